"""fp32 attention in blocks of 128 rows whose wavefronts share every key tile: a ragged last block of rows, one row
past it, one key more or less than a tile in every segment, slots in reverse order, grouped heads, the fewest
ranges, V's largest entries growing along the keys (the block's scale is raised while tiles wait in the buffers);
against the float64 oracle at the parity bars."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2602_10825_amd import build, synth
from tests.test_gpu_parity import check_attend, run_attend

DRIVER = r"""
#include "attend_split.hpp"
extern "C" __attribute__((visibility("default"))) int shared(int A, int L_c, int L_clean, int H_q, int R) {
    const FcAttendPlan p = fc_attend_plan_f32(A, L_c, L_clean, H_q, true);
    return p.narrow[R - 1] ? 0 : p.splits[R - 1];
}
"""
# (H_q, H_k, d, A, L_c, L_clean, recompute list)
SHAPES = [
    (48, 48, 64, 2, 128, 1600, [0, 1]), (12, 12, 128, 4, 385, 1025, [0, 2, 3]), (24, 6, 128, 2, 383, 639, [1]),
    (24, 24, 64, 3, 384, 1, [0, 1, 2]), (24, 12, 128, 2, 511, 95, [0, 1]),
]


@pytest.fixture(scope="module")
def shared(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.hip", d / "plan.so"
    src.write_text(DRIVER)
    subprocess.run([build.HIPCC, "--offload-host-only", *build.FLAGS, "-shared", str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).shared


def test_the_shapes_are_run_by_blocks_that_share_their_tiles(shared):
    """Asked of the plan, so that a change of its costs cannot take the cases below elsewhere unseen; every range count
    is at least three (the bound on what one accumulator adds up)."""
    for H_q, _, _, A, L_c, L_clean, rec in SHAPES:
        assert shared(A, L_c, L_clean, H_q, len(rec)) >= 3, (H_q, A, L_c, L_clean)


@pytest.mark.gpu
@pytest.mark.parametrize("grow", [False, True])
@pytest.mark.parametrize("H_q,H_k,d,A,L_c,L_clean,rec", SHAPES)
def test_shared_tiles(H_q, H_k, d, A, L_c, L_clean, rec, grow):
    wl = synth.Workload("shared", "f32", H_q, H_k, d, A, L_c, L_clean, 1)
    a = synth.attend_inputs(wl, seed=L_c)
    a["active_off"] = a["active_off"][::-1]
    if grow:
        rng = np.random.default_rng(L_c)
        a["v_cache"] *= np.logspace(-9, 6, wl.capacity, dtype=np.float32)[None, :, None]
        a["v_cache"][:, :70] = 0
        a["v_new"] *= (10.0 ** rng.uniform(-3, 8, A * L_c)).astype(np.float32)[:, None, None]
        a["k_cache"] *= (10.0 ** rng.uniform(-6, 0.1, wl.capacity)).astype(np.float32)[None, :, None]
        a["q"] *= (10.0 ** rng.uniform(-4, 0.2, a["q"].shape[0])).astype(np.float32)[:, None, None]
    got, ref, res, ref_lse, *_ = run_attend(wl, a, rec)
    check_attend(wl, got, ref, res, ref_lse, len(rec))
