"""fp32 attention in blocks of 128 rows whose wavefronts share every key tile: a ragged last block of rows, one row
past it, one key more or less than a tile in every segment, slots in reverse order, grouped heads, the fewest
ranges, V's largest entries growing along the keys (the block's scale is raised while tiles wait in the buffers);
against the float64 oracle at the parity bars."""
import ctypes
import subprocess

import numpy as np
import pytest
import torch

from paper_2602_10825_amd import binding as B
from paper_2602_10825_amd import build, synth
from tests.test_gpu_parity import DEV, check_attend, dev, run_attend

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


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [np.inf, -np.inf])
@pytest.mark.parametrize("H_q,H_k,d,A,L_c,L_clean,rec", [SHAPES[4], (2, 1, 64, 2, 40, 300, [0, 1]), (4, 4, 128, 1, 33, 70, [0])])
def test_an_infinite_value_spoils_its_own_column(H_q, H_k, d, A, L_c, L_clean, rec, bad):
    """Both forms scale V by its largest entry: an infinity must not reach the other columns through the
    scale.  They are then the bits of the call with a zero in its place."""
    wl = synth.Workload("shared", "f32", H_q, H_k, d, A, L_c, L_clean, 1)
    a = synth.attend_inputs(wl, seed=9)
    a["v_cache"] = a["v_cache"].copy()
    outs = []
    for value in (0.0, bad):
        a["v_cache"][0, L_clean // 2, 5] = value
        with np.errstate(invalid="ignore"):
            outs.append(run_attend(wl, a, rec)[0])
    zero, got = (o.reshape(-1, H_q, d) for o in outs)
    group = H_q // H_k
    assert not np.isfinite(got[:, :group, 5]).any()
    got[:, :group, 5] = zero[:, :group, 5]
    assert np.isfinite(zero).all() and np.array_equal(got, zero)


@pytest.mark.gpu
def test_workspaces_too_small_for_shared_tiles():
    """Less room than the query asks for: 32-row blocks with their keys split where that fits, undivided below.  The
    same products in another grouping, sums of at most 4096 terms: 1e-5 of the norm."""
    H_q, H_k, d, A, L_c, L_clean, rec = SHAPES[1]
    wl = synth.Workload("shared", "f32", H_q, H_k, d, A, L_c, L_clean, 1)
    a = synth.attend_inputs(wl, seed=2)
    idx = torch.arange(A, dtype=torch.int32, device=DEV)
    n = torch.tensor([A], dtype=torch.int32, device=DEV)
    q, k, v = dev(a["q"], "f32"), dev(a["k_cache"], "f32"), dev(a["v_cache"], "f32")
    need = B.lib().flowcache_attend_workspace(A, L_c, H_q, H_k, d, 0, 50)
    outs = []
    for size in (need, need - 256, need // 3, need // 8, 256):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        r = B.flowcache_attend(q, None, None, k, v, L_c, L_clean, a["active_off"], idx, n, workspace=ws)
        outs.append(r["out"].cpu().numpy())
    for o in outs[1:]:
        assert np.linalg.norm(o - outs[0]) <= 1e-5 * np.linalg.norm(outs[0])
