"""fp32 attention in blocks of 256 rows whose wavefronts share every key tile, in every form of the launch: a ragged last
block of rows, one row past a block, one key more or less than a tile in every segment, slots in reverse order, grouped
heads, split blocks that do not divide evenly among the XCDs, a launch that runs 32-row blocks for other recompute counts, values that grow along the keys; against the float64
oracle at the parity bars."""
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
extern "C" __attribute__((visibility("default"))) int form(int A, int L_c, int L_clean, int H_q, int d, int R) {
    const FcAttendPlan p = fc_attend_plan_f32(A, L_c, L_clean, H_q, true, d);
    if (p.narrow[R - 1]) return 0;
    const int S = p.splits[R - 1];
    return S == 1 ? 1 : fc_wide_shape(R, H_q * ((L_c + kWideRows - 1) / kWideRows), S).full == 0 ? 2 : 3;
}
"""
NARROW, WHOLE, ALL_SPLIT, LAST_SPLIT = range(4)
# (H_q, H_k, d, A, L_c, L_clean, recompute list), form
FORMS = [
    ((24, 24, 64, 2, 256, 640, [0, 1]), ALL_SPLIT), ((12, 12, 128, 4, 385, 1025, [0, 1, 2, 3]), ALL_SPLIT),
    ((24, 6, 128, 2, 383, 639, [1]), ALL_SPLIT), ((12, 12, 128, 4, 385, 1025, [0, 2, 3]), NARROW),
    ((24, 12, 128, 2, 511, 95, [0, 1]), ALL_SPLIT), ((96, 96, 64, 1, 257, 129, [0]), WHOLE),
    ((24, 4, 64, 4, 330, 333, [0, 1, 2, 3]), WHOLE), ((48, 12, 64, 2, 600, 40, [0, 1]), LAST_SPLIT),
    ((64, 8, 64, 2, 520, 100, [0, 1]), LAST_SPLIT),
    ((3, 1, 128, 3, 900, 5000, [0, 1, 2]), ALL_SPLIT), ((1, 1, 128, 3, 1500, 2500, [0, 1, 2]), ALL_SPLIT),
    ((48, 48, 64, 2, 128, 1600, [0, 1]), NARROW), ((24, 24, 64, 3, 384, 1, [0, 1, 2]), NARROW),
]
SHAPES = [shape for shape, _ in FORMS]


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.hip", d / "plan.so"
    src.write_text(DRIVER)
    subprocess.run([build.HIPCC, "--offload-host-only", *build.FLAGS, "-shared", str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so)).form


def test_the_shapes_are_run_in_these_forms(form):
    """Asked of the plan, so that a change of its costs cannot take the cases below elsewhere unseen."""
    for (H_q, _, d, A, L_c, L_clean, rec), want in FORMS:
        assert form(A, L_c, L_clean, H_q, d, len(rec)) == want, (H_q, A, L_c, L_clean)


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
    """An infinity has no parts, so its wavefronts form their sums with fp32 products: its column is infinite, the others
    are those of the call with a zero in its place, up to the rounding of the other products."""
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
    assert (got[:, :group, 5] == bad).all()
    got[:, :group, 5] = zero[:, :group, 5]
    assert np.isfinite(zero).all() and np.abs(got - zero).max() <= 1e-5 * np.abs(zero).max()


@pytest.mark.gpu
def test_workspaces_too_small_for_the_partials():
    """Less room than the plan's partials take: the keys stay undivided.  The same products in another grouping, sums of
    at most 4096 terms: 1e-5 of the norm."""
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


@pytest.mark.gpu
@pytest.mark.parametrize("H_q,H_k,d,A", [(96, 8, 64, 1), (48, 4, 128, 2)])
def test_long_ranges_add_up_as_many_tiles(form, H_q, H_k, d, A):
    """More units than compute units on a long cache: a wavefront adds up 1272 tiles or more.  O is rounded once per tile, by
    2^-24 at most, and a random walk of that ends below 2^-24 sqrt(1300 / 3) = 1.25e-6 of the sum (earlier sums are
    smaller); scores and exponentials are off by some 2^-23 each, 3e-7 of a sum of many."""
    L_c, L_clean = 700, 40000
    assert form(A, L_c, L_clean, H_q, d, A) == LAST_SPLIT
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d)
    n = L_clean + A * L_c
    q, k, v = (torch.randn(s, generator=gen, device=DEV) for s in ((A * L_c, H_q, d), (H_k, n, d), (H_k, n, d)))
    idx, count = torch.arange(A, dtype=torch.int32, device=DEV), torch.tensor([A], dtype=torch.int32, device=DEV)
    out = B.flowcache_attend(q, None, None, k, v, L_c, L_clean, [L_clean + i * L_c for i in range(A)], idx, count)["out"]
    for h in (0, H_q // 2 - 1, H_q - 1):
        hk = h // (H_q // H_k)
        for c in range(A):
            seen = L_clean + (c + 1) * L_c
            s = q[c * L_c:(c + 1) * L_c, h].double() @ k[hk, :seen].double().T * d ** -0.5
            ref = torch.softmax(s, -1) @ v[hk, :seen].double()
            err = (out[c * L_c:(c + 1) * L_c, h].double() - ref).norm() / ref.norm()
            assert float(err) <= 1.5e-6, (h, c, float(err))
