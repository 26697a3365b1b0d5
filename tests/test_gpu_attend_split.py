"""The attention kernels that divide a block's keys over its wavefronts and, where a launch has few
query rows, over several blocks: row tiles of 32, key tiles of 32, key ranges per block.  The sizes
sit at the edges of those (one row, one key, a tile more or less, fewer tiles than wavefronts,
ranges that split inside a segment), against the float64 oracle at the bars of the parity tests."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import binding as B
from paper_2602_10825_amd import synth
from tests.test_attend_plan import driver  # noqa: F401  (fixture: the launch plan, compiled for the CPU)
from tests.test_gpu_parity import DEV, check_attend, dev, run_attend

pytestmark = pytest.mark.gpu

# (H_q, H_k, d, A, L_c, L_clean, recompute list)
SHAPES = [
    (1, 1, 64, 1, 1, 0, [0]),                 # one row, one key
    (2, 1, 128, 2, 31, 1, [0, 1]),            # a tile less one
    (2, 2, 128, 1, 33, 31, [0]),              # a tile and one; ragged end of both segments
    (1, 1, 128, 3, 32, 255, [2]),             # exactly one row tile, eight key tiles in the clean region
    (4, 2, 64, 2, 65, 1025, [1]),             # two ranges and more
    (1, 1, 128, 2, 5, 9000, [0, 1]),          # few rows, long context: the most ranges
    (3, 1, 64, 16, 40, 700, [0, 3, 15]),      # ranges over many segments
    (8, 8, 128, 4, 321, 64, [0, 1, 2, 3]),    # enough rows that fp32 splits nothing over blocks
    (12, 12, 64, 2, 513, 3000, [0, 1]),       # 256-row units, all of them split (bf16)
    (24, 24, 64, 2, 1400, 700, [0, 1]),       # more 256-row units than compute units: the last round split
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H_q,H_k,d,A,L_c,L_clean,rec", SHAPES)
def test_attend_split_edges(dtype, H_q, H_k, d, A, L_c, L_clean, rec):
    wl = synth.Workload("split", dtype, H_q, H_k, d, A, L_c, L_clean, 1)
    a = synth.attend_inputs(wl, seed=L_c)
    got, ref, res, ref_lse, *_ = run_attend(wl, a, rec)
    check_attend(wl, got, ref, res, ref_lse, len(rec))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attend_without_room_for_partials(dtype):
    """A workspace too small for the partials, or not aligned for them, leaves the keys of a unit in one
    block."""
    wl = synth.Workload("split", dtype, 2, 2, 64, 2, 48, 4000, 1)
    a = synth.attend_inputs(wl, seed=3)
    idx = torch.tensor([1, -1], dtype=torch.int32, device=DEV)
    n = torch.tensor([1], dtype=torch.int32, device=DEV)
    q, k, v = dev(a["q"], dtype), dev(a["k_cache"], dtype), dev(a["v_cache"], dtype)
    need = B.lib().flowcache_attend_workspace(wl.A, wl.L_c, wl.H_q, wl.H_k, wl.d, 0, 50)
    outs = []
    for ws in (torch.empty(need, dtype=torch.uint8, device=DEV), torch.empty(256, dtype=torch.uint8, device=DEV),
               torch.empty(need + 8, dtype=torch.uint8, device=DEV)[8:], torch.empty(need + 1, dtype=torch.uint8, device=DEV)[1:]):
        r = B.flowcache_attend(q, None, None, k, v, wl.L_c, wl.L_clean, a["active_off"], idx, n, workspace=ws)
        outs.append((r["out"][:wl.L_c].float().cpu().numpy(), r["lse"][:, :wl.L_c].cpu().numpy()))
    # the same products summed in another grouping: fp32 sums of at most 4096 terms, and for bf16 one
    # rounding of weights and outputs each
    tol = 1e-5 if dtype == "f32" else 1e-2
    for x, y in zip(outs[0], outs[1]):
        assert np.linalg.norm(x - y) <= tol * np.linalg.norm(y)
    for other in outs[2:]:
        assert all(np.array_equal(x, y) for x, y in zip(other, outs[1]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_importance_needs_no_room_for_partials(dtype):
    """With mass the workspace has to hold what the importance needs and no more: one sized for other
    lengths (shorter chunks may ask for more partials) is not refused."""
    wl = synth.Workload("split", dtype, 2, 2, 64, 2, 48, 4000, 1)
    a = synth.attend_inputs(wl, seed=4)
    idx = torch.tensor([0, 1], dtype=torch.int32, device=DEV)
    n = torch.tensor([2], dtype=torch.int32, device=DEV)
    q, k, v = dev(a["q"], dtype), dev(a["k_cache"], dtype), dev(a["v_cache"], dtype)
    L = B.lib()
    least = 256 + L.flowcache_attention_mass_workspace(40, wl.H_q, wl.H_k, wl.d, 4000)
    full = L.flowcache_attend_workspace(wl.A, wl.L_c, wl.H_q, wl.H_k, wl.d, 4000, 40)
    assert least < full
    outs = []
    for nbytes in (full, least):
        ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        r = B.flowcache_attend(q, None, None, k, v, wl.L_c, wl.L_clean, a["active_off"], idx, n, mass_len=4000,
                               obs_window=40, workspace=ws)
        outs.append((r["out"].float().cpu().numpy(), r["mass"].cpu().numpy()))
    assert np.array_equal(outs[0][1], outs[1][1])
    tol = 1e-5 if dtype == "f32" else 1e-2        # as above
    assert np.linalg.norm(outs[0][0] - outs[1][0]) <= tol * np.linalg.norm(outs[0][0])
    with pytest.raises(B.FlowCacheError):
        B.flowcache_attend(q, None, None, k, v, wl.L_c, wl.L_clean, a["active_off"], idx, n, mass_len=4000,
                           obs_window=40, workspace=torch.empty(least - 1, dtype=torch.uint8, device=DEV))


NARROW, WHOLE, ALL_SPLIT, LAST_SPLIT = range(4)


@pytest.mark.parametrize("H_q,H_k,d,A,L_c,L_clean,form", [
    (4, 2, 128, 3, 328, 1000, NARROW), (2, 2, 64, 2, 70, 3000, NARROW),
    (24, 24, 128, 3, 450, 601, WHOLE), (24, 4, 64, 4, 330, 333, WHOLE),
    (12, 12, 64, 2, 513, 3000, ALL_SPLIT), (12, 3, 128, 2, 600, 3001, ALL_SPLIT),
    (24, 24, 64, 2, 1400, 700, LAST_SPLIT), (24, 6, 128, 2, 1300, 701, LAST_SPLIT),
])
def test_every_form_when_later_keys_dwarf_earlier_ones(driver, H_q, H_k, d, A, L_c, L_clean, form):
    """Scores that grow along the keys by far more than 2^40, in the clean region and again in the active
    chunks, so that the exponents' reference is raised in the middle of a run, in every form of the bf16
    launch; the slots lie in reverse order, so every segment ends in its own ragged tile.  The plan is
    asked for the form, so that a change of its costs cannot take a case elsewhere unseen."""
    assert ctypes.CDLL(driver).form(A, L_c, L_clean, H_q, d, A) == form
    wl = synth.Workload("grow", "bf16", H_q, H_k, d, A, L_c, L_clean, 1)
    a = synth.attend_inputs(wl, seed=L_c)
    a["active_off"] = a["active_off"][::-1]
    ramp = np.linspace(0.05, 30.0, wl.capacity)[None, :, None]
    a["k_cache"] = synth.to_storage((O.widen(a["k_cache"]) * ramp).astype(np.float32), "bf16")
    grow = np.linspace(20.0, 60.0, A * L_c)[:, None, None]
    a["k_new"] = synth.to_storage((O.widen(a["k_new"]) * grow).astype(np.float32), "bf16")
    got, ref, res, ref_lse, *_ = run_attend(wl, a, list(range(A)))
    err = np.abs(got - ref)                      # outputs are O(1), a few keys dominate each row: relative bars
    assert np.sqrt((err ** 2).sum()) / np.sqrt((ref ** 2).sum()) <= 1e-2
    assert err.max() <= 2e-2 * max(1.0, np.abs(ref).max())
    assert np.abs(res["lse"].cpu().numpy()[:, :A * L_c] - ref_lse).max() <= 2e-2 * np.abs(ref_lse).max()


@pytest.mark.parametrize("H_q,H_k,d,A,L_c,L_clean", [
    (2, 1, 64, 2, 40, 300), (2, 2, 128, 1, 33, 1000), (4, 4, 128, 2, 300, 2100), (6, 3, 64, 2, 400, 1500)])
def test_f32_operands_of_any_magnitude(H_q, H_k, d, A, L_c, L_clean):
    """fp32 operands are split into two f16 parts after scaling by powers of two: per query row, per key, and for V by
    the largest entry so far, which here grows along the keys (its scale is raised again and again), with rows of
    zeros, a first tile of zeros and subnormal entries.  Each entry is held to 2^-23 and a few thousand terms are
    added up: the parity bars, per row."""
    wl = synth.Workload("magnitude", "f32", H_q, H_k, d, A, L_c, L_clean, 1)
    a = synth.attend_inputs(wl, seed=7)
    rng = np.random.default_rng(5)
    rows = lambda n, lo, hi: (10.0 ** rng.uniform(lo, hi, n)).astype(np.float32)
    a["q"] *= rows(a["q"].shape[0], -4, 0.3)[:, None, None]
    a["k_cache"] *= rows(wl.capacity, -6, 0.1)[None, :, None]
    a["k_cache"][:, 5::7] = 0
    a["v_cache"] *= np.logspace(-12, 9, wl.capacity, dtype=np.float32)[None, :, None]
    a["v_cache"][:, :40] = 0
    a["v_cache"][:, 50:60] = 1e-41
    a["v_new"] *= rows(A * L_c, -3, 10)[:, None, None]
    a["q"][3] = 0
    got, ref, res, ref_lse, *_ = run_attend(wl, a, list(range(A)))
    check_attend(wl, got, ref, res, ref_lse, A)
