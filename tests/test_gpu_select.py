"""Selection of the top-B keys: heads up to 4096 keys go to one block, longer ones to a histogram over a
bracket taken from 128 sampled keys, with a list of at most 4096 candidates and, in LDS, comparison of at
most 256.  Lengths and budgets sit at those edges.  With lambda = 1 and no pooling the score is the
importance itself, so the cases can put the wanted key where they like: inside the bracket, below or
above it (the sampled positions hold the other values), among ties.  Whole
numbers: exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import binding as B
from paper_2602_10825_amd import synth
from tests.test_gpu_parity import DEV, dev

pytestmark = pytest.mark.gpu


def sampled(L):
    q = np.arange(128, dtype=np.uint64)
    jitter = ((q * 2654435761) & 0xFFFFFFFF) >> 12
    return (q * L // 128 + jitter % (L // 128)).astype(np.int64)


def importance(kind, L, rng):
    if kind == "even":
        return rng.random(L)
    if kind == "skewed":
        return np.exp(12.0 * rng.standard_normal(L))
    if kind == "plateaus":                  # eleven values
        return rng.integers(0, 11, L) / 11.0
    if kind == "equal":
        return np.full(L, 0.25)
    if kind == "signed":                    # a bracket with zero inside
        return rng.standard_normal(L)
    m = rng.random(L)
    m[sampled(L)] = (2.0 if kind == "below" else -2.0) + rng.random(128)
    return m


@pytest.mark.parametrize("kind,L,budget", [
    ("even", 2, 1), ("even", 257, 256), ("even", 1312, 984), ("even", 4096, 4095), ("even", 4096, 1),
    ("skewed", 4095, 2000), ("plateaus", 4096, 1234), ("equal", 3000, 77),
    ("even", 4097, 4096), ("even", 4097, 1), ("skewed", 20001, 15000), ("skewed", 50000, 100),
    ("plateaus", 20000, 9000), ("plateaus", 4100, 300), ("equal", 20000, 12345),
    ("below", 20001, 10000), ("above", 20001, 10000),     # more candidates outside than the list holds
    ("below", 4200, 4150), ("above", 4200, 40),           # few enough for it
    ("signed", 50000, 20000), ("signed", 50000, 24000), ("signed", 50000, 25000),
])
def test_selection_by_importance_alone(kind, L, budget):
    rng = np.random.default_rng(L + budget)
    k = synth.to_storage(rng.standard_normal((2, L, 64)).astype(np.float32), "bf16")
    mass = np.stack([importance(kind, L, rng) for _ in range(2)]).astype(np.float32)
    kept = B.flowcache_kv_select(dev(k, "bf16"), L, budget, torch.from_numpy(mass).to(DEV), 1, 1.0)
    ref = np.stack([O.select_top_b(m.astype(np.float64), budget) for m in mass])
    assert np.array_equal(kept.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype,d,L,budget,pool_k", [
    ("bf16", 128, 4096, 3000, 7), ("bf16", 128, 4097, 3000, 7), ("f32", 64, 700, 350, 9), ("f32", 128, 9000, 4500, 3),
    ("bf16", 64, 5000, 2500, 141), ("bf16", 64, 5000, 2500, 385), ("f32", 64, 4200, 900, 257),
    ("bf16", 64, 5000, 2500, 387),        # a window wider than what LDS holds beside a block's tokens
    ("bf16", 64, 129, 128, 7), ("bf16", 64, 700, 385, 7), ("bf16", 64, 9001, 8000, 7),   # tiles of 128 rows
])
def test_selection_with_redundancy(dtype, d, L, budget, pool_k):
    rng = np.random.default_rng(L)
    k = synth.to_storage(rng.standard_normal((2, L, d)).astype(np.float32), dtype)
    v = synth.to_storage(rng.standard_normal((2, L, d)).astype(np.float32), dtype)
    mass = (rng.exponential(size=(2, L)) ** 2).astype(np.float32)
    mass /= mass.sum(1, keepdims=True)
    kc, vc = dev(k, dtype), dev(v, dtype)
    kept = B.flowcache_kv_compress(kc, vc, L, budget, torch.from_numpy(mass).to(DEV), pool_k, 0.07)
    rk, rk_k, rk_v, _ = O.kv_compress(k, v, L, budget, mass, pool_k, 0.07)
    assert np.array_equal(kept.cpu().numpy(), rk)
    assert np.array_equal(B.to_host(kc), rk_k) and np.array_equal(B.to_host(vc), rk_v)


@pytest.mark.parametrize("L,budget,lam", [(51000, 25500, 0.2), (51000, 25500, 0.3), (51000, 40800, 0.5),
                                          (51000, 40800, 0.7), (20001, 16000, 0.7)])
def test_selection_with_scores_of_both_signs(L, budget, lam):
    """The wanted score close to zero, where importance and redundancy balance."""
    rng = np.random.default_rng(5)
    k = synth.to_storage(rng.standard_normal((2, L, 64)).astype(np.float32), "bf16")
    mass = (rng.exponential(size=(2, L)) ** 2).astype(np.float32)
    mass /= mass.sum(1, keepdims=True)
    ref = np.stack([O.select_top_b(O.selection_scores(O.widen(k[h]), mass[h], 7, lam), budget) for h in range(2)])
    for _ in range(3):
        kept = B.flowcache_kv_select(dev(k, "bf16"), L, budget, torch.from_numpy(mass).to(DEV), 7, lam)
        assert np.array_equal(kept.cpu().numpy(), ref)


@pytest.mark.parametrize("H,d,L,budget", [(1, 64, 200, 100),          # one tile: the second ticket is past the end
                                          (8, 128, 5000, 4096),       # 512 tiles: one ticket per block
                                          (9, 128, 4200, 4096),       # 576: some blocks draw a second tile
                                          (3, 64, 40000, 39000),      # 915 of 128 rows, nearly all of them waiting
                                          (10, 128, 17000, 16384),    # 2560: five per block, rows requested early
                                          (24, 64, 16000, 13500),     # 2544: not
                                          (4, 128, 12000, 10240)])    # 160 per head: early again
def test_compaction_draws_every_tile_once(H, d, L, budget):
    """All wavefronts of a block work on the block's first ticket, whatever the second one is."""
    g = torch.Generator(device=DEV).manual_seed(L)
    k0, v0 = (torch.randn((H, L + 64, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
    kept = torch.stack([torch.randperm(L, generator=g, device=DEV)[:budget].sort().values for _ in range(H)]).int()
    rows = kept.long()[..., None].expand(H, budget, d)
    for _ in range(10):
        k, v = k0.clone(), v0.clone()
        B.flowcache_kv_compact(k, v, L, budget, kept, check_status=True)
        for x, x0 in ((k, k0), (v, v0)):
            assert torch.equal(x[:, :budget], x0.gather(1, rows)) and torch.equal(x[:, budget:], x0[:, budget:])


@pytest.mark.parametrize("kind,L,budget", [
    ("256", 1500, 100), ("257", 1500, 100), ("256", 4096, 256), ("257", 4096, 258), ("256", 300, 257), ("outlier", 2000, 700),
    ("outlier", 2000, 1), ("signed", 1312, 984), ("signed", 4096, 2000), ("signed", 257, 128), ("tiny", 1000, 400),
])
def test_first_cut_of_short_heads(kind, L, budget):
    """Heads of at most 4096 keys are cut into 2048 bins of equal width in the score first; what the wanted bin
    holds is compared with each other up to 256 keys, and otherwise the digits of the keys decide: a bin of exactly
    256 and 257 nearly equal scores, one outlier that leaves all others in one bin, scores of both signs, and
    subnormal scores."""
    rng = np.random.default_rng(L + budget)
    m = rng.random((2, L)).astype(np.float32)
    if kind in ("256", "257"):                # bins of 0.49: the n scores at 1.5 have one to themselves
        n = min(int(kind), L - 2)
        m[:, :n] = np.float32(1.5) + rng.permutation(n).astype(np.float32) * np.float32(2.0 ** -22)
        m[:, n] = 1000.0
        m = np.take_along_axis(m, rng.permuted(np.tile(np.arange(L), (2, 1)), axis=1), 1)
    elif kind == "outlier":
        m[:, 77] = 1e30
    elif kind == "signed":
        m = rng.standard_normal((2, L)).astype(np.float32)
    else:
        m *= np.float32(1e-41)
    k = synth.to_storage(rng.standard_normal((2, L, 64)).astype(np.float32), "bf16")
    kept = B.flowcache_kv_select(dev(k, "bf16"), L, budget, torch.from_numpy(m).to(DEV), 1, 1.0)
    assert np.array_equal(kept.cpu().numpy(), np.stack([O.select_top_b(x.astype(np.float64), budget) for x in m]))
