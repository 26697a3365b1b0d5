"""First digit of the selection (select_bins.hpp), compiled for the CPU: no GPU needed."""
import ctypes
import subprocess

import numpy as np
import pytest

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import build

DRIVER = r"""
#include "select_bins.hpp"
extern "C" {
#pragma GCC visibility push(default)
int edges(const uint64_t* sample, int budget, int L, uint64_t* edge) {   // sample: descending
    const FcBracket b = fc_bracket(budget, L);
    for (int i = 0; i < kEdges; ++i) edge[i] = ~0ull;
    for (int r = b.top; r <= b.bottom; ++r) edge[b.bottom - r] = sample[r];
    return b.bottom - b.top;
}
int even_shift(const uint64_t* edge, int n) {
    const int sh = fc_even_shift(edge, n);
    for (int i = 0; i < 64; ++i)
        if (fc_crowded(edge, n, sh, i)) return -1;
    return sh;
}
void digits(const uint64_t* k, int m, const uint64_t* edge, int n, int sh, uint32_t* out) {
    for (int i = 0; i < m; ++i) out[i] = fc_first_digit(k[i], edge, n, sh);
}
void bin_keys(uint32_t bin, const uint64_t* edge, int n, int sh, uint64_t* range) {
    fc_bin_keys(bin, edge, n, sh, range, range + 1);
}
}
"""


@pytest.fixture(scope="module")
def bins(tmp_path_factory):
    d = tmp_path_factory.mktemp("bins")
    src, so = d / "bins.hip", d / "bins.so"
    src.write_text(DRIVER)
    subprocess.run([build.HIPCC, "--offload-host-only", *build.FLAGS, "-shared", str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def ptr(a):
    return ctypes.c_void_p(a.ctypes.data)


def keys_of(score):
    b = (np.asarray(score, dtype=np.float64) + 0.0).view(np.uint64)
    return np.where(b >> np.uint64(63), ~b, b | np.uint64(1 << 63))


def sampled(L):
    q = np.arange(128, dtype=np.uint64)
    return (q * L // 128 + (((q * 2654435761) & 0xFFFFFFFF) >> 12) % (L // 128)).astype(np.int64)


def first_digit(bins, key, budget, sample):
    edge, down = np.empty(64, dtype=np.uint64), np.ascontiguousarray(np.sort(sample)[::-1])
    n = bins.edges(ptr(down), budget, len(key), ptr(edge))
    sh = bins.even_shift(ptr(edge), n)
    key, out = np.ascontiguousarray(key), np.empty(len(key), dtype=np.uint32)
    bins.digits(ptr(key), len(key), ptr(edge), n, sh, ptr(out))
    return out, edge, n, sh


@pytest.mark.parametrize("kind", ["normal", "exponents", "plateaus", "equal", "bits", "ends", "narrow"])
@pytest.mark.parametrize("L,budget", [(4097, 1), (4097, 4096), (9000, 4500), (20001, 300), (20001, 19000)])
def test_digits_ascend_with_the_keys_and_bins_are_ranges(bins, kind, L, budget):
    rng = np.random.default_rng(L + budget)
    if kind == "bits":
        key = rng.integers(0, 1 << 64, L, dtype=np.uint64)
    elif kind == "ends":                    # the lowest and highest keys there are
        key = rng.choice(np.array([0, 1, (1 << 64) - 2, (1 << 64) - 1, 1 << 63], dtype=np.uint64), L)
    else:
        key = keys_of({"normal": rng.standard_normal(L), "plateaus": rng.integers(-3, 4, L) / 7.0, "narrow": 1.0 + rng.random(L),
                        "equal": np.full(L, -0.5),
                       "exponents": np.sign(rng.standard_normal(L)) * np.exp(100 * rng.standard_normal(L))}[kind])
    dgt, edge, n, sh = first_digit(bins, key, budget, key[sampled(L)])
    order = np.argsort(key, kind="stable")
    assert 28 <= n <= 56 and dgt.max() < 512
    assert np.all(np.diff(dgt[order].astype(np.int64)) >= 0)
    assert np.all((dgt == 0) == (key < edge[0])) and np.all((dgt == 511) == (key > edge[n]))
    rang = np.empty(2, dtype=np.uint64)
    for b in np.unique(dgt):
        bins.bin_keys(int(b), ptr(edge), n, sh, ptr(rang))
        with np.errstate(over="ignore"):
            assert np.array_equal(key - rang[0] <= rang[1], dgt == b), int(b)


@pytest.mark.parametrize("lam", [0.0, 0.07, 0.2, 0.3, 0.5, 0.7, 1.0])
def test_few_keys_share_the_wanted_digit(bins, lam):
    """At every weight of the importance, also where scores of both signs surround the wanted one, the
    keys that the select looks at again fit its list of 4096; bins of equal width over the whole bracket put up
    to 20000 of them into one."""
    rng = np.random.default_rng(5)
    L = 51000
    red = O.redundancy(rng.standard_normal((L, 64)).astype(np.float32))
    both = set()
    for imp in (rng.exponential(size=L) ** 2, np.exp(3 * rng.standard_normal(L)),
                np.where(rng.random(L) < 0.02, 1.0, 1e-9) * rng.random(L)):
        imp = (imp / imp.sum()).astype(np.float32).astype(np.float64)
        for pool in (1, 7):
            score = lam * O.maxpool1d(imp, pool) - (1.0 - lam) * red
            for budget in (5000, 25500, 40800, 48000):
                key = keys_of(score)
                dgt, _, _, sh = first_digit(bins, key, budget, key[sampled(L)])
                wanted = dgt[np.argsort(key)[L - budget]]
                both.add(sh < 0)
                assert (dgt == wanted).sum() <= max(4096, (score == np.sort(score)[L - budget]).sum())
    assert False in both and (True in both or lam == 0.0)     # equal widths, and bins that follow the sample
