"""fp32 attention and importance over the range of a float.  An fp32 product keeps every operand's 24 bits whatever its
neighbours are, so each entry of an output may be off by no more than the parity bar (1e-5) times the sum of the
magnitudes that it is made of: one value column, or one key without weight, far larger than the rest; a key that takes
nearly all the weight and has no value; channels in which queries are tiny and keys huge; entries close to the
largest float; an infinite entry.  Both forms of the attention launch."""
import numpy as np
import pytest
import torch

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import binding as B
from tests.test_gpu_parity import DEV, dev

pytestmark = pytest.mark.gpu

# (H_q, H_k, d, A, L_c, L_clean): 32-row blocks, then blocks of rows that share their key tiles
SHAPES = [(2, 1, 64, 2, 40, 300), (4, 4, 128, 1, 33, 70), (24, 12, 128, 2, 511, 95), (24, 24, 64, 2, 256, 640)]
BAR = 1e-5


def inputs(H_q, H_k, d, A, L_c, L_clean, seed=3):
    rng = np.random.default_rng(seed)
    n = L_clean + A * L_c
    normal = lambda *s: rng.standard_normal(s).astype(np.float32)
    return normal(A * L_c, H_q, d), normal(H_k, n, d), normal(H_k, n, d)


def attend(q, k, v, A, L_c, L_clean):
    off = [L_clean + i * L_c for i in range(A)]
    idx, n = torch.arange(A, dtype=torch.int32, device=DEV), torch.tensor([A], dtype=torch.int32, device=DEV)
    r = B.flowcache_attend(dev(q, "f32"), None, None, dev(k, "f32"), dev(v, "f32"), L_c, L_clean, off, idx, n)
    return r["out"].cpu().numpy().astype(np.float64), r["lse"].cpu().numpy()


def check(shape, q, k, v, k_ref=None, factor=1.0):
    """Every entry against float64, relative to the sum of its terms' magnitudes."""
    H_q, H_k, d, A, L_c, L_clean = shape
    off, rec = [L_clean + i * L_c for i in range(A)], list(range(A))
    k_ref = k if k_ref is None else k_ref
    ref, ref_lse = O.attend(q, k_ref, v, L_clean, off, L_c, rec)
    size, _ = O.attend(q, k_ref, np.abs(v), L_clean, off, L_c, rec)
    got, lse = attend(q, k, v, A, L_c, L_clean)
    worst = np.abs(got - ref) / np.where(size > 0, size, 1.0)
    assert worst.max() <= factor * BAR, worst.max()       # (a NaN fails too)
    assert np.abs(lse - ref_lse).max() <= factor * BAR * max(1.0, np.abs(ref_lse).max())


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("power", [20, 24, 40, 100, -100, -118])
def test_a_value_column_of_another_magnitude(shape, power):
    q, k, v = inputs(*shape)
    v[:, :, 5] *= np.float32(2.0 ** power)
    check(shape, q, k, v)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("power", [24, 60])
def test_a_huge_value_without_weight(shape, power):
    """One key scores about 200 below the others in every row: 2^60 times its weight is nothing."""
    H_q, H_k, d, A, L_c, L_clean = shape
    q, k, v = inputs(*shape)
    q[:, :, 0] = 8.0
    k[:, :, 0] = 0.0
    for key in (2, L_clean // 2):
        k[:, key, 0] = -200.0 * np.sqrt(d) / 8.0
        v[:, key] *= np.float32(2.0 ** power)
    check(shape, q, k, v)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bits", [20, 30])
def test_a_key_that_takes_the_weight_and_has_no_value(shape, bits):
    H_q, H_k, d, A, L_c, L_clean = shape
    q, k, v = inputs(*shape)
    q[:, :, 0] = 8.0
    k[:, :, 0] = 0.0
    k[:, 1, 0] = bits * np.log(2.0) * np.sqrt(d) / 8.0
    v[:, 1] = 0.0
    check(shape, q, k, v)


@pytest.mark.parametrize("shape", SHAPES)
def test_channels_of_opposite_magnitude(shape):
    """Half of the channels carry keys of 2^30 and queries of 2^-30: scores are O(1), and each product counts."""
    q, k, v = inputs(*shape)
    half = shape[2] // 2
    q[:, :, :half] *= np.float32(2.0 ** -30)
    k[:, :, :half] *= np.float32(2.0 ** 30)
    check(shape, q, k, v)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("power", [100, 120, -100, -120])
def test_keys_of_another_magnitude_than_the_queries(shape, power):
    q, k, v = inputs(*shape)
    check(shape, (q * np.float32(2.0 ** -power)).astype(np.float32), (k * np.float32(2.0 ** power)).astype(np.float32), v)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("magnitude", [1e33, 1e35, 1e36])
def test_values_near_the_largest_float(shape, magnitude):
    """Weights are at most 1 before they are divided by their sum, so sums of values of 1e36 are finite."""
    q, k, v = inputs(*shape)
    check(shape, q, k, v * np.float32(magnitude))


@pytest.mark.parametrize("shape", SHAPES)
def test_the_largest_float_as_a_value(shape):
    q, k, v = inputs(*shape)
    v[:, 7, 3] = np.finfo(np.float32).max
    v[:, 8, 4] = -np.finfo(np.float32).max
    check(shape, q, k, v)


@pytest.mark.parametrize("shape", SHAPES)
def test_infinite_entries(shape):
    """A key whose score is minus infinity has no weight; an infinite value makes its column infinite and nothing else."""
    H_q, H_k, d, A, L_c, L_clean = shape
    q, k, v = inputs(*shape)
    q[:, :, 0] = np.abs(q[:, :, 0]) + 0.1
    far = k.copy()
    far[:, 9, 0] = -1e6
    k[:, 9, 0] = -np.inf
    check(shape, q, k, v, k_ref=far)
    q, k, v = inputs(*shape)
    plain, _ = attend(q, k, v, A, L_c, L_clean)
    v[:, 9, 5] = np.inf
    got, _ = attend(q, k, v, A, L_c, L_clean)
    assert (got[:, :, 5] == np.inf).all()
    # the same sums in the other columns, perhaps by another path
    others = np.arange(d) != 5
    assert np.abs(got[:, :, others] - plain[:, :, others]).max() <= BAR * np.abs(plain).max()


# ------------------------------------------------------------------ importance
# (d, H_q, H_k, W, L): merged with and without the launch between the passes; two and four tiles of rows, and few rows
MASS_SHAPES = [(64, 4, 1, 50, 512), (128, 2, 2, 40, 3000), (128, 8, 2, 130, 900), (64, 2, 2, 3, 3000)]


def check_mass(d, H_q, H_k, W, L, q, k, k_ref=None):
    got = B.flowcache_attention_mass(dev(q, "f32"), dev(k, "f32"), L).cpu().numpy().astype(np.float64)
    ref = O.attention_mass(q, k if k_ref is None else k_ref, L)
    assert (np.abs(got - ref) / np.where(ref > 1e-30, ref, 1.0)).max() <= BAR, (d, W, L)


@pytest.mark.parametrize("d,H_q,H_k,W,L", MASS_SHAPES)
@pytest.mark.parametrize("kind", ["channels", "apart", "keys large", "keys small", "infinite", "far apart", "very far apart"])
def test_importance_over_the_range(d, H_q, H_k, W, L, kind):
    rng = np.random.default_rng(W)
    q = rng.standard_normal((W, H_q, d)).astype(np.float32)
    k = rng.standard_normal((H_k, L, d)).astype(np.float32)
    k_ref, half = None, d // 2
    if kind == "channels":
        q[:, :, :half] *= np.float32(2.0 ** -30)
        k[:, :, :half] *= np.float32(2.0 ** 30)
    elif kind == "apart":                        # huge entries that never meet: scores of zero and of O(1)
        q[::2, :, :half], q[::2, :, half:] = 1e25, 0.0
        k[:, ::3, :half], k[:, ::3, half:] = 0.0, 1e25
        q[1::2, :, half:] *= np.float32(1e-25)
        k[:, 1::3, :half] = k[:, 2::3, :half] = 0.0
    elif kind == "keys large":
        q, k = q * np.float32(2.0 ** -120), k * np.float32(2.0 ** 120)
    elif kind == "keys small":
        q, k = q * np.float32(2.0 ** 100), k * np.float32(2.0 ** -100)
    elif kind == "far apart":                    # scores to 1e13, by far the most of a row in one key
        q, k = np.float32(2.0 ** 20) * q, np.float32(2.0 ** 20) * k
    elif kind == "very far apart":               # and to 1e32
        q, k = np.float32(2.0 ** 52) * q, np.float32(2.0 ** 52) * k
    else:
        q[:, :, 0] = np.abs(q[:, :, 0]) + 0.1
        k_ref = k.copy()
        k_ref[:, 9, 0] = -1e6
        k[:, 9, 0] = -np.inf
    check_mass(d, H_q, H_k, W, L, q.astype(np.float32), k.astype(np.float32), k_ref)
