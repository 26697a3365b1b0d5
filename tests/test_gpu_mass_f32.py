"""fp32 importance mass on the matrix cores: 32 rows (pass 1) or 32 keys (pass 2) stay in a wavefront, eight
wavefronts to a block, key ranges over blocks.  Sizes at the edges: one row and one key, a tile of rows or
keys more or less, fewer key tiles than wavefronts, several ranges, one to eight wavefronts on the same
keys, tiles with rows of several query heads, and the one-thread-per-key kernels for few rows; against the float64 oracle at its usual bars."""
import numpy as np
import pytest
import torch

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import binding as B
from tests._checks import assert_mass_close
from tests.test_gpu_parity import DEV, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H_q,H_k,W,L,grow", [
    (128, 1, 1, 1, 1, 1.0),
    (64, 2, 1, 32, 31, 1.0), (128, 2, 2, 33, 33, 1.0),
    (64, 4, 1, 50, 512, 1.0),         # eight row tiles over the heads of one key head
    (128, 12, 12, 50, 4000, 1.0),     # ranges of pass 1
    (64, 1, 1, 65, 511, 1.0),         # two groups, one range
    (128, 2, 1, 130, 1100, 4.0),      # scores that grow along the keys
    (64, 24, 24, 20, 6000, 4.0),      # enough key blocks that no two wavefronts share one
    (128, 1, 1, 300, 3000, 1.0),
    (128, 3, 3, 1, 1000, 1.0), (64, 2, 1, 1, 257, 4.0), (64, 1, 1, 2, 3000, 4.0),   # one thread per key
    (64, 3, 1, 1, 257, 1.0), (128, 2, 2, 3, 257, 1.0),
    (64, 16, 4, 1, 8191, 1.0), (64, 16, 4, 1, 8192, 1.0),   # four rows of four heads: the last length of that
    (128, 8, 8, 4, 8200, 1.0), (64, 16, 8, 4, 12289, 4.0),  # four and eight rows, long
    (64, 16, 8, 4, 12287, 1.0), (128, 16, 8, 5, 600, 1.0),  # tiles that hold rows of several heads of one key head
    (64, 12, 3, 9, 1100, 1.0), (128, 8, 2, 65, 300, 1.0), (64, 6, 2, 11, 40, 1.0),
])
def test_mass_f32(d, H_q, H_k, W, L, grow):
    rng = np.random.default_rng(L + W)
    q = rng.standard_normal((W, H_q, d)).astype(np.float32)
    k = rng.standard_normal((H_k, L + 9, d)).astype(np.float32)
    k[:, L // 2:] *= grow
    k[:, L:] *= 100.0                 # past the scored range: must not count
    got = B.flowcache_attention_mass(dev(q, "f32"), dev(k, "f32"), L).cpu().numpy().astype(np.float64)
    assert_mass_close(got, O.attention_mass(q, k, L), "f32", f"W={W} L={L}")


def test_mass_f32_of_more_rows_than_a_grid_dimension_has_blocks():
    """65536 tiles of 32 rows and one row more; the reference in float64 on the device."""
    W, L, d = 65536 * 32 + 1, 8, 64
    g = torch.Generator(device=DEV).manual_seed(1)
    q = torch.randn((W, 1, d), generator=g, device=DEV)
    k = torch.randn((1, L, d), generator=g, device=DEV)
    got = B.flowcache_attention_mass(q, k, L).double()
    ref = sum(torch.softmax(x[:, 0].double() @ k[0].double().T * d ** -0.5, 1).sum(0) for x in q.split(1 << 18)) / W
    # a lane adds W / 32 / 8 terms one after the other: at most that many roundings of 2^-24, far fewer as
    # they go both ways; a tenth of that bound
    assert float((got[0] - ref).abs().max() / ref.min()) <= 0.1 * (W / 256) * 2.0 ** -24


@pytest.mark.parametrize("d,H_q,H_k,W,L", [(64, 4, 1, 64, 1024), (64, 4, 1, 65, 1290), (128, 2, 2, 40, 256), (128, 1, 1, 257, 900)])
def test_mass_f32_rows_and_keys_of_any_magnitude(d, H_q, H_k, W, L):
    """Queries and keys are split into two f16 parts after scaling by powers of two, per row and per key: rows of zeros,
    of subnormal numbers and of magnitudes over 30 decimal orders whose scores stay O(1); up to eight tiles of rows and
    four partials per row are merged without the launch between the passes, more with it.  The usual bars."""
    rng = np.random.default_rng(W)
    q = rng.standard_normal((W, H_q, d)).astype(np.float32)
    k = rng.standard_normal((H_k, L, d)).astype(np.float32)
    k *= (10.0 ** rng.uniform(-8, 0.2, L)).astype(np.float32)[None, :, None]
    q *= (10.0 ** rng.uniform(-20, 0.2, W)).astype(np.float32)[:, None, None]
    k[:, 3::5] = 0
    k[:, 4::50] *= np.float32(1e-35)
    q[::7] = 0
    q[1::9] *= np.float32(1e-20)
    got = B.flowcache_attention_mass(dev(q, "f32"), dev(k, "f32"), L).cpu().numpy().astype(np.float64)
    assert_mass_close(got, O.attention_mass(q, k, L), "f32", f"W={W} L={L}")
