"""fp32 importance mass on the matrix cores: 32 rows (pass 1) or 32 keys (pass 2) stay in a wavefront, eight
wavefronts to a block, key ranges over blocks.  Sizes at the edges: one row and one key, a tile of rows or
keys more or less, fewer key tiles than wavefronts, several ranges, one to eight wavefronts on the same
keys, and the one-thread-per-key kernels for one or two rows; against the float64 oracle at its usual bars."""
import numpy as np
import pytest

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import binding as B
from tests._checks import assert_mass_close
from tests.test_gpu_parity import dev

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
    (64, 3, 1, 1, 257, 1.0), (128, 2, 2, 3, 257, 1.0),                              # and just past it
])
def test_mass_f32(d, H_q, H_k, W, L, grow):
    rng = np.random.default_rng(L + W)
    q = rng.standard_normal((W, H_q, d)).astype(np.float32)
    k = rng.standard_normal((H_k, L + 9, d)).astype(np.float32)
    k[:, L // 2:] *= grow
    k[:, L:] *= 100.0                 # past the scored range: must not count
    got = B.flowcache_attention_mass(dev(q, "f32"), dev(k, "f32"), L).cpu().numpy().astype(np.float64)
    assert_mass_close(got, O.attention_mass(q, k, L), "f32", f"W={W} L={L}")
