"""Importance mass for more than 64 observation rows in bf16: wavefronts of 64 resident rows (pass 1) or
keys (pass 2), 2, 4 or 8 to a block, and tiles of 64 passing rows.  Sizes at the edges of those, of
the key ranges of pass 1 and of the block widths, against the float64 oracle at its usual bars; and
scores that grow along the keys, so that the reference point of the sums is raised on the way."""
import numpy as np
import pytest

from oracle import flowcache_oracle as O
from paper_2602_10825_amd import binding as B
from paper_2602_10825_amd import synth
from tests._checks import assert_mass_close
from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H_q,H_k,W,L,grow", [
    (128, 1, 1, 65, 1, 1.0),          # one key
    (128, 2, 1, 128, 63, 1.0),        # two full groups, a tile less one; grouped heads
    (64, 2, 2, 129, 65, 1.0),         # three groups in a block of four, a tile and one
    (128, 1, 1, 257, 511, 1.0),       # five groups in a block of eight; one range
    (64, 4, 2, 193, 1025, 1.0),       # two ranges, the second one key longer than whole tiles
    (128, 2, 2, 577, 1217, 1.0),      # ten groups: a second block with two
    (128, 1, 1, 70, 9001, 12.0),      # many ranges; the scores of the second half are twelvefold
    (128, 4, 4, 300, 3000, 12.0),
    (64, 16, 16, 66, 16500, 1.0),     # blocks of 8 wavefronts in pass 2, ragged end
    (64, 8, 8, 80, 17000, 1.0),       # blocks of 4
])
def test_mass_of_many_rows(d, H_q, H_k, W, L, grow):
    rng = np.random.default_rng(L + W)
    q = synth.to_storage(rng.standard_normal((W, H_q, d)).astype(np.float32), "bf16")
    k = rng.standard_normal((H_k, L + 9, d)).astype(np.float32)
    k[:, L // 2:] *= grow
    k[:, L:] *= 100.0                 # past the scored range: must not count
    k = synth.to_storage(k, "bf16")
    got = B.flowcache_attention_mass(dev(q, "bf16"), dev(k, "bf16"), L).cpu().numpy().astype(np.float64)
    assert_mass_close(got, O.attention_mass(q, k, L), "bf16", f"W={W} L={L}")
