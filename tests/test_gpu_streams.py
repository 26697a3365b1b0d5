"""Calls enqueued on another stream than the current one (`stream=`), without a workspace of the caller's."""
import pytest
import torch

from paper_2602_10825_amd import binding as B
from paper_2602_10825_amd import synth
from tests.test_gpu_parity import DEV, dev

pytestmark = pytest.mark.gpu


def calls(side):
    """name -> a call on `side`, or on the current stream for None"""
    wl = synth.Workload("streams", "bf16", 2, 2, 64, 2, 48, 4000, 1)
    a = synth.attend_inputs(wl, seed=6)
    idx, n = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in ([1, -1], [1]))
    q, k, v = (dev(a[x], "bf16") for x in ("q", "k_cache", "v_cache"))
    mass = torch.rand((2, 4000), device=DEV)
    return {
        "attend": lambda: B.flowcache_attend(q, None, None, k, v, wl.L_c, wl.L_clean, a["active_off"], idx, n,
                                             stream=side)["out"][:wl.L_c],
        "mass": lambda: B.flowcache_attention_mass(q[:50].contiguous(), k, 4000, stream=side),
        "select": lambda: B.flowcache_kv_select(k, 4000, 2000, mass, stream=side),
    }


@pytest.mark.parametrize("name", ["attend", "mass", "select"])
def test_scratch_is_not_handed_out_while_the_other_stream_uses_it(name, monkeypatch):
    side = torch.cuda.Stream()
    scratch = []
    make = B._workspace

    def spy(*args):
        scratch.append(make(*args))
        return scratch[-1]

    torch.manual_seed(1)
    want = calls(None)[name]().clone()
    torch.manual_seed(1)
    call = calls(side)[name]
    torch.cuda.synchronize()
    monkeypatch.setattr(B, "_workspace", spy)
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)               # some milliseconds ahead of the call
    got = call()
    ptr, nbytes = scratch[0].data_ptr(), scratch[0].numel()
    scratch.clear()                                 # given back while `side` has not begun
    again = [torch.empty(nbytes, dtype=torch.uint8, device=DEV) for _ in range(4)]
    for t in again:
        assert t.data_ptr() + nbytes <= ptr or ptr + nbytes <= t.data_ptr()
        t.fill_(255)
    side.synchronize()
    assert torch.equal(got, want)
