"""The calls a denoising program makes on this library, over the sizes it makes them at.

Four kinds of case, each one pass through the public binding:

``tick``      one layer's share of a denoising tick in which something is recomputed: change metric,
              decision and gather; the new K/V into their cache slots and the chunk-causal attention;
              cached-activation store / apply.  With ``mass`` the attention also emits the importance.
``reuse``     a tick in which every chunk is past warm-up and drifting slowly, so that the stack is
              skipped: decision (per chunk, or the uniform policy) and cached-activation apply.  Most
              ticks of a run are of this kind.
``mass``      importance of the cached keys for a window of observation queries (Eq. (9)).
``compress``  scoring, top-B selection and in-place compaction at a chunk commit, by token or by
              groups of tokens (a latent frame).

The shapes are those of the repository's workloads: a MAGI-1-like layer (24 x 128, chunks of 6 x 30 x
52 = 9360 tokens), a SkyReels-V2-1.3B-like layer (12 x 128, chunks of 5 x 34 x 60 = 10200 tokens), the
tiny fp32 step of the smoke test and the reduced ragged shapes of the tests.
"""
import math

import torch

from paper_2602_10825_amd import binding as B

DEV = "cuda"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
WARMUP_M, POOL_K, LAMBDA = 4, 7, 0.07


def _tick(name, dtype, H_q, H_k, d, A, R, L_c, L_clean, eps=0.1, mass=False):
    return {"name": name, "kind": "tick", "dtype": dtype, "H_q": H_q, "H_k": H_k, "d": d, "A": A, "R": R,
            "L_c": L_c, "L_clean": L_clean, "eps": eps, "mass": mass}


def _reuse(name, dtype, width, A, L_c, policy, eps=0.1):
    return {"name": name, "kind": "reuse", "dtype": dtype, "width": width, "A": A, "L_c": L_c,
            "policy": policy, "eps": eps}


def _mass(name, dtype, H_q, H_k, d, W, L):
    return {"name": name, "kind": "mass", "dtype": dtype, "H_q": H_q, "H_k": H_k, "d": d, "W": W, "L": L}


def _compress(name, dtype, H, d, L, budget, group, keys):
    return {"name": name, "kind": "compress", "dtype": dtype, "H": H, "d": d, "L": L, "budget": budget,
            "group": group, "keys": keys}


def listed():
    return [
        # the smallest step: four query heads on one key head, two chunks of 2 x 8 x 8 tokens, fp32
        _tick("tick tiny f32", "f32", 4, 1, 64, 2, 2, 128, 512, eps=0.05, mass=True),
        # fp32 at the size of a small layer; no length is a multiple of a tile
        _tick("tick ragged f32", "f32", 12, 12, 128, 2, 2, 1021, 4083),
        # small bf16 layer with grouped heads and ragged lengths, one of three chunks recomputed
        _tick("tick small grouped", "bf16", 8, 2, 128, 3, 1, 328, 1000),
        # head dimension 64, many short chunks in the window (a frame of 34 x 60 tokens each)
        _tick("tick d64 window 5", "bf16", 24, 24, 64, 5, 2, 2040, 8160),
        # SkyReels-like layer, only the newest chunk recomputed: the usual tick that computes at all
        _tick("tick skyreels newest", "bf16", 12, 12, 128, 2, 1, 10200, 40800),
        # MAGI-1-like layer, every chunk recomputed: the largest step
        _tick("tick magi all", "bf16", 24, 24, 128, 4, 4, 9360, 74880, eps=0.015),
        # the tick that skips the stack, MAGI-1-like activations
        _reuse("reuse magi", "bf16", 24 * 128, 4, 9360, "chunk"),
        # the default observation window (50 rows) over a full cache at a commit
        _mass("mass skyreels 50", "bf16", 12, 12, 128, 50, 51000),
        # frame-level observation queries: a fifth of a chunk
        _mass("mass magi frame", "bf16", 24, 24, 128, 1872, 74880),
        # commit of a reduced model: launches count
        _compress("compress small", "bf16", 4, 128, 1312, 984, 1, "normal"),
        # commits at full length: steady state of a four-chunk budget, and half of the cache dropped
        _compress("compress skyreels", "bf16", 12, 128, 51000, 40800, 1, "heavy"),
        _compress("compress magi", "bf16", 24, 128, 74880, 37440, 1, "clustered"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; lengths are odd as often as not."""
    kind = rng.choice(("tick", "tick", "tick", "reuse", "mass", "compress", "compress"))
    dtype = "bf16" if rng.random() < 0.75 else "f32"
    d = rng.choice((64, 128, 128))
    H_k = rng.choice((1, 2, 4, 8, 12, 12, 24))
    H_q = H_k * rng.choice((1, 1, 1, 2, 4)) if H_k <= 8 else H_k
    if kind == "tick":
        A = rng.choice((1, 2, 2, 3, 4, 4, 6))
        R = rng.randint(1, A)
        most = 4.0e13 if dtype == "bf16" else 1.5e11      # costs no more than the largest listed tick
        while True:
            c = _tick("", dtype, H_q, H_k, d, A, R, _log(rng, 64, 10200), _log(rng, 256, 74880),
                      eps=rng.choice((0.015, 0.05, 0.1)), mass=rng.random() < 0.3)
            if work(c)["flops"] <= most:
                break
    elif kind == "reuse":
        c = _reuse("", dtype, H_q * d, rng.choice((1, 2, 4, 4, 8)), _log(rng, 64, 9360),
                   rng.choice(("chunk", "chunk", "uniform")))
    elif kind == "mass":
        W = rng.choice((1, 32, 50, 50, 64)) if rng.random() < 0.6 else _log(rng, 65, 2040)
        most = 1.7e12 if dtype == "bf16" else 2.0e10
        while True:
            c = _mass("", dtype, H_q, H_k, d, W, _log(rng, 500, 84240))
            if work(c)["flops"] <= most:
                break
    else:
        L = _log(rng, 600, 84240)
        group = rng.choice((1, 1, 1, 1, rng.choice((60, 65, 208))))
        L = max(2, L // group) * group
        budget = max(1, int(L // group * rng.uniform(0.4, 0.95))) * group
        c = _compress("", dtype, H_k, d, L, budget, group, rng.choice(("normal", "clustered", "heavy")))
    del c["name"]
    return c


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(dtype)


def _keys(g, kind, H, L, d, dtype):
    """Key rows: independent; 32 cluster centres with small scatter; or heavy-tailed with near copies."""
    if kind == "normal":
        return _normal(g, (H, L, d), dtype)
    if kind == "clustered":
        centre = torch.randn((H, 32, d), generator=g, device=DEV)
        which = torch.randint(0, 32, (H, L, 1), generator=g, device=DEV).expand(H, L, d)
        return (torch.gather(centre, 1, which) + 0.1 * torch.randn((H, L, d), generator=g, device=DEV)).to(dtype)
    k = torch.randn((H, L, d), generator=g, device=DEV)
    chi = torch.zeros((H, L, d), device=DEV)
    for _ in range(3):                                    # Student-t with three degrees of freedom
        chi += torch.randn((H, L, d), generator=g, device=DEV) ** 2
    k /= (chi / 3.0).sqrt_()
    copied = torch.rand((H, L, 1), generator=g, device=DEV) < 0.2
    near = torch.roll(k, 977 % L, 1)
    near = near + 0.01 * near.abs().mean() * torch.randn((H, L, d), generator=g, device=DEV)
    return torch.where(copied, near, k).to(dtype)


def _importance(g, H, L):
    """Positive, heavy-tailed, rows sum to one, with plateaus."""
    m = torch.empty((H, L), device=DEV).exponential_(generator=g) ** 2
    flat = torch.rand((H, L), generator=g, device=DEV) < 1.0 / 16
    m = torch.where(flat, torch.roll(m, 1, 1), m)
    return (m / m.sum(1, keepdim=True)).contiguous()


def _drift(g, A, elems, dtype):
    """Activations of two consecutive ticks; each chunk has its own, small, rate of change."""
    x_prev = _normal(g, (A, elems), dtype)
    sigma = 1e-3 * torch.exp(torch.rand((A, 1), generator=g, device=DEV))
    noise = torch.randn((A, elems), generator=g, device=DEV)
    return (x_prev.float() + sigma * noise).to(dtype), x_prev


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    g = _generator(seed)
    dtype = DTYPES[case["dtype"]]
    code = B.FC_BF16 if case["dtype"] == "bf16" else B.FC_F32
    L = B.lib()
    s = {"case": case}
    if case["kind"] in ("tick", "reuse"):
        A, L_c = case["A"], case["L_c"]
        width = case["width"] if case["kind"] == "reuse" else case["H_q"] * case["d"]
        s["x_cur"], s["x_prev"] = _drift(g, A, L_c * width, dtype)
        s["x_compact"] = torch.zeros_like(s["x_cur"])
        s["residual"] = _normal(g, (A, L_c * width), dtype)
        s["full"] = torch.zeros_like(s["x_cur"])
        s["ws_decide"] = _workspace(L.flowcache_chunk_decide_workspace(A, L_c * width))
        uniform = case.get("policy") == "uniform"
        s["acc"] = torch.zeros(1 if uniform else A, dtype=torch.float64, device=DEV)
        # the newest R chunks of a tick are in warm-up and recompute; the others are past it
        fresh = case["R"] if case["kind"] == "tick" else 0
        steps = [WARMUP_M + 8] * (A - fresh) + [1] * fresh
        s["step_idx"] = torch.tensor(steps, dtype=torch.int32, device=DEV)
    if case["kind"] == "tick":
        H_q, H_k, d, L_clean = case["H_q"], case["H_k"], case["d"], case["L_clean"]
        s["q"] = _normal(g, (A * L_c, H_q, d), dtype)
        s["k_new"] = _normal(g, (A * L_c, H_k, d), dtype)
        s["v_new"] = _normal(g, (A * L_c, H_k, d), dtype)
        s["k_cache"] = _normal(g, (H_k, L_clean + A * L_c, d), dtype)
        s["v_cache"] = _normal(g, (H_k, L_clean + A * L_c, d), dtype)
        s["active_off"] = [L_clean + i * L_c for i in range(A)]
        s["out"] = torch.zeros_like(s["q"])
        s["mass_len"] = L_clean if case["mass"] else 0
        s["ws_attend"] = _workspace(L.flowcache_attend_workspace(A, L_c, H_q, H_k, d, s["mass_len"], 50))
    elif case["kind"] == "mass":
        s["q_obs"] = _normal(g, (case["W"], case["H_q"], case["d"]), dtype)
        s["k_cache"] = _normal(g, (case["H_k"], case["L"] + case["L"] // 4, case["d"]), dtype)
        s["ws"] = _workspace(L.flowcache_attention_mass_workspace(case["W"], case["H_q"], case["H_k"], case["d"],
                                                                  case["L"]))
    elif case["kind"] == "compress":
        H, d, n = case["H"], case["d"], case["L"]
        tail = n // 4                                     # the slots of the chunks in flight
        s["k_cache"] = torch.cat([_keys(g, case["keys"], H, n, d, dtype), _normal(g, (H, tail, d), dtype)], 1)
        s["v_cache"] = _normal(g, (H, n + tail, d), dtype)
        s["mass"] = _importance(g, H, n)
        s["kept"] = torch.zeros((H, case["budget"]), dtype=torch.int32, device=DEV)
        if case["group"] > 1:
            s["ws"] = _workspace(L.flowcache_kv_compress_grouped_workspace(H, n, d, case["budget"], case["group"],
                                                                           code))
        else:
            s["ws"] = _workspace(L.flowcache_kv_compress_workspace(H, n, d, case["budget"], code))
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "mass":
        return B.flowcache_attention_mass(s["q_obs"], s["k_cache"], case["L"], workspace=s["ws"])
    if case["kind"] == "compress":
        if case["group"] > 1:
            kept = B.flowcache_kv_compress_grouped(s["k_cache"], s["v_cache"], case["L"], case["budget"],
                                                   case["group"], s["mass"], POOL_K, LAMBDA, kept_idx=s["kept"],
                                                   workspace=s["ws"])
        else:
            kept = B.flowcache_kv_compress(s["k_cache"], s["v_cache"], case["L"], case["budget"], s["mass"],
                                           POOL_K, LAMBDA, kept_idx=s["kept"], workspace=s["ws"])
        return kept, s["k_cache"], s["v_cache"]
    decide = B.flowcache_uniform_decide if case.get("policy") == "uniform" else B.flowcache_chunk_decide
    dec = decide(s["x_cur"], s["x_prev"], s["step_idx"], WARMUP_M, case["eps"], s["acc"],
                 x_compact=s["x_compact"], workspace=s["ws_decide"])
    y, att = None, {}
    if case["kind"] == "tick":
        att = B.flowcache_attend(s["q"], s["k_new"], s["v_new"], s["k_cache"], s["v_cache"], case["L_c"],
                                 case["L_clean"], s["active_off"], dec["recompute_idx"], dec["n_recompute"],
                                 out=s["out"], want_lse=False, mass_len=s["mass_len"], workspace=s["ws_attend"])
        y = s["out"].view(case["A"], -1)
    full = B.flowcache_residual_apply(s["x_cur"], y, s["residual"], dec["recompute_idx"], dec["n_recompute"],
                                      out=s["full"])
    return {"decision": dec, "out": att.get("out"), "mass": att.get("mass"), "residual": s["residual"],
            "full": full, "k_cache": s.get("k_cache"), "v_cache": s.get("v_cache")}


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "mass":
        # K and the queries read, the importance written; one product Q K^T
        keys = case["H_k"] * case["L"]
        return {"bytes": keys * (case["d"] * e + 4) + case["W"] * case["H_q"] * case["d"] * e,
                "flops": 2 * case["W"] * case["H_q"] * case["L"] * case["d"]}
    if case["kind"] == "compress":
        # K once for the scores, the kept rows of K and V read and written, importance and index list
        row = case["d"] * e
        return {"bytes": case["H"] * (case["L"] * (row + 4) + case["budget"] * (4 * row + 4)),
                "flops": 6 * case["H"] * case["L"] * case["d"]}
    A, L_c = case["A"], case["L_c"]
    width = case["width"] if case["kind"] == "reuse" else case["H_q"] * case["d"]
    R = case["R"] if case["kind"] == "tick" else 0
    x = L_c * width * e
    # both activations read and the full layout written; a reused chunk reads its difference, a
    # recomputed one is gathered and stores its difference
    nbytes = A * 3 * x + (A - R) * x + R * 2 * x
    flops = 3 * A * L_c * width
    if case["kind"] == "tick":
        H_q, H_k, d, L_clean = case["H_q"], case["H_k"], case["d"], case["L_clean"]
        seen = [L_clean + (c + 1) * L_c for c in range(A - R, A)]
        nbytes += 2 * R * x                               # queries in, attention out
        nbytes += 2 * 2 * R * L_c * H_k * d * e           # new K/V in and into their slots
        nbytes += 2 * max(seen) * H_k * d * e             # the visible keys and values
        flops += 4 * H_q * d * L_c * sum(seen)
        if case["mass"]:
            nbytes += H_k * L_clean * 4
            flops += 2 * min(50, L_c) * H_q * L_clean * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what was measured against the same path in float64: fp32 softmax sums of the
    importance 4e-7 (largest entry 1.3e-6), fp32 attention 1.5e-6 (9e-6), bf16 attention 2.4e-3 (1.0e-2, the
    rounding of the weights and of the output).  Positions, counts and moved bytes are exact in every
    kind; the compression's outputs are nothing else, and the float64 sums of the decisions differ by
    their order alone."""
    if case["kind"] == "compress":
        return "exact"
    if case["kind"] == "reuse":
        return {"rel": 1e-12, "max": 1e-11}
    if case["kind"] == "mass":
        return {"rel": 2e-6, "max": 6e-6}
    return {"rel": 1e-2, "max": 4e-2} if case["dtype"] == "bf16" else {"rel": 6e-6, "max": 4e-5}
