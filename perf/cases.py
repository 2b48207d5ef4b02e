"""The work that users of this library have it do, as timed cases.

A case names an entry point of paper_2607_02963_amd.pdec and its sizes; the
kinds are
  step      attn_step: one decode step of one video
  ragged    attn_step_ragged: one decode step over a batch of videos
  loop      decode_step: consecutive steps with the cache append fused in
  rope      rope_kv_append, then attn_step: a step from unrotated q and k
  prefill   attn_prefill / attn_prefill_ragged: whole branches at once
  causal    attn_prefill of one stream over an empty prefix: the prefix's own
            causal attention
  train     attn_prefill, then attn_prefill_backward: one training step of
            the attention
  ground    segment_grounding
  aggregate aggregate

Shapes: videos of up to 256 frames give prefixes of thousands to tens of
thousands of tokens, about 13 event streams per video with about 42 tokens
each (captions of about 549 tokens per video), 28 query heads over 4 kv heads
of width 128 as in a 7B Omni-LLM.  Queries and keys are normal with a spread
that gives scaled scores a standard deviation of about 1.5 nats, so a softmax
row has keys that matter and keys that do not; values are normal * 0.5.
"""
import math
import random

import torch

from paper_2607_02963_amd import pdec

Q_SIGMA, K_SIGMA, V_SIGMA = 1.5, 1.0, 0.5
THETA = 1000000.0


def listed():
    return [
        # The smallest call: a float32 check-sized step, where launches and latency are all there is.
        {"name": "step_f32_tiny", "kind": "step", "dtype": "f32", "H_q": 4, "H_kv": 1, "D": 64, "L": 256, "E": 4,
         "own": 15, "ended": 0, "plan": 0},
        # The full head layout in float32 (a precision reference run of a decode).
        {"name": "step_f32_4k", "kind": "step", "dtype": "f32", "H_q": 28, "H_kv": 4, "D": 128, "L": 4095, "E": 13,
         "own": 42, "ended": 0, "plan": 0},
        # An ordinary step: a short video, 8 event streams.
        {"name": "step_8k", "kind": "step", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "L": 8192, "E": 8,
         "own": 64, "ended": 0, "plan": 0},
        # The library's headline step: a long video, 32 streams.
        {"name": "step_32k", "kind": "step", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "L": 32768, "E": 32,
         "own": 128, "ended": 0, "plan": 0},
        # A serving batch: 16 videos of their own lengths and stream counts.
        {"name": "ragged_16", "kind": "ragged", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "V": 16,
         "L_lo": 4096, "L_hi": 16384, "E_lo": 4, "E_hi": 24, "own": 96, "ended": 3, "plan": 0},
        # Eight consecutive steps of a decode loop, the cache append fused in.
        {"name": "loop_16k", "kind": "loop", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "L": 16384, "E": 16,
         "own": 48, "ended": 2, "steps": 8},
        # One step as a model calls it: rotate and append, then attend (an odd prefix, the mean stream count).
        {"name": "rope_step_12k", "kind": "rope", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "L": 12001,
         "E": 13, "own": 42, "ended": 1},
        # Teacher-forced branches (scoring, training forward): the mean video over a long prefix.
        {"name": "prefill_32k", "kind": "prefill", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "V": 1,
         "L_lo": 32768, "L_hi": 32768, "E_lo": 13, "E_hi": 13, "N": 48, "ended": 0, "cross": 0},
        # The prefix's own causal attention: the prefill of a long video.
        {"name": "causal_16k", "kind": "causal", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "L": 16384},
        # One training step of the attention: forward and every gradient.
        {"name": "train_32k", "kind": "train", "dtype": "bf16", "H_q": 28, "H_kv": 4, "D": 128, "L": 32768, "E": 13,
         "N": 48, "ended": 0},
        # Segment grounding of 32 event tokens over a long video's audio-visual tokens.
        {"name": "ground_32k", "kind": "ground", "K": 32, "N": 32704, "S": 128, "d": 256},
        # Attention-guided aggregation of the same tokens into the event tokens.
        {"name": "aggregate_32k", "kind": "aggregate", "mode": "attention", "K": 32, "N": 32704, "S": 128,
         "hidden": 3584, "H_q": 28, "H_kv": 4, "D": 128},
    ]


HEADS = [(28, 4), (28, 4), (28, 4), (16, 2), (8, 8), (7, 1), (32, 8), (40, 8)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Sizes over the ranges the library is used in; both head widths, several head layouts, odd lengths."""
    kind = rng.choice(["step", "step", "step", "ragged", "loop", "rope", "prefill", "prefill", "causal", "causal",
                       "train", "train", "ground", "aggregate"])
    H_q, H_kv = rng.choice(HEADS)
    D = rng.choice([128, 128, 128, 64])
    c = {"kind": kind, "dtype": "bf16", "H_q": H_q, "H_kv": H_kv, "D": D}
    if kind == "step":
        if rng.random() < 0.25:
            c["dtype"] = "f32"
        c.update(L=_log(rng, 200, 8000 if c["dtype"] == "f32" else 40000), E=_log(rng, 1, 48), own=_log(rng, 1, 200),
                 ended=0, plan=0)
        c["ended"] = rng.randint(0, c["E"] // 4)
        if rng.random() < 0.2:
            c["plan"] = rng.randint(1, 4) if c["E"] * 4 <= c["L"] else 0
    elif kind == "ragged":
        lo = _log(rng, 300, 8000)
        c.update(V=rng.randint(2, 16), L_lo=lo, L_hi=2 * lo + 1, E_lo=rng.randint(1, 6), E_hi=rng.randint(7, 24),
                 own=_log(rng, 4, 128), ended=rng.randint(0, 2), plan=0)
    elif kind == "loop":
        c.update(L=_log(rng, 500, 32000), E=_log(rng, 1, 32), own=_log(rng, 1, 100), ended=0,
                 steps=rng.randint(3, 8))
    elif kind == "rope":
        c.update(L=_log(rng, 500, 32000), E=_log(rng, 1, 32), own=_log(rng, 1, 100), ended=0)
    elif kind == "prefill":
        lo = _log(rng, 300, 16000)
        V = rng.choice([1, 1, 1, 2, 5])
        c.update(V=V, L_lo=lo, L_hi=lo if V == 1 else 2 * lo, E_lo=1 if V > 1 else 13, E_hi=13,
                 N=_log(rng, 6, 100), ended=rng.randint(0, 1), cross=int(rng.random() < 0.25))
    elif kind == "causal":
        c.update(L=_log(rng, 300, 16000))
    elif kind == "train":
        if rng.random() < 0.4:
            c.update(L=0, E=1, N=_log(rng, 200, 4000), ended=0)  # a whole text's causal attention
        else:
            c.update(L=_log(rng, 300, 16000), E=_log(rng, 2, 24), N=_log(rng, 6, 80), ended=rng.randint(0, 1))
    elif kind == "ground":
        c = {"kind": kind, "K": _log(rng, 1, 64), "N": _log(rng, 500, 64000), "S": _log(rng, 8, 256),
             "d": rng.choice([64, 128, 256])}
    else:
        c = {"kind": kind, "mode": rng.choice(["uniform", "learned", "attention"]), "K": _log(rng, 1, 64),
             "N": _log(rng, 500, 33000), "S": _log(rng, 8, 256), "hidden": rng.choice([2048, 3584, 1536, 1000]),
             "H_q": H_q, "H_kv": H_kv, "D": D}
    return c


# ---- structure and inputs ----

def _structure(c, seed):
    """Lengths of the case on the host: (prefix_lens, events_per_video, event_lens, cap).  A batch's stream counts
    are the case's, its prefix and stream lengths the seed's."""
    r = random.Random(1000003 * seed + 17)
    if c["kind"] in ("ragged", "prefill"):
        prefix = [r.randint(c["L_lo"], c["L_hi"]) for _ in range(c["V"])]
        counts = random.Random(131 * c["V"] + c["E_hi"])
        events = [counts.randint(c["E_lo"], c["E_hi"]) for _ in range(c["V"])]
    elif c["kind"] == "causal":
        prefix, events = [0], [1]
    else:
        prefix, events = [c["L"]], [c["E"]]
    SE = sum(events)
    if c["kind"] == "causal":
        return prefix, events, [c["L"]], c["L"]
    if c["kind"] in ("prefill", "train"):  # branches are padded to the longest: some are shorter
        N = c["N"]
        own = [N if SE == 1 or r.random() < 0.5 else r.randint(max(1, N // 2), N) for _ in range(SE)]
        cap = N
    else:
        own = [r.randint(0, c["own"]) + (1 if c["kind"] in ("step", "ragged") else 0) for _ in range(SE)]
        cap = c["own"] + 1 + c.get("steps", 0)
    for e in r.sample(range(SE), min(c.get("ended", 0), SE - 1)):
        own[e] = 0
    return prefix, events, own, cap


def _cum(v):
    out = [0]
    for x in v:
        out.append(out[-1] + x)
    return out


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, sigma, dtype):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * sigma).to(dtype)


def _ints(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _segments(c, seed):
    r = random.Random(1000003 * seed + 29)
    cuts = sorted(r.randint(0, c["N"]) for _ in range(c["S"] - 1))
    if c["S"] * 16 < c["N"]:  # time segments of about equal length, as frames give
        step = c["N"] / c["S"]
        cuts = sorted(min(c["N"], max(0, int((i + 1 + r.uniform(-0.2, 0.2)) * step))) for i in range(c["S"] - 1))
    return [0] + cuts + [c["N"]]


def _inputs(c, seed):
    """Every input tensor of the case."""
    g, bf = _generator(seed), torch.bfloat16
    if c["kind"] == "ground":
        cu = _segments(c, seed)
        ev, p = _normal(g, (c["K"], c["d"]), 0.5, torch.float32), _normal(g, (c["N"], c["d"]), 0.5, torch.float32)
        for i in range(c["K"]):  # each event resembles the tokens of one segment, as trained features do
            u = _normal(g, (c["d"],), 1.0, torch.float32)
            u /= u.norm()
            ev[i] += 2.0 * u
            s = (3 * i) % c["S"]
            p[cu[s]:cu[s + 1]] += 0.25 * u
        return {"g": ev.to(bf), "p": p.to(bf), "cu": _ints(cu), "cu_host": cu}
    if c["kind"] == "aggregate":
        cu, r = _segments(c, seed), random.Random(1000003 * seed + 31)
        sal = torch.zeros((c["K"], c["S"]), dtype=torch.uint8)
        for i in range(c["K"] - (c["K"] > 1)):  # runs of consecutive segments; the last event has none
            run = r.randint(1, min(8, c["S"]))
            at = r.randint(0, c["S"] - run)
            sal[i, at:at + run] = 1
        st = {"g": _normal(g, (c["K"], c["hidden"]), 0.5, bf), "x": _normal(g, (c["N"], c["hidden"]), 0.5, bf),
              "cu": _ints(cu), "cu_host": cu, "sal": sal.cuda()}
        if c["mode"] == "attention":
            st["q"] = _normal(g, (c["H_q"], c["D"]), 1.0, bf)
            st["k"] = _normal(g, (c["N"], c["H_kv"], c["D"]), 1.0, bf)
            st["lse"] = math.log(c["N"]) + 0.5 + torch.rand(c["H_q"], generator=g, device="cuda") - 0.5
        elif c["mode"] == "learned":
            st["scores"] = torch.rand(c["N"], generator=g, device="cuda") * 0.95 + 0.05
        return st
    prefix, events, own, cap = _structure(c, seed)
    dt = torch.float32 if c["dtype"] == "f32" else bf
    SE, SL, H_q, H_kv, D = sum(events), sum(prefix), c["H_q"], c["H_kv"], c["D"]
    N = {"prefill": c.get("N"), "train": c.get("N"), "causal": c.get("L")}.get(c["kind"])
    rows = (SE, H_q, D) if N is None else (SE, N, H_q, D)
    st = {"q": _normal(g, rows, Q_SIGMA, dt), "kp": _normal(g, (SL, H_kv, D), K_SIGMA, dt),
          "vp": _normal(g, (SL, H_kv, D), V_SIGMA, dt), "ke": _normal(g, (SE, cap, H_kv, D), K_SIGMA, dt),
          "ve": _normal(g, (SE, cap, H_kv, D), V_SIGMA, dt), "lens": _ints(own), "own": own, "prefix": prefix,
          "events": events, "cap": cap}
    if len(prefix) > 1:
        st["cup"], st["cue"] = _ints(_cum(prefix)), _ints(_cum(events))
    else:
        st["plen"] = _ints(prefix)
    if c["kind"] == "train":
        st["dout"] = _normal(g, rows, 0.5, dt)
    if c["kind"] in ("loop", "rope"):
        n = c.get("steps", 1)
        st["qs"] = _normal(g, (n, SE, H_q, D), Q_SIGMA, dt)
        st["kn"] = _normal(g, (n, SE, H_kv, D), K_SIGMA, dt)
        st["vn"] = _normal(g, (n, SE, H_kv, D), V_SIGMA, dt)
        st["live"] = _ints([0 if own[e] == 0 and c["ended"] else 1 for e in range(SE)])
        st["live_host"] = st["live"].tolist()
    if c["kind"] == "rope":
        st["pos"] = _ints([prefix[0]])
    return st


def prepare(case, seed):
    """Inputs, and the outputs and workspaces that a program keeps between calls."""
    c = case
    st = _inputs(c, seed)
    st["case"] = c
    dev = {"device": "cuda"}
    if c["kind"] == "ground":
        st["scores"] = torch.empty((c["K"], c["S"]), dtype=torch.float32, **dev)
        st["salient"] = torch.empty((c["K"], c["S"]), dtype=torch.uint8, **dev)
        ws = pdec.grounding_workspace_size(c["K"], c["N"], c["S"], c["d"])
    elif c["kind"] == "aggregate":
        st["out"] = torch.empty_like(st["g"])
        st["weights"] = torch.empty(c["N"], dtype=torch.float32, **dev) if c["mode"] == "attention" else None
        heads = (c["H_q"], c["H_kv"], c["D"]) if c["mode"] == "attention" else (0, 0, 0)
        ws = pdec.aggregation_workspace_size(c["K"], c["N"], c["S"], c["hidden"], c["mode"], *heads)
    else:
        q = st["q"]
        whole = q.dim() == 4
        st["out"] = torch.empty_like(q)
        st["lse"] = torch.empty(q.shape[:-1], dtype=torch.float32, **dev)
        code = pdec.PDEC_DTYPE_F32 if c["dtype"] == "f32" else pdec.PDEC_DTYPE_BF16
        V, bound = len(st["prefix"]), max(st["prefix"])
        dims = pdec.make_dims(q.shape[0], c["H_q"], c["H_kv"], c["D"], st["cap"], bound, code,
                              max_events_per_video=max(st["events"]) if V > 1 else 0,
                              prefix_tokens=st["kp"].shape[0] if V > 1 else 0,
                              plan_mask=int(c.get("plan", 0) > 0), plan_per_stream=c.get("plan", 0),
                              queries_per_stream=q.shape[1] if whole else 0, cross_causal=c.get("cross", 0))
        ws = pdec.workspace_size(dims, V)
        if c["kind"] == "train":
            st["bws"] = torch.empty(max(pdec.backward_workspace_size(dims), 16), dtype=torch.uint8, **dev)
        if c["kind"] == "loop":
            st["outs"] = [torch.empty_like(st["qs"][0]) for _ in range(c["steps"])]
            st["lses"] = [torch.empty_like(st["lse"]) for _ in range(c["steps"])]
            st["counts"] = [torch.empty_like(st["lens"]) for _ in range(2)]
    st["ws"] = torch.empty(max(ws, 256), dtype=torch.uint8, **dev)
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "ground":
        return pdec.segment_grounding(st["g"], st["p"], st["cu"], 0.5, scores=st["scores"], salient=st["salient"],
                                      workspace=st["ws"])
    if kind == "aggregate":
        out = pdec.aggregate(st["g"], st["x"], st["cu"], st["sal"], c["mode"], scores=st.get("scores"),
                             q=st.get("q"), k=st.get("k"), lse=st.get("lse"), weights=st["weights"], out=st["out"],
                             workspace=st["ws"])
        return (out, st["weights"])
    if kind == "step":
        return pdec.attn_step(st["q"], st["kp"], st["vp"], st["ke"], st["ve"], st["lens"], st["plen"],
                              out=st["out"], lse=st["lse"], workspace=st["ws"], plan_mask=int(c["plan"] > 0),
                              plan_per_stream=c["plan"])
    if kind == "ragged":
        return pdec.attn_step_ragged(st["q"], st["kp"], st["vp"], st["cup"], st["ke"], st["ve"], st["lens"],
                                     st["cue"], max_prefix_len=max(st["prefix"]),
                                     max_events_per_video=max(st["events"]), out=st["out"], lse=st["lse"],
                                     workspace=st["ws"])
    if kind == "loop":
        lens = st["lens"]
        for s in range(c["steps"]):
            after = st["counts"][s % 2]
            pdec.decode_step(st["qs"][s], st["kp"], st["vp"], st["kn"][s], st["vn"][s], st["ke"], st["ve"], lens,
                             after, st["live"], prefix_lens=st["plen"], out=st["outs"][s], lse=st["lses"][s],
                             workspace=st["ws"])
            lens = after
        return {"out": st["outs"], "lse": st["lses"], "lens": lens, "k": st["ke"], "v": st["ve"]}
    if kind == "rope":
        q, lens = st["qs"][0].clone(), st["lens"].clone()  # both are changed by the call
        pdec.rope_kv_append(q, st["kn"][0], st["vn"][0], st["ke"], st["ve"], lens, st["pos"], st["live"],
                            theta=THETA)
        out, lse = pdec.attn_step(q, st["kp"], st["vp"], st["ke"], st["ve"], lens, st["plen"], out=st["out"],
                                  lse=st["lse"], workspace=st["ws"])
        return {"out": out, "lse": lse, "q": q, "lens": lens, "k": st["ke"], "v": st["ve"]}
    if kind == "prefill" and "cup" in st:
        return pdec.attn_prefill_ragged(st["q"], st["kp"], st["vp"], st["cup"], st["ke"], st["ve"], st["lens"],
                                        st["cue"], max_prefix_len=max(st["prefix"]),
                                        max_events_per_video=max(st["events"]), out=st["out"], lse=st["lse"],
                                        workspace=st["ws"], cross=c["cross"])
    out, lse = pdec.attn_prefill(st["q"], st["kp"], st["vp"], st["ke"], st["ve"], st["lens"], st["plen"],
                                 out=st["out"], lse=st["lse"], workspace=st["ws"], cross=c.get("cross", 0))
    if kind != "train":
        return out, lse
    grads = pdec.attn_prefill_backward(st["q"], st["kp"], st["vp"], st["ke"], st["ve"], st["lens"], st["plen"], out,
                                       lse, st["dout"], workspace=st["bws"])
    return (out, lse, *grads)


# ---- what a pass cannot do without ----

def work(case):
    """Bytes: every input that the call has to see read once, every output written once.  Flops: the matrix
    products (2 per multiply-add) over the visible (row, key) pairs.  Lengths drawn from a seed count at their
    mean."""
    c = case
    if c["kind"] == "ground":
        K, N, S, d = c["K"], c["N"], c["S"], c["d"]
        return {"bytes": 2 * (N + K) * d + 5 * K * S + 4 * (S + 1), "flops": 2 * K * N * d}
    if c["kind"] == "aggregate":
        K, N, S, h = c["K"], c["N"], c["S"], c["hidden"]
        b, f = 2 * N * h + 4 * K * h + K * S + 4 * (S + 1), 2 * N * h
        if c["mode"] == "attention":
            b += 2 * N * c["H_kv"] * c["D"] + 4 * N
            f += 2 * N * c["H_q"] * c["D"]
        return {"bytes": b, "flops": f}
    es = 4 if c["dtype"] == "f32" else 2
    H_q, H_kv, D = c["H_q"], c["H_kv"], c["D"]
    row, qrow = 2 * H_kv * D * es, H_q * (2 * D * es + 4)
    if c["kind"] == "causal":
        L = c["L"]
        return {"bytes": L * (row + qrow), "flops": 4 * D * H_q * L * (L + 1) // 2}
    if c["kind"] in ("prefill", "train"):
        V = c.get("V", 1)
        L = c["L"] if "L" in c else (c["L_lo"] + c["L_hi"]) / 2
        E = c["E"] if "E" in c else (c["E_lo"] + c["E_hi"]) / 2
        N, live = c["N"], 1 - c["ended"] / (V * E)
        keys = N * L + N * (N + 1) / 2 * (1 + c.get("cross", 0) * (E - 1))
        b = V * (L * row + E * N * (row + qrow))
        f = 4 * D * H_q * V * E * live * keys
        if c["kind"] == "train":  # five products; q, k, v, out, lse, dout in, float32 gradients out
            b += L * 3 * row + E * N * (3 * row + qrow + H_q * D * (es + 4))
            f += 10 * D * H_q * E * live * keys
        return {"bytes": int(b), "flops": int(f)}
    V = c.get("V", 1)
    L = c["L"] if "L" in c else (c["L_lo"] + c["L_hi"]) / 2
    E = c["E"] if "E" in c else (c["E_lo"] + c["E_hi"]) / 2
    n, steps = c["own"] / 2 + 1, c.get("steps", 1)
    live = 1 - c["ended"] / (V * E)
    b = V * (L * row + E * (live * n * row + qrow))
    f = 4 * D * H_q * V * E * live * (L + n)
    if c["kind"] in ("loop", "rope"):
        b += E * 2 * row
    return {"bytes": int(steps * b), "flops": int(steps * f)}


def tolerance(case):
    # Measured against float64 (see exact): float32 steps 3e-7 to 9e-7; bf16 outputs 2.1e-3 to 2.9e-3 (the rounding
    # of the probabilities, of the partial states and of the result); gradients 1.4e-3 to 1.8e-3 (p and ds in bf16);
    # grounding scores 1.2e-7 (float32 sums); aggregation 1.5e-3 to 1.7e-3 (the rounding of the result).
    if case["kind"] == "ground":
        return {"rel": 1e-5, "differ": 0.002}
    if case.get("dtype") == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ---- the same results in 64 bits ----

def _attention(st, c, q, lens, ke, ve):
    """out, lse in float64 for q [SE, N, H_q, D], lens the rows of each stream's cache that are attended."""
    SE, N, H_q, D = q.shape
    H_kv = st["kp"].shape[1]
    G = H_q // H_kv
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.full(q.shape[:3], -math.inf, dtype=torch.float64, device="cuda")
    cup, cue = _cum(st["prefix"]), _cum(st["events"])
    T, cross, decode = c.get("plan", 0), c.get("cross", 0), N == 1
    for v in range(len(st["prefix"])):
        E, L = cue[v + 1] - cue[v], cup[v + 1] - cup[v]
        for g in range(H_kv):
            kp, vp = st["kp"][cup[v]:cup[v + 1], g].double(), st["vp"][cup[v]:cup[v + 1], g].double()
            for f in range(E):
                e = cue[v] + f
                if lens[e] <= 0:
                    continue
                others = [x for x in range(E) if x != f] if cross and not decode else []
                step = max(1, int(1.5e8 // (G * (L + lens[e]))))
                for j0 in range(0, N, step):
                    j1 = min(N, j0 + step)
                    n = lens[e] if decode else min(lens[e], j1)
                    ks, vs = [kp, ke[e, :n, g].double()], [vp, ve[e, :n, g].double()]
                    j = torch.arange(j0, j1, device="cuda")[:, None]
                    t = torch.arange(n, device="cuda")[None]
                    see = [torch.ones((j1 - j0, L), dtype=torch.bool, device="cuda"),
                           (t <= j) | torch.full_like(t, decode, dtype=torch.bool)]
                    if T:
                        p = torch.arange(L, device="cuda") - (L - E * T)
                        see[0] &= (p < 0) | ((p >= f * T) & (p < (f + 1) * T))
                    for x in others:
                        m = min(max(lens[cue[v] + x], 0), j1)
                        ks.append(ke[cue[v] + x, :m, g].double())
                        vs.append(ve[cue[v] + x, :m, g].double())
                        see.append(torch.arange(m, device="cuda")[None] < j)
                    k, val, see = torch.cat(ks), torch.cat(vs), torch.cat(see, 1)
                    rows = q[e, j0:j1, g * G:(g + 1) * G].double().reshape(-1, D)
                    s = rows @ k.t() / math.sqrt(D)
                    s.masked_fill_(~see.repeat_interleave(G, 0), -math.inf)
                    z = torch.logsumexp(s, 1, keepdim=True)
                    o = torch.exp(s.sub_(z)) @ val
                    out[e, j0:j1, g * G:(g + 1) * G] = o.reshape(j1 - j0, G, D)
                    lse[e, j0:j1, g * G:(g + 1) * G] = z.reshape(j1 - j0, G)
    return out, lse


def _gradients(st, q, lens, out, lse):
    """dq, dk_prefix, dv_prefix, dk_event, dv_event in float64 (one video)."""
    E, N, H_q, D = q.shape
    H_kv, L = st["kp"].shape[1], st["kp"].shape[0]
    G, tau = H_q // H_kv, 1.0 / math.sqrt(D)
    z = {n: torch.zeros(st[n].shape, dtype=torch.float64, device="cuda") for n in ("q", "kp", "vp", "ke", "ve")}
    for g in range(H_kv):
        kp, vp = st["kp"][:, g].double(), st["vp"][:, g].double()
        for e in range(E):
            if lens[e] <= 0:
                continue
            n = min(lens[e], N)
            k, v = torch.cat([kp, st["ke"][e, :n, g].double()]), torch.cat([vp, st["ve"][e, :n, g].double()])
            step = max(1, int(1.0e8 // (G * (L + n))))
            for j0 in range(0, N, step):
                at = (e, slice(j0, min(N, j0 + step)), slice(g * G, (g + 1) * G))
                w = min(N, j0 + step) - j0
                rows, do = q[at].double().reshape(-1, D), st["dout"][at].double().reshape(-1, D)
                s = rows @ k.t() * tau
                hide = torch.arange(n, device="cuda")[None] > torch.arange(j0, j0 + w, device="cuda")[:, None]
                s[:, L:].masked_fill_(hide.repeat_interleave(G, 0), -math.inf)
                p = torch.exp(s - lse[at].reshape(-1, 1))
                ds = p * (do @ v.t() - (do * out[at].reshape(-1, D)).sum(1, keepdim=True)) * tau
                z["q"][at] = (ds @ k).reshape(w, G, D)
                dk, dv = ds.t() @ rows, p.t() @ do
                z["kp"][:, g] += dk[:L]
                z["vp"][:, g] += dv[:L]
                z["ke"][e, :n, g] += dk[L:]
                z["ve"][e, :n, g] += dv[L:]
    return tuple(z[n] for n in ("q", "kp", "vp", "ke", "ve"))


def _append(st, c, s, lens, ke, ve, kn):
    """The live streams' new rows in the caches; the counts after it."""
    after = []
    for e, n in enumerate(lens):
        live = st["live_host"][e]
        if live and n < st["cap"]:
            ke[e, n], ve[e, n] = kn[e], st["vn"][s, e]
            n += 1
        after.append(n if live else 0)
    return after


def _rotate(x, pos):
    """Rotate-half at position pos[e] of x [SE, heads, D], rounded to x's type."""
    h = x.shape[-1] // 2
    freq = torch.tensor(THETA, dtype=torch.float64, device="cuda") ** (
        -2.0 * torch.arange(h, device="cuda", dtype=torch.float64) / (2 * h))
    ang = pos.double()[:, None, None] * freq
    a, b = x[..., :h].double(), x[..., h:].double()
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1).to(x.dtype)


def exact(case, seed):
    c, st = case, _inputs(case, seed)
    if c["kind"] == "ground":
        sim, cu = st["g"].double() @ st["p"].double().t(), st["cu_host"]
        scores = torch.stack([sim[:, cu[s]:cu[s + 1]].sum(1) for s in range(c["S"])], 1)
        return scores, (scores > 0.5 * scores.max(1, keepdim=True).values).to(torch.uint8)
    if c["kind"] == "aggregate":
        cu, weights = st["cu_host"], None
        w = torch.ones(c["N"], dtype=torch.float64, device="cuda")
        if c["mode"] == "learned":
            w = st["scores"].double()
        elif c["mode"] == "attention":
            G = c["H_q"] // c["H_kv"]
            s = torch.stack([st["k"][:, h // G].double() @ st["q"][h].double() for h in range(c["H_q"])])
            w = weights = torch.exp(s / math.sqrt(c["D"]) - st["lse"].double()[:, None]).mean(0)
        out = st["g"].double()
        for i in range(c["K"]):
            at = [n for s in range(c["S"]) if st["sal"][i, s] for n in range(cu[s], cu[s + 1])]
            if at:
                at = torch.tensor(at, device="cuda")
                out[i] += (w[at] @ st["x"][at].double()) / w[at].sum()
        return out, weights
    lens = st["own"]
    if c["kind"] in ("step", "ragged"):
        out, lse = _attention(st, c, st["q"][:, None], lens, st["ke"], st["ve"])
        return out[:, 0], lse[:, 0]
    if c["kind"] == "loop":
        outs, lses = [], []
        for s in range(c["steps"]):
            lens = _append(st, c, s, lens, st["ke"], st["ve"], st["kn"][s])
            out, lse = _attention(st, c, st["qs"][s][:, None], lens, st["ke"], st["ve"])
            outs.append(out[:, 0])
            lses.append(lse[:, 0])
        return {"out": outs, "lse": lses, "lens": _ints(lens), "k": st["ke"], "v": st["ve"]}
    if c["kind"] == "rope":
        pos = st["lens"] + st["prefix"][0]
        live = st["live"].bool()[:, None, None]
        q = torch.where(live, _rotate(st["qs"][0], pos), st["qs"][0])
        lens = _append(st, c, 0, lens, st["ke"], st["ve"], _rotate(st["kn"][0], pos))
        out, lse = _attention(st, c, q[:, None], lens, st["ke"], st["ve"])
        return {"out": out[:, 0], "lse": lse[:, 0], "q": q, "lens": _ints(lens), "k": st["ke"], "v": st["ve"]}
    out, lse = _attention(st, c, st["q"], lens, st["ke"], st["ve"])
    if c["kind"] != "train":
        return out, lse
    return (out, lse, *_gradients(st, st["q"], lens, out, lse))
