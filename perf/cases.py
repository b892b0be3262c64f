"""The work that programs have this library do, as cases that can be timed and checked.

A case is a dict of plain values.  prepare() makes what a serving program holds before the call (caches at their
budget, the next tokens, weights, the context), run() is one pass through the public calls, exact() the same result
in 64-bit arithmetic by plain torch.  Five kinds of work ("op"):

  step    one decode step: a token per (layer, KV head) list enters, every entry is rescored, the cache is evicted
          down to the global budget and attended.  Layouts: "ragged" (a new compact cache every step), "inplace"
          (compacted inside the cache), "paged".
  chunk   one chunk of a chunked prefill: many tokens enter, rescoring, selection, eviction; no attention.
  first   the first eviction behind a long prefill: score, select, compact and attend (or move to pages).
  attn    one token's attention, called layer by layer as a model's forward pass calls it, hard or soft
          (the form the gates are trained with, together with the occupancy sum of its capacity loss).
  gate    log beta of new tokens: one token per sequence, a batch or short chunk, a prefill chunk.
"""
import math

import torch

import paper_2605_09649_amd as kv

RING = 64      # decode steps whose inputs differ; longer runs come back to the first
ROOM = 64      # free slots behind a segment for the in-place step, evened out after as many steps

_LLAMA = dict(layers=32, kv_heads=8, q_heads=32, head_dim=128)


def listed():
    return [
        # a small model's decode step: nothing but latency and launches
        dict(name="step_tiny", op="step", layout="ragged", seqs=1, layers=4, kv_heads=4, q_heads=8, head_dim=64,
             tokens=2048, per_list=64, horizon=1, z_mean=3.0, layer_std=0.0, evidence=0.0, visual=0.0),
        # long-context decode of one sequence (128 K tokens, 6.25 % kept): the benchmark's step
        dict(name="step_long", op="step", layout="ragged", seqs=1, **_LLAMA, tokens=131072, per_list=8192, horizon=1,
             z_mean=3.5, layer_std=0.0, evidence=0.02, visual=0.0),
        # vision-language decode of two sequences, seven query heads per KV head, lookahead horizon 2
        dict(name="step_vlm", op="step", layout="ragged", seqs=2, layers=28, kv_heads=4, q_heads=28, head_dim=128,
             tokens=20480, per_list=2048, horizon=2, z_mean=3.0, layer_std=0.0, evidence=0.0, visual=0.2),
        # a serving batch: sixteen sequences of different lengths
        dict(name="step_batch16", op="step", layout="ragged", seqs=16, **_LLAMA, tokens=16384, per_list=2048, horizon=1,
             z_mean=3.0, layer_std=0.0, evidence=0.0, visual=0.0),
        # 32 K tokens, 12.5 % kept, compacted inside the cache; layers compete unevenly
        dict(name="step_inplace", op="step", layout="inplace", seqs=1, **_LLAMA, tokens=32768, per_list=4096, horizon=1,
             z_mean=3.0, layer_std=0.5, evidence=0.0, visual=0.0),
        # the long-context step on pages
        dict(name="step_paged", op="step", layout="paged", seqs=1, **_LLAMA, tokens=131072, per_list=8192, horizon=1,
             z_mean=3.5, layer_std=0.0, evidence=0.02, visual=0.0),
        # multi-turn serving: a 4096-token chunk of four conversations that are at their budget
        dict(name="chunk_multiturn", op="chunk", layout="ragged", seqs=4, **_LLAMA, tokens=24576, per_list=8192,
             n_new=4096, horizon=1, z_mean=3.0, layer_std=0.0, evidence=0.0, visual=0.0),
        # the first eviction behind a 128 K prefill
        dict(name="first_long", op="first", layout="ragged", seqs=1, **_LLAMA, tokens=131072, per_list=8192, horizon=1,
             z_mean=3.5, layer_std=0.0, evidence=0.02, visual=0.0),
        # attention of one token over an evicted cache, a call per layer
        dict(name="attn_layers", op="attn", layout="ragged", soft=False, seqs=1, **_LLAMA, tokens=32768, per_list=4096,
             horizon=1, z_mean=3.0, layer_std=0.5, evidence=0.0, visual=0.0),
        # the gates of one new token, of a batch (or short chunk) of 64, of a prefill chunk; weights prepared once
        dict(name="gate_token", op="gate", n_tok=1, layers=32, kv_heads=8, d_model=4096, d_g=512, d_p=128, horizon=1,
             prepared=True),
        dict(name="gate_batch64", op="gate", n_tok=64, layers=32, kv_heads=8, d_model=4096, d_g=512, d_p=128, horizon=2,
             prepared=True),
        dict(name="gate_prefill", op="gate", n_tok=4096, layers=32, kv_heads=8, d_model=4096, d_g=512, d_p=128, horizon=1,
             prepared=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "chunk", "first", "attn", "attn", "gate", "gate", "gate"])
    if op == "gate":
        n_tok = _log_int(rng, 1, 4096)
        return dict(op="gate", n_tok=n_tok, layers=_log_int(rng, 2, 32), kv_heads=rng.randint(1, 8),
                    d_model=256 * rng.randint(4, 16), d_g=64 * rng.choice([1, 2, 3, 4, 4, 6, 8, 8, 8]),
                    d_p=rng.choice([32, 64, 100, 128]), horizon=rng.choice([0, 1, 2]), prepared=rng.random() < 0.75)
    layers, kv_heads, group = _log_int(rng, 2, 36), rng.randint(1, 8), rng.randint(1, 8)
    head_dim = rng.choice([64, 128, 128])
    seqs = rng.choice([1, 1, 1, 2, 3, 8]) if op in ("step", "chunk") else rng.choice([1, 1, 2])
    most = {"step": 4_000_000, "chunk": 3_000_000, "first": 400_000, "attn": 3_000_000}[op]
    lists = seqs * layers * kv_heads
    per_list = _log_int(rng, 40, min(16384, max(60, most // lists)))
    tokens = int(per_list * rng.choice([3.0, 8.0, 16.0]) * rng.uniform(0.8, 1.2)) + rng.randint(1, 9)
    case = dict(op=op, layout=rng.choice(["ragged", "ragged", "inplace", "paged"]) if op == "step" else
                rng.choice(["ragged", "ragged", "paged"]), seqs=seqs, layers=layers, kv_heads=kv_heads,
                q_heads=kv_heads * group, head_dim=head_dim, tokens=tokens, per_list=per_list,
                horizon=rng.choice([1, 1, 2]), z_mean=rng.choice([3.0, 3.5]), layer_std=rng.choice([0.0, 0.5]),
                evidence=rng.choice([0.0, 0.02]), visual=rng.choice([0.0, 0.2]))
    if op == "chunk":
        case["n_new"] = max(1, min(4096, int(per_list * rng.uniform(0.1, 1.0))))
    if op == "attn":
        case["soft"] = case["layout"] == "ragged" and rng.random() < 0.4
    return case


# ---- inputs --------------------------------------------------------------------------------------------------------

def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + salt) % (1 << 62))


def _log_beta(z):
    return (-torch.log1p(torch.exp(-z))).float()


def _log_tail(lb, horizon):
    """log(sum_{k < horizon} beta^k), what a horizon other than 1 adds to a token's constants."""
    total, term, beta = 0.0, 1.0, torch.exp(lb.double())
    for _ in range(horizon):
        total, term = total + term, term * beta
    return torch.log(total).float()


def _score(lb, pos, now, horizon):
    """The score of the method in fp32: one multiply, or one fused multiply-add (exact in 64 bits before it is rounded)."""
    age = (now + 1 - pos).float()
    if horizon == 1:
        return age * lb
    return (age.double() * lb.double() + _log_tail(lb, horizon).double()).float()


def _first_b(score, budget):
    """Mask of the `budget` largest scores of one sequence; the earlier entry wins among equals (storage order)."""
    keep = torch.zeros(score.numel(), dtype=torch.bool, device=score.device)
    keep[torch.sort(score, descending=True, stable=True).indices[:budget]] = True
    return keep


def _prefilled(case, seed, seq):
    """log beta [lists of a sequence][tokens of this sequence]: gate logits with layers, near-permanent tokens and a
    block of visual tokens as the case says.  A batch's sequences are of different lengths."""
    g = _gen(seed, 100 + seq)
    L, H = case["layers"], case["kv_heads"]
    T = case["tokens"] if seq == 0 else case["tokens"] - (seq * 2654435761 % 1000) * (case["tokens"] - case["per_list"]) // 1500
    z = torch.randn(L * H, T, generator=g, device="cuda", dtype=torch.float64) * 1.5 + case["z_mean"]
    if case["layer_std"]:
        z += (torch.randn(L, generator=g, device="cuda", dtype=torch.float64) * case["layer_std"]).repeat_interleave(H)[:, None]
    if case["visual"]:
        a, b = T // 20, T // 20 + int(T * case["visual"])
        z[:, a:b] = torch.randn(L * H, b - a, generator=g, device="cuda", dtype=torch.float64) * 2.0 + 1.5
    if case["evidence"]:
        there = torch.rand(T, generator=g, device="cuda") < case["evidence"]
        z = torch.where(there[None], torch.randn(L * H, T, generator=g, device="cuda", dtype=torch.float64) + 8.0, z)
    return _log_beta(z)


def _lists(case, seed, evicted):
    """(log beta, pos, length of every list, newest position of every sequence), lists one after the other; `evicted`:
    as the eviction at the end of the prefill left them."""
    lbs, poss, lens, now = [], [], [], []
    for seq in range(case["seqs"]):
        lb = _prefilled(case, seed, seq)
        n, T = lb.shape
        pos = torch.arange(T, dtype=torch.int32, device="cuda").expand(n, T)
        now.append(T - 1)
        if evicted:
            keep = _first_b(_score(lb, pos, T - 1, case["horizon"]).reshape(-1), case["per_list"] * n).view(n, T)
            lbs.append(lb[keep])
            poss.append(pos[keep])
            lens.append(keep.sum(1))
        else:
            lbs.append(lb.reshape(-1))
            poss.append(pos.reshape(-1))
            lens.append(torch.full((n,), T, device="cuda"))
    return torch.cat(lbs), torch.cat(poss), torch.cat(lens), now


def _rows(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _cache(case, seed, room, evicted=True):
    """A ragged cache with `room` free slots behind every list, as a dict of tensors, and the newest positions."""
    lb, pos, lens, now = _lists(case, seed, evicted)
    nseg, n = lens.numel(), lb.numel()
    start = torch.cumsum(lens + room, 0) - (lens + room)
    cap = n + nseg * room
    at = torch.arange(n, device="cuda") + torch.repeat_interleave(torch.arange(nseg, device="cuda") * room, lens)
    c = dict(log_beta=torch.zeros(cap, device="cuda"), pos=torch.zeros(cap, dtype=torch.int32, device="cuda"),
             seg_start=start.long(), seg_len=lens.int())
    c["log_beta"][at], c["pos"][at] = lb, pos
    if case["horizon"] != 1:
        c["log_tail"] = torch.zeros(cap, device="cuda")
        c["log_tail"][at] = _log_tail(lb, case["horizon"])
    del at, lb, pos
    g = _gen(seed, 1)
    c["k"], c["v"] = _rows(g, cap, case["head_dim"]), _rows(g, cap, case["head_dim"])
    return c, now


def _next_tokens(case, seed, n_new, ring):
    """`ring` calls' worth of new tokens and queries."""
    nseg = case["seqs"] * case["layers"] * case["kv_heads"]
    g, D = _gen(seed, 2), case["head_dim"]
    got = []
    for _ in range(ring):
        d = dict(k=_rows(g, nseg, n_new, D), v=_rows(g, nseg, n_new, D),
                 lb=_log_beta(torch.randn(nseg, n_new, generator=g, device="cuda", dtype=torch.float64) * 1.5 + case["z_mean"]),
                 q=_rows(g, case["seqs"], case["layers"], case["q_heads"], D))
        d["lt"] = _log_tail(d["lb"], case["horizon"]) if case["horizon"] != 1 else None
        got.append(d)
    return got


def _clock(case, now, n_new):
    """One int32 buffer that holds the new tokens' positions of every list and each sequence's newest position, so that
    one addition moves a decode loop on."""
    per = case["layers"] * case["kv_heads"]
    ends = torch.tensor(now, dtype=torch.int32, device="cuda")
    new = (ends[:, None] - n_new + 1 + torch.arange(n_new, dtype=torch.int32, device="cuda")).repeat_interleave(per, 0)
    buf = torch.cat([new.reshape(-1), ends])
    return buf, buf[:new.numel()], buf[new.numel():]


# ---- prepare and run -----------------------------------------------------------------------------------------------

def prepare(case, seed):
    s = _prepare_gate(case, seed) if case["op"] == "gate" else _prepare_cache(case, seed)
    s["case"] = case
    return s


def _prepare_gate(case, seed):
    d = _gate_inputs(case, seed)
    gate = kv.Gate(d["w1"], d["c1"], d["w2"], d["c2"], d["w_g"], d["b_g"])
    L, H, n = case["layers"], case["kv_heads"], case["n_tok"]
    ctx = kv.Context(1, L, H, H, 128, 1024)
    s = dict(ctx=ctx, gate=gate, x=d["x"], prepared=None,
             scratch=torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n, L), dtype=torch.uint8, device="cuda"),
             lb=torch.zeros(n, L, H, device="cuda"), lt=torch.zeros(n, L, H, device="cuda") if case["horizon"] != 1 else None)
    if case["prepared"]:
        s["prepared"] = torch.empty(kv.kvtrim_gate_prepared_bytes(gate, L, H), dtype=torch.uint8, device="cuda")
        kv.kvtrim_gate_prepare(ctx, gate, s["prepared"])
    return s


def _gate_inputs(case, seed):
    """Weights and token representations with the spreads that give gate logits around 3.5 +- 1.5."""
    g = _gen(seed, 3)
    L, H, dm, dg, dp = (case[n] for n in ("layers", "kv_heads", "d_model", "d_g", "d_p"))

    def rn(*shape):
        return torch.randn(*shape, generator=g, device="cuda")
    return dict(w1=(rn(L, dg, dm) / dm ** 0.5).bfloat16(), c1=rn(L, dg) * 0.1, w2=(rn(L, H, dp, dg) / dg ** 0.5).bfloat16(),
                c2=rn(L, H, dp) * 0.1, w_g=rn(dp) * 2.5 / dp ** 0.5, b_g=3.5, x=_rows(g, L, case["n_tok"], dm))


def _prepare_cache(case, seed):
    S, L, H, Hq, D = (case[n] for n in ("seqs", "layers", "kv_heads", "q_heads", "head_dim"))
    op, layout, tail = case["op"], case["layout"], case["horizon"] != 1
    nseg, n_new = S * L * H, case.get("n_new", 1)
    room = {"step": ROOM if layout == "inplace" else 1, "chunk": n_new}.get(op, 0)
    if layout == "paged":
        room = 0
    c, now = _cache(case, seed, room, evicted=op != "first")
    src = kv.Cache(**c)
    s = dict(i=0, nseg=nseg, per=L * H, room=room, cur=src, scale=D ** -0.5,
             budget=torch.full((S,), case["per_list"] * L * H, dtype=torch.int64, device="cuda"),
             out=torch.zeros(S, L, Hq, D, device="cuda"), lse=torch.zeros(S, L, Hq, device="cuda"),
             kept=torch.zeros(nseg, dtype=torch.int32, device="cuda"), thr=torch.zeros(S, dtype=torch.int32, device="cuda"))
    kept_rows = case["per_list"] * nseg
    s["ring"] = _next_tokens(case, seed, n_new, {"step": RING, "chunk": 2}.get(op, 1))
    s["clock"], s["pos_new"], s["now"] = _clock(case, now, n_new)
    slots = src.cap
    if layout == "paged":
        # a pool with a quarter more pages than a dense packing needs, three more per list and the chunk's own
        rows = kept_rows + (n_new * nseg if op == "chunk" else 0)
        pages = int(1.25 * rows / kv.PAGE_SIZE) + 3 * nseg + 64
        longest = int(src.seg_len.max()) + n_new
        s["pages"] = kv.PagedCache(nseg, D, pages, 2 * (longest // kv.PAGE_SIZE) + 32, with_tail=tail)
        slots = max(slots, s["pages"].slots)
    elif op != "attn":
        s["nxt"] = kv.Cache.empty(nseg, D, kept_rows + nseg * room, with_tail=tail)
    s["score"] = torch.zeros(slots, device="cuda")
    s["keep"] = torch.zeros(slots, dtype=torch.uint8, device="cuda")
    s["ctx"] = ctx = kv.Context(S, L, H, Hq, D, slots)
    if op == "attn":
        s["occ"] = torch.zeros(S, dtype=torch.float64, device="cuda")
    if layout == "paged" and op != "first":
        s["keep"].fill_(1)
        kv.kvtrim_paged_build(ctx, src, s["keep"][:src.cap], src.seg_len, s["pages"])
        s["cur"] = src = None
    if op == "step":
        # the context has seen an eviction of this cache, as in a decode loop
        if layout == "paged":
            kv.kvtrim_paged_score_select(ctx, s["pages"], s["now"], s["budget"] - s["per"], s["score"], s["keep"], s["kept"], s["thr"])
        else:
            kv.kvtrim_score_select(ctx, src, s["now"], s["budget"] - s["per"], s["score"], s["keep"], s["kept"], s["thr"])
    return s


def run(s):
    return {"gate": _run_gate, "step": _run_step, "chunk": _run_chunk, "first": _run_first, "attn": _run_attn}[s["case"]["op"]](s)


def _run_gate(s):
    c = s["case"]
    if s["prepared"] is None:
        kv.kvtrim_gate_forward(s["ctx"], s["gate"], s["x"], c["n_tok"], 0, c["layers"], c["horizon"], s["scratch"], s["lb"], s["lt"])
    else:
        kv.kvtrim_gate_forward_prepared(s["ctx"], s["gate"], s["prepared"], s["x"], c["n_tok"], 0, c["layers"], c["horizon"],
                                        s["scratch"], s["lb"], s["lt"])
    return {"log_beta": s["lb"]} if s["lt"] is None else {"log_beta": s["lb"], "log_tail": s["lt"]}


def _entries(c):
    return {n: getattr(c, n) for n in ("k", "v", "log_beta", "pos", "log_tail", "seg_start", "seg_len") if getattr(c, n) is not None}


def _run_step(s):
    c, i = s["case"], s["i"]
    new = s["ring"][i % RING]
    s["i"] = i + 1
    s["clock"].add_(1)
    if c["layout"] == "paged":
        # where a row sits in the pool depends on the order in which pages were freed: the results are the step's outputs
        kv.kvtrim_paged_decode_step(s["ctx"], s["pages"], new["k"], new["v"], new["lb"], s["pos_new"], s["now"], s["budget"],
                                    s["score"], s["keep"], s["kept"], new["q"], 0, c["layers"], s["scale"], s["out"], s["lse"],
                                    s["thr"], new["lt"], s["per"])
        return {"out": s["out"], "lse": s["lse"], "kept": s["kept"], "thr": s["thr"], "live": s["pages"].seg_live}
    cur, nxt = s["cur"], s["nxt"]
    if c["layout"] == "inplace" and i % ROOM != ROOM - 1:
        kv.kvtrim_decode_step_inplace(s["ctx"], cur, new["k"], new["v"], new["lb"], s["pos_new"], 1, s["now"], s["budget"],
                                      s["score"], s["keep"], s["kept"], nxt, new["q"], 0, c["layers"], s["scale"], s["out"],
                                      s["lse"], s["thr"], new["lt"], s["per"])
        return {"out": s["out"], "lse": s["lse"], "kept": s["kept"], "thr": s["thr"], "cache": _entries(cur)}
    kv.kvtrim_decode_step(s["ctx"], cur, new["k"], new["v"], new["lb"], s["pos_new"], 1, s["now"], s["budget"], s["score"],
                          s["keep"], s["kept"], nxt, s["room"], new["q"], 0, c["layers"], s["scale"], s["out"], s["lse"],
                          s["thr"], new["lt"], s["per"])
    s["cur"], s["nxt"] = nxt, cur
    return {"out": s["out"], "lse": s["lse"], "kept": s["kept"], "thr": s["thr"], "cache": _entries(nxt)}


def _run_chunk(s):
    c, i = s["case"], s["i"]
    n, new = c["n_new"], s["ring"][i % 2]
    s["i"] = i + 1
    s["clock"].add_(n)
    if c["layout"] == "paged":
        p = s["pages"]
        kv.kvtrim_paged_append(s["ctx"], p, new["k"], new["v"], new["lb"], s["pos_new"], new["lt"], n)
        kv.kvtrim_paged_score_select(s["ctx"], p, s["now"], s["budget"], s["score"], s["keep"], s["kept"], s["thr"])
        kv.kvtrim_paged_evict(s["ctx"], p, s["keep"])
        return {"kept": s["kept"], "thr": s["thr"], "live": p.seg_live}
    cur, nxt = s["cur"], s["nxt"]
    kv.kvtrim_append_compact(s["ctx"], cur, new["k"], new["v"], new["lb"], s["pos_new"], n, s["now"], s["budget"], s["score"],
                             s["keep"], s["kept"], nxt, n, s["thr"], new["lt"])
    s["cur"], s["nxt"] = nxt, cur
    return {"kept": s["kept"], "thr": s["thr"], "cache": _entries(nxt)}


def _run_first(s):
    c, src, q = s["case"], s["cur"], s["ring"][0]["q"]
    kv.kvtrim_score_select(s["ctx"], src, s["now"], s["budget"], s["score"], s["keep"], s["kept"], s["thr"])
    got = {"out": s["out"], "lse": s["lse"], "kept": s["kept"], "thr": s["thr"]}
    if c["layout"] == "paged":
        p = s["pages"]
        kv.kvtrim_paged_build(s["ctx"], src, s["keep"], s["kept"], p)
        kv.kvtrim_paged_attn(s["ctx"], p, q, 0, c["layers"], s["scale"], s["out"], s["lse"])
        return dict(got, live=p.seg_live)
    kv.kvtrim_compact_attn(s["ctx"], src, s["keep"], s["kept"], s["nxt"], s["room"], q, 0, c["layers"], s["scale"], s["out"], s["lse"])
    return dict(got, score=s["score"], keep=s["keep"], cache=_entries(s["nxt"]))


def _run_attn(s):
    c, q = s["case"], s["ring"][0]["q"]
    for layer in range(c["layers"]):
        if c["layout"] == "paged":
            kv.kvtrim_paged_attn(s["ctx"], s["pages"], q, layer, layer + 1, s["scale"], s["out"], s["lse"])
        elif c["soft"]:
            kv.kvtrim_decode_attn_soft(s["ctx"], s["cur"], q, s["now"], layer, layer + 1, s["scale"], s["out"], s["lse"])
        else:
            kv.kvtrim_decode_attn(s["ctx"], s["cur"], q, layer, layer + 1, s["scale"], s["out"], s["lse"])
    if not c["soft"]:
        return {"out": s["out"], "lse": s["lse"]}
    kv.kvtrim_occupancy(s["ctx"], s["cur"], s["now"], s["occ"])
    return {"out": s["out"], "lse": s["lse"], "occ": s["occ"]}


# ---- what a pass cannot do without, and what it must give -----------------------------------------------------------

def work(case):
    if case["op"] == "gate":
        n, L, H, dm, dg, dp = (case[k] for k in ("n_tok", "layers", "kv_heads", "d_model", "d_g", "d_p"))
        second = L * H * (4 * dg if case["prepared"] else 2 * dg * dp)      # folded vectors, or the second layer's weights
        return {"bytes": 2 * L * dg * dm + second + 2 * n * L * dm + 4 * n * L * H * (1 if case["horizon"] == 1 else 2),
                "flops": 2.0 * n * L * dg * (dm + H)}
    nseg, D, tail = case["seqs"] * case["layers"] * case["kv_heads"], case["head_dim"], 4 * (case["horizon"] != 1)
    heads = case["seqs"] * case["layers"] * case["q_heads"]
    kept, n_new = nseg * case["per_list"], case.get("n_new", 1)
    row, attend = 4 * D + 8 + tail, 6 * D * heads
    score = 8 + tail + 4 + 1                                                 # constants in, score and mask out
    flops = 4.0 * D * kept * heads / nseg
    if case["op"] == "attn":
        return {"bytes": kept * (4 * D + 8 * case["soft"]) + attend, "flops": flops}
    if case["op"] == "chunk":
        # every survivor is read and written once; on pages only the new rows are
        rows = 2 * kept * row if case["layout"] == "ragged" else 2 * nseg * n_new * row
        return {"bytes": rows + (kept + nseg * n_new) * score, "flops": 2.0 * (kept + nseg * n_new)}
    if case["op"] == "first":
        n = sum(_prefill_len(case, seq) for seq in range(case["seqs"])) * (nseg // case["seqs"])
        return {"bytes": n * score + 2 * kept * row + attend, "flops": flops}
    # a decode step: out of place every survivor is written as well (in place the rows behind an eviction, which depend on it)
    rows = kept * row * 2 if case["layout"] == "ragged" else kept * 4 * D + 2 * nseg * row
    return {"bytes": rows + (kept + nseg) * score + attend, "flops": flops}


def _prefill_len(case, seq):
    return case["tokens"] if seq == 0 else case["tokens"] - (seq * 2654435761 % 1000) * (case["tokens"] - case["per_list"]) // 1500


def tolerance(case):
    # Scores, selections and moved rows come out bit for bit.  Attention: probabilities enter the second product with 16
    # mantissa bits or more, everything else is fp32 (1.5e-6 to 2.1e-6 off the 64-bit result).  Gate: bf16 products summed
    # in fp32 over up to 4096 terms, u kept to 16 bits or more (1e-7 to 6e-7 off).
    if case["op"] == "chunk":
        return "exact"
    if case["op"] == "gate":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 1e-5, "max": 1e-4}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------

def exact(case, seed):
    if case["op"] == "gate":
        return _exact_gate(case, seed)
    if case["op"] == "chunk":
        return None                                     # rows and whole numbers, compared bit for bit
    S, L, H, Hq, D = (case[n] for n in ("seqs", "layers", "kv_heads", "q_heads", "head_dim"))
    op, layout, G = case["op"], case["layout"], Hq // H
    room = (ROOM if layout == "inplace" else 1) if op == "step" and layout != "paged" else 0
    c, now = _cache(case, seed, room, evicted=op != "first")
    new = _next_tokens(case, seed, 1, 1)[0]
    starts, lens = c["seg_start"].tolist(), c["seg_len"].tolist()
    out = torch.zeros(S, L, Hq, D, dtype=torch.float64, device="cuda")
    lse = torch.full((S, L, Hq), -math.inf, dtype=torch.float64, device="cuda")
    occ = torch.zeros(S, dtype=torch.float64, device="cuda")
    per = L * H
    for seq in range(S):
        spans = [(starts[g], lens[g]) for g in range(seq * per, (seq + 1) * per)]
        entered = op == "step"
        t = now[seq] + entered
        keep = None
        if op != "attn":
            lb, pos = [], []
            for g, (a, n) in enumerate(spans):
                lb += [c["log_beta"][a:a + n]] + ([new["lb"][seq * per + g]] if entered else [])
                pos += [c["pos"][a:a + n]] + ([torch.full((1,), t, dtype=torch.int32, device="cuda")] if entered else [])
            keep = _first_b(_score(torch.cat(lb), torch.cat(pos), t, case["horizon"]), case["per_list"] * per)
            del lb, pos
        at = 0
        for g, (a, n) in enumerate(spans):
            k, v, lb, pos = (c[x][a:a + n] for x in ("k", "v", "log_beta", "pos"))
            if keep is not None:
                m = keep[at:at + n + entered]
                at += n + entered
                k, v = k[m[:n]], v[m[:n]]
                if entered:
                    i = seq * per + g
                    k, v = torch.cat([k, new["k"][i][m[n:]]]), torch.cat([v, new["v"][i][m[n:]]])
            if k.shape[0] == 0:
                continue
            layer, head = g // H, g % H
            z = new["q"][seq, layer, head * G:(head + 1) * G].double() @ k.double().t() * D ** -0.5
            if op == "attn" and case["soft"]:
                bias = (t - pos).double() * lb.double()
                z = z + bias
                occ[seq] += torch.exp(bias).sum()
            lse[seq, layer, head * G:(head + 1) * G] = torch.logsumexp(z, 1)
            out[seq, layer, head * G:(head + 1) * G] = torch.softmax(z, 1) @ v.double()
    got = {"out": out, "lse": lse}
    if op == "attn":
        return dict(got, occ=occ) if case["soft"] else got
    got.update(kept=None, thr=None)
    if layout == "paged":
        return dict(got, live=None)
    return dict(got, score=None, keep=None, cache=None) if op == "first" else dict(got, cache=None)


def _exact_gate(case, seed):
    d = _gate_inputs(case, seed)
    L, H, n = case["layers"], case["kv_heads"], case["n_tok"]
    lb = torch.zeros(n, L, H, dtype=torch.float64, device="cuda")
    for layer in range(L):
        u = d["x"][layer].double() @ d["w1"][layer].double().t() + d["c1"][layer].double()
        u = u * torch.sigmoid(u)
        for h in range(H):
            p = u @ d["w2"][layer, h].double().t() + d["c2"][layer, h].double()
            lb[:, layer, h] = torch.nn.functional.logsigmoid(p @ d["w_g"].double() + d["b_g"])
    if case["horizon"] == 1:
        return {"log_beta": lb}
    beta = torch.exp(lb)
    tail = -torch.log1p(-beta) if case["horizon"] == 0 else torch.log(sum(beta ** k for k in range(case["horizon"])))
    return {"log_beta": lb, "log_tail": tail}
