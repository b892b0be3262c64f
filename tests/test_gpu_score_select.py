"""GPU parity of kvtrim_score_select (stages 1 + 2 in one call) against the oracle's score + full sort:
scores, mask, per-segment counts and threshold key bit for bit, in both of its forms - the radix passes with the
score fused into the first (evict_hint 0) and the decode-step form (candidate list + ranking, with its single-block
fallback) - through whole decode loops (the rest of the step runs too, so a wrong mask would also show in the
compacted cache and the attention)."""
import numpy as np
import pytest
import torch

import kvtrim_inputs as ki
import oracle
import paper_2605_09649_amd as kv
from harness import run_steps_both
from helpers import host_cache, live_mask

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ATTN_TOL = 5e-3


def check(results, what=""):
    for i, r in enumerate(results):
        assert r["status"] == 0, (what, i, r)
        assert r["score_equal"], (what, i, "score bits differ")
        assert r["keep_equal"], (what, i, "selection differs")
        assert r["cache_equal"], (what, i, "compacted cache differs")
        assert r["attn_err"] <= ATTN_TOL and r["lse_err"] <= 2e-3 and r["lse_inf_equal"], (what, i, r)


def wl(S, L, H, G, D):
    return ki.Workload("t", 0, S, L, H, G * H, D, (0,) * S, (0,) * S, 1, 3.0, 1.5)


@pytest.mark.parametrize("hint", [0, 16])
def test_tiny_workload_full_loop(hint):
    w = ki.workload("tiny")                                       # 16 segments: 16 evictions per step once at the budget
    res = run_steps_both(w, steps=16, budget=w.budget, device=DEV, fused=True, hint=hint)
    check(res, hint)
    listed, fallback = res[-1]["path_counts"]
    if hint:
        # the first call has no bound yet (single-block select), the second starts from the bound that one left;
        # from then on the candidate list must carry every step: scores only decay and 16 entries go per step
        assert fallback <= 2 and listed >= 14, (listed, fallback)
    else:
        assert listed == 0 and fallback == 0


@pytest.mark.parametrize("name,prefill,steps", [("llama", 700, 6), ("long", 900, 6), ("vlm", 640, 6), ("multiturn", 600, 4)])
def test_scaled_down_workloads_decode_step_form(name, prefill, steps):
    w = ki.workload(name, prefill=prefill)
    res = run_steps_both(w, steps=steps, budget=w.budget, device=DEV, fused=True, hint=w.n_layers * w.n_kv_heads)
    check(res, name)
    listed, fallback = res[-1]["path_counts"]
    assert listed >= (steps - 2) * w.n_seq - fallback and fallback <= 2 * w.n_seq, (listed, fallback)


def test_radix_passes_leave_the_bound_the_decode_step_form_starts_from():
    # first eviction from the prefill through the radix passes (hint 0), decode steps after it with a hint: the
    # first of them already finds its candidates listed, no sequence ever takes the single-block fallback
    for name, prefill in (("long", 2000), ("vlm", 900)):
        w = ki.workload(name, prefill=prefill)
        per_seq = w.n_layers * w.n_kv_heads
        res = run_steps_both(w, steps=6, budget=w.budget, device=DEV, fused=True, hint=[0, per_seq])
        check(res, name)
        listed, fallback = res[-1]["path_counts"]
        assert fallback == 0 and listed == 5 * w.n_seq, (name, listed, fallback)


@pytest.mark.parametrize("horizon", [2, 0])
def test_lookahead_horizon_tail_enters_the_fused_score(horizon):
    w = ki.workload("tiny", prefill=500)
    for hint in (0, 16):
        check(run_steps_both(w, steps=5, budget=w.budget, device=DEV, fused=True, hint=hint, horizon=horizon), (horizon, hint))


@pytest.mark.parametrize("hint", [0, 4, 60])
@pytest.mark.parametrize("S,L,H,G,D", [(1, 2, 2, 1, 128), (2, 2, 1, 7, 128), (3, 1, 2, 3, 64), (1, 2, 1, 4, 128)])
def test_ragged_segments_spanning_several_blocks(S, L, H, G, D, hint):
    w = wl(S, L, H, G, D)
    rng = np.random.default_rng(S * 1000 + G * 10 + D)
    seg_len = rng.integers(0, 20000, w.nseg)                      # more than one 8192-entry share per segment
    seg_len[rng.integers(0, w.nseg)] = 0
    seg_len[rng.integers(0, w.nseg)] = 8192 * 2 + 1
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=G)
    per_seq = [int(seg_len[s * L * H:(s + 1) * L * H].sum()) for s in range(S)]
    budget = [max(1, n // 3) for n in per_seq]
    check(run_steps_both(w, steps=4, budget=budget, device=DEV, cache_dict=c, now0=now.numpy(), fused=True, hint=hint))


def test_budget_changes_from_step_to_step_and_nothing_to_evict():
    # budget far above the count (nothing evicted, the threshold is the lowest key), then at the count, then a
    # drop to a third (many evictions: the list cannot hold them, the fallback runs), then steady, then zero
    w = wl(2, 2, 2, 2, 64)
    rng = np.random.default_rng(8)
    seg_len = rng.integers(50, 900, w.nseg)
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=3)
    n0 = [int(seg_len[:4].sum()), int(seg_len[4:].sum())]
    steps = [[10 ** 9, 10 ** 9], [n0[0] + 8, n0[1]], [n0[0] // 3, n0[1] - 5], [n0[0] // 3, n0[1] - 5], [n0[0] // 3, n0[1] - 5],
             [n0[0] // 3 + 2, n0[1] - 9], [0, n0[1] - 9], [5, 0]]
    res = run_steps_both(w, steps=len(steps), budget=[10 ** 9, 10 ** 9], device=DEV, cache_dict=c, now0=now.numpy(), fused=True,
                         hint=8, budget_per_step=steps)
    check(res)


@pytest.mark.parametrize("levels", [1, 2, 5])
def test_quantised_retention_gives_ties_at_the_threshold_every_step(levels):
    # few distinct log beta values: whole groups of entries share a score, the threshold falls inside a group in
    # every step and (segment, position) decides - one level: pure recency, every segment ties with every other
    w = wl(2, 2, 3, 2, 64)
    rng = np.random.default_rng(40 + levels)
    seg_len = rng.integers(100, 1500, w.nseg)
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=levels, pos_stride_max=1)
    g = torch.Generator().manual_seed(levels)
    c["log_beta"] = -(torch.randint(0, levels, c["log_beta"].shape, generator=g).to(torch.float32) + 1.0) * 0.125
    budget = [int(seg_len[:6].sum()) // 2, int(seg_len[6:].sum()) - 7]
    for hint in (0, 6, 200):
        clone = {k: (v.clone() if torch.is_tensor(v) else v) for k, v in c.items()}
        check(run_steps_both(w, steps=5, budget=budget, device=DEV, cache_dict=clone, now0=now.numpy(), fused=True, hint=hint),
              (levels, hint))


@pytest.mark.parametrize("seed,long_segments", [(s, False) for s in range(24)] + [(s, True) for s in range(12)])
def test_random_configuration(seed, long_segments):
    from test_gpu_random_sweep import random_case
    w, c, now, budgets = random_case(seed, long_segments=long_segments)
    for hint in (0, 1 + seed % 7, 900):
        clone = {k: (v.clone() if torch.is_tensor(v) else v) for k, v in c.items()}
        res = run_steps_both(w, steps=len(budgets), budget=[max(b[s] for b in budgets) for s in range(w.n_seq)], device=DEV,
                             cache_dict=clone, now0=now.numpy(), fused=True, hint=hint, budget_per_step=budgets)
        check(res, (seed, hint))


@pytest.mark.parametrize("S,L,H", [(600, 1, 2), (1100, 1, 1)])
def test_many_short_sequences(S, L, H):
    rng = np.random.default_rng(77 + S)
    w = ki.Workload("m", 0, S, L, H, 2 * H, 64, (0,) * S, (0,) * S, 1, 3.0, 1.5)
    seg_len = rng.integers(0, 41, w.nseg)
    seg_len[rng.random(w.nseg) < 0.1] = 0
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=S, pos_stride_max=2)
    g = torch.Generator().manual_seed(S)
    c["log_beta"] = -(torch.randint(0, 3, c["log_beta"].shape, generator=g).to(torch.float32)) * 0.25
    per_seq = [int(seg_len[s * L * H:(s + 1) * L * H].sum()) for s in range(S)]
    budget = [0 if rng.random() < 0.05 else int(rng.integers(1, max(2, n + 3))) for n in per_seq]
    for hint in (0, 2):
        clone = {k: (v.clone() if torch.is_tensor(v) else v) for k, v in c.items()}
        check(run_steps_both(w, steps=3, budget=budget, device=DEV, cache_dict=clone, now0=now.numpy(), fused=True, hint=hint), (S, hint))


def test_the_context_is_shared_by_unrelated_caches():
    # the carried bound belongs to the context, not to a cache: alternating two unrelated caches on one context makes
    # the bound useless (too low or far too high) - results must not depend on it
    w = wl(1, 2, 2, 2, 64)
    caches = []
    for salt, scale in ((1, 1.0), (2, 30.0)):
        c, now = ki.ragged_cache(w, [3000, 10, 5000, 2222], reserve=1, salt=salt)
        c["log_beta"] = c["log_beta"] * scale
        caches.append((c, now))
    cap = max(c["cap"] for c, _ in caches)
    ctx = kv.Context(1, 2, 2, 4, 64, cap)
    score = torch.zeros(cap, dtype=torch.float32, device=DEV)
    keep = torch.zeros(cap, dtype=torch.uint8, device=DEV)
    kept = torch.zeros(w.nseg, dtype=torch.int32, device=DEV)
    thr = torch.zeros(1, dtype=torch.int32, device=DEV)
    for rnd in range(3):
        for c, now in caches:
            hc = host_cache(w, c)
            n = int(hc.seg_len.sum())
            budget = np.array([n - 4 - rnd], np.int64)
            now_np = now.numpy() + rnd
            s_ref = oracle.score(hc, now_np)
            keep_ref, kept_ref, thr_ref = oracle.select(hc, s_ref, budget)
            dc = kv.Cache.from_dict(c, DEV)
            kv.kvtrim_score_select(ctx, dc, torch.from_numpy(now_np).to(DEV), torch.from_numpy(budget).to(DEV), score, keep,
                                   kept, thr, evict_hint=4)
            assert kv.kvtrim_poll_error(ctx) == 0
            live = live_mask(hc)
            assert np.array_equal(score[:hc.cap].cpu().numpy()[live].view(np.uint32), s_ref[live].view(np.uint32))
            assert np.array_equal(keep[:hc.cap].cpu().numpy()[live], keep_ref[live])
            assert np.array_equal(kept.cpu().numpy(), kept_ref)
            assert np.array_equal(thr.cpu().numpy().view(np.uint32), thr_ref)


def test_bad_segment_table_is_reported():
    w = wl(1, 1, 2, 2, 64)
    c, now = ki.ragged_cache(w, [100, 100], reserve=1, salt=1)
    c["seg_len"][0] = 150                                         # runs into the next segment
    dc = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(1, 1, 2, 4, 64, dc.cap)
    score = torch.zeros(dc.cap, dtype=torch.float32, device=DEV)
    keep = torch.zeros(dc.cap, dtype=torch.uint8, device=DEV)
    kept = torch.zeros(2, dtype=torch.int32, device=DEV)
    bud = torch.tensor([50], dtype=torch.int64, device=DEV)
    for hint in (0, 2):
        kv.kvtrim_score_select(ctx, dc, now.to(DEV), bud, score, keep, kept, None, evict_hint=hint)
        assert kv.kvtrim_poll_error(ctx) == -6


def select_repeatedly(w, lens, log_beta, evictions, calls):
    """A cache of which every call evicts `evictions` entries per sequence: one selection by the radix passes, then
    `calls` decode-step ones, all against the oracle.  Returns the path counts."""
    start = np.concatenate([[0], np.cumsum(lens + 1)[:-1]])
    cap = int((lens + 1).sum())
    c = {"k": torch.zeros(cap, 64, dtype=torch.bfloat16), "v": torch.zeros(cap, 64, dtype=torch.bfloat16),
         "log_beta": torch.from_numpy(log_beta(cap, start)).float(),
         "pos": torch.from_numpy((np.arange(cap) - np.repeat(start, lens + 1)).astype(np.int32)),
         "seg_start": torch.from_numpy(start), "seg_len": torch.from_numpy(lens.astype(np.int32)), "cap": cap}
    now = np.full(w.n_seq, int(lens.max()), dtype=np.int32)
    hc = host_cache(w, c)
    score = oracle.score(hc, now)
    budget = lens.reshape(w.n_seq, -1).sum(1) - evictions
    keep, kept, thr = oracle.select(hc, score, budget)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, 64, cap)
    dc = kv.Cache.from_dict(c, DEV)
    live = live_mask(hc)
    args = [torch.from_numpy(now).to(DEV), torch.from_numpy(budget).to(DEV), torch.zeros(cap, dtype=torch.float32, device=DEV),
            torch.zeros(cap, dtype=torch.uint8, device=DEV), torch.zeros(w.nseg, dtype=torch.int32, device=DEV),
            torch.zeros(w.n_seq, dtype=torch.int32, device=DEV)]
    for call in range(1 + calls):
        args[3].fill_(7)
        kv.kvtrim_score_select(ctx, dc, *args, evict_hint=evictions if call else 0)
        assert kv.kvtrim_poll_error(ctx) == 0
        assert np.array_equal(args[2].cpu().numpy()[live].view(np.uint32), score[live].view(np.uint32))
        k = args[3].cpu().numpy()
        assert np.array_equal(k[live], keep[live]) and np.all(k[~live] == 7)
        assert np.array_equal(args[4].cpu().numpy(), kept)
        assert np.array_equal(args[5].cpu().numpy().view(np.uint32), thr)
    return kv.kvtrim_select_path_counts(ctx)


def test_a_hot_layer_of_a_batch_stays_on_the_candidate_list():
    # 2048 segments, several to a scanning block; nearly all candidates (about 900 per sequence) come from the 16 neighbouring
    # segments of one layer, which must not share one block's sub-list (256 entries)
    w = wl(4, 32, 16, 1, 64)
    lens = np.full(w.nseg, 9)
    for s in range(4):
        lens[s * 512 + 80:s * 512 + 96] = 70

    def log_beta(cap, start):
        rng = np.random.default_rng(9)
        lb = -0.001 * rng.random(cap)
        for s in range(4):
            a, b = start[s * 512 + 80], start[s * 512 + 96]
            lb[a:b] = -1.0 - rng.random(b - a)
        return lb
    assert select_repeatedly(w, lens, log_beta, 300, 3) == (3 * 4, 0)


def test_one_hot_segment_of_a_batch_stays_on_the_candidate_list():
    # 320 segments, two to a block; all candidates of a sequence (some 600) come from one segment: more than a sub-list's 256
    # entries
    w = wl(5, 8, 8, 1, 64)
    lens = np.full(w.nseg, 40)
    lens[37::64] = 3000
    rng = np.random.default_rng(10)

    def log_beta(cap, start):
        lb = -0.0001 * rng.random(cap)
        for g in range(37, w.nseg, 64):
            lb[start[g]:start[g + 1]] = -1.0 - rng.random(start[g + 1] - start[g])
        return lb
    assert select_repeatedly(w, lens, log_beta, 150, 3) == (3 * 5, 0)


@pytest.mark.parametrize("S,H,evictions", [(260, 16, 490),        # about 1490 candidates per sequence: more than a block stages
                                           (260, 16, 8)])         # ... few, but a selection from scratch leaves the bound far off
def test_sequences_of_few_segments_stay_on_the_candidate_list(S, H, evictions):
    w = wl(S, 1, H, 1, 64)
    rng = np.random.default_rng(evictions)
    lens = rng.integers(140, 161, w.nseg)
    assert select_repeatedly(w, lens, lambda cap, start: -rng.random(cap), evictions, 3) == (3 * S, 0)


@pytest.mark.parametrize("cap,offset", [(1 << 21, 0), ((1 << 21) + 5, 0), ((1 << 21) - 1, 0), ((1 << 21) + 3, 1)])
def test_tails_enter_the_scores_of_large_caches(cap, offset):
    # the first pass loads log beta, positions and tails four entries at a time where the arrays are 16-byte aligned; segments that
    # begin and end at any entry, one of them empty, free entries behind the last
    w = wl(2, 2, 3, 1, 64)
    rng = np.random.default_rng(cap % 1000 + offset)
    lens = rng.integers(100000, 170001, w.nseg)
    lens[[1, 7]] = [0, 3]
    lens[11] += cap - 9 - w.nseg - int(lens.sum())
    start = np.concatenate([[0], np.cumsum(lens + 1)[:-1]])
    c = {"k": torch.zeros(cap, 64, dtype=torch.bfloat16), "v": torch.zeros(cap, 64, dtype=torch.bfloat16),
         "log_beta": torch.from_numpy(-np.log1p(np.exp(-(rng.standard_normal(cap) * 1.5 + 3)))).float(),
         "pos": torch.from_numpy((np.arange(cap) - np.repeat(np.append(start, cap - 9), np.append(lens + 1, 9))).astype(np.int32)),
         "seg_start": torch.from_numpy(start), "seg_len": torch.from_numpy(lens.astype(np.int32)), "cap": cap}
    c["log_tail"] = ki.log_tail_of(c["log_beta"], 2)
    now = np.array([int(lens[:6].max()), int(lens[6:].max())], dtype=np.int32)
    hc = host_cache(w, c)
    score = oracle.score(hc, now)
    budget = np.array([int(lens[:6].sum()) // 9, int(lens[6:].sum()) // 2])
    keep, kept, thr = oracle.select(hc, score, budget)

    def on_gpu(t):
        b = torch.zeros(t.numel() + offset, dtype=t.dtype, device=DEV)[offset:]
        return b.copy_(t)
    dc = kv.Cache(c["k"].to(DEV), c["v"].to(DEV), on_gpu(c["log_beta"]), on_gpu(c["pos"]), c["seg_start"].to(DEV),
                  c["seg_len"].to(DEV), on_gpu(c["log_tail"]))
    ctx = kv.Context(2, 2, 3, 3, 64, cap)
    live = live_mask(hc)
    s = torch.full((cap,), 7.0, device=DEV)
    k = torch.full((cap,), 7, dtype=torch.uint8, device=DEV)
    n, t = torch.zeros(w.nseg, dtype=torch.int32, device=DEV), torch.zeros(2, dtype=torch.int32, device=DEV)
    kv.kvtrim_score_select(ctx, dc, torch.from_numpy(now).to(DEV), torch.from_numpy(budget).to(DEV), s, k, n, t)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert np.array_equal(s.cpu().numpy()[live].view(np.uint32), score[live].view(np.uint32))
    assert np.array_equal(k.cpu().numpy()[live], keep[live]) and np.array_equal(n.cpu().numpy(), kept)
    assert np.array_equal(t.cpu().numpy().view(np.uint32), thr)


# The selection of small caches in one launch (k_sel_small) against the general kernels, which kvtrim_select_global_noalloc always
# runs, and the oracle: a block for a sequence and up to sixteen that meet, a second tile of a wavefront's entries (from 8192 a
# block on), lists at and over a wavefront's 64 entries, sequences of very different lengths and without entries, ties that
# have to be ranked inside a wavefront, over wavefronts and over blocks, infinities, budgets from below 0 to above all; behind
# one another on one context, whose counters and histograms every call leaves as it found them.
@pytest.mark.parametrize("S,L,H,lens", [
    (1, 1, 1, [1]), (1, 2, 2, [0, 63, 64, 65]), (1, 2, 4, [1024, 1025, 0, 1, 511, 513, 4000, 1117]), (1, 1, 3, [8191, 0, 2]),
    (1, 5, 4, [880]), (1, 3, 2, [20000, 1, 0, 23000, 700, 1]), (1, 1, 2, [130000, 130001]), (1, 128, 8, [33, 1, 0, 100]),
    (2, 1, 2, [5, 40000, 0, 0]), (3, 2, 2, [9000, 0, 100, 64, 0, 0, 0, 0, 1, 8192, 3, 50000]), (8, 1, 3, [100, 7, 2000]),
    (15, 1, 1, [1500, 0, 17000, 1, 2]), (16, 1, 2, [300, 5, 0, 900])])
@pytest.mark.parametrize("levels", [0, 3])
def test_one_launch_selection_equals_the_general_kernels(S, L, H, lens, levels):
    w = ki.Workload("t", 0, S, L, H, H, 64, (0,) * S, (0,) * S, 1, 3.0, 1.5)
    seg_len = [lens[g % len(lens)] for g in range(w.nseg)]
    c, now = ki.ragged_cache(w, seg_len, reserve=2, salt=S + levels)
    if levels:                                                   # few different scores, both zeros and minus infinity
        g = torch.Generator().manual_seed(7)
        c["log_beta"] = -torch.randint(0, levels, c["log_beta"].shape, generator=g).float()
        c["log_beta"][torch.rand(c["log_beta"].shape, generator=g) < 0.01] = -np.inf
        c["pos"] = torch.minimum(c["pos"], torch.tensor(50, dtype=torch.int32))
    hc = host_cache(w, c)
    src = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(S, L, H, H, 64, hc.cap)
    cfg = (S, L, H, H, 64, hc.cap)
    per = L * H
    full = np.array([sum(seg_len[s * per:(s + 1) * per]) for s in range(S)], dtype=np.int64)
    ref_score = oracle.score(hc, now.numpy())
    for part, budget in enumerate([full // 3, full // 3, full - full // 97, np.maximum(full // 2 - np.arange(S), 0), full * 0, full + 5, -np.ones(S, dtype=np.int64), full // 16 + 1]):
        keep, kept, thr = oracle.select(hc, ref_score, budget)
        bud = torch.from_numpy(np.ascontiguousarray(budget)).to(DEV)

        def outputs():
            return (torch.full((hc.cap,), 7, dtype=torch.uint8, device=DEV), torch.full((w.nseg,), 9, dtype=torch.int32, device=DEV),
                    torch.full((S,), 9, dtype=torch.int32, device=DEV))
        score = torch.full((hc.cap,), 99.0, device=DEV)
        a, b, d = outputs(), outputs(), outputs()
        kv.kvtrim_score_select(ctx, src, now.to(DEV), bud, score, *a)
        kv.kvtrim_select_global(ctx, src, score, bud, *b)
        status = torch.zeros(1, dtype=torch.int32, device=DEV)
        kv.kvtrim_select_global_noalloc(cfg, src, score, bud, *d, status)
        assert kv.kvtrim_poll_error(ctx) == 0 and int(status.item()) == 0
        for x, y, z in zip(a, b, d):
            assert torch.equal(x, z) and torch.equal(y, z), part
        assert np.array_equal(a[1].cpu().numpy(), kept) and np.array_equal(a[2].cpu().numpy().view(np.uint32), thr)
        k, sc = a[0].cpu().numpy(), score.cpu().numpy()
        outside = np.ones(hc.cap, dtype=bool)
        for st, n in zip(c["seg_start"].tolist(), seg_len):
            assert np.array_equal(k[st:st + n], keep[st:st + n])
            assert np.array_equal(sc[st:st + n].view(np.uint32), ref_score[st:st + n].view(np.uint32))
            outside[st:st + n] = False
        assert np.all(k[outside] == 7) and np.all(sc[outside] == 99.0)


def test_one_launch_selection_of_an_unusable_table_selects_nothing():
    w = ki.Workload("t", 0, 3, 2, 2, 2, 64, (0,) * 3, (0,) * 3, 1, 3.0, 1.5)
    c, now = ki.ragged_cache(w, [9000, 10] * 6, reserve=1, salt=1)
    src = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(3, 2, 2, 2, 64, src.cap)
    src.seg_len[7] = 10 ** 6                                     # in the second sequence
    bud = torch.full((3,), 100, dtype=torch.int64, device=DEV)
    keep = torch.full((src.cap,), 7, dtype=torch.uint8, device=DEV)
    kept, thr = torch.full((12,), 9, dtype=torch.int32, device=DEV), torch.zeros(3, dtype=torch.int32, device=DEV)
    score = torch.zeros(src.cap, device=DEV)
    kv.kvtrim_score_select(ctx, src, now.to(DEV), bud, score, keep, kept, thr)
    assert kv.kvtrim_poll_error(ctx) == -6                       # KVTRIM_ELAYOUT
    assert torch.all(keep == 7) and torch.all(kept == 0) and torch.all(thr == -1)


# A sequence's blocks need not be on the chip together: one that has looked KVTRIM_SEL_WAIT times without seeing all of the others does the
# whole selection, and those that come later leave.  At 0 the first to arrive takes over in every call, at 1 and 3 now one and now none.
@pytest.mark.parametrize("wait", [0, 1, 3])
@pytest.mark.parametrize("S,L,H,lens", [
    (1, 2, 4, [1024, 1025, 0, 1, 511, 513, 4000, 1117]), (1, 1, 2, [130000, 130001]), (1, 128, 8, [33, 1, 0, 100]),
    (3, 2, 2, [9000, 0, 100, 64, 0, 0, 0, 0, 1, 8192, 3, 50000]), (15, 1, 1, [1500, 0, 17000, 1, 2])])
def test_one_launch_selection_by_a_block_that_does_not_wait(S, L, H, lens, wait, monkeypatch):
    monkeypatch.setenv("KVTRIM_SEL_WAIT", str(wait))
    for levels in (0, 3):
        test_one_launch_selection_equals_the_general_kernels(S, L, H, lens, levels)


def test_one_launch_selections_on_many_streams_beside_large_kernels():
    # a context and a stream each, calls of up to sixteen blocks that meet, beside products that fill the chip: whichever blocks get
    # onto it together, every call has its own selection
    w = ki.Workload("t", 0, 1, 4, 4, 4, 64, (0,), (0,), 1, 3.0, 1.5)
    streams = [torch.cuda.Stream() for _ in range(12)]
    busy = torch.cuda.Stream()
    m = torch.randn(4096, 4096, device=DEV).bfloat16()
    sets = []
    for i in range(len(streams)):
        c, now = ki.ragged_cache(w, [3000 + 500 * i + 77 * g for g in range(16)], reserve=1, salt=i)
        src = kv.Cache.from_dict(c, DEV)
        bud = torch.tensor([int(sum(c["seg_len"].tolist())) // (2 + i % 3)], dtype=torch.int64, device=DEV)
        out = [torch.zeros(src.cap, device=DEV), torch.zeros(src.cap, dtype=torch.uint8, device=DEV), torch.zeros(16, dtype=torch.int32, device=DEV),
               torch.zeros(1, dtype=torch.int32, device=DEV)]
        want = oracle.select(host_cache(w, c), oracle.score(host_cache(w, c), now.numpy()), bud.cpu().numpy())
        sets.append((kv.Context(1, 4, 4, 4, 64, src.cap), src, now.to(DEV), bud, out, want, c))
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(30):
            m @ m
    for call in range(25):
        for st, (ctx, src, now, bud, out, want, c) in zip(streams, sets):
            kv.kvtrim_score_select(ctx, src, now, bud, *out, stream=st)
    torch.cuda.synchronize()
    for ctx, src, now, bud, (score, keep, kept, thr), (keep_ref, kept_ref, thr_ref), c in sets:
        assert kv.kvtrim_poll_error(ctx) == 0
        assert np.array_equal(kept.cpu().numpy(), kept_ref) and np.array_equal(thr.cpu().numpy().view(np.uint32), thr_ref)
        k = keep.cpu().numpy()
        for s, n in zip(c["seg_start"].tolist(), c["seg_len"].tolist()):
            assert np.array_equal(k[s:s + n], keep_ref[s:s + n])
