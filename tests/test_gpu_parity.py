"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element.

Selection and compaction must match bit for bit; attention within
max|o_gpu - o_ref| / max|o_ref| <= 5e-3 (bf16 inputs, fp32 accumulation).
"""
import math

import numpy as np
import pytest
import torch

import kvtrim_inputs as ki
import oracle
import paper_2605_09649_amd as kv
from harness import attn_error, compare_caches, device_cache_to_host, run_multiturn_both, run_steps_both
from helpers import bf16_bits, host_cache, live_mask

pytestmark = pytest.mark.gpu
ATTN_TOL = 5e-3
DEV = "cuda:0"


def check(results):
    for i, r in enumerate(results):
        assert r["status"] == 0, (i, r)
        assert r["score_equal"], (i, "score bits differ")
        assert r["keep_equal"], (i, "selection differs")
        assert r["cache_equal"], (i, "compacted cache differs")
        assert r["attn_err"] <= ATTN_TOL, (i, r["attn_err"])
        assert r["lse_err"] <= 2e-3 and r["lse_inf_equal"], (i, r)


def wl(S, L, H, G, D, name="t"):
    return ki.Workload(name, 0, S, L, H, G * H, D, (0,) * S, (0,) * S, 1, 3.0, 1.5)


# ---------------------------------------------------------------------------------- whole loop

@pytest.mark.parametrize("fused", [False, True])
def test_tiny_workload_full_loop(fused):
    w = ki.workload("tiny")                       # L4 H4 G2 D64, 2048 prefilled, B = 1024, 16 steps
    check(run_steps_both(w, steps=16, budget=w.budget, device=DEV, fused=fused))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("name,prefill,steps", [("llama", 700, 3), ("long", 900, 3), ("vlm", 640, 3),
                                                ("multiturn", 600, 2)])
def test_scaled_down_workloads(name, prefill, steps, fused):
    w = ki.workload(name, prefill=prefill)
    check(run_steps_both(w, steps=steps, budget=w.budget, device=DEV, fused=fused))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("S,L,H,G,D", [(1, 2, 2, 1, 128), (2, 2, 1, 7, 128), (1, 1, 3, 8, 64), (3, 1, 2, 3, 64),
                                       (1, 2, 2, 5, 128), (1, 1, 2, 6, 128), (1, 2, 1, 4, 128), (1, 1, 2, 2, 64)])
def test_ragged_segments_spanning_several_chunks(S, L, H, G, D, fused):
    w = wl(S, L, H, G, D)
    rng = np.random.default_rng(S * 1000 + G * 10 + D)
    seg_len = rng.integers(0, 6000, w.nseg)
    seg_len[rng.integers(0, w.nseg)] = 0          # an empty segment
    seg_len[rng.integers(0, w.nseg)] = 2048 * 2 + 1
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=G)
    per_seq = [int(seg_len[s * L * H:(s + 1) * L * H].sum()) for s in range(S)]
    budget = [max(1, n // 3) for n in per_seq]
    check(run_steps_both(w, steps=2, budget=budget, device=DEV, cache_dict=c, now0=now.numpy(), fused=fused))


@pytest.mark.parametrize("fused", [False, True])
def test_multi_turn_chunked_prefill_then_decode(fused):
    # the multi-turn configuration scaled down: sequences of different lengths grow by prefill chunks (ragged last
    # chunks are padded with negative positions), the cache is rescored, selected and compacted after every chunk,
    # then a few tokens are decoded; four turns, per-sequence budgets
    w = wl(3, 2, 2, 2, 64)
    lengths = [700, 180, 411]
    res = run_multiturn_both(w, lengths, chunk=64, decode_per_turn=3, budget=[160, 10 ** 6, 96], device=DEV, fused=fused)
    assert len(res) > 20 and any("decode" in r["what"] for r in res)
    for r in res:
        assert r["status"] == 0 and r["score_equal"] and r["keep_equal"] and r["cache_equal"], r
        if "attn_err" in r:
            assert r["attn_err"] <= ATTN_TOL and r["lse_err"] <= 2e-3, r


@pytest.mark.parametrize("D", [64, 128])
def test_multi_turn_chunks_in_one_call(D):
    # the same flow with every chunk step done by kvtrim_append_compact (metadata appended, rows moved once, from
    # the caller's buffers to the compacted cache): scores, mask, counts, threshold and cache as the oracle's four stages
    w = wl(3, 2, 2, 2, D)
    res = run_multiturn_both(w, [700, 180, 411], chunk=64, decode_per_turn=2, budget=[160, 10 ** 6, 96], device=DEV,
                             one_call_chunks=True)
    assert sum("chunk" in r["what"] for r in res) > 10
    for r in res:
        assert r["status"] == 0 and r["score_equal"] and r["keep_equal"] and r["cache_equal"], r
        if "attn_err" in r:
            assert r["attn_err"] <= ATTN_TOL and r["lse_err"] <= 2e-3, r


def test_multi_turn_chunks_in_one_call_sixteen_sequences():
    w = ki.workload("multiturn", prefill=1024)                   # S16 L32 Hkv8 Hq32 D128, lengths in [64, 1024]
    res = run_multiturn_both(w, list(w.prefill), chunk=256, decode_per_turn=1, budget=[96 * 32 * 8] * 16, device=DEV,
                             turns=2, one_call_chunks=True)
    for r in res:
        assert r["status"] == 0 and r["score_equal"] and r["keep_equal"] and r["cache_equal"], r


@pytest.mark.parametrize("horizon", [1, 2, 0])
def test_append_compact_on_a_ragged_cache(horizon):
    # one call on a cache with gapped positions and an empty segment: sequence 0 brings a full chunk, sequence 1 a
    # ragged one (padding rows behind its 11 tokens); with a lookahead horizon the new tokens bring their tail constant
    w = wl(2, 2, 3, 2, 128)
    rng = np.random.default_rng(5 + horizon)
    seg_len = rng.integers(1, 300, w.nseg)
    seg_len[3] = 0
    n_new, per_seq = 37, w.n_layers * w.n_kv_heads
    c, now = ki.ragged_cache(w, seg_len, reserve=n_new, salt=9)
    c = ki.with_horizon(c, horizon)
    inp = ki.chunk_inputs(w, n_new, "cpu", 3)
    lt_new = None if horizon == 1 else ki.log_tail_of(inp["log_beta_new"], horizon)
    take = [n_new, 11]
    pos_new = np.full((w.nseg, n_new), -1, np.int32)
    for s in range(2):
        pos_new[s * per_seq:(s + 1) * per_seq, :take[s]] = int(now[s]) + np.arange(take[s])
    now_after = (now.numpy() + np.array(take) - 1).astype(np.int32)
    n_seq_entries = [int(seg_len[s * per_seq:(s + 1) * per_seq].sum()) + take[s] * per_seq for s in range(2)]
    budget = np.array([n_seq_entries[0] // 2, n_seq_entries[1] - 5], np.int64)
    cap = c["cap"]
    # ---- oracle: the four stages
    hc = host_cache(w, c)
    oracle.append(hc, bf16_bits(inp["k_new"]), bf16_bits(inp["v_new"]), inp["log_beta_new"].numpy(), pos_new,
                  log_tail_new=None if lt_new is None else lt_new.numpy())
    s_ref = oracle.score(hc, now_after)
    k_ref, kept_ref, thr_ref = oracle.select(hc, s_ref, budget)
    hc_next = oracle.compact(hc, k_ref, cap, 1)
    # ---- GPU: one call
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, w.head_dim, cap)
    src = kv.Cache.from_dict(c, DEV)
    dst = kv.Cache.empty(w.nseg, w.head_dim, cap, DEV, with_tail=horizon != 1)
    score = torch.zeros(cap, dtype=torch.float32, device=DEV)
    keep = torch.zeros(cap, dtype=torch.uint8, device=DEV)
    kept = torch.zeros(w.nseg, dtype=torch.int32, device=DEV)
    thr = torch.zeros(w.n_seq, dtype=torch.int32, device=DEV)
    kv.kvtrim_append_compact(ctx, src, inp["k_new"].to(DEV), inp["v_new"].to(DEV), inp["log_beta_new"].to(DEV),
                             torch.from_numpy(pos_new).to(DEV), n_new, torch.from_numpy(now_after).to(DEV),
                             torch.from_numpy(budget).to(DEV), score, keep, kept, dst, 1, thr_key_out=thr,
                             log_tail_new=None if lt_new is None else lt_new.to(DEV))
    assert kv.kvtrim_poll_error(ctx) == 0
    live = live_mask(hc)
    assert np.array_equal(score.cpu().numpy()[live].view(np.uint32), s_ref[live].view(np.uint32))
    assert np.array_equal(keep.cpu().numpy()[live], k_ref[live]) and np.array_equal(kept.cpu().numpy(), kept_ref)
    assert np.array_equal(thr.cpu().numpy().view(np.uint32), thr_ref)
    assert compare_caches(device_cache_to_host(w, dst), hc_next)
    assert int(kept_ref.sum()) == int(budget.sum())


def test_append_compact_argument_checks():
    w = wl(1, 1, 1, 1, 64)
    nseg, cap = 1, 64
    ctx = kv.Context(1, 1, 1, 1, 64, cap)
    a, b = kv.Cache.empty(nseg, 64, cap, DEV), kv.Cache.empty(nseg, 64, cap, DEV)
    t = lambda *shape, dt=torch.float32: torch.zeros(*shape, dtype=dt, device=DEV)
    k_new, lb, pos = t(1, 4, 64, dt=torch.bfloat16), t(1, 4), t(1, 4, dt=torch.int32)
    now, budget = t(1, dt=torch.int32), t(1, dt=torch.int64)
    score, keep, kept = t(cap), t(cap, dt=torch.uint8), t(nseg, dt=torch.int32)
    with pytest.raises(kv.KvtrimError):                           # source and destination share buffers
        kv.kvtrim_append_compact(ctx, a, k_new, k_new, lb, pos, 4, now, budget, score, keep, kept, a, 0)
    with pytest.raises(kv.KvtrimError):                           # no tokens
        kv.kvtrim_append_compact(ctx, a, k_new, k_new, lb, pos, 0, now, budget, score, keep, kept, b, 0)
    with pytest.raises(kv.KvtrimError):                           # a missing output
        kv.kvtrim_append_compact(ctx, a, k_new, k_new, lb, pos, 4, now, budget, None, keep, kept, b, 0)
    with pytest.raises(kv.KvtrimError):                           # the tail constant without a cache that carries it
        kv.kvtrim_append_compact(ctx, a, k_new, k_new, lb, pos, 4, now, budget, score, keep, kept, b, 0, log_tail_new=lb)
    assert kv.kvtrim_poll_error(ctx) == 0


def test_multi_turn_chunked_sixteen_sequences():
    w = ki.workload("multiturn", prefill=1024)                   # S16 L32 Hkv8 Hq32 D128, lengths in [64, 1024]
    per_head = 96
    res = run_multiturn_both(w, list(w.prefill), chunk=256, decode_per_turn=2, budget=[per_head * 32 * 8] * 16, device=DEV,
                             turns=2)
    for r in res:
        assert r["status"] == 0 and r["score_equal"] and r["keep_equal"] and r["cache_equal"], r
        if "attn_err" in r:
            assert r["attn_err"] <= ATTN_TOL and r["lse_err"] <= 2e-3, r


@pytest.mark.parametrize("fused", [False, True])
def test_one_giant_segment_and_many_empty_ones(fused):
    w = wl(1, 2, 4, 4, 128)
    seg_len = [0, 0, 0, 70001, 0, 0, 3, 0]
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=3)
    check(run_steps_both(w, steps=2, budget=[20011], device=DEV, cache_dict=c, now0=now.numpy(), fused=fused))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("horizon", [2, 5, 0])
def test_lookahead_horizon_scores_through_the_whole_loop(horizon, fused):
    # Sec. 4.2: horizon T-t = 2 is the paper's inference default, 0 stands for the limit T-t -> infinity
    w = ki.workload("tiny", prefill=700)
    check(run_steps_both(w, steps=6, budget=w.budget, device=DEV, fused=fused, horizon=horizon))
    w = ki.workload("llama", prefill=600)
    check(run_steps_both(w, steps=2, budget=w.budget, device=DEV, fused=fused, horizon=horizon))


def test_horizon_tail_must_be_consistent_between_caches():
    w = wl(1, 1, 2, 2, 64)
    c, now = ki.ragged_cache(w, [10, 10], salt=1)
    ctx = kv.Context(1, 1, 2, 4, 64, 32)
    src = kv.Cache.from_dict(ki.with_horizon(c, 2), DEV)
    dst = kv.Cache.empty(2, 64, 32, DEV)                                  # no tail in the destination
    keep = torch.ones(32, dtype=torch.uint8, device=DEV)
    kept = torch.tensor([10, 10], dtype=torch.int32, device=DEV)
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_compact(ctx, src, keep, kept, dst, 1)
    new = ki.decode_inputs(w, 0)
    with pytest.raises(kv.KvtrimError):                                   # tail required for this cache
        kv.kvtrim_append(ctx, src, new["k_new"].to(DEV), new["v_new"].to(DEV), new["log_beta_new"].to(DEV),
                         torch.zeros(2, dtype=torch.int32, device=DEV), 1)


@pytest.mark.parametrize("G,D", [(4, 128), (8, 128), (6, 64)])
@pytest.mark.parametrize("roomy", [True, False])
def test_fused_call_with_a_layer_range_and_sparse_mask(roomy, G, D):
    # compaction + attention in one call on a mask that keeps about one entry in five, layers [1, 3) only.  With a
    # destination of at least a quarter of the source the fused kernel works a block per chunk of the source; with a
    # tight one the library expects few survivors and works a block per chunk of the destination - same results
    # either way.
    w = wl(2, 3, 2, G, D)
    rng = np.random.default_rng(21)
    seg_len = rng.integers(0, 2500, w.nseg)
    c, _ = ki.ragged_cache(w, seg_len, salt=21)
    hc = host_cache(w, c)
    keep_np = (rng.random(hc.cap) < 0.2).astype(np.uint8)
    kept_np = np.array([keep_np[s:s + n].sum() for s, n in zip(hc.seg_start, hc.seg_len)], np.int32)
    dst_cap = hc.cap // 2 if roomy else int(kept_np.sum()) + 2 * w.nseg
    assert (dst_cap >= hc.cap // 4) == roomy
    dst_ref = oracle.compact(hc, keep_np, dst_cap, 2)
    q = ki.decode_inputs(w, 3)["q"]
    scale = 1.0 / math.sqrt(D)
    ref, ref_lse = oracle.attend(dst_ref, bf16_bits(q), scale)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, D, hc.cap)
    dst = kv.Cache.empty(w.nseg, D, dst_cap, DEV)
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    kv.kvtrim_compact_attn(ctx, kv.Cache.from_dict(c, DEV), torch.from_numpy(keep_np).to(DEV),
                           torch.from_numpy(kept_np).to(DEV), dst, 2, q.to(DEV), 1, 3, scale, out, lse)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert compare_caches(device_cache_to_host(w, dst), dst_ref)
    o = out.cpu().numpy()
    assert np.all(o[:, 0] == 99.0)
    assert attn_error(o[:, 1:3], ref[:, 1:3]) <= ATTN_TOL
    fin = np.isfinite(ref_lse[:, 1:3])
    assert np.abs(lse.cpu().numpy()[:, 1:3][fin] - ref_lse[:, 1:3][fin]).max() <= 2e-3


@pytest.mark.parametrize("D,horizon", [(128, 1), (64, 1), (128, 2)])
def test_sparse_selection_in_stage_three_alone_gathers_by_destination_chunk(D, horizon):
    # a destination under a quarter of the source: the row mover works a block per 128-row chunk of the DESTINATION
    # (the fused kernel's gathering instance with no layer to attend).  One entry in sixteen survives on average; some
    # source chunks keep nothing, some keep every entry, segments end in ragged chunks, one segment is empty.
    w = wl(2, 2, 3, 2, D)
    rng = np.random.default_rng(77 + D + horizon)
    seg_len = rng.integers(1, 6000, w.nseg)
    seg_len[3] = 0
    seg_len[5] = 128 * 9 + 1
    c, _ = ki.ragged_cache(w, seg_len, salt=33)
    c = ki.with_horizon(c, horizon)
    hc = host_cache(w, c)
    keep_np = (rng.random(hc.cap) < 1.0 / 16).astype(np.uint8)
    s5 = int(hc.seg_start[5])
    keep_np[s5 + 128:s5 + 3 * 128] = 1                            # two chunks that keep everything
    keep_np[s5 + 4 * 128:s5 + 6 * 128] = 0                        # two that keep nothing
    keep_np[s5 + 9 * 128] = 1                                     # the one-entry tail chunk
    kept_np = np.array([keep_np[s:s + n].sum() for s, n in zip(hc.seg_start, hc.seg_len)], np.int32)
    dst_cap = int(kept_np.sum()) + 3 * w.nseg
    assert dst_cap < hc.cap // 4
    dst_ref = oracle.compact(hc, keep_np, dst_cap, 3)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, D, hc.cap)
    dst = kv.Cache.empty(w.nseg, D, dst_cap, DEV, with_tail=horizon != 1)
    kv.kvtrim_compact(ctx, kv.Cache.from_dict(c, DEV), torch.from_numpy(keep_np).to(DEV), torch.from_numpy(kept_np).to(DEV),
                      dst, 3)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert compare_caches(device_cache_to_host(w, dst), dst_ref)


@pytest.mark.parametrize("G,D,horizon,many", [(4, 128, 1, False), (1, 128, 2, False), (5, 128, 1, False), (3, 128, 1, True),
                                              (2, 64, 1, False), (4, 64, 2, False)])
def test_sparse_selection_in_the_fused_call_gathers_by_destination_chunk(G, D, horizon, many):
    # compaction + attention in one call with a destination under a quarter of the source and a group of query heads
    # the one-shot kernel serves: its gathering instance runs, a block per 128-row chunk of the DESTINATION reading the
    # source rows the compaction scan has listed.  One entry in sixteen survives on average; some source chunks keep
    # nothing, some everything, one segment is empty, one keeps nothing, one keeps exactly one chunk's worth, segments
    # end in ragged chunks; `many`: more than 1024 segments (the scan's prefix kernel).  Layers [1, 3) attend.
    w = wl(2, 180 if many else 3, 3, G, D)
    rng = np.random.default_rng(1000 + 16 * G + D + horizon)
    seg_len = rng.integers(1, 700 if many else 6000, w.nseg)
    seg_len[3] = 0
    seg_len[5] = 128 * 9 + 1
    seg_len[7] = 300
    seg_len[9] = 128 * 20
    c, _ = ki.ragged_cache(w, seg_len, salt=35)
    c = ki.with_horizon(c, horizon)
    hc = host_cache(w, c)
    keep_np = (rng.random(hc.cap) < 1.0 / 16).astype(np.uint8)
    s5, s7, s9 = int(hc.seg_start[5]), int(hc.seg_start[7]), int(hc.seg_start[9])
    keep_np[s5 + 128:s5 + 3 * 128] = 1                            # two source chunks that keep everything
    keep_np[s5 + 4 * 128:s5 + 6 * 128] = 0                        # two that keep nothing
    keep_np[s5 + 9 * 128] = 1                                     # the one-entry tail chunk
    keep_np[s7:s7 + 300] = 0                                      # a segment that keeps nothing
    keep_np[s9:s9 + 128 * 20] = 0
    keep_np[s9 + 5:s9 + 128 * 20:20] = 1                          # exactly 128 survivors: one full destination chunk
    kept_np = np.array([keep_np[s:s + n].sum() for s, n in zip(hc.seg_start, hc.seg_len)], np.int32)
    assert kept_np[7] == 0 and kept_np[9] == 128
    dst_cap = int(kept_np.sum()) + 2 * w.nseg
    assert dst_cap < hc.cap // 4
    dst_ref = oracle.compact(hc, keep_np, dst_cap, 2)
    q = ki.decode_inputs(w, 3)["q"]
    scale = 1.0 / math.sqrt(D)
    ref, ref_lse = oracle.attend(dst_ref, bf16_bits(q), scale)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, D, hc.cap)
    dst = kv.Cache.empty(w.nseg, D, dst_cap, DEV, with_tail=horizon != 1)
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    keep_d, kept_d = torch.from_numpy(keep_np).to(DEV), torch.from_numpy(kept_np).to(DEV)
    kv.kvtrim_profile_begin(ctx, (1 << kv.binding.N_KERNELS) - 1)
    kv.kvtrim_compact_attn(ctx, kv.Cache.from_dict(c, DEV), keep_d, kept_d, dst, 2, q.to(DEV), 1, 3, scale, out, lse)
    times = kv.kvtrim_profile_end(ctx)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert times["k_cmp_attn"][1] == 1 and "k_cmp_copy" not in times      # the fused kernel ran, not the two stages
    assert compare_caches(device_cache_to_host(w, dst), dst_ref)
    o = out.cpu().numpy()
    assert np.all(o[:, 0] == 99.0)
    assert attn_error(o[:, 1:3], ref[:, 1:3]) <= ATTN_TOL
    fin = np.isfinite(ref_lse[:, 1:3])
    assert np.abs(lse.cpu().numpy()[:, 1:3][fin] - ref_lse[:, 1:3][fin]).max() <= 2e-3
    assert np.all(np.isneginf(lse.cpu().numpy()[:, 1:3][~fin]))
    # a mask with more survivors than `kept` says is reported (as that, not as a failed HIP call)
    keep_bad = keep_np.copy()
    keep_bad[s7:s7 + 300] = 1
    guard = kv.Cache.empty(w.nseg, D, dst_cap, DEV, with_tail=horizon != 1)
    kv.kvtrim_compact_attn(ctx, kv.Cache.from_dict(c, DEV), torch.from_numpy(keep_bad).to(DEV), kept_d, guard, 2, q.to(DEV),
                           1, 3, scale, out, lse)
    assert kv.kvtrim_poll_error(ctx) == -5                         # KVTRIM_EMISMATCH
    assert kv.kvtrim_poll_error(ctx) == 0


# ---------------------------------------------------------------------------------- degenerate budgets, ties

def run_select_compact(w, c, now, budget, score_override=None, reserve=1):
    """One score -> select -> compact on both sides; returns (gpu results, oracle results)."""
    hc = host_cache(w, c)
    total = int(hc.seg_len.sum())
    dst_cap = min(int(sum(budget)), total) + w.nseg * reserve + 4
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, w.head_dim, max(hc.cap, dst_cap))
    src = kv.Cache.from_dict(c, DEV)
    dst = kv.Cache.empty(w.nseg, w.head_dim, dst_cap, DEV)
    score = torch.zeros(hc.cap, dtype=torch.float32, device=DEV)
    keep = torch.full((hc.cap,), 7, dtype=torch.uint8, device=DEV)
    kept = torch.zeros(w.nseg, dtype=torch.int32, device=DEV)
    thr = torch.zeros(w.n_seq, dtype=torch.int32, device=DEV)
    kv.kvtrim_score(ctx, src, now.to(DEV), score)
    score_ref = oracle.score(hc, now.numpy())
    if score_override is not None:
        score_ref = score_override.copy()
        score.copy_(torch.from_numpy(score_override))
    b = torch.tensor(budget, dtype=torch.int64, device=DEV)
    kv.kvtrim_select_global(ctx, src, score, b, keep, kept, thr)
    kv.kvtrim_compact(ctx, src, keep, kept, dst, reserve)
    assert kv.kvtrim_poll_error(ctx) == 0
    keep_ref, kept_ref, thr_ref = oracle.select(hc, score_ref, np.array(budget, np.int64))
    dst_ref = oracle.compact(hc, keep_ref, dst_cap, reserve)
    live = live_mask(hc)
    assert np.array_equal(score.cpu().numpy()[live].view(np.uint32), score_ref[live].view(np.uint32))
    assert np.array_equal(keep.cpu().numpy()[live], keep_ref[live])
    assert np.array_equal(kept.cpu().numpy(), kept_ref)
    assert np.array_equal(thr.cpu().numpy().view(np.uint32), thr_ref)
    assert compare_caches(device_cache_to_host(w, dst), dst_ref)
    return kept_ref


@pytest.mark.parametrize("frac", [0.0, 1.0, 2.0, 0.5])
def test_budget_zero_full_and_above_full(frac):
    w = wl(2, 2, 2, 2, 64)
    rng = np.random.default_rng(11)
    seg_len = rng.integers(0, 3000, w.nseg)
    c, now = ki.ragged_cache(w, seg_len, salt=5)
    per_seq = [int(seg_len[s * 4:(s + 1) * 4].sum()) for s in range(2)]
    kept = run_select_compact(w, c, now, [int(frac * n) for n in per_seq])
    for s in range(2):
        assert kept[s * 4:(s + 1) * 4].sum() == min(int(frac * per_seq[s]), per_seq[s])


def test_all_scores_equal_keeps_the_first_entries_in_storage_order():
    w = wl(1, 2, 2, 2, 64)
    seg_len = [3000, 2500, 4100, 100]
    c, now = ki.ragged_cache(w, seg_len, salt=6)
    score = np.full(sum(seg_len) + 4, -3.0, np.float32)
    for B in (1, 2999, 3000, 3001, 5500, 7777, 9699, 9700):
        kept = run_select_compact(w, c, now, [B], score_override=score)
        expect, left = [], B
        for n in seg_len:
            expect.append(min(n, left))
            left -= expect[-1]
        assert kept.tolist() == expect


def test_heavy_ties_signed_zeros_and_infinities():
    w = wl(2, 1, 3, 2, 64)
    rng = np.random.default_rng(12)
    seg_len = rng.integers(1000, 5000, w.nseg)
    c, now = ki.ragged_cache(w, seg_len, salt=7)
    cap = int(seg_len.sum()) + w.nseg
    vals = np.array([-np.inf, -7.5, -7.5, -1e-20, -0.0, 0.0, -2.0000002, -2.0], np.float32)
    score = rng.choice(vals, size=cap).astype(np.float32)
    for frac in (0.1, 0.37, 0.5, 0.93):
        budget = [int(frac * seg_len[:3].sum()), int(frac * seg_len[3:].sum())]
        run_select_compact(w, c, now, budget, score_override=score)


def test_keys_differing_only_in_low_bits():
    w = wl(1, 1, 2, 2, 64)
    seg_len = [5000, 5000]
    c, now = ki.ragged_cache(w, seg_len, salt=8)
    rng = np.random.default_rng(13)
    bits = (np.float32(-1.5).view(np.uint32) + rng.integers(0, 1 << 9, sum(seg_len) + 2).astype(np.uint32))
    score = bits.view(np.float32)
    for B in (1, 100, 4999, 9000):
        run_select_compact(w, c, now, [B], score_override=score)


# ---------------------------------------------------------------------------------- attention alone

@pytest.mark.parametrize("D,G", [(128, 4), (128, 7), (64, 2), (128, 1), (64, 8)])
def test_attention_against_oracle_and_layer_ranges(D, G):
    w = wl(2, 3, 2, G, D)
    rng = np.random.default_rng(D + G)
    seg_len = rng.integers(0, 1500, w.nseg)
    seg_len[0] = 0
    seg_len[1] = 1
    seg_len[2] = 257
    c, _ = ki.ragged_cache(w, seg_len, salt=9)
    hc = host_cache(w, c)
    dc = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, D, hc.cap)
    q = ki.decode_inputs(w, 0)["q"]
    scale = 1.0 / math.sqrt(D)
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), scale)
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    kv.kvtrim_decode_attn(ctx, dc, q.to(DEV), 0, w.n_layers, scale, out, lse)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert attn_error(out.cpu().numpy(), ref) <= ATTN_TOL
    o = out.cpu().numpy()
    assert np.all(o[0, 0, :G] == 0.0)                                   # empty segment
    assert np.isneginf(lse.cpu().numpy()[0, 0, :G]).all()
    fin = np.isfinite(ref_lse)
    assert np.abs(lse.cpu().numpy()[fin] - ref_lse[fin]).max() <= 2e-3
    # a layer range writes only its layers
    out2 = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    kv.kvtrim_decode_attn(ctx, dc, q.to(DEV), 1, 2, scale, out2, None)
    o2 = out2.cpu().numpy()
    assert np.all(o2[:, 0] == 99.0) and np.all(o2[:, 2] == 99.0)
    # (the rows are shared out among the kernel's blocks per call, so the order of the fp32 sums - not their terms -
    # depends on the layer range)
    assert attn_error(o2[:, 1], o[:, 1]) <= 2e-6


@pytest.mark.parametrize("blocks", [1, 2, 3, 7, 50, 100000])
def test_attention_for_any_size_of_the_fixed_grid(blocks, monkeypatch):
    # the attention kernel's blocks share the chunk table in equal parts of 64 rows and leave one partial result per
    # block and segment; whatever the number of blocks (a tuning knob read when the context is created) - one block
    # that walks everything, shares that end inside a chunk or inside a segment, more blocks than chunks - the
    # merge must find exactly those partial results
    monkeypatch.setenv("KVTRIM_ATT_BLOCKS", str(blocks))
    w = wl(2, 2, 2, 4, 128)
    seg_len = [3000, 0, 513, 64, 1, 2049, 700, 5000]
    c, _ = ki.ragged_cache(w, seg_len, salt=21)
    hc = host_cache(w, c)
    dc = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, 128, hc.cap)
    q = ki.decode_inputs(w, 0)["q"]
    scale = 1.0 / math.sqrt(128)
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), scale)
    for rng in ((0, 2), (1, 2)):
        out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
        lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
        kv.kvtrim_decode_attn(ctx, dc, q.to(DEV), rng[0], rng[1], scale, out, lse)
        assert kv.kvtrim_poll_error(ctx) == 0
        o, l = out.cpu().numpy()[:, rng[0]:rng[1]], lse.cpu().numpy()[:, rng[0]:rng[1]]
        assert attn_error(o, ref[:, rng[0]:rng[1]]) <= ATTN_TOL, (blocks, rng)
        fin = np.isfinite(ref_lse[:, rng[0]:rng[1]])
        assert np.abs(l[fin] - ref_lse[:, rng[0]:rng[1]][fin]).max() <= 2e-3
        assert np.array_equal(np.isneginf(l), ~fin)


@pytest.mark.parametrize("seed", range(8))
def test_attention_on_random_shapes_ranges_and_grids(seed, monkeypatch):
    # random segment lengths (many empty or tiny ones beside long ones), a random layer range and a random number of
    # blocks for the attention kernel's fixed grid: the shares of the blocks start and end anywhere
    rng = np.random.default_rng(1000 + seed)
    S, L, H = int(rng.integers(1, 4)), int(rng.integers(1, 4)), int(rng.integers(1, 4))
    G, D = int(rng.choice([1, 2, 4, 7])), int(rng.choice([64, 128]))
    monkeypatch.setenv("KVTRIM_ATT_BLOCKS", str(int(rng.choice([1, 2, 3, 5, 9, 17, 40, 768]))))
    w = wl(S, L, H, G, D)
    kinds = rng.integers(0, 5, w.nseg)
    seg_len = np.where(kinds == 0, 0, np.where(kinds == 1, rng.integers(1, 70, w.nseg),
                       np.where(kinds == 2, rng.integers(400, 700, w.nseg), rng.integers(1000, 6000, w.nseg))))
    c, _ = ki.ragged_cache(w, seg_len, salt=30 + seed)
    hc = host_cache(w, c)
    dc = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(S, L, H, H * G, D, hc.cap)
    q = ki.decode_inputs(w, seed)["q"]
    scale = 1.0 / math.sqrt(D)
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), scale)
    lb = int(rng.integers(0, L))
    le = int(rng.integers(lb + 1, L + 1))
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    kv.kvtrim_decode_attn(ctx, dc, q.to(DEV), lb, le, scale, out, lse)
    assert kv.kvtrim_poll_error(ctx) == 0
    o, l = out.cpu().numpy(), lse.cpu().numpy()
    outside = [x for x in range(L) if not lb <= x < le]
    assert np.all(o[:, outside] == 99.0) and np.all(l[:, outside] == 99.0)
    if np.abs(ref[:, lb:le]).max() > 0:
        assert attn_error(o[:, lb:le], ref[:, lb:le]) <= ATTN_TOL, (seed, seg_len.tolist(), lb, le)
    else:
        assert np.all(o[:, lb:le] == 0.0)
    fin = np.isfinite(ref_lse[:, lb:le])
    assert np.array_equal(np.isneginf(l[:, lb:le]), ~fin)
    if fin.any():
        assert np.abs(l[:, lb:le][fin] - ref_lse[:, lb:le][fin]).max() <= 2e-3


def test_attention_with_large_logits_stays_finite():
    w = wl(1, 1, 1, 4, 128)
    c, _ = ki.ragged_cache(w, [900], salt=10)
    c["k"] *= 6.0
    hc = host_cache(w, c)
    q = ki.decode_inputs(w, 1)["q"] * 6.0
    ctx = kv.Context(1, 1, 1, 4, 128, hc.cap)
    ref, _ = oracle.attend(hc, bf16_bits(q), 1.0)
    out = torch.zeros(ref.shape, dtype=torch.float32, device=DEV)
    kv.kvtrim_decode_attn(ctx, kv.Cache.from_dict(c, DEV), q.to(DEV), 0, 1, 1.0, out, None)
    o = out.cpu().numpy()
    assert np.isfinite(o).all() and attn_error(o, ref) <= ATTN_TOL


# ---------------------------------------------------------------------------------- error paths (kernels exit normally)

def test_device_side_errors_are_reported_and_nothing_overflows():
    w = wl(1, 1, 4, 2, 64)
    seg_len = [300, 10, 0, 500]
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=14)
    cap = sum(seg_len) + 4
    ctx = kv.Context(1, 1, 4, 8, 64, cap)
    src = kv.Cache.from_dict(c, DEV)
    keep = torch.ones(cap, dtype=torch.uint8, device=DEV)
    kept = torch.tensor(seg_len, dtype=torch.int32, device=DEV)
    small = kv.Cache.empty(4, 64, 700, DEV)
    small.k.fill_(1.0)
    kv.kvtrim_compact(ctx, src, keep, kept, small, 1)
    assert kv.kvtrim_poll_error(ctx) == -4                               # KVTRIM_ECAP
    assert torch.all(small.k == 1.0)                                     # nothing was written
    assert kv.kvtrim_poll_error(ctx) == 0                                # flag cleared
    big = kv.Cache.empty(4, 64, cap, DEV)
    wrong = kept.clone()
    wrong[0] -= 1
    kv.kvtrim_compact(ctx, src, keep, wrong, big, 1)
    assert kv.kvtrim_poll_error(ctx) == -5                               # KVTRIM_EMISMATCH
    # appending two tokens where one slot is reserved
    new = ki.decode_inputs(w, 0)
    two = lambda t: torch.stack([t, t], 1).contiguous().to(DEV)
    before = src.seg_len.clone()
    kv.kvtrim_append(ctx, src, two(new["k_new"]), two(new["v_new"]), two(new["log_beta_new"]),
                     torch.zeros(4, 2, dtype=torch.int32, device=DEV), 2)
    assert kv.kvtrim_poll_error(ctx) == -4
    assert torch.equal(src.seg_len, before)
    # an inconsistent segment table
    bad = kv.Cache(src.k, src.v, src.log_beta, src.pos, src.seg_start, torch.tensor([300, 10, 0, 900], dtype=torch.int32, device=DEV))
    score = torch.zeros(cap, dtype=torch.float32, device=DEV)
    kv.kvtrim_score(ctx, bad, now.to(DEV), score)
    kv.kvtrim_select_global(ctx, bad, score, torch.tensor([5], dtype=torch.int64, device=DEV), keep, kept)
    assert kv.kvtrim_poll_error(ctx) == -6                               # KVTRIM_ELAYOUT


@pytest.mark.parametrize("nseg", [6, 1500])
def test_compaction_rejects_overlapping_segments_and_leaves_the_destination_alone(nseg):
    # a segment that runs into its successor (still inside the buffers) must not reach the row movers, in either
    # form of the compaction scan (one block per segment summing all segments itself: up to 1024 segments; a prefix
    # kernel first: more); and a destination that is too small is left untouched, segment table included
    w = wl(1, 1, nseg, 1, 64)
    seg_len = [20] * nseg
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=3)
    cap = c["cap"]
    ctx = kv.Context(1, 1, nseg, nseg, 64, cap + 64)
    src = kv.Cache.from_dict(c, DEV)
    keep = torch.ones(cap, dtype=torch.uint8, device=DEV)
    kept = torch.tensor(seg_len, dtype=torch.int32, device=DEV)
    q = torch.zeros(1, 1, nseg, 64, dtype=torch.bfloat16, device=DEV)
    out = torch.zeros(1, 1, nseg, 64, dtype=torch.float32, device=DEV)

    def fresh(n):
        d = kv.Cache.empty(nseg, 64, n, DEV)
        d.k.fill_(1.0)
        d.seg_start.fill_(-7)
        d.seg_len.fill_(-7)
        return d

    small = fresh(sum(seg_len) + nseg - 1)                        # one slot short
    for call in ("compact", "compact_attn"):
        if call == "compact":
            kv.kvtrim_compact(ctx, src, keep, kept, small, 1)
        else:
            kv.kvtrim_compact_attn(ctx, src, keep, kept, small, 1, q, 0, 1, 0.125, out)
        assert kv.kvtrim_poll_error(ctx) == -4                    # KVTRIM_ECAP
        assert torch.all(small.k == 1.0) and torch.all(small.seg_start == -7) and torch.all(small.seg_len == -7)
    lens = src.seg_len.clone()
    lens[2] = 25                                                  # 4 entries into segment 3's range
    bad = kv.Cache(src.k, src.v, src.log_beta, src.pos, src.seg_start, lens)
    kept_bad = kept.clone()
    kept_bad[2] = 25
    big = fresh(cap + 64)
    for call in ("compact", "compact_attn", "inplace"):
        if call == "compact":
            kv.kvtrim_compact(ctx, bad, keep, kept_bad, big, 1)
        elif call == "compact_attn":
            kv.kvtrim_compact_attn(ctx, bad, keep, kept_bad, big, 1, q, 0, 1, 0.125, out)
        else:
            spare = kv.Cache.empty(nseg, 64, cap, DEV)
            before = bad.k.clone()
            kv.kvtrim_compact_attn_inplace(ctx, bad, keep, kept_bad, spare, q, 0, 1, 0.125, out)
            assert torch.equal(bad.k, before)
        assert kv.kvtrim_poll_error(ctx) == -6                    # KVTRIM_ELAYOUT
        assert torch.all(big.k == 1.0) and torch.all(big.seg_len == -7)


def test_host_side_argument_checks():
    ctx = kv.Context(1, 1, 2, 4, 64, 100)
    c = kv.Cache.empty(2, 64, 100, DEV)
    too_big = kv.Cache.empty(2, 64, 101, DEV)
    score = torch.zeros(101, dtype=torch.float32, device=DEV)
    now = torch.zeros(1, dtype=torch.int32, device=DEV)
    with pytest.raises(kv.KvtrimError) as e:
        kv.kvtrim_score(ctx, too_big, now, score)
    assert e.value.status == -1
    keep = torch.zeros(100, dtype=torch.uint8, device=DEV)
    kept = torch.zeros(2, dtype=torch.int32, device=DEV)
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_compact(ctx, c, keep, kept, c, 1)                      # src == dst
    q = torch.zeros(1, 1, 4, 64, dtype=torch.bfloat16, device=DEV)
    out = torch.zeros(1, 1, 4, 64, dtype=torch.float32, device=DEV)
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_decode_attn(ctx, c, q, 0, 2, 0.125, out)               # layer range beyond L
    with pytest.raises(kv.KvtrimError):
        kv.Context(1, 1, 2, 4, 96, 100)


def test_results_are_deterministic_across_runs():
    w = ki.workload("llama", prefill=500)
    a = run_steps_both(w, steps=2, budget=w.budget, device=DEV)
    b = run_steps_both(w, steps=2, budget=w.budget, device=DEV)
    check(a)
    assert [r["attn_err"] for r in a] == [r["attn_err"] for r in b]


# ---------------------------------------------------------------------------------- soft attention, occupancy

@pytest.mark.parametrize("D,G,S", [(128, 4, 1), (64, 2, 2), (128, 7, 2)])
def test_soft_retention_gated_attention_and_occupancy(D, G, S):
    w = wl(S, 2, 2, G, D)
    rng = np.random.default_rng(D + G + S)
    seg_len = rng.integers(0, 1800, w.nseg)
    seg_len[1] = 0
    c, now = ki.ragged_cache(w, seg_len, salt=40 + G)
    hc = host_cache(w, c)
    dc = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, D, hc.cap)
    q = ki.decode_inputs(w, 2)["q"]
    scale = 1.0 / math.sqrt(D)
    now_np = now.numpy() + 3
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), scale, soft_now=now_np)
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    now_dev = torch.from_numpy(now_np).to(DEV)
    kv.kvtrim_decode_attn_soft(ctx, dc, q.to(DEV), now_dev, 0, w.n_layers, scale, out, lse)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert attn_error(out.cpu().numpy(), ref) <= ATTN_TOL
    fin = np.isfinite(ref_lse)
    assert np.abs(lse.cpu().numpy()[fin] - ref_lse[fin]).max() <= 2e-3
    assert np.array_equal(np.isneginf(lse.cpu().numpy()), np.isneginf(ref_lse))
    # the soft form differs from the hard one on this input, and beta = 1 makes them coincide
    hard, _ = oracle.attend(hc, bf16_bits(q), scale)
    assert attn_error(out.cpu().numpy(), hard) > 10 * ATTN_TOL
    ones = dict(c)
    ones["log_beta"] = torch.zeros_like(c["log_beta"])
    out1 = torch.zeros_like(out)
    out2 = torch.zeros_like(out)
    d1 = kv.Cache.from_dict(ones, DEV)
    kv.kvtrim_decode_attn_soft(ctx, d1, q.to(DEV), now_dev, 0, w.n_layers, scale, out1)
    kv.kvtrim_decode_attn(ctx, d1, q.to(DEV), 0, w.n_layers, scale, out2)
    assert torch.equal(out1, out2)
    # occupancy
    occ = torch.zeros(S, dtype=torch.float64, device=DEV)
    kv.kvtrim_occupancy(ctx, dc, now_dev, occ)
    np.testing.assert_allclose(occ.cpu().numpy(), oracle.occupancy(hc, now_np), rtol=2e-6)


def test_many_segments_take_the_prefix_kernel_and_report_errors():
    # more than 1024 segments: the segment prefixes of the compaction come from one extra block instead of a
    # reduction in every block; results and device-side errors must be the same
    w = wl(9, 8, 16, 1, 64)                                        # 1152 segments
    rng = np.random.default_rng(77)
    seg_len = rng.integers(0, 40, w.nseg)
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=8)
    per_seq = [int(seg_len[s * 128:(s + 1) * 128].sum()) for s in range(9)]
    check(run_steps_both(w, steps=2, budget=[max(1, n // 2) for n in per_seq], device=DEV, cache_dict=c, now0=now.numpy(),
                         fused=True))
    hc = host_cache(w, c)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, w.head_dim, hc.cap)
    src = kv.Cache.from_dict(c, DEV)
    keep = torch.ones(hc.cap, dtype=torch.uint8, device=DEV)
    kept = torch.from_numpy(hc.seg_len.copy()).to(DEV)
    small = kv.Cache.empty(w.nseg, w.head_dim, int(hc.seg_len.sum()) // 2, DEV)
    kv.kvtrim_compact(ctx, src, keep, kept, small, 0)
    assert kv.kvtrim_poll_error(ctx) == -4                         # destination too small
    roomy = kv.Cache.empty(w.nseg, w.head_dim, hc.cap, DEV)
    kept[5] += 1
    kv.kvtrim_compact(ctx, src, keep, kept, roomy, 0)
    assert kv.kvtrim_poll_error(ctx) == -5                         # kept disagrees with the mask
    kept[5] -= 1
    kv.kvtrim_compact(ctx, src, keep, kept, roomy, 0)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert compare_caches(device_cache_to_host(w, roomy), oracle.compact(hc, np.ones(hc.cap, np.uint8), hc.cap, 0))


@pytest.mark.parametrize("S,L,H,G,D,layers", [(257, 4, 4, 2, 64, (0, 4)),       # 4112 segments: the table kernel runs first
                                              (256, 4, 4, 2, 64, (0, 4)),       # 4096: every block adds up the lengths itself
                                              (512, 3, 4, 1, 64, (1, 2)),       # ... of a layer range of a longer table
                                              (1, 2, 2, 3, 128, (0, 2))])
def test_attention_over_many_segments(S, L, H, G, D, layers):
    # segments of 0 to 150 entries (under, at and over a round of 64 rows), so that shares end everywhere in them
    w = wl(S, L, H, G, D)
    rng = np.random.default_rng(S + L)
    seg_len = rng.choice([0, 1, 15, 16, 17, 63, 64, 65, 128, 150], w.nseg)
    c, _ = ki.ragged_cache(w, seg_len, salt=41)
    hc = host_cache(w, c)
    ctx = kv.Context(S, L, H, H * G, D, hc.cap)
    q = ki.decode_inputs(w, 0)["q"]
    scale = 1.0 / math.sqrt(D)
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), scale)
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    kv.kvtrim_decode_attn(ctx, kv.Cache.from_dict(c, DEV), q.to(DEV), *layers, scale, out, lse)
    assert kv.kvtrim_poll_error(ctx) == 0
    inside, outside = slice(*layers), [x for x in range(L) if not layers[0] <= x < layers[1]]
    o, l = out.cpu().numpy(), lse.cpu().numpy()
    assert np.all(o[:, outside] == 99.0) and np.all(l[:, outside] == 99.0)
    assert attn_error(o[:, inside], ref[:, inside]) <= ATTN_TOL
    fin = np.isfinite(ref_lse[:, inside])
    assert np.array_equal(np.isneginf(l[:, inside]), ~fin)
    assert np.abs(l[:, inside][fin] - ref_lse[:, inside][fin]).max() <= 2e-3


def test_attention_on_a_bad_table_outside_the_layer_range_gives_no_result():
    # a segment table that overlaps in a layer that is not asked for: the call reports it and writes nothing
    w = wl(1, 2, 2, 2, 64)
    c, _ = ki.ragged_cache(w, [100, 200, 300, 50], salt=42)
    ctx = kv.Context(1, 2, 2, 4, 64, c["cap"])
    q = ki.decode_inputs(w, 0)["q"].to(DEV)
    out = torch.full((1, 2, 4, 64), 99.0, dtype=torch.float32, device=DEV)
    c["seg_len"][0] = 150
    kv.kvtrim_decode_attn(ctx, kv.Cache.from_dict(c, DEV), q, 1, 2, 0.125, out, None)
    assert kv.kvtrim_poll_error(ctx) == -6                               # KVTRIM_ELAYOUT
    assert torch.all(out == 99.0)


# Rounds of 128 rows, shares that start at multiples of 128 to 16 rows, segments of one round undivided, merges in tiles of
# RG * 16 results (16 at 8 heads and D = 128, 64 at one head), at most 64 segments and 128 KB of results a segment in one
# launch: lengths on both sides of each, 64 and 65 segments, and the same call again on counters that the first left behind.
@pytest.mark.parametrize("S,H,G,D,lens,soft", [
    (1, 16, 4, 128, [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 130, 255, 256, 257, 2100], False),
    (1, 2, 8, 128, [5000, 100], False),                           # 39 results to merge, more than two tiles of 16: in groups of 32
    (1, 1, 1, 64, [9000], True),                                  # 70 results: a tile of 64 and the rest
    (1, 3, 3, 128, [0, 0, 4097], True),
    (4, 16, 2, 64, [40, 0, 300, 16], False),                      # 64 segments, most shorter than a round
    (5, 13, 2, 64, [40, 0, 300, 16], False),                      # 65: two launches
    (2, 2, 4, 128, [0], False)])                                  # nothing retained at all
def test_attention_of_small_calls_at_the_edges_of_their_shares(S, H, G, D, lens, soft):
    w = wl(S, 2, H, G, D)
    seg_len = [lens[g % len(lens)] for g in range(w.nseg)]
    c, now = ki.ragged_cache(w, seg_len, reserve=1, salt=50 + G)
    hc = host_cache(w, c)
    dc = kv.Cache.from_dict(c, DEV)
    ctx = kv.Context(S, 2, H, H * G, D, hc.cap)
    q = ki.decode_inputs(w, 1)["q"]
    now_np = now.numpy() + 2
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), 0.1, soft_now=now_np if soft else None)
    out = torch.full(ref.shape, 99.0, dtype=torch.float32, device=DEV)
    lse = torch.full(ref_lse.shape, 99.0, dtype=torch.float32, device=DEV)
    now_dev, qd = torch.from_numpy(now_np).to(DEV), q.to(DEV)

    def call(cache, layer, lse=lse):
        if soft:
            kv.kvtrim_decode_attn_soft(ctx, cache, qd, now_dev, layer, layer + 1, 0.1, out, lse)
        else:
            kv.kvtrim_decode_attn(ctx, cache, qd, layer, layer + 1, 0.1, out, lse)

    # a table that is unusable, and the sticky flag it leaves: no result, and nothing counted
    bad_len = dc.seg_len.clone()
    bad_len[w.nseg - 1] = 10 ** 6
    call(kv.Cache(dc.k, dc.v, dc.log_beta, dc.pos, dc.seg_start, bad_len), 0)
    call(dc, 1)
    assert torch.all(out == 99.0) and torch.all(lse == 99.0)
    assert kv.kvtrim_poll_error(ctx) == -6                               # KVTRIM_ELAYOUT
    got = []
    for again in range(3):
        out.fill_(99.0)
        for layer in range(2):
            call(dc, layer, lse if again < 2 else None)
        assert kv.kvtrim_poll_error(ctx) == 0
        got.append(out.cpu().numpy())
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
    fin = np.isfinite(ref_lse)
    l = lse.cpu().numpy()
    assert np.array_equal(np.isneginf(l), ~fin) and np.all(got[0][~fin] == 0.0)
    if fin.any():
        assert attn_error(got[0], ref) <= ATTN_TOL
        assert np.abs(l[fin] - ref_lse[fin]).max() <= 2e-3


# One launch goes by the mean list; a list far longer than that has more results than one block merges (four tiles of 16 at 8
# heads and D = 128): groups of 32 meet first.  64 and 65 results (one group more, of one result), two long lists that
# share a block, several wide groups, tiles of 64 results, a longest list that is all of the call; hard, soft and on pages.
@pytest.mark.parametrize("H,G,D,lens", [
    (4, 8, 128, [8319, 0, 0, 0]), (4, 8, 128, [0, 8320, 0, 0]), (8, 8, 128, [0, 9000, 9001, 0, 0, 1, 0, 0]),
    (16, 4, 128, [30000] + [17] * 15), (32, 1, 64, [3] * 31 + [34000]), (16, 3, 64, [0] * 8 + [26001, 129] + [0] * 6)])
def test_attention_of_a_list_that_outgrows_the_others(H, G, D, lens):
    w = wl(1, 1, H, G, D)
    c, now = ki.ragged_cache(w, lens, reserve=1, salt=70 + G)
    hc = host_cache(w, c)
    dc = kv.Cache.from_dict(c, DEV)
    n_pages = sum((n + 127) // 128 for n in lens)
    pages = kv.PagedCache(H, D, n_pages + 3, (max(lens) + 127) // 128, DEV)
    ctx = kv.Context(1, 1, H, H * G, D, max(hc.cap, pages.slots))
    q = ki.decode_inputs(w, 1)["q"]
    qd, now_np = q.to(DEV), now.numpy() + 2
    now_dev = torch.from_numpy(now_np).to(DEV)
    kv.kvtrim_paged_build(ctx, dc, torch.ones(hc.cap, dtype=torch.uint8, device=DEV), dc.seg_len, pages)
    assert kv.kvtrim_poll_error(ctx) == 0
    for soft, call in ((False, lambda o, l: kv.kvtrim_decode_attn(ctx, dc, qd, 0, 1, 0.1, o, l)),
                       (True, lambda o, l: kv.kvtrim_decode_attn_soft(ctx, dc, qd, now_dev, 0, 1, 0.1, o, l)),
                       (False, lambda o, l: kv.kvtrim_paged_attn(ctx, pages, qd, 0, 1, 0.1, o, l))):
        ref, ref_lse = oracle.attend(hc, bf16_bits(q), 0.1, soft_now=now_np if soft else None)
        fin = np.isfinite(ref_lse)
        got = []
        for again in range(3):                                    # on the counters that the call before left
            out, lse = (torch.full(r.shape, 99.0, device=DEV) for r in (ref, ref_lse))
            call(out, lse)
            assert kv.kvtrim_poll_error(ctx) == 0
            got.append((out.cpu().numpy(), lse.cpu().numpy()))
        assert all(np.array_equal(x, y) for g in got[1:] for x, y in zip(g, got[0]))
        o, l = got[0]
        assert attn_error(o, ref) <= ATTN_TOL and np.abs(l[fin] - ref_lse[fin]).max() <= 2e-3
        assert np.array_equal(np.isneginf(l), ~fin) and np.all(o[~fin] == 0.0)


# A list of up to three rounds of 128 rows (four at D = 64) is one block's: lengths on both sides of the line, short lists whose
# blocks also take the beginning or the end of a long one, and nothing else; hard, soft and on pages.
@pytest.mark.parametrize("H,G,D,lens", [
    (8, 4, 128, [384, 385, 383, 129, 256, 257, 1, 0]), (12, 8, 128, [384] * 5 + [3000] + [385] * 3 + [384, 2000, 384]),
    (8, 6, 64, [512, 513, 511, 385, 384, 640, 0, 127]), (3, 1, 64, [512, 2100, 512]), (1, 2, 128, [384])])
def test_attention_of_lists_that_one_block_takes(H, G, D, lens):
    test_attention_of_a_list_that_outgrows_the_others(H, G, D, lens)


# On pages a round less from 17 lists on (9 at D = 64): the lists of the last round are divided there, ragged ones stay whole.
@pytest.mark.parametrize("H,D,lens", [(16, 128, [384, 257, 300, 100]), (17, 128, [384, 257, 300, 256, 255]), (40, 128, [384, 0, 129]),
                                      (8, 64, [512, 385, 400]), (9, 64, [512, 385, 384, 1]), (33, 64, [500, 130, 384])])
def test_attention_on_pages_of_many_lists_of_few_rounds(H, D, lens):
    test_attention_of_a_list_that_outgrows_the_others(H, 4, D, [lens[i % len(lens)] for i in range(H)])


# out and lse are arrays of floats and need no more than their alignment, also where the last block of a segment merges:
# attention of a small call (2200 and 40 rows a list), of the row mover (18 chunks and 1), of segments that one block writes
@pytest.mark.parametrize("G,D", [(4, 128), (3, 64)])
def test_attention_results_may_lie_at_any_float(G, D):
    w = wl(1, 2, 2, G, D)
    lens = [2200, 40, 1100, 130]
    c, now = ki.ragged_cache(w, lens, reserve=1, salt=60 + G)
    hc = host_cache(w, c)
    dc, dst = kv.Cache.from_dict(c, DEV), kv.Cache.empty(w.nseg, D, hc.cap, DEV)
    ctx = kv.Context(1, 2, 2, 2 * G, D, hc.cap)
    q = ki.decode_inputs(w, 1)["q"]
    ref, ref_lse = oracle.attend(hc, bf16_bits(q), 0.1)
    qd = q.to(DEV)
    keep = torch.ones(hc.cap, dtype=torch.uint8, device=DEV)
    kept = torch.tensor(lens, dtype=torch.int32, device=DEV)

    def layers(out, lse):
        for layer in range(2):
            kv.kvtrim_decode_attn(ctx, dc, qd, layer, layer + 1, 0.1, out, lse)

    def mover(out, lse):
        kv.kvtrim_compact_attn(ctx, dc, keep, kept, dst, 0, qd, 0, 2, 0.1, out, lse)
    for call in (layers, mover):
        first = None
        for off in range(4):
            bufs = [torch.full((r.size + 8,), 99.0, device=DEV) for r in (ref, ref_lse)]
            out, lse = (b[off:off + r.size].view(r.shape) for b, r in zip(bufs, (ref, ref_lse)))
            assert out.data_ptr() % 16 == 4 * off
            call(out, lse)
            assert kv.kvtrim_poll_error(ctx) == 0
            got = [b.cpu().numpy() for b in bufs]
            for g, r in zip(got, (ref, ref_lse)):
                assert np.all(g[:off] == 99.0) and np.all(g[off + r.size:] == 99.0), (call.__name__, off)
            got = [g[off:off + r.size].reshape(r.shape) for g, r in zip(got, (ref, ref_lse))]
            assert attn_error(got[0], ref) <= ATTN_TOL and np.abs(got[1] - ref_lse).max() <= 2e-3
            first = first or got
            assert all(np.array_equal(a, b) for a, b in zip(first, got)), (call.__name__, off)


@pytest.mark.parametrize("reserve,lens", [
    (3, [0, 1, 15, 16, 17, 127, 128, 129]),                  # under, at and over a lane's 16 mask bytes and a chunk; every start misaligned differently
    (1, [1023, 1024, 1025, 2047, 2048, 2049, 4095, 8]),      # ... a wavefront's load (8 chunks) and a selection chunk
    (2, [65536, 65537, 131072, 131073, 5, 70000, 1, 3]),     # ... half a tile and a tile of 1024 chunks of the scan
])
@pytest.mark.parametrize("keep_part", [2, 40])               # a block per source chunk / the gathering form
def test_selection_and_compaction_at_the_edges_of_their_tiles(reserve, lens, keep_part):
    w = wl(1, 2, 4, 2, 64)
    c, now = ki.ragged_cache(w, lens, reserve=reserve, salt=50)
    hc = host_cache(w, c)
    total = sum(lens)
    budget = np.array([max(total // keep_part, 1)], dtype=np.int64)
    score = oracle.score(hc, now.numpy())
    keep, kept, thr = oracle.select(hc, score, budget)
    ctx = kv.Context(1, 2, 4, 8, 64, hc.cap)
    src = kv.Cache.from_dict(c, DEV)
    d_score = torch.zeros(hc.cap, dtype=torch.float32, device=DEV)
    d_keep = torch.full((hc.cap,), 7, dtype=torch.uint8, device=DEV)
    d_kept = torch.zeros(w.nseg, dtype=torch.int32, device=DEV)
    d_thr = torch.zeros(1, dtype=torch.int32, device=DEV)
    kv.kvtrim_score_select(ctx, src, now.to(DEV), torch.from_numpy(budget).to(DEV), d_score, d_keep, d_kept, d_thr)
    dst = kv.Cache.empty(w.nseg, 64, int(kept.sum()) + w.nseg * reserve, DEV)
    kv.kvtrim_compact(ctx, src, d_keep, d_kept, dst, reserve)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert np.array_equal(d_kept.cpu().numpy(), kept)
    assert int(d_thr.cpu().numpy().view(np.uint32)[0]) == int(thr[0])
    k = d_keep.cpu().numpy()
    inside = np.zeros(hc.cap, dtype=bool)
    starts, cursor = c["seg_start"].tolist(), 0
    for g, (s, n) in enumerate(zip(starts, lens)):
        inside[s:s + n] = True
        assert np.array_equal(k[s:s + n], keep[s:s + n])
        m = torch.from_numpy(keep[s:s + n].astype(bool))
        here = slice(cursor, cursor + int(kept[g]))
        for name in ("k", "v", "log_beta", "pos"):
            assert torch.equal(getattr(dst, name)[here].cpu(), c[name][s:s + n][m])
        cursor += int(kept[g]) + reserve
    assert np.all(k[~inside] == 7)                           # slots outside the segments are not written


@pytest.mark.parametrize("cap", [1, 3, 4, 5])
def test_more_segments_than_a_long_mask_needs_over_a_handful_of_entries(cap):
    # the chunk bound (a chunk per segment) asks for the mask kernel's long form, whose 16-byte loads a cache of fewer
    # than four entries must not see
    w = wl(2, 32, 130, 1, 64)                                # 8320 segments
    seg_len = np.zeros(w.nseg, dtype=np.int64)
    seg_len[[5, 4159, 4160, 8319, 17][:cap]] = 1
    c, now = ki.ragged_cache(w, seg_len, reserve=0, salt=51)
    hc = host_cache(w, c)
    assert hc.cap == cap
    budget = np.array([1, 1], dtype=np.int64)
    score = oracle.score(hc, now.numpy())
    keep, kept, thr = oracle.select(hc, score, budget)
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, 64, cap)
    d_score = torch.zeros(cap, dtype=torch.float32, device=DEV)
    d_keep = torch.full((cap,), 7, dtype=torch.uint8, device=DEV)
    d_kept = torch.zeros(w.nseg, dtype=torch.int32, device=DEV)
    d_thr = torch.zeros(2, dtype=torch.int32, device=DEV)
    kv.kvtrim_score_select(ctx, kv.Cache.from_dict(c, DEV), now.to(DEV), torch.from_numpy(budget).to(DEV), d_score, d_keep, d_kept, d_thr)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert np.array_equal(d_score.cpu().numpy().view(np.uint32), score.view(np.uint32))
    assert np.array_equal(d_keep.cpu().numpy(), keep) and np.array_equal(d_kept.cpu().numpy(), kept)
    assert np.array_equal(d_thr.cpu().numpy().view(np.uint32), thr)


@pytest.mark.parametrize("keep_part", [2, 40])               # a block per source chunk / the gathering form
def test_compaction_of_many_segments_at_the_edges_of_their_tiles(keep_part):
    # more than 1024 segments: the scan takes a segment in tiles of 256 chunks = 32768 entries
    w = wl(9, 8, 16, 1, 64)                                  # 1152 segments
    rng = np.random.default_rng(keep_part)
    seg_len = rng.choice([0, 1, 15, 16, 127, 128, 129, 300], w.nseg)
    for g, n in {0: 32767, 3: 32768, 4: 32769, 700: 65537, 1151: 33000}.items():
        seg_len[g] = n
    c, _ = ki.ragged_cache(w, seg_len, reserve=1, salt=52)
    hc = host_cache(w, c)
    keep = np.zeros(hc.cap, np.uint8)
    kept = np.zeros(w.nseg, np.int32)
    for g, (s, n) in enumerate(zip(hc.seg_start, hc.seg_len)):
        keep[s:s + n] = rng.random(n) < 1 / keep_part
        kept[g] = keep[s:s + n].sum()
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, 64, hc.cap)
    dst = kv.Cache.empty(w.nseg, 64, int(kept.sum()) + w.nseg, DEV)
    args = (ctx, kv.Cache.from_dict(c, DEV), torch.from_numpy(keep).to(DEV), torch.from_numpy(kept).to(DEV), dst, 1)
    kv.kvtrim_compact(*args)
    assert kv.kvtrim_poll_error(ctx) == 0
    assert compare_caches(device_cache_to_host(w, dst), oracle.compact(hc, keep, dst.cap, 1))


@pytest.mark.parametrize("shift", [0, 1])                    # the mask kernel's long form / a score array it cannot load 16 bytes from
def test_long_mask_over_uneven_segments(shift):
    # 8400 segments, so that a block walks runs of chunks: across empty, tiny and longer ones (2049: two chunks) and from
    # sequence to sequence - one with an ordinary threshold, one that keeps nothing, one with ties to rank inside the runs,
    # one that keeps everything; the last group of four entries ends behind the arrays
    w = wl(4, 30, 70, 1, 64)
    rng = np.random.default_rng(53)
    seg_len = rng.choice([0, 1, 3, 4, 5, 7, 2049], w.nseg, p=[.2, .2, .2, .1, .1, .19, .01])
    seg_len[-1] = 7
    seg_len[0] += (3 - int((seg_len + 1).sum())) % 4
    start = np.concatenate([[0], np.cumsum(seg_len + 1)[:-1]])
    cap = int((seg_len + 1).sum())
    assert cap % 4 == 3
    log_beta = -rng.random(cap).astype(np.float32)
    log_beta[start[2 * 2100]:start[3 * 2100]] = -0.25 * rng.integers(1, 3, start[3 * 2100] - start[2 * 2100])
    c = {"k": torch.zeros(cap, 64, dtype=torch.bfloat16), "v": torch.zeros(cap, 64, dtype=torch.bfloat16),
         "log_beta": torch.from_numpy(log_beta), "pos": torch.from_numpy((np.arange(cap) - np.repeat(start, seg_len + 1)).astype(np.int32)),
         "seg_start": torch.from_numpy(start), "seg_len": torch.from_numpy(seg_len.astype(np.int32)), "cap": cap}
    hc = host_cache(w, c)
    per_seq = seg_len.reshape(4, -1).sum(1)
    budget = np.array([per_seq[0] // 3, 0, per_seq[2] // 2, per_seq[3]], dtype=np.int64)
    score = oracle.score(hc, np.full(4, 3000, dtype=np.int32))
    keep, kept, thr = oracle.select(hc, score, budget)
    live = live_mask(hc)
    d_score = torch.zeros(cap + shift, dtype=torch.float32, device=DEV)
    d_score[shift:].copy_(torch.from_numpy(score))
    ctx = kv.Context(w.n_seq, w.n_layers, w.n_kv_heads, w.n_q_heads, 64, cap)
    d_keep = torch.full((cap,), 7, dtype=torch.uint8, device=DEV)
    d_kept = torch.zeros(w.nseg, dtype=torch.int32, device=DEV)
    d_thr = torch.zeros(4, dtype=torch.int32, device=DEV)
    kv.kvtrim_select_global(ctx, kv.Cache.from_dict(c, DEV), d_score[shift:], torch.from_numpy(budget).to(DEV), d_keep, d_kept, d_thr)
    assert kv.kvtrim_poll_error(ctx) == 0
    k = d_keep.cpu().numpy()
    assert np.array_equal(k[live], keep[live]) and np.all(k[~live] == 7)
    assert np.array_equal(d_kept.cpu().numpy(), kept)
    assert np.array_equal(d_thr.cpu().numpy().view(np.uint32), thr)
    tied = score[live & (np.arange(cap) >= start[2 * 2100]) & (np.arange(cap) < start[3 * 2100])]
    last = np.sort(tied)[::-1][budget[2] - 1]
    assert (tied == last).sum() > 1 and (tied >= last).sum() > budget[2]   # (fewer survive than tie at the threshold)


# The error against 64 bits of a list of several rounds that one block takes is that of a list divided into rounds: kvtrim_compact_attn on
# the same rows, which has a maximum for every 16 of them and a partial result for every 128.  Both lose what a probability loses
# as two bf16 terms, 1.5e-6 of the result as a mean over 640 heads; with one maximum for all rounds it was 4 to 18 % more at these
# lengths, and means over such samples differ by less than 1 %.
@pytest.mark.parametrize("D,rows", [(128, 128), (128, 240), (128, 300), (128, 384), (128, 385), (64, 240), (64, 384), (64, 500), (64, 512), (64, 513)])
def test_attention_error_of_undivided_lists_is_that_of_divided_ones(D, rows):
    H = G = 8
    n = H * rows
    err = np.zeros(4)
    for seed in range(10):
        g = torch.Generator(device=DEV).manual_seed(1000 * seed + rows)
        k, v = (torch.randn(n, D, generator=g, device=DEV).bfloat16() for _ in range(2))
        q = torch.randn(1, 1, H * G, D, generator=g, device=DEV).bfloat16()
        lens = torch.full((H,), rows, dtype=torch.int32, device=DEV)
        c = kv.Cache(k, v, torch.zeros(n, device=DEV), torch.arange(rows, dtype=torch.int32, device=DEV).repeat(H), torch.arange(H, device=DEV) * rows, lens)
        pages = (rows + 127) // 128
        pc, dst = kv.PagedCache(H, D, H * pages, pages, DEV), kv.Cache.empty(H, D, n, DEV)
        ctx = kv.Context(1, 1, H, H * G, D, max(n, pc.slots))
        keep = torch.ones(n, dtype=torch.uint8, device=DEV)
        now = torch.full((1,), rows, dtype=torch.int32, device=DEV)
        kv.kvtrim_paged_build(ctx, c, keep, lens, pc)
        out = [torch.zeros(1, 1, H * G, D, device=DEV) for _ in range(4)]
        lse = [torch.zeros(1, 1, H * G, device=DEV) for _ in range(4)]
        s = D ** -0.5
        kv.kvtrim_decode_attn(ctx, c, q, 0, 1, s, out[0], lse[0])
        kv.kvtrim_decode_attn_soft(ctx, c, q, now, 0, 1, s, out[1], lse[1])   # (beta = 1: the same sums)
        kv.kvtrim_paged_attn(ctx, pc, q, 0, 1, s, out[2], lse[2])
        kv.kvtrim_compact_attn(ctx, c, keep, lens.clone(), dst, 0, q, 0, 1, s, out[3], lse[3])
        assert kv.kvtrim_poll_error(ctx) == 0
        kd, vd, qd = (x.cpu().double().view(H, -1, D) for x in (k, v, q))
        z = torch.matmul(qd, kd.transpose(1, 2).contiguous()) * s
        ref = torch.matmul(torch.softmax(z, -1), vd)
        for i in range(4):
            err[i] += float((out[i].cpu().double().view(H, G, D) - ref).norm() / ref.norm()) / 10
            assert float((lse[i].cpu().double().view(H, G) - torch.logsumexp(z, -1)).abs().max()) < 5e-6
    assert np.all(err[:3] <= 1.02 * err[3]) and err[3] < 1.7e-6, err


# Tiles whose largest logits lie far apart, in both directions and with a tile that counts for nothing: in a list of several rounds each
# is relative to its own, or 2^8 below the tile's before.  V up to 1e37: the sums stay below what they are relative to the largest.
@pytest.mark.parametrize("D,rows", [(128, 384), (128, 300), (64, 512)])
@pytest.mark.parametrize("step", [-30.0, -5.0, 5.0, 30.0, -300.0, 300.0])
def test_attention_of_undivided_lists_with_rising_and_falling_logits(D, rows, step):
    H, G = 4, 3
    n = H * rows
    g = torch.Generator().manual_seed(rows)
    k, v = (torch.randn(n, D, generator=g) for _ in range(2))
    q = torch.randn(H * G, D, generator=g)
    q[:, 0] = 8.0
    k[:, 0] = (torch.arange(rows) // 128).float().repeat(H) * step * D ** 0.5 / 8.0   # (logits a round apart by `step`)
    v *= 1e37 / 4
    k, v, q = k.bfloat16(), v.bfloat16(), q.bfloat16()
    lens = torch.full((H,), rows, dtype=torch.int32, device=DEV)
    c = kv.Cache(k.to(DEV), v.to(DEV), torch.zeros(n, device=DEV), torch.arange(rows, dtype=torch.int32).repeat(H).to(DEV), torch.arange(H, device=DEV) * rows, lens)
    ctx = kv.Context(1, 1, H, H * G, D, n)
    out, lse = torch.zeros(1, 1, H * G, D, device=DEV), torch.zeros(1, 1, H * G, device=DEV)
    kv.kvtrim_decode_attn(ctx, c, q.view(1, 1, H * G, D).to(DEV), 0, 1, D ** -0.5, out, lse)
    assert kv.kvtrim_poll_error(ctx) == 0
    kd, vd, qd = (x.double().view(H, -1, D) for x in (k, v, q))
    z = torch.matmul(qd, kd.transpose(1, 2).contiguous()) * D ** -0.5
    ref = torch.matmul(torch.softmax(z, -1), vd)
    got = out.cpu().double().view(H, G, D)
    assert torch.isfinite(got).all() and float((got - ref).norm() / ref.norm()) < 2e-4   # (logits of hundreds in fp32)
    assert float((lse.cpu().double().view(H, G) - torch.logsumexp(z, -1)).abs().max()) < 2e-4


# The row mover's q.k on the matrix cores (out of place, and in place with many heads) is no less accurate than as packed dot products,
# which the in-place form takes with few heads: logits of +-10, where the sum over the columns shows in the result.
@pytest.mark.parametrize("D,G", [(128, 1), (128, 4), (128, 6), (64, 2)])
def test_row_mover_error_with_large_logits(D, G):
    H, rows = 32, 1000
    n = H * rows
    err = np.zeros(2)
    for seed in range(6):
        g = torch.Generator(device=DEV).manual_seed(seed)
        k, v = (torch.randn(n, D, generator=g, device=DEV).bfloat16() for _ in range(2))
        q = (3.0 * torch.randn(1, 1, H * G, D, generator=g, device=DEV)).bfloat16()
        lens = torch.full((H,), rows, dtype=torch.int32, device=DEV)
        c = kv.Cache(k, v, torch.zeros(n, device=DEV), torch.arange(rows, dtype=torch.int32, device=DEV).repeat(H), torch.arange(H, device=DEV) * rows, lens)
        dst, ctx = kv.Cache.empty(H, D, n, DEV), kv.Context(1, 1, H, H * G, D, n)
        keep = torch.ones(n, dtype=torch.uint8, device=DEV)
        out = [torch.zeros(1, 1, H * G, D, device=DEV) for _ in range(2)]
        kv.kvtrim_compact_attn(ctx, c, keep, lens.clone(), dst, 0, q, 0, 1, D ** -0.5, out[0])
        kv.kvtrim_compact_attn_inplace(ctx, c, keep, lens.clone(), dst, q, 0, 1, D ** -0.5, out[1])
        assert kv.kvtrim_poll_error(ctx) == 0
        kd, vd, qd = (x.cpu().double().view(H, -1, D) for x in (k, v, q))
        ref = torch.matmul(torch.softmax(torch.matmul(qd, kd.transpose(1, 2).contiguous()) * D ** -0.5, -1), vd)
        for i in range(2):
            err[i] += float((out[i].cpu().double().view(H, G, D) - ref).norm() / ref.norm()) / 6
    assert err[0] <= 1.03 * err[1], err                           # (as one chain of MFMAs 1.05 at D = 64, 1.15 to 1.2 at 128)
