// Stage 2: one global top-B selection per sequence (Sec. 4.2, eviction rule) - the general form, for any
// number of evictions (the decode-step form, which looks only for the few lowest entries, is in k_fastsel.hip).
//
// Exact selection by a three-pass most-significant-digit radix select (11 + 11 + 10 bits)
// on the order-preserving uint32 image of the fp32 score.  Each pass builds per-block
// histograms in LDS and merges them with device-scope atomics into replicated global histograms.
// Every block of pass p + 1 finds the digit of pass p itself, by walking the merged histogram of
// pass p in its prologue; behind the last pass a block per sequence fixes the final digit, the
// threshold key and the tie quota.
// The first pass can compute the score on the fly (stage 1 fused: it reads log beta and the
// position instead of a score array and writes the score out as it goes).
// Entries above the threshold are kept; entries equal to it are kept in storage order
// (segment ascending, position ascending = layer, head, position) until the budget is
// met.  When every entry equal to the threshold fits (the usual case) the mask is a plain
// comparison; otherwise an ordered count of ties per chunk and an exclusive scan over the
// chunks rank them.  Small caches take all of this in one launch (k_sel_small, below).
#include <type_traits>

#include "kvtrim_device.h"

namespace kvtrim {

constexpr int SEL_THREADS = 256;      // mask kernel: one chunk per block, 8 entries per thread
constexpr int CNT_THREADS = 1024;
constexpr int HIST_THREADS = 1024;    // histogram passes: few fat blocks, so that few device-scope
constexpr int HIST_BLOCKS = HIST_BLOCKS_MAX;   // atomics meet on one address when the LDS histograms are merged
                                      // (the merged histogram is also kept in HIST_REPLICAS copies)
constexpr int PLAN_TABLE_BLOCKS = 8;  // blocks of the plan kernel that share the filling of the chunk table
constexpr int PLAN_ZERO_BLOCKS = 8;   // extra blocks of the plan kernel that clear the histograms
constexpr int MASK_BLOCKS = 1536;     // most blocks of the mask kernel's long form (six per compute unit, what fits at once)
constexpr int MASK_LONG = 8192;       // chunks from which it pays (16 K chunks: 30 us against 57; 6 K: 17.9 against 15.4)

// The sequence that chunk `ch` belongs to.
__device__ __forceinline__ int seq_of_chunk(const int32_t* prefix, const Shape& sh, int ch) {
    int lo = 0, hi = sh.n_seq;                                    // prefix[lo * segs] <= ch < prefix[hi * segs]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid * sh.segs_per_seq] <= ch) lo = mid;
        else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(1024) void k_sel_plan(CacheView c, Shape sh, const int64_t* __restrict__ budget,
                                                   Workspace ws, int32_t* __restrict__ kept_out,
                                                   uint32_t* __restrict__ thr_out, int hist_blocks) {
    if (blockIdx.x >= PLAN_TABLE_BLOCKS) {     // clear the (replicated) histograms of the three passes
        const int64_t n = (int64_t)3 * HIST_REPLICAS * sh.n_seq * RADIX_BINS;   // 65536 sequences: 3.2 G words
        for (int64_t i = (blockIdx.x - PLAN_TABLE_BLOCKS) * blockDim.x + threadIdx.x; i < n; i += (gridDim.x - PLAN_TABLE_BLOCKS) * blockDim.x)
            ws.hist[i] = 0;
        return;
    }
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < DONE_WORDS; i += blockDim.x) ws.done[i] = 0;
        for (int g = threadIdx.x; g < sh.nseg; g += blockDim.x) kept_out[g] = 0;
    }
    // (one block filled the table of 33.5 M entries - 16 K chunks - in 16.5 us; eight take 6)
    const int total = build_chunk_table(c.seg_len, c.seg_start, sh.nseg, [](int) { return true; }, SEL_CHUNK, c.cap,
                                        ws.sel_chunk_prefix, ws.sel_desc, ws.max_sel_chunks, ws.sel_entry_prefix, ws.err,
                                        (int)blockIdx.x, PLAN_TABLE_BLOCKS);
    if (blockIdx.x != 0) return;
    if ((int)threadIdx.x < hist_blocks) {                         // chunk range of every histogram block
        const int cpb = (total + hist_blocks - 1) / hist_blocks;
        const int c0 = min(total, (int)threadIdx.x * cpb), c1 = min(total, c0 + cpb);
        int4 r = make_int4(c0, c1, 0, -1);
        if (c0 < c1) {
            r.z = seq_of_chunk(ws.sel_chunk_prefix, sh, c0);
            r.w = seq_of_chunk(ws.sel_chunk_prefix, sh, c1 - 1);
        }
        ws.sel_blk[threadIdx.x] = r;
    }
    for (int seq = threadIdx.x; seq < sh.n_seq; seq += blockDim.x) {
        const int64_t n = ws.sel_entry_prefix[(seq + 1) * sh.segs_per_seq] - ws.sel_entry_prefix[seq * sh.segs_per_seq];
        int64_t b = budget[seq];
        if (b < 0) b = 0;
        SelState st;
        st.prefix = 0;
        st.thr_key = 0xFFFFFFFFu;
        st.count = n;
        st.want = b < n ? b : n;
        st.rank = st.want;
        st.tie_quota = 0;
        st.keep_none = st.want == 0;
        st.need_rank = 0;
        ws.sel[seq] = st;                                         // final slot (what the count and mask kernels read)
        ws.sel[sh.n_seq + seq] = st;                              // state before the first digit
        if (thr_out) thr_out[seq] = 0xFFFFFFFFu;                  // stands for a sequence that keeps nothing
    }
}

// One digit of the threshold key: walks the merged histogram of pass P (the sum of its replicas) of sequence
// `seq` from the top bin down to the bin that holds the entry of rank st.rank (1-based, descending key order)
// and returns the state with that digit appended.  Called by all threads of a 1024-thread block.
template <int P>
__device__ __forceinline__ SelState next_digit(const uint32_t* __restrict__ hist_pass, int n_seq, int seq, SelState st,
                                               int64_t* lds64, SelState* s_state) {
    constexpr int NB = P == 2 ? 1024 : 2048;
    constexpr int PER = NB / 1024;                                // bins per thread (1 or 2), thread 0 owns the highest bins
    const int tid = threadIdx.x;
    uint32_t cnt[PER];
    int64_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int bin = NB - 1 - (tid * PER + i);
        uint32_t v = 0;
#pragma unroll
        for (int r = 0; r < HIST_REPLICAS; ++r) v += hist_pass[((size_t)r * n_seq + seq) * RADIX_BINS + bin];
        cnt[i] = v;
        mine += v;
    }
    int64_t tot;
    int64_t above = block_excl_scan<int64_t>(mine, lds64, &tot);
    if (above < st.rank && st.rank <= above + mine) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (st.rank <= above + cnt[i]) {
                const uint32_t bin = NB - 1 - (tid * PER + i);
                const int bits = P == 2 ? RADIX_BITS2 : (P == 1 ? RADIX_BITS1 : RADIX_BITS0);
                SelState o = st;
                o.prefix = (st.prefix << bits) | bin;
                o.rank = st.rank - above;
                *s_state = o;
                break;
            }
            above += cnt[i];
        }
    }
    __syncthreads();
    const SelState o = *s_state;
    __syncthreads();                                              // s_state may be written again by the next call
    return o;
}

// Histogram of the next digit over the entries whose higher digits equal the prefix found so
// far.  A block takes a contiguous range of chunks and walks it as a flat range of entry slots
// (every load independent of the previous one); its LDS histogram is flushed per sequence.
// SHIFT = log2 of the chunk size of the table (2048-entry chunks of a ragged cache, 128-slot pages of a
// paged one); PAGED: a slot counts only if its position is not negative.
// SCORE (first pass of a ragged cache only): the score is computed here from log beta and the position (Eq.
// global_score in log domain, exactly as k_score does) and written to score_w; `score` is not read.
// VEC (ragged caches whose arrays are all 16-byte aligned): a chunk is walked in ALIGNED groups of four entries -
// 16-byte loads, four times the bytes in flight of the entry-by-entry walk.  A group may begin before the chunk or
// end behind it (segments start anywhere): what lies outside [first, first + n) is loaded and ignored; the one group
// that would reach past the end of the arrays is read entry by entry.
struct Quad {
    int64_t a;        // first entry of the aligned group
    int lo, hi;       // its entries a + lo .. a + hi - 1 belong to the chunk (lo == hi: none)
    bool whole;       // all four can be loaded (the group ends inside the arrays)
};
__device__ __forceinline__ Quad quad_of(const ChunkDesc& d, int q, int64_t cap) {
    Quad r;
    r.a = (d.first & ~(int64_t)3) + 4 * (int64_t)q;
    const int64_t end = d.first + d.n;
    r.lo = (int)(d.first > r.a ? d.first - r.a : 0);
    const int64_t h = end - r.a;
    r.hi = h < r.lo ? r.lo : (h < 4 ? (int)h : 4);
    r.whole = r.a + 4 <= cap;
    return r;
}
template <typename T>
__device__ __forceinline__ void load_quad(const T* __restrict__ base, const Quad& q, T (&v)[4]) {
    struct alignas(16) T4 { T x, y, z, w; };
    // (a group with nothing of the chunk, or reaching past the arrays, loads the arrays' first four entries instead)
    const T4 x = *reinterpret_cast<const T4*>(base + ((q.whole && q.lo < q.hi) ? q.a : 0));
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
}
template <typename T>
__device__ __forceinline__ void reload_quad_tail(const T* __restrict__ base, const Quad& q, T (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i >= q.lo && i < q.hi) v[i] = base[q.a + i];
}

template <int PASS, int SHIFT, bool PAGED, bool SCORE = false>
__global__ __launch_bounds__(HIST_THREADS, 8) void k_sel_hist(const float* __restrict__ score, Shape sh,
                                                           Workspace ws, SelTables tb,
                                                           CacheView c, const int32_t* __restrict__ now,
                                                           float* __restrict__ score_w, bool vec) {
    static_assert(!SCORE || (PASS == 0 && !PAGED), "the score is fused into the first pass over a ragged cache only");
    constexpr int NB = PASS == 2 ? 1024 : 2048;
    constexpr int HIST_TILE = 64;
    __shared__ uint32_t h[NB];
    __shared__ ChunkDesc s_desc[HIST_TILE];
    __shared__ int64_t lds64[17];
    __shared__ SelState s_state;
    const int tid = threadIdx.x;
    const int4 rng = ws.sel_blk[blockIdx.x];
    const int c0 = rng.x, c1 = rng.y;
    uint32_t* hist_pass = ws.hist + (size_t)PASS * HIST_REPLICAS * sh.n_seq * RADIX_BINS;
    uint32_t* hist = hist_pass + (size_t)(blockIdx.x % HIST_REPLICAS) * sh.n_seq * RADIX_BINS;

    if (c0 < c1) {
        for (int i = tid; i < NB; i += HIST_THREADS) h[i] = 0;
        const int seq_lo = rng.z, seq_hi = rng.w;
        for (int seq = seq_lo; seq <= seq_hi; ++seq) {
            const int a = max(c0, tb.prefix[seq * sh.segs_per_seq]);
            const int b = min(c1, tb.prefix[(seq + 1) * sh.segs_per_seq]);
            if (a >= b) continue;
            if (!SCORE && ws.sel[seq].keep_none) continue;        // (with SCORE the pass still has the scores to write)
            const int t1 = SCORE ? now[seq] + 1 : 0;
            // The digits fixed so far: every block derives them itself from the previous pass's merged histogram
            // (a few microseconds of L2 reads, the same for all blocks) instead of waiting for that pass's last
            // block to do it, which put "last block done" detection and the walk on the critical path of every pass.
            // (slots of ws.sel: [0] final, [1] after the plan, [2] after the first digit, [3] after the second)
            SelState st = ws.sel[(size_t)(PASS > 1 ? PASS : 1) * sh.n_seq + seq];
            if (PASS > 0) {
                st = next_digit<(PASS > 0 ? PASS - 1 : 0)>(ws.hist + (size_t)(PASS - 1) * HIST_REPLICAS * sh.n_seq * RADIX_BINS,
                                                          sh.n_seq, seq, st, lds64, &s_state);
            }
            if (PASS > 0 && tid == 0) ws.sel[(size_t)(PASS + 1) * sh.n_seq + seq] = st;   // the same value from every block
            const uint32_t prefix = st.prefix;
            // the descriptors of a tile of chunks go through LDS so that the score loads of a
            // thread do not depend on anything loaded inside the loop and are all in flight at once
            for (int t0 = a; t0 < b; t0 += HIST_TILE) {
                const int nt = min(HIST_TILE, b - t0);
                __syncthreads();
                if (tid < nt) s_desc[tid] = tb.desc[t0 + tid];
                __syncthreads();
                if (PAGED) {
                    // pages are whole, 16-byte aligned chunks: four slots per load
#pragma unroll 4
                    for (int s4 = tid; s4 < (nt << (SHIFT - 2)); s4 += HIST_THREADS) {
                        const ChunkDesc d = s_desc[s4 >> (SHIFT - 2)];
                        const int64_t e = d.first + ((s4 & ((1 << (SHIFT - 2)) - 1)) << 2);
                        const float4 sc = *reinterpret_cast<const float4*>(score + e);
                        const float v[4] = {sc.x, sc.y, sc.z, sc.w};
                        int bin[4];
                        bool hit[4];
                        bool any = false;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            hit[i] = digit_of<PASS>(key_of_score(v[i]), prefix, &bin[i]);
                            any |= hit[i];
                        }
                        if (any) {                                // the positions are looked at only where a prefix matches
                            const int4 ps = *reinterpret_cast<const int4*>(tb.pos + e);
                            const int p[4] = {ps.x, ps.y, ps.z, ps.w};
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (hit[i] && p[i] >= 0) atomicAdd(&h[bin[i]], 1u);
                        }
                    }
                } else if (vec) {
                    constexpr int QPC = (1 << (SHIFT - 2)) + 1;   // aligned groups of four that can overlap a chunk
                    constexpr int U = SCORE ? 2 : 4;              // groups a thread has in flight
                    for (int q0 = tid; q0 < nt * QPC; q0 += HIST_THREADS * U) {
                        Quad qd[U];
                        float sv[U][4];
                        int pv[U][4];
                        float lbv[U][4], ltv[U][4];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int qi = q0 + u * HIST_THREADS;
                            const int cidx = qi < nt * QPC ? qi / QPC : 0;
                            ChunkDesc d = s_desc[cidx];
                            if (qi >= nt * QPC) d.n = 0;
                            qd[u] = quad_of(d, qi - cidx * QPC, c.cap);
                            if (SCORE) {
                                load_quad(c.pos, qd[u], pv[u]);
                                load_quad(c.log_beta, qd[u], lbv[u]);
                                if (c.log_tail) load_quad(c.log_tail, qd[u], ltv[u]);
                            } else {
                                load_quad(score, qd[u], sv[u]);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const Quad& q = qd[u];
                            if (q.lo >= q.hi) continue;
                            if (!q.whole) {                       // (once per array at most)
                                if (SCORE) {
                                    reload_quad_tail(c.pos, q, pv[u]);
                                    reload_quad_tail(c.log_beta, q, lbv[u]);
                                    if (c.log_tail) reload_quad_tail(c.log_tail, q, ltv[u]);
                                } else {
                                    reload_quad_tail(score, q, sv[u]);
                                }
                            }
                            if (SCORE) {
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const float dt = (float)(t1 - pv[u][i]);
                                    sv[u][i] = c.log_tail ? __fmaf_rn(dt, lbv[u][i], ltv[u][i]) : __fmul_rn(dt, lbv[u][i]);
                                }
                                if (q.whole && q.lo == 0 && q.hi == 4) {
                                    *reinterpret_cast<float4*>(score_w + q.a) = make_float4(sv[u][0], sv[u][1], sv[u][2], sv[u][3]);
                                } else {
#pragma unroll
                                    for (int i = 0; i < 4; ++i)
                                        if (i >= q.lo && i < q.hi) score_w[q.a + i] = sv[u][i];
                                }
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                int bin;
                                if (i >= q.lo && i < q.hi && digit_of<PASS>(key_of_score(sv[u][i]), prefix, &bin)) atomicAdd(&h[bin], 1u);
                            }
                        }
                    }
                } else {
#pragma unroll 8
                    for (int slot = tid; slot < (nt << SHIFT); slot += HIST_THREADS) {
                        const ChunkDesc d = s_desc[slot >> SHIFT];
                        const int j = slot & ((1 << SHIFT) - 1);
                        if (j < d.n) {
                            int bin;
                            float sv;
                            if (SCORE) {
                                const int64_t e = d.first + j;
                                const float dt = (float)(t1 - c.pos[e]);
                                sv = c.log_tail ? __fmaf_rn(dt, c.log_beta[e], c.log_tail[e]) : __fmul_rn(dt, c.log_beta[e]);
                                score_w[e] = sv;
                            } else {
                                sv = score[d.first + j];
                            }
                            if (digit_of<PASS>(key_of_score(sv), prefix, &bin)) atomicAdd(&h[bin], 1u);
                        }
                    }
                }
            }
            __syncthreads();
            for (int i = tid; i < NB; i += HIST_THREADS) {
                const uint32_t v = h[i];
                if (v) {
                    atomicAdd(&hist[(size_t)seq * RADIX_BINS + i], v);
                    h[i] = 0;
                }
            }
            // (the next kernel finds this pass's digit itself)
        }
    }
}

// Behind the last pass, one block per sequence: the final digit, hence the threshold key, how many of the entries equal
// to it survive and whether those have to be ranked in order; and the bound that the decode-step selection starts from
// at its next call (k_fastsel.hip): a key with about 2 (k + 1) retained entries between it and the threshold
// (seed_distance).  The entry of that rank is walked down the three histograms as far as it shares the threshold's
// digits (below that the histograms count other buckets); where it leaves them, the upper edge of its bucket is taken.
// All three histograms are asked for at once, and both ranks are looked up in the same three scans.  (This used to be
// done by the last block of the last pass to arrive: two fences, then four walks one after the other, 35 to 40 us
// behind the pass whatever its size; the kernel takes 6 to 7.)
__global__ __launch_bounds__(HIST_THREADS) void k_sel_final(Shape sh, Workspace ws, uint32_t* __restrict__ thr_out) {
    __shared__ int64_t lds64[17];
    __shared__ int64_t s_rank[3][2];                              // per digit: rank inside the bin, of the threshold / of the bound
    __shared__ uint32_t s_bin[3][2], s_cnt;
    const int tid = threadIdx.x, seq = blockIdx.x;
    const SelState st = ws.sel[(size_t)sh.n_seq + seq];           // before the first digit
    if (st.keep_none) return;
    // thread 0 owns the highest bins; bins of the first two passes go two to a thread
    uint32_t c0[2] = {0, 0}, c1[2] = {0, 0}, c2 = 0;
    const size_t pass = (size_t)HIST_REPLICAS * sh.n_seq * RADIX_BINS;
#pragma unroll
    for (int r = 0; r < HIST_REPLICAS; ++r) {
        const uint32_t* h = ws.hist + ((size_t)r * sh.n_seq + seq) * RADIX_BINS;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            c0[i] += h[2047 - (2 * tid + i)];
            c1[i] += h[pass + 2047 - (2 * tid + i)];
        }
        c2 += h[2 * pass + 1023 - tid];
    }
    const bool seed = ws.fl_cap > 0 && st.count > st.want;
    int64_t rank_b = st.want - seed_distance(st.count - st.want, sh.segs_per_seq, ws.fl_cap);
    rank_b = rank_b >= 1 ? rank_b : 1;
    // the bin with the entries of rank ra / rb (1-based, from the top) of one digit: into s_bin[d], s_rank[d]
    auto find = [&](int d, const uint32_t* cnt, int per, int nb, int64_t ra, int64_t rb) {
        int64_t mine = 0, tot;
        for (int i = 0; i < per; ++i) mine += cnt[i];
        int64_t above = block_excl_scan<int64_t>(mine, lds64, &tot);
        for (int i = 0; i < per; ++i) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t r = k ? rb : ra;
                if (above < r && r <= above + cnt[i]) {
                    s_bin[d][k] = nb - 1 - (tid * per + i);
                    s_rank[d][k] = r - above;
                    if (k == 0 && d == 2) s_cnt = cnt[i];
                }
            }
            above += cnt[i];
        }
        __syncthreads();
    };
    find(0, c0, 2, 2048, st.rank, rank_b);
    find(1, c1, 2, 2048, s_rank[0][0], s_rank[0][1]);             // (the bound's only if it shares the first digit; else not used)
    find(2, &c2, 1, 1024, s_rank[1][0], s_rank[1][1]);
    if (tid != 0) return;
    SelState fin = st;
    fin.prefix = (((s_bin[0][0] << RADIX_BITS1) | s_bin[1][0]) << RADIX_BITS2) | s_bin[2][0];
    fin.rank = s_rank[2][0];
    fin.thr_key = fin.prefix;
    fin.tie_quota = fin.rank;
    fin.need_rank = fin.rank < (int64_t)s_cnt;                    // fewer survive than tie at the threshold
    if (fin.need_rank) atomicOr((int*)&ws.done[127], 1);
    if (thr_out) thr_out[seq] = fin.thr_key;
    ws.sel[seq] = fin;
    if (seed) {
        uint64_t key;
        if (s_bin[0][1] != s_bin[0][0]) key = ((uint64_t)s_bin[0][1] + 1) << 21;
        else if (s_bin[1][1] != s_bin[1][0]) key = ((((uint64_t)s_bin[0][1] << RADIX_BITS1) | s_bin[1][1]) + 1) << 10;
        else key = (uint64_t)((((s_bin[0][1] << RADIX_BITS1) | s_bin[1][1]) << RADIX_BITS2) | s_bin[2][1]) + 1;
        ws.fast_hi[seq] = key > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)key;
    }
}

// Only runs when, for some sequence, the entries equal to the threshold do not all fit.  Per
// chunk of such a sequence: entries above the threshold (credited to the segment) and entries
// equal to it; the last block then turns the per-chunk tie counts into exclusive prefixes per
// sequence and credits the ties that fit into the quota to their segments.
__global__ __launch_bounds__(CNT_THREADS) void k_sel_count(const float* __restrict__ score, Shape sh,
                                                           Workspace ws, SelTables tb,
                                                           int32_t* __restrict__ kept_out) {
    __shared__ int64_t lds64[17];
    __shared__ int32_t lds32[17];
    __shared__ int s_list[CNT_THREADS];
    __shared__ int s_n, is_last;
    if (ws.done[127] == 0) return;                                // uniform over the grid
    const int tid = threadIdx.x;
    for_each_ranked_seq(ws.sel, sh.n_seq, s_list, &s_n, [&](int seq) {
        const uint32_t thr_key = ws.sel[seq].thr_key;
        const int cb = tb.prefix[seq * sh.segs_per_seq], ce = tb.prefix[(seq + 1) * sh.segs_per_seq];
        for (int ch = cb + blockIdx.x; ch < ce; ch += gridDim.x) {
            const ChunkDesc d = tb.desc[ch];
            int gt = 0, eq = 0;
            for (int j = tid; j < d.n; j += CNT_THREADS) {
                const uint32_t key = key_of_score(score[d.first + j]);
                gt += key > thr_key;
                eq += key == thr_key;
            }
            gt = block_sum<int32_t>(gt, lds32);
            eq = block_sum<int32_t>(eq, lds32);
            if (tid == 0) {
                if (gt) atomicAdd(&kept_out[d.seg], gt);
                ws.chunk_eq[ch] = eq;
            }
        }
    });
    __syncthreads();
    if (tid == 0) is_last = arrive_last(ws.done + 32 * 3);
    __syncthreads();
    if (!is_last) return;
    __threadfence();

    for_each_ranked_seq(ws.sel, sh.n_seq, s_list, &s_n, [&](int seq) {
        const int cb = tb.prefix[seq * sh.segs_per_seq];
        const int ce = tb.prefix[(seq + 1) * sh.segs_per_seq];
        const int64_t quota = ws.sel[seq].tie_quota;
        int64_t running = 0;
        for (int base = cb; base < ce; base += CNT_THREADS) {
            const int cc = base + tid;
            int64_t v = cc < ce ? (int64_t)__hip_atomic_load(&ws.chunk_eq[cc], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            int64_t tot;
            int64_t ex = block_excl_scan<int64_t>(v, lds64, &tot);
            if (cc < ce) {
                const int64_t tbase = running + ex;
                ws.chunk_tie_base[cc] = tbase;
                if (v > 0 && tbase < quota) {
                    const int64_t take = min(v, quota - tbase);
                    atomicAdd(&kept_out[tb.desc[cc].seg], (int32_t)take);
                }
            }
            running += tot;
        }
    });
}

// The mask of one chunk entry by entry, for the cases the fast walk below does not take; returns how many survivors of
// this thread still have to be credited to the segment (none where the count kernel has done it).
__device__ __forceinline__ int mask_chunk(const float* __restrict__ score, const Workspace& ws, uint8_t* __restrict__ keep,
                                          const ChunkDesc& d, int ch, const SelState& st, int32_t* lds32) {
    const int tid = threadIdx.x;
    const float* s = score + d.first;
    uint8_t* kp = keep + d.first;
    if (st.keep_none) {
        for (int j = tid; j < d.n; j += SEL_THREADS) kp[j] = 0;
        return 0;
    }
    if (!st.need_rank) {                                          // every tie survives
        int n = 0;
#pragma unroll 8
        for (int j = tid; j < d.n; j += SEL_THREADS) {
            const bool k = key_of_score(s[j]) >= st.thr_key;
            kp[j] = k;
            n += k;
        }
        return n;
    }
    const int64_t tbase = ws.chunk_tie_base[ch];
    const int eq_total = ws.chunk_eq[ch];
    if (eq_total == 0 || tbase + eq_total <= st.tie_quota) {     // every tie of this chunk survives
        for (int j = tid; j < d.n; j += SEL_THREADS) kp[j] = key_of_score(s[j]) >= st.thr_key;
        return 0;
    }
    if (tbase >= st.tie_quota) {                                  // no tie of this chunk survives
        for (int j = tid; j < d.n; j += SEL_THREADS) kp[j] = key_of_score(s[j]) > st.thr_key;
        return 0;
    }
    // the quota runs out inside this chunk: rank the ties in order
    int64_t running = tbase;
    for (int base = 0; base < d.n; base += SEL_THREADS) {         // uniform trip count
        const int j = base + tid;
        uint32_t key = 0;
        int is_eq = 0;
        if (j < d.n) {
            key = key_of_score(s[j]);
            is_eq = key == st.thr_key;
        }
        int32_t tot;
        int32_t ex = block_excl_scan<int32_t>(is_eq, lds32, &tot);
        if (j < d.n) kp[j] = key > st.thr_key || (is_eq && running + ex < st.tie_quota);
        running += tot;
    }
    return 0;
}

// keep[e] = key > thr, or key == thr and the entry is among the first `quota` ties of its
// sequence in (segment, position) order.  When every tie fits (the usual case) the kernel also
// counts the survivors of its chunk into kept_out; otherwise the count kernel has done that.
// A segment is stored in position order, so the ties are ranked by storage order (exclusive tie
// counts per chunk).
// A block takes a run of consecutive chunks.  VEC (many chunks; score 16-byte, keep 4-byte aligned): a chunk is walked in
// aligned groups of four entries - a 16-byte load and one 4-byte store each, entry by entry where the group leaves the
// chunk - and the next chunk's descriptor and scores are asked for before the current ones are used; survivors are
// counted in registers and added to their segment once per run.  Otherwise a block per chunk, entry by entry: a chain of
// five latencies per 2048 entries, which many chunks pay eight times over (33.5 M entries, 168 MB: 57 us, now 30).
template <bool VEC>
__global__ __launch_bounds__(SEL_THREADS) void k_sel_mask(const float* __restrict__ score, Shape sh,
                                                          Workspace ws, SelTables tb, uint8_t* __restrict__ keep,
                                                          int32_t* __restrict__ kept_out, int64_t cap) {
    __shared__ int32_t lds32[17];
    const int tid = threadIdx.x;
    const int total = tb.prefix[sh.nseg];
    const int per = (total + (int)gridDim.x - 1) / (int)gridDim.x;
    const int ch0 = (int)blockIdx.x * per, ch1 = min(total, ch0 + per);
    if (ch0 >= ch1) return;
    constexpr int QT = SEL_CHUNK / 4 / SEL_THREADS;               // groups per thread; an unaligned chunk has one more
    ChunkDesc d = tb.desc[ch0], dn = d;
    float v[QT][4], vn[QT][4];
    auto load = [&](const ChunkDesc& cd, float (&x)[QT][4]) {
#pragma unroll
        for (int u = 0; u < QT; ++u) load_quad(score, quad_of(cd, tid + u * SEL_THREADS, cap), x[u]);
    };
    if (VEC) load(d, v);
    int seq = -1, n = 0;
    SelState st;
    auto credit = [&](int seg) {                                  // the run of chunks of segment `seg` has ended
        const int sum = block_sum<int32_t>(n, lds32);
        if (tid == 0 && sum) atomicAdd(&kept_out[seg], sum);
        n = 0;
    };
    for (int ch = ch0; ch < ch1; ++ch) {
        if (ch + 1 < ch1) {
            dn = tb.desc[ch + 1];
            if (VEC) load(dn, vn);
        }
        if (d.seg / sh.segs_per_seq != seq) {                     // (uniform)
            seq = d.seg / sh.segs_per_seq;
            st = ws.sel[seq];
        }
        if (VEC && !st.keep_none && !st.need_rank) {              // every tie survives
            auto put = [&](const Quad& q, const float (&x)[4]) {
                uint32_t word = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool k = key_of_score(x[i]) >= st.thr_key;
                    word |= (uint32_t)k << (8 * i);
                    if (i >= q.lo && i < q.hi) n += k;
                }
                if (q.lo == 0 && q.hi == 4) {
                    *reinterpret_cast<uint32_t*>(keep + q.a) = word;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (i >= q.lo && i < q.hi) keep[q.a + i] = (uint8_t)(word >> (8 * i));
                }
            };
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                const Quad q = quad_of(d, tid + u * SEL_THREADS, cap);
                if (!q.whole) reload_quad_tail(score, q, v[u]);   // (once per array at most)
                put(q, v[u]);
            }
            if (tid == 0) {                                       // an unaligned full chunk: its last group
                const Quad q = quad_of(d, QT * SEL_THREADS, cap);
                if (q.lo < q.hi) {
                    float x[4];
                    load_quad(score, q, x);
                    if (!q.whole) reload_quad_tail(score, q, x);
                    put(q, x);
                }
            }
        } else {
            n += mask_chunk(score, ws, keep, d, ch, st, lds32);
        }
        if (ch + 1 == ch1 || dn.seg != d.seg) credit(d.seg);
        d = dn;
#pragma unroll
        for (int u = 0; u < QT; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[u][i] = vn[u][i];
    }
}

// The whole selection of a small cache in one launch: a sequence's entries are one flat range (segment after segment), shared
// equally by some of the SMALL_BLOCKS blocks and in them by the wavefronts, so a wavefront's keys lie in registers and
// the order of ties is the order of blocks, wavefronts and lanes.  The same three digits as above; between two of them
// the blocks of a sequence meet: each adds its histogram to the sequence's in memory, counts itself, and reads that when all
// have.
// What this replaces is seven dependent launches of 2 to 8 us each, whatever the size.
//
// Nothing says that the blocks of a launch are on the chip together (they are not on a stream that may use a few compute units
// only, or beside kernels that fill the chip), so a block waits for none that may not have started.  Where the blocks of a
// sequence meet first, one that has looked `wait` times without seeing all of them takes the sequence over: it does the
// whole selection itself, as a sequence of one block is done, and those that come to the meeting behind its mark leave.  Once all
// have met without such a mark all are running, and the later meetings end by themselves.
constexpr int SMALL_THREADS = 1024, SMALL_ITEMS = 8, SMALL_SEGS = 1024;
constexpr int SMALL_ONE = SMALL_THREADS * SMALL_ITEMS;            // entries up to which a sequence is one block's
// Most entries a block may have to walk when one sequence has them all: two tiles of its wavefronts.  us a call of kvtrim_score_select, in
// seven launches / in one: 1500 entries 30.2 / 8.0, 17.6 K 30.9 / 16.0, 88 K 32.5 / 17.2, 130 K 31.9 / 17.3, 200 K 32.4 / 24.9, but
// 400 K 36.8 / 47.7; 2 sequences of 85 K each 32.6 / 24.8; 4 of 25 K 32.7 / 17.6; 8 of 15 K 32.9 / 22.3, one with nine tenths 33.3 /
// 25.3 (a fixed two blocks for each: 17 and 70); 1024 lists of 4 entries 37.6 / 23.1, of 16 37.8 / 24.7; all scores equal, 88 K 48.8 / 38.3.
// A block that takes a sequence over: 100 K 43, 200 K 240.
constexpr int64_t SMALL_MOST = 2 * SMALL_ONE;
constexpr uint32_t SMALL_TAKEN = 1u << 31;                        // in a sequence's arrivals: one block does it all

// ONE: a grid of a block for each sequence, which meet nobody: half the registers (two of 64 to a compute unit; the others take
// 106 to 115, and held to 64 they spill: 88 K entries 26.8 us for 17.4).
template <bool SCORE, bool ONE>
__global__ __launch_bounds__(SMALL_THREADS, ONE ? 8 : 4) void k_sel_small(const float* __restrict__ score_in, CacheView c, const int32_t* __restrict__ now,
                                                             float* __restrict__ score_out, const int64_t* __restrict__ budget, Shape sh,
                                                             uint32_t* __restrict__ meet, uint32_t* __restrict__ hist, uint32_t* __restrict__ fast_hi,
                                                             int fl_cap, uint32_t wait, int32_t* __restrict__ err, uint8_t* __restrict__ keep,
                                                             int32_t* __restrict__ kept_out, uint32_t* __restrict__ thr_out) {
    constexpr int NW = SMALL_THREADS / 64;
    __shared__ uint32_t h[RADIX_BINS];
    __shared__ uint32_t s_before[SMALL_SEGS], s_len[SMALL_SEGS], s_start[SMALL_SEGS];
    __shared__ int s_kept[SMALL_SEGS];
    __shared__ int32_t lds32[17];
    __shared__ int64_t s_rank[3][2];                              // per digit: rank inside the bin, of the threshold / of the bound
    __shared__ uint32_t s_bin[3][2], s_cnt;
    __shared__ int s_bad, s_met, s_total[SMALL_BLOCKS];
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int segs = sh.segs_per_seq;
    auto len_of = [&](int g, int64_t* start, bool* bad) {
        const int len = c.seg_len[g];
        const int64_t st = c.seg_start[g], nx = c.seg_start[min(g + 1, sh.nseg - 1)], nxt = g + 1 < sh.nseg ? nx : c.cap;
        *start = st;
        if (len >= 0 && st >= 0 && st + len <= c.cap && st + len <= nxt) return len;
        *bad = true;
        return 0;
    };
    bool bad = false;
    int len = 0;
    int64_t start = 0;
    int seq = ONE ? (int)blockIdx.x : 0, part = ONE ? 0 : (int)blockIdx.x, bpq = ONE ? 1 : (int)gridDim.x;
    if (tid < segs) len = len_of(seq * segs + tid, &start, &bad);   // (of the first sequence; usually the only one)
    if (tid == 0) s_bad = 0;
    if (tid < SMALL_BLOCKS) s_total[tid] = 0;
    for (int i = tid; i < RADIX_BINS; i += SMALL_THREADS) h[i] = 0;
    if (ONE && sh.n_seq > 1) {
        int64_t st;
        for (int g = tid; g < sh.nseg; g += SMALL_THREADS) len_of(g, &st, &bad);
    }
    if (!ONE && sh.n_seq > 1) {
        // the grid's blocks are dealt out by the sequences' lengths: one each, the others in proportion, none for fewer than SMALL_ONE entries
        __syncthreads();
        for (int g = tid; g < sh.nseg; g += SMALL_THREADS) {
            int64_t st;
            const int n = len_of(g, &st, &bad);
            if (n) atomicAdd(&s_total[g / segs], n);
        }
        __syncthreads();
        const int mine = lane < sh.n_seq ? s_total[min(lane, SMALL_BLOCKS - 1)] : 0;
        const float all = (float)max(wave_sum(mine), 1);
        const int more = min((int)((float)((int)gridDim.x - sh.n_seq) * ((float)mine / all)), (mine + SMALL_ONE - 1) / SMALL_ONE - 1);   // (sums to the rest at most)
        const int nb = lane < sh.n_seq ? 1 + max(more, 0) : 0, first = wave_incl_scan(nb) - nb;
        const uint64_t at = __ballot(lane < sh.n_seq && first <= (int)blockIdx.x && (int)blockIdx.x < first + nb);
        if (at == 0) return;                                      // a block to spare (the whole block, and nobody waits for it)
        seq = __ffsll((long long)at) - 1;
        part = (int)blockIdx.x - lane_value(first, seq);
        bpq = lane_value(nb, seq);
        len = 0;
        if (tid < segs) len = len_of(seq * segs + tid, &start, &bad);
    }
    const int g0 = seq * segs;
    const int64_t bud = budget[seq];
    const int t1 = SCORE ? now[seq] + 1 : 0;
    int32_t tot;
    const int32_t before = block_excl_scan<int32_t>(len, lds32, &tot);   // (its barriers stand between s_bad = 0 and = 1)
    if (bad) s_bad = 1;
    if (tid < segs) {
        s_before[tid] = (uint32_t)before;
        s_len[tid] = (uint32_t)len;
        s_start[tid] = (uint32_t)start;
        s_kept[tid] = 0;
    }
    auto clear_kept = [&]() {                                     // (the survivors are added by all blocks)
        if (part == 0 && tid < segs) __hip_atomic_store(&kept_out[g0 + tid], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    __syncthreads();
    if (s_bad) {                                                  // an unusable table anywhere (every block finds it): no selection at all
        clear_kept();
        if (tid == 0) {
            atomicOr(err, ERR_LAYOUT);
            if (part == 0 && thr_out) thr_out[seq] = 0xFFFFFFFFu;
        }
        return;
    }
    if (!ONE && sh.n_seq == 1) bpq = min(bpq, max(1, (tot + SMALL_ONE - 1) / SMALL_ONE));
    if (part >= bpq) return;
    const uint32_t total = (uint32_t)tot;
    const int64_t want = bud < 0 ? 0 : (bud < (int64_t)total ? bud : (int64_t)total);
    const int dealt = bpq;
    uint32_t* word = meet + (size_t)seq * 2 * SMALL_STRIDE;       // arrivals; SMALL_STRIDE behind: blocks that have left
#pragma unroll 1
    for (;;) {                                                    // (once more for a block that takes the sequence over)
    // the wavefront's entries: [w0, w1) of the sequence
    const uint32_t share = (total + (uint32_t)(bpq * NW) * 64 - 1) / ((uint32_t)(bpq * NW) * 64) * 64, wno = (uint32_t)(part * NW + wave);
    const uint32_t w0 = min(total, wno * share), w1 = min(total, w0 + share);
    int sl0 = -1;                                                 // the segment of entry w0 + lane
    for (int b = 0; b < segs; b += 64) sl0 += __popcll(__ballot(b + lane < segs && s_before[min(b + lane, segs - 1)] <= w0));
    sl0 = max(sl0, 0);

    // a tile of the wavefront's entries: which segment they belong to and where they lie
    struct Tile {
        int seg[SMALL_ITEMS];
        uint32_t at[SMALL_ITEMS];
        bool in[SMALL_ITEMS];
    };
    auto place = [&](uint32_t b, int& sl, Tile& t) {
#pragma unroll
        for (int u = 0; u < SMALL_ITEMS; ++u) {
            const uint32_t i = b + u * 64 + lane;
            t.in[u] = i < w1;
            if (t.in[u])
                while (i >= s_before[sl] + s_len[sl]) ++sl;
            t.seg[u] = sl;
            t.at[u] = t.in[u] ? s_start[sl] + (i - s_before[sl]) : 0u;
        }
    };
    // (behind the first tile the keys come from the scores again, which this block has written itself or which are the input)
    auto keys = [&](const Tile& t, uint32_t (&k)[SMALL_ITEMS]) {
        float v[SMALL_ITEMS];
#pragma unroll
        for (int u = 0; u < SMALL_ITEMS; ++u) v[u] = t.in[u] ? (SCORE ? (const float*)score_out : score_in)[t.at[u]] : 0.f;
#pragma unroll
        for (int u = 0; u < SMALL_ITEMS; ++u) k[u] = key_of_score(v[u]);
    };
    if (bpq == 1) clear_kept();
    Tile t0;
    uint32_t key[SMALL_ITEMS];
    int sl_rest = sl0;                                            // the segment where the second tile begins
    place(w0, sl_rest, t0);
    constexpr uint32_t STEP = 64 * SMALL_ITEMS;
    auto count = [&](int u, const Tile& t, uint32_t bin) {
        if (t.in[u]) atomicAdd(&h[bin], 1u);
    };
    // ---- first digit, with the scores
    if (SCORE) {
        int sl = sl_rest;
        Tile t = t0;
        for (uint32_t b = w0;; b += STEP) {
            int pv[SMALL_ITEMS];
            float lb[SMALL_ITEMS], lt[SMALL_ITEMS];
#pragma unroll
            for (int u = 0; u < SMALL_ITEMS; ++u) {
                pv[u] = t.in[u] ? c.pos[t.at[u]] : 0;
                lb[u] = t.in[u] ? c.log_beta[t.at[u]] : 0.f;
                lt[u] = t.in[u] && c.log_tail ? c.log_tail[t.at[u]] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < SMALL_ITEMS; ++u) {
                const float dt = (float)(t1 - pv[u]);
                const float sv = c.log_tail ? __fmaf_rn(dt, lb[u], lt[u]) : __fmul_rn(dt, lb[u]);
                if (t.in[u]) score_out[t.at[u]] = sv;
                const uint32_t k = key_of_score(sv);
                if (b == w0) key[u] = k;
                count(u, t, k >> 21);
            }
            if (b + STEP >= w1) break;
            place(b + STEP, sl, t);
        }
    } else {
        keys(t0, key);
#pragma unroll
        for (int u = 0; u < SMALL_ITEMS; ++u) count(u, t0, key[u] >> 21);
    }
    // the entries behind the first tile, a tile at a time
    auto rest = [&](auto&& use) {
        int sl = sl_rest;
        for (uint32_t b = w0 + STEP; b < w1; b += STEP) {
            Tile t;
            uint32_t k[SMALL_ITEMS];
            place(b, sl, t);
            keys(t, k);
            use(t, k);
        }
    };
    if (!SCORE) rest([&](const Tile& t, const uint32_t (&k)[SMALL_ITEMS]) {
#pragma unroll
        for (int u = 0; u < SMALL_ITEMS; ++u) count(u, t, k[u] >> 21);
    });

    uint32_t round = 0;
    constexpr int MET = 0, TAKE_OVER = 1, LEAVE = 2;
    auto all_here = [&]() {                                       // ... and everything they have stored past the caches is
        ++round;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            atomicAdd(word, 1u);
            const uint32_t all = round * (uint32_t)bpq;
            uint32_t v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), looked = 0;
            int met = MET;
            while (v < all) {
                if (round == 1 && looked++ >= wait) {
                    const uint32_t was = atomicCAS(word, v, v | SMALL_TAKEN);
                    if (was == v) {
                        met = TAKE_OVER;
                        break;
                    }
                    v = was;                                      // (another block has come, or taken over)
                    continue;
                }
                __builtin_amdgcn_s_sleep(1);
                v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (met == MET && v & SMALL_TAKEN) met = LEAVE;       // (the mark is above any count)
            s_met = met;
        }
        __syncthreads();
    };
    // the sequence's histogram of digit d; the bins with the entries of rank ra / rb (1-based, from the top)
    auto find = [&](auto pass, int64_t ra, int64_t rb) {
        constexpr int d = decltype(pass)::value, NB = d == 2 ? 1024 : 2048, PER = NB / SMALL_THREADS;
        uint32_t cnt[PER];
        uint32_t* g = hist + ((size_t)seq * 3 + d) * RADIX_BINS;
        __syncthreads();
        // thread 0 owns the highest bins
        if (!ONE && bpq > 1) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t v = h[i * SMALL_THREADS + tid];
                if (v) atomicAdd(&g[i * SMALL_THREADS + tid], v);
            }
            all_here();
            if (d == 0 && s_met != MET) return;
            if constexpr (PER == 2) {
                const uint64_t two = __hip_atomic_load(reinterpret_cast<const uint64_t*>(g + NB - 2 - 2 * tid), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                cnt[0] = (uint32_t)(two >> 32);
                cnt[1] = (uint32_t)two;
            } else {
                cnt[0] = __hip_atomic_load(&g[NB - 1 - tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
#pragma unroll
            for (int i = 0; i < PER; ++i) cnt[i] = h[NB - 1 - (tid * PER + i)];
        }
        int32_t sum = 0, all;
#pragma unroll
        for (int i = 0; i < PER; ++i) sum += (int32_t)cnt[i];
        int32_t above = block_excl_scan<int32_t>(sum, lds32, &all);
#pragma unroll
        for (int i = 0; i < PER; ++i) h[i * SMALL_THREADS + tid] = 0;   // (read by all: the scan's barriers)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t r = k ? rb : ra;
                if (above < r && r <= (int64_t)above + cnt[i]) {
                    s_bin[d][k] = NB - 1 - (tid * PER + i);
                    s_rank[d][k] = r - above;
                    if (k == 0 && d == 2) s_cnt = cnt[i];
                }
            }
            above += (int32_t)cnt[i];
        }
        __syncthreads();
    };
    const bool none = want == 0;
    const int64_t gone = (int64_t)total - want;
    int64_t rank_b = want - seed_distance(gone, segs, fl_cap);    // (the bound of the decode-step selection: as k_sel_final leaves it)
    rank_b = rank_b >= 1 ? rank_b : 1;
    uint32_t thr = 0xFFFFFFFFu;
    int64_t quota = 0;
    bool need_rank = false;
    uint32_t tie0 = 0;                                            // ties of the sequence before this wavefront's
    if (none) {
        if (bpq > 1) clear_kept();
    } else {
        find(std::integral_constant<int, 0>{}, want, rank_b);
        if (!ONE && bpq > 1 && s_met == LEAVE) break;
        if (!ONE && bpq > 1 && s_met == TAKE_OVER) {
            bpq = 1;
            part = 0;
            for (int i = tid; i < RADIX_BINS; i += SMALL_THREADS) h[i] = 0;
            __syncthreads();
            continue;
        }
        if (bpq > 1) clear_kept();                                // (the others add theirs two meetings later)
        const uint32_t p0 = s_bin[0][0];
        auto digit1 = [&](const Tile& t, const uint32_t (&k)[SMALL_ITEMS]) {
#pragma unroll
            for (int u = 0; u < SMALL_ITEMS; ++u)
                if (k[u] >> 21 == p0) count(u, t, k[u] >> 10 & 2047u);
        };
        digit1(t0, key);
        rest(digit1);
        find(std::integral_constant<int, 1>{}, s_rank[0][0], s_rank[0][1]);
        const uint32_t p1 = p0 << RADIX_BITS1 | s_bin[1][0];
        auto digit2 = [&](const Tile& t, const uint32_t (&k)[SMALL_ITEMS]) {
#pragma unroll
            for (int u = 0; u < SMALL_ITEMS; ++u)
                if (k[u] >> 10 == p1) count(u, t, k[u] & 1023u);
        };
        digit2(t0, key);
        rest(digit2);
        find(std::integral_constant<int, 2>{}, s_rank[1][0], s_rank[1][1]);
        thr = p1 << RADIX_BITS2 | s_bin[2][0];
        quota = s_rank[2][0];
        need_rank = quota < (int64_t)s_cnt;                       // fewer survive than tie at the threshold
        if (need_rank) {
            uint32_t n = 0;
            auto ties = [&](const Tile& t, const uint32_t (&k)[SMALL_ITEMS]) {
#pragma unroll
                for (int u = 0; u < SMALL_ITEMS; ++u) n += (uint32_t)__popcll(__ballot(t.in[u] && k[u] == thr));
            };
            ties(t0, key);
            rest(ties);
            int32_t mine;
            tie0 = (uint32_t)block_excl_scan<int32_t>(lane == 0 ? (int32_t)n : 0, lds32, &mine);
            tie0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)tie0);
            if (!ONE && bpq > 1) {
                uint32_t* tcount = hist + (size_t)sh.n_seq * 3 * RADIX_BINS + (size_t)seq * SMALL_BLOCKS;
                if (tid == 0) __hip_atomic_store(&tcount[part], (uint32_t)mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                all_here();
                for (int p = 0; p < part; ++p) tie0 += __hip_atomic_load(&tcount[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    // ---- the mask, and the survivors of every segment
    int64_t tie = (int64_t)tie0;
    auto mask = [&](const Tile& t, const uint32_t (&k)[SMALL_ITEMS]) {
#pragma unroll
        for (int u = 0; u < SMALL_ITEMS; ++u) {
            bool kf = !none && t.in[u] && (need_rank ? k[u] > thr : k[u] >= thr);
            if (need_rank) {
                const bool eq = t.in[u] && k[u] == thr;
                const uint64_t m = __ballot(eq);
                if (eq) kf = tie + __popcll(m & ((1ull << lane) - 1ull)) < quota;
                tie += __popcll(m);
            }
            if (t.in[u]) keep[t.at[u]] = kf;
            uint64_t left = __ballot(kf);
            while (left) {                                        // segment by segment (usually one)
                const int g = __builtin_amdgcn_readlane(t.seg[u], __ffsll((long long)left) - 1);
                const uint64_t same = __ballot(kf && t.seg[u] == g);
                if (lane == 0) atomicAdd(&s_kept[g], __popcll(same));
                left &= ~same;
            }
        }
    };
    mask(t0, key);
    rest(mask);
    __syncthreads();
    if (tid < segs && s_kept[tid]) atomicAdd(&kept_out[g0 + tid], s_kept[tid]);
    if (part == 0 && tid == 0) {
        if (thr_out) thr_out[seq] = thr;
        if (!none && fl_cap > 0 && gone > 0) {
            uint64_t b;
            if (s_bin[0][1] != s_bin[0][0]) b = ((uint64_t)s_bin[0][1] + 1) << 21;
            else if (s_bin[1][1] != s_bin[1][0]) b = ((((uint64_t)s_bin[0][1] << RADIX_BITS1) | s_bin[1][1]) + 1) << 10;
            else b = (uint64_t)((((s_bin[0][1] << RADIX_BITS1) | s_bin[1][1]) << RADIX_BITS2) | s_bin[2][1]) + 1;
            fast_hi[seq] = b > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)b;
        }
    }
    if (none) return;                                             // (they did not meet)
    break;
    }
    if (ONE || dealt == 1) return;
    if (tid == 0) s_bad = atomicAdd(word + SMALL_STRIDE, 1u) == (uint32_t)dealt - 1u;
    __syncthreads();
    if (!s_bad) return;                                           // the last to leave: nobody waits or reads any more
    for (int i = tid; i < 3 * RADIX_BINS; i += SMALL_THREADS) hist[(size_t)seq * 3 * RADIX_BINS + i] = 0;
    if (tid < 2) __hip_atomic_store(word + tid * SMALL_STRIDE, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Blocks of a selection in one launch, 0 where it takes the general way.
static int small_blocks(const kvtrim_ctx* ctx, int64_t cap) {
    const Shape& sh = ctx->shape;
    if (!ctx->sel_meet || sh.n_seq > SMALL_BLOCKS || sh.segs_per_seq > SMALL_SEGS) return 0;
    if (cap > (SMALL_BLOCKS + 1 - sh.n_seq) * SMALL_MOST) return 0;
    const int64_t blocks = sh.n_seq - 1 + (cap + SMALL_ONE - 1) / SMALL_ONE;
    return (int)(blocks < SMALL_BLOCKS ? blocks : SMALL_BLOCKS);
}

static void launch_select_final(kvtrim_ctx* ctx, uint32_t* thr, hipStream_t st) {
    ProfScope prof(ctx, K_SEL_FINAL, st);
    hipLaunchKernelGGL(k_sel_final, dim3(ctx->shape.n_seq), dim3(HIST_THREADS), 0, st, ctx->shape, ctx->ws, thr);
}

// The three histogram passes over a paged cache whose chunk table (one chunk per page) is in tb;
// the plan, the tie count and the mask of the paged layout live in k_paged.hip.
void launch_select_passes_paged(kvtrim_ctx* ctx, const float* score, const SelTables& tb, int hist_blocks,
                                int pass, uint32_t* thr, hipStream_t st) {
    const Shape& sh = ctx->shape;
    const Workspace& ws = ctx->ws;
    if (pass == 0) {
        ProfScope prof(ctx, K_SEL_HIST0, st);
        hipLaunchKernelGGL((k_sel_hist<0, 7, true>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, score, sh, ws, tb, CacheView(), nullptr, nullptr, false);
    } else if (pass == 1) {
        ProfScope prof(ctx, K_SEL_HIST1, st);
        hipLaunchKernelGGL((k_sel_hist<1, 7, true>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, score, sh, ws, tb, CacheView(), nullptr, nullptr, false);
    } else {
        ProfScope prof(ctx, K_SEL_HIST2, st);
        hipLaunchKernelGGL((k_sel_hist<2, 7, true>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, score, sh, ws, tb, CacheView(), nullptr, nullptr, false);
        launch_select_final(ctx, thr, st);
    }
}

// now != NULL: stage 1 is fused into the first pass, which writes the scores to score_w.
static kvtrim_status launch_select_impl(kvtrim_ctx* ctx, const CacheView& c, const float* score, const int32_t* now,
                                        float* score_w, const int64_t* budget, uint8_t* keep, int32_t* kept,
                                        uint32_t* thr, hipStream_t st) {
    const Shape& sh = ctx->shape;
    const Workspace& ws = ctx->ws;
    if (const int blocks = small_blocks(ctx, c.cap)) {
        ProfScope prof(ctx, K_SEL_SMALL, st);
        const dim3 grid(blocks), block(SMALL_THREADS);
#define KVTRIM_SMALL(scores, one) hipLaunchKernelGGL((k_sel_small<scores, one>), grid, block, 0, st, scores ? (const float*)nullptr : score, c, now, scores ? score_w : (float*)nullptr, \
                           budget, sh, ctx->sel_meet, ctx->sel_small, ws.fast_hi, ws.fl_cap, (uint32_t)ctx->sel_wait, ws.err, keep, kept, thr)
        if (blocks == sh.n_seq) {
            if (now) KVTRIM_SMALL(true, true);
            else KVTRIM_SMALL(false, true);
        } else {
            if (now) KVTRIM_SMALL(true, false);
            else KVTRIM_SMALL(false, false);
        }
#undef KVTRIM_SMALL
        KVTRIM_HIP(ctx, hipGetLastError());
        return KVTRIM_OK;
    }
    const int64_t max_chunks = c.cap / SEL_CHUNK + sh.nseg;      // bound on the chunk count
    const int n_chunk_blocks = (int)max_chunks;
    const int hist_blocks = (int)(max_chunks < HIST_BLOCKS ? (max_chunks < 1 ? 1 : max_chunks) : HIST_BLOCKS);
    SelTables tb;
    tb.desc = ws.sel_desc;
    tb.prefix = ws.sel_chunk_prefix;
    tb.pos = nullptr;
    // 16-byte loads need every array they touch aligned (and at least one group of four entries)
    const bool vec = c.cap >= 4 && ((((uintptr_t)score) | ((uintptr_t)score_w) | ((uintptr_t)c.pos) | ((uintptr_t)c.log_beta) |
                                     ((uintptr_t)c.log_tail)) & 15) == 0;
    { ProfScope prof(ctx, K_SEL_PLAN, st);
      hipLaunchKernelGGL(k_sel_plan, dim3(PLAN_TABLE_BLOCKS + PLAN_ZERO_BLOCKS), dim3(1024), 0, st, c, sh, budget, ws, kept, thr, hist_blocks); }
    { ProfScope prof(ctx, K_SEL_HIST0, st);
      if (now)
          hipLaunchKernelGGL((k_sel_hist<0, SEL_SHIFT, false, true>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, (const float*)nullptr, sh, ws, tb, c, now, score_w, vec);
      else
          hipLaunchKernelGGL((k_sel_hist<0, SEL_SHIFT, false>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, score, sh, ws, tb, c, nullptr, nullptr, vec); }
    { ProfScope prof(ctx, K_SEL_HIST1, st);
      hipLaunchKernelGGL((k_sel_hist<1, SEL_SHIFT, false>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, score, sh, ws, tb, c, nullptr, nullptr, vec); }
    { ProfScope prof(ctx, K_SEL_HIST2, st);
      hipLaunchKernelGGL((k_sel_hist<2, SEL_SHIFT, false>), dim3(hist_blocks), dim3(HIST_THREADS), 0, st, score, sh, ws, tb, c, nullptr, nullptr, vec); }
    launch_select_final(ctx, thr, st);
    { ProfScope prof(ctx, K_SEL_COUNT, st);
      hipLaunchKernelGGL(k_sel_count, dim3(n_chunk_blocks < 256 ? n_chunk_blocks : 256), dim3(CNT_THREADS), 0, st, score, sh, ws, tb, kept); }
    { ProfScope prof(ctx, K_SEL_MASK, st);
      // (cap >= 4: a group of four that is not whole loads the array's first four entries in its place)
      if (n_chunk_blocks >= MASK_LONG && c.cap >= 4 && (((uintptr_t)score) & 15) == 0 && (((uintptr_t)keep) & 3) == 0)
          hipLaunchKernelGGL(k_sel_mask<true>, dim3(MASK_BLOCKS), dim3(SEL_THREADS), 0, st, score, sh, ws, tb, keep, kept, c.cap);
      else
          hipLaunchKernelGGL(k_sel_mask<false>, dim3(n_chunk_blocks), dim3(SEL_THREADS), 0, st, score, sh, ws, tb, keep, kept, c.cap); }
    KVTRIM_HIP(ctx, hipGetLastError());
    return KVTRIM_OK;
}

kvtrim_status launch_select(kvtrim_ctx* ctx, const CacheView& c, const float* score, const int64_t* budget,
                            uint8_t* keep, int32_t* kept, uint32_t* thr, hipStream_t st) {
    return launch_select_impl(ctx, c, score, nullptr, nullptr, budget, keep, kept, thr, st);
}

kvtrim_status launch_score_select_general(kvtrim_ctx* ctx, const CacheView& c, const int32_t* now, const int64_t* budget,
                                          float* score, uint8_t* keep, int32_t* kept, uint32_t* thr, hipStream_t st) {
    return launch_select_impl(ctx, c, score, now, score, budget, keep, kept, thr, st);
}

}  // namespace kvtrim
