// Stages 1 + 2 for decode steps (Sec. 4.2: Eq. global_score and the global eviction rule) in two kernels, on pages in one; the
// first of them, in its STEP form, is also the first kernel of the one-call decode step.
//
// A decode step evicts a handful of entries per sequence - as many as it appended - so the selection is the
// search for the FEW LOWEST entries of the total order (key descending, segment ascending, position ascending),
// not a general top-B.  The pass that computes the scores lists every entry whose key lies below a bound `hi`
// carried over from the previous call; if the list holds at least k + 1 entries (k = count - min(budget, count)
// evictions), the k + 1 lowest entries of the whole sequence are the k + 1 lowest of the list, because every entry
// that is not listed has a key >= hi > every listed key.  The last block to finish a sequence ("last block done",
// one arrival counter per sequence) ranks the list - a few hundred entries - and publishes the last retained
// entry of the order as (key, segment, position); the mask kernel compares every entry with that triple (on pages the scanning
// blocks write the mask as if all survived and the last block clears what goes: one kernel).
//
// The bound adapts by itself: the next bound is the key of about the 3(k+1)-th lowest entry of the current
// list.  Scores only decay from step to step (beta <= 1, Eq. global_score) and new tokens enter with the highest
// scores, so the 2(k+1) retained entries below that key are below it at the next step as well: with a steady
// number of evictions per step the list can never come up short.  Nothing depends on the bound for correctness:
// a list that is short (first call, a budget or workload change), too long for its buffer, or with too many equal
// keys at the threshold makes the last block run a plain three-pass radix select over the sequence on its own
// (slow - one block reads every score three times - but rare) which also re-seeds the bound.
#include "kvtrim_paged_device.h"

namespace kvtrim {

constexpr int VMCNT_0 = 0x0F70;                                   // s_waitcnt: loads and stores done, the other counters as they are
constexpr int FAST_ITEMS = FL_CAP_MAX / FAST_THREADS;             // list entries a thread of the resolving block holds
constexpr int FAST_SUB = 16;                                      // sub-lists / group words per sequence
constexpr int FAST_STAGE = 1024;                                  // candidates a block of one segment stages in LDS
constexpr int FAST_PIECE_SHIFT = 6;                               // ... 64 of which go on one sub-list before the next is taken
constexpr int FAST_BATCH = 8;                                     // entries a thread loads before it uses any of them ...
constexpr int SLOW_BATCH = 4;                                     // ... in the single-block select (eight took the scoring kernel's registers from 72 to 86)
constexpr int FAST_BIN_DIRECT = 256;                              // a bin of at most this many entries is ranked directly
static_assert(FAST_ITEMS * FAST_THREADS == FL_CAP_MAX, "list capacity must be a multiple of the block size");

// A segment as the kernels see it (seg_view): empty, with *bad set, when its table entry is unusable - negative, beyond the buffers
// or overlapping its successor.  STEP: its entries [len_old, len) are this step's new tokens - up to the first
// padding row (negative position), none if the segment has no room for them (kvtrim_append's rule) - whose
// metadata is read from the new-token buffers by every block, never from the cache.
// PAGED: the segment's entries are the slots of its pages in block-table order (entry j = slot j % 128 of the table's
// page j / 128; start = the table's row); slots with a negative position are empty and `live` counts the others.
struct SegView {
    int64_t start;
    int len_old;
    int len;
    int live;
};

// What a block of k_fast_scan walks: a segment or a part of one / several segments / a whole sequence / one too, or a part of a long one
constexpr int DEAL_SEGMENT = 0, DEAL_MULTI = 1, DEAL_WHOLE = 2, DEAL_PARTS = 3;
constexpr int SCAN_RAGGED = 0, SCAN_STEP = 1, SCAN_PAGED = 2;     // what k_fast_scan walks over
constexpr int WHOLE_ENTRIES = FAST_THREADS * FAST_BATCH;          // a batch for every lane of a block

template <int KIND>
__device__ __forceinline__ SegView seg_view(const CacheView& c, int g, int nseg, const StepArgs& sa, bool* bad, bool* nocap) {
    constexpr bool STEP = KIND == SCAN_STEP;
    SegView v;
    if (KIND == SCAN_PAGED) {
        const int npg = sa.pg.seg_pages[g], live = sa.pg.seg_live[g];
        v.start = (int64_t)g * sa.pg.max_pps;
        if (npg < 0 || npg > sa.pg.max_pps || live < 0 || (int64_t)live > (int64_t)npg * KVTRIM_PAGE_SIZE) {
            *bad = true;
            v.len_old = v.len = v.live = 0;
            return v;
        }
        v.len_old = v.len = npg * KVTRIM_PAGE_SIZE;
        v.live = live;
        return v;
    }
    // (everything is asked for at once: a new token's position behind the table's check was a second round trip)
    const int len = c.seg_len[g];
    const int64_t st = c.seg_start[g], nx = c.seg_start[min(g + 1, nseg - 1)];
    const int32_t* pn = STEP ? sa.pos_new + (int64_t)g * sa.n_new : nullptr;
    const int first_new = STEP && sa.n_new > 0 ? pn[0] : -1;
    const int64_t nxt = g + 1 < nseg ? nx : c.cap;
    v.start = st;
    if (len < 0 || st < 0 || st + len > c.cap || st + len > nxt) {
        *bad = true;
        v.len_old = v.len = v.live = 0;
        return v;
    }
    v.len_old = v.len = len;
    if (STEP) {
        int cnt = first_new >= 0;
        if (cnt)
            while (cnt < sa.n_new && pn[cnt] >= 0) ++cnt;
        if (st + len + cnt > nxt || nxt > c.cap) {
            if (cnt) *nocap = true;
            cnt = 0;
        }
        v.len = len + cnt;
    }
    v.live = v.len;
    return v;
}

// a is evicted before b: lower key first; among equal keys the later (segment, position) first
__device__ __forceinline__ bool evicted_before(uint32_t ka, int sa, int pa, uint32_t kb, int sb, int pb) {
    if (ka != kb) return ka < kb;
    if (sa != sb) return sa > sb;
    return pa > pb;
}

struct ResolveShared {
    uint32_t h[2048];
    int64_t lds64[17];
    int32_t lds32[17];
    uint32_t red_u[16];
    int bin, bin_m, cnt, gather_n, found_seg, found_pos, digit;
    int64_t before, rank_in;
    uint32_t found_key, bin_count;
    uint32_t g_key[FAST_BIN_DIRECT];
    int32_t g_seg[FAST_BIN_DIRECT], g_pos[FAST_BIN_DIRECT];
};

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_min(uint32_t v) {         // with a lane's own value where there is no other
    return min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false));
}
// over the row of 16 lanes that ends at lane `last`, in all lanes of the wavefront
__device__ __forceinline__ uint32_t row_min(uint32_t v, int last) {
    v = dpp_min<0x111, 0xF>(v);
    v = dpp_min<0x112, 0xF>(v);
    v = dpp_min<0x114, 0xF>(v);
    v = dpp_min<0x118, 0xF>(v);
    return lane_value(v, last);
}
__device__ __forceinline__ uint32_t block_min_u32(uint32_t v, uint32_t* red) {
    v = dpp_min<0x111, 0xF>(v);                                   // inside the rows of 16 lanes, then across them (as wave_incl_scan)
    v = dpp_min<0x112, 0xF>(v);
    v = dpp_min<0x114, 0xF>(v);
    v = dpp_min<0x118, 0xF>(v);
    v = dpp_min<0x142, 0xA>(v);
    v = dpp_min<0x143, 0xC>(v);
    __syncthreads();
    if (lane_id() == 63) red[threadIdx.x >> 6] = v;
    __syncthreads();
    static_assert(FAST_THREADS / 64 == 16, "a lane of a row for every wavefront");
    return row_min(red[lane_id() & 15], 15);
}

// Walks an LDS histogram of NB bins from the top bin down to the one that holds the entry of rank `rank`
// (1-based, descending digit order).  Results in sm->digit, sm->rank_in (rank inside the bin), sm->bin_count.
template <int NB>
__device__ __forceinline__ void walk_from_top(ResolveShared* sm, int64_t rank) {
    constexpr int PER = NB / FAST_THREADS;                        // 2 or 1 bins per thread, thread 0 owns the highest
    const int tid = threadIdx.x;
    uint32_t cnt[PER];
    int64_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        cnt[i] = sm->h[NB - 1 - (tid * PER + i)];
        mine += cnt[i];
    }
    int64_t tot;
    int64_t above = block_excl_scan<int64_t>(mine, sm->lds64, &tot);
    if (above < rank && rank <= above + mine) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (rank <= above + cnt[i]) {
                sm->digit = NB - 1 - (tid * PER + i);
                sm->rank_in = rank - above;
                sm->bin_count = cnt[i];
                break;
            }
            above += cnt[i];
        }
    }
    __syncthreads();
}

// Where the key of an entry comes from: log beta and the position (stage 1, Eq. global_score in log domain - one fp32
// multiply, or one fused multiply-add with the cached horizon tail).  Both are inputs of the call, so any block may
// read any entry at any time.
template <int KIND>
struct KeySource {
    static constexpr bool STEP = KIND == SCAN_STEP, PAGED = KIND == SCAN_PAGED;
    const float* lb;
    const float* lt;
    const int32_t* pos;
    const float* lb_new;
    const float* lt_new;
    const int32_t* pos_new;
    int n_new;
    int t1;
    const int32_t* bt;                                            // PAGED: the block tables and the pool's page count
    int n_pages;
    // where entry j of the segment lies in the cache's arrays (not for a STEP's new tokens); *bad_page: the block
    // table names a page outside the pool (the page is clamped into it)
    __device__ __forceinline__ int64_t place(const SegView& v, int j, bool* bad_page) const {
        if (!PAGED) return v.start + j;
        int pg = bt[v.start + (j >> 7)];
        if (pg < 0 || pg >= n_pages) {
            *bad_page = true;
            pg = pg < 0 ? 0 : n_pages - 1;
        }
        return (int64_t)pg * KVTRIM_PAGE_SIZE + (j & (KVTRIM_PAGE_SIZE - 1));
    }
    // entry j of segment g: false for an empty slot (PAGED), else its position and score
    __device__ __forceinline__ bool entry_at(int g, const SegView& v, int j, int* p_out, float* s_out) const {
        float b, t = 0.f;
        int p;
        if (STEP && j >= v.len_old) {
            const int64_t i = (int64_t)g * n_new + (j - v.len_old);
            p = pos_new[i];
            b = lb_new[i];
            if (lt) t = lt_new[i];
        } else {
            bool bp = false;
            const int64_t e = place(v, j, &bp);
            p = pos[e];
            if (PAGED && p < 0) return false;
            b = lb[e];
            if (lt) t = lt[e];
        }
        *p_out = p;
        const float dt = (float)(t1 - p);
        *s_out = lt ? __fmaf_rn(dt, b, t) : __fmul_rn(dt, b);
        return true;
    }
    // the same for entries j0, j0 + stride, ... of a batch (those behind the segment's end are not live): all loads of a kind are
    // under way together
    __device__ __forceinline__ void batch_at(int g, const SegView& v, int j0, int stride, int (&slot)[SLOW_BATCH], bool (&live)[SLOW_BATCH],
                                             int (&p)[SLOW_BATCH], float (&s)[SLOW_BATCH]) const {
        float b[SLOW_BATCH], t[SLOW_BATCH];
        bool bp = false;
#pragma unroll
        for (int u = 0; u < SLOW_BATCH; ++u) {                    // (places are below 2^31 - and those of new tokens, at most STEP_MAX_NEW of 2^20 segments)
            const int j = j0 + u * stride;
            slot[u] = STEP && j >= v.len_old ? g * n_new + (j - v.len_old) : (j < v.len ? (int)place(v, j, &bp) : 0);
        }
#pragma unroll
        for (int u = 0; u < SLOW_BATCH; ++u) {
            const int j = j0 + u * stride;
            const bool in = j < v.len, isnew = STEP && j >= v.len_old;
            p[u] = in ? (isnew ? pos_new : pos)[slot[u]] : 0;
            b[u] = in ? (isnew ? lb_new : lb)[slot[u]] : 0.f;
            t[u] = in && lt ? (isnew ? lt_new : lt)[slot[u]] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < SLOW_BATCH; ++u) {
            const float dt = (float)(t1 - p[u]);
            s[u] = lt ? __fmaf_rn(dt, b[u], t[u]) : __fmul_rn(dt, b[u]);
            live[u] = j0 + u * stride < v.len && (!PAGED || p[u] >= 0);
        }
    }
};

// What a pass does with the entries besides counting them: nothing, or what the function does with a batch of a segment's entries
// (a wavefront's 64 of a place in the batch lie next to one another, on pages in one page).
struct NoVisit {
    static constexpr bool ANY = false;
    __device__ __forceinline__ void operator()(int, const int*, const bool*, const int*, const float*) const {}
};
template <typename F>
struct Visit {
    static constexpr bool ANY = true;
    const F& f;
    __device__ __forceinline__ void operator()(int g, const int* slot, const bool* live, const int* pos, const float* score) const { f(g, slot, live, pos, score); }
};

// One digit of a most-significant-digit radix select over all entries of the sequence, by this block alone: sixteen segments
// at a time, a wavefront to each if they are all short, else all wavefronts to one after the other.  (The chain of loads
// to a list's first entry is a microsecond, and a batch's loads must not wait for one another: kvtrim_paged_score_select with
// a list that is no use, 256 lists of 1000 entries 1690 us -> 548, 4 of 500 K 10.2 ms -> 5.1.)
constexpr int SLOW_SHORT = 8192;
template <int PASS, int KIND, typename V = NoVisit>
__device__ __forceinline__ void slow_pass(const KeySource<KIND>& ks, const CacheView& c, const Shape& sh,
                                          const StepArgs& sa, int seq, uint32_t prefix, ResolveShared* sm, const V& visit = V()) {
    constexpr int NB = PASS == 2 ? 1024 : 2048, NW = FAST_THREADS / 64;
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __syncthreads();
    for (int i = tid; i < NB; i += FAST_THREADS) sm->h[i] = 0;
    __syncthreads();
    auto walk = [&](int g, int first, int stride) {
        bool bad = false, nocap = false;
        const SegView v = seg_view<KIND>(c, g, sh.nseg, sa, &bad, &nocap);
        const int len = v.len;
        for (int j0 = first; j0 < len; j0 += stride * SLOW_BATCH) {
            float sv[SLOW_BATCH];
            bool lv[SLOW_BATCH];
            int pv[SLOW_BATCH], slot[SLOW_BATCH];
            ks.batch_at(g, v, j0, stride, slot, lv, pv, sv);
#pragma unroll
            for (int u = 0; u < SLOW_BATCH; ++u) {
                int bin;
                if (lv[u] && digit_of<PASS>(key_of_score(sv[u]), prefix, &bin)) atomicAdd(&sm->h[bin], 1u);
            }
            if (V::ANY) visit(g, slot, lv, pv, sv);
        }
    };
    const int g0 = seq * sh.segs_per_seq, g1 = g0 + sh.segs_per_seq;
    for (int g = g0; g < g1; g += NW) {
        bool bad = false, nocap = false;
        int len = 0;
        if (lane < NW && g + lane < g1) len = KIND == SCAN_PAGED ? sa.pg.seg_pages[g + lane] * KVTRIM_PAGE_SIZE : seg_view<KIND>(c, g + lane, sh.nseg, sa, &bad, &nocap).len;
        if (!__any(len > SLOW_SHORT)) {
            if (g + wave < g1) walk(g + wave, lane, 64);
        } else {
            for (int i = 0; i < NW && g + i < g1; ++i) walk(g + i, tid, FAST_THREADS);
        }
    }
    __syncthreads();
}

// Key of the entry of rank `rank` (1-based, descending key order) of the sequence; *rank_in = its rank among the
// entries with that key, *ties = how many entries have that key.  The first pass shows every entry to `visit`, which may
// empty slots of entries that come behind the one looked for.
template <int KIND, typename V = NoVisit>
__device__ __forceinline__ uint32_t slow_radix(const KeySource<KIND>& ks, const CacheView& c, const Shape& sh,
                                               const StepArgs& sa, int seq, int64_t rank, ResolveShared* sm,
                                               int64_t* rank_in, uint32_t* ties, const V& visit = V()) {
    slow_pass<0>(ks, c, sh, sa, seq, 0, sm, visit);
    walk_from_top<2048>(sm, rank);
    uint32_t prefix = (uint32_t)sm->digit;
    rank = sm->rank_in;
    slow_pass<1>(ks, c, sh, sa, seq, prefix, sm);
    walk_from_top<2048>(sm, rank);
    prefix = (prefix << RADIX_BITS1) | (uint32_t)sm->digit;
    rank = sm->rank_in;
    slow_pass<2>(ks, c, sh, sa, seq, prefix, sm);
    walk_from_top<1024>(sm, rank);
    prefix = (prefix << RADIX_BITS2) | (uint32_t)sm->digit;
    *rank_in = sm->rank_in;
    *ties = sm->bin_count;
    __syncthreads();
    return prefix;
}

// One digit of the radix select over the positions of segment g's entries with key == key_thr (taken as
// 0x7fffffff - position, so that the smallest position is the largest): narrows *prefix and *rank.
template <int PASS, int KIND>
__device__ __forceinline__ void tie_pos_pass(const KeySource<KIND>& ks, int g, const SegView& v, uint32_t key_thr,
                                             uint32_t* prefix, int64_t* rank, ResolveShared* sm) {
    constexpr int NB = PASS == 2 ? 1024 : 2048;
    const int tid = threadIdx.x;
    __syncthreads();
    for (int i = tid; i < NB; i += FAST_THREADS) sm->h[i] = 0;
    __syncthreads();
    for (int j = tid; j < v.len; j += FAST_THREADS) {
        int pj, bin;
        float sc;
        if (ks.entry_at(g, v, j, &pj, &sc) && key_of_score(sc) == key_thr &&
            digit_of<PASS>(0x7fffffffu - (uint32_t)pj, *prefix, &bin))
            atomicAdd(&sm->h[bin], 1u);
    }
    __syncthreads();
    walk_from_top<NB>(sm, *rank);
    *prefix = PASS == 0 ? (uint32_t)sm->digit : (*prefix << (PASS == 1 ? RADIX_BITS1 : RADIX_BITS2)) | (uint32_t)sm->digit;
    *rank = sm->rank_in;
}

// The `quota`-th entry (1-based) with key == key_thr in (segment ascending, position ascending) order:
// result in sm->found_seg / sm->found_pos.  The caller guarantees that it exists.
template <int KIND>
__device__ __forceinline__ void slow_tie_walk(const KeySource<KIND>& ks, const CacheView& c, const Shape& sh,
                                              const StepArgs& sa, int seq, uint32_t key_thr, int64_t quota,
                                              ResolveShared* sm) {
    const int tid = threadIdx.x;
    int64_t need = quota;
    auto is_tie = [&](int g, const SegView& v, int j, int* p) {
        float sc;
        return j < v.len && ks.entry_at(g, v, j, p, &sc) && key_of_score(sc) == key_thr;
    };
    for (int g = seq * sh.segs_per_seq; g < (seq + 1) * sh.segs_per_seq; ++g) {
        bool bad = false, nocap = false;
        const SegView v = seg_view<KIND>(c, g, sh.nseg, sa, &bad, &nocap);
        const int len = v.len;
        int mine = 0, p;
        for (int j = tid; j < len; j += FAST_THREADS) mine += is_tie(g, v, j, &p);
        const int in_seg = block_sum<int32_t>(mine, sm->lds32);
        if (need > in_seg) {
            need -= in_seg;
            continue;
        }
        if (KIND == SCAN_PAGED) {
            // the entry is in this segment, whose slots are in no particular order: the need-th smallest position
            // among its ties is the need-th largest of 0x7fffffff - position - three digits, as for the keys
            uint32_t prefix = 0;
            int64_t rank = need;
            tie_pos_pass<0>(ks, g, v, key_thr, &prefix, &rank, sm);
            tie_pos_pass<1>(ks, g, v, key_thr, &prefix, &rank, sm);
            tie_pos_pass<2>(ks, g, v, key_thr, &prefix, &rank, sm);
            __syncthreads();
            if (tid == 0) {
                sm->found_seg = g;
                sm->found_pos = (int)(0x7fffffffu - prefix);
            }
            __syncthreads();
            return;
        }
        // the entry is in this segment: entries are stored in position order
        int64_t running = 0;
        for (int base = 0; base < len; base += FAST_THREADS) {    // uniform trip count
            const int j = base + tid;
            int pj = 0;
            const int is_eq = is_tie(g, v, j, &pj);
            int32_t tot;
            const int32_t ex = block_excl_scan<int32_t>(is_eq, sm->lds32, &tot);
            if (is_eq && running + ex == need - 1) {
                sm->found_seg = g;
                sm->found_pos = pj;
            }
            running += tot;
            if (running >= need) break;                           // uniform: tot comes from LDS
        }
        __syncthreads();
        return;
    }
    __syncthreads();
}

// loads and stores that bypass the caches which are not coherent across the chip (what one block writes this way
// and has seen acknowledged, another block reads this way without any fence)
template <typename T>
__device__ __forceinline__ T ld_dev(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void st_dev(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Several segments to a block: a segment's own threads walk its first `limit` entries (scan_grid), and then all threads of
// the block together what is left of the longer ones.  (With a wavefront per segment the longest of 16 lists would set
// the time of the block, and the lists of a global budget are uneven: one of 60 K entries among 4096 of 500, 840 us with
// the single-block select that its own sub-list's overflow brought, 230 without, now 48.)  Returns the segments of block blk
// of a sequence's bpq (bit: their group) of which something may be left - every wavefront finds out for itself, so no
// barrier is needed.
template <int KIND>
__device__ __forceinline__ uint32_t long_segments(const CacheView& c, const StepArgs& sa, const Shape& sh, int seq, int bpq, int blk,
                                                  int spb, int limit) {
    const int s = lane_id() * bpq + blk;
    int64_t most = 0;                                             // entries the segment has at most
    if (lane_id() < spb && s < sh.segs_per_seq) {
        const int g = seq * sh.segs_per_seq + s;
        most = KIND == SCAN_PAGED ? (int64_t)sa.pg.seg_pages[g] * KVTRIM_PAGE_SIZE : (int64_t)c.seg_len[g] + (KIND == SCAN_STEP ? sa.n_new : 0);
    }
    return (uint32_t)__ballot(most > limit);
}

// What the one-call decode step needs besides the scan, for the 16 segments from seg0 on, a wavefront each: the segment's
// new tokens enter the source cache, and its part of the row mover's chunk table is written.  Both are read by the next
// kernel only.  (A block per segment of 1024 threads was half the grid of the scoring kernel: at 4096 segments its
// blocks alone took eight rounds of the chip.)
__device__ __forceinline__ void write_step_tables(const CacheView& c, const Shape& sh, const Workspace& ws, const StepArgs& sa,
                                                  int seg0, int32_t* lds32 /* [17] */) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int seg = seg0 + wave;
    const bool mine = seg < sh.nseg;
    bool bad = false, nocap = false;                              // (reported by the scanning blocks)
    SegView v{};
    if (mine) v = seg_view<SCAN_STEP>(c, seg, sh.nseg, sa, &bad, &nocap);
    // the chunks of the segments before the block's are counted here
    int before = 0;
    for (int g = tid; g < seg0; g += FAST_THREADS) {
        bool b2 = false, n2 = false;
        before += (seg_view<SCAN_STEP>(c, g, sh.nseg, sa, &b2, &n2).len + CMP_CHUNK - 1) / CMP_CHUNK;
    }
    if (mine) {
        // ---- this segment's new tokens enter the source cache (rows: 16 bytes per lane; metadata)
        const int cnt_new = v.len - v.len_old, vpr = sh.head_dim / 8;
        const uint4* kn = reinterpret_cast<const uint4*>(sa.k_new) + (int64_t)seg * sa.n_new * vpr;
        const uint4* vn = reinterpret_cast<const uint4*>(sa.v_new) + (int64_t)seg * sa.n_new * vpr;
        uint4* kd = reinterpret_cast<uint4*>(sa.src.k) + (v.start + v.len_old) * vpr;
        uint4* vd = reinterpret_cast<uint4*>(sa.src.v) + (v.start + v.len_old) * vpr;
        for (int i = lane; i < cnt_new * vpr; i += 64) {
            kd[i] = kn[i];
            vd[i] = vn[i];
        }
        if (lane < cnt_new) {                                     // (n_new <= STEP_MAX_NEW)
            const int64_t e = v.start + v.len_old + lane, ni = (int64_t)seg * sa.n_new + lane;
            sa.src.log_beta[e] = sa.lb_new[ni];
            if (c.log_tail) sa.src.log_tail[e] = sa.lt_new[ni];
            sa.src.pos[e] = sa.pos_new[ni];
        }
    }
    before = block_sum<int32_t>(before, lds32);
    const int nch = (v.len + CMP_CHUNK - 1) / CMP_CHUNK;          // (0 behind the last segment)
    __syncthreads();
    if (lane == 0) lds32[wave] = nch;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before += lds32[w];
    if (!mine) return;
    for (int ch = lane; ch < nch; ch += 64) {
        ChunkDesc d;
        d.first = v.start + (int64_t)ch * CMP_CHUNK;
        d.n = min(CMP_CHUNK, v.len - ch * CMP_CHUNK);
        d.seg = seg;
        ws.cmp_desc[before + ch] = d;
    }
    if (lane == 0) {
        ws.cmp_chunk_prefix[seg] = before;
        if (seg == sh.nseg - 1) ws.cmp_chunk_prefix[sh.nseg] = before + nch;
        if (!sa.inplace) ws.step_len[seg] = v.len;                // (in place: the sequence's last block leaves the survivors' count there)
    }
}
static_assert(STEP_MAX_NEW <= 64, "a lane per new token");

// Stage 1 is computed here, and written to score_out.
// STEP: the decode step in one call.  Every block scores its segments' new tokens from the new-token
// buffers; more blocks, behind the scanning ones of the grid, write their rows and metadata into the source cache and
// the row mover's chunk table (write_step_tables).  The last block of a sequence also leaves
// what the compaction needs: survivors per segment, the destination's segment table and - when the evicted entries
// are on the candidate list - per chunk of 128 entries the number of entries it loses and per segment a record with
// the start of its survivors in the destination and the indices of its evicted entries, from which a block of the
// row mover places its chunk's survivors itself (and writes its mask bytes).  After the single-block select, or
// with more evictions than the lists hold, it writes the whole mask and a destination offset per chunk instead.
//
// Cross-block traffic inside the kernel: the candidate lists, their counters, the lowest keys and the arrival
// counters.  All of it is written with device-scope atomics or write-through stores whose acknowledgement the
// writer waits for before it arrives, and read with device-scope loads - so no block needs a fence, which on this
// chip means a write-back of a whole L2.  The scores written here are read by the NEXT kernel only; the
// single-block select, which has to look at every entry, recomputes them from the call's inputs.
template <int KIND, int DEAL>
__global__ __launch_bounds__(FAST_THREADS) void k_fast_scan(CacheView c, const int32_t* __restrict__ now,
                                                            float* score_out,
                                                            const int64_t* __restrict__ budget, Shape sh, Workspace ws,
                                                            int bps, int spb_arg, int limit, int32_t* __restrict__ kept_out,
                                                            uint32_t* __restrict__ thr_out, StepArgs sa) {
    constexpr bool STEP = KIND == SCAN_STEP, PAGED = KIND == SCAN_PAGED, MULTI = DEAL == DEAL_MULTI, WHOLE = DEAL >= DEAL_WHOLE, PARTS = DEAL == DEAL_PARTS;
    __shared__ ResolveShared sm;
    __shared__ int s_last, s_ncand;
    __shared__ uint32_t s_base[FAST_SUB];
    // This block's candidates, before they go to the list; the last block of a sequence reuses the space (STEP).  A block of
    // several segments, which may be all of its sequence, stages as many as the list holds.
    constexpr int STAGE = DEAL == DEAL_SEGMENT ? FAST_STAGE : FL_CAP_MAX;
    constexpr int STAGE_AT = WHOLE ? 5 * FAST_STAGE : 0;          // (WHOLE: behind the tables, which it needs from the beginning)
    constexpr bool IDX = STEP || PAGED;                           // where a candidate lies: its index in the segment (STEP), its slot (PAGED)
    __shared__ int32_t s_pool[STAGE_AT + (IDX ? 4 : 3) * STAGE];
    uint32_t* c_key = reinterpret_cast<uint32_t*>(s_pool + STAGE_AT);
    int32_t* c_pos = s_pool + STAGE_AT + STAGE;
    int32_t* c_seg = s_pool + STAGE_AT + 2 * STAGE;
    int32_t* c_idx = s_pool + STAGE_AT + (IDX ? 3 : 2) * STAGE;
    // tables of the sequence's segments (STEP, WHOLE): entries before it, length, chunks before it, start, entries in the cache
    uint32_t* s_before = reinterpret_cast<uint32_t*>(s_pool);
    uint32_t* s_len = reinterpret_cast<uint32_t*>(s_pool) + FAST_STAGE;
    uint32_t* s_chb = reinterpret_cast<uint32_t*>(s_pool) + 2 * FAST_STAGE;
    uint32_t* s_start = reinterpret_cast<uint32_t*>(s_pool) + 3 * FAST_STAGE;
    uint32_t* s_old = reinterpret_cast<uint32_t*>(s_pool) + (WHOLE ? 4 : 0) * FAST_STAGE;
    __shared__ int s_ev[STEP ? STEP_MAX_SEGS : 1], s_off[STEP ? STEP_MAX_SEGS : 1];
    __shared__ int s_seqcnt[STEP ? STEP_MAX_SEQS + 1 : 1];        // entries before each sequence
    static_assert(STEP_MAX_EVICT < 1 << 16 && STEP_MAX_SEGS <= FAST_STAGE && STEP_MAX_SEGS <= FAST_THREADS && STEP_MAX_EVICT <= FAST_STAGE, "the step's tables reuse the staging space, one segment per thread");
    const int tid = threadIdx.x;
    // bps blocks share a segment, or (MULTI: bps = 1) spb segments of a sequence share a block, FAST_THREADS / spb threads to
    // each (whole wavefronts).  A block takes every bpq-th segment, so that neighbouring segments - a layer's, whose
    // candidates come in the same steps - are staged by different blocks.  STEP: behind the scanning blocks the grid has blocks
    // that only write the segments' tables, a wavefront per segment.
    // WHOLE: a block walks all segments of its sequence; PARTS: of a sequence of more than a batch up to bps (= gridDim.y)
    // blocks walk a part each, and a shorter one's other blocks have nothing to do.
    const int spb = MULTI ? spb_arg : 1;
    const int bpq = WHOLE ? 1 : (sh.segs_per_seq + spb - 1) / spb * bps;   // scanning blocks per sequence
    const bool tables_only = STEP && (int)blockIdx.x >= sh.n_seq * bpq;
    const int threads = FAST_THREADS / spb, group = tid / threads, gt = tid % threads;
    const int seq = tables_only ? 0 : (int)blockIdx.x / bpq;
    const int blk_in_seq = tables_only ? 0 : (int)blockIdx.x % bpq;
    const int part = blk_in_seq % bps;
    const int seg_in_seq = MULTI ? group * bpq + blk_in_seq : blk_in_seq / bps;
    const bool no_seg = !tables_only && seg_in_seq >= sh.segs_per_seq;   // (a block may have a group to spare)
    const int own_seg = seq * sh.segs_per_seq + min(seg_in_seq, sh.segs_per_seq - 1);
    // Device-scope atomics on one line are served one after the other (some 5 ns each), so the blocks of a sequence do
    // not meet on one word: the list is kept in up to FAST_SUB sub-lists with a counter each, the lowest key and the
    // arrivals in FAST_SUB group words (then one top-level arrival per group), and every word lies on a
    // line of its own (256 segments of 4096 entries: 2.2 us from the end of the scores to a place on the list instead of 3.7).
    const int nblk = bpq;
    const int nsub_log = nblk < FAST_SUB ? 31 - __clz(nblk) : 4;   // (a power of two: no division to find a slot's sub-list)
    static_assert(FAST_SUB == 16 && FAST_SUB == FAST_THREADS / 64, "the resolving block has a wavefront for every sub-list");
    const int nsub = 1 << nsub_log;
    const int sub = blk_in_seq & (nsub - 1);
    if (tid == 0) s_ncand = 0;
    __syncthreads();
    // the tables-only blocks take no part in the scan, so a sequence's last block never waits for them
    if (tables_only) {
        if (PARTS && blockIdx.y > 0) return;
        write_step_tables(c, sh, ws, sa, ((int)blockIdx.x - sh.n_seq * bpq) * (FAST_THREADS / 64), sm.lds32);
        return;
    }
    bool bad = false, nocap = false;
    SegView own{};
    if (!WHOLE) own = seg_view<KIND>(c, own_seg, sh.nseg, sa, &bad, &nocap);
    const int own_len = no_seg ? 0 : own.len;
    if (!WHOLE && gt == 0 && part == 0 && !no_seg && (bad || nocap)) atomicOr(ws.err, bad ? ERR_LAYOUT : ERR_CAP);
    const uint32_t hi = ws.fast_hi[seq];
    const uint32_t cap = (uint32_t)ws.fl_cap;
    const uint32_t subcap = cap >> nsub_log;                      // entries per sub-list
    uint32_t* lk = ws.fl_key + (size_t)seq * cap;
    int32_t* ls = ws.fl_seg + (size_t)seq * cap;
    int32_t* lp = ws.fl_pos + (size_t)seq * cap;
    int32_t* li = ws.fl_idx + (size_t)seq * cap;
    const uint32_t wstride = (uint32_t)ws.fast_stride;
    uint32_t* sub_count = ws.fl_count + (size_t)seq * FAST_SUB * wstride;
    uint32_t* grp_min = ws.fast_min + (size_t)seq * FAST_SUB * wstride;
    uint32_t* done = ws.fast_done + (size_t)seq * (FAST_SUB + 1) * wstride;
    KeySource<KIND> ks;
    ks.bt = sa.pg.block_table;
    ks.n_pages = sa.pg.n_pages;
    ks.lb = c.log_beta;
    ks.lt = c.log_tail;
    ks.pos = c.pos;
    ks.lb_new = sa.lb_new;
    ks.lt_new = sa.lt_new;
    ks.pos_new = sa.pos_new;
    ks.n_new = sa.n_new;
    ks.t1 = now[seq] + 1;
    // (the mask then needs no selection; a vector load, for which nothing waits before the first scores are there: 0.5 us of 47)
    const bool none_stays = PAGED && ld_dev(&budget[seq]) <= 0;

    const int g0 = seq * sh.segs_per_seq;
    // STEP: one scan over the segments of the batch (1024 at a time): entries and chunks before each, so the entries of every
    // sequence (the destination of a sequence starts behind all earlier ones) and this sequence's part of the tables
    // fall out of it.  (The staging space is free once the block has arrived; entries of a cache are below 2^31.)
    auto step_tables = [&]() {
        uint64_t carry = 0;                                       // entries in the upper, chunks in the lower 28 bits
        for (int base = 0; base < sh.nseg; base += FAST_THREADS) {
            const int g = base + tid;
            uint64_t v = 0;
            SegView sv{};
            bool b2 = false, n2 = false;
            if (g < sh.nseg) {
                sv = seg_view<KIND>(c, g, sh.nseg, sa, &b2, &n2);
                v = (uint64_t)sv.len << 28 | (uint64_t)((sv.len + CMP_CHUNK - 1) / CMP_CHUNK);
            }
            uint64_t tot;
            const uint64_t ex = carry + block_excl_scan<uint64_t>(v, reinterpret_cast<uint64_t*>(sm.lds64), &tot);
            carry += tot;
            if (sh.n_seq == 1) {
                if (g == 0) s_seqcnt[0] = 0;
            } else if (g < sh.nseg && g % sh.segs_per_seq == 0) {
                s_seqcnt[g / sh.segs_per_seq] = (int)(uint32_t)(ex >> 28);
            }
            if (g >= g0 && g < g0 + sh.segs_per_seq) {
                if (!PARTS) kept_out[g] = 0;
                s_start[g - g0] = (uint32_t)sv.start;
                s_len[g - g0] = (uint32_t)sv.len;
                s_chb[g - g0] = (uint32_t)(ex & 0xFFFFFFFu);
                if (WHOLE) {
                    s_before[g - g0] = (uint32_t)(ex >> 28);
                    s_old[g - g0] = (uint32_t)sv.len_old;
                    if (b2 || n2) atomicOr(ws.err, b2 ? ERR_LAYOUT : ERR_CAP);
                }
            }
        }
        if (tid == 0) s_seqcnt[sh.n_seq] = (int)(uint32_t)(carry >> 28);
        __syncthreads();
    };

    // what the ranking and the step's tables count in, long before they do
    auto clear_lds = [&]() {
        sm.h[tid] = 0;
        if (tid == 0) sm.gather_n = 0;
        if (STEP) s_ev[tid] = 0;
    };
    static_assert(!STEP || STEP_MAX_SEGS == FAST_THREADS, "a counter per thread");
    int64_t cnt = 0;                                              // entries of the sequence (not STEP: of this thread's segments)
    uint32_t key[FAST_ITEMS];
    int sg[FAST_ITEMS], ps[FAST_ITEMS], ix[FAST_ITEMS];
    bool valid[FAST_ITEMS], listed[FAST_ITEMS];
    bool sub_overflow = false;
    int live_mine = 0;                                            // PAGED, WHOLE: live entries of segment g0 + tid
    uint32_t n_list = 0, min_key = 0xFFFFFFFFu;
    if constexpr (WHOLE) {
        // ---- the whole sequence: its entries as one flat range, in equal shares of whole 64s to the wavefronts, so that it
        // does not matter how they are spread over the segments; a lane follows the table from entry to entry
        uint32_t total;
        clear_lds();
        if (STEP) {
            step_tables();
            total = (uint32_t)s_seqcnt[seq + 1] - (uint32_t)s_seqcnt[seq];
        } else {
            SegView sv{};
            bool b2 = false, n2 = false;
            if (tid < sh.segs_per_seq) {
                sv = seg_view<KIND>(c, g0 + tid, sh.nseg, sa, &b2, &n2);
                // (a sequence's first block always takes part.  One without a part is not waited for: it may read the tables while the
                // resolving block shortens them, and see a page count and a live count that do not belong together.  It
                // then counts fewer entries than there were, and still finds no part for itself)
                if (b2 && (!PARTS || blockIdx.y == 0)) atomicOr(ws.err, ERR_LAYOUT);
                if (!PAGED && !PARTS) kept_out[g0 + tid] = 0;     // the mask kernel adds its counts
                if (PAGED) live_mine = sv.live;
                cnt = sv.live;
            }
            int32_t tot;
            const int32_t ex = block_excl_scan<int32_t>(sv.len, sm.lds32, &tot);
            if (tid < sh.segs_per_seq) {
                s_before[tid] = (uint32_t)ex;
                s_len[tid] = (uint32_t)sv.len;
                s_start[tid] = (uint32_t)sv.start;
            }
            total = (uint32_t)tot;
            __syncthreads();
        }
        const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        constexpr uint32_t NW = FAST_THREADS / 64;
        const uint32_t first_before = STEP ? (uint32_t)s_seqcnt[seq] : 0u;
        uint32_t share = (total + NW * 64 - 1) / (NW * 64) * 64, w = (uint32_t)wave, parts = 1;
        if (PARTS) {
            if (total > WHOLE_ENTRIES) {
                parts = min((uint32_t)bps, (total - 1) / WHOLE_ENTRIES + 1);
                share = (total + parts * NW * 64 - 1) / (parts * NW * 64) * 64;
                w += blockIdx.y * NW;
            }
            if (blockIdx.y >= parts) return;                      // (the whole block: there is no part for it)
        }
        const uint32_t i0 = first_before + min(total, w * share), i1 = first_before + min(total, (w + 1) * share);
        int sl = -1;                                              // the segment of this lane's entry
        for (int base = 0; base < sh.segs_per_seq; base += 64)
            sl += __popcll(__ballot(base + lane < sh.segs_per_seq && s_before[min(base + lane, sh.segs_per_seq - 1)] <= i0));
        sl = max(sl, 0);
        uint32_t mn = 0xFFFFFFFFu;
        for (uint32_t b0 = i0; b0 < i1; b0 += 64 * FAST_BATCH) {
            float sv[FAST_BATCH];
            int pv[FAST_BATCH], seg[FAST_BATCH], jj[FAST_BATCH];
            int64_t at[FAST_BATCH], sat[FAST_BATCH];              // where the entry lies in the arrays, and its score
            bool isnew[FAST_BATCH], in[FAST_BATCH];
            bool bad_page = false;
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                const uint32_t i = b0 + u * 64 + lane;
                in[u] = i < i1;
                if (in[u])
                    while (i >= s_before[sl] + s_len[sl]) ++sl;
                seg[u] = sl;
                jj[u] = in[u] ? (int)(i - s_before[sl]) : 0;
                isnew[u] = STEP && in[u] && jj[u] >= (int)s_old[sl];
                SegView v{};
                v.start = PAGED ? (int64_t)(g0 + sl) * sa.pg.max_pps : (int64_t)s_start[sl];
                sat[u] = in[u] ? ks.place(v, jj[u], &bad_page) : 0;
                at[u] = isnew[u] ? (int64_t)(g0 + sl) * sa.n_new + (jj[u] - (int)s_old[sl]) : sat[u];
            }
            if (PAGED && bad_page) atomicOr(ws.err, ERR_LAYOUT);
            float lbv[FAST_BATCH], ltv[FAST_BATCH];
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                pv[u] = in[u] ? (isnew[u] ? sa.pos_new : c.pos)[at[u]] : 0;
                lbv[u] = in[u] ? (isnew[u] ? sa.lb_new : c.log_beta)[at[u]] : 0.f;
                ltv[u] = (in[u] && c.log_tail) ? (isnew[u] ? sa.lt_new : c.log_tail)[at[u]] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                const float dt = (float)(ks.t1 - pv[u]);
                sv[u] = c.log_tail ? __fmaf_rn(dt, lbv[u], ltv[u]) : __fmul_rn(dt, lbv[u]);
                if (PAGED && pv[u] < 0) sv[u] = 0.f;              // an empty slot's score reads 0
                if (in[u]) score_out[sat[u]] = sv[u];
                const uint32_t k2 = key_of_score(sv[u]);
                const bool live = in[u] && (!PAGED || pv[u] >= 0);
                if (PAGED && in[u]) st_dev(&sa.keep_out[sat[u]], (uint8_t)(live && !none_stays));
                if (live) mn = min(mn, k2);
                if (live && k2 < hi) {
                    const int slot = atomicAdd(&s_ncand, 1);
                    if (slot < STAGE) {
                        c_key[slot] = k2;
                        c_pos[slot] = pv[u];
                        c_seg[slot] = g0 + seg[u];
                        if (IDX) c_idx[slot] = STEP ? jj[u] : (int)sat[u];
                    }
                }
            }
        }
        min_key = block_min_u32(mn, sm.red_u);                    // (its barriers also complete s_ncand and the staged entries)
        if (PARTS && parts > 1) {
            // The blocks of a long sequence meet on its list in memory, each with one place for all it has staged (they are 8 at
            // most), and the last takes the list into its LDS, as if it had walked the sequence alone.
            const int ncand = s_ncand;
            uint32_t* k_list = ws.fl_key + (size_t)seq * cap;
            int32_t* s_list = ws.fl_seg + (size_t)seq * cap;
            int32_t* p_list = ws.fl_pos + (size_t)seq * cap;
            int32_t* i_list = ws.fl_idx + (size_t)seq * cap;
            const size_t at_word = (size_t)seq * (uint32_t)ws.fast_stride;
            uint32_t* count = ws.fl_count + FAST_SUB * at_word;
            uint32_t* lowest = ws.fast_min + FAST_SUB * at_word;
            uint32_t* arrived = ws.fast_done + (FAST_SUB + 1) * at_word;
            if (tid == 0) {
                if (min_key != 0xFFFFFFFFu) atomicMin(lowest, min_key);
                s_base[0] = ncand ? atomicAdd(count, ncand > STAGE ? cap + 1u : (uint32_t)ncand) : 0u;
            }
            __syncthreads();
            for (int i = tid; i < ncand && ncand <= STAGE; i += FAST_THREADS) {
                const uint32_t slot = s_base[0] + (uint32_t)i;
                if (slot < cap) {
                    st_dev(&k_list[slot], c_key[i]);
                    st_dev(&s_list[slot], c_seg[i]);
                    st_dev(&p_list[slot], c_pos[i]);
                    if (IDX) st_dev(&i_list[slot], c_idx[i]);
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this thread's list entries are acknowledged ...
            __syncthreads();                                      // ... and so are the whole block's, before it arrives
            if (tid == 0) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // (thread 0's own atomics above have returned)
                s_last = atomicAdd(arrived, 1u) == parts - 1u;
            }
            __syncthreads();
            if (!s_last) return;
            const uint32_t n = ld_dev(count);
            min_key = ld_dev(lowest);
            for (uint32_t i = tid; i < n && n <= cap; i += FAST_THREADS) {   // (cap <= STAGE)
                c_key[i] = ld_dev(&k_list[i]);
                c_seg[i] = ld_dev(&s_list[i]);
                c_pos[i] = ld_dev(&p_list[i]);
                if (IDX) c_idx[i] = ld_dev(&i_list[i]);
            }
            __syncthreads();                                      // every thread has read the per-call words ...
            if (tid == 0) {                                       // ... which go back to "between calls"
                s_ncand = n <= cap ? (int)n : STAGE + 1;
                atomicExch(arrived, 0u);
                atomicExch(count, 0u);
                atomicExch(lowest, 0xFFFFFFFFu);
            }
            __syncthreads();
        }
        if (PARTS && !PAGED && tid < sh.segs_per_seq) kept_out[g0 + tid] = 0;   // (here: by the block that will write the counts, no other)
        if (PAGED && tid < sh.segs_per_seq) st_dev(&kept_out[g0 + tid], live_mine);
        n_list = (uint32_t)s_ncand;
        sub_overflow = n_list > (uint32_t)STAGE;
#pragma unroll
        for (int u = 0; u < FAST_ITEMS; ++u) {
            const int i = u * FAST_THREADS + tid;
            valid[u] = !sub_overflow && (uint32_t)i < n_list;
            listed[u] = valid[u];
            key[u] = valid[u] ? c_key[i] : 0u;
            sg[u] = valid[u] ? c_seg[i] : 0;
            ps[u] = valid[u] ? c_pos[i] : 0;
            ix[u] = IDX && valid[u] ? c_idx[i] : 0;
        }
    }
    // ---- every entry of this block's share: score, and onto the list if its key is below the bound
    if constexpr (!WHOLE) {
        uint32_t mn = 0xFFFFFFFFu;
        SegView sv0 = own;
        int seg = own_seg, first = part * threads + gt, stride = bps * threads;
        int len = MULTI ? min(own_len, limit) : own_len;
        uint32_t todo = MULTI ? long_segments<KIND>(c, sa, sh, seq, bpq, blk_in_seq, spb, limit) : 0;
        for (;;) {                                                // the threads' own segments, then (MULTI) what is left of long ones
        const int64_t start = sv0.start;
        // batches of FAST_BATCH entries per thread: all loads of a batch are issued before any of them is used
        for (int j0 = first; j0 < len; j0 += stride * FAST_BATCH) {
            float sv[FAST_BATCH];
            int pv[FAST_BATCH];
            int64_t at[FAST_BATCH];                               // where the entry lies in the arrays
            bool bad_page = false;
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                const int j = j0 + u * stride;
                const bool isnew = STEP && j >= sv0.len_old;
                at[u] = isnew ? (int64_t)seg * sa.n_new + (j - sv0.len_old) : (j < len ? ks.place(sv0, j, &bad_page) : 0);
            }
            if (PAGED && bad_page) atomicOr(ws.err, ERR_LAYOUT);
            float lbv[FAST_BATCH], ltv[FAST_BATCH];
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                const int j = j0 + u * stride;
                const bool in = j < len;
                const bool isnew = STEP && j >= sv0.len_old;
                pv[u] = in ? (isnew ? sa.pos_new : c.pos)[at[u]] : 0;
                lbv[u] = in ? (isnew ? sa.lb_new : c.log_beta)[at[u]] : 0.f;
                ltv[u] = (in && c.log_tail) ? (isnew ? sa.lt_new : c.log_tail)[at[u]] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                const int j = j0 + u * stride;
                const float dt = (float)(ks.t1 - pv[u]);
                sv[u] = c.log_tail ? __fmaf_rn(dt, lbv[u], ltv[u]) : __fmul_rn(dt, lbv[u]);
                if (PAGED && pv[u] < 0) sv[u] = 0.f;              // an empty slot's score reads 0
                if (j < len) score_out[STEP ? start + j : at[u]] = sv[u];
            }
#pragma unroll
            for (int u = 0; u < FAST_BATCH; ++u) {
                const int j = j0 + u * stride;
                const uint32_t key = key_of_score(sv[u]);
                const bool live = j < len && (!PAGED || pv[u] >= 0);
                if (PAGED && j < len) st_dev(&sa.keep_out[at[u]], (uint8_t)(live && !none_stays));
                if (live) mn = min(mn, key);
                if (live && key < hi) {                           // rare: a few hundred entries per sequence and call
                    const int slot = atomicAdd(&s_ncand, 1);
                    if (slot < STAGE) {
                        c_key[slot] = key;
                        c_pos[slot] = pv[u];
                        c_seg[slot] = seg;
                        if (IDX) c_idx[slot] = STEP ? j : (int)at[u];
                    }
                }
            }
        }
        if (!MULTI || todo == 0) break;                           // (uniform)
        seg = seq * sh.segs_per_seq + __builtin_ctz(todo) * bpq + blk_in_seq;
        todo &= todo - 1;
        bool b2 = false, n2 = false;                              // (reported by the segment's own threads)
        sv0 = seg_view<KIND>(c, seg, sh.nseg, sa, &b2, &n2);
        first = limit + tid;
        stride = FAST_THREADS;
        len = sv0.len;
        }
        mn = block_min_u32(mn, sm.red_u);                         // (its barriers also complete s_ncand and the staged entries)
        const int ncand = s_ncand;
        // One reservation per block; MULTI: one per 64 candidates (more where the sub-lists are few), in neighbouring sub-lists, so
        // that a block with the segments of a hot layer does not fill its own.  A block with more candidates than it can
        // stage makes its sub-list overflow.
        int shift = MULTI ? FAST_PIECE_SHIFT : 31;
        while (MULTI && nsub << shift < min(ncand, STAGE)) ++shift;
        const int npiece = ncand > STAGE || !MULTI ? min(ncand, 1) : (ncand + (1 << shift) - 1) >> shift;
        auto list_of = [&](int p) { return sub + p < nsub ? sub + p : sub + p - nsub; };
        if (tid == 0 && mn != 0xFFFFFFFFu) atomicMin(&grp_min[sub * wstride], mn);
        if (tid < npiece)
            s_base[tid] = atomicAdd(&sub_count[list_of(tid) * wstride], ncand > STAGE ? cap + 1u : (uint32_t)(MULTI ? min(1 << shift, ncand - (tid << shift)) : ncand));
        __syncthreads();
        if (ncand > 0 && ncand <= STAGE) {
            for (int i = tid; i < ncand; i += FAST_THREADS) {
                const int p = MULTI ? i >> shift : 0;
                const uint32_t slot = s_base[p] + (uint32_t)(MULTI ? i - (p << shift) : i);
                if (slot < subcap) {
                    const size_t at = (size_t)list_of(p) * subcap + slot;
                    st_dev(&lk[at], c_key[i]);
                    st_dev(&ls[at], c_seg[i]);
                    st_dev(&lp[at], c_pos[i]);
                    if (IDX) st_dev(&li[at], c_idx[i]);
                }
            }
        }
    }
    // ---- PAGED: the scanning blocks have written the mask as if everything survived (a byte for every slot, listed or not: a list
    // may hold fewer than lie below the bound), or nothing where the budget is zero.  Here the bytes of what goes are cleared, the
    // survivors counted and, in the decode step in one call, the eviction applied: a slot that goes becomes empty, the live counts
    // of its page and segment go down, and a page left without a live entry goes back to the free list.  Of the other blocks
    // only those without a part (PARTS) may still read this sequence's tables, and they report nothing.
    // What the scanning blocks wrote of the mask has left their caches (st_dev, and acknowledged before they arrived),
    // so it does not come back over what is written here.  (A mask kernel that also evicted, and the tidying in the
    // attention's merge kernel, took 4 to 9 us: on pages 256 lists of 8192 entries 204.1 -> 201.4 us a step, 20 of 756 31.9 -> 27.9.)
    __shared__ int s_nrel, s_rel[PAGED ? FAST_BIN_DIRECT : 1];    // segments that lost pages (one may be there more than once)
    // n live entries of segment g go (mask bytes, positions and the page's live count are the caller's)
    auto take_out = [&](int g, int n) {
        atomicSub(&kept_out[g], n);
        if (sa.pg.evict) atomicSub(&sa.pg.seg_live[g], n);
    };
    auto release_page = [&](int g, int page) {
        sa.pg.page_owner[page] = -2;
        const int i = atomicAdd(&s_nrel, 1);
        if (i < FAST_BIN_DIRECT) s_rel[i] = g;
    };
    // before the first entry is taken out: the live counts stored as survivors and the scanning blocks' bytes are in place
    auto take_out_begin = [&]() {
        __builtin_amdgcn_s_waitcnt(VMCNT_0);
        if (tid == 0) s_nrel = 0;
        __syncthreads();
    };
    // a wavefront to a segment
    auto tidy_paged = [&]() {
        __syncthreads();
        const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int nrel = none_stays ? FAST_BIN_DIRECT + 1 : s_nrel;
        if (nrel > FAST_BIN_DIRECT) {
            for (int i = wave; i < sh.segs_per_seq; i += FAST_THREADS / 64) tidy_segment_by_wave(sa.pg, g0 + i, none_stays, ws.err);
            return;
        }
        for (int i = wave; i < nrel; i += FAST_THREADS / 64) {
            const int g = s_rel[i];
            bool twice = false;                                   // (whoever comes first in the list does it)
            for (int b = 0; b < i; b += 64) twice |= __any(b + lane < i && s_rel[min(b + lane, FAST_BIN_DIRECT - 1)] == g);
            if (!twice) tidy_segment_by_wave(sa.pg, g, false, ws.err);
        }
    };
    uint32_t word = 0;
    const int lane = lane_id();
    // The resolving block's wavefronts share the sub-lists equally, a sub-list each when there are 16: a thread holds slots
    // slot0, slot0 + 64, ... of its wavefront's.  The first 128 of a wavefront are asked for before the counter is known
    // and the rest only if it reaches them.
    const int wave_of = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t my_sub = (uint32_t)wave_of >> (4 - nsub_log);
    const uint32_t slot0 = ((uint32_t)wave_of & ((16u >> nsub_log) - 1u)) * (64 * FAST_ITEMS) + (uint32_t)lane;
    auto load_slot = [&](int u) {
        const uint32_t i = slot0 + u * 64;
        if (i < subcap) {
            const uint32_t at = my_sub * subcap + i;
            key[u] = ld_dev(&lk[at]);
            sg[u] = ld_dev(&ls[at]);
            ps[u] = ld_dev(&lp[at]);
            if (IDX) ix[u] = ld_dev(&li[at]);
        }
    };
    if constexpr (!WHOLE) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // this thread's list entries are acknowledged ...
    __syncthreads();                                              // ... and so are the whole block's, before it arrives
    if (tid == 0) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // (thread 0's own atomics above have returned)
        int last = 0;
        if (nblk <= 2 * FAST_SUB) {                               // few enough to meet on one word
            last = atomicAdd(&done[0], 1u) == (unsigned)nblk - 1u;
        } else {
            const int grp = blk_in_seq % FAST_SUB;
            const unsigned gsize = (unsigned)(nblk - grp + FAST_SUB - 1) / FAST_SUB;   // blocks of the sequence with this group number
            if (atomicAdd(&done[(1 + grp) * wstride], 1u) == gsize - 1u) last = atomicAdd(&done[0], 1u) == FAST_SUB - 1u;
        }
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;

    // ---- the last block of the sequence: everything of the sequence has been scored and listed.
    // All it needs is requested at once: the sub-list counters, the lowest keys, the first half of every sub-list (whether
    // a slot holds an entry is known once the counters are here), the segment lengths, the budget.  From here on one
    // compute unit works alone, so what counts is the chain: scans by DPP, one of them over all segments of the batch
    // and one for the destination, the counters a lane per word, no reduction for the key range (256 segments of 4096
    // entries, the whole kernel: 28.6 -> 22.8 us; 16 segments of 65: 21.5 -> 15.6).
    clear_lds();
    // (a lane per word: 0..15 the sub-lists' counters, 16..31 the groups' lowest keys)
    word = 0xFFFFFFFFu;
    if (lane < FAST_SUB) word = lane < nsub ? ld_dev(&sub_count[lane * wstride]) : 0u;
    else if (lane < 2 * FAST_SUB) word = ld_dev(&grp_min[(lane - FAST_SUB) * wstride]);
#pragma unroll
    for (int u = 0; u < FAST_ITEMS; ++u) {
        key[u] = 0;
        sg[u] = ps[u] = ix[u] = 0;
        if (u < FAST_ITEMS / 2) load_slot(u);
    }
    }
    int64_t bud = budget[seq];
    const int sq_other = sh.n_seq <= 64 ? lane : tid;             // (n_seq <= FAST_THREADS in a STEP)
    const int64_t bud_other = STEP && sh.n_seq > 1 ? budget[min(sq_other, sh.n_seq - 1)] : 0;
    int64_t step_before = 0, step_total = 0;                      // STEP: destination entries before this sequence / of all sequences
    int step_chunks_before = 0;                                   // STEP: chunks of the sequences before this one
    int my_len = 0;                                               // STEP: length and start of segment g0 + tid (one segment of the sequence per thread)
    uint32_t my_start = 0;
    int32_t step_ctot = 0;                                        // STEP: chunks of the sequence
    if (STEP) {
        if (!WHOLE) step_tables();
        step_chunks_before = (int)s_chb[0];
        if (tid < sh.segs_per_seq) {
            my_len = (int)s_len[tid];
            my_start = s_start[tid];
        }
        const int last_seg = sh.segs_per_seq - 1;
        step_ctot = (int32_t)s_chb[last_seg] - step_chunks_before + ((int)s_len[last_seg] + CMP_CHUNK - 1) / CMP_CHUNK;
        cnt = (int64_t)((uint32_t)s_seqcnt[seq + 1] - (uint32_t)s_seqcnt[seq]);
        auto need_of = [&](int sq, int64_t b) {                   // destination entries of a sequence
            const int64_t n = (int64_t)((uint32_t)s_seqcnt[sq + 1] - (uint32_t)s_seqcnt[sq]);
            if (b < 0) b = 0;
            return (b < n ? b : n) + (int64_t)sa.reserve * sh.segs_per_seq;
        };
        if (sh.n_seq == 1) {
            step_total = need_of(0, bud);
        } else {
            // (up to 64 sequences: every wavefront by itself)
            const int sq = sh.n_seq <= 64 ? lane : tid;
            const int64_t need = sq < sh.n_seq ? need_of(sq, bud_other) : 0;
            if (sh.n_seq <= 64) {
                const int64_t in = wave_incl_scan(need);
                step_total = lane_value(in, 63);
                step_before = lane_value(in - need, seq);
            } else {
                const int64_t ex = block_excl_scan<int64_t>(need, sm.lds64, &step_total);
                if (tid == seq) sm.before = ex;
                __syncthreads();
                step_before = sm.before;
                __syncthreads();
            }
        }
    } else if (!WHOLE) {
        for (int g = g0 + tid; g < g0 + sh.segs_per_seq; g += FAST_THREADS) {
            bool b2 = false, n2 = false;
            const int n = seg_view<KIND>(c, g, sh.nseg, sa, &b2, &n2).live;
            cnt += n;
            if (PAGED) st_dev(&kept_out[g], n);                   // (what is evicted is taken from it below)
            else kept_out[g] = 0;                                 // the mask kernel adds its counts
        }
    }
    if (bud < 0) bud = 0;
    if constexpr (!WHOLE) {
#pragma unroll
    for (int u = 0; u < FAST_ITEMS; ++u) {
        if (u == 0) {                                             // (lanes 0..15: the counters, 16..31: the lowest keys)
            sub_overflow = __any(lane < FAST_SUB && word > subcap);
            n_list = lane_value(row_incl_scan(min(word, subcap)), FAST_SUB - 1);
            min_key = row_min(word, 2 * FAST_SUB - 1);
        }
        valid[u] = slot0 + u * 64 < min(lane_value(word, (int)my_sub), subcap);
        listed[u] = valid[u];
        if (u >= FAST_ITEMS / 2 && __any(valid[u])) load_slot(u);
    }
    }
    if (STEP) {
        // The per-chunk eviction counts of this sequence are cleared long before they are needed: the stores (write-through: the
        // counts are added with device-scope atomics) complete while the candidates are ranked.  Whatever was asked for has
        // to be here first: loads and stores are counted together, so a load that is waited for behind these waits for them too.
        __builtin_amdgcn_s_waitcnt(VMCNT_0);
        if (sa.inplace || step_total <= sa.dst.cap)
            for (int i = tid; i < step_ctot; i += FAST_THREADS) st_dev(&ws.step_chunk_ev[step_chunks_before + i], 0u);
    }
    // every listed key lies in [lowest key of the sequence, bound): no reduction over the list is needed
    uint32_t lo = min_key, hi_k = hi - 1u;
    if (!STEP) {
        cnt = block_sum<int64_t>(cnt, sm.lds64);                  // entries of the sequence
    }
    const int64_t want = bud < cnt ? bud : cnt;
    const int64_t k = cnt - want;                                 // entries to evict
    FastSel out;
    out.mode = FSEL_THRESHOLD;
    out.key_thr = 0xFFFFFFFFu;
    out.seg_thr = 0x7fffffff;
    out.pos_thr = 0x7fffffff;
    uint32_t next_hi = hi;
    bool used_fallback = false;
    if (want == 0) {
        out.mode = FSEL_NONE;
    } else if (k == 0) {
        out.mode = FSEL_ALL;
        out.key_thr = min_key;                                    // key of the last entry of the order
    } else {
        bool solved = false;
        if (!sub_overflow && (int64_t)n_list >= k + 1 && n_list <= cap) {
            // -- rank the list: the entry of rank k (0-based, eviction order) is the last retained one
            int r = (int)k;                                       // (k < n_list <= FL_CAP_MAX)
            bool first = true;
#pragma unroll 1
            for (int round = 0; round < 5; ++round) {             // every round narrows the key range by a factor of 1024
                const uint32_t range = hi_k - lo;
                const int shift = range < 1024u ? 0 : 32 - __clz(range) - 10;
                if (!first) {                                     // (the first time they were cleared long ago)
                    __syncthreads();
                    sm.h[tid] = 0;
                    if (tid == 0) sm.gather_n = 0;
                    __syncthreads();
                }
#pragma unroll
                for (int u = 0; u < FAST_ITEMS; ++u)
                    if (valid[u]) atomicAdd(&sm.h[(key[u] - lo) >> shift], 1u);
                __syncthreads();
                const int32_t v = (int32_t)sm.h[tid];
                int32_t tot;
                const int32_t ex = block_excl_scan<int32_t, true>(v, sm.lds32, &tot);
                if (ex <= r && r < ex + v) {
                    sm.bin = tid;
                    sm.before = ex;
                    sm.cnt = v;
                }
                if (first) {
                    const int m = min(3 * ((int)k + 1), tot - 1);
                    if (ex <= m && m < ex + v) sm.bin_m = tid;
                }
                __syncthreads();
                const int bin = sm.bin, bcnt = sm.cnt;
                const int before = (int)sm.before;
                if (first) {
                    // next bound: the upper edge of the bin that holds the entry of rank min(3(k+1), n - 1);
                    // doubled distance from the threshold's bin when the list was too short to reach that rank
                    uint64_t edge = (uint64_t)lo + (((uint64_t)sm.bin_m + 1) << shift);
                    if ((int64_t)tot - 1 < 3 * (k + 1)) edge += edge - ((uint64_t)lo + ((uint64_t)bin << shift));
                    next_hi = edge > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)edge;
                    first = false;
                }
                if (bcnt <= FAST_BIN_DIRECT) {
                    // few entries in the bin: rank them directly on the whole triple
#pragma unroll
                    for (int u = 0; u < FAST_ITEMS; ++u) {
                        if (valid[u] && (int)((key[u] - lo) >> shift) == bin) {
                            const int slot = atomicAdd(&sm.gather_n, 1);
                            sm.g_key[slot] = key[u];
                            sm.g_seg[slot] = sg[u];
                            sm.g_pos[slot] = ps[u];
                        }
                    }
                    if (STEP || PAGED) __builtin_amdgcn_s_waitcnt(VMCNT_0);   // (the zeros, the live counts: see `sparse` below)
                    __syncthreads();
                    if (bcnt == 1) {                              // nothing to rank
                        out.key_thr = sm.g_key[0];
                        out.seg_thr = sm.g_seg[0];
                        out.pos_thr = sm.g_pos[0];
                        solved = true;
                        break;
                    }
                    {
                        // four threads to an entry (bcnt <= 256 = a quarter of the block), each against every fourth
                        // of the others; the triples are compared without branches, so the loop's LDS reads do not
                        // wait for one another (with the short-circuit form an iteration took three dependent reads)
                        static_assert(4 * FAST_BIN_DIRECT <= FAST_THREADS, "four threads rank one entry");
                        const int me = min(tid >> 2, bcnt - 1);
                        const uint32_t mk = sm.g_key[me];
                        const int ms = sm.g_seg[me], mp = sm.g_pos[me];
                        int rank = 0;
                        for (int j = tid & 3; j < bcnt; j += 4) {
                            const uint32_t kj = sm.g_key[j];
                            const int sj = sm.g_seg[j], pj = sm.g_pos[j];
                            rank += (int)((kj < mk) | ((kj == mk) & ((sj > ms) | ((sj == ms) & (pj > mp)))));
                        }
                        rank += __shfl_xor(rank, 1, 64);
                        rank += __shfl_xor(rank, 2, 64);
                        if ((tid >> 2) < bcnt && (tid & 3) == 0 && rank == r - before) {
                            sm.found_key = mk;
                            sm.found_seg = ms;
                            sm.found_pos = mp;
                        }
                    }
                    __syncthreads();
                    out.key_thr = sm.found_key;
                    out.seg_thr = sm.found_seg;
                    out.pos_thr = sm.found_pos;
                    solved = true;
                    break;
                }
                if (shift == 0) break;                            // too many equal keys at the threshold: the plain select below
                const uint32_t nlo = lo + ((uint32_t)bin << shift);
#pragma unroll
                for (int u = 0; u < FAST_ITEMS; ++u) valid[u] = valid[u] && (int)((key[u] - lo) >> shift) == bin;
                lo = nlo;
                const uint64_t top = (uint64_t)nlo + ((1ull << shift) - 1ull);
                hi_k = top < (uint64_t)hi_k ? (uint32_t)top : hi_k;
                r -= before;
            }
        }
        if (!solved) {
            // -- plain radix select by this block alone; also the bound for the next call
            used_fallback = true;
            __syncthreads();
            int64_t rank_in;
            uint32_t ties;
            const uint32_t key_thr = slow_radix(ks, c, sh, sa, seq, want, &sm, &rank_in, &ties);
            out.key_thr = key_thr;
            if (rank_in < (int64_t)ties) {                        // only the first rank_in of the equal keys survive
                slow_tie_walk(ks, c, sh, sa, seq, key_thr, rank_in, &sm);
                out.seg_thr = sm.found_seg;
                out.pos_thr = sm.found_pos;
            }
            __syncthreads();
            const int64_t above = seed_distance(k, sh.segs_per_seq, ws.fl_cap);
            const int64_t rank_b = want - above >= 1 ? want - above : 1;
            int64_t unused_r;
            uint32_t unused_t, key_b;
            if constexpr (PAGED) {
                // what goes is taken out on the way
                take_out_begin();
                auto visit = [&](int g, const int* slot, const bool* live, const int* pos, const float* score) {
                    int page_left[SLOW_BATCH], n[SLOW_BATCH], all = 0;
#pragma unroll
                    for (int u = 0; u < SLOW_BATCH; ++u) {        // (counters that are waited for are asked for together)
                        const bool gone = live[u] && evicted_before(key_of_score(score[u]), g, pos[u], out.key_thr, out.seg_thr, out.pos_thr);
                        const uint64_t m = __ballot(gone);
                        n[u] = gone && (m & ((1ull << lane) - 1ull)) == 0 ? __popcll(m) : 0;   // (in the first of them)
                        all += __popcll(m);
                        if (gone) sa.keep_out[slot[u]] = 0;
                        if (gone && sa.pg.evict) sa.pg.pos[slot[u]] = -1;
                        page_left[u] = 1;
                        if (n[u] && sa.pg.evict) page_left[u] = atomicSub(&sa.pg.page_live[slot[u] / KVTRIM_PAGE_SIZE], n[u]) - n[u];
                    }
                    if (all && lane == 0) take_out(g, all);       // (lane 0 has an entry of every batch)
#pragma unroll
                    for (int u = 0; u < SLOW_BATCH; ++u)
                        if (page_left[u] <= 0) release_page(g, slot[u] / KVTRIM_PAGE_SIZE);
                };
                key_b = slow_radix(ks, c, sh, sa, seq, rank_b, &sm, &unused_r, &unused_t, Visit<decltype(visit)>{visit});
            } else {
                key_b = slow_radix(ks, c, sh, sa, seq, rank_b, &sm, &unused_r, &unused_t);
            }
            next_hi = key_b == 0xFFFFFFFFu ? key_b : key_b + 1u;
        }
    }
    if (out.mode != FSEL_THRESHOLD) __syncthreads();              // every thread has read the per-call words (a ranking had barriers)
    if (!WHOLE && tid <= FAST_SUB) {                              // ... which go back to "between calls"
        st_dev(&done[tid * wstride], 0u);
        if (tid < FAST_SUB) {
            st_dev(&sub_count[tid * wstride], 0u);
            st_dev(&grp_min[tid * wstride], 0xFFFFFFFFu);
        }
    }
    if (tid == 0) {
        if (out.mode == FSEL_THRESHOLD) atomicAdd(&ws.fast_stat[used_fallback ? 1 : 0], 1ull);
        ws.fast_sel[seq] = out;
        if (thr_out) thr_out[seq] = out.mode == FSEL_NONE ? 0xFFFFFFFFu : out.key_thr;
        if (out.mode == FSEL_THRESHOLD) ws.fast_hi[seq] = next_hi;
    }
    if constexpr (PAGED) {
        if (out.mode == FSEL_ALL) return;
        if (out.mode == FSEL_NONE) {
            __builtin_amdgcn_s_waitcnt(VMCNT_0);                  // (the live counts of other threads)
            __syncthreads();
            for (int i = tid; i < sh.segs_per_seq; i += FAST_THREADS) {
                kept_out[g0 + i] = 0;
                if (sa.pg.evict) sa.pg.seg_live[g0 + i] = 0;
            }
            if (!none_stays) return;                              // (there was nothing)
        } else if (!used_fallback) {
            take_out_begin();
#pragma unroll
            for (int u = 0; u < FAST_ITEMS; ++u) {
                if (!listed[u] || !evicted_before(key[u], sg[u], ps[u], out.key_thr, out.seg_thr, out.pos_thr)) continue;
                sa.keep_out[ix[u]] = 0;
                take_out(sg[u], 1);
                if (!sa.pg.evict) continue;
                sa.pg.pos[ix[u]] = -1;
                const int page = ix[u] / KVTRIM_PAGE_SIZE;
                if (atomicSub(&sa.pg.page_live[page], 1) <= 1) release_page(sg[u], page);
            }
        }
        if (sa.pg.evict) tidy_paged();
        return;
    }
    if (!STEP) return;

    // ---- STEP: what the row mover needs: survivors per segment, the destination's segment table, a destination
    // offset per chunk of 128 entries (flagged when the chunk loses nothing) and the keep mask of the chunks that do
    // lose entries.  Entry (g, position p, key) survives iff it is not behind the last retained entry `out`.
    if (STEP) {
        if (!sa.inplace && step_total > sa.dst.cap) {             // every sequence's last block takes the same decision
            if (tid == 0) atomicOr(ws.err, ERR_CAP);
            return;
        }
        const int nsg = sh.segs_per_seq;
        // The evicted entries are among the listed ones unless the single-block select ran; they are handed over as
        // lists, so there must not be too many (nothing retained at all also takes the other route).
        const bool sparse = out.mode == FSEL_ALL || (out.mode == FSEL_THRESHOLD && !used_fallback && k <= STEP_MAX_EVICT);
        const int32_t ctot = step_ctot;
        uint32_t* chunk_ev = ws.step_chunk_ev + step_chunks_before;   // this sequence's chunks
        if (sparse) {
            // What the row mover gets: per chunk the number of entries it loses (a byte; almost all 0), per segment a
            // record - where its survivors start in the destination, and the indices of its evicted entries.  From
            // these a block of the row mover places its chunk itself: survivors of chunk ch of segment g start at
            // dst_start[g] + 128 ch - (evicted entries of g before the chunk).
            // (The zeros of the per-chunk counts were acknowledged before a barrier of the ranking; FSEL_ALL adds none.)
            bool ev[FAST_ITEMS];
            int ev_slot[FAST_ITEMS];
#pragma unroll
            for (int u = 0; u < FAST_ITEMS; ++u) {
                ev[u] = out.mode == FSEL_THRESHOLD && listed[u] && evicted_before(key[u], sg[u], ps[u], out.key_thr, out.seg_thr, out.pos_thr);
                ev_slot[u] = 0;
                if (ev[u]) {
                    const int sl = sg[u] - g0;
                    ev_slot[u] = atomicAdd(&s_ev[sl], 1);
                    atomicAdd(&ws.step_chunk_ev[s_chb[sl] + ix[u] / CMP_CHUNK], 1u);
                }
            }
            __syncthreads();
            const int my_ev = tid < nsg ? s_ev[tid] : 0;
            // evicted entries (at most STEP_MAX_EVICT) and destination entries of the segments before, in one scan
            uint64_t tot;
            const uint64_t ex = block_excl_scan<uint64_t, true>(tid < nsg ? (uint64_t)((int64_t)(my_len - my_ev) + sa.reserve) << 16 | (uint64_t)my_ev : 0,
                                                                reinterpret_cast<uint64_t*>(sm.lds64), &tot);
            const int32_t eex = (int32_t)(ex & 0xFFFFu);
            const int64_t nex = (int64_t)(ex >> 16);
            if (tid < nsg) {
                const int g = g0 + tid;
                s_off[tid] = eex;
                kept_out[g] = my_len - my_ev;
                StepSegRec* rec = ws.step_rec + g;
                if (sa.inplace) {                                 // the segment keeps its start; the row mover commits the new length
                    rec->dst_start = (int64_t)my_start;
                    ws.step_len[g] = my_len - my_ev;
                } else {
                    sa.dst.seg_start[g] = step_before + nex;
                    sa.dst.seg_len[g] = my_len - my_ev;
                    rec->dst_start = step_before + nex;
                }
                rec->cnt = my_ev;
                rec->off = eex;
            }
            __syncthreads();
            int32_t* evl = ws.step_evl + (size_t)seq * STEP_MAX_EVICT;
#pragma unroll
            for (int u = 0; u < FAST_ITEMS; ++u) {
                if (ev[u]) {
                    const int sl = sg[u] - g0;
                    evl[s_off[sl] + ev_slot[u]] = ix[u];
                    if (ev_slot[u] < STEP_REC_IDX) ws.step_rec[g0 + sl].idx[ev_slot[u]] = ix[u];
                }
            }
        } else {
            // after the single-block select (or with very many evictions) the evicted entries are not listed: one more
            // pass over the sequence leaves the keep mask and, per chunk of 128 entries, where its survivors go
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (the zeros written earlier have landed)
            __syncthreads();
            for (int i = tid; i < ctot; i += FAST_THREADS) st_dev(&chunk_ev[i], STEP_CHUNK_DENSE);   // "look at the mask and the table"
            int64_t cursor = step_before;
            int cb = step_chunks_before;
            const int lane = lane_id(), wave = tid >> 6;
            for (int g = g0; g < g0 + nsg; ++g) {
                bool b2 = false, n2 = false;
                const SegView v = seg_view<KIND>(c, g, sh.nseg, sa, &b2, &n2);
                if (sa.inplace) cursor = v.start;                 // the segment keeps its start
                int64_t running = 0;
                for (int t0 = 0; t0 < v.len; t0 += FAST_THREADS) {   // tiles of 8 chunks
                    const int j = t0 + tid;
                    bool kf = false;
                    if (j < v.len) {
                        if (out.mode == FSEL_THRESHOLD) {
                            int pj;
                            float sj;
                            ks.entry_at(g, v, j, &pj, &sj);
                            const uint32_t kk = key_of_score(sj);
                            kf = !evicted_before(kk, g, pj, out.key_thr, out.seg_thr, out.pos_thr);
                        } else {
                            kf = out.mode == FSEL_ALL;
                        }
                        sa.keep_out[v.start + j] = kf;
                    }
                    const int wc = __popcll(__ballot(kf));
                    __syncthreads();
                    if (lane == 0) sm.h[wave] = wc;               // 16 wavefronts = 8 chunks of two
                    __syncthreads();
                    if (tid < FAST_THREADS / CMP_CHUNK) {
                        const int chl = t0 / CMP_CHUNK + tid;     // chunk of the segment
                        if (chl * CMP_CHUNK < v.len) {
                            int64_t ex = 0;
                            for (int i = 0; i < tid; ++i) ex += sm.h[2 * i] + sm.h[2 * i + 1];
                            const int here = sm.h[2 * tid] + sm.h[2 * tid + 1];
                            const int n = min(CMP_CHUNK, v.len - chl * CMP_CHUNK);
                            ws.cmp_chunk_dst[cb + chl] = (cursor + running + ex) | (here == n ? CMP_DST_FULL : 0);
                        }
                    }
                    int tile = 0;
                    for (int i = 0; i < FAST_THREADS / 64; ++i) tile += sm.h[i];
                    running += tile;
                }
                if (tid == 0) {
                    kept_out[g] = (int32_t)running;
                    if (sa.inplace) {
                        ws.step_len[g] = (int32_t)running;
                    } else {
                        sa.dst.seg_start[g] = cursor;
                        sa.dst.seg_len[g] = (int32_t)running;
                    }
                }
                cursor += running + sa.reserve;
                cb += (v.len + CMP_CHUNK - 1) / CMP_CHUNK;
            }
        }
    }
}

// keep[e] from the published triple; survivors per segment are added to kept_out (zeroed by k_fast_scan).
template <bool MULTI>
__global__ __launch_bounds__(FAST_THREADS) void k_fast_mask(CacheView c, const float* __restrict__ score, Shape sh,
                                                            Workspace ws, int bps, int spb_arg, int limit, uint8_t* __restrict__ keep,
                                                            int32_t* __restrict__ kept_out) {
    __shared__ int32_t lds32[17];
    // dealt as in k_fast_scan
    const int spb = MULTI ? spb_arg : 1, threads = FAST_THREADS / spb;
    const int tid = (int)threadIdx.x % threads;
    int seg, part;
    bool no_seg = false;
    const int bpq = (sh.segs_per_seq + spb - 1) / spb * bps;
    if (MULTI) {                                                  // (bps = 1)
        const int seg_in_seq = (int)threadIdx.x / threads * bpq + (int)blockIdx.x % bpq;
        no_seg = seg_in_seq >= sh.segs_per_seq;
        seg = (int)blockIdx.x / bpq * sh.segs_per_seq + min(seg_in_seq, sh.segs_per_seq - 1);
        part = 0;
    } else {
        seg = (int)blockIdx.x / bps;
        part = (int)blockIdx.x % bps;
    }
    const int seq = seg / sh.segs_per_seq;
    int stride = bps * threads;
    const StepArgs sa{};
    bool bad = false, nocap = false;
    SegView v = seg_view<SCAN_RAGGED>(c, seg, sh.nseg, sa, &bad, &nocap);
    int len = no_seg ? 0 : v.len;
    const FastSel fs = ws.fast_sel[seq];
    int n = 0, first = part * threads + tid;
    if (MULTI) len = min(len, limit);
    uint32_t todo = MULTI ? long_segments<SCAN_RAGGED>(c, sa, sh, seq, bpq, (int)blockIdx.x % bpq, spb, limit) : 0;
    for (;;) {                                                    // as in k_fast_scan
    const bool seg_before = seg < fs.seg_thr, seg_same = seg == fs.seg_thr;
    for (int j0 = first; j0 < len; j0 += stride * FAST_BATCH) {
        float sv[FAST_BATCH];
#pragma unroll
        for (int u = 0; u < FAST_BATCH; ++u) {
            const int j = j0 + u * stride;
            sv[u] = (j < len && fs.mode == FSEL_THRESHOLD) ? score[v.start + j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < FAST_BATCH; ++u) {
            const int j = j0 + u * stride;
            if (j >= len) continue;
            bool kf = fs.mode == FSEL_ALL;
            if (fs.mode == FSEL_THRESHOLD) {
                const uint32_t key = key_of_score(sv[u]);
                kf = key > fs.key_thr;
                if (key == fs.key_thr) kf = seg_before || (seg_same && c.pos[v.start + j] <= fs.pos_thr);
            }
            keep[v.start + j] = kf;
            n += kf;
        }
    }
    if (!MULTI) {
        n = block_sum<int32_t>(n, lds32);
        if (tid == 0 && n) atomicAdd(&kept_out[seg], n);
    } else {                                                      // (a wavefront's threads share a segment)
        n = wave_sum(n);
        if (lane_id() == 0 && n) atomicAdd(&kept_out[seg], n);
    }
    if (!MULTI || todo == 0) break;
    seg = seq * sh.segs_per_seq + __builtin_ctz(todo) * bpq + (int)blockIdx.x % bpq;
    todo &= todo - 1;
    v = seg_view<SCAN_RAGGED>(c, seg, sh.nseg, sa, &bad, &nocap);
    first = limit + (int)threadIdx.x;
    stride = FAST_THREADS;
    len = v.len;
    n = 0;
    }
}

// How the blocks of k_fast_scan and k_fast_mask are dealt: several to a segment of more than FAST_ENTRIES_PER_BLOCK
// entries; several segments of a sequence to a block when a block each would be more than are resident at once (one of
// k_fast_scan's per compute unit, two of k_fast_mask's) - a block of k_fast_scan lives 8 to 10 us whatever it has to do, so
// 4096 segments of 2048 entries took sixteen rounds of the chip: 202 us, with sixteen segments to a block 43.
// Of a long segment its own threads walk twice the mean capacity of a segment, and two batches at least; a whole number of
// pages, so that a wavefront's entries stay in one.
struct ScanGrid {
    int deal, bps, spb, limit;
    unsigned blocks, parts = 1;
};
// A whole sequence to a block, which then neither lists its candidates in memory nor meets other blocks: up to a batch of
// FAST_BATCH entries for every lane of its wavefronts.  One-call steps in us, against a block per segment or several
// segments to a block: 16 lists of 65 entries 24.2 / 26.6, 64 of 101 27.2 / 29.2, 4 of 1901 25.9 / 29.4, eight sequences
// of 16 lists of 501 38.5 / 40.9; but with two batches the walk has no other blocks to hide behind: 2 x 18 lists of 1152
// 38.3 / 34.9, 88 lists of 297 35.2 / 28.8.  That is a mean: nothing says that a batch's sequences are alike, the longest may be
// all of it.  Beyond two batches in all the grid therefore has more blocks for each sequence, as many as the longest could
// use and a compute unit each has (for more than 128 sequences none: those are better off with a block each whatever their
// lengths, 200 sequences of 288 entries, nine tenths of all in one 75.5 / 100.6).  Lists of 500 for four sequences, alike / one
// with nine tenths / with half: 27.7, 29.0, 29.8 us, dealt by segments 31.0, 30.8, 31.0, a block for each whatever its length 27.4,
// 36.1, 30.6; for eight 31.9, 33.6, 34.6 (34.5, 34.9, 34.4; 31.5, 52.9, 34.5); 64 sequences of 16 lists of 60, four blocks for each at most,
// 34.6, 44.9, 34.8 (40.2, 42.7, 40.8; 34.0, 57.0, 34.1).  The separate instance, because what a sequence of
// one block never needs costs it 0.5 us all the same.
constexpr int64_t WHOLE_CAP = 8 * WHOLE_ENTRIES;
static int whole_parts(const Shape& sh, int64_t cap, int resident, int64_t max_pps) {   // blocks for a sequence; 0: dealt in another way
    if (sh.segs_per_seq > STEP_MAX_SEGS || sh.n_seq > STEP_MAX_SEQS || cap / sh.n_seq > WHOLE_ENTRIES || cap > WHOLE_CAP) return 0;
    if (sh.segs_per_seq * max_pps >= 1 << 24) return 0;           // (a sequence's slots are counted in 32 bits)
    const int64_t most = (cap + WHOLE_ENTRIES - 1) / WHOLE_ENTRIES, room = resident / sh.n_seq;
    return cap <= 2 * WHOLE_ENTRIES || room < 2 ? 1 : (int)(most < room ? most : room);
}
static ScanGrid scan_grid(const Shape& sh, int64_t cap, int resident, bool whole, int64_t max_pps = 0) {
    ScanGrid g;
    if (const int parts = whole ? whole_parts(sh, cap, resident, max_pps) : 0) return ScanGrid{parts > 1 ? DEAL_PARTS : DEAL_WHOLE, parts, 1, 0, (unsigned)sh.n_seq, (unsigned)parts};
    const int64_t bps = cap / ((int64_t)sh.nseg * FAST_ENTRIES_PER_BLOCK);
    g.bps = (int)(bps < 1 ? 1 : (bps > 64 ? 64 : bps));
    g.spb = 1;
    auto per_seq = [&](int spb) { return (int64_t)((sh.segs_per_seq + spb - 1) / spb); };
    while (bps < 1 && g.spb < FAST_THREADS / 64 && sh.n_seq * per_seq(g.spb) > resident && 2 * g.spb <= sh.segs_per_seq) g.spb *= 2;
    g.blocks = (unsigned)(sh.n_seq * per_seq(g.spb) * g.bps);
    g.deal = g.spb > 1 ? DEAL_MULTI : DEAL_SEGMENT;
    // (several to a block: a mean below FAST_ENTRIES_PER_BLOCK, so the limit is below 2^15)
    const int64_t mean2 = 2 * (cap / sh.nseg), batches = 2 * (FAST_THREADS / g.spb) * FAST_BATCH;
    g.limit = g.spb == 1 ? 0 : (int)(((mean2 > batches ? mean2 : batches) + KVTRIM_PAGE_SIZE - 1) / KVTRIM_PAGE_SIZE * KVTRIM_PAGE_SIZE);
    return g;
}
constexpr int SCAN_RESIDENT = 256, MASK_RESIDENT = 512;

template <int KIND>
static void launch_scan(const ScanGrid& g, const CacheView& c, const int32_t* now, float* score, const int64_t* budget, const Shape& sh,
                        const Workspace& ws, int32_t* kept, uint32_t* thr, const StepArgs& sa, unsigned more_blocks, hipStream_t st) {
#define KVTRIM_DEAL(d) hipLaunchKernelGGL((k_fast_scan<KIND, d>), dim3(g.blocks + more_blocks, g.parts), dim3(FAST_THREADS), 0, st, c, now, score, budget, sh, ws, g.bps, g.spb, g.limit, kept, thr, sa)
    if (g.deal == DEAL_WHOLE) KVTRIM_DEAL(DEAL_WHOLE);
    else if (g.deal == DEAL_PARTS) KVTRIM_DEAL(DEAL_PARTS);
    else if (g.deal == DEAL_MULTI) KVTRIM_DEAL(DEAL_MULTI);
    else KVTRIM_DEAL(DEAL_SEGMENT);
#undef KVTRIM_DEAL
}

kvtrim_status launch_score_select(kvtrim_ctx* ctx, const CacheView& c, const int32_t* now, const int64_t* budget,
                                  float* score, uint8_t* keep, int32_t* kept, uint32_t* thr, int64_t evict_hint,
                                  hipStream_t st) {
    const Shape& sh = ctx->shape;
    const Workspace& ws = ctx->ws;
    // the list has to hold about 3 (k + 1) entries for k evictions, spread unevenly over its sub-lists
    if (evict_hint <= 0 || 8 * (evict_hint + 1) > (int64_t)ws.fl_cap)
        return launch_score_select_general(ctx, c, now, budget, score, keep, kept, thr, st);
    const dim3 block(FAST_THREADS);
    const ScanGrid sg = scan_grid(sh, c.cap, SCAN_RESIDENT, true);
    { ProfScope prof(ctx, K_FAST_SCAN, st);
      launch_scan<SCAN_RAGGED>(sg, c, now, score, budget, sh, ws, kept, thr, StepArgs(), 0, st); }
    { ProfScope prof(ctx, K_FAST_MASK, st);
      const ScanGrid mg = scan_grid(sh, c.cap, MASK_RESIDENT, false);
      if (mg.spb > 1) hipLaunchKernelGGL(k_fast_mask<true>, dim3(mg.blocks), block, 0, st, c, (const float*)score, sh, ws, mg.bps, mg.spb, mg.limit, keep, kept);
      else hipLaunchKernelGGL(k_fast_mask<false>, dim3(mg.blocks), block, 0, st, c, (const float*)score, sh, ws, mg.bps, mg.spb, mg.limit, keep, kept); }
    KVTRIM_HIP(ctx, hipGetLastError());
    return KVTRIM_OK;
}

// The decode-step form over a paged cache (`pool`: the page pool's arrays, cap = its slots) in one kernel, walking every segment's
// slots through its block table.  The caller has checked that the hint fits the list.
kvtrim_status launch_score_select_paged(kvtrim_ctx* ctx, const CacheView& pool, const PagedArgs& pg, const int32_t* now,
                                        const int64_t* budget, float* score, uint8_t* keep, int32_t* kept, uint32_t* thr,
                                        hipStream_t st) {
    const ScanGrid sg = scan_grid(ctx->shape, pool.cap, SCAN_RESIDENT, true, pg.max_pps);
    StepArgs sa{};
    sa.pg = pg;
    sa.keep_out = keep;
    ProfScope prof(ctx, K_FAST_SCAN, st);
    launch_scan<SCAN_PAGED>(sg, pool, now, score, budget, ctx->shape, ctx->ws, kept, thr, sa, 0, st);
    KVTRIM_HIP(ctx, hipGetLastError());
    return KVTRIM_OK;
}

// The scoring kernel of the one-call decode step (the caller has checked that the step fits its limits).
kvtrim_status launch_step_scan(kvtrim_ctx* ctx, const CacheView& c, const int32_t* now, const int64_t* budget, float* score,
                               int32_t* kept, uint32_t* thr, const StepArgs& sa, hipStream_t st) {
    const Shape& sh = ctx->shape;
    const ScanGrid sg = scan_grid(sh, c.cap, SCAN_RESIDENT, true);
    const unsigned tables = (unsigned)((sh.nseg + FAST_THREADS / 64 - 1) / (FAST_THREADS / 64));
    ProfScope prof(ctx, K_FAST_SCAN, st);
    launch_scan<SCAN_STEP>(sg, c, now, score, budget, sh, ctx->ws, kept, thr, sa, tables, st);
    KVTRIM_HIP(ctx, hipGetLastError());
    return KVTRIM_OK;
}

}  // namespace kvtrim
