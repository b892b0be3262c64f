// Stage 3: stable stream compaction of the retained entries into a tight ragged cache.
//
// k_cmp_scan  one block per segment: counts the mask per 128-entry chunk, scans the counts inside
//             the segment and derives the destination segment table from `kept`.
// k_cmp_copy  one block of 8 wavefronts per chunk: a ballot/prefix over the chunk's mask
//             ranks the survivors; every wavefront then moves at most 16 rows in ONE batch of
//             loads followed by one batch of stores (16 bytes per lane, whole rows per 16
//             lanes, non-temporal) and ends.  Short-lived wavefronts measured ~10 % faster on
//             this chip than wavefronts that loop over several batches.
#include "kvtrim_device.h"

#include <type_traits>

namespace kvtrim {

constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_LANE = 16;          // mask bytes per lane and load: a wavefront's load covers 8 chunks
constexpr int SCAN_GROUP = 64 * SCAN_LANE / CMP_CHUNK;
constexpr int SCAN_BATCH = 64 / SCAN_GROUP;   // loads with which a block's wavefronts cover a tile of as many chunks as it has threads: 8
static_assert(SCAN_LANE * 8 == CMP_CHUNK, "eight lanes to a chunk");

// bit i set where byte i of the 16 is not zero
typedef uint32_t scan_v4 __attribute__((ext_vector_type(4), aligned(1)));   // (16 bytes at any address)
__device__ __forceinline__ uint32_t nonzero_bytes(const scan_v4& w) {
    auto four = [](uint32_t x) {
        const uint32_t t = ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) >> 7) & 0x01010101u;
        return (t * 0x01020408u) >> 24 & 15u;
    };
    return four(w.x) | four(w.y) << 4 | four(w.z) << 8 | four(w.w) << 12;
}

// Sums four values over the block (1024 threads) with one barrier; every thread gets every sum.  Each step of the first
// two halves what a lane still has to add up, so that a wavefront takes 7 shuffles instead of 24, and the 16 wavefronts'
// sums are added by shuffles as well: with eight values one after the other and every thread reading 128 sums from LDS
// this was most of k_cmp_scan at a thousand segments (1024 segments of 12 K entries: 51 us, now 29.5).
__device__ __forceinline__ void block_sum_4(int64_t (&v)[4], int64_t* lds /* [64] */) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const bool up = lane & 32, odd = lane & 16;
    int64_t a = (up ? v[2] : v[0]) + __shfl_xor(up ? v[0] : v[2], 32, 64);
    const int64_t b = (up ? v[3] : v[1]) + __shfl_xor(up ? v[1] : v[3], 32, 64);
    a = (odd ? b : a) + __shfl_xor(odd ? a : b, 16, 64);          // lanes 16 k .. 16 k + 15 hold value k
#pragma unroll
    for (int s = 8; s >= 1; s >>= 1) a += __shfl_xor(a, s, 64);
    if ((lane & 15) == 0) lds[wave * 4 + (lane >> 4)] = a;
    __syncthreads();
    a = lds[lane];                                                // value lane % 4 of wavefront lane / 4
#pragma unroll
    for (int s = 32; s >= 4; s >>= 1) a += __shfl_xor(a, s, 64);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __shfl(a, k, 64);
}

// With many segments the per-block reduction over all segments below costs more than a launch: one block
// then scans the segments once and leaves, per segment, the first chunk (ws.cmp_chunk_prefix) and the first
// destination entry (dst.seg_start) - the two values k_cmp_scan would otherwise derive in every block.
// inplace: the survivors stay in their segment's own region (dst is the same cache): the segment starts stand as
// they are and there is no capacity to check.
__global__ __launch_bounds__(SCAN_THREADS) void k_cmp_prefix(CacheView src, const int32_t* __restrict__ kept,
                                                             CacheViewMut dst, int reserve, int align, Shape sh,
                                                             Workspace ws, int inplace, int gat) {
    __shared__ int64_t lds64[17];
    __shared__ int s_bad_layout, s_bad_kept;
    const int tid = threadIdx.x, nseg = sh.nseg;
    if (tid == 0) s_bad_layout = s_bad_kept = 0;
    __syncthreads();
    int64_t chunks = 0, entries = 0, runs = 0;
    for (int base = 0; base < nseg; base += SCAN_THREADS) {
        const int i = base + tid;
        int64_t nch = 0, need = 0, nrun = 0;
        if (i < nseg) {
            const int len = src.seg_len[i];
            const int64_t st = src.seg_start[i];
            const int kp = kept[i];
            const int64_t nxt = i + 1 < nseg ? src.seg_start[i + 1] : src.cap;
            if (len < 0 || st < 0 || st + len > src.cap || st + len > nxt) s_bad_layout = 1;
            if (kp < 0 || kp > len) s_bad_kept = 1;
            nch = len > 0 ? ((int64_t)len + CMP_CHUNK - 1) / CMP_CHUNK : 0;
            need = ((int64_t)kp + reserve + align - 1) / align * align;
            nrun = gat && len > 0 ? ((int64_t)kp + CMP_CHUNK - 1) / CMP_CHUNK : 0;
        }
        int64_t tot_c, tot_e;
        const int64_t ex_c = block_excl_scan<int64_t>(nch, lds64, &tot_c);
        const int64_t ex_e = block_excl_scan<int64_t>(need, lds64, &tot_e);
        if (i < nseg) {
            ws.cmp_chunk_prefix[i] = (int32_t)min(chunks + ex_c, (int64_t)0x7fffffff);
            // (parked in the workspace: the destination is written only once the capacity check below has passed)
            if (!inplace) ws.pg_seg_start[i] = entries + ex_e;
        }
        chunks += tot_c;
        entries += tot_e;
        if (gat) {                                                // uniform over the block
            int64_t tot_r;
            const int64_t ex_r = block_excl_scan<int64_t>(nrun, lds64, &tot_r);
            if (i < nseg) ws.att_chunk_prefix[i] = (int32_t)min(runs + ex_r, (int64_t)0x7fffffff);
            runs += tot_r;
        }
    }
    __syncthreads();
    const bool bad_layout = s_bad_layout || chunks > ws.max_cmp_chunks || runs > ws.max_att_chunks, bad_kept = s_bad_kept != 0;
    if (tid == 0) {
        if (bad_layout || bad_kept || (!inplace && entries > dst.cap)) {
            atomicOr(ws.err, bad_layout ? ERR_LAYOUT : (bad_kept ? ERR_MISMATCH : ERR_CAP));
            ws.cmp_chunk_prefix[nseg] = 0;
            if (gat) ws.att_chunk_prefix[nseg] = 0;
        } else {
            ws.cmp_chunk_prefix[nseg] = (int32_t)chunks;
            if (gat) ws.att_chunk_prefix[nseg] = (int32_t)runs;
        }
    }
    if (!inplace && !(bad_layout || bad_kept || entries > dst.cap)) {
        __syncthreads();                                          // the parked starts are this block's own writes
        for (int i = tid; i < nseg; i += SCAN_THREADS) dst.seg_start[i] = ws.pg_seg_start[i];
    }
}

// Behind k_cmp_prefix (more than 1024 segments) a block of 256 threads takes a segment: the kernel needs some 80 registers,
// with which a compute unit holds one block of 1024 threads but five of 256.
constexpr int PRE_THREADS = 256;

// PRE: k_cmp_prefix has run (segment prefixes and the checks over all segments are done).
// gat: the table of the DESTINATION's 128-row chunks (ws.att_chunk_prefix / ws.att_desc) and the source row of every
// destination row (ws.gat_src) are written as well, for the gathering instance of the fused kernel that follows.
template <bool PRE, int THREADS>
__global__ __launch_bounds__(THREADS) void k_cmp_scan(CacheView src, const uint8_t* __restrict__ keep,
                                                           const int32_t* __restrict__ kept, CacheViewMut dst,
                                                           int reserve, int align, Shape sh, Workspace ws, int inplace,
                                                           int gat) {
    static_assert(PRE || THREADS == SCAN_THREADS, "a thread per segment sums the prefixes");
    __shared__ int64_t lds64[17];
    __shared__ int64_t lds_n[64];
    __shared__ int s_bad;                                         // 1: a segment table entry, 2: a count that no mask can have
    __shared__ int s_cnt[THREADS];
    __shared__ int s_ex[THREADS];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int g = blockIdx.x;
    const int nseg = sh.nseg;
    if (!PRE) {
        if (tid == 0) s_bad = 0;
        __syncthreads();
    }

    // Order of the memory traffic: (1) this segment's own table entry; (2) in one round, the table entries of all
    // segments (for the prefixes; !PRE) and the mask bytes of this segment's first THREADS chunks; then
    // arithmetic only; (3) the stores.  A decode-step segment is done after two dependent round trips.
    const int len_raw = src.seg_len[g];
    const int64_t start = src.seg_start[g];
    const bool own_ok = len_raw >= 0 && start >= 0 && start + len_raw <= src.cap;   // (checked for all segments below / by k_cmp_prefix)
    const int len = own_ok ? len_raw : 0;
    const int nch = len > 0 ? (len + CMP_CHUNK - 1) / CMP_CHUNK : 0;
    const uint8_t* kp = keep + start;

    int64_t chunks_before, dst_before, runs_before = 0;
    int o_len = 0, o_kp = 0;                                      // !PRE: table entry of segment `tid`
    int64_t o_st = 0;
    if (PRE) {
        // One decision for the whole block: another block of this launch may raise the flag (a mask that disagrees
        // with `kept`) between the reads of two wavefronts, and a block that lost some of its wavefronts would scan
        // counts that were never written.
        __shared__ int s_err;
        if (tid == 0) s_err = __hip_atomic_load(ws.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_err != 0) return;
        chunks_before = ws.cmp_chunk_prefix[g];
        dst_before = dst.seg_start[g];
        if (gat) runs_before = ws.att_chunk_prefix[g];
    } else if (tid < nseg) {                                      // (nseg <= THREADS without k_cmp_prefix)
        o_len = src.seg_len[tid];
        o_st = src.seg_start[tid];
        o_kp = kept[tid];
    }

    // Mask bytes of one tile of THREADS chunks: load u of a wavefront covers the 8 chunks from (16 u + wave) * 8 on, 16
    // bytes per lane (at any address: a segment starts anywhere), all of them asked for at once.  They stay in registers
    // as one bit per entry, for the counts and (gat) for the row numbers.  (A wavefront per chunk with two byte loads per
    // lane, twice over for the row numbers, took 46 us for the 33.5 M entries of a first eviction; now 18.)
    // A lane whose 16 bytes reach past the segment's end reads the segment's last 16 and shifts them into place.
    // In two halves, the first of which - 512 chunks - is under way while the prefixes are summed.
    scan_v4 w[SCAN_BATCH / 2];
    uint32_t bits[SCAN_BATCH];
    // (below 2^31: a tile starts at a multiple of THREADS chunks inside a segment of at most 2^31 - 4096 entries)
    auto first_of = [&](int tile0, int u) { return (tile0 + (u * (THREADS / 64) + wave) * SCAN_GROUP) * CMP_CHUNK; };
    auto request = [&](int tile0, int half) {
#pragma unroll
        for (int u = 0; u < SCAN_BATCH / 2; ++u) {
            const int64_t j0 = first_of(tile0, half * (SCAN_BATCH / 2) + u);
            w[u] = scan_v4{0, 0, 0, 0};
            if (j0 < len) {                                       // (uniform)
                if (len >= SCAN_LANE) {
                    w[u] = *reinterpret_cast<const scan_v4*>(kp + min(j0 + lane * SCAN_LANE, (int64_t)len - SCAN_LANE));
                } else if (lane == 0) {
                    uint64_t lo = 0, hi = 0;
                    for (int i = 0; i < len; ++i) (i < 8 ? lo : hi) |= (uint64_t)kp[i] << (8 * (i & 7));
                    w[u] = scan_v4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
                }
            }
        }
    };
    auto count = [&](int tile0, auto half) {                      // survivors per chunk of half a tile into s_cnt
#pragma unroll
        for (int i = 0; i < SCAN_BATCH / 2; ++i) {
            constexpr int first = decltype(half)::value * (SCAN_BATCH / 2);
            const int u = first + i;
            if (first_of(tile0, u) >= len) {                      // (uniform; nothing there, and nobody reads the counts)
                bits[u] = 0;
                continue;
            }
            const int64_t over = (int64_t)first_of(tile0, u) + lane * SCAN_LANE - ((int64_t)len - SCAN_LANE);   // bytes past the end
            bits[u] = nonzero_bytes(w[i]);
            if (over > 0 && len >= SCAN_LANE) bits[u] = over < SCAN_LANE ? bits[u] >> over : 0u;
            int n = __popc(bits[u]);
            n += __shfl_xor(n, 1, 64);
            n += __shfl_xor(n, 2, 64);
            n += __shfl_xor(n, 4, 64);
            if ((lane & 7) == 0) s_cnt[(u * (THREADS / 64) + wave) * SCAN_GROUP + (lane >> 3)] = n;
        }
    };
    request(0, 0);                                                // in flight while the prefixes are summed

    if (!PRE) {
        // chunks and destination entries of the segments before g, and the totals
        int64_t acc[4] = {0, 0, 0, 0};   // chunks (before g in the low, all in the high half), destination chunks (alike), dst entries before g, all
        bool bl = false, bk = false;
        if (tid < nseg) {
            const int i = tid;
            const int64_t o_nxt = i + 1 < nseg ? src.seg_start[i + 1] : src.cap;
            bl = o_len < 0 || o_st < 0 || o_st + o_len > src.cap || o_st + o_len > o_nxt;
            bk = o_kp < 0 || o_kp > o_len;
            // (both below 2^24 for a segment that is inside the buffers; the sums count only if none is bad)
            const int64_t nc = o_len > 0 && !bl ? ((int64_t)o_len + CMP_CHUNK - 1) / CMP_CHUNK : 0;
            const int64_t nrun = gat && o_len > 0 && !bl && !bk ? ((int64_t)o_kp + CMP_CHUNK - 1) / CMP_CHUNK : 0;
            const int64_t need = ((int64_t)o_kp + reserve + align - 1) / align * align;   // align = 1 unless pages are built
            acc[0] = nc << 32 | (i < g ? nc : 0);
            acc[1] = nrun << 32 | (i < g ? nrun : 0);
            acc[2] = i < g ? need : 0;
            acc[3] = need;
        }
        if (bl || bk) atomicOr(&s_bad, bl ? 1 : 2);
        block_sum_4(acc, lds_n);
        chunks_before = acc[0] & 0xffffffff;
        dst_before = acc[2];
        runs_before = acc[1] & 0xffffffff;
        const int64_t dst_total = acc[3], chunks_total = acc[0] >> 32;
        const bool bad_layout = (s_bad & 1) || chunks_total > ws.max_cmp_chunks || (acc[1] >> 32) > ws.max_att_chunks, bad_kept = s_bad & 2;
        if (inplace) dst_before = start;                          // the segment keeps its place
        if (bad_layout || bad_kept || (!inplace && dst_total > dst.cap)) {   // every block takes the same decision
            if (tid == 0) {
                atomicOr(ws.err, bad_layout ? ERR_LAYOUT : (bad_kept ? ERR_MISMATCH : ERR_CAP));
                if (g == 0) {
                    ws.cmp_chunk_prefix[nseg] = 0;
                    if (gat) ws.att_chunk_prefix[nseg] = 0;
                }
            }
            return;
        }
    }

    const int cbase = (int)chunks_before;
    int64_t gat_slots = 0;                                        // gat: slots of this segment in ws.gat_src
    if (gat) {                                                    // the chunks of the DESTINATION segment, for the gathering fused kernel
        const int rlen = own_ok ? kept[g] : 0;
        const int nrun = len > 0 && rlen > 0 ? (rlen + CMP_CHUNK - 1) / CMP_CHUNK : 0;
        gat_slots = (int64_t)nrun * CMP_CHUNK;
        for (int u = tid; u < nrun; u += THREADS) {
            ChunkDesc d;
            d.first = dst_before + (int64_t)u * CMP_CHUNK;
            d.n = min(CMP_CHUNK, rlen - u * CMP_CHUNK);
            d.seg = g;
            ws.att_desc[runs_before + u] = d;
        }
        if (tid == 0 && !PRE) {
            ws.att_chunk_prefix[g] = (int32_t)runs_before;
            if (g == nseg - 1) ws.att_chunk_prefix[nseg] = (int32_t)(runs_before + nrun);
        }
    }

    // Tiles of THREADS chunks: counts (phase 1, above), then a thread per chunk - exclusive scan of the counts,
    // destination offset and descriptor of every chunk (phase 2).
    int64_t running = 0;
    for (int tile0 = 0; tile0 < nch; tile0 += THREADS) {
        const int tile_n = min(THREADS, nch - tile0);
        __syncthreads();                                          // s_cnt of the previous tile has been read
        if (tile0 > 0) request(tile0, 0);                         // (the first one is already here)
        count(tile0, std::integral_constant<int, 0>());
        request(tile0, 1);
        count(tile0, std::integral_constant<int, 1>());
        __syncthreads();
        const int ch = tile0 + tid;
        const int64_t v = tid < tile_n ? s_cnt[tid] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan<int64_t>(v, lds64, &tot);
        if (tid < tile_n) {
            const int n = min(CMP_CHUNK, len - ch * CMP_CHUNK);
            // a chunk that loses nothing is marked: its mover needs neither the mask nor the ranks
            ws.cmp_chunk_dst[cbase + ch] = (dst_before + running + ex) | (v == n ? CMP_DST_FULL : 0);
            ChunkDesc d;
            d.first = start + (int64_t)ch * CMP_CHUNK;
            d.n = n;
            d.seg = g;
            ws.cmp_desc[cbase + ch] = d;
        }
        if (gat) {
            // the source row of every destination row, in slots of CMP_CHUNK per destination chunk (the segment's
            // chunks are consecutive, so row r of the segment has slot runs_before * CMP_CHUNK + r)
            s_ex[tid] = (int)(running + ex);
            __syncthreads();
            int32_t* slots = ws.gat_src + runs_before * CMP_CHUNK;
#pragma unroll
            for (int u = 0; u < SCAN_BATCH; ++u) {
                const int cl = (u * (THREADS / 64) + wave) * SCAN_GROUP + (lane >> 3);
                const int n = __popc(bits[u]);
                int before = n;                                   // survivors of the chunk up to this lane's, then before them
                int o = __shfl_up(before, 1, 8);
                if ((lane & 7) >= 1) before += o;
                o = __shfl_up(before, 2, 8);
                if ((lane & 7) >= 2) before += o;
                o = __shfl_up(before, 4, 8);
                if ((lane & 7) >= 4) before += o;
                int64_t r = (int64_t)s_ex[cl] + before - n;
                const int32_t row = (int32_t)(start + ((int64_t)tile0 + cl) * CMP_CHUNK + (lane & 7) * SCAN_LANE);
                // (a mask with more survivors than `kept` says - reported below - must not leave the segment's slots)
                for (uint32_t m = bits[u]; m; m &= m - 1, ++r)
                    if (r >= 0 && r < gat_slots) slots[r] = row + __builtin_ctz(m);
            }
        }
        running += tot;
    }
    if (gat) {
        // the slots behind the segment's last row, up to the end of its last chunk, name a row that exists
        for (int64_t r = running + tid; r < gat_slots; r += THREADS) ws.gat_src[runs_before * CMP_CHUNK + r] = (int32_t)start;
    }
    if (tid == 0) {
        if (running != kept[g]) atomicOr(ws.err, ERR_MISMATCH);
        if (!inplace) {                                           // (in place the other blocks are still reading the lengths:
            dst.seg_start[g] = dst_before;                        //  the mover's last kernel commits them)
            dst.seg_len[g] = kept[g];
        }
        if (!PRE) {
            ws.cmp_chunk_prefix[g] = cbase;
            if (g == nseg - 1) ws.cmp_chunk_prefix[nseg] = cbase + nch;
        }
    }
}

typedef unsigned v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 ld16_nt(const uint4* p) {
    v4u t = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void st16_nt(uint4* p, uint4 v) {
    v4u t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<v4u*>(p));
}

// NEW: the K/V rows of a segment's entries from old_len[seg] on are not in src but in k_new / v_new
// ([nseg][n_new][D], entry old_len + i of segment g = row g * n_new + i): a chunk of tokens whose metadata has
// been appended to src goes from the caller's buffers straight to its place in dst.
template <int D, bool NEW>
__global__ __launch_bounds__(CMP_THREADS) void k_cmp_copy(CacheView src, const uint8_t* __restrict__ keep,
                                                          CacheViewMut dst, Shape sh, Workspace ws,
                                                          const uint16_t* __restrict__ k_new,
                                                          const uint16_t* __restrict__ v_new, int n_new,
                                                          const int32_t* __restrict__ old_len) {
    constexpr int VPR = D / 8;                    // 16-byte vectors per row
    constexpr int RPI = 64 / VPR;                 // rows moved by one wavefront instruction
    constexpr int BATCH = CMP_WAVE_ROWS / RPI;    // instructions per wavefront: 4 (D=128) or 2 (D=64)
    __shared__ int wave_cnt[CMP_CHUNK / 64];
    __shared__ int list[CMP_CHUNK];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int ch = blockIdx.x;
    // (what the tables hold at or beyond `total` is not used; the grid never exceeds them)
    const ChunkDesc d = ws.cmp_desc[ch];
    const int64_t dbase = ws.cmp_chunk_dst[ch] & ~CMP_DST_FULL;   // first destination entry of its survivors
    const int err = __hip_atomic_load(ws.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ch >= ws.cmp_chunk_prefix[sh.nseg] || err != 0) return;
    const int64_t sbase = d.first;                                // first source entry of the chunk
    // NEW: index of the chunk's first entry in its segment, and where the segment's new entries begin
    const int64_t seg_off = NEW ? sbase - src.seg_start[d.seg] : 0;
    const int64_t first_new = NEW ? old_len[d.seg] : 0;
    const int64_t new_base = NEW ? (int64_t)d.seg * n_new - first_new : 0;   // + index in the segment = row of k_new
    // the first CMP_CHUNK threads rank the survivors; an entry's metadata is asked for with its mask byte
    int rank = 0;
    bool flag = false;
    float md_lb = 0.f, md_lt = 0.f;
    int md_pos = 0;
    if (tid < CMP_CHUNK) {
        const bool in = tid < d.n;
        const uint8_t kb = in ? keep[sbase + tid] : (uint8_t)0;
        if (in) {
            md_lb = src.log_beta[sbase + tid];
            if (src.log_tail) md_lt = src.log_tail[sbase + tid];
            md_pos = src.pos[sbase + tid];
        }
        flag = kb != 0;
        const uint64_t mask = __ballot(flag);
        rank = mbcnt(mask);
        if (lane == 0) wave_cnt[wave] = __popcll(mask);
    }
    __syncthreads();
    int cnt = 0;
#pragma unroll
    for (int w = 0; w < CMP_CHUNK / 64; ++w) {
        if (w < wave && tid < CMP_CHUNK) rank += wave_cnt[w];
        cnt += wave_cnt[w];
    }
    if (flag) {
        list[rank] = tid;
        dst.log_beta[dbase + rank] = md_lb;
        if (src.log_tail) dst.log_tail[dbase + rank] = md_lt;
        dst.pos[dbase + rank] = md_pos;
    }
    __syncthreads();
    const int r0 = wave * CMP_WAVE_ROWS;                          // this wavefront's rows of the survivor list
    if (r0 >= cnt) return;
    const uint4* sk = reinterpret_cast<const uint4*>(src.k);
    const uint4* sv = reinterpret_cast<const uint4*>(src.v);
    uint4* dk = reinterpret_cast<uint4*>(dst.k);
    uint4* dv = reinterpret_cast<uint4*>(dst.v);
    const int sub = lane / VPR, col = lane % VPR;
    uint4 kk[BATCH], vv[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
        const int e = list[min(r0 + u * RPI + sub, cnt - 1)];     // clamped: loads stay on live rows
        const bool fresh = NEW && seg_off + e >= first_new;
        const int64_t row = (fresh ? new_base + seg_off + e : sbase + e) * VPR + col;
        kk[u] = ld16_nt((fresh ? reinterpret_cast<const uint4*>(k_new) : sk) + row);
        vv[u] = ld16_nt((fresh ? reinterpret_cast<const uint4*>(v_new) : sv) + row);
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
        const int r = r0 + u * RPI + sub;
        if (r < cnt) {
            const int64_t de = (dbase + r) * VPR + col;
            st16_nt(dk + de, kk[u]);
            st16_nt(dv + de, vv[u]);
        }
    }
}

void launch_cmp_scan_aligned(kvtrim_ctx* ctx, const CacheView& src, const uint8_t* keep, const int32_t* kept,
                             const CacheViewMut& dst, int32_t reserve, int32_t align, hipStream_t st, bool gat) {
    ProfScope prof(ctx, K_CMP_SCAN, st);
    const int g = gat ? 1 : 0;
    if (ctx->shape.nseg > 1024) {                                 // see k_cmp_prefix
        hipLaunchKernelGGL(k_cmp_prefix, dim3(1), dim3(SCAN_THREADS), 0, st, src, kept, dst, reserve, align, ctx->shape, ctx->ws, 0, g);
        hipLaunchKernelGGL((k_cmp_scan<true, PRE_THREADS>), dim3(ctx->shape.nseg), dim3(PRE_THREADS), 0, st, src, keep, kept, dst, reserve,
                           align, ctx->shape, ctx->ws, 0, g);
    } else {
        hipLaunchKernelGGL((k_cmp_scan<false, SCAN_THREADS>), dim3(ctx->shape.nseg), dim3(SCAN_THREADS), 0, st, src, keep, kept, dst, reserve,
                           align, ctx->shape, ctx->ws, 0, g);
    }
}

// The tables for a compaction inside the cache itself: every segment keeps its start, chunk ch's survivors go to
// ws.cmp_chunk_dst[ch] = seg_start + survivors of the segment's earlier chunks; nothing of the cache is written.
void launch_cmp_scan_inplace(kvtrim_ctx* ctx, const CacheViewMut& c, const uint8_t* keep, const int32_t* kept, hipStream_t st) {
    ProfScope prof(ctx, K_CMP_SCAN, st);
    CacheView src;
    src.k = c.k; src.v = c.v; src.log_beta = c.log_beta; src.pos = c.pos;
    src.seg_start = c.seg_start; src.seg_len = c.seg_len; src.cap = c.cap; src.log_tail = c.log_tail;
    if (ctx->shape.nseg > 1024) {
        hipLaunchKernelGGL(k_cmp_prefix, dim3(1), dim3(SCAN_THREADS), 0, st, src, kept, c, 0, 1, ctx->shape, ctx->ws, 1, 0);
        hipLaunchKernelGGL((k_cmp_scan<true, PRE_THREADS>), dim3(ctx->shape.nseg), dim3(PRE_THREADS), 0, st, src, keep, kept, c, 0, 1,
                           ctx->shape, ctx->ws, 1, 0);
    } else {
        hipLaunchKernelGGL((k_cmp_scan<false, SCAN_THREADS>), dim3(ctx->shape.nseg), dim3(SCAN_THREADS), 0, st, src, keep, kept, c, 0, 1,
                           ctx->shape, ctx->ws, 1, 0);
    }
}

void launch_cmp_scan(kvtrim_ctx* ctx, const CacheView& src, const uint8_t* keep, const int32_t* kept,
                     const CacheViewMut& dst, int32_t reserve, hipStream_t st) {
    launch_cmp_scan_aligned(ctx, src, keep, kept, dst, reserve, 1, st);
}

kvtrim_status launch_compact(kvtrim_ctx* ctx, const CacheView& src, const uint8_t* keep, const int32_t* kept,
                             const CacheViewMut& dst, int32_t reserve, hipStream_t st) {
    launch_cmp_scan_aligned(ctx, src, keep, kept, dst, reserve, 1, st, gather_fits(ctx, src.cap, dst.cap));
    return launch_cmp_copy(ctx, src, keep, dst, st);
}

// The row mover alone (the tables of k_cmp_scan must be in the workspace - with gat = gather_fits(...), which decides
// here which mover runs).
kvtrim_status launch_cmp_copy(kvtrim_ctx* ctx, const CacheView& src, const uint8_t* keep, const CacheViewMut& dst,
                              hipStream_t st) {
    const Shape& sh = ctx->shape;
    const Workspace& ws = ctx->ws;
    const int64_t max_chunks = src.cap / CMP_CHUNK + sh.nseg;
    if (max_chunks > 0) {
        ProfScope prof(ctx, K_CMP_COPY, st);
        const dim3 grid((unsigned)max_chunks), block(CMP_THREADS);
        if (gather_fits(ctx, src.cap, dst.cap))                   // few survivors per chunk: a block per chunk of the destination
            return launch_gather_rows(ctx, src, dst, st);
        if (sh.head_dim == 128)
            hipLaunchKernelGGL((k_cmp_copy<128, false>), grid, block, 0, st, src, keep, dst, sh, ws, nullptr, nullptr, 0, nullptr);
        else
            hipLaunchKernelGGL((k_cmp_copy<64, false>), grid, block, 0, st, src, keep, dst, sh, ws, nullptr, nullptr, 0, nullptr);
    }
    KVTRIM_HIP(ctx, hipGetLastError());
    return KVTRIM_OK;
}

constexpr size_t THREE_BLOCKS_LDS = 40960;                        // and what the kernel itself uses: three blocks to a compute unit's 160 KB
kvtrim_status launch_cmp_copy_new(kvtrim_ctx* ctx, const CacheView& src, const uint8_t* keep, const CacheViewMut& dst,
                                  const uint16_t* k_new, const uint16_t* v_new, int32_t n_new, const int32_t* old_len,
                                  hipStream_t st) {
    const Shape& sh = ctx->shape;
    const Workspace& ws = ctx->ws;
    const int64_t max_chunks = src.cap / CMP_CHUNK + sh.nseg;
    if (max_chunks > 0) {
        ProfScope prof(ctx, K_CMP_COPY, st);
        const dim3 grid((unsigned)max_chunks), block(CMP_THREADS);
        // Two blocks a compute unit where most entries stay (mover_lds): a cache at its budget keeps as many as it held, half of all
        // if the new ones are not more than those.  256 lists, chunks of 1024 into 8192 440 us (with four blocks 448), 4096 into
        // 4096 251 (253); but four sequences, 4096 into 2048 547, with four 498.  Rows of 128 bytes: three blocks where two
        // thirds stay: 1024 into 8192 239 us (with four blocks 249, two 240), 4096 into four times 8192 883 (913, 936); 4000 into
        // 4000 164 (158, 178).
        const int64_t fresh = (int64_t)sh.nseg * n_new;
        const bool most_stay = src.cap >= (sh.head_dim == 128 ? 2 : 3) * fresh;
        if (sh.head_dim == 128)
            hipLaunchKernelGGL((k_cmp_copy<128, true>), grid, block, most_stay ? mover_lds(128, 0, max_chunks) : 0, st, src, keep, dst, sh, ws, k_new, v_new, n_new, old_len);
        else
            hipLaunchKernelGGL((k_cmp_copy<64, true>), grid, block, most_stay && max_chunks >= MOVER_BLOCKS ? THREE_BLOCKS_LDS : 0, st, src, keep, dst, sh, ws, k_new, v_new, n_new, old_len);
    }
    KVTRIM_HIP(ctx, hipGetLastError());
    return KVTRIM_OK;
}

}  // namespace kvtrim
