// Device code of the paged layout that more than one kernel file uses: the view of a paged cache, the chunk
// table over its block tables, and the tidying of a block table after an eviction.
#pragma once
#include "kvtrim_device.h"

namespace kvtrim {

constexpr int P = KVTRIM_PAGE_SIZE;

constexpr int PG_TABLE_BLOCKS = 16;        // blocks that share the building of a chunk table
constexpr int ATT_PAGE_GROUP = 4;          // an attention call takes at most this many pages per slot of the partial-result buffer

// ---------------------------------------------------------------------------------------------
// Chunk table of a paged cache for the selection: the pages of every segment, in segment order, one chunk per page.
// prefix[g] = first chunk of segment g, prefix[nseg] = number of chunks, desc = {first slot of the page, page size,
// segment}; entry_prefix counts the live entries of the segments before g.
// Built by `nparts` blocks: every block scans the per-segment counts (a few thousand integers),
// block `part` fills the descriptors of the segments g = part (mod nparts), one wavefront per
// segment, and block 0 writes the prefixes.  Returns the number of chunks.  Counts that do not
// fit raise ERR_LAYOUT and leave the table empty; a page id out of range raises it too and is
// clamped, so that no reader leaves the pool.
__device__ __forceinline__ int build_page_table(const PagedView& pc, int nseg, int32_t* prefix, ChunkDesc* desc,
                                                int64_t max_chunks, int64_t* entry_prefix, int32_t* err, int part, int nparts) {
    __shared__ uint64_t s_scan[17];
    __shared__ int s_bad;
    __shared__ int s_c0[1024], s_n[1024];
    const int tid = threadIdx.x;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    uint64_t carry = 0;
    for (int base = 0; base < nseg; base += blockDim.x) {
        const int g = base + tid;
        uint64_t v = 0;
        int npg = 0;
        if (g < nseg) {
            npg = pc.seg_pages[g];
            const int live = pc.seg_live[g];
            if (npg < 0 || npg > pc.max_pps || live < 0 || (int64_t)live > (int64_t)npg * P) {
                s_bad = 1;
                npg = 0;
            } else {
                v = ((uint64_t)live << 32) | (uint64_t)npg;
            }
        }
        uint64_t tot;
        const uint64_t ex = carry + block_excl_scan<uint64_t>(v, s_scan, &tot);
        carry += tot;
        const int c0 = (int)(ex & 0xffffffffu);
        if (g < nseg && part == 0) {
            prefix[g] = c0;
            entry_prefix[g] = (int64_t)(ex >> 32);
        }
        s_c0[tid] = c0;
        s_n[tid] = npg;
        __syncthreads();
        if (!s_bad && (int64_t)(carry & 0xffffffffu) <= max_chunks) {
            const int lane = lane_id(), wave = tid >> 6, nw = blockDim.x >> 6;
            const int ntile = min((int)blockDim.x, nseg - base);
            const int first_t = ((part - base) % nparts + nparts) % nparts;      // first t with (base + t) = part (mod nparts)
            for (int t = first_t + wave * nparts; t < ntile; t += nw * nparts) {
                const int gg = base + t, cc = s_c0[t], nn = s_n[t];
                const int64_t row = (int64_t)gg * pc.max_pps;
                bool bad_page = false;
                for (int i = lane; i < nn; i += 64) {
                    const int pg = pc.block_table[row + i];
                    bad_page |= pg < 0 || pg >= pc.n_pages;
                    ChunkDesc d;
                    d.seg = gg;
                    d.first = (int64_t)min(max(pg, 0), pc.n_pages - 1) * P;
                    d.n = P;
                    desc[cc + i] = d;
                }
                if (__any(bad_page) && lane == 0) atomicOr(err, ERR_LAYOUT);
            }
        }
        __syncthreads();
    }
    const int64_t total = (int64_t)(carry & 0xffffffffu);
    if (s_bad || total > max_chunks) {
        if (part == 0) {
            if (tid == 0) atomicOr(err, ERR_LAYOUT);
            for (int g = tid; g <= nseg; g += blockDim.x) {
                prefix[g] = 0;
                entry_prefix[g] = 0;
            }
        }
        __syncthreads();
        return 0;
    }
    if (tid == 0 && part == 0) {
        prefix[nseg] = (int32_t)total;
        entry_prefix[nseg] = (int64_t)(carry >> 32);
    }
    __syncthreads();
    return (int)total;
}

// A block of THREADS threads tidies segment g: the pages marked for release leave its block table (order of
// the others kept) and return to the free list.  A released page that is still in the table is harmless to a
// reader - every slot of it is empty - so this may run any time after the eviction and before the next append.
template <int THREADS>
__device__ __forceinline__ void tidy_segment(const PagedView& pc, int g, int32_t* err) {
    __shared__ int32_t lds32[17];
    __shared__ int32_t s_page[THREADS];
    const int tid = threadIdx.x;
    const int npg = pc.seg_pages[g];
    if (npg < 0 || npg > pc.max_pps) {
        if (tid == 0) atomicOr(err, ERR_LAYOUT);
        return;
    }
    int32_t* bt = pc.block_table + (int64_t)g * pc.max_pps;
    int out = 0;
    for (int base = 0; base < npg; base += THREADS) {                    // read a tile, then write it: out <= base
        const int i = base + tid;
        int page = -1;
        bool alive = false;
        if (i < npg) {
            page = bt[i];
            if (page >= 0 && page < pc.n_pages) {
                alive = pc.page_owner[page] == g;
                if (!alive && pc.page_owner[page] == -2) {          // release
                    pc.page_owner[page] = -1;
                    pc.page_live[page] = 0;
                    const int idx = atomicAdd(pc.n_free, 1);
                    if (idx >= 0 && idx < pc.n_pages) pc.free_list[idx] = page;
                }
            }
        }
        int32_t tot;
        const int32_t ex = block_excl_scan<int32_t>(alive ? 1 : 0, lds32, &tot);
        s_page[tid] = page;
        __syncthreads();
        if (alive) bt[out + ex] = s_page[tid];
        __syncthreads();
        out += tot;
    }
    if (tid == 0) pc.seg_pages[g] = out;
}

// The same by a wavefront, a few tiles of 64 pages at a time.  all: every page goes with all that is in it, whatever it is marked as.
__device__ __forceinline__ void tidy_segment_by_wave(const PagedView& pc, int g, bool all, int32_t* err) {
    constexpr int TILES = 4;
    const int lane = lane_id(), npg = pc.seg_pages[g];
    if (npg < 0 || npg > pc.max_pps) {
        if (lane == 0) atomicOr(err, ERR_LAYOUT);
        return;
    }
    int32_t* bt = pc.block_table + (int64_t)g * pc.max_pps;
    const uint64_t below = (1ull << lane) - 1ull;
    int out = 0;
    for (int base = 0; base < npg; base += 64 * TILES) {                 // read a tile, then write it: out <= base
        int page[TILES], owner[TILES];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int i = base + 64 * t + lane;
            page[t] = i < npg ? bt[i] : -1;
            if (page[t] >= pc.n_pages) page[t] = -1;
        }
#pragma unroll
        for (int t = 0; t < TILES; ++t) owner[t] = page[t] < 0 ? -1 : all ? -2 : pc.page_owner[page[t]];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const bool goes = owner[t] == -2, stays = owner[t] == g;
            const uint64_t mg = __ballot(goes), ms = __ballot(stays);
            if (all) {
                for (uint64_t m = mg; m; m &= m - 1) {
                    const int pg = __builtin_amdgcn_readlane(page[t], __ffsll((long long)m) - 1);
                    reinterpret_cast<int2*>(pc.pos + (int64_t)pg * P)[lane] = make_int2(-1, -1);
                }
            }
            if (mg) {
                int at = 0;
                if (lane == 0) at = atomicAdd(pc.n_free, __popcll(mg));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(mg & below);
                if (goes) {
                    pc.page_owner[page[t]] = -1;
                    pc.page_live[page[t]] = 0;
                    if (at >= 0 && at < pc.n_pages) pc.free_list[at] = page[t];
                }
            }
            if (stays) bt[out + __popcll(ms & below)] = page[t];
            out += __popcll(ms);
        }
    }
    if (lane == 0) pc.seg_pages[g] = out;
}

}  // namespace kvtrim
