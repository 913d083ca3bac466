// Binning of the depth-ordered Gaussians into supers (blocks of 4 x 4 tiles,
// 64 x 64 pixels) for gfx950.
//
// A super's list holds every Gaussian whose tile rectangle meets the super,
// in depth order, with a 16-bit mask of the super's tiles that the rectangle
// covers; a tile's list is the entries of its super whose mask has the
// tile's bit, in the same order.  The forward blend filters its super's list
// as it walks it, so no (Gaussian, tile) pair is ever written: on 300K
// Gaussians at 1352 x 1014 (34M pairs, of which the blend walks 3%) a
// Gaussian takes 11 super entries of 6 bytes instead of 114 pairs of 4.
// Against the pair list (binned chunk by chunk, every pair written), render
// and renderer backward of 1M Gaussians at 1920 x 1080 went from 2.42 to
// 1.95 ms, the 300K training step from 1.34 to 1.20 ms, a novel view of a
// 300K surface scene (4 pairs a Gaussian) from 0.57 to 0.46 ms.  4 x 4 tiles:
// the mask fits 16 bits, and a tile filters 1.6 list entries for each of its
// own where Gaussians are 10 tiles wide, 6 where they are 2 wide.
//
// Three launches: the counts per (super, chunk of 512 Gaussians), each
// super's exclusive scan over the chunks, and the scatter.  Which of a wave's
// 64 Gaussians meet a super is the AND of two words, those that meet its
// column and those that meet its row (cover_words), whatever the size of the
// rectangles; the counts and the ranks inside a chunk are popcounts of them.
#include <algorithm>

#include "kernels.h"

namespace gs3 {

namespace {

constexpr int kBigRect = 32;     // supers walked by one thread (16 or 64: 6% or 1% more render time at 1M Gaussians)
constexpr int kMaxCols = 64;     // supers of the widest view (4096 pixels)
constexpr int kPartRows = 64;    // rows of supers whose words are in LDS at a time, at most
constexpr int kPartSupers = 512; // supers of a scatter workgroup, at most
constexpr int kScatterBlocks = 512;   // its workgroups, at least where the rows of supers can be cut
constexpr int kWords = kSuperChunk / 64;

struct SRect {
    int x0, y0, x1, y1;   // supers; empty when x0 > x1
};

__device__ __forceinline__ SRect super_rect(uint2 r) {
    return SRect{(int)(r.x & 0xFFFFu) >> kSuperShift, (int)(r.x >> 16) >> kSuperShift,
                 (int)(r.y & 0xFFFFu) >> kSuperShift, (int)(r.y >> 16) >> kSuperShift};
}

__device__ __forceinline__ bool empty_rect(uint2 r) { return (r.x & 0xFFFFu) > (r.y & 0xFFFFu); }

// The tiles of super (sx, sy) that tile rectangle r covers: bit 4 ly + lx.
__device__ __forceinline__ uint32_t tile_mask(uint2 r, int sx, int sy) {
    constexpr int D = kSuperDim;
    const int lx0 = max((int)(r.x & 0xFFFFu) - D * sx, 0), lx1 = min((int)(r.y & 0xFFFFu) - D * sx, D - 1);
    const int ly0 = max((int)(r.x >> 16) - D * sy, 0), ly1 = min((int)(r.y >> 16) - D * sy, D - 1);
    const uint32_t cols = ((1u << (lx1 + 1)) - 1u) & ~((1u << lx0) - 1u);
    const uint32_t rows = ((1u << (D * (ly1 + 1))) - 1u) & ~((1u << (D * ly0)) - 1u);
    return (cols * 0x1111u) & rows;
}

// Orders a wave's own LDS accesses for the compiler (they complete in issue order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f(e, sx, sy) for every super of rows [y0, y1) that the rectangles of a wave's
// Gaussians meet (e: position in the chunk, r: tile rectangle).  A rectangle of
// more than kBigRect supers is walked by the whole wave, so a few large
// Gaussians do not leave one lane looping.
template <class F>
__device__ __forceinline__ void for_supers(uint2 r, int e, int lane, int y0, int y1, F f) {
    SRect q = super_rect(r);
    q.y0 = max(q.y0, y0);
    q.y1 = min(q.y1, y1 - 1);
    const int w = q.x1 - q.x0 + 1;
    const int cnt = empty_rect(r) || q.y0 > q.y1 ? 0 : w * (q.y1 - q.y0 + 1);
    if (cnt <= kBigRect) {
        int sx = q.x0, sy = q.y0;
        for (int k = 0; k < cnt; k++) {
            f(e, sx, sy);
            if (++sx > q.x1) {
                sx = q.x0;
                sy++;
            }
        }
    }
    uint64_t big = __ballot(cnt > kBigRect);
    while (big) {
        const int l = __builtin_ctzll(big);
        big &= big - 1;
        const int bx0 = __builtin_amdgcn_readlane(q.x0, l), by0 = __builtin_amdgcn_readlane(q.y0, l);
        const int bw = __builtin_amdgcn_readlane(w, l), bc = __builtin_amdgcn_readlane(cnt, l);
        const int be = __builtin_amdgcn_readlane(e, l);
        for (int k = lane; k < bc; k += 64) f(be, bx0 + k % bw, by0 + k / bw);
    }
}

// Bit l of cols[sx] and rows[sy - y0]: the rectangle of the wave's Gaussian l
// meets column sx and row sy of supers, rows y0 <= sy < y1 <= y0 + kPartRows.
// A Gaussian sets its own bits, or, where one of the wave is large or the columns
// and rows are few, a column or a row is asked of all at once.  The latter
// alone takes 17 us of counting for 14 where Gaussians meet two or three supers
// (502K surfaces at 1920 x 1080), the former 17 for 15 with one super (1M).
constexpr int kLoopExtent = 16;
__device__ __forceinline__ void cover_words(uint2 r, int supers_x, int y0, int y1, int lane, uint64_t* cols,
                                            uint64_t* rows) {
    SRect q = super_rect(r);
    q.y0 = max(q.y0, y0);
    q.y1 = min(q.y1, y1 - 1);
    if (empty_rect(r)) q = SRect{1, 1, 0, 0};
    if (supers_x + y1 - y0 <= kLoopExtent || __ballot(q.x1 - q.x0 + q.y1 - q.y0 > kLoopExtent)) {
        uint64_t mine = 0;
        for (int x = 0; x < supers_x; x++) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(q.x0 <= x) & __builtin_amdgcn_ballot_w64(x <= q.x1);
            mine = lane == x ? m : mine;
        }
        cols[lane] = mine;
        for (int y = y0; y < y1; y++) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(q.y0 <= y) & __builtin_amdgcn_ballot_w64(y <= q.y1);
            mine = lane == y - y0 ? m : mine;
        }
        rows[lane] = mine;   // the words past the last row are not read
    } else {
        cols[lane] = 0;
        rows[lane] = 0;
        wave_lds_fence();
        for (int x = q.x0; x <= q.x1; x++) atomicOr(reinterpret_cast<unsigned long long*>(cols + x), 1ull << lane);
        for (int y = q.y0; y <= q.y1; y++) atomicOr(reinterpret_cast<unsigned long long*>(rows + y - y0), 1ull << lane);
    }
}

// Counts per super of one chunk of the depth order, hist[super][chunk]; the
// tile rectangles gathered into depth order; and the chunk's number of
// (Gaussian, tile) pairs.  Counters that every Gaussian adds to in each super
// it meets took 56 us for 8 with 20K view-filling ones (1920 x 1080).
__global__ __launch_bounds__(kSuperChunk) void k_super_count(const uint32_t* __restrict__ order, int64_t n,
                                                             const uint2* __restrict__ rect, int supers_x, int nsuper,
                                                             int64_t nchunks, uint2* __restrict__ srect,
                                                             uint32_t* __restrict__ hist, uint64_t* __restrict__ ksum) {
    __shared__ uint64_t s_cols[kWords][kMaxCols], s_rows[kWords][kPartRows];
    __shared__ uint64_t s_k[kSuperChunk / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * kSuperChunk + threadIdx.x;
    uint2 r = make_uint2(1u, 0u);
    if (e < n) {
        r = rect[order[e]];
        srect[e] = r;
    }
    const int supers_y = nsuper / supers_x;
    for (int y0 = 0; y0 < supers_y; y0 += kPartRows) {
        const int y1 = min(y0 + kPartRows, supers_y);
        if (y0) __syncthreads();   // the previous rows' words are no longer read
        cover_words(r, supers_x, y0, y1, lane, s_cols[w], s_rows[w]);
        __syncthreads();
        for (int s = y0 * supers_x + (int)threadIdx.x; s < y1 * supers_x; s += kSuperChunk) {
            const int y = s / supers_x, x = s - y * supers_x;
            uint32_t c = 0u;
#pragma unroll
            for (int q = 0; q < kWords; q++) c += (uint32_t)__popcll(s_cols[q][x] & s_rows[q][y - y0]);
            hist[(int64_t)s * nchunks + blockIdx.x] = c;
        }
    }
    uint64_t k = 0;
    if (!empty_rect(r))
        k = (uint64_t)((r.y & 0xFFFFu) - (r.x & 0xFFFFu) + 1u) * (uint64_t)((r.y >> 16) - (r.x >> 16) + 1u);
    for (int off = 32; off > 0; off >>= 1) k += __shfl_xor(k, off, 64);
    if (lane == 0) s_k[w] = k;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int q = 0; q < kSuperChunk / 64; q++) t += s_k[q];
        ksum[blockIdx.x] = t;
    }
}

// Block s < nsuper: exclusive scan of hist[s][0..nchunks) in place, the
// super's entries to len[s].  The last block adds up the chunks' pairs into
// *total and flags an overflow.
__global__ __launch_bounds__(256) void k_super_scan(uint32_t* __restrict__ hist, const uint64_t* __restrict__ ksum,
                                                    int64_t nchunks, int nsuper, uint64_t cap, uint32_t* __restrict__ len,
                                                    uint64_t* __restrict__ total, int* __restrict__ overflow) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if ((int)blockIdx.x == nsuper) {
        __shared__ uint64_t s_t[4];
        uint64_t k = 0;
        for (int64_t c = threadIdx.x; c < nchunks; c += 256) k += ksum[c];
        for (int off = 32; off > 0; off >>= 1) k += __shfl_xor(k, off, 64);
        if (lane == 0) s_t[w] = k;
        __syncthreads();
        if (threadIdx.x == 0) {
            k = s_t[0] + s_t[1] + s_t[2] + s_t[3];
            *total = k;
            if (k > cap) atomicOr(overflow, 1);
        }
        return;
    }
    __shared__ uint32_t s_w[2][4];
    uint32_t* h = hist + (int64_t)blockIdx.x * nchunks;
    uint32_t carry = 0u;
    int par = 0;
    for (int64_t c0 = 0; c0 < nchunks; c0 += 256, par ^= 1) {
        const int64_t c = c0 + threadIdx.x;
        const uint32_t v = c < nchunks ? h[c] : 0u;
        const uint32_t x = wave_incl_scan_u32(v);
        if (lane == 63) s_w[par][w] = x;
        __syncthreads();   // the other half of s_w is still read by slower waves of the previous round
        uint32_t pre = carry;
        for (int k = 0; k < 4; k++) {
            if (k < w) pre += s_w[par][k];
            carry += s_w[par][k];
        }
        if (c < nchunks) h[c] = pre + x - v;
    }
    if (threadIdx.x == 0) len[blockIdx.x] = carry;
}

// Scatter of one chunk into the supers of some rows: entry (id, tile mask) of
// every super its Gaussians meet, at the super's start + the entries of earlier
// chunks + the rank among the chunk's Gaussians that meet the super (a popcount
// of the words below).
//
// Few entries for a super (under kDense): the entries are first put in list
// order in LDS, kEntries at a time, each by its Gaussian's thread, so that
// consecutive lanes write consecutive slots of a super's segment (a dozen or two
// entries): stored straight from the Gaussian's thread every lane wrote to
// another segment, and those requests bounded the kernel (1M Gaussians at 1920 x
// 1080, 18M entries: 292 -> 129 us; 300K at 1352 x 1014: 49 -> 33 us; with under
// two entries a Gaussian the detour costs 1-2 us).  What is left is the loops
// over the supers of the widest Gaussian of each wave; with a bit per Gaussian
// and super set by such a loop, too, in place of the words, it was 134 us for 100
// and 37 for 31.
//
// Many: a wave takes a super at a time and its lanes the Gaussians, 64 at a
// time, whose entries follow each other in the list.  Each round through LDS
// walks every rectangle: with that alone, view-filling Gaussians (20K at 1920 x
// 1080, 10M entries) took 3376 us, 25 this way.
//
// Grid (chunks, parts): where there are few chunks, the rows of supers are cut
// into parts (2000 Gaussians at 4096 x 1024, four chunks: 198 -> 14 us).  The
// workgroups of chunk 0 also write the supers' starts, and the first of them
// the longest-first order (sorder, when set: scheduling only) and resets the
// walked-block counter *pool.
constexpr int kEntries = 6144;   // with the other arrays three workgroups share a CU's LDS
constexpr int kDense = 48;       // entries for a super from which it is listed by a wave: six a word
__global__ __launch_bounds__(kSuperChunk) void k_super_scatter(
    const uint32_t* __restrict__ order, int64_t n, const uint2* __restrict__ srect, int supers_x, int nsuper,
    int rows_per, int64_t nchunks, const uint32_t* __restrict__ hist, const uint32_t* __restrict__ len, uint32_t cap,
    uint32_t* __restrict__ ids, uint16_t* __restrict__ masks, uint32_t* __restrict__ start, int* __restrict__ sorder,
    uint32_t* __restrict__ pool, uint32_t pool0) {
    constexpr int NW = kSuperChunk / 64;
    __shared__ uint64_t s_cols[kWords][kMaxCols], s_rows[kWords][kPartRows];
    __shared__ uint16_t s_pre[kPartSupers][kWords];
    __shared__ uint32_t s_base[kPartSupers];   // first slot of this chunk's entries of the super
    __shared__ uint32_t s_loc[kPartSupers];    // and their first place in the chunk's list
    __shared__ uint32_t s_xy[kPartSupers];     // the super's column and row
    __shared__ uint2 s_rect[kSuperChunk];
    __shared__ uint32_t s_id[kSuperChunk];
    __shared__ uint32_t s_ent[kEntries];       // chunk position | super << 16
    __shared__ uint64_t s_w[NW], s_b[NW];
    __shared__ uint32_t s_l[NW];
    static_assert(kPartSupers == kSuperChunk, "one thread per super of a part");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t g = (int64_t)blockIdx.x * kSuperChunk + threadIdx.x;
    const int me = (int)threadIdx.x;
    const int y0 = (int)blockIdx.y * rows_per, y1 = min(y0 + rows_per, nsuper / supers_x);
    const int b0 = y0 * supers_x, nb = (y1 - y0) * supers_x;   // the part's supers
    uint2 r = make_uint2(1u, 0u);
    if (g < n) {
        r = srect[g];
        s_id[me] = order[g];
    }
    s_rect[me] = r;
    if (blockIdx.x == 0 && blockIdx.y == 0 && me == 0) {
        pool[0] = pool0;
        pool[1] = 0u;
    }
    const int s = b0 + me, y = s / supers_x, x = s - y * supers_x;
    const uint64_t v = me < nb ? (uint64_t)len[s] : 0;
    const uint32_t before = me < nb ? hist[(int64_t)s * nchunks + blockIdx.x] : 0u;
    uint64_t below = 0;   // entries of the supers before the part's
    for (int k = me; k < b0; k += kSuperChunk) below += len[k];
    uint64_t z = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t u = __shfl_up(z, off, 64);
        if (lane >= off) z += u;
    }
    for (int off = 32; off > 0; off >>= 1) below += __shfl_xor(below, off, 64);
    if (lane == 63) s_w[w] = z;
    if (lane == 0) s_b[w] = below;
    s_xy[me] = (uint32_t)x | ((uint32_t)y << 16);
    cover_words(r, supers_x, y0, y1, lane, s_cols[w], s_rows[w]);
    __syncthreads();
    uint32_t run = 0u;
    if (me < nb) {
        uint64_t first = z - v;
        for (int k = 0; k < NW; k++) first += s_b[k] + (k < w ? s_w[k] : 0);
        const uint64_t at = first + before;
        s_base[me] = at < (uint64_t)cap ? (uint32_t)at : cap;
        if (blockIdx.x == 0) start[s] = first < (uint64_t)cap ? (uint32_t)first : cap;
#pragma unroll
        for (int k = 0; k < kWords; k++) {
            s_pre[me][k] = (uint16_t)run;
            run += (uint32_t)__popcll(s_cols[k][x] & s_rows[k][y - y0]);
        }
    }
    const uint32_t lx = wave_incl_scan_u32(run);
    if (lane == 63) s_l[w] = lx;
    __syncthreads();
    uint32_t loc = lx - run, total = 0u;
    for (int k = 0; k < NW; k++) {
        if (k < w) loc += s_l[k];
        total += s_l[k];
    }
    if (total >= (uint32_t)(kDense * nb)) {
        uint32_t id[kWords];
        uint2 rc[kWords];
#pragma unroll
        for (int k = 0; k < kWords; k++) {
            id[k] = s_id[64 * k + lane];
            rc[k] = s_rect[64 * k + lane];
        }
        for (int q = w; q < nb; q += NW) {
            const uint32_t xy = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_xy[q]);
            const int sx = (int)(xy & 0xFFFFu), sy = (int)(xy >> 16);
            uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_base[q]);
#pragma unroll
            for (int k = 0; k < kWords; k++) {
                const uint64_t m = uniform64(s_cols[k][sx] & s_rows[k][sy - y0]);
                const uint32_t slot = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                // base <= cap < 2^31 and the rank is below kSuperChunk: no wrap
                if (__builtin_amdgcn_inverse_ballot_w64(m) && slot < cap) {
                    ids[slot] = id[k];
                    masks[slot] = (uint16_t)tile_mask(rc[k], sx, sy);
                }
                at += (uint32_t)__popcll(m);
            }
        }
    } else {
        s_loc[me] = loc;
        for (uint32_t w0 = 0; w0 < total; w0 += kEntries) {
            __syncthreads();   // s_loc written; the previous round's entries are no longer read
            for_supers(r, me, lane, y0, y1, [&](int e, int sx, int sy) {
                const int q = sy * supers_x + sx - b0;
                // e is one of this wave's Gaussians
                const uint64_t under = s_cols[w][sx] & s_rows[w][sy - y0] & ((1ull << (e & 63)) - 1ull);
                const uint32_t at = s_loc[q] + s_pre[q][w] + (uint32_t)__popcll(under) - w0;
                if (at < (uint32_t)kEntries) s_ent[at] = (uint32_t)e | ((uint32_t)q << 16);
            });
            __syncthreads();
            const uint32_t m = min((uint32_t)kEntries, total - w0);
            for (uint32_t i = me; i < m; i += kSuperChunk) {
                const uint32_t t = s_ent[i], q = t >> 16, e = t & 0xFFFFu, xy = s_xy[q];
                const uint32_t slot = s_base[q] + (w0 + i - s_loc[q]);
                if (slot < cap) {
                    ids[slot] = s_id[e];
                    masks[slot] = (uint16_t)tile_mask(s_rect[e], (int)(xy & 0xFFFFu), (int)(xy >> 16));
                }
            }
        }
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && sorder) {
        __syncthreads();   // s_base is no longer read
        // longest list first, on a half-octave scale
        uint32_t* cnt = s_base;
        for (int b = me; b < 66; b += kSuperChunk) cnt[b] = 0u;
        __syncthreads();
        for (int k = me; k < nsuper; k += kSuperChunk) atomicAdd(&cnt[work_bucket(len[k])], 1u);
        __syncthreads();
        if (me == 0) {
            uint32_t acc = 0u;
            for (int b = 65; b >= 0; b--) {
                const uint32_t c = cnt[b];
                cnt[b] = acc;
                acc += c;
            }
        }
        __syncthreads();
        for (int k = me; k < nsuper; k += kSuperChunk) sorder[atomicAdd(&cnt[work_bucket(len[k])], 1u)] = k;
    }
}

// The tile-major lists of a view with few tiles, for the narrow blends: each
// tile's workgroup counts the entries of its super's list with the tile's bit,
// takes that many slots of the walked blocks' room (the order of the tiles
// there is any), and writes them in order.  A wave takes a stretch of the list,
// so the workgroup meets twice only, with eight loads of a lane in flight (one
// at a time: 17 -> 8 us at 50K Gaussians and 256 tiles, a launch's 5 us among
// them).  Also clears tile_walk.
constexpr int kListThreads = 1024;
__global__ __launch_bounds__(kListThreads) void k_super_lists(const uint32_t* __restrict__ ids,
                                                              const uint16_t* __restrict__ masks,
                                                              const uint32_t* __restrict__ start,
                                                              const uint32_t* __restrict__ len, uint32_t cap,
                                                              int supers_x, int tiles_x, uint64_t slots,
                                                              unsigned long long* __restrict__ pool,
                                                              uint32_t* __restrict__ list, uint2* __restrict__ ranges,
                                                              uint32_t* __restrict__ tile_walk) {
    constexpr int NW = kListThreads / 64;
    __shared__ uint32_t s_n[NW];
    __shared__ uint64_t s_at;
    const int tile = blockIdx.x, tx = tile % tiles_x, ty = tile / tiles_x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int s = (ty >> kSuperShift) * supers_x + (tx >> kSuperShift);
    const int bit = (ty % kSuperDim) * kSuperDim + tx % kSuperDim;
    const uint32_t c0 = start[s], c1 = min(cap, c0 + len[s]);
    const uint32_t per = ((c1 - c0 + NW * 64 - 1) / (NW * 64)) * 64, b0 = min(c1, c0 + w * per), b1 = min(c1, b0 + per);
    constexpr int U = 8;   // loads in flight
    uint32_t n = 0u;
    for (uint32_t b = b0; b < b1; b += 64 * U) {
        uint32_t m[U];
#pragma unroll
        for (int u = 0; u < U; u++) m[u] = b + 64 * u + lane < b1 ? masks[b + 64 * u + lane] : 0u;
#pragma unroll
        for (int u = 0; u < U; u++) n += (uint32_t)__popcll(__ballot((m[u] >> bit) & 1u));
    }
    if (lane == 0) s_n[w] = n;
    __syncthreads();
    uint32_t before = 0u, total = 0u;
    for (int k = 0; k < NW; k++) {
        if (k < w) before += s_n[k];
        total += s_n[k];
    }
    if (threadIdx.x == 0) {
        // past the room only when the pairs overflowed
        const uint64_t at = atomicAdd(pool, (unsigned long long)total);
        s_at = at;
        ranges[tile] = make_uint2((uint32_t)min(at, slots), (uint32_t)min(at + total, slots));
        tile_walk[tile] = 0u;
    }
    __syncthreads();
    uint64_t at = s_at + before;
    for (uint32_t b = b0; b < b1; b += 64 * U) {
        uint32_t m[U], id[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t i = b + 64 * u + lane;
            m[u] = i < b1 ? masks[i] : 0u;
            id[u] = i < b1 ? ids[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const bool on = (m[u] >> bit) & 1u;
            const uint64_t bal = __ballot(on);
            const uint64_t k = at + (uint64_t)__popcll(bal & ((1ull << lane) - 1ull));
            if (on && k < slots) list[k] = id[u];
            at += (uint64_t)__popcll(bal);
        }
    }
}

// Pairs per tile (inspection): one workgroup per super counts its masks.
__global__ __launch_bounds__(256) void k_super_tile_counts(const uint16_t* __restrict__ masks,
                                                           const uint32_t* __restrict__ start,
                                                           const uint32_t* __restrict__ len, uint32_t cap, int supers_x,
                                                           int tiles_x, int tiles_y, uint32_t* __restrict__ ttot) {
    constexpr int T = kSuperDim * kSuperDim;
    __shared__ uint32_t s_cnt[T];
    if (threadIdx.x < T) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t c0 = start[blockIdx.x], c1 = min(cap, c0 + len[blockIdx.x]);
    for (uint32_t b = c0; b < c1; b += 256) {
        const uint32_t i = b + threadIdx.x;
        const uint32_t m = i < c1 ? masks[i] : 0u;
#pragma unroll
        for (int t = 0; t < T; t++) {
            const uint32_t c = (uint32_t)__popcll(__ballot((m >> t) & 1u));
            if (c && (threadIdx.x & 63) == 0) atomicAdd(&s_cnt[t], c);
        }
    }
    __syncthreads();
    if (threadIdx.x < T) {
        const int tx = ((int)blockIdx.x % supers_x) * kSuperDim + (int)threadIdx.x % kSuperDim;
        const int ty = ((int)blockIdx.x / supers_x) * kSuperDim + (int)threadIdx.x / kSuperDim;
        if (tx < tiles_x && ty < tiles_y) ttot[ty * tiles_x + tx] = s_cnt[threadIdx.x];
    }
}

// The tile-major pair list (inspection): one workgroup per tile filters its
// super's list in order.
__global__ __launch_bounds__(256) void k_super_pairs(const uint32_t* __restrict__ ids, const uint16_t* __restrict__ masks,
                                                     const uint32_t* __restrict__ start, const uint32_t* __restrict__ len,
                                                     uint32_t cap, int supers_x, int tiles_x,
                                                     const uint2* __restrict__ ranges, const uint32_t* __restrict__ key,
                                                     uint64_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out) {
    __shared__ uint32_t s_c[2][4];
    const int tile = blockIdx.x, tx = tile % tiles_x, ty = tile / tiles_x;
    const int s = (ty >> kSuperShift) * supers_x + (tx >> kSuperShift);
    const int bit = (ty % kSuperDim) * kSuperDim + tx % kSuperDim;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t c0 = start[s], c1 = min(cap, c0 + len[s]);
    const uint2 rg = ranges[tile];
    uint32_t pos = rg.x;
    int par = 0;
    for (uint32_t b = c0; b < c1; b += 256, par ^= 1) {
        const uint32_t i = b + threadIdx.x;
        const bool on = i < c1 && ((masks[i] >> bit) & 1u);
        const uint64_t bal = __ballot(on);
        if (lane == 0) s_c[par][w] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t at = pos + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        for (int k = 0; k < 4; k++) {
            if (k < w) at += s_c[par][k];
            pos += s_c[par][k];
        }
        if (on && at < rg.y) {
            const uint32_t id = ids[i];
            if (vals_out) vals_out[at] = id;
            if (keys_out) keys_out[at] = ((uint64_t)tile << 32) | key[id];
        }
    }
}

}  // namespace

int64_t super_chunks(int64_t n) { return (n + kSuperChunk - 1) / kSuperChunk; }

int super_count_of(int tiles) { return (tiles + kSuperDim - 1) / kSuperDim; }

void super_bin(const Launch& L, const uint32_t* order, int64_t n, const uint2* rect, int tiles_x, int tiles_y,
               uint64_t cap, uint32_t pool0, uint2* srect, uint32_t* hist, uint64_t* ksum, uint64_t* total,
               int* overflow, const SuperDev& sd, int* sorder) {
    if (n <= 0) return;
    const int64_t nchunks = super_chunks(n);
    const int nsuper = sd.supers_x * super_count_of(tiles_y);
    if (L.prof) L.prof->begin("bin_count", L.st);
    hipLaunchKernelGGL(k_super_count, dim3((unsigned)nchunks), dim3(kSuperChunk), 0, L.st, order, n, rect, sd.supers_x,
                       nsuper, nchunks, srect, hist, ksum);
    if (L.prof) L.prof->end(L.st);
    if (L.prof) L.prof->begin("scan", L.st);
    hipLaunchKernelGGL(k_super_scan, dim3((unsigned)nsuper + 1), dim3(256), 0, L.st, hist, ksum, nchunks, nsuper, cap,
                       sd.len, total, overflow);
    if (L.prof) L.prof->end(L.st);
    if (L.prof) L.prof->begin("bin_scatter", L.st);
    // parts of whole rows, as many as give two workgroups per CU
    const int supers_y = super_count_of(tiles_y);
    const int64_t want = std::min<int64_t>(supers_y, (kScatterBlocks + nchunks - 1) / nchunks);
    const int rows = std::min(std::min((int)((supers_y + want - 1) / want), kPartSupers / sd.supers_x), kPartRows);
    const unsigned parts = (unsigned)((supers_y + rows - 1) / rows);
    hipLaunchKernelGGL(k_super_scatter, dim3((unsigned)nchunks, parts), dim3(kSuperChunk), 0, L.st, order, n, srect,
                       sd.supers_x, nsuper, rows, nchunks, hist, sd.len, (uint32_t)cap, sd.ids, sd.masks, sd.start,
                       sorder, sd.pool, pool0);
    if (L.prof) L.prof->end(L.st);
}

void super_lists(const Launch& L, const SuperDev& sd, int tiles_x, int ntiles, uint2* ranges, uint32_t* tile_walk) {
    if (L.prof) L.prof->begin("tile_ranges", L.st);
    hipLaunchKernelGGL(k_super_lists, dim3((unsigned)ntiles), dim3(kListThreads), 0, L.st, sd.ids, sd.masks, sd.start,
                       sd.len, sd.cap, sd.supers_x, tiles_x, (uint64_t)sd.max_blocks * kWalkBlock,
                       reinterpret_cast<unsigned long long*>(sd.pool), sd.walked, ranges, tile_walk);
    if (L.prof) L.prof->end(L.st);
}

void super_tile_counts(const Launch& L, const SuperDev& sd, int tiles_x, int tiles_y, uint32_t* ttot) {
    hipLaunchKernelGGL(k_super_tile_counts, dim3((unsigned)(sd.supers_x * super_count_of(tiles_y))), dim3(256), 0, L.st,
                       sd.masks, sd.start, sd.len, sd.cap, sd.supers_x, tiles_x, tiles_y, ttot);
}

void super_pairs(const Launch& L, const SuperDev& sd, int tiles_x, int tiles_y, const uint2* ranges,
                 const uint32_t* key, uint64_t* keys_out, uint32_t* vals_out) {
    hipLaunchKernelGGL(k_super_pairs, dim3((unsigned)(tiles_x * tiles_y)), dim3(256), 0, L.st, sd.ids, sd.masks,
                       sd.start, sd.len, sd.cap, sd.supers_x, tiles_x, ranges, key, keys_out, vals_out);
}

}  // namespace gs3
