// Tile rasterizer of 3D Gaussians for gfx950 (Sec. 3.2: Eq. 2-4), forward
// and adjoint, plus the Gaussian transform of Sec. 4.1 fused into the
// per-Gaussian kernels.
#include <type_traits>

#include "kernels.h"

namespace gs3 {

namespace {

__device__ __forceinline__ uint32_t pack16(int lo, int hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }

// ---------------------------------------------------------------------------
// preprocess: transform, covariance (Eq. 2), EWA projection (Eq. 3), conic,
// pixel box, tile rectangle, depth key, SH colour, tile count.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_preprocess(GaussDev g, CamDev cam, float4* __restrict__ rec,
                                                    uint32_t* __restrict__ key, uint2* __restrict__ rect,
                                                    uint32_t* __restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= g.n) return;
    Geo o;
    if (!geo_forward(g, cam, i, o)) {
        key[i] = 0xFFFFFFFFu;
        if (count) count[i] = 0;
        rect[i] = make_uint2(1u, 0u);
        rec[3 * i + 0] = make_float4(0.f, 0.f, 0.f, 0.f);
        rec[3 * i + 1] = make_float4(0.f, 0.f, 0.f, 0.f);
        rec[3 * i + 2] = make_float4(0.f, __uint_as_float(pack16(1, 1)), __uint_as_float(0u), 0.f);
        return;
    }
    ColourCtx cc;
    colour_forward(g, cam, i, o, cc);
    const float A = o.c / o.det, B = -o.b / o.det, C = o.a / o.det;
    const float op = opacity_of(g.opac[i]);
    rec[3 * i + 0] = make_float4(o.u, o.v, A, B);
    rec[3 * i + 1] = make_float4(C, op, fmaxf(cc.raw[0], 0.f), fmaxf(cc.raw[1], 0.f));
    rec[3 * i + 2] = make_float4(fmaxf(cc.raw[2], 0.f), __uint_as_float(pack16(o.x0, o.y0)),
                                 __uint_as_float(pack16(o.x1, o.y1)), -logf(255.0f * op));
    const int tx0 = o.x0 / kTile, ty0 = o.y0 / kTile, tx1 = o.x1 / kTile, ty1 = o.y1 / kTile;
    rect[i] = make_uint2(pack16(tx0, ty0), pack16(tx1, ty1));
    if (count) count[i] = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
    key[i] = __float_as_uint(o.t[2]);
}

// ---------------------------------------------------------------------------
// radix64 ordering: one (tile << 32 | depth bits, index) pair per covered
// tile, in Gaussian order, then a 64-bit LSD sort and a boundary scan.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_emit(int64_t n, const uint32_t* __restrict__ key,
                                              const uint2* __restrict__ rect, const uint64_t* __restrict__ offs,
                                              int tiles_x, uint64_t cap, uint64_t* __restrict__ keys,
                                              uint32_t* __restrict__ vals) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t k = key[i];
    if (k == 0xFFFFFFFFu) return;
    const uint2 r = rect[i];
    const int tx0 = r.x & 0xFFFF, ty0 = r.x >> 16, tx1 = r.y & 0xFFFF, ty1 = r.y >> 16;
    uint64_t off = offs[i];
    for (int ty = ty0; ty <= ty1; ty++)
        for (int tx = tx0; tx <= tx1; tx++) {
            if (off < cap) {
                keys[off] = ((uint64_t)(ty * tiles_x + tx) << 32) | k;
                vals[off] = (uint32_t)i;
            }
            off++;
        }
}

__global__ __launch_bounds__(256) void k_gpos_from_pairs(const uint64_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ vals, int64_t K,
                                                         const uint2* __restrict__ rect,
                                                         const uint64_t* __restrict__ goff, int tiles_x, uint64_t cap,
                                                         uint32_t* __restrict__ gpos) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= K) return;
    const uint32_t id = vals[p];
    const uint32_t t = (uint32_t)(keys[p] >> 32);
    const int tx = (int)(t % (uint32_t)tiles_x), ty = (int)(t / (uint32_t)tiles_x);
    const uint2 r = rect[id];
    const int tx0 = r.x & 0xFFFF, ty0 = r.x >> 16, tx1 = r.y & 0xFFFF;
    const uint64_t k = goff[id] + (uint64_t)((ty - ty0) * (tx1 - tx0 + 1) + (tx - tx0));
    if (k < cap) gpos[k] = (uint32_t)p;
}

__global__ __launch_bounds__(256) void k_zero_ranges(uint2* ranges, int ntiles) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < ntiles) ranges[t] = make_uint2(0u, 0u);
}

__global__ __launch_bounds__(256) void k_ranges_from_keys(const uint64_t* __restrict__ keys, int64_t K,
                                                          uint2* __restrict__ ranges) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    const uint32_t t = (uint32_t)(keys[k] >> 32);
    if (k == 0 || (uint32_t)(keys[k - 1] >> 32) != t) ranges[t].x = (uint32_t)k;
    if (k == K - 1 || (uint32_t)(keys[k + 1] >> 32) != t) ranges[t].y = (uint32_t)(k + 1);
}

// ---------------------------------------------------------------------------
// depth-first ordering.  The Gaussians are first sorted by (depth bits,
// index) and their tile rectangles gathered into that order.  The sorted
// sequence is cut into chunks of kBinChunk.  A workgroup stages one chunk's
// rectangles in LDS; each of its waves owns one tile row.  Pass 1 counts
// pairs per (chunk, tile); an exclusive scan of the counts gives each
// (chunk, tile) segment its first slot; pass 2 lists the chunk's Gaussians
// spanning the row in depth order and writes, column by column, the indices
// of those covering the column at consecutive slots of the segment.  Inside
// a tile the result is ordered by (chunk, position in chunk), i.e. by
// (depth bits, index): the order a stable (tile, depth) sort gives.
// ---------------------------------------------------------------------------
#ifndef GS3_BIN_ROWS
#define GS3_BIN_ROWS 8
#endif
constexpr int kBinRowsPerBlock = GS3_BIN_ROWS;   // one wave per tile row
constexpr int kBinThreads = 64 * kBinRowsPerBlock;

// Workgroups are dealt round-robin to the eight XCDs (linear id mod 8), each
// with its own L2.  The binning passes give each XCD a contiguous eighth of
// the chunks of every row block, so the (tile, chunk) segments that follow
// each other in a tile's list (about a dozen entries each) are written
// through the same L2 and merge into whole lines there, instead of eight L2s
// writing back partial lines of each other's segments.  nchunks is a
// multiple of 8 (bin_chunks); the padding chunks are empty.
__device__ __forceinline__ void bin_block(int64_t nchunks, int& rowblock, int64_t& chunk) {
    const int64_t per = nchunks >> 3;
    const int64_t b = blockIdx.x;
    const int64_t k = b >> 3;
    rowblock = (int)(k / per);
    chunk = (b & 7) * per + k % per;
}

__global__ __launch_bounds__(256) void k_bin_gather(const uint32_t* __restrict__ order, int64_t n,
                                                    const uint2* __restrict__ rect, const uint32_t* __restrict__ count,
                                                    const uint64_t* __restrict__ goff, uint32_t cap,
                                                    uint2* __restrict__ srect, uint32_t* __restrict__ sgoff) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const uint32_t id = order[e];
    srect[e] = count[id] ? rect[id] : make_uint2(0xFFFF0000u, 0u);   // empty: no row spans
    const uint64_t go = goff[id];
    sgoff[e] = go < (uint64_t)cap ? (uint32_t)go : cap;
}

// Counting pass of the depth-first binning: for a tile row (one wave) and a
// chunk of depth-ordered Gaussians, how many of the chunk's Gaussians have a
// tile rectangle covering each tile of the row.  Every covering Gaussian
// adds +1 at its first column and -1 past its last to an LDS difference
// array; a prefix sum over the row's columns gives the counts (the same
// coverage test the scatter applies tile by tile).  The counts are stored
// chunk-major, so a wave writes its row as consecutive words.  A workgroup
// takes kCountGroup consecutive chunks of one row block.
constexpr int kCountGroup = 8;   // bin_chunks is a multiple of 8

__global__ __launch_bounds__(kBinThreads) void k_bin_count(const uint2* __restrict__ srect, int64_t n, int tiles_x,
                                                           int tiles_y, int64_t nchunks, uint32_t* __restrict__ hist) {
    const int64_t ntiles = (int64_t)tiles_x * tiles_y;
    __shared__ uint2 s_rect[kBinChunk];
    __shared__ int s_diff[kBinRowsPerBlock][kMaxTilesX + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t ngroups = nchunks / kCountGroup;
    const int64_t group = (int64_t)blockIdx.x % ngroups;
    const int rowblock = (int)((int64_t)blockIdx.x / ngroups);
    const int row = rowblock * kBinRowsPerBlock + w;
    for (int64_t chunk = group * kCountGroup; chunk < (group + 1) * kCountGroup; chunk++) {
        const int64_t e0 = chunk * kBinChunk;
        const int m = (int)min((int64_t)kBinChunk, n - e0);   // <= 0 for the padding chunks
        __syncthreads();   // the previous chunk's rectangles are no longer read
        for (int e = threadIdx.x; e < m; e += kBinThreads) s_rect[e] = srect[e0 + e];
        for (int k = lane; k <= kMaxTilesX; k += 64) s_diff[w][k] = 0;
        __syncthreads();
        if (row >= tiles_y) continue;
        for (int e = lane; e < m; e += 64) {
            const uint2 r = s_rect[e];
            if ((int)(r.x >> 16) <= row && row <= (int)(r.y >> 16)) {
                atomicAdd(&s_diff[w][r.x & 0xFFFFu], 1);
                atomicAdd(&s_diff[w][(r.y & 0xFFFFu) + 1u], -1);
            }
        }
        // the wave's atomics are done before its reads below (LDS operations of
        // one wave complete in order); lane l takes columns 4 l .. 4 l + 3
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int a[4];
        int t = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            t += s_diff[w][4 * lane + k];
            a[k] = t;
        }
        const int x = (int)wave_incl_scan_u32((uint32_t)t);   // inclusive scan of the lane totals
        const int pre = x - t;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int tx = 4 * lane + k;
            const uint32_t v = (uint32_t)(pre + a[k]);
            if (tx < tiles_x) hist[chunk * ntiles + (int64_t)row * tiles_x + tx] = v;
        }
    }
}

// Start slots of the tiles in the tile-major list: ranges[t] = [s, s + len)
// from the exclusive scan of the tile totals, clamped to cap.
// Tile-major exclusive prefix of the chunk-major counts.  A thread owns one
// tile and a segment of kBinScanSeg chunks, so every load and store of a
// warp-wide step touches consecutive tiles of one chunk: (1) segment sums,
// (2) per tile, the exclusive prefix over its segments and its total,
// (3) an exclusive scan of the tile totals (scan_u32_to_u64), (4) each
// segment's chunks walked again from the tile's and the segment's offset.
constexpr int kBinScanSeg = 32;

__global__ __launch_bounds__(256) void k_bin_scan_part(const uint32_t* __restrict__ hist, int64_t nchunks, int ntiles,
                                                       int64_t nseg, uint32_t* __restrict__ part) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= ntiles) return;
    for (int64_t sg = blockIdx.y; sg < nseg; sg += gridDim.y) {
        const int64_t c0 = sg * kBinScanSeg;
        const int64_t c1 = min(c0 + kBinScanSeg, nchunks);
        uint32_t s = 0u;
        for (int64_t c = c0; c < c1; c++) s += hist[c * ntiles + t];
        part[sg * ntiles + t] = s;
    }
}

__global__ __launch_bounds__(256) void k_bin_scan_tiles(uint32_t* __restrict__ part, int64_t nseg, int ntiles,
                                                        uint32_t* __restrict__ ttot) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= ntiles) return;
    uint32_t run = 0u;   // a tile holds at most one pair per Gaussian (< 2^31)
    for (int64_t sg = 0; sg < nseg; sg++) {
        const uint32_t v = part[sg * ntiles + t];
        part[sg * ntiles + t] = run;
        run += v;
    }
    ttot[t] = run;
}

__global__ __launch_bounds__(256) void k_bin_scan_base(const uint32_t* __restrict__ hist, int64_t nchunks, int ntiles,
                                                       int64_t nseg, const uint32_t* __restrict__ part,
                                                       const uint64_t* __restrict__ toff, uint32_t cap,
                                                       uint32_t* __restrict__ base) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= ntiles) return;
    for (int64_t sg = blockIdx.y; sg < nseg; sg += gridDim.y) {
        const int64_t c0 = sg * kBinScanSeg;
        const int64_t c1 = min(c0 + kBinScanSeg, nchunks);
        uint64_t run = toff[t] + part[sg * ntiles + t];
        for (int64_t c = c0; c < c1; c++) {
            base[c * ntiles + t] = run < (uint64_t)cap ? (uint32_t)run : cap;
            run += hist[c * ntiles + t];
        }
    }
}

// Scatter pass, one wave per (tile row, chunk of depth-ordered Gaussians):
// the wave lists the chunk's Gaussians whose rectangle spans its row, in
// depth order, and holds that list in registers, 64 Gaussians per group
// (lane = position in the group).  It then walks the row's columns: at
// column tx the Gaussians covering tx find their rank among the covering
// ones by a ballot and a masked bit count, and write their indices at
// consecutive slots from the (chunk, tile) segment's first slot.  One store
// instruction therefore fills one segment (about a dozen consecutive
// words) instead of touching a dozen tiles' lists, and every tile's entries
// keep the depth order.  The first slot of each (chunk, tile) segment comes
// from `base` in [chunk][tile] layout (clamped to cap).
constexpr int kBinGroups = kBinChunk / 64;   // register groups of the covering list
static_assert(kBinChunk % 64 == 0, "the covering list is held in groups of 64");

__global__ __launch_bounds__(kBinThreads) void k_bin_rows(const uint32_t* __restrict__ order, int64_t n,
                                                  const uint2* __restrict__ srect, const uint32_t* __restrict__ sgoff,
                                                  int tiles_x, int tiles_y, int64_t nchunks,
                                                  const uint32_t* __restrict__ base, uint32_t cap,
                                                  uint32_t* __restrict__ vals, uint32_t* __restrict__ gpos) {
    // A segment's slots start at min(first slot, cap) and run at most
    // kBinChunk past it, so with cap < 2^31 they never wrap; slots at or
    // past cap are not written.
    __shared__ uint2 s_rect[kBinChunk];
    __shared__ uint32_t s_id[kBinChunk];
    __shared__ uint32_t s_goff[kBinChunk];
    __shared__ uint32_t s_cov[kBinRowsPerBlock][kBinChunk];   // chunk positions of the row's covering Gaussians
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int rowblock;
    int64_t chunk;
    bin_block(nchunks, rowblock, chunk);
    const int row = rowblock * kBinRowsPerBlock + w;
    const int64_t e0 = chunk * kBinChunk;
    const int m = (int)min((int64_t)kBinChunk, n - e0);
    for (int e = threadIdx.x; e < m; e += kBinThreads) {
        s_id[e] = order[e0 + e];
        s_rect[e] = srect[e0 + e];
        s_goff[e] = sgoff[e0 + e];
    }
    __syncthreads();
    if (row >= tiles_y) return;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;   // lanes under this one
    // 1. the chunk's Gaussians spanning this row, in depth order
    int G = 0;
    for (int eb = 0; eb < m; eb += 64) {
        const int e = eb + lane;
        bool cov = false;
        if (e < m) {
            const uint2 r = s_rect[e];
            cov = (int)(r.x >> 16) <= row && row <= (int)(r.y >> 16);
        }
        const uint64_t bal = __ballot(cov);
        if (cov) s_cov[w][G + __popcll(bal & below)] = (uint32_t)e;
        G += __popcll(bal);
    }
    if (G == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // 2. the list in registers: column span, index and the slot of column 0
    // of this row in the Gaussian's own pair range
    int lo[kBinGroups], hi[kBinGroups];
    uint32_t gid[kBinGroups], gk[kBinGroups];
    int cmin = 1 << 30, cmax = -1;
#pragma unroll
    for (int gi = 0; gi < kBinGroups; gi++) {
        lo[gi] = 1 << 30;
        hi[gi] = -1;
        gid[gi] = 0u;
        gk[gi] = 0u;
        const int k = 64 * gi + lane;
        if (64 * gi < G && k < G) {
            const uint32_t e = s_cov[w][k];
            const uint2 r = s_rect[e];
            lo[gi] = (int)(r.x & 0xFFFFu);
            hi[gi] = (int)(r.y & 0xFFFFu);   // < tiles_x
            gid[gi] = s_id[e];
            gk[gi] = s_goff[e] + (uint32_t)(row - (int)(r.x >> 16)) * (uint32_t)(hi[gi] - lo[gi] + 1) -
                     (uint32_t)lo[gi];
            cmin = min(cmin, lo[gi]);
            cmax = max(cmax, hi[gi]);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        cmin = min(cmin, __shfl_xor(cmin, off));
        cmax = max(cmax, __shfl_xor(cmax, off));
    }
    cmin = __builtin_amdgcn_readfirstlane(cmin);
    cmax = __builtin_amdgcn_readfirstlane(cmax);
    const int ngr = (G + 63) >> 6;
    // 3. the columns the list covers; lane l of colb[cg] holds the first
    // slot of column 64 cg + l
    const uint32_t* brow = base + chunk * ((int64_t)tiles_x * tiles_y) + (int64_t)row * tiles_x;
    uint32_t colb[kMaxTilesX / 64];
#pragma unroll
    for (int cg = 0; cg < kMaxTilesX / 64; cg++) {
        const int tx = 64 * cg + lane;
        colb[cg] = (tx < tiles_x && cg * 64 <= cmax) ? min(brow[tx], cap) : cap;
    }
#pragma unroll
    for (int cg = 0; cg < kMaxTilesX / 64; cg++) {
        if (64 * cg > cmax) break;
        const int t0 = max(cmin, 64 * cg), t1 = min(cmax, 64 * cg + 63);
        for (int tx = t0; tx <= t1; tx++) {
            uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)colb[cg], tx - 64 * cg);
#pragma unroll
            for (int gi = 0; gi < kBinGroups; gi++) {
                if (gi >= ngr) break;
                const uint64_t bal =
                    __builtin_amdgcn_ballot_w64(lo[gi] <= tx) & __builtin_amdgcn_ballot_w64(tx <= hi[gi]);
                // rank among the covering lanes below this one
                const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                const uint32_t slot = pos + rank;
                if (__builtin_amdgcn_inverse_ballot_w64(bal) && slot < cap) {
                    vals[slot] = gid[gi];
                    const uint32_t kk = gk[gi] + (uint32_t)tx;
                    if (kk < cap) gpos[kk] = slot;
                }
                pos += (uint32_t)__popcll(bal);
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_ranges_from_hist(const uint32_t* __restrict__ base,
                                                          const uint64_t* __restrict__ total, int ntiles, uint64_t cap,
                                                          uint2* __restrict__ ranges, int* __restrict__ overflow) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    const uint64_t K = *total;
    if (t == 0 && K > cap) atomicOr(overflow, 1);
    if (t >= ntiles) return;
    // chunk 0's row of the bases: the first slot of every tile (clamped to cap)
    const uint32_t s = base[t];
    const uint32_t e = t + 1 < ntiles ? base[t + 1] : (uint32_t)(K < cap ? K : cap);
    ranges[t] = make_uint2(s, e);
}

// Longest-first tile schedule: tiles bucketed by the work they carry (list
// length for the forward, walked entries for the backward) on a half-octave
// scale, heaviest bucket first, so the long tiles start in the first wave of
// workgroups instead of trailing the launch.  One workgroup; the order inside
// a bucket is whatever the atomics give (it only affects scheduling).
__global__ __launch_bounds__(1024) void k_tile_order(const uint2* __restrict__ ranges,
                                                     const uint32_t* __restrict__ walk, int ntiles,
                                                     int* __restrict__ order) {
    __shared__ uint32_t cnt[kOrderBuckets], off[kOrderBuckets];
    for (int b = threadIdx.x; b < kOrderBuckets; b += blockDim.x) cnt[b] = 0u;
    __syncthreads();
    for (int t = threadIdx.x; t < ntiles; t += blockDim.x) {
        const uint32_t w = walk ? walk[t] : ranges[t].y - ranges[t].x;
        atomicAdd(&cnt[work_bucket(w)], 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0u;
        for (int b = kOrderBuckets - 1; b >= 0; b--) {
            off[b] = acc;
            acc += cnt[b];
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < ntiles; t += blockDim.x) {
        const uint32_t w = walk ? walk[t] : ranges[t].y - ranges[t].x;
        order[atomicAdd(&off[work_bucket(w)], 1u)] = t;
    }
}

// ---------------------------------------------------------------------------
// blend forward (Eq. 4): one workgroup per 16x16 tile, one pixel per thread;
// the tile's Gaussian records are staged through LDS 256 at a time.
//
// kSuper: the tile's entries are those of its super's list whose mask has the
// tile's bit.  The workgroup filters the list 256 entries at a time into a
// queue of indices in LDS (the next 256 masks and indices are loaded while
// the current batch is evaluated) and evaluates the queue in batches of 256
// (fewer at the end of the list).  Each batch's indices are kept in a walked
// block for the backward.  Otherwise the entries are vals[ranges[tile]).
//
// Bound by instruction issue where the launch fills the chip (300K uniform at 1352 x
// 1014: the vector ALUs in 0.69 of the cycles, and three scalar instructions for
// four of theirs) and by the latency of one wave's chain where it does not.  So a wave takes a square of 8 x 8
// pixels and evaluates only the staged entries that can reach it
// (quads_reached, a bit per entry and quadrant: at the benchmark scene less
// than half of the (wave, entry) visits of 16 x 4 pixels without the test),
// four at a time, since their exponents do not depend on each other (two at a
// time 0.5-3% slower, eight 2-4% slower on the large views).  Per launch,
// 16 x 4 pixels and every entry -> this: 300K uniform at 1352 x 1014 227 ->
// 139 us, 1M at 1920 x 1080 407 -> 228, 300K surfaces 298 -> 168, 50K
// surfaces at 256 x 256 486 -> 225, 2K at 64 x 64 129 -> 53 us.
// ---------------------------------------------------------------------------
constexpr int kFwdGroup = 4;   // entries whose exponents are evaluated together
template <bool kSuper>
__global__ __launch_bounds__(kBlendThreads, 7) void k_blend_fwd(CamDev cam, const uint2* __restrict__ ranges,
                                                             const uint32_t* __restrict__ vals,
                                                             const float4* __restrict__ rec, float* __restrict__ image,
                                                             float* __restrict__ T_final, uint32_t* __restrict__ last_out,
                                                             uint32_t* __restrict__ tile_walk,
                                                             const int* __restrict__ order,
                                                             uint64_t* __restrict__ taken, SuperDev sd, int nsuper) {
    constexpr int NT = kBlendThreads, NW = NT / 64;
    static_assert(kWalkBlock == NT, "a walked block holds one batch");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int tx, ty, tile, sup = 0;
    if (kSuper) {
        // the tiles of a super on one XCD (workgroup b runs on XCD b mod 8):
        // they read the same list and mostly the same records
        constexpr int T = kSuperDim * kSuperDim;
        const int x = blockIdx.x & 7, k = blockIdx.x >> 3;
        const int place = (k / T) * 8 + x, local = k % T;
        if (place >= nsuper) return;
        sup = order[place];
        tx = (sup % sd.supers_x) * kSuperDim + local % kSuperDim;
        ty = (sup / sd.supers_x) * kSuperDim + local / kSuperDim;
        if (tx >= cam.tiles_x || ty >= cam.tiles_y) return;
        tile = ty * cam.tiles_x + tx;
    } else {
        tile = order[blockIdx.x];
        tx = tile % cam.tiles_x;
        ty = tile / cam.tiles_x;
    }
    __shared__ uint32_t s_walk;
    __shared__ float4 s_w0[NT];
    __shared__ float4 s_w1[NT];
    __shared__ float4 s_w2[NT];   // blend_stage_w2 form
    __shared__ uint32_t s_q[kSuper ? 2 * NT : 1];   // queue of indices
    __shared__ uint32_t s_n[2][NW];                 // entries each wave adds to it
    __shared__ uint64_t s_reach[NW][NW];            // [quadrant][word]: staged entries that can reach its pixels
    __shared__ uint64_t s_taken[NW][NW];            // [word][quadrant]: entries a pixel of the quadrant took
    __shared__ uint32_t s_live[NW], s_blk;           // bit 0: pixels left, bit 1: took an entry of the batch
    __shared__ uint64_t s_over[NW];                 // [word]: staged entries with an infinite colour
    const int tx0p = tx * kTile, ty0p = ty * kTile;
    // wave w: the 8 x 8 quadrant (w & 1, w >> 1) of the tile
    const int lx = quad_x(w, lane), ly = quad_y(w, lane);
    const int px = tx0p + lx, py = ty0p + ly;
    const float fpx = (float)px, fpy = (float)py;
    const uint32_t sel = (1u << lx) | (1u << (16 + ly));   // column and row bits in the box masks
    float T = 1.0f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
    uint32_t last = 0u;
    // lanes whose pixel is in the image and has not stopped
    uint64_t alive = __builtin_amdgcn_ballot_w64(px < cam.W && py < cam.H);
    if (tid == 0) s_walk = 0u;
    // list cursor: the super's entries [c, cend) are not filtered yet; mk, id
    // hold this thread's entry c + tid
    uint32_t c = 0u, cend = 0u, mk = 0u, nid = 0u;
    uint32_t queued = 0u;
    int par = 0;
    uint32_t tbit = 0u;
    if (kSuper) {
        c = sd.start[sup];
        cend = min(sd.cap, c + sd.len[sup]);
        tbit = 1u << ((ty % kSuperDim) * kSuperDim + tx % kSuperDim);
        if (c + tid < cend) {
            mk = sd.masks[c + tid];
            nid = sd.ids[c + tid];
        }
    } else {
        const uint2 rg = ranges[tile];
        c = rg.x;
        cend = rg.y;
    }
    uint32_t blk = (uint32_t)tile, lastblk = (uint32_t)tile;   // walked blocks
    for (uint32_t eb = 0;;) {   // eb: entries staged so far
        uint32_t myid = 0u;
        uint32_t cnt_u;
        int64_t word = 0;   // first word of the batch in `taken` (kSuper: the block's, known later)
        if (kSuper) {
            while (queued < (uint32_t)NT && c < cend) {
                const bool on = (mk & tbit) != 0u && c + tid < cend;
                const uint64_t bal = __ballot(on);
                if (lane == 0) s_n[par][w] = (uint32_t)__popcll(bal);
                __syncthreads();
                uint32_t at = queued + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
#pragma unroll
                for (int k = 0; k < NW; k++) {
                    if (k < w) at += s_n[par][k];
                    queued += s_n[par][k];
                }
                if (on) s_q[at] = nid;   // at < NT - 1 + NT
                par ^= 1;
                c += NT;
                if (c + tid < cend) {
                    mk = sd.masks[c + tid];
                    nid = sd.ids[c + tid];
                }
            }
            if (queued == 0u) break;
            cnt_u = min((uint32_t)NT, queued);
            __syncthreads();
            if ((uint32_t)tid < cnt_u) myid = s_q[tid];
        } else {
            if (c >= cend) break;
            cnt_u = min((uint32_t)NT, cend - c);
            if ((uint32_t)tid < cnt_u) myid = vals[c + tid];
            word = taken_word(ranges[tile].x, tile) + (eb >> 6);
            c += cnt_u;
        }
        uint32_t reach = 0u;   // quadrants this thread's entry can reach
        bool over = false;
        if ((uint32_t)tid < cnt_u) {
            const float4 r0 = rec[3 * (int64_t)myid + 0], r1 = rec[3 * (int64_t)myid + 1];
            const float4 r2 = rec[3 * (int64_t)myid + 2];
            s_w0[tid] = r0;
            s_w1[tid] = r1;
            s_w2[tid] = blend_stage_w2(r2, tx0p, ty0p);
            reach = quads_reached(r0, r1, r2, tx0p, ty0p);
            over = colour_overflows(r1, r2);
        }
        const uint64_t overb = __builtin_amdgcn_ballot_w64(over);
        if (lane == 0) s_over[w] = overb;
#pragma unroll
        for (int q = 0; q < NW; q++) {
            const uint64_t b = __builtin_amdgcn_ballot_w64((reach >> q) & 1u);
            if (lane == 0) s_reach[q][w] = b;
        }
        uint32_t rest = 0u;   // the queue's entries past this batch move to its front
        if (kSuper && (uint32_t)tid + NT < queued) rest = s_q[NT + tid];
        __syncthreads();
        if (kSuper) {
            if ((uint32_t)tid + NT < queued) s_q[tid] = rest;
            queued -= cnt_u;
            // a block for this batch (the first is the tile's own); the
            // answer is needed only after the evaluation
            if (tid == 0 && eb != 0u) blk = atomicAdd(sd.pool, 1u);
        }
        uint64_t tk = 0ull;   // the word's entries a pixel of the wave takes
        {
            // branch-free per-pixel body over a group of entries: the
            // exponents and opacities of the group are independent of each
            // other, so their latencies overlap; only the transmittance
            // passes from entry to entry.  Every lane evaluates, lane masks
            // (wave-uniform) keep the state of pixels that do not take the
            // contribution.
            auto eval = [&](auto G, const int* j, int& tj) {
                constexpr int kG = decltype(G)::value;
                float power[kG], alpha[kG];
                float4 w1[kG];
                float cb[kG];
                uint64_t okm[kG], bm[kG];
                uint64_t any = 0ull, band = 0ull;
#pragma unroll
                for (int i = 0; i < kG; i++) {
                    const float4 w0 = s_w0[j[i]], w2 = s_w2[j[i]];
                    w1[i] = s_w1[j[i]];
                    cb[i] = w2.x;
                    const uint32_t box = __float_as_uint(w2.w);
                    float adx2, bdx;
                    blend_dx_terms(fpx - w0.x, w0, adx2, bdx);
                    power[i] = blend_power(adx2, bdx, fpy - w0.y, w1[i].x);
                    // pixels inside the exponent band at w2.y..w2.z take the exact test
                    const uint64_t pm = alive & __builtin_amdgcn_ballot_w64((box & sel) == sel) &
                                        __builtin_amdgcn_ballot_w64(power[i] <= 0.0f) &
                                        __builtin_amdgcn_ballot_w64(power[i] >= w2.y);
                    bm[i] = pm & __builtin_amdgcn_ballot_w64(power[i] < w2.z);
                    okm[i] = pm & ~bm[i];
                    any |= pm;
                    band |= bm[i];
                }
                if (band) {
#pragma unroll
                    for (int i = 0; i < kG; i++)
                        okm[i] |= bm[i] & __builtin_amdgcn_ballot_w64(blend_exact_test(power[i], w1[i].y));
                }
                if (!any) return;   // no pixel of the wave takes an entry: nothing changes
#pragma unroll
                for (int i = 0; i < kG; i++) alpha[i] = fminf(0.99f, w1[i].y * __expf(power[i]));
#pragma unroll
                for (int i = 0; i < kG; i++) {
                    const float Tn = T * (1.0f - alpha[i]);
                    const uint64_t ok = okm[i] & alive;   // a pixel may have stopped inside the group
                    const uint64_t stop = ok & __builtin_amdgcn_ballot_w64(Tn < 1e-4f);
                    const bool take = __builtin_amdgcn_inverse_ballot_w64(ok & ~stop);
                    tj = (ok & ~stop) != 0ull ? j[i] & 63 : tj;
                    set_bit(tk, tj);
                    alive &= ~stop;
                    const float wgt = take ? alpha[i] * T : 0.0f;
                    // an entry by itself may have an infinite colour, which weight zero does not take away
                    const float n0 = c0 + wgt * w1[i].z, n1 = c1 + wgt * w1[i].w, n2 = c2 + wgt * cb[i];
                    c0 = kG > 1 || take ? n0 : c0;
                    c1 = kG > 1 || take ? n1 : c1;
                    c2 = kG > 1 || take ? n2 : c2;
                    T = take ? Tn : T;
                    last = take ? eb + (uint32_t)j[i] + 1u : last;
                }
            };
            // the entries that can reach the wave's pixels, in order; the
            // wave leaves once all its pixels have stopped.  One by one where
            // an infinite colour is among them
#pragma unroll 1
            for (int q = 0; q < NW; q++) {
                tk = 0ull;
                uint64_t m = uniform64(alive ? s_reach[w][q] : 0ull);
                const int group = (m & uniform64(s_over[q])) ? NT : kFwdGroup;
                // the last entry taken; until there is one, the first visited
                // (a bit too many costs the backward a visit)
                int tj = __builtin_ctzll(m | (1ull << 63));
                auto next = [&]() {
                    const int b = __builtin_ctzll(m);
                    clear_bit(m, b);
                    return 64 * q + b;
                };
                int left = __popcll(m);
#pragma unroll 1
                for (; left >= group && alive; left -= kFwdGroup) {
                    int j[kFwdGroup];
#pragma unroll
                    for (int i = 0; i < kFwdGroup; i++) j[i] = next();
                    eval(std::integral_constant<int, kFwdGroup>{}, j, tj);
                }
#pragma unroll 1
                for (; left > 0 && alive; left--) {
                    const int j[1] = {next()};
                    eval(std::integral_constant<int, 1>{}, j, tj);
                }
                if (lane == 0) s_taken[q][w] = tk;
            }
        }
        const uint64_t took = __builtin_amdgcn_ballot_w64(last > eb);
        if (lane == 0) s_live[w] = (alive != 0ull ? 1u : 0u) | (took != 0ull ? 2u : 0u);
        if (kSuper && tid == 0) {
            if (blk >= sd.max_blocks) blk = 0xFFFFFFFFu;   // only when the pairs overflowed
            if (eb != 0u && blk != 0xFFFFFFFFu) sd.prev[blk] = s_blk;
            s_blk = blk;
        }
        __syncthreads();
        bool keep = true;   // the batch's taken bits have a place
        if (kSuper) {
            const uint32_t b = s_blk;
            keep = b != 0xFFFFFFFFu;
            if ((uint32_t)tid < cnt_u && keep) sd.walked[(int64_t)b * kWalkBlock + tid] = myid;
            word = (int64_t)b * (kWalkBlock / 64);
        }
        // a tile-major list's words past the tile's last entry are another tile's
        if (keep && tid < NW * NW && 64u * (tid / NW) < cnt_u)
            taken[(word + tid / NW) * NW + tid % NW] = s_taken[tid / NW][tid % NW];
        const uint32_t state = s_live[0] | s_live[1] | s_live[2] | s_live[3];
        if (kSuper && (state & 2u)) lastblk = s_blk;   // the last contributor's so far
        eb += cnt_u;
        if (!(state & 1u)) break;
    }
    const int64_t P = (int64_t)cam.W * cam.H;
    if (px < cam.W && py < cam.H) {
        const int64_t p = (int64_t)py * cam.W + px;
        image[p] = c0 + T * cam.bg[0];
        image[P + p] = c1 + T * cam.bg[1];
        image[2 * P + p] = c2 + T * cam.bg[2];
        T_final[p] = T;
        last_out[p] = last;
    }
    __syncthreads();
    if (last) atomicMax(&s_walk, last);
    __syncthreads();
    if (tid == 0) {
        // no block to walk back through: the backward skips the tile (the
        // pairs overflowed, which the render reports)
        const bool lost = kSuper && lastblk == 0xFFFFFFFFu;
        tile_walk[tile] = lost ? 0u : s_walk;
        if (kSuper) sd.tile_blk[tile] = lost ? (uint32_t)tile : lastblk;
    }
}

// ---------------------------------------------------------------------------
// blend backward: walk the tile list from the last contributor of any pixel
// down to the first, recover T_i = T_{i+1} / (1 - alpha_i), keep the colour
// accumulated behind each contributor, sum each Gaussian's nine gradient
// terms over a wave's pixels (reduce-scatter), then over the tile's waves in
// LDS, before one global atomic per term and tile.
//
// Bound by VALU issue on large views (0.95 of the cycles, 300K uniform at 1352 x
// 1014).  Each wave has the forward's 8 x 8
// quadrant and visits exactly the entries of which the forward noted that a
// pixel of the quadrant took them (`taken`, a bit per entry and quadrant), so
// next to no visit is in vain; kBwdGroup entries are evaluated together
// (their exponents, opacities and reciprocals do not depend on each other;
// the transmittance and the colour behind pass from entry to entry).  Four
// together gain 2-3% where one wave has a SIMD to itself and lose 1-2% on the
// large views.  Per launch, 16 x 4 pixels with per-wave box tests -> this:
// 300K uniform at 1352 x 1014 259 -> 214 us, 1M at 1920 x 1080 442 -> 355,
// 502K surfaces (opacity too) 444 -> 297, 50K surfaces at 256 x 256 619 ->
// 331, 2K at 64 x 64 161 -> 95 us.
// ---------------------------------------------------------------------------
// kRecords: write each walked entry's nine sums to the compact record buffer
// (fixed summation order; gathered per Gaussian by the preprocess backward),
// atomics only past its capacity; otherwise one global atomic per term and
// (tile, Gaussian).  kOpacity: also reduce the opacity term.
// factors of the nine reduced terms: the conic terms are summed as dx^2,
// dx dy and dy^2 (powers of two: the scaling is exact)
constexpr int kBwdBatch = 128;   // entries staged per batch (LDS: about 200 B each)
constexpr int kBwdGroup = 2;     // entries evaluated and reduced together
static_assert(kBwdGroup % 2 == 0, "entries are reduced two at a time");
__constant__ float kConicScale[9] = {1.f, 1.f, -0.5f, -1.f, -0.5f, 1.f, 1.f, 1.f, 1.f};

// A batch's sums of the waves (s_g, [wave][term][entry]; on: the entries each
// wave visited, [word][wave]): out(entry, term, sum).  A lane has one term of an entry
// throughout and a wave seven entries at a time, so the rounds need no
// divisions, a round's LDS reads are independent, and an entry's nine atomics
// are adjacent lanes on adjacent addresses (one or two cache lines).  The mean
// terms come from the sums of dp dx and dp dy (the neighbouring lane's) and
// the entry's conic (A, B, C).  Against a division, the wave masks one by one
// and a branch for the mean terms in every round, the whole backward went from
// 156 to 128 us at 50K Gaussians and 256 x 256, from 220 to 208 at 300K and
// 1352 x 1014, from 295 to 288 at 502K and 1080p (rounds unrolled: 214 and
// 305, for the registers); the narrow backward with records from 54 to 52 at 5K
// and 200 x 152.
template <int NW, int KB, bool kOpacity, class Conic, class Out>
__device__ __forceinline__ void sum_batch(int cnt, int w, int lane, const uint64_t (&on)[2][NW],
                                          const float (&s_g)[NW][9][KB + 1], Conic conic, Out out) {
    constexpr int kPer = 7, kRounds = (KB + kPer * NW - 1) / (kPer * NW);
    const int l = min(lane, 62) / 9, k = min(lane, 62) - 9 * l;
    const bool none = !kOpacity && k == 5;
    const float scale = kConicScale[k];
    const int other = k == 0 ? lane + 1 : k == 1 ? lane - 1 : lane;
#pragma unroll 1
    for (int i = 0; i < kRounds; i++) {
        if (kPer * NW * i >= cnt) break;
        const int e0 = (i * NW + w) * kPer + l, e = min(e0, KB - 1);
        const uint32_t* words = reinterpret_cast<const uint32_t*>(&on[e >> 6][0]) + ((e >> 5) & 1);
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < NW; q++) {
            const float g = s_g[q][k][e];
            v += (words[2 * q] >> (e & 31)) & 1u ? g : 0.f;
        }
        const float o = __shfl(v, other);
        const float3 c = conic(e);
        const float m = c.y * o + (k == 0 ? c.x : c.z) * v;
        v = none ? 0.f : k <= 1 ? m : v * scale;
        if (lane < 63 && e0 < cnt) out(e, k, v);
    }
}

template <bool kSuper, bool kRecords, bool kOpacity>
__global__ __launch_bounds__(kBlendThreads) void k_blend_bwd(CamDev cam, const uint2* __restrict__ ranges,
                                                             const uint32_t* __restrict__ vals,
                                                             const float4* __restrict__ rec,
                                                             const float* __restrict__ d_image,
                                                             const float* __restrict__ T_final,
                                                             const uint32_t* __restrict__ last_in,
                                                             const uint32_t* __restrict__ tile_walk,
                                                             const uint32_t* __restrict__ walk_off,
                                                             float* __restrict__ grec, uint32_t grec_cap,
                                                             float* __restrict__ accum, const int* __restrict__ order,
                                                             const uint64_t* __restrict__ taken, SuperDev sd) {
    constexpr int NT = kBlendThreads, NW = NT / 64;
    constexpr int KB = kBwdBatch;
    static_assert(KB == 128, "two mask words per batch");
    static_assert(kWalkBlock % KB == 0, "a batch lies in one walked block");
    __shared__ float4 s_w0[KB];
    __shared__ float4 s_w1[KB];
    __shared__ float4 s_w2[KB];   // blend_stage_w2 form
    __shared__ uint32_t s_id[KB];
    __shared__ uint64_t s_taken[2][NW];    // the batch's taken bits, [word][quadrant]
    __shared__ uint32_t s_over[2];         // colours of the batch that have overflowed
    __shared__ float s_g[NW][9][KB + 1];   // per-wave sums, [wave][term][entry] (padded: term rows on distinct banks)
    const int tile = order[blockIdx.x];
    const uint32_t maxlast = tile_walk[tile];
    if (maxlast == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    const int tx0p = tx * kTile, ty0p = ty * kTile;
    const int lx = quad_x(w, lane), ly = quad_y(w, lane);
    const int px = tx0p + lx, py = ty0p + ly;
    const float fpx = (float)px, fpy = (float)py;
    const uint32_t sel = (1u << lx) | (1u << (16 + ly));   // column and row bits in the box masks
    // kSuper: the block holding the batch (the forward's tile_blk, then prev)
    const uint32_t start = kSuper ? 0u : ranges[tile].x;
    uint32_t blk = kSuper ? sd.tile_blk[tile] : 0u;
    const uint32_t woff = kRecords ? walk_off[tile] : 0u;
    const int64_t P = (int64_t)cam.W * cam.H;
    // gb: dL/dC . (colour behind the current contributor), the only use of
    // that colour (dL/dalpha_i = T_i (dL/dC . c_i - gb)); it starts at the
    // background and moves to alpha c + (1 - alpha) b past each contributor
    float T = 1.0f, g0 = 0.f, g1 = 0.f, g2 = 0.f;
    uint32_t last = 0u;
    if (px < cam.W && py < cam.H) {
        const int64_t p = (int64_t)py * cam.W + px;
        T = T_final[p];
        last = last_in[p];
        g0 = d_image[p];
        g1 = d_image[P + p];
        g2 = d_image[2 * P + p];
    }
    float gb = g0 * cam.bg[0] + g1 * cam.bg[1] + g2 * cam.bg[2];
    // reduce-scatter terms: the image-space mean terms summed as dp dx and
    // dp dy (the conic is applied to the sums per entry), the conic terms,
    // r, g, b; lane group (lane >> 3) holds term (lane >> 3)
    const int my_term = lane >> 3;
    const int my_slot = my_term < 5 ? my_term : my_term + 1;   // index in the nine-term layout
    for (int64_t jb = ((int64_t)(maxlast - 1) / KB) * KB; jb >= 0; jb -= KB) {
        const uint32_t e = (uint32_t)jb + tid;
        bool over = false;
        if (tid < KB && e < maxlast) {
            const uint32_t id = kSuper ? sd.walked[(int64_t)blk * kWalkBlock + (e % kWalkBlock)] : vals[start + e];
            const float4 r0 = rec[3 * (int64_t)id + 0], r1 = rec[3 * (int64_t)id + 1], r2 = rec[3 * (int64_t)id + 2];
            s_id[tid] = id;
            s_w0[tid] = r0;
            s_w1[tid] = r1;
            s_w2[tid] = blend_stage_w2(r2, tx0p, ty0p);
            over = colour_overflows(r1, r2);
        }
        const uint64_t overb = __builtin_amdgcn_ballot_w64(over);
        if (lane == 0 && w < 2) s_over[w] = overb != 0ull ? 1u : 0u;
        if (tid >= KB && tid < KB + 2 * NW) {
            const int t = tid - KB, wd = t / NW;
            const int64_t word = (kSuper ? (int64_t)blk * (kWalkBlock / 64) + ((jb % kWalkBlock) >> 6)
                                         : taken_word(start, tile) + (jb >> 6)) + wd;
            // entries past the last contributor are not staged: the forward's
            // bit for an entry it visited before any was taken may lie there
            const int64_t left = (int64_t)maxlast - jb - 64 * wd;
            const uint64_t some = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1ull : 0ull;
            s_taken[wd][t % NW] = some ? taken[word * NW + t % NW] & some : 0ull;
        }
        if (kSuper && jb > 0 && jb % kWalkBlock == 0) blk = sd.prev[blk];
        __syncthreads();
        const int cnt = (int)min((int64_t)KB, (int64_t)maxlast - jb);
        // kG entries, last first: this thread's pixel walks back past them
        // (its transmittance and behind-colour state), and their eight terms
        // are summed over the wave
        auto walk = [&](auto G, const int* j) {
            constexpr int kG = decltype(G)::value;
            float power[kG], dx[kG], dy[kG], G_[kG], raw[kG], inv[kG], cb[kG];
            float4 w1[kG];
            // lane masks (wave-uniform): okm the lanes whose pixel takes the
            // entry, bm those whose exponent lies in the band where the exact
            // test decides
            uint64_t okm[kG], bm[kG], band = 0ull;
#pragma unroll
            for (int i = 0; i < kG; i++) {
                const float4 w0 = s_w0[j[i]], w2 = s_w2[j[i]];
                w1[i] = s_w1[j[i]];
                cb[i] = w2.x;
                const uint32_t box = __float_as_uint(w2.w);
                dx[i] = fpx - w0.x;
                dy[i] = fpy - w0.y;
                float adx2, bdx;
                blend_dx_terms(dx[i], w0, adx2, bdx);
                power[i] = blend_power(adx2, bdx, dy[i], w1[i].x);
                const uint64_t pm = __builtin_amdgcn_ballot_w64((uint32_t)jb + (uint32_t)j[i] < last) &
                                    __builtin_amdgcn_ballot_w64((box & sel) == sel) &
                                    __builtin_amdgcn_ballot_w64(power[i] <= 0.0f) &
                                    __builtin_amdgcn_ballot_w64(power[i] >= w2.y);
                bm[i] = pm & __builtin_amdgcn_ballot_w64(power[i] < w2.z);
                okm[i] = pm & ~bm[i];
                band |= bm[i];
            }
            if (band) {
#pragma unroll
                for (int i = 0; i < kG; i++)
                    okm[i] |= bm[i] & __builtin_amdgcn_ballot_w64(blend_exact_test(power[i], w1[i].y));
            }
#pragma unroll
            for (int i = 0; i < kG; i++) {
                G_[i] = __expf(power[i]);
                raw[i] = w1[i].y * G_[i];
                // T recovery T_i = T_{i+1} / (1 - alpha_i), with the hardware reciprocal (1 ulp)
                inv[i] = __builtin_amdgcn_rcpf(1.0f - fminf(0.99f, raw[i]));
            }
            float gr[kG][8], gop[kG];
#pragma unroll
            for (int i = 0; i < kG; i++) {
                // branch-free: selects keep the state of pixels that this
                // Gaussian does not reach
                const bool ok = __builtin_amdgcn_inverse_ballot_w64(okm[i]);
                T = ok ? T * inv[i] : T;
                const float aok = ok ? fminf(0.99f, raw[i]) : 0.0f;   // zero: the pixel's state is kept
                const float wgt = aok * T;
                const float d = (g0 * w1[i].z + g1 * w1[i].w + g2 * cb[i]) - gb;
                const float dal = T * d;
                const float gn = gb + aok * d;
                gb = kG > 1 || ok ? gn : gb;   // see the forward: opacity zero does not take an infinite colour away
                const bool unclamped =
                    __builtin_amdgcn_inverse_ballot_w64(okm[i] & __builtin_amdgcn_ballot_w64(raw[i] < 0.99f));
                const float dp = unclamped ? dal * raw[i] : 0.0f;
                gop[i] = unclamped ? dal * G_[i] : 0.0f;
                // d power / d(u, v) = (A dx + B dy, B dx + C dy): the sums of
                // dp dx and dp dy take A, B, C after the reduction; the conic
                // terms -dx^2 / 2, -dx dy, -dy^2 / 2 get their constant
                // factors there too (kConicScale)
                const float ax = dp * dx[i], ay = dp * dy[i];
                gr[i][0] = ax;
                gr[i][1] = ay;
                gr[i][2] = ax * dx[i];
                gr[i][3] = ax * dy[i];
                gr[i][4] = ay * dy[i];
                gr[i][5] = g0 * wgt;
                gr[i][6] = g1 * wgt;
                gr[i][7] = g2 * wgt;
            }
            float red[kG];
            if constexpr (kG == 1) {
                red[0] = wave_reduce_scatter8(gr[0], lane);
            } else {
#pragma unroll
                for (int i = 0; i < kG; i += 2) wave_reduce_scatter8x2(gr[i], gr[i + 1], lane, red[i], red[i + 1]);
            }
            if ((lane & 7) == 0) {
#pragma unroll
                for (int i = 0; i < kG; i++) s_g[w][my_slot][j[i]] = red[i];
            }
            if (kOpacity) {
#pragma unroll
                for (int i = 0; i < kG; i++) {
                    const float o = wave_sum_dpp(gop[i]);
                    if (lane == 8) s_g[w][5][j[i]] = o;
                }
            }
        };
        const int group = __builtin_amdgcn_readfirstlane(s_over[0] | s_over[1]) ? KB : kBwdGroup;
#pragma unroll 1
        for (int wd = 1; wd >= 0; wd--) {
            uint64_t m = uniform64(s_taken[wd][w]);
            auto next = [&]() {
                const int b = 63 - __builtin_clzll(m);
                clear_bit(m, b);
                return 64 * wd + b;
            };
            int left = __popcll(m);
#pragma unroll 1
            for (; left >= group; left -= kBwdGroup) {
                int j[kBwdGroup];
#pragma unroll
                for (int i = 0; i < kBwdGroup; i++) j[i] = next();
                walk(std::integral_constant<int, kBwdGroup>{}, j);
            }
#pragma unroll 1
            for (; left > 0; left--) {
                const int j[1] = {next()};
                walk(std::integral_constant<int, 1>{}, j);
            }
        }
        __syncthreads();
        // term k of entry e summed over the waves that took it
        auto over_waves = [&](int k, int e, uint32_t on) -> float {
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < NW; q++) v += (on >> q) & 1u ? s_g[q][k][e] : 0.f;
            return v;
        };
        auto taken_by = [&](int e) -> uint32_t {
            uint32_t on = 0u;
#pragma unroll
            for (int q = 0; q < NW; q++) on |= (uint32_t)((s_taken[e >> 6][q] >> (e & 63)) & 1ull) << q;
            return on;
        };
        // the mean terms from the sums of dp dx and dp dy and the entry's conic (A, B, C)
        auto entry_term = [&](int k, int e, uint32_t on) -> float {
            const float v = over_waves(k, e, on);
            if (k <= 1) {
                const float o = over_waves(1 - k, e, on);
                const float4 w0 = s_w0[e];
                const float C = s_w1[e].x;
                return k == 0 ? w0.z * v + w0.w * o : w0.w * o + C * v;
            }
            return v * kConicScale[k];
        };
        if (kRecords) {
            if (tid < cnt) {
                const uint32_t widx = woff + (uint32_t)jb + tid;   // compact index of this walked entry
                const bool fits = widx < grec_cap;
                const uint32_t on = taken_by(tid);
#pragma unroll
                for (int k = 0; k < 9; k++) {
                    if (!kOpacity && k == 5) {
                        if (fits) grec[(int64_t)k * grec_cap + widx] = 0.f;
                        continue;
                    }
                    const float v = entry_term(k, tid, on);
                    if (fits)
                        grec[(int64_t)k * grec_cap + widx] = v;
                    else if (v != 0.f)
                        atomicAdd(accum + 9 * (int64_t)s_id[tid] + k, v);
                }
            }
        } else {
            sum_batch<NW, KB, kOpacity>(
                cnt, w, lane, s_taken, s_g, [&](int e) { return make_float3(s_w0[e].z, s_w0[e].w, s_w1[e].x); },
                [&](int e, int k, float v) {
                    if (v != 0.f) atomicAdd(accum + 9 * (int64_t)s_id[e] + k, v);
                });
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Narrow blends, for views of few tiles.  With a tile or two to a CU, the
// 8 x 8 blends above leave one wave or two to a SIMD and run at the latency of
// its chain, entry after entry.  Here a tile has 16 waves: a wave takes a block of
// 4 x 4 pixels, and its four 16-lane rows evaluate four entries (slots) at a
// time, one entry to a row, each lane one pixel of it.  The opacities of the
// four slots are then exchanged between the rows (permlane swaps), and every
// row walks the four in order for the transmittance, so the results are the
// same as entry by entry.  A block of 16 pixels is reached by half as many
// entries as a quadrant of 64 where the Gaussians are small, and the
// exponents, tests and gradient terms of four entries cost one evaluation.
// A workgroup takes a quarter of a tile (8 x 8 pixels, four waves), so that
// the longest tile, which bounds such launches, is spread over four CUs: at 50K
// surfaces and 256 x 256 a tile walks 388 entries on average and 2742 at most.
// The quarters read tile-major lists (k_super_lists writes them for views of
// few tiles) and stop each by itself.  Only the backward with gradient records
// keeps a tile to a workgroup, for a record holds the whole tile's sums.  What
// is left is the latency of the longest quarter's one wave per SIMD.  Per
// launch, 8 x 8 pixels a wave -> a workgroup a tile -> a quarter, 50K surfaces
// at 256 x 256: forward 226 -> 118 -> 82 us (and 8 for the lists), backward 331
// -> 196 -> 128; 2K uniform at 64 x 64: 54 -> 32 -> 20 (and 5), 95 -> 55 -> 33.
// Where they are chosen: narrow_tiles.
// ---------------------------------------------------------------------------
constexpr int kNarrowThreads = 1024;    // a workgroup a tile: a wave per 4 x 4 block, block w at (w & 3, w >> 2)
constexpr int kQuarterThreads = 256;    // a workgroup a quarter, four blocks
constexpr int kQuarterWaves = kQuarterThreads / 64;
constexpr int kSlots = 4;
__device__ __forceinline__ int quarter_block(int quarter, int w) {
    return (2 * (quarter >> 1) + (w >> 1)) * 4 + 2 * (quarter & 1) + (w & 1);
}

// x of the four rows (slots) of a wave, each in every row: s[k] holds, in lane
// l, the value of lane 16 k + (l & 15).
__device__ __forceinline__ void rows_all(float x, float s[kSlots]) {
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));   // rows 0 1 0 1, rows 2 3 2 3
    float a1 = a, b1 = b;
    asm volatile(
        "s_nop 1\n\t"
        "v_permlane16_swap_b32 %0, %1\n\t"
        "v_permlane16_swap_b32 %2, %3"
        : "+v"(a), "+v"(a1), "+v"(b), "+v"(b1));
    s[0] = a;
    s[1] = a1;
    s[2] = b;
    s[3] = b1;
}

// Eight values per lane -> their sums over each row of 16 lanes: afterwards
// lane i of the row holds the sum of term row_term(i).
__device__ __forceinline__ int row_term(int i) { return ((i >> 3) & 1) * 4 + ((i >> 2) & 1) * 2 + ((i >> 1) & 1); }
template <int kCtrl>
__device__ __forceinline__ float row_halve(float lo, float hi, bool up) {
    const float keep = up ? hi : lo, send = up ? lo : hi;
    return keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), kCtrl, 0xF,
                                                                        0xF, false));
}
__device__ __forceinline__ float row_reduce_scatter8(const float v[8], int i) {
    float a[4], b[2];
#pragma unroll
    for (int k = 0; k < 4; k++) a[k] = row_halve<0x128>(v[k], v[4 + k], i & 8);        // row_ror:8, lane i ^ 8
#pragma unroll
    for (int k = 0; k < 2; k++) b[k] = row_halve<0x141>(a[k], a[2 + k], i & 4);        // row_half_mirror, lane i ^ 7
    const float c = row_halve<0x4E>(b[0], b[1], i & 2);                                // quad_perm [2,3,0,1]
    return dpp_add<0xB1, 0xF>(c);                                                      // quad_perm [1,0,3,2]
}

// Whether an entry in LDS form (s_a, s_b of the narrow blends, box mask) can
// reach 4 x 4 block b of the tile: quads_reached for a block.
__device__ __forceinline__ bool block_reached(const float4& a, const float4& b, uint32_t box, int blk, int tx0p, int ty0p) {
    const int bx = 4 * (blk & 3), by = 4 * (blk >> 2);
    const uint32_t cols = (box >> bx) & 15u, rows = (box >> (16 + by)) & 15u;
    const float A = a.z, B = a.w, C = b.x, k = -2.0f * b.z;
    const bool cut = A * C <= 250.0f * (A * C - B * B);
    // spans of the box inside the block (the bits are contiguous)
    const int x0 = tx0p + bx + __ffs(cols) - 1, x1 = tx0p + bx + 31 - __clz(cols);
    const int y0 = ty0p + by + __ffs(rows) - 1, y1 = ty0p + by + 31 - __clz(rows);
    const bool meets = conic_reaches(A, B, C, k, (float)x0 - a.x, (float)x1 - a.x, (float)y0 - a.y, (float)y1 - a.y);
    return (cols != 0u) & (rows != 0u) & (!cut | meets);
}

// The records of the narrow blends in LDS: (u, v, A, B), (C, opacity, band
// lower edge, band upper edge), colour, box mask; one past the last is an
// entry no pixel takes.  The opacity of an entry whose colour may be infinite is
// negated: the lists' builders read that word anyway, and its magnitude is
// free (a flag of the batch beside the records cost the forward 5% on long lists).
template <int N>
struct NarrowRecs {
    float4 a[N + 1], b[N + 1], col[N + 1];
    uint32_t box[N + 1];
    __device__ __forceinline__ void put(int j, const float4& r0, const float4& r1, const float4& r2, int tx0p, int ty0p) {
        const float4 w2 = blend_stage_w2(r2, tx0p, ty0p);
        a[j] = r0;
        b[j] = make_float4(r1.x, colour_overflows(r1, r2) ? -r1.y : r1.y, w2.y, w2.z);
        col[j] = make_float4(r1.z, r1.w, w2.x, 0.f);
        box[j] = __float_as_uint(w2.w);
    }
    __device__ __forceinline__ void put_none(int j) {
        a[j] = b[j] = col[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        box[j] = 0u;
    }
};

// A batch's records on their way from a tile-major list to LDS: the ids are
// loaded two batches ahead and the records one, so neither is waited for.
struct Ahead {
    float4 r0, r1, r2;
    uint32_t id, next;   // of the records, and of the batch after
    __device__ __forceinline__ void records(const float4* __restrict__ rec) {
        r0 = rec[3 * (int64_t)id];
        r1 = rec[3 * (int64_t)id + 1];
        r2 = rec[3 * (int64_t)id + 2];
    }
};

__global__ __launch_bounds__(kQuarterThreads) void k_blend_fwd_narrow(CamDev cam, const uint2* __restrict__ ranges,
                                                                      const uint32_t* __restrict__ vals,
                                                                      const float4* __restrict__ rec,
                                                                      float* __restrict__ image,
                                                                      float* __restrict__ T_final,
                                                                      uint32_t* __restrict__ last_out,
                                                                      uint32_t* __restrict__ tile_walk) {
    constexpr int NB = kQuarterThreads, NW = kQuarterWaves;   // NB entries a batch
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tile = blockIdx.x >> 2, quarter = blockIdx.x & 3;
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    __shared__ NarrowRecs<NB> s_r;
    __shared__ __align__(8) uint16_t s_list[NW][NB + 3 * kSlots];   // entries that reach the wave's block, in order
    __shared__ uint32_t s_live[2];
    const int tx0p = tx * kTile, ty0p = ty * kTile;
    const int row = lane >> 4, pix = lane & 15, block = quarter_block(quarter, w);
    const int lx = 4 * (block & 3) + (pix & 3), ly = 4 * (block >> 2) + (pix >> 2);
    const int px = tx0p + lx, py = ty0p + ly;
    const float fpx = (float)px, fpy = (float)py;
    const uint32_t sel = (1u << lx) | (1u << (16 + ly));
    float T = 1.0f, c = 0.f;                          // c: the channel of the lane's row (none in row 3)
    uint32_t last = 0u;                               // of the lane's slot
    uint64_t alive = __builtin_amdgcn_ballot_w64(px < cam.W && py < cam.H);
    const uint2 rg = ranges[tile];
    const uint32_t n = rg.y - rg.x;
    const uint32_t* const list = vals + rg.x;
    Ahead ahead;
    if ((uint32_t)tid < n) {
        ahead.id = list[tid];
        if ((uint32_t)tid + NB < n) ahead.next = list[tid + NB];
        ahead.records(rec);
    }
    if (tid == 0) s_r.put_none(NB);
    int par = 0;
    for (uint32_t eb = 0; eb < n; eb += NB, par ^= 1) {
        const uint32_t cnt_u = min((uint32_t)NB, n - eb);
        if ((uint32_t)tid < cnt_u) s_r.put(tid, ahead.r0, ahead.r1, ahead.r2, tx0p, ty0p);
        if (tid == 0) s_live[par] = 0u;
        if (eb + NB + tid < n) {
            ahead.id = ahead.next;
            if (eb + 2 * NB + tid < n) ahead.next = list[eb + 2 * NB + tid];
            ahead.records(rec);
        }
        __syncthreads();
        if (alive) {
            int listed = 0;
            uint64_t over = 0ull;   // listed entries with an infinite colour, which weight zero does not take away
#pragma unroll
            for (int q = 0; q < NB / 64; q++) {
                const int j = 64 * q + lane;
                const float4 ra = s_r.a[j], rb = s_r.b[j];
                const uint64_t m = __builtin_amdgcn_ballot_w64((uint32_t)j < cnt_u &&
                                                               block_reached(ra, rb, s_r.box[j], block, tx0p, ty0p));
                over |= m & __builtin_amdgcn_ballot_w64(rb.y < 0.0f);
                if ((m >> lane) & 1ull) s_list[w][listed + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)j;
                listed += __popcll(m);
            }
            if (lane < 3 * kSlots) s_list[w][listed + lane] = (uint16_t)NB;   // a last group of fewer entries, and two more
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // four entries' opacities; the next four's records are on their
            // way from LDS meanwhile (a heavy quarter has a wave per SIMD)
            struct Four {
                float as[kSlots], col[kSlots];   // opacity 0 in the lanes that do not take their entry
                uint64_t ok;
                int j;
            };
            struct Rec {
                float4 ra, rb;
                float col[kSlots];   // the colours of the four slots, this row's channel
                uint32_t box;
                int j;
            };
            auto four_at = [&](int g) { return *reinterpret_cast<const uint64_t*>(&s_list[w][g]); };
            auto load = [&](uint64_t l) {
                Rec v;
                v.j = (int)((l >> (16 * row)) & 0xFFFFu);
                v.ra = s_r.a[v.j];
                v.rb = s_r.b[v.j];
                v.box = s_r.box[v.j];
#pragma unroll
                for (int s = 0; s < kSlots; s++)
                    v.col[s] = reinterpret_cast<const float*>(&s_r.col[(l >> (16 * s)) & 0xFFFFu])[row];
                return v;
            };
            auto eval = [&](const Rec& r) {
                Four v;
                v.j = r.j;
                const float4 ra = r.ra, rb = r.rb;
                const uint32_t box = r.box;
#pragma unroll
                for (int s = 0; s < kSlots; s++) v.col[s] = r.col[s];
                float adx2, bdx;
                blend_dx_terms(fpx - ra.x, ra, adx2, bdx);
                const float power = blend_power(adx2, bdx, fpy - ra.y, rb.x);
                const uint64_t pm = alive & __builtin_amdgcn_ballot_w64((box & sel) == sel) &
                                    __builtin_amdgcn_ballot_w64(power <= 0.0f) &
                                    __builtin_amdgcn_ballot_w64(power >= rb.z);
                const uint64_t bm = pm & __builtin_amdgcn_ballot_w64(power < rb.w);
                v.ok = pm & ~bm;
                if (bm) v.ok |= bm & __builtin_amdgcn_ballot_w64(blend_exact_test(power, fabsf(rb.y)));
                rows_all(__builtin_amdgcn_inverse_ballot_w64(v.ok) ? fminf(0.99f, fabsf(rb.y) * __expf(power)) : 0.0f, v.as);
                return v;
            };
            Rec ahead4 = load(four_at(0));
            uint64_t l = four_at(kSlots);
            // with one, every group takes the branch that selects
            const float stop_below = over ? __builtin_huge_valf() : 1e-4f;
#pragma unroll 1
            for (int g = 0; g < listed && alive; g += kSlots) {
                const Four cur = eval(ahead4);
                ahead4 = load(l);
                l = four_at(g + 2 * kSlots);
                if (!cur.ok) continue;
                // opacity 0 leaves the transmittance and the colour as they
                // are (T is never below the stop's 1e-4)
                float Ts[kSlots + 1];
                Ts[0] = T;
#pragma unroll
                for (int s = 0; s < kSlots; s++) Ts[s + 1] = Ts[s] * (1.0f - cur.as[s]);
                uint64_t own = cur.ok;   // lanes whose own slot's entry is taken
                if ((alive & __builtin_amdgcn_ballot_w64(Ts[kSlots] < stop_below)) == 0ull) {
#pragma unroll
                    for (int s = 0; s < kSlots; s++) c += (cur.as[s] * Ts[s]) * cur.col[s];
                    T = Ts[kSlots];
                } else {   // a pixel stops among the four, or may meet an infinite colour
                    uint64_t taken = 0ull;
#pragma unroll
                    for (int s = 0; s < kSlots; s++) {
                        const float Tn = T * (1.0f - cur.as[s]);
                        const uint64_t stop = alive & __builtin_amdgcn_ballot_w64(Tn < 1e-4f);
                        const uint64_t takem = alive & ~stop;
                        const bool take = __builtin_amdgcn_inverse_ballot_w64(takem);
                        const float cn = c + (cur.as[s] * T) * cur.col[s];
                        c = take && cur.as[s] != 0.0f ? cn : c;
                        T = take ? Tn : T;
                        alive = takem;
                        taken |= takem & (0xFFFFull << (16 * s));
                    }
                    own &= taken;
                }
                last = __builtin_amdgcn_inverse_ballot_w64(own) ? eb + (uint32_t)cur.j + 1u : last;
            }
        }
        if (lane == 0 && alive) s_live[par] = 1u;
        __syncthreads();
        if (s_live[par] == 0u) break;
    }
    const int64_t P = (int64_t)cam.W * cam.H;
    if (px < cam.W && py < cam.H) {
        const int64_t p = (int64_t)py * cam.W + px;
        if (row < 3) image[row * P + p] = c + T * (row == 0 ? cam.bg[0] : row == 1 ? cam.bg[1] : cam.bg[2]);
        else T_final[p] = T;
    }
    // the pixel's last contributor: the latest of its four slots
    last = max(last, (uint32_t)__shfl_xor((int)last, 16));
    last = max(last, (uint32_t)__shfl_xor((int)last, 32));
    if (row == 3 && px < cam.W && py < cam.H) last_out[(int64_t)py * cam.W + px] = last;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) last = max(last, (uint32_t)__shfl_xor((int)last, off));
    if (lane == 0 && last) atomicMax(tile_walk + tile, last);
}

// kRecords: a workgroup a tile (its entries' records hold the whole tile's
// sums); else a quarter.
template <bool kRecords, bool kOpacity>
__global__ __launch_bounds__(kRecords ? kNarrowThreads : kQuarterThreads) void k_blend_bwd_narrow(
    CamDev cam, const uint2* __restrict__ ranges, const uint32_t* __restrict__ vals, const float4* __restrict__ rec,
    const float* __restrict__ d_image, const float* __restrict__ T_final, const uint32_t* __restrict__ last_in,
    const uint32_t* __restrict__ walk_off, float* __restrict__ grec, uint32_t grec_cap, float* __restrict__ accum) {
    constexpr int NT = kRecords ? kNarrowThreads : kQuarterThreads, NW = NT / 64, KB = kBwdBatch;
    static_assert(KB == 128 && KB <= NT, "two words, and a thread per entry");
    __shared__ NarrowRecs<KB> s_r;
    __shared__ uint32_t s_id[KB];
    __shared__ uint64_t s_reach[2][NW];
    __shared__ uint16_t s_list[NW][KB + 3 * kSlots];
    __shared__ float s_g[NW][9][KB + 1];   // per-wave sums, [wave][term][entry]; the last is no entry's
    __shared__ uint32_t s_last[NW];
    const int tile = kRecords ? blockIdx.x : blockIdx.x >> 2;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    const int tx0p = tx * kTile, ty0p = ty * kTile;
    const int row = lane >> 4, pix = lane & 15, block = kRecords ? w : quarter_block(blockIdx.x & 3, w);
    const int lx = 4 * (block & 3) + (pix & 3), ly = 4 * (block >> 2) + (pix >> 2);
    const int px = tx0p + lx, py = ty0p + ly;
    const float fpx = (float)px, fpy = (float)py;
    const uint32_t sel = (1u << lx) | (1u << (16 + ly));
    const uint32_t woff = kRecords ? walk_off[tile] : 0u;
    const int64_t P = (int64_t)cam.W * cam.H;
    float T = 1.0f, g0 = 0.f, g1 = 0.f, g2 = 0.f;
    uint32_t last = 0u;
    if (px < cam.W && py < cam.H) {
        const int64_t p = (int64_t)py * cam.W + px;
        T = T_final[p];
        last = last_in[p];
        g0 = d_image[p];
        g1 = d_image[P + p];
        g2 = d_image[2 * P + p];
    }
    float gb = g0 * cam.bg[0] + g1 * cam.bg[1] + g2 * cam.bg[2];   // see k_blend_bwd
    uint32_t wlast = last;   // the block's last contributor
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) wlast = max(wlast, (uint32_t)__shfl_xor((int)wlast, off));
    wlast = __builtin_amdgcn_readfirstlane(wlast);
    const int term = row_term(pix);
    const int slot9 = term < 5 ? term : term + 1;   // index in the nine-term layout
    if (lane == 0) s_last[w] = wlast;
    if (tid == 0) s_r.put_none(KB);
    __syncthreads();
    uint32_t maxlast = 0u;
#pragma unroll
    for (int k = 0; k < NW; k++) maxlast = max(maxlast, s_last[k]);
    if (maxlast == 0) return;
    const uint32_t* const list = vals + ranges[tile].x;
    const int64_t top = ((int64_t)(maxlast - 1) / KB) * KB;
    Ahead ahead;   // walking back: the batch below is the next
    if (tid < KB) {
        if (top >= KB) ahead.next = list[top - KB + tid];
        if (top + tid < (int64_t)maxlast) {
            ahead.id = list[top + tid];
            ahead.records(rec);
        }
    }
    for (int64_t jb = top; jb >= 0; jb -= KB) {
        const int cnt = (int)min((int64_t)KB, (int64_t)maxlast - jb);
        if (tid < cnt) {
            s_id[tid] = ahead.id;
            s_r.put(tid, ahead.r0, ahead.r1, ahead.r2, tx0p, ty0p);
        }
        if (tid < KB && jb >= KB) {
            ahead.id = ahead.next;
            if (jb >= 2 * KB) ahead.next = list[jb - 2 * KB + tid];
            ahead.records(rec);
        }
        __syncthreads();
        // the block's entries, last first, up to its last contributor; the
        // words keep the entries that are visited
        int listed = 0;
        const int64_t before = (int64_t)wlast - jb;
#pragma unroll
        for (int q = 1; q >= 0; q--) {
            const int j = 64 * q + lane;
            const int64_t left = min(before, (int64_t)cnt) - 64 * q;
            uint64_t m = 0ull;
            if (left > 0) {
                const float4 ra = s_r.a[j], rb = s_r.b[j];
                m = __builtin_amdgcn_ballot_w64(lane < left && block_reached(ra, rb, s_r.box[j], block, tx0p, ty0p));
            }
            const int n = __popcll(m);
            if ((m >> lane) & 1ull)
                s_list[w][listed + n - 1 - __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)j;
            listed += n;
            if (lane == 0) s_reach[q][w] = m;
        }
        if (lane < 3 * kSlots) s_list[w][listed + lane] = (uint16_t)KB;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // four entries up to their opacities and colour terms; see the forward
        struct Four {
            float as[kSlots], ds[kSlots];   // opacity zero: the pixel's state is kept
            float al, raw, G, dx, dy;       // the lane's own slot
            uint64_t ok;
            int j;
        };
        struct Rec {
            float4 ra, rb, rc;
            uint32_t box;
            int j;
        };
        auto load = [&](int j) { return Rec{s_r.a[j], s_r.b[j], s_r.col[j], s_r.box[j], j}; };
        auto eval = [&](const Rec& r) {
            Four v;
            v.j = r.j;
            const float4 ra = r.ra, rb = r.rb, rc = r.rc;
            const uint32_t box = r.box;
            v.dx = fpx - ra.x;
            v.dy = fpy - ra.y;
            float adx2, bdx;
            blend_dx_terms(v.dx, ra, adx2, bdx);
            const float power = blend_power(adx2, bdx, v.dy, rb.x);
            const uint64_t pm = __builtin_amdgcn_ballot_w64((uint32_t)jb + (uint32_t)v.j < last) &
                                __builtin_amdgcn_ballot_w64((box & sel) == sel) &
                                __builtin_amdgcn_ballot_w64(power <= 0.0f) & __builtin_amdgcn_ballot_w64(power >= rb.z);
            const uint64_t bm = pm & __builtin_amdgcn_ballot_w64(power < rb.w);
            v.ok = pm & ~bm;
            if (bm) v.ok |= bm & __builtin_amdgcn_ballot_w64(blend_exact_test(power, fabsf(rb.y)));
            v.G = __expf(power);
            v.raw = fabsf(rb.y) * v.G;
            v.al = __builtin_amdgcn_inverse_ballot_w64(v.ok) ? fminf(0.99f, v.raw) : 0.0f;
            rows_all(v.al, v.as);
            // zero where the entry is not taken: opacity zero does not take an infinite colour away
            rows_all(__builtin_amdgcn_inverse_ballot_w64(v.ok) ? g0 * rc.x + g1 * rc.y + g2 * rc.z : 0.0f, v.ds);
            return v;
        };
        Rec ahead4 = load(s_list[w][row]);
        int j = s_list[w][kSlots + row];
#pragma unroll 1
        for (int g = 0; g < listed; g += kSlots) {
            const Four cur = eval(ahead4);
            ahead4 = load(j);
            j = s_list[w][g + 2 * kSlots + row];
            float red = 0.f, redop = 0.f;
            if (cur.ok) {
                float To = 0.f, d = 0.f;   // transmittance before, and colour term of, the lane's own slot
#pragma unroll
                for (int s = 0; s < kSlots; s++) {
                    // T recovery T_i = T_{i+1} / (1 - alpha_i), with the hardware reciprocal (1 ulp)
                    T *= __builtin_amdgcn_rcpf(1.0f - cur.as[s]);
                    const float di = cur.ds[s] - gb;
                    gb += cur.as[s] * di;
                    To = row == s ? T : To;
                    d = row == s ? di : d;
                }
                const float wgt = cur.al * To;
                const float dal = To * d;
                const bool unclamped =
                    __builtin_amdgcn_inverse_ballot_w64(cur.ok & __builtin_amdgcn_ballot_w64(cur.raw < 0.99f));
                const float dp = unclamped ? dal * cur.raw : 0.0f;
                const float ax = dp * cur.dx, ay = dp * cur.dy;   // terms: see k_blend_bwd
                const float t8[8] = {ax, ay, ax * cur.dx, ax * cur.dy, ay * cur.dy, g0 * wgt, g1 * wgt, g2 * wgt};
                red = row_reduce_scatter8(t8, pix);
                if (kOpacity) {
                    float o = unclamped ? dal * cur.G : 0.0f;
                    o = dpp_add<0xB1, 0xF>(o);
                    o = dpp_add<0x4E, 0xF>(o);
                    o = dpp_add<0x141, 0xF>(o);
                    redop = dpp_add<0x140, 0xF>(o);   // row_mirror
                }
            }
            if ((pix & 1) == 0) s_g[w][slot9][cur.j] = red;
            if (kOpacity && pix == 1) s_g[w][5][cur.j] = redop;
        }
        __syncthreads();
        sum_batch<NW, KB, kOpacity>(
            cnt, w, lane, s_reach, s_g, [&](int e) { return make_float3(s_r.a[e].z, s_r.a[e].w, s_r.b[e].x); },
            [&](int e, int k, float v) {
                const uint32_t widx = woff + (uint32_t)jb + e;   // compact index of this walked entry
                if (kRecords && widx < grec_cap)
                    grec[(int64_t)k * grec_cap + widx] = v;
                else if (v != 0.f)
                    atomicAdd(accum + 9 * (int64_t)s_id[e] + k, v);
            });
        __syncthreads();
    }
}

__device__ __forceinline__ void quat_rot_adj(const float q[4], const float g[9], float d[4]) {
    const float w = q[0], x = q[1], y = q[2], z = q[3];
    d[0] += 2.f * (-z * g[1] + y * g[2] + z * g[3] - x * g[5] - y * g[6] + x * g[7]);
    d[1] += 2.f * (y * g[1] + z * g[2] + y * g[3] - 2.f * x * g[4] - w * g[5] + z * g[6] + w * g[7] - 2.f * x * g[8]);
    d[2] += 2.f * (-2.f * y * g[0] + x * g[1] + w * g[2] + x * g[3] + z * g[5] - w * g[6] + z * g[7] - 2.f * y * g[8]);
    d[3] += 2.f * (-2.f * z * g[0] - w * g[1] + x * g[2] + w * g[3] - 2.f * z * g[4] + y * g[5] + x * g[6] + y * g[7]);
}

// ---------------------------------------------------------------------------
// preprocess backward: chain the per-Gaussian 2D gradients through the conic
// inverse, EWA (with J depending on the camera-space mean), the covariance,
// the colour (SH and its view direction) and the transform.
// ---------------------------------------------------------------------------
template <bool kRecords>
__global__ __launch_bounds__(256) void k_preprocess_bwd(GaussDev g, CamDev cam, float* __restrict__ accum,
                                                        GatherDev ga, GradsDev out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.n) return;
    // the blend's sums, left zero for the next backward
    float a9[9];
    for (int k = 0; k < 9; k++) a9[k] = accum[9 * i + k];
    for (int k = 0; k < 9; k++) accum[9 * i + k] = 0.f;
    Geo o;
    if (!geo_forward(g, cam, i, o)) return;
    ColourCtx cc;
    colour_forward(g, cam, i, o, cc);
    // the nine 2D gradient terms: the sums (records: those past the buffer)
    // plus this Gaussian's walked entries, visited in its tile-rectangle order
    if constexpr (kRecords) {
        // four entries at a time, whose chains of loads run side by side (5K
        // Gaussians at 200 x 152, with a wave a workgroup: 29 -> 20 us).  Bound by
        // the lanes' lines where rectangles are large, so a lane loads for an entry
        // that was walked only: 40K Gaussians at 1920 x 1080, one pair in fifteen
        // walked, 920 us with every lane loading, 786 so, 814 one at a time
        constexpr int U = 4;
        const uint2 r = ga.rect[i];
        const int tx0 = r.x & 0xFFFF, ty0 = r.x >> 16, tx1 = r.y & 0xFFFF, ty1 = r.y >> 16;
        const uint64_t k0 = ga.goff[i];
        const int n = (tx1 - tx0 + 1) * (ty1 - ty0 + 1);
        int tx = tx0, ty = ty0;
        for (int e = 0; e < n; e += U) {
            uint32_t widx[U];
            bool on[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int t = ty * cam.tiles_x + tx;   // past the rectangle: its last tile
                on[u] = e + u < n && k0 + e + u < ga.cap;
                const uint32_t rel = (on[u] ? ga.gpos[k0 + e + u] : 0u) - ga.ranges[t].x;
                on[u] = on[u] && rel < ga.tile_walk[t];
                widx[u] = on[u] ? ga.walk_off[t] + rel : 0u;
                on[u] = on[u] && widx[u] < ga.grec_cap;
                const bool wrap = tx == tx1;
                if (!(wrap && ty == ty1)) {
                    tx = wrap ? tx0 : tx + 1;
                    ty += wrap ? 1 : 0;
                }
            }
            float v[U][9];
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (on[u]) {
#pragma unroll
                    for (int c = 0; c < 9; c++) v[u][c] = ga.grec[(int64_t)c * ga.grec_cap + widx[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < U; u++)
#pragma unroll
                for (int c = 0; c < 9; c++) a9[c] = on[u] ? a9[c] + v[u][c] : a9[c];
        }
    }
    const float du = a9[0], dv = a9[1], dA = a9[2], dB = a9[3], dC = a9[4], dop = a9[5];
    const float drgb[3] = {a9[6], a9[7], a9[8]};
    if (out.d_uv) { out.d_uv[2 * i] += du; out.d_uv[2 * i + 1] += dv; }
    if (out.vgrad) {
        // gradient with respect to the normalised-device-coordinate mean
        const float gx = du * (0.5f * (float)cam.W), gy = dv * (0.5f * (float)cam.H);
        out.vgrad[i] += sqrtf(gx * gx + gy * gy);
        out.vcount[i] += 1.0f;
    }
    if (out.d_conic) { out.d_conic[3 * i] += dA; out.d_conic[3 * i + 1] += dB; out.d_conic[3 * i + 2] += dC; }
    if (out.d_opacity) out.d_opacity[i] += dop;
    if (out.d_rgb) for (int k = 0; k < 3; k++) out.d_rgb[3 * i + k] += drgb[k];
    if (out.d_opac) {
        const float op = opacity_of(g.opac[i]);
        out.d_opac[i] += dop * op * (1.0f - op);
    }
    float dm[3] = {0.f, 0.f, 0.f};
    float dRp[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float dRh[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    // colour
    float gch[3];
    for (int k = 0; k < 3; k++) gch[k] = cc.raw[k] > 0.f ? drgb[k] : 0.f;
    float wk[16];
    switch (g.sh_degree) {
        case 3: sh_weights<16>(g.sh + i * 48, gch, wk); break;
        case 1: sh_weights<4>(g.sh + i * 12, gch, wk); break;
        case 2: sh_weights<9>(g.sh + i * 27, gch, wk); break;
        default: sh_weights<1>(g.sh + i * 3, gch, wk); break;
    }
    // a Gaussian that no pixel saw leaves its row as it is
    if (out.d_sh && (gch[0] != 0.f || gch[1] != 0.f || gch[2] != 0.f)) {
        float Y[16];
        sh_basis(g.sh_degree, cc.dl[0], cc.dl[1], cc.dl[2], Y);
        switch (g.sh_degree) {
            case 3: sh_accumulate<16>(out.d_sh + i * 48, gch, Y); break;
            case 1: sh_accumulate<4>(out.d_sh + i * 12, gch, Y); break;
            case 2: sh_accumulate<9>(out.d_sh + i * 27, gch, Y); break;
            default: sh_accumulate<1>(out.d_sh + i * 3, gch, Y); break;
        }
    }
    float gdl[3];
    sh_grad(g.sh_degree, cc.dl[0], cc.dl[1], cc.dl[2], wk, gdl[0], gdl[1], gdl[2]);
    float ddir[3];
    if (g.dq) {
        for (int k = 0; k < 3; k++) ddir[k] = cc.Ml[k] * gdl[0] + cc.Ml[3 + k] * gdl[1] + cc.Ml[6 + k] * gdl[2];
        // Ml = Rh Rp^T, dMl = gdl dir^T:  dRh = dMl Rp, dRp = dMl^T Rh
        for (int r = 0; r < 3; r++)
            for (int k = 0; k < 3; k++) {
                dRh[3 * r + k] += gdl[r] * (cc.dir[0] * o.Rp[k] + cc.dir[1] * o.Rp[3 + k] + cc.dir[2] * o.Rp[6 + k]);
                dRp[3 * r + k] += cc.dir[r] * (gdl[0] * cc.Rh[k] + gdl[1] * cc.Rh[3 + k] + gdl[2] * cc.Rh[6 + k]);
            }
    } else {
        ddir[0] = gdl[0]; ddir[1] = gdl[1]; ddir[2] = gdl[2];
    }
    {
        const float pd = ddir[0] * cc.dir[0] + ddir[1] * cc.dir[1] + ddir[2] * cc.dir[2];
        for (int k = 0; k < 3; k++) dm[k] += (ddir[k] - cc.dir[k] * pd) / cc.wn;
    }

    // conic (A, B, C) = (c, -b, a) / det
    const float a = o.a, b = o.b, c = o.c, det = o.det, id2 = 1.0f / (det * det), idt = 1.0f / det;
    const float da = dA * (-c * c * id2) + dB * (b * c * id2) + dC * (idt - a * c * id2);
    const float db = dA * (2.f * b * c * id2) + dB * (-idt - 2.f * b * b * id2) + dC * (2.f * a * b * id2);
    const float dc = dA * (idt - a * c * id2) + dB * (a * b * id2) + dC * (-a * a * id2);
    // Sigma2 = T Sigma T^T: G2 = [[da, db/2], [db/2, dc]]
    const float G00 = da, G01 = 0.5f * db, G11 = dc;
    const float T0[3] = {o.T00, o.T01, o.T02}, T1[3] = {o.T10, o.T11, o.T12};
    const float S[9] = {o.S00, o.S01, o.S02, o.S01, o.S11, o.S12, o.S02, o.S12, o.S22};
    float dS[9];
    for (int p = 0; p < 3; p++)
        for (int q = 0; q < 3; q++)
            dS[3 * p + q] = T0[p] * (G00 * T0[q] + G01 * T1[q]) + T1[p] * (G01 * T0[q] + G11 * T1[q]);
    // dT = 2 G2 T Sigma
    float TS0[3], TS1[3];
    for (int q = 0; q < 3; q++) {
        TS0[q] = T0[0] * S[q] + T0[1] * S[3 + q] + T0[2] * S[6 + q];
        TS1[q] = T1[0] * S[q] + T1[1] * S[3 + q] + T1[2] * S[6 + q];
    }
    float dT0[3], dT1[3];
    for (int q = 0; q < 3; q++) {
        dT0[q] = 2.f * (G00 * TS0[q] + G01 * TS1[q]);
        dT1[q] = 2.f * (G01 * TS0[q] + G11 * TS1[q]);
    }
    const float* R = cam.R;
    const float dj00 = dT0[0] * R[0] + dT0[1] * R[1] + dT0[2] * R[2];
    const float dj02 = dT0[0] * R[6] + dT0[1] * R[7] + dT0[2] * R[8];
    const float dj11 = dT1[0] * R[3] + dT1[1] * R[4] + dT1[2] * R[5];
    const float dj12 = dT1[0] * R[6] + dT1[1] * R[7] + dT1[2] * R[8];
    const float tx = o.t[0], ty = o.t[1], tz = o.t[2], itz = 1.0f / tz, itz2 = itz * itz;
    const float fx = cam.fx, fy = cam.fy;
    float dtx = 0.f, dty = 0.f, dtz = 0.f;
    dtz += dj00 * (-fx * itz2) + dj11 * (-fy * itz2) + dj02 * (fx * o.txc * itz2) + dj12 * (fy * o.tyc * itz2);
    const float dtxc = dj02 * (-fx * itz), dtyc = dj12 * (-fy * itz);
    if (!o.clx) { dtx += dtxc * itz; dtz += -dtxc * tx * itz2; }
    if (!o.cly) { dty += dtyc * itz; dtz += -dtyc * ty * itz2; }
    dtx += du * fx * itz;
    dty += dv * fy * itz;
    dtz += -du * fx * tx * itz2 - dv * fy * ty * itz2;
    for (int k = 0; k < 3; k++) dm[k] += R[k] * dtx + R[3 + k] * dty + R[6 + k] * dtz;

    // Sigma = M M^T with M = Rp diag(s): dM = 2 dS M
    float M[9];
    for (int r = 0; r < 3; r++)
        for (int k = 0; k < 3; k++) M[3 * r + k] = o.Rp[3 * r + k] * o.s[k];
    float ds[3] = {0.f, 0.f, 0.f};
    for (int r = 0; r < 3; r++)
        for (int k = 0; k < 3; k++) {
            const float dMrk = 2.f * (dS[3 * r] * M[k] + dS[3 * r + 1] * M[3 + k] + dS[3 * r + 2] * M[6 + k]);
            dRp[3 * r + k] += dMrk * o.s[k];
            ds[k] += dMrk * o.Rp[3 * r + k];
        }
    if (out.d_log_scales)
        for (int k = 0; k < 3; k++) out.d_log_scales[3 * i + k] += ds[k] * o.s[k];

    // rotations -> quaternions
    float dqp[4] = {0.f, 0.f, 0.f, 0.f}, dqh[4] = {0.f, 0.f, 0.f, 0.f};
    quat_rot_adj(o.qp, dRp, dqp);
    if (g.dq) {
        quat_rot_adj(o.qh, dRh, dqh);
        const float bw = o.dh[0], bx = o.dh[1], by = o.dh[2], bz = o.dh[3];
        const float aw = o.qh[0], ax = o.qh[1], ay = o.qh[2], az = o.qh[3];
        // q' = qh (x) dh; gradient with respect to qh is Rb^T dqp, to dh is La^T dqp
        dqh[0] += bw * dqp[0] + bx * dqp[1] + by * dqp[2] + bz * dqp[3];
        dqh[1] += -bx * dqp[0] + bw * dqp[1] - bz * dqp[2] + by * dqp[3];
        dqh[2] += -by * dqp[0] + bz * dqp[1] + bw * dqp[2] - bx * dqp[3];
        dqh[3] += -bz * dqp[0] - by * dqp[1] + bx * dqp[2] + bw * dqp[3];
        float ddh[4];
        ddh[0] = aw * dqp[0] + ax * dqp[1] + ay * dqp[2] + az * dqp[3];
        ddh[1] = -ax * dqp[0] + aw * dqp[1] + az * dqp[2] - ay * dqp[3];
        ddh[2] = -ay * dqp[0] - az * dqp[1] + aw * dqp[2] + ax * dqp[3];
        ddh[3] = -az * dqp[0] + ay * dqp[1] - ax * dqp[2] + aw * dqp[3];
        if (out.d_dq) {
            const float pd = o.dh[0] * ddh[0] + o.dh[1] * ddh[1] + o.dh[2] * ddh[2] + o.dh[3] * ddh[3];
            const bool nz = o.dn > 1e-12f;
            for (int k = 0; k < 4; k++)
                out.d_dq[4 * i + k] += nz ? (ddh[k] - o.dh[k] * pd) / o.dn : ddh[k] / o.dn;
        }
    } else {
        for (int k = 0; k < 4; k++) dqh[k] += dqp[k];
    }
    if (out.d_quats && o.qn > 0.f) {
        const float pd = o.qh[0] * dqh[0] + o.qh[1] * dqh[1] + o.qh[2] * dqh[2] + o.qh[3] * dqh[3];
        for (int k = 0; k < 4; k++) out.d_quats[4 * i + k] += (dqh[k] - o.qh[k] * pd) / o.qn;
    }
    for (int k = 0; k < 3; k++) {
        if (out.d_means) out.d_means[3 * i + k] += dm[k];
        if (out.d_dmu) out.d_dmu[3 * i + k] += dm[k];
    }
}

__global__ __launch_bounds__(256) void k_debug_keys(const uint2* __restrict__ ranges, const uint32_t* __restrict__ vals,
                                                    const uint32_t* __restrict__ key, int ntiles,
                                                    uint64_t* __restrict__ keys_out) {
    const int t = blockIdx.x;
    if (t >= ntiles) return;
    const uint2 r = ranges[t];
    for (uint32_t e = r.x + threadIdx.x; e < r.y; e += 256) keys_out[e] = ((uint64_t)t << 32) | key[vals[e]];
}

__global__ __launch_bounds__(256) void k_debug_records(int64_t n, const float4* __restrict__ rec,
                                                       int32_t* __restrict__ box, float* __restrict__ rec9) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float4 a = rec[3 * i], b = rec[3 * i + 1], c = rec[3 * i + 2];
    if (box) {
        const uint32_t b0 = __float_as_uint(c.y), b1 = __float_as_uint(c.z);
        box[4 * i + 0] = b0 & 0xFFFF; box[4 * i + 1] = b0 >> 16;
        box[4 * i + 2] = b1 & 0xFFFF; box[4 * i + 3] = b1 >> 16;
    }
    if (rec9) {
        float v[9] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x};
        for (int k = 0; k < 9; k++) rec9[9 * i + k] = v[k];
    }
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

void preprocess(const Launch& L, const GaussDev& g, const CamDev& cam, float4* rec, uint32_t* key, uint2* rect,
                uint32_t* count) {
    if (g.n <= 0) return;
    if (L.prof) L.prof->begin("preprocess_fwd", L.st);
    hipLaunchKernelGGL(k_preprocess, dim3(blocks_for(g.n, 256)), dim3(256), 0, L.st, g, cam, rec, key, rect, count);
    if (L.prof) L.prof->end(L.st);
}

void emit_pairs(const Launch& L, int64_t n, const uint32_t* key, const uint2* rect, const uint64_t* offs, int tiles_x,
                uint64_t cap, uint64_t* keys, uint32_t* vals) {
    if (n <= 0) return;
    if (L.prof) L.prof->begin("emit_keys", L.st);
    hipLaunchKernelGGL(k_emit, dim3(blocks_for(n, 256)), dim3(256), 0, L.st, n, key, rect, offs, tiles_x, cap, keys,
                       vals);
    if (L.prof) L.prof->end(L.st);
}

void ranges_from_keys(const Launch& L, const uint64_t* keys, int64_t K, int ntiles, uint2* ranges) {
    if (L.prof) L.prof->begin("tile_ranges", L.st);
    hipLaunchKernelGGL(k_zero_ranges, dim3(blocks_for(ntiles, 256)), dim3(256), 0, L.st, ranges, ntiles);
    if (K > 0)
        hipLaunchKernelGGL(k_ranges_from_keys, dim3(blocks_for(K, 256)), dim3(256), 0, L.st, keys, K, ranges);
    if (L.prof) L.prof->end(L.st);
}

void bin_gather(const Launch& L, const uint32_t* order, int64_t n, const uint2* rect, const uint32_t* count,
                const uint64_t* goff, uint64_t cap, uint2* srect, uint32_t* sgoff) {
    if (n <= 0) return;
    if (L.prof) L.prof->begin("bin_gather", L.st);
    hipLaunchKernelGGL(k_bin_gather, dim3(blocks_for(n, 256)), dim3(256), 0, L.st, order, n, rect, count, goff,
                       (uint32_t)std::min<uint64_t>(cap, 0xFFFFFFFFull), srect, sgoff);
    if (L.prof) L.prof->end(L.st);
}

int64_t bin_chunks(int64_t n) { return (((n + kBinChunk - 1) / kBinChunk) + 7) / 8 * 8; }

static dim3 bin_grid(int64_t nchunks, int tiles_y) {
    return dim3((unsigned)(nchunks * ((tiles_y + kBinRowsPerBlock - 1) / kBinRowsPerBlock)));
}

void bin_count(const Launch& L, int64_t n, const uint2* srect, int tiles_x, int tiles_y, uint32_t* hist) {
    const int64_t nchunks = n > 0 ? bin_chunks(n) : 0;
    if (nchunks == 0) return;
    if (L.prof) L.prof->begin("bin_count", L.st);
    const unsigned grid = (unsigned)((nchunks / kCountGroup) * ((tiles_y + kBinRowsPerBlock - 1) / kBinRowsPerBlock));
    hipLaunchKernelGGL(k_bin_count, dim3(grid), dim3(kBinThreads), 0, L.st, srect, n, tiles_x, tiles_y, nchunks, hist);
    if (L.prof) L.prof->end(L.st);
}

int64_t bin_scan_part_words(int64_t nchunks, int ntiles) {
    return ((nchunks + kBinScanSeg - 1) / kBinScanSeg) * (int64_t)ntiles;
}

void bin_scan(const Launch& L, const uint32_t* hist, int64_t nchunks, int ntiles, uint32_t cap, uint32_t* base,
              uint64_t* total, uint32_t* part, uint32_t* ttot, uint64_t* toff, uint64_t* tmp) {
    if (nchunks <= 0 || ntiles <= 0) return;
    if (L.prof) L.prof->begin("scan", L.st);
    const int64_t nseg = (nchunks + kBinScanSeg - 1) / kBinScanSeg;
    const dim3 grid((unsigned)((ntiles + 255) / 256), (unsigned)std::min<int64_t>(nseg, 65535));
    hipLaunchKernelGGL(k_bin_scan_part, grid, dim3(256), 0, L.st, hist, nchunks, ntiles, nseg, part);
    hipLaunchKernelGGL(k_bin_scan_tiles, dim3((unsigned)((ntiles + 255) / 256)), dim3(256), 0, L.st, part, nseg,
                       ntiles, ttot);
    if (L.prof) L.prof->end(L.st);
    scan_u32_to_u64(L, ttot, ntiles, toff, total, tmp);
    if (L.prof) L.prof->begin("scan", L.st);
    hipLaunchKernelGGL(k_bin_scan_base, grid, dim3(256), 0, L.st, hist, nchunks, ntiles, nseg, part, toff, cap, base);
    if (L.prof) L.prof->end(L.st);
}

void bin_scatter(const Launch& L, const uint32_t* order, int64_t n, const uint2* srect, const uint32_t* sgoff,
                 int tiles_x, int tiles_y, const uint32_t* base, uint64_t cap, uint32_t* vals, uint32_t* gpos) {
    const int64_t nchunks = n > 0 ? bin_chunks(n) : 0;
    if (nchunks == 0) return;
    if (L.prof) L.prof->begin("bin_scatter", L.st);
    hipLaunchKernelGGL(k_bin_rows, bin_grid(nchunks, tiles_y), dim3(kBinThreads), 0, L.st, order, n, srect, sgoff,
                       tiles_x, tiles_y, nchunks, base, (uint32_t)cap, vals, gpos);
    if (L.prof) L.prof->end(L.st);
}

void gpos_from_pairs(const Launch& L, const uint64_t* keys, const uint32_t* vals, int64_t K, const uint2* rect,
                     const uint64_t* goff, int tiles_x, uint64_t cap, uint32_t* gpos) {
    if (K <= 0) return;
    hipLaunchKernelGGL(k_gpos_from_pairs, dim3(blocks_for(K, 256)), dim3(256), 0, L.st, keys, vals, K, rect, goff,
                       tiles_x, cap, gpos);
}

void ranges_from_hist(const Launch& L, const uint32_t* base, const uint64_t* total, int ntiles, uint64_t cap,
                      uint2* ranges, int* overflow) {
    if (L.prof) L.prof->begin("tile_ranges", L.st);
    hipLaunchKernelGGL(k_ranges_from_hist, dim3(blocks_for(ntiles, 256)), dim3(256), 0, L.st, base, total, ntiles, cap,
                       ranges, overflow);
    if (L.prof) L.prof->end(L.st);
}


void tile_order(const Launch& L, const uint2* ranges, const uint32_t* walk, int ntiles, int* order) {
    if (L.prof) L.prof->begin("tile_order", L.st);
    hipLaunchKernelGGL(k_tile_order, dim3(1), dim3(1024), 0, L.st, ranges, walk, ntiles, order);
    if (L.prof) L.prof->end(L.st);
}

// Views of at most two tiles per CU take the narrow blends.  Render / backward
// of 50K surface Gaussians (us), 8 x 8 against narrow: 100 tiles 383 / 450
// against 165 / 180, 256 tiles 276 / 320 against 132 / 126, 529 tiles 200 / 209
// against 117 / 92; of 50K uniform ones: 256 tiles 96 / 69 against 84 / 46, 529
// tiles 91 / 65 against 96 / 57, 784 tiles 91 / 62 against 106 / 70, 1620
// tiles 105 / 83 against 148 / 130: with many tiles of like lists the 8 x 8
// blends fill the SIMDs, and evaluate a large Gaussian's pixels 64 at a time.
// With gradient records the backward keeps a tile to a workgroup: at most one
// per CU (400 uniform tiles 108 / 71 against 114 / 88).  Without, the backward's
// LDS lets six workgroups share a CU, 384 tiles in all; the quarters past those
// start in raster order as others end.  Even where the longest tiles come last
// that costs less than 8 x 8 blends, longest first: surfaces in the far corner of
// the view, 50K at 400, 480 and 512 tiles 487 / 570, 470 / 523 and 159 / 162
// against 193 / 236, 193 / 237 and 109 / 81, 200K at 506 tiles 1177 / 1480
// against 403 / 640.
bool narrow_tiles(int ntiles, bool records) { return ntiles <= (records ? kNarrowTiles / 2 : kNarrowTiles); }

void blend_forward(const Launch& L, const CamDev& cam, const uint2* ranges, const uint32_t* vals, const float4* rec,
                   float* image, float* T_final, uint32_t* last, uint32_t* tile_walk, const int* order, uint64_t* taken,
                   const SuperDev* supers, bool narrow) {
    const int ntiles = cam.tiles_x * cam.tiles_y;
    if (L.prof) L.prof->begin("blend_fwd", L.st);
    if (narrow) {
        hipLaunchKernelGGL(k_blend_fwd_narrow, dim3(4u * (unsigned)ntiles), dim3(kQuarterThreads), 0, L.st, cam, ranges,
                           vals, rec, image, T_final, last, tile_walk);
    } else if (supers) {
        const int nsuper = supers->supers_x * super_count_of(cam.tiles_y);
        const unsigned grid = (unsigned)((nsuper + 7) / 8 * 8 * kSuperDim * kSuperDim);
        hipLaunchKernelGGL((k_blend_fwd<true>), dim3(grid), dim3(kBlendThreads), 0, L.st, cam, ranges, vals, rec, image,
                           T_final, last, tile_walk, order, taken, *supers, nsuper);
    } else {
        hipLaunchKernelGGL((k_blend_fwd<false>), dim3((unsigned)ntiles), dim3(kBlendThreads), 0, L.st, cam, ranges, vals,
                           rec, image, T_final, last, tile_walk, order, taken, SuperDev{}, 0);
    }
    if (L.prof) L.prof->end(L.st);
}

void blend_backward(const Launch& L, const CamDev& cam, const uint2* ranges, const uint32_t* vals, const float4* rec,
                    const float* d_image, const float* T_final, const uint32_t* last, const GatherDev& ga,
                    float* accum, bool want_opacity, const int* order, const uint64_t* taken, const SuperDev* supers,
                    bool narrow) {
    const int ntiles = cam.tiles_x * cam.tiles_y;
    if (L.prof) L.prof->begin("blend_bwd", L.st);
    const bool records = ga.grec_cap > 0;
    if (narrow) {
        auto kern = records ? (want_opacity ? k_blend_bwd_narrow<true, true> : k_blend_bwd_narrow<true, false>)
                            : (want_opacity ? k_blend_bwd_narrow<false, true> : k_blend_bwd_narrow<false, false>);
        hipLaunchKernelGGL(kern, dim3((records ? 1u : 4u) * (unsigned)ntiles),
                           dim3(records ? kNarrowThreads : kQuarterThreads), 0, L.st, cam, ranges, vals, rec, d_image,
                           T_final, last, ga.walk_off, ga.grec, (uint32_t)ga.grec_cap, accum);
        if (L.prof) L.prof->end(L.st);
        return;
    }
    // gradient records are kept with a tile-major list only
    auto kern = supers ? (want_opacity ? k_blend_bwd<true, false, true> : k_blend_bwd<true, false, false>)
                : records ? (want_opacity ? k_blend_bwd<false, true, true> : k_blend_bwd<false, true, false>)
                          : (want_opacity ? k_blend_bwd<false, false, true> : k_blend_bwd<false, false, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)ntiles), dim3(kBlendThreads), 0, L.st, cam, ranges, vals, rec, d_image, T_final, last, ga.tile_walk, ga.walk_off, ga.grec,
                       (uint32_t)ga.grec_cap, accum, order, taken, supers ? *supers : SuperDev{});
    if (L.prof) L.prof->end(L.st);
}

void preprocess_backward(const Launch& L, const GaussDev& g, const CamDev& cam, float* accum,
                         const GatherDev& ga, const GradsDev& out) {
    if (g.n <= 0) return;
    if (L.prof) L.prof->begin("preprocess_bwd", L.st);
    // a wave a workgroup where there are too few for every CU
    const int nt = g.n < 256 * 256 ? 64 : 256;
    hipLaunchKernelGGL(ga.grec_cap > 0 ? k_preprocess_bwd<true> : k_preprocess_bwd<false>, dim3(blocks_for(g.n, nt)),
                       dim3(nt), 0, L.st, g, cam, accum, ga, out);
    if (L.prof) L.prof->end(L.st);
}

void debug_keys(const Launch& L, const uint2* ranges, const uint32_t* vals, const uint32_t* key, int ntiles,
                uint64_t* keys_out) {
    hipLaunchKernelGGL(k_debug_keys, dim3((unsigned)ntiles), dim3(256), 0, L.st, ranges, vals, key, ntiles, keys_out);
}

void debug_records(const Launch& L, int64_t n, const float4* rec, int32_t* box, float* rec9) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_debug_records, dim3(blocks_for(n, 256)), dim3(256), 0, L.st, n, rec, box, rec9);
}

}  // namespace gs3
