// Neural Transformation Cache on gfx950 (Sec. 4.1, Eq. 5):
//   (dmu, dq) = MLP(h(mu)),  h = multi-resolution hash encoding,
//   MLP = 32 -> 64 (ReLU) -> 64 (ReLU) -> 7, no biases.
//
// Work unit: a batch of 16 points per wave.  Lane l owns point l % 16 and
// levels 4 (l / 16) .. 4 (l / 16) + 3 of the encoding, so the 64 lanes cover
// the 16 x 16 (point, level) pairs of a batch.  Activations go through LDS in
// [point][feature] layout; every layer is a 16 x 16 MFMA tile product
// (v_mfma_f32_16x16x16 f16 / bf16, or 16x16x4 f32), weights staged once per
// workgroup in LDS.  The backward pass recomputes the forward and
// propagates the output gradient through the three layers, each wave on its
// own batch; then the four waves accumulate the weight gradients of the
// four batches with MFMA (contraction over each batch's 16 points) in FP32
// registers, each wave a quarter of the weight tiles; the encoding gradient
// goes to the per-entry sums of the table gradient over the prepared lists, or
// is added to the table's parts in LDS (very large tables: with global
// atomics).
//
// Half-precision backward: each activation-gradient stage is rescaled by a
// power of two so that its largest magnitude in the batch sits near 2^13
// before it is rounded to FP16/BF16; the FP32 results are unscaled exactly.
#include <algorithm>

#include "kernels.h"
#include "ntc.h"

namespace gs3 {

namespace {

// points of a slice of the contribution lists: whole groups of 256
__host__ __device__ __forceinline__ int64_t csr_slice(int64_t n, int slices) {
    return ((n + slices - 1) / slices + 255) / 256 * 256;
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef __bf16 b4v __attribute__((ext_vector_type(4)));

struct PF32 {
    using S = float;
    using AF = float;
    static constexpr int KPL = 1;
    static constexpr int KSTEP = 4;
    __device__ static f4v mfma(AF a, AF b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static S cvt(float x) { return x; }
    __device__ static float tof(S x) { return x; }
    static constexpr bool kScaled = false;
};
struct PF16 {
    using S = _Float16;
    using AF = h4v;
    static constexpr int KPL = 4;
    static constexpr int KSTEP = 16;
    __device__ static f4v mfma(AF a, AF b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0); }
    __device__ static S cvt(float x) { return (S)x; }
    __device__ static float tof(S x) { return (float)x; }
    static constexpr bool kScaled = true;
};
struct PBF16 {
    using S = __bf16;
    using AF = b4v;
    static constexpr int KPL = 4;
    static constexpr int KSTEP = 16;
    __device__ static f4v mfma(AF a, AF b, f4v c) {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
    __device__ static S cvt(float x) { return (S)x; }
    __device__ static float tof(S x) { return (float)x; }
    static constexpr bool kScaled = true;
};

// A or B fragment, elements base[row * ld + k0 + i] (contiguous in k)
template <class P>
__device__ __forceinline__ typename P::AF frag_k_contig(const typename P::S* base, int ld, int row, int k0) {
    typename P::AF f;
    if constexpr (P::KPL == 1) {
        f = base[row * ld + k0];
    } else {
#pragma unroll
        for (int i = 0; i < P::KPL; i++) f[i] = base[row * ld + k0 + i];
    }
    return f;
}
// Fragment with elements base[(k0 + i) * ld + c0 + (lane & 15)] (strided in
// k), k0 the same for the 16 lanes of a group: in the half types one
// transposing read, to which lane j of a group gives the place of four columns
// of row j / 4.
template <class P>
__device__ __forceinline__ typename P::AF frag_k_strided(const typename P::S* base, int ld, int c0, int k0, int lane) {
    const int j = lane & 15;
    if constexpr (P::KPL == 1) {
        return base[k0 * ld + c0 + j];
    } else {
        typedef short s4v __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s4v lds_s4v;
        const typename P::S* at = base + (k0 + (j >> 2)) * ld + c0 + 4 * (j & 3);   // 8-byte aligned
        return __builtin_bit_cast(typename P::AF, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)at));
    }
}

// four consecutive elements, 4-element aligned
template <class P>
__device__ __forceinline__ void store4(typename P::S* at, const typename P::S v[4]) {
    typedef typename P::S s4 __attribute__((ext_vector_type(4)));
    *reinterpret_cast<s4*>(at) = s4{v[0], v[1], v[2], v[3]};
}

// Inside the batch loops each wave works on its own activation arrays in LDS
// (the staged weights are read-only there), so the waves of a workgroup only
// order their own LDS accesses: a wave-level barrier that keeps the compiler
// from moving LDS accesses across it (a wave's LDS operations complete in
// issue order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Row strides (elements) of the LDS arrays; +4 breaks bank regularity.
constexpr int kMlpParams = 64 * 32 + 64 * 64 + 7 * 64;
constexpr int LD32 = 32 + 4;
constexpr int LD64 = 64 + 4;
constexpr int LD16 = 16 + 4;
constexpr int kWaves = 4;
constexpr int kPts = 16;

// the two features of a table entry; the entry's byte offset fits in 32 bits
// (at most 2^26 entries), so the load takes a scalar base and a 32-bit offset
template <class P>
__device__ __forceinline__ float2 load2(const typename P::S* table, uint32_t entry) {
    const unsigned char* base = reinterpret_cast<const unsigned char*>(table);
    const uint32_t off = entry * (uint32_t)(2 * sizeof(typename P::S));
    if constexpr (sizeof(typename P::S) == 4) {
        return *reinterpret_cast<const float2*>(base + off);
    } else {
        typedef typename P::S s2v __attribute__((ext_vector_type(2)));
        const s2v v = *reinterpret_cast<const s2v*>(base + off);
        return make_float2(P::tof(v.x), P::tof(v.y));
    }
}

// normalised position; false when outside [0, 1]^3 (the point is discarded)
__device__ __forceinline__ bool ntc_normalise(const NtcDev& nd, const float* mu, float x[3]) {
#pragma clang fp contract(off)
    bool in = true;
    for (int k = 0; k < 3; k++) {
        x[k] = (mu[k] - nd.aabb_min[k]) * nd.inv_ext[k];
        in = in && (x[k] >= 0.0f) && (x[k] <= 1.0f);
    }
    return in;
}

// corner entries and trilinear weights of level lv
__device__ __forceinline__ void ntc_corners(const NtcDev& nd, int lv, const float x[3], uint32_t ent[8], float wt[8]) {
    float w[3];
    uint32_t i0[3];
    {
#pragma clang fp contract(off)
        const int N = nd.res[lv];
        const float fN = (float)N;
        for (int k = 0; k < 3; k++) {
            const float p = x[k] * fN;
            int c = (int)floorf(p);
            c = c > N - 1 ? N - 1 : c;
            c = c < 0 ? 0 : c;
            i0[k] = (uint32_t)c;
            w[k] = p - (float)c;
        }
    }
    const int N1 = nd.res[lv] + 1;
    const bool dense = (nd.dense_mask >> lv) & 1u;
#pragma unroll
    for (int c = 0; c < 8; c++) {
        const uint32_t vx = i0[0] + (c & 1), vy = i0[1] + ((c >> 1) & 1), vz = i0[2] + ((c >> 2) & 1);
        uint32_t idx;
        if (dense)
            idx = vx + (uint32_t)N1 * (vy + (uint32_t)N1 * vz);
        else
            idx = ((vx * 1u) ^ (vy * 2654435761u) ^ (vz * 805459861u)) & nd.T_mask;
        ent[c] = (uint32_t)nd.off[lv] + idx;
        wt[c] = ((c & 1) ? w[0] : 1.0f - w[0]) * (((c >> 1) & 1) ? w[1] : 1.0f - w[1]) *
                (((c >> 2) & 1) ? w[2] : 1.0f - w[2]);
    }
}

template <class P>
using Pair = typename P::S __attribute__((ext_vector_type(2)));

// The weights to LDS, by 256 threads.  Every load is issued before the first
// store (pairs: what the parameters' alignment allows); with a load and its
// store per round, the rounds' latencies add up to a third of a launch on few
// points.
template <class P>
__device__ __forceinline__ void load_weights(const typename P::S* __restrict__ mlp, typename P::S* sW1,
                                             typename P::S* sW2, typename P::S* sW3, typename P::S* sW1t,
                                             typename P::S* sW2t, typename P::S* sW3t) {
    using S = typename P::S;
    constexpr int kPairs = kMlpParams / 2, kN = (kPairs + 255) / 256;
    constexpr int kW2 = 64 * 32 / 2 / 256, kW3 = kW2 + 64 * 64 / 2 / 256;   // first rounds of W2 and W3
    static_assert(kW2 * 256 == 64 * 32 / 2 && (kW3 - kW2) * 256 == 64 * 64 / 2 && kN == kW3 + 1, "whole rounds");
    const int t = threadIdx.x;
    Pair<P> v[kN];
#pragma unroll
    for (int u = 0; u < kN; u++)
        v[u] = t + 256 * u < kPairs ? reinterpret_cast<const Pair<P>*>(mlp)[t + 256 * u] : Pair<P>{P::cvt(0.f), P::cvt(0.f)};
    auto put = [](S* a, S* at, int r, int c, int ld, int ldt, Pair<P> x) {
        if (a) {
            a[r * ld + c] = x.x;
            a[r * ld + c + 1] = x.y;
        }
        if (at) {
            at[c * ldt + r] = x.x;
            at[(c + 1) * ldt + r] = x.y;
        }
    };
#pragma unroll
    for (int u = 0; u < kW2; u++) put(sW1, sW1t, (t + 256 * u) / 16, (t + 256 * u) % 16 * 2, LD32, LD64, v[u]);
#pragma unroll
    for (int u = kW2; u < kW3; u++) {
        const int k = t + 256 * (u - kW2);
        put(sW2, sW2t, k / 32, k % 32 * 2, LD64, LD64, v[u]);
    }
    // W3 has 7 rows; rows 7 .. 15 are zero
    put(sW3, sW3t, t / 32, t % 32 * 2, LD64, LD16, v[kW3]);
    put(sW3, sW3t, 8 + t / 32, t % 32 * 2, LD64, LD16, Pair<P>{P::cvt(0.f), P::cvt(0.f)});
}

// D (16 x 16, rows m0.., cols = points) += W[m0..m0+15][0..K) X[p][0..K)
template <class P, int K>
__device__ __forceinline__ f4v layer_tile(const typename P::S* W, int ldw, int m0, const typename P::S* X, int ldx,
                                          int lane) {
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    const int row = lane & 15, g = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < K / P::KSTEP; ks++) {
        const int k0 = ks * P::KSTEP + P::KPL * g;
        acc = P::mfma(frag_k_contig<P>(W, ldw, m0 + row, k0), frag_k_contig<P>(X, ldx, row, k0), acc);
    }
    return acc;
}
// The same with W^T, from W in the half types and from a transposed copy Wt in
// float, whose transposed reads would meet on the banks.
template <class P, int K>
__device__ __forceinline__ f4v layer_tile_t(const typename P::S* W, int ldw, const typename P::S* Wt, int ldt, int m0,
                                            const typename P::S* X, int ldx, int lane) {
    if constexpr (P::KPL == 1) return layer_tile<P, K>(Wt, ldt, m0, X, ldx, lane);
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    const int row = lane & 15, g = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < K / P::KSTEP; ks++) {
        const int k0 = ks * P::KSTEP + P::KPL * g;
        acc = P::mfma(frag_k_strided<P>(W, ldw, m0, k0, lane), frag_k_contig<P>(X, ldx, row, k0), acc);
    }
    return acc;
}
// A layer's outputs (ReLU, rounded) of a lane, to LDS and kept in v.
template <class P>
__device__ __forceinline__ void relu_out(const f4v& a, typename P::S* at, typename P::S v[4]) {
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = P::cvt(fmaxf(a[r], 0.f));
    store4<P>(at, v);
}

// encode this lane's 4 levels of its point into X[p][8 g .. 8 g + 7]
template <class P>
__device__ __forceinline__ void encode_lane(const NtcDev& nd, const typename P::S* __restrict__ table,
                                            const float x[3], int g, typename P::S* X, int p) {
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int lv = 4 * g + j;
        uint32_t ent[8];
        float wt[8];
        ntc_corners(nd, lv, x, ent, wt);
        float e0 = 0.f, e1 = 0.f;
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const float2 v = load2<P>(table, ent[c]);
            e0 += wt[c] * v.x;
            e1 += wt[c] * v.y;
        }
        X[p * LD32 + 2 * lv] = P::cvt(e0);
        X[p * LD32 + 2 * lv + 1] = P::cvt(e1);
    }
}

// The encoding in memory: [level][point][2], so that a wave that encodes one
// level stores consecutive words.
template <class P>
__device__ __forceinline__ void enc_put(typename P::S* enc, int64_t n, int lv, int64_t pt, typename P::S a,
                                        typename P::S b) {
    reinterpret_cast<Pair<P>*>(enc)[lv * n + pt] = Pair<P>{a, b};
}
// a lane's eight values: levels 4 g .. 4 g + 3 of point pt
template <class P>
__device__ __forceinline__ void enc_get(const typename P::S* enc, int64_t n, int g, int64_t pt, typename P::S v[8]) {
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const Pair<P> w = reinterpret_cast<const Pair<P>*>(enc)[(4 * g + j) * n + pt];
        v[2 * j] = w.x;
        v[2 * j + 1] = w.y;
    }
}

// The encoding of many points: a workgroup holds one level of the table in
// LDS, an entry a word, and encodes its slice of the points from there.  From
// global memory a point's 128 corners are that many L2 requests, some 320 a
// ns; LDS serves them several times faster, and what bounds the kernel now is
// the arithmetic of the corners.  300K points in fp16, encoding and MLP: 109
// us with points in random order and 58 in Morton order -> 44 (encoding 24,
// MLP 20); 50K 27 and 19 -> 16.  The float table's levels do not fit: as two
// passes over a feature each, 300K points took 115 us for 123 and 95.
constexpr int kEncEntries = 32768;   // entries of a level in LDS (128 KB)
template <class P>
__global__ __launch_bounds__(1024) void k_ntc_encode(NtcDev nd, const typename P::S* __restrict__ table,
                                                     const float* __restrict__ means, int64_t n, int slices,
                                                     typename P::S* __restrict__ enc) {
    static_assert(sizeof(Pair<P>) == 4, "an entry is a word");
    __shared__ uint32_t s_t[kEncEntries];
    // a slice's workgroups have the same blockIdx.x mod 8, hence the same XCD,
    // whose L2 then holds the slice's means (slices is a multiple of 8)
    const int slice = blockIdx.x % slices, lv = blockIdx.x / slices;
    const int size = (int)nd.level_size(lv);
    const uint32_t first = (uint32_t)nd.off[lv];
    {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(table) + first;
        int k = threadIdx.x;
        for (; k + 7 * 1024 < size; k += 8 * 1024) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) v[u] = src[k + 1024 * u];
#pragma unroll
            for (int u = 0; u < 8; u++) s_t[k + 1024 * u] = v[u];
        }
        for (; k < size; k += 1024) s_t[k] = src[k];
    }
    __syncthreads();
    const int64_t per = (n + slices - 1) / slices, p1 = min(n, (slice + 1) * per);
    int64_t pt = slice * per + threadIdx.x;
    float mu[3] = {0.f, 0.f, 0.f};
    auto load = [&](int64_t q) {
        if (q < p1) {
            mu[0] = means[3 * q];
            mu[1] = means[3 * q + 1];
            mu[2] = means[3 * q + 2];
        }
    };
    load(pt);
    for (; pt < p1; pt += 1024) {
        float x[3];
        const bool in = ntc_normalise(nd, mu, x);
        load(pt + 1024);   // a round ahead
        float e0 = 0.f, e1 = 0.f;
        if (in) {
            uint32_t ent[8];
            float wt[8];
            ntc_corners(nd, lv, x, ent, wt);
#pragma unroll
            for (int c = 0; c < 8; c++) {
                const Pair<P> v = __builtin_bit_cast(Pair<P>, s_t[ent[c] - first]);
                e0 += wt[c] * P::tof(v.x);
                e1 += wt[c] * P::tof(v.y);
            }
        }
        enc_put<P>(enc, n, lv, pt, P::cvt(e0), P::cvt(e1));
    }
}

// kGiven: enc holds the points' encoding; else they are encoded here, and the
// encoding is stored in enc, if given, for the backward.
template <class P, bool kGiven>
__global__ __launch_bounds__(256, 4) void k_ntc_fwd(NtcDev nd, const typename P::S* __restrict__ table,
                                                 const typename P::S* __restrict__ mlp, const float* __restrict__ means,
                                                 int64_t n, float* __restrict__ dmu, float* __restrict__ dq,
                                                 typename P::S* __restrict__ enc) {
    using S = typename P::S;
    __shared__ __align__(16) S sW1[64 * LD32], sW2[64 * LD64], sW3[16 * LD64];
    __shared__ __align__(16) S sX[kWaves][kPts * LD32], sH1[kWaves][kPts * LD64], sH2[kWaves][kPts * LD64];
    load_weights<P>(mlp, sW1, sW2, sW3, nullptr, nullptr, nullptr);
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = lane & 15, g = lane >> 4;
    S* X = sX[w];
    S* H1 = sH1[w];
    S* H2 = sH2[w];
    const int64_t nb = (n + kPts - 1) / kPts;
    // each batch's inputs are loaded one round ahead
    float nmu[3] = {0.f, 0.f, 0.f};
    S nenc[8];
    auto prefetch = [&](int64_t bb) {
        const int64_t q = (bb + w) * kPts + p;
        if (bb < nb && q < n) {
            nmu[0] = means[3 * q];
            nmu[1] = means[3 * q + 1];
            nmu[2] = means[3 * q + 2];
            if constexpr (kGiven) enc_get<P>(enc, n, g, q, nenc);
        }
    };
    prefetch((int64_t)blockIdx.x * kWaves);
    for (int64_t b0 = (int64_t)blockIdx.x * kWaves; b0 < nb; b0 += (int64_t)gridDim.x * kWaves) {
        const int64_t pt = (b0 + w) * kPts + p;
        const bool valid = pt < n;
        float x[3] = {0.f, 0.f, 0.f};
        bool in = false;
        if (valid) in = ntc_normalise(nd, nmu, x);
        if constexpr (!kGiven) prefetch(b0 + (int64_t)gridDim.x * kWaves);
        wave_sync();   // previous batch's reads of X done
        if (kGiven && valid) {
#pragma unroll
            for (int j = 0; j < 8; j++) X[p * LD32 + 8 * g + j] = nenc[j];
        } else if (!kGiven && in) {
            encode_lane<P>(nd, table, x, g, X, p);
        } else {
            for (int j = 0; j < 8; j++) X[p * LD32 + 8 * g + j] = P::cvt(0.f);
        }
        if constexpr (kGiven) prefetch(b0 + (int64_t)gridDim.x * kWaves);
        wave_sync();
        if (!kGiven && enc && valid) {
#pragma unroll
            for (int j = 0; j < 4; j++)
                enc_put<P>(enc, n, 4 * g + j, pt, X[p * LD32 + 8 * g + 2 * j], X[p * LD32 + 8 * g + 2 * j + 1]);
        }
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            const f4v a = layer_tile<P, 32>(sW1, LD32, mt * 16, X, LD32, lane);
            S v[4];
            relu_out<P>(a, H1 + p * LD64 + mt * 16 + 4 * g, v);
        }
        wave_sync();
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            const f4v a = layer_tile<P, 64>(sW2, LD64, mt * 16, H1, LD64, lane);
            S v[4];
            relu_out<P>(a, H2 + p * LD64 + mt * 16 + 4 * g, v);
        }
        wave_sync();
        const f4v o = layer_tile<P, 64>(sW3, LD64, 0, H2, LD64, lane);
        if (valid && g < 2) {
            if (g == 0) {
                dmu[3 * pt + 0] = in ? o[0] : 0.f;
                dmu[3 * pt + 1] = in ? o[1] : 0.f;
                dmu[3 * pt + 2] = in ? o[2] : 0.f;
                dq[4 * pt + 0] = in ? o[3] : 1.f;
            } else {
                dq[4 * pt + 1] = in ? o[0] : 0.f;
                dq[4 * pt + 2] = in ? o[1] : 0.f;
                dq[4 * pt + 3] = in ? o[2] : 0.f;
            }
        }
    }
}

// v or its neighbour's by a DPP pattern, the larger (lanes without one keep v)
template <int kCtrl, int kRows>
__device__ __forceinline__ float dpp_max(float v) {
    const int i = __float_as_int(v);
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(i, i, kCtrl, kRows, 0xF, false)));
}
__device__ __forceinline__ float wave_max(float v) {   // patterns as in wave_sum_dpp
    v = dpp_max<0xB1, 0xF>(v);
    v = dpp_max<0x4E, 0xF>(v);
    v = dpp_max<0x141, 0xF>(v);
    v = dpp_max<0x140, 0xF>(v);
    v = dpp_max<0x142, 0xA>(v);
    v = dpp_max<0x143, 0xC>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// exponent k of the power of two 2^k with max * 2^k in [2^12, 2^13); 0 when
// max is 0 or not finite
__device__ __forceinline__ int pow2_exp(float mx) {
    if (!(mx > 0.f) || !isfinite(mx)) return 0;
    int e;
    frexpf(mx, &e);   // mx = f 2^e, f in [0.5, 1)
    return 13 - e;
}

// the scale exponents stay inside the normal range of float, so 2^k and
// 2^-k are exact
__device__ __forceinline__ int clamp_exp(int k) { return k < -126 ? -126 : (k > 126 ? 126 : k); }

// The encoding gradient goes to `denc` (level-major, n x 32 floats), for the
// per-entry gather of the prepared contribution lists or the scatter.
//
// Each iteration takes four batches, one per wave.  Phase A (each wave on its
// own batch): the encoding, the forward layers, the output gradient and the
// activation gradients of the three layers, all kept in the wave's LDS
// arrays (activations and gradients side by side), and the encoding
// gradient.  Phase B (after a workgroup barrier): the weight gradients of
// all four batches, split between the waves by output rows (wave w: the 16
// rows 16 w.. of dW1 and dW2 and the 16 columns 16 w.. of dW3), so a wave
// holds 7 accumulator tiles instead of 28 and the register file leaves room
// for more than one wave per SIMD.
// Two workgroups' registers per SIMD and LDS per CU; bound by instructions
// issued (by either of a SIMD's two waves in 7 cycles of 10, the vector ALU in 4),
// so fragments strided in the points are read transposed (four 2-byte
// reads and their packing each, else), W1 and W2 are read either way from one
// copy, a lane keeps its activations for the masks, and with two waves to a
// SIMD the accumulators need no AGPRs (184 moves from them): 300K points fp16
// 62 -> 47 us, 20,011 bf16 with the encoding 22 -> 19.
//
// kScatter (means without lists, tables of more than kLdsParts parts): a lane
// adds the gradients of its four levels to the table with global atomics, whose
// rate of some 20 per ns bounds the launch; the rest hides behind them (a
// launch of their own for the atomics, on the stored encoding gradient: 300K
// points at T = 2^17 4.19 for 3.91 ms, at 2^19 4.23 for 3.92).
template <class P, bool kScatter>
__global__ __launch_bounds__(256, 2) void k_ntc_bwd(NtcDev nd, const typename P::S* __restrict__ table,
                                                 const typename P::S* __restrict__ mlp, const float* __restrict__ means,
                                                 int64_t n, const float* __restrict__ d_dmu,
                                                 const float* __restrict__ d_dq, float* __restrict__ g_part,
                                                 float* __restrict__ denc,
                                                 const typename P::S* __restrict__ enc_in,
                                                 float* __restrict__ g_table) {
    using S = typename P::S;
    constexpr bool kCopies = P::KPL == 1;   // transposed copies of W1 and W2: see layer_tile_t
    constexpr int kWElems = 64 * LD32 + 64 * LD64 + 64 * LD16 + (kCopies ? 32 * LD64 + 64 * LD64 : 0);
    __shared__ __align__(16) S sWraw[kWElems];
    S* sW1 = sWraw;
    S* sW2 = sW1 + 64 * LD32;
    S* sW3t = sW2 + 64 * LD64;
    S* sW1t = kCopies ? sW3t + 64 * LD16 : nullptr;
    S* sW2t = kCopies ? sW1t + 32 * LD64 : nullptr;
    // per wave: encoding, activations, their gradients, output gradient
    __shared__ __align__(16) S sX[kWaves][kPts * LD32], sH1[kWaves][kPts * LD64], sH2[kWaves][kPts * LD64];
    __shared__ __align__(16) S sD1[kWaves][kPts * LD64], sD2[kWaves][kPts * LD64];
    __shared__ __align__(16) S sO[kWaves][kPts * LD16];
    __shared__ int sK[kWaves][3];   // each batch's scale exponents k0, k1, k2
    load_weights<P>(mlp, sW1, sW2, nullptr, sW1t, sW2t, sW3t);
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = lane & 15, g = lane >> 4, col = lane & 15;
    S* X = sX[w];
    S* H1 = sH1[w];
    S* H2 = sH2[w];
    S* D1 = sD1[w];
    S* D2 = sD2[w];
    S* O = sO[w];
    // this wave's weight-gradient tiles: dW1 rows 16 w.. (2 column tiles),
    // dW2 rows 16 w.. (4 column tiles), dW3 columns 16 w..
    f4v gW1[2], gW2[4], gW3;
    for (int a = 0; a < 2; a++) gW1[a] = f4v{0.f, 0.f, 0.f, 0.f};
    for (int a = 0; a < 4; a++) gW2[a] = f4v{0.f, 0.f, 0.f, 0.f};
    gW3 = f4v{0.f, 0.f, 0.f, 0.f};
    // the level slices this lane writes in the level-major encoding gradient:
    // levels 2 g and 8 + 2 g (and the level after each)
    float2* const dlev[2] = {reinterpret_cast<float2*>(denc) + (int64_t)(2 * g) * n,
                             reinterpret_cast<float2*>(denc) + (int64_t)(8 + 2 * g) * n};
    const int64_t nb = (n + kPts - 1) / kPts;
    // the inputs of this wave's batch are loaded one round ahead, so that
    // their latency overlaps the previous round's work
    float nmu[3] = {0.f, 0.f, 0.f}, ndv[4] = {0.f, 0.f, 0.f, 0.f};
    S nenc[8];
    auto prefetch = [&](int64_t bb) {
        const int64_t q = (bb + w) * kPts + p;
        if (bb < nb && q < n) {
            nmu[0] = means[3 * q];
            nmu[1] = means[3 * q + 1];
            nmu[2] = means[3 * q + 2];
            if (enc_in) enc_get<P>(enc_in, n, g, q, nenc);
            if (g == 0) {
                ndv[0] = d_dmu[3 * q];
                ndv[1] = d_dmu[3 * q + 1];
                ndv[2] = d_dmu[3 * q + 2];
                ndv[3] = d_dq[4 * q];
            } else if (g == 1) {
                ndv[0] = d_dq[4 * q + 1];
                ndv[1] = d_dq[4 * q + 2];
                ndv[2] = d_dq[4 * q + 3];
            }
        }
    };
    prefetch((int64_t)blockIdx.x * kWaves);
    for (int64_t b0 = (int64_t)blockIdx.x * kWaves; b0 < nb; b0 += (int64_t)gridDim.x * kWaves) {
        // ---------------- phase A: this wave's batch ----------------
        const int64_t pt = (b0 + w) * kPts + p;
        const bool valid = pt < n;   // false for every lane of a wave past the last batch
        float x[3] = {0.f, 0.f, 0.f};
        bool in = false;
        if (valid) in = ntc_normalise(nd, nmu, x);
        // 1. encoding: the forward's, when it kept it, else recomputed
        if (enc_in && valid) {
#pragma unroll
            for (int j = 0; j < 8; j++) X[p * LD32 + 8 * g + j] = nenc[j];
        } else if (in) {
            encode_lane<P>(nd, table, x, g, X, p);
        } else {
            for (int j = 0; j < 8; j++) X[p * LD32 + 8 * g + j] = P::cvt(0.f);
        }
        // output gradient (lanes of group 0 own the 7 outputs of their point)
        float dv[4] = {0.f, 0.f, 0.f, 0.f};
        if (in && g <= 1) {
#pragma unroll
            for (int r = 0; r < 4; r++) dv[r] = ndv[r];
        }
        prefetch(b0 + (int64_t)gridDim.x * kWaves);
        // the activation gradients of this batch are held scaled by 2^k0,
        // 2^k1, 2^k2 (exact powers of two; the weight gradients unscale them)
        int k0 = 0;
        if (P::kScaled)
            k0 = clamp_exp(pow2_exp(wave_max(fmaxf(fmaxf(fabsf(dv[0]), fabsf(dv[1])), fmaxf(fabsf(dv[2]), fabsf(dv[3]))))));
        const float s0 = ldexpf(1.0f, k0);
        {
            S v[4];
            for (int r = 0; r < 4; r++) v[r] = P::cvt(dv[r] * s0);   // rows 8..15 stay zero
            store4<P>(O + p * LD16 + 4 * g, v);
        }
        wave_sync();
        // 2. forward recompute; a lane's activations stay for the masks
        S h1[4][4], h2[4][4];
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            const f4v a = layer_tile<P, 32>(sW1, LD32, mt * 16, X, LD32, lane);
            relu_out<P>(a, H1 + p * LD64 + mt * 16 + 4 * g, h1[mt]);
        }
        wave_sync();
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            const f4v a = layer_tile<P, 64>(sW2, LD64, mt * 16, H1, LD64, lane);
            relu_out<P>(a, H2 + p * LD64 + mt * 16 + 4 * g, h2[mt]);
        }
        wave_sync();
        // 3. dH2 = (W3^T dO) * [H2 > 0]
        f4v d2[4];
        float m2 = 0.f;
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            d2[mt] = layer_tile<P, 16>(sW3t, LD16, mt * 16, O, LD16, lane);
            for (int r = 0; r < 4; r++) {
                const bool on = P::tof(h2[mt][r]) > 0.f;
                d2[mt][r] = on ? d2[mt][r] : 0.f;
                m2 = fmaxf(m2, fabsf(d2[mt][r]));
            }
        }
        int k1 = k0;
        if (P::kScaled) k1 = clamp_exp(k0 + pow2_exp(wave_max(m2)));
        {
            const float f = ldexpf(1.0f, k1 - k0);
            for (int mt = 0; mt < 4; mt++) {
                S v[4];
                for (int r = 0; r < 4; r++) v[r] = P::cvt(d2[mt][r] * f);
                store4<P>(D2 + p * LD64 + mt * 16 + 4 * g, v);
            }
        }
        wave_sync();
        // 4. dH1 = (W2^T dH2) * [H1 > 0]
        f4v d1[4];
        float m1 = 0.f;
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            d1[mt] = layer_tile_t<P, 64>(sW2, LD64, sW2t, LD64, mt * 16, D2, LD64, lane);
            for (int r = 0; r < 4; r++) {
                const bool on = P::tof(h1[mt][r]) > 0.f;
                d1[mt][r] = on ? d1[mt][r] : 0.f;
                m1 = fmaxf(m1, fabsf(d1[mt][r]));
            }
        }
        int k2 = k1;
        if (P::kScaled) k2 = clamp_exp(k1 + pow2_exp(wave_max(m1)));
        {
            const float f = ldexpf(1.0f, k2 - k1);
            for (int mt = 0; mt < 4; mt++) {
                S v[4];
                for (int r = 0; r < 4; r++) v[r] = P::cvt(d1[mt][r] * f);
                store4<P>(D1 + p * LD64 + mt * 16 + 4 * g, v);
            }
        }
        if (lane == 0) {
            sK[w][0] = k0;
            sK[w][1] = k1;
            sK[w][2] = k2;
        }
        wave_sync();
        // 5. dX = W1^T dH1: the encoding gradient
        {
            const float inv = ldexpf(1.0f, -k2);
#pragma unroll
            for (int mt = 0; mt < 2; mt++) {
                const f4v e = layer_tile_t<P, 64>(sW1, LD32, sW1t, LD64, mt * 16, D1, LD64, lane);
                if constexpr (kScatter) {
                    if (in) {
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            uint32_t ent[8];
                            float wt[8];
                            ntc_corners(nd, 8 * mt + 2 * g + j, x, ent, wt);
                            const float e0 = e[2 * j] * inv, e1 = e[2 * j + 1] * inv;
#pragma unroll
                            for (int c = 0; c < 8; c++) {
                                atomicAdd(g_table + 2 * (int64_t)ent[c], wt[c] * e0);
                                atomicAdd(g_table + 2 * (int64_t)ent[c] + 1, wt[c] * e1);
                            }
                        }
                    }
                } else if (valid) {
                    // level-major [level][point][2]: one level's slice (8 n bytes)
                    // stays cache-resident while the gather walks that level
                    float2* d = dlev[mt] + pt;
                    d[0] = make_float2(e[0] * inv, e[1] * inv);
                    d[n] = make_float2(e[2] * inv, e[3] * inv);   // level lv + 1
                }
            }
        }
        __syncthreads();
        // ---------------- phase B: weight gradients of the four batches ----------------
#pragma unroll
        for (int b = 0; b < kWaves; b++) {
            const float inv0 = ldexpf(1.0f, -sK[b][0]);
            const float inv1 = ldexpf(1.0f, -sK[b][1]);
            const float inv2 = ldexpf(1.0f, -sK[b][2]);
            // dW3[o][m] += sum_p dO[p][o] H2[p][m], columns m = 16 w..
            {
                f4v t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < kPts / P::KSTEP; ks++) {
                    const int kk = ks * P::KSTEP + P::KPL * g;
                    t = P::mfma(frag_k_strided<P>(sO[b], LD16, 0, kk, lane),
                                frag_k_strided<P>(sH2[b], LD64, w * 16, kk, lane), t);
                }
                gW3 += t * inv0;
            }
            // dW2[m][k] += sum_p dH2[p][m] H1[p][k], rows m = 16 w..
#pragma unroll
            for (int nt = 0; nt < 4; nt++) {
                f4v t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < kPts / P::KSTEP; ks++) {
                    const int kk = ks * P::KSTEP + P::KPL * g;
                    t = P::mfma(frag_k_strided<P>(sD2[b], LD64, w * 16, kk, lane),
                                frag_k_strided<P>(sH1[b], LD64, nt * 16, kk, lane), t);
                }
                gW2[nt] += t * inv1;
            }
            // dW1[m][k] += sum_p dH1[p][m] X[p][k], rows m = 16 w..
#pragma unroll
            for (int nt = 0; nt < 2; nt++) {
                f4v t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < kPts / P::KSTEP; ks++) {
                    const int kk = ks * P::KSTEP + P::KPL * g;
                    t = P::mfma(frag_k_strided<P>(sD1[b], LD64, w * 16, kk, lane),
                                frag_k_strided<P>(sX[b], LD32, nt * 16, kk, lane), t);
                }
                gW1[nt] += t * inv2;
            }
        }
        __syncthreads();   // phase B's reads done before the next batches are written
    }
    // weight-gradient partials of this workgroup: every wave writes its own
    // tiles (they are disjoint and cover the MLP's parameters once)
    float* out = g_part + (int64_t)blockIdx.x * kMlpParams;
    for (int nt = 0; nt < 2; nt++)
        for (int r = 0; r < 4; r++) out[(w * 16 + 4 * g + r) * 32 + nt * 16 + col] = gW1[nt][r];
    for (int nt = 0; nt < 4; nt++)
        for (int r = 0; r < 4; r++) out[64 * 32 + (w * 16 + 4 * g + r) * 64 + nt * 16 + col] = gW2[nt][r];
    for (int r = 0; r < 4; r++)
        if (4 * g + r < 7) out[64 * 32 + 64 * 64 + (4 * g + r) * 64 + w * 16 + col] = gW3[r];
}

// The table cut into parts of one level, for the kernels that hold a part in
// LDS and read the points again for each.
constexpr int kLdsEntries = 8192;    // entries of a part: two doubles each (128 KB),
constexpr int kListEntries = 32768;  // or a counter each (128 KB)
constexpr int kLdsParts = 128;       // most parts of the table for which the points are read again

struct TableParts {
    int level[kLdsParts];
    int first[kLdsParts];   // first entry of the part in its level
    int size[kLdsParts];
    int count = 0;
};

static bool table_parts(const NtcDev& nd, int part, TableParts& tp) {
    for (int lv = 0; lv < 16; lv++) {
        const int64_t size = nd.level_size(lv);
        for (int64_t f = 0; f < size; f += part) {
            if (tp.count == kLdsParts) return false;
            tp.level[tp.count] = lv;
            tp.first[tp.count] = (int)f;
            tp.size[tp.count++] = (int)std::min<int64_t>(part, size - f);
        }
    }
    return true;
}

// ---------------------------------------------------------------------------
// Per-frame contribution lists.  The means are frozen during Stage 1, so
// every (point, level, corner) contribution to the table gradient has a fixed
// entry and a fixed trilinear weight for the whole frame.  They are sorted
// by entry once; each iteration then sums, per entry, weight x encoding
// gradient of the contributing points (no atomics, fixed summation order).
//
// The lists are built by counting: a workgroup counts a slice of the points
// into the entries of one part of the table in LDS, the counts of (slice,
// entry) are turned into first slots (entry by entry, slice by slice), and a
// workgroup per (part, slice) walks its points in order with the slots in LDS
// and stores each contribution where its entry's counter says.  Its sixteen
// waves take a group of 64 points each and compute its corners and store on
// their own; only the slots are taken in turn, group after group (s_turn).  A
// wave's LDS operations are done in order, so a list is ordered by groups of 64
// points, then corner, then the order in which the LDS serves the lanes of one
// instruction.  The ISA leaves that order open; no other wave has a part in it,
// and on this chip it depends on the addresses alone: the same means give the
// same lists (the sort below orders them by construction).  Bound by the scattered 8-byte stores (an entry's list is one of
// 32768 that a workgroup appends to, more lines than an L2 holds) and, with
// points in spatial order, by the atomics of lanes on one entry.  300K points,
// T = 2^15, with the means' Morton reorder: 1.85 ms with a radix sort of (entry,
// contribution) pairs -> 0.53 ms.  The placing alone, against four waves that
// meet at a barrier for every turn: 284 -> 256 us (random order 474 -> 456), 2000
// points 44 -> 19.  Lanes of one entry counted as one: 256 -> 538; the table in
// two passes of half the entries: 315.  Tables of more than kLdsParts parts (T
// above 2^18) still take the sort.
// ---------------------------------------------------------------------------
// Points from which the lists are kept slice by slice (backward of points in
// Morton order all over the box, on surfaces, and in random order; entry by
// entry and slice by slice: 100K 81 78 86 and 86 85 88 us, 150K 105 96 117 and
// 120 115 123, 200K 142 130 163 and 136 136 134, 300K 210 204 264 and 176 178
// 174, 600K 427 398 572 and 338 336 342).
constexpr int64_t kChunkMin = 220000;
constexpr int kChunkPoints = 79 * 256;   // points of a slice at most: 158 KB of LDS in k_csr_chunk
static_assert(kChunkPoints <= 1 << 15 && kListEntries <= 1 << 15, "chunk_word");

// a contribution's word in lists kept slice by slice: entry of the level, point of the slice
__device__ __forceinline__ uint32_t chunk_word(uint32_t entry, uint32_t point) { return entry << 15 | point; }

__global__ __launch_bounds__(1024) void k_csr_count(NtcDev nd, TableParts tp, const float* __restrict__ means, int64_t n,
                                                    int slices, int64_t entries, uint32_t* __restrict__ cnt) {
    __shared__ uint32_t s_n[kListEntries];
    const int part = blockIdx.x / slices, slice = blockIdx.x % slices;
    const int lv = tp.level[part], size = tp.size[part];
    const uint32_t first = (uint32_t)nd.off[lv] + (uint32_t)tp.first[part];
    for (int k = threadIdx.x; k < size; k += 1024) s_n[k] = 0u;
    __syncthreads();
    const int64_t per = csr_slice(n, slices), p0 = slice * per, p1 = min(n, p0 + per);
    const int64_t rows = (per + 1023) / 1024;   // points of one thread, next to each other: see k_table_lds
    for (int64_t r = 0; r < rows; r++) {
        const int64_t pt = p0 + (int64_t)threadIdx.x * rows + r;
        if (pt >= p1) break;
        const float mu[3] = {means[3 * pt], means[3 * pt + 1], means[3 * pt + 2]};
        float x[3];
        if (!ntc_normalise(nd, mu, x)) continue;
        uint32_t ent[8];
        float wt[8];
        ntc_corners(nd, lv, x, ent, wt);
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const uint32_t k = ent[c] - first;
            if (k < (uint32_t)size) atomicAdd(&s_n[k], 1u);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < size; k += 1024) cnt[(int64_t)slice * entries + first + k] = s_n[k];
    if (blockIdx.x == 0 && threadIdx.x == 0) cnt[slices * entries] = 0u;   // the lists' end, once scanned
}

// contributions per entry
__global__ __launch_bounds__(256) void k_csr_totals(const uint32_t* __restrict__ cnt, int slices, int64_t entries,
                                                    uint32_t* __restrict__ total) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= entries) return;
    uint32_t s = 0u;
    for (int k = 0; k < slices; k++) s += cnt[k * entries + e];
    total[e] = s;
}

// first[e] (exclusive scan of the totals) -> rows[e] and, in place of each
// (slice, entry) count, its first slot
__global__ __launch_bounds__(256) void k_csr_slots(uint32_t* __restrict__ cnt, int slices, int64_t entries,
                                                   const uint32_t* __restrict__ first, uint2* __restrict__ rows) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= entries) return;
    uint32_t run = first[e];
    const uint32_t begin = run;
    for (int k = 0; k < slices; k++) {
        const uint32_t v = cnt[k * entries + e];
        cnt[k * entries + e] = run;
        run += v;
    }
    rows[e] = make_uint2(begin, run);
}

constexpr int kPlaceThreads = 1024;
__global__ __launch_bounds__(kPlaceThreads) void k_csr_place(NtcDev nd, TableParts tp, const float* __restrict__ means,
                                                             int64_t n, int slices, int64_t entries,
                                                             const uint32_t* __restrict__ slot, bool chunked,
                                                             uint2* __restrict__ pw) {
    constexpr int NW = kPlaceThreads / 64;
    __shared__ uint32_t s_at[kListEntries];
    __shared__ int s_turn;   // the group of 64 points that takes its slots next
    const int part = blockIdx.x / slices, slice = blockIdx.x % slices;
    const int lv = tp.level[part], size = tp.size[part];
    const uint32_t first = (uint32_t)nd.off[lv] + (uint32_t)tp.first[part];
    const uint32_t* src = slot + (int64_t)slice * entries + first;
    for (int k = threadIdx.x; k < size; k += kPlaceThreads) s_at[k] = src[k];
    if (threadIdx.x == 0) s_turn = 0;
    __syncthreads();
    const int64_t per = csr_slice(n, slices), p0 = slice * per, p1 = min(n, p0 + per);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int groups = p1 > p0 ? (int)((p1 - p0 + 63) / 64) : 0;
    float mu[3] = {0.f, 0.f, 0.f};
    auto load = [&](int64_t pt) {
        if (pt < p1) {
            mu[0] = means[3 * pt];
            mu[1] = means[3 * pt + 1];
            mu[2] = means[3 * pt + 2];
        }
    };
    load(p0 + 64 * w + lane);
    for (int g = w; g < groups; g += NW) {
        const int64_t pt = p0 + 64 * (int64_t)g + lane;
        float x[3];
        const bool in = ntc_normalise(nd, mu, x) && pt < p1;
        load(pt + 64 * NW);   // the next group's means arrive during this one's work
        uint32_t ent[8];
        float wt[8];
        ntc_corners(nd, lv, x, ent, wt);
        // the groups' turns come in order, each ends before the next begins,
        // and the wave of every group is on the CU: the wait ends
        while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&s_turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != g)
            __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        uint32_t at[8];
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const uint32_t k = ent[c] - first;
            at[c] = 0u;
            if (in && k < (uint32_t)size) at[c] = atomicAdd(&s_at[k], 1u);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // the wave's LDS operations are done
        if (lane == 0) __hip_atomic_store(&s_turn, g + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // the means are waited for here: behind the stores, the wait would be theirs too
        asm volatile("" : "+v"(mu[0]), "+v"(mu[1]), "+v"(mu[2]));
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const uint32_t k = ent[c] - first;
            if (in && k < (uint32_t)size)
                pw[at[c]] = make_uint2(chunked ? chunk_word(k, (uint32_t)(pt - p0))
                                               : ((uint32_t)pt << 7) | ((uint32_t)lv << 3) | (uint32_t)c,
                                       __float_as_uint(wt[c]));
        }
    }
}

// The sort, for large tables: contributions keyed by entry.
__global__ __launch_bounds__(256) void k_csr_contrib(NtcDev nd, const float* __restrict__ means, int64_t n,
                                                     uint32_t sentinel, uint32_t* __restrict__ key,
                                                     uint32_t* __restrict__ pid) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;   // (point, level)
    if (t >= n * 16) return;
    const int64_t pt = t >> 4;
    const int lv = (int)(t & 15);
    const float mu[3] = {means[3 * pt], means[3 * pt + 1], means[3 * pt + 2]};
    float x[3];
    const bool in = ntc_normalise(nd, mu, x);
    uint32_t ent[8];
    float wt[8];
    ntc_corners(nd, lv, x, ent, wt);
    for (int c = 0; c < 8; c++) {
        key[8 * t + c] = in ? (uint32_t)ent[c] : sentinel;
        pid[8 * t + c] = ((uint32_t)pt << 7) | ((uint32_t)lv << 3) | (uint32_t)c;
    }
}

__global__ __launch_bounds__(256) void k_csr_rows(const uint32_t* __restrict__ key, int64_t m, uint32_t sentinel,
                                                  uint2* __restrict__ rows) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= m) return;
    const uint32_t e = key[k];
    if (e == sentinel) return;
    if (k == 0 || key[k - 1] != e) rows[e].x = (uint32_t)k;
    if (k == m - 1 || key[k + 1] != e) rows[e].y = (uint32_t)(k + 1);
}

__global__ __launch_bounds__(256) void k_csr_weights(NtcDev nd, const float* __restrict__ means,
                                                     const uint32_t* __restrict__ key, const uint32_t* __restrict__ pid,
                                                     int64_t m, uint32_t sentinel, uint2* __restrict__ pw) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= m) return;
    const uint32_t c = pid[k];
    if (key[k] == sentinel) {
        pw[k] = make_uint2(c, 0u);
        return;
    }
    const int64_t pt = c >> 7;
    const int lv = (c >> 3) & 15, corner = c & 7;
    const float mu[3] = {means[3 * pt], means[3 * pt + 1], means[3 * pt + 2]};
    float x[3];
    ntc_normalise(nd, mu, x);
    uint32_t ent[8];
    float wt[8];
    ntc_corners(nd, lv, x, ent, wt);
    pw[k] = make_uint2(c, __float_as_uint(wt[corner]));
}

// 16 lanes per table entry: the entry's (point, weight) contributions are
// read 16 at a time (coalesced, one 8-byte load each), each lane gathers its
// point's encoding gradient, and the group sums with DPP (pairs, quads,
// half-row and row mirror): fixed order.
//
// Every level takes the same number of contributions (8 per point) and reads
// only its own slice of the encoding gradient (n x 8 bytes).  Workgroups are
// handed to the 8 XCDs in turn, so workgroup b runs on XCD b mod 8; the grid
// gives XCD x the entries of levels x and 15 - x (a coarse level with few,
// long rows and a fine one with many short rows), one level after the other.
// Each XCD then fetches two slices of the encoding gradient into its own L2
// instead of all sixteen.  The placement is a performance choice only: the
// result does not depend on where a workgroup runs.
constexpr int kGatherLanes = 16;
constexpr int kGatherEntries = 256 / kGatherLanes;   // entries per workgroup
constexpr int kXcds = 8;

struct GatherLevels {
    int64_t begin[16];   // first entry of each level
    int64_t end[16];     // one past its last entry
};


// The per-workgroup weight-gradient rows summed into dst: workgroup b of 256
// takes a range of columns of a slice of the rows, one atomic per (slice,
// column).  The kernels over the prepared lists end with these workgroups, for
// both only wait for the backward and a launch of its own costs 4-5 us.
constexpr int kPartSlice = 32;
struct PartSums {
    const float* part;
    int nparts;
    float* dst;
    int64_t first;   // the launch's first workgroup of them
    __host__ __device__ static constexpr int cols() { return (kMlpParams + 255) / 256; }
    int64_t blocks() const { return (int64_t)cols() * ((nparts + kPartSlice - 1) / kPartSlice); }
};

__device__ __forceinline__ void sum_parts(const PartSums& ps, int b) {
    const int k = b % PartSums::cols() * 256 + threadIdx.x;
    if (k >= kMlpParams) return;
    const int b0 = b / PartSums::cols() * kPartSlice;
    const int b1 = min(b0 + kPartSlice, ps.nparts);
    // eight loads in flight, summed in order
    float s = 0.f;
    int r = b0;
    for (; r + 8 <= b1; r += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = ps.part[(int64_t)(r + u) * kMlpParams + k];
#pragma unroll
        for (int u = 0; u < 8; u++) s += v[u];
    }
    for (; r < b1; r++) s += ps.part[(int64_t)r * kMlpParams + k];
    atomicAdd(ps.dst + k, s);
}

__global__ __launch_bounds__(256) void k_reduce_parts(PartSums ps) { sum_parts(ps, blockIdx.x); }

// The weighted encoding gradients of contributions k, k + G, ... below end,
// four independent loads in flight per lane.
template <int G>
__device__ __forceinline__ float2 gather_stride(const uint2* __restrict__ pw, const float* __restrict__ denc, int64_t n,
                                                uint32_t k, uint32_t end) {
    float a0 = 0.f, a1 = 0.f;
    auto enc = [&](uint32_t c) {
        return *reinterpret_cast<const float2*>(denc + 2 * ((int64_t)((c >> 3) & 15) * n + (c >> 7)));
    };
    for (; k + 3 * G < end; k += 4 * G) {
        const uint2 c0 = pw[k], c1 = pw[k + G], c2 = pw[k + 2 * G], c3 = pw[k + 3 * G];
        const float2 d0 = enc(c0.x), d1 = enc(c1.x), d2 = enc(c2.x), d3 = enc(c3.x);
        const float w0 = __uint_as_float(c0.y), w1 = __uint_as_float(c1.y);
        const float w2 = __uint_as_float(c2.y), w3 = __uint_as_float(c3.y);
        a0 += w0 * d0.x;
        a1 += w0 * d0.y;
        a0 += w1 * d1.x;
        a1 += w1 * d1.y;
        a0 += w2 * d2.x;
        a1 += w2 * d2.y;
        a0 += w3 * d3.x;
        a1 += w3 * d3.y;
    }
    for (; k < end; k += G) {
        const uint2 c = pw[k];
        const float2 d = enc(c.x);
        const float wk = __uint_as_float(c.y);
        a0 += wk * d.x;
        a1 += wk * d.y;
    }
    return make_float2(a0, a1);
}

// Row r summed by 16 lanes; lane 0 of them (sub 0) holds the sum.
__device__ __forceinline__ float2 gather_row16(const uint2* __restrict__ pw, const float* __restrict__ denc, int64_t n,
                                               uint2 r, int sub) {
    float2 a = gather_stride<16>(pw, denc, n, r.x + sub, r.y);
    a.x = dpp_add<0xB1, 0xF>(a.x);    // quad_perm [1,0,3,2]
    a.x = dpp_add<0x4E, 0xF>(a.x);    // quad_perm [2,3,0,1]
    a.x = dpp_add<0x141, 0xF>(a.x);   // row_half_mirror
    a.x = dpp_add<0x140, 0xF>(a.x);   // row_mirror: lane 0 of the row holds the sum
    a.y = dpp_add<0xB1, 0xF>(a.y);
    a.y = dpp_add<0x4E, 0xF>(a.y);
    a.y = dpp_add<0x141, 0xF>(a.y);
    a.y = dpp_add<0x140, 0xF>(a.y);
    return a;
}

static int64_t gather_blocks(const GatherLevels& gl, int lv) {
    return (gl.end[lv] - gl.begin[lv] + kGatherEntries - 1) / kGatherEntries;
}

__global__ __launch_bounds__(256) void k_csr_gather(GatherLevels gl, const uint2* __restrict__ rows,
                                                    const uint2* __restrict__ pw, const float* __restrict__ denc,
                                                    int64_t n, float* __restrict__ g_table, PartSums ps) {
    if ((int64_t)blockIdx.x >= ps.first) {
        sum_parts(ps, (int)(blockIdx.x - ps.first));
        return;
    }
    const int x = (int)(blockIdx.x % kXcds);
    int64_t j = blockIdx.x / kXcds;   // this workgroup's place among its XCD's
    int lv = x;
    const int64_t na = (gl.end[lv] - gl.begin[lv] + kGatherEntries - 1) / kGatherEntries;
    if (j >= na) {
        j -= na;
        lv = 15 - x;
    }
    const int64_t e = gl.begin[lv] + j * kGatherEntries + threadIdx.x / kGatherLanes;
    const bool valid = e < gl.end[lv];
    const int sub = threadIdx.x % kGatherLanes;
    uint2 r = make_uint2(0u, 0u);
    if (valid) r = rows[e];
    const float2 a = gather_row16(pw, denc, n, r, sub);
    if (sub == 0 && valid && r.y > r.x) {
        g_table[2 * e] += a.x;
        g_table[2 * e + 1] += a.y;
    }
}

// The same for few points, where most entries have a contribution or none: a
// lane sums an entry of up to kShortRow contributions alone, and the longer
// ones of a wave then take 16 lanes each.  Bound by the latency of loads that
// follow each other, in a quarter of the waves.  Not more entries to a wave,
// or its long ones queue up: backwards of 2000 and 4096 points in fp16, points
// all over the box, on surfaces and in a corner of it: 32 30 32 and 35 32 43
// us with 16 lanes an entry, 18 22 29 and 23 26 46 with 32 entries to a wave,
// 21 20 28 and 24 24 42 with 16.  8192 points 37 35 70 and 31 30 71, and from
// there on the corner loses (14000: 113 and 141), hence the line at two
// contributions an entry (6900 points at T = 2^15).
constexpr uint32_t kShortRow = 8;
constexpr int64_t kShortMean = 2;   // mean contributions of an entry up to which lanes take entries alone
constexpr int kShortEntries = 16;   // entries of a wave
__global__ __launch_bounds__(256) void k_csr_gather_short(int64_t entries, const uint2* __restrict__ rows,
                                                          const uint2* __restrict__ pw, const float* __restrict__ denc,
                                                          int64_t n, float* __restrict__ g_table, PartSums ps) {
    if ((int64_t)blockIdx.x >= ps.first) {
        sum_parts(ps, (int)(blockIdx.x - ps.first));
        return;
    }
    const int lane = threadIdx.x & 63;
    const int64_t e0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kShortEntries, e = e0 + lane;
    const uint2 r = lane < kShortEntries && e < entries ? rows[e] : make_uint2(0u, 0u);
    float2* const out = reinterpret_cast<float2*>(g_table);
    const bool lone = r.y - r.x <= kShortRow;
    if (lone && r.y > r.x) {
        const float2 a = gather_stride<1>(pw, denc, n, r.x, r.y), o = out[e];
        out[e] = make_float2(o.x + a.x, o.y + a.y);
    }
    const int sub = lane & 15, q = lane >> 4;
    for (uint64_t m = __ballot(!lone); m;) {   // the wave's next four long rows
        uint64_t t = m;
        for (int k = 0; k < q; k++) t &= t - 1;
        const int src = t ? __builtin_ctzll(t) : 0;
        uint2 l = make_uint2((uint32_t)__shfl((int)r.x, src), (uint32_t)__shfl((int)r.y, src));
        if (!t) l.y = l.x;
        const float2 a = gather_row16(pw, denc, n, l, sub);
        if (sub == 0 && t) {
            const float2 o = out[e0 + src];
            out[e0 + src] = make_float2(o.x + a.x, o.y + a.y);
        }
        for (int k = 0; k < 4; k++) m &= m - 1;
    }
}

// The same for many points, whose lists are kept slice by slice: a workgroup
// holds a slice of the points of one level in LDS and sums the level's entries
// over it into the slice's row of part.  The list is read in order, so the
// next part of it is in flight while one is summed: a lane takes kRun
// contributions that follow each other, stores the sums of the entries that
// lie inside them, and the entries that reach over lanes, rounds and waves are
// put together from the ends (a segmented scan over the lanes, a carry per
// wave, thread 0 over the waves).  A fixed order throughout.  k_csr_gather's 8
// bytes a contribution come from all over the level, a 128-byte line of the L2
// each; here they are read once, and the list's 8 bytes a contribution (65 us
// of 300K points' 97, at the rate of a large copy) are what is left.  300K
// points with k_chunk_sum, random and Morton order: 198 and 148 -> 110 and 118
// us.
constexpr int kRun = 8;
constexpr uint32_t kNoEntry = 0x1FFFFu;   // past the end of the list, with a point that is there
typedef uint32_t pw2 __attribute__((ext_vector_type(4), aligned(8)));   // two contributions

template <int kCtrl, int kRows>
__device__ __forceinline__ void seg_step(float& x, float& y, uint32_t& f) {
    const float px = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, kRows, 0xF, false));
    const float py = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), kCtrl, kRows, 0xF, false));
    const uint32_t pf = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, kCtrl, kRows, 0xF, false);
    x += f ? 0.f : px;
    y += f ? 0.f : py;
    f |= pf;
}

__global__ __launch_bounds__(1024) void k_csr_chunk(NtcDev nd, int64_t n, int slices, int64_t entries,
                                                    const uint32_t* __restrict__ starts, const uint2* __restrict__ pw,
                                                    const float* __restrict__ denc, float2* __restrict__ part) {
    constexpr int NW = 16;
    __shared__ float2 s_d[kChunkPoints];
    __shared__ uint32_t s_first[NW], s_last[NW];    // a wave's first and last entry
    __shared__ float2 s_fsum[NW], s_lsum[NW];       // and their sums
    const int slice = blockIdx.x % slices, lv = blockIdx.x / slices;
    const int64_t per = csr_slice(n, slices), p0 = slice * per;
    const int m = (int)max((int64_t)0, min(n, p0 + per) - p0);
    const int size = (int)nd.level_size(lv), tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t* const st = starts + slice * entries + nd.off[lv];
    float2* const out = part + slice * entries + nd.off[lv];
    // the waves take equal parts of the list, in whole rounds
    constexpr uint32_t kRound = 64 * kRun;
    const uint32_t total = st[size] - st[0], perw = (total + NW * kRound - 1) / (NW * kRound) * kRound;
    const uint32_t a = min(total, w * perw), b = min(total, a + perw);
    const uint2* const list = pw + st[0];
    uint32_t nx[kRun];
    float nw[kRun];
    auto load = [&](uint32_t r) {   // the lane's contributions of the round at r
        const uint32_t k = r + lane * kRun;
        if (k + kRun <= b) {
#pragma unroll
            for (int i = 0; i < kRun; i += 2) {
                const pw2 v = *reinterpret_cast<const pw2*>(list + k + i);
                nx[i] = v.x;
                nw[i] = __uint_as_float(v.y);
                nx[i + 1] = v.z;
                nw[i + 1] = __uint_as_float(v.w);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kRun; i++) {
                const bool in = k + i < b;
                const uint2 v = in ? list[k + i] : make_uint2(chunk_word(kNoEntry, 0u), 0u);
                nx[i] = v.x;
                nw[i] = __uint_as_float(v.y);
            }
        }
    };
    load(a);
    {
        const float2* src = reinterpret_cast<const float2*>(denc) + lv * n + p0;
        int k = tid;
        for (; k + 3 * 1024 < m; k += 4 * 1024) {
            float2 v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) v[u] = src[k + 1024 * u];
#pragma unroll
            for (int u = 0; u < 4; u++) s_d[k + 1024 * u] = v[u];
        }
        for (; k < m; k += 1024) s_d[k] = src[k];
    }
    for (int k = tid; k < size; k += 1024) out[k] = make_float2(0.f, 0.f);   // entries without a contribution
    __syncthreads();
    uint32_t first = kNoEntry, ckey = kNoEntry;
    float cx = 0.f, cy = 0.f;
    auto store = [&](uint32_t e, float x, float y) {   // an entry's whole sum in this wave
        if (e == first)
            s_fsum[w] = make_float2(x, y);   // it may have begun in the wave before
        else
            out[e] = make_float2(x, y);
    };
    for (uint32_t r = a; r < b; r += kRound) {
        uint32_t key[kRun];
        float px[kRun], py[kRun];
#pragma unroll
        for (int i = 0; i < kRun; i++) {
            key[i] = nx[i] >> 15;
            const float2 d = s_d[nx[i] & 0x7FFFu];
            px[i] = nw[i] * d.x;
            py[i] = nw[i] * d.y;
        }
        load(min(r + kRound, b));
        if (r == a) first = (uint32_t)__builtin_amdgcn_readfirstlane((int)key[0]);
        float x = px[0], y = py[0], hx = 0.f, hy = 0.f;
        bool pass = true;   // one entry so far
#pragma unroll
        for (int i = 1; i < kRun; i++) {
            const bool cut = key[i] != key[i - 1];
            if (cut && !pass) out[key[i - 1]] = make_float2(x, y);
            hx = cut && pass ? x : hx;
            hy = cut && pass ? y : hy;
            pass = pass && !cut;
            x = (cut ? 0.f : x) + px[i];
            y = (cut ? 0.f : y) + py[i];
        }
        const uint32_t tail = key[kRun - 1];
        uint32_t before = (uint32_t)__shfl_up((int)tail, 1);   // the last entry of the lane before
        before = lane == 0 ? ckey : before;
        const bool cont = key[0] == before;
        uint32_t f = pass && cont ? 0u : 1u;
        if (lane == 0 && !f) {
            x += cx;
            y += cy;
        }
        seg_step<0x111, 0xF>(x, y, f);   // row_shr 1, 2, 4, 8
        seg_step<0x112, 0xF>(x, y, f);
        seg_step<0x114, 0xF>(x, y, f);
        seg_step<0x118, 0xF>(x, y, f);
        seg_step<0x142, 0xA>(x, y, f);   // row_bcast 15 into rows 1 and 3
        seg_step<0x143, 0xC>(x, y, f);   // row_bcast 31 into rows 2 and 3
        float bx = __shfl_up(x, 1), by = __shfl_up(y, 1);
        bx = lane == 0 ? cx : bx;
        by = lane == 0 ? cy : by;
        if (!cont && before != kNoEntry) store(before, bx, by);
        if (!pass) store(key[0], hx + (cont ? bx : 0.f), hy + (cont ? by : 0.f));
        ckey = (uint32_t)__builtin_amdgcn_readlane((int)tail, 63);
        cx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
        cy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), 63));
    }
    if (lane == 0) {
        s_first[w] = first;
        s_last[w] = ckey;
        s_lsum[w] = make_float2(cx, cy);
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t key = kNoEntry;
        float2 sum = make_float2(0.f, 0.f);
        for (int k = 0; k < NW; k++) {
            if (s_first[k] == kNoEntry) break;   // no contributions here and after
            const bool one = s_first[k] == s_last[k];   // a single entry in the wave
            const float2 head = one ? s_lsum[k] : s_fsum[k];
            if (key == s_first[k]) {
                sum = make_float2(sum.x + head.x, sum.y + head.y);
            } else {
                if (key != kNoEntry) out[key] = sum;
                key = s_first[k];
                sum = head;
            }
            if (!one) {
                out[key] = sum;
                key = s_last[k];
                sum = s_lsum[k];
            }
        }
        if (key != kNoEntry) out[key] = sum;
    }
}

// The slices' sums added to the table gradient, slice by slice.
__global__ __launch_bounds__(256) void k_chunk_sum(const float2* __restrict__ part, int slices, int64_t entries,
                                                   float2* __restrict__ g_table, PartSums ps) {
    if ((int64_t)blockIdx.x >= ps.first) {
        sum_parts(ps, (int)(blockIdx.x - ps.first));
        return;
    }
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= entries) return;
    float2 a = make_float2(0.f, 0.f);
    int k = 0;
    for (; k + 8 <= slices; k += 8) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = part[(k + u) * entries + e];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            a.x += v[u].x;
            a.y += v[u].y;
        }
    }
    for (; k < slices; k++) {
        const float2 v = part[k * entries + e];
        a.x += v.x;
        a.y += v.y;
    }
    const float2 o = g_table[e];
    g_table[e] = make_float2(o.x + a.x, o.y + a.y);
}

// Table gradient of means that were not prepared: every (point, level) adds
// its eight corners' weighted encoding gradient to the level's entries.  A
// workgroup holds kLdsEntries entries of one level (a part) in LDS, adds the
// corners of its slice of the points that fall there with LDS atomics, and
// adds the sums to the table gradient, lane after lane on consecutive
// addresses.  Global atomics straight from the points each go to a line of
// their own, and the L2s take only some 20 of those per ns.  The sums are
// doubles: ds_add_f64 takes 3 to 6 lanes per clock of a CU on random entries
// where ds_add_f32 takes a third of one (measured).  Neighbouring lanes take
// points that lie apart, since points in spatial order fall on the same
// entries and their atomics would queue up.  20,011 points in bf16:
// 290 -> 45 us for backward and table gradient; 300K points in Morton order in
// fp16: 4.88 -> 0.40 ms.

__global__ __launch_bounds__(1024) void k_table_lds(NtcDev nd, TableParts tp, const float* __restrict__ means, int64_t n,
                                                    int slices, const float* __restrict__ denc,
                                                    float* __restrict__ g_table) {
    __shared__ double s_g[2 * kLdsEntries];
    const int part = blockIdx.x / slices, slice = blockIdx.x % slices;
    const int lv = tp.level[part], size = tp.size[part];
    const uint32_t first = (uint32_t)nd.off[lv] + (uint32_t)tp.first[part];
    for (int k = threadIdx.x; k < 2 * size; k += 1024) s_g[k] = 0.0;
    __syncthreads();
    const int64_t per = (n + slices - 1) / slices, p0 = slice * per, p1 = min(n, p0 + per);
    const int64_t rows = (per + 1023) / 1024;   // points of one thread, next to each other
    for (int64_t r = 0; r < rows; r++) {
        const int64_t pt = p0 + (int64_t)threadIdx.x * rows + r;
        if (pt >= p1) break;
        const float mu[3] = {means[3 * pt], means[3 * pt + 1], means[3 * pt + 2]};
        float xn[3];
        if (!ntc_normalise(nd, mu, xn)) continue;
        const float2 e = reinterpret_cast<const float2*>(denc)[(int64_t)lv * n + pt];
        uint32_t ent[8];
        float wt[8];
        ntc_corners(nd, lv, xn, ent, wt);
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const uint32_t k = ent[c] - first;
            if (k < (uint32_t)size) {
                atomicAdd(&s_g[2 * k], (double)(wt[c] * e.x));
                atomicAdd(&s_g[2 * k + 1], (double)(wt[c] * e.y));
            }
        }
    }
    __syncthreads();
    float* out = g_table + 2 * (int64_t)first;
    for (int k = threadIdx.x; k < 2 * size; k += 1024) {
        const float v = (float)s_g[k];
        if (v != 0.f) atomicAdd(out + k, v);
    }
}

template <class P>
__global__ __launch_bounds__(256) void k_ntc_adam(float* __restrict__ p, float* __restrict__ gr, float* __restrict__ m,
                                                  float* __restrict__ v, typename P::S* __restrict__ work, int64_t n,
                                                  float lr, float b1, float b2, float eps, float bc1, float bc2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float g = gr[i];
    const float mi = b1 * m[i] + (1.f - b1) * g;
    const float vi = b2 * v[i] + (1.f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    p[i] = pi;
    gr[i] = 0.f;
    if (work) work[i] = P::cvt(pi);
}

template <class P>
__global__ __launch_bounds__(256) void k_to_work(const float* __restrict__ p, typename P::S* __restrict__ work,
                                                 int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) work[i] = P::cvt(p[i]);
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ gr,
                                              float* __restrict__ m, float* __restrict__ v, int64_t n, float lr,
                                              float b1, float b2, float eps, float bc1, float bc2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float g = gr[i];
    const float mi = b1 * m[i] + (1.f - b1) * g;
    const float vi = b2 * v[i] + (1.f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// Eq. 7 per point, plus per-block partial sums of the loss
__global__ __launch_bounds__(256) void k_warmup(const float* __restrict__ dmu, const float* __restrict__ dq, int64_t n,
                                                float* __restrict__ gmu, float* __restrict__ gq,
                                                double* __restrict__ bsum) {
    __shared__ double s[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double L = 0.0;
    if (i < n) {
        const float invn = 1.0f / (float)n;
        float a = 0.f;
        for (int k = 0; k < 3; k++) {
            const float d = dmu[3 * i + k];
            a += fabsf(d);
            gmu[3 * i + k] = (d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f)) * invn;
        }
        const float w = dq[4 * i], x = dq[4 * i + 1], y = dq[4 * i + 2], z = dq[4 * i + 3];
        const float n2 = w * w + x * x + y * y + z * z;
        float c2 = 0.f;
        if (n2 > 0.f) {
            c2 = w * w / n2;
            const float i4 = 1.0f / (n2 * n2);
            gq[4 * i] = -(2.f * w * (n2 - w * w) * i4) * invn;
            gq[4 * i + 1] = (2.f * w * w * x * i4) * invn;
            gq[4 * i + 2] = (2.f * w * w * y * i4) * invn;
            gq[4 * i + 3] = (2.f * w * w * z * i4) * invn;
        } else {
            for (int k = 0; k < 4; k++) gq[4 * i + k] = 0.f;
        }
        L = (double)a - (double)c2;
    }
    for (int off = 32; off > 0; off >>= 1) L += __shfl_xor(L, off, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = L;
    __syncthreads();
    if (threadIdx.x == 0) bsum[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

__global__ __launch_bounds__(256) void k_warmup_finalize(const double* __restrict__ bsum, int64_t nb, int64_t n,
                                                         float* __restrict__ loss) {
    __shared__ double s[4];
    double a = 0.0;
    for (int64_t k = threadIdx.x; k < nb; k += 256) a += bsum[k];
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) loss[0] = (float)((s[0] + s[1] + s[2] + s[3]) / (double)n);
}

inline unsigned nblk(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// Whether the encoding of prepared means, which the forward keeps for the
// backward anyway, gets a launch of its own: the half types' levels, where
// they fit in its LDS, from so many points that the loads of the tables and
// the launch pay (fp16, random and Morton order: 8192 points 11 and 10 us in
// one launch, 11 in two; 20,011 16 and 13, 12 in two).  Without preparation
// there is no place for it but a workspace of the context, and such forwards
// write none: they may run beside each other and beside backwards, on other
// streams (300K points in Morton order 58 us so, 44 in two launches).
constexpr int64_t kEncPoints = 16384;
bool encode_apart(const NtcDev& nd, int64_t n) {
    bool fits = n >= kEncPoints;
    for (int lv = 0; lv < 16; lv++) fits = fits && nd.level_size(lv) <= kEncEntries;
    return fits;
}

template <class P>
void fwd_impl(const Launch& L, const NtcDev& nd, const void* table, const void* mlp, const float* means, int64_t n,
              float* dmu, float* dq, void* enc_out) {
    using S = typename P::S;
    const S* t = (const S*)table;
    const S* w = (const S*)mlp;
    // four workgroups per CU are resident (LDS-bound) on 256 CUs: one round of
    // workgroups, each looping over its share of the batches
    const dim3 grid((unsigned)std::min<int64_t>((n + kPts * kWaves - 1) / (kPts * kWaves), 1024));
    if constexpr (sizeof(S) == 2) {
        if (enc_out && encode_apart(nd, n)) {
            constexpr int kSlices = 16;   // times 16 levels: one workgroup per CU (the LDS holds one)
            hipLaunchKernelGGL((k_ntc_encode<P>), dim3(16 * kSlices), dim3(1024), 0, L.st, nd, t, means, n, kSlices,
                               (S*)enc_out);
            hipLaunchKernelGGL((k_ntc_fwd<P, true>), grid, dim3(256), 0, L.st, nd, t, w, means, n, dmu, dq, (S*)enc_out);
            return;
        }
    }
    hipLaunchKernelGGL((k_ntc_fwd<P, false>), grid, dim3(256), 0, L.st, nd, t, w, means, n, dmu, dq, (S*)enc_out);
}

// Table gradient from the encoding gradient, per entry over the prepared lists
// or scattered, and the sums of the weight-gradient rows.
void table_grad(const Launch& L, const NtcDev& nd, const float* means, int64_t n, const NtcCsr* csr, const float* denc,
                float* g_table, PartSums ps) {
    const auto with_parts = [&](int64_t blocks) {
        ps.first = blocks;
        return dim3((unsigned)(blocks + ps.blocks()));
    };
    if (!csr) {
        TableParts tp;
        if (table_parts(nd, kLdsEntries, tp)) {   // else the backward has scattered it
            // about one workgroup per CU (the LDS holds one) for few points,
            // a slice per 8192 points for many, so that the coarse levels'
            // workgroups, whose atomics queue up, do not trail the launch
            // (300K points: 4 slices 763 us, 8 565, 35 400; 20K: 4 slices 81
            // us for the whole pass, 8 85, 17 100)
            const int64_t few = std::min<int64_t>(256 / tp.count, (n + 1023) / 1024);
            const int slices = (int)std::max<int64_t>(std::max<int64_t>(few, n / 8192), 1);
            hipLaunchKernelGGL(k_table_lds, dim3((unsigned)(tp.count * slices)), dim3(1024), 0, L.st, nd, tp, means, n,
                               slices, denc, g_table);
        }
        ps.first = 0;
        hipLaunchKernelGGL(k_reduce_parts, dim3((unsigned)ps.blocks()), dim3(256), 0, L.st, ps);
        return;
    }
    if (csr->slices > 0) {
        hipLaunchKernelGGL(k_csr_chunk, dim3((unsigned)(16 * csr->slices)), dim3(1024), 0, L.st, nd, n, csr->slices,
                           csr->entries, csr->starts, csr->pw, denc, csr->part);
        const dim3 grid = with_parts(nblk(csr->entries, 256));
        hipLaunchKernelGGL(k_chunk_sum, grid, dim3(256), 0, L.st, csr->part, csr->slices, csr->entries,
                           reinterpret_cast<float2*>(g_table), ps);
        return;
    }
    if (128 * n <= kShortMean * csr->entries) {
        const dim3 grid = with_parts(nblk(csr->entries, 4 * kShortEntries));
        hipLaunchKernelGGL(k_csr_gather_short, grid, dim3(256), 0, L.st, csr->entries, csr->rows, csr->pw, denc, n, g_table,
                           ps);
        return;
    }
    GatherLevels gl;
    for (int lv = 0; lv < 16; lv++) {
        gl.begin[lv] = nd.off[lv];
        gl.end[lv] = lv < 15 ? nd.off[lv + 1] : csr->entries;
    }
    int64_t per_xcd = 0;
    for (int x = 0; x < kXcds; x++) per_xcd = std::max(per_xcd, gather_blocks(gl, x) + gather_blocks(gl, 15 - x));
    const dim3 grid = with_parts(per_xcd * kXcds);
    hipLaunchKernelGGL(k_csr_gather, grid, dim3(256), 0, L.st, gl, csr->rows, csr->pw, denc, n, g_table, ps);
}

template <class P>
void bwd_impl(const Launch& L, const NtcDev& nd, const void* table, const void* mlp, const float* means, int64_t n,
              const float* d_dmu, const float* d_dq, float* g_table, float* g_mlp, float* g_part, int max_parts,
              const NtcCsr* csr, float* denc, const void* enc_in) {
    const int64_t nb = (n + kPts - 1) / kPts;
    // max_parts is two per CU: the half-precision kernels fit two workgroups
    // on a CU, the float32 one (twice the LDS) one
    const int parts = sizeof(typename P::S) == 4 ? max_parts / 2 : max_parts;
    const unsigned grid = (unsigned)std::min<int64_t>((nb + kWaves - 1) / kWaves, parts);
    auto kern = denc ? k_ntc_bwd<P, false> : k_ntc_bwd<P, true>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, L.st, nd, (const typename P::S*)table, (const typename P::S*)mlp,
                       means, n, d_dmu, d_dq, g_part, denc, (const typename P::S*)enc_in, g_table);
    if (L.prof) L.prof->end(L.st);
    if (L.prof) L.prof->begin("ntc_scatter", L.st);
    table_grad(L, nd, means, n, csr, denc, g_table, PartSums{g_part, (int)grid, g_mlp, 0});
    if (L.prof) L.prof->end(L.st);
}

}  // namespace

int ntc_mlp_params() { return kMlpParams; }

void ntc_forward(const Launch& L, int precision, const NtcDev& nd, const void* table, const void* mlp,
                 const float* means, int64_t n, float* dmu, float* dq, void* enc_out) {
    if (n <= 0) return;
    if (L.prof) L.prof->begin("ntc_fwd", L.st);
    if (precision == 1)
        fwd_impl<PF16>(L, nd, table, mlp, means, n, dmu, dq, enc_out);
    else if (precision == 2)
        fwd_impl<PBF16>(L, nd, table, mlp, means, n, dmu, dq, enc_out);
    else
        fwd_impl<PF32>(L, nd, table, mlp, means, n, dmu, dq, enc_out);
    if (L.prof) L.prof->end(L.st);
}

void ntc_backward(const Launch& L, int precision, const NtcDev& nd, const void* table, const void* mlp,
                  const float* means, int64_t n, const float* d_dmu, const float* d_dq, float* g_table, float* g_mlp,
                  float* g_part, int max_parts, const NtcCsr* csr, float* scratch, const void* enc_in) {
    if (n <= 0) return;
    // without preparation the points go through the scratch a part at a time,
    // or their gradients straight to a large table
    TableParts tp;
    const bool scatter = !csr && !table_parts(nd, kLdsEntries, tp);
    const int64_t step = csr || scatter ? n : kScatterPoints;
    for (int64_t p0 = 0; p0 < n; p0 += step) {
        const int64_t m = std::min(step, n - p0);
        float* denc = csr ? csr->denc : scatter ? nullptr : scratch;
        if (L.prof) L.prof->begin("ntc_bwd", L.st);
        if (precision == 1)
            bwd_impl<PF16>(L, nd, table, mlp, means + 3 * p0, m, d_dmu + 3 * p0, d_dq + 4 * p0, g_table, g_mlp, g_part,
                           max_parts, csr, denc, enc_in);
        else if (precision == 2)
            bwd_impl<PBF16>(L, nd, table, mlp, means + 3 * p0, m, d_dmu + 3 * p0, d_dq + 4 * p0, g_table, g_mlp, g_part,
                            max_parts, csr, denc, enc_in);
        else
            bwd_impl<PF32>(L, nd, table, mlp, means + 3 * p0, m, d_dmu + 3 * p0, d_dq + 4 * p0, g_table, g_mlp, g_part,
                           max_parts, csr, denc, enc_in);
    }
}

bool ntc_csr_chunked(const NtcDev& nd, int64_t n) {
    bool fits = n >= kChunkMin;
    for (int lv = 0; lv < 16; lv++) fits = fits && nd.level_size(lv) <= kListEntries;
    return fits;
}

int64_t ntc_csr_slices(const NtcDev& nd, int64_t n) {
    // a workgroup per level and slice, whole rounds of one per CU
    if (ntc_csr_chunked(nd, n)) return 16 * ((n + 16 * kChunkPoints - 1) / (16 * kChunkPoints));
    TableParts tp;
    if (!table_parts(nd, kListEntries, tp)) return 0;
    // one workgroup per CU (the LDS holds one), a slice of at least 1024 points
    return std::max<int64_t>(1, std::min<int64_t>(256 / tp.count, (n + 1023) / 1024));
}

void ntc_csr_build(const Launch& L, const NtcDev& nd, const float* means, int64_t n, NtcCsr& csr, const CsrScratch& w) {
    if (L.prof) L.prof->begin("ntc_prepare", L.st);
    Launch inner{L.st, nullptr};
    TableParts tp;
    if (table_parts(nd, kListEntries, tp)) {
        const int slices = (int)ntc_csr_slices(nd, n);
        const unsigned grid = (unsigned)(tp.count * slices);
        hipLaunchKernelGGL(k_csr_count, dim3(grid), dim3(1024), 0, L.st, nd, tp, means, n, slices, csr.entries, w.cnt);
        csr.slices = 0;
        if (ntc_csr_chunked(nd, n)) {
            csr.slices = slices;
            csr.starts = w.cnt;
            scan_u32_to_u32(inner, w.cnt, slices * csr.entries + 1, w.cnt, w.tmp, w.tmp + 1);
        } else {
            hipLaunchKernelGGL(k_csr_totals, dim3(nblk(csr.entries, 256)), dim3(256), 0, L.st, w.cnt, slices,
                               csr.entries, w.first);
            scan_u32_to_u32(inner, w.first, csr.entries, w.first, w.tmp, w.tmp + 1);
            hipLaunchKernelGGL(k_csr_slots, dim3(nblk(csr.entries, 256)), dim3(256), 0, L.st, w.cnt, slices,
                               csr.entries, w.first, csr.rows);
        }
        hipLaunchKernelGGL(k_csr_place, dim3(grid), dim3(kPlaceThreads), 0, L.st, nd, tp, means, n, slices, csr.entries, w.cnt,
                           csr.slices > 0, csr.pw);
        if (L.prof) L.prof->end(L.st);
        return;
    }
    csr.slices = 0;
    const int64_t m = n * 128;
    const uint32_t sentinel = (uint32_t)csr.entries;
    int bits = 1;
    while (((int64_t)1 << bits) <= csr.entries) bits++;
    uint32_t* keys[2] = {w.keys[0], w.keys[1]};
    uint32_t* vals[2] = {w.vals[0], w.vals[1]};
    hipLaunchKernelGGL(k_csr_contrib, dim3(nblk(n * 16, 256)), dim3(256), 0, L.st, nd, means, n, sentinel, keys[0],
                       vals[0]);
    const int r = radix_sort_u32(inner, keys, vals, m, bits, w.hist, w.tmp);
    fill_u32(inner, reinterpret_cast<uint32_t*>(csr.rows), 0u, 2 * csr.entries);
    hipLaunchKernelGGL(k_csr_rows, dim3(nblk(m, 256)), dim3(256), 0, L.st, keys[r], m, sentinel, csr.rows);
    hipLaunchKernelGGL(k_csr_weights, dim3(nblk(m, 256)), dim3(256), 0, L.st, nd, means, keys[r], vals[r], m, sentinel,
                       csr.pw);
    if (L.prof) L.prof->end(L.st);
}

// SplitMix64 (Steele, Lea and Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014) used as a counter-based generator: output i of
// the stream seeded with `seed` is the generator's mixing function applied to
// seed + (i + 1) * 0x9E3779B97F4A7C15.
__device__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Parameter i = bound * (2u - 1) with u the top 24 bits of output i over
// 2^24 (exact in float32, so 2u - 1 is exact and the product rounds once).
// bound: b_table for the table, then b_w1 / b_w2 / b_w3 for the three
// weight matrices (n_w1, n_w2 entries; the rest W3).
__global__ __launch_bounds__(256) void k_ntc_init(float* __restrict__ p, int64_t n, int64_t n_table, int64_t n_w1,
                                                  int64_t n_w2, float b_table, float b_w1, float b_w2, float b_w3,
                                                  uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t j = i - n_table;
    const float b = j < 0 ? b_table : j < n_w1 ? b_w1 : j < n_w1 + n_w2 ? b_w2 : b_w3;
    const float u = (float)(uint32_t)(splitmix64_at(seed, (uint64_t)i) >> 40) * 0x1p-24f;
    p[i] = b * (2.0f * u - 1.0f);
}

void ntc_init(const Launch& L, float* p, int64_t n, int64_t n_table, uint64_t seed) {
    // U(-1e-4, 1e-4) for the table (instant-NGP's), Kaiming-uniform
    // U(-sqrt(6 / fan_in), +sqrt(6 / fan_in)) for W1 (fan-in 32), W2, W3 (64)
    const float b_table = 1e-4f, b_w1 = (float)sqrt(6.0 / 32.0), b_w2 = (float)sqrt(6.0 / 64.0);
    if (n <= 0) return;
    hipLaunchKernelGGL(k_ntc_init, dim3(nblk(n, 256)), dim3(256), 0, L.st, p, n, n_table, (int64_t)64 * 32,
                       (int64_t)64 * 64, b_table, b_w1, b_w2, b_w2, seed);
}

void ntc_adam(const Launch& L, int precision, float* p, float* g, float* m, float* v, void* work, int64_t n, float lr,
              float b1, float b2, float eps, float bc1, float bc2) {
    if (L.prof) L.prof->begin("ntc_adam", L.st);
    if (precision == 1)
        hipLaunchKernelGGL((k_ntc_adam<PF16>), dim3(nblk(n, 256)), dim3(256), 0, L.st, p, g, m, v, (_Float16*)work, n,
                           lr, b1, b2, eps, bc1, bc2);
    else if (precision == 2)
        hipLaunchKernelGGL((k_ntc_adam<PBF16>), dim3(nblk(n, 256)), dim3(256), 0, L.st, p, g, m, v, (__bf16*)work, n,
                           lr, b1, b2, eps, bc1, bc2);
    else
        hipLaunchKernelGGL((k_ntc_adam<PF32>), dim3(nblk(n, 256)), dim3(256), 0, L.st, p, g, m, v, (float*)nullptr, n,
                           lr, b1, b2, eps, bc1, bc2);
    if (L.prof) L.prof->end(L.st);
}

void ntc_refresh_work(const Launch& L, int precision, const float* p, void* work, int64_t n) {
    if (precision == 1)
        hipLaunchKernelGGL((k_to_work<PF16>), dim3(nblk(n, 256)), dim3(256), 0, L.st, p, (_Float16*)work, n);
    else if (precision == 2)
        hipLaunchKernelGGL((k_to_work<PBF16>), dim3(nblk(n, 256)), dim3(256), 0, L.st, p, (__bf16*)work, n);
}

void adam(const Launch& L, float* p, const float* g, float* m, float* v, int64_t n, int step, float lr, float b1,
          float b2, float eps) {
    if (n <= 0) return;
    const float bc1 = (float)(1.0 - pow((double)b1, (double)step));
    const float bc2 = (float)(1.0 - pow((double)b2, (double)step));
    if (L.prof) L.prof->begin("adam", L.st);
    hipLaunchKernelGGL(k_adam, dim3(nblk(n, 256)), dim3(256), 0, L.st, p, g, m, v, n, lr, b1, b2, eps, bc1, bc2);
    if (L.prof) L.prof->end(L.st);
}

void warmup_loss(const Launch& L, const float* dmu, const float* dq, int64_t n, float* loss, float* gmu, float* gq,
                 double* bsum) {
    if (n <= 0) return;
    if (L.prof) L.prof->begin("warmup_loss", L.st);
    const unsigned nb = nblk(n, 256);
    hipLaunchKernelGGL(k_warmup, dim3(nb), dim3(256), 0, L.st, dmu, dq, n, gmu, gq, bsum);
    hipLaunchKernelGGL(k_warmup_finalize, dim3(1), dim3(256), 0, L.st, bsum, (int64_t)nb, n, loss);
    if (L.prof) L.prof->end(L.st);
}

}  // namespace gs3
