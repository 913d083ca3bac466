// NTC launchers (internal to libgs3.so).
#pragma once
#include "kernels.h"

namespace gs3 {

// Shape of the hash encoding, passed by value to kernels.
struct NtcDev {
    int res[16];           // grid resolution per level
    int64_t off[16];       // first table entry of each level
    uint32_t dense_mask;   // bit l set: level l is stored densely
    uint32_t T_mask;       // 2^log2_T - 1
    float aabb_min[3];
    float inv_ext[3];
    __host__ __device__ int64_t level_size(int lv) const {
        const int64_t r = (int64_t)res[lv] + 1;
        return (dense_mask >> lv) & 1u ? r * r * r : (int64_t)T_mask + 1;
    }
};

// Per-frame contribution lists of the table gradient (see ntc.hip).
struct NtcCsr {
    int64_t entries = 0;      // table entries
    uint2* rows = nullptr;    // [entries]: [start, end) into pw
    uint2* pw = nullptr;      // (point << 7 | level << 3 | corner, float bits of the trilinear weight), by entry
    float* denc = nullptr;    // [16 levels][n][2] encoding gradient of the current backward
    // lists kept slice by slice (many points), instead of rows: starts[slice][entry] of them
    // in pw and the lists' end, and the slices' sums of the current backward
    int slices = 0;
    uint32_t* starts = nullptr;
    float2* part = nullptr;
};

int ntc_mlp_params();
// points whose encoding gradient a backward without preparation holds at a
// time (32 MB of scratch)
constexpr int64_t kScatterPoints = 1 << 18;
// Scratch of the list building: cnt (slices x entries + 1) and first (entries)
// when ntc_csr_slices gives a number of slices, else (0) the sort's ping-pong
// buffers of n * 128 u32 each and hist, radix_hist_words(n * 128); tmp holds
// the scan's words of either + 1.
struct CsrScratch {
    uint32_t* cnt = nullptr;
    uint32_t* first = nullptr;
    uint32_t* keys[2] = {nullptr, nullptr};
    uint32_t* vals[2] = {nullptr, nullptr};
    uint32_t* hist = nullptr;
    uint64_t* tmp = nullptr;
};
int64_t ntc_csr_slices(const NtcDev& nd, int64_t n);
bool ntc_csr_chunked(const NtcDev& nd, int64_t n);   // lists slice by slice
void ntc_csr_build(const Launch& L, const NtcDev& nd, const float* means, int64_t n, NtcCsr& csr, const CsrScratch& w);
// enc_out (optional, n x 32 values of the working precision): the forward
// also stores the points' encoding there, in the order that the backward reads
void ntc_forward(const Launch& L, int precision, const NtcDev& nd, const void* table, const void* mlp,
                 const float* means, int64_t n, float* dmu, float* dq, void* enc_out);
// g_part holds max_parts x ntc_mlp_params() floats; without csr, scratch holds
// min(n, kScatterPoints) x 32 floats; enc_in (optional, with csr): the
// encoding a forward with the same parameters and means stored, used instead
// of recomputing it
void ntc_backward(const Launch& L, int precision, const NtcDev& nd, const void* table, const void* mlp,
                  const float* means, int64_t n, const float* d_dmu, const float* d_dq, float* g_table, float* g_mlp,
                  float* g_part, int max_parts, const NtcCsr* csr, float* scratch, const void* enc_in);
void ntc_adam(const Launch& L, int precision, float* p, float* g, float* m, float* v, void* work, int64_t n, float lr,
              float b1, float b2, float eps, float bc1, float bc2);
// float32 master parameters [table | W1 | W2 | W3] from a counter-based
// generator (SplitMix64) seeded with `seed`
void ntc_init(const Launch& L, float* p, int64_t n, int64_t n_table, uint64_t seed);
void ntc_refresh_work(const Launch& L, int precision, const float* p, void* work, int64_t n);
void warmup_loss(const Launch& L, const float* dmu, const float* dq, int64_t n, float* loss, float* gmu, float* gq,
                 double* bsum);

}  // namespace gs3
