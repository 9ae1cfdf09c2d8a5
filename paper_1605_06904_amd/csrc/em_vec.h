// Shared pieces of the vector EM kernels of libprojmotif (gfx950): the launch
// arguments and the helpers of a workgroup of four waves that takes one model.
#pragma once

#include <math.h>

#include "pm_common.h"

namespace pm {

struct EmArgs {
    pm_inst one;                // the instance, when inst is NULL
    const pm_inst *inst;        // batch: instance table, or NULL
    const int32_t *item_inst;   // batch: instance of every trial item
    const pm_bucket *buckets;   // batch: the models' buckets (their items)
    const double *theta0;
    const double *bg;
    const int64_t *n_dev;
    double *theta_out;
    double *J;
    double *llr;
    int32_t *sites;
    int64_t B;
    int l, iters;
    int site_stride;  // sites row length (t, or the largest t of a batch)
    double beta;
    int model;        // PM_OOPS, PM_ZOOPS or PM_TCM
    double mix0;      // ZOOPS gamma or TCM lambda of theta0
    double *mix_out;  // [B] mixing parameter of the final E-step, or NULL
    int seq_cap;      // LDS words reserved for the packed input (0: read from global)
    int off_cap;      // LDS offsets reserved (0: read from global)
    int tile_pct;     // tiled form: see tile_takes (0: never)
    int fp32;         // tiled form: sites by FP32 scores
};

// Whether the tiled form (em_tile.h) takes a call of n models: its time goes by
// rounds of sixteen models per CU, full or not, and a full round takes pct
// hundredths of the time that the workgroup-per-model form takes for as many
// models.  One form takes all models of a call, so that equal models have
// equal results.
constexpr int64_t kTileRound = 16 * 256;
__host__ __device__ inline bool tile_takes(int64_t n, int pct)
{
    return pct > 0 && (n + kTileRound - 1) / kTileRound * kTileRound * pct <= 100 * n;
}

constexpr int kEmThreads = 256;
constexpr int kEmWaves = kEmThreads / 64;

template <typename T>
__device__ __forceinline__ T ninf();
template <>
__device__ __forceinline__ float ninf<float>() { return -INFINITY; }
template <>
__device__ __forceinline__ double ninf<double>() { return -INFINITY; }

__device__ __forceinline__ float ex(float v) { return expf(v); }
__device__ __forceinline__ double ex(double v) { return exp(v); }
__device__ __forceinline__ float lg1p(float v) { return log1pf(v); }
__device__ __forceinline__ double lg1p(double v) { return log1p(v); }

// ln(e^u + e^v), e^{-inf} = 0
template <typename T>
__device__ __forceinline__ T log_add(T u, T v)
{
    if (u == ninf<T>()) return v;
    if (v == ninf<T>()) return u;
    const T d = u - v;
    return (d > 0 ? u : v) + lg1p(ex(d > 0 ? -d : d));
}

template <int WAVES = kEmWaves, typename V>
__device__ __forceinline__ V block_sum(V v, V *red)
{
    v = wave_sum(v);
    if (lane_id() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    V r = red[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) r += red[w];
    __syncthreads();
    return r;
}

__device__ __forceinline__ int64_t wave_min_i64(int64_t v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        int64_t u = __shfl_xor(v, o);
        v = u < v ? u : v;
    }
    return v;
}

// the DNA form (em_dna.h) of four and eight waves (four: l <= 24); a.seq_cap and
// a.off_cap are set, lds their bytes
int launch_em_dna_f64_w4(const EmArgs &a, size_t lds, hipStream_t st);
int launch_em_dna_f64_w8(const EmArgs &a, size_t lds, hipStream_t st);
int launch_em_dna_f32_w4(const EmArgs &a, size_t lds, hipStream_t st);
int launch_em_dna_f32_w8(const EmArgs &a, size_t lds, hipStream_t st);
// the tiled form (em_tile.h)
int launch_em_tile(const EmArgs &a, hipStream_t st);      // OOPS and ZOOPS
int launch_em_tile_tcm(const EmArgs &a, hipStream_t st);

}  // namespace pm
