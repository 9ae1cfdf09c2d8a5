// a7 - a9 for protein models on the matrix cores: the precision form with a
// 20-letter one-hot.
//
// E-step scores of a tile of 16 windows for 16 models: S = OneHot . W with
// contraction index kappa = 20 p + sigma (position p, letter sigma), 20 l of
// them padded to NK blocks of 64.  M-step counts: C = OneHot^T . Z, rows kappa
// (4 NK tiles of 16), contraction over 32 windows.  One FP16 value per non-0/1
// operand (the log-odds W and the posteriors Z), FP32 accumulation.  The
// per-sequence log-sum-exp is FP64: each lane keeps an FP64 sum of its terms
// 2^(S - ref) against a whole-number reference (so that moving it rescales the
// sum exactly), the lanes and waves of a model are combined in FP64 and the
// logarithm is FP64; LLR and J are FP64.
//
// A workgroup of four waves takes 64 models (four groups of 16) of one
// instance.  What bounds the one-hot side is forming and moving its operands,
// 25 times sparser than a DNA one-hot is, so each is formed once per
// workgroup and used for all 64 models:
//  - E-step: the waves take different blocks of 32 windows, each for all 64
//    models (their log-odds stay in registers).  A position's 20 columns are
//    five groups of four with at most one 1, inside the 2-of-4 pattern of
//    v_smfmac_f32_16x16x64_f16.  Stored as one dword per group ((1, 0) or
//    (0, 1) of the pair of letters that holds the symbol, or zero), five per
//    symbol, the expanded sequence holds every window's operand as it is: lane
//    (window r, group g) of block kk reads the dwords 5 w + 16 kk + 4 g ..
//    + 3 and the index field of those four groups.
//  - M-step: the waves take different row tiles, each for all windows and
//    models; the posteriors pass through LDS in the layout the E-step leaves
//    and the M-step reads.  Row (p, sigma) of the one-hot is the bitmap of
//    letter sigma's places in the sequence, shifted by p: a lane reads the
//    bitmap, and a table of 256 turns its eight windows' bits into halves.
// Every sequence is swept twice, for its log-sum-exp (in the final E-step also
// the best start) and, with exactly normalised posteriors, for the counts,
// which stay in registers across the sequences.
//
// 16 384 models of the (20,6) workload (t = 30, n = 1000), 5 iterations:
// 32.1 ms with dense operands of both steps rebuilt in LDS for every window
// pair and read by every wave for its own 16 models.
//
// Lane layout (lane L, r = L % 16, g = L / 16):
//   E-step A: window row r, kappa 64 kk + 16 g .. + 15; B: model r, kappa
//   64 kk + 8 g .. + 7 and 64 kk + 32 + 8 g .. + 7; D: model r, windows
//   4g .. 4g+3 of the tile;
//   M-step A: kappa row 16 rt + r, windows w_j (j < 8) = 4g + j (tile 0) and
//   16 + 4g + j - 4 (tile 1), exactly the windows of the lane's E-step outputs.
#include <math.h>

#include "pm_common.h"

namespace pm {

typedef _Float16 half8p __attribute__((ext_vector_type(8)));
typedef _Float16 half16p __attribute__((ext_vector_type(16)));
typedef float float4p __attribute__((ext_vector_type(4)));

constexpr int kPW = 4;           // waves per workgroup
constexpr int kPG = 4;           // groups of 16 models per workgroup
constexpr int kPSymMax = 2048;   // longest sequence (symbols)
constexpr int kPTMax = 64;       // most sequences
constexpr int kPSymPad = 96;     // symbols past the end that a window's padded operand reaches
constexpr float kPLog2e = 1.4426950408889634f;
constexpr float kPRefSlack = 60.0f;  // a lane's reference moves when a score passes it by more

struct EmProtArgs {
    const uint32_t *packed;
    const int64_t *offsets;
    const double *theta0;
    const double *bg;
    const int64_t *n_dev;
    double *theta_out;
    double *J;
    double *llr;
    int32_t *sites;
    int64_t B;
    int t, l, iters;
    int nsym;    // symbols the LDS holds of a sequence (longest one and padding)
    double beta;
};

// dynamic LDS, one region: the expanded sequence and the posteriors during the
// sweeps; the log-odds before them; the counts after them
__host__ __device__ inline int prot_bit_words(int nsym) { return nsym / 32 + 8; }
__host__ __device__ inline int prot_seq_bytes(int nsym)
{
    return (nsym * 30 + 21 * 4 * prot_bit_words(nsym) + 15) / 16 * 16;
}
template <int NK>
__host__ __device__ inline int prot_lds_bytes(int nsym)
{
    const int sweep = prot_seq_bytes(nsym) + 2 * kPW * kPG * 64 * 16, wts = kPG * NK * 2 * 64 * 16,
              cnt = 64 * NK * 64 * 4;
    const int a = sweep > wts ? sweep : wts;
    return a > cnt ? a : cnt;
}

// eight FP16 halves, 1.0 at the set bits of an 8-bit mask
__device__ __forceinline__ uint4 mask8_halves(uint32_t mk)
{
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        w[q] = (((mk >> (2 * q)) & 1u) ? 0x3C00u : 0u) | (((mk >> (2 * q + 1)) & 1u) ? 0x3C000000u : 0u);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// 64 NK contraction rows; the log-odds of 64 models take 32 NK registers and
// the wave's counts 16 NK: one wave per SIMD
template <int NK>
__global__ void __launch_bounds__(64 * kPW, 1) k_em_prot(const EmProtArgs a)
{
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ __align__(16) uint4 lut[256];
    __shared__ double psum[kPW][64];    // a wave's sum of 2^(S - pref) per model
    __shared__ float pref[kPW][64];
    __shared__ float pbest[kPW][64];    // final E-step: a wave's best score and window
    __shared__ int pwin[kPW][64];
    __shared__ double prior_s[64];
    __shared__ double lbg[20];          // ln of the background frequencies

    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    int64_t nvalid = a.n_dev ? *a.n_dev : a.B;
    if (nvalid > a.B) nvalid = a.B;
    const int64_t b0 = (int64_t)blockIdx.x * 16 * kPG;
    if (b0 >= nvalid) return;  // uniform over the workgroup
    const int l = a.l, t = a.t, AL = 20 * l, nk = 20 * l, nsym = a.nsym, nbw = prot_bit_words(nsym);
    const double beta = a.beta;
    uint32_t *X = reinterpret_cast<uint32_t *>(dyn);           // [nsym][5]
    uint16_t *XI = reinterpret_cast<uint16_t *>(X + 5 * nsym); // [nsym][5] index fields of groups j .. j + 3
    uint32_t *bits = reinterpret_cast<uint32_t *>(dyn + (nsym * 30 + 3) / 4 * 4);  // [21][nbw], row 20 empty
    uint4 *post = reinterpret_cast<uint4 *>(dyn + prot_seq_bytes(nsym));   // [2][block][group][lane]
    lut[tid] = mask8_halves(tid);
    if (tid < 20) lbg[tid] = log(a.bg[tid]);
    __syncthreads();

    // the wave's row tiles wv NK .. wv NK + NK - 1: this lane's row of each, as
    // the byte offset of its letter's bitmap (times 32) and its shift
    uint32_t row[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const int kap = 16 * (NK * wv + i) + r;
        row[i] = (uint32_t)((kap < nk ? kap % 20 : 20) * nbw * 4) << 5 | (uint32_t)(kap < nk ? kap / 20 : 0);
    }

    // sequence i expanded in LDS (all users of the previous one are done)
    auto expand = [&](int64_t s0, int n) {
        for (int u0 = 64 * wv; u0 < nsym; u0 += 64 * kPW) {
            const int u = u0 + lane;
            const int e = u < n ? (int)prot_sym(a.packed, s0 + u) : 32;
            const int e1 = u + 1 < n ? (int)prot_sym(a.packed, s0 + u + 1) : 32;
            if (u < nsym) {
                const uint32_t v = 0x3C00u << ((e & 1) * 16);
#pragma unroll
                for (int q = 0; q < 5; ++q) X[5 * u + q] = (e >> 2) == q ? v : 0u;
                const uint32_t f = (e & 2) ? 0xEu : 0x4u, f1 = (e1 & 2) ? 0xEu : 0x4u;
                XI[5 * u] = (uint16_t)(f * 0x1111u);
                XI[5 * u + 1] = (uint16_t)(f * 0x1111u);
                XI[5 * u + 2] = (uint16_t)(f * 0x111u + f1 * 0x1000u);
                XI[5 * u + 3] = (uint16_t)(f * 0x11u + f1 * 0x1100u);
                XI[5 * u + 4] = (uint16_t)(f + f1 * 0x1110u);
            }
            uint32_t lo = 0, hi = 0;  // lane q < 20: letter q's places among these 64
#pragma unroll
            for (int q = 0; q < 20; ++q) {
                const uint64_t m = __ballot(e == q);
                if (lane == q) {
                    lo = (uint32_t)m;
                    hi = (uint32_t)(m >> 32);
                }
            }
            if (lane < 21) {
                bits[lane * nbw + u0 / 32] = lo;
                bits[lane * nbw + u0 / 32 + 1] = hi;
            }
        }
        // past the last 64 symbols: no letter
        const int w1 = (nsym + 63) / 64 * 2;
        for (int q = tid; q < 21 * (nbw - w1); q += 64 * kPW) bits[q / (nbw - w1) * nbw + w1 + q % (nbw - w1)] = 0u;
    };

    half16p Wb[kPG][NK];
    // scores of the windows w0 .. w0 + 31 for the 64 models, from `init`
    auto estep = [&](int w0, const float (&init)[kPG], float4p (&S)[2][kPG]) {
#pragma unroll
        for (int q = 0; q < kPG; ++q)
            S[0][q] = S[1][q] = float4p{init[q], init[q], init[q], init[q]};
        const int j0 = 5 * (w0 + r) + 4 * g;
        const uint32_t *x = X + j0;
        const uint16_t *xi = XI + j0;
        // the operands of block kk + 1 load while block kk multiplies; nothing
        // else is moved ahead (all blocks' operands at once would not fit)
        uint4 v[2];
        int ix[2];
        auto load = [&](int kk) {
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2) {
                const int j = 16 * kk + 80 * t2;
                v[t2] = make_uint4(x[j], x[j + 1], x[j + 2], x[j + 3]);
                ix[t2] = xi[j];
            }
        };
        load(0);
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            const half8p A0 = __builtin_bit_cast(half8p, v[0]), A1 = __builtin_bit_cast(half8p, v[1]);
            const int i0 = ix[0], i1 = ix[1];
            if (kk + 1 < NK) load(kk + 1);
#pragma unroll
            for (int q = 0; q < kPG; ++q) {
                S[0][q] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(A0, Wb[q][kk], S[0][q], i0, 0, 0);
                S[1][q] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(A1, Wb[q][kk], S[1][q], i1, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    for (int it = 0; it <= a.iters; ++it) {
        const bool last = it == a.iters;
        const double *src = it == 0 ? a.theta0 : a.theta_out;
        // ---- log-odds (log2 units) of the wave's own 16 models and their
        // prior, through LDS to all four waves; one half block at a time (an
        // unrolled build would keep all its loads in flight in registers)
        {
            uint4 *wts = reinterpret_cast<uint4 *>(dyn);  // [group][2 NK][lane]
            const int64_t b = b0 + 16 * wv + r;
            const bool vb = b < nvalid;
            double prior = 0;
#pragma unroll 1
            for (int kh = 0; kh < 2 * NK; ++kh) {
                half8p hv;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int kap = 32 * kh + 8 * g + j;
                    float w = 0.f;
                    if (kap < nk && vb) {
                        const int p = kap / 20, sg = kap - 20 * p;
                        const double th = src[b * AL + sg * l + p];
                        if (it == 0) a.theta_out[b * AL + sg * l + p] = th;
                        const double lt = log(th);
                        w = (float)((lt - lbg[sg]) * (double)kPLog2e);
                        prior += a.bg[sg] * lt;
                    }
                    hv[j] = (_Float16)w;
                }
                wts[(wv * 2 * NK + kh) * 64 + lane] = __builtin_bit_cast(uint4, hv);
            }
            prior += __shfl_xor(prior, 16);
            prior += __shfl_xor(prior, 32);
            if (g == 0) prior_s[16 * wv + r] = prior;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kPG; ++q)
#pragma unroll
                for (int kk = 0; kk < NK; ++kk) {
                    const half8p h0 = __builtin_bit_cast(half8p, wts[(q * 2 * NK + 2 * kk) * 64 + lane]);
                    const half8p h1 = __builtin_bit_cast(half8p, wts[(q * 2 * NK + 2 * kk + 1) * 64 + lane]);
                    Wb[q][kk] = __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                }
        }

        float4p C[NK][kPG];
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
            for (int q = 0; q < kPG; ++q) C[i][q] = float4p{0.f, 0.f, 0.f, 0.f};
        double llr = 0;  // of model `lane`, the same in every wave

        for (int i = 0; i < t; ++i) {
            const int64_t s0 = a.offsets[i];
            const int n = (int)(a.offsets[i + 1] - s0), L = n - l + 1, nb = (L + 31) / 32;
            __syncthreads();  // the previous users of the LDS region are done
            expand(s0, n);
            __syncthreads();

            // ---- log-sum-exp of the sequence (the best start too in the final
            // E-step): the wave's blocks wv, wv + 4, ...
            float ref[kPG], bestv[kPG];
            double sm[kPG];
            int besti[kPG];
#pragma unroll
            for (int q = 0; q < kPG; ++q) {
                ref[q] = 0.f;
                sm[q] = 0.0;
                bestv[q] = -INFINITY;
                besti[q] = 0;
            }
            for (int blk = wv; blk < nb; blk += kPW) {
                const int w0 = 32 * blk;
                float4p S[2][kPG];
                const float init[kPG] = {-ref[0], -ref[1], -ref[2], -ref[3]};
                estep(w0, init, S);
                if (w0 + 32 > L) {
#pragma unroll
                    for (int q = 0; q < kPG; ++q)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if (w0 + 4 * g + j >= L) S[0][q][j] = -INFINITY;
                            if (w0 + 16 + 4 * g + j >= L) S[1][q][j] = -INFINITY;
                        }
                }
                float top[kPG];
                bool move = blk == wv;  // the first block sets the reference
#pragma unroll
                for (int q = 0; q < kPG; ++q) {
                    top[q] = fmaxf(fmaxf(fmaxf(S[0][q][0], S[0][q][1]), fmaxf(S[0][q][2], S[0][q][3])),
                                   fmaxf(fmaxf(S[1][q][0], S[1][q][1]), fmaxf(S[1][q][2], S[1][q][3])));
                    move |= top[q] > kPRefSlack;
                }
                if (last) {
#pragma unroll
                    for (int q = 0; q < kPG; ++q)
                        if (__ballot(top[q] + ref[q] > bestv[q])) {
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                const float v = (u < 4 ? S[0][q][u & 3] : S[1][q][u & 3]) + ref[q];
                                if (v > bestv[q]) {
                                    bestv[q] = v;
                                    besti[q] = w0 + 16 * (u >> 2) + 4 * g + (u & 3);
                                }
                            }
                        }
                }
                if (__ballot(move)) {
                    // whole numbers: the rescaled sums are exact
#pragma unroll
                    for (int q = 0; q < kPG; ++q) {
                        const bool mv = top[q] > -INFINITY && (blk == wv || top[q] > kPRefSlack);
                        const float d = mv ? ceilf(top[q]) : 0.f;
                        sm[q] = ldexp(sm[q], -(int)d);
                        ref[q] += d;
                        S[0][q] -= d;
                        S[1][q] -= d;
                    }
                }
#pragma unroll
                for (int q = 0; q < kPG; ++q) {
                    float e[8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        e[j] = __builtin_amdgcn_exp2f(S[0][q][j]);
                        e[4 + j] = __builtin_amdgcn_exp2f(S[1][q][j]);
                    }
                    sm[q] += (double)(((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])));
                }
            }
            // the four lanes of each model (a lane without a window has the
            // reference 0 and the sum 0, which changes nothing), then the waves
#pragma unroll
            for (int q = 0; q < kPG; ++q) {
                float M = sm[q] > 0 ? ref[q] : -INFINITY;
                M = fmaxf(M, __shfl_xor(M, 16));
                M = fmaxf(M, __shfl_xor(M, 32));
                double part = sm[q] > 0 ? ldexp(sm[q], (int)(ref[q] - M)) : sm[q];
                part += __shfl_xor(part, 16);
                part += __shfl_xor(part, 32);
                if (last && a.sites) {
#pragma unroll
                    for (int o = 16; o <= 32; o <<= 1) {
                        const float ov = __shfl_xor(bestv[q], o);
                        const int oi = __shfl_xor(besti[q], o);
                        if (ov > bestv[q] || (ov == bestv[q] && oi < besti[q])) {
                            bestv[q] = ov;
                            besti[q] = oi;
                        }
                    }
                }
                if (g == 0) {
                    psum[wv][16 * q + r] = part;
                    pref[wv][16 * q + r] = M;
                    pbest[wv][16 * q + r] = bestv[q];
                    pwin[wv][16 * q + r] = besti[q];
                }
            }
            __syncthreads();
            // model `lane`, in every wave
            float M = fmaxf(fmaxf(pref[0][lane], pref[1][lane]), fmaxf(pref[2][lane], pref[3][lane]));
            double tot = 0;
#pragma unroll
            for (int w = 0; w < kPW; ++w) {
                const double p = psum[w][lane];
                tot += p > 0 ? ldexp(p, (int)(pref[w][lane] - M)) : p;
            }
            const double lz = (double)M + log2(tot);  // log2 of the sum of 2^S
            llr += lz * 0.6931471805599453 - log((double)L);
            if (last) {
                if (a.sites && wv == 0 && b0 + lane < nvalid) {
                    float bv = pbest[0][lane];
                    int bi = pwin[0][lane];
#pragma unroll
                    for (int w = 1; w < kPW; ++w)
                        if (pbest[w][lane] > bv || (pbest[w][lane] == bv && pwin[w][lane] < bi)) {
                            bv = pbest[w][lane];
                            bi = pwin[w][lane];
                        }
                    a.sites[(b0 + lane) * t + i] = bi;
                }
                continue;
            }

            // ---- exactly normalised posteriors and their counts, four blocks a
            // step; the buffers alternate, so one barrier per step is enough
            float nlz[kPG];
#pragma unroll
            for (int q = 0; q < kPG; ++q) nlz[q] = -__shfl((float)lz, 16 * q + r);
            for (int s = 0; kPW * s < nb; ++s) {
                uint4 *buf = post + (s & 1) * kPW * kPG * 64;
                const int blk = kPW * s + wv, w0 = 32 * blk;
                if (blk < nb) {
                    float4p S[2][kPG];
                    estep(w0, nlz, S);
#pragma unroll
                    for (int q = 0; q < kPG; ++q) {
                        half8p h;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            float e0 = __builtin_amdgcn_exp2f(S[0][q][j]), e1 = __builtin_amdgcn_exp2f(S[1][q][j]);
                            if (w0 + 32 > L) {
                                if (w0 + 4 * g + j >= L) e0 = 0.f;
                                if (w0 + 16 + 4 * g + j >= L) e1 = 0.f;
                            }
                            h[j] = (_Float16)e0;
                            h[4 + j] = (_Float16)e1;
                        }
                        buf[(wv * kPG + q) * 64 + lane] = __builtin_bit_cast(uint4, h);
                    }
                }
                __syncthreads();
                const int have = nb - kPW * s < kPW ? nb - kPW * s : kPW;  // blocks of this step
#pragma unroll 1
                for (int k = 0; k < have; ++k) {
                    half8p Z[kPG];
#pragma unroll
                    for (int q = 0; q < kPG; ++q) Z[q] = __builtin_bit_cast(half8p, buf[(k * kPG + q) * 64 + lane]);
                    const uint8_t *bk = reinterpret_cast<const uint8_t *>(bits + kPW * s + k);
#pragma unroll
                    for (int i2 = 0; i2 < NK; ++i2) {
                        const uint32_t *bw = reinterpret_cast<const uint32_t *>(bk + (row[i2] >> 5));
                        const uint32_t m = (__builtin_amdgcn_alignbit(bw[1], bw[0], row[i2]) >> (4 * g)) & 0x000F000Fu;
                        const half8p Am = __builtin_bit_cast(half8p, lut[(m | (m >> 12)) & 0xFFu]);
#pragma unroll
                        for (int q = 0; q < kPG; ++q)
                            C[i2][q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Am, Z[q], C[i2][q], 0, 0, 0);
                    }
                }
            }
        }
        if (wv == 0 && b0 + lane < nvalid) {
            a.J[(b0 + lane) * (a.iters + 1) + it] = llr + beta * prior_s[lane];
            if (a.llr) a.llr[(b0 + lane) * (a.iters + 1) + it] = llr;
        }
        if (last) break;

        // ---- counts to LDS, every column of a model divided by its own total:
        // the lane is the model, the waves take columns
        __syncthreads();
        float *cnt = reinterpret_cast<float *>(dyn);  // [64 NK rows][64 models]
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
            for (int q = 0; q < kPG; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) cnt[(16 * (NK * wv + i) + 4 * g + j) * 64 + 16 * q + r] = C[i][q][j];
        __syncthreads();
        const int64_t b = b0 + lane;
        if (b < nvalid)
            for (int p = wv; p < l; p += kPW) {
                double s = 0;
                for (int c = 0; c < 20; ++c) s += (double)cnt[(20 * p + c) * 64 + lane];
                const double tot = s + beta;
                for (int c = 0; c < 20; ++c)
                    a.theta_out[b * AL + c * l + p] = ((double)cnt[(20 * p + c) * 64 + lane] + beta * a.bg[c]) / tot;
            }
        __syncthreads();  // theta^(it+1) visible to every lane before it is read
    }
}

template <int NK>
static int launch_prot(const EmProtArgs &a, hipStream_t st)
{
    const int64_t groups = (a.B + 16 * kPG - 1) / (16 * kPG);
    const int lds = prot_lds_bytes<NK>(a.nsym);
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute((const void *)k_em_prot<NK>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    hipLaunchKernelGGL(k_em_prot<NK>, dim3((unsigned)groups), dim3(64 * kPW), lds, st, a);
    PM_LAUNCHED();
    return PM_OK;
}

int em_refine_prot(const pm_seqs *S, int32_t l, const double *theta0, const double *bg, int64_t B,
                   const int64_t *n_dev, int32_t iters, double beta, double *theta_out, double *J_out,
                   double *llr_out, int32_t *sites_out, hipStream_t st)
{
    if (l > 24) return fail(PM_ERANGE, "the protein matrix-core form takes l <= 24");
    if (S->t > kPTMax) return fail(PM_ERANGE, "the protein matrix-core form takes t <= %d", kPTMax);
    if (S->n_max > kPSymMax) return fail(PM_ERANGE, "the protein matrix-core form takes n_i <= %d", kPSymMax);
    EmProtArgs a{};
    a.packed = S->packed;
    a.offsets = S->offsets;
    a.theta0 = theta0;
    a.bg = bg;
    a.n_dev = n_dev;
    a.theta_out = theta_out;
    a.J = J_out;
    a.llr = llr_out;
    a.sites = sites_out;
    a.B = B;
    a.t = S->t;
    a.l = l;
    a.iters = iters;
    a.beta = beta;
    a.nsym = (S->n_max + kPSymPad + 1) / 2 * 2;
    switch ((20 * l + 63) / 64) {
    case 1: return launch_prot<1>(a, st);
    case 2: return launch_prot<2>(a, st);
    case 3: return launch_prot<3>(a, st);
    case 4: return launch_prot<4>(a, st);
    case 5: return launch_prot<5>(a, st);
    case 6: return launch_prot<6>(a, st);
    case 7: return launch_prot<7>(a, st);
    default: return launch_prot<8>(a, st);
    }
}

}  // namespace pm
