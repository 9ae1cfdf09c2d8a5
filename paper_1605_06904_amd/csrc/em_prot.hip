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
// A workgroup of eight waves takes 64 models (four groups of 16) of one
// instance: four waves (one per SIMD) do the E-step and hand the posteriors to
// four that keep the counts.  Apart, the log-odds of a wave (16 NK registers)
// or its counts (16 NK) leave room for the operands under way at two waves per
// SIMD; together they spilled at every sequence, and with eight E-step waves
// (three per SIMD) the operands under way did.  What bounds the one-hot side is forming and moving its operands,
// 25 times sparser than a DNA one-hot is, so each is formed once per
// workgroup and used for all 64 models:
//  - E-step: a pair of waves takes a block of 32 windows, each for 32 of the
//    models.  A position's 20 columns are
//    five groups of four with at most one 1, inside the 2-of-4 pattern of
//    v_smfmac_f32_16x16x64_f16.  Stored as one dword per group ((1, 0) or
//    (0, 1) of the pair of letters that holds the symbol, or zero), five per
//    symbol, the expanded sequence holds every window's operand as it is: lane
//    (window r, group g) of block kk reads the dwords 5 w + 16 kk + 4 g ..
//    + 3 and the index field of those four groups.
//  - M-step: the four waves take different row tiles, each for all windows and
//    models, one step of four blocks behind the E-step; the posteriors pass through LDS in the layout the E-step leaves
//    and the M-step reads.  Row (p, sigma) of the one-hot is the bitmap of
//    letter sigma's places in the sequence, shifted by p: a lane reads the
//    bitmap, and a table of 256 turns its eight windows' bits into halves.
// Every sequence is swept twice, for its log-sum-exp (in the final E-step also
// the best start) and, with exactly normalised posteriors, for the counts,
// which stay in registers across the sequences.
//
// 16 384 models of the (20,6) workload (t = 30, n = 1000), 5 iterations:
// 32.1 ms with dense operands of both steps rebuilt in LDS for every window
// pair and read by every wave for its own 16 models; 8.1 ms with every wave
// doing both steps (a wave per SIMD with all registers, or two), 6.3 ms so: an
// E-step wave is the longest in every step (about 2 100 cycles per block, of
// which 450 are its matrix instructions).
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

constexpr int kPWE = 4;          // waves of the E-step
constexpr int kPWM = 4;          // waves of the M-step
constexpr int kPW = kPWE + kPWM;
constexpr int kPG = 4;           // groups of 16 models per workgroup
constexpr int kPB = 4;           // blocks of 32 windows per step
constexpr int kPP = kPWE / 2;    // pairs of E-step waves, a block of windows at a time each
constexpr int kPE = 2;           // groups of an E-step wave
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
    const int sweep = prot_seq_bytes(nsym) + 2 * kPB * kPG * 64 * 16, wts = kPG * NK * 2 * 64 * 16,
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

struct ProtShared {
    uint4 lut[256];
    double psum[kPP][64];  // a wave pair's sums of 2^(S - pref) per model
    float pref[kPP][64];
    float pbest[kPP][64];  // final E-step: its best score and window
    int pwin[kPP][64];
    double prior[64];
    double lbg[20];  // ln of the background frequencies
    int64_t offs[kPTMax + 1];
    uint32_t pk[2 * 256];  // packed words of the sequence to expand
};

// The whole refinement, as an E-step (ESTEP) or an M-step wave; both pass the
// same barriers.
template <int NK, bool ESTEP>
__device__ __forceinline__ void prot_wave(const EmProtArgs &a, uint8_t *dyn, ProtShared &sh, int wv, int64_t nvalid,
                                          int64_t b0)
{
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int eb = wv >> 1, eh = wv & 1;  // E-step: the wave's pair and its half of the models
    const int l = a.l, t = a.t, AL = 20 * l, nk = 20 * l, nsym = a.nsym, nbw = prot_bit_words(nsym);
    const double beta = a.beta;
    uint32_t *X = reinterpret_cast<uint32_t *>(dyn);           // [nsym][5]
    uint16_t *XI = reinterpret_cast<uint16_t *>(X + 5 * nsym); // [nsym][5] index fields of groups j .. j + 3
    uint32_t *bits = reinterpret_cast<uint32_t *>(dyn + (nsym * 30 + 3) / 4 * 4);  // [21][nbw], row 20 empty
    uint4 *post = reinterpret_cast<uint4 *>(dyn + prot_seq_bytes(nsym));   // [2][block][group][lane]

    // the packed words of a sequence: loaded into a register one sequence ahead
    // (at most 2048 symbols: 343 words, one per thread)
    uint32_t pw = 0;
    auto words_ahead = [&](int i) {
        const int64_t w0 = sh.offs[i] / 6, w1 = (sh.offs[i + 1] - 1) / 6;
        if (tid < 512) pw = a.packed[min(w0 + tid, w1)];
    };
    words_ahead(0);

    // sequence i expanded in LDS (all users of the previous one are done)
    auto expand = [&](int i, int n) {
        const int first = (int)(sh.offs[i] % 6);  // the first symbol's place in its word
        if (tid < 512) sh.pk[tid] = pw;
        __syncthreads();
        words_ahead(i + 1 < t ? i + 1 : 0);
        for (int u0 = 64 * wv; u0 < nsym; u0 += 64 * kPW) {
            const int u = u0 + lane;
            const int e = u < n ? (int)prot_sym(sh.pk, first + u) : 32;
            const int e1 = u + 1 < n ? (int)prot_sym(sh.pk, first + u + 1) : 32;
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

    // ---- M-step waves: the row tiles (wv - kPWE) NK .. + NK - 1; this lane's
    // row of each, as the byte offset of its letter's bitmap (times 32) and its
    // shift, and the counts of all 64 models
    constexpr int NM = ESTEP ? 1 : NK;
    uint32_t row[NM];
    float4p C[NM][kPG];
    if (!ESTEP) {
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int kap = 16 * (NK * (wv - kPWE) + i) + r;
            row[i] = (uint32_t)((kap < nk ? kap % 20 : 20) * nbw * 4) << 5 | (uint32_t)(kap < nk ? kap / 20 : 0);
        }
    }
    // counts of the `have` blocks of step s.  Operands come by two dependent LDS
    // reads, the bitmap and the table of halves: the bitmaps of the whole step
    // are read first (the lane's eight windows of block k as byte k of ent), and
    // the table is read kLutAhead row tiles ahead of the matrix instructions.
    auto consume = [&](int s, int have) {
        const uint4 *buf = post + (s & 1) * kPB * kPG * 64;
        const uint8_t *b0k = reinterpret_cast<const uint8_t *>(bits + kPB * s);
        uint32_t ent[NM];
        constexpr int kBatch = 4;
#pragma unroll
        for (int i0 = 0; i0 < NM; i0 += kBatch) {
            uint32_t v[kBatch][kPB + 1];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (i0 + u < NM) {
                    const uint32_t *bw = reinterpret_cast<const uint32_t *>(b0k + (row[i0 + u < NM ? i0 + u : 0] >> 5));
#pragma unroll
                    for (int k = 0; k <= kPB; ++k) v[u][k] = bw[k];
                }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (i0 + u < NM) {
                    const int i = i0 + u < NM ? i0 + u : 0;
                    uint32_t e = 0;
#pragma unroll
                    for (int k = 0; k < kPB; ++k) {
                        const uint32_t m = (__builtin_amdgcn_alignbit(v[u][k + 1], v[u][k], row[i]) >> (4 * g)) & 0x000F000Fu;
                        e |= ((m | (m >> 12)) & 0xFFu) << (8 * k);
                    }
                    ent[i] = e;
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        constexpr int kLutAhead = NM < 3 ? NM : 3;
#pragma unroll 1
        for (int k = 0; k < have; ++k) {
            half8p Z[kPG], Am[kLutAhead + 1];
            auto lut_of = [&](int i) { return __builtin_bit_cast(half8p, sh.lut[(ent[i] >> (8 * k)) & 0xFFu]); };
#pragma unroll
            for (int i = 0; i < kLutAhead; ++i) Am[i] = lut_of(i);
#pragma unroll
            for (int q = 0; q < kPG; ++q) Z[q] = __builtin_bit_cast(half8p, buf[(k * kPG + q) * 64 + lane]);
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                if (i + kLutAhead < NM) Am[(i + kLutAhead) % (kLutAhead + 1)] = lut_of(i + kLutAhead < NM ? i + kLutAhead : 0);
#pragma unroll
                for (int q = 0; q < kPG; ++q)
                    C[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Am[i % (kLutAhead + 1)], Z[q], C[i][q], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // ---- E-step waves: log-odds of 32 models
    half16p Wb[kPE][ESTEP ? NK : 1];
    // scores of the windows w0 .. w0 + 31 for the wave's models, from `init`
    auto estep = [&](int w0, const float (&init)[kPE], float4p (&S)[2][kPE]) {
        if (ESTEP) {
#pragma unroll
            for (int q = 0; q < kPE; ++q) S[0][q] = S[1][q] = float4p{init[q], init[q], init[q], init[q]};
            const int j0 = 5 * (w0 + r) + 4 * g;
            const uint32_t *x = X + j0;
            const uint16_t *xi = XI + j0;
            // the operands of the next three blocks of columns load while one
            // multiplies; nothing else is moved ahead (all at once would not fit)
            constexpr int D = 4;
            uint4 v[D][2];
            int ix[D][2];
            auto load = [&](int kk) {
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {
                    const int j = 16 * kk + 80 * t2;
                    v[kk % D][t2] = make_uint4(x[j], x[j + 1], x[j + 2], x[j + 3]);
                    ix[kk % D][t2] = xi[j];
                }
            };
#pragma unroll
            for (int kk = 0; kk < D - 1 && kk < NK; ++kk) load(kk);
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                if (kk + D - 1 < NK) load(kk + D - 1);
#pragma unroll
                for (int q = 0; q < kPE; ++q)
#pragma unroll
                    for (int t2 = 0; t2 < 2; ++t2)
                        S[t2][q] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(
                            __builtin_bit_cast(half8p, v[kk % D][t2]), Wb[q][ESTEP ? kk : 0], S[t2][q], ix[kk % D][t2],
                            0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    for (int it = 0; it <= a.iters; ++it) {
        const bool last = it == a.iters;
        const double *src = it == 0 ? a.theta0 : a.theta_out;
        // ---- log-odds (log2 units) and prior of group wv's models, through LDS to
        // the waves that take them; one half block at a time (an unrolled build would keep all its loads in
        // flight in registers)
        uint4 *wts = reinterpret_cast<uint4 *>(dyn);  // [group][2 NK][lane]
        if (ESTEP) {
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
                        w = (float)((lt - sh.lbg[sg]) * (double)kPLog2e);
                        prior += a.bg[sg] * lt;
                    }
                    hv[j] = (_Float16)w;
                }
                wts[(wv * 2 * NK + kh) * 64 + lane] = __builtin_bit_cast(uint4, hv);
            }
            prior += __shfl_xor(prior, 16);
            prior += __shfl_xor(prior, 32);
            if (g == 0) sh.prior[16 * wv + r] = prior;
        } else {
#pragma unroll
            for (int i = 0; i < NM; ++i)
#pragma unroll
                for (int q = 0; q < kPG; ++q) C[i][q] = float4p{0.f, 0.f, 0.f, 0.f};
        }
        __syncthreads();
        if (ESTEP) {
#pragma unroll
            for (int q = 0; q < kPE; ++q)
#pragma unroll
                for (int kk = 0; kk < NK; ++kk) {
                    const uint4 *w = wts + ((kPE * eh + q) * 2 * NK + 2 * kk) * 64 + lane;
                    const half8p h0 = __builtin_bit_cast(half8p, w[0]), h1 = __builtin_bit_cast(half8p, w[64]);
                    Wb[q][ESTEP ? kk : 0] =
                        __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                }
        }
        double llr = 0;  // of model `lane`, the same in every wave

        for (int i = 0; i < t; ++i) {
            const int n = __builtin_amdgcn_readfirstlane((int)(sh.offs[i + 1] - sh.offs[i]));
            const int L = n - l + 1, nb = (L + 31) / 32, steps = (nb + kPB - 1) / kPB;
            __syncthreads();  // the previous users of the LDS region are done
            expand(i, n);
            __syncthreads();
            if (ESTEP) {
                // ---- log-sum-exp of the sequence (the best start too in the final
                // E-step): the pair's blocks eb, eb + 2, ...
                float ref[kPE], bestv[kPE];
                double sm[kPE];
                int besti[kPE];
#pragma unroll
                for (int q = 0; q < kPE; ++q) {
                    ref[q] = 0.f;
                    sm[q] = 0.0;
                    bestv[q] = -INFINITY;
                    besti[q] = 0;
                }
                for (int blk = eb; blk < nb; blk += kPP) {
                    const int w0 = 32 * blk;
                    float4p S[2][kPE];
                    const float init[kPE] = {-ref[0], -ref[1]};
                    estep(w0, init, S);
                    if (w0 + 32 > L) {
#pragma unroll
                        for (int q = 0; q < kPE; ++q)
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                if (w0 + 4 * g + j >= L) S[0][q][j] = -INFINITY;
                                if (w0 + 16 + 4 * g + j >= L) S[1][q][j] = -INFINITY;
                            }
                    }
                    float top[kPE];
                    bool move = blk == eb;  // the first block sets the reference
#pragma unroll
                    for (int q = 0; q < kPE; ++q) {
                        top[q] = fmaxf(fmaxf(fmaxf(S[0][q][0], S[0][q][1]), fmaxf(S[0][q][2], S[0][q][3])),
                                       fmaxf(fmaxf(S[1][q][0], S[1][q][1]), fmaxf(S[1][q][2], S[1][q][3])));
                        move |= top[q] > kPRefSlack;
                    }
                    if (last) {
#pragma unroll
                        for (int q = 0; q < kPE; ++q)
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
                        for (int q = 0; q < kPE; ++q) {
                            const bool mv = top[q] > -INFINITY && (blk == eb || top[q] > kPRefSlack);
                            const float d = mv ? ceilf(top[q]) : 0.f;
                            sm[q] = ldexp(sm[q], -(int)d);
                            ref[q] += d;
                            S[0][q] -= d;
                            S[1][q] -= d;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < kPE; ++q) {
                        double e[8];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            e[j] = (double)__builtin_amdgcn_exp2f(S[0][q][j]);
                            e[4 + j] = (double)__builtin_amdgcn_exp2f(S[1][q][j]);
                        }
                        sm[q] += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
                    }
                }
                // the four lanes of each model (a lane without a window has the
                // reference 0 and the sum 0, which changes nothing), then the waves
#pragma unroll
                for (int q = 0; q < kPE; ++q) {
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
                        sh.psum[eb][16 * (kPE * eh + q) + r] = part;
                        sh.pref[eb][16 * (kPE * eh + q) + r] = M;
                        sh.pbest[eb][16 * (kPE * eh + q) + r] = bestv[q];
                        sh.pwin[eb][16 * (kPE * eh + q) + r] = besti[q];
                    }
                }
            }
            __syncthreads();
            // model `lane`, in every wave
            const float M = fmaxf(sh.pref[0][lane], sh.pref[1][lane]);
            static_assert(kPP == 2, "two pairs");
            double tot = 0;
#pragma unroll
            for (int w = 0; w < kPP; ++w) {
                const double p = sh.psum[w][lane];
                tot += p > 0 ? ldexp(p, (int)(sh.pref[w][lane] - M)) : p;
            }
            const double lz = (double)M + log2(tot);  // log2 of the sum of 2^S
            // a sum that is not a number (a zero in theta, whose log-odds the one-hot
            // multiplies by 0): log-likelihood -inf
            llr += (lz == lz ? lz : -INFINITY) * 0.6931471805599453 - log((double)L);
            if (last) {
                if (a.sites && wv == 0 && b0 + lane < nvalid) {
                    float bv = sh.pbest[0][lane];
                    int bi = sh.pwin[0][lane];
#pragma unroll
                    for (int w = 1; w < kPP; ++w)
                        if (sh.pbest[w][lane] > bv || (sh.pbest[w][lane] == bv && sh.pwin[w][lane] < bi)) {
                            bv = sh.pbest[w][lane];
                            bi = sh.pwin[w][lane];
                        }
                    a.sites[(b0 + lane) * t + i] = bi;
                }
                continue;
            }

            // ---- exactly normalised posteriors and their counts, four blocks a
            // step, the M-step waves one step behind; the buffers alternate, so one
            // barrier per step is enough
            float nlz[kPE];
#pragma unroll
            for (int q = 0; q < kPE; ++q) nlz[q] = -__shfl((float)lz, 16 * (kPE * eh + q) + r);
            for (int s = 0; s <= steps; ++s) {
                if (ESTEP) {
                    uint4 *buf = post + (s & 1) * kPB * kPG * 64;
#pragma unroll 1
                    for (int k = eb; k < kPB && kPB * s + k < nb; k += kPP) {
                        const int w0 = 32 * (kPB * s + k);
                        float4p S[2][kPE];
                        estep(w0, nlz, S);
#pragma unroll
                        for (int q = 0; q < kPE; ++q) {
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
                            buf[(k * kPG + kPE * eh + q) * 64 + lane] = __builtin_bit_cast(uint4, h);
                        }
                    }
                } else if (s > 0) {
                    consume(s - 1, min(nb - kPB * (s - 1), kPB));
                }
                __syncthreads();
            }
        }
        if (wv == 0 && b0 + lane < nvalid) {
            a.J[(b0 + lane) * (a.iters + 1) + it] = llr + beta * sh.prior[lane];
            if (a.llr) a.llr[(b0 + lane) * (a.iters + 1) + it] = llr;
        }
        if (last) break;

        // ---- counts to LDS, every column of a model divided by its own total:
        // the lane is the model, the waves take columns
        float *cnt = reinterpret_cast<float *>(dyn);  // [64 NK rows][64 models]
        if (!ESTEP) {
#pragma unroll
            for (int i = 0; i < NM; ++i)
#pragma unroll
                for (int q = 0; q < kPG; ++q)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        cnt[(16 * (NK * (wv - kPWE) + i) + 4 * g + j) * 64 + 16 * q + r] = C[i][q][j];
        }
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
__global__ void __launch_bounds__(64 * kPW, 2) k_em_prot(const EmProtArgs a)
{
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ __align__(16) ProtShared sh;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t nvalid = a.n_dev ? *a.n_dev : a.B;
    if (nvalid > a.B) nvalid = a.B;
    const int64_t b0 = (int64_t)blockIdx.x * 16 * kPG;
    if (b0 >= nvalid) return;  // uniform over the workgroup
    if (tid < 256) sh.lut[tid] = mask8_halves(tid);
    if (tid < 20) sh.lbg[tid] = log(a.bg[tid]);
    for (int i = tid; i <= a.t; i += 64 * kPW) sh.offs[i] = a.offsets[i];
    __syncthreads();
    if (wv < kPWE) prot_wave<NK, true>(a, dyn, sh, wv, nvalid, b0);
    else prot_wave<NK, false>(a, dyn, sh, wv, nvalid, b0);
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
