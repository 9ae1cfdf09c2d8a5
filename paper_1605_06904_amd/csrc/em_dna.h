// a7 - a9 for DNA models on the vector units: OOPS, ZOOPS and TCM EM in FP64
// or FP32 (see em.hip for the protein form and projmotif.h for the models).
// Included by one source per precision and number of waves.
//
// One workgroup of four or eight waves per model; a wave takes whole sequences
// and a lane takes windows.  Sequences are summed by eight slots whatever the
// waves, so that a model's result does not depend on their number.  What bounds this is LDS traffic per window: scoring is
// a table read per position and the M-step a table update per position.
// Both go by three letters at a time here: the E-step reads ceil(l/3) tables
// of 64 three-letter sums (formed once per iteration from the l columns), and
// the M-step adds each posterior to one entry of ceil(l/3) tables of 64, from
// which the letter counts are summed at the end of the iteration.  Against a
// read and an update per position this is a third of the LDS operations, and
// an update's 64 lanes fall on 64 entries instead of on four, whose updates
// the LDS takes one after another.  The updates are FP64 in both precisions:
// the LDS's FP32 additions took several times as long (4 096 ZOOPS models of
// the (18,6) workload, 10 iterations: 27.7 ms with FP32 updates, 7.5 with
// FP64 ones).  Measured against a read and an update per position: those
// models 84.5 -> 7.5 ms, a (15,4) pass in FP64 (20 000 models, 5 iterations)
// 45.3 -> 11.3 ms; the LDS is then busy 88% of the time, three quarters of it
// with the updates.
//
// A sequence of up to 64 kNC windows is scored once: its scores stay in
// registers, the log-sum-exp is formed against its largest score, and the
// same exponentials, times one factor per sequence, are the posteriors.
// Longer sequences are scored twice.
#pragma once

#include <algorithm>

#include "dna3.h"
#include "em_vec.h"

namespace pm {

constexpr int kNC = 16;    // windows a lane holds in registers
constexpr int kSlots = 8;  // sequences i, i + 8, .. are summed together

// the score of a window: ceil(l/3) table reads
template <typename T, int NG, int Q = 0>
__device__ __forceinline__ T score3(const Win &w, const T *W3)
{
    const T v = W3[64 * Q + three_letters<Q>(w)];
    if constexpr (Q + 1 < NG) return v + score3<T, NG, Q + 1>(w, W3);
    else return v;
}

template <int NG, int Q = 0>
__device__ __forceinline__ void scatter3(const Win &w, double z, double *C3)
{
    atomicAdd(&C3[64 * Q + three_letters<Q>(w)], z);
    if constexpr (Q + 1 < NG) scatter3<NG, Q + 1>(w, z, C3);
}

// the score as a sum over positions in order: decides between best starts
// whose three-letter sums are within rounding of each other
template <typename T>
__device__ __forceinline__ T score_in_order(const Win &w, const T *wt, int l)
{
    T s = 0;
    for (int p = 0; p < l; ++p) s += wt[dna_at(w.hi, w.lo, p) * l + p];
    return s;
}

template <typename T>
__device__ __forceinline__ T eps();
template <>
__device__ __forceinline__ float eps<float>() { return 1.1920929e-7f; }
template <>
__device__ __forceinline__ double eps<double>() { return 2.220446049250313e-16; }

template <typename T, int NG, int MODEL, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, NG == 8 && WAVES == 4 ? 2 : 4) k_em_dna(const EmArgs a)
{
    constexpr int kThreads = 64 * WAVES;
    const int64_t b = blockIdx.x;
    int64_t nvalid = a.n_dev ? *a.n_dev : a.B;
    if (nvalid > a.B) nvalid = a.B;
    if (b >= nvalid || tile_takes(nvalid, a.tile_pct)) return;

    __shared__ double th[4 * 32];
    __shared__ T wt[4 * 32];                 // log-odds of every letter and position
    __shared__ T W3[64 * NG];                // their sums over three positions
    __shared__ double C3[kSlots][64 * NG];   // posteriors by three letters, per slot
    __shared__ double csum[64 * NG];         // the same over the slots
    __shared__ double red[WAVES], llr_slot[kSlots];
    __shared__ double colsum[32];
    __shared__ double ztot;
    extern __shared__ __align__(16) uint32_t dyn[];
    uint32_t *seq = dyn;
    int64_t *offs = reinterpret_cast<int64_t *>(dyn + ((a.seq_cap + 1) & ~1));

    const pm_inst I = a.inst ? a.inst[a.item_inst[a.buckets[b].trial]] : a.one;
    const int tid = threadIdx.x, wv = tid >> 6, lane = lane_id();
    const int l = a.l, t = I.t, AL = 4 * l;
    const double beta = a.beta;
    const int seq_words = a.seq_cap ? (int)((I.n_total + 15) / 16 + 4) : 0;

    for (int i = tid; i < AL; i += kThreads) th[i] = a.theta0[b * AL + i];
    for (int i = tid; i < seq_words; i += kThreads) seq[i] = I.packed[i];
    if (a.off_cap)
        for (int i = tid; i <= t; i += kThreads) offs[i] = I.offsets[i];
    __syncthreads();
    const uint32_t *W = a.seq_cap ? seq : I.packed;
    const int64_t *O = a.off_cap ? offs : I.offsets;

    // mixing parameter of ZOOPS (gamma) or TCM (lambda); OOPS has none
    double mix = a.mix0;
    for (int it = 0; it <= a.iters; ++it) {
        const bool last = it == a.iters;
        const double lmix = MODEL == PM_OOPS ? 0.0 : log(mix), lnone = MODEL == PM_OOPS ? 0.0 : log1p(-mix);
        double pr = 0;
        for (int i = tid; i < AL; i += kThreads) {
            const int c = i / l;
            const double v = th[i];
            wt[i] = (T)(log(v) - log(a.bg[c]));
            if (beta != 0) pr += a.bg[c] * log(v);
        }
        for (int i = tid; i < kSlots * 64 * NG; i += kThreads) (&C3[0][0])[i] = 0;
        pr = block_sum<WAVES>(pr, red);  // includes the barrier that publishes wt
        for (int e = tid; e < 64 * NG; e += kThreads) {
            const int p = e / 64 * 3;
            T v = wt[((e >> 4) & 3) * l + p];
            if (p + 1 < l) v += wt[((e >> 2) & 3) * l + p + 1];
            if (p + 2 < l) v += wt[(e & 3) * l + p + 2];
            W3[e] = v;
        }
        __syncthreads();
        // how far a three-letter sum and the sum in order can be apart
        T tol = 0;
        if (last) {
            T m = 0;
            if (lane < l)
                for (int c = 0; c < 4; ++c) m = fmax(m, fabs(wt[c * l + lane]));
            tol = wave_sum(m) * (T)(2 * 32) * eps<T>();
        }

        for (int slot = wv; slot < kSlots; slot += WAVES) {
            double *ac = C3[slot];
            double llr_w = 0;
            for (int i = slot; i < t; i += kSlots) {
                const int64_t s0 = O[i];
                const int L = (int)(O[i + 1] - s0) - l + 1;
                if (MODEL == PM_TCM) {
                    // every window its own two-component mixture: one sweep gives
                    // its log-likelihood term, its posterior and its counts
                    const T lm = (T)lmix, ln0 = (T)lnone;
                    double lsum = 0;
                    T bv = ninf<T>();
                    int64_t ba = 0;
                    for (int x = lane; x < L; x += 64) {
                        const Win w = load_win(W, s0 + x);
                        const T s = score3<T, NG>(w, W3);
                        // the larger component, and what the other is of it (a NaN
                        // score, or an infinite one, makes its posterior NaN)
                        const T v = lm + s;
                        const bool site = !(v <= ln0);
                        const T e = v == ninf<T>() ? (T)0 : ln0 == ninf<T>() ? (T)0 : ex(site ? ln0 - v : v - ln0);
                        lsum += (double)((site ? v : ln0) + lg1p(e));
                        if (last) {
                            const T so = score_in_order(w, wt, l);
                            if (so > bv) {
                                bv = so;
                                ba = x;
                            }
                            continue;
                        }
                        const T z = (site ? (T)1 + (v - v) : e) / ((T)1 + e);
                        scatter3<NG>(w, z, ac);
                    }
                    llr_w += wave_sum(lsum);
                    if (last && a.sites) {
                        const T bm = wave_max(bv);
                        const int64_t cand = wave_min_i64(bv == bm ? ba : INT64_MAX);
                        // reported when that window's posterior is at least 1/2
                        const bool keep = (double)bm + lmix >= lnone;
                        if (lane == 0) a.sites[b * a.site_stride + i] = keep ? (int32_t)cand : -1;
                    }
                    continue;
                }
                // windows past the end read the last one and score -inf
                auto win_at = [&](int x) { return load_win(W, s0 + (x < L ? x : L - 1)); };
                const bool held = L <= 64 * kNC;
                T s[kNC];
                T mx = ninf<T>();
                double sm = 0;  // FP64 sum of exponentials in both precisions
                if (held) {
#pragma unroll
                    for (int c = 0; c < kNC; ++c) {
                        s[c] = ninf<T>();
                        if (64 * c < L) {
                            const int x = 64 * c + lane;
                            const T v = score3<T, NG>(win_at(x), W3);
                            s[c] = x < L ? v : ninf<T>();
                            mx = s[c] > mx ? s[c] : mx;
                        }
                    }
                } else {
                    for (int x = lane; x < L; x += 64) {
                        const T v = score3<T, NG>(win_at(x), W3);
                        mx = v > mx ? v : mx;
                    }
                }
                const T M = wave_max(mx);
                const T Mr = M > ninf<T>() ? M : (T)0;  // no finite score: every term is 0, not NaN
                if (held) {
#pragma unroll
                    for (int c = 0; c < kNC; ++c)
                        if (64 * c < L) {
                            const T e = ex(s[c] - Mr);
                            sm += s[c] > ninf<T>() ? (double)e : 0.0;
                            if (!last) s[c] = e;
                        }
                } else {
                    for (int x = lane; x < L; x += 64) {
                        const T v = score3<T, NG>(win_at(x), W3);
                        sm += v > ninf<T>() ? (double)ex(v - Mr) : 0.0;
                    }
                }
                const double Ssum = wave_sum(sm);
                const double lse = (double)M + log(Ssum);
                // OOPS: LLR_i = LSE_i - ln L_i, Z = e^{s - LSE_i}.  ZOOPS: the
                // sequence holds no site with probability 1 - gamma, so
                // LLR_i = ln((1 - gamma) + gamma e^{LSE_i} / L_i) and
                // Z = gamma e^s / (L_i e^{LLR_i}); q_i = sum_a Z is its site mass
                double li, f, qi = 1.0;  // Z = f e^{s - Mr}
                if (MODEL == PM_ZOOPS) {
                    const double lsite = lmix - log((double)L) + lse;
                    li = log_add(lnone, lsite);
                    qi = exp(lsite - li);
                    f = Ssum > 0 ? qi / Ssum : qi;  // (no finite score: no counts)
                } else {
                    li = lse - log((double)L);
                    f = 1.0 / Ssum;
                }
                llr_w += li;
                if (last) {
                    if (a.sites) {
                        T bv = ninf<T>();
                        int64_t ba = 0;
                        auto consider = [&](int x) {
                            const T so = score_in_order(win_at(x), wt, l);
                            if (so > bv) {
                                bv = so;
                                ba = x;
                            }
                        };
                        if (held) {
                            uint32_t near = 0;
#pragma unroll
                            for (int c = 0; c < kNC; ++c)
                                if (64 * c + lane < L && s[c] >= M - tol) near |= 1u << c;
                            for (; near; near &= near - 1) consider(64 * (__ffs(near) - 1) + lane);
                        } else {
                            for (int x = lane; x < L; x += 64)
                                if (score3<T, NG>(win_at(x), W3) >= M - tol) consider(x);
                        }
                        const T bm = wave_max(bv);
                        const int64_t cand = wave_min_i64(bv == bm ? ba : INT64_MAX);
                        if (lane == 0) a.sites[b * a.site_stride + i] = qi >= 0.5 ? (int32_t)cand : -1;
                    }
                } else {
                    const T fz = (T)f;
                    if (held) {
#pragma unroll
                        for (int c = 0; c < kNC; ++c)
                            if (64 * c + lane < L) scatter3<NG>(load_win(W, s0 + 64 * c + lane), s[c] * fz, ac);
                    } else {
                        for (int x = lane; x < L; x += 64) {
                            const Win w = win_at(x);
                            scatter3<NG>(w, ex(score3<T, NG>(w, W3) - Mr) * fz, ac);
                        }
                    }
                }
            }
            if (lane == 0) llr_slot[slot] = llr_w;  // (the same in every lane)
        }
        __syncthreads();
        double llr = 0;
        for (int w = 0; w < kSlots; ++w) llr += llr_slot[w];
        if (tid == 0) {
            a.J[b * (a.iters + 1) + it] = llr + beta * pr;
            if (a.llr) a.llr[b * (a.iters + 1) + it] = llr;
        }
        if (!last) {
            // counts of the slots, then of every letter and position, in FP64
            for (int e = tid; e < 64 * NG; e += kThreads) {
                double cs = 0;
#pragma unroll
                for (int w = 0; w < kSlots; ++w) cs += C3[w][e];
                csum[e] = cs;
            }
            __syncthreads();
            for (int i = tid; i < AL; i += kThreads) {
                const int c = i / l, p = i % l;
                const int sh = 4 - 2 * (p % 3);          // the letter's field in an entry's number
                const int rest = (1 << sh) - 1;
                const double *cq = csum + 64 * (p / 3);
                double cs = 0;
                for (int u = 0; u < 16; ++u) cs += cq[((u & ~rest) << 2) | (c << sh) | (u & rest)];
                th[i] = cs;
            }
            __syncthreads();
            // theta' = (counts + beta*bg) / (t + beta); every column's counts sum
            // to t, so dividing by the column's own total is the same update and
            // keeps each column exactly on the simplex under rounding
            for (int p = tid; p < l; p += kThreads) {
                double tot = 0;
                for (int c = 0; c < 4; ++c) tot += th[c * l + p];
                colsum[p] = tot + beta;
                if (p == 0) ztot = tot;
            }
            __syncthreads();
            for (int i = tid; i < AL; i += kThreads) th[i] = (th[i] + beta * a.bg[i / l]) / colsum[i % l];
            // the mixing parameter's update: the posterior mass (every
            // column's counts total it) over t sequences (ZOOPS) or x windows
            // (TCM), capped at 1 against rounding
            if (MODEL == PM_ZOOPS) mix = fmin(1.0, ztot / (double)t);
            else if (MODEL == PM_TCM) mix = fmin(1.0, ztot / (double)I.x);
            __syncthreads();
        }
    }
    for (int i = tid; i < AL; i += kThreads) a.theta_out[b * AL + i] = th[i];
    if (tid == 0 && a.mix_out) a.mix_out[b] = mix;
}

template <typename T, int NG, int WAVES>
static void launch_waves(const EmArgs &a, size_t lds, hipStream_t st)
{
    // the largest number of models that is this form's (tile_takes)
    int64_t most = a.B;
    if (tile_takes(a.B, a.tile_pct)) {
        most = 1;
        for (int64_t r = 1; (r - 1) * kTileRound < a.B; ++r) {
            const int64_t n = std::min({a.B, r * kTileRound, (r * kTileRound * a.tile_pct + 99) / 100 - 1});
            if (n > (r - 1) * kTileRound) most = std::max(most, n);
        }
    }
    const dim3 grid((unsigned)most);
    if (a.model == PM_OOPS) hipLaunchKernelGGL((k_em_dna<T, NG, PM_OOPS, WAVES>), grid, dim3(64 * WAVES), lds, st, a);
    else if (a.model == PM_ZOOPS) hipLaunchKernelGGL((k_em_dna<T, NG, PM_ZOOPS, WAVES>), grid, dim3(64 * WAVES), lds, st, a);
    else hipLaunchKernelGGL((k_em_dna<T, NG, PM_TCM, WAVES>), grid, dim3(64 * WAVES), lds, st, a);
}

// the kernel for l positions; four waves only up to eight tables (launch_em_dna)
template <typename T, int WAVES>
static int launch_positions(const EmArgs &a, size_t lds, hipStream_t st)
{
    switch ((a.l + 2) / 3) {
    case 1: launch_waves<T, 1, WAVES>(a, lds, st); break;
    case 2: launch_waves<T, 2, WAVES>(a, lds, st); break;
    case 3: launch_waves<T, 3, WAVES>(a, lds, st); break;
    case 4: launch_waves<T, 4, WAVES>(a, lds, st); break;
    case 5: launch_waves<T, 5, WAVES>(a, lds, st); break;
    case 6: launch_waves<T, 6, WAVES>(a, lds, st); break;
    case 7: launch_waves<T, 7, WAVES>(a, lds, st); break;
    case 8: launch_waves<T, 8, WAVES>(a, lds, st); break;
    default:
        if constexpr (WAVES == 8) {
            if (a.l <= 27) launch_waves<T, 9, WAVES>(a, lds, st);
            else if (a.l <= 30) launch_waves<T, 10, WAVES>(a, lds, st);
            else launch_waves<T, 11, WAVES>(a, lds, st);
        }
    }
    PM_LAUNCHED();
    return PM_OK;
}

}  // namespace pm
