// a7 - a9 for many DNA models of one instance in FP64: OOPS, ZOOPS and TCM EM
// of sixteen models at a time, the M-step on the FP64 matrix instructions.
// Included by one source per sequence model.
//
// em_dna.h gives a model a workgroup, and its time goes to LDS updates of 64
// lanes that meet on the same entries of a table.  Here a workgroup holds the
// tables of sixteen models, a wave takes four windows of a sequence at once,
// and lane 16 g + m looks at window g for model m:
//  * a score is a read of ceil(l/3) three-letter tables as there, but the
//    sixteen lanes of a window read sixteen consecutive entries, so that the
//    four rows rarely meet on a bank;
//  * the posteriors of the step are, as they lie, the right operand of
//    v_mfma_f64_16x16x4_f64; its left operand says which of the four letters
//    stands at each of four positions in the four windows (formed from the
//    lane's own window), and the sixteen results a lane's model gets per
//    instruction are the counts of those letters: ceil(l/4) instructions per
//    step and no LDS updates at all.
// The waves of a workgroup share the windows of each sequence.  Posteriors are
// formed against a reference that no score passes (the sum of every position's
// largest log-odds), unnormalised over a sequence, and the sequence's counts
// are scaled by one factor at its end, when the waves have exchanged their
// sums.  Should a sum be so small that terms may have been lost, the sequence
// is swept again against its largest score.
//
// Bound by the matrix instructions (68 cycles each, in which the SIMD issues no
// vector instruction) and, about even, by the vector work of a step, mostly
// the exponential: a step of four windows takes 128 cycles of a CU at l = 15,
// 122 by the count of its instructions.  Twelve waves, whose registers hold a
// sequence's counts and the totals up to l = 24; with sixteen (l = 18: 5.2
// instead of 4.2 ms) they go to memory, eight are too few (l = 14: 3.4 instead
// of 3.2 ms).  Measured against the workgroup per model, 4096 models, 20
// sequences of 1000, 10 iterations: FP64 OOPS of l = 14, 18, 22: 6.9, 7.6, 8.9
// -> 3.2, 3.7, 4.5 ms; ZOOPS in FP32, l = 18: 7.5 -> 3.8 ms; TCM in FP64: 6.2,
// 6.8, 8.0 -> 3.7, 4.1, 4.7 ms; a (15,4) pass of 20 600 models, 5 iterations
// (six rounds of which the last is nearly empty): 11.4 -> 7.3 ms.  FP32 calls
// take this form too: all arithmetic in FP64, sites by FP32 scores.
//
// It needs sixteen models per CU to fill the chip (tile_takes).
#pragma once

#include <utility>

#include "dna3.h"
#include "em_vec.h"

namespace pm {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kTileModels = 16;

// e^x for x <= 0 (or a rounding above): x = (64 k + j) ln 2 / 64 + r, T[j] =
// 2^(j / 64), and the Taylor series of e^r to r^5 (remainder below 2^-54)
__device__ __forceinline__ double exp_le0(double x, const double *T)
{
    const double n = rint(x * 92.33248261893597);
    double r = fma(n, -0.6931471805599453 / 64, x);
    r = fma(n, -2.3190468138462996e-17 / 64, r);
    double p = 1.0 / 120.0;
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0) * r;
    const int k = (int)n;
    const double v = T[k & 63];
    return x < -800.0 ? 0.0 : ldexp(fma(v, p, v), k >> 6);
}

// smallest sequence sum (against the highest reference) that has lost nothing:
// terms 2^-53 below it are still normal numbers
constexpr double kTileSumMin = 1e-280;

// over the four windows of a step
__device__ __forceinline__ double over_windows(double v)
{
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// the score of the window at code for the lane's model (W3m: its first entry)
template <int NG, int Q = 0>
__device__ __forceinline__ double tile_score(const uint8_t *code, const double *W3m)
{
    const double v = W3m[(64 * Q + code[3 * Q]) * kTileModels];
    if constexpr (Q + 1 < NG) return v + tile_score<NG, Q + 1>(code, W3m);
    else return v;
}

// counts of the step's windows with posteriors P: tile T holds positions 4 T ..
// 4 T + 3; code is at the lane's position of the first, letter its letter on top
template <int NT>
__device__ __forceinline__ void tile_counts(const uint8_t *code, uint32_t letter, double P, f64x4 (&acc)[NT])
{
#pragma unroll
    for (int T = 0; T < NT; ++T) {
        const double is = __hiloint2double((code[4 * T] ^ letter) < 16u ? 0x3ff00000 : 0, 0);
        acc[T] = __builtin_amdgcn_mfma_f64_16x16x4f64(is, P, acc[T], 0, 0, 0);
    }
}

constexpr int kTileSums = 64;  // sequences whose sums are kept for their logarithms
constexpr int kTilePad = 64;  // symbols looked at past the end of the input, at most

// LDS of a workgroup, in bytes, without the input's codes
template <int NG, int NT, int NW>
constexpr size_t tile_lds()
{
    return (size_t)8 * (64 + kTileModels * (64 * NG + 4 * 4 * NT + 2 * 4 * NT + 2 * NW + 2 * kTileSums + 1)) +
           (size_t)4 * kTileModels * NW;
}

template <int NG, int NT, int NW, bool TCM>
__global__ void __launch_bounds__(64 * NW, NW / 4) k_em_tile(const EmArgs a)
{
    constexpr int M = kTileModels, LP = 4 * NT;
    int64_t nvalid = a.n_dev ? *a.n_dev : a.B;
    if (nvalid > a.B) nvalid = a.B;
    const int64_t b0 = (int64_t)blockIdx.x * M;
    if (!tile_takes(nvalid, a.tile_pct) || b0 >= nvalid) return;  // uniform over the workgroup

    extern __shared__ __align__(16) uint8_t lds[];
    double *W3 = reinterpret_cast<double *>(lds);  // [NG][64][M] three-letter sums; then the waves' counts
    double *wt = W3 + 64 * NG * M;                 // [LP][4][M] log-odds
    double *top = wt + 4 * LP * M;                 // [LP][M] largest log-odds of a position
    double *pri = top + LP * M;                    // [LP][M] share of the prior
    double *part = pri + LP * M;                   // [NW][M] sums over a wave's windows
    double *bestv = part + NW * M;                 // [NW][M] best window of a wave: score
    double *sums = bestv + NW * M;                 // [kTileSums][M] sums of sequences
    double *refs = sums + kTileSums * M;           // [kTileSums][M] and their references
    double *mass = refs + kTileSums * M;           // [M]
    int32_t *besti = reinterpret_cast<int32_t *>(mass + M);     // [NW][M] and place
    double *exps = reinterpret_cast<double *>(besti + NW * M);  // [64] 2^(j / 64)
    uint8_t *codes = reinterpret_cast<uint8_t *>(exps + 64);        // the three letters from every symbol on

    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, m = lane & 15;
    const pm_inst &I = a.one;
    const int l = a.l, t = I.t, AL = 4 * l;
    const double beta = a.beta;
    const int64_t b = b0 + m, bc = b < nvalid ? b : nvalid - 1;  // lanes past the end repeat the last model
    const bool vb = b < nvalid;
    const double bgl = a.bg[g], lbg = log(bgl);  // the lane's letter is g wherever positions go by waves
    const uint32_t letter = (uint32_t)(m & 3) << 4;
    const int64_t *O = I.offsets;
    const int n_codes = (int)I.n_total + kTilePad;
    for (int i = tid; i < n_codes; i += 64 * NW) codes[i] = i < I.n_total ? (uint8_t)(load_win(I.packed, i).hi >> 26) : 0;
    if (tid < 64) exps[tid] = exp2((double)tid / 64.0);
    const double *W3m = W3 + m;

    // Groups of waves that take a sequence each, round by round: fewer rounds
    // end less often with a barrier, but wait for their longest sequence.  In
    // windows per wave; a round's end costs about as much as 16 of them.
    int groups = 1;
    for (int G = 1, best = 0; G <= 4; G *= 2) {
        int cost = 0;
        for (int i = 0; i < t; i += G) {
            int longest = 0;
            for (int k = i; k < min(t, i + G); ++k) longest = max(longest, (int)(O[k + 1] - O[k]) - l + 1);
            cost += ((longest * G + NW - 1) / NW + 7) / 8 * 8 + 16;
        }
        if (G == 1 || cost < best) {
            best = cost;
            groups = G;
        }
    }
    groups = __builtin_amdgcn_readfirstlane(groups);
    const int gw = NW / groups, grp = wv / gw, w_grp = wv % gw, rounds = (t + groups - 1) / groups;

    // position p of the models from theta: log-odds, their largest, the prior
    auto column = [&](int p, double th) {
        const double lt = log(th), w = lt - lbg;
        wt[(4 * p + g) * M + m] = w;
        double mx = fmax(w, __shfl_xor(w, 16));
        mx = fmax(mx, __shfl_xor(mx, 32));
        const double pr = beta != 0 ? over_windows(bgl * lt) : 0.0;
        if (g == 0) {
            top[p * M + m] = mx;
            pri[p * M + m] = pr;
        }
    };
    for (int p = wv; p < LP; p += NW) {
        if (p < l) {
            const double th = a.theta0[bc * AL + g * l + p];
            column(p, th);
            if (a.iters == 0 && vb) a.theta_out[b * AL + g * l + p] = th;
        } else {
            wt[(4 * p + g) * M + m] = 0;
        }
    }
    double mix = a.mix0;
    __syncthreads();

    for (int it = 0; it <= a.iters; ++it) {
        const bool last = it == a.iters;
        const double lmix = a.model == PM_OOPS ? 0.0 : log(mix), lnone = a.model == PM_OOPS ? 0.0 : log1p(-mix);
        for (int e = tid; e < 64 * M; e += 64 * NW) {
            const int em = e & 15, u = e >> 4;
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                double v = wt[(12 * q + (u >> 4)) * M + em];
                if (3 * q + 1 < LP) v += wt[(12 * q + 4 + ((u >> 2) & 3)) * M + em];
                if (3 * q + 2 < LP) v += wt[(12 * q + 8 + (u & 3)) * M + em];
                W3[64 * M * q + e] = v;
            }
        }
        double ref = 0, prior = 0;
        for (int p = 0; p < l; ++p) {
            ref += top[p * M + m];
            prior += pri[p * M + m];
        }
        __syncthreads();

        f64x4 acc[NT], tot[NT];
#pragma unroll
        for (int T = 0; T < NT; ++T) tot[T] = f64x4{0, 0, 0, 0};
        double llr = 0;
        const double c0 = mix * exp(ref);
        for (int r = 0; r < rounds; ++r) {
            const int i = r * groups + grp;
            const bool has = i < t;  // uniform over the wave; all waves meet the barriers
            const int64_t s0 = has ? O[i] : 0;
            const int L = has ? __builtin_amdgcn_readfirstlane((int)(O[i + 1] - s0)) - l + 1 : 0;
            const int per = ((L + gw - 1) / gw + 7) & ~7;
            const int lo = w_grp * per, hi = min(L, lo + per);
            const uint8_t *at = codes + s0 + g;            // window g of the step at w0: at[w0]
            const uint8_t *pos = at + (m >> 2);            // and the lane's position of it
            if (last && a.sites) {
                // the best window, by scores summed in order in the caller's precision
                double bv = ninf<double>();
                int ba = 0;
                for (int w0 = lo; w0 < hi; w0 += 4) {
                    const int w = w0 + g;
                    double s = 0;
                    if (a.fp32) {
                        float sf = 0;
                        for (int p = 0; p < l; ++p) sf += (float)wt[(4 * p + (at[w0 + p] >> 4)) * M + m];
                        s = sf;
                    } else {
                        for (int p = 0; p < l; ++p) s += wt[(4 * p + (at[w0 + p] >> 4)) * M + m];
                    }
                    if (w < hi && s > bv) {
                        bv = s;
                        ba = w;
                    }
                }
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) {
                    const double v = __shfl_xor(bv, o);
                    const int at = __shfl_xor(ba, o);
                    if (v > bv || (v == bv && at < ba)) {
                        bv = v;
                        ba = at;
                    }
                }
                if (g == 0) {
                    bestv[wv * M + m] = bv;
                    besti[wv * M + m] = ba;
                }
            }
            // over the group's waves: the earliest of the best windows; kept if
            // `keep` says so
            auto site = [&](auto keep) {
                if (!has || w_grp != 0 || g != 0) return;
                double bv = ninf<double>();
                int ba = 0;
                for (int w = wv; w < wv + gw; ++w) {
                    const double v = bestv[w * M + m];
                    if (v > bv) {
                        bv = v;
                        ba = besti[w * M + m];
                    }
                }
                if (vb) a.sites[b * a.site_stride + i] = keep(bv) ? ba : -1;
            };
            if (TCM) {
                // every window its own two-component mixture: with e what the
                // smaller component is of the larger, its log-likelihood is the
                // larger plus ln(1 + e), the logarithms taken of products
                double prod = 1.0;
                int terms = 0;
                auto posterior = [&](int w0) {
                    const double v = lmix + tile_score<NG>(at + w0, W3m);
                    const bool site = !(v <= lnone);  // (a NaN or infinite score: a NaN posterior)
                    const double e = v == ninf<double>() || lnone == ninf<double>()
                                         ? 0.0
                                         : exp_le0(site ? lnone - v : v - lnone, exps);
                    const double d = 1.0 + e;
                    double y = __builtin_amdgcn_rcp(d);  // 1 / d, 1 <= d <= 2
                    y = fma(fma(-d, y, 1.0), y, y);
                    y = fma(fma(-d, y, 1.0), y, y);
                    const bool in = w0 + g < hi;
                    llr += in ? site ? v : lnone : 0.0;
                    prod *= in ? d : 1.0;
                    return in ? site ? y + (v - v) : e * y : 0.0;
                };
                for (int w0 = lo; w0 < hi; w0 += 8) {
                    const double P0 = posterior(w0), P1 = posterior(w0 + 4);
                    if (!last) {
                        tile_counts<NT>(pos + w0, letter, P0, tot);
                        tile_counts<NT>(pos + w0 + 4, letter, P1, tot);
                    }
                    if (++terms == 256) {
                        llr += log(prod);
                        prod = 1.0;
                        terms = 0;
                    }
                }
                llr += log(prod);
                if (last && a.sites) {
                    __syncthreads();
                    // reported when that window's posterior is at least 1/2
                    site([&](double bv) { return bv + lmix >= lnone; });
                    __syncthreads();
                }
                continue;
            }
            // the wave's windows against reference rf: their sum, and counts
            auto sweep = [&](double rf, bool skip_nan) {
                double sum = 0;
#pragma unroll
                for (int T = 0; T < NT; ++T) acc[T] = f64x4{0, 0, 0, 0};
                for (int w0 = lo; w0 < hi; w0 += 8) {
                    const double e0 = exp_le0(tile_score<NG>(at + w0, W3m) - rf, exps);
                    const double e1 = exp_le0(tile_score<NG>(at + w0 + 4, W3m) - rf, exps);
                    const double P0 = w0 + g < hi ? e0 : 0.0, P1 = w0 + 4 + g < hi ? e1 : 0.0;
                    sum += skip_nan && !(P0 == P0) ? 0.0 : P0;
                    sum += skip_nan && !(P1 == P1) ? 0.0 : P1;
                    if (!last) {
                        tile_counts<NT>(pos + w0, letter, P0, acc);
                        tile_counts<NT>(pos + w0 + 4, letter, P1, acc);
                    }
                }
                sum = over_windows(sum);
                if (g == 0) part[wv * M + m] = sum;
                __syncthreads();
                sum = 0;
                for (int w = wv - w_grp; w < wv - w_grp + gw; ++w) sum += part[w * M + m];
                return sum;
            };
            double rf = ref, sum = sweep(ref, false);
            const bool low = has && !(sum >= kTileSumMin);
            if (__syncthreads_or(low)) {
                double mx = ninf<double>();
                for (int w0 = lo; w0 < hi; w0 += 4) {
                    const double s = tile_score<NG>(at + w0, W3m);
                    mx = w0 + g < hi && s > mx ? s : mx;
                }
                mx = fmax(mx, __shfl_xor(mx, 16));
                mx = fmax(mx, __shfl_xor(mx, 32));
                if (g == 0) part[wv * M + m] = mx;
                __syncthreads();
                for (int w = wv - w_grp; w < wv - w_grp + gw; ++w) mx = fmax(mx, part[w * M + m]);
                __syncthreads();
                // no finite score: every term and the sum are 0 (the log of the sum
                // -inf), against any finite reference
                if (low) rf = mx > ninf<double>() ? mx : 0.0;
                sum = sweep(rf, low);
                __syncthreads();
            }
            if (has && w_grp == 0 && g == 0) {
                sums[(i % kTileSums) * M + m] = sum;
                refs[(i % kTileSums) * M + m] = rf;
            }
            // OOPS: Z = e^{s - rf} / sum.  ZOOPS: the sequence holds a site with
            // probability q = c sum / (c sum + (1 - mix) L), c = mix e^rf, and Z =
            // q e^{s - rf} / sum; by logarithms where those leave FP64's range
            double qi = 1.0, f = 1.0 / sum;
            if (a.model == PM_ZOOPS && has) {
                const double cs = (low ? mix * exp(rf) : c0) * sum, no = (1.0 - mix) * (double)L;
                const bool by_log = !(cs > 1e-290 && cs < 1e290);
                qi = cs / (cs + no);
                if (__ballot(by_log)) {
                    const double lsite = lmix - log((double)L) + rf + log(sum);
                    if (by_log) qi = exp(lsite - log_add(lnone, lsite));
                    if (!(sum > 0)) sum = 1.0;  // no finite score: qi = 0 and no counts
                }
                f = qi / sum;
            }
            if (last) {
                if (a.sites) {
                    site([&](double) { return qi >= 0.5; });
                    __syncthreads();
                }
            } else if (has) {
#pragma unroll
                for (int T = 0; T < NT; ++T) tot[T] += acc[T] * f;
            }
            // ---- log-likelihoods of the kept sums: OOPS' ln(sum e^rf / L),
            // ZOOPS' ln((1 - mix) + mix sum e^rf / L)
            const int i1 = min(t, (r + 1) * groups);  // sequences done
            if (i1 % kTileSums == 0 || i1 == t) {
                const int i0 = (i1 - 1) / kTileSums * kTileSums;
                __syncthreads();
                for (int e = tid; e < (i1 - i0) * M; e += 64 * NW) {  // (e % M is m)
                    const int k = i0 + e / M;
                    const double lse = refs[e] + log(sums[e]) - log((double)(O[k + 1] - O[k] - l + 1));
                    sums[e] = a.model == PM_ZOOPS ? log_add(lnone, lmix + lse) : lse;
                }
                __syncthreads();
                for (int e = 0; e < i1 - i0; ++e) llr += sums[e * M + m];
                __syncthreads();
            }
        }
        if (TCM) {  // over the lanes' and the waves' windows
            llr = over_windows(llr);
            if (g == 0) part[wv * M + m] = llr;
            __syncthreads();
            llr = 0;
            for (int w = 0; w < NW; ++w) llr += part[w * M + m];
        }
        if (tid < M && vb) {
            a.J[b * (a.iters + 1) + it] = llr + beta * prior;
            if (a.llr) a.llr[b * (a.iters + 1) + it] = llr;
        }
        if (last) break;
        // ---- counts over the waves, four of them at a time through the tables'
        // LDS, in the waves' order: lane 16 c + m of position p's wave gets
        // letter c of model m
        constexpr int NP = (LP + NW - 1) / NW;
        double cs[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) cs[k] = 0;
        for (int w4 = 0; w4 < NW; w4 += 4) {
            __syncthreads();
            if (wv >= w4 && wv < w4 + 4)
#pragma unroll
                for (int T = 0; T < NT; ++T)
#pragma unroll
                    for (int r = 0; r < 4; ++r) W3[((wv - w4) * LP + 4 * T + r) * 64 + lane] = tot[T][r];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int p = wv + NW * k;
                if (p < l)
                    for (int w = 0; w < 4; ++w) cs[k] += W3[(w * LP + p) * 64 + lane];
            }
        }
        // theta' = (counts + beta*bg) / (t + beta); every column's counts sum to
        // t, so dividing by the column's own total is the same update and keeps
        // each column exactly on the simplex under rounding
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int p = wv + NW * k;
            if (p < l) {
                const double tp = over_windows(cs[k]);
                if (p == 0 && g == 0) mass[m] = tp;
                const double th = (cs[k] + beta * bgl) / (tp + beta);
                if (it + 1 == a.iters && vb) a.theta_out[b * AL + g * l + p] = th;
                column(p, th);
            }
        }
        __syncthreads();
        // the mixing parameter's update, capped at 1 against rounding
        if (a.model == PM_ZOOPS) mix = fmin(1.0, mass[m] / (double)t);
        else if (a.model == PM_TCM) mix = fmin(1.0, mass[m] / (double)I.x);
    }
    if (tid < M && vb && a.mix_out) a.mix_out[b] = mix;
}

template <int NG, int NT, int NW, bool TCM>
static int launch_tile_shape(const EmArgs &a, hipStream_t st)
{
    const size_t lds = tile_lds<NG, NT, NW>() + (size_t)a.one.n_total + kTilePad;
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)k_em_tile<NG, NT, NW, TCM>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  device_lds_bytes());
        (void)hipGetLastError();
        attr = true;
    }
    const dim3 grid((unsigned)((a.B + kTileModels - 1) / kTileModels));
    hipLaunchKernelGGL((k_em_tile<NG, NT, NW, TCM>), grid, dim3(64 * NW), lds, st, a);
    PM_LAUNCHED();
    return PM_OK;
}

template <bool TCM>
static int launch_tile(const EmArgs &a, hipStream_t st)
{
    if (a.l <= 12) return launch_tile_shape<4, 3, 12, TCM>(a, st);
    if (a.l <= 15) return launch_tile_shape<5, 4, 12, TCM>(a, st);
    if (a.l <= 16) return launch_tile_shape<6, 4, 12, TCM>(a, st);
    if (a.l <= 18) return launch_tile_shape<6, 5, 12, TCM>(a, st);
    if (a.l <= 20) return launch_tile_shape<7, 5, 12, TCM>(a, st);
    if (a.l <= 21) return launch_tile_shape<7, 6, 12, TCM>(a, st);
    return launch_tile_shape<8, 6, 12, TCM>(a, st);
}

}  // namespace pm
