// Gibbs site sampling as the local optimiser of a bucket, in place of EM.
//
// Sec. 1 and Sec. 3 of the paper name Gibbs sampling beside EM as the local
// search that PROJECTION seeds; the sampler is the site sampler of Lawrence
// et al. (cited there).  Per model: start from the best start of every
// sequence under the bucket's theta0; a sweep visits the sequences in order
// and redraws each one's start from the motif model of the other t-1 sites
// (pseudocounts beta * bg); the alignment of largest log-odds score F over
// the start and every sweep is the answer.  Random numbers come from
// Philox4x64-10 (Salmon et al., SC'11) keyed by the seed, one block per
// (sweep, sequence, model), so any model's chain is reproducible on its own.
//
// One wave per model, four models (one instance) per workgroup; the packed
// instance is staged in LDS once for the four.  A draw scores the sequence's
// starts in contiguous chunks per lane (lane order = start order), so a wave
// scan of the lanes' weight sums gives every lane's running sum and the lane
// holding the drawn start finds it in its chunk.  All arithmetic is FP64.
//
// DNA (k_gibbs_dna): a start's weight is a product of l ratios
// theta / bg, so it is formed as a product of ceil(l/3) entries of tables of
// 64 three-letter products, with no logarithm or exponential per start; the
// ratios themselves take t values per letter and are looked up.  A lane's
// weights (up to 16 starts) stay in registers from the sum to the walk, its
// windows come from one window shifted along, and the sweep's random numbers
// are formed by one lane per sequence.  4 096 chains of the (18,6) workload,
// 10 sweeps: 33.9 ms by a dependent pair of LDS reads per position and start,
// three times per draw, with an exponential per start and the random number
// formed in every lane, 1.64 ms this way (LDS reads of the tables bound it).
// Where l ratios could leave the FP64 range
// (kGibbsLogRange) the tables hold sums of logarithms instead.
#include <math.h>

#include "dna3.h"

namespace pm {

constexpr int kGibbsWaves = 4;
constexpr int kGibbsThreads = kGibbsWaves * kWave;
constexpr int kGibbsMaxT = 512;

struct GibbsArgs {
    pm_inst one;
    const double *theta0;
    const double *bg;
    const int64_t *n_dev;
    double *theta_out;
    double *F;
    int32_t *sites;
    int64_t B;
    int l, sweeps;
    double beta;
    uint64_t seed;
    int seq_cap;  // LDS words of the packed input (0: global)
    int off_cap;  // LDS offsets (0: global)
};

__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t lo0 = M0 * c[0], hi0 = __umul64hi(M0, c[0]);
        const uint64_t lo1 = M1 * c[2], hi1 = __umul64hi(M1, c[2]);
        const uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
        k0 += 0x9E3779B97F4A7C15ull;
        k1 += 0xBB67AE8584CAA73Bull;
    }
}

// uniform in [0, 1) with 53 random bits for (sweep, sequence, model)
__device__ __forceinline__ double gibbs_uniform(uint64_t seed, int sweep, int i, int64_t model)
{
    uint64_t c[4] = {(uint64_t)sweep, (uint64_t)i, (uint64_t)model, 0};
    philox4x64_10(c, seed, 0);
    return (double)(c[0] >> 11) * (1.0 / 9007199254740992.0);
}

// LDS written by lanes of the wave before, read by other lanes after: the
// hardware takes a wave's LDS operations in order, and the fences (no
// instructions at this scope) keep the compiler from holding a value that
// another lane has changed
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// score of start a of the sequence beginning at symbol s0 under table Wt
__device__ __forceinline__ double start_score(const uint32_t *W, int64_t s0, int64_t a, const double *Wt, int l)
{
    double v = 0;
    for (int p = 0; p < l; ++p) v += Wt[prot_sym(W, s0 + a + p) * l + p];
    return v;
}

// F = sum n ln(theta / bg) over entries with n > 0, theta = (n + beta bg)/(t + beta)
__device__ __forceinline__ double alignment_F(const int32_t *n, const double *bg, int A, int l, int t, double beta)
{
    double f = 0;
    for (int e = lane_id(); e < A * l; e += kWave) {
        const int c = e / l;
        if (n[e] > 0) f += (double)n[e] * log(((double)n[e] + beta * bg[c]) / ((double)t + beta) / bg[c]);
    }
    return wave_sum(f);
}

// (value, index) with the larger value, the smaller index on ties
__device__ __forceinline__ void wave_argmax(double &v, int64_t &ix)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(v, o);
        const int64_t oi = __shfl_xor(ix, o);
        if (ov > v || (ov == v && oi < ix)) {
            v = ov;
            ix = oi;
        }
    }
}

// Protein models.
__global__ void __launch_bounds__(kGibbsThreads) k_gibbs(const GibbsArgs g)
{
    extern __shared__ __align__(16) uint32_t dyn[];
    __shared__ double Wt[kGibbsWaves][20 * 32];
    __shared__ double bgs[20];
    __shared__ int32_t cnt[kGibbsWaves][20 * 32];
    __shared__ int32_t cur[kGibbsWaves][kGibbsMaxT];
    __shared__ int32_t bst[kGibbsWaves][kGibbsMaxT];

    const pm_inst &I = g.one;
    const int tid = threadIdx.x, wv = tid / kWave, lane = lane_id();
    constexpr int A = 20;
    const int l = g.l, AL = A * l, t = I.t;
    uint32_t *seq = dyn;
    int64_t *offs = reinterpret_cast<int64_t *>(dyn + ((g.seq_cap + 1) & ~1));
    const int seq_words = g.seq_cap ? (int)((I.n_total + 5) / 6 + 4) : 0;
    for (int i = tid; i < seq_words; i += kGibbsThreads) seq[i] = I.packed[i];
    if (g.off_cap)
        for (int i = tid; i <= t; i += kGibbsThreads) offs[i] = I.offsets[i];
    for (int c = tid; c < A; c += kGibbsThreads) bgs[c] = g.bg[c];
    __syncthreads();
    const uint32_t *W = g.seq_cap ? seq : I.packed;
    const int64_t *O = g.off_cap ? offs : I.offsets;

    int64_t nvalid = g.n_dev ? *g.n_dev : g.B;
    if (nvalid > g.B) nvalid = g.B;
    const int64_t b = (int64_t)blockIdx.x * kGibbsWaves + wv;
    if (b >= nvalid) return;  // whole waves leave; no workgroup barrier follows

    double *Tw = Wt[wv];
    int32_t *n = cnt[wv];
    int32_t *cs = cur[wv];
    int32_t *bs = bst[wv];
    const double beta = g.beta;

    // start: the best start of every sequence under theta0 (first on ties)
    for (int e = lane; e < AL; e += kWave) Tw[e] = log(g.theta0[b * AL + e]) - log(bgs[e / l]);
    wave_sync();
    for (int i = 0; i < t; ++i) {
        const int64_t s0 = O[i], L = O[i + 1] - s0 - l + 1;
        double bv = -INFINITY;
        int64_t ba = lane < L ? lane : INT64_MAX;  // (no finite score: the first start)
        for (int64_t a = lane; a < L; a += kWave) {
            const double v = start_score(W, s0, a, Tw, l);
            if (v > bv) {
                bv = v;
                ba = a;
            }
        }
        wave_argmax(bv, ba);
        if (lane == 0) cs[i] = (int32_t)ba;
    }
    for (int e = lane; e < AL; e += kWave) n[e] = 0;
    wave_sync();
    for (int i = 0; i < t; ++i)
        if (lane < l) atomicAdd(&n[(int)prot_sym(W, O[i] + cs[i] + lane) * l + lane], 1);
    wave_sync();
    double Fb = alignment_F(n, bgs, A, l, t, beta);
    const int it1 = g.sweeps + 1;
    if (g.F && lane == 0) g.F[b * it1] = Fb;
    for (int i = lane; i < t; i += kWave) bs[i] = cs[i];

    const double tm1 = (double)(t - 1) + beta;
    for (int r = 0; r < g.sweeps; ++r) {
        for (int i = 0; i < t; ++i) {
            const int64_t s0 = O[i], L = O[i + 1] - s0 - l + 1;
            // the other t-1 sites' model
            wave_sync();
            if (lane < l) atomicSub(&n[(int)prot_sym(W, s0 + cs[i] + lane) * l + lane], 1);
            wave_sync();
            for (int e = lane; e < AL; e += kWave) {
                const int c = e / l;
                Tw[e] = log(((double)n[e] + beta * bgs[c]) / tm1) - log(bgs[c]);
            }
            wave_sync();
            // lane chunks of consecutive starts
            const int64_t C = (L + kWave - 1) / kWave;
            const int64_t a0 = min(L, (int64_t)lane * C), a1 = min(L, a0 + C);
            double mx = -INFINITY;
            for (int64_t a = a0; a < a1; ++a) mx = fmax(mx, start_score(W, s0, a, Tw, l));
            mx = wave_max(mx);
            double part = 0;
            for (int64_t a = a0; a < a1; ++a) part += exp(start_score(W, s0, a, Tw, l) - mx);
            // running sums over the lanes in start order
            double incl = part;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const double v = __shfl_up(incl, o);
                if (lane >= o) incl += v;
            }
            const double tot = __shfl(incl, kWave - 1);
            const double target = gibbs_uniform(g.seed, r, i, b) * tot;
            const uint64_t over = __ballot(incl > target);
            int64_t pick = L - 1;
            if (over) {
                const int who = __builtin_ctzll(over);
                int64_t found = L - 1;
                if (lane == who) {
                    double run = incl - part;
                    for (int64_t a = a0; a < a1; ++a) {
                        run += exp(start_score(W, s0, a, Tw, l) - mx);
                        if (run > target) {
                            found = a;
                            break;
                        }
                    }
                }
                pick = __shfl(found, who);
            }
            if (lane == 0) cs[i] = (int32_t)pick;
            wave_sync();
            if (lane < l) atomicAdd(&n[(int)prot_sym(W, s0 + pick + lane) * l + lane], 1);
            wave_sync();
        }
        const double Fr = alignment_F(n, bgs, A, l, t, beta);
        if (g.F && lane == 0) g.F[b * it1 + r + 1] = Fr;
        if (Fr > Fb) {
            Fb = Fr;
            for (int i = lane; i < t; i += kWave) bs[i] = cs[i];
        }
        wave_sync();
    }
    // the best alignment's model and sites
    for (int e = lane; e < AL; e += kWave) n[e] = 0;
    wave_sync();
    for (int i = 0; i < t; ++i)
        if (lane < l) atomicAdd(&n[(int)prot_sym(W, O[i] + bs[i] + lane) * l + lane], 1);
    wave_sync();
    for (int e = lane; e < AL; e += kWave)
        g.theta_out[b * AL + e] = ((double)n[e] + beta * bgs[e / l]) / ((double)t + beta);
    if (g.sites)
        for (int i = lane; i < t; i += kWave) g.sites[b * t + i] = bs[i];
}

constexpr int kGibbsHeld = 16;            // starts a lane holds in registers
constexpr double kGibbsLogRange = 600.0;  // largest |ln| of a start's weight taken as a product

// a window of 32 symbols and the 16 that follow, shifted along symbol by symbol
struct Slide {
    Win w;
    uint32_t next;
};

__device__ __forceinline__ Slide slide_at(const uint32_t *W, int64_t P)
{
    const int64_t wi = P >> 4;
    const uint32_t r = (uint32_t)(P & 15) << 1;
    const uint32_t w0 = W[wi], w1 = W[wi + 1], w2 = W[wi + 2], w3 = W[wi + 3];
    Slide s;
    s.w.hi = (uint32_t)((((uint64_t)w0 << 32) | w1) >> (32 - r));
    s.w.lo = (uint32_t)((((uint64_t)w1 << 32) | w2) >> (32 - r));
    s.next = (uint32_t)((((uint64_t)w2 << 32) | w3) >> (32 - r));
    return s;
}

__device__ __forceinline__ void slide(Slide &s)
{
    s.w.hi = (s.w.hi << 2) | (s.w.lo >> 30);
    s.w.lo = (s.w.lo << 2) | (s.next >> 30);
    s.next <<= 2;
}

// product (or sum) of the window's ceil(l/3) table entries
template <int NG, bool PROD, int Q = 0>
__device__ __forceinline__ double weight3(const Win &w, const double *T3)
{
    const double v = T3[64 * Q + three_letters<Q>(w)];
    if constexpr (Q + 1 < NG) {
        const double r = weight3<NG, PROD, Q + 1>(w, T3);
        return PROD ? v * r : v + r;
    } else {
        return v;
    }
}

// the tables of three letters from the columns Tw (4 x l), by one wave
template <int NG, bool PROD>
__device__ __forceinline__ void tables3(const double *Tw, int l, double *T3)
{
    const int e = lane_id();
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int p = 3 * q;
        double v = Tw[(e >> 4) * l + p];
        if (p + 1 < l) v = PROD ? v * Tw[((e >> 2) & 3) * l + p + 1] : v + Tw[((e >> 2) & 3) * l + p + 1];
        if (p + 2 < l) v = PROD ? v * Tw[(e & 3) * l + p + 2] : v + Tw[(e & 3) * l + p + 2];
        T3[64 * q + e] = v;
    }
}

// One draw: the start, 0 <= start < L, that the uniform u picks among the L
// starts of the sequence at symbol s0 by their weights.
template <int NG, bool PROD>
__device__ int64_t draw_start(const uint32_t *W, int64_t s0, int L, const double *T3, double u)
{
    const int lane = lane_id();
    // lane chunks of consecutive starts; a lane past the end reads the last one
    const int C = (L + kWave - 1) / kWave;
    const int a0 = min(L, lane * C), a1 = min(L, a0 + C);
    const bool held = C <= kGibbsHeld;
    double e[kGibbsHeld], mx = -INFINITY, part = 0;
    if (held) {
        Slide s = slide_at(W, s0 + min(a0, L - 1));
#pragma unroll
        for (int c = 0; c < kGibbsHeld; ++c) {
            e[c] = PROD ? 0.0 : -INFINITY;
            if (c < C) {
                const double v = weight3<NG, PROD>(s.w, T3);
                if (a0 + c < a1) e[c] = v;
                slide(s);
            }
        }
    }
    auto weight = [&](int a) {
        const double v = weight3<NG, PROD>(load_win(W, s0 + a), T3);
        return PROD ? v : exp(v - mx);
    };
    if (!PROD) {
        if (held) {
#pragma unroll
            for (int c = 0; c < kGibbsHeld; ++c) mx = fmax(mx, e[c]);
        } else {
            for (int a = a0; a < a1; ++a) mx = fmax(mx, weight3<NG, PROD>(load_win(W, s0 + a), T3));
        }
        mx = wave_max(mx);
        if (held)
#pragma unroll
            for (int c = 0; c < kGibbsHeld; ++c) e[c] = exp(e[c] - mx);
    }
    if (held) {
#pragma unroll
        for (int c = 0; c < kGibbsHeld; ++c) part += e[c];
    } else {
        for (int a = a0; a < a1; ++a) part += weight(a);
    }
    // running sums over the lanes in start order
    const double incl = wave_incl_sum(part);
    const double target = u * __shfl(incl, kWave - 1);
    const uint64_t over = __ballot(incl > target);
    if (!over) return L - 1;
    const int who = __builtin_ctzll(over);
    double run = incl - part;
    int found = -1;
    if (held) {
#pragma unroll
        for (int c = 0; c < kGibbsHeld; ++c) {
            run += e[c];
            if (found < 0 && a0 + c < a1 && run > target) found = a0 + c;
        }
    } else if (lane == who) {
        for (int a = a0; a < a1 && found < 0; ++a) {
            run += weight(a);
            if (run > target) found = a;
        }
    }
    if (found < 0) found = L - 1;
    return __shfl(found, who);
}

template <int NG>
__global__ void __launch_bounds__(kGibbsThreads, 4) k_gibbs_dna(const GibbsArgs g)
{
    extern __shared__ __align__(16) uint32_t dyn[];
    __shared__ double Tws[kGibbsWaves][4 * 32];   // ln theta0/bg, then the ratios (or their logarithms)
    __shared__ double T3s[kGibbsWaves][64 * NG];
    __shared__ int32_t cnt[kGibbsWaves][4 * 32];
    __shared__ double bgs[4];

    const pm_inst &I = g.one;
    const int tid = threadIdx.x, wv = tid / kWave, lane = lane_id();
    const int l = g.l, AL = 4 * l, t = I.t;
    const double beta = g.beta, tm1 = (double)(t - 1) + beta;
    uint32_t *seq = dyn;
    int64_t *offs = reinterpret_cast<int64_t *>(dyn + ((g.seq_cap + 1) & ~1));
    double *R = reinterpret_cast<double *>(offs + g.off_cap);  // [4][t + 1]: ratio of n sites with the letter
    int32_t *cs = reinterpret_cast<int32_t *>(R + 4 * (t + 1)) + 2 * wv * t, *bs = cs + t;
    const int seq_words = g.seq_cap ? (int)((I.n_total + 15) / 16 + 4) : 0;
    for (int i = tid; i < seq_words; i += kGibbsThreads) seq[i] = I.packed[i];
    if (g.off_cap)
        for (int i = tid; i <= t; i += kGibbsThreads) offs[i] = I.offsets[i];
    if (tid < 4) bgs[tid] = g.bg[tid];
    __syncthreads();
    // every ratio lies between beta / tm1 (no site) and 1 / bg
    double low = 1.0;
    for (int c = 0; c < 4; ++c) low = fmin(low, bgs[c]);
    const bool prod = l * fmax(fabs(log(beta / tm1)), fabs(log(low))) < kGibbsLogRange;
    for (int i = tid; i < 4 * (t + 1); i += kGibbsThreads) {
        const int c = i / (t + 1), n = i % (t + 1);
        const double th = ((double)n + beta * bgs[c]) / tm1;
        R[i] = prod ? th / bgs[c] : log(th) - log(bgs[c]);
    }
    __syncthreads();
    const uint32_t *W = g.seq_cap ? seq : I.packed;
    const int64_t *O = g.off_cap ? offs : I.offsets;

    int64_t nvalid = g.n_dev ? *g.n_dev : g.B;
    if (nvalid > g.B) nvalid = g.B;
    const int64_t b = (int64_t)blockIdx.x * kGibbsWaves + wv;
    if (b >= nvalid) return;  // whole waves leave; no workgroup barrier follows

    double *Tw = Tws[wv], *T3 = T3s[wv];
    int32_t *n = cnt[wv];

    // start: the best start of every sequence under theta0 (first on ties).
    // Starts whose three-letter sum is within rounding of the largest are
    // decided by their sum over the positions in order.
    for (int e = lane; e < AL; e += kWave) Tw[e] = log(g.theta0[b * AL + e]) - log(bgs[e / l]);
    wave_sync();
    tables3<NG, false>(Tw, l, T3);
    wave_sync();
    double tol = 0;
    if (lane < l)
        for (int c = 0; c < 4; ++c) tol = fmax(tol, fabs(Tw[c * l + lane]));
    tol = wave_sum(tol) * 64 * 2.220446049250313e-16;
    for (int i = 0; i < t; ++i) {
        const int64_t s0 = O[i];
        const int L = (int)(O[i + 1] - s0) - l + 1;
        double mx = -INFINITY;
        for (int a = lane; a < L; a += kWave) mx = fmax(mx, weight3<NG, false>(load_win(W, s0 + a), T3));
        mx = wave_max(mx);
        double bv = -INFINITY;
        int64_t ba = lane < L ? lane : INT64_MAX;  // (no finite score: the first start)
        for (int a = lane; a < L; a += kWave) {
            const Win w = load_win(W, s0 + a);
            if (weight3<NG, false>(w, T3) >= mx - tol) {
                double v = 0;
                for (int p = 0; p < l; ++p) v += Tw[dna_at(w.hi, w.lo, p) * l + p];
                if (v > bv) {
                    bv = v;
                    ba = a;
                }
            }
        }
        wave_argmax(bv, ba);
        if (lane == 0) cs[i] = (int32_t)ba;
    }
    for (int e = lane; e < AL; e += kWave) n[e] = 0;
    wave_sync();
    for (int i = 0; i < t; ++i)
        if (lane < l) atomicAdd(&n[dna_sym(W, O[i] + cs[i] + lane) * l + lane], 1);
    wave_sync();
    for (int e = lane; e < AL; e += kWave) Tw[e] = R[e / l * (t + 1) + n[e]];
    double Fb = alignment_F(n, bgs, 4, l, t, beta);
    const int it1 = g.sweeps + 1;
    if (g.F && lane == 0) g.F[b * it1] = Fb;
    for (int i = lane; i < t; i += kWave) bs[i] = cs[i];

    // one site's letters taken out of (d = -1) or put into (d = 1) the counts,
    // with their ratios
    auto site = [&](int64_t P, int d) {
        wave_sync();
        if (lane < l) {
            const int c = (int)dna_sym(W, P + lane), e = c * l + lane, k = n[e] + d;
            n[e] = k;
            Tw[e] = R[c * (t + 1) + k];
        }
        wave_sync();
    };
    for (int r = 0; r < g.sweeps; ++r) {
        double us = 0;
        for (int i = 0; i < t; ++i) {
            if (i % kWave == 0) us = gibbs_uniform(g.seed, r, i + lane, b);
            const double u = __shfl(us, i % kWave);
            const int64_t s0 = O[i];
            const int L = (int)(O[i + 1] - s0) - l + 1;
            site(s0 + cs[i], -1);  // the other t-1 sites' model
            int64_t pick;
            if (prod) {
                tables3<NG, true>(Tw, l, T3);
                wave_sync();
                pick = draw_start<NG, true>(W, s0, L, T3, u);
            } else {
                tables3<NG, false>(Tw, l, T3);
                wave_sync();
                pick = draw_start<NG, false>(W, s0, L, T3, u);
            }
            if (lane == 0) cs[i] = (int32_t)pick;
            site(s0 + pick, 1);
        }
        const double Fr = alignment_F(n, bgs, 4, l, t, beta);
        if (g.F && lane == 0) g.F[b * it1 + r + 1] = Fr;
        if (Fr > Fb) {
            Fb = Fr;
            for (int i = lane; i < t; i += kWave) bs[i] = cs[i];
        }
        wave_sync();
    }
    // the best alignment's model and sites
    for (int e = lane; e < AL; e += kWave) n[e] = 0;
    wave_sync();
    for (int i = 0; i < t; ++i)
        if (lane < l) atomicAdd(&n[dna_sym(W, O[i] + bs[i] + lane) * l + lane], 1);
    wave_sync();
    for (int e = lane; e < AL; e += kWave)
        g.theta_out[b * AL + e] = ((double)n[e] + beta * bgs[e / l]) / ((double)t + beta);
    if (g.sites)
        for (int i = lane; i < t; i += kWave) g.sites[b * t + i] = bs[i];
}

template <int NG>
static void launch_dna_groups(const GibbsArgs &g, dim3 grid, size_t lds, hipStream_t st)
{
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute((const void *)k_gibbs_dna<NG>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_gibbs_dna<NG>, grid, dim3(kGibbsThreads), lds, st, g);
}

static void launch_gibbs_dna(const GibbsArgs &g, dim3 grid, size_t lds, hipStream_t st)
{
    switch ((g.l + 2) / 3) {
    case 1: launch_dna_groups<1>(g, grid, lds, st); break;
    case 2: launch_dna_groups<2>(g, grid, lds, st); break;
    case 3: launch_dna_groups<3>(g, grid, lds, st); break;
    case 4: launch_dna_groups<4>(g, grid, lds, st); break;
    case 5: launch_dna_groups<5>(g, grid, lds, st); break;
    case 6: launch_dna_groups<6>(g, grid, lds, st); break;
    case 7: launch_dna_groups<7>(g, grid, lds, st); break;
    case 8: launch_dna_groups<8>(g, grid, lds, st); break;
    case 9: launch_dna_groups<9>(g, grid, lds, st); break;
    case 10: launch_dna_groups<10>(g, grid, lds, st); break;
    default: launch_dna_groups<11>(g, grid, lds, st); break;
    }
}

}  // namespace pm

using namespace pm;

extern "C" int gibbs_refine(const pm_seqs *S, int32_t l, const double *theta0, const double *bg, int64_t B,
                            const int64_t *n_dev, int32_t sweeps, double beta, uint64_t seed, double *theta_out,
                            double *F_out, int32_t *sites_out, void *stream)
{
    clear_error();
    int rc = check_seqs(S, l);
    if (rc) return rc;
    if (B < 0 || sweeps < 0) return fail(PM_EINVAL, "need B >= 0 and sweeps >= 0");
    if (!(beta > 0)) return fail(PM_EINVAL, "Gibbs sampling needs beta > 0 (a start's weight would be 0)");
    if (S->t > kGibbsMaxT) return fail(PM_ERANGE, "t = %d above the sampler's %d sequences", S->t, kGibbsMaxT);
    if (B > ((int64_t)1 << 36)) return fail(PM_ERANGE, "B too large");
    if (B > 0 && (!theta0 || !bg || !theta_out)) return fail(PM_EINVAL, "NULL buffer");
    if (B == 0) return PM_OK;
    GibbsArgs g{};
    g.one = inst_of(S, l);
    g.theta0 = theta0;
    g.bg = bg;
    g.n_dev = n_dev;
    g.theta_out = theta_out;
    g.F = F_out;
    g.sites = sites_out;
    g.B = B;
    g.l = l;
    g.sweeps = sweeps;
    g.beta = beta;
    g.seed = seed;
    const int64_t nw = pm_packed_words(S->alphabet, S->n_total);
    g.seq_cap = nw * 4 <= 48 * 1024 ? (int)nw : 0;
    g.off_cap = (S->t + 1) * 8 <= 8 * 1024 ? S->t + 1 : 0;
    const size_t lds = ((g.seq_cap + 1) & ~1) * 4 + (size_t)g.off_cap * 8;
    const int64_t blocks = (B + kGibbsWaves - 1) / kGibbsWaves;
    const dim3 grid((unsigned)blocks);
    if (S->alphabet == 4)
        launch_gibbs_dna(g, grid, lds + (size_t)4 * (S->t + 1) * 8 + (size_t)2 * kGibbsWaves * S->t * 4,
                         as_stream(stream));
    else
        hipLaunchKernelGGL(k_gibbs, grid, dim3(kGibbsThreads), lds, as_stream(stream), g);
    PM_LAUNCHED();
    return PM_OK;
}
