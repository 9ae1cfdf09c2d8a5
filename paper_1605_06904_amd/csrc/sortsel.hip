// a3 + a4 + a5 without a count table: enriched buckets of key spaces too
// large for LDS histograms (DNA k up to 16, protein k up to 7).
//
// Alg. 2 step 3 defines a bucket by the l-mers that share a projected k-mer
// and keeps it when it holds at least s of them (Sec. 6).  The |Sigma|^k
// table of PROJECTION1 (Sec. 5.2) stops fitting on-chip long before keys stop
// fitting 32 bits; the paper's own answer to that space problem is its K2
// kernel (Sec. 6: every l-mer compared with every other, O(x^2) work).  Here
// a trial's buckets come from sorting instead: one workgroup owns one
// (trial, key-range slice), counts the slice's keys in a coarse LDS histogram
// of 4096 key ranges, takes the leading ranges whose windows fit an LDS
// buffer of 8192 (key, window) pairs, gathers those pairs, sorts them with a
// bitonic network, and reads buckets off the runs of equal keys, in key order
// with members in window order -- the same lists as the count-table path.
// A range with more windows than the buffer holds is narrowed (finer coarse
// bins) until it is a single key, which then forms its bucket directly.
// With s >= 2 most windows of such key spaces are alone with their key and
// leave before the sort: a filter finds the keys that may occur twice, a trial
// is one slice, and the sort is of what passes it, commonly some dozens of
// pairs.  1000 trials of the (18,6) workload, k = 14, s = 2: 2740 us without it,
// 362 with one look, 238 with a second one over what passed; bound by the keys,
// formed once per pass, and the LDS atomics of the first look.  Kernels of their
// own for the two forms: without the filter's code the other one takes 3 to 10%
// less.
// Nothing but the bucket records and members reaches HBM; like the fused
// count-table path, one pass counts (per-slice totals, scanned on the device)
// and a second identical pass writes.
#include <algorithm>

#include "hash_dev.h"

namespace pm {

constexpr int kSortCap = 8192;     // (key, window) pairs sorted at once
constexpr int kFiltCap = 4096;     // the same behind the filter
constexpr int kFiltLog = 18;       // log2 bits of the filter's first bitmap (it lies in the buffer)
static_assert(kFiltCap * 64 == 1 << kFiltLog, "the bitmap lies in the sort buffer");
constexpr int kFiltWindows = 24;   // filtered windows per thread whose keys stay in registers
// The filter needs keys that are rarely met twice: at least this many keys per
// window, from where on what passes still fits the buffer.  Random DNA, k = 8,
// s = 2, unfiltered against filtered: 300 trials of 20 000 windows (3.3 keys per
// window) 970 and 576 us, 150 of 30 000 (2.2) 750 and 734, of 40 000 (1.6) 1213
// and 1280, of 80 000 (0.8) 3040 and 4100.  A trial is not one slice where
// there are fewer trials than CUs: 12 trials of 80 000 windows, k = 9, 788 us in
// four slices, 271 in 20.
constexpr int64_t kFiltSparse = 2;
constexpr int64_t kSortCUs = 256;
constexpr int kCoarseLog = 12;
constexpr int kCoarseBins = 1 << kCoarseLog;  // key ranges of the coarse histogram
constexpr int kCtlWords = 64;      // block-scan partials and round state
constexpr int kSortWaves = kHashThreads / kWave;

struct HsortArgs {
    HashArgs h;
    uint32_t s;
    uint64_t slice_width;           // keys per slice (the last one may be shorter)
    int64_t *tot_b, *tot_m;         // [items * nslices]
    const int64_t *base_b, *base_m; // [items * nslices] (EMIT)
    pm_bucket *buckets;
    uint32_t *members;
    int64_t cap_b, cap_m;
};

// Exclusive prefix of (a, b) over the workgroup's threads, in thread order;
// tot_* receive the workgroup totals.  ctl holds 2 * kSortWaves words.
__device__ __forceinline__ void block_excl_scan2(uint32_t &a, uint32_t &b, uint32_t *ctl, uint32_t &tot_a,
                                                 uint32_t &tot_b)
{
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const uint32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
    if (lane == kWave - 1) {
        ctl[2 * wave] = ia;
        ctl[2 * wave + 1] = ib;
    }
    __syncthreads();
    uint32_t pa = 0, pb = 0, sa = 0, sb = 0;
    for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t va = ctl[2 * w], vb = ctl[2 * w + 1];
        if (w < wave) {
            pa += va;
            pb += vb;
        }
        sa += va;
        sb += vb;
    }
    a = pa + ia - a;
    b = pb + ib - b;
    tot_a = sa;
    tot_b = sb;
    __syncthreads();
}

// (the second look's bitmap of kCoarseBins words has two bits for one of the second bitmap)
static_assert(kCoarseLog + 5 - 1 == kFiltLog - 2, "the second look shares the second bitmap");
// the filter's second bitmap: 2^kFiltFold bits of the first share one of it
constexpr int kFiltFold = 2;
__host__ __device__ constexpr int filt_words2(int log2_bits) { return 1 << (log2_bits - kFiltFold - 5); }

// smallest shift whose 2^sh-wide bins cover `range` keys in kCoarseBins bins
__device__ __forceinline__ int coarse_shift(uint64_t range)
{
    int sh = 0;
    while (((range + (1ull << sh) - 1) >> sh) > (uint64_t)kCoarseBins) ++sh;
    return sh;
}

template <int A, int K, bool EMIT, bool FILT>
__global__ void __launch_bounds__(kHashThreads) k_hsort(const HsortArgs g)
{
    const HashArgs &a = g.h;
    extern __shared__ __align__(16) uint32_t smem[];
    const int slice = blockIdx.x % a.nslices;
    const int j = blockIdx.x / a.nslices;
    const int tid = threadIdx.x;
    const int64_t e = (int64_t)blockIdx.x;  // (item, slice) entry

    if (EMIT && g.tot_b[e] == 0) return;  // counted: nothing to write
    const uint32_t mask = a.masks[j];
    if (!mask_ok(a, mask)) {
        if (tid == 0) {
            if (slice == 0 && a.status) atomicOr(a.status, PM_STATUS_BAD_MASK);
            if (!EMIT) g.tot_b[e] = g.tot_m[e] = 0;
        }
        return;
    }
    constexpr uint32_t cap = FILT ? kFiltCap : kSortCap;
    uint64_t *buf = reinterpret_cast<uint64_t *>(smem);  // [cap]
    uint32_t *hist = smem + 2 * cap;                      // [kCoarseBins]
    uint32_t *ctl = hist + kCoarseBins;                   // [kCtlWords]
    uint32_t *twice = ctl + kCtlWords;                    // filter's second bitmap
    uint32_t *seq = twice + (FILT ? filt_words2(kFiltLog) : 0);
    int32_t *wst = reinterpret_cast<int32_t *>(seq + a.seq_cap);
    const Staged st = stage_input<A>(a, j, seq, wst);
    int pos[K];
    kept_positions<A, K>(mask, pos);
    const int64_t x = st.I.x;
    const uint64_t s_lo = (uint64_t)slice * g.slice_width;
    const uint64_t s_hi = min((uint64_t)a.nb, s_lo + g.slice_width);
    const int sh0 = coarse_shift(s_hi > s_lo ? s_hi - s_lo : 1);
    const int64_t bb = EMIT ? g.base_b[e] : 0, mb = EMIT ? g.base_m[e] : 0;
    int64_t rb = 0, rm = 0;  // buckets and members of this entry so far
    uint64_t lo = s_lo;
    int sh = sh0;
    __syncthreads();

    // A bucket's key occurs at least twice where s >= 2: a bitmap of hashed keys
    // whose bit is found set marks the key's bit in a second one, and only
    // windows with that bit are looked at further (keys met once pass by
    // coincidence, in about one window of ten).  Commonly they all fit the sort
    // buffer, and the slice is done after one look at its windows and one at
    // the keys kept from it.
    auto hashed = [&](uint64_t key) { return ((uint32_t)key * 0x9E3779B1u) >> (32 - kFiltLog); };
    auto marked = [&](uint64_t key) {
        if (!FILT) return true;
        const uint32_t h = hashed(key) >> kFiltFold;
        return ((twice[h >> 5] >> (h & 31u)) & 1u) != 0;
    };
    bool whole = false;  // the slice's pairs are in buf
    uint32_t n_whole = 0;
    if constexpr (FILT) {
        uint32_t *once = smem;  // the sort buffer's words
        for (int b = tid; b < (1 << kFiltLog) / 32; b += kHashThreads) once[b] = 0;
        for (int b = tid; b < filt_words2(kFiltLog); b += kHashThreads) twice[b] = 0;
        if (tid == 0) ctl[2 * kSortWaves + 2] = 0;
        __syncthreads();
        const bool all_keys = s_lo == 0 && s_hi >= (uint64_t)a.nb;
        auto mark = [&](uint64_t key) {
            if (!all_keys && (key < s_lo || key >= s_hi)) return;
            const uint32_t h = hashed(key);
            if ((atomicOr(once + (h >> 5), 1u << (h & 31u)) >> (h & 31u)) & 1u)
                atomicOr(twice + (h >> (kFiltFold + 5)), 1u << ((h >> kFiltFold) & 31u));
        };
        auto gather = [&](uint64_t key, int64_t w, bool in) {
            const bool hit = in && (all_keys || (key >= s_lo && key < s_hi)) && marked(key);
            const uint64_t m = __ballot(hit);
            if (!m) return;
            const int first = __ffsll((unsigned long long)m) - 1;
            uint32_t slot = 0;
            if (lane_id() == first) slot = atomicAdd(ctl + 2 * kSortWaves + 2, (uint32_t)__popcll(m));
            slot = (uint32_t)__builtin_amdgcn_readlane((int)slot, first) +
                   (uint32_t)__popcll(m & ((1ull << lane_id()) - 1));
            if (hit && slot < cap) buf[slot] = (key << 32) | (uint64_t)w;
        };
        uint32_t held[kFiltWindows];
        int i = 0;
#pragma unroll
        for (int q = 0; q < kFiltWindows; ++q) {
            const int64_t w = (int64_t)q * kHashThreads + tid;
            held[q] = 0;
            if (w < x) {
                held[q] = (uint32_t)window_key<A, K>(a, st, pos, w, i);
                mark(held[q]);
            }
        }
        const int i_held = i;
        for (int64_t w = (int64_t)kFiltWindows * kHashThreads + tid; w < x; w += kHashThreads)
            mark(window_key<A, K>(a, st, pos, w, i));
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kFiltWindows; ++q) {
            const int64_t w = (int64_t)q * kHashThreads + tid;
            gather(held[q], w, w < x);
        }
        i = i_held;
        for (int64_t w0 = (int64_t)kFiltWindows * kHashThreads; w0 < x; w0 += kHashThreads) {
            const int64_t w = w0 + tid;
            gather(w < x ? window_key<A, K>(a, st, pos, w, i) : 0u, w, w < x);
        }
        __syncthreads();
        n_whole = ctl[2 * kSortWaves + 2];
        whole = n_whole <= cap;
        __syncthreads();
        if (whole && n_whole > kWave) {
            // again over the pairs, by another hash into the coarse histogram's
            // words: of the keys met once one in fifty is left, and the sort is
            // of some dozens of pairs instead of a thousand or two
            constexpr int kPer = kFiltCap / kHashThreads;
            uint64_t mine[kPer];
            auto hashed2 = [](uint64_t pair) { return ((uint32_t)(pair >> 32) * 0xB5297A4Du) >> (32 - kCoarseLog - 5); };
            for (int b = tid; b < kCoarseBins; b += kHashThreads) hist[b] = 0;
            for (int b = tid; b < filt_words2(kFiltLog); b += kHashThreads) twice[b] = 0;
            if (tid == 0) ctl[2 * kSortWaves + 2] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const uint32_t p = tid + q * kHashThreads;
                mine[q] = p < n_whole ? buf[p] : 0;
                if (p < n_whole) {
                    const uint32_t h = hashed2(mine[q]);
                    if ((atomicOr(hist + (h >> 5), 1u << (h & 31u)) >> (h & 31u)) & 1u)
                        atomicOr(twice + (h >> 6), 1u << ((h >> 1) & 31u));
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const uint32_t h = hashed2(mine[q]) >> 1;
                if (tid + q * kHashThreads < n_whole && ((twice[h >> 5] >> (h & 31u)) & 1u))
                    buf[atomicAdd(ctl + 2 * kSortWaves + 2, 1u)] = mine[q];
            }
            __syncthreads();
            n_whole = ctl[2 * kSortWaves + 2];
            __syncthreads();
        }
    }

    while (lo < s_hi) {
        uint64_t hi = s_hi;
        uint32_t n = n_whole;
        if (!whole) {
        const uint64_t r_hi = min(s_hi, lo + ((uint64_t)kCoarseBins << sh));
        const uint32_t nbins = (uint32_t)((r_hi - lo + (1ull << sh) - 1) >> sh);
        // 1. coarse histogram of the keys in [lo, r_hi)
        for (int b = tid; b < kCoarseBins; b += kHashThreads) hist[b] = 0;
        if (tid == 0) ctl[2 * kSortWaves] = 0xffffffffu;
        __syncthreads();
        {
            int i = 0;
            for (int64_t w = tid; w < x; w += kHashThreads) {
                const uint64_t key = window_key<A, K>(a, st, pos, w, i);
                if (key >= lo && key < r_hi && marked(key)) atomicAdd(hist + (uint32_t)((key - lo) >> sh), 1u);
            }
        }
        __syncthreads();
        // 2. the leading bins whose windows fit the sort buffer
        constexpr int kPer = kCoarseBins / kHashThreads;
        uint32_t c[kPer], sum = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            c[q] = hist[tid * kPer + q];
            sum += c[q];
        }
        uint32_t excl = sum, dummy = 0, total = 0, dtot = 0;
        block_excl_scan2(excl, dummy, ctl, total, dtot);
        {
            uint32_t run = excl;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                run += c[q];
                if (run > cap) {
                    atomicMin(ctl + 2 * kSortWaves, (uint32_t)(tid * kPer + q));
                    break;
                }
            }
        }
        __syncthreads();
        const uint32_t first_over = ctl[2 * kSortWaves];
        const uint32_t take = min(first_over, nbins);
        // windows in the taken bins: the prefix up to bin `take`
        if (tid == 0) ctl[2 * kSortWaves + 1] = 0;
        __syncthreads();
        {
            uint32_t run = excl;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const uint32_t b = tid * kPer + q;
                if (b < take) run += c[q];
            }
            if (tid * kPer < take && (tid + 1) * kPer >= take) ctl[2 * kSortWaves + 1] = run;
        }
        __syncthreads();
        n = take > 0 ? ctl[2 * kSortWaves + 1] : 0;
        const uint32_t c_first = hist[0];
        __syncthreads();

        if (take == 0) {
            if (sh > 0) {  // the first bin alone is too large: look at it in finer bins
                sh = sh > 12 ? sh - 12 : 0;
                continue;
            }
            // a single key with more windows than the buffer: its own bucket,
            // members in window order by an ordered compaction
            if (c_first >= g.s) {
                if (EMIT) {
                    const int64_t idx = bb + rb;
                    if (tid == 0 && idx < g.cap_b)
                        g.buckets[idx] = pm_bucket{(uint32_t)j, (uint32_t)lo, c_first, (uint32_t)(mb + rm)};
                    int i = 0;
                    uint32_t placed = 0;
                    for (int64_t w0 = 0; w0 < x; w0 += kHashThreads) {
                        const int64_t w = w0 + tid;
                        const bool hit = w < x && window_key<A, K>(a, st, pos, w, i) == lo;
                        uint32_t f = hit ? 1u : 0u, d0 = 0, tot = 0, d1 = 0;
                        block_excl_scan2(f, d0, ctl, tot, d1);
                        const int64_t ms = mb + rm + placed + f;
                        if (hit && ms < g.cap_m) g.members[ms] = (uint32_t)w;
                        placed += tot;
                    }
                }
                rb += 1;
                rm += c_first;
            }
            lo += 1;
            sh = sh0;
            continue;
        }
        hi = min(r_hi, lo + ((uint64_t)take << sh));
        if (n > 0) {
            // 3. gather the (key, window) pairs of [lo, hi)
            if (tid == 0) ctl[2 * kSortWaves + 2] = 0;
            __syncthreads();
            {
                int i = 0;
                for (int64_t w = tid; w < x; w += kHashThreads) {
                    const uint64_t key = window_key<A, K>(a, st, pos, w, i);
                    if (key >= lo && key < hi && marked(key)) {
                        const uint32_t slot = atomicAdd(ctl + 2 * kSortWaves + 2, 1u);
                        buf[slot] = (key << 32) | (uint64_t)w;
                    }
                }
            }
        }
        }
        if (n > 0) {
            // sort the pairs
            uint32_t P = 64;
            while (P < n) P <<= 1;
            for (uint32_t q = n + tid; q < P; q += kHashThreads) buf[q] = ~0ull;
            __syncthreads();
            for (uint32_t kk = 2; kk <= P; kk <<= 1) {
                for (uint32_t jj = kk >> 1; jj > 0; jj >>= 1) {
                    for (uint32_t q = tid; q < P / 2; q += kHashThreads) {
                        const uint32_t i0 = ((q & ~(jj - 1)) << 1) | (q & (jj - 1));
                        const uint32_t i1 = i0 | jj;
                        const uint64_t u = buf[i0], v = buf[i1];
                        const bool up = (i0 & kk) == 0;
                        if ((u > v) == up) {
                            buf[i0] = v;
                            buf[i1] = u;
                        }
                    }
                    __syncthreads();
                }
            }
            // 4. runs of equal keys, in order; each thread starts the runs that
            // begin in its chunk
            const uint32_t chunk = (n + kHashThreads - 1) / kHashThreads;
            const uint32_t c0 = min(n, tid * chunk), c1 = min(n, c0 + chunk);
            uint32_t nbk = 0, nmem = 0;
            for (uint32_t q = c0; q < c1; ++q) {
                const uint32_t key = (uint32_t)(buf[q] >> 32);
                if (q > 0 && (uint32_t)(buf[q - 1] >> 32) == key) continue;
                uint32_t len = 1;
                while (q + len < n && (uint32_t)(buf[q + len] >> 32) == key) ++len;
                if (len >= g.s) {
                    nbk += 1;
                    nmem += len;
                }
            }
            uint32_t bi = nbk, mi = nmem, tb = 0, tm = 0;
            block_excl_scan2(bi, mi, ctl, tb, tm);
            if (EMIT) {
                for (uint32_t q = c0; q < c1; ++q) {
                    const uint32_t key = (uint32_t)(buf[q] >> 32);
                    if (q > 0 && (uint32_t)(buf[q - 1] >> 32) == key) continue;
                    uint32_t len = 1;
                    while (q + len < n && (uint32_t)(buf[q + len] >> 32) == key) ++len;
                    if (len < g.s) continue;
                    const int64_t idx = bb + rb + bi;
                    const int64_t first = mb + rm + mi;
                    if (idx < g.cap_b) g.buckets[idx] = pm_bucket{(uint32_t)j, key, len, (uint32_t)first};
                    for (uint32_t r = 0; r < len; ++r)
                        if (first + r < g.cap_m) g.members[first + r] = (uint32_t)buf[q + r];
                    bi += 1;
                    mi += len;
                }
            }
            rb += tb;
            rm += tm;
            __syncthreads();
        }
        lo = hi;
        sh = sh0;
    }
    if (!EMIT && tid == 0) {
        g.tot_b[e] = rb;
        g.tot_m[e] = rm;
    }
}

template <int A, int K, bool EMIT, bool FILT>
static int launch_hsort(const HsortArgs &g, size_t lds, int blocks, hipStream_t st)
{
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_hsort<A, K, EMIT, FILT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  device_lds_bytes());
        (void)hipGetLastError();
        attr_set = true;
    }
    hipLaunchKernelGGL((k_hsort<A, K, EMIT, FILT>), dim3(blocks), dim3(kHashThreads), lds, st, g);
    PM_LAUNCHED();
    return PM_OK;
}

// run-time (alphabet, k) -> compile-time kernel: DNA k 8..16, protein k 4..7
template <bool FILT, int K>
static int dispatch_hsort(int alphabet, int k, bool emit, const HsortArgs &g, size_t lds, int blocks, hipStream_t st)
{
    if constexpr (K > 16) {
        return fail(PM_ERANGE, "k=%d not supported by the sorted selection", k);
    } else {
        if (k != K) return dispatch_hsort<FILT, K + 1>(alphabet, k, emit, g, lds, blocks, st);
        if (alphabet == 4) {
            if constexpr (K >= kSortKMinDna)
                return emit ? launch_hsort<4, K, true, FILT>(g, lds, blocks, st)
                            : launch_hsort<4, K, false, FILT>(g, lds, blocks, st);
            return fail(PM_ERANGE, "k=%d below the sorted selection's range for DNA", k);
        }
        if constexpr (K >= kSortKMinProt && K <= 7)
            return emit ? launch_hsort<20, K, true, FILT>(g, lds, blocks, st)
                        : launch_hsort<20, K, false, FILT>(g, lds, blocks, st);
        return fail(PM_ERANGE, "k=%d outside the sorted selection's range for protein", k);
    }
}

// LDS bytes and slices for the largest instance; 0 after fail()
static size_t hsort_layout(HashArgs &a, int64_t x_max, int64_t nw_max, int t_max)
{
    const int lds_max = device_lds_bytes();
    const int64_t sw = staged_words(a.A, nw_max);
    a.off_cap = (t_max + 1) * 4 <= 8 * 1024 ? t_max + 1 : 0;
    a.seq_cap = sw * 4 <= 48 * 1024 && (a.A == 4 || a.off_cap) ? (int)sw : 0;
    a.hist_words = 0;
    a.slice_bins = 0;
    // slices of the key range sized for about half a sort buffer of windows
    // each when keys spread evenly
    int64_t ns = (2 * x_max + kSortCap - 1) / kSortCap;
    if (ns < 1) ns = 1;
    if (ns > a.nb) ns = a.nb;
    a.nslices = (int)ns;
    const size_t bytes = (size_t)(2 * kSortCap + kCoarseBins + kCtlWords + a.seq_cap + a.off_cap) * 4;
    if ((int64_t)bytes > lds_max) {
        fail(PM_ERANGE, "input too large for the sorted selection's LDS budget");
        return 0;
    }
    return bytes;
}

static size_t hsort_ws_bytes(int64_t entries) { return entries < 0 ? 0 : (size_t)entries * 4 * sizeof(int64_t) + 256; }

static int64_t hsort_entries(HashArgs a, int32_t items, int64_t x_max, int64_t nw_max, int t_max)
{
    if (!hsort_layout(a, x_max, nw_max, t_max)) return -1;
    return (int64_t)items * a.nslices;
}

int hsort_check_k(int A, int k)
{
    if (A == 4 && (k < kSortKMinDna || k > 16))
        return fail(PM_ERANGE, "the sorted selection takes DNA k from %d to 16 (k=%d)", kSortKMinDna, k);
    if (A == 20 && (k < kSortKMinProt || k > 7))
        return fail(PM_ERANGE, "the sorted selection takes protein k from %d to 7 (k=%d)", kSortKMinProt, k);
    return PM_OK;
}

size_t hsort_workspace(int A, int l, int k, int32_t items, int64_t x_max, int64_t nw_max, int t_max)
{
    HashArgs a{};
    a.A = A;
    a.nb = ipow(A, k);
    a.l = l;
    a.k = k;
    return hsort_ws_bytes(hsort_entries(a, items, x_max, nw_max, t_max));
}

int hsort_run(HashArgs &a, int A, int32_t items, int64_t x_max, int64_t nw_max, int t_max, uint32_t s,
              pm_bucket *buckets, int64_t cap_b, uint32_t *members, int64_t cap_m, int64_t *n_out, void *ws,
              size_t ws_bytes, hipStream_t st)
{
    if (int rc = hsort_check_k(A, a.k)) return rc;
    size_t lds = hsort_layout(a, x_max, nw_max, t_max);
    if (!lds) return PM_ERANGE;
    if (x_max >= (int64_t)1 << 31) return fail(PM_ERANGE, "more than 2^31 windows in one instance");
    int64_t entries = (int64_t)items * a.nslices;
    if (entries > 0x7fffffff) return fail(PM_ERANGE, "too many trials x slices");
    if (ws_bytes < hsort_ws_bytes(entries))
        return fail(PM_EINVAL, "workspace of %zu bytes, need %zu", ws_bytes, hsort_ws_bytes(entries));
    if (((uintptr_t)ws & 7) != 0) return fail(PM_EINVAL, "workspace must be 8-byte aligned");
    HsortArgs g{};
    const bool filtered = s >= 2 && kFiltSparse * x_max <= a.nb;
    if (filtered) {
        // as many windows per slice as a bitmap of the (halved)
        // buffer's bits takes at one key in ten bits, but as many slices as
        // there are CUs for; never more slices
        lds -= (size_t)(2 * (kSortCap - kFiltCap) - filt_words2(kFiltLog)) * 4;
        const int64_t per = (int64_t)kFiltWindows * kHashThreads;
        a.nslices = (int)std::max<int64_t>(
            1, std::min<int64_t>(a.nslices, std::max<int64_t>((x_max + per - 1) / per, kSortCUs / std::max(items, 1))));
        entries = (int64_t)items * a.nslices;
    }
    int64_t *w = static_cast<int64_t *>(ws);
    g.h = a;
    g.s = s;
    g.slice_width = ((uint64_t)a.nb + a.nslices - 1) / a.nslices;
    g.tot_b = w;
    g.tot_m = w + entries;
    g.base_b = w + 2 * entries;
    g.base_m = w + 3 * entries;
    g.buckets = buckets;
    g.members = members;
    g.cap_b = cap_b;
    g.cap_m = cap_m;
    const auto launch = [&](bool emit) {
        return filtered ? dispatch_hsort<true, 1>(A, a.k, emit, g, lds, (int)entries, st)
                        : dispatch_hsort<false, 1>(A, a.k, emit, g, lds, (int)entries, st);
    };
    if (int rc = launch(false)) return rc;
    const TotScan ts{g.tot_b, g.tot_m, w + 2 * entries, w + 3 * entries, entries, cap_b, cap_m, n_out, a.status};
    if (int rc = launch_tot_scan(ts, st)) return rc;
    if (cap_b == 0 && cap_m == 0) return PM_OK;  // sizing only
    return launch(true);
}

}  // namespace pm
