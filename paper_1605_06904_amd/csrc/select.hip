// a5 (enriched-bucket selection and member lists) and a6 (profiles, theta^0).
//
// The paper finds enriched buckets by comparing every k-mer with every other
// one (Sec. 6, quadratic work) to avoid a |Sigma|^k table.  On MI355X the dense
// counts already sit in HBM (the histogram of projection_hash), so selection
// reads them once: a counting pass per trial writes the number of passing
// bins, their total size and a bitmap of the passing keys (one bit per key);
// projection_hash_select has its hash kernel write these instead.  After a
// scan of the per-trial totals, one workgroup per trial loads its bitmap into
// LDS, gathers the counts of the passing keys only, scans them into bucket
// numbers and first member slots, and places the member windows in window
// order.  A trial of few members lists its passing windows per wave quarter
// in LDS and places them from the lists (should a quarter overflow its list,
// or where the key space is small, by a stable counting sort over chunks of
// windows: per-wave counts by LDS atomics, then each wave groups its passing
// windows by key, every bucket keeping its next free slot per wave in LDS).  A
// trial of many members or buckets collects its members in any order in LDS
// and ranks them within their buckets.
#include <algorithm>

#include "pm_common.h"

namespace pm {

struct SelWs {
    int64_t *ne;      // [m] enriched buckets per trial
    int64_t *ms;      // [m] members per trial
    int64_t *bb;      // [m] first bucket of the trial
    int64_t *mb;      // [m] first member slot of the trial
    int64_t *n_heavy; // [1] trials with more buckets than the first emit launch takes
    int64_t *qctr;    // [4] next units of the heavy launches (their work queues' heads, [0] and [1]), and
                      // whether the second has anything to do ([2])
    int32_t *heavy;   // [m] those trials, in order; kHasBig set: buckets are left to the second launch
    int64_t *nep;     // [m][parts] buckets of each part of a trial's bins (parts > 1)
    int64_t *msp;     // [m][parts] their members
    uint64_t *bits;   // [m][nwb] passing keys: bit key % 64 of word key / 64
};

// parts of a trial's bins counted by separate workgroups: enough workgroups
// (about 16 384) that the launch does not end on a partly filled wave of
// them, each part at least 32 bitmap words
static int sel_parts(int32_t m, int64_t nwb)
{
    int64_t p = (16384 + (int64_t)m - 1) / std::max<int64_t>(m, 1);
    p = std::min<int64_t>(p, std::max<int64_t>(1, nwb / 32));
    return (int)std::max<int64_t>(1, std::min<int64_t>(p, 64));
}

static size_t sel_head_bytes(int32_t m, int64_t nwb)
{
    return (size_t)m * 4 * sizeof(int64_t) + 5 * sizeof(int64_t) + (((size_t)m * 4 + 7) & ~(size_t)7) +
           (size_t)m * sel_parts(m, nwb) * 2 * sizeof(int64_t);
}

static size_t sel_ws_bytes(int32_t m, int64_t nwb)
{
    return sel_head_bytes(m, nwb) + (size_t)m * nwb * 8 + 256;
}

static SelWs carve(void *ws, int32_t m, int64_t nwb)
{
    char *p = static_cast<char *>(ws);
    SelWs w;
    w.ne = reinterpret_cast<int64_t *>(p);
    w.ms = w.ne + m;
    w.bb = w.ms + m;
    w.mb = w.bb + m;
    w.n_heavy = w.mb + m;
    w.qctr = w.n_heavy + 1;
    w.heavy = reinterpret_cast<int32_t *>(w.qctr + 4);
    w.nep = reinterpret_cast<int64_t *>(p + (size_t)m * 4 * sizeof(int64_t) + 5 * sizeof(int64_t) +
                                        (((size_t)m * 4 + 7) & ~(size_t)7));
    w.msp = w.nep + (int64_t)m * sel_parts(m, nwb);
    w.bits = reinterpret_cast<uint64_t *>(p + sel_head_bytes(m, nwb));
    return w;
}

struct SelArgs {
    pm_inst one;               // the instance, when inst is NULL
    const pm_inst *inst;       // batch: instance table, or NULL
    const int32_t *item_inst;  // batch: instance of every trial item
    const uint32_t *keys;
    const uint32_t *counts;
    pm_bucket *buckets;
    uint32_t *members;
    int64_t *n_out;
    uint32_t *status;
    SelWs ws;
    int64_t nb, cap_b, cap_m;
    int64_t light;             // k_sel_emit: members of a trial it takes at most
    int32_t m;                 // trials (items)
    uint32_t s;
    int nwb;    // bitmap words, ceil(nb / 64)
    int cb;     // buckets whose cursors the LDS holds
    int parts;  // k_sel_count: workgroups per trial
    int room;   // k_sel_emit_heavy, k_sel_emit_cursors: bytes of LDS for rows and list or cursors
    int cursors;  // k_sel_emit_cursors follows k_sel_emit_heavy
};

// per (trial, part of its bins): number of passing bins, their total size
// and the bitmap words of the passing keys.  Lane i of a wave reads bins 4i ..
// 4i+3 of 256 as one 16-byte load, and the four ballots (one per bin of the
// load) become four words in lane-major order: bit 16q + i of word g is bin
// 64g + 4i + q.  The emit pass puts the words in key order.
__global__ void __launch_bounds__(256) k_sel_count(const SelArgs a)
{
    const int j = blockIdx.x / a.parts, part = blockIdx.x % a.parts;
    const int wv = threadIdx.x >> 6, lane = lane_id();
    const uint4 *cnt = reinterpret_cast<const uint4 *>(a.counts + (int64_t)j * a.nb);  // nb % 4 == 0
    uint64_t *bits = a.ws.bits + (int64_t)j * a.nwb;
    const uint32_t smin = a.s > 1u ? a.s : 1u;  // a bin passes with at least max(s, 1) l-mers
    constexpr int U = 4;                        // 256-bin groups per wave at a time
    const int64_t n4 = a.nb / 4;
    const int64_t per = ((a.nwb + a.parts - 1) / a.parts + 4 * U - 1) / (4 * U) * (4 * U);  // words per part
    const int64_t w_lo = part * per, w_hi = std::min<int64_t>(a.nwb, w_lo + per);
    uint32_t ne = 0, ms = 0;  // ne counts whole ballots (the same in every lane); a trial has fewer than 2^32 windows
    for (int64_t g0 = w_lo / 4 + (int64_t)wv * U; 4 * g0 < w_hi; g0 += 4 * U) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = (g0 + u) * 64 + lane;  // 16-byte load index
            v[u] = 4 * (g0 + u) < w_hi && i < n4 ? cnt[i] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            uint64_t bal[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool p = c[q] >= smin;
                bal[q] = __ballot(p);
                ne += (uint32_t)__popcll(bal[q]);
                ms += p ? c[q] : 0u;
            }
            const int64_t wi = 4 * (g0 + u) + lane;
            if (lane < 4 && wi < w_hi) {
                const int sh = 16 * lane;
                bits[wi] = ((bal[0] >> sh) & 0xffffull) | (((bal[1] >> sh) & 0xffffull) << 16) |
                           (((bal[2] >> sh) & 0xffffull) << 32) | (((bal[3] >> sh) & 0xffffull) << 48);
            }
        }
    }
    const uint32_t mst = wave_sum(ms);
    __shared__ uint64_t red[2][4];
    if (lane == 0) {
        red[0][wv] = ne;
        red[1][wv] = mst;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t tb = (int64_t)(red[0][0] + red[0][1] + red[0][2] + red[0][3]);
        const int64_t tm = (int64_t)(red[1][0] + red[1][1] + red[1][2] + red[1][3]);
        if (a.parts > 1) {
            a.ws.nep[(int64_t)j * a.parts + part] = tb;
            a.ws.msp[(int64_t)j * a.parts + part] = tm;
        } else {
            a.ws.ne[j] = tb;
            a.ws.ms[j] = tm;
        }
    }
}

// bit i of a 16-bit value moved to bit 4i
__device__ __forceinline__ uint64_t spread4(uint64_t x)
{
    uint64_t v = x & 0xffffull;
    v = (v | (v << 24)) & 0x000000ff000000ffull;
    v = (v | (v << 12)) & 0x000f000f000f000full;
    v = (v | (v << 6)) & 0x0303030303030303ull;
    v = (v | (v << 3)) & 0x1111111111111111ull;
    return v;
}

// a bitmap word from lane-major order (bit 16q + i: key 4i + q) to key order
__device__ __forceinline__ uint64_t word_in_key_order(uint64_t b)
{
    return spread4(b) | (spread4(b >> 16) << 1) | (spread4(b >> 32) << 2) | (spread4(b >> 48) << 3);
}

// whether a trial of few buckets has so many members that they are listed and
// ranked; ranking takes a bucket's members times themselves, so not where
// buckets are large (protein k = 2, 85 members a bucket: 420 us placed by
// chunks, 1900 ranked)
__device__ __forceinline__ bool heavy_members(int64_t buckets, int64_t members, int64_t light)
{
    return members > light && members <= 32 * buckets;
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// exclusive scan of per-trial (or per trial-slice) totals, one workgroup:
// bases of every entry, the required totals in n_out, capacity status, and
// on request the list of heavy entries
__global__ void __launch_bounds__(1024) k_tot_scan(const TotScan a)
{
    // four entries per thread and step; one barrier per step (the waves' sums
    // alternate between two buffers), every thread keeping the totals so far.
    // One workgroup, so bound by latency: 6000 entries took 47 us in steps of
    // 1024 entries scanned through LDS, 11 this way
    constexpr int P = 4;
    __shared__ double sums[2][2][16];  // (whole numbers below 2^53)
    __shared__ uint32_t sums_h[2][16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
    int64_t done[3] = {0, 0, 0};  // buckets, members, heavy entries before this step
    int buf = 0;
    for (int64_t base = 0; base < a.n; base += 1024 * P, buf ^= 1) {
        const int64_t j0 = base + (int64_t)threadIdx.x * P;
        int64_t ve[P], vm[P], s[3] = {0, 0, 0};
        uint32_t h = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int64_t j = j0 + i;
            ve[i] = vm[i] = 0;
            if (j < a.n) {
                if (a.parts > 1) {
                    for (int q = 0; q < a.parts; ++q) {
                        ve[i] += a.ne[j * a.parts + q];
                        vm[i] += a.ms[j * a.parts + q];
                    }
                    a.ne_sum[j] = ve[i];
                    a.ms_sum[j] = vm[i];
                } else {
                    ve[i] = a.ne[j];
                    vm[i] = a.ms[j];
                }
                if (a.heavy && (ve[i] > a.heavy_above || heavy_members(ve[i], vm[i], a.heavy_members))) h |= 1u << i;
            }
            s[0] += ve[i];
            s[1] += vm[i];
        }
        s[2] = __popc(h);
        double v[2];
        const uint32_t vh = wave_incl_scan((uint32_t)s[2]);
#pragma unroll
        for (int q = 0; q < 2; ++q) v[q] = wave_incl_sum((double)s[q]);
        if (lane == 63) {
            sums[buf][0][wave] = v[0];
            sums[buf][1][wave] = v[1];
            sums_h[buf][wave] = vh;
        }
        __syncthreads();
        int64_t before[3];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double w = wave_incl_sum(lane < 16 ? sums[buf][q][lane] : 0.0);
            before[q] = done[q] + (int64_t)(v[q] + (wave > 0 ? read_lane(w, wave - 1) : 0.0)) - s[q];
            done[q] += (int64_t)read_lane(w, 15);
        }
        const uint32_t wh = wave_incl_scan(lane < 16 ? sums_h[buf][lane] : 0u);
        before[2] = done[2] + vh + (wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)wh, wave - 1) : 0u) - s[2];
        done[2] += (uint32_t)__builtin_amdgcn_readlane((int)wh, 15);
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int64_t j = j0 + i;
            if (j >= a.n) break;
            a.bb[j] = before[0];
            a.mb[j] = before[1];
            before[0] += ve[i];
            before[1] += vm[i];
            if ((h >> i) & 1u) a.heavy[before[2]++] = (int32_t)j;
        }
    }
    if (threadIdx.x == 0) {
        a.n_out[0] = done[0];
        a.n_out[1] = done[1];
        if ((done[0] > a.cap_b || done[1] > a.cap_m) && a.status) atomicOr(a.status, PM_STATUS_CAPACITY);
        if (a.heavy) a.n_heavy[0] = done[2];
    }
}

int launch_tot_scan(const TotScan &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_tot_scan, dim3(1), dim3(1024), 0, st, a);
    PM_LAUNCHED();
    return PM_OK;
}

// exclusive prefix sums of n pairs of u32 values in place (256 threads)
__device__ __forceinline__ void block_excl_scan_pair(uint32_t *v0, uint32_t *v1, int n, uint32_t *tmp)
{
    const int tid = threadIdx.x, wv = tid >> 6, per = (n + 255) / 256;
    const int lo = min(n, tid * per), hi = min(n, lo + per);
    uint32_t s0 = 0, s1 = 0;
    for (int i = lo; i < hi; ++i) {
        s0 += v0[i];
        s1 += v1[i];
    }
    const uint32_t i0 = wave_incl_scan(s0), i1 = wave_incl_scan(s1);
    if (lane_id() == 63) {
        tmp[wv] = i0;
        tmp[4 + wv] = i1;
    }
    __syncthreads();
    uint32_t r0 = i0 - s0, r1 = i1 - s1;
    for (int w = 0; w < wv; ++w) {
        r0 += tmp[w];
        r1 += tmp[4 + w];
    }
    for (int i = lo; i < hi; ++i) {
        const uint32_t x0 = v0[i], x1 = v1[i];
        v0[i] = r0;
        v1[i] = r1;
        r0 += x0;
        r1 += x1;
    }
    __syncthreads();
}

// ---------------------------------------------------------------- members
constexpr int kSelU = 8;                   // window loads in flight per lane
constexpr int kSelChunk = 4 * 64 * kSelU;  // windows per workgroup step
constexpr int kSelBitsMin = 6;             // flagged lanes from which a wave groups by key bits
constexpr uint32_t kNoSlot = 0xffffffffu;
constexpr int kSelListCap = 256;           // passing windows each wave may list in a trial of few members

struct Group {
    int head;       // lowest lane holding the same key
    uint32_t rank;  // lanes below this one holding the same key
    uint32_t n;     // lanes holding the key (set at the head)
};

// Groups the flagged lanes of a wave by key (keys below 2^nbits).  With few
// flagged lanes, one ballot per distinct key; with many, each lane's peers
// (the flagged lanes holding its key) as the AND, over the nbits bits of the
// key, of the lanes that agree with it on that bit: VALU and scalar work only,
// where a sort across the wave was a chain of dependent cross-lane moves.
// Both give the same answer.
__device__ __forceinline__ Group group_by_key(bool flag, uint32_t key, int nbits)
{
    const int lane = lane_id();
    const uint64_t bal = __ballot(flag);
    Group g{lane, 0u, 0u};
    if (__popcll(bal) < kSelBitsMin) {
        uint64_t left = bal;
        while (left) {
            const int leader = __ffsll((unsigned long long)left) - 1;
            const uint32_t lk = __shfl(key, leader);
            const uint64_t peers = __ballot(flag && key == lk);
            if ((peers >> lane) & 1ull) {
                g.head = leader;
                g.rank = (uint32_t)__popcll(peers & lanemask_lt());
                g.n = (uint32_t)__popcll(peers);
            }
            left &= ~peers;
        }
        return g;
    }
    uint64_t peers = bal;
    for (int b = 0; b < nbits; ++b) {
        const bool bit = (key >> b) & 1u;
        const uint64_t on = __ballot(bit);
        peers &= bit ? on : ~on;
    }
    if (flag) {
        g.head = __ffsll((unsigned long long)peers) - 1;
        g.rank = (uint32_t)__popcll(peers & lanemask_lt());
        g.n = (uint32_t)__popcll(peers);
    }
    return g;
}

// bucket number of a passing key within its trial
__device__ __forceinline__ uint32_t local_bucket(const uint64_t *bm, const uint32_t *wcnt, uint32_t key)
{
    const uint32_t wd = key >> 6;
    return wcnt[wd] + (uint32_t)__popcll(bm[wd] & ((1ull << (key & 63u)) - 1ull));
}

// Bucket records and member lists of trial j, which has ne in 1 .. cb passing
// keys, by one workgroup of four waves.  Member cursors: rows[q][bucket] in
// LDS.
__device__ void emit_trial(const SelArgs &a, int j, int64_t ne, uint64_t *bm, uint32_t *tmp)
{
    uint32_t *wcnt = reinterpret_cast<uint32_t *>(bm + a.nwb);  // [nwb] -> buckets before the word
    uint32_t *wsz = wcnt + a.nwb;                               // [nwb] -> members before the word
    uint32_t *rows = wsz + a.nwb;                               // [4][cb]
    const int tid = threadIdx.x, wv = tid >> 6, lane = lane_id();
    const int cb = a.cb;
    const uint32_t *cnt = a.counts + (int64_t)j * a.nb;
    const uint64_t *bits = a.ws.bits + (int64_t)j * a.nwb;
    const int64_t bbase = a.ws.bb[j], mbase = a.ws.mb[j];
    const pm_inst I = a.inst ? a.inst[a.item_inst[j]] : a.one;

    // ---- the bitmap, and per word the total size of its passing buckets: a
    // wave takes four groups of 64 words at once (one load each) and gathers
    // the counts of eight non-empty words at a time
    for (int base = wv * 64; base < a.nwb; base += 4 * 256) {
        uint64_t b[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int wi = base + 256 * it + lane;
            b[it] = wi < a.nwb ? bits[wi] : 0ull;
        }
#pragma unroll
        for (int it = 0; it < 4; ++it)
            if (__ballot(b[it] != 0ull)) b[it] = word_in_key_order(b[it]);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int w0 = base + 256 * it, wi = w0 + lane;
            uint32_t sz = 0;
            uint64_t nz = __ballot(b[it] != 0ull);
            while (nz) {
                constexpr int G = 8;
                int idx[G];
                uint32_t c[G];
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    idx[u] = nz ? __ffsll((unsigned long long)nz) - 1 : -1;
                    nz &= nz - 1ull;
                }
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    c[u] = 0u;
                    if (idx[u] >= 0) {
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b[it], idx[u]);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b[it] >> 32), idx[u]);
                        if (((((uint64_t)hi << 32) | lo) >> lane) & 1ull)
                            c[u] = cnt[(int64_t)(w0 + idx[u]) * 64 + lane];
                    }
                }
#pragma unroll
                for (int u = 0; u < G; ++u)
                    if (idx[u] >= 0) {
                        const uint32_t t = wave_sum(c[u]);
                        if (lane == idx[u]) sz = t;
                    }
            }
            if (wi < a.nwb) {
                bm[wi] = b[it];
                wcnt[wi] = (uint32_t)__popcll(b[it]);
                wsz[wi] = sz;
            }
        }
    }
    __syncthreads();
    block_excl_scan_pair(wcnt, wsz, a.nwb, tmp);

    // ---- bucket records in key order (a word's buckets are its set lanes),
    // and every bucket's cursor row: its first slot, then zeros; the counts of
    // eight non-empty words are read at a time
    for (int w0 = wv * 64; w0 < a.nwb; w0 += 256) {
        const int wi = w0 + lane;
        uint64_t nz = __ballot(wi < a.nwb && bm[wi] != 0ull);
        while (nz) {
            constexpr int G = 8;
            int wd[G];
            uint32_t c[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                wd[u] = nz ? w0 + __ffsll((unsigned long long)nz) - 1 : -1;
                nz &= nz - 1ull;
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                c[u] = 0u;
                if (wd[u] >= 0 && ((bm[wd[u]] >> lane) & 1ull)) c[u] = cnt[(uint32_t)wd[u] * 64u + (uint32_t)lane];
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                if (wd[u] < 0) continue;
                const int w = wd[u];
                const uint64_t wb = bm[w];
                const bool set = (wb >> lane) & 1ull;
                const uint32_t key = (uint32_t)w * 64u + (uint32_t)lane;
                const uint32_t frel = wsz[w] + wave_incl_scan(c[u]) - c[u];  // first slot within the trial
                const uint32_t bi = wcnt[w] + (uint32_t)__popcll(wb & lanemask_lt());
                const int64_t b = bbase + bi;
                if (set) {
                    if (b < a.cap_b) a.buckets[b] = pm_bucket{(uint32_t)j, key, c[u], (uint32_t)(mbase + frel)};
                    rows[bi] = frel;
                    rows[cb + bi] = rows[2 * cb + bi] = rows[3 * cb + bi] = 0u;
                }
            }
        }
    }
    __syncthreads();

    const uint32_t *kj = a.keys + I.key_base + (int64_t)(j - I.first_item) * I.x;
    const int64_t x = I.x;
    const int64_t nb = a.nb;
    // the bitmap as 32-bit words (little-endian halves of the 64-bit ones)
    const uint32_t *bm32 = reinterpret_cast<const uint32_t *>(bm);
    const uint32_t nb32 = (uint32_t)nb;
    const int nbits = 32 - __builtin_clz(nb32 - 1u);  // key bits (|Sigma|^k >= 4)
    auto passing = [&](uint32_t key) { return key < nb32 && ((bm32[key >> 5] >> (key & 31u)) & 1u); };

    if (a.ws.ms[j] <= 4 * kSelListCap) {
        // few members: each wave lists the passing windows of its quarter of
        // the trial in order (no barrier), then one wave places the four lists,
        // which together are in window order, with the buckets' cursors (row 0)
        uint32_t *lw = rows + cb;                // [4][cap] windows
        uint32_t *lk = lw + 4 * kSelListCap;     // [4][cap] their keys
        const int64_t lo = x * wv / 4, hi = x * (wv + 1) / 4;
        uint32_t n = 0;
        uint32_t nk[kSelU];
#pragma unroll
        for (int u = 0; u < kSelU; ++u) {
            const int64_t w = lo + 64 * u + lane;
            nk[u] = w < hi ? kj[w] : 0u;
        }
        for (int64_t wb = lo; wb < hi; wb += 64 * kSelU) {
            uint32_t kk[kSelU];
#pragma unroll
            for (int u = 0; u < kSelU; ++u) kk[u] = nk[u];
            if (wb + 64 * kSelU < hi) {
#pragma unroll
                for (int u = 0; u < kSelU; ++u) {
                    const int64_t w = wb + 64 * kSelU + 64 * u + lane;
                    nk[u] = w < hi ? kj[w] : 0u;
                }
            }
#pragma unroll
            for (int u = 0; u < kSelU; ++u) {
                const int64_t w = wb + 64 * u + lane;
                const bool f = w < hi && passing(kk[u]);
                const uint64_t bal = __ballot(f);
                if (bal == 0ull) continue;
                const uint32_t pos = n + (uint32_t)__popcll(bal & lanemask_lt());
                if (f && pos < (uint32_t)kSelListCap) {
                    lw[wv * kSelListCap + pos] = (uint32_t)w;
                    lk[wv * kSelListCap + pos] = kk[u];
                }
                n += (uint32_t)__popcll(bal);
            }
        }
        if (lane == 0) tmp[wv] = n;
        __syncthreads();
        const uint32_t n0 = tmp[0], n1 = tmp[1], n2 = tmp[2], n3 = tmp[3];
        const uint32_t cap = (uint32_t)kSelListCap;
        if (n0 <= cap && n1 <= cap && n2 <= cap && n3 <= cap) {
            if (wv == 0) {
                const uint32_t e1 = n0, e2 = e1 + n1, e3 = e2 + n2, total = e3 + n3;
                for (uint32_t e0 = 0; e0 < total; e0 += 64) {
                    const uint32_t e = e0 + (uint32_t)lane;
                    const bool valid = e < total;
                    const uint32_t q = (e >= e1) + (e >= e2) + (e >= e3);
                    const uint32_t at = q * cap + e - (q == 0 ? 0u : q == 1 ? e1 : q == 2 ? e2 : e3);
                    const uint32_t w = valid ? lw[at] : 0u, key = valid ? lk[at] : 0u;
                    const Group g = group_by_key(valid, key, nbits);
                    uint32_t old = kNoSlot;
                    if (valid && g.head == lane) {
                        const uint32_t bi = local_bucket(bm, wcnt, key);
                        if (bbase + bi < a.cap_b) {
                            old = rows[bi];
                            rows[bi] = old + g.n;
                        }
                    }
                    old = __shfl(old, g.head);
                    if (valid && old != kNoSlot) {
                        const int64_t slot = mbase + old + g.rank;
                        if (slot < a.cap_m) a.members[slot] = w;
                    }
                }
            }
            return;
        }
        // a quarter held more than its list: the chunked placement below, with
        // rows 1-3 (which the lists overwrote) cleared again
        for (int64_t bi = tid; bi < ne; bi += 256) rows[cb + bi] = rows[2 * cb + bi] = rows[3 * cb + bi] = 0u;
        __syncthreads();
    }
    {
        // chunks of 2048 windows, wave q owning the q-th quarter of each: rows
        // 1-3 count the members of waves 0-2 per bucket, a sweep turns rows
        // 0-3 into each wave's first slot, the waves place their members, and
        // wave 3's row, now the first free slot, becomes row 0 again
        // the next chunk's keys are loaded while this one is placed
        const bool sparse = a.ws.ms[j] < x / 256;
        uint32_t nk[kSelU];
#pragma unroll
        for (int u = 0; u < kSelU; ++u) {
            const int64_t w = (int64_t)wv * 64 * kSelU + 64 * u + lane;
            nk[u] = w < x ? kj[w] : 0u;
        }
        for (int64_t c0 = 0; c0 < x; c0 += kSelChunk) {
            const int64_t wb = c0 + (int64_t)wv * 64 * kSelU;
            uint32_t kk[kSelU];
#pragma unroll
            for (int u = 0; u < kSelU; ++u) kk[u] = nk[u];
            if (c0 + kSelChunk < x) {
#pragma unroll
                for (int u = 0; u < kSelU; ++u) {
                    const int64_t w = wb + kSelChunk + 64 * u + lane;
                    nk[u] = w < x ? kj[w] : 0u;
                }
            }
            uint32_t fl = 0;  // bit u: this lane's window of step u passes
            if (c0 + kSelChunk <= x) {
#pragma unroll
                for (int u = 0; u < kSelU; ++u) fl |= passing(kk[u]) ? 1u << u : 0u;
            } else {
                const int left = (int)(x - wb);  // windows of this wave in the last chunk
#pragma unroll
                for (int u = 0; u < kSelU; ++u) fl |= 64 * u + lane < left && passing(kk[u]) ? 1u << u : 0u;
            }
            // a chunk without members is passed over, where there can be some
            if (sparse && !__syncthreads_or(fl != 0u)) continue;
            if (wv < 3) {
                // counts only: one LDS atomic per member, no grouping
#pragma unroll
                for (int u = 0; u < kSelU; ++u)
                    if ((fl >> u) & 1u) atomicAdd(rows + (wv + 1) * cb + local_bucket(bm, wcnt, kk[u]), 1u);
            }
            __syncthreads();
            for (int64_t bi = tid; bi < ne; bi += 256) {
                const uint32_t r1 = rows[bi] + rows[cb + bi];
                const uint32_t r2 = r1 + rows[2 * cb + bi];
                rows[cb + bi] = r1;
                rows[2 * cb + bi] = r2;
                rows[3 * cb + bi] += r2;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kSelU; ++u) {
                const bool f = (fl >> u) & 1u;
                if (__ballot(f) == 0ull) continue;
                const Group g = group_by_key(f, kk[u], nbits);
                uint32_t old = kNoSlot;
                if (f && g.head == lane) {
                    const uint32_t bi = local_bucket(bm, wcnt, kk[u]);
                    if (bbase + bi < a.cap_b) {
                        uint32_t *r = rows + wv * cb + bi;
                        old = *r;
                        *r = old + g.n;
                    }
                }
                old = __shfl(old, g.head);
                if (f && old != kNoSlot) {
                    const int64_t slot = mbase + old + g.rank;
                    if (slot < a.cap_m) a.members[slot] = (uint32_t)(wb + 64 * u + lane);
                }
            }
            __syncthreads();
            for (int64_t bi = tid; bi < ne; bi += 256) {
                rows[bi] = rows[3 * cb + bi];
                rows[cb + bi] = rows[2 * cb + bi] = rows[3 * cb + bi] = 0u;
            }
            __syncthreads();
        }
        return;
    }
}

// one workgroup per trial of few members whose buckets fit the LDS rows
__global__ void __launch_bounds__(256) k_sel_emit(const SelArgs a)
{
    extern __shared__ __align__(16) uint64_t bm[];
    __shared__ uint32_t tmp[256];
    const int j = blockIdx.x;
    if (j == 0 && threadIdx.x < 3) a.ws.qctr[threadIdx.x] = 0;  // of the heavy launches after this one
    const int64_t ne = a.ws.ne[j];
    if (ne == 0 || ne > a.cb || heavy_members(ne, a.ws.ms[j], a.light)) return;
    emit_trial(a, j, ne, bm, tmp);
}

// Many buckets.  The placement above (stable, by grouping the lanes of a wave)
// is a serial chain per wave, and its four cursors of every bucket leave room
// for few waves on a CU.  Here sixteen waves take a trial and place members in
// any order: an LDS atomic on a bucket's one cursor gives a place in a list in
// LDS, and when the list stands, every member counts the smaller windows of
// its bucket's piece of it, which is its rank.  A bucket holds few members (s
// and somewhat more), so that is a handful of LDS reads, and slots are written
// side by side.  A bucket of more than kHeavyBig members is left out of the
// list: k_sel_emit_cursors places it, or in small instances a wave that goes
// through the windows for it.
//
// Keys, counts and first slots go by a thread per bucket, so that a trial
// waits for its counts once, not once for every few bitmap words.  A trial
// whose buckets or members exceed the LDS (split between rows and list by the
// trial's members per bucket) goes by ranges of them, every one reading the
// trial's keys again (from the caches).  LDS for two workgroups per CU where
// the bitmap leaves it.  Bound by latencies and LDS accesses.  Measured on 6000
// trials of uneven instances (k = 7, s = 3, 26000 windows each; most are
// members): 2320 us placed by groups, 730 so; on 2000 protein trials (k = 4, s = 3, 29430 windows, 160000 bins,
// 1500 buckets): 1190 and 214.
constexpr int kHeavyThreads = 1024;
constexpr int kHeavyStatic = 3072;       // at least the launch's static LDS
constexpr int kHeavyWaves = kHeavyThreads / 64;
constexpr int kHeavyU = 8;               // key loads in flight per lane
constexpr uint32_t kHeavyBig = 128;
constexpr int kHeavyBigs = 256;          // big buckets of a range: the list's places / kHeavyBig at most
constexpr uint32_t kNotListed = 0x80000000u;
constexpr int32_t kHasBig = INT32_MIN;
// k_sel_emit_cursors is launched for instances of more windows: below, no trial
// of more than kSelChunk / 2 buckets is dense, and big buckets are few
constexpr int64_t kCursorWindows = 32 * kSelChunk / 2;

// trials placed by k_sel_emit_cursors alone: ranking takes a bucket's members
// times themselves (see heavy_members)
__device__ __forceinline__ bool heavy_dense(int64_t buckets, int64_t members) { return members > 32 * buckets; }
constexpr uint16_t kNoBucket = 0xffffu;

// exclusive prefix sums of n values in place, v[n] receiving the total
// (1024 threads)
__device__ __forceinline__ void heavy_scan(uint32_t *v, int n, uint32_t *part)
{
    const int tid = threadIdx.x, wv = tid >> 6, per = (n + kHeavyThreads - 1) / kHeavyThreads;
    const int lo = min(n, tid * per), hi = min(n, lo + per);
    uint32_t s = 0;
    for (int i = lo; i < hi; ++i) s += v[i];
    const uint32_t incl = wave_incl_scan(s);
    if (lane_id() == 63) part[wv] = incl;
    __syncthreads();
    uint32_t run = incl - s + wave_sum(lane_id() < wv ? part[lane_id()] : 0u);
    for (int i = lo; i < hi; ++i) {
        const uint32_t x = v[i];
        v[i] = run;
        run += x;
    }
    if (tid == kHeavyThreads - 1) v[n] = run;
    __syncthreads();
}

// the last i in lo + 1 .. n with v[i] - v[lo] <= room, lo + 1 if there is none
// (v ascending; the whole wave calls)
__device__ __forceinline__ int heavy_reach(const uint32_t *v, int lo, int n, uint32_t room)
{
    const uint32_t base = v[lo];
    if (v[n] - base <= room) return n;
    int at = lo + 1;
    for (int span = n - at; span > 0;) {  // the answer lies in at .. at + span
        const int step = (span + 63) / 64, i = min(at + (lane_id() + 1) * step, n);
        const int fit = __popcll(__ballot(v[i] - base <= room));
        at = min(at + fit * step, n);
        span = step - 1;
    }
    return at;
}

// trial j (ne passing keys); of several workgroups that share it, number `part`
// of `parts` takes every parts-th range; *seen (LDS): non-zero if there were big
// buckets
__device__ __forceinline__ void emit_heavy(const SelArgs &a, int j, int64_t ne, int part, int parts, uint64_t *bm,
                                           uint32_t *seen)
{
    __shared__ uint32_t scan[kHeavyWaves];
    __shared__ uint32_t big_key[kHeavyBigs], big_first[kHeavyBigs], n_big;
    uint32_t *wcnt = reinterpret_cast<uint32_t *>(bm + a.nwb);  // [nwb + 1] -> buckets before the word
    uint32_t *lds = wcnt + a.nwb + 1;                           // [room / 4]
    // rows of 8 bytes and list places of 6, shared out by members per bucket
    const int64_t ms = a.ws.ms[j];
    const int rcap = (int)max((int64_t)64, min((int64_t)0xfff0, (int64_t)a.room * ne / (8 * ne + 6 * (ms + ms / 32))));
    const uint32_t lcap = (uint32_t)((a.room - 8 * rcap - 4) / 6) & ~1u;
    uint32_t *cur = lds;                                        // [rcap] key, then next list place
    uint32_t *first = cur + rcap;                               // [rcap + 1] first slot within the rows' buckets
    uint32_t *lw = first + rcap + 1;                            // [lcap] windows
    uint16_t *lb = reinterpret_cast<uint16_t *>(lw + lcap);     // [lcap] their buckets (rows)
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = lane_id();
    const uint32_t big = min(kHeavyBig, lcap);
    const uint32_t *cnt = a.counts + (int64_t)j * a.nb;
    const uint64_t *bits = a.ws.bits + (int64_t)j * a.nwb;
    const int64_t bbase = a.ws.bb[j], mbase = a.ws.mb[j];
    const pm_inst I = a.inst ? a.inst[a.item_inst[j]] : a.one;
    const uint32_t *kj = a.keys + I.key_base + (int64_t)(j - I.first_item) * I.x;
    const uint32_t x = (uint32_t)I.x;  // below 2^31

    for (int w = tid; w < a.nwb; w += kHeavyThreads) {
        const uint64_t b = word_in_key_order(bits[w]);
        bm[w] = b;
        wcnt[w] = (uint32_t)__popcll(b);
    }
    __syncthreads();
    heavy_scan(wcnt, a.nwb, scan);

    uint32_t m_rows = 0;  // members before the rows' buckets
    int r = 0;
    for (int w0 = 0, w1; w0 < a.nwb; w0 = w1) {
        // ---- the buckets of as many words as there are rows for
        w1 = heavy_reach(wcnt, w0, a.nwb, (uint32_t)rcap);
        const uint32_t b0 = wcnt[w0];
        const int n = (int)(wcnt[w1] - b0);  // at most rcap: a word has 64
        if (n == 0) continue;
        for (int u = tid; u < 4 * (w1 - w0); u += kHeavyThreads) {
            const int w = w0 + (u >> 2), sh = 16 * (u & 3);
            const uint64_t b = bm[w];
            uint32_t at = wcnt[w] - b0 + (uint32_t)__popcll(b & ((1ull << sh) - 1ull));
            for (uint32_t q = (uint32_t)(b >> sh) & 0xffffu; q; q &= q - 1u)
                cur[at++] = (uint32_t)w * 64u + (uint32_t)(sh + __ffs((int)q) - 1);
        }
        if (tid == 0) n_big = 0;
        __syncthreads();
        for (int i0 = tid; i0 < n; i0 += 4 * kHeavyThreads) {
            uint32_t c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = i0 + u * kHeavyThreads < n ? cnt[cur[i0 + u * kHeavyThreads]] : 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u * kHeavyThreads < n) first[i0 + u * kHeavyThreads] = c[u];
        }
        __syncthreads();
        heavy_scan(first, n, scan);
        if (part == 0)
            for (int i = tid; i < n; i += kHeavyThreads) {
                const int64_t b = bbase + b0 + i;
                const uint32_t f = first[i];
                if (b < a.cap_b)
                    a.buckets[b] = pm_bucket{(uint32_t)j, cur[i], first[i + 1] - f, (uint32_t)(mbase + m_rows + f)};
            }
        for (int i0 = 0, i1; i0 < n; i0 = i1, ++r) {
            // ---- a range of them whose members the list takes (or one bucket)
            i1 = heavy_reach(first, i0, n, lcap);
            if (r % parts != part) continue;
            const uint32_t f0 = first[i0], nm = min(first[i1] - f0, lcap);
            for (uint32_t p = tid; p < nm; p += kHeavyThreads) lb[p] = kNoBucket;
            for (int i = tid; i < i1; i += kHeavyThreads) {  // (the thread that read the key above)
                if (i < i0) continue;
                const uint32_t f = first[i], c = first[i + 1] - f;
                const bool kept = bbase + b0 + i < a.cap_b;
                if (kept && c > big) {
                    const uint32_t q = atomicAdd(&n_big, 1u);
                    if (q < (uint32_t)kHeavyBigs) {
                        big_key[q] = cur[i];
                        big_first[q] = f;
                    }
                }
                cur[i] = kept && c <= big ? f - f0 : kNotListed;
            }
            __syncthreads();
            // ---- the list: each member of the range's listed buckets
            uint32_t nk[kHeavyU];  // the next step's keys, loaded ahead
            auto load_keys = [&](uint32_t wb) {
#pragma unroll
                for (int u = 0; u < kHeavyU; ++u) {
                    const uint32_t w = wb + kHeavyThreads * u + tid;
                    nk[u] = w < x ? kj[w] : 0xffffffffu;
                }
            };
            load_keys(0);
            const uint32_t wn = (uint32_t)(w1 - w0), in = (uint32_t)(i1 - i0), lo = b0 + (uint32_t)i0;
            for (uint32_t wb = 0; wb < x; wb += kHeavyThreads * kHeavyU) {
                uint32_t kk[kHeavyU];
#pragma unroll
                for (int u = 0; u < kHeavyU; ++u) kk[u] = nk[u];
                load_keys(wb + kHeavyThreads * kHeavyU);
#pragma unroll
                for (int u = 0; u < kHeavyU; ++u) {
                    const uint32_t wd = kk[u] >> 6;  // 0xffffffff, where there is no window or key, is in no range
                    if (wd - (uint32_t)w0 >= wn) continue;
                    const uint64_t m = bm[wd];
                    if (!((m >> (kk[u] & 63u)) & 1ull)) continue;
                    const uint32_t i = wcnt[wd] + (uint32_t)__popcll(m & ((1ull << (kk[u] & 63u)) - 1ull)) - lo;
                    if (i >= in) continue;
                    const uint32_t p = atomicAdd(cur + i0 + i, 1u);
                    if (p < lcap) {
                        lw[p] = wb + kHeavyThreads * u + tid;
                        lb[p] = (uint16_t)(i0 + i);
                    }
                }
            }
            __syncthreads();
            // ---- ranks and slots
            for (uint32_t p = tid; p < nm; p += kHeavyThreads) {
                const uint32_t i = lb[p];
                if (i == kNoBucket) continue;
                // (to the last place taken: the caller's counts may exceed the keys')
                const uint32_t f = first[i], w = lw[p], q0 = f - f0, q1 = min(cur[i], lcap);
                uint32_t rank = 0;
                for (uint32_t q = q0; q < q1; q += 4) {
                    uint32_t v[4];
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) v[k] = lw[min(q + k, q1 - 1)];
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) rank += q + k < q1 && v[k] < w ? 1u : 0u;
                }
                const int64_t slot = mbase + m_rows + f + rank;
                if (slot < a.cap_m) a.members[slot] = w;
            }
            // ---- big buckets: a wave finds a key's windows in order
            const uint32_t nb = a.cursors ? 0u : min(n_big, (uint32_t)kHeavyBigs);
            for (uint32_t q = wv; q < nb; q += kHeavyWaves) {
                const uint32_t key = big_key[q];
                int64_t slot = mbase + m_rows + big_first[q];
                for (uint32_t wb = 0; wb < x; wb += 64 * kHeavyU) {
                    uint32_t kk[kHeavyU];
#pragma unroll
                    for (int u = 0; u < kHeavyU; ++u) {
                        const uint32_t w = wb + 64 * u + lane;
                        kk[u] = w < x ? kj[w] : 0xffffffffu;
                    }
#pragma unroll
                    for (int u = 0; u < kHeavyU; ++u) {
                        const uint64_t hit = __ballot(kk[u] == key);
                        const int64_t at = slot + __popcll(hit & lanemask_lt());
                        if (kk[u] == key && at < a.cap_m) a.members[at] = wb + 64 * u + lane;
                        slot += __popcll(hit);
                    }
                }
            }
            __syncthreads();
            if (tid == 0) {
                *seen |= n_big;
                n_big = 0;
            }
            __syncthreads();
        }
        m_rows += first[n];
        __syncthreads();
    }
}

// the trials with more buckets than the rows above or more members than the
// short lists (on an uneven batch such trials took 140 us placed by chunks, and
// cost nothing to be seen among the others here), listed by the scan: a
// fixed grid of workgroups takes them from a work queue (trials differ in size
// by an order of magnitude).  Where they are fewer than the workgroups the
// chip holds, up to eight share a trial's ranges.
__global__ void __launch_bounds__(kHeavyThreads, 8) k_sel_emit_heavy(const SelArgs a)
{
    extern __shared__ __align__(16) uint64_t bm[];
    __shared__ int64_t claim;
    __shared__ uint32_t seen;
    const int64_t nh = *a.ws.n_heavy;
    if (nh == 0) return;  // no queue traffic
    const int parts = (int)(nh >= gridDim.x ? 1 : min((int64_t)8, ((int64_t)gridDim.x + nh - 1) / nh));
    unsigned long long *q = reinterpret_cast<unsigned long long *>(a.ws.qctr);
    for (;;) {
        if (threadIdx.x == 0) claim = (int64_t)atomicAdd(q, 1ull);
        __syncthreads();
        const int64_t un = claim;
        __syncthreads();
        if (un >= nh * parts) break;  // every workgroup ends here once the queue is past its end
        const int j = a.ws.heavy[un % nh] & ~kHasBig, part = (int)(un / nh);
        const int64_t ne = a.ws.ne[j];
        const int64_t ms = a.ws.ms[j];
        if (threadIdx.x == 0) seen = a.cursors && heavy_dense(ne, ms);
        // a trial that fits the LDS is one range
        if (!(a.cursors && heavy_dense(ne, ms)) && (part == 0 || 8 * ne + 7 * ms + 1024 > a.room))  // uniform
            emit_heavy(a, j, ne, part, parts, bm, &seen);
        if (a.cursors && threadIdx.x == 0 && seen) {
            atomicOr(a.ws.heavy + claim % *a.ws.n_heavy, kHasBig);
            a.ws.qctr[2] = 1;
        }
    }
}

// Buckets of many members, by cursors: a stable placement in two passes over
// the windows, of which each of the sixteen waves takes a sixteenth (it counts
// the buckets' members; the counts of the waves give each its first slots; it
// places its members in order).  All buckets of a dense trial, with their
// records, and the big ones of the others.  A trial goes by ranges of as many
// buckets as the LDS has cursors for.  Bound by LDS accesses: a key's bucket is
// one read of a table where the range's keys are few enough (three dependent
// reads by the bitmap), and lanes that meet on a bucket show by the value that
// the cursor has after the step, so that only those are put in order by ballots.
// Whole selection of 256 DNA trials of 200 000 windows (k = 6, 49 members per
// bucket) 1410 us so, 1670 by ranks, 1180 by four waves' cursors; of 1024 such
// trials 4700, 5930 and 4560 (all members' slots lie apart: bound by their
// writes); of 64 trials of 520 000 (127 per bucket) 1050, 26 000 and 2110.  At
// 24 per bucket (1024 trials of 100 000) ranks take 2010, four waves' cursors
// 2710; the line between the two lies at 32 (heavy_dense).
constexpr int kCursorU = 8;  // windows per lane and step
constexpr int kMapKeys = 10240;

__device__ __forceinline__ int cursor_rows(int room) { return (room - 4 - 2 * kMapKeys) / (8 + 4 * kHeavyWaves); }

__device__ __forceinline__ void emit_cursors(const SelArgs &a, int j, int64_t ne, bool dense, int part, int parts,
                                             uint64_t *bm)
{
    __shared__ uint32_t scan[kHeavyWaves];
    __shared__ uint32_t n_big;
    uint32_t *wcnt = reinterpret_cast<uint32_t *>(bm + a.nwb);  // [nwb + 1] -> buckets before the word
    uint32_t *num = wcnt + a.nwb + 1;                           // [rcap] key, then number of the row's bucket
    const int rcap = cursor_rows(a.room);
    uint32_t *first = num + rcap;                               // [rcap + 1] first slot within the rows' buckets
    uint32_t *cursors = first + rcap + 1;                       // [kHeavyWaves][numbers] next slots
    uint16_t *map = reinterpret_cast<uint16_t *>(cursors + kHeavyWaves * rcap);  // [kMapKeys] numbers by key
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = lane_id();
    const uint32_t *cnt = a.counts + (int64_t)j * a.nb;
    const uint64_t *bits = a.ws.bits + (int64_t)j * a.nwb;
    const int64_t bbase = a.ws.bb[j], mbase = a.ws.mb[j];
    const pm_inst I = a.inst ? a.inst[a.item_inst[j]] : a.one;
    const uint32_t *kj = a.keys + I.key_base + (int64_t)(j - I.first_item) * I.x;
    const uint32_t x = (uint32_t)I.x;  // below 2^31
    const uint32_t lo = (uint32_t)((uint64_t)x * wv / kHeavyWaves), hi = (uint32_t)((uint64_t)x * (wv + 1) / kHeavyWaves);

    for (int w = tid; w < a.nwb; w += kHeavyThreads) {
        const uint64_t b = word_in_key_order(bits[w]);
        bm[w] = b;
        wcnt[w] = (uint32_t)__popcll(b);
    }
    __syncthreads();
    heavy_scan(wcnt, a.nwb, scan);

    int64_t slot0 = mbase;  // first slot of the rows' buckets
    for (int w0 = 0, w1, r = 0; w0 < a.nwb; w0 = w1) {
        // ---- the buckets of as many words as there are rows for
        w1 = heavy_reach(wcnt, w0, a.nwb, (uint32_t)rcap);
        const uint32_t b0 = wcnt[w0], wn = (uint32_t)(w1 - w0);
        const int n = (int)(wcnt[w1] - b0);  // at most rcap: a word has 64
        if (n == 0) continue;
        for (uint32_t u = tid; u < 4 * wn; u += kHeavyThreads) {
            const int w = w0 + (int)(u >> 2), sh = 16 * (u & 3);
            const uint64_t b = bm[w];
            uint32_t at = wcnt[w] - b0 + (uint32_t)__popcll(b & ((1ull << sh) - 1ull));
            for (uint32_t q = (uint32_t)(b >> sh) & 0xffffu; q; q &= q - 1u)
                num[at++] = (uint32_t)w * 64u + (uint32_t)(sh + __ffs((int)q) - 1);
        }
        if (tid == 0) n_big = 0;
        const uint32_t k0 = 64u * (uint32_t)w0, kn = 64u * wn;  // the range's keys
        const bool mapped = kn <= (uint32_t)kMapKeys;
        if (mapped)
            for (uint32_t d = tid; d < kn; d += kHeavyThreads) map[d] = 0xffffu;
        __syncthreads();
        for (int i = tid; i < n; i += kHeavyThreads) first[i] = cnt[num[i]];
        __syncthreads();
        heavy_scan(first, n, scan);
        for (int i = tid; i < n; i += kHeavyThreads) {
            const int64_t b = bbase + b0 + i;
            const uint32_t f = first[i], c = first[i + 1] - f;
            const bool kept = b < a.cap_b;
            if (kept && dense && part == 0) a.buckets[b] = pm_bucket{(uint32_t)j, num[i], c, (uint32_t)(slot0 + f)};
            const uint32_t q = kept && (dense || c > kHeavyBig) ? atomicAdd(&n_big, 1u) : 0xffffffffu;
            if (mapped) map[num[i] - k0] = (uint16_t)q;
            num[i] = q;
        }
        __syncthreads();
        const uint32_t nq = n_big;
        // a trial's ranges are shared by `parts` workgroups; a range without big
        // buckets needs none
        if (nq > 0 && r++ % parts == part) {
            uint32_t *mine = cursors + wv * nq;
            // the number of a key's bucket (nq or more: none)
            auto number = [&](uint32_t key) {
                // (0xffffffff, where there is no window or key, is in no range)
                if (mapped) return key - k0 < kn ? (uint32_t)map[key - k0] : 0xffffffffu;
                const uint32_t wd = key >> 6;
                if (wd - (uint32_t)w0 >= wn) return 0xffffffffu;
                const uint64_t m = bm[wd];
                if (!((m >> (key & 63u)) & 1ull)) return 0xffffffffu;
                return num[wcnt[wd] + (uint32_t)__popcll(m & ((1ull << (key & 63u)) - 1ull)) - b0];
            };
            uint32_t nk[kCursorU];  // the next step's keys, loaded ahead
            auto load_keys = [&](uint32_t wb) {
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) {
                    const uint32_t w = wb + 64 * u + lane;
                    nk[u] = w < hi ? kj[w] : 0xffffffffu;
                }
            };
            for (uint32_t e = tid; e < kHeavyWaves * nq; e += kHeavyThreads) cursors[e] = 0;
            load_keys(lo);
            __syncthreads();
            for (uint32_t wb = lo; wb < hi; wb += 64 * kCursorU) {
                uint32_t q[kCursorU];
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) q[u] = nk[u];
                load_keys(wb + 64 * kCursorU);
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) q[u] = number(q[u]);
#pragma unroll
                for (int u = 0; u < kCursorU; ++u)
                    if (q[u] < nq) atomicAdd(mine + q[u], 1u);
            }
            load_keys(lo);
            __syncthreads();
            for (int i = tid; i < n; i += kHeavyThreads) {
                const uint32_t q = num[i];
                if (q >= nq) continue;
                uint32_t run = first[i], c[kHeavyWaves];
#pragma unroll
                for (int w = 0; w < kHeavyWaves; ++w) c[w] = cursors[w * nq + q];
#pragma unroll
                for (int w = 0; w < kHeavyWaves; ++w) {
                    cursors[w * nq + q] = run;
                    run += c[w];
                }
            }
            __syncthreads();
            for (uint32_t wb = lo; wb < hi; wb += 64 * kCursorU) {
                uint32_t q[kCursorU], old[kCursorU], now[kCursorU];
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) q[u] = nk[u];
                load_keys(wb + 64 * kCursorU);
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) q[u] = number(q[u]);
                // the steps in order: a wave's LDS operations complete in order
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) {
                    old[u] = 0;
                    now[u] = 1;
                    if (q[u] < nq) {
                        old[u] = __hip_atomic_fetch_add(mine + q[u], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        now[u] = __hip_atomic_load(mine + q[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
#pragma unroll
                for (int u = 0; u < kCursorU; ++u) {
                    uint64_t met = __ballot(now[u] != old[u] + 1u);
                    while (met) {
                        // lanes of one bucket, all but one of which see a larger
                        // value: their slots in lane order
                        const uint32_t b = (uint32_t)__builtin_amdgcn_readlane(
                            (int)q[u], __ffsll((unsigned long long)met) - 1);
                        const uint64_t peers = __ballot(q[u] == b);
                        if (q[u] == b)
                            old[u] = now[u] - (uint32_t)__popcll(peers) + (uint32_t)__popcll(peers & lanemask_lt());
                        met &= ~peers;
                    }
                    const int64_t slot = slot0 + old[u];
                    if (q[u] < nq && slot < a.cap_m) a.members[slot] = wb + 64 * u + lane;
                }
            }
        }
        __syncthreads();
        slot0 += first[n];
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kHeavyThreads, 4) k_sel_emit_cursors(const SelArgs a)
{
    extern __shared__ __align__(16) uint64_t bm[];
    __shared__ int64_t claim;
    if (a.ws.qctr[2] == 0) return;
    const int64_t nh = *a.ws.n_heavy;
    const int parts = (int)(nh >= gridDim.x ? 1 : min((int64_t)8, ((int64_t)gridDim.x + nh - 1) / nh));
    unsigned long long *q = reinterpret_cast<unsigned long long *>(a.ws.qctr + 1);
    for (;;) {
        if (threadIdx.x == 0) claim = (int64_t)atomicAdd(q, 1ull);
        __syncthreads();
        const int64_t un = claim;
        __syncthreads();
        if (un >= nh * parts) break;  // every workgroup ends here once the queue is past its end
        const int32_t entry = a.ws.heavy[un % nh];
        const int j = entry & ~kHasBig, part = (int)(un / nh);
        const int64_t ne = a.ws.ne[j];
        const bool dense = heavy_dense(ne, a.ws.ms[j]);
        if (!dense && entry >= 0) continue;  // uniform over the workgroup
        // a trial that fits the LDS is one range
        if (part > 0 && ne <= cursor_rows(a.room)) continue;
        emit_cursors(a, j, ne, dense, part, parts, bm);
    }
}

// ---------------------------------------------------------------- a6
struct ProfArgs {
    pm_inst one;               // the instance, when inst is NULL
    const pm_inst *inst;       // batch: instance table, or NULL
    const int32_t *item_inst;  // batch: instance of every trial item
    const pm_bucket *buckets;
    const uint32_t *members;
    const int64_t *n_dev;
    uint32_t *profile;
    int64_t B, cap_m;
    int l, A;
};

// SW lanes per bucket (16 for l <= 16, else 32; 64 / SW buckets per wave);
// lane j of a bucket's group owns column j
template <int SW>
__global__ void __launch_bounds__(256) k_profile(const ProfArgs a)
{
    constexpr int NB = 64 / SW;  // buckets per wave
    __shared__ uint32_t cnt[4][NB][20 * SW];
    const int wv = threadIdx.x >> 6, lane = lane_id(), sub = lane / SW, j = lane % SW;
    const int64_t b = ((int64_t)blockIdx.x * 4 + wv) * NB + sub;
    int64_t nvalid = a.n_dev ? *a.n_dev : a.B;
    if (nvalid > a.B) nvalid = a.B;
    if (((int64_t)blockIdx.x * 4 + wv) * NB >= nvalid) return;  // the wave's first bucket (uniform)
    const bool live = b < nvalid;
    uint32_t *C = cnt[wv][sub];
    for (int i = j; i < a.A * SW; i += SW) C[i] = 0;
    pm_bucket bk{0u, 0u, 0u, 0u};
    if (live) bk = a.buckets[b];
    const pm_inst I = a.inst ? a.inst[a.item_inst[live ? bk.trial : 0]] : a.one;
    const int64_t lm1 = a.l - 1;
    const uint32_t size = live && (int64_t)bk.first + bk.size <= a.cap_m ? bk.size : 0u;
    // SW members at a time: lane j finds where member j starts, then every
    // column lane reads the members' symbols one after another
    uint32_t most = size;  // the wave's largest bucket
#pragma unroll
    for (int o = SW; o < 64; o <<= 1) {
        const uint32_t t = __shfl_xor(most, o);
        most = t > most ? t : most;
    }
    for (uint32_t r0 = 0; r0 < most; r0 += SW) {
        const uint32_t nr = size > r0 ? (size - r0 < (uint32_t)SW ? size - r0 : (uint32_t)SW) : 0u;
        int64_t Pm = 0;
        if ((uint32_t)j < nr) {
            const int64_t w = a.members[(int64_t)bk.first + r0 + j];
            int lo = 0, hi = I.t;  // last sequence whose first window <= w
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (I.offsets[mid] - (int64_t)mid * lm1 <= w) lo = mid;
                else hi = mid;
            }
            Pm = w + (int64_t)lo * lm1;
        }
        const uint32_t nmost = most - r0 < (uint32_t)SW ? most - r0 : (uint32_t)SW;
        for (uint32_t r = 0; r < nmost; ++r) {
            const int64_t P = __shfl(Pm, sub * SW + (int)r);
            if (r < nr && j < a.l) {
                const uint32_t code = a.A == 4 ? dna_sym(I.packed, P + j) : prot_sym(I.packed, P + j);
                C[code * SW + j] += 1;
            }
        }
    }
    if (!live) return;
    uint32_t *out = a.profile + b * a.A * a.l;
    for (int c = 0; c < a.A; ++c)
        if (j < a.l) out[c * a.l + j] = C[c * SW + j];
}

// one thread per (bucket, column): the bucket's size from column 0, then the
// column's A letters
__global__ void k_theta_init(const uint32_t *__restrict__ prof, const int64_t *n_dev, int64_t B, int A,
                             int l, const double *__restrict__ bg, double beta, double *__restrict__ th)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t b = g <= 0xffffffffll ? (int64_t)((uint32_t)g / (uint32_t)l) : g / l;
    int64_t nvalid = n_dev ? *n_dev : B;
    if (nvalid > B) nvalid = B;
    if (b >= nvalid) return;
    const int p = (int)(g - b * l);
    const int64_t per = (int64_t)A * l;
    const uint32_t *P = prof + b * per;
    double *T = th + b * per;
    double size = 0;
    for (int cc = 0; cc < A; ++cc) size += P[cc * l];
    for (int c = 0; c < A; ++c) T[c * l + p] = (P[c * l + p] + beta * bg[c]) / (size + beta);
}

}  // namespace pm

using namespace pm;

// |Sigma|^k for the count-table selection, or -1 above 2^19 bins
static int64_t sel_bins(int A, int k)
{
    if ((A != 4 && A != 20) || k < 1) return -1;
    int64_t nb = 1;
    for (int i = 0; i < k; ++i) {
        nb *= A;
        if (nb > (1ll << 19)) return -1;
    }
    return nb;
}

extern "C" size_t pm_select_workspace(int32_t alphabet, int32_t k, int32_t m, int64_t cap_buckets)
{
    const int64_t nb = sel_bins(alphabet, k);
    if (nb < 0 || m < 0 || cap_buckets < 0) return 0;
    return sel_ws_bytes(m, (nb + 63) / 64);  // member cursors live in LDS: no per-bucket space
}

// dynamic LDS of the emit kernels: bitmap, word scans, cursor row 0, then
// rows 1-3 or the member lists of a trial with few members
static size_t sel_emit_lds(int64_t nwb, int64_t cb)
{
    return (size_t)(16 * nwb + 4 * cb + 4 * std::max<int64_t>(3 * cb, 8 * kSelListCap));
}

// counted: the bitmap and the per-trial totals are already in the workspace
// (projection_hash_select's hash pass wrote them), so no counting pass
static int select_launch(SelArgs &a, int64_t x_max, hipStream_t st, bool counted = false)
{
    const int64_t nwb = (a.nb + 63) / 64;
    a.nwb = (int)nwb;
    a.parts = counted ? 1 : sel_parts(a.m, nwb);
    if (!counted) {
        hipLaunchKernelGGL(k_sel_count, dim3((unsigned)((int64_t)a.m * a.parts)), dim3(256), 0, st, a);
        PM_LAUNCHED();
    }
    // the first emit launch keeps its LDS near 20 KB (eight workgroups per CU)
    // and takes the trials whose buckets fit there, a second one the rest, from
    // a list the scan writes
    const int64_t ne_bound = std::min<int64_t>(a.nb, x_max / std::max<uint32_t>(a.s, 1u));
    const int64_t lds_max = device_lds_bytes() - kHeavyStatic;
    const int64_t cb_a = std::max<int64_t>(
        1, std::min<int64_t>(std::min<int64_t>(ne_bound, kSelChunk / 2), std::max<int64_t>(256, (20480 - 16 * nwb) / 16)));
    // counts not written by projection_hash may pass anywhere
    const bool heavy = a.nb > cb_a;
    a.light = heavy ? 4 * kSelListCap : INT64_MAX;
    TotScan ts{a.ws.ne, a.ws.ms, a.ws.bb, a.ws.mb, a.m, a.cap_b, a.cap_m, a.n_out, a.status};
    if (a.parts > 1) {
        ts.ne = a.ws.nep;
        ts.ms = a.ws.msp;
        ts.parts = a.parts;
        ts.ne_sum = a.ws.ne;
        ts.ms_sum = a.ws.ms;
    }
    if (heavy) {
        ts.heavy = a.ws.heavy;
        ts.n_heavy = a.ws.n_heavy;
        ts.heavy_above = cb_a;
        ts.heavy_members = a.light;
    }
    if (int rc = launch_tot_scan(ts, st)) return rc;
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)k_sel_emit, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
        (void)hipFuncSetAttribute((const void *)k_sel_emit_heavy, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds_max);
        (void)hipFuncSetAttribute((const void *)k_sel_emit_cursors, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds_max);
        (void)hipGetLastError();  // an unsupported attribute must not poison the launch check
        attr = true;
    }
    a.cb = (int)cb_a;
    hipLaunchKernelGGL(k_sel_emit, dim3(a.m), dim3(256), sel_emit_lds(nwb, cb_a), st, a);
    PM_LAUNCHED();
    if (heavy) {
        // two workgroups per CU while the bitmap and its scan leave them a
        // third of their LDS
        const int64_t half = (device_lds_bytes() / 2 - kHeavyStatic) & ~(int64_t)7;
        const int64_t lds = half - 12 * nwb >= half / 3 ? half : lds_max & ~(int64_t)7;
        a.room = (int)(lds - 12 * nwb - 8);
        const int grid = (int)std::min<int64_t>(8 * (int64_t)a.m, lds == half ? 512 : 256);
        a.cursors = x_max > kCursorWindows;
        hipLaunchKernelGGL(k_sel_emit_heavy, dim3(grid), dim3(kHeavyThreads), (size_t)lds, st, a);
        PM_LAUNCHED();
        if (a.cursors) {
            const int64_t all = lds_max & ~(int64_t)7;
            a.room = (int)(all - 12 * nwb - 8);
            const int grid1 = (int)std::min<int64_t>(8 * (int64_t)a.m, 256);
            hipLaunchKernelGGL(k_sel_emit_cursors, dim3(grid1), dim3(kHeavyThreads), (size_t)all, st, a);
            PM_LAUNCHED();
        }
    }
    return PM_OK;
}

static int check_select_args(int A, int k, int32_t items, const uint32_t *keys, const uint32_t *counts,
                             const int64_t *n_out, void *ws, size_t ws_bytes, pm_bucket *buckets,
                             int64_t cap_buckets, uint32_t *members, int64_t cap_members)
{
    if (items < 1) return fail(PM_EINVAL, "m must be >= 1");
    if (sel_bins(A, k) < 0) return fail(PM_ERANGE, "|Sigma|^k above 2^19");
    if (!keys || !counts || !n_out || !ws) return fail(PM_EINVAL, "keys, counts, n_out and ws are required");
    if (cap_buckets < 0 || cap_members < 0) return fail(PM_EINVAL, "negative capacity");
    if ((cap_buckets > 0 && !buckets) || (cap_members > 0 && !members))
        return fail(PM_EINVAL, "NULL output with a non-zero capacity");
    if (cap_members > 0xffffffffll) return fail(PM_ERANGE, "cap_members must be below 2^32");
    if (ws_bytes < pm_select_workspace(A, k, items, cap_buckets)) return fail(PM_EINVAL, "workspace too small");
    if (reinterpret_cast<uintptr_t>(ws) & 7) return fail(PM_EINVAL, "workspace must be 8-byte aligned");
    return PM_OK;
}

namespace pm {

int check_select_ws(int A, int k, int32_t items, const uint32_t *keys, const uint32_t *counts,
                    const int64_t *n_out, void *ws, size_t ws_bytes, pm_bucket *buckets, int64_t cap_buckets,
                    uint32_t *members, int64_t cap_members)
{
    return check_select_args(A, k, items, keys, counts, n_out, ws, ws_bytes, buckets, cap_buckets, members,
                             cap_members);
}

__global__ void k_sel_zero(int64_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

int select_counted_prepare(void *ws, int32_t m, int A, int k, SelCounted *out, hipStream_t st)
{
    const int64_t nb = sel_bins(A, k), nwb = (nb + 63) / 64;
    const SelWs w = carve(ws, m, nwb);
    // ne and ms are adjacent: [m] each
    hipLaunchKernelGGL(k_sel_zero, dim3((unsigned)((2 * (int64_t)m + 255) / 256)), dim3(256), 0, st, w.ne,
                       2 * (int64_t)m);
    PM_LAUNCHED();
    *out = SelCounted{w.bits, w.ne, w.ms, nwb};
    return PM_OK;
}

int select_counted(const pm_inst &one, const pm_inst *inst, const int32_t *item_inst, int A, int k,
                   const uint32_t *keys, const uint32_t *counts, int32_t m, uint32_t s, pm_bucket *buckets,
                   int64_t cap_buckets, uint32_t *members, int64_t cap_members, int64_t *n_out, void *ws,
                   uint32_t *status, int64_t x_max, hipStream_t st)
{
    SelArgs a{};
    a.one = one;
    a.inst = inst;
    a.item_inst = item_inst;
    a.keys = keys;
    a.counts = counts;
    a.buckets = buckets;
    a.members = members;
    a.n_out = n_out;
    a.status = status;
    a.nb = sel_bins(A, k);
    a.ws = carve(ws, m, (a.nb + 63) / 64);
    a.cap_b = cap_buckets;
    a.cap_m = cap_members;
    a.m = m;
    a.s = s;
    return select_launch(a, x_max, st, true);
}

}  // namespace pm

extern "C" int bucket_select(const pm_seqs *S, int32_t l, int32_t k, const uint32_t *keys,
                             const uint32_t *counts, int32_t m, uint32_t s, pm_bucket *buckets,
                             int64_t cap_buckets, uint32_t *members, int64_t cap_members,
                             int64_t *n_out, void *ws, size_t ws_bytes, uint32_t *status, void *stream)
{
    clear_error();
    int rc = check_seqs(S, l);
    if (rc) return rc;
    if (k < 1 || k > l) return fail(PM_EINVAL, "need 1 <= k <= l");
    if ((rc = check_select_args(S->alphabet, k, m, keys, counts, n_out, ws, ws_bytes, buckets, cap_buckets, members,
                                cap_members)))
        return rc;
    SelArgs a{};
    a.one = inst_of(S, l);
    a.keys = keys;
    a.counts = counts;
    a.buckets = buckets;
    a.members = members;
    a.n_out = n_out;
    a.status = status;
    a.nb = sel_bins(S->alphabet, k);
    a.ws = carve(ws, m, (a.nb + 63) / 64);
    a.cap_b = cap_buckets;
    a.cap_m = cap_members;
    a.m = m;
    a.s = s;
    return select_launch(a, a.one.x, as_stream(stream));
}

extern "C" int bucket_select_batch(const pm_batch *B, const uint32_t *keys, const uint32_t *counts, uint32_t s,
                                   pm_bucket *buckets, int64_t cap_buckets, uint32_t *members,
                                   int64_t cap_members, int64_t *n_out, void *ws, size_t ws_bytes,
                                   uint32_t *status, void *stream)
{
    clear_error();
    BatchInfo info;
    int rc = check_batch(B, &info);
    if (rc) return rc;
    if ((rc = check_select_args(B->alphabet, B->k, B->items, keys, counts, n_out, ws, ws_bytes, buckets, cap_buckets,
                                members, cap_members)))
        return rc;
    SelArgs a{};
    a.inst = B->inst;
    a.item_inst = B->item_inst;
    a.keys = keys;
    a.counts = counts;
    a.buckets = buckets;
    a.members = members;
    a.n_out = n_out;
    a.status = status;
    a.nb = sel_bins(B->alphabet, B->k);
    a.ws = carve(ws, B->items, (a.nb + 63) / 64);
    a.cap_b = cap_buckets;
    a.cap_m = cap_members;
    a.m = B->items;
    a.s = s;
    return select_launch(a, info.x_max, as_stream(stream));
}

static int profile_launch(const ProfArgs &a, hipStream_t st)
{
    if (a.l <= 16) {
        hipLaunchKernelGGL(k_profile<16>, dim3((unsigned)((a.B + 15) / 16)), dim3(256), 0, st, a);
    } else {
        hipLaunchKernelGGL(k_profile<32>, dim3((unsigned)((a.B + 7) / 8)), dim3(256), 0, st, a);
    }
    PM_LAUNCHED();
    return PM_OK;
}

extern "C" int bucket_profile(const pm_seqs *S, int32_t l, const pm_bucket *buckets,
                              const uint32_t *members, int64_t cap_members, int64_t B,
                              const int64_t *n_dev, uint32_t *profile, void *stream)
{
    clear_error();
    int rc = check_seqs(S, l);
    if (rc) return rc;
    if (B < 0) return fail(PM_EINVAL, "B must be >= 0");
    if (B == 0) return PM_OK;
    if (!buckets || !members || !profile) return fail(PM_EINVAL, "NULL buffer");
    ProfArgs a{};
    a.one = inst_of(S, l);
    a.buckets = buckets;
    a.members = members;
    a.n_dev = n_dev;
    a.profile = profile;
    a.B = B;
    a.cap_m = cap_members;
    a.l = l;
    a.A = S->alphabet;
    return profile_launch(a, as_stream(stream));
}

extern "C" int bucket_profile_batch(const pm_batch *Bt, const pm_bucket *buckets, const uint32_t *members,
                                    int64_t cap_members, int64_t B, const int64_t *n_dev, uint32_t *profile,
                                    void *stream)
{
    clear_error();
    int rc = check_batch(Bt, nullptr);
    if (rc) return rc;
    if (B < 0) return fail(PM_EINVAL, "B must be >= 0");
    if (B == 0) return PM_OK;
    if (!buckets || !members || !profile) return fail(PM_EINVAL, "NULL buffer");
    ProfArgs a{};
    a.inst = Bt->inst;
    a.item_inst = Bt->item_inst;
    a.buckets = buckets;
    a.members = members;
    a.n_dev = n_dev;
    a.profile = profile;
    a.B = B;
    a.cap_m = cap_members;
    a.l = Bt->l;
    a.A = Bt->alphabet;
    return profile_launch(a, as_stream(stream));
}

extern "C" int theta_init(int32_t alphabet, int32_t l, const uint32_t *profile, int64_t B,
                          const int64_t *n_dev, const double *bg, double beta, double *theta0,
                          void *stream)
{
    clear_error();
    if (alphabet != 4 && alphabet != 20) return fail(PM_EINVAL, "alphabet must be 4 or 20");
    if (l < 1 || l > 32) return fail(PM_EINVAL, "need 1 <= l <= 32");
    if (B < 0 || beta < 0) return fail(PM_EINVAL, "need B >= 0 and beta >= 0");
    if (B == 0) return PM_OK;
    if (!profile || !bg || !theta0) return fail(PM_EINVAL, "NULL buffer");
    const int64_t total = B * l;
    const int threads = 256;
    hipLaunchKernelGGL(k_theta_init, dim3((unsigned)((total + threads - 1) / threads)), dim3(threads), 0,
                       as_stream(stream), profile, n_dev, B, alphabet, l, bg, beta, theta0);
    PM_LAUNCHED();
    return PM_OK;
}
