// a7 - a9 on the matrix cores: OOPS EM of DNA models as one-hot contractions.
//
// For a tile of windows and a group of 16 models the E-step scores are a
// product of the windows' one-hot encoding (4l columns, entries 0/1) with the
// models' log-odds (4l x 16):  S = OneHot . W.  The M-step counts are the
// transposed product with the posteriors:  C = OneHot^T . P.  Per sequence
// the posteriors are a softmax over windows, so one pass over a sequence is
// an attention-like sweep with a reference maximum and rescaled accumulators.
//
// Arithmetic: the E-step on v_smfmac_f32_16x16x64_f16 (the one-hot operand as
// the 2-of-4 sparse one, see Tiles), the M-step on v_mfma_f32_16x16x32_f16.
// The one-hot side is exact in FP16.
// The other side is split in two FP16 halves, x = hi + lo with
// hi = fp16(x) and lo = fp16(x - hi), both multiplied by the same one-hot
// operand, so every product is exact and the operand carries about 22
// significant bits; sums are FP32.  The single-FP16 form (SPLIT = false) keeps
// only hi: half the matrix-core work, 11-bit operands.  Scores are kept in
// log2 units (W = log2 theta - log2 bg by the hardware FP32 logarithm, about
// 2^-23 relative, inside the 22 bits the split halves carry; the prior term of
// J adds those logarithms in FP64) so the softmax uses the hardware exp2.  The per-sequence
// log-sum-exp is FP64: the posterior terms 2^(S - ref) are FP32 exp2 of FP32
// scores; the eight a lane holds for one window pair are added in FP32 (three
// levels), and these pair partials are accumulated over the whole sequence in
// FP64, so the error does not grow with the sequence length; the four lane
// groups are combined with FP64 shuffles and the logarithm is FP64, as are
// the objective and the final comparison.
//
// Lane layout of one 16x16x32 MFMA (lane L, r = L % 16, g = L / 16):
//   A operand: row r, the g-th group of 8 contraction indices;
//   B operand: column r, the same 8 contraction indices;
//   D:         column r, rows 4g .. 4g+3;
// of one 16x16x64 sparse MFMA:
//   A operand: row r, of the indices 16g .. 16g+15 two in every four (8 values
//              and their places, 2 bits each);
//   B operand: column r, indices 8g .. 8g+7 and 32+8g .. 32+8g+7.
// E-step: rows = 16 windows, columns = 16 models, contraction = (position,
// letter) pairs, position-major, 16 positions (a fragment) per instruction.
// M-step: rows = 16 (position, letter) pairs, columns =
// models, contraction = 32 windows (two E tiles); lane (r, g) carries windows
// 4g..4g+3 of the first tile and of the second, exactly the rows its E-step
// outputs hold, so posteriors feed the M-step without leaving registers.
//
// Softmax reference: scores leave the E-step already shifted by the current
// reference (the accumulator starts at -reference), and the reference moves
// only when a score passes it by more than kSlack, so the common path needs
// neither a cross-lane maximum nor a rescale.  It starts just under the
// sequence's largest score of the previous iteration (sweep).  Posteriors enter the M-step as
// 2^(S - ref + kPOff) <= 2^(kPOff + kSlack) = 2^15, inside the FP16 range.
// The reference moves by whole numbers, so every rescale (of the count
// accumulators and of the FP64 sums) is an exact power of two.
//
// Work split: a workgroup of four waves takes 64 G models of one instance, G
// groups of 16 per wave; the groups of a wave share every A operand (the
// one-hot tables), so G = 2 halves the table reads and builds per model and
// gives each wave two independent E-step/softmax/M-step chains to interleave.
// The four waves sweep the same windows in step; the one-hot tables of PPB
// window pairs sit in LDS per step (double-buffered, one barrier per PPB
// pairs).  With a workspace, k_em_tables builds every pair's tables once per
// call and the EM kernel copies each step's into LDS, loading the next step's
// while it computes; without one, the workgroup builds them itself from the
// packed instance in global memory.  (G, PPB) is the tunable tile
// shape: em_autotune times the variants on the caller's models and records
// the fastest per (ceil(l/4), precision) class.
//
// What bounds it: no pipe alone.  Counters of (18,6), 89 000 models, 10
// iterations, default shape: the matrix pipe is busy 37% of the time and the
// vector unit 56%; a wave issues in 36% of its cycles, waits for an issue slot
// (with two others on its SIMD) in 37%, and for data or a barrier in 27%.  An
// MFMA takes two of the vector unit's issue slots (8 cycles) and overlaps the
// rest of its 16, so a pair of 16 MFMAs and 44 vector instructions, 8 of them
// exponentials, would take about 350 cycles of a SIMD; 600 are measured at
// three waves per SIMD.  Measured on that workload: 12.0 ms with the dense
// E-step, references started from the lowest score and two FP64 logarithms
// per sequence; 11.8 with the sparse E-step (16 instead of 20 MFMAs a pair),
// 10.3 in a timing copy whose references never move.  (15,4) batch of 24
// instances: 18.1 -> 15.4 ms; single FP16, (21,7), 16 384 models, 5 iterations:
// 6.8 -> 6.3 ms, 3.8 ms in three parts.  The slots one after the other cost
// 1 to 3% (10.48 -> 10.58 ms, 15.2 -> 15.6 ms) against one sum over all
// sequences.
#include <math.h>
#include <stddef.h>
#include <stdlib.h>

#include "pm_common.h"

namespace pm {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half16 __attribute__((ext_vector_type(16)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
// counts that wait in theta_out's entries
typedef float float4_in __attribute__((ext_vector_type(4), aligned(8), may_alias));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // one 16-byte table quad

struct EmMfmaArgs {
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
    int64_t nwords;  // packed words (reads are clamped below this)
    int t, l, iters;
    int site_stride; // sites row length (t, or the largest t of a batch)
    int split;       // 1: two FP16 halves per operand; 0: one FP16 value
    double beta;
    // batch: the instance table and the workgroup plan (k_em_plan), or NULL
    const pm_inst *inst;
    const int64_t *plan;
    int P;
    // precomputed one-hot tables (k_em_tables), or NULL to build them in the
    // kernel; tbase: first slot of every instance of a batch (NULL: one instance)
    const uint8_t *tables;
    const int64_t *tbase;
    // instances of at most mcap sequences keep every sequence's largest score
    // of the previous iteration in LDS (0: none)
    int mcap;
};

// workgroups of a launch that takes mw models per workgroup: whole groups of
// the B models, or, for a batch, the plan's count bounded by one partly filled
// group per instance
static inline int64_t em_groups(const EmMfmaArgs &a, int mw)
{
    const int64_t full = (a.B + mw - 1) / mw;
    return a.inst ? full + a.P : full;
}

// Workgroup plan of a batch: the instances in decreasing order of windows
// (the longest sweeps start first), each cut into groups of 16 kWaves G
// consecutive buckets (the models of one workgroup).  Layout: wg_start[P + 1] (first workgroup of each rank),
// b0[P], b1[P] (bucket range of each instance), order[P] (instance of each rank).
struct PlanView {
    const int64_t *wg_start, *b0, *b1, *order;
};
__host__ __device__ inline PlanView plan_view(const int64_t *plan, int P)
{
    return PlanView{plan, plan + P + 1, plan + 2 * P + 1, plan + 3 * P + 1};
}

constexpr int kWaves = 4;  // waves (groups of 16 models) per part of a workgroup
// A model's sequences are summed in em_slots slots (i, i + slots, ..), whose
// counts and log-likelihoods are added in order at the end of an iteration: a
// model's result does not depend on what else the launch holds.  A launch whose
// models alone would leave SIMDs idle (em_parts) takes the slots side by side,
// as parts of a workgroup of kWaves waves each with their own tables and
// counts (and one group of models per wave); else they follow each other, the
// counts of all but the last waiting in theta_out, which the iteration has read
// and not yet written.
constexpr int kPartThreads = 64 * kWaves;
__device__ __forceinline__ int part_thread() { return (int)(threadIdx.x % kPartThreads); }
// tile shape 10 G + PPB: G groups of 16 models per wave, PPB window pairs
// built per workgroup barrier
constexpr int kShapeDefault = 14;  // untuned
// the form in parts: one group of models per wave, kPartsPPB window pairs
constexpr int kPartsPPB = 4;
constexpr int kShapeParts = 100 + 10 + kPartsPPB;
constexpr int shape_groups(int shape) { return shape / 10 % 10; }
constexpr int kMaxMT2 = 6;         // G = 2 for ceil(l/4) <= 6 (registers)
constexpr float kPOff = 3.0f;
constexpr float kSlack = 12.0f;
// A known sequence's reference starts this far below its largest score of the
// iteration before (rounded up): room for it to fall by kBelow bits (else the
// iteration is repeated) and to rise by kSlack - kBelow (else the reference
// moves).  On the (12,4) to (24,7) shapes the largest score of a sequence
// changes by -8 to +8 bits from theta0 to theta1 (medians near +2, 1% beyond
// -6 and +5) and by less than 6 bits either way afterwards.
constexpr float kBelowFirst = 8.0f;  // iteration 1
constexpr float kBelow = 5.0f;       // later ones
// smallest largest shifted score of such a sweep: what a reference that moves
// leaves at least (kPOff - 1), so that the FP16 halves of the small terms keep
// as many bits
constexpr float kTopMin = kPOff - 1.0f;
static_assert(kTopMin == 2.0f, "terms of 2^2 and more");

// 32 DNA symbols starting at P (MSB-first) as hi (P..P+15) and lo (P+16..P+31).
// CLAMP: reads clamped below nw (global memory); otherwise the buffer is padded.
template <bool CLAMP>
__device__ __forceinline__ void dna32(const uint32_t *w, int64_t P, int64_t nw, uint32_t &hi, uint32_t &lo)
{
    const int64_t wi = P >> 4;
    const uint32_t r = (uint32_t)(P & 15) << 1;
    uint32_t w0, w1, w2;
    if (CLAMP) {
        w0 = w[wi < nw ? wi : nw - 1];
        w1 = w[wi + 1 < nw ? wi + 1 : nw - 1];
        w2 = w[wi + 2 < nw ? wi + 2 : nw - 1];
    } else {
        w0 = w[wi];
        w1 = w[wi + 1];
        w2 = w[wi + 2];
    }
    hi = (uint32_t)((((uint64_t)w0 << 32) | w1) >> (32 - r));
    lo = (uint32_t)((((uint64_t)w1 << 32) | w2) >> (32 - r));
}

// where a workgroup's one-hot tables come from
constexpr int kSrcGlobal = 0;  // built in the kernel from the packed instance (no workspace)
constexpr int kSrcPre = 2;     // copied from tables precomputed once per call (k_em_tables)

// Precomputed tables: pair j (windows 32j .. 32j+31) of sequence i of an
// instance sits in slot i + floor(W_i / 32) + j, W_i = offsets[i] - i (l - 1)
// being the sequence's first window in the instance's window numbering.  A
// sequence of L_i windows ends at slot i + floor((W_i + L_i) / 32) at most, so
// the slots of different sequences never overlap and an instance needs at
// most t + ceil(x / 32) of them (a few stay unused).
__host__ __device__ inline int64_t em_inst_slots(int64_t t, int64_t x) { return t + (x + 31) / 32; }

__device__ __forceinline__ int64_t seq_slot0(const int64_t *offsets, int i, int l)
{
    return i + (offsets[i] - (int64_t)i * (l - 1)) / 32;
}

// fp16(p - hi) for two values whose fp16 roundings are packed in hi2
__device__ __forceinline__ uint32_t split_lo(uint32_t hi2, float p0, float p1)
{
    uint32_t r;
    asm volatile(
        "v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]\n\t"
        "v_fma_mixhi_f16 %0, %1, -1.0, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
        : "=&v"(r)
        : "v"(hi2), "v"(p0), "v"(p1));
    return r;
}

__device__ __forceinline__ uint32_t pack_hi(float p0, float p1)
{
    return __builtin_bit_cast(uint32_t, half2v{(_Float16)p0, (_Float16)p1});
}

// E-step contraction for MT M-tiles (4 MT positions).  A window's one-hot has
// one 1 in every four columns (a position's letters), which is inside the
// 2-of-4 pattern of the sparse matrix instruction, so the E-step runs on
// v_smfmac_f32_16x16x64_f16: 16 positions per instruction where the dense
// form takes 8, at the same rate.  Of a position's four letters the A operand
// stores the pair that holds the symbol (letters 0, 1 or 2, 3: the index
// field) as (1, 0) or (0, 1).  A fragment covers 16 positions, position 4g+i
// of it in lane group g; a last fragment of at most 8 positions (eight)
// repeats them in groups 2, 3, so that the split form's hi and lo halves
// share one instruction.
template <int MT>
struct Tiles {
    static constexpr int FULL = MT / 4;                        // fragments of 16 positions
    static constexpr int REST = 4 * MT % 16;                   // positions of the last one
    static constexpr bool EIGHT = REST == 4 || REST == 8;      // repeated in groups 2, 3
    static constexpr int NF = FULL + (REST != 0 ? 1 : 0);      // fragments of a window
    static constexpr int CX = 4 * MT;       // count rows (positions) of a model
    static constexpr int NE = 4 * MT + 12;  // M-step table entries a pair reads
    static constexpr int NEV = MT <= 4 ? 44 : MT <= 6 ? 52 : 60;  // E-step entries a pair reads
    // up to 24 positions the index fields have room behind the E-step entries
    // (dword e: those of entries e and e + 16, the two tiles of a pair);
    // beyond, an entry keeps the high bytes of its eight halves and its field
    static constexpr bool BYTES = MT > 6;
    // matrix instructions per tile: hi and lo of every fragment, one for both
    // in a repeated one
    static constexpr int ops(bool split) { return split ? 2 * NF - (EIGHT ? 1 : 0) : NF; }
};

// one-hot tables of one window pair: the symbols at s0 + a0 + e
template <int MT>
struct alignas(16) PairTables {
    uint32_t ev[64][4];           // E-step entries: symbols e .. e+3, then the index fields
    uint4 mt8[Tiles<MT>::NE][4];  // [e][c]: symbols e..e+3 and e+16..e+19 == c
};
static_assert(Tiles<4>::NEV * 16 + 28 * 4 <= 1024 && Tiles<6>::NEV * 16 + 36 * 4 <= 1024, "room for the index fields");
// 16-byte quads of one pair's tables: at most 256, one per thread of a workgroup
template <int MT>
constexpr int kTabQuads = (int)(sizeof(PairTables<MT>) / 16);
static_assert(kTabQuads<8> <= 256, "one quad per thread");

// The index field of four symbols (8 bits, first on top): for each, the
// first on the lowest nibble, its pair of letters as two 2-bit row numbers.
__device__ __forceinline__ uint32_t index_field(uint32_t y)
{
    uint32_t f = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) f |= ((y >> (7 - 2 * i)) & 1u ? 0xEu : 0x4u) << (4 * i);
    return f;
}

// lut[y]: four FP16 halves, half q = 1.0 where 2-bit field q of y (from the top)
// is zero.  With y = (4 symbols) ^ (c * 0x55) that is the one-hot of letter c.
__device__ __forceinline__ void build_lut(uint2 *lut)
{
    const uint32_t y = part_thread();  // the parts of a workgroup write the same
    uint32_t h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = ((y >> (6 - 2 * q)) & 3u) ? 0u : 0x3C00u;
    lut[y] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
}

// Workgroup-cooperative build: thread (e = tid / 4, c = tid % 4) writes
// mt8[e][c] (e < NE) and word c of E-step entry e, or a dword of the index
// fields behind the entries.
template <int MT, bool CLAMP>
__device__ __forceinline__ void build_tables(const uint32_t *W, int64_t nw, int64_t base, const uint2 *lut,
                                             PairTables<MT> &T)
{
    const int tid = part_thread(), e = tid >> 2;
    const uint32_t c = tid & 3u;
    uint32_t hi, lo;
    dna32<CLAMP>(W, base + e, nw, hi, lo);
    if (e < Tiles<MT>::NE) {
        const uint32_t cc = c * 0x55u;
        const uint2 u0 = lut[(hi >> 24) ^ cc], u1 = lut[(lo >> 24) ^ cc];
        T.mt8[e][c] = make_uint4(u0.x, u0.y, u1.x, u1.y);
    }
    const uint32_t y = hi >> 24;  // symbols e .. e+3
    if (Tiles<MT>::BYTES) {
        uint32_t v = 0;
        if (c < 2) {
            // halves of symbols 2c, 2c+1: high byte of 1.0 in the half of the letter's parity
            v = (0x3Cu << (((y >> (6 - 4 * c)) & 1u) * 8)) | (0x3C0000u << (((y >> (4 - 4 * c)) & 1u) * 8));
        } else if (c == 2) {
            v = index_field(y);
        }
        T.ev[e][c] = v;
    } else {
        constexpr int NEV = Tiles<MT>::NEV;
        if (e < NEV) T.ev[e][c] = 0x3C00u << (((y >> (6 - 2 * c)) & 1u) << 4);
        // entry e's thread c == 0 also writes dword e of the index fields
        if (c == 0 && e < 4 * (64 - NEV))
            (&T.ev[NEV][0])[e] = index_field(y) | (index_field(lo >> 24) << 16);
    }
}

struct SeqState {
    float4v neg;  // kPOff - mref in every component: the E-step accumulators' start
    float mref;   // reference (log2 units) of the scores
    float top;    // largest shifted score so far
    double srun;  // this lane's share of sum 2^(S - mref + kPOff), in FP64
    float bestv;  // final E-step: best score and window of this lane
    int besti;
};

// LDS byte offsets of this lane's fragments within a pair's tables, formed
// once per sequence: the E-step entry of window r and position 4g, the same
// for a repeated fragment (position 4 (g & 1)), M-step A
struct FragOff {
    uint32_t a, a_eight, m;
};

// the A operand of an E-step fragment: stored values and index field
struct SparseA {
    half8 v;
    int ix;
};

// the operands of fragment f for the two tiles of a pair
template <int MT>
__device__ __forceinline__ void sparse_frag(const char *tb, const FragOff &fo, int f, SparseA (&A)[2])
{
    const bool eight = Tiles<MT>::EIGHT && f == Tiles<MT>::FULL;
    const uint32_t off = (eight ? fo.a_eight : fo.a) + 256u * f;
    if (Tiles<MT>::BYTES) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            const uint4 q = *reinterpret_cast<const uint4 *>(tb + off + 256 * t2);
            // bytes to halves: (0, b0, 0, b1)
            uint4 w;
            w.x = __builtin_amdgcn_perm(0u, q.x, 0x010C000Cu);
            w.y = __builtin_amdgcn_perm(0u, q.x, 0x030C020Cu);
            w.z = __builtin_amdgcn_perm(0u, q.y, 0x010C000Cu);
            w.w = __builtin_amdgcn_perm(0u, q.y, 0x030C020Cu);
            A[t2].v = __builtin_bit_cast(half8, w);
            A[t2].ix = (int)q.z;
        }
    } else {
        // one dword for both tiles, the second's in the high half
        const int ix = *reinterpret_cast<const int *>(tb + 16 * Tiles<MT>::NEV + off / 4);
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            A[t2].v = *reinterpret_cast<const half8 *>(tb + off + 256 * t2);
            A[t2].ix = ix;
        }
    }
}

template <int MT, int TILE>
__device__ __forceinline__ float4v smfma(const SparseA &A, half16 W, float4v S)
{
    // the field's half of the dword: the second tile's is the high one
    return __builtin_amdgcn_smfmac_f32_16x16x64_f16(A.v, W, S, A.ix, 0, TILE == 1 && !Tiles<MT>::BYTES ? 1 : 0);
}

// One pair of 16-window tiles (windows a0 .. a0+31 of one sequence) for this
// wave's G groups of 16 models; the groups share the A operands.
template <int MT, bool LAST, bool TAIL, bool SPLIT, int G>
__device__ __forceinline__ void tile_pair(int a0, int L, const PairTables<MT> &T, const FragOff &fo,
                                          const half16 (&Wb)[G][Tiles<MT>::ops(SPLIT)], float4v (&O)[G][MT],
                                          SeqState (&st)[G])
{
    constexpr int NF = Tiles<MT>::NF;
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const char *tb = reinterpret_cast<const char *>(&T);
    SparseA Ae[NF][2];
#pragma unroll
    for (int f = 0; f < NF; ++f) sparse_frag<MT>(tb, fo, f, Ae[f]);
    // E-step, already shifted: S' = S - (mref - kPOff); one chain per tile and group
    float4v S0[G], S1[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        S0[q] = st[q].neg;
        S1[q] = st[q].neg;
    }
#pragma unroll
    for (int op = 0; op < Tiles<MT>::ops(SPLIT); ++op)
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int f = SPLIT ? op / 2 : op;
            S0[q] = smfma<MT, 0>(Ae[f][0], Wb[q][op], S0[q]);
            S1[q] = smfma<MT, 1>(Ae[f][1], Wb[q][op], S1[q]);
        }
    half8 Am[MT];
    if (!LAST) {
        // M-step A operand: row (position pm, letter cm); windows 4g..4g+3 of both tiles
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)  // mt8[4g + 4mt + r/4][r % 4]
            Am[mt] = *reinterpret_cast<const half8 *>(tb + fo.m + mt * 256);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
        if (TAIL) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (a0 + 4 * g + u >= L) S0[q][u] = -INFINITY;
                if (a0 + 16 + 4 * g + u >= L) S1[q][u] = -INFINITY;
            }
        }
        // the largest shifted score of the sequence so far: passes the slack, or
        // the best start, only when one of these eight does
        const float top = fmaxf(fmaxf(fmaxf(fmaxf(fmaxf(fmaxf(fmaxf(fmaxf(st[q].top, S0[q][0]), S0[q][1]), S0[q][2]),
                                S0[q][3]), S1[q][0]), S1[q][1]), S1[q][2]), S1[q][3]);
        st[q].top = top;
        // a new best start is rare: the eight scores are looked at one by one
        // only where their maximum passes the best so far
        if (LAST && __ballot(top - st[q].neg[0] > st[q].bestv)) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float v = (u < 4 ? S0[q][u & 3] : S1[q][u & 3]) - st[q].neg[0];
                if (v > st[q].bestv) {
                    st[q].bestv = v;
                    st[q].besti = a0 + 16 * (u >> 2) + 4 * g + (u & 3);
                }
            }
        }
        if (__builtin_expect(__ballot(top > kPOff + kSlack) != 0, 0)) {
            // rare: move the reference up to the model's new maximum
            float tm = fmaxf(top, __shfl_xor(top, 16));
            tm = fmaxf(tm, __shfl_xor(tm, 32));
            // a whole number of binades, so that the rescales below are exact
            const float d = tm > kPOff + kSlack ? ceilf(tm - kPOff) : 0.f;
            const float al = __builtin_amdgcn_exp2f(-d);
            st[q].srun *= (double)al;
            if (!LAST)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) O[q][mt] *= al;
            S0[q] -= d;
            S1[q] -= d;
            st[q].top -= d;
            st[q].mref += d;
            const float n = kPOff - st[q].mref;  // exactly what the scores are shifted by
            st[q].neg = float4v{n, n, n, n};
        }
        float S[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            S[j] = S0[q][j];
            S[4 + j] = S1[q][j];
        }
        float P[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) P[u] = __builtin_amdgcn_exp2f(S[u]);
        // the lane's eight terms of this pair (a three-level FP32 tree, relative
        // error at most 3 * 2^-24), accumulated over the sequence in FP64
        st[q].srun += (double)(((P[0] + P[1]) + (P[2] + P[3])) + ((P[4] + P[5]) + (P[6] + P[7])));
        if (!LAST) {
            uint4 h;
            h.x = pack_hi(P[0], P[1]);
            h.y = pack_hi(P[2], P[3]);
            h.z = pack_hi(P[4], P[5]);
            h.w = pack_hi(P[6], P[7]);
            const half8 Ph = __builtin_bit_cast(half8, h);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                O[q][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Am[mt], Ph, O[q][mt], 0, 0, 0);
            if (SPLIT) {
                uint4 lw;
                lw.x = split_lo(h.x, P[0], P[1]);
                lw.y = split_lo(h.y, P[2], P[3]);
                lw.z = split_lo(h.z, P[4], P[5]);
                lw.w = split_lo(h.w, P[6], P[7]);
                const half8 Pl = __builtin_bit_cast(half8, lw);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    O[q][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Am[mt], Pl, O[q][mt], 0, 0, 0);
            }
        }
    }
}

// This thread's quads of the tables of the PPB window pairs starting at
// window a0 of sequence i (kSrcPre): loaded into registers one step ahead of
// their use, written to LDS at the step that uses them.
template <int MT, int PPB>
__device__ __forceinline__ void fetch_tables(const EmMfmaArgs &a, int slot0, int L, int a0, u32x4 (&pf)[PPB])
{
    // every load is unconditional and in bounds (a pair past the sequence's
    // end re-reads the step's first pair, threads past the quads re-read the
    // last one), which keeps pf in registers; only the LDS writes are guarded
    constexpr int NQ = kTabQuads<MT>;
    const int q = part_thread() < NQ ? part_thread() : NQ - 1;
    // slot0 and L are scalars: one scalar base, one lane offset for all loads
    const u32x4 *src = reinterpret_cast<const u32x4 *>(a.tables) + ((int64_t)slot0 + a0 / 32) * NQ;
#pragma unroll
    for (int u = 0; u < PPB; ++u) pf[u] = (src + (a0 + 32 * u < L ? u : 0) * NQ)[(uint32_t)q];
}

// windows and first table slot of sequence i of the instance whose first slot
// is tb (kSrcPre), as scalars (a launch has fewer than 2^31 slots)
__device__ __forceinline__ void seq_slots(const EmMfmaArgs &a, int64_t tb, int i, int &L, int &slot0)
{
    L = __builtin_amdgcn_readfirstlane((int)(a.offsets[i + 1] - a.offsets[i])) - a.l + 1;
    slot0 = __builtin_amdgcn_readfirstlane((int)(tb + seq_slot0(a.offsets, i, a.l)));
}

// A model's log-likelihood over the sequences so far: sum of log2 references
// and exponents (multiples of 2^-23 below 2^29, so exact in any order), and the
// product of the mantissas of its sums (its logarithm is taken once per
// iteration).
struct LogSum {
    double e, m;
    // the product of another slot's mantissas multiplied in
    __device__ __forceinline__ void join(double om)
    {
        const double p = om * m;
        e += (double)__builtin_amdgcn_frexp_exp(p);
        m = __builtin_amdgcn_frexp_mant(p);
    }
};

// One sequence: every window pair (tables built by the whole workgroup, or
// copied from the precomputed ones), then the per-sequence log-sum-exp and
// counts, or, in the final E-step, the best start of every model.  acc[q]:
// the count accumulators of group q.  kSrcPre: pf holds this thread's quads of
// the sequence's first step on entry and the first step of sequence `next` (the
// slot's next one, the next slot's first, or the part's first for the next
// iteration) on return.
//
// mprev: this lane's slots (one per group) of the sequence's largest score in
// the previous iteration (NULL: not kept).  The reference starts `below` under
// it (known[q]), so that it seldom moves: a move costs a wave about a window
// pair's time, and when all models start from their lowest score some model of
// the 16 moves in most pairs of a sequence's first third.  A model whose
// scores all stay under kTopMin of such a start would lose bits of its
// posteriors: low[q] is set, and the caller repeats the iteration with that
// model's references from its lowest score (again: the others start as they
// did before, from the slot's high byte).
template <int MT, int SRC, bool LAST, bool SPLIT, int PPB, int G>
__device__ __forceinline__ void sweep(const EmMfmaArgs &a, const uint32_t *W, const uint2 *lut, int i, int64_t bw,
                                      int64_t nvalid, PairTables<MT> *tabs, int &parity, int64_t tb,
                                      u32x4 (&pf)[PPB], int next, float (*acc)[16][Tiles<MT>::CX][4],
                                      const half16 (&Wb)[G][Tiles<MT>::ops(SPLIT)], const float (&mlow)[G],
                                      int16_t *mprev, const bool (&known)[G], float below, bool again, bool (&low)[G],
                                      LogSum (&llr)[G])
{
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int64_t s0 = a.offsets[i];
    const int L = (int)(a.offsets[i + 1] - s0) - a.l + 1;
    static_assert(offsetof(PairTables<MT>, mt8) == 1024, "M-step fragments follow the 1 KB of E-step ones");
    const FragOff fo{(uint32_t)(r + 4 * g) * 16u, (uint32_t)(r + 4 * (g & 1)) * 16u,
                     1024u + (uint32_t)((4 * g + (r >> 2)) * 4 + (r & 3)) * 16u};
    // kSrcPre: this sequence's and the next one's size and first slot, formed
    // once here rather than at every step
    int sl = 0, sln = 0, Ls = 0, Ln = 0;
    if constexpr (SRC == kSrcPre) {
        seq_slots(a, tb, i, Ls, sl);
        seq_slots(a, tb, next, Ln, sln);
    }
    float4v O[G][MT];
    SeqState st[G];
    int prev[G];  // largest score of the previous iteration
#pragma unroll
    for (int q = 0; q < G; ++q) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) O[q][mt] = float4v{0.f, 0.f, 0.f, 0.f};
        prev[q] = mprev ? (again ? mprev[16 * q] >> 8 : (int)(int8_t)mprev[16 * q]) : 0;
        const float m0 = known[q] ? (float)prev[q] - below : mlow[q], n0 = kPOff - m0;
        st[q] = SeqState{float4v{n0, n0, n0, n0}, m0, -INFINITY, 0.0, -INFINITY, 0};
    }
    for (int a0 = 0; a0 < L; a0 += 32 * PPB) {
        PairTables<MT> *T = tabs + PPB * parity;
        parity ^= 1;
        if constexpr (SRC == kSrcPre) {
#pragma unroll
            for (int u = 0; u < PPB; ++u)
                if (a0 + 32 * u < L && part_thread() < kTabQuads<MT>)
                    reinterpret_cast<u32x4 *>(&T[u])[part_thread()] = pf[u];
        } else {
#pragma unroll
            for (int u = 0; u < PPB; ++u)
                if (a0 + 32 * u < L)
                    build_tables<MT, SRC == kSrcGlobal>(W, a.nwords, s0 + a0 + 32 * u, lut, T[u]);
        }
        __syncthreads();
        if constexpr (SRC == kSrcPre) {
            // the next step's quads (this sequence's, or the next sequence's
            // first) load while this step computes
            const int na = a0 + 32 * PPB;
            if (na < Ls) fetch_tables<MT, PPB>(a, sl, Ls, na, pf);
            else fetch_tables<MT, PPB>(a, sln, Ln, 0, pf);
        }
#pragma unroll
        for (int u = 0; u < PPB; ++u) {
            const int b0 = a0 + 32 * u;
            if (b0 + 32 <= L) tile_pair<MT, LAST, false, SPLIT, G>(b0, L, T[u], fo, Wb, O, st);
            else if (b0 < L) tile_pair<MT, LAST, true, SPLIT, G>(b0, L, T[u], fo, Wb, O, st);
        }
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
        // the sequence's largest score, to the next whole number, for the next
        // iteration (every lane of the model holds the same)
        if (mprev) {
            float tp = st[q].top;
            tp = fmaxf(tp, __shfl_xor(tp, 16));
            tp = fmaxf(tp, __shfl_xor(tp, 32));
            low[q] |= known[q] && !(tp >= kTopMin);
            const float m = fminf(fmaxf(ceilf(st[q].mref + tp - kPOff), -128.f), 127.f);
            mprev[16 * q] = (int16_t)(((int)m & 0xff) | (prev[q] << 8));
        }
        // the model's sum over the sequence's windows: the four lane groups'
        // FP64 partials combined in FP64
        double sr = st[q].srun;
        sr += __shfl_xor(sr, 16);
        sr += __shfl_xor(sr, 32);
        const double m = __builtin_amdgcn_frexp_mant(sr) * llr[q].m;
        llr[q].e += (double)st[q].mref + (double)(__builtin_amdgcn_frexp_exp(sr) + __builtin_amdgcn_frexp_exp(m));
        llr[q].m = __builtin_amdgcn_frexp_mant(m);
        if (!LAST) {
            double x = __builtin_amdgcn_rcp(sr);
            x = fma(fma(-sr, x, 1.0), x, x);
            x = fma(fma(-sr, x, 1.0), x, x);
            const float inv = (float)x;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float4v *dst = reinterpret_cast<float4v *>(&acc[q][r][4 * mt + g][0]);
                *dst += O[q][mt] * inv;
            }
        } else if (a.sites) {
            float bv = st[q].bestv;
            int bi = st[q].besti;
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float ov = __shfl_xor(bv, o);
                const int oi = __shfl_xor(bi, o);
                if (ov > bv || (ov == bv && oi < bi)) {
                    bv = ov;
                    bi = oi;
                }
            }
            const int64_t b = bw + 16 * q + r;
            if (g == 0 && b < nvalid) a.sites[b * a.site_stride + i] = bi;
        }
    }
}

// static LDS of a workgroup and the waves per SIMD to compile for: three when
// the registers of ceil(l/4) <= 5 allow it and three workgroups' LDS (with 6 KB
// of headroom each) fit the 160 KB of a CU, else two
template <int MT, int PPB, int G>
constexpr int em_part_lds()
{
    return 2 * PPB * (int)sizeof(PairTables<MT>) + kWaves * G * 16 * Tiles<MT>::CX * 16;
}
template <int MT, int PPB, int G>
constexpr int em_static_lds()
{
    return em_part_lds<MT, PPB, G>() + 256 * (int)sizeof(uint2);
}
// LDS of one sequence's largest scores: a whole number per model
template <int G>
constexpr int kPrevBytes = kWaves * G * 16 * 2;
// Instances of up to this many sequences keep them: up to ceil(l/4) = 5 the
// workgroups of a CU leave as much LDS in every tile shape, and a limit of
// its own per shape would make results depend on the shape.
constexpr int kPrevT = 60;
template <int MT, int PPB, int G>
constexpr int em_waves_per_simd()
{
    return MT <= 5 && 3 * (em_static_lds<MT, PPB, G>() + 6 * 1024) <= 160 * 1024 ? 3 : 2;
}
// slots of the sequences, and parts of a workgroup of several: a wave per SIMD
// each, as many as the registers of ceil(l/4) allow
constexpr int em_slots(int mt, bool split) { return mt <= 5 || (mt == 6 && !split) ? 3 : 2; }

// G groups of 16 models per wave, kWaves waves per part; PARTS: several parts
template <int MT, int SRC, bool SPLIT, int PPB, int G, bool PARTS>
__global__ void __launch_bounds__((PARTS ? kPartThreads * em_slots(MT, SPLIT) : kPartThreads),
                                  (PARTS ? em_slots(MT, SPLIT) : em_waves_per_simd<MT, PPB, G>()))
k_em_mfma(const EmMfmaArgs a0)
{
    constexpr int NF = Tiles<MT>::NF, CX = Tiles<MT>::CX, MW = 16 * kWaves * G;
    typedef float Acc[kWaves][G][16][CX][4];
    __shared__ __align__(16) uint2 lut[SRC == kSrcGlobal ? 256 : 1];
    __shared__ float lbg2[4];  // log2 bg[c], formed once for every iteration's log-odds
    // per part: tables [2 PPB] and counts; then [mcap][models of the workgroup]
    extern __shared__ __align__(16) uint8_t dynlds[];
    constexpr int kPart = em_part_lds<MT, PPB, G>();
    const int parts = PARTS ? (int)(blockDim.x / kPartThreads) : 1;
    const int part = PARTS ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kPartThreads)) : 0;
    PairTables<MT> *tabs = reinterpret_cast<PairTables<MT> *>(dynlds + part * kPart);
    auto acc_of = [&](int q) -> Acc & {
        return *reinterpret_cast<Acc *>(dynlds + q * kPart + 2 * PPB * (int)sizeof(PairTables<MT>));
    };
    Acc &accs = acc_of(part);
    int16_t *prevs = reinterpret_cast<int16_t *>(dynlds + parts * kPart);

    const int wv = part_thread() >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    EmMfmaArgs a = a0;
    int64_t b0, nvalid, tb = 0;
    if (a0.inst) {
        // batch: find this workgroup's instance rank, largest r with wg_start[r] <= wg
        const PlanView pv = plan_view(a0.plan, a0.P);
        const int64_t wg = blockIdx.x;
        if (wg >= pv.wg_start[a0.P]) return;
        int lo = 0, hi = a0.P;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pv.wg_start[mid] <= wg) lo = mid;
            else hi = mid;
        }
        const int p = (int)pv.order[lo];
        const pm_inst I = a0.inst[p];
        a.packed = I.packed;
        a.offsets = I.offsets;
        a.t = I.t;
        a.nwords = (I.n_total + 15) / 16 + 4;
        tb = a0.tbase ? a0.tbase[p] : 0;
        b0 = pv.b0[p] + (wg - pv.wg_start[lo]) * MW;
        nvalid = pv.b1[p] < b0 + MW ? pv.b1[p] : b0 + MW;
    } else {
        nvalid = a.n_dev ? *a.n_dev : a.B;
        if (nvalid > a.B) nvalid = a.B;
        b0 = (int64_t)blockIdx.x * MW;
        if (b0 >= nvalid) return;  // uniform over the workgroup
    }
    const uint32_t *W = a.packed;
    const uint2 *lutp = nullptr;
    u32x4 pf[PPB];
    if constexpr (SRC == kSrcPre) {
        int L0, sl0;
        seq_slots(a, tb, part < a.t ? part : 0, L0, sl0);
        fetch_tables<MT, PPB>(a, sl0, L0, 0, pf);  // the first step of the first sweep
    } else {
        build_lut(lut);
        lutp = lut;
    }
    // by the same FP32 logarithm as the models' log2 theta, so that theta = bg
    // gives log-odds of exactly zero
    if (threadIdx.x < 4) lbg2[threadIdx.x] = __builtin_amdgcn_logf((float)a.bg[threadIdx.x]);
    __syncthreads();
    const int64_t bw = b0 + 16 * G * wv;
    float (*acc)[16][CX][4] = accs[wv];
    const int l = a.l, t = a.t, AL = 4 * l;
    const double beta = a.beta;
    int parity = 0;
    int16_t *mprev = t <= a.mcap ? prevs + 16 * G * wv + r : nullptr;
    // sum of ln L_i over the sequences
    double lnL = 0;
    for (int i = lane; i < t; i += 64) lnL += log((double)((int)(a.offsets[i + 1] - a.offsets[i]) - l + 1));
    lnL = wave_sum(lnL);
    // a step has one barrier: a part with fewer steps than another waits at the
    // barriers of those it does not have
    int idle = 0;
    if (parts > 1) {
        int mine = 0, most = 0;
        for (int q = 0; q < parts; ++q) {
            int n = 0;
            for (int i = q + parts * lane; i < t; i += 64 * parts)
                n += ((int)(a.offsets[i + 1] - a.offsets[i]) - l + 32 * PPB) / (32 * PPB);
            n = wave_sum(n);
            most = n > most ? n : most;
            mine = q == part ? n : mine;
        }
        idle = __builtin_amdgcn_readfirstlane(most - mine);
    }

    constexpr int slots = em_slots(MT, SPLIT);
    const int used = t < slots ? t : slots;  // those that hold sequences
    half16 Wb[G][Tiles<MT>::ops(SPLIT)];
    for (int it = 0; it <= a.iters; ++it) {
        const bool last = it == a.iters;
        const double *src = it == 0 ? a.theta0 : a.theta_out;
        // ---- log-odds (log2 units) of the lane's E-step B operands: model r of
        // group q, of every fragment positions 2g, 2g+1 (entries 0..7: letters 0..3
        // of both) and 8+2g, 8+2g+1 (entries 8..15), split in two FP16 halves, one
        // operand each; a repeated fragment has positions 2g, 2g+1 only, hi in
        // entries 0..7 and lo in 8..15 of one operand.  Every position is held once
        // across the four lane groups, so the prior and the lowest score are lane
        // sums over them
        double prior[G];
        float mlow[G];
        // the lane's position base goes through an empty asm statement so that
        // the index arithmetic below is formed here each iteration rather than
        // hoisted out of the loop into registers the sweeps need
        int g2 = 2 * g;
        asm volatile("" : "+v"(g2));
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int64_t b = bw + 16 * q + r;
            const bool vb = b < nvalid;
            double pr = 0;
            float wmin = 0.f;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const bool eight = Tiles<MT>::EIGHT && f == Tiles<MT>::FULL;
                half16 hi = {}, lo = {};
#pragma unroll
                for (int h = 0; h < (eight ? 2 : 4); ++h) {
                    const int p = 16 * f + 8 * (h >> 1) + g2 + (h & 1);
                    float mn = 0.f;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float w = 0.f;
                        if (p < l && vb) {
                            const double th = src[b * AL + c * l + p];
                            if (it == 0) a.theta_out[b * AL + c * l + p] = th;
                            // log2 theta by the hardware FP32 logarithm (about 2^-23
                            // relative, within what the split FP16 halves carry)
                            const float l2 = __builtin_amdgcn_logf((float)th);
                            w = l2 - lbg2[c];
                            pr += a.bg[c] * (double)l2;  // log2 units
                        }
                        mn = c == 0 ? w : fminf(mn, w);
                        const _Float16 wh = (_Float16)w;
                        hi[4 * h + c] = wh;
                        lo[4 * h + c] = (_Float16)(w - (float)wh);
                    }
                    wmin += mn;
                }
                if (eight) {
                    if (SPLIT)
#pragma unroll
                        for (int j = 0; j < 8; ++j) hi[8 + j] = lo[j];
                    Wb[q][SPLIT ? 2 * f : f] = hi;
                } else if (SPLIT) {
                    Wb[q][2 * f] = hi;
                    Wb[q][SPLIT ? 2 * f + 1 : f] = lo;
                } else {
                    Wb[q][f] = hi;
                }
            }
            pr += __shfl_xor(pr, 16);
            pr += __shfl_xor(pr, 32);
            wmin += __shfl_xor(wmin, 16);
            wmin += __shfl_xor(wmin, 32);
            prior[q] = pr * 0.6931471805599453;  // natural log
            // lowest possible score, a little below to absorb rounding
            mlow[q] = wmin - 1.0f;
        }
        LogSum ls[G];
        double mant[G];        // the earlier slots' mantissas
        uint32_t lows[G] = {};  // bit 8 + k: the model was low in slot k; bit k: when the iteration was repeated for it
        const float below = it == 1 ? kBelowFirst : kBelow;
        for (bool again = false;; again = true) {
            // ---- clear the count accumulators (own entries)
#pragma unroll
            for (int q = 0; q < G; ++q) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    *reinterpret_cast<float4v *>(&acc[q][r][4 * mt + g][0]) = float4v{0.f, 0.f, 0.f, 0.f};
                ls[q] = LogSum{0.0, 1.0};
                mant[q] = 1.0;
            }
            __syncthreads();  // tables free
            // slot by slot (the slot of sequence i is i % slots)
            for (int i = part, k = part; i < t;) {
                const bool end = i + slots >= t;  // of the slot
                const int next = !end ? i + slots : k + parts < used ? k + parts : part;
                bool known[G], low[G] = {};
#pragma unroll
                for (int q = 0; q < G; ++q) known[q] = mprev && it > 0 && !((lows[q] >> k) & 1u);
                int16_t *mp = mprev ? mprev + (int64_t)i * MW : nullptr;
                if (last)
                    sweep<MT, SRC, true, SPLIT, PPB, G>(a, W, lutp, i, bw, nvalid, tabs, parity, tb, pf, next, acc, Wb,
                                                        mlow, mp, known, below, again, low, ls);
                else
                    sweep<MT, SRC, false, SPLIT, PPB, G>(a, W, lutp, i, bw, nvalid, tabs, parity, tb, pf, next, acc, Wb,
                                                         mlow, mp, known, below, again, low, ls);
#pragma unroll
                for (int q = 0; q < G; ++q) lows[q] |= low[q] ? 256u << k : 0u;
                i = next;
                if (!end) continue;
                if (PARTS || k + 1 >= used) break;
                // ---- this slot's counts (own entries) wait in the model's rows of
                // theta_out, four letters together; the next slot's start from zero
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    const double em = ls[q].m;
                    ls[q].m = mant[q];
                    ls[q].join(em);
                    mant[q] = ls[q].m;
                    ls[q].m = 1.0;
                }
                if (!last) {
                    // (addresses formed on the spot, from an opaque thread number,
                    // rather than kept in registers that the sweeps need)
                    int u = part_thread();
                    asm volatile("" : "+v"(u));
                    #pragma unroll 1
                    for (int j = 0; j < MT * G; ++j) {
                        const int q = j / MT, p = 4 * (j % MT) + u % 64 / 16;
                        const int64_t b = b0 + u / 64 * (16 * G) + 16 * q + u % 16;
                        float4v *own = reinterpret_cast<float4v *>(&accs[u / 64][q][u % 16][p][0]);
                        if (p < l && b < nvalid)
                            reinterpret_cast<float4_in *>(a.theta_out + b * AL)[k * l + p] = *own;
                        *own = float4v{0.f, 0.f, 0.f, 0.f};
                    }
                }
                ++k;
            }
            for (int k = 0; k < idle; ++k) __syncthreads();
            // repeated at most once: the low models then start from their lowest score
            if (!mprev || it == 0 || again) break;
            bool any = false;
#pragma unroll
            for (int q = 0; q < G; ++q) {
                any |= lows[q] != 0u;
                lows[q] >>= 8;
            }
            if (!__syncthreads_or(any)) break;
        }
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const double em = ls[q].m;
            ls[q].m = mant[q];
            ls[q].join(em);
        }
        // the parts' log-likelihoods, added in order (through the tables' LDS,
        // which nobody reads any more after the barrier)
        if (parts > 1) {
            LogSum *comb = reinterpret_cast<LogSum *>(dynlds);  // [part][models of the workgroup]
            __syncthreads();
            if (g == 0) comb[part * MW + 16 * wv + r] = ls[0];
            __syncthreads();
            ls[0] = LogSum{0.0, 1.0};
            for (int q = 0; q < parts; ++q) {
                const LogSum o = comb[q * MW + 16 * wv + r];
                ls[0].e += o.e;
                ls[0].join(o.m);
            }
        }
        double llr[G];
#pragma unroll
        for (int q = 0; q < G; ++q)
            llr[q] = (ls[q].e - (double)t * (double)kPOff) * 0.6931471805599453 + log(ls[q].m) - lnL;
        // ---- objective of theta^it, then the M-step (own entries; the parts share
        // the positions)
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int64_t b = bw + 16 * q + r;
            const bool vb = b < nvalid;
            if (g == 0 && vb && part == 0) {
                a.J[b * (a.iters + 1) + it] = llr[q] + beta * prior[q];
                if (a.llr) a.llr[b * (a.iters + 1) + it] = llr[q];
            }
            if (!PARTS && !last && used > 1) {
                // the slots' counts in order; every lane of the wave has read what
                // waits in its models' rows before any writes them
                const float4_in *wait = reinterpret_cast<const float4_in *>(a.theta_out + b * AL);
                #pragma unroll 1
                for (int mt = 0; mt < MT; ++mt) {
                    const int p = 4 * mt + g;
                    if (p < l && vb) {
                        float4v cn = wait[p];
                        if (used > 2) cn += wait[l + p];
                        float4v *own = reinterpret_cast<float4v *>(&acc[q][r][p][0]);
                        *own = cn + *own;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            if (!last && vb) {
                #pragma unroll 1
                for (int mt = part; mt < MT; mt += parts) {
                    const int p = 4 * mt + g;
                    if (p < l) {
                        float4v cn = *reinterpret_cast<const float4v *>(&acc_of(0)[wv][q][r][p][0]);
                        for (int k = 1; k < parts; ++k)
                            cn += *reinterpret_cast<const float4v *>(&acc_of(k)[wv][q][r][p][0]);
                        // every column's counts sum to t: normalising by the column's
                        // own total is the same update and stays on the simplex
                        const double tot = (double)cn[0] + (double)cn[1] + (double)cn[2] + (double)cn[3] + beta;
                        #pragma unroll 1
                        for (int c = 0; c < 4; ++c)
                            a.theta_out[b * AL + c * l + p] = ((double)cn[c] + beta * a.bg[c]) / tot;
                    }
                }
            }
        }
        // theta^(it+1) visible to the lanes that read it: a lane's log-odds
        // entries were normalised by other lanes of its wave
        __syncthreads();
    }
}

// One workgroup per table slot: the one-hot tables of one window pair in the
// layout the EM kernel copies into LDS.  Batch: the slot's instance from
// tbase (first slot of every instance, ascending).  Slots past a sequence's
// last pair are left untouched; nothing reads them.
struct EmTabArgs {
    pm_inst one;           // the instance when inst is NULL
    const pm_inst *inst;   // batch instance table, or NULL
    const int64_t *tbase;  // batch: [P + 1]
    int P, l;
    int64_t nslots;        // slots of the launch
    int64_t nwords_one;    // packed words of `one` (reads are clamped below)
    uint8_t *tables;
};

template <int MT>
__global__ void __launch_bounds__(256) k_em_tables(const EmTabArgs a)
{
    __shared__ __align__(16) uint2 lut[256];
    const int64_t slot = blockIdx.x;
    if (slot >= a.nslots) return;
    pm_inst I = a.one;
    int64_t rel = slot, nw = a.nwords_one;
    if (a.inst) {
        if (slot >= a.tbase[a.P]) return;
        int lo = 0, hi = a.P;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.tbase[mid] <= slot) lo = mid;
            else hi = mid;
        }
        I = a.inst[lo];
        rel = slot - a.tbase[lo];
        nw = (I.n_total + 15) / 16 + 4;
    }
    // the sequence: largest i with seq_slot0(i) <= rel (seq_slot0 increases with i)
    int lo = 0, hi = I.t;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seq_slot0(I.offsets, mid, a.l) <= rel) lo = mid;
        else hi = mid;
    }
    const int64_t j = rel - seq_slot0(I.offsets, lo, a.l);
    const int64_t s0 = I.offsets[lo];
    const int L = (int)(I.offsets[lo + 1] - s0) - a.l + 1;
    if (32 * j >= L) return;  // uniform over the workgroup
    build_lut(lut);
    __syncthreads();
    build_tables<MT, true>(I.packed, nw, s0 + 32 * j, lut, reinterpret_cast<PairTables<MT> *>(a.tables)[slot]);
}

static size_t pair_table_bytes(int mt) { return 1024 + (size_t)(4 * mt + 12) * 64; }
static_assert(sizeof(PairTables<1>) == 1024 + 16 * 64 && sizeof(PairTables<8>) == 1024 + 44 * 64, "table size");

static int launch_em_tables(const EmTabArgs &t, hipStream_t st)
{
    if (t.nslots < 1) return PM_OK;
    switch ((t.l + 3) / 4) {
    case 1: hipLaunchKernelGGL(k_em_tables<1>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    case 2: hipLaunchKernelGGL(k_em_tables<2>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    case 3: hipLaunchKernelGGL(k_em_tables<3>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    case 4: hipLaunchKernelGGL(k_em_tables<4>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    case 5: hipLaunchKernelGGL(k_em_tables<5>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    case 6: hipLaunchKernelGGL(k_em_tables<6>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    case 7: hipLaunchKernelGGL(k_em_tables<7>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    default: hipLaunchKernelGGL(k_em_tables<8>, dim3((unsigned)t.nslots), dim3(256), 0, st, t); break;
    }
    PM_LAUNCHED();
    return PM_OK;
}

static int64_t seqs_slots(const pm_seqs *S, int l) { return em_inst_slots(S->t, S->n_total - (int64_t)S->t * (l - 1)); }

size_t em_tables_workspace(const pm_seqs *S, int32_t l)
{
    return (size_t)seqs_slots(S, l) * pair_table_bytes((l + 3) / 4);
}

// precomputed tables of one instance into ws (checked size), a.tables set
static int prepare_tables(EmMfmaArgs &a, const pm_seqs *S, int l, void *ws, size_t ws_bytes, hipStream_t st)
{
    a.tables = nullptr;
    if (!ws) return PM_OK;
    const size_t need = em_tables_workspace(S, l);
    if (ws_bytes < need) return fail(PM_EINVAL, "workspace of %zu bytes, the one-hot tables need %zu", ws_bytes, need);
    if (((uintptr_t)ws & 15) != 0) return fail(PM_EINVAL, "workspace must be 16-byte aligned");
    EmTabArgs t{};
    t.one.offsets = S->offsets;
    t.one.packed = S->packed;
    t.one.n_total = S->n_total;
    t.one.t = S->t;
    t.l = l;
    t.nslots = seqs_slots(S, l);
    t.nwords_one = pm_packed_words(S->alphabet, S->n_total);
    t.tables = static_cast<uint8_t *>(ws);
    const int rc = launch_em_tables(t, st);
    if (rc != PM_OK) return rc;
    a.tables = t.tables;
    return PM_OK;
}

constexpr int kCUs = 256;

// Parts of a launch's workgroups: the slots side by side where every CU has a
// workgroup of 64 models at most, else one.  16 384 models of the (21,7)
// workload in single FP16, one workgroup per CU: 6.3 ms in one part, 3.8 in
// three; just above (16 500 to 24 500 models, 3 iterations) 5.7 ms in one part
// against 6.1 in two, and on (18,6) in split FP16 1.55 against 1.65.  Where the
// number of models is on the device, or an instance's last workgroup may be
// partly filled, the capacity may be more than there is: up to twice as much
// still goes in parts, which cost 0 to 6% if it is full ((18,6): two rounds of
// 0.81 ms against 1.52 to 1.64 in one part) and take half the time if it is not.
static int em_parts(const EmMfmaArgs &a)
{
    const int slots = em_slots((a.l + 3) / 4, a.split != 0);
    if (em_groups(a, 16 * kWaves) > (a.inst || a.n_dev ? 2 * kCUs : kCUs)) return 1;
    return a.site_stride < slots ? a.site_stride : slots;
}

template <int MT, bool SPLIT, int PPB, int G, bool PARTS = false>
static int launch_em_mfma(const EmMfmaArgs &a, hipStream_t st)
{
    const int64_t groups = em_groups(a, 16 * kWaves * G);
    EmMfmaArgs b = a;
    b.mcap = a.site_stride < kPrevT ? a.site_stride : kPrevT;  // site_stride: the most sequences of an instance
    const int parts = PARTS ? em_parts(a) : 1;  // (PARTS: launch_shape has seen more than one)
    const size_t lds = (size_t)parts * em_part_lds<MT, PPB, G>() + (size_t)b.mcap * kPrevBytes<G>;
    const dim3 grid((unsigned)groups), block(kPartThreads * parts);
    auto kernel = a.tables ? k_em_mfma<MT, kSrcPre, SPLIT, PPB, G, PARTS> : k_em_mfma<MT, kSrcGlobal, SPLIT, PPB, G, PARTS>;
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, grid, block, lds, st, b);
    PM_LAUNCHED();
    return PM_OK;
}

// tile shape in use per (ceil(l/4) - 1, split), coded 10 G + PPB; 0 = untuned.
// With kShapeSet: set by the caller, and taken by every launch
static int g_shape[8][2];
constexpr int kShapeSet = 256;

static int &shape_of(int l, bool split) { return g_shape[(l + 3) / 4 - 1][split ? 1 : 0]; }

static bool shape_ok(int shape, int l)
{
    const int G = shape / 10, ppb = shape % 10;
    return (ppb == 1 || ppb == 2 || ppb == 4) && (G == 1 || (G == 2 && (l + 3) / 4 <= kMaxMT2));
}

static int tuned_shape(int l, bool split)
{
    const int v = shape_of(l, split) & ~kShapeSet;
    return v ? v : kShapeDefault;
}

template <bool SPLIT, int PPB, int G, bool PARTS = false>
static int dispatch_mt(const EmMfmaArgs &a, hipStream_t st)
{
    switch ((a.l + 3) / 4) {
    case 1: return launch_em_mfma<1, SPLIT, PPB, G, PARTS>(a, st);
    case 2: return launch_em_mfma<2, SPLIT, PPB, G, PARTS>(a, st);
    case 3: return launch_em_mfma<3, SPLIT, PPB, G, PARTS>(a, st);
    case 4: return launch_em_mfma<4, SPLIT, PPB, G, PARTS>(a, st);
    case 5: return launch_em_mfma<5, SPLIT, PPB, G, PARTS>(a, st);
    case 6: return launch_em_mfma<6, SPLIT, PPB, G, PARTS>(a, st);
    case 7: if (G == 1) return launch_em_mfma<7, SPLIT, PPB, 1, PARTS>(a, st); break;
    default: if (G == 1) return launch_em_mfma<8, SPLIT, PPB, 1, PARTS>(a, st); break;
    }
    return fail(PM_EINVAL, "tile shape with %d model groups per wave needs l <= %d", G, 4 * kMaxMT2);
}

template <bool SPLIT>
static int dispatch_shape(const EmMfmaArgs &a, hipStream_t st, int shape)
{
    switch (shape) {
    case kShapeParts: return dispatch_mt<SPLIT, kPartsPPB, 1, true>(a, st);
    case 11: return dispatch_mt<SPLIT, 1, 1>(a, st);
    case 12: return dispatch_mt<SPLIT, 2, 1>(a, st);
    case 14: return dispatch_mt<SPLIT, 4, 1>(a, st);
    case 21: return dispatch_mt<SPLIT, 1, 2>(a, st);
    case 22: return dispatch_mt<SPLIT, 2, 2>(a, st);
    default: return dispatch_mt<SPLIT, 4, 2>(a, st);
    }
}

// the tile shape a launch runs in: in parts where those pay, unless the caller
// has set a shape; else the recorded one
static int launch_shape(const EmMfmaArgs &a)
{
    if (!(shape_of(a.l, a.split != 0) & kShapeSet) && em_parts(a) > 1) return kShapeParts;
    const int shape = tuned_shape(a.l, a.split != 0);
    return shape_ok(shape, a.l) ? shape : 10 + shape % 10;
}

static int dispatch_em_mfma(const EmMfmaArgs &a, hipStream_t st, int shape)
{
    return a.split ? dispatch_shape<true>(a, st, shape) : dispatch_shape<false>(a, st, shape);
}

int em_refine_mfma(const pm_seqs *S, int32_t l, const double *theta0, const double *bg, int64_t B,
                   const int64_t *n_dev, int32_t iters, double beta, double *theta_out, double *J_out,
                   double *llr_out, int32_t *sites_out, void *ws, size_t ws_bytes, bool split, hipStream_t st)
{
    EmMfmaArgs a{};
    a.split = split;
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
    a.nwords = pm_packed_words(S->alphabet, S->n_total);
    a.t = S->t;
    a.site_stride = S->t;
    a.l = l;
    a.iters = iters;
    a.beta = beta;
    const int rc = prepare_tables(a, S, l, ws, ws_bytes, st);
    if (rc != PM_OK) return rc;
    return dispatch_em_mfma(a, st, launch_shape(a));
}

// One workgroup: each instance's bucket range (buckets ascend by item), its
// workgroup count, the largest-first order of the instances and the scan of
// the counts in that order.
__global__ void __launch_bounds__(1024) k_em_plan(const pm_inst *inst, int P, const pm_bucket *buckets,
                                                 const int64_t *n_dev, int64_t Bcap, int mw, int64_t *plan,
                                                 int64_t *tbase)
{
    const PlanView pv = plan_view(plan, P);
    int64_t *wg_start = const_cast<int64_t *>(pv.wg_start), *b0 = const_cast<int64_t *>(pv.b0);
    int64_t *b1 = const_cast<int64_t *>(pv.b1), *order = const_cast<int64_t *>(pv.order);
    int64_t nvalid = n_dev ? *n_dev : Bcap;
    if (nvalid > Bcap) nvalid = Bcap;
    // bucket range of every instance: first bucket whose item is >= first_item
    for (int p = threadIdx.x; p < P; p += 1024) {
        for (int side = 0; side < 2; ++side) {
            const int64_t item = (int64_t)inst[p].first_item + (side ? inst[p].m : 0);
            int64_t lo = 0, hi = nvalid;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if ((int64_t)buckets[mid].trial < item) lo = mid + 1;
                else hi = mid;
            }
            (side ? b1 : b0)[p] = lo;
        }
    }
    // rank by windows, descending, ties by index
    for (int p = threadIdx.x; p < P; p += 1024) {
        const int64_t xp = inst[p].x;
        int r = 0;
        for (int q = 0; q < P; ++q) {
            const int64_t xq = inst[q].x;
            r += (xq > xp || (xq == xp && q < p)) ? 1 : 0;
        }
        order[r] = p;
    }
    __syncthreads();
    // exclusive scan of the workgroup counts in rank order (serial: P is small)
    if (threadIdx.x == 0) {
        int64_t run = 0;
        for (int r = 0; r < P; ++r) {
            wg_start[r] = run;
            const int p = (int)order[r];
            run += (b1[p] - b0[p] + mw - 1) / mw;
        }
        wg_start[P] = run;
        // first precomputed-table slot of every instance, in instance order
        if (tbase) {
            int64_t sl = 0;
            for (int p = 0; p < P; ++p) {
                tbase[p] = sl;
                sl += em_inst_slots(inst[p].t, inst[p].x);
            }
            tbase[P] = sl;
        }
    }
}

// batch workspace: the plan, the instances' first table slots, the tables
static size_t plan_bytes(int32_t P) { return ((size_t)(4 * (int64_t)P + 1) * sizeof(int64_t) + 255) / 256 * 256; }
static size_t tbase_bytes(int32_t P) { return ((size_t)(P + 1) * sizeof(int64_t) + 255) / 256 * 256; }
static int64_t batch_slots(const pm_batch *Bt)
{
    int64_t sl = 0;
    for (int p = 0; p < Bt->P; ++p) sl += em_inst_slots(Bt->inst_host[p].t, Bt->inst_host[p].x);
    return sl;
}

size_t em_batch_workspace(const pm_batch *Bt, bool tables)
{
    if (Bt->P < 1) return 0;
    size_t n = plan_bytes(Bt->P) + tbase_bytes(Bt->P);
    if (tables) n += (size_t)batch_slots(Bt) * pair_table_bytes((Bt->l + 3) / 4);
    return n;
}

int em_refine_mfma_batch(const pm_batch *Bt, int64_t nw_max, int t_max, const pm_bucket *buckets,
                         const double *theta0, const double *bg, int64_t B, const int64_t *n_dev, int32_t iters,
                         double beta, double *theta_out, double *J_out, double *llr_out, int32_t *sites_out,
                         void *ws, bool split, hipStream_t st)
{
    uint8_t *w = static_cast<uint8_t *>(ws);
    int64_t *plan = reinterpret_cast<int64_t *>(w);
    int64_t *tbase = reinterpret_cast<int64_t *>(w + plan_bytes(Bt->P));
    uint8_t *tables = w + plan_bytes(Bt->P) + tbase_bytes(Bt->P);
    EmMfmaArgs a{};
    a.split = split;
    a.inst = Bt->inst;
    a.plan = plan;
    a.P = Bt->P;
    a.tables = tables;
    a.tbase = tbase;
    a.theta0 = theta0;
    a.bg = bg;
    a.n_dev = n_dev;
    a.theta_out = theta_out;
    a.J = J_out;
    a.llr = llr_out;
    a.sites = sites_out;
    a.B = B;
    a.site_stride = t_max;
    a.l = Bt->l;
    a.iters = iters;
    a.beta = beta;
    const int shape = launch_shape(a);
    hipLaunchKernelGGL(k_em_plan, dim3(1), dim3(1024), 0, st, Bt->inst, Bt->P, buckets, n_dev, B,
                       16 * kWaves * shape_groups(shape), plan, tbase);
    PM_LAUNCHED();
    EmTabArgs tt{};
    tt.inst = Bt->inst;
    tt.tbase = tbase;
    tt.P = Bt->P;
    tt.l = Bt->l;
    tt.nslots = batch_slots(Bt);
    tt.tables = tables;
    const int rc = launch_em_tables(tt, st);
    if (rc != PM_OK) return rc;
    (void)nw_max;
    // every instance wastes at most one partly filled group
    return dispatch_em_mfma(a, st, shape);
}

int em_autotune_mfma(const pm_seqs *S, int32_t l, const double *theta0, const double *bg, int64_t B, int32_t iters,
                     double beta, bool split, double *theta_out, double *J_out, void *ws, size_t ws_bytes,
                     int32_t *choice, hipStream_t st)
{
    EmMfmaArgs a{};
    a.split = split;
    a.packed = S->packed;
    a.offsets = S->offsets;
    a.theta0 = theta0;
    a.bg = bg;
    a.theta_out = theta_out;
    a.J = J_out;
    a.B = B;
    a.nwords = pm_packed_words(S->alphabet, S->n_total);
    a.t = S->t;
    a.site_stride = S->t;
    a.l = l;
    a.iters = iters;
    a.beta = beta;
    const int prc = prepare_tables(a, S, l, ws, ws_bytes, st);
    if (prc != PM_OK) return prc;
    hipEvent_t e0, e1;
    PM_TRY(hipEventCreate(&e0));
    PM_TRY(hipEventCreate(&e1));
    float best_ms = 0.f;
    int best = 0, rc = PM_OK;
    for (const int shape : {11, 12, 14, 21, 22, 24}) {
        if (!shape_ok(shape, l)) continue;
        float ms = 0.f;
        rc = dispatch_em_mfma(a, st, shape);  // warm-up
        if (rc == PM_OK && hipEventRecord(e0, st) != hipSuccess) rc = fail(PM_EDEVICE, "hipEventRecord failed");
        if (rc == PM_OK) rc = dispatch_em_mfma(a, st, shape);
        if (rc == PM_OK && hipEventRecord(e1, st) != hipSuccess) rc = fail(PM_EDEVICE, "hipEventRecord failed");
        if (rc == PM_OK && hipEventSynchronize(e1) != hipSuccess) rc = fail(PM_EDEVICE, "hipEventSynchronize failed");
        if (rc == PM_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = fail(PM_EDEVICE, "hipEventElapsedTime failed");
        if (rc != PM_OK) break;
        if (best == 0 || ms < best_ms) {
            best = shape;
            best_ms = ms;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != PM_OK) return rc;
    shape_of(l, split) = best;
    if (choice) *choice = best;
    return PM_OK;
}

int em_tuned_shape(int32_t l, bool split) { return tuned_shape(l, split); }

int em_record_shape(int32_t l, bool split, int32_t shape)
{
    if (!shape_ok(shape, l))
        return fail(PM_EINVAL, "tile shape %d is not one of 11, 12, 14, 21, 22, 24 (G = 2 needs l <= %d)", shape,
                    4 * kMaxMT2);
    shape_of(l, split) = shape | kShapeSet;
    return PM_OK;
}


}  // namespace pm
