// The label-looping decoder (paper Algorithm 3, Sec. 3.2; TDT Sec. 3.3) as a chain of
// exchanges: two for the predictor side of a label, one for every joint pass.  decode.hip holds the
// general kernel and explains the phases P (predictor step), Q (products with the new predictor state),
// J (joint pass) and D (decision); this one runs the same phases for the default loops (label-looping,
// precomputed projections) of groups of at most kLabelMaxHyps hypotheses with reductions of the compiled
// lengths (label_form), and is built for the length of the chain: an exchange between workgroups is about
// 1.4 us whatever it carries, so what matters is how many dependent steps there are between them and how
// few instructions each takes.  Config 2 at B = 32, a label with one joint pass, microseconds by a time line
// of one workgroup: P 0.7; the pass set up while the hidden state travels 0.9, and 0.8 until it is there; Q
// 1.1; on to the joint pass 0.5, and 0.6 until the projected output is there; J 2.9; cells gathered 1.1; D 1.6
// with the top of the next label (10.2 with the time stamps; about 8 a label without).
//
//   * No barriers between workgroups.  Every exchanged word says itself whether it is there: rows
//     of the hidden state and of the projected predictor output start out as a bit pattern that no
//     result has, argmax / softmax cells as zero.  A reader loads what it needs and loads it again
//     until all of it is there, so data and "it is complete" travel together (measured for 32
//     workgroups all exchanging 10 KB: 1.45 us against 2.08 us with flags that are polled before
//     the data is loaded).  Words are put back by their writer once everybody has read them; see
//     "Reuse of the exchange buffers" below.
//   * A workgroup owns its column tiles of the predictor-side matrices for the whole call.  The four
//     gates of a unit meet in the workgroup that updates the unit's cell, so the recurrent
//     pre-activations and the cell state never leave its LDS; only h is exchanged (bfloat16, one layer: as the three terms its
//     readers multiply, split once by whoever updates the cell).
//   * A group's hypotheses wait for each other's searches only until enough of them do: half, without a predictor a third, with
//     deeper LSTMs two thirds or four fifths (see "patience").
//   * The control state of a hypothesis (frame, label count, last labels, score ...) lives in lane g
//     of every wavefront, the lists of active and searching hypotheses are 64-bit masks: a decision
//     is taken by every wavefront on its own, without a workgroup barrier or LDS list.
//   * Four wavefronts a workgroup, one per SIMD.  What a label costs beside the exchanges is the number
//     of instructions in a row, and two wavefronts that share a SIMD take turns at them.  It also
//     leaves 512 registers a lane, and the weights stay in them: those of phase Q for the whole call (one
//     layer; float32's longest form with two rounds: the first), those of a joint pass while its work
//     items cover the same column tiles, which a group's plans seldom change (stateless, and one layer but
//     for two rounds in bfloat16).  Scalar registers are short: 100 to 400 scalar values of a form are
//     kept in lanes of vector registers and moved back where they are used.
//   * Every wavefront multiplies its own quarter of the reduction for all column tiles.  So no two
//     wavefronts need the same activation: each loads and waits for its quarter of the rows, and
//     only the partial sums are shared (rows staged in LDS for all wavefronts, with the barrier that
//     takes: config 2 at B = 1 648 us against 610; stateless at B = 128 3.11 ms against 2.70).  Where there is
//     one LSTM layer or none, a wavefront's rows of a joint pass change lanes through LDS of its own (stages_rows) and are
//     split between the products of the step before (split_and_multiply); so do rows of the hidden state in float32, while in
//     bfloat16 with one layer they arrive as the operands they are multiplied as (plane_base).
//
// Reuse of the exchange buffers.  Every workgroup of a group publishes something in every joint
// exchange (a workgroup without work item: a word of its own that everybody waits for), after it
// has finished reading all earlier exchanges.  So a workgroup that has read joint exchange j knows
// what all others have read, and puts its own words of that back.  The stores complete before it publishes joint
// exchange j + 1 (every wavefront waits for its stores before the workgroup barrier that precedes
// publishing), and the next readers of those words come only behind that exchange.  What is known to have been read:
//   * Cells: those of joint exchange j - 2 (those of j - 1 not for certain: the score terms found in it are summed while
//     j's cells travel).  They rotate through four buffers.
//   * Rows of the hidden state: this predictor step's.  They alternate between two buffers by step.
//   * Projected rows where LDS has two areas (one layer, not OWN): this step's, which alternate by step as well.  Every workgroup
//     stages the rows of those who took the step before it publishes the step's first joint exchange -- a workgroup without a work item,
//     too, though it has no use for them in that pass: a hypothesis that goes on searching is scored behind later steps,
//     with the row it has, by workgroups that may have had no item until then, and by that time the row is put back.  (Where
//     nobody goes on early, `patience` zero, every row belongs to the step at hand and stays until it ends.)
//   * Projected rows of the other LSTM forms (OWN), which are read in every pass: a hypothesis' own last one.  It stays through
//     as many steps of others as the hypothesis searches; which of the two buffers it is in is kept per hypothesis (`own`), and
//     it is put back while the hypothesis' next one is made, since all have read it in the pass that found the label.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "tdt_internal.h"
#include "decode_state.h"
#include "exchange.h"
#include "split.h"
#include "tile_gemm.h"
#include "terms.h"

namespace tdt {
namespace {

constexpr unsigned kAbsent = 0xffffffffu;   // an exchanged float that is not there yet (a NaN no result is stored as)
constexpr int kWidePart = 2 * (4 * CT + 8);       // WIDE: floats per wavefront and row of a tile in the partial sums, at least (all uses)
constexpr int kWideTiles = 16;                    // ... column tiles of the predictor side with a place there, at most
constexpr int wide_part(int tiles) { return tiles * CT + 4 > kWidePart ? tiles * CT + 4 : kWidePart; }
constexpr int wide_tiles(int part) { return (part - 4) / CT; }
static_assert(kNowhere >= 2ll * TDT_MAX_LSTM_LAYERS * kMaxGrid * kLabelMaxHyps * kLabelLongest * 4, "the largest exchange buffer");
constexpr int kPackRows = 4;                // up to this many rows the three planes of a tile share its 16 rows
constexpr int kPairRows = 8;                // up to this many rows two planes do (one LSTM layer)
static_assert(plane_rows(kPackRows) == kPackRows && plane_rows(kPairRows) == kPairRows, "planes");

typedef unsigned v4u __attribute__((ext_vector_type(4)));

// What differs between the element types: a fragment is 1 KiB = 16 columns x KS inputs, E of them a lane.
// The product of 16 rows and 16 columns is formed with the weights as the left operand: lane l then
// holds four neighbouring columns, (l / 16) * 4 .. + 3, of row l % 16.
template <typename WT> struct Frags;
template <> struct Frags<uint16_t> {
    static constexpr int KS = 32, E = 8, PL = 3;
    typedef bf16x8 A;
    __device__ static f32x4 mma(const A &a, const v4u &b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(&b), a, c, 0, 0, 0);
    }
};
template <> struct Frags<float> {
    static constexpr int KS = 16, E = 4, PL = 1;
    typedef f32x4 A;
    __device__ static f32x4 mma(const A &a, const v4u &b, f32x4 c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b.x), a.x, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b.y), a.y, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b.z), a.z, c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b.w), a.w, c, 0, 0, 0);
    }
};

__device__ inline float present(float v) { return __float_as_uint(v) == kAbsent ? __uint_as_float(0x7fc00000u) : v; }
__device__ inline void st_co32(int *p, int v) { __hip_atomic_store((TDT_GLOBAL int *)p, v, __ATOMIC_RELAXED, TDT_AGENT); }
__device__ inline void st_co4(float *p, float4 v)   // two 8-byte stores of agent scope
{
    unsigned long long *q = reinterpret_cast<unsigned long long *>(p);
    st_co64(q, (unsigned long long)__float_as_uint(v.x) | ((unsigned long long)__float_as_uint(v.y) << 32));
    st_co64(q + 1, (unsigned long long)__float_as_uint(v.z) | ((unsigned long long)__float_as_uint(v.w) << 32));
}
// Buffer descriptor of `bytes` bytes of device memory from `base` on, the same in every lane.  A load
// then takes a lane offset and a scalar offset, so that the addresses of many loads of one array
// cost one scalar addition each; reads beyond the end give zeros.
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *base, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
__device__ inline float4 as_float4(v4u v)
{
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ inline unsigned umax4(v4u v) { return max(max(v.x, v.y), max(v.z, v.w)); }
// agent scope: what another workgroup writes (see ld_co4)
__device__ inline v4u ldx4(__amdgpu_buffer_rsrc_t rs, int lane_off, int off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(rs, lane_off, off, 16 /* sc1 */);
}
// what no workgroup writes while the kernel runs
__device__ inline v4u ldg4(const float *row, int off)
{
    return *(const TDT_GLOBAL v4u *)(reinterpret_cast<const char *>(row) + (unsigned)off);
}
// Gives registers a value without an instruction.  An array of which a pass fills only a part needs it:
// what is not filled would otherwise be the value of the pass before, held in registers all the way.
template <typename T, int N> __device__ inline void any_value(T (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "=v"(x[i]));
}
template <typename T, int M, int N> __device__ inline void any_value(T (&x)[M][N])
{
#pragma unroll
    for (int i = 0; i < M; ++i) any_value(x[i]);
}
template <typename T, int M, int N> __device__ inline void any_acc(T (&x)[M][N])
{
#pragma unroll
    for (int i = 0; i < M * N; ++i) asm volatile("" : "=a"(x[i / N][i % N]));
}
// a value the compiler must not compute ahead of the loop it is used in (it would be kept, and
// spilled, through the whole label loop for the sake of an addition)
__device__ inline int here(int v)
{
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
}
// Reductions over the 16 lanes of a row, in all of them: a rotation is an operand's, so a step is one instruction
// (with row_allreduce five: copy, move across lanes, canonicalise) and the two wait states ahead of it.
#define TDT_ROW_STEPS(op)                                                          \
    "s_nop 1\n\t" op " %0, %0, %0 row_ror:1 row_mask:0xf bank_mask:0xf\n\t"       \
    "s_nop 1\n\t" op " %0, %0, %0 row_ror:2 row_mask:0xf bank_mask:0xf\n\t"       \
    "s_nop 1\n\t" op " %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"       \
    "s_nop 1\n\t" op " %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf"
__device__ inline float row_max(float v)
{
    asm(TDT_ROW_STEPS("v_max_f32_dpp") : "+v"(v));
    return v;
}
__device__ inline float row_sum(float v)
{
    asm(TDT_ROW_STEPS("v_add_f32_dpp") : "+v"(v));
    return v;
}
__device__ inline int row_min(int v)
{
    asm(TDT_ROW_STEPS("v_min_i32_dpp") : "+v"(v));
    return v;
}
// sum over the lanes that share l % 32, in both
__device__ inline float sum_over_halves(float v)
{
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}
// sum / maximum over the lanes that share l % 16, in all of them
__device__ inline float sum_over_rows(float v)
{
    auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}
__device__ inline unsigned long long max_over_rows(unsigned long long v)
{
    auto lo = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(v >> 32), (unsigned)(v >> 32), false, false);
    unsigned long long a = lo[0] | ((unsigned long long)hi[0] << 32), b = lo[1] | ((unsigned long long)hi[1] << 32);
    v = a > b ? a : b;
    lo = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    hi = __builtin_amdgcn_permlane32_swap((unsigned)(v >> 32), (unsigned)(v >> 32), false, false);
    a = lo[0] | ((unsigned long long)hi[0] << 32);
    b = lo[1] | ((unsigned long long)hi[1] << 32);
    return a > b ? a : b;
}
// 1 / (1 + exp(-x)) on the hardware exponential and reciprocal, the latter with one Newton step.  The
// exponential is kept finite, so that the step sees no infinity, by the minimum that hands a NaN on
// (v_minimum3_f32: one instruction, like the one that does not).  Error against 64 bits over 4 million
// points of [-90, 90]: 9.2e-8 absolute at most, 1.87e-8 rms, the same as with a correctly rounded reciprocal.
__device__ inline float sigmoid(float x)
{
    const float d = 1.0f + __builtin_elementwise_minimum(__expf(-x), 1e38f), r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(-d, r, 1.0f), r, r);
}

// ---- Rows on their way to the matrix cores (stages_rows: one LSTM layer or stateless, four wavefronts).  A wavefront
// multiplies its own stretch of the reduction of all 16 rows, and lane l feeds part l / 16 of row l % 16.
// Loaded like that, 16 lanes in a row ask for 16 different rows, and a compute unit takes in one 64-byte
// piece a clock: 1.1 us for the 40 KB of 16 rows of 640 floats, twice or three times in every pass (rows
// of the encoder, of the projected predictor output, in float32 of the hidden state).  Eight lanes on 128 bytes of a row
// are four times as fast (0.33 us; 4 wavefronts x 10 loads of 16 bytes a lane, 256 workgroups, all from L2).
// So rows are loaded that way and change lanes through LDS, in an area of the wavefront's own: no barrier.
// With the split between the products below, one case timed alone on both sides: stateless at B = 128 2.74 -> 2.42
// ms, config 2 at B = 32 1.53 -> 1.47 ms, at B = 128 2.51 -> 2.39 ms, config 3 at B = 32 0.62 -> 0.59 ms.
constexpr bool stages_rows(int layers, int nw) { return layers < 2 && nw == 4; }
constexpr int staged_row(int nk, int ks) { return nk * ks + 4; }   // floats (padded: 16 rows start in 16 different banks)
// a second area for the predictor's rows, which then stay from pass to pass of a label
constexpr bool two_areas(int nk, int ks) { return nk * ks <= 160; }
__host__ __device__ constexpr int pred_area_rows(int layers, int hyps_per_cluster) { return layers == 1 && hyps_per_cluster <= 8 ? 8 : 16; }

// how a joint pass with n searching hypotheses is cut (tabulated per n when the kernel starts)
struct LabelPlan {
    short Kw, n_tiles, n_cg, tpg;
    int rcp_kw;
    short ti0, cg0;   // this workgroup's first work item
};

struct LabelShared {
    LabelPlan plan[kLabelMaxHyps + 1];
    unsigned long long rowb[kLabelRowsPerPass];    // best label of each row (or shares of it, see the gather)
    unsigned long long rowd[kLabelRowsPerPass];    // frame step of the best duration class of each row
    unsigned long long rowl[kLabelRowsPerPass];    // softmax share of each row (groups of one workgroup only)
    int res_a[kLabelRowsPerPass], res_d[kLabelRowsPerPass];   // passes of more than 64 rows: label, frame step
    int gid[kLabelMaxHyps];
    int durations[TDT_MAX_DURATIONS];
    int aborted;
    long long tk[5], tk_last, tk_start;   // profiling builds: P, Q, J, D, waits
};

// LAYERS: 0: stateless predictor; 1: one LSTM layer, a workgroup's column tiles fit one round and the
// group one row tile (every thread then has fixed places to write its results to); 2: any LSTM.
// NW: wavefronts.  Four, or (WIDE) eight for output layers of many thousands of columns, see wide_rows.
// TQ: column tiles of a round of the predictor-side products; stateless: of a joint pass's first round; eight wavefronts: those of the
// one round of one layer (wide_round), or the steps of the predictor's reduction, whose column tiles then are lists.
// QROWS: most rows of the hidden state that are multiplied at once (kPairRows: see few_products).
template <typename WT, int LAYERS, bool CHUNKED, int NK, int NW, int TQ, int QROWS>
__global__ __launch_bounds__(NW * 64, NW / 4) void label_kernel(DecodeParams p)
{
    typedef Frags<WT> F;
    typedef typename F::A AFrag;
    constexpr int PL = F::PL, KS = F::KS, NL = F::E / 4;   // NL: 16-byte loads of float32 for a lane's part of a step
    constexpr bool LSTM = LAYERS > 0, DEEP = LAYERS > 1, WIDE = NW == 8;
    constexpr int THREADS = NW * 64;
    constexpr int kClearer = NW - 2;                          // the wavefront that puts cells back (the last one sums scores meanwhile)
    constexpr int TR = label_tiles(NK);                       // column tiles per round of a joint pass
    constexpr int TJ = LAYERS == 0 && !WIDE ? TQ : TR;        // ... per its first round
    constexpr int JH = TJ > 4 ? 2 : 1;                        // which is looked at four tiles, four columns a thread, at a time
    constexpr int QPR = THREADS / RT;                         // threads that share a row of a round, four columns each
    constexpr bool LISTS = WIDE && LSTM && TQ <= NK;          // eight wavefronts, the predictor's column tiles as lists
    static_assert(!WIDE || (LAYERS != 1 && (!LSTM || LISTS || TQ * CT <= QPR * 4)), "eight wavefronts: any LSTM or none, a round is one pass of the threads");
    constexpr bool ONE_ROUND = WIDE && LSTM && !LISTS;        // ... one layer and one round of them (wide_round)
    constexpr int NQ = LISTS ? TQ : NK;                       // steps of the predictor's reduction
    constexpr int PLQ = TQ * CT + 4, PLJ = TJ * CT + 4;   // floats per row of the partial sums (padded: 16 rows, 64 banks)
    constexpr int KI = (NK * NW * KS + 255) / 256;  // 16-byte loads per lane for a whole row
    constexpr bool STAGED = stages_rows(LAYERS, NW);          // rows go through LDS, see stage_rows
    constexpr int C32 = NK * KS / 32, LDX = staged_row(NK, KS);   // 128-byte pieces of a wavefront's stretch of a row, floats of a staged row
    constexpr bool TWO = two_areas(NK, KS);
    constexpr bool TWO_ROUNDS = LAYERS == 1 && TQ > TR;       // phase Q has two rounds
    // Weights of a joint pass's later rounds have registers of their own, and a thread asks for all its partial sums at
    // once.  Not in deeper LSTMs, which keep no weights and where both cost (two layers, bfloat16, B = 32, 1760 us,
    // without 1727; float32, reductions to 64, B = 12, 448, 441) -- but for float32's longest form (1853, 1890) --
    // nor, the registers, where phase Q's second round has them (see "Weights that stay").
    constexpr bool OWN2 = DEEP ? PL == 1 && NK > 4 : !(TWO_ROUNDS && PL == 3);
    // Hypotheses that have found a label need not wait for all that search, see "patience".  Not with float32's
    // shortest reductions, whose small models have long windows (the smallest benchmark model 150 us a call, with it 155).
    constexpr bool MERGES = !(PL == 1 && NK <= 4);
    // Rows of the projected predictor output are read from the exchange buffers in every pass (where there are two
    // areas they stay staged), so a row stays there until its hypothesis' next one: see "own".
    constexpr bool OWN = LSTM && !(LAYERS == 1 && TWO);
    constexpr bool PLANES = PL == 3 && LAYERS == 1;   // the hidden state travels as its terms, see plane_base
    constexpr bool FEW = QROWS < RT;                  // ... float32: see few_products
    static_assert(!FEW || (PL == 1 && LAYERS == 1 && QROWS == kPairRows), "few_products");
    constexpr bool EARLY_GATES = LAYERS == 1 && (PL == 3 || FEW || !CHUNKED);   // see request_gates
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    __shared__ LabelShared S;

    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Called where a phase starts: what the phase derives from the thread's index is computed there.
    // Without it the compiler computes all of it once ahead of the label loop, a hundred registers that
    // it then spills.
    auto fresh = [&]() __attribute__((always_inline)) {
        asm volatile("" : "+v"(tid));
        lane = tid & 63;
    };
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int ncl = p.n_clusters;
    const int C = gridDim.x / ncl;
    // which group, and which place in it: as in decode.hip, every die hosts the same ranks of
    // every group, so that its L2 keeps the columns those ranks multiply by
    int cl, rank;
    if (gridDim.x % kXcds == 0) {
        const int die = blockIdx.x % kXcds, j = blockIdx.x / kXcds;
        const int per = (int)(gridDim.x / kXcds) / ncl;
        if (j < per * ncl) {
            cl = j % ncl;
            rank = die * per + j / ncl;
        } else {
            const int e = (j - per * ncl) * kXcds + die;
            if (e >= ncl * (C - kXcds * per)) return;   // an empty slot: not part of any group
            cl = e % ncl;
            rank = kXcds * per + e / ncl;
        }
    } else {
        cl = blockIdx.x % ncl;
        rank = blockIdx.x / ncl;
    }
    const int B = p.B, T = p.T, H = p.H, V = p.V, D = p.D, O = p.O, VL = p.VL;
    const bool big_blanks = p.multi_blank != 0;
    const int hpc = p.hyps_per_cluster, b0 = cl * hpc, Bw = ncl * hpc;
    // the group's hypotheses: dealt by length, longest first, as in decode.hip
    const bool ranked = ncl > 1 && B <= kMaxRankedBatch;
    int G;
    if (ranked) {
        const int full = B / ncl, rem = B % ncl;
        const int pos_in_last = (full & 1) ? ncl - 1 - cl : cl;
        G = full + (pos_in_last < rem ? 1 : 0);
    } else {
        G = B - b0;
        if (G > hpc) G = hpc;
    }
    if (G <= 0) return;   // the whole group leaves together
    if (ranked) {
        int *lens = reinterpret_cast<int *>(dyn_lds);
        for (int b = tid; b < B; b += THREADS) lens[b] = min(max(p.enc_len[b], 0), T);
        __syncthreads();
        for (int b = tid; b < B; b += THREADS) {
            const int lb = lens[b];
            int r = 0;
            for (int b2 = 0; b2 < B; ++b2) {
                const int l2 = lens[b2];
                r += (l2 > lb || (l2 == lb && b2 < b)) ? 1 : 0;
            }
            const int round = r / ncl, pos = r - round * ncl;
            if (((round & 1) ? ncl - 1 - pos : pos) == cl) S.gid[round] = b;
        }
        __syncthreads();   // the lengths are not needed any more
    } else {
        if (tid < G) S.gid[tid] = b0 + tid;
    }
    const int Hp = p.h_pred, L = DEEP && !ONE_ROUND ? p.pred_layers : 1;

    // ---- LDS: in deeper LSTMs of few hypotheses the tile of packed rows (bfloat16); the partial sums of a round -- of the predictor side and of a joint
    // pass, which may start while the former are still read; every wavefront's staged rows (STAGED; eight
    // wavefronts: over the partial sums); and what this workgroup keeps of its own units: recurrent
    // pre-activations, cell state, (chunks) hidden state
    const int ldb = ActTile<WT>::row_elems(p.kseg_max);
    WT *const planes = reinterpret_cast<WT *>(dyn_lds);
    float *const part_q = reinterpret_cast<float *>(dyn_lds + (PL == 3 && DEEP && !LISTS && hpc <= kPackRows ? RT * ldb * sizeof(WT) : 0));   // [NW][16][PLQ]
    float *const part_j = part_q + (LSTM && !WIDE ? NW * RT * PLQ : 0);                                              // [NW][16][PLJ]
    for (int i = tid; i < p.lds_bytes / 16; i += THREADS)
        reinterpret_cast<uint4 *>(dyn_lds)[i] = make_uint4(0, 0, 0, 0);

    // ---- this workgroup's column tiles of the predictor side, and with its W_hh tiles a stretch of hidden
    // units (see pred_share)
    const int nst_h = (Hp + KS - 1) / KS, nst_j = (H + KS - 1) / KS;   // fragments per tile
    const int NT_A = (H + CT - 1) / CT, NT_B = LSTM ? (Hp + 3) / 4 : 0;
    const PredShare share = pred_share(DEEP, NT_A, NT_B, Hp, C, rank);
    const int qt0 = share.qt0, na = share.na, r0 = share.r0, nr = share.nr, nq = na + nr;
    const int u0 = share.u0, U = share.U, QT = (NT_A + NT_B + C - 1) / C;
    const int Upad = (DEEP ? (NT_B + C - 1) / C : QT) * 4;
    const int xp_rows = STAGED && TWO ? pred_area_rows(LAYERS, hpc) : 0;
    float *const xs = part_j + NW * RT * (WIDE ? p.wide_part : PLJ);             // staged rows: [NW][16 + xp_rows][LDX]
    static_assert(!WIDE || RT * LDX <= RT * kWidePart, "wide: a wavefront's rows lie over its share of the partial sums");
    float *const xe = WIDE ? part_q + wave * RT * LDX : xs + wave * (RT + xp_rows) * LDX, *const xp = xe + (TWO ? RT * LDX : 0);
    float4 *const rg_l = reinterpret_cast<float4 *>(xs + (STAGED ? NW * (RT + xp_rows) * LDX : 0));               // [L][hpc][Upad]
    float *const c_l = reinterpret_cast<float *>(rg_l + (size_t)(LSTM ? L * hpc * Upad : 0));
    float *const h_l = c_l + (LSTM ? L * hpc * Upad : 0);                                 // (chunks only)

    const int rows_cap = p.rows_per_cluster;
    float *const hx = p.hbuf;         // [2][L][Bw][Hp]
    float *const px = p.pred_proj;    // [2][Bw][H]
    const int cells = p.cells_per_cluster;   // joint cells of one buffer (work items x 16)
    // The words of the joint exchanges lie behind one another (label_words, some eight megabytes at most) and are reached through
    // one descriptor: a lane offset and a scalar offset instead of 64-bit sums of pointers, of which a pass needed some
    // twenty.  Byte offsets of this group's, and the bytes of one of their kRowBufs buffers:
    auto behind = [&](const unsigned long long *q) { return (int)((q - p.row_lab) * sizeof(unsigned long long)); };
    const int jb_n = cells * 8, jd_n = 2 * rows_cap * 8, jh_n = C * 8;
    const int jb = cl * kRowBufs * jb_n;                          // packed (logit, ~label)
    const int jl = behind(p.row_lse) + jb;                        // (largest logit, sum of exp)
    const int jd = behind(p.row_dur) + cl * kRowBufs * jd_n;      // packed (logit, ~duration class)
    const int jh = behind(p.present) + cl * (kRowBufs + 1) * jh_n;   // workgroups without a work item (the last: state has been read)
    const __amdgpu_buffer_rsrc_t crs = buffer_of(p.row_lab, (size_t)behind(p.present) + (size_t)ncl * (kRowBufs + 1) * jh_n);
    auto ld_word = [&](int lane_off, int off) __attribute__((always_inline)) { return ld_word64(crs, lane_off, off); };
    auto st_word = [&](int lane_off, int off, unsigned long long v) __attribute__((always_inline)) { st_word64(crs, lane_off, off, v); };

    // ---- Alg. 3 lines 3-4.  Lane g of every wavefront holds hypothesis g of the group
    __syncthreads();
    const bool mine = lane < G;
    int gid = mine ? S.gid[lane] : 0;   // (read again where it is needed)
    int len = mine ? p.enc_len[gid] : 0, status = 0;
    if (len < 0) { len = 0; status = TDT_HYP_LEN_CLAMPED; }
    if (len > T) { len = T; status = TDT_HYP_LEN_CLAMPED; }
    int time = 0, sym = 0, last = V, last2 = V, olen = 0;
    float score = 0.0f;   // (of the hypotheses whose scores this workgroup sums: slot % C == rank)
    bool started = false;
    if (CHUNKED && mine) {
        started = p.st_started[gid] != 0;
        time = max(p.st_time[gid], 0);
        if (started) {
            last = min(max(p.st_last[gid], 0), V);
            last2 = min(max(p.st_last2[gid], 0), V);
        }
    }
    bool active = mine && time < len;
    const unsigned long long carried = CHUNKED ? __ballot(active && started) : 0ull;   // bring a state along
    const unsigned long long took_part = __ballot(active);
    started = started || active;
    if (tid < TDT_MAX_DURATIONS) S.durations[tid] = p.durations[tid];
    if (tid == 0) {
#if TDT_TRACE
        g_tr_n = 0;
        g_tr_on = 0;
#endif
        S.aborted = 0;
        for (int a = 0; a < 5; ++a) S.tk[a] = 0;
        S.tk_last = S.tk_start = wall_clock64();
    }
    enum { kTkP = 0, kTkQ, kTkJ, kTkD, kTkBar };
    auto lap = [&](int bucket) {   // profiling builds only: see decode.hip
        if (TDT_PHASE_TIMERS && tid == 0) {
            const long long now = wall_clock64();
            S.tk[bucket] += now - S.tk_last;
            S.tk_last = now;
        }
    };
    if (CHUNKED) {   // rank 0 writes the new state when everybody has read the old one
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) st_word(rank * 8, jh + kRowBufs * jh_n, 1ull);
    }
    const unsigned long long owned = __ballot(mine && lane % C == rank);   // whose scores this workgroup sums

    // ---- how a joint pass is cut, per number of searching hypotheses
    const int NT = (O + CT - 1) / CT;
    {
        const int rows_auto = label_joint_rows(C, NT, p.joint_tiles, hpc);
        for (int n = tid + 1; n <= G; n += THREADS) {
            const int Kw = label_window(n, p.window, rows_auto, rows_cap, C, NT);
            const int n_tiles = (n * Kw + RT - 1) / RT;
            int n_cg, tpg;
            split_tiles(C, WIDE ? 1 : n_tiles, NT, C, n_cg, tpg);   // (wide: a workgroup takes its columns of all rows)
            LabelPlan pl;
            pl.Kw = (short)Kw;
            pl.rcp_kw = ((1 << 20) + Kw - 1) / Kw;
            pl.n_tiles = (short)n_tiles;
            pl.n_cg = (short)n_cg;
            pl.tpg = (short)tpg;
            pl.ti0 = (short)(rank / n_cg);
            pl.cg0 = (short)(rank % n_cg);
            S.plan[n] = pl;
        }
    }
    __syncthreads();

    // ---- Algorithm 3's inner loop ends when nobody searches any more: a group's label takes as many joint passes as its
    // longest search, and who has found one waits.  Here it ends, after any pass, as soon as those
    // who wait are as many as those who search (no predictor: half as many): they take their predictor step, and
    // the next pass scores both.  A hypothesis' own sequence of steps is the same; the group's joint passes are fewer, for more
    // predictor steps of fewer hypotheses.  Replays of decoded hypotheses (7 to 16 of a group; labels in bursts, and drawn on 3 to 60
    // % of the frames) take 0.82 to 1.00 of the lock step's time with this rule, with a step after every pass that found
    // one 0.82 to 1.24 (predictor and joint pass at their measured times).  Not with a caller's window, which asks for the steps
    // as they are printed, nor with long ones, of which a search takes one.  us a call, in lock step / now: RNN-T B = 32 987 / 943,
    // B = 128 1986 / 1850, TDT B = 32 494 / 448, stateless B = 128 1979 / 1782, multi-blank B = 27 521 / 504; one or two
    // hypotheses a group 235 / 237.  (One has nobody to wait for and a long window: a pass has a row tile at least.)
    // Deeper LSTMs, whose predictor step is two joint passes and more: four times as many as search; twice, where the output
    // layer is streamed and few rows are no shorter pass (two layers, 640 units, B = 32, 1761 us, with two to one 1796, four to one
    // 1766; B = 128 3205, 3207, 3149; 8198 outputs, B = 96, 3804, 3475, three to one 3507; config 5 29489, 27752).  Reductions
    // over 640, one layer: joint width 1024, B = 32, 1876 / 1751; TDT, B = 64, 1302 / 1128.
    const int patience = MERGES && p.window == 0 && uni(S.plan[G].Kw) < kLongWindow ? (LSTM || WIDE ? 1 : 2) : 0;
    constexpr int kCrowd = !DEEP ? 1 : WIDE ? 2 : 4;

    unsigned st_pred_passes = 0, st_joint_passes = 0;
    long long st_pred_rows = 0, st_joint_rows = 0;

    // A wavefront whose data is not there yet: every 64th time it looks whether to give up.
    auto give_up = [&](unsigned &spins, long long &since) -> bool {
        if (spins == 0) since = wall_clock64();
        if ((++spins & 63u) != 0u) return false;
        int stop = 0;
        if (lane == 0) {
            if (__hip_atomic_load(p.abort_flag, __ATOMIC_RELAXED, TDT_AGENT)) {
                stop = 1;
            } else if (wall_clock64() - since > p.timeout_ticks) {
                __hip_atomic_store(p.abort_flag, 1, __ATOMIC_RELAXED, TDT_AGENT);
                stop = 1;
            }
        }
        stop = uni(stop);
        if (stop && lane == 0) S.aborted = 1;
        return stop != 0;
    };
    // Reads rows until no word of them is absent: read() requests them, leaves them where its caller wants
    // them and returns the largest word.  The intrinsic behind ldx4 does not say that what it reads changes;
    // the statement in front of it does, so that every turn issues the loads again.
    auto until_there = [&](auto read) __attribute__((always_inline)) {
        unsigned spins = 0;
        long long since = 0;
#pragma clang loop unroll(disable)
        for (;;) {
            asm volatile("" ::: "memory");
            const unsigned mx = read();
            if (__ballot(mx == kAbsent) == 0ull || give_up(spins, since)) break;
        }
    };
    // waits until the words of every lane are there (zero: not yet) and returns them
    auto wait_word = [&](int lane_off, int off) __attribute__((always_inline)) {
        unsigned spins = 0;
        long long since = 0;
        for (;;) {
            asm volatile("" ::: "memory");   // (see until_there)
            const unsigned long long x = ld_word(lane_off, off);
            if (__ballot(x == 0ull) == 0ull || give_up(spins, since)) return x;
        }
    };

    // ---- which steps of a reduction of nst steps this wavefront takes: a contiguous stretch, the
    // first nst % NW wavefronts one step more
    const int hs0 = wave * (nst_h / NW) + min(wave, nst_h % NW), hsn = nst_h / NW + (wave < nst_h % NW ? 1 : 0);
    const int js0 = wave * (nst_j / NW) + min(wave, nst_j % NW), jsn = nst_j / NW + (wave < nst_j % NW ? 1 : 0);
    // ---- weight fragments of a round; tile_off(t): byte offset of tile t among the fragment-major
    // copies
    const __amdgpu_buffer_rsrc_t wrs = buffer_of(p.packed, p.packed_bytes);
    auto fetch = [&](auto &b, int n, int s0, int sn, auto tile_off) __attribute__((always_inline)) {
        constexpr int TT = sizeof(b) / (NK * sizeof(v4u));
        if constexpr (PL == 3 && !WIDE) any_acc(b);
        else any_value(b);
#pragma unroll
        for (int t = 0; t < TT; ++t)
            if (t < n) {   // uniform
                const int w = tile_off(t) + s0 * 1024;
#pragma unroll
                for (int s = 0; s < NK; ++s)   // (a step beyond the wavefront's share: zeros, by an offset beyond the buffer)
                    b[t][s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, s < sn ? lane * 16 : ~0xff, w + (s < sn ? s : 0) * 1024, 0);
            }
    };
    // The round's products, into this wavefront's share of the partial sums.  The tile count is rounded up to what is compiled (what stands in the registers of the other tiles is multiplied
    // too, and nobody looks at it): without branches between them the products of the tiles overlap.
    // PACKED: the planes of a row are rows of one tile.
    // float32, short reductions, sn: steps of this wavefront (the others' weights are zeros, and a product takes 32 cycles: a joint width
    // of 64 has one step a wavefront where four are compiled, a call of the smallest benchmark model 262 us, now 228; where ten
    // are compiled the branches cost more: float32 at B = 16 1.46 ms, with them 1.53).
    auto products_of = [&](auto packed_tag, auto count, const AFrag (&a)[NK][PL], const auto &b, auto tiles, int sn, float *part) __attribute__((always_inline)) {
        constexpr bool PACKED = decltype(packed_tag)::value;
        constexpr int PLD = decltype(tiles)::value * CT + 4;
        constexpr int N = decltype(count)::value, NC = PL == 1 || PACKED || N < 4 ? 2 : 1;   // chains per tile
        float *const pw = part + (size_t)wave * RT * PLD + (lane & 15) * PLD + (lane >> 4) * 4;
        if constexpr (WIDE) {   // (half the registers a lane: two tiles at a time; the other wavefront of the SIMD fills the gaps)
#pragma unroll
            for (int t = 0; t < N; t += 2) {
                f32x4 c[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                for (int s = 0; s < NK; ++s)
#pragma unroll
                    for (int pl = PACKED ? 0 : PL - 1; pl >= 0; --pl)
#pragma unroll
                        for (int u = 0; u < 2; ++u) c[u] = F::mma(a[s][pl], b[t + u][s], c[u]);
#pragma unroll
                for (int u = 0; u < 2; ++u) *reinterpret_cast<f32x4 *>(pw + (t + u) * CT) = c[u];
                __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
        f32x4 c[N][NC];
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int ch = 0; ch < NC; ++ch) c[t][ch] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        // (the remainders of all steps first: they are small, and what they are added to is small then)
#pragma unroll
        for (int k = 0; k < NK * (PACKED ? 1 : PL); ++k) {
            const int s = k < NK * (PL - 1) && !PACKED ? k / (PL - 1 > 0 ? PL - 1 : 1) : k % NK;
            const int pl = k < NK * (PL - 1) && !PACKED ? PL - 1 - k % (PL - 1 > 0 ? PL - 1 : 1) : 0;
            if (PL > 1 || NK > 4 || s < sn)   // uniform
#pragma unroll
                for (int t = 0; t < N; ++t) c[t][k % NC] = F::mma(a[s][pl], b[t][s], c[t][k % NC]);
        }
#pragma unroll
        for (int t = 0; t < N; ++t) {
            f32x4 sum = c[t][0];
            if (NC > 1) sum = sum + c[t][NC - 1];
            *reinterpret_cast<f32x4 *>(pw + t * CT) = sum;
        }
    };
    auto products = [&](auto packed_tag, const AFrag (&a)[NK][PL], const auto &b, int n, auto tiles, int sn, float *part) __attribute__((always_inline)) {
        constexpr int TT = sizeof(b) / (NK * sizeof(v4u));
        constexpr int H2 = WIDE ? (TT + 2) / 4 * 2 : TT / 2;   // (wide: pairs)
        const std::integral_constant<int, H2> half{};
        const std::integral_constant<int, TT> all{};
        if (n <= H2) products_of(packed_tag, half, a, b, tiles, sn, part);
        else products_of(packed_tag, all, a, b, tiles, sn, part);
    };
    // ---- activation fragments.  A wavefront multiplies its own stretch of the reduction only.  In the deep
    // form of four wavefronts it loads that stretch of all 16 rows straight into the registers the matrix
    // cores read, lane l part l / 16 of every step of row l % 16 (up to kPackRows rows of the hidden state: see
    // load_packed); in the others rows are staged (stage_rows).
    // Byte offset of a lane's part of step s in a row of K inputs; parts beyond the row's end read its last
    // inputs again (they meet zeros in the weights, but must be numbers).
    auto part_of = [&](int s, int s0, int K) __attribute__((always_inline)) {
        return min((s0 + s) * KS + (lane >> 4) * F::E, K - F::E) * (int)sizeof(float);
    };
    // bfloat16: x == hi + lo + lo2 as in ActTile::split3, two elements packed per instruction.  A term is taken off its
    // element by a product with (-1, 0) or (0, -1) of the packed pair (terms.h).
    // That instruction runs where products do and waits for them, so a split beside products uses two.
    const std::true_type beside_products{};
    const std::false_type alone{};
    const MinusOne minus;
    auto split = [&](const float (&x0)[F::E], AFrag (&a)[PL], auto beside) __attribute__((always_inline)) {
        if constexpr (PL == 3) {
            float x[F::E];
#pragma unroll
            for (int e = 0; e < F::E; ++e) x[e] = x0[e];
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
                v4u o;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    o[e] = top_halves(x[2 * e], x[2 * e + 1]);
                a[pl] = *reinterpret_cast<const AFrag *>(&o);
                if (pl < 2)
#pragma unroll
                    for (int e = 0; e < F::E; ++e) {
                        if constexpr (decltype(beside)::value) x[e] -= __uint_as_float(__float_as_uint(x[e]) & 0xffff0000u);
                        else x[e] = less_term(o[e / 2], e % 2 ? minus.high : minus.low, x[e]);
                    }
            }
        } else {
            a[0] = AFrag{x0[0], x0[1], x0[2], x0[3]};
        }
    };
    // staged rows: eight lanes take 128 bytes of a row; this lane's are inputs i * 32 + lane % 8 * 4 .. + 3 of the wavefront's stretch of rows
    // lane / 8 and lane / 8 + 8 (inputs beyond the row's end: its last ones again)
    auto flat_off = [&](int i, int s0, int K) __attribute__((always_inline)) {
        return min(s0 * KS + i * 32 + (lane & 7) * 4, K - 4) * (int)sizeof(float);
    };
    // nothing of what one lane stores is read by another lane ahead of it: LDS accesses of a wavefront
    // are carried out in order, this keeps the compiler to that order
    auto lds_order = []() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    };
    // (rows: which of them; the others keep what they have)
    auto stage_some = [&](float *x, const v4u (&v)[2 * C32], bool upper, unsigned rows) __attribute__((always_inline)) {
        float *const at = x + (lane >> 3) * LDX + (lane & 7) * 4;
        rows >>= lane >> 3;
        lds_order();
        if (rows & 1u)
#pragma unroll
            for (int i = 0; i < C32; ++i) *reinterpret_cast<v4u *>(at + i * 32) = v[i];
        if (upper && (rows >> 8 & 1u))   // (upper: uniform)
#pragma unroll
            for (int i = 0; i < C32; ++i) *reinterpret_cast<v4u *>(at + 8 * LDX + i * 32) = v[C32 + i];
        lds_order();
    };
    auto stage_rows = [&](float *x, const v4u (&v)[2 * C32], bool upper) __attribute__((always_inline)) {
        float *const at = x + (lane >> 3) * LDX + (lane & 7) * 4;
        lds_order();
#pragma unroll
        for (int i = 0; i < C32; ++i) *reinterpret_cast<v4u *>(at + i * 32) = v[i];
        if (upper)   // uniform
#pragma unroll
            for (int i = 0; i < C32; ++i) *reinterpret_cast<v4u *>(at + 8 * LDX + i * 32) = v[C32 + i];
        lds_order();
    };
    // part l / 16 of step s of a staged row
    auto staged = [&](const float *x, int row, int s, int l) __attribute__((always_inline)) {
        return *reinterpret_cast<const float4 *>(x + row * LDX + s * KS + (lane >> 4) * F::E + l * 4);
    };
    // up to kPackRows rows: through LDS, where plane pl of row i is row pl * kPackRows + i
    auto load_packed = [&](AFrag (&a)[NK][PL], int s0, int sn) __attribute__((always_inline)) {
        const WT *row = planes + (lane & 15) * ldb;
#pragma unroll
        for (int s = 0; s < NK; ++s)
            a[s][0] = *reinterpret_cast<const AFrag *>(row + (s < sn ? (s0 + s) * KS + (lane >> 4) * F::E : ldb - F::E));
    };
    // The first round's products (bfloat16, staged rows) while the rows are split: source(s, x) reads this lane's
    // inputs of step s.  The matrix cores take 16 cycles a product and the wavefront issues an instruction every
    // 4 to 5, so the split of step s + 1 goes between the products of step s -- of its remainders: a product of first
    // terms is added to a sum of all remainders.  Error of 640 products against 64 bits, rms for a logit of 1: 6.71e-8,
    // with a chain of accumulators for each of the three terms 6.93e-8, with one chain step by step 1.22e-7.
    auto split_and_multiply = [&](auto count, auto source, AFrag (&a)[NK][PL], const auto &b, auto tiles, float *part) __attribute__((always_inline)) {
        constexpr int PLD = decltype(tiles)::value * CT + 4, N = decltype(count)::value;
        float *const pw = part + (size_t)wave * RT * PLD + (lane & 15) * PLD + (lane >> 4) * 4;
        f32x4 c[N];
#pragma unroll
        for (int t = 0; t < N; ++t) c[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        float x[2][F::E];
        source(0, x[0]);
        if (NK > 1) source(1, x[1]);
        split(x[0], a[0], alone);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            if (s + 1 < NK) split(x[(s + 1) & 1], a[s + 1], beside_products);
            if (s + 2 < NK) source(s + 2, x[s & 1]);
#pragma unroll
            for (int pl = PL - 1; pl > 0; --pl)
#pragma unroll
                for (int t = 0; t < N; ++t) c[t] = F::mma(a[s][pl], b[t][s], c[t]);
            if (s + 1 < NK)
#pragma unroll
                for (int i = 0; i < N * (PL - 1); ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // a product
                    __builtin_amdgcn_sched_group_barrier(0x002, (60 + N * (PL - 1) - 1) / (N * (PL - 1)), 0);   // its share of the split
                }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = 0; s < NK; ++s)
#pragma unroll
            for (int t = 0; t < N; ++t) c[t] = F::mma(a[s][0], b[t][s], c[t]);
#pragma unroll
        for (int t = 0; t < N; ++t) *reinterpret_cast<f32x4 *>(pw + t * CT) = c[t];
    };
    const std::true_type packed_rows{};
    const std::false_type full_rows{};
    // four neighbouring columns of a row of the partial sums, summed over the wavefronts
    auto gather = [&](auto tiles, const float *part, int row, int quad) __attribute__((always_inline)) {
        constexpr int PLD = decltype(tiles)::value * CT + 4;
        const float *q = part + (size_t)row * PLD + quad * 4;
        float4 x[NW];   // (all on their way before the first is looked at)
#pragma unroll
        for (int w = 0; w < NW; ++w) x[w] = *reinterpret_cast<const float4 *>(q + (size_t)w * RT * PLD);
        if (!WIDE && (!DEEP || OWN2)) __builtin_amdgcn_sched_barrier(0);
        float4 v = x[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            v.x += x[w].x;
            v.y += x[w].y;
            v.z += x[w].z;
            v.w += x[w].w;
        }
        return v;
    };
    const std::integral_constant<int, TQ> q_tiles{};
    const std::integral_constant<int, TR> r_tiles{};
    const std::integral_constant<int, TJ> j_tiles{};
    // inputs k .. k+3 of packed row i
    auto put = [&](int i, int k, float4 v) __attribute__((always_inline)) {
        WT *o = planes + i * ldb + k;
        float x0 = v.x, x1 = v.y, x2 = v.z, x3 = v.w;
        auto top = [](float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); };
        auto pack = [](float lo, float hi) {
            return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
        };
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            *reinterpret_cast<uint2 *>(o + pl * kPackRows * ldb) = make_uint2(pack(x0, x1), pack(x2, x3));
            if (pl < 2) {
                x0 -= top(x0);
                x1 -= top(x1);
                x2 -= top(x2);
                x3 -= top(x3);
            }
        }
    };
    const bool qpack = PL == 3 && ((DEEP && !LISTS) || PLANES) && hpc <= kPackRows, qpair = FEW || (PLANES && !qpack && hpc <= kPairRows);
    // bfloat16, one layer: the hidden state travels as the three terms of its values, in the order in which the matrix cores
    // take them.  Whoever updates a cell splits it, once, and a reader of the exchange buffers has its operands in
    // registers as soon as they are there: no rows to change lanes, no split.  Plane row `pl * RP + g` is term pl of hypothesis g,
    // RP the rows of a plane: with up to four hypotheses four, and all terms are rows of one tile of sixteen; up to eight eight, a tile
    // and a half; else sixteen.  A step of 32 inputs is 64 bytes a plane row: a lane's eight inputs of plane row r are the 16 bytes
    // at (lane / 16 * 3 RP + r) * 16.  Absent is a pair of terms that are all ones, which no two terms are: a NaN is stored as the one of
    // which they are not.  Before, every reader had rows of float32 change lanes through LDS and split them, and ten
    // workgroups of 51 had all of W_pred (see pred_share).  Both with the encoder's rows staged early (planes_of), and the table
    // rows requested early (request_gates), us a call on the same utterances: config 2 at B = 1 528 / 503, B = 32 847 / 814, B = 128 2017 / 1942,
    // 32 chunked streams 1811 / 1732, TDT B = 7 289 / 274, B = 32 454 / 441.
    const int RP = plane_rows(hpc), hstep = plane_step(hpc), plane_buffer = plane_bytes(Hp, hpc);
    auto plane_base = [&](int buffer) { return (buffer * ncl + cl) * plane_buffer; };
    // Products of the first `count` tiles that `b` holds with the plane rows `v` (NT tiles of them), smallest terms first
    auto plane_products = [&](auto count, const auto &v, const auto &b, auto tiles, float *part) __attribute__((always_inline)) {
        constexpr int PLD = decltype(tiles)::value * CT + 4, N = decltype(count)::value;
        constexpr int NT = sizeof(v) / sizeof(v[0]);
        float *const pw = part + (size_t)wave * RT * PLD + (lane & 15) * PLD + (lane >> 4) * 4;
        f32x4 c[N];
#pragma unroll
        for (int t = 0; t < N; ++t) c[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = NT - 1; i >= 0; --i)
#pragma unroll
            for (int s = 0; s < NK; ++s)
#pragma unroll
                for (int t = 0; t < N; ++t) c[t] = F::mma(*reinterpret_cast<const AFrag *>(&v[i][s]), b[t][s], c[t]);
#pragma unroll
        for (int t = 0; t < N; ++t) *reinterpret_cast<f32x4 *>(pw + t * CT) = c[t];
    };

    // float32, one layer, few rows: sixteen products of four columns and four rows at a time (v_mfma_f32_4x4x1_16b_f32,
    // 8 cycles) instead of one of sixteen and sixteen over four inputs (32 cycles, four a step and tile, whatever
    // rows there are).  A lane's part of a fragment is column l % 16 and inputs l / 16 * 4 .. + 3 of the step, so the
    // products are those of four columns with four rows over one input in four, and every lane ends with its four
    // neighbouring columns of row l % 4 over a quarter of the wavefront's inputs.  Quarters are added up in pairs, and lie
    // in the partial sums as planes of up to eight rows do: half q of row i is row q * 8 + i.  Four rows at a time; a form of its
    // own, because rows for both kinds of products were 22 registers more than there are.  What bounds it are the matrix cores: four
    // tiles and 160 inputs a wavefront took 5120 cycles, now 1280 per four rows (see few_rows for which groups).  Config 2's model in
    // float32, B = 16, four rows a group, 1305 / 1179 us.  Error of 640 products against 64 bits, rms for a result of 1: 1.69e-7 / 1.27e-7 (shorter
    // chains: tests/test_sum_orders.py forms both sums).
    auto few_products = [&](const auto &b0, const auto &b1, auto tiles, float *part) __attribute__((always_inline)) {
        constexpr int PLD = decltype(tiles)::value * CT + 4, N = TWO_ROUNDS ? 2 * TR : TR;
#pragma clang loop unroll(disable)
        for (int r = 0; r < hpc; r += 4) {   // uniform
            float *const pw = part + (size_t)wave * RT * PLD + (r + (lane & 3) + ((lane >> 4) & 1) * kPairRows) * PLD + ((lane >> 2) & 3) * 4;
            constexpr int AHEAD = 3;   // steps of the rows on their way (registers)
            float4 x[AHEAD];
#pragma unroll
            for (int s = 0; s < AHEAD; ++s) x[s] = staged(xe, r + (lane & 3), s, 0);
            f32x4 c[N];
#pragma unroll
            for (int t = 0; t < N; ++t) c[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < NK; ++s) {
                const float4 y4 = x[s % AHEAD];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < N; ++t) {
                        const float y = e == 0 ? y4.x : e == 1 ? y4.y : e == 2 ? y4.z : y4.w;
                        const float w = __uint_as_float(t < TR ? b0[t % TR][s][e] : b1[t % TR][s][e]);
                        c[t] = __builtin_amdgcn_mfma_f32_4x4x1f32(w, y, c[t], 0, 0, 0);
                    }
                if (s + AHEAD < NK) x[s % AHEAD] = staged(xe, r + (lane & 3), s + AHEAD, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int t = 0; t < N; ++t) {
                f32x4 sum;
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] = sum_over_halves(c[t][e]);
                if (lane < 32) *reinterpret_cast<f32x4 *>(pw + t * CT) = sum;
            }
        }
    };

    // byte offsets of this workgroup's predictor-side tiles (the fragment-major copies)
    const int hbytes = nst_h * 1024, jbytes = nst_j * 1024;
    auto q_tile = [&](int t) {
        return t < na ? p.off_w_pred + (qt0 + t) * hbytes : p.off_w_hh[L - 1] + (r0 + t - na) * hbytes;
    };

    // the four columns a thread takes of a round of phase Q (packed: a wavefront holds one row, in four places)
    auto q_quad = [&]() { return qpack ? (wave / kPackRows) * 16 + (lane & 15) : tid % QPR; };

    // the LSTM cell of one unit: new cell value and new hidden value
    auto cell = [&](float4 g4, float c_old, float &cn, float &hn) __attribute__((always_inline)) {
        const float ig = sigmoid(g4.x), fg = sigmoid(g4.y);
        const float gg = 2.0f * sigmoid(2.0f * g4.z) - 1.0f;
        const float og = sigmoid(g4.w);
        cn = fg * c_old + ig * gg;
        hn = og * (2.0f * sigmoid(2.0f * cn) - 1.0f);
    };

    // what lane l reads of a whole row: inputs l*4 + kk*256 .. + 3, or the row's last ones again
    auto hoff = [&](int kk) { return min(lane * 4 + kk * 256, Hp - 4) * (int)sizeof(float); };
    const __amdgpu_buffer_rsrc_t hrs = buffer_of(hx, PLANES ? (size_t)planes_covered(ncl, Hp, hpc, NK) : (size_t)2 * L * Bw * Hp * sizeof(float));
    const __amdgpu_buffer_rsrc_t prs = buffer_of(px, (size_t)2 * Bw * H * sizeof(float));
    const __amdgpu_buffer_rsrc_t brs = buffer_of(p.b_out, (size_t)O * sizeof(float));
    auto h_source = [&](int s, float (&x)[F::E]) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const float4 y = staged(xe, lane & 15, s, l);
            x[l * 4] = y.x;
            x[l * 4 + 1] = y.y;
            x[l * 4 + 2] = y.z;
            x[l * 4 + 3] = y.w;
        }
    };
    // Row tile tq of this label iteration's hidden state (row0: the group's first row in the exchange
    // buffer): loads, waits, splits.  For a row without an active hypothesis nothing is loaded where rows are
    // staged, elsewhere it repeats one that has (nobody looks at its results).
    auto stage_h = [&](auto &a, int row0, int tq, unsigned long long in_tile) __attribute__((always_inline)) {
        constexpr int NA = sizeof(a) / sizeof(a[0]);   // (steps: NQ)
        const int any = __ffsll((long long)in_tile) - 1;
        if (DEEP && qpack) {   // a wavefront takes a row
            if constexpr (PL == 3 && DEEP && !LISTS) {
                v4u v[KI];
                const bool row = wave < kPackRows;   // uniform
                const int off = (row0 + (row && ((in_tile >> wave) & 1ull) ? wave : any)) * Hp * (int)sizeof(float);
                until_there([&]() __attribute__((always_inline)) {
                    unsigned mx = 0;
#pragma unroll
                    for (int kk = 0; kk < KI; ++kk) v[kk] = ldx4(hrs, hoff(kk), off);
#pragma unroll
                    for (int kk = 0; kk < KI; ++kk) mx = max(mx, umax4(v[kk]));
                    return mx;
                });
                TR(11);
                if (row)
#pragma unroll
                for (int kk = 0; kk < KI; ++kk)   // (lanes beyond the row's end write its last inputs again)
                    put(wave, hoff(kk) / (int)sizeof(float), as_float4(v[kk]));
                __syncthreads();
                TR(13);
                fresh();
                load_packed(a, hs0, hsn);
            }
        } else {
            if constexpr (STAGED) {
                v4u v[2 * C32];
                int off[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {   // (nothing is loaded for a row without an active hypothesis)
                    const int g = h * 8 + (lane >> 3);
                    off[h] = (in_tile >> g) & 1ull ? (row0 + g) * Hp * (int)sizeof(float) : kNowhere;
                }
                const bool upper = (in_tile >> 8) != 0ull;
                until_there([&]() __attribute__((always_inline)) {
                    unsigned mx = 0;
#pragma unroll
                    for (int i = 0; i < C32; ++i) v[i] = ldx4(hrs, off[0] + flat_off(i, hs0, Hp), 0);
                    if (upper)
#pragma unroll
                        for (int i = 0; i < C32; ++i) v[C32 + i] = ldx4(hrs, off[1] + flat_off(i, hs0, Hp), 0);
#pragma unroll
                    for (int i = 0; i < C32; ++i) mx = max(mx, umax4(v[i]));
                    if (upper)
#pragma unroll
                        for (int i = 0; i < C32; ++i) mx = max(mx, umax4(v[C32 + i]));
                    return mx;
                });
                TR(11);
                stage_rows(xe, v, upper);
                if constexpr (!FEW)
#pragma unroll
                    for (int s = 0; s < NK; ++s) {
                        float x[F::E];
                        h_source(s, x);
                        split(x, a[s], alone);
                    }
                return;
            }
            v4u v[NA][NL];
            int off[NA];
            const int g = (in_tile >> (lane & 15)) & 1ull ? lane & 15 : any;
            const int row = (row0 + tq * RT + g) * Hp * (int)sizeof(float);
#pragma unroll
            for (int s = 0; s < NA; ++s) off[s] = LISTS && s >= hsn ? kNowhere : row + part_of(s, hs0, Hp);
            until_there([&]() __attribute__((always_inline)) {
                unsigned mx = 0;
#pragma unroll
                for (int s = 0; s < NA; ++s)
#pragma unroll
                    for (int l = 0; l < NL; ++l) v[s][l] = ldx4(hrs, off[s] + l * 16, 0);
#pragma unroll
                for (int s = 0; s < NA; ++s)
#pragma unroll
                    for (int l = 0; l < NL; ++l) mx = max(mx, umax4(v[s][l]));
                return mx;
            });
            TR(11);
#pragma unroll
            for (int s = 0; s < NA; ++s) {
                float x[F::E];
#pragma unroll
                for (int e = 0; e < F::E; ++e) x[e] = __uint_as_float(v[s][e / 4][e % 4]);
                split(x, a[s], alone);
            }
        }
    };

    // this thread's first two cells (hypothesis, unit), and the h-th from base on
    auto cell_at = [&](int idx) { return U > 0 ? (idx / U) << 16 | (idx - idx / U * U) : kLabelMaxHyps << 16; };
    const int place0 = cell_at(tid), place1 = cell_at(tid + THREADS);
    auto place = [&](int base, int h, int &g, int &u) __attribute__((always_inline)) {
        const int at = base > 0 ? cell_at(base + h * THREADS + tid) : h == 0 ? place0 : place1;
        g = at >> 16;
        u = at & 0xffff;
    };
    int par = 0;                     // which buffer this label's rows go through
    unsigned jpass = 0;              // joint exchanges so far
    int prev_items = 0, prev_tiles = 0, prev_cg = 1;   // the last pass: work items, row tiles, column groups
    int prev2_items = 0, prev2_tiles = 0, clr_items = 0, clr_tiles = 0;   // the two before it
    unsigned long long act_prev = 0ull;        // who took part in the previous label's rows
    bool first = true, ok = true;
    unsigned long long needm = 0ull;           // who searches
    // (OWN) which of the two buffers hypothesis g's newest row of the projected predictor output is in.  The other one's is put
    // back while the newest is made: all have read it in the pass in which the hypothesis found its label.
    unsigned long long own = 0ull;
    auto p_row = [&](int g, int other) __attribute__((always_inline)) { return ((int)(own >> g & 1ull) ^ other) * Bw + b0 + g; };
    int dcg0 = -1, dcg1 = -1, dcg_tpg = 0;   // the column groups of dcg_tpg tiles that hold duration outputs (at most two: there are at most 16)

    // puts back what this workgroup wrote in the label iteration before (see the head of the file)
    auto clear_rows = [&](unsigned long long act) __attribute__((always_inline)) {
        const int pb = par ^ 1;
        const int hrow = Hp * (int)sizeof(float), jrow = H * (int)sizeof(float);
        if (U > 0)
#pragma clang loop unroll(disable)
            for (int base = 0; base < G * U; base += 2 * THREADS)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    int g, u;
                    place(base, h, g, u);
                    const int off = g < G && ((act_prev >> g) & 1ull) ? (b0 + g) * hrow + (u0 + u) * (int)sizeof(float) : kNowhere;
                    if (base + h * THREADS < G * U)   // uniform
#pragma clang loop unroll(disable)
                        for (int l = 0; l < L; ++l)
                            __builtin_amdgcn_raw_buffer_store_b32(kAbsent, hrs, off, (pb * L + l) * Bw * hrow, 16 /* sc1 */);
                }
        if (na > 0) {
            const int c = (tid & 15) * 4, nc = min(na * CT, H - qt0 * CT);   // (H is a multiple of 8)
            const v4u absent = {kAbsent, kAbsent, kAbsent, kAbsent};
#pragma clang loop unroll(disable)
            for (int c0 = 0; c0 < nc; c0 += 64)
#pragma clang loop unroll(disable)
                for (int g = tid >> 4; g < G; g += THREADS / 16)
                    if (((act >> g) & 1ull) && c0 + c < nc)
                        __builtin_amdgcn_raw_buffer_store_b128(absent, prs, p_row(g, 1) * jrow + (qt0 * CT + c0 + c) * (int)sizeof(float),
                                                               0, 16 /* sc1 */);
        }
    };
    // ... and its cells of the joint pass two before the last
    auto clear_cells = [&]() __attribute__((always_inline)) {
        if (C > 1 && jpass > 2 && wave == kClearer) {   // uniform
            const int pb = (int)((jpass - 3) & (kRowBufs - 1));
            const int stride = WIDE ? prev_cg : C;   // (wide: the same split in every pass)
            const int cell = (lane & 16 ? jl : jb) + (lane & 15) * 8;
            if (rank < stride)
#pragma clang loop unroll(disable)
            for (int it = rank; it < clr_items; it += stride)
                if (lane < 2 * RT) st_word(cell, pb * jb_n + it * RT * 8, 0ull);
            if (D > 0)   // (whoever wrote them: the words of a row tile are put back by rank ti)
#pragma clang loop unroll(disable)
                for (int ti = rank; ti < clr_tiles; ti += C)
                    if (lane < 2 * RT) st_word(lane * 8, jd + pb * jd_n + ti * RT * 16, 0ull);
            if (rank >= (WIDE ? stride : clr_items) && lane == 0) st_word(rank * 8, jh + pb * jh_n, 0ull);
        }
    };

    // ---- score terms of the labels found in the last pass, summed while the next pass's cells travel.
    // A hypothesis' score is summed by the workgroup of rank slot % C.
    bool pend = false;       // lane g: hypothesis g has a term to add
    int pend_row = 0;        // the row its label was found in
    float pend_m = 0.0f;     // that row's largest label logit
    auto finish_scores = [&]() {
        unsigned long long m = __ballot(pend) & owned;
        while (m != 0ull) {   // uniform
            const int g = __ffsll((long long)m) - 1;
            m &= m - 1ull;
            const int r = __builtin_amdgcn_readlane(pend_row, g);
            const float rowm = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pend_m), g));
            float s = 0.0f;
#pragma clang loop unroll(disable)
            for (int c0 = 0; c0 < prev_cg; c0 += 64) {
                const int c = min(c0 + lane, prev_cg - 1);
                const unsigned long long x =
                    C == 1 ? S.rowl[r]
                           : wait_word(c * RT * 8, jl + (int)((jpass - 1) & (kRowBufs - 1)) * jb_n + ((r >> 4) * prev_cg * RT + (r & 15)) * 8);
                const float cm = __uint_as_float((unsigned)x), cs = __uint_as_float((unsigned)(x >> 32));
                if (c0 + lane < prev_cg && cs > 0.0f) s += cs * __expf(cm - rowm);
            }
            s = wave_sum(s);
            s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), 63));
            if (lane == g) score -= logf(s);   // log_softmax at the maximum = -log(sum exp(l - max))
        }
        pend = false;
    };

    // ---- the work item at hand.  Lane i (of every 16) holds row i of its tile: the row of enc_proj, the
    // hypothesis, and which of the searching ones that is
    int ti = 0, cg = 0, tile0 = 0, n_ct = 0;
    int erow_l = 0, g_l = 0, q_l = 0;
    bool have_p = false;    // (TWO) this label's projected predictor output is staged
    int slot_of = 0;        // lane q: the q-th searching hypothesis
    int Kw = 1, rcp_kw = 1, n_tiles = 0, n_cg = 1, tpg = 1, items = 0, M = 0, ti0 = 0, cg0 = 0;
    auto plan_pass = [&](unsigned long long needm) __attribute__((always_inline)) {
        const int n_need = __popcll(needm);
        const LabelPlan lp = S.plan[n_need];
        // the searching hypotheses, packed to the front
        const bool need = (needm >> lane) & 1ull;
        const int to = need ? __popcll(needm & ((1ull << lane) - 1ull)) : 63;
        slot_of = __builtin_amdgcn_ds_permute(to * 4, lane);
        Kw = uni(lp.Kw);
        n_tiles = uni(lp.n_tiles);
        n_cg = uni(lp.n_cg);
        tpg = uni(lp.tpg);
        rcp_kw = uni(lp.rcp_kw);
        ti0 = uni(lp.ti0);
        cg0 = uni(lp.cg0);
        items = n_tiles * n_cg;
        M = n_need * Kw;
    };
    auto set_rows = [&]() __attribute__((always_inline)) {
        const int r = min(ti * RT + (lane & 15), M - 1);   // (a row beyond the last repeats it)
        const int q = (r * rcp_kw) >> 20;                  // r / Kw
        q_l = q;
        g_l = __builtin_amdgcn_ds_bpermute(q * 4, slot_of) & 63;
        const int f = __builtin_amdgcn_ds_bpermute(g_l * 4, time) + (r - q * Kw);
        // (every lane has to take part in every permute: what an inactive lane holds reads as zero)
        const int len_r = __builtin_amdgcn_ds_bpermute(g_l * 4, len), gid_r = S.gid[g_l];
        erow_l = gid_r * T + (f < len_r ? f : 0);   // (a frame beyond its utterance's end reads frame 0)
    };
    auto set_item = [&](int it) __attribute__((always_inline)) {
        ti = ti0;
        cg = cg0;
        if (it != rank) {
            ti = it / here(n_cg);   // (the division's preparation stays in here)
            cg = it - ti * n_cg;
        }
        tile0 = cg * tpg;
        n_ct = min(tpg, NT - tile0);
        set_rows();
    };

    // ---- LAYERS == 1: where this thread's results of phase Q go -- four columns of one row per half of
    // a round -- and its cell.  Offsets into the exchange buffers; beyond their end where there is
    // nothing to write, so that the stores need no branch.
    constexpr int QH = TQ > 4 ? 2 : 1;   // halves of a round: four tiles, four columns a thread
    auto q_hyp = [&]() { return qpack ? wave : qpair ? wave * 2 + ((lane >> 4) & 1) : tid >> 4; };
    int q_off[2] = {kNowhere, kNowhere}, q_unit[2] = {-1, -1}, h_off[2] = {kNowhere, kNowhere}, h_off2[2] = {kNowhere, kNowhere}, c_g[2], c_u[2];
    float4 q_bias[2];
    // ... and the place in the exchange buffers (its scalar part; OWN: in the lane's offset), of the newest row and the one before
    auto q_base = [&](int other) { return OWN ? 0 : ((par ^ other) * Bw + b0) * H * (int)sizeof(float); };
    auto q_at = [&](int h, unsigned long long act, int other) __attribute__((always_inline)) {
        if (!OWN) return q_off[h];
        const int g = q_hyp();   // (at most 16 hypotheses; q_off holds g rows already)
        return ((unsigned)act >> g & 1u) && q_off[h] != kNowhere ? q_off[h] + (p_row(g, other) - g) * H * (int)sizeof(float) : kNowhere;
    };
    if constexpr (LAYERS == 1) {
        const int quad = lane & 15, g = q_hyp();
#pragma unroll
        for (int h = 0; h < QH; ++h) {
            const int t = h * 4 + (quad >> 2), col = (qt0 + t) * CT + (quad & 3) * 4, u = (t - na) * 4 + (quad & 3);
            const bool row = g < G && lane < (qpack ? 16 : qpair ? 32 : 64);
            if (row && t < na && col < H) q_off[h] = (g * H + col) * (int)sizeof(float);
            if (row && t >= na && t < nq && u < U) q_unit[h] = g * Upad + u;
            q_bias[h] = *reinterpret_cast<const float4 *>(p.b_pred + (t < na && col < H ? col : 0));
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int idx = tid + h * THREADS;
            c_g[h] = U > 0 ? min(idx / max(U, 1), kLabelMaxHyps - 1) : kLabelMaxHyps - 1;
            c_u[h] = U > 0 ? idx - idx / max(U, 1) * U : 0;
            if (U > 0 && idx < G * U) {
                if constexpr (PLANES) {   // (of two neighbours the one stores the pairs of first and of last terms, the other those between)
                    const int k = u0 + c_u[h], odd = k & 1;
                    h_off[h] = (k >> 5) * hstep + ((k >> 3 & 3) * 3 * RP + odd * RP + c_g[h]) * 16 + (k & 6) * 2;
                    if (!odd) h_off2[h] = h_off[h] + 2 * RP * 16;
                } else {
                    h_off[h] = (c_g[h] * Hp + u0 + c_u[h]) * (int)sizeof(float);
                }
            }
        }
    }
    // ---- WIDE: R row tiles from tile tb on against this workgroup's columns.  What bounds a pass over
    // an output layer of many thousands of columns is the stream of weights into a compute unit
    // (64 bytes a clock) and, from two row tiles on, its matrix cores (three products per weight
    // fragment and row tile).  So: two row tiles share one stream; a wavefront keeps the activations
    // of its eighth of the reduction in registers and reads of the weights only that eighth; a batch
    // of TB tiles is multiplied while the next one is on its way into the registers it leaves, step by step, and the
    // sums of the one before go through LDS into running statistics, two columns a thread, by pieces between
    // the products of the batch's second half: the barrier they need stands in its middle, where no
    // wavefront waits for another's last product.  The three planes of a product share one accumulator, smallest first within a
    // step (registers); score error against 64 bits at 8198 outputs, joint width 1024: 2.2e-6 rms per root of
    // a label count, 2.8e-6 in decode.hip's streaming pass, which keeps three and adds the smallest first.
    // Measured at 8198 outputs, joint width 1024, 16 workgroups a group (33 tiles each), a call at B = 256: 33.6
    // ms; with rows staged by 128-byte pieces 32.4; the next batch's weights requested step by step as well (not
    // all at the end of a batch) 31.9; the barrier in the middle as well 30.3.  Two row tiles take 0.95 us a
    // batch of two tiles, of which the matrix cores need 0.8 (96 products a SIMD, 18 cycles each at 2.1 GHz);
    // one takes 1.2 us a batch of four (the stream of weights alone 1.05 us: 126 GB/s a compute unit).
    auto wide_rows = [&](auto rtag, int tb, int jbb, int jlb, int jdb) __attribute__((always_inline)) {
        constexpr int R = decltype(rtag)::value, TB = 4 / R, PW = TB * CT + 4;
        constexpr int CPT = 2, QR = TB * CT / CPT;   // columns a thread looks at, threads of a row
        constexpr int PB = NW * R * RT * PW;         // floats of a buffer of partial sums (of two)
        static_assert(2 * PB <= NW * RT * kWidePart, "two buffers");
        fresh();
        TR(40);
        v4u b[TB][NK];
        const int last_t = n_ct - 1;
        auto fetch_tile = [&](auto &bt, int t) __attribute__((always_inline)) {   // tile t, or the last
            const int w = p.off_w_out + (tile0 + min(t, last_t)) * jbytes + js0 * 1024;
#pragma unroll
            for (int s = 0; s < NK; ++s)
                bt[s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, s < jsn ? lane * 16 : ~0xff, w + (s < jsn ? s : 0) * 1024, 0);
        };
        AFrag a[R][NK][PL];
        {
            // rows change lanes through LDS as in the other forms, one row tile after the other in one area (the partial
            // sums', which nobody looks at between the row tiles)
            v4u e[R][2 * C32], q[R][2 * C32];
            int po[R][2], prow[R];
            bool upper[R];   // more than eight hypotheses in the row tile
#pragma unroll
            for (int r = 0; r < R; ++r) {
                any_value(q[r]);
                ti = tb + r;
                set_rows();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int er = __builtin_amdgcn_ds_bpermute((h * 8 + (lane >> 3)) * 4, erow_l);
                    const float *at = p.enc_proj + (size_t)(unsigned)er * H;
#pragma unroll
                    for (int i = 0; i < C32; ++i) e[r][h * C32 + i] = ldg4(at, flat_off(i, js0, H));
                }
                const int q0 = uni(q_l), q1 = __builtin_amdgcn_readlane(q_l, 15);
                prow[r] = q_l - q0;
                upper[r] = q1 - q0 >= 8;
#pragma unroll
                for (int h = 0; h < 2; ++h) {   // (rows beyond the last: the last again)
                    const int g = __builtin_amdgcn_ds_bpermute(min(q0 + h * 8 + (lane >> 3), q1) * 4, slot_of) & 63;
                    if constexpr (LSTM) {
                        po[r][h] = p_row(g, 0) * H * (int)sizeof(float);
                    } else if (h == 0 || upper[r]) {
                        const int lab = __builtin_amdgcn_ds_bpermute(g * 4, last), lab2 = __builtin_amdgcn_ds_bpermute(g * 4, last2);
                        const float *t = p.pred_tab + (size_t)(p.pred_layers == 2 ? lab2 : lab) * H;
#pragma unroll
                        for (int i = 0; i < C32; ++i) q[r][h * C32 + i] = ldg4(t, flat_off(i, js0, H));
                        if (p.pred_layers == 2) {
                            t = p.pred_tab + ((size_t)(V + 1) + lab) * H;
#pragma unroll
                            for (int i = 0; i < C32; ++i) {
                                const float4 y = as_float4(ldg4(t, flat_off(i, js0, H))), z = as_float4(q[r][h * C32 + i]);
                                q[r][h * C32 + i] = v4u{__float_as_uint(z.x + y.x), __float_as_uint(z.y + y.y),
                                                        __float_as_uint(z.z + y.z), __float_as_uint(z.w + y.w)};
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < TB; ++t) fetch_tile(b[t], t);
            if constexpr (LSTM) {
                until_there([&]() __attribute__((always_inline)) {
                    unsigned mx = 0;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
#pragma unroll
                        for (int i = 0; i < C32; ++i) q[r][i] = ldx4(prs, po[r][0] + flat_off(i, js0, H), 0);
                        if (upper[r])
#pragma unroll
                            for (int i = 0; i < C32; ++i) q[r][C32 + i] = ldx4(prs, po[r][1] + flat_off(i, js0, H), 0);
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
#pragma unroll
                        for (int i = 0; i < C32; ++i) mx = max(mx, umax4(q[r][i]));
                        if (upper[r])
#pragma unroll
                            for (int i = 0; i < C32; ++i) mx = max(mx, umax4(q[r][C32 + i]));
                    }
                    return mx;
                });
                lap(kTkBar);
                TR(41);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float4 z[NK][NL];
                stage_rows(xe, q[r], upper[r]);
#pragma unroll
                for (int s = 0; s < NK; ++s)
#pragma unroll
                    for (int l = 0; l < NL; ++l) z[s][l] = staged(xe, prow[r], s, l);
                stage_rows(xe, e[r], true);
#pragma unroll
                for (int s = 0; s < NK; ++s) {
                    float x[F::E];
#pragma unroll
                    for (int l = 0; l < NL; ++l) {
                        const float4 y = staged(xe, lane & 15, s, l);
                        x[l * 4] = fmaxf(y.x + z[s][l].x, 0.0f);
                        x[l * 4 + 1] = fmaxf(y.y + z[s][l].y, 0.0f);
                        x[l * 4 + 2] = fmaxf(y.z + z[s][l].z, 0.0f);
                        x[l * 4 + 3] = fmaxf(y.w + z[s][l].w, 0.0f);
                    }
                    split(x, a[r][s], alone);
                }
            }
        }
        fresh();
        TR(42);
        const int row = tid / QR, quad = tid % QR;   // this thread's row (of R * 16) and columns of a batch
        constexpr float kNone = -3.4e38f;
        float rm = kNone, rs = 0.0f, rdm = -INFINITY;
        int ra = 0x7fffffff, rda = 0;
        f32x4 acc[TB][R];
        float bias[CPT], x4[CPT];
        // The products of batch k; each tile's registers then take the same tile of the next batch.  Of the
        // eight groups of products every one is followed by a piece of other work (piece(0) .. piece(7)):
        // the other wavefront of the SIMD multiplies meanwhile.
        auto multiply = [&](int k, auto piece) __attribute__((always_inline)) {
            const int bo = ((tile0 + k * TB) * CT + quad * CPT) * (int)sizeof(float);
#pragma unroll
            for (int e = 0; e < CPT; ++e) bias[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(brs, bo + e * 4, 0, 0));
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int r = 0; r < R; ++r) acc[t][r] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int g = 0; g < 8; ++g) {   // R == 1: two tiles, one step a group; R == 2: two tiles, half a step (three products each)
                const int t = R == 1 ? g / NK * 2 : 0, s = R == 1 ? g % NK : g / 2;
#pragma unroll
                for (int pl = PL - 1; pl >= 0; --pl)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int r = R == 1 ? 0 : g % 2;
                        acc[t + u][r] = F::mma(a[r][s][pl], b[t + u][s], acc[t + u][r]);
                    }
                if (R == 1 || g % 2 == 1)   // this step's weights of the next batch
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int w = p.off_w_out + (tile0 + min((k + 1) * TB + t + u, last_t)) * jbytes + js0 * 1024;
                        b[t + u][s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, s < jsn ? lane * 16 : ~0xff, w + (s < jsn ? s : 0) * 1024, 0);
                    }
                piece(g);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto store = [&](int k) __attribute__((always_inline)) {
            float *const pw = part_q + (k & 1) * PB + (size_t)wave * R * RT * PW + (lane & 15) * PW + (lane >> 4) * 4;
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int r = 0; r < R; ++r) *reinterpret_cast<f32x4 *>(pw + r * RT * PW + t * CT) = acc[t][r];
        };
        // what is done with the sums of batch k, in eight pieces
        typedef float VC __attribute__((ext_vector_type(CPT)));
        VC lv[NW];
        float lg[CPT], lm, lx[CPT + 1], bb[CPT];
        auto look = [&](int k, int step) __attribute__((always_inline)) {
            if (step == 0) {
                const float *q = part_q + (k & 1) * PB + (size_t)row * PW + quad * CPT;
#pragma unroll
                for (int w = 0; w < NW; ++w) lv[w] = *reinterpret_cast<const VC *>(q + (size_t)w * R * RT * PW);
            } else if (step == 2) {
#pragma unroll
                for (int w = 0; w < NW; w += 2) lv[w] = lv[w] + lv[w + 1];
            } else if (step == 3) {
                lv[0] = (lv[0] + lv[2]) + (lv[4] + lv[6]);
            } else if (step == 4) {
                // (no branches: columns that are not there, and logits that are no numbers, count as kNone, and what
                // stands beside a largest logit of kNone vanishes with the first real one)
                const int t = k * TB + quad * CPT / CT, col0 = t < n_ct ? (tile0 + t) * CT + quad * CPT % CT : O;
                lm = rm;
#pragma unroll
                for (int e = 0; e < CPT; ++e) {   // (columns ascend: '>' keeps the first maximum)
                    x4[e] = lv[0][e] + bb[e];
                    lg[e] = fmaxf(col0 + e <= VL ? x4[e] : kNone, kNone);
                    ra = lg[e] > lm ? col0 + e : ra;
                    lm = fmaxf(lm, lg[e]);
                }
            } else if (step == 5) {
                lx[CPT] = __expf(rm - lm);
#pragma unroll
                for (int e = 0; e < CPT; ++e) lx[e] = __expf(lg[e] - lm);
                rm = lm;
            } else if (step == 6) {
                rs *= lx[CPT];
#pragma unroll
                for (int e = 0; e < CPT; ++e) rs += lx[e];
            }
        };
        auto durations = [&](int k) __attribute__((always_inline)) {
            if (cg >= dcg0 && cg <= dcg1) {   // (uniform; never without a duration head)
                const int t = k * TB + quad * CPT / CT, col0 = t < n_ct ? (tile0 + t) * CT + quad * CPT % CT : O;
#pragma unroll
                for (int e = 0; e < CPT; ++e)
                    if (col0 + e > VL && col0 + e < O && x4[e] > rdm) { rdm = x4[e]; rda = col0 + e - (VL + 1); }
            }
        };
        const int batches = (n_ct + TB - 1) / TB;
        multiply(0, [](int) {});
        TR(43);
        __syncthreads();   // the partial sums are not read any more (phase Q, the rows before)
        store(0);
#pragma clang loop unroll(disable)
        for (int k = 1; k < batches; ++k) {
#pragma unroll
            for (int e = 0; e < CPT; ++e) bb[e] = bias[e];
            multiply(k, [&](int g) __attribute__((always_inline)) {
                if (g == 3) __syncthreads();
                if (g > 3) {
                    constexpr int per = (8 + 6 - 3) / (7 - 3);
#pragma unroll
                    for (int st = (g - 3 - 1) * per; st < (g - 3) * per; ++st) look(k - 1, st);
                }
            });
            durations(k - 1);
            store(k);   // (into the buffer that was looked at before the barrier)
            TR(44);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < CPT; ++e) bb[e] = bias[e];
#pragma unroll
        for (int step = 0; step < 8; ++step) look(batches - 1, step);
        durations(batches - 1);
        // the threads of a row
        auto fmax2 = [](float x, float y) { return fmaxf(x, y); };
        auto imin2 = [](int x, int y) { return min(x, y); };
        auto fadd2 = [](float x, float y) { return x + y; };
        auto over_row = [&](auto v, auto op) __attribute__((always_inline)) {
            v = row_allreduce(v, op);
            if constexpr (QR == 32) {   // (two rows of lanes)
                unsigned u;
                __builtin_memcpy(&u, &v, 4);
                const auto x = __builtin_amdgcn_permlane16_swap(u, u, false, false);
                decltype(v) y, z;
                const unsigned x0 = x[0], x1 = x[1];
                __builtin_memcpy(&y, &x0, 4);
                __builtin_memcpy(&z, &x1, 4);
                v = op(y, z);
            }
            return v;
        };
        const float m = over_row(rm, fmax2);
        const int am = over_row(rm == m ? ra : 0x7fffffff, imin2);
        const float sum = over_row(rs * __expf(rm - m), fadd2);
        float dm = -INFINITY;
        int da = 0;
        if (cg >= dcg0 && cg <= dcg1) {
            dm = over_row(rdm, fmax2);
            da = over_row(rdm == dm ? rda : 0x7fffffff, imin2);
        }
        TR(45);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (words put back earlier have arrived ...
        __syncthreads();                                   // ... those of all wavefronts)
        if (quad == 0) {
            const int i = row & 15, tr = tb + row / RT, o = (tr * n_cg + cg) * RT + i;
            const unsigned long long best = m > kNone ? pack_best(m, am) : 1ull;
            const unsigned long long bd = dm > -INFINITY ? pack_best(dm, da) : 1ull;
            const unsigned long long lse = (unsigned long long)__float_as_uint(m) |
                                           ((unsigned long long)__float_as_uint(m > kNone ? sum : 0.0f) << 32);
            if (C > 1) {
                st_word(o * 8, jbb, best);
                if (cg == dcg0) st_word((tr * 2 * RT + i) * 8, jdb, bd);
                else if (cg == dcg1) st_word(((tr * 2 + 1) * RT + i) * 8, jdb, bd);
                st_word(o * 8, jlb, lse);
            } else {
                S.rowb[tr * RT + i] = best;
                S.rowl[tr * RT + i] = lse;
                S.rowd[tr * RT + i] = (unsigned)S.durations[unpack_index(bd) & (TDT_MAX_DURATIONS - 1)];
            }
        }
        lap(kTkJ);
    };

    // Weights that stay (see the head of the file).  Phase Q's, of both rounds where it has two; those of a joint pass's
    // first round; and of its second where items have two, in stateless groups and in groups of so few workgroups
    // that phase Q has two rounds as well.  Registers hold two of the four kinds in bfloat16 and three in float32's
    // longest form.  bfloat16: phase Q's (config 2 at B = 128, the joint rounds' and none of phase Q's 1555 us, 18 registers
    // in scratch, phase Q's first round only 1507, both 1502; 1024 units and joint width, B = 24, 7388, 7314, 7067; all
    // kept 1700 and more).  Float32: not phase Q's second, requested for every label behind its table row (config 2's
    // model, B = 16, 1207; with it, 53 registers in scratch, 1249).  Nothing kept, the code before, against
    // what one round of phase Q keeps: stateless at B = 128 2.42 ms, 2.19; config 2 at B = 32 1.47 ms, 1.32, at B = 1 375 us,
    // 351.
    constexpr bool KEEP1 = STAGED && !(TWO_ROUNDS && PL == 3), KEEP2 = KEEP1 && (LAYERS == 0 || TWO_ROUNDS), KEEPQ2 = PL == 3 || NK <= 4;
    v4u bq[TR][NK], bq2_kept[TR][NK];   // LAYERS == 1: the predictor-side weights, of the first TR tiles and of the others
    auto fetch_second = [&](auto &w) __attribute__((always_inline)) { fetch(w, nq - TR, hs0, hsn, [&](int t) { return q_tile(TR + t); }); };
    if constexpr (LAYERS == 1) fetch(bq, min(nq, TR), hs0, hsn, q_tile);
    if constexpr (TWO_ROUNDS && KEEPQ2) fetch_second(bq2_kept);
    v4u b[TJ][NK];    // the first column tiles of the work item at hand, and which
    v4u b2[TR][NK];   // ... and those of later rounds
    v4u bias0[JH], bias1[1];
    int in_b = -1, in_b2 = -1;
    // LAYERS == 1: the table rows of this thread's cells, by the last labels of their hypotheses.  They are requested as soon as a
    // pass is known to be the label's last, ahead of what else is left to do of it -- but for chunks in float32 with more than few rows,
    // where they are registers too many (640 units and joint width, B = 64, 1820 / 1809 us; 256, 1470 / 1455).
    v4u t4[2];
    any_value(t4);
    auto request_gates = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (h == 0 || G * U > THREADS) {   // uniform
                const int lab = __builtin_amdgcn_ds_bpermute(c_g[h] * 4, last);
                t4[h] = *(const TDT_GLOBAL v4u *)(p.emb_gates + ((size_t)lab * Hp + u0 + c_u[h]) * 4);
            }
    };
    if constexpr (EARLY_GATES) request_gates();
#pragma clang loop unroll(disable)
    while (ok) {   // ---- Alg. 3 line 5: while any hypothesis is active
        const unsigned long long alive = __ballot(active);
        if (alive == 0ull) break;
        const unsigned long long act = alive & ~needm;   // who takes a predictor step: not those in the middle of a search
        if (OWN) own ^= act;
        st_pred_passes += 1;
#if TDT_TRACE
        if (tid == 0) g_tr_on = (st_pred_passes >= 20 && st_pred_passes < 24);
#endif
        TR(1);
        st_pred_rows += __popcll(CHUNKED && first ? act & ~carried : act);
        // who will search in the first joint pass (in a chunk a hypothesis may only be here for the
        // predictor step of its last label)
        bool need = active && !(CHUNKED && (time >= len || (status & TDT_HYP_TRUNCATED)));
        needm = CHUNKED ? __ballot(need) : alive;

        // the projected encoder frames of a work item: this wavefront's stretch of its rows
        v4u e4[NK][NL], ev[2 * C32];   // (not wide; staged: ev)
        have_p = false;
        auto request_rows = [&]() __attribute__((always_inline)) {
            if constexpr (STAGED) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int e = __builtin_amdgcn_ds_bpermute((h * 8 + (lane >> 3)) * 4, erow_l);
                    const float *er = p.enc_proj + (size_t)(unsigned)e * H;
#pragma unroll
                    for (int i = 0; i < C32; ++i) ev[h * C32 + i] = ldg4(er, flat_off(i, js0, H));
                }
                return;
            }
            const float *er = p.enc_proj + (size_t)(unsigned)erow_l * H;
#pragma unroll
            for (int s = 0; s < NK; ++s)
#pragma unroll
                for (int l = 0; l < NL; ++l) e4[s][l] = ldg4(er, part_of(s, js0, H) + l * 16);
        };
        fresh();
        v4u bq2_now[TR][NK];
        auto &bq2 = KEEPQ2 ? bq2_kept : bq2_now;
        if constexpr (LAYERS == 1) {
            // ---- P: the cell update (one or two units a thread).  W_ih * emb[label] + b is a table row, requested behind the decision
            // (request_gates); W_hh * h was formed by this workgroup when h was new.
            const bool two_cells = G * U > THREADS;   // uniform
            if constexpr (!EARLY_GATES) request_gates();
            __builtin_amdgcn_sched_barrier(0);
            if (TWO_ROUNDS && !KEEPQ2) fetch_second(bq2);   // (they take about as long to leave as the row to arrive)
            __builtin_amdgcn_sched_barrier(0);
            // (waited for here, in all lanes: behind a branch that some lanes or workgroups skip the compiler takes the
            // loads for pending still and waits for what was sent after them, the published hidden state)
            asm volatile("" ::"v"(t4[0]), "v"(t4[1]));
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (h == 0 || two_cells) {
                    const bool there = h_off[h] != kNowhere && ((act >> c_g[h]) & 1ull);
                    float hn = 0.0f;
                    if (there) {
                        const int o = c_g[h] * Upad + c_u[h];
                        float cn;
                        if (CHUNKED && first && ((carried >> c_g[h]) & 1ull)) {
                            const size_t src = (size_t)S.gid[c_g[h]] * Hp + u0 + c_u[h];
                            hn = p.st_h[src];
                            cn = p.st_c[src];
                        } else {
                            const float4 r4 = rg_l[o], x = as_float4(t4[h]);
                            cell(make_float4(r4.x + x.x, r4.y + x.y, r4.z + x.z, r4.w + x.w), c_l[o], cn, hn);
                        }
                        c_l[o] = cn;
                        if (CHUNKED) h_l[o] = hn;
                    }
                    if constexpr (PLANES) {
                        // (in all lanes: neighbours exchange terms.  A NaN becomes the one whose terms are not all ones.)
                        hn = hn == hn ? hn : __uint_as_float(0x7fc00000u);
                        const float r = hn - __uint_as_float(__float_as_uint(hn) & 0xffff0000u);
                        const float r2 = r - __uint_as_float(__float_as_uint(r) & 0xffff0000u);
                        auto neighbour = [](float x) { return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), 0xb1, 0xf, 0xf, false)); };   // quad_perm 1 0 3 2
                        const bool odd = tid & 1;
                        const float from = neighbour(odd ? hn : r), from2 = neighbour(r2);
                        const unsigned w0 = top_halves(odd ? from : hn, odd ? r : from), w1 = top_halves(r2, from2);
                        const int at = plane_base(par);
                        __builtin_amdgcn_raw_buffer_store_b32(w0, hrs, there ? h_off[h] : kNowhere, at, 16 /* sc1 */);
                        __builtin_amdgcn_raw_buffer_store_b32(w1, hrs, there ? h_off2[h] : kNowhere, at, 16 /* sc1 */);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(present(hn)), hrs, there ? h_off[h] : kNowhere,
                                                              (par * Bw + b0) * Hp * (int)sizeof(float), 16 /* sc1 */);
                    }
                }
        }
        if constexpr (DEEP) {
            // ---- P: the first layer's cell update.  W_ih * emb[label] + b is a table row,
            // W_hh * h was formed by this workgroup when h was new.
#pragma clang loop unroll(disable)
            for (int base = 0; base < G * U; base += 2 * THREADS) {   // uniform
                int g[2], u[2];
                v4u t4[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {   // (both table rows are requested before either is used)
                    place(base, h, g[h], u[h]);
                    const int lab = __builtin_amdgcn_ds_bpermute(min(g[h], kLabelMaxHyps - 1) * 4, last);
                    t4[h] = *(const TDT_GLOBAL v4u *)(p.emb_gates + ((size_t)lab * Hp + u0 + u[h]) * 4);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (g[h] < G && ((act >> g[h]) & 1ull)) {
                        const int o = g[h] * Upad + u[h];
                        float cn, hn;
                        if (CHUNKED && first && ((carried >> g[h]) & 1ull)) {
                            const size_t src = (size_t)S.gid[g[h]] * Hp + u0 + u[h];
                            hn = p.st_h[src];
                            cn = p.st_c[src];
                        } else {
                            const float4 r4 = rg_l[o], x = as_float4(t4[h]);
                            cell(make_float4(r4.x + x.x, r4.y + x.y, r4.z + x.z, r4.w + x.w), c_l[o], cn, hn);
                        }
                        c_l[o] = cn;
                        if (CHUNKED) h_l[o] = hn;
                        st_co(hx + ((size_t)par * L * Bw + b0 + g[h]) * Hp + u0 + u[h], present(hn));
                    }
            }
        }
        if constexpr (LSTM) {
            TR(2);
            // ---- while the hidden state travels: what was exchanged for the label before is put back, and the first joint
            // pass is set up
            fresh();
            if constexpr (LAYERS == 1) {
                const v4u absent = {kAbsent, kAbsent, kAbsent, kAbsent};
                const int pb = (par ^ 1) * Bw + b0;
                const int h_at = PLANES ? plane_base(par ^ 1) : pb * Hp * (int)sizeof(float);
                __builtin_amdgcn_raw_buffer_store_b32(kAbsent, hrs, h_off[0], h_at, 16 /* sc1 */);
                if (PLANES) __builtin_amdgcn_raw_buffer_store_b32(kAbsent, hrs, h_off2[0], h_at, 16 /* sc1 */);
                if (G * U > THREADS) {
                    __builtin_amdgcn_raw_buffer_store_b32(kAbsent, hrs, h_off[1], h_at, 16 /* sc1 */);
                    if (PLANES) __builtin_amdgcn_raw_buffer_store_b32(kAbsent, hrs, h_off2[1], h_at, 16 /* sc1 */);
                }
                __builtin_amdgcn_raw_buffer_store_b128(absent, prs, q_at(0, act, 1), q_base(1), 16 /* sc1 */);
                if (QH > 1 && nq > 4) __builtin_amdgcn_raw_buffer_store_b128(absent, prs, q_at(1, act, 1), q_base(1), 16 /* sc1 */);
            } else {
                clear_rows(act);
            }
            clear_cells();
            if (needm != 0ull) {
                plan_pass(needm);
                set_item(rank);   // (a workgroup without a work item: never used)
                if (!WIDE && rank < items) request_rows();
            }
            TR(3);
            if (wave == NW - 1) finish_scores();
            fresh();
            TR(10);
            lap(kTkP);
            if constexpr (LAYERS == 1) {
                // ---- Q
                // What a thread takes of the sums of half h, four columns of a row.
                // Planes: a wavefront takes a row, or two, its lanes one tile row each, and the planes are added up.
                auto look = [&](int h) __attribute__((always_inline)) {
                    const int quad = lane & 15, row = qpack   ? wave + (lane >> 4) * kPackRows
                                                      : qpair ? wave * 2 + ((lane >> 4) & 1) + (lane >> 5) * kPairRows
                                                              : tid >> 4;
                    float4 v = gather(q_tiles, part_q, row, h * 16 + quad);
                    if (qpack) {   // (rows 12 .. 15 of a packed tile are nobody's)
                        v.x = sum_over_rows(lane < 48 ? v.x : 0.0f);
                        v.y = sum_over_rows(lane < 48 ? v.y : 0.0f);
                        v.z = sum_over_rows(lane < 48 ? v.z : 0.0f);
                        v.w = sum_over_rows(lane < 48 ? v.w : 0.0f);
                    } else if (qpair) {
                        v.x = sum_over_halves(v.x);
                        v.y = sum_over_halves(v.y);
                        v.z = sum_over_halves(v.z);
                        v.w = sum_over_halves(v.w);
                    }
                    const v4u o = {__float_as_uint(present(v.x + q_bias[h].x)), __float_as_uint(present(v.y + q_bias[h].y)),
                                   __float_as_uint(present(v.z + q_bias[h].z)), __float_as_uint(present(v.w + q_bias[h].w))};
                    __builtin_amdgcn_raw_buffer_store_b128(o, prs, q_at(h, act, 0), q_base(0), 16 /* sc1 */);
                    if (q_unit[h] >= 0 && ((unsigned)act >> q_hyp() & 1u)) rg_l[q_unit[h]] = v;   // the four gates of one unit
                };
                if constexpr (PLANES) {
                    // The encoder's rows are staged behind the first look for the hidden state, ahead of which they were requested: a wait
                    // for it is a wait for them, and behind phase Q staging them was 1.5 % of a call.
                    bool rows_wait = needm != 0ull && rank < items;
                    // (A copy of everything up to the published results for each number of tiles: with one behind them that all three lead to,
                    // which needs no more than their tags, calls were 3.5 % slower.)
                    auto planes_of = [&](auto nt) __attribute__((always_inline)) {
                        constexpr int NT = decltype(nt)::value;
                        v4u v[NT][NK];
                        int off[NT][NK];
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            const int r = t * RT + (lane & 15), g = r & (RP - 1);
                            const bool row = r < 3 * RP && ((unsigned)act >> g & 1u);
#pragma unroll
                            for (int s = 0; s < NK; ++s)   // (zeros where there is nothing)
                                off[t][s] = row && s < hsn && (hs0 + s) * 32 + (lane >> 4) * 8 < Hp ? ((lane >> 4) * 3 * RP + r) * 16 : kNowhere;
                        }
                        // (reductions to 640: formed ahead of the loop that polls; in it they are a selection a step and turn, config 2 at B = 1
                        // 500 / 495 us.  Longer ones: see planes_covered.)
                        const int first_at = plane_base(par) + hs0 * hstep;
                        int at[NK];
                        any_value(at);
                        if constexpr (NK <= 5)
#pragma unroll
                            for (int s = 0; s < NK; ++s) at[s] = here(first_at + plane_step_at(hstep, hsn, s));
                        until_there([&]() __attribute__((always_inline)) {
                            unsigned mx = 0;
#pragma unroll
                            for (int t = 0; t < NT; ++t)
#pragma unroll
                                for (int s = 0; s < NK; ++s) v[t][s] = ldx4(hrs, off[t][s], NK <= 5 ? at[s] : first_at + s * hstep);
                            if (rows_wait) {   // uniform
                                stage_rows(xe, ev, true);
                                rows_wait = false;
                            }
#pragma unroll
                            for (int t = 0; t < NT; ++t)
#pragma unroll
                                for (int s = 0; s < NK; ++s) mx = max(mx, umax4(v[t][s]));
                            return mx;
                        });
                        TR(11);
                        lap(kTkBar);
                        plane_products(r_tiles, v, bq, q_tiles, part_q);
                        if (TWO_ROUNDS && nq > TR) plane_products(r_tiles, v, bq2, q_tiles, part_q + TR * CT);   // uniform
                        TR(14);
                        __syncthreads();
                        look(0);
                        if (QH > 1 && nq > 4) look(1);
                        TR(16);
                    };
                    if (nq > 0) {
                        if (qpack) planes_of(std::integral_constant<int, 1>{});
                        else if (qpair) planes_of(std::integral_constant<int, 2>{});
                        else planes_of(std::integral_constant<int, 3>{});
                    } else if (rows_wait) {
                        stage_rows(xe, ev, true);
                    }
                } else if (nq > 0) {
                    AFrag a[NK][PL];
                    stage_h(a, par * Bw + b0, 0, act);
                    lap(kTkBar);
                    fresh();
                    TR(14);
                    if constexpr (FEW) {
                        few_products(bq, bq2, q_tiles, part_q);
                    } else if constexpr (TQ == TR) {
                        products(full_rows, a, bq, nq, q_tiles, hsn, part_q);
                    } else {
                        products_of(full_rows, r_tiles, a, bq, q_tiles, hsn, part_q);
                        if (nq > TR) products_of(full_rows, r_tiles, a, bq2, q_tiles, hsn, part_q + TR * CT);
                    }
                    TR(15);
                    __syncthreads();
                    TR(16);
                    fresh();
#pragma unroll
                    for (int h = 0; h < QH; ++h)
                        if (h == 0 || nq > 4) look(h);   // uniform
                }
            }
            const int ntq = (G + RT - 1) / RT;
            // ---- eight wavefronts: the column tiles that a row tile of a layer's h is multiplied by are two lists, what somebody waits
            // for -- the next layer's input product with its cells, at the top W_pred -- and the recurrent product for the
            // next label, which is formed while the first one's results travel.  What bounds a list is the stream of its
            // weights (64 bytes a clock, at some 1.7 GHz: ten tiles of 640 inputs 1.9 us, the list takes 2.5) and, with all
            // sixteen rows, nearly as many cycles of the matrix cores.  So the weights run through registers of two tiles from
            // list to list, requested step by step where they have been multiplied, steps that a wavefront has not are left out,
            // and a list has one look at its sums.  Rounds of six tiles, fetched, multiplied and looked at one after the other, took a
            // label of two layers 30 us where it now takes 20: 8198 outputs, 640 units, B = 256, 27.7 / 25.4 ms; B = 110, 7.76
            // / 6.84 ms; B = 32, 3.53 / 3.40 ms; B = 1, 418 / 415 us.  Registers of four tiles are no faster (B = 256 25.6 ms, two
            // 25.5; B = 32 3.56, 3.41), nor is a compiled reduction of four steps where there are three (25.9).
            if constexpr (LISTS) {
                constexpr int TS = 2;
                const int room = wide_tiles(p.wide_part), PLW = room * CT + 4;
                v4u b[TS][NQ];
                // (The scalar offset is made uniform by hand: the compiler does not see that it is, and put a loop over the wavefront's different
                // values, of which there is one, around every request.  Joint width 1024, B = 32, one layer of 640 units 682 / 666 us, two 1110
                // / 1074, in chunks 1863 / 1794; 1024 units, two layers, in chunks, where four registers were in scratch memory, 1970 / 1842.)
                auto request = [&](int u, int s, int n, int base) __attribute__((always_inline)) {   // tile u of the n that start at base, or nothing
                    const int w = uni(base + (u < n ? u : 0) * hbytes + (hs0 + (s < hsn ? s : 0)) * 1024);
                    b[u][s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, u < n && s < hsn ? lane * 16 : ~0xff, w, 0);
                };
                auto request_all = [&](int n, int base) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < TS; ++u)
#pragma unroll
                        for (int s = 0; s < NQ; ++s) request(u, s, n, base);
                };
                // One list, and which tiles follow it, of a tile of `rows` rows.  pre(t, i, j): what use(t, i, j, sums, pre, out, off) takes beside
                // the sums of row i's columns j * 4 .. + 3 of tile t (rows and tiles that are not there as well); publish(out, off)
                // takes place in all lanes: behind a branch its stores would be waited for with the weights.
                auto list = [&](const AFrag (&a)[NQ][PL], int rows, int n, int base, int n_next, int base_next, auto pre, auto use, auto publish) __attribute__((always_inline)) {
                    if (n == 0) request_all(n_next, base_next);
#pragma clang loop unroll(disable)
                    for (int t1 = 0; t1 < n; t1 += room) {   // as many tiles as there is room for
                        const int np = min(room, n - t1), n4 = np * 4;
                        const int rn1 = t1 + room < n ? n - t1 - room : n_next, rat1 = t1 + room < n ? base + (t1 + room) * hbytes : base_next;
                        fresh();
                        TR(14);
                        // a thread looks at four columns of a row, or two times four: idx / n4 and the rest
                        const int rcp = uni((int)(1048576.0f * __builtin_amdgcn_rcpf((float)n4)) + 2);
                        int row[2], quad[2];
                        float4 extra[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int idx = h * THREADS + tid;
                            row[h] = (idx * rcp) >> 20;
                            quad[h] = idx - row[h] * n4;
                            extra[h] = pre(t1 + (quad[h] >> 2), row[h], quad[h] & 3);
                        }
                        float *const pw = part_q + (size_t)wave * RT * PLW + (lane & 15) * PLW + (lane >> 4) * 4;
#pragma clang loop unroll(disable)
                        for (int t0 = 0; t0 < np; t0 += TS) {
                            const int rn = t0 + TS < np ? np - t0 - TS : rn1, rat = t0 + TS < np ? base + (t1 + t0 + TS) * hbytes : rat1;
                            f32x4 c[TS];
#pragma unroll
                            for (int u = 0; u < TS; ++u) c[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                            for (int s = 0; s < NQ; ++s) {
                                if (s < NK / 2 || s < hsn)   // uniform
#pragma unroll
                                    for (int pl = PL - 1; pl >= 0; --pl)
#pragma unroll
                                        for (int u = 0; u < TS; ++u) c[u] = F::mma(a[s][pl], b[u][s], c[u]);
#pragma unroll
                                for (int u = 0; u < TS; ++u) request(u, s, rn, rat);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                            if (t0 == 0) __syncthreads();   // the partial sums before are not read any more
#pragma unroll
                            for (int u = 0; u < TS; ++u)
                                if (t0 + u < np) *reinterpret_cast<f32x4 *>(pw + (t0 + u) * CT) = c[u];
                        }
                        TR(15);
                        __syncthreads();
                        TR(16);
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            v4u out = {0u, 0u, 0u, 0u};
                            int off = kNowhere;
                            if (h == 0 || rows * n4 > THREADS) {   // uniform
                                const float *q = part_q + (size_t)min(row[h], RT - 1) * PLW + quad[h] * 4;
                                f32x4 v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                                for (int w0 = 0; w0 < NW; w0 += NW / 2) {   // (registers: half of them at a time)
                                    f32x4 x[NW / 2];
#pragma unroll
                                    for (int w = 0; w < NW / 2; ++w) x[w] = *reinterpret_cast<const f32x4 *>(q + (size_t)(w0 + w) * RT * PLW);
#pragma unroll
                                    for (int w = 0; w < NW / 2; ++w) v = w0 + w == 0 ? x[0] : v + x[w];
                                    __builtin_amdgcn_sched_barrier(0);
                                }
                                use(t1 + (quad[h] >> 2), row[h], quad[h] & 3, make_float4(v.x, v.y, v.z, v.w), extra[h], out, off);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                            publish(out, off);
                        }
                    }
                };
                auto first_of = [&](int l, int &n, int &base) __attribute__((always_inline)) {   // what layer l's h is multiplied by first
                    const bool top = l == L - 1;
                    n = top ? na : nr;
                    base = here((top ? p.off_w_pred + qt0 * hbytes : p.off_w_ih[l + 1] + r0 * hbytes));
                };
                int n0, base0;
                first_of(0, n0, base0);
                request_all(n0, base0);
#pragma clang loop unroll(disable)
                for (int l = 0; l < L; ++l) {
                    const bool top = l == L - 1;
                    first_of(l, n0, base0);
                    int n_up = 0, base_up = 0;
                    if (!top) first_of(l + 1, n_up, base_up);
                    const int base1 = here(p.off_w_hh[l] + r0 * hbytes);
#pragma clang loop unroll(disable)
                    for (int tq = 0; tq < ntq; ++tq) {
                        const unsigned long long in_tile = act >> (tq * RT) & 0xffffull;
                        if (in_tile == 0ull) continue;   // nobody active here (uniform over the group)
                        const bool more = tq + 1 < ntq && act >> (tq * RT + RT) != 0ull;   // another row tile of this layer
                        AFrag a[NQ][PL];
                        stage_h(a, (par * L + l) * Bw + b0, tq, in_tile);
                        lap(kTkBar);
                        const int rows = min(RT, G - tq * RT);
                        auto of_row = [&](int i, int &g) __attribute__((always_inline)) {   // row i is that of an active hypothesis, g
                            g = tq * RT + min(i, RT - 1);
                            return i < RT && g < G && ((act >> g) & 1ull);
                        };
                        if (!top) {
                            const float *const bl = p.b_lstm[l + 1] + u0;
                            list(a, rows, n0, base0, nr, base1,
                                 [&](int t, int, int j) __attribute__((always_inline)) {
                                     const int u = min(t * 4 + j, max(U - 1, 0));
                                     return make_float4(bl[u], bl[Hp + u], bl[2 * Hp + u], bl[3 * Hp + u]);
                                 },
                                 [&](int t, int i, int j, float4 v, float4 bias, v4u &out, int &off) __attribute__((always_inline)) {
                                     const int u = t * 4 + j;
                                     int g;
                                     const bool there = of_row(i, g) && u < U;
                                     const int o = there ? ((l + 1) * hpc + g) * Upad + u : 0;
                                     const float4 r4 = rg_l[o];
                                     float cn, hn;
                                     cell(make_float4(v.x + r4.x + bias.x, v.y + r4.y + bias.y, v.z + r4.z + bias.z, v.w + r4.w + bias.w),
                                          c_l[o], cn, hn);
                                     if (CHUNKED && first && there && ((carried >> g) & 1ull)) {
                                         const size_t at = ((size_t)(l + 1) * B + S.gid[g]) * Hp + u0 + u;
                                         hn = p.st_h[at];
                                         cn = p.st_c[at];
                                     }
                                     if (there) {
                                         c_l[o] = cn;
                                         if (CHUNKED) h_l[o] = hn;
                                     }
                                     out.x = __float_as_uint(present(hn));
                                     off = there ? (((par * L + l + 1) * Bw + b0 + g) * Hp + u0 + u) * (int)sizeof(float) : kNowhere;
                                 },
                                 [&](const v4u &out, int off) __attribute__((always_inline)) {
                                     __builtin_amdgcn_raw_buffer_store_b32(out.x, hrs, off, 0, 16 /* sc1 */);
                                 });
                        } else {
                            list(a, rows, n0, base0, nr, base1,
                                 [&](int t, int, int j) __attribute__((always_inline)) {
                                     return *reinterpret_cast<const float4 *>(p.b_pred + min((qt0 + t) * CT + j * 4, H - 4));
                                 },
                                 [&](int t, int i, int j, float4 v, float4 bias, v4u &out, int &off) __attribute__((always_inline)) {
                                     const int col = (qt0 + t) * CT + j * 4;
                                     int g;
                                     const bool there = of_row(i, g) && t < na && col < H;
                                     out = v4u{__float_as_uint(present(v.x + bias.x)), __float_as_uint(present(v.y + bias.y)),
                                               __float_as_uint(present(v.z + bias.z)), __float_as_uint(present(v.w + bias.w))};
                                     off = there ? (p_row(g, 0) * H + col) * (int)sizeof(float) : kNowhere;
                                 },
                                 [&](const v4u &out, int off) __attribute__((always_inline)) {
                                     __builtin_amdgcn_raw_buffer_store_b128(out, prs, off, 0, 16 /* sc1 */);
                                 });
                        }
                        list(a, rows, nr, base1, more ? n0 : n_up, more ? base0 : base_up,
                             [](int, int, int) __attribute__((always_inline)) { return make_float4(0.0f, 0.0f, 0.0f, 0.0f); },
                             [&](int t, int i, int j, float4 v, float4, v4u &, int &) __attribute__((always_inline)) {
                                 const int u = t * 4 + j;
                                 int g;
                                 if (of_row(i, g) && u < U) rg_l[(l * hpc + g) * Upad + u] = v;
                             },
                             [](const v4u &, int) __attribute__((always_inline)) {});
                        lap(kTkQ);   // (behind every wait what followed it: the next one starts here)
                    }
                }
            }
            // ---- deeper layers: W_ih . [h of the layer below] + what W_hh . h left here
            if constexpr (DEEP && !LISTS)
#pragma clang loop unroll(disable)
            for (int l = 0; l < L; ++l) {
                const int row0 = (par * L + l) * Bw + b0;
                const bool top = l == L - 1;
                // What this layer's h is multiplied by.  Below the top: first the next layer's input
                // product (its cell follows at once), then the recurrent product for the next label;
                // the top layer: the list of W_pred and W_hh tiles in order.
                const int kinds = top ? 1 : 2, n_all = top ? nq : nr;
                v4u b[TQ][NK];
                float4 qbias;
                auto fetch_round = [&](int kind, int t0) __attribute__((always_inline)) {
                    const int n = min(TQ, n_all - t0);
                    const int w = here(top ? 0 : (kind == 0 ? p.off_w_ih[l + 1] : p.off_w_hh[l]) + (r0 + t0) * hbytes);
                    fetch(b, n, hs0, hsn, [&](int t) { return top ? q_tile(t0 + t) + w : w + t * hbytes; });
                    const int t = t0 + (q_quad() >> 2), col = (qt0 + t) * CT + (lane & 3) * 4;
                    qbias = *reinterpret_cast<const float4 *>(p.b_pred + (t < na && col < H ? col : 0));
                };
                bool loaded = false;   // the registers hold the fragments of the first round
#pragma clang loop unroll(disable)
                for (int tq = 0; tq < ntq && n_all > 0; ++tq) {
                    const unsigned long long in_tile = act >> (tq * RT) & 0xffffull;
                    if (in_tile == 0ull) continue;   // nobody active here (uniform over the group)
                    if (!loaded) fetch_round(0, 0);   // while the rows are on their way
                    loaded = !WIDE && top && n_all <= TQ;
                    AFrag a[NK][PL];
                    any_value(a);
                    stage_h(a, row0, tq, in_tile);
                    lap(kTkBar);
                    fresh();
#pragma clang loop unroll(disable)
                    for (int kind = 0; kind < kinds; ++kind) {
                        const bool input = !top && kind == 0;
#pragma clang loop unroll(disable)
                        for (int t0 = 0; t0 < n_all; t0 += TQ) {
                            const int n = min(TQ, n_all - t0);
                            TR(14);
                            if (qpack) products(packed_rows, a, b, n, q_tiles, hsn, part_q);
                            else products(full_rows, a, b, n, q_tiles, hsn, part_q);
                            TR(15);
                            const float4 bias = qbias;
                            if (t0 + TQ < n_all) fetch_round(kind, t0 + TQ);   // while the results are looked at
                            else if (kind + 1 < kinds) fetch_round(kind + 1, 0);
                            __syncthreads();
                            TR(16);
                            fresh();
                            // a thread takes four columns of a row; packed: a wavefront takes a row, its
                            // lanes one plane each, and the planes are added up
                            const int quad = q_quad(), i = qpack ? wave % kPackRows : tid / QPR, g = tq * RT + i;
                            float4 v = gather(q_tiles, part_q, qpack ? i + (lane >> 4) * kPackRows : i, quad);
                            if (qpack) {
                                if (lane >= 48) v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                                v.x = sum_over_rows(v.x);
                                v.y = sum_over_rows(v.y);
                                v.z = sum_over_rows(v.z);
                                v.w = sum_over_rows(v.w);
                            }
                            if (g < G && ((act >> g) & 1ull) && quad < n * 4 && (!qpack || lane < 16)) {
                                const int t = t0 + (quad >> 2);
                                if (top && t < na) {   // projected predictor output
                                    const int col = (qt0 + t) * CT + (quad & 3) * 4;
                                    if (col < H)
                                        st_co4(px + (size_t)p_row(g, 0) * H + col,
                                               make_float4(present(v.x + bias.x), present(v.y + bias.y),
                                                           present(v.z + bias.z), present(v.w + bias.w)));
                                } else {   // the four gates of one unit
                                    const int u = (top ? t - na : t) * 4 + (quad & 3);
                                    if (u < U) {
                                        if (!input) {
                                            rg_l[((size_t)l * hpc + g) * Upad + u] = v;
                                        } else {
                                            const int o = ((l + 1) * hpc + g) * Upad + u;
                                            const float *bl = p.b_lstm[l + 1] + u0 + u;
                                            const float4 r4 = rg_l[o];
                                            float cn, hn;
                                            if (CHUNKED && first && ((carried >> g) & 1ull)) {
                                                const size_t at = ((size_t)(l + 1) * B + S.gid[g]) * Hp + u0 + u;
                                                hn = p.st_h[at];
                                                cn = p.st_c[at];
                                            } else {
                                                cell(make_float4(v.x + r4.x + bl[0], v.y + r4.y + bl[Hp],
                                                                 v.z + r4.z + bl[2 * Hp], v.w + r4.w + bl[3 * Hp]),
                                                     c_l[o], cn, hn);
                                            }
                                            c_l[o] = cn;
                                            if (CHUNKED) h_l[o] = hn;
                                            st_co(hx + (((size_t)par * L + l + 1) * Bw + b0 + g) * Hp + u0 + u,
                                                  present(hn));
                                        }
                                    }
                                }
                            }
                            // (the partial sums are written again behind the next barrier only if another
                            // round, row tile or layer follows; a joint pass has its own)
                            if (t0 + TQ < n_all || kind + 1 < kinds || tq + 1 < ntq || l + 1 < L) __syncthreads();
                        }
                    }
                    lap(kTkQ);   // (behind every wait what followed it: the next one starts here)
                }
            }
            TR(17);
            lap(kTkQ);
        }
        if (CHUNKED) {
            active = need;
            if (needm == 0ull) {   // nobody scores a frame any more: the loop ends at its test
                act_prev = act;
                first = false;
                par ^= 1;
                continue;
            }
        }
        if constexpr (!LSTM) plan_pass(needm);
        // (TWO, LSTM) this label's rows of the projected predictor output are staged; the others' are still there
        auto take_p = [&](unsigned long long rows, v4u (&v)[2 * C32]) __attribute__((always_inline)) {
            int off[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int g = h * 8 + (lane >> 3);
                off[h] = (rows >> g) & 1ull ? (par * Bw + b0 + g) * H * (int)sizeof(float) : kNowhere;
            }
            const bool upper = (rows >> 8) != 0ull;
            until_there([&]() __attribute__((always_inline)) {
                unsigned mx = 0;
#pragma unroll
                for (int i = 0; i < C32; ++i) v[i] = ldx4(prs, off[0] + flat_off(i, js0, H), 0);
                if (upper)
#pragma unroll
                    for (int i = 0; i < C32; ++i) v[C32 + i] = ldx4(prs, off[1] + flat_off(i, js0, H), 0);
#pragma unroll
                for (int i = 0; i < C32; ++i) mx = max(mx, umax4(v[i]));
                if (upper)
#pragma unroll
                    for (int i = 0; i < C32; ++i) mx = max(mx, umax4(v[C32 + i]));
                return mx;
            });
            lap(kTkBar);
            stage_some(xp, v, upper, (unsigned)rows);
        };
        // ---- inner loop (Alg. 3 line 12): joint passes until nobody searches any more, or those who wait are enough
        // (see "patience")
#pragma clang loop unroll(disable)
        for (bool again = false; needm != 0ull; again = true) {
            fresh();
            // (a group of one workgroup: this pass writes over what the terms of the last one are summed from)
            if (C == 1 && (!LSTM || again) && wave == NW - 1) finish_scores();
            if (again) plan_pass(needm);
            const int buf = (int)(jpass & (kRowBufs - 1));
            ++jpass;
            st_joint_passes += 1;
            st_joint_rows += M;
            const int jbb = jb + buf * jb_n, jlb = jl + buf * jb_n, jdb = jd + buf * jd_n, jhb = jh + buf * jh_n;
            if (D > 0 && tpg != dcg_tpg) {   // uniform
                dcg_tpg = tpg;
                dcg0 = ((VL + 1) / CT) / tpg;
                dcg1 = ((O - 1) / CT) / tpg;
            }

            // ---- J
#pragma clang loop unroll(disable)
            for (int it = rank; !WIDE && it < items; it += C) {
                if (!LSTM || again || it != rank) {
                    set_item(it);
                    request_rows();
                }
                v4u p4[NK][NL], pv[2 * C32];
                any_value(pv);
                int po[NK];
                bool upper = false;   // more than eight rows of the predictor's
                const bool load_p = !LSTM || !have_p;
                // the predictor's rows: of the group's hypotheses (LSTM), of those in this row tile (stateless); one area and an
                // LSTM: each lane its own row's part, as it is fed (few of the 16 rows are different ones, so they take few of the
                // requests that made rows go through LDS, and the way through the encoder's area twice is saved: 1024
                // units and joint width, B = 24, 7067 us, 6996; joint width 648, 576 units, two frames a pass, 4779, 4670)
                constexpr bool DIRECT = STAGED && LSTM && !TWO;
                if constexpr (STAGED && LSTM && TWO) {
                } else if constexpr (STAGED && !LSTM) {
                    const int q0 = uni(q_l), q1 = __builtin_amdgcn_readlane(q_l, 15);
                    upper = q1 - q0 >= 8;
                    const float *t0[2], *t1[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {   // (rows beyond the last: the last again)
                        const int g = __builtin_amdgcn_ds_bpermute(min(q0 + h * 8 + (lane >> 3), q1) * 4, slot_of) * 4;
                        const int lab = __builtin_amdgcn_ds_bpermute(g, last), lab2 = __builtin_amdgcn_ds_bpermute(g, last2);
                        // one label of context: its table row; two: the older label's table, then the newest label's
                        t0[h] = p.pred_tab + (size_t)(p.pred_layers == 2 ? lab2 : lab) * H;
                        t1[h] = p.pred_tab + ((size_t)(V + 1) + lab) * H;
                    }
#pragma unroll
                    for (int i = 0; i < C32; ++i) pv[i] = ldg4(t0[0], flat_off(i, js0, H));
                    if (upper)
#pragma unroll
                        for (int i = 0; i < C32; ++i) pv[C32 + i] = ldg4(t0[1], flat_off(i, js0, H));
                    if (p.pred_layers == 2) {
                        auto add_row = [&](v4u &x, const float *t, int i) __attribute__((always_inline)) {
                            const float4 y = as_float4(ldg4(t, flat_off(i, js0, H))), z = as_float4(x);
                            x = v4u{__float_as_uint(z.x + y.x), __float_as_uint(z.y + y.y), __float_as_uint(z.z + y.z),
                                    __float_as_uint(z.w + y.w)};
                        };
#pragma unroll
                        for (int i = 0; i < C32; ++i) add_row(pv[i], t1[0], i);
                        if (upper)
#pragma unroll
                            for (int i = 0; i < C32; ++i) add_row(pv[C32 + i], t1[1], i);
                    }
                } else {
                    const int row = p_row(g_l, 0) * H * (int)sizeof(float);
#pragma unroll
                    for (int s = 0; s < NK; ++s) po[s] = row + part_of(s, js0, H);
                }
                // weights, and biases of this thread's four columns (zeros beyond the last)
                auto fetch_round = [&](auto &w, auto &bias, int t0) __attribute__((always_inline)) {
                    const int wbase = here(p.off_w_out + (tile0 + t0) * jbytes);
                    fetch(w, min((int)(sizeof(w) / sizeof(w[0])), n_ct - t0), js0, jsn, [&](int t) { return wbase + t * jbytes; });
#pragma unroll
                    for (int h = 0; h < (int)(sizeof(bias) / sizeof(v4u)); ++h)
                        bias[h] = __builtin_amdgcn_raw_buffer_load_b128(
                            brs, ((tile0 + t0) * CT + h * 64 + (lane & 15) * 4) * (int)sizeof(float), 0, 0);
                };
                auto key = [&](int t0, int most) { return (tile0 + t0) * 16 + min(most, n_ct - t0); };   // which tiles, and how many
                if (!KEEP1 || in_b != key(0, TJ)) {
                    fetch_round(b, bias0, 0);
                    in_b = key(0, TJ);
                }
                if (KEEP2 && n_ct > TJ && in_b2 != key(TJ, TR)) {
                    fetch_round(b2, bias1, TJ);
                    in_b2 = key(TJ, TR);
                }
                TR(20);
                const bool to_stage = !PLANES || again || it != rank;   // (else phase Q has)
                if constexpr (STAGED && !DIRECT) {
                    if (TWO && to_stage) stage_rows(xe, ev, true);
                    if (load_p) {
                        if constexpr (LSTM) {
                            take_p(act, pv);
                        } else {
                            stage_rows(xp, pv, upper);
                        }
                        have_p = true;
                    }
                    if (!TWO) {   // one area: the predictor's rows make way for the encoder's
                        const int prow = q_l - uni(q_l);
#pragma unroll
                        for (int s = 0; s < NK; ++s)
#pragma unroll
                            for (int l = 0; l < NL; ++l) {
                                const float4 y = staged(xp, prow, s, l);
                                p4[s][l] = v4u{__float_as_uint(y.x), __float_as_uint(y.y), __float_as_uint(y.z), __float_as_uint(y.w)};
                            }
                        stage_rows(xe, ev, true);
                    }
                } else {
                    if (DIRECT && to_stage) stage_rows(xe, ev, true);
                    until_there([&]() __attribute__((always_inline)) {
                        unsigned mx = 0;
#pragma unroll
                        for (int s = 0; s < NK; ++s)
#pragma unroll
                            for (int l = 0; l < NL; ++l) p4[s][l] = ldx4(prs, po[s] + l * 16, 0);
#pragma unroll
                        for (int s = 0; s < NK; ++s)
#pragma unroll
                            for (int l = 0; l < NL; ++l) mx = max(mx, umax4(p4[s][l]));
                        return mx;
                    });
                    lap(kTkBar);
                }
                TR(22);
                AFrag a[NK][PL];
                constexpr bool STREAMED = STAGED && PL == 3;
                const int prow = LSTM ? g_l : q_l - uni(q_l);   // (staged: where the predictor's row of this lane's row is)
                auto j_source = [&](int s, float (&x)[F::E]) __attribute__((always_inline)) {
#pragma unroll
                    for (int l = 0; l < NL; ++l) {
                        const float4 y = STAGED ? staged(xe, lane & 15, s, l) : as_float4(e4[s][l]);
                        const float4 z = STAGED && TWO ? staged(xp, prow, s, l) : as_float4(p4[s][l]);
                        x[l * 4] = fmaxf(y.x + z.x, 0.0f);
                        x[l * 4 + 1] = fmaxf(y.y + z.y, 0.0f);
                        x[l * 4 + 2] = fmaxf(y.z + z.z, 0.0f);
                        x[l * 4 + 3] = fmaxf(y.w + z.w, 0.0f);
                    }
                };
                if (KEEP1 && !KEEP2 && n_ct > TJ) fetch_round(b2, bias1, TJ);
                if constexpr (STREAMED) {
                    // (all tiles: they are paid for by the split -- but half of them in the stateless form for small items, whose
                    // passes of one or two tiles an item would else be slower than with the split ahead of the products: one
                    // frame a pass, 128 hypotheses in two groups, 46.7 ms that way, 47.6 with all four, 46.1; the form
                    // with eight has no registers left for a third copy of the products)
                    const std::integral_constant<int, (TR + 1) / 2> half{};
                    if (JH > 1 && n_ct <= TR) split_and_multiply(r_tiles, j_source, a, b, j_tiles, part_j);
                    else if (LAYERS == 0 && JH == 1 && TR > 2 && n_ct <= TR / 2) split_and_multiply(half, j_source, a, b, j_tiles, part_j);
                    else split_and_multiply(j_tiles, j_source, a, b, j_tiles, part_j);
                } else {
#pragma unroll
                    for (int s = 0; s < NK; ++s) {
                        float x[F::E];
                        j_source(s, x);
                        split(x, a[s], alone);
                    }
                }
                TR(24);
                fresh();
                // 16 lanes share a row and take four neighbouring columns each; running statistics
                const int i = tid >> 4, quad = lane & 15;
                float rm = -INFINITY, rs = 0.0f, rsm = -INFINITY, rdm = -INFINITY;
                int ra = 0x7fffffff, rda = 0;
                // the sum of exp(logit - largest) of a round is added up when the next round is over or the
                // largest logit has been published
                float lg[4 * JH];
#pragma unroll
                for (int e = 0; e < 4 * JH; ++e) lg[e] = -INFINITY;
                auto fold_sums = [&]() __attribute__((always_inline)) {   // relative to rm, the largest so far
                    float s = 0.0f;
#pragma unroll
                    for (int e = 0; e < 4 * JH; ++e) s += lg[e] > -INFINITY ? __expf(lg[e] - rm) : 0.0f;
                    s = row_sum(s);
                    rs = (rs > 0.0f ? rs * __expf(rsm - rm) : 0.0f) + s;
                    rsm = rm;
                };
#pragma clang loop unroll(disable)
                for (int t0 = 0, next = TJ; t0 < n_ct; t0 = next, next += TR) {
                    const int n = min(next - t0, n_ct - t0);
                    TR(25);
                    if (OWN2 && t0 > 0) products(full_rows, a, b2, n, j_tiles, jsn, part_j);
                    else if (!STREAMED || t0 > 0) products(full_rows, a, b, n, j_tiles, jsn, part_j);
                    float4 bb[JH];
#pragma unroll
                    for (int h = 0; h < JH; ++h) bb[h] = as_float4(OWN2 && h == 0 && t0 > 0 ? bias1[0] : bias0[h]);
                    TR(26);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (words put back earlier have arrived)
                    __syncthreads();
                    TR(27);
                    if ((!KEEP1 || t0 > 0) && next < n_ct) {   // the next round's weights, while this one's results are looked at
                        if constexpr (OWN2) {
                            fetch_round(b2, bias1, next);
                            in_b2 = key(next, TR);
                        } else {
                            fetch_round(b, bias0, next);
                        }
                    }
                    if (t0 > 0) fold_sums();
                    float x4[4 * JH], m = -INFINITY;
                    int am = 0x7fffffff, col0[JH];
#pragma unroll
                    for (int h = 0; h < JH; ++h) {
                        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        if (h == 0 || n > 4) v = gather(j_tiles, part_j, i, h * 16 + quad);   // uniform
                        x4[h * 4] = v.x + bb[h].x;
                        x4[h * 4 + 1] = v.y + bb[h].y;
                        x4[h * 4 + 2] = v.z + bb[h].z;
                        x4[h * 4 + 3] = v.w + bb[h].w;
                        col0[h] = h * 16 + quad < n * 4 ? (tile0 + t0) * CT + h * 64 + quad * 4 : O;
                    }
#pragma unroll
                    for (int e = 0; e < 4 * JH; ++e) {
                        const int col = col0[e / 4] + e % 4;
                        lg[e] = col <= VL ? x4[e] : -INFINITY;
                        am = lg[e] > m ? col : am;
                        m = lg[e] > m ? lg[e] : m;
                    }
                    const float mrow = row_max(m);
                    am = row_min(m == mrow ? am : 0x7fffffff);
                    ra = mrow > rm ? am : ra;   // rounds ascend through the columns: '>' keeps the first maximum
                    rm = fmaxf(rm, mrow);
                    if (cg >= dcg0 && cg <= dcg1) {   // (uniform; never without a duration head)
                        float dm = -INFINITY;
                        int da = 0x7fffffff;
#pragma unroll
                        for (int e = 0; e < 4 * JH; ++e) {
                            const int col = col0[e / 4] + e % 4;
                            if (col > VL && col < O && x4[e] > dm) { dm = x4[e]; da = col - (VL + 1); }
                        }
                        const float drow = row_max(dm);
                        da = row_min(dm == drow ? da : 0x7fffffff);
                        if (drow > rdm) { rdm = drow; rda = da; }
                    }
                    if (next < n_ct) __syncthreads();   // before the partial sums are written again
                }
                TR(28);
                // (no label column, or no logit that is a number: below every label, but present)
                const unsigned long long best = rm > -INFINITY ? pack_best(rm, ra) : 1ull;
                const unsigned long long bd = rdm > -INFINITY ? pack_best(rdm, rda) : 1ull;
                if (C > 1 && quad == 0) {
                    st_word(i * 8, jbb + it * RT * 8, best);
                    if (cg == dcg0) st_word(i * 8, jdb + ti * 2 * RT * 8, bd);
                    else if (cg == dcg1) st_word(i * 8, jdb + (ti * 2 + 1) * RT * 8, bd);
                }
                fold_sums();
                if (quad == 0) {
                    if (!(rm > -INFINITY)) rs = 0.0f;
                    const unsigned long long lse =
                        (unsigned long long)__float_as_uint(rm) | ((unsigned long long)__float_as_uint(rs) << 32);
                    if (C > 1) {
                        st_word(i * 8, jlb + it * RT * 8, lse);
                    } else {
                        S.rowb[ti * RT + i] = best;
                        S.rowl[ti * RT + i] = lse;
                        S.rowd[ti * RT + i] = (unsigned)S.durations[unpack_index(bd) & (TDT_MAX_DURATIONS - 1)];
                    }
                }
                if (it + C < items) __syncthreads();   // the next item writes the partial sums again
                lap(kTkJ);
            }
            if constexpr (WIDE) {
                if (rank < n_cg) {
                    if (LSTM && !again) __syncthreads();   // (phase Q's partial sums are not read any more)
                    tile0 = rank * tpg;
                    n_ct = min(tpg, NT - tile0);
                    cg = rank;
#pragma clang loop unroll(disable)
                    for (int t = 0; t < n_tiles; t += 2) {
                        const std::integral_constant<int, 1> one{};
                        const std::integral_constant<int, 2> two{};
                        if (t + 1 < n_tiles) wide_rows(two, t, jbb, jlb, jdb);
                        else wide_rows(one, t, jbb, jlb, jdb);
                    }
                }
            }
            const int busy = WIDE ? n_cg : items;   // workgroups with a work item (or more)
            if (rank >= busy) {   // no work item: say that this workgroup has come this far
                if constexpr (MERGES && LSTM && !OWN)
                    if (patience > 0 && !have_p) {   // (it may have one when these rows are scored again)
                        v4u pv[2 * C32];
                        any_value(pv);
                        take_p(act, pv);
                        have_p = true;
                    }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (tid == 0) st_word(rank * 8, jhb, 1ull);
            }
            TR(29);
            lap(kTkJ);

            // ---- while the cells travel: the score terms of the pass before
            fresh();
            if (C > 1 && (!LSTM || again)) {   // (an LSTM's first pass: summed while the hidden state travelled)
                --jpass;   // (finish_scores looks at the last pass)
                if (wave == NW - 1) finish_scores();
                ++jpass;
            }
            // ---- gather the cells: a wavefront takes one row tile, or a share of its column groups;
            // lane = (column group modulo 4, row)
            const int wsh = n_tiles == 1 && n_cg > 8 ? 2 : n_tiles <= 2 && n_cg > 4 ? 1 : 0, wpt = 1 << wsh;
            if (C > 1) {
                const int i = (lane & 15) * 8;
#pragma clang loop unroll(disable)
                for (int tw = wave; tw < n_tiles << wsh; tw += NW) {   // (more than once only for many row tiles)
                    const int tt = tw >> wsh, wq = tw & (wpt - 1);
                    const int src = jbb + tt * n_cg * RT * 8;
                    unsigned long long best = 0ull;
                    const int step = 4 << wsh;
                    // Words a lane takes at a time: four, or six where four would leave out some of 17 to 24 column groups and
                    // ask for them when the others have come (config 2 at B = 32, 17 groups, 1.33 ms, with six 1.27, eight
                    // 1.29; at B = 1, 22 groups, 352 us, with six 338, five 356).  Not beyond: of 65 groups a second turn asks
                    // for the last alone, while six words would have every wavefront of the group ask for it over and over
                    // (one frame a pass in one group, 32 hypotheses, 21.0 ms, with six 22.9).  For the same reason a
                    // lane that has no fifth or sixth word asks for its first again (config 3 522 us, now 515).
                    auto gather_cells = [&](auto words) __attribute__((always_inline)) {
                        constexpr int N = decltype(words)::value;
#pragma clang loop unroll(disable)
                        for (int cb = wq * 4; cb < n_cg; cb += N * step) {   // uniform
                            unsigned long long x[N];
                            unsigned spins = 0;
                            long long since = 0;
                            for (;;) {
                                bool all = true;
                                asm volatile("" ::: "memory");   // (see until_there)
#pragma unroll
                                for (int e = 0; e < N; ++e) {
                                    const int c = cb + (lane >> 4) + e * step;
                                    x[e] = ld_word(i + (e > 3 && c >= n_cg ? cb + (lane >> 4) : min(c, n_cg - 1)) * (RT * 8), src);
                                }
#pragma unroll
                                for (int e = 0; e < N; ++e) all = all & (x[e] != 0ull);
                                if (__ballot(!all) == 0ull || give_up(spins, since)) break;
                            }
#pragma unroll
                            for (int e = 0; e < N; ++e) best = x[e] > best ? x[e] : best;
                        }
                    };
                    const std::integral_constant<int, 4> four{};
                    const std::integral_constant<int, 6> six{};
                    if (n_cg <= 4 * step || n_cg > 24) gather_cells(four);
                    else gather_cells(six);
                    best = max_over_rows(best);
                    if (lane < RT) S.rowb[(wq * n_tiles + tt) * RT + lane] = best;
                }
                if (D > 0) {   // the duration head's words: one or two column groups
                    const int two = dcg1 != dcg0 ? RT : 0;
#pragma clang loop unroll(disable)
                    for (int rb = (NW - 1 - wave) * 64; rb < n_tiles * RT; rb += THREADS) {   // uniform
                        const int r = min(rb + lane, n_tiles * RT - 1);
                        const int q = ((r >> 4) * 2 * RT + (r & 15)) * 8;
                        unsigned long long x = wait_word(q, jdb);
                        if (two) {
                            const unsigned long long y = wait_word(q + two * 8, jdb);
                            x = x > y ? x : y;
                        }
                        S.rowd[r] = (unsigned)S.durations[unpack_index(x) & (TDT_MAX_DURATIONS - 1)];   // the frame step
                    }
                }
                if (busy < C && wave == 1)   // the workgroups without a work item
#pragma clang loop unroll(disable)
                    for (int c = busy; c < C; c += 64) wait_word(min(c + lane, C - 1) * 8, jhb);
            }
            TR(31);
            __syncthreads();
            TR(32);
            lap(kTkBar);
            // ---- D: every wavefront takes the same decisions.  Rows of passes of up to 64 rows sit in
            // lanes; larger passes are first brought together in LDS
            fresh();
            const int w_rows = n_tiles * RT, stop = S.aborted;
            auto row_result = [&](int r, int &ra, int &step, unsigned long long &best) __attribute__((always_inline)) {
                best = S.rowb[r];
                if (wpt > 1) {   // uniform; two shares or four, all on their way before the first is looked at
                    const unsigned long long x = S.rowb[w_rows + r], y = S.rowb[(wpt - 2) * w_rows + r], z = S.rowb[(wpt - 1) * w_rows + r];
                    best = x > best ? x : best;
                    best = y > best ? y : best;
                    best = z > best ? z : best;
                }
                ra = unpack_index(best);
                if ((unsigned)ra > (unsigned)VL) ra = V;   // (no logit of the row is a number)
                // the frame step that goes with the decision: from the duration head (Sec. 3.3) or,
                // multi-blank, from the symbol: the blank one frame, big blank i its increment
                step = 0;
                if (D > 0) step = (int)(unsigned)S.rowd[r];
                else if (big_blanks) step = ra < V ? 0 : ra == V ? 1 : S.durations[(ra - V - 1) & (TDT_MAX_DURATIONS - 1)];
            };
            const bool plain = D == 0 && !big_blanks;
            const int nv = need ? min(Kw, len - time) : 0;   // >= 1 where it searches
            const int base = __popcll(needm & ((1ull << lane) - 1ull)) * Kw;   // lane g: its first row
            int w = 0, k = V, dk = 0;
            unsigned kb = 0;
            bool found = false;
            if (M <= 64) {
                int ra, step;
                unsigned long long best;
                row_result(lane < M ? lane : 0, ra, step, best);
                if (plain) {   // Alg. 3 lines 10 / 18: a blank moves one frame on
                    const unsigned long long nb = __ballot(lane < M && ra < V);
                    const unsigned long long sub = need ? (nb >> base) & (nv >= 64 ? ~0ull : (1ull << nv) - 1ull) : 0ull;
                    found = sub != 0ull;
                    w = found ? __ffsll((long long)sub) - 1 : nv;
                } else {
                    const int code = ra < V ? 0 : max(step, 1);   // frames a non-label moves on; 0: a label
                    bool go = need;
                    while (__ballot(go) != 0ull) {   // (selections: branches on lanes are three times the instructions)
                        const int x = __builtin_amdgcn_ds_bpermute(((base + w) & 63) * 4, code);
                        found = found | (go & (x == 0));
                        w += go ? x : 0;
                        go = go & (x != 0) & (w < nv);
                    }
                }
                const int at = ((base + (found ? w : 0)) & 63) * 4;
                k = __builtin_amdgcn_ds_bpermute(at, ra);
                kb = (unsigned)__builtin_amdgcn_ds_bpermute(at, (int)(unsigned)(best >> 32));
                if (!plain) dk = __builtin_amdgcn_ds_bpermute(at, step);
            } else {
                for (int r = tid; r < M; r += THREADS) {
                    int ra, step;
                    unsigned long long best;
                    row_result(r, ra, step, best);
                    S.res_a[r] = ra;
                    S.res_d[r] = step;
                    S.rowb[r] = best;   // (one share per row tile in passes of this size)
                }
                __syncthreads();
                while (need && w < nv) {
                    if (S.res_a[base + w] < V) { found = true; break; }
                    const int d_ = S.res_d[base + w];
                    w += plain ? 1 : d_ > 0 ? d_ : 1;
                }
                if (found) {
                    k = S.res_a[base + w];
                    dk = S.res_d[base + w];
                    kb = (unsigned)(S.rowb[base + w] >> 32);
                }
            }
            ok = uni(stop) == 0;
            if (!ok) break;
            // ---- Alg. 3 line 20, Sec. 3.1 add_results (selections: a branch costs more than what it skips)
            {
                const bool moved = need & ((w > 0) | !found);
                const int frame = time + w;
                found = found & need;
                if (rank == 0 && wave == 0 && found) {
                    const int gid = S.gid[lane];
                    p.out_labels[(size_t)gid * p.u_cap + olen] = k;
                    p.out_frames[(size_t)gid * p.u_cap + olen] = frame;
                }
                sym = (moved ? 0 : sym) + (found ? 1 : 0);
                olen += found ? 1 : 0;
                last2 = found ? last : last2;
                last = found ? k : last;
                const int dk1 = ((dk == 0) & (sym >= p.max_symbols)) ? 1 : dk;
                const int step = found ? dk1 : 0;
                time = need ? frame + step : time;
                sym = step > 0 ? 0 : sym;
                const bool full = found & (olen >= p.u_cap), more = time < len;
                status |= full ? TDT_HYP_TRUNCATED : 0;
                // (chunks: a hypothesis that has found a label takes one more predictor step, which its
                // state carries on)
                active = need ? (found & CHUNKED) | (more & !full) : active;
                need = need & !found & more;
            }
            pend = found;
            pend_row = base + w;
            pend_m = unpack_value((unsigned long long)kb << 32);
            needm = __ballot(need);
            // (through a scalar register: what leaves a loop on a condition the compiler can't prove the same in all lanes makes
            // everything the loop counts a lane's own)
            const int enough = uni(patience > 0 && __popcll(__ballot(active) & ~needm) * patience >= __popcll(needm) * kCrowd ? 1 : 0);
            TR(33);
            // everybody has read the pass two before this one: its cells are put back (behind the label's
            // last pass: while the next label's hidden state travels)
            clr_items = prev2_items;
            clr_tiles = prev2_tiles;
            prev2_items = prev_items;
            prev2_tiles = prev_tiles;
            prev_items = items;
            prev_tiles = n_tiles;
            prev_cg = n_cg;
            if (!LSTM || (needm != 0ull && enough == 0)) {
                fresh();
                clear_cells();
            }
            TR(34);
            lap(kTkD);
            if (enough != 0) break;
        }
        if (!ok) break;
        if constexpr (EARLY_GATES) request_gates();
        act_prev = act;
        first = false;
        par ^= 1;
    }
    if (ok && wave == NW - 1) finish_scores();

    // ---- what the next chunk takes up
    if (CHUNKED) {
        if (ok && rank == 0 && wave == 0)
            for (int c = 0; c < C; c += 64) wait_word(min(c + lane, C - 1) * 8, jh + kRowBufs * jh_n);
        __syncthreads();
        ok = ok && uni(S.aborted) == 0;
    }
    if (CHUNKED && ok) {
        if constexpr (LSTM) {
            for (int idx = tid; idx < G * U; idx += THREADS) {
                const int g = idx / U, u = idx - g * U;
                if ((took_part >> g) & 1ull)
                    for (int l = 0; l < L; ++l) {
                        const size_t dst = ((size_t)l * B + S.gid[g]) * Hp + u0 + u;
                        p.st_h[dst] = h_l[(l * hpc + g) * Upad + u];
                        p.st_c[dst] = c_l[(l * hpc + g) * Upad + u];
                    }
            }
        }
        if (rank == 0 && wave == 0 && mine) {
            gid = S.gid[lane];
            p.st_started[gid] = started;
            // frames of the next chunk already stepped over; a hypothesis stopped at its label
            // capacity gives up the rest of this chunk
            p.st_time[gid] = max(time - len, 0);
            p.st_last[gid] = last;
            p.st_last2[gid] = last2;
        }
    }
    gid = mine ? S.gid[lane] : 0;
    if (wave == NW - 1 && ((owned >> lane) & 1ull)) p.out_score[gid] = score;   // (the wavefront that summed it)
    // Rank 0 writes labels, lengths and status, but a score is summed elsewhere, and that workgroup may have
    // given up where rank 0 went on to the end.  It adds its mark behind the call's abort flag; rank 0 looks
    // at the flag once more behind its own stores: either it sees the flag or the mark comes later.
    if (rank != 0 && wave == NW - 1 && uni(S.aborted) != 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if ((owned >> lane) & 1ull) atomicOr(&p.out_status[gid], TDT_HYP_ABORTED);
        if (lane == 0 && p.out_stats) atomicAdd((unsigned long long *)&p.out_stats[TDT_STAT_ABORT], 1ull);
    }
    if (rank == 0 && wave == 0) {
        if (mine) {
            p.out_len[gid] = olen;
            st_co32(&p.out_status[gid], status | (ok ? 0 : TDT_HYP_ABORTED));
        }
        if (C > 1) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (__hip_atomic_load(p.abort_flag, __ATOMIC_RELAXED, TDT_AGENT) && mine)
                atomicOr(&p.out_status[gid], TDT_HYP_ABORTED);
        }
        if (tid == 0 && p.out_stats) {
            auto add = [&](int slot, long long v) {
                atomicAdd((unsigned long long *)&p.out_stats[slot], (unsigned long long)v);
            };
            add(TDT_STAT_PRED_PASSES, (long long)st_pred_passes);
            add(TDT_STAT_PRED_ROWS, st_pred_rows);
            add(TDT_STAT_JOINT_PASSES, (long long)st_joint_passes);
            add(TDT_STAT_JOINT_ROWS, st_joint_rows);
            atomicMax((unsigned long long *)&p.out_stats[TDT_STAT_OUTER_MAX], (unsigned long long)st_pred_passes);
            atomicMax((unsigned long long *)&p.out_stats[TDT_STAT_JOINT_PASSES_MAX],
                      (unsigned long long)st_joint_passes);
            if (!ok) add(TDT_STAT_ABORT, 1);
            if (TDT_PHASE_TIMERS && cl == TDT_TIMER_GROUP) {   // where one group's time went, in wall-clock ticks
                add(TDT_STAT_TICKS_PRED, S.tk[kTkP]);
                add(TDT_STAT_TICKS_PROJ, S.tk[kTkQ]);
                add(TDT_STAT_TICKS_JOINT, S.tk[kTkJ]);
                add(TDT_STAT_TICKS_DECIDE, S.tk[kTkD]);
                add(TDT_STAT_TICKS_BARRIER, S.tk[kTkBar]);
                add(TDT_STAT_TICKS_TOTAL, wall_clock64() - S.tk_start);
            }
        }
    }
}

constexpr size_t kLabelDynLds = kLdsBytes - sizeof(LabelShared) - 256;   // (the rest: what the compiler adds)

int label_kseg(const tdt_weights_t *w)
{
    return w->pred_kind == TDT_PRED_LSTM && w->h_pred > w->h_joint ? w->h_pred : w->h_joint;
}

template <typename WT, int LAYERS, int NK, int NW, int TQ, int QROWS = RT> const void *label_form_of(bool chunked)
{
    return chunked ? (const void *)label_kernel<WT, LAYERS, true, NK, NW, TQ, QROWS>
                   : (const void *)label_kernel<WT, LAYERS, false, NK, NW, TQ, QROWS>;
}
template <typename WT, int NK> const void *label_fn(int layers, int tq, bool few, bool chunked)
{
    constexpr int TR = label_tiles(NK);
    if (layers > 1) return label_form_of<WT, 2, NK, 4, TR>(chunked);
    if constexpr (Frags<WT>::PL == 1)
        if (layers == 1 && few)
            return tq > TR ? label_form_of<WT, 1, NK, 4, 2 * TR, kPairRows>(chunked) : label_form_of<WT, 1, NK, 4, TR, kPairRows>(chunked);
    if (layers == 1) return tq > TR ? label_form_of<WT, 1, NK, 4, 2 * TR>(chunked) : label_form_of<WT, 1, NK, 4, TR>(chunked);
    if constexpr (first_tiles(Frags<WT>::PL == 3, NK) > TR)
        if (tq > TR) return label_form_of<WT, 0, NK, 4, first_tiles(true, NK)>(chunked);
    return label_form_of<WT, 0, NK, 4, TR>(chunked);
}
const void *label_wide_fn(bool lstm, int round, int pred_steps, bool chunked)   // (bfloat16)
{
    if (!lstm) return label_form_of<uint16_t, 0, 4, 8, 4>(chunked);
    if (round > 0) return label_form_of<uint16_t, 2, 4, 8, kWideRound>(chunked);
    return pred_steps <= 3 ? label_form_of<uint16_t, 2, 4, 8, 3>(chunked) : label_form_of<uint16_t, 2, 4, 8, 4>(chunked);
}
struct LabelForm {
    const void *fn;   // null: none
    int nk, nw, tq, layers;   // steps of the reduction per wavefront, wavefronts, TQ, LAYERS
};
// item: column tiles of a usual work item of a joint pass.  A stateless group where that is at most a round's four takes four
// in the first round too, or two where an item has no more (one frame a pass, 128 hypotheses in three groups,
// 37.7 ms with eight, 35.8; before there were eight 36.4).
LabelForm label_form(const tdt_weights_t *w, bool chunked, bool wide, int hyps_per_cluster, int C, int item)
{
    const bool lstm = w->pred_kind == TDT_PRED_LSTM;
    LabelForm f{nullptr, 0, wide ? 8 : 4, 0, lstm ? 2 : 0};
    // bfloat16: steps of 32 inputs (reductions of up to 640 and 1024), float32: of 16 (256 and 640; for 1024,
    // 16 steps a wavefront, the rows of two operands and the weights of a round would take more than the 512
    // registers of a lane: 128 and 128 in a joint pass, 256 more for the round of phase Q held meanwhile)
    const int kseg = label_kseg(w);
    if (wide) {
        f.nk = 4;
        if (lstm && wide_round(w->pred_layers, (w->h_joint + CT - 1) / CT, (w->h_pred + 3) / 4, C)) f.tq = kWideRound;
        if (w->dtype == 1 && label_steps(true, kseg, f.nw) <= f.nk) f.fn = label_wide_fn(lstm, f.tq, label_steps(true, w->h_pred, f.nw), chunked);
        return f;
    }
    f.nk = label_nk(w->dtype == 1, kseg);
    if (f.nk == 0) return f;
    bool few = false;
    f.tq = label_tiles(f.nk);
    if (!lstm && item > f.tq) f.tq = first_tiles(w->dtype == 1, f.nk);
    if (lstm && w->pred_layers == 1) {
        const int nt_a = (w->h_joint + CT - 1) / CT, nt_b = (w->h_pred + 3) / 4;
        if (one_layer_form(f.nk, nt_a, nt_b, C, hyps_per_cluster, kLabelThreads)) {
            f.layers = 1;
            const int per_wg = (nt_a + nt_b + C - 1) / C;
            few = few_rows(f.nk, per_wg, hyps_per_cluster, w->h_pred);   // (float32)
            if (per_wg > f.tq) f.tq *= 2;
        }
    }
    if (w->dtype == 1)
        f.fn = f.nk == 5 ? label_fn<uint16_t, 5>(f.layers, f.tq, few, chunked) : label_fn<uint16_t, 8>(f.layers, f.tq, few, chunked);
    else f.fn = f.nk == 4 ? label_fn<float, 4>(f.layers, f.tq, few, chunked) : label_fn<float, 10>(f.layers, f.tq, few, chunked);
    return f;
}

}  // namespace

// lists of column tiles (f.nw == 8, f.tq == 0): with room for as many column tiles of partial sums as wide_part floats hold
static size_t label_lds_bytes(const tdt_weights_t *w, const LabelForm &f, bool chunked, int hyps_per_cluster, int C, int wide_part = kWidePart)
{
    size_t n = 0;
    if (w->dtype == 1 && f.layers > 1 && (f.nw < 8 || f.tq > 0) && hyps_per_cluster <= kPackRows)
        n = (size_t)RT * ActTile<uint16_t>::row_elems(label_kseg(w)) * sizeof(uint16_t);
    if (f.nw == 8) {
        n += (size_t)f.nw * RT * wide_part * sizeof(float);
    } else {
        if (w->pred_kind == TDT_PRED_LSTM) n += (size_t)f.nw * RT * (f.tq * CT + 4) * sizeof(float);
        n += (size_t)f.nw * RT * ((f.layers == 0 ? f.tq : label_tiles(f.nk)) * CT + 4) * sizeof(float);
    }
    if (stages_rows(f.layers, f.nw)) {
        const int ks = w->dtype == 1 ? 32 : 16, rows = RT + (two_areas(f.nk, ks) ? pred_area_rows(f.layers, hyps_per_cluster) : 0);
        n += (size_t)f.nw * rows * staged_row(f.nk, ks) * sizeof(float);
    }
    if (w->pred_kind == TDT_PRED_LSTM) {
        const int tiles = (w->h_pred + 3) / 4 + (f.layers == 1 ? (w->h_joint + CT - 1) / CT : 0);
        const size_t units = (size_t)w->pred_layers * hyps_per_cluster * ((tiles + C - 1) / C) * 4;
        n += units * (4 + 1 + (chunked ? 1 : 0)) * sizeof(float);
    }
    return (n + 15) / 16 * 16;
}

#if TDT_TRACE
hipError_t copy_trace_label(long long *out, int n)
{
    return hipMemcpyFromSymbol(out, HIP_SYMBOL(g_trace), (size_t)n * sizeof(long long));
}
#endif

bool label_kernel_takes(const tdt_weights_t *w, bool chunked, bool wide, int hyps_per_cluster, int C)
{
    if (hyps_per_cluster > kLabelMaxHyps) return false;
    const LabelForm f = label_form(w, chunked, wide, hyps_per_cluster, C, 64);   // (the larger of two for a stateless model)
    if (!f.fn) return false;
    const size_t dyn = label_lds_bytes(w, f, chunked, hyps_per_cluster, C);
    const size_t lens = (size_t)kMaxRankedBatch * sizeof(int);   // (the batch's lengths while they are ranked)
    if (packed_layout(w).total >= ((size_t)1 << 31)) return false;   // offsets among the copies are 32 bits
    return dyn >= lens && dyn <= kLabelDynLds;
}

hipError_t launch_label(const DecodeParams &p, const tdt_weights_t *w, bool chunked, bool wide, int grid,
                        hipStream_t stream)
{
    // the LDS limit of a compiled form is raised once per device (to all a workgroup can have)
    static std::mutex mu;
    static const void *ready[64][64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    const int C = grid / p.n_clusters;
    const int item = w->pred_kind == TDT_PRED_LSTM || wide
                         ? 0 : usual_item(C, (p.O + CT - 1) / CT, p.hyps_per_cluster, p.window, p.joint_tiles, p.rows_per_cluster);
    const LabelForm f = label_form(w, chunked, wide, p.hyps_per_cluster, C, item);
    const void *fn = f.fn;
    if (!fn) return hipErrorInvalidValue;
    {
        std::lock_guard<std::mutex> lock(mu);
        int i = 0;
        while (i < 64 && ready[dev][i] && ready[dev][i] != fn) ++i;
        if (i == 64 || !ready[dev][i]) {
            e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kLabelDynLds);
            if (e != hipSuccess) return e;
            if (i < 64) ready[dev][i] = fn;
        }
    }
    DecodeParams pc = p;
    pc.kseg_max = label_kseg(w);
    // (lists: the most column tiles a workgroup has of one matrix, or as many as LDS has room for)
    int tiles = 0;
    if (f.nw == 8 && f.layers > 0 && f.tq == 0) {
        tiles = std::max(((w->h_joint + CT - 1) / CT + C - 1) / C, ((w->h_pred + 3) / 4 + C - 1) / C);
        tiles = std::min(tiles, kWideTiles);
        while (tiles > 0 && label_lds_bytes(w, f, chunked, p.hyps_per_cluster, C, wide_part(tiles)) > kLabelDynLds) --tiles;
    }
    pc.wide_part = wide_part(tiles);
    pc.lds_bytes = (int)label_lds_bytes(w, f, chunked, p.hyps_per_cluster, C, pc.wide_part);
    void *args[] = {&pc};
    // A group of one workgroup waits for nobody, so its workgroups need not all be resident.  A cooperative launch, which
    // sees to that, goes through another queue: 11 us from the kernel before to this one and 11 to the next (the
    // smallest benchmark model's call 229 us, now 210).
    if (grid == p.n_clusters) return hipLaunchKernel(fn, dim3(grid), dim3(f.nw * 64), args, (unsigned)pc.lds_bytes, stream);
    return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(f.nw * 64), args, (unsigned)pc.lds_bytes, stream);
}

}  // namespace tdt
