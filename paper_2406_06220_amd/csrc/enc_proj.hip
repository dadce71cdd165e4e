// Dense projections computed once per call, before the label loop starts:
//   encoder projection (paper Sec. 3.4; the precomputation at line 2 of Algorithm 3)
//     out[r][n] = sum_k enc[r][k] * w_enc[n][k] + b_enc[n]
//   and, with the same kernel, what the predictor side can tabulate per label: the first LSTM
//   layer's input product w_ih[0] * emb[label] + b_lstm[0], or -- for a stateless predictor,
//   whose output is nothing but embeddings of the last labels -- its whole projection into the
//   joint space, one table per context position: w_pred[:, c*E .. (c+1)*E) * emb_c[label]
//   (the last table with b_pred added).
// A dense contraction over all B*T frames, so it runs on the matrix cores:
// bf16 operands, fp32 accumulation, fp32 output (v_mfma_f32_32x32x16_bf16).
// Both operands are K-contiguous ("NT" GEMM), which is the layout the MFMA lane
// mapping wants: lane l supplies row (l % 32), k-slice (l / 32) * 8 .. + 7.
#include "tdt_internal.h"

#include <mutex>
#include <type_traits>

namespace tdt {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

constexpr int BM = 128, BN = 128, BK = 64;   // workgroup tile
constexpr int GEMM_THREADS = 256;            // 4 wavefronts, each a 64x64 sub-tile

// A tile row is 128 bytes, half of the 64 four-byte LDS banks; rows r and r + 1 lie in different
// halves.  16-byte chunk c of row r is stored at chunk c ^ ((r >> 1) & 7), so that the 16 rows a
// quarter of a wavefront reads for one k-slice (same c, consecutive r) fall on 16 different
// chunk positions, i.e. on all 64 banks.
__device__ inline int lds_off(int row, int chunk) { return row * BK + ((chunk ^ ((row >> 1) & 7)) << 3); }

// One product C = A * W^T + bias and the workgroups it takes.  Rows of W are ldw apart (a
// slice of the columns of a wider matrix can be multiplied); bias may be null.
// With `lens` the rows are the frames of B utterances of T frames each, of which only the first
// min(max(lens[b], 0), T) of utterance b are multiplied (Alg. 3 line 2 projects the encoder
// output; frames beyond an utterance's length are never looked at, so they are neither read nor
// written): the workgroups then walk the valid frames in order, 128 at a time, and M = B * T only
// bounds their number.
struct LinearProblem {
    const void *A, *W;   // both bfloat16 or both float32
    const float *bias;
    float *C;
    long long M;
    int N, K, ldw;
    // row tiles are dealt to 1 << deal_shift dies: all of them, or one (tiles in order).  (Among the first 64 bytes, which every kernel
    // loads: behind them the first tile waits for a second line of arguments, 28 x 10 tiles of 64 x 64 9.0 us, not 8.8.)
    int deal_shift;
    const int32_t *lens;
    int B, T, group;
    unsigned blocks;
};
constexpr int kMaxProblems = 3;   // products one preparation launch can hold
struct LinearBatch {
    LinearProblem q[kMaxProblems];
};

// the row of W (and the bias) that column c of the output is the product with.  GROUPED: group may be
// set (columns that belong together then leave as whole rows, not as scattered words)
template <bool GROUPED> __device__ inline int source_column(const LinearProblem &q, int c)
{
    if (!GROUPED || q.group == 0) return c;
    const int kinds = q.N / q.group;
    return c % kinds * q.group + c / kinds;
}

// The output tile of workgroup `block`: its row tile and its column tile.  Consecutive workgroups go to
// consecutive XCDs, each with an L2 of its own, so the workgroups that share a row tile of `A` (all its
// column tiles) are given to one XCD: row tiles are dealt round robin to the XCDs, and the j-th workgroup of an
// XCD takes column tile j % nt_n of that XCD's (j / nt_n)-th row tile.  `A` then comes from HBM once instead of
// once per XCD; `W` is small and stays in every L2.  Few row tiles may be taken in order (tiles_in_order).
__device__ inline void tile_of(const LinearProblem &q, unsigned block, int nt_n, long long &mt, int &nt)
{
    const unsigned j = block >> q.deal_shift;
    mt = ((long long)(j / nt_n) << q.deal_shift) + (block & ((1u << q.deal_shift) - 1u));
    nt = (int)(j % nt_n);
}

// Which frames rows m0 .. m0 + ROWS - 1 of the packed sequence of valid frames are: row_of[i] =
// b * T + t, or -1 beyond the last valid frame.  Called by all THREADS threads of a workgroup;
// returns false (for all of them) if the tile holds no valid frame at all.  Every thread sums a
// stretch of the utterances' lengths, the stretches' sums are scanned across the workgroup, and
// each row finds its utterance by a search over the stretches and a walk through its stretch.
// (The two halves are functions of their own for workgroups that look for the rows of several tiles.)
template <int THREADS>
__device__ inline int scan_lengths(const int32_t *lens, int B, int T, int per, int *scan, int *wsum)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b_lo = min(tid * per, B), b_hi = min(b_lo + per, B);
    int mine = 0;   // B * T < 2^31, so every sum of lengths fits an int
    for (int b = b_lo; b < b_hi; ++b) mine += min(max(lens[b], 0), T);
    int v = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    if (lane == 63) wsum[wave] = v;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        if (w < wave) base += wsum[w];
        total += wsum[w];
    }
    scan[tid] = base + v - mine;   // valid frames before stretch tid
    __syncthreads();
    return total;
}
template <int THREADS>   // m is less than the number of valid frames
__device__ inline long long find_row(const int32_t *lens, int T, int B, int per, const int *scan, int m)
{
    int lo = 0, hi = THREADS - 1;   // the last stretch that starts at or before m
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (scan[mid] <= m) lo = mid; else hi = mid - 1;
    }
    int before = scan[lo], b = min(lo * per, B);
    // (stretches of one utterance: it is the one, others start later or are empty)
    while (per > 1) {   // ends, because m is a valid frame
        const int len = min(max(lens[b], 0), T);
        if (m < before + len) break;
        before += len;
        ++b;
    }
    return (long long)b * T + (m - before);
}
template <int ROWS, int THREADS = GEMM_THREADS>
__device__ inline bool valid_row_map(const int32_t *lens, int B, int T, long long m0, long long *row_of, int *scan,
                                     int *wsum)
{
    const int tid = threadIdx.x, per = (B + THREADS - 1) / THREADS;
    const int total = scan_lengths<THREADS>(lens, B, T, per, scan, wsum);
    if (m0 >= total) return false;
    if (tid < ROWS) row_of[tid] = m0 + tid < total ? find_row<THREADS>(lens, T, B, per, scan, (int)m0 + tid) : -1;
    return true;
}

// the 128 x 128 output tile of workgroup `block` (of q.blocks) of one product
template <bool GROUPED> __device__ inline void gemm_tile_bf16(const LinearProblem &q, unsigned block)
{
    const uint16_t *__restrict__ A = static_cast<const uint16_t *>(q.A);
    const uint16_t *__restrict__ W = static_cast<const uint16_t *>(q.W);
    const float *__restrict__ bias = q.bias;
    float *__restrict__ C = q.C;
    const long long M = q.M;
    const int N = q.N, K = q.K, ldw = q.ldw;
    // the operand tiles (two buffers each) and, once the products are done, the output tile on
    // its way to memory share one block of LDS
    constexpr int CLD = BN + 4;   // floats per row of the output tile (padded: rows 8 apart meet other banks)
    constexpr size_t kTileBytes = 2 * (size_t)(BM + BN) * BK * sizeof(uint16_t);
    constexpr size_t kOutBytes = (size_t)BM * CLD * sizeof(float);
    __shared__ __align__(16) unsigned char lds_raw[kOutBytes > kTileBytes ? kOutBytes : kTileBytes];
    uint16_t (*As)[BM * BK] = reinterpret_cast<uint16_t (*)[BM * BK]>(lds_raw);
    uint16_t (*Bs)[BN * BK] = reinterpret_cast<uint16_t (*)[BN * BK]>(lds_raw + 2 * (size_t)BM * BK * sizeof(uint16_t));
    float *Cs = reinterpret_cast<float *>(lds_raw);
    __shared__ long long row_of[BM];   // source / destination row of each row of the tile, -1: none
    __shared__ int scan[GEMM_THREADS], wsum[GEMM_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int nt_n = (N + BN - 1) / BN;
    long long mt;
    int nt;
    tile_of(q, block, nt_n, mt, nt);
    const long long m0 = mt * BM;
    const int n0 = nt * BN;
    if (m0 >= M) return;   // the last round of row tiles may be partial (uniform over the workgroup)
    if (q.lens) {
        if (!valid_row_map<BM>(q.lens, q.B, q.T, m0, row_of, scan, wsum)) return;   // uniform
    } else if (tid < BM) {
        row_of[tid] = m0 + tid < M ? m0 + tid : -1;
    }
    __syncthreads();

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // Two register sets and two LDS buffers: K tile kt is multiplied from LDS while tile kt + 1
    // sits in (or is still on its way into) one register set and tile kt + 2 is being requested
    // into the other -- at this kernel's few hundred bytes per flop-microsecond it is the number
    // of bytes in flight per compute unit that decides how much of the HBM rate it gets.
    uint4 ra[2][4], rb[2][4];
    // What this thread loads of every K tile: 16-byte chunk kc of four rows of each operand.
    // The loads themselves are unconditional -- a row or chunk that does not exist is read from
    // one that does (row 0, the last chunk) and replaced by zeros on its way into LDS -- because
    // a load inside a block that depends on the lane makes the compiler wait for every load
    // still in flight before it issues the next, and the two K tiles in flight become one.
    const int kc = tid & 7;
    const uint16_t *a_src[4], *w_src[4];
    bool a_ok[4], w_ok[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = (tid + j * GEMM_THREADS) >> 3;
        const long long ar = row_of[row];
        const int n = n0 + row;
        a_ok[j] = ar >= 0;
        w_ok[j] = n < N;
        a_src[j] = A + (a_ok[j] ? ar : 0) * K;
        w_src[j] = W + (long long)(w_ok[j] ? source_column<GROUPED>(q, n) : 0) * ldw;
    }
    auto load_tiles = [&](int k0, uint4 (&xa)[4], uint4 (&xb)[4]) {
        const int k = min(k0 + kc * 8, K - 8);   // K is a multiple of 8
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            xa[j] = *reinterpret_cast<const uint4 *>(a_src[j] + k);
            xb[j] = *reinterpret_cast<const uint4 *>(w_src[j] + k);
        }
    };
    auto store_tiles = [&](int buf, int k0, const uint4 (&xa)[4], const uint4 (&xb)[4]) {
        const bool k_ok = k0 + kc * 8 < K;
        // (masks, not a choice between two values: a choice between the register set and a
        // constant becomes a choice between two addresses, which puts the set into scratch memory)
        auto keep = [](uint4 v, bool ok) {
            const unsigned m = ok ? 0xffffffffu : 0u;
            return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
        };
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = (tid + j * GEMM_THREADS) >> 3;
            *reinterpret_cast<uint4 *>(As[buf] + lds_off(row, kc)) = keep(xa[j], a_ok[j] && k_ok);
            *reinterpret_cast<uint4 *>(Bs[buf] + lds_off(row, kc)) = keep(xb[j], w_ok[j] && k_ok);
        }
    };
    auto products = [&](int buf) {
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            const int chunk = s * 2 + (lane >> 5);
            bf16x8 a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int ar = wm * 64 + i * 32 + (lane & 31);
                const int br = wn * 64 + i * 32 + (lane & 31);
                a[i] = *reinterpret_cast<const bf16x8 *>(As[buf] + lds_off(ar, chunk));
                b[i] = *reinterpret_cast<const bf16x8 *>(Bs[buf] + lds_off(br, chunk));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };

    // The same products with the requests for a later K tile dealt out between them, one after
    // every two products (step s asks for the thread's s-th chunk of both operands), so that
    // the compute unit's address path takes them one by one instead of eight in a row.
    auto products_and_loads = [&](int buf, int k0, uint4 (&xa)[4], uint4 (&xb)[4]) __attribute__((always_inline)) {
        static_assert(BK / 16 == 4, "one chunk of each operand per k step");
        const int k = min(k0 + kc * 8, K - 8);
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            const int chunk = s * 2 + (lane >> 5);
            bf16x8 a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int ar = wm * 64 + i * 32 + (lane & 31);
                const int br = wn * 64 + i * 32 + (lane & 31);
                a[i] = *reinterpret_cast<const bf16x8 *>(As[buf] + lds_off(ar, chunk));
                b[i] = *reinterpret_cast<const bf16x8 *>(Bs[buf] + lds_off(br, chunk));
            }
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc[0][1], 0, 0, 0);
            xa[s] = *reinterpret_cast<const uint4 *>(a_src[s] + k);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc[1][1], 0, 0, 0);
            xb[s] = *reinterpret_cast<const uint4 *>(w_src[s] + k);
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);   // the step's four fragments from LDS
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // two products
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // one request
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
    };

    const int nk = (K + BK - 1) / BK;
    load_tiles(0, ra[0], rb[0]);
    if (nk > 1) load_tiles(BK, ra[1], rb[1]);
    store_tiles(0, 0, ra[0], rb[0]);
    __syncthreads();
    // Two K tiles per trip, so that the register sets are named at compile time; one workgroup
    // barrier per K tile (the buffer written after the products was last read before the
    // previous barrier).  The trips that have all their tiles run without a branch: behind a
    // branch, even a uniform one, the compiler no longer knows how many loads are in flight and
    // waits for all of them where the older set would do.  (The fence keeps the older set's way
    // into LDS behind the products.)
    int kt = 0;
    for (; kt + 4 <= nk; kt += 2) {
        products_and_loads(0, (kt + 2) * BK, ra[0], rb[0]);
        __builtin_amdgcn_sched_barrier(0);
        store_tiles(1, (kt + 1) * BK, ra[1], rb[1]);
        __syncthreads();
        products_and_loads(1, (kt + 3) * BK, ra[1], rb[1]);
        __builtin_amdgcn_sched_barrier(0);
        store_tiles(0, (kt + 2) * BK, ra[0], rb[0]);
        __syncthreads();
    }
    for (; kt < nk; kt += 2) {   // the last one to three tiles
        if (kt + 2 < nk) load_tiles((kt + 2) * BK, ra[0], rb[0]);
        products(0);
        if (kt + 1 < nk) store_tiles(1, (kt + 1) * BK, ra[1], rb[1]);
        __syncthreads();
        if (kt + 1 < nk) {
            if (kt + 3 < nk) load_tiles((kt + 3) * BK, ra[1], rb[1]);
            products(1);
            if (kt + 2 < nk) store_tiles(0, (kt + 2) * BK, ra[0], rb[0]);
            __syncthreads();
        }
    }

    // accumulator register e of lane l is row 8*(e/4) + 4*(l/32) + e%4, column l%32
    // The output tile goes through LDS so that it leaves as whole rows: a lane then stores 16
    // bytes, half a wavefront one 512-byte row, and the row's destination is looked up once per
    // row instead of once per element.  (The operand tiles are dead: every wavefront has passed
    // the barrier that followed the last products.)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = wm * 64 + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                Cs[r * CLD + wn * 64 + j * 32 + (lane & 31)] = acc[i][j][e];
            }
    __syncthreads();
    {
        const int c4 = (lane & 31) * 4;                 // this lane's four columns of the tile
        const int n = n0 + c4;
        float4 bn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (bias && n < N) {                            // N is a multiple of 8, so n + 3 < N too
            if (!GROUPED || q.group == 0) bn = *reinterpret_cast<const float4 *>(bias + n);
            else bn = make_float4(bias[source_column<GROUPED>(q, n)], bias[source_column<GROUPED>(q, n + 1)], bias[source_column<GROUPED>(q, n + 2)],
                                  bias[source_column<GROUPED>(q, n + 3)]);
        }
#pragma unroll 4
        for (int it = 0; it < BM / (2 * GEMM_THREADS / 64); ++it) {
            const int r = (it * (GEMM_THREADS / 64) + wave) * 2 + (lane >> 5);
            const long long dst = row_of[r];
            float4 v = *reinterpret_cast<const float4 *>(Cs + r * CLD + c4);
            v.x += bn.x;
            v.y += bn.y;
            v.z += bn.z;
            v.w += bn.w;
            if (dst >= 0 && n < N) *reinterpret_cast<float4 *>(C + dst * N + n) = v;
        }
    }
}

__global__ __launch_bounds__(GEMM_THREADS, 2) void enc_proj_bf16_kernel(LinearProblem q)
{
    gemm_tile_bf16<false>(q, blockIdx.x);
}

// The same product for small problems: 64 x 64 output tile, four wavefronts of 32 x 32.  Where the 128 x
// 128 tiles do not fill the chip a product lasts as long as one workgroup's walk along K, and a step of
// that is the latency of its loads: so four register sets are in flight instead of two, and a tile has
// a quarter of the work.  K tiles come in fours (tiles beyond the end are zeros).
// Measured (this against 128 x 128 tiles): 50 x 640 x 512 7.5 us, 10.5; 200 x 1024 x 1024 10.5 us, 16.3;
// 3200 x 640 x 512 (125 tiles of 128 x 128) 10.5 us, 11.9; 2400 x 1024 x 1024 (152) 15.2 us, 17.5; but 5000 x
// 640 x 512 (200) 12.7 us, 12.4, and 3600 x 1024 x 1024 (232) 19.7 us, 18.5 -- the border is between.
constexpr int SM = 64, SN = 64;
__global__ __launch_bounds__(GEMM_THREADS, 4) void enc_proj_bf16_small_kernel(LinearProblem q)
{
    const unsigned block = blockIdx.x;
    const uint16_t *__restrict__ A = static_cast<const uint16_t *>(q.A);
    const uint16_t *__restrict__ W = static_cast<const uint16_t *>(q.W);
    const int N = q.N, K = q.K, ldw = q.ldw;
    constexpr int D = 4, CLD = SN + 4;
    __shared__ __align__(16) unsigned char lds_raw[2 * (SM + SN) * BK * sizeof(uint16_t)];
    static_assert(sizeof(lds_raw) >= SM * CLD * sizeof(float), "the output tile reuses the operand buffers");
    uint16_t *const As = reinterpret_cast<uint16_t *>(lds_raw), *const Bs = As + 2 * SM * BK;
    float *const Cs = reinterpret_cast<float *>(lds_raw);
    __shared__ long long row_of[SM];
    __shared__ int scan[GEMM_THREADS], wsum[GEMM_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int nt_n = (N + SN - 1) / SN;
    long long mt;
    int nt;
    tile_of(q, block, nt_n, mt, nt);
    const long long m0 = mt * SM;
    const int n0 = nt * SN;
    if (m0 >= q.M) return;
    if (q.lens) {
        if (!valid_row_map<SM>(q.lens, q.B, q.T, m0, row_of, scan, wsum)) return;   // uniform
    } else if (tid < SM) {
        row_of[tid] = m0 + tid < q.M ? m0 + tid : -1;
    }
    __syncthreads();
    // (unconditional loads, zeros by mask: see gemm_tile_bf16)
    const int kc = tid & 7;
    const uint16_t *a_src[2], *w_src[2];
    bool a_ok[2], w_ok[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = (tid >> 3) + h * 32, n = n0 + row;
        const long long ar = row_of[row];
        a_ok[h] = ar >= 0;
        w_ok[h] = n < N;
        a_src[h] = A + (a_ok[h] ? ar : 0) * K;
        w_src[h] = W + (long long)(w_ok[h] ? n : 0) * ldw;
    }
    uint4 xa[D][2], xw[D][2];
    auto load = [&](int set, int k0) __attribute__((always_inline)) {
        const int k = min(k0 + kc * 8, K - 8);   // K is a multiple of 8
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            xa[set][h] = *reinterpret_cast<const uint4 *>(a_src[h] + k);
            xw[set][h] = *reinterpret_cast<const uint4 *>(w_src[h] + k);
        }
    };
    auto store = [&](int set, int buf, int k0) __attribute__((always_inline)) {
        const bool k_ok = k0 + kc * 8 < K;
        auto keep = [](uint4 v, bool ok) {
            const unsigned m = ok ? 0xffffffffu : 0u;
            return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
        };
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int o = lds_off((tid >> 3) + h * 32, kc);
            *reinterpret_cast<uint4 *>(As + buf * (SM * BK) + o) = keep(xa[set][h], a_ok[h] && k_ok);
            *reinterpret_cast<uint4 *>(Bs + buf * (SN * BK) + o) = keep(xw[set][h], w_ok[h] && k_ok);
        }
    };
    f32x16 acc[2];   // (even and odd steps: two chains)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, d * BK);
    for (int k0 = 0; k0 < K; k0 += D * BK) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int buf = d & 1;
            store(d, buf, k0 + d * BK);   // (last read before the barrier of the tile before)
            load(d, k0 + (D + d) * BK);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < BK / 16; ++s) {
                const int chunk = s * 2 + (lane >> 5);
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(As + buf * (SM * BK) + lds_off(wm * 32 + (lane & 31), chunk));
                const bf16x8 b = *reinterpret_cast<const bf16x8 *>(Bs + buf * (SN * BK) + lds_off(wn * 32 + (lane & 31), chunk));
                acc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[s & 1], 0, 0, 0);
            }
        }
    }
    __syncthreads();
    // whole rows leave through LDS, as in gemm_tile_bf16
#pragma unroll
    for (int e = 0; e < 16; ++e)
        Cs[(wm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * CLD + wn * 32 + (lane & 31)] = acc[0][e] + acc[1][e];
    __syncthreads();
    const int c4 = (tid & 15) * 4, n = n0 + c4;
    if (n >= N) return;   // (N is a multiple of 8)
    float4 bn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (q.bias) bn = *reinterpret_cast<const float4 *>(q.bias + n);
#pragma unroll
    for (int r = tid >> 4; r < SM; r += GEMM_THREADS / 16) {
        const long long dst = row_of[r];
        float4 v = *reinterpret_cast<const float4 *>(Cs + r * CLD + c4);
        v.x += bn.x;
        v.y += bn.y;
        v.z += bn.z;
        v.w += bn.w;
        if (dst >= 0) *reinterpret_cast<float4 *>(q.C + dst * N + n) = v;
    }
}

// ---------------------------------------------------------------------------
// The same product for large problems: 256 x 256 output tile, 4 wavefronts, each 128 x 128
// ---------------------------------------------------------------------------
// What bounds it is the LDS and the wait for memory.  At 128 x 128 outputs a wavefront eight fragments feed
// sixteen MFMAs (128 x 64: six feed eight), so a K tile takes 1024 of its 2048 MFMA cycles of the LDS for fragments,
// and the operands go straight into LDS: two buffers of a K tile, filled two steps ahead.
//   * One workgroup of one wavefront a SIMD per compute unit, and it stays: it walks through its tiles without
//     a pause in the requests, and the stores of a tile drain during the products of the next.
//   * The accumulators are all 256 accumulation registers.  Products are written as assembly so that they stay
//     there: the compiler moved them to and fro (some 500 spills).  They go to LDS from where they are.
//   * The fragments of a k step are read during the products of the step before, also across the barrier of a K tile.
//   * Requests are assembly, too: the compiler waits for all of them ahead of every read of LDS.  What is in
//     flight is counted by hand where it matters, see the wait ahead of the barrier.
//   * The L2 of the die has A's lines fetched four steps ahead, one lane a line; the workgroups that share the rows
//     share the lines (61 x 1487 frames 187 -> 170 us, 256 x 1500 705 -> 655).
//   * The output leaves in 128-byte pieces past the caches (non-temporal), and workgroups start apart, so that
//     they do not all write at once: 170 -> 158 us, 655 -> 632.
// Against 8 wavefronts of 128 x 64 that passed their operands through registers, a workgroup a tile, 1024 x 1024, us:
// 66749 valid rows 203 -> 156, 289033 738 -> 640, 33216 117 -> 87, 31750 90 -> 73; 92759 x 1280 x 512 213 -> 163.
// Halving the tiles of a last round that leaves half the workgroups idle was no better (156 -> 162, 33216 rows the same).
constexpr int GM = 256, GN = 256, BIG_THREADS = 256;
constexpr int BIG_MAPS = 4;               // row maps: of the tile that is multiplied and of up to two that are requested
struct BigShared {
    float out[BIG_THREADS / 64][32 * 32];   // a block of a wavefront's outputs
    float bias[BIG_MAPS][GN];
    float unused[BIG_THREADS];   // what look_ahead fetches
    long long row_of[BIG_MAPS][GM];
    int scan[BIG_THREADS], wsum[BIG_THREADS / 64];
};
constexpr size_t kBigBufBytes = (size_t)(GM + GN) * BK * sizeof(uint16_t);   // one K tile of both operands
constexpr size_t kBigLdsBytes = 2 * kBigBufBytes + sizeof(BigShared);
constexpr int kBigGrid = 256;             // one workgroup a compute unit
__device__ const uint4 kZeroChunk = {0, 0, 0, 0};

// Requests BYTES bytes a lane from `src`: lane l's land at byte `at` + l * BYTES of LDS.  (The compiler reserves m0, so it
// warns of a statement that says it changes it; saying so keeps it from relying on a value that it put there itself.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES> __device__ inline void into_lds(const void *src, unsigned at)
{
    static_assert(BYTES == 4 || BYTES == 16, "");
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(at) : "m0", "memory");
    else
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" : : "v"(src), "s"(at) : "m0", "memory");
}
#pragma clang diagnostic pop

__global__ __launch_bounds__(BIG_THREADS, 1) void enc_proj_bf16_big_kernel(LinearProblem q)
{
    extern __shared__ __align__(16) unsigned char big_lds[];
    typedef __attribute__((address_space(3))) unsigned char LdsByte;
    BigShared &sh = *reinterpret_cast<BigShared *>(big_lds + 2 * kBigBufBytes);
    const int N = q.N, K = q.K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const unsigned nt_n = N / GN;
    const int nk = (K + BK - 1) / BK;

    // rows of the product, and a scan of the lengths they are found by (see valid_row_map)
    int per = 0;
    long long rows = q.M;
    if (q.lens) {
        per = (q.B + BIG_THREADS - 1) / BIG_THREADS;
        rows = scan_lengths<BIG_THREADS>(q.lens, q.B, q.T, per, sh.scan, sh.wsum);
    }
    // this workgroup's tiles: the die-aware order of the 128 x 128 kernel, a grid apart
    auto tile_index = [&](int i) { return (blockIdx.x + (unsigned)i * gridDim.x) / kXcds; };
    auto row_tile = [&](int i) { return (long long)(tile_index(i) / nt_n) * kXcds + blockIdx.x % kXcds; };
    auto column = [&](int i) { return (int)(tile_index(i) % nt_n) * GN; };
    auto map_rows = [&](int i) {
        const long long m = row_tile(i) * GM + tid;
        long long src = -1;
        if (m < rows) src = q.lens ? find_row<BIG_THREADS>(q.lens, q.T, q.B, per, sh.scan, (int)m) : m;
        sh.row_of[i % BIG_MAPS][tid] = src;
    };
    int n_tiles = 0;
    while (row_tile(n_tiles) * GM < rows) ++n_tiles;
    if (n_tiles == 0) return;   // uniform over the workgroup

    // this lane's part of every K tile: the 16-byte chunk that lands at place lane % 8 of rows
    // j * 32 + wave * 8 + lane / 8 (LDS takes a wavefront's 64 chunks in a row)
    const int row0 = wave * 8 + (lane >> 3), kc = (lane & 7) ^ ((row0 >> 1) & 7);
    const uint16_t *a_src[8], *w_src[8];
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(LdsByte *)big_lds);
    const uint16_t *ahead;   // the line that this lane has L2 fetch ahead of the requests
    auto sources = [&](int i) {
        const int n0 = column(i);
        const long long mine = sh.row_of[i % BIG_MAPS][min(GM - 1, wave * 64 + (int)(lane / nt_n * nt_n) + n0 / GN)];
        ahead = static_cast<const uint16_t *>(q.A) + (mine >= 0 ? mine : 0) * K;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const long long ar = sh.row_of[i % BIG_MAPS][row0 + j * 32];
            a_src[j] = static_cast<const uint16_t *>(q.A) + (ar >= 0 ? ar : 0) * K + kc * 8;
            w_src[j] = static_cast<const uint16_t *>(q.W) + (long long)(n0 + row0 + j * 32) * q.ldw + kc * 8;
        }
    };
    auto look_ahead = [&](int k) __attribute__((always_inline)) {
        const uint16_t *src = ahead + (k < nk ? k * BK : 0);
        const unsigned at = lds0 + (unsigned)(2 * kBigBufBytes + offsetof(BigShared, unused)) + wave * 256;
        into_lds<4>(src, at);
    };
    auto past_the_end = [&]() {   // the last K tile, where it is not a whole one
        if ((nk - 1) * BK + kc * 8 >= K) {
#pragma unroll
            for (int j = 0; j < 8; ++j) a_src[j] = w_src[j] = reinterpret_cast<const uint16_t *>(&kZeroChunk);
        }
    };
    const unsigned lds_wave = lds0 + wave * 8 * BK * 2;
    auto request = [&](int idx, unsigned buf) __attribute__((always_inline)) {
        const int j = idx & 7;
        const uint16_t *&src = idx < 8 ? a_src[j] : w_src[j];
        const unsigned at = lds_wave + buf + (idx < 8 ? 0 : GM * BK * 2) + j * 32 * BK * 2;
        into_lds<16>(src, at);
        src += BK;
    };

    // lane's fragments: row l % 32 of each 32 x 32 block, chunk s * 2 + l / 32
    const int r32 = lane & 31, sw = (r32 >> 1) & 7;
    const unsigned a_at = (wm * 128 + r32) * (BK * 2), b_at = (GM + wn * 128 + r32) * (BK * 2);
    bf16x8 fa[2][4], fb[2][4];
    auto fragment = [&](int set, int s, int f, unsigned buf) __attribute__((always_inline)) {   // in the order the products need them
        const unsigned c = ((s * 2 + (lane >> 5)) ^ sw) * 16 + buf;
        const bool is_a = f == 0 || f > 4;
        const int i = f == 0 ? 0 : f <= 4 ? f - 1 : f - 4;
        const bf16x8 v = *reinterpret_cast<const bf16x8 *>(big_lds + (is_a ? a_at : b_at) + c + i * 32 * BK * 2);
        if (is_a) fa[set][i] = v; else fb[set][i] = v;
    };

    f32x16 acc[4][4];
    auto product = [&](int x, int set) __attribute__((always_inline)) {
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc[x >> 2][x & 3]) : "v"(fb[set][x & 3]), "v"(fa[set][x >> 2]));
    };
    auto first_product = [&](int x) __attribute__((always_inline)) {
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=a"(acc[x >> 2][x & 3]) : "v"(fb[0][x & 3]), "v"(fa[0][x >> 2]));
    };

    const int steps = n_tiles * nk;
    // Workgroups that write at the same time wait for each other's stores, so they start apart (where there is
    // more than one round of tiles): up to about the time of a tile, those with most tiles first.
    const unsigned slots = gridDim.x / kXcds, all = (unsigned)((rows + GM - 1) / GM + kXcds - 1) / kXcds * nt_n;
    const unsigned rounds = (all + slots - 1) / slots;
    const unsigned naps = rounds > 1 ? blockIdx.x / kXcds / 4 * nk * min(rounds - 1, 4u) : 0;   // of 128 cycles
    for (unsigned z = 0; z < naps; ++z) __builtin_amdgcn_s_sleep(2);
    map_rows(0);
    if (nk == 1 && n_tiles > 1) map_rows(1);
    __syncthreads();
    // the tile and K tile that are requested next, two steps ahead of the products
    int ti = 0, tk = 0;
    auto request_bias = [&](int i) __attribute__((always_inline)) {
        const float *src = q.bias ? q.bias + column(i) + tid : reinterpret_cast<const float *>(&kZeroChunk);
        const unsigned at = lds0 + (unsigned)(2 * kBigBufBytes + offsetof(BigShared, bias)) + (i % BIG_MAPS) * GN * 4 + wave * 256;
        into_lds<4>(src, at);
    };
    auto advance = [&]() { if (++tk == nk) { tk = 0; ++ti; } };
    auto aim = [&]() {
        if (tk == 0) {
            sources(ti);
            request_bias(ti);
        }
        if (tk == nk - 1 && K % BK != 0) past_the_end();
    };
    aim();
#pragma unroll
    for (int idx = 0; idx < 16; ++idx) request(idx, 0);
    advance();
    if (steps > 1) {
        aim();
#pragma unroll
        for (int idx = 0; idx < 16; ++idx) request(idx, (unsigned)kBigBufBytes);
        advance();
        asm volatile("s_waitcnt vmcnt(16)" : : : "memory");
    } else {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
#pragma unroll
    for (int f = 0; f < 8; ++f) fragment(0, 0, f, 0);

    int g = 0;
    bool stored = false;   // 64 stores of the tile before came behind the requests of the next step
    for (int tile = 0; tile < n_tiles; ++tile) {
        for (int kt = 0; kt < nk; ++kt, ++g) {
            const unsigned buf = (g & 1) * (unsigned)kBigBufBytes;
            const bool more = g + 2 < steps;
            if (more && tk == 0) map_rows(ti);
            if (kt == 0) {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    __builtin_amdgcn_sched_barrier(0);
                    first_product(x);
                    if (x < 8) fragment(1, 1, x, buf);
                }
            } else {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    __builtin_amdgcn_sched_barrier(0);
                    product(x, 0);
                    if (x < 8) fragment(1, 1, x, buf);
                }
            }
#pragma unroll
            for (int s = 1; s < 3; ++s) {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    __builtin_amdgcn_sched_barrier(0);
                    product(x, s & 1);
                    if (x < 8) fragment((s + 1) & 1, s + 1, x, buf);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // The next step's K tile has landed, and nobody reads this step's any more.  What may be in flight is
            // younger: one look ahead, or the 64 stores of the tile before.
            if (kt == 0 && stored) asm volatile("s_waitcnt vmcnt(63) lgkmcnt(0)" : : : "memory");
            else if (kt == 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");
            else asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)" : : : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" : : : "memory");
            if (more) {
                aim();
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) a_src[j] = w_src[j] = reinterpret_cast<const uint16_t *>(&kZeroChunk);
            }
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                __builtin_amdgcn_sched_barrier(0);
                product(x, 1);
                if (x < 8) fragment(0, 0, x, buf ^ (unsigned)kBigBufBytes);
                request(x, buf);
            }
            look_ahead(tk + 2);
            __builtin_amdgcn_sched_barrier(0);
            advance();
        }
        asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");   // the last products are written
        // (the compiler does not see that a product takes so long: what reads one has to stay behind the wait)
#pragma unroll
        for (int x = 0; x < 16; ++x) asm volatile("" : "+a"(acc[x >> 2][x & 3]));
        // accumulator register e of lane l is row l % 32, column 8 * (e / 4) + 4 * (l / 32) + e % 4 of its block: a
        // block passes through LDS of the wavefront's own (chunks placed as in lds_off) and leaves as 128-byte pieces
        float *const stage = sh.out[wave];
        const int col = lane & 7, n = column(tile) + wn * 128 + col * 4;
        const long long *const row_of = sh.row_of[tile % BIG_MAPS] + wm * 128 + (lane >> 3);
        auto store = [&](auto whole) __attribute__((always_inline)) {
            constexpr bool WHOLE = decltype(whole)::value;
            float *out[4];
            bool ok[4];
            f32x4 y[2][4], bn[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                bn[j] = *reinterpret_cast<const f32x4 *>(sh.bias[tile % BIG_MAPS] + wn * 128 + j * 32 + col * 4);
#pragma unroll
            for (int x = 0; x <= 16; ++x) {
                __builtin_amdgcn_sched_barrier(0);
                if (x < 16) {
                    const f32x16 &v = acc[x >> 2][x & 3];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        *reinterpret_cast<f32x4 *>(stage + r32 * 32 + (((2 * e + (lane >> 5)) ^ sw) << 2)) =
                            f32x4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
                    asm volatile("" : : : "memory");
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        y[x & 1][e] = *reinterpret_cast<const f32x4 *>(
                            stage + (e * 8 + (lane >> 3)) * 32 + ((col ^ ((e * 4 + (lane >> 4)) & 7)) << 2));
                    asm volatile("" : : : "memory");
                }
                __builtin_amdgcn_sched_barrier(0);
                if (x == 0) continue;
                const int i = (x - 1) >> 2, j = (x - 1) & 3;
                if (j == 0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const long long dst = row_of[i * 32 + e * 8];
                        ok[e] = WHOLE || dst >= 0;
                        out[e] = q.C + dst * N + n;
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x4 v = y[(x - 1) & 1][e] + bn[j];
                    if (ok[e]) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(out[e] + j * 32));
                }
            }
        };
        stored = row_tile(tile) * GM + GM <= rows;
        if (stored) store(std::true_type{}); else store(std::false_type{});
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");   // (what is still on its way into LDS)
}

// ---------------------------------------------------------------------------
// fragment-major copies of the streamed matrices
// ---------------------------------------------------------------------------
struct PackJob {
    const void *src;
    uint4 *dst;
    int N, K, gate_h;   // gate_h > 0: LSTM gate matrix of gate_h hidden units
    int steps;
    int first;   // its first fragment in the batch
};
constexpr int kMaxPackJobs = 3 + 2 * TDT_MAX_LSTM_LAYERS;
struct PackBatch {
    PackJob j[kMaxPackJobs];
    int n;
    int elem;   // bytes per element: 2 (a step is 32 inputs) or 4 (16 inputs)
    int frags;
};

// Block `blk` of `nblk` blocks of 256 threads copies its share of the fragments, a wavefront one at a
// time, so that which matrix, tile and step it is is worked out once per KiB and not per lane.
__device__ inline void pack_fragments(const PackBatch &b, unsigned blk, unsigned nblk)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = 16 / b.elem, j = lane & 15;   // inputs per lane
    for (int frag = (int)blk * 4 + wave; frag < b.frags; frag += (int)nblk * 4) {
        int ji = 0;
        while (ji + 1 < b.n && frag >= b.j[ji + 1].first) ++ji;
        const PackJob &q = b.j[ji];
        const int local = frag - q.first, tile = local / q.steps, step = local - tile * q.steps;
        const int k = (step * 4 + (lane >> 4)) * per;
        const int unit = tile * 4 + (j >> 2);
        const int row = q.gate_h > 0 ? (j & 3) * q.gate_h + unit : tile * 16 + j;
        const bool ok = (q.gate_h > 0 ? unit < q.gate_h : row < q.N) && k < q.K;   // (K % 8 == 0)
        uint4 v = make_uint4(0, 0, 0, 0);
        if (ok) v = *reinterpret_cast<const uint4 *>(static_cast<const char *>(q.src) + ((size_t)row * q.K + k) * b.elem);
        q.dst[(size_t)local * 64 + lane] = v;
    }
}

__global__ __launch_bounds__(256) void pack_weights_kernel(PackBatch b) { pack_fragments(b, blockIdx.x, gridDim.x); }

PackBatch pack_batch(const tdt_weights_t *w, const PackedLayout &pl, bool on_the_fly, void *packed)
{
    PackBatch b{};
    b.elem = w->dtype == 1 ? 2 : 4;
    if (pl.total == 0) return b;
    const bool lstm = w->pred_kind == TDT_PRED_LSTM;
    auto add = [&](const void *src, const PackedMatrix &m, int N, int K, int gate_h) {
        PackJob &q = b.j[b.n++];
        q.src = src;
        q.dst = reinterpret_cast<uint4 *>(static_cast<char *>(packed) + m.offset);
        q.N = N;
        q.K = K;
        q.gate_h = gate_h;
        q.steps = m.steps;
        q.first = b.frags;
        b.frags += m.tiles * m.steps;   // (dimensions of at most 2^24 x 2048: fits)
    };
    // what a call does not multiply by stays unpacked: the encoder projection and, with a
    // stateless predictor, its projection are products of the kernel only when it projects on the fly
    if (on_the_fly) add(w->w_enc, pl.w_enc, w->h_joint, w->d_enc, 0);
    if (on_the_fly || lstm) add(w->w_pred, pl.w_pred, w->h_joint, w->h_pred, 0);
    add(w->w_out, pl.w_out, w->vocab + 1 + w->n_dur, w->h_joint, 0);
    for (int l = 0; lstm && l < w->pred_layers; ++l) {
        if (l > 0) add(w->w_ih[l], pl.w_ih[l], 4 * w->h_pred, w->h_pred, w->h_pred);
        add(w->w_hh[l], pl.w_hh[l], 4 * w->h_pred, w->h_pred, w->h_pred);
    }
    return b;
}
unsigned pack_blocks_for(const PackBatch &b)
{
    const int blocks = (b.frags + 3) / 4;
    return (unsigned)(blocks < 1024 ? blocks : 1024);
}

// float32 models: 64 x 64 output tile, four wavefronts of 32 x 32 on v_mfma_f32_32x32x2_f32 (exact
// products, float32 accumulation).  A lane holds four consecutive inputs of its row (one 16-byte LDS
// read) and feeds them to four products.  Small tiles, because a call has few rows: at config 2's
// widths the table of 1025 labels makes 680 of them.  Bound by the float32 matrix rate (157 TFLOP/s).
// Measured: the 1025 x 2560 x 640 table and a projection of 3000 x 640 x 512, two launches of a
// vector-ALU kernel, 240 us; here together with the copies and the clearing 91 us.
constexpr int FM = 64, FN = 64, FK = 32, FLD = FK + 4;   // (rows padded by 16 bytes)

template <bool GROUPED> __device__ inline void gemm_tile_f32(const LinearProblem &q, unsigned block)
{
    const float *__restrict__ A = static_cast<const float *>(q.A);
    const float *__restrict__ W = static_cast<const float *>(q.W);
    const int N = q.N, K = q.K, ldw = q.ldw;
    __shared__ __align__(16) float As[2][FM * FLD], Ws[2][FN * FLD];
    __shared__ long long row_of[FM];
    __shared__ int scan[GEMM_THREADS], wsum[GEMM_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int nt_n = (N + FN - 1) / FN;
    long long mt;
    int nt;
    tile_of(q, block, nt_n, mt, nt);
    const long long m0 = mt * FM;
    const int n0 = nt * FN;
    if (m0 >= q.M) return;
    if (q.lens) {
        if (!valid_row_map<FM>(q.lens, q.B, q.T, m0, row_of, scan, wsum)) return;   // uniform
    } else if (tid < FM) {
        row_of[tid] = m0 + tid < q.M ? m0 + tid : -1;
    }
    __syncthreads();
    // this thread's part of every K tile: 16-byte chunk kc of two rows of each operand (unconditional
    // loads, zeros by mask: see gemm_tile_bf16)
    const int kc = tid & 7;
    const float *a_src[2], *w_src[2];
    bool a_ok[2], w_ok[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = (tid >> 3) + h * 32, n = n0 + row;
        const long long ar = row_of[row];
        a_ok[h] = ar >= 0;
        w_ok[h] = n < N;
        a_src[h] = A + (a_ok[h] ? ar : 0) * K;
        w_src[h] = W + (long long)(w_ok[h] ? source_column<GROUPED>(q, n) : 0) * ldw;
    }
    float4 xa[2], xw[2];
    auto load = [&](int k0) {
        const int k = min(k0 + kc * 4, K - 4);   // K is a multiple of 8
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            xa[h] = *reinterpret_cast<const float4 *>(a_src[h] + k);
            xw[h] = *reinterpret_cast<const float4 *>(w_src[h] + k);
        }
    };
    auto keep = [](float4 v, bool ok) {
        return make_float4(ok ? v.x : 0.0f, ok ? v.y : 0.0f, ok ? v.z : 0.0f, ok ? v.w : 0.0f);
    };
    auto store = [&](int buf, int k0) {
        const bool k_ok = k0 + kc * 4 < K;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int o = ((tid >> 3) + h * 32) * FLD + kc * 4;
            *reinterpret_cast<float4 *>(As[buf] + o) = keep(xa[h], a_ok[h] && k_ok);
            *reinterpret_cast<float4 *>(Ws[buf] + o) = keep(xw[h], w_ok[h] && k_ok);
        }
    };
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    const int nk = (K + FK - 1) / FK;
    load(0);
    store(0, 0);
    if (nk > 1) load(FK);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) store((kt + 1) & 1, (kt + 1) * FK);   // (last read before the barrier that ended tile kt - 1)
        if (kt + 2 < nk) load((kt + 2) * FK);
        const float *a = As[kt & 1] + (wm * 32 + (lane & 31)) * FLD + (lane >> 5) * 4;
        const float *w = Ws[kt & 1] + (wn * 32 + (lane & 31)) * FLD + (lane >> 5) * 4;
#pragma unroll
        for (int s = 0; s < FK / 8; ++s) {
            const float4 x = *reinterpret_cast<const float4 *>(a + s * 8), y = *reinterpret_cast<const float4 *>(w + s * 8);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc, 0, 0, 0);
        }
        __syncthreads();
    }
    // accumulator register e of lane l is row 8*(e/4) + 4*(l/32) + e%4, column l%32
    const int n = n0 + wn * 32 + (lane & 31);
    if (n >= N) return;
    const float bn = q.bias ? q.bias[source_column<GROUPED>(q, n)] : 0.0f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const long long dst = row_of[wm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)];
        if (dst >= 0) q.C[dst * N + n] = acc[e] + bn;
    }
}

__global__ __launch_bounds__(GEMM_THREADS) void enc_proj_f32_kernel(LinearProblem q) { gemm_tile_f32<false>(q, blockIdx.x); }

// Everything a decode call needs before its decode kernel, in one launch: the encoder
// projection, the per-label tables of the predictor side (a product with blocks == 0 is
// absent), and the clearing of the workspace's zero region and of the statistics.  The tasks
// are independent; a workgroup takes its task from its index.  A product's die-aware order of tiles takes no more
// than that local indexes which are alike modulo the dies run on one die; which die that is depends on the
// workgroups ahead, whose number is any (products in order have no whole rounds of the dies).
template <bool BF16>
__global__ __launch_bounds__(GEMM_THREADS, 2) void prepare_kernel(LinearBatch batch, PackBatch pack, unsigned pack_blocks,
                                                              uint4 *zero, size_t n16, uint4 *ones, size_t n16_ones,
                                                              long long *out_stats)
{
    unsigned b = blockIdx.x, used = 0;
#pragma unroll
    for (int i = 0; i < kMaxProblems; ++i) {
        if (b < batch.q[i].blocks) {
            if constexpr (BF16) gemm_tile_bf16<true>(batch.q[i], b);
            else gemm_tile_f32<true>(batch.q[i], b);
            return;
        }
        b -= batch.q[i].blocks;
        used += batch.q[i].blocks;
    }
    if (b < pack_blocks) {   // the fragment-major copies of the matrices the decode kernel streams
        pack_fragments(pack, b, pack_blocks);
        return;
    }
    b -= pack_blocks;
    used += pack_blocks;
    const unsigned zb = b, nzb = gridDim.x - used;
    for (size_t i = (size_t)zb * GEMM_THREADS + threadIdx.x; i < n16; i += (size_t)nzb * GEMM_THREADS)
        zero[i] = make_uint4(0, 0, 0, 0);
    for (size_t i = (size_t)zb * GEMM_THREADS + threadIdx.x; i < n16_ones; i += (size_t)nzb * GEMM_THREADS)
        ones[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (out_stats && zb == 0 && threadIdx.x < TDT_STAT_COUNT) out_stats[threadIdx.x] = 0;
}

}  // namespace

// the order of a problem's square tiles, and the workgroups that makes
static void order_tiles(LinearProblem &q, int tile, TileLaunch launch)
{
    const long long row_tiles = (q.M + tile - 1) / tile, column_tiles = (q.N + tile - 1) / tile;
    const long long rounds = (row_tiles + kXcds - 1) / kXcds;
    const bool in_order = tiles_in_order(launch, row_tiles, column_tiles);
    static_assert(kXcds == 1 << 3, "a power of two");
    q.deal_shift = in_order ? 0 : 3;
    q.blocks = (unsigned)((in_order ? row_tiles : rounds * kXcds) * column_tiles);
}

constexpr long long kSmallTiles = 160;   // up to this many 128 x 128 tiles a product takes 64 x 64 tiles, see enc_proj_bf16_small_kernel
static long long tiles_of(const LinearProblem &q) { return (q.M + BM - 1) / BM * ((q.N + BN - 1) / BN); }

static LinearProblem linear_problem(int dtype, const void *a, int64_t rows, int K, const void *w, int ldw, int N,
                                    const float *bias, int group, float *out)
{
    LinearProblem q{};
    q.A = a;
    q.W = w;
    q.bias = bias;
    q.C = out;
    q.M = rows;
    q.N = N;
    q.K = K;
    q.ldw = ldw;
    q.group = group;
    return q;
}

// Products that take the 256 x 256 kernel (a launch of its own: it has its own workgroup size and LDS footprint)
static bool takes_big_tiles(const LinearProblem &q)
{
    return q.group == 0 && q.N % GN == 0 && big_tiles(q.lens != nullptr, q.M, q.N / GN);
}

static hipError_t launch_big_tiles(LinearProblem q, hipStream_t stream)
{
    static std::mutex mu;
    static bool ready[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!ready[dev]) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(enc_proj_bf16_big_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBigLdsBytes);
            if (e != hipSuccess) return e;
            ready[dev] = true;
        }
    }
    const long long row_tiles = (q.M + GM - 1) / GM, rounds = (row_tiles + kXcds - 1) / kXcds;
    const long long tiles = rounds * kXcds * (q.N / GN);
    q.blocks = (unsigned)(tiles < kBigGrid ? tiles : kBigGrid);
    hipLaunchKernelGGL(enc_proj_bf16_big_kernel, dim3(q.blocks), dim3(BIG_THREADS), kBigLdsBytes, stream, q);
    return hipGetLastError();
}

hipError_t launch_prepare(const void *enc, const int32_t *enc_len, int B, int T, const tdt_weights_t *w,
                          float *enc_proj, float *emb_gates, float *pred_tab, const PackedLayout &pl,
                          bool on_the_fly, void *packed, const ClearRanges &clear, long long *out_stats,
                          hipStream_t stream)
{
    const bool bf16 = w->dtype == 1;
    LinearBatch batch{};
    int n = 0;
    // (B == 0: no encoder projection in this launch)
    batch.q[n] = linear_problem(w->dtype, enc, (int64_t)B * T, w->d_enc, w->w_enc, w->d_enc, w->h_joint, w->b_enc, 0, enc_proj);
    batch.q[n].lens = enc_len;
    batch.q[n].B = B;
    batch.q[n].T = T;
    const bool apart = bf16 && takes_big_tiles(batch.q[n]);   // not part of the launch below
    if (apart) {
        const hipError_t e = launch_big_tiles(batch.q[n], stream);
        if (e != hipSuccess) return e;
    }
    ++n;
    if (w->pred_kind == TDT_PRED_LSTM) {   // stored [label][unit][gate]
        batch.q[n++] = linear_problem(w->dtype, w->emb, w->vocab + 1, w->emb_dim, w->w_ih[0], w->emb_dim, 4 * w->h_pred,
                                      w->b_lstm[0], w->h_pred, emb_gates);
    } else if (pred_tab) {
        const size_t E = (size_t)w->emb_dim, rows_tab = (size_t)w->vocab + 1, esz = bf16 ? 2 : 4;
        for (int c = 0; c < w->pred_layers; ++c)
            batch.q[n++] = linear_problem(w->dtype, static_cast<const char *>(w->emb) + c * rows_tab * E * esz,
                                          (int64_t)rows_tab, w->emb_dim,
                                          static_cast<const char *>(w->w_pred) + c * E * esz, w->h_pred, w->h_joint,
                                          c == w->pred_layers - 1 ? w->b_pred : nullptr, 0,
                                          pred_tab + c * rows_tab * w->h_joint);
    }
    unsigned blocks = 0;
    for (int i = apart ? 1 : 0; i < n; ++i) {
        order_tiles(batch.q[i], bf16 ? BM : FM, TileLaunch::kPrepare);
        blocks += batch.q[i].blocks;
    }
    const size_t n16 = clear.zero_bytes / 16, n16_ones = clear.ones_bytes / 16;
    size_t zb = ((n16 > n16_ones ? n16 : n16_ones) + GEMM_THREADS - 1) / GEMM_THREADS;
    if (zb > 256) zb = 256;
    if (zb < 1) zb = 1;
    const PackBatch pack = pack_batch(w, pl, on_the_fly, packed);
    const unsigned pb = pack.frags > 0 ? pack_blocks_for(pack) : 0;
    const dim3 grid(blocks + pb + (unsigned)zb);
    if (bf16)
        hipLaunchKernelGGL(prepare_kernel<true>, grid, dim3(GEMM_THREADS), 0, stream, batch, pack, pb,
                           static_cast<uint4 *>(clear.zero), n16, static_cast<uint4 *>(clear.ones), n16_ones, out_stats);
    else
        hipLaunchKernelGGL(prepare_kernel<false>, grid, dim3(GEMM_THREADS), 0, stream, batch, pack, pb,
                           static_cast<uint4 *>(clear.zero), n16, static_cast<uint4 *>(clear.ones), n16_ones, out_stats);
    return hipGetLastError();
}

static hipError_t launch_problem(int dtype, LinearProblem q, hipStream_t stream)
{
    if (q.M <= 0) return hipSuccess;
    if (dtype == 1 && takes_big_tiles(q)) return launch_big_tiles(q, stream);
    if (dtype == 1 && tiles_of(q) <= kSmallTiles) {
        order_tiles(q, SM, TileLaunch::kSmall);
        hipLaunchKernelGGL(enc_proj_bf16_small_kernel, dim3(q.blocks), dim3(GEMM_THREADS), 0, stream, q);
    } else if (dtype == 1) {
        order_tiles(q, BM, TileLaunch::kOwn);
        hipLaunchKernelGGL(enc_proj_bf16_kernel, dim3(q.blocks), dim3(GEMM_THREADS), 0, stream, q);
    } else {
        order_tiles(q, FM, TileLaunch::kOwn);
        hipLaunchKernelGGL(enc_proj_f32_kernel, dim3(q.blocks), dim3(GEMM_THREADS), 0, stream, q);
    }
    return hipGetLastError();
}

hipError_t launch_encoder_projection_valid(const void *enc, const int32_t *enc_len, int B, int T,
                                           const tdt_weights_t *w, float *out, hipStream_t stream)
{
    LinearProblem q = linear_problem(w->dtype, enc, (int64_t)B * T, w->d_enc, w->w_enc, w->d_enc, w->h_joint, w->b_enc, 0, out);
    q.lens = enc_len;
    q.B = B;
    q.T = T;
    return launch_problem(w->dtype, q, stream);
}

hipError_t launch_encoder_projection(const void *enc, int64_t rows, const tdt_weights_t *w,
                                     float *out, hipStream_t stream)
{
    return launch_problem(w->dtype, linear_problem(w->dtype, enc, rows, w->d_enc, w->w_enc, w->d_enc, w->h_joint, w->b_enc, 0, out),
                          stream);
}

namespace {
PackedMatrix place(size_t &off, int tiles, int K, int per_step)
{
    PackedMatrix m;
    m.offset = off;
    m.tiles = tiles;
    m.steps = (K + per_step - 1) / per_step;
    off += (size_t)m.tiles * m.steps * 1024;
    return m;
}
}  // namespace

PackedLayout packed_layout(const tdt_weights_t *w)
{
    PackedLayout pl{};
    size_t off = 0;
    const bool lstm = w->pred_kind == TDT_PRED_LSTM;
    const int ps = w->dtype == 1 ? 32 : 16;   // inputs per step: 64 bytes of a row
    // (float32: only label_loop.hip multiplies by copies, and it never projects on the fly)
    if (w->dtype == 1) pl.w_enc = place(off, (w->h_joint + 15) / 16, w->d_enc, ps);
    pl.w_pred = place(off, (w->h_joint + 15) / 16, w->h_pred, ps);
    pl.w_out = place(off, (w->vocab + 1 + w->n_dur + 15) / 16, w->h_joint, ps);
    for (int l = 0; lstm && l < w->pred_layers; ++l) {
        // the first layer's input product is a per-label table: its matrix is not streamed
        if (l > 0) pl.w_ih[l] = place(off, (w->h_pred + 3) / 4, w->h_pred, ps);
        pl.w_hh[l] = place(off, (w->h_pred + 3) / 4, w->h_pred, ps);
    }
    pl.total = off;
    return pl;
}

// the copies in a launch of their own (calls that reuse the projections of an earlier call)
hipError_t launch_pack_weights(const tdt_weights_t *w, const PackedLayout &pl, bool on_the_fly, void *packed,
                               hipStream_t stream)
{
    const PackBatch b = pack_batch(w, pl, on_the_fly, packed);
    if (b.frags == 0) return hipSuccess;
    hipLaunchKernelGGL(pack_weights_kernel, dim3(pack_blocks_for(b)), dim3(256), 0, stream, b);
    return hipGetLastError();
}

}  // namespace tdt
