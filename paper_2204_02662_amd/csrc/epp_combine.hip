// Combination stage of the backward pass on the active rows only (Alg. 1, backward loop):
//     W' = Y^T (x) X'      (F_in x F_out, a sum over vertices)
//     Y' = X' (x) W^T      (one row per vertex)
// Theorem 1 makes every row of X' outside N^k zero, so both products run over the ascending id
// list of N^k only: the rows are gathered (and, for Y', scattered) by vertex id, everything
// else is a dense contraction and runs on the matrix cores in fp32 (v_mfma_f32_32x32x2_f32; two
// widths of 65 to 128 and many rows in bfloat16 parts, epp_combine_split.hip).
//
// Widths of up to 128 (every weight matrix of an ordinary model) have kernels of their own, further down:
// the whole product of a pair of rows fits a wavefront's registers, so nothing but W goes through LDS.
//
// For wider ones both kernels give a workgroup of four wavefronts, arranged WM x WN, an output tile of
// 32 WM BM x 32 WN BN, every wavefront BM x BN accumulator blocks of 32 x 32, and step through
// the contraction 32 at a time: the operand tiles of the next step are fetched into registers
// while the matrix cores work on the current ones in LDS.  The arrangement follows the matrix:
// 2 x 2 wavefronts with up to 2 x 2 blocks each for wide outputs, 4 x 1 (a 128 x 32 tile) when
// one side has at most 32 columns, as the weight matrices of a GCN with 16 hidden units or a
// few classes do.
//
// Operand layout of the 32x32x2 instruction: lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32]; element j of its accumulator is C[8 (j / 4) + 4 (l / 32) + j % 4][l % 32].

#include <algorithm>

#include "epp_internal.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kBlock = 256;
constexpr int kStep = 32;   // contraction step
constexpr int kMaxWidth = 4096;
constexpr int kMinChunkRows = 256;
constexpr int64_t kNoChunkLimit = (int64_t)1 << 40;

typedef float float4v __attribute__((ext_vector_type(4)));

// Four consecutive floats of a row; VEC: one 16-byte access (the caller has checked that widths
// are multiples of four and bases 16-byte aligned), else element by element up to `valid`.
template <bool VEC>
__device__ __forceinline__ float4v load4(const float* __restrict__ p, int valid) {
    if constexpr (VEC) {
        return valid > 0 ? *reinterpret_cast<const float4v*>(p) : float4v{0.f, 0.f, 0.f, 0.f};
    } else {
        float4v v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < valid) v[i] = p[i];
        return v;
    }
}

// Thread mapping of all tile loads: eight threads per row, four consecutive floats each, so a
// row segment of 32 floats is one 128-byte access and a thread needs one vertex id per row.

// Y'[id, n] = sum_k X'[id, k] W[n, k] for the ids of one tile of 32 WM BM rows and 32 WN BN columns n.
template <int WM, int WN, int BM, int BN, bool VEC>
__global__ __launch_bounds__(kBlock) void k_input_gradient(const int32_t* __restrict__ ids, int64_t n_rows,
                                                           const float* __restrict__ G, int Fo,
                                                           const float* __restrict__ W, int Fi,
                                                           float* __restrict__ Yg) {
    static_assert(WM * WN == 4, "four wavefronts per workgroup");
    constexpr int TM = 32 * WM * BM, TN = 32 * WN * BN;
    constexpr int NA = TM / 32, NB = TN / 32;  // rows per thread and step
    __shared__ float As[TM][kStep + 1];   // X' rows of the tile, [row][k]
    __shared__ float Bs[kStep][TN + 1];   // W^T, [k][n]
    __shared__ int64_t sid[TM];           // vertex of each tile row, -1 past the end
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = w % WM, wn = w / WM;
    const int64_t row0 = (int64_t)blockIdx.x * TM;
    const int n0 = blockIdx.y * TN;
    for (int r = t; r < TM; r += kBlock) {
        const int64_t row = row0 + r;
        sid[r] = row < n_rows ? (ids ? (int64_t)ids[row] : row) : -1;
    }
    __syncthreads();
    const int tr = t >> 3, k = 4 * (t & 7);
    int64_t oa[NA], ob[NB];  // element offset of this thread's piece at k0 = 0; -1: no such row
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int64_t id = sid[tr + 32 * i];
        oa[i] = id >= 0 ? id * Fo + k : -1;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int n = n0 + tr + 32 * i;
        ob[i] = n < Fi ? (int64_t)n * Fo + k : -1;
    }
    float4v ra[NA], rb[NB];
    auto fetch = [&](int k0) {
        const int valid = Fo - (k0 + k);
#pragma unroll
        for (int i = 0; i < NA; ++i) ra[i] = load4<VEC>(G + (oa[i] >= 0 ? oa[i] + k0 : 0), oa[i] >= 0 ? valid : 0);
#pragma unroll
        for (int i = 0; i < NB; ++i) rb[i] = load4<VEC>(W + (ob[i] >= 0 ? ob[i] + k0 : 0), ob[i] >= 0 ? valid : 0);
    };
    floatx16 acc[BM][BN] = {};
    fetch(0);
    for (int k0 = 0; k0 < Fo; k0 += kStep) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) As[tr + 32 * i][k + c] = ra[i][c];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) Bs[k + c][tr + 32 * i] = rb[i][c];
        __syncthreads();
        if (k0 + kStep < Fo) fetch(k0 + kStep);
#pragma unroll
        for (int kk = 0; kk < kStep; kk += 2) {
            float a[BM], b[BN];
#pragma unroll
            for (int bm = 0; bm < BM; ++bm) a[bm] = As[32 * (BM * wm + bm) + (lane & 31)][kk + (lane >> 5)];
#pragma unroll
            for (int bn = 0; bn < BN; ++bn) b[bn] = Bs[kk + (lane >> 5)][32 * (BN * wn + bn) + (lane & 31)];
#pragma unroll
            for (int bm = 0; bm < BM; ++bm)
#pragma unroll
                for (int bn = 0; bn < BN; ++bn)
                    acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[bm], b[bn], acc[bm][bn], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < BN; ++bn) {
            const int n = n0 + 32 * (BN * wn + bn) + (lane & 31);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int i = 8 * (j / 4) + 4 * (lane >> 5) + (j % 4);
                const int64_t id = sid[32 * (BM * wm + bm) + i];
                if (id >= 0 && n < Fi) Yg[id * Fi + n] = acc[bm][bn][j];
            }
        }
}

// partial[chunk][m][n] = sum over the chunk's rows of Y[id, m] X'[id, n], one tile of 32 WM BM x 32 WN BN.
// The vertex id of a row is fetched one step before the row itself, so that the row loads of a
// step never wait for an id.
template <int WM, int WN, int BM, int BN, bool VEC>
__global__ __launch_bounds__(kBlock) void k_weight_gradient(const int32_t* __restrict__ ids, int64_t n_rows,
                                                            int64_t rows_per_chunk, const float* __restrict__ Y,
                                                            int Fi, const float* __restrict__ G, int Fo,
                                                            float* __restrict__ partial) {
    static_assert(WM * WN == 4, "four wavefronts per workgroup");
    constexpr int TM = 32 * WM * BM, TN = 32 * WN * BN;
    constexpr int NA = TM / 32, NB = TN / 32;  // 4-float pieces per thread and step
    __shared__ __attribute__((aligned(16))) float As[kStep][TM];   // Y rows, [row][m]
    __shared__ __attribute__((aligned(16))) float Bs[kStep][TN];   // X' rows, [row][n]
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = w % WM, wn = w / WM;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.z * TN;
    const int64_t first = (int64_t)blockIdx.x * rows_per_chunk;
    const int64_t last = std::min<int64_t>(first + rows_per_chunk, n_rows);
    const int tr = t >> 3, c4 = 4 * (t & 7);
    auto vertex = [&](int64_t r) -> int64_t { return r < last ? (ids ? (int64_t)ids[r] : r) : -1; };
    float4v ra[NA], rb[NB];
    auto fetch = [&](int64_t id) {
        const float* y = Y + (id >= 0 ? id * Fi + m0 + c4 : 0);
        const float* g = G + (id >= 0 ? id * Fo + n0 + c4 : 0);
#pragma unroll
        for (int i = 0; i < NA; ++i) ra[i] = load4<VEC>(y + 32 * i, id >= 0 ? Fi - (m0 + c4 + 32 * i) : 0);
#pragma unroll
        for (int i = 0; i < NB; ++i) rb[i] = load4<VEC>(g + 32 * i, id >= 0 ? Fo - (n0 + c4 + 32 * i) : 0);
    };
    floatx16 acc[BM][BN] = {};
    int64_t id_next = -1;
    if (first < last) {
        fetch(vertex(first + tr));
        id_next = vertex(first + kStep + tr);
    }
    for (int64_t r0 = first; r0 < last; r0 += kStep) {
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<float4v*>(&As[tr][c4 + 32 * i]) = ra[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<float4v*>(&Bs[tr][c4 + 32 * i]) = rb[i];
        __syncthreads();
        if (r0 + kStep < last) {
            fetch(id_next);
            id_next = vertex(r0 + 2 * kStep + tr);
        }
#pragma unroll
        for (int kk = 0; kk < kStep; kk += 2) {
            float a[BM], b[BN];
#pragma unroll
            for (int bm = 0; bm < BM; ++bm) a[bm] = As[kk + (lane >> 5)][32 * (BM * wm + bm) + (lane & 31)];
#pragma unroll
            for (int bn = 0; bn < BN; ++bn) b[bn] = Bs[kk + (lane >> 5)][32 * (BN * wn + bn) + (lane & 31)];
#pragma unroll
            for (int bm = 0; bm < BM; ++bm)
#pragma unroll
                for (int bn = 0; bn < BN; ++bn)
                    acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[bm], b[bn], acc[bm][bn], 0, 0, 0);
        }
        __syncthreads();
    }
    float* __restrict__ mine = partial + (int64_t)blockIdx.x * Fi * Fo;
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < BN; ++bn) {
            const int n = n0 + 32 * (BN * wn + bn) + (lane & 31);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int m = m0 + 32 * (BM * wm + bm) + 8 * (j / 4) + 4 * (lane >> 5) + (j % 4);
                if (m < Fi && n < Fo) mine[(int64_t)m * Fo + n] = acc[bm][bn][j];
            }
        }
}

// ---------------------------------------------------------------- widths of up to 128
// Loads of a lane's share of a row: BLOCKS floats, one for each 32-wide block of the width.  VEC: they
// are consecutive (lane p holds BLOCKS p, BLOCKS p + 1, ..: one wide load; the blocks then interleave,
// which only permutes the products' rows or columns and is undone when they are written); else
// float 32 i + p of block i, element by element, for widths that BLOCKS does not divide.  Lanes past
// the width read what is there: their products are never written.
template <int BLOCKS, bool VEC>
__device__ __forceinline__ void load_share(const float* __restrict__ row, int width, int p, float (&x)[BLOCKS]) {
    if constexpr (VEC) {
        typedef float vec_t __attribute__((ext_vector_type(BLOCKS), aligned(4)));
        const vec_t v = *reinterpret_cast<const vec_t*>(row + (BLOCKS * p < width ? BLOCKS * p : 0));
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) x[i] = v[i];
    } else {
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) x[i] = row[32 * i + p < width ? 32 * i + p : 0];
    }
}
template <int BLOCKS, bool VEC>
__device__ __forceinline__ int share_index(int block, int p) { return VEC ? BLOCKS * p + block : 32 * block + p; }

// partial[chunk] = sum over the chunk's rows of Y[id, :]^T X'[id, :], widths of at most 32 MT and 32 NT.
//
// The contraction runs over the rows, and both operands of v_mfma_f32_32x32x2_f32 want lane l to hold
// one feature (l % 32) of row l / 32 of a pair: which is how a row lies in memory.  So nothing goes through
// LDS: every wavefront takes its own rows, loads its operands straight into registers (one 16-byte load
// per lane and operand for a pair of rows of 128), D pairs ahead of the matrix core, and keeps the whole
// F_in x F_out product in its accumulators.  The wavefronts of a workgroup add theirs through LDS, in 32 bits, in pairs
// and in a fixed order, once at the end; sums of workgroups are added in double.  That is two additions behind a chain
// that is a quarter as long as a workgroup's: against 64 bits the error over 7 to 4.6 M rows and widths of 3 to 128 is
// half that of one chain per workgroup on average, and nowhere larger.
// Bound by HBM where a width is 16 (4.9 TB/s), by the launch with the few rows that 128 x 128 has here.
// Measured against tiles staged through LDS, partial sums included: 128 x 16, 3.9 M rows 0.53 -> 0.46 ms; 16 x 41, 250,000 rows 55 -> 29 us; 16 x 3, 400 rows 14.1 -> 6.4 us;
// 96 x 96, 869 / 30,000 / 100,000 rows 26 -> 14.6 / 33 -> 29 / 53 -> 59 us.
template <int MT, int NT, bool VA, bool VB>
__global__ __launch_bounds__(kBlock, MT * NT >= 16 ? 1 : 2) void k_weight_gradient_rows(
    const int32_t* __restrict__ ids, int64_t n_rows, int64_t rows_per_wave, const float* __restrict__ Y, int Fi,
    const float* __restrict__ G, int Fo, float* __restrict__ out) {
    // columns of Y, hence rows of W', that are this workgroup's
    const int m0 = blockIdx.y * 32 * MT, rows = std::min(Fi - m0, 32 * MT);
    Y += m0;
    constexpr int D = 8, WAVES = kBlock / 64;  // pairs of rows in flight, wavefronts
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, p = lane & 31, half = lane >> 5;
    const int64_t first = ((int64_t)blockIdx.x * WAVES + wave) * rows_per_wave;
    const int64_t last = std::min<int64_t>(first + rows_per_wave, n_rows);
    // (one block leaves room for four sums, of every fourth pair each: as many chains as 16 wavefronts would have)
    constexpr int CHAINS = MT * NT == 1 ? 4 : 1;
    floatx16 chain[CHAINS][MT][NT] = {};
    auto& acc = chain[0];
    // lane i (of the first 2 D) holds the vertex of row r + i; rows past the end repeat the last one
    // (without `ids` the load is of something else and not used: a branch around it would make every
    // step wait for all loads)
    const int32_t* __restrict__ id_src = ids ? ids : reinterpret_cast<const int32_t*>(Y);
    auto place = [&](int64_t r) -> int { return (int)std::min<int64_t>(r + (lane & (2 * D - 1)), last - 1); };
    auto vertices = [&](int64_t r) -> int { return id_src[place(r)]; };
    float a[D][MT], b[D][NT];
    auto fetch = [&](int d, int v) {
        const int v0 = __builtin_amdgcn_readlane(v, 2 * d), v1 = __builtin_amdgcn_readlane(v, 2 * d + 1);
        const int64_t id = half ? v1 : v0;
        load_share<MT, VA>(Y + id * Fi, rows, p, a[d]);
        load_share<NT, VB>(G + id * Fo, Fo, p, b[d]);
    };
    if (first < last) {
        // (loads in the order in which the loop issues them, so that the loop's waits count the same
        // loads whichever way it is entered)
        const int v0 = vertices(first);
        int v = vertices(first + 2 * D);
        __builtin_amdgcn_sched_barrier(0);
        const int now = ids ? v0 : place(first);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            fetch(d, now);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int64_t r = first; r < last; r += 2 * D) {
            if (r + 2 * D > last) {  // rows past the end count nothing: both factors zero
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const bool in = r + 2 * d + half < last;
#pragma unroll
                    for (int i = 0; i < MT; ++i) a[d][i] = in ? a[d][i] : 0.0f;
#pragma unroll
                    for (int j = 0; j < NT; ++j) b[d][j] = in ? b[d][j] : 0.0f;
                }
            }
            // a pair's registers are filled again as soon as the matrix core has taken them, so that a
            // fetch has the products of D - 1 pairs to arrive in, and its address arithmetic hides
            // behind those of its own (the last step fetches rows that are not used)
            const int next = ids ? v : place(r + 2 * D);
            v = vertices(r + 4 * D);
#pragma unroll
            for (int d = 0; d < D; ++d) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        chain[d % CHAINS][i][j] =
                            __builtin_amdgcn_mfma_f32_32x32x2f32(a[d][i], b[d][j], chain[d % CHAINS][i][j], 0, 0, 0);
                fetch(d, next);
                __builtin_amdgcn_sched_barrier(0);  // (left alone, all products come first and all fetches last)
            }
        }
    }
    if constexpr (CHAINS == 4) acc[0][0] = (acc[0][0] + chain[1][0][0]) + (chain[2][0][0] + chain[3][0][0]);
    // Each wavefront adds and writes its share of the blocks: wavefront o those numbered o kShare .. (o + 1) kShare - 1, row
    // by row; the others hand theirs over through LDS, kPass blocks of every owner at a time.  (Handed on from one half of
    // the wavefronts to the other until one has them all, and written by that one, 128 x 128 took 20 us more.)
    static_assert(WAVES == 4, "added in pairs");
    constexpr int B = MT * NT, kOwners = B < WAVES ? B : WAVES, kShare = B / kOwners, kPass = kShare > 2 ? 2 : 1;
    __shared__ float4v sums[kOwners * kPass * (WAVES - 1)][4 * 64];
    const int w = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
    for (int h = 0; h < kShare; h += kPass) {
        if (h > 0) __syncthreads();  // `sums` is written again
#pragma unroll
        for (int o = 0; o < kOwners; ++o) {
            if (w == o) continue;
#pragma unroll
            for (int g = 0; g < kPass; ++g) {
                const floatx16& x = acc[(o * kShare + h + g) / NT][(o * kShare + h + g) % NT];
                float4v* __restrict__ to = sums[(o * kPass + g) * (WAVES - 1) + (w < o ? w : w - 1)] + lane;
#pragma unroll
                for (int q = 0; q < 4; ++q) to[q * 64] = float4v{x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int o = 0; o < kOwners; ++o) {
            if (w != o) continue;
#pragma unroll
            for (int g = 0; g < kPass; ++g) {
                floatx16& x = acc[(o * kShare + h + g) / NT][(o * kShare + h + g) % NT];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4v* __restrict__ from = sums[(o * kPass + g) * (WAVES - 1)] + q * 64 + lane;
                    const float4v y0 = from[0], y1 = from[4 * 64], y2 = from[2 * 4 * 64];
#pragma unroll
                    for (int c = 0; c < 4; ++c) x[4 * q + c] = (x[4 * q + c] + y0[c]) + (y1[c] + y2[c]);
                }
            }
        }
    }
    float* __restrict__ mine = out + ((int64_t)blockIdx.x * Fi + m0) * Fo;
#pragma unroll
    for (int o = 0; o < kOwners; ++o) {
        if (w != o) continue;
        // (kShare divides NT: blocks of one row)
        const int i = o * kShare / NT, j0 = o * kShare % NT;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int m = share_index<MT, VA>(i, 8 * (e / 4) + 4 * half + (e % 4));
            if (m >= rows) continue;
            float* __restrict__ row = mine + m * Fo;
            if constexpr (VB && kShare > 1) {
                typedef float vec_t __attribute__((ext_vector_type(kShare), aligned(4)));
                vec_t v;
#pragma unroll
                for (int g = 0; g < kShare; ++g) v[g] = acc[i][j0 + g][e];
                const int n = NT * p + j0;  // (Fo is a multiple of NT)
                if (n < Fo) *reinterpret_cast<vec_t*>(row + n) = v;
            } else {
#pragma unroll
                for (int g = 0; g < kShare; ++g) {
                    const int n = share_index<NT, VB>(j0 + g, p);
                    if (n < Fo) row[n] = acc[i][j0 + g][e];
                }
            }
        }
    }
}

// W' of few rows in one launch: a workgroup of 16 wavefronts forms 32 x 32 of it from all rows, a sixteenth of them a wavefront, which has all its
// operands on their way at once; the wavefronts' sums meet in LDS and are added in double.
// Bound by the launch, the two loads behind each other and the lines that one CU gets through; partial sums need a second launch to add
// them (us, 16 x 3 / 32 x 32 / 41 x 41 / 64 x 64 / 128 x 128; 8 rows 3.2 / 3.4 / 3.8 / 3.9 / 4.7 -> 2.5 / 2.5 / 2.6 / 2.6 / 2.7, 64 rows 3.0 / 3.3 / 6.1 / 6.0 /
// 4.7 -> 3.0 / 3.0 / 3.1 / 3.2 / 3.3, 128 rows 5.4 / 5.7 / 6.1 / 6.0 / 7.0 -> 3.3 / 3.3 / 3.4 / 3.4 / 3.5, 384 rows 5.2 / 5.5 / 6.0 / 5.9 / 7.2 ->
// 4.9 / 4.8 / 5.3 / 5.1 / 5.1; from 450 on not for every width: 5.2 / 5.6 / 6.0 / 5.9 / 7.3 against 5.6 / 5.6 / 5.8 / 5.7 / 5.7, 512 rows 5.2 against 5.8 at
// 16 x 3).  Error against 64 bits 4e-8 to 7e-8 for 5e-8 to 9e-8.
constexpr int kFewWaves = 16, kFewRows = 384;
__global__ __launch_bounds__(64 * kFewWaves) void k_weight_gradient_few(const int32_t* __restrict__ ids, int n_rows, int rows_per_wave,
                                                                        const float* __restrict__ Y, int Fi,
                                                                        const float* __restrict__ G, int Fo, float* __restrict__ Wg) {
    constexpr int PAIRS = kFewRows / kFewWaves / 2, CHAINS = 4;
    __shared__ float part[kFewWaves][16 * 64];
    const int m0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
    const int lane = threadIdx.x & 63, p = lane & 31, half = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = wave * rows_per_wave, mine = std::min(rows_per_wave, n_rows - first);  // (0 or less: none)
    // (lanes past a width read what is there: their products are never written)
    const float* __restrict__ y = Y + (m0 + p < Fi ? m0 + p : 0);
    const float* __restrict__ g = G + (n0 + p < Fo ? n0 + p : 0);
    floatx16 chain[CHAINS] = {};
    if (mine > 0) {
        // lane i holds the vertex of row i; the row behind an odd number's last is that one again, with both factors zero
        const int row = first + std::min(lane, mine - 1), v = ids ? ids[row] : row;
        float a[PAIRS], b[PAIRS];
#pragma unroll
        for (int d = 0; d < PAIRS; ++d) {
            a[d] = b[d] = 0.0f;
            if (2 * d < mine) {
                const int v0 = __builtin_amdgcn_readlane(v, 2 * d), v1 = __builtin_amdgcn_readlane(v, 2 * d + 1);
                const int64_t id = half ? v1 : v0;
                a[d] = y[id * Fi];
                b[d] = g[id * Fo];
            }
        }
#pragma unroll
        for (int d = 0; d < PAIRS; ++d) {
            if (2 * d >= mine) continue;
            const bool in = 2 * d + half < mine;
            chain[d % CHAINS] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? a[d] : 0.0f, in ? b[d] : 0.0f, chain[d % CHAINS], 0, 0, 0);
        }
    }
    const floatx16 sum = (chain[0] + chain[1]) + (chain[2] + chain[3]);
#pragma unroll
    for (int e = 0; e < 16; ++e) part[wave][e * 64 + lane] = sum[e];
    __syncthreads();
    const int m = m0 + 8 * (wave / 4) + 4 * half + wave % 4, n = n0 + p;  // element `wave` of the accumulators
    if (m >= Fi || n >= Fo) return;
    double total = 0.0;
#pragma unroll
    for (int w = 0; w < kFewWaves; ++w) total += (double)part[w][threadIdx.x];
    Wg[(int64_t)m * Fo + n] = (float)total;
}

// Y'[id, n] = sum_k X'[id, k] W[n, k], widths of at most 128 (F_out = k) and 32 NT (F_in = n).
//
// W stays in LDS for the whole launch, in the order in which the matrix core takes it: the workgroups
// are persistent, each wavefront takes 32 rows at a time and loads them straight into registers, lane l
// its own row l % 32, four floats at a time (lanes l and l + 32 alternate: the contraction's order is free as
// long as both operands follow it), the next 32 rows while the matrix core works on these.  One
// 16-byte LDS read feeds four instructions, and no barrier is left in the loop.  Bound by HBM where a width is 16
// (4.9 TB/s).
// Measured against tiles of both operands staged through LDS: 128 x 16, 3.9 M rows 0.55 -> 0.46 ms; 16 x 41, 250,000 rows 27 -> 21 us; 16 x 3, 382 rows 5.4 -> 3.0 us;
// 96 x 96, 869 / 30,000 / 100,000 rows 11.9 -> 11.8 / 14.0 -> 14.0 / 38 -> 38 us (18.0 / 20.1 / 51 with W brought into
// LDS a float and a row at a time, and 16 chunks for 12).
template <int KC, int NT>  // KC: chunks of 8 floats of a row
__global__ __launch_bounds__(kBlock, 2) void k_input_gradient_rows(const int32_t* __restrict__ ids, int64_t n_rows,
                                                                   const float* __restrict__ G, int Fo,
                                                                   const float* __restrict__ W, int Fi,
                                                                   float* __restrict__ Yg) {
    const int n0 = blockIdx.y * 32 * NT, cols = std::min(Fi - n0, 32 * NT);  // columns of Y' that are this workgroup's
    W += (int64_t)n0 * Fo;
    Yg += n0;
    __shared__ float4v Ws[KC * 2 * NT * 32];  // [chunk][half][n]: W[n, 8 chunk + 4 half ..]
    __shared__ float4v out_all[kBlock / 64][32 * 8];  // 32 rows x 32 columns of results, private to a wavefront
    const int lane = threadIdx.x & 63, p = lane & 31, half = lane >> 5;
    typedef float vec_t __attribute__((ext_vector_type(4), aligned(4)));
    {   // W: a wavefront takes 16 rows x 16 columns at a time, so that a lane of four reads 64 bytes of a row and 16 of
        // them write 256 bytes of LDS; all loads before the first write
        constexpr int kSteps = (KC * NT + kBlock / 64 - 1) / (kBlock / 64);  // of KC NT such pieces
        float4v w[kSteps];
        const int top = std::max(Fo - 4, 0);
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int blk = i * (kBlock / 64) + (threadIdx.x >> 6);
            const int k = 16 * (blk % (KC / 2)) + 4 * (lane & 3), n = 16 * (blk / (KC / 2)) + (lane >> 2);
            const float* __restrict__ row = W + (int64_t)std::min(n, cols - 1) * Fo;
            if (Fo >= 4) {
                w[i] = *reinterpret_cast<const vec_t*>(row + std::min(k, top));
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) w[i][c] = row[std::min(c, Fo - 1)];
            }
        }
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int blk = i * (kBlock / 64) + (threadIdx.x >> 6);
            const int k = 16 * (blk % (KC / 2)) + 4 * (lane & 3), n = 16 * (blk / (KC / 2)) + (lane >> 2);
            // (the last columns of a row were read together with those before them)
            const int late = k - std::min(k, top);
            float4v x;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float y = w[i][c];
                if (c < 3 && late == 1) y = w[i][c + 1];
                if (c < 2 && late == 2) y = w[i][c + 2];
                if (c < 1 && late == 3) y = w[i][c + 3];
                x[c] = n < cols && k + c < Fo ? y : 0.0f;
            }
            if (KC * NT % (kBlock / 64) == 0 || n < 32 * NT) Ws[(k / 4) * (NT * 32) + n] = x;
        }
    }
    __syncthreads();
    const int64_t n_tiles = (n_rows + 31) / 32, step = (int64_t)gridDim.x * (kBlock / 64);
    auto vertex = [&](int64_t tile) -> int {
        const int64_t r = std::min<int64_t>(tile * 32 + p, n_rows - 1);
        return ids ? ids[r] : (int)r;
    };
    auto fetch = [&](float4v (&x)[KC], int v) {
        const float* __restrict__ row = G + (int64_t)v * Fo;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const int k = 8 * c + 4 * half;
            if (k + 4 <= Fo) {
                x[c] = *reinterpret_cast<const vec_t*>(row + k);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) x[c][i] = k + i < Fo ? row[k + i] : 0.0f;
            }
        }
    };
    auto process = [&](const float4v (&x)[KC], int64_t tile, int v) {
        floatx16 acc[NT] = {};
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            float4v w[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) w[j] = Ws[((c * 2 + half) * NT + j) * 32 + p];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[c][i], w[j][i], acc[j], 0, 0, 0);
            if (c % 2) __builtin_amdgcn_sched_barrier(0);  // (all of W read ahead would not fit the registers)
        }
        // 32 columns at a time through LDS, so that a store carries 16 bytes per lane and whole 128-byte
        // lines: single floats are four times as many stores as the counter of outstanding accesses holds,
        // and four columns of a lane's own row each are 32-byte pieces of lines (1.41 and 1.50 ms)
        float4v* __restrict__ ov = out_all[threadIdx.x >> 6];
        float* __restrict__ of = reinterpret_cast<float*>(ov);
        int vr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) vr[q] = __shfl(v, 8 * q + (lane >> 3), 64);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < 16; ++e) of[(8 * (e / 4) + 4 * half + (e % 4)) * 32 + p] = acc[j][e];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int n = 32 * j + 4 * (lane & 7);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4v y = ov[64 * q + lane];
                if (tile * 32 + 8 * q + (lane >> 3) >= n_rows) continue;
                float* __restrict__ o = Yg + (int64_t)vr[q] * Fi + n;
                if (n + 4 <= cols) {
                    *reinterpret_cast<vec_t*>(o) = y;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n + i < cols) o[i] = y[i];
                }
            }
        }
    };
    int64_t tile = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (tile >= n_tiles) return;
    float4v x0[KC], x1[KC];
    int v0 = vertex(tile), v1 = tile + step < n_tiles ? vertex(tile + step) : 0;
    fetch(x0, v0);
    for (;;) {
        const bool more = tile + step < n_tiles;
        int v2 = 0;
        if (more) {
            fetch(x1, v1);
            if (tile + 2 * step < n_tiles) v2 = vertex(tile + 2 * step);
        }
        process(x0, tile, v0);
        if (!more) break;
        tile += step;
        const bool again = tile + step < n_tiles;
        int v3 = 0;
        if (again) {
            fetch(x0, v2);
            if (tile + 2 * step < n_tiles) v3 = vertex(tile + 2 * step);
        }
        process(x1, tile, v1);
        if (!again) break;
        tile += step;
        v0 = v2;
        v1 = v3;
    }
}

// W'[e] = sum over chunks: LANES threads per element take every LANES-th chunk each, accumulate in double, and are added in a
// fixed order (the result does not depend on timing).  What bounds it is the chain of loads that a thread waits for, eight at a
// time, and then what a workgroup of E elements leaves of a line: a thousand partial sums want many lanes, large products wide
// elements, small ones more workgroups.
template <int E, int THREADS>
__global__ __launch_bounds__(THREADS) void k_weight_gradient_reduce(const float* __restrict__ partial, int n_chunks,
                                                                    int64_t total, float* __restrict__ Wg) {
    constexpr int LANES = THREADS / E;
    __shared__ double part[LANES][E + 1];
    const int el = threadIdx.x % E, cl = threadIdx.x / E;
    const int64_t e = (int64_t)blockIdx.x * E + el;
    double s = 0.0;
    if (e < total) {
        for (int c = cl; c < n_chunks; c += 8 * LANES) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = c + i * LANES < n_chunks ? partial[(c + i * LANES) * total + e] : 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) s += (double)x[i];
        }
    }
    part[cl][el] = s;
    __syncthreads();
    if (cl < 16) {  // (reads and writes no rows but those of its own remainder by 16)
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < LANES / 16; ++i) sum += part[cl + 16 * i][el];
        part[cl][el] = sum;
    }
    __syncthreads();
    if (cl == 0 && e < total) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += part[i][el];
        Wg[e] = (float)sum;
    }
}
template <int E, int THREADS>
void launch_reduce(const float* part, int64_t chunks, int64_t total, float* Wg, hipStream_t s) {
    static_assert(THREADS / E >= 16, "the last sum takes 16 lanes");
    hipLaunchKernelGGL((k_weight_gradient_reduce<E, THREADS>), dim3((unsigned)((total + E - 1) / E)), dim3(THREADS), 0, s, part,
                       (int)chunks, total, Wg);
}

// 16-byte row accesses need widths that are multiples of four and aligned bases.
bool aligned4(int Fa, int Fb, const void* a, const void* b) {
    return Fa % 4 == 0 && Fb % 4 == 0 && ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0;
}

// Output tile of a launch, by the extents of the two tiled dimensions (m is always "long" for the
// input gradient, whose rows are the active vertices).
enum TileShape { T128x128, T128x64, T64x128, T128x32, T32x128 };
TileShape tile_shape(int m, int n) {
    if (n <= 32 && m > 32) return T128x32;
    if (m <= 32 && n > 32) return T32x128;
    if (m > 64) return n > 64 ? T128x128 : T128x64;
    return T64x128;
}
void tile_dims(TileShape t, int* tm, int* tn) {
    static const int dims[5][2] = {{128, 128}, {128, 64}, {64, 128}, {128, 32}, {32, 128}};
    *tm = dims[t][0];
    *tn = dims[t][1];
}

int check_widths(int Fi, int Fo) {
    if (Fi < 1 || Fo < 1 || Fi > kMaxWidth || Fo > kMaxWidth) {
        epp_set_error("widths F_in=%d F_out=%d outside [1, %d]", Fi, Fo, kMaxWidth);
        return EPP_ERR_INVALID_ARG;
    }
    return EPP_OK;
}

// Row set of the products: N^k, or every vertex for k = -1.
int row_set(const epp_paths* p, int k, const int32_t** ids, int64_t* count) {
    if (k == -1) {
        *ids = nullptr;
        *count = p->n;
        return EPP_OK;
    }
    return epp_active_ids(p, k, ids, count);
}

// Widths that the kernels without operand tiles take (and their number of 32-wide blocks).
constexpr int kNarrow = 128;
bool narrow(int Fi, int Fo) { return Fi <= kNarrow && Fo <= kNarrow; }
int blocks_of(int F) { return F > 64 ? 4 : (F > 32 ? 2 : 1); }

// Workgroups of k_input_gradient_rows<kc, nt> that a CU holds at once (by its registers; four at most, with which the
// memory is busy).  More of them than the chip holds would run after the others, each for as long (96 x 39, 400,000
// rows: 81 us with 1,024 workgroups, 72 with 768).
int resident(int kc, int nt) {
    if (kc >= 16) return 2;
    if (kc == 12) return nt == 1 ? 3 : 2;
    if (kc == 8) return nt == 4 ? 2 : 3;
    return nt == 4 ? 3 : 4;
}

// Blocks of 32 columns of Y' (nt in all) that a workgroup of k_input_gradient_rows takes, 128 rows a round: fewer where the chip would
// not be full.  A wavefront's products then follow each other in a chain a half or a quarter as long, and a workgroup brings that much
// less of W into LDS (us, 1 / 2 / 4 blocks; 128 x 128, 11 rows 5.5 / 8.1 / 13.2, 2,000 6.3 / 9.0 / 14.5, 8,000 7.3 / 9.5 / 14.9, 12,000
// 11.4 / 10.2 / 15.2, 16,000 12.2 / 11.0 / 15.8, 24,000 16.3 / 17.4 / 17.8, 32,000 23.5 / 18.4 / 18.6; 64 x 64, 2,000 4.2 / 5.5, 16,000 4.7 / 6.1,
// 24,000 6.9 / 6.3).  Up to 16 floats a row leave a wavefront little to do but wait (128 x 16, 24,000 rows 5.3 / 5.7 / 5.8, 32,000 6.7 / 6.5 / 6.5).
int columns_at_once(int64_t tiles, int kc, int nt) {
    const int64_t blocks = (tiles + 3) / 4, most = kc <= 2 ? 768 : 256;
    int per = 1;
    while (per < nt && blocks * (nt / per) > most) per *= 2;
    return per;
}

// (where the rows have to run through one CU faster than partial sums are added: k_weight_gradient_few)
bool few_rows(int64_t n_rows, int Fi, int Fo) { return n_rows > 0 && n_rows <= kFewRows && narrow(Fi, Fo); }

// How the rows are cut into partial sums (at most `max_chunks` of them); not for few rows.
struct Chunks {
    int64_t per;    // rows per chunk; narrow widths: rows per wavefront
    int64_t count;  // partial sums
};
Chunks chunking(int64_t n_rows, int Fi, int Fo, int64_t max_chunks) {
    Chunks c;
    if (narrow(Fi, Fo)) {
        const int tiles = blocks_of(Fi) * blocks_of(Fo);
        // Four wavefronts.  Many rows: two rounds of the chip where a wavefront fills its SIMD, else four.  Up to 65,536:
        // one round, 16 rows per wavefront at least (one batch of fetches), as what a launch takes is then the rows that
        // follow each other in a wavefront, and what the partial sums cost to write and add (64 rows a wavefront, or
        // 16 wavefronts for up to 1,024 rows -> this: 869 rows, 64 x 64 24.7 -> 7.5 us, 16 x 16 11.6 -> 6.6, 96 x 96
        // 40.7 -> 14.6; 30,000 rows, 64 x 64 16.0 -> 15.2, 96 x 96 46 -> 29).  One block: half as many partial sums, until
        // that is 64 rows a wavefront (32 x 32, 16,000 rows 9.1 -> 8.2 us).
        if (n_rows <= 65536) {
            const int64_t chains = tiles == 1 ? 512 : 1024;
            c.per = std::max<int64_t>((n_rows + chains - 1) / chains, 16);
            if (tiles == 1) c.per = std::min<int64_t>(c.per, 64);  // (256 partial sums at most, whatever the widths)
        } else {
            const int64_t want = std::min<int64_t>(tiles >= 8 ? 512 : 1024, std::max<int64_t>(max_chunks, 1));
            c.per = std::max<int64_t>((n_rows + 4 * want - 1) / (4 * want), 64);
        }
        c.per = (c.per + 1) / 2 * 2;
        c.count = (n_rows + 4 * c.per - 1) / (4 * c.per);
        return c;
    }
    // operand tiles: enough chunks to fill the chip a few times over, whole steps each
    int tm, tn;
    tile_dims(tile_shape(Fi, Fo), &tm, &tn);
    const int64_t tiles = (int64_t)((Fi + tm - 1) / tm) * ((Fo + tn - 1) / tn);
    const int64_t want = std::min(std::max<int64_t>(1, 2048 / tiles), std::max<int64_t>(max_chunks, 1));
    c.per = std::max<int64_t>((n_rows + want - 1) / want, kMinChunkRows);
    c.per = (c.per + kStep - 1) / kStep * kStep;
    c.count = (n_rows + c.per - 1) / c.per;
    return c;
}

// Blocks of 32 columns of Y (mt in all) that a workgroup of k_weight_gradient_rows takes, for the same reason, while a wavefront has few
// rows (us, 1 / 2 / 4 blocks, partial sums added; 128 x 128, 2,000 rows 8.7 / 10.2 / 14.7, 8,000 15.4 / 15.8 / 19.9, 12,000 17.1 /
// 18.0 / 20.2, 16,000 20.2 / 18.4 / 22.9; 64 x 128, 16,000 14.4 / 14.8, 50,000 21.9 / 19.4; 64 x 64, 2,000 6.5 / 7.4, 8,000 9.0 / 9.8, 12,000 9.4 /
// 9.2; 128 x 16, 4,000 6.9 / 7.2 / 7.8, 12,000 8.7 / 8.8 / 8.2).
int rows_at_once(const Chunks& c, int mt, int nt) {
    const int64_t most = nt == 4 ? 768 : 256;
    int at_once = c.per <= 16 ? 1 : mt;
    while (at_once < mt && c.count * (mt / at_once) > most) at_once *= 2;
    return at_once;
}

template <int MT, int NT, bool VA, bool VB>
void launch_rows_wg(const Chunks& c, const int32_t* ids, int64_t n_rows, const float* Y, int Fi, const float* G, int Fo,
                    float* out, hipStream_t s) {
    hipLaunchKernelGGL((k_weight_gradient_rows<MT, NT, VA, VB>), dim3((unsigned)c.count, (unsigned)((Fi + 32 * MT - 1) / (32 * MT))),
                       dim3(256), 0, s, ids, n_rows, c.per, Y, Fi, G, Fo, out);
}
template <int MT, bool VA>
void launch_rows_wg_n(const Chunks& c, const int32_t* ids, int64_t n_rows, const float* Y, int Fi, const float* G, int Fo,
                      float* out, hipStream_t s) {
    const int nt = blocks_of(Fo);
    if (nt == 1) launch_rows_wg<MT, 1, VA, false>(c, ids, n_rows, Y, Fi, G, Fo, out, s);
    else if (nt == 2 && Fo % 2 == 0) launch_rows_wg<MT, 2, VA, true>(c, ids, n_rows, Y, Fi, G, Fo, out, s);
    else if (nt == 2) launch_rows_wg<MT, 2, VA, false>(c, ids, n_rows, Y, Fi, G, Fo, out, s);
    else if (Fo % 4 == 0) launch_rows_wg<MT, 4, VA, true>(c, ids, n_rows, Y, Fi, G, Fo, out, s);
    else launch_rows_wg<MT, 4, VA, false>(c, ids, n_rows, Y, Fi, G, Fo, out, s);
}

}  // namespace

extern "C" int64_t epp_weight_gradient_workspace(const epp_paths_t* paths, int k, int F_in, int F_out) {
    if (!paths) { epp_set_error("NULL argument"); return EPP_ERR_INVALID_ARG; }
    if (k < -1 || k > paths->L) { epp_set_error("k=%d outside [-1, %d]", k, paths->L); return EPP_ERR_INVALID_ARG; }
    if (check_widths(F_in, F_out) != EPP_OK) return EPP_ERR_INVALID_ARG;
    const int64_t n_rows = k < 0 ? paths->n : paths->set_size[k];
    const int64_t sums = few_rows(n_rows, F_in, F_out) ? 1 : std::max<int64_t>(chunking(n_rows, F_in, F_out, kNoChunkLimit).count, 1);
    return sums * F_in * F_out * (int64_t)sizeof(float);
}

namespace {

// Both weight-gradient entry points: partial sums of at most `max_chunks` blocks of rows go to
// `part` (max_chunks * F_in * F_out floats at least), a second kernel adds them in a fixed order.
int weight_gradient(const epp_paths* paths, int k, const float* Y, int F_in, const float* grad_X, int F_out,
                    float* grad_W, float* part, int64_t max_chunks, hipStream_t s) {
    const int32_t* ids = nullptr;
    int64_t n_rows = 0;
    EPP_TRY(row_set(paths, k, &ids, &n_rows));
    if (few_rows(n_rows, F_in, F_out)) {
        const int per = ((int)n_rows + 2 * kFewWaves - 1) / (2 * kFewWaves) * 2;
        hipLaunchKernelGGL(k_weight_gradient_few, dim3((unsigned)((F_in + 31) / 32), (unsigned)((F_out + 31) / 32)), dim3(64 * kFewWaves), 0, s,
                           ids, (int)n_rows, per, Y, F_in, grad_X, F_out, grad_W);
        EPP_HIP_TRY(hipGetLastError());
        return EPP_OK;
    }
    const Chunks c = chunking(n_rows, F_in, F_out, max_chunks);
    const int64_t per = c.per, chunks = c.count;
    if (epp_split_weight_gradient(F_in, F_out, n_rows)) {
        epp_launch_weight_gradient_split(chunks, 4 * per, ids, n_rows, Y, F_in, grad_X, F_out, part, s);
    } else if (chunks > 0 && narrow(F_in, F_out)) {
        const int mt = rows_at_once(c, blocks_of(F_in), blocks_of(F_out));
        if (mt == 1) launch_rows_wg_n<1, false>(c, ids, n_rows, Y, F_in, grad_X, F_out, part, s);
        else if (mt == 2 && F_in % 2 == 0) launch_rows_wg_n<2, true>(c, ids, n_rows, Y, F_in, grad_X, F_out, part, s);
        else if (mt == 2) launch_rows_wg_n<2, false>(c, ids, n_rows, Y, F_in, grad_X, F_out, part, s);
        else if (F_in % 4 == 0) launch_rows_wg_n<4, true>(c, ids, n_rows, Y, F_in, grad_X, F_out, part, s);
        else launch_rows_wg_n<4, false>(c, ids, n_rows, Y, F_in, grad_X, F_out, part, s);
    } else if (chunks > 0) {
        const TileShape shape = tile_shape(F_in, F_out);
        int tm, tn;
        tile_dims(shape, &tm, &tn);
        const dim3 grid((unsigned)chunks, (unsigned)((F_in + tm - 1) / tm), (unsigned)((F_out + tn - 1) / tn));
        const bool vec = aligned4(F_in, F_out, Y, grad_X);
#define EPP_LAUNCH_WG(WM, WN, BM, BN)                                                                            \
    do {                                                                                                         \
        if (vec)                                                                                                 \
            hipLaunchKernelGGL((k_weight_gradient<WM, WN, BM, BN, true>), grid, dim3(kBlock), 0, s, ids, n_rows, \
                               per, Y, F_in, grad_X, F_out, part);                                               \
        else                                                                                                     \
            hipLaunchKernelGGL((k_weight_gradient<WM, WN, BM, BN, false>), grid, dim3(kBlock), 0, s, ids, n_rows, \
                               per, Y, F_in, grad_X, F_out, part);                                               \
    } while (0)
        switch (shape) {
            case T128x128: EPP_LAUNCH_WG(2, 2, 2, 2); break;
            case T128x64: EPP_LAUNCH_WG(2, 2, 2, 1); break;
            case T64x128: EPP_LAUNCH_WG(2, 2, 1, 2); break;
            case T128x32: EPP_LAUNCH_WG(4, 1, 1, 1); break;
            case T32x128: EPP_LAUNCH_WG(1, 4, 1, 1); break;
        }
#undef EPP_LAUNCH_WG
    }
    const int64_t total = (int64_t)F_in * F_out;
    // Up to 128 partial sums are one round of loads for workgroups of 256 threads.  More, in workgroups of 1,024 (4 or 16 elements by 256
    // threads -> this): 250 of 41 x 41 / 64 x 64 / 128 x 128 4.5 / 6.2 / 7.6 -> 2.6 / 3.9 / 5.1 us; 1,021 of 16 x 16 / 16 x 41 / 64 x 16 / 64 x 47 /
    // 64 x 64 6.8 / 7.3 / 7.8 / 15.2 / 18.4 -> 4.6 / 5.1 / 4.9 / 8.8 / 7.7; 512 of 96 x 96 / 128 x 128 14.6 / 16.2 -> 7.6 / 8.4 (4 TB/s).  The number of
    // elements makes 64 to 512 workgroups of 16 x 16 to 128 x 128.
    if (chunks <= 128) {
        if (total >= 4096) launch_reduce<16, 256>(part, chunks, total, grad_W, s);
        else launch_reduce<4, 256>(part, chunks, total, grad_W, s);
    } else if (total >= 8192) {
        launch_reduce<32, 1024>(part, chunks, total, grad_W, s);
    } else if (total >= 4096) {
        launch_reduce<16, 1024>(part, chunks, total, grad_W, s);
    } else if (total >= 1024) {
        launch_reduce<8, 1024>(part, chunks, total, grad_W, s);
    } else {
        launch_reduce<4, 1024>(part, chunks, total, grad_W, s);
    }
    EPP_HIP_TRY(hipGetLastError());
    return EPP_OK;
}

}  // namespace

extern "C" int epp_weight_gradient(epp_paths_t* paths, int k, const float* Y, int F_in, const float* grad_X, int F_out,
                                   float* grad_W, void* workspace, int64_t workspace_bytes, epp_stream_t stream) {
    if (!paths || !Y || !grad_X || !grad_W || !workspace) { epp_set_error("NULL argument"); return EPP_ERR_INVALID_ARG; }
    if (k < -1 || k > paths->L) { epp_set_error("k=%d outside [-1, %d]", k, paths->L); return EPP_ERR_INVALID_ARG; }
    EPP_TRY(check_widths(F_in, F_out));
    const int64_t need = epp_weight_gradient_workspace(paths, k, F_in, F_out);
    if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 15)) {
        epp_set_error("workspace of %lld bytes (need %lld, 16-byte aligned)", (long long)workspace_bytes, (long long)need);
        return EPP_ERR_INVALID_ARG;
    }
    return weight_gradient(paths, k, Y, F_in, grad_X, F_out, grad_W, static_cast<float*>(workspace), kNoChunkLimit,
                           (hipStream_t)stream);
}

// ---- the entry point that allocates nothing --------------------------------------------------
// Partial sums of epp_weight_gradient_static: a file-scope device array instead of a caller's
// workspace.  Every GPU the library runs on holds its own copy until the process ends.  In host
// code the array's name is only a handle for the symbol lookup; the device address of the current
// GPU's copy comes from hipGetSymbolAddress, once per device, and is what the kernels receive.
constexpr size_t kStaticScratchBytes = 32u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
float* g_scratch_ptr[kMaxDevices] = {};  // per device; written once (the same value by any thread that races)
}  // namespace

int epp_static_scratch(float** ptr) {
    int dev = -1;
    EPP_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) { epp_set_error("device index %d not supported", dev); return EPP_ERR_INVALID_ARG; }
    float* p = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        void* addr = nullptr;
        EPP_HIP_TRY(hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch)));
        if (!addr) { epp_set_error("the static scratch array has no device address"); return EPP_ERR_HIP; }
        p = static_cast<float*>(addr);
        __atomic_store_n(&g_scratch_ptr[dev], p, __ATOMIC_RELEASE);
    }
    *ptr = p;
    return EPP_OK;
}

extern "C" int epp_weight_gradient_static(epp_paths_t* paths, int k, const float* Y, int F_in, const float* grad_X,
                                          int F_out, float* grad_W, epp_stream_t stream) {
    if (!paths || !Y || !grad_X || !grad_W) { epp_set_error("NULL argument"); return EPP_ERR_INVALID_ARG; }
    if (k < -1 || k > paths->L) { epp_set_error("k=%d outside [-1, %d]", k, paths->L); return EPP_ERR_INVALID_ARG; }
    EPP_TRY(check_widths(F_in, F_out));
    const int64_t block_bytes = (int64_t)F_in * F_out * (int64_t)sizeof(float);
    if (block_bytes > (int64_t)kStaticScratchBytes) {
        epp_set_error("F_in * F_out = %lld exceeds the %lld elements the static scratch array holds; use "
                      "epp_weight_gradient with a workspace", (long long)F_in * F_out,
                      (long long)(kStaticScratchBytes / sizeof(float)));
        return EPP_ERR_TOO_LARGE;
    }
    float* part = nullptr;
    EPP_TRY(epp_static_scratch(&part));
    // as many blocks of rows as fit the array; every block is written in full before the second
    // kernel reads it, so nothing left over from an earlier call is ever read
    return weight_gradient(paths, k, Y, F_in, grad_X, F_out, grad_W, part, (int64_t)kStaticScratchBytes / block_bytes,
                           (hipStream_t)stream);
}

extern "C" int epp_input_gradient(epp_paths_t* paths, int k, const float* grad_X, int F_out, const float* W, int F_in,
                                  float* grad_Y, epp_stream_t stream) {
    if (!paths || !grad_X || !W || !grad_Y) { epp_set_error("NULL argument"); return EPP_ERR_INVALID_ARG; }
    if (k < -1 || k > paths->L) { epp_set_error("k=%d outside [-1, %d]", k, paths->L); return EPP_ERR_INVALID_ARG; }
    EPP_TRY(check_widths(F_in, F_out));
    hipStream_t s = (hipStream_t)stream;
    const int32_t* ids = nullptr;
    int64_t n_rows = 0;
    EPP_TRY(row_set(paths, k, &ids, &n_rows));
    if (n_rows == 0) return EPP_OK;
    if (epp_split_input_gradient(F_in, F_out, n_rows)) {
        epp_launch_input_gradient_split(ids, n_rows, grad_X, F_out, W, F_in, grad_Y, s);
        EPP_HIP_TRY(hipGetLastError());
        return EPP_OK;
    }
    const int kc = (F_out + 7) / 8, nt = blocks_of(F_in);
    // (many rows of more than 48 floats onto one block of columns are left to the operand tiles: 16 x 64, 100,000 /
    // 400,000 / 2 M rows 10.0 / 28 / 123 us against 11.9 / 32 / 169, 32 x 128, 60,000 rows 11.1 against 13.0; not so 16 x 41,
    // 250,000 rows 27 against 21, nor 16 x 64, 30,000 rows 5.5 against 5.2)
    if (narrow(F_in, F_out) && !(nt == 1 && F_out > 48 && n_rows >= 50000)) {
        // persistent workgroups, as many as the chip holds at once
        const int64_t tiles = (n_rows + 31) / 32;
        // few rows: the columns in pieces of `per` blocks, a workgroup each
        const int per = columns_at_once(tiles, kc, nt);
        const unsigned pieces = (unsigned)((F_in + 32 * per - 1) / (32 * per));
        dim3 grid;
        auto blocks = [&](int at_once) { grid = dim3((unsigned)std::min<int64_t>((tiles + 3) / 4, at_once), pieces); };
#define EPP_LAUNCH_IGR(KC)                                                                                           \
    do {                                                                                                             \
        blocks(256 * resident(KC, per));                                                                             \
        if (per == 1)                                                                                                \
            hipLaunchKernelGGL((k_input_gradient_rows<KC, 1>), grid, dim3(kBlock), 0, s, ids, n_rows, grad_X, F_out, \
                               W, F_in, grad_Y);                                                                     \
        else if (per == 2)                                                                                           \
            hipLaunchKernelGGL((k_input_gradient_rows<KC, 2>), grid, dim3(kBlock), 0, s, ids, n_rows, grad_X, F_out, \
                               W, F_in, grad_Y);                                                                     \
        else                                                                                                         \
            hipLaunchKernelGGL((k_input_gradient_rows<KC, 4>), grid, dim3(kBlock), 0, s, ids, n_rows, grad_X, F_out, \
                               W, F_in, grad_Y);                                                                     \
    } while (0)
        if (kc <= 2) EPP_LAUNCH_IGR(2);
        else if (kc <= 4) EPP_LAUNCH_IGR(4);
        else if (kc <= 6) EPP_LAUNCH_IGR(6);
        else if (kc <= 8) EPP_LAUNCH_IGR(8);
        else if (kc <= 12) EPP_LAUNCH_IGR(12);
        else EPP_LAUNCH_IGR(16);
#undef EPP_LAUNCH_IGR
        EPP_HIP_TRY(hipGetLastError());
        return EPP_OK;
    }
    // rows are the long dimension: 128 of them per tile
    const TileShape shape = tile_shape(1 << 20, F_in);
    int tm, tn;
    tile_dims(shape, &tm, &tn);
    const dim3 grid((unsigned)((n_rows + tm - 1) / tm), (unsigned)((F_in + tn - 1) / tn));
    const bool vec = aligned4(F_out, F_out, grad_X, W);  // both operands are read along F_out
#define EPP_LAUNCH_IG(WM, WN, BM, BN)                                                                              \
    do {                                                                                                           \
        if (vec)                                                                                                   \
            hipLaunchKernelGGL((k_input_gradient<WM, WN, BM, BN, true>), grid, dim3(kBlock), 0, s, ids, n_rows,    \
                               grad_X, F_out, W, F_in, grad_Y);                                                    \
        else                                                                                                       \
            hipLaunchKernelGGL((k_input_gradient<WM, WN, BM, BN, false>), grid, dim3(kBlock), 0, s, ids, n_rows,   \
                               grad_X, F_out, W, F_in, grad_Y);                                                    \
    } while (0)
    switch (shape) {
        case T128x128: EPP_LAUNCH_IG(2, 2, 2, 2); break;
        case T128x64: EPP_LAUNCH_IG(2, 2, 2, 1); break;
        default: EPP_LAUNCH_IG(4, 1, 1, 1); break;  // T128x32
    }
#undef EPP_LAUNCH_IG
    EPP_HIP_TRY(hipGetLastError());
    return EPP_OK;
}
