// The products of the combination stage (epp_combine.hip) for two widths of 65 to 128 and many rows, where
// v_mfma_f32_32x32x2_f32 and not memory is the bound: on v_mfma_f32_32x32x16_bf16, which takes sixteen times the products
// a cycle, with every float split into three bfloat16 parts.
//
// x = h + m + l with h = bf16(x), m = bf16(x - h), l = x - h - m: both differences are exact, and so is l as a bfloat16 (24 bits
// less the 8 + 1 of each part before).  The bf16 instruction takes parts and products below 2^-126 as zero.  So x is 2^23 times the operand,
// by which every part of every float, denormal ones too, is above that, and every product that counts beside a result; sums go back
// by 2^-46.
//
// Of the nine products of two split floats six are formed; ml, lm and ll are at most 2^-24 of the product together.  Sums are in 32 bits,
// in two chains: hh, and the five small ones, added at the end.  (In one chain the matrix core drops the small products' low bits
// against a sum that has all of its own, always downwards: a bias of 2e-7 of a sum of 4,480 terms, which does not average out over
// thousands of such sums as errors do.)  Relative error of sums of 16 / 128 / 512 / 4,480 products of normal numbers against 64 bits (formed
// in one piece for this): fp32 instruction 7.3 / 20 / 41 / 120 e-8, one chain 3.3 / 16 / 34 / 104, two 3.2 / 6.5 / 13 / 42.  It is as
// large as the fp32 instruction's for W' where all products are positive (a million rows 3.05e-8, 2.94e-8), and larger in sums of one to
// three products: for one at most 2.1 x 2^-24 of the result (measured 1.8; fp32 1), on average the same (2.60e-8, 2.53e-8).
//
// What overflows in this is formed again with the fp32 instruction, 32 rows of Y' or a wavefront's part of W' at a time: rows of Y' whose
// largest magnitudes multiply to 2^66 or have 2^97 among them, parts of W' that came out infinite or NaN.  (So infinities are
// where fp32 has them, and NaN in the same rows and columns.)  These take about two and a half times as long as
// the others: a million rows of 128 x 128 620 to 700 / 550 to 600 us.
//
// 4.6 M rows, fp32 kernels -> this, timed in turn, 20 calls in a row, W' with the sum of its partial sums / Y': 128 x 128 1335 / 1424 -> 1203 /
// 1048 us, 96 x 96 1263 / 1039 -> 1091 / 744, 65 x 67 1230 / 1066 -> 996 / 700 (another card 1144 / 1015, 1039 / 727, 955 / 689).
// What bounds them is the card's power: at 128 x 128 the matrix core is busy 42 / 50 % of the cycles, at 1.65 to 2.1 / 1.55 to 1.9 GHz (fp32
// instruction 82 / 78 %, at 2.07).
//
// Operand layout of the 32x32x16 instruction: lane l supplies A[l % 32][8 (l / 32) ..] and B[8 (l / 32) ..][l % 32], eight
// elements; its accumulator is that of 32x32x2.

#include <algorithm>

#include "epp_internal.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));  // global accesses need no more
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr float kUp = 0x1p23f, kDown = 0x1p-46f;            // of both operands, of their products
constexpr float kMost = 0x1p120f, kMostProduct = 0x1p112f;  // of scaled operands (128 such products are 2^119)

// Three parts of eight floats, two to a word.
struct Parts { uintx4 h, m, l; };
__device__ __forceinline__ bf16x8 operand(uintx4 x) { return __builtin_bit_cast(bf16x8, x); }
__device__ __forceinline__ unsigned two_bf16(float x, float y) { return __builtin_bit_cast(unsigned, bf16x2{(__bf16)x, (__bf16)y}); }
// x - one of two bfloat16, in one instruction (the product with the other is a zero, or NaN beside one that is not finite).  The factors
// come from a register: as constants in the instruction they were taken for others.
__device__ __forceinline__ float less(float x, unsigned w, unsigned factors) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, factors), x, false);
}
template <class X>  // of x(i) kUp, x(i) the i-th of eight floats; `most`, if given, becomes the largest magnitude so far (NaN are passed over)
__device__ __forceinline__ Parts split(X x, float* most = nullptr) {
    Parts r;
    unsigned low = 0x0000BF80u, high = 0xBF800000u;  // -1 for one of two
    asm("" : "+s"(low), "+s"(high));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x(2 * i) * kUp, b = x(2 * i + 1) * kUp;
        if (most) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(*most) : "v"(a), "v"(b));
        r.h[i] = two_bf16(a, b);
        const float a1 = less(a, r.h[i], low), b1 = less(b, r.h[i], high);
        r.m[i] = two_bf16(a1, b1);
        r.l[i] = two_bf16(less(a1, r.m[i], low), less(b1, r.m[i], high));
    }
    return r;
}
__device__ __forceinline__ float most_of_wave(float x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = fmaxf(x, __shfl_xor(x, d, 64));
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
// Whether nothing overflows, from the largest magnitudes of what is multiplied.
__device__ __forceinline__ bool in_range(float most_a, float most_b) {
    return most_a < kMost && most_b < kMost && most_a * most_b < kMostProduct;
}

// The six products of N blocks: b's with a.
template <int N>
__device__ __forceinline__ void add_products(floatx16* sum, floatx16* small, const Parts (&a)[N], const Parts& b) {
#define EPP_MFMA(to, x, y)  \
    _Pragma("unroll") for (int j = 0; j < N; ++j) to[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(a[j].x), operand(b.y), to[j], 0, 0, 0)
    EPP_MFMA(small, l, h);
    EPP_MFMA(sum, h, h);
    EPP_MFMA(small, h, l);
    EPP_MFMA(small, m, m);
    EPP_MFMA(small, m, h);
    EPP_MFMA(small, h, m);
#undef EPP_MFMA
}

// partial[workgroup] = sum over the workgroup's rows of Y[id, :]^T X'[id, :].
//
// 16 rows at a time: a thread loads one feature of eight of them (256 consecutive bytes of a row per instruction, D steps ahead), splits
// them, which is what the instruction wants of a lane, and leaves its parts in LDS; then every wavefront adds a quarter of
// the product, 64 x 64.  A row is read and split once.  Sums of kSplitPiece rows at a time are formed, checked and added to the
// workgroup's: the error of the chain then stays below that of the fp32 instruction also where all products have one sign.
constexpr int kSplitPiece = 2304;
__global__ __launch_bounds__(256, 2) void k_weight_gradient_split(const int32_t* __restrict__ ids, int n_rows, int rows_per_group,
                                                                  const float* __restrict__ Y, int Fi, const float* __restrict__ G,
                                                                  int Fo, float* __restrict__ out) {
    constexpr int D = 3;  // steps of 16 rows in flight
    __shared__ uintx4 parts[2][3][2][256];  // [step][part][half][feature of Y, then of X' from 128 on]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), p = lane & 31, half = lane >> 5;
    const int64_t group_first = (int64_t)blockIdx.x * rows_per_group;
    if (group_first >= n_rows) return;
    const int group_last = (int)std::min<int64_t>(group_first + rows_per_group, n_rows);
    // what the thread loads: eight rows of every step, one feature of Y and one of X' (past the width the last one: its products
    // are never written)
    const int rows = 8 * (wave >> 1), feature = 64 * (wave & 1) + lane;
    const int fa = std::min(feature, Fi - 1), fb = std::min(feature, Fo - 1);
    // what it multiplies
    const int m0 = 64 * (wave & 1), n0 = 64 * (wave >> 1);
    float* __restrict__ mine = out + (int64_t)blockIdx.x * Fi * Fo;
    // (without `ids` the load is of something else and not used: a branch around it would make a step wait for all loads)
    const int32_t* __restrict__ id_src = ids ? ids : reinterpret_cast<const int32_t*>(Y);
    int buffer = 0;  // (goes on from piece to piece)
    for (int first = (int)group_first; first < group_last; first += kSplitPiece) {
        const int last = std::min(first + kSplitPiece, group_last);
        // Lane i (of eight) holds the vertex of the thread's i-th row of a step (rows past the end repeat the last one), from D steps before
        // that row is loaded, so that the wait for it is not one for rows that were asked for later.
        auto place = [&](int r) { return std::min(r + rows + (lane & 7), last - 1); };
        float a[D][8], b[D][8];
        auto fetch = [&](int d, int v) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int64_t id = __builtin_amdgcn_readlane(v, i);
                a[d][i] = (Y + id * Fi)[fa];
                b[d][i] = (G + id * Fo)[fb];
            }
        };
        int vertex[D];
        floatx16 sum[2][2] = {}, small[2][2] = {};  // [block of X'][block of Y]
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int v = id_src[place(first + 16 * d)];
            fetch(d, ids ? v : place(first + 16 * d));
            vertex[d] = id_src[place(first + 16 * (d + D))];
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int r0 = first; r0 < last; r0 += 16 * D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int r = r0 + 16 * d;
                if (r + 16 > last) {  // rows past the end count nothing
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        a[d][i] = r + rows + i < last ? a[d][i] : 0.0f;
                        b[d][i] = r + rows + i < last ? b[d][i] : 0.0f;
                    }
                }
                {
                    const Parts x = split([&](int i) { return a[d][i]; });
                    parts[buffer][0][wave >> 1][feature] = x.h;
                    parts[buffer][1][wave >> 1][feature] = x.m;
                    parts[buffer][2][wave >> 1][feature] = x.l;
                    const Parts z = split([&](int i) { return b[d][i]; });
                    parts[buffer][0][wave >> 1][128 + feature] = z.h;
                    parts[buffer][1][wave >> 1][128 + feature] = z.m;
                    parts[buffer][2][wave >> 1][128 + feature] = z.l;
                }
                __builtin_amdgcn_sched_barrier(0);
                fetch(d, ids ? vertex[d] : place(r + 16 * D));
                __builtin_amdgcn_sched_barrier(0);
                vertex[d] = id_src[place(r + 16 * 2 * D)];
                // (a wavefront writes to this buffer again only after the next step's barrier, behind which all have read it)
                __syncthreads();
                auto read = [&](int f) {
                    return Parts{parts[buffer][0][half][f], parts[buffer][1][half][f], parts[buffer][2][half][f]};
                };
                const Parts x[2] = {read(m0 + p), read(m0 + 32 + p)};
#pragma unroll
                for (int j = 0; j < 2; ++j) add_products(sum[j], small[j], x, read(128 + n0 + 32 * j + p));
                buffer ^= 1;
            }
        }
        bool finite = true;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                sum[j][i] = (sum[j][i] + small[j][i]) * kDown;
#pragma unroll
                for (int e = 0; e < 16; ++e) finite &= fabsf(sum[j][i][e]) < INFINITY;
            }
        if (__ballot(!finite)) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) sum[j][i] = floatx16{};
            constexpr int P = 8;  // pairs of rows at a time
            auto ids_of = [&](int r) { return id_src[std::min(r + (lane & (2 * P - 1)), last - 1)]; };
            int ahead = ids_of(first);
            for (int r = first; r < last; r += 2 * P) {
                const int now = ahead;
                ahead = ids_of(r + 2 * P);
                float x[P][2], z[P][2];
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const int at = std::min(r + 2 * q + half, last - 1);
                    const int64_t v = ids ? (half ? __builtin_amdgcn_readlane(now, 2 * q + 1) : __builtin_amdgcn_readlane(now, 2 * q)) : at;
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        x[q][u] = (Y + v * Fi)[std::min(m0 + 32 * u + p, Fi - 1)];
                        z[q][u] = (G + v * Fo)[std::min(n0 + 32 * u + p, Fo - 1)];
                    }
                }
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const bool in = r + 2 * q + half < last;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            sum[j][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? x[q][i] : 0.0f, in ? z[q][j] : 0.0f, sum[j][i], 0, 0, 0);
                }
            }
        }
        int m1 = m0 + 4 * half;
        asm volatile("" : "+v"(m1));  // (the places' offsets are not kept in registers through the loop)
        auto element = [&](int i, int j, int e) {
            return std::min(m1 + 32 * i + 8 * (e / 4) + e % 4, Fi - 1) * Fo + std::min(n0 + 32 * j + p, Fo - 1);
        };
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (first > (int)group_first) {
                    float before[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) before[e] = mine[element(i, j, e)];
#pragma unroll
                    for (int e = 0; e < 16; ++e) sum[j][i][e] += before[e];
                }
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (m1 + 32 * i + 8 * (e / 4) + e % 4 < Fi && n0 + 32 * j + p < Fo) mine[element(i, j, e)] = sum[j][i][e];
            }
    }
}

// Y'[id, n] = sum_k X'[id, k] W[n, k] for F_out of at most 16 KS (k), F_in of at most 32 NT (n).
//
// W's parts stay in LDS for the whole launch, in the order in which the matrix core takes them; a workgroup fills a CU and is
// persistent.  A wavefront takes 32 rows at a time, of which a lane loads its own row l % 32, four floats at a time (lanes l
// and l + 32 alternate), the next 32 rows' as soon as it has split these.  The rows are the columns of the instruction's
// result, so that a lane has four consecutive floats of its row at a time; they go through LDS to be stored in whole lines.
constexpr int kSplitThreads = 512, kSplitWaves = kSplitThreads / 64;
// FULL: F_in is 32 NT.  (Stores under no condition: behind others the next rows' wait could not tell how many there are, and would be
// for all of them.)
template <int KS, int NT, bool FULL>
__global__ __launch_bounds__(kSplitThreads, 2) void k_input_gradient_split(const int32_t* __restrict__ ids, int64_t n_rows,
                                                                           const float* __restrict__ G, int Fo,
                                                                           const float* __restrict__ W, int Fi,
                                                                           float* __restrict__ Yg) {
    constexpr int N = 32 * NT;
    __shared__ uintx4 Ws[3][KS * 2 * N];  // [part][step][half][n]
    __shared__ unsigned w_most;           // bits of W's largest magnitude (NaN are passed over)
    __shared__ float4v out_all[kSplitWaves][32 * 8];  // 32 rows x 32 columns of results, private to a wavefront
    const int lane = threadIdx.x & 63, p = lane & 31, half = lane >> 5;
    // Element i (of four) of the quadruple that starts at k; the last ones of a row start at F_out - 4 and have what comes
    // before k as zeros in W.
    const int top = Fo - 4;
    if (threadIdx.x == 0) w_most = 0;
    __syncthreads();
    float most_w = 0.0f;
    for (int i = threadIdx.x; i < KS * 2 * N; i += kSplitThreads) {
        const int n = i / (KS * 2), s = i % (KS * 2) / 2, h = i % 2;
        const float* __restrict__ row = W + (int64_t)std::min(n, Fi - 1) * Fo;
        float x[8];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int k = 16 * s + 8 * q + 4 * h, from = std::min(k, top);
            const float4u w = *reinterpret_cast<const float4u*>(row + from);
#pragma unroll
            for (int c = 0; c < 4; ++c) x[4 * q + c] = n < Fi && k < Fo && from + c >= k ? w[c] : 0.0f;
        }
        const Parts w = split([&](int j) { return x[j]; }, &most_w);
        Ws[0][(s * 2 + h) * N + n] = w.h;
        Ws[1][(s * 2 + h) * N + n] = w.m;
        Ws[2][(s * 2 + h) * N + n] = w.l;
    }
    most_w = most_of_wave(most_w);
    if (lane == 0) atomicMax(&w_most, __float_as_uint(most_w));
    __syncthreads();
    most_w = __uint_as_float(__builtin_amdgcn_readfirstlane(w_most));

    const int64_t n_tiles = (n_rows + 31) / 32, step = (int64_t)gridDim.x * kSplitWaves;
    auto vertex = [&](int64_t tile) -> int {
        const int64_t r = std::min<int64_t>(tile * 32 + p, n_rows - 1);
        return ids ? ids[r] : (int)r;
    };
    auto quad = [&](const float* __restrict__ row, int c) {  // (F_out is above 16 (KS - 2))
        const int k = 8 * c + 4 * half;
        return *reinterpret_cast<const float4u*>(row + (8 * c + 8 <= 16 * (KS - 2) ? k : std::min(k, top)));
    };
    int64_t tile = (int64_t)blockIdx.x * kSplitWaves + (threadIdx.x >> 6);
    if (tile >= n_tiles) return;
    float4v x[2 * KS];
    int v = vertex(tile), next = vertex(std::min(tile + step, n_tiles - 1));
    {
        const float* __restrict__ row = G + (int64_t)v * Fo;
#pragma unroll
        for (int c = 0; c < 2 * KS; ++c) {
            x[c] = quad(row, c);
            __builtin_amdgcn_sched_barrier(0);  // (in the order of the loop's loads, whose waits then count the same ones)
        }
    }
    for (; tile < n_tiles; tile += step) {
        const float* __restrict__ next_row = G + (int64_t)next * Fo;
        const int after = vertex(std::min(tile + 2 * step, n_tiles - 1));
        floatx16 sum[NT] = {}, small[NT] = {};
        float most = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const Parts b = split([&](int i) { return x[2 * s + i / 4][i % 4]; }, &most);
            // (behind the last tile these are read once more and not used)
            x[2 * s] = quad(next_row, 2 * s);
            x[2 * s + 1] = quad(next_row, 2 * s + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int at = (s * 2 + half) * N + 32 * j + p;
                const Parts w[1] = {{Ws[0][at], Ws[1][at], Ws[2][at]}};
                add_products(sum + j, small + j, w, b);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) sum[j] = (sum[j] + small[j]) * kDown;
        if (__ballot(!in_range(most, most_w))) {
#pragma unroll
            for (int j = 0; j < NT; ++j) sum[j] = floatx16{};
            const float* __restrict__ row = G + (int64_t)v * Fo;
            for (int k0 = 0; k0 < Fo; k0 += 8) {
                const int k = k0 + 4 * half, from = std::min(k, top);
                const float4u g = *reinterpret_cast<const float4u*>(row + from);
                float4u w[NT];
#pragma unroll
                for (int j = 0; j < NT; ++j) w[j] = *reinterpret_cast<const float4u*>(W + (int64_t)std::min(32 * j + p, Fi - 1) * Fo + from);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool in = k < Fo && from + c >= k;
#pragma unroll
                    for (int j = 0; j < NT; ++j)  // (columns past F_in are not written)
                        sum[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? w[j][c] : 0.0f, in ? g[c] : 0.0f, sum[j], 0, 0, 0);
                }
            }
        }
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));  // (what follows from it is not kept in registers through the products)
        float4v* __restrict__ ov = out_all[t >> 6];
        const int l = t & 63, own = l & 31, upper = l >> 5;
        int vr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) vr[q] = __shfl(v, 8 * q + (l >> 3), 64);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            __builtin_amdgcn_wave_barrier();
            // (quadruple c of row r lies at place c ^ r % 8, so that the rows' accesses spread over the banks)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ov[own * 8 + ((2 * q + upper) ^ (own & 7))] = float4v{sum[j][4 * q], sum[j][4 * q + 1], sum[j][4 * q + 2], sum[j][4 * q + 3]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int n = 32 * j + 4 * (l & 7);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = 8 * q + (l >> 3);
                const float4v y = ov[r * 8 + ((l & 7) ^ (r & 7))];
                // (rows past the end are the last one once more, and so are their results)
                float* __restrict__ o = Yg + (int64_t)vr[q] * Fi + n;
                if (FULL || n + 4 <= Fi) {
                    *reinterpret_cast<float4u*>(o) = y;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n + i < Fi) o[i] = y[i];
                }
            }
        }
        v = next;
        next = after;
    }
}

}  // namespace

// One width of up to 64 leaves memory the bound (128 x 64: 12 instructions for 768 bytes), and fewer rows the launch.  fp32 kernels -> this
// in us, W' with the sum of its partial sums: 128 x 128, 10,000 / 20,000 / 40,000 / 100,000 rows 21.9 -> 21.8, 29.0 -> 21.9, 32.5 -> 25.7,
// 61 -> 43; 65 x 67 20.1 -> 17.4, 27.8 -> 18.7, 31.7 -> 24.2, 62 -> 39; 65 x 128, 16,400 rows 26.4 -> 19.5.  Y', 20,000 / 40,000 / 100,000:
// 16.7 -> 18.4, 27.5 -> 19.0, 51 -> 31.6; 65 x 67 12.2 -> 11.1, 19.5 -> 12.1, 35.8 -> 21.5; 65 x 128, 33,000 rows 24.8 -> 15.4.  (W' of up to 65,536
// rows is cut into 256 workgroups, as the fp32 kernel wants it; two fit a CU here, and 512 have not been tried.)
static bool split_widths(int Fi, int Fo) { return Fi > 64 && Fo > 64 && Fi <= 128 && Fo <= 128; }
bool epp_split_weight_gradient(int Fi, int Fo, int64_t n_rows) { return split_widths(Fi, Fo) && n_rows > 16384; }
bool epp_split_input_gradient(int Fi, int Fo, int64_t n_rows) { return split_widths(Fi, Fo) && n_rows > 32768; }

void epp_launch_weight_gradient_split(int64_t groups, int64_t rows_per_group, const int32_t* ids, int64_t n_rows, const float* Y,
                                      int Fi, const float* G, int Fo, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_weight_gradient_split, dim3((unsigned)groups), dim3(256), 0, s, ids, (int)n_rows, (int)rows_per_group, Y, Fi, G,
                       Fo, out);
}

void epp_launch_input_gradient_split(const int32_t* ids, int64_t n_rows, const float* G, int Fo, const float* W, int Fi, float* Yg,
                                     hipStream_t s) {
    const int64_t tiles = (n_rows + 31) / 32;
    const dim3 grid((unsigned)std::min<int64_t>((tiles + kSplitWaves - 1) / kSplitWaves, 256)), block(kSplitThreads);
#define EPP_LAUNCH(KS, NT)                                                                                                      \
    do {                                                                                                                        \
        if (Fi == 32 * NT)                                                                                                      \
            hipLaunchKernelGGL((k_input_gradient_split<KS, NT, true>), grid, block, 0, s, ids, n_rows, G, Fo, W, Fi, Yg);       \
        else                                                                                                                    \
            hipLaunchKernelGGL((k_input_gradient_split<KS, NT, false>), grid, block, 0, s, ids, n_rows, G, Fo, W, Fi, Yg);      \
    } while (0)
    if (Fo <= 96) {
        if (Fi <= 96) EPP_LAUNCH(6, 3);
        else EPP_LAUNCH(6, 4);
    } else {
        if (Fi <= 96) EPP_LAUNCH(8, 3);
        else EPP_LAUNCH(8, 4);
    }
#undef EPP_LAUNCH
}
