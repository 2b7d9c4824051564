// Gather-reduce over whole rows (Alg. 2, aggregation loop): small paths, and very narrow rows.
//
// On a small path the group kernel (epp_aggregate.hip) is bound by launches and dependent loads, not by
// what it moves: two kernels of about 5 us each (groups, then the rows cut by their boundaries), and in
// the first a chain of group table -> row id and pairs -> LDS -> gathers.  Here a row is processed
// whole, so that nothing is left to add up afterwards and no table has to be built beforehand:
//   * T lanes read a source row, four floats each (the last of them steps back so that it ends at
//     the row's end: rows of any width are read 16 bytes at a time; a row of three floats or less is
//     one access); P such slots share a row's entries, U at a time each, and add their sums by
//     exchanging lanes;
//   * a row of more than `limit` entries is left to the whole workgroup, which takes the long rows
//     among its own one after the other;
//   * a row of more than a few steps of a workgroup is cut into chunks, one workgroup each, at the
//     front of the grid, and the last of them to be done adds the chunks' sums.
// The order of the additions depends on the path and the width only: equal inputs give equal bits.
//
// Bound by the address units where the sources lie in L2: a slot's pairs are therefore loaded by its lanes, one each, and handed
// on between them; every lane used to load all four (us, before / now / groups: 1.3 M entries, 60,000 sources, F = 16: 27.6 /
// 24.6 / 29.2, F = 32: 34.4 / 29.0 / 36.1; 7.1 M, 1.1 M sources, F = 16: 120 / 103 / 115; 13,938, 2,708 sources, F = 16:
// 7.4 / 6.8 / 12.2; 4.6 M, 89,000, F = 4: 37 / 36 / 50).

#include <cstdlib>

#include "epp_internal.h"

namespace {

constexpr int kBlock = 256;
constexpr int kU = 4;  // entries in flight per slot (eight cost half the wavefronts in flight and gain nothing)

typedef int int2v __attribute__((ext_vector_type(2)));

// VEC floats at 4-byte alignment (global accesses need no more): one access of 4 VEC bytes.  (Three
// floats element by element: a vector of three is read and written as one of four.)
template <int VEC>
__device__ __forceinline__ void load_frag(const float* __restrict__ p, float (&x)[VEC]) {
    if constexpr (VEC == 1 || VEC == 3) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) x[i] = p[i];
    } else {
        typedef float vec_t __attribute__((ext_vector_type(VEC), aligned(4)));
        const vec_t v = *reinterpret_cast<const vec_t*>(p);
#pragma unroll
        for (int i = 0; i < VEC; ++i) x[i] = v[i];
    }
}
template <int VEC>
__device__ __forceinline__ void store_frag(float* __restrict__ p, const float (&x)[VEC]) {
    if constexpr (VEC == 1 || VEC == 3) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) p[i] = x[i];
    } else {
        typedef float vec_t __attribute__((ext_vector_type(VEC), aligned(4)));
        vec_t v;
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = x[i];
        *reinterpret_cast<vec_t*>(p) = v;
    }
}

struct RowArgs {
    const int2v* cv;
    const int32_t* rowptr;
    const int32_t* row_ids;  // NULL: identity
    int n_rows;
    int user;                // which of a cut row's counts is this width's
    const float* in;
    float* out;
    int F;
    int log2p;               // slots per row
    int limit;               // longest row that is not left to the workgroup
    int log2_chunk;          // 2^: entries of a chunk, and the longest row that is not cut into chunks
    int has_long;            // some row is longer than `limit`
    int chunk_blocks;        // workgroups that take one chunk of a cut row each, before the others
    LongRow* long_rows;
    const int* long_head;
    float* pieces;           // the chunks' sums, F floats each
    // launch for the inner path that shares the arrays only
    const float* zero;           // what an entry that is not the inner path's gathers
    const unsigned int* only;    // bitmap of the inner path's rows
};

// Entry u of a step, of which every lane of a slot has loaded its share: lane i of the slot's first
// four those numbered i, i + 4, ..
template <int LOG2T, int N>
__device__ __forceinline__ int2v step_entry(const int2v (&mine)[N], int u) {
    if constexpr (LOG2T == 0) return mine[u];
    else if constexpr (LOG2T == 1) {  // (two slots in four lanes)
        const int2v e = mine[u >> 1];
        return u & 1 ? int2v{__builtin_amdgcn_mov_dpp(e.x, 0xF5, 0xF, 0xF, true), __builtin_amdgcn_mov_dpp(e.y, 0xF5, 0xF, 0xF, true)}
                     : int2v{__builtin_amdgcn_mov_dpp(e.x, 0xA0, 0xF, 0xF, true), __builtin_amdgcn_mov_dpp(e.y, 0xA0, 0xF, 0xF, true)};
    } else {
        const int2v e = mine[0];
        switch (u) {  // quad_perm:[u,u,u,u]
            case 0: return int2v{__builtin_amdgcn_mov_dpp(e.x, 0x00, 0xF, 0xF, true), __builtin_amdgcn_mov_dpp(e.y, 0x00, 0xF, 0xF, true)};
            case 1: return int2v{__builtin_amdgcn_mov_dpp(e.x, 0x55, 0xF, 0xF, true), __builtin_amdgcn_mov_dpp(e.y, 0x55, 0xF, 0xF, true)};
            case 2: return int2v{__builtin_amdgcn_mov_dpp(e.x, 0xAA, 0xF, 0xF, true), __builtin_amdgcn_mov_dpp(e.y, 0xAA, 0xF, 0xF, true)};
            default: return int2v{__builtin_amdgcn_mov_dpp(e.x, 0xFF, 0xF, 0xF, true), __builtin_amdgcn_mov_dpp(e.y, 0xFF, 0xF, 0xF, true)};
        }
    }
}

// acc = sum of the entries j0, j0 + 1, .. (U at a time, `step` apart) of [j0, p1).  The pairs of the
// next step are fetched while the rows of this one are on their way, each by one lane of the slot, which hands it to the others.
//
// A step that reaches past p1 gathers the last entry again, with weight zero, and one that belongs to the outer
// path only gathers zeros.  That adds zero, or NaN where the row or the weight holds an infinity.  EXACT clears both
// factors in the last step, which costs a path of 7,000 entries 0.2 us of 4.1; without it the caller looks at
// the sums, and forms those that are not numbers again from the slot's own entries alone (add_own_entries).
template <int VEC, int LOG2T, int U, bool INNER, bool EXACT>
__device__ __forceinline__ void add_entries(const RowArgs& a, const float* __restrict__ src, int j0, int p1, int step,
                                            float (&acc)[VEC]) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.0f;
    if (j0 >= p1) return;
    constexpr int kSharers = LOG2T >= 2 ? 4 : 1 << LOG2T, kMine = U / kSharers;
    static_assert(U == 4, "one step of a slot is what four lanes load");
    const int q = (int)threadIdx.x & (kSharers - 1);
    int2v mine[kMine];
#pragma unroll
    for (int k = 0; k < kMine; ++k) mine[k] = a.cv[min(j0 + k * kSharers + q, p1 - 1)];
    for (int j = j0; j < p1; j += step) {
        int2v e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) e[u] = step_entry<LOG2T>(mine, u);
        float x[U][VEC];
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* p = src + (size_t)(e[u].x & kEntCol) * (size_t)a.F;
            if constexpr (INNER) p = (e[u].x & kEntOuterOnly) ? a.zero : p;
            load_frag<VEC>(p, x[u]);
            w[u] = j + u < p1 ? __int_as_float(e[u].y) : 0.0f;
            if constexpr (INNER && EXACT) w[u] = (e[u].x & kEntOuterOnly) ? 0.0f : w[u];
        }
        if (j + step < p1) {
#pragma unroll
            for (int k = 0; k < kMine; ++k) mine[k] = a.cv[min(j + step + k * kSharers + q, p1 - 1)];
        }
        if (EXACT && j + U > p1) {
            asm volatile("");  // (keeps the branch)
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) x[u][i] = j + u < p1 ? x[u][i] : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = fmaf(w[u], x[u][i], acc[i]);
        }
    }
}

template <int VEC, int U, bool INNER>
__device__ __forceinline__ void add_own_entries(const RowArgs& a, const float* __restrict__ src, int j0, int p1, int step,
                                                float (&acc)[VEC]) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.0f;
    for (int j = j0; j < p1; j += step) {
        for (int q = j; q < min(j + U, p1); ++q) {
            const int2v own = a.cv[q];
            if constexpr (INNER) {
                if (own.x & kEntOuterOnly) continue;
            }
            float x[VEC];
            load_frag<VEC>(src + (size_t)(own.x & kEntCol) * (size_t)a.F, x);
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = fmaf(__int_as_float(own.y), x[i], acc[i]);
        }
    }
}

template <int VEC>
__device__ __forceinline__ bool not_numbers(const float (&acc)[VEC]) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < VEC; i += 2) bad |= (bool)__builtin_isunordered(acc[i], acc[i + 1 < VEC ? i + 1 : i]);
    return bad;
}

// o[f ..] of the calling thread's lanes = sum of what the slots of the workgroup add up each: acc = add(f).  Only the first
// wavefront writes, PIECE: past the L2, for workgroups on other XCDs.
template <int VEC, int LOG2T, bool PIECE, class Add>
__device__ __forceinline__ void sum_by_workgroup(const RowArgs& a, float* __restrict__ o, float (*part)[(1 << LOG2T) * VEC], Add add) {
    constexpr int T = 1 << LOG2T;
    const int t = threadIdx.x & (T - 1);
    for (int f0 = 0; f0 < a.F; f0 += T * VEC) {
        const bool fok = f0 + t * VEC < a.F;
        const int f = fok ? min(f0 + t * VEC, a.F - VEC) : 0;
        float acc[VEC];
        add(f, acc);
#pragma unroll
        for (int d = T; d < 64; d <<= 1) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], d, 64);
        }
        if ((threadIdx.x & 63) < T) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) part[threadIdx.x >> 6][t * VEC + i] = acc[i];
        }
        __syncthreads();
        if (threadIdx.x < T && fok) {
            float r[VEC];
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                float sum = part[0][t * VEC + i];
#pragma unroll
                for (int w = 1; w < kBlock / 64; ++w) sum += part[w][t * VEC + i];
                r[i] = sum;
            }
            if constexpr (PIECE) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) __hip_atomic_store(o + f + i, r[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                store_frag<VEC>(o + f, r);
            }
        }
        __syncthreads();  // `part` is written again
    }
}

// One chunk of a cut row.  The workgroup that is the last of the row's to be done adds the chunks' sums, in an order that depends on their
// number alone (a launch of its own for that took 4 to 5 us and the gap before it: an epoch of 88,784 vertices, F = 16 / 39, and what
// comes before it 177 -> 167 us, the backward loop of 1.1 M vertices, F = 16 / 41, 228.6 -> 223.1).
// Sums are written and read past the L2, of which every XCD has its own: relaxed atomics of agent scope, which this GPU's instructions do
// that with (sc1), and a wait for the writes to have arrived before they are counted.  The language orders relaxed atomics of different
// words by fences alone; a release here and an acquire by the last workgroup are the same order with the whole L2 written back and
// dropped (223.9 -> 231.3 us of that loop, the blog graph's import and first epoch 112.6 -> 122.8).  A test reads the instructions.
template <int VEC, int LOG2T, bool INNER>
__device__ __forceinline__ void sum_chunk(const RowArgs& a, float (*part)[(1 << LOG2T) * VEC], int* was) {
    const int b = (int)blockIdx.x;
    // classes from the longest rows' down, as many workgroups for each row of one as its longest row has chunks
    const int lane = threadIdx.x & 63, c = EPP_NCLASS - 1 - (lane & (EPP_NCLASS - 1));
    const int rows_of_class = a.long_head[c * kLongApart], place_of_class = a.long_head[c * kLongApart + 1];
    const int width = c > a.log2_chunk ? rows_of_class << (c - a.log2_chunk) : 0;
    int upto = width;
#pragma unroll
    for (int d = 1; d < EPP_NCLASS; d <<= 1) {
        const int below = __shfl_up(upto, d, EPP_NCLASS);
        if ((lane & (EPP_NCLASS - 1)) >= d) upto += below;
    }
    const int k = __ffsll((long long)__ballot(b < upto)) - 1;
    if (k < 0) return;
    const int log2 = EPP_NCLASS - 1 - k - a.log2_chunk, j = b - __builtin_amdgcn_readlane(upto - width, k), q = j & ((1 << log2) - 1);
    LongRow* const h = a.long_rows + __builtin_amdgcn_readlane(place_of_class, k) + (j >> log2);
    const int row_begin = h->begin, row_end = h->end, v = h->v;
    const int count = (row_end - row_begin + (1 << a.log2_chunk) - 1) >> a.log2_chunk;
    if (q >= count) return;
    const int begin = row_begin + (q << a.log2_chunk), end = min(begin + (1 << a.log2_chunk), row_end);
    const int slot = threadIdx.x >> LOG2T;
    constexpr int kSlots = kBlock >> LOG2T, kAhead = 4;
    sum_by_workgroup<VEC, LOG2T, true>(a, a.pieces + (size_t)b * a.F, part, [&](int f, float (&acc)[VEC]) {
        add_entries<VEC, LOG2T, kU, INNER, true>(a, a.in + f, begin + slot * kU, end, kSlots * kU, acc);
    });
    if (threadIdx.x < 64) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0) *was = (int)atomicInc(&h->done[a.user], (unsigned)count - 1u);  // (0 again behind the last one)
    }
    __syncthreads();
    if (*was != count - 1) return;
    if constexpr (INNER) {
        if (!((a.only[v >> 5] >> (v & 31)) & 1u)) return;
    }
    const float* __restrict__ pieces = a.pieces + (size_t)(b - q) * a.F;
    sum_by_workgroup<VEC, LOG2T, false>(a, a.out + (size_t)v * a.F, part, [&](int f, float (&acc)[VEC]) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = 0.0f;
        for (int p = slot; p < count; p += kAhead * kSlots) {
            float x[kAhead][VEC];
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int i = 0; i < VEC; ++i)
                    x[u][i] = __hip_atomic_load(pieces + (size_t)min(p + u * kSlots, count - 1) * a.F + f + i, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int i = 0; i < VEC; ++i)
                    if (p + u * kSlots < count) acc[i] += x[u][i];
        }
    });
}

template <int VEC, int LOG2T, bool INNER>
__global__ __launch_bounds__(kBlock, 7) void k_aggregate_rows(RowArgs a) {
    constexpr int T = 1 << LOG2T;
    __shared__ int list[kBlock];
    __shared__ int count;
    __shared__ float part[kBlock / 64][T * VEC];
    if ((int)blockIdx.x < a.chunk_blocks) {
        sum_chunk<VEC, LOG2T, INNER>(a, part, &count);
        return;
    }
    const int t = threadIdx.x & (T - 1), slot = threadIdx.x >> LOG2T;
    const int P = 1 << a.log2p, sub = slot & (P - 1);
    const int r = ((int)blockIdx.x - a.chunk_blocks) * (kBlock >> (LOG2T + a.log2p)) + (slot >> a.log2p);
    const bool has = r < a.n_rows;
    const int p0 = has ? a.rowptr[r] : 0, p1 = has ? a.rowptr[r + 1] : 0;
    const int v = has ? (a.row_ids ? a.row_ids[r] : r) : 0;
    const bool is_long = p1 - p0 > a.limit;
    bool write = has && !is_long && sub == 0;
    if constexpr (INNER) write = write && ((a.only[v >> 5] >> (v & 31)) & 1u);
    if (a.has_long) {
        if (threadIdx.x == 0) count = 0;
        __syncthreads();
        if (is_long && p1 - p0 <= (1 << a.log2_chunk) && t == 0 && sub == 0) list[atomicAdd(&count, 1)] = r;
    }
    bool bad = false;
    for (int f0 = 0; f0 < a.F; f0 += T * VEC) {
        const bool fok = f0 + t * VEC < a.F;
        const int f = fok ? min(f0 + t * VEC, a.F - VEC) : 0;
        float acc[VEC];
        add_entries<VEC, LOG2T, kU, INNER, false>(a, a.in + f, p0 + sub * kU, is_long ? p0 : p1, P * kU, acc);
        for (int d = T; d < T * P; d <<= 1) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], d, 64);
        }
        bad |= not_numbers<VEC>(acc);  // (the same in all slots of the row)
        if (write && fok) store_frag<VEC>(a.out + (size_t)v * a.F + f, acc);
    }
    if (__builtin_expect(bad, 0)) {
        // (a second look at everything, so that nothing of it is kept in registers through the loop above)
        unsigned thread = threadIdx.x;
        asm volatile("" : "+v"(thread));
        const int ot = thread & (T - 1), os = thread >> LOG2T, osub = os & (P - 1);
        const int orow = ((int)blockIdx.x - a.chunk_blocks) * (kBlock >> (LOG2T + a.log2p)) + (os >> a.log2p);
        const int begin = a.rowptr[orow], end = a.rowptr[orow + 1], ov = a.row_ids ? a.row_ids[orow] : orow;
        bool owrite = osub == 0;
        if constexpr (INNER) owrite = owrite && ((a.only[ov >> 5] >> (ov & 31)) & 1u);
        for (int f0 = 0; f0 < a.F; f0 += T * VEC) {
            const bool fok = f0 + ot * VEC < a.F;
            const int f = fok ? min(f0 + ot * VEC, a.F - VEC) : 0;
            float acc[VEC];
            add_own_entries<VEC, kU, INNER>(a, a.in + f, begin + osub * kU, end, P * kU, acc);
            for (int d = T; d < T * P; d <<= 1) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], d, 64);
            }
            if (owrite && fok) store_frag<VEC>(a.out + (size_t)ov * a.F + f, acc);
        }
    }
    if (!a.has_long) return;
    __syncthreads();
    const int n_long = count;
    for (int k = 0; k < n_long; ++k) {
        const int lr = list[k], q0 = a.rowptr[lr], q1 = a.rowptr[lr + 1];
        const int lv = a.row_ids ? a.row_ids[lr] : lr;
        if constexpr (INNER) {
            if (!((a.only[lv >> 5] >> (lv & 31)) & 1u)) continue;  // (uniform)
        }
        sum_by_workgroup<VEC, LOG2T, false>(a, a.out + (size_t)lv * a.F, part, [&](int f, float (&acc)[VEC]) {
            add_entries<VEC, LOG2T, kU, INNER, true>(a, a.in + f, q0 + slot * kU, q1, (kBlock >> LOG2T) * kU, acc);
        });
    }
}

__global__ __launch_bounds__(kBlock) void k_list_long_rows(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ row_ids,
                                                           int n_rows, LongRows list) {
    __shared__ int found[2 * EPP_NCLASS];
    const int r = blockIdx.x * kBlock + threadIdx.x;
    const int p0 = r < n_rows ? rowptr[r] : 0, p1 = r < n_rows ? rowptr[r + 1] : 0;
    list_long_rows(list, r < n_rows && row_ids ? row_ids[r] : r, p0, p1 - p0, found);
    if (blockIdx.x == 0) place_long_rows(list);
}

template <int VEC, int LOG2T>
void launch(const RowArgs& a, hipStream_t s) {
    const int per_block = kBlock >> (LOG2T + a.log2p);
    const dim3 grid((unsigned)(a.chunk_blocks + (a.n_rows + per_block - 1) / per_block));
    if (a.zero) hipLaunchKernelGGL((k_aggregate_rows<VEC, LOG2T, true>), grid, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_aggregate_rows<VEC, LOG2T, false>), grid, dim3(kBlock), 0, s, a);
}

}  // namespace

// Lanes per source row, and the entries of a chunk: eight steps of the workgroup.
static int lanes_log2(int F) {
    const int frags = (F + 3) / 4;
    int l = 0;
    while ((1 << l) < frags && l < 6) ++l;
    return l;
}
static int chunk_log2(int F) { return 13 - lanes_log2(F); }
static_assert((1 << 13) == 8 * kBlock * kU, "chunk length");

// Which paths run here.  Rows of 16 bytes and less always: the group kernel's lanes then each carry a
// group of their own and read pairs far apart (this kernel's time over the group kernel's at 20 / 90 / 200 to 230 M entries,
// 0.25 to 8 M sources, both models: F = 1 0.37 to 0.80, F = 2 0.38 to 0.85, F = 4 0.42 to 0.88, growing with the matrix and
// the entries; F = 3, whose groups have four lanes, 0.74 to 0.91 / 0.88 to 1.06 / 0.92 to 1.02).
// Rows of up to 64 bytes up to 10 (F <= 8) and 5 M entries, and where launches do not run on tiles (epp_tiles.hip) as far as the
// group kernel, which reads copies of 32 or 64 bytes instead, needs at least as long (over its time, 5 to 46 M entries, 0.02 to 6 M
// vertices, both models): 8 floats 0.50 to 0.95 everywhere; 5 to 7 up to 30 M entries 0.67 to 0.98, beyond to 1.13; 9 and 10 up to 20 M
// 0.76 to 1.03, beyond to 1.18; 11 to 13 up to 12 M 0.61 to 1.01, beyond to 1.30; 14 and 15 up to 8 M 0.79 to 1.03, beyond to 1.44; 16 up to
// 12 M 0.59 to 0.94.
// Rows of up to 256 bytes while the second kernel and the chain of loads still show: at 16 M floats of gathered rows in any
// case; up to 100 M, where the source matrix of 110 MB still stays in the memory-side cache, if the group kernel has to read
// rows across the ends of lines (F = 17 to 31: 0.63 to 1.10, at most 1.02 in nine of ten; above 32, if rows are no whole number of 16 bytes, 0.74
// to 1.20 and 0.93 on average; at 3 to 7 M vertices' rows of 140 MB and more 0.9 to 1.3); up to 64 M of 40 MB at F = 32 (0.60 to 0.91) and
// 48 M at F = 64 (0.73 to 0.94).  The group kernel's aligned loads are as fast or faster for other multiples of 4 (F = 36 to 60, 16 to
// 100 M: 0.73 to 1.53).
constexpr int64_t kMostNarrow = 48000000;   // entries: no path of more runs here at more than 4 floats a row, 8 floats having the most
constexpr int64_t kMostGathered = 100000000;  // floats of gathered rows, at more than 16 floats a row
bool epp_rows_kernel_fits(const epp_path* p, int F) {
    if (const char* e = std::getenv("EPP_TUNE_ROWS")) {  // 0: never, 2: always (tests, measurements)
        if (*e == '0') return false;
        if (*e == '2') return p->nnz <= (1 << 30);
    }
    if (epp_group_layout_asked()) return false;
    if (F <= 4) return p->nnz <= (1 << 30);
    if (F <= 16 && p->nnz <= (F <= 8 ? 10000000 : 5000000)) return true;
    if (F > 16 && p->nnz * F <= 16000000) return true;
    if (epp_group_table_asked()) return false;
    double any_delay;
    if (F <= 16) {
        const int64_t most = F <= 7 ? 30000000 : F == 8 ? kMostNarrow : F <= 10 ? 20000000 : F <= 13 || F == 16 ? 12000000 : 8000000;
        return p->nnz <= most && epp_tile_lanes(p, F, &any_delay) == 0;
    }
    if (F > 64) return false;
    if (F == 32 || F == 64) return p->nnz * F <= (F == 32 ? 64000000 : 48000000) && p->n_src * F <= 10000000;
    return (F < 32 || F % 4 != 0) && p->nnz * F <= kMostGathered && p->n_src * F <= 28000000;
}

// The path's own list takes no launch of its own.  It goes down to the shortest chunks that launches on this many entries have, those
// of the widest rows that the rule above lets run here, since a place for every row that there could be is 32 bytes for every
// 2^(log2 - 1) entries; but not below 2^9: wider rows than 64 floats run here on up to 250,000 entries only, and list for themselves.  Import and first epoch of
// the blog graph (4.2 M entries, F = 16 / 39): 153.5 us with the rows listed width by width, 120.2 with the path's own list.
size_t epp_plan_long_rows(int64_t nnz, LongRows* l) {
    *l = LongRows{};
    if (nnz > kMostNarrow) return 0;
    int widest = 16;  // (in steps that change the chunks: one more lane a row)
    while (widest < 64 && nnz * (widest + 1) <= kMostGathered) widest *= 2;
    l->log2 = chunk_log2(widest);
    l->nnz = (int)nnz;
    return (size_t)l->first_place(EPP_NCLASS) * sizeof(LongRow);
}

int epp_build_rows_plan(epp_path* p, int F, hipStream_t s, RowsPlan** out) {
    *out = nullptr;
    // rows of 2^(c-1) < length <= 2^c are counted in class c
    const int c0 = chunk_log2(F);
    int64_t n_chunks = 0;
    for (int c = c0 + 1; c < EPP_NCLASS; ++c) n_chunks += p->len_hist[c] << (c - c0);
    if (n_chunks == 0) return EPP_OK;
    RowsPlan* q = new RowsPlan();
    struct Guard { RowsPlan* q; ~Guard() { delete q; } } guard{q};
    LongRows list = p->long_rows;
    size_t at = 0;
    // (up to kLongUsers widths of a path take its list; the others each make one of their own)
    while (q->user < kLongUsers && ((p->long_rows_taken >> q->user) & 1u)) ++q->user;
    const bool listed = list.rows && list.log2 <= c0 && q->user < kLongUsers;
    if (!listed) q->user = 0;
    if (!listed) {
        list.log2 = c0;
        list.nnz = (int)p->nnz;
        at = kLongHeadBytes + DevArena::rounded((size_t)list.first_place(EPP_NCLASS) * sizeof(LongRow));
    }
    EPP_TRY(q->store.alloc(at + (size_t)n_chunks * F * 4, epp_alloc_of(p)));
    if (!listed) {
        list.head = q->store.as<int>();
        list.rows = reinterpret_cast<LongRow*>(q->store.as<char>() + kLongHeadBytes);
        EPP_HIP_TRY(hipMemsetAsync(list.head, 0, kLongHeadBytes, s));
        hipLaunchKernelGGL(k_list_long_rows, dim3((unsigned)((p->n_stream_rows + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                           p->rowptr.as<int32_t>(), p->row_ids.p ? p->row_ids.as<int32_t>() : nullptr, (int)p->n_stream_rows, list);
        EPP_HIP_TRY(hipGetLastError());
    }
    // (also where nothing was launched: launches may run on another stream than the one whose work the block of memory was last used by)
    EPP_HIP_TRY(hipStreamSynchronize(s));
    q->rows = list.rows;
    q->head = list.head;
    q->pieces = reinterpret_cast<float*>(q->store.as<char>() + at);
    if (listed) {
        q->taken = &p->long_rows_taken;
        p->long_rows_taken |= 1u << q->user;
    }
    q->n_chunks = (int)n_chunks;  // (an upper bound: a workgroup whose chunk its row does not have ends at once)
    guard.q = nullptr;
    *out = q;
    return EPP_OK;
}

int epp_launch_rows(const epp_path* p, const RowsPlan* plan, const float* in, float* out, int F, hipStream_t s,
                    const unsigned int* inner_rows) {
    if (p->n_stream_rows == 0) return EPP_OK;
    RowArgs a;
    a.cv = reinterpret_cast<const int2v*>(p->cv.p);
    a.rowptr = p->rowptr.as<int32_t>();
    a.row_ids = p->row_ids.p ? p->row_ids.as<int32_t>() : nullptr;
    a.n_rows = (int)p->n_stream_rows;
    a.user = plan ? plan->user : 0;
    a.in = in;
    a.out = out;
    a.F = F;
    a.zero = inner_rows ? p->zero_block.as<float>() : nullptr;
    a.only = inner_rows;
    const int log2t = lanes_log2(F);
    // as many slots per row as its entries keep busy on average, but no more wavefronts than a few rounds
    // of the chip, more of them the less each gathers (a round costs the whole chain of loads; F = 64,
    // 1.5 M entries: 62 us against 90 us with a wavefront per row, where one slot's chain would not be longer)
    const double per_row = (double)p->nnz / (double)p->n_stream_rows;
    int log2p = 0;
    while (log2p + log2t < 6 && (double)(kU << log2p) < per_row) ++log2p;
    while (log2p > 0 && (p->n_stream_rows << (log2t + log2p)) >> 6 > (262144 >> log2t)) --log2p;
    a.log2p = log2p;
    a.log2_chunk = chunk_log2(F);
    a.limit = std::min((8 * kU) << log2p, 1 << a.log2_chunk);
    a.has_long = p->max_len > a.limit;
    a.chunk_blocks = plan ? plan->n_chunks : 0;
    a.long_rows = plan ? plan->rows : nullptr;
    a.long_head = plan ? plan->head : nullptr;
    a.pieces = plan ? plan->pieces : nullptr;
    if (F >= 4) {
        switch (log2t) {
            case 0: launch<4, 0>(a, s); break;
            case 1: launch<4, 1>(a, s); break;
            case 2: launch<4, 2>(a, s); break;
            case 3: launch<4, 3>(a, s); break;
            case 4: launch<4, 4>(a, s); break;
            case 5: launch<4, 5>(a, s); break;
            default: launch<4, 6>(a, s); break;
        }
    } else if (F == 3) {
        launch<3, 0>(a, s);
    } else if (F == 2) {
        launch<2, 0>(a, s);
    } else {
        launch<1, 0>(a, s);
    }
    EPP_HIP_TRY(hipGetLastError());
    return EPP_OK;
}
