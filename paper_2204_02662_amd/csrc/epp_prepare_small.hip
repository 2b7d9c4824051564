// Execution path preparing (Sec. 4) for small graphs in ONE kernel launch.
//
// On a graph of a few thousand vertices the general construction (epp_prepare.hip) is all
// overhead: about fifteen launches, a host wait and an allocation per level, against microseconds
// of work.  Preparing on the fly (Sec. 6: the paths are built inside the first epoch) only pays if
// the construction costs a few epochs' worth of savings, and on such graphs an epoch saves
// microseconds.  Here one workgroup of 1024 threads builds every level with the frontier
// bitmaps, the keep-mask of the entries and their prefix counts in LDS; the host makes one
// allocation before (worst-case sizes: the whole handle is a megabyte or two), one launch, and one
// wait after, for the sizes.  Same results as the general construction, bit for bit (tested).
//
// Limits: n, |V_t| <= 65,536 and nnz <= 131,072 (one LDS word per 64 vertices and thread, two per
// 64 entries and thread), L <= 32; of these, the graphs on which it is the faster of the two.

#include <algorithm>
#include <cstring>

#include "epp_internal.h"

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxItems = 65536;           // vertices
constexpr int kWords = kMaxItems / 64;     // = kThreads: one bitmap word per thread
constexpr int kMaxEntries = 2 * kMaxItems;
constexpr int kEntryWords = kMaxEntries / 64;  // = 2 * kThreads: two keep-mask words per thread
constexpr int kStatWords = EPP_NCLASS + 1; // histogram + longest row
constexpr int kLevelWords = 3 + kStatWords; // kept entries, rows, "set did not change", statistics
constexpr int kRowEnd = kEntRowEnd;
constexpr int kBatch = 8;                  // independent loads in flight per lane in the streaming loops
constexpr int kMaskBatch = 16;             // ... of the keep-mask pass (one register per load)

__device__ __forceinline__ unsigned long long low_mask(int lane) { return (1ull << lane) - 1ull; }
__device__ __forceinline__ int length_class(int len) { return len <= 1 ? 0 : 32 - __clz(len - 1); }

// Position of the k-th (0-based) set bit of m (m has more than k set bits).
__device__ __forceinline__ int select_bit(unsigned long long m, int k) {
    int pos = 0;
#pragma unroll
    for (int half = 32; half >= 1; half >>= 1) {
        const int c = __popcll(m & ((1ull << half) - 1ull));
        if (k >= c) { k -= c; m >>= half; pos += half; }
    }
    return pos;
}

// Largest w in [0, count) with pre[w] <= j (pre is non-decreasing, pre[0] == 0 <= j).
__device__ __forceinline__ int last_not_above(const int* pre, int count, int j) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= j) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Exclusive scan of one value per thread over the workgroup; *total = sum.  (Two barriers.)
__device__ __forceinline__ int block_scan(int x, int* wave_sum /* LDS, kWaves + 1 */, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    __syncthreads();  // wave_sum may still be read from the scan before
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int s = wave_sum[w];
        if (w < wave) base += s;
        all += s;
    }
    *total = all;
    return base + incl - x;
}

// Is it cheaper to look `items` items up one by one than to walk `words` words of which they are the bits?
__device__ __forceinline__ bool by_item(int items, int words) {
    return (items + kThreads - 1) / kThreads * 130 < (words + kWaves - 1) / kWaves * 25;
}

struct SmallArgs {
    int n, nnz, n_train, L;
    int cv_stride, ids_stride, ptr_stride, bm_stride;  // per-level strides of the output arrays, in elements
    const int32_t* rowptr;
    const int32_t* col;
    const float* val;
    const int32_t* train_ids;
    unsigned long long* bitmaps;  // (L + 1) x n_words
    int32_t* set0_ids;            // n
    int2* cv;                     // L x nnz
    int32_t* row_ids;             // L x n
    int32_t* out_rowptr;          // L x (n + 1)
    long long* result;            // pinned host words: [0] error bits, [1] |N^0|, then kLevelWords per level
    PinnedWords::Signal signal;   // .. that they, and everything else, are written
};

// HELD: for graphs of at most kHeldItems vertices and kHeldEntries entries.
template <bool HELD>
__global__ void k_prepare_small(SmallArgs a);

// Everything that the workgroup has written is there, for the host and for kernels on any stream.
__device__ __forceinline__ void all_written(const SmallArgs& a) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (every wavefront's stores are in this XCD's L2)
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence_system();
        epp_raise(a.signal);
    }
}

template <>
__global__ __launch_bounds__(kThreads) void k_prepare_small<false>(SmallArgs a) {
    __shared__ unsigned long long bm_cur[kWords + 1], bm_next[kWords], keep[kEntryWords];
    __shared__ unsigned int ends[2 * kEntryWords];  // one bit per kept entry: the last of its row
    __shared__ int wpre[kEntryWords], rpre[kWords];
    __shared__ int wave_sum[kWaves + 1];
    __shared__ int hist[EPP_NCLASS];
    __shared__ int s_max, s_err, s_differs;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_words = (a.n + 63) >> 6, n_seg = (a.nnz + 63) >> 6;

    bm_cur[tid] = 0ull;
    if (tid == 0) {
        bm_cur[kWords] = 0ull;  // what an id that is no vertex looks up
        s_err = 0;
    }
    __syncthreads();
    // N^0 = V_t (Property 1); the row pointer must rise from 0 to nnz
    // (the column ids are range-checked where the first level loads them)
    {
        for (int i0 = tid; i0 < a.n_train; i0 += kThreads * kBatch) {
            int v[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) v[i] = i0 + i * kThreads < a.n_train ? a.train_ids[i0 + i * kThreads] : 0;
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                if (i0 + i * kThreads >= a.n_train) continue;
                if (v[i] < 0 || v[i] >= a.n) atomicOr(&s_err, 2);
                else atomicOr(&bm_cur[v[i] >> 6], 1ull << (v[i] & 63));
            }
        }
    }
    for (int v0 = tid; v0 < a.n; v0 += kThreads * kBatch) {
        int p0[kBatch], p1[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int v = v0 + i * kThreads;
            p0[i] = v < a.n ? a.rowptr[v] : 0;
            p1[i] = v < a.n ? a.rowptr[v + 1] : 0;
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int v = v0 + i * kThreads;
            if (v < a.n && (p0[i] < 0 || p1[i] < p0[i] || p1[i] > a.nnz || (v == 0 && p0[i] != 0) || (v == a.n - 1 && p1[i] != a.nnz)))
                atomicOr(&s_err, 1);
        }
    }
    __syncthreads();
    if (s_err) {  // uniform: nothing is indexed with unchecked values
        if (tid == 0) a.result[0] = s_err;
        all_written(a);
        return;
    }
    {   // ascending ids of N^0
        int total;
        const unsigned long long m = bm_cur[tid];
        const int base = block_scan(__popcll(m), wave_sum, &total);
        wpre[tid] = base;
        __syncthreads();
        for (int w = wave; w < n_words; w += kWaves) {
            const unsigned long long mm = bm_cur[w];
            if ((mm >> lane) & 1ull) a.set0_ids[wpre[w] + __popcll(mm & low_mask(lane))] = w * 64 + lane;
        }
        if (tid < n_words) a.bitmaps[tid] = m;
        if (tid == 0) {
            a.result[0] = 0;
            a.result[1] = total;
        }
    }

    for (int k = 0; k < a.L; ++k) {
        int2* __restrict__ cv = a.cv + (size_t)k * a.cv_stride;
        int32_t* __restrict__ row_ids = a.row_ids + (size_t)k * a.ids_stride;
        int32_t* __restrict__ orp = a.out_rowptr + (size_t)k * a.ptr_stride;
        __syncthreads();
        bm_next[tid] = 0ull;
        for (int i = tid; i < 2 * n_seg; i += kThreads) ends[i] = 0u;
        if (tid < EPP_NCLASS) hist[tid] = 0;
        if (tid == 0) { s_max = 0; s_differs = 0; }
        // keep-mask of the entries: is the column in N^k?  (kMaskBatch words per step and wavefront:
        // the column loads of a step are issued together, their latency is paid once.)  An id
        // outside [0, n) finds a zero; the first level reports it.
        unsigned int top = 0;
        const unsigned int* bm32 = reinterpret_cast<const unsigned int*>(bm_cur);  // (4-byte lookups: half the bank conflicts)
        for (int w0 = wave * kMaskBatch; w0 < n_seg; w0 += kWaves * kMaskBatch) {
            int c[kMaskBatch];
            if ((w0 + kMaskBatch) * 64 <= a.nnz) {
#pragma unroll
                for (int i = 0; i < kMaskBatch; ++i) c[i] = a.col[(w0 + i) * 64 + lane];
                if (k == 0) {
#pragma unroll
                    for (int i = 0; i < kMaskBatch; ++i) top = max(top, (unsigned int)c[i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < kMaskBatch; ++i) {
                    const int e = (w0 + i) * 64 + lane;
                    c[i] = kMaxItems;
                    if (e < a.nnz) {
                        c[i] = a.col[e];
                        if (k == 0) top = max(top, (unsigned int)c[i]);
                    }
                }
            }
            unsigned long long out = 0ull;
#pragma unroll
            for (int i = 0; i < kMaskBatch; ++i) {
                const unsigned int x = min((unsigned int)c[i], (unsigned int)kMaxItems);
                const unsigned long long m = __ballot((bm32[x >> 5] >> (x & 31)) & 1u);
                if (lane == i) out = m;
            }
            if (lane < kMaskBatch && w0 + lane < n_seg) keep[w0 + lane] = out;
        }
        const bool bad = top >= (unsigned int)a.n;
        if (k == 0 && bad) atomicOr(&s_err, 4);
        __syncthreads();
        if (k == 0 && s_err) {  // uniform
            if (tid == 0) a.result[0] = s_err;
            all_written(a);
            return;
        }
        int kept;
        {   // prefix counts of the keep-mask words: two consecutive words per thread
            const int c0 = 2 * tid < n_seg ? __popcll(keep[2 * tid]) : 0;
            const int c1 = 2 * tid + 1 < n_seg ? __popcll(keep[2 * tid + 1]) : 0;
            const int wbase = block_scan(c0 + c1, wave_sum, &kept);
            wpre[2 * tid] = wbase;
            wpre[2 * tid + 1] = wbase + c0;
        }
        __syncthreads();
        auto kept_before = [&](int p) -> int {
            return p >= a.nnz ? kept : wpre[p >> 6] + __popcll(keep[p >> 6] & low_mask(p & 63));
        };
        // filtered list of every vertex; a vertex whose list is not empty is in N^{k+1}
        // (the 64 lanes of a wavefront hold the 64 vertices of one bitmap word: one ballot per word)
        int longest = 0;
        auto count_row = [&](int v, int ra, int rb) {
            const bool member = v < a.n && rb > ra;
            const unsigned long long word = __ballot(member);
            if (lane == 0 && (v >> 6) < n_words) bm_next[v >> 6] = word;
            if (member) {
                const int len = rb - ra;
                atomicOr(&ends[(rb - 1) >> 5], 1u << ((rb - 1) & 31));
                atomicAdd(&hist[length_class(len)], 1);
                longest = max(longest, len);
            }
        };
        for (int v0 = tid; v0 - lane < a.n; v0 += kThreads * kBatch) {
            int p0[kBatch], p1[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const int v = v0 + i * kThreads;
                p0[i] = v < a.n ? a.rowptr[v] : a.nnz;
                p1[i] = v < a.n ? a.rowptr[v + 1] : a.nnz;
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                if (v0 - lane + i * kThreads >= a.n) break;  // (uniform)
                count_row(v0 + i * kThreads, kept_before(p0[i]), kept_before(p1[i]));
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) longest = max(longest, __shfl_xor(longest, d, 64));
        if (lane == 0 && longest > 0) atomicMax(&s_max, longest);
        __syncthreads();  // bm_next and the row ends are complete
        // Stable compaction of (col, val), word by word: a kept entry's place is its word's prefix count plus
        // the kept ones before it in the word.  Where little is kept, entry by entry instead: slot j
        // of the path belongs to the word whose prefix count is the last one not above j, and is that
        // word's (j - prefix)-th set bit (some 130 instructions per entry and thread, against 14
        // per word and wavefront, whose number this one workgroup is bound by).
        if (by_item(kept, n_seg)) {
            for (int j = tid; j < kept; j += kThreads) {
                const int w = last_not_above(wpre, n_seg, j), e = w * 64 + select_bit(keep[w], j - wpre[w]);
                const int flag = (ends[j >> 5] >> (j & 31)) & 1u ? kRowEnd : 0;
                cv[j] = make_int2(a.col[e] | flag, __float_as_int(a.val[e]));
            }
        } else {
            for (int w0 = wave; w0 < n_seg; w0 += kWaves * kBatch) {
                unsigned long long m[kBatch];
                int2 x[kBatch];
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    const int w = w0 + i * kWaves;
                    m[i] = w < n_seg ? keep[w] : 0ull;
                    if ((m[i] >> lane) & 1ull) x[i] = make_int2(a.col[w * 64 + lane], __float_as_int(a.val[w * 64 + lane]));
                }
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    if (!((m[i] >> lane) & 1ull)) continue;
                    const int j = wpre[w0 + i * kWaves] + __popcll(m[i] & low_mask(lane));
                    if ((ends[j >> 5] >> (j & 31)) & 1u) x[i].x |= kRowEnd;
                    cv[j] = x[i];
                }
            }
        }
        int R;
        const int rbase = block_scan(tid < n_words ? __popcll(bm_next[tid]) : 0, wave_sum, &R);
        rpre[tid] = rbase;
        if (tid < n_words && bm_next[tid] != bm_cur[tid]) s_differs = 1;
        __syncthreads();
        // rows of the path (in the same two ways)
        auto put_row = [&](int r, int v) {
            row_ids[r] = v;
            orp[r] = kept_before(a.rowptr[v]);
        };
        if (by_item(R, n_words)) {
            for (int r = tid; r < R; r += kThreads) {
                const int w = last_not_above(rpre, n_words, r);
                put_row(r, w * 64 + select_bit(bm_next[w], r - rpre[w]));
            }
        } else {
            for (int w = wave; w < n_words; w += kWaves) {
                const unsigned long long m = bm_next[w];
                if ((m >> lane) & 1ull) put_row(rpre[w] + __popcll(m & low_mask(lane)), w * 64 + lane);
            }
        }
        long long* res = a.result + 2 + (size_t)k * kLevelWords;
        if (tid == 0) {
            orp[R] = kept;
            res[0] = kept;
            res[1] = R;
            res[2] = s_differs ? 0 : 1;
            res[3 + EPP_NCLASS] = s_max;
        }
        if (tid < EPP_NCLASS) res[3 + tid] = hist[tid];
        if (tid < n_words) a.bitmaps[(size_t)(k + 1) * a.bm_stride + tid] = bm_next[tid];
        __syncthreads();
        bm_cur[tid] = bm_next[tid];
    }
    all_written(a);
}

// The same for graphs whose columns, weights and row pointer fit the registers: thread t of wavefront w holds entry t % 64 of the words
// w, w + 16, .. of the entries, and the vertices t, t + 1024, .., which is where the keep-mask, the compaction and the rows want
// them.  Every wavefront adds up the words' counts for itself, and what a level writes has two buffers, so that a level takes two
// barriers.  Bound by the latency of what one level's LDS accesses and barriers wait for.
//
// A citation graph of 2,708 vertices and 13,200 entries, two levels: 26.4 us with columns and row pointer in LDS, twelve barriers a level
// and the weights read per level, 14.5 us like this (prepared and one epoch 59.5 -> 47.7).  With twice the registers, for 8,192 vertices
// and 32,768 entries, they no longer fit and it is the slower one (4,000 vertices, 28,000 entries 106 -> 110 us).
constexpr int kHeldItems = 4096, kHeldEntries = 16384;
constexpr int kHistCopies = 16;  // (64 lanes on a few counters would wait for each other)

// Sum over the lanes up to this one; largest of all lanes, in lane 63 (data moves between lanes without LDS).
template <class F>
__device__ __forceinline__ int over_lanes(int x, F f) {
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false));  // row_shr:1
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false));  // row_shr:2
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false));  // row_shr:4
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false));  // row_shr:8
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false));  // row_bcast:15
    x = f(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return x;
}
__device__ __forceinline__ int sum_up_to_lane(int x) { return over_lanes(x, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ int largest_of_lanes(int x) { return over_lanes(x, [](int a, int b) { return max(a, b); }); }  // (none is negative)

// Bits before the words of N = 64 PER: lane l has those before the words PER l + wave % PER, of which a wavefront's words w, w + 16, ..
// are some (word_at); all[word], if given, becomes those before every word.
template <int PER>
__device__ __forceinline__ int bits_before(const unsigned long long* words, int wave, int& mine, int* all) {
    const int lane = threadIdx.x & 63;
    int c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] = sum;
        sum += __popcll(words[PER * lane + q]);
    }
    const int incl = sum_up_to_lane(sum);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] += incl - sum;
        if (all) all[PER * lane + q] = c[q];
        if (wave % PER == q) mine = c[q];
    }
    return __builtin_amdgcn_readlane(incl, 63);
}
template <int PER>
__device__ __forceinline__ int word_at(int mine, int wave, int i) { return __builtin_amdgcn_readlane(mine, wave / PER + kWaves / PER * i); }
// Set bits of m below this lane.
__device__ __forceinline__ int bits_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

template <>
__global__ __launch_bounds__(kThreads) void k_prepare_small<true>(SmallArgs a) {
    constexpr int COLS = kHeldEntries / kThreads, ROWS = kHeldItems / kThreads;  // words of entries and of vertices per wavefront
    constexpr int kSegs = COLS * kWaves, kRowWords = ROWS * kWaves;
    constexpr int kPerSeg = kSegs / 64, kPerRow = kRowWords / 64;
    static_assert(kSegs % 64 == 0 && kRowWords % 64 == 0 && kWaves % kPerSeg == 0 && COLS <= 32, "");
    __shared__ unsigned long long bm[2][kRowWords + 1];  // N^k and N^{k+1}, in turns; the last word stays empty
    __shared__ unsigned long long keep[kSegs];
    __shared__ unsigned int ends[2][2 * kSegs];  // one bit per kept entry: the last of its row
    __shared__ int before[kSegs];                // kept entries before every word (each wavefront writes, and reads, all of them)
    __shared__ int hist[2][kHistCopies][EPP_NCLASS + 1];
    __shared__ int s_max[2], s_err;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_words = (a.n + 63) >> 6;

    int c[COLS], p0[ROWS], p1[ROWS];
    float val[COLS];
#pragma unroll
    for (int i = 0; i < COLS; ++i) c[i] = tid + i * kThreads < a.nnz ? a.col[tid + i * kThreads] : kRowWords * 64;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const int v = tid + j * kThreads;
        p0[j] = v < a.n ? a.rowptr[v] : a.nnz;
        p1[j] = v < a.n ? a.rowptr[v + 1] : a.nnz;
    }
    for (int i = tid; i < 2 * (kRowWords + 1); i += kThreads) (&bm[0][0])[i] = 0ull;
    for (int i = tid; i < 2 * 2 * kSegs; i += kThreads) (&ends[0][0])[i] = 0u;
    for (int i = tid; i < 2 * kHistCopies * (EPP_NCLASS + 1); i += kThreads) (&hist[0][0][0])[i] = 0;
    if (tid < 2) s_max[tid] = 0;
    if (tid == 0) s_err = 0;
    __syncthreads();
    // N^0 = V_t (Property 1); the row pointer must rise from 0 to nnz
    for (int i0 = tid; i0 < a.n_train; i0 += kThreads * kBatch) {
        int v[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) v[i] = i0 + i * kThreads < a.n_train ? a.train_ids[i0 + i * kThreads] : 0;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (i0 + i * kThreads >= a.n_train) continue;
            if (v[i] < 0 || v[i] >= a.n) atomicOr(&s_err, 2);
            else atomicOr(&bm[0][v[i] >> 6], 1ull << (v[i] & 63));
        }
    }
    int t = tid;
    asm volatile("" : "+v"(t));  // (a register pair for each of the comparisons, kept from above, does not fit)
#pragma unroll
    for (int i = 0; i < COLS; ++i) val[i] = t + i * kThreads < a.nnz ? a.val[t + i * kThreads] : 0.0f;
    int wrong = 0;
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int i = 0; i < COLS; ++i) wrong |= t + i * kThreads < a.nnz && (unsigned)c[i] >= (unsigned)a.n ? 4 : 0;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const int v = tid + j * kThreads;
        if (v < a.n && (p0[j] < 0 || p1[j] < p0[j] || p1[j] > a.nnz || (v == 0 && p0[j] != 0) || (v == a.n - 1 && p1[j] != a.nnz)))
            wrong |= 1;
    }
    if (wrong) atomicOr(&s_err, wrong);
    __syncthreads();
    if (s_err) {  // uniform: nothing is indexed with unchecked values
        if (tid == 0) a.result[0] = s_err;
        all_written(a);
        return;
    }
    {   // ascending ids of N^0
        int base;
        const int total = bits_before<kPerRow>(bm[0], wave, base, nullptr);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const unsigned long long m = bm[0][wave + j * kWaves];
            const int at = word_at<kPerRow>(base, wave, j) + bits_below(m);
            if ((m >> lane) & 1ull) a.set0_ids[at] = tid + j * kThreads;
        }
        if (tid < n_words) a.bitmaps[tid] = bm[0][tid];
        if (tid == 0) {
            a.result[0] = 0;
            a.result[1] = total;
        }
    }

    for (int k = 0; k < a.L; ++k) {
        int2* __restrict__ cv = a.cv + (size_t)k * a.cv_stride;
        int32_t* __restrict__ row_ids = a.row_ids + (size_t)k * a.ids_stride;
        int32_t* __restrict__ orp = a.out_rowptr + (size_t)k * a.ptr_stride;
        const int now = k & 1;
        // (what follows from them is not kept in registers from level to level)
#pragma unroll
        for (int i = 0; i < COLS; ++i) asm volatile("" : "+v"(c[i]));
#pragma unroll
        for (int j = 0; j < ROWS; ++j) asm volatile("" : "+v"(p0[j]), "+v"(p1[j]));
        // keep-mask of the entries: is the column in N^k?
        const unsigned int* bm32 = reinterpret_cast<const unsigned int*>(bm[now]);  // (4-byte lookups: half the bank conflicts)
        unsigned mine = 0u;  // bit i: the thread's i-th entry is kept
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
            const unsigned in = (bm32[c[i] >> 5] >> (c[i] & 31)) & 1u;
            mine |= in << i;
            const unsigned long long m = __ballot(in);
            if (lane == 0) keep[wave + i * kWaves] = m;
        }
        __syncthreads();
        int word_base;
        const int kept = bits_before<kPerSeg>(keep, wave, word_base, before);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        auto kept_before = [&](int p) -> int {
            return p >= a.nnz ? kept : before[p >> 6] + __popcll(keep[p >> 6] & low_mask(p & 63));
        };
        // filtered list of every vertex; a vertex whose list is not empty is in N^{k+1}
        int begin[ROWS], longest = 0;
        unsigned member = 0u;  // bit j: the thread's j-th vertex is in N^{k+1}
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            begin[j] = kept_before(p0[j]);
            const int end = kept_before(p1[j]), len = end - begin[j];
            const unsigned long long m = __ballot(len > 0);
            if (lane == 0) bm[now ^ 1][wave + j * kWaves] = m;
            if (len > 0) {
                member |= 1u << j;
                atomicOr(&ends[now][(end - 1) >> 5], 1u << ((end - 1) & 31));
                atomicAdd(&hist[now][lane & (kHistCopies - 1)][length_class(len)], 1);
                longest = max(longest, len);
            }
        }
        longest = largest_of_lanes(longest);
        if (lane == 63 && longest > 0) atomicMax(&s_max[now], longest);
        __syncthreads();
        // stable compaction of (col, val): a kept entry's place is its word's count plus the kept ones before it in the word
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
            const bool in = (mine >> i) & 1u;
            const int j = word_at<kPerSeg>(word_base, wave, i) + bits_below(__ballot(in));
            if (in) cv[j] = make_int2(c[i] | ((ends[now][j >> 5] >> (j & 31)) & 1u ? kRowEnd : 0), __float_as_int(val[i]));
        }
        // rows of the path
        int row_base;
        const int R = bits_before<kPerRow>(bm[now ^ 1], wave, row_base, nullptr);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const bool in = (member >> j) & 1u;
            const int r = word_at<kPerRow>(row_base, wave, j) + bits_below(__ballot(in));
            if (in) {
                row_ids[r] = tid + j * kThreads;
                orp[r] = begin[j];
            }
        }
        bool differs = false;
#pragma unroll
        for (int w = 0; w < kRowWords; w += 64) differs |= bm[0][w + lane] != bm[1][w + lane];
        differs = __ballot(differs) != 0ull;
        long long* res = a.result + 2 + (size_t)k * kLevelWords;
        if (tid == 0) {
            orp[R] = kept;
            res[0] = kept;
            res[1] = R;
            res[2] = differs ? 0 : 1;
            res[3 + EPP_NCLASS] = s_max[now];
        }
        if (tid < EPP_NCLASS) {
            int sum = 0;
#pragma unroll
            for (int i = 0; i < kHistCopies; ++i) sum += hist[now][i][tid];
            res[3 + tid] = sum;
        }
        if (tid < n_words) a.bitmaps[(size_t)(k + 1) * a.bm_stride + tid] = bm[now ^ 1][tid];
        // for the next level (nobody reads these any more: all have been at the barrier behind this level's keep-mask)
        for (int i = tid; i < 2 * kSegs; i += kThreads) ends[now ^ 1][i] = 0u;
        for (int i = tid; i < kHistCopies * (EPP_NCLASS + 1); i += kThreads) (&hist[now ^ 1][0][0])[i] = 0;
        if (tid == 0) s_max[now ^ 1] = 0;
    }
    all_written(a);
}

}  // namespace

bool epp_prepare_small_fits(const epp_csr_t* g, int64_t n_train, int L) {
    // (one workgroup's time grows with the graph, the general construction's hardly does below a million
    // entries: 83 to 103 us against 124 at 10,000 vertices and 64,000 entries, 103 to 131 against 122 at
    // 10,000 and 117,000, 121 to 155 against 123 at 20,000 and 117,000, two levels each)
    return g->n <= kMaxItems && g->nnz <= kMaxEntries && g->nnz + 3 * g->n <= 140000 && n_train <= kMaxItems && L <= 32 &&
           g->n > 0;
}

int epp_prepare_small(const epp_csr_t* g, const int32_t* train_ids, int64_t n_train, int L, const epp_alloc_t* alloc,
                      hipStream_t s, epp_paths_t** out) {
    const int64_t n = g->n, nnz = g->nnz, n_words = (n + 63) / 64;
    epp_paths* P = new epp_paths();
    struct Guard { epp_paths* p; ~Guard() { delete p; } } guard{P};
    P->L = L;
    P->n = n;
    if (alloc && alloc->alloc && alloc->free) P->alloc = *alloc;
    const epp_alloc_t* al = epp_alloc_of(P);
    P->bitmaps.resize(L + 1);
    P->set_size.assign(L + 1, 0);
    P->path.assign(L, nullptr);

    // one allocation for the whole handle (worst-case sizes), carved into 256-byte aligned pieces
    const size_t result_words = 2 + (size_t)L * kLevelWords;
    const size_t bm_bytes = (size_t)n_words * 8, cv_bytes = (size_t)std::max<int64_t>(nnz, 1) * 8,
                 ids_bytes = (size_t)n * 4, ptr_bytes = (size_t)(n + 1) * 4;
    DevArena arena;
    EPP_TRY(arena.reserve((size_t)(L + 1) * DevArena::rounded(bm_bytes) + DevArena::rounded(ids_bytes) +
                          (size_t)L * (DevArena::rounded(cv_bytes) + DevArena::rounded(ids_bytes) + DevArena::rounded(ptr_bytes)), al));
    // (every level's arrays start 256-byte aligned: the strides are the rounded sizes)
    DevBuf bm_all, set0, cv_all, ids_all, ptr_all;
    arena.take(&bm_all, (size_t)(L + 1) * DevArena::rounded(bm_bytes));
    arena.take(&set0, ids_bytes);
    arena.take(&cv_all, (size_t)L * DevArena::rounded(cv_bytes));
    arena.take(&ids_all, (size_t)L * DevArena::rounded(ids_bytes));
    arena.take(&ptr_all, (size_t)L * DevArena::rounded(ptr_bytes));
    PinnedWords pinned;
    EPP_TRY(pinned.get(result_words));
    long long* host = pinned.p;

    SmallArgs a;
    a.n = (int)n;
    a.nnz = (int)nnz;
    a.n_train = (int)n_train;
    a.L = L;
    a.cv_stride = (int)(DevArena::rounded(cv_bytes) / 8);
    a.ids_stride = (int)(DevArena::rounded(ids_bytes) / 4);
    a.ptr_stride = (int)(DevArena::rounded(ptr_bytes) / 4);
    a.bm_stride = (int)(DevArena::rounded(bm_bytes) / 8);
    a.rowptr = g->rowptr;
    a.col = g->col;
    a.val = g->val;
    a.train_ids = train_ids;
    a.bitmaps = bm_all.as<unsigned long long>();
    a.set0_ids = set0.as<int32_t>();
    a.cv = cv_all.as<int2>();
    a.row_ids = ids_all.as<int32_t>();
    a.out_rowptr = ptr_all.as<int32_t>();
    a.signal = pinned.signal();
    a.result = host;  // (the kernel writes a few dozen words there itself: a copy would be a launch of its own)
    if (n <= kHeldItems && nnz <= kHeldEntries) hipLaunchKernelGGL(k_prepare_small<true>, dim3(1), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL(k_prepare_small<false>, dim3(1), dim3(kThreads), 0, s, a);
    EPP_HIP_TRY(hipGetLastError());
    EPP_TRY(pinned.wait(s));
    if (host[0] != 0) {
        if (host[0] & 2) { epp_set_error("training id outside [0, %lld)", (long long)n); return EPP_ERR_OUT_OF_RANGE_ID; }
        if (host[0] & 4) { epp_set_error("a column id lies outside [0, %lld)", (long long)n); return EPP_ERR_OUT_OF_RANGE_ID; }
        epp_set_error("the row pointer does not rise from 0 to nnz");
        return EPP_ERR_INVALID_ARG;
    }
    for (int k = 0; k <= L; ++k) P->bitmaps[k].view(bm_all.as<unsigned long long>() + (size_t)k * a.bm_stride, bm_bytes);
    P->set_size[0] = host[1];
    P->set0_ids.view(set0.p, (size_t)host[1] * 4);
    for (int k = 0; k < L; ++k) {
        const long long* res = host + 2 + (size_t)k * kLevelWords;
        const int l = L - 1 - k;
        epp_path* p = new epp_path();
        P->path[l] = p;
        p->n = n;
        p->alloc = P->alloc;
        p->pool = &P->pool;
        p->rows_pool = &P->rows_pool;
        p->sources = P->bitmaps[k].as<unsigned long long>();
        p->n_src = P->set_size[k];
        p->nnz = res[0];
        p->n_rows = p->n_stream_rows = res[1];
        P->set_size[k + 1] = res[1];
        p->cv.view(cv_all.as<int2>() + (size_t)k * a.cv_stride, (size_t)res[0] * 8);
        p->row_ids.view(ids_all.as<int32_t>() + (size_t)k * a.ids_stride, (size_t)res[1] * 4);
        p->rowptr.view(ptr_all.as<int32_t>() + (size_t)k * a.ptr_stride, (size_t)(res[1] + 1) * 4);
        for (int c = 0; c < EPP_NCLASS; ++c) p->len_hist[c] = res[3 + c];
        p->max_len = res[3 + EPP_NCLASS];
        // fixed point: N^{k+1} == N^k makes every deeper layer this very path
        if (res[2] && k + 1 < L) {
            for (int j = k + 1; j < L; ++j) {
                P->set_size[j + 1] = P->set_size[k + 1];
                P->path[L - 1 - j] = p;
            }
            break;
        }
    }
    P->store = std::move(arena.store);
    guard.p = nullptr;
    *out = P;
    return EPP_OK;
}
