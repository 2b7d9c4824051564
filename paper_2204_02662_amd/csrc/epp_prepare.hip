// Execution path preparing on the GPU (Sec. 4): frontier expansion from the training set
// (Theorem 1's sets N^k), stable extraction of the filtered neighbour lists, row
// renumbering and prefix-sum compaction into compact CSR.  Hand-written for gfx950, wave64.
//
// One level k -> k+1 is two streaming passes over the edge array and two over the rows:
//   edge_mask     keep[j] = (col[j] in N^k) as one 64-bit ballot per 64 edges, the kept edges before
//                 each of them in its tile of 2048, and the tile's count
//   scan          exclusive scan of the tile counts
//   row_flags     filtered row pointer of every vertex from those counts; a vertex is in
//                 N^{k+1} iff its filtered list is non-empty -> next bitmap, members per 256 vertices
//   scan          exclusive scan of the member counts; its last act is to hand the level's five
//                 numbers (kept edges, members, errors, relation of N^k to N^{k+1}) to the host
//   rows_compact  ascending ids of N^{k+1}, compact row pointer, row-length statistics
//   edge_extract  stable compaction of (col, val) through the ballots
// The host waits once per level, for those numbers, and then allocates the level's arrays.
// All kept entries belong to rows of N^{k+1} by definition, so compacting the edge array
// alone yields the path's entries in canonical order.

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "epp_internal.h"

namespace {

constexpr int kBlock = 256;
constexpr int kSegsPerTile = 32;  // 32 ballots of 64 edges = 2048 edges
constexpr int kWordsPerTile = 64;  // bitmap words per workgroup (at most kBlock)
// Numbers of one level: [0] kept entries, [1] rows, [2] input errors (below), [3] N^k is not inside
// N^{k+1}, [4] N^k differs from N^{k+1}, [5] |N^0| (first level)
constexpr int kLevelWords = 8;
constexpr int kErrRowptr = 1, kErrCol = 2, kErrTrain = 4;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ unsigned long long low_mask(int lane) { return (1ull << lane) - 1ull; }

// Inclusive scan across the 64 lanes of a wavefront.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive scan over the 256 threads of a workgroup; *total receives the block sum.
__device__ __forceinline__ int block_exclusive_scan(int x, int* total) {
    __shared__ int wave_sum[4];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    int incl = wave_inclusive_scan(x);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) base += wave_sum[w];
        all += wave_sum[w];
    }
    __syncthreads();
    *total = all;
    return base + incl - x;
}

// N^0 = V_t as a bitmap; ids outside [0, n) raise the error flag instead of being written.
__global__ __launch_bounds__(kBlock) void k_mark_training(const int32_t* __restrict__ ids, int64_t n_ids, int64_t n,
                                                          unsigned int* __restrict__ bitmap32,
                                                          int* __restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_ids) return;
    int32_t v = ids[i];
    if (v < 0 || v >= n) { atomicOr(err, kErrTrain); return; }
    atomicOr(&bitmap32[v >> 5], 1u << (v & 31));
}

// The same, with the ascending ids and their number, by one workgroup that keeps the bitmap in LDS: for up to
// kSetVertices vertices and kSetIds training ids (marking, counting, scanning and listing are four
// launches of 4.5 us otherwise, whatever they process).  It also clears the results of the kernels to come (`clear`, up to kSetClear
// bytes; a memset is a launch of 5 us with the gap before it).
constexpr int kSetVertices = 524288, kSetIds = 65536;
constexpr size_t kSetClear = 262144;
__global__ __launch_bounds__(1024) void k_training_set(const int32_t* __restrict__ ids, int n_ids, int n,
                                                       unsigned long long* __restrict__ bitmap, int32_t* __restrict__ ids_out,
                                                       long long* count, int* err, ulonglong2* clear, int clear_pairs) {
    __shared__ unsigned long long bits[kSetVertices / 64];
    __shared__ int wave_sum[16];
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id(), n_words = (n + 63) >> 6;
    for (int i = tid; i < clear_pairs; i += 1024) clear[i] = make_ulonglong2(0ull, 0ull);
    for (int w = tid; w < n_words; w += 1024) bits[w] = 0ull;
    __syncthreads();
    unsigned int* bits32 = reinterpret_cast<unsigned int*>(bits);
    for (int i0 = tid; i0 < n_ids; i0 += 8 * 1024) {
        int v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = i0 + j * 1024 < n_ids ? ids[i0 + j * 1024] : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (i0 + j * 1024 >= n_ids) continue;
            if (v[j] < 0 || v[j] >= n) atomicOr(err, kErrTrain);
            else atomicOr(&bits32[v[j] >> 5], 1u << (v[j] & 31));
        }
    }
    __syncthreads();
    // consecutive words per thread, so that a scan of the threads' counts places every word
    const int per = (n_words + 1023) / 1024, w0 = min(tid * per, n_words), w1 = min(w0 + per, n_words);
    int mine = 0;
    for (int w = w0; w < w1; ++w) mine += __popcll(bits[w]);
    const int incl = wave_inclusive_scan(mine);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int at = incl - mine, all = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) at += wave_sum[w];
        all += wave_sum[w];
    }
    for (int w = w0; w < w1; ++w) {
        unsigned long long m = bits[w];
        bitmap[w] = m;
        for (; m; m &= m - 1ull) ids_out[at++] = w * 64 + __ffsll((long long)m) - 1;
    }
    if (tid == 0) *count = all;
}

struct MaskArgs {
    const int32_t* col;
    int64_t nnz, n_seg, n_tiles;
    int n;
    const unsigned int* bitmap;     // N^k
    int first_id, n_ids;            // ids looked up by this pass
    const unsigned long long* known;  // entries kept without a lookup (NULL: none; may be `mask` itself)
    int all;                        // N^k holds every vertex: every entry is kept, nothing is looked up
    int check;                      // range-check the columns (the first pass over the array)
    int count;                      // last pass of the level: write the counts
    unsigned long long* mask;
    uint16_t* seg_off;              // kept entries of the tile before each segment
    int* tile_count;
    int* err;
};

// keep-mask of every 64-edge segment, kept entries per tile and before each segment of a tile.  A
// wavefront owns a tile of 2048 entries and issues all its column loads, then all lookups, back to
// back, so that the dependent latencies are paid once.
//
// What bounds it: the lookups.  64 lanes look 64 different words up, which from L2 costs the address
// unit one cycle and more per lane: 250 G lookups/s on the whole chip, 0.52 ms for the 140 M
// entries of a co-purchase graph whose columns stream in 0.12 ms.  LDS serves a wavefront's 64
// words in a few cycles.  So a workgroup first copies a window of the bitmap into LDS (WORDS words:
// 1.28 M ids fit) and streams its tiles past it; where the graph has more vertices, one pass per
// window, each adding its finds to the mask.  A pass re-reads the columns (0.12 ms), so from three windows on
// k_edge_mask_folded takes over where the set is sparse or dense enough, and past three the
// lookups through L2 (k_edge_mask_far) otherwise.
//
// `known`: if N^{k-1} is a subset of N^k (always the case when every vertex has a self-loop), an
// entry kept at the previous level has its column in N^{k-1}, hence in N^k, and is kept again.  The
// next window of a level is handed the mask so far in the same way.
//
// Columns are range-checked by the first pass: an id outside [0, n) raises an error bit; it is
// never used as an index.
__device__ __forceinline__ unsigned long long lane_word(unsigned long long x, int i) {
    return (unsigned int)__builtin_amdgcn_readlane((int)x, i) |
           ((unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(x >> 32), i) << 32);
}

// Mask words and counts of a tile (lane i holds segment i's) to memory.
__device__ __forceinline__ void store_tile(const MaskArgs& a, int64_t tile, bool mine, unsigned long long out, int off, int run) {
    const int lane = lane_id();
    const int64_t seg = tile * kSegsPerTile + lane;
    if (mine) {
        a.mask[seg] = out;
        if (a.count) a.seg_off[seg] = (uint16_t)off;
    }
    if (a.count && lane == 0) a.tile_count[tile] = run;
}

// THREADS: 1,024, or 256 where the tiles are few and sixteen wavefronts would share one of a few CUs (0.5 M entries 9.3 -> 5.5 us, 4.2 M
// 10.0 -> 9.6).
template <int WORDS, int THREADS>
__global__ __launch_bounds__(THREADS) void k_edge_mask(MaskArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned int bits[WORDS + 4];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    {
        const int words = (a.n_ids + 31) >> 5, total = ((a.n + 63) >> 6) * 2 - (a.first_id >> 5);
        const unsigned int* __restrict__ src = a.bitmap + (a.first_id >> 5);
        for (int i = 4 * (int)threadIdx.x; i < words; i += 4 * THREADS) {
            uint4 x = make_uint4(0, 0, 0, 0);
            if (i + 4 <= total) {
                x = *reinterpret_cast<const uint4*>(src + i);
            } else {
                if (i < total) x.x = src[i];
                if (i + 1 < total) x.y = src[i + 1];
                if (i + 2 < total) x.z = src[i + 2];
            }
            *reinterpret_cast<uint4*>(bits + i) = x;
        }
        if (threadIdx.x == 0) bits[WORDS] = 0u;  // what every id outside the window looks up
        __syncthreads();
    }
    const int64_t step = (int64_t)gridDim.x * (THREADS / 64);
    for (int64_t tile = (int64_t)blockIdx.x * (THREADS / 64) + wave; tile < a.n_tiles; tile += step) {
        const int64_t seg0 = tile * kSegsPerTile;
        const bool mine = lane < kSegsPerTile && seg0 + lane < a.n_seg;
        const unsigned long long known = (a.known && mine) ? a.known[seg0 + lane] : 0ull;
        int c[kSegsPerTile];
        const int32_t* __restrict__ col = a.col + seg0 * 64 + lane;
        if ((seg0 + kSegsPerTile) * 64 <= a.nnz) {
#pragma unroll
            for (int i = 0; i < kSegsPerTile; ++i) c[i] = __builtin_nontemporal_load(col + i * 64);
        } else {
#pragma unroll
            for (int i = 0; i < kSegsPerTile; ++i) c[i] = (seg0 + i) * 64 + lane < a.nnz ? col[i * 64] : -1;
        }
        if (a.check) {
            unsigned int top = 0;  // (a negative id is a large unsigned one; so is the filler past the end)
#pragma unroll
            for (int i = 0; i < kSegsPerTile; ++i)
                top = max(top, (seg0 + i) * 64 + lane < a.nnz ? (unsigned int)c[i] : 0u);
            if (top >= (unsigned int)a.n) atomicOr(a.err, kErrCol);
        }
        unsigned int w[kSegsPerTile];
#pragma unroll
        for (int i = 0; i < kSegsPerTile; ++i) {
            c[i] -= a.first_id;
            w[i] = bits[(unsigned int)c[i] < (unsigned int)a.n_ids ? (unsigned int)c[i] >> 5 : WORDS];
        }
        unsigned long long out = 0ull;
        int off = 0, run = 0;
#pragma unroll
        for (int i = 0; i < kSegsPerTile; ++i) {
            const unsigned long long m = __ballot((w[i] >> (c[i] & 31)) & 1u) | lane_word(known, i);
            if (lane == i) {
                out = m;
                off = run;
            }
            run += __popcll(m);
        }
        store_tile(a, tile, mine, out, off, run);
    }
}

// Bit g of `folded`: whether any of the 2^shift ids (4 or 8) from g 2^shift on is in the set, or (ALL_OF) all of them are.
template <bool ALL_OF>
__global__ __launch_bounds__(kBlock) void k_fold_bitmap(const unsigned int* __restrict__ bitmap, int words, int shift, int out_words,
                                                        unsigned int* __restrict__ folded) {
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i >= out_words) return;
    unsigned int out = 0u;
    for (int k = 0; k < 1 << shift; ++k) {
        const int j = (i << shift) + k;
        unsigned int x = j < words ? bitmap[j] : 0u;
        if (ALL_OF) x = ~x;
        for (int t = 0; t < shift; ++t) x |= x >> (1 << t);
        // bits 0, 2^shift, .. to the front
        if (shift == 2) {
            x &= 0x11111111u;
            x = (x | x >> 3) & 0x03030303u;
            x = (x | x >> 6) & 0x000F000Fu;
            x = (x | x >> 12) & 0x000000FFu;
        } else {
            x &= 0x01010101u;
            x = (x | x >> 7) & 0x00030003u;
            x = (x | x >> 14) & 0x0000000Fu;
        }
        out |= x << (k * (32 >> shift));
    }
    folded[i] = ALL_OF ? ~out : out;
}

// The same for graphs of three windows and more, in one pass: the folded bitmap in LDS settles most ids (none of a
// group in the set, or, ALL_OF, all of them), the others are looked up through L2 while the columns stream in.  140 M entries
// with 15 / 25 % of them looked up: 0.21 / 0.25 ms (two windows 0.24, all looked up 0.52).  Preparation of three layers, 284 M
// entries, 8.4 M vertices: 4.36 -> 3.69 ms; 122 M, 4.5 M: 2.51 -> 1.95; of two, 76 M, 5 M: 1.48 -> 1.20.
template <int WORDS, bool ALL_OF>
__global__ __launch_bounds__(1024) void k_edge_mask_folded(MaskArgs a, const unsigned int* __restrict__ folded, int shift) {
    __shared__ __attribute__((aligned(16))) unsigned int bits[WORDS];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int words = (((a.n - 1) >> shift) >> 5) + 1;  // (at most WORDS; `folded` has room for whole quadruples)
    for (int i = 4 * (int)threadIdx.x; i < words; i += 4 * 1024)
        *reinterpret_cast<uint4*>(bits + i) = *reinterpret_cast<const uint4*>(folded + i);
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * 16;
    for (int64_t tile = (int64_t)blockIdx.x * 16 + wave; tile < a.n_tiles; tile += step) {
        const int64_t seg0 = tile * kSegsPerTile;
        const bool mine = lane < kSegsPerTile && seg0 + lane < a.n_seg;
        const unsigned long long known = (a.known && mine) ? a.known[seg0 + lane] : 0ull;
        int c[kSegsPerTile];
        const int32_t* __restrict__ col = a.col + seg0 * 64 + lane;
        if ((seg0 + kSegsPerTile) * 64 <= a.nnz) {
#pragma unroll
            for (int i = 0; i < kSegsPerTile; ++i) c[i] = __builtin_nontemporal_load(col + i * 64);
        } else {
#pragma unroll
            for (int i = 0; i < kSegsPerTile; ++i) c[i] = (seg0 + i) * 64 + lane < a.nnz ? col[i * 64] : -1;
        }
        if (a.check) {
            unsigned int top = 0;
#pragma unroll
            for (int i = 0; i < kSegsPerTile; ++i)
                top = max(top, (seg0 + i) * 64 + lane < a.nnz ? (unsigned int)c[i] : 0u);
            if (top >= (unsigned int)a.n) atomicOr(a.err, kErrCol);
        }
        unsigned long long out = 0ull;
        int off = 0, run = 0;
        constexpr int kHalf = kSegsPerTile / 2;
#pragma unroll
        for (int h = 0; h < kSegsPerTile; h += kHalf) {
            unsigned int in = 0u, open = 0u, w[kHalf];  // entries that are in the set; that are looked up
#pragma unroll
            for (int i = 0; i < kHalf; ++i) {
                const int id = c[h + i];
                const bool valid = (unsigned int)id < (unsigned int)a.n;
                const unsigned int g = valid ? (unsigned int)id >> shift : 0u;
                const bool bit = valid && ((bits[g >> 5] >> (g & 31)) & 1u);
                const bool look = (ALL_OF ? valid && !bit : bit) && !((lane_word(known, h + i) >> lane) & 1ull);
                if (ALL_OF && bit) in |= 1u << i;
                if (look) open |= 1u << i;
                w[i] = a.bitmap[look ? id >> 5 : 0];
            }
#pragma unroll
            for (int i = 0; i < kHalf; ++i) {
                const bool found = ((open >> i) & 1u) && ((w[i] >> (c[h + i] & 31)) & 1u);
                const unsigned long long m = __ballot(found || ((in >> i) & 1u)) | lane_word(known, h + i);
                if (lane == h + i) {
                    out = m;
                    off = run;
                }
                run += __popcll(m);
            }
        }
        store_tile(a, tile, mine, out, off, run);
    }
}

// The same with the lookups through L2, where known entries are neither loaded nor looked up; and, with
// `all`, the mask of a set that holds every vertex.
__global__ __launch_bounds__(kBlock) void k_edge_mask_far(MaskArgs a) {
    constexpr int kHalf = kSegsPerTile / 2;
    const int lane = lane_id();
    const int64_t step = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t tile = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); tile < a.n_tiles; tile += step) {
        const int64_t seg0 = tile * kSegsPerTile;
        const bool mine = lane < kSegsPerTile && seg0 + lane < a.n_seg;
        if (a.all) {
            const int64_t left = a.nnz - (seg0 + lane) * 64;
            store_tile(a, tile, mine, left >= 64 ? ~0ull : low_mask((int)max(left, (int64_t)0)), lane * 64,
                       (int)min(a.nnz - seg0 * 64, (int64_t)kSegsPerTile * 64));
            continue;
        }
        const unsigned long long known = (a.known && mine) ? a.known[seg0 + lane] : 0ull;
        unsigned long long out = 0ull;
        int off = 0, run = 0;
        bool bad = false;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int c[kHalf];
#pragma unroll
            for (int i = 0; i < kHalf; ++i) {
                const int64_t e = (seg0 + h * kHalf + i) * 64 + lane;
                const bool want = e < a.nnz && !((lane_word(known, h * kHalf + i) >> lane) & 1ull);
                c[i] = want ? __builtin_nontemporal_load(a.col + e) : -1;
                bad |= want && (c[i] < 0 || c[i] >= a.n);
            }
            unsigned int w[kHalf];
#pragma unroll
            for (int i = 0; i < kHalf; ++i) w[i] = (c[i] >= 0 && c[i] < a.n) ? a.bitmap[c[i] >> 5] : 0u;
#pragma unroll
            for (int i = 0; i < kHalf; ++i) {
                const int sg = h * kHalf + i;
                const unsigned long long m = __ballot((w[i] >> (c[i] & 31)) & 1u) | lane_word(known, sg);
                if (lane == sg) {
                    out = m;
                    off = run;
                }
                run += __popcll(m);
            }
        }
        if (a.check && bad) atomicOr(a.err, kErrCol);
        store_tile(a, tile, mine, out, off, run);
    }
}

// Exclusive scan of `n` counts (per-tile numbers of kept entries or set bits).  A workgroup of
// 1024 threads, kScanPerThread consecutive counts each, scans a chunk of kScanChunk counts;
// k_scan_counts walks all chunks in one workgroup (short arrays), the three-kernel form scans
// the chunks in parallel, then the chunk sums, then adds the chunk offsets.
constexpr int kScanPerThread = 8;
constexpr int kScanChunk = 1024 * kScanPerThread;

// Scans in[base .. base + kScanChunk) into out, starting from `carry`; returns the chunk's sum
// to every thread.  Called by all 1024 threads of the workgroup.  (The arrays are 16-byte aligned.)
__device__ __forceinline__ int scan_chunk(const int* __restrict__ in, int* __restrict__ out, int64_t n, int64_t base,
                                          int carry) {
    __shared__ int wave_sum[16];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanPerThread;
    const bool whole = i0 + kScanPerThread <= n;
    int x[kScanPerThread];
    int mine = 0;
    if (whole) {
#pragma unroll
        for (int j = 0; j < kScanPerThread; j += 4) {
            const int4 v = *reinterpret_cast<const int4*>(in + i0 + j);
            x[j] = v.x; x[j + 1] = v.y; x[j + 2] = v.z; x[j + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kScanPerThread; ++j) x[j] = i0 + j < n ? in[i0 + j] : 0;
    }
#pragma unroll
    for (int j = 0; j < kScanPerThread; ++j) mine += x[j];
    const int incl = wave_inclusive_scan(mine);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int off = carry, all = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) off += wave_sum[w];
        all += wave_sum[w];
    }
    __syncthreads();  // wave_sum is reused by the next call
    off += incl - mine;
#pragma unroll
    for (int j = 0; j < kScanPerThread; ++j) {
        const int v = x[j];
        x[j] = off;
        off += v;
    }
    if (whole) {
#pragma unroll
        for (int j = 0; j < kScanPerThread; j += 4)
            *reinterpret_cast<int4*>(out + i0 + j) = make_int4(x[j], x[j + 1], x[j + 2], x[j + 3]);
    } else {
#pragma unroll
        for (int j = 0; j < kScanPerThread; ++j)
            if (i0 + j < n) out[i0 + j] = x[j];
    }
    return all;
}

// With `level` (the numbers of a level, of which *total is one) and `host` (pinned): all of them are
// handed to the host.
__global__ __launch_bounds__(1024) void k_scan_counts(const int* __restrict__ in, int* __restrict__ out, int64_t n,
                                                      long long* total, const long long* level, long long* host) {
    int carry = 0;
    for (int64_t base = 0; base < n; base += kScanChunk) carry += scan_chunk(in, out, n, base, carry);
    if (threadIdx.x == 0) {
        *total = carry;
        if (host) {
            for (int i = 0; i < kLevelWords; ++i) host[i] = level + i == total ? (long long)carry : level[i];
        }
    }
}

__global__ __launch_bounds__(1024) void k_scan_chunks(const int* __restrict__ in, int* __restrict__ out, int64_t n,
                                                      int* __restrict__ chunk_sum) {
    const int all = scan_chunk(in, out, n, (int64_t)blockIdx.x * kScanChunk, 0);
    if (threadIdx.x == 0) chunk_sum[blockIdx.x] = all;
}

__global__ __launch_bounds__(1024) void k_scan_add_offsets(int* __restrict__ out, int64_t n,
                                                           const int* __restrict__ chunk_base) {
    const int off = chunk_base[blockIdx.x];
    const int64_t i0 = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPerThread;
#pragma unroll
    for (int j = 0; j < kScanPerThread; ++j)
        if (i0 + j < n) out[i0 + j] += off;
}

// Members of a level's set N^{k+1} before a vertex: bitmap, and the members before every 256 vertices.
struct Members {
    const unsigned long long* bitmap;
    const int* base;
    __device__ __forceinline__ int before(int v, int n) const {
        if (v >= n) v = n - 1;
        const int w0 = (v >> 8) * 4, w = v >> 6;
        int r = base[v >> 8];
        for (int i = w0; i < w; ++i) r += __popcll(bitmap[i]);
        return r + __popcll(bitmap[w] & low_mask(v & 63));
    }
};

// Copies of a path's statistics, which the workgroups are dealt to, so that no word is added to by more than 64 of them: atomics at one
// address follow each other at 20 to 40 ns.  (k_rows_compact, one copy and 512 workgroups at most
// -> 32 and 2,048: 89,000 vertices 8.6 -> 5.4 us, 1.1 M 16.0 -> 8.8.)
// A copy: EPP_NCLASS counts, then the longest row.
constexpr int kStatWords = EPP_NCLASS + 1;
template <int COPIES>
__device__ __forceinline__ unsigned long long* my_stats(unsigned long long* stats) { return stats + (blockIdx.x % COPIES) * kStatWords; }
// The sum of the copies' word i; of the last word the largest.
template <int COPIES>
__host__ __device__ inline unsigned long long stat_word(const unsigned long long* __restrict__ stats, int i) {
    unsigned long long x = 0ull;
#pragma unroll
    for (int c = 0; c < COPIES; ++c) {
        const unsigned long long y = stats[c * kStatWords + i];
        x = i < EPP_NCLASS ? x + y : std::max(x, y);
    }
    return x;
}
constexpr unsigned kRowBlocks = 2048;  // of k_rows_compact
constexpr int kRowCopies = 32;
constexpr int kImportCopies = 8;  // (they all go to the host)

// Where the kept entries of a level go: mask, and the counts before a tile and inside it.
struct Kept {
    const unsigned long long* mask;
    const uint16_t* seg_off;
    const int* tile_base;
    __device__ __forceinline__ int before_seg(int64_t seg) const { return tile_base[seg / kSegsPerTile] + seg_off[seg]; }
};

// Stable compaction of the kept entries into interleaved (col, val) pairs: a kept entry of
// segment s goes to (kept entries before s) + (kept entries before it in the segment).  With
// `inner.mask` (the keep-mask of the level before, a subset of this one) the entries that level did
// not keep get the kEntOuterOnly mark: the path of the level before will run on this array;
// inner_pos[q / 64] then receives, for every 64th entry q, how many entries before it that level kept.
//
// The last kept entry of every row gets the row-end flag: a workgroup looks through the path's rows that
// overlap its tile (tile_row[t]: the vertex of the tile's first entry) for those that end in it, while its
// entries are in flight.  They are 2,050 at most, as none of them is empty: the vertices in between can be
// millions.  (A kernel of its own that set the flags in the finished array took 0.1 ms for 2.4 M rows:
// a read and a write of 128 bytes for each.)
//
// TWO: a second level's entries, without marks, from the same read of the columns and values.
//
// The last one of a construction hands the levels' statistics to the host (pinned memory; a copy behind it is a launch of 6 us).
//
// Runs at the rate of a copy: 140 M entries in 0.41 ms, with 19 M of another level 0.46 ms; those by themselves took 0.23 ms, as
// nearly every line of the arrays holds some of them.  (What concerns a segment is fetched by one lane
// and read from there as a scalar; vector loads of it cost 0.45 ms more.)
struct Extracted {
    Kept kept;
    Members members;
    const int* ptr;
    int n_rows, total;
    int2* cv;
};
template <bool TWO>
__global__ __launch_bounds__(kBlock) void k_edge_extract(const int32_t* __restrict__ col, const float* __restrict__ val,
                                                         int64_t n_seg, Extracted a, Kept inner, int* __restrict__ inner_pos,
                                                         Extracted b, const int* __restrict__ tile_row, int n,
                                                         const unsigned long long* __restrict__ stats, int levels,
                                                         unsigned long long* __restrict__ host) {
    if (blockIdx.x == 0) {  // (none where `levels` is 0)
        for (int i = threadIdx.x; i < levels * kStatWords; i += kBlock)
            host[i] = stat_word<kRowCopies>(stats + i / kStatWords * kRowCopies * kStatWords, i % kStatWords);
    }
    constexpr int kPerWave = kSegsPerTile / 4;
    __shared__ unsigned int row_end[TWO ? 2 : 1][kSegsPerTile * 2];  // one bit per kept entry of the tile
    if (threadIdx.x < kSegsPerTile * 2) {
        row_end[0][threadIdx.x] = 0u;
        if constexpr (TWO) row_end[1][threadIdx.x] = 0u;
    }
    const int lane = lane_id();
    const int64_t seg0 = (int64_t)blockIdx.x * kSegsPerTile + (threadIdx.x >> 6) * kPerWave;
    // lane i fetches what concerns segment i; it is read from there as a scalar below
    unsigned long long am = 0ull, bm = 0ull, im = 0ull;
    int ab = 0, bb = 0, ib = 0;
    if (lane < kPerWave && seg0 + lane < n_seg) {
        am = a.kept.mask[seg0 + lane];
        ab = a.kept.before_seg(seg0 + lane);
        if constexpr (TWO) {
            bm = b.kept.mask[seg0 + lane];
            bb = b.kept.before_seg(seg0 + lane);
        }
        if (inner.mask) {
            im = inner.mask[seg0 + lane];
            ib = inner.before_seg(seg0 + lane);
        }
    }
    int2 x[kPerWave];
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) {
        const int64_t e = (seg0 + i) * 64 + lane;
        if ((lane_word(TWO ? am | bm : am, i) >> lane) & 1ull) x[i] = make_int2(col[e], __float_as_int(val[e]));
    }
    const bool last_tile = blockIdx.x + 1 == gridDim.x;
    const int a_base = a.kept.tile_base[blockIdx.x], a_limit = last_tile ? a.total : a.kept.tile_base[blockIdx.x + 1];
    int b_base = 0, b_limit = 0;
    if constexpr (TWO) {
        b_base = b.kept.tile_base[blockIdx.x];
        b_limit = last_tile ? b.total : b.kept.tile_base[blockIdx.x + 1];
    }
    __syncthreads();
    auto ends = [&](const Extracted& o, int base, int limit, unsigned int* __restrict__ bits) {
        if (limit <= base) return;
        // (the row of the next tile's first entry may end in this one, if that entry is not kept)
        const int r0 = o.members.before(tile_row[blockIdx.x], n);
        const int r1 = last_tile ? o.n_rows : min(o.members.before(tile_row[blockIdx.x + 1], n) + 1, o.n_rows);
        for (int r = r0 + (int)threadIdx.x; r < r1; r += kBlock) {
            const int q = o.ptr[r + 1];
            if (q > base && q <= limit) atomicOr(&bits[(q - 1 - base) >> 5], 1u << ((q - 1 - base) & 31));
        }
    };
    ends(a, a_base, a_limit, row_end[0]);
    if constexpr (TWO) ends(b, b_base, b_limit, row_end[1]);
    __syncthreads();
    auto put = [&](const Extracted& o, int base, const unsigned int* __restrict__ bits, int2 e, int q) {
        if ((bits[(q - base) >> 5] >> ((q - base) & 31)) & 1u) e.x |= kEntRowEnd;
        o.cv[q] = e;
    };
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) {
        const unsigned long long m = lane_word(am, i);
        const int q = __builtin_amdgcn_readlane(ab, i) + __popcll(m & low_mask(lane));
        if constexpr (TWO) {
            const unsigned long long own = lane_word(bm, i);
            if ((own >> lane) & 1ull)
                put(b, b_base, row_end[TWO], x[i], __builtin_amdgcn_readlane(bb, i) + __popcll(own & low_mask(lane)));
        }
        if (inner.mask) {  // (uniform)
            const unsigned long long in = lane_word(im, i);
            if (!((in >> lane) & 1ull)) x[i].x |= kEntOuterOnly;
            if (((m >> lane) & 1ull) && (q & 63) == 0)
                inner_pos[q >> 6] = __builtin_amdgcn_readlane(ib, i) + __popcll(in & low_mask(lane));
        }
        if ((m >> lane) & 1ull) put(a, a_base, row_end[0], x[i], q);
    }
}

// Filtered row pointer of every vertex, membership of N^{k+1}, members per 256 vertices, and how
// N^{k+1} relates to N^k; with `tile_row`, also the row of every tile's first entry.  A row pointer that does not rise from 0 to nnz raises an error bit; no
// index outside the mask arrays is formed.
__global__ __launch_bounds__(kBlock) void k_row_flags(const int32_t* __restrict__ rowptr, int64_t n, int64_t nnz, Kept kept,
                                                      long long* level, int* __restrict__ newptr,
                                                      const unsigned long long* __restrict__ bitmap_cur,
                                                      unsigned long long* __restrict__ bitmap_next,
                                                      int* __restrict__ row_count, int* __restrict__ tile_row) {
    __shared__ int wave_cnt[kBlock / 64], wave_rel[kBlock / 64];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int total = (int)level[0];  // kept entries of the level (the host has not read it yet)
    auto kept_before = [&](int64_t p) -> int {
        if (p < 0 || p >= nnz) return total;
        return kept.before_seg(p >> 6) + __popcll(kept.mask[p >> 6] & low_mask((int)(p & 63)));
    };
    const int p0 = v < n ? rowptr[v] : (int)nnz;
    int p1 = __shfl_down(p0, 1, 64);
    if (lane == 63) p1 = v + 1 <= n ? rowptr[v + 1] : (int)nnz;
    const int a = kept_before(p0);
    int b = __shfl_down(a, 1, 64);
    if (lane == 63) b = kept_before(p1);
    bool flag = false;
    int64_t t0 = 0, t1 = 0;  // tiles whose first entry is the row's
    if (v < n) {
        if (v == n - 1) p1 = rowptr[n];
        if (p0 < 0 || p1 < p0 || p1 > nnz || (v == 0 && p0 != 0) || (v == n - 1 && p1 != nnz))
            atomicOr(reinterpret_cast<int*>(level + 2), kErrRowptr);
        newptr[v] = a;
        if (v == n - 1) newptr[n] = total;
        flag = b > a;
        if (tile_row && p0 >= 0 && p1 > p0 && p1 <= nnz) {  // (first level: the rows of the tiles' first entries)
            constexpr int kTile = kSegsPerTile * 64;
            t0 = ((int64_t)p0 + kTile - 1) / kTile;
            t1 = ((int64_t)p1 + kTile - 1) / kTile;
        }
    }
    if (tile_row) for_range_by_wave(t0, t1, [&](int64_t t, int lane_of_row) { tile_row[t] = (int)(v - lane + lane_of_row); });
    const unsigned long long bal = __ballot(flag);
    if (lane == 0) {
        const bool in = v < n;
        if (in) bitmap_next[v >> 6] = bal;
        const unsigned long long cur = in ? bitmap_cur[v >> 6] : 0ull;
        wave_cnt[wave] = __popcll(bal);
        wave_rel[wave] = ((cur & ~bal) ? 1 : 0) | (cur != bal ? 2 : 0);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int cnt = 0, rel = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            cnt += wave_cnt[w];
            rel |= wave_rel[w];
        }
        row_count[blockIdx.x] = cnt;
        if (rel & 1) level[3] = 1;  // (plain stores: every writer stores the same value)
        if (rel & 2) level[4] = 1;
    }
}

// Adds a row to the workgroup's histogram (one copy per wavefront, so that at most 64 lanes queue at
// a counter).
constexpr int kHists = kBlock / 64;
__device__ __forceinline__ void add_length(int* __restrict__ h, int len) {
    atomicAdd(&h[(threadIdx.x >> 6) * EPP_NCLASS + length_class(len)], 1);
}
__device__ __forceinline__ void clear_lengths(int* __restrict__ h, int* __restrict__ mx) {
    for (int i = threadIdx.x; i < kHists * EPP_NCLASS; i += kBlock) h[i] = 0;
    if (threadIdx.x == 0) *mx = 0;
    __syncthreads();
}
// The workgroup's counts and longest row to the statistics in memory (few workgroups: their atomics
// meet at the same 33 words).
__device__ __forceinline__ void flush_lengths(const int* __restrict__ h, int* __restrict__ mx, int my_max,
                                              unsigned long long* __restrict__ hist, int* __restrict__ max_len) {
    if (my_max) atomicMax(mx, my_max);
    __syncthreads();
    if (threadIdx.x < EPP_NCLASS) {
        int c = 0;
#pragma unroll
        for (int w = 0; w < kHists; ++w) c += h[w * EPP_NCLASS + threadIdx.x];
        if (c) atomicAdd(&hist[threadIdx.x], (unsigned long long)c);
    }
    if (threadIdx.x == 0 && *mx) atomicMax(max_len, *mx);
}
constexpr unsigned kStatBlocks = 512;
// Ascending ids of N^{k+1}, compact row pointer, row-length statistics and the list of long rows; a workgroup takes 256 vertices at a time.
__global__ __launch_bounds__(kBlock) void k_rows_compact(const unsigned long long* __restrict__ bitmap, int64_t n,
                                                         const int* __restrict__ row_base, const int* __restrict__ newptr,
                                                         int32_t* __restrict__ ids, int32_t* __restrict__ ptr_out,
                                                         int64_t n_set, int total_nnz,
                                                         unsigned long long* __restrict__ stats, LongRows list) {
    __shared__ int h[kHists * EPP_NCLASS], found[2 * EPP_NCLASS];
    __shared__ int mx;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    clear_lengths(h, &mx);
    int my_max = 0;
    const int64_t tiles = (n + kBlock - 1) / kBlock, n_words = (n + 63) >> 6;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        int at = row_base[t];
        unsigned long long m = 0ull;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            const unsigned long long x = t * 4 + w < n_words ? bitmap[t * 4 + w] : 0ull;
            if (w < wave) at += __popcll(x);
            if (w == wave) m = x;
        }
        const int64_t v = t * kBlock + threadIdx.x;
        int p = 0, len = 0;
        if ((m >> lane) & 1ull) {
            const int r = at + __popcll(m & low_mask(lane));
            p = newptr[v];
            len = newptr[v + 1] - p;
            ids[r] = (int32_t)v;
            ptr_out[r] = p;
            my_max = max(my_max, len);
            add_length(h, len);
        }
        if (list.rows) list_long_rows(list, (int)v, p, len, found);
    }
    stats = my_stats<kRowCopies>(stats);
    flush_lengths(h, &mx, my_max, stats, reinterpret_cast<int*>(stats + EPP_NCLASS));
    if (blockIdx.x == 0 && threadIdx.x == 0) ptr_out[n_set] = total_nnz;
    if (blockIdx.x == 0 && list.rows) place_long_rows(list);
}

__global__ __launch_bounds__(kBlock) void k_bitmap_count(const unsigned long long* __restrict__ bitmap, int64_t n_words,
                                                         int* __restrict__ tile_count) {
    int64_t w = (int64_t)blockIdx.x * kWordsPerTile + threadIdx.x;
    int c = threadIdx.x < kWordsPerTile && w < n_words ? __popcll(bitmap[w]) : 0;
    int total;
    (void)block_exclusive_scan(c, &total);
    if (threadIdx.x == 0) tile_count[blockIdx.x] = total;
}

// Ascending ids of the set bits; optionally the compact row pointer gathered from newptr.
__global__ __launch_bounds__(kBlock) void k_bitmap_compact(const unsigned long long* __restrict__ bitmap,
                                                           int64_t n_words, const int* __restrict__ tile_base,
                                                           const int* __restrict__ newptr, int32_t* __restrict__ ids,
                                                           int32_t* __restrict__ ptr_out, int64_t n_set,
                                                           int total_nnz) {
    __shared__ int wbase[kWordsPerTile];
    int64_t w = (int64_t)blockIdx.x * kWordsPerTile + threadIdx.x;
    int c = threadIdx.x < kWordsPerTile && w < n_words ? __popcll(bitmap[w]) : 0;
    int total;
    const int before = block_exclusive_scan(c, &total);
    if (threadIdx.x < kWordsPerTile) wbase[threadIdx.x] = before;
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int tb = tile_base[blockIdx.x];
    for (int i = wave; i < kWordsPerTile; i += 4) {
        int64_t ww = (int64_t)blockIdx.x * kWordsPerTile + i;
        if (ww >= n_words) break;
        unsigned long long m = bitmap[ww];
        if ((m >> lane) & 1ull) {
            int r = tb + wbase[i] + __popcll(m & low_mask(lane));
            int32_t v = (int32_t)(ww * 64 + lane);
            ids[r] = v;
            if (ptr_out) ptr_out[r] = newptr[v];
        }
    }
    if (ptr_out && blockIdx.x == 0 && threadIdx.x == 0) ptr_out[n_set] = total_nnz;
}

// Row-length histogram by class and the maximal length.
__global__ __launch_bounds__(kBlock) void k_len_hist(const int32_t* __restrict__ rowptr, int64_t n_rows,
                                                     unsigned long long* __restrict__ hist, int* __restrict__ max_len) {
    __shared__ int h[kHists * EPP_NCLASS];
    __shared__ int mx;
    clear_lengths(h, &mx);
    int my_max = 0;
    const int64_t span = (int64_t)gridDim.x * kBlock;
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < n_rows; r += span) {
        const int len = rowptr[r + 1] - rowptr[r];
        my_max = max(my_max, len);
        add_length(h, len);
    }
    flush_lengths(h, &mx, my_max, hist, max_len);
}

// Interleave a plain CSR's (col, val) into pairs (all-active graph).
// A column outside [0, n) raises bit 1 of *err (if given) and is stored as 0.
__global__ __launch_bounds__(kBlock) void k_interleave(const int32_t* __restrict__ col, const float* __restrict__ val,
                                                       int64_t nnz, int64_t n, int2* __restrict__ cv,
                                                       int* __restrict__ err) {
    int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= nnz) return;
    int32_t c = col[e];
    if (c < 0 || c >= n) {
        if (err) atomicOr(err, 2);
        c = 0;
    }
    cv[e] = make_int2(c, __float_as_int(val[e]));
}

// Row pointer of a whole graph: must rise from 0 to nnz (bit 0 of *err otherwise).
__global__ __launch_bounds__(kBlock) void k_check_rowptr(const int32_t* __restrict__ rowptr, int64_t n, int64_t nnz,
                                                         int* __restrict__ err) {
    int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (v >= n) return;
    const int64_t p0 = rowptr[v], p1 = rowptr[v + 1];
    if (p0 < 0 || p1 < p0 || p1 > nnz || (v == 0 && p0 != 0) || (v == n - 1 && p1 != nnz)) atomicOr(err, 1);
}

// A path in canonical form, into the caller's arrays (any of which may be NULL), in one launch: the
// first entry_blocks workgroups write the entries without their flags, kExportSegs segments of 64
// per wavefront, the others the row ids (NULL: 0 .. n_rows - 1) and the row pointer.
//
// INNER: the path is an inner one that shares these entries.  Its entries are those without the
// kEntOuterOnly mark, in the same order; inner_pos (recorded when the array was extracted) says
// where a segment's entries go, so one pass over the array is enough.
//
// Runs at the rate of a copy: 140 M entries (1.1 GB read, 1.1 GB written) in 0.4 to 0.47 ms.  (A
// wavefront per inner row, with a search for the row, took 6.3 ms.)
constexpr int kExportSegs = 4;
template <bool INNER>
__global__ __launch_bounds__(kBlock) void k_export(const int2* __restrict__ cv, int64_t nnz,
                                                   const int* __restrict__ inner_pos, int64_t out_nnz, unsigned entry_blocks,
                                                   int32_t* __restrict__ col, float* __restrict__ val,
                                                   const int32_t* __restrict__ row_ids, const int32_t* __restrict__ rowptr,
                                                   int64_t n_rows, int32_t* __restrict__ ids_out,
                                                   int32_t* __restrict__ ptr_out) {
    if (blockIdx.x >= entry_blocks) {
        const int64_t r = (int64_t)(blockIdx.x - entry_blocks) * kBlock + threadIdx.x;
        if (ids_out && r < n_rows) ids_out[r] = row_ids ? row_ids[r] : (int32_t)r;
        if (ptr_out && r <= n_rows) ptr_out[r] = rowptr[r];
        return;
    }
    const int64_t seg0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * kExportSegs;
    const int lane = lane_id();
    int2 x[kExportSegs];
    int at[kExportSegs];
#pragma unroll
    for (int i = 0; i < kExportSegs; ++i) {
        const int64_t e = (seg0 + i) * 64 + lane;
        x[i] = e < nnz ? cv[e] : make_int2(kEntOuterOnly, 0);
        if constexpr (INNER) at[i] = (seg0 + i) * 64 < nnz ? inner_pos[seg0 + i] : 0;
    }
#pragma unroll
    for (int i = 0; i < kExportSegs; ++i) {
        int64_t j = (seg0 + i) * 64 + lane;
        bool keep = j < nnz;
        if constexpr (INNER) {
            keep = !(x[i].x & kEntOuterOnly);
            j = at[i] + __popcll(__ballot(keep) & low_mask(lane));
            keep &= j < out_nnz;  // (only guards against arrays that do not belong together)
        }
        if (keep) {
            if (col) col[j] = x[i].x & kEntCol;
            if (val) val[j] = __int_as_float(x[i].y);
        }
    }
}

// Flag the last entry of every (non-empty) row in bit 31 of its column id.
__global__ __launch_bounds__(kBlock) void k_mark_row_ends(const int32_t* __restrict__ rowptr, int64_t n_rows,
                                                          int2* __restrict__ cv) {
    int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= n_rows) return;
    const int32_t end = rowptr[r + 1];
    if (end > rowptr[r]) cv[end - 1].x |= kEntRowEnd;
}

// Bitmap of the vertices with a non-empty (invert = 0) or empty (invert = 1) list.
__global__ __launch_bounds__(kBlock) void k_nonempty_bitmap(const int32_t* __restrict__ rowptr, int64_t n, int invert,
                                                            unsigned long long* __restrict__ bitmap) {
    int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    bool flag = false;
    if (v < n) flag = (rowptr[v + 1] > rowptr[v]) != (invert != 0);
    unsigned long long bal = __ballot(flag);
    if (lane_id() == 0 && (v >> 6) < ((n + 63) >> 6)) bitmap[v >> 6] = bal;
}

inline unsigned grid_for(int64_t n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }

// out = exclusive scan of in[0 .. n), *total = sum.  `tmp` holds two arrays of a number per chunk.
inline int64_t scan_tmp_stride(int64_t n) { return ((n + kScanChunk - 1) / kScanChunk + 3) & ~(int64_t)3; }
inline size_t scan_tmp_bytes(int64_t n) { return (size_t)(2 * scan_tmp_stride(n)) * sizeof(int); }
// `level`, `host`: see k_scan_counts.
void scan_counts(const int* in, int* out, int64_t n, long long* total, int* tmp, hipStream_t s,
                 const long long* level = nullptr, long long* host = nullptr) {
    const int64_t chunks = (n + kScanChunk - 1) / kScanChunk;
    if (chunks <= 4) {
        hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, s, in, out, n, total, (const long long*)level, host);
        return;
    }
    int* chunk_sum = tmp;
    int* chunk_base = tmp + scan_tmp_stride(n);
    hipLaunchKernelGGL(k_scan_chunks, dim3((unsigned)chunks), dim3(1024), 0, s, in, out, n, chunk_sum);
    hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, s, (const int*)chunk_sum, chunk_base, chunks, total,
                       level, host);
    hipLaunchKernelGGL(k_scan_add_offsets, dim3((unsigned)chunks), dim3(1024), 0, s, out, n, (const int*)chunk_base);
}

int validate_csr(const epp_csr_t* g) {
    if (!g) { epp_set_error("graph is NULL"); return EPP_ERR_INVALID_ARG; }
    if (g->n < 0 || g->nnz < 0) { epp_set_error("negative graph size"); return EPP_ERR_INVALID_ARG; }
    if (g->n >= kMaxVertices || g->nnz >= 0x7FFFFFFFll) {
        epp_set_error("graph too large: n=%lld (limit 2^29-1) nnz=%lld (limit 2^31-1)", (long long)g->n,
                      (long long)g->nnz);
        return EPP_ERR_TOO_LARGE;
    }
    if (!g->rowptr || (g->nnz > 0 && (!g->col || !g->val))) {
        epp_set_error("graph arrays are NULL");
        return EPP_ERR_INVALID_ARG;
    }
    return EPP_OK;
}

// Ascending ids of a bitmap (and optionally the compact row pointer).  Returns the count.
int compact_bitmap(const DevBuf& bitmap, int64_t n, const int* newptr, int total_nnz, DevBuf* ids, DevBuf* ptr_out,
                   int64_t* count, DevBuf& tile_cnt, DevBuf& tile_base, DevBuf& dev_total, PinnedWords& hs,
                   const epp_alloc_t* al, hipStream_t s) {
    const int64_t n_words = (n + 63) / 64;
    const unsigned tiles = grid_for(n_words, kWordsPerTile);
    long long R = 0;
    if (tiles) {
        hipLaunchKernelGGL(k_bitmap_count, dim3(tiles), dim3(kBlock), 0, s, bitmap.as<unsigned long long>(), n_words,
                           tile_cnt.as<int>());
        hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, s, tile_cnt.as<int>(), tile_base.as<int>(),
                           (int64_t)tiles, dev_total.as<long long>(), (const long long*)nullptr, (long long*)nullptr);
        EPP_HIP_TRY(hipMemcpyAsync(hs.p, dev_total.p, sizeof(long long), hipMemcpyDeviceToHost, s));
        EPP_HIP_TRY(hipStreamSynchronize(s));
        R = hs.p[0];
    }
    *count = R;
    if (!ids) return EPP_OK;
    EPP_TRY(ids->alloc((size_t)R * sizeof(int32_t), al));
    if (ptr_out) EPP_TRY(ptr_out->alloc((size_t)(R + 1) * sizeof(int32_t), al));
    if (tiles) {
        hipLaunchKernelGGL(k_bitmap_compact, dim3(tiles), dim3(kBlock), 0, s, bitmap.as<unsigned long long>(), n_words,
                           tile_base.as<int>(), newptr, ids->as<int32_t>(),
                           ptr_out ? ptr_out->as<int32_t>() : nullptr, (int64_t)R, total_nnz);
    } else if (ptr_out) {
        EPP_HIP_TRY(hipMemsetAsync(ptr_out->p, 0, sizeof(int32_t), s));
    }
    EPP_HIP_TRY(hipGetLastError());
    return EPP_OK;
}

constexpr int kFoldedWords = 39936;

// keep-mask of one level: windows of the bitmap in LDS, or lookups through L2 (see k_edge_mask).
void launch_edge_mask(const epp_csr_t* g, int64_t n_seg, unsigned n_tiles, const unsigned int* bitmap,
                      const unsigned long long* known, bool all, bool check, double share, double known_share, unsigned int* folded,
                      unsigned long long* mask, uint16_t* seg_off, int* tile_count, int* err, hipStream_t s) {
    constexpr int kSmall = 8192, kLarge = kFoldedWords;  // words: 32 KB (two workgroups per CU), 156 KB (one)
    MaskArgs a;
    a.col = g->col;
    a.nnz = g->nnz;
    a.n_seg = n_seg;
    a.n_tiles = n_tiles;
    a.n = (int)g->n;
    a.bitmap = bitmap;
    a.known = known;
    a.all = all;
    a.mask = mask;
    a.seg_off = seg_off;
    a.tile_count = tile_count;
    a.err = err;
    const int64_t window = g->n <= kSmall * 32 ? kSmall * 32 : kLarge * 32;
    const int64_t passes = (g->n + window - 1) / window;
    // (copying the folded bitmap into every CU's LDS takes as long as 6 M lookups through L2)
    if (!all && (passes == 3 || (passes > 3 && g->nnz >= 6000000))) {
        int shift = 2;
        while (((g->n - 1) >> shift) >= (int64_t)kLarge * 32) ++shift;
        const double any = 1.0 - std::pow(1.0 - share, 1 << shift), not_all = 1.0 - std::pow(share, 1 << shift);
        // (as if an entry's column were any vertex, and its neighbours' membership nothing to do with its own)
        const double looked_up = std::min(any, not_all);
        if (shift <= 3 && looked_up < (passes > 3 ? 0.6 * (1.0 - known_share) : 0.4)) {
            const bool all_of = not_all < any;
            const int words = (int)((g->n + 31) >> 5), out_words = (int)(((((g->n - 1) >> shift) >> 5) + 4) & ~3ll);
            hipLaunchKernelGGL(all_of ? k_fold_bitmap<true> : k_fold_bitmap<false>, dim3(grid_for(out_words, kBlock)), dim3(kBlock), 0, s,
                               bitmap, words, shift, out_words, folded);
            a.first_id = 0;
            a.n_ids = a.n;
            a.check = check;
            a.count = 1;
            hipLaunchKernelGGL((all_of ? k_edge_mask_folded<kLarge, true> : k_edge_mask_folded<kLarge, false>),
                               dim3(std::min(grid_for(n_tiles, 16), 256u)), dim3(1024), 0, s, a, folded, shift);
            return;
        }
    }
    if (all || passes > 3) {
        a.first_id = 0;
        a.n_ids = a.n;
        a.check = check;
        a.count = 1;
        hipLaunchKernelGGL(k_edge_mask_far, dim3(std::min(grid_for(n_tiles, kBlock / 64), 16384u)), dim3(kBlock), 0, s, a);
        return;
    }
    for (int64_t w = 0; w < passes; ++w) {
        a.first_id = (int)(w * window);
        a.n_ids = (int)std::min(window, g->n - w * window);
        a.check = check && w == 0;
        a.count = w == passes - 1;
        if (w > 0) a.known = mask;
        if (window == kSmall * 32 && n_tiles <= 2048)
            hipLaunchKernelGGL((k_edge_mask<kSmall, 256>), dim3(grid_for(n_tiles, 4)), dim3(256), 0, s, a);
        else if (window == kSmall * 32)
            hipLaunchKernelGGL((k_edge_mask<kSmall, 1024>), dim3(std::min(grid_for(n_tiles, 16), 512u)), dim3(1024), 0, s, a);
        else
            hipLaunchKernelGGL((k_edge_mask<kLarge, 1024>), dim3(std::min(grid_for(n_tiles, 16), 256u)), dim3(1024), 0, s, a);
    }
}

// An imported path, copied and checked in one launch: the first row_blocks workgroups take the rows,
// the others a tile of kImportTile entries each.
//
// Rows: an error bit if ids do not ascend, the pointer decreases, a row is empty or the end points are
// wrong; another for an id outside [0, n).  They are counted into the row-length statistics and set in
// the bitmap of the row set.  Ids ascend, so neighbouring lanes share bitmap words: the bits of a
// word are gathered by a segmented scan across the wavefront and set by its last lane, one atomic per
// word instead of one per row.
//
// Entries: columns in range, interleaved with the weights; the last entry of every row gets the
// row-end flag.  A tile's first row is found by a search with 256 probes a step, and as no row is
// empty at most kImportTile + 1 of them concern it (whatever an invalid pointer holds).
struct ImportArgs {
    const int32_t *row_ids, *rowptr, *col;
    const float* val;
    int64_t n_rows, nnz, n;
    int32_t *ids_out, *ptr_out;
    int2* cv;
    unsigned int* bitmap32;
    unsigned long long* stats;
    int* err;
    unsigned row_blocks;
    LongRows list;
};
constexpr int kImportTile = 2048;
// The workgroups of several paths in one launch, each path's behind those of the one before.
constexpr int kImportPaths = 4;
struct ImportPaths {
    ImportArgs path[kImportPaths];
    unsigned end[kImportPaths];
};
__global__ __launch_bounds__(kBlock) void k_import_path(ImportPaths all) {
    unsigned block = blockIdx.x;
    int at = 0;
    while (at < kImportPaths - 1 && blockIdx.x >= all.end[at]) block = blockIdx.x - all.end[at++];
    const ImportArgs& a = all.path[at];
    __shared__ int h[kHists * EPP_NCLASS], found[2 * EPP_NCLASS];
    __shared__ int mx;
    __shared__ unsigned int row_end[kImportTile / 32];
    const int lane = lane_id();
    if (block >= a.row_blocks) {
        const int64_t e0 = (int64_t)(block - a.row_blocks) * kImportTile;
        constexpr int kPer = kImportTile / kBlock;
        int2 x[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int64_t e = e0 + i * kBlock + threadIdx.x;
            x[i] = e < a.nnz ? make_int2(a.col[e], __float_as_int(a.val[e])) : make_int2(0, 0);
        }
        if (threadIdx.x < kImportTile / 32) row_end[threadIdx.x] = 0u;
        int64_t lo = 0, hi = a.n_rows;  // the row of entry e0: the last one that starts at or before it
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + kBlock - 1) / kBlock, r = lo + (int64_t)threadIdx.x * step;
            const int below = __syncthreads_count(r < hi && a.rowptr[r] <= e0);
            lo += (int64_t)max(below - 1, 0) * step;
            hi = std::min<int64_t>(lo + step, hi);
        }
        __syncthreads();
        for (int64_t r = lo + threadIdx.x; r < std::min<int64_t>(lo + kImportTile + 1, a.n_rows); r += kBlock) {
            const int64_t end = (int64_t)a.rowptr[r + 1] - 1 - e0;
            if (end >= 0 && end < kImportTile) atomicOr(&row_end[end >> 5], 1u << (end & 31));
        }
        __syncthreads();
        bool bad = false;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int t = i * kBlock + threadIdx.x;
            if (e0 + t >= a.nnz) continue;
            if (x[i].x < 0 || x[i].x >= a.n) {
                bad = true;
                x[i].x = 0;
            }
            if ((row_end[t >> 5] >> (t & 31)) & 1u) x[i].x |= kEntRowEnd;
            a.cv[e0 + t] = x[i];
        }
        if (bad) atomicOr(a.err, kErrCol);
        return;
    }
    clear_lengths(h, &mx);
    int my_max = 0, bad = 0;
    const int64_t span = (int64_t)a.row_blocks * kBlock;
    // (one index past the rows, for the end of the pointer; the whole workgroup enters every iteration)
    for (int64_t base = (int64_t)block * kBlock; base <= a.n_rows; base += span) {
        const int64_t r = base + threadIdx.x;
        const bool row = r < a.n_rows;
        const int p = r <= a.n_rows ? a.rowptr[r] : 0;
        const int v = row ? a.row_ids[r] : -1;
        const int prev = row && r > 0 ? a.row_ids[r - 1] : -1;
        const int len = row ? a.rowptr[r + 1] - p : 0;
        if (r <= a.n_rows) a.ptr_out[r] = p;
        if ((r == 0 && p != 0) || (r == a.n_rows && p != a.nnz)) bad |= kErrRowptr;
        bool in = false;
        if (row) {
            a.ids_out[r] = v;
            in = v >= 0 && v < a.n;
            if (!in) bad |= kErrCol;
            if (prev >= v || len <= 0) bad |= kErrRowptr;
            my_max = max(my_max, len);
        }
        const int word = in ? v >> 5 : -1;
        unsigned int b = in ? 1u << (v & 31) : 0u;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned int other = __shfl_up(b, d, 64);
            const int other_word = __shfl_up(word, d, 64);
            if (lane >= d && other_word == word) b |= other;
        }
        const int next_word = __shfl_down(word, 1, 64);
        if (in && (lane == 63 || next_word != word)) atomicOr(&a.bitmap32[word], b);
        if (row && len > 0) add_length(h, len);
        if (a.list.rows) list_long_rows(a.list, v, p, row ? len : 0, found);
    }
    if (bad) atomicOr(a.err, bad);
    if (block == 0 && a.list.rows) place_long_rows(a.list);
    unsigned long long* const stats = my_stats<kImportCopies>(a.stats);
    flush_lengths(h, &mx, my_max, stats, reinterpret_cast<int*>(stats + EPP_NCLASS));
}

// *outside = 1 if an entry's column is not in the bitmap.  Bound by the lookups, which come from L2 (250 G/s), eight in
// flight per lane.
constexpr int kCheckPer = 8;
__global__ __launch_bounds__(kBlock) void k_columns_inside(const int2* __restrict__ cv, int64_t nnz,
                                                           const unsigned int* __restrict__ bitmap32, int* __restrict__ outside) {
    const int64_t e0 = (int64_t)blockIdx.x * (kBlock * kCheckPer) + threadIdx.x;
    int c[kCheckPer];
    unsigned int w[kCheckPer];
#pragma unroll
    for (int i = 0; i < kCheckPer; ++i) c[i] = cv[min(e0 + i * kBlock, nnz - 1)].x & kEntCol;
#pragma unroll
    for (int i = 0; i < kCheckPer; ++i) w[i] = bitmap32[c[i] >> 5];
    unsigned int in = 1u;
#pragma unroll
    for (int i = 0; i < kCheckPer; ++i) in &= w[i] >> (c[i] & 31);
    if (!(in & 1u)) *outside = 1;  // (every writer stores the same value)
}

// N^0 as a bitmap and its ascending ids; *count receives their number.  `clear`, `clear_bytes`: what is cleared before (256 bytes
// or a multiple, `count` and `err` among them, not the bitmap).
int launch_training_set(const int32_t* train_ids, int64_t n_train, int64_t n, const DevBuf& bitmap, void* ids_out,
                        int* tile_cnt, int* tile_base, int* scan_tmp, long long* count, int* err, void* clear, size_t clear_bytes,
                        hipStream_t s) {
    if (n_train > 0 && n > 0 && n <= kSetVertices && n_train <= kSetIds && clear_bytes <= kSetClear) {
        hipLaunchKernelGGL(k_training_set, dim3(1), dim3(1024), 0, s, train_ids, (int)n_train, (int)n,
                           bitmap.as<unsigned long long>(), static_cast<int32_t*>(ids_out), count, err, static_cast<ulonglong2*>(clear),
                           (int)(clear_bytes / sizeof(ulonglong2)));
        return EPP_OK;
    }
    EPP_HIP_TRY(hipMemsetAsync(clear, 0, clear_bytes, s));
    EPP_HIP_TRY(hipMemsetAsync(bitmap.p, 0, bitmap.bytes, s));
    if (n_train == 0) return EPP_OK;
    const int64_t n_words = (n + 63) / 64;
    const unsigned tiles = grid_for(n_words, kWordsPerTile);
    hipLaunchKernelGGL(k_mark_training, dim3(grid_for(n_train, kBlock)), dim3(kBlock), 0, s, train_ids, n_train, n,
                       bitmap.as<unsigned int>(), err);
    if (n == 0) return EPP_OK;
    hipLaunchKernelGGL(k_bitmap_count, dim3(tiles), dim3(kBlock), 0, s, bitmap.as<unsigned long long>(), n_words, tile_cnt);
    scan_counts(tile_cnt, tile_base, tiles, count, scan_tmp, s);
    hipLaunchKernelGGL(k_bitmap_compact, dim3(tiles), dim3(kBlock), 0, s, bitmap.as<unsigned long long>(), n_words, tile_base,
                       (const int*)nullptr, static_cast<int32_t*>(ids_out), (int32_t*)nullptr, (int64_t)0, 0);
    return EPP_OK;
}

// Message and code for the error bits raised by the input checks (bit 0 row pointer, bit 1 ids).
long long env_share_pct() {
    const char* e = std::getenv("EPP_TUNE_SHARE_PCT");
    return (e && *e) ? std::atoll(e) : 95;
}

// Memory of a path's rows, whose numbers are known: row ids | row pointer | list of long rows, each 256-byte aligned.  `head`: cleared, of that
// list, and stays with it.
int alloc_rows(epp_path* p, char* head, const epp_alloc_t* al) {
    const size_t ids_bytes = (size_t)p->n_rows * 4, ptr_bytes = (size_t)(p->n_rows + 1) * 4, list_bytes = epp_plan_long_rows(p->nnz, &p->long_rows);
    const size_t ptr_at = DevArena::rounded(ids_bytes), list_at = ptr_at + DevArena::rounded(ptr_bytes);
    EPP_TRY(p->store.alloc(list_at + list_bytes, al));
    p->row_ids.view(p->store.p, ids_bytes);
    p->rowptr.view(p->store.as<char>() + ptr_at, ptr_bytes);
    if (list_bytes) {
        p->long_rows.rows = reinterpret_cast<LongRow*>(p->store.as<char>() + list_at);
        p->long_rows.head = reinterpret_cast<int*>(head);
    }
    return EPP_OK;
}

int input_error(int bits, int64_t n) {
    if (bits & 2) { epp_set_error("a column id lies outside [0, %lld)", (long long)n); return EPP_ERR_OUT_OF_RANGE_ID; }
    epp_set_error("the row pointer does not rise from 0 to nnz");
    return EPP_ERR_INVALID_ARG;
}

}  // namespace

// Pinned blocks of every host thread that is inside a call: a list of idle ones, so that calls do
// not each pay for a pinned allocation and its release (together 0.1 ms).  At most kIdlePinned stay
// in the list; the rest goes back to the runtime.
namespace {
constexpr size_t kPinnedBlock = 4096, kIdlePinned = 16;
std::mutex g_pinned_lock;
PinnedWords::Block g_pinned_idle[kIdlePinned];
size_t g_pinned_count = 0;
}  // namespace

int PinnedWords::get(size_t need) {
    if (need <= kPinnedBlock) {
        std::lock_guard<std::mutex> hold(g_pinned_lock);
        if (g_pinned_count) block = g_pinned_idle[--g_pinned_count];
    }
    p = block.words;
    count = std::max(need, kPinnedBlock);
    // (behind the words the one that a signal is given by)
    if (!p && hipHostMalloc((void**)&p, (count + 1) * sizeof(long long), hipHostMallocPortable | hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        p = nullptr;
        epp_set_error("pinned host allocation failed");
        return EPP_ERR_ALLOC;
    }
    block.words = p;
    return EPP_OK;
}

PinnedWords::~PinnedWords() {
    if (!p) return;
    if (count == kPinnedBlock) {
        std::lock_guard<std::mutex> hold(g_pinned_lock);
        if (g_pinned_count < kIdlePinned) {
            g_pinned_idle[g_pinned_count++] = block;
            return;
        }
    }
    if (block.mark) (void)hipEventDestroy(block.mark);
    (void)hipHostFree(p);
}

PinnedWords::Signal PinnedWords::signal() {
    static std::atomic<long long> tickets{0};
    ticket = ++tickets;
    __atomic_store_n(p + count, 0ll, __ATOMIC_RELAXED);
    return Signal{p + count, ticket};
}

int PinnedWords::wait(hipStream_t s) {
    // (A hipStreamSynchronize soon after this would put such a mark on the stream itself, and wait for it: prepared and synchronised 41 us
    // without, 33 with it, 38 with hipStreamSynchronize in place of the signal.  Without it nothing is wrong.)
    int device = -1;
    if (hipGetDevice(&device) == hipSuccess && (!block.mark || block.device != device)) {
        if (block.mark) (void)hipEventDestroy(block.mark);
        block.device = device;
        if (hipEventCreateWithFlags(&block.mark, hipEventDisableTiming) != hipSuccess) block.mark = nullptr;
    }
    if (block.mark) (void)hipEventRecord(block.mark, s);
    (void)hipGetLastError();
    // (not for ever: after 10 ms, or where no kernel will raise it, the runtime says what the stream does)
    const auto end = std::chrono::steady_clock::now() + std::chrono::milliseconds(10);
    do {
        for (int i = 0; i < 64; ++i) {
            if (__atomic_load_n(p + count, __ATOMIC_ACQUIRE) == ticket) return EPP_OK;
            __builtin_ia32_pause();
        }
    } while (std::chrono::steady_clock::now() < end);
    const hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess && block.mark) {  // (it may be part of a capture that this ended)
        (void)hipEventDestroy(block.mark);
        block.mark = nullptr;
    }
    EPP_HIP_TRY(e);
    return EPP_OK;
}

size_t epp_scan_tmp_bytes(int64_t n) { return scan_tmp_bytes(n); }
void epp_scan_exclusive(const int* in, int* out, int64_t n, long long* total, int* tmp, hipStream_t s) {
    scan_counts(in, out, n, total, tmp, s);
}

void epp_path_set_stats(epp_path* p, const unsigned long long* host) {
    for (int c = 0; c < EPP_NCLASS; ++c) p->len_hist[c] = (int64_t)host[c];
    int mx;
    std::memcpy(&mx, &host[EPP_NCLASS], sizeof(int));
    p->max_len = mx;
}

int epp_path_finish(epp_path* p, hipStream_t s) {
    DevBuf stats;
    EPP_TRY(stats.alloc((EPP_NCLASS + 1) * sizeof(unsigned long long), epp_alloc_of(p)));
    EPP_HIP_TRY(hipMemsetAsync(stats.p, 0, stats.bytes, s));
    if (p->n_rows > 0) {
        // canonical rows: the all-active graph counts its empty rows too
        const int32_t* ptr = p->all_rows ? p->full_rowptr.as<int32_t>() : p->rowptr.as<int32_t>();
        hipLaunchKernelGGL(k_len_hist, dim3(std::min(grid_for(p->n_rows, kBlock), kStatBlocks)), dim3(kBlock), 0, s, ptr,
                           p->n_rows, stats.as<unsigned long long>(),
                           reinterpret_cast<int*>(stats.as<unsigned long long>() + EPP_NCLASS));
        EPP_HIP_TRY(hipGetLastError());
    }
    unsigned long long host[EPP_NCLASS + 1];
    EPP_HIP_TRY(hipMemcpyAsync(host, stats.p, sizeof(host), hipMemcpyDeviceToHost, s));
    EPP_HIP_TRY(hipStreamSynchronize(s));
    epp_path_set_stats(p, host);
    if (p->n_stream_rows > 0) {
        hipLaunchKernelGGL(k_mark_row_ends, dim3(grid_for(p->n_stream_rows, kBlock)), dim3(kBlock), 0, s,
                           p->rowptr.as<int32_t>(), p->n_stream_rows, p->cv.as<int2>());
        EPP_HIP_TRY(hipGetLastError());
    }
    return EPP_OK;  // the callers synchronise once, before they return the handle
}

extern "C" int epp_prepare(const epp_csr_t* g, const int32_t* train_ids, int64_t n_train, int L,
                           const epp_alloc_t* alloc, epp_stream_t stream, epp_paths_t** out) {
    if (!out) { epp_set_error("out is NULL"); return EPP_ERR_INVALID_ARG; }
    *out = nullptr;
    EPP_TRY(validate_csr(g));
    if (L < 1) { epp_set_error("L must be >= 1 (got %d)", L); return EPP_ERR_INVALID_ARG; }
    if (n_train < 0 || (n_train > 0 && !train_ids)) { epp_set_error("bad training set"); return EPP_ERR_INVALID_ARG; }
    hipStream_t s = (hipStream_t)stream;
    {   // set-up of this GPU's static scratch array (used by epp_weight_gradient_static)
        float* unused = nullptr;
        EPP_TRY(epp_static_scratch(&unused));
    }
    // small graphs: one launch builds everything (EPP_TUNE_SMALL_PREPARE=0 forces the general construction)
    if (epp_prepare_small_fits(g, n_train, L)) {
        const char* e = std::getenv("EPP_TUNE_SMALL_PREPARE");
        if (!(e && e[0] == '0')) return epp_prepare_small(g, train_ids, n_train, L, alloc, s, out);
    }
    const int64_t n = g->n, nnz = g->nnz;
    if (n == 0 && nnz > 0) return input_error(kErrCol, n);
    const int64_t n_words = (n + 63) / 64;
    const int64_t n_seg = (nnz + 63) / 64;
    const unsigned edge_tiles = grid_for(n_seg, kSegsPerTile);
    const unsigned word_tiles = grid_for(n_words, kWordsPerTile);
    const unsigned row_tiles = grid_for(n, kBlock);

    // pinned words: the numbers of the level being built, then every level's statistics
    PinnedWords hs;
    EPP_TRY(hs.get(kLevelWords + (size_t)L * kStatWords));
    epp_paths* P = new epp_paths();
    struct Guard {  // (on an error: nothing may still be writing to what is given back)
        epp_paths* p;
        hipStream_t s;
        ~Guard() {
            if (!p) return;
            (void)hipStreamSynchronize(s);
            delete p;
        }
    } guard{P, s};
    P->L = L;
    P->n = n;
    if (alloc && alloc->alloc && alloc->free) P->alloc = *alloc;
    const epp_alloc_t* al = epp_alloc_of(P);
    P->bitmaps.resize(L + 1);
    P->set_size.assign(L + 1, 0);
    P->path.assign(L, nullptr);
    // bitmaps of all sets, the ids of N^0 (at most one per training id) and what the levels count in one allocation
    const size_t bm_bytes = (size_t)n_words * 8;
    const size_t set0_bytes = (size_t)std::min(n_train, n) * 4;
    const size_t level_bytes = DevArena::rounded((size_t)L * ((kLevelWords + kRowCopies * kStatWords) * 8 + kLongHeadBytes));
    EPP_TRY(P->store.alloc((size_t)(L + 1) * DevArena::rounded(bm_bytes) + DevArena::rounded(set0_bytes) + level_bytes, al));
    for (int k = 0; k <= L; ++k) P->bitmaps[k].view(P->store.as<char>() + (size_t)k * DevArena::rounded(bm_bytes), bm_bytes);
    void* set0 = P->store.as<char>() + (size_t)(L + 1) * DevArena::rounded(bm_bytes);

    // all temporaries of the construction come from one allocation
    // (keep-mask, its counts and the members before every 256 vertices three times: the entries of a level are extracted
    // once the next level has shown whether the two paths share them, and then wait for the next extraction)
    constexpr int kAlive = 3;
    DevBuf mask[kAlive], seg_off[kAlive], tile_base[kAlive], folded, tile_cnt, row_cnt, row_base[kAlive], scan_tmp, newptr, tile_row;
    const size_t cnt_bytes = (size_t)std::max(std::max(edge_tiles, word_tiles), 1u) * 4;
    const size_t row_bytes = (size_t)std::max(row_tiles, 1u) * 4;
    const size_t tmp_bytes = scan_tmp_bytes(std::max<int64_t>(edge_tiles, row_tiles));
    DevArena arena;
    EPP_TRY(arena.reserve(kAlive * (DevArena::rounded((size_t)n_seg * 8) + DevArena::rounded((size_t)n_seg * 2) +
                                    DevArena::rounded(cnt_bytes) + DevArena::rounded(row_bytes)) +
                          DevArena::rounded(kFoldedWords * 4) + 2 * DevArena::rounded(cnt_bytes) + DevArena::rounded(row_bytes) + DevArena::rounded(tmp_bytes) +
                          DevArena::rounded((size_t)(n + 1) * 4), al));
    for (int i = 0; i < kAlive; ++i) {
        arena.take(&mask[i], (size_t)n_seg * 8);
        arena.take(&seg_off[i], (size_t)n_seg * 2);
        arena.take(&tile_base[i], cnt_bytes);
        arena.take(&row_base[i], row_bytes);
    }
    arena.take(&folded, kFoldedWords * 4);
    arena.take(&newptr, (size_t)(n + 1) * 4);
    arena.take(&tile_cnt, cnt_bytes);
    arena.take(&row_cnt, row_bytes);
    arena.take(&scan_tmp, tmp_bytes);
    arena.take(&tile_row, cnt_bytes);
    long long* const d_levels = reinterpret_cast<long long*>(static_cast<char*>(set0) + DevArena::rounded(set0_bytes));
    unsigned long long* const d_stats = reinterpret_cast<unsigned long long*>(d_levels + (size_t)L * kLevelWords);
    char* const d_long = reinterpret_cast<char*>(d_stats + (size_t)L * kRowCopies * kStatWords);

    // N^0 = V_t (Property 1) and its ascending ids (the other sets are the row ids of the paths)
    EPP_TRY(launch_training_set(train_ids, n_train, n, P->bitmaps[0], set0, tile_cnt.as<int>(), tile_base[0].as<int>(),
                                scan_tmp.as<int>(), d_levels + 5, reinterpret_cast<int*>(d_levels + 2), d_levels, level_bytes, s));
    EPP_HIP_TRY(hipGetLastError());

    // Shared entries: the path of a level runs on the arrays of the next level's path if nearly
    // all of that path's entries are its own too (the extra entries are skipped one by one at
    // run time, so the inner layer pays for them; EPP_TUNE_SHARE_PCT, default 95, 0: never).
    // A level's entries are therefore extracted only when the next level's count is known: not
    // at all if it shares them, and the outer path's extraction marks the entries that are not
    // the inner path's.  Every other level at most: a path whose marks serve an inner path
    // keeps its own arrays.
    std::vector<epp_path*> built;  // in level order, for the statistics
    struct Waiting { epp_path* p = nullptr; int level = 0; };
    Waiting pending;  // path whose entries are not extracted yet
    Waiting due;      // .. and have arrays of their own for certain: the next extraction takes them along
    auto kept_of = [&](int slot) {
        return Kept{mask[slot].as<unsigned long long>(), seg_off[slot].as<uint16_t>(), tile_base[slot].as<int>()};
    };
    auto extracted = [&](const Waiting& w) {
        const int slot = w.level % kAlive;
        return Extracted{kept_of(slot), Members{P->bitmaps[w.level + 1].as<unsigned long long>(), row_base[slot].as<int>()},
                         w.p->rowptr.as<int>(), (int)w.p->n_rows, (int)w.p->nnz, w.p->cv.as<int2>()};
    };
    unsigned long long* const h_stats = reinterpret_cast<unsigned long long*>(hs.p) + kLevelWords;
    auto extract = [&](epp_path* q, int level, bool marks_inner, bool last) -> int {
        // the entries in an allocation of their own (it can be given back once every prepared width
        // runs on a reconstructed copy)
        EPP_TRY(q->cv.alloc((size_t)q->nnz * sizeof(int2), al));
        if (marks_inner) EPP_TRY(q->inner_pos.alloc((size_t)((q->nnz + 63) / 64) * 4, al));
        if (due.p) EPP_TRY(due.p->cv.alloc((size_t)due.p->nnz * sizeof(int2), al));
        if (edge_tiles) {
            const Extracted a = extracted(Waiting{q, level});
            const Kept inner = marks_inner ? kept_of((level + kAlive - 1) % kAlive) : Kept{nullptr, nullptr, nullptr};
            if (due.p)
                hipLaunchKernelGGL(k_edge_extract<true>, dim3(edge_tiles), dim3(kBlock), 0, s, g->col, g->val, n_seg, a, inner,
                                   q->inner_pos.as<int>(), extracted(due), tile_row.as<int>(), (int)n, d_stats, last ? L : 0, h_stats);
            else
                hipLaunchKernelGGL(k_edge_extract<false>, dim3(edge_tiles), dim3(kBlock), 0, s, g->col, g->val, n_seg, a, inner,
                                   q->inner_pos.as<int>(), a, tile_row.as<int>(), (int)n, d_stats, last ? L : 0, h_stats);
        }
        due = Waiting{};
        EPP_HIP_TRY(hipGetLastError());
        return EPP_OK;
    };
    const long long share_pct = env_share_pct();
    bool nested = false;  // N^{k-1} lies in N^k
    for (int k = 0; k < L; ++k) {
        const int l = L - 1 - k;  // rows N^{k+1} = N^{L-l}, sources N^k = N^{L-l-1}
        const int slot = k % kAlive;
        epp_path* p = new epp_path();
        P->path[l] = p;
        built.push_back(p);
        p->n = n;
        p->alloc = P->alloc;
        p->pool = &P->pool;
        p->rows_pool = &P->rows_pool;
        p->sources = P->bitmaps[k].as<unsigned long long>();
        long long* d_level = d_levels + (size_t)k * kLevelWords;
        if (edge_tiles) {
            const bool all = k > 0 && P->set_size[k] == n;
            launch_edge_mask(g, n_seg, edge_tiles, P->bitmaps[k].as<unsigned int>(),
                             k > 0 && nested ? mask[(k + kAlive - 1) % kAlive].as<unsigned long long>() : nullptr, all, k == 0,
                             (double)(k > 0 ? P->set_size[k] : std::min(n_train, n)) / (double)n,
                             k > 0 && nested ? (double)built[k - 1]->nnz / (double)nnz : 0.0, folded.as<unsigned int>(),
                             mask[slot].as<unsigned long long>(), seg_off[slot].as<uint16_t>(), tile_cnt.as<int>(),
                             reinterpret_cast<int*>(d_level + 2), s);
            scan_counts(tile_cnt.as<int>(), tile_base[slot].as<int>(), (int64_t)edge_tiles, d_level, scan_tmp.as<int>(), s);
        }
        if (n > 0) {
            hipLaunchKernelGGL(k_row_flags, dim3(row_tiles), dim3(kBlock), 0, s, g->rowptr, n, nnz, kept_of(slot), d_level,
                               newptr.as<int>(), P->bitmaps[k].as<unsigned long long>(),
                               P->bitmaps[k + 1].as<unsigned long long>(), row_cnt.as<int>(),
                               k == 0 ? tile_row.as<int>() : (int*)nullptr);
            scan_counts(row_cnt.as<int>(), row_base[slot].as<int>(), (int64_t)row_tiles, d_level + 1, scan_tmp.as<int>(), s, d_level,
                        hs.p);
        } else {
            EPP_HIP_TRY(hipMemcpyAsync(hs.p, d_level, kLevelWords * sizeof(long long), hipMemcpyDeviceToHost, s));
        }
        EPP_HIP_TRY(hipGetLastError());
        EPP_HIP_TRY(hipStreamSynchronize(s));
        if (hs.p[2] & kErrTrain) {
            epp_set_error("training id outside [0, %lld)", (long long)n);
            return EPP_ERR_OUT_OF_RANGE_ID;
        }
        if (hs.p[2] != 0) return input_error((int)hs.p[2], n);
        if (k == 0) {
            P->set_size[0] = hs.p[5];
            P->set0_ids.view(set0, (size_t)hs.p[5] * 4);
        }
        const long long kept = hs.p[0], R = hs.p[1];
        const bool next_nested = hs.p[3] == 0, fixed_point = hs.p[4] == 0;
        p->n_src = P->set_size[k];
        p->nnz = kept;
        p->n_rows = R;
        p->n_stream_rows = R;  // every row of a path has at least one entry
        P->set_size[k + 1] = R;
        EPP_TRY(alloc_rows(p, d_long + (size_t)k * kLongHeadBytes, al));
        if (n > 0) {
            hipLaunchKernelGGL(k_rows_compact, dim3(std::min(row_tiles, kRowBlocks)), dim3(kBlock), 0, s,
                               P->bitmaps[k + 1].as<unsigned long long>(), n, row_base[slot].as<int>(), newptr.as<int>(),
                               p->row_ids.as<int32_t>(), p->rowptr.as<int32_t>(), (int64_t)R, (int)kept,
                               d_stats + (size_t)k * kRowCopies * kStatWords, p->long_rows);
            EPP_HIP_TRY(hipGetLastError());
        } else {
            EPP_HIP_TRY(hipMemsetAsync(p->rowptr.p, 0, sizeof(int32_t), s));
        }
        epp_path* q = pending.p;  // the path of the level before, if its entries still wait
        if (q && nested && share_pct > 0 && q->nnz > 0 && q->nnz * 100 >= kept * share_pct) {
            EPP_TRY(p->zero_block.alloc(256, al));
            EPP_HIP_TRY(hipMemsetAsync(p->zero_block.p, 0, 256, s));
            p->has_inner = true;
            q->outer = p;
            q->inner_rows = P->bitmaps[k].as<unsigned int>();  // its rows are N^k
            EPP_TRY(extract(p, k, true, k + 1 == L || fixed_point));
            pending.p = nullptr;
        } else {
            // (at most one is due: the next level extracts this one's entries, or its own that this one shares)
            if (q && due.p) EPP_TRY(extract(q, pending.level, false, false));
            else if (q) due = pending;
            pending = Waiting{p, k};
        }
        nested = next_nested;
        // Fixed point: N^{k+1} == N^k means every further set is the same set, so every deeper
        // layer (rows and sources both equal to it) has exactly this path; share it.
        if (k + 1 < L && fixed_point) {
            for (int j = k + 1; j < L; ++j) {
                EPP_HIP_TRY(hipMemcpyAsync(P->bitmaps[j + 1].p, P->bitmaps[k + 1].p, P->bitmaps[k + 1].bytes,
                                           hipMemcpyDeviceToDevice, s));
                P->set_size[j + 1] = P->set_size[k + 1];
                P->path[L - 1 - j] = p;
            }
            break;
        }
    }
    if (pending.p) EPP_TRY(extract(pending.p, pending.level, false, true));
    if (!edge_tiles) std::memset(h_stats, 0, (size_t)L * kStatWords * 8);  // (no entry, no row)
    EPP_HIP_TRY(hipStreamSynchronize(s));
    for (size_t k = 0; k < built.size(); ++k)
        epp_path_set_stats(built[k], h_stats + k * kStatWords);
    guard.p = nullptr;
    *out = P;
    return EPP_OK;
}

extern "C" int epp_prepare_full(const epp_csr_t* g, const epp_alloc_t* alloc, epp_stream_t stream,
                                epp_path_t** out) {
    if (!out) { epp_set_error("out is NULL"); return EPP_ERR_INVALID_ARG; }
    *out = nullptr;
    EPP_TRY(validate_csr(g));
    hipStream_t s = (hipStream_t)stream;
    epp_path* p = new epp_path();
    struct Guard { epp_path* p; ~Guard() { delete p; } } guard{p};
    p->n = g->n;
    p->n_rows = g->n;
    p->nnz = g->nnz;
    p->n_src = g->n;
    p->all_rows = true;
    if (alloc && alloc->alloc && alloc->free) p->alloc = *alloc;
    const epp_alloc_t* al = epp_alloc_of(p);
    EPP_TRY(p->full_rowptr.alloc((size_t)(g->n + 1) * 4, al));
    EPP_TRY(p->cv.alloc((size_t)g->nnz * sizeof(int2), al));
    {   // streamed form: the vertices with non-empty lists, ascending, with a compact row pointer
        PinnedWords hs;
        EPP_TRY(hs.get(64));
        DevBuf bitmap, tile_cnt, tile_base, dev_total, err;
        const int64_t n_words = (g->n + 63) / 64;
        const size_t tiles = std::max<size_t>(grid_for(n_words, kWordsPerTile), 1);
        DevArena arena;
        EPP_TRY(arena.reserve(DevArena::rounded((size_t)n_words * 8) + 2 * DevArena::rounded(tiles * 4) +
                              2 * DevArena::rounded(16), al));
        arena.take(&bitmap, (size_t)n_words * 8);
        arena.take(&tile_cnt, tiles * 4);
        arena.take(&tile_base, tiles * 4);
        arena.take(&dev_total, sizeof(long long));
        arena.take(&err, sizeof(int));
        // the caller's arrays are checked before anything is indexed with them
        EPP_HIP_TRY(hipMemsetAsync(err.p, 0, sizeof(int), s));
        if (g->n > 0)
            hipLaunchKernelGGL(k_check_rowptr, dim3(grid_for(g->n, kBlock)), dim3(kBlock), 0, s, g->rowptr, g->n, g->nnz,
                               err.as<int>());
        if (g->nnz > 0)
            hipLaunchKernelGGL(k_interleave, dim3(grid_for(g->nnz, kBlock)), dim3(kBlock), 0, s, g->col, g->val, g->nnz,
                               g->n, p->cv.as<int2>(), err.as<int>());
        EPP_HIP_TRY(hipGetLastError());
        EPP_HIP_TRY(hipMemcpyAsync(hs.p, err.p, sizeof(int), hipMemcpyDeviceToHost, s));
        EPP_HIP_TRY(hipStreamSynchronize(s));
        int herr;
        std::memcpy(&herr, hs.p, sizeof(int));
        if (g->n == 0 && g->nnz > 0) herr |= 2;
        if (herr) return input_error(herr, g->n);
        EPP_HIP_TRY(hipMemcpyAsync(p->full_rowptr.p, g->rowptr, (size_t)(g->n + 1) * 4, hipMemcpyDeviceToDevice, s));
        if (g->n > 0) {
            hipLaunchKernelGGL(k_nonempty_bitmap, dim3(grid_for(g->n, kBlock)), dim3(kBlock), 0, s, g->rowptr, g->n, 0,
                               bitmap.as<unsigned long long>());
            EPP_HIP_TRY(hipGetLastError());
        }
        EPP_TRY(compact_bitmap(bitmap, g->n, g->rowptr, (int)g->nnz, &p->row_ids, &p->rowptr, &p->n_stream_rows,
                               tile_cnt, tile_base, dev_total, hs, al, s));
        p->n_empty_rows = g->n - p->n_stream_rows;
        if (p->n_empty_rows == 0) {
            EPP_HIP_TRY(hipStreamSynchronize(s));
            p->row_ids.release();  // identity
        } else {
            hipLaunchKernelGGL(k_nonempty_bitmap, dim3(grid_for(g->n, kBlock)), dim3(kBlock), 0, s, g->rowptr, g->n, 1,
                               bitmap.as<unsigned long long>());
            EPP_HIP_TRY(hipGetLastError());
            int64_t cnt = 0;
            EPP_TRY(compact_bitmap(bitmap, g->n, nullptr, 0, &p->empty_rows, nullptr, &cnt, tile_cnt, tile_base,
                                   dev_total, hs, al, s));
            EPP_HIP_TRY(hipStreamSynchronize(s));
        }
    }
    EPP_TRY(epp_path_finish(p, s));
    EPP_HIP_TRY(hipStreamSynchronize(s));
    guard.p = nullptr;
    *out = p;
    return EPP_OK;
}

extern "C" int epp_paths_import(int64_t n, int L, const int32_t* train_ids, int64_t n_train,
                                const epp_path_arrays_t* layers, const epp_alloc_t* alloc, epp_stream_t stream,
                                epp_paths_t** out) {
    if (!out) { epp_set_error("out is NULL"); return EPP_ERR_INVALID_ARG; }
    *out = nullptr;
    if (L < 1 || !layers) { epp_set_error("L must be >= 1 and layers non-NULL"); return EPP_ERR_INVALID_ARG; }
    if (n < 0 || n_train < 0 || (n_train > 0 && !train_ids)) { epp_set_error("bad sizes"); return EPP_ERR_INVALID_ARG; }
    if (n >= kMaxVertices) { epp_set_error("graph too large: n=%lld (limit 2^29-1)", (long long)n); return EPP_ERR_TOO_LARGE; }
    for (int l = 0; l < L; ++l) {
        const epp_path_arrays_t& a = layers[l];
        if (a.n_rows < 0 || a.n_rows > n || a.nnz < 0 || !a.rowptr || (a.n_rows > 0 && !a.row_ids) ||
            (a.nnz > 0 && (!a.col || !a.val)) || (a.n_rows == 0 && a.nnz != 0)) {
            epp_set_error("layer %d: inconsistent sizes or NULL arrays", l);
            return EPP_ERR_INVALID_ARG;
        }
        if (a.nnz >= 0x7FFFFFFFll) { epp_set_error("layer %d: nnz=%lld (limit 2^31-1)", l, (long long)a.nnz); return EPP_ERR_TOO_LARGE; }
    }
    hipStream_t s = (hipStream_t)stream;
    {   // set-up of this GPU's static scratch array (used by epp_weight_gradient_static)
        float* unused = nullptr;
        EPP_TRY(epp_static_scratch(&unused));
    }
    const int64_t n_words = (n + 63) / 64;
    // words: [0] errors, [1] |N^0|, then every layer's statistics
    constexpr size_t kLayerWords = kImportCopies * kStatWords;
    const size_t res_words = 2 + (size_t)L * kLayerWords;
    PinnedWords hs;
    EPP_TRY(hs.get(res_words));
    epp_paths* P = new epp_paths();
    struct Guard {  // (on an error: nothing may still be writing to what is given back)
        epp_paths* p;
        hipStream_t s;
        ~Guard() {
            if (!p) return;
            (void)hipStreamSynchronize(s);
            delete p;
        }
    } guard{P, s};
    P->L = L;
    P->n = n;
    if (alloc && alloc->alloc && alloc->free) P->alloc = *alloc;
    const epp_alloc_t* al = epp_alloc_of(P);
    P->bitmaps.resize(L + 1);
    P->set_size.assign(L + 1, 0);
    P->path.assign(L, nullptr);
    // bitmaps (cleared), ids of N^0 (at most one per training id), results, counts of the long rows (cleared)
    const size_t bm_bytes = (size_t)n_words * 8, set0_bytes = (size_t)std::min(n_train, n) * 4;
    const size_t tiles = std::max<size_t>(grid_for(n_words, kWordsPerTile), 1);
    const size_t clear_bytes = (size_t)(L + 1) * DevArena::rounded(bm_bytes) + DevArena::rounded(res_words * 8 + (size_t)L * kLongHeadBytes);
    EPP_TRY(P->store.alloc(clear_bytes + DevArena::rounded(set0_bytes), al));
    for (int k = 0; k <= L; ++k) P->bitmaps[k].view(P->store.as<char>() + (size_t)k * DevArena::rounded(bm_bytes), bm_bytes);
    long long* d_res = reinterpret_cast<long long*>(P->store.as<char>() + (size_t)(L + 1) * DevArena::rounded(bm_bytes));
    char* const d_long = reinterpret_cast<char*>(d_res + res_words);
    void* set0 = P->store.as<char>() + clear_bytes;
    int* d_err = reinterpret_cast<int*>(d_res);
    DevArena arena;
    DevBuf tile_cnt, tile_base, scan_tmp;
    EPP_TRY(arena.reserve(2 * DevArena::rounded(tiles * 4) + DevArena::rounded(scan_tmp_bytes(tiles)), al));
    arena.take(&tile_cnt, tiles * 4);
    arena.take(&tile_base, tiles * 4);
    arena.take(&scan_tmp, scan_tmp_bytes(tiles));
    EPP_TRY(launch_training_set(train_ids, n_train, n, P->bitmaps[0], set0, tile_cnt.as<int>(), tile_base.as<int>(), scan_tmp.as<int>(),
                                d_res + 1, d_err, P->store.as<char>() + DevArena::rounded(bm_bytes),
                                clear_bytes - DevArena::rounded(bm_bytes), s));
    ImportPaths all;
    int held = 0;
    unsigned blocks = 0;
    for (int l = L - 1; l >= 0; --l) {
        const epp_path_arrays_t& a = layers[l];
        const int k = L - l - 1;
        epp_path* p = new epp_path();
        P->path[l] = p;
        p->n = n;
        p->alloc = P->alloc;
        p->pool = &P->pool;
        p->rows_pool = &P->rows_pool;
        p->sources = P->bitmaps[k].as<unsigned long long>();
        p->sources_checked = false;
        p->n_rows = p->n_stream_rows = a.n_rows;
        p->nnz = a.nnz;
        P->set_size[k + 1] = a.n_rows;
        // (the entries in an allocation of their own: see epp_prepare)
        EPP_TRY(alloc_rows(p, d_long + (size_t)l * kLongHeadBytes, al));
        EPP_TRY(p->cv.alloc((size_t)a.nnz * sizeof(int2), al));
        ImportArgs& q = all.path[held];
        q.row_ids = a.row_ids;
        q.rowptr = a.rowptr;
        q.col = a.col;
        q.val = a.val;
        q.n_rows = a.n_rows;
        q.nnz = a.nnz;
        q.n = n;
        q.ids_out = p->row_ids.as<int32_t>();
        q.ptr_out = p->rowptr.as<int32_t>();
        q.cv = p->cv.as<int2>();
        q.bitmap32 = P->bitmaps[k + 1].as<unsigned int>();
        q.stats = reinterpret_cast<unsigned long long*>(d_res + 2 + (size_t)l * kLayerWords);
        q.err = d_err;
        q.row_blocks = std::min(grid_for(a.n_rows + 1, kBlock), kStatBlocks);
        q.list = p->long_rows;
        blocks += q.row_blocks + grid_for(a.nnz, kImportTile);
        all.end[held++] = blocks;
        if (l > 0 && held < kImportPaths) continue;
        for (int i = held; i < kImportPaths; ++i) all.end[i] = blocks;
        hipLaunchKernelGGL(k_import_path, dim3(blocks), dim3(kBlock), 0, s, all);
        EPP_HIP_TRY(hipGetLastError());
        held = 0;
        blocks = 0;
    }
    EPP_HIP_TRY(hipMemcpyAsync(hs.p, d_res, res_words * 8, hipMemcpyDeviceToHost, s));
    EPP_HIP_TRY(hipStreamSynchronize(s));
    const int herr = (int)hs.p[0];
    if (herr & (kErrCol | kErrTrain)) { epp_set_error("an id lies outside [0, %lld)", (long long)n); return EPP_ERR_OUT_OF_RANGE_ID; }
    if (herr) { epp_set_error("path arrays are not in canonical form"); return EPP_ERR_INVALID_ARG; }
    P->set_size[0] = hs.p[1];
    P->set0_ids.view(set0, (size_t)hs.p[1] * 4);
    for (int l = 0; l < L; ++l) {
        P->path[l]->n_src = P->set_size[L - l - 1];
        const unsigned long long* const copies = reinterpret_cast<const unsigned long long*>(hs.p) + 2 + (size_t)l * kLayerWords;
        unsigned long long stats[kStatWords];
        for (int i = 0; i < kStatWords; ++i) stats[i] = stat_word<kImportCopies>(copies, i);
        epp_path_set_stats(P->path[l], stats);
    }
    guard.p = nullptr;
    *out = P;
    return EPP_OK;
}

int epp_check_sources(epp_path* p, hipStream_t s) {
    if (p->sources_checked || !p->sources || p->nnz == 0) return EPP_OK;
    PinnedWords host;
    DevBuf outside;
    EPP_TRY(host.get(1));
    EPP_TRY(outside.alloc(sizeof(int), epp_alloc_of(p)));
    EPP_HIP_TRY(hipMemsetAsync(outside.p, 0, sizeof(int), s));
    hipLaunchKernelGGL(k_columns_inside, dim3(grid_for(p->nnz, kBlock * kCheckPer)), dim3(kBlock), 0, s, p->cv.as<int2>(),
                       p->nnz, reinterpret_cast<const unsigned int*>(p->sources), outside.as<int>());
    EPP_HIP_TRY(hipGetLastError());
    host.p[0] = 0;
    EPP_HIP_TRY(hipMemcpyAsync(host.p, outside.p, sizeof(int), hipMemcpyDeviceToHost, s));
    EPP_HIP_TRY(hipStreamSynchronize(s));
    if (host.p[0] != 0) p->sources = nullptr;  // any row may be gathered
    p->sources_checked = true;
    return EPP_OK;
}

extern "C" int epp_num_layers(const epp_paths_t* p) {
    if (!p) { epp_set_error("paths is NULL"); return EPP_ERR_INVALID_ARG; }
    return p->L;
}

extern "C" epp_path_t* epp_get_path(epp_paths_t* p, int l) {
    if (!p || l < 0 || l >= p->L) { epp_set_error("no such layer"); return nullptr; }
    return p->path[l];
}

extern "C" int epp_path_export(const epp_path_t* p, int32_t* row_ids, int32_t* rowptr, int32_t* col, float* val,
                               epp_stream_t stream) {
    if (!p) { epp_set_error("path is NULL"); return EPP_ERR_INVALID_ARG; }
    hipStream_t s = (hipStream_t)stream;
    epp_path* o = p->outer ? p->outer : const_cast<epp_path*>(p);  // the path whose array holds the entries
    const bool entries = (col || val) && p->nnz > 0;
    if (entries) EPP_TRY(epp_ensure_canonical(o, s));
    const unsigned eb = entries ? grid_for(o->nnz, kBlock * kExportSegs) : 0;
    const unsigned rb = (row_ids || rowptr) ? grid_for(p->n_rows + 1, kBlock) : 0;
    if (eb + rb > 0) {
        const int32_t* ids = p->all_rows ? nullptr : p->row_ids.as<int32_t>();
        const int32_t* ptr = p->all_rows ? p->full_rowptr.as<int32_t>() : p->rowptr.as<int32_t>();
        if (p->outer)
            hipLaunchKernelGGL(k_export<true>, dim3(eb + rb), dim3(kBlock), 0, s, o->cv.as<int2>(), o->nnz,
                               o->inner_pos.as<int>(), p->nnz, eb, col, val, ids, ptr, p->n_rows, row_ids, rowptr);
        else
            hipLaunchKernelGGL(k_export<false>, dim3(eb + rb), dim3(kBlock), 0, s, o->cv.as<int2>(), o->nnz,
                               (const int*)nullptr, p->nnz, eb, col, val, ids, ptr, p->n_rows, row_ids, rowptr);
    }
    EPP_HIP_TRY(hipGetLastError());
    EPP_HIP_TRY(hipStreamSynchronize(s));
    // (an entry array that was rebuilt for this call only is given back again)
    epp_release_canonical_if_unused(p->outer ? p->outer : const_cast<epp_path*>(p));
    return EPP_OK;
}

extern "C" int epp_active_set_export(const epp_paths_t* p, int k, int32_t* ids, int64_t* count, epp_stream_t stream) {
    if (!p || !count) { epp_set_error("NULL argument"); return EPP_ERR_INVALID_ARG; }
    if (k < 0 || k > p->L) { epp_set_error("k=%d outside [0, %d]", k, p->L); return EPP_ERR_INVALID_ARG; }
    hipStream_t s = (hipStream_t)stream;
    if (!ids) { *count = p->set_size[k]; return EPP_OK; }
    if (*count < p->set_size[k]) {
        epp_set_error("ids buffer holds %lld entries, need %lld", (long long)*count, (long long)p->set_size[k]);
        return EPP_ERR_INVALID_ARG;
    }
    PinnedWords hs;
    EPP_TRY(hs.get(64));
    DevBuf tile_cnt, tile_base, dev_total, tmp;
    const size_t tiles = std::max<size_t>(grid_for((p->n + 63) / 64, kWordsPerTile), 1);
    const epp_alloc_t* al = epp_alloc_of(p);
    EPP_TRY(tile_cnt.alloc(tiles * 4, al));
    EPP_TRY(tile_base.alloc(tiles * 4, al));
    EPP_TRY(dev_total.alloc(sizeof(long long), al));
    int64_t c = 0;
    EPP_TRY(compact_bitmap(p->bitmaps[k], p->n, nullptr, 0, &tmp, nullptr, &c, tile_cnt, tile_base, dev_total, hs, al, s));
    if (c > 0) EPP_HIP_TRY(hipMemcpyAsync(ids, tmp.p, (size_t)c * 4, hipMemcpyDeviceToDevice, s));
    EPP_HIP_TRY(hipStreamSynchronize(s));
    *count = c;
    return EPP_OK;
}

int epp_active_ids(const epp_paths* p, int k, const int32_t** ids, int64_t* count) {
    if (k < 0 || k > p->L) { epp_set_error("k=%d outside [0, %d]", k, p->L); return EPP_ERR_INVALID_ARG; }
    *count = p->set_size[k];
    // N^k, k >= 1, is the row set of SG_{L-k}; N^0 was compacted when the handle was made
    *ids = k > 0 ? p->path[p->L - k]->row_ids.as<int32_t>() : p->set0_ids.as<int32_t>();
    return EPP_OK;
}

extern "C" void epp_destroy_paths(epp_paths_t* p) { delete p; }
extern "C" void epp_destroy_path(epp_path_t* p) { delete p; }
