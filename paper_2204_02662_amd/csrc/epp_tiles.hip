// Gather-reduce in source order: tiles of rows whose sums stay in LDS (Alg. 2, aggregation loop), for paths whose
// source rows do not fit the L2s.
//
// The group kernel (epp_aggregate.hip) takes entries row after row, so every XCD gathers from everywhere at any time and
// an L2 of 4 MB serves next to nothing (2.4 M sources, F = 64: 11 % of the lines); the rest runs at the 60 G lines/s
// that the fabric gives.  Here a wavefront owns a tile of 79 to 255 rows, whose sums lie in LDS, and takes the
// tile's entries in the order of their sources.  The 256 wavefronts of an XCD therefore sweep the source matrix
// together, and a source row that one of them has fetched is still in L2 when the others come to it.
//
//   * The rows are dealt to the tiles by length: tiles that run at the same time hold rows of nearly the same lengths, hence
//     as many entries each, and keep abreast by themselves (a sweep that falls behind finds its lines in L2 and
//     catches up).  It also puts the long rows into few tiles, which is where most entries share a sweep.  (2.4 M sources,
//     F = 64: rows dealt at random 4.4 ms a launch, by length 2.8.)
//   * A row of more than kSplitMax entries is cut into parts, each with every so-manieth kChunk entries, so that every
//     part spans all sources; the parts' sums go to an array that a second kernel adds up.
//   * 2^k lanes of 16 bytes read a source row's slice (a "slot"); a wavefront carries several slots, which share its
//     tile.  A tile's list is cut into batches of 64 entries, each sorted by row and dealt to the slots so that
//     one step of the wavefront never touches a row twice: then LDS is read, added to and written without atomics
//     (ds_add_f32 takes 190 cycles a wavefront here), in an order that depends on the path alone.
//   * Eight wavefronts of 159 rows fill a CU's LDS.  Sixteen of 79 drift apart (26 % instead of 46 % of the lines in
//     L2: 3.9 ms), four are bound by the instructions of one wavefront per SIMD.
//   * Wide rows are taken in slices, one after the other: the narrower the slice, the more rows fit LDS and the more sources L2,
//     at the price of reading the entries once per slice.

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "epp_internal.h"

namespace {

constexpr int kTileWaves = 8;            // wavefronts of a workgroup, which fills a CU's LDS
constexpr int kTilesAtOnce = 256 * kTileWaves;  // tiles of a generation, which run at the same time
constexpr int kSplitMax = 512;           // longest row that is not cut into parts (and a part's entries, at most)
constexpr int kPiece = 32;               // entries of a row (on average) that are added up before their sum is added to the row's
constexpr int kTileBins = 128;           // length classes by which rows are dealt
constexpr unsigned kTogether = 64;       // consecutive tiles that are prepared on one XCD
constexpr int kChunk = 4;                // entries of a cut row that stay together
constexpr int kBuckets = 1024;           // source ranges into which a tile's entries are sorted
constexpr int kRowsPerBlock = 1024, kListBlock = 256;
constexpr int kColBits = 23;             // of an entry's first word; then 8 bits row of the tile, 1 bit "not the inner path's"
constexpr unsigned kColMask23 = (1u << kColBits) - 1;

typedef int int2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));  // global accesses need no more

// LANES lanes of 16 bytes per slot: rows whose sums a wavefront keeps (one more takes what fills up a batch)
constexpr int tile_rows(int lanes) { return lanes == 4 ? 255 : lanes == 8 ? 159 : 79; }
// How a batch is taken, by its two bits of `care`: two steps at a time (0 turns), or one at a time in so many turns.
constexpr int care_turns(int lanes, unsigned care) {
    return lanes == 4 ? (care == 0 ? 1 : care == 1 ? 2 : care == 2 ? 4 : 16)
                      : (care == 0 ? 0 : care == 1 ? 1 : care == 2 ? 2 : 64 / lanes);
}
// entries of one row that it may hold
constexpr int care_limit(int lanes, unsigned care) {
    return care_turns(lanes, care) == 0 ? lanes / 2 : care_turns(lanes, care) * lanes;
}

// Steps that a wavefront makes one after the other for a batch, beyond those of a batch that needs no care.
constexpr int care_steps(int lanes, unsigned care) { return care_turns(lanes, care) == 0 ? lanes / 2 : lanes * care_turns(lanes, care); }
constexpr int care_delay(int lanes, unsigned care) { return care_steps(lanes, care) - care_steps(lanes, 0); }

int env_int(const char* name, int dflt) {
    const char* v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : dflt;
}

// Entries of part p of a row of `len` entries cut into `parts`: chunks p, p + parts, ..
__host__ __device__ inline int parts_of(int len, int split) { return len <= split ? 1 : (len + split - 1) / split; }
__host__ __device__ inline int part_len(int len, int parts, int p) {
    const int chunks = (len + kChunk - 1) / kChunk;
    const int mine = (chunks - p + parts - 1) / parts;
    return mine * kChunk - ((chunks - 1) % parts == p ? chunks * kChunk - len : 0);
}

// Length class, the longest rows first: exact up to 32 entries, then eight classes per octave.
__device__ __forceinline__ int tile_bin(int len) {
    const int e = 31 - __clz(len);
    const int up = len < 32 ? len : 32 + (e - 5) * 8 + ((len >> (e - 3)) & 7);
    return kTileBins - 1 - min(up, kTileBins - 1);
}

// ------------------------------------------------------------------------------------------ preparation
// Sums over the lanes up to this one (data moves between lanes without LDS).
__device__ __forceinline__ int sum_up_to_lane(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return x;
}

// A workgroup takes kRowsPerBlock consecutive rows, a wavefront a quarter of them, 64 at a time: f(row's first entry,
// its entries, its parts (0: no row), its vertex's index r) by every lane.
template <class F>
__device__ __forceinline__ void for_block_rows(const int32_t* __restrict__ rowptr, int64_t n_rows, int split, F f) {
    constexpr int kPerWave = kRowsPerBlock / (kListBlock / 64);
    const int64_t base = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6) * kPerWave + (threadIdx.x & 63);
    for (int i = 0; i < kPerWave; i += 64) {
        const int64_t r = base + i;
        const int begin = r < n_rows ? rowptr[r] : 0, len = r < n_rows ? rowptr[r + 1] - begin : 0;
        f(begin, len, len > 0 ? parts_of(len, split) : 0, r);
    }
}

// f(entries, part, ..) for the parts of every lane's row, by its wavefront where they are many; `begin`, `parts` and `to`
// are handed on as the row's lane has them.
template <class F>
__device__ __forceinline__ void for_parts(int len, int parts, int begin, int to, F f) {
    for (int p = 0; p < (parts > 8 ? 0 : parts); ++p) f(part_len(len, parts, p), p, begin, parts, to);
    for (unsigned long long todo = __ballot(parts > 8); todo; todo &= todo - 1ull) {
        const int l = __ffsll((long long)todo) - 1;
        const int its_len = __shfl(len, l, 64), its_parts = __shfl(parts, l, 64);
        const int its_begin = __shfl(begin, l, 64), its_to = __shfl(to, l, 64);
        for (int p = (int)(threadIdx.x & 63); p < its_parts; p += 64)
            f(part_len(its_len, its_parts, p), p, its_begin, its_parts, its_to);
    }
}

// What the order of the ids will do to the batches of k_tile_sort: *delay is the sum of care_delay over kOrderSamples batches, each
// that of a random entry.  Every workgroup counts 8,192 random entries per range of the sources (whole lines of 16), so that it knows
// which ranges fill a batch of a tile between them.  A lane of one wavefront then draws an entry and looks up how many of its row (or part of
// one) lie in the entry's batch, if all rows of the tile are as long.  Batches hold several rows, of which the one with the most
// entries counts, so this is somewhat less than what the sort finds (mean delay, sort / sampled, 8 lanes: narrow band 60 / 59, communities
// 58 / 48 and 6.5 / 3.0, by degree 12.3 / 10.4 and 4.0 / 3.0, random order 0.07 / 0.01).  Bound by latency, 35 to 40 us.
constexpr int kOrderBlocks = 256, kOrderThreads = 1024, kOrderReads = 8;
constexpr int kOrderSamples = kOrderBlocks * 64;  // (a wavefront each: more of them on a CU would wait for its address units)
__host__ __device__ inline bool too_slow(unsigned delay, double max_delay) { return (double)delay > max_delay * kOrderSamples; }
__device__ __forceinline__ unsigned scrambled(unsigned x) {
    x = (x ^ (x >> 16)) * 0x7FEB352Du;
    x = (x ^ (x >> 15)) * 0x846CA68Bu;
    return x ^ (x >> 16);
}
template <int LANES>
__global__ __launch_bounds__(kOrderThreads) void k_tile_order(const int2v* __restrict__ cv, int64_t nnz, const int32_t* __restrict__ rowptr,
                                                              int64_t n_rows, int split, int shift, unsigned int* __restrict__ delay) {
    static_assert(kBuckets == kOrderThreads, "a thread per range");
    __shared__ int before[kBuckets], wave_sum[kOrderThreads / 64];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    before[t] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kOrderReads; ++i) {
        const unsigned x = scrambled((blockIdx.x * kOrderReads + i) * (kOrderThreads / 16) + (t >> 4));
        const int64_t e = (int64_t)(((unsigned long long)x * (unsigned long long)nnz) >> 32);
        atomicAdd(&before[(cv[std::min<int64_t>((e & ~15ll) + (t & 15), nnz - 1)].x & kEntCol) >> shift], 1);
    }
    __syncthreads();
    const int mine = before[t], incl = sum_up_to_lane(mine);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int sum = incl - mine;
    for (int w = 0; w < wave; ++w) sum += wave_sum[w];
    before[t] = sum;
    __syncthreads();
    if (wave > 0) return;
    const unsigned x = scrambled(0x80000000u | (blockIdx.x * 64 + t));
    const int64_t e = (int64_t)(((unsigned long long)x * (unsigned long long)nnz) >> 32);
    int64_t lo = 0, hi = n_rows;  // the last row that begins at or before entry e
    while (hi - lo > 1) {
        const int64_t step = std::max<int64_t>((hi - lo) / 8, 1);
        int past = 0;
#pragma unroll
        for (int i = 1; i < 8; ++i) past += lo + i * step < hi && rowptr[std::min(lo + i * step, hi - 1)] <= e;
        if (past < 7) hi = std::min(hi, lo + (past + 1) * step);
        lo += past * step;
    }
    const int begin = rowptr[lo], len = rowptr[lo + 1] - begin, parts = parts_of(len, split), at = (int)e - begin;
    const int part = at / kChunk % parts, m = part_len(len, parts, part), here = at / kChunk / parts * kChunk + at % kChunk;
    // batch of the part's entry k, if a tile's rows all have m entries
    const float batches = (float)(tile_rows(LANES) * m) / (64.0f * kOrderThreads * kOrderReads);
    auto batch_of = [&](int k) {
        const int col = cv[begin + part * kChunk + k / kChunk * parts * kChunk + k % kChunk].x & kEntCol;
        return (int)((float)before[col >> shift] * batches);
    };
    const int batch = batch_of(here);
    int first = 0, top = here, low = here + 1, end = m;  // [first, top] and [low, end] hold the ends of its entries of that batch
    while (first < top || low < end) {
        const int mid0 = (first + top) >> 1, mid1 = (low + end) >> 1;
        const int b0 = batch_of(min(mid0, m - 1)), b1 = batch_of(min(mid1, m - 1));
        if (first < top) {
            if (b0 < batch) first = mid0 + 1; else top = mid0;
        }
        if (low < end) {
            if (b1 <= batch) low = mid1 + 1; else end = mid1;
        }
    }
    const int most = end - first;
    int steps = 0;
#pragma unroll
    for (unsigned c = 0; c < 3; ++c)
        if (most > care_limit(LANES, c)) steps = care_delay(LANES, c + 1);
    steps = sum_up_to_lane(steps);
    if (lane == 63 && steps) atomicAdd(delay, (unsigned)steps);
}

// Rows (parts of cut rows counted one by one) per length class, of every workgroup; totals: rows, parts of cut rows,
// cut rows; then the delay of k_tile_order, with which nothing is done if it is too long.
__global__ __launch_bounds__(kListBlock) void k_tile_count(const int32_t* __restrict__ rowptr, int64_t n_rows, int split,
                                                           unsigned int* __restrict__ block_hist,
                                                           unsigned int* __restrict__ totals, double max_delay) {
    if (too_slow(totals[3], max_delay)) return;
    __shared__ unsigned int h[kTileBins], t[3];
    if (threadIdx.x < kTileBins) h[threadIdx.x] = 0;
    if (threadIdx.x < 3) t[threadIdx.x] = 0;
    __syncthreads();
    for_block_rows(rowptr, n_rows, split, [&](int, int len, int parts, int64_t) {
        for_parts(len, parts, 0, 0, [&](int m, int, int, int, int) { atomicAdd(&h[tile_bin(m)], 1u); });
        if (parts > 0) atomicAdd(&t[0], (unsigned)parts);
        if (parts > 1) {
            atomicAdd(&t[1], (unsigned)parts);
            atomicAdd(&t[2], 1u);
        }
    });
    __syncthreads();
    if (threadIdx.x < kTileBins) block_hist[blockIdx.x * kTileBins + threadIdx.x] = h[threadIdx.x];
    if (threadIdx.x < 3 && t[threadIdx.x]) atomicAdd(&totals[threadIdx.x], t[threadIdx.x]);
}

// A workgroup per class: the class's rows before every workgroup of k_tile_count, and in all of them.
__global__ __launch_bounds__(256) void k_tile_classes(unsigned int* __restrict__ block_hist, int n_blocks,
                                                      unsigned int* __restrict__ hist,
                                                      const unsigned int* __restrict__ totals, double max_delay) {
    if (too_slow(totals[3], max_delay)) return;
    __shared__ unsigned int wave_sum[4];
    const int bin = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned before = 0;
    for (int b0 = 0; b0 < n_blocks; b0 += 256) {
        const int b = b0 + (int)threadIdx.x;
        const unsigned x = b < n_blocks ? block_hist[b * kTileBins + bin] : 0u;
        const unsigned incl = (unsigned)sum_up_to_lane((int)x);
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        unsigned mine = before + incl - x;
        for (int w = 0; w < 4; ++w) {
            if (w < wave) mine += wave_sum[w];
            before += wave_sum[w];
        }
        if (b < n_blocks) block_hist[b * kTileBins + bin] = mine;
        __syncthreads();
    }
    if (threadIdx.x == 0) hist[bin] = before;
}

struct TileBins { unsigned first[kTileBins]; };  // rank of the first row of every class
struct CutRow { int v, first, count; };          // vertex, its first part's place and their number
// Of a rank: the row's first entry (-1: no row), which of its parts, where its sum goes, parts << 10 | entries of this one.
struct Dealt { int first, part, target, parts_len; };

// Rank of a tile's row.
__device__ __forceinline__ int64_t dealt_at(int tile, int local, int tile_rows, int at_once) {
    const int gen = tile / at_once;
    return ((int64_t)gen * tile_rows + local) * at_once + (tile - gen * at_once);
}

// Deals the rows: rank k goes to tile k % at_once of its generation, so that the ranks of a tile lie at_once apart.
// Within a class rows are ranked in their order (a wavefront counts its own; lanes that add to one counter are served in
// their order), so that two handles of one path run the same additions.  Only where the parts' sums lie depends on timing.
__global__ __launch_bounds__(kListBlock) void k_tile_deal(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ row_ids,
                                                          int64_t n_rows, int split, int n, TileBins bins,
                                                          const unsigned int* __restrict__ block_hist,
                                                          unsigned int* __restrict__ places,  // [0] parts, [1] cut rows
                                                          Dealt* __restrict__ dealt, CutRow* __restrict__ cut) {
    constexpr int kWaves = kListBlock / 64;
    __shared__ unsigned int h[kWaves][kTileBins], t[2], place[2];
    for (int i = threadIdx.x; i < kWaves * kTileBins; i += kListBlock) h[i / kTileBins][i % kTileBins] = 0;
    if (threadIdx.x < 2) t[threadIdx.x] = 0;
    __syncthreads();
    unsigned int* __restrict__ mine = h[threadIdx.x >> 6];
    for_block_rows(rowptr, n_rows, split, [&](int, int len, int parts, int64_t) {
        for_parts(len, parts, 0, 0, [&](int m, int, int, int, int) { atomicAdd(&mine[tile_bin(m)], 1u); });
        if (parts > 1) { atomicAdd(&t[0], (unsigned)parts); atomicAdd(&t[1], 1u); }
    });
    __syncthreads();
    // (one place in each list for all of the workgroup's parts and cut rows together)
    if (threadIdx.x < kTileBins) {
        unsigned rank = bins.first[threadIdx.x] + block_hist[blockIdx.x * kTileBins + threadIdx.x];
        for (int w = 0; w < kWaves; ++w) {
            const unsigned m = h[w][threadIdx.x];
            h[w][threadIdx.x] = rank;
            rank += m;
        }
    }
    if (threadIdx.x < 2) {
        place[threadIdx.x] = t[threadIdx.x] ? atomicAdd(&places[threadIdx.x], t[threadIdx.x]) : 0u;
        t[threadIdx.x] = 0;
    }
    __syncthreads();
    for_block_rows(rowptr, n_rows, split, [&](int begin, int len, int parts, int64_t r) {
        int to = len > 0 ? (row_ids ? row_ids[r] : (int)r) : 0;
        if (parts > 1) {
            const int first = (int)(place[0] + atomicAdd(&t[0], (unsigned)parts));
            cut[place[1] + atomicAdd(&t[1], 1u)] = CutRow{to, first, parts};
            to = n + first;
        }
        for_parts(len, parts, begin, to, [&](int m, int p, int its_begin, int its_parts, int its_to) {
            dealt[atomicAdd(&mine[tile_bin(m)], 1u)] = Dealt{its_begin, p, its_to + p, its_parts << 10 | m};
        });
    });
}

// Batches of 64 entries per tile.
__global__ __launch_bounds__(64) void k_tile_sizes(const Dealt* __restrict__ dealt, int tile_rows, int at_once, int n_tiles,
                                                   int* __restrict__ batches) {
    const int tile = (int)(blockIdx.x * 64 + threadIdx.x);
    if (tile >= n_tiles) return;
    const int64_t first = dealt_at(tile, 0, tile_rows, at_once);
    int sum = 0;
#pragma unroll 8
    for (int i = 0; i < tile_rows; ++i) {
        const Dealt r = dealt[first + (int64_t)i * at_once];
        sum += r.first < 0 ? 0 : r.parts_len & 1023;
    }
    batches[tile] = (sum + 63) / 64;
}

// One workgroup per tile: its entries into the order of their sources (kBuckets ranges of them), then into batches.
//
// A tile of at most kSortMax entries is read once, into registers; a larger one is counted first, then taken in rounds,
// each a range of the sources.  A wavefront takes its share of the rows 64 entries at a time and counts for itself; lanes that
// add to one counter are served in their order.  A range's entries are therefore in the order of the rows, whatever the
// timing, and so are the additions of a launch.  The entries that fill up the last batch have weight zero and a row of
// their own.
//
// A batch's 64 entries are sorted by row and dealt to (step, slot): place i goes to step i % steps of slot i / steps.
// Two entries of one row then share a step only if the row has more than `steps` entries in the batch; they lie fewer
// than t slots apart if it has at most t * steps, and then a step is safe in t turns, of every t-th slot each.  Two steps
// half as many apart share no row if none has more than half as many entries.  The launch learns from two bits of
// `care` how it has to take the batch.
//
// *bad is set where that cannot be done: more than kSortMax entries of a tile in one range, or, in a tile that takes more
// than one round, columns that do not ascend along a row.  Workgroups that start after that do nothing.
constexpr int kSortThreads = 512, kSortWaves = kSortThreads / 64;
constexpr int kSortMax = 5632;
constexpr int kSortPer = (kSortMax / kSortWaves + kSplitMax - 1 + 63) / 64;  // entries per lane: a wavefront's share and all of one row but one

// Of a row (part): its first entry, from one chunk of it to the next, its entries, and the (negative) number of the
// round's entries before it less those of it that are already taken.
struct TileRow { int first, step, len, before; };

__device__ __forceinline__ int tile_entry(const TileRow& r, int k) {
    return r.first + (int)((unsigned)k / kChunk) * r.step + (int)((unsigned)k % kChunk);
}

template <int LANES>
__global__ __launch_bounds__(kSortThreads, 4) void k_tile_sort(const int2v* __restrict__ cv, const Dealt* __restrict__ dealt, int at_once,
                                                               const int32_t* __restrict__ first_batch, int fine_shift,
                                                               int32_t* __restrict__ target, int* __restrict__ longest,
                                                               int2v* __restrict__ ent, unsigned int* __restrict__ care,
                                                               int* __restrict__ bad) {
    constexpr int kRows = tile_rows(LANES);
    static_assert(kRows < 256 && kRows < kSortThreads && kRows % 4 == 3, "");
    __shared__ int2v buf[kSortMax + 64];
    // entries per range: of the round and of two wavefronts a word, 16 bits each, then their places; of the tile, up to the range's end
    __shared__ unsigned count[kSortWaves / 2][kBuckets];
    __shared__ int upto[kBuckets];
    __shared__ TileRow row_of[kRows];
    __shared__ int from[kRows], start[kRows + 1];    // first entry of the round, its place among the round's entries
    __shared__ int wave_sum[kSortWaves];
    __shared__ int row_count_all[kSortWaves][256];
    __shared__ int stop;
    // (consecutive tiles hold the parts of one row and read the same lines: kTogether of them run on one XCD)
    const unsigned turn = blockIdx.x >> 3;
    const int tile = (int)(((turn / kTogether) * 8 + (blockIdx.x & 7)) * kTogether + turn % kTogether);
    const int b0 = first_batch[tile];
    const int t = (int)threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if (t == 0) stop = __hip_atomic_load(bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    TileRow mine = {0, kChunk, 0, 0};
    if (t < kRows) {
        const Dealt r = dealt[dealt_at(tile, t, kRows, at_once)];
        if (r.first >= 0) mine = TileRow{r.first + r.part * kChunk, (r.parts_len >> 10) * kChunk, r.parts_len & 1023, 0};
        target[(size_t)tile * kRows + t] = r.target;
        if (t == 0) longest[tile] = mine.len;  // (about: a tile's first row is of its highest length class)
    }
    // sums of x over the threads before this one and over all
    auto scan = [&](int x, int& total) {
        const int incl = sum_up_to_lane(x);
        __syncthreads();  // (wave_sum may still be read)
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        int before = incl - x;
        total = 0;
        for (int w = 0; w < kSortWaves; ++w) {
            if (w < wave) before += wave_sum[w];
            total += wave_sum[w];
        }
        total = __builtin_amdgcn_readfirstlane(total);
        return before;
    };
    // the row of the round's entry `pos`: the last one that starts at or before it and is not empty
    auto row_at = [&](int pos) {  // (a fixed number of steps, so that several searches run side by side)
        int at = 0;
#pragma unroll
        for (int step = 128; step > 0; step >>= 1) {
            if (at + step < kRows && start[at + step] <= pos) at += step;
        }
        return at;
    };
    int all;
    {
        const int before = scan(mine.len, all);
        mine.before = -before;
        if (t < kRows) { start[t] = before; from[t] = 0; row_of[t] = mine; }
        if (t == 0) start[kRows] = all;
    }
    __syncthreads();
    if (stop || all == 0) return;  // (its places have no rows)
    const bool whole = all <= kSortMax;
    // fewer and larger ranges where a batch spans several of them anyway
    int buckets = kBuckets, shift = fine_shift;
    while (buckets > 256 && buckets > all / 8) { buckets /= 2; ++shift; }
    const int per = max(buckets / kSortThreads, 1), mine0 = min(t * per, buckets), mine1 = min(mine0 + per, buckets);
    if (!whole) {
        for (int i = t; i < buckets; i += kSortThreads) upto[i] = 0;
        __syncthreads();
        constexpr int kAtOnce = 8;  // (with one search and load after the other the kernel took 15 % more)
        for (int pos0 = t; pos0 < all; pos0 += kAtOnce * kSortThreads) {
            int col[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                const int pos = min(pos0 + i * kSortThreads, all - 1);
                const TileRow row = row_of[row_at(pos)];
                col[i] = cv[tile_entry(row, pos + row.before)].x & kEntCol;
            }
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i)
                if (pos0 + i * kSortThreads < all) atomicAdd(&upto[col[i] >> shift], 1);
        }
        __syncthreads();
        int sum = 0, total;
#pragma unroll 1
        for (int i = mine0; i < mine1; ++i) sum += upto[i];
        int before = scan(sum, total);
#pragma unroll 1
        for (int i = mine0; i < mine1; ++i) { before += upto[i]; upto[i] = before; }
        __syncthreads();
    }
    int lo_bucket = 0, carry = 0, done = b0;  // (the same in all threads)
    while (true) {
        int hi_bucket = buckets;
        if (!whole) {  // as many ranges as fit
            const int limit = (lo_bucket ? upto[lo_bucket - 1] : 0) + kSortMax;
            int lo = lo_bucket, hi = buckets;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (upto[mid] <= limit) lo = mid + 1; else hi = mid;
            }
            hi_bucket = __builtin_amdgcn_readfirstlane(lo);
            if (hi_bucket == lo_bucket) {
                if (t == 0) atomicOr(bad, 1);
                return;
            }
        }
        const bool last = hi_bucket == buckets;
        int begin = 0, end = mine.len;
        if (!whole && t < kRows) {
            begin = from[t];
            if (!last) {
                int lo = begin;
                while (lo < end) {
                    const int mid = (lo + end) >> 1;
                    if (((cv[tile_entry(mine, mid)].x & kEntCol) >> shift) < hi_bucket) lo = mid + 1; else end = mid;
                }
            }
        }
        int here;
        {
            const int before = scan(t < kRows ? end - begin : 0, here);
            if (t < kRows) { start[t] = before; row_of[t].before = begin - before; }
            if (t == 0) start[kRows] = here;
        }
        for (int i = t; i < buckets; i += kSortThreads) {
            for (int w = 0; w < kSortWaves / 2; ++w) count[w][i] = 0;
        }
        __syncthreads();
        if (here > kSortMax) {  // (rows that do not ascend)
            if (t == 0) atomicOr(bad, 1);
            return;
        }
        // the wavefront's rows: those that start in its share of the places
        const int share = (here + kSortWaves - 1) / kSortWaves;
        auto first_place = [&](int w) {  // of the first row that starts at or after place w * share
            int lo = 0, hi = kRows;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (start[mid] < w * share) lo = mid + 1; else hi = mid;
            }
            return __builtin_amdgcn_readfirstlane(lo);
        };
        const int r0 = first_place(wave), r1 = wave == kSortWaves - 1 ? kRows : first_place(wave + 1);
        const int p0 = __builtin_amdgcn_readfirstlane(start[r0]), p1 = __builtin_amdgcn_readfirstlane(start[r1]);
        unsigned* __restrict__ my_count = count[wave >> 1];
        const int half = (wave & 1) * 16;
        int2v e[kSortPer];
        int at[kSortPer];  // row, then (also) the place inside the range
#pragma unroll
        for (int i = 0; i < kSortPer; ++i) {
            const int pos = p0 + i * 64 + lane;
            e[i] = int2v{0, 0};
            at[i] = 0;
            if (p0 + i * 64 < p1) {
                const int r = row_at(min(pos, p1 - 1));
                at[i] = r;
                const TileRow row = row_of[r];
                e[i] = cv[tile_entry(row, min(pos, p1 - 1) + row.before)];
            }
        }
        bool out_of_range = false;
#pragma unroll
        for (int i = 0; i < kSortPer; ++i) {
            if (p0 + i * 64 < p1) {
                const bool valid = p0 + i * 64 + lane < p1;
                const int bucket = (e[i].x & kEntCol) >> shift;
                if (!whole) out_of_range |= bucket < lo_bucket || bucket >= hi_bucket;
                unsigned place = 0;
                if (valid) place = atomicAdd(&my_count[bucket], 1u << half);
                at[i] = (at[i] << 16) | (int)((place >> half) & 0xFFFFu);
            }
        }
        if (out_of_range) atomicOr(bad, 1);
        __syncthreads();
        {
            int sum = 0, total;
#pragma unroll 1
            for (int i = mine0; i < mine1; ++i) {
                for (int w = 0; w < kSortWaves / 2; ++w) sum += (int)((count[w][i] & 0xFFFFu) + (count[w][i] >> 16));
            }
            unsigned before = (unsigned)(scan(sum, total) + carry);
#pragma unroll 1
            for (int i = mine0; i < mine1; ++i) {  // a range's entries in the order of the wavefronts
                for (int w = 0; w < kSortWaves / 2; ++w) {
                    const unsigned c = count[w][i], odd = before + (c & 0xFFFFu);
                    count[w][i] = before | odd << 16;
                    before = odd + (c >> 16);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSortPer; ++i) {
            if (p0 + i * 64 + lane < p1) {
                int x = e[i].x;
                asm volatile("" : "+v"(x));  // (formed again: columns and ranges kept since above would not fit the registers)
                const unsigned col = (unsigned)(x & kEntCol);
                buf[((my_count[col >> shift] >> half) & 0xFFFFu) + (at[i] & 0xFFFF)] =
                    int2v{(int)(col | ((unsigned)(at[i] >> 16) << kColBits) | (x & kEntOuterOnly ? 0x80000000u : 0u)), e[i].y};
            }
        }
        const int filled = carry + here;
        const int batches = last ? (filled + 63) / 64 : filled / 64;
        if (last && t < 64 && filled + t < batches * 64) {
            const int2v any = cv[tile_entry(row_of[0], 0)];  // (a source that the launch reads anyway)
            buf[filled + t] = int2v{(int)((unsigned)(any.x & kEntCol) | ((unsigned)kRows << kColBits) |
                                          (any.x & kEntOuterOnly ? 0x80000000u : 0u)), 0};
        }
        __syncthreads();
        for (int i = wave; i < batches; i += kSortWaves) {
            const int2v x = buf[i * 64 + lane];
            const unsigned row = ((unsigned)x.x >> kColBits) & 255u;
            // entries per row, their places, and how many of its own row are before an entry
            int* __restrict__ n_of = row_count_all[wave];
            int4* __restrict__ quad = reinterpret_cast<int4*>(n_of) + lane;
            __builtin_amdgcn_wave_barrier();
            *quad = int4{0, 0, 0, 0};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int before = atomicAdd(&n_of[row], 1);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int4 n = *quad;
            int most = max(max(n.x, n.y), n.z);
            if (lane * 4 + 3 != kRows) most = max(most, n.w);
            const int sum = n.x + n.y + n.z + n.w;
            const int first = sum_up_to_lane(sum) - sum;
            *quad = int4{first, first + n.x, first + n.x + n.y, first + n.x + n.y + n.z};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int place = n_of[row] + before;
            unsigned level = 0;
#pragma unroll
            for (unsigned c = 0; c < 3; ++c)
                if (__ballot(most > care_limit(LANES, c))) level = c + 1;
            const int b = done + i;
            if (level && lane == 0) atomicOr(&care[b >> 4], level << (2 * (b & 15)));
            __builtin_nontemporal_store(x, ent + (int64_t)b * 64 + place);
        }
        if (last) return;
        done += batches;
        carry = filled - batches * 64;
        lo_bucket = hi_bucket;
        const int2v rest = t < carry ? buf[batches * 64 + t] : int2v{0, 0};
        __syncthreads();
        if (t < carry) buf[t] = rest;
        if (t < kRows) from[t] = end;
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------ launch
struct TileArgs {
    const int2v* ent;
    const int32_t* first_batch;   // per tile, then their number
    const unsigned int* care;     // two bits per batch (k_tile_sort)
    const int32_t* target;        // per row of a tile: vertex, n + place of a part's sum, or -1
    const int* longest;           // per tile: entries of its rows, about at most
    const float* in;
    float* out;
    float* parts;                 // sums of the cut rows' parts, F floats each
    unsigned records;             // bytes from a slice's first row to the end of its last one
    int n, F;
    int lanes;                    // of a slot that hold part of a slice
    int ld;                       // floats from one row of `in` to the next
    int64_t slice_step;           // and from one slice of a row to the next
    int blocks;                   // workgroups per slice
    const float* zero;            // launch for the inner path that shares the arrays: 256 zero bytes
    const unsigned int* inner_rows;
};

constexpr unsigned kNowhere = 0xFFFFFF00u;  // place of a source row that is not there: behind all that are
constexpr int kRawBuffer = 0x00020000;      // a buffer of bytes, loads behind whose end give zero

// Copies the source rows slice by slice: all rows of the first slice, `stride` quadruples apart, of which `q` are used
// (zeros behind F), then those of the next.  Rows that are not in the bitmap `sources` (NULL: all are) are left
// out.  One workgroup per word of the bitmap.
__global__ __launch_bounds__(kListBlock) void k_pack_slices(const float* __restrict__ in, int64_t n, int F, int q, int stride,
                                                            int slices, const unsigned long long* __restrict__ sources,
                                                            float* __restrict__ out) {
    const unsigned long long mine = sources ? sources[blockIdx.x] : ~0ull;
    if (!mine) return;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int rows = (int)std::min<int64_t>(n - r0, 64);
    for (int s = 0; s < slices; ++s) {
        float4v* __restrict__ dst = reinterpret_cast<float4v*>(out) + ((int64_t)s * n + r0) * stride;
        for (int i = threadIdx.x; i < rows * q; i += kListBlock) {
            const int r = i / q, k = i - r * q, f = (s * q + k) * 4;
            if (!((mine >> r) & 1)) continue;
            const float* __restrict__ x = in + (r0 + r) * F + f;
            float4v v = {0.0f, 0.0f, 0.0f, 0.0f};
            if (f + 4 <= F) {
                v = *reinterpret_cast<const float4u*>(x);
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (f + c < F) v[c] = x[c];
            }
            dst[r * stride + k] = v;
        }
    }
}

// A wavefront per tile and slice.  Where the sources' lines miss L2, these bound it (2.4 M sources, 140 M entries, F = 64: 93 G
// lines/s, half of which miss; the group kernel's launch takes 4620 us, this one 3080), and the further a wavefront runs ahead, the
// less it finds there; where they hit, it waits for latency.  So its gathers go out AHEAD pairs of steps (of kSlots entries each) before
// their additions, in a window that rolls over the batches (2 batches of 4 lanes), or, AHEAD = 0, a batch at a time.  tile_ahead
// has the rule and the figures.
//
// What is formed per entry is what a step cannot share: the lanes of a slot hold its entries' weights and the places of their source
// rows and sums, and the additions take them from there by DPP; the gathers are buffer loads with a 32-bit offset.  (Formed by every
// lane for itself, with 64-bit addresses, a batch of 64 entries and 16 lanes a slot was 280 instructions instead of 206; 114 M entries,
// 233 K sources, F = 41: 1390 -> 1310 us.)  FAR: rows that lie further apart than such an offset reaches.
//
// A sum is formed in LDS over a part of the sweep at a time, and those sums in registers, where a lane has those of the rows that it
// will write.  A part holds kPiece entries of a row whose sources lie anywhere; the rounding error then grows like that of a sum of
// 32 + 16 terms, not of 512: over 20 all-active launches (both models, ids in random order, 22 to 288 M entries, F = 16 to 128) it is
// 0.63 to 0.89 of the group kernel's against 64 bits.  A row whose sources all lie in one part is one chain of up to kSplitMax, 0.99 to
// 1.6 of it; paths of such rows stay on the group table (k_tile_order).  Adding up in LDS alone would be no faster (within 3 %, the
// spread of the runs).
template <int LANES, int AHEAD, bool INNER, bool FAR>
__global__ __launch_bounds__(kTileWaves * 64, 2) void k_aggregate_tiles(TileArgs a) {
    constexpr int kRows = tile_rows(LANES), kSlots = 64 / LANES, kSteps = LANES;
    constexpr int kPairs = kSteps / 2;
    constexpr int kTakes = LANES == 4 ? 2 : 1;  // batches in flight
    static_assert(AHEAD == (LANES == 4 ? kTakes * kPairs : AHEAD) && AHEAD <= kTakes * kPairs, "a step's registers are those that it frees");
    constexpr unsigned kNoRow = FAR ? ~0u : kNowhere;
    constexpr int kShares = LANES == 8 ? 2 : 1;  // entries of a batch that a lane holds
    typedef __attribute__((address_space(1))) const float4u* gvec_ptr;
    __shared__ float4v sums_all[kTileWaves][(kRows + 1) * LANES];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int slot = lane / LANES, l = lane % LANES;
    const int slice = blockIdx.x / a.blocks;
    const int tile = (blockIdx.x - slice * a.blocks) * kTileWaves + wave;
    float4v* __restrict__ sums = sums_all[wave];
    const int f = l < a.lanes ? (slice * a.lanes + l) * 4 : a.F;  // (a lane without a share reads its neighbour's)
    const int b0 = a.first_batch[tile], b1 = a.first_batch[tile + 1];
    if (b0 == b1) return;  // (its places have no rows; nothing below waits for another wavefront)
    for (int i = lane; i < (kRows + 1) * LANES; i += 64) sums[i] = float4v{};
    const float* __restrict__ src = a.in + slice * a.slice_step;
    const unsigned ld = (unsigned)a.ld * (FAR ? 1u : 4u), share = (unsigned)min(l, a.lanes - 1) * (FAR ? 4u : 16u);
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(src), 0, (int)a.records, kRawBuffer);
    // (8 lanes: the entries of steps 0 to 3, then of 4 to 7, in each of a slot's two quads)
    const int2v* __restrict__ ent = a.ent + (int64_t)b0 * 64 + (LANES == 8 ? slot * 8 + (l & 3) : lane);
    const int last = b1 - b0 - 1, pieces = min((a.longest[tile] + kPiece - 1) / kPiece, last + 1);
    // Entries and their two bits of `care` are loaded one batch before they are used.  (Behind the end the last batch is gathered
    // again, from L2.)
    struct Entries { int2v e[kShares]; };
    auto entries = [&](int b) {
        Entries x;
#pragma unroll
        for (int i = 0; i < kShares; ++i) x.e[i] = __builtin_nontemporal_load(ent + min(b, last) * 64 + i * 4);
        return x;
    };
    auto cares = [&](int b) { return a.care[(b0 + min(b, last)) >> 4]; };
    // Of a batch in flight: what its gathers give, and of the entries that a lane holds the weight and the place of the row's sum.
    struct Shares { float w[kShares]; int at[kShares]; };
    struct { float4u x[kSteps]; Shares own; unsigned care; } flight[kTakes];
    unsigned place[kShares];  // and of the source row, of the batch that is being gathered
    Entries ahead = entries(0);
    auto put = [&](int b, Shares& own) {  // the entries of batch b, and loads those of the next
        const Entries here = ahead;
        ahead = entries(b + 1);
        __builtin_amdgcn_sched_barrier(0);  // (before the gathers that come next, so that waiting for it is not waiting for them)
#pragma unroll
        for (int i = 0; i < kShares; ++i) {
            const int x = here.e[i].x;
            own.at[i] = (int)(((unsigned)x >> kColBits) & 255u) * LANES * 16;
            own.w[i] = __int_as_float(here.e[i].y);
            place[i] = __umul24((unsigned)x & kColMask23, ld);
            if constexpr (INNER) {
                if (x < 0) { place[i] = kNoRow; own.w[i] = 0.0f; }
            }
        }
    };
    // Step j's value of a lane's slot: one of the slot's lanes has it, and an addition or a product takes it from there.  (Handed
    // on through LDS, as the words of an entry were at first, entries took a place there that rows can use, and 2 to 9 % of a launch.)
    auto of_step = [&](auto J, const auto (&v)[kShares]) {
        constexpr int j = decltype(J)::value;
        const int x = __builtin_bit_cast(int, v[LANES == 8 ? j >> 2 : 0]);
        int y;
        if constexpr (LANES == 16) y = __builtin_amdgcn_update_dpp(0, x, 0x150 + j, 0xF, 0xF, true);  // row_newbcast:j
        else y = __builtin_amdgcn_update_dpp(0, x, (j & 3) * 0x55, 0xF, 0xF, true);                   // quad_perm:[j,j,j,j]
        return __builtin_bit_cast(std::remove_const_t<std::remove_reference_t<decltype(v[0])>>, y);
    };
    auto gather = [&](auto& fl, auto J) {
        const unsigned at = of_step(J, place);
        if constexpr (FAR) {
            gvec_ptr p = (gvec_ptr)(src + (at + share));  // (32 bits: the number of vertices times ld is below 2^32)
            if constexpr (INNER) p = at == kNoRow ? (gvec_ptr)(a.zero + l * 4) : p;
            fl.x[J] = *p;
        } else {
            fl.x[J] = __builtin_bit_cast(float4u, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)(at + share), 0, 0));
        }
    };
    // (always in this order: the wait for one gather is then not for another that was made later)
    auto gather_two = [&](auto& fl, auto J, auto K) {
        gather(fl, J);
        __builtin_amdgcn_sched_barrier(0x7);  // (arithmetic may cross)
        gather(fl, K);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto sum_at = [&](auto& fl, auto J) {
        return reinterpret_cast<float4v*>(reinterpret_cast<char*>(sums) + (of_step(J, fl.own.at) + l * 16));
    };
    auto plus = [&](auto& fl, auto J, float4v& sum) {
        const float w = of_step(J, fl.own.w);
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = fmaf(w, fl.x[J][i], sum[i]);
    };
    auto for_steps = [&](auto f) {  // for the first half of them, a constant each, and that of the other half
        auto g = [&](auto J) { f(J, std::integral_constant<int, decltype(J)::value + kSteps / 2>{}); };
        g(std::integral_constant<int, 0>{});
        g(std::integral_constant<int, 1>{});
        if constexpr (kSteps >= 8) { g(std::integral_constant<int, 2>{}); g(std::integral_constant<int, 3>{}); }
        if constexpr (kSteps >= 16) {
            g(std::integral_constant<int, 4>{});
            g(std::integral_constant<int, 5>{});
            g(std::integral_constant<int, 6>{});
            g(std::integral_constant<int, 7>{});
        }
    };
    auto take = [&](int b, auto& fl) {
        const unsigned how = __builtin_amdgcn_readfirstlane(fl.care >> (2 * ((b0 + b) & 15))) & 3u;
        fl.care = cares(b + kTakes);
        Shares next;  // of the batch whose gathers go out meanwhile
        if constexpr (AHEAD == 0) {
            put(b, fl.own);
            for_steps([&](auto J, auto K) {
                gather(fl, J);
                gather(fl, K);
            });
        }
        auto refill = [&](auto J) {  // (the gathers go to registers that the additions have freed)
            if constexpr (AHEAD > 0) {
                constexpr int j = decltype(J)::value + AHEAD, q = j % kPairs;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (q == 0) put(b + kTakes, next);
                gather_two(fl, std::integral_constant<int, q>{}, std::integral_constant<int, q + kPairs>{});
            }
        };
        const int turns = how == 0 ? 1 : how == 1 ? care_turns(LANES, 1) : how == 2 ? care_turns(LANES, 2) : care_turns(LANES, 3);
        const int mine = slot & (turns - 1);
        auto in_turns = [&](auto J) {
            float4v* const p = sum_at(fl, J);
            const float w = of_step(J, fl.own.w);
            for (int t = 0; t < turns; ++t) {
                if (mine == t) {
                    float4v sum = *p;
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[i] = fmaf(w, fl.x[J][i], sum[i]);
                    *p = sum;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        };
        // (in LDS a wavefront's operations execute in order)
        auto add_two = [&](auto J, auto K) {
            float4v* const p0 = sum_at(fl, J);
            float4v* const p1 = sum_at(fl, K);
            float4v s0 = *p0;
            if constexpr (care_turns(LANES, 0) == 1) {
                plus(fl, J, s0);
                *p0 = s0;
                float4v s1 = *p1;
                plus(fl, K, s1);
                *p1 = s1;
            } else {
                float4v s1 = *p1;
                plus(fl, J, s0);
                plus(fl, K, s1);
                *p0 = s0;
                *p1 = s1;
            }
        };
        if constexpr (AHEAD > 0) {  // (one order of loads whichever way a batch is taken: the waits count them)
            for_steps([&](auto J, auto K) {
                if (how == 0) {
                    add_two(J, K);
                } else {
                    in_turns(J);
                    in_turns(K);
                }
                refill(J);
            });
        } else if (how == 0) {
            for_steps([&](auto J, auto K) { add_two(J, K); });
        } else {
            for_steps([&](auto J, auto K) {
                in_turns(J);
                in_turns(K);
            });
        }
        if constexpr (AHEAD > 0) fl.own = next;
    };
#pragma unroll
    for (int d = 0; d < kTakes; ++d) {
        flight[d].care = cares(d);
        if constexpr (AHEAD > 0) {
            put(d, flight[d].own);
            for_steps([&](auto J, auto K) {
                if constexpr (decltype(J)::value < AHEAD) gather_two(flight[d], J, K);
            });
        }
    }
    constexpr int kOwn = (kRows + 1) / kSlots;
    static_assert(kOwn * kSlots == kRows + 1, "");
    float4v whole[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) whole[i] = float4v{};
    int b = 0;
    for (int piece = 1; piece <= pieces; ++piece) {
        const int upto = (int)((int64_t)(last + 1) * piece / pieces);
        for (; b < upto; b += kTakes) {
#pragma unroll
            for (int d = 0; d < kTakes; ++d)
                if (d == 0 || b + d <= last) take(b + d, flight[d]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            whole[i] += sums[lane + i * 64];
            sums[lane + i * 64] = float4v{};
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    // (all places are looked up at once: one after the other they would hold the sweep up)
    int to[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int r = slot + i * kSlots;
        to[i] = a.target[(size_t)tile * kRows + min(r, kRows - 1)];
        if (r >= kRows || f >= a.F) to[i] = -1;
    }
    if constexpr (INNER) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i)
            if (to[i] >= 0 && to[i] < a.n && !((a.inner_rows[to[i] >> 5] >> (to[i] & 31)) & 1u)) to[i] = -1;
    }
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        if (to[i] < 0) continue;
        float* __restrict__ o = to[i] < a.n ? a.out + (size_t)to[i] * (size_t)a.F : a.parts + (size_t)(to[i] - a.n) * (size_t)a.F;
        if (f + 4 <= a.F) {
            __builtin_nontemporal_store((float4u)whole[i], reinterpret_cast<float4u*>(o + f));
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                if (f + c < a.F) o[f + c] = whole[i][c];
        }
    }
}

// out[v, :] = sum of the parts of a cut row, in their order: 2^log2T lanes of 16 bytes a row, four loads in flight.
// A row with more than kFewSums of them is left to a wavefront, whose teams of lanes take every so-manieth one and
// exchange their sums between lanes, one with more than kManySums to the whole workgroup.  Bound by memory: 2.9 M sums of
// 128 floats in 278 us.
constexpr int kFewSums = 16, kManySums = 256;
__global__ __launch_bounds__(kListBlock) void k_tile_add_parts(const CutRow* __restrict__ cut, int n_cut, int F, int log2T,
                                                               const float* __restrict__ parts,
                                                               const unsigned int* __restrict__ only_bits,
                                                               float* __restrict__ out) {
    constexpr int kWaves = kListBlock / 64;
    __shared__ CutRow list[kListBlock];
    __shared__ int n_long;
    __shared__ float4v sum_of[kWaves][64];
    const int T = 1 << log2T, lane = threadIdx.x & (T - 1), wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) n_long = 0;
    __syncthreads();
    const int at = (int)((blockIdx.x * kListBlock + threadIdx.x) >> log2T);
    if (at < n_cut) {
        const CutRow c = cut[at];
        if (only_bits && !((only_bits[c.v >> 5] >> (c.v & 31)) & 1u)) {
            // not a row of the inner path
        } else if (c.count > kFewSums) {
            if (lane == 0) list[atomicAdd(&n_long, 1)] = c;
        } else {
            for (int f0 = lane * 4; f0 < F; f0 += T * 4) {
                const int f = min(f0, F - 4);
                const float* __restrict__ x0 = parts + (size_t)c.first * F + f;
                float4u s = *reinterpret_cast<const float4u*>(x0);
                for (int p = 1; p < c.count; p += 4) {
                    float4u x[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const float4u*>(x0 + (size_t)min(p + i, c.count - 1) * F);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (p + i < c.count) s += x[i];
                }
                *reinterpret_cast<float4u*>(out + (size_t)c.v * F + f) = s;
            }
        }
    }
    __syncthreads();
    const int longs = n_long;
    for (int i = 0; i < longs; ++i) {
        const CutRow c = list[i];
        const bool all = c.count > kManySums;
        if (!all && (i & (kWaves - 1)) != wave) continue;
        const int team = (all ? (int)threadIdx.x : (int)(threadIdx.x & 63)) >> log2T, teams = (all ? kListBlock : 64) >> log2T;
        for (int base = 0; base < F; base += T * 4) {
            const int f0 = base + lane * 4, f = min(f0, F - 4);
            float4u s = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int p = team; p < c.count; p += 8 * teams) {
                float4u x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    x[j] = *reinterpret_cast<const float4u*>(parts + (size_t)(c.first + min(p + j * teams, c.count - 1)) * F + f);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (p + j * teams < c.count) s += x[j];
            }
            for (int d = T; d < 64; d <<= 1) {
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] += __shfl_xor(s[j], d, 64);
            }
            if (all) {  // (the same for every wavefront, like the barriers below)
                sum_of[wave][threadIdx.x & 63] = s;
                __syncthreads();
                if (wave == 0) {
                    for (int w = 1; w < kWaves; ++w) s += sum_of[w][lane];
                }
                __syncthreads();  // `sum_of` is written again
            }
            if (team == 0 && f0 < F) *reinterpret_cast<float4u*>(out + (size_t)c.v * F + f) = s;
        }
    }
}

struct TileShape { int slices, quads, stride; bool packed; };

unsigned blocks_for(int64_t items, int per) { return (unsigned)((items + per - 1) / per); }

template <int LANES>
void sort_tiles(TilePlan* q, const int2v* cv, const Dealt* dealt, int shift, int* bad, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_sort<LANES>, dim3((unsigned)q->n_tiles), dim3(kSortThreads), 0, s, cv, dealt, q->at_once,
                       q->first_batch, shift, q->target, q->longest, reinterpret_cast<int2v*>(q->ent), q->care, bad);
}

template <int LANES>
void sample_order(const epp_path* p, int split, int shift, unsigned int* delay, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_order<LANES>, dim3(kOrderBlocks), dim3(kOrderThreads), 0, s, reinterpret_cast<const int2v*>(p->cv.p), p->nnz,
                       p->rowptr.as<int32_t>(), p->n_stream_rows, split, shift, delay);
}

template <int LANES, int AHEAD>
void launch_tiles(const TileArgs& a, int slices, hipStream_t s) {
    const dim3 grid((unsigned)(a.blocks * slices)), block(kTileWaves * 64);
    const bool far = a.records == 0;
    if (a.zero) {
        if (far) hipLaunchKernelGGL((k_aggregate_tiles<LANES, AHEAD, true, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_aggregate_tiles<LANES, AHEAD, true, false>), grid, block, 0, s, a);
    } else {
        if (far) hipLaunchKernelGGL((k_aggregate_tiles<LANES, AHEAD, false, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_aggregate_tiles<LANES, AHEAD, false, false>), grid, block, 0, s, a);
    }
}

}  // namespace

// How launches take rows of F floats: slices of `quads` quadruples, which lie `stride` quadruples apart where the rows
// are copied first.  A slice should touch as few 128-byte lines as it can fill, so that all is copied that does not
// lie that way already (F = 24, 274 M entries, 2.4 M sources: 2687 us copied, 4251 read across the lines' ends).
static TileShape tile_shape(int F, int lanes) {
    const int quads = (F + 3) / 4;
    TileShape t;
    t.slices = (quads + lanes - 1) / lanes;
    t.quads = (quads + t.slices - 1) / t.slices;
    t.stride = 1;
    while (t.stride < t.quads) t.stride *= 2;
    if (t.stride == 16 && t.quads <= 12) t.stride = 12;  // (two lines either way)
    t.packed = F % 4 != 0 || t.slices * t.quads != quads || t.quads != t.stride;
    return t;
}

size_t epp_tile_packed_bytes(const epp_path* p, int F, int lanes) {
    const TileShape t = tile_shape(F, lanes);
    return t.packed ? (size_t)p->n * t.slices * t.stride * 16 : 0;
}

// ------------------------------------------------------------------------------------------------ which paths
// What a launch costs is estimated from how often each source is referenced, and that from the row-length classes, as
// if the sources were referenced as unequally as the rows are long (on a symmetric graph they are).
struct Sources {
    int classes = 0;
    double count[EPP_NCLASS], share[EPP_NCLASS];  // sources; part of all references that goes to one of them
    double rows[EPP_NCLASS], len[EPP_NCLASS];     // rows and their mean length, the longest first
    explicit Sources(const epp_path* p) {
        double all = 0.0;
        const double per_row = (double)p->n_src / (double)std::max<int64_t>(p->n_stream_rows, 1);
        for (int c = EPP_NCLASS - 1; c >= 0; --c) {
            const double r = (double)(p->len_hist[c] - (c == 0 ? p->n_empty_rows : 0));
            if (r <= 0.0) continue;
            rows[classes] = r;
            len[classes] = c == 0 ? 1.0 : 0.72 * (double)(1ll << c);
            all += r * len[classes++];
        }
        for (int i = 0; i < classes; ++i) {
            count[i] = rows[i] * per_row;
            share[i] = len[i] / (all * per_row);
            len[i] *= (double)p->nnz / all;
        }
    }
    // groups of `per` sources that so many references touch
    double touched(double references, double per) const {
        double d = 0.0;
        for (int i = 0; i < classes; ++i) d -= count[i] / per * std::expm1(-share[i] * per * references);
        return d;
    }
    // references that a cache of so many sources serves, the least recently used one giving way
    double cached(double sources) const {
        double all = 0.0, lo = 0.0, hi = 60.0, hit = 0.0;  // (octaves of references between two uses)
        for (int i = 0; i < classes; ++i) all += count[i];
        if (all <= sources) return 1.0;
        for (int i = 0; i < 16; ++i) {
            const double mid = 0.5 * (lo + hi);
            (touched(std::exp2(mid), 1.0) < sources ? lo : hi) = mid;
        }
        for (int i = 0; i < classes; ++i) hit -= count[i] * share[i] * std::expm1(-share[i] * std::exp2(lo));
        return hit;
    }
};

constexpr double kLinesOfL2 = 32768.0;

// Microseconds of a launch on the group table (or its partitioned copy).
static double group_launch_us(const epp_path* p, const Sources& src, int F) {
    double best = 1e30;
    const int packed = F <= 16 ? std::max(8, F > 8 ? 16 : 8) : (F + 15) / 16 * 16;
    for (const int ld : {F, packed}) {
        if (ld == packed && best < 1e30 && packed == F) break;
        const double lines = epp_lines_per_row(F, ld), hit = src.cached(kLinesOfL2 / lines);
        const double copy = ld == F ? 0.0 : 4.0 * (double)p->n * (F + ld) * 2.5e-7;
        best = std::min(best, 1e-6 * (double)p->nnz * (3.8 + lines * (3.0 * hit + 12.8 * (1.0 - hit))) + copy);
    }
    return 16.0 + best + 1e-6 * (double)p->n_stream_rows * (16.0 + 0.66 * F);
}

// .. and on tiles of so many lanes a slot.
struct Sweeps { double count, missed; };  // and the source rows' lines that they fetch from beyond L2, a line a row
static Sweeps tile_sweeps(const Sources& src, int lanes, double per_line) {
    const double capacity = (double)kTilesAtOnce * tile_rows(lanes);
    // the longest rows first: each XCD touches the sources of an eighth of a sweep's entries
    Sweeps s = {0.0, 0.0};
    double room = capacity, entries = 0.0;
    auto sweep = [&] {
        s.missed += std::min(8.0 * src.touched(entries / 8.0, per_line), entries);
        s.count += 1.0;
        entries = 0.0;
        room = capacity;
    };
    for (int i = 0; i < src.classes; ++i) {
        const double cut = std::max(1.0, src.len[i] / kSplitMax), len = src.len[i] / cut;
        for (double left = src.rows[i] * cut; left > 0.0;) {
            const double take = std::min(left, room);
            entries += take * len;
            left -= take;
            room -= take;
            if (room <= 0.0) sweep();
        }
    }
    if (entries > 0.0) sweep();
    return s;
}

// Pairs of steps that a launch's gathers are ahead of its additions (k_aggregate_tiles), by the part of its gathers that is expected to
// miss L2, a line a row (us with 0 / 2 / 3 / 4 pairs; ids in random order, all-active;
// sources, entries, missed):
//   16 lanes, F = 64: 262 K sources, 60 M entries, 0.03 missed 752 / 881 / 733 / 712, F = 48 686 / 875 / 724 / 707; 233 K, 115 M, 0.03 1265 /
//   1624 / 1337 / 1311; 1 M, 179 M, 0.07 2290 / 2626 / 2233 / 2257; 0.4 M, 44 M, 0.17 768 / 736 / 669 / 715; 4.2 M, 133 M, 0.21 2352 / 2450 /
//   2232 / 2293; 8.4 M, 149 M, 0.31 3180 / 3208 / 3014 / 3128; 3 M, 270 M, 0.49 7084 / 6468 / 6653 / 7196; 5 M, 139 M, 0.70 4406 / 4247 / 4201 / 4397.
//   8 lanes, F = 32: 262 K, 60 M, 0.024 439 / 527 / 422 / 409; 1 M, 179 M, 0.05 1301 / 1541 / 1252 / 1247; 0.4 M, 44 M, 0.11 384 / 418 / 369 / 372; 4.2 M, 0.16
//   1201 / 1336 / 1198 / 1225; 1 M, 89 M, 0.21 809 / 857 / 806 / 851; 8.4 M, 0.25 1592 / 1709 / 1601 / 1640; 3 M, 0.37 2710 / 2746 / 2804 / 3064; 5 M,
//   0.61 2044 / 1971 / 2018 / 2105; 2.4 M, 140 M,
//   F = 64 3220 / 3082 / 3142 / 3431; dense ones, 1.1 M, 252 M, 0.12 1.09 to 1.15 of a batch at a time with 4.
// 16 lanes that hardly miss: a batch at a time is the fastest over the three launches below 0.06 together (2703; 3 pairs 2794, 4 pairs 2730),
// not in each.  Two pairs, which only half of the gathers missing pays for (6468 of 6653), are no kernel for 16 lanes.
// 4 lanes need both batches in flight everywhere (114 M entries, 233 K sources, F = 16: 697 us without, 575 with one, 541 with two).
static int tile_ahead(int lanes, double missed) {
    if (lanes == 4) return 4;
    if (lanes == 8) return missed < 0.10 ? 4 : missed < 0.33 ? 3 : 2;
    return missed < 0.06 ? 0 : 3;
}
// Whether there is such a kernel (epp_launch_tiles): a switch of the environment may ask for any number.
static bool tile_ahead_built(int lanes, int ahead) {
    return lanes == 4 ? ahead == 4 : lanes == 8 ? ahead >= 2 && ahead <= 4 : ahead == 0 || ahead == 3;
}

static double tile_launch_us(const epp_path* p, const Sources& src, int F, int lanes) {
    struct Cost { double launch, sweep, entry, line_cached, line_missed, row, copy; };  // us; ps per entry, line, row and byte
    const Cost c = lanes == 4 ? Cost{45, 10.2, 2.5, 2.3, 19.6, 0.0, 0.36} : lanes == 8 ? Cost{76, 1.7, 6.5, 0.38, 10.7, 0.84, 0.29}
                                                                        : Cost{41, 3.4, 9.4, 0.90, 14.6, 0.22, 0.17};
    const TileShape t = tile_shape(F, lanes);
    const double per_line = std::max(1.0, 8.0 / t.stride), lines = std::max(1.0, t.stride == 12 ? 2.0 : t.stride / 8.0);
    const Sweeps sw = tile_sweeps(src, lanes, per_line);
    const double sweeps = sw.count, missed = sw.missed;
    const double nnz = (double)p->nnz;
    double us = c.launch + 1e-6 * (double)p->n_stream_rows * F * c.row +
                t.slices * (sweeps * c.sweep + 1e-6 * (nnz * c.entry + lines * ((nnz - missed) * c.line_cached + missed * c.line_missed)));
    if (t.packed) us += 8.0 + 4e-6 * c.copy * ((double)p->n_src * F + (double)p->n * t.slices * t.stride * 4);
    return us;
}

// Whether launches of width F run on tiles, and of how many lanes a slot.  The constants above were fitted to 544
// paths and widths (all-active, and 0.5 to 30 % training vertices; 65 K to 8.4 M vertices, 1.6 to 274 M entries, both models, F =
// 8 to 128), which they meet within 8 to 16 % (root mean square).  Of 487 of them that the row kernel does not take, launches by
// this rule need 0.86 of the group kernel's time on average, 1.12 at worst; always the better one would need 0.83.
// Some of them (us, group kernel / tiles of 4, 8 and 16 lanes): 274 M entries, 2.4 M sources, F = 64: 8866 / 12056 / 5550 /
// 7246; F = 16: 4940 / 2425 / 2587; 228 M, 8.4 M, R-MAT, F = 128: 12290 / - / 8960 / 8560; not taken: 19 M of 2.4 M, F = 128:
// 1547 / - / 1446 / 1442; 65 M of 8.4 M, F = 41: 2726 / 4699 / 4376 / 3603.
// Of 540 other paths and widths (ids in random order, 4 to 240 M entries, F = 5 to 160) 162 are taken, in 0.70 of the time on average,
// 1.11 at worst (R-MAT, 165,000 sources, F = 88).
// Among 8 and 16 lanes, slices of 33 to 48 floats on 16 (t.stride == 12), three quarters of whose lines they fill, take 0.92 of that: of 101
// launches the choice is then 0.01 % behind the better one, 0.4 % without (2.4 M sources, 140 M entries, F = 47: 3640 on 8, 3440 on 16).
// The tiles cost 9 to 11 us per million entries to prepare, which five launches have to repay.  Rows of up to 32 floats have to be
// estimated to save kNarrowSaves a launch besides: beyond that width the group kernel prepares a partitioned copy of skewed graphs, which
// costs as much as tiles, but here a group table of 20 us, and a run that ends soon pays for the difference (import and one epoch, F =
// 5 / 32, 31 M entries: 422 us without tiles, 891 with them; F = 32, 79 M: 1493, 2007; F = 16 / 41, 114 M: 1.1 ms more once, 0.37 ms less
// per epoch).  Preparation and one launch of the 162 run at 0.34 to 0.84 of the speed without tiles up to 32 floats, 0.71 to 2.0 up to
// 64, 1.04 to 2.4 beyond; narrow ones are repaid by 1.3 to 5.3 launches.  Fewer sources than
// 100,000 nearly fit the L2s together: the estimate of what hits them is not good enough there (65,000, 23 M entries, F = 96:
// 527 / - / 732 / 633, estimated 758 / - / 602 / 617), but for rows of 64 bytes and less, which four lanes gather faster from L2
// too (51,000, 30 M entries, F = 16: 269 / 181, estimated 230 / 202; 84,000, 118 M: 1085 / 691).
constexpr double kNarrowSaves = 400.0;  // us
// All of that is for ids in random order, where hardly a row has more than a few of a batch's 64 entries.  Where neighbours have
// neighbouring ids, rows fill batches by themselves, and their additions wait for each other: a band of 500 ids, 50 M entries, 1 M
// sources, F = 64: 1569 us on groups, 4677 on 8 lanes; communities of 20,000 ids with hubs, 116 M entries, F = 64: 3657 / 10191; ids by
// degree, 114 M entries, 233,000 sources, F = 16: 950 / 1540, F = 128: 2902 / 3990.  So the build first samples the batches
// (k_tile_order) and stops where their mean delay uses up what the launch would save.  Mean delay in steps, sampled: random order 0.01
// at most; a band of 200,000 ids 0.1; 2.4 M vertices by degree 1.9 to 3; 233,000 by degree 6 to 10; the narrow band 55 to 60.
// Such a step costs 35e-6 us a batch in the last case and 50 to 140e-6 in those before, where the estimates of the gathers are off,
// too: with 60e-6 the F = 128 above would be taken, with 100e-6 no launch of 56 paths and widths in 14 orders took more than 1.04 of
// the group kernel's time.
constexpr double kStepUs = 1e-4;

int epp_tile_lanes(const epp_path* p, int F, double* max_delay) {
    *max_delay = 1e30;
    const int mode = env_int("EPP_TUNE_TILES", 1);  // 0: never, 1: where it pays, 2: wherever it can be (tests)
    if (mode == 0 || F < 5 || p->nnz == 0) return 0;
    // (a source's id has 23 bits in an entry, and its row's place in the matrix 32)
    if (p->n > (1ll << kColBits) || (p->n - 1) * (int64_t)F >= (1ll << 32)) return 0;
    if (mode == 2) {
        const int lanes = env_int("EPP_TUNE_TILE_LANES", 8);
        return lanes == 4 || lanes == 16 ? lanes : 8;
    }
    if (epp_group_table_asked()) return 0;
    if (p->nnz < 4'000'000 || p->n_src < (F <= 16 ? 40'000 : 100'000)) return 0;
    const Sources src(p);
    const double groups = group_launch_us(p, src, F);
    int lanes = 0;
    double best = 1e30, ranked = 1e30;
    for (const int l : {4, 8, 16}) {
        const TileShape t = tile_shape(F, l);
        if (t.slices > 8) continue;
        const double us = tile_launch_us(p, src, F, l), rank = t.stride == 12 ? 0.92 * us : us;
        best = std::min(best, us);
        if (rank < ranked) { ranked = rank; lanes = l; }
    }
    const double need = std::max({0.1 * groups, 20.0 + 2e-6 * (double)p->nnz, F > 32 ? 0.0 : kNarrowSaves});
    const double spare = groups - need - best;
    if (spare <= 0.0) return 0;
    *max_delay = spare / (tile_shape(F, lanes).slices * (double)p->nnz / 64.0 * kStepUs);
    return lanes;
}

int epp_build_tiles(epp_path* p, int lanes, double max_delay, hipStream_t s, TilePlan** out) {
    *out = nullptr;
    const int rows_per_tile = tile_rows(lanes);
    const int64_t R = p->n_stream_rows;
    const int split = std::min(std::max(env_int("EPP_TUNE_TILE_SPLIT", kSplitMax), 8), kSplitMax);
    const epp_alloc_t* al = epp_alloc_of(p);
    const int32_t* rowptr = p->rowptr.as<int32_t>();
    const int2v* cv = reinterpret_cast<const int2v*>(p->cv.p);

    int shift = 0;
    while (((p->n - 1) >> shift) >= kBuckets) ++shift;

    // rows per length class, and the order of the ids
    DevArena counts;
    DevBuf hist, totals, places, block_hist;
    const unsigned blocks = blocks_for(R, kRowsPerBlock);
    const size_t b_hist = (size_t)blocks * kTileBins * 4;
    EPP_TRY(counts.reserve(3 * DevArena::rounded(kTileBins * 4) + DevArena::rounded(b_hist), al));
    counts.take(&totals, kTileBins * 4);
    counts.take(&places, kTileBins * 4);
    counts.take(&hist, kTileBins * 4);
    counts.take(&block_hist, b_hist);
    EPP_HIP_TRY(hipMemsetAsync(totals.p, 0, 2 * DevArena::rounded(kTileBins * 4), s));
    PinnedWords host;
    EPP_TRY(host.get(kTileBins));
    if (lanes == 4) sample_order<4>(p, split, shift, totals.as<unsigned>() + 3, s);
    else if (lanes == 8) sample_order<8>(p, split, shift, totals.as<unsigned>() + 3, s);
    else sample_order<16>(p, split, shift, totals.as<unsigned>() + 3, s);
    hipLaunchKernelGGL(k_tile_count, dim3(blocks), dim3(kListBlock), 0, s, rowptr, R, split, block_hist.as<unsigned>(),
                       totals.as<unsigned>(), max_delay);
    hipLaunchKernelGGL(k_tile_classes, dim3(kTileBins), dim3(256), 0, s, block_hist.as<unsigned>(), (int)blocks, hist.as<unsigned>(),
                       totals.as<unsigned>(), max_delay);
    EPP_HIP_TRY(hipGetLastError());
    unsigned* const h = reinterpret_cast<unsigned*>(host.p);  // the classes, then the totals
    EPP_HIP_TRY(hipMemcpyAsync(h, hist.p, kTileBins * 4, hipMemcpyDeviceToHost, s));
    EPP_HIP_TRY(hipMemcpyAsync(h + kTileBins, totals.p, 4 * 4, hipMemcpyDeviceToHost, s));
    EPP_HIP_TRY(hipStreamSynchronize(s));
    TileOrder& order = p->tile_order[tile_order_of(lanes)];
    order.delay = (double)h[kTileBins + 3] / kOrderSamples;
    if (too_slow(h[kTileBins + 3], max_delay)) return EPP_OK;
    TileBins bins;
    unsigned rank = 0;
    for (int b = 0; b < kTileBins; ++b) { bins.first[b] = rank; rank += h[b]; }
    const int64_t n_rows = h[kTileBins], n_parts = h[kTileBins + 1], n_cut = h[kTileBins + 2];
    if (p->n + n_parts >= 0x7FFFFFFFll || n_rows == 0) return EPP_OK;

    TilePlan* q = new TilePlan();
    struct Guard {  // (on an error: nothing may still be writing to what is given back)
        TilePlan* q;
        hipStream_t s;
        ~Guard() {
            if (!q) return;
            (void)hipStreamSynchronize(s);
            delete q;
        }
    } guard{q, s};
    q->at_once = std::max(env_int("EPP_TUNE_TILES_AT_ONCE", kTilesAtOnce) / 512, 1) * 512;  // (whole groups of kTogether tiles per XCD)
    const int64_t rows_at_once = (int64_t)q->at_once * rows_per_tile;
    q->lanes = lanes;
    q->ahead = env_int("EPP_TUNE_TILE_AHEAD", -1);
    if (!tile_ahead_built(lanes, q->ahead)) q->ahead = tile_ahead(lanes, tile_sweeps(Sources(p), lanes, 1.0).missed / (double)p->nnz);
    q->far = env_int("EPP_TUNE_TILE_FAR", 0) != 0;
    q->n_tiles = (int)((n_rows + rows_at_once - 1) / rows_at_once * q->at_once);
    q->n_parts = n_parts;
    q->n_cut = (int)n_cut;
    q->max_batches = (int)(p->nnz / 64 + q->n_tiles);  // (every tile's last batch may be filled up)
    const size_t n_places = (size_t)q->n_tiles * rows_per_tile;
    const size_t b_ent = DevArena::rounded((size_t)q->max_batches * 512), b_first = DevArena::rounded((size_t)(q->n_tiles + 1) * 4),
                 b_target = DevArena::rounded(n_places * 4), b_longest = DevArena::rounded((size_t)q->n_tiles * 4), b_care = DevArena::rounded(((size_t)q->max_batches / 16 + 1) * 4),
                 b_cut = DevArena::rounded((size_t)n_cut * sizeof(CutRow));
    EPP_TRY(q->store.alloc(b_ent + b_first + b_target + b_longest + b_care + b_cut, al));
    char* at = q->store.as<char>();
    q->ent = at;
    q->first_batch = reinterpret_cast<int32_t*>(at += b_ent);
    q->target = reinterpret_cast<int32_t*>(at += b_first);
    q->longest = reinterpret_cast<int*>(at += b_target);
    q->care = reinterpret_cast<unsigned*>(at += b_longest);
    q->cut = at += b_care;

    DevArena tmp;
    DevBuf dealt, batches, scan_tmp, total;
    EPP_TRY(tmp.reserve(DevArena::rounded(n_places * sizeof(Dealt)) + DevArena::rounded((size_t)q->n_tiles * 4) +
                        DevArena::rounded(epp_scan_tmp_bytes(q->n_tiles)) + 256, al));
    tmp.take(&dealt, n_places * sizeof(Dealt));
    tmp.take(&batches, (size_t)q->n_tiles * 4);
    tmp.take(&scan_tmp, epp_scan_tmp_bytes(q->n_tiles));
    tmp.take(&total, 8);
    EPP_HIP_TRY(hipMemsetAsync(dealt.p, 0xFF, n_places * sizeof(Dealt), s));
    EPP_HIP_TRY(hipMemsetAsync(q->care, 0, b_care, s));
    hipLaunchKernelGGL(k_tile_deal, dim3(blocks), dim3(kListBlock), 0, s, rowptr, p->row_ids.p ? p->row_ids.as<int32_t>() : nullptr, R,
                       split, (int)p->n, bins, block_hist.as<unsigned>(), places.as<unsigned>(), dealt.as<Dealt>(),
                       static_cast<CutRow*>(q->cut));
    hipLaunchKernelGGL(k_tile_sizes, dim3(blocks_for(q->n_tiles, 64)), dim3(64), 0, s, dealt.as<Dealt>(), rows_per_tile,
                       q->at_once, q->n_tiles, batches.as<int>());
    epp_scan_exclusive(batches.as<int>(), q->first_batch, q->n_tiles, total.as<long long>(), scan_tmp.as<int>(), s);
    // (the scan's last element is the total; little endian)
    EPP_HIP_TRY(hipMemcpyAsync(q->first_batch + q->n_tiles, total.p, 4, hipMemcpyDeviceToDevice, s));
    int* const bad = totals.as<int>();  // (what it held has been read)
    EPP_HIP_TRY(hipMemsetAsync(bad, 0, 4, s));
    if (lanes == 4) sort_tiles<4>(q, cv, dealt.as<Dealt>(), shift, bad, s);
    else if (lanes == 8) sort_tiles<8>(q, cv, dealt.as<Dealt>(), shift, bad, s);
    else sort_tiles<16>(q, cv, dealt.as<Dealt>(), shift, bad, s);
    EPP_HIP_TRY(hipMemcpyAsync(h, bad, 4, hipMemcpyDeviceToHost, s));
    EPP_HIP_TRY(hipGetLastError());
    EPP_HIP_TRY(hipStreamSynchronize(s));  // (the temporaries go, too)
    if (h[0]) {
        order.unfit = true;
        return EPP_OK;
    }
    guard.q = nullptr;
    *out = q;
    return EPP_OK;
}

int epp_launch_tiles(const epp_path* p, const TilePlan* q, float* parts, const float* in, float* packed, float* out, int F,
                     hipStream_t s, const unsigned long long* sources, const unsigned int* inner_rows) {
    const TileShape t = tile_shape(F, q->lanes);
    if (t.packed) {
        hipLaunchKernelGGL(k_pack_slices, dim3(blocks_for(p->n, 64)), dim3(kListBlock), 0, s, in, p->n, F, t.quads, t.stride, t.slices, sources,
                           packed);
    }
    TileArgs a;
    a.ent = static_cast<const int2v*>(q->ent);
    a.first_batch = q->first_batch;
    a.care = q->care;
    a.target = q->target;
    a.longest = q->longest;
    a.in = t.packed ? packed : in;
    a.out = out;
    a.parts = parts;
    a.n = (int)p->n;
    a.F = F;
    a.lanes = t.quads;
    a.ld = t.packed ? t.stride * 4 : F;
    a.slice_step = t.packed ? p->n * t.stride * 4 : t.quads * 4;
    a.blocks = q->n_tiles / kTileWaves;
    const int64_t bytes = ((p->n - 1) * (int64_t)a.ld + t.quads * 4) * 4;
    a.records = bytes <= (int64_t)kNowhere && !q->far ? (unsigned)bytes : 0u;
    a.zero = inner_rows ? p->zero_block.as<float>() : nullptr;
    a.inner_rows = inner_rows;
    switch (q->lanes * 16 + q->ahead) {  // (all that tile_ahead_built lets through)
        case 4 * 16 + 4: launch_tiles<4, 4>(a, t.slices, s); break;
        case 8 * 16 + 2: launch_tiles<8, 2>(a, t.slices, s); break;
        case 8 * 16 + 3: launch_tiles<8, 3>(a, t.slices, s); break;
        case 8 * 16 + 4: launch_tiles<8, 4>(a, t.slices, s); break;
        case 16 * 16 + 0: launch_tiles<16, 0>(a, t.slices, s); break;
        case 16 * 16 + 3: launch_tiles<16, 3>(a, t.slices, s); break;
        default: epp_set_error("no kernel for tiles of %d lanes, %d ahead", q->lanes, q->ahead); return EPP_ERR_INVALID_ARG;
    }
    if (q->n_cut > 0) {
        int log2T = 0;
        while (log2T < 6 && (4 << log2T) < F) ++log2T;
        hipLaunchKernelGGL(k_tile_add_parts, dim3(blocks_for((int64_t)q->n_cut << log2T, kListBlock)), dim3(kListBlock), 0, s,
                           static_cast<const CutRow*>(q->cut), q->n_cut, F, log2T, parts, inner_rows, out);
    }
    EPP_HIP_TRY(hipGetLastError());
    return EPP_OK;
}
