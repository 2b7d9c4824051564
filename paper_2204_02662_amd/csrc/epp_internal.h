// Internal declarations shared by the translation units of libepp (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "epp.h"

#define EPP_NCLASS 32

// An entry of a path is the pair (column word, weight bits).  The column word holds the source's
// vertex id in its low 29 bits and three flags:
constexpr int kEntRowEnd = (int)0x80000000u;  // last entry of its row
constexpr int kEntCold = 0x40000000;           // rarely referenced source: gathered with streaming loads
constexpr int kEntOuterOnly = 0x20000000;      // not an entry of the inner path that shares this array (below)
constexpr int kEntCol = 0x1FFFFFFF;
constexpr long long kMaxVertices = 0x20000000ll;  // vertex ids must leave the flag bits free

// f(i, lane) for the i of every lane's range [i0, i1): by the lane itself while they are few, else by the whole
// wavefront (all lanes call this): one long row must not make one lane do the work of thousands.
template <class F>
__device__ __forceinline__ void for_range_by_wave(int64_t i0, int64_t i1, F f) {
    const bool many = i1 - i0 > 8;
    if (!many) {
        for (int64_t i = i0; i < i1; ++i) f(i, (int)(threadIdx.x & 63));
    }
    for (unsigned long long todo = __ballot(many); todo; todo &= todo - 1ull) {
        const int l = __ffsll((long long)todo) - 1;
        const int64_t first = __shfl(i0, l, 64), last = __shfl(i1, l, 64);
        for (int64_t i = first + (int)(threadIdx.x & 63); i < last; i += 64) f(i, l);
    }
}

void epp_set_error(const char* fmt, ...);

#define EPP_HIP_TRY(expr)                                                                           \
    do {                                                                                            \
        hipError_t epp_e_ = (expr);                                                                 \
        if (epp_e_ != hipSuccess) {                                                                 \
            epp_set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(epp_e_), __FILE__,      \
                          __LINE__);                                                                \
            return EPP_ERR_HIP;                                                                     \
        }                                                                                           \
    } while (0)

#define EPP_TRY(expr)                  \
    do {                               \
        int epp_rc_ = (expr);          \
        if (epp_rc_ != EPP_OK) return epp_rc_; \
    } while (0)

// Device allocation that frees itself; `bytes` is kept for the footprint report.  The memory
// comes from the caller's allocator (epp_alloc_t, the handle keeps a copy) or, without one, from
// hipMalloc.  A buffer can also be a view of part of another allocation (temporaries carved from
// one arena: every hipMalloc / hipFree pair costs about 0.15 ms, hipFree waits for the device).
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    bool owned = true;
    epp_alloc_t via = {nullptr, nullptr, nullptr};  // allocator that owns p (alloc == NULL: hipMalloc)
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    DevBuf(DevBuf&& o) noexcept : p(o.p), bytes(o.bytes), owned(o.owned), via(o.via) { o.p = nullptr; o.bytes = 0; }
    DevBuf& operator=(DevBuf&& o) noexcept {
        if (this != &o) { release(); p = o.p; bytes = o.bytes; owned = o.owned; via = o.via; o.p = nullptr; o.bytes = 0; }
        return *this;
    }
    ~DevBuf() { release(); }
    int alloc(size_t n, const epp_alloc_t* a) {
        release();
        if (n == 0) n = 4;  // keep a valid pointer for empty arrays
        if (a && a->alloc && a->free) {
            p = a->alloc(n, a->ctx);
            if (!p || (reinterpret_cast<uintptr_t>(p) & 255)) {
                if (p) a->free(p, a->ctx);
                p = nullptr;
                epp_set_error("the caller's allocator gave no 256-byte aligned block of %zu bytes", n);
                return EPP_ERR_ALLOC;
            }
            via = *a;
        } else {
            if (hipMalloc(&p, n) != hipSuccess) {
                (void)hipGetLastError();
                p = nullptr;
                epp_set_error("device allocation of %zu bytes failed", n);
                return EPP_ERR_ALLOC;
            }
            via = {nullptr, nullptr, nullptr};
        }
        bytes = n;
        owned = true;
        return EPP_OK;
    }
    void view(void* ptr, size_t n) {  // memory owned by someone who outlives this view
        release();
        p = ptr;
        bytes = n;
        owned = false;
    }
    void release() {
        if (p && owned) {
            if (via.alloc) via.free(p, via.ctx);
            else (void)hipFree(p);
        }
        p = nullptr;
        bytes = 0;
        owned = true;
    }
    template <class T> T* as() const { return static_cast<T*>(p); }
};

// Bump allocator over one device allocation (256-byte aligned pieces).
struct DevArena {
    DevBuf store;
    size_t used = 0;
    static size_t rounded(size_t n) { return (std::max<size_t>(n, 4) + 255) & ~(size_t)255; }
    int reserve(size_t total, const epp_alloc_t* a) { used = 0; return store.alloc(total, a); }
    void take(DevBuf* b, size_t n) {
        b->view(static_cast<char*>(store.p) + used, n);
        used += rounded(n);
    }
};

// Group table of one path for one group size gs (neighbour grouping, Sec. 2.2): the path's
// entry array is cut into groups of gs consecutive entries; group g covers entries
// [g * gs, min((g + 1) * gs, nnz)).
struct Schedule {
    int gs = 0;
    int64_t n_groups = 0;
    int64_t n_split_rows = 0;  // rows cut by a group boundary (summed from the groups' partial rows)
    DevBuf store;              // the allocation behind the two tables
    DevBuf group_row;          // int32[n_groups] row holding the group's first entry; bit 31: starts inside it
    DevBuf cut_rows;           // int32[n_split_rows] (path-row indices)
    // Partial rows of the groups, per width F: float[n_groups][2][F].  Slot 0 of a group holds the
    // sum of the tail of a row that began in an earlier group, slot 1 the sum of the row still
    // open at the group's end.  Written by every launch before it is read; sized at schedule time
    // so that a launch never allocates.
    struct Pieces { int F; DevBuf buf; };
    std::vector<Pieces*> pieces;
    ~Schedule() { for (Pieces* q : pieces) delete q; }
    float* pieces_for(int F) const {
        for (const Pieces* q : pieces)
            if (q->F == F) return q->buf.as<float>();
        return nullptr;
    }
    int ensure_pieces(int F, const epp_alloc_t* a) {
        if (pieces_for(F) || n_split_rows == 0) return EPP_OK;
        Pieces* q = new Pieces();
        q->F = F;
        if (q->buf.alloc((size_t)n_groups * 2 * (size_t)F * sizeof(float), a) != EPP_OK) { delete q; return EPP_ERR_ALLOC; }
        pieces.push_back(q);
        return EPP_OK;
    }
    void drop_pieces(int F) {  // (hipFree waits for the device; a caller's allocator must be stream-ordered)
        for (size_t i = 0; i < pieces.size(); ++i)
            if (pieces[i]->F == F) { delete pieces[i]; pieces.erase(pieces.begin() + i); return; }
    }
    size_t bytes() const {
        size_t b = store.bytes;
        for (const Pieces* q : pieces) b += q->buf.bytes;
        return b;
    }
};

// Scratch memory of a launch that the paths of one handle share: a handle is used by one call at
// a time, so two of its paths never need their scratch at once.  Buffers only ever get added (a
// captured HIP graph may hold the address of an older one), unless the width they were added for has
// not been prepared; a request is served by the smallest
// buffer that is large enough, else by a new one, sized an eighth above the request at most so
// that paths of nearly equal size end up on one buffer.
struct ScratchPool {
    std::vector<DevBuf*> bufs;
    const void* accounted_by = nullptr;  // the path whose footprint report includes the pool
    ~ScratchPool() { for (DevBuf* b : bufs) delete b; }
    int get(size_t bytes, const epp_alloc_t* al, void** out) {
        DevBuf* best = nullptr;
        for (DevBuf* b : bufs)
            if (b->bytes >= bytes && (!best || b->bytes < best->bytes)) best = b;
        if (!best) {
            size_t step = 256;
            while (step * 16 <= bytes) step *= 2;  // an eighth of the leading power of two
            best = new DevBuf();
            if (best->alloc((bytes + step - 1) / step * step, al) != EPP_OK) { delete best; return EPP_ERR_ALLOC; }
            bufs.push_back(best);
        }
        *out = best->p;
        return EPP_OK;
    }
    void keep_first(size_t n) {
        for (; bufs.size() > n; bufs.pop_back()) delete bufs.back();
    }
    size_t bytes() const {
        size_t b = 0;
        for (const DevBuf* x : bufs) b += x->bytes;
        return b;
    }
};

// Source-partitioned layout of a path for one width ("reconstructed" execution path, Sec. 6's
// pre-processing step, re-derived for a GPU of 8 XCDs with private L2s).  The entries of the long
// rows whose source is among the most referenced ones are moved into 8 sections by partition of the
// source; section x is processed by XCD x only, whose L2 then holds only the source rows of
// partition x.  All other entries form the last section.  A row that has entries in several
// sections becomes one virtual row per section; each writes a partial row to `vpart`, and a last
// kernel adds a vertex's partial rows in section order.
struct Partition {
    DevBuf cv2;        // int2[nnz] entries, section after section, canonical order inside a section
    DevBuf vptr;       // int32[n_vrows + 1] entry range of every virtual row
    DevBuf tgt;        // int32[n_vrows] vertex id (< n) or n + slot in vpart
    int64_t n_vrows = 0;
    DevBuf mvert;      // int32[n_split] vertex of every row that is cut into sections
    DevBuf mptr;       // int32[n_split + 1] its slots in vpart
    int64_t n_split = 0, n_slots = 0;
    float* vpart = nullptr;  // float[n_slots][F], in the handle's scratch pool
    // what is needed to put the entries back into canonical order (the path may give its canonical
    // entry array back while every prepared width runs on a reconstructed copy)
    DevBuf srow, tile_first, tile_row;  // cut rows, their first tile, the row of every tile
    DevBuf toff;       // int32[9 * n_tiles] place of every tile in every section
    DevBuf sec4;       // section of every entry of the cut rows, 4 bits each, rows byte-aligned
    DevBuf sec_off;    // int32[n_split] first byte of a cut row in sec4
    DevBuf whole_off;  // int32[rows] place of a row that is not cut (-1: cut)
    int64_t n_tiles = 0;
    int sec_g[10] = {};    // first group of every section, then n_groups
    int64_t hot_entries = 0;  // entries in the eight hot sections
    Schedule* sched = nullptr;  // groups over (vptr, cv2)
    ~Partition() { delete sched; }
    size_t bytes() const {
        return cv2.bytes + vptr.bytes + tgt.bytes + mvert.bytes + mptr.bytes + srow.bytes + tile_first.bytes +
               tile_row.bytes + toff.bytes + sec4.bytes + sec_off.bytes + whole_off.bytes + (sched ? sched->bytes() : 0);
    }
};

// A row that the row kernel (epp_rows.hip) may cut into chunks: vertex, entries; for each of the widths that may use the list, 0, and during
// a launch how many chunks it has summed.  Every width counts for itself: widths cut a row into different numbers of chunks, and launches
// of two of them may be in flight at once.
constexpr int kLongUsers = 5;
struct LongRow { int v, begin, end; unsigned done[kLongUsers]; };
static_assert(sizeof(LongRow) == 32, "a row of the list lies in one line");
// The rows of a path of `nnz` entries with more than 2^log2 of them, those of every length class (2^(c-1) < length <= 2^c) beside each
// other, in any order, behind a place for every row that the shorter classes could have.
struct LongRows {
    LongRow* rows = nullptr;  // (NULL: not listed)
    int* head = nullptr;      // per class, kLongApart ints apart: how many, first place (cleared before they are listed)
    int log2 = 0, nnz = 0;
    __host__ __device__ int first_place(int c) const {
        int at = 0;
        for (int i = log2 + 1; i < c; ++i) at += nnz >> (i - 1);
        return at;
    }
};
constexpr int kLongApart = 16;
constexpr size_t kLongHeadBytes = EPP_NCLASS * kLongApart * sizeof(int);

__device__ __forceinline__ int length_class(int len) { return len <= 1 ? 0 : 32 - __clz(len - 1); }

// One row (or none, len = 0) of every thread of a workgroup, which all call this.  One atomic per workgroup and class: they follow each
// other at 20 to 40 ns.  `found`: 2 EPP_NCLASS ints of LDS.  (No row gets a place that its class does not have, whatever the lengths.)
__device__ __forceinline__ void list_long_rows(const LongRows& l, int v, int begin, int len, int* __restrict__ found) {
    const bool is_long = len > (1 << l.log2);
    if (!__syncthreads_or(is_long)) return;
    if (threadIdx.x < EPP_NCLASS) found[threadIdx.x] = 0;
    __syncthreads();
    const int c = length_class(len), at = is_long ? atomicAdd(&found[c], 1) : 0;
    __syncthreads();
    if (threadIdx.x < EPP_NCLASS && found[threadIdx.x])
        found[EPP_NCLASS + threadIdx.x] = atomicAdd(&l.head[threadIdx.x * kLongApart], found[threadIdx.x]);
    __syncthreads();
    if (!is_long) return;
    const int first = l.first_place(c), place = found[EPP_NCLASS + c] + at;
    if (place < l.nnz >> (c - 1)) l.rows[first + place] = LongRow{v, begin, begin + len, {}};
}
// The first places, by one workgroup of those that list.
__device__ __forceinline__ void place_long_rows(const LongRows& l) {
    if (threadIdx.x < EPP_NCLASS) l.head[threadIdx.x * kLongApart + 1] = l.first_place((int)threadIdx.x);
}

// What the row kernel needs to know of the rows that one workgroup should not take alone: they are cut into chunks, whose sums the last
// workgroup of the row's adds.
struct RowsPlan {
    DevBuf store;  // the pieces, and the rows where the path has no list of them, or none with a count to spare
    LongRow* rows = nullptr;
    const int* head = nullptr;
    float* pieces = nullptr;  // float[n_chunks][F]
    int n_chunks = 0;
    int user = 0;             // which of a row's counts is this width's
    unsigned* taken = nullptr;  // the path's list is used: the path's bits of the counts that are
    ~RowsPlan() { if (taken) *taken &= ~(1u << user); }
};

// What a build of tiles has shown about the order of a path's entries, whichever the width; per number of lanes.
struct TileOrder {
    bool unfit = false;   // they cannot be laid out
    double delay = -1.0;  // steps by which entries of one row delay a batch on average; -1: not known
};
inline int tile_order_of(int lanes) { return lanes == 4 ? 0 : lanes == 8 ? 1 : 2; }

// Tiles of rows whose sums a launch keeps in LDS while it takes their entries in source order (epp_tiles.hip); serves
// all widths that want the same lanes per source row.
struct TilePlan {
    DevBuf store;                    // the allocation behind the arrays
    int lanes = 0;                   // per slot
    int ahead = 0;                   // how far a launch's gathers run ahead of its additions
    bool far = false;                // launches take the addresses of far rows at any size (tests)
    int at_once = 0;                 // tiles that run at the same time, among which the rows are dealt
    int n_tiles = 0, max_batches = 0, n_cut = 0;
    int64_t n_parts = 0;
    void* ent = nullptr;             // int2[64 * batches]
    int32_t* first_batch = nullptr;  // [n_tiles + 1]
    int32_t* target = nullptr;       // [n_tiles * rows of a tile]
    int* longest = nullptr;          // [n_tiles]
    unsigned int* care = nullptr;    // two bits per batch
    void* cut = nullptr;             // rows that are cut into parts
};

struct epp_path {
    int64_t n = 0;       // vertices of the input graph
    int64_t n_rows = 0;  // R: rows of the path in canonical form (all-active graph: n)
    int64_t nnz = 0;
    int64_t n_src = 0;
    const unsigned long long* sources = nullptr;  // bitmap of the source vertices (owned by the handle); NULL: all
    bool sources_checked = true;  // every column is in it (an imported path: not known before epp_check_sources)
    int64_t max_len = 0;
    int64_t len_hist[EPP_NCLASS] = {};
    bool all_rows = false;       // all-active graph (handle from epp_prepare_full)
    // Streamed form: only rows with at least one entry, in ascending vertex order.
    int64_t n_stream_rows = 0;
    DevBuf store;                // one allocation behind row_ids, rowptr, long_rows and cv where they are views of it
    LongRows long_rows;          // (a path of a construction or an import, where the row kernel may ask for it)
    unsigned long_rows_taken = 0;  // which of its rows' counts belong to a width
    DevBuf row_ids;              // int32[n_stream_rows] vertex of each streamed row; unset: identity
    DevBuf rowptr;               // int32[n_stream_rows + 1]
    DevBuf cv;                   // int2[nnz]: (column word, weight bits)
    // Shared entries (Sec. 4: consecutive execution paths of a model overlap almost entirely once the
    // active sets approach saturation).  With N^{k-1} inside N^k, every entry of the path one level
    // further in is an entry of this one, in the same order.  Such an inner path can do without entry
    // arrays of its own: it keeps its row ids and row pointer (canonical form, export, combination
    // stage) and runs on this path's arrays, group tables and reconstructed copies, skipping the
    // entries that carry kEntOuterOnly and the rows left without any entry.
    epp_path* outer = nullptr;            // set on the inner path: the path whose entries it shares
    const unsigned int* inner_rows = nullptr;  // set on the inner path: bitmap of its rows (owned by the handle)
    bool has_inner = false;               // set on the outer path: kEntOuterOnly marks are in place
    DevBuf zero_block;                    // outer path: 256 zero bytes, what a skipped entry gathers
    DevBuf inner_pos;                     // outer path: int32[ceil(nnz / 64)] entries of the inner path before every 64th entry
    bool has_cold = false;       // entries of rarely referenced sources carry the cold flag
    int cold_F = 0;              // width the cold flags were chosen for (the largest prepared width that marks)
    epp_alloc_t alloc = {nullptr, nullptr, nullptr};  // the caller's allocator (alloc == NULL: hipMalloc)
    ScratchPool own_pool;        // launch scratch of a path that belongs to no epp_paths handle
    ScratchPool* pool = &own_pool;  // the handle's pool for the paths of an epp_paths handle
    ScratchPool own_rows;           // the same for packed source rows (needed together with the other's)
    ScratchPool* rows_pool = &own_rows;
    // all-active graph only
    DevBuf full_rowptr;          // int32[n + 1] as given (for export)
    int64_t n_empty_rows = 0;
    DevBuf empty_rows;           // int32[n_empty_rows] vertices with empty lists
    std::vector<Schedule*> scheds;
    std::vector<TilePlan*> tile_plans;
    TileOrder tile_order[3];
    // per-width choices
    // prepared: epp_path_prepare_width has been called; rows: launches run the row kernel, which needs no
    // group table (sched may be NULL then) and a plan only where some row is very long; slices: XCD feature slicing; part: source-partitioned layout
    // of this width, if it pays (owned by the path)
    struct WidthCfg {
        int F;
        int forced_gs = 0;
        bool prepared = false, rows = false;
        RowsPlan* plan = nullptr;
        Schedule* sched = nullptr;
        int log2_slices = 0;
        Partition* part = nullptr;
        TilePlan* tiles = nullptr;    // launches run on tiles (no group table then, but for the if-else baseline's)
        float* tile_parts = nullptr;  // sums of the cut rows' parts, in the handle's scratch pool
        float* packed = nullptr;  // the launch first copies its source rows to this place, `ld` floats apart
        int ld = 0;               // (NULL, F: it reads them where they are)
    };
    std::vector<WidthCfg> widths;
    int last_F = 0;
    ~epp_path() {
        for (Schedule* s : scheds) delete s;
        for (TilePlan* t : tile_plans) delete t;
        for (auto& w : widths) { delete w.part; delete w.plan; }
    }
};

struct epp_paths {
    int L = 0;
    int64_t n = 0;
    std::vector<DevBuf> bitmaps;    // L+1 bitmaps of N^k, uint64 words
    std::vector<int64_t> set_size;  // |N^k|
    std::vector<epp_path*> path;    // index l; once the sets stop growing, deeper layers share one object
    DevBuf set0_ids;                // ascending ids of N^0 (the other sets are path rows)
    DevBuf store;                   // the allocation that the bitmaps (small graphs: all arrays) are views of
    ScratchPool pool, rows_pool;    // launch scratch shared by the paths
    epp_alloc_t alloc = {nullptr, nullptr, nullptr};
    ~epp_paths() {
        for (size_t i = 0; i < path.size(); ++i) {
            bool seen = false;
            for (size_t j = 0; j < i; ++j) seen |= (path[j] == path[i]);
            if (!seen) delete path[i];
        }
    }
};

// Pinned host words that the device writes and the host reads after a wait; a lease on a block of a
// process-wide list (prepare.hip).
struct PinnedWords {
    long long* p = nullptr;
    size_t count = 0;
    PinnedWords() = default;
    PinnedWords(const PinnedWords&) = delete;
    PinnedWords& operator=(const PinnedWords&) = delete;
    int get(size_t need);
    ~PinnedWords();
    // A kernel that is all that a call launches may raise this signal when everything that it writes is written, and the host then looks at
    // a word of the block instead of asking the runtime, which knows 5 us later (prepared on 2,700 vertices 34.5 -> 29.2 us).
    // Not for calls of several launches: these then wait, unknown to the runtime, for the next hipStreamSynchronize, which takes 20 us
    // more from eight of them on (signals in export, import and the levels of a preparation: exported and synchronised 25 -> 32 us, prepared
    // on 20,000 vertices and synchronised 122 -> 141, imported and one epoch over a group table 193 -> 211).
    struct Signal { long long* flag; long long ticket; };
    Signal signal();
    int wait(hipStream_t s);
    long long ticket = 0;
    struct Block { long long* words = nullptr; hipEvent_t mark = nullptr; int device = -1; } block;  // (mark: an event of that GPU)
};
__device__ __forceinline__ void epp_raise(PinnedWords::Signal g) {  // (by one thread, whose own words it releases)
    __hip_atomic_store(g.flag, g.ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// prepare.hip
// histogram + max length of a built path (waits for them), row-end flags
int epp_path_finish(epp_path* p, hipStream_t s);
void epp_path_set_stats(epp_path* p, const unsigned long long* host);
// ascending vertex ids of N^k (device, owned by `p`); allocates nothing, never waits
int epp_active_ids(const epp_paths* p, int k, const int32_t** ids, int64_t* count);

// Whether an imported path's columns all lie in its source set; where they do not, `sources` is given up.  Once per path.
int epp_check_sources(epp_path* p, hipStream_t s);

// prepare_small.hip: the whole construction in one launch, for graphs of at most 65,536 vertices and 131,072 entries
bool epp_prepare_small_fits(const epp_csr_t* g, int64_t n_train, int L);
int epp_prepare_small(const epp_csr_t* g, const int32_t* train_ids, int64_t n_train, int L, const epp_alloc_t* alloc,
                      hipStream_t s, epp_paths_t** out);

// combine.hip
// device address of the static scratch array on the current GPU (symbol lookup once per device;
// no allocation).  Handles are created with the GPU current, so they resolve it up front.
int epp_static_scratch(float** ptr);

// combine_split.hip: whether these products are taken in bfloat16 parts; the launches (W': `groups` partial products of
// rows_per_group rows each)
bool epp_split_weight_gradient(int Fi, int Fo, int64_t n_rows);
bool epp_split_input_gradient(int Fi, int Fo, int64_t n_rows);
void epp_launch_weight_gradient_split(int64_t groups, int64_t rows_per_group, const int32_t* ids, int64_t n_rows, const float* Y,
                                      int Fi, const float* G, int Fo, float* out, hipStream_t s);
void epp_launch_input_gradient_split(const int32_t* ids, int64_t n_rows, const float* G, int Fo, const float* W, int Fi, float* Yg,
                                     hipStream_t s);

// aggregate.hip
int epp_build_schedule(epp_path* p, int gs, hipStream_t s, Schedule** out);
// inner_rows != NULL: the launch serves the inner path that shares p's entries (bitmap of its rows)
int epp_launch_aggregate(epp_path* p, Schedule* sc, int log2_slices, const float* in, float* out, int F, hipStream_t s,
                         const unsigned int* row_bits = nullptr, const unsigned int* src_bits = nullptr,
                         const Partition* part = nullptr, const unsigned int* inner_rows = nullptr,
                         float* packed = nullptr, int ld = 0, const unsigned long long* sources = nullptr);
double epp_lines_per_row(int F, int ld);           // 128-byte lines that a row of F floats touches on average, rows ld floats apart
// Whether a switch of the environment asks for what only the group kernel has: a layout of its entries; that, a group size or a
// choice of the copied source rows.
bool epp_group_layout_asked();
bool epp_group_table_asked();
int epp_packed_stride(const epp_path* p, int F);  // floats from row to row of packed source rows; F: not packed
// rows.hip: one launch that processes rows whole, for small paths
bool epp_rows_kernel_fits(const epp_path* p, int F);
int epp_build_rows_plan(epp_path* p, int F, hipStream_t s, RowsPlan** out);  // *out = NULL: none needed
// rows.hip: the list of long rows that whoever builds a path of `nnz` entries makes along with it: which rows, where the classes lie (*l,
// without memory); returns the bytes it takes, 0: none
size_t epp_plan_long_rows(int64_t nnz, LongRows* l);
int epp_launch_rows(const epp_path* p, const RowsPlan* plan, const float* in, float* out, int F, hipStream_t s, const unsigned int* inner_rows);
// group table over any (row pointer, entry count); not registered with the path
int epp_build_schedule_over(const epp_path* p, const int32_t* rowptr, int64_t n_rows, int64_t nnz, int gs, hipStream_t s,
                            Schedule** out);
int epp_default_group_size(const epp_path* p, int F);
int epp_zero_empty_rows(const epp_path* p, float* out, int F, hipStream_t s);
// ld: floats from one source row to the next.  Where the memory for it is missing, marks and partition are left out.
int epp_tune_locality(epp_path* p, int F, int ld, int gs, bool may_partition, hipStream_t s, int* log2_slices, Partition** part);

// tiles.hip: lanes per source row of a launch on tiles (0: it runs on the group table) and the longest delay of a batch
// with which that pays, bytes of the copy of the source rows that it makes (0: none)
int epp_tile_lanes(const epp_path* p, int F, double* max_delay);
size_t epp_tile_packed_bytes(const epp_path* p, int F, int lanes);
// *out = NULL: these entries cannot be laid out, or their batches would be delayed by more than max_delay (p->tile_order keeps both)
int epp_build_tiles(epp_path* p, int lanes, double max_delay, hipStream_t s, TilePlan** out);
int epp_launch_tiles(const epp_path* p, const TilePlan* q, float* parts, const float* in, float* packed, float* out, int F,
                     hipStream_t s, const unsigned long long* sources, const unsigned int* inner_rows);

// partition.hip
int epp_partition_hot_rows(double lines);  // source rows of width F the eight L2s hold together
// share of the gathers it has to save (epp_build_partition)
inline double epp_partition_score_needed(const epp_path* p) { return p->nnz < 5 * p->n_stream_rows ? 0.20 : 0.12; }
// source-partitioned layout of `p` for width F and group size gs, or *out = NULL where it does not pay
// `unstreamed` (or NULL): bitmap of the sources whose entries stay unmarked in the last section; the
// copy then sets the streamed-source marks itself, whatever the canonical array carries
int epp_build_partition(epp_path* p, int F, int gs, const unsigned int* hot_bitmap, const unsigned int* unstreamed,
                        hipStream_t s, Partition** out);

// partition.hip: canonical entry array of `p` rebuilt from a reconstructed copy, if it was given back
int epp_ensure_canonical(epp_path* p, hipStream_t s);
// gives the canonical entry array back if every prepared width runs on a reconstructed copy
void epp_release_canonical_if_unused(epp_path* p);
// would it be given back if width F_with_copy (0: none) had a reconstructed copy and were prepared?
bool epp_canonical_unused(const epp_path* p, int F_with_copy);

// prepare.hip: exclusive scan of n ints (*total, device, receives the sum); tmp: epp_scan_tmp_bytes(n)
size_t epp_scan_tmp_bytes(int64_t n);
void epp_scan_exclusive(const int* in, int* out, int64_t n, long long* total, int* tmp, hipStream_t s);
inline const epp_alloc_t* epp_alloc_of(const epp_path* p) { return p->alloc.alloc ? &p->alloc : nullptr; }
inline const epp_alloc_t* epp_alloc_of(const epp_paths* p) { return p->alloc.alloc ? &p->alloc : nullptr; }
