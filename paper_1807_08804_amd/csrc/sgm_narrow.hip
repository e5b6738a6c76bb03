// Persistent per-query kernel (gfx950): each slot workgroup takes queries
// from a queue and runs the whole filtering-and-joining pipeline of one query
// (thesis Alg. 3.1) with barrier-separated phases, in its own slot of device
// memory, then leaves the slot's bitmaps zeroed for the next query. Filter
// steps over many candidates or long rows are shared: the owner posts them on
// a board and the launch's idle workgroups (extra ones, and slot workgroups
// whose queue ran dry) claim chunks of them.
//
// Phases (thesis Ch. 3):
//   root candidates  -- kernel_check / kernel_collect of Alg. 3.2, part of the
//                       first explore step (a range of the graph's vertices
//                       in type order);
//   explore          -- kernel_explore of Alg. 3.2 along the spanning tree;
//   refine           -- Sec. "Candidate Nodes Refinement" (prune only);
//   candidate edges  -- Sec. "Joining Phase", two-step output per key;
//   join             -- edge order of Sec. "Joining Phase", one query vertex
//                       per level, rows staged through LDS offsets;
//   ordering         -- rows sorted by a packed key of candidate ranks.
// Candidate lists are kept alongside the bitmaps (a push that sets a new bit
// appends to the list), so no phase scans all V vertices. When a query
// outgrows the slot (list, slab or LDS capacities), the workgroup clears its
// slot and reports kNeedWide; the host then runs the multi-kernel path.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sgm_device.h"
#include "sgm_narrow.h"
#include "sgm_share.h"

namespace sgm {
namespace {

constexpr int NT = kNarrowThreads;
constexpr int NW = NT / 64;
constexpr int kBigCap = 256;         // LDS list of items for the whole workgroup
// A step with at least kLongShare rows beyond its flat window shares them
// too, kLongChunk rows per chunk, one wave per row.
constexpr int32_t kLongShare = 32;
constexpr int32_t kLongChunk = 16;
constexpr int32_t kRevMin = 256;      // candidates of u before a reverse check can pay
constexpr int32_t kRevMaxCand = 4096; // neighbours with at most this many candidates
constexpr int kListSortCap = 8192;    // int32 entries sorted in LDS
constexpr int kRowSortCap = 2048;     // final rows sorted in LDS (u64 key + int32 index);
                                      // more rows use radix passes in the slab

struct Smem {
    int64_t sh[NW + 1];
    int64_t slab_used;
    int64_t ectot[SGM_MAX_QE];
    int32_t *ec_cnt[SGM_MAX_QE];
    int32_t *ec_offs[SGM_MAX_QE];
    int32_t *ec_vals[SGM_MAX_QE];
    int32_t cnt[SGM_MAX_QV];
    int32_t eckey[SGM_MAX_QE];      // key vertex the join needs for each edge
    int32_t ecbuilt[SGM_MAX_QE];    // key vertex of the table built first
    int32_t jorder[SGM_MAX_QV], jpos[SGM_MAX_QV];
    int32_t lv_ext[SGM_MAX_QV], lv_first[SGM_MAX_QV], lv_nchk[SGM_MAX_QV];
    int32_t chk[SGM_MAX_QE];
    int32_t big[kBigCap];
    int32_t pairoff[NT];
    int32_t rowlo[NT];
    JLevel jl;                 // the join level being built
    int32_t wnok[2][NW];       // shared join levels: rows per wave of a block of pairs
    int64_t wbase[2];          // and the block's first output row
    unsigned long long cnt64;  // rows of a counting level
    int32_t abort_;
    int32_t q;
    int64_t slab_cap;  // this query's slab (see k_narrow)
    int64_t below_top; // a last join level placed at the slab's top: the slab used below it (-1: none)
    int32_t *table;    // the join's last table
    int32_t nev;
    int32_t nbig;
    int32_t ngiant;
    int32_t nnbl;
    int32_t nmarks;
    int32_t ndef;  // candidates whose pushes go to row segments
    int32_t retired;  // this slot gave up on a shared step (see HelpJob::dirty)
    int32_t unsorted; // ordering: some key is above the next one
    int32_t hostord;  // the final table is left in the slab for the host to order
    int32_t keybits;
    int64_t pin_off;  // byte offset of that table in the slab
    const int32_t *tableptr;
    const int32_t *listptr;  // the key columns' sorted candidate lists beside it
    unsigned long long rowhit;  // item_wg: listed rows with a matching entry
    int32_t hq, hch;            // helper: board entry and chunk claimed (-1: none)
    int8_t qsrc[SGM_MAX_QE], qdst[SGM_MAX_QE];  // the query's edges, staged for join_order
    uint64_t revmask;
    NQuery query;           // the descriptor, staged for its many small reads
    NTest nbl[SGM_MAX_QE + 1];  // neighbours a step still tests (and a reverse test)
    // What filtering has established so far. ver[v] counts the changes of
    // C(v); okv[2 e + s] is the version of one endpoint's candidates for
    // which every candidate of the other (s = 0: the source of query edge e,
    // 1: its destination) is known to have a matching neighbour, or -1.
    int32_t ver[SGM_MAX_QV];
    int32_t okv[2 * SGM_MAX_QE];
    int32_t skippar;  // the step's test against its parent is known to hold
    int32_t removed;
    int32_t rdrop;  // candidates a step's reverse tests removed
    int32_t ctr;
    int32_t empty;
    // per-query outcome, written to global memory by thread 0 at the end
    int32_t status;
    int32_t reason;
    int32_t cand[SGM_MAX_QV];
    int32_t bitsn[SGM_MAX_QV];
    int32_t kdepth;  // steps of the key columns' binary searches
    int32_t ocol[SGM_MAX_QV];  // table position of each output column
    int32_t nout;              // output columns (the projected ones)
    const int32_t *rkl[SGM_MAX_QV];  // list each key column ranks into (LDS copy if it fits)
    int64_t level_rows[SGM_MAX_QV];
    int64_t nrows;
    int64_t offset;
    int64_t need;
    unsigned long long bytes;  // algorithmic bytes moved (see add_bytes)
    int64_t t[5];              // wall clock at the phase boundaries
    unsigned long long pb[5];  // bytes at the phase boundaries
};

// Scratch LDS (g_dyn), 46 KB: with the rest a workgroup stays within 64 KB,
// and two workgroups per CU remain resident (registers allow no more). List
// sorting uses [0, 32 KB); the final ordering keeps keys and indices
// (bitonic) or digit counts (radix) in [0, 24 KB) and stages the candidate
// lists its keys rank into at [24 KB, 46 KB).
constexpr size_t kDynLds = 46 << 10;
constexpr size_t kStageOff = 24 << 10;
constexpr int32_t kStageInts = (int32_t)((kDynLds - kStageOff) / sizeof(int32_t));
static_assert(sizeof(int32_t) * kListSortCap <= kDynLds, "list sort space");
static_assert((sizeof(uint64_t) + sizeof(int32_t)) * kRowSortCap <= kStageOff, "row sort space");
static_assert(kDynLds + sizeof(Smem) + sizeof(NArgs) <= (64 << 10), "LDS per workgroup");
static_assert(8 * 256 * sizeof(int32_t) <= kStageOff, "radix counts");

// The workgroup's LDS, at file scope: a query's phases and the shared tiers
// are functions that are not inlined, each with registers of its own, and
// reach it as LDS too; they rebuild their context from the launch's arguments
// kept here. In one body, 750 KB of code, the small steps paid for the large
// tiers' spills; the split leaves a seventh of the code and shortens the
// large steps (six cyclic queries on 4M vertices 96 -> 73 ms, with the shared
// giant rows and reverse tests by marks that it made room for; queries of a
// few candidates within 2 %). A call into a large tier saves registers to
// scratch memory, most of what a launch of small queries writes.
__shared__ Smem g_s;
__shared__ NArgs g_args;
__shared__ __align__(16) unsigned char g_dyn[kDynLds];

struct Ctx {
    // the launch's graph, read in place from the kernel arguments (a copy in
    // the context would live in scratch memory: its adjacency pointers are
    // chosen by direction at run time)
    const DevGraph &g;
    int32_t lcap;
    int64_t slab_bytes;
    int32_t *out;
    int64_t out_cap;
    unsigned long long *out_used;
    int32_t *host_out;
    int64_t host_cap;
    const NQuery *Q;
    uint64_t *bits;     // slot bitmaps [(SGM_MAX_QV + 1) * nwords]
    uint64_t *scratch;  // the extra bitmap of the slot
    int32_t *lists;     // slot lists [SGM_MAX_QV * lcap]
    char *slab;
    int64_t *trace;     // this query's step events, or null
    int32_t gmax;       // most lanes per key of an edge table
    int32_t wg_rows;    // rows longer than this get the whole workgroup
    int32_t join_policy;
    int32_t *marks;     // pushes into the scratch bitmap, while filtering (slab)
    HelpJob *job;       // this slot's entry on the helper board
    int32_t *hctr;      // posted shared steps, slot workgroups done
    int32_t help_items; // share filter steps of at least this many candidates (0: never)
    int32_t q;          // index of the query in the batch
    int32_t nslot, ngrid;  // slot workgroups, all workgroups of the launch
    int64_t help_wait;  // polls of a shared step's completion before giving up
    int64_t host_order_rows;  // final tables of this many rows go to the host (0: none)
    __device__ uint64_t *B(int u) const { return bits + (int64_t)u * g.nwords; }
    __device__ int32_t *L(int u) const { return lists + (int64_t)u * lcap; }
};

// slab_cap: the slot's slab below tables its earlier queries of the launch
// left for the host to order (the whole slab otherwise)
__device__ __forceinline__ Ctx slot_ctx(const NArgs &a, int slot,
                                        int32_t q, int64_t slab_cap) {
    const int32_t nwords = a.g.nwords;
    uint64_t *bits = a.bits + (int64_t)slot * (SGM_MAX_QV + 1) * nwords;
    int32_t *lists = a.lists + (int64_t)slot * SGM_MAX_QV * a.lcap;
    char *slab = a.slab + (int64_t)slot * a.slab_bytes;
    return Ctx{a.g,  a.lcap, slab_cap, a.out, a.out_cap, a.out_used, a.host_out, a.host_cap, &g_s.query,
               bits, bits + (int64_t)SGM_MAX_QV * nwords, lists, slab,
               a.trace ? a.trace + (int64_t)q * SGM_TRACE_CAP : nullptr, a.group_lanes,
               a.wg_rows, a.join_policy,
               // while filtering the slab holds the long-row overflow list in
               // [0, 4 lcap) bytes and the marks in [4 lcap, 8 lcap)
               (int32_t *)(slab + 4 * (int64_t)a.lcap), a.board ? a.board + slot : nullptr, a.hctr,
               a.help_items, q, a.nslot, a.ngrid, a.help_wait, a.host_order_rows};
}

// A copy from LDS of what is the same in every lane, in scalar registers.
template <class T>
__device__ __forceinline__ T uniform_copy(const T &in) {
    static_assert(sizeof(T) % 4 == 0, "copied as ints");
    int32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &in, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    T out;
    __builtin_memcpy(&out, w, sizeof(T));
    return out;
}

template <class T>
__device__ __forceinline__ T uniform(T x) {
    return uniform_copy(x);
}

// Pointers to device memory, known as such (read back from LDS they could
// point anywhere, and every access through them would be a flat one).
template <class T>
__device__ __forceinline__ void in_memory(T *&p) {
    p = (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// The launch's arguments, inside a function that is not inlined.
__device__ __forceinline__ NArgs own_args() {
    NArgs a = uniform_copy(g_args);
    DevGraph &g = a.g;
    in_memory(g.out_off);
    in_memory(g.in_off);
    in_memory(g.out_adj);
    in_memory(g.in_adj);
    in_memory(g.vrow);
    in_memory(g.tverts);
    in_memory(g.trow);
    in_memory(g.tdeg);
    in_memory(g.vinfo);
    in_memory(g.out_ta);
    in_memory(g.out_tb);
    in_memory(g.in_ta);
    in_memory(g.in_tb);
    in_memory(g.hub_of);
    in_memory(g.hub_toff);
    in_memory(a.bits);
    in_memory(a.lists);
    in_memory(a.slab);
    in_memory(a.out);
    in_memory(a.trace);
    in_memory(a.board);
    in_memory(a.hctr);
    return a;
}

// The slot workgroup's context for its current query, inside a function that
// is not inlined.
#define SGM_OWN_CTX(c)                                                                    \
    const NArgs c##_args = own_args();                                                    \
    Ctx c = slot_ctx(c##_args, blockIdx.x, __builtin_amdgcn_readfirstlane(g_s.q),         \
                     uniform_copy(g_s.slab_cap))

__device__ __forceinline__ bool aborted(const Ctx &c) { return g_s.abort_ != 0; }

// Algorithmic byte accounting: every phase adds the global-memory words its
// algorithm must read or write (adjacency entries 8 B, neighbour tests 4 B,
// list / table / edge-table ints 4 B, bitmap words 8 B), not what caches
// happen to serve.
__device__ __forceinline__ void add_bytes(Ctx &c, uint64_t b) {
    if (b) atomicAdd(&g_s.bytes, (unsigned long long)b);
}

// wave-reduced variant: every lane of the wave must call it
__device__ __forceinline__ void add_bytes_wave(Ctx &c, uint64_t b) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) b += __shfl_xor(b, o, 64);
    if ((threadIdx.x & 63) == 0) add_bytes(c, b);
}

// step event (uniform call; thread 0 records)
__device__ __forceinline__ void ev(Ctx &c, int code) {
    if (c.trace && threadIdx.x == 0) {
        const int k = g_s.nev++;
        if (k < SGM_TRACE_CAP) c.trace[k] = (int64_t)(wall_clock64() << 8) | code;
    }
}

// Phase boundary i (0 start, 1 filtered, 2 edge tables built, 3 joined,
// 4 ordered and written): its clock and the bytes counted so far. Callers
// have passed a barrier since the phase's last byte count.
__device__ __forceinline__ void mark(Ctx &c, int i) {
    if (threadIdx.x == 0) {
        g_s.t[i] = wall_clock64();
        g_s.pb[i] = g_s.bytes;
    }
}

// Lowest slab offset of a table left for the host: the slot's later
// queries keep the filter's overflow list, marks, deferred list and row
// segments ([0, 12 lcap) and beyond) plus 4 MB below it.
__device__ __forceinline__ int64_t kPinFloor(const Ctx &c) {
    return 16ll * c.lcap + (4ll << 20);
}

// All threads call; returns the same pointer everywhere (nullptr + abort on
// overflow).
__device__ __forceinline__ char *slab_alloc(Ctx &c, int64_t bytes) {
    __syncthreads();
    const int64_t off = (g_s.slab_used + 255) & ~(int64_t)255;
    char *p = (off + bytes <= c.slab_bytes) ? c.slab + off : nullptr;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (p) g_s.slab_used = off + bytes;
        else g_s.abort_ = kWhySlab;
    }
    __syncthreads();
    return p;
}

// Counters a filter step updates: in the workgroup's LDS, or on the helper
// board while several workgroups share the step.
struct LdsCtr {
    __device__ int32_t *cnt(int v) const { return &g_s.cnt[v]; }
    __device__ int32_t *nbig() const { return &g_s.nbig; }
    __device__ int32_t *removed() const { return &g_s.removed; }
    __device__ int32_t *nmarks() const { return &g_s.nmarks; }
    __device__ int32_t *ndef() const { return &g_s.ndef; }
    __device__ int32_t *abort_() const { return &g_s.abort_; }
    __device__ bool failed() const { return __atomic_load_n(&g_s.abort_, __ATOMIC_RELAXED) != 0; }
};
struct BoardCtr {
    HelpJob *j;
    __device__ int32_t *cnt(int v) const { return &j->cnt[v]; }
    __device__ int32_t *nbig() const { return &j->nbig; }
    __device__ int32_t *removed() const { return &j->removed; }
    __device__ int32_t *nmarks() const { return &j->nmarks; }
    __device__ int32_t *ndef() const { return &j->ndef; }
    __device__ int32_t *abort_() const { return &j->abort_; }
    __device__ bool failed() const { return false; }  // a chunk is short: the owner looks
};

// Set bit x; on a newly set bit append x to list tl, or, for a push into
// the scratch bitmap (tl == nullptr: the parent's marks), to the marks list.
template <class K>
__device__ __forceinline__ void push_bit(Ctx &c, const K &k, uint64_t *tb, int32_t *tl, int v,
                                         int32_t x) {
    const uint64_t m = 1ull << (x & 63);
    uint64_t *w = tb + (x >> 6);
    if (__atomic_load_n(w, __ATOMIC_RELAXED) & m) return;
    const uint64_t old = atomicOr((unsigned long long *)w, m);
    if (old & m) return;
    if (tl) {
        const int32_t p = atomicAdd(k.cnt(v), 1);
        if (p < c.lcap) tl[p] = x;
        else *k.abort_() = kWhyList;
    } else {
        // marks are parent candidates, so at most lcap of them
        c.marks[atomicAdd(k.nmarks(), 1)] = x;
    }
}

__device__ __forceinline__ void push_bit(Ctx &c, uint64_t *tb, int32_t *tl, int v, int32_t x) {
    push_bit(c, LdsCtr{}, tb, tl, v, x);
}

// push_bit for up to four entries per lane (hk: push xk), appending the
// newly set ones with one counter update per wave: the lanes that reach
// this call take consecutive places in the order of their lane index. The
// four reads, then the four atomics, are in flight together.
template <class K, bool look = true>
__device__ __forceinline__ void push4(Ctx &c, const K &k, uint64_t *tb, int32_t *tl, int v,
                                      bool h0, int32_t x0, bool h1, int32_t x1, bool h2,
                                      int32_t x2, bool h3, int32_t x3) {
    bool h[4] = {h0, h1, h2, h3};
    const int32_t x[4] = {x0, x1, x2, x3};
    if (look) {
        uint64_t was[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            was[q] = __atomic_load_n(tb + (h[q] ? x[q] >> 6 : 0), __ATOMIC_RELAXED);
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] = h[q] && !((was[q] >> (x[q] & 63)) & 1ull);
    }
    unsigned long long old[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        old[q] = ~0ull;
        if (h[q]) old[q] = atomicOr((unsigned long long *)(tb + (x[q] >> 6)), 1ull << (x[q] & 63));
    }
    const bool n0 = !((old[0] >> (x0 & 63)) & 1ull), n1 = !((old[1] >> (x1 & 63)) & 1ull);
    const bool n2 = !((old[2] >> (x2 & 63)) & 1ull), n3 = !((old[3] >> (x3 & 63)) & 1ull);
    const int cnt = (int)n0 + (int)n1 + (int)n2 + (int)n3;
    const uint64_t b0 = __ballot(cnt & 1), b1 = __ballot(cnt & 2), b2 = __ballot(cnt & 4);
    const int tot = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
    if (tot == 0) return;
    const uint64_t lt = lanemask_lt(threadIdx.x & 63);
    const int pre = __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt);
    const int leader = __ffsll((unsigned long long)__ballot(1)) - 1;
    int32_t base = 0;
    if ((int)(threadIdx.x & 63) == leader) base = atomicAdd(tl ? k.cnt(v) : k.nmarks(), tot);
    base = __builtin_amdgcn_readlane(base, leader);
    int32_t p = base + pre;
    if (tl) {
        // a list may outgrow its capacity: the query then leaves the slot
        if (n0) { if (p < c.lcap) tl[p] = x0; else *k.abort_() = kWhyList; ++p; }
        if (n1) { if (p < c.lcap) tl[p] = x1; else *k.abort_() = kWhyList; ++p; }
        if (n2) { if (p < c.lcap) tl[p] = x2; else *k.abort_() = kWhyList; ++p; }
        if (n3) { if (p < c.lcap) tl[p] = x3; else *k.abort_() = kWhyList; }
    } else {
        // marks are parent candidates, so at most lcap of them
        if (n0) c.marks[p++] = x0;
        if (n1) c.marks[p++] = x1;
        if (n2) c.marks[p++] = x2;
        if (n3) c.marks[p] = x3;
    }
}

// entry i of a row ending at end, or an in-range dummy (vertex 0, no
// relation) past the end
__device__ __forceinline__ int2 adj_at(const int2 *adj, int32_t i, int32_t end) {
    return i < end ? adj[i] : make_int2(0, -1);
}

__device__ __forceinline__ bool nbr_hit(const Ctx &c, const NTest &d, int2 e) {
    if (!adj_rel_ok(c.g, e, d.rel) || !adj_type_ok(c.g, e, d.label)) return false;
    if (d.pin >= 0 && e.x != d.pin) return false;
    if (d.mode == 0) return bit_test(c.B(d.v), e.x);
    if (d.mode == 2) return true;
    const int2 vi = c.g.vinfo[e.x];
    return (d.label < 0 || vi.x == d.label) && (vi.y & 255) >= (d.qdeg & 255) &&
           (vi.y >> 8) >= (d.qdeg >> 8);
}

// Keep only the list entries whose bit is still set, preserving order.
__device__ __forceinline__ void list_from_bits(Ctx &c, int u);

// Zero the bitmap words of u's n listed candidates: one by one, or all words
// in order when the list is longer (a list of millions took one workgroup
// milliseconds of scattered stores).
__device__ __forceinline__ void clear_words(Ctx &c, int u, int32_t n) {
    uint64_t *b = c.B(u);
    const int32_t *l = c.L(u);
    if (n > c.g.nwords / 4) {
        for (int32_t w = threadIdx.x; w < c.g.nwords; w += NT) b[w] = 0ull;
    } else {
#pragma unroll 4
        for (int32_t i = threadIdx.x; i < n; i += NT) b[l[i] >> 6] = 0ull;
    }
}

__device__ __forceinline__ void compact_list(Ctx &c, int u) {
    if (g_s.cnt[u] > c.g.nwords) {
        // longer than the bitmap: read that instead
        list_from_bits(c, u);
        return;
    }
    int32_t *l = c.L(u);
    const uint64_t *b = c.B(u);
    __syncthreads();
    const int32_t n = g_s.cnt[u];
    int64_t out = 0;
    // eight consecutive entries per thread, their reads and bit tests all in
    // flight before the block scan; entries keep their order
    constexpr int kI = 8;
    for (int32_t base = 0; base < n; base += kI * NT) {
        const int32_t i0 = base + threadIdx.x * kI;
        int32_t x[kI];
#pragma unroll
        for (int k = 0; k < kI; ++k) x[k] = i0 + k < n ? l[i0 + k] : 0;
        bool keep[kI];
        int32_t cnt = 0;
#pragma unroll
        for (int k = 0; k < kI; ++k) {
            keep[k] = i0 + k < n && bit_test(b, x[k]);
            cnt += keep[k] ? 1 : 0;
        }
        int64_t tot;
        int64_t p = out + block_excl_scan<NW>(cnt, g_s.sh, &tot);
        // the block scan's barriers ordered every read of this round before
        // these writes, which stay at or below the entries just read
#pragma unroll
        for (int k = 0; k < kI; ++k)
            if (keep[k]) l[p++] = x[k];
        out += tot;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        g_s.cnt[u] = (int32_t)out;
        add_bytes(c, 12ull * n + 4ull * out);
    }
    __syncthreads();
}

// Rebuild list u from its bitmap in ascending order (O(V/64) words).
__device__ __forceinline__ void list_from_bits(Ctx &c, int u) {
    __syncthreads();
    const int32_t nwords = c.g.nwords;
    const uint64_t *src = c.B(u);
    int32_t *l = c.L(u);
    int64_t out = 0;
    // eight consecutive words per thread, all read before any is used (a
    // dependent read per block scan would leave the workgroup waiting)
    constexpr int kW = 8;
    for (int32_t base = 0; base < nwords; base += kW * NT) {
        const int32_t w0 = base + threadIdx.x * kW;
        uint64_t wd[kW];
#pragma unroll
        for (int k = 0; k < kW; ++k) wd[k] = w0 + k < nwords ? src[w0 + k] : 0ull;
        int32_t cnt = 0;
#pragma unroll
        for (int k = 0; k < kW; ++k) {
            cnt += __popcll(wd[k]);
        }
        int64_t tot;
        const int64_t ex = block_excl_scan<NW>(cnt, g_s.sh, &tot);
        if (out + tot > c.lcap) {
            if (threadIdx.x == 0) g_s.abort_ = kWhyList;
            break;  // uniform: tot and out are block-uniform
        }
        int64_t p = out + ex;
#pragma unroll
        for (int k = 0; k < kW; ++k) {
            uint64_t word = wd[k];
            while (word) {
                l[p++] = (w0 + k) * 64 + __builtin_ctzll(word);
                word &= word - 1ull;
            }
        }
        out += tot;
    }
    __syncthreads();
    if (threadIdx.x == 0 && !g_s.abort_) {
        g_s.cnt[u] = (int32_t)out;
        add_bytes(c, 8ull * nwords + 4ull * out);
    }
    __syncthreads();
}

// Sort list u ascending (LDS bitonic, or a rebuild from the bitmap).
__device__ __forceinline__ void sort_list(Ctx &c, int u) {
    __syncthreads();
    const int32_t n = g_s.cnt[u];
    if (n <= 1) return;
    int32_t N = 1, lg = 0;
    while (N < n) {
        N <<= 1;
        ++lg;
    }
    // barrier rounds of a bitonic network vs. an ordered rebuild from the
    // bitmap (two barriers per NT words)
    const int64_t cost_bitonic = (int64_t)lg * (lg + 1) / 2 * ((N / 2 + NT - 1) / NT);
    const int64_t cost_bits = 2 * ((c.g.nwords + 8 * NT - 1) / (8 * NT));
    if (n > kListSortCap || cost_bits < cost_bitonic) {
        list_from_bits(c, u);
        return;
    }
    int32_t *l = c.L(u);
    int32_t *t = (int32_t *)g_dyn;
    for (int32_t i = threadIdx.x; i < N; i += NT) t[i] = i < n ? l[i] : INT32_MAX;
    __syncthreads();
    for (int32_t size = 2; size <= N; size <<= 1) {
        for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
            for (int32_t i = threadIdx.x; i < N / 2; i += NT) {
                const int32_t lo = 2 * i - (i & (stride - 1));
                const int32_t hi = lo + stride;
                const bool up = (lo & size) == 0;
                const int32_t x = t[lo], y = t[hi];
                if ((x > y) == up) {
                    t[lo] = y;
                    t[hi] = x;
                }
            }
            __syncthreads();
        }
    }
    for (int32_t i = threadIdx.x; i < n; i += NT) l[i] = t[i];
    if (threadIdx.x == 0) add_bytes(c, 8ull * n);
    __syncthreads();
}

// ---------------------------------------------------------------------------
// filtering: one explore / refine step (Alg. 3.2 kernel_explore; refinement)
// ---------------------------------------------------------------------------

__device__ __forceinline__ void row_of(const DevGraph &g, int32_t up, int dir, int32_t *beg,
                                       int32_t *end) {
    const int4 r = g.vrow[up];
    *beg = dir ? r.z : r.x;
    *end = dir ? r.w : r.y;
}

// First index in [b, e) where less() no longer holds (e if none); the same
// arguments in all 64 lanes, all active. Each round reads 64 places at once:
// three dependent reads where a binary search of a hub's row takes 15 to 20.
template <class F>
__device__ __forceinline__ int32_t wave_bound(int32_t b, int32_t e, F less) {
    const int lane = threadIdx.x & 63;
    while (e - b > 64) {
        const int64_t len = e - b;
        auto at = [&](int l) { return b + (int32_t)((int64_t)(l + 1) * len / 65); };
        const int n = __popcll(__ballot(less(at(lane))));
        const int32_t nb = n == 0 ? b : at(n - 1) + 1;
        if (n < 64) e = at(n);
        b = nb;
    }
    return b + __popcll(__ballot(b + lane < e && less(b + lane)));
}

// Entries of candidate up's row that can pass test d: a hub row (at least
// kHubRow entries) tested against a typed query vertex is read from its
// copy sorted by the other end's type (then by relation for a labelled
// test), restricted to that type (and relation); any other row in full.
// Every entry left out fails the test (wrong type or relation), so the
// outcome is the full row's; the slice keeps the other ends ascending.
template <bool UNI = true>
__device__ __forceinline__ const int2 *test_row(const Ctx &c, int32_t up, const NTest &d,
                                                int32_t *beg, int32_t *end) {
    const DevGraph &g = c.g;
    row_of(g, up, d.dir, beg, end);
    const int2 *adj = g.adj(d.dir);
    if (g.hub_types == 0 || *end - *beg < kHubRow) return adj;
    const int32_t t = d.label;
    if (t < 0 || t + 1 >= g.hub_types) return adj;
    const int32_t h = g.hub_of[up];
    const int order = d.rel >= 0 ? 0 : 1;
    const int32_t *toff = g.hub_toff + ((int64_t)(h * 2 + d.dir) * 2 + order) * g.hub_types;
    int32_t b = *beg + toff[t], e = *beg + toff[t + 1];
    const int2 *arr = g.tab(d.dir, order);
    if (d.rel >= 0) {
        // the type's entries are sorted by relation: its relation's range
        if (UNI) {
            const int32_t b0 = b;
            b = wave_bound(b0, e, [&](int32_t i) { return (arr[i].y & g.rel_mask) < d.rel; });
            e = wave_bound(b0, e, [&](int32_t i) { return (arr[i].y & g.rel_mask) <= d.rel; });
            *beg = b;
            *end = e;
            return arr;
        }
        int32_t lo = b, hi = e;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if ((arr[mid].y & g.rel_mask) < d.rel) lo = mid + 1;
            else hi = mid;
        }
        int32_t lo2 = lo, hi2 = e;
        while (lo2 < hi2) {
            const int32_t mid = (lo2 + hi2) >> 1;
            if ((arr[mid].y & g.rel_mask) <= d.rel) lo2 = mid + 1;
            else hi2 = mid;
        }
        b = lo;
        e = lo2;
    }
    *beg = b;
    *end = e;
    return arr;
}

// Candidate up leaves its set (ub; null: a step that only looks, see
// filter_step's reverse tests).
template <class K>
__device__ __forceinline__ void drop_item(const K &k, uint64_t *ub, int32_t up) {
    if (!ub) return;
    atomicAnd((unsigned long long *)&ub[up >> 6], ~(1ull << (up & 63)));
    atomicAdd(k.removed(), 1);
}

// Whole workgroup on one candidate (uniform call). Prune: the candidate
// survives if every listed query edge has a matching neighbour; explore
// then pushes every matching neighbour.
__device__ __forceinline__ int32_t max_row(const DevGraph &g, const NTest *nb, int ncount, int32_t up);

template <class K>
__device__ __forceinline__ void item_wg_k(Ctx &c, const K &k, const NStep &st, const NTest *nb,
                                          int ncount, int32_t up, uint64_t *ub, uint64_t &fb,
                                          int32_t *defer = nullptr) {
    const DevGraph &g = c.g;
    if (ncount <= 16 && max_row(g, nb, ncount, up) <= 4 * NT) {
        // Every listed row fits one pass: all rows are read and tested at
        // once (bit 4j + k of `hits`: entry threadIdx.x + k NT of row j
        // matches), one barrier decides whether the candidate lives, and
        // pushes replay the recorded hits.
        if (threadIdx.x == 0) g_s.rowhit = 0ull;
        __syncthreads();
        uint64_t hits = 0, seen = 0;
        for (int j = 0; j < ncount; ++j) {
            const NTest d = nb[j];
            const int2 *adj = g.adj(d.dir);
            int32_t beg, end;
            row_of(g, up, d.dir, &beg, &end);
            const int32_t i = beg + threadIdx.x;
            const int2 e0 = adj_at(adj, i, end), e1 = adj_at(adj, i + NT, end);
            const int2 e2 = adj_at(adj, i + 2 * NT, end), e3 = adj_at(adj, i + 3 * NT, end);
            const uint64_t h = (uint64_t)((i < end) & nbr_hit(c, d, e0)) |
                               (uint64_t)((i + NT < end) & nbr_hit(c, d, e1)) << 1 |
                               (uint64_t)((i + 2 * NT < end) & nbr_hit(c, d, e2)) << 2 |
                               (uint64_t)((i + 3 * NT < end) & nbr_hit(c, d, e3)) << 3;
            if (h) atomicOr(&g_s.rowhit, 1ull << j);
            hits |= h << (4 * j);
            seen += end - beg;
        }
        __syncthreads();
        const bool alive = __popcll(g_s.rowhit) == ncount;
        __syncthreads();  // rowhit is read by all before the next candidate clears it
        if (!alive) {
            if (threadIdx.x == 0) {
                drop_item(k, ub, up);
                fb += 20ull + 12ull * seen;
            }
            return;
        }
        if (st.push)
            for (int j = 0; j < ncount; ++j) {
                const uint32_t hj = (uint32_t)(hits >> (4 * j)) & 15u;
                if (!hj) continue;
                const NTest d = nb[j];
                const int2 *adj = g.adj(d.dir);
                int32_t beg, end;
                row_of(g, up, d.dir, &beg, &end);
                uint64_t *tb = d.mode == 0 ? c.scratch : c.B(d.v);
                int32_t *tl = d.mode == 0 ? nullptr : c.L(d.v);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((hj >> q) & 1u) push_bit(c, k, tb, tl, d.v, adj[beg + threadIdx.x + q * NT].x);
            }
        if (threadIdx.x == 0) fb += 20ull + 12ull * seen;
        return;
    }
    bool alive = true;
    uint64_t seen = 0;
    for (int j = 0; j < ncount && alive; ++j) {
        const NTest d = nb[j];
        if (d.known) continue;
        int32_t beg, end;
        const int2 *adj = test_row(c, up, d, &beg, &end);
        bool found = false;
        for (int32_t base = beg; base < end; base += 4 * NT) {
            bool hit = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int32_t i = base + q * NT + threadIdx.x;
                if (i < end) hit |= nbr_hit(c, d, adj[i]);
            }
            seen += min(4 * NT, end - base);
            if (__syncthreads_or(hit)) {
                found = true;
                break;
            }
        }
        alive = found;
    }
    if (!alive) {
        if (threadIdx.x == 0) {
            drop_item(k, ub, up);
            fb += 20ull + 12ull * seen;
        }
        return;
    }
    if (st.push && defer) {
        if (threadIdx.x == 0) {
            defer[atomicAdd(k.ndef(), 1)] = up;
            fb += 20ull + 12ull * seen;
        }
        return;
    }
    if (st.push) {
        for (int j = 0; j < ncount; ++j) {
            const NTest d = nb[j];
            int32_t beg, end;
            const int2 *adj = test_row(c, up, d, &beg, &end);
            uint64_t *tb = d.mode == 0 ? c.scratch : c.B(d.v);
            int32_t *tl = d.mode == 0 ? nullptr : c.L(d.v);
            seen += end - beg;
            for (int32_t base = beg; base < end; base += 8 * NT) {
                // eight independent loads in flight per thread; a row's
                // neighbours are distinct, so their bits are set without a
                // look first
                const int32_t i = base + threadIdx.x;
                int2 e[8];
                bool h[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) e[q] = adj_at(adj, i + q * NT, end);
#pragma unroll
                for (int q = 0; q < 8; ++q) h[q] = (i + q * NT < end) && nbr_hit(c, d, e[q]);
                push4<K, false>(c, k, tb, tl, d.v, h[0], e[0].x, h[1], e[1].x,
                                     h[2], e[2].x, h[3], e[3].x);
                push4<K, false>(c, k, tb, tl, d.v, h[4], e[4].x, h[5], e[5].x,
                                     h[6], e[6].x, h[7], e[7].x);
            }
        }
    }
    if (threadIdx.x == 0) fb += 20ull + 12ull * seen;
}

__device__ __forceinline__ void item_wg(Ctx &c, const NStep &st, const NTest *nb, int ncount, int32_t up,
                                        uint64_t *ub, uint64_t &fb, int32_t *defer = nullptr) {
    item_wg_k(c, LdsCtr{}, st, nb, ncount, up, ub, fb, defer);
}

// One wave on one candidate (wave-uniform call, no workgroup barrier), four
// loads in flight per lane; same outcome as item_wg.
__device__ __forceinline__ void item_wave(Ctx &c, const NStep &st, const NTest *nb, int ncount,
                                          int32_t up, uint64_t *ub, uint64_t &fb,
                                          int32_t *defer = nullptr) {
    const DevGraph &g = c.g;
    const int lane = threadIdx.x & 63;
    bool alive = true;
    uint64_t seen = 0;
    for (int j = 0; j < ncount && alive; ++j) {
        const NTest d = nb[j];
        if (d.known) continue;
        int32_t beg, end;
        const int2 *adj = test_row(c, up, d, &beg, &end);
        bool found = false;
        for (int32_t base = beg; base < end; base += 256) {
            const int32_t i = base + lane;
            const int2 e0 = i < end ? adj[i] : make_int2(-1, -1);
            const int2 e1 = i + 64 < end ? adj[i + 64] : make_int2(-1, -1);
            const int2 e2 = i + 128 < end ? adj[i + 128] : make_int2(-1, -1);
            const int2 e3 = i + 192 < end ? adj[i + 192] : make_int2(-1, -1);
            const bool hit = (e0.x >= 0 && nbr_hit(c, d, e0)) || (e1.x >= 0 && nbr_hit(c, d, e1)) ||
                             (e2.x >= 0 && nbr_hit(c, d, e2)) || (e3.x >= 0 && nbr_hit(c, d, e3));
            seen += min(256, end - base);
            if (__ballot(hit)) {
                found = true;
                break;
            }
        }
        alive = found;
    }
    if (!alive) {
        if (lane == 0) {
            drop_item(LdsCtr{}, ub, up);
            fb += 20ull + 12ull * seen;
        }
        return;
    }
    if (st.push && defer) {
        // the pushes go to row segments that several workgroups share
        if (lane == 0) {
            defer[atomicAdd(&g_s.ndef, 1)] = up;
            fb += 20ull + 12ull * seen;
        }
        return;
    }
    if (st.push)
        for (int j = 0; j < ncount; ++j) {
            const NTest d = nb[j];
            int32_t beg, end;
            const int2 *adj = test_row(c, up, d, &beg, &end);
            uint64_t *tb = d.mode == 0 ? c.scratch : c.B(d.v);
            int32_t *tl = d.mode == 0 ? nullptr : c.L(d.v);
            seen += end - beg;
            for (int32_t base = beg; base < end; base += 256) {
                const int32_t i = base + lane;
                const int2 e0 = i < end ? adj[i] : make_int2(-1, -1);
                const int2 e1 = i + 64 < end ? adj[i + 64] : make_int2(-1, -1);
                const int2 e2 = i + 128 < end ? adj[i + 128] : make_int2(-1, -1);
                const int2 e3 = i + 192 < end ? adj[i + 192] : make_int2(-1, -1);
                if (e0.x >= 0 && nbr_hit(c, d, e0)) push_bit(c, tb, tl, d.v, e0.x);
                if (e1.x >= 0 && nbr_hit(c, d, e1)) push_bit(c, tb, tl, d.v, e1.x);
                if (e2.x >= 0 && nbr_hit(c, d, e2)) push_bit(c, tb, tl, d.v, e2.x);
                if (e3.x >= 0 && nbr_hit(c, d, e3)) push_bit(c, tb, tl, d.v, e3.x);
            }
        }
    if (lane == 0) fb += 20ull + 12ull * seen;
}

// longest adjacency row a candidate scans for the listed query edges
__device__ __forceinline__ int32_t max_row(const DevGraph &g, const NTest *nb, int ncount, int32_t up) {
    const int4 r = g.vrow[up];
    int32_t m = 0;
    for (int j = 0; j < ncount; ++j) m = max(m, nb[j].dir ? r.w - r.z : r.y - r.x);
    return m;
}

// lanes per key of an edge table for n keys: a power of two in [1, gmax], the
// most that leaves no lane without a key
__device__ __forceinline__ int lanes_for(int32_t n, int gmax) {
    int G = gmax;
    while (G > 1 && (int64_t)G * n > NT) G >>= 1;
    return G;
}

// Flat scan of several adjacency rows by one wave: the entries of up to 64
// segments (a candidate's row for one test) are laid end to end and dealt to
// the lanes, so a wave's time follows the sum of its rows, not the longest
// one. pre: where each segment starts; adr: what turns a position into an
// index of the adjacency array.
// Longer rows go to a wider tier: many candidates share a wave's scan, and
// its few long rows would hold the others back while other waves idle (rows
// of about 300, 28 queries one at a time: 3.4 ms at 512, 2.7 at 256). A tier
// more costs 10 us a step, so it begins where the rows pay for it: 300,000
// vertices with rows of 20 to 200, 28 queries one at a time 2.64 ms at 96,
// 2.36 at 256; a dense graph's 59 queries 8.9 ms at either. A wave with one
// candidate takes more.
constexpr int kFlatRow = 256;
constexpr int kFlatRowOne = 512;
struct FlatLds {
    int32_t pre[64], adr[64];
};

// orders this wave's LDS accesses before the call against those after it
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lane l's segment: len entries from adjacency index beg, positions
// [*pos, *pos + len). Returns the total.
__device__ __forceinline__ int32_t flat_begin(FlatLds *w, int32_t beg, int32_t len, int lane,
                                              int32_t *pos) {
    const int32_t inc = wave_incl_scan32(len, lane);
    wave_sync();  // the reads of the scan before
    w->pre[lane] = inc - len;
    w->adr[lane] = beg - (inc - len);
    *pos = inc - len;
    wave_sync();
    return __builtin_amdgcn_readlane(inc, 63);
}

// Do the positions [p, p + 64), lane i's match in bit i of `hits`, hold a
// match of this lane's segment [pos, pos + len)? (A segment's entries sit on
// consecutive lanes, so the wave's ballot answers for all 64 segments; one
// shared word of hit bits took an LDS atomic per matching entry, all on one
// address.)
__device__ __forceinline__ bool flat_found(uint64_t hits, int32_t p, int32_t pos, int32_t len) {
    const int32_t lo = max(pos - p, 0), hi = min(pos + len - p, 64);
    if (lo >= hi) return false;
    return (hits >> lo) << (64 - (hi - lo)) != 0ull;
}

// Segments of positions e[q] (the last one that starts at or before each).
__device__ __forceinline__ void flat_owner(const FlatLds *w, const int32_t (&e)[4], int (&o)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = 0;
#pragma unroll
    for (int st = 32; st > 0; st >>= 1)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (w->pre[o[q] + st] <= e[q]) o[q] += st;
}

__device__ __forceinline__ FlatLds *flat_lds(Ctx &c) {
    return (FlatLds *)g_dyn + (threadIdx.x >> 6);
}

// The first step of a query with an unpinned root takes its candidates from
// the graph's vertices in type order (DevGraph::tverts), not from a list: the
// root's type is a contiguous range of them, its row extents lie beside it
// (trow), and only the survivors enter the root's list and bitmap. Building
// the whole type's list and bitmap first, as every other vertex of the type
// was then dropped from them, cost the large graph's queries 80 us for one
// workgroup before the step began, and a sweep of all vertices per batch.
// root: degree bounds of such a step (least out-degree | least in-degree
// << 8 | 1 << 16 when they are read from vinfo: a compressed graph's bounds
// are not its row lengths), -1 for a step over a list.
__device__ __forceinline__ bool root_ok(const DevGraph &g, int32_t root, int32_t up, int4 vr) {
    int32_t od = vr.y - vr.x, id = vr.w - vr.z;
    if (root >> 16) {
        const int32_t y = g.vinfo[up].y;
        od = y & 255;
        id = y >> 8;
    }
    return od >= (root & 255) && id >= ((root >> 8) & 255);
}

// Candidates that pass to the overflow list at the start of the slab, which
// no phase uses while filtering (lcap entries).
template <class K>
__device__ __forceinline__ void to_overflow(Ctx &c, const K &k, int32_t up) {
    const int32_t p = atomicAdd(k.nbig(), 1);
    if (p < c.lcap) ((int32_t *)c.slab)[p] = up;
    else *k.abort_() = kWhyList;
}

// Survivors of a root step (the lanes in m) into u's list and bitmap.
template <class K>
__device__ __forceinline__ void keep_root(Ctx &c, const K &k, int u, uint64_t *ub, uint64_t m,
                                          int32_t up, int lane) {
    if (!m) return;
    int32_t p = 0;
    if (lane == 0) p = atomicAdd(k.cnt(u), __popcll(m));
    p = __builtin_amdgcn_readlane(p, 0) + __popcll(m & lanemask_lt(lane));
    if ((m >> lane) & 1ull) {
        if (p < c.lcap) c.L(u)[p] = up;
        else *k.abort_() = kWhyList;
        atomicOr((unsigned long long *)&ub[up >> 6], 1ull << (up & 63));
    }
}

// One wave, candidates ul[i0, i1) (at most 64, one per lane), the tests one
// after the other: a candidate that fails one reads no row for the next.
template <class K>
__device__ __forceinline__ void wave_items(Ctx &c, const K &k, int u, int32_t root, bool push,
                                           const NTest *nb, int ncount, const int32_t *ul,
                                           int32_t i0, int32_t i1, uint64_t *ub, int32_t bigdeg,
                                           uint64_t &fb) {
    const DevGraph &g = c.g;
    const int lane = threadIdx.x & 63;
    FlatLds *w = flat_lds(c);
    bool have = i0 + lane < i1;
    const int32_t up = have ? ul[i0 + lane] : 0;
    const int4 vr = root < 0 ? g.vrow[up] : have ? g.trow[(ul - g.tverts) + i0 + lane] : make_int4(0, 0, 0, 0);
    if (root >= 0) have = have && root_ok(g, root, up, vr);
    int32_t maxd = 0;
    for (int j = 0; j < ncount; ++j) maxd = max(maxd, nb[j].dir ? vr.w - vr.z : vr.y - vr.x);
    const bool over = have && maxd > bigdeg;
    if (over) {
        to_overflow(c, k, up);
        have = false;
    }
    const uint64_t overs = root >= 0 ? __ballot(over) : 0ull;  // candidates until a later tier drops them
    const uint64_t todo = __ballot(have);
    uint64_t alive = todo;
    int64_t seen = 0;
    const bool direct = push && ncount == 1;  // one scan finds and pushes
    for (int pass = 0; pass < (push && !direct ? 2 : 1); ++pass)
        for (int j = 0; j < ncount && alive; ++j) {
            const NTest d = nb[j];
            if (pass == 0 && d.known && !direct) continue;  // pushes only
            const int2 *adj = g.adj(d.dir);
            const bool on = (alive >> lane) & 1ull;
            int32_t beg = d.dir ? vr.z : vr.x;
            int32_t len = on ? (d.dir ? vr.w : vr.y) - beg : 0;
            const bool pushing = pass == 1 || direct;
            bool found = false;
            if (!pushing && d.label < 0 && d.pin < 0) {
                // a test that most entries pass: each lane's first four
                // entries first, and only the rest of the others' rows
                int2 en[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) en[q] = q < len ? adj[beg + q] : make_int2(0, -1);
#pragma unroll
                for (int q = 0; q < 4; ++q) found |= q < len && nbr_hit(c, d, en[q]);
                seen += 4;
                beg += 4;
                len = found ? 0 : max(len - 4, 0);
            }
            const uint64_t early = __ballot(found);
            int32_t pos;
            const int32_t T = flat_begin(w, beg, len, lane, &pos);
            uint64_t *tb = d.mode == 0 ? c.scratch : c.B(d.v);
            int32_t *tl = d.mode == 0 ? nullptr : c.L(d.v);
            seen += T;
            for (int32_t base = 0; base < T; base += 256) {
                int32_t e[4];
                int o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] = base + q * 64 + lane;
                flat_owner(w, e, o);
                uint64_t done = 0;
                if (!pushing && base > 0) {
                    // candidates found alive need no further entries
                    done = __ballot(found);
                    if (((alive & ~early) & ~done) == 0) break;
                }
                int2 en[4];
                bool h[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h[q] = e[q] < T && !((done >> o[q]) & 1ull);
                    en[q] = h[q] ? adj[w->adr[o[q]] + e[q]] : make_int2(0, -1);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) h[q] = h[q] && nbr_hit(c, d, en[q]);
                if (pass == 0)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        found |= flat_found(__ballot(h[q]), base + q * 64, pos, len);
                if (pushing)
                    push4(c, k, tb, tl, d.v, h[0], en[0].x, h[1], en[1].x, h[2], en[2].x, h[3],
                          en[3].x);
            }
            if (pass == 0) alive = __ballot(found);
        }
    if (root >= 0) {
        keep_root(c, k, u, ub, alive | overs, up, lane);
        if (lane == 0) fb += 20ull * (i1 - i0) + 12ull * seen;
        return;
    }
    const uint64_t dead = ub ? todo & ~alive : 0ull;
    if ((dead >> lane) & 1ull)
        atomicAnd((unsigned long long *)&ub[up >> 6], ~(1ull << (up & 63)));
    if (lane == 0) {
        if (dead) atomicAdd(k.removed(), __popcll(dead));
        fb += 20ull * __popcll(todo) + 12ull * seen;
    }
}

// One wave, few candidates: every row of every test at once (the candidates
// times the tests are at most 64 segments), so a step's chain is one read of
// the row extents, one of the entries and one of what they are tested
// against. Matches among the first 256 entries are pushed from registers.
template <class K>
__device__ __forceinline__ void wave_few(Ctx &c, const K &k, int u, int32_t root, bool push,
                                         const NTest *nb, int ncount, const int32_t *ul,
                                         int32_t i0, int32_t i1, uint64_t *ub, int32_t bigdeg,
                                         uint64_t &fb) {
    const DevGraph &g = c.g;
    const int lane = threadIdx.x & 63;
    FlatLds *w = flat_lds(c);
    const int n = i1 - i0;
    // item = lane / ncount by a 16-bit reciprocal (exact for lane < 64)
    const uint32_t inv = (65536u + (uint32_t)ncount - 1u) / (uint32_t)ncount;
    const int it = (int)(((uint32_t)lane * inv) >> 16), tj = lane - it * ncount;
    bool have = it < n;
    const int32_t up = have ? ul[i0 + it] : 0;
    const int4 vr = g.vrow[up];
    if (root >= 0) have = have && root_ok(g, root, up, vr);
    const int dir = nb[tj].dir;
    const int32_t beg = dir ? vr.z : vr.x, end = dir ? vr.w : vr.y;
    // this candidate's segments among the wave's, and those that decide
    const uint64_t mine = (ncount == 64 ? ~0ull : (1ull << ncount) - 1ull) << (it * ncount & 63);
    const uint64_t need = mine & ~__ballot(nb[tj].known);
    bool over = false;
    if (__ballot(have && end - beg > bigdeg) & mine) {
        over = have && tj == 0;
        if (over) to_overflow(c, k, up);
        have = false;
    }
    const bool todo = have;
    const int32_t len = have ? end - beg : 0;
    int32_t pos;
    const int32_t T = flat_begin(w, beg, len, lane, &pos);
    bool alive = false, found = false;
    for (int pass = 0; pass < (push && T > 256 ? 2 : 1); ++pass) {
        uint64_t live = 0;  // segments of surviving candidates
        if (pass == 1) live = __ballot(alive);
        for (int32_t base = 0; base < T; base += 256) {
            int32_t e[4];
            int o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) e[q] = base + q * 64 + lane;
            flat_owner(w, e, o);
            int2 en[4];
            bool h[4];
            NTest d[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int oi = (int)(((uint32_t)o[q] * inv) >> 16);
                d[q] = nb[o[q] - oi * ncount];
                h[q] = e[q] < T && (pass == 0 || ((live >> o[q]) & 1ull));
                const int2 *adj = g.adj(d[q].dir);
                en[q] = h[q] ? adj[w->adr[o[q]] + e[q]] : make_int2(0, -1);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) h[q] = h[q] && nbr_hit(c, d[q], en[q]);
            if (pass == 0)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    found |= flat_found(__ballot(h[q]), base + q * 64, pos, len);
            if (push && T <= 256) {
                alive = todo;
                alive &= (__ballot(found) & need) == need;
                live = __ballot(alive);
            }
            if (push && (pass == 1 || T <= 256)) {
                // all bits first, then each target's newly set ones take
                // consecutive places with one counter update
                unsigned long long old[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    old[q] = ~0ull;
                    if (h[q] && ((live >> o[q]) & 1ull))
                        old[q] = atomicOr((unsigned long long *)((d[q].mode == 0 ? c.scratch : c.B(d[q].v)) +
                                                                 (en[q].x >> 6)),
                                          1ull << (en[q].x & 63));
                }
                int tq[4];  // test of the entry's segment, -1: nothing new
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int oi = (int)(((uint32_t)o[q] * inv) >> 16);
                    tq[q] = (old[q] >> (en[q].x & 63)) & 1ull ? -1 : o[q] - oi * ncount;
                }
                for (int j = 0; j < ncount; ++j) {
                    uint64_t m[4];
                    int tot = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        m[q] = __ballot(tq[q] == j);
                        tot += __popcll(m[q]);
                    }
                    if (tot == 0) continue;
                    const int v = nb[j].v;
                    const bool marks = nb[j].mode == 0;
                    int32_t p = 0;
                    if (lane == 0) p = atomicAdd(marks ? k.nmarks() : k.cnt(v), tot);
                    p = __builtin_amdgcn_readlane(p, 0);
                    int32_t *tl = marks ? c.marks : c.L(v);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int32_t at = p + __popcll(m[q] & lanemask_lt(lane));
                        if (tq[q] == j) {
                            // marks are parent candidates, at most lcap
                            if (at < c.lcap) tl[at] = en[q].x;
                            else *k.abort_() = kWhyList;
                        }
                        p += __popcll(m[q]);
                    }
                }
            }
        }
        if (pass == 0) {
            alive = todo;
            alive &= (__ballot(found) & need) == need;
        }
    }
    if (root >= 0) {
        keep_root(c, k, u, ub, __ballot(tj == 0 && (alive || over)), up, lane);
        if (lane == 0) fb += 20ull * n + 12ull * (uint64_t)T;
        return;
    }
    const bool drop = ub && todo && !alive && tj == 0;
    if (drop) atomicAnd((unsigned long long *)&ub[up >> 6], ~(1ull << (up & 63)));
    const uint64_t dead = __ballot(drop);
    if (lane == 0) {
        if (dead) atomicAdd(k.removed(), __popcll(dead));
        fb += 20ull * n + 12ull * (uint64_t)T;
    }
}

// Candidates [it0, it1) of u's list (ul, bitmap ub), dealt to the waves: a
// candidate lacking a matching neighbour for one of the ncount tests is
// dropped; with push, the neighbours of the others that pass a test are
// pushed. Candidates with a row above kFlatRow entries go to the overflow
// list at the start of the slab for a wider tier (nodefer: a shared pass
// over long rows, one wave per row up to wg_rows, which the whole workgroup
// would take next; longer ones stay with the owner, whose pushes become
// shared row segments). Counters go to k.
template <class K>
__device__ __forceinline__ void filter_items(Ctx &c, const K &k, int u, int32_t root, bool push,
                                             const NTest *nb, int ncount, const int32_t *ul,
                                             uint64_t *ub, int32_t it0, int32_t it1,
                                             uint64_t &fb, bool nodefer = false) {
    const int wid = threadIdx.x >> 6;
    const int32_t per = nodefer ? 1 : min(64, (it1 - it0 + NW - 1) / NW);
    const int32_t bigdeg = nodefer ? max(4096, c.wg_rows) : per == 1 ? kFlatRowOne : kFlatRow;
    for (int32_t i = it0 + wid * per; i < it1 && !k.failed(); i += NW * per) {
        const int32_t e = min(it1, i + per);
        // few candidates and several tests: all their rows at once; the
        // rows of long-row passes are read test by test, which stops at the
        // first match
        if (!nodefer && ncount > 1 && (e - i) * ncount <= 64)
            wave_few(c, k, u, root, push, nb, ncount, ul, i, e, ub, bigdeg, fb);
        else
            wave_items(c, k, u, root, push, nb, ncount, ul, i, e, ub, bigdeg, fb);
    }
}

// A root that few vertices of its range reach (root_sparse): the vertices of
// ul[i0, i1) that have the degrees it asks for, into u's list and bitmap. The
// bounds alone cost two bytes a vertex here, eight vertices to a load and two
// to a comparison, the next round's loads under way; in a root step each 64
// vertices cost a wave's turn, 8 ns a vertex alone. (500,000 vertices of which
// none has 12 out-edges: 213 -> 115 us a call, 4.0 -> 0.4 ms in a served
// query's one workgroup.)
constexpr int kSparseLoads = 4;
constexpr int32_t kSparseRound = kSparseLoads * 512;  // vertices a wave takes at once
constexpr int32_t kSparseShare = 1 << 16;  // range from which the scan is shared
template <class K>
__device__ __forceinline__ void sparse_scan(Ctx &c, const K &k, int u, int32_t root,
                                            const int32_t *ul, int32_t i0, int32_t i1,
                                            uint64_t &fb) {
    const int lane = threadIdx.x & 63;
    // place i of the range is entry i + shift of deg, which starts at a
    // multiple of eight vertices in type order
    const int64_t p0 = ul - c.g.tverts;
    const int32_t shift = (int32_t)(p0 & 7), end = i1 + shift;
    const uint4 *deg = (const uint4 *)(c.g.tdeg + (p0 - shift));
    const uint32_t top = 0x80808080u, least = (uint32_t)(root & 0xffff) * 0x10001u;
    uint4 next[kSparseLoads];
    auto load = [&](int32_t at) {
#pragma unroll
        for (int q = 0; q < kSparseLoads; ++q) {
            const int32_t e = at + (q * 64 + lane) * 8;
            next[q] = e < end ? deg[e >> 3] : make_uint4(0, 0, 0, 0);
        }
    };
    int32_t at = ((i0 + shift) & ~7) + (int32_t)(threadIdx.x >> 6) * kSparseRound;
    load(at);
    for (; at < end; at += NW * kSparseRound) {
        // both bytes of a vertex's word at least the bounds: bit 7 of each
        uint32_t hit[kSparseLoads * 4], any = 0;
#pragma unroll
        for (int q = 0; q < kSparseLoads * 4; ++q) {
            const uint4 x = next[q >> 2];
            const uint32_t w = (q & 3) == 0 ? x.x : (q & 3) == 1 ? x.y : (q & 3) == 2 ? x.z : x.w;
            const uint32_t ge = ((w | top) - least) & top;
            hit[q] = ge & (ge >> 8) & 0x00800080u;
            any |= hit[q];
        }
        load(at + NW * kSparseRound);
        if (lane == 0) fb += 2ull * min(kSparseRound, end - at);
        if (__ballot(any != 0) == 0ull) continue;
        uint32_t ok = 0;  // bit 8 q + r: entry r of load q
#pragma unroll
        for (int q = 0; q < kSparseLoads * 4; ++q) {
            const int32_t i = at + ((q >> 2) * 64 + lane) * 8 + (q & 3) * 2 - shift;
            ok |= (uint32_t)((hit[q] & 0x80u) && i >= i0 && i < i1) << (2 * q);
            ok |= (uint32_t)((hit[q] >> 16) && i + 1 >= i0 && i + 1 < i1) << (2 * q + 1);
        }
        const int32_t n = __popc(ok), inc = wave_incl_scan32(n, lane);
        int32_t p = 0;
        if (lane == 63) p = atomicAdd(k.cnt(u), inc);
        p = __builtin_amdgcn_readlane(p, 63) + inc - n;
        for (; ok; ok &= ok - 1u) {
            const int b = __builtin_ctz(ok);
            const int32_t v = ul[at + ((b >> 3) * 64 + lane) * 8 + (b & 7) - shift];
            if (p < c.lcap) c.L(u)[p++] = v;
            else *k.abort_() = kWhyList;
            atomicOr((unsigned long long *)&c.B(u)[v >> 6], 1ull << (v & 63));
        }
    }
}

// Empty polls in a row before a helper leaves (helping is optional, so
// leaving early only costs speed; about a second of polling). The owner of
// a shared step polls its completion count at most NArgs::help_wait times
// (default 4M) before it gives up: an error, since every claimed chunk
// finishes in bounded time.
constexpr int64_t kHelpIdle = 1ll << 20;

// Claim word of a posted step, and a claim's outcome.
__device__ __forceinline__ unsigned long long claim_word(uint32_t seq, int32_t nch) {
    return ((unsigned long long)(seq & 0xffffffu) << 40) | ((unsigned long long)nch << 20);
}
__device__ __forceinline__ uint32_t claim_seq(unsigned long long w) { return (uint32_t)(w >> 40); }
__device__ __forceinline__ int32_t claim_nch(unsigned long long w) {
    return (int32_t)((w >> 20) & 0xfffffull);
}
__device__ __forceinline__ int32_t claim_next(unsigned long long w) {
    return (int32_t)(w & 0xfffffull);
}
// Take one chunk of board entry j (thread 0): the returned claim word's next
// field is the chunk, which exists if it is below the chunk field. The step
// named by the word stays posted, with fixed parameters, until every chunk
// taken from it is reported done.
__device__ __forceinline__ unsigned long long take_chunk(HelpJob *j) {
    return atomicAdd(&j->claim, 1ull);
}

// Row segments: pushes of long rows of surviving candidates, kSegEntries
// entries of one row and one neighbour test per segment, one pass of a
// whole workgroup each.
constexpr int32_t kSegEntries = 8 * NT;

// The pushes of segment sg = (candidate, test index, first entry, end) of a
// row (whole workgroup). A row's neighbours are distinct, so bits are set
// without a look first.
template <class K>
__device__ __forceinline__ void push_segment(Ctx &c, const K &k, const NTest *nb, int4 sg,
                                             uint64_t &fb) {
    const NTest d = nb[sg.y];
    int32_t rb, re;  // the segment indexes the array test_row picks for its row
    const int2 *adj = test_row(c, sg.x, d, &rb, &re);
    uint64_t *tb = d.mode == 0 ? c.scratch : c.B(d.v);
    int32_t *tl = d.mode == 0 ? nullptr : c.L(d.v);
    for (int32_t base = sg.z; base < sg.w; base += kSegEntries) {
        const int32_t i = base + threadIdx.x;
        int2 e[8];
        bool h[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = adj_at(adj, i + q * NT, sg.w);
#pragma unroll
        for (int q = 0; q < 8; ++q) h[q] = (i + q * NT < sg.w) && nbr_hit(c, d, e[q]);
        push4<K, false>(c, k, tb, tl, d.v, h[0], e[0].x, h[1], e[1].x, h[2], e[2].x, h[3], e[3].x);
        push4<K, false>(c, k, tb, tl, d.v, h[4], e[4].x, h[5], e[5].x, h[6], e[6].x, h[7], e[7].x);
    }
    if (threadIdx.x == 0) fb += 12ull * (uint64_t)(sg.w - sg.z);
}

// Segments of the rows of the nd deferred candidates into seg (at most cap);
// the count, or -1 if they do not fit (uniform).
__device__ __forceinline__ int32_t build_segments(Ctx &c, const NTest *nb, int ncount,
                                                  const int32_t *def, int32_t nd, int4 *seg,
                                                  int64_t cap) {
    int64_t carry = 0;
    for (int32_t base = 0; base < nd; base += NT) {
        const int32_t i = base + threadIdx.x;
        int32_t cnt = 0;
        if (i < nd)
            for (int j = 0; j < ncount; ++j) {
                int32_t b, e;
                test_row<false>(c, def[i], nb[j], &b, &e);
                cnt += (e - b + kSegEntries - 1) / kSegEntries;
            }
        int64_t tot;
        const int64_t ex = block_excl_scan<NW>(cnt, g_s.sh, &tot);
        if (i < nd && carry + tot <= cap) {
            int64_t p = carry + ex;
            for (int j = 0; j < ncount; ++j) {
                int32_t b, e;
                test_row<false>(c, def[i], nb[j], &b, &e);
                for (int32_t x = b; x < e; x += kSegEntries)
                    seg[p++] = make_int4(def[i], j, x, min(e, x + kSegEntries));
            }
        }
        carry += tot;
    }
    __syncthreads();
    return carry <= cap ? (int32_t)carry : -1;
}

__device__ __forceinline__ void ec_chunk(Ctx &c, const EcJob &E, HelpJob *j, int32_t i0, int32_t i1,
                                         int G, uint64_t &fb);

// A filter step shared with the launch's idle workgroups through this
// slot's board entry: the counters move to the entry, the work is cut into
// nch chunks that the owner and its helpers claim (kind 0: K candidates of
// u's list; kind 1: one row segment each; see HelpJob), and the owner waits
// for the chunks its helpers claimed before taking the counters back.
template <class W>
__device__ __forceinline__ void shared_run(Ctx &c, int kind, const NStep &st, const NTest *nb,
                                           int ncount, const int32_t *ul, uint64_t *ub,
                                           int32_t n_items, int32_t K, int G, int32_t nch,
                                           const int4 *seg, const EcJob *ecj, bool nodefer,
                                           int32_t root, const int32_t *def, W work) {
    HelpJob *j = c.job;
    if (threadIdx.x == 0) {
        for (int v = 0; v < SGM_MAX_QV; ++v) j->cnt[v] = g_s.cnt[v];
        j->nbig = 0;
        j->removed = 0;
        j->nmarks = g_s.nmarks;
        j->abort_ = 0;
        j->bytes = 0ull;
        j->done = 0;
        j->kind = kind;
        j->nodefer = nodefer;
        j->root = root;
        j->seg = seg;
        j->ul = ul;
        j->chunk = K;
        j->q = c.q;
        j->n_items = n_items;
        j->G = G;
        j->ncount = ncount;
        j->nodrop = ub == nullptr;
        j->ndef = g_s.ndef;
        j->defer = def != nullptr;
        j->st = st;
        for (int i = 0; i < ncount; ++i) j->nbl[i] = nb[i];
        if (ecj) {
            j->ecj = *ecj;
            j->jrows = 0ull;
        }
        const uint32_t seq =
            claim_seq(__hip_atomic_load(&j->claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) + 1u;
        // parameters, and the slot's lists and bitmaps, before the claim word
        __threadfence();
        atomicExch(&j->claim, claim_word(seq, nch));
        atomicAdd(&c.hctr[0], 1);
    }
    __syncthreads();
    int32_t own = 0, claimed = nch;  // (thread 0's: chunks that will be reported)
    for (;;) {
        if (threadIdx.x == 0) {
            const int32_t failed =
                __hip_atomic_load(&j->abort_, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned long long w = take_chunk(j);
            if (failed && claim_next(w) < claim_nch(w)) {
                // the query leaves the slot: no chunk beyond those taken (this
                // one, which is reported without work, among them)
                const unsigned long long v = atomicExch(&j->claim, claim_word(claim_seq(w), 0));
                claimed = min(claim_next(v), nch);
                ++own;
                w = 0ull;
            }
            g_s.hch = claim_next(w) < claim_nch(w) ? claim_next(w) : -1;
        }
        __syncthreads();
        const int32_t ch = g_s.hch;
        __syncthreads();
        if (ch < 0) break;
        work(j, ch);
        ++own;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // the owner's own chunks need no fence: it reads them itself
        int32_t got = atomicAdd(&j->done, own) + own;
        int64_t n = 0;
        while (got < claimed && n < c.help_wait) {
            __builtin_amdgcn_s_sleep(1);
            got = __hip_atomic_load(&j->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ++n;
        }
        if (got < claimed) {
            // give up: no further claims on the step (a claim against zero
            // chunks fails), and the slot stays out of use until the next
            // launch clears it, since chunks claimed earlier may still write
            // its bitmaps and lists
            const uint32_t seq = claim_seq(
                __hip_atomic_load(&j->claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            atomicExch(&j->claim, claim_word(seq, 0));
            atomicExch(&j->dirty, 1);
            g_s.retired = 1;
        }
        __threadfence();
        atomicSub(&c.hctr[0], 1);
        for (int v = 0; v < SGM_MAX_QV; ++v)
            g_s.cnt[v] = __hip_atomic_load(&j->cnt[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        g_s.nbig += __hip_atomic_load(&j->nbig, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        g_s.removed += __hip_atomic_load(&j->removed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        g_s.ndef = __hip_atomic_load(&j->ndef, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        g_s.nmarks = __hip_atomic_load(&j->nmarks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t ab = __hip_atomic_load(&j->abort_, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ab) g_s.abort_ = ab;
        if (got < claimed) g_s.abort_ = kWhyHelp;
        add_bytes(c, __hip_atomic_load(&j->bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __syncthreads();
}

__device__ __forceinline__ void shared_job(Ctx &c, int kind, const NStep &st, const NTest *nb,
                                           int ncount, const int32_t *ul, uint64_t *ub,
                                           int32_t n_items, int32_t K, int G, int32_t nch,
                                           const int4 *seg, uint64_t &fb,
                                           const EcJob *ecj = nullptr, bool nodefer = false,
                                           int32_t root = -1, int32_t *def = nullptr) {
    shared_run(c, kind, st, nb, ncount, ul, ub, n_items, K, G, nch, seg, ecj, nodefer, root, def,
               [&](HelpJob *j, int32_t ch) {
        if (kind == 0)
            filter_items(c, BoardCtr{j}, st.u, root, st.push != 0, nb, ncount, ul, ub, ch * K,
                         min(n_items, ch * K + K), fb, nodefer);
        else if (kind == 3)
            ec_chunk(c, *ecj, j, ch * K, min(n_items, ch * K + K), G, fb);
        else if (kind == 4)
            item_wg_k(c, BoardCtr{j}, st, nb, ncount, ul[ch], ub, fb, def);
        else
            push_segment(c, BoardCtr{j}, nb, seg[ch], fb);
    });
}

// Workgroups that can help this slot now: the launch's extra ones and the
// slot workgroups whose queue ran dry (uniform).
__device__ __forceinline__ int32_t helpers_now(Ctx &c) {
    if (c.help_items <= 0) return 0;
    if (c.ngrid > c.nslot) return c.ngrid - c.nslot;
    __syncthreads();
    if (threadIdx.x == 0)
        g_s.hch = c.ngrid - c.nslot +
                   __hip_atomic_load(&c.hctr[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int32_t h = g_s.hch;
    __syncthreads();
    return h;
}

// The candidates of a sparse root (uniform), shared from kSparseShare vertices.
__device__ __attribute__((noinline)) void sparse_root() {
    SGM_OWN_CTX(c);
    const int u = uniform(c.Q->root);
    const int32_t root = uniform(c.Q->pred[u].qout) | uniform(c.Q->pred[u].qin) << 8;
    const int32_t *ul = c.g.tverts + uniform(c.Q->root_lo);
    const int32_t n = uniform(c.Q->root_hi) - uniform(c.Q->root_lo);
    uint64_t fb = 0;
    if (c.help_items > 0 && c.job && n >= kSparseShare) {
        const int32_t K = chunk_items(n, helpers_now(c), NW * kSparseRound, 1 << 16);
        NStep st{};
        st.u = (int8_t)u;
        shared_run(c, 5, st, nullptr, 0, ul, nullptr, n, K, 64, chunk_count(n, K), nullptr, nullptr,
                   false, root, nullptr, [&](HelpJob *j, int32_t ch) {
            sparse_scan(c, BoardCtr{j}, u, root, ul, ch * K, min(n, ch * K + K), fb);
        });
    } else {
        sparse_scan(c, LdsCtr{}, u, root, ul, 0, n, fb);
    }
    add_bytes_wave(c, fb);
    __syncthreads();
}

// Where the wave and workgroup tiers of a pushing step list the candidates
// whose pushes become shared row segments, when helpers exist and the slab
// has room beyond the overflow list and the marks; else nullptr (uniform).
__device__ __forceinline__ int32_t *defer_list(Ctx &c, const NStep &st) {
    if (!st.push || c.help_items <= 0) return nullptr;
    if (c.slab_bytes < 12 * (int64_t)c.lcap + 64 * (int64_t)sizeof(int4)) return nullptr;
    if (helpers_now(c) <= 0) return nullptr;
    return (int32_t *)(c.slab + 8 * (int64_t)c.lcap);
}

// The candidates ul[0, n_items) through a step's tests, in tiers: waves over
// rows laid end to end; one wave per long row; the workgroup per row above
// wg_rows; the pushes of the last two as row segments. Each tier is shared
// with idle workgroups when it has enough to do (from one place: a copy of
// the shared tiers' code per tier made the kernel twice as large). ub: the
// bitmap the dropped candidates leave (null: none is dropped). The step's
// counters are zero on entry (from: the tier to start with).
__device__ __forceinline__ void filter_pass(Ctx &c, const NStep &st, int32_t root, const NTest *nb,
                                            int ncount, const int32_t *ul, uint64_t *ub,
                                            int32_t n_items, int32_t from, uint64_t &fb) {
    const DevGraph &g = c.g;
    const int u = st.u;
    const int lane = threadIdx.x & 63;
    // slab while filtering, in units of 4 lcap bytes: overflow list, marks,
    // deferred list, then the lists of rows and the row segments
    int32_t *ov = (int32_t *)c.slab;
    const bool room = c.slab_bytes >= 16 * (int64_t)c.lcap;
    int32_t *rows = (int32_t *)(c.slab + 12 * (int64_t)c.lcap);
    const bool can = c.help_items > 0 && c.job;
    // a step resumed at its pushes has listed them already
    int32_t *def = from == 3 ? (int32_t *)(c.slab + 8 * (int64_t)c.lcap) : nullptr;
    for (int tier = from; tier < 4; ++tier) {
        if (tier > 0) {
            // A step that has failed goes no further: the query leaves the
            // slot, and after a give-up a helper may still hold a chunk of
            // the tier before, so nothing more may be posted on the board
            // entry. (Every wave reads the word before the tier can set it.)
            __syncthreads();
            const bool failed = aborted(c);
            __syncthreads();
            if (failed) return;
        }
        // what the tier shares: kind (-1: nothing), items, chunk size, chunks
        int kind = -1;
        int32_t nsh = 0, K = 1, nch = 0;
        const int32_t *items = rows;
        const int4 *seg = nullptr;
        if (tier == 0) {
            // a step of many candidates is shared whether or not workgroups
            // are idle yet (in a batch they become idle while it runs)
            if (can && n_items >= c.help_items) {
                const int32_t helpers = helpers_now(c);
                kind = 0;
                items = ul;
                nsh = n_items;
                K = chunk_items(n_items, helpers, 64, 512);
                nch = chunk_count(n_items, K);
            } else {
                filter_items(c, LdsCtr{}, u, root, st.push != 0, nb, ncount, ul, ub, 0, n_items, fb);
            }
        } else if (tier == 1) {
            const int32_t nl = min(g_s.nbig, c.lcap);
            if (nl == 0) return;
            def = defer_list(c, st);
            ev(c, SGM_EV_LONGROWS);
            if (can && room && nl >= kLongShare) {
                // many long rows: one wave per row up to wg_rows entries,
                // shared like a step of many candidates (the rows move to a
                // list of their own; longer ones come back to the overflow
                // list)
                for (int32_t i = threadIdx.x; i < nl; i += NT) rows[i] = ov[i];
                __syncthreads();
                if (threadIdx.x == 0) g_s.nbig = 0;
                kind = 0;
                nsh = nl;
                K = kLongChunk;
                nch = (nl + kLongChunk - 1) / kLongChunk;
            }
        } else if (tier == 2) {
            // one wave per long row; rows above wg_rows get the whole
            // workgroup (listed in the slab where it has room), and so does
            // every row when there are fewer than waves
            const int32_t nbig = min(g_s.nbig, c.lcap);
            int32_t *giant = room ? rows : g_s.big;
            const int32_t gcap = room ? c.lcap : kBigCap;
            for (int32_t b = threadIdx.x >> 6; b < nbig; b += NW) {
                const int32_t up = ov[b];
                if (n_items <= NW || max_row(g, nb, ncount, up) > c.wg_rows) {
                    int32_t p = 0;
                    if (lane == 0) p = atomicAdd(&g_s.ngiant, 1);
                    p = __shfl(p, 0, 64);
                    if (p < gcap) {
                        if (lane == 0) giant[p] = up;
                        continue;
                    }
                    // list full: this wave handles the row itself
                }
                item_wave(c, st, nb, ncount, up, ub, fb, def);
            }
            __syncthreads();
            const int32_t ngiant = min(g_s.ngiant, gcap);
            if (ngiant >= 2 && room && can && n_items > NW && (!st.push || def)) {
                // one workgroup each, shared; the rows of a pushing step's
                // survivors then go out as shared row segments. (A step over
                // 81 hub rows: 2.6 ms by the owner alone, most of it the
                // tests.)
                kind = 4;
                nsh = nch = ngiant;
            } else {
                for (int32_t b = 0; b < ngiant; ++b) item_wg(c, st, nb, ncount, giant[b], ub, fb, def);
            }
        } else {
            // the deferred pushes (by this workgroup alone when they do not
            // fit the slab)
            const int32_t nd = g_s.ndef;
            if (!def || nd == 0) return;
            // room in the slab, and no more chunks than a claim word counts
            const int64_t cap = min((c.slab_bytes - 12 * (int64_t)c.lcap) / (int64_t)sizeof(int4),
                                    (int64_t)kMaxChunks);
            const int32_t nseg = build_segments(c, nb, ncount, def, nd, (int4 *)rows, cap);
            if (nseg > 0) {
                kind = 1;
                items = nullptr;
                seg = (const int4 *)rows;
                nch = nseg;
            } else {
                for (int32_t i = 0; i < nd; ++i)
                    for (int j = 0; j < ncount; ++j) {
                        int32_t b, e;
                        test_row(c, def[i], nb[j], &b, &e);
                        push_segment(c, LdsCtr{}, nb, make_int4(def[i], j, b, e), fb);
                    }
                __syncthreads();
            }
        }
        if (kind >= 0)
            shared_job(c, kind, st, nb, ncount, items, ub, nsh, K, 64, nch, seg, fb, nullptr,
                       tier == 1, tier == 0 ? root : -1, kind == 4 ? def : nullptr);
    }
}

// Intersect p's candidates with the pushed marks (all of them candidates of
// p): the marks are the intersection, so unless nothing left, its bitmap and
// list are rebuilt from them. Clears the scratch bitmap; true if p lost
// candidates (uniform).
__device__ __forceinline__ bool keep_marked(Ctx &c, int p) {
    uint64_t *pb = c.B(p);
    int32_t *pl = c.L(p);
    const int32_t n = g_s.cnt[p], nm = g_s.nmarks;
    const int32_t nwords = c.g.nwords;
    if (nm > nwords / 4) {
        // many marks: the scratch bitmap holds them, word by word (one by one,
        // a scattered atomic and a scattered store each: six cyclic queries
        // on 4M vertices 41.5 ms instead of 39.8)
#pragma unroll 4
        for (int32_t w = threadIdx.x; w < nwords; w += NT) {
            const uint64_t m = c.scratch[w];
            if (nm < n) pb[w] = m;
            c.scratch[w] = 0ull;
        }
        if (nm < n)
#pragma unroll 4
            for (int32_t i = threadIdx.x; i < nm; i += NT) pl[i] = c.marks[i];
    } else {
        if (nm < n) {
            clear_words(c, p, n);
            __syncthreads();
#pragma unroll 4
            for (int32_t i = threadIdx.x; i < nm; i += NT) {
                const int32_t x = c.marks[i];
                atomicOr((unsigned long long *)&pb[x >> 6], 1ull << (x & 63));
                pl[i] = x;
            }
        }
#pragma unroll 4
        for (int32_t i = threadIdx.x; i < nm; i += NT) c.scratch[c.marks[i] >> 6] = 0ull;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        g_s.cnt[p] = nm;
        add_bytes(c, nm < n ? 12ull * n + 24ull * nm : 12ull * nm);
    }
    __syncthreads();
    return nm < n;
}

// The tiers of a step beyond its first few candidates' short rows, in a
// function of its own (see g_s). from: the tier to start with. Returns the
// bytes of this thread's work.
__device__ __attribute__((noinline)) uint64_t filter_far(int step_u, int push, int parent, int first,
                                                         int32_t root, int32_t from) {
    SGM_OWN_CTX(c);
    const NStep st{(int8_t)__builtin_amdgcn_readfirstlane(step_u), (int8_t)__builtin_amdgcn_readfirstlane(push),
                   (int8_t)__builtin_amdgcn_readfirstlane(parent), 0,
                   (int16_t)__builtin_amdgcn_readfirstlane(first), 0};
    root = __builtin_amdgcn_readfirstlane(root);
    from = __builtin_amdgcn_readfirstlane(from);
    const int u = st.u;
    uint64_t *ub = c.B(u);
    const int32_t *ul = root < 0 ? c.L(u) : c.g.tverts + c.Q->root_lo;
    const int32_t n_items = root < 0 ? g_s.cnt[u] : c.Q->root_hi - c.Q->root_lo;
    uint64_t fb = 0;
    const int ncount = g_s.nnbl;
    // Reverse tests first: the neighbour's candidates push the members of
    // C(u) they reach over the edge, and those stay. What an explore step
    // does for its parent, with nothing dropped from C(v).
    for (uint64_t rm = g_s.revmask;;) {
        const bool rev = rm != 0;
        if (!rev && ncount == 0 && root < 0) break;
        const NNbr d = c.Q->nbr[st.first + (rev ? __builtin_ctzll(rm) : 0)];
        if (rev && threadIdx.x == 0) {
            NTest *rt = g_s.nbl + SGM_MAX_QE;
            rt->v = (int8_t)u;
            rt->dir = 1 - d.dir;
            rt->mode = 0;
            rt->known = 0;
            rt->rel = d.rel;
            rt->label = c.Q->pred[u].label;
            rt->pin = c.Q->pred[u].pin;
            rt->qdeg = 0;
        }
        if (rev) __syncthreads();
        const int32_t n = g_s.cnt[u];
        filter_pass(c, rev ? NStep{d.v, 1, (int8_t)u, 0, 0, 0} : st, rev ? -1 : root,
                    g_s.nbl + (rev ? SGM_MAX_QE : 0), rev ? 1 : ncount, rev ? c.L(d.v) : ul,
                    rev ? nullptr : ub, rev ? g_s.cnt[d.v] : root < 0 ? n : n_items, from, fb);
        if (!rev) break;
        __syncthreads();
        // The marks of a failed pass may be incomplete. (The abort word is read
        // between barriers only: at the head of the loop a fast wave's pushes
        // could already have set it when a slow one looked, and the waves
        // would have parted before a barrier.)
        if (aborted(c)) break;
        keep_marked(c, u);
        if (threadIdx.x == 0) g_s.rdrop += n - g_s.cnt[u];
        if (threadIdx.x == 0) {
            g_s.nbig = 0;
            g_s.ngiant = 0;
            g_s.nmarks = 0;
            g_s.ndef = 0;
        }
        __syncthreads();
        rm &= rm - 1;
    }
    return fb;
}

// compact_list of more than a few entries, likewise.
__device__ __attribute__((noinline)) void compact_far(int u) {
    SGM_OWN_CTX(c);
    compact_list(c, __builtin_amdgcn_readfirstlane(u));
}

// One step; returns the number of candidates it removed from C(u) (uniform).
// root: -1, or the first step of a query with an unpinned root (see root_ok).
__device__ __forceinline__ int32_t filter_step(Ctx &c, const NStep &st, int32_t root = -1) {
    const DevGraph &g = c.g;
    const int u = st.u;
    uint64_t *ub = c.B(u);
    const int32_t *ul = root < 0 ? c.L(u) : g.tverts + c.Q->root_lo;
    const int32_t n_items = root < 0 ? g_s.cnt[u] : c.Q->root_hi - c.Q->root_lo;
    uint64_t fb = 0;  // algorithmic bytes of this thread's work
    // A test known to hold is left out: every candidate of u was found (or
    // pushed) with a matching neighbour in C(v), C(v) has not changed since
    // and C(u) only shrinks. Refinement repeats the tree edges that the
    // exploration has just established, so a query whose candidates are down
    // to a few runs hardly any of its refine steps. An explore step's test
    // against its parent is kept for what it pushes, except for a parent with
    // a single candidate: what it would push is that candidate, as long as
    // any candidate of u survives.
    const bool in = (int)(threadIdx.x & 63) < st.count;
    const NNbr td = c.Q->nbr[st.first + (in ? threadIdx.x & 63 : 0)];
    const bool known = in && td.mode == 0 && g_s.okv[2 * td.e + td.dir] == g_s.ver[td.v];
    if (!st.push && __popcll(__ballot(known)) == st.count) return 0;  // every wave alike
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        if (lane == 0) {
            g_s.nbig = 0;
            g_s.ngiant = 0;
            g_s.removed = 0;
            g_s.rdrop = 0;
            g_s.nmarks = 0;
            g_s.ndef = 0;
        }
        const bool spar = known && st.push && g_s.cnt[td.v] == 1;
        bool keep = in && !spar && (st.push || !known);
        // In prune-only steps over many candidates, a neighbour with few
        // candidates whose rows together are shorter than u's list is
        // checked from its side instead.
        uint64_t rm = 0;
        if (!st.push && n_items >= kRevMin) {
            const int32_t nvl = g_s.cnt[td.v];
            uint64_t cand = __ballot(keep && nvl <= kRevMaxCand && nvl < n_items);
            while (cand) {
                const int j = __builtin_ctzll(cand);
                cand &= cand - 1;
                const int v = __builtin_amdgcn_readlane((int)td.v, j);
                const int dir = __builtin_amdgcn_readlane((int)td.dir, j);
                // reverse cost: v's list plus its rows, against at least one
                // read per candidate of u forward
                const int32_t nv = g_s.cnt[v];
                const int32_t *off = g.off(!dir);
                const int32_t *vl = c.L(v);
                int64_t sum = nv;
                for (int32_t b = 0; b < nv && sum <= n_items; b += 64) {
                    int32_t len = 0;
                    if (b + lane < nv) {
                        const int32_t y = vl[b + lane];
                        len = off[y + 1] - off[y];
                    }
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) len += __shfl_xor(len, o, 64);
                    sum += len;
                }
                if (sum <= n_items) rm |= 1ull << j;
            }
            keep = keep && !((rm >> lane) & 1ull);
        }
        // The tests in the order of what they cost and drop: relation and
        // type (or a pin) given, type, relation, neither, and last a parent
        // test kept for its pushes alone.
        const VPred &p = c.Q->pred[td.v];
        const int32_t lab = p.label, pin = p.pin;
        const int rank = known ? 4 : lab >= 0 || pin >= 0 ? (td.rel >= 0 || pin >= 0 ? 0 : 1)
                                                          : (td.rel >= 0 ? 2 : 3);
        int at = 0, n = 0;
#pragma unroll
        for (int r = 0; r < 5; ++r) {
            const uint64_t m = __ballot(keep && rank == r);
            if (rank == r) at = n + __popcll(m & lanemask_lt(lane));
            n += __popcll(m);
        }
        if (keep) {
            // the edge itself is one in-edge (dir 0) or out-edge of the
            // neighbour: often all the degree its vertex asks for
            const bool degok = td.dir ? p.qout <= 1 && p.qin == 0 : p.qin <= 1 && p.qout == 0;
            NTest &t = g_s.nbl[at];
            t.v = td.v;
            t.dir = td.dir;
            t.mode = (int8_t)(td.mode == 1 && degok && g.typed_adj && !c.Q->homo ? 2 : td.mode);
            t.known = known;
            t.rel = td.rel;
            t.label = lab;
            t.pin = pin;
            t.qdeg = p.qout | p.qin << 8;
        }
        const uint64_t sp = __ballot(spar);
        if (lane == 0) {
            g_s.revmask = rm;
            g_s.nnbl = n;
            g_s.skippar = sp != 0;
        }
    }
    __syncthreads();
    const int par = g_s.skippar ? -1 : st.parent;  // parent this step's marks intersect
    const int ncount = g_s.nnbl;
    if (n_items <= NW && g_s.revmask == 0) {
        // a handful of candidates: a wave each; those with a long row the
        // whole workgroup
        if (ncount > 0 || root >= 0)
            filter_items(c, LdsCtr{}, u, root, st.push != 0, g_s.nbl, ncount, ul, ub, 0, n_items, fb);
        __syncthreads();
        const int32_t nl = g_s.nbig;
        if (nl) {
            int32_t *def = defer_list(c, st);
            for (int32_t b = 0; b < nl; ++b)
                item_wg(c, st, g_s.nbl, ncount, ((const int32_t *)c.slab)[b], ub, fb, def);
            __syncthreads();
            if (def && g_s.ndef) fb += filter_far(u, st.push, st.parent, st.first, root, 3);
        }
    } else {
        fb += filter_far(u, st.push, st.parent, st.first, root, 0);
    }
    add_bytes_wave(c, fb);
    __syncthreads();
    // A step that failed leaves counts past the lists they belong to (a root
    // step appends its survivors as it goes, and counts them on past lcap):
    // nothing below may read a list by them. The query leaves the slot.
    if (aborted(c)) return 0;
    const bool shrunk = g_s.removed != 0 || g_s.rdrop != 0;
    if (g_s.removed) {
        const int32_t n = g_s.cnt[u];
        if (n <= 64) {
            // one wave's worth
            if (threadIdx.x < 64) {
                int32_t *l = c.L(u);
                const int32_t x = (int32_t)threadIdx.x < n ? l[threadIdx.x] : 0;
                const bool keep = (int32_t)threadIdx.x < n && bit_test(ub, x);
                const uint64_t m = __ballot(keep);
                if (keep) l[__popcll(m & lanemask_lt(threadIdx.x))] = x;
                if (threadIdx.x == 0) {
                    g_s.cnt[u] = __popcll(m);
                    add_bytes(c, 12ull * n + 4ull * __popcll(m));
                }
            }
            __syncthreads();
        } else {
            compact_far(u);
        }
    }
    bool pshrunk = false;  // the parent lost candidates
    if (par >= 0) {
        pshrunk = keep_marked(c, par);
    } else if (g_s.skippar && g_s.cnt[u] == 0) {
        // no candidate left to push the parent's single one
        const int p = st.parent;
        if (threadIdx.x == 0) {
            c.B(p)[c.L(p)[0] >> 6] = 0ull;
            g_s.cnt[p] = 0;
        }
        pshrunk = true;
        __syncthreads();
    }
    if (threadIdx.x < 64) {
        // what the step established: each test for all of C(u), and after an
        // explore step the other way round too (the children's and the
        // parent's candidates are the neighbours its survivors pushed)
        if (threadIdx.x == 0) {
            if (shrunk) ++g_s.ver[u];
            if (pshrunk) ++g_s.ver[st.parent];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (in) {
            g_s.okv[2 * td.e + td.dir] = g_s.ver[td.v];
            if (st.push) g_s.okv[2 * td.e + 1 - td.dir] = g_s.ver[u];
        }
    }
    const int32_t removed = g_s.removed + g_s.rdrop;
    __syncthreads();
    return removed;
}

// ---------------------------------------------------------------------------
// candidate edges (Sec. "Joining Phase"): for each key (a candidate of the
// key vertex, sorted), the sorted candidates of the other endpoint joined to
// it by a matching data edge. Space per key comes from the data degrees, so
// one pass writes the table: vals[off[i] .. off[i] + num[i]).
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool ec_hit(const DevGraph &g, int32_t rel, int32_t olabel,
                                       const uint64_t *other, const int2 *adj, int32_t beg,
                                       int32_t i, int32_t key) {
    const int2 e = adj[i];
    if (!adj_type_ok(g, e, olabel)) return false;
    if (rel >= 0) {
        if (!adj_rel_ok(g, e, rel)) return false;
    } else if (i > beg && adj[i - 1].x == e.x) {
        return false;  // same neighbour under another relation: one pair
    }
    return e.x != key && bit_test(other, e.x);
}

// first position in row adj[beg, end) (sorted by neighbour id, then
// relation) whose neighbour id is >= x
__device__ __forceinline__ int32_t row_lower_bound(const int2 *adj, int32_t beg, int32_t end,
                                                   int32_t x) {
    while (beg < end) {
        const int32_t mid = beg + ((end - beg) >> 1);
        if (adj[mid].x < x) beg = mid + 1;
        else end = mid;
    }
    return beg;
}

// does the row hold neighbour x under relation rel (-1: any relation)?
__device__ __forceinline__ bool row_has(const DevGraph &g, const int2 *adj, int32_t beg,
                                        int32_t end, int32_t x, int32_t rel) {
    for (int32_t i = row_lower_bound(adj, beg, end, x); i < end && adj[i].x == x; ++i)
        if (adj_rel_ok(g, adj[i], rel)) return true;
    return false;
}

// The same, one value for the whole wave (uniform call).
__device__ __forceinline__ bool wave_row_has(const DevGraph &g, const int2 *adj, int32_t beg,
                                             int32_t end, int32_t x, int32_t rel) {
    const int32_t b = wave_bound(beg, end, [&](int32_t i) { return adj[i].x < x; });
    // (a neighbour has one entry per relation: a few at most)
    for (int32_t i = b; i < end; i += 64) {
        const int32_t j = i + (int32_t)(threadIdx.x & 63);
        const int2 e = j < end ? adj[j] : make_int2(-1, -1);
        if (__ballot(e.x == x && adj_rel_ok(g, e, rel))) return true;
        if (__ballot(e.x != x)) return false;
    }
    return false;
}
constexpr int32_t kProbeOne = 4;  // values up to which a wave looks them up one by one

// Looking each of `no` candidates up in a row of `len` entries costs about
// no * log2(len) reads against len for a scan of the row.
__device__ __forceinline__ bool probe_cheaper(int32_t no, int32_t len) {
    return (int64_t)no * (33 - __clz(len | 1)) < (int64_t)len;
}

__device__ __forceinline__ uint64_t probe_bytes(int32_t no, int32_t len) {
    return (uint64_t)no * (4ull + 8ull * (uint64_t)(33 - __clz(len | 1)));
}

// one key, whole workgroup: the other endpoint's sorted candidates that the
// key's row holds, in order (the lookup form of ec_key_wg)
__device__ __forceinline__ int64_t ec_probe_wg(Ctx &c, int32_t rel, const int32_t *ol, int32_t no,
                                               const int2 *adj, int32_t beg, int32_t end, int32_t k,
                                               int32_t *dst) {
    int64_t n = 0;
    if (no <= kProbeOne) {
        // every wave does the same searches; the first one writes
        for (int32_t i = 0; i < no; ++i) {
            const int32_t x = ol[i];
            if (x == k || !wave_row_has(c.g, adj, beg, end, x, rel)) continue;
            if (threadIdx.x == 0) dst[n] = x;
            ++n;
        }
        return n;
    }
    for (int32_t base = 0; base < no; base += NT) {
        const int32_t i = base + threadIdx.x;
        const int32_t x = i < no ? ol[i] : -1;
        const bool hit = x >= 0 && x != k && row_has(c.g, adj, beg, end, x, rel);
        int64_t tot;
        const int64_t p = n + block_excl_scan<NW>(hit ? 1 : 0, g_s.sh, &tot);
        if (hit) dst[p] = x;
        n += tot;
    }
    return n;
}

// one key, one wave (wave-uniform call): lookup form of ec_key_wave
__device__ __forceinline__ int64_t ec_probe_wave(const Ctx &c, int32_t rel, const int32_t *ol, int32_t no,
                                                 const int2 *adj, int32_t beg, int32_t end,
                                                 int32_t k, int32_t *dst) {
    const int lane = threadIdx.x & 63;
    int64_t n = 0;
    if (no <= kProbeOne) {
        // a handful of values: the wave searches for one at a time
        for (int32_t i = 0; i < no; ++i) {
            const int32_t x = ol[i];
            if (x == k || !wave_row_has(c.g, adj, beg, end, x, rel)) continue;
            if (lane == 0) dst[n] = x;
            ++n;
        }
        return n;
    }
    for (int32_t base = 0; base < no; base += 64) {
        const int32_t i = base + lane;
        const int32_t x = i < no ? ol[i] : -1;
        const bool hit = x >= 0 && x != k && row_has(c.g, adj, beg, end, x, rel);
        const uint64_t bm = __ballot(hit);
        if (hit) dst[n + __popcll(bm & lanemask_lt(lane))] = x;
        n += __popcll(bm);
    }
    return n;
}

// one key, whole workgroup, ordered compaction in chunks of 4*NT entries
__device__ __forceinline__ int64_t ec_key_wg(Ctx &c, int32_t rel, int32_t olabel, const uint64_t *ob, const int2 *adj,
                             int32_t beg, int32_t end, int32_t k, int32_t *dst) {
    int64_t n = 0;
    for (int32_t base = beg; base < end; base += 4 * NT) {
        const int32_t i0 = base + 4 * threadIdx.x;
        uint32_t h = 0;  // bit t: entry i0 + t matches
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (i0 + t < end && ec_hit(c.g, rel, olabel, ob, adj, beg, i0 + t, k)) h |= 1u << t;
        int64_t tot;
        int64_t p = n + block_excl_scan<NW>(__popc(h), g_s.sh, &tot);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if ((h >> t) & 1u) dst[p++] = adj[i0 + t].x;
        n += tot;
    }
    return n;
}

// one key, one wave (wave-uniform call), same ordered output as ec_key_wg
__device__ __forceinline__ int64_t ec_key_wave(const Ctx &c, int32_t rel, int32_t olabel, const uint64_t *ob, const int2 *adj,
                                               int32_t beg, int32_t end, int32_t k, int32_t *dst) {
    const int lane = threadIdx.x & 63;
    int64_t n = 0;
    for (int32_t base = beg; base < end; base += 256) {
        const int32_t i0 = base + 4 * lane;
        uint32_t h = 0;  // bit t: entry i0 + t matches
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (i0 + t < end && ec_hit(c.g, rel, olabel, ob, adj, beg, i0 + t, k)) h |= 1u << t;
        const int32_t inc = wave_incl_scan32(__popc(h), lane);
        int64_t p = n + inc - __popc(h);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if ((h >> t) & 1u) dst[p++] = adj[i0 + t].x;
        n += __shfl(inc, 63, 64);
    }
    return n;
}

// Keys [i0, i1) of a table build, G lanes per key; keys whose rows are
// longer than 64 * G entries go to E.ovl (counted by *nbig) for the wave
// tier. Returns the entries this thread's groups wrote (on their first lane).
__device__ __forceinline__ int64_t ec_keys(const Ctx &c, const EcJob &Ej, int32_t i0, int32_t i1,
                                           int G, int32_t *nbig, uint64_t &fb) {
    const EcJob E = Ej;  // once, before the stores below
    const int32_t *off = c.g.off(E.dir);
    const int2 *adj = c.g.adj(E.dir);
    const int NGr = NT / G;
    const int lane = threadIdx.x & 63, gl = lane & (G - 1), gb = lane & ~(G - 1);
    const uint64_t gmask = (G == 64 ? ~0ull : ((1ull << G) - 1ull)) << gb;
    const int32_t bigdeg = 64 * G;
    int64_t mytot = 0;
    for (int32_t it = i0 + (int32_t)threadIdx.x / G; it < i1; it += NGr) {
        const int32_t k = E.keys[it];
        const int32_t beg = off[k], end = off[k + 1];
        if (end - beg > bigdeg) {
            if (gl == 0) E.ovl[atomicAdd(nbig, 1)] = it;
            continue;
        }
        int32_t *dst = E.vals + E.degoff[it];
        int32_t n = 0;
        for (int32_t base = beg; base < end; base += G) {
            const int32_t i = base + gl;
            const bool hit = i < end && ec_hit(c.g, E.rel, E.olabel, E.ob, adj, beg, i, E.homo ? -1 : k);
            const uint64_t bm = __ballot(hit) & gmask;
            if (hit) dst[n + __popcll(bm & lanemask_lt(lane))] = adj[i].x;
            n += __popcll(bm);
        }
        if (gl == 0) {
            E.num[it] = n;
            mytot += n;
            fb += 16ull + 12ull * (end - beg) + 4ull * n;
        }
    }
    return mytot;
}

// Long keys E.items[i0, i1), one wave each (scan or lookup, whichever
// reads less); keys with rows above wg_rows go to E.ovl for the owner's
// workgroup tier. Returns the entries written (on lane 0 of each wave).
__device__ __forceinline__ int64_t ec_long_keys(const Ctx &c, const EcJob &Ej, int32_t i0,
                                                int32_t i1, int32_t *ngiant, uint64_t &fb) {
    const EcJob E = Ej;
    const int32_t *off = c.g.off(E.dir);
    const int2 *adj = c.g.adj(E.dir);
    const int lane = threadIdx.x & 63;
    int64_t mytot = 0;
    for (int32_t b = i0 + (int32_t)(threadIdx.x >> 6); b < i1; b += NW) {
        const int32_t it = E.items[b];
        const int32_t k = E.keys[it];
        const int32_t beg = off[k], end = off[k + 1];
        if (end - beg > c.wg_rows) {
            if (lane == 0) E.ovl[atomicAdd(ngiant, 1)] = it;
            continue;
        }
        const bool probe = probe_cheaper(E.no, end - beg);
        int32_t *dst = E.vals + E.degoff[it];
        const int32_t ks = E.homo ? -1 : k;  // -1: the key may pair with itself
        const int64_t n = probe ? ec_probe_wave(c, E.rel, E.ol, E.no, adj, beg, end, ks, dst)
                                : ec_key_wave(c, E.rel, E.olabel, E.ob, adj, beg, end, ks, dst);
        if (lane == 0) {
            E.num[it] = (int32_t)n;
            mytot += n;
            fb += 16ull + 4ull * n + (probe ? probe_bytes(E.no, end - beg) : 12ull * (end - beg));
        }
    }
    return mytot;
}

// Keys with rows above wg_rows, E.items[i0, i1), the whole workgroup each.
// Returns the entries written (on thread 0).
__device__ __forceinline__ int64_t ec_giant_keys(Ctx &c, const EcJob &Ej, int32_t i0, int32_t i1,
                                                 uint64_t &fb) {
    const EcJob E = Ej;
    const int32_t *off = c.g.off(E.dir);
    const int2 *adj = c.g.adj(E.dir);
    int64_t mytot = 0;
    for (int32_t b = i0; b < i1; ++b) {
        const int32_t it = E.items[b];
        const int32_t k = E.keys[it];
        const int32_t beg = off[k], end = off[k + 1];
        const bool probe = probe_cheaper(E.no, end - beg);
        int32_t *dst = E.vals + E.degoff[it];
        const int32_t ks = E.homo ? -1 : k;
        const int64_t n = probe ? ec_probe_wg(c, E.rel, E.ol, E.no, adj, beg, end, ks, dst)
                                : ec_key_wg(c, E.rel, E.olabel, E.ob, adj, beg, end, ks, dst);
        if (threadIdx.x == 0) {
            E.num[it] = (int32_t)n;
            mytot += n;
            fb += 16ull + 4ull * n + (probe ? probe_bytes(E.no, end - beg) : 12ull * (end - beg));
        }
    }
    return mytot;
}

// One chunk of a shared table build (owner or helper): the keys, and the
// chunk's entry count added to the board.
__device__ __forceinline__ void ec_chunk(Ctx &c, const EcJob &E, HelpJob *j, int32_t i0, int32_t i1,
                                         int G, uint64_t &fb) {
    int64_t t = E.tier == 2   ? ec_giant_keys(c, E, i0, i1, fb)
                : E.tier == 1 ? ec_long_keys(c, E, i0, i1, &j->nbig, fb)
                              : ec_keys(c, E, i0, i1, G, &j->nbig, fb);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if ((threadIdx.x & 63) == 0 && t) atomicAdd(&j->jrows, (unsigned long long)t);
}

// One shared pass of a table build (nch chunks of K items); adds the
// entries written to mytot (thread 0). False when the owner gave up on its
// helpers: the query is aborted (and rerun) and the build stops, since key
// lists of unreported chunks may be incomplete.
__device__ __forceinline__ bool ec_shared(Ctx &c, int e, const EcJob &E, int32_t n_items,
                                          int32_t K, int G, const int32_t *ovl, uint64_t &fb,
                                          int64_t &mytot) {
    shared_job(c, 3, NStep{}, nullptr, 0, nullptr, nullptr, n_items, K, G,
               (n_items + K - 1) / K, nullptr, fb, &E);
    if (aborted(c)) {
        if (threadIdx.x == 0) {
            g_s.ectot[e] = 0;
            g_s.slab_used = (int64_t)((const char *)ovl - c.slab);
        }
        __syncthreads();
        return false;
    }
    if (threadIdx.x == 0)
        mytot += (int64_t)__hip_atomic_load(&c.job->jrows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return true;
}

// Build the table of query edge e keyed by `key` (dir 0: keys are sources).
// Sets s.ec_offs/ec_cnt/ec_vals[e], s.eckey[e] and s.ectot[e]. Tiers: G
// lanes per key; one wave per key for rows above 64 G entries; the whole
// workgroup per key above wg_rows. With a helper board, each tier with
// enough keys is shared like a filter step (its chunks write disjoint keys
// of the one-pass layout).
__device__ __forceinline__ void ec_build(Ctx &c, int e, int key, int other, int dir) {
    const DevGraph &g = c.g;
    const int32_t *keys = c.L(key);
    const int32_t nk = g_s.cnt[key];
    const uint64_t *ob = c.B(other);
    const int32_t *ol = c.L(other);  // sorted
    const int32_t no = g_s.cnt[other];
    const int32_t rel = c.Q->elabel[e];
    const int32_t *off = g.off(dir);
    const int2 *adj = g.adj(dir);
    int32_t *degoff = (int32_t *)slab_alloc(c, 4ll * nk + 4);
    int32_t *num = (int32_t *)slab_alloc(c, 4ll * nk + 4);
    if (!degoff || !num) return;
    // exclusive scan of the keys' degrees: space per key
    int64_t carry = 0;
    for (int32_t base = 0; base < nk; base += NT) {
        const int32_t i = base + threadIdx.x;
        const int32_t d = i < nk ? off[keys[i] + 1] - off[keys[i]] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan<NW>(d, g_s.sh, &tot);
        if (i < nk) degoff[i] = (int32_t)(carry + ex);
        carry += tot;
    }
    int32_t *vals = (int32_t *)slab_alloc(c, 4 * carry + 4);
    if (!vals) return;
    // keys with long rows, for the wave and workgroup tiers; given back
    // to the slab at the end
    int32_t *ovl = (int32_t *)slab_alloc(c, 4ll * nk + 4);
    if (!ovl) return;
    if (threadIdx.x == 0) {
        degoff[nk] = (int32_t)carry;
        g_s.ec_offs[e] = degoff;
        g_s.ec_cnt[e] = num;
        g_s.ec_vals[e] = vals;
        g_s.eckey[e] = key;
        g_s.nbig = 0;
        g_s.ngiant = 0;
    }
    __syncthreads();
    int64_t mytot = 0;
    uint64_t fb = 0;
    const bool can_share = c.help_items > 0 && c.job;
    const int32_t homo = c.Q->homo;
    const int32_t olabel = c.Q->pred[other].label;
    const EcJob E{keys, degoff, num, vals, ovl, ob, ol, nullptr, nk, rel, dir, no, 0, olabel, homo};
    if (nk <= NW) {
        // a handful of keys: one wave each, rows above wg_rows get the
        // whole workgroup
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (wave < nk) {
            const int32_t k = keys[wave];
            const int32_t beg = off[k], end = off[k + 1];
            if (end - beg > c.wg_rows) {
                if (lane == 0) g_s.big[atomicAdd(&g_s.ngiant, 1)] = wave;  // at most NW
            } else {
                const bool probe = probe_cheaper(no, end - beg);
                const int32_t ks = homo ? -1 : k;
                const int64_t n = probe ? ec_probe_wave(c, rel, ol, no, adj, beg, end, ks, vals + degoff[wave])
                                        : ec_key_wave(c, rel, olabel, ob, adj, beg, end, ks, vals + degoff[wave]);
                if (lane == 0) {
                    num[wave] = (int32_t)n;
                    mytot += n;
                    fb += 16ull + 4ull * n + (probe ? probe_bytes(no, end - beg) : 12ull * (end - beg));
                }
            }
        }
    }
    // tiers: G lanes per key, one wave per long key, one workgroup per key
    // with a row above wg_rows; each shared from the same place when it has
    // enough keys
    for (int tier = nk <= NW ? 2 : 0; tier < 3; ++tier) {
        const int lane = threadIdx.x & 63;
        EcJob E1 = E;
        E1.tier = tier;
        int32_t nsh = 0, K = 1;  // items to share (0: none), per chunk
        int G = 64;
        if (tier == 0) {
            if (can_share && nk >= c.help_items) {
                const int32_t helpers = helpers_now(c);
                nsh = nk;
                K = chunk_items(nk, helpers, 64, 512);
                G = lanes_for(K, c.gmax);
            } else {
                mytot += ec_keys(c, E, 0, nk, lanes_for(nk, c.gmax), &g_s.nbig, fb);
            }
        } else if (tier == 1) {
            __syncthreads();
            const int32_t nl = g_s.nbig;
            if (can_share && nl >= kLongShare) {
                // the keys move to a list of their own; rows longer than
                // wg_rows come back to ovl
                int32_t *items = (int32_t *)slab_alloc(c, 4ll * nl + 4);
                if (!items) return;
                for (int32_t i = threadIdx.x; i < nl; i += NT) items[i] = ovl[i];
                __syncthreads();
                if (threadIdx.x == 0) g_s.nbig = 0;
                E1.items = items;
                nsh = nl;
                K = kLongChunk;
            }
        } else {
            __syncthreads();
            const int32_t nbig = nk <= NW ? 0 : g_s.nbig;
            for (int32_t b = threadIdx.x >> 6; b < nbig; b += NW) {
                const int32_t it = ovl[b];
                const int32_t k = keys[it];
                const int32_t beg = off[k], end = off[k + 1];
                if (end - beg > c.wg_rows) {
                    int32_t p = 0;
                    if (lane == 0) p = atomicAdd(&g_s.ngiant, 1);
                    p = __shfl(p, 0, 64);
                    if (p < kBigCap) {
                        if (lane == 0) g_s.big[p] = it;
                        continue;
                    }
                }
                const bool probe = probe_cheaper(no, end - beg);
                const int32_t ks = homo ? -1 : k;
                const int64_t n = probe ? ec_probe_wave(c, rel, ol, no, adj, beg, end, ks, vals + degoff[it])
                                        : ec_key_wave(c, rel, olabel, ob, adj, beg, end, ks, vals + degoff[it]);
                if (lane == 0) {
                    num[it] = (int32_t)n;
                    mytot += n;
                    fb += 16ull + 4ull * n + (probe ? probe_bytes(no, end - beg) : 12ull * (end - beg));
                }
            }
            __syncthreads();
            const int32_t ngiant = min(g_s.ngiant, kBigCap);
            if (can_share && ngiant >= 2) {
                int32_t *items = (int32_t *)slab_alloc(c, 4ll * ngiant + 4);
                if (!items) return;
                for (int32_t i = threadIdx.x; i < ngiant; i += NT) items[i] = g_s.big[i];
                __syncthreads();
                E1.items = items;
                nsh = ngiant;
                G = NT;
            } else if (ngiant > 0) {
                E1.items = g_s.big;
                mytot += ec_giant_keys(c, E1, 0, ngiant, fb);
            }
        }
        if (nsh > 0 && !ec_shared(c, e, E1, nsh, K, G, ovl, fb, mytot)) return;
    }
    add_bytes_wave(c, fb);
    int64_t tot;
    block_excl_scan<NW>(mytot, g_s.sh, &tot);
    if (threadIdx.x == 0) {
        g_s.ectot[e] = tot;
        g_s.slab_used = (int64_t)((char *)ovl - c.slab);  // the last allocation
    }
    __syncthreads();
}

__device__ __attribute__((noinline)) void ec_build_far(int e, int key, int other, int dir) {
    SGM_OWN_CTX(c);
    ec_build(c, __builtin_amdgcn_readfirstlane(e), __builtin_amdgcn_readfirstlane(key),
             __builtin_amdgcn_readfirstlane(other), __builtin_amdgcn_readfirstlane(dir));
}

// Tables of the edges in `mask` whose key vertex has up to kFewKeys
// candidates, with rows of at most wg_rows entries (dir as in ec_build),
// built together: one wave per (edge, key) and one slab allocation for all of
// them, instead of the barriers and allocations of a full build per edge (8 us
// each). Returns the edges built (uniform). Uses the dynamic LDS, which no
// other phase holds meanwhile.
constexpr int kFewKeys = 8;
static_assert(SGM_MAX_QE * kFewKeys <= NT, "a thread per (edge, key)");

__device__ __forceinline__ uint64_t ec_build_few(Ctx &c, uint64_t mask, int dir) {
    const DevGraph &g = c.g;
    const NQuery &Q = *c.Q;
    Smem &s = g_s;
    const int2 *adj = g.adj(dir);
    // per thread t = (edge t / kFewKeys, key t % kFewKeys), for the waves
    struct Task {
        int32_t key, beg, end, at;  // at: first value in the edge's array
    };
    Task *task = (Task *)g_dyn;                      // [NT]
    int32_t *esz = (int32_t *)(task + NT);           // [SGM_MAX_QE] bytes of each table, 0: not here
    int32_t *epos = esz + SGM_MAX_QE;                // [SGM_MAX_QE] byte offset in the allocation
    int32_t *list = epos + SGM_MAX_QE;               // [NT] tasks
    int32_t *meta = list + NT;                       // [0] tasks, [1] bytes
    const int t = threadIdx.x, e = t / kFewKeys, i = t % kFewKeys;
    const int lane = t & 63, wid = t >> 6;
    const bool in = e < Q.m && ((mask >> e) & 1ull);
    const int kv = in ? (dir ? Q.edst[e] : Q.esrc[e]) : 0;
    const int32_t nk = in ? s.cnt[kv] : 0;
    const bool on = in && nk <= kFewKeys && i < nk;
    int32_t len = 0;
    Task tk{-1, 0, 0, 0};
    if (on) {
        tk.key = c.L(kv)[i];
        const int4 r = g.vrow[tk.key];
        tk.beg = dir ? r.z : r.x;
        tk.end = dir ? r.w : r.y;
        len = tk.end - tk.beg;
    }
    // the edge's rows side by side; a row above wg_rows leaves the edge out
    const uint64_t grp = 0xffull << (lane & ~(kFewKeys - 1));
    const bool big = (__ballot(on && len > min(c.wg_rows, 32768)) & grp) != 0;
    int32_t inc = len;
#pragma unroll
    for (int o = 1; o < kFewKeys; o <<= 1) {
        const int32_t y = __shfl_up(inc, o, kFewKeys);
        if (i >= o) inc += y;
    }
    const int32_t sum = __shfl(inc, kFewKeys - 1, kFewKeys);
    tk.at = inc - len;
    const bool here = on && !big;
    if (t == 0) meta[0] = 0;
    // offsets [nk + 1], counts [nk], values [sum], rounded to 16 bytes
    if (i == 0 && e < SGM_MAX_QE) esz[e] = here ? (4 * (2 * nk + 1 + sum) + 15) & ~15 : 0;
    task[t] = tk;
    __syncthreads();
    if (here) list[atomicAdd(&meta[0], 1)] = t;
    if (wid == 0) {
        // exclusive scan of the tables' sizes
        const int32_t sz = esz[lane];
        const int32_t ic = wave_incl_scan32(sz, lane);
        epos[lane] = ic - sz;
        if (lane == 63) meta[1] = ic;
        if (sz) s.ectot[lane] = 0;
    }
    __syncthreads();
    const int32_t nt = meta[0];
    if (nt == 0) return 0ull;
    char *base = slab_alloc(c, meta[1]);
    if (!base) return 0ull;
    if (here) {
        int32_t *degoff = (int32_t *)(base + epos[e]);
        degoff[i] = tk.at;
        if (i == nk - 1) degoff[nk] = sum;
        if (i == 0) {
            s.ec_offs[e] = degoff;
            s.ec_cnt[e] = degoff + nk + 1;
            s.ec_vals[e] = degoff + 2 * nk + 1;
            s.eckey[e] = kv;
        }
    }
    __syncthreads();
    uint64_t fb = 0;
    for (int q = wid; q < nt; q += NW) {
        const int ti = list[q], ed = ti / kFewKeys, ki = ti % kFewKeys;
        const Task w = task[ti];
        const int other = dir ? Q.esrc[ed] : Q.edst[ed];
        const int32_t no = s.cnt[other], rel = Q.elabel[ed], wl = w.end - w.beg;
        int32_t *vals = s.ec_vals[ed] + w.at;
        const bool probe = probe_cheaper(no, wl);
        const int32_t ks = Q.homo ? -1 : w.key;
        const int64_t n = probe ? ec_probe_wave(c, rel, c.L(other), no, adj, w.beg, w.end, ks, vals)
                                : ec_key_wave(c, rel, Q.pred[other].label, c.B(other), adj, w.beg, w.end, ks, vals);
        if (lane == 0) {
            s.ec_cnt[ed][ki] = (int32_t)n;
            if (n) atomicAdd((unsigned long long *)&s.ectot[ed], (unsigned long long)n);
            fb += 28ull + 4ull * n + (probe ? probe_bytes(no, wl) : 12ull * wl);
        }
    }
    add_bytes_wave(c, fb);
    uint64_t built = 0;
    for (int q = 0; q < Q.m; ++q) built |= (uint64_t)(esz[q] != 0) << q;
    __syncthreads();
    return built;
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = min(x, (uint64_t)__shfl_xor(x, o, 64));
    return x;
}

// Join order of Sec. "Joining Phase", by wave 0 with one query edge per
// lane: start from the source of the edge with the fewest candidate edges;
// bind one new vertex per level through the cheapest edge with exactly one
// bound endpoint (policy 1: first the new vertex with the most edges to
// bound vertices), the earliest edge on ties; all other unused edges between
// the new vertex and bound vertices are checks of that level.
__device__ __forceinline__ void join_order(Ctx &c) {
    if (threadIdx.x >= 64) return;
    const NQuery &Q = *c.Q;
    Smem &s = g_s;
    const int lane = threadIdx.x;
    const bool has = lane < Q.m;
    const int xs = has ? s.qsrc[lane] : 0, xd = has ? s.qdst[lane] : 0;
    const uint64_t cost = has ? (uint64_t)min(s.ectot[lane], (int64_t)((1ll << 52) - 1)) : 0ull;
    uint32_t vis = 0;   // bound query vertices
    uint64_t used = 0;  // consumed query edges
    int ext = (int)(wave_min_u64(has ? (cost << 6) | (uint64_t)lane : ~0ull) & 63);
    int w = s.qsrc[ext];
    if (lane == 0) s.jorder[0] = w;
    vis |= 1u << w;
    int nc = 0;
    for (int lv = 0; lv < Q.n - 1; ++lv) {
        const bool va = (vis >> xs) & 1u, vb = (vis >> xd) & 1u;
        if (lv > 0) {
            const bool cand = has && !((used >> lane) & 1ull) && va != vb;
            const int wv = va ? xd : xs;  // the endpoint a candidate would bind
            int links = 0;
            if (c.join_policy == 1)
                for (int x = 0; x < Q.n; ++x) {
                    const uint64_t m = __ballot(cand && wv == x);
                    if (wv == x) links = __popcll(m);
                }
            const uint64_t key =
                cand ? ((uint64_t)(63 - links) << 58) | (cost << 6) | (uint64_t)lane : ~0ull;
            ext = (int)(wave_min_u64(key) & 63);
        }
        w = ((vis >> s.qsrc[ext]) & 1u) ? s.qdst[ext] : s.qsrc[ext];
        used |= 1ull << ext;
        const bool chk = has && !((used >> lane) & 1ull) &&
                         ((xs == w && ((vis >> xd) & 1u)) || (xd == w && ((vis >> xs) & 1u)));
        const uint64_t cm = __ballot(chk);
        if (chk) s.chk[nc + __popcll(cm & lanemask_lt(lane))] = lane;
        if (lane == 0) {
            s.lv_ext[lv] = ext;
            s.lv_first[lv] = nc;
            s.lv_nchk[lv] = __popcll(cm);
            s.jorder[lv + 1] = w;
        }
        nc += __popcll(cm);
        used |= cm;
        vis |= 1u << w;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < Q.n) s.jpos[s.jorder[lane]] = lane;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (has) s.eckey[lane] = s.jpos[xs] < s.jpos[xd] ? xs : xd;
}

// Shared join levels: a chunk is one block of NT parent rows, or 1/nsub of
// its pairs (every nsub-th block of NT pairs) when the level's pairs are
// few rows with long fan-outs; about kJoinChunkPairs pairs per chunk. A
// level of at least kJoinSharePairs pairs is shared with the launch's idle
// workgroups (those that become idle while it runs join in too).
constexpr int64_t kJoinChunkPairs = 16384;
constexpr int64_t kJoinSharePairs = 2 * kJoinChunkPairs;
constexpr int kJoinMaxSub = 64;
// blocks of rows from which a level counted row by row is shared
constexpr int64_t kCountShareBlocks = 4;
// blocks of pairs whose accepted rows take one output reservation (shared
// levels): up to 4 NT pairs, staged per wave in LDS
constexpr int kJoinGroup = 4;

// A level's block of parent rows, staged in LDS behind the waves' staged
// output rows: every pair tests its new value against the whole row and every
// accepted pair copies it, which from global memory was a chain of k dependent
// reads per pair (a 14-column level of 22,000 pairs: 1.0 ms in one workgroup).
constexpr int kJoinStageRows = NW * 512 * (int)sizeof(int32_t);
static_assert(kJoinStageRows + NT * (SGM_MAX_QV - 1) * sizeof(int32_t) <= kDynLds, "parent rows");

// Pair i of a block: its row rr within the block of parent rows (the last
// whose pair offset is <= pi), its new value x, and whether the extended
// row passes the injectivity test and every check edge of the level
// (Sec. "Joining Phase").
__device__ __forceinline__ bool join_pair(const Smem &s, const JLevel &L, const int32_t *rows,
                                          int64_t pi, int32_t *rr_out, int32_t *x_out,
                                          uint64_t &jb) {
    int32_t a0 = 0;
#pragma unroll
    for (int st = NT / 2; st > 0; st >>= 1)
        if (s.pairoff[a0 + st] <= pi) a0 += st;
    const int32_t x = L.evals[s.rowlo[a0] + (pi - s.pairoff[a0])];
    const int k = L.k;
    const int32_t *row = rows + a0 * k;
    bool ok = true;
    for (uint32_t m = L.cmask; m; m &= m - 1) ok &= row[__builtin_ctz(m)] != x;
    for (int ci = 0; ci < L.nchk && ok; ++ci) {
        // the check edge's values for the row's key vertex hold x
        const JChk &h = L.chk[ci];
        const int32_t kval = row[h.col];
        const int32_t i = lower_bound_i32(h.kl, 0, h.nkl, kval);
        if (i >= h.nkl || h.kl[i] != kval) {
            ok = false;
        } else {
            const int32_t vlo = h.offs[i], vhi = vlo + h.cnt[i];
            const int32_t jx = lower_bound_i32(h.vals, vlo, vhi, x);
            ok = jx < vhi && h.vals[jx] == x;
        }
    }
    jb += 4ull + 4ull * k + 24ull * L.nchk + (ok && !L.count ? 4ull * (k + 1) : 0ull);
    *rr_out = a0;
    *x_out = x;
    return ok;
}

// Copy a wave's n staged output rows (parent row within the block, new
// value) to out[base, base + n), consecutive lanes on consecutive ints.
__device__ __forceinline__ void join_put(const JLevel &L, const int32_t *rows, const int32_t *wrr,
                                         const int32_t *wx, int n, int64_t base, int lane) {
    const int k = L.k, w = k + 1;
    // e / w by a 16-bit reciprocal: exact for e < 4096, w <= 16
    const uint32_t inv = (65536u + (uint32_t)w - 1u) / (uint32_t)w;
    int32_t *dst = L.out + base * w;
#pragma unroll 4
    for (int e = lane; e < n * w; e += 64) {
        const int rw = (int)(((uint32_t)e * inv) >> 16);
        const int cc = e - rw * w;
        dst[e] = cc < k ? rows[wrr[rw] * k + cc] : wx[rw];
    }
}

// Rows [r0, r1) of join level L (at most NT of them): each row's fan-out
// (the candidate-edge count of its parent vertex's value), then its pairs
// in blocks of NT, the accepted rows appended to L.out.
// Owner alone (SHARED false): every block of pairs, output places by one
// LDS atomic per wave. SHARED: the blocks sub, sub + nsub, ... only, and
// the accepted rows of up to kJoinGroup of them take their places with one
// device-scope atomic on *gctr.
// A counting level (L.count, the last of a count-only query) writes no rows:
// its accepted pairs are counted, and without check edges not even looked at,
// since a row's pairs are its fan-out less the values of the row itself that
// its candidate edges hold. Counts go to s.cnt64, or to *gctr when SHARED.
template <bool SHARED>
__device__ __forceinline__ void join_rows(Ctx &c, const JLevel &L, int64_t r0, int64_t r1,
                                          int32_t sub, int32_t nsub, unsigned long long *gctr,
                                          int32_t *gabort, uint64_t &jb) {
    Smem &s = g_s;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t r = r0 + threadIdx.x;
    int32_t *rows = (int32_t *)(g_dyn + kJoinStageRows);
    {
        const int32_t *src = L.table + r0 * L.k;
        const int nint = (int)(r1 - r0) * L.k;
#pragma unroll 4
        for (int i = threadIdx.x; i < nint; i += NT) rows[i] = src[i];
    }
    __syncthreads();
    int32_t fan = 0, lo = 0;
    if (r < r1) {
        const int32_t pv = rows[threadIdx.x * L.k + L.cp];
        const int32_t i = lower_bound_i32(L.pk, 0, L.npk, pv);
        if (i < L.npk && L.pk[i] == pv) {
            lo = L.eoffs[i];
            fan = L.ecnt[i];
        }
        jb += 16ull + 4ull * (32 - __clz(L.npk | 1));
    }
    if (L.count && L.nchk == 0) {
        int64_t mine = fan;
        const int32_t *row = rows + threadIdx.x * L.k;
        if (fan > 0)
            for (uint32_t m = L.cmask; m; m &= m - 1) {
                const int32_t x = row[__builtin_ctz(m)];
                const int32_t j = lower_bound_i32(L.evals, lo, lo + fan, x);
                mine -= j < lo + fan && L.evals[j] == x;
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
        if (lane == 0 && mine) atomicAdd(SHARED ? gctr : &s.cnt64, (unsigned long long)mine);
        __syncthreads();
        return;
    }
    int64_t tot;
    const int64_t ex = block_excl_scan<NW>(fan, s.sh, &tot);
    if (tot > INT32_MAX) {
        // more pairs than a block's offsets hold: the multi-kernel path
        if (threadIdx.x == 0) {
            if (SHARED) atomicExch(gabort, kWhySlab);
            else s.abort_ = kWhySlab;
            s.need = INT64_MAX;
        }
        __syncthreads();
        return;
    }
    if (!SHARED && !L.count && L.rows <= NT && tot > kPairSlack * L.cap) {
        // the level's only block of rows: its pairs bound the level, so a
        // level that could not fit even a much larger slot stops here
        if (threadIdx.x == 0) {
            s.abort_ = kWhySlab;
            s.need = (int64_t)((const char *)L.out - c.slab) + tot * 4 * (L.k + 1);
        }
        __syncthreads();
        return;
    }
    s.pairoff[threadIdx.x] = (int32_t)ex;
    s.rowlo[threadIdx.x] = lo;
    __syncthreads();
    int32_t *wrr = (int32_t *)g_dyn + wid * 512;  // this wave's staged rows
    int32_t *wx = wrr + 256;
    if (L.count) {
        const int64_t nblk = (tot + NT - 1) / NT;
        int64_t mine = 0;
        for (int64_t bi = SHARED ? sub : 0; bi < nblk; bi += SHARED ? nsub : 1) {
            const int64_t pi = bi * NT + threadIdx.x;
            int32_t rr, x;
            mine += pi < tot && join_pair(s, L, rows, pi, &rr, &x, jb);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
        if (lane == 0 && mine) atomicAdd(SHARED ? gctr : &s.cnt64, (unsigned long long)mine);
    } else if (!SHARED) {
        for (int64_t pb = 0; pb < tot; pb += NT) {
            const int64_t pi = pb + threadIdx.x;
            int32_t rr = 0, x = 0;
            const bool ok = pi < tot && join_pair(s, L, rows, pi, &rr, &x, jb);
            const uint64_t bm = __ballot(ok);
            const int nok = __popcll(bm);
            int32_t base = 0;
            const int leader = bm ? __builtin_ctzll(bm) : 0;
            if (bm && lane == leader) base = atomicAdd(&s.ctr, nok);
            base = __shfl(base, leader, 64);
            if (ok) {
                const int j = __popcll(bm & lanemask_lt(lane));
                wrr[j] = rr;
                wx[j] = x;
            }
            wave_sync();
            if ((int64_t)base + nok > L.cap) {
                if (lane == 0) s.abort_ = kWhySlab;
            } else {
                join_put(L, rows, wrr, wx, nok, base, lane);
            }
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        const int64_t nblk = (tot + NT - 1) / NT;
        int par = 0;
        for (int64_t i0 = sub; i0 < nblk; i0 += (int64_t)nsub * kJoinGroup, par ^= 1) {
            int wn = 0;
            for (int t = 0; t < kJoinGroup; ++t) {
                const int64_t bi = i0 + (int64_t)t * nsub;
                if (bi >= nblk) break;
                const int64_t pi = bi * NT + threadIdx.x;
                int32_t rr = 0, x = 0;
                const bool ok = pi < tot && join_pair(s, L, rows, pi, &rr, &x, jb);
                const uint64_t bm = __ballot(ok);
                if (ok) {
                    const int j = wn + __popcll(bm & lanemask_lt(lane));
                    wrr[j] = rr;
                    wx[j] = x;
                }
                wn += __popcll(bm);
            }
            wave_sync();
            // one reservation for the group's accepted rows (two buffers: a
            // wave may run one group ahead)
            if (lane == 0) s.wnok[par][wid] = wn;
            __syncthreads();
            if (threadIdx.x == 0) {
                int32_t t = 0;
                for (int w = 0; w < NW; ++w) t += s.wnok[par][w];
                s.wbase[par] = t ? (int64_t)atomicAdd(gctr, (unsigned long long)t) : 0;
            }
            __syncthreads();
            int64_t base = s.wbase[par];
            for (int w = 0; w < wid; ++w) base += s.wnok[par][w];
            if (base + wn > L.cap) {
                if (lane == 0 && wn) atomicExch(gabort, kWhySlab);
            } else {
                join_put(L, rows, wrr, wx, wn, base, lane);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
}

// Chunk ch of a shared level: its block of parent rows and its share of
// that block's pairs.
__device__ __forceinline__ void join_chunk(Ctx &c, const JLevel &L, int32_t ch,
                                           unsigned long long *gctr, int32_t *gabort,
                                           uint64_t &jb) {
    const int64_t b = ch / L.nsub;
    const int64_t r0 = b * NT;
    join_rows<true>(c, L, r0, min(L.rows, r0 + NT), ch % L.nsub, L.nsub, gctr, gabort, jb);
}

// A join level shared through this slot's board entry (kind 2): the level's
// view goes to the entry, its parent rows are cut into nch chunks that the
// owner and idle workgroups claim, output rows are placed through the
// entry's counter; the owner waits for the chunks its helpers claimed (the
// same protocol as a shared filter step) and takes the row count into
// s.ctr.
__device__ __forceinline__ void shared_join(Ctx &c, int32_t nch, uint64_t &jb) {
    HelpJob *j = c.job;
    Smem &s = g_s;
    {
        const uint64_t *src = (const uint64_t *)&s.jl;
        uint64_t *dst = (uint64_t *)&j->jl;
        for (int i = threadIdx.x; i < (int)(sizeof(JLevel) / 8); i += NT) dst[i] = src[i];
    }
    if (threadIdx.x == 0) {
        j->jrows = 0ull;
        j->abort_ = 0;
        j->bytes = 0ull;
        j->done = 0;
        j->kind = 2;
        j->chunk = 0;
        j->q = c.q;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t seq =
            claim_seq(__hip_atomic_load(&j->claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) + 1u;
        // the level's view, tables and edge tables before the claim word
        __threadfence();
        atomicExch(&j->claim, claim_word(seq, nch));
        atomicAdd(&c.hctr[0], 1);
    }
    __syncthreads();
    int32_t own = 0;
    for (;;) {
        if (threadIdx.x == 0) {
            const unsigned long long w = take_chunk(j);
            s.hch = claim_next(w) < claim_nch(w) ? claim_next(w) : -1;
        }
        __syncthreads();
        const int32_t ch = s.hch;
        __syncthreads();
        if (ch < 0) break;
        join_chunk(c, s.jl, ch, &j->jrows, &j->abort_, jb);
        ++own;
    }
    ev(c, SGM_EV_SHARED);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t got = atomicAdd(&j->done, own) + own;
        int64_t n = 0;
        while (got < nch && n < c.help_wait) {
            __builtin_amdgcn_s_sleep(1);
            got = __hip_atomic_load(&j->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ++n;
        }
        if (got < nch) {
            // give up as a filter step does: no further claims, and the
            // slot stays out of use until the next launch clears it
            const uint32_t seq = claim_seq(
                __hip_atomic_load(&j->claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            atomicExch(&j->claim, claim_word(seq, 0));
            atomicExch(&j->dirty, 1);
            s.retired = 1;
        }
        // the helpers' rows, written before their reports
        __threadfence();
        atomicSub(&c.hctr[0], 1);
        const unsigned long long placed =
            __hip_atomic_load(&j->jrows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s.cnt64 = placed;
        s.ctr = (int32_t)min((unsigned long long)s.jl.cap, placed);
        const int32_t ab = __hip_atomic_load(&j->abort_, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ab) s.abort_ = ab;
        if (!s.jl.count && placed > (unsigned long long)s.jl.cap) s.abort_ = kWhySlab;
        if (got < nch) s.abort_ = kWhyHelp;
        add_bytes(c, __hip_atomic_load(&j->bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __syncthreads();
}

__device__ __attribute__((noinline)) uint64_t shared_join_far(int32_t nch) {
    SGM_OWN_CTX(c);
    uint64_t jb = 0;
    shared_join(c, __builtin_amdgcn_readfirstlane(nch), jb);
    return jb;
}

// ---------------------------------------------------------------------------
// final ordering helpers
// ---------------------------------------------------------------------------

// Sort key of a row: the ranks of its values within their (sorted) candidate
// lists, concatenated in query-vertex order (s.bitsn bits each; a column of
// a single candidate has rank 0 and no bits). The binary searches of up to
// eight columns advance together, so their probes are independent loads;
// s.kdepth steps bring every search to its end.
__device__ __forceinline__ uint64_t row_key(const Ctx &c, const int32_t *row) {
    const Smem &s = g_s;
    const int n = c.Q->n;
    const int depth = s.kdepth;
    uint64_t key = 0;
    for (int u0 = 0; u0 < n; u0 += 8) {
        int32_t x[8], lo[8], len[8];
        const int32_t *lst[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int u = u0 + j;
            const bool on = u < n && s.bitsn[u] > 0;
            lst[j] = on ? s.rkl[u] : nullptr;
            x[j] = on ? row[s.jpos[u]] : 0;
            lo[j] = 0;
            len[j] = on ? s.cnt[u] : 0;
        }
        for (int it = 0; it < depth; ++it) {
            int32_t v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = len[j] > 0 ? lst[j][lo[j] + (len[j] >> 1)] : 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int32_t h = len[j] >> 1;
                if (len[j] > 0 && v[j] < x[j]) {
                    lo[j] += h + 1;
                    len[j] -= h + 1;
                } else {
                    len[j] = h;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int u = u0 + j;
            if (u < n && s.bitsn[u] > 0) key = (key << s.bitsn[u]) | (uint64_t)lo[j];
        }
    }
    return key;
}

// Sort keys of the rows r0 + q NT (q < kKeyRows) below `rows`, as row_key,
// column by column: a column's probes are the same steps for every row and
// lane (each row's value is in its list), through LDS where its list is
// staged, and the rows' probes are the independent loads. For more rows than
// threads, where row_key's eight columns at once cost a wave 11 us per row
// whatever the columns (20,763 rows of nine key columns: 521 us in one
// workgroup, now 136).
constexpr int kKeyRows = 4;

__device__ __forceinline__ void row_keys(const Ctx &c, const int32_t *table, int k, int64_t r0,
                                         int64_t rows, uint64_t *key) {
    const Smem &s = g_s;
    const int32_t *stage = (const int32_t *)(g_dyn + kStageOff);
    const int n = uniform(c.Q->n);
#pragma unroll
    for (int q = 0; q < kKeyRows; ++q) key[q] = 0;
    for (int u = 0; u < n; ++u) {
        const int b = uniform(s.bitsn[u]);
        if (b == 0) continue;
        const int32_t m = uniform(s.cnt[u]), col = uniform(s.jpos[u]);
        const int32_t *lst = uniform(s.rkl[u]);
        int32_t x[kKeyRows], lo[kKeyRows];
#pragma unroll
        for (int q = 0; q < kKeyRows; ++q) {
            const int64_t r = r0 + q * NT;
            x[q] = table[(r < rows ? r : 0) * k + col];
            lo[q] = 0;
        }
        if (lst != c.L(u)) {
            const int32_t *l = stage + (lst - stage);
            for (int32_t len = m; len > 1;) {
                const int32_t h = len >> 1;
#pragma unroll
                for (int q = 0; q < kKeyRows; ++q) lo[q] += l[lo[q] + h - 1] < x[q] ? h : 0;
                len -= h;
            }
        } else {
            const int32_t *l = c.L(u);
            for (int32_t len = m; len > 1;) {
                const int32_t h = len >> 1;
#pragma unroll
                for (int q = 0; q < kKeyRows; ++q) lo[q] += l[lo[q] + h - 1] < x[q] ? h : 0;
                len -= h;
            }
        }
#pragma unroll
        for (int q = 0; q < kKeyRows; ++q) key[q] = (key[q] << b) | (uint64_t)lo[q];
    }
}

// Point rkl[u] at the sorted candidate list of every key column, copying
// the lists into LDS while they fit (binary searches then stay on chip).
__device__ __forceinline__ void stage_key_lists(Ctx &c) {
    int32_t *stage = (int32_t *)(g_dyn + kStageOff);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t used = 0;
        for (int u = 0; u < c.Q->n; ++u) {
            const int32_t m = g_s.cnt[u];
            if (g_s.bitsn[u] > 0 && used + m <= kStageInts) {
                g_s.rkl[u] = stage + used;
                used += m;
            } else {
                g_s.rkl[u] = c.L(u);
            }
        }
    }
    __syncthreads();
    for (int u = 0; u < c.Q->n; ++u) {
        int32_t *dst = const_cast<int32_t *>(g_s.rkl[u]);
        if (dst == c.L(u)) continue;
        const int32_t *src = c.L(u);
        for (int32_t i = threadIdx.x; i < g_s.cnt[u]; i += NT) dst[i] = src[i];
    }
    __syncthreads();
}

// One stable 8-bit LSD pass of the whole workgroup. Wave w owns a contiguous
// segment of the input: per-wave digit counts, one scan in (digit, wave)
// order, then every wave places its segment in order without further
// workgroup barriers (64 elements at a time, ranked within the wave by
// matching digits through ballots; four chunks' loads in flight).
__device__ __forceinline__ void wg_radix_pass(Ctx &c, const uint64_t *kin, const int32_t *iin,
                                              uint64_t *kout, int32_t *iout, int64_t n,
                                              int shift) {
    int32_t *cnt = (int32_t *)g_dyn;  // [NW][256] counts, then running offsets
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t seg = ((n + NW - 1) / NW + 63) & ~(int64_t)63;
    const int64_t lo = min(n, wid * seg), hi = min(n, lo + seg);
    __syncthreads();
    for (int i = threadIdx.x; i < NW * 256; i += NT) cnt[i] = 0;
    __syncthreads();
    for (int64_t i = lo + lane; i < hi; i += 64) atomicAdd(&cnt[wid * 256 + ((kin[i] >> shift) & 255)], 1);
    __syncthreads();
    {
        // digit-major exclusive scan; thread d < 256 owns digit d
        int32_t col[NW];
        int64_t sum = 0;
        if (threadIdx.x < 256)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                col[w] = cnt[w * 256 + threadIdx.x];
                sum += col[w];
            }
        int64_t tot;
        int64_t run = block_excl_scan<NW>(sum, g_s.sh, &tot);
        if (threadIdx.x < 256)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                cnt[w * 256 + threadIdx.x] = (int32_t)run;
                run += col[w];
            }
    }
    __syncthreads();
    int32_t *mine = cnt + wid * 256;
    for (int64_t b = lo; b < hi; b += 256) {
        uint64_t kv[4];
        int32_t iv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = b + q * 64 + lane;
            kv[q] = i < hi ? kin[i] : 0ull;
            iv[q] = i < hi ? iin[i] : 0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool valid = b + q * 64 + lane < hi;
            const int d = (int)((kv[q] >> shift) & 255);
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint64_t m = __ballot((d >> t) & 1);
                peers &= ((d >> t) & 1) ? m : ~m;
            }
            const int rk = __popcll(peers & lanemask_lt(lane));
            if (valid) {
                const int64_t p = (int64_t)mine[d] + rk;
                kout[p] = kv[q];
                iout[p] = iv[q];
            }
            // every lane has read its offset before the digit's first lane
            // advances it (one wave, program order)
            if (valid && rk == 0) mine[d] += __popcll(peers);
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// one query
// ---------------------------------------------------------------------------

__device__ __forceinline__ void clear_slot(Ctx &c, bool full) {
    __syncthreads();
    const int n = c.Q->n;
    const int32_t nwords = c.g.nwords;
    if (full) {
        for (int u = 0; u < n; ++u)
            for (int32_t w = threadIdx.x; w < nwords; w += NT) c.B(u)[w] = 0ull;
        for (int32_t w = threadIdx.x; w < nwords; w += NT) c.scratch[w] = 0ull;
    } else {
        for (int u = 0; u < n; ++u) clear_words(c, u, g_s.cnt[u]);
    }
    __syncthreads();
}

// The one row over single-candidate query vertices vert(0 .. k): their
// candidates to out[0 .. k), and level_rows[i] = 1 while the first i + 1 of
// them are distinct (or may repeat), else 0. Ends without a barrier.
template <class F>
__device__ __forceinline__ void single_row(Ctx &c, int32_t *out, int k, F vert) {
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x;
    const int32_t x = lane < k ? c.L(vert(lane))[0] : -1 - lane;
    uint32_t dup = 0;  // lanes that repeat an earlier one
    if (!c.Q->homo)
        for (int i = 0; i + 1 < k; ++i)
            dup |= (uint32_t)__ballot(lane > i && x == __builtin_amdgcn_readlane(x, i));
    if (lane < k) {
        out[lane] = x;
        g_s.level_rows[lane] = (dup & ((2u << lane) - 1u)) == 0;
    }
}

// A query's phases, each in a function of its own (see g_s).

// Filtering: root candidates, exploration, refinement.
__device__ __attribute__((noinline)) void filter_phase() {
    SGM_OWN_CTX(c);
    const DevGraph &g = c.g;
    Smem &s = g_s;
    const NQuery &Q = s.query;
    const int n = uniform(Q.n);
    // root candidates
    const int root = Q.root;
    // (a sparse root's are listed already: its step is one over a list)
    const int32_t rootq = Q.root_lo < 0 || Q.root_sparse ? -1
                                        : Q.pred[root].qout | Q.pred[root].qin << 8 | (Q.homo ? 1 << 16 : 0);
    if (rootq < 0) {
        if (threadIdx.x == 0) {
            const int32_t pin = Q.pred[root].pin;
            if (pin >= 0 && pin < g.V && vpred(g, Q.pred[root], pin)) {
                c.B(root)[pin >> 6] |= 1ull << (pin & 63);
                c.L(root)[0] = pin;
                s.cnt[root] = 1;
            }
        }
        __syncthreads();
    }
    ev(c, SGM_EV_ROOT);
    // Explore along the spanning tree, then refinement rounds: one loop, so
    // that the kernel holds the steps' code once. (A single query vertex has
    // no step; an unpinned one takes its whole range in one without tests.)
    const bool alone = Q.n_init == 0 && rootq >= 0;
    const int n_exp = alone ? 1 : Q.n_init;
    const int rounds = Q.n_ref > 0 ? (Q.refine_rounds < 0 ? 32 : Q.refine_rounds) : 0;
    int removed = 0;
    for (int i = 0, r = 0; i < n_exp + (r < rounds ? Q.n_ref : 0) && !aborted(c);) {
        const NStep st = alone ? NStep{(int8_t)root, 1, -1, 0, 0, 0} : Q.steps[i];
        // the first step is the root's
        removed += filter_step(c, st, i == 0 ? rootq : -1);
        const bool exploring = i < n_exp;
        ev(c, exploring ? SGM_EV_EXPLORE : SGM_EV_REFINE);
        if (exploring) removed = 0;
        if (++i == n_exp + Q.n_ref && r < rounds) {
            // a round is over
            ++r;
            if (r < rounds && !(Q.refine_rounds < 0 && removed == 0)) i = n_exp;
            removed = 0;
        }
    }
}

// Candidate edges and join levels: the rows found and their table.
__device__ __attribute__((noinline)) void match_phase() {
    SGM_OWN_CTX(c);
    Smem &s = g_s;
    const NQuery &Q = s.query;
    const int n = uniform(Q.n);
    int64_t rows = 0;
    int32_t *table = nullptr;
    for (int u = 0; u < n && !aborted(c); ++u)
        if (s.cnt[u] > 1) sort_list(c, u);
    ev(c, SGM_EV_LISTS);
    if (Q.m == 0) {
        table = c.L(0);
        rows = s.cnt[0];
        if (threadIdx.x == 0) {
            s.jorder[0] = 0;
            s.jpos[0] = 0;
        }
        __syncthreads();
    } else if (!aborted(c)) {
        // candidate edges keyed by each edge's source: totals for the order
        // (dir 0), then the edges the join looks up by their destination
        // again, keyed so (dir 1)
        bool join = false;
        int pre = 0;
        uint64_t todo = Q.m == 64 ? ~0ull : (1ull << Q.m) - 1ull;
        for (int dir = 0; dir < 2 && todo && !aborted(c); ++dir) {
            const uint64_t few = ec_build_few(c, todo, dir);
            if (few) ev(c, SGM_EV_EDGES);
            for (int e = 0; e < Q.m && !aborted(c); ++e) {
                if (!(((todo & ~few) >> e) & 1ull)) continue;
                ec_build_far(e, dir ? Q.edst[e] : Q.esrc[e], dir ? Q.esrc[e] : Q.edst[e], dir);
                ev(c, SGM_EV_EDGES);
            }
            __syncthreads();
            if (dir == 1) break;
            bool none = false, single = true;
            for (int e = 0; e < Q.m; ++e) none |= s.ectot[e] == 0;
            for (int u = 0; u < n; ++u) single &= s.cnt[u] == 1;
            if (aborted(c) || none) break;
            if (single) {
                // One candidate per query vertex and its pair in every
                // edge table: those candidates are the only possible
                // row, and a match exactly when they are distinct. The
                // join binds the vertices in index order.
                int32_t *one_row = (int32_t *)slab_alloc(c, 4ll * n);
                if (!one_row) break;
                mark(c, 2);
                single_row(c, one_row, n, [&](int u) { return u; });
                if (threadIdx.x < n) {
                    s.jorder[threadIdx.x] = threadIdx.x;
                    s.jpos[threadIdx.x] = threadIdx.x;
                }
                if (threadIdx.x == 0) {
                    s.nrows = s.level_rows[n - 1];
                    add_bytes(c, 8ull * n);
                }
                __syncthreads();
                table = one_row;
                rows = s.nrows;
                ev(c, SGM_EV_LEVEL);
                break;
            }
            join = true;
            if (threadIdx.x < Q.m) s.ecbuilt[threadIdx.x] = s.eckey[threadIdx.x];
            __syncthreads();
            join_order(c);
            __syncthreads();
            ev(c, SGM_EV_ORDER);
            // The join's leading vertices of one candidate each make one
            // row (every edge between them holds its pair, or the query
            // had ended): no level and no re-keyed table is run for them.
            while (pre < n && s.cnt[s.jorder[pre]] == 1) ++pre;
            todo = 0;
            for (int e = 0; e < Q.m; ++e)
                if (s.eckey[e] != s.ecbuilt[e] && (s.jpos[Q.esrc[e]] >= pre || s.jpos[Q.edst[e]] >= pre))
                    todo |= 1ull << e;
        }
        if (join && !aborted(c)) {
            // join levels
            mark(c, 2);
            table = c.L(s.jorder[0]);
            rows = s.cnt[s.jorder[0]];
            if (threadIdx.x == 0) s.level_rows[0] = rows;
            int k = 1;
            if (pre > 1 && !aborted(c)) {
                int32_t *row = (int32_t *)slab_alloc(c, 4ll * pre);
                if (row) {
                    single_row(c, row, pre, [&](int i) { return s.jorder[i]; });
                    __syncthreads();
                    table = row;
                    rows = s.level_rows[pre - 1];
                    k = pre;
                    ev(c, SGM_EV_LEVEL);
                }
            }
            for (int lv = k - 1; lv < n - 1 && !aborted(c) && rows > 0; ++lv) {
                const bool counting = Q.count_only && lv == n - 2;
                const int ext = s.lv_ext[lv];
                const int p = s.eckey[ext];
                const int cp = s.jpos[p];
                const int32_t *pk = c.L(p);
                const int32_t npk = s.cnt[p];
                const int32_t *eoffs = s.ec_offs[ext];
                const int32_t *ecnt = s.ec_cnt[ext];
                const int32_t *evals = s.ec_vals[ext];
                in_memory(eoffs);
                in_memory(ecnt);
                in_memory(evals);
                const int nchk = s.lv_nchk[lv];
                const int cfirst = s.lv_first[lv];
                // output capacity: what is left of the slab
                __syncthreads();
                const int64_t used0 = (s.slab_used + 255) & ~(int64_t)255;
                const int64_t left = c.slab_bytes - used0;
                int64_t cap = left / (4 * (k + 1));
                if (cap <= 0) {
                    if (threadIdx.x == 0) s.abort_ = kWhySlab;
                    __syncthreads();
                    break;
                }
                if (threadIdx.x == 0) {
                    s.ctr = 0;
                    s.cnt64 = 0ull;
                }
                __syncthreads();
                // the level's pairs bound its rows: a level that could not
                // fit even a much larger slot stops here rather than
                // after filling this one
                int64_t pairs = -1;
                const bool may_share = c.job && c.help_items > 0;
                // a block of rows whose pairs could reach a shared or a
                // host-ordered level (rows times the extension edge's
                // candidate edges bound them) counts them here too
                if (counting && nchk == 0) {
                    // counted row by row, shared by rows
                    pairs = rows;
                } else if (rows > NT || rows * s.ectot[ext] >= kJoinSharePairs) {
                    int64_t mp = 0;
                    for (int64_t r = threadIdx.x; r < rows; r += NT) {
                        const int32_t pv = table[r * k + cp];
                        const int32_t i = lower_bound_i32(pk, 0, npk, pv);
                        if (i < npk && pk[i] == pv) mp += ecnt[i];
                    }
                    block_excl_scan<NW>(mp, s.sh, &pairs);
                    if (!counting && pairs > kPairSlack * cap) {
                        if (threadIdx.x == 0) {
                            s.abort_ = kWhySlab;
                            s.need = used0 + pairs * 4 * (k + 1);
                        }
                        __syncthreads();
                        break;
                    }
                }
                // A last level that may reach the size the host orders
                // goes to the top of the slab (its pairs bound its rows),
                // with room above for the key columns' candidate lists:
                // the slot's later queries keep the slab below it.
                int32_t *out = nullptr;
                if (counting) cap = INT32_MAX;  // no rows are written
                if (!counting && lv == n - 2 && c.host_order_rows > 0 && pairs >= c.host_order_rows) {
                    int64_t lint = 0;
                    for (int u = 0; u < n; ++u) lint += s.cnt[u];
                    const int64_t tneed = (pairs * 4 * (k + 1) + 255) & ~(int64_t)255;
                    const int64_t lneed = (4 * lint + 256 * (n + 1)) & ~(int64_t)255;
                    const int64_t at = (c.slab_bytes - tneed - lneed) & ~(int64_t)255;
                    if (at >= kPinFloor(c) && at >= used0) {
                        out = (int32_t *)(c.slab + at);
                        cap = pairs;
                        if (threadIdx.x == 0) s.below_top = used0;
                        __syncthreads();
                        if (threadIdx.x == 0) s.slab_used = at + pairs * 4 * (k + 1);
                        __syncthreads();
                    }
                }
                if (!out && !counting) out = (int32_t *)slab_alloc(c, cap * 4 * (k + 1));
                if (!out && !counting) {
                    if (threadIdx.x == 0) s.abort_ = kWhySlab;
                    __syncthreads();
                    break;
                }
                // the level's view (parent column, edge tables of its
                // extension and check edges, output), the same for the
                // owner and for helpers
                __syncthreads();
                if (threadIdx.x == 0) {
                    JLevel &L = s.jl;
                    L.table = table;
                    L.rows = rows;
                    L.k = k;
                    L.cp = cp;
                    L.pk = pk;
                    L.npk = npk;
                    L.eoffs = eoffs;
                    L.ecnt = ecnt;
                    L.evals = evals;
                    L.nchk = nchk;
                    for (int ci = 0; ci < nchk; ++ci) {
                        const int e = s.chk[cfirst + ci];
                        const int kv = s.eckey[e];
                        L.chk[ci] = JChk{c.L(kv), s.ec_offs[e], s.ec_cnt[e], s.ec_vals[e],
                                         s.cnt[kv], s.jpos[kv]};
                    }
                    L.out = out;
                    L.cap = cap;
                    L.count = counting;
                    // columns the new value may repeat: those of a vertex
                    // that can hold a candidate of the new one
                    const int w = s.jorder[lv + 1];
                    uint32_t cm = 0;
                    for (int i = 0; i < k && !Q.homo; ++i) {
                        const int32_t a = Q.pred[s.jorder[i]].label, b = Q.pred[w].label;
                        if (a < 0 || b < 0 || a == b) cm |= 1u << i;
                    }
                    L.cmask = cm;
                }
                // a level of many pairs is shared (whether or not
                // workgroups are idle yet: those that become idle join)
                const int64_t nrb = (rows + NT - 1) / NT;
                int64_t nsub = 1;
                if (may_share && pairs >= kJoinSharePairs)
                    nsub = min((int64_t)kJoinMaxSub,
                               max((int64_t)1, (pairs + nrb * kJoinChunkPairs - 1) /
                                                   (nrb * kJoinChunkPairs)));
                // (a counting level without check edges: blocks of rows)
                if (counting && nchk == 0) nsub = 1;
                const bool share =
                    may_share && nrb * nsub <= kMaxChunks &&
                    (counting && nchk == 0 ? nrb >= kCountShareBlocks : pairs >= kJoinSharePairs);
                if (threadIdx.x == 0) s.jl.nsub = (int32_t)nsub;
                __syncthreads();
                uint64_t jb = 0;  // algorithmic bytes of this thread's rows and pairs
                if (share) {
                    jb += shared_join_far((int32_t)(nrb * nsub));
                } else {
                    for (int64_t rbase = 0; rbase < rows && !aborted(c); rbase += NT)
                        join_rows<false>(c, s.jl, rbase, min(rows, rbase + NT), 0, 1,
                                         nullptr, nullptr, jb);
                }
                add_bytes(c, jb);
                __syncthreads();
                rows = counting ? (int64_t)s.cnt64 : (int64_t)s.ctr;
                if (threadIdx.x == 0) s.level_rows[lv + 1] = rows;
                // give back the unused part of the table allocation
                __syncthreads();
                if (threadIdx.x == 0 && !s.abort_ && !counting)
                    s.slab_used = (int64_t)((char *)out - c.slab) + rows * 4 * (k + 1);
                __syncthreads();
                ev(c, SGM_EV_LEVEL);
                table = out;
                ++k;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        s.nrows = rows;
        s.table = table;
    }
}

// Ordering and output of the rows found.
__device__ __attribute__((noinline)) void order_phase() {
    SGM_OWN_CTX(c);
    Smem &s = g_s;
    const NQuery &Q = s.query;
    const int n = uniform(Q.n);
    int64_t rows = uniform(s.nrows);
    int32_t *table = uniform(s.table);
    in_memory(table);
    // ordering: key = concatenated candidate ranks in column order 0..n-1;
    // a projection (thesis Ch. 3, Sec. "GpSense") keys and keeps only
    // its columns
    __syncthreads();
    if (threadIdx.x == 0) {
        int tb = 0, no = 0, depth = 0;
        for (int u = 0; u < n; ++u) {
            const bool kept = Q.proj == 0u || ((Q.proj >> u) & 1u);
            int b = 0;
            while (kept && (1ll << b) < s.cnt[u]) ++b;
            s.bitsn[u] = b;
            tb += b;
            if (kept) s.ocol[no++] = s.jpos[u];
            // a lower bound over m entries ends after bit_length(m) halvings
            if (b > 0) depth = max(depth, 32 - __clz(s.cnt[u]));
        }
        s.ctr = tb;
        s.nout = no;
        s.kdepth = depth;
    }
    __syncthreads();
    if (s.ctr > 64 && rows > 1) {
        if (threadIdx.x == 0) {
            s.status = kNeedWide;
            s.reason = kWhyKey;
        }
        return;
    }
    const int tb = s.ctr;
    const int k = n;
    const int no = s.nout;
    int32_t *idx;
    const uint64_t *skeys = nullptr;  // the sorted keys (rows > 1)
    // A large final table in the slab, with room below it for the slot's
    // later queries: the key columns' sorted candidate lists go beside
    // it and the host orders it (and collapses a projection) with
    // whole-GPU kernels after the launch; one workgroup would spend
    // milliseconds on the keys, the passes and the gather.
    int64_t toff = (int64_t)((const char *)table - c.slab);
    if (c.host_order_rows > 0 && rows >= c.host_order_rows && toff >= 0 &&
        toff < c.slab_bytes) {
        int64_t lint = 0;
        for (int u = 0; u < n; ++u)
            if (s.bitsn[u] > 0) lint += s.cnt[u];
        int32_t *lst = nullptr;
        const int64_t tbytes = (rows * k * 4 + 255) & ~(int64_t)255;
        const int64_t top = ((c.slab_bytes - 4 * lint) & ~(int64_t)255) - tbytes;
        if (toff >= kPinFloor(c)) {
            lst = (int32_t *)slab_alloc(c, 4 * lint);
        } else if (top >= kPinFloor(c) && top > toff) {
            // too low in the slab to keep for the host: move it up to
            // the top, lists above it; overlapping, so the chunks go
            // from the end (every read of a chunk before its writes)
            int32_t *dst = (int32_t *)(c.slab + top);
            const int64_t nint = rows * k;
            for (int64_t end = nint; end > 0; end -= 4 * NT) {
                const int64_t beg = end - 4 * NT > 0 ? end - 4 * NT : 0;
                int32_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t i = beg + q * NT + threadIdx.x;
                    v[q] = i < end ? table[i] : 0;
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t i = beg + q * NT + threadIdx.x;
                    if (i < end) dst[i] = v[q];
                }
                __syncthreads();
            }
            if (threadIdx.x == 0) add_bytes(c, 8ull * nint);
            table = dst;
            toff = top;
            lst = (int32_t *)(c.slab + top + tbytes);
        }
        if (lst) {
            int64_t o = 0;
            for (int u = 0; u < n; ++u) {
                if (s.bitsn[u] == 0) continue;
                const int32_t *src = c.L(u);
                for (int32_t i = threadIdx.x; i < s.cnt[u]; i += NT) lst[o + i] = src[i];
                o += s.cnt[u];
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                s.hostord = 1;
                s.keybits = tb;
                s.pin_off = toff;
                s.tableptr = table;
                s.listptr = lst;
                add_bytes(c, 8ull * lint);
            }
            __syncthreads();
            ev(c, SGM_EV_SORT);
            return;
        }
    }
    if (rows > 1) stage_key_lists(c);
    if (s.below_top >= 0 && rows > kRowSortCap) {
        // the last level sits at the slab's top but stayed on this
        // workgroup: its sort buffers go into the slab below it
        __syncthreads();
        if (threadIdx.x == 0) s.slab_used = s.below_top;
        __syncthreads();
        c.slab_bytes = toff;
    }
    if (rows == 1) {
        int32_t *ix = (int32_t *)g_dyn;
        if (threadIdx.x == 0) ix[0] = 0;
        __syncthreads();
        idx = ix;
    } else if (rows <= kRowSortCap) {
        // bitonic network in LDS
        uint64_t *keys = (uint64_t *)g_dyn;
        int32_t *ix = (int32_t *)(g_dyn + sizeof(uint64_t) * kRowSortCap);
        int32_t N = 1;
        while (N < rows) N <<= 1;
        if (rows <= NT) {
            for (int32_t r = threadIdx.x; r < N; r += NT) {
                keys[r] = r < rows ? row_key(c, table + (int64_t)r * k) : ~0ull;
                ix[r] = r;
            }
        } else {
            static_assert(kRowSortCap <= kKeyRows * NT, "one round");
            uint64_t key[kKeyRows];
            row_keys(c, table, k, threadIdx.x, rows, key);
#pragma unroll
            for (int q = 0; q < kKeyRows; ++q) {
                const int32_t r = threadIdx.x + q * NT;
                if (r < N) {
                    keys[r] = r < rows ? key[q] : ~0ull;
                    ix[r] = r;
                }
            }
        }
        __syncthreads();
        for (int32_t size = 2; size <= N; size <<= 1) {
            for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
                for (int32_t i = threadIdx.x; i < N / 2; i += NT) {
                    const int32_t lo = 2 * i - (i & (stride - 1));
                    const int32_t hi = lo + stride;
                    const bool up = (lo & size) == 0;
                    // ties (a key of all ones against the padding)
                    // by row index, so padding stays last
                    const uint64_t x = keys[lo], y = keys[hi];
                    const bool gt = x > y || (x == y && ix[lo] > ix[hi]);
                    if (gt == up) {
                        keys[lo] = y;
                        keys[hi] = x;
                        const int32_t t = ix[lo];
                        ix[lo] = ix[hi];
                        ix[hi] = t;
                    }
                }
                __syncthreads();
            }
        }
        idx = ix;
        skeys = keys;
    } else {
        // LSD radix on (key, row) pairs in the slab, 8 bits per pass
        uint64_t *ka = (uint64_t *)slab_alloc(c, 8 * rows);
        uint64_t *kb = (uint64_t *)slab_alloc(c, 8 * rows);
        int32_t *ia = (int32_t *)slab_alloc(c, 4 * rows);
        int32_t *ib = (int32_t *)slab_alloc(c, 4 * rows);
        if (!ka || !kb || !ia || !ib) {
            if (threadIdx.x == 0) {
                s.status = kNeedWide;
                s.reason = kWhySlab;
            }
            return;
        }
        if (threadIdx.x == 0) s.unsorted = 0;
        for (int64_t r0 = threadIdx.x; r0 < rows; r0 += kKeyRows * NT) {
            uint64_t key[kKeyRows];
            row_keys(c, table, k, r0, rows, key);
#pragma unroll
            for (int q = 0; q < kKeyRows; ++q) {
                const int64_t r = r0 + q * NT;
                if (r < rows) {
                    ka[r] = key[q];
                    ia[r] = (int32_t)r;
                }
            }
        }
        __syncthreads();
        // a join that bound the key columns in key order has left the
        // rows in order already: then no pass is needed
        bool down = false;
        for (int64_t r = threadIdx.x; r + 1 < rows; r += NT) down |= ka[r] > ka[r + 1];
        if (down) s.unsorted = 1;
        __syncthreads();
        if (threadIdx.x == 0) add_bytes(c, 8ull * rows);
        const bool passes = s.unsorted != 0;
        for (int sh = 0; passes && sh < tb; sh += 8) {
            wg_radix_pass(c, ka, ia, kb, ib, rows, sh);
            uint64_t *tk = ka;
            ka = kb;
            kb = tk;
            int32_t *ti = ia;
            ia = ib;
            ib = ti;
        }
        if (threadIdx.x == 0 && passes) add_bytes(c, 24ull * rows * ((tb + 7) / 8));
        idx = ia;
        skeys = ka;
    }
    if (Q.proj && rows > 1) {
        // equal projected rows now have equal, adjacent keys: keep the
        // first row of each run (in-place compaction of the order)
        int64_t kept = 0;
        for (int64_t base = 0; base < rows; base += NT) {
            const int64_t i = base + threadIdx.x;
            const bool head = i < rows && (i == 0 || skeys[i] != skeys[i - 1]);
            const int32_t v = i < rows ? idx[i] : 0;
            int64_t tot;
            const int64_t ex = block_excl_scan<NW>((int64_t)(head ? 1 : 0), s.sh, &tot);
            if (head) idx[kept + ex] = v;
            kept += tot;
            __syncthreads();
        }
        if (threadIdx.x == 0) add_bytes(c, 16ull * rows);
        rows = kept;
        if (threadIdx.x == 0) s.nrows = rows;
        __syncthreads();
    }
    ev(c, SGM_EV_SORT);
    if (threadIdx.x == 0) {
        const unsigned long long need = (unsigned long long)rows * no;
        const unsigned long long off = atomicAdd(c.out_used, need);
        s.offset = (off + need <= (unsigned long long)c.out_cap) ? (int64_t)off : -1;
    }
    __syncthreads();
    const int64_t off = s.offset;
    if (off < 0) {
        if (threadIdx.x == 0) s.status = kOutFull;
    } else {
        // one wave per 64 output rows: consecutive lanes write
        // consecutive ints of the rows, columns back in query-vertex
        // order; e / no by a 16-bit reciprocal (exact for e < 64 no,
        // no <= 16)
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        const uint32_t inv = (65536u + (uint32_t)no - 1u) / (uint32_t)no;
        int32_t *arena = off + rows * no <= c.host_cap ? c.host_out : c.out;
        for (int64_t r0 = (int64_t)wid * 64; r0 < rows; r0 += NT) {
            const int32_t my = r0 + lane < rows ? idx[r0 + lane] : 0;
            const int nr = (int)min((int64_t)64, rows - r0);
            int32_t *dst = arena + off + r0 * no;
            const int ne = nr * no;
            for (int e0 = 0; e0 < ne; e0 += 256) {
                // four gathers in flight per lane; every lane takes part
                // in the shuffles
                int32_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int e = e0 + q * 64 + lane;
                    const int r = min(63, (int)(((uint32_t)e * inv) >> 16));
                    const int32_t src = __shfl(my, r, 64);
                    v[q] = e < ne ? table[(int64_t)src * k + s.ocol[e - r * no]] : 0;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (e0 + q * 64 + lane < ne) dst[e0 + q * 64 + lane] = v[q];
            }
        }
        if (threadIdx.x == 0) add_bytes(c, 20ull * rows * no);
    }
}

// The output of a query with one row: nothing to order (2 us less than the
// ordering phase takes to find that out).
__device__ __forceinline__ void one_row_out(Ctx &c) {
    Smem &s = g_s;
    ev(c, SGM_EV_SORT);
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const uint32_t all = (1u << c.Q->n) - 1u;
        const uint32_t kept = c.Q->proj ? c.Q->proj & all : all;
        const int no = __popc(kept);
        unsigned long long off = 0;
        if (lane == 0) {
            off = atomicAdd(c.out_used, (unsigned long long)no);
            const bool fits = off + no <= (unsigned long long)c.out_cap;
            s.offset = fits ? (int64_t)off : -1;
            if (!fits) s.status = kOutFull;
            add_bytes(c, fits ? 20ull * no : 0ull);
        }
        off = __shfl(off, 0, 64);
        if (off + no <= (unsigned long long)c.out_cap && lane < c.Q->n && ((kept >> lane) & 1u)) {
            int32_t *arena = (int64_t)off + no <= c.host_cap ? c.host_out : c.out;
            arena[off + __popc(kept & ((1u << lane) - 1u))] = s.table[s.jpos[lane]];
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void run_query(Ctx &c) {
    Smem &s = g_s;
    const NQuery &Q = s.query;
    const int n = Q.n;
    if (threadIdx.x < SGM_MAX_QV) {
        s.cnt[threadIdx.x] = 0;
        s.cand[threadIdx.x] = 0;
        s.level_rows[threadIdx.x] = 0;
        s.jorder[threadIdx.x] = -1;
    }
    if (threadIdx.x < SGM_MAX_QV) s.ver[threadIdx.x] = 0;
    if (threadIdx.x < 2 * SGM_MAX_QE) s.okv[threadIdx.x] = -1;
    if (threadIdx.x < SGM_MAX_QE) {
        s.ectot[threadIdx.x] = 0;
        s.qsrc[threadIdx.x] = threadIdx.x < Q.m ? (int8_t)Q.esrc[threadIdx.x] : 0;
        s.qdst[threadIdx.x] = threadIdx.x < Q.m ? (int8_t)Q.edst[threadIdx.x] : 0;
    }
    if (threadIdx.x < 5) {
        s.t[threadIdx.x] = 0;
        s.pb[threadIdx.x] = 0ull;
    }
    if (threadIdx.x == 0) {
        s.hostord = 0;
        s.keybits = 0;
        s.tableptr = nullptr;
        s.listptr = nullptr;
        s.abort_ = 0;
        s.slab_used = 0;
        s.below_top = -1;
        s.empty = 0;
        s.status = SGM_OK;
        s.reason = 0;
        s.nrows = 0;
        s.offset = 0;
        s.need = 0;
        s.bytes = 0;
        if (Q.fault) s.status = kFault;
    }
    if (Q.fault) {
        // a failure injected from the host: this query alone ends with a
        // device error, as a fault confined to it would
        __syncthreads();
        return;
    }
    __syncthreads();
    mark(c, 0);
    ev(c, SGM_EV_START);
    if (Q.root_sparse) sparse_root();
    filter_phase();
    __syncthreads();
    mark(c, 1);
    if (aborted(c)) {
        clear_slot(c, true);
        if (threadIdx.x == 0) {
            s.status = kNeedWide;
            s.reason = s.abort_;
        }
        return;
    }
    if (threadIdx.x == 0)
        for (int u = 0; u < n; ++u) {
            s.cand[u] = s.cnt[u];
            if (s.cnt[u] == 0) s.empty = 1;
        }
    __syncthreads();
    if (!s.empty) match_phase();
    __syncthreads();
    mark(c, 3);
    if (aborted(c)) {
        clear_slot(c, true);
        if (threadIdx.x == 0) {
            s.status = kNeedWide;
            s.reason = s.abort_;
        }
        return;
    }
    // a count-only query is done (its last level wrote no table)
    if (s.nrows > 0 && !Q.count_only) {
        if (s.nrows == 1 && (c.host_order_rows <= 0 || c.host_order_rows > 1)) one_row_out(c);
        else order_phase();
        __syncthreads();
    }
    const bool ended = s.status != kNeedWide;
    if (ended) ev(c, SGM_EV_OUTPUT);
    clear_slot(c, false);
    if (ended) mark(c, 4);
}

// Chunks of the step posted on board entry e, starting with chunk ch, until
// the step has none left; then the chunks are reported done (one release
// fence for all of them).
__device__ __forceinline__ void help_step(const NArgs &a, int e, int32_t ch) {
    Smem &s = g_s;
    HelpJob *j = a.board + e;
    // the parameters stay fixed while this workgroup holds unreported chunks
    const NStep st = j->st;
    const int32_t K = j->chunk, G = j->G, n_items = j->n_items, ncount = j->ncount;
    int32_t *def = j->defer ? (int32_t *)(a.slab + (int64_t)e * a.slab_bytes + 8 * (int64_t)a.lcap) : nullptr;
    const bool nodrop = j->nodrop != 0;
    const int kind = j->kind;
    const int4 *seg = j->seg;
    const int32_t *hul = j->ul;
    const bool nodefer = j->nodefer != 0;
    const int32_t root = j->root;
    if ((int)threadIdx.x < ncount) {
        s.nbl[threadIdx.x] = j->nbl[threadIdx.x];
    }
    if (kind == 2) {
        const uint64_t *src = (const uint64_t *)&j->jl;
        uint64_t *dst = (uint64_t *)&s.jl;
        for (int i = threadIdx.x; i < (int)(sizeof(JLevel) / 8); i += NT) dst[i] = src[i];
    }
    __syncthreads();
    Ctx c = slot_ctx(a, e, j->q, a.slab_bytes);
    c.trace = nullptr;
    uint64_t fb = 0;
    int32_t n = 0;
    while (ch >= 0) {
        if (kind == 0) {
            filter_items(c, BoardCtr{j}, st.u, root, st.push != 0, s.nbl, ncount, hul, nodrop ? nullptr : c.B(st.u), ch * K,
                          min(n_items, ch * K + K), fb, nodefer);
        } else if (kind == 1) {
            push_segment(c, BoardCtr{j}, s.nbl, seg[ch], fb);
        } else if (kind == 3) {
            ec_chunk(c, j->ecj, j, ch * K, min(n_items, ch * K + K), G, fb);
        } else if (kind == 4) {
            item_wg_k(c, BoardCtr{j}, st, s.nbl, ncount, hul[ch], nodrop ? nullptr : c.B(st.u), fb, def);
        } else if (kind == 5) {
            sparse_scan(c, BoardCtr{j}, st.u, root, hul, ch * K, min(n_items, ch * K + K), fb);
        } else {
            join_chunk(c, s.jl, ch, &j->jrows, &j->abort_, fb);
        }
        ++n;
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long w = take_chunk(j);
            s.hch = claim_next(w) < claim_nch(w) ? claim_next(w) : -1;
        }
        __syncthreads();
        ch = s.hch;
        __syncthreads();
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) fb += __shfl_xor(fb, o, 64);
    if ((threadIdx.x & 63) == 0 && fb) atomicAdd(&j->bytes, (unsigned long long)fb);
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        atomicAdd(&j->done, n);
    }
}

__device__ __attribute__((noinline)) void help_step_far(int e, int32_t ch) {
    const NArgs a = own_args();
    help_step(a, __builtin_amdgcn_readfirstlane(e), __builtin_amdgcn_readfirstlane(ch));
}

// Helpers: claim chunks of posted steps until every slot workgroup has run
// out of queries (or after kHelpIdle empty polls in a row).
__device__ __forceinline__ void help_loop(const NArgs &a) {
    Smem &s = g_s;
    const int lane = threadIdx.x & 63;
    int64_t idle = 0;
    for (;;) {
        if (threadIdx.x < 64) {
            int32_t e = -2, ch = -1;  // e: -2 nothing found, -1 leave
            const int32_t done =
                __hip_atomic_load(&a.hctr[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int32_t posted =
                __hip_atomic_load(&a.hctr[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (done >= a.nslot) e = -1;
            else if (posted > 0) {
                // entries with an open chunk, 64 at a time from a rotating start
                for (int base = 0; base < a.nslot && e == -2; base += 64) {
                    const int k = base + lane;
                    const int en = (k + (int)blockIdx.x) % a.nslot;
                    bool open = false;
                    if (k < a.nslot) {
                        const unsigned long long w = __hip_atomic_load(
                            &a.board[en].claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        open = claim_next(w) < claim_nch(w);
                    }
                    uint64_t m = __ballot(open);
                    while (m && e == -2) {
                        const int l = __ffsll((unsigned long long)m) - 1;
                        m &= m - 1;
                        const int cand = (base + l + (int)blockIdx.x) % a.nslot;
                        int32_t got = -1;
                        if (lane == 0) {
                            const unsigned long long w = take_chunk(a.board + cand);
                            if (claim_next(w) < claim_nch(w)) {
                                got = claim_next(w);
                                // the step's parameters and the owner's data
                                __threadfence();
                            }
                        }
                        got = __shfl(got, 0, 64);
                        if (got >= 0) {
                            e = cand;
                            ch = got;
                        }
                    }
                }
            }
            if (lane == 0) {
                s.hq = e;
                s.hch = ch;
            }
        }
        __syncthreads();
        const int32_t e = s.hq, ch = s.hch;
        __syncthreads();
        if (e == -1) break;
        if (e < 0) {
            if (++idle > kHelpIdle) break;
            // quick polls right after work, slower ones while owners run
            // phases they do not share
            if (idle < 64) __builtin_amdgcn_s_sleep(2);
            else __builtin_amdgcn_s_sleep(32);
            continue;
        }
        idle = 0;
        help_step_far(e, ch);
    }
}

// A workgroup's last act: no workgroup reads a counter after counting itself
// out, so the last one out can zero them all.
__device__ __forceinline__ void leave(const NArgs &a) {
    if (threadIdx.x != 0 || !a.left) return;
    if (atomicAdd(a.left, 1) != (int)gridDim.x - 1) return;
    atomicExch(a.queue, 0);
    atomicExch(a.out_used, 0ull);
    atomicExch(&a.hctr[0], 0);
    atomicExch(&a.hctr[1], 0);
    atomicExch(a.left, 0);
}

__global__ __launch_bounds__(NT, 4) void k_narrow(NArgs a) {
    Smem &s = g_s;
    if (threadIdx.x == 0) g_args = a;
    __syncthreads();
    const bool help = a.help_items > 0 && a.board != nullptr;
    if ((int)blockIdx.x >= a.nslot) {
        if (help) help_loop(a);
        leave(a);
        return;
    }
    if (threadIdx.x == 0) {
        s.retired = 0;
        s.hq = a.board ? __hip_atomic_load(&a.board[blockIdx.x].dirty, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT)
                       : 0;
    }
    __syncthreads();
    if (s.hq) {
        // an earlier launch left this slot after giving up on a shared step
        // (helpers may have written any of its bitmaps since): clear it all
        uint64_t *bits = a.bits + (int64_t)blockIdx.x * (SGM_MAX_QV + 1) * a.g.nwords;
        const int64_t nb = (int64_t)(SGM_MAX_QV + 1) * a.g.nwords;
        for (int64_t w = threadIdx.x; w < nb; w += NT) bits[w] = 0ull;
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();
            atomicExch(&a.board[blockIdx.x].dirty, 0);
        }
    }
    int64_t slab_cap = a.slab_bytes;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s.q = atomicAdd(a.queue, 1);
        __syncthreads();
        const int32_t q = s.q;
        if (q >= a.nq) break;
        const NQuery &Qd = a.qs[q];
        const NQuery &Q = s.query;
        NResult &R = a.res[q];
        if (s.retired) {
            // the slot is out of use: the query is reported for a rerun
            if (threadIdx.x == 0) {
                R.status = kNeedWide;
                R.reason = kWhyHelp;
                R.n_cols = Qd.n;
                R.n_rows = 0;
                R.offset = 0;
                for (int u = 0; u < SGM_MAX_QV; ++u) {
                    R.cand[u] = 0;
                    R.level_rows[u] = 0;
                    R.join_order[u] = -1;
                }
                for (int e = 0; e < SGM_MAX_QE; ++e) R.ec[e] = 0;
                R.bytes = 0;
                R.need = 0;
                for (int i = 0; i < 4; ++i) R.ticks[i] = R.pbytes[i] = 0;
                R.host_order = 0;
            }
            continue;
        }
        if (threadIdx.x == 0) s.slab_cap = slab_cap;
        Ctx c = slot_ctx(a, blockIdx.x, q, slab_cap);
        static_assert(sizeof(NQuery) % 4 == 0, "staged as ints");
        for (int i = threadIdx.x; i < (int)(sizeof(NQuery) / 4); i += NT)
            ((int32_t *)&s.query)[i] = ((const int32_t *)&Qd)[i];
        if (threadIdx.x == 0) s.nev = 0;
        __syncthreads();
        run_query(c);
        __syncthreads();
        if (s.hostord) slab_cap = s.pin_off;  // keep that table until the launch ends
        // the result is put together in LDS and leaves in whole lines
        NResult &L = *(NResult *)g_dyn;
        const int t = threadIdx.x;
        if (t < SGM_MAX_QV) {
            L.cand[t] = t < Q.n ? s.cand[t] : 0;
            L.level_rows[t] = t < Q.n ? s.level_rows[t] : 0;
            L.join_order[t] = t < Q.n ? s.jorder[t] : -1;
        }
        if (t < SGM_MAX_QE) L.ec[t] = t < Q.m ? s.ectot[t] : 0;
        if (t == 0) {
            L.status = s.status;
            L.reason = s.reason;
            L.n_cols = Q.n;
            L.pad = 0;
            L.n_rows = s.status == SGM_OK ? s.nrows : 0;
            L.offset = s.offset;
            L.bytes = (int64_t)s.bytes;
            L.need = s.need;
            L.host_order = s.hostord;
            L.key_bits = s.keybits;
            L.table_ptr = (int64_t)(uintptr_t)s.tableptr;
            L.list_ptr = (int64_t)(uintptr_t)s.listptr;
            // phases a query skipped carry the time and bytes of the
            // previous mark
            int64_t prev = s.t[0];
            unsigned long long pbp = 0ull;
            for (int i = 1; i < 5; ++i) {
                const bool hit = s.t[i] != 0;
                const int64_t ti = hit ? s.t[i] : prev;
                const unsigned long long bi = hit ? s.pb[i] : pbp;
                L.ticks[i - 1] = ti - prev;
                L.pbytes[i - 1] = (int64_t)(bi - pbp);
                prev = ti;
                pbp = bi;
            }
        }
        __syncthreads();
        static_assert(sizeof(NResult) % 4 == 0, "copied as ints");
        for (int i = t; i < (int)(sizeof(NResult) / 4); i += NT)
            ((int32_t *)&R)[i] = ((const int32_t *)&L)[i];
    }
    if (help) {
        if (threadIdx.x == 0) atomicAdd(&a.hctr[1], 1);
        help_loop(a);
    }
    leave(a);
}

// Zeroes the launch's counters: the work queue, the output arena's use and
// the helper counters.
__global__ void k_reset(unsigned long long *ctr) {
    if (threadIdx.x < 3) ctr[threadIdx.x] = 0ull;
}

}  // namespace

hipError_t launch_narrow(hipStream_t s, const NArgs &a, int grid) {
    NArgs arg = a;
    void *args[] = {&arg};
    return hipLaunchKernel((const void *)k_narrow, dim3(grid), dim3(NT), args, 0, s);
}

void launch_reset(hipStream_t s, unsigned long long *ctr) {
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, s, ctr);
}

}  // namespace sgm
