// gwfa_kernels.hip -- device code of the graph wavefront alignment library
// for AMD CDNA4 (gfx950).
//
// One persistent workgroup aligns one query at a time, taking queries from a
// device work queue.  Per score s it runs the paper's loop (Section 2.4):
//   EXPAND  (Algorithm 3): insertion / deletion / mismatch candidates of every
//           diagonal of F_s, merged per diagonal, admitted when they beat the
//           diagonal's record;
//   EXTEND  (Algorithm 2): every admitted diagonal slides along its vertex by
//           the exact-match run (2-bit packed XOR + count-leading-zeros, 32
//           bases per step); a diagonal reaching the end of vertex v creates
//           (u, k+|v|) at offset 0 on every out-edge (v,u) not seen before, at
//           the same score (cost 0), and those are extended in further rounds;
//   END     (extension mode): stop at the first score at which a wavefront
//           cell has consumed the whole query;
//   PRUNE   (Algorithm 4, optional) or the learned keep/drop network.
//
// The wavefront F_s is a list sorted by (v, k).  The expansion is
// owner-computes: output diagonal k' of vertex v is produced by the present
// source with the smallest k among k'-1, k', k'+1, and those sources are the
// source's neighbours in the sorted list, so the expansion reads no table
// except at the two ends of a run of consecutive diagonals (where the record
// of a diagonal outside F_s decides).  Each wave expands a part of the list
// and writes its outputs, in order, into a part of the new one; diagonals
// created by crossings are ranked and merged in.  Lists of at most 64 entries
// are run by one wave in LDS.
//
// Records of the paper's wavefront set H~ (kept for the life of a query):
// pages of 32 consecutive diagonals of one vertex, found through an
// open-addressing directory keyed (v, k >> 5).  A record word is
// (generation << 32 | offset): a word whose generation is not the current
// query's is "never seen", so pages need no initialisation.  A record holds
// the diagonal's offset when it left the wavefront (reached the vertex end,
// consumed the query, or was pruned) -- the only diagonals outside F_s that
// can still be candidates.
//
// Global form (an end vertex v_e): the end test is Algorithm 1's, the cell
// (|q|, v_e, |v_e|); diagonals that consumed the query go on by deletions
// and crossings; an empty wavefront means v_e cannot be reached.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "gwfa_internal.h"
#include "gwfa_mlp_dev.h"

namespace gwfa_dev {

using namespace gwfa_nn;

typedef unsigned long long ull;

constexpr int PAGE = 32;
constexpr int32_t CLAIM_BASE = 0x40000000;   // record value while a crossing round claims it
constexpr int F_GROW = 1;   // directory / trace capacity exceeded: restart with a bigger one
constexpr int F_LIST = 2;   // list / candidate capacity exceeded: re-run on a larger tier
// Crossing entries sorted in LDS (virtual merge) up to this many per
// workgroup of `block` lanes; larger sets are sorted in the arena.
constexpr int xs_lds(int block) { return block >= 256 ? 1024 : 4 * block; }
// Each wave of the expansion writes the sort key of every SAMP-th entry of its
// part of the list into LDS (nsamp keys for the workgroup): the merge then
// finds an entry's place in that part by a search in LDS and one round of at
// most SAMP-1 loads.
constexpr int SAMP = 8;
constexpr int nsamp(int block) { return block >= 256 ? 1024 : (block >= 128 ? 256 : 128); }
// A list's storage: its main entries are written by the waves of the
// workgroup, each into a part of its own, at most three per source entry, so
// 3 list_cap places hold any list of up to list_cap entries; the crossing
// entries follow at place 3 list_cap.
constexpr int MAIN_X = 3;
// The exact mode stages the crossing rounds' data in LDS: up to xstage(block)
// diagonals claimed by one round (read back by the next round's extension)
// and up to twice as many crossing candidates (read back by the claims); the
// rest goes through the arena.
constexpr int xstage(int block) { return block >= 512 ? 256 : (block >= 256 ? 128 : 64); }


struct Page {
    ull R[PAGE];    // (gen << 32) | record offset (or CLAIM_BASE + round)
    ull Wc[PAGE];   // (gen << 32) | W: max walk length of a round's crossings
};
static_assert(sizeof(Page) == 512, "page layout");

__device__ __forceinline__ ull mkR(uint32_t gen, int32_t r) { return ((ull)gen << 32) | (ull)(uint32_t)r; }
__device__ __forceinline__ uint32_t rgen(ull w) { return (uint32_t)(w >> 32); }
__device__ __forceinline__ int32_t rval(ull w) { return (int32_t)(uint32_t)(w & 0xffffffffull); }

__device__ __forceinline__ ull dkey(int32_t v, int32_t kp) {
    return ((ull)(uint32_t)(v + 1) << 32) | (ull)(uint32_t)(kp + 0x40000000);
}
__device__ __forceinline__ ull skey(int32_t v, int32_t k) {   // sort key of a diagonal
    return ((ull)(uint32_t)v << 32) | (ull)(uint32_t)(k + 0x40000000);
}
__device__ __forceinline__ uint32_t dhash(ull key) {
    return (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 32);
}

// 32 bases starting at base index p of a 2-bit MSB-first packed store.
__device__ __forceinline__ ull win32(const ull* __restrict__ w, int64_t p) {
    const int64_t wi = p >> 5;
    const int sh = (int)(p & 31) * 2;
    const ull a = w[wi];
    const ull b = w[wi + 1];
    return (a << sh) | ((b >> 1) >> (63 - sh));
}

// LCP of q[qp ...] and label[sp ...], at most lim bases.  Each step
// compares up to four consecutive 32-base windows; they share words (window j
// spans words j and j+1 of the step), so a step loads five words per
// sequence, all issued together: a long exact run costs one memory round trip
// per 128 bases.  Word indices are clamped to qmax / smax, the word after the
// one holding the range's last base (both stores end with two words of
// padding, so that word exists): a window that starts inside the range never
// reaches past it, and the words clamped are never used.
__device__ __forceinline__ int32_t lcp(const ull* __restrict__ qw, int64_t qp, int64_t qmax, const ull* __restrict__ sw,
                                       int64_t sp, int64_t smax, int32_t lim, uint32_t& chunks) {
    int32_t l = 0;
    const int qs = (int)((qp & 31) * 2), ss = (int)((sp & 31) * 2);
    while (l < lim) {
        const int32_t rem = lim - l;
        const int64_t qi = (qp + l) >> 5, si = (sp + l) >> 5;
        ull a[5], b[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            a[j] = qw[min(qi + j, qmax)];
            b[j] = sw[min(si + j, smax)];
        }
        int32_t m = 0;
        bool stop = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!stop && 32 * j < rem) {
                ++chunks;
                const ull xq = (a[j] << qs) | ((a[j + 1] >> 1) >> (63 - qs));
                const ull xs = (b[j] << ss) | ((b[j + 1] >> 1) >> (63 - ss));
                const ull x = xq ^ xs;
                if (x) { m += (int32_t)(__clzll((long long)x) >> 1); stop = true; }
                else m += 32;
            }
        }
        if (m >= rem) return lim;
        l += m;
        if (stop) return l;
    }
    return l;
}

// Finds or inserts a key, going on from `c`, a value read from slot h earlier (it
// may be stale: a slot only ever goes from empty to a key, and an empty slot
// is claimed by compare-and-swap, which sees the current value); counts
// insertions in *n_ins.  -1 when the table is full.
__device__ int dir_settle(ull* dir, uint32_t mask, ull key, uint32_t h, ull c, int* n_ins) {
    for (uint32_t p = 0; p <= mask; ++p) {
        if (p > 0) c = __hip_atomic_load(&dir[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (c == key) return (int)h;
        if (c == 0) {
            const ull old = atomicCAS(&dir[h], 0ull, key);
            if (old == 0) { atomicAdd(n_ins, 1); return (int)h; }
            if (old == key) return (int)h;
        }
        h = (h + 1) & mask;
    }
    return -1;
}
// The same from the key's home slot.
__device__ __forceinline__ int dir_insert(ull* dir, uint32_t mask, ull key, int* n_ins) {
    const uint32_t h = dhash(key) & mask;
    return dir_settle(dir, mask, key, h, __hip_atomic_load(&dir[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), n_ins);
}

// Exclusive prefix sum of x >= 0 over the 64 lanes of the wave, plus the
// total.  Bit plane b adds 2^b times the number of lower lanes that have
// bit b set (ballot + mbcnt): no data moves between lanes, one ballot per
// bit plane in use (the counts here are small: outputs, claims, keeps).
__device__ __forceinline__ int wave_excl_scan(int x, int& total) {
    uint32_t rem = (uint32_t)x;
    int ex = 0, tot = 0;
    for (int b = 0; __ballot(rem != 0u); ++b, rem >>= 1) {
        const ull m = __ballot(rem & 1u);
        ex += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) << b;
        tot += __popcll(m) << b;
    }
    total = tot;
    return ex;
}

// Reserves cnt consecutive slots of an LDS counter (one atomic per wave,
// order between waves unspecified).  All lanes of the wave must call it.
__device__ __forceinline__ int wave_alloc(int cnt, int* counter) {
    int total;
    const int ex = wave_excl_scan(cnt, total);
    int base = 0;
    if (__lane_id() == 0 && total > 0) base = atomicAdd(counter, total);
    // lane 0's value to every lane: a lane read (one ALU instruction), not a
    // permute through LDS
    base = __builtin_amdgcn_readlane(base, 0);
    return base + ex;
}

// Workgroup barrier for phases that exchange only LDS data: waits for this
// wave's LDS operations, not for its outstanding global stores (which the
// full __syncthreads() would drain).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A 64-bit value that is the same in every lane, as a scalar.
__device__ __forceinline__ int64_t uniform64(int64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Exclusive prefix sum over the whole block in thread order (keeps lists
// sorted).  All threads must call it.
template <int BLOCK>
__device__ __forceinline__ int block_excl_scan(int x, int& total, int* scan) {
    constexpr int NW = BLOCK / 64;
    int wt;
    const int ex = wave_excl_scan(x, wt);
    const int w = threadIdx.x >> 6;
    if (NW == 1) { total = __builtin_amdgcn_readfirstlane(wt); return ex; }
    if (__lane_id() == 0) scan[w] = wt;
    lds_barrier();
    int off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int y = scan[i];
        off += (i < w) ? y : 0;
        tot += y;
    }
    lds_barrier();
    total = __builtin_amdgcn_readfirstlane(tot);   // block-uniform: kept in a scalar register
    return off + ex;
}

// A wavefront list: per entry the diagonal (v, k), its offset o and record
// page d in one 16-byte word, the walk length W and the trace index t in
// arrays of their own (each moved only by the modes that use it).  The label
// length l and base b of v are kept only for the diagonals a crossing round
// creates, by their number among them (their extension in the next round then
// needs no lookup); every other reader takes them from the graph's per-vertex
// label record.  Bit 31 of the page word is set when o = |v|, so that the
// expansion's sources need no label.
struct Lists {
    int4* e;          // (v, k, o, d)
    int32_t *w, *t, *l;
    int64_t* b;
};
constexpr int32_t AT_END = (int32_t)0x80000000;
__device__ __forceinline__ int32_t page_word(int32_t d, int32_t o, int32_t Lv) { return o == Lv ? d | AT_END : d; }
__device__ __forceinline__ int32_t page_of(int32_t w) { return w & ~AT_END; }
// The diagonal (v, k) of entry i (the first 8 bytes of its word).
__device__ __forceinline__ int2 vk_of(const Lists& L, int32_t i) {
    return *reinterpret_cast<const int2*>(&L.e[i]);
}
// Label base of a per-vertex label record.
__device__ __forceinline__ int64_t lab_base(int4 lab) {
    return (int64_t)(((uint64_t)(uint32_t)lab.y << 32) | (uint32_t)lab.x);
}

// LDS lists of the narrow path (narrow_scores): the list being expanded (slots
// 2 .. n+1, two sentinels on each side), the list being built and the crossing
// candidates.  Entries carry their vertex's label base and length.
struct Narrow {
    static constexpr int N = 64;       // entries of a list: one per lane of the wave
    static constexpr int C = 48;       // crossing candidates kept here, the rest in the arena
    static constexpr int R = 128;      // the expansion's candidates: up to 63 waiting and 63 of a step
    int4 ie[N + 4];
    int4 oe[N];
    int2 ring[R];                      // offset; source, slot and which source decides
    int64_t ib[N + 4], ob[N], cb[C];
    int32_t iw[N + 4], it[N + 4], il[N + 4];
    int32_t ow[N], ot[N], ol[N];
    int32_t cu[C], ck[C], cw[C], ct[C], cl[C];
};

// Candidate outputs of the expansion, in list order: (v, k, offset with bit 31
// set when the diagonal's record has to be checked, page or -1 when it has to
// be looked up), trace index, walk length.
template <bool TRACK>
struct CandRing {
    static constexpr int N = 128;
    int4 e[N];
    int32_t t[N];
    int32_t w[TRACK ? N : 1];
};

// Workgroup LDS, sized for the workgroup (merge keys, the staged batch) and
// the mode (the network's weights only where it runs).
template <int BLOCK, int MODE>
struct Shared {
    using Ring = CandRing<(MODE > 0)>;
    static constexpr int XS = xs_lds(BLOCK);
    static constexpr int NW = BLOCK / 64;
    static constexpr int SEGS = nsamp(BLOCK) / NW;   // samples of one part
    static constexpr int XC = MODE == 0 ? xstage(BLOCK) : 0;       // claimed diagonals staged
    static constexpr int CS = MODE == 0 ? 2 * xstage(BLOCK) : 0;   // crossing candidates staged
    int32_t read;
    int32_t n_out;    // entries in the list being built (outputs, then crossing entries)
    int32_t ncand;
    int32_t dirn;     // pages created
    int32_t mn;       // trace entries created
    int32_t flags;
    int32_t found;
    int32_t iend;     // largest end row reached (free end gap in the query)
    int32_t amax;
    int32_t imax;
    int32_t dropped;
    int32_t tend;
    uint32_t gen;
    ull endkey;
    ull chunks;
    ull cross;
    ull adm;
    ull mlp;
    ull tick[4];      // wall-clock ticks per phase (thread 0)
    ull acc[16];      // counters of the queries this workgroup has finished
    int32_t scan[16];
    ull samp[nsamp(BLOCK)]; // sort keys of entries 0, SAMP, 2 SAMP, ... of each part, written by the expansion
    // the parts of the list (Parts): first entry, first place, entries, first key
    int32_t partL[NW], partP[NW], partN[NW];
    int32_t newN[NW];       // entries of the parts being built
    ull partK[NW];
    // what the narrow path is called with and what it hands back (narrow_scores)
    int32_t nr_code, nr_s, nr_n, nr_n1, nr_round, nr_vmx, nr_list, nr_r;
    uint32_t nr_mask;
    int64_t nr_work, nr_arena;
    // The narrow path's lists share the storage of the wide path's arrays: a
    // score runs on one of the two.
    union {
        struct {
            ull skeys[XS];          // merge: keys of the crossing entries, then the bitmap of their merged positions
            int32_t sidx[XS];       // crossing entries in merged order
            int32_t xcnt[XS];       // merge: merged positions, then the bits below each word of the bitmap
            int32_t csu[CS + 1], csk[CS + 1], cst[CS + 1];   // crossing candidates: target, diagonal, trace index
            union {
                Ring ring[NW];      // expansion: each wave's candidates waiting to be extended
                struct {            // crossing rounds: claimed diagonals (vertex, diagonal, page, label length,
                                    // predecessor's trace index, label base)
                    int32_t xsv[XC + 1], xsk[XC + 1], xsd[XC + 1], xsl[XC + 1], xst[XC + 1];
                    int64_t xsb[XC + 1];
                };
            };
        };
        Narrow nw;
    };
    alignas(16) uint16_t mlpw[MODE >= 2 ? 4808 : 8];   // pruning network (bfloat16), loaded once per launch
    float mscale[8];        // feature scales
};

// The workgroup's LDS: one variable per instantiation, named through this
// function by the kernel and by the narrow path (a function of its own).
template <int BLOCK, int MODE>
__device__ __forceinline__ Shared<BLOCK, MODE>& lds() {
    __shared__ Shared<BLOCK, MODE> S;
    return S;
}

// The launch arguments as the kernel received them, in constant memory.
typedef const __attribute__((address_space(4))) KArgs* KernArg;
__device__ __forceinline__ KernArg kernarg() { return (KernArg)__builtin_amdgcn_kernarg_segment_ptr(); }
// The same through a pointer the compiler cannot follow: what is read through
// it is loaded (scalar cache) where it is used.  Read directly, every argument
// and every pointer made from one stays in scalar registers for the whole
// kernel, and with about 250 such values the compiler moves them to and from
// vector lanes in every inner loop.
__device__ __forceinline__ const KArgs& fresh_args() {
    KernArg p = kernarg();
    asm volatile("" : "+s"(p));
    return *(const KArgs*)p;
}

// Per-query view of the arena and of the read.
struct Q {
    const ull* rd;
    int64_t q0;
    int32_t qlen, vs;
    int32_t j0, j1;   // start window: the walk starts after the first j bases of vs, j0 <= j <= j1
    int32_t ve;       // end vertex (global form) or -1 (extension mode)
    int32_t ilo;      // end rows: ilo .. qlen (qlen minus the free end gap in the query)
    bool wfree;       // global form: the walk may end anywhere inside ve
    ull* dir;
    Page* pages;
    ull* mkey;
    int32_t* Tv;
    int32_t* Tt;
    uint32_t mask;
    uint32_t gen;
    bool tb, track;   // traced walks; walk lengths and lags tracked (pruning, dumps)
};

// The arena's parts and the launch's read store, from (fresh) arguments.
__device__ __forceinline__ void bind_q(Q& q, const KArgs& A, char* arena) {
    q.rd = A.rd;
    q.dir = reinterpret_cast<ull*>(arena + A.o_dir);
    q.pages = reinterpret_cast<Page*>(arena + A.o_pages);
    q.mkey = reinterpret_cast<ull*>(arena + A.o_mkey);
    q.Tv = reinterpret_cast<int32_t*>(arena + A.o_tv);
    q.Tt = reinterpret_cast<int32_t*>(arena + A.o_tt);
    q.tb = A.traceback != 0;
}
// View of query r in a workgroup's arena (mask and gen are set per attempt).
// The query's parameters are the same in every lane: readfirstlane keeps them
// in scalar registers (and tests on them branches of the whole wave).
template <int MODE>
__device__ __forceinline__ Q make_q(const KArgs& A, char* arena, int r) {
    Q q;
    q.q0 = uniform64(A.rd_off[r]);
    q.qlen = __builtin_amdgcn_readfirstlane((int32_t)(A.rd_off[r + 1] - q.q0));
    q.vs = __builtin_amdgcn_readfirstlane(A.v_start[r]);
    q.ve = __builtin_amdgcn_readfirstlane(A.v_end ? A.v_end[r] : A.end_vertex);
    q.j0 = __builtin_amdgcn_readfirstlane(A.v_off ? A.v_off[r] : 0);
    q.j1 = __builtin_amdgcn_readfirstlane(A.v_off_hi ? A.v_off_hi[r] : q.j0);
    q.ilo = max(0, q.qlen - A.end_free);
    q.wfree = A.walk_free != 0;
    bind_q(q, A, arena);
    q.track = MODE >= 1;   // the launch picks MODE >= 1 when pruning or dumping
    q.mask = 0;
    q.gen = 0;
    return q;
}
// List j (0 or 1) of an arena: entry words, W and t (MAIN_X + 1 times list_cap
// places), the crossing diagonals' labels (list_cap places).
__device__ __forceinline__ Lists list_of(const KArgs& A, char* arena, int j) {
    const int64_t lcap = A.list_cap, n = (MAIN_X + 1) * lcap;
    int32_t* p = reinterpret_cast<int32_t*>(arena + A.o_lists) + (int64_t)j * LIST_WORDS * lcap;
    Lists x;
    x.e = reinterpret_cast<int4*>(p);
    x.w = p + 4 * n; x.t = p + 5 * n; x.l = p + 6 * n;
    x.b = reinterpret_cast<int64_t*>(p + 6 * n + lcap);
    return x;
}
// Where the main entries of a list are: part w (written by wave w) holds
// entries L[w] .. L[w+1]-1 at places from P[w].  In scalar registers.
template <int NW>
struct Parts {
    int32_t L[NW], D[NW];   // first entry, place minus entry
    template <class SH>
    __device__ __forceinline__ explicit Parts(const SH& S) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            L[w] = __builtin_amdgcn_readfirstlane(S.partL[w]);
            D[w] = __builtin_amdgcn_readfirstlane(S.partP[w]) - L[w];
        }
    }
    __device__ __forceinline__ int32_t place(int32_t i) const {
        int32_t d = D[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) d = i >= L[w] ? D[w] : d;
        return i + d;
    }
};
// A list in one part, from place 0.
template <int NW, class SH>
__device__ __forceinline__ void one_part(SH& S, int32_t n) {
    if (threadIdx.x < NW) {
        S.partL[threadIdx.x] = threadIdx.x == 0 ? 0 : n;
        S.partP[threadIdx.x] = threadIdx.x == 0 ? 0 : n;
        S.partN[threadIdx.x] = threadIdx.x == 0 ? n : 0;
    }
}

template <class SH>
__device__ __forceinline__ int32_t trace_push_from(const Q& q, SH& S, int32_t v, int32_t tprev, ull probe);
// Algorithm 5: T gets (v, t) unless the pair is already there; the index of
// the pair's slot in the de-duplication map is its trace index.
template <class SH>
__device__ __forceinline__ int32_t trace_push(const Q& q, SH& S, int32_t v, int32_t tprev) {
    return trace_push_from(q, S, v, tprev,
                           __hip_atomic_load(&q.mkey[dhash(dkey(v, tprev)) & q.mask], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT));
}
// The same, given the value an earlier read found in the pair's first map
// slot (so that the read can go out with other loads).
template <class SH>
__device__ __forceinline__ int32_t trace_push_from(const Q& q, SH& S, int32_t v, int32_t tprev, ull probe) {
    const int ms = dir_settle(q.mkey, q.mask, dkey(v, tprev), dhash(dkey(v, tprev)) & q.mask, probe, &S.mn);
    if (ms < 0) { atomicOr(&S.flags, F_GROW); return -1; }
    // the slot's (v, tprev) is fixed by its key, so every inserter may write it
    q.Tv[ms] = v;
    q.Tt[ms] = tprev;
    return ms;
}

// Whether the front cell (v, o) of a diagonal can end a walk (the label of v
// has Lv bases): extension mode, any cell; global form, the last cell of ve,
// or any cell of ve when the walk's end gap is free.  A cell (v, 0) ends a
// walk only as the start cell (vs, 0).
__device__ __forceinline__ bool ends_walk(const Q& q, int32_t v, int32_t o, int32_t Lv) {
    if (q.ve >= 0 && (v != q.ve || (!q.wfree && o != Lv))) return false;
    return o >= 1 || (v == q.vs && q.j0 == 0);
}

// Records an extended diagonal: its record word when it is new or reached
// the vertex end, the end test and the pruning reductions; returns the number
// of out-edges to cross (0 unless the vertex end was reached).
template <class SH>
__device__ __forceinline__ int record_entry(const Q& q, SH& S, int32_t v, int32_t k, int32_t o, int32_t W,
                                            int32_t d, bool mark, int32_t Lv, int32_t deg, int2& lmax) {
    const int32_t i = k + o;
    // the record is written when the diagonal is new or may leave the
    // wavefront: at the vertex end, or with the query consumed (no mismatch
    // can advance it; in the global form the search goes on past i = |q|)
    if (mark || o == Lv || i == q.qlen) q.pages[d].R[k & 31] = mkR(q.gen, o);
    // end test: extension mode, any cell of the last query row; global form,
    // the cell at the end of the end vertex (Algorithm 1), or any cell of
    // the end vertex with a free end gap in the walk.  Offset-0 cells end a
    // walk only at the start cell (vs, 0): another one is the copy of a
    // predecessor's last cell.  With a free end gap in the query every row
    // from ilo on ends: the largest row reached is found here, its smallest
    // end cell once the score is complete.
    if (i >= q.ilo && ends_walk(q, v, o, Lv)) {
        S.found = 1;
        if (q.ilo < q.qlen) atomicMax(&S.iend, i);
        else atomicMin(&S.endkey, ((ull)(uint32_t)v << 32) | (uint32_t)o);
    }
    // Algorithm 4's a = i + W~ and the furthest row: this lane's maxima of the
    // score, reduced over the wave and the workgroup once the score is extended
    if (q.track) {
        lmax.x = max(lmax.x, i + W);
        lmax.y = max(lmax.y, i);
    }
    return (o == Lv) ? deg : 0;
}

// Extends one admitted diagonal (Algorithm 2) and records it.
template <class SH>
__device__ __forceinline__ int extend_entry(const KArgs& A, const Q& q, SH& S, int32_t v, int32_t k,
                                            int32_t& o, int32_t& W, int32_t d, bool mark, int64_t sb,
                                            int32_t Lv, int32_t deg, uint32_t& chunks, int2& lmax) {
    const int32_t i = k + o;
    const int32_t lim = min(q.qlen - i, Lv - o);
    const int32_t l = lcp(q.rd, q.q0 + i, ((q.q0 + q.qlen) >> 5) + 1, A.seg, sb + o, ((sb + Lv) >> 5) + 1, lim, chunks);
    o += l;
    W += l;
    return record_entry(q, S, v, k, o, W, d, mark, Lv, deg, lmax);
}

// Crossing candidate c: target u, diagonal k2 in u, walk length W, trace
// index t.  The first SH::CS (exact mode) go to LDS, the rest to the arena.
template <class SH>
__device__ __forceinline__ void put_cand(SH& S, const KArgs& A, int32_t* cu, int32_t* ck, int32_t* cW, int32_t* ct,
                                         int c, int32_t u, int32_t k2, int32_t W, int32_t t) {
    if (c < SH::CS) {
        S.csu[c] = u; S.csk[c] = k2; S.cst[c] = t;
    } else if (c < A.cand_cap) {
        cu[c] = u; ck[c] = k2; cW[c] = W; ct[c] = t;
    } else {
        atomicOr(&S.flags, F_LIST);
    }
}
// The candidates for the out-edges of a vertex whose out-edge record is vi
// (first edge, degree, first two targets), from slot c on.  Only the edges
// after the second need loads, in a branch of their own that ends by waiting
// for them: with a load inside the loop over all edges, or one possibly in
// flight after it, the compiler made the wave wait for every outstanding
// memory operation (the output stores and the next batch's entries among
// them) before each candidate, on every vertex.
template <class SH>
__device__ __forceinline__ void put_out_edges(SH& S, const KArgs& A, int32_t* cu, int32_t* ck, int32_t* cW,
                                              int32_t* ct, int c, int4 vi, int32_t k2, int32_t W, int32_t t) {
    const int deg = vi.y;
    if (deg > 0) put_cand(S, A, cu, ck, cW, ct, c, vi.z, k2, W, t);
    if (deg > 1) put_cand(S, A, cu, ck, cW, ct, c + 1, vi.w, k2, W, t);
    if (deg > 2) {
        for (int e = 2; e < deg; ++e) put_cand(S, A, cu, ck, cW, ct, c + e, A.out_dst[vi.x + e], k2, W, t);
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): no load of this branch outlives it
    }
}

// Bitonic sort of n keys (+ payload) in place, ascending; n is a power of 2.
// LDS=true when keys and payload are in LDS (stages then need LDS barriers only).
template <int BLOCK, bool LDS>
__device__ void bitonic(ull* keys, int32_t* idx, int n) {
    for (int kk = 2; kk <= n; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n; i += BLOCK) {
                const int p = i ^ j;
                if (p > i) {
                    const ull a = keys[i], b = keys[p];
                    const bool up = (i & kk) == 0;
                    if ((a > b) == up) {
                        keys[i] = b; keys[p] = a;
                        const int32_t t = idx[i]; idx[i] = idx[p]; idx[p] = t;
                    }
                }
            }
            if (LDS) lds_barrier(); else __syncthreads();
        }
    }
}

// Number of main entries of the list whose key is below a key, in two steps, so
// that the caller can put work between the loads and their use.  issue(): the
// part, by the parts' first keys; a search of the part's sampled keys in LDS
// (samp[j] = key of entry SAMP*j); the loads of the SAMP-1 entries between two
// samples, all together.  count(): how many of those are below.  Beyond the
// sampled entries issue() searches the list itself and leaves nothing to count.
struct LowerBound {
    int32_t c, a, b;      // entries below so far; entries a .. b-1 of the part are open
    int2 x[SAMP - 1];
    template <class SH>
    __device__ __forceinline__ void issue(const SH& S, const Lists& L, ull key) {
        int w = 0;                               // the last part whose first key is below key
#pragma unroll
        for (int j = 1; j < SH::NW; ++j)
            if (S.partN[j] > 0 && S.partK[j] < key) w = j;
        const int32_t n = S.partN[w], place = S.partP[w];
        const ull* const samp = S.samp + w * SH::SEGS;
        const int32_t ns = min((int32_t)SH::SEGS, (n + SAMP - 1) / SAMP);
        int32_t lo = 0, hi = ns;                 // samples below key
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (samp[mid] < key) lo = mid + 1; else hi = mid;
        }
        a = lo > 0 ? SAMP * (lo - 1) + 1 : 0;    // entry a-1 is below key
        b = min(SAMP * lo, n);                   // entry b is not below key (or b = n)
        if (lo == ns && SAMP * ns < n) {         // past the sampled entries
            int32_t h2 = n;
            while (a < h2) {
                const int32_t mid = (a + h2) >> 1;
                const int2 y = vk_of(L, place + mid);
                if (skey(y.x, y.y) < key) a = mid + 1; else h2 = mid;
            }
            b = a;
        }
        c = S.partL[w] + a;
        // every lane loads all SAMP-1 keys (indices clamped to the part)
#pragma unroll
        for (int32_t j = 0; j < SAMP - 1; ++j) x[j] = vk_of(L, place + max(min(a + j, n - 1), 0));
    }
    __device__ __forceinline__ int32_t count(ull key) const {
        int32_t r = c;
#pragma unroll
        for (int32_t j = 0; j < SAMP - 1; ++j) r += (a + j < b && skey(x[j].x, x[j].y) < key) ? 1 : 0;
        return r;
    }
};

// Merged view of a list whose main entries are sorted and whose crossing
// entries (unsorted in memory) have known merged positions: a bitmap over the
// merged positions (bit p & 63 of word p >> 6 set when position p holds a
// crossing entry), the number of bits set below each word, and the crossing
// entries in merged order.  The place of merged position p takes two
// independent LDS reads and a count; xb is the place of crossing entry 0.
template <int NW>
__device__ __forceinline__ int32_t merged_place(const ull* bm, const int32_t* pre, const int32_t* xidx,
                                                const Parts<NW>& parts, int32_t xb, int32_t p) {
    const ull word = bm[p >> 6];
    const int b = p & 63;
    const int32_t c = pre[p >> 6] + __popcll(word & ((1ull << b) - 1));
    return ((word >> b) & 1) ? xb + xidx[c] : parts.place(p - c);
}

__device__ __forceinline__ int32_t lower_bound_keys(const ull* keys, int32_t n, ull key) {
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (keys[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Copies entry i of a to slot j of b; W moves only when a pruning mode reads
// it, t only when walks are traced.
__device__ __forceinline__ void copy_entry(const Lists& a, int32_t i, const Lists& b, int32_t j, bool w, bool t) {
    b.e[j] = a.e[i];
    if (w) b.w[j] = a.w[i];
    if (t) b.t[j] = a.t[i];
}

// ---------------------------------------------------------------------------
// Learned keep/drop of wavefront diagonals.
//
// Eight features of a diagonal whose front cell is (i, v, off) at score s,
// with walk length W (a = i + W as in Algorithm 4), the largest a and i of the
// wavefront, the label length |v| and out-degree of v:
//   0 log1p(a_max - a)      lag behind the furthest diagonal
//   1 log1p(s)              score
//   2 log1p(outdeg(v))
//   3 log1p(i_max - i)      distance from the query frontier
//   4 log1p(|v| - off)      bases left in the vertex
//   5 sign * log1p(|W - i|) walk/query drift (deletions minus insertions)
//   6 i / |q|               progress
//   7 log1p(|q| - i)        query left
// each multiplied by a per-feature scale and rounded to bfloat16 before the
// network (gwfa_mlp_dev.h) scores the diagonal.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void entry_features(float* f, int32_t s, int32_t i, int32_t W, int32_t off, int32_t Lv,
                                               int32_t deg, int32_t amax, int32_t imax, int32_t qlen) {
    f[0] = log1pf((float)(amax - (i + W)));
    f[1] = log1pf((float)s);
    f[2] = log1pf((float)deg);
    f[3] = log1pf((float)(imax - i));
    f[4] = log1pf((float)(Lv - off));
    const int32_t dr = W - i;
    f[5] = dr >= 0 ? log1pf((float)dr) : -log1pf((float)(-dr));
    f[6] = qlen > 0 ? (float)i / (float)qlen : 0.0f;
    f[7] = log1pf((float)(qlen - i));
}

// ---------------------------------------------------------------------------
// Narrow wavefronts: scores whose lists have at most 64 entries are run by one
// wave on lists in LDS, with no barrier and one memory round trip per score
// (records, windows, out-edges and their labels together) and one per crossing
// round, where the wide path takes about eight (list, labels, records, stores
// drained before each barrier, list again for the merge and the pruning).
// Pruned runs and short reads stay here: a score of Algorithm 4 on the 1 Mb DAG
// has 5 entries, and its wide cost is round trips and about 1,500 instructions
// per wave, whatever the number of lanes at work.  Each lane makes one output
// diagonal's candidate (three slots of 21 source entries per step) and then
// extends one, so the windows, records and extension are written once.
// Bound now half by instructions (about 630 a score, one wave after the other
// on its SIMD) and half by the round trips: 2.2 us a score with 5 entries, 3 us
// with 16 waves on the CU, against 4.6 and 7.7 us on the wide path.  20,000
// reads of 10 kb on the 1 Mb DAG, Algorithm 4 (64 lanes): 15.9 -> 6.3 ms.  LDS is
// kept small enough for 16 one-wave workgroups on a CU (10,240 bytes each; the
// same code with 11,088 was 10% slower).
// Entered at 48 entries or fewer: from 49 on the next list usually exceeds 64
// and the score would be started here only to be handed over.
// ---------------------------------------------------------------------------
constexpr int NARROW_IN = 48;   // lists entering the narrow path; it leaves above Narrow::N
// how the narrow path left
constexpr int NR_WIDE = 0;      // (not run)
constexpr int NR_ROUNDS = 1;    // score nr_s outgrew it: nr_n entries in list 0, S.ncand candidates left to claim
constexpr int NR_END = 2;       // the query is done, status nr_n
constexpr int NR_FLAGS = 3;     // capacity exceeded, flags nr_n

__device__ __forceinline__ int lanes_below(ull m) {   // set bits of m below this lane
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ int64_t readlane64(int64_t x, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)(uint64_t)x, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)x >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
// LDS written by some lanes of the wave is read by others: the DS operations
// of a wave execute in order, so only the compiler has to keep the order.
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Largest x of the wave, in every lane's scalar registers: six steps of
// data-parallel moves (within rows of 16, then from row to row).
__device__ __forceinline__ int32_t wave_max(int32_t x) {
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x111, 0xf, 0xf, false));   // row_shr:1, 2, 4, 8
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1, 3
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2, 3
    return __builtin_amdgcn_readlane(x, 63);
}

// Continues the exact-match runs of the lanes with `more` (at query base qp,
// label base sp, at most rem bases).  One run is compared by the whole wave,
// 2,048 bases per memory round trip (a run between two errors of an accurate
// read is hundreds of bases; one lane alone compares 128 per round trip);
// several are taken four at a time, 16 lanes and 512 bases each.
__device__ __forceinline__ int32_t wave_extend(const ull* __restrict__ seg, const Q& q, bool more, int64_t qp, int64_t sp,
                                               int32_t rem, uint32_t& chunks) {
    ull need = __ballot(more);
    if (!need) return 0;
    const int lane = __lane_id();
    int32_t ext = 0;
    if ((need & (need - 1)) == 0) {
        const int l = __builtin_ctzll(need);
        const int64_t uq = readlane64(qp, l), us = readlane64(sp, l);
        const int32_t ur = __builtin_amdgcn_readlane(rem, l);
        int32_t e = 0;
        uint32_t w = 0;
        for (;;) {
            const int32_t off = e + 32 * lane;
            const bool in = off < ur;
            const int32_t o = in ? off : 0;
            const ull x = win32(q.rd, uq + o) ^ win32(seg, us + o);
            const int32_t rl = min(32, ur - off);
            const int32_t m = min(x ? (int32_t)(__clzll((long long)x) >> 1) : 32, rl);
            const ull bad = __ballot(in && m < rl);
            if (bad) {
                const int f = __builtin_ctzll(bad);
                e += 32 * f + __builtin_amdgcn_readlane(m, f);
                w += f + 1;
                break;
            }
            const int32_t g = min(ur - e, 2048);
            e += g;
            w += (uint32_t)(g + 31) >> 5;
            if (e >= ur) break;
        }
        if (lane == l) { ext = e; chunks += w; }
        return ext;
    }
    while (need) {
        // the run this lane's 16 work on (without one: they stand at the first
        // run, whose bases are in the stores; a lane without a run may be past them)
        int l = __builtin_ctzll(need);
        bool on = true;
        need &= need - 1;
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            const bool any = need != 0;
            const int b = any ? __builtin_ctzll(need) : 0;
            if ((lane >> 4) == j) { l = any ? b : l; on = any; }
            need &= need - 1;
        }
        const int64_t uq = __shfl(qp, l, 64), us = __shfl(sp, l, 64);
        const int32_t lr = __shfl(rem, l, 64);       // by every lane: a lane that sits an exchange out is read as 0
        const int32_t ur = on ? lr : 0;
        int32_t e = 0;
        uint32_t w = 0;
        bool go = on;
        while (__ballot(go)) {
            const int32_t off = e + 32 * (lane & 15);
            const bool in = go && off < ur;
            const int32_t o = in ? off : 0;
            const ull x = win32(q.rd, uq + o) ^ win32(seg, us + o);
            const int32_t rl = min(32, ur - off);
            const int32_t m = min(x ? (int32_t)(__clzll((long long)x) >> 1) : 32, rl);
            const ull bad = (__ballot(in && m < rl) >> (lane & 48)) & 0xffffull;
            const int f = bad ? __builtin_ctzll(bad) : 0;
            const int32_t mf = __shfl(m, (lane & 48) + f, 64);
            if (go) {
                if (bad) {
                    e += 32 * f + mf;
                    w += f + 1;
                    go = false;
                } else {
                    const int32_t g = min(ur - e, 512);
                    e += g;
                    w += (uint32_t)(g + 31) >> 5;
                    go = e < ur;
                }
            }
        }
        // back to the runs' lanes: lane l's run was taken by the group whose lanes name it
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int lj = __builtin_amdgcn_readlane(l, 16 * j);
            const int32_t ej = __builtin_amdgcn_readlane(e, 16 * j);
            const uint32_t wj = __builtin_amdgcn_readlane(w, 16 * j);
            if (__builtin_amdgcn_readlane((int)on, 16 * j) && lane == lj) { ext = ej; chunks += wj; }
        }
    }
    return ext;
}

__device__ __forceinline__ ull dir_load(const ull* tab, uint32_t h) {
    return __hip_atomic_load(&tab[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Length of the common prefix of q[qp ..] and label[sp ..], at most 64 bases
// (three words of each, loaded together).  `any`: qp and sp are bases of the
// query and the label; the stores' two words of padding then hold the third
// word, else (an empty rest at the end of the store) the second is read twice.
__device__ __forceinline__ int32_t first64(const ull* __restrict__ seg, const Q& q, int64_t qp, int64_t sp, bool any) {
    const ull *qw = q.rd + (qp >> 5), *sw = seg + (sp >> 5);
    const int qs = (int)((qp & 31) * 2), ss = (int)((sp & 31) * 2);
    const ull a0 = qw[0], a1 = qw[1], a2 = qw[any ? 2 : 1], b0 = sw[0], b1 = sw[1], b2 = sw[any ? 2 : 1];
    const ull x0 = ((a0 << qs) | ((a1 >> 1) >> (63 - qs))) ^ ((b0 << ss) | ((b1 >> 1) >> (63 - ss)));
    const ull x1 = ((a1 << qs) | ((a2 >> 1) >> (63 - qs))) ^ ((b1 << ss) | ((b2 >> 1) >> (63 - ss)));
    return x0 ? (int32_t)(__clzll((long long)x0) >> 1) : 32 + (x1 ? (int32_t)(__clzll((long long)x1) >> 1) : 32);
}
// A vertex's out-edges: first edge, degree, first two targets, and those
// targets' labels.
struct Out {
    int4 vi, l0, l1;
};
__device__ __forceinline__ Out load_out(const int4* __restrict__ vinfo, const int4* __restrict__ vsucc, int32_t v,
                                        bool want) {
    Out o;
    o.vi = make_int4(0, 0, -1, -1);
    o.l0 = o.l1 = make_int4(0, 0, 0, 0);
    if (want) {
        o.vi = vinfo[v];
        o.l0 = vsucc[2 * (int64_t)v];
        o.l1 = vsucc[2 * (int64_t)v + 1];
    }
    return o;
}
// Finds or creates the keys of the lanes with `act` in an open-addressing table
// that only this wave changes meanwhile: c is what was read from slot h.  No
// compare-and-swap: lanes that find the same slot empty settle it among
// themselves, the lowest first.  Returns the slot (-1: the table is full);
// `made`: this lane's key was not there.
template <class SH>
__device__ __forceinline__ int wave_settle(ull* tab, uint32_t mask, ull key, uint32_t h, ull c, bool act, bool& made,
                                           SH& S, bool trace = false) {
    const int lane = __lane_id();
    int slot = act && c == key ? (int)h : -1, n = 0;
    bool todo = act && c != key;
    made = false;
    for (uint32_t p = 0; __ballot(todo); ++p) {
        ull em = __ballot(todo && c == 0);
        while (em) {
            const int f = __builtin_ctzll(em);
            const uint32_t hf = (uint32_t)__builtin_amdgcn_readlane((int)h, f);
            const ull kf = (ull)readlane64((int64_t)key, f);
            const bool here = todo && c == 0 && h == hf;
            em &= ~__ballot(here);
            if (lane == f) __hip_atomic_store(&tab[hf], kf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (here) {
                if (key == kf) { slot = (int)hf; made = true; todo = false; }
                else c = kf;   // taken now
            }
            ++n;
        }
        if (p > mask) break;
        if (todo) {
            h = (h + 1) & mask;
            c = dir_load(tab, h);
            if (c == key) { slot = (int)h; todo = false; }
        }
    }
    if (n > 0 && lane == 0) {
        if (trace) S.mn += n; else S.dirn += n;
    }
    return slot;
}
// Appends the crossing candidates of the lanes with `at_end` (vertex v, target
// diagonal k2, walk length W, trace index t) to the nc there are: with their
// labels in LDS, beyond Narrow::C (a list that leaves the narrow path) in the
// arena.  o: v's out-edges where they have been loaded (`have`).
template <class SH>
__device__ __forceinline__ void put_crossings(SH& S, const KArgs& A, Narrow& L, int32_t* cu, int32_t* ck, int32_t* cW,
                                              int32_t* ct, int32_t& nc, bool at_end, Out o, bool have, int32_t v,
                                              int32_t k2, int32_t W, int32_t t) {
    if (__ballot(at_end && !have)) {
        const Out x = load_out(A.vinfo, A.vsucc, v, at_end && !have);
        if (at_end && !have) o = x;
    }
    const int deg = at_end ? o.vi.y : 0;
    int tot;
    const int c = nc + wave_excl_scan(deg, tot);
    nc += __builtin_amdgcn_readfirstlane(tot);
    for (int j = 0; j < deg; ++j) {
        const int32_t u = j == 0 ? o.vi.z : (j == 1 ? o.vi.w : A.out_dst[o.vi.x + j]);
        if (c + j < Narrow::C) {
            const int4 lab = j == 0 ? o.l0 : (j == 1 ? o.l1 : A.vlab[u]);
            L.cu[c + j] = u; L.ck[c + j] = k2; L.ct[c + j] = t; L.cw[c + j] = W;
            L.cl[c + j] = lab.z; L.cb[c + j] = lab_base(lab);
        } else if (c + j < A.cand_cap) {
            cu[c + j] = u; ck[c + j] = k2; cW[c + j] = W; ct[c + j] = t;
        } else {
            atomicOr(&S.flags, F_LIST);
        }
    }
}

// Runs scores from S.nr_s on as long as the lists stay narrow; called by the
// 64 lanes of wave 0.  List nr_list (nr_n entries, read through the merge's
// bitmap when nr_vmx) is the source of score s > 0, or holds the start
// entries (s = 0).  What is left for the wide path goes to list 0.  A
// function of its own: inlined, its scalars and the wide loop's do not fit
// the scalar registers together and the wide loop spills vector registers.
template <int BLOCK, int MODE>
__device__ __attribute__((noinline)) void narrow_scores(int64_t karg) {
    using SH = Shared<BLOCK, MODE>;
    SH& S = lds<BLOCK, MODE>();
    const KArgs& A = *(const KArgs*)(KernArg)uniform64(karg);
    char* const arena = (char*)uniform64(S.nr_arena);
    Q q = make_q<MODE>(A, arena, __builtin_amdgcn_readfirstlane(S.nr_r));
    q.mask = __builtin_amdgcn_readfirstlane(S.nr_mask);
    q.gen = __builtin_amdgcn_readfirstlane(S.gen);
    const int32_t half = (int32_t)((q.mask + 1) >> 1);
    int32_t s = __builtin_amdgcn_readfirstlane(S.nr_s), n = __builtin_amdgcn_readfirstlane(S.nr_n);
    const int32_t vmx = __builtin_amdgcn_readfirstlane(S.nr_vmx);
    const int32_t xb = MAIN_X * A.list_cap;
    const Lists L0 = list_of(A, arena, 0), Ls = list_of(A, arena, __builtin_amdgcn_readfirstlane(S.nr_list));
    int32_t* cu = reinterpret_cast<int32_t*>(arena + A.o_cand);
    int32_t *ck = cu + A.cand_cap, *cW = cu + 2 * (int64_t)A.cand_cap, *ct = cu + 3 * (int64_t)A.cand_cap;
    uint32_t chunks = 0;
    constexpr bool LEARN = MODE >= 2;
    constexpr int SRC = 21;             // sources per step (three output slots each)
    Narrow& L = S.nw;
    const int lane = __lane_id();
    const int li = lane / 3, lj = lane - 3 * li;
    // the arguments every score reads, held in scalar registers (from constant
    // memory the compiler would load them again at each use, and wait)
    const int4 *vinfo = A.vinfo, *vsucc = A.vsucc;
    const ull* seg = A.seg;
    int32_t max_score = A.max_score, a_diff = MODE == 1 && A.prune == GWFA_PRUNE_HEURISTIC ? A.a_diff : 0x7fffffff;
    asm volatile("" : "+s"(vinfo), "+s"(vsucc), "+s"(seg), "+s"(max_score), "+s"(a_diff));
    const ull t_in = wall_clock64();
    ull t_rounds = 0;
    int64_t work = 0;
    int32_t adm = 0, cross = 0, dropped = 0, evals = 0;
    int code = NR_WIDE, val = 0, round = 0;
    int32_t n1 = 0, ntot = 0, nc = 0;
    int2 lmax = make_int2(0, 0);
    // ---- the list from memory
    {
        int4 e = make_int4(-1, 0, 0, 0);
        int32_t w = 0, t = -1, l = 0;
        int64_t b = 0;
        if (lane < n) {
            const Parts<SH::NW> parts(S);
            const int32_t p = s == 0 ? xb + lane
                                     : (vmx ? merged_place(S.skeys, S.xcnt, S.sidx, parts, xb, lane) : parts.place(lane));
            e = Ls.e[p];
            e.w = page_of(e.w);
            if (q.track) w = Ls.w[p];
            if (q.tb) t = Ls.t[p];
            const int4 lab = A.vlab[e.x];
            l = lab.z;
            b = lab_base(lab);
        }
        wave_lds_order();   // the bitmap (same storage) is read before the lists are written
        if (s == 0) {
            L.oe[lane] = e; L.ow[lane] = 0; L.ot[lane] = t; L.ol[lane] = l; L.ob[lane] = b;
        } else {
            L.ie[lane + 2] = e; L.iw[lane + 2] = w; L.it[lane + 2] = t; L.il[lane + 2] = l; L.ib[lane + 2] = b;
        }
        if (lane < 2) {
            L.ie[lane] = make_int4(-1, 0, 0, 0);
            L.ie[lane + 66] = make_int4(-1, 0, 0, 0);
        }
        wave_lds_order();
    }
    for (;;) {
        n1 = 0;
        nc = 0;
        lmax = make_int2(0, 0);
        if (s > 0) {
            if (lane == 0) { S.found = 0; S.iend = -1; S.endkey = ~0ull; }
            // ========== EXPAND + EXTEND ==========
            // sources: three output slots of 21 entries per step; the candidates
            // go to a ring in list order, and 64 of them at a time (usually all
            // of the score's) are extended, one per lane
            int32_t head = 0, fill = 0;
            for (int32_t c0 = 0; c0 < n; c0 += SRC) {
                const bool src = lane < 3 * SRC && c0 + li < n;
                const int32_t si = min(c0 + li, n - 1) + 2;
                const int4 em2 = L.ie[si - 2], em1 = L.ie[si - 1], e0 = L.ie[si], ep1 = L.ie[si + 1], ep2 = L.ie[si + 2];
                const int32_t v = e0.x, k = e0.y;
                const int32_t Lv = L.il[si];
                const bool pm1 = em1.x == v && em1.y == k - 1;
                const bool pm2 = pm1 ? (em2.x == v && em2.y == k - 2) : (em1.x == v && em1.y == k - 2);
                const bool pp1 = ep1.x == v && ep1.y == k + 1;
                const int4 ez = pp1 ? ep2 : ep1;
                const bool pp2 = ez.x == v && ez.y == k + 2;
                // output diagonal kk; its sources: kk-1 (insertion), kk (mismatch), kk+1 (deletion)
                const int32_t kk = k - 1 + lj;
                const bool own = src && (lj == 2 || (!pm1 && (lj == 1 || !pm2)));
                const bool hasB = lj == 1 || (lj == 2 && pp1);
                const bool hasC = lj == 0 || (lj == 1 ? pp1 : pp2);
                const int bi = lj == 1 ? si : si + 1;
                const int ci = lj == 0 ? si : (lj == 1 || !pp1 ? si + 1 : si + 2);
                const int32_t oB = lj == 1 ? e0.z : ep1.z;
                const int32_t oC = lj == 0 ? e0.z : (lj == 1 ? ep1.z : ez.z);
                const int32_t W0 = q.track ? L.iw[si] : 0, WB = q.track ? L.iw[bi] : 0, WC = q.track ? L.iw[ci] : 0;
                int32_t bo = -1, bw = -1, from = si << 1;   // the deciding source's slot, and whether it adds a walk base
                if (lj == 2 && k + e0.z < q.qlen) { bo = e0.z; bw = W0; }
                if (hasB && kk + oB < q.qlen && oB < Lv && (oB + 1 > bo || (oB + 1 == bo && WB + 1 > bw))) {
                    bo = oB + 1; bw = WB + 1; from = (bi << 1) | 1;
                }
                if (hasC && oC < Lv && (oC + 1 > bo || (oC + 1 == bo && WC + 1 > bw))) {
                    bo = oC + 1; bw = WC + 1; from = (ci << 1) | 1;
                }
                const bool cand = own && bo > (hasB ? oB : -1);
                const ull cm = __ballot(cand);
                if (cand)   // source and slot (the diagonal and its page follow), whether its record decides
                    L.ring[(head + fill + lanes_below(cm)) & (Narrow::R - 1)] =
                        make_int2(bo, si | (lj << 8) | (from << 10) | (hasB ? 0 : 1 << 20));
                fill += __popcll(cm);
                wave_lds_order();
                while (fill >= 64 || (fill > 0 && c0 + SRC >= n)) {
                    const int cnt = min(fill, 64);
                    const bool act = lane < cnt;
                    const int2 c = L.ring[(head + (act ? lane : 0)) & (Narrow::R - 1)];
                    head += cnt;
                    fill -= cnt;
                    const int32_t sj = c.y & 255, j = (c.y >> 8) & 3;
                    const int4 se = L.ie[sj];
                    const int32_t lv = L.il[sj];
                    const int64_t sb = L.ib[sj];
                    const int32_t sv = se.x, sk = se.y - 1 + j, b0 = c.x;
                    const bool chk = act && (c.y >> 20);   // the diagonal's record decides
                    const int32_t fr = (c.y >> 11) & 127;
                    const int32_t ct0 = q.tb ? L.it[fr] : -1, cw0 = q.track ? L.iw[fr] + ((c.y >> 10) & 1) : 0;
                    const bool far = chk && (sk >> 5) != (se.y >> 5);
                    int pg = chk || j == 1 ? se.w : L.ie[sj + 1].w;
                    // directory, record, out-edges, successors' labels and windows in one
                    // round of loads; a diagonal on another page than its source is looked
                    // for in its key's home slot
                    const ull key = dkey(sv, sk >> 5);
                    const uint32_t h = dhash(key) & q.mask;
                    const ull dprobe = far ? dir_load(q.dir, h) : key;
                    const int32_t m = act ? min(q.qlen - (sk + b0), lv - b0) : 0;
                    const ull rw = q.pages[far ? (int)h : pg].R[sk & 31];
                    const Out o1 = load_out(vinfo, vsucc, sv, act && lv - b0 <= 64);
                    const int64_t qp = q.q0 + (m > 0 ? sk + b0 : 0), sp = sb + (m > 0 ? b0 : 0);
                    int32_t lx = first64(seg, q, qp, sp, m > 0);
                    ull r2 = rw;
                    if (__ballot(far)) {
                        bool made;
                        const int f = wave_settle(q.dir, q.mask, key, h, dprobe, far, made, S);
                        if (far) {
                            pg = f;
                            if (made) r2 = 0;
                            else if (f >= 0 && f != (int)h) r2 = q.pages[f].R[sk & 31];
                        }
                    }
                    const bool rec = chk && pg >= 0 && rgen(r2) == q.gen;
                    const bool ov = act && !(rec && b0 <= rval(r2));
                    lx = ov ? min(lx, m) : 0;
                    if (ov && m > 0) chunks += lx >= 32 && m > 32 ? 2 : 1;
                    lx += wave_extend(seg, q, lx == 64 && m > 64, qp + 64, sp + 64, m - 64, chunks);
                    const ull om = __ballot(ov);
                    const int32_t p = n1 + lanes_below(om);
                    n1 += __popcll(om);
                    int ncr = 0;
                    const int32_t o = b0 + lx, W = cw0 + lx;
                    if (ov) {
                        if (pg < 0) {
                            atomicOr(&S.flags, F_GROW);
                        } else {
                            ncr = record_entry(q, S, sv, sk, o, W, pg, chk && !rec, lv, o == lv ? 1 : 0, lmax);
                            if (p < Narrow::N) {
                                L.oe[p] = make_int4(sv, sk, o, pg); L.ol[p] = lv; L.ob[p] = sb;
                                if (q.track) L.ow[p] = W;
                                if (q.tb) L.ot[p] = ct0;
                            } else {   // more than a narrow list: it goes on in the wide path
                                L0.e[p] = make_int4(sv, sk, o, page_word(pg, o, lv));
                                if (q.track) L0.w[p] = W;
                                if (q.tb) L0.t[p] = ct0;
                                if ((p & (SAMP - 1)) == 0) S.samp[p / SAMP] = skey(sv, sk);
                            }
                        }
                    }
                    if (__ballot(ncr != 0)) put_crossings(S, A, L, cu, ck, cW, ct, nc, ncr != 0, o1, lv - b0 <= 64, sv, sk + lv, W, ct0);
                    wave_lds_order();
                }
            }
            adm += n1;
        }
        wave_lds_order();
        // ========== crossings, in rounds ==========
        int32_t xhi = n1;
        if (s == 0) {
            // the start entries: extended where they stand, their trace records are there
            const bool act = lane < n;
            const int ix = act ? lane : 0;
            const int4 e = L.oe[ix];
            const int32_t lv = L.ol[ix], t = q.tb ? L.ot[ix] : -1;
            const int64_t sb = L.ob[ix];
            const int32_t m = act ? min(q.qlen - (e.y + e.z), lv - e.z) : 0;
            const bool near = lv - e.z <= 64;
            const Out o1 = load_out(vinfo, vsucc, e.x, act && near);
            const int64_t qp = q.q0 + (m > 0 ? e.y + e.z : 0), sp = sb + (m > 0 ? e.z : 0);
            int32_t lx = min(first64(seg, q, qp, sp, m > 0), m);
            if (m > 0) chunks += lx >= 32 && m > 32 ? 2 : 1;
            lx += wave_extend(seg, q, lx == 64 && m > 64, qp + 64, sp + 64, m - 64, chunks);
            const int32_t o = e.z + lx;
            int ncr = 0;
            if (act) {
                ncr = record_entry(q, S, e.x, e.y, o, lx, e.w, true, lv, o == lv ? 1 : 0, lmax);
                L.oe[lane].z = o;
                if (q.track) L.ow[lane] = lx;
            }
            if (__ballot(ncr != 0)) put_crossings(S, A, L, cu, ck, cW, ct, nc, ncr != 0, o1, near, e.x, e.y + lv, lx, t);
            xhi = n;
            wave_lds_order();
        }
        bool timed = false;
        ull tr = 0;
        for (round = 0;; ++round) {
            const int f1 = __builtin_amdgcn_readfirstlane(S.flags | ((S.dirn > half || S.mn > half) ? F_GROW : 0));
            if (f1) { code = NR_FLAGS; val = f1; break; }
            if (xhi + nc > Narrow::N || nc > Narrow::C) { code = NR_ROUNDS; break; }   // may outgrow the narrow lists
            if (nc == 0) break;
            if (!timed) { timed = true; tr = wall_clock64(); }
            // Claim and extend in one step: a candidate carries its vertex's label
            // (from its predecessor's out-edge record), so that the directory, the
            // record at the key's home slot, the trace map and the windows are read
            // together, before it is known whether the diagonal was seen.  One wave
            // holds every candidate, so equal ones meet here and no atomic is
            // needed: the lowest lane takes the diagonal, with the largest W.
            const bool act = lane < nc;
            const int ci = act ? lane : 0;
            const int32_t u = L.cu[ci], kc = L.ck[ci], tc = q.tb ? L.ct[ci] : -1;
            const int32_t lv = L.cl[ci];
            const int64_t sb = L.cb[ci];
            int32_t wc = q.track ? L.cw[ci] : 0;
            const ull key = dkey(u, kc >> 5), tkey = dkey(u, tc);
            const uint32_t h = dhash(key) & q.mask, th = dhash(tkey) & q.mask;
            const ull dprobe = dir_load(q.dir, h);
            const ull wh = __hip_atomic_load(&q.pages[h].R[kc & 31], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const ull tprobe = q.tb ? dir_load(q.mkey, th) : 0ull;
            const int32_t m = act ? min(q.qlen - kc, lv) : 0;
            const Out o1 = load_out(vinfo, vsucc, u, act && lv <= 64);
            const int64_t qp = q.q0 + (m > 0 ? kc : 0), sp = sb;
            int32_t lx = min(first64(seg, q, qp, sp, m > 0), m);
            // seen, when the page is there and holds a record of this query
            bool fresh = act && !(dprobe == key && rgen(wh) == q.gen);
            ull walk = __ballot(fresh && dprobe != key && dprobe != 0);   // another key's slot: look further
            uint32_t hs = h;
            ull dp = dprobe;
            while (walk) {
                const bool mine = (walk >> lane) & 1;
                if (mine) { hs = (hs + 1) & q.mask; dp = dir_load(q.dir, hs); }
                const bool hit = mine && dp == key;
                if (hit && rgen(__hip_atomic_load(&q.pages[hs].R[kc & 31], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == q.gen)
                    fresh = false;
                walk = __ballot(mine && dp != key && dp != 0 && hs != h);
            }
            ull todo = __ballot(fresh), lead = 0;
            while (todo) {
                const int f = __builtin_ctzll(todo);
                const ull same = __ballot(fresh && u == __builtin_amdgcn_readlane(u, f) &&
                                          kc == __builtin_amdgcn_readlane(kc, f));
                lead |= 1ull << f;
                todo &= ~same;
                if (q.track && (same & (same - 1))) {
                    int32_t wm = (same >> lane) & 1 ? wc : 0;
                    for (int j = 32; j >= 1; j >>= 1) wm = max(wm, __shfl_xor(wm, j, 64));
                    if (lane == f) wc = wm;
                }
            }
            nc = 0;
            if (lead) {
                const bool ld = (lead >> lane) & 1;
                bool made;
                const int ds = wave_settle(q.dir, q.mask, key, hs, dp, ld, made, S);
                if (ld && m > 0) chunks += lx >= 32 && m > 32 ? 2 : 1;
                lx += wave_extend(seg, q, ld && lx == 64 && m > 64, qp + 64, sp + 64, m - 64, chunks);
                int32_t t = -1;
                if (q.tb) {   // Algorithm 5: T gets (u, tc) unless the pair is there
                    t = wave_settle(q.mkey, q.mask, tkey, th, tprobe, ld, made, S, true);
                    if (ld && t >= 0) { q.Tv[t] = u; q.Tt[t] = tc; }
                }
                const int32_t W = wc + lx;
                int ncr = 0;
                if (ld) {
                    if (ds < 0 || (q.tb && t < 0)) {
                        atomicOr(&S.flags, F_GROW);
                    } else {
                        ncr = record_entry(q, S, u, kc, lx, W, ds, true, lv, lx == lv ? 1 : 0, lmax);
                        const int32_t p = xhi + lanes_below(lead);
                        L.oe[p] = make_int4(u, kc, lx, ds);
                        L.ol[p] = lv; L.ob[p] = sb;
                        if (q.track) L.ow[p] = W;
                        if (q.tb) L.ot[p] = t;
                    }
                }
                const int add = __popcll(lead);
                xhi += add;
                cross += add;
                wave_lds_order();   // the candidates are read before the next ones are written
                if (__ballot(ncr != 0)) put_crossings(S, A, L, cu, ck, cW, ct, nc, ncr != 0, o1, lv <= 64, u, kc + lv, W, t);
                wave_lds_order();
            }
        }
        if (timed) t_rounds += wall_clock64() - tr;
        ntot = xhi;
        if (code != NR_WIDE) break;
        work += ntot;
        int32_t amax = 0, imax = 0;
        if (q.track) {
            amax = wave_max(lmax.x);
            if (LEARN) imax = wave_max(lmax.y);
        }
        // this lane's entry of the score's list: outputs first, then crossing entries
        const bool ent = lane < ntot;
        const int li2 = ent ? lane : 0;
        const int4 e = L.oe[li2];
        const int32_t eW = q.track ? L.ow[li2] : 0, eT = q.tb ? L.ot[li2] : -1, eL = L.ol[li2];
        const int64_t eB = L.ob[li2];
        // ========== end test ==========
        if (__builtin_amdgcn_readfirstlane(S.found)) {
            int32_t iend = q.qlen;
            if (q.ilo < q.qlen) {
                iend = __builtin_amdgcn_readfirstlane(S.iend);
                if (ent && e.y + e.z == iend && ends_walk(q, e.x, e.z, eL))
                    atomicMin(&S.endkey, ((ull)(uint32_t)e.x << 32) | (uint32_t)e.z);
                wave_lds_order();
            }
            if (q.tb) {
                const int32_t ev = (int32_t)(S.endkey >> 32), eo = (int32_t)(S.endkey & 0xffffffffull);
                if (lane == 0) S.tend = -1;
                wave_lds_order();
                if (ent && e.x == ev && e.z == eo && e.y + eo == iend) S.tend = eT;
            }
            code = NR_END; val = GWFA_ST_OK;
            break;
        }
        if (max_score >= 0 && s >= max_score) { code = NR_END; val = GWFA_ST_MAX_SCORE; break; }
        if (ntot == 0) { code = NR_END; val = q.ve >= 0 ? GWFA_ST_UNREACHABLE : GWFA_ST_MAX_SCORE; break; }
        if (q.ve < 0 && s > q.qlen + 1) { code = NR_END; val = GWFA_ST_MAX_SCORE; break; }
        // ========== merge of the crossing entries, and Algorithm 4 ==========
        {
            bool keep = ent;
            if (MODE == 1 && amax > a_diff) {
                keep = ent && amax - (e.y + e.z + eW) < a_diff;
                const ull dm = __ballot(ent && !keep);
                if (ent && !keep) q.pages[e.w].R[e.y & 31] = mkR(q.gen, e.z);   // the record stays
                dropped += __popcll(dm);
            }
            const ull km = __ballot(keep);
            const ull lowm = n1 >= 64 ? ~0ull : (1ull << n1) - 1;
            const ull mo = km & lowm;
            ull mc = km & ~lowm;
            const ull key = skey(e.x, e.y);
            int32_t pos = lanes_below(mo);        // kept outputs before this one (crossing entries: set below)
            if (mc) {
                const bool crossing = lane >= n1;
                int32_t cnt = 0, outs = 0;
                while (mc) {
                    const int f = __builtin_ctzll(mc);
                    mc &= mc - 1;
                    const ull kf = (ull)readlane64((int64_t)key, f);
                    cnt += kf < key ? 1 : 0;
                    const int32_t b = __popcll(__ballot(key < kf) & mo);
                    if (lane == f) outs = b;
                }
                pos = (crossing ? outs : pos) + cnt;
            }
            n = __popcll(km);
            wave_lds_order();
            if (keep) {
                L.ie[pos + 2] = e; L.il[pos + 2] = eL; L.ib[pos + 2] = eB;
                if (q.track) L.iw[pos + 2] = eW;
                if (q.tb) L.it[pos + 2] = eT;
            }
            if (lane < 2) L.ie[n + 2 + lane] = make_int4(-1, 0, 0, 0);
            wave_lds_order();
        }
        // ========== learned keep/drop ==========
        if (LEARN && A.prune == GWFA_PRUNE_LEARNED && n >= A.mlp_gate && (s % A.mlp_period) == 0) {
            const bool live = lane < n;
            const int ix = (live ? lane : 0) + 2;
            const int4 c = L.ie[ix];
            const int32_t cw2 = L.iw[ix], cl = L.il[ix], c_t = q.tb ? L.it[ix] : -1;
            const int64_t cb = L.ib[ix];
            const int32_t i = c.y + c.z;
            float f[8];
            entry_features(f, s, i, cw2, c.z, cl, vinfo[c.x].y, amax, imax, q.qlen);
            const float z = mlp_logit_wave(f, S.mscale, S.mlpw);
            const bool keep = live && (z >= A.keep_threshold || i + cw2 == amax);   // the furthest diagonal stays
            if (live && !keep) q.pages[c.w].R[c.y & 31] = mkR(q.gen, c.z);
            const ull km = __ballot(keep);
            evals += n;
            dropped += n - __popcll(km);
            n = __popcll(km);
            const int32_t pos = lanes_below(km);
            wave_lds_order();
            if (keep) {
                L.ie[pos + 2] = c; L.iw[pos + 2] = cw2; L.il[pos + 2] = cl; L.ib[pos + 2] = cb;
                if (q.tb) L.it[pos + 2] = c_t;
            }
            if (lane < 2) L.ie[n + 2 + lane] = make_int4(-1, 0, 0, 0);
            wave_lds_order();
        }
        ++s;
    }
    // ========== what is left for the wide path ==========
    if (code == NR_ROUNDS) {
        if (q.track) lmax = make_int2(wave_max(lmax.x), wave_max(lmax.y));
        if (lane < min(ntot, Narrow::N)) {
            const int4 e = L.oe[lane];
            const int32_t p = lane < n1 ? lane : xb + lane - n1;
            L0.e[p] = make_int4(e.x, e.y, e.z, page_word(e.w, e.z, L.ol[lane]));
            if (q.track) L0.w[p] = L.ow[lane];
            if (q.tb) L0.t[p] = L.ot[lane];
            if (lane < n1 && (lane & (SAMP - 1)) == 0) S.samp[lane / SAMP] = skey(e.x, e.y);
        }
        // the candidates to where the wide path looks for them
        const int cj = min(lane, Narrow::C - 1);
        const int32_t u2 = L.cu[cj], k2 = L.ck[cj], w2 = q.track ? L.cw[cj] : 0, t2 = L.ct[cj];
        wave_lds_order();
        if (lane < min(nc, Narrow::C)) put_cand(S, A, cu, ck, cW, ct, lane, u2, k2, w2, t2);
        for (int c = Narrow::C + lane; c < min(nc, (int)SH::CS); c += 64) {
            S.csu[c] = cu[c]; S.csk[c] = ck[c]; S.cst[c] = ct[c];
        }
        one_part<SH::NW>(S, n1);
        if (lane == 0) {
            S.ncand = nc; S.n_out = ntot; S.nr_n1 = n1; S.nr_round = round;
            S.amax = lmax.x; S.imax = lmax.y;
        }
        val = ntot;
    }
    for (int j = 32; j >= 1; j >>= 1) chunks += __shfl_xor(chunks, j, 64);
    if (lane == 0) {
        S.chunks += (ull)chunks;
        S.nr_code = code; S.nr_s = s; S.nr_n = val; S.nr_work = work;
        S.adm += (ull)adm; S.cross += (ull)cross; S.dropped += dropped;
        if (LEARN) S.mlp += (ull)evals;
        const ull t_out = wall_clock64();
        S.tick[0] += t_out - t_in - t_rounds;
        S.tick[1] += t_rounds;
    }
}

// ---------------------------------------------------------------------------
// EXPAND (Algorithm 3) + EXTEND of what it admits, on lists of any size.
//
// Every wave takes a part of the source list (whole groups of 64 entries, in
// order) and runs through it on its own, with no barrier until the end.
//   Sources: one entry per lane.  An output diagonal k' is owned by the
// present source with the smallest k among k'-1, k', k'+1, and those are the
// source's neighbours in the list, which the lanes exchange by whole-wave
// shifts (the group before and the group after fill in at the ends); each
// source makes up to three candidates, which go to the wave's ring in LDS in
// list order.  The next group's entries and labels are loaded meanwhile.
//   Outputs: whenever the ring holds 64 candidates, one per lane: labels are
// loaded, then the windows they lead to, out-edge records and records, the run
// is extended, and the outputs are written behind the wave's previous ones (at
// most three per source, so the part's place in the new list is known from the
// start).
// Before, a block staged 256 entries in LDS, each lane computed three output
// slots of which one is taken on average, and three barriers and a scan
// ordered the outputs of every batch (800 vector instructions a wave and
// batch; here about 160 per 64 sources and 220 per 64 outputs).  What bounds
// it now: the two round trips of a batch and its stores.  On the 1 Mb and the
// 10 Mb workload the waves wait 66 and 72% of their cycles, with the vector
// units 50% busy and 381 and 927 cycles to a read of the L2, of which 52 and
// 38% hit; the latter moves 5.2 TB/s, as much as a copy (a record word is read
// for every candidate, also where it decides nothing).  The registers (128,
// four waves a SIMD) leave room for no deeper queue.  Per call: 20,000 reads on the 1 Mb DAG 135.5 -> 115 ms, 3,001 noisy reads on the
// 10 Mb graph 459 -> 397 ms (its hardest read takes most of that alone), 500
// reads of 100 kb through loops 518 -> 237 ms (its lists of 25,000 to 50,000
// entries are merged by the bitmap now, which holds 65,536 positions instead
// of 32,768).
// ---------------------------------------------------------------------------
// x of the lane below (above), `edge` in lane 0 (63)
__device__ __forceinline__ int32_t lane_below(int32_t x, int32_t edge) {
    return __builtin_amdgcn_update_dpp(edge, x, 0x138, 0xf, 0xf, false);   // wave_shr:1
}
__device__ __forceinline__ int32_t lane_above(int32_t x, int32_t edge) {
    return __builtin_amdgcn_update_dpp(edge, x, 0x130, 0xf, 0xf, false);   // wave_shl:1
}
__device__ __forceinline__ int32_t rdl(int32_t x, int l) { return __builtin_amdgcn_readlane(x, l); }

template <int BLOCK, int MODE>
__device__ __forceinline__ void expand_part(const KArgs& A, const Q& q, Shared<BLOCK, MODE>& S, const Lists& Ls,
                                            const Lists& Ld, int32_t n, int32_t vmx, int32_t* cu, int32_t* ck,
                                            int32_t* cW, int32_t* ct, uint32_t& chunks, int2& lmax) {
    using SH = Shared<BLOCK, MODE>;
    constexpr int NW = SH::NW;
    const int lane = __lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    typename SH::Ring& R = S.ring[wv];
    const Parts<NW> parts(S);
    const int32_t xb = MAIN_X * A.list_cap;
    const int4* __restrict__ vinfo = A.vinfo;
    const int4* __restrict__ vlab = A.vlab;
    const ull* __restrict__ seg = A.seg;
    auto part_lo = [&](int w) { return w >= NW ? n : (int32_t)(((int64_t)n * w / NW) & ~63); };
    const int32_t lo = part_lo(wv), hi = part_lo(wv + 1);
    const int32_t place0 = MAIN_X * lo;
    int32_t nout = 0;            // outputs written
    int32_t head = 0, fill = 0;  // the ring
    ull* const samp = S.samp + wv * SH::SEGS;

    struct Ent { int4 e; int32_t w, t; };
    // the entries at merged positions base + lane (base a multiple of 64)
    auto fetch = [&](int32_t base, Ent& x, int from = 0) {
        x.e = make_int4(-1, 0, 0, 0);
        x.w = 0;
        x.t = -1;
        if (base + lane < n && lane >= from) {
            int32_t p;
            if (vmx) {
                const ull word = uniform64(S.skeys[base >> 6]);
                const int32_t c = S.xcnt[base >> 6] + lanes_below(word);
                p = ((word >> lane) & 1) ? xb + S.sidx[c] : parts.place(base + lane - c);
            } else {
                p = parts.place(base + lane);
            }
            x.e = Ls.e[p];
            if (q.track) x.w = Ls.w[p];
            if (q.tb) x.t = Ls.t[p];
        }
    };
    // Batches of up to 64 candidates, one per lane.  PIPE: in two stages behind
    // the sources, `one` with its labels on the way, `two` its first windows,
    // out-edges and records; a batch is finished two groups after it was taken, so
    // both round trips pass under the work on the groups between.  Where a wave's
    // part is long: 1 Mb DAG 122.3 -> 118.8 ms, 10 Mb graph 429 -> 406 ms against
    // one batch after the other (both at 256 lanes).  Not with eight waves, where
    // parts are of one or two groups and the empty stages cost more than they
    // hide: 50 reads of 1 kb 297 -> 305 us, 500 reads through loops 236 -> 238 ms
    // with it.
    constexpr bool PIPE = NW < 8;
    struct Taken {
        int n;                   // candidates (0: none)
        int4 c;                  // the ring's entry
        int32_t t, w;
        int4 lab;
    };
    Taken one, two;
    int4 vi;
    ull rw, dp;                  // record (at the key's home slot when the page is not known), that slot's key
    ull a0, a1, b0, b1;          // first window's words
    one.n = 0;
    two.n = 0;
    // the batch whose windows are here
    auto finish = [&]() {
        if (!PIPE || two.n > 0) {
            const bool act = lane < two.n;
            const int32_t v = two.c.x, kk = two.c.y, bo = two.c.z & 0x7fffffff;
            const bool chk = two.c.z < 0;
            int d = two.c.w;
            if (PIPE && __ballot(act && d < 0)) {
                // a missing page means no record: the output is admitted and needs
                // the page, so it is created now
                const ull key = dkey(v, kk >> 5);
                const uint32_t h = dhash(key) & q.mask;
                if (act && d < 0) {
                    d = dp == key ? (int)h : dir_settle(q.dir, q.mask, key, h, dp, &S.dirn);
                    if (d >= 0 && d != (int)h) rw = q.pages[d].R[kk & 31];
                    else if (dp != key) rw = 0;      // not there when the record was read: never seen
                }
            }
            const int32_t Lv = two.lab.z;
            const int64_t sb = lab_base(two.lab);
            const int32_t i = kk + bo;
            const int32_t m = act ? min(q.qlen - i, Lv - bo) : 0;
            const int qs = (int)((q.q0 + i) & 31) * 2, ss = (int)((sb + bo) & 31) * 2;
            const ull x = ((a0 << qs) | ((a1 >> 1) >> (63 - qs))) ^ ((b0 << ss) | ((b1 >> 1) >> (63 - ss)));
            const bool rec = chk && d >= 0 && rgen(rw) == q.gen;
            const bool ov = act && !(rec && bo <= rval(rw));
            int32_t lx = 0;
            if (ov && m > 0) {
                ++chunks;
                lx = min(x ? (int32_t)(__clzll((long long)x) >> 1) : 32, m);
            }
            lx += wave_extend(seg, q, lx == 32 && m > 32, q.q0 + i + 32, sb + bo + 32, m - 32, chunks);
            const ull om = __ballot(ov);
            const int32_t o = bo + lx, W = two.w + lx;
            int ncr = 0;
            if (ov) {
                if (d < 0) {
                    atomicOr(&S.flags, F_GROW);
                } else {
                    ncr = record_entry(q, S, v, kk, o, W, d, chk && !rec, Lv, o == Lv ? vi.y : 0, lmax);
                    const int32_t j = nout + lanes_below(om);
                    Ld.e[place0 + j] = make_int4(v, kk, o, page_word(d, o, Lv));
                    if (q.track) Ld.w[place0 + j] = W;
                    if (q.tb) Ld.t[place0 + j] = two.t;
                    if ((j & (SAMP - 1)) == 0 && j < SAMP * SH::SEGS) samp[j / SAMP] = skey(v, kk);
                    if (j == 0) S.partK[wv] = skey(v, kk);
                }
            }
            nout += __popcll(om);
            // crossing candidates of the whole wave in one allocation, skipped when
            // no lane reached a vertex end
            if (__ballot(ncr != 0)) {
                const int cp = wave_alloc(ncr, &S.ncand);
                if (ncr) put_out_edges(S, A, cu, ck, cW, ct, cp, vi, kk + Lv, W, two.t);
            }
        }
    };
    // the windows of the batch whose labels are here (a lane without bases to
    // compare reads the first words)
    auto windows = [&]() {
        if (!PIPE || two.n > 0) {
            const int32_t bo = two.c.z & 0x7fffffff, i = two.c.y + bo;
            const bool any = lane < two.n && i < q.qlen && bo < two.lab.z;
            const ull* const qp = q.rd + ((q.q0 + (any ? i : 0)) >> 5);
            const ull* const sp = seg + ((lab_base(two.lab) + (any ? bo : 0)) >> 5);
            a0 = qp[0]; a1 = qp[1];
            b0 = sp[0]; b1 = sp[1];
        }
    };
    // its out-edges and records
    auto records = [&]() {
        if (!PIPE || two.n > 0) {
            vi = vinfo[two.c.x];
            if (PIPE) {
                const uint32_t h = dhash(dkey(two.c.x, two.c.y >> 5)) & q.mask;
                dp = 0;
                if (lane < two.n && two.c.w < 0) dp = __hip_atomic_load(&q.dir[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                rw = q.pages[two.c.w < 0 ? (int)h : two.c.w].R[two.c.y & 31];
            } else {
                if (lane < two.n && two.c.w < 0) two.c.w = dir_insert(q.dir, q.mask, dkey(two.c.x, two.c.y >> 5), &S.dirn);
                rw = q.pages[max(two.c.w, 0)].R[two.c.y & 31];
            }
        }
    };
    // the next candidates of the ring
    auto take = [&]() {
        one.n = min(fill, 64);
        if (!PIPE || one.n > 0) {
            const bool act = lane < one.n;
            const int ri = (head + (act ? lane : 0)) & (SH::Ring::N - 1);
            one.c = R.e[ri];
            one.t = q.tb ? R.t[ri] : -1;
            one.w = q.track ? R.w[ri] : 0;
            one.lab = vlab[one.c.x];
            head = (head + one.n) & (SH::Ring::N - 1);
            fill -= one.n;
        }
    };

    Ent cur, nxt, nn;
    int32_t pv1 = -1, pk1 = 0, pv2 = -1, pk2 = 0;   // the two entries before the group
    if (lo < hi) {
        fetch(lo, cur);
        fetch(lo + 64, nxt);
        if (lo > 0) {
            Ent b;
            fetch(lo - 64, b, 62);
            pv1 = rdl(b.e.x, 63); pk1 = rdl(b.e.y, 63);
            pv2 = rdl(b.e.x, 62); pk2 = rdl(b.e.y, 62);
        }
    }
    for (int32_t g = lo; g < hi; g += 64) {
        fetch(g + 128, nn);
        // all 64 sources at once, or 16 at a time when the ring has no room for
        // so many candidates (made again then: they are not kept over the batches)
        for (int sub = 0, width = 64; sub < 64;) {
        asm volatile("" : "+v"(cur.e.y));
        const int32_t v = cur.e.x, k = cur.e.y, o0 = cur.e.z, ds0 = page_of(cur.e.w);
        const int32_t vm1 = lane_below(v, pv1), km1 = lane_below(k, pk1);
        const int32_t vm2 = lane_below(vm1, pv2), km2 = lane_below(km1, pk2);
        const int32_t vp1 = lane_above(v, rdl(nxt.e.x, 0)), kp1 = lane_above(k, rdl(nxt.e.y, 0));
        const int32_t op1 = lane_above(o0, rdl(nxt.e.z, 0)), dw1 = lane_above(cur.e.w, rdl(nxt.e.w, 0));
        const int32_t dw2 = lane_above(dw1, rdl(nxt.e.w, 1));
        const int32_t vp2 = lane_above(vp1, rdl(nxt.e.x, 1)), kp2 = lane_above(kp1, rdl(nxt.e.y, 1));
        const int32_t op2 = lane_above(op1, rdl(nxt.e.z, 1));
        const int32_t W0 = cur.w, t0 = cur.t;
        const int32_t wp1 = q.track ? lane_above(W0, rdl(nxt.w, 0)) : 0;
        const int32_t wp2 = q.track ? lane_above(wp1, rdl(nxt.w, 1)) : 0;
        const int32_t tp1 = q.tb ? lane_above(t0, rdl(nxt.t, 0)) : -1;
        const int32_t tp2 = q.tb ? lane_above(tp1, rdl(nxt.t, 1)) : -1;
        const bool valid = g + lane < hi && (unsigned)(lane - sub) < (unsigned)width;
        const int32_t i0 = k + o0;
        // k-2, k-1 (k+1, k+2) of the same vertex are adjacent in the sorted list
        const bool pm1 = vm1 == v && km1 == k - 1;
        const bool pm2 = pm1 ? (vm2 == v && km2 == k - 2) : (vm1 == v && km1 == k - 2);
        const bool pp1 = vp1 == v && kp1 == k + 1;
        const bool pp2 = pp1 ? (vp2 == v && kp2 == k + 2) : (vp1 == v && kp1 == k + 2);
        const int32_t o2 = pp1 ? op2 : op1, W2 = pp1 ? wp2 : wp1, t2 = pp1 ? tp2 : tp1;
        // before the vertex end (o < |v|)
        const bool in0 = cur.e.w >= 0, in1 = dw1 >= 0, in2 = (pp1 ? dw2 : dw1) >= 0;
        const int32_t dp1 = page_of(dw1);
        const int sl = k & 31;
        // output k-1 (this source owns it when k-1 and k-2 are absent): deletion
        const bool h0 = valid && !pm1 && !pm2 && in0;
        // output k (owned when k-1 is absent): mismatch, deletion from k+1
        int32_t b1 = -1, w1 = -1, t1 = -1;
        if (i0 < q.qlen && in0) { b1 = o0 + 1; w1 = W0 + 1; t1 = t0; }
        if (pp1 && in1 && (op1 + 1 > b1 || (op1 + 1 == b1 && wp1 + 1 > w1))) { b1 = op1 + 1; w1 = wp1 + 1; t1 = tp1; }
        const bool h1 = valid && !pm1 && b1 > o0;
        // output k+1 (always owned): insertion, mismatch at k+1, deletion from k+2
        int32_t b2 = -1, w2 = -1, t2o = -1;
        if (i0 < q.qlen) { b2 = o0; w2 = W0; t2o = t0; }
        if (pp1 && k + 1 + op1 < q.qlen && in1 && (op1 + 1 > b2 || (op1 + 1 == b2 && wp1 + 1 > w2))) {
            b2 = op1 + 1; w2 = wp1 + 1; t2o = tp1;
        }
        if (pp2 && in2 && (o2 + 1 > b2 || (o2 + 1 == b2 && W2 + 1 > w2))) { b2 = o2 + 1; w2 = W2 + 1; t2o = t2; }
        const bool h2 = valid && b2 > (pp1 ? op1 : -1);
        const int4 c0 = make_int4(v, k - 1, (o0 + 1) | (int32_t)0x80000000, sl > 0 ? ds0 : -1);
        const int4 c1 = make_int4(v, k, b1, ds0);
        const int4 c2 = make_int4(v, k + 1, pp1 ? b2 : (b2 | (int32_t)0x80000000), pp1 ? dp1 : (sl < 31 ? ds0 : -1));
        // into the ring, in list order; whenever 64 are there they are extended
        const ull m0 = __ballot(h0), m1 = __ballot(h1), m2 = __ballot(h2);
        const int total = __popcll(m0) + __popcll(m1) + __popcll(m2);
        if (fill + total > SH::Ring::N) { width = 16; continue; }   // at most 48 of 16 lanes
        int x = head + fill + lanes_below(m0) + lanes_below(m1) + lanes_below(m2);
        auto put = [&](bool h, const int4& c, int32_t w, int32_t t) {
            if (h) {
                const int r = x & (SH::Ring::N - 1);
                R.e[r] = c;
                if (q.tb) R.t[r] = t;
                if (q.track) R.w[r] = w;
            }
            x += h ? 1 : 0;
        };
        put(h0, c0, W0 + 1, t0);
        put(h1, c1, w1, t1);
        put(h2, c2, w2, t2o);
        fill += total;
        sub += width;
        if (sub >= 64) {
            pv1 = rdl(v, 63); pk1 = rdl(k, 63);
            pv2 = rdl(v, 62); pk2 = rdl(k, 62);
        }
        const bool flush = sub >= 64 && g + 64 >= hi;
        wave_lds_order();
        while (fill >= 64 || (flush && (fill > 0 || (PIPE && (one.n > 0 || two.n > 0))))) {
            if (PIPE) { finish(); two = one; windows(); records(); take(); }
            else      { take(); two = one; records(); windows(); finish(); }
        }
        wave_lds_order();
        }
        cur = nxt;
        nxt = nn;
    }
    if (lane == 0) {
        S.newN[wv] = nout;
        if (nout) atomicAdd(&S.adm, (ull)nout);
    }
}

// MODE 0: exact; 1: walk lengths tracked (Algorithm 4); 2: trace dump (and
// the learned keep/drop); 3: learned keep/drop without the dump.  Each mode
// is its own instantiation so that the registers of what it does not use
// are not allocated.
template <int BLOCK, int MODE>
__device__ void align_read(char* __restrict__ arena, int r, Shared<BLOCK, MODE>& S) {
    using SH = Shared<BLOCK, MODE>;
    constexpr bool LEARN = MODE >= 2;
    constexpr bool DUMP = MODE == 2;
    constexpr bool NARROW = !DUMP;
    const int tid = threadIdx.x;
    const int64_t t_begin = (int64_t)wall_clock64();
    // Every query here passed the screen pass (k_screen): its start vertex,
    // start window and end vertex are in range.
    Q q = make_q<MODE>(fresh_args(), arena, r);
    int cap_log2 = 8;
    {
        const KArgs& A = fresh_args();
        const int64_t want = ((int64_t)q.qlen / 32 + 1) * A.dir_factor;
        while (cap_log2 < A.dir_log2_max && ((int64_t)1 << cap_log2) < want) ++cap_log2;
    }
    int status = -1;
    int32_t s = 0;
    int32_t clip = 0;         // query bases left unaligned (free end gap)
    int cur = 1;
    int32_t n_cur = 0;
    int32_t vmx = 0;          // crossing entries of the source list merged virtually
    constexpr int NW = SH::NW;
    // merged positions of crossing entries: a bitmap over the list in the keys'
    // storage (64 positions per key slot) and the bits below each word
    uint32_t* const vm_bits = reinterpret_cast<uint32_t*>(S.skeys);
    int32_t* const vm_pre = S.xcnt;
    int64_t work = 0;
    uint32_t chunks = 0;
    for (;;) {   // attempts with a growing directory
        const uint32_t mask = (1u << cap_log2) - 1;
        const int32_t half = (int32_t)((mask + 1) >> 1);
        const KArgs& A0 = fresh_args();
        const int32_t dir_log2_max = A0.dir_log2_max;
        bind_q(q, A0, arena);
        q.mask = mask;
        for (uint32_t i = tid; i <= mask; i += BLOCK) {
            q.dir[i] = 0;
            if (q.tb) q.mkey[i] = 0;
        }
        if (tid == 0) {
            uint32_t* hdr = reinterpret_cast<uint32_t*>(arena + A0.o_hdr);
            const uint32_t g = hdr[0] + 1;
            hdr[0] = g;
            S.gen = g;
            S.n_out = 0; S.ncand = 0; S.dirn = 0; S.mn = 0; S.flags = 0;
            S.chunks = 0; S.cross = 0; S.adm = 0; S.mlp = 0; S.dropped = 0;
            S.found = 0; S.iend = -1; S.endkey = ~0ull; S.amax = 0; S.imax = 0;
            S.tick[0] = S.tick[1] = S.tick[2] = S.tick[3] = 0;
        }
        __syncthreads();
        q.gen = __builtin_amdgcn_readfirstlane(S.gen);
        // score 0 starts from the start cells (0, vs, j), j0 <= j <= j1: diagonal
        // -j at offset j, sorted by k (t = 0 is j1).  A start's trace record is
        // (vs, -1 - j), so the traced walk tells where it started.
        {
            const int32_t nst = q.j1 - q.j0 + 1;
            const Lists L0 = list_of(A0, arena, 0);
            const int64_t sb0 = A0.seg_off[q.vs];
            const int32_t lv0 = (int32_t)(A0.seg_off[q.vs + 1] - sb0);
            for (int32_t t = tid; t < min(nst, (int32_t)A0.list_cap); t += BLOCK) {
                const int32_t j = q.j1 - t;
                const int ds = dir_insert(q.dir, mask, dkey(q.vs, (-j) >> 5), &S.dirn);
                if (ds < 0) atomicOr(&S.flags, F_GROW);
                const int32_t t0 = q.tb ? trace_push(q, S, q.vs, -1 - j) : -1;
                const int32_t p = MAIN_X * A0.list_cap + t;
                L0.e[p] = make_int4(q.vs, -j, j, ds);
                L0.w[p] = 0; L0.t[p] = t0;
                L0.b[t] = sb0; L0.l[t] = lv0;
            }
            if (tid == 0) {
                S.n_out = min(nst, (int32_t)A0.list_cap);
                if (nst > A0.list_cap) atomicOr(&S.flags, F_LIST);
            }
        }
        one_part<NW>(S, 0);
        __syncthreads();
        // a start window that does not fit restarts with more working memory
        const int f0 = __builtin_amdgcn_readfirstlane(S.flags | ((S.dirn > half || S.mn > half) ? F_GROW : 0));
        const int32_t n_start = __builtin_amdgcn_readfirstlane(S.n_out);
        __syncthreads();
        cur = 1;
        n_cur = 0;
        vmx = 0;
        s = 0;
        work = 0;
        status = -1;
        int rflags = f0;
        chunks = 0;
        for (;; ++s) {
            if (f0) break;
            // ========== narrow wavefronts: wave 0 alone, on LDS lists ==========
            bool outgrown = false;    // the narrow path left this score to the crossing rounds below
            if (NARROW && (s > 0 ? n_cur : n_start) <= NARROW_IN) {
                if (tid == 0) {
                    S.nr_s = s; S.nr_n = s > 0 ? n_cur : n_start; S.nr_vmx = vmx; S.nr_list = s > 0 ? cur : 0;
                    S.nr_r = r; S.nr_mask = mask; S.nr_arena = (int64_t)(uintptr_t)arena;
                }
                __syncthreads();      // the list is complete before wave 0 reads it
                if (tid < 64) narrow_scores<BLOCK, MODE>((int64_t)(uintptr_t)kernarg());
                __syncthreads();
                const int nr = __builtin_amdgcn_readfirstlane(S.nr_code);
                const int32_t val = __builtin_amdgcn_readfirstlane(S.nr_n);
                s = __builtin_amdgcn_readfirstlane(S.nr_s);
                work += uniform64(S.nr_work);
                vmx = 0;
                if (nr == NR_FLAGS) { rflags = val; break; }
                if (nr == NR_END) {
                    status = val;
                    if (val == GWFA_ST_OK && q.ilo < q.qlen) clip = q.qlen - __builtin_amdgcn_readfirstlane(S.iend);
                    break;
                }
                outgrown = true;
                cur = 1;              // list 0 is under construction
                n_cur = val;
            }
            const KArgs& A = fresh_args();
            bind_q(q, A, arena);
            // read here for the loops below: the compiler does not move a load from
            // these arguments out of a branch
            const int4* __restrict__ vinfo = A.vinfo;
            const int4* __restrict__ vlab = A.vlab;
            const int32_t list_cap = A.list_cap;
            const int32_t xb = MAIN_X * list_cap;   // place of a list's crossing entry 0
            auto LL = [&](int j) -> Lists { return list_of(A, arena, j); };
            int32_t* const cu = reinterpret_cast<int32_t*>(arena + A.o_cand);
            const int64_t cc = A.cand_cap;
            int32_t *const ck = cu + cc, *const cW = cu + 2 * cc, *const ct = cu + 3 * cc;
            const int nb = 1 - cur;
            const Lists Ld = LL(nb);
            int32_t n1 = 0;           // diagonals produced by the expansion
            int2 lmax = make_int2(0, 0);   // this lane's largest a = i + W~ and i of the score (tracked modes)
            ull tk = wall_clock64();
            if (outgrown) {
                n1 = __builtin_amdgcn_readfirstlane(S.nr_n1);
            } else if (s > 0) {
                if (tid == 0) { S.found = 0; S.iend = -1; S.endkey = ~0ull; S.amax = 0; S.imax = 0; }
                __syncthreads();
                expand_part<BLOCK, MODE>(A, q, S, LL(cur), Ld, n_cur, vmx, cu, ck, cW, ct, chunks, lmax);
                __syncthreads();
                // the new list's parts
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const int32_t c = S.newN[w];
                    if (tid == w) {
                        S.partL[w] = n1;
                        S.partP[w] = MAIN_X * (int32_t)(((int64_t)n_cur * w / NW) & ~63);
                        S.partN[w] = c;
                    }
                    n1 += c;
                }
                n1 = __builtin_amdgcn_readfirstlane(n1);
                if (n1 > list_cap && tid == 0) atomicOr(&S.flags, F_LIST);
                n1 = min(n1, list_cap);   // not set in that branch: it has to stay a scalar
                if (tid == 0) S.n_out = n1;
            }
            if (tid == 0) { const ull t2 = wall_clock64(); S.tick[0] += t2 - tk; tk = t2; }
            // ========== crossings (Algorithm 2, same score, cost 0), in rounds ==========
            int32_t xlo = n1, xhi = (s == 0) ? n_start : n1;
            if (outgrown) xlo = xhi = n_cur;   // extended already; their candidates are next
            const int32_t preset_hi = (s == 0) ? n_start : 0;   // the start entries have their W and t
            const int32_t unkeyed = xhi - n1;                   // crossing entries made before these rounds
            bool restart = false;
            for (int round = outgrown ? __builtin_amdgcn_readfirstlane(S.nr_round) : 0;; ++round) {
                // (1) extend the diagonals created by the previous round
                for (int32_t base = xlo; base < xhi; base += BLOCK) {
                    const int32_t idx = base + tid;
                    int ncr = 0;
                    int32_t k2 = 0, W = 0, t = 0;
                    int4 vi = make_int4(0, 0, -1, -1);
                    if (idx < xhi) {
                        // the entry carries its vertex's label (set when it was claimed),
                        // so the extension's first loads go out with the out-edge range
                        int32_t v, k, d, o, Lv;
                        int64_t sb;
                        if (round > 0 && idx - xlo < SH::XC) {   // claimed by the previous round, at offset 0
                            const int32_t j = idx - xlo;
                            v = S.xsv[j]; k = S.xsk[j]; d = S.xsd[j]; o = 0; Lv = S.xsl[j]; sb = S.xsb[j];
                            t = q.tb ? S.xst[j] : -1;
                        } else {
                            const int4 e = Ld.e[xb + idx - n1];
                            v = e.x; k = e.y; d = e.w; o = e.z;
                            sb = Ld.b[idx - n1];
                            Lv = Ld.l[idx - n1];
                            W = (q.track || idx < preset_hi) ? Ld.w[xb + idx - n1] : 0;
                            t = (q.tb || idx < preset_hi) ? Ld.t[xb + idx - n1] : -1;
                        }
                        if (idx >= preset_hi && q.track) W = rval(q.pages[d].Wc[k & 31]);
                        vi = vinfo[v];
                        // Algorithm 5's push: its map slot is read with the extension's
                        // loads, the push itself follows the extension
                        const bool push = q.tb && idx >= preset_hi;
                        const ull tprobe = __hip_atomic_load(&q.mkey[push ? (dhash(dkey(v, t)) & q.mask) : 0],
                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ncr = extend_entry(A, q, S, v, k, o, W, d, true, sb, Lv, vi.y, chunks, lmax);
                        if (idx >= preset_hi) t = push ? trace_push_from(q, S, v, t, tprobe) : -1;
                        *reinterpret_cast<int2*>(&Ld.e[xb + idx - n1].z) = make_int2(o, page_word(d, o, Lv));
                        if (q.track) Ld.w[xb + idx - n1] = W;
                        if (q.tb) Ld.t[xb + idx - n1] = t;
                        k2 = k + Lv;
                    }
                    if (__ballot(ncr != 0)) {
                        const int cp = wave_alloc(ncr, &S.ncand);
                        if (ncr) put_out_edges(S, A, cu, ck, cW, ct, cp, vi, k2, W, t);
                    }
                }
                __syncthreads();
                const int32_t nc = __builtin_amdgcn_readfirstlane(S.ncand);
                const int f1 = __builtin_amdgcn_readfirstlane(S.flags | ((S.dirn > half || S.mn > half) ? F_GROW : 0));
                __syncthreads();
                if (tid == 0) S.ncand = 0;
                if (f1) { rflags = f1; restart = true; break; }
                if (nc == 0) break;
                // (2) claim never-seen diagonals (no record of this query); every
                // predecessor of this round folds its W into the slot with a max
                const ull mine = mkR(q.gen, CLAIM_BASE + round);
                for (int32_t base = 0; base < nc; base += BLOCK) {
                    const int32_t c = base + tid;
                    int claim = 0;
                    int ds = -1;
                    int64_t csb = 0;
                    int32_t cLv = 0;
                    int32_t u = 0, kc = 0, wc = 0, tc = -1;
                    if (c < nc) {
                        if (c < SH::CS) {
                            u = S.csu[c]; kc = S.csk[c]; tc = S.cst[c];
                        } else {
                            u = cu[c]; kc = ck[c]; wc = cW[c]; tc = ct[c];
                        }
                        // the target's label (stored with the entry when it is claimed),
                        // the directory slot and the record word in the page of that
                        // slot, read together: the page is almost always at its key's
                        // home slot (found there, or inserted there), and only when it
                        // is not is the record read again from the slot found.  The
                        // early read sees what a later one would: in this phase the
                        // word changes only by the claims' compare-and-swaps, which
                        // compare against the value read.
                        const ull key = dkey(u, kc >> 5);
                        const uint32_t h = dhash(key) & mask;
                        const ull probe = __hip_atomic_load(&q.dir[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const int4 lab = vlab[u];
                        const ull wh = __hip_atomic_load(&q.pages[h].R[kc & 31], __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                        csb = lab_base(lab);
                        cLv = lab.z;
                        ds = dir_settle(q.dir, mask, key, h, probe, &S.dirn);
                        if (ds < 0) {
                            atomicOr(&S.flags, F_GROW);
                        } else {
                            ull* rp = &q.pages[ds].R[kc & 31];
                            const ull w = (ds == (int)h) ? wh
                                                         : __hip_atomic_load(rp, __ATOMIC_RELAXED,
                                                                             __HIP_MEMORY_SCOPE_AGENT);
                            bool part = false;
                            if (rgen(w) != q.gen) {
                                const ull old = atomicCAS(rp, w, mine);
                                if (old == w) { claim = 1; part = true; }
                                else if (old == mine) part = true;
                            } else if (w == mine) {
                                part = true;
                            }
                            if (part && q.track) atomicMax(&q.pages[ds].Wc[kc & 31], mkR(q.gen, wc));
                        }
                    }
                    const int pos = wave_alloc(claim, &S.n_out);
                    if (claim) {
                        if (pos < list_cap) {
                            const int32_t x = pos - n1;
                            Ld.e[xb + x] = make_int4(u, kc, 0, ds);
                            if (x < SH::XS) S.skeys[x] = skey(u, kc);   // for the merge
                            Ld.l[x] = cLv; Ld.b[x] = csb;
                            if (q.track) Ld.w[xb + x] = wc;
                            if (q.tb) Ld.t[xb + x] = tc;
                            const int32_t j = pos - xhi;
                            if (j < SH::XC) {
                                S.xsv[j] = u; S.xsk[j] = kc; S.xsd[j] = ds; S.xsl[j] = cLv; S.xsb[j] = csb; S.xst[j] = tc;
                            }
                        } else {
                            atomicOr(&S.flags, F_LIST);
                        }
                    }
                }
                __syncthreads();
                const int32_t xn = __builtin_amdgcn_readfirstlane(S.n_out);
                const int f2 = __builtin_amdgcn_readfirstlane(S.flags | ((S.dirn > half) ? F_GROW : 0));
                __syncthreads();
                if (f2) { rflags = f2; restart = true; break; }
                xlo = xhi;
                xhi = xn;
                if (tid == 0) S.cross += (ull)(xhi - xlo);
            }
            if (restart) break;
            if (tid == 0) { const ull t2 = wall_clock64(); S.tick[1] += t2 - tk; tk = t2; }
            const int32_t ntot = xhi;
            work += ntot;
            if (q.track) {   // one update of the score's maxima per wave
                for (int m = 32; m >= 1; m >>= 1) {
                    lmax.x = max(lmax.x, __shfl_xor(lmax.x, m, 64));
                    lmax.y = max(lmax.y, __shfl_xor(lmax.y, m, 64));
                }
                if (__lane_id() == 0) {
                    atomicMax(&S.amax, __builtin_amdgcn_readfirstlane(lmax.x));
                    atomicMax(&S.imax, __builtin_amdgcn_readfirstlane(lmax.y));
                }
            }
            __syncthreads();
            const int found = __builtin_amdgcn_readfirstlane(S.found);
            const int32_t iend = q.ilo < q.qlen ? __builtin_amdgcn_readfirstlane(S.iend) : q.qlen;
            const int32_t amax = __builtin_amdgcn_readfirstlane(S.amax);
            const int32_t imax = __builtin_amdgcn_readfirstlane(S.imax);
            __syncthreads();
            // ========== end test (extension mode) ==========
            if (found) {
                status = GWFA_ST_OK;
                clip = q.qlen - iend;
                if (q.ilo < q.qlen) {
                    // the end cells of row iend (all of them are in this score's list)
                    const Parts<NW> parts(S);
                    for (int32_t idx = tid; idx < ntot; idx += BLOCK) {
                        const int4 e = Ld.e[idx < n1 ? parts.place(idx) : xb + idx - n1];
                        const int32_t v = e.x, o = e.z;
                        if (e.y + o == iend && ends_walk(q, v, o, vlab[v].z))
                            atomicMin(&S.endkey, ((ull)(uint32_t)v << 32) | (uint32_t)o);
                    }
                    __syncthreads();
                }
                if (q.tb) {
                    if (tid == 0) S.tend = -1;
                    __syncthreads();
                    const int32_t ev = (int32_t)(S.endkey >> 32), eo = (int32_t)(S.endkey & 0xffffffffull);
                    const Parts<NW> parts(S);
                    for (int32_t idx = tid; idx < ntot; idx += BLOCK) {
                        const int32_t p = idx < n1 ? parts.place(idx) : xb + idx - n1;
                        const int4 e = Ld.e[p];
                        if (e.x == ev && e.z == eo && e.y + eo == iend) S.tend = Ld.t[p];
                    }
                    __syncthreads();
                }
                break;
            }
            if (A.max_score >= 0 && s >= A.max_score) { status = GWFA_ST_MAX_SCORE; break; }
            // global form: an empty wavefront means the end vertex cannot be
            // reached.  Extension mode: cannot happen for valid input (the
            // query can always be inserted); a guard so that every workgroup
            // finishes.
            if (ntot == 0) { status = q.ve >= 0 ? GWFA_ST_UNREACHABLE : GWFA_ST_MAX_SCORE; break; }
            if (q.ve < 0 && s > q.qlen + 1) { status = GWFA_ST_MAX_SCORE; break; }
            // ========== merge the crossing diagonals into the sorted list ==========
            // Small sets (<= Shared::XS, in lists of up to 64 Shared::XS entries)
            // are merged virtually: their keys are ranked in LDS and each gets
            // its merged position (its rank among the crossing keys plus the
            // number of expansion outputs below it); the next pass reads the list
            // through a bitmap of those positions.  Larger sets are sorted in the
            // arena and the list is rewritten merged.
            const int32_t m = ntot - n1;
            vmx = 0;
            if (m > 0) {
                if (m > A.sort_cap) { rflags = F_LIST; break; }
                if (m <= SH::XS && ntot <= 64 * SH::XS) {
                    // rank of each crossing key among them (the keys are distinct
                    // diagonals), counted against every key read from LDS by all
                    // lanes at once: two barriers, where a sorting network would
                    // take one per stage.  Bound by its round trips: the keys are
                    // left here by the claims instead of read back, and the list's
                    // keys around each are on the way during the ranking.  10 Mb
                    // graph, 3,001 reads 409 -> 397 ms, 1 Mb DAG 118.8 -> 115.5
                    // ms, 50 reads of 1 kb 302 -> 295 us.
                    // (keys of the entries claimed here are in place already)
                    if (unkeyed > 0) {
                        for (int i = tid; i < unkeyed; i += BLOCK) {
                            const int2 a = vk_of(Ld, xb + i);
                            S.skeys[i] = skey(a.x, a.y);
                        }
                        __syncthreads();
                    }
                    for (int i = tid; i < m; i += BLOCK) {
                        const ull ki = S.skeys[i];
                        LowerBound lb;
                        lb.issue(S, Ld, ki);
                        int32_t rk = 0;
                        // sixteen keys per step, read together (one LDS round trip per
                        // step instead of one per key)
                        int j = 0;
                        for (; j + 16 <= m; j += 16) {
                            ull x[16];
#pragma unroll
                            for (int u = 0; u < 16; ++u) x[u] = S.skeys[j + u];
#pragma unroll
                            for (int u = 0; u < 16; ++u) rk += x[u] < ki ? 1 : 0;
                        }
                        for (; j < m; ++j) rk += S.skeys[j] < ki ? 1 : 0;
                        S.sidx[rk] = i;
                        S.xcnt[rk] = rk + lb.count(ki);
                    }
                    __syncthreads();
                    // the merged positions as a bitmap over the list, in the keys'
                    // storage, then the number of bits below each word, in the
                    // positions' (both no longer needed by then): the passes over
                    // this list find an entry's place from two words
                    {
                        const int32_t nw = (ntot + 63) >> 6;
                        for (int32_t w = tid; w < 2 * nw; w += BLOCK) vm_bits[w] = 0u;
                        lds_barrier();
                        for (int32_t j = tid; j < m; j += BLOCK) {
                            const int32_t pj = S.xcnt[j];
                            atomicOr(&vm_bits[pj >> 5], 1u << (pj & 31));
                        }
                        lds_barrier();
                        const int32_t kw = (nw + BLOCK - 1) / BLOCK;   // words per thread, in order
                        const int32_t w0 = min(tid * kw, nw), w1 = min(w0 + kw, nw);
                        int nbits = 0;
                        for (int32_t w = w0; w < w1; ++w) nbits += __popcll(S.skeys[w]);
                        int tot;
                        int below = block_excl_scan<BLOCK>(nbits, tot, S.scan);
                        for (int32_t w = w0; w < w1; ++w) {
                            vm_pre[w] = below;
                            below += __popcll(S.skeys[w]);
                        }
                        lds_barrier();
                    }
                    vmx = m;
                    cur = nb;
                } else {
                    int N = 1;
                    while (N < m) N <<= 1;
                    if (N > A.sort_cap) { rflags = F_LIST; break; }
                    ull* const gkeys = reinterpret_cast<ull*>(arena + A.o_sort);
                    int32_t* const gidx = reinterpret_cast<int32_t*>(gkeys + A.sort_cap);
                    for (int i = tid; i < N; i += BLOCK) {
                        ull key = ~0ull;
                        if (i < m) {
                            const int2 a = vk_of(Ld, xb + i);
                            key = skey(a.x, a.y);
                        }
                        gkeys[i] = key;
                        gidx[i] = i;
                    }
                    __syncthreads();
                    bitonic<BLOCK, false>(gkeys, gidx, N);
                    const Lists Lm = LL(cur);
                    const Parts<NW> parts(S);
                    for (int32_t j = tid; j < n1; j += BLOCK) {
                        const int32_t p = parts.place(j);
                        const int2 a = vk_of(Ld, p);
                        copy_entry(Ld, p, Lm, j + lower_bound_keys(gkeys, m, skey(a.x, a.y)), q.track, q.tb);
                    }
                    for (int32_t x = tid; x < m; x += BLOCK) {
                        const ull key = gkeys[x];
                        LowerBound lb;
                        lb.issue(S, Ld, key);
                        copy_entry(Ld, xb + gidx[x], Lm, x + lb.count(key), q.track, q.tb);
                    }
                    __syncthreads();
                    one_part<NW>(S, ntot);
                    __syncthreads();
                }
            } else {
                cur = nb;
            }
            if (tid == 0) { const ull t2 = wall_clock64(); S.tick[2] += t2 - tk; tk = t2; }
            n_cur = ntot;
            // ========== pruning (Algorithm 4) ==========
            if ((MODE == 1 || MODE == 2) && A.prune == GWFA_PRUNE_HEURISTIC && amax > A.a_diff) {
                const Lists Ls = LL(cur);
                const Lists Lp = LL(1 - cur);
                const Parts<NW> parts(S);
                int32_t outbase = 0;
                int dropped = 0;
                for (int32_t base = 0; base < n_cur; base += BLOCK) {
                    const int32_t idx = base + tid;
                    int keep = 0;
                    int32_t ph = idx;
                    if (idx < n_cur) {
                        ph = vmx ? merged_place(S.skeys, vm_pre, S.sidx, parts, xb, idx) : parts.place(idx);
                        const int4 e = Ls.e[ph];
                        const int32_t a = e.y + e.z + Ls.w[ph];
                        keep = (amax - a < A.a_diff) ? 1 : 0;
                        if (!keep) {   // the diagonal keeps its offset as its record
                            q.pages[page_of(e.w)].R[e.y & 31] = mkR(q.gen, e.z);
                            ++dropped;
                        }
                    }
                    int total;
                    const int pos = block_excl_scan<BLOCK>(keep, total, S.scan);
                    if (keep) copy_entry(Ls, ph, Lp, outbase + pos, q.track, q.tb);
                    outbase += total;
                }
                if (dropped) atomicAdd(&S.dropped, dropped);
                cur = 1 - cur;
                n_cur = outbase;
                vmx = 0;
                one_part<NW>(S, n_cur);
                __syncthreads();
                if (tid == 0) S.tick[3] += wall_clock64() - tk;
            }
            // ========== trace dump and learned keep/drop ==========
            const bool run_mlp = LEARN && A.prune == GWFA_PRUNE_LEARNED && n_cur >= A.mlp_gate && (s % A.mlp_period) == 0;
            if (LEARN && ((DUMP && A.dump) || run_mlp)) {
                const Lists Ls = LL(cur);
                const Lists Lp = LL(1 - cur);
                const Parts<NW> parts(S);
                int32_t outbase = 0;
                int dropped = 0, evals = 0;
                for (int32_t base = 0; base < n_cur; base += BLOCK) {
                    const int32_t idx = base + tid;
                    const bool live = idx < n_cur;
                    int keep = 0;
                    int32_t ph = idx;
                    int rec = 0;
                    float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    int32_t v = 0, k = 0, o = 0, dp = 0, W = 0, i = 0;
                    if (live) {
                        ph = vmx ? merged_place(S.skeys, vm_pre, S.sidx, parts, xb, idx) : parts.place(idx);
                        const int4 e = Ls.e[ph];
                        v = e.x; k = e.y; o = e.z; dp = page_of(e.w); W = Ls.w[ph];
                        i = k + o;
                        const int32_t Lv = vlab[v].z;
                        entry_features(f, s, i, W, o, Lv, vinfo[v].y, amax, imax, q.qlen);
                        rec = (DUMP && A.dump) ? 1 : 0;
                        keep = 1;
                    }
                    if (run_mlp) {
                        // the whole wave scores its 64 entries together (matrix cores)
                        const float z = mlp_logit_wave(f, S.mscale, S.mlpw);
                        if (live) {
                            ++evals;
                            keep = (z >= A.keep_threshold || i + W == amax) ? 1 : 0;   // the furthest diagonal stays
                            if (!keep) {
                                q.pages[dp].R[k & 31] = mkR(q.gen, o);   // record kept, as in Algorithm 4
                                ++dropped;
                            }
                        }
                    }
                    if (DUMP && A.dump) {
                        // one global atomic per wave
                        int tot;
                        const int ex = wave_excl_scan(rec, tot);
                        ull b0 = 0;
                        if (__lane_id() == 0 && tot > 0) b0 = atomicAdd(A.dump_count, (ull)tot);
                        b0 = __shfl(b0, 0, 64);
                        const ull slot = b0 + (ull)ex;
                        if (rec && (int64_t)slot < A.dump_cap) {
                            float* dr = A.dump + slot * 16;
#pragma unroll
                            for (int j = 0; j < 8; ++j) dr[j] = f[j];
                            int32_t* di = reinterpret_cast<int32_t*>(dr + 8);
                            di[0] = r; di[1] = s; di[2] = i; di[3] = v; di[4] = o; di[5] = W; di[6] = k;
                            di[7] = (A.tier << 8) | cap_log2;   // attempt: later attempts of a query supersede
                        }
                    }
                    if (run_mlp) {
                        int total;
                        const int pos = block_excl_scan<BLOCK>(keep, total, S.scan);
                        if (keep) copy_entry(Ls, ph, Lp, outbase + pos, q.track, q.tb);
                        outbase += total;
                    }
                }
                if (run_mlp) {
                    if (dropped) atomicAdd(&S.dropped, dropped);
                    if (evals) atomicAdd(&S.mlp, (ull)evals);
                    cur = 1 - cur;
                    n_cur = outbase;
                    vmx = 0;
                    __syncthreads();
                    one_part<NW>(S, n_cur);
                }
                __syncthreads();
            }
        }
        if (status >= 0 || !(rflags)) break;
        // capacity exceeded: grow the directory if possible, else give up
        __syncthreads();
        if ((rflags & F_GROW) && !(rflags & F_LIST) && cap_log2 < dir_log2_max) {
            cap_log2 = min(cap_log2 + 2, dir_log2_max);
            continue;
        }
        status = GWFA_ST_ARENA;
        break;
    }
    if (chunks) atomicAdd(&S.chunks, (ull)chunks);
    __syncthreads();
    // ========== results and walk (Algorithm 6) ==========
    if (tid == 0) {
        const KArgs& A = fresh_args();
        bind_q(q, A, arena);
        gwfa_result* const out = A.res + r;
        out->t_begin = t_begin;
        out->t_end = (int64_t)wall_clock64();
        out->status = status;
        out->n_scores = s + 1;
        out->work = work;
        out->path_off = -1;
        out->path_len = 0;
        out->start_off = q.j0;
        out->clip = clip;
        if (status == GWFA_ST_OK) {
            out->dist = s;
            out->end_v = (int32_t)(S.endkey >> 32);
            out->end_off = (int32_t)(S.endkey & 0xffffffffull);
            if (q.tb && S.tend >= 0) {
                // a chain visits each trace slot at most once: at most mask+1 steps
                const int32_t lim = (int32_t)q.mask + 1;
                int32_t len = 0, first = -1;
                for (int32_t t = S.tend; t >= 0 && len <= lim; t = q.Tt[t]) { ++len; first = t; }
                // the first record's predecessor field holds -1 - (start offset)
                if (first >= 0 && q.Tt[first] < 0) out->start_off = -1 - q.Tt[first];
                const ull pos = atomicAdd(A.path_cursor, (ull)len);
                out->path_len = len;
                if ((int64_t)pos + len <= A.path_cap && A.path_buf) {
                    int32_t j = len - 1;
                    for (int32_t t = S.tend; t >= 0 && j >= 0; t = q.Tt[t]) A.path_buf[pos + (j--)] = q.Tv[t];
                    out->path_off = (int64_t)pos;
                }
            }
        } else {
            out->dist = -1; out->end_v = -1; out->end_off = -1;
            if (status == GWFA_ST_ARENA && A.retry) {
                const int ri = atomicAdd(A.retry_count, 1);
                A.retry[ri] = r;
            }
        }
        // this workgroup's counters (flush_stats)
        S.acc[0] += (ull)work;
        S.acc[1] += S.cross;
        S.acc[2] += (ull)S.dirn;
        S.acc[3] += S.chunks;
        S.acc[4] += S.adm;
        S.acc[6] += S.mlp;
        S.acc[7] += (ull)S.dropped;
        S.acc[8] += (ull)(s + 1);
        for (int i = 0; i < 4; ++i) S.acc[9 + i] += S.tick[i];
    }
    __syncthreads();
}

// Waves per SIMD the compiler must allow: 4 (128 registers), for the network's
// instantiations 3 (168; one-wave workgroups 2: their LDS, with the network's
// weights, lets 8 onto a CU), 2 for the dump instantiation; a 512-lane
// workgroup of the tracked modes fills a CU alone: it takes the whole register
// file instead of spilling.
constexpr int waves_per_simd(int block, int mode) {
    return mode == 2 ? 2 : (block >= 512 ? (mode == 0 ? 4 : 1) : (mode == 3 ? (block == 64 ? 2 : 3) : 4));
}
// Query r as if it had outgrown this tier.
__device__ void leave_to_next(const KArgs& A, int r) {
    gwfa_result* const out = A.res + r;
    const int64_t t = (int64_t)wall_clock64();
    out->t_begin = t; out->t_end = t;
    out->dist = -1; out->end_v = -1; out->end_off = -1; out->status = GWFA_ST_ARENA;
    out->path_off = -1; out->path_len = 0; out->n_scores = 0; out->work = 0;
    out->start_off = A.v_off ? A.v_off[r] : 0; out->clip = 0;
    if (A.retry) A.retry[atomicAdd(A.retry_count, 1)] = r;
}

template <int BLOCK, int MODE>
__global__ __launch_bounds__(BLOCK, waves_per_simd(BLOCK, MODE)) void k_align(KArgs A) {
    constexpr bool LEARN = MODE >= 2;
    Shared<BLOCK, MODE>& S = lds<BLOCK, MODE>();
    char* arena = A.arena + (int64_t)blockIdx.x * A.arena_stride;
    if constexpr (LEARN) {
        if (A.prune == GWFA_PRUNE_LEARNED) {
            for (int i = threadIdx.x; i < MLP_N; i += BLOCK) S.mlpw[i] = A.mlp_w[i];
            if (threadIdx.x < 8) S.mscale[threadIdx.x] = A.mlp_scale[threadIdx.x];
            __syncthreads();
        }
    }
    if (threadIdx.x < 16) S.acc[threadIdx.x] = 0;
    // The work queue: query ridx of `order` (-1: turned away by the screen pass,
    // -2 - r: query r is left to the next tier).
    // Device atomics on one address take their turns (7 ns each), so a batch
    // with many queries per workgroup is dealt out by Q_SLOTS counters, every
    // Q_SLOTS-th query each; a workgroup goes on to the next counter when one
    // has run out.  Small batches use one: the last, empty, takes cost a round
    // trip each.
    const int n_q = A.n_reads;
    const int slots = n_q > 4 * (int)gridDim.x ? Q_SLOTS : 1;
    int slot = (int)blockIdx.x % slots, left = slots;
    while (left > 0) {
        if (threadIdx.x == 0) S.read = atomicAdd(&A.queue[Q_STRIDE * slot], 1);
        __syncthreads();
        const int64_t ridx = queue_place(__builtin_amdgcn_readfirstlane(S.read), slots, slot);
        __syncthreads();
        if (ridx < n_q) {
            const int r = __builtin_amdgcn_readfirstlane(A.order ? A.order[ridx] : (int)ridx);
            if (r >= 0) align_read<BLOCK, MODE>(arena, r, S);
            else if (r < -1 && threadIdx.x == 0) leave_to_next(A, -2 - r);
        } else {
            --left;
            slot = slot + 1 == slots ? 0 : slot + 1;
        }
    }
    // counters: once per workgroup, on one of STAT_SLOTS lines.  Twelve atomics
    // per query on one line bounded short queries (87 ns a query, whatever the
    // number of workgroups: 20,011 seeded reads of 200 bases 1.9 ms, 0.4 without them).
    if (threadIdx.x < 16 && A.stats && S.acc[threadIdx.x])
        atomicAdd(&A.stats[16 * (blockIdx.x % STAT_SLOTS) + threadIdx.x], S.acc[threadIdx.x]);
}

// Screen pass, before the alignment kernel, one thread per place of the work
// queue: a query whose start vertex, start window (0 <= j0 <= j1 <= |v_s|) or
// end vertex is out of range gets its result here, with status
// GWFA_ST_BAD_INPUT, and leaves -1 in its place of `valid`; the others are
// listed there, so that the alignment kernel only ever takes queries whose
// parameters index the graph in bounds.  A query r expected to need more pages
// than half the tier's directory (a run ends there) is listed as -2 - r; where
// more than 1 in 64 are, so are all: the next tier runs after this one, and a
// batch on both takes the sum of two long reads' times (900 reads of 10-120 kb
// at lag 400, 17% of them too long: 220 ms split by length, 129 on the next tier
// alone), while the few of a large batch matter less than its rest.  It also
// resets the queue and the call's counters (20,011 queries: 6 us; 60 us when one workgroup
// compacted the list, and a launch of its own for the reset).
__device__ __forceinline__ void reset_counters(int32_t* queue, ull* path_cursor, int32_t* retry_count, ull* dump_count) {
    if (threadIdx.x < Q_SLOTS) queue[Q_STRIDE * threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        if (path_cursor) *path_cursor = 0;
        if (retry_count) *retry_count = 0;
        if (dump_count) *dump_count = 0;
    }
}
__global__ __launch_bounds__(SCREEN) void k_screen(KArgs A, int32_t* valid) {
    if (blockIdx.x == 0) reset_counters(A.queue, A.path_cursor, A.retry_count, A.dump_count);
    const int32_t idx = (int32_t)blockIdx.x * SCREEN + (int32_t)threadIdx.x;
    const bool any = idx < A.n_reads;
    const int32_t r = any ? (A.order ? A.order[idx] : idx) : 0;
    bool leave = false;
    if (A.pages_per_vtx > 0.0f) {
        const float most = (float)(1 << (A.dir_log2_max - 1)) / (A.vtx_per_base * A.pages_per_vtx);   // bases
        auto big = [&](int32_t x) { return (float)(A.rd_off[x + 1] - A.rd_off[x]) > most; };
        // the batch, by up to SCREEN places spread over it (the same in every workgroup)
        const int32_t m = min(SCREEN, A.n_reads);
        bool seen = false;
        if ((int32_t)threadIdx.x < m) {
            const int32_t j = (int32_t)((int64_t)threadIdx.x * A.n_reads / m);
            seen = big(A.order ? A.order[j] : j);
        }
        const int n_big = __syncthreads_count(seen);
        leave = 64 * n_big > m || big(r);
    }
    if (!any) return;
    const int32_t vs = A.v_start[r];
    const int32_t ve = A.v_end ? A.v_end[r] : A.end_vertex;
    const int32_t j0 = A.v_off ? A.v_off[r] : 0;
    const int32_t j1 = A.v_off_hi ? A.v_off_hi[r] : j0;
    bool good = vs >= 0 && vs < A.n_vtx && ve >= -1 && ve < A.n_vtx && !(A.v_end && ve < 0) && j0 >= 0 && j1 >= j0;
    if (good) good = (int64_t)j1 <= A.seg_off[vs + 1] - A.seg_off[vs];
    if (!good) {
        gwfa_result* out = A.res + r;
        const int64_t t = (int64_t)wall_clock64();
        out->t_begin = t; out->t_end = t;
        out->dist = -1; out->end_v = -1; out->end_off = -1; out->status = GWFA_ST_BAD_INPUT;
        out->path_off = -1; out->path_len = 0; out->n_scores = 0; out->work = 0;
        out->start_off = j0; out->clip = 0;
    }
    valid[idx] = good ? (leave ? -2 - r : r) : -1;
}

// Four ASCII bases (the first in the low byte) -> 8 bits, the first base in
// the high bits; A/a 0, C/c 1, G/g 2, T/t 3 come from bits 1-2 of the code
// point ((c >> 1) ^ (c >> 2)).  *bad gets a bit for every other byte.
__device__ __forceinline__ uint32_t pack4(uint32_t x, uint32_t& bad) {
    const uint32_t u = x & 0xDFDFDFDFu;   // upper case
    // 0x80 in every zero byte of v (exact: no carry crosses a byte)
    auto zb = [](uint32_t v) { return ~(((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v | 0x7F7F7F7Fu); };
    const uint32_t ok = zb(u ^ 0x41414141u) | zb(u ^ 0x43434343u) | zb(u ^ 0x47474747u) | zb(u ^ 0x54545454u);
    bad |= ok ^ 0x80808080u;
    const uint32_t m = ((x >> 1) ^ (x >> 2)) & 0x03030303u;
    return ((m & 0xFFu) << 6) | (((m >> 8) & 0xFFu) << 4) | (((m >> 16) & 0xFFu) << 2) | (m >> 24);
}

// ASCII -> 2-bit packed words.  One thread per 16 bases (one 16-byte load,
// so a wave reads 1 KiB contiguously); lane pairs join their halves into one
// 64-bit word (the even lane holds the first 16 bases).
__global__ void k_pack(const uint8_t* __restrict__ ascii, int64_t n, ull* __restrict__ out, int64_t n_words,
                       int32_t* err) {
    const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t b0 = h * 16;
    uint32_t half = 0, bad = 0;
    if (h < 2 * n_words) {
        if (b0 + 16 <= n && ((reinterpret_cast<uintptr_t>(ascii + b0) & 15) == 0)) {
            const uint4 x = *reinterpret_cast<const uint4*>(ascii + b0);
            half = (pack4(x.x, bad) << 24) | (pack4(x.y, bad) << 16) | (pack4(x.z, bad) << 8) | pack4(x.w, bad);
        } else {
            for (int j = 0; j < 16; ++j) {
                const int64_t bi = b0 + j;
                uint32_t code = 0;
                if (bi < n) {
                    const uint32_t c = ascii[bi];
                    const uint32_t u = c & 0xdfu;
                    bad |= (u != 'A' && u != 'C' && u != 'G' && u != 'T');
                    code = ((c >> 1) ^ (c >> 2)) & 3u;
                }
                half = (half << 2) | code;
            }
        }
    }
    // every lane takes part in the exchange (blocks are whole waves, and lane
    // pairs never straddle a wave)
    const uint32_t other = __shfl_xor(half, 1, 64);
    if (h < 2 * n_words && (h & 1) == 0) out[h >> 1] = ((ull)half << 32) | other;
    if (bad && err) atomicExch(err, (int32_t)GWFA_ERR_ALPHABET);
}

// Working memory of the entry point that allocates nothing: one copy per
// device, held from the library's first use on that device to the end of the
// process.  Host code never names it directly (there it is only a stand-in
// for the device symbol): gwfa_static_scratch looks its address up.
static __device__ __align__(256) unsigned char scratch[STATIC_BYTES];

__global__ void k_zero(ull* p, int64_t n_words) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// Before a re-run: the walks' and the records' cursors go on.
__global__ void k_reset(int32_t* queue, int32_t* retry_count) { reset_counters(queue, nullptr, retry_count, nullptr); }

}  // namespace gwfa_dev

// ---------------------------------------------------------------------------
// launch helpers (called from the host code)
// ---------------------------------------------------------------------------
namespace {
template <int L>
void launch_modes(const KArgs& A, int mode, int groups, hipStream_t st) {
    if (mode == 3) { hipLaunchKernelGGL((gwfa_dev::k_align<L, 3>), dim3(groups), dim3(L), 0, st, A); return; }
    if (mode == 2) { hipLaunchKernelGGL((gwfa_dev::k_align<L, 2>), dim3(groups), dim3(L), 0, st, A); return; }
    if (mode == 1) hipLaunchKernelGGL((gwfa_dev::k_align<L, 1>), dim3(groups), dim3(L), 0, st, A);
    else hipLaunchKernelGGL((gwfa_dev::k_align<L, 0>), dim3(groups), dim3(L), 0, st, A);
}
}  // namespace

hipError_t gwfa_launch_align(const KArgs& A, int lanes, int groups, hipStream_t st) {
    // the trace dump and the learned keep/drop live in their own instantiations
    const int mode = A.dump != nullptr ? 2
                     : (A.prune == GWFA_PRUNE_LEARNED ? 3 : (A.prune != GWFA_PRUNE_NONE ? 1 : 0));
    (void)hipGetLastError();   // the launch status below must not report an older, unrelated error
    switch (lanes) {
    case 64: launch_modes<64>(A, mode, groups, st); break;
    case 128: launch_modes<128>(A, mode, groups, st); break;
    case 256: launch_modes<256>(A, mode, groups, st); break;
    case 512: launch_modes<512>(A, mode, groups, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int gwfa_align_blocks_per_cu(int lanes, int prune) {
    int nb = 0;
    hipError_t e = hipErrorInvalidValue;
    auto ask = [&](auto* exact, auto* heuristic, auto* learned) {
        const void* f = prune == GWFA_PRUNE_LEARNED ? (const void*)learned
                        : (prune != GWFA_PRUNE_NONE ? (const void*)heuristic : (const void*)exact);
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, lanes, 0);
    };
    using namespace gwfa_dev;
    switch (lanes) {
    case 64: ask(k_align<64, 0>, k_align<64, 1>, k_align<64, 3>); break;
    case 128: ask(k_align<128, 0>, k_align<128, 1>, k_align<128, 3>); break;
    case 256: ask(k_align<256, 0>, k_align<256, 1>, k_align<256, 3>); break;
    case 512: ask(k_align<512, 0>, k_align<512, 1>, k_align<512, 3>); break;
    default: break;
    }
    return (e == hipSuccess && nb > 0) ? nb : 0;
}

hipError_t gwfa_launch_pack(const uint8_t* ascii, int64_t n, unsigned long long* out, int64_t n_words, int32_t* err,
                            hipStream_t st) {
    if (n_words <= 0) return hipSuccess;
    const int tpb = 256;
    const int64_t blocks = (2 * n_words + tpb - 1) / tpb;   // one thread per 16 bases
    (void)hipGetLastError();
    hipLaunchKernelGGL(gwfa_dev::k_pack, dim3((unsigned)blocks), dim3(tpb), 0, st, ascii, n, out, n_words, err);
    return hipGetLastError();
}

void* gwfa_static_scratch(int device) {
    static std::mutex mu;
    static void* ptr[64] = {};
    std::lock_guard<std::mutex> lock(mu);
    if (device < 0 || device >= 64) return nullptr;
    if (ptr[device]) return ptr[device];
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(gwfa_dev::scratch)) != hipSuccess || !p) return nullptr;
    // generation 0 everywhere (record words of generation 0 read as "never
    // seen"); done once, before any alignment on this device uses it
    (void)hipGetLastError();
    hipLaunchKernelGGL(gwfa_dev::k_zero, dim3(2048), dim3(256), 0, nullptr, (unsigned long long*)p, STATIC_BYTES / 8);
    if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) return nullptr;
    ptr[device] = p;
    return p;
}

hipError_t gwfa_launch_screen(const KArgs& A, int32_t* valid, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(gwfa_dev::k_screen, dim3((unsigned)screen_blocks(A.n_reads)), dim3(SCREEN), 0, st, A, valid);
    return hipGetLastError();
}

hipError_t gwfa_launch_reset(int32_t* queue, int32_t* retry_count, hipStream_t st) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(gwfa_dev::k_reset, dim3(1), dim3(64), 0, st, queue, retry_count);
    return hipGetLastError();
}
