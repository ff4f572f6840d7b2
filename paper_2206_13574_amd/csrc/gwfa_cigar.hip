// gwfa_cigar.hip -- base-level alignment of each query against the walk the
// graph alignment traced (the last step the paper leaves to a pairwise
// aligner, noting that it is cheap).
//
// One persistent workgroup per query, the largest distances first: the walk's
// string T (the labels of the walk, the first one from start_off, the last one
// cut at end_off) is spelled into a 2-bit packed buffer, then a pairwise
// wavefront alignment (the score-ordered diagonal recurrence of Eq. 2 on a
// single path: mismatch, insertion, deletion, then extension by the
// exact-match run) finds an optimal global alignment of q and T, and a
// traceback turns the stored wavefronts into CIGAR operations.
//
// The cost is at most the query's graph distance D, so wavefront s only needs
// the diagonals k = j - i (i query bases, j bases of T consumed) that can be
// reached with s edits and can still reach the end's diagonal with D - s:
// -s <= k <= s and |k - kend| <= D - s.  That is half of the full triangle,
// and every diagonal kept has its three sources kept.  Row s is stored at
// row_at(s) of the workgroup's buffer.
//
// Where the packed query, T and two wavefronts fit LDS (k_cigar<.., true>) a
// score is one pass over LDS and one barrier; each cell's start and source go
// to memory for the traceback, which reads 8 scores per memory round trip.
// Longer queries keep them in memory.  Operation words are
// (length << 4) | op with op 7 ('=', match), 8 ('X', mismatch), 1 ('I', query
// base absent from the walk), 2 ('D', walk base absent from the query), 4
// ('S', query bases left unaligned by a free end gap in the query), as in
// SAM/BAM.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gwfa_internal.h"

namespace gwfa_cig {

typedef unsigned long long ull;
constexpr int32_t NEG = -(1 << 30);
constexpr uint32_t OP_EQ = 7, OP_X = 8, OP_I = 1, OP_D = 2, OP_S = 4;

__device__ __forceinline__ ull win32(const ull* __restrict__ w, int64_t p) {
    const int64_t wi = p >> 5;
    const int sh = (int)(p & 31) * 2;
    return (w[wi] << sh) | ((w[wi + 1] >> 1) >> (63 - sh));
}

// exact-match run of q[qp ...] and t[tp ...], at most lim bases, 32 at a time
__device__ int32_t run_len(const ull* __restrict__ q, int64_t qp, const ull* __restrict__ t, int64_t tp, int32_t lim) {
    int32_t l = 0;
    while (l < lim) {
        const ull x = win32(q, qp + l) ^ win32(t, tp + l);
        const int32_t m = x ? (int32_t)(__clzll((long long)x) >> 1) : 32;
        if (l + m >= lim) return lim;
        l += m;
        if (x) return l;
    }
    return l;
}

// The diagonals of wavefront s that are kept, and where its row is stored:
// at most 2 min(s, D - s) + 1 of them, rows packed by that bound.
struct Band {
    int32_t D, kend;
    __device__ __forceinline__ int32_t lo(int32_t s) const { return max(-s, kend - (D - s)); }
    __device__ __forceinline__ int32_t hi(int32_t s) const { return min(s, kend + (D - s)); }
    __device__ __forceinline__ int64_t row_at(int32_t s) const {
        const int64_t h = D / 2, a = s, b = D - (int64_t)s + 1;
        return a <= h ? a * a : (h + 1) * (h + 1) + (D - h) * (D - h) - b * b;
    }
};

// the three sources of diagonal k at the next score (Eq. 2 on one path), from
// row Wp of the diagonals lo..hi; NEG if absent
__device__ __forceinline__ void sources(const int32_t* Wp, int32_t lo, int32_t hi, int32_t k, int32_t qlen,
                                        int32_t tlen, int32_t& mis, int32_t& ins, int32_t& del) {
    mis = ins = del = NEG;
    if (k >= lo && k <= hi) {                     // mismatch: (i, j) -> (i+1, j+1)
        const int32_t i0 = Wp[k - lo];
        if (i0 >= 0 && i0 < qlen && i0 + k < tlen) mis = i0 + 1;
    }
    if (k + 1 >= lo && k + 1 <= hi) {             // query base alone: (i, j) -> (i+1, j), from k+1
        const int32_t i1 = Wp[k + 1 - lo];
        if (i1 >= 0 && i1 < qlen) ins = i1 + 1;
    }
    if (k - 1 >= lo && k - 1 <= hi) {             // walk base alone: (i, j) -> (i, j+1), from k-1
        const int32_t i2 = Wp[k - 1 - lo];
        if (i2 >= 0 && i2 + k - 1 < tlen) del = i2;
    }
}

// The operations of one query, from the end: run-length merged in registers,
// each finished one stored by lane 0.
struct Ops {
    uint32_t* out;
    int32_t n = 0;           // stored
    uint32_t op = 0;
    int32_t len = 0;         // the run being built
    __device__ __forceinline__ void emit(uint32_t o, int32_t l) {
        if (l <= 0) return;
        if (o != op) flush();
        op = o;
        len += l;
    }
    __device__ __forceinline__ void flush() {
        if (len > 0) {
            if (threadIdx.x == 0) out[n] = ((uint32_t)len << 4) | op;
            ++n;
            len = 0;
        }
    }
};

struct Shared {
    int32_t read;
    int32_t done[2];         // by parity of the score, so that one barrier a score is enough
    int32_t n_ops;
    int64_t pos;
    int32_t scan[16];
    int64_t carry;
};

// The query's result as scalars: every field is read by one lane and
// broadcast, so that every branch on it is a branch of the whole workgroup.
struct UniRes {
    int32_t dist, end_off, status, path_len, start_off, clip;
    int64_t path_off;
};
__device__ __forceinline__ int64_t uni64(int64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ UniRes load_res(const gwfa_result* p) {
    UniRes u;
    u.dist = __builtin_amdgcn_readfirstlane(p->dist);
    u.end_off = __builtin_amdgcn_readfirstlane(p->end_off);
    u.status = __builtin_amdgcn_readfirstlane(p->status);
    u.path_len = __builtin_amdgcn_readfirstlane(p->path_len);
    u.start_off = __builtin_amdgcn_readfirstlane(p->start_off);
    u.clip = __builtin_amdgcn_readfirstlane(p->clip);
    u.path_off = uni64(p->path_off);
    return u;
}

// Barrier for phases that exchange only LDS data (stores to memory stay in
// flight).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Persistent loop over the queries.  No query leaves the loop body early
// (no continue, no return): a per-query exit in front of the queue fetch
// (thread 0's atomic, then a barrier) lets the compiler send the other lanes
// straight back to that barrier while thread 0 waits outside the loop, and
// the workgroup never fetches again.  Every branch that decides the loop's
// course is on values the whole workgroup shares (scalar registers).
//
// 4,001 reads of 8 kb (1-8% errors): 4.4 ms, bound by the scores of its hardest
// query (LDS latency and a barrier each); 28.7 ms before, with the full
// triangle, rows, query and T in memory, two barriers a score and one thread
// tracing back with read-modify-writes of its operations.
template <int BLOCK, bool LDS>
__global__ __launch_bounds__(BLOCK) void k_cigar(CigArgs A) {
    __shared__ Shared S;
    extern __shared__ ull dyn[];
    char* arena = A.arena + (int64_t)blockIdx.x * A.arena_stride;
    ull* const Tg = reinterpret_cast<ull*>(arena);
    int64_t* P = reinterpret_cast<int64_t*>(arena + A.o_pref);
    int32_t* W = reinterpret_cast<int32_t*>(arena + A.o_wf);
    uint32_t* ops = reinterpret_cast<uint32_t*>(arena + A.o_ops);
    // LDS: query, T, two rows
    ull* const Ql = dyn;
    ull* const Tl = Ql + A.lds_q;
    int32_t* const rows = reinterpret_cast<int32_t*>(Tl + A.lds_t);
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) S.read = atomicAdd(A.queue, 1);
        __syncthreads();
        const int ri = __builtin_amdgcn_readfirstlane(S.read);
        __syncthreads();
        if (ri >= A.n_reads) break;
        const int r = __builtin_amdgcn_readfirstlane(A.order[ri]);
        const UniRes res = load_res(A.res + r);
        const int64_t q0 = uni64(A.rd_off[r]);
        const int32_t qfull = __builtin_amdgcn_readfirstlane((int32_t)(A.rd_off[r + 1] - q0));
        // the graph alignment covers q[0, qfull - clip); the rest is soft-clipped
        const int32_t qlen = qfull - res.clip;
        const bool usable = res.status == GWFA_ST_OK && res.path_off >= 0 && res.path_len > 0 && res.dist >= 0 &&
                            res.dist <= A.max_d && qfull <= A.max_q && res.start_off >= 0 && res.clip >= 0 &&
                            qlen >= 0;
        if (!usable) {
            if (tid == 0) { A.cigar_off[r] = -1; A.cigar_len[r] = -1; }
        } else {
            const int32_t* walk = A.path_buf + res.path_off;
            const int32_t L = res.path_len;
            const int32_t j0 = res.start_off;
            // ---- prefix offsets of the walk's vertices in T (block scan in chunks)
            if (tid == 0) S.carry = 0;
            __syncthreads();
            for (int32_t b = 0; b < L; b += BLOCK) {
                const int32_t j = b + tid;
                int64_t len = 0;
                if (j < L) {
                    const int32_t v = walk[j];
                    len = (j == L - 1) ? (int64_t)res.end_off : (A.seg_off[v + 1] - A.seg_off[v]);
                    if (j == 0) len = max(len - j0, (int64_t)0);   // the first vertex starts at j0
                }
                // inclusive scan over the block (the lengths fit in 32 bits per vertex)
                int32_t x = (int32_t)len;
                for (int d = 1; d < 64; d <<= 1) {
                    const int32_t y = __shfl_up(x, d, 64);
                    if (__lane_id() >= d) x += y;
                }
                if (__lane_id() == 63) S.scan[tid >> 6] = x;
                __syncthreads();
                int64_t before = S.carry;
                for (int w = 0; w < (tid >> 6); ++w) before += S.scan[w];
                if (j < L) P[j + 1] = before + x;
                if (j == 0) P[0] = 0;
                __syncthreads();
                if (tid == 0) {
                    int64_t tot = 0;
                    for (int w = 0; w < BLOCK / 64; ++w) tot += S.scan[w];
                    S.carry += tot;
                }
                __syncthreads();
            }
            const int64_t tlen64 = uni64(S.carry);
            if (tlen64 > (int64_t)A.max_t) {
                if (tid == 0) { A.cigar_off[r] = -1; A.cigar_len[r] = -3; }
            } else {
                const int32_t tlen = (int32_t)tlen64;
                const ull* const qw = LDS ? Ql : A.rd;
                const int64_t qb = LDS ? (q0 & 31) : q0;   // the query's first base in qw
                ull* const T = LDS ? Tl : Tg;
                if (LDS) {
                    const int32_t w0 = (int32_t)((qb + qlen) >> 5) + 2;
                    for (int32_t w = tid; w < w0; w += BLOCK) Ql[w] = A.rd[(q0 >> 5) + w];
                }
                // ---- spell T, 2-bit packed, 32 bases per word, plus two zero words
                const int32_t tw = tlen / 32 + 2;
                for (int32_t w = tid; w < tw; w += BLOCK) {
                    ull word = 0;
                    int64_t p = (int64_t)w * 32;
                    if (p < tlen) {
                        int32_t lo = 0, hi = L - 1;          // last vertex j with P[j] <= p
                        while (lo < hi) {
                            const int32_t mid = (lo + hi + 1) >> 1;
                            if (P[mid] <= p) lo = mid; else hi = mid - 1;
                        }
                        int32_t j = lo;
                        for (int b = 0; b < 32 && p < tlen;) {
                            while (j + 1 < L && P[j + 1] <= p) ++j;
                            const int64_t g = A.seg_off[walk[j]] + (j == 0 ? j0 : 0) + (p - P[j]);
                            const int n = (int)min((int64_t)(32 - b), P[j + 1] - p);   // bases of this vertex
                            ull x = win32(A.seg, g);
                            if (n < 32) x &= ~(~0ull >> (2 * n));
                            word |= x >> (2 * b);
                            b += n;
                            p += n;
                        }
                    }
                    T[w] = word;
                }
                const int32_t kend = tlen - qlen;
                const Band B{res.dist, kend};
                if (tid == 0) S.done[0] = S.done[1] = -1;
                __syncthreads();
                // ---- wavefronts
                // (a cost of at most D implies |kend| <= D)
                int32_t s = 0, done = -1;
                if (kend >= -B.D && kend <= B.D) {
                    const int32_t l = run_len(qw, qb, T, 0, min(qlen, tlen));   // by every thread: one value
                    if (tid == 0) {
                        if (LDS) rows[0] = l; else W[0] = l;
                    }
                    done = __builtin_amdgcn_readfirstlane((kend == 0 && l == qlen) ? 0 : -1);
                    if (LDS) lds_barrier(); else __syncthreads();
                    while (done < 0 && s < B.D) {
                        ++s;
                        const int32_t plo = B.lo(s - 1), phi = B.hi(s - 1), lo = B.lo(s), hi = B.hi(s);
                        int32_t* const Wg = W + B.row_at(s);
                        const int32_t* const Wp = LDS ? rows + ((s - 1) & 1) * A.lds_row : W + B.row_at(s - 1);
                        int32_t* const Ws = LDS ? rows + (s & 1) * A.lds_row : Wg;
                        for (int32_t k = lo + tid; k <= hi; k += BLOCK) {
                            int32_t mis, ins, del;
                            sources(Wp, plo, phi, k, qlen, tlen, mis, ins, del);
                            const int32_t v = max(mis, max(ins, del));
                            int32_t i = v;
                            if (v >= 0) i += run_len(qw, qb + v, T, (int64_t)v + k, min(qlen - v, tlen - v - k));
                            Ws[k - lo] = v < 0 ? NEG : i;
                            // for the traceback: where the cell's run starts and its source
                            if (LDS) Wg[k - lo] = (v << 2) | (mis == v ? 0 : (ins == v ? 1 : 2));
                            if (k == kend && i == qlen) S.done[s & 1] = s;
                        }
                        if (LDS) lds_barrier(); else __syncthreads();
                        done = __builtin_amdgcn_readfirstlane(S.done[s & 1]);
                    }
                }
                __syncthreads();   // the rows are in memory
                if (done < 0) {
                    if (tid == 0) { A.cigar_off[r] = -1; A.cigar_len[r] = -3; }
                } else {
                    // ---- traceback, by wave 0: operations from the end, run-length merged
                    if (tid < 64) {
                        Ops o{ops};
                        o.emit(OP_S, qfull - qlen);
                        int32_t k = kend, i = qlen, ss = done;
                        if (LDS) {
                            // lane l holds the cell at score ss - x, x = floor(sqrt(l)), diagonal
                            // k + l - x(x+1): every cell the next eight steps can reach
                            const int x = (tid >= 1) + (tid >= 4) + (tid >= 9) + (tid >= 16) + (tid >= 25) + (tid >= 36) +
                                          (tid >= 49);
                            const int dk = tid - x * (x + 1);
                            while (ss > 0) {
                                int32_t c = 0;
                                const int32_t sx = ss - x, kx = k + dk;
                                if (sx > 0 && kx >= B.lo(sx) && kx <= B.hi(sx)) c = W[B.row_at(sx) + kx - B.lo(sx)];
                                const int32_t k0 = k;
                                const int steps = min(ss, 8);
                                for (int y = 0; y < steps; ++y) {
                                    const int32_t cell = __builtin_amdgcn_readlane(c, y * (y + 1) + k - k0);
                                    const int32_t v = cell >> 2, op = cell & 3;
                                    o.emit(OP_EQ, i - v);
                                    if (op == 0) { o.emit(OP_X, 1); i = v - 1; }
                                    else if (op == 1) { o.emit(OP_I, 1); i = v - 1; k += 1; }
                                    else { o.emit(OP_D, 1); i = v; k -= 1; }
                                }
                                ss -= steps;
                            }
                        } else {
                            for (; ss > 0; --ss) {
                                int32_t mis, ins, del;
                                sources(W + B.row_at(ss - 1), B.lo(ss - 1), B.hi(ss - 1), k, qlen, tlen, mis, ins, del);
                                const int32_t v = __builtin_amdgcn_readfirstlane(max(mis, max(ins, del)));
                                const int op = __builtin_amdgcn_readfirstlane(mis == v ? 0 : (ins == v ? 1 : 2));
                                o.emit(OP_EQ, i - v);
                                if (op == 0) { o.emit(OP_X, 1); i = v - 1; }
                                else if (op == 1) { o.emit(OP_I, 1); i = v - 1; k += 1; }
                                else { o.emit(OP_D, 1); i = v; k -= 1; }
                            }
                        }
                        o.emit(OP_EQ, i);
                        o.flush();
                        if (tid == 0) {
                            S.n_ops = o.n;
                            S.pos = (int64_t)atomicAdd(A.cigar_cursor, (ull)o.n);
                        }
                    }
                    __syncthreads();
                    // ---- reversed into the output
                    const int32_t n = __builtin_amdgcn_readfirstlane(S.n_ops);
                    const int64_t pos = uni64(S.pos);
                    const bool fits = pos + n <= A.cigar_cap;
                    if (fits)
                        for (int32_t x = tid; x < n; x += BLOCK) A.cigar[pos + x] = ops[n - 1 - x];
                    if (tid == 0) {
                        A.cigar_off[r] = fits ? pos : -1;
                        A.cigar_len[r] = fits ? n : -2;
                    }
                }
            }
        }
        __syncthreads();
    }
}

__global__ void k_cig_reset(int32_t* queue, ull* cursor) {
    if (threadIdx.x == 0 && blockIdx.x == 0) { *queue = 0; *cursor = 0; }
}

}  // namespace gwfa_cig

// words of a workgroup's wavefront rows for distances up to d (Band::row_at)
int64_t gwfa_cigar_row_words(int64_t d) {
    const int64_t h = d / 2;
    return (h + 1) * (h + 1) + (d - h) * (d - h);
}

int64_t gwfa_cigar_lds_bytes(const CigArgs& A) { return 8 * ((int64_t)A.lds_q + A.lds_t) + 2 * 4 * (int64_t)A.lds_row; }

hipError_t gwfa_launch_cigar(const CigArgs& A, int groups, int lanes, int lds_bytes, hipStream_t st) {
    using namespace gwfa_cig;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_cig_reset, dim3(1), dim3(64), 0, st, A.queue, A.cigar_cursor);
    if (lds_bytes > 0) {
        const void* f = lanes == 512 ? (const void*)k_cigar<512, true> : (const void*)k_cigar<256, true>;
        if (lds_bytes > 48 << 10) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
            if (e != hipSuccess) return e;
        }
        if (lanes == 512) hipLaunchKernelGGL((k_cigar<512, true>), dim3(groups), dim3(512), lds_bytes, st, A);
        else hipLaunchKernelGGL((k_cigar<256, true>), dim3(groups), dim3(256), lds_bytes, st, A);
    } else {
        hipLaunchKernelGGL((k_cigar<256, false>), dim3(groups), dim3(256), 0, st, A);
    }
    return hipGetLastError();
}
