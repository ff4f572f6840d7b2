// gwfa_internal.h -- launch arguments shared by the host code and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gwfa.h"

// Counters are kept on several lines, summed when they are read.
constexpr int STAT_SLOTS = 64;
// Counters of the work queue, on lines of their own.
constexpr int Q_SLOTS = 8, Q_STRIDE = 32;
// Place in the work queue of take `taken` of counter `slot`; an empty take's
// may lie past 2^31.
__host__ __device__ constexpr int64_t queue_place(int32_t taken, int slots, int slot) {
    return (int64_t)taken * slots + slot;
}
// Workgroups of the screen pass, SCREEN places each.
constexpr int SCREEN = 256;
constexpr int64_t screen_blocks(int32_t n_reads) { return ((int64_t)n_reads + SCREEN - 1) / SCREEN; }

struct KArgs {
    // graph (device)
    const unsigned long long* seg;   // packed labels
    const int64_t* seg_off;          // n_vtx+1 base offsets
    const int32_t* out_off;          // n_vtx+1 CSR offsets
    const int32_t* out_dst;          // n_edge targets
    const int4* vinfo;               // n_vtx: first out-edge index, out-degree, first and second target (-1: none)
    const int4* vlab;                // n_vtx: label base (low, high 32 bits), label length, 0
    const int4* vsucc;               // 2 n_vtx: vlab of the first and the second target (zeros: none)
    int32_t n_vtx;
    // queries (device)
    const unsigned long long* rd;    // packed queries
    const int64_t* rd_off;           // n_reads+1 base offsets
    const int32_t* v_start;
    const int32_t* v_off;            // per-query start offsets in the start vertex, or null (all 0)
    const int32_t* v_off_hi;         // per-query end of a free start window, or null (= v_off)
    const int32_t* order;            // work-queue order (-1: no query, -2 - r: r is left to the next tier) or null
    const int32_t* v_end;            // per-query end vertices (global form) or null
    int32_t end_vertex;              // end vertex of every query (global form) or -1
    int32_t n_reads;
    // outputs (device)
    gwfa_result* res;
    int32_t* path_buf;
    int64_t path_cap;
    unsigned long long* path_cursor;
    int32_t* queue;                  // Q_SLOTS counters, Q_STRIDE apart
    unsigned long long* stats;       // STAT_SLOTS lines of 16 counters, or null
    int32_t* retry;                  // queries that overflowed (or null)
    int32_t* retry_count;
    // options
    int32_t prune, a_diff, traceback, max_score;
    float keep_threshold;
    int32_t mlp_gate, mlp_period;
    int32_t end_free;                // free end gap in the query (trailing bases)
    int32_t walk_free;               // global form: the walk may end anywhere inside the end vertex
    const uint16_t* mlp_w;           // bf16 weights (device) or null
    const float* mlp_scale;          // 8 feature scales (device) or null
    float* dump;                     // per-entry trace records (16 x 4 bytes) or null
    int64_t dump_cap;
    unsigned long long* dump_count;
    int32_t tier;                    // working-memory tier of this launch (tags dump records)
    // working memory: one arena per workgroup
    char* arena;
    int64_t arena_stride;
    int32_t dir_log2_max, dir_factor, list_cap, cand_cap, sort_cap;
    int64_t o_hdr, o_dir, o_pages, o_mkey, o_tv, o_tt, o_lists, o_cand, o_sort;
    // queries expected to need more pages than this tier has are left to the
    // next: vertices per base of the graph, pages per vertex of the walk (0: all are tried)
    float vtx_per_base, pages_per_vtx;
};

// 4-byte words of one wavefront list per entry of its capacity (gwfa_kernels.hip,
// list_of): 4 places of 24 bytes (3 for the main entries, 1 for the crossing
// entries) and the crossing entries' 12-byte labels
constexpr int64_t LIST_WORDS = 4 * 6 + 3;

hipError_t gwfa_launch_align(const KArgs& A, int lanes, int groups, hipStream_t st);
// resident workgroups per compute unit of a pruning mode's alignment kernel (0 if unknown)
int gwfa_align_blocks_per_cu(int lanes, int prune);
hipError_t gwfa_launch_pack(const uint8_t* ascii, int64_t n, unsigned long long* out, int64_t n_words,
                            int32_t* err, hipStream_t st);
// resets the queue and the retry counter before a re-run
hipError_t gwfa_launch_reset(int32_t* queue, int32_t* retry_count, hipStream_t st);
// Working memory of the entry point that allocates nothing
// (gwfa_align_batch_static_dev): a file-scope device array of STATIC_BYTES
// per device holding a header (queue, counters), the screened query list
// (at most STATIC_MAX_READS queries) and one fixed tier of per-workgroup
// arenas (record directory of 2^STATIC_DIR_LOG2 pages, wavefront lists of
// STATIC_LIST_CAP entries).
constexpr int64_t STATIC_BYTES = (int64_t)512 << 20;
constexpr int32_t STATIC_MAX_READS = 1 << 20;
constexpr int32_t STATIC_DIR_LOG2 = 14;
constexpr int32_t STATIC_LIST_CAP = 8192;
constexpr int64_t STATIC_HDR = 4096;   // retry counter, path cursor, queue (STATIC_QUEUE)
constexpr int64_t STATIC_QUEUE = 1024;
// Device address of the static array on `device` (the current device),
// looked up and cleared once per device and process; null if that fails.
void* gwfa_static_scratch(int device);

// per-query parameter check before the alignment: results of the queries
// that are out of range (GWFA_ST_BAD_INPUT) and the work queue's list, `valid`;
// resets the queue, A.path_cursor, A.retry_count and A.dump_count
hipError_t gwfa_launch_screen(const KArgs& A, int32_t* valid, hipStream_t st);

// pruning network: training and batch inference (gwfa_mlp.hip)
struct Scale8 {
    float s[8];
};
int64_t gwfa_mlp_scratch_floats();
hipError_t gwfa_launch_mlp_grad(const float* feat, int64_t stride, const Scale8& scale, const uint8_t* label,
                                int64_t n, float pos_weight, const uint16_t* w, float* scr, float* grad, float* loss,
                                hipStream_t st);
hipError_t gwfa_launch_mlp_adam(float* master, float* m1, float* m2, const float* grad, uint16_t* wb, float lr,
                                float beta1, float beta2, float eps, float bc1, float bc2, hipStream_t st);
hipError_t gwfa_launch_mlp_cast(const float* src, uint16_t* dst, int64_t n, hipStream_t st);
hipError_t gwfa_launch_mlp_logits(const float* feat, int64_t stride, const Scale8& scale, int64_t n,
                                  const uint16_t* w, float* out, hipStream_t st);

// base-level alignment along the traced walks (gwfa_cigar.hip)
struct CigArgs {
    const unsigned long long* seg;   // packed labels
    const int64_t* seg_off;
    const unsigned long long* rd;    // packed queries
    const int64_t* rd_off;
    int32_t n_reads;
    const gwfa_result* res;
    const int32_t* path_buf;
    uint32_t* cigar;
    int64_t cigar_cap;
    unsigned long long* cigar_cursor;
    int64_t* cigar_off;
    int32_t* cigar_len;
    int32_t* queue;
    char* arena;                     // one region per workgroup
    int64_t arena_stride, o_pref, o_wf, o_ops;
    int32_t max_d, max_q, max_t;     // capacities of the regions
    const int32_t* order;            // queries, the largest distances first
    int32_t lds_q, lds_t, lds_row;   // LDS words of the query and of T (64 bits), entries of a wavefront row
};
int64_t gwfa_cigar_row_words(int64_t d);
int64_t gwfa_cigar_lds_bytes(const CigArgs& A);
// lds_bytes: dynamic LDS of the variant that keeps queries there, 0 for the other
hipError_t gwfa_launch_cigar(const CigArgs& A, int groups, int lanes, int lds_bytes, hipStream_t st);
