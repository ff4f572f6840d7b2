// Stand-in for the HIP runtime and the kernels, so that the library's host
// code (gwfa_host.cpp, compiled by g++ with this file) runs on a machine
// without a GPU.  Device memory is counted, not used: an allocation of up to
// 64 MiB is host memory, a larger one an address nobody reads.  Launches of
// the alignment kernel are logged; each leaves as many queries to be re-run
// as the test asked for at its directory size.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <vector>

#include "gwfa.h"
#include "gwfa_internal.h"

// Host allocations of the library of at least this size fail.
static size_t new_limit = SIZE_MAX;
void* operator new(size_t n) {
    if (n >= new_limit) throw std::bad_alloc();
    return malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

namespace {
struct Block { size_t bytes; bool real; };
std::map<uintptr_t, Block> blocks;
size_t total = (size_t)288 << 30, used = 0, largest = SIZE_MAX;
uintptr_t next_addr = (uintptr_t)1 << 46;
hipError_t last = hipSuccess;
int failed = 0;
bool capturing = false;
int overflow[32];
struct Launch { KArgs A; int lanes, groups; };
std::vector<Launch> launches, captured;
int64_t cig_bytes = 0, cig_groups = 0;

bool readable(const void* p) {
    auto it = blocks.upper_bound((uintptr_t)p);
    if (it == blocks.begin()) return true;
    --it;
    return it->second.real || (uintptr_t)p >= it->first + it->second.bytes;
}
void run(const Launch& l) {
    launches.push_back(l);
    const int k = l.A.retry ? std::min(overflow[l.A.dir_log2_max], l.A.n_reads) : 0;
    *l.A.retry_count = k;
    for (int i = 0; i < k; ++i) l.A.retry[i] = i;
}
}  // namespace

extern "C" {
void fake_memory(int64_t bytes) { total = (size_t)bytes; }
void fake_largest(int64_t bytes) { largest = bytes < 0 ? SIZE_MAX : (size_t)bytes; }   // largest block to be had
void fake_new_limit(int64_t bytes) { new_limit = bytes < 0 ? SIZE_MAX : (size_t)bytes; }
int64_t fake_used() { return (int64_t)used; }
void fake_overflow(int dir_log2, int queries) { overflow[dir_log2] = queries; }
void fake_clear() { launches.clear(); last = hipSuccess; }
int fake_launches() { return (int)launches.size(); }
// directory size, lanes, groups, queries, records' tier, whether the arenas are allocated, a query's bytes
void fake_launch(int i, int64_t* out) {
    const Launch& l = launches[i];
    auto it = blocks.find((uintptr_t)l.A.arena);
    const bool live = it != blocks.end() && it->second.bytes >= (size_t)l.A.arena_stride * (size_t)l.groups;
    const int64_t v[7] = {l.A.dir_log2_max, l.lanes, l.groups, l.A.n_reads, l.A.tier, live, l.A.arena_stride};
    memcpy(out, v, sizeof v);
}
int64_t fake_screen_blocks(int32_t n) { return screen_blocks(n); }
int64_t fake_queue_place(int32_t taken, int32_t slots, int32_t slot) { return queue_place(taken, slots, slot); }
int64_t fake_cigar_groups() { return cig_groups; }
int fake_failed() { return failed; }      // allocations refused so far
int fake_last_error() { return (int)last; }

hipError_t hipMalloc(void** p, size_t n) {
    if (capturing || used + n > total || n > largest) { ++failed; return last = hipErrorOutOfMemory; }
    const bool real = n <= (size_t)64 << 20;
    *p = real ? calloc(1, n + 1) : (void*)next_addr;
    if (!real) next_addr += (n + 8191) / 4096 * 4096;
    blocks[(uintptr_t)*p] = Block{n, real};
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    auto it = blocks.find((uintptr_t)p);
    if (it == blocks.end()) return last = hipErrorInvalidValue;
    used -= it->second.bytes;
    if (it->second.real) free(p);
    blocks.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n + 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { if (readable(p)) memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    if (n && readable(d) && readable(s)) memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = total - used; *t = total; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)(uintptr_t)64; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    capturing = true;
    captured.clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    capturing = false;
    *g = (hipGraph_t)(uintptr_t)128;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *x = (hipGraphExec_t) new std::vector<Launch>(captured);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    for (const Launch& l : *(std::vector<Launch>*)x) run(l);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete (std::vector<Launch>*)x; return hipSuccess; }
}  // extern "C"

// ---- the kernels' launches
hipError_t gwfa_launch_align(const KArgs& A, int lanes, int groups, hipStream_t) {
    if (capturing) captured.push_back(Launch{A, lanes, groups});
    else run(Launch{A, lanes, groups});
    return hipSuccess;
}
int gwfa_align_blocks_per_cu(int lanes, int prune) { return std::min(16, (prune == 2 ? 512 : 1024) / lanes); }
hipError_t gwfa_launch_pack(const uint8_t*, int64_t, unsigned long long*, int64_t, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t gwfa_launch_reset(int32_t*, int32_t* retry_count, hipStream_t) {
    *retry_count = 0;
    return hipSuccess;
}
void* gwfa_static_scratch(int) { static char base[8192]; return base; }
hipError_t gwfa_launch_screen(const KArgs& A, int32_t*, hipStream_t) {
    if (!capturing) *A.retry_count = 0;
    return hipSuccess;
}
int64_t gwfa_mlp_scratch_floats() { return 1024; }
hipError_t gwfa_launch_mlp_grad(const float*, int64_t, const Scale8&, const uint8_t*, int64_t, float, const uint16_t*,
                                float*, float*, float*, hipStream_t) { return hipSuccess; }
hipError_t gwfa_launch_mlp_adam(float*, float*, float*, const float*, uint16_t*, float, float, float, float, float, float,
                                hipStream_t) { return hipSuccess; }
hipError_t gwfa_launch_mlp_cast(const float*, uint16_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t gwfa_launch_mlp_logits(const float*, int64_t, const Scale8&, int64_t, const uint16_t*, float*, hipStream_t) {
    return hipSuccess;
}
int64_t gwfa_cigar_row_words(int64_t d) { const int64_t h = d / 2; return (h + 1) * (h + 1) + (d - h) * (d - h); }
int64_t gwfa_cigar_lds_bytes(const CigArgs& A) { return 8 * ((int64_t)A.lds_q + A.lds_t) + 8 * (int64_t)A.lds_row; }
hipError_t gwfa_launch_cigar(const CigArgs&, int groups, int, int, hipStream_t) { cig_groups = groups; return hipSuccess; }
