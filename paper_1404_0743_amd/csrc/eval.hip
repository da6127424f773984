// eval.hip -- C ABI of the endgame solver: arbitrary boards solved to the
// full board over all 256 quadrant rotations (Section VIII serial solver),
// binned by number of empty cells on the device.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <set>

#include "internal.h"

namespace pg {

static std::mutex g_pool_mutex;
static std::set<int> g_pool_ready;

// Keep stream-ordered allocations pooled instead of returning them to the
// driver after every call.
void keep_pool(int dev)
{
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    if (g_pool_ready.count(dev)) return;
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) {
        uint64_t big = ~0ull;
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &big);
    }
    g_pool_ready.insert(dev);
}

int eval_grid(int *grid)
{
    static int cached[64] = {0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 64 && cached[dev]) {
        *grid = cached[dev];
        return 0;
    }
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    // workgroups with a layer slot of their own for roots with 9 or 10 empty
    // cells, and those of the server's batches with 8 to 10: two per CU, as the
    // LDS of one root with 8 allows
    *grid = std::max(1, 2 * cus);
    if (dev < 64) cached[dev] = *grid;
    keep_pool(dev);
    return 0;
}

struct EvalAlloc {
    void *base = nullptr;
    EvalScratch S;
};

static int eval_alloc(size_t n, int grid, hipStream_t st, EvalAlloc *A)
{
    const size_t ints = 64;
    grid = (int)std::min<size_t>(n, (size_t)grid);  // a layer slot per workgroup, no more of them than roots
    const size_t glayer = (size_t)grid * 2 * kDagGlobalLayer * 64;
    const size_t bytes = glayer + ints * 4 + 64 + n * 4 + n + 256;
    hipError_t e = hipMallocAsync(&A->base, bytes, st);
    if (e != hipSuccess) return hip_fail(e, "hipMallocAsync(eval scratch)");
    char *p = (char *)A->base;
    A->S.global_layers = (uint4 *)p;
    p += glayer;
    A->S.count = (int *)p;
    A->S.start = A->S.count + 16;
    A->S.cursor = A->S.count + 32;
    p += ints * 4;
    static_assert(kEvalCounters * sizeof(unsigned long long) <= 64, "queue counters");
    A->S.counter = (unsigned long long *)p;
    p += 64;
    A->S.order = (int *)p;
    p += n * 4;
    A->S.empties = (uint8_t *)p;
    A->S.global_slots = grid;
    return 0;
}

// Scratch bytes of one endgame batch of n roots (deep: some root has 9 or
// 10 empty cells and needs the global layer buffers).
size_t eval_scratch_bytes(size_t n, int grid, bool deep)
{
    return (deep ? (size_t)grid * 2 * kDagGlobalLayer * 64 : 0) + 64 * 4 + 32 + n * 5 + 256;
}

// Enqueue one batch whose roots all belong to endgame class cls (see
// launch_eval_direct): one queue counter and, for roots with 9 or 10 empty
// cells, the global layer slots; no binning.
int eval_enqueue_class(const uint64_t *boards, size_t n, uint4 *out, int cls, bool deep, int grid,
                       hipStream_t st)
{
    DevTables T;
    int rc = device_tables(&T);
    if (rc) return rc;
    void *base = nullptr;
    const size_t glayer = deep ? (size_t)grid * 2 * kDagGlobalLayer * 64 : 0;
    hipError_t e = hipMallocAsync(&base, glayer + 256, st);
    if (e != hipSuccess) return hip_fail(e, "hipMallocAsync(eval scratch)");
    uint4 *gl = deep ? (uint4 *)base : nullptr;
    unsigned long long *counter = (unsigned long long *)((char *)base + glayer);
    e = launch_eval_direct(boards, (int)n, out, cls, counter, gl, grid, T, st);
    (void)hipFreeAsync(base, st);
    if (e != hipSuccess) return hip_fail(e, "eval launch");
    return 0;
}

}  // namespace pg

using namespace pg;

extern "C" {

int pentago_eval_batch(const pentago_board *boards, size_t n, pentago_superinfo *out,
                       int32_t *status, void *hip_stream)
{
    if (n && (!boards || !out)) return fail(PENTAGO_EINVAL, "NULL boards or out");
    if (n > (size_t)1 << 30) return fail(PENTAGO_ERANGE, "more than 2^30 boards");
    if (n == 0) return 0;
    DevTables T;
    int rc = device_tables(&T);
    if (rc) return rc;
    int grid;
    rc = eval_grid(&grid);
    if (rc) return rc;
    const hipStream_t st = (hipStream_t)hip_stream;
    EvalAlloc A;
    rc = eval_alloc(n, grid, st, &A);
    if (rc) return rc;
    const hipError_t e = launch_eval((const uint64_t *)boards, n, (uint4 *)out, A.S, status, T, st);
    (void)hipFreeAsync(A.base, st);
    if (e != hipSuccess) return hip_fail(e, "eval launch");
    return 0;
}

int pentago_autotune_eval(const pentago_board *boards, size_t n, pentago_superinfo *out, void *hip_stream,
                          int threads[2], float *best_ms)
{
    if (n && (!boards || !out)) return fail(PENTAGO_EINVAL, "NULL boards or out");
    if (n > (size_t)1 << 30) return fail(PENTAGO_ERANGE, "more than 2^30 boards");
    if (n == 0) return 0;
    const hipStream_t st = (hipStream_t)hip_stream;
    int dev = 0, cus = 0, grid = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    int rc = eval_grid(&grid);
    if (rc) return rc;
    // the classes these boards have roots of: a batch that goes without binning
    // reaches none of their kernels
    int roots[kEvalThreadClasses] = {0, 0, 0};
    if (n > (size_t)eval_few_boards(cus, (int)std::min<size_t>(n, (size_t)grid))) {
        EvalAlloc A;
        rc = eval_alloc(n, grid, st, &A);
        if (rc) return rc;
        int start[16];
        e = launch_eval_bin((const uint64_t *)boards, n, A.S, nullptr, (uint4 *)out, st);
        if (e == hipSuccess) e = hipMemcpyAsync(start, A.S.start, sizeof(start), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        (void)hipFreeAsync(A.base, st);
        if (e != hipSuccess) return hip_fail(e, "eval launch");
        roots[0] = start[8];
        roots[1] = start[7] - start[8];
        roots[2] = start[6] - start[7];
    }
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess)
        return fail(PENTAGO_EDEVICE, "hipEventCreate");
    auto time = [&] {
        rc = pentago_eval_batch(boards, n, out, nullptr, hip_stream);  // warm-up
        float t = 1e30f;
        for (int rep = 0; rep < 3 && rc == 0; rep++) {
            (void)hipEventRecord(a, st);
            rc = pentago_eval_batch(boards, n, out, nullptr, hip_stream);
            (void)hipEventRecord(b, st);
            if (hipEventSynchronize(b) != hipSuccess) rc = fail(PENTAGO_EDEVICE, "hipEventSynchronize");
            float ms = 0;
            (void)hipEventElapsedTime(&ms, a, b);
            t = std::min(t, ms);
        }
        return t;
    };
    float best = time();
    // The classes' launches follow one another, so each size is tried by itself;
    // it changes where that gains 2 %, more than repeated runs differ.
    for (int cls = 0; cls < kEvalThreadClasses && rc == 0; cls++) {
        if (roots[cls] == 0) continue;
        const int kept = get_eval_class_threads(cls);
        set_eval_class_threads(cls, 768 - kept);
        const float t = time();
        if (rc == 0 && t < 0.98f * best) best = t;
        else set_eval_class_threads(cls, kept);
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (rc) return rc;
    if (threads) {
        threads[0] = get_eval_class_threads(1);
        threads[1] = get_eval_class_threads(2);
    }
    if (best_ms) *best_ms = best;
    return rc;
}

int pentago_eval_batch_grouped(const pentago_board *boards, size_t n, pentago_superinfo *out,
                               int32_t *status, void *hip_stream)
{
    if (n && (!boards || !out)) return fail(PENTAGO_EINVAL, "NULL boards or out");
    if (n > (size_t)1 << 30) return fail(PENTAGO_ERANGE, "more than 2^30 boards");
    if (n == 0) return 0;
    DevTables T;
    int rc = device_tables(&T);
    if (rc) return rc;
    int grid;
    rc = eval_grid(&grid);
    if (rc) return rc;
    const hipStream_t st = (hipStream_t)hip_stream;
    EvalAlloc A;
    rc = eval_alloc(n, grid, st, &A);
    if (rc) return rc;
    hipError_t e = launch_eval_bin((const uint64_t *)boards, n, A.S, status, (uint4 *)out, st);
    int start[16];
    if (e == hipSuccess) e = hipMemcpyAsync(start, A.S.start, sizeof(start), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    for (int k = 10; k >= 0 && e == hipSuccess; k--) {
        const int first = start[k];
        const int count = (k == 0 ? start[11] : start[k - 1]) - first;
        e = launch_eval_group((const uint64_t *)boards, k, first, count, (uint4 *)out, A.S, T, st);
    }
    (void)hipFreeAsync(A.base, st);
    if (e != hipSuccess) return hip_fail(e, "eval launch");
    return 0;
}

}  // extern "C"
