/* Ragged (mixed-size) batches: device-side grouping by size and one launch
 * per size class (see kernels_ragged.h). */
#include <cstddef>
#include <cstring>

#include "kernels_ragged.h"

namespace lupp {

/* Grouping by size, in two kernels. Workgroup g owns the contiguous chunk of
 * systems [g*chunk, (g+1)*chunk), chunk a multiple of the workgroup: the first
 * kernel counts the sizes of every chunk (RaggedPlan::part), the second sums
 * these counts for the plan and for the place of its own systems in the bins.
 * No global atomics and nothing to clear; every call writes all it reads.
 *
 * What it costs is latency, not the 12 bytes per system it moves: a launch of
 * a few microseconds per kernel, atomics of many workgroups on 32 addresses.
 * Hence few, large workgroups, and the 32-entry plan by scans of one wave in
 * every workgroup of the second kernel. Four kernels (clear, count with
 * global atomics on up to 1024 workgroups of 256, plan by one thread, scatter)
 * took 22 us for 20,000 systems, 50 for 250,000 and 60 for 2,000,000; these two
 * take 10, 10 and 18. */
__device__ __forceinline__ void ragged_chunk(const RaggedArgs &a, int64_t &c0, int64_t &c1)
{
    const int64_t chunk = ((a.batch + gridDim.x - 1) / gridDim.x + kGroupThreads - 1) / kGroupThreads *
                          kGroupThreads;
    c0 = (int64_t)blockIdx.x * chunk;
    c1 = c0 + chunk < a.batch ? c0 + chunk : a.batch;
}

/* systems of each size in the chunk, privatised in LDS */
__global__ void __launch_bounds__(kGroupThreads) k_ragged_hist(RaggedArgs a)
{
    __shared__ int h[32];
    if (threadIdx.x < 32) h[threadIdx.x] = 0;
    __syncthreads();
    int64_t c0, c1;
    ragged_chunk(a, c0, c1);
#pragma unroll 4
    for (int64_t s = c0 + threadIdx.x; s < c1; s += kGroupThreads) {
        const int n = a.n[s];
        if (n >= 1 && n <= 32) atomicAdd(&h[n - 1], 1);
    }
    __syncthreads();
    if (threadIdx.x < 32) a.plan->part[blockIdx.x][threadIdx.x] = h[threadIdx.x];
}

/* The plan, bins in descending size (work items per bin follow the lane count
 * of the size), and the system indices in their bins: chunk by chunk within a
 * bin, in any order within a chunk (systems are independent). */
__global__ void __launch_bounds__(kGroupThreads) k_ragged_scatter(RaggedArgs a)
{
    /* by size - 1: systems, those of earlier chunks, next index of this chunk */
    __shared__ int total[32], before[32], next[32];
    RaggedPlan *plan = a.plan;
    const int tid = (int)threadIdx.x;
    if (tid < 32) total[tid] = before[tid] = 0;
    __syncthreads();
    {
        int tot = 0, bef = 0;
#pragma unroll 4
        for (int g = tid >> 5; g < (int)gridDim.x; g += kGroupThreads / 32) {
            const int v = plan->part[g][tid & 31];
            tot += v;
            bef += g < (int)blockIdx.x ? v : 0;
        }
        atomicAdd(&total[tid & 31], tot);
        atomicAdd(&before[tid & 31], bef);
    }
    __syncthreads();
    if (tid < 32) {
        /* lane i holds size 32 - i: inclusive scans over descending sizes */
        const int n = 32 - tid, c = total[n - 1];
        const int per = ragged_per_item(a.lanes[n]);
        const int it = (c + per - 1) / per;
        int cs = c, is = it;
        for (int d = 1; d < 32; d *= 2) {
            const int cu = __shfl_up(cs, d, 32), iu = __shfl_up(is, d, 32);
            cs += tid >= d ? cu : 0;
            is += tid >= d ? iu : 0;
        }
        next[n - 1] = cs - c + before[n - 1];
        if (blockIdx.x == 0) {
            plan->count[n] = c;
            plan->bin_start[n] = cs - c;
            plan->item_start[n] = is - it;
            if (n == ragged_class_hi(ragged_class_of(n))) plan->class_start[ragged_class_of(n)] = is - it;
            if (n == 1) plan->class_start[kRaggedClasses] = is;
        }
    }
    __syncthreads();
    int64_t c0, c1;
    ragged_chunk(a, c0, c1);
#pragma unroll 4
    for (int64_t s = c0 + tid; s < c1; s += kGroupThreads) {
        const int n = a.n[s];
        if (n >= 1 && n <= 32) a.sorted[atomicAdd(&next[n - 1], 1)] = (int32_t)s;
        else a.info[s] = -1;
    }
}

hipError_t ragged_one_launch(int n, const RaggedArgs &a, int items, hipStream_t st);

/* Workspace of the allocating entry point. Calls on one context may come on
 * different streams: `done` is recorded after each call's last kernel, and
 * the next call on another stream waits for it before its grouping kernels
 * rewrite the plan and `sorted` (which the earlier call's solve
 * kernels may still be reading). */
struct RaggedWs {
    RaggedPlan *plan = nullptr;
    int32_t *sorted = nullptr;
    int64_t cap = 0;
    hipEvent_t done = nullptr;
    hipStream_t last = nullptr;
    bool used = false;
};

RaggedWs *ragged_ws_create() { return new RaggedWs; }

void ragged_ws_destroy(RaggedWs *ws)
{
    if (ws == nullptr) return;
    if (ws->done) {
        hipEventSynchronize(ws->done);
        hipEventDestroy(ws->done);
    }
    hipFree(ws->sorted);
    hipFree(ws->plan);
    delete ws;
}

/* Workgroups for at most `items` work items of class c. A workgroup without an
 * item costs 0.22 ns, which a batch of small sizes pays for every class it does
 * not use. Up to kOnePer possible items (14 us) there is a workgroup for each;
 * beyond, a workgroup takes up to ragged_class_items. 2000000 systems of n = 1 /
 * 2 / 3 / 2..4, us: ds_bpermute kernels on resident grids 98 / 101 / 130 / 205,
 * a workgroup for each possible item 121 / 130 / 146 / 213, this 104 / 110 / 127 /
 * 196; n = 17..21, whose workgroups do take several items, 4370, 2735, 2940. At
 * 1000000 systems the second form was no slower than the first any more. */
static unsigned ragged_grid(int c, int64_t items)
{
    constexpr int64_t kOnePer = 65536;
    return (unsigned)(items <= kOnePer ? items : (items + ragged_class_items(c) - 1) / ragged_class_items(c));
}

int ragged_enqueue(RaggedPlan *plan, int32_t *sorted, const uint8_t *lanes, int64_t batch,
                   const int32_t *n, const int64_t *offA, const int64_t *offB, double *A, double *b,
                   int32_t *ipiv, int32_t *info, bool factors, bool per_size, hipStream_t st)
{
    RaggedArgs a{batch, n, offA, offB, A, b, ipiv, info, factors ? 1 : 0, sorted, plan, 0, {}};
    for (int m = 0; m <= 32; ++m) a.lanes[m] = m >= 1 ? lanes[m] : 1;
    const int64_t full = (batch + kGroupThreads - 1) / kGroupThreads;
    const unsigned blocks = (unsigned)(full < kGroupBlocks ? full : kGroupBlocks);
    hipLaunchKernelGGL(k_ragged_hist, dim3(blocks), dim3(kGroupThreads), 0, st, a);
    hipLaunchKernelGGL(k_ragged_scatter, dim3(blocks), dim3(kGroupThreads), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e);
    if (!per_size) {
        /* for as many items as a class can have: every system in its size with
         * the fewest systems per item, and one item that is not full per size;
         * in launches of at most kMaxItems (a multiple of ragged_class_items) */
        constexpr int64_t kMaxItems = (int64_t)1 << 23;
        hipError_t (*const launch[kRaggedClasses])(const RaggedArgs &, unsigned, hipStream_t) = {
            ragged_c0_launch, ragged_c1_launch, ragged_c2_launch};
        for (int c = 0; c < kRaggedClasses && e == hipSuccess; ++c) {
            int per = kRaggedThreads;
            for (int m = ragged_class_lo(c); m <= ragged_class_hi(c); ++m)
                per = ragged_per_item(a.lanes[m]) < per ? ragged_per_item(a.lanes[m]) : per;
            const int64_t most = batch / per + (ragged_class_hi(c) - ragged_class_lo(c) + 1);
            for (int64_t i0 = 0; i0 < most && e == hipSuccess; i0 += kMaxItems) {
                a.item0 = (int32_t)i0;
                e = launch[c](a, ragged_grid(c, most - i0 < kMaxItems ? most - i0 : kMaxItems), st);
            }
        }
        return hip_err(e);
    }
    /* one launch per size: the host reads the plan (a synchronisation) */
    RaggedPlan h;
    e = hipMemcpyAsync(&h, plan, offsetof(RaggedPlan, part), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_err(e);
    for (int m = 32; m >= 1; --m) {
        const int per = ragged_per_item(a.lanes[m]);
        const int items = (h.count[m] + per - 1) / per;
        e = ragged_one_launch(m, a, items, st);
        if (e != hipSuccess) return hip_err(e);
    }
    return 0;
}

int ragged_launch_impl(RaggedWs *ws, const uint8_t *lanes, int64_t batch, const int32_t *n,
                       const int64_t *offA, const int64_t *offB, double *A, double *b,
                       int32_t *ipiv, int32_t *info, bool factors, bool per_size, hipStream_t st)
{
    if (batch > 0x7fffffff) return LUPP_E_UNSUPPORTED;
    hipError_t e = hipSuccess;
    if (ws->done == nullptr) {
        e = hipEventCreateWithFlags(&ws->done, hipEventDisableTiming);
        if (e != hipSuccess) return hip_err(e);
    }
    if (ws->cap < batch) {
        if (ws->sorted) {
            /* the previous call, on whatever stream, must be done with it */
            e = hipEventSynchronize(ws->done);
            if (e != hipSuccess) return hip_err(e);
            hipFree(ws->sorted);
            ws->sorted = nullptr;
            ws->cap = 0;
        }
        const int64_t cap = batch < 65536 ? 65536 : batch;
        e = hipMalloc(&ws->sorted, (size_t)cap * sizeof(int32_t));
        if (e != hipSuccess) return e == hipErrorOutOfMemory ? LUPP_E_NOMEM : hip_err(e);
        ws->cap = cap;
    }
    if (ws->plan == nullptr) {
        e = hipMalloc(&ws->plan, sizeof(RaggedPlan));
        if (e != hipSuccess) return hip_err(e);
    }
    /* a call being captured into a graph is ordered by the graph, not by
     * the eager event chain */
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(st, &cs);
    if (e != hipSuccess) return hip_err(e);
    const bool capturing = cs != hipStreamCaptureStatusNone;
    if (!capturing && ws->used && ws->last != st) {
        e = hipStreamWaitEvent(st, ws->done, 0);
        if (e != hipSuccess) return hip_err(e);
    }
    const int rc = ragged_enqueue(ws->plan, ws->sorted, lanes, batch, n, offA, offB, A, b, ipiv,
                                  info, factors, per_size, st);
    if (capturing) return rc;
    e = hipEventRecord(ws->done, st);
    ws->last = st;
    ws->used = true;
    return rc != 0 ? rc : hip_err(e);
}

/* offsets of a packed single-size batch: system s at s*n*n (matrix) and s*n
 * (right-hand side, pivots) */
__global__ void __launch_bounds__(256) k_ragged_uniform(int64_t batch, int n, int32_t *nv,
                                                        int64_t *offA, int64_t *offB)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= batch) return;
    nv[s] = n;
    offA[s] = s * n * n;
    offB[s] = s * n;
}

int ragged_autotune_impl(RaggedWs *ws, uint8_t *lanes, int n, int64_t batch, const double *A,
                         const double *b, int reps, int *best, float *best_ms, hipStream_t st)
{
    const size_t nA = (size_t)batch * n * n, nB = (size_t)batch * n;
    double *wA = nullptr, *wB = nullptr;
    int32_t *wN = nullptr, *wP = nullptr, *wI = nullptr;
    int64_t *oA = nullptr, *oB = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = 0;
    hipError_t e = hipMalloc(&wA, nA * 8);
    if (e == hipSuccess) e = hipMalloc(&wB, nB * 8);
    if (e == hipSuccess) e = hipMalloc(&wN, (size_t)batch * 4);
    if (e == hipSuccess) e = hipMalloc(&wP, nB * 4);
    if (e == hipSuccess) e = hipMalloc(&wI, (size_t)batch * 4);
    if (e == hipSuccess) e = hipMalloc(&oA, (size_t)batch * 8);
    if (e == hipSuccess) e = hipMalloc(&oB, (size_t)batch * 8);
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e != hipSuccess) rc = e == hipErrorOutOfMemory ? LUPP_E_NOMEM : hip_err(e);
    if (rc == 0) {
        hipLaunchKernelGGL(k_ragged_uniform, dim3((unsigned)((batch + 255) / 256)), dim3(256), 0, st,
                           batch, n, wN, oA, oB);
        e = hipGetLastError();
        if (e != hipSuccess) rc = hip_err(e);
    }
    const uint8_t keep = lanes[n];
    int pick = 0;
    float pick_ms = 3.0e38f;
    const int cands[6] = {1, 2, 4, 8, 16, 32};
    for (int c = 0; c < 6 && rc == 0; ++c) {
        if (!ragged_lanes_ok(n, cands[c])) continue;
        lanes[n] = (uint8_t)cands[c];
        float t[64];
        const int r_total = reps + 1 < 64 ? reps + 1 : 64;
        for (int r = 0; r < r_total && rc == 0; ++r) {
            e = hipMemcpyAsync(wA, A, nA * 8, hipMemcpyDeviceToDevice, st);
            if (e == hipSuccess) e = hipMemcpyAsync(wB, b, nB * 8, hipMemcpyDeviceToDevice, st);
            if (e == hipSuccess) e = hipEventRecord(e0, st);
            if (e != hipSuccess) { rc = hip_err(e); break; }
            rc = ragged_launch_impl(ws, lanes, batch, wN, oA, oB, wA, wB, wP, wI, true, false, st);
            if (rc != 0) break;
            e = hipEventRecord(e1, st);
            if (e == hipSuccess) e = hipEventSynchronize(e1);
            if (e == hipSuccess) e = hipEventElapsedTime(&t[r], e0, e1);
            if (e != hipSuccess) rc = hip_err(e);
        }
        if (rc != 0) break;
        /* median of the timed repetitions (the first run is a warm-up) */
        for (int i = 1; i < r_total; ++i)
            for (int j = i + 1; j < r_total; ++j)
                if (t[j] < t[i]) { const float x = t[i]; t[i] = t[j]; t[j] = x; }
        const float med = t[1 + (r_total - 1) / 2];
        if (med < pick_ms) { pick_ms = med; pick = cands[c]; }
    }
    lanes[n] = (rc == 0 && pick != 0) ? (uint8_t)pick : keep;
    if (rc == 0) {
        if (best) *best = pick;
        if (best_ms) *best_ms = pick_ms;
    }
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    hipFree(wA);
    hipFree(wB);
    hipFree(wN);
    hipFree(wP);
    hipFree(wI);
    hipFree(oA);
    hipFree(oB);
    return rc;
}

}  // namespace lupp
