/* Mixed-size (ragged) batches (Section 4.1: a size-aware dispatcher picks the
 * specialised solver for each problem size).
 *
 * Systems are grouped by size on the device: a histogram, a plan that lays
 * the size bins out in descending n (costliest work first) and cuts each bin
 * into work items of one workgroup round, and a scatter of system indices
 * into the bins. The solve is then one launch per size class - classes of
 * sizes with the same register budget, so that each class runs at the
 * occupancy its largest size allows - with one workgroup per work item (in very
 * large batches a few items per workgroup), or one launch per size.
 *
 * System s: matrix column-major at A + offA[s] (lda = n[s]), right-hand side
 * and pivots at offset offB[s], info[s].
 */
#ifndef LUPP_KERNELS_RAGGED_H
#define LUPP_KERNELS_RAGGED_H

#include <utility>

#include "internal.h"
#include "kernels_seg.h"
#include "lupp_segments.h"

namespace lupp {

constexpr int kRaggedWaves = 4;       /* wave64s per workgroup */
constexpr int kRaggedThreads = 64 * kRaggedWaves;

/* Size classes of the ragged and grouped kernels, largest sizes first, each
 * the sizes with one register budget of the 16-lane solver (seg_shape): 22..32
 * (168 VGPRs, 3 waves per SIMD), 17..21 (128, 4 waves) and 1..16 (128). */
constexpr int kRaggedClasses = 3;
__host__ __device__ constexpr int ragged_class_lo(int c) { return c == 0 ? 22 : (c == 1 ? 17 : 1); }
__host__ __device__ constexpr int ragged_class_hi(int c) { return c == 0 ? 32 : (c == 1 ? 21 : 16); }
__host__ __device__ constexpr int ragged_class_of(int n) { return n >= 22 ? 0 : (n >= 17 ? 1 : 2); }
/* waves per SIMD each class kernel is compiled for */
__host__ __device__ constexpr int ragged_class_waves(int c) { return c == 0 ? 3 : 4; }

/* grouping kernels: at most this many workgroups of this many threads */
constexpr int kGroupBlocks = 256, kGroupThreads = 1024;

/* work items a workgroup of a class kernel takes at most. The loop over them
 * costs class 0 more registers than it has (44 bytes per lane of scratch), and
 * class 2, whose items hold twice the systems, 2 to 6% also where each
 * workgroup has one item. */
__host__ __device__ constexpr int ragged_class_items(int c) { return c == 1 ? 4 : 1; }

struct RaggedPlan {
    int32_t count[33];      /* systems of each size */
    int32_t bin_start[33];  /* first index of each size in `sorted` */
    int32_t item_start[33]; /* first work item of each size */
    /* work items of class c: class_start[c] .. class_start[c + 1] - 1 */
    int32_t class_start[kRaggedClasses + 1];
    int32_t part[kGroupBlocks][32]; /* systems of size m + 1 in each grouping chunk */
};

struct RaggedArgs {
    int64_t batch;
    const int32_t *n;
    const int64_t *offA, *offB;
    double *A, *b;
    int32_t *ipiv, *info;
    int factors;
    int32_t *sorted;
    RaggedPlan *plan;
    int32_t item0; /* first work item of this launch within its class */
    /* lanes per system for each size (ragged_lanes_ok). Words, not bytes:
     * 4-byte-aligned kernel arguments are read by scalar loads, where a byte
     * array is loaded into vector registers (and, in the looping
     * kernels, spilled to scratch memory) */
    int32_t lanes[33];
};

/* systems one workgroup solves at once with T lanes per system: one work
 * item (measured: four rounds per item ran 2-11% slower than one, the
 * workgroup's next loads then waiting for its previous solve) */
__host__ __device__ constexpr int ragged_per_round(int T)
{
    return T == 1 ? kRaggedThreads : kRaggedWaves * (64 / T);
}

__host__ __device__ constexpr int ragged_per_item(int T) { return ragged_per_round(T); }

/* LDS doubles of a wave: the solver records of its segments, for the size and
 * lane count of LO..HI that takes most */
template <int LO, int HI>
__host__ __device__ constexpr int ragged_lds()
{
    int most = 2;
    if constexpr (LO <= HI) {
        for (int T = 2; T <= 16; T *= 2)
            if (ragged_lanes_ok(LO, T)) {
                const int d = 64 / T * seg_lds<LO>::kStride;
                most = d > most ? d : most;
            }
        const int rest = ragged_lds<LO + 1, HI>();
        most = rest > most ? rest : most;
    }
    return most;
}

/* Where the j-th system of a work item lives: matrix (column-major, leading
 * dimension lda()), right-hand side, pivots and info. */
struct SysPtrs {
    double *A, *b;
    int32_t *ipiv, *info;
};

/* Ragged batches: the item's systems are entries of the sorted index list,
 * each at its own offsets, packed (lda = n). */
template <int N>
struct RaggedLoc {
    const RaggedArgs &a;
    const int32_t *idx;
    __device__ __forceinline__ SysPtrs sys(int j) const
    {
        const int64_t s = idx[j];
        return {a.A + a.offA[s], a.b + a.offB[s], a.ipiv + a.offB[s], a.info + s};
    }
    __device__ __forceinline__ int64_t lda() const { return N; }
};

/* The lane number, computed where it stands: kept out of the registers that
 * live across the work-item loop and the solves. */
__device__ __forceinline__ int fresh_lane()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

/* the wave's number in its workgroup (uniform) */
__device__ __forceinline__ int ragged_wave()
{
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

/* Solve the cnt (>= 1) systems of one work item with the whole workgroup, T
 * lanes per system (T == 1: one thread per system). Threads or segments
 * without a system point at system 0, load zeros and store nothing. lds: the
 * wave's solver records (ragged_lds), its own whatever the size: the waves of a
 * workgroup go from item to item without waiting for each other. W: waves per
 * SIMD of the kernel. */
template <int N, int T, int W, typename Loc>
__device__ __forceinline__ void solve_item(const Loc &loc, int cnt, int factors, double *lds)
{
    const int64_t lda = loc.lda();
    if constexpr (T == 1) {
        const int i = threadIdx.x;
        const bool act = i < cnt;
        const SysPtrs p = loc.sys(act ? i : 0); /* cnt >= 1: system 0 exists */
        double m[N][N], x[N];
        int piv[N];
        static_for<0, N>([&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            static_for<0, N>([&](auto ic) __attribute__((always_inline)) {
                constexpr int ii = decltype(ic)::value;
                m[j][ii] = act ? p.A[ii + j * lda] : 0.0;
            });
            x[j] = act ? p.b[j] : 0.0;
        });
        const int inf = thread_getrf_solve<N, true>(m, x, piv);
        if (act) {
            if (factors) {
                static_for<0, N>([&](auto jc) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value;
                    static_for<0, N>([&](auto ic) __attribute__((always_inline)) {
                        constexpr int ii = decltype(ic)::value;
                        p.A[ii + j * lda] = m[j][ii];
                    });
                });
            }
            static_for<0, N>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                p.ipiv[k] = piv[k];
                if (inf == 0) p.b[k] = x[k];
            });
            *p.info = inf;
        }
    } else {
        constexpr int K = lanes_shape<N, T>::K;
        constexpr bool PF = seg_shape<N, T>::waves(seg_shape<N, T>::kNeed + 28) >= W;
        constexpr int SPW = 64 / T;
        const int wave = ragged_wave();
        /* rebuilt after the solve, with the system's pointers, so that neither
         * stays live across it */
        int g, t;
        bool act;
        auto set_geometry = [&]() __attribute__((always_inline)) {
            const int lane = fresh_lane();
            g = lane / T;
            t = lane % T;
            act = wave * SPW + g < cnt;
        };
        set_geometry();
        double m[K][N], x[K];
        int pos[K];
        {
            const SysPtrs p = loc.sys(act ? wave * SPW + g : 0); /* cnt >= 1: system 0 exists */
            static_for<0, K>([&](auto sc) __attribute__((always_inline)) {
                constexpr int sl = decltype(sc)::value;
                const int r = t + sl * T;
                const bool ok = act && r < N;
                pos[sl] = r < N ? r : -1;
                static_for<0, N>([&](auto jc) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value;
                    m[sl][j] = ok ? p.A[r + j * lda] : 0.0;
                });
                x[sl] = ok ? p.b[r] : 0.0;
            });
        }
        double *rec = lds + g * seg_lds<N>::kStride;
        const int inf = seg_getrf_solve<N, T, false, seg_shape<N, T>::CH, PF>(m, x, pos, rec);
        set_geometry();
        rec = lds + g * seg_lds<N>::kStride;
        if (act) {
            const SysPtrs p = loc.sys(wave * SPW + g);
            const int *seq = reinterpret_cast<const int *>(rec + seg_lds<N>::kPos);
            static_for<0, K>([&](auto sc) __attribute__((always_inline)) {
                constexpr int sl = decltype(sc)::value;
                if (factors && pos[sl] >= 0) {
                    static_for<0, N>([&](auto jc) __attribute__((always_inline)) {
                        constexpr int j = decltype(jc)::value;
                        p.A[pos[sl] + j * lda] = m[sl][j];
                    });
                }
                const int r = t + sl * T;
                if (r < N) {
                    if (inf == 0) p.b[r] = rec[r];
                    p.ipiv[r] = seq[r] + 1;
                }
            });
            if (t == 0) *p.info = inf;
        }
    }
}

template <int N, int T, int W>
__device__ __forceinline__ void ragged_item(const RaggedArgs &a, int first, int cnt, double *lds)
{
    /* uniform: in scalar registers across the solve */
    const int at = __builtin_amdgcn_readfirstlane(a.plan->bin_start[N] + first);
    const RaggedLoc<N> loc{a, opaque_ptr(a.sorted + at)};
    solve_item<N, T, W>(loc, cnt, a.factors, lds);
}

template <int N, int T, int W>
__device__ __forceinline__ void ragged_run_item_t(const RaggedArgs &a, int it, double *lds)
{
    const int first = __builtin_amdgcn_readfirstlane((it - a.plan->item_start[N]) * ragged_per_item(T));
    const int rest = __builtin_amdgcn_readfirstlane(a.plan->count[N] - first);
    if (rest > 0) ragged_item<N, T, W>(a, first, rest < ragged_per_item(T) ? rest : ragged_per_item(T), lds);
}

template <int N, int T, int W>
__device__ __forceinline__ bool ragged_try_lanes(const RaggedArgs &a, int lanes, int it, double *lds)
{
    if constexpr (ragged_lanes_ok(N, T)) {
        if (lanes == T) {
            ragged_run_item_t<N, T, W>(a, it, lds);
            return true;
        }
    }
    return false;
}

/* Solve the work item `it` of size N (all threads of the workgroup) with the
 * lane count the table gives for N (uniform across the workgroup). */
template <int N, int W>
__device__ __forceinline__ void ragged_run_item(const RaggedArgs &a, int it, double *lds)
{
    if constexpr (N > kRaggedSmallMax) {
        /* 16 lanes: the only count compiled for these sizes (ragged_lanes_ok) */
        ragged_run_item_t<N, 16, W>(a, it, lds);
    } else {
        const int lanes = __builtin_amdgcn_readfirstlane((int)a.lanes[N]);
        (void)(ragged_try_lanes<N, 1, W>(a, lanes, it, lds) || ragged_try_lanes<N, 2, W>(a, lanes, it, lds) ||
               ragged_try_lanes<N, 4, W>(a, lanes, it, lds) || ragged_try_lanes<N, 8, W>(a, lanes, it, lds) ||
               ragged_try_lanes<N, 16, W>(a, lanes, it, lds));
    }
}

/* One size per launch: workgroup b solves work item b of size N. */
template <int N>
__global__ void __launch_bounds__(kRaggedThreads)
    __attribute__((amdgpu_waves_per_eu(ragged_class_waves(ragged_class_of(N))))) k_ragged_one(RaggedArgs a)
{
    __shared__ __align__(16) double lds[kRaggedWaves][ragged_lds<N, N>()];
    const int it = a.plan->item_start[N] + (int)xcd_block(blockIdx.x, gridDim.x);
    ragged_run_item<N, ragged_class_waves(ragged_class_of(N))>(a, it, lds[ragged_wave()]);
}

template <int N, int W>
__device__ __forceinline__ bool ragged_try(const RaggedArgs &a, int n, int it, double *lds)
{
    if (n != N) return false;
    ragged_run_item<N, W>(a, it, lds);
    return true;
}

template <int LO, int W, int... Ns>
__device__ __forceinline__ void ragged_dispatch(const RaggedArgs &a, int n, int it, double *lds,
                                                std::integer_sequence<int, Ns...>)
{
    (void)(ragged_try<LO + Ns, W>(a, n, it, lds) || ...);
}

/* Work item i of class C (sizes LO..HI) in this launch; false past the last.
 * The size of an item is the smallest m whose first item is at or before it
 * (empty sizes start where the next one does). */
template <int C>
__device__ __forceinline__ bool ragged_class_item(const RaggedArgs &a, int i, double *lds)
{
    constexpr int LO = ragged_class_lo(C), HI = ragged_class_hi(C);
    const RaggedPlan *plan = a.plan;
    const int c0 = __builtin_amdgcn_readfirstlane(plan->class_start[C] + a.item0);
    const int left = __builtin_amdgcn_readfirstlane(plan->class_start[C + 1] - c0);
    if (i >= left) return false;
    const int it = c0 + i;
    int n = HI;
    for (int m = HI - 1; m >= LO; --m)
        if (plan->item_start[m] <= it) n = m;
    n = __builtin_amdgcn_readfirstlane(n);
    ragged_dispatch<LO, ragged_class_waves(C)>(a, n, it, lds, std::make_integer_sequence<int, HI - LO + 1>{});
    return true;
}

/* Work items a.item0 + b, b + G, ... (at most ragged_class_items) of class C by
 * workgroup b of G, largest sizes first. Neighbouring workgroups go to the XCDs
 * in turn, so each XCD gets the same mix of sizes: with one contiguous range of
 * items per XCD the first one had all the largest systems. The host does not
 * know how many items a class has, so the grid follows the bound that the batch
 * size gives (ragged_grid), and workgroups without an item end at once.
 *
 * Nothing may live across the solves but the item's number: the arguments are
 * read anew through a pointer the compiler cannot follow, and the kernel that
 * loops is compiled without the hoisting of constants out of loops (NO_HOIST in
 * build.py), which kept 41 registers alive across the solve and put 48 bytes per
 * lane into scratch memory. A second item is slower than a second workgroup all
 * the same (its loads wait for the first one's stores, which count on the same
 * counter: 2000000 systems of n = 17..21 2789 against 2956 us): only very large
 * batches have one. */
template <int C>
__device__ __forceinline__ void ragged_class(const RaggedArgs &direct)
{
    __shared__ __align__(16) double lds[kRaggedWaves][ragged_lds<ragged_class_lo(C), ragged_class_hi(C)>()];
    int i = (int)blockIdx.x;
    if constexpr (ragged_class_items(C) == 1) {
        (void)ragged_class_item<C>(direct, i, lds[ragged_wave()]);
    } else {
#pragma clang loop unroll(disable)
        for (int r = 0; r < ragged_class_items(C); ++r, i += (int)gridDim.x) {
            auto args = (const __attribute__((address_space(4))) RaggedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(args));
            if (!ragged_class_item<C>(*(const RaggedArgs *)args, i, lds[ragged_wave()])) return;
        }
    }
}

/* ------------------------------------------------------------------------ */
/* Grouped batches: up to kMaxGroups uniform batches, each with its own size,  */
/* pointers and strides (AoS), solved by one launch per size class. The host   */
/* knows every group's size, so no grouping kernels and no work counter are   */
/* needed: workgroup w takes work item w, and the group table (kernel          */
/* arguments, read with scalar loads) gives its group.                         */
/* ------------------------------------------------------------------------ */
constexpr int kMaxGroups = 32;

struct GroupDesc {
    double *A, *b;
    int32_t *ipiv, *info;
    int64_t lda, sA, sB, batch;
    int32_t n, lanes;
    int32_t item0;   /* first work item of the group in its launch */
    int32_t factors; /* write the factors back (else A is only read) */
};

struct GroupedArgs {
    int32_t ngroups, pad;
    GroupDesc g[kMaxGroups]; /* ascending item0 */
};

/* System s of a group: matrix at A + s*sA (leading dimension lda), right-hand
 * side at b + s*sB, pivots at ipiv + s*n, info[s]. */
template <int N>
struct GroupLoc {
    const GroupDesc &g;
    int64_t first;
    __device__ __forceinline__ SysPtrs sys(int j) const
    {
        const int64_t s = first + j;
        return {g.A + s * g.sA, g.b + s * g.sB, g.ipiv + s * N, g.info + s};
    }
    __device__ __forceinline__ int64_t lda() const { return g.lda; }
};

/* systems of one grouped work item: one round of the workgroup */
__host__ __device__ constexpr int grouped_per_item(int T) { return ragged_per_round(T); }

template <int N, int T, int W>
__device__ __forceinline__ bool grouped_try_lanes(const GroupDesc &g, int lanes, int local,
                                                  int factors, double *lds)
{
    if constexpr (ragged_lanes_ok(N, T)) {
        if (lanes == T) {
            const int64_t first = (int64_t)local * grouped_per_item(T);
            const int64_t rest = g.batch - first;
            const int cnt = (int)(rest < grouped_per_item(T) ? rest : grouped_per_item(T));
            solve_item<N, T, W>(GroupLoc<N>{g, first}, cnt, factors, lds);
            return true;
        }
    }
    return false;
}

template <int N, int W>
__device__ __forceinline__ bool grouped_try(const GroupDesc &g, int n, int local, int factors,
                                            double *lds)
{
    if (n != N) return false;
    if constexpr (N > kRaggedSmallMax) {
        (void)grouped_try_lanes<N, 16, W>(g, 16, local, factors, lds); /* the only count compiled */
    } else {
        const int lanes = __builtin_amdgcn_readfirstlane(g.lanes);
        (void)(grouped_try_lanes<N, 1, W>(g, lanes, local, factors, lds) ||
               grouped_try_lanes<N, 2, W>(g, lanes, local, factors, lds) ||
               grouped_try_lanes<N, 4, W>(g, lanes, local, factors, lds) ||
               grouped_try_lanes<N, 8, W>(g, lanes, local, factors, lds) ||
               grouped_try_lanes<N, 16, W>(g, lanes, local, factors, lds));
    }
    return true;
}

template <int LO, int W, int... Ns>
__device__ __forceinline__ void grouped_dispatch(const GroupDesc &g, int n, int local, int factors,
                                                 double *lds, std::integer_sequence<int, Ns...>)
{
    (void)(grouped_try<LO + Ns, W>(g, n, local, factors, lds) || ...);
}

/* Work item `it` of a grouped launch over the sizes of class C (all threads of
 * the workgroup; items to workgroups in launch order, as in
 * ragged_class): find its group (uniform), then solve its systems. */
template <int C>
__device__ __forceinline__ void grouped_run(const GroupedArgs &a, int it)
{
    constexpr int LO = ragged_class_lo(C), HI = ragged_class_hi(C);
    __shared__ __align__(16) double lds[kRaggedWaves][ragged_lds<LO, HI>()];
    int gi = 0;
    for (int k = 1; k < a.ngroups; ++k)
        if (it >= a.g[k].item0) gi = k;
    gi = __builtin_amdgcn_readfirstlane(gi);
    const GroupDesc &g = a.g[gi];
    grouped_dispatch<LO, ragged_class_waves(C)>(g, __builtin_amdgcn_readfirstlane(g.n), it - g.item0,
                                                g.factors, lds[ragged_wave()],
                                                std::make_integer_sequence<int, HI - LO + 1>{});
}

/* Grouped kernels (grouped_c0.hip .. grouped_c2.hip), one per size class:
 * one workgroup per work item. */
hipError_t grouped_c0_launch(const GroupedArgs &a, unsigned items, hipStream_t st);
hipError_t grouped_c1_launch(const GroupedArgs &a, unsigned items, hipStream_t st);
hipError_t grouped_c2_launch(const GroupedArgs &a, unsigned items, hipStream_t st);

/* Ragged kernels (ragged_c0.hip .. ragged_c2.hip: separate translation units,
 * compiled in parallel), one per size class: `grid` workgroups each. */
hipError_t ragged_c0_launch(const RaggedArgs &a, unsigned grid, hipStream_t st);
hipError_t ragged_c1_launch(const RaggedArgs &a, unsigned grid, hipStream_t st);
hipError_t ragged_c2_launch(const RaggedArgs &a, unsigned grid, hipStream_t st);

}  // namespace lupp

#define LUPP_RAGGED_ONE_INSTANCE(N)                                                 \
    namespace lupp {                                                               \
    hipError_t ragged_one_launch_##N(const RaggedArgs &a, int items, hipStream_t st)   \
    {                                                                              \
        if (items <= 0) return hipSuccess;                                         \
        hipLaunchKernelGGL((k_ragged_one<N>), dim3((unsigned)items), dim3(kRaggedThreads), 0, st, a); \
        return hipGetLastError();                                                  \
    }                                                                              \
    }

#endif
