/* Lanes-per-system batched solve in strict and FMA arithmetic (Section 3.2,
 * multi-threaded solvers): T lanes of a wave64 share one system and solve it
 * with seg_getrf_solve (lupp_segments.h). AoS layout here, the interleaved
 * one in kernels_seg_soa.h; tile-local pivoting keeps the kernels of
 * kernels_lanes.h and kernels_lanes_soa.h.
 *
 * Wave w of the workgroup serves systems (block*wpb + w)*(64/T) + g for
 * segments g = 0..64/T-1; lane t of segment g loads rows t, t+T, ...: T
 * consecutive doubles of a column per load. Lanes past the end of the batch
 * and phantom rows use an out-of-range buffer offset: they load zeros and
 * store nothing. */
#ifndef LUPP_KERNELS_SEG_H
#define LUPP_KERNELS_SEG_H

#include "internal.h"
#include "lupp_segments.h"

namespace lupp {

/* Register budget of the solve per (n, T): the matrix takes 2*K*n VGPRs, one
 * chunk of 4 columns of the two pivot rows and what else is live in a step
 * 28 + 6*K (a fit to what the compiler allocates), a second chunk in flight 16
 * more. The kernels are compiled for the most waves per SIMD that leaves no scratch
 * memory (a spilled n = 32 instance ran at half the speed); chunks of 4
 * columns are fetched ahead where that costs no wave. */
template <int N, int T>
struct seg_shape {
    static constexpr int K = (N + T - 1) / T;
    static constexpr int waves(int vgprs)
    {
        return vgprs <= 64 ? 8 : vgprs <= 72 ? 7 : vgprs <= 80 ? 6 : vgprs <= 96 ? 5 :
               vgprs <= 128 ? 4 : vgprs <= 168 ? 3 : vgprs <= 256 ? 2 : 1;
    }
    static constexpr int kNeed = 2 * K * N + 28 + 6 * K; /* one chunk of 4 columns */
    static constexpr int W = waves(kNeed);
    static constexpr bool PF = waves(kNeed + 16) == W;
    static constexpr int CH = 4;
};

template <int N, int T, bool F>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(seg_shape<N, T>::W, seg_shape<N, T>::W)))
    k_seg(SolveArgs a, int factors)
{
    using Sh = seg_shape<N, T>;
    constexpr int K = Sh::K, SPW = 64 / T;
    __shared__ __align__(16) double lds[4 * SPW * seg_lds<N>::kStride];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t sys0 = ((int64_t)xcd_block(blockIdx.x, gridDim.x) * (blockDim.x >> 6) + wave) * SPW;
    const int64_t rem = a.batch - sys0;
    const int nvalid = (int)(rem <= 0 ? 0 : (rem < SPW ? rem : SPW));

    /* Lane geometry: rebuilt after the solve from a fenced copy of the lane
     * number, so that none of it stays live across the solve. */
    int lane = (int)__lane_id(), g, t;
    auto set_geometry = [&]() __attribute__((always_inline)) {
        g = lane / T;
        t = lane % T;
    };
    set_geometry();

    double *baseA = a.A + sys0 * a.sA;
    double *baseB = a.b + sys0 * a.sB;
    const uint32_t bytesA = (uint32_t)(nvalid * a.sA * 8), bytesB = (uint32_t)(nvalid * a.sB * 8);
    double m[K][N], x[K];
    int pos[K];
    {
        uint32_t vo[K];
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            const int r = t + s * T;
            pos[s] = r < N ? r : -1;
            vo[s] = (g < nvalid && r < N) ? (uint32_t)(((uint32_t)g * (uint32_t)a.sA + r) * 8) : kOutOfRange;
        });
        static_for<0, N>(LUPP_SF(jc) {
            constexpr int j = decltype(jc)::value;
            const auto rc = make_rsrc(baseA + j * a.lda, bytesA);
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                m[s][j] = buf_load_f64(rc, vo[s], 0);
            });
        });
        const auto rB = make_rsrc(baseB, bytesB);
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            const int r = t + s * T;
            x[s] = buf_load_f64(rB, (g < nvalid && r < N) ? (uint32_t)(((uint32_t)g * (uint32_t)a.sB + r) * 8) : kOutOfRange, 0);
        });
    }

    double *rec = lds + (wave * SPW + g) * seg_lds<N>::kStride;
    const int inf = seg_getrf_solve<N, T, F, Sh::CH, Sh::PF>(m, x, pos, rec);

    settle(lane);
    set_geometry();
    rec = lds + (wave * SPW + g) * seg_lds<N>::kStride;
    baseA = opaque_ptr(baseA);
    baseB = opaque_ptr(baseB);
    const bool active = g < nvalid;
    if (factors) {
        uint32_t vo[K];
        /* slot s holds row pos[s] of the LAPACK-ordered factors */
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            vo[s] = (active && pos[s] >= 0) ? (uint32_t)(((uint32_t)g * (uint32_t)a.sA + pos[s]) * 8) : kOutOfRange;
        });
        static_for<0, N>(LUPP_SF(jc) {
            constexpr int j = decltype(jc)::value;
            const auto rc = make_rsrc(baseA + j * a.lda, bytesA);
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                buf_store_f64(rc, vo[s], 0, m[s][j]);
            });
        });
    }
    const int *ipl = reinterpret_cast<const int *>(rec + seg_lds<N>::kPos);
    const auto rBs = make_rsrc(baseB, bytesB);
    const auto rP = make_rsrc(a.ipiv + sys0 * N, (uint32_t)(nvalid * N * 4));
    static_for<0, K>(LUPP_SF(sc) {
        constexpr int s = decltype(sc)::value;
        const int r = t + s * T;
        const bool ok = active && r < N;
        const int rr = r < N ? r : 0;
        buf_store_f64(rBs, ok && inf == 0 ? (uint32_t)(((uint32_t)g * (uint32_t)a.sB + r) * 8) : kOutOfRange, 0, rec[rr]);
        buf_store_i32(rP, ok ? (uint32_t)((g * N + r) * 4) : kOutOfRange, 0, ipl[rr] + 1);
    });
    const auto rI = make_rsrc(a.info + sys0, (uint32_t)nvalid * 4u);
    buf_store_i32(rI, (active && t == 0) ? (uint32_t)g * 4u : kOutOfRange, 0, inf);
}

}  // namespace lupp

#endif
