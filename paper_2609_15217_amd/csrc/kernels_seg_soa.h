/* Lanes-per-system batched solve in strict and FMA arithmetic for the
 * interleaved (SoA) layout: the staging of kernels_lanes_soa.h (a workgroup
 * moves the matrices of 16 consecutive systems through LDS in whole 128-byte
 * lines) around the solver of lupp_segments.h. Measured against the
 * ds_bpermute solver in the same staging (200000 systems, solution only, us):
 * n = 16 with 8 lanes 160 -> 129, n = 24 539 -> 391 (8 lanes against 16),
 * n = 32 with 16 lanes 872 -> 737. One workgroup holds 16/(64/T) waves, whose
 * solver records reuse the staging tile.
 * Other numbers of systems per workgroup: see seg_soa_systems (32) and
 * seg_soa_by_8. */
#ifndef LUPP_KERNELS_SEG_SOA_H
#define LUPP_KERNELS_SEG_SOA_H

#include "kernels_lanes_soa.h"
#include "kernels_seg.h"

namespace lupp {

/* Systems per workgroup. Writing the factors is bound by memory, and 256
 * contiguous bytes per element instead of 128 are written faster, above all
 * where ldbatch is no multiple of 16, so that every row starts inside a line,
 * or a power of two. Measured with 8 lanes, 16 -> 32 systems, us, at 2^20
 * systems with ldbatch 2^20 + 192, 300007 dense and 2^19 dense: n = 14:
 * 781 -> 731, 273 -> 238, 428 -> 384; n = 16: 1031 -> 935, 356 -> 308,
 * 553 -> 487; n = 18: 1341 -> 1341, 424 -> 403, 737 -> 686; n = 20:
 * 1585 -> 1596, 526 -> 482, 903 -> 827. The line lies where that no longer
 * holds for all of them: n = 17 (24 staged rows of 17): 1220 -> 1248,
 * 380 -> 376, 684 -> 641; n = 22: 2020 -> 2136, 633 -> 647, 1142 -> 1117;
 * n = 24: 2308 -> 2388, 764 -> 741, 1344 -> 1271; n = 13 and less did not
 * change (249 -> 247). Without the factors the larger workgroup only waits
 * longer at its barriers (n = 24: 1945 -> 2055 and 586 -> 618), and with 16
 * lanes its eight waves would be the only ones of a compute unit. */
template <int N, int T>
constexpr int seg_soa_systems(bool factors)
{
    return factors && T == 8 && N >= 14 && N <= 20 && N != 17 ? 32 : 16;
}

template <int N, int T, bool F, int SYS>
__global__ void __launch_bounds__((soa_shape<N, T, SYS>::NT))
    __attribute__((amdgpu_waves_per_eu(seg_shape<N, T>::W, seg_shape<N, T>::W)))
    k_seg_soa(SolveArgs a, int factors)
{
    using Sh = soa_shape<N, T, SYS>;
    constexpr int S = Sh::S, K = Sh::K, NP = Sh::NP, CJ = Sh::CJ, NCH = Sh::NCH;
    constexpr int QB = NP / T; /* cooperative accesses per column and thread */
    /* the staging tile; between the staging phases each wave's share holds its
     * segments' solver records */
    constexpr int SEG = seg_lds<N>::kStride;
    constexpr int TILE = CJ * NP * S > S * SEG ? CJ * NP * S : S * SEG;
    __shared__ __align__(16) double tile[TILE];
    __shared__ double xb[NP * S];
    __shared__ int ipl[NP * S];
    __shared__ int infl[S];

    int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t sys0 = (int64_t)xcd_block(blockIdx.x, gridDim.x) * S;
    const int64_t rem = a.batch - sys0;
    const int nvalid = (int)(rem < S ? rem : S);

    /* Lane geometry, all derived from tid (rebuilt after the solve from a
     * fenced copy of tid, so that none of it stays live across the solve):
     * lane side: segment g, lane t of the segment, system yl, rows t + s*T;
     * cooperative side: system yw, rows ci0 + multiples of T. */
    int g, t, yl, yw, ci0;
    auto set_geometry = [&]() __attribute__((always_inline)) {
        const int lane = tid & 63;
        g = lane / T;
        t = lane % T;
        yl = wave * Sh::SPW + g;
        yw = tid & (S - 1);
        ci0 = tid >> Sh::LOG_S;
    };
    set_geometry();

    /* The cooperative rows of a wave are ci0 = cw .. cw + 64/S - 1, so each
     * descriptor is based at the wave's first row (a uniform address) and
     * its extent spans 64/S rows: the per-lane offsets stay below 2^31
     * bytes for any ldbatch under 2^31 / (8 * (64/S - 1) + 8). */
    const int cw = (wave * 64) >> Sh::LOG_S;
    double *baseA = a.A + sys0 + (int64_t)cw * a.sA;
    double *baseB = a.b + sys0 + (int64_t)cw * a.sB;
    const int64_t colA = a.lda * a.sA;
    constexpr int RW = 64 / S; /* cooperative rows per wave */
    const uint32_t bytesA = (uint32_t)(((int64_t)(RW - 1) * a.sA + nvalid) * 8);
    const uint32_t bytesB = (uint32_t)(((int64_t)(RW - 1) * a.sB + nvalid) * 8);
    auto coop_off = [&](int64_t ld, int w) __attribute__((always_inline)) {
        return yw < nvalid ? (uint32_t)(((int64_t)(ci0 - cw) * ld + yw) * w) : kOutOfRange;
    };
    uint32_t vA = coop_off(a.sA, 8), vB = coop_off(a.sB, 8);
    /* per-lane offset of the cooperative row ci0 + ib (out of range for rows past n) */
    auto rowv = [&](uint32_t v, int ib) -> uint32_t {
        return (ib + T <= N || ci0 < N - ib) ? v : kOutOfRange;
    };
    /* LDS index of the cooperative element (chunk column c, row block ib) */
    auto cidx = [&](int c, int ib) { const int i = ci0 + ib; return (c * NP + i) * S + (yw ^ soa_sw<N, T, SYS>(i)); };
    /* LDS index of a lane-side element (chunk column c, row i) */
    auto lidx = [&](int c, int i) { return (c * NP + i) * S + (yl ^ soa_sw<N, T, SYS>(i)); };

    /* ---------------------------------------------------------- load */
    double m[K][N];
    double x[K];
    int pos[K];
    static_for<0, K>(LUPP_SF(sc) {
        constexpr int s = decltype(sc)::value;
        pos[s] = t + s * T < N ? t + s * T : -1;
    });
    /* the loads of column chunk c + LA are issued before chunk c is
     * transposed, so LA + 1 chunks are in flight per wave while the staging
     * registers of a chunk die as its matrix registers fill (the whole
     * matrix in flight would hold 2*n*n/T extra VGPRs: a wave per SIMD) */
    double v[N * QB];
    double vb[QB];
    auto load_chunk = [&](auto chc) __attribute__((always_inline)) {
        constexpr int ch = decltype(chc)::value;
        if constexpr (ch < NCH) {
            constexpr int j0 = ch * CJ;
            constexpr int cj = (j0 + CJ <= N) ? CJ : N - j0;
            static_for<j0 * QB, (j0 + cj) * QB>(LUPP_SF(qc) {
                constexpr int q = decltype(qc)::value;
                constexpr int j = q / QB, ib = (q % QB) * T;
                const auto rc = make_rsrc(baseA + (int64_t)j * colA + (int64_t)ib * a.sA, bytesA);
                v[q] = buf_load_f64(rc, rowv(vA, ib), 0);
            });
        }
    };
    static_for<0, Sh::LA>(load_chunk);
    {
        static_for<0, QB>(LUPP_SF(qc) {
            constexpr int ib = decltype(qc)::value * T;
            vb[decltype(qc)::value] =
                buf_load_f64(make_rsrc(baseB + (int64_t)ib * a.sB, bytesB), rowv(vB, ib), 0);
        });
    }
    static_for<0, NCH>(LUPP_SF(chc) {
        constexpr int ch = decltype(chc)::value;
        load_chunk(std::integral_constant<int, ch + Sh::LA>{});
        constexpr int j0 = ch * CJ;
        constexpr int cj = (j0 + CJ <= N) ? CJ : N - j0;
        static_for<0, cj * QB>(LUPP_SF(qc) {
            constexpr int q = decltype(qc)::value;
            tile[cidx(q / QB, (q % QB) * T)] = v[j0 * QB + q];
        });
        if constexpr (ch == NCH - 1) {
            static_for<0, QB>(LUPP_SF(qc) {
                constexpr int q = decltype(qc)::value;
                xb[cidx(0, q * T)] = vb[q];
            });
        }
        __syncthreads();
        static_for<0, cj>(LUPP_SF(cc) {
            constexpr int c = decltype(cc)::value;
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                m[s][j0 + c] = tile[lidx(c, t + s * T)];
            });
        });
        if constexpr (ch == NCH - 1) {
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                x[s] = xb[lidx(0, t + s * T)];
            });
        }
        __syncthreads();
    });

    /* ---------------------------------------------------------- solve */
    const int inf = seg_getrf_solve<N, T, F, seg_shape<N, T>::CH, seg_shape<N, T>::PF>(m, x, pos, tile + yl * SEG);

    /* ---------------------------------------------------------- store */
    baseA = opaque_ptr(baseA);
    baseB = opaque_ptr(baseB);
    const int64_t sAs = opaque_i64(a.sA), sBs = opaque_i64(a.sB);
    settle(tid);
    set_geometry();
    vA = coop_off(sAs, 8);
    vB = coop_off(sBs, 8);
    {
        const double *rec = tile + yl * SEG;
        const int *seq = reinterpret_cast<const int *>(rec + seg_lds<N>::kPos);
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            const int r = t + s * T;
            if (r < N) {
                xb[lidx(0, r)] = rec[r];
                ipl[lidx(0, r)] = seq[r] + 1;
            }
        });
        if (t == 0) infl[yl] = inf;
    }
    __syncthreads(); /* every record is read before the tile is staged again */
    if (factors) {
        static_for<0, NCH>(LUPP_SF(chc) {
            constexpr int j0 = decltype(chc)::value * CJ;
            constexpr int cj = (j0 + CJ <= N) ? CJ : N - j0;
            /* slot s holds row pos[s] of the LAPACK-ordered factors */
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                if (pos[s] >= 0) {
                    static_for<0, cj>(LUPP_SF(cc) {
                        constexpr int c = decltype(cc)::value;
                        tile[lidx(c, pos[s])] = m[s][j0 + c];
                    });
                }
            });
            __syncthreads();
            static_for<0, cj * QB>(LUPP_SF(qc) {
                constexpr int q = decltype(qc)::value;
                constexpr int c = q / QB, ib = (q % QB) * T;
                const auto rc = make_rsrc(baseA + (int64_t)(j0 + c) * colA + (int64_t)ib * sAs, bytesA);
                buf_store_f64(rc, rowv(vA, ib), 0, tile[cidx(c, ib)]);
            });
            __syncthreads();
        });
    }
    {
        const bool ok = infl[yw] == 0;
        int32_t *baseP = a.ipiv + sys0 + (int64_t)cw * sAs;
        const uint32_t bytesP = (uint32_t)(((int64_t)(RW - 1) * sAs + nvalid) * 4);
        const uint32_t vP = coop_off(sAs, 4);
        static_for<0, QB>(LUPP_SF(qc) {
            constexpr int ib = decltype(qc)::value * T;
            buf_store_f64(make_rsrc(baseB + (int64_t)ib * sBs, bytesB), ok ? rowv(vB, ib) : kOutOfRange,
                          0, xb[cidx(0, ib)]);
            buf_store_i32(make_rsrc(baseP + (int64_t)ib * sAs, bytesP), rowv(vP, ib), 0,
                          ipl[cidx(0, ib)]);
        });
        const auto ri = make_rsrc(a.info + sys0, (uint32_t)nvalid * 4u);
        if (tid < S) buf_store_i32(ri, (uint32_t)tid * 4u, 0, infl[tid]);
    }
}

template <int N, int T, int SYS>
hipError_t launch_seg_soa(const SolveArgs &a, bool factors, hipStream_t st)
{
    using Sh = soa_shape<N, T, SYS>;
    const dim3 grid((unsigned)((a.batch + Sh::S - 1) / Sh::S));
    const dim3 block(Sh::NT);
    if (a.fma) hipLaunchKernelGGL((k_seg_soa<N, T, true, SYS>), grid, block, 0, st, a, (int)factors);
    else hipLaunchKernelGGL((k_seg_soa<N, T, false, SYS>), grid, block, 0, st, a, (int)factors);
    return hipGetLastError();
}

/* Whether an interleaved batch with 16 or 32 lanes runs 8 systems per
 * workgroup. A small batch is bound by the steps' chain and by the row writes
 * of one compute unit's LDS, which all its waves share: half the waves per
 * workgroup spread better over the 256 compute units. Each line is then read
 * by two workgroups, neighbours on one XCD, the second time from its L2.
 * Measured, us, 16 -> 8 systems, solution only (with the factors alike):
 * 32 lanes, 1000 / 4096 / 5003 / 10000 / 30000 systems: n = 21: 20.9 -> 15.8,
 * 20.4 -> 20.2, 29.8 -> 26.2, 36.0 -> 31.8, 77 -> 71; n = 32: 33.2 -> 23.2,
 * 32.5 -> 32.7, 52.5 -> 44.6, 68 -> 58, 155 -> 140. 16 lanes: n = 21:
 * 21.4 -> 17.8, 22.1 -> 22.9, 30.2 -> 27.9, 34.7 -> 31.9, 70 -> 68; n = 32:
 * 34.3 -> 28.3, 34.9 -> 38.4, 53.5 -> 48.6, 63 -> 58, 136 -> 133, and 16000
 * systems 81 -> 87: with 16 lanes only where the busiest compute unit gets an
 * eighth fewer systems. From 32768 systems on the dispatcher has other
 * entries. The strides must keep a wave's 8 rows within 2^31 bytes (16
 * systems: 4 rows). */
template <int T>
bool seg_soa_by_8(const SolveArgs &a)
{
    constexpr int64_t kCUs = 256, kSmall = 32768, kSpan = (int64_t)1 << 31;
    if (a.batch >= kSmall || (7 * a.sA + 8) * 8 >= kSpan || (7 * a.sB + 8) * 8 >= kSpan) return false;
    if (T == 32) return true;
    auto busiest = [&](int64_t s) { return ((a.batch + s - 1) / s + kCUs - 1) / kCUs * s; };
    return busiest(8) * 8 <= busiest(16) * 7;
}

/* kSoa: whether the interleaved kernels are built too */
template <int N, int T, bool kSoa = true>
hipError_t launch_seg(const SolveArgs &a, int layout, bool factors, int wpb, hipStream_t st)
{
    if (layout == LUPP_SOA) {
        if constexpr (kSoa) {
            if constexpr (T >= 16)
                if (seg_soa_by_8<T>(a)) return launch_seg_soa<N, T, 8>(a, factors, st);
            return factors ? launch_seg_soa<N, T, seg_soa_systems<N, T>(true)>(a, factors, st)
                           : launch_seg_soa<N, T, seg_soa_systems<N, T>(false)>(a, factors, st);
        } else {
            return hipErrorNotSupported;
        }
    }
    const int w = wpb > 0 ? wpb : 4;
    const int64_t per_block = (int64_t)w * (64 / T);
    const dim3 grid((unsigned)((a.batch + per_block - 1) / per_block));
    const dim3 block(64 * w);
    if (a.fma) hipLaunchKernelGGL((k_seg<N, T, true>), grid, block, 0, st, a, (int)factors);
    else hipLaunchKernelGGL((k_seg<N, T, false>), grid, block, 0, st, a, (int)factors);
    return hipGetLastError();
}

}  // namespace lupp

#endif
