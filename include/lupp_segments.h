/* Lanes-per-system LU with partial pivoting through LDS, HIP for gfx950
 * (CDNA4, wave64): T lanes of a wave (a "segment") share one system, as
 * lanes_getrf_solve of lupp_device.h does, with the same arithmetic contract
 * (Section 2.2; Section 3.2, several rows per thread), so the results are the
 * same bits. What differs is how the lanes cooperate.
 *
 * What bounds a solve of this kind on gfx950 is instruction issue, not
 * arithmetic: at n = 32 only 2100 of the 7400 vector instructions per wave of
 * the ds_bpermute form were multiplies and subtracts of the elimination; the
 * rest chose the pivot, gathered the pivot row and kept the positions, and
 * its two ds_bpermute per broadcast double kept LDS busy half of the time.
 * This form issues 4414 (counted with the factors written):
 *
 *   - The wave's candidates and owners are 64-bit wave masks in SGPRs, kept
 *     by scalar instructions, one mask per row slot. Masked work runs under
 *     `s_mov_b64 exec, mask` in short asm blocks: no compares or selects per
 *     step, and none of the branches of divergent regions.
 *   - The pivot search compares the high 32 bits of |a_rk| (v_max_i32 with
 *     DPP: one instruction per level instead of five for doubles). Only if two
 *     candidates of a segment share the largest high word does a second
 *     search over the low words, then the positions, decide. A finite |x| as
 *     an integer orders as the number does, so the choice is the exact one.
 *   - Two elimination steps share one broadcast: after step k only the next
 *     column is updated, then step k + 1 finds its pivot, and both pivot rows
 *     go to the segment's LDS record with one masked write per row slot.
 *     Every lane reads both rows (same address for all lanes of a segment: a
 *     conflict-free ds_read_b128), applies step k to row k + 1 itself (one
 *     multiply-subtract per column) and updates its rows with both. Every
 *     element still receives the same rounded operations in the same order.
 *   - Divisions by one pivot share its reciprocal (two Newton-Raphson steps
 *     from v_rcp_f64); the quotient is then corrected with its exact residual
 *     (Markstein's method, as in the correctly rounded division the compiler
 *     emits, whose scaling steps do nothing in the range checked for). A zero
 *     numerator has the exact quotient q = +-0 and residual 0. A wave with
 *     another pivot or numerator outside 2^-400 .. 2^400 takes true divisions
 *     instead.
 *
 * Measured (262144 systems of N(0, 1) entries, packed, strict mode, us, solution
 * only / with factors; the ds_bpermute form -> this one): n = 32: 1187 / 1264 ->
 * 850 / 932; n = 24: 703 / 704 -> 518 / 541 (16 lanes), 456 / 582 (8 lanes). At
 * n = 32 (solution only, 2^20 systems) the vector units are busy 58% of the
 * time and LDS 54%; a wave spends 24% of its life waiting to issue an LDS
 * instruction.
 *
 * LDS traffic decides the shape of the broadcast: a masked ds_write_b128 costs
 * 13.7 cycles of the CU's LDS whatever the number of active lanes, a
 * broadcast ds_read_b128 4.1, a ds_bpermute_b32 6 (measured).
 */
#ifndef LUPP_SEGMENTS_H
#define LUPP_SEGMENTS_H

#include "lupp_device.h"

namespace lupp {

/* LDS of one segment, in doubles: two pivot rows of kRow entries (n columns
 * and the right-hand side; even, so that pairs are 16-byte aligned), then
 * the n int32 positions (with room to spare). The stride is an odd number of
 * 16-byte units: the segments of a wave then read from different banks. */
template <int N>
struct seg_lds {
    static constexpr int kRow = (N + 2) & ~1;
    static constexpr int kPos = 2 * kRow;
    static constexpr int kMin = (kPos + (N + 2) / 2 + 1) & ~1;
    static constexpr int kStride = (kMin / 2) % 2 == 1 ? kMin : kMin + 2;
};

typedef double seg_pair __attribute__((ext_vector_type(2)));

/* Orders the wave's LDS accesses in the compiler (LDS serves one wave's
 * accesses in order, so no instruction is needed). */
__device__ __forceinline__ void seg_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__device__ __forceinline__ int seg_hi_abs(double v)
{
    return __builtin_bit_cast(int2, v).y & 0x7fffffff;
}

__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

__device__ __forceinline__ unsigned lds_addr(const void *p)
{
    return (unsigned)(size_t)(const __attribute__((address_space(3))) void *)p;
}

/* Maximum over aligned groups of 2^(L+1) lanes given the maxima over groups
 * of 2^L (the exchange patterns of pair_u32). */
template <int L>
__device__ __forceinline__ int seg_max_round(int v)
{
    if constexpr (L == 0) return max(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));
    else if constexpr (L == 1) return max(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));
    else if constexpr (L == 2) return max(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));
    else if constexpr (L == 3) return max(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true));
    else {
        auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        return max((int)r[0], (int)r[1]);
    }
}

template <int T>
__device__ __forceinline__ int seg_max(int v)
{
    if constexpr (T > 1) v = seg_max_round<0>(v);
    if constexpr (T > 2) v = seg_max_round<1>(v);
    if constexpr (T > 4) v = seg_max_round<2>(v);
    if constexpr (T > 8) v = seg_max_round<3>(v);
    if constexpr (T > 16) v = seg_max_round<4>(v);
    return v;
}

/* x, z, p = m ? (xs, zs, ps) : (x, z, p) per lane, by a wave mask (asm: the
 * compiler would turn a chain of selects between register-array elements into
 * an indexed scratch access). A vector instruction may read a mask that a
 * vector compare has written only two wait states later, and the compiler's
 * hazard pass does not look inside asm: hence the s_nop. */
__device__ __forceinline__ void mask_select(uint64_t m, double &x, double xs, double &z, double zs,
                                            int &p, int ps)
{
    int2 u = __builtin_bit_cast(int2, x), v = __builtin_bit_cast(int2, z);
    const int2 us = __builtin_bit_cast(int2, xs), vs = __builtin_bit_cast(int2, zs);
    asm("s_nop 1\n\t"
        "v_cndmask_b32_e64 %0, %0, %5, %10\n\tv_cndmask_b32_e64 %1, %1, %6, %10\n\t"
        "v_cndmask_b32_e64 %2, %2, %7, %10\n\tv_cndmask_b32_e64 %3, %3, %8, %10\n\t"
        "v_cndmask_b32_e64 %4, %4, %9, %10"
        : "+&v"(u.x), "+&v"(u.y), "+&v"(v.x), "+&v"(v.y), "+&v"(p)
        : "v"(us.x), "v"(us.y), "v"(vs.x), "v"(vs.y), "v"(ps), "s"(m));
    x = __builtin_bit_cast(double, u);
    z = __builtin_bit_cast(double, v);
}

/* Masked blocks: the wave enters with every lane active, works in the lanes of
 * m, and leaves with every lane active again. volatile keeps them in program
 * order, which also bounds the registers in flight. */
#define LUPP_IN "s_mov_b64 exec, %[m]\n\t"
#define LUPP_OUT "s_mov_b64 exec, -1"
#define LUPP_MUL_SUB(i) \
    "v_mul_f64 %[t], %[l], %[u" #i "]\n\tv_add_f64 %[a" #i "], %[a" #i "], -%[t]\n\t"
#define LUPP_FMA_SUB(i) "v_fma_f64 %[a" #i "], -%[l], %[u" #i "], %[a" #i "]\n\t"
#define LUPP_RW(i) [a##i] "+v"(a[i])
#define LUPP_RD(i) [u##i] "v"(u[i])

/* a[i] = a[i] - l * u[i] for i < C, in the lanes of m */
template <bool kFMA, int C>
__device__ __forceinline__ void masked_msub(uint64_t m, double l, double *a, const double *u)
{
    double t;
    if constexpr (C == 1) {
        if constexpr (kFMA)
            asm volatile(LUPP_IN LUPP_FMA_SUB(0) LUPP_OUT
                         : LUPP_RW(0) : [l] "v"(l), LUPP_RD(0), [m] "s"(m));
        else
            asm volatile(LUPP_IN LUPP_MUL_SUB(0) LUPP_OUT
                         : LUPP_RW(0), [t] "=&v"(t) : [l] "v"(l), LUPP_RD(0), [m] "s"(m));
    } else if constexpr (C == 2) {
        if constexpr (kFMA)
            asm volatile(LUPP_IN LUPP_FMA_SUB(0) LUPP_FMA_SUB(1) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1)
                         : [l] "v"(l), LUPP_RD(0), LUPP_RD(1), [m] "s"(m));
        else
            asm volatile(LUPP_IN LUPP_MUL_SUB(0) LUPP_MUL_SUB(1) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1), [t] "=&v"(t)
                         : [l] "v"(l), LUPP_RD(0), LUPP_RD(1), [m] "s"(m));
    } else if constexpr (C == 4) {
        if constexpr (kFMA)
            asm volatile(LUPP_IN LUPP_FMA_SUB(0) LUPP_FMA_SUB(1) LUPP_FMA_SUB(2) LUPP_FMA_SUB(3) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1), LUPP_RW(2), LUPP_RW(3)
                         : [l] "v"(l), LUPP_RD(0), LUPP_RD(1), LUPP_RD(2), LUPP_RD(3), [m] "s"(m));
        else
            asm volatile(LUPP_IN LUPP_MUL_SUB(0) LUPP_MUL_SUB(1) LUPP_MUL_SUB(2) LUPP_MUL_SUB(3) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1), LUPP_RW(2), LUPP_RW(3), [t] "=&v"(t)
                         : [l] "v"(l), LUPP_RD(0), LUPP_RD(1), LUPP_RD(2), LUPP_RD(3), [m] "s"(m));
    } else if constexpr (C > 0) {
        constexpr int H = C > 4 ? 4 : 2;
        masked_msub<kFMA, H>(m, l, a, u);
        masked_msub<kFMA, C - H>(m, l, a + H, u + H);
    }
}

/* Both steps of a pair: a[i] -= l0 * u0[i] in the lanes of m0, then
 * a[i] -= l1 * u1[i] in the lanes of m1, in one block (one change of the
 * execution mask less than two blocks) */
#define LUPP_MUL_SUB1(i) \
    "v_mul_f64 %[t], %[h], %[w" #i "]\n\tv_add_f64 %[a" #i "], %[a" #i "], -%[t]\n\t"
#define LUPP_FMA_SUB1(i) "v_fma_f64 %[a" #i "], -%[h], %[w" #i "], %[a" #i "]\n\t"
#define LUPP_IN1 "s_mov_b64 exec, %[n]\n\t"
#define LUPP_RD1(i) [w##i] "v"(w[i])
template <bool kFMA, int C>
__device__ __forceinline__ void masked_msub2(uint64_t m, double l, const double *u, uint64_t n,
                                             double h, const double *w, double *a)
{
    double t;
    if constexpr (C == 1) {
        if constexpr (kFMA)
            asm volatile(LUPP_IN LUPP_FMA_SUB(0) LUPP_IN1 LUPP_FMA_SUB1(0) LUPP_OUT
                         : LUPP_RW(0)
                         : [l] "v"(l), [h] "v"(h), LUPP_RD(0), LUPP_RD1(0), [m] "s"(m), [n] "s"(n));
        else
            asm volatile(LUPP_IN LUPP_MUL_SUB(0) LUPP_IN1 LUPP_MUL_SUB1(0) LUPP_OUT
                         : LUPP_RW(0), [t] "=&v"(t)
                         : [l] "v"(l), [h] "v"(h), LUPP_RD(0), LUPP_RD1(0), [m] "s"(m), [n] "s"(n));
    } else if constexpr (C == 2) {
        if constexpr (kFMA)
            asm volatile(LUPP_IN LUPP_FMA_SUB(0) LUPP_FMA_SUB(1) LUPP_IN1 LUPP_FMA_SUB1(0) LUPP_FMA_SUB1(1) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1)
                         : [l] "v"(l), [h] "v"(h), LUPP_RD(0), LUPP_RD(1), LUPP_RD1(0), LUPP_RD1(1),
                           [m] "s"(m), [n] "s"(n));
        else
            asm volatile(LUPP_IN LUPP_MUL_SUB(0) LUPP_MUL_SUB(1) LUPP_IN1 LUPP_MUL_SUB1(0) LUPP_MUL_SUB1(1) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1), [t] "=&v"(t)
                         : [l] "v"(l), [h] "v"(h), LUPP_RD(0), LUPP_RD(1), LUPP_RD1(0), LUPP_RD1(1),
                           [m] "s"(m), [n] "s"(n));
    } else if constexpr (C == 4) {
        if constexpr (kFMA)
            asm volatile(LUPP_IN LUPP_FMA_SUB(0) LUPP_FMA_SUB(1) LUPP_FMA_SUB(2) LUPP_FMA_SUB(3)
                         LUPP_IN1 LUPP_FMA_SUB1(0) LUPP_FMA_SUB1(1) LUPP_FMA_SUB1(2) LUPP_FMA_SUB1(3) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1), LUPP_RW(2), LUPP_RW(3)
                         : [l] "v"(l), [h] "v"(h), LUPP_RD(0), LUPP_RD(1), LUPP_RD(2), LUPP_RD(3),
                           LUPP_RD1(0), LUPP_RD1(1), LUPP_RD1(2), LUPP_RD1(3), [m] "s"(m), [n] "s"(n));
        else
            asm volatile(LUPP_IN LUPP_MUL_SUB(0) LUPP_MUL_SUB(1) LUPP_MUL_SUB(2) LUPP_MUL_SUB(3)
                         LUPP_IN1 LUPP_MUL_SUB1(0) LUPP_MUL_SUB1(1) LUPP_MUL_SUB1(2) LUPP_MUL_SUB1(3) LUPP_OUT
                         : LUPP_RW(0), LUPP_RW(1), LUPP_RW(2), LUPP_RW(3), [t] "=&v"(t)
                         : [l] "v"(l), [h] "v"(h), LUPP_RD(0), LUPP_RD(1), LUPP_RD(2), LUPP_RD(3),
                           LUPP_RD1(0), LUPP_RD1(1), LUPP_RD1(2), LUPP_RD1(3), [m] "s"(m), [n] "s"(n));
    } else if constexpr (C > 0) {
        constexpr int H = C > 4 ? 4 : 2;
        masked_msub2<kFMA, H>(m, l, u, n, h, w, a);
        masked_msub2<kFMA, C - H>(m, l, u + H, n, h, w + H, a + H);
    }
}

/* d = fma(e, y, q), d = y, in the lanes of m */
__device__ __forceinline__ void masked_fma(uint64_t m, double &d, double e, double y, double q)
{
    asm volatile(LUPP_IN "v_fma_f64 %[d], %[e], %[y], %[q]\n\t" LUPP_OUT
                 : [d] "+v"(d) : [e] "v"(e), [y] "v"(y), [q] "v"(q), [m] "s"(m));
}

__device__ __forceinline__ void masked_mov(uint64_t m, double &d, double y)
{
    asm volatile(LUPP_IN "v_mov_b64 %[d], %[y]\n\t" LUPP_OUT : [d] "+v"(d) : [y] "v"(y), [m] "s"(m));
}

/* LDS writes in the lanes of m: doubles OFF, OFF + 1, ... from address p */
template <int OFF>
__device__ __forceinline__ void masked_put1(uint64_t m, unsigned p, double x)
{
    asm volatile(LUPP_IN "ds_write_b64 %[p], %[x] offset:%[o]\n\t" LUPP_OUT
                 :: [p] "v"(p), [x] "v"(x), [m] "s"(m), [o] "n"(8 * OFF) : "memory");
}

template <int OFF>
__device__ __forceinline__ void masked_put2(uint64_t m, unsigned p, double x, double y)
{
    asm volatile(LUPP_IN "ds_write2_b64 %[p], %[x], %[y] offset0:%[o0] offset1:%[o1]\n\t" LUPP_OUT
                 :: [p] "v"(p), [x] "v"(x), [y] "v"(y), [m] "s"(m), [o0] "n"(OFF), [o1] "n"(OFF + 1)
                 : "memory");
}

template <int OFF>
__device__ __forceinline__ void masked_put4(uint64_t m, unsigned p, double x, double y, double z,
                                            double w)
{
    asm volatile(LUPP_IN "ds_write2_b64 %[p], %[x], %[y] offset0:%[o0] offset1:%[o1]\n\t"
                 "ds_write2_b64 %[p], %[z], %[w] offset0:%[o2] offset1:%[o3]\n\t" LUPP_OUT
                 :: [p] "v"(p), [x] "v"(x), [y] "v"(y), [z] "v"(z), [w] "v"(w), [m] "s"(m),
                    [o0] "n"(OFF), [o1] "n"(OFF + 1), [o2] "n"(OFF + 2), [o3] "n"(OFF + 3)
                 : "memory");
}

template <int OFF>
__device__ __forceinline__ void masked_put8(uint64_t m, unsigned p, double x0, double x1, double x2,
                                            double x3, double x4, double x5, double x6, double x7)
{
    asm volatile(LUPP_IN "ds_write2_b64 %[p], %[x0], %[x1] offset0:%[o0] offset1:%[o1]\n\t"
                 "ds_write2_b64 %[p], %[x2], %[x3] offset0:%[o2] offset1:%[o3]\n\t"
                 "ds_write2_b64 %[p], %[x4], %[x5] offset0:%[o4] offset1:%[o5]\n\t"
                 "ds_write2_b64 %[p], %[x6], %[x7] offset0:%[o6] offset1:%[o7]\n\t" LUPP_OUT
                 :: [p] "v"(p), [x0] "v"(x0), [x1] "v"(x1), [x2] "v"(x2), [x3] "v"(x3), [x4] "v"(x4),
                    [x5] "v"(x5), [x6] "v"(x6), [x7] "v"(x7), [m] "s"(m), [o0] "n"(OFF),
                    [o1] "n"(OFF + 1), [o2] "n"(OFF + 2), [o3] "n"(OFF + 3), [o4] "n"(OFF + 4),
                    [o5] "n"(OFF + 5), [o6] "n"(OFF + 6), [o7] "n"(OFF + 7)
                 : "memory");
}

/* int32 at byte offset BYTE */
template <int BYTE>
__device__ __forceinline__ void masked_put_i32(uint64_t m, unsigned p, int x)
{
    asm volatile(LUPP_IN "ds_write_b32 %[p], %[x] offset:%[o]\n\t" LUPP_OUT
                 :: [p] "v"(p), [x] "v"(x), [m] "s"(m), [o] "n"(BYTE) : "memory");
}

/* Factor (and solve, on info == 0) the system of each segment of the wave.
 * a[s][j], b[s]: row t + s*T (t: lane of the segment), column j and right-hand
 * side; rec: the segment's seg_lds<N>::kStride doubles of LDS, 16-byte
 * aligned; pos[s]: the row index, or -1 for a phantom row. The whole wave
 * calls this with every lane active; lanes without a system hold zeros.
 * On return pos[s] is the row's position in the LAPACK-ordered factors (a[s]
 * holds that row), rec[r] the solution entry r (info == 0; all lanes of the
 * wave may read it), and the int32 at rec + kPos the interchange sequence,
 * 0-based. b is overwritten. CH: pivot-row columns fetched at a time, one
 * chunk ahead of its use where PF is set (2 x 4*CH or 1 x 4*CH VGPRs). */
template <int N, int T, bool kFMA, int CH, bool PF>
__device__ __forceinline__ int seg_getrf_solve(double (&a)[(N + T - 1) / T][N],
                                               double (&b)[(N + T - 1) / T],
                                               int (&pos)[(N + T - 1) / T], double *rec)
{
    constexpr int K = lanes_shape<N, T>::K, SPW = 64 / T;
    constexpr int RS = seg_lds<N>::kRow, IP = seg_lds<N>::kPos * 8;
    constexpr int LO = (1023 - 400) << 20, HI = (1023 + 400) << 20;
    static_assert(CH % 2 == 0, "chunks start at even columns");
    const unsigned rp = lds_addr(rec);
    const int *ipl = reinterpret_cast<const int *>(rec + seg_lds<N>::kPos);
    int info = 0;
    uint64_t cand[K], odd = 0; /* odd: lanes that saw a value out of range */
    double ry[K];              /* reciprocal of the row's pivot */
    static_for<0, K>(LUPP_SF(sc) {
        constexpr int s = decltype(sc)::value;
        cand[s] = __ballot(pos[s] >= 0);
        ry[s] = 0.0;
    });

    /* pivot of column k: hit[s] = the lanes whose slot s is the pivot row,
     * taken out of the candidates; key: high words, M: their maximum. A NaN (a
     * finite matrix may overflow into one) has the largest key and is found
     * first; with has_nan it is the pivot if it is the row at position k and
     * passed over otherwise, as in a scan for a larger magnitude. */
    auto search = [&](auto kc, int (&key)[K], int &M, uint64_t (&hit)[K], auto has_nan) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        int lm = -1;
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            int c = seg_hi_abs(a[s][k]);
            if constexpr (decltype(has_nan)::value) {
                const bool is = a[s][k] != a[s][k];
                c = is ? (pos[s] == k ? 0x7fffffff : -1) : c;
            }
            key[s] = in_mask(cand[s]) ? c : -1;
            lm = s == 0 ? key[0] : max(lm, key[s]);
        });
        M = seg_max<T>(lm);
        int nhit = 0;
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            hit[s] = __ballot(key[s] == M);
            nhit += __builtin_popcountll(hit[s]);
        });
        /* every segment has a candidate, so SPW hits are one per segment */
        if (__builtin_expect(nhit != SPW, 0)) {
            int lv[K], l = 0, pm = 0;
            bool h[K];
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                /* the low word, ordered as a signed integer */
                lv[s] = (int)((unsigned)__builtin_bit_cast(int2, a[s][k]).x ^ 0x80000000u);
                h[s] = key[s] == M;
                const int c = h[s] ? lv[s] : (int)0x80000000;
                l = s == 0 ? c : max(l, c);
            });
            const int L = seg_max<T>(l);
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                h[s] = h[s] & (lv[s] == L);
                const int c = h[s] ? 64 - pos[s] : 0;
                pm = s == 0 ? c : max(pm, c);
            });
            const int P = seg_max<T>(pm);
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                hit[s] = __ballot(h[s] & (64 - pos[s] == P));
            });
        }
        static_for<0, K>(LUPP_SF(sc) { cand[decltype(sc)::value] &= ~hit[decltype(sc)::value]; });
    };
    /* positions after step k, its pivot row found at position q: finished rows
     * are marked 64 + their final position */
    auto place = [&](auto kc, const uint64_t (&hit)[K], int q) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            pos[s] = in_mask(hit[s]) ? 64 + k : (pos[s] == k ? q : pos[s]);
            settle(pos[s]);
        });
    };
    /* takes back search and place of step k */
    auto unplace = [&](auto kc, const uint64_t (&hit)[K], int q) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            pos[s] = in_mask(hit[s]) ? q : (pos[s] == q ? k : pos[s]);
            cand[s] |= hit[s];
        });
    };
    /* the lanes whose pivot pv (as found, a NaN before any number) is zero;
     * again(): takes the step back, searches with has_nan and does it anew */
    auto check_pivot = [&](auto kc, const double &pv, auto again) __attribute__((always_inline)) -> uint64_t {
        constexpr int k = decltype(kc)::value;
        uint64_t z = __ballot(__builtin_amdgcn_class(pv, 0x63)); /* zeros and NaN */
        if (__builtin_expect(z != 0, 0)) {
            if (__ballot(pv != pv) != 0) again();
            z = __ballot(pv == 0.0);
            info = (pv == 0.0 && info == 0) ? k + 1 : info;
        }
        settle(info);
        return z;
    };
    auto reciprocal = [](double v) __attribute__((always_inline)) -> double {
        double y = __builtin_amdgcn_rcp(v);
        y = __builtin_fma(__builtin_fma(-v, y, 1.0), y, y);
        return __builtin_fma(__builtin_fma(-v, y, 1.0), y, y);
    };
    /* multipliers: a[s][k] = a[s][k] / pv, correctly rounded, in the lanes m[s];
     * the pivot rows keep the reciprocal for the back substitution */
    auto scale = [&](auto kc, const int (&key)[K], int M, const uint64_t (&m)[K],
                     const uint64_t (&hit)[K], double pv) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        const uint64_t big = __ballot(M > HI);
        uint64_t bad = big;
        static_for<0, K>(LUPP_SF(sc) {
            bad |= __ballot((unsigned)key[decltype(sc)::value] < (unsigned)LO);
        });
        double y = reciprocal(pv);
        static_for<0, K>(LUPP_SF(sc) { masked_mov(hit[decltype(sc)::value], ry[decltype(sc)::value], y); });
        if (__builtin_expect(bad == 0, 1)) {
            double q[K], e[K];
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                q[s] = a[s][k] * y;
                e[s] = __builtin_fma(-pv, q[s], a[s][k]);
            });
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                masked_fma(m[s], a[s][k], e[s], y, q[s]);
            });
        } else {
            /* zeros, the usual case, are none of the values out of range */
            bad = big;
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                bad |= __ballot(((unsigned)key[s] < (unsigned)LO) & (a[s][k] != 0.0));
            });
            if (bad == 0) {
                /* q is the zero of the quotient's sign; a as the residual keeps it so */
                settle(y);
                static_for<0, K>(LUPP_SF(sc) {
                    constexpr int s = decltype(sc)::value;
                    const double q = a[s][k] * y, e = __builtin_fma(-pv, q, a[s][k]);
                    masked_fma(m[s], a[s][k], a[s][k] == 0.0 ? a[s][k] : e, y, q);
                });
            } else {
                odd |= bad;
                static_for<0, K>(LUPP_SF(sc) {
                    constexpr int s = decltype(sc)::value;
                    masked_mov(m[s], a[s][k], a[s][k] / pv); /* one division at a time */
                });
            }
        }
    };

    static_for<0, N / 2>(LUPP_SF(kkc) {
        constexpr int k = 2 * decltype(kkc)::value;
        constexpr std::integral_constant<int, k> k0{};
        constexpr std::integral_constant<int, k + 1> k1{};
        int key[K], M;
        uint64_t h0[K], h1[K], m0[K], m1[K];

        /* step k: its pivot row's entries k and k + 1 go out at once */
        seg_pair p0;
        auto first = [&](auto has_nan) __attribute__((always_inline)) {
            search(k0, key, M, h0, has_nan);
            double x = a[0][k], z = a[0][k + 1];
            int p = pos[0];
            uint64_t own = h0[0];
            static_for<1, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                mask_select(h0[s], x, a[s][k], z, a[s][k + 1], p, pos[s]);
                own |= h0[s];
            });
            masked_put2<k>(own, rp, x, z);
            masked_put_i32<IP + 4 * k>(own, rp, p);
            seg_order();
            p0 = *reinterpret_cast<const seg_pair *>(rec + k);
        };
        first(std::false_type{});
        place(k0, h0, ipl[k]);
        const uint64_t z0 = check_pivot(k0, p0.x, [&]() __attribute__((always_inline)) {
            unplace(k0, h0, ipl[k]);
            first(std::true_type{});
            place(k0, h0, ipl[k]);
        });
        const uint64_t n0 = ~z0;
        static_for<0, K>(LUPP_SF(sc) { m0[decltype(sc)::value] = cand[decltype(sc)::value] & n0; });
        scale(k0, key, M, m0, h0, p0.x);
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            const double u[1] = {p0.y};
            masked_msub<kFMA, 1>(m0[s], a[s][k], &a[s][k + 1], u);
        });

        /* step k + 1: both pivot rows from column k on, row k + 1 with its
         * multiplier and without step k's update */
        constexpr int NC = (N - k - 2 + CH - 1) / CH;
        double u0[2][CH + 1], u1[2][CH + 1];
        auto fetch = [&](auto cc) __attribute__((always_inline)) {
            constexpr int c = decltype(cc)::value;
            constexpr int j0 = k + 2 + c * CH;
            constexpr int j1 = (j0 + CH < N) ? j0 + CH : N;
            if constexpr (c < NC) static_for<j0 / 2, (j1 + 1) / 2>(LUPP_SF(pc) {
                constexpr int j = 2 * decltype(pc)::value;
                const seg_pair v = *reinterpret_cast<const seg_pair *>(rec + j);
                const seg_pair w = *reinterpret_cast<const seg_pair *>(rec + RS + j);
                u0[c & 1][j - j0] = v.x;
                u0[c & 1][j + 1 - j0] = v.y;
                u1[c & 1][j - j0] = w.x;
                u1[c & 1][j + 1 - j0] = w.y;
            });
        };
        seg_pair p1; /* multiplier, pivot */
        double y0[1], y1[1];
        auto second = [&](auto has_nan) __attribute__((always_inline)) {
            search(k1, key, M, h1, has_nan);
            seg_order();
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                const unsigned r = in_mask(h1[s]) ? rp + RS * 8 : rp;
                const uint64_t m = h0[s] | h1[s];
                masked_put_i32<IP + 4 * (k + 1)>(h1[s], rp, pos[s]);
                auto val = [&](auto jc) __attribute__((always_inline)) -> double {
                    constexpr int c = decltype(jc)::value;
                    if constexpr (c < N) return a[s][c];
                    else return b[s];
                };
                constexpr int cols = N + 1 - k, full = cols / 8 * 8;
                static_for<0, cols / 8>(LUPP_SF(pc) {
                    constexpr int j = k + 8 * decltype(pc)::value;
                    masked_put8<j>(m, r, val(std::integral_constant<int, j>{}), val(std::integral_constant<int, j + 1>{}),
                                   val(std::integral_constant<int, j + 2>{}), val(std::integral_constant<int, j + 3>{}),
                                   val(std::integral_constant<int, j + 4>{}), val(std::integral_constant<int, j + 5>{}),
                                   val(std::integral_constant<int, j + 6>{}), val(std::integral_constant<int, j + 7>{}));
                });
                static_for<0, (cols - full + 3) / 4>(LUPP_SF(pc) {
                    constexpr int j = k + full + 4 * decltype(pc)::value;
                    const double x = val(std::integral_constant<int, j>{});
                    if constexpr (j + 3 <= N) {
                        masked_put4<j>(m, r, x, val(std::integral_constant<int, j + 1>{}),
                                       val(std::integral_constant<int, j + 2>{}),
                                       val(std::integral_constant<int, j + 3>{}));
                    } else {
                        if constexpr (j + 1 <= N) masked_put2<j>(m, r, x, val(std::integral_constant<int, j + 1>{}));
                        else masked_put1<j>(m, r, x);
                        if constexpr (j + 2 <= N) masked_put1<j + 2>(m, r, val(std::integral_constant<int, j + 2>{}));
                    }
                });
            });
            seg_order();
            p1 = *reinterpret_cast<const seg_pair *>(rec + RS + k);
            y0[0] = rec[N];
            y1[0] = rec[RS + N];
            if constexpr (PF) fetch(std::integral_constant<int, 0>{});
        };
        second(std::false_type{});
        place(k1, h1, ipl[k + 1]);
        const uint64_t z1 = check_pivot(k1, p1.y, [&]() __attribute__((always_inline)) {
            unplace(k1, h1, ipl[k + 1]);
            second(std::true_type{});
            place(k1, h1, ipl[k + 1]);
        });
        static_for<0, K>(LUPP_SF(sc) { m1[decltype(sc)::value] = cand[decltype(sc)::value] & ~z1; });
        scale(k1, key, M, m1, h1, p1.y);
        /* row k + 1 takes step k's update unless that pivot was zero */
        masked_msub<kFMA, 1>(n0, p1.x, y1, y0);
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            masked_msub2<kFMA, 1>(m0[s], a[s][k], y0, m1[s], a[s][k + 1], y1, &b[s]);
        });
        static_for<0, NC>(LUPP_SF(cc) {
            constexpr int c = decltype(cc)::value;
            constexpr int j0 = k + 2 + c * CH;
            constexpr int j1 = (j0 + CH < N) ? j0 + CH : N;
            fetch(std::integral_constant<int, PF ? c + 1 : c>{});
            masked_msub<kFMA, j1 - j0>(n0, p1.x, u1[c & 1], u0[c & 1]);
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                masked_msub2<kFMA, j1 - j0>(m0[s], a[s][k], u0[c & 1], m1[s], a[s][k + 1], u1[c & 1],
                                            &a[s][j0]);
            });
        });
        seg_order();
    });
    if constexpr (N % 2 == 1) {
        /* the last row of an odd size: one candidate, nothing left to update */
        constexpr int k = N - 1;
        static_for<0, K>(LUPP_SF(sc) {
            constexpr int s = decltype(sc)::value;
            masked_put1<k>(cand[s], rp, a[s][k]);
            masked_put_i32<IP + 4 * k>(cand[s], rp, pos[s]);
            pos[s] = in_mask(cand[s]) ? 64 + k : pos[s];
        });
        seg_order();
        const double pv = rec[k];
        info = (pv == 0.0 && info == 0) ? N : info;
        const int h = seg_hi_abs(pv);
        odd |= __ballot((h < LO || h > HI) && pv != 0.0);
        const double y = reciprocal(pv);
        static_for<0, K>(LUPP_SF(sc) { masked_mov(cand[decltype(sc)::value], ry[decltype(sc)::value], y); });
    }
    static_for<0, K>(LUPP_SF(sc) {
        constexpr int s = decltype(sc)::value;
        pos[s] = pos[s] >= 0 ? (pos[s] & 63) : -1;
    });

    /* Back substitution, column j descending: the row at position j divides,
     * its x_j goes to rec[j], the rows above eliminate it. Divisions take the
     * kept reciprocals; they are exact while every pivot (checked: odd) is in
     * range and every x_j (checked afterwards, so also every numerator) is in
     * range or has the numerator +0. A wave where one is not substitutes again
     * from the saved right-hand side with true divisions. */
    if (__ballot(info == 0) != 0) {
        double b0[K];
        static_for<0, K>(LUPP_SF(sc) { b0[decltype(sc)::value] = b[decltype(sc)::value]; });
        auto subst = [&](auto exact) __attribute__((always_inline)) {
            uint64_t above[K];
            static_for<0, K>(LUPP_SF(sc) {
                above[decltype(sc)::value] = __ballot(pos[decltype(sc)::value] >= 0);
            });
            static_for_down<0, N>(LUPP_SF(jc) {
                constexpr int j = decltype(jc)::value;
                static_for<0, K>(LUPP_SF(sc) {
                    constexpr int s = decltype(sc)::value;
                    const uint64_t own = __ballot(pos[s] == j);
                    above[s] &= ~own;
                    double x;
                    if constexpr (decltype(exact)::value) {
                        x = b[s] / a[s][j];
                    } else {
                        const double q = b[s] * ry[s];
                        x = __builtin_fma(__builtin_fma(-a[s][j], q, b[s]), ry[s], q);
                    }
                    masked_put1<j>(own, rp, x);
                });
                if constexpr (j > 0) {
                    const double x[1] = {rec[j]};
                    static_for<0, K>(LUPP_SF(sc) {
                        constexpr int s = decltype(sc)::value;
                        masked_msub<kFMA, 1>(above[s], a[s][j], &b[s], x);
                    });
                }
            });
            seg_order();
        };
        uint64_t redo = odd;
        if (redo == 0) {
            subst(std::false_type{});
            /* b[s] is the row's numerator now: +0 gives the zero of the right
             * sign, -0 may not */
            uint64_t out[K];
            static_for<0, K>(LUPP_SF(sc) {
                constexpr int s = decltype(sc)::value;
                const int h = seg_hi_abs(rec[pos[s] >= 0 ? pos[s] : 0]);
                out[s] = __ballot(info == 0 && (h < (1023 - 300) << 20 || h > (1023 + 300) << 20));
                redo |= out[s];
            });
            if (__builtin_expect(redo != 0, 0)) {
                redo = 0;
                static_for<0, K>(LUPP_SF(sc) {
                    constexpr int s = decltype(sc)::value;
                    redo |= out[s] & __ballot(pos[s] >= 0 && __builtin_bit_cast(uint64_t, b[s]) != 0);
                });
            }
            static_for<0, K>(LUPP_SF(sc) { b[decltype(sc)::value] = b0[decltype(sc)::value]; });
        }
        if (__builtin_expect(redo != 0, 0)) subst(std::true_type{});
    }
    return info;
}

#undef LUPP_IN
#undef LUPP_OUT
#undef LUPP_MUL_SUB
#undef LUPP_FMA_SUB
#undef LUPP_RW
#undef LUPP_RD
#undef LUPP_IN1
#undef LUPP_MUL_SUB1
#undef LUPP_FMA_SUB1
#undef LUPP_RD1

}  // namespace lupp

#endif
