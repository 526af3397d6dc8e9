// Device pieces of the matrix-core pair sums (FP32 and FP64): the a operand's
// layout, the MFMA of each type and the sum of a wave's tiles over a range of
// partner columns.
#pragma once

#include "srm3_device.hpp"
#include "srm3_internal.hpp"

namespace srm3 {

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Layout of the a operand (re, re + im, im - re) of support column ic, row kk:
// FP32 keeps three kappa-contiguous planes (a block's rows load as wide scalar
// loads); FP64 interleaves the three values per row, padded to four, so that
// rows load one at a time and the scalar register window stays small.
template <typename T> struct ALayout;
template <> struct ALayout<float> {
    static constexpr int ES = 1;       // element stride between rows
    static constexpr int NS = 3;       // slots per (column, row)
    __device__ static long plane(const Geometry &g) { return static_cast<long>(g.ncw) * g.nkp; }
};
template <> struct ALayout<double> {
    static constexpr int ES = 4;
    static constexpr int NS = 4;
    __device__ static long plane(const Geometry &) { return 1; }
};

// Per-precision pieces of the matrix-core pair sum: the 16x16x4 MFMA and its
// output row layout, the a
// operand layout (FP32: three kappa-contiguous planes; FP64: the three values
// of a (column, row) side by side, rows 32 bytes apart) and whether the sums
// are flushed into two-sum pairs (FP32 only).
template <typename T> struct MfmaT;
template <> struct MfmaT<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static constexpr bool COMP = true;
    static constexpr bool PLANAR = true;
    static constexpr unsigned ROW_BYTES = 4;
    __device__ static v4 mfma(float x, float y, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); }
    __device__ static int drow(int q, int e) { return 4 * q + e; }   // output row of lane group q, element e
    __device__ static float aload(brsrc r, unsigned voff, unsigned soff) { return bload32(r, voff, soff); }
};
template <> struct MfmaT<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static constexpr bool COMP = false;
    static constexpr bool PLANAR = false;
    static constexpr unsigned ROW_BYTES = 32;
    __device__ static v4 mfma(double x, double y, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0); }
    __device__ static int drow(int q, int e) { return q + 4 * e; }   // rows interleaved (checked on the device)
    __device__ static double aload(brsrc r, unsigned voff, unsigned soff) { return bload64(r, voff, soff); }
};

// A wave's RT x CT tiles of one realization (output rows from 16 RT rg, columns
// c0 .. c0 + 16 CT - 1) over the partner columns i0 .. i1: P1, P2, P3 += the
// three real products.  after(n) runs after every four columns, n kappa splits
// each.  FP64 leaves row tiles past the grid's rows out.  PRIO: issue each split's
// MFMAs at raised wave priority.
template <typename T, int RT, int CT, bool PRIO, class After>
__device__ __forceinline__ void mfma_columns(const Geometry &g, const typename vec<T>::v2 *__restrict__ zrow_b,
                                             const T *__restrict__ zcol_b,
                                             const typename vec<T>::v2 *__restrict__ wtab, int rg, int c0, int i0, int i1,
                                             typename MfmaT<T>::v4 (&P1)[RT][CT], typename MfmaT<T>::v4 (&P2)[RT][CT],
                                             typename MfmaT<T>::v4 (&P3)[RT][CT], const After &after)
{
    using T2 = typename vec<T>::v2;
    using M = MfmaT<T>;
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int K0 = rg * 16 * RT;
    const int Wm1 = g.W - 1;
    const int kk_max = min(K0 + 16 * RT - 1, g.nk - 1);
    const int jk_end = kk_max / 2;   // last kappa split any row of the wave uses
    const int jb = K0 / 2;           // splits below jb are at full weight for every row

    const long lines = static_cast<long>(g.nk) * g.nc;
    const long plane = static_cast<long>(g.ncw) * g.nkp;
    // b rows through a buffer resource (uniform row offset, per-lane column).
    // The a planes' resource starts `shift` rows before them: per-lane offsets
    // stay fixed for a partner step and the split moves the uniform offset
    // (shift - jk rows, never negative).  Reads of rows a split does not use
    // stay inside the plan's workspace (the phase rows precede the a planes);
    // their values (not necessarily finite) are replaced by zero, skipped with
    // their tile, or land in an output row that is not stored.
    const unsigned row_bytes = static_cast<unsigned>(g.nc * sizeof(T2));
    const brsrc zb = make_brsrc(zrow_b, static_cast<unsigned>(lines * sizeof(T2)));
    const int shift = jk_end + 2;
    constexpr unsigned RS = M::ROW_BYTES;   // bytes between kappa rows of one a value
    const brsrc za = make_brsrc(reinterpret_cast<const char *>(zcol_b) - static_cast<long>(shift) * RS,
                                static_cast<unsigned>(ALayout<T>::NS * plane * sizeof(T) + (shift + 64) * RS));
    // bytes between the three a values of one (column, row)
    const unsigned plane_bytes = M::PLANAR ? static_cast<unsigned>(plane * sizeof(T)) : static_cast<unsigned>(sizeof(T));

    // Partner step iw0 (4 columns): the lane's a-plane byte offset (row
    // K0 + li of column ic, plane 0), its b column offsets and weights.
    auto setup = [&](int s0, unsigned &ao, unsigned (&bo)[CT], T2 (&w)[CT]) {
        const int iw = s0 + lq;
        const int ic = min(iw + Wm1, g.ncw - 1);
        ao = static_cast<unsigned>(ic * g.nkp + K0 + li) * RS;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int col = c0 + 16 * c + li;
            const int jw = col - (g.nw - 1) - iw;
            const bool ok = col < g.nc && iw <= Wm1 && jw > -g.W && jw < g.W;
            w[c].x = T(0);
            w[c].y = T(0);
            if (ok) w[c] = wtab[static_cast<long>(iw + Wm1) * g.ncw + (jw + Wm1)];
            bo[c] = ok ? static_cast<unsigned>(jw + g.nw - 1) * static_cast<unsigned>(sizeof(T2)) : 0u;
        }
    };
    // operands of split jk: b phases per column tile, a planes per row tile
    auto load_split = [&](T2 (&zs)[CT], T (&as)[RT][3], unsigned ao, const unsigned (&bo)[CT], int jk) {
#pragma unroll
        for (int c = 0; c < CT; ++c) zs[c] = bload(zb, bo[c], static_cast<unsigned>(jk) * row_bytes, T(0));
        const unsigned so = static_cast<unsigned>(shift - jk) * RS;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const unsigned o = ao + 16u * RS * r;
            as[r][0] = M::aload(za, o, so);
            as[r][1] = M::aload(za, o + plane_bytes, so);
            as[r][2] = M::aload(za, o + 2 * plane_bytes, so);
        }
    };
    auto split = [&](int jk, bool tail, const unsigned (&bo)[CT], const T2 (&wc)[CT], const T2 (&zc)[CT],
                     const T (&ac)[RT][3]) {
        T bs[CT], bi[CT], br[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const T Br = fma_(wc[c].x, zc[c].x, -wc[c].y * zc[c].y);
            const T Bi = fma_(wc[c].x, zc[c].y, wc[c].y * zc[c].x);
            bs[c] = Br + Bi;
            bi[c] = Bi;
            br[c] = Br;
        }
        // PRIO: the split's MFMAs at raised wave priority, so that a wave that
        // reaches them issues them back to back while the other waves of the
        // SIMD do their VALU work
        if (PRIO) __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            // no row of this tile is stored (the branch costs FP32 6 % at 100x333 lines)
            if (!M::COMP && r > 0 && K0 + 16 * r >= g.nk) continue;
            if (tail && 2 * jk > K0 + 16 * r + 15) continue;   // no row of this tile uses the split
            T x0 = ac[r][0], x1 = ac[r][1], x2 = ac[r][2];
            if (tail) {
                // rows above the split keep their values, the split's own row
                // is halved, rows below it are replaced by zero (a select, not
                // a product: the values read there lie outside the a planes
                // and need not be finite)
                const int kk = K0 + 16 * r + li;
                const T h = 2 * jk == kk ? T(0.5) : T(1);
                const bool use = 2 * jk <= kk;
                x0 = use ? x0 * h : T(0);
                x1 = use ? x1 * h : T(0);
                x2 = use ? x2 * h : T(0);
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                P1[r][c] = M::mfma(x0, bs[c], P1[r][c]);
                P2[r][c] = M::mfma(x1, bi[c], P2[r][c]);
                P3[r][c] = M::mfma(x2, br[c], P3[r][c]);
            }
        }
        if (PRIO) __builtin_amdgcn_s_setprio(0);
    };

    for (int iw0 = i0; iw0 <= i1; iw0 += 4) {
        unsigned ao;
        unsigned boff[CT];
        T2 wc[CT];
        setup(iw0, ao, boff, wc);
        // two operand sets: even splits in set 0, odd ones in set 1; each
        // split first requests the next split's operands (the scheduling
        // barrier keeps those loads ahead of this split's MFMAs; past the
        // last split they read unused rows)
        T2 z0[CT], z1[CT];
        T a0[RT][3], a1[RT][3];
        load_split(z0, a0, ao, boff, 0);
        auto pair = [&](int jk, bool tail, bool both) {
            load_split(z1, a1, ao, boff, jk + 1);
            __builtin_amdgcn_sched_barrier(0);
            split(jk, tail, boff, wc, z0, a0);
            if (!both) return;
            load_split(z0, a0, ao, boff, jk + 2);
            __builtin_amdgcn_sched_barrier(0);
            split(jk + 1, tail, boff, wc, z1, a1);
        };
        // jb = K0 / 2 is even: the bulk ends on a set-0 split
        int jk = 0;
        for (; jk < jb; jk += 2) pair(jk, false, true);      // every row of the wave at full weight
        for (; jk + 1 <= jk_end; jk += 2) pair(jk, true, true);
        if (jk <= jk_end) pair(jk, true, false);
        after(jk_end + 1);
    }
}

}  // namespace srm3
