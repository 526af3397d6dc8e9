// The weighted frequency autoconvolution of the kappa-DFT pair sum,
//     Y[q][kw] = sum_{iw} Wh(iw, kw) Z[q][iw] Z[q][kw - iw]
// over the sheared half table Wh (each unordered frequency pair once).
#include <algorithm>

#include "srm3_device.hpp"
#include "srm3_internal.hpp"

namespace srm3 {

namespace {

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

struct YpairArgs {
    const void *Z;      // [B][M][ncw] phase DFTs along kappa
    void *Y;            // [B][M][nca]
    const void *wh;     // [wh_rows][nca] sheared half table, zero rows after row ncw - 1
    int M, W, nca, kw0, wh_rows;
    int batch, n_qtiles, n_ctiles, per_xcd;
    int one_sided;      // partners i_w <= k_omega only (both partners >= 0)
};

// A wave owns 64 consecutive output columns (one per lane) and R DFT rows q,
// and walks the partner frequencies i_w in chunks of C steps.  The b operand
// Z[q][kw - i_w] of lane l at step i_w is element e = e0 + l - i_w of row q, so
// a chunk reads a window of 64 + C - 1 elements per row, staged in the wave's
// own slice of LDS (no barrier: the wave alone writes and reads its slice).
// The a operand Z[q][i_w] is the same for all lanes and comes through scalar
// loads, or with ALDS from the wave's LDS slice; the weight row W_h[i_w][.] is read once per step for
// all R rows, two steps ahead.  Steps past the last partner meet zero weights
// (zero rows after the table, or pairs outside the support) and the last
// partner's a operand.  Per term: t = a b (4 operations), acc += w t (4 FMAs).
//
// Bound by the vector ALUs (8 operations per term, 9.0 issued: busy all of the
// cycles at 256x1024, where the clock falls to 2.1 GHz).  Buffer loads took the
// window's address arithmetic away, scalar loads one of two LDS reads per term:
// 256x1024, batch 64, FP32 16.1 -> 14.8 ms for the whole call (14.5 with the
// column transforms that came after); the process of 4096 frequencies, 4096
// realizations 6.3 -> 5.8.  Column tiles in the outer order (fewer passes over the
// weights, but every wave's rows fall out of the scalar cache): 24 ms.
constexpr int kY2Rows = 8;   // DFT rows per wave
constexpr int kWaves = 4;    // per block

template <typename T, int R, int C, bool ALDS>
__global__ __launch_bounds__(64 * kWaves) void ypair2_kernel(YpairArgs a)
{
    using T2 = typename vec<T>::v2;
    constexpr int LW = 64 + C;   // staged elements per row (64 + C - 1 used)
    constexpr unsigned E = sizeof(T2);
    extern __shared__ unsigned char smem_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    T2 *ldsb = reinterpret_cast<T2 *>(smem_raw) + wave * (R * LW + (ALDS ? C * R : 0));
    T2 *ldsa = ldsb + R * LW;   // ALDS: [step][row]
    // a block: one column tile, kWaves consecutive q tiles (one per wave), so
    // that its waves read the same weight rows at about the same time
    const int bid = blockIdx.x;
    const int work = (bid % kXcds) * a.per_xcd + bid / kXcds;
    const int n_qgroups = (a.n_qtiles + kWaves - 1) / kWaves;
    const int per_b = n_qgroups * a.n_ctiles;
    if (work >= a.batch * per_b) return;
    const int b = work / per_b;
    const int rem = work - b * per_b;
    const int qg = rem / a.n_ctiles;
    const int ct = rem - qg * a.n_ctiles;
    const int qt = qg * kWaves + wave;
    if (qt >= a.n_qtiles) return;
    const int cc0 = ct * 64;
    const int W = a.W, ncw = 2 * W - 1, q0 = qt * R;
    const int rows = min(R, a.M - q0);
    const T2 *Zq = uniform_ptr(static_cast<const T2 *>(a.Z) + (static_cast<long>(b) * a.M + q0) * ncw);
    const int kw_lo = a.kw0 + cc0;
    const int kw_hi = a.kw0 + min(cc0 + 64, a.nca) - 1;
    const int iw_lo = max(-W + 1, (kw_lo + 1) >> 1);
    const int iw_hi = min(W - 1, a.one_sided ? kw_hi : kw_hi + W - 1);
    const int nchunk = __builtin_amdgcn_readfirstlane(iw_hi >= iw_lo ? (iw_hi - iw_lo + C) / C : 0);
    // rows past the last read that one, lanes past a row's ends get a vector
    // offset past the buffer (and load zero)
    const unsigned row_bytes = static_cast<unsigned>(ncw) * E;
    const brsrc zr = make_brsrc(Zq, static_cast<unsigned>(rows) * row_bytes);
    const unsigned wrow_bytes = static_cast<unsigned>(a.nca) * E;
    const brsrc wr = make_brsrc(a.wh, static_cast<unsigned>(a.wh_rows) * wrow_bytes);
    const unsigned wcol = static_cast<unsigned>(cc0 + lane) * E;

    T accr[R], acci[R], sumr[R], sumi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) accr[r] = acci[r] = sumr[r] = sumi[r] = T(0);

    for (int ch = 0; ch < nchunk; ++ch) {
        const int iwc = iw_lo + ch * C;
        // b window: lane l at chunk step s reads index l + C - 1 - s of row r
        const int e_lo = kw_lo + W - 1 - (iwc + C - 1);
        const int e0 = e_lo + lane, e1 = e0 + 64;
        const unsigned v0 = e0 >= 0 && e0 < ncw ? static_cast<unsigned>(e0) * E : ~31u;
        const unsigned v1 = e1 >= 0 && e1 < ncw ? static_cast<unsigned>(e1) * E : ~31u;
        T2 z0[R], z1[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned ro = static_cast<unsigned>(ypair_row(r, rows)) * row_bytes;
            z0[r] = bload(zr, v0, ro, T(0));
            z1[r] = bload(zr, v1, ro, T(0));
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ldsb[r * LW + lane] = z0[r];
            if (lane < C) ldsb[r * LW + 64 + lane] = z1[r];
        }
        const int ic0 = iwc + W - 1;
        if constexpr (ALDS) {
            static_assert(64 % R == 0 && C * R % 64 == 0, "staging shape");
            const int r = ypair_row(lane % R, rows);
#pragma unroll
            for (int i = 0; i < C * R / 64; ++i) {
                const int ic = ic0 + lane / R + 64 / R * i;
                ldsa[i * 64 + lane] =
                    bload(zr, ic < ncw ? static_cast<unsigned>(r) * row_bytes + static_cast<unsigned>(ic) * E : ~31u, 0u, T(0));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        auto load_w = [&](int s) { return bload(wr, wcol, static_cast<unsigned>(ic0 + s) * wrow_bytes, T(0)); };
        auto load_a = [&](T2 (&av)[2][R], int s) {
            if constexpr (ALDS) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int r = 0; r < R; ++r) av[u][r] = ldsa[(s + u) * R + r];
                return;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const cptr<T> p = as_const(reinterpret_cast<const T *>(Zq)) + 2 * min(ic0 + s + u, ncw - 1);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const long o = 2 * static_cast<long>(ypair_row(r, rows)) * ncw;
                    av[u][r].x = p[o];
                    av[u][r].y = p[o + 1];
                }
            }
        };
        auto pair = [&](const T2 (&av)[2][R], const T2 (&w)[2], int s) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const T2 *bp = ldsb + (lane + C - 1 - s - u);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const T2 bv = bp[r * LW];
                    const T tr = fma_(av[u][r].x, bv.x, -(av[u][r].y * bv.y));
                    const T ti = fma_(av[u][r].x, bv.y, av[u][r].y * bv.x);
                    accr[r] = fma_(w[u].x, tr, accr[r]);
                    accr[r] = fma_(-w[u].y, ti, accr[r]);
                    acci[r] = fma_(w[u].x, ti, acci[r]);
                    acci[r] = fma_(w[u].y, tr, acci[r]);
                }
            }
        };
        T2 a0[2][R], w0[2], w1[2];
        w0[0] = load_w(0);
        w0[1] = load_w(1);
        if constexpr (!ALDS) {
            // a two steps ahead, in two sets of scalar registers (FP32 only: see launch_ypair)
            T2 a1[2][R];
            load_a(a0, 0);
            for (int s = 0; s < C; s += 4) {
                load_a(a1, s + 2);
                w1[0] = load_w(s + 2);
                w1[1] = load_w(s + 3);
                pair(a0, w0, s);
                load_a(a0, s + 4);
                w0[0] = load_w(s + 4);
                w0[1] = load_w(s + 5);
                pair(a1, w1, s + 2);
            }
        } else {
#pragma unroll 2
            for (int s = 0; s < C; s += 2) {
                load_a(a0, s);
                w1[0] = load_w(s + 2);
                w1[1] = load_w(s + 3);
                pair(a0, w0, s);
                w0[0] = w1[0];
                w0[1] = w1[1];
            }
        }
        // the slice is rewritten by the next chunk only after these reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (ch & 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                sumr[r] += accr[r];
                sumi[r] += acci[r];
                accr[r] = acci[r] = T(0);
            }
        }
    }
    T2 *Y = static_cast<T2 *>(a.Y) + static_cast<long>(b) * a.M * a.nca;
    const int cc = cc0 + lane;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (cc < a.nca && q0 + r < a.M) {
            T2 v;
            v.x = sumr[r] + accr[r];
            v.y = sumi[r] + acci[r];
            Y[static_cast<long>(q0 + r) * a.nca + cc] = v;
        }
    }
}

template <typename T, bool ALDS>
hipError_t ypair_t(YpairArgs y, hipStream_t st)
{
    y.n_qtiles = (y.M + kY2Rows - 1) / kY2Rows;
    y.n_ctiles = (y.nca + 63) / 64;
    const long blocks = static_cast<long>(y.batch) * ((y.n_qtiles + kWaves - 1) / kWaves) * y.n_ctiles;
    y.per_xcd = static_cast<int>((blocks + kXcds - 1) / kXcds);
    const size_t lds = static_cast<size_t>(kWaves) * kY2Rows * (64 + kYpairChunk + (ALDS ? kYpairChunk : 0)) *
                       sizeof(typename vec<T>::v2);
    ypair2_kernel<T, kY2Rows, kYpairChunk, ALDS>
        <<<dim3(static_cast<unsigned>(static_cast<long>(y.per_xcd) * kXcds)), 64 * kWaves, lds, st>>>(y);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ypair(int precision, const Geometry &g, const KfftGeom &k, const void *Z, void *Y, const void *wh,
                        int batch, hipStream_t st)
{
    YpairArgs y{};
    y.Z = Z;
    y.Y = Y;
    y.wh = wh;
    // one kappa line: the realizations are the rows ([B][1][.] == [B][.])
    y.M = k.M == 1 ? batch : k.M;
    y.batch = k.M == 1 ? 1 : batch;
    y.W = g.W;
    y.nca = k.nca;
    y.kw0 = k.kw0;
    y.wh_rows = k.wh_rows;
    y.one_sided = k.one_sided;
    // FP64: a in LDS.  Scalar loads of it take the scalar registers of two steps,
    // so they are not requested ahead: 256x1024 lines, one realization, 0.65 ms,
    // LDS 0.49; eight 3.68, 3.06; 32x2048 x 4 1.22, 0.79; the process 4096x4096 11.9,
    // 8.9 (both staged in LDS through registers of 64-bit addresses, before: 0.58,
    // 3.85, 1.08, 11.0).
    if (precision == SRM3_FP64) return ypair_t<double, true>(y, st);
    // FP32: the scalar loads of a pay while the waves of a launch share its rows
    // in the scalar cache, in large kappa-DFTs, not in small ones nor the process,
    // whose rows lie far apart (scalar loads, LDS, in ms a call): 256x1024 lines
    // with 2048 waves 0.47, 0.38, 8192 1.10, 1.00, 16384 1.92, 1.89, 131072 14.57,
    // 14.70; 256x256 with 8192 0.362, 0.356, 16384 0.620, 0.634; 512x512 with 8192
    // 0.605, 0.581, 16384 1.033, 1.043, 65536 4.01, 4.09; 32x2048 (M = 64) with
    // 32768 7.39, 7.14; the process 4096x4096 6.45, 5.73, 1000x513 0.295, 0.191.
    // Both sum alike, bitwise.
    const long waves = static_cast<long>(y.batch) * ((y.M + kY2Rows - 1) / kY2Rows) * ((y.nca + 63) / 64);
    const bool scalar = !k.one_sided && waves >= 16384;
    return scalar ? ypair_t<float, false>(y, st) : ypair_t<float, true>(y, st);
}

}  // namespace srm3
