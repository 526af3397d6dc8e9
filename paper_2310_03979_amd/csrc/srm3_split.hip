// The FP32 direct-form pair sum as Toeplitz products of split phases on the
// FP16 matrix cores, and the phase kernel that lays out its operands.
//
// Unordered pairs are split by frequency: for output line k = (kk, kw),
//     T_k = sum_{iw >= kw - iw} f(iw) W(iw, kw - iw) sum_{jk <= kk} z[kk - jk][iw] z[jk][kw - iw],
// f = 1 for iw > jw = kw - iw and 1/2 for iw == jw (there the ordered kappa
// splits count every pair twice and the self pair once, whose other half the
// assembly adds).  For one partner column iw the inner sum is a product of the
// lower-triangular Toeplitz matrix of column iw with the phase columns jw, and
// its operands are raw phase factors (times line factors of moderate range),
// so that each splits into two FP16 parts,
//     2^10 z = hi + lo + e,  |e| <= 2^-24 2^10 for |z| <= 1,
// so that three FP16 products (hi hi + hi lo + lo hi) with FP32 accumulation
// replace one FP32 product: 12 FP16 multiply-adds per pair term at 16 times
// the FP32 matrix rate.  A product drops lo lo and the two e: below 1.5 x 2^-23
// of the largest factors' product.  The weight is applied in FP32, once per
// output and partner column, and the weighted products are summed in FP32 on
// three levels: groups of columns, items, tiles.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "srm3_device.hpp"
#include "srm3_internal.hpp"

namespace srm3 {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

constexpr float kSplitScale = 1024.0f;            // z is held times 2^10
constexpr float kSplitUnscale = 1.0f / 1024.0f;   // applied to W and to the sums

// ---------------------------------------------------------------------------
// Phases with the split operand: the tiles of phase_kernel (64 frequencies x
// 64 rows), the same words and phase rows; the four FP16 parts are staged in
// LDS and written along kappa, eight rows per store.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void phase_split_kernel(SeedChunk seeds, const uint64_t *__restrict__ seeds_dev,
                                                          int b0, Geometry g, float2 *__restrict__ zrow,
                                                          _Float16 *__restrict__ zh, const double *__restrict__ lr)
{
    constexpr int TR = 64;
    __shared__ _Float16 at[4][64][TR + 2];   // odd dword stride: columns on distinct banks
    __shared__ __align__(16) uint32_t wt[TR][68];
    __shared__ double2 ptab[256];
    phase_table_fill(ptab);
    const int bl = blockIdx.z;
    const int b = b0 + bl;
    const int k0 = blockIdx.y * TR;
    const uint64_t seed = seeds_dev ? seeds_dev[b] : seeds.s[bl];
    const int q0 = floor_div4(-(g.nw - 1)) + 16 * static_cast<int>(blockIdx.x);
    const int kw0 = 4 * q0;
    {
        const int gi = threadIdx.x & 15;
        const int q = q0 + gi;
        const bool live = 4 * q + 3 >= -(g.nw - 1) && 4 * q <= g.nw - 1;
#pragma unroll
        for (int i = 0; i < TR / 16; ++i) {
            const int kt = (threadIdx.x >> 4) + 16 * i;
            const int kk = k0 + kt;
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            if (live && kk < g.nk) phase_words(kk, q, seed, w);
            *reinterpret_cast<uint4 *>(&wt[kt][4 * gi]) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    __syncthreads();   // words and phase table
    const int ct = threadIdx.x & 63;
    const int c = kw0 + ct + g.nw - 1;
    const int ic0 = kw0 + g.W - 1;   // support column of the tile's first column
    const bool planes = ic0 + 63 >= 0 && ic0 < g.ncw;
#pragma unroll 4
    for (int i = 0; i < TR / 4; ++i) {
        const int kt = (threadIdx.x >> 6) + 4 * i;
        const int kk = k0 + kt;
        double s = 0.0, co = 0.0;   // rows past n_kappa hold zero
        if (c >= 0 && c < g.nc && kk < g.nk) {
            const long l = static_cast<long>(kk) * g.nc + c;
            phase_line(wt[kt][ct], ptab, lr, l, co, s);
            zrow[static_cast<long>(b) * g.nk * g.nc + l] =
                make_float2(static_cast<float>(co), static_cast<float>(s));
        }
        if (planes) {
            const double sr = co * static_cast<double>(kSplitScale), si = s * static_cast<double>(kSplitScale);
            const _Float16 rh = static_cast<_Float16>(sr), ih = static_cast<_Float16>(si);
            at[0][ct][kt] = rh;
            at[1][ct][kt] = static_cast<_Float16>(sr - static_cast<double>(rh));
            at[2][ct][kt] = ih;
            at[3][ct][kt] = static_cast<_Float16>(si - static_cast<double>(ih));
        }
    }
    if (!planes) return;
    __syncthreads();
    const int nk8 = split_nk8(g.nk), seg = split_seg(g.nk);
    _Float16 *zb = zh + static_cast<size_t>(b) * (split_operand_bytes(g.nk, g.ncw) / 2);
    if (k0 == 0) {
        const int ic = ic0 + static_cast<int>(threadIdx.x >> 2);
        if (ic >= 0 && ic < g.ncw)
            *reinterpret_cast<half8 *>(zb + (static_cast<long>(ic) * 4 + (threadIdx.x & 3)) * seg) = half8(static_cast<_Float16>(0));
    }
    // 64 columns x 4 parts x 8 groups of eight rows
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int t = threadIdx.x + 256 * i;
        const int gr = t & 7, pl = (t >> 3) & 3, col = t >> 5;
        const int ic = ic0 + col, kk = k0 + 8 * gr;
        if (ic < 0 || ic >= g.ncw || kk >= nk8) continue;
        half8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = at[pl][col][8 * gr + e];
        *reinterpret_cast<half8 *>(zb + (static_cast<long>(ic) * 4 + pl) * seg + 8 + kk) = v;
    }
}

// ---------------------------------------------------------------------------
// Pair sum.
//
// A block of eight waves owns a tile of RS = 32 NV output rows x CB = 256 / NV
// output columns and walks the partner columns iw.  Wave (v, cw) owns two
// 16-row tiles, v and the v-th from the end (so that the triangular work is
// shared evenly), x two 16-column tiles.  The kappa splits go in passes of
// JB = RS rows of the b operand (one pass per 256 rows):
//  - b: the phase columns jw = kw - iw of the tile are a window that moves by
//    one column per iw, kept in a ring in LDS (JB rows x 4
//    parts each); one column is loaded per iw.
//  - a: the Toeplitz blocks of column iw are shifted copies of it.  LDS holds
//    for every start s the eight values z[s .. s + 7] of each part, so that any
//    block is read with aligned 16-byte loads.
// Both are double buffered against one barrier per iw.  b is stored reversed
// in groups of eight, so that a's eight values ascend.
// v_mfma_f32_16x16x32_f16: lane l, i = l % 16, q = l / 16 holds A[i][8q + e]
// and B[8q + e][i], e = 0..7, and D[4q + e][i], e = 0..3.
// LDS banks: 16-byte reads go in groups of 16 lanes, 0-3, 12-15, 20-27 and so
// on, over 64 banks; the ring's stride (32 bytes past a multiple of 256) and
// the swizzled starts (bit 3 flipped by bit 4) put every group on distinct
// banks.
//
// Work item: one tile x split_chunk partner columns.  Items are taken from a
// queue in order (chunk by chunk over all tiles) and each adds its sums to the
// tile's in `tout` after the item of the previous chunk has, so the sum does
// not depend on which blocks run the items or on how many requests share the
// launch.  The wait ends: an item is taken only after all items before it were
// taken by running blocks, and the first unfinished one waits for nothing.
//
// Bound by the chip's power: at 256x1024 (batch 64) the pair sum takes 60 ms
// (FP32 16x16x4 MFMAs: 169 ms) with the matrix cores busy 72 % of the cycles at
// 1.99 GHz (counters; 36 ms of MFMA issue at 2.4 GHz), at 512x8192 (support 2048,
// batch 16) 295 ms (817), 75 % at 1.94.  Taking a quarter of the MFMAs out gains
// 18 %, a third of the LDS reads 6 %, the weights 3 %.
// Tried: 64 x 32 outputs per wave in passes of 128 rows (72 ms: a second pass
// over the partner columns, spills); both operands of the next step in a
// second register set (spills, 100 ms); 32x32x16 MFMAs (7 % slower).
// ---------------------------------------------------------------------------
// Partner columns of an item, by the support alone: 64 (0.15 ms at 256 rows;
// 128 leave single calls short of items, 64x128 lines 0.156 -> 0.254 ms), more
// where a tile would have over 64 items, each of which rounds its sum once.
__host__ __device__ inline int split_chunk(int W) { return 64 * ((2 * W - 1 + 4095) / 4096); }
// FP32 sums of this many columns are added to the item's: a column rounds a sum
// of eight, not of the whole item.  Relative error of the coefficients (root
// mean square, against 64 bits) with one sum per item, so, and in the FP32
// MFMAs' form: 32x512 lines 2.2e-7, 1.5e-7, 2.1e-7; 64x2048 2.8e-7, 1.7e-7,
// 2.1e-7; 256x1024 2.4e-7, 1.5e-7, 4.0e-7.  Groups of 4 the same; the time too.
constexpr int kSplitGroup = 8;

template <int NV> struct SplitShape {
    static constexpr int RS = 32 * NV;              // rows of a tile
    static constexpr int CB = 256 / NV;             // columns of a tile
    static constexpr int JB = RS;                   // b rows per pass
    static constexpr int KS = JB / 32;              // MFMA steps per pass
    static constexpr int RING = CB + 8;              // (a multiple of 8: wrapped columns keep their banks)
    static constexpr int PART = JB * 2;             // bytes of one part of a ring column
    static constexpr int COL = 4 * PART + 32;       // ring column stride
    static constexpr int NS = RS + JB;              // starts held of the a column
    static constexpr int EPART = NS * 16;
    static constexpr int EBUF = 4 * EPART;
    static constexpr int LDS = RING * COL + 2 * EBUF;
};

struct SplitArgs {
    const void *zh;      // [B] operands (split_operand_bytes)
    const void *wtab;    // [ncw][ncw] float2
    void *tout;          // [B][nk][nc] float2
    Geometry g;
    int n_rs, n_cg;      // tiles along kappa and frequency
    int tiles;           // batch * n_rs * n_cg
    int n_items;
    unsigned *queue;     // next item, zero at launch
    unsigned *done;      // chunks committed per tile, zero at launch
    const PReq *reqs;    // with items: the requests and their work list
    const PItem *items;
};

// Partner columns of a tile: iw from lo to hi (empty: hi < lo).
__host__ __device__ inline void split_range(int nw, int nc, int W, int cb, int cg, int &lo, int &hi)
{
    const int k0 = cg * cb - (nw - 1);
    const int k1 = (cg * cb + cb - 1 < nc - 1 ? cg * cb + cb - 1 : nc - 1) - (nw - 1);
    const int half = k0 >= 0 ? (k0 + 1) / 2 : -(-k0 / 2);   // ceil(k0 / 2)
    lo = half > -(W - 1) ? half : -(W - 1);
    hi = k1 + W - 1 < W - 1 ? k1 + W - 1 : W - 1;
}

__host__ __device__ inline int split_chunks(const Geometry &g, int cb, int cg)
{
    int lo, hi;
    split_range(g.nw, g.nc, g.W, cb, cg, lo, hi);
    return hi < lo ? 1 : (hi - lo) / split_chunk(g.W) + 1;
}

// (the 16-byte loads of a's starts are aligned to two bytes only)
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ uint4v load16(brsrc r, unsigned voff, unsigned soff)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(voff), static_cast<int>(soff), 0);
    uint4v u;
    __builtin_memcpy(&u, &v, sizeof u);
    return u;
}
constexpr int kCoherent = 16;   // sc1: agent scope
template <int AUX = 0>
__device__ __forceinline__ float2v load8(brsrc r, unsigned voff, unsigned soff)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, static_cast<int>(voff), static_cast<int>(soff), AUX);
    float2v f;
    __builtin_memcpy(&f, &v, sizeof f);
    return f;
}
__device__ __forceinline__ void store8(brsrc r, unsigned voff, float2v f)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, f), r, static_cast<int>(voff), 0, kCoherent);
}
#else
__device__ inline void store8(brsrc, unsigned, float2v) {}
__device__ inline uint4v load16(brsrc, unsigned, unsigned) { return uint4v{}; }
constexpr int kCoherent = 0;
template <int AUX = 0>
__device__ inline float2v load8(brsrc, unsigned, unsigned) { return float2v{}; }
#endif

// Slot of start x in the a buffer (see above).
__device__ __forceinline__ int eslot(int x) { return x ^ ((x >> 1) & 8); }

struct SplitGeom {
    int nk, nw, W, nc;
};

template <int NV>
__device__ __forceinline__ void split_item(unsigned char *smem, const SplitGeom &g, const char *zh,
                                           const char *wtab, float2v *tout, int rs, int cg, int chunk,
                                           unsigned *done)
{
    using S = SplitShape<NV>;
    unsigned char *const ring = smem;
    unsigned char *const ebuf = smem + S::RING * S::COL;
    const int tid = threadIdx.x;
    const int lane = tid & 63, li = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int v = wave % NV, cw = wave / NV;
    const int seg = split_seg(g.nk);
    const int Wm1 = g.W - 1;
    int lo, hi;
    split_range(g.nw, g.nc, g.W, S::CB, cg, lo, hi);
    const int ch = split_chunk(g.W);
    const int iw0 = lo + chunk * ch;
    const int iw1 = min(iw0 + ch, hi + 1);
    if (chunk > 0 && iw0 > hi) return;   // this tile has fewer chunks

    const int k0 = cg * S::CB - (g.nw - 1);   // frequency of the tile's first column
    const int R0 = rs * S::RS;
    const int rows = min(S::RS, g.nk - R0);
    // the wave's row tiles: rt[1] = v-th from the end, rt[0] = v (if another)
    const int nt = (rows + 15) >> 4;
    const int rt[2] = {v, nt - 1 - v};
    const int col0 = cg * S::CB + 32 * cw + li;
    const int kw0 = col0 - (g.nw - 1);                   // frequency of the lane's first column
    const unsigned col_bytes = static_cast<unsigned>(seg) * 8u;   // of a column's four parts
    const unsigned ncw = 2u * Wm1 + 1u;
    const brsrc zr = make_brsrc(zh, ncw * col_bytes + 16u), wr = make_brsrc(wtab, ncw * ncw * 8u);

    // sums of the item, and of its last (up to kSplitGroup) columns
    float tre[2][2][4], tim[2][2][4], gre[2][2][4], gim[2][2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) tre[m][c][e] = tim[m][c][e] = gre[m][c][e] = gim[m][c][e] = 0.0f;

    // staging of the a column: thread t takes the starts t, t + 512, .. of the four parts
    constexpr int ET = (4 * S::NS + 511) / 512;
    // staging of a b column: threads 256 .. 256 + JB / 2 - 1 take 16 bytes each
    const int bt = tid - 256;
    constexpr int BG = S::JB / 8;
    const int bg = bt & (BG - 1), bp = bt / BG;
    const bool btask = bt >= 0 && bt < 4 * BG;

    const int n_pass = iw1 > iw0 ? (R0 + rows + S::JB - 1) / S::JB : 0;
    for (int J = 0; J < n_pass; ++J) {
        const int D = R0 - S::JB * J;
        // Lane offsets of the a column's starts (bytes from the column), and
        // their slots.  Starts whose eight values are all past the rows, and b
        // rows or columns that do not exist, read a column's eight zeros.
        unsigned e_off[ET];
#pragma unroll
        for (int i = 0; i < ET; ++i) {
            const int t = tid + 512 * i, p = t / S::NS, k = eslot(t - p * S::NS) + D - S::JB;
            e_off[i] = split_start(g.nk, p, k);
        }
        auto load_e = [&](int iw, uint4v (&x)[ET]) {
#pragma unroll
            for (int i = 0; i < ET; ++i) x[i] = load16(zr, e_off[i], static_cast<unsigned>(iw + Wm1) * col_bytes);
        };
        auto store_e = [&](int buf, const uint4v (&x)[ET]) {
#pragma unroll
            for (int i = 0; i < ET; ++i) {
                const int t = tid + 512 * i;
                if (t < 4 * S::NS) *reinterpret_cast<uint4v *>(ebuf + buf * S::EBUF + t * 16) = x[i];
            }
        };
        // 16 bytes of column jw: the thread's part and rows of the pass
        const unsigned b_off = split_start(g.nk, bp, S::JB * J + 8 * bg);
        auto load_b = [&](int jw) {
            const bool ok = jw > -g.W && jw < g.W;
            return load16(zr, ok ? b_off : 0u, ok ? static_cast<unsigned>(jw + Wm1) * col_bytes : 0u);
        };
        // the order of its eight values reversed, the im parts negated
        auto reversed = [](const uint4v &x, int p) {
            const unsigned sign = p >= 2 ? 0x80008000u : 0u;
            uint4v r;
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_alignbit(x[3 - i], x[3 - i], 16) ^ sign;
            return r;
        };
        // weights of the lane's two columns; scale_w drops those of no pair
        auto load_w = [&](int iw, float2v (&w)[2]) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int jw = kw0 + 16 * c - iw;
                w[c] = load8(wr, static_cast<unsigned>(min(max(jw + Wm1, 0), 2 * Wm1)) * 8u,
                             static_cast<unsigned>(iw + Wm1) * ncw * 8u);
            }
        };
        auto scale_w = [&](int iw, float2v (&w)[2]) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int jw = kw0 + 16 * c - iw;
                const bool ok = jw > -g.W && jw <= iw && kw0 + 16 * c < g.nw;
                const float f = ok ? (jw == iw ? 0.5f * kSplitUnscale : kSplitUnscale) : 0.0f;
                w[c].x *= f;
                w[c].y *= f;
            }
        };
        // the ring's first window: columns k0 - iw0 + n in slot n, n < CB
        for (int t = tid; t < S::CB * 4 * BG; t += 512) {
            const int gq = t & (BG - 1), p = (t / BG) & 3, n = t / (4 * BG);
            const int jw = k0 - iw0 + n, j = S::JB * J + 8 * gq;
            const bool ok = jw > -g.W && jw < g.W;
            const uint4v x = load16(zr, ok ? static_cast<unsigned>(jw + Wm1) * col_bytes + split_start(g.nk, p, j) : 0u, 0u);
            *reinterpret_cast<uint4v *>(ring + n * S::COL + p * S::PART + gq * 16) = reversed(x, p);
        }
        // weights of the products held, and of the next column
        float2v w[2] = {float2v{0.0f, 0.0f}, float2v{0.0f, 0.0f}}, wn[2];
        load_w(iw0, wn);
        {
            uint4v x[ET];
            load_e(iw0, x);
            store_e(0, x);
        }
        __syncthreads();

        // MFMA steps of the wave's tiles: 16 rt + 15 + D >= 32 ks, at most KS
        auto steps = [&](int r) { return min(S::KS, (16 * r + 15 + D) / 32 + 1); };
        const int n_hi = rt[1] >= v && 16 * rt[1] + 15 + D >= 0 ? steps(rt[1]) : 0;
        const int n_lo = rt[1] > v && 16 * v + 15 + D >= 0 ? steps(v) : 0;
        int slot[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) slot[c] = (32 * cw + 16 * c + li) * S::COL + lq * 16;
        int new_slot = (S::RING - 1) * S::COL;   // where the next iw's column goes
        int ea[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) ea[m] = eslot(16 * max(rt[m], 0) + li - 8 * lq + S::JB - 7) * 16;
        for (int iw = iw0; iw < iw1; ++iw) {
            const int buf = (iw - iw0) & 1;
            float4v pre[2][2], pia[2][2], pib[2][2];   // re = pre, im = pia - pib (the ring holds -im of b)
        // G += W P
        auto update = [&]() {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float pr = pre[m][c][e], pi = pia[m][c][e] - pib[m][c][e];
                        gre[m][c][e] = __builtin_fmaf(w[c].x, pr, gre[m][c][e]);
                        gre[m][c][e] = __builtin_fmaf(-w[c].y, pi, gre[m][c][e]);
                        gim[m][c][e] = __builtin_fmaf(w[c].x, pi, gim[m][c][e]);
                        gim[m][c][e] = __builtin_fmaf(w[c].y, pr, gim[m][c][e]);
                    }
        };
            const bool more = iw + 1 < iw1;
            uint4v ex[ET], bx;
            if (more) {
                load_e(iw + 1, ex);
                if (btask) bx = load_b(k0 - iw - 1);
            }
            {
                const unsigned char *eb = ebuf + buf * S::EBUF;
                // operands of one step: parts re hi, re lo, im hi, im lo
                half8 a0[4], a1[4], b[2][4];
                auto load_bf = [&](half8 (&bf)[2][4], int ks) {
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            bf[c][p] = *reinterpret_cast<const half8 *>(ring + slot[c] + p * S::PART + ks * 64);
                };
                auto load_af = [&](half8 (&af)[4], int m, int ks) {
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        af[p] = *reinterpret_cast<const half8 *>(eb + ea[m] + p * S::EPART - ks * 512);
                };
                auto tile_step = [&](auto first, int m, const half8 (&af)[4]) {
                    constexpr bool FIRST = decltype(first)::value;
                    const float4v zero{0.0f, 0.0f, 0.0f, 0.0f};
#define SRM3_MF(x, y, acc) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, acc, 0, 0, 0)
#define SRM3_MF0(x, y, acc) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, FIRST ? zero : acc, 0, 0, 0)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        SRM3_MF0(af[1], b[c][0], pre[m][c]);
                        SRM3_MF0(af[1], b[c][2], pib[m][c]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        SRM3_MF(af[0], b[c][1], pre[m][c]);
                        SRM3_MF(af[0], b[c][3], pib[m][c]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        SRM3_MF(af[0], b[c][0], pre[m][c]);
                        SRM3_MF(af[0], b[c][2], pib[m][c]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        SRM3_MF(af[3], b[c][2], pre[m][c]);
                        SRM3_MF0(af[3], b[c][0], pia[m][c]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        SRM3_MF(af[2], b[c][3], pre[m][c]);
                        SRM3_MF(af[2], b[c][1], pia[m][c]);
                    }
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        SRM3_MF(af[2], b[c][2], pre[m][c]);
                        SRM3_MF(af[2], b[c][0], pia[m][c]);
                    }
#undef SRM3_MF
#undef SRM3_MF0
                };
                // steps of both tiles, then those of tile 1 alone (operands
                // requested past the last step are unused entries)
                auto step_both = [&](auto first, int ks) {
                    load_af(a0, 0, ks);
                    __builtin_amdgcn_sched_barrier(0);
                    tile_step(first, 1, a1);
                    load_af(a1, 1, ks + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    tile_step(first, 0, a0);
                    load_bf(b, ks + 1);
                };
                auto step_one = [&](auto first, int ks) {
                    tile_step(first, 1, a1);
                    load_bf(b, ks + 1);
                    load_af(a1, 1, ks + 1);
                };
                load_bf(b, 0);
                load_af(a1, 1, 0);
                int ks = 1;
                step_both(std::true_type{}, 0);   // (every wave: a tile it does not have is not stored)
                for (; ks < n_lo; ++ks) step_both(std::false_type{}, ks);
                for (; ks < n_hi; ++ks) step_one(std::false_type{}, ks);
                scale_w(iw, wn);
                w[0] = wn[0];
                w[1] = wn[1];
                if (more) load_w(iw + 1, wn);
                update();
                if (((iw - iw0) & (kSplitGroup - 1)) == kSplitGroup - 1 || !more) {
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int c = 0; c < 2; ++c)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                tre[m][c][e] += gre[m][c][e];
                                tim[m][c][e] += gim[m][c][e];
                                gre[m][c][e] = gim[m][c][e] = 0.0f;
                            }
                }
            }
            if (more) {
                store_e(buf ^ 1, ex);
                if (btask) *reinterpret_cast<uint4v *>(ring + new_slot + bp * S::PART + bg * 16) = reversed(bx, bp);
                new_slot = new_slot == 0 ? (S::RING - 1) * S::COL : new_slot - S::COL;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    slot[c] -= S::COL;
                    if (slot[c] < 0) slot[c] += S::RING * S::COL;
                }
            }
            __syncthreads();
        }
    }

    // commit: add to the sums of the chunks before this one
    if (chunk > 0) {
        if (tid == 0) wait_count(done, static_cast<unsigned>(chunk));
        __syncthreads();
    }
    // (lines outside the grid get an offset past the buffer: they load zero and are not stored)
    const brsrc tr = make_brsrc(tout, static_cast<unsigned>(g.nk) * static_cast<unsigned>(g.nc) * 8u);
    auto offset = [&](int m, int c, int e) {
        const int kk = R0 + 16 * rt[m] + 4 * lq + e, col = col0 + 16 * c;
        const bool ok = rt[1] >= v && (m == 1 || rt[1] > v) && kk < g.nk && col < g.nc;
        return ok ? (static_cast<unsigned>(kk) * static_cast<unsigned>(g.nc) + static_cast<unsigned>(col)) * 8u : ~15u;
    };
    float2v old[2][2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) old[m][c][e] = chunk > 0 ? load8<kCoherent>(tr, offset(m, c, e), 0u) : float2v{0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                store8(tr, offset(m, c, e), float2v{__builtin_fmaf(tre[m][c][e], kSplitUnscale, old[m][c][e].x),
                                                    __builtin_fmaf(tim[m][c][e], kSplitUnscale, old[m][c][e].y)});
    wait_stores();
    __syncthreads();
    if (tid == 0) set_count(done, static_cast<unsigned>(chunk + 1));
}

// Row waves of a tile: the fewest that hold the grid's rows (64, 128, 256),
// so that small grids do not multiply rows they do not have.
__host__ __device__ inline int split_nv(int nk) { return nk <= 64 ? 2 : (nk <= 128 ? 4 : 8); }
__host__ __device__ inline int split_cols(int nk) { return 256 / split_nv(nk); }

template <int NV>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void pairsum_split_kernel(SplitArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_item[2];
    for (int turn = 0;; turn ^= 1) {
        // (two slots: a skipped item has no barrier between its read and the next write)
        if (threadIdx.x == 0) s_item[turn] = static_cast<int>(atomicAdd(a.queue, 1u));
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(s_item[turn]);
        if (item >= a.n_items) return;
        SplitGeom g;
        int rs, cg, chunk, tile;
        const char *zh, *wtab;
        float2v *tout;
        if (a.items) {
            const PItem it = a.items[item];
            const PReq &r = a.reqs[__builtin_amdgcn_readfirstlane(it.req)];
            g = SplitGeom{__builtin_amdgcn_readfirstlane(r.g.nk), __builtin_amdgcn_readfirstlane(r.g.nw),
                          __builtin_amdgcn_readfirstlane(r.g.W), __builtin_amdgcn_readfirstlane(r.g.nc)};
            rs = __builtin_amdgcn_readfirstlane(it.kb & 0xFFFF);
            chunk = __builtin_amdgcn_readfirstlane(it.kb >> 16);
            cg = __builtin_amdgcn_readfirstlane(it.cg);
            tile = __builtin_amdgcn_readfirstlane(it.pad);
            zh = uniform_ptr(static_cast<const char *>(r.zcol));
            wtab = uniform_ptr(static_cast<const char *>(r.wtab));
            tout = uniform_ptr(static_cast<float2v *>(r.tsum));
        } else {
            g = SplitGeom{a.g.nk, a.g.nw, a.g.W, a.g.nc};
            chunk = item / a.tiles;
            tile = item - chunk * a.tiles;
            // heaviest row tiles first, realizations innermost
            const int batch = a.tiles / (a.n_rs * a.n_cg);
            const int t = tile / batch, b = tile - t * batch;
            rs = a.n_rs - 1 - t / a.n_cg;
            cg = t - (t / a.n_cg) * a.n_cg;
            zh = static_cast<const char *>(a.zh) + static_cast<size_t>(b) * split_operand_bytes(g.nk, 2 * g.W - 1);
            wtab = static_cast<const char *>(a.wtab);
            tout = static_cast<float2v *>(a.tout) + static_cast<long>(b) * g.nk * g.nc;
        }
        split_item<NV>(smem, g, zh, wtab, tout, rs, cg, chunk, a.done + tile);
    }
}

int split_row_tiles(const Geometry &g) { return (g.nk + 32 * split_nv(g.nk) - 1) / (32 * split_nv(g.nk)); }
int split_col_tiles(const Geometry &g) { return (g.nc + split_cols(g.nk) - 1) / split_cols(g.nk); }

template <int NV>
hipError_t launch_split_t(const SplitArgs &a, hipStream_t st)
{
    // one block per CU (LDS)
    const int blocks = std::min(a.n_items, kCus);
    pairsum_split_kernel<NV><<<dim3(static_cast<unsigned>(blocks)), 512, SplitShape<NV>::LDS, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_split(int nv, const SplitArgs &a, hipStream_t st)
{
    switch (nv) {
    case 2: return launch_split_t<2>(a, st);
    case 4: return launch_split_t<4>(a, st);
    default: return launch_split_t<8>(a, st);
    }
}

template <int NV>
hipError_t prepare_split_t()
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&pairsum_split_kernel<NV>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, SplitShape<NV>::LDS);
}

}  // namespace

// Below 32 rows half of every 64-row tile would be idle and the operand region
// too small.
bool split_supported(const Geometry &g, int precision) { return precision == SRM3_FP32 && g.nk >= kSplitMinRows; }

hipError_t launch_phases_split(const Geometry &g, const uint64_t *seeds, const uint64_t *seeds_dev, int batch,
                               const Workspace &ws, const double *lr, hipStream_t st)
{
    const int chunk = seeds_dev ? 65535 : kMaxSeedsPerLaunch;
    for (int b0 = 0; b0 < batch; b0 += chunk) {
        const int nb = std::min(chunk, batch - b0);
        SeedChunk sc{};
        if (!seeds_dev)
            for (int i = 0; i < nb; ++i) sc.s[i] = seeds[b0 + i];
        const int kwb = 4 * floor_div4(-(g.nw - 1));
        const unsigned gx = static_cast<unsigned>((g.nw - kwb + 63) / 64);
        const unsigned gy = static_cast<unsigned>((split_nk8(g.nk) + 63) / 64);
        phase_split_kernel<<<dim3(gx, gy, nb), 256, 0, st>>>(sc, seeds_dev, b0, g, static_cast<float2 *>(ws.zrow),
                                                             static_cast<_Float16 *>(ws.zcol), lr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pairsum_split(const Geometry &g, const void *wtab, int batch, const Workspace &ws, hipStream_t st)
{
    const int cb = split_cols(g.nk);
    SplitArgs a{};
    a.zh = ws.zcol;
    a.wtab = wtab;
    a.tout = ws.tsum;
    a.g = g;
    a.n_rs = split_row_tiles(g);
    a.n_cg = split_col_tiles(g);
    a.tiles = batch * a.n_rs * a.n_cg;
    int chunks = 1;
    for (int cg = 0; cg < a.n_cg; ++cg) chunks = std::max(chunks, split_chunks(g, cb, cg));
    a.n_items = a.tiles * chunks;
    // the counters live in the transform workspace, which nothing uses before the t-transform
    a.queue = static_cast<unsigned *>(ws.g);
    a.done = a.queue + 1;
    const hipError_t e = launch_fill_u32(a.queue, 1 + static_cast<size_t>(a.tiles), 0u, st);
    if (e != hipSuccess) return e;
    return launch_split(split_nv(g.nk), a, st);
}

hipError_t launch_pairsum_split_items(const void *reqs, const void *items, const WorkItems &n, int tiles,
                                      unsigned *counters, hipStream_t st)
{
    hipError_t e = launch_fill_u32(counters, split_counter_words(tiles), 0u, st);
    SplitArgs a{};
    a.reqs = static_cast<const PReq *>(reqs);
    a.done = counters + kSplitShapes;
    for (int i = 0; i < kSplitShapes && e == hipSuccess; ++i) {
        a.items = static_cast<const PItem *>(items) + n.begin[i];
        a.n_items = n.begin[i + 1] - n.begin[i];
        a.queue = counters + i;
        if (a.n_items > 0) e = launch_split(8 >> i, a, st);
    }
    return e;
}

int split_shape(const Geometry &g) { return split_nv(g.nk) == 8 ? 0 : (split_nv(g.nk) == 4 ? 1 : 2); }

std::vector<WorkTile> split_tiles(const Geometry &g, int req)
{
    const int rsize = 32 * split_nv(g.nk), cb = split_cols(g.nk);
    std::vector<WorkTile> v;
    for (int rs = 0; rs < split_row_tiles(g); ++rs) {
        const double r0 = static_cast<double>(rs) * rsize, r1 = std::min<double>(g.nk, r0 + rsize);
        for (int cg = 0; cg < split_col_tiles(g); ++cg) {
            int lo, hi;
            split_range(g.nw, g.nc, g.W, cb, cg, lo, hi);
            const double terms = 0.5 * (r1 * (r1 + 1) - r0 * (r0 + 1)) * cb * std::max(1, hi - lo + 1);
            v.push_back({req, rs, cg, split_chunks(g, cb, cg), terms});
        }
    }
    std::stable_sort(v.begin(), v.end(), [](const WorkTile &a, const WorkTile &b) { return a.cost > b.cost; });
    return v;
}

void WorkList::add(int shape, const std::vector<WorkTile> &tiles)
{
    double c = 0.0;
    for (const WorkTile &t : tiles) c += t.cost;
    if (!tiles.empty()) runs_[shape].push_back({tiles, c});
    n_tiles_ += static_cast<int>(tiles.size());
}

std::vector<unsigned char> WorkList::items(WorkItems *n)
{
    std::vector<PItem> out;
    int tile0 = 0;
    for (int i = 0; i < kSplitShapes; ++i) {
        n->begin[i] = static_cast<int>(out.size());
        std::stable_sort(runs_[i].begin(), runs_[i].end(), [](const Run &a, const Run &b) { return a.cost > b.cost; });
        for (const Run &r : runs_[i]) {
            int chunks = 1;
            for (const WorkTile &t : r.tiles) chunks = std::max(chunks, t.items());
            for (int c = 0; c < chunks; ++c)
                for (size_t k = 0; k < r.tiles.size(); ++k) {
                    const WorkTile &t = r.tiles[k];
                    const int chunk = t.chunks == 0 ? kTileWhole : c;
                    if (c < t.items())
                        out.push_back({t.req, t.rs | static_cast<int>(static_cast<unsigned>(chunk) << 16), t.cg, tile0 + static_cast<int>(k)});
                }
            tile0 += static_cast<int>(r.tiles.size());
        }
    }
    n->begin[kSplitShapes] = static_cast<int>(out.size());
    std::vector<unsigned char> bytes(out.size() * sizeof(PItem));
    if (!out.empty()) std::memcpy(bytes.data(), out.data(), bytes.size());
    return bytes;
}

hipError_t prepare_split()
{
    hipError_t e = prepare_split_t<2>();
    if (e == hipSuccess) e = prepare_split_t<4>();
    if (e == hipSuccess) e = prepare_split_t<8>();
    return e;
}

}  // namespace srm3
