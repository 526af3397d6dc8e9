// The FP64 direct-form pair sum on the matrix cores (see srm3_mfma.hpp for the
// products): tiles of 16 RT rows x 16 CT columns of outputs, the partner columns
// in chunks, a chunk to a block of four waves.
//
// A tile's sum is that of its chunks in order, a chunk's that of its four
// quarters in order; both partitions depend on the grid alone, so a realization
// has the same bits in every launch.  An item is a chunk, added to the tile's
// sum in memory after the chunk before it (an ordered addition, about 10 us from
// one block to the next); or a chunk whose sum goes to a slab of its own, the
// slabs being added afterwards; or a whole tile.  Items with ordered additions
// are taken from a queue in order, chunk by chunk over all tiles, so the first
// unfinished one waits for nothing; the others are the launch's blocks.
//
// Bound by the FP64 matrix cores where rows and realizations fill them (256x1024
// lines, 64 realizations: 318 ms, 62 TFLOP/s in the three products of a pair
// term) and by the chain of additions and its tail in small calls.
// With a wave to a chunk instead, each chunk added to memory by its wave (four
// times the additions; batches and the server ran whole tiles, one wave each):
// that batch 328 ms, 32x64 lines x 64 0.31 ms (now 0.10), 16x333 x 8 1.07
// (0.10), 24 mixed grids of 64x128 to 256x1024 in a batch 64 (20.5).
#include <algorithm>

#include "srm3_mfma.hpp"

namespace srm3 {

namespace {

constexpr int kWaves = 4;
constexpr int kWholeWork = 160;   // see whole_tiles

// Most partner columns of a chunk, by the grid alone.  The smallest grids take
// 32 (the four-column steps of an MFMA, two to a wave), or 64 where these would
// be many in a row: 32x64 lines, one realization, 0.054 ms (64: 0.066, 16:
// 0.049), 64x64 0.067 (0.091, 0.056; 64 realizations 0.203, 0.198, 0.214), but
// 24x333 x 8 0.32 (0.19).  Above, 128 while a tile has few kappa splits to a
// column, 64 from 64 rows on: 32x1024, one realization, 0.23 (64: 0.44), 64x512
// 0.23 (0.19), 256x128 0.43 (0.25), 256x1024 x 16 79.7 (78.8).  The line between
// the two: 32x128 with 128 0.091 (32: 0.056), 32x333 x 8 with 32 0.33 (128: 0.18).
__host__ __device__ inline int f64_chunk_max(const Geometry &g)
{
    if (g.nk < 8) return 128;   // (a chunk of 32 is hardly longer than the meeting of its waves)
    if (g.nk * g.nc <= 16384) return g.ncw <= 256 ? 32 : 64;
    return g.nk < 64 ? 128 : 64;
}

// The chunks of the column tile from column c0 on: partner columns lo .. hi in
// `chunks` chunks of 4 sub columns, a quarter (sub, a multiple of 4) for each
// wave.  By the grid alone, so that the sums are the same in every launch.
struct F64Range {
    int lo, hi, sub, chunks;
};

__host__ __device__ inline F64Range f64_range(const Geometry &g, int c0, int cols)
{
    const int Wm1 = g.W - 1;
    const int k0 = c0 - (g.nw - 1), k1 = (c0 + cols - 1 < g.nc - 1 ? c0 + cols - 1 : g.nc - 1) - (g.nw - 1);
    F64Range r;
    r.lo = k0 - Wm1 > -Wm1 ? k0 - Wm1 : -Wm1;
    r.hi = k1 + Wm1 < Wm1 ? k1 + Wm1 : Wm1;
    const int n = r.hi >= r.lo ? r.hi - r.lo + 1 : 1;
    const int m = (n + f64_chunk_max(g) - 1) / f64_chunk_max(g);
    r.sub = (n + 16 * m - 1) / (16 * m) * 4;
    r.chunks = (n + 4 * r.sub - 1) / (4 * r.sub);
    return r;
}

struct F64Args {
    const void *zrow;   // [B][nk][nc] double2
    const void *zcol;   // [B][ncw][nkp][4] double
    const void *wtab;   // [ncw][ncw] double2
    void *tout;         // [B][nk][nc] double2
    Geometry g;
    int batch, n_rg, n_ct;
    int tiles;          // batch * n_rg * n_ct
    int n_items;        // tiles, or tiles * chunks of the widest
    int whole;          // an item is a whole tile
    unsigned *queue;    // next item, zero at launch; or null: item blockIdx.x (no additions in order)
    unsigned *done;     // chunks added per tile, zero at launch
    double2 *slabs;     // or null: [chunks][batch][nk][nc], each chunk's sums apart (added by sum_slabs_kernel)
    const PReq *reqs;   // with items: the requests and their work list
    const PItem *items;
};

// One tile's chunks chunk0 .. chunk1 - 1.  The waves' sums of a chunk meet in
// LDS, row tile by row tile, and are added in their order; every thread has CT
// outputs of each row tile.  ordered: added onto the sums of the chunks before
// in tout, counted by `done`.
template <int RT, int CT>
__device__ __forceinline__ void f64_item(double2 *red, const Geometry &g, const double2 *zrow, const double *zcol,
                                         const double2 *wtab, double2 *tout, int rg, int c0, const F64Range &rng,
                                         int chunk0, int chunk1, bool ordered, unsigned *done)
{
    using M = MfmaT<double>;
    using V4 = M::v4;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K0 = 16 * RT * rg;
    double2 *const tot = red + kWaves * CT * 256 + tid;   // (in registers it would spill)
    for (int chunk = chunk0; chunk < chunk1; ++chunk) {
        V4 P1[RT][CT], P2[RT][CT], P3[RT][CT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) P1[r][c] = P2[r][c] = P3[r][c] = V4{0.0, 0.0, 0.0, 0.0};
        const int i0 = rng.lo + (4 * chunk + wave) * rng.sub;
        mfma_columns<double, RT, CT, true>(g, zrow, zcol, wtab, rg, c0, i0, min(rng.hi, i0 + rng.sub - 1), P1, P2, P3,
                                           [](int) {});
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (r > 0 || chunk > chunk0) __syncthreads();   // the reads of the sums before
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    red[((wave * CT + c) * 4 + e) * 64 + lane] =
                        make_double2(P1[r][c][e] - P2[r][c][e], P1[r][c][e] + P3[r][c][e]);
            __syncthreads();
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                double2 s = red[c * 256 + tid];   // (thread: element tid / 64 of lane tid % 64)
#pragma unroll
                for (int w = 1; w < kWaves; ++w) {
                    const double2 x = red[(w * CT + c) * 256 + tid];
                    s.x += x.x;
                    s.y += x.y;
                }
                if (chunk > chunk0) {
                    const double2 t = tot[(r * CT + c) * 256];
                    s.x += t.x;
                    s.y += t.y;
                }
                tot[(r * CT + c) * 256] = s;
            }
        }
    }
    if (ordered && chunk0 > 0) {
        if (tid == 0) wait_count(done, static_cast<unsigned>(chunk0));
        __syncthreads();
    }
    double2 old[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            old[r][c] = make_double2(0.0, 0.0);
            const int kk = K0 + 16 * r + M::drow(lq, wave), col = c0 + 16 * c + li;
            if (ordered && chunk0 > 0 && kk < g.nk && col < g.nc) {
                const double2 *p = tout + static_cast<long>(kk) * g.nc + col;
                old[r][c].x = coherent_load(&p->x);
                old[r][c].y = coherent_load(&p->y);
            }
        }
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int kk = K0 + 16 * r + M::drow(lq, wave), col = c0 + 16 * c + li;
            if (kk >= g.nk || col >= g.nc) continue;
            double2 v = tot[(r * CT + c) * 256];
            double2 *p = tout + static_cast<long>(kk) * g.nc + col;
            if (!ordered) {
                *p = v;
                continue;
            }
            if (chunk0 > 0) {
                v.x += old[r][c].x;
                v.y += old[r][c].y;
            }
            coherent_store(&p->x, v.x);
            coherent_store(&p->y, v.y);
        }
    if (ordered) wait_stores();
    __syncthreads();   // (and the reads of `red`)
    if (ordered && tid == 0) set_count(done, static_cast<unsigned>(chunk1));
}

template <int RT, int CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void pairsum_f64_kernel(F64Args a)
{
    __shared__ double2 red[(kWaves + RT) * CT * 256];   // the waves' sums of a row tile, and the tile's
    __shared__ int s_item[2];
    for (int turn = 0;; turn ^= 1) {
        // (two slots: a skipped item has no barrier between its read and the next write)
        int item = static_cast<int>(blockIdx.x);
        if (a.queue) {
            if (threadIdx.x == 0) s_item[turn] = static_cast<int>(atomicAdd(a.queue, 1u));
            __syncthreads();
            item = __builtin_amdgcn_readfirstlane(s_item[turn]);
        } else if (turn) {
            return;
        }
        if (item >= a.n_items) return;
        int rg, ct, chunk, tile;
        if (a.items) {
            const PItem it = a.items[item];
            const PReq &q = a.reqs[__builtin_amdgcn_readfirstlane(it.req)];
            const Geometry g = q.g;
            rg = __builtin_amdgcn_readfirstlane(it.kb & 0xFFFF);
            chunk = __builtin_amdgcn_readfirstlane(it.kb >> 16);   // kTileWhole: all
            ct = __builtin_amdgcn_readfirstlane(it.cg);
            tile = __builtin_amdgcn_readfirstlane(it.pad);
            const F64Range rng = f64_range(g, 16 * CT * ct, 16 * CT);
            const bool whole = chunk == kTileWhole;
            f64_item<RT, CT>(red, g, static_cast<const double2 *>(uniform_ptr(q.zrow)),
                             static_cast<const double *>(uniform_ptr(q.zcol)),
                             static_cast<const double2 *>(uniform_ptr(q.wtab)),
                             static_cast<double2 *>(uniform_ptr(q.tsum)), rg, 16 * CT * ct, rng, whole ? 0 : chunk,
                             whole ? rng.chunks : chunk + 1, !whole, a.done + tile);
            continue;
        }
        chunk = a.whole ? 0 : item / a.tiles;
        tile = item - chunk * a.tiles;
        // heaviest row groups first, realizations innermost
        const int k = tile / a.batch, b = tile - k * a.batch;
        rg = a.n_rg - 1 - k / a.n_ct;
        ct = k - (k / a.n_ct) * a.n_ct;
        const Geometry &g = a.g;
        const F64Range rng = f64_range(g, 16 * CT * ct, 16 * CT);
        if (!a.whole && chunk >= rng.chunks) continue;
        const long lines = static_cast<long>(g.nk) * g.nc, plane = static_cast<long>(g.ncw) * g.nkp;
        f64_item<RT, CT>(red, g, static_cast<const double2 *>(a.zrow) + b * lines,
                         static_cast<const double *>(a.zcol) + b * ALayout<double>::NS * plane,
                         static_cast<const double2 *>(a.wtab),
                         a.slabs ? a.slabs + (static_cast<long>(chunk) * a.batch + b) * lines
                                 : static_cast<double2 *>(a.tout) + b * lines,
                         rg, 16 * CT * ct, rng, chunk, a.whole ? rng.chunks : chunk + 1, !a.whole && !a.slabs,
                         a.done + tile);
    }
}

// The chunks' sums, added in the order of the other forms.
__global__ __launch_bounds__(256) void sum_slabs_kernel(const double2 *__restrict__ slabs, Geometry g, int batch,
                                                        int cols, double2 *__restrict__ tout)
{
    const long n = static_cast<long>(batch) * g.nk * g.nc;
    const long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const int col = static_cast<int>(i % g.nc);
    const int chunks = f64_range(g, col / cols * cols, cols).chunks;
    double2 t = slabs[i];
    for (int c = 1; c < chunks; ++c) {
        const double2 x = slabs[c * n + i];
        t.x += x.x;
        t.y += x.y;
    }
    tout[i] = t;
}

int widest_chunks(const Geometry &g, int cols)
{
    int chunks = 1;
    for (int c0 = 0; c0 < g.nc; c0 += cols) chunks = std::max(chunks, f64_range(g, c0, cols).chunks);
    return chunks;
}

// Work of a tile: pair terms of its live row tiles, empty parts of products included.
double tile_cost(const Geometry &g, int rt, int cols, int rg, int ct)
{
    const F64Range r = f64_range(g, cols * ct, cols);
    const int live = std::min(rt, (g.nk - 16 * rt * rg + 15) / 16);
    return static_cast<double>(std::min(16 * rt * (rg + 1) - 1, g.nk - 1) / 2 + 1) * 16 * live * cols * std::max(1, r.hi - r.lo + 1);
}

// Whether the grid's tiles are run whole, by one block each: where the work of
// a chunk (kappa splits x row tiles x columns of a wave, of the heaviest tile)
// is short beside an ordered addition, or, in launches of many tiles, not long.
// 12x333 lines, 64 realizations: whole 0.38 ms, chunks 0.41; 8x333 x 512 1.87,
// 2.47; 1x4096 x 64 12.9, 25.5; 32x64 x 512 0.41, 0.43; but 16x1024 x 8 0.67,
// 0.58 and 24x333 x 8 0.31, 0.19.
bool whole_tiles(const Geometry &g, const MfmaShape &m, long tiles)
{
    const int rg = (g.nk - 1) / (16 * m.rt), cols = 16 * m.ct;
    const int live = (g.nk - 16 * m.rt * rg + 15) / 16;
    int sub = 4;
    for (int c0 = 0; c0 < g.nc; c0 += cols) sub = std::max(sub, f64_range(g, c0, cols).sub);
    const long work = static_cast<long>((g.nk - 1) / 2 + 1) * live * sub;
    return widest_chunks(g, cols) == 1 || work <= kWholeWork || (work <= 2 * kWholeWork && tiles >= 6 * kCus);
}

template <int RT, int CT>
hipError_t launch_t(const F64Args &a, hipStream_t st)
{
    const int blocks = a.queue ? std::min(a.n_items, 3 * kCus) : a.n_items;
    pairsum_f64_kernel<RT, CT><<<dim3(static_cast<unsigned>(blocks)), 64 * kWaves, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_shape(int shape, const F64Args &a, hipStream_t st)
{
    switch (shape) {
    case 1: return launch_t<2, 1>(a, st);
    case 2: return launch_t<1, 2>(a, st);
    default: return launch_t<2, 2>(a, st);
    }
}

}  // namespace

size_t f64_slab_bytes(const Geometry &g, int shape, int batch)
{
    const int chunks = widest_chunks(g, 16 * mfma_shape(SRM3_FP64, shape).ct);
    return chunks > 1 ? static_cast<size_t>(chunks) * batch * g.nk * g.nc * sizeof(double2) : 0;
}

hipError_t launch_pairsum_f64(const Geometry &g, int shape, const void *wtab, int batch, const Workspace &ws,
                              const Slabs &slabs, hipStream_t st)
{
    const MfmaShape m = mfma_shape(SRM3_FP64, shape);
    const int cols = 16 * m.ct;
    F64Args a{};
    a.wtab = wtab;
    a.g = g;
    a.n_rg = (g.nk + 16 * m.rt - 1) / (16 * m.rt);
    a.n_ct = (g.nc + cols - 1) / cols;
    const int chunks = widest_chunks(g, cols);
    const bool slabs_fit = chunks > 1 && slabs.p && f64_slab_bytes(g, shape, batch) <= slabs.n;
    // (slabs where whole tiles would leave CUs idle: 8x64 lines, one realization,
    // 0.042 ms, whole 0.068; 64 realizations, 256 tiles, 0.070, whole 0.058)
    const long all = static_cast<long>(batch) * a.n_rg * a.n_ct;
    a.whole = whole_tiles(g, m, all) && !(slabs_fit && all < kCus);
    const long lines = static_cast<long>(g.nk) * g.nc, n = lines * batch;
    if (!a.whole && slabs_fit) a.slabs = static_cast<double2 *>(slabs.p);
    // realizations of one launch: its items are counted in 32 bits
    const int per = mfma_queue_batch(static_cast<long>(a.n_rg) * a.n_ct * chunks);
    for (int b0 = 0; b0 < batch; b0 += per) {
        a.batch = std::min(per, batch - b0);
        a.zrow = static_cast<const double2 *>(ws.zrow) + b0 * lines;
        a.zcol = static_cast<const double *>(ws.zcol) + b0 * static_cast<long>(a_slots(SRM3_FP64)) * g.ncw * g.nkp;
        a.tout = static_cast<double2 *>(ws.tsum) + b0 * lines;
        a.tiles = a.batch * a.n_rg * a.n_ct;
        a.n_items = a.whole ? a.tiles : a.tiles * chunks;
        hipError_t e = hipSuccess;
        if (!a.whole && !a.slabs) {
            // the counters live in the transform workspace, which nothing uses before the t-transform
            a.queue = static_cast<unsigned *>(ws.g);
            a.done = a.queue + 1;
            e = launch_fill_u32(a.queue, f64_counter_words(a.tiles), 0u, st);
        }
        if (e == hipSuccess) e = launch_shape(shape, a, st);
        if (e != hipSuccess) return e;
    }
    if (a.slabs)   // (one launch: they hold the whole call)
        sum_slabs_kernel<<<dim3(static_cast<unsigned>((n + 255) / 256)), 256, 0, st>>>(a.slabs, g, batch, cols,
                                                                                        static_cast<double2 *>(ws.tsum));
    return hipGetLastError();
}

hipError_t launch_pairsum_f64_items(int shape, const void *reqs, const void *items, int n_items, int tiles,
                                    unsigned *counters, hipStream_t st)
{
    const hipError_t e = launch_fill_u32(counters, f64_counter_words(tiles), 0u, st);
    if (e != hipSuccess) return e;
    F64Args a{};
    a.reqs = static_cast<const PReq *>(reqs);
    a.items = static_cast<const PItem *>(items);
    a.n_items = n_items;
    a.queue = counters;
    a.done = counters + 1;
    return launch_shape(shape, a, st);
}

std::vector<WorkTile> f64_tiles(const Geometry &g, int shape, int req)
{
    const MfmaShape m = mfma_shape(SRM3_FP64, shape);
    const int cols = 16 * m.ct;
    const bool whole = whole_tiles(g, m, 0);
    std::vector<WorkTile> v;
    for (int rg = 0; rg * 16 * m.rt < g.nk; ++rg)
        for (int ct = 0; ct * cols < g.nc; ++ct)
            v.push_back({req, rg, ct, whole ? 0 : f64_range(g, cols * ct, cols).chunks, tile_cost(g, m.rt, cols, rg, ct)});
    std::stable_sort(v.begin(), v.end(), [](const WorkTile &a, const WorkTile &b) { return a.cost > b.cost; });
    return v;
}

}  // namespace srm3
