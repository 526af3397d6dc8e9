// Device pieces shared by the kernel sources: phase factors of lines and the
// descriptors of persistent work lists.
#pragma once

#include "srm3_internal.hpp"

namespace srm3 {

// Read-only data that does not change while a kernel runs, in the constant
// address space: uniform loads through such a pointer become scalar loads even
// where the kernel stores elsewhere earlier (the persistent loop).
// (The host pass of the compiler only parses kernel bodies; it sees plain
// pointers.)
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;
#else
template <typename T>
using cptr = const T *;
#endif

template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T *p)
{
    return (cptr<T>)p;
}

// A pointer that every lane of the wave holds, taken from the first lane so
// that address arithmetic on it stays scalar.
template <typename T>
__device__ __forceinline__ T *uniform_ptr(T *p)
{
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v));
    const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v >> 32));
    return reinterpret_cast<T *>((static_cast<unsigned long long>(hi) << 32) | lo);
}

// Device memory in the global address space: loads through such a pointer are
// global (not flat) loads also where the pointer itself was read from memory.
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using gptr = const __attribute__((address_space(1))) T *;
template <typename T>
using gmut = __attribute__((address_space(1))) T *;
#else
template <typename T>
using gptr = const T *;
template <typename T>
using gmut = T *;
#endif

// Buffer loads: a uniform resource, a per-lane byte offset and a uniform byte
// offset, so stepping the uniform one costs no vector address arithmetic.  A
// per-lane offset past the buffer loads zero; the uniform offset takes no part
// in that check, so it stays within the buffer.
#if defined(__HIP_DEVICE_COMPILE__)
using brsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ brsrc make_brsrc(const void *p, unsigned bytes)
{
    // the resource lives in scalar registers (the base is wave-uniform);
    // word 3 of a gfx9 raw buffer resource: 32-bit data format, no swizzle
    return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(const_cast<void *>(p)), static_cast<short>(0),
                                             static_cast<int>(__builtin_amdgcn_readfirstlane(bytes)), 0x00020000);
}
#else
struct brsrc {
    const void *p;
};
__device__ inline brsrc make_brsrc(const void *p, unsigned) { return brsrc{p}; }
#endif

#if defined(__HIP_DEVICE_COMPILE__)
// (The loaded vector is copied out whole: extracting its lanes one by one has
// been folded by the compiler into a single-dword load.)
__device__ __forceinline__ float2 bload(brsrc r, unsigned voff, unsigned soff, float)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, static_cast<int>(voff), static_cast<int>(soff), 0);
    static_assert(sizeof(v) == sizeof(float2), "b64 load is two floats");
    float2 f;
    __builtin_memcpy(&f, &v, sizeof(f));
    return f;
}
__device__ __forceinline__ double2 bload(brsrc r, unsigned voff, unsigned soff, double)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(voff), static_cast<int>(soff), 0);
    static_assert(sizeof(v) == sizeof(double2), "b128 load is two doubles");
    double2 d;
    __builtin_memcpy(&d, &v, sizeof(d));
    return d;
}
__device__ __forceinline__ float bload32(brsrc r, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, static_cast<int>(voff),
                                                                          static_cast<int>(soff), 0));
}
__device__ __forceinline__ double bload64(brsrc r, unsigned voff, unsigned soff)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, static_cast<int>(voff), static_cast<int>(soff), 0);
    double d;
    __builtin_memcpy(&d, &v, sizeof(d));
    return d;
}
#else
__device__ inline float2 bload(brsrc, unsigned, unsigned, float) { return float2{}; }
__device__ inline double2 bload(brsrc, unsigned, unsigned, double) { return double2{}; }
__device__ inline float bload32(brsrc, unsigned, unsigned) { return 0.0f; }
__device__ inline double bload64(brsrc, unsigned, unsigned) { return 0.0; }
#endif

// ---------------------------------------------------------------------------
// Phase factor e^{i phi} of a 32-bit fixed-point phase u (phi = 2 pi u / 2^32)
// in FP64, shared by every kernel that draws phases: the top 8 bits select
// e^{2 pi i (u >> 24) / 256} from a 256-entry table (FP64 sincospi, built in
// LDS by each block), the low 24 bits give theta = 2 pi (u mod 2^24) / 2^32 <
// 2 pi / 256, whose cosine and sine come from their Taylor series through
// theta^6 and theta^7 (the next terms are below 1e-17), and the two factors
// are multiplied: a few ulp of FP64, for a fraction of a sincos.  The
// arithmetic is written out in fma() calls so that no call site can contract
// it differently (phases drawn by different kernels agree bitwise).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void phase_table_fill(double2 *tab)
{
    for (int m = threadIdx.x; m < 256; m += blockDim.x) {
        double sn, cs;
        sincospi(static_cast<double>(m) * (1.0 / 128.0), &sn, &cs);
        tab[m] = make_double2(cs, sn);
    }
}

__device__ __forceinline__ void phase_cs(uint32_t u, const double2 *tab, double &c, double &s)
{
    const double2 t = tab[u >> 24];
    const double th = static_cast<double>(u & 0xFFFFFFu) * 1.4629180792671596e-09;   // 2 pi / 2^32
    const double t2 = th * th;
    const double ct = fma(t2, fma(t2, fma(t2, -1.0 / 720.0, 1.0 / 24.0), -0.5), 1.0);
    const double st = th * fma(t2, fma(t2, fma(t2, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), 1.0);
    // explicit fused products: every kernel that inlines this rounds alike
    c = fma(t.x, ct, -(t.y * st));
    s = fma(t.y, ct, t.x * st);
}

// Phase words.  One Philox4x32-10 call (key = the realization's seed) serves
// the four consecutive frequencies k_omega = 4 q .. 4 q + 3 of row k_kappa:
// counter (k_kappa, q, 0, 0), word k_omega - 4 q.  q = floor(k_omega / 4).
// ---------------------------------------------------------------------------
__host__ __device__ inline int floor_div4(int kw) { return (kw >= 0 ? kw : kw - 3) / 4; }

__device__ __forceinline__ void phase_words(int kk, int q, uint64_t seed, uint32_t (&w)[4])
{
    philox_words4(static_cast<uint32_t>(kk), static_cast<uint32_t>(q), 0u, 0u, seed, w);
}

// Phase factor of a line with its per-line complex factor rho_k (if any).
__device__ __forceinline__ void phase_line(uint32_t u, const double2 *ptab, const double *__restrict__ lr, long l,
                                           double &co, double &s)
{
    phase_cs(u, ptab, co, s);
    if (lr) {
        // per-line complex bicoherence factor rho_k carried by the phase factor
        const double xr = lr[2 * l], xi = lr[2 * l + 1];
        const double cr = fma(co, xr, -(s * xi)), ci = fma(co, xi, s * xr);   // fused as in phase_cs
        co = cr;
        s = ci;
    }
}

// Ordered additions to a sum by several blocks, counted: one waits until n are
// counted, adds, and counts itself once its stores are done.  With fences around
// them, one addition in a launch of 3072 waves cost over 200 us.  Without, the
// order rests on three properties of gfx942 and gfx950 that the language does
// not promise: every access to the sums and the counters has agent scope (sc1:
// loads are not served from an XCD's own copy, stores are written through to
// where the other XCDs read), so no cache holds a line to write back or
// invalidate; s_waitcnt waits until a wave's stores have been acknowledged from
// there, before any wave of the block passes the barrier and the count is
// stored; and loads are issued in program order, those of the sums after the
// load that returned the count.  The compiler is kept from moving them by empty
// asm statements that clobber memory.
__device__ __forceinline__ unsigned load_count(const unsigned *count)
{
    return __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void wait_count(const unsigned *count, unsigned n)
{
    while (load_count(count) < n) __builtin_amdgcn_s_sleep(8);
    asm volatile("" ::: "memory");
}

// Wait for the wave's own stores.
__device__ __forceinline__ void wait_stores()
{
    asm volatile("" ::: "memory");
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0);
#endif
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void set_count(unsigned *count, unsigned n)
{
    __hip_atomic_store(count, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ T coherent_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void coherent_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Descriptor of one request of a persistent launch, and one of its work items.
struct PReq {
    Geometry g;
    const void *zrow;
    const void *zcol;
    void *tsum;
    const void *wtab;
    int n_ctiles;
    int pad;
};
struct PItem {
    int req, kb, cg, pad;
};

}  // namespace srm3
