// Device helpers shared by the lattice kernels of libmdlbm (forward and
// adjoint): storage formats, D3Q19 equilibrium, moments, BGK collision with
// Guo forcing, and lattice indexing.  Internal to the library.
#pragma once

#include "lbm_internal.h"
#include "lbm_stencil.h"

namespace mdlbm {


// Per-node moments (rho - 1, u) in the storage's arithmetic.
struct alignas(16) Mom64 {
    double d, x, y, z;
};
struct alignas(8) Mom16 {
    __half2 a, b;
};

template <int S>
struct St;
template <>
struct St<LBM_STORE_F64> {
    using T = double;
    using A = double;
    using M = Mom64;
    static constexpr bool dev = false;
    static __device__ __forceinline__ double ld(const double* p, float) { return *p; }
    static __device__ __forceinline__ double ld_nt(const double* p, float) { return __builtin_nontemporal_load(p); }
    static __device__ __forceinline__ void st(double* p, double v, float) { *p = v; }
    // as stored, without the scale of half deviations
    static __device__ __forceinline__ double raw(const double* p) { return *p; }
    static __device__ __forceinline__ void put(double* p, double v) { *p = v; }
    static __device__ __forceinline__ void put_nt(double* p, double v) { __builtin_nontemporal_store(v, p); }
    static constexpr bool scaled = false;
    static __device__ __forceinline__ void st_mom(M* p, double d, double x, double y, double z, float)
    {
        *p = Mom64{d, x, y, z};
    }
    static __device__ __forceinline__ void ld_mom(const M* p, float, double& d, double& x, double& y,
                                                  double& z)
    {
        const Mom64 m = *p;
        d = m.d, x = m.x, y = m.y, z = m.z;
    }
};
template <>
struct St<LBM_STORE_F32> {
    using T = float;
    using A = float;
    using M = float4;
    static constexpr bool dev = true;
    static __device__ __forceinline__ float ld(const float* p, float) { return *p; }
    static __device__ __forceinline__ float ld_nt(const float* p, float) { return __builtin_nontemporal_load(p); }
    static __device__ __forceinline__ void st(float* p, float v, float) { *p = v; }
    static __device__ __forceinline__ float raw(const float* p) { return *p; }
    static __device__ __forceinline__ void put(float* p, float v) { *p = v; }
    static __device__ __forceinline__ void put_nt(float* p, float v) { __builtin_nontemporal_store(v, p); }
    static constexpr bool scaled = false;
    static __device__ __forceinline__ void st_mom(M* p, float d, float x, float y, float z, float)
    {
        *p = make_float4(d, x, y, z);
    }
    static __device__ __forceinline__ void ld_mom(const M* p, float, float& d, float& x, float& y,
                                                  float& z)
    {
        const float4 m = *p;
        d = m.x, x = m.y, y = m.z, z = m.w;
    }
};
template <>
struct St<LBM_STORE_F16> {
    using T = __half;
    using A = float;
    using M = Mom16;
    static constexpr bool dev = true;
    static __device__ __forceinline__ float ld(const __half* p, float inv)
    {
        return __half2float(*p) * inv;
    }
    static __device__ __forceinline__ float ld_nt(const __half* p, float inv)
    {
        return (float)__builtin_nontemporal_load(reinterpret_cast<const _Float16*>(p)) * inv;
    }
    static __device__ __forceinline__ void st(__half* p, float v, float sc)
    {
        *p = __float2half_rn(v * sc);
    }
    static __device__ __forceinline__ float raw(const __half* p) { return __half2float(*p); }
    static __device__ __forceinline__ void put(__half* p, float v) { *p = __float2half_rn(v); }
    static __device__ __forceinline__ void put_nt(__half* p, float v)
    {
        __builtin_nontemporal_store((_Float16)v, reinterpret_cast<_Float16*>(p));
    }
    static constexpr bool scaled = true;
    static __device__ __forceinline__ void st_mom(M* p, float d, float x, float y, float z, float sc)
    {
        Mom16 m;
        m.a = __floats2half2_rn(d * sc, x * sc);
        m.b = __floats2half2_rn(y * sc, z * sc);
        *p = m;
    }
    static __device__ __forceinline__ void ld_mom(const M* p, float inv, float& d, float& x, float& y,
                                                  float& z)
    {
        const Mom16 m = *p;
        const float2 a = __half22float2(m.a), b = __half22float2(m.b);
        d = a.x * inv, x = a.y * inv, y = b.x * inv, z = b.y * inv;
    }
};

template <class A>
__device__ __forceinline__ A W(int i);
template <>
__device__ __forceinline__ double W<double>(int i) { return wgt(i); }
template <>
__device__ __forceinline__ float W<float>(int i) { return wgtf(i); }

// Equilibrium of direction i in the storage's form:
//   plain:      feq = w rho (1 + 3 e.u + 4.5 (e.u)^2 - 1.5 u.u)
//   deviation:  feq - w = w (drho + rho (3 e.u + 4.5 (e.u)^2 - 1.5 u.u)).
template <bool DEV, class A>
__device__ __forceinline__ A eq_i(int i, A drho, A rho, A ux, A uy, A uz)
{
    const A eu = A(cx(i)) * ux + A(cy(i)) * uy + A(cz(i)) * uz;
    const A uu = ux * ux + uy * uy + uz * uz;
    const A poly = A(3) * eu + A(4.5) * eu * eu - A(1.5) * uu;
    if constexpr (DEV)
        return W<A>(i) * (drho + rho * poly);
    else
        return W<A>(i) * rho * (A(1) + poly);
}

// Moments of the values v[19] in the storage's form; `shift` is +1/2 for
// pre-collision populations (u = (sum f e + F/2)/rho) and -1/2 for
// post-collision ones (the collision turned the momentum into rho u + F/2).
template <bool DEV, class A>
__device__ __forceinline__ void moments(const A* v, A shift, const A* F, A& drho, A& rho, A& ux,
                                        A& uy, A& uz)
{
    A s = A(0), jx = A(0), jy = A(0), jz = A(0);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        s += v[i];
        if (cx(i)) jx += A(cx(i)) * v[i];
        if (cy(i)) jy += A(cy(i)) * v[i];
        if (cz(i)) jz += A(cz(i)) * v[i];
    }
    if constexpr (DEV) {
        drho = s;
        rho = A(1) + s;
    } else {
        rho = s;
        drho = s - A(1);
    }
    const A ir = A(1) / rho;
    ux = (jx + shift * F[0]) * ir;
    uy = (jy + shift * F[1]) * ir;
    uz = (jz + shift * F[2]) * ir;
}

// e_i . (x, y, z) for a direction known at compile time (after unrolling): the
// zero components take no part, since 0 * x may not be dropped by the compiler.
template <class A>
__device__ __forceinline__ A edot(int i, A x, A y, A z)
{
    A r = A(0);
    bool any = false;
    if (cx(i)) {
        r = cx(i) > 0 ? x : -x;
        any = true;
    }
    if (cy(i)) {
        const A t = cy(i) > 0 ? y : -y;
        r = any ? r + t : t;
        any = true;
    }
    if (cz(i)) {
        const A t = cz(i) > 0 ? z : -z;
        r = any ? r + t : t;
    }
    return r;
}

// BGK collision with Guo forcing, in place:
//   f+ = f + omega (feq - f) + (1 - omega/2) w [3 (e - u) + 9 (e.u) e].F
//      = f + omega (w X - f)
// over the opposite pairs (i, i + 1), e_{i+1} = -e_i.  With go = 1/omega - 1/2,
// g = rho u + go F and h = rho u + 2 go F,
//   X = drho - 3/2 rho u.u - 3 go u.F + 9/2 (e.u)(e.h) + 3 (e.g)
// (rho in place of drho for plain populations), of which only the last term
// changes its sign within a pair: about 145 multiply-adds a node.  (A sum per
// direction with the products by zero components, which the compiler may not
// drop, took the FP32 kernel to 687 vector instructions a wave instead of
// about 200.)  The error of f+ against 64 bits is 1.1e-7 in FP32 deviations
// where the sum per direction had 1.4e-7; in FP64, against 80 bits and relative to
// the largest value, 4.9e-17 for f+, 7.1e-17 for rho and 3.1e-17 for u (6.4e-17,
// 1.2e-16 and 4.7e-17; with the diagonals summed last 5.4e-17, 9.1e-17, 3.2e-17).
// With SCALED the populations come and go multiplied by `scale` (half
// deviations as stored): the moments are unscaled and the node's few common
// factors scaled, instead of every population twice.
template <bool DEV, class A, bool SCALED = false>
__device__ __forceinline__ void collide(A* v, A omega, A go, const A* F, A& drho, A& ux, A& uy,
                                        A& uz, A inv = A(1), A scale = A(1))
{
    // (directions 1 to 6 are the axes; the diagonals, the smallest, sum first)
    A s = v[7] + v[8];
    A jx = v[1] - v[2], jy = v[3] - v[4], jz = v[5] - v[6];
#pragma unroll
    for (int i = 7; i < kQ; i += 2) {
        if (i > 7) s += v[i] + v[i + 1];
        const A m = v[i] - v[i + 1];
        if (cx(i)) jx = cx(i) > 0 ? jx + m : jx - m;
        if (cy(i)) jy = cy(i) > 0 ? jy + m : jy - m;
        if (cz(i)) jz = cz(i) > 0 ? jz + m : jz - m;
    }
    s = v[0] + (((v[1] + v[2]) + (v[3] + v[4]) + (v[5] + v[6])) + s);
    if constexpr (SCALED) {
        s *= inv;
        jx *= inv;
        jy *= inv;
        jz *= inv;
    }
    A rho;
    if constexpr (DEV) {
        drho = s;
        rho = A(1) + s;
    } else {
        rho = s;
        drho = s - A(1);
    }
    const A ir = A(1) / rho;
    ux = (jx + A(0.5) * F[0]) * ir;
    uy = (jy + A(0.5) * F[1]) * ir;
    uz = (jz + A(0.5) * F[2]) * ir;
    const A go2 = go + go;
    A gx = rho * ux + go * F[0], gy = rho * uy + go * F[1], gz = rho * uz + go * F[2];
    A hx = rho * ux + go2 * F[0], hy = rho * uy + go2 * F[1], hz = rho * uz + go2 * F[2];
    const A uu = ux * ux + uy * uy + uz * uz;
    const A uF = ux * F[0] + uy * F[1] + uz * F[2];
    A c = (DEV ? drho : rho) - (A(1.5) * rho * uu + A(3) * go * uF);
    if constexpr (SCALED) {
        c *= scale;
        gx *= scale;
        gy *= scale;
        gz *= scale;
        hx *= scale;
        hy *= scale;
        hz *= scale;
    }
    v[0] += omega * (W<A>(0) * c - v[0]);
#pragma unroll
    for (int i = 1; i < kQ; i += 2) {
        const A eu = edot(i, ux, uy, uz), eg = edot(i, gx, gy, gz), eh = edot(i, hx, hy, hz);
        const A even = (A(4.5) * eu) * eh + c;
        v[i] += omega * (W<A>(i) * (A(3) * eg + even) - v[i]);
        v[i + 1] += omega * (W<A>(i) * (A(-3) * eg + even) - v[i + 1]);
    }
}

// Coordinates of a node from its index: division by the invariant nx and ny
// as a multiplication and a shift (exact for indices below 2^31).
__device__ __forceinline__ uint32_t fdiv(uint32_t n, uint32_t m, uint32_t sh)
{
    return (uint32_t)(((uint64_t)n * m) >> sh);
}
__device__ __forceinline__ void node_xyz(uint32_t node, const Geom& g, uint32_t& x, uint32_t& y,
                                         uint32_t& z)
{
    const uint32_t yz = fdiv(node, g.div_m[0], g.div_s[0]);
    x = node - yz * (uint32_t)g.n[0];
    z = fdiv(yz, g.div_m[1], g.div_s[1]);
    y = yz - z * (uint32_t)g.n[1];
}

// Offsets of (c-1, c, c+1) along one axis and whether each lies in the domain.
__device__ __forceinline__ void axis3(uint32_t c, uint32_t n, int per, uint32_t mul,
                                      uint32_t o[3], bool v[3])
{
    o[1] = c * mul;
    v[1] = true;
    if (c > 0) {
        o[0] = (c - 1) * mul;
        v[0] = true;
    } else {
        o[0] = (n - 1) * mul;
        v[0] = per != 0;
    }
    if (c + 1 < n) {
        o[2] = (c + 1) * mul;
        v[2] = true;
    } else {
        o[2] = 0;
        v[2] = per != 0;
    }
}

// The pre-collision populations of node first + threadIdx.x (first: the
// workgroup's first node, the same for all its threads), pulled from x - e_i;
// beyond a wall the node's own opposite population (static halfway
// bounce-back).  Every thread of a wave calls it; `on`: the node wants them.
//
// A wave whose nodes all lie off the y and z faces takes its sources at
// offsets that are the same for every lane: the plane, the shift by e_y and
// e_z and the workgroup's first node go into the scalar base address, and
// three vector offsets (x - 1, x, x + 1, wrapped within the row) serve all
// directions, so a load costs no vector arithmetic.  Lanes at an x wall load
// their five (D3Q19) opposite populations again.  Waves that touch a y or z
// face (3% of them at 128^3, 1% at 512^3) form each lane's address.  Half
// deviations keep their scale.
template <int S>
__device__ __forceinline__ void pull_node(const typename St<S>::T* __restrict__ src, const Geom& g,
                                          uint32_t first, bool on, typename St<S>::A f[kQ])
{
    using T = typename St<S>::T;
    constexpr uint32_t es = sizeof(T);
    const uint32_t cell = first + threadIdx.x;
    const uint32_t nx = g.n[0], ny = g.n[1], nz = g.n[2];
    uint32_t x, y, z;
    node_xyz(cell, g, x, y, z);
    const bool face = y == 0u || y + 1u >= ny || z == 0u || z + 1u >= nz;
    if (!__any(on && face)) {
        if (!on) return;
        const uint32_t t = threadIdx.x;
        // byte offsets from `nx` nodes before the workgroup's first
        const uint32_t o0 = (t + nx) * es;
        const uint32_t om = x > 0u ? o0 - es : (t + 2u * nx - 1u) * es;
        const uint32_t op = x + 1u < nx ? o0 + es : (t + 1u) * es;
        const T* b0 = src + ((int64_t)first - (int64_t)nx);
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const int64_t shift = (int64_t)cy(i) * nx + (int64_t)cz(i) * ((int64_t)nx * ny);
            const char* b = reinterpret_cast<const char*>(b0 + ((int64_t)i * g.stride - shift));
            const uint32_t o = cx(i) > 0 ? om : (cx(i) < 0 ? op : o0);
            f[i] = St<S>::raw(reinterpret_cast<const T*>(b + o));
        }
        if (!g.per[0]) {
            auto own = [&](int i) {
                const char* b = reinterpret_cast<const char*>(b0 + (int64_t)opp(i) * g.stride);
                return St<S>::raw(reinterpret_cast<const T*>(b + o0));
            };
            if (x == 0u) {
#pragma unroll
                for (int i = 1; i < kQ; ++i)
                    if (cx(i) > 0) f[i] = own(i);
            }
            if (x + 1u == nx) {
#pragma unroll
                for (int i = 1; i < kQ; ++i)
                    if (cx(i) < 0) f[i] = own(i);
            }
        }
        return;
    }
    if (!on) return;
    uint32_t ox[3], oy[3], oz[3];
    bool vx[3], vy[3], vz[3];
    axis3(x, nx, g.per[0], 1u, ox, vx);
    axis3(y, ny, g.per[1], nx, oy, vy);
    axis3(z, nz, g.per[2], nx * ny, oz, vz);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        const int sx = 1 - cx(i), sy = 1 - cy(i), sz = 1 - cz(i);
        const bool ok = vx[sx] && vy[sy] && vz[sz];
        const int64_t at = ok ? (int64_t)i * g.stride + (ox[sx] + oy[sy] + oz[sz])
                              : (int64_t)opp(i) * g.stride + cell;
        f[i] = St<S>::raw(src + at);
    }
}

// The populations of node first + threadIdx.x into every plane of dst (a
// scalar base address and one vector offset for all planes); half deviations
// come scaled.
template <int S, bool NT>
__device__ __forceinline__ void store_node(typename St<S>::T* __restrict__ dst, const Geom& g,
                                           uint32_t first, const typename St<S>::A f[kQ])
{
    using T = typename St<S>::T;
    const uint32_t o = threadIdx.x * (uint32_t)sizeof(T);
    T* b0 = dst + first;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        char* b = reinterpret_cast<char*>(b0 + (int64_t)i * g.stride);
        if constexpr (NT)
            St<S>::put_nt(reinterpret_cast<T*>(b + o), f[i]);
        else
            St<S>::put(reinterpret_cast<T*>(b + o), f[i]);
    }
}

__device__ __forceinline__ double image_coord(int c, int L, int per, double center)
{
    if (!per) return (double)c;
    const double d = (double)c - center;
    if (d > 0.5 * L) return (double)(c - L);
    if (d < -0.5 * L) return (double)(c + L);
    return (double)c;
}

__device__ __forceinline__ bool wrap3(int c[3], const Geom& g)
{
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (c[a] < 0 || c[a] >= g.n[a]) {
            if (g.per[a])
                c[a] = c[a] < 0 ? c[a] + g.n[a] : c[a] - g.n[a];
            else
                ok = false;
        }
    }
    return ok;
}

__device__ __forceinline__ uint32_t node_of(const int c[3], const Geom& g)
{
    return (uint32_t)c[0] + (uint32_t)g.n[0] * ((uint32_t)c[1] + (uint32_t)g.n[1] * (uint32_t)c[2]);
}

// The equilibrium of a moving direction d known at run time (eu = e_d.u,
// uu = u.u), in the storage's form as eq_i.
template <bool DEV, class A>
__device__ __forceinline__ A eq_moving(A w, A drho, A rho, A eu, A uu)
{
    const A poly = A(3) * eu + A(4.5) * eu * eu - A(1.5) * uu;
    if constexpr (DEV)
        return w * (drho + rho * poly);
    else
        return w * rho * (A(1) + poly);
}

// Sums of six values over a wave: lane k (k < 6) gets the sum of v[k] over all
// lanes (lanes 6 and 7 zero).  Each of the first three exchanges halves the number
// of values a lane carries, so ten exchanges do what 36 would value by value.
__device__ __forceinline__ double shfl_xor(double v, int m) { return __shfl_xor(v, m, 64); }

template <class V>
__device__ __forceinline__ V wave_sum6(const V v[6])
{
    const int lane = threadIdx.x & 63;
    V a[4];
    {
        // lanes with bit 2 set keep values 4-7
        const bool up = lane & 4;
        const V w[8] = {v[0], v[1], v[2], v[3], v[4], v[5], V{}, V{}};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const V give = up ? w[k] : w[k + 4], keep = up ? w[k + 4] : w[k];
            a[k] = keep + shfl_xor(give, 4);
        }
    }
    V b[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const bool up = lane & 2;
        const V give = up ? a[k] : a[k + 2], keep = up ? a[k + 2] : a[k];
        b[k] = keep + shfl_xor(give, 2);
    }
    const bool up = lane & 1;
    V s = (up ? b[1] : b[0]) + shfl_xor(up ? b[0] : b[1], 1);
    s = s + shfl_xor(s, 8);
    s = s + shfl_xor(s, 16);
    s = s + shfl_xor(s, 32);
    return s;
}

// The force and torque sums of the step under way, which k_boundary adds to,
// and where they go: n = 6 np numbers, doubles or exact 128-bit integers.
struct ForceSums {
    double* sums;
    unsigned long long* fx;
    double* FT;
    uint32_t n;
};

__device__ __forceinline__ double force_sum(const double* sums, const unsigned long long* fx, int64_t i)
{
    return fx ? (double)(int64_t)fx[2 * i + 1] * 0x1p-16 + (double)fx[2 * i] * 0x1p-80 : sums[i];
}

// Finished sums to FT, by the whole grid of a one-dimensional kernel; they are
// left zero for the next step (a launch of its own to clear them took 1-3 us a
// step, with the exact sums three took 10).
__device__ __forceinline__ void settle_sums(const ForceSums& s)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < s.n; i += gridDim.x * blockDim.x) {
        s.FT[i] = force_sum(s.sums, s.fx, i);
        if (s.fx)
            s.fx[2 * (int64_t)i] = s.fx[2 * (int64_t)i + 1] = 0ull;
        else
            s.sums[i] = 0.0;
    }
}

// The counters of a classification whose lists are complete.
struct CounterReport {
    uint32_t* ctr;
    const uint32_t* set;  // this classification's words
    uint32_t* host;       // the pinned block, or null: latch instead
    const int64_t* loff;
    int np;
    uint32_t cand_cap, refill_cap;
};

// To the host block: the head line and the first word of every cursor line.
// Or, after an asynchronous classification: its box check and any list overflow
// (a count above its capacity) into the deferred word, which no classification
// clears.  By the whole grid of a one-dimensional kernel: a line a thread, and no
// round of lines after another (k_refill with nothing to refill, read back and
// latched, by its last wave alone and by all: 200 bodies 4 us either way, 1000
// 14.7 and 12.3 -> 5.6 and 4.4, 27 000 352 and 327 -> 79 and 4.6).  The host
// reads its block after it has waited for the stream.
__device__ __forceinline__ void report_counters(const CounterReport& r)
{
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x), threads = (int)(gridDim.x * blockDim.x);
    if (r.host) {
        if (t < kStageHead) r.host[t] = r.ctr[t];
        for (int i = t; i < 2 * r.np; i += threads) {
            const int64_t at = kStageHead + (int64_t)i * kCursorPad;
            r.host[at] = r.ctr[at];
        }
        return;
    }
    uint32_t bad = 0;
    for (int p = t; p < r.np; p += threads) {
        const uint32_t nl = r.ctr[kStageHead + (int64_t)p * kCursorPad];
        const uint32_t nc = r.ctr[kStageHead + (int64_t)(r.np + p) * kCursorPad];
        if ((int64_t)nl > r.loff[p + 1] - r.loff[p] || nc > r.cand_cap) bad = kDeferredOverflow;
    }
    if (t == 0) {
        if (r.set[kSetRefill] > r.refill_cap) bad |= kDeferredOverflow;
        bad |= r.set[kSetErr] & 0xFFu;
    }
    if (bad) atomicOr(r.ctr + kCtrDeferred, bad);
}

inline CounterReport counter_report(const lbm_ctx* c, bool host)
{
    return CounterReport{c->ctr, c->ctr + kCtrSet[c->ctr_set], host ? c->host_stage : nullptr,
                         c->lay->off_dev, c->cfg.n_particles, (uint32_t)c->cand_cap,
                         (uint32_t)c->refill_cap};
}

}  // namespace mdlbm
