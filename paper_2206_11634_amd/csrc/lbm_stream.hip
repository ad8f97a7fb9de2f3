// Lattice kernels of libmdlbm for gfx950: fused pull-stream + BGK collision,
// link reconstruction (VIBB / halfway) with momentum-exchange forces, local
// refilling, and population import/export.
//
// Storage formats (template parameter S):
//   LBM_STORE_F64  f_i in double, arithmetic in double (the plain method);
//   LBM_STORE_F32  h_i = f_i - w_i in float, arithmetic in float;
//   LBM_STORE_F16  h_i * scale in half, arithmetic in float.
// Deviations keep the O(1) weights out of the stored values, so the rounding
// error of a stored population is relative to |f - w| (a few 1e-3 at the
// Mach numbers of interest) rather than to f.
//
// Layout: plane i of a buffer starts at element i * stride, x fastest.  Every
// collision also stores the node's moments (rho - 1, u) into a moment plane,
// so a link needs two populations and two moment vectors instead of the 38
// populations of x_f and x_ff.  Every kernel is bound by HBM traffic; none of
// them is a contraction, so there is no MFMA here.  A solid node's plane-i slot serves as the "ghost" that holds
// the reconstructed population f_i(x_f, t+1) of the one fluid node
// x_f = x_s + e_i that pulls from it, so the bulk kernel needs no link lookup.
#include <algorithm>

#include "lbm_internal.h"
#include "lbm_stencil.h"
#include "lbm_kernels.h"

namespace mdlbm {
namespace {

// Workgroups are dispatched round-robin over the 8 XCDs.  Each XCD takes
// runs of 128 consecutive workgroups (32768 nodes), the runs of the 8 XCDs
// interleaved: the cache lines neighbouring workgroups share (the +-1 shifts
// in x) mostly stay in one XCD's L2, while the workgroups in flight still
// cover one window of each plane.  Measured on the 512^3 step: 1.9% faster
// than one contiguous eighth of the lattice per XCD, 4% faster than plain
// round-robin.  Grids not divisible into such runs keep the eighths.
__device__ __forceinline__ uint32_t xcd_block()
{
    constexpr uint32_t kRun = 128u;
    const uint32_t per = gridDim.x >> 3;
    const uint32_t k = blockIdx.x >> 3;
    if (per % kRun) return (blockIdx.x & 7u) * per + k;
    return (k / kRun) * (8u * kRun) + (blockIdx.x & 7u) * kRun + (k % kRun);
}

// ---------------------------------------------------------------------------
// Bulk: one thread per node, pull f_i(x - e_i), collide, store.  Bound by HBM:
// FP32 3.7-4.3 ms on 512^3 by where the buffers lie in memory (153 + 16 B a node,
// 5.3-6.1 TB/s; fixed from their allocation on, a copy of the same buffers makes
// 6.2), FP64 7.4-8.3 ms, FP32 D3Q15 3.0-3.4 ms; fewer workgroups a compute unit,
// six waves a SIMD for FP64 and other runs of workgroups gained nothing that held.
// Small lattices are bound by the latency of the flag and population loads
// (48x40x44: 4.8 us FP32, 7.2 us FP64).  With an address per lane and direction
// (687 vector instructions a wave instead of about 200; FP64 112 registers
// instead of 88) 3.83 (where 3.75), 7.5 (7.4), 3.0-3.3 ms, 5.5 and 7.7 us.
// ---------------------------------------------------------------------------
template <int S, bool NT>
__global__ __launch_bounds__(256) void k_stream_collide(const typename St<S>::T* __restrict__ src,
                                                        typename St<S>::T* __restrict__ dst,
                                                        typename St<S>::M* __restrict__ mom,
                                                        const uint8_t* __restrict__ flag, Geom g,
                                                        Phys ph, ForceSums sums)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    settle_sums(sums);
    const uint32_t first = xcd_block() * 256u;
    const uint32_t cell = first + threadIdx.x;
    if (cell >= g.ncell) return;
    const bool fluid = flag[cell] == 0;
    // A solid node's slots are only ever read as link ghosts, which the
    // boundary kernel writes before they are pulled.  Storing the rest state
    // keeps every cache line of the wave fully written (partially written
    // lines cost far more HBM time than the bytes saved) and keeps stale
    // values from evolving inside the bodies.  Fluid and solid lanes of a wave
    // share the stores below.
    A f[kQ];
    A drho = A(0), ux = A(0), uy = A(0), uz = A(0);
#pragma unroll
    for (int i = 0; i < kQ; ++i) f[i] = DEV ? A(0) : W<A>(i);
    if (__any(fluid)) {
        pull_node<S>(src, g, first, fluid, f);
        if (fluid) {
            A F[3];
            A om, go;
            if constexpr (DEV) {
                F[0] = ph.Ff[0], F[1] = ph.Ff[1], F[2] = ph.Ff[2];
                om = ph.omegaf, go = ph.gof;
            } else {
                F[0] = ph.F[0], F[1] = ph.F[1], F[2] = ph.F[2];
                om = ph.omega, go = ph.go;
            }
            collide<DEV, A, St<S>::scaled>(f, om, go, F, drho, ux, uy, uz, A(ph.inv_scale), A(ph.scale));
        }
    }
    store_node<S, NT>(dst, g, first, f);
    St<S>::st_mom(mom + cell, drho, ux, uy, uz, ph.scale);
}

// FP16 deviation storage, two x-neighbouring nodes per thread: the stores
// and the pulls along directions with e_x = 0 move a pair of values per lane
// (half2) instead of one.  Pulls with e_x != 0 start at an odd node and
// are loaded per node.  The arithmetic per node is that of k_stream_collide.
// Requires an even nx (pairs never straddle a row).  Addresses as pull_node's:
// the wave's common offset in the scalar base, three vector offsets.  Bound by
// HBM: 2.1-2.26 ms on 512^3 (77 + 8 B a node, 5.0-5.4 TB/s), 28.5 us on 128^3; with an
// address per lane and direction and a sum per direction in the collision
// (1345 vector instructions a wave) 2.31 ms and 35 us.
__device__ __forceinline__ void pull_pair(const __half* __restrict__ src, const Geom& g,
                                          uint32_t first, bool on, float f0[kQ], float f1[kQ])
{
    const uint32_t t2 = 2u * threadIdx.x, cell = first + t2;
    const uint32_t nx = g.n[0], ny = g.n[1], nz = g.n[2];
    uint32_t x, y, z;
    node_xyz(cell, g, x, y, z);
    const bool face = y == 0u || y + 1u >= ny || z == 0u || z + 1u >= nz;
    const bool slow = __any(on && face);  // uniform over the wave
    if (!on) return;
    auto both = [](const void* p) { return __half22float2(*static_cast<const __half2*>(p)); };
    auto one = [](const void* p) { return __half2float(*static_cast<const __half*>(p)); };
    if (!slow) {
        const uint32_t o0 = (t2 + nx) * 2u;
        const uint32_t om = x > 0u ? o0 - 2u : (t2 + 2u * nx - 1u) * 2u;
        const uint32_t op = x + 2u < nx ? o0 + 4u : (t2 + 2u) * 2u;
        const __half* b0 = src + ((int64_t)first - (int64_t)nx);
        const bool wall0 = !g.per[0] && x == 0u, wall1 = !g.per[0] && x + 2u == nx;
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const int64_t shift = (int64_t)cy(i) * nx + (int64_t)cz(i) * ((int64_t)nx * ny);
            const char* b = reinterpret_cast<const char*>(b0 + ((int64_t)i * g.stride - shift));
            if (cx(i) == 0) {
                const float2 v = both(b + o0);
                f0[i] = v.x;
                f1[i] = v.y;
            } else if (cx(i) > 0) {
                f0[i] = one(wall0 ? reinterpret_cast<const char*>(b0 + (int64_t)opp(i) * g.stride) + o0
                                  : b + om);
                f1[i] = one(b + o0);
            } else {
                f0[i] = one(b + o0 + 2);
                f1[i] = one(wall1 ? reinterpret_cast<const char*>(b0 + (int64_t)opp(i) * g.stride) + o0 + 2
                                  : b + op);
            }
        }
        return;
    }
    uint32_t ox0[3], ox1[3], oy[3], oz[3];
    bool vx0[3], vx1[3], vy[3], vz[3];
    axis3(x, nx, g.per[0], 1u, ox0, vx0);
    axis3(x + 1u, nx, g.per[0], 1u, ox1, vx1);
    axis3(y, ny, g.per[1], nx, oy, vy);
    axis3(z, nz, g.per[2], nx * ny, oz, vz);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        const int sx = 1 - cx(i), sy = 1 - cy(i), sz = 1 - cz(i);
        const uint32_t row = oy[sy] + oz[sz];
        const int64_t pl = (int64_t)i * g.stride, own = (int64_t)opp(i) * g.stride + cell;
        if (cx(i) == 0) {
            const float2 v = both(src + (vy[sy] && vz[sz] ? pl + ox0[1] + row : own));
            f0[i] = v.x;
            f1[i] = v.y;
        } else {
            f0[i] = one(src + (vx0[sx] && vy[sy] && vz[sz] ? pl + ox0[sx] + row : own));
            f1[i] = one(src + (vx1[sx] && vy[sy] && vz[sz] ? pl + ox1[sx] + row : own + 1));
        }
    }
}

template <bool NT>
__global__ __launch_bounds__(256, 6) void k_stream_collide_x2(const __half* __restrict__ src,
                                                           __half* __restrict__ dst,
                                                           Mom16* __restrict__ mom,
                                                           const uint8_t* __restrict__ flag,
                                                           Geom g, Phys ph, ForceSums sums)
{
    settle_sums(sums);
    const uint32_t first = xcd_block() * 512u;
    const uint32_t cell = first + 2u * threadIdx.x;
    if (cell >= g.ncell) return;
    const uint16_t fl = *reinterpret_cast<const uint16_t*>(flag + cell);
    const bool solid0 = (fl & 0xFFu) != 0, solid1 = (fl >> 8) != 0;
    float f0[kQ], f1[kQ];
    float d0 = 0.0f, x0 = 0.0f, y0 = 0.0f, z0 = 0.0f, d1 = 0.0f, x1 = 0.0f, y1 = 0.0f, z1 = 0.0f;
#pragma unroll
    for (int i = 0; i < kQ; ++i) f0[i] = f1[i] = 0.0f;
    const bool on = !(solid0 && solid1);
    if (__any(on)) {
        pull_pair(src, g, first, on, f0, f1);
        const float F[3] = {ph.Ff[0], ph.Ff[1], ph.Ff[2]};
        // (solid pairs collide the rest state: zeros, or the force's share,
        // cleared below)
        collide<true, float, true>(f0, ph.omegaf, ph.gof, F, d0, x0, y0, z0, ph.inv_scale, ph.scale);
        collide<true, float, true>(f1, ph.omegaf, ph.gof, F, d1, x1, y1, z1, ph.inv_scale, ph.scale);
        if (solid0) {
            // rest state, as k_stream_collide stores at solid nodes
#pragma unroll
            for (int i = 0; i < kQ; ++i) f0[i] = 0.0f;
            d0 = x0 = y0 = z0 = 0.0f;
        }
        if (solid1) {
#pragma unroll
            for (int i = 0; i < kQ; ++i) f1[i] = 0.0f;
            d1 = x1 = y1 = z1 = 0.0f;
        }
    }
    const uint32_t o = 4u * threadIdx.x;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        char* b = reinterpret_cast<char*>(dst + first + (int64_t)i * g.stride);
        typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
        const __half2 v = __floats2half2_rn(f0[i], f1[i]);
        if constexpr (NT)
            __builtin_nontemporal_store(*reinterpret_cast<const half2_t*>(&v), reinterpret_cast<half2_t*>(b + o));
        else
            *reinterpret_cast<__half2*>(b + o) = v;
    }
    struct alignas(16) M2 {
        Mom16 a, b;
    } m;
    m.a.a = __floats2half2_rn(d0 * ph.scale, x0 * ph.scale);
    m.a.b = __floats2half2_rn(y0 * ph.scale, z0 * ph.scale);
    m.b.a = __floats2half2_rn(d1 * ph.scale, x1 * ph.scale);
    m.b.b = __floats2half2_rn(y1 * ph.scale, z1 * ph.scale);
    *reinterpret_cast<M2*>(mom + cell) = m;
}

// ---------------------------------------------------------------------------
// Links: one thread per link record, one workgroup per 256-record chunk.
// With many bodies bound by the lines its gathers touch (c. 5.7 GB read for
// 26.4 M links on 512^3: every population line that holds a surface node, once;
// 1.39 ms whatever the instruction count); with few by one wave's chain of
// loads and instructions, so directions come from tables and coordinates from
// multiplications (640 instructions instead of 2450, most of them compares of
// the run-time direction): 5.6 us for one or two bodies, before 10.
// ---------------------------------------------------------------------------
// Exact force sums: a term v becomes the 128-bit two's-complement integer
// v * 2^80 rounded toward zero (hi: the signed upper word, lo: the lower);
// integer sums do not depend on their order.  Returns true, with v taken as
// zero, for a term that is not finite or not below 2^46.
__device__ __forceinline__ bool to_fixed(double v, uint64_t& lo, int64_t& hi)
{
    const bool bad = !(fabs(v) < 0x1p46);
    const double a = bad ? 0.0 : fabs(v) * 0x1p16;  // exact: a power of two
    const double h = floor(a);
    const uint64_t H = (uint64_t)h;
    const uint64_t L = (uint64_t)((a - h) * 0x1p64);  // a - h in [0, 1), exact for a >= 0
    if (v < 0.0 && !bad) {
        lo = 0ull - L;
        hi = (int64_t)(0ull - H - (L != 0ull ? 1ull : 0ull));
    } else {
        lo = L;
        hi = (int64_t)H;
    }
    return bad;
}
struct Fixed {
    uint64_t lo;
    int64_t hi;
};
__device__ __forceinline__ Fixed operator+(const Fixed& a, const Fixed& b)
{
    const uint64_t s = a.lo + b.lo;
    return Fixed{s, (int64_t)((uint64_t)a.hi + (uint64_t)b.hi + (s < a.lo ? 1u : 0u))};
}
__device__ __forceinline__ Fixed shfl_xor(const Fixed& v, int m)
{
    return Fixed{(uint64_t)__shfl_xor((unsigned long long)v.lo, m, 64),
                 (int64_t)__shfl_xor((long long)v.hi, m, 64)};
}

template <int S, bool EXACT>
__global__ __launch_bounds__(256) void k_boundary(typename St<S>::T* __restrict__ f,
                                                  const typename St<S>::M* __restrict__ mom,
                                                  const LinkRec* __restrict__ links,
                                                  const uint32_t* __restrict__ cursor,
                                                  const int64_t* __restrict__ loff,
                                                  const uint32_t* __restrict__ chunk,
                                                  PartDev P, double* __restrict__ sums,
                                                  unsigned long long* __restrict__ FX, Geom g,
                                                  Phys ph, uint32_t* __restrict__ numeric)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    // one workgroup per 256-record chunk of the link layout (chunks do not
    // straddle particles; a wave per 64 records gained nothing at any size)
    const int64_t g0 = (int64_t)blockIdx.x * 256;
    // (every record of a chunk is allocated: it loads beside the particle's
    // index, and counts only if it lies below the particle's link count)
    const LinkRec r = links[g0 + threadIdx.x];
    const int p = (int)chunk[blockIdx.x];
    const int64_t cnt = min(loff[p + 1] - loff[p], (int64_t)cursor[(int64_t)p * kCursorPad]);
    if (g0 - loff[p] >= cnt) return;  // uniform over the block
    const int64_t l = g0 - loff[p] + threadIdx.x;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    if (l < cnt) {
        const int d = r.d, db = opp_moving(d);
        int e[3];
        dir_of(d, e);
        uint32_t ux, uy, uz;
        node_xyz(r.node, g, ux, uy, uz);
        const double xp[3] = {P.pos[3 * p], P.pos[3 * p + 1], P.pos[3 * p + 2]};
        const double vp[3] = {P.vel[3 * p], P.vel[3 * p + 1], P.vel[3 * p + 2]};
        const double wp[3] = {P.omega[3 * p], P.omega[3 * p + 1], P.omega[3 * p + 2]};
        int cn[3] = {(int)ux - e[0], (int)uy - e[1], (int)uz - e[2]};
        wrap3(cn, g);  // for a missing point beyond a wall the node is virtual
        double rr[3], uw[3];
        const double ed[3] = {(double)e[0], (double)e[1], (double)e[2]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            // periodic axes are wrapped by wrap3; a node beyond a wall keeps
            // its raw coordinate (a virtual missing force point)
            const double Xn = image_coord(cn[a], g.n[a], g.per[a], xp[a]);
            const double Xw = Xn + r.q * ed[a];
            rr[a] = Xw - xp[a];
        }
        uw[0] = vp[0] + (wp[1] * rr[2] - wp[2] * rr[1]);
        uw[1] = vp[1] + (wp[2] * rr[0] - wp[0] * rr[2]);
        uw[2] = vp[2] + (wp[0] * rr[1] - wp[1] * rr[0]);
        double out, in;
        if (r.kind == LBM_LINK_MISSING) {
            // treatment 2: equilibrium at (rho0, u_w) on both sides
            const double w = wgt_moving<double>(d);
            const double eu = ed[0] * uw[0] + ed[1] * uw[1] + ed[2] * uw[2];
            const double uu = uw[0] * uw[0] + uw[1] * uw[1] + uw[2] * uw[2];
            out = eq_moving<false, double>(w, 0.0, ph.rho0, eu, uu);
            in = eq_moving<false, double>(w, 0.0, ph.rho0, -eu, uu);
        } else {
            // x_f: its outgoing population and moments at time t
            const A ea[3] = {A(e[0]), A(e[1]), A(e[2])};
            const A w = wgt_moving<A>(d);
            const typename St<S>::T* fd = f + (int64_t)d * g.stride;
            const uint32_t xf = node_of(cn, g);
            const A fdf = St<S>::ld(fd + xf, ph.inv_scale);
            A drf, uf[3];
            St<S>::ld_mom(mom + xf, ph.inv_scale, drf, uf[0], uf[1], uf[2]);
            const A rf = A(1) + drf;
            const A uwa[3] = {A(uw[0]), A(uw[1]), A(uw[2])};
            // 6 w rho_f e_{opp d}.u_w
            const A mw = A(-6) * w * rf * (ea[0] * uwa[0] + ea[1] * uwa[1] + ea[2] * uwa[2]);
            A unk;
            if (r.kind == LBM_LINK_VIBB) {
                int cf[3] = {cn[0] - e[0], cn[1] - e[1], cn[2] - e[2]};
                wrap3(cf, g);
                const uint32_t xff = node_of(cf, g);
                const A fdff = St<S>::ld(fd + xff, ph.inv_scale);
                A drff, uff[3];
                St<S>::ld_mom(mom + xff, ph.inv_scale, drff, uff[0], uff[1], uff[2]);
                const A rff = A(1) + drff;
                const A q = A(r.q);
                const bool low = q <= A(0.5);
                const A tq = A(2) * q, oq = A(1) - A(2) * q;
                auto eq = [&](A dr, A rh, const A u[3]) {
                    return eq_moving<DEV, A>(w, dr, rh, ea[0] * u[0] + ea[1] * u[1] + ea[2] * u[2],
                                             u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
                };
                // non-equilibrium part extrapolated to x_d (Eq. neqd), or for
                // q > 1/2 under treatment bit 8 held at its x_f value
                const bool hold = ph.neq_split && !low;
                const A fneq = (hold ? A(1) : tq) * (fdf - eq(drf, rf, uf)) +
                               (hold ? A(0) : oq) * (fdff - eq(drff, rff, uff));
                // density at x_d (Eq. rhod)
                const A drd = low ? tq * drf + oq * drff : drf;
                const A rd = low ? tq * rf + oq * rff : rf;
                // u*_d from x_f and x_ff (q <= 1/2) or the wall, u**_d from
                // x_ff and the wall
                const A iq1 = A(1) / (A(1) + q);
                const A a1 = low ? tq : (A(1) - q) / q, a2 = low ? oq : (tq - A(1)) / q;
                const A b1 = (A(1) - q) * iq1, b2 = tq * iq1;
                A ud[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const A us = a1 * uf[a] + a2 * (low ? uff[a] : uwa[a]);
                    const A uss = b1 * uff[a] + b2 * uwa[a];
                    ud[a] = (us + A(2) * uss) * A(1.0 / 3.0);
                }
                unk = eq(drd, rd, ud) + fneq + mw;
            } else {
                // treatment 1: halfway bounce-back with the moving-wall term
                unk = fdf + mw;
            }
            St<S>::st(f + (int64_t)db * g.stride + r.node, unk, ph.scale);
            out = (double)fdf;
            in = (double)unk;
            if constexpr (DEV) {
                out += wgt_moving<double>(d);
                in += wgt_moving<double>(d);
            }
        }
        // Galilean-invariant momentum exchange (Eq. mem)
        double t[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) t[a] = (ed[a] - uw[a]) * out + (ed[a] + uw[a]) * in;
        acc[0] = t[0];
        acc[1] = t[1];
        acc[2] = t[2];
        acc[3] = rr[1] * t[2] - rr[2] * t[1];
        acc[4] = rr[2] * t[0] - rr[0] * t[2];
        acc[5] = rr[0] * t[1] - rr[1] * t[0];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if constexpr (EXACT) {
        // per link in 128-bit integers, then wave, workgroup and the
        // particle's accumulator (the carry of the low word's atomic goes
        // into the high word's)
        Fixed v[6];
        bool bad = false;
#pragma unroll
        for (int k = 0; k < 6; ++k) bad = to_fixed(acc[k], v[k].lo, v[k].hi) || bad;
        if (__ballot(bad) && lane == 0) atomicOr(numeric, 1u);  // reported by the next classification
        __shared__ Fixed red[4][6];
        const Fixed sum = wave_sum6(v);
        if (lane < 6) red[wv][lane] = sum;
        __syncthreads();
        if (threadIdx.x < 6) {
            Fixed s = red[0][threadIdx.x];
            for (int w = 1; w < 4; ++w) s = s + red[w][threadIdx.x];
            unsigned long long* a = FX + 2 * (6 * (int64_t)p + threadIdx.x);
            const unsigned long long old = atomicAdd(a, (unsigned long long)s.lo);
            const unsigned long long carry = old + s.lo < old ? 1ull : 0ull;
            atomicAdd(a + 1, (unsigned long long)s.hi + carry);
        }
    } else {
        __shared__ double red[4][6];
        const double sum = wave_sum6(acc);
        if (lane < 6) red[wv][lane] = sum;
        __syncthreads();
        if (threadIdx.x < 6) {
            const double s = (red[0][threadIdx.x] + red[1][threadIdx.x]) +
                             (red[2][threadIdx.x] + red[3][threadIdx.x]);
            atomicAdd(sums + 6 * p + threadIdx.x, s);
            if (!isfinite(s)) atomicOr(numeric, 1u);  // reported by the next classification
        }
    }
}

// ---------------------------------------------------------------------------
// Refill: one thread per node uncovered since the previous classification.
// The count is read on the device (the list's cursor, at most cap), so the
// launch needs no read-back; a grid of at most a few thousand waves strides over
// the list (64 nodes a workgroup spread its gathers over more compute units than
// 256: 200 bodies 20 -> 11 us, 1000 in 512^3 42 -> 16), which also
// reports the classification's counters.  Each node reads only the previous
// populations and owners and writes only its own populations and moments, so
// running the kernel again over a longer list (after the list has grown) gives
// the same values at the nodes of the first run.  Bound by the latency of one node's
// chain: each neighbour's owner and population load once (the bounce-back of
// direction i reads what the streaming of opp(i) would), all before the first
// use: 4.3-5.2 us for a few nodes, 10 us for 60 bodies in FP64, where 38
// populations and 36 owners with wrapped coordinates took 10-15 and 21 us.
// ---------------------------------------------------------------------------
template <int S>
__device__ __forceinline__ void refill_node(const typename St<S>::T* __restrict__ prev,
                                            typename St<S>::T* __restrict__ cur,
                                            typename St<S>::M* __restrict__ mom,
                                            const RefillRec r,
                                            const uint32_t* __restrict__ own_prev,
                                            const PartDev& P, const Geom& g, const Phys& ph)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    const int p = r.part;
    // the wrapped neighbours x - e_i, whether each lies in the lattice, its
    // owner and its f_i; x + e_i and its f_opp(i) are those of opp(i)
    uint32_t x[3];
    node_xyz(r.node, g, x[0], x[1], x[2]);
    uint32_t o[3][3];
    bool in[3][3];
    axis3(x[0], g.n[0], g.per[0], 1u, o[0], in[0]);
    axis3(x[1], g.n[1], g.per[1], g.n[0], o[1], in[1]);
    axis3(x[2], g.n[2], g.per[2], (uint32_t)g.n[0] * (uint32_t)g.n[1], o[2], in[2]);
    A a[kQ];
    uint32_t own[kQ];
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
        const uint32_t n = o[0][1 - cx(i)] + o[1][1 - cy(i)] + o[2][1 - cz(i)];
        a[i] = St<S>::ld(prev + (int64_t)i * g.stride + n, ph.inv_scale);
        own[i] = own_prev[n];
    }
    double rr[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double xp = P.pos[3 * p + k];
        rr[k] = image_coord((int)x[k], g.n[k], g.per[k], xp) - xp;
    }
    const double wp[3] = {P.omega[3 * p], P.omega[3 * p + 1], P.omega[3 * p + 2]};
    const A un[3] = {A(P.vel[3 * p] + (wp[1] * rr[2] - wp[2] * rr[1])),
                     A(P.vel[3 * p + 1] + (wp[2] * rr[0] - wp[0] * rr[2])),
                     A(P.vel[3 * p + 2] + (wp[0] * rr[1] - wp[1] * rr[0]))};
    const A r0 = A(ph.rho0), dr0 = A(ph.rho0 - 1.0);
    const A uu = un[0] * un[0] + un[1] * un[1] + un[2] * un[2];
    bool fluid[kQ];
#pragma unroll
    for (int i = 1; i < kQ; ++i)
        fluid[i] = in[0][1 - cx(i)] && in[1][1 - cy(i)] && in[2][1 - cz(i)] && own[i] == kFluid;
    A v[kQ];
    v[0] = eq_moving<DEV, A>(W<A>(0), dr0, r0, A(0), uu);
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
        const A eu = edot(i, un[0], un[1], un[2]);
        v[i] = fluid[i]        ? a[i]                                          // streamed
               : fluid[opp(i)] ? a[opp(i)] + A(6) * W<A>(i) * r0 * eu          // bounced back
                               : eq_moving<DEV, A>(W<A>(i), dr0, r0, eu, uu);  // equilibrium
    }
    A F[3];
    A om, go;
    if constexpr (DEV) {
        F[0] = ph.Ff[0], F[1] = ph.Ff[1], F[2] = ph.Ff[2];
        om = ph.omegaf, go = ph.gof;
    } else {
        F[0] = ph.F[0], F[1] = ph.F[1], F[2] = ph.F[2];
        om = ph.omega, go = ph.go;
    }
    A drho, ux, uy, uz;
    collide<DEV, A>(v, om, go, F, drho, ux, uy, uz);
#pragma unroll
    for (int i = 0; i < kQ; ++i) St<S>::st(cur + (int64_t)i * g.stride + r.node, v[i], ph.scale);
    St<S>::st_mom(mom + r.node, drho, ux, uy, uz, ph.scale);
}

template <int S>
__global__ __launch_bounds__(64) void k_refill(const typename St<S>::T* __restrict__ prev,
                                                typename St<S>::T* __restrict__ cur,
                                                typename St<S>::M* __restrict__ mom,
                                                const RefillRec* __restrict__ rec,
                                                const uint32_t* __restrict__ cursor, uint32_t cap,
                                                const uint32_t* __restrict__ err,
                                                const uint32_t* __restrict__ own_prev, PartDev P,
                                                Geom g, Phys ph, CounterReport report)
{
    if (report.ctr) report_counters(report);
    if (*err) return;  // the classification's box check failed: nothing was listed
    const uint32_t cnt = min(*cursor, cap);
    for (uint32_t l = blockIdx.x * 64u + threadIdx.x; l < cnt; l += gridDim.x * 64u)
        refill_node<S>(prev, cur, mom, rec[l], own_prev, P, g, ph);
}

// ---------------------------------------------------------------------------
// Import / export
// ---------------------------------------------------------------------------
template <int S>
__global__ void k_init_eq(typename St<S>::T* f, typename St<S>::M* mom, Geom g, Phys ph, double u0x,
                          double u0y, double u0z)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
    if (cell >= g.ncell) return;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        const A v = eq_i<DEV, A>(i, A(ph.rho0 - 1.0), A(ph.rho0), A(u0x), A(u0y), A(u0z));
        St<S>::st(f + (int64_t)i * g.stride + cell, v, ph.scale);
    }
    // the initial populations count as post-collision ones: u = (rho0 u0 - F/2) / rho0
    St<S>::st_mom(mom + cell, A(ph.rho0 - 1.0), A(u0x - 0.5 * ph.F[0] / ph.rho0),
                  A(u0y - 0.5 * ph.F[1] / ph.rho0), A(u0z - 0.5 * ph.F[2] / ph.rho0), ph.scale);
}

template <int S>
__global__ void k_get(const typename St<S>::T* f, double* out, Geom g, Phys ph)
{
    const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
    if (cell >= g.ncell) return;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        double v = (double)St<S>::ld(f + (int64_t)i * g.stride + cell, ph.inv_scale);
        if constexpr (St<S>::dev) v += wgt(i);
        out[(int64_t)i * g.ncell + cell] = v;
    }
}

template <int S>
__global__ void k_set(typename St<S>::T* f, typename St<S>::M* mom, const double* in, Geom g,
                      Phys ph)
{
    using A = typename St<S>::A;
    const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
    if (cell >= g.ncell) return;
    double rho = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        const double fi = in[(int64_t)i * g.ncell + cell];
        rho += fi;
        jx += cx(i) * fi;
        jy += cy(i) * fi;
        jz += cz(i) * fi;
        double v = fi;
        if constexpr (St<S>::dev) v -= wgt(i);
        St<S>::st(f + (int64_t)i * g.stride + cell, A(v), ph.scale);
    }
    // the given populations are post-collision: u = (sum f e - F/2) / rho
    St<S>::st_mom(mom + cell, A(rho - 1.0), A((jx - 0.5 * ph.F[0]) / rho),
                  A((jy - 0.5 * ph.F[1]) / rho), A((jz - 0.5 * ph.F[2]) / rho), ph.scale);
}

__global__ void k_split(const double* FT, double* F, double* T, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    for (int a = 0; a < 3; ++a) {
        F[3 * i + a] = FT[6 * i + a];
        T[3 * i + a] = FT[6 * i + 3 + a];
    }
}

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + 255) / 256); }

template <template <int> class Fn, class... Args>
hipError_t dispatch(int storage, Args&&... args)
{
    switch (storage) {
    case LBM_STORE_F64: return Fn<LBM_STORE_F64>::run(args...);
    case LBM_STORE_F32: return Fn<LBM_STORE_F32>::run(args...);
    case LBM_STORE_F16: return Fn<LBM_STORE_F16>::run(args...);
    default: return hipErrorInvalidValue;
    }
}

template <int S>
struct RunInit {
    static hipError_t run(lbm_ctx* c, void* f)
    {
        hipLaunchKernelGGL(k_init_eq<S>, dim3(blocks_for(c->geom.ncell)), dim3(256), 0, c->stream,
                           (typename St<S>::T*)f, (typename St<S>::M*)c->mom, c->geom, c->phys,
                           c->cfg.u0[0], c->cfg.u0[1], c->cfg.u0[2]);
        return hipGetLastError();
    }
};

template <int S>
struct RunSC {
    static hipError_t run(lbm_ctx* c, const void* src, void* dst)
    {
        const ForceSums sums{c->sums, c->FX, c->FT, 6u * (uint32_t)c->cfg.n_particles};
        // Populations stored past the cache (non-temporal) where two levels and the
        // moments do not fit the 256 MB memory-side cache: a level written through
        // it only pushes out what the next step would find there.  Same buffers,
        // cached and past it, us: below the line 112^3 FP32 36.3 and 43.0, 128^3
        // FP16 28.7 and 38.4, 88^3 FP64 35.5 and 45.9; above, 128^3 FP32 71 and 67,
        // 104^3 FP64 76.0 and 69.7, 152^3 FP16 67.2 and 62.0, 256^3 281.5 and
        // 275.7, 512^3 2325 and 2258.  From twice the cache on it is even for FP32
        // and FP64 (-3 to +2 % by the buffers' place), which stay cached.
        const int64_t bytes = 2 * c->sizes.population_bytes + c->sizes.moment_bytes;
        const bool nt = bytes > ((int64_t)1 << 28) && (S == LBM_STORE_F16 || bytes < ((int64_t)1 << 29));
        // FP16 only: for FP32 the pair kernel was measured slower (4.8 against
        // 4.4 ms on 512^3)
        if constexpr (S == LBM_STORE_F16) {
            if (c->geom.n[0] % 2 == 0) {
                uint32_t nb = blocks_for(c->geom.ncell / 2);
                nb = (nb + 7u) & ~7u;
                hipLaunchKernelGGL((nt ? k_stream_collide_x2<true> : k_stream_collide_x2<false>), dim3(nb), dim3(256), 0, c->stream,
                                   (const typename St<S>::T*)src, (typename St<S>::T*)dst,
                                   (typename St<S>::M*)c->mom, c->flag, c->geom, c->phys, sums);
                return hipGetLastError();
            }
        }
        uint32_t nb = blocks_for(c->geom.ncell);
        nb = (nb + 7u) & ~7u;  // whole rounds over the 8 XCDs
        hipLaunchKernelGGL((nt ? k_stream_collide<S, true> : k_stream_collide<S, false>), dim3(nb), dim3(256), 0, c->stream,
                           (const typename St<S>::T*)src, (typename St<S>::T*)dst,
                           (typename St<S>::M*)c->mom, c->flag, c->geom, c->phys, sums);
        return hipGetLastError();
    }
};

template <int S>
struct RunBC {
    static hipError_t run(lbm_ctx* c, void* f, const PartDev& P)
    {
        if (c->cfg.n_particles == 0 || c->link_max == 0 || c->lay->chunks() == 0)
            return hipSuccess;
        hipLaunchKernelGGL((c->FX ? k_boundary<S, true> : k_boundary<S, false>),
                           dim3((uint32_t)c->lay->chunks()), dim3(256), 0, c->stream,
                           (typename St<S>::T*)f, (const typename St<S>::M*)c->mom, c->links,
                           c->link_cursor, c->lay->off_dev, c->lay->chunk_dev, P, c->sums, c->FX,
                           c->geom, c->phys, c->numeric);
        return hipGetLastError();
    }
};

template <int S>
struct RunRefill {
    static hipError_t run(lbm_ctx* c, const void* fprev, void* fcur, const uint32_t* own_prev,
                          const PartDev& P, Report report)
    {
        const uint32_t nb = std::min<uint32_t>((uint32_t)((c->refill_cap + 63) / 64), 4096u);
        const CounterReport r = report == Report::none ? CounterReport{} : counter_report(c, report == Report::host);
        hipLaunchKernelGGL(k_refill<S>, dim3(nb), dim3(64), 0, c->stream,
                           (const typename St<S>::T*)fprev, (typename St<S>::T*)fcur,
                           (typename St<S>::M*)c->mom, c->refill, c->refill_cursor,
                           (uint32_t)c->refill_cap, c->err, own_prev, P, c->geom, c->phys, r);
        return hipGetLastError();
    }
};

template <int S>
struct RunGet {
    static hipError_t run(lbm_ctx* c, const void* f, double* out)
    {
        hipLaunchKernelGGL(k_get<S>, dim3(blocks_for(c->geom.ncell)), dim3(256), 0, c->stream,
                           (const typename St<S>::T*)f, out, c->geom, c->phys);
        return hipGetLastError();
    }
};

// Density and velocity of every node from the moment plane, in FP64.
template <int S>
__global__ __launch_bounds__(256) void k_get_moments(const typename St<S>::M* __restrict__ mom,
                                                     double* __restrict__ rho,
                                                     double* __restrict__ u, Geom g, Phys ph)
{
    using A = typename St<S>::A;
    const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
    if (cell >= g.ncell) return;
    A d, ux, uy, uz;
    St<S>::ld_mom(mom + cell, ph.inv_scale, d, ux, uy, uz);
    rho[cell] = 1.0 + (double)d;
    u[3 * (int64_t)cell] = (double)ux;
    u[3 * (int64_t)cell + 1] = (double)uy;
    u[3 * (int64_t)cell + 2] = (double)uz;
}

template <int S>
struct RunMoments {
    static hipError_t run(lbm_ctx* c, double* rho, double* u)
    {
        hipLaunchKernelGGL(k_get_moments<S>, dim3(blocks_for(c->geom.ncell)), dim3(256), 0,
                           c->stream, (const typename St<S>::M*)c->mom, rho, u, c->geom, c->phys);
        return hipGetLastError();
    }
};

template <int S>
struct RunSet {
    static hipError_t run(lbm_ctx* c, void* f, const double* in)
    {
        hipLaunchKernelGGL(k_set<S>, dim3(blocks_for(c->geom.ncell)), dim3(256), 0, c->stream,
                           (typename St<S>::T*)f, (typename St<S>::M*)c->mom, in, c->geom, c->phys);
        return hipGetLastError();
    }
};

}  // namespace

namespace MDLBM_QNS {

hipError_t launch_init_equilibrium(lbm_ctx* c, void* f)
{
    return dispatch<RunInit>(c->cfg.storage, c, f);
}
hipError_t launch_stream_collide(lbm_ctx* c, const void* src, void* dst)
{
    return dispatch<RunSC>(c->cfg.storage, c, src, dst);
}
hipError_t launch_boundary(lbm_ctx* c, void* f, const PartDev& P)
{
    return dispatch<RunBC>(c->cfg.storage, c, f, P);
}
hipError_t launch_refill(lbm_ctx* c, const void* fprev, void* fcur, const uint32_t* own_prev,
                         const PartDev& P, Report report)
{
    return dispatch<RunRefill>(c->cfg.storage, c, fprev, fcur, own_prev, P, report);
}
hipError_t launch_get_populations(lbm_ctx* c, const void* f, double* out)
{
    return dispatch<RunGet>(c->cfg.storage, c, f, out);
}
hipError_t launch_set_populations(lbm_ctx* c, void* f, const double* in)
{
    return dispatch<RunSet>(c->cfg.storage, c, f, in);
}
hipError_t launch_get_moments(lbm_ctx* c, double* rho, double* u)
{
    return dispatch<RunMoments>(c->cfg.storage, c, rho, u);
}
hipError_t launch_split_forces(const lbm_ctx* c, double* F, double* T)
{
    const int n = c->cfg.n_particles;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_split, dim3(blocks_for(n)), dim3(256), 0, c->stream, c->FT, F, T, n);
    return hipGetLastError();
}

}  // namespace MDLBM_QNS
}  // namespace mdlbm
