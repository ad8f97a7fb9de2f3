// Adjoint of the lattice step (differentiation form; not part of the paper).
//
// With the geometry schedule held fixed, one taped step maps the populations
// f(n) (fluid nodes of the owners at n) to f(n+1) (fluid nodes of the owners
// at n+1): link reconstruction from f(n), pull streaming and BGK + Guo
// collision of the fluid nodes of n, and refilling + collision of the nodes
// uncovered between n and n+1.  The objective adds, per step, the momentum
// exchange force and torque of every particle weighted by (wF, wT).
//
// One adjoint step n <- n+1 runs three kernels:
//  1. k_adj_node   per node x fluid at n: recompute its pulled pre-collision
//                  populations, apply the transposed collision Jacobian to
//                  lambda(n+1) -> Lambda (the adjoint of the pre-collision
//                  populations), accumulate dJ/dtau, dJ/dF; then (every node)
//                  push Lambda to the entries of lambda(n) that x read: entry
//                  (j, x - e_j), of which x is the only writer (x itself for
//                  entries read through a wall); and list the nodes refilled
//                  between n and n+1;
//     k_adj_refill the same for the listed nodes, whose pre-collision
//                  populations come from the refill rules; also dJ/dv of the
//                  wall velocity in those rules;
//  2. k_adj_links  per link: adjoint of its reconstructed population (Lambda
//                  of the fluid node that pulled the ghost slot, left in
//                  lambda(n) at the solid node, plus the objective), transposed
//                  through VIBB / halfway by a reverse sweep and added to lambda(n) at x_f and x_ff with atomics; momentum-
//                  exchange and missing-point objective terms; dJ/dv, dJ/dF.
// Arithmetic is that of the storage (double for FP64, float otherwise);
// parameter gradients are summed in FP64.
#include <algorithm>
#include <type_traits>

#include "lbm_internal.h"
#include "lbm_stencil.h"
#include "lbm_kernels.h"

namespace mdlbm {
namespace {

// The reconstructed population of a link and its transposed derivative: the
// formulas of the forward link kernel (VIBB, Eqs. eqneq, neqd, rhod, u*_d,
// u**_d, u_d; or halfway bounce-back) followed by one reverse sweep, which
// costs about as much as the value (13 tangents carried forward took some 1000
// more instructions a link).
template <class A>
struct LinkIn {
    A fdf, rf, uf[3];     // x_f: outgoing population, density, velocity
    A fdff, rff, uff[3];  // x_ff
    A uw[3], q;
};
// d value / d of each input (of the same names).
template <class A>
using LinkGrad = LinkIn<A>;

template <bool DEV, class A>
__device__ __forceinline__ A link_value(int kind, A w, const A e[3], const LinkIn<A>& x,
                                        bool neq_split, LinkGrad<A>& g)
{
    const A euw = e[0] * x.uw[0] + e[1] * x.uw[1] + e[2] * x.uw[2];
    const A w6 = A(-6) * w;
    const A mw = w6 * x.rf * euw;
    g.fdf = A(1);
    g.rf = w6 * euw;
    g.fdff = g.rff = g.q = A(0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        g.uf[a] = g.uff[a] = A(0);
        g.uw[a] = w6 * x.rf * e[a];
    }
    if (kind != LBM_LINK_VIBB) return x.fdf + mw;
    // the equilibrium at (r, u) less its weight, 1 + its polynomial, and the
    // factors of its derivative in u: w r (3 + 9 e.u) e - 3 w r u
    auto eq = [&](A r, const A u[3], A& p1, A& eu) {
        eu = e[0] * u[0] + e[1] * u[1] + e[2] * u[2];
        const A poly = A(3) * eu + A(4.5) * eu * eu -
                       A(1.5) * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
        p1 = A(1) + poly;
        return DEV ? w * ((r - A(1)) + r * poly) : w * (r + r * poly);
    };
    const A q = x.q;
    const bool low = q <= A(0.5), hold = neq_split && !low;
    const A tq = A(2) * q, oq = A(1) - tq;
    const A n1 = hold ? A(1) : tq, n2 = hold ? A(0) : oq;
    const A iq = A(1) / q, i1 = A(1) / (A(1) + q);
    const A c1 = (A(1) - q) * iq, c2 = (tq - A(1)) * iq, c3 = (A(1) - q) * i1, c4 = tq * i1;
    const A third = A(1.0 / 3.0);
    A pf, pff, pd, ef, eff, ed, ud[3];
    const A nf = x.fdf - eq(x.rf, x.uf, pf, ef), nff = x.fdff - eq(x.rff, x.uff, pff, eff);
    const A rd = low ? tq * x.rf + oq * x.rff : x.rf;
    const A a1 = low ? tq : c1, a2 = low ? oq : c2;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const A us = a1 * x.uf[a] + a2 * (low ? x.uff[a] : x.uw[a]);
        ud[a] = (us + A(2) * (c3 * x.uff[a] + c4 * x.uw[a])) * third;
    }
    const A value = eq(rd, ud, pd, ed) + n1 * nf + n2 * nff + mw;
    g.fdf = n1;
    g.fdff = n2;
    g.rf += w * (pd * (low ? tq : A(1)) - n1 * pf);
    g.rff = w * (pd * (low ? oq : A(0)) - n2 * pff);
    g.q = (hold ? A(0) : A(2) * (nf - nff)) + (low ? A(2) * w * pd * (x.rf - x.rff) : A(0));
    const A kd = w * rd * (A(3) + A(9) * ed), ld = A(-3) * w * rd;
    const A kf = n1 * w * x.rf * (A(3) + A(9) * ef), lf = A(-3) * n1 * w * x.rf;
    const A kff = n2 * w * x.rff * (A(3) + A(9) * eff), lff = A(-3) * n2 * w * x.rff;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const A du = third * (kd * e[a] + ld * ud[a]);  // d value / d (us + 2 uss)
        g.uf[a] = du * a1 - (kf * e[a] + lf * x.uf[a]);
        g.uff[a] = du * ((low ? oq : A(0)) + A(2) * c3) - (kff * e[a] + lff * x.uff[a]);
        g.uw[a] += du * ((low ? A(0) : c2) + A(2) * c4);
        const A dus = low ? A(2) * (x.uf[a] - x.uff[a]) : (x.uw[a] - x.uf[a]) * iq * iq;
        g.q += du * (dus + A(4) * (x.uw[a] - x.uff[a]) * i1 * i1);
    }
    return value;
}

// Metaball sum of one particle at X (world coordinates of the image nearest
// the particle), its gradient in X, and its derivative for a small rotation
// of the body about its centre xp: each point x_i moves by dtheta x (x_i - xp),
// so dM/dtheta = sum_i (x_i - xp) x dm_i/dx_i with dm_i/dx_i = -grad_X m_i.
__device__ __forceinline__ void metaball_grad(const double* pts, const double* K, int i0, int i1,
                                              const double X[3], const double xp[3], double& M,
                                              double gM[3], double gR[3])
{
    M = 0.0;
    gM[0] = gM[1] = gM[2] = 0.0;
    gR[0] = gR[1] = gR[2] = 0.0;
    for (int i = i0; i < i1; ++i) {
        const double r[3] = {X[0] - pts[3 * i], X[1] - pts[3 * i + 1], X[2] - pts[3 * i + 2]};
        const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
        const double t = K[i] / r2;
        M += t;
        const double s = -2.0 * t / r2;
        gM[0] += s * r[0];
        gM[1] += s * r[1];
        gM[2] += s * r[2];
        const double b[3] = {pts[3 * i] - xp[0], pts[3 * i + 1] - xp[1], pts[3 * i + 2] - xp[2]};
        // (x_i - xp) x (-s r)
        gR[0] -= s * (b[1] * r[2] - b[2] * r[1]);
        gR[1] -= s * (b[2] * r[0] - b[0] * r[2]);
        gR[2] -= s * (b[0] * r[1] - b[1] * r[0]);
    }
}

// Pose data of one taped step for the geometry terms of the adjoint, and
// where the per-particle derivatives go.  Prescribed trajectories: the pose
// gradients of each step (stride 6: x, theta) and one dJ/dv for all steps
// (stride 3); free motion: the state adjoints of the steps (stride 12: x,
// theta, v, omega).
struct GeoArgs {
    const double* wpts = nullptr;   // world control points of the step's pose
    const double* K = nullptr;
    const double* c0 = nullptr;
    const int32_t* off = nullptr;
    int exact_q = 0;
    double* g_links = nullptr;      // dJ/d(x_p, theta_p) of the pose the links used
    double* g_refill = nullptr;     // dJ/dx_p of the pose the refill used
    int gstride = 6;
    double* v_links = nullptr;      // dJ/dv_p seen by the links (null: grad + 4)
    double* v_refill = nullptr;     // dJ/dv_p seen by the refill (null: grad + 4)
    int vstride = 3;
    double* w_links = nullptr;      // dJ/domega_p seen by the links (null: not kept)
    double* w_refill = nullptr;     // dJ/domega_p seen by the refill (null: not kept)
};

// Sum NV doubles over a block of T threads and add sum k to *out(k) (one
// atomic each).
template <int T, int NV, class Out>
__device__ __forceinline__ void block_add(const double (&v)[NV], Out out)
{
    static_assert(T == 64 || T == 256, "one wave or four");
    constexpr int NG = (NV + 5) / 6;
    __shared__ double red[4][6 * NG];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        double t[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) t[m] = 6 * k + m < NV ? v[6 * k + m < NV ? 6 * k + m : 0] : 0.0;
        const double s = wave_sum6(t);
        if constexpr (T == 64) {
            if (lane < 6 && 6 * k + lane < NV && s != 0.0) atomicAdd(out(6 * k + lane), s);
        } else {
            if (lane < 6) red[wv][6 * k + lane] = s;
        }
    }
    if constexpr (T == 64) return;
    __syncthreads();
    if (threadIdx.x < NV) {
        const double s = (red[0][threadIdx.x] + red[1][threadIdx.x]) +
                         (red[2][threadIdx.x] + red[3][threadIdx.x]);
        if (s != 0.0) atomicAdd(out((int)threadIdx.x), s);
    }
}

// ---------------------------------------------------------------------------
// 1. transposed collision per node, pushed to lambda(n)
// ---------------------------------------------------------------------------

// Lambda = (d post / d pre)^T lambda for BGK + Guo at the pre-collision state
// pre, in closed form: Lambda_j = (1 - omega) lambda_j + omega a
// + H . (e_j - u) / rho, kept as (1 - omega) lambda_j + c + e_j . h.  Returns
// the coefficients; adds dJ/dF (3) and dJ/dtau to acc.
template <class A>
struct AdjCoef {
    A om1, c, h[3];  // Lambda_j = om1 lambda_j + c + e_j.h
    __device__ __forceinline__ A operator()(int j, A lam_j) const
    {
        return j == 0 ? om1 * lam_j + c : om1 * lam_j + (c + edot(j, h[0], h[1], h[2]));
    }
};

template <bool DEV, class A>
__device__ __forceinline__ AdjCoef<A> adj_collide(const A lam[kQ], const A pre[kQ], const Phys& ph,
                                                  double acc[4])
{
    A F[3];
    A om;
    if constexpr (DEV) {
        F[0] = ph.Ff[0], F[1] = ph.Ff[1], F[2] = ph.Ff[2];
        om = ph.omegaf;
    } else {
        F[0] = ph.F[0], F[1] = ph.F[1], F[2] = ph.F[2];
        om = ph.omega;
    }
    // sums over the opposite pairs: populations, and the weighted moments of
    // lambda, m0 = sum w l, m1 = sum w l e, m2 = sum w l e e: the sums over i
    // of the equilibrium's and the forcing's derivatives are polynomials in u
    // and F with these coefficients
    A s = pre[0], jx = A(0), jy = A(0), jz = A(0);
    A lsum = lam[0], m0 = W<A>(0) * lam[0], m1[3] = {A(0), A(0), A(0)};
    A mxx = A(0), myy = A(0), mzz = A(0), mxy = A(0), mxz = A(0), myz = A(0);
#pragma unroll
    for (int i = 1; i < kQ; i += 2) {
        s += pre[i] + pre[i + 1];
        const A m = pre[i] - pre[i + 1];
        const A lp = lam[i] + lam[i + 1];
        lsum += lp;
        const A p = W<A>(i) * lp, d = W<A>(i) * (lam[i] - lam[i + 1]);
        m0 += p;
        if (cx(i)) {
            jx += cx(i) > 0 ? m : -m;
            m1[0] += cx(i) > 0 ? d : -d;
            mxx += p;
        }
        if (cy(i)) {
            jy += cy(i) > 0 ? m : -m;
            m1[1] += cy(i) > 0 ? d : -d;
            myy += p;
        }
        if (cz(i)) {
            jz += cz(i) > 0 ? m : -m;
            m1[2] += cz(i) > 0 ? d : -d;
            mzz += p;
        }
        if (cx(i) && cy(i)) mxy += cx(i) * cy(i) > 0 ? p : -p;
        if (cx(i) && cz(i)) mxz += cx(i) * cz(i) > 0 ? p : -p;
        if (cy(i) && cz(i)) myz += cy(i) * cz(i) > 0 ? p : -p;
    }
    A drho, rho;
    if constexpr (DEV) {
        drho = s;
        rho = A(1) + s;
    } else {
        rho = s;
        drho = s - A(1);
    }
    const A ir = A(1) / rho;
    const A u[3] = {(jx + A(0.5) * F[0]) * ir, (jy + A(0.5) * F[1]) * ir, (jz + A(0.5) * F[2]) * ir};
    const A uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const A uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2];
    const A gf = A(1) - A(0.5) * om;
    // dJ/domega = sum (lambda - mean)(feq - pre - S/2): the second factor sums
    // to zero over i, so lambda may be centred on its mean, which keeps the
    // sum free of the cancellation of a large common adjoint density.  feq -
    // S/2 = w [drho - 3/2 rho u.u + 3/2 u.F + 9/2 (e.u)(e.h) + 3 e.g] with g =
    // rho u - F/2, h = rho u - F (rho in place of drho for plain populations).
    const A lbar = lsum * A(1.0 / kQ);
    const A c = (DEV ? drho : rho) - (A(1.5) * rho * uu - A(1.5) * uF);
    const A g[3] = {rho * u[0] - A(0.5) * F[0], rho * u[1] - A(0.5) * F[1], rho * u[2] - A(0.5) * F[2]};
    const A h[3] = {rho * u[0] - F[0], rho * u[1] - F[1], rho * u[2] - F[2]};
    A dom = (lam[0] - lbar) * (W<A>(0) * c - pre[0]);
#pragma unroll
    for (int i = 1; i < kQ; i += 2) {
        const A eu = edot(i, u[0], u[1], u[2]), eg = edot(i, g[0], g[1], g[2]),
                eh = edot(i, h[0], h[1], h[2]);
        const A even = (A(4.5) * eu) * eh + c;
        dom += (lam[i] - lbar) * (W<A>(i) * (A(3) * eg + even) - pre[i]);
        dom += (lam[i + 1] - lbar) * (W<A>(i) * (A(-3) * eg + even) - pre[i + 1]);
    }
    const A m2u[3] = {mxx * u[0] + mxy * u[1] + mxz * u[2], mxy * u[0] + myy * u[1] + myz * u[2],
                      mxz * u[0] + myz * u[1] + mzz * u[2]};
    const A m2F[3] = {mxx * F[0] + mxy * F[1] + mxz * F[2], mxy * F[0] + myy * F[1] + myz * F[2],
                      mxz * F[0] + myz * F[1] + mzz * F[2]};
    const A m1u = m1[0] * u[0] + m1[1] * u[1] + m1[2] * u[2];
    const A um2u = u[0] * m2u[0] + u[1] * m2u[1] + u[2] * m2u[2];
    // a = sum w l P_i with P_i = 1 + 3 e.u + 4.5 (e.u)^2 - 1.5 u.u
    const A a = m0 * (A(1) - A(1.5) * uu) + A(3) * m1u + A(4.5) * um2u;
    AdjCoef<A> co;
    co.om1 = A(1) - om;
    A hu = A(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const A B = rho * (A(3) * m1[k] + A(9) * m2u[k] - A(3) * u[k] * m0);
        const A G = A(-3) * F[k] * m0 + A(9) * m2F[k];
        const A Fd = A(3) * m1[k] - A(3) * u[k] * m0 + A(9) * m2u[k];
        const A H = om * B + gf * G;
        co.h[k] = H * ir;
        hu += co.h[k] * u[k];
        acc[k] += (double)(co.h[k] * A(0.5) + gf * Fd);
    }
    co.c = om * a - hu;
    acc[3] += -(double)om * (double)om * (double)dom;  // dtau = -omega^2 domega
    return co;
}

// Every node x.  A node fluid at n and n + 1 recomputes its pulled
// pre-collision populations and takes the transposed collision; then x pushes
// Lambda to the entries of lambda(n) it read.  Entry (j, y) is written by
// exactly one node: x = y + e_j when that lies inside the lattice, else y
// itself (read through a wall).  Its value is Lambda_j(x) for a node x fluid
// at n (for a solid y that is the adjoint of the ghost slot, which the link
// kernel takes and clears), and zero otherwise; k_adj_refill then rewrites the
// entries its refilled nodes read.
//
// Bound by memory where the lattice exceeds the caches: f and lambda(n + 1)
// read, lambda(n) written, owners, 3 x 76 + 8 bytes a node in FP32, 79 us at
// 128^3 (6.3 TB/s; 97 with everything through the memory-side cache; 105 before
// sums over opposite pairs took the place of 19 terms each).  NT: the taped
// level is loaded and the planes with e_x = 0 are stored past that cache (the
// shifted planes' lines, written by two waves, have to meet in a cache: 100 us
// with all stores past it).  A small FP64 box (48 x 40 x 44) takes 12.4 us (14.0 before).
template <int S, bool NT>
__global__ __launch_bounds__(256) void k_adj_node(const typename St<S>::T* __restrict__ f,
                                                  const uint32_t* __restrict__ own0,
                                                  const uint32_t* __restrict__ own1,
                                                  const typename St<S>::A* __restrict__ lam1,
                                                  typename St<S>::A* __restrict__ lam0, Geom g,
                                                  Phys ph, double* grad, AdjList list)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};  // dJ/dF (3), dJ/dtau
    bool refilled = false;
    if (cell < g.ncell) {
        const uint32_t o0 = own0[cell], o1 = own1[cell];
        const bool live = o0 == kFluid && o1 == kFluid;
        // a node refilled between n and n + 1 leaves the entries it read from
        // nodes fluid at n to k_adj_refill, so the two kernels write disjoint
        // entries
        refilled = o0 != kFluid && o1 == kFluid;
        const uint32_t nx = g.n[0], ny = g.n[1];
        uint32_t x, y, z;
        node_xyz(cell, g, x, y, z);
        uint32_t ox[3], oy[3], oz[3];
        bool vx[3], vy[3], vz[3];
        axis3(x, nx, g.per[0], 1u, ox, vx);
        axis3(y, ny, g.per[1], nx, oy, vy);
        axis3(z, g.n[2], g.per[2], nx * ny, oz, vz);
        // the entry that x reads in direction j: (j, x - e_j), or through a
        // wall its own (opp j)
        auto entry = [&](int j) -> int64_t {
            const int sx = 1 - cx(j), sy = 1 - cy(j), sz = 1 - cz(j);
            return vx[sx] && vy[sy] && vz[sz] ? (int64_t)j * g.stride + (ox[sx] + oy[sy] + oz[sz])
                                              : (int64_t)opp(j) * g.stride + cell;
        };
        A lam[kQ] = {};
        AdjCoef<A> co{};
        if (live) {
            A pre[kQ];
#pragma unroll
            for (int i = 0; i < kQ; ++i) {
                lam[i] = lam1[(int64_t)i * g.stride + cell];
                pre[i] = NT ? St<S>::ld_nt(f + entry(i), ph.inv_scale) : St<S>::ld(f + entry(i), ph.inv_scale);
            }
            co = adj_collide<DEV, A>(lam, pre, ph, acc);
        }
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            const A v = live ? co(j, lam[j]) : A(0);
            const int sx = 1 - cx(j), sy = 1 - cy(j), sz = 1 - cz(j);
            if (!(refilled && j > 0 && vx[sx] && vy[sy] && vz[sz] &&
                  own0[ox[sx] + oy[sy] + oz[sz]] == kFluid)) {
                if (NT && cx(j) == 0)
                    __builtin_nontemporal_store(v, lam0 + entry(j));
                else
                    lam0[entry(j)] = v;
            }
        }
    }
    // list the refilled nodes for k_adj_refill (one atomic per wave); the
    // count may pass the capacity, which the host checks after the adjoint
    const uint64_t m = __ballot(refilled);
    if (m) {  // uniform over the wave
        const int lane = threadIdx.x & 63;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(list.count, (uint32_t)__popcll(m));
        base = __shfl(base, 0, 64);
        const uint32_t idx = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (refilled && idx < list.cap) list.node[idx] = cell;
    }
    block_add<256>(acc, [=](int k) { return grad + k; });
}

// Nodes refilled between n and n + 1 (solid at n, fluid at n + 1): their
// pre-collision populations follow the refill rules (streamed from a node
// fluid at n, bounce-back of the opposite streamed population with the wall
// term, or the equilibrium at (rho0, u_wall)); transposed collision, dJ/dF,
// dJ/dtau, and dJ/dv of the wall velocity in the bounce-back and equilibrium
// rules.  The entries (j, x - e_j) of lambda(n) at nodes fluid at n get the
// adjoint of the streamed f_j, plus that of the bounce-back of direction
// opp(j) unless x + e_j was fluid.
//
// Few nodes, so the time is one wave's chain of loads and arithmetic.  Each
// neighbour and its owner load once, all before the first use (the upstream
// candidate of i is the downstream one of opp i): 22 -> 10 us at 128^3 FP32
// with one body, 15 -> 8 us in 48 x 40 x 44 FP64.
template <int S>
__global__ __launch_bounds__(256) void k_adj_refill(const typename St<S>::T* __restrict__ f,
                                                    const uint32_t* __restrict__ own0,
                                                    const typename St<S>::A* __restrict__ lam1,
                                                    typename St<S>::A* __restrict__ lam0,
                                                    const double* pos1, const double* vel1,
                                                    const double* om1, Geom g, Phys ph,
                                                    double* grad, GeoArgs ga, AdjList list)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const uint32_t cnt = min(*list.count, list.cap);
    for (uint32_t l = blockIdx.x * 256u + threadIdx.x; l < cnt; l += gridDim.x * 256u) {
        const uint32_t cell = list.node[l];
        const int p = (int)own0[cell];
        // neighbours x - e_i with their owners and f_i, each once (x + e_i and
        // f_opp(i) are those of opp(i)), before any use
        uint32_t xc[3];
        node_xyz(cell, g, xc[0], xc[1], xc[2]);
        uint32_t o[3][3];
        bool in[3][3];
        axis3(xc[0], g.n[0], g.per[0], 1u, o[0], in[0]);
        axis3(xc[1], g.n[1], g.per[1], g.n[0], o[1], in[1]);
        axis3(xc[2], g.n[2], g.per[2], (uint32_t)g.n[0] * (uint32_t)g.n[1], o[2], in[2]);
        A lam[kQ], pre[kQ], fa[kQ];
        uint32_t nu[kQ], ow[kQ];
        lam[0] = lam1[cell];
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
            lam[i] = lam1[(int64_t)i * g.stride + cell];
            nu[i] = o[0][1 - cx(i)] + o[1][1 - cy(i)] + o[2][1 - cz(i)];
            fa[i] = St<S>::ld(f + (int64_t)i * g.stride + nu[i], ph.inv_scale);
            ow[i] = own0[nu[i]];
        }
        double rr[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double xp = pos1[3 * p + a];
            rr[a] = image_coord((int)xc[a], g.n[a], g.per[a], xp) - xp;
        }
        const double wp[3] = {om1[3 * p], om1[3 * p + 1], om1[3 * p + 2]};
        const A un[3] = {A(vel1[3 * p] + (wp[1] * rr[2] - wp[2] * rr[1])),
                         A(vel1[3 * p + 1] + (wp[2] * rr[0] - wp[0] * rr[2])),
                         A(vel1[3 * p + 2] + (wp[0] * rr[1] - wp[1] * rr[0]))};
        const A r0 = A(ph.rho0), dr0 = A(ph.rho0 - 1.0);
        const A uu = un[0] * un[0] + un[1] * un[1] + un[2] * un[2];
        uint32_t fl = 0;  // bit i: x - e_i lies in the lattice and was fluid at n
#pragma unroll
        for (int i = 1; i < kQ; ++i)
            if (in[0][1 - cx(i)] && in[1][1 - cy(i)] && in[2][1 - cz(i)] && ow[i] == kFluid) fl |= 1u << i;
        // per direction: streamed, bounced back, or the equilibrium
        pre[0] = eq_moving<DEV, A>(W<A>(0), dr0, r0, A(0), uu);
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
            const A eu = edot(i, un[0], un[1], un[2]);
            pre[i] = (fl >> i) & 1u        ? fa[i]
                     : (fl >> opp(i)) & 1u ? fa[opp(i)] + A(6) * W<A>(i) * r0 * eu
                                           : eq_moving<DEV, A>(W<A>(i), dr0, r0, eu, uu);
        }
        const AdjCoef<A> co = adj_collide<DEV, A>(lam, pre, ph, acc);
        A Lp[kQ];
#pragma unroll
        for (int j = 0; j < kQ; ++j) Lp[j] = co(j, lam[j]);
        // d pre_j / d u_new: 6 w rho0 e_j for the bounce-back rule, d feq_j(rho0,
        // u_new)/du = w rho0 ((3 + 9 e.u) e - 3 u) for the equilibrium
        // (summed in double)
        double dva[3] = {0.0, 0.0, 0.0}, su = (double)(A(-3) * W<A>(0) * r0 * Lp[0]);
#pragma unroll
        for (int j = 1; j < kQ; ++j) {
            const bool bounced = !((fl >> j) & 1u) && ((fl >> opp(j)) & 1u);
            const bool equi = !((fl >> j) & 1u) && !bounced;
            const A t = W<A>(j) * r0 * Lp[j];
            const double k = (double)(
                bounced ? A(6) * t : (equi ? t * (A(3) + A(9) * edot(j, un[0], un[1], un[2])) : A(0)));
            if (cx(j)) dva[0] += cx(j) > 0 ? k : -k;
            if (cy(j)) dva[1] += cy(j) > 0 ? k : -k;
            if (cz(j)) dva[2] += cz(j) > 0 ? k : -k;
            su += equi ? (double)(A(-3) * t) : 0.0;
        }
        const double dv[3] = {dva[0] + su * (double)un[0], dva[1] + su * (double)un[1],
                              dva[2] + su * (double)un[2]};
        double* vout = ga.v_refill ? ga.v_refill + (int64_t)ga.vstride * p : grad + 4 + 3 * p;
        for (int k = 0; k < 3; ++k)
            if (dv[k] != 0.0) atomicAdd(vout + k, dv[k]);
        if (ga.g_refill) {
            // u_new = v + omega x (x - x_p): dJ/dx_p = -(dJ/du_new) x omega
            const double gx[3] = {-(dv[1] * wp[2] - dv[2] * wp[1]), -(dv[2] * wp[0] - dv[0] * wp[2]),
                                  -(dv[0] * wp[1] - dv[1] * wp[0])};
            for (int k = 0; k < 3; ++k)
                if (gx[k] != 0.0) atomicAdd(ga.g_refill + (int64_t)ga.gstride * p + k, gx[k]);
        }
        if (ga.w_refill) {
            // dJ/domega = (x - x_p) x dJ/du_new
            const double gw[3] = {rr[1] * dv[2] - rr[2] * dv[1], rr[2] * dv[0] - rr[0] * dv[2],
                                  rr[0] * dv[1] - rr[1] * dv[0]};
            for (int k = 0; k < 3; ++k)
                if (gw[k] != 0.0) atomicAdd(ga.w_refill + (int64_t)ga.vstride * p + k, gw[k]);
        }
        // entries read through the streaming rule of direction j (x - e_j fluid
        // at n): f_j(x - e_j) also fed the bounce-back of opp(j) when x + e_j
        // was not fluid
#pragma unroll
        for (int j = 1; j < kQ; ++j)
            if ((fl >> j) & 1u) {
                const bool bb = !((fl >> opp(j)) & 1u);
                lam0[(int64_t)j * g.stride + nu[j]] = bb ? Lp[j] + Lp[opp(j)] : Lp[j];
            }
    }
    block_add<256>(acc, [=](int k) { return grad + k; });
}

// ---------------------------------------------------------------------------
// 2. links: reconstruction, momentum exchange and missing points
// ---------------------------------------------------------------------------
// With GEO, also dJ/dx_p of the pose the links were built from, with the
// link set held fixed: through q (Eq. appq, or Eq. calq by the implicit
// function theorem), which moves the VIBB weights and the wall point
// x_w = x_n + q e, and through the lever arm r = x_w - x_p of the torque
// weight and of u_w = v + omega x r.
template <int S, bool GEO, int T>
__global__ __launch_bounds__(T) void k_adj_links(const typename St<S>::T* __restrict__ f,
                                                   const LinkRec* __restrict__ links,
                                                   const uint32_t* __restrict__ cursor,
                                                   const int64_t* __restrict__ loff,
                                                   const uint32_t* __restrict__ chunk,
                                                   const double* pos,
                                                   const double* vel, const double* om,
                                                   typename St<S>::A* lam0, const double* wts,
                                                   Geom g, Phys ph, double* grad, GeoArgs ga)
{
    using A = typename St<S>::A;
    constexpr bool DEV = St<S>::dev;
    // one or four workgroups per 256-record chunk of the step's link layout (a
    // chunk's records are all allocated: they load beside the particle's index)
    const int64_t g0 = (int64_t)blockIdx.x * T;
    const LinkRec r = links[g0 + threadIdx.x];
    const int p = (int)chunk[blockIdx.x / (256 / T)];
    const int64_t cnt = min(loff[p + 1] - loff[p], (int64_t)cursor[(int64_t)p * kCursorPad]);
    if (g0 - loff[p] >= cnt) return;  // uniform over the block
    const int64_t l = g0 - loff[p] + threadIdx.x;
    // dJ/dF (3), dJ/dv_p (3), dJ/dx_p (3, GEO), dJ/dtheta_p (3, GEO),
    // dJ/domega_p (3, GEO)
    double acc[15] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (l < cnt) {
        const int d = r.d, db = opp_moving(d);
        int e[3];
        dir_of(d, e);
        const double ed[3] = {(double)e[0], (double)e[1], (double)e[2]};
        uint32_t sx, sy, sz;
        node_xyz(r.node, g, sx, sy, sz);
        int cn[3] = {(int)sx - e[0], (int)sy - e[1], (int)sz - e[2]};
        wrap3(cn, g);
        double rr[3], uw[3], Wv[3], Xn[3];
        const double xp[3] = {pos[3 * p], pos[3 * p + 1], pos[3 * p + 2]};
        const double wp[3] = {om[3 * p], om[3 * p + 1], om[3 * p + 2]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            Xn[a] = image_coord(cn[a], g.n[a], g.per[a], xp[a]);
            rr[a] = Xn[a] + r.q * ed[a] - xp[a];
        }
        uw[0] = vel[3 * p] + (wp[1] * rr[2] - wp[2] * rr[1]);
        uw[1] = vel[3 * p + 1] + (wp[2] * rr[0] - wp[0] * rr[2]);
        uw[2] = vel[3 * p + 2] + (wp[0] * rr[1] - wp[1] * rr[0]);
        // objective weight of this force point: wF + wT x r (J = F.wF + (r x F).wT)
        const double* wF = wts + 6 * p;
        const double wT[3] = {wts[6 * p + 3], wts[6 * p + 4], wts[6 * p + 5]};
        Wv[0] = wF[0] + (wT[1] * rr[2] - wT[2] * rr[1]);
        Wv[1] = wF[1] + (wT[2] * rr[0] - wT[0] * rr[2]);
        Wv[2] = wF[2] + (wT[0] * rr[1] - wT[1] * rr[0]);
        // weights of the outgoing and incoming population in J
        double d_out = 0.0, d_in = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            d_out += (ed[a] - uw[a]) * Wv[a];
            d_in += (ed[a] + uw[a]) * Wv[a];
        }
        // geometry terms: t = the link's momentum-exchange vector, G = dJ/du_w
        // of the link (all paths), dq = dJ/dq through the reconstruction
        double tv[3] = {0, 0, 0}, G[3] = {0, 0, 0}, dq = 0.0;
        if (r.kind == LBM_LINK_MISSING) {
            // J = [(e_d - u_w) feq_d(rho0, u_w) - (e_db - u_w) feq_db(rho0, u_w)] . W
            const double w = wgt_moving<double>(d), wr = w * ph.rho0;
            const double eu = ed[0] * uw[0] + ed[1] * uw[1] + ed[2] * uw[2];
            const double uu = uw[0] * uw[0] + uw[1] * uw[1] + uw[2] * uw[2];
            const double fo = eq_moving<false, double>(w, 0.0, ph.rho0, eu, uu);
            const double fi = eq_moving<false, double>(w, 0.0, ph.rho0, -eu, uu);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                G[a] = -Wv[a] * (fo - fi) + d_out * wr * (ed[a] * (3.0 + 9.0 * eu) - 3.0 * uw[a]) +
                       d_in * wr * (ed[a] * (9.0 * eu - 3.0) - 3.0 * uw[a]);
                tv[a] = (ed[a] - uw[a]) * fo + (ed[a] + uw[a]) * fi;
                acc[3 + a] = G[a];
            }
        } else {
            A F[3];
            if constexpr (DEV) {
                F[0] = ph.Ff[0], F[1] = ph.Ff[1], F[2] = ph.Ff[2];
            } else {
                F[0] = ph.F[0], F[1] = ph.F[1], F[2] = ph.F[2];
            }
            const uint32_t xf = node_of(cn, g);
            const bool vibb = r.kind == LBM_LINK_VIBB;
            uint32_t xff = xf;
            if (vibb) {
                int cf[3] = {cn[0] - e[0], cn[1] - e[1], cn[2] - e[2]};
                wrap3(cf, g);
                xff = node_of(cf, g);
            }
            // (halfway links load x_f twice: one batch either way)
            A v[kQ], vv[kQ];
#pragma unroll
            for (int i = 0; i < kQ; ++i) {
                v[i] = St<S>::ld(f + (int64_t)i * g.stride + xf, ph.inv_scale);
                vv[i] = St<S>::ld(f + (int64_t)i * g.stride + xff, ph.inv_scale);
            }
            LinkIn<A> x;
            LinkGrad<A> gk;
            A dr;
            x.fdf = St<S>::ld(f + (int64_t)d * g.stride + xf, ph.inv_scale);
            x.fdff = St<S>::ld(f + (int64_t)d * g.stride + xff, ph.inv_scale);
            // the node kernel left the adjoint of the ghost slot (x_s, opp d),
            // which x_f pulled, in lambda(n) at x_s; take it and clear it
            A* ghost = lam0 + (int64_t)db * g.stride + r.node;
            const A lu = *ghost + A(d_in);
            *ghost = A(0);
            moments<DEV, A>(v, A(-0.5), F, dr, x.rf, x.uf[0], x.uf[1], x.uf[2]);
            moments<DEV, A>(vv, A(-0.5), F, dr, x.rff, x.uff[0], x.uff[1], x.uff[2]);
#pragma unroll
            for (int a = 0; a < 3; ++a) x.uw[a] = A(uw[a]);
            x.q = A(r.q);
            const A ea[3] = {A(e[0]), A(e[1]), A(e[2])};
            const A unk = link_value<DEV, A>(r.kind, wgt_moving<A>(d), ea, x, ph.neq_split != 0, gk);
            // momentum exchange of this link: [(e_d - u_w) out - (e_db - u_w) in] . W
            double out = (double)x.fdf, inn = (double)unk;
            if constexpr (DEV) {
                out += wgt_moving<double>(d);
                inn += wgt_moving<double>(d);
            }
            // adjoint of the reconstructed value (lu): the fluid node that
            // pulled the ghost slot, plus the objective; pushed to the
            // populations of x_f and x_ff through f_d and the moments
            auto push = [&](uint32_t node, A gf, A gr, const A gu[3], const A u[3], A rho) {
                const A ir = A(1) / rho;
                const A hx = gu[0] * ir, hy = gu[1] * ir, hz = gu[2] * ir;
                const A c = gr - (hx * u[0] + hy * u[1] + hz * u[2]);
                atomicAdd(lam0 + (int64_t)d * g.stride + node, gf);
#pragma unroll
                for (int j = 0; j < kQ; ++j)
                    atomicAdd(lam0 + (int64_t)j * g.stride + node, j ? c + edot(j, hx, hy, hz) : c);
                acc[0] -= (double)(hx * A(0.5));
                acc[1] -= (double)(hy * A(0.5));
                acc[2] -= (double)(hz * A(0.5));
            };
            const A gf3[3] = {lu * gk.uf[0], lu * gk.uf[1], lu * gk.uf[2]};
            push(xf, lu * gk.fdf + A(d_out), lu * gk.rf, gf3, x.uf, x.rf);
            if (vibb) {
                const A gff3[3] = {lu * gk.uff[0], lu * gk.uff[1], lu * gk.uff[2]};
                push(xff, lu * gk.fdff, lu * gk.rff, gff3, x.uff, x.rff);
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                tv[a] = (ed[a] - uw[a]) * out + (ed[a] + uw[a]) * inn;
                G[a] = -(out - inn) * Wv[a] + (double)(lu * gk.uw[a]);
                acc[3 + a] = G[a];
            }
            if constexpr (GEO) dq = (double)(lu * gk.q);
        }
        if constexpr (GEO) {
            // dJ/dr: torque weight (wT x r).t and u_w = v + omega x r
            double Jr[3];
            Jr[0] = (tv[1] * wT[2] - tv[2] * wT[1]) + (G[1] * wp[2] - G[2] * wp[1]);
            Jr[1] = (tv[2] * wT[0] - tv[0] * wT[2]) + (G[2] * wp[0] - G[0] * wp[2]);
            Jr[2] = (tv[0] * wT[1] - tv[1] * wT[0]) + (G[0] * wp[1] - G[1] * wp[0]);
            dq += Jr[0] * e[0] + Jr[1] * e[1] + Jr[2] * e[2];
            // dq/dx_p and dq/dtheta_p: translating the body by dx moves M(X)
            // by -grad M(X).dx; a small rotation moves it by dM/dtheta
            const int i0 = ga.off[p], i1 = ga.off[p + 1];
            const double c0 = ga.c0[p];
            double qx[3], qt[3];
            if (ga.exact_q) {
                const double Xw[3] = {Xn[0] + r.q * e[0], Xn[1] + r.q * e[1], Xn[2] + r.q * e[2]};
                double M, gM[3], gR[3];
                metaball_grad(ga.wpts, ga.K, i0, i1, Xw, xp, M, gM, gR);
                const double ge = gM[0] * e[0] + gM[1] * e[1] + gM[2] * e[2];
                for (int a = 0; a < 3; ++a) {
                    qx[a] = gM[a] / ge;
                    qt[a] = -gR[a] / ge;
                }
            } else {
                const double Xs[3] = {Xn[0] + e[0], Xn[1] + e[1], Xn[2] + e[2]};
                double Mn, Ms, gn[3], gs[3], rn[3], rs[3];
                metaball_grad(ga.wpts, ga.K, i0, i1, Xn, xp, Mn, gn, rn);
                metaball_grad(ga.wpts, ga.K, i0, i1, Xs, xp, Ms, gs, rs);
                const double den = (Ms - Mn) * (Ms - Mn);
                const double an = (c0 - Ms) / den, as = (Mn - c0) / den;
                for (int a = 0; a < 3; ++a) {
                    qx[a] = -(an * gn[a] + as * gs[a]);
                    qt[a] = an * rn[a] + as * rs[a];
                }
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                acc[6 + a] = dq * qx[a] - Jr[a];
                acc[9 + a] = dq * qt[a];
            }
            // u_w = v + omega x r: dJ/domega = r x G
            acc[12] = rr[1] * G[2] - rr[2] * G[1];
            acc[13] = rr[2] * G[0] - rr[0] * G[2];
            acc[14] = rr[0] * G[1] - rr[1] * G[0];
        }
    }
    if constexpr (GEO) {
        double* gl = ga.g_links + (int64_t)ga.gstride * p;
        double* vl = ga.v_links ? ga.v_links + (int64_t)ga.vstride * p : grad + 4 + 3 * p;
        double* wl = ga.w_links + (int64_t)ga.vstride * p;
        auto out = [=](int k) {
            double* o = k < 3 ? grad + k : vl + (k - 3);
            o = k < 6 ? o : gl + (k - 6);
            return k < 12 ? o : wl + (k - 12);
        };
        if (ga.w_links) {
            block_add<T>(acc, out);
        } else {
            double a12[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) a12[k] = acc[k];
            block_add<T>(a12, out);
        }
    } else {
        double a6[6] = {acc[0], acc[1], acc[2], acc[3], acc[4], acc[5]};
        block_add<T>(a6, [=](int k) { return k < 3 ? grad + k : grad + 4 + 3 * p + (k - 3); });
    }
}

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + 255) / 256); }

// Up to one chunk per CU the link adjoint runs a wave per workgroup: its
// gathers and its scattered atomics go lane by lane through a CU's address
// unit, and one chunk's four waves then use four of them (one body in 128^3
// FP32: 30.7 -> 18.8 us; two in 48 x 40 x 44 FP64 with the poses: 23.7 -> 13.2).
// With 500 chunks and more the four-wave workgroup, with a quarter of the
// per-body sums, is as fast or faster (500: 96 us against 101; 20000: 3.12 ms
// against 3.28).
constexpr uint32_t kWaveChunks = 256;

template <int S>
struct RunAdj {
    static hipError_t run(lbm_ctx* c, const TapeStep& ts, const uint32_t* own1, const double* pos1,
                          const double* vel1, const double* om1, const void* lam1,
                          void* lam0, const double* wts, double* grad, const GeoArgs& ga,
                          const AdjList& list, int parts)
    {
        using T = typename St<S>::T;
        using A = typename St<S>::A;
        // Where two adjoint fields and a taped level outgrow the 256 MB memory-side
        // cache, the taped level, which nothing reads again, and the planes stored
        // whole go past it, and lambda stays for the next step.  Node, refill and
        // link kernels of a 16-step window of one body, cached and past it, us:
        // below the line 104^3 FP32 69.0 and 71.9, 80^3 FP64 66.7 and 67.5, 112^3
        // FP16 76.3 and 77.9; above 112^3 FP32 92.8 and 84.5, 128^3 127.7 and 108.9,
        // 96^3 FP64 108.0 and 87.4, 128^3 226 and 211, 160^3 FP16 192 and 181; from
        // four times the cache on even (200^3 FP32 441 and 456, FP16 359 and 361,
        // 160^3 FP64 411 and 397), so cached there.
        const int64_t bytes = (int64_t)sizeof(A) * 2 * kQ * c->geom.stride + (int64_t)c->sizes.population_bytes;
        const bool nt = bytes > ((int64_t)1 << 28) && bytes < ((int64_t)1 << 30);
        if (parts & kAdjNode)
            hipLaunchKernelGGL((nt ? k_adj_node<S, true> : k_adj_node<S, false>),
                               dim3(blocks_for(c->geom.ncell)), dim3(256), 0,
                               c->stream, (const T*)ts.f, ts.own_use, own1, (const A*)lam1, (A*)lam0,
                               c->geom, c->phys, grad, list);
        if (parts & kAdjRefill) {
            // a grid that one round of resident workgroups covers
            const uint32_t nb = std::min<uint32_t>(blocks_for(list.cap), 512u);
            hipLaunchKernelGGL(k_adj_refill<S>, dim3(nb), dim3(256), 0, c->stream, (const T*)ts.f,
                               ts.own_use, (const A*)lam1, (A*)lam0, pos1, vel1, om1, c->geom, c->phys,
                               grad, ga, list);
        }
        if ((parts & kAdjLinks) && c->cfg.n_particles > 0 && ts.link_max > 0 && ts.lay &&
            ts.lay->chunks() > 0) {
            const int np = c->cfg.n_particles;
            const uint32_t nch = (uint32_t)ts.lay->chunks();
            auto go = [&](auto geo, auto threads) {
                constexpr int T_ = decltype(threads)::value;
                hipLaunchKernelGGL((k_adj_links<S, decltype(geo)::value, T_>), dim3(nch * (256 / T_)),
                                   dim3(T_), 0, c->stream, (const T*)ts.f, ts.links_use, ts.cursor,
                                   ts.lay->off_dev, ts.lay->chunk_dev, ts.part, ts.part + 3 * np,
                                   ts.part + 6 * np, (A*)lam0, wts, c->geom, c->phys, grad, ga);
            };
            using One = std::integral_constant<int, 64>;
            using Four = std::integral_constant<int, 256>;
            const bool waves = nch <= kWaveChunks;
            if (ga.g_links)
                waves ? go(std::true_type{}, One{}) : go(std::true_type{}, Four{});
            else
                waves ? go(std::false_type{}, One{}) : go(std::false_type{}, Four{});
        }
        return hipGetLastError();
    }
};

// One taped step in one launch: the owner plane and the links; and by the first
// threads the small arrays: the first word of every link cursor line, the
// particle state (position, velocity, angular velocity, world control points,
// quaternion, F^h and T^h of the step), and the DEM state the next dem_step
// starts from (pair records, wall records, carried contact sums; the pair
// records' keys).
__global__ __launch_bounds__(256) void k_tape(CopySeg own, CopySeg links, uint32_t* __restrict__ tcur, const uint32_t* __restrict__ cur,
                       double* __restrict__ part, const double* __restrict__ pos,
                       const double* __restrict__ vel, const double* __restrict__ om,
                       const double* __restrict__ wpts, const double* __restrict__ quat,
                       const double* __restrict__ sums,
                       const unsigned long long* __restrict__ fx, int np, int nctrl,
                       double* __restrict__ dem, int32_t* __restrict__ dem_key,
                       const double* __restrict__ hpp, const double* __restrict__ hpw,
                       const double* __restrict__ fc, const int32_t* __restrict__ hkey)
{
    const int i = (int)(blockIdx.x * 256u + threadIdx.x);
    copy_segment(own, (uint64_t)i, (uint64_t)gridDim.x * 256u);
    copy_segment(links, (uint64_t)i, (uint64_t)gridDim.x * 256u);
    if (i < np) tcur[(int64_t)i * kCursorPad] = cur[(int64_t)i * kCursorPad];
    if (i < 3 * np) {
        part[i] = pos[i];
        part[3 * np + i] = vel[i];
        part[6 * np + i] = om[i];
    }
    if (i < 3 * nctrl) part[9 * np + i] = wpts[i];
    double* tq = part + 9 * np + 3 * nctrl;
    if (quat && i < 4 * np) tq[i] = quat[i];
    if (i < 6 * np) tq[4 * np + i] = force_sum(sums, fx, i);
    const int npp = np * kPairSlots;
    if (i < 8 * npp) dem[i] = hpp[i];
    if (i < 48 * np) dem[8 * npp + i] = hpw[i];
    if (i < 6 * np) dem[8 * npp + 48 * np + i] = fc[i];
    if (i < npp) dem_key[i] = hkey[i];
}

}  // namespace

namespace MDLBM_QNS {

hipError_t launch_tape(lbm_ctx* c, TapeStep& t, const lbm_particles* P, const CopySeg& own,
                       const CopySeg& links)
{
    const int np = c->cfg.n_particles, nctrl = c->cfg.n_ctrl;
    // a thread per number of the small arrays, and as many as copy the large
    // ones well
    const uint64_t n = np ? std::max<uint64_t>({8 * (uint64_t)np * kPairSlots, 48 * (uint64_t)np,
                                                3 * (uint64_t)nctrl})
                          : 1;
    const uint64_t most = std::min<uint64_t>(std::max(own.bytes, links.bytes) / 16, 2048 * 256);
    hipLaunchKernelGGL(k_tape, dim3((uint32_t)((std::max(n, most) + 255) / 256)), dim3(256), 0,
                       c->stream, own, links, t.cursor, c->link_cursor, t.part, P ? P->pos : nullptr,
                       P ? P->vel : nullptr, P ? P->omega : nullptr, P ? P->world_pts : nullptr,
                       P ? P->quat : nullptr, c->sums, c->FX, np, np ? nctrl : 0, t.dem, t.dem_key,
                       c->hist_pp, c->hist_pw, c->fc, c->hist_key);
    return hipGetLastError();
}

hipError_t launch_adjoint_step(lbm_ctx* c, const TapeStep& ts, const uint32_t* own1,
                               const double* pos1, const double* vel1, const double* om1,
                               const void* lam1, void* lam0, const double* wts,
                               double* grad, const lbm_particles* P, const AdjOut& out,
                               const AdjList& list, int parts)
{
    GeoArgs ga;
    const int np = c->cfg.n_particles;
    ga.wpts = ts.part + 9 * np;
    ga.K = P->K;
    ga.c0 = P->c0;
    ga.off = P->ctrl_off;
    ga.exact_q = (c->cfg.treatments & LBM_TREAT_EXACT_Q) ? 1 : 0;
    ga.g_links = out.g_links;
    ga.g_refill = out.g_refill;
    ga.gstride = out.gstride;
    ga.v_links = out.v_links;
    ga.v_refill = out.v_refill;
    ga.w_links = out.w_links;
    ga.w_refill = out.w_refill;
    ga.vstride = out.vstride;
    switch (c->cfg.storage) {
    case LBM_STORE_F64:
        return RunAdj<LBM_STORE_F64>::run(c, ts, own1, pos1, vel1, om1, lam1, lam0, wts, grad, ga,
                                          list, parts);
    case LBM_STORE_F32:
        return RunAdj<LBM_STORE_F32>::run(c, ts, own1, pos1, vel1, om1, lam1, lam0, wts, grad, ga,
                                          list, parts);
    case LBM_STORE_F16:
        return RunAdj<LBM_STORE_F16>::run(c, ts, own1, pos1, vel1, om1, lam1, lam0, wts, grad, ga,
                                          list, parts);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace MDLBM_QNS
}  // namespace mdlbm
