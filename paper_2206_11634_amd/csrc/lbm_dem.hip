// Metaball DEM of libmdlbm in FP64 on the GPU (Sec. 2.1, with the
// sub-cycling of Sec. 2.3.4): velocity Verlet for translation, Euler's
// equations in the principal body frame for rotation, linear spring-dashpot
// normal force and Coulomb-limited tangential spring, metaball-metaball
// contacts by Newton-Raphson on grad(M_i + M_j) = 0 (Eqs. opt, grad, cp, k0,
// contactprop) and metaball-wall contacts by Newton on the in-plane gradient
// (Eqs. metawall, metawallcp, k, contactprop2).
//
// The work is latency-bound (chains of FP64 operations on a few thousand
// particles at most), not HBM-bound.  Up to kBlockParticles particles one
// workgroup runs the whole call: the broad phase and every substep, with
// barriers where more particles take a launch; the first wave moves the
// particles (a lane each) and takes their wall contacts (a lane each), the other
// waves take the candidate pairs (kPairLanes lanes each), and what a substep hands
// over lies in LDS.  Beyond, k_open, the broad phase (on the cell grid from
// kGridMinParticles on), one k_substep a substep and k_close.  Both half kicks
// around a substep's start act in the body frame, with one rotation matrix a pose
// and Euler's terms as products of two components; half angles come from their
// series.
// Measured, microseconds a call of ten substeps (in parentheses a thread per
// pair, per pair test and per particle's cells, 23 launches whatever the count):
//   1 sphere 13.5 (83), 2 flat metaballs 36 (153), 64 packed spheres 69 (173),
//   1000 metaballs of the 512^3 run 190 (535), packed spheres 1000: 121 (226),
//   2548: 123 (420), 8000: 137 (462), 27 000: 310 (745); a body of 64 points in a
//   corner of three walls 267 (752; 1063 with its wall contacts one after the
//   other on the body's lane and their coordinates picked from all three).
#include <algorithm>
#include <mutex>

#include "lbm_fp64.h"
#include "lbm_internal.h"

namespace mdlbm {
namespace {

constexpr int kHist = 8;  // active, xi[3], warm start[3], pad
constexpr int kMaxPts = 64;

struct DemP {
    double kn, etan, kt, etat, mu, ctol, ntol2;
    int niter;
    double g[3];
    double rhof;
};

__device__ __forceinline__ void cross3(const double a[3], const double b[3], double c[3])
{
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ __forceinline__ double dot3(const double a[3], const double b[3])
{
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

__device__ __forceinline__ void rotmat(const double q[4], double R[9])
{
    const double w = q[0], x = q[1], y = q[2], z = q[3];
    R[0] = 1 - 2 * (y * y + z * z);
    R[1] = 2 * (x * y - w * z);
    R[2] = 2 * (x * z + w * y);
    R[3] = 2 * (x * y + w * z);
    R[4] = 1 - 2 * (x * x + z * z);
    R[5] = 2 * (y * z - w * x);
    R[6] = 2 * (x * z - w * y);
    R[7] = 2 * (y * z + w * x);
    R[8] = 1 - 2 * (x * x + y * y);
}

// Sum over the G lanes of a pair's group (2 or 4 lanes of a quad, exchanged by
// quad permutes; the same bits in each of them).
template <int CTRL>
__device__ __forceinline__ double quad_perm(double v)
{
    union {
        double d;
        int w[2];
    } u;
    u.d = v;
    u.w[0] = __builtin_amdgcn_mov_dpp(u.w[0], CTRL, 0xf, 0xf, true);
    u.w[1] = __builtin_amdgcn_mov_dpp(u.w[1], CTRL, 0xf, 0xf, true);
    return u.d;
}
template <int G>
__device__ __forceinline__ double gsum(double v)
{
    static_assert(G == 1 || G == 2 || G == 4, "a group is part of a quad");
    if constexpr (G >= 2) v += quad_perm<0xB1>(v);  // lanes 1 0 3 2
    if constexpr (G >= 4) v += quad_perm<0x4E>(v);  // lanes 2 3 0 1
    return v;
}

// Terms of one control point at distance r: its share of M, grad M (negated:
// s r with s = 2 K / r^4) and the upper triangle of the Hessian.
__device__ __forceinline__ void add_point(double K, const double r[3], double i2, double& M,
                                          double g[3], double H[6])
{
    const double t = K * i2, s = 2.0 * t * i2, q = 4.0 * s * i2;
    M += t;
    g[0] -= s * r[0];
    g[1] -= s * r[1];
    g[2] -= s * r[2];
    const double q0 = q * r[0], q1 = q * r[1], q2 = q * r[2];
    H[0] += q0 * r[0] - s;
    H[1] += q0 * r[1];
    H[2] += q0 * r[2];
    H[3] += q1 * r[1] - s;
    H[4] += q1 * r[2];
    H[5] += q2 * r[2] - s;
}

// dx = -H^-1 g for a symmetric H (upper triangle).
__device__ __forceinline__ bool solve3(const double H[6], const double g[3], double dx[3])
{
    const double a = H[0], b = H[1], c = H[2], d = H[3], e = H[4], f = H[5];
    const double c00 = d * f - e * e, c01 = c * e - b * f, c02 = b * e - c * d;
    const double c11 = a * f - c * c, c12 = b * c - a * e, c22 = a * d - b * b;
    const double det = a * c00 + b * c01 + c * c02;
    if (!(fabs(det) > 0.0) || !isfinite(det)) return false;
    const double s = -fast_rcp(det);
    dx[0] = s * (c00 * g[0] + c01 * g[1] + c02 * g[2]);
    dx[1] = s * (c01 * g[0] + c11 * g[1] + c12 * g[2]);
    dx[2] = s * (c02 * g[0] + c12 * g[1] + c22 * g[2]);
    return true;
}

__device__ __forceinline__ double reach(const PartDev& P, int p)
{
    return reach_of(P.body_pts, P.K, P.off[p], P.off[p + 1]);
}

// Normal spring-dashpot (clamped at zero) and tangential spring with Coulomb
// limit; updates the spring xi; returns the force on body i.
__device__ __forceinline__ void contact_force(const DemP& c, double delta, const double n[3],
                                              const double vrel[3], double dt, double xi[3],
                                              double Fi[3])
{
    const double vn = dot3(vrel, n);
    double Fn = c.kn * delta - c.etan * vn;
    if (Fn < 0.0) Fn = 0.0;
    double vt[3], Ft[3];
    for (int a = 0; a < 3; ++a) vt[a] = vrel[a] - vn * n[a];
    const double xin = dot3(xi, n);
    for (int a = 0; a < 3; ++a) xi[a] = xi[a] - xin * n[a] + vt[a] * dt;
    for (int a = 0; a < 3; ++a) Ft[a] = -c.kt * xi[a] - c.etat * vt[a];
    const double ft2 = dot3(Ft, Ft), lim = c.mu * Fn;
    // |Ft| > lim, of either sign
    if (ft2 > lim * fabs(lim) && ft2 > 0.0) {
        const double s = lim * fast_rsqrt(ft2), ik = 1.0 / c.kt;
        for (int a = 0; a < 3; ++a) {
            Ft[a] *= s;
            xi[a] = -(Ft[a] + c.etat * vt[a]) * ik;
        }
    }
    for (int a = 0; a < 3; ++a) Fi[a] = Fn * n[a] + Ft[a];
}

// A particle's state and constants in registers.
struct Body {
    double x[3], q[4], v[3], w[3];  // centre, orientation, velocity, angular velocity
    double R[9], wb[3];             // rotation of q, angular velocity in the body frame
    double F[3], T[3];              // F^h + relative gravity, T^h
    double hm, hI[3], kI[3];        // half step over the mass and the moments; of Euler's terms
    int c0, c1;                     // control points
};

__device__ __forceinline__ void to_body(Body& b)
{
    for (int i = 0; i < 3; ++i) b.wb[i] = b.R[i] * b.w[0] + b.R[3 + i] * b.w[1] + b.R[6 + i] * b.w[2];
}
__device__ __forceinline__ void to_world(Body& b)
{
    for (int i = 0; i < 3; ++i)
        b.w[i] = b.R[3 * i] * b.wb[0] + b.R[3 * i + 1] * b.wb[1] + b.R[3 * i + 2] * b.wb[2];
}

__device__ __forceinline__ Body load_body(const PartDev& P, int p, const double* FTh, const DemP& c,
                                          double h)
{
    Body b;
    const double m = P.mass[p];
    const double mrel = m - c.rhof * P.volume[p];
    b.hm = h / m;
    b.c0 = P.off[p];
    b.c1 = P.off[p + 1];
    double I[3];
    for (int a = 0; a < 3; ++a) {
        b.x[a] = P.pos[3 * p + a];
        b.v[a] = P.vel[3 * p + a];
        b.w[a] = P.omega[3 * p + a];
        I[a] = P.inertia[3 * p + a];
        b.hI[a] = h / I[a];
        b.F[a] = FTh[6 * p + a] + mrel * c.g[a];
        b.T[a] = FTh[6 * p + 3 + a];
    }
    // (w x I w)_0 = (I_2 - I_1) w_1 w_2, and so on
    for (int a = 0; a < 3; ++a) b.kI[a] = b.hI[a] * (I[(a + 2) % 3] - I[(a + 1) % 3]);
    for (int a = 0; a < 4; ++a) b.q[a] = P.quat[4 * p + a];
    rotmat(b.q, b.R);
    to_body(b);
    return b;
}

// What half a kick under F, T and the contact sum fc adds to v and, without
// Euler's terms, to the angular velocity in the body frame.
struct Kick {
    double v[3], w[3];
};

__device__ __forceinline__ Kick kick_of(const Body& b, const double fc[6])
{
    Kick k;
    double T[3];
    for (int a = 0; a < 3; ++a) {
        k.v[a] = b.hm * (b.F[a] + fc[a]);
        T[a] = b.T[a] + fc[3 + a];
    }
    for (int a = 0; a < 3; ++a)
        k.w[a] = b.hI[a] * (b.R[a] * T[0] + b.R[3 + a] * T[1] + b.R[6 + a] * T[2]);
    return k;
}

// Half a kick: of the velocity, and of the rotation by one explicit or four
// fixed-point sweeps of Euler's equations.
__device__ __forceinline__ void kick_v(Body& b, const Kick& k)
{
    for (int a = 0; a < 3; ++a) b.v[a] += k.v[a];
}
template <bool IMPLICIT>
__device__ __forceinline__ void kick_w(Body& b, const Kick& k)
{
    double w0[3];
    for (int a = 0; a < 3; ++a) w0[a] = b.wb[a] + k.w[a];
#pragma unroll
    for (int it = 0; it < (IMPLICIT ? 4 : 1); ++it) {
        const double p0 = b.wb[1] * b.wb[2], p1 = b.wb[2] * b.wb[0], p2 = b.wb[0] * b.wb[1];
        b.wb[0] = w0[0] - b.kI[0] * p0;
        b.wb[1] = w0[1] - b.kI[1] * p1;
        b.wb[2] = w0[2] - b.kI[2] * p2;
    }
}

// The centre's drift over dt.
__device__ __forceinline__ void move(Body& b, double dt, const Geom& g)
{
    for (int a = 0; a < 3; ++a) {
        double x = b.x[a] + dt * b.v[a];
        if (g.per[a]) {
            if (x >= (double)g.n[a]) x -= g.n[a];
            else if (x < 0.0) x += g.n[a];
        }
        b.x[a] = x;
    }
}

// The rotation over dt (w and wb both hold the angular velocity).
__device__ __forceinline__ void rotate(Body& b, double dt)
{
    // cos(t) and sin(t) / |w| of half the angle t = |w| dt / 2
    const double z = (0.25 * dt * dt) * dot3(b.w, b.w);
    double dq[4], s;
    if (z < kSmallAngle2) {
        dq[0] = cos_series(z);
        s = (0.5 * dt) * sinc_series(z);
    } else {
        const double wn = sqrt(dot3(b.w, b.w));
        double sn;
        sincos(0.5 * wn * dt, &sn, &dq[0]);
        s = sn / wn;
    }
    for (int a = 0; a < 3; ++a) dq[1 + a] = s * b.w[a];
    const double* q = b.q;
    double qn[4];
    qn[0] = dq[0] * q[0] - dq[1] * q[1] - dq[2] * q[2] - dq[3] * q[3];
    qn[1] = dq[0] * q[1] + dq[1] * q[0] + dq[2] * q[3] - dq[3] * q[2];
    qn[2] = dq[0] * q[2] - dq[1] * q[3] + dq[2] * q[0] + dq[3] * q[1];
    qn[3] = dq[0] * q[3] + dq[1] * q[2] - dq[2] * q[1] + dq[3] * q[0];
    const double in = fast_rsqrt(qn[0] * qn[0] + qn[1] * qn[1] + qn[2] * qn[2] + qn[3] * qn[3]);
    for (int a = 0; a < 4; ++a) b.q[a] = qn[a] * in;
    rotmat(b.q, b.R);
    to_body(b);
}

// The world control points of the pose, from and to arrays indexed alike; N
// points' loads go before the first store, which could alias them (from global
// memory N = 4: a call's substep of 200 metaballs 4.5 us, point by point 5.7).
template <int N>
__device__ __forceinline__ void place_points(const Body& b, int i0, int i1, const double* body,
                                             double* world)
{
    for (int i = i0; i < i1; i += N) {
        double r[N][3];
#pragma unroll
        for (int k = 0; k < N; ++k)
            for (int a = 0; a < 3; ++a) r[k][a] = body[3 * (int64_t)min(i + k, i1 - 1) + a];
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (i + k < i1)
                for (int a = 0; a < 3; ++a)
                    world[3 * (int64_t)(i + k) + a] =
                        b.x[a] + (b.R[3 * a] * r[k][0] + b.R[3 * a + 1] * r[k][1] + b.R[3 * a + 2] * r[k][2]);
    }
}

__device__ __forceinline__ void store_body(const PartDev& P, int p, const Body& b, bool pose)
{
    for (int a = 0; a < 3; ++a) {
        P.vel[3 * p + a] = b.v[a];
        P.omega[3 * p + a] = b.w[a];
        if (pose) P.pos[3 * p + a] = b.x[a];
    }
    if (pose)
        for (int a = 0; a < 4; ++a) P.quat[4 * p + a] = b.q[a];
}

// What a contact reads of a particle at the current substep.
struct Kin {
    double x[3], v[3], w[3], rs, reach;
    const double* K;  // its control points' weights
    int n;            // their number
};

__device__ __forceinline__ void clear_record(double* h)
{
    for (int k = 0; k < kHist; ++k) h[k] = 0.0;
}

// Whether a pair is within reach; sh takes the second centre to its image
// nearest the first.
__device__ __forceinline__ bool near_pair(const double xi[3], const double xj[3], double far,
                                          const Geom& g, double sh[3])
{
    double dv[3];
    for (int a = 0; a < 3; ++a) {
        const double d = xj[a] - xi[a];
        sh[a] = 0.0;
        if (g.per[a]) {
            const double L = g.n[a];
            if (d > 0.5 * L) sh[a] = -L;
            else if (d < -0.5 * L) sh[a] = L;
        }
        dv[a] = d + sh[a];
    }
    return !(dot3(dv, dv) > far * far);
}

// Contact of pair (A, B) within reach, A the lower index, record h of A:
// Newton on grad(M_A + M_B) = 0 from the recorded point or the closest pair
// of control points (point(u, r, K): world coordinates and weight of point u of
// the pair, A's, then B's at their image nearest A), the contact test and the
// force.  The G lanes of a group share a pair: each sums every G-th control
// point of the two bodies (kept in registers up to 4 a lane), and all follow the
// same branches on the same bits.  A contact's force on A and the torques of it
// about A and, the other way, B go to emit(F, tA, tB) on the group's first lane.
template <int G, class Point, class Emit>
__device__ __forceinline__ void pair_item(const Kin& A, const Kin& B, const double sh[3], Point&& point,
                                          double* h, const DemP& c, double dt, int l, Emit&& emit)
{
    const double *xi = A.x, *xj = B.x;
    const double rsi = A.rs, rsj = B.rs;
    const double active = h[0];
    const int ni = A.n, nj = B.n, nt = ni + nj;
    constexpr int R = G == 2 ? 1 : 4;  // two lanes: two spheres
    double pr[R][3], kr[R];
    const bool regs = nt <= G * R;
    if (regs) {
        // (the last point again beyond the end: no branch between the loads)
#pragma unroll
        for (int k = 0; k < R; ++k) point(min(l + G * k, nt - 1), pr[k], kr[k]);
    }
    double x[3];
    if (active != 0.0) {
        for (int a = 0; a < 3; ++a) x[a] = xi[a] + h[4 + a];
    } else {
        double best = INFINITY;
        int at = 0x7fffffff;
        for (int t = l; t < ni * nj; t += G) {
            double p[3], q[3], K, d2 = 0.0;
            point(t / nj, p, K);
            point(ni + t % nj, q, K);
            for (int a = 0; a < 3; ++a) d2 += (p[a] - q[a]) * (p[a] - q[a]);
            if (d2 < best) {
                best = d2;
                at = t;
            }
        }
        // the first of the closest
#pragma unroll
        for (int m = 1; m < G; m <<= 1) {
            const double ob = __shfl_xor(best, m, 64);
            const int oa = __shfl_xor(at, m, 64);
            if (ob < best || (ob == best && oa < at)) {
                best = ob;
                at = oa;
            }
        }
        if (at == 0x7fffffff) at = 0;
        double p[3], q[3], K;
        point(at / nj, p, K);
        point(ni + at % nj, q, K);
        for (int a = 0; a < 3; ++a) x[a] = 0.5 * (p[a] + q[a]);
    }
    bool conv = false;
    for (int it = 0; it < c.niter; ++it) {
        double M = 0.0, gg[3] = {0, 0, 0}, H[6] = {0, 0, 0, 0, 0, 0}, dx[3];
        if (regs) {
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (l + G * k < nt) {
                    const double r[3] = {x[0] - pr[k][0], x[1] - pr[k][1], x[2] - pr[k][2]};
                    add_point(kr[k], r, fast_rcp(dot3(r, r)), M, gg, H);
                }
        } else {
            for (int u = l; u < nt; u += G) {
                double r[3], K;
                point(u, r, K);
                for (int a = 0; a < 3; ++a) r[a] = x[a] - r[a];
                add_point(K, r, fast_rcp(dot3(r, r)), M, gg, H);
            }
        }
        if constexpr (G > 1) {
            for (int a = 0; a < 3; ++a) gg[a] = gsum<G>(gg[a]);
            for (int a = 0; a < 6; ++a) H[a] = gsum<G>(H[a]);
        }
        if (!solve3(H, gg, dx)) break;
        for (int a = 0; a < 3; ++a) x[a] += dx[a];
        if (dot3(dx, dx) < c.ntol2) {
            conv = true;
            break;
        }
    }
    if (!conv) {
        if (l == 0) clear_record(h);
        return;
    }
    // M and grad M of each body at the stationary point
    double MA = 0.0, MB = 0.0, gA[3] = {0, 0, 0}, gB[3] = {0, 0, 0};
    auto field = [&](int u, double K, const double p[3]) __attribute__((always_inline)) {
        const double r[3] = {x[0] - p[0], x[1] - p[1], x[2] - p[2]};
        const double i2 = fast_rcp(dot3(r, r)), t = K * i2, s = 2.0 * t * i2;
        if (u < ni) {
            MA += t;
            for (int a = 0; a < 3; ++a) gA[a] -= s * r[a];
        } else {
            MB += t;
            for (int a = 0; a < 3; ++a) gB[a] -= s * r[a];
        }
    };
    if (regs) {
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (l + G * k < nt) field(l + G * k, kr[k], pr[k]);
    } else {
        for (int u = l; u < nt; u += G) {
            double p[3], K;
            point(u, p, K);
            field(u, K, p);
        }
    }
    if constexpr (G > 1) {
        MA = gsum<G>(MA);
        MB = gsum<G>(MB);
        for (int a = 0; a < 3; ++a) {
            gA[a] = gsum<G>(gA[a]);
            gB[a] = gsum<G>(gB[a]);
        }
    }
    if (l != 0) return;
    // both bodies' fields above ctol at the stationary point (Eq. opt); the
    // separation is signed along the common line of the two projections of
    // Eq. cp, n = (grad M_i - grad M_j)/|.| from body j to body i, so that a
    // stationary point already inside one internal body (two flat faces
    // meeting at an angle) reads as an overlap rather than as no contact;
    // overlaps beyond 2 (R_si + R_sj) are stationary points inside a body,
    // where the projection of Eq. k0 does not hold, and are not contacts
    if (!(MA > c.ctol && MB > c.ctol)) return clear_record(h);
    const double qA = (1.0 - MA) * fast_rcp(dot3(gA, gA)), qB = (1.0 - MB) * fast_rcp(dot3(gB, gB));
    double xa[3], dd[3], n[3];
    for (int a = 0; a < 3; ++a) {
        xa[a] = x[a] + qA * gA[a];
        dd[a] = xa[a] - (x[a] + qB * gB[a]);
        n[a] = gA[a] - gB[a];
    }
    const double n2 = dot3(n, n);
    if (!(n2 > 0.0)) return clear_record(h);
    const double un = fast_rsqrt(n2);
    for (int a = 0; a < 3; ++a) n[a] = n[a] * un;
    const double delta = rsi + rsj - dot3(dd, n);
    if (!(delta <= 2.0 * (rsi + rsj))) return clear_record(h);
    h[0] = 1.0;
    for (int a = 0; a < 3; ++a) h[4 + a] = x[a] - xi[a];
    if (delta <= 0.0) {
        h[1] = h[2] = h[3] = 0.0;
        return;
    }
    double xcp[3], ra[3], rb[3];
    for (int a = 0; a < 3; ++a) {
        xcp[a] = xa[a] - (rsi - 0.5 * delta) * n[a];
        ra[a] = xcp[a] - xi[a];
        rb[a] = xcp[a] - (xj[a] + sh[a]);
    }
    double ca[3], cb[3], vrel[3], Fi[3], ti[3], tj[3], spring[3] = {h[1], h[2], h[3]};
    cross3(A.w, ra, ca);
    cross3(B.w, rb, cb);
    for (int a = 0; a < 3; ++a) vrel[a] = (A.v[a] + ca[a]) - (B.v[a] + cb[a]);
    contact_force(c, delta, n, vrel, dt, spring, Fi);
    for (int a = 0; a < 3; ++a) h[1 + a] = spring[a];
    cross3(ra, Fi, ti);
    cross3(rb, Fi, tj);
    emit(Fi, ti, tj);
}

// Component a of v (a known at run time).
__device__ __forceinline__ double component(const double v[3], int a)
{
    return a == 0 ? v[0] : (a == 1 ? v[1] : v[2]);
}

// Whether a particle whose centre lies at xa along axis ax can touch that
// axis's wall on a side.
__device__ __forceinline__ bool near_wall(double xa, double lim, int ax, int side, const Geom& g)
{
    return !((side ? (double)g.n[ax] - 0.5 - xa : xa + 0.5) > lim);
}

// Contact of particle A with wall (ax, side) near it, record h: in-plane Newton
// for the point of the wall plane where M is largest, the contact test and the
// force; the force and its torque go to emit(F, t).  pa(u, r): point u along the
// wall's normal axis and the two after it.
template <int R, class PA, class Emit>
__device__ __forceinline__ void wall_contact(const Kin& A, PA&& pa, double* h, int ax, int side,
                                             const DemP& c, double dt, const Geom& g, Emit&& emit)
{
    const double plane = side ? g.n[ax] - 0.5 : -0.5, sgn = side ? -1.0 : 1.0;
    const int t1 = (ax + 1) % 3, t2 = (ax + 2) % 3;
    const double xa = component(A.x, ax), x1 = component(A.x, t1), x2 = component(A.x, t2);
    const double active = h[0];
    const int ni = A.n;
    // the points along (ax, t1, t2), up to R in registers: a loop that reads them
    // from memory again waits for each (1000 metaballs, some near a wall: 36 us a
    // substep, 17 from registers); from LDS (R = 0) the loop is as good
    double pr[R ? R : 1][3], kr[R ? R : 1];
    const bool regs = R && ni <= R && ni > 0;
    auto load = [&](int u, double r[3], double& K) __attribute__((always_inline)) {
        pa(u, r);
        K = A.K[u];
    };
    if (regs) {
#pragma unroll
        for (int k = 0; k < R; ++k) load(min(k, ni - 1), pr[k], kr[k]);
    }
    auto each = [&](auto&& fn) __attribute__((always_inline)) {
        if (regs) {
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k < ni) fn(pr[k], kr[k]);
        } else {
            for (int u = 0; u < ni; ++u) {
                double p[3], K;
                load(u, p, K);
                fn(p, K);
            }
        }
    };
    double y1, y2;
    if (active != 0.0) {
        y1 = x1 + h[4 + t1];
        y2 = x2 + h[4 + t2];
    } else {
        double best = INFINITY;
        y1 = y2 = 0.0;
        bool first = true;
        each([&](const double p[3], double) __attribute__((always_inline)) {
            const double dd = fabs(p[0] - plane);
            if (dd < best || first) {
                best = dd;
                y1 = p[1];
                y2 = p[2];
            }
            first = false;
        });
    }
    bool conv = false;
    for (int it = 0; it < c.niter; ++it) {
        double M = 0.0, gr[3] = {0, 0, 0}, H[6] = {0, 0, 0, 0, 0, 0};
        each([&](const double p[3], double K) __attribute__((always_inline)) {
            const double r[3] = {plane - p[0], y1 - p[1], y2 - p[2]};
            add_point(K, r, fast_rcp(dot3(r, r)), M, gr, H);
        });
        const double h11 = H[3], h12 = H[4], h22 = H[5];
        const double det = h11 * h22 - h12 * h12;
        if (!(fabs(det) > 0.0) || !isfinite(det)) break;
        const double s = -fast_rcp(det);
        const double d1 = s * (h22 * gr[1] - h12 * gr[2]);
        const double d2 = s * (h11 * gr[2] - h12 * gr[1]);
        y1 += d1;
        y2 += d2;
        if (d1 * d1 + d2 * d2 < c.ntol2) {
            conv = true;
            break;
        }
    }
    if (!conv) return clear_record(h);
    double M = 0.0, gr[3] = {0, 0, 0};
    each([&](const double p[3], double K) __attribute__((always_inline)) {
        const double r[3] = {plane - p[0], y1 - p[1], y2 - p[2]};
        const double i2 = fast_rcp(dot3(r, r)), t = K * i2, s = 2.0 * t * i2;
        M += t;
        for (int a = 0; a < 3; ++a) gr[a] -= s * r[a];
    });
    if (!(sgn * gr[0] > 0.0)) return clear_record(h);
    const double rel[3] = {plane - xa, y1 - x1, y2 - x2};
    h[0] = 1.0;
    h[4 + ax] = rel[0];
    h[4 + t1] = rel[1];
    h[4 + t2] = rel[2];
    const double qR = (1.0 - M) * fast_rcp(dot3(gr, gr));
    const double delta = A.rs - sgn * (qR * gr[0]);
    if (delta <= 0.0) {
        h[1] = h[2] = h[3] = 0.0;
        return;
    }
    // back in (x, y, z)
    double n[3], ra[3];
    for (int a = 0; a < 3; ++a) {
        n[a] = a == ax ? sgn : 0.0;
        ra[a] = (a == ax ? rel[0] : (a == t1 ? rel[1] : rel[2])) - 0.5 * delta * n[a];
    }
    double ca[3], vrel[3], Fi[3], tq[3], spring[3] = {h[1], h[2], h[3]};
    cross3(A.w, ra, ca);
    for (int a = 0; a < 3; ++a) vrel[a] = A.v[a] + ca[a];
    contact_force(c, delta, n, vrel, dt, spring, Fi);
    cross3(ra, Fi, tq);
    for (int a = 0; a < 3; ++a) h[1 + a] = spring[a];
    emit(Fi, tq);
}

// ---------------------------------------------------------------------------
// Broad phase.  Pair (i, j) is a candidate of a dem_step call of duration T
// when the centres are within the reach radii, R_s and a skin that covers the
// relative displacement of the call, (|v_i| + |v_j|) T + 1/2 (velocities
// change by far less than 1/4 lu per lattice step under the accelerations of
// a stable run), i.e. within bound_i + bound_j with bound = reach + R_s +
// |v| T + 1/4.  A pair outside it cannot come into reach during the call.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool within(const double xi[3], const double* xj, double lim,
                                       const Geom& g)
{
    double d2 = 0.0;
    for (int a = 0; a < 3; ++a) {
        double d = xj[a] - xi[a];
        if (g.per[a]) {
            const double L = g.n[a];
            if (d > 0.5 * L) d -= L;
            else if (d < -0.5 * L) d += L;
        }
        d2 += d * d;
    }
    return sqrt(d2) <= lim;
}

// The contact records of particle i, one per lane of its wave (lanes below
// kPairSlots): each holds its partner's index + 1, 0 when free (zeroed state is
// empty).  Only i's wave touches i's records.
struct Slots {
    int32_t key;
    bool full;  // a candidate found no free record
};

// The candidates among the wave's 64 partners (lane's partner jj, `take` when
// it is one) find their record or claim a free one, in ascending lane order.
__device__ __forceinline__ void claim(Slots& s, bool take, int jj)
{
    const int lane = threadIdx.x & 63;
    uint64_t m = __ballot(take);
    while (m) {
        const int src = __ffsll((unsigned long long)m) - 1;
        m &= m - 1;
        const int32_t k = __builtin_amdgcn_readlane(jj, src) + 1;
        if (__ballot(s.key == k)) continue;  // has its record
        const uint64_t free = __ballot(lane < kPairSlots && s.key == 0);
        if (!free) {
            s.full = true;
            continue;
        }
        if (lane == __ffsll((unsigned long long)free) - 1) s.key = k;
    }
}

// What a call of many particles keeps of each between its launches, one or two
// lines a particle: its constants (half step over the mass and the moments,
// Euler's terms, F^h + relative gravity, T^h, R_s, reach, points), its state at
// two substeps in turn (x, v, q, angular velocity in the body frame), and the
// contact sums of three.
constexpr int kCon = 16, kState = 16, kSums = 8;
struct Ws {
    double* con;
    double* st[2];
    double* sum[3];
};
inline Ws ws_of(double* at, int n)
{
    Ws w;
    w.con = at;
    w.st[0] = at + (int64_t)kCon * n;
    w.st[1] = w.st[0] + (int64_t)kState * n;
    for (int k = 0; k < 3; ++k) w.sum[k] = w.st[1] + (int64_t)kState * n + (int64_t)kSums * n * k;
    return w;
}
static_assert(kDemStateDoubles == kCon + 2 * kState + 3 * kSums, "work space of a particle");

__device__ __forceinline__ void save_state(double* st, const Body& b)
{
    for (int a = 0; a < 3; ++a) {
        st[a] = b.x[a];
        st[3 + a] = b.v[a];
        st[10 + a] = b.wb[a];
    }
    for (int a = 0; a < 4; ++a) st[6 + a] = b.q[a];
}
// The body without its rotation matrix, and its contact view.
__device__ __forceinline__ Body load_state(const double* con, const double* st)
{
    Body b;
    b.hm = con[0];
    for (int a = 0; a < 3; ++a) {
        b.F[a] = con[1 + a];
        b.T[a] = con[4 + a];
        b.hI[a] = con[7 + a];
        b.kI[a] = con[10 + a];
        b.x[a] = st[a];
        b.v[a] = st[3 + a];
        b.wb[a] = st[10 + a];
    }
    for (int a = 0; a < 4; ++a) b.q[a] = st[6 + a];
    const int2 pts = *reinterpret_cast<const int2*>(con + 15);
    b.c0 = pts.x;
    b.c1 = pts.y;
    return b;
}

// Every particle's reach, candidate bound, constants, state and carried contact
// sum; the pair list emptied.
__global__ __launch_bounds__(64) void k_open(PartDev P, const double* FTh, const double* fc, DemP c,
                                             double dt, double T, double* rch, double* bound, Ws w,
                                             uint32_t* count)
{
    const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (p == 0) *count = 0u;
    if (p >= P.n) return;
    const Body b = load_body(P, p, FTh, c, 0.5 * dt);
    double f[6];
    for (int k = 0; k < 6; ++k) f[k] = fc[6 * p + k];
    const double rs = P.rs[p], r = reach(P, p);
    rch[p] = r;
    bound[p] = r + rs + sqrt(dot3(b.v, b.v)) * T + 0.25;
    double* con = w.con + (int64_t)kCon * p;
    con[0] = b.hm;
    for (int a = 0; a < 3; ++a) {
        con[1 + a] = b.F[a];
        con[4 + a] = b.T[a];
        con[7 + a] = b.hI[a];
        con[10 + a] = b.kI[a];
    }
    con[13] = rs;
    con[14] = r;
    *reinterpret_cast<int2*>(con + 15) = make_int2(b.c0, b.c1);
    save_state(w.st[1] + (int64_t)kState * p, b);
    for (int k = 0; k < 6; ++k) {
        w.sum[2][(int64_t)kSums * p + k] = f[k];
        w.sum[0][(int64_t)kSums * p + k] = 0.0;
    }
}

// The cells around c along an axis of nc: lo, lo + 1, ... (n of them), wrapped
// on a periodic axis (each once), clipped at walls.
struct Around {
    int lo, n, nc;
    __device__ __forceinline__ int cell(int k) const
    {
        const int v = lo + k;
        return v < 0 ? v + nc : (v >= nc ? v - nc : v);
    }
};
__device__ __forceinline__ Around around(int c, int nc, int per)
{
    if (per) return nc >= 3 ? Around{c - 1, 3, nc} : Around{0, nc, nc};
    const int lo = max(c - 1, 0);
    return Around{lo, min(c + 1, nc - 1) - lo + 1, nc};
}

// Candidate pairs of one dem_step call, a wave per particle i: the records of
// pairs that are candidates no more are released (zeroed, slot freed), the
// candidates j > i find their record or claim a free one (a particle with more
// candidate partners than slots latches kDeferredSlots; the pair is left out),
// and the pairs with a record are appended as slot << 32 | i << 16 | j, one
// atomic per workgroup of 16 particles (8000 atomics on the one count, one a
// wave, took 90 us).  With GRID the partners are those of the cells around i's
// (every accepted pair lies within H, and cells are at least H wide), else all.
// A wave per particle keeps the walk short and needs no atomic on a record.
__device__ __forceinline__ int grid_cell(const double pos[3], const Geom& g, const int32_t* gdim,
                                         const double* gsize, int c3[3])
{
    for (int a = 0; a < 3; ++a) {
        double x = pos[a];
        if (g.per[a] && !(x >= 0.0 && x <= (double)g.n[a]))
            x -= (double)g.n[a] * floor(x / (double)g.n[a]);  // into [0, n]
        const int k = (int)floor(x * gsize[a]);
        c3[a] = min(max(k, 0), gdim[a] - 1);
    }
    return c3[0] + gdim[0] * (c3[1] + gdim[1] * c3[2]);
}

template <bool GRID>
__global__ __launch_bounds__(1024) void k_pairs(PartDev P, double* hist, int32_t* key,
                                               const double* bound, Geom g, const int32_t* gdim,
                                               const double* gsize, const uint32_t* gstart,
                                               const uint32_t* gitem, uint64_t* list,
                                               uint32_t* count, uint32_t* deferred)
{
    __shared__ uint32_t found[16], base0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int id = (int)(blockIdx.x * 16u) + wave;
    const bool on = id < P.n;  // uniform over the wave
    const int i = on ? id : 0;
    const double xi[3] = {P.pos[3 * i], P.pos[3 * i + 1], P.pos[3 * i + 2]};
    const double bi = bound[i];
    Slots s{0, false};
    if (on && lane < kPairSlots) {
        s.key = key[(int64_t)i * kPairSlots + lane];
        if (s.key > 0 && !within(xi, P.pos + 3 * (s.key - 1), bi + bound[s.key - 1], g)) {
            clear_record(hist + ((int64_t)i * kPairSlots + lane) * kHist);
            s.key = 0;
        }
    }
    if constexpr (GRID) {
        // a lane per cell around i's; their particles flattened over the wave
        int c3[3];
        grid_cell(xi, g, gdim, gsize, c3);
        const Around A0 = around(c3[0], gdim[0], g.per[0]), A1 = around(c3[1], gdim[1], g.per[1]),
                     A2 = around(c3[2], gdim[2], g.per[2]);
        uint32_t first = 0, cnt = 0;
        const int r = lane % 3, t = (lane / 3) % 3, u = lane / 9;
        if (on && r < A0.n && t < A1.n && u < A2.n) {
            const int cell = A0.cell(r) + gdim[0] * (A1.cell(t) + gdim[1] * A2.cell(u));
            first = gstart[cell];
            cnt = gstart[cell + 1] - first;
        }
        uint32_t incl = cnt;
        for (int o = 1; o < 32; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        const uint32_t total = __shfl(incl, 26, 64);  // lanes from 27 on add nothing
        const uint32_t shift = first - (incl - cnt);  // item of flat index k: k + shift
        for (uint32_t k0 = 0; k0 < total; k0 += 64u) {
            const uint32_t k = k0 + (uint32_t)lane;
            int c = 0;  // the cell of flat index k: the number of cells that end at or before it
            for (int step = 16; step > 0; step >>= 1)
                if (__shfl(incl, min(c + step, 27) - 1, 64) <= k && c + step <= 26) c += step;
            const uint32_t sh = __shfl(shift, c, 64);
            const int j = k < total ? (int)gitem[k + sh] : -1;
            claim(s, j > i && within(xi, P.pos + 3 * j, bi + bound[j], g), j);
        }
    } else {
        for (int j0 = on ? i + 1 : P.n; j0 < P.n; j0 += 64) {
            const int j = j0 + lane;
            claim(s, j < P.n && within(xi, P.pos + 3 * j, bi + bound[j], g), j);
        }
    }
    if (on && lane < kPairSlots) key[(int64_t)i * kPairSlots + lane] = s.key;
    if (s.full && lane == 0) atomicOr(deferred, kDeferredSlots);
    const uint64_t m = __ballot(s.key != 0);
    if (lane == 0) found[wave] = (uint32_t)__popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int w = 0; w < 16; ++w) total += found[w];
        base0 = total ? atomicAdd(count, total) : 0u;
    }
    __syncthreads();
    uint32_t base = base0;
    for (int w = 0; w < wave; ++w) base += found[w];
    if (s.key != 0)
        list[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] =
            ((uint64_t)lane << 32) | ((uint64_t)i << 16) | (uint64_t)(s.key - 1);
}

// The cell width and the grid's shape from the particles, by one workgroup of
// 1024; the number of cells on every thread.
__device__ __forceinline__ int grid_shape(const PartDev& P, const double* rch, double T, const Geom& g,
                                          int32_t* gdim, double* gsize, int64_t gcap)
{
    __shared__ double red[2][16];
    __shared__ int ncell;
    double h = 0.0, v = 0.0;
    // (four particles' loads at once; the last particle again beyond the end)
    for (int p0 = (int)threadIdx.x; p0 < P.n; p0 += 4 * (int)blockDim.x) {
        double r[4], s[4], vp[4][3];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int p = min(p0 + k * (int)blockDim.x, P.n - 1);
            r[k] = rch[p];
            s[k] = P.rs[p];
            for (int a = 0; a < 3; ++a) vp[k][a] = P.vel[3 * p + a];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            h = fmax(h, r[k] + s[k]);
            v = fmax(v, dot3(vp[k], vp[k]));
        }
    }
    for (int m = 32; m >= 1; m >>= 1) {
        h = fmax(h, __shfl_xor(h, m, 64));
        v = fmax(v, __shfl_xor(v, m, 64));
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wv] = h;
        red[1][wv] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double hm = 0.0, vm = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            hm = fmax(hm, red[0][w]);
            vm = fmax(vm, red[1][w]);
        }
        // the largest accepted distance, with a margin for rounding
        double H = (2.0 * hm + 2.0 * sqrt(vm) * T + 0.5) * (1.0 + 1e-9) + 1e-9;
        int nc[3];
        int64_t total = 1;
        for (int it = 0; it < 64; ++it) {
            total = 1;
            for (int a = 0; a < 3; ++a) {
                nc[a] = max(1, (int)floor((double)g.n[a] / H));
                total *= nc[a];
            }
            if (total <= gcap) break;
            H *= 1.25;  // more cells than the arrays hold: wider cells
        }
        for (int a = 0; a < 3; ++a) {
            gdim[a] = nc[a];
            gsize[a] = (double)nc[a] / (double)g.n[a];
        }
        gdim[3] = (int32_t)total;
        ncell = (int)total;
    }
    __syncthreads();
    return ncell;
}

// The whole grid by one workgroup, up to kGridBlock particles: shape, counts and
// starts in LDS, and the particles by cell (15 us at 8000; a launch each for
// the shape, the counts, the starts and the scatter, as beyond, 21 and three
// gaps).
constexpr int kGridBlock = 16384, kGridBlockCells = 8192;

__global__ __launch_bounds__(1024) void k_grid_block(PartDev P, const double* rch, double T, Geom g,
                                                     int32_t* gdim, double* gsize, uint32_t* gstart,
                                                     uint32_t* gitem, int64_t gcap)
{
    constexpr int kEach = kGridBlock / 1024, kCells = kGridBlockCells / 1024;
    __shared__ uint32_t count[kGridBlockCells];
    __shared__ uint32_t wsum[16];
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
#pragma unroll
    for (int k = 0; k < kCells; ++k) count[tid + 1024 * k] = 0u;
    const int C = grid_shape(P, rch, T, g, gdim, gsize, min(gcap, (int64_t)kGridBlockCells));
    int cell[kEach];
    uint32_t rank[kEach];
    const int32_t nc[3] = {gdim[0], gdim[1], gdim[2]};
    const double per_node[3] = {gsize[0], gsize[1], gsize[2]};
#pragma unroll
    for (int k0 = 0; k0 < kEach; k0 += 4) {
        if (1024 * k0 >= P.n) continue;  // uniform
        double x[4][3];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            for (int a = 0; a < 3; ++a) x[k][a] = P.pos[3 * min(tid + 1024 * (k0 + k), P.n - 1) + a];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int c3[3];
            cell[k0 + k] = grid_cell(x[k], g, nc, per_node, c3);
            if (tid + 1024 * (k0 + k) < P.n) rank[k0 + k] = atomicAdd(count + cell[k0 + k], 1u);
        }
    }
    __syncthreads();
    // exclusive starts: each thread's kCells cells, then the wave and the block
    uint32_t own[kCells], sum = 0;
#pragma unroll
    for (int k = 0; k < kCells; ++k) {
        own[k] = sum;
        sum += count[kCells * tid + k];
    }
    uint32_t incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t before = incl - sum;
    for (int w = 0; w < wv; ++w) before += wsum[w];
#pragma unroll
    for (int k = 0; k < kCells; ++k) count[kCells * tid + k] = before + own[k];
    __syncthreads();
    for (int i = tid; i < C; i += 1024) gstart[i] = count[i];
    if (tid == 0) gstart[C] = (uint32_t)P.n;
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int p = tid + 1024 * k;
        if (p < P.n) gitem[count[cell[k]] + rank[k]] = (uint32_t)p;
    }
}

// One workgroup: the grid's shape, and the counts cleared.
__global__ __launch_bounds__(1024) void k_grid_setup(PartDev P, const double* rch, double T,
                                                     Geom g, int32_t* gdim,
                                                     double* gsize, uint32_t* gcount, int64_t gcap)
{
    const int ncell = grid_shape(P, rch, T, g, gdim, gsize, gcap);
    for (int i = (int)threadIdx.x; i <= ncell; i += (int)blockDim.x) gcount[i] = 0u;
}

__global__ __launch_bounds__(256) void k_grid_count(PartDev P, Geom g, const int32_t* gdim,
                                                    const double* gsize, uint32_t* gcount)
{
    const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (p >= P.n) return;
    int c3[3];
    atomicAdd(gcount + grid_cell(P.pos + 3 * p, g, gdim, gsize, c3), 1u);
}

// One workgroup: exclusive starts of the cells in place (gcount[C] = n),
// and the scatter cursors.
__global__ __launch_bounds__(1024) void k_grid_scan(const int32_t* gdim, uint32_t* gcount,
                                                    uint32_t* gcursor)
{
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t carry;
    const int C = gdim[3];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry = 0u;
    __syncthreads();
    for (int b0 = 0; b0 < C; b0 += (int)blockDim.x) {
        const int i = b0 + (int)threadIdx.x;
        const uint32_t x = i < C ? gcount[i] : 0u;
        uint32_t incl = x;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (int w = 0; w < wv; ++w) before += wsum[w];
        const uint32_t excl = before + incl - x;
        __syncthreads();  // every thread has read carry and wsum
        if (i < C) {
            gcount[i] = excl;
            gcursor[i] = excl;
        }
        if (threadIdx.x == blockDim.x - 1) carry = excl + x;
        __syncthreads();
    }
    if (threadIdx.x == 0) gcount[C] = carry;
}

__global__ __launch_bounds__(256) void k_grid_scatter(PartDev P, Geom g, const int32_t* gdim,
                                                      const double* gsize, uint32_t* gcursor,
                                                      uint32_t* gitem)
{
    const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (p >= P.n) return;
    int c3[3];
    const uint32_t slot = atomicAdd(gcursor + grid_cell(P.pos + 3 * p, g, gdim, gsize, c3), 1u);
    gitem[slot] = (uint32_t)p;
}

// ---------------------------------------------------------------------------
// Substeps, many particles
// ---------------------------------------------------------------------------

// One substep in one launch: whoever needs a particle's new state forms it from
// the last substep's state and contact sum (the second half kick of that
// substep, but not before the first, then the first half kick, the drift and
// the rotation), so no launch in between has to.  The first workgroups take
// the particles (a thread per particle and wall of a non-periodic axis; the
// first of each particle keeps the new state and clears the next contact sum),
// the others stride over the listed pairs, G lanes each: the positions first,
// and only for a pair within reach the rotations, one body to a lane and
// exchanged between neighbouring lanes.  What bounds it is the one chain of a
// pair or wall in contact (loads, Newton, additions), so a launch less and the
// points in registers tell.  Against a launch for the contacts and one for the
// advance, ten substeps: 1000 metaballs 235 -> 190 us, 125 186 -> 163, 100
// spheres 112 -> 101, 8000 packed ones 156 -> 136; with several waves for every
// SIMD the state that each pair forms again is no longer free: 27 000 spheres
// 302 -> 310.
template <bool FIRST>
__device__ __forceinline__ void advance_centre(Body& b, const double f[6], double dt, const Geom& g)
{
    const Kick k = kick_of(b, f);
    if (!FIRST) kick_v(b, k);
    kick_v(b, k);
    move(b, dt, g);
}
template <bool FIRST>
__device__ __forceinline__ void advance_rotation(Body& b, const double f[6], double dt)
{
    rotmat(b.q, b.R);
    const Kick k = kick_of(b, f);
    if (!FIRST) kick_w<true>(b, k);
    kick_w<false>(b, k);
    to_world(b);
    rotate(b, dt);
}

// (spheres: two waves a SIMD, 8000 of them 142 -> 136 us, 27 000 399 -> 310;
// metaballs: the points take the registers)
template <int G, bool FIRST>
__global__ __launch_bounds__(256, G == 2 ? 2 : 1) void k_substep(PartDev P, Ws w, int s, double* hist, double* hist_w,
                                                 DemP c, double dt, Geom g, const uint64_t* list,
                                                 const uint32_t* count, uint32_t own_blocks, int n_axes,
                                                 int ax0, int ax1, int ax2)
{
    const double *con = w.con, *st = w.st[(s + 1) & 1], *sum = w.sum[(s + 2) % 3];
    double *out = w.st[s & 1], *add_to = w.sum[s % 3], *next = w.sum[(s + 1) % 3];
    auto sums_of = [&](int p, double f[6]) {
        for (int k = 0; k < 6; ++k) f[k] = sum[(int64_t)kSums * p + k];
    };
    auto kin_of = [&](const Body& b, int p) {
        Kin k;
        for (int a = 0; a < 3; ++a) {
            k.x[a] = b.x[a];
            k.v[a] = b.v[a];
            k.w[a] = b.w[a];
        }
        k.rs = con[(int64_t)kCon * p + 13];
        k.reach = con[(int64_t)kCon * p + 14];
        k.K = P.K + b.c0;
        k.n = min(b.c1 - b.c0, kMaxPts);
        return k;
    };
    // world coordinates of control point u of a body with centre x, matrix R
    auto world = [&](const double x[3], const double R[9], int c0, int u, double r[3]) {
        const double* bp = P.body_pts + 3 * (int64_t)(c0 + u);
        for (int a = 0; a < 3; ++a)
            r[a] = x[a] + (R[3 * a] * bp[0] + R[3 * a + 1] * bp[1] + R[3 * a + 2] * bp[2]);
    };
    if (blockIdx.x < own_blocks) {
        const int t = (int)(blockIdx.x * 256u + threadIdx.x);
        const int per = max(2 * n_axes, 1);
        if (t >= P.n * per) return;
        const int i = t / per, k = (t % per) >> 1, side = t & 1;
        const int ax = k == 0 ? ax0 : (k == 1 ? ax1 : ax2);
        Body b = load_state(con + (int64_t)kCon * i, st + (int64_t)kState * i);
        double f[6];
        sums_of(i, f);
        double* h = hist_w + ((int64_t)i * 6 + 2 * ax + side) * kHist;
        const double active = n_axes ? h[0] : 0.0;
        const double lim = con[(int64_t)kCon * i + 13] + con[(int64_t)kCon * i + 14];
        advance_centre<FIRST>(b, f, dt, g);
        const bool keep = t % per == 0, near = n_axes && near_wall(component(b.x, ax), lim, ax, side, g);
        if (keep || near) {
            advance_rotation<FIRST>(b, f, dt);
            if (keep) {
                save_state(out + (int64_t)kState * i, b);
                for (int a = 0; a < 6; ++a) next[(int64_t)kSums * i + a] = 0.0;
            }
            if (near)
                wall_contact<G == 2 ? 1 : 8>(kin_of(b, i),
                             [&](int u, double r[3]) {
                                 double p[3];
                                 world(b.x, b.R, b.c0, u, p);
                                 r[0] = component(p, ax);
                                 r[1] = component(p, (ax + 1) % 3);
                                 r[2] = component(p, (ax + 2) % 3);
                             },
                             h, ax, side, c, dt, g, [&](const double F[3], const double tq[3]) {
                                 for (int a = 0; a < 3; ++a) {
                                     atomicAdd(add_to + (int64_t)kSums * i + a, F[a]);
                                     atomicAdd(add_to + (int64_t)kSums * i + 3 + a, tq[a]);
                                 }
                             });
        }
        if (!near && active != 0.0) clear_record(h);
        return;
    }
    // the wave's contacts, gathered so that consecutive lanes add the twelve
    // numbers of one: the sums of a particle lie in one line, and six lanes'
    // additions to it are one request (a lane that adds its own contact's
    // numbers one after the other makes twelve: 8000 packed spheres 15.2 us a
    // substep's contacts, 8.0 of them without any addition; so 9.4)
    constexpr int kPairs = 64 / G;
    __shared__ double add[4][12 * kPairs];
    __shared__ int who[4][2 * kPairs];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l = lane % G;
    double* wa = add[wave];
    int* ww = who[wave];
    const uint32_t n = *count;
    const uint32_t stride = (gridDim.x - own_blocks) * (256u / G);
    for (uint32_t t0 = (blockIdx.x - own_blocks) * (256u / G) + (uint32_t)(wave * kPairs); t0 < n;
         t0 += stride) {  // uniform over the wave
        const uint32_t t = t0 + (uint32_t)(lane / G);
        int i = 0, j = 0;
        double v[12];
        bool on = false;
        if (t < n) {
            const uint64_t e = list[t];
            i = (int)((e >> 16) & 0xffffu), j = (int)(e & 0xffffu);
            double* h = hist + ((int64_t)i * kPairSlots + (int)(e >> 32)) * kHist;
            const double active = h[0];
            Body A = load_state(con + (int64_t)kCon * i, st + (int64_t)kState * i);
            Body B = load_state(con + (int64_t)kCon * j, st + (int64_t)kState * j);
            double fA[6], fB[6], sh[3];
            sums_of(i, fA);
            sums_of(j, fB);
            Kin kA = kin_of(A, i), kB = kin_of(B, j);
            advance_centre<FIRST>(A, fA, dt, g);
            advance_centre<FIRST>(B, fB, dt, g);
            // (a body without points is an error, reported: it touches nothing)
            if (near_pair(A.x, B.x, kA.reach + kB.reach + kA.rs + kB.rs, g, sh) && kA.n > 0 && kB.n > 0) {
                // odd lanes turn B, even lanes A (the same branch for a group)
                const bool second = l & 1;
                Body M = second ? B : A;
                double f[6];
                for (int k = 0; k < 6; ++k) f[k] = second ? fB[k] : fA[k];
                advance_rotation<FIRST>(M, f, dt);
                for (int k = 0; k < 9; ++k) {
                    const double o = quad_perm<0xB1>(M.R[k]);
                    A.R[k] = second ? o : M.R[k];
                    B.R[k] = second ? M.R[k] : o;
                }
                for (int a = 0; a < 3; ++a) {
                    const double o = quad_perm<0xB1>(M.w[a]);
                    kA.w[a] = second ? o : M.w[a];
                    kB.w[a] = second ? M.w[a] : o;
                    kA.x[a] = A.x[a], kA.v[a] = A.v[a];
                    kB.x[a] = B.x[a], kB.v[a] = B.v[a];
                }
                auto point = [&](int u, double r[3], double& K) __attribute__((always_inline)) {
                    const bool of_b = u >= kA.n;
                    const int at = of_b ? B.c0 + (u - kA.n) : A.c0 + u;
                    const double* bp = P.body_pts + 3 * (int64_t)at;
                    const double b0 = bp[0], b1 = bp[1], b2 = bp[2];
                    K = P.K[at];
                    for (int a = 0; a < 3; ++a) {
                        const double x = of_b ? B.x[a] + sh[a] : A.x[a];
                        r[a] = x + ((of_b ? B.R[3 * a] : A.R[3 * a]) * b0 +
                                    (of_b ? B.R[3 * a + 1] : A.R[3 * a + 1]) * b1 +
                                    (of_b ? B.R[3 * a + 2] : A.R[3 * a + 2]) * b2);
                    }
                };
                pair_item<G>(kA, kB, sh, point, h, c, dt, l,
                             [&](const double F[3], const double ti[3], const double tj[3]) {
                                 on = true;
                                 for (int a = 0; a < 3; ++a) {
                                     v[a] = F[a];
                                     v[3 + a] = ti[a];
                                     v[6 + a] = -F[a];
                                     v[9 + a] = -tj[a];
                                 }
                             });
            } else if (active != 0.0 && l == 0) {
                // out of reach: forget the pair's contact (read one double
                // instead of writing eight when the record is zero already)
                clear_record(h);
            }
        }
        const uint64_t m = __ballot(on);
        if (!m) continue;
        if (on) {
            const int r = __popcll(m & ((1ull << lane) - 1ull));
            for (int k = 0; k < 12; ++k) wa[12 * r + k] = v[k];
            ww[2 * r] = i;
            ww[2 * r + 1] = j;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int total = 12 * __popcll(m);
        for (int u = lane; u < total; u += 64) {
            const int q = u / 6;
            atomicAdd(add_to + (int64_t)kSums * ww[q] + (u - 6 * q), wa[u]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// The last substep's second half kick, and the caller's arrays.
__global__ __launch_bounds__(64) void k_close(PartDev P, Ws w, int n_sub, double* fc)
{
    const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (p >= P.n) return;
    Body b = load_state(w.con + (int64_t)kCon * p, w.st[(n_sub + 1) & 1] + (int64_t)kState * p);
    const double* sum = w.sum[(n_sub + 2) % 3] + (int64_t)kSums * p;
    double f[6];
    for (int k = 0; k < 6; ++k) f[k] = sum[k];
    rotmat(b.q, b.R);
    const Kick k = kick_of(b, f);
    kick_v(b, k);
    kick_w<true>(b, k);
    to_world(b);
    for (int a = 0; a < 6; ++a) fc[6 * p + a] = f[a];
    store_body(P, p, b, true);
    place_points<4>(b, b.c0, b.c1, P.body_pts, P.wpts);
}

// ---------------------------------------------------------------------------
// A whole dem_step call in one workgroup
// ---------------------------------------------------------------------------
constexpr int kBlockThreads = 512;
// Most control points of such a call (they and the records fill the 64 KB of
// LDS a workgroup may declare; bodies with more take the launches).
constexpr int kBlockPoints = 384;
// Lanes that share a pair: the Newton chain of one lane over the 4 to 12
// points of two metaballs is what a substep waits for (32-43 us at 1000
// metaballs, about 16 with four lanes).
constexpr int kPairLanes = 4;

// Groups of pair lanes: every wave but the first.
constexpr int kPairGroups = (kBlockThreads - 64) / kPairLanes;

__global__ __launch_bounds__(kBlockThreads) void k_dem_block(PartDev P, double* hist, double* hist_w,
                                                             int32_t* key, const double* FTh,
                                                             double* fc, uint64_t* list, DemP c,
                                                             int n_sub, double dt, Geom g,
                                                             uint32_t* deferred)
{
    __shared__ double pos[3 * kBlockParticles], vel[3 * kBlockParticles], om[3 * kBlockParticles];
    __shared__ double sum[6 * kBlockParticles], rs[kBlockParticles], rch[kBlockParticles];
    __shared__ double bound[kBlockParticles];
    __shared__ double body[3 * kBlockPoints], world[3 * kBlockPoints], K[kBlockPoints];
    __shared__ double wall[6 * kBlockParticles * kHist];  // the particles' wall records
    __shared__ double rec[kPairGroups * kHist];           // the groups' first pairs' records
    __shared__ int32_t off[kBlockParticles + 1];
    __shared__ uint16_t items[6 * kBlockParticles];       // the first wave's wall contacts
    __shared__ uint32_t npairs;
    const int tid = (int)threadIdx.x, lane = tid & 63, n = P.n;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto kin = [&](int i) {
        Kin k;
        for (int a = 0; a < 3; ++a) {
            k.x[a] = pos[3 * i + a];
            k.v[a] = vel[3 * i + a];
            k.w[a] = om[3 * i + a];
        }
        k.rs = rs[i];
        k.reach = rch[i];
        k.K = K + off[i];
        k.n = min(off[i + 1] - off[i], kMaxPts);
        return k;
    };
    auto points = [&](int i, int ax) {
        const double *p = world + 3 * off[i], *p0 = p + ax, *p1 = p + (ax + 1) % 3, *p2 = p + (ax + 2) % 3;
        return [=](int u, double r[3]) {
            r[0] = p0[3 * u], r[1] = p1[3 * u], r[2] = p2[3 * u];
        };
    };
    const int p0 = P.off[0], np = min(P.off[n] - p0, kBlockPoints);
    if (tid == 0) {
        npairs = 0u;
        if (P.off[n] - p0 > kBlockPoints) atomicOr(deferred, kDeferredPoints);
    }
    if (tid <= n) off[tid] = min(P.off[tid] - p0, kBlockPoints);
    for (int i = tid; i < np; i += kBlockThreads) K[i] = P.K[p0 + i];
    for (int i = tid; i < 3 * np; i += kBlockThreads) body[i] = P.body_pts[3 * (int64_t)p0 + i];
    for (int i = tid; i < 6 * n * kHist; i += kBlockThreads) wall[i] = hist_w[i];
    if (tid < n) {
        double v2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            pos[3 * tid + a] = P.pos[3 * tid + a];
            const double v = P.vel[3 * tid + a];
            v2 += v * v;
        }
        rs[tid] = P.rs[tid];
        rch[tid] = reach(P, tid);
        bound[tid] = rch[tid] + rs[tid] + sqrt(v2) * ((double)n_sub * dt) + 0.25;
    }
    __syncthreads();
    // candidate pairs, as k_pairs
    for (int i = wave; i < n; i += kBlockThreads / 64) {
        const double xi[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
        Slots s{0, false};
        if (lane < kPairSlots) {
            s.key = key[i * kPairSlots + lane];
            const int j = s.key - 1;
            if (s.key > 0 && !within(xi, pos + 3 * j, bound[i] + bound[j], g)) {
                clear_record(hist + ((int64_t)i * kPairSlots + lane) * kHist);
                s.key = 0;
            }
        }
        for (int j0 = i + 1; j0 < n; j0 += 64) {
            const int j = j0 + lane;
            claim(s, j < n && within(xi, pos + 3 * min(j, n - 1), bound[i] + bound[min(j, n - 1)], g), j);
        }
        if (lane < kPairSlots) key[i * kPairSlots + lane] = s.key;
        if (s.full && lane == 0) atomicOr(deferred, kDeferredSlots);
        const uint64_t m = __ballot(s.key != 0);
        uint32_t base = 0;
        if (lane == 0 && m) base = atomicAdd(&npairs, (uint32_t)__popcll(m));
        base = __shfl(base, 0, 64);
        if (s.key != 0)
            list[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] =
                ((uint64_t)lane << 32) | ((uint64_t)i << 16) | (uint64_t)(s.key - 1);
    }
    __syncthreads();
    // the first wave moves the particles and takes their wall contacts, the
    // others take the pairs (the same barriers on both sides: two a substep,
    // none if there are no pairs)
    const bool pairs = __builtin_amdgcn_readfirstlane((int)npairs) > 0;
    if (wave == 0) {
        const bool on = tid < n;
        uint32_t live = 0;  // wall records that are not zero
        double lim = 0.0;   // how near a wall must be to be touched
        Body b{};
        double f[6] = {0, 0, 0, 0, 0, 0};
        if (on) {
            b = load_body(P, tid, FTh, c, 0.5 * dt);
            for (int k = 0; k < 6; ++k) f[k] = fc[6 * tid + k];
            const Kick k0 = kick_of(b, f);
            kick_v(b, k0);
            kick_w<false>(b, k0);
            for (int k = 0; k < 6; ++k) live |= wall[(6 * tid + k) * kHist] != 0.0 ? 1u << k : 0u;
            lim = rch[tid] + rs[tid];
        }
        for (int sub = 0; sub < n_sub; ++sub) {
            if (on) {
                to_world(b);
                move(b, dt, g);
                rotate(b, dt);
                place_points<1>(b, off[tid], off[tid + 1], body, world);
                for (int a = 0; a < 3; ++a) {
                    pos[3 * tid + a] = b.x[a];
                    vel[3 * tid + a] = b.v[a];
                    om[3 * tid + a] = b.w[a];
                }
                for (int k = 0; k < 6; ++k) sum[6 * tid + k] = 0.0;
            }
            if (pairs) __syncthreads();
            uint32_t near = 0;  // as near_wall
            if (on)
                for (int ax = 0; ax < 3; ++ax)
                    if (!g.per[ax]) {
                        if (!(b.x[ax] + 0.5 > lim)) near |= 1u << (2 * ax);
                        if (!((double)g.n[ax] - 0.5 - b.x[ax] > lim)) near |= 2u << (2 * ax);
                    }
            const uint32_t todo = near | live;
            live = near;
            if (__any(todo != 0u)) {
                // the wave's bodies and walls listed, one to a lane: a body in a
                // corner waits for one contact, not for three one after the other
                int total = 0;
                for (int k = 0; k < 6; ++k) {
                    const bool is = (todo >> k) & 1u;
                    const uint64_t m = __ballot(is);
                    if (is)
                        items[total + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                            (uint16_t)(tid << 4 | k << 1 | (int)((near >> k) & 1u));
                    total += __popcll(m);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                for (int t = tid; t < total; t += 64) {
                    const int i = items[t] >> 4, k = (items[t] >> 1) & 7;
                    double* h = wall + (6 * i + k) * kHist;
                    if (items[t] & 1)
                        wall_contact<0>(kin(i), points(i, k >> 1), h, k >> 1, k & 1, c, dt, g,
                                     [&](const double F[3], const double t[3]) {
                                         for (int a = 0; a < 3; ++a) {
                                             atomicAdd(sum + 6 * i + a, F[a]);
                                             atomicAdd(sum + 6 * i + 3 + a, t[a]);
                                         }
                                     });
                    else
                        clear_record(h);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            if (pairs) __syncthreads();
            if (on) {
                for (int k = 0; k < 6; ++k) f[k] = sum[6 * tid + k];
                const Kick k = kick_of(b, f);
                kick_v(b, k);
                kick_w<true>(b, k);
                if (sub + 1 < n_sub) {
                    kick_v(b, k);
                    kick_w<false>(b, k);
                }
            }
        }
        if (on) {
            to_world(b);
            store_body(P, tid, b, true);
            for (int k = 0; k < 6; ++k) fc[6 * tid + k] = f[k];
        }
    } else if (pairs) {
        const int group = kPairGroups - 1 - (tid - 64) / kPairLanes, l = tid % kPairLanes;
        auto adder = [&](int i, int j) {
            return [&, i, j](const double F[3], const double ti[3], const double tj[3]) {
                for (int a = 0; a < 3; ++a) {
                    atomicAdd(sum + 6 * i + a, F[a]);
                    atomicAdd(sum + 6 * j + a, -F[a]);
                    atomicAdd(sum + 6 * i + 3 + a, ti[a]);
                    atomicAdd(sum + 6 * j + 3 + a, -tj[a]);
                }
            };
        };
        auto contact = [&](int i, int j, double* h) {
            const Kin a = kin(i), b = kin(j);
            double sh[3];
            auto point = [&](int u, double r[3], double& Ku) __attribute__((always_inline)) {
                const bool of_b = u >= a.n;
                const int at = of_b ? off[j] + (u - a.n) : off[i] + u;
                for (int k = 0; k < 3; ++k) r[k] = world[3 * at + k] + (of_b ? sh[k] : 0.0);
                Ku = K[at];
            };
            if (near_pair(a.x, b.x, a.reach + b.reach + a.rs + b.rs, g, sh) && a.n > 0 && b.n > 0)
                pair_item<kPairLanes>(a, b, sh, point, h, c, dt, l, adder(i, j));
            else if (l == 0 && h[0] != 0.0)
                clear_record(h);  // out of reach: forget the pair's contact
        };
        const int total = (int)npairs;
        const bool mine = group < total;
        const uint64_t e0 = mine ? list[group] : 0;
        const int i0 = (int)((e0 >> 16) & 0xffffu), j0 = (int)(e0 & 0xffffu);
        double* h0 = rec + group * kHist;
        double* g0 = hist + ((int64_t)i0 * kPairSlots + (int)(e0 >> 32)) * kHist;
        if (mine)
            for (int k = l; k < kHist; k += kPairLanes) h0[k] = g0[k];
        for (int sub = 0; sub < n_sub; ++sub) {
            __syncthreads();
            if (mine) contact(i0, j0, h0);
            for (int t = group + kPairGroups; t < total; t += kPairGroups) {
                const uint64_t e = list[t];
                const int i = (int)((e >> 16) & 0xffffu), j = (int)(e & 0xffffu);
                contact(i, j, hist + ((int64_t)i * kPairSlots + (int)(e >> 32)) * kHist);
            }
            __syncthreads();
        }
        if (mine)
            for (int k = l; k < kHist; k += kPairLanes) g0[k] = h0[k];
    }
    __syncthreads();
    if (n_sub > 0)
        for (int i = tid; i < 3 * np; i += kBlockThreads) P.wpts[3 * (int64_t)p0 + i] = world[i];
    for (int i = tid; i < 6 * n * kHist; i += kBlockThreads) hist_w[i] = wall[i];
}

}  // namespace

hipError_t launch_dem(lbm_ctx* ctx, const PartDev& P, int n_sub, double dt, const dem_params& prm,
                      const DemScratch& ws)
{
    const int np = P.n;
    if (np == 0) return hipSuccess;
    DemP c;
    c.kn = prm.kn;
    c.etan = prm.eta_n;
    c.kt = prm.kt;
    c.etat = prm.eta_t;
    c.mu = prm.mu_s;
    c.ctol = prm.ctol;
    c.ntol2 = step_tol2(prm.newton_tol);
    c.niter = prm.newton_iter;
    for (int a = 0; a < 3; ++a) c.g[a] = prm.gravity[a];
    c.rhof = prm.rho_f;
    uint32_t* deferred = ctx->ctr + kCtrDeferred;
    const Geom& g = ctx->geom;
    // lbm_config.n_ctrl picks the path; a context that does not state it (fewer
    // points than particles) takes the launches, which go by ctrl_off alone
    const int n_ctrl = ctx->cfg.n_ctrl;
    if (np <= kBlockParticles && n_ctrl >= np && n_ctrl <= kBlockPoints) {
        hipLaunchKernelGGL(k_dem_block, dim3(1), dim3(kBlockThreads), 0, ctx->stream, P, ctx->hist_pp,
                           ctx->hist_pw, ctx->hist_key, ctx->FT, ctx->fc, ws.pairs, c, n_sub, dt, g,
                           deferred);
        return hipGetLastError();
    }
    const uint32_t bp = (uint32_t)(np + 63) / 64, bw = (uint32_t)(np + 15) / 16;
    const double T = (double)n_sub * dt;
    const Ws w = ws_of(ws.state, np);
    hipLaunchKernelGGL(k_open, dim3(bp), dim3(64), 0, ctx->stream, P, ctx->FT, ctx->fc, c, dt, T, ws.reach,
                       ws.bound, w, ws.count);
    if (ws.gcount && np >= kGridMinParticles) {
        if (np <= kGridBlock) {
            hipLaunchKernelGGL(k_grid_block, dim3(1), dim3(1024), 0, ctx->stream, P, ws.reach, T, g,
                               ws.gdim, ws.gsize, ws.gcount, ws.gitem, ws.gcap);
        } else {
            const uint32_t bn = (uint32_t)((np + 255) / 256);
            hipLaunchKernelGGL(k_grid_setup, dim3(1), dim3(1024), 0, ctx->stream, P, ws.reach, T, g,
                               ws.gdim, ws.gsize, ws.gcount, ws.gcap);
            hipLaunchKernelGGL(k_grid_count, dim3(bn), dim3(256), 0, ctx->stream, P, g, ws.gdim,
                               ws.gsize, ws.gcount);
            hipLaunchKernelGGL(k_grid_scan, dim3(1), dim3(1024), 0, ctx->stream, ws.gdim, ws.gcount,
                               ws.gcursor);
            hipLaunchKernelGGL(k_grid_scatter, dim3(bn), dim3(256), 0, ctx->stream, P, g, ws.gdim,
                               ws.gsize, ws.gcursor, ws.gitem);
        }
        hipLaunchKernelGGL(k_pairs<true>, dim3(bw), dim3(1024), 0, ctx->stream, P, ctx->hist_pp,
                           ctx->hist_key, ws.bound, g, ws.gdim, ws.gsize, ws.gcount, ws.gitem,
                           ws.pairs, ws.count, deferred);
    } else {
        hipLaunchKernelGGL(k_pairs<false>, dim3(bw), dim3(1024), 0, ctx->stream, P, ctx->hist_pp,
                           ctx->hist_key, ws.bound, g, nullptr, nullptr, nullptr, nullptr, ws.pairs,
                           ws.count, deferred);
    }
    int axes[3] = {0, 0, 0}, n_axes = 0;
    for (int a = 0; a < 3; ++a)
        if (!g.per[a]) axes[n_axes++] = a;
    const uint32_t wb = (uint32_t)(((int64_t)np * std::max(2 * n_axes, 1) + 255) / 256);
    // lanes for eight pairs a particle (more stride over the list)
    // (spheres: two control points a pair)
    const bool spheres = n_ctrl == np;
    const int lanes = spheres ? 2 : kPairLanes;
    const uint32_t pb = (uint32_t)std::min<int64_t>(((int64_t)np * 8 * lanes + 255) / 256, 2048);
    for (int s = 0; s < n_sub; ++s) {
        const auto substep = spheres ? (s ? k_substep<2, false> : k_substep<2, true>)
                                     : (s ? k_substep<kPairLanes, false> : k_substep<kPairLanes, true>);
        hipLaunchKernelGGL(substep, dim3(wb + pb), dim3(256), 0, ctx->stream, P, w, s, ctx->hist_pp,
                           ctx->hist_pw, c, dt, g, ws.pairs, ws.count, wb, n_axes, axes[0], axes[1],
                           axes[2]);
    }
    hipLaunchKernelGGL(k_close, dim3(bp), dim3(64), 0, ctx->stream, P, w, n_sub, ctx->fc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The allocation-free work space of dem_step_noalloc: one static array per
// device (module-scope device memory, loaded with the code object), laid out
// as the pair count (first 512 bytes), the reach and the candidate bound of up
// to kNoAllocParticles particles, then up to kNoAllocParticles * kPairSlots pair
// entries and the particles' states and sums.  Host code never uses the array's
// name as an address: the device address is looked up once per device and kept.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t kNoAllocHead = 64;  // 8-byte words before the reach
constexpr size_t kNoAllocWords =
    kNoAllocHead + (2 + kPairSlots + kDemStateDoubles) * (size_t)kNoAllocParticles;
__device__ __align__(256) uint64_t scratch[kNoAllocWords];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint64_t* g_scratch_dev[kMaxDevices] = {};
}  // namespace

hipError_t dem_noalloc_setup()
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_dev[dev]) return hipSuccess;
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_dev[dev] = static_cast<uint64_t*>(ptr);
    return hipSuccess;
}

bool dem_noalloc_scratch(int dev, DemScratch* out)
{
    if (dev < 0 || dev >= kMaxDevices) return false;
    uint64_t* base;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        base = g_scratch_dev[dev];
    }
    if (!base) return false;
    out->count = reinterpret_cast<uint32_t*>(base);
    out->reach = reinterpret_cast<double*>(base + kNoAllocHead);
    out->bound = out->reach + kNoAllocParticles;
    out->pairs = base + kNoAllocHead + 2 * kNoAllocParticles;
    out->state = reinterpret_cast<double*>(out->pairs + kNoAllocParticles * kPairSlots);
    return true;
}

}  // namespace mdlbm
