// FP64 geometry kernels of libmdlbm for gfx950: node classification against
// the metaball bodies {M_p >= c0_p} (Eq. metaball), link records with the
// wall fraction q of Eq. (appq), and detection of nodes to refill (Sec. 2.3.3).
//
// These decisions must be bit-identical to any other IEEE implementation of
// the same convention, so this file is built with -ffp-contract=off and every
// metaball value is evaluated as
//     r2 = (dx*dx + dy*dy) + dz*dz,   M = ((0 + K_0/r2_0) + K_1/r2_1) + ...
// in IEEE double with correctly rounded division.
//
// Work is organised per particle: a particle's nodes lie in a ball of radius
// R <= h - 1 about x_p (a rigorous bound from the metaball weights), inside the
// box of (2h+1)^3 nodes around floor(x_p).  One workgroup takes one z plane
// of the box.  Coordinates are unwrapped, so on a periodic axis they are exactly
// the node's image nearest x_p (the box is narrower than half the period).
#pragma clang fp contract(off)

#include <algorithm>

#include "lbm_internal.h"
#include "lbm_stencil.h"
#include "lbm_kernels.h"

namespace mdlbm {
namespace {

constexpr int kMaxCtrl = 64;

// Control points (x, y, z, K) of particle p staged in LDS.
__device__ __forceinline__ int stage_ctrl(const PartDev& P, int p, double* sp)
{
    const int a = P.off[p], n = min(P.off[p + 1] - a, kMaxCtrl);
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        sp[4 * i + 0] = P.wpts[3 * (int64_t)(a + i) + 0];
        sp[4 * i + 1] = P.wpts[3 * (int64_t)(a + i) + 1];
        sp[4 * i + 2] = P.wpts[3 * (int64_t)(a + i) + 2];
        sp[4 * i + 3] = P.K[a + i];
    }
    __syncthreads();
    return n;
}

// (four quotients in flight; the sum takes them in order)
__device__ __forceinline__ double metaball(const double* sp, int n, double X, double Y, double Z)
{
    auto term = [&](int i) {
        const double dx = X - sp[4 * i + 0];
        const double dy = Y - sp[4 * i + 1];
        const double dz = Z - sp[4 * i + 2];
        const double r2 = (dx * dx + dy * dy) + dz * dz;
        return sp[4 * i + 3] / r2;
    };
    double M = 0.0;
    int i = 0;
    for (; i + 4 <= n; i += 4) {
        const double a = term(i), b = term(i + 1), c = term(i + 2), d = term(i + 3);
        M = (((M + a) + b) + c) + d;
    }
    for (; i < n; ++i) M = M + term(i);
    return M;
}

// The same, point by point from global memory, where it is rarely needed.
__device__ __forceinline__ double metaball_rare(const double* w, const double* K, int n, double X,
                                                double Y, double Z)
{
    double M = 0.0;
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const double dx = X - w[3 * i + 0];
        const double dy = Y - w[3 * i + 1];
        const double dz = Z - w[3 * i + 2];
        const double r2 = (dx * dx + dy * dy) + dz * dz;
        M = M + K[i] / r2;
    }
    return M;
}

__device__ __forceinline__ uint32_t node_idx(const int c[3], const Geom& g)
{
    return (uint32_t)c[0] + (uint32_t)g.n[0] * ((uint32_t)c[1] + (uint32_t)g.n[1] * (uint32_t)c[2]);
}

// An unwrapped coordinate beyond the lattice, wrapped onto a periodic axis.
__device__ __forceinline__ int wrap_axis(int v, int n)
{
    v += v < 0 ? n : -n;
    return v >= 0 && v < n ? v : ((v % n) + n) % n;
}

// Wrap unwrapped coordinates onto the lattice; false beyond a wall.
__device__ __forceinline__ bool wrap_cell(const int ii[3], const Geom& g, int c[3])
{
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int v = ii[a];
        if (v < 0 || v >= g.n[a]) {
            if (g.per[a])
                v = wrap_axis(v, g.n[a]);
            else
                ok = false;
        }
        c[a] = v;
    }
    return ok;
}

// Visit the nodes of z plane `plane` of the box in the square around
// the ball (x_p, R)'s circle there, 32 x 8 nodes a workgroup and two such tiles
// at once: fn(node, on) for each tile, called by every lane of a wave together
// (on: the node exists and lies in the ball).  A wave per row with the row's
// FP64 ends first, one row after the other, was a longer chain.
template <class Fn>
__device__ __forceinline__ void walk_ball_plane(const double* ball, int h, int plane, const Geom& g,
                                                Fn&& fn)
{
    const double bx = ball[0], by = ball[1], bz = ball[2], R = ball[3];
    const int zi = (int)floor(bz) - h + plane;
    const double dz = (double)zi - bz;
    const double r2z = R * R - dz * dz;
    if (r2z < 0.0) return;  // uniform over the block
    const double ry = sqrt(r2z);
    const int ylo = (int)ceil(by - ry), yhi = (int)floor(by + ry);
    const int xlo = (int)ceil(bx - ry), xhi = (int)floor(bx + ry);
    for (int y0 = ylo + (int)(threadIdx.x >> 5); y0 - (int)(threadIdx.x >> 5) <= yhi; y0 += 16)
        for (int x = xlo + (int)(threadIdx.x & 31); x - (int)(threadIdx.x & 31) <= xhi; x += 32) {
            uint32_t node[2];
            bool on[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int ii[3] = {x, y0 + 8 * k, zi};
                const double dx = (double)ii[0] - bx, dy = (double)ii[1] - by;
                int c[3];
                on[k] = dx * dx + dy * dy <= r2z && wrap_cell(ii, g, c);
                node[k] = on[k] ? node_idx(c, g) : 0u;
            }
            fn(node, on);
        }
}

// Wave-wide exclusive offset of `count` within a reservation of `total`
// slots taken from *cursor by lane 63.  Every lane of the wave must call it.
__device__ __forceinline__ uint32_t wave_reserve(uint32_t count, uint32_t* cursor)
{
    const int lane = threadIdx.x & 63;
    uint32_t incl = count;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    const uint32_t total = __shfl(incl, 63, 64);
    uint32_t base = 0;
    if (lane == 63 && total != 0) base = atomicAdd(cursor, total);
    base = __shfl(base, 63, 64);
    return base + incl - count;
}

// Block (bx, by) of a gx x gy work grid launched as the first `blocks`, a
// multiple of 8, workgroups of a 1D grid.  The hardware hands workgroup b to XCD b % 8; mapping XCD k to
// the k-th eighth of the work keeps all blocks of a particle (by) on one XCD,
// so the owner rows its candidates share are fetched into one L2.  False for
// the padding workgroups.
__device__ __forceinline__ bool xcd_tile(uint32_t blocks, uint32_t gx, uint32_t gy, uint32_t& bx,
                                         uint32_t& by)
{
    const uint32_t per = blocks >> 3;
    const uint32_t logical = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if (logical >= gx * gy) return false;
    bx = logical % gx;
    by = logical / gx;
    return true;
}

// ---------------------------------------------------------------------------

// Box origin and body radius of every particle, and input checks.  At
// distance d > max|x_i - x_p| from the centre, M <= B(d) = sum K_i/(d - |x_i - x_p|)^2,
// which decreases in d, so the body lies within the root R of B(R) = c0.  The
// box must hold the ball of radius h - 1 (B(h-1) < c0); R itself lets the
// kernels skip box cells that cannot be solid.
__device__ __forceinline__ double wave_sum_d(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// v of lane j (the same j on every lane).
__device__ __forceinline__ float lane_of(float v, int j)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}

// Box and radius of particle p by one wave, a lane per control point (n <= 64).
__device__ __forceinline__ void box_of(const PartDev& P, int p, int h, double* ball, uint32_t* err,
                                       const Geom& g, const double* ball_prev, double* quat_prev,
                                       uint32_t* inc_bad)
{
    const int lane = threadIdx.x;
    uint32_t bad = 0;
    double xp[3];
    for (int a = 0; a < 3; ++a) {
        xp[a] = P.pos[3 * p + a];
        if (!(xp[a] == xp[a]) || (g.per[a] && !(xp[a] >= 0.0 && xp[a] < (double)g.n[a]))) bad |= 1u;
    }
    const int a0 = P.off[p], n = P.off[p + 1] - a0;
    if (n < 1 || n > kMaxCtrl) bad |= 8u;
    const double c0 = P.c0[p];
    if (!(c0 > 0.0)) bad |= 2u;
    // this lane's control point: distance to the centre and weight
    double ri = 0.0, Ki = 0.0;
    if (lane < min(n, kMaxCtrl)) {
        Ki = P.K[a0 + lane];
        if (!(Ki > 0.0)) bad |= 2u;
        double r2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double d = P.wpts[3 * (int64_t)(a0 + lane) + a] - xp[a];
            r2 += d * d;
        }
        ri = sqrt(r2);
    }
    double rmax = ri;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) rmax = fmax(rmax, __shfl_xor(rmax, o, 64));
    auto bound = [&](double d) {
        const double t = d - ri;
        return wave_sum_d(Ki > 0.0 ? Ki / (t * t) : 0.0);
    };
    const double lim = (double)(h - 1);
    double R = lim;
    if (!(lim > rmax) || !(bound(lim) < c0)) {
        bad |= 4u;
    } else {
        // B decreases beyond rmax.  A 64-way search in FP32 closes in on its
        // root: the lanes test 64 points of (lo, hi], each summing B over the
        // control points itself, and the first below c0 becomes hi; five
        // rounds reach FP32's spacing.  The FP64 sum then has to pass at the
        // radius found, widened past the FP32 sum's error; else the box's own
        // bound, tested above, stands.
        const int nn = min(n, kMaxCtrl);
        const float rf = (float)ri, Kf = (float)Ki, cf = (float)c0 * 0.9999f;
        float lo = (float)rmax, hi = (float)lim;
        for (int round = 0; round < 5; ++round) {
            const float step = (hi - lo) * (1.0f / 64.0f);
            const float d = lane == 63 ? hi : lo + step * (float)(lane + 1);
            float B = 0.0f;
            for (int j = 0; j < nn; ++j) {
                const float t = d - lane_of(rf, j);
                B += lane_of(Kf, j) * __builtin_amdgcn_rcpf(t * t);
            }
            const uint64_t pass = __ballot(B < cf);
            if (!pass) break;  // uniform; hi keeps its bound
            const int first = __ffsll((unsigned long long)pass) - 1;
            const float nh = lane_of(d, first), nl = lane_of(d, first > 0 ? first - 1 : 0);
            hi = nh;
            if (first > 0) lo = nl;
        }
        const double near = (double)hi * (1.0 + 1e-5) + 1e-5;
        if (near > rmax && near < lim && bound(near) < c0) R = near;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) bad |= __shfl_xor(bad, o, 64);
    if (lane == 0) {
        ball[4 * p + 0] = xp[0];
        ball[4 * p + 1] = xp[1];
        ball[4 * p + 2] = xp[2];
        ball[4 * p + 3] = R + 1e-6;
        if (bad) atomicOr(err, bad);
        if (inc_bad) {
            // how far a body point within R + 2 of the centre moved since the
            // previous classification: the centre's displacement plus
            // (R + 2) times the rotation angle between the two orientations
            double d2 = 0.0;
            for (int a = 0; a < 3; ++a) {
                double d = xp[a] - ball_prev[4 * p + a];
                if (g.per[a]) {
                    if (d > 0.5 * g.n[a]) d -= g.n[a];
                    else if (d < -0.5 * g.n[a]) d += g.n[a];
                }
                d2 += d * d;
            }
            const double* q = P.quat + 4 * p;
            double* qp = quat_prev + 4 * p;
            const double dot = fabs(q[0] * qp[0] + q[1] * qp[1] + q[2] * qp[2] + q[3] * qp[3]);
            const double ang = 2.0 * acos(fmin(1.0, dot));
            const double D = sqrt(d2) + (R + 2.0) * ang;
            // a solid node off the candidate list has M >= c0 wherever within
            // the lattice's largest |e| of it; a node moved by less than that
            // stays solid
            if (!(D < 0.9 * (double)kMaxSpeedUp - 1e-3)) atomicOr(inc_bad, 1u);
            for (int a = 0; a < 4; ++a) qp[a] = q[a];
        }
    }
}

// The first kernel of a classification, a column of workgroups per particle:
// the first of a column resets the particle's candidate count (that of the
// previous classification is kept for its lists) and finds its box, the others,
// given a plane to clear, clear a z plane of its ball of two classifications ago
// (also where the check of the boxes fails: that plane is not in use, and the
// next attempt clears it again).  The link counts are those that lbm_step runs
// by until the check has passed, so k_mark resets them.  One launch for the chain
// of three that a small run waited 12 us for.
__global__ __launch_bounds__(256) void k_begin(PartDev P, int h, double* ball, uint32_t* err, Geom g,
                                               const double* ball_prev, double* quat_prev,
                                               uint32_t* inc_bad, uint32_t* cand_cursor,
                                               uint32_t* cand_prev_count, uint32_t* own,
                                               const double* ball_clear)
{
    const int p = blockIdx.y;
    if (blockIdx.x > 0) {
        walk_ball_plane(ball_clear + 4 * p, h, (int)blockIdx.x - 1, g,
                        [&](const uint32_t* node, const bool* on) {
#pragma unroll
                            for (int k = 0; k < 2; ++k)
                                if (on[k]) own[node[k]] = kFluid;
                        });
        return;
    }
    if (threadIdx.x >= 64) return;
    if (threadIdx.x == 0) {
        const int64_t at = (int64_t)p * kCursorPad;
        if (cand_prev_count) cand_prev_count[p] = cand_cursor[at];
        cand_cursor[at] = 0;
    }
    box_of(P, p, h, ball, err, g, ball_prev, quat_prev, inc_bad);
}

// Node owners: the lowest particle index with M_p >= c0_p.
//
// Which nodes are visited.  If every control point lies farther than
// rho = sqrt(sum_i K_i / c0) from a node, M_p < c0 there, so p's body lies
// in the union of the balls (x_i, rho); it also lies in the ball (x_p, R) of
// k_begin.  One workgroup takes one z plane of p's box: for every row y of the
// plane it takes the x range of the union's hull on that row intersected with
// the centre ball, cuts it into segments of 8 nodes, lists them in LDS (a
// prefix sum over the rows places them) and hands them to its lanes, so a lane
// finds its node by one LDS read and few lanes idle at row ends.  The ranges
// are FP32 and widened by more than their error: with coordinates relative to
// o off by at most (3h + 1) 2^-24, squares and their sums are off by less than
// (2h + 4)^2 2^-21 and ends by less than (2h + 4) 2^-21; a node visited in vain
// is decided as not solid.
//
// How a node is decided.  The FP64 sum alone decides, bit for bit; an FP32
// estimate settles the nodes far from the decision.  The estimate works in
// coordinates relative to o = floor(x_p) (node offsets are exact integers,
// control points are rounded once, |x_i - o| <= R + 1 < h), so each
// coordinate difference is off by at most delta = (2h + 4) 2^-24.  At a
// distance r >= g = 0.0085 (2h + 4) from every control point the relative
// error of r^2 is below 2.83 delta / r + 3 2^-24 <= 2e-5, of a term
// K_i / r^2 (hardware reciprocal, 1 ulp) below 2.2e-5 and of the sum below
// 2.6e-5 for up to 64 points.  So outside a relative band of 1e-4 around c0
// the estimate decides what the FP64 sum decides; nodes in the band, or
// within g of a control point, or of a box with h > 127, take the FP64 sum.
//
// Candidates for links.  M_p at any lattice neighbour (|e| <= E: sqrt 2 for
// D3Q19, sqrt 3 for D3Q15) is at least sum_i K_i / (r_i + E)^2.  A solid
// node where the FP32 value of this bound (E rounded up) clears c0 by the
// same margin (its relative error stays below 3.5e-5 for h <= 127: the
// r_i + E terms are never small) has M_p >= c0 at every neighbour, hence no
// link of any kind, and is left off p's candidate list; and it is solid.  Every
// other solid node of p goes on the list.  The bound and the estimate take the
// same distances, so one loop over the points forms both: the bound first, and
// the estimate only outside the interior, loops twice over the points of bodies
// whose points lie apart (a classification of 200 bodies of 64 points in a cube
// 0.9 diameters wide 397 us, bound first 421, estimate first 397 before; of 1000
// 824, 881 and 971; six points each 223, 228 and 369).
//
// Bound by the arithmetic of the visited nodes and of each plane's preparation
// where bodies are many (1000 in 512^3: 285 us; 425 with FP64 row ends, a
// binary search for each node's row and the bound after the estimate), by the
// chain of one plane's steps where they are few (one body: 6.4 us, before 7.1).
template <int T>
__global__ __launch_bounds__(T, 8) void k_mark(const uint32_t* __restrict__ err, uint32_t* own, const double* ball, int h, PartDev P,
                                              Geom g, uint8_t* flag, int store_flag, uint32_t* cand,
                                              int64_t cap, uint32_t* cursors, uint32_t* link_cursor,
                                              uint32_t* other_set)
{
    if (*err) return;  // the boxes failed their check: leave every plane and count as it is
    if (blockIdx.x == 0) {
        // (the lowest plane lies beyond the ball, whose radius is below h)
        if (threadIdx.x == 0) link_cursor[(int64_t)blockIdx.y * kCursorPad] = 0u;
        if (blockIdx.y == 0 && threadIdx.x < kSetWords) other_set[threadIdx.x] = 0u;
        return;
    }
    constexpr int kSegs = 8 * T;           // segments of 8 nodes listed at a time
    constexpr uint32_t kCandBuf = 8 * T;
    __shared__ float4 sf[kMaxCtrl];
    __shared__ uint32_t seg[kSegs];  // row, first x (both from the box's corner)
    __shared__ int wsum[4];
    __shared__ uint32_t cbuf[kCandBuf];  // this plane's candidates, in walk order
    __shared__ uint32_t ccount, gbase;
    const int p = blockIdx.y;
    const double bx = ball[4 * p + 0], by = ball[4 * p + 1], bz = ball[4 * p + 2];
    const double R = ball[4 * p + 3];
    const int ox = (int)floor(bx), oy = (int)floor(by), oz = (int)floor(bz);
    const int zi = oz - h + (int)blockIdx.x;
    const double dzc = (double)zi - bz;
    const double r2z = R * R - dzc * dzc;
    if (r2z < 0.0) return;  // uniform over the block
    const int S = 2 * h + 1;
    const int a0 = P.off[p], n = min(P.off[p + 1] - a0, kMaxCtrl);
    const double c0 = P.c0[p];
    const double* wp = P.wpts + 3 * (int64_t)a0;
    const double* Kp = P.K + a0;
    for (int i = threadIdx.x; i < n; i += T) {
        const double dz = (double)zi - wp[3 * i + 2];
        sf[i] = make_float4((float)(wp[3 * i] - (double)ox), (float)(wp[3 * i + 1] - (double)oy),
                            (float)(dz * dz), (float)Kp[i]);
    }
    if (threadIdx.x == 0) ccount = 0;
    __syncthreads();
    const float c0f = (float)c0;
    float ksum = 0.0f;
    for (int i = 0; i < n; ++i) ksum += sf[i].w;
    const float span = (float)(2 * h + 4), slack = span * 0x1p-21f, slack2 = span * span * 0x1p-20f;
    const float rho2 = ksum / c0f * 1.00002f + slack2;
    // rows: thread t takes rows rpt t .. rpt t + rpt - 1, rpt up to 4
    const int rpt = (S + T - 1) / T;
    const float bxf = (float)(bx - (double)ox), byf = (float)(by - (double)oy);
    const float r2zf = (float)r2z * 1.000001f + slack2;
    uint32_t span8[4];  // first x from the box's corner << 16 | segments
    int tsum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int r = rpt * (int)threadIdx.x + k;
        span8[k] = 0;
        if (k < rpt && r < S) {
            const float Y = (float)(r - h), dyc = Y - byf;
            const float r2x = r2zf - dyc * dyc;
            if (r2x >= 0.0f) {
                const float rx = __builtin_amdgcn_sqrtf(r2x) * 1.000001f + slack;
                float lo = 3e38f, hi = -3e38f;
                for (int i = 0; i < n; ++i) {
                    const float4 q = sf[i];
                    const float dy = Y - q.y;
                    const float rem = rho2 - (dy * dy + q.z);
                    if (rem >= 0.0f) {
                        const float w = __builtin_amdgcn_sqrtf(rem) * 1.000001f + slack;
                        lo = fminf(lo, q.x - w);
                        hi = fmaxf(hi, q.x + w);
                    }
                }
                lo = ceilf(fmaxf(lo - slack, bxf - rx));
                hi = floorf(fminf(hi + slack, bxf + rx));
                if (hi >= lo) {  // some control-point ball meets the row
                    const int x = max((int)lo, -h);
                    const int c = (min((int)hi, h) - x + 8) >> 3;
                    span8[k] = (uint32_t)(x + h) << 16 | (uint32_t)c;
                    tsum += c;
                }
            }
        }
    }
    // block-wide exclusive scan of the per-thread sums
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = tsum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    int off = incl - tsum, total;
    if constexpr (T == 64) {
        total = __shfl(incl, 63, 64);
    } else {
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        for (int w = 0; w < wv; ++w) off += wsum[w];
        total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    }
    if (total == 0) return;  // uniform over the block

    uint32_t* list = cand + (int64_t)p * cap;
    uint32_t* cursor = cursors + (int64_t)p * kCursorPad;
    const float c0hi = c0f * 1.0001f, c0lo = c0f * 0.9999f;
    const float gr = fmaxf(0.5f, 0.0085f * (float)(2 * h + 4));
    const float guard2 = h <= 127 ? gr * gr : 3.0e38f;
    for (int s0 = 0; s0 < total; s0 += kSegs) {
        int at = off - s0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (k < rpt) {
                const uint32_t row = (uint32_t)(rpt * (int)threadIdx.x + k) << 16;
                const uint32_t x = span8[k] >> 16;
                for (uint32_t i = 0; i < (span8[k] & 0xFFFFu); ++i, ++at)
                    if (at >= 0 && at < kSegs) seg[at] = row | (x + 8u * i);
            }
        }
        __syncthreads();
        const int nodes = 8 * min(total - s0, kSegs);
        for (int j0 = 0; j0 < nodes; j0 += T) {
            const int j = j0 + (int)threadIdx.x;
            bool keep = false;
            uint32_t node = 0;
            if (j < nodes) {
                const uint32_t sg = seg[j >> 3];
                const int xr = (int)(sg & 0xFFFFu) - h + (j & 7), yr = (int)(sg >> 16) - h;
                const int ii[3] = {ox + xr, oy + yr, zi};
                int c[3];
                if (wrap_cell(ii, g, c)) {
                    node = node_idx(c, g);
                    const float X = (float)xr, Y = (float)yr;
                    float Mf = 0.0f, m2 = 3.0e38f, lb = 0.0f;
                    for (int i = 0; i < n; ++i) {
                        const float4 q = sf[i];
                        const float dx = X - q.x, dy = Y - q.y;
                        const float r2 = fmaf(dx, dx, fmaf(dy, dy, q.z));
                        Mf = fmaf(q.w, __builtin_amdgcn_rcpf(r2), Mf);
                        m2 = fminf(m2, r2);
                        const float t = __builtin_amdgcn_sqrtf(r2) + kMaxSpeedUp;
                        lb = fmaf(q.w, __builtin_amdgcn_rcpf(t * t), lb);
                    }
                    const bool interior = h <= 127 && lb >= c0hi;
                    const bool settled = Mf >= c0hi || Mf <= c0lo;  // false for NaN
                    bool solid = interior || Mf >= c0hi;
                    if (!interior && (m2 < guard2 || !settled))
                        solid = metaball_rare(wp, Kp, n, (double)ii[0], (double)ii[1],
                                              (double)ii[2]) >= c0;
                    if (solid) {
                        atomicMin(own + node, (uint32_t)p);
                        if (store_flag) flag[node] = 1;
                        keep = !interior;
                    }
                }
            }
            // candidates gather in LDS so that the plane's list stays contiguous
            // and in row order (neighbouring candidates then share owner rows in
            // k_links); a full buffer spills lanes straight to the list
            const uint64_t m = __ballot(keep);
            if (m) {  // uniform over the wave
                uint32_t wbase = 0;
                if (lane == 0) wbase = atomicAdd(&ccount, (uint32_t)__popcll(m));
                wbase = __shfl(wbase, 0, 64);
                if (keep) {
                    const uint32_t idx = wbase + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    if (idx < kCandBuf) {
                        cbuf[idx] = node;
                    } else {
                        const uint32_t slot = atomicAdd(cursor, 1u);
                        if (slot < cap) list[slot] = node;
                    }
                }
            }
        }
        __syncthreads();
    }
    const uint32_t nb = min(ccount, (uint32_t)kCandBuf);
    if (threadIdx.x == 0) gbase = nb ? atomicAdd(cursor, nb) : 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nb; i += T)
        if (gbase + i < cap) list[gbase + i] = cbuf[i];
}

// Over the previous balls: flags of the new classification and the nodes that
// particle p covered before and that are fluid now.
struct Finish {
    const uint32_t* own_prev;
    const double* ball;  // the previous classification's
    uint8_t* flag;
    RefillRec* rec;
    int64_t cap;
    uint32_t* cursor;
};

__device__ __forceinline__ void finish_plane(const Finish& F, const uint32_t* own_new, int p, int h,
                                             int plane, const Geom& g)
{
    const int lane = threadIdx.x & 63;
    walk_ball_plane(F.ball + 4 * p, h, plane, g, [&](const uint32_t* node, const bool* on) {
        uint32_t now[2], was[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            now[k] = on[k] ? own_new[node[k]] : 0u;
            was[k] = on[k] ? F.own_prev[node[k]] : kFluid;
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (on[k]) F.flag[node[k]] = now[k] != kFluid;
            const bool refill = now[k] == kFluid && was[k] == (uint32_t)p;
            const uint64_t m = __ballot(refill);
            if (!m) continue;  // uniform over the wave
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(F.cursor, (uint32_t)__popcll(m));
            base = __shfl(base, 0, 64);
            const uint32_t slot = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            if (refill && slot < F.cap) {
                F.rec[slot].node = node[k];
                F.rec[slot].part = (uint32_t)p;
            }
        }
    });
}

// q of Eq. (calq): the root of g(q) = M(x_n + q e_d) - c0 on [0, 1] (g(0) < 0
// <= g(1)), by Newton-Raphson from the estimate of Eq. (appq), kept inside the
// bracket of the sign change (a step that leaves it becomes the midpoint),
// stopping on a step below 1e-13 or after 60 steps.  Along the line
// dM/dq = sum_i -2 K_i ((x - x_i) . e_d) / r_i^4.  Every value is formed in
// the order written (this file has no contraction), so any IEEE
// implementation of the same sequence gets the same bits.
__device__ double exact_q(const double* sp, int n, const double Xn[3], const int e[3], double c0,
                          double Mn, double Ms)
{
    double a = 0.0, b = 1.0;
    double q = (c0 - Mn) / (Ms - Mn);
    for (int it = 0; it < 60; ++it) {
        double M = 0.0, dM = 0.0;
        for (int i = 0; i < n; ++i) {
            const double dx = (Xn[0] + q * (double)e[0]) - sp[4 * i + 0];
            const double dy = (Xn[1] + q * (double)e[1]) - sp[4 * i + 1];
            const double dz = (Xn[2] + q * (double)e[2]) - sp[4 * i + 2];
            const double r2 = (dx * dx + dy * dy) + dz * dz;
            const double t = sp[4 * i + 3] / r2;
            const double se = (dx * (double)e[0] + dy * (double)e[1]) + dz * (double)e[2];
            M = M + t;
            dM = dM - ((2.0 * t) * se) / r2;
        }
        const double g = M - c0;
        if (g == 0.0) break;
        if (g < 0.0)
            a = q;
        else
            b = q;
        double qn = q - g / dM;
        if (!(qn > a && qn < b)) qn = 0.5 * (a + b);
        if (fabs(qn - q) < 1e-13) {
            q = qn;
            break;
        }
        q = qn;
    }
    return q;
}

// Link records of the candidate nodes of p (those p owns), written
// direction-major within each wave: the links of one direction over a run of
// neighbouring candidates are contiguous, so the link kernel's gathers
// coalesce.  Each lane first finds the link directions of its candidate; the
// wave then lists its (direction, candidate) pairs in LDS in that order and
// gives one to each lane (candidate data by lane shuffles), so the FP64 work of
// q runs on full waves.  A grid of a few workgroups per particle strides over
// the list.
// With few particles a wave takes cpw = 12 candidates instead of 64: at about
// five links each one round of the lanes then, and more waves where the list is
// too small to fill the chip.
//
// One body is bound by the chain of loads, quotients and the cursor's atomic
// (8.6 us; 14.4 with directions compared at run time, the list's k-th link
// searched by each lane, the quotients of M one after the other and 16
// candidates a wave), many by issue and gathers (1000 in 512^3: 444 us, before
// 575; 60 with exact fractions 38 us, before 48).
// FINISH: workgroups after the links' take the planes of finish_plane, which
// need nothing of the links (200 bodies 28.5 us together; apart 27.4 and 9.5).
template <bool FINISH>
__global__ __launch_bounds__(256, FINISH ? 5 : 6) void k_links(const uint32_t* __restrict__ err, const uint32_t* own, const double* ball, PartDev P,
                                               Geom g, const uint32_t* cand, int64_t cand_cap,
                                               const uint32_t* cand_cursors, LinkRec* links,
                                               const int64_t* __restrict__ loff,
                                               uint32_t* cursors, int treat, uint32_t gx,
                                               uint32_t cpw, uint32_t link_blocks, Finish F, int h)
{
    if (*err) return;  // the boxes failed their check: leave every plane as it is
    __shared__ double sp[4 * kMaxCtrl];
    __shared__ uint16_t pairs[4][64 * (kQ - 1)];  // per wave: direction << 6 | lane
    if constexpr (FINISH)
        if (blockIdx.x >= link_blocks) {  // uniform over the block
            const uint32_t b = blockIdx.x - link_blocks, S = 2u * (uint32_t)h + 1u;
            finish_plane(F, own, (int)(b / S), h, (int)(b % S), g);
            return;
        }
    uint32_t bx, by;
    if (!xcd_tile(link_blocks, gx, (uint32_t)P.n, bx, by)) return;  // uniform over the block
    const int p = (int)by;
    const uint32_t count = min((uint32_t)cand_cap, cand_cursors[(int64_t)p * kCursorPad]);
    const uint32_t chunk = 4u * cpw;  // candidates of one workgroup per round
    if (bx * chunk >= count) return;  // uniform over the block
    const int n = stage_ctrl(P, p, sp);
    const double c0 = P.c0[p];
    const double B[3] = {ball[4 * p], ball[4 * p + 1], ball[4 * p + 2]};  // loaded once
    const uint32_t* list = cand + (int64_t)p * cand_cap;
    LinkRec* out = links + loff[p];
    const int64_t cap = loff[p + 1] - loff[p];  // p's segment
    uint32_t* cursor = cursors + (int64_t)p * kCursorPad;
    const int lane = threadIdx.x & 63;
    uint16_t* pl = pairs[threadIdx.x >> 6];
    for (uint32_t base0 = bx * chunk; base0 < count; base0 += gx * chunk) {
        const uint32_t k = base0 + (threadIdx.x >> 6) * cpw + (uint32_t)lane;
        uint32_t node = 0, mask = 0, fmask = 0;  // link directions; those with x_f fluid
        int u[3] = {0, 0, 0};  // unwrapped: the image nearest the particle centre
        if ((uint32_t)lane < cpw && k < count) {
            node = list[k];
            uint32_t c[3], o[3][3];
            bool in[3][3];
            node_xyz(node, g, c[0], c[1], c[2]);
            axis3(c[0], g.n[0], g.per[0], 1u, o[0], in[0]);
            axis3(c[1], g.n[1], g.per[1], g.n[0], o[1], in[1]);
            axis3(c[2], g.n[2], g.per[2], (uint32_t)g.n[0] * (uint32_t)g.n[1], o[2], in[2]);
            // the node's owner and its neighbours' in one batch of loads
            // (each from a valid address), before any branch on them
            const uint32_t self = own[node];
            uint32_t onv[kQ];
#pragma unroll
            for (int d = 1; d < kQ; ++d)
                onv[d] = own[o[0][1 - cx(d)] + o[1][1 - cy(d)] + o[2][1 - cz(d)]];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                u[a] = (int)c[a];
                if (g.per[a]) {
                    const double d = (double)u[a] - B[a];
                    if (d > 0.5 * g.n[a]) u[a] -= g.n[a];
                    else if (d < -0.5 * g.n[a]) u[a] += g.n[a];
                }
            }
            if (self == (uint32_t)p) {
                uint32_t rest = 0;  // neither p's nor fluid: of another body or beyond a wall
#pragma unroll
                for (int d = 1; d < kQ; ++d) {
                    const bool ok = in[0][1 - cx(d)] && in[1][1 - cy(d)] && in[2][1 - cz(d)];
                    if (ok && onv[d] == kFluid) fmask |= 1u << d;
                    if (!ok || (onv[d] != kFluid && onv[d] != (uint32_t)p)) rest |= 1u << d;
                }
                mask = fmask;
                if (treat & LBM_TREAT_MISSING)
                    while (rest) {
                        const int d = __ffs(rest) - 1;
                        rest &= rest - 1u;
                        int e[3];
                        dir_of(d, e);
                        if (metaball(sp, n, (double)(u[0] - e[0]), (double)(u[1] - e[1]),
                                     (double)(u[2] - e[2])) < c0)
                            mask |= 1u << d;
                    }
            }
        }
        // direction-major list of the wave's links
        uint32_t total = 0;
#pragma unroll
        for (int d = 1; d < kQ; ++d) {
            const bool on = (mask >> d) & 1u;
            const uint64_t m = __ballot(on);
            if (on)
                pl[total + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    (uint16_t)(d << 6 | lane);
            total += (uint32_t)__popcll(m);
        }
        if (total == 0) continue;  // uniform over the wave
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t wbase = 0;
        if (lane == 0) wbase = atomicAdd(cursor, total);
        double Ms = 0.0;
        if (mask) Ms = metaball(sp, n, (double)u[0], (double)u[1], (double)u[2]);
        wbase = __shfl(wbase, 0, 64);
        for (uint32_t j0 = 0; j0 < total; j0 += 64) {
            const uint32_t j = j0 + (uint32_t)lane;
            const uint32_t e16 = j < total ? pl[j] : 64u;
            const int src = (int)(e16 & 63u), d = (int)(e16 >> 6);
            const uint32_t snode = __shfl(node, src, 64);
            const int su[3] = {__shfl(u[0], src, 64), __shfl(u[1], src, 64), __shfl(u[2], src, 64)};
            const double sMs = __shfl(Ms, src, 64);
            const uint32_t sfmask = __shfl(fmask, src, 64);
            if (j < total) {
                int e[3];
                dir_of(d, e);
                int kind = LBM_LINK_MISSING;
                if ((sfmask >> d) & 1u) {  // x_f exists and is fluid
                    // x_ff = x_s - 2 e (u lies within half a period of the
                    // lattice: one wrap)
                    int cff[3];
                    bool okf = true;
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        int v = su[a] - 2 * e[a];
                        if (v < 0 || v >= g.n[a]) {
                            if (g.per[a])
                                v = wrap_axis(v, g.n[a]);
                            else
                                okf = false;
                        }
                        cff[a] = v;
                    }
                    const bool ff = okf && own[node_idx(cff, g)] == kFluid;
                    kind = ((treat & LBM_TREAT_VIBB) && ff) ? LBM_LINK_VIBB : LBM_LINK_HALFWAY;
                }
                const double Xn[3] = {(double)(su[0] - e[0]), (double)(su[1] - e[1]),
                                      (double)(su[2] - e[2])};
                const double Mn = metaball(sp, n, Xn[0], Xn[1], Xn[2]);
                const uint32_t slot = wbase + j;
                if (slot < cap) {
                    LinkRec r;
                    r.node = snode;
                    r.part = (uint16_t)p;
                    r.d = (uint8_t)d;
                    r.kind = (uint8_t)kind;
                    r.q = (treat & LBM_TREAT_EXACT_Q) ? exact_q(sp, n, Xn, e, c0, Mn, sMs)
                                                      : (c0 - Mn) / (sMs - Mn);
                    out[slot] = r;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Flags and refill list from the whole lattice (four consecutive nodes per
// thread, 16-byte owner loads), used when the balls cover most of the lattice
// and a coalesced sweep is cheaper.
__global__ __launch_bounds__(256) void k_finish_all(const uint32_t* __restrict__ err, const uint32_t* own_prev,
                                                    const uint32_t* own_new, Geom g, uint8_t* flag,
                                                    RefillRec* rec, int64_t cap, uint32_t* cursor,
                                                    const uint32_t* inc_bad)
{
    if (*err) return;  // the boxes failed their check: leave every plane as it is
    if (inc_bad && *inc_bad == 0u) return;  // the candidate pass did the work
    // grid-stride over groups of four nodes (a bounded grid: when the
    // candidate pass did the work, its workgroups only read the word above)
    for (uint32_t base0 = blockIdx.x * 1024u; base0 < g.ncell; base0 += gridDim.x * 1024u) {
        const uint32_t base = base0 + threadIdx.x * 4u;
        uint32_t on[4] = {kFluid, kFluid, kFluid, kFluid}, op[4] = {kFluid, kFluid, kFluid, kFluid};
        if (base + 3u < g.ncell) {
            const uint4 a = *reinterpret_cast<const uint4*>(own_new + base);
            const uint4 b = *reinterpret_cast<const uint4*>(own_prev + base);
            on[0] = a.x, on[1] = a.y, on[2] = a.z, on[3] = a.w;
            op[0] = b.x, op[1] = b.y, op[2] = b.z, op[3] = b.w;
            *reinterpret_cast<uchar4*>(flag + base) =
                make_uchar4(on[0] != kFluid, on[1] != kFluid, on[2] != kFluid, on[3] != kFluid);
        } else {
            for (int k = 0; k < 4; ++k)
                if (base + k < g.ncell) {
                    on[k] = own_new[base + k];
                    op[k] = own_prev[base + k];
                    flag[base + k] = on[k] != kFluid;
                }
        }
        uint32_t cnt = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) cnt += (op[k] != kFluid && on[k] == kFluid) ? 1u : 0u;
        uint32_t slot = wave_reserve(cnt, cursor);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (op[k] != kFluid && on[k] == kFluid) {
                if (slot < cap) {
                    rec[slot].node = base + k;
                    rec[slot].part = op[k];
                }
                ++slot;
            }
    }
}

// Dense mode, bodies moved less than the guard of k_begin: the flags of the
// nodes that left a body and the refill list, from the previous
// classification's candidate lists (a node solid then and fluid now was
// within reach of the old surface, hence a candidate).  New solid nodes got
// their flag from k_mark.  One workgroup per (chunk, particle).
__global__ __launch_bounds__(256) void k_finish_cand(const uint32_t* __restrict__ err,
                                                     const uint32_t* __restrict__ inc_bad,
                                                     const uint32_t* __restrict__ own_prev,
                                                     const uint32_t* __restrict__ own_new,
                                                     const uint32_t* __restrict__ cand,
                                                     int64_t cand_cap,
                                                     const uint32_t* __restrict__ counts,
                                                     uint8_t* flag, RefillRec* rec, int64_t cap,
                                                     uint32_t* cursor)
{
    if (*err || *inc_bad) return;  // the lattice sweep does the work
    const int p = blockIdx.y;
    const uint32_t cnt = min((uint32_t)cand_cap, counts[p]);
    for (uint32_t i0 = blockIdx.x * 256u; i0 < cnt; i0 += gridDim.x * 256u) {
        const uint32_t i = i0 + threadIdx.x;
        bool left = false;
        uint32_t node = 0;
        if (i < cnt) {
            node = cand[(int64_t)p * cand_cap + i];
            // a node in two bodies is on both lists: its owner's list takes it
            left = own_prev[node] == (uint32_t)p && own_new[node] == kFluid;
            if (left) flag[node] = 0;
        }
        uint32_t slot = wave_reserve(left ? 1u : 0u, cursor);
        if (left && slot < cap) {
            rec[slot].node = node;
            rec[slot].part = (uint32_t)p;
        }
    }
}

// A first classification has no refill whose launch could report.
__global__ __launch_bounds__(256) void k_latch_deferred(CounterReport r) { report_counters(r); }

__global__ void k_owner_export(const uint32_t* own, int32_t* out, uint32_t ncell)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= ncell) return;
    const uint32_t o = own[i];
    out[i] = o == kFluid ? 0 : (int32_t)o + 1;
}

__global__ void k_link_export(const LinkRec* links, const uint32_t* cursors,
                              const int64_t* loff, const uint32_t* chunk,
                              const int64_t* offsets, int32_t* node, int8_t* d, int8_t* kind,
                              int32_t* part, double* q)
{
    // one workgroup per 256-record chunk of the layout
    const int p = (int)chunk[blockIdx.x];
    const int64_t gi = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t l = gi - loff[p];
    const int64_t cnt = min(loff[p + 1] - loff[p], (int64_t)cursors[(int64_t)p * kCursorPad]);
    if (l >= cnt) return;
    const LinkRec r = links[gi];
    const int64_t o = offsets[p] + l;
    node[o] = (int32_t)r.node;
    d[o] = (int8_t)r.d;
    kind[o] = (int8_t)r.kind;
    part[o] = (int32_t)r.part;
    q[o] = r.q;
}

inline uint32_t blocks_for(int64_t n) { return (uint32_t)((n + 255) / 256); }

}  // namespace

namespace MDLBM_QNS {

hipError_t launch_begin(lbm_ctx* c, const PartDev& P, int slot, int slot_prev, bool inc,
                        uint32_t* own, int slot_clear)
{
    const int np = c->cfg.n_particles;
    if (np == 0) return hipSuccess;
    c->use_counters(c->ctr_set ^ 1);
    if (own && c->dense) {
        const hipError_t e = hipMemsetAsync(own, 0xFF, sizeof(uint32_t) * (size_t)c->geom.ncell, c->stream);
        if (e != hipSuccess) return e;
        own = nullptr;
    }
    hipLaunchKernelGGL(k_begin, dim3(own ? 1 + c->box.S : 1, np), dim3(own ? 256 : 64), 0, c->stream, P,
                       c->box.h, c->ball_hist + (int64_t)slot * 4 * np, c->err, c->geom,
                       c->ball_hist + (int64_t)slot_prev * 4 * np, c->quat_prev,
                       inc ? c->inc : nullptr, c->cand_cursor, c->cand_prev_count,
                       own, c->ball_hist + (int64_t)slot_clear * 4 * np);
    return hipGetLastError();
}

// From 4096 planes a wave per plane fills the chip, and the preparation of a
// plane is done by one wave, not four (200 bodies in 256^3: 12.4 us against 15.2,
// 1000 in 512^3 317 against 354, and 285 since the interior bound shares the
// estimate's loop); below, four waves share a plane's nodes (60 bodies: 8.9 us
// against 11.0, two 8.1 against 11.6).  Boxes beyond 256 rows take four waves (a lane keeps four rows).
constexpr int64_t kWavePlanes = 4096;

hipError_t launch_mark(lbm_ctx* c, uint32_t* own, const PartDev& P, int slot, bool inc)
{
    const int np = c->cfg.n_particles;
    if (np == 0) return hipSuccess;
    // in dense mode the lattice sweep of k_finish_all writes every flag,
    // unless the candidate pass runs (then the solid nodes' flags come from
    // here)
    const bool waves = (int64_t)c->box.S * np >= kWavePlanes && c->box.S <= 256;
    hipLaunchKernelGGL(waves ? k_mark<64> : k_mark<256>, dim3(c->box.S, np), dim3(waves ? 64 : 256), 0,
                       c->stream, c->err, own, c->ball_hist + (int64_t)slot * 4 * np, c->box.h, P,
                       c->geom, c->flag, (c->dense && !inc) ? 0 : 1, c->cand, c->cand_cap,
                       c->cand_cursor, c->link_cursor, c->ctr + kCtrSet[c->ctr_set ^ 1]);
    return hipGetLastError();
}

// The flags and refills of dense mode.
static hipError_t launch_finish_dense(lbm_ctx* c, const uint32_t* own_prev, const uint32_t* own_new,
                                      int np_prev, bool inc)
{
    if (inc) {
        // the candidate pass, or, should k_begin have found a body that moved
        // too far, the lattice sweep (each kernel checks the word)
        const uint32_t nb =
            (uint32_t)std::min<int64_t>(std::max<int64_t>(1, (c->cand_prev_cap + 255) / 256), 64);
        hipLaunchKernelGGL(k_finish_cand, dim3(nb, np_prev), dim3(256), 0, c->stream, c->err, c->inc,
                           own_prev, own_new, c->cand_prev, c->cand_prev_cap, c->cand_prev_count,
                           c->flag, c->refill, c->refill_cap, c->refill_cursor);
    }
    // 2048 workgroups (eight per compute unit) stride over the lattice
    const uint32_t nb = (uint32_t)std::min<int64_t>(((int64_t)c->geom.ncell + 1023) / 1024, 2048);
    hipLaunchKernelGGL(k_finish_all, dim3(nb), dim3(256), 0, c->stream, c->err, own_prev, own_new,
                       c->geom, c->flag, c->refill, c->refill_cap, c->refill_cursor,
                       inc ? c->inc : nullptr);
    return hipGetLastError();
}

hipError_t launch_finish_links(lbm_ctx* c, const uint32_t* own_prev, const uint32_t* own_new,
                               const PartDev& P, int slot, int slot_prev, bool inc, bool finish,
                               bool links)
{
    const int np = c->cfg.n_particles;
    if (np == 0) return hipSuccess;
    if (finish && c->dense) {
        const hipError_t e = launch_finish_dense(c, own_prev, own_new, np, inc);
        if (e != hipSuccess) return e;
        finish = false;
    }
    if (!finish && !links) return hipSuccess;
    // few particles: 12 candidates per wave and up to 96 workgroups each (60
    // bodies with exact fractions: 38 us; 42 with 16, 44 with 24)
    const uint32_t cpw = np <= 64 ? 12u : 64u;
    const int64_t chunk = 4 * (int64_t)cpw;
    const uint32_t per =
        (uint32_t)std::min<int64_t>(np <= 64 ? 96 : 16, (c->cand_cap + chunk - 1) / chunk);
    const uint32_t nb = links ? (per * (uint32_t)np + 7u) & ~7u : 0u;
    const uint32_t nf = finish ? (uint32_t)c->box.S * (uint32_t)np : 0u;
    const Finish F{own_prev, c->ball_hist + (int64_t)slot_prev * 4 * np, c->flag, c->refill,
                   c->refill_cap, c->refill_cursor};
    hipLaunchKernelGGL(finish ? k_links<true> : k_links<false>, dim3(nb + nf), dim3(256), 0,
                       c->stream, c->err, own_new,
                       c->ball_hist + (int64_t)slot * 4 * np, P, c->geom, c->cand, c->cand_cap,
                       c->cand_cursor, c->links, c->lay->off_dev, c->link_cursor,
                       c->cfg.treatments, per, cpw, nb, F, c->box.h);
    return hipGetLastError();
}

hipError_t launch_latch_deferred(lbm_ctx* c)
{
    hipLaunchKernelGGL(k_latch_deferred, dim3(blocks_for(std::max(c->cfg.n_particles, 1))), dim3(256), 0,
                       c->stream, counter_report(c, false));
    return hipGetLastError();
}

hipError_t launch_owner_export(const lbm_ctx* c, const uint32_t* own, int32_t* out)
{
    hipLaunchKernelGGL(k_owner_export, dim3(blocks_for(c->geom.ncell)), dim3(256), 0, c->stream,
                       own, out, c->geom.ncell);
    return hipGetLastError();
}

hipError_t launch_link_export(const lbm_ctx* c, int32_t* node, int8_t* d, int8_t* kind,
                              int32_t* part, double* q, const int64_t* offsets_dev)
{
    const int np = c->cfg.n_particles;
    if (np == 0 || c->link_max == 0 || c->lay->chunks() == 0) return hipSuccess;
    hipLaunchKernelGGL(k_link_export, dim3((uint32_t)c->lay->chunks()), dim3(256), 0, c->stream,
                       c->links, c->link_cursor, c->lay->off_dev, c->lay->chunk_dev, offsets_dev,
                       node, d, kind, part, q);
    return hipGetLastError();
}

}  // namespace MDLBM_QNS
}  // namespace mdlbm
