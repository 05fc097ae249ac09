// adjoint.hip -- reverse (discrete adjoint) sweep of the IFDLBM step: the
// gradient of a cavity objective with respect to the top angle theta, the
// power-law index n and the lid speed U.
//
// One time step maps the state (f-hat, Lambda) at t to the state at t + dt
// through Steps (2)-(6) of Section 4:
//   A  every node:     moments (Eqs. 2.10-2.11), equilibrium (Eq. 2.8), the
//                      lagged power-law lambda (Eqs. 2.12-2.14, 1.4), f-hat+
//                      and f-bar+ (Eqs. 2.15-2.16);
//   B  interior:       f-bar = f-bar+ - dt/2 S[f-bar+] (Eq. 3.7);
//   BH every node:     f(t + dt/2) = f-bar + dt/(4 lambda + dt) (f_eq - f-bar)
//                      (Eq. 2.17), wall nodes first taking f-bar by
//                      non-equilibrium extrapolation from the inward node;
//   C  interior:       f-hat(t + dt) = f-hat+ - dt S[f(t + dt/2)] (Eq. 3.6);
//   CB wall nodes:     extrapolation of the new f-hat from the inward node.
// S_k[phi] = c_k,xi M_xi(phi_k) + c_k,eta M_eta(phi_k) with the mixed difference
// of Eqs. (2.5)-(2.7) and the contravariant velocity of Eq. (3.6).
//
// The adjoint step takes the adjoint of the state at t + dt and returns that
// of the state at t, walking the stages backwards: CB, C, BH, B, A.  Each
// stage's transpose is written out by hand.  Stencil stages are transposed
// as gathers: node m collects, from every interior node x whose stencil reads
// m, the weight x gives to m (which depends on the upwind side chosen at x)
// times x's adjoint; the wall extrapolation is transposed the same way, the
// inward node collecting from the wall nodes that copy it.  The forward
// quantities a step needs (f-bar+, lambda, f-bar, f(t + dt/2)) are recomputed
// from the stored state at t, in FP64.  All stages of a step run in one kernel
// over tiles of nodes with their halo.
//
// Parameter adjoints are accumulated as those of the primitive quantities:
// cot(theta) through the metric terms a_j = 1/(1 + 2 eta_j cot), s_i = cot
// (2 xi_i - 1) (Eqs. 3.2-3.8.2) and the Jacobian of the objective; the time
// step (whose CFL rule may involve cot); 3K (Eq. 2.15.1); the exponent
// (n - 1)/2 of Eq. (1.4); the lid velocity (Eq. 1.5); and, at the initial
// state of Step (1), the initial lambda and the lid row's equilibrium.  Each
// kernel reduces them per block into its own slot of a running FP64 sum, so
// the result does not depend on scheduling.
#include <cmath>
#include <type_traits>
#include <vector>

#include "ifdlbm_internal.h"

namespace ifd {

namespace {

constexpr int kB = 256;   // threads per block

// accumulators of the primitive parameter adjoints
enum Acc { A_COT = 0, A_DT, A_K3, A_EXPO, A_ULID, A_LAM0, A_N };
// one slot of block sums per kernel that contributes
enum Slot { S_OBJ = 0, S_STEP, S_INIT, S_N };

struct AdjParams {
    int nx, ny, pitch;
    int64_t plane;       // of a stored state
    double dt, K3, expo, g2min, mix, ulid, inv2dxi, inv2deta, dxi, deta;
    const double* geo;   // a_j [ny], s_i [nx], d a_j / d cot [ny], d s_i / d cot [nx]
    double* acc;         // [S_N][blocks][A_N]
    int blocks;
};

__device__ __forceinline__ bool node_of(const AdjParams& p, int& i, int& j)
{
    const int n = blockIdx.x * kB + threadIdx.x;
    if (n >= p.nx * p.ny) return false;
    j = n / p.nx;
    i = n - j * p.nx;
    return true;
}

__device__ __forceinline__ bool interior(const AdjParams& p, int i, int j)
{
    return i >= 1 && j >= 1 && i <= p.nx - 2 && j <= p.ny - 2;
}

__device__ __forceinline__ int64_t at(const AdjParams& p, int i, int j) { return (int64_t)j * p.nx + i; }

// Block sum of up to A_N accumulators, added by thread 0 into slot `slot`
// of this block (each (slot, block) pair has one writer per launch and
// launches are stream-ordered).
__device__ void accumulate(const AdjParams& p, int slot, const double (&v)[A_N])
{
    __shared__ double sh[A_N][kB];
#pragma unroll
    for (int q = 0; q < A_N; ++q) sh[q][threadIdx.x] = v[q];
    __syncthreads();
    for (int w = kB / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int q = 0; q < A_N; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double* a = p.acc + ((int64_t)slot * p.blocks + blockIdx.x) * A_N;
#pragma unroll
        for (int q = 0; q < A_N; ++q) a[q] += sh[q][0];
    }
}

// ------------------------------------------------ local transposes (FP64)

// Transpose of moments(): (P-bar, ux-bar, uy-bar) at u -> g-bar.
// P = 0.6 sum_{k>0} g_k - 0.4 |u|^2, u = sum c_k g_k.
__device__ __forceinline__ void moments_t(double ux, double uy, double Pb, double uxb, double uyb, double gb[9])
{
    const double ax = uxb - 0.8 * ux * Pb, ay = uyb - 0.8 * uy * Pb, s = 0.6 * Pb;
    gb[0] = 0.0;
#pragma unroll
    for (int k = 1; k < 9; ++k) gb[k] = cxk(k) * ax + cyk(k) * ay + s;
}

// Transpose of equilibrium(): e-bar -> (P-bar, ux-bar, uy-bar), added.
// e_0 = -5/3 P - 2/3 |u|^2; e_k = w_k (3 P - 1.5 |u|^2 + 3 c.u + 4.5 (c.u)^2).
__device__ __forceinline__ void equilibrium_t(double ux, double uy, const double eb[9], double& Pb, double& uxb,
                                              double& uyb)
{
    Pb += -5.0 / 3.0 * eb[0];
    uxb += -4.0 / 3.0 * ux * eb[0];
    uyb += -4.0 / 3.0 * uy * eb[0];
#pragma unroll
    for (int k = 1; k < 9; ++k) {
        const double w = k < 5 ? 1.0 / 9.0 : 1.0 / 36.0, cx = cxk(k), cy = cyk(k);
        const double cu = cx * ux + cy * uy, we = w * eb[k], dq = 3.0 + 9.0 * cu;
        Pb += 3.0 * we;
        uxb += we * (-3.0 * ux + dq * cx);
        uyb += we * (-3.0 * uy + dq * cy);
    }
}

// Transpose of extrapolate(x_nb, uwall): x_b-bar -> x_nb-bar (added) and
// uwall-bar (returned).  x_b = e(P, uwall, 0) + x_nb - e(P, u_nb), (P, u_nb) =
// moments(x_nb).
__device__ __forceinline__ double extrapolate_t(const double xnb[9], double uwall, const double xbb[9], double xnbb[9])
{
    double P, ux, uy;
    moments(xnb, P, ux, uy);
    double Pb = 0.0, uwb = 0.0, uwyb = 0.0, uxb = 0.0, uyb = 0.0;
    equilibrium_t(uwall, 0.0, xbb, Pb, uwb, uwyb);
    double m[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) m[k] = -xbb[k];
    equilibrium_t(ux, uy, m, Pb, uxb, uyb);
    double gb[9];
    moments_t(ux, uy, Pb, uxb, uyb, gb);
#pragma unroll
    for (int k = 0; k < 9; ++k) xnbb[k] += xbb[k] + gb[k];
    return uwb;
}

// Weight of phi(i + o) in 2h M(phi)(i) (Eqs. 2.5-2.7) for the upwind side
// `pos` (contravariant velocity >= 0) and the first-order fallbacks at
// i = 1 (lo) and i = N - 2 (hi); the forward form is mixed_diff_2h.
__device__ __forceinline__ double stencil_weight(int o, bool pos, bool lo, bool hi, double eps)
{
    const double u = 1.0 - eps;
    switch (o) {
    case -2: return pos && !lo ? u : 0.0;
    case -1: return -eps + (pos ? (lo ? -2.0 * u : -4.0 * u) : 0.0);
    case 0: return pos ? (lo ? 2.0 * u : 3.0 * u) : (hi ? -2.0 * u : -3.0 * u);
    case 1: return eps + (!pos ? (hi ? 2.0 * u : 4.0 * u) : 0.0);
    default: return !pos && !hi ? -u : 0.0;
    }
}

// The q-th of the wall nodes that may extrapolate from the interior node (i, j): the edge node on the side wall, the
// one on the bottom or lid, and the corner.  False where the node is not next to that wall.
__device__ __forceinline__ bool wall_of(const AdjParams& p, int i, int j, int q, int& wi, int& wj)
{
    const int di = i == 1 ? -1 : (i == p.nx - 2 ? 1 : 0), dj = j == 1 ? -1 : (j == p.ny - 2 ? 1 : 0);
    wi = q == 1 ? i : i + di;
    wj = q == 0 ? j : j + dj;
    return (q == 1 || di) && (q == 0 || dj);
}

// ------------------------------------------------------- adjoint stages

// Objective, Eq. (5.1): J = sum 1/2 w_i w_j dxi deta J_j |u|^2, J_j = 1 + 2
// eta_j cot.  Writes the block sums of J (slot S_OBJ, accumulator A_N - 1 is
// not used: J goes to `jpart`) and the state adjoint at the final step.
__global__ __launch_bounds__(kB) void a_objective(AdjParams p, double cot, const double* st, double* fbar,
                                                  double* lbar, double* jpart)
{
    __shared__ double sj[kB];
    double v[A_N] = {};
    double jl = 0.0;
    int i, j;
    if (node_of(p, i, j)) {
        const int64_t id = at(p, i, j), pl = (int64_t)p.nx * p.ny;
        double g[9], P, ux, uy;
        for (int k = 0; k < 9; ++k) g[k] = st[k * pl + id];
        moments(g, P, ux, uy);
        const double wi = (i == 0 || i == p.nx - 1) ? 0.5 : 1.0, wj = (j == 0 || j == p.ny - 1) ? 0.5 : 1.0;
        const double w = wi * wj * p.dxi * p.deta, eta = j * p.deta, Jj = 1.0 + 2.0 * eta * cot;
        const double uu = ux * ux + uy * uy;
        jl = 0.5 * w * Jj * uu;
        v[A_COT] = w * eta * uu;
        double gb[9];
        moments_t(ux, uy, 0.0, w * Jj * ux, w * Jj * uy, gb);
        for (int k = 0; k < 9; ++k) fbar[k * pl + id] = gb[k];
        lbar[id] = 0.0;
    }
    sj[threadIdx.x] = jl;
    __syncthreads();
    for (int w = kB / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sj[threadIdx.x] += sj[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) jpart[blockIdx.x] = sj[0];
    accumulate(p, S_OBJ, v);
}

// One adjoint step of a tile of 12 x 12 nodes: from the adjoint of the state
// at t + dt (fb_in, lb_in) to that of the state at t (fb_out, lb_out).  One
// workgroup holds the tile and four more nodes on every side, one per thread,
// and walks them through the forward stages and back, each stage's values in
// LDS: a node's distance from the tile is at most 4 for A and CB^T, 2 for B,
// BH, C^T, BH^T and the wall transpose (one more for the wall nodes next to
// those), 0 for B^T and A^T.  Parameter adjoints are summed over the nodes of
// the tile proper.
// Bound by the chain of a thread: 2230 vector and 245 LDS instructions of a
// wavefront on 129 x 129 nodes (1660 and 227 clear of the walls), 55 % of its
// time spent waiting (dependent FP64 instructions, LDS, five barriers, 16 to 36
// spilled registers): 20 us on 33 x 33 and 21 us on 129 x 129 nodes, where the
// nine launches of a stage each, through HBM, took 105 us.  Tiles of 8 x 8 recompute more halo (50 against 45 us per
// step of the whole adjoint on 129 x 129 before the walls' loops left their
// arrays), tiles of 16 x 16 leave 168 registers per thread, which spill (59 us).
constexpr int kTile = 12, kHalo = 4, kSide = kTile + 2 * kHalo;
constexpr int kNodes = kSide * kSide, kThreads = (kNodes + kWaveLanes - 1) / kWaveLanes * kWaveLanes;

struct AdjLds {
    double bp[9][kNodes];   // f-bar+
    // moving populations k = 1 .. 8 in plane k - 1
    double fh[8][kNodes];   // f(t + dt/2)
    double G[8][kNodes];    // adjoint of the new f-hat, then of f-bar
    double X[8][kNodes];    // adjoint of the half-step input
};

// 2h times the mixed difference at a node from points `step` apart: eps * central + (1 - eps) * upwind on the points
// sorted by the upwind side (a1 one behind, a2 two behind, f1 one ahead), without a branch; edge: the second upwind
// point leaves the grid (first-order form, as with the linear ghost 2 a1 - c0).
__device__ __forceinline__ double mixed_at(const double* x, int step, bool pos, bool edge, double eps)
{
    const int u = pos ? -step : step;
    const double c0 = x[0], a1 = x[u], f1 = x[-u], far = x[2 * u];
    const double a2 = edge ? 2.0 * a1 - c0 : far;
    const double m = eps * (f1 - a1) + (1.0 - eps) * (3.0 * c0 - 4.0 * a1 + a2);
    return pos ? m : -m;
}

// Tiles [xa, xb) x [ya, yb) of the tx x ty ones keep clear of the walls and the nodes next to them: they take the
// kernel without wall handling.  EDGE runs the frame around them, or every tile where that is one launch less.
struct TileFrame {
    int tx, ty, xa, xb, ya, yb;
    __host__ __device__ int edge_tiles() const { return tx * ty - (xb - xa) * (yb - ya); }
    __device__ void tile(bool edge, int b, int& x, int& y) const
    {
        const int w = xb - xa, h = yb - ya;
        if (!edge) {
            x = xa + b % w;
            y = ya + b / w;
            return;
        }
        const int side = tx - w, mid = h * side;   // the rows below, beside and above the inner tiles
        if (b < ya * tx || b >= ya * tx + mid) {
            const int c = b < ya * tx ? b : b - mid + h * tx;
            x = c % tx;
            y = c / tx;
            return;
        }
        const int c = b - ya * tx, q = c % side;
        x = q < xa ? q : q + w;
        y = ya + c / side;
    }
};

template <int PREC, bool EDGE>
__global__ __launch_bounds__(kThreads, 2) void k_adjoint_step(AdjParams p, TileFrame fr, const typename Storage<PREC>::F* st,
                                                        const typename Storage<PREC>::L* lst,
                                                        const typename Storage<PREC>::F* st1, const double* fb_in,
                                                        const double* lb_in, double* fb_out, double* lb_out)
{
    using S = Storage<PREC>;
    __shared__ AdjLds sh;
    double v[A_N] = {};
    int bx, by;
    fr.tile(EDGE, (int)blockIdx.x, bx, by);
    bx = __builtin_amdgcn_readfirstlane(bx);
    by = __builtin_amdgcn_readfirstlane(by);
    const int nx = p.nx, ny = p.ny, t = min((int)threadIdx.x, kNodes - 1), lx = t % kSide, ly = t / kSide;
    const int i0 = bx * kTile, j0 = by * kTile;
    const int i = i0 - kHalo + lx, j = j0 - kHalo + ly;
    const bool grid = !EDGE || (i >= 0 && j >= 0 && i < nx && j < ny);
    const bool in = !EDGE || interior(p, i, j), wall = grid && !in;
    // the inward node of a wall node
    const int ci = EDGE ? min(max(i, 1), nx - 2) : i, cj = EDGE ? min(max(j, 1), ny - 2) : j;
    auto dist = [&](int x, int y) { return max(max(i0 - x, x - (i0 + kTile - 1)), max(j0 - y, y - (j0 + kTile - 1))); };
    const bool near = grid && dist(ci, cj) <= 2;   // B, BH and their transposes
    const bool own = grid && dist(i, j) <= 0;      // the tile proper
    const int64_t pl = (int64_t)nx * ny;
    const int gi = EDGE ? min(max(i, 0), nx - 1) : i, gj = EDGE ? min(max(j, 0), ny - 1) : j;
    const int64_t id = at(p, gi, gj), rid = (int64_t)gj * p.pitch + gi;

    double g[9], gadj[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) g[k] = (double)S::load(st, k * p.plane + rid, k);
    const double lam_old = (double)lst[rid];
    int64_t again = 0;   // an offset the compiler does not know, so that it loads the state again
    asm volatile("" : "+s"(again));
#pragma unroll
    for (int k = 0; k < 9; ++k) gadj[k] = in ? fb_in[k * pl + id] : 0.0;   // wall f-hat+ is not used
    const double lbar = lb_in[id];
    const double aj = p.geo[gj], ajd = p.geo[ny + nx + gj];          // a_j, d a_j / d cot
    const double si = p.geo[ny + gi], sid = p.geo[2 * ny + nx + gi];  // s_i, d s_i / d cot

    const double acj = EDGE ? p.geo[cj] : aj, sci = EDGE ? p.geo[ny + ci] : si;
    // s of the columns whose xi stencils read this node
    double sc[5];
#pragma unroll
    for (int o = -2; o <= 2; ++o) sc[o + 2] = p.geo[ny + (EDGE ? min(max(i - o, 0), nx - 1) : i - o)];

    // ------------------------------------------------------------- A
    double lam, pw, m, Q, r, pxx, pyy, pxy, P, ux, uy;
    bool floor;
    moments(g, P, ux, uy);
    const Equilibrium<double> eq(P, ux, uy);
    {
        double n[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) n[k] = eq.from(k, g[k]);
        const double s58 = (n[5] + n[6]) + (n[7] + n[8]);
        pxx = (n[1] + n[3]) + s58;
        pyy = (n[2] + n[4]) + s58;
        pxy = (n[5] - n[6]) + (n[7] - n[8]);
        Q = pxx * pxx + 2.0 * pxy * pxy + pyy * pyy;
        r = 1.0 / (2.0 * lam_old + p.dt);
        const double gamma2 = 18.0 * Q * r * r;
        floor = !(gamma2 > p.g2min);
        m = floor ? p.g2min : gamma2;
        pw = pow_pos<double>(m, p.expo);   // the power of the FP64 step: lambda as the trajectory took it
        lam = p.K3 * pw;
        const double bb = 1.5 * p.dt / (2.0 * lam + p.dt);
#pragma unroll
        for (int k = 0; k < 9; ++k) sh.bp[k][t] = g[k] - bb * n[k];
    }
    // CB^T: the adjoint of the interior values of the new state: its own plus what the wall nodes extrapolated from
    // this node hand back
    if (EDGE && in && (i == 1 || j == 1 || i == nx - 2 || j == ny - 2)) {
        double x[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) x[k] = (double)S::load(st1, k * p.plane + rid, k);
#pragma unroll 1
        for (int q = 0; q < 3; ++q) {
            int wi, wj;
            if (!wall_of(p, i, j, q, wi, wj)) continue;
            double xb[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) xb[k] = fb_in[k * pl + at(p, wi, wj)];
            const double uwb = extrapolate_t(x, wj == ny - 1 ? p.ulid : 0.0, xb, gadj);
            if (own && wj == ny - 1) v[A_ULID] += uwb;
        }
    }
#pragma unroll
    for (int k = 1; k < 9; ++k) sh.G[k - 1][t] = gadj[k];
    sh.X[0][t] = 0.0;   // read past the last plane of G by wall nodes three away from the tile, with zero weight
    __syncthreads();

    // --------------------------------------------------------- B, BH
    const int ct = t + (ci - i) + (cj - j) * kSide;   // the inward node in the tile
    double x[9], hc = 0.0, den = 1.0;
    double uxh = 0.0, uyh = 0.0, dh[9];   // velocity of the half-step input and e - x
    if (near) {
        x[0] = sh.bp[0][ct];
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            const double* plane = &sh.bp[k][ct];
            const double c = acj * ((double)cxk(k) - (double)cyk(k) * sci);
            double str = c * (mixed_at(plane, 1, c >= 0.0, EDGE && ci == (c >= 0.0 ? 1 : nx - 2), p.mix) * p.inv2dxi);
            if (cyk(k) != 0)
                str += (double)cyk(k) * (mixed_at(plane, kSide, cyk(k) > 0, EDGE && cj == (cyk(k) > 0 ? 1 : ny - 2), p.mix) * p.inv2deta);
            x[k] = plane[0] - 0.5 * p.dt * str;
            __builtin_amdgcn_sched_barrier(0);   // keeps the reads of later populations from being moved up
        }
        if (EDGE && wall) extrapolate(x, j == ny - 1 ? p.ulid : 0.0, x);
        double Ph;
        moments(x, Ph, uxh, uyh);
        const Equilibrium<double> eh(Ph, uxh, uyh);
        den = 4.0 * lam + p.dt;
        hc = p.dt / den;
#pragma unroll
        for (int k = 0; k < 9; ++k) dh[k] = eh.minus(k, x[k]);
#pragma unroll
        for (int k = 1; k < 9; ++k) sh.fh[k - 1][t] = x[k] + hc * dh[k];
    }
    __syncthreads();

    // Transposed stencil of population k at this node: the sum over the interior nodes ix = i - o and jx = j - o whose
    // stencils read it of their y times the weight they give to it.  The weights of all other nodes are zero; what is
    // read for them is finite (the tile's row wraps, or plane 0 of X).
    auto stencil_t = [&](const double* y, int k) {
        double sx = 0.0;
        if (!EDGE || (j >= 1 && j <= ny - 2)) {
#pragma unroll
            for (int o = -2; o <= 2; ++o) {
                const int ix = i - o;
                const double d = (double)cxk(k) - (double)cyk(k) * sc[o + 2];
                double w = stencil_weight(o, d >= 0.0, EDGE && ix == 1, EDGE && ix == nx - 2, p.mix);
                if (EDGE && (ix < 1 || ix > nx - 2)) w = 0.0;
                sx += (y[-o] * d) * w;
            }
            sx *= aj * p.inv2dxi;
        }
        if (cyk(k) != 0 && (!EDGE || (i >= 1 && i <= nx - 2))) {
            double se = 0.0;
#pragma unroll
            for (int o = -2; o <= 2; ++o) {
                const int jx = j - o;
                double w = stencil_weight(o, cyk(k) > 0, EDGE && jx == 1, EDGE && jx == ny - 2, p.mix);
                if (EDGE && (jx < 1 || jx > ny - 2)) w = 0.0;
                se += y[-o * kSide] * w;
            }
            sx += se * ((double)cyk(k) * p.inv2deta);
        }
        return sx;
    };
    // Adjoints of dt and cot through the stream term of one interior node: y_k is the adjoint of -scale dt S_k.
    auto stream_adjoint = [&](const double (*tile)[kNodes], const double (&y)[9], double scale) {
        double sdt = 0.0, scot = 0.0;
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            const double* plane = &tile[k - 1][t];
            const double d = (double)cxk(k) - (double)cyk(k) * si, c = aj * d;
            const double mxi = mixed_at(plane, 1, c >= 0.0, EDGE && i == (c >= 0.0 ? 1 : nx - 2), p.mix) * p.inv2dxi;
            double str = c * mxi;
            if (cyk(k) != 0)
                str += (double)cyk(k) * (mixed_at(plane, kSide, cyk(k) > 0, EDGE && j == (cyk(k) > 0 ? 1 : ny - 2), p.mix) * p.inv2deta);
            sdt += y[k] * str;
            scot += y[k] * ((ajd * d - aj * (double)cyk(k) * sid) * mxi);
            __builtin_amdgcn_sched_barrier(0);   // keeps the reads of later populations from being moved up
        }
        v[A_DT] -= scale * sdt;
        v[A_COT] -= scale * p.dt * scot;
    };

    // ----------------------------------------------------- C^T, BH^T
    double xb[9], lb = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) xb[k] = 0.0;
    if (near) {
        double eb[9], hcb = 0.0;
        eb[0] = 0.0;   // population 0 is not streamed: its half-step adjoint is zero
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            const double y = -p.dt * stencil_t(&sh.G[k - 1][t], k);
            xb[k] = (1.0 - hc) * y;
            eb[k] = hc * y;
            hcb += y * dh[k];
            __builtin_amdgcn_sched_barrier(0);   // keeps the reads of later populations from being moved up
        }
        double Pb = 0.0, uxb = 0.0, uyb = 0.0, mb[9];
        equilibrium_t(uxh, uyh, eb, Pb, uxb, uyb);
        moments_t(uxh, uyh, Pb, uxb, uyb, mb);
#pragma unroll
        for (int k = 1; k < 9; ++k) xb[k] += mb[k];
        lb = hcb * (-4.0 * p.dt / (den * den));
        if (own) v[A_DT] += hcb * (4.0 * lam / (den * den));
    }
    if (own && in) stream_adjoint(sh.fh, gadj, 1.0);
#pragma unroll
    for (int k = 1; k < 9; ++k) sh.X[k - 1][t] = xb[k];
    __syncthreads();

    // wall transpose of BH: adjoint of f-bar at interior nodes, over G
    if (EDGE && in && near && (i == 1 || j == 1 || i == nx - 2 || j == ny - 2)) {
#pragma unroll 1
        for (int q = 0; q < 3; ++q) {
            int wi, wj;
            if (!wall_of(p, i, j, q, wi, wj)) continue;
            const int tw = t + (wi - i) + (wj - j) * kSide;
            double y[9];
            y[0] = 0.0;
#pragma unroll
            for (int k = 1; k < 9; ++k) y[k] = sh.X[k - 1][tw];
            const double uwb = extrapolate_t(x, wj == ny - 1 ? p.ulid : 0.0, y, xb);
            if (own && wj == ny - 1) v[A_ULID] += uwb;
        }
    }
#pragma unroll
    for (int k = 1; k < 9; ++k) sh.G[k - 1][t] = in ? xb[k] : 0.0;
    __syncthreads();

    // the stored state again: not held in registers since stage A
#pragma unroll
    for (int k = 0; k < 9; ++k) g[k] = (double)S::load(st, k * p.plane + rid + again, k);
    // the weights of the transposed stencils are formed again in B^T: held from C^T on they would take 80 registers
#pragma unroll
    for (int o = 0; o < 5; ++o) asm volatile("" : "+v"(sc[o]));
    // ------------------------------------------------------ B^T, A^T
    if (own) {
        double yb[9];
        yb[0] = 0.0;
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            yb[k] = (in ? xb[k] : 0.0) - 0.5 * p.dt * stencil_t(&sh.G[k - 1][t], k);
            __builtin_amdgcn_sched_barrier(0);   // keeps the reads of later populations from being moved up
        }
        if (in) stream_adjoint(sh.bp + 1, xb, 0.5);
        const double R = 1.0 / (2.0 * lam + p.dt), bh = 2.0 * p.dt * R, bb = 1.5 * p.dt * R;
        // f-hat+ = g + bh (e - g), f-bar+ = g + bb (e - g)
        double gb[9], eb[9], bhb = 0.0, bbb = 0.0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const double yh = gadj[k];
            gb[k] = (1.0 - bh) * yh + (1.0 - bb) * yb[k];
            eb[k] = bh * yh + bb * yb[k];
            const double d = eq.minus(k, g[k]);
            bhb += yh * d;
            bbb += yb[k] * d;
        }
        const double Rb = 2.0 * p.dt * bhb + 1.5 * p.dt * bbb;
        v[A_DT] += 2.0 * R * bhb + 1.5 * R * bbb - Rb * R * R;
        const double lamb = lb + lbar - 2.0 * Rb * R * R;
        // lambda = K3 m^expo
        v[A_K3] = lamb * pw;
        v[A_EXPO] = lamb * lam * log(m);
        double lam_old_b = 0.0;
        if (!floor) {
            const double gb2 = lamb * lam * p.expo / m;
            const double Qb = gb2 * 18.0 * r * r, rb = gb2 * 36.0 * Q * r;
            lam_old_b = -2.0 * rb * r * r;
            v[A_DT] -= rb * r * r;
            const double pxxb = 2.0 * pxx * Qb, pyyb = 2.0 * pyy * Qb, pxyb = 4.0 * pxy * Qb;
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                const double cx = cxk(k), cy = cyk(k);
                const double nb = cx * cx * pxxb + cx * cy * pxyb + cy * cy * pyyb;
                gb[k] += nb;
                eb[k] -= nb;
            }
        }
        double Pb = 0.0, uxb = 0.0, uyb = 0.0, mb[9];
        equilibrium_t(ux, uy, eb, Pb, uxb, uyb);
        moments_t(ux, uy, Pb, uxb, uyb, mb);
#pragma unroll
        for (int k = 0; k < 9; ++k) fb_out[k * pl + id] = gb[k] + mb[k];
        lb_out[id] = lam_old_b;
    }
    // sums over the tile: each wavefront, then the wavefronts, in a fixed order
    __shared__ double sums[kThreads / kWaveLanes][A_N];
#pragma unroll
    for (int q = 0; q < A_N; ++q) {
        if (q == A_LAM0) continue;   // none in a step
        double sv = v[q];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sv += __shfl_xor(sv, off, kWaveLanes);
        if (threadIdx.x % kWaveLanes == 0) sums[threadIdx.x / kWaveLanes][q] = sv;
    }
    __syncthreads();
    if ((int)threadIdx.x < A_N && threadIdx.x != A_LAM0) {
        double sv = 0.0;
#pragma unroll
        for (int w = 0; w < kThreads / kWaveLanes; ++w) sv += sums[w][t];
        p.acc[((int64_t)S_STEP * p.blocks + by * fr.tx + bx) * A_N + t] += sv;
    }
}

// Step (1)^T: f-hat = e(0, u) with u = (U, 0) on the lid row, Lambda = lam0.
__global__ __launch_bounds__(kB) void a_initial(AdjParams p, const double* fbar, const double* lbar)
{
    double v[A_N] = {};
    int i, j;
    if (node_of(p, i, j)) {
        const int64_t id = at(p, i, j), pl = (int64_t)p.nx * p.ny;
        v[A_LAM0] = lbar[id];
        if (j == p.ny - 1) {
            double eb[9], Pb = 0.0, uxb = 0.0, uyb = 0.0;
            for (int k = 0; k < 9; ++k) eb[k] = fbar[k * pl + id];
            equilibrium_t(p.ulid, 0.0, eb, Pb, uxb, uyb);
            v[A_ULID] = uxb;
        }
    }
    accumulate(p, S_INIT, v);
}

}  // namespace

// --------------------------------------------------------------- host side

struct AdjointSweep::Impl {
    AdjParams p{};
    double cot = 0.0;
    size_t nn = 0, nb = 0;
    int prec = 0, cur = 0;
    TileFrame frame{};
    double *geo = nullptr, *acc = nullptr, *jpart = nullptr;
    double *fbar[2] = {nullptr, nullptr}, *lbar[2] = {nullptr, nullptr};   // adjoint of the state, before and after a step
};

AdjointSweep::AdjointSweep() : d(new Impl) {}

AdjointSweep::~AdjointSweep() { delete d; }

namespace {

struct SweepSizes {
    size_t nn, nb, tx, ty, slots;   // slots: accumulators of one kind
    explicit SweepSizes(const CavityDesc& c)
        : nn((size_t)c.nx * c.ny), nb((nn + kB - 1) / kB), tx((size_t)(c.nx + kTile - 1) / kTile),
          ty((size_t)(c.ny + kTile - 1) / kTile), slots(tx * ty > nb ? tx * ty : nb)
    {
    }
};

}  // namespace

// doubles: metric tables, accumulators, objective partial sums, two adjoint states
size_t AdjointSweep::work_doubles(const CavityDesc& c)
{
    const SweepSizes z(c);
    return 2 * (size_t)(c.nx + c.ny) + S_N * z.slots * A_N + z.nb + 20 * z.nn;
}

hipError_t AdjointSweep::init(const CavityDesc& c, int prec, double* work, hipStream_t s)
{
    Impl& m = *d;
    const SweepSizes z(c);
    m.cot = c.cot;
    m.nn = z.nn;
    m.nb = z.nb;
    m.prec = prec;
    // a tile and its halo are clear of the walls' neighbours: T b - 4 >= 2 and T (b + 1) + 4 <= n - 2
    auto inner_end = [](int n, int lo) { return n >= 2 * kTile + 6 ? (n - 6) / kTile : lo; };
    TileFrame& fr = m.frame;
    fr = {(int)z.tx, (int)z.ty, 1, inner_end(c.nx, 1), 1, inner_end(c.ny, 1)};
    // while every tile has a CU of its own, one launch of the general kernel is the shorter
    if (fr.tx * fr.ty <= 256 || fr.xb <= fr.xa || fr.yb <= fr.ya) fr.xa = fr.xb = fr.ya = fr.yb = 0;
    std::vector<double> geo(2 * (c.nx + c.ny));
    for (int j = 0; j < c.ny; ++j) {
        const double eta = j * c.deta, a = 1.0 / (1.0 + 2.0 * c.cot * eta);
        geo[j] = a;
        geo[c.ny + c.nx + j] = -2.0 * eta * a * a;
    }
    for (int i = 0; i < c.nx; ++i) {
        const double w = (double)(2 * i - (c.nx - 1)) / (double)(c.nx - 1);
        geo[c.ny + i] = c.cot * w;
        geo[2 * c.ny + c.nx + i] = w;
    }
    auto take = [&](size_t n) {
        double* q = work;
        work += n;
        return q;
    };
    m.geo = take(geo.size());
    m.acc = take(S_N * z.slots * A_N);
    m.jpart = take(z.nb);
    for (int b = 0; b < 2; ++b) {
        m.fbar[b] = take(9 * z.nn);
        m.lbar[b] = take(z.nn);
    }
    hipError_t e = hipMemcpyAsync(m.geo, geo.data(), geo.size() * sizeof(double), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemsetAsync(m.acc, 0, S_N * z.slots * A_N * sizeof(double), s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);   // geo lives on the host's stack
    AdjParams& p = m.p;
    p.nx = c.nx;
    p.ny = c.ny;
    p.pitch = c.pitch;
    p.plane = c.plane;
    p.dt = c.dt;
    p.K3 = 3.0 * c.K;
    p.expo = c.expo;
    p.g2min = c.g2min;
    p.mix = c.mix;
    p.ulid = c.u_lid;
    p.inv2dxi = c.inv2dxi;
    p.inv2deta = c.inv2deta;
    p.dxi = c.dxi;
    p.deta = c.deta;
    p.geo = m.geo;
    p.acc = m.acc;
    p.blocks = (int)z.slots;
    return e;
}

hipError_t AdjointSweep::objective(const double* state, hipStream_t s)
{
    Impl& m = *d;
    hipLaunchKernelGGL(a_objective, dim3(m.nb), dim3(kB), 0, s, m.p, m.cot, state, m.fbar[m.cur], m.lbar[m.cur], m.jpart);
    return hipGetLastError();
}

hipError_t AdjointSweep::step_back(const void* f, const void* l, const void* f1, hipStream_t s)
{
    Impl& m = *d;
    auto go = [&](auto prec) {
        constexpr int P = decltype(prec)::value;
        using F = typename Storage<P>::F;
        auto launch = [&](auto kernel, int tiles) {
            hipLaunchKernelGGL(kernel, dim3(tiles), dim3(kThreads), 0, s, m.p, m.frame, static_cast<const F*>(f),
                               static_cast<const typename Storage<P>::L*>(l), static_cast<const F*>(f1), m.fbar[m.cur],
                               m.lbar[m.cur], m.fbar[m.cur ^ 1], m.lbar[m.cur ^ 1]);
        };
        const int edge = m.frame.edge_tiles(), inner = m.frame.tx * m.frame.ty - edge;
        if (inner > 0) launch(k_adjoint_step<P, false>, inner);
        launch(k_adjoint_step<P, true>, edge);
    };
    // the FP32 modes store alike
    switch (m.prec) {
    case P_FP64: go(std::integral_constant<int, P_FP64>{}); break;
    case P_FP16DEV: go(std::integral_constant<int, P_FP16DEV>{}); break;
    default: go(std::integral_constant<int, P_FP32>{}); break;
    }
    m.cur ^= 1;
    return hipGetLastError();
}

hipError_t AdjointSweep::finish(const CavityDesc& c, double dt_dcot, double lam0_dU, double K_dn, double K_dU,
                                hipStream_t s, double* J, double grad[3])
{
    Impl& m = *d;
    hipLaunchKernelGGL(a_initial, dim3(m.nb), dim3(kB), 0, s, m.p, m.fbar[m.cur], m.lbar[m.cur]);
    hipError_t e = hipGetLastError();
    std::vector<double> acc((size_t)S_N * m.p.blocks * A_N), jp(m.nb);
    if (e == hipSuccess) e = hipMemcpyAsync(acc.data(), m.acc, acc.size() * sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(jp.data(), m.jpart, jp.size() * sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    double t[A_N] = {};
    for (size_t q = 0; q < (size_t)S_N * m.p.blocks; ++q)
        for (int a = 0; a < A_N; ++a) t[a] += acc[q * A_N + a];
    double j = 0.0;
    for (double x : jp) j += x;
    *J = j;
    const double dcot_dtheta = -(1.0 + c.cot * c.cot);
    grad[0] = (t[A_COT] + t[A_DT] * dt_dcot) * dcot_dtheta;
    grad[1] = 3.0 * t[A_K3] * K_dn + 0.5 * t[A_EXPO];
    grad[2] = 3.0 * t[A_K3] * K_dU + t[A_ULID] + t[A_LAM0] * lam0_dU;
    return hipSuccess;
}

}  // namespace ifd
