// gradient.hip -- derivative of a cavity objective with respect to the top
// angle theta (radians), the power-law index n and the lid speed U, by
// forward (tangent-linear) differentiation of the discrete IFDLBM step.
//
// Every quantity of the step carries its value and its three partial
// derivatives (Dual<3>, FP64).  The parameters enter through the metric terms
// a_j = 1/(1 + 2 eta_j cot theta), s_i = cot theta (2 xi_i - 1) (Eqs. 3.2-3.8.2),
// the time step (CFL rule on the contravariant speed 1 + cot theta), the
// consistency K = U^(2-n) / Re (Eq. 2.15.1), the exponent (n - 1)/2 of
// Eq. (1.4), the lid velocity (Eq. 1.5) and the initial lambda U / (Re c_s^2).
// The objective is the kinetic energy of Eq. (5.1) after n_steps steps.  With
// three parameters the tangent sweep costs about four forward runs and needs
// no stored trajectory; the derivative is that of the discrete objective, the
// same one a reverse sweep would return.
#include <cmath>
#include <mutex>
#include <string>
#include <vector>

#include "dual.h"
#include "ifdlbm_internal.h"

namespace ifd {

using D3 = Dual<3>;

namespace {

// A quantity that depends on theta only (metric terms, time step): value and theta derivative.
struct Th {
    double v, d;
};

struct TParams {
    int nx, ny;
    double mix, g2min, inv2dxi, inv2deta;
    Th dt, cot;
    D3 K, expo, ulid, lam0;
    double dxi, deta;
};

// ------------------------------------------------ arithmetic of the step
// Written out for what is a constant (four products), what depends on theta
// only (five) and what carries all three derivatives (seven).

__device__ __forceinline__ D3 times(double a, const D3& x)
{
    D3 r;
    r.v = a * x.v;
#pragma unroll
    for (int q = 0; q < 3; ++q) r.d[q] = a * x.d[q];
    return r;
}

__device__ __forceinline__ D3 axpy(double a, const D3& x, const D3& y)   // a x + y
{
    D3 r;
    r.v = __builtin_fma(a, x.v, y.v);
#pragma unroll
    for (int q = 0; q < 3; ++q) r.d[q] = __builtin_fma(a, x.d[q], y.d[q]);
    return r;
}

__device__ __forceinline__ D3 muladd(const D3& a, const D3& b, const D3& c)   // a b + c
{
    D3 r;
    r.v = __builtin_fma(a.v, b.v, c.v);
#pragma unroll
    for (int q = 0; q < 3; ++q) r.d[q] = __builtin_fma(a.d[q], b.v, __builtin_fma(a.v, b.d[q], c.d[q]));
    return r;
}

__device__ __forceinline__ D3 muladd(const Th& a, const D3& b, const D3& c)   // a b + c
{
    D3 r;
    r.v = __builtin_fma(a.v, b.v, c.v);
#pragma unroll
    for (int q = 0; q < 3; ++q) r.d[q] = __builtin_fma(a.v, b.d[q], c.d[q]);
    r.d[0] = __builtin_fma(a.d, b.v, r.d[0]);
    return r;
}

// Eqs. (2.10)-(2.11) on deviations (see moments in lbm_device.h)
__device__ __forceinline__ void moments_t(const D3 (&g)[9], D3& P, D3& ux, D3& uy)
{
    ux = (g[1] - g[3]) + (g[5] - g[6]) - (g[7] - g[8]);
    uy = (g[2] - g[4]) + (g[5] + g[6]) - (g[7] + g[8]);
    const D3 s = ((g[1] + g[2]) + (g[3] + g[4])) + ((g[5] + g[6]) + (g[7] + g[8]));
    P.v = 0.6 * s.v - 0.4 * (ux.v * ux.v + uy.v * uy.v);
#pragma unroll
    for (int q = 0; q < 3; ++q) P.d[q] = 0.6 * s.d[q] - 0.8 * (ux.v * ux.d[q] + uy.v * uy.d[q]);
}

// Eq. (2.8) (see Equilibrium in lbm_device.h)
struct EquilibriumT {
    D3 base, e0, ux, uy;
    __device__ __forceinline__ EquilibriumT(const D3& P, const D3& x, const D3& y) : ux(x), uy(y)
    {
        D3 uu;
        uu.v = x.v * x.v + y.v * y.v;
#pragma unroll
        for (int q = 0; q < 3; ++q) uu.d[q] = 2.0 * (x.v * x.d[q] + y.v * y.d[q]);
        base = axpy(-1.5, uu, times(3.0, P));
        e0 = axpy(-5.0 / 3.0, P, times(-2.0 / 3.0, uu));
    }
    // e_k + s v for s = 1 or -1
    __device__ __forceinline__ D3 plus(int k, double s, const D3& v) const
    {
        if (k == 0) return axpy(s, v, e0);
        const D3 cu = k == 1 ? ux : k == 2 ? uy : k == 3 ? -ux : k == 4 ? -uy : k == 5 ? ux + uy : k == 6 ? uy - ux : k == 7 ? -(ux + uy) : ux - uy;
        const double w = k < 5 ? 1.0 / 9.0 : 1.0 / 36.0, slope = 3.0 + 9.0 * cu.v;
        D3 r;
        r.v = __builtin_fma(w, __builtin_fma(cu.v, __builtin_fma(4.5, cu.v, 3.0), base.v), s * v.v);
#pragma unroll
        for (int q = 0; q < 3; ++q) r.d[q] = __builtin_fma(w, __builtin_fma(slope, cu.d[q], base.d[q]), s * v.d[q]);
        return r;
    }
};

// Non-equilibrium extrapolation onto a wall node (see extrapolate in lbm_device.h)
__device__ __forceinline__ void extrapolate_t(D3 (&x)[9], const D3& uwall)
{
    D3 P, ux, uy;
    moments_t(x, P, ux, uy);
    const EquilibriumT nb(P, ux, uy), wall(P, uwall, D3(0.0));
#pragma unroll
    for (int k = 0; k < 9; ++k) x[k] = wall.plus(k, -1.0, nb.plus(k, -1.0, x[k]));
}

// scale dt / (m lam + dt), the relaxation coefficients of Eqs. (2.15)-(2.17)
__device__ __forceinline__ D3 relax_coef(double scale, const Th& dt, double m, const D3& lam)
{
    const double r = 1.0 / (m * lam.v + dt.v), b = scale * dt.v * r;
    D3 o;
    o.v = b;
#pragma unroll
    for (int q = 0; q < 3; ++q) o.d[q] = -b * r * m * lam.d[q];
    o.d[0] += (scale - b) * r * dt.d;
    return o;
}

// Steps (2)-(4): lambda (Eqs. 2.12-2.14, 1.4, every parameter differentiated: no Newtonian shortcut, as d mu / d n != 0
// at n = 1), f-bar+ (Eq. 2.16) and f-hat+ (Eq. 2.15, over g) of a node.  The power is the library's, within an ulp: that
// of the step kernels (about two) saves 2 % of a sweep of 129 x 129 nodes, but takes the root-mean-square error of
// (J, dJ/d theta, dJ/dn, dJ/dU) over 14 cavities, against extended precision, from (1.07, 0.39, 34, 1.13) to (1.10, 0.43,
// 36, 1.14) e-15.
__device__ __forceinline__ void collide_t(D3 (&g)[9], const D3& lam_old, const TParams& c, D3 (&bp)[9], D3& lam)
{
    D3 P, ux, uy, n[9];
    moments_t(g, P, ux, uy);
    const EquilibriumT eq(P, ux, uy);
#pragma unroll
    for (int k = 0; k < 9; ++k) n[k] = eq.plus(k, -1.0, g[k]);   // e - g
    const D3 s58 = (n[5] + n[6]) + (n[7] + n[8]);
    const D3 pxx = (n[1] + n[3]) + s58, pyy = (n[2] + n[4]) + s58, pxy = (n[5] - n[6]) + (n[7] - n[8]);
    const double r = 1.0 / (2.0 * lam_old.v + c.dt.v);
    const double Q = pxx.v * pxx.v + 2.0 * pxy.v * pxy.v + pyy.v * pyy.v, g2 = 18.0 * Q * r * r;
    const bool floored = !(g2 > c.g2min);
    const double m = floored ? c.g2min : g2, pw = pow(m, c.expo.v), lm = log(m);
    lam.v = 3.0 * c.K.v * pw;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double dr = -r * r * (2.0 * lam_old.d[q] + (q == 0 ? c.dt.d : 0.0));
        const double dQ = 2.0 * (pxx.v * pxx.d[q] + 2.0 * pxy.v * pxy.d[q] + pyy.v * pyy.d[q]);
        const double dg2 = floored ? 0.0 : 18.0 * r * (dQ * r + 2.0 * Q * dr);
        lam.d[q] = 3.0 * pw * (c.K.d[q] + c.K.v * (c.expo.v * dg2 / m + lm * c.expo.d[q]));
    }
    const D3 b_hat = relax_coef(2.0, c.dt, 2.0, lam), b_bar = times(0.75, b_hat);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        bp[k] = muladd(b_bar, n[k], g[k]);
        g[k] = muladd(b_hat, n[k], g[k]);
    }
}

// One step of a tile of T x T nodes with every derivative, as step_tile.hip
// does it: the workgroup holds the tile and four more nodes on every side, one
// per thread; f-bar+ and then f(t + dt/2) in LDS (a plane per population and
// component), f-hat+ in registers.  Bound by the chain of about 2500 vector
// instructions of a wavefront, mostly FP64, with 40 % (33 x 33) to 54 % (129 x
// 129) of its time spent waiting.  Five launches of a stage each through HBM
// took 44 us per step on 33 x 33 and 47 us on 129 x 129 nodes; tiles of 8 take 17
// and 29 us (342 registers, one wavefront per SIMD), tiles of 12, with less halo
// and two wavefronts per SIMD, 25 and 27 us (256 registers, 78 more spilled).
constexpr int kHalo = 4;
constexpr int side_of(int T) { return T + 2 * kHalo; }
constexpr int threads_of(int T) { return (side_of(T) * side_of(T) + kWaveLanes - 1) / kWaveLanes * kWaveLanes; }

template <int T>
struct TangentLds {
    static constexpr int kSide = side_of(T);
    double x[9][4][kSide * kSide];
    __device__ __forceinline__ void put(int k, int t, const D3& a)
    {
        x[k][0][t] = a.v;
#pragma unroll
        for (int q = 0; q < 3; ++q) x[k][q + 1][t] = a.d[q];
    }
    __device__ __forceinline__ D3 get(int k, int t) const
    {
        D3 a(x[k][0][t]);
#pragma unroll
        for (int q = 0; q < 3; ++q) a.d[q] = x[k][q + 1][t];
        return a;
    }
};

// 2h times the mixed difference (Eqs. 2.5-2.7) of population k at a node from points u apart, u pointing upwind; edge:
// the second upwind point leaves the grid (first-order form).
template <int T>
__device__ __forceinline__ D3 mixed_t(const TangentLds<T>& sh, int k, int t, int u, bool edge, double eps)
{
    D3 r;
    double* out[4] = {&r.v, &r.d[0], &r.d[1], &r.d[2]};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double* x = &sh.x[k][q][t];
        const double c0 = x[0], a1 = x[u], f1 = x[-u], far = x[2 * u];
        const double a2 = edge ? 2.0 * a1 - c0 : far;
        *out[q] = eps * (f1 - a1) + (1.0 - eps) * (3.0 * c0 - 4.0 * a1 + a2);
    }
    return r;
}

// base_k - sdt c_k . grad phi_k of the moving populations (Eqs. 3.4, 3.6, 3.7) at a node of the tile
template <int T, typename Base>
__device__ __forceinline__ void transport_t(const TangentLds<T>& sh, const TParams& c, int t, int i, int j, const Th& a,
                                            const Th& s, const Th& sdt, Base base, D3 (&out)[9])
{
    constexpr int kSide = side_of(T);
#pragma unroll
    for (int k = 1; k < 9; ++k) {
        const double cx = cxk(k), cy = cyk(k), d = cx - cy * s.v;
        // |c_xi| times the difference along the upwind direction; the theta derivative of c_xi is kept where c_xi is
        // zero (the upwind side is then the c >= 0 one, as in the forward step)
        const bool pos = d >= 0.0;
        const double sg = pos ? c.inv2dxi : -c.inv2dxi;
        const Th cxi{a.v * d * sg, (a.d * d - a.v * cy * s.d) * sg};
        D3 term = muladd(cxi, mixed_t(sh, k, t, pos ? -1 : 1, i == (pos ? 1 : c.nx - 2), c.mix), D3(0.0));
        if (cyk(k) > 0) term = axpy(c.inv2deta, mixed_t(sh, k, t, -kSide, j == 1, c.mix), term);
        if (cyk(k) < 0) term = axpy(c.inv2deta, mixed_t(sh, k, t, kSide, j == c.ny - 2, c.mix), term);
        out[k] = muladd(Th{-sdt.v, -sdt.d}, term, base(k));
        __builtin_amdgcn_sched_barrier(0);   // keeps the reads of later populations from being moved up (registers)
    }
}

template <int T>
__global__ __launch_bounds__(threads_of(T), T == 8 ? 1 : 2) void t_step(TParams c, const D3* fin, const D3* lin, const D3* geo,
                                                                         D3* fout, D3* lout)
{
    constexpr int kSide = side_of(T), kNodes = kSide * kSide;
    __shared__ TangentLds<T> sh;
    const int nx = c.nx, ny = c.ny, t = min((int)threadIdx.x, kNodes - 1), lx = t % kSide, ly = t / kSide;
    const int tx = (nx + T - 1) / T, by = (int)blockIdx.x / tx, bx = (int)blockIdx.x - by * tx;
    const int i0 = bx * T, j0 = by * T, i = i0 - kHalo + lx, j = j0 - kHalo + ly;
    const int64_t pl = (int64_t)nx * ny;
    // the nearest node of the grid: threads outside it compute a node that nothing reads
    const int64_t id = (int64_t)min(max(j, 0), ny - 1) * nx + min(max(i, 0), nx - 1);
    const bool grid = i >= 0 && j >= 0 && i < nx && j < ny;
    const bool wall = grid && (i == 0 || j == 0 || i == nx - 1 || j == ny - 1);
    const int ci = min(max(i, 1), nx - 2), cj = min(max(j, 1), ny - 2), ct = t + (ci - i) + (cj - j) * kSide;
    auto dist = [&](int x, int y) { return max(max(i0 - x, x - (i0 + T - 1)), max(j0 - y, y - (j0 + T - 1))); };
    const bool near = grid && dist(i, j) <= 2, own = grid && dist(i, j) <= 0;
    D3 g[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) g[k] = fin[k * pl + id];
    const D3 lam_old = lin[id], ga = geo[cj], gs = geo[ny + ci];
    const Th a{ga.v, ga.d[0]}, s{gs.v, gs.d[0]};

    // A
    D3 lam;
    {
        D3 bp[9];
        collide_t(g, lam_old, c, bp, lam);
#pragma unroll
        for (int k = 0; k < 9; ++k) sh.put(k, t, bp[k]);
    }
    if (own) lout[id] = lam;
    __syncthreads();
    // B and Eq. (2.17)
    D3 x[9];
    if (near) {
        x[0] = sh.get(0, ct);
        transport_t(sh, c, ct, ci, cj, a, s, Th{0.5 * c.dt.v, 0.5 * c.dt.d}, [&](int k) { return sh.get(k, ct); }, x);
        if (wall) extrapolate_t(x, j == ny - 1 ? c.ulid : D3(0.0));
        D3 P, ux, uy;
        moments_t(x, P, ux, uy);
        const EquilibriumT eq(P, ux, uy);
        const D3 b = relax_coef(1.0, c.dt, 4.0, lam);
#pragma unroll
        for (int k = 1; k < 9; ++k) x[k] = muladd(b, eq.plus(k, -1.0, x[k]), x[k]);
    }
    __syncthreads();
    if (near)
#pragma unroll
        for (int k = 1; k < 9; ++k) sh.put(k, t, x[k]);
    __syncthreads();
    // C: f-hat+ is in g
    if (own && !wall) transport_t(sh, c, t, i, j, a, s, c.dt, [&](int k) { return g[k]; }, g);
    // walls from their inward nodes, which may belong to another tile: those recompute nothing, the wall node is left
    // to the tile of its inward node
    const bool walls = i0 <= 1 || j0 <= 1 || i0 + T >= nx - 1 || j0 + T >= ny - 1;
    if (own && !wall) {
#pragma unroll
        for (int k = 0; k < 9; ++k) fout[k * pl + id] = g[k];
    }
    if (walls) {
        __syncthreads();
        if (own && !wall)
#pragma unroll
            for (int k = 0; k < 9; ++k) sh.put(k, t, g[k]);
        __syncthreads();
        if (wall && dist(ci, cj) <= 0) {
#pragma unroll
            for (int k = 0; k < 9; ++k) x[k] = sh.get(k, ct);
            extrapolate_t(x, j == ny - 1 ? c.ulid : D3(0.0));
#pragma unroll
            for (int k = 0; k < 9; ++k) fout[k * pl + id] = x[k];
        }
    }
}

__device__ inline bool node(const TParams& c, int& i, int& j)
{
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= c.nx * c.ny) return false;
    j = n / c.nx;
    i = n - j * c.nx;
    return true;
}

__global__ __launch_bounds__(256) void t_init(TParams c, D3* f, D3* l)
{
    int i, j;
    if (!node(c, i, j)) return;
    const int64_t id = (int64_t)j * c.nx + i, pl = (int64_t)c.nx * c.ny;
    const EquilibriumT eq(D3(0.0), j == c.ny - 1 ? c.ulid : D3(0.0), D3(0.0));
    for (int k = 0; k < 9; ++k) f[k * pl + id] = eq.plus(k, 1.0, D3(0.0));
    l[id] = c.lam0;
}

// Eq. (5.1) per block: 1/2 |u|^2 w_i w_j J_j dxi deta with J_j = 1 + 2 eta_j cot(theta).
__global__ __launch_bounds__(256) void t_energy(TParams c, const D3* f, D3* part)
{
    __shared__ double sh[4][256];
    int i, j;
    D3 e(0.0);
    if (node(c, i, j)) {
        const int64_t id = (int64_t)j * c.nx + i, pl = (int64_t)c.nx * c.ny;
        D3 g[9], P, ux, uy;
        for (int k = 0; k < 9; ++k) g[k] = f[k * pl + id];
        moments_t(g, P, ux, uy);
        const double wi = (i == 0 || i == c.nx - 1) ? 0.5 : 1.0;
        const double wj = (j == 0 || j == c.ny - 1) ? 0.5 : 1.0;
        D3 J(1.0 + 2.0 * j * c.deta * c.cot.v);
        J.d[0] = 2.0 * j * c.deta * c.cot.d;
        e = D3(0.5 * wi * wj * c.dxi * c.deta) * J * (ux * ux + uy * uy);
    }
    sh[0][threadIdx.x] = e.v;
    for (int q = 0; q < 3; ++q) sh[q + 1][threadIdx.x] = e.d[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 4; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        D3 s(sh[0][0]);
        for (int q = 0; q < 3; ++q) s.d[q] = sh[q + 1][0];
        part[blockIdx.x] = s;
    }
}

}  // namespace

namespace {

// Parameters of the step and the metric tables a_j, s_i, each with its derivatives with respect to
// (theta [rad], n, U).
void tangent_params(int nx, int ny, double re, double n, double theta_deg, double u_lid, double cfl, double mix,
                    double gamma_min, int dt_rule, TParams& P, std::vector<D3>& geo)
{
    const double th = theta_deg * (M_PI / 180.0);
    const double C = theta_deg == 90.0 ? 0.0 : 1.0 / std::tan(th);
    const double dC = -(1.0 + C * C);   // d cot / d theta
    const double U = std::fabs(u_lid), sgnU = u_lid < 0 ? -1.0 : 1.0;
    const double dxi = 1.0 / (nx - 1), deta = 1.0 / (ny - 1);
    P.nx = nx;
    P.ny = ny;
    P.dxi = dxi;
    P.deta = deta;
    P.cot = {C, dC};
    if (dt_rule == 1 || 1.0 / deta > (1.0 + C) / dxi) {
        P.dt = {dt_rule == 1 ? cfl * std::min(dxi, deta) : cfl * deta, 0.0};
    } else {
        const double dt = cfl * dxi / (1.0 + C);
        P.dt = {dt, -dt / (1.0 + C) * dC};
    }
    const double K = std::pow(U, 2.0 - n) / re;
    {
        double d[3] = {0, -K * std::log(U), (2.0 - n) * K / U * sgnU};
        P.K = D3::make(K, d);
    }
    {
        double d[3] = {0, 0.5, 0};
        P.expo = D3::make(0.5 * (n - 1.0), d);
    }
    P.g2min = gamma_min * gamma_min;
    P.mix = mix;
    {
        double d[3] = {0, 0, 1.0};
        P.ulid = D3::make(u_lid, d);
    }
    P.inv2dxi = 0.5 / dxi;
    P.inv2deta = 0.5 / deta;
    {
        double d[3] = {0, 0, 3.0 / re * sgnU};
        P.lam0 = D3::make(3.0 * U / re, d);
    }
    geo.resize(ny + nx);
    for (int j = 0; j < ny; ++j) {
        const double eta = j * deta, a = 1.0 / (1.0 + 2.0 * C * eta);
        double d[3] = {-2.0 * eta * a * a * dC, 0, 0};
        geo[j] = D3::make(a, d);
    }
    for (int i = 0; i < nx; ++i) {
        const double w = (double)(2 * i - (nx - 1)) / (double)(nx - 1);
        double d[3] = {w * dC, 0, 0};
        geo[ny + i] = D3::make(C * w, d);
    }
}

// Work arrays of one cavity, packed [k][j][i]: the state twice (nine planes and lambda each), the metric tables a_j,
// s_i, the energy partial sums.
struct TBuf {
    D3 *f[2], *l[2], *geo, *part;
};

size_t work_elems(int nx, int ny)
{
    const size_t nn = (size_t)nx * ny;
    return 20 * nn + (size_t)nx + (size_t)ny + (nn + 255) / 256;
}

// The arrays carved from one workspace of work_elems(nx, ny) values.
TBuf carve(D3* w, size_t nn, size_t ngeo)
{
    TBuf b{};
    auto take = [&](size_t n) {
        D3* q = w;
        w += n;
        return q;
    };
    for (int q = 0; q < 2; ++q) {
        b.f[q] = take(9 * nn);
        b.l[q] = take(nn);
    }
    b.geo = take(ngeo);
    b.part = take((nn + 255) / 256);
    return b;
}

// The sweep in a given workspace: Step (1), n_steps steps with their derivatives, Eq. (5.1).  Every
// work array is written before it is read, so the workspace needs no clearing.
hipError_t tangent_run(const TParams& P, const std::vector<D3>& geo, D3* work, int64_t n_steps, hipStream_t s,
                       double* J, double* grad, std::string& err)
{
    const size_t nn = (size_t)P.nx * P.ny, nb = (nn + 255) / 256;
    const TBuf b = carve(work, nn, geo.size());
    auto failed = [&](hipError_t e, const char* what) {
        err = std::string("gradient: ") + what + ": " + hipGetErrorString(e);
        return e;
    };
    hipError_t e = hipMemcpyAsync(b.geo, geo.data(), geo.size() * sizeof(D3), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return failed(e, "metric tables to the device");
    const dim3 g(nb), blk(256);
    // tiles of 8 while each has a CU of its own (see t_step)
    const int tile = ((P.nx + 7) / 8) * ((P.ny + 7) / 8) <= 256 ? 8 : 12;
    const auto step = tile == 8 ? t_step<8> : t_step<12>;
    const int threads = tile == 8 ? threads_of(8) : threads_of(12);
    // one dimension: tall grids have more rows of tiles than the 65536 workgroups of a launch's second dimension
    const dim3 tiles((unsigned)((P.nx + tile - 1) / tile) * (unsigned)((P.ny + tile - 1) / tile));
    hipLaunchKernelGGL(t_init, g, blk, 0, s, P, b.f[0], b.l[0]);
    if ((e = hipGetLastError()) != hipSuccess) return failed(e, "Step (1) launch");
    int cur = 0;
    for (int64_t t = 0; t < n_steps; ++t) {
        hipLaunchKernelGGL(step, tiles, dim3(threads), 0, s, P, b.f[cur], b.l[cur], b.geo, b.f[cur ^ 1], b.l[cur ^ 1]);
        cur ^= 1;
        if ((t & 1023) == 1023 && (e = hipGetLastError()) != hipSuccess) return failed(e, "step launch");
    }
    hipLaunchKernelGGL(t_energy, g, blk, 0, s, P, b.f[cur], b.part);
    if ((e = hipGetLastError()) != hipSuccess) return failed(e, "step or energy launch");
    std::vector<D3> part(nb);
    e = hipMemcpyAsync(part.data(), b.part, nb * sizeof(D3), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return failed(e, "energy partial sums to the host");
    D3 sum(0.0);
    for (const D3& x : part) sum += x;
    *J = sum.v;
    for (int q = 0; q < 3; ++q) grad[q] = sum.d[q];
    return hipSuccess;
}

// Work arrays of ifdlbm_gradient_noalloc: one array per GPU, held until the process ends.  Host code must not
// use this name as a device address: the address of each GPU's copy comes from hipGetSymbolAddress.
constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array (looked up on the first call on each device).
hipError_t scratch_of_current_device(void** out, std::string& err)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        err = std::string("hipGetDevice: ") + hipGetErrorString(e);
        return e;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        err = "device index beyond the library's table of scratch arrays";
        return hipErrorInvalidDevice;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
            return e != hipSuccess ? e : hipErrorInvalidSymbol;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

// The grids that ifdlbm_gradient_noalloc accepts are those of its documented limit of 48 values per node, which its
// work arrays (20 per node) stay well within.
size_t tangent_workspace_elems(int nx, int ny)
{
    const size_t nn = (size_t)nx * ny;
    return 48 * nn + (size_t)nx + (size_t)ny + (nn + 255) / 256;
}

size_t tangent_scratch_capacity_elems() { return kScratchBytes / sizeof(D3); }

// Host driver; returns a HIP error or hipSuccess and fills J and grad[3].  The work arrays live in one
// allocation made and freed here, or, with use_scratch, in the current device's scratch array.
hipError_t tangent_kinetic_energy(int nx, int ny, double re, double n, double theta_deg, double u_lid, double cfl,
                                  double mix, double gamma_min, int dt_rule, int64_t n_steps, hipStream_t s, double* J,
                                  double* grad, std::string& err, bool use_scratch)
{
    TParams P;
    std::vector<D3> geo;
    tangent_params(nx, ny, re, n, theta_deg, u_lid, cfl, mix, gamma_min, dt_rule, P, geo);
    D3* work = nullptr;
    hipError_t e = hipSuccess;
    if (use_scratch) {
        if (tangent_workspace_elems(nx, ny) > tangent_scratch_capacity_elems()) {
            err = "grid too large for the scratch array";
            return hipErrorInvalidValue;
        }
        void* p = nullptr;
        e = scratch_of_current_device(&p, err);
        if (e != hipSuccess) return e;
        work = static_cast<D3*>(p);
    } else {
        e = hipMalloc(reinterpret_cast<void**>(&work), work_elems(nx, ny) * sizeof(D3));
        if (e != hipSuccess) {
            err = std::string("gradient: ") + hipGetErrorString(e);
            return e;
        }
    }
    e = tangent_run(P, geo, work, n_steps, s, J, grad, err);
    if (!use_scratch) (void)hipFree(work);
    return e;
}

}  // namespace ifd
