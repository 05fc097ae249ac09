// step_tile.hip -- one launch per IFDLBM time step (arXiv:2306.07603,
// Section 4, Steps (2)-(6)) for batches too small to fill the GPU with the row
// march (step_fused.hip, step_block.hip): one node per thread.
//
// Work item: a tile of output columns [i0, i1) and rows [j0, j1) of one
// cavity, at most (LX - 8) x (LY - 8) nodes.  The workgroup holds the nodes
// i0 - 4 .. and j0 - 4 .. , LX x LY of them, NPT per thread, and carries each
// through the three stages of the step:
//   A  (all nodes)         moments, lambda (Step 2), f-bar+ (Eq. 2.16) into
//                          LDS, f-hat+ (Eq. 2.15) in registers
//   B  (outputs and 2 more f-bar(t + dt/2) by Eq. (3.7) from the LDS tile,
//       on every side)     walls by extrapolation, f(t + dt/2) by Eq. (2.17)
//                          back into the same LDS tile
//   C  (outputs)           f-hat(t + dt) by Eq. (3.6), walls by extrapolation
//                          (Step 6), store, residual sums of Eq. (2.19)
// What bounds it: for one small cavity the chain of one step, 340 vector
// instructions of a wavefront in FP32SRF and 370 in FP64 behind two dependent
// loads, with 70 % of its time spent waiting (5.2 us per step of a 33 x 33
// FP32SRF cavity and 5.7 us in FP64, against 35.0 us of the FP32 march, whose
// items are chains of at least 16 rows); on large batches the issue of vector
// instructions (shape 2 in FP32SRF: 63 % of the peak on 1025^2, 79 % on 12 x 513^2).  The halo is recomputed: a 24 x 24 tile runs stage A on
// 1.8 and stage B on 1.4 times its nodes, so past a few million nodes (in FP64
// half a million) the march with its 1.3 wins (choose_kernel in api.hip holds the measured line).
//
// Every node is rounded as the march rounds it (the same stage functions and
// the same order in the stencils), so which of the two runs never shows in
// the results.
#include "ifdlbm_internal.h"
#include "step_common.h"

namespace ifd {
namespace {

template <typename T> __device__ __forceinline__ const T* tile_geo(const StepArgs& a);
template <> __device__ __forceinline__ const double* tile_geo<double>(const StepArgs& a) { return a.geo; }
template <> __device__ __forceinline__ const float* tile_geo<float>(const StepArgs& a) { return a.geo32; }

// One node's view of the LDS tile: byte offsets of the node's neighbours in a
// plane.  The upwind side of a population follows the sign of its xi-velocity
// a_j d_k, d_k = c_kx - c_ky s_i (Eqs. 3.2-3.8.2), opposite for the members of
// the pairs (2, 4), (5, 7) and (6, 8): the first member reads a1 (one behind),
// a2 (two behind) and f1 (one ahead), the second f1, f2 and a1.
template <typename T, int LX>
struct TileView {
    static constexpr uint32_t E = sizeof(T);
    uint32_t low2;                            // two rows below the node
    uint32_t a1[3], f1[3], a2[3], f2[3];
    T ad[3];                                  // |d|
    bool edge_l, edge_r, edge_b, edge_t;      // next to the left / right wall, bottom, lid
    bool edge_p[3], edge_m[3];                // the second upwind point of the pairs leaves the grid

    __device__ __forceinline__ TileView(int node, int i, int j, int nx, int ny, T s)
        : low2((uint32_t)(node - 2 * LX) * E), edge_l(i == 1), edge_r(i == nx - 2), edge_b(j == 1), edge_t(j == ny - 2)
    {
        const T d[3] = {-s, T(1) - s, T(-1) - s};   // d of k = 2, 5, 6
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const bool pos = d[c] >= T(0);
            const uint32_t own = (uint32_t)node * E, u = pos ? 0u - E : E;
            a1[c] = own + u;
            a2[c] = own + 2u * u;
            f1[c] = own - u;
            f2[c] = own - 2u * u;
            ad[c] = pos ? d[c] : -d[c];
            edge_p[c] = pos ? edge_l : edge_r;
            edge_m[c] = pos ? edge_r : edge_l;
        }
    }
};

// out[k] = base[k] - sx a_j d_k D_xi - sy D_eta of the node of view v for the
// moving populations (the transport of step_fused.hip): mx carries sx a_j, my
// carries sy, and the values are read from the LDS tile.  EDGE: the tile
// holds nodes next to a wall; where their second upwind point leaves the grid
// the value read there (inside the tile's array) is not used.
template <bool EDGE, int LX, int N, typename T, typename Base>
__device__ __forceinline__ void tile_transport(const T (*tile)[N], const TileView<T, LX>& v, const MixedWeights<T>& mx,
                                               const MixedWeights<T>& my, Base base, T (&out)[9])
{
    constexpr uint32_t E = sizeof(T);
#pragma unroll
    for (int k = 1; k < 9; ++k) {
        auto at = [&](uint32_t off, int dx, int dy) {
            return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(&tile[k][0]) + off + (uint32_t)(dy * LX + dx) * E);
        };
        const T c0 = at(v.low2, 0, 2);
        T a1, a2, f1, w;
        bool edge;
        if (k == 1 || k == 3) {
            const int u = k == 1 ? -1 : 1;
            a1 = at(v.low2, u, 2);
            a2 = at(v.low2, 2 * u, 2);
            f1 = at(v.low2, -u, 2);
            w = T(1);
            edge = k == 1 ? v.edge_l : v.edge_r;
        } else {
            const int pr = (k == 2 || k == 4) ? 0 : ((k == 5 || k == 7) ? 1 : 2);
            const bool first = k == 2 || k == 5 || k == 6;
            a1 = at(first ? v.a1[pr] : v.f1[pr], 0, 0);
            a2 = at(first ? v.a2[pr] : v.f2[pr], 0, 0);
            f1 = at(first ? v.f1[pr] : v.a1[pr], 0, 0);
            w = v.ad[pr];
            edge = first ? v.edge_p[pr] : v.edge_m[pr];
        }
        T r = xi_term(base(k, c0), w, mx, a2, a1, c0, f1, EDGE && edge);
        if (cyk(k) > 0) r = eta_term(r, my, at(v.low2, 0, 0), at(v.low2, 0, 1), c0, at(v.low2, 0, 3), EDGE && v.edge_b);
        if (cyk(k) < 0) r = eta_term(r, my, at(v.low2, 0, 4), at(v.low2, 0, 3), c0, at(v.low2, 0, 1), EDGE && v.edge_t);
        out[k] = r;
        // FP64, the larger tiles: keep the reads of later populations from being moved up (registers, see k_tile)
        if constexpr (sizeof(T) == 8 && LX > 16)
            if (k % 2 == 0) __builtin_amdgcn_sched_barrier(0);
    }
}

// The work item of one workgroup.  EDGE: nodes of the tile's half-step region
// are on or next to a wall.
template <int PREC, bool RES, bool IMPL, bool EDGE, int LX, int LY, int NPT>
__device__ __forceinline__ void tile_item(const StepArgs& a, const StripItem& it, const CavityDesc& c,
                                          typename Storage<PREC>::T (*tile)[LX * LY], double (&acc)[kPartials])
{
    using S = Storage<PREC>;
    using T = typename S::T;
    using V = typename S::V;
    using F = typename S::F;
    using L = typename S::L;
    constexpr int N = LX * LY, RT = LY / NPT;   // NPT nodes of a thread are RT rows apart
    const int nx = c.nx, ny = c.ny, pitch = c.pitch;
    const int lx = (int)threadIdx.x % LX, ly = (int)threadIdx.x / LX;
    const int i = it.i0 - kHaloCols + lx;
    const int64_t plane = c.plane;
    const F* f = static_cast<const F*>(a.f_in) + c.f_off;
    const L* l = static_cast<const L*>(a.l_in) + c.l_off;
    const T* geo = tile_geo<T>(a) + c.geo_off;
    const int ic = min(max(i, 0), nx - 1), ci = EDGE ? min(max(i, 1), nx - 2) : ic;
    auto row = [&](int r) { return it.j0 - kHaloCols + ly + r * RT; };
    auto inner_row = [&](int r) { return EDGE ? min(max(row(r), 1), ny - 2) : min(max(row(r), 0), ny - 1); };
    // the nearest node of the grid: threads outside it compute a node that nothing reads
    auto node_id = [&](int r) { return (uint32_t)(min(max(row(r), 0), ny - 1) * pitch + ic); };

    F raw[NPT][9];
    V lam[NPT];
    T aj[NPT];
#pragma unroll
    for (int r = 0; r < NPT; ++r) {
#pragma unroll
        for (int k = 0; k < 9; ++k) raw[r][k] = plane_at(f + k * plane, node_id(r));
        lam[r] = V(plane_at(l, node_id(r)));
        aj[r] = geo[inner_row(r)];
    }
    const T si = geo[ny + ci];
    const PowerLaw<V> pl(c);
    const T dt = T(c.dt), eps = T(c.mix), ulid = T(c.u_lid);
    auto wall_of = [&](int r) { return EDGE && (i <= 0 || row(r) <= 0 || i >= nx - 1 || row(r) >= ny - 1); };
    auto in_b = [&](int r) {
        return i >= max(it.i0 - 2, 0) && i < min(it.i1 + 2, nx) && row(r) >= max(it.j0 - 2, 0) && row(r) < min(it.j1 + 2, ny);
    };
    auto out_of = [&](int r) { return i >= it.i0 && i < it.i1 && row(r) >= it.j0 && row(r) < it.j1; };
    // the inward node of a wall node, the node itself elsewhere: the difference stencils of stage B
    auto inward_node = [&](int r) { return (ly + r * RT + inner_row(r) - row(r)) * LX + lx + ci - i; };
    auto own_node = [&](int r) { return (ly + r * RT) * LX + lx; };

    // ---------------------------------------------------------------- A
    T g[NPT][9], hp[NPT][9];
#pragma unroll
    for (int r = 0; r < NPT; ++r) {
        T bp[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) g[r][k] = S::cvt(raw[r][k], k);
        V l_new;
        collide<S, IMPL>(g[r], lam[r], pl, bp, hp[r], l_new);
        lam[r] = l_new;
#pragma unroll
        for (int k = 0; k < 9; ++k) tile[k][own_node(r)] = bp[k];
        if (out_of(r)) plane_at(static_cast<L*>(a.l_out) + c.l_off, node_id(r)) = L(l_new);
    }
    __syncthreads();

    // ---------------------------------------------------------------- B
    T fh[NPT][9];
#pragma unroll
    for (int r = 0; r < NPT; ++r)
        if (in_b(r)) {
            T fb[9];
            const TileView<T, LX> v(inward_node(r), ci, inner_row(r), nx, ny, si);
            const MixedWeights<T> mx(eps, T(0.5) * dt * T(c.inv2dxi) * aj[r]), my(eps, T(0.5) * dt * T(c.inv2deta));
            fb[0] = tile[0][inward_node(r)];
            tile_transport<EDGE, LX, N>(tile, v, mx, my, [](int, T c0) { return c0; }, fb);
            if (wall_of(r)) extrapolate(fb, row(r) == ny - 1 ? ulid : T(0), fb);
            half_step(fb, lam[r], pl.dt, fh[r]);
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NPT; ++r)
        if (in_b(r)) {
#pragma unroll
            for (int k = 1; k < 9; ++k) tile[k][own_node(r)] = fh[r][k];
        }
    __syncthreads();

    // ---------------------------------------------------------------- C
    T gn[NPT][9];
    double fin[NPT][S::kExactFinal ? 9 : 1];   // exact final update (FP32SRF): the FP64 sum of each population
#pragma unroll
    for (int r = 0; r < NPT; ++r)
        if (out_of(r) && !wall_of(r)) {
            const TileView<T, LX> v(inward_node(r), ci, inner_row(r), nx, ny, si);
            const MixedWeights<T> mx(eps, dt * T(c.inv2dxi) * aj[r]), my(eps, dt * T(c.inv2deta));
            gn[r][0] = hp[r][0];
            tile_transport<EDGE, LX, N>(tile, v, mx, my, [&](int k, T) { return hp[r][k]; }, gn[r]);
            if constexpr (S::kExactFinal) {
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    fin[r][k] = (double)g[r][k] + (double)gn[r][k];
                    gn[r][k] = T(fin[r][k]);
                }
            }
        }
    if (EDGE && (it.i0 == 0 || it.j0 == 0 || it.i1 == nx || it.j1 == ny)) {
        // walls from their inward nodes, which belong to the same tile
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NPT; ++r)
            if (out_of(r) && !wall_of(r)) {
#pragma unroll
                for (int k = 0; k < 9; ++k) tile[k][own_node(r)] = gn[r][k];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NPT; ++r)
            if (out_of(r) && wall_of(r)) {
                T src[9];
#pragma unroll
                for (int k = 0; k < 9; ++k) src[k] = tile[k][inward_node(r)];
                extrapolate(src, row(r) == ny - 1 ? ulid : T(0), gn[r]);
                if constexpr (S::kExactFinal) {
#pragma unroll
                    for (int k = 0; k < 9; ++k) fin[r][k] = (double)gn[r][k];
                }
            }
    }
    F* fo = static_cast<F*>(a.f_out) + c.f_off;
    const uint32_t skey = S::kStochastic ? step_key(a.seed_ctr[0], a.step) : 0u, ckey = S::kStochastic ? cavity_key(it.cav) : 0u;
#pragma unroll
    for (int r = 0; r < NPT; ++r)
        if (out_of(r)) {
            const NodeWords nw(skey, ckey, node_id(r));
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                if constexpr (S::kExactFinal)
                    plane_at(fo + k * plane, node_id(r)) = encode_state<S>(fin[r][k], k, &nw);
                else
                    plane_at(fo + k * plane, node_id(r)) = encode_state<S>(gn[r][k], k, &nw);
            }
            if (RES) {
                T old[3];
                moments(g[r], old[0], old[1], old[2]);
                const double ref[2] = {a.res_ref[2 * it.cav], a.res_ref[2 * it.cav + 1]};
                residual_add(gn[r], old, ref, acc);
            }
        }
}

// Tiles away from the walls take a copy of the code without wall handling (vector instructions of a wavefront of 128
// nodes in FP32SRF: 918 on 1025^2, where 9 % of the tiles are at a wall, 1048 on 513^2, where 17 % are).  Four wavefronts per SIMD (128 registers) are asked for where tiles queue up on
// the CUs: in FP64 that and the fences of tile_transport took 64 x 513^2 from 1885 to 1305 us per step in shape 1.  The
// small tile of shape 0 runs one round, where more registers are faster (5.7 against 6.4 us on 33 x 33).
template <int PREC, bool RES, bool IMPL, int LX, int LY, int NPT>
__global__ __launch_bounds__(LX* LY / NPT, LX > 16 ? 4 : 1) void k_tile(StepArgs a, const StripItem* items, int w0)
{
    constexpr int NT = LX * LY / NPT;
    __shared__ typename Storage<PREC>::T tile[9][LX * LY];
    const StripItem it = items[w0 + (int)blockIdx.x];
    if (it.unit < 0) return;   // padding of a per-XCD queue
    const CavityDesc c = a.desc[it.cav];
    double acc[kPartials];
#pragma unroll
    for (int q = 0; q < kPartials; ++q) acc[q] = 0.0;
    if (it.i0 <= 3 || it.j0 <= 3 || it.i1 >= c.nx - 3 || it.j1 >= c.ny - 3)
        tile_item<PREC, RES, IMPL, true, LX, LY, NPT>(a, it, c, tile, acc);
    else
        tile_item<PREC, RES, IMPL, false, LX, LY, NPT>(a, it, c, tile, acc);
    if (RES) {
        // sum of each wavefront, then of the wavefronts, in a fixed order
        __shared__ double sums[NT / kWaveLanes][kPartials];
        const int t = threadIdx.x;
        const double ws = wave_sums(acc);
        if (t % kWaveLanes < kPartials) sums[t / kWaveLanes][t % kWaveLanes] = ws;
        __syncthreads();
        if (t < kPartials) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NT / kWaveLanes; ++w) s += sums[w][t];
            a.partial[(int64_t)it.unit * kPartials + t] = s;
        }
    }
}

template <int PREC, bool IMPL, int LX, int LY, int NPT>
hipError_t tile(const StepArgs& a, const StripItem* items, int w0, int nw, bool residual, hipStream_t s)
{
    if (nw <= 0) return hipSuccess;
    if (residual)
        hipLaunchKernelGGL((k_tile<PREC, true, IMPL, LX, LY, NPT>), dim3(nw), dim3(LX * LY / NPT), 0, s, a, items, w0);
    else
        hipLaunchKernelGGL((k_tile<PREC, false, IMPL, LX, LY, NPT>), dim3(nw), dim3(LX * LY / NPT), 0, s, a, items, w0);
    return hipGetLastError();
}

template <int PREC, bool IMPL>
hipError_t tile_shape(int shape, const StepArgs& a, const StripItem* items, int w0, int nw, bool residual, hipStream_t s)
{
    // two nodes per thread where the registers of two fit four wavefronts per SIMD: FP32 arithmetic
    constexpr int kNodes = sizeof(typename Storage<PREC>::T) == 8 ? 1 : 2;
    switch (shape) {
    case 0: return tile<PREC, IMPL, kTileCols[0] + 8, kTileRows[0] + 8, 1>(a, items, w0, nw, residual, s);
    case 1: return tile<PREC, IMPL, kTileCols[1] + 8, kTileRows[1] + 8, 1>(a, items, w0, nw, residual, s);
    case 2: return tile<PREC, IMPL, kTileCols[2] + 8, kTileRows[2] + 8, kNodes>(a, items, w0, nw, residual, s);
    }
    return hipErrorInvalidValue;
}

template <bool IMPL>
hipError_t tile_prec(int shape, int prec, const StepArgs& a, const StripItem* items, int w0, int nw, bool residual,
                     hipStream_t s)
{
    switch (prec) {
    case P_FP64: return tile_shape<P_FP64, IMPL>(shape, a, items, w0, nw, residual, s);
    case P_FP32: return tile_shape<P_FP32, IMPL>(shape, a, items, w0, nw, residual, s);
    case P_FP16DEV: return tile_shape<P_FP16DEV, IMPL>(shape, a, items, w0, nw, residual, s);
    case P_FP32X: return tile_shape<P_FP32X, IMPL>(shape, a, items, w0, nw, residual, s);
    case P_FP32SR: return tile_shape<P_FP32SR, IMPL>(shape, a, items, w0, nw, residual, s);
    case P_FP32SRF: return tile_shape<P_FP32SRF, IMPL>(shape, a, items, w0, nw, residual, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_tile_step(int shape, int prec, bool implicit_lambda, const StepArgs& a, const StripItem* items, int w0,
                            int nw, bool residual, hipStream_t s)
{
    return implicit_lambda ? tile_prec<true>(shape, prec, a, items, w0, nw, residual, s)
                           : tile_prec<false>(shape, prec, a, items, w0, nw, residual, s);
}

}  // namespace ifd
