// step_block.hip -- one launch per IFDLBM time step (arXiv:2306.07603,
// Section 4, Steps (2)-(6)) in FP64 arithmetic: workgroups of four wavefronts
// that march up the rows of a strip four at a time.
//
// Work item: output columns [i0, i1) and rows [j0, j1) of one cavity, at most
// kStripOut columns; the 64 lanes of every wavefront hold columns i0 - 4 ..
// i0 + 59, and wavefront w the rows j0 - 4 + 4 n + w.  Chunk n of the march:
//   A  each wavefront's row: moments, lambda (Step 2, stored), f-bar+
//      (Eq. 2.16) into an LDS ring of the last eight rows, f-hat+ (Eq. 2.15)
//      kept in registers; the next chunk's row is fetched
//   B  two rows lower: f-bar(t + dt/2) by Eq. (3.7), walls by extrapolation,
//      f(t + dt/2) by Eq. (2.17) into a second ring
//   C  four rows lower, the row whose f-hat+ the wavefront kept one chunk ago:
//      f-hat(t + dt) by Eq. (3.6), walls (Step 6), store, residual sums
// with a barrier after A and after B.  The rings of the one-wavefront march of
// step_fused.hip live in registers, which in FP64 takes 430 of them, one
// wavefront per SIMD and a third of the instructions in register moves; here
// they are in LDS (70 KiB), two workgroups share a CU and two wavefronts a SIMD.
// Microseconds per FP64 step, that march against this one (each at its segment
// length): 64 x 513^2 946 / 925, 200 x 257^2 794 / 776, 16 x 513^2 290 / 260,
// one 1025^2 93 / 62; against the tiles where those were chosen before,
// 13 x 257^2 64 / 56, 4 x 513^2 70 / 62.  Not bound by one thing (counters, 64
// x 513^2 and the 256-cavity batch alike): vector instructions, 580 per row and
// wavefront, are issued at 35 .. 37 % of the peak rate (FP64 ones, at the 5.2
// cycles they were measured to take, for 45 .. 49 % of the time), and the two
// wavefronts of a SIMD spend 51 % of their time waiting, 3 % of it for LDS
// issue: for the loads of a chunk and at its two barriers.  The residual
// variants hold nine more values from chunk to chunk and spill 73 to 87
// registers (13 x 257^2 with residual sums 72.5 us, without 56.0).
#include "ifdlbm_internal.h"
#include "step_common.h"

namespace ifd {
namespace {

constexpr int kWaves = 4;         // wavefronts of a workgroup, rows of a chunk
constexpr int kRing = kWaves + 4;   // ring rows

// Workgroup barrier that orders LDS only: the loads of the next rows stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct BlockLds {
    double bar[kRing][9][kWaveLanes];    // f-bar+
    double half[kRing][8][kWaveLanes];   // f(t + dt/2), populations 1 .. 8
};

// The xi neighbours of a lane: byte offsets in a row of one population.  The upwind side of a population follows the
// sign of its xi-velocity a_j d_k, d_k = c_kx - c_ky s_i (Eqs. 3.2-3.8.2), opposite for the members of the pairs
// (2, 4), (5, 7) and (6, 8): the first member reads a1 (one behind), a2 (two behind) and f1 (one ahead), the second
// f1, f2 and a1.
template <typename T>
struct XiColumn {
    static constexpr uint32_t E = sizeof(T);
    uint32_t own;
    uint32_t a1[3], f1[3], a2[3], f2[3];
    T ad[3];                                  // |d|
    bool edge_l, edge_r, edge_p[3], edge_m[3];
    __device__ __forceinline__ XiColumn(int column, int i, int nx, T s)
        : own((uint32_t)column * E), edge_l(i == 1), edge_r(i == nx - 2)
    {
        const T d[3] = {-s, T(1) - s, T(-1) - s};   // d of k = 2, 5, 6
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const bool pos = d[c] >= T(0);
            const uint32_t u = pos ? 0u - E : E;
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

// Transport of one node of a ring row (the transport of step_fused.hip); rows: LDS byte offsets of population 1 of the
// rows two below .. two above.  EDGE: the node may be next to a wall (low / high: bottom / lid).
template <bool EDGE, typename T, typename Base>
__device__ __forceinline__ void ring_transport(const char* lds, const uint32_t (&rows)[5], bool low, bool high,
                                               const XiColumn<T>& v, const MixedWeights<T>& mx, const MixedWeights<T>& my,
                                               Base base, T (&out)[9])
{
    constexpr uint32_t E = sizeof(T), P = kWaveLanes * E;
    uint32_t y[5], a1[3], f1[3], a2[3], f2[3];
#pragma unroll
    for (int q = 0; q < 5; ++q) y[q] = rows[q] + v.own;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a1[c] = rows[2] + v.a1[c];
        f1[c] = rows[2] + v.f1[c];
        a2[c] = rows[2] + v.a2[c];
        f2[c] = rows[2] + v.f2[c];
    }
    const uint32_t x0 = y[2] - 2 * E;
#pragma unroll
    for (int k = 1; k < 9; ++k) {
        auto at = [&](uint32_t off) { return *reinterpret_cast<const T*>(lds + off + (uint32_t)(k - 1) * P); };
        const T c0 = at(y[2]);
        T b1, b2, h1, w;
        bool edge;
        if (k == 1 || k == 3) {
            const int u = k == 1 ? -1 : 1;
            b1 = at(x0 + (2 + u) * E);
            b2 = at(x0 + (2 + 2 * u) * E);
            h1 = at(x0 + (2 - u) * E);
            w = T(1);
            edge = k == 1 ? v.edge_l : v.edge_r;
        } else {
            const int pr = (k == 2 || k == 4) ? 0 : ((k == 5 || k == 7) ? 1 : 2);
            const bool first = k == 2 || k == 5 || k == 6;
            b1 = at(first ? a1[pr] : f1[pr]);
            b2 = at(first ? a2[pr] : f2[pr]);
            h1 = at(first ? f1[pr] : a1[pr]);
            w = v.ad[pr];
            edge = first ? v.edge_p[pr] : v.edge_m[pr];
        }
        T r = xi_term(base(k, c0), w, mx, b2, b1, c0, h1, EDGE && edge);
        if (cyk(k) > 0) r = eta_term(r, my, at(y[0]), at(y[1]), c0, at(y[3]), EDGE && low);
        if (cyk(k) < 0) r = eta_term(r, my, at(y[4]), at(y[3]), c0, at(y[1]), EDGE && high);
        out[k] = r;
    }
}

template <int PREC, bool RES, bool IMPL>
__global__ __launch_bounds__(kWaves* kWaveLanes, 2) void k_block(StepArgs a, const StripItem* items, int w0)
{
    using S = Storage<PREC>;
    using T = typename S::T;
    using V = typename S::V;
    using F = typename S::F;
    using L = typename S::L;
    static_assert(sizeof(T) == 8 && !S::kExactFinal, "FP64 arithmetic: the FP32 modes take the march of step_fused.hip");
    constexpr int R = kWaves, D = kRing, W = kWaveLanes;
    constexpr uint32_t E = sizeof(T);
    __shared__ BlockLds sh;
    const StripItem it = items[w0 + (int)blockIdx.x];
    if (it.unit < 0) return;   // padding of a per-XCD queue
    const CavityDesc c = a.desc[it.cav];
    const int nx = c.nx, ny = c.ny, pitch = c.pitch;
    const int lane = threadIdx.x % W, w = __builtin_amdgcn_readfirstlane(threadIdx.x / W);
    const int i = it.i0 - kHaloCols + lane;
    const int ic = min(max(i, 0), nx - 1), ci = min(max(i, 1), nx - 2);
    const F* f = static_cast<const F*>(a.f_in) + c.f_off;
    F* fo = static_cast<F*>(a.f_out) + c.f_off;
    const L* l = static_cast<const L*>(a.l_in) + c.l_off;
    L* lo = static_cast<L*>(a.l_out) + c.l_off;
    const int64_t plane = c.plane;
    const T* geo = a.geo + c.geo_off;
    const PowerLaw<V> pl(c);
    const T dt = T(c.dt), eps = T(c.mix), ulid = T(c.u_lid);
    const T sx = dt * T(c.inv2dxi), sx_b = T(0.5) * dt * T(c.inv2dxi);
    const MixedWeights<T> my_b(eps, T(0.5) * dt * T(c.inv2deta)), my_c(eps, dt * T(c.inv2deta));
    const XiColumn<T> v(ci - i + lane, ci, nx, geo[ny + ci]);
    const bool b_col = i >= max(it.i0 - 2, 0) && i < min(it.i1 + 2, nx);
    const bool out_col = i >= it.i0 && i < it.i1;
    const bool side = i <= 0 || i >= nx - 1;
    const bool walls = it.i0 == 0 || it.i1 == nx, edge_x = it.i0 <= 3 || it.i1 >= nx - 3;
    const uint32_t skey = S::kStochastic ? step_key(a.seed_ctr[0], a.step) : 0u, ckey = S::kStochastic ? cavity_key(it.cav) : 0u;
    double acc[kPartials];
#pragma unroll
    for (int q = 0; q < kPartials; ++q) acc[q] = 0.0;
    double ref[2] = {0.0, 0.0};
    if (RES) {
        ref[0] = a.res_ref[2 * it.cav];
        ref[1] = a.res_ref[2 * it.cav + 1];
    }
    const int t0 = it.j0 - 4;
    const int a_lo = max(t0, 0), a_hi = min(it.j1 + 3, ny - 1);          // rows of stage A
    const int b_lo = max(it.j0 - 2, 0), b_hi = min(it.j1 + 1, ny - 1);   // rows of stage B
    const int c_lo = max(it.j0, 1), c_hi = min(it.j1 - 1, ny - 2);       // interior output rows
    const int chunks = (it.j1 - it.j0 + 8 + R - 1) / R;
    // stage B takes this chunk's row where the two above it are there, else the last chunk's; stage C the last chunk's
    const bool b_now = w <= R - 3;
    const char* lds_bar = reinterpret_cast<const char*>(&sh.bar[0][1][0]);
    const char* lds_half = reinterpret_cast<const char*>(&sh.half[0][0][0]);
    auto slot_of = [&](int r) { return (uint32_t)(r - t0 + 2 * D) % (uint32_t)D; };

    F raw[9];
    L lraw;
    auto fetch = [&](int row) {
        const uint32_t id = (uint32_t)(min(max(row, a_lo), a_hi) * pitch + ic);
#pragma unroll
        for (int k = 0; k < 9; ++k) raw[k] = plane_at(f + k * plane, id);
        lraw = plane_at(l, id);
    };
    fetch(t0 + w);
    T hc[9], gc[9];        // f-hat+ and the stored g of the previous chunk's row
    V lc = V(1);
#pragma unroll
    for (int k = 0; k < 9; ++k) hc[k] = gc[k] = T(0);

#pragma unroll 1
    for (int n = 0; n < chunks; ++n) {
        const int row = t0 + n * R + w;
        // ------------------------------------------------------------ A
        T g[9], hp[9];
        V lam = V(1);
#pragma unroll
        for (int k = 0; k < 9; ++k) g[k] = S::cvt(raw[k], k);
        if (row >= a_lo && row <= a_hi) {
            T bp[9];
            collide<S, IMPL>(g, V(lraw), pl, bp, hp, lam);
            const uint32_t s = slot_of(row);
#pragma unroll
            for (int k = 0; k < 9; ++k) sh.bar[s][k][lane] = bp[k];
            if (out_col && row >= it.j0 && row < it.j1) plane_at(lo, (uint32_t)(row * pitch + i)) = L(lam);
        } else {
#pragma unroll
            for (int k = 0; k < 9; ++k) hp[k] = T(0);
        }
        if (n + 1 < chunks) fetch(row + R);
        lds_barrier();
        // ------------------------------------------------------------ B
        const int q = b_now ? row : row - R;
        if (q >= b_lo && q <= b_hi) {
            const V lam_b = b_now ? lam : lc;
            auto stage_b = [&](auto edge) {
                constexpr bool EDGE = decltype(edge)::value;
                const int cq = EDGE ? min(max(q, 1), ny - 2) : q;
                uint32_t rows[5];
#pragma unroll
                for (int y = 0; y < 5; ++y) rows[y] = slot_of(cq + y - 2) * (9 * W * E);
                const MixedWeights<T> mx(eps, sx_b * geo[cq]);
                if (b_col) {
                    T fb[9], fh[9];
                    fb[0] = *reinterpret_cast<const T*>(lds_bar + rows[2] + v.own - W * E);
                    ring_transport<EDGE>(lds_bar, rows, cq == 1, cq == ny - 2, v, mx, my_b, [](int, T c0) { return c0; }, fb);
                    if (EDGE && (side || q == 0 || q == ny - 1)) extrapolate(fb, q == ny - 1 ? ulid : T(0), fb);
                    half_step(fb, lam_b, pl.dt, fh);
                    const uint32_t s = slot_of(q);
#pragma unroll
                    for (int k = 1; k < 9; ++k) sh.half[s][k - 1][lane] = fh[k];
                }
            };
            if (edge_x || q <= 1 || q >= ny - 2)
                stage_b(std::true_type{});
            else
                stage_b(std::false_type{});
        }
        lds_barrier();
        // ------------------------------------------------------------ C
        const int p = row - R;
        if (p >= c_lo && p <= c_hi) {
            auto store = [&](int r, const T(&x)[9]) {
                const uint32_t id = (uint32_t)(r * pitch + i);
                const NodeWords nw(skey, ckey, id);
#pragma unroll
                for (int k = 0; k < 9; ++k) plane_at(fo + k * plane, id) = encode_state<S>(x[k], k, &nw);
            };
            auto stage_c = [&](auto edge) {
                constexpr bool EDGE = decltype(edge)::value;
                uint32_t rows[5];
#pragma unroll
                for (int y = 0; y < 5; ++y) rows[y] = slot_of(p + y - 2) * (8 * W * E);
                const MixedWeights<T> mx(eps, sx * geo[p]);
                T gn[9];
                if (out_col && !(EDGE && side)) {
                    gn[0] = hc[0];
                    ring_transport<EDGE>(lds_half, rows, p == 1, p == ny - 2, v, mx, my_c, [&](int k, T) { return hc[k]; }, gn);
                }
                T src[9];   // extrapolation source: the inward node's value for side lanes, the lane's own elsewhere
                if constexpr (EDGE) {
#pragma unroll
                    for (int k = 0; k < 9; ++k) src[k] = gn[k];
                    if (walls) {
#pragma unroll
                        for (int k = 0; k < 9; ++k) src[k] = __shfl(gn[k], lane + ci - i, W);
                        if (side && out_col) extrapolate(src, T(0), gn);
                    }
                }
                if (out_col) {
                    store(p, gn);
                    if (RES) {
                        T old[3];
                        moments(gc, old[0], old[1], old[2]);
                        residual_add(gn, old, ref, acc);
                    }
                }
                if constexpr (EDGE) {
                    // the wall rows with the rows next to them (Eq. 1.5)
                    auto wall_row = [&](int r, T u) {
                        T x[9];
                        extrapolate(src, u, x);
                        if (out_col) {
                            store(r, x);
                            if (RES) {
                                T o[9], old[3];
#pragma unroll
                                for (int k = 0; k < 9; ++k) o[k] = S::cvt(plane_at(f + k * plane, (uint32_t)(r * pitch + i)), k);
                                moments(o, old[0], old[1], old[2]);
                                residual_add(x, old, ref, acc);
                            }
                        }
                    };
                    if (p == 1 && it.j0 == 0) wall_row(0, T(0));
                    if (p == ny - 2 && it.j1 == ny) wall_row(ny - 1, ulid);
                }
            };
            if (edge_x || p == 1 || p == ny - 2)
                stage_c(std::true_type{});
            else
                stage_c(std::false_type{});
        }
        lc = lam;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            hc[k] = hp[k];
            gc[k] = g[k];
        }
    }
    if (RES) {
        // sum of each wavefront, then of the wavefronts, in a fixed order
        __shared__ double sums[R][kPartials];
        const double ws = wave_sums(acc);
        if (lane < kPartials) sums[w][lane] = ws;
        __syncthreads();
        if (threadIdx.x < kPartials) {
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < R; ++u) s += sums[u][threadIdx.x];
            a.partial[(int64_t)it.unit * kPartials + threadIdx.x] = s;
        }
    }
}

template <int PREC, bool IMPL>
hipError_t block(const StepArgs& a, const StripItem* items, int w0, int nw, bool residual, hipStream_t s)
{
    if (nw <= 0) return hipSuccess;
    if (residual)
        hipLaunchKernelGGL((k_block<PREC, true, IMPL>), dim3(nw), dim3(kWaves * kWaveLanes), 0, s, a, items, w0);
    else
        hipLaunchKernelGGL((k_block<PREC, false, IMPL>), dim3(nw), dim3(kWaves * kWaveLanes), 0, s, a, items, w0);
    return hipGetLastError();
}

template <bool IMPL>
hipError_t block_prec(int prec, const StepArgs& a, const StripItem* items, int w0, int nw, bool residual, hipStream_t s)
{
    switch (prec) {
    case P_FP64: return block<P_FP64, IMPL>(a, items, w0, nw, residual, s);
    case P_FP32X: return block<P_FP32X, IMPL>(a, items, w0, nw, residual, s);
    case P_FP32SR: return block<P_FP32SR, IMPL>(a, items, w0, nw, residual, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_block_step(int prec, bool implicit_lambda, const StepArgs& a, const StripItem* items, int w0, int nw,
                             bool residual, hipStream_t s)
{
    return implicit_lambda ? block_prec<true>(prec, a, items, w0, nw, residual, s)
                           : block_prec<false>(prec, a, items, w0, nw, residual, s);
}

}  // namespace ifd
