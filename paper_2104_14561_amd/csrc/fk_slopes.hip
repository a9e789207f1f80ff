// fk_slopes.hip -- the slope pass (F^n of Eq. (e36)) and its launchers.
#include "fk_device.h"

namespace fk {
namespace {

// Slope pass for step n over work items [first, first + count): table items
// (kind 1 + a) fill the (sin, cos) table of axis a; region items (kind 0)
// write record[node] = (u, g_0, .., g_{d-1}) for nodes of the instance's
// reachable box [blo, blo + blen), numbered along the box.
//
// Bound: one read of u and one record write per node (20 bytes in FP32, 3D:
// 9 us for 129^3 at the 4.7 TB/s of a large copy), so the work per node is
// kept below that.  A region item's start is decoded once on the scalar unit
// and a lane's offset in it with reciprocal multiplications; spacings enter as
// inverses (one division per axis is left, of the harmonic mean); the box is
// numbered across its rows, so that rows of 129 nodes do not leave half of a
// 256-thread workgroup idle.  129^3 FP32: 57 us with a workgroup per row and
// three divisions per axis, 24 us now; the FP32 part of the 64-instance batch
// 31 us, now 22 us.
template <typename T, int D, bool TW>
__global__ void __launch_bounds__(kBlock) k_slopes(PlanDev P, int n, int first, int count,
                                                   const T *__restrict__ u,
                                                   T *__restrict__ packed)
{
    constexpr int PS = RecStride<D>::value;
    using R = typename RecT<T, PS>::type;
    const WorkRange wr = work_range(first, count);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = P.slope_work[w];
        const DevInst &I = P.inst[it.inst];
        if (it.kind > 0) {
            if ((int)threadIdx.x >= it.count) continue;
            const int a = it.kind - 1;
            const int i = it.first + threadIdx.x;
            const double arg = trig_arg(I, time_factors(P, n, it.inst), a,
                                        P.coords[I.coord_off[a] + i]);
            P.trig[I.coord_off[a] + i] = make_double2(sin(arg), cos(arg));
            continue;
        }
        const T *ui = u + I.node_off;
        R *rec = reinterpret_cast<R *>(packed) + I.node_off;
        // start of the item inside the box (uniform), then lane offsets
        const int ll = I.blen[D - 1], lm = D == 3 ? I.blen[1] : 1;
        const int row0 = D == 1 ? 0 : it.first / ll;
        const int in0 = D == 1 ? it.first : it.first - row0 * ll;
        const int pl0 = D == 3 ? row0 / lm : 0;
        const int mid0 = D == 3 ? row0 - pl0 * lm : 0;
        const bool small = ll < (1 << 14) && lm < (1 << 14);   // fast_div's range
        const unsigned long long rl = fast_recip(ll), rm = fast_recip(lm);
        auto at = [&](int o) {
            int idx[3] = {0, 0, 0};
            int e = in0 + o;
            if constexpr (D == 1) {
                idx[0] = I.blo[0] + e;
            } else {
                const int dr = small ? fast_div(e, rl) : e / ll;
                idx[D - 1] = I.blo[D - 1] + e - dr * ll;
                if constexpr (D == 2) {
                    idx[0] = I.blo[0] + row0 + dr;
                } else {
                    const int m = mid0 + dr;
                    const int dp = small ? fast_div(m, rm) : m / lm;
                    idx[1] = I.blo[1] + m - dp * lm;
                    idx[0] = I.blo[0] + pl0 + dp;
                }
            }
            int st[3];
            int node = 0;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                st[a] = a == D - 1 ? 1 : (int)I.stride[a];
                node += idx[a] * st[a];
            }
            T g[3] = {T(0), T(0), T(0)};
#pragma unroll
            for (int a = 0; a < D; ++a) {
                int il, ic, ir;
                T rl_, rr_;
                slope_stencil<T>(I, P.coords, a, idx[a], il, ic, ir, rl_, rr_);
                const int base = node - idx[a] * st[a];
                g[a] = pchip<T>(ui[base + il * st[a]], ui[base + ic * st[a]], ui[base + ir * st[a]], rl_, rr_);
            }
            R r;
            r.x = ui[node];
            r.y = g[0];
            if constexpr (PS == 4) {
                r.z = g[1];
                r.w = g[2];
                // R2 twist: the PCHIP slope along axis 1 of the axis-0 slope field in
                // 2D (the one-dimensional rule composed in increasing axis order);
                // in 3D the four twist fields in the node's second record
                if constexpr (TW && D == 2) r.w = twist_2d<T>(I, P.coords, ui, idx);
                if constexpr (TW && D == 3) {
                    T tw[4];
                    twist_3d<T>(I, P.coords, ui, idx, tw);
                    R q;
                    q.x = tw[0]; q.y = tw[1]; q.z = tw[2]; q.w = tw[3];
                    reinterpret_cast<R *>(P.packed2)[I.node_off + node] = q;
                }
            }
            rec[node] = r;
        };
        if (it.count == 4 * kBlock) {
            // the four nodes of a thread side by side, for the loads in flight
#pragma unroll
            for (int k = 0; k < 4; ++k) at(k * kBlock + (int)threadIdx.x);
        } else {
            for (int o = threadIdx.x; o < it.count; o += kBlock) at(o);
        }
    }
}

}  // namespace

hipError_t launch_slopes(const PlanDev &P, bool f32, int n, const void *u, void *packed,
                         hipStream_t s)
{
    if (P.n_slope_work == 0) return hipSuccess;
    if (P.retab && P.retab_step) {
        const hipError_t e = launch_runaway_tables(P, n, s);
        if (e != hipSuccess) return e;
    }
#define FK_SLOPES(TW_)                                                                          \
    FK_DISPATCH_D(P.d,                                                                          \
        if (f32) k_slopes<float, D, TW_><<<P.slope_grid, kBlock, 0, s>>>(P, n, 0, P.n_slope_work, (const float *)u, (float *)packed); \
        else k_slopes<double, D, TW_><<<P.slope_grid, kBlock, 0, s>>>(P, n, 0, P.n_slope_work, (const double *)u, (double *)packed))
    if (P.hermite2) {
        FK_SLOPES(true);
    } else {
        FK_SLOPES(false);
    }
#undef FK_SLOPES
    return hipGetLastError();
}

hipError_t launch_tables(const PlanDev &P, int n, hipStream_t s)
{
    if (P.retab && P.retab_step) {
        const hipError_t e = launch_runaway_tables(P, n, s);
        if (e != hipSuccess) return e;
    }
    if (P.n_table_work == 0) return hipSuccess;
    const int g = P.n_table_work >= 8 ? (P.n_table_work + 7) / 8 * 8 : P.n_table_work;
    FK_DISPATCH_D(P.d,
        k_slopes<double, D, false><<<g, kBlock, 0, s>>>(P, n, 0, P.n_table_work, nullptr, nullptr));
    return hipGetLastError();
}

}  // namespace fk
