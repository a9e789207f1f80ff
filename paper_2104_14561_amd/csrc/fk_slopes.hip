// fk_slopes.hip -- the slope pass (F^n of Eq. (e36)), its transpose, and their
// launchers.
#include "fk_device.h"

namespace fk {
namespace {

// Decoding of a region item: nodes of the instance's reachable box numbered
// along the box from the item's start.  The start is uniform (scalar unit), a
// lane's offset takes reciprocal multiplications.
template <int D> struct BoxItem {
    int ll, lm, row0, in0, pl0, mid0;
    bool small;
    unsigned long long rl, rm;
    __device__ BoxItem(const DevInst &I, int first)
    {
        ll = I.blen[D - 1];
        lm = D == 3 ? I.blen[1] : 1;
        row0 = D == 1 ? 0 : first / ll;
        in0 = D == 1 ? first : first - row0 * ll;
        pl0 = D == 3 ? row0 / lm : 0;
        mid0 = D == 3 ? row0 - pl0 * lm : 0;
        small = ll < (1 << 14) && lm < (1 << 14);   // fast_div's range
        rl = fast_recip(ll);
        rm = fast_recip(lm);
    }
    __device__ void index(const DevInst &I, int o, int *idx) const
    {
        const int e = in0 + o;
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
    }
};

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
// three divisions per axis, 23 us now; the FP32 part of the 64-instance batch
// 31 us, now 20 us with u in the L2 and 24 without.
//
// Several columns (Algorithm 1) in one launch: column c = blockIdx.y, its field
// at u + c * ustride, its records at packed + c * pstride.
template <typename T, int D, bool TW>
__global__ void __launch_bounds__(kBlock) k_slopes(PlanDev P, int n, int first, int count,
                                                   const T *__restrict__ u,
                                                   T *__restrict__ packed,
                                                   long long ustride, long long pstride)
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
        const T *ui = u + blockIdx.y * ustride + I.node_off;
        R *rec = reinterpret_cast<R *>(packed + blockIdx.y * pstride) + I.node_off;
        const BoxItem<D> box(I, it.first);
        auto at = [&](int o) {
            int idx[3] = {0, 0, 0};
            box.index(I, o, idx);
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
        if (it.count == 2 * kBlock) {
            // the two nodes of a thread side by side, for the loads in flight
#pragma unroll
            for (int k = 0; k < 2; ++k) at(k * kBlock + (int)threadIdx.x);
        } else {
            for (int o = threadIdx.x; o < it.count; o += kBlock) at(o);
        }
    }
}

// The step's last pass of the transpose over the region items: from mu (per
// node the cotangents of u and of the slopes) the cotangent of u,
//   lam[m] = mu_u[m] + sum_a (J_a(u)^T mu_a)[m],
// gathered: node m along axis a belongs to the slope stencils centred at m - 1,
// m and m + 1 (an end node's slope to its inner neighbour's stencil).  Exit
// nodes and images get 0, a node with images their cotangents too.
//
// Bound: one read of mu and u and one write of lam (24 bytes per node in FP32,
// 3D) and the nine slope derivatives of a node.  It was three launches (value,
// scatter with nine atomic adds per node, fold) which also cleared mu for the
// next step; the gather of the tiles now stores instead of adding.  129^3 in
// FP32: 75 us in three launches, 42 now, the gather 41 and 30 us; the FP32 part
// of the 64-instance batch 49 and 18.5 us.
template <typename T, int D>
__global__ void __launch_bounds__(kBlock) k_slopes_T(PlanDev P, int first, int count,
                                                     const T *__restrict__ u,
                                                     const T *__restrict__ mu,
                                                     T *__restrict__ lam)
{
    constexpr int PS = RecStride<D>::value;
    using R = typename RecT<T, PS>::type;
    const WorkRange wr = work_range(first, count);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = P.slope_work[w];
        const DevInst &I = P.inst[it.inst];
        const T *ui = u + I.node_off;
        const T *mi = mu + I.node_off * PS;
        const BoxItem<D> box(I, it.first);
        for (int o = threadIdx.x; o < it.count; o += kBlock) {
            int idx[3] = {0, 0, 0}, st[3];
            box.index(I, o, idx);
            int node = 0, img = 0;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                st[a] = a == D - 1 ? 1 : (int)I.stride[a];
                node += idx[a] * st[a];
                if (I.periodic[a] && idx[a] == 0) img |= 1 << a;
            }
            if (P.chi[I.node_off + node] != 0) {
                lam[I.node_off + node] = T(0);
                continue;
            }
            // field f of node j's images along the axes of mask
            auto images = [&](int j, int mask, int f) {
                T s = T(0);
                for (int k = 1; k < (1 << D); ++k) {
                    if ((k & ~mask) != 0) continue;
                    int jj = j;
                    for (int a = 0; a < D; ++a)
                        if (k & (1 << a)) jj += (I.n[a] - 1) * st[a];
                    s += mi[(long long)jj * PS + f];
                }
                return s;
            };
            const R rc = reinterpret_cast<const R *>(mi)[node];
            T acc = rc.x;
            if (img != 0) acc += images(node, img, 0);
            const T uc = ui[node];
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const int na = I.n[a], i = idx[a], base = node - i * st[a];
                const bool per = I.periodic[a] != 0;
                const int mask = img & ~(1 << a);
                // node at distance k along the axis (clamped: without weight there)
                auto pos = [&](int k) {
                    int p = i + k;
                    if (per) p = p < 0 ? p + na - 1 : (p >= na - 1 ? p - (na - 1) : p);
                    else p = min(max(p, 0), na - 1);
                    return p;
                };
                const int p0 = pos(-1), p2 = pos(1);
                const T um2 = ui[base + pos(-2) * st[a]], um1 = ui[base + p0 * st[a]];
                const T up1 = ui[base + p2 * st[a]], up2 = ui[base + pos(2) * st[a]];
                const bool in0 = per || i >= 2, in1 = per || (i >= 1 && i <= na - 2), in2 = per || i <= na - 3;
                T own = rc.y;
                if constexpr (PS == 4) own = a == 0 ? rc.y : (a == 1 ? rc.z : rc.w);
                const T *ma = mi + 1 + a;
                T m0 = ma[(long long)(base + p0 * st[a]) * PS], m1 = own;
                T m2 = ma[(long long)(base + p2 * st[a]) * PS];
                // near an end the stencils centred here also serve the end node (or
                // the image of node 0), and images along other axes count
                if (mask != 0 || (per ? i <= 1 || i >= na - 2 : i <= 2 || i >= na - 3)) {
                    auto more = [&](int p, int own_node) {
                        T m = T(0);
                        if (mask != 0) m += images(own_node, mask, 1 + a);
                        auto end = [&](int q) {
                            const int j = base + q * st[a];
                            m += ma[(long long)j * PS];
                            if (mask != 0) m += images(j, mask, 1 + a);
                        };
                        if (per) {
                            if (p == 0) end(na - 1);
                        } else {
                            if (p == 1) end(0);
                            if (p == na - 2) end(na - 1);
                        }
                        return m;
                    };
                    m0 += more(p0, base + p0 * st[a]);
                    m1 += more(i, node);
                    m2 += more(p2, base + p2 * st[a]);
                }
                m0 = in0 ? m0 : T(0);
                m1 = in1 ? m1 : T(0);
                m2 = in2 ? m2 : T(0);
                // inverse spacings of the cells m - 2 .. m + 1
                T r0, r1, r2, r3;
                if (I.affine[a]) {
                    r0 = r1 = r2 = r3 = (T)I.inv_h[a];
                } else {
                    const double *x = P.coords + I.coord_off[a];
                    auto inv = [&](int p) { return T(1) / (T)(x[p + 1] - x[p]); };
                    auto cell = [&](int k) {
                        int p = i + k;
                        if (per) p = p < 0 ? p + na - 1 : (p >= na - 1 ? p - (na - 1) : p);
                        return min(max(p, 0), na - 2);
                    };
                    r0 = inv(cell(-2));
                    r1 = inv(cell(-1));
                    r2 = inv(cell(0));
                    r3 = inv(cell(1));
                }
                // m dF/d(left difference) / h_l and m dF/d(right difference) / h_r;
                // 0 where a divided difference vanishes, including differences that
                // are rounding noise of a flat stretch (below 2^-30 of the values; in
                // FP32 that is exact equality)
                auto part = [&](T vl, T vc, T vr, T rl, T rr, T m, T &cl, T &cr) {
                    constexpr T tau = T(0x1p-30);
                    constexpr T tiny = sizeof(T) == 8 ? T(0x1p-1000) : T(0x1p-110f);
                    const T el = vc - vl, er = vr - vc;
                    const T dl = el * rl, dr = er * rr;
                    bool ok = m != T(0) && dl * dr > T(0);
                    if constexpr (sizeof(T) == 8)
                        ok = ok && fabs(el) > tau * (fabs(vc) + fabs(vl)) && fabs(er) > tau * (fabs(vr) + fabs(vc));
                    // as 2 dr^2 / (dl + dr)^2: squares that underflow (a front's far
                    // tail) count as the quotient of what is left of them
                    const T den = (dl + dr) * (dl + dr);
                    const T inv = T(1) / den;
                    T gl = T(2) * dr * dr * inv, gr = T(2) * dl * dl * inv;
                    if (ok && den < tiny) {
                        gl = T(2) * dr * dr / den;
                        gr = T(2) * dl * dl / den;
                    }
                    cl = ok ? gl * (m * rl) : T(0);
                    cr = ok ? gr * (m * rr) : T(0);
                };
                T cl, cr;
                part(um2, um1, uc, r0, r1, m0, cl, cr);
                acc += cr;
                part(um1, uc, up1, r1, r2, m1, cl, cr);
                acc += cl - cr;
                part(uc, up1, up2, r2, r3, m2, cl, cr);
                acc -= cl;
            }
            lam[I.node_off + node] = acc;
        }
    }
}

// mu <- 0 over the region items (plans whose tiles do not all pass the gather).
template <typename T, int D>
__global__ void __launch_bounds__(kBlock) k_mu_clear(PlanDev P, int first, int count, T *__restrict__ mu)
{
    constexpr int PS = RecStride<D>::value;
    using R = typename RecT<T, PS>::type;
    const WorkRange wr = work_range(first, count);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = P.slope_work[w];
        const DevInst &I = P.inst[it.inst];
        R *mr = reinterpret_cast<R *>(mu) + I.node_off;
        const BoxItem<D> box(I, it.first);
        for (int o = threadIdx.x; o < it.count; o += kBlock) {
            int idx[3] = {0, 0, 0};
            box.index(I, o, idx);
            int node = 0;
#pragma unroll
            for (int a = 0; a < D; ++a) node += idx[a] * (a == D - 1 ? 1 : (int)I.stride[a]);
            R z;
            z.x = z.y = T(0);
            if constexpr (PS == 4) z.z = z.w = T(0);
            mr[node] = z;
        }
    }
}

}  // namespace

hipError_t launch_adjoint_slopes_T(const PlanDev &P, bool f32, const void *u, void *mu,
                                   void *lam_next, hipStream_t s)
{
    // every node that an adjoint step can touch lies in the reachable boxes
    // (the active region widened by the reach and the slope stencil)
    const int first = P.n_table_work, count = P.n_slope_work - P.n_table_work;
    if (count <= 0) return hipSuccess;
    FK_DISPATCH_D(P.d,
        if (f32) {
            k_slopes_T<float, D><<<P.slope_grid, kBlock, 0, s>>>(P, first, count, (const float *)u, (const float *)mu, (float *)lam_next);
            if (!P.adj.fresh) k_mu_clear<float, D><<<P.slope_grid, kBlock, 0, s>>>(P, first, count, (float *)mu);
        } else {
            k_slopes_T<double, D><<<P.slope_grid, kBlock, 0, s>>>(P, first, count, (const double *)u, (const double *)mu, (double *)lam_next);
            if (!P.adj.fresh) k_mu_clear<double, D><<<P.slope_grid, kBlock, 0, s>>>(P, first, count, (double *)mu);
        });
    return hipGetLastError();
}

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
        if (f32) k_slopes<float, D, TW_><<<P.slope_grid, kBlock, 0, s>>>(P, n, 0, P.n_slope_work, (const float *)u, (float *)packed, 0, 0); \
        else k_slopes<double, D, TW_><<<P.slope_grid, kBlock, 0, s>>>(P, n, 0, P.n_slope_work, (const double *)u, (double *)packed, 0, 0))
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
        k_slopes<double, D, false><<<g, kBlock, 0, s>>>(P, n, 0, P.n_table_work, nullptr, nullptr, 0, 0));
    return hipGetLastError();
}

hipError_t launch_slopes_mc(const PlanDev &P, bool f32, int n, const void *u, long long ustride,
                            void *packed, long long pstride, int nc, hipStream_t s)
{
    const int first = P.n_table_work, count = P.n_slope_work - P.n_table_work;
    if (count <= 0) return hipSuccess;
    const dim3 g(P.slope_grid, nc);
    FK_DISPATCH_D(P.d,
        if (f32) k_slopes<float, D, false><<<g, kBlock, 0, s>>>(P, n, first, count, (const float *)u, (float *)packed, ustride, pstride);
        else k_slopes<double, D, false><<<g, kBlock, 0, s>>>(P, n, first, count, (const double *)u, (double *)packed, ustride, pstride));
    return hipGetLastError();
}

}  // namespace fk
