// fk_ent.hip -- separable step in entry form: 3D plans with face kinds other
// than exit-1, node-dependent diffusion (the runaway model) or axes that are
// not affine, box region.
#include "fk_sep.h"

namespace fk {
namespace {

constexpr int kEntThreads = 64;

// Per-coordinate tables of the runaway model at step n (Section 4.3, Eq.
// (ex32d)).  Momentum: gamma p / tau, the drift's own terms, E / p,
// 1 / (tau gamma), 2 C_B / p^2, the scales of p and (without sqrt(1 - xi^2))
// xi, exp(-(p / Delta_p)^2).  Pitch: 1 - xi^2, its root, E xi.  Radius: the
// drift V, dD/dr and the scale of r, the last two without the momentum factor.
__global__ void __launch_bounds__(kBlock) k_runaway_tables(PlanDev P, int n)
{
#pragma clang fp contract(off)
    for (int i = 0; i < P.n_inst; ++i) {
        const DevInst &I = P.inst[i];
        if (!I.sdiff) continue;
        const double *p = I.coef, *tf = time_factors(P, n, i);
        const double E = tf[0], nu = tf[1], vT = tf[2], delta = tf[3];
        const double sq = sqrt(2.0 * P.dt);
        const int total = I.n[0] + I.n[1] + I.n[2];
        for (int e = blockIdx.x * kBlock + threadIdx.x; e < total; e += gridDim.x * kBlock) {
            const int a = e < I.n[0] ? 0 : (e < I.n[0] + I.n[1] ? 1 : 2);
            const int k = e - (a > 0 ? I.n[0] : 0) - (a > 1 ? I.n[1] : 0);
            const double x = coord(I, P.coords, a, k);
            double *t = P.retab + (I.coord_off[a] + k) * kReTab;
            if (a == 0) {
                const double gam = sqrt(1.0 + (delta * x) * (delta * x));
                const double y = x / gam;
                const double phi = erf(y);
                const double dphi = 2.0 / sqrt(M_PI) * exp(-y * y);
                const double psi = (phi - y * dphi) / (2.0 * y * y);
                const double dpsi = dphi - 2.0 * psi / y;
                const double k2 = nu * vT * vT;
                const double CA = k2 * psi / y;
                const double CB = 0.5 * k2 / y * (p[2] + phi - psi + 0.5 * y * y * pow(delta, 4.0));
                const double CF = 2.0 * nu * vT * psi;
                const double dCA = k2 * (dpsi * y - psi) / (y * y) / (gam * gam * gam);
                t[0] = gam * x / p[1];
                t[1] = 2.0 * CA / x + dCA - CF;
                t[2] = E / x;
                t[3] = 1.0 / (p[1] * gam);
                t[4] = 2.0 * CB / (x * x);
                t[5] = sqrt(2.0 * CA) * sq;
                t[6] = sqrt(2.0 * CB) / x * sq;
                t[7] = exp(-(x / p[8]) * (x / p[8]));
            } else if (a == 1) {
                const double om = 1.0 - x * x;
                t[0] = om;
                t[1] = sqrt(om > 0.0 ? om : 0.0);
                t[2] = E * x;
            } else {
                const double th = tanh((x - p[6]) / p[7]);
                t[0] = x > p[6] ? p[9] : 0.0;
                t[1] = 0.5 * p[10] * (1.0 - th * th) / p[7];
                t[2] = sqrt(2.0 * (0.5 * p[10] * (1.0 + th))) * sq;
            }
        }
    }
}

// Thread per node.  Per axis at most 2 Q* entries (node, V, S) in the thread's
// LDS columns, the nodes of the landing cells in the order of the GH nodes: a
// cell equal to the last one adds to its two entries, the next cell shares one
// (reflected points may repeat a node, as entries of their own).  The record
// contraction then reads the product of the entry counts, at most (2 Q*)^3 =
// 8 Q*^3, the landing points' own, and far fewer where the points of an axis
// share cells.  Exits are per axis (a box region); the lowest exiting axis
// gives a point's value, so the masses of value 1 and 0 are sums over the axis
// of (all inside below) x (out here) x (any above).
//
// Bound: latency and the evaluations (49 x 41 x 128, Q* = 4, FP32: 3.75
// wavefronts per SIMD, the plan's own number; 2000 vector instructions and 112
// record reads each).  So the innermost axis' entries stay in registers and the
// reads of a row are issued together (54 us against 72 from LDS, four at a
// time), the model's functions come from tables (183 -> 116 registers) and one
// wavefront is a workgroup: 36 us.  The points' own form took 119 us.
template <typename T, int QS>
__global__ void __launch_bounds__(64) k_step_ent3(
    const PlanDev P, int n, const DevInst *__restrict__ insts, const WorkItem *__restrict__ work,
    const int *__restrict__ nodes, const double2 *__restrict__ trig, const double *__restrict__ coords,
    const T *__restrict__ packed, T *__restrict__ u_out)
{
    constexpr int BS = kEntThreads, NE = 2 * QS;
    using R = typename RecT<T, 4>::type;
    using V2 = typename Vec2T<T>::type;
    __shared__ V2 ev[2][NE][BS];
    __shared__ unsigned short en[2][NE][BS];
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    T wsum = T(0);
#pragma unroll
    for (int q = 0; q < QS; ++q) wsum += w1[q];
    constexpr int NS = kBlock / BS;
    const int tid = threadIdx.x;
    const WorkRange wr = work_range(0, P.n_ent_work * NS);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w / NS];
        const int t = (w % NS) * BS + tid;
        if (t >= it.count) continue;
        const DevInst &I = insts[it.inst];
        const int node = nodes[it.first + t];
        int idx[3];
        split_node<3>(I, node, idx);
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const T uref = ri[node].x;
        double c[3], S[3];
        if (I.sdiff) {
            runaway_centre_tab(I, coords, P.retab, idx, P.dt, c, S);
        } else {
            node_centre<3>(I, coords, time_factors(P, n, it.inst), trig, idx, P.dt, c);
            S[0] = S[1] = S[2] = I.S;
        }
        T in[3], o1[3], o0[3];
        // the entries of axis a into LDS columns m; their number
        const auto entries = [&](int a, int m) {
            int wl = -2, k2 = 0;
            in[a] = o1[a] = o0[a] = T(0);
#pragma unroll
            for (int q = 0; q < QS; ++q) {
                const AxisEval e = eval_axis_faces(I, coords, a, c[a], ga[q], S[a]);
                const T wq = w1[q];
                if (e.ex) {
                    if (e.exv == 0.0) o0[a] += wq;
                    else o1[a] += wq;
                    continue;
                }
                in[a] += wq;
                const T s = (T)e.s, h = (T)e.h;
                T v0, v1, d0, d1;
                unit_basis<T>(s, v0, v1, d0, d1);
                V2 x0, x1;
                x0.x = wq * v0;
                x0.y = wq * h * d0;
                x1.x = wq * v1;
                x1.y = wq * h * d1;
                if (e.k == wl || e.k == wl + 1) {
                    // entries k2 - 2 and k2 - 1 hold wl and wl + 1
                    const bool same = e.k == wl;
                    V2 *p0 = &ev[m][k2 - (same ? 2 : 1)][tid];
                    V2 y0 = *p0;
                    y0.x += x0.x;
                    y0.y += x0.y;
                    *p0 = y0;
                    if (same) {
                        V2 y1 = ev[m][k2 - 1][tid];
                        y1.x += x1.x;
                        y1.y += x1.y;
                        ev[m][k2 - 1][tid] = y1;
                    } else {
                        ev[m][k2][tid] = x1;
                        en[m][k2][tid] = (unsigned short)(e.k + 1);
                        ++k2;
                    }
                } else {
                    ev[m][k2][tid] = x0;
                    en[m][k2][tid] = (unsigned short)e.k;
                    ev[m][k2 + 1][tid] = x1;
                    en[m][k2 + 1][tid] = (unsigned short)(e.k + 1);
                    k2 += 2;
                }
                wl = e.k;
            }
            return k2;
        };
        // innermost axis: entries in registers, those past the thread's last
        // repeat its first node with zero weight
        const int cin = entries(2, 0);
        V2 bin[NE];
        int kin[NE];
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const bool has = k < cin;
            bin[k] = ev[0][k][tid];
            kin[k] = en[0][k][tid];
            bin[k].x = has ? bin[k].x : T(0);
            bin[k].y = has ? bin[k].y : T(0);
            kin[k] = has ? kin[k] : (k == 0 ? 0 : kin[0]);
        }
        // the largest count of the wave
        int cmax = 0;
#pragma unroll
        for (int k = 0; k < NE; ++k) cmax += __ballot(cin > k) != 0 ? 1 : 0;
        const int n0 = entries(0, 0), c1 = entries(1, 1);
        const int c0 = cin > 0 ? n0 : 0;
        // exit masses
        const T em1 = o1[0] * wsum * wsum + in[0] * (o1[1] * wsum + in[1] * o1[2]);
        const T em0 = o0[0] * wsum * wsum + in[0] * (o0[1] * wsum + in[1] * o0[2]);
        const int st0 = (int)I.stride[0], st1 = (int)I.stride[1];
        T acc = T(0);
        for (int i = 0; i < c0; ++i) {
            const V2 e0 = ev[0][i][tid];
            const R *r0 = ri + en[0][i][tid] * st0;
            T sv = T(0), sg = T(0);
            for (int j = 0; j < c1; ++j) {
                const V2 e1 = ev[1][j][tid];
                const R *r1 = r0 + en[1][j][tid] * st1;
                R r[NE];
#pragma unroll
                for (int k = 0; k < NE; ++k)
                    if (k < cmax) r[k] = r1[kin[k]];
                T tv = T(0), t0 = T(0), t1 = T(0);
#pragma unroll
                for (int k = 0; k < NE; ++k)
                    if (k < cmax) {
                        tv = fma_t(bin[k].x, r[k].x - uref, fma_t(bin[k].y, r[k].w, tv));
                        t0 = fma_t(bin[k].x, r[k].y, t0);
                        t1 = fma_t(bin[k].x, r[k].z, t1);
                    }
                sv += e1.x * tv + e1.y * t1;
                sg += e1.x * t0;
            }
            acc += e0.x * sv + e0.y * sg;
        }
        const T v = uref + acc + em1 * (T(1) - uref) - em0 * uref;
        flag_nonfinite(P.flags, v);
        store_node<3, T>(I, idx, node, v, u_out);
    }
}

template <typename T, int QS>
hipError_t ent_launch(const PlanDev &P, int n, const void *packed, void *u_out, hipStream_t s)
{
    constexpr int BS = kEntThreads;
    k_step_ent3<T, QS><<<P.ent_grid * (kBlock / BS), BS, 0, s>>>(
        P, n, P.inst, P.ent_work, P.ent_nodes, P.trig, P.coords, (const T *)packed, (T *)u_out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_runaway_tables(const PlanDev &P, int n, hipStream_t s)
{
    if (!P.retab) return hipSuccess;
    k_runaway_tables<<<8, kBlock, 0, s>>>(P, n);
    return hipGetLastError();
}

hipError_t launch_step_ent3(const PlanDev &P, bool f32, int n, const void *packed, void *u_out, hipStream_t s)
{
#define FK_QS(v) case v: return f32 ? ent_launch<float, v>(P, n, packed, u_out, s) : ent_launch<double, v>(P, n, packed, u_out, s);
    switch (P.qs) { FK_QS(2) FK_QS(3) FK_QS(4) FK_QS(5) FK_QS(6) }
#undef FK_QS
    return hipErrorInvalidValue;
}

}  // namespace fk
