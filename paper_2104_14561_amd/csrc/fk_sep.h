// fk_sep.h -- the separable form of the step on affine axes, in two and three
// dimensions.
//
// For a node none of whose landing points can reach a ball boundary the tensor
// rule factorises: the row of A_n over the footprint [o0, o0 + L0) x
// [o1, o1 + L1) is built from per-axis vectors
//   V_a[l] = sum_q w_q (H00(s_q) [l = k_q] + H01(s_q) [l = k_q + 1])
//   S_a[l] = the same with the slope basis h H10, h H11
// (q over the GH nodes that stay inside on axis a, k_q the landing cell
// counted from the first one), so a step reads L0 L1 records instead of 4 Q*^2.
#pragma once

#include "fk_device.h"

#include <type_traits>

namespace fk {
namespace {

template <typename T> struct Vec2T;
template <> struct Vec2T<float> { using type = float2; };
template <> struct Vec2T<double> { using type = double2; };

__device__ inline float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Value and slope basis of a cell at position s, the slope basis without its
// factor h: (1 + 2s)(1-s)^2, s^2 (3 - 2s), s (1-s)^2, -s^2 (1-s).  (H00 as
// 1 - H01 would save two operations but loses the relative accuracy of a small
// weight: the far nodes of a footprint then carry the rounding of a large one.)
template <typename T>
__device__ inline void unit_basis(T s, T &v0, T &v1, T &d0, T &d1)
{
    const T om = T(1) - s;
    const T s2 = s * s, om2 = om * om;
    v0 = om2 * (T(1) + T(2) * s);
    v1 = s2 * (T(3) - T(2) * s);
    d0 = s * om2;
    d1 = -(om * s2);
}

// Vectors of one axis of one node into the caller's LDS column col[l * BS],
// l = -1 .. L (rows -1 and L are guards: a landing cell can be one off the
// bound by the rounding of the position, with a vanishing weight there).  The
// landing position is taken relative to the node, in cells (x_k = k step + lo
// exactly on an affine axis): t_q = b dt / h + a_q S / h.  That is three FP64
// operations per GH node where coordinates, comparisons with the neighbouring
// nodes and the subtraction from the cell's node take some twenty, and its
// rounding is relative to the few cells of the displacement instead of the
// axis' length.  Exits on a non-periodic axis are decided on the coordinate
// z = c + S a_q itself (every product rounded, as everywhere); m and x are the
// weights inside and outside (EX), summed apart: the exit mass as a difference
// from the sum of all weights would carry that sum's rounding.
template <typename T, int QS, int BS, bool EX>
__device__ inline void sep_vectors(const DevInst &I, int a, int idx, double bdt, int L,
                                   const double *__restrict__ ga, const T *__restrict__ w1,
                                   typename Vec2T<T>::type *col, int &o, T &m, T &x)
{
#pragma clang fp contract(off)
    using V2 = typename Vec2T<T>::type;
    const double sh = I.S * I.inv_h[a];
    const double bh = bdt * I.inv_h[a];
    const double f0 = floor(fma_t(ga[0], sh, bh));
    const double br = bh - f0;
    o = idx + (int)f0;
    const bool per = I.periodic[a] != 0;
    double c = 0.0, lo = 0.0, hi = 0.0;
    if constexpr (EX) {
        lo = I.lo[a];
        hi = I.hi[a];
        c = ((idx == I.n[a] - 1) ? hi : (double)idx * I.step[a] + lo) + bdt;
    }
    V2 z;
    z.x = T(0);
    z.y = T(0);
    for (int j = -1; j <= L; ++j) col[j * BS] = z;
    m = x = T(0);
#pragma unroll
    for (int q = 0; q < QS; ++q) {
        const double t = fma_t(ga[q], sh, br);
        const double fl = floor(t);
        const T s = (T)(t - fl);
        const int l = (int)fl;
        T w = w1[q];
        if constexpr (EX) {
            const double zq = c + I.S * ga[q];
            if (!per && (zq <= lo || zq >= hi)) {
                x += w;
                w = T(0);
            }
            m += w;
        }
        T v0, v1, d0, d1;
        unit_basis<T>(s, v0, v1, d0, d1);
        V2 *e = col + l * BS;
        V2 e0 = e[0], e1 = e[BS];
        e0.x = fma_t(w, v0, e0.x);
        e0.y = fma_t(w, d0, e0.y);
        e1.x = fma_t(w, v1, e1.x);
        e1.y = fma_t(w, d1, e1.y);
        e[0] = e0;
        e[BS] = e1;
    }
}

// A node's value over its inside landing points alone, one after another, on the
// coordinates of affine axes.  The separable kernels also read records without
// weight, exiting points' own among them in the grouped ones, and 0 times a value
// that is not finite is NaN: nodes whose sum is not finite are taken again so
// (retake), and depend on the records their points touch and no others (a caller's
// field may hold NaN or infinity outside the region).
template <typename T, int D, int QS, bool TW>
__device__ inline T point_value(const PlanDev &P, int n, int inst, const DevInst &I, int node,
                                const double2 *__restrict__ trig, const T *__restrict__ packed)
{
#pragma clang fp contract(off)
    using R = typename RecT<T, 4>::type;
    const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
    const R *qi = TW && D == 3 ? reinterpret_cast<const R *>(P.packed2) + I.node_off : nullptr;
    int idx[3];
    split_node<D>(I, node, idx);
    const T uref = ri[node].x;
    double b[3];
    drift<D>(I, time_factors(P, n, inst), trig, idx, b);
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    double c[3];
#pragma unroll
    for (int a = 0; a < D; ++a)
        c[a] = ((idx[a] == I.n[a] - 1) ? I.hi[a] : (double)idx[a] * I.step[a] + I.lo[a]) + b[a] * P.dt;
    const bool ball = I.region_kind == 1;
    T acc = T(0), em = T(0);
#pragma unroll 1
    for (int q = 0; q < P.n_quad; ++q) {
        int qq[3], r = q;
#pragma unroll
        for (int a = D - 1; a >= 0; --a) {
            qq[a] = r % QS;
            r /= QS;
        }
        T w = T(1);
        bool ex = false;
        double d2 = 0.0;
        int base = 0;
        Basis<T> B[3];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const AxisEval e = eval_axis_affine(I, a, c[a], ga[qq[a]]);
            w *= w1[qq[a]];
            ex = ex || e.ex;
            d2 = a == 0 ? e.dz2 : d2 + e.dz2;
            base += e.k * (a == D - 1 ? 1 : (int)I.stride[a]);
            B[a] = hermite<T>(e.s, e.h);
        }
        if (ex || (ball && d2 >= I.r2)) {
            em += w;
            continue;
        }
        // corner by corner: its records times the bases of the axes' sides
        T pt = T(0);
#pragma unroll 1
        for (int k = 0; k < (1 << D); ++k) {
            const bool c0 = (k >> (D - 1)) & 1, c1 = (k >> (D - 2)) & 1, c2 = D == 3 && (k & 1);
            const int at = base + (c0 ? (int)I.stride[0] : 0) + (c1 ? (D == 3 ? (int)I.stride[1] : 1) : 0) + (c2 ? 1 : 0);
            const T v0 = c0 ? B[0].v1 : B[0].v0, d0 = c0 ? B[0].d1 : B[0].d0;
            const T v1 = c1 ? B[1].v1 : B[1].v0, d1 = c1 ? B[1].d1 : B[1].d0;
            const R r = ri[at];
            if constexpr (D == 2) {
                pt += v1 * (v0 * (r.x - uref) + d0 * r.y) + d1 * (v0 * r.z + (TW ? d0 * r.w : T(0)));
            } else {
                const T v2 = c2 ? B[2].v1 : B[2].v0, d2_ = c2 ? B[2].d1 : B[2].d0;
                T a0 = v0 * (r.x - uref) + d0 * r.y, a1 = v0 * r.z, a2 = v0 * r.w, a12 = T(0);
                if constexpr (TW) {
                    const R t = qi[at];   // (t01, t02, t12, t012)
                    a1 += d0 * t.x;
                    a2 += d0 * t.y;
                    a12 = v0 * t.z + d0 * t.w;
                }
                pt += v2 * (v1 * a0 + d1 * a1) + d2_ * (v1 * a2 + d1 * a12);
            }
        }
        acc += w * pt;
    }
    return uref + acc + em * (T(1) - uref);
}

// The nodes of this thread whose stored value is not finite, once more.  A loop of
// its own behind the step's, which finite fields never enter: inside that loop it
// takes 4 to 30 registers and up to a wave per SIMD.  NPB threads' nodes per
// workgroup, NS workgroups to a work item, this thread's number `slot`.
template <typename T, int D, int QS, bool TW, int NPB, int NS>
__device__ inline void retake(const PlanDev &P, int n, int n_work, int slot, const DevInst *__restrict__ insts,
                              const WorkItem *__restrict__ work, const int *__restrict__ nodes,
                              const double2 *__restrict__ trig, const T *__restrict__ packed, T *u_out)
{
    const WorkRange wr = work_range(0, n_work * NS);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w / NS];
        const int t = (w % NS) * NPB + slot;
        if (t >= it.count) continue;
        const DevInst &I = insts[it.inst];
        const int node = nodes[it.first + t];
        if (isfinite((double)u_out[I.node_off + node])) continue;
        const T v = point_value<T, D, QS, TW>(P, n, it.inst, I, node, trig, packed);
        flag_nonfinite(P.flags, v);
        int idx[3];
        split_node<D>(I, node, idx);
        store_node<D, T>(I, idx, node, v, u_out);
    }
}

// Thread per node.  The axis-1 vectors move from the thread's LDS column to
// registers, the axis-0 vectors then take the column's place and are read one
// row at a time; a row is L1 records against the axis-1 vectors, its loop
// unrolled for the instance's L1 rounded up to threes (a loop that leaves
// after three records keeps only three reads in flight).  Column and row
// positions past the grid carry no weight and are clamped.  BS threads share
// a 256-node work item (128 in the wide FP64 class: its columns are 32 bytes
// per footprint node and thread, and two workgroups must fit a CU's LDS).
// TW: the R2 interpolant (the twist field in the records' fourth entry).
//
// Bound: the L1 record reads, 16 cycles of a CU per 16-byte record of a wave
// (FP64 32), L0 L1 of them per node against 4 Q*^2 in the per-point form, and
// about as much VALU issue.  64-instance batch (Q* = 8), per step: the FP32 part
// 63 us over the classes and 62 by points for the nodes near the discs and those
// of about 15 nodes on both axes (k_step_pt2), the FP64 part 109 and 29 us; a
// thread per node over the landing points took 182 and 223 us for all of them.
// From 16 nodes per axis on a footprint holds more records than the points read;
// the host draws the line where the form stops being faster.
template <typename T, int QS, int L, int BS, bool TW>
__global__ void __launch_bounds__(BS) k_step_sep2(
    const PlanDev P, int n, int n_work, const DevInst *__restrict__ insts,
    const WorkItem *__restrict__ work, const int *__restrict__ nodes,
    const double2 *__restrict__ trig, const T *__restrict__ packed, T *__restrict__ u_out)
{
    static_assert(L % 3 == 0, "rows are read in threes");
    using R = typename RecT<T, 4>::type;
    using V2 = typename Vec2T<T>::type;
    __shared__ V2 lv[L + 2][BS];
    V2 *col = &lv[1][threadIdx.x];
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    T wsum = T(0);
#pragma unroll
    for (int q = 0; q < QS; ++q) wsum += w1[q];
    // BS < 256: consecutive workgroups take the parts of a work item
    constexpr int NS = kBlock / BS;
    bool bad = false;
    const WorkRange wr = work_range(0, n_work * NS);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w / NS];
        const int t = (w % NS) * BS + (int)threadIdx.x;
        if (t >= it.count) continue;
        const DevInst &I = insts[it.inst];
        const int node = nodes[it.first + t];
        int idx[3];
        split_node<2>(I, node, idx);
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const T uref = ri[node].x;
        double b[3];
        drift<2>(I, time_factors(P, n, it.inst), trig, idx, b);
        const bool interior = it.kind == 1;   // host: no landing point can exit
        const int L0 = min(I.sep_l[0], L), L1 = min(I.sep_l[1], L);
        int o0, o1;
        T m0, m1, x0, x1, emass = T(0);
        T V1[L], S1[L];
        if (interior) sep_vectors<T, QS, BS, false>(I, 1, idx[1], b[1] * P.dt, L1, ga, w1, col, o1, m1, x1);
        else sep_vectors<T, QS, BS, true>(I, 1, idx[1], b[1] * P.dt, L1, ga, w1, col, o1, m1, x1);
        const T h0 = (T)I.step[0], h1 = (T)I.step[1];
#pragma unroll
        for (int j = 0; j < L; ++j) {
            V1[j] = T(0);
            S1[j] = T(0);
            if (j < L1) {
                const V2 e = col[j * BS];
                V1[j] = e.x;
                S1[j] = e.y * h1;
            }
        }
        if (interior) {
            sep_vectors<T, QS, BS, false>(I, 0, idx[0], b[0] * P.dt, L0, ga, w1, col, o0, m0, x0);
        } else {
            sep_vectors<T, QS, BS, true>(I, 0, idx[0], b[0] * P.dt, L0, ga, w1, col, o0, m0, x0);
            emass = x0 * wsum + m0 * x1;
        }
        const int s0 = (int)I.stride[0], n0 = I.n[0], n1 = I.n[1];
        const int per0 = I.periodic[0], per1 = I.periodic[1];
        T acc = T(0);
        // LR: columns read, L1 rounded up to threes
        auto rows = [&](auto lr) {
            constexpr int LR = decltype(lr)::value;
            auto row = [&](const R *rr, auto &&at, const V2 &e) {
                T tv = T(0), tg = T(0);
#pragma unroll
                for (int j = 0; j < LR; ++j) {
                    const R r = rr[at(j)];
                    tv += V1[j] * (r.x - uref) + S1[j] * r.z;
                    tg += V1[j] * r.y;
                    if constexpr (TW) tg += S1[j] * r.w;
                }
                acc += e.x * tv + (e.y * h0) * tg;
            };
            if (__all(o1 >= 0 && o1 + LR <= n1)) {
                // every lane's columns lie on the grid: one address per row
                const R *rc = ri + o1;
                for (int i = 0; i < L0; ++i)
                    row(rc + wrap_index(o0 + i, n0, per0) * s0, [](int j) { return j; }, col[i * BS]);
            } else {
                for (int i = 0; i < L0; ++i)
                    row(ri + wrap_index(o0 + i, n0, per0) * s0,
                        [&](int j) { return wrap_index(o1 + j, n1, per1); }, col[i * BS]);
            }
        };
        if (L > 6 || L1 > 3) rows(std::integral_constant<int, L>{});
        else rows(std::integral_constant<int, 3>{});
        const T v = uref + acc + emass * (T(1) - uref);
        bad = bad || !isfinite((double)v);
        store_node<2, T>(I, idx, node, v, u_out);
    }
    if (__builtin_expect(bad, 0)) retake<T, 2, QS, TW, BS, kBlock / BS>(P, n, n_work, threadIdx.x, insts, work, nodes, trig, packed, u_out);
}

// Q*^2 landing points by a group of GL = pow2(Q*) lanes per node, lane l taking
// the axis-1 GH node l, for the nodes that the separable form does not take (a
// landing point can reach the ball, or the footprint holds too many records).  A
// lane evaluates one landing coordinate per axis; the axis-0 ones (cell row,
// weighted bases, squared distance) are shared through LDS and walked in
// order, the lane's own column bases applied once at the end, 16 multiply-adds
// per point.  Positions are relative to the node, as above; exits are decided
// on the coordinates, a face exit as an infinite squared distance, so that one
// comparison per point remains.  An exiting point reads the node's own cell
// with no weight (a branch per point would hold back the next point's reads).
//
// A lane holds one column's data instead of Q* (a thread per node takes 108 to
// 156 VGPRs, three to four waves per SIMD).  Lanes next to each other take
// nodes next to each other, the same GH node, so that their records share
// lines (the nodes near the discs of the 64-instance batch in FP32, 57 us with a
// node's lanes side by side, 48 so; 301^2, points spread over 45 cells: 25 and 20
// us).  The same nodes a thread per node: FP32 54, FP64 52 us, here 48 and 29.
template <typename T, int QS, bool TW>
__global__ void __launch_bounds__(kBlock) k_step_pt2(
    const PlanDev P, int n, int n_work, const DevInst *__restrict__ insts,
    const WorkItem *__restrict__ work, const int *__restrict__ nodes,
    const double2 *__restrict__ trig, const T *__restrict__ packed, T *__restrict__ u_out)
{
#pragma clang fp contract(off)
    using R = typename RecT<T, 4>::type;
    constexpr int GL = QS <= 2 ? 2 : (QS <= 4 ? 4 : 8);
    constexpr int NPB = kBlock / GL;
    struct Row { T x0, x1, d0, d1; };
    constexpr int NW = kWave / GL;
    __shared__ Row rows[GL][NPB];
    __shared__ double rd2[GL][NPB];
    __shared__ int roff[GL][NPB];
    const int wl = threadIdx.x % kWave;
    const int lane = wl / NW, slot = threadIdx.x / kWave * NW + wl % NW;
    const int q = lane < QS ? lane : QS - 1;   // idle lanes repeat the last one, unweighted
    const double gq = P.gh_a[q];
    const T wq = lane < QS ? weights1<T>(P)[q] : T(0);
    bool bad = false;
    const WorkRange wr = work_range(0, n_work);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w];
        const DevInst &I = insts[it.inst];
        const bool valid = slot < it.count;
        const int node = nodes[it.first + (valid ? slot : 0)];
        int idx[3];
        split_node<2>(I, node, idx);
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const T uref = ri[node].x;
        double b[3];
        drift<2>(I, time_factors(P, n, it.inst), trig, idx, b);
        const bool interior = it.kind == 1;
        const bool ball = I.region_kind == 1;
        const double r2 = ball ? I.r2 : HUGE_VAL;
        // one landing coordinate: cell, position, squared distance (infinite: exit)
        auto axis = [&](int a, int &k, T &s, double &d2) {
            const double t = fma_t(gq, I.S * I.inv_h[a], b[a] * P.dt * I.inv_h[a]);
            int kk = idx[a] + (int)floor(t);
            if (!I.periodic[a]) kk = min(max(kk, 0), I.n[a] - 2);
            s = (T)(t - (double)(kk - idx[a]));
            if (I.periodic[a]) kk += kk < 0 ? I.n[a] - 1 : (kk > I.n[a] - 2 ? 1 - I.n[a] : 0);
            k = kk;
            d2 = 0.0;
            if (!interior) {
                const double x = (idx[a] == I.n[a] - 1) ? I.hi[a] : (double)idx[a] * I.step[a] + I.lo[a];
                const double c = x + b[a] * P.dt;
                const double z = c + I.S * gq;
                const double dz = z - I.center[a];
                d2 = ball ? dz * dz : 0.0;
                if (!I.periodic[a] && (z <= I.lo[a] || z >= I.hi[a])) d2 = HUGE_VAL;
            }
        };
        const int s0 = (int)I.stride[0];
        int k0, k1;
        T s, v0, v1, e0, e1;
        double d2;
        axis(0, k0, s, d2);
        unit_basis<T>(s, v0, v1, e0, e1);
        const T wh = wq * (T)I.step[0];
        rows[lane][slot] = {wq * v0, wq * v1, wh * e0, wh * e1};
        rd2[lane][slot] = d2;
        roff[lane][slot] = k0 * s0;
        axis(1, k1, s, d2);
        unit_basis<T>(s, v0, v1, e0, e1);
        // lanes of a node belong to one wave: its LDS writes precede its reads
        __builtin_amdgcn_wave_barrier();
        // column sums: u and the axis-0 slope (c), the axis-1 slope (g)
        T c0 = T(0), c1 = T(0), g0 = T(0), g1 = T(0), pex = T(0);
#pragma unroll 4
        for (int q0 = 0; q0 < QS; ++q0) {
            Row rw = rows[q0][slot];
            int off = roff[q0][slot] + k1;
            if (!interior) {
                const bool ex = rd2[q0][slot] + d2 >= r2;
                if (ex) {
                    pex += rw.x0 + rw.x1;
                    rw = {T(0), T(0), T(0), T(0)};
                    off = node;
                }
            }
            const R *p = ri + off;
            const R p00 = p[0], p01 = p[1], p10 = p[s0], p11 = p[s0 + 1];
            c0 = fma_t(rw.x0, p00.x - uref, c0);
            c1 = fma_t(rw.x0, p01.x - uref, c1);
            c0 = fma_t(rw.x1, p10.x - uref, c0);
            c1 = fma_t(rw.x1, p11.x - uref, c1);
            c0 = fma_t(rw.d0, p00.y, c0);
            c1 = fma_t(rw.d0, p01.y, c1);
            c0 = fma_t(rw.d1, p10.y, c0);
            c1 = fma_t(rw.d1, p11.y, c1);
            g0 = fma_t(rw.x0, p00.z, g0);
            g1 = fma_t(rw.x0, p01.z, g1);
            g0 = fma_t(rw.x1, p10.z, g0);
            g1 = fma_t(rw.x1, p11.z, g1);
            if constexpr (TW) {
                g0 = fma_t(rw.d0, p00.w, g0);
                g1 = fma_t(rw.d0, p01.w, g1);
                g0 = fma_t(rw.d1, p10.w, g0);
                g1 = fma_t(rw.d1, p11.w, g1);
            }
        }
        __builtin_amdgcn_wave_barrier();
        T acc = wq * (v0 * c0 + v1 * c1 + (T)I.step[1] * (e0 * g0 + e1 * g1));
        T emass = wq * pex;
#pragma unroll
        for (int off = kWave / 2; off >= NW; off >>= 1) {
            acc += __shfl_xor(acc, off, kWave);
            emass += __shfl_xor(emass, off, kWave);
        }
        if (!valid || lane != 0) continue;
        const T v = uref + acc + emass * (T(1) - uref);
        bad = bad || !isfinite((double)v);
        store_node<2, T>(I, idx, node, v, u_out);
    }
    if (__builtin_expect(bad, 0)) retake<T, 2, QS, TW, NPB, 1>(P, n, n_work, slot, insts, work, nodes, trig, packed, u_out);
}

// A whole backward step of a small 2D plan in one launch: a workgroup takes a
// patch of 256 / GL nodes, builds the records (u, slopes) of the patch and its
// reach in LDS from u, the (sin, cos) of its coordinates beside them, and then
// works as k_step_pt2 (GL lanes per node, lane l the axis-1 GH node l; a lane has
// one landing position per axis, taken on the coordinates), every record read
// from LDS.  Slopes of a patch's reach are computed by each
// workgroup that needs them, which costs less than the launch that would share
// them as long as the reach is a few patches.
// Bound: the chain of one workgroup (one item each) and the launch (4 us).
// 513 x 257 with a disc (28 thousand active nodes, Q* = 8) in FP32: 6.8 us against
// 5.1 + 10.5 us in two launches; 129 x 33 periodic in FP64 6.0 against 4.1 + 7.9 us.
template <typename T, int QS, bool TW>
__global__ void __launch_bounds__(kBlock) k_step_small2(
    const PlanDev P, int n, const DevInst *__restrict__ insts, const WorkItem *__restrict__ work,
    const TileBox *__restrict__ tiles, const int *__restrict__ nodes, const T *__restrict__ u_in,
    T *__restrict__ u_out)
{
#pragma clang fp contract(off)
    using R = typename RecT<T, 4>::type;
    constexpr int GL = small_lanes(QS), NPB = kBlock / GL;
    struct Row { T x0, x1, d0, d1; };
    extern __shared__ __align__(16) unsigned char smem_raw[];
    R *rec = reinterpret_cast<R *>(smem_raw);
    __shared__ Row rows[NPB][GL];
    __shared__ double rd2[NPB][GL];
    __shared__ int roff[NPB][GL];
    __shared__ double2 trig[2][kSmallPatch];
    const WorkItem it = work[blockIdx.x];
    const TileBox tb = tiles[blockIdx.x];
    const DevInst &I = insts[it.inst];
    const double *tf = time_factors(P, n, it.inst);
    const T *ui = u_in + I.node_off;
    const int e1 = tb.ext[1], cells = tb.ext[0] * e1, s0 = (int)I.stride[0];
    const unsigned long long re = fast_recip(e1);
    // the patch's coordinates on the last wave, the records on all
    const int c0 = tb.pad, c1 = tb.soff;   // first row and column of the patch
    const int tl = (int)threadIdx.x - (kBlock - 64);
    if (tl >= 0 && I.coef_kind != 0) {
        const int a = tl >= kSmallPatch ? 1 : 0, i = tl - a * kSmallPatch;
        const int k = (a ? c1 : c0) + i;
        if (a < 2 && i < kSmallPatch && tl < 2 * kSmallPatch && k < I.n[a]) {
            const double arg = trig_arg(I, tf, a, P.coords[I.coord_off[a] + k]);
            trig[a][i] = make_double2(sin(arg), cos(arg));
        }
    }
    for (int e = threadIdx.x; e < cells; e += kBlock) {
        const int r = fast_div(e, re), c = e - r * e1;
        int idx[3] = {wrap_index(tb.lo[0] + r, I.n[0], I.periodic[0]),
                      wrap_index(tb.lo[1] + c, I.n[1], I.periodic[1]), 0};
        R o;
        o.x = ui[idx[0] * s0 + idx[1]];
        T g[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            int il, ic, ir;
            T rl, rr;
            slope_stencil<T>(I, P.coords, a, idx[a], il, ic, ir, rl, rr);
            const int b = a == 0 ? idx[1] : idx[0] * s0, st = a == 0 ? s0 : 1;
            g[a] = pchip<T>(ui[b + il * st], ui[b + ic * st], ui[b + ir * st], rl, rr);
        }
        o.y = g[0];
        o.z = g[1];
        o.w = T(0);
        if constexpr (TW) o.w = twist_2d<T>(I, P.coords, ui, idx);
        rec[e] = o;
    }
    __syncthreads();
    const int lane = threadIdx.x % GL, slot = threadIdx.x / GL;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int q = lane < QS ? lane : QS - 1;   // idle lanes repeat the last one, unweighted
    const double gq = P.gh_a[q];
    const T wq = lane < QS ? weights1<T>(P)[q] : T(0);
    const bool valid = slot < it.count;
    const int node = nodes[it.first + (valid ? slot : 0)];
    int idx[3];
    split_node<2>(I, node, idx);
    const int own = (idx[0] - tb.lo[0]) * e1 + (idx[1] - tb.lo[1]);
    const T uref = rec[own].x;
    double b[2];
    if (I.coef_kind == 0) {
        b[0] = I.coef[0];
        b[1] = I.coef[1];
    } else {
        drift_2d(I, tf, trig[0][idx[0] - c0], trig[1][idx[1] - c1], b);
    }
    const bool interior = it.kind == 1;
    const bool ball = I.region_kind == 1;
    const double r2 = ball ? I.r2 : HUGE_VAL;
    // one landing coordinate: cell (unwrapped, inside the tile), position,
    // squared distance (infinite: exit)
    auto axis = [&](int a, int &k, T &s, double &d2) {
        const double x = (idx[a] == I.n[a] - 1) ? I.hi[a] : (double)idx[a] * I.step[a] + I.lo[a];
        const AxisEval e = eval_axis_affine(I, a, x + b[a] * P.dt, gq);
        int kk = e.k;
        if (I.periodic[a]) kk += kk < tb.lo[a] ? I.n[a] - 1 : (kk > tb.lo[a] + tb.ext[a] - 2 ? 1 - I.n[a] : 0);
        k = min(max(kk, tb.lo[a]), tb.lo[a] + tb.ext[a] - 2) - tb.lo[a];
        s = (T)e.s;
        d2 = e.ex ? HUGE_VAL : (ball ? e.dz2 : 0.0);
    };
    int k0, k1;
    T s, v0, v1, f0, f1;
    double d2;
    axis(0, k0, s, d2);
    unit_basis<T>(s, v0, v1, f0, f1);
    const T wh = wq * (T)I.step[0];
    rows[slot][lane] = {wq * v0, wq * v1, wh * f0, wh * f1};
    rd2[slot][lane] = d2;
    roff[slot][lane] = k0 * e1;
    axis(1, k1, s, d2);
    unit_basis<T>(s, v0, v1, f0, f1);
    // lanes of a node belong to one wave: its LDS writes precede its reads
    __builtin_amdgcn_wave_barrier();
    T a0 = T(0), a1 = T(0), g0 = T(0), g1 = T(0), pex = T(0);
#pragma unroll 4
    for (int q0 = 0; q0 < QS; ++q0) {
        Row rw = rows[slot][q0];
        const int off = roff[slot][q0] + k1;
        if (!interior && rd2[slot][q0] + d2 >= r2) {
            pex += rw.x0 + rw.x1;
            rw = {T(0), T(0), T(0), T(0)};
        }
        const R *p = rec + off;
        const R p00 = p[0], p01 = p[1], p10 = p[e1], p11 = p[e1 + 1];
        a0 = fma_t(rw.x0, p00.x - uref, a0);
        a1 = fma_t(rw.x0, p01.x - uref, a1);
        a0 = fma_t(rw.x1, p10.x - uref, a0);
        a1 = fma_t(rw.x1, p11.x - uref, a1);
        a0 = fma_t(rw.d0, p00.y, a0);
        a1 = fma_t(rw.d0, p01.y, a1);
        a0 = fma_t(rw.d1, p10.y, a0);
        a1 = fma_t(rw.d1, p11.y, a1);
        g0 = fma_t(rw.x0, p00.z, g0);
        g1 = fma_t(rw.x0, p01.z, g1);
        g0 = fma_t(rw.x1, p10.z, g0);
        g1 = fma_t(rw.x1, p11.z, g1);
        if constexpr (TW) {
            g0 = fma_t(rw.d0, p00.w, g0);
            g1 = fma_t(rw.d0, p01.w, g1);
            g0 = fma_t(rw.d1, p10.w, g0);
            g1 = fma_t(rw.d1, p11.w, g1);
        }
    }
    T acc = wq * (v0 * a0 + v1 * a1 + (T)I.step[1] * (f0 * g0 + f1 * g1));
    T emass = wq * pex;
    acc = group_sum<GL>(acc);
    emass = group_sum<GL>(emass);
    if (!valid || lane != 0) return;
    const T v = uref + acc + emass * (T(1) - uref);
    store_node<2, T>(I, idx, node, v, u_out);
    if (__builtin_expect(!isfinite((double)v), 0)) {
        // the inside points alone (see point_value); all of it anew from the wave's and
        // the workgroup's number, so that no vector register is held for it before
        int wg = blockIdx.x;
        asm volatile("" : "+s"(wg));
        const int again = (wave * kWave + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u))) / GL;
        const WorkItem jt = work[wg];
        const TileBox tc = tiles[wg];
        const DevInst &J = insts[jt.inst];
        const int nd = nodes[jt.first + again];
        int id[3];
        split_node<2>(J, nd, id);
        const T u0 = rec[(id[0] - tc.lo[0]) * tc.ext[1] + (id[1] - tc.lo[1])].x;
        double bb[2];
        if (J.coef_kind == 0) {
            bb[0] = J.coef[0];
            bb[1] = J.coef[1];
        } else {
            drift_2d(J, time_factors(P, n, jt.inst), trig[0][id[0] - tc.pad], trig[1][id[1] - tc.soff], bb);
        }
        T sum = T(0), em = T(0);
#pragma unroll 1
        for (int q = 0; q < QS * QS; ++q) {
            const int q0 = q / QS, q1 = q - q0 * QS;
            const double x = (id[1] == J.n[1] - 1) ? J.hi[1] : (double)id[1] * J.step[1] + J.lo[1];
            const AxisEval e = eval_axis_affine(J, 1, x + bb[1] * P.dt, P.gh_a[q1]);
            const Row rw = rows[again][q0];
            const T w = weights1<T>(P)[q1];
            if (e.ex || (J.region_kind == 1 && rd2[again][q0] + e.dz2 >= J.r2) || rd2[again][q0] == HUGE_VAL) {
                em += w * (rw.x0 + rw.x1);
                continue;
            }
            int k = e.k;
            if (J.periodic[1]) k += k < tc.lo[1] ? J.n[1] - 1 : (k > tc.lo[1] + tc.ext[1] - 2 ? 1 - J.n[1] : 0);
            k = min(max(k, tc.lo[1]), tc.lo[1] + tc.ext[1] - 2) - tc.lo[1];
            const Basis<T> Y = hermite<T>(e.s, e.h);
            const R *p = rec + (roff[again][q0] + k);
            T pt = T(0);
#pragma unroll 1
            for (int c = 0; c < 4; ++c) {
                const R r = p[(c & 1) + (c >> 1) * tc.ext[1]];
                const T X = c & 2 ? rw.x1 : rw.x0, Xd = c & 2 ? rw.d1 : rw.d0;
                const T Yv = c & 1 ? Y.v1 : Y.v0, Yd = c & 1 ? Y.d1 : Y.d0;
                pt += Yv * (X * (r.x - u0) + Xd * r.y) + Yd * (X * r.z + (TW ? Xd * r.w : T(0)));
            }
            sum += w * pt;
        }
        const T v1 = u0 + sum + em * (T(1) - u0);
        flag_nonfinite(P.flags, v1);
        store_node<2, T>(J, id, nd, v1, u_out);
    }
}

// The separable step in three dimensions.  The axis-2 vectors are in registers, those of
// axes 0 and 1 in two LDS columns; an (i, j) row of the footprint is L2
// records against the axis-2 vectors.  Footprints up to 4 nodes (UN) unroll
// the rows, wider ones loop over the instance's own L0 x L1.  TW: the R2
// interpolant, the nodes' twist records beside the others.
// Bound: vector issue (3170 vector instructions for a wave's four nodes per lane
// at 129^3, 42 of the 67 us below at 4 cycles each), then the record gathers.
// 129^3 ABC flow (3-node footprints, Q* = 6) in FP32: 67 us, 116 us with the
// vectors selected by cell in registers and the coordinate form of the landing
// points; 65^3 with the R2 interpolant 16 us against 457 us over the landing
// points; 65^3 in FP64 with 6 x 6 x 9 footprints 114 against 597 us.
template <typename T, int QS, int L, int BS, bool TW>
__global__ void __launch_bounds__(BS, sizeof(T) == 8 && L == 4 && TW ? 2 : 1) k_step_sep3(
    const PlanDev P, int n, int n_work, const DevInst *__restrict__ insts,
    const WorkItem *__restrict__ work, const int *__restrict__ nodes,
    const double2 *__restrict__ trig, const T *__restrict__ packed, T *__restrict__ u_out)
{
    using R = typename RecT<T, 4>::type;
    using V2 = typename Vec2T<T>::type;
    constexpr bool UN = L <= 4;
    __shared__ V2 lv[2][L + 2][BS];
    V2 *cA = &lv[0][1][threadIdx.x], *cB = &lv[1][1][threadIdx.x];
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    T wsum = T(0);
#pragma unroll
    for (int q = 0; q < QS; ++q) wsum += w1[q];
    constexpr int NS = kBlock / BS;
    bool bad = false;
    const WorkRange wr = work_range(0, n_work * NS);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w / NS];
        const int t = (w % NS) * BS + (int)threadIdx.x;
        if (t >= it.count) continue;
        const DevInst &I = insts[it.inst];
        const int node = nodes[it.first + t];
        int idx[3];
        split_node<3>(I, node, idx);
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const R *qi = TW ? reinterpret_cast<const R *>(P.packed2) + I.node_off : nullptr;
        const T uref = ri[node].x;
        double b[3];
        drift<3>(I, time_factors(P, n, it.inst), trig, idx, b);
        const bool interior = it.kind == 1;
        const int L0 = UN ? L : min(I.sep_l[0], L), L1 = UN ? L : min(I.sep_l[1], L);
        const int L2 = UN ? L : min(I.sep_l[2], L);
        int o0, o1, o2;
        T m0, m1, m2, x0, x1, x2, emass = T(0);
        T V2_[L], S2_[L];
        auto vectors = [&](int a, int La, V2 *col, int &o, T &m, T &x) {
            if (interior || I.periodic[a])
                sep_vectors<T, QS, BS, false>(I, a, idx[a], b[a] * P.dt, La, ga, w1, col, o, m, x);
            else
                sep_vectors<T, QS, BS, true>(I, a, idx[a], b[a] * P.dt, La, ga, w1, col, o, m, x);
            if (I.periodic[a]) m = wsum;
        };
        vectors(2, L2, cA, o2, m2, x2);
        const T h0 = (T)I.step[0], h1 = (T)I.step[1], h2 = (T)I.step[2];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            V2_[k] = T(0);
            S2_[k] = T(0);
            if (k < L2) {
                const V2 e = cA[k * BS];
                V2_[k] = e.x;
                S2_[k] = e.y * h2;
            }
        }
        vectors(0, L0, cA, o0, m0, x0);
        vectors(1, L1, cB, o1, m1, x1);
        if (!interior) emass = x0 * wsum * wsum + m0 * (x1 * wsum + m1 * x2);
        const int s0 = (int)I.stride[0], s1 = (int)I.stride[1];
        const int n0 = I.n[0], n1 = I.n[1], n2 = I.n[2];
        const int per0 = I.periodic[0], per1 = I.periodic[1], per2 = I.periodic[2];
        T acc = T(0);
        auto contract = [&](int o2b, auto &&at) {
            auto rows = [&](int i) {
                const V2 e0 = cA[i * BS];
                const int b0 = wrap_index(o0 + i, n0, per0) * s0 + o2b;
                T sv = T(0), sg = T(0);
                auto row = [&](int j) {
                    const V2 e1 = cB[j * BS];
                    const int bb = b0 + wrap_index(o1 + j, n1, per1) * s1;
                    T tv = T(0), t0 = T(0), t1 = T(0), t01 = T(0);
#pragma unroll
                    for (int k = 0; k < L; ++k) {
                        const R r = ri[bb + at(k)];
                        tv += V2_[k] * (r.x - uref) + S2_[k] * r.w;
                        t0 += V2_[k] * r.y;
                        t1 += V2_[k] * r.z;
                        if constexpr (TW) {
                            // (t01, t02, t12, t012): slope bases of their axis sets
                            const R g = qi[bb + at(k)];
                            t0 += S2_[k] * g.y;
                            t1 += S2_[k] * g.z;
                            t01 += V2_[k] * g.x + S2_[k] * g.w;
                        }
                    }
                    const T d1 = e1.y * h1;
                    sv += e1.x * tv + d1 * t1;
                    sg += e1.x * t0;
                    if constexpr (TW) sg += d1 * t01;
                };
                if constexpr (UN) {
#pragma unroll
                    for (int j = 0; j < L; ++j) row(j);
                } else {
                    for (int j = 0; j < L1; ++j) row(j);
                }
                acc += e0.x * sv + (e0.y * h0) * sg;
            };
            if constexpr (UN && !TW) {
#pragma unroll
                for (int i = 0; i < L; ++i) rows(i);
            } else {
                for (int i = 0; i < L0; ++i) rows(i);
            }
        };
        if (__all(o2 >= 0 && o2 + L <= n2)) contract(o2, [](int k) { return k; });
        else contract(0, [&](int k) { return wrap_index(o2 + k, n2, per2); });
        const T v = uref + acc + emass * (T(1) - uref);
        bad = bad || !isfinite((double)v);
        store_node<3, T>(I, idx, node, v, u_out);
    }
    if (__builtin_expect(bad, 0)) retake<T, 3, QS, TW, BS, kBlock / BS>(P, n, n_work, threadIdx.x, insts, work, nodes, trig, packed, u_out);
}

}  // namespace
}  // namespace fk
