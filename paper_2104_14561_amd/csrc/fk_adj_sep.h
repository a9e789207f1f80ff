// fk_adj_sep.h -- the transposed step of separable nodes (affine axes), a
// thread per node, in two and three dimensions.
//
// The transposed row of A_n over the footprint is the outer product of the
// per-axis vectors (V, S) of fk_sep.h times lam_j; it is added to the work
// item's LDS tile.  The theta-gradient needs the derivatives of
//   F = sum_box V_0 V_1 [V_2] u + (slope terms)
// with respect to each axis' landing position.  They are taken after the sums:
// F depends on axis a through A_a[l] = dF / dV_a[l] and B_a[l] = dF / dS_a[l]
// (the records contracted over the other axes), so
//   dF/dz_a = sum_q w_q (H00' A_a[k_q] + H01' A_a[k_q+1] + H10' B_a[k_q] + H11' B_a[k_q+1]),
// and the same with w_q a_q for the derivative along the GH node.  A record
// then costs 3 d - 1 multiply-adds beside the step's own instead of 3 (d + 1)
// against derivative vectors, and no such vectors are built.
#pragma once

#include "fk_sep.h"

namespace fk {
namespace {

// dF/dz and its GH-weighted counterpart on one axis from the sums (A, B) in
// the caller's LDS column (entries -1 .. L, the guards finite), the landing
// positions as in sep_vectors.
template <typename T, int QS, int BS, bool EX>
__device__ inline void sep_gradient(const DevInst &I, int a, int idx, double bdt,
                                    const double *__restrict__ ga, const T *__restrict__ w1,
                                    const typename Vec2T<T>::type *col, T &G, T &H)
{
#pragma clang fp contract(off)
    using V2 = typename Vec2T<T>::type;
    const double sh = I.S * I.inv_h[a];
    const double bh = bdt * I.inv_h[a];
    const double br = bh - floor(__builtin_fma(ga[0], sh, bh));
    const T rh = (T)I.inv_h[a];
    const bool per = I.periodic[a] != 0;
    double c = 0.0, lo = 0.0, hi = 0.0;
    if constexpr (EX) {
        lo = I.lo[a];
        hi = I.hi[a];
        c = ((idx == I.n[a] - 1) ? hi : (double)idx * I.step[a] + lo) + bdt;
    }
    G = H = T(0);
#pragma unroll
    for (int q = 0; q < QS; ++q) {
        const double t = __builtin_fma(ga[q], sh, br);
        const double fl = floor(t);
        const T s = (T)(t - fl);
        T w = w1[q];
        if constexpr (EX) {
            const double zq = c + I.S * ga[q];
            if (!per && (zq <= lo || zq >= hi)) w = T(0);
        }
        const V2 *e = col + (int)fl * BS;
        const V2 e0 = e[0], e1 = e[BS];
        const T s2 = s * s;
        const T zv = T(6) * (s - s2) * rh;                      // H01' = -H00'
        const T zd1 = T(3) * s2 - T(2) * s;
        const T zd0 = zd1 + T(1) - T(2) * s;
        const T g = w * fma_t(zv, e1.x - e0.x, fma_t(zd0, e0.y, zd1 * e1.y));
        G += g;
        H = fma_t((T)ga[q], g, H);
    }
}

// 2D.  LDS: one column of (V, S) pairs per thread, then the tile.  A row's
// (V0, S0) entry is replaced by its sums (A0, B0) once it is done; the column
// sums (A1, B1) are registers and take the column over at the end.  Entries
// past the node's footprint carry no weight: along the row they may fall on
// any later entry of the tile (the host leaves L entries behind it), outside
// the tile's rows or before its first column they are clamped.  Bound: the LDS
// adds, 8.4 cycles of a CU per wave instruction at best, about 11 here (lanes
// whose footprints start differently meet; left out, the FP32 classes of the
// batch take 10 to 16 us instead of 39 to 46).
template <typename T, int QS, int L, int BS>
__global__ void __launch_bounds__(BS) k_adjoint_sep2(
    const PlanDev P, int n, int n_work, const DevInst *__restrict__ insts,
    const WorkItem *__restrict__ work, const TileBox *__restrict__ tiles,
    const int *__restrict__ nodes, const double2 *__restrict__ trig,
    const T *__restrict__ packed, const T *__restrict__ lam, T *__restrict__ mu,
    double *__restrict__ grad)
{
    constexpr int D = 2, PS = 4;
    using R = typename RecT<T, PS>::type;
    using V2 = typename Vec2T<T>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[kBlock / 64][kThetaSlots];
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    const WorkRange wr = work_range(0, n_work);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w];
        const DevInst &I = insts[it.inst];
        const int L0 = min(I.sep_l[0], L), L1 = min(I.sep_l[1], L);
        V2 *col = reinterpret_cast<V2 *>(smem_raw) + BS + threadIdx.x;
        double *const tmem = reinterpret_cast<double *>(smem_raw) +
                             (max(L0, L1) + 2) * BS * (sizeof(V2) / 8);
        MuTile<T, D> tile;
        tile.init(tmem, tiles[w]);
        tile.clear();
        __syncthreads();
        double gth[kThetaSlots];
        for (int kk = 0; kk < kThetaSlots; ++kk) gth[kk] = 0.0;
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const double *tf = time_factors(P, n, it.inst);
        const bool interior = it.kind == 1;
        for (int t = threadIdx.x; t < it.count; t += BS) {
            const int node = nodes[it.first + t];
            const T Lm = lam[I.node_off + node];
            if (Lm == T(0)) continue;
            int idx[3];
            split_node<D>(I, node, idx);
            const T uref = ri[node].x;
            double b[3];
            drift<D>(I, tf, trig, idx, b);
            const double b0 = b[0] * P.dt, b1 = b[1] * P.dt;
            int o0, o1;
            T m, mx;
            T V1[L], S1[L], A1[L], B1[L];
            if (interior) sep_vectors<T, QS, BS, false>(I, 1, idx[1], b1, L1, ga, w1, col, o1, m, mx);
            else sep_vectors<T, QS, BS, true>(I, 1, idx[1], b1, L1, ga, w1, col, o1, m, mx);
            const T h0 = (T)I.step[0], h1 = (T)I.step[1];
#pragma unroll
            for (int j = 0; j < L; ++j) {
                V1[j] = S1[j] = A1[j] = B1[j] = T(0);
                if (j < L1) {
                    const V2 e = col[j * BS];
                    V1[j] = e.x;
                    S1[j] = e.y * h1;
                }
            }
            if (interior) sep_vectors<T, QS, BS, false>(I, 0, idx[0], b0, L0, ga, w1, col, o0, m, mx);
            else sep_vectors<T, QS, BS, true>(I, 0, idx[0], b0, L0, ga, w1, col, o0, m, mx);
            const int s0 = (int)I.stride[0], n0 = I.n[0], n1 = I.n[1];
            const int per0 = I.periodic[0], per1 = I.periodic[1];
            const int tr0 = o0 - tile.lo[0], tc0 = o1 - tile.lo[1];
            const int pitch = tile.pitch, plane = tile.plane;
            auto rows = [&](auto lr) {
                constexpr int LR = decltype(lr)::value;
                // t_first + tat(j): entry of column j in the tile's row
                auto row = [&](int i, const R *rr, auto &&at, int t_first, auto &&tat) {
                    const V2 e = col[i * BS];
                    const T v0 = e.x, q0 = e.y * h0;
                    const T lv = Lm * v0, ls = Lm * q0;
                    double *t0 = tmem + (min(max(tr0 + i, 0), tile.ext[0] - 1) * pitch + t_first);
                    double *t1 = t0 + plane, *t2 = t1 + plane;
                    T tA = T(0), tB = T(0);
#pragma unroll
                    for (int j = 0; j < LR; ++j) {
                        const R r = rr[at(j)];
                        const T u = r.x - uref;
                        tA = fma_t(V1[j], u, fma_t(S1[j], r.z, tA));
                        tB = fma_t(V1[j], r.y, tB);
                        A1[j] = fma_t(v0, u, fma_t(q0, r.y, A1[j]));
                        B1[j] = fma_t(v0, r.z, B1[j]);
                        const int e = tat(j);
                        lds_add(t0 + e, (double)(lv * V1[j]));
                        lds_add(t1 + e, (double)(ls * V1[j]));
                        lds_add(t2 + e, (double)(lv * S1[j]));
                    }
                    V2 ab;
                    ab.x = tA;
                    ab.y = tB;
                    col[i * BS] = ab;
                };
                if (__all(o1 >= 0 && o1 + LR <= n1)) {
                    const R *rc = ri + o1;
                    for (int i = 0; i < L0; ++i)
                        row(i, rc + wrap_index(o0 + i, n0, per0) * s0, [](int j) { return j; },
                            tc0, [](int j) { return j; });
                } else {
                    for (int i = 0; i < L0; ++i)
                        row(i, ri + wrap_index(o0 + i, n0, per0) * s0,
                            [&](int j) { return wrap_index(o1 + j, n1, per1); },
                            0, [&](int j) { return max(tc0 + j, 0); });
                }
            };
            if (L > 6 || L1 > 3) rows(std::integral_constant<int, L>{});
            else rows(std::integral_constant<int, 3>{});
            T Gz[3] = {T(0), T(0), T(0)}, Hz[3] = {T(0), T(0), T(0)};
            if (interior) sep_gradient<T, QS, BS, false>(I, 0, idx[0], b0, ga, w1, col, Gz[0], Hz[0]);
            else sep_gradient<T, QS, BS, true>(I, 0, idx[0], b0, ga, w1, col, Gz[0], Hz[0]);
#pragma unroll
            for (int j = 0; j < L; ++j)
                if (j < L1) {
                    V2 ab;
                    ab.x = A1[j];
                    ab.y = B1[j];
                    col[j * BS] = ab;
                }
            if (interior) sep_gradient<T, QS, BS, false>(I, 1, idx[1], b1, ga, w1, col, Gz[1], Hz[1]);
            else sep_gradient<T, QS, BS, true>(I, 1, idx[1], b1, ga, w1, col, Gz[1], Hz[1]);
            double gn[kThetaSlots];
            for (int kk = 0; kk < kThetaSlots; ++kk) gn[kk] = 0.0;
            node_theta<D, T>(P, I, tf, trig, idx, Lm, Gz, Hz, gn);
            for (int kk = 0; kk < kThetaSlots; ++kk) gth[kk] += gn[kk];
        }
        __syncthreads();
        tile.template flush<PS>(I, mu, (T *)P.adj.stage);
        reduce_theta(red, gth, grad, it.inst);
        __syncthreads();
    }
}

// Per landing point in 2D (positions relative to the node, one exit comparison
// per point: fk_sep.h).  A work item's nodes go 64 at a time, a lane per node
// and a wave per axis-1 GH node.  Each wave evaluates one axis-0 GH node of the
// 64 nodes and shares it through LDS (cell row, weighted bases and derivative
// bases, squared distance); then each walks the Q* rows against its own column.
// A lane holds one column (all of a node's columns took 100 to 180 VGPRs), the
// rows' record reads overlap, and the twelve tile entries of a point are adds
// of 64 neighbouring nodes to neighbouring entries.  (With the columns across
// the lanes instead, as in the forward step, adds of one instruction meet in
// one entry: the FP32 part of the batch took twice as long.)  The
// theta-gradient is linear in a node's sums, so that the waves' parts are added
// in the workgroup's reduction.  Per point: the row sums against the column
// (for axis 0), the column sums over the rows (for axis 1, applied once at the
// end).  Landing cells outside the tile (a tile that does not fit, a periodic
// seam) go to global memory.  Bound: the LDS adds, as above.
template <typename T, int QS>
__global__ void __launch_bounds__(64 * QS, sizeof(T) == 4 ? 6 : 2) k_adjoint_pt2(
    const PlanDev P, int n, int n_work, const DevInst *__restrict__ insts,
    const WorkItem *__restrict__ work, const TileBox *__restrict__ tiles,
    const int *__restrict__ nodes, const double2 *__restrict__ trig,
    const T *__restrict__ packed, const T *__restrict__ lam, T *__restrict__ mu,
    double *__restrict__ grad)
{
#pragma clang fp contract(off)
    constexpr int D = 2, PS = 4;
    using R = typename RecT<T, PS>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[QS][kThetaSlots];
    __shared__ R rx[QS][64], rz[QS][64];   // (x0, x1, p0, p1); (zv, zd0, zd1, -)
    __shared__ double rd[QS][64];          // squared distance (infinite: exit)
    __shared__ int rk[QS][64];             // cell row
    double *const tmem = reinterpret_cast<double *>(smem_raw);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    const double gq = ga[wave];
    const T wq = w1[wave];
    const WorkRange wr = work_range(0, n_work);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w];
        const DevInst &I = insts[it.inst];
        MuTile<T, D> tile;
        tile.init(tmem, tiles[w]);
        tile.clear();
        double gth[kThetaSlots];
        for (int kk = 0; kk < kThetaSlots; ++kk) gth[kk] = 0.0;
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const double *tf = time_factors(P, n, it.inst);
        const bool interior = it.kind == 1;
        const bool ball = I.region_kind == 1;
        const double r2 = ball ? I.r2 : HUGE_VAL;
        const int s0 = (int)I.stride[0], plane = tile.plane, pitch = tile.pitch;
        const T h0 = (T)I.step[0], h1 = (T)I.step[1], rh0 = (T)I.inv_h[0], rh1 = (T)I.inv_h[1];
        for (int base = 0; base < it.count; base += 64) {
            const bool valid = base + lane < it.count;
            const int node = nodes[it.first + (valid ? base + lane : 0)];
            const T Lm = valid ? lam[I.node_off + node] : T(0);
            int idx[3];
            split_node<D>(I, node, idx);
            const T uref = ri[node].x;
            double b[3];
            drift<D>(I, tf, trig, idx, b);
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
            int k0, k1;
            T s, v0, v1, d0, d1;
            double d2;
            axis(0, k0, s, d2);
            unit_basis<T>(s, v0, v1, d0, d1);
            {
                const T s2 = s * s, zd1 = T(3) * s2 - T(2) * s;
                R x, z;
                x.x = wq * v0;
                x.y = wq * v1;
                x.z = wq * h0 * d0;
                x.w = wq * h0 * d1;
                z.x = wq * (T(6) * (s - s2) * rh0);     // H01' = -H00'
                z.y = wq * (zd1 + T(1) - T(2) * s);
                z.z = wq * zd1;
                z.w = T(0);
                rx[wave][lane] = x;
                rz[wave][lane] = z;
                rd[wave][lane] = d2;
                rk[wave][lane] = k0;
            }
            axis(1, k1, s, d2);
            unit_basis<T>(s, v0, v1, d0, d1);
            const T y0 = wq * v0, y1 = wq * v1, f0 = wq * h1 * d0, f1 = wq * h1 * d1;
            // lam times the column's bases, for the tile
            const T ly0 = Lm * y0, ly1 = Lm * y1, lf0 = Lm * f0, lf1 = Lm * f1;
            const int tc = k1 - tile.lo[1];
            const bool cin = tile.use && tc >= 0 && tc + 1 < tile.ext[1];
            __syncthreads();   // the rows, and the cleared tile
            T c0 = T(0), c1 = T(0), g0 = T(0), g1 = T(0);   // column sums over the rows
            T G0 = T(0), H0 = T(0);
            if (Lm != T(0)) {
#pragma unroll 2
                for (int q0 = 0; q0 < QS; ++q0) {
                    if (!interior && rd[q0][lane] + d2 >= r2) continue;
                    const R x = rx[q0][lane], z = rz[q0][lane];
                    const int kr = rk[q0][lane];
                    const int off = kr * s0 + k1;
                    const R *p = ri + off;
                    const R p00 = p[0], p01 = p[1], p10 = p[s0], p11 = p[s0 + 1];
                    const T u00 = p00.x - uref, u01 = p01.x - uref, u10 = p10.x - uref, u11 = p11.x - uref;
                    const T a0 = fma_t(y0, u00, fma_t(y1, u01, fma_t(f0, p00.z, f1 * p01.z)));
                    const T a1 = fma_t(y0, u10, fma_t(y1, u11, fma_t(f0, p10.z, f1 * p11.z)));
                    const T b0 = fma_t(y0, p00.y, y1 * p01.y), b1 = fma_t(y0, p10.y, y1 * p11.y);
                    const T g = fma_t(z.x, a1 - a0, fma_t(z.y, b0, z.z * b1));
                    G0 += g;
                    H0 = fma_t((T)ga[q0], g, H0);
                    c0 = fma_t(x.x, u00, fma_t(x.y, u10, fma_t(x.z, p00.y, fma_t(x.w, p10.y, c0))));
                    c1 = fma_t(x.x, u01, fma_t(x.y, u11, fma_t(x.z, p01.y, fma_t(x.w, p11.y, c1))));
                    g0 = fma_t(x.x, p00.z, fma_t(x.y, p10.z, g0));
                    g1 = fma_t(x.x, p01.z, fma_t(x.y, p11.z, g1));
                    const int tr = kr - tile.lo[0];
                    if (cin && tr >= 0 && tr + 1 < tile.ext[0]) {
                        double *tp = tmem + (tr * pitch + tc);
                        lds_add(tp, (double)(x.x * ly0));
                        lds_add(tp + 1, (double)(x.x * ly1));
                        lds_add(tp + pitch, (double)(x.y * ly0));
                        lds_add(tp + pitch + 1, (double)(x.y * ly1));
                        tp += plane;
                        lds_add(tp, (double)(x.z * ly0));
                        lds_add(tp + 1, (double)(x.z * ly1));
                        lds_add(tp + pitch, (double)(x.w * ly0));
                        lds_add(tp + pitch + 1, (double)(x.w * ly1));
                        tp += plane;
                        lds_add(tp, (double)(x.x * lf0));
                        lds_add(tp + 1, (double)(x.x * lf1));
                        lds_add(tp + pitch, (double)(x.y * lf0));
                        lds_add(tp + pitch + 1, (double)(x.y * lf1));
                    } else {
                        T *mp = mu + (I.node_off + off) * PS;
                        const int sp = s0 * PS;
                        atomicAdd(mp, x.x * ly0);
                        atomicAdd(mp + PS, x.x * ly1);
                        atomicAdd(mp + sp, x.y * ly0);
                        atomicAdd(mp + sp + PS, x.y * ly1);
                        atomicAdd(mp + 1, x.z * ly0);
                        atomicAdd(mp + PS + 1, x.z * ly1);
                        atomicAdd(mp + sp + 1, x.w * ly0);
                        atomicAdd(mp + sp + PS + 1, x.w * ly1);
                        atomicAdd(mp + 2, x.x * lf0);
                        atomicAdd(mp + PS + 2, x.x * lf1);
                        atomicAdd(mp + sp + 2, x.y * lf0);
                        atomicAdd(mp + sp + PS + 2, x.y * lf1);
                    }
                }
                const T s2 = s * s, zd1 = T(3) * s2 - T(2) * s;
                const T zv = T(6) * (s - s2) * rh1, zd0 = zd1 + T(1) - T(2) * s;
                const T G1 = wq * fma_t(zv, c1 - c0, fma_t(zd0, g0, zd1 * g1));
                const T Gz[3] = {G0, G1, T(0)}, Hz[3] = {H0, (T)gq * G1, T(0)};
                double gn[kThetaSlots];
                for (int kk = 0; kk < kThetaSlots; ++kk) gn[kk] = 0.0;
                node_theta<D, T>(P, I, tf, trig, idx, Lm, Gz, Hz, gn);
                for (int kk = 0; kk < kThetaSlots; ++kk) gth[kk] += gn[kk];
            }
            __syncthreads();   // the rows are rewritten, or the tile is complete
        }
        tile.template flush<PS>(I, mu, (T *)P.adj.stage);
        reduce_theta(red, gth, grad, it.inst);
        __syncthreads();
    }
}

// 3D.  LDS: per thread a column of (V0, S0) pairs, replaced by (A0, B0) row by
// row, one of (V1, S1) and one of the sums (A1, B1); the axis-2 vectors and
// sums are registers.  Footprints up to 4 nodes (UN) unroll the rows and keep
// (A1, B1) in registers too; in FP32 with 3-node footprints four workgroups fit
// a CU (126 VGPRs, 40 KB).  Bound at 129^3: vector issue (1917 vector
// instructions per wave of 64 nodes, at 4 cycles 102 of the 162 us below), then
// the adds: a wave takes 4 rows of 16 nodes (8 rows of 8 met two by two on the LDS
// banks, 16.4 cycles per add).
// 129^3 ABC flow (3-node footprints) in FP32: 369 us with derivative vectors per
// axis (224 VGPRs), 208 with sums, 182 in rows of 16 and a cell's fields flushed
// together, 162 with the fourth workgroup; 65^3 in FP64 with 6 x 6 x 9 footprints
// 390 us against 47.7 ms per landing point (a tile of that reach did not fit LDS,
// and every add went to global memory).  Columns and tile leave room for one
// workgroup of 128 threads a CU there, two waves on four SIMDs with nothing to
// hide a latency behind: the vector issue alone is 106 us on the two SIMDs, the
// 27 thousand LDS instructions of a CU 95 to 124 us at 8.4 to 11 cycles.
template <typename T, int QS, int L, int BS>
__global__ void __launch_bounds__(BS, (sizeof(T) == 4 && L == 3) ? 4 : 1) k_adjoint_sep3(
    const PlanDev P, int n, int n_work, const DevInst *__restrict__ insts,
    const WorkItem *__restrict__ work, const TileBox *__restrict__ tiles,
    const int *__restrict__ nodes, const double2 *__restrict__ trig,
    const T *__restrict__ packed, const T *__restrict__ lam, T *__restrict__ mu,
    double *__restrict__ grad)
{
    constexpr int D = 3, PS = 4;
    constexpr bool UN = L <= 4;
    using R = typename RecT<T, PS>::type;
    using V2 = typename Vec2T<T>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[kBlock / 64][kThetaSlots];
    const double *ga = P.gh_a;
    const T *w1 = weights1<T>(P);
    const WorkRange wr = work_range(0, n_work);
    for (int w = wr.begin; w < wr.end; w += wr.step) {
        const WorkItem it = work[w];
        const DevInst &I = insts[it.inst];
        const int L0 = UN ? L : min(I.sep_l[0], L), L1 = UN ? L : min(I.sep_l[1], L);
        const int L2 = UN ? L : min(I.sep_l[2], L);
        // columns (guards at both ends): axis 0, axis 1, axis-1 sums; the axis-2
        // vectors and sums pass through the first and second together; unrolled,
        // the first's upper and the second's lower guard are one
        V2 *cA = reinterpret_cast<V2 *>(smem_raw) + BS + threadIdx.x;
        const int nA = max(L0, L2) + (UN ? 1 : 2), nB = L1 + 2;
        V2 *cB = cA + nA * BS, *cC = cB + nB * BS;
        double *const tmem = reinterpret_cast<double *>(smem_raw) +
                             (nA + (UN ? 1 : 2) * nB) * BS * (sizeof(V2) / 8);
        MuTile<T, D> tile;
        tile.init(tmem, tiles[w]);
        tile.clear();
        __syncthreads();
        double gth[kThetaSlots];
        for (int kk = 0; kk < kThetaSlots; ++kk) gth[kk] = 0.0;
        const R *ri = reinterpret_cast<const R *>(packed) + I.node_off;
        const double *tf = time_factors(P, n, it.inst);
        const bool interior = it.kind == 1;
        for (int t = threadIdx.x; t < it.count; t += BS) {
            const int node = nodes[it.first + t];
            const T Lm = lam[I.node_off + node];
            if (Lm == T(0)) continue;
            int idx[3];
            split_node<D>(I, node, idx);
            const T uref = ri[node].x;
            double b[3];
            drift<D>(I, tf, trig, idx, b);
            const double bd[3] = {b[0] * P.dt, b[1] * P.dt, b[2] * P.dt};
            int o0, o1, o2;
            T m, mx;
            T V2_[L], S2_[L], A2[L], B2[L];
            T A1[UN ? L : 1], B1[UN ? L : 1];
            auto vectors = [&](int a, int La, V2 *col, int &o) {
                if (interior || I.periodic[a])
                    sep_vectors<T, QS, BS, false>(I, a, idx[a], bd[a], La, ga, w1, col, o, m, mx);
                else
                    sep_vectors<T, QS, BS, true>(I, a, idx[a], bd[a], La, ga, w1, col, o, m, mx);
            };
            auto gradient = [&](int a, const V2 *col, T &G, T &H) {
                if (interior || I.periodic[a])
                    sep_gradient<T, QS, BS, false>(I, a, idx[a], bd[a], ga, w1, col, G, H);
                else
                    sep_gradient<T, QS, BS, true>(I, a, idx[a], bd[a], ga, w1, col, G, H);
            };
            vectors(2, L2, cA, o2);
            const T h0 = (T)I.step[0], h1 = (T)I.step[1], h2 = (T)I.step[2];
#pragma unroll
            for (int k = 0; k < L; ++k) {
                V2_[k] = S2_[k] = A2[k] = B2[k] = T(0);
                if (k < L2) {
                    const V2 e = cA[k * BS];
                    V2_[k] = e.x;
                    S2_[k] = e.y * h2;
                }
            }
            vectors(0, L0, cA, o0);
            vectors(1, L1, cB, o1);
            V2 z;
            z.x = z.y = T(0);
            if constexpr (UN) {
#pragma unroll
                for (int j = 0; j < L; ++j) A1[j] = B1[j] = T(0);
            } else {
                for (int j = -1; j <= L1; ++j) cC[j * BS] = z;
            }
            const int s0 = (int)I.stride[0], s1 = (int)I.stride[1];
            const int n0 = I.n[0], n1 = I.n[1], n2 = I.n[2];
            const int per0 = I.periodic[0], per1 = I.periodic[1], per2 = I.periodic[2];
            const int t0 = o0 - tile.lo[0], t1 = o1 - tile.lo[1], t2 = o2 - tile.lo[2];
            const int pitch = tile.pitch, plane = tile.plane;
            auto box = [&](int o2b, auto &&at, int t_first, auto &&tat) {
                auto slab = [&](int i) {
                    const V2 e0 = cA[i * BS];
                    const T v0 = e0.x, q0 = e0.y * h0;
                    const int r0 = wrap_index(o0 + i, n0, per0) * s0 + o2b;
                    const int p0 = min(max(t0 + i, 0), tile.ext[0] - 1) * tile.ext[1];
                    T A0 = T(0), B0 = T(0);
                    auto row = [&](int j) {
                        const V2 e1 = cB[j * BS];
                        const T v1 = e1.x, q1 = e1.y * h1;
                        const R *rr = ri + (r0 + wrap_index(o1 + j, n1, per1) * s1);
                        double *d0 = tmem + ((p0 + min(max(t1 + j, 0), tile.ext[1] - 1)) * pitch + t_first);
                        double *d1 = d0 + plane, *d2 = d1 + plane, *d3 = d2 + plane;
                        const T vv = v0 * v1, sv = q0 * v1, vs = v0 * q1;
                        const T fa = Lm * vv, fb = Lm * sv, fc = Lm * vs;
                        T su = T(0), s_0 = T(0), s_1 = T(0);
#pragma unroll
                        for (int k = 0; k < L; ++k) {
                            const R r = rr[at(k)];
                            const T u = r.x - uref;
                            su = fma_t(V2_[k], u, fma_t(S2_[k], r.w, su));
                            s_0 = fma_t(V2_[k], r.y, s_0);
                            s_1 = fma_t(V2_[k], r.z, s_1);
                            A2[k] = fma_t(vv, u, fma_t(sv, r.y, fma_t(vs, r.z, A2[k])));
                            B2[k] = fma_t(vv, r.w, B2[k]);
                            const int e = tat(k);
                            lds_add(d0 + e, (double)(fa * V2_[k]));
                            lds_add(d1 + e, (double)(fb * V2_[k]));
                            lds_add(d2 + e, (double)(fc * V2_[k]));
                            lds_add(d3 + e, (double)(fa * S2_[k]));
                        }
                        A0 = fma_t(v1, su, fma_t(q1, s_1, A0));
                        B0 = fma_t(v1, s_0, B0);
                        const T a1 = fma_t(v0, su, q0 * s_0), b1_ = v0 * s_1;
                        if constexpr (UN) {
                            A1[j] += a1;
                            B1[j] += b1_;
                        } else {
                            V2 e = cC[j * BS];
                            e.x += a1;
                            e.y += b1_;
                            cC[j * BS] = e;
                        }
                    };
                    if constexpr (UN) {
#pragma unroll
                        for (int j = 0; j < L; ++j) row(j);
                    } else {
                        for (int j = 0; j < L1; ++j) row(j);
                    }
                    V2 ab;
                    ab.x = A0;
                    ab.y = B0;
                    cA[i * BS] = ab;
                };
                for (int i = 0; i < L0; ++i) slab(i);
            };
            if (__all(o2 >= 0 && o2 + L <= n2))
                box(o2, [](int k) { return k; }, t2, [](int k) { return k; });
            else
                box(0, [&](int k) { return wrap_index(o2 + k, n2, per2); }, 0,
                    [&](int k) { return max(t2 + k, 0); });
            T Gz[3], Hz[3];
            gradient(0, cA, Gz[0], Hz[0]);
            if constexpr (UN) {
#pragma unroll
                for (int j = 0; j < L; ++j) {
                    V2 ab;
                    ab.x = A1[j];
                    ab.y = B1[j];
                    cB[j * BS] = ab;
                }
                gradient(1, cB, Gz[1], Hz[1]);
            } else {
                gradient(1, cC, Gz[1], Hz[1]);
            }
#pragma unroll
            for (int k = 0; k < L; ++k)
                if (k < L2) {
                    V2 ab;
                    ab.x = A2[k];
                    ab.y = B2[k];
                    cA[k * BS] = ab;
                }
            gradient(2, cA, Gz[2], Hz[2]);
            double gn[kThetaSlots];
            for (int kk = 0; kk < kThetaSlots; ++kk) gn[kk] = 0.0;
            node_theta<D, T>(P, I, tf, trig, idx, Lm, Gz, Hz, gn);
            for (int kk = 0; kk < kThetaSlots; ++kk) gth[kk] += gn[kk];
        }
        __syncthreads();
        tile.template flush<PS>(I, mu, (T *)P.adj.stage);
        reduce_theta(red, gth, grad, it.inst);
        __syncthreads();
    }
}

}  // namespace
}  // namespace fk
