// fk_line.hip -- several backward steps of one-dimensional plans in one launch.
#include "fk_sep.h"

namespace fk {
namespace {

constexpr int kLineThreads = 1024;
constexpr int kLineLanes = 4;   // lanes per node, each a quarter of the GH nodes

// Sum over the four lanes of a quad, by lane permutation inside the VALU.
template <int CTRL> __device__ inline float quad_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ inline double quad_add(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
template <typename T> __device__ inline T quad_sum(T v)
{
    v = quad_add<0xb1>(v);          // lanes 1, 0, 3, 2
    return quad_add<0x4e>(v);       // lanes 2, 3, 0, 1
}

// Steps n_hi - 1 .. n_lo (u^{n_hi} -> u^{n_lo}) of one instance per workgroup.
// The records (u, g) of the instance stay in LDS, two buffers used in turn:
// a step writes the new values into the other buffer and the slopes follow
// there, two barriers per step.  The drift of a one-dimensional problem is
// constant, so that on an affine axis the landing cells and weighted bases of
// the GH nodes, relative to the node, are the same for every node and step:
// they are registers.  What depends on the node is which points exit, a bit
// mask per node and lane taken from the coordinates once.
//
// u^m goes to store + (m / every - shift) stride whenever every divides m, and
// u^{n_lo} to u_out (each may be null).
//
// ONE: at most 256 nodes, so that a thread keeps one node for all steps and the
// exits (and a cell that the rounding put one off the axis) fold into its
// registers' weights; more nodes loop, with the mask looked up.
//
// Bound: the chain of a step (two barriers, a division in the slope, the LDS
// reads) and the issue of its 16 waves; one launch replaces 2 (n_hi - n_lo).
// 201 nodes, Q* = 16, FP64: 0.89 us a step (1.8 with the mask looked up and the
// sums through LDS permutations) against 16 us in two launches.
template <typename T, int QS, bool ONE>
__global__ void __launch_bounds__(kLineThreads) k_line_steps(
    const PlanDev P, int n_hi, int n_lo, int nmax, const T *__restrict__ u_in,
    T *__restrict__ u_out, T *__restrict__ store, int every, int shift, long long stride)
{
#pragma clang fp contract(off)
    using V2 = typename Vec2T<T>::type;
    constexpr int G = kLineLanes, NQ = (QS + G - 1) / G, NG = kLineThreads / G;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V2 *recs = reinterpret_cast<V2 *>(smem_raw);                       // [2][nmax]
    unsigned char *mask = reinterpret_cast<unsigned char *>(recs + 2 * nmax);   // [nmax][G]
    unsigned char *cls = mask + nmax * G;                              // [nmax]
    const DevInst &I = P.inst[blockIdx.x];
    const int n = I.n[0], tid = threadIdx.x, lane = tid % G, grp = tid / G;
    const bool per = I.periodic[0] != 0, ball = I.region_kind == 1;
    const T *w1 = weights1<T>(P);
    const double bdt = I.coef[0] * P.dt;
    const T h = (T)I.step[0], ih = (T)I.inv_h[0];
    int off[NQ];
    T y0[NQ], y1[NQ], f0[NQ], f1[NQ], wq[NQ];
    double zq[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int q = lane + i * G < QS ? lane + i * G : QS - 1;
        wq[i] = lane + i * G < QS ? w1[q] : T(0);
        const double t = fma_t(P.gh_a[q], I.S * I.inv_h[0], bdt * I.inv_h[0]);
        const double fl = floor(t);
        T v0, v1, d0, d1;
        unit_basis<T>((T)(t - fl), v0, v1, d0, d1);
        off[i] = (int)fl;
        y0[i] = wq[i] * v0;
        y1[i] = wq[i] * v1;
        f0[i] = wq[i] * h * d0;
        f1[i] = wq[i] * h * d1;
        zq[i] = I.S * P.gh_a[q];
    }
    bool odd = false;   // some value of the first field is not finite
    for (int j = tid; j < n; j += kLineThreads) {
        const T u = u_in[I.node_off + j];
        odd = odd || !isfinite((double)u);
        recs[j].x = u;
        cls[j] = P.chi[I.node_off + j];
    }
    for (int j = grp; j < n; j += NG) {
        const double x = (j == n - 1) ? I.hi[0] : (double)j * I.step[0] + I.lo[0];
        const double c = x + bdt;
        unsigned int m = 0;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const double z = c + zq[i];
            const double dz = z - I.center[0];
            const bool ex = (!per && (z <= I.lo[0] || z >= I.hi[0])) || (ball && dz * dz >= I.r2);
            m |= ex ? 1u << i : 0u;
        }
        mask[j * G + lane] = (unsigned char)m;
    }
    const int any_odd = __builtin_amdgcn_readfirstlane(__syncthreads_or(odd));
    if constexpr (ONE) {
        // the value of node j's inside landing point q
        auto point = [&](const V2 *r, int j, int q, T uref) -> T {
            const double t = fma_t(P.gh_a[q], I.S * I.inv_h[0], bdt * I.inv_h[0]);
            const double fl = floor(t);
            T v0, v1, d0, d1;
            unit_basis<T>((T)(t - fl), v0, v1, d0, d1);
            int k = j + (int)fl;
            if (per) k += k < 0 ? n - 1 : (k > n - 2 ? 1 - n : 0);
            const V2 a = r[min(max(k, 0), n - 2)], b = r[min(max(k, 0), n - 2) + 1];
            if (k < 0) return w1[q] * (a.x - uref);
            if (k > n - 2) return w1[q] * (b.x - uref);
            return w1[q] * (v0 * (a.x - uref) + v1 * (b.x - uref) + h * (d0 * a.y + d1 * b.y));
        };
        const int j = grp;
        const bool act = j < n && cls[j] == 0;
        int kc[NQ];
        T em = T(0);
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const bool ex = j < n && ((mask[j * G + lane] >> i) & 1u);
            int k = j + off[i];
            if (per) k += k < 0 ? n - 1 : (k > n - 2 ? 1 - n : 0);
            kc[i] = act ? min(max(k, 0), n - 2) : 0;
            if (!act || ex || k != kc[i]) {
                if (act && ex) em += wq[i];
                y0[i] = act && !ex && k < 0 ? wq[i] : T(0);
                y1[i] = act && !ex && k > n - 2 ? wq[i] : T(0);
                f0[i] = f1[i] = T(0);
            }
        }
        // this thread's slope node (tid < n) and its stencil
        int il = 0, ic = 0, ir = 0;
        T rl, rr;
        if (tid < n) slope_stencil<T>(I, P.coords, 0, tid, il, ic, ir, rl, rr);
        const bool writes = lane == 0 && j < n && (act || cls[j] != 2);
        const bool image = lane == 0 && per && j == 0 && act;
        const T fix = j < n && (cls[j] & 5) == 1 ? T(1) : T(0);
        em = quad_sum(em);
        // all steps; check: the first field holds values that are not finite
        auto steps = [&](auto check) {
            int cur = 0;
            for (int m = n_hi - 1; m >= n_lo; --m) {
                V2 *r = recs + cur * nmax, *rn = recs + (1 - cur) * nmax;
                if (tid < n) r[tid].y = pchip<T>(r[il].x, r[ic].x, r[ir].x, ih, ih);
                __syncthreads();
                const T uref = act ? r[j].x : T(0);
                T acc = T(0);
    #pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    const V2 a = r[kc[i]], b = r[kc[i] + 1];
                    acc = fma_t(y0[i], a.x - uref, fma_t(y1[i], b.x - uref, fma_t(f0[i], a.y, fma_t(f1[i], b.y, acc))));
                }
                acc = quad_sum(acc);
                if (check.value && act && !isfinite((double)acc)) {
                    // a record without weight may have held a value that is not finite:
                    // the inside points alone
                    acc = T(0);
    #pragma unroll 1
                    for (int q = lane, i = 0; q < QS; q += G, ++i) {
                        if ((mask[j * G + lane] >> i) & 1u) continue;
                        acc += point(r, j, q, uref);
                    }
                    acc = quad_sum(acc);
                }
                if (writes) {
                    const T v = act ? uref + acc + em * (T(1) - uref) : fix;
                    flag_nonfinite(P.flags, v);
                    rn[j].x = v;
                    if (image) rn[n - 1].x = v;
                    if (store != nullptr && m % every == 0) {
                        T *out = store + (long long)(m / every - shift) * stride + I.node_off;
                        out[j] = v;
                        if (image) out[n - 1] = v;
                    }
                    if (u_out != nullptr && m == n_lo) {
                        u_out[I.node_off + j] = v;
                        if (image) u_out[I.node_off + n - 1] = v;
                    }
                }
                __syncthreads();
                cur = 1 - cur;
            }
        };
        if (any_odd) steps(std::true_type{});
        else steps(std::false_type{});
        return;
    }
    // value of an inactive node (an exit node's, 0 or 1; an image of an active
    // node takes its original's, below)
    auto fixed = [&](int j) { return (T)((cls[j] & 5) == 1 ? 1 : 0); };
    int cur = 0;
    for (int m = n_hi - 1; m >= n_lo; --m) {
        V2 *r = recs + cur * nmax, *rn = recs + (1 - cur) * nmax;
        for (int j = tid; j < n; j += kLineThreads) {
            int il, ic, ir;
            T rl, rr;
            slope_stencil<T>(I, P.coords, 0, j, il, ic, ir, rl, rr);
            r[j].y = pchip<T>(r[il].x, r[ic].x, r[ir].x, ih, ih);
        }
        __syncthreads();
        const bool keep = store != nullptr && m % every == 0;
        T *out = keep ? store + (long long)(m / every - shift) * stride + I.node_off
                      : (m == n_lo && u_out ? u_out + I.node_off : nullptr);
        T *out2 = keep && m == n_lo && u_out ? u_out + I.node_off : nullptr;
        auto put = [&](int j, T v) {
            rn[j].x = v;
            if (out) out[j] = v;
            if (out2) out2[j] = v;
        };
        for (int j = grp; j < n; j += NG) {
            if (cls[j] != 0) {
                if (lane == 0 && cls[j] != 2) put(j, fixed(j));
                continue;
            }
            const T uref = r[j].x;
            const unsigned int mk = mask[j * G + lane];
            T acc = T(0), em = T(0);
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                int k = j + off[i];
                if (per) k += k < 0 ? n - 1 : (k > n - 2 ? 1 - n : 0);
                const int kc = min(max(k, 0), n - 2);
                const V2 a = r[kc], b = r[kc + 1];
                T v = fma_t(y0[i], a.x - uref, fma_t(y1[i], b.x - uref, fma_t(f0[i], a.y, f1[i] * b.y)));
                // an inside point whose cell the rounding put one off the axis: its end node
                if (k != kc) v = wq[i] * ((k < 0 ? a.x : b.x) - uref);
                const bool ex = (mk >> i) & 1u;
                acc += ex ? T(0) : v;
                em += ex ? wq[i] : T(0);
            }
            acc = quad_sum(acc);
            em = quad_sum(em);
            if (lane == 0) {
                const T v = uref + acc + em * (T(1) - uref);
                flag_nonfinite(P.flags, v);
                put(j, v);
                if (per && j == 0) put(n - 1, v);
            }
        }
        __syncthreads();
        cur = 1 - cur;
    }
}

template <typename T, int QS>
hipError_t line_launch(const PlanDev &P, int nmax, int n_hi, int n_lo, const void *u_in, void *u_out,
                       void *store, int every, int shift, hipStream_t s)
{
    const size_t lds = line_lds(nmax, sizeof(T) == 4);
    if (nmax <= kLineThreads / kLineLanes) {
        k_line_steps<T, QS, true><<<P.n_inst, kLineThreads, lds, s>>>(
            P, n_hi, n_lo, nmax, (const T *)u_in, (T *)u_out, (T *)store, every, shift, P.n_nodes);
        return hipGetLastError();
    }
    // (the limit is the process': every plan sets the same value, the longest axis')
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_line_steps<T, QS, false>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)line_lds(kLineNodes, sizeof(T) == 4));
    k_line_steps<T, QS, false><<<P.n_inst, kLineThreads, lds, s>>>(
        P, n_hi, n_lo, nmax, (const T *)u_in, (T *)u_out, (T *)store, every, shift, P.n_nodes);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_line_steps(const PlanDev &P, bool f32, int nmax, int n_hi, int n_lo, const void *u_in,
                             void *u_out, void *store, int every, int shift, hipStream_t s)
{
#define FK_QS(v) case v: return f32 ? line_launch<float, v>(P, nmax, n_hi, n_lo, u_in, u_out, store, every, shift, s) \
                                    : line_launch<double, v>(P, nmax, n_hi, n_lo, u_in, u_out, store, every, shift, s);
    switch (P.qs) { FK_QS(2) FK_QS(3) FK_QS(4) FK_QS(5) FK_QS(6) FK_QS(7) FK_QS(8) FK_QS(10) FK_QS(12) FK_QS(16) }
#undef FK_QS
    return hipErrorInvalidValue;
}

}  // namespace fk
