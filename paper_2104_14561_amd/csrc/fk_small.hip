// fk_small.hip -- launcher of the one-launch step of small 2D plans.
#include "fk_sep.h"

namespace fk {
namespace {

template <typename T, int QS>
hipError_t small_launch(const PlanDev &P, int n, const void *u_in, void *u_out, hipStream_t s)
{
    if (P.hermite2)
        k_step_small2<T, QS, true><<<P.n_small_work, kBlock, P.small_lds, s>>>(
            P, n, P.inst, P.small_work, P.small_tiles, P.small_nodes, (const T *)u_in, (T *)u_out);
    else
        k_step_small2<T, QS, false><<<P.n_small_work, kBlock, P.small_lds, s>>>(
            P, n, P.inst, P.small_work, P.small_tiles, P.small_nodes, (const T *)u_in, (T *)u_out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_step_small2(const PlanDev &P, bool f32, int n, const void *u_in, void *u_out,
                              hipStream_t s)
{
#define FK_QS(v) case v: return f32 ? small_launch<float, v>(P, n, u_in, u_out, s) : small_launch<double, v>(P, n, u_in, u_out, s);
    switch (P.qs) { FK_QS(2) FK_QS(3) FK_QS(4) FK_QS(5) FK_QS(6) FK_QS(7) FK_QS(8) }
#undef FK_QS
    return hipErrorInvalidValue;
}

}  // namespace fk
