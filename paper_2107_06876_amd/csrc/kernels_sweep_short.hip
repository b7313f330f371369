// The half-iteration of sweep.h for factor rows of up to 128 entries.
#include "sweep.h"

namespace lcn {

hipError_t launch_short_sweep(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                              double *partial, unsigned long long *cnt, hipStream_t s)
{
    if (h.lp == 64)
        launch_sweep_columns<1>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    else
        launch_sweep_columns<2>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    return hipGetLastError();
}

}  // namespace lcn
