// The half-iteration of sweep.h for factor rows of 129 to 256 entries.
#include "sweep.h"

namespace lcn {

hipError_t launch_mid_sweep(const PassSide &S, const Handle &h, int mode, const FuseArgs &F, bool fused_in, int groups,
                              double *partial, unsigned long long *cnt, hipStream_t s)
{
    if (h.lp == 192)
        launch_sweep_columns<3>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    else
        launch_sweep_columns<4>(S, h, mode, F, fused_in, groups, partial, cnt, s);
    return hipGetLastError();
}

}  // namespace lcn
