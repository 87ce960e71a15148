// Score kernels for head_dim = 64. Instantiated (32-row blocks per wave, waves per workgroup): 1,1 1,2 1,4 1,7 1,8 2,4 2,7, and 3,6 for sweep 1.
#include "score_impl.h"

namespace audiokv {

hipError_t launch_score_d64(int which, const Geom& g, int NB, int WR, const score_detail::SweepArgs& a, hipStream_t s)
{
    using namespace score_detail;
    if (NB == 1 && WR == 1) return launch_sweep<64, 1, 1>(which, g, a, s);
    if (NB == 1 && WR == 2) return launch_sweep<64, 1, 2>(which, g, a, s);
    if (NB == 1 && WR == 4) return launch_sweep<64, 1, 4>(which, g, a, s);
    if (NB == 1 && WR == 7) return launch_sweep<64, 1, 7>(which, g, a, s);
    if (NB == 1 && WR == 8) return launch_sweep<64, 1, 8>(which, g, a, s);
    if (NB == 2 && WR == 4) return launch_sweep<64, 2, 4>(which, g, a, s);
    if (NB == 2 && WR == 7) return launch_sweep<64, 2, 7>(which, g, a, s);
    if (NB == 3 && WR == 6) return launch_sweep<64, 3, 6, false>(which, g, a, s);
    return hipErrorInvalidValue;
}

}  // namespace audiokv
