// The joint backward grids of tile width 128 whose blocks of keys are taken in shares.
#include "fa_bwd_joint.h"

namespace fa {

template hipError_t launch_joint_shares<128, false>(const BwdArgs&, int, hipStream_t);
template hipError_t launch_joint_shares<128, true>(const BwdArgs&, int, hipStream_t);

}  // namespace fa
