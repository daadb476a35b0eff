// The joint backward grids of tile width 64 whose blocks of keys are taken in shares.
#include "fa_bwd_joint.h"

namespace fa {

template hipError_t launch_joint_shares<64, false>(const BwdArgs&, int, hipStream_t);
template hipError_t launch_joint_shares<64, true>(const BwdArgs&, int, hipStream_t);

}  // namespace fa
