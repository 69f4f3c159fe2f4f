// The dK/dV pass at head_dim 128 (one workgroup per compute unit with the whole register file), softmax weights: the
// instantiations of hta_bwd_dkdv.h that are compiled with the scheduling strategy favouring instruction-level parallelism
// (build.py), with the launch for the keys behind the history where there are real-time tokens.  The pointwise kernel spills
// under that strategy (20 bytes per lane) and stays with the default one in hta_bwd_bf16.hip.
#include "hta_bwd_dkdv.h"

namespace hta {

hipError_t launch_bwd_dkdv128_bf16(const Params& p, hipStream_t s) { return launch_dkdv_as<128, 4, false>(p, s); }

}  // namespace hta
