// Four-env rollout kernel (rollout_four.hpp): bf16 actors of more than 32 stocks.
#include "rollout_four.hpp"

namespace tpk {
namespace four {
template hipError_t launch_type<true, 8>(RolloutArgs &, hipStream_t);
}  // namespace four
}  // namespace tpk
