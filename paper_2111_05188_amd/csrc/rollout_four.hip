// Four-env rollout kernel (rollout_four.hpp): fp32 actors of up to 32 stocks,
// and the dispatch.
#include "rollout_four.hpp"

namespace tpk {
namespace four {
extern template hipError_t launch_type<false, 8>(RolloutArgs &, hipStream_t);
extern template hipError_t launch_type<true, 2>(RolloutArgs &, hipStream_t);
extern template hipError_t launch_type<true, 8>(RolloutArgs &, hipStream_t);
template hipError_t launch_type<false, 2>(RolloutArgs &, hipStream_t);
}  // namespace four

hipError_t launch_rollout_four(RolloutArgs &a, hipStream_t s)
{
    const bool small = a.env.n <= 32;   // two stocks a lane of the trade, or eight
    if (a.lay.dtype == TP_BF16)
        return small ? four::launch_type<true, 2>(a, s) : four::launch_type<true, 8>(a, s);
    return small ? four::launch_type<false, 2>(a, s) : four::launch_type<false, 8>(a, s);
}

}  // namespace tpk
