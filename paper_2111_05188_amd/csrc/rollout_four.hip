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

// The shape alone decides, so that an env's results are the same bits whatever
// the number of envs and agents in the call.  fp32: every width it holds (the
// VALU layers took 1.3 to 3.5 times as long, 1 to 65,536 envs).  bf16: the
// shapes at which no env count is slower than on the generic kernel: first
// layers to 384 wide (wider ones, with 16 envs a workgroup, spill), second ones
// to 768, and rows of 16 envs that fit the LDS.  us a lockstep step (64 steps
// with reset and GAE), generic kernel -> this one, at 64, 2,048, 4,096 and
// 16,384 envs:
//   31-128-128-5      9.9,  9.9,  9.9, 39 ->  2.7,  3.0,  3.7, 14
//   301-256-256-30   12.7, 12.8, 13.0, 51 ->  4.8,  5.4,  7.0, 27
//   301-384-384-30   15.7, 15.9, 16.1, 63 ->  7.3,  8.4,  9.7, 38
//   1001-384-384-100 20.2, 20.6, 21.1, 83 -> 12.5, 14.6, 17.2, 68
//   1281-384-512-128 23.3, 23.5, 24.5, 96 -> 17.0, 18.6, 21.7, 86
// Past the line, with 8 envs a workgroup: 301-512-512-30 at 64 envs 153 us for
// eight steps -> 100, but 618 -> 973 at 16,384; 1001-384-1024-100 at 2,056 envs
// (16 a workgroup) 3% slower.
bool rollout_four_shape(const PackedLayout &P)
{
    if (P.dtype == TP_F32) return P.four;
    if (P.H1 > 384 || P.H2 > 768) return false;
    const four::Tiles t = four::tiles(P);
    four::Plan plan;
    return four::make_plan(P, 16, t.GT, t.TW, (int)LDS_LIMIT, &plan);
}

hipError_t launch_rollout_four(RolloutArgs &a, hipStream_t s)
{
    const bool small = a.env.n <= 32;   // two stocks a lane of the trade, or eight
    if (a.lay.dtype == TP_BF16)
        return small ? four::launch_type<true, 2>(a, s) : four::launch_type<true, 8>(a, s);
    return small ? four::launch_type<false, 2>(a, s) : four::launch_type<false, 8>(a, s);
}

}  // namespace tpk
