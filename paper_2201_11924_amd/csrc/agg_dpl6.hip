// Instantiates the aggregation kernels for 6 disparities per lane.
#include "aggregate_impl.h"

namespace ss {

hipError_t launch_agg_dpl6(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s)
{
    return wide ? launch_aggregation_lanes<6, true>(a, q, grid, hl, s) : launch_aggregation_lanes<6, false>(a, q, grid, hl, s);
}

}  // namespace ss
