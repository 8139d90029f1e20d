// Instantiates the aggregation kernels for 1 disparities per lane.
#include "aggregate_impl.h"

namespace ss {

hipError_t launch_agg_dpl1(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s)
{
    return wide ? launch_aggregation_lanes<1, true>(a, q, grid, hl, s) : launch_aggregation_lanes<1, false>(a, q, grid, hl, s);
}

}  // namespace ss
