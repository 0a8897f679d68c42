// dugks_tile_f64.hip -- the tile kernel, FP64 T2.
#include "dugks_tile_impl.h"

template void dugks::launch_tile<double, dugks::STAGE_T2>(const dugks_plan*, const dugks::StageBufs<double>&,
                                                       int64_t, hipStream_t);
