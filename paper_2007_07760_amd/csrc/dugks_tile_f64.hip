// dugks_tile_f64.hip -- the tile kernel in FP64.
#include "dugks_tile_impl.h"

template void dugks::launch_tile<double>(const dugks_plan*, int, const dugks::StageBufs<double>&,
                                       int64_t, hipStream_t);
