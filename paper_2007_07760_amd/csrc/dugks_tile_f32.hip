// dugks_tile_f32.hip -- the tile kernel in FP32.
#include "dugks_tile_impl.h"

template void dugks::launch_tile<float>(const dugks_plan*, int, const dugks::StageBufs<float>&,
                                       int64_t, hipStream_t);
