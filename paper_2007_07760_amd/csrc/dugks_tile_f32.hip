// dugks_tile_f32.hip -- the tile kernel, FP32 T2.
#include "dugks_tile_impl.h"

template void dugks::launch_tile<float, dugks::STAGE_T2>(const dugks_plan*, const dugks::StageBufs<float>&,
                                                       int64_t, hipStream_t);
