// dugks_tile_f64_t3s3.hip -- the tile kernel, the stages of FP64 T3S3.
#include "dugks_tile_impl.h"

template void dugks::launch_tile<double, dugks::STAGE_A>(const dugks_plan*, const dugks::StageBufs<double>&,
                                                      int64_t, hipStream_t);
template void dugks::launch_tile<double, dugks::STAGE_B>(const dugks_plan*, const dugks::StageBufs<double>&,
                                                      int64_t, hipStream_t);
