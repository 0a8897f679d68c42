// dugks_tile_f32_batch.hip -- the batch tile kernel in FP32.
#include "dugks_tile_batch_impl.h"

template void dugks::launch_batch_tile<float>(const dugks::BatchDev&, int, bool, int, hipStream_t);
