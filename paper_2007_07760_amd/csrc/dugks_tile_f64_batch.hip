// dugks_tile_f64_batch.hip -- the batch tile kernel in FP64.
#include "dugks_tile_batch_impl.h"

template void dugks::launch_batch_tile<double>(const dugks::BatchDev&, int, bool, int, hipStream_t);
