// dugks_tile_batch_impl.h -- launches of the batch tile kernel (instantiated per
// precision in dugks_tile_*_batch.hip; private to the library).
#pragma once

#include <type_traits>

#include "dugks_batch_impl.h"
#include "dugks_plan.h"
#include "dugks_tile.h"

namespace dugks {

// f(recon, mass fix, stage, rows) with compile-time arguments, for the batch
// kernels (the narrow patches)
template <int R, int STAGE, typename F>
static void batch_rows(bool mfix, F&& f) {
  if (mfix)
    f(std::integral_constant<int, R>{}, std::true_type{}, std::integral_constant<int, STAGE>{},
      std::integral_constant<int, MASS_GROUP>{});
  else
    f(std::integral_constant<int, R>{}, std::false_type{}, std::integral_constant<int, STAGE>{},
      std::integral_constant<int, 4>{});
}
template <int R, typename F>
static void batch_stages(int scheme, bool mfix, F&& f) {
  if (scheme == DUGKS_T3S3) {   // the two stages, in turn
    batch_rows<R, STAGE_A>(mfix, f);
    batch_rows<R, STAGE_B>(mfix, f);
  } else {
    batch_rows<R, STAGE_T2>(mfix, f);
  }
}
template <typename F>
static void batch_forms(int recon, int scheme, bool mfix, F&& f) {
  switch (recon) {
    case DUGKS_CENTRAL2: batch_stages<DUGKS_CENTRAL2>(scheme, mfix, f); break;
    case DUGKS_UPWIND3: batch_stages<DUGKS_UPWIND3>(scheme, mfix, f); break;
    default: batch_stages<DUGKS_CENTRAL4>(scheme, mfix, f); break;
  }
}

template <typename T>
void launch_batch_tile(const BatchDev& D, int recon, bool mfix, int scheme, hipStream_t s) {
  batch_forms(recon, scheme, mfix, [&](auto R, auto MF, auto ST, auto TR) {
    hipLaunchKernelGGL((batch_tile_kernel<T, R.value, MF.value, ST.value, TR.value>),
                       dim3(D.tile_blocks), dim3(LANES * tile_cell_rows(R.value, TR.value)), 0, s,
                       static_cast<const GridDesc<T>*>(D.desc), D.steps, D.ctl);
  });
}

template <typename T>
int batch_tile_occupancy(int recon, bool mfix, int scheme, int* per_cu) {
  int rc = DUGKS_OK;
  *per_cu = 1 << 30;
  batch_forms(recon, scheme, mfix, [&](auto R, auto MF, auto ST, auto TR) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n,
            reinterpret_cast<const void*>(
                &batch_tile_kernel<T, R.value, MF.value, ST.value, TR.value>),
            LANES * tile_cell_rows(R.value, TR.value), 0) != hipSuccess)
      rc = DUGKS_EDEVICE;
    *per_cu = std::min(*per_cu, n);
  });
  return rc;
}

}  // namespace dugks
