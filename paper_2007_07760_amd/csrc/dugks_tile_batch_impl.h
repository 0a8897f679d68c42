// dugks_tile_batch_impl.h -- launches of the batch tile kernel (instantiated per
// precision in dugks_tile_*_batch.hip; private to the library).
#pragma once

#include <type_traits>

#include "dugks_batch_impl.h"
#include "dugks_plan.h"
#include "dugks_tile.h"

namespace dugks {

// f(recon, mass fix, stage, rows) with compile-time arguments, for the batch
// kernels (the narrow patches) of tiles of `rows` rows (see block_tile_rows)
template <typename T, int R, int STAGE, typename F>
static void batch_rows(bool mfix, int rows, F&& f) {
  using std::integral_constant;
  constexpr int scheme = STAGE == STAGE_T2 ? DUGKS_T2 : DUGKS_T3S3;
  if (mfix) {
    f(integral_constant<int, R>{}, std::true_type{}, integral_constant<int, STAGE>{},
      integral_constant<int, MASS_GROUP>{});
    return;
  }
  if constexpr (tall_tiles(sizeof(T), R, scheme)) {
    if (rows == 8) {
      f(integral_constant<int, R>{}, std::false_type{}, integral_constant<int, STAGE>{},
        integral_constant<int, 8>{});
      return;
    }
  }
  f(integral_constant<int, R>{}, std::false_type{}, integral_constant<int, STAGE>{},
    integral_constant<int, 4>{});
}
template <typename T, int R, typename F>
static void batch_stages(int scheme, bool mfix, int rows, F&& f) {
  if (scheme == DUGKS_T3S3) {   // the two stages, in turn
    batch_rows<T, R, STAGE_A>(mfix, rows, f);
    batch_rows<T, R, STAGE_B>(mfix, rows, f);
  } else {
    batch_rows<T, R, STAGE_T2>(mfix, rows, f);
  }
}
template <typename T, typename F>
static void batch_forms(int recon, int scheme, bool mfix, int rows, F&& f) {
  switch (recon) {
    case DUGKS_CENTRAL2: batch_stages<T, DUGKS_CENTRAL2>(scheme, mfix, rows, f); break;
    case DUGKS_UPWIND3: batch_stages<T, DUGKS_UPWIND3>(scheme, mfix, rows, f); break;
    default: batch_stages<T, DUGKS_CENTRAL4>(scheme, mfix, rows, f); break;
  }
}

template <typename T>
void launch_batch_tile(const BatchDev& D, int recon, bool mfix, int scheme, hipStream_t s) {
  batch_forms<T>(recon, scheme, mfix, D.tile, [&](auto R, auto MF, auto ST, auto TR) {
    hipLaunchKernelGGL((batch_tile_kernel<T, R.value, MF.value, ST.value, TR.value>),
                       dim3(D.tile_blocks), dim3(LANES * tile_cell_rows(R.value, TR.value)), 0, s,
                       static_cast<const GridDesc<T>*>(D.desc), D.steps, D.ctl);
  });
}

}  // namespace dugks
