// dugks_tile_impl.h -- launches of the tile kernel on one grid (instantiated per
// precision and stage in dugks_tile_*.hip; private to the library).
#pragma once

#include "dugks_plan.h"
#include "dugks_tile.h"

namespace dugks {

template <typename T, int R, bool MFIX, int STAGE, bool VARR, int TR>
static void tile_go(const StepArgs<T>& a, const StageBufs<T>& q, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((tile_kernel<T, R, MFIX, STAGE, VARR, TR>), dim3(a.nlogical),
                     dim3(LANES * tile_cell_rows(R, TR)), 0, s, a, n, q.src, q.dst, q.dst2, q.aux,
                     q.cf, q.tabx, q.taby, q.uv, q.part, q.prev, q.hdr);
}

template <typename T, int R, int STAGE, bool VARR>
static void tile_rows_go(const dugks_plan* P, const StepArgs<T>& a, const StageBufs<T>& q,
                         int64_t n, hipStream_t s) {
  if (P->p.flags & DUGKS_FLAG_MASS_FIX) {
    tile_go<T, R, true, STAGE, VARR, MASS_GROUP>(a, q, n, s);
    return;
  }
  if constexpr (wide(R)) {
    if (P->tile == 10) {
      tile_go<T, R, false, STAGE, VARR, 10>(a, q, n, s);
      return;
    }
  }
  if constexpr (tall_tiles(sizeof(T), R, STAGE == STAGE_T2 ? DUGKS_T2 : DUGKS_T3S3)) {
    if (P->tile == 8) {
      tile_go<T, R, false, STAGE, VARR, 8>(a, q, n, s);
      return;
    }
  }
  tile_go<T, R, false, STAGE, VARR, 4>(a, q, n, s);
}

template <typename T, int R, int STAGE>
static void tile_vel_go(const dugks_plan* P, const StepArgs<T>& a, const StageBufs<T>& q,
                        int64_t n, hipStream_t s) {
  if constexpr (R == DUGKS_UPWIND5) {   // T2, analytic velocities (see validate)
    if constexpr (STAGE == STAGE_T2) tile_rows_go<T, R, STAGE, false>(P, a, q, n, s);
  } else if (P->p.vel_kind == DUGKS_VEL_ARRAYS) {
    tile_rows_go<T, R, STAGE, true>(P, a, q, n, s);
  } else {
    tile_rows_go<T, R, STAGE, false>(P, a, q, n, s);
  }
}

template <typename T, int STAGE>
static void tile_recon_go(const dugks_plan* P, const StepArgs<T>& a, const StageBufs<T>& q,
                          int64_t n, hipStream_t s) {
  switch (P->p.recon) {
    case DUGKS_CENTRAL2: tile_vel_go<T, DUGKS_CENTRAL2, STAGE>(P, a, q, n, s); break;
    case DUGKS_UPWIND3: tile_vel_go<T, DUGKS_UPWIND3, STAGE>(P, a, q, n, s); break;
    case DUGKS_CENTRAL4: tile_vel_go<T, DUGKS_CENTRAL4, STAGE>(P, a, q, n, s); break;
    default: tile_vel_go<T, DUGKS_UPWIND5, STAGE>(P, a, q, n, s); break;
  }
}

template <typename T, int STAGE>
void launch_tile(const dugks_plan* P, const StageBufs<T>& q, int64_t n, hipStream_t s) {
  StepArgs<T> a = step_args<T>(P, STAGE);
  a.seg_rows = P->tile;
  a.nsegs = (P->p.ny + P->tile - 1) / P->tile;
  a.nlogical = a.nstrips * a.nsegs;
  tile_recon_go<T, STAGE>(P, a, q, n, s);
}

}  // namespace dugks
