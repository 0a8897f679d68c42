// dugks_batch_impl.h -- pieces of the batch path shared by the batch entry
// points and the allocation-free multi-grid step (private to the library).
#pragma once

#include <string.h>

#include <algorithm>

#include "dugks_common.h"
#include "dugks_kernels.h"
#include "dugks_plan.h"

namespace dugks {

// Device memory one batch step works on: descriptors, step counters, slot
// status, the work-list control block and the queue heads.
struct BatchDev {
  const void* desc;
  SlotStep* steps;
  int32_t* status;
  BatchCtl* ctl;
  unsigned* head;
  int nslots;        // finish-kernel blocks (one per slot)
  int grid_blocks;   // resident wavefronts of the persistent kernel
  int tile;          // rows of the block tiles the list holds; 0: marching tiles
  int tile_blocks;   // blocks of the tile kernel: NQUEUE x the longest queue, or more
};

// One batch step (finish = true) or the step kernels alone, on `s`, for grids
// of one precision / reconstruction / mass-fix flag / time scheme.
int launch_batch(const BatchDev& D, int precision, int recon, bool mfix, int scheme,
                 hipStream_t s, bool finish);

// The most 16-row marching tiles (of all grids together) for which the block
// tiles are taken: where they meet the marching tiles of the batch's choice (8
// or 16 rows), measured on the first grids of a mix of sides 32-512 (us per
// step, block / marching tiles): FP32 corrected upwind-3 841 tiles 37.9 / 38.4,
// 1143 45.6 / 44.4, T3S3 841 73.8 / 73.9, central-4 1305 53.7 / 54.9, 1538 61.0 /
// 58.5; FP64 upwind-3 1305 63.0 / 65.6, 1538 74.2 / 70.1, central-4 1305 82.2 /
// 86.3, 1538 93.7 / 87.8, T3S3 463 68.2 / 71.7, 841 111 / 101.
inline int64_t batch_tile_limit(int precision, int recon, int scheme) {
  if (recon == DUGKS_CENTRAL4) return precision == DUGKS_F32 ? 1350 : 1400;
  if (precision == DUGKS_F32) return 900;
  return scheme == DUGKS_T3S3 ? 600 : 1350;
}

// The step kernels of launch_batch for a list of block tiles.
template <typename T>
void launch_batch_tile(const BatchDev& D, int recon, bool mfix, int scheme, hipStream_t s);

// Resident wavefronts per CU of the batch step kernel of that kind.
int batch_occupancy(int precision, int recon, bool mfix, int scheme, int* per_cu);

// The descriptor of one grid (plan, state), its tiles `rows` high.
template <typename T>
inline GridDesc<T> make_grid_desc(const dugks_plan* P, void* state, int rows) {
  GridDesc<T> d;
  memset(&d, 0, sizeof(d));
  if (!P) return d;
  const Layout& L = P->L;
  const bool t3 = P->p.scheme == DUGKS_T3S3;
  d.a = step_args<T>(P, t3 ? STAGE_A : STAGE_T2);
  d.b = step_args<T>(P, t3 ? STAGE_B : STAGE_T2);
  const int seg = std::min(rows, P->p.ny);
  for (StepArgs<T>* a : {&d.a, &d.b}) {
    a->seg_rows = seg;
    a->nsegs = (P->p.ny + seg - 1) / seg;
    a->nlogical = a->nstrips * a->nsegs;
    a->ileave = 1;   // unused: a batch takes its tiles from its work queues
    a->clen = a->nsegs;
  }
  if (t3) {
    d.mid = at<T>(state, L.off_mid);
    d.q = at<T>(state, L.off_q);
    d.cf2 = at<T>(state, L.off_coef2);
  }
  d.buf[0] = at<T>(state, L.off_buf[0]);
  d.buf[1] = at<T>(state, L.off_buf[1]);
  d.cf = at<T>(state, L.off_coef);
  d.tabx = at<T>(state, L.off_tabx);
  d.taby = at<T>(state, L.off_taby);
  d.hdr = at<StateHeader>(state, 0);
  d.part = at<double>(state, L.off_groups);
  d.ncells = (double)P->p.nx * (double)P->p.ny;
  d.strip_part = at<double>(state, L.off_strips);
  d.groups_per_strip = L.ngroups;
  d.nstrips = L.tl.nstrips;
  return d;
}

}  // namespace dugks
