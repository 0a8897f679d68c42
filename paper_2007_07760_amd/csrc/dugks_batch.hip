// dugks_batch.hip -- C ABI of batches (include/dugks.h): many independent
// grids of one precision and reconstruction advanced by one persistent kernel,
// replayed from a captured hipGraph, with a measured choice of tile height.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "dugks_common.h"
#include "dugks_kernels.h"
#include "dugks_plan.h"
#include "dugks_batch_impl.h"

using namespace dugks;

namespace {

constexpr int NSTAGE = 3;   // pinned staging buffers in flight

// Tile heights the autotuner tries (whole mass groups; 0: the batch's own choice).
constexpr int TUNE_ROWS[] = {0, 16, 24, 32, 48, 64, 96, 128, 192, 256};
constexpr int DEFAULT_ROWS = 64;   // reported until the first commit chooses

struct Slot {
  const dugks_plan* plan = nullptr;
  void* state = nullptr;
  int64_t step = 0, target = 0;
  int64_t until = 0;                  // the batch's step (see done) it stops at
  bool step_dirty = false;
};

}  // namespace

namespace dugks {

template <typename T, int R, bool MFIX>
static int launch_batch_step(const BatchDev& D, int scheme, hipStream_t s, bool finish) {
  const GridDesc<T>* desc = static_cast<const GridDesc<T>*>(D.desc);
  if (D.tile) {
    launch_batch_tile<T>(D, R, MFIX, scheme, s);
  } else if (scheme == DUGKS_T3S3) {   // the two stages over every tile, in turn
    hipLaunchKernelGGL((batch_step_kernel<T, R, MFIX, STAGE_A>), dim3(D.grid_blocks),
                       dim3(LANES), 0, s, desc, D.steps, D.ctl, D.head);
    hipLaunchKernelGGL((batch_step_kernel<T, R, MFIX, STAGE_B>), dim3(D.grid_blocks),
                       dim3(LANES), 0, s, desc, D.steps, D.ctl, D.head);
  } else {
    hipLaunchKernelGGL((batch_step_kernel<T, R, MFIX>), dim3(D.grid_blocks), dim3(LANES), 0, s,
                       desc, D.steps, D.ctl, D.head);
  }
  if (finish)
    hipLaunchKernelGGL((batch_finish_kernel<T, MFIX>), dim3(D.nslots), dim3(FIX_THREADS), 0, s,
                       desc, D.steps, D.head, D.status);
  return hip_status(hipGetLastError());
}

int launch_batch(const BatchDev& D, int precision, int recon, bool mfix, int scheme,
                 hipStream_t s, bool finish) {
#define DUGKS_BATCH(TT, RR)                                                    \
  return mfix ? launch_batch_step<TT, RR, true>(D, scheme, s, finish)          \
              : launch_batch_step<TT, RR, false>(D, scheme, s, finish)
#define DUGKS_BATCH_R(TT)                                        \
  switch (recon) {                                               \
    case DUGKS_CENTRAL2: DUGKS_BATCH(TT, DUGKS_CENTRAL2);        \
    case DUGKS_UPWIND3: DUGKS_BATCH(TT, DUGKS_UPWIND3);          \
    default: DUGKS_BATCH(TT, DUGKS_CENTRAL4);                    \
  }
  if (precision == DUGKS_F64) {
    DUGKS_BATCH_R(double)
  } else {
    DUGKS_BATCH_R(float)
  }
#undef DUGKS_BATCH_R
#undef DUGKS_BATCH
}

template <typename T, int R, bool MFIX>
static int occupancy(int* per_cu, int scheme) {
  if (scheme == DUGKS_T3S3) {   // the smaller of the two stages' residencies
    int a = 0, b = 0;
    int rc = hip_status(hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &a, reinterpret_cast<const void*>(&batch_step_kernel<T, R, MFIX, STAGE_A>), LANES, 0));
    if (!rc)
      rc = hip_status(hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &b, reinterpret_cast<const void*>(&batch_step_kernel<T, R, MFIX, STAGE_B>), LANES,
          0));
    *per_cu = std::min(a, b);
    return rc;
  }
  return hip_status(hipOccupancyMaxActiveBlocksPerMultiprocessor(
      per_cu, reinterpret_cast<const void*>(&batch_step_kernel<T, R, MFIX>), LANES, 0));
}

int batch_occupancy(int precision, int recon, bool mfix, int scheme, int* per_cu) {
#define DUGKS_OCC(TT, RR)                                   \
  return mfix ? occupancy<TT, RR, true>(per_cu, scheme)     \
              : occupancy<TT, RR, false>(per_cu, scheme)
#define DUGKS_OCC_R(TT)                                 \
  switch (recon) {                                      \
    case DUGKS_CENTRAL2: DUGKS_OCC(TT, DUGKS_CENTRAL2);  \
    case DUGKS_UPWIND3: DUGKS_OCC(TT, DUGKS_UPWIND3);    \
    default: DUGKS_OCC(TT, DUGKS_CENTRAL4);              \
  }
  if (precision == DUGKS_F64) {
    DUGKS_OCC_R(double)
  } else {
    DUGKS_OCC_R(float)
  }
#undef DUGKS_OCC_R
#undef DUGKS_OCC
}

}  // namespace dugks

struct dugks_batch {
  int cap = 0, precision = 0, recon = 0;
  int scheme = DUGKS_T2;              // every attached plan's time scheme
  bool mfix = false;
  int device = 0;
  size_t desc_bytes = 0;              // sizeof(GridDesc<T>)
  // device memory owned by the batch
  void* d_desc = nullptr;             // GridDesc<T>[cap]
  SlotStep* d_steps = nullptr;        // [cap]
  int32_t* d_status = nullptr;        // [cap] status of each slot's state
  BatchCtl* d_ctl = nullptr;
  unsigned* d_head = nullptr;
  BatchItem* d_items = nullptr;
  size_t items_cap = 0;
  // host side
  std::vector<Slot> slots;
  std::vector<BatchItem> items;
  std::vector<int32_t> qstart;        // queue q: items [qstart[q], qstart[q + 1])
  int nq = 1;
  bool desc_dirty = true;
  int64_t done = 0;                   // steps issued
  int rows = DEFAULT_ROWS;            // height of the marching tiles
  int tile = 0;                       // rows of the list's block tiles; 0: marching tiles
  bool given = false;                 // the height is the caller's (or the autotuner's)
  bool given_tile = false;            // choice, with block tiles while the grids are
                                      // few; else each commit chooses
  int grid_blocks = 0;                // resident wavefronts of the persistent kernel
  int tile_blocks = 0;                // NQUEUE x the longest queue of block tiles
  // pinned staging ring: [ctl][desc table][steps][items]
  void* stage[NSTAGE] = {};
  size_t stage_bytes[NSTAGE] = {};
  hipEvent_t stage_ev[NSTAGE] = {};
  int stage_next = 0;
  // graphs of K steps, one per kind of tiles
  hipStream_t cap_stream = nullptr;
  struct Graph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int k = 0;
    int blocks = 0;                   // of its tile kernels: no fewer than the list needs
  } graphs[3];                        // marching tiles, block tiles of 4 and 8 rows
  // replaced graphs whose replays may still be running: until `over` has passed
  struct Retired {
    hipGraph_t graph;
    hipGraphExec_t exec;
    hipEvent_t over;
  };
  std::vector<Retired> retired;
};

namespace {

template <typename T>
GridDesc<T> make_desc(const Slot& s, int rows) {
  return make_grid_desc<T>(s.plan, s.state, rows);
}

// Whether a list of marching tiles of `rows` rows is more than two rounds of the
// resident wavefronts, of grids that stop at different steps of the batch.  (Of
// up to two rounds, a queue left alone is one for the quarter of the wavefronts
// that reach it.)
bool uneven_rounds(const dugks_batch* B, int rows) {
  int64_t first = -1, tiles = 0;
  bool differ = false;
  for (const Slot& s : B->slots) {
    if (!s.plan) continue;
    const int64_t left = std::max<int64_t>(s.until - B->done, 0);
    differ = differ || (first >= 0 && left != first);
    first = left;
    tiles += (int64_t)s.plan->nstrips * ((s.plan->p.ny + rows - 1) / rows);
  }
  return differ && tiles > 2 * (int64_t)B->grid_blocks;
}

struct Keyed {
  int h;         // rows of the tile
  BatchItem it;
};

// Every grid's tiles, segment by segment, cut into NQUEUE equal bands, one per
// queue (starting at another queue for each slot): the queues stay equal also
// when some grids have reached their targets.
void spread_tiles(const dugks_batch* B, int rows, std::vector<Keyed>* queue) {
  for (int k = 0; k < B->cap; k++) {
    const Slot& s = B->slots[k];
    if (!s.plan) continue;
    const int ny = s.plan->p.ny, nstrips = s.plan->nstrips;
    const int seg = std::min(rows, ny);
    const int64_t n = (int64_t)nstrips * ((ny + seg - 1) / seg);
    for (int64_t i = 0; i < n; i++)
      queue[(i * NQUEUE / n + k) % NQUEUE].push_back(
          {std::min(seg, ny - (int)(i / nstrips) * seg), {k, (int32_t)i}});
  }
}

// The grids' tiles, the largest grid first and each grid's segment by segment,
// laid end to end and cut at equal shares of the marched rows, so a queue holds
// whole small grids or a band of segments of a large one: tiles that share halos
// stay in one XCD's L2.
void share_tiles(const dugks_batch* B, int rows, std::vector<Keyed>* queue) {
  std::vector<std::pair<int64_t, int>> order;   // (marched rows, slot)
  int64_t total = 0;
  for (int k = 0; k < B->cap; k++) {
    const Slot& s = B->slots[k];
    if (!s.plan) continue;
    const int ny = s.plan->p.ny;
    const int seg = std::min(rows, ny);
    const int64_t nsegs = (ny + seg - 1) / seg;
    order.push_back({(int64_t)s.plan->nstrips * (ny + 5 * nsegs), k});
    total += order.back().first;
  }
  std::stable_sort(order.begin(), order.end(),
                   [](const std::pair<int64_t, int>& a, const std::pair<int64_t, int>& b) {
                     return a.first > b.first;
                   });
  int q = 0;
  int64_t done = 0;
  for (const auto& o : order) {
    const int k = o.second;
    const Slot& s = B->slots[k];
    const int ny = s.plan->p.ny, nstrips = s.plan->nstrips;
    const int seg = std::min(rows, ny);
    const int nsegs = (ny + seg - 1) / seg;
    for (int g = 0; g < nsegs; g++) {
      const int h = std::min(seg, ny - g * seg);
      for (int st = 0; st < nstrips; st++) {
        // up to the queue's share of the work (the last queue takes the rest)
        while (q < NQUEUE - 1 && done + h + 5 > total * (q + 1) / NQUEUE) q++;
        queue[q].push_back({h, {k, g * nstrips + st}});
        done += h + 5;
      }
    }
  }
}

// The work list for tiles of `rows` rows, cut into NQUEUE queues of about equal
// work (one per XCD); within a queue the taller tiles come first, so that the
// short ones fill the tail.  A block of the tile kernel takes one item of its
// XCD's queue, so every queue gets a band of each grid, and so it does where
// marching wavefronts take several tiles each and the grids stop at different
// steps: once a queue's grids have stopped, a seventh of its wavefronts goes on to
// each of the others.  128 of 1024 corrected FP32 grids of 256^2 going on, us per
// step with whole grids in a queue / bands: 652 / 317 (FP64 1008 / 453), 32 of 256
// grids 187 / 78.  While all run, bands cost up to 1 % at the default heights (4 %
// for central-4 of hardly more than two rounds) and 2-5 % at 64 rows.
void build_items(dugks_batch* B, int rows) {
  std::vector<Keyed> queue[NQUEUE];
  if (B->tile || uneven_rounds(B, rows))
    spread_tiles(B, rows, queue);
  else
    share_tiles(B, rows, queue);
  B->items.clear();
  B->qstart.assign(NQUEUE + 1, 0);
  size_t most = 1;
  for (int q = 0; q < NQUEUE; q++) {
    if (!B->tile)
      std::stable_sort(queue[q].begin(), queue[q].end(),
                       [](const Keyed& a, const Keyed& b) { return a.h > b.h; });
    for (const Keyed& k : queue[q]) B->items.push_back(k.it);
    B->qstart[q + 1] = (int32_t)B->items.size();
    most = std::max(most, queue[q].size());
  }
  B->nq = B->items.empty() ? 1 : NQUEUE;
  B->tile_blocks = B->tile ? NQUEUE * (int)most : 0;
}

int ensure_items_cap(dugks_batch* B, size_t n, hipStream_t s) {
  if (n <= B->items_cap) return DUGKS_OK;
  // in-flight steps may still read the old list
  if (hipStreamSynchronize(s) != hipSuccess) return DUGKS_EDEVICE;
  if (B->d_items) (void)hipFree(B->d_items);
  B->d_items = nullptr;
  B->items_cap = 0;
  size_t cap = std::max<size_t>(n, 2 * n);
  if (hipMalloc(&B->d_items, cap * sizeof(BatchItem)) != hipSuccess) return DUGKS_EDEVICE;
  B->items_cap = cap;
  return DUGKS_OK;
}

// Copy the descriptor table, the changed step counters and the work list to
// the device (asynchronous, through the pinned staging ring).
template <typename T>
int upload(dugks_batch* B, hipStream_t s) {
  int rc = ensure_items_cap(B, std::max<size_t>(B->items.size(), 1), s);
  if (rc) return rc;
  const size_t off_desc = 256;
  const size_t off_steps = align_up(off_desc + B->cap * sizeof(GridDesc<T>), 256);
  const size_t off_status = align_up(off_steps + B->cap * sizeof(SlotStep), 256);
  const size_t off_items = align_up(off_status + B->cap * sizeof(int32_t), 256);
  const size_t need = off_items + B->items.size() * sizeof(BatchItem);
  const int j = B->stage_next;
  B->stage_next = (j + 1) % NSTAGE;
  if (hipEventSynchronize(B->stage_ev[j]) != hipSuccess) return DUGKS_EDEVICE;
  if (B->stage_bytes[j] < need) {
    if (B->stage[j]) (void)hipHostFree(B->stage[j]);
    B->stage[j] = nullptr;
    B->stage_bytes[j] = 0;
    if (hipHostMalloc(&B->stage[j], 2 * need, hipHostMallocDefault) != hipSuccess)
      return DUGKS_EDEVICE;
    B->stage_bytes[j] = 2 * need;
  }
  char* h = static_cast<char*>(B->stage[j]);
  BatchCtl* ctl = reinterpret_cast<BatchCtl*>(h);
  ctl->items = B->d_items;
  ctl->nitems = (int32_t)B->items.size();
  ctl->nq = B->nq;
  for (int q = 0; q <= NQUEUE; q++)
    ctl->qstart[q] = q < (int)B->qstart.size() ? B->qstart[q] : ctl->nitems;
  hipError_t e;
  if ((e = hipMemcpyAsync(B->d_ctl, ctl, sizeof(BatchCtl), hipMemcpyHostToDevice, s)))
    return hip_status(e);
  if (B->desc_dirty) {
    GridDesc<T>* dt = reinterpret_cast<GridDesc<T>*>(h + off_desc);
    for (int k = 0; k < B->cap; k++)
      dt[k] = make_desc<T>(B->slots[k], B->tile ? B->tile : B->rows);
    if ((e = hipMemcpyAsync(B->d_desc, dt, B->cap * sizeof(GridDesc<T>), hipMemcpyHostToDevice,
                            s)))
      return hip_status(e);
    B->desc_dirty = false;
  }
  SlotStep* st = reinterpret_cast<SlotStep*>(h + off_steps);
  int32_t* ss = reinterpret_cast<int32_t*>(h + off_status);
  for (int k = 0; k < B->cap; k++) {
    Slot& sl = B->slots[k];
    if (!sl.step_dirty) continue;
    st[k].n = sl.step;
    st[k].target = sl.target;
    ss[k] = DUGKS_OK;   // a newly attached (or cleared) slot has no status yet
    if ((e = hipMemcpyAsync(B->d_steps + k, st + k, sizeof(SlotStep), hipMemcpyHostToDevice,
                            s)) ||
        (e = hipMemcpyAsync(B->d_status + k, ss + k, sizeof(int32_t), hipMemcpyHostToDevice, s)))
      return hip_status(e);
    sl.step_dirty = false;
  }
  if (!B->items.empty()) {
    BatchItem* it = reinterpret_cast<BatchItem*>(h + off_items);
    memcpy(it, B->items.data(), B->items.size() * sizeof(BatchItem));
    if ((e = hipMemcpyAsync(B->d_items, it, B->items.size() * sizeof(BatchItem),
                            hipMemcpyHostToDevice, s)))
      return hip_status(e);
  }
  return hip_status(hipEventRecord(B->stage_ev[j], s));
}

// finish = false: the step kernel alone, which writes only the next-step
// buffers and mass partials of each active slot (used to time tilings; the
// state is unchanged, since the finish kernel never runs)
int batch_launch(dugks_batch* B, hipStream_t s, bool finish, int blocks) {
  const BatchDev D{B->d_desc, B->d_steps, B->d_status, B->d_ctl, B->d_head, B->cap,
                   B->grid_blocks, B->tile, blocks};
  return launch_batch(D, B->precision, B->recon, B->mfix, B->scheme, s, finish);
}

// The kind and height of the tiles.  Where the caller has given none, as for one
// grid (see default_tile_rows and tile_kernel_default in dugks_abi.hip), by the
// number of 16-row marching tiles of all grids together; 8 rows where those still
// make one round (24 of a mix of FP32 grids: 45.5 us a step against 52.3 at 16).  A
// batch too small to fill the chip is bound by one tile's latency: us per step with
// 64-row marching tiles / now, FP32 corrected: one 64^2 grid 164 / 12.5, eight 128^2
// 176 / 16.6, 16 grids of sides 32-512 178 / 39; 64 of them 175 / 76, 256 239 / 211.
// A given height of 8 asks for block tiles; of more grids than those are good for it
// is marched (256 grids of the mix, block tiles / march: FP32 corrected 416 / 340, FP64
// 598 / 535).
void choose_tiles(dugks_batch* B) {
  auto count = [B](int rows) {
    int64_t n = 0;
    for (const Slot& s : B->slots)
      if (s.plan) n += (int64_t)s.plan->nstrips * ((s.plan->p.ny + rows - 1) / rows);
    return n;
  };
  const int rows0 = B->rows, tile0 = B->tile;
  const int64_t n16 = count(16);
  const bool block = (!B->given || B->given_tile) &&
                     n16 <= batch_tile_limit(B->precision, B->recon, B->scheme);
  B->tile = block ? block_tile_rows(B->precision == DUGKS_F64 ? 8 : 4, B->recon, B->scheme,
                                    B->mfix, count(4))
                  : 0;
  if (!B->given) {
    B->rows = count(8) <= B->grid_blocks ? 8 : 16;
    if (n16 > B->grid_blocks && n16 < 2 * (int64_t)B->grid_blocks)
      while (B->rows < 256 && count(B->rows) > B->grid_blocks) B->rows += MASS_GROUP;
  }
  if (B->rows != rows0 || B->tile != tile0) B->desc_dirty = true;
}

int commit(dugks_batch* B, hipStream_t s) {
  choose_tiles(B);
  build_items(B, B->tile ? B->tile : B->rows);
  return B->precision == DUGKS_F64 ? upload<double>(B, s) : upload<float>(B, s);
}

void drop(const dugks_batch::Retired& r) {
  (void)hipGraphExecDestroy(r.exec);
  (void)hipGraphDestroy(r.graph);
  if (r.over) (void)hipEventDestroy(r.over);
}

// A graph is replaced while its last replay may be running (work list and steps
// are only queued), and an executable graph has to outlive its replays: kept
// until an event behind them on `s` has passed (batch calls follow one another
// in stream order).  Under a capture of the caller's, until the batch goes.  At
// most RETIRED_MAX wait, then the oldest is waited for.
constexpr size_t RETIRED_MAX = 16;
void retire(dugks_batch* B, dugks_batch::Graph* G, hipStream_t s) {
  dugks_batch::Retired r{G->graph, G->exec, nullptr};
  G->exec = nullptr;
  G->graph = nullptr;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
  if (hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
      hipEventCreateWithFlags(&r.over, hipEventDisableTiming) == hipSuccess &&
      hipEventRecord(r.over, s) != hipSuccess) {
    (void)hipEventDestroy(r.over);
    r.over = nullptr;
  }
  B->retired.push_back(r);
  std::vector<dugks_batch::Retired> keep;
  size_t waiting = 0;
  for (const auto& o : B->retired) waiting += o.over != nullptr;
  for (const auto& o : B->retired) {
    if (o.over && (hipEventQuery(o.over) == hipSuccess ||
                   (waiting > RETIRED_MAX && hipEventSynchronize(o.over) == hipSuccess))) {
      drop(o);
      waiting--;
    } else {
      keep.push_back(o);
    }
  }
  B->retired.swap(keep);
}

void release(dugks_batch* B) {
  for (const auto& r : B->retired) drop(r);
  for (dugks_batch::Graph& g : B->graphs) {
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
  }
  if (B->cap_stream) (void)hipStreamDestroy(B->cap_stream);
  for (int j = 0; j < NSTAGE; j++) {
    if (B->stage_ev[j]) {
      (void)hipEventSynchronize(B->stage_ev[j]);
      (void)hipEventDestroy(B->stage_ev[j]);
    }
    if (B->stage[j]) (void)hipHostFree(B->stage[j]);
  }
  if (B->d_items) (void)hipFree(B->d_items);
  if (B->d_desc) (void)hipFree(B->d_desc);
  if (B->d_steps) (void)hipFree(B->d_steps);
  if (B->d_status) (void)hipFree(B->d_status);
  if (B->d_ctl) (void)hipFree(B->d_ctl);
  if (B->d_head) (void)hipFree(B->d_head);
}

// The graph of k steps over the kind of tiles the list holds.  A graph's tile
// kernels have a power of two of blocks per queue, so that it is captured again
// only when the list has outgrown it.
int capture_graph(dugks_batch* B, int k, hipStream_t s, hipGraphExec_t* exec) {
  dugks_batch::Graph& G = B->graphs[B->tile / 4];
  *exec = G.exec;
  if (G.exec && G.k == k && G.blocks >= B->tile_blocks) return DUGKS_OK;
  if (G.exec) retire(B, &G, s);
  if (hipStreamBeginCapture(B->cap_stream, hipStreamCaptureModeRelaxed) != hipSuccess)
    return DUGKS_EDEVICE;
  int rc = DUGKS_OK;
  G.blocks = NQUEUE;
  while (G.blocks < B->tile_blocks) G.blocks *= 2;
  for (int j = 0; j < k && rc == DUGKS_OK; j++)
    rc = batch_launch(B, B->cap_stream, true, G.blocks);
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(B->cap_stream, &g);
  if (rc || e != hipSuccess || !g) {
    if (g) (void)hipGraphDestroy(g);
    return DUGKS_EDEVICE;
  }
  G.graph = g;
  if (hipGraphInstantiate(&G.exec, g, nullptr, nullptr, 0) != hipSuccess) {
    (void)hipGraphDestroy(g);
    G.exec = nullptr;
    G.graph = nullptr;
    return DUGKS_EDEVICE;
  }
  G.k = k;
  *exec = G.exec;
  return DUGKS_OK;
}

}  // namespace

// ================================================================== C ABI
extern "C" {

int dugks_batch_create(int32_t capacity, int32_t precision, int32_t recon, uint32_t flags,
                       dugks_batch** out) {
  if (!out) return DUGKS_EINVAL;
  *out = nullptr;
  if (capacity < 1 || capacity > 65536 || precision < 0 || precision > 1 || recon < 0 ||
      recon > 3 || (flags & ~(DUGKS_FLAG_MASS_FIX | DUGKS_BATCH_T3S3)))
    return DUGKS_EINVAL;
  if (recon == DUGKS_UPWIND5) return DUGKS_EUNSUPPORTED;   // single grids only
  dugks_batch* B = new (std::nothrow) dugks_batch();
  if (!B) return DUGKS_ENOMEM;
  B->cap = capacity;
  B->precision = precision;
  B->recon = recon;
  B->mfix = (flags & DUGKS_FLAG_MASS_FIX) != 0;
  B->scheme = (flags & DUGKS_BATCH_T3S3) ? DUGKS_T3S3 : DUGKS_T2;
  B->slots.resize(capacity);
  B->desc_bytes = precision == DUGKS_F64 ? sizeof(GridDesc<double>) : sizeof(GridDesc<float>);
  int rc = DUGKS_OK;
  int per_cu = 0, ncu = 0;
  if (hipGetDevice(&B->device) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, B->device) !=
          hipSuccess ||
      (rc = batch_occupancy(B->precision, B->recon, B->mfix, B->scheme, &per_cu)) !=
          DUGKS_OK ||
      per_cu < 1 || ncu < 1 ||
      hipMalloc(&B->d_desc, capacity * B->desc_bytes) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&B->d_steps), capacity * sizeof(SlotStep)) !=
          hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&B->d_status), capacity * sizeof(int32_t)) !=
          hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&B->d_ctl), sizeof(BatchCtl)) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&B->d_head), HEAD_BYTES) != hipSuccess ||
      hipMemset(B->d_desc, 0, capacity * B->desc_bytes) != hipSuccess ||
      hipMemset(B->d_steps, 0, capacity * sizeof(SlotStep)) != hipSuccess ||
      hipMemset(B->d_status, 0, capacity * sizeof(int32_t)) != hipSuccess ||
      hipMemset(B->d_ctl, 0, sizeof(BatchCtl)) != hipSuccess ||
      hipMemset(B->d_head, 0, HEAD_BYTES) != hipSuccess ||
      hipStreamCreateWithFlags(&B->cap_stream, hipStreamNonBlocking) != hipSuccess) {
    release(B);
    delete B;
    return rc ? rc : DUGKS_EDEVICE;
  }
  for (int j = 0; j < NSTAGE; j++)
    if (hipEventCreateWithFlags(&B->stage_ev[j], hipEventDisableTiming) != hipSuccess) {
      release(B);
      delete B;
      return DUGKS_EDEVICE;
    }
  if (hipDeviceSynchronize() != hipSuccess) {
    release(B);
    delete B;
    return DUGKS_EDEVICE;
  }
  B->grid_blocks = per_cu * ncu;
  *out = B;
  return DUGKS_OK;
}

void dugks_batch_destroy(dugks_batch* batch) {
  if (!batch) return;
  (void)hipDeviceSynchronize();
  release(batch);
  delete batch;
}

int dugks_batch_set(dugks_batch* batch, int32_t slot, const dugks_plan* plan, void* state,
                    int64_t step, int64_t target) {
  if (!batch || slot < 0 || slot >= batch->cap || !plan || !state || !aligned(state) ||
      step < 0 || target < step)
    return DUGKS_EINVAL;
  if (plan->p.precision != batch->precision || plan->p.recon != batch->recon ||
      ((plan->p.flags & DUGKS_FLAG_MASS_FIX) != 0) != batch->mfix ||
      plan->p.scheme != batch->scheme)
    return DUGKS_EINVAL;
  if (plan->p.vel_kind == DUGKS_VEL_ARRAYS) return DUGKS_EUNSUPPORTED;
  Slot& s = batch->slots[slot];
  s.plan = plan;
  s.state = state;
  s.step = step;
  s.target = target;
  s.until = target - step > INT64_MAX - batch->done ? INT64_MAX : batch->done + (target - step);
  s.step_dirty = true;
  batch->desc_dirty = true;
  return DUGKS_OK;
}

int dugks_batch_clear(dugks_batch* batch, int32_t slot) {
  if (!batch || slot < 0 || slot >= batch->cap) return DUGKS_EINVAL;
  Slot& s = batch->slots[slot];
  s = Slot();
  s.step_dirty = true;   // (n, target) = (0, 0): idle
  batch->desc_dirty = true;
  return DUGKS_OK;
}

int dugks_batch_commit(dugks_batch* batch, void* stream) {
  if (!batch) return DUGKS_EINVAL;
  return commit(batch, static_cast<hipStream_t>(stream));
}

int dugks_batch_step(dugks_batch* batch, int64_t nsteps, int32_t graph_steps, void* stream) {
  if (!batch || nsteps < 0 || graph_steps < 0 || graph_steps > 4096) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  int64_t left = nsteps;
  if (graph_steps > 1 && nsteps >= graph_steps) {
    hipGraphExec_t exec = nullptr;
    int rc = capture_graph(batch, graph_steps, s, &exec);
    if (rc) return rc;
    for (; left >= graph_steps; left -= graph_steps) {
      if (hipGraphLaunch(exec, s) != hipSuccess) return DUGKS_EDEVICE;
      batch->done += graph_steps;
    }
  }
  for (; left > 0; left--) {
    int rc = batch_launch(batch, s, true, batch->tile_blocks);
    if (rc) return rc;
    batch->done++;
  }
  return DUGKS_OK;
}

int dugks_batch_steps(const dugks_batch* batch, int64_t* out, void* stream) {
  if (!batch || !out) return DUGKS_EINVAL;
  return hip_status(hipMemcpyAsync(out, batch->d_steps, batch->cap * sizeof(SlotStep),
                                   hipMemcpyDefault, static_cast<hipStream_t>(stream)));
}

int dugks_batch_status(const dugks_batch* batch, int32_t* out, void* stream) {
  if (!batch || !out) return DUGKS_EINVAL;
  return hip_status(hipMemcpyAsync(out, batch->d_status, batch->cap * sizeof(int32_t),
                                   hipMemcpyDefault, static_cast<hipStream_t>(stream)));
}

int dugks_batch_tile_rows(const dugks_batch* batch) { return batch ? batch->rows : -1; }

int dugks_batch_set_tile_rows(dugks_batch* batch, int32_t rows) {
  if (!batch || rows < MASS_GROUP || rows > 65536 || rows % MASS_GROUP) return DUGKS_EINVAL;
  batch->rows = rows;
  batch->given = true;
  batch->given_tile = rows <= TILE_MAX_ROWS;
  batch->desc_dirty = true;
  return DUGKS_OK;
}

int dugks_batch_tune(dugks_batch* batch, int32_t reps, int32_t* rows_out, void* stream) {
  if (!batch || reps < 1 || reps > 1000) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return DUGKS_EDEVICE;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return DUGKS_EDEVICE;
  }
  int rc = DUGKS_OK;
  const int rows0 = batch->rows;
  const bool given0 = batch->given, given_tile0 = batch->given_tile;
  // the batch's own choice first, then the heights of the march
  float own_ms = -1.0f, best_ms = -1.0f;
  int own = 0, best = rows0;
  bool own_tile = false;
  for (int rows : TUNE_ROWS) {
    batch->given = rows != 0;
    batch->given_tile = false;
    if (rows) batch->rows = rows;
    batch->desc_dirty = true;
    if ((rc = commit(batch, s))) break;
    // one untimed pass, then the timed passes
    if ((rc = batch_launch(batch, s, false, batch->tile_blocks))) break;
    // the step kernels alone leave the queue heads at their ends: rewind them
    if (hipMemsetAsync(batch->d_head, 0, HEAD_BYTES, s) != hipSuccess) {
      rc = DUGKS_EDEVICE;
      break;
    }
    (void)hipEventRecord(e0, s);
    for (int r = 0; r < reps && rc == DUGKS_OK; r++) {
      rc = batch_launch(batch, s, false, batch->tile_blocks);
      if (!rc && hipMemsetAsync(batch->d_head, 0, HEAD_BYTES, s) != hipSuccess)
        rc = DUGKS_EDEVICE;
    }
    (void)hipEventRecord(e1, s);
    if (rc || hipEventSynchronize(e1) != hipSuccess) {
      rc = rc ? rc : DUGKS_EDEVICE;
      break;
    }
    float ms = 0.0f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    if (!rows) {
      own_ms = ms;
      own_tile = batch->tile != 0;
      own = batch->rows;
    } else if (best_ms < 0.0f || ms < best_ms) {
      best_ms = ms;
      best = rows;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) {   // as it was
    batch->rows = rows0;
    batch->given = given0;
    batch->given_tile = given_tile0;
  } else {
    batch->given = true;
    batch->given_tile = own_tile && own_ms <= best_ms;
    batch->rows = !own_tile && own_ms <= best_ms ? own : best;
    best = batch->rows;
  }
  batch->desc_dirty = true;
  int rc2 = commit(batch, s);
  if (!rc) rc = rc2;
  if (!rc && rows_out) *rows_out = best;
  return rc;
}

}  // extern "C"
