// dugks_noalloc.hip -- dugks_step_many_noalloc (include/dugks.h): the batch
// step of many grids for callers that cannot allocate device memory.  It runs
// the batch kernels of dugks_batch.hip; what a batch keeps in device memory of
// its own lives here in one fixed file-scope device array per GPU.
#include <string.h>

#include <algorithm>
#include <mutex>

#include "dugks_batch_impl.h"
#include "dugks_common.h"
#include "dugks_kernels.h"
#include "dugks_plan.h"

using namespace dugks;

namespace {

// dugks_step_many_noalloc keeps what a batch keeps in its own device memory --
// descriptors, step counters, slot status, the work list and its control block
// with the queue heads -- in one file-scope device array of NOALLOC_BYTES per
// GPU, filled by small set-up kernels whose inputs travel as kernel arguments
// (no host staging buffer, no allocation).  Layout of the array:
constexpr int NOALLOC_GRIDS = 256;
constexpr size_t NOALLOC_BYTES = size_t(1) << 20;
constexpr size_t NA_CTL = 0, NA_HEAD = 256, NA_STEPS = NA_HEAD + HEAD_BYTES;
constexpr size_t NA_STATUS = NA_STEPS + NOALLOC_GRIDS * sizeof(SlotStep);
constexpr size_t NA_DESC = (NA_STATUS + NOALLOC_GRIDS * sizeof(int32_t) + 255) / 256 * 256;
constexpr size_t NA_ITEMS =
    (NA_DESC + NOALLOC_GRIDS * sizeof(GridDesc<double>) + 255) / 256 * 256;
constexpr int64_t NOALLOC_ITEMS = (int64_t)((NOALLOC_BYTES - NA_ITEMS) / sizeof(BatchItem));
static_assert(sizeof(GridDesc<double>) >= sizeof(GridDesc<float>), "descriptor sizes");
static_assert(NOALLOC_ITEMS == 115680, "the limit include/dugks.h states");
static_assert(sizeof(BatchCtl) <= NA_HEAD - NA_CTL, "control block");
static_assert(NA_STEPS % 256 == 0, "alignment");

// descriptors of up to DESC_CHUNK grids, by value
constexpr int DESC_CHUNK = 8;
template <typename T>
struct DescChunk {
  GridDesc<T> d[DESC_CHUNK];
  SlotStep st[DESC_CHUNK];
  int first, count;
};
static_assert(sizeof(DescChunk<double>) <= 4096, "kernel argument size");

template <typename T>
__global__ __launch_bounds__(64) void noalloc_desc_kernel(DescChunk<T> c, unsigned char* base) {
  const int k = threadIdx.x;
  if (k >= c.count) return;
  GridDesc<T>* desc = reinterpret_cast<GridDesc<T>*>(base + NA_DESC);
  SlotStep* steps = reinterpret_cast<SlotStep*>(base + NA_STEPS);
  int32_t* status = reinterpret_cast<int32_t*>(base + NA_STATUS);
  desc[c.first + k] = c.d[k];
  steps[c.first + k] = c.st[k];
  status[c.first + k] = DUGKS_OK;
}

// the work list, in pieces: item i of piece p (start[p] <= i < start[p + 1]) is
// tile first[p] + i - start[p] of grid[p]; queue q holds items [qstart[q],
// qstart[q + 1]).  A grid is one piece, or one per queue it reaches into.  One
// thread also writes the control block and rewinds the queue heads
constexpr int NOALLOC_PIECES = NOALLOC_GRIDS + NQUEUE - 1;
struct ItemPieces {
  int32_t qstart[NQUEUE + 1];
  int32_t n;
  int32_t start[NOALLOC_PIECES + 1];
  int32_t grid[NOALLOC_PIECES];
  int32_t first[NOALLOC_PIECES];
};
static_assert(sizeof(ItemPieces) <= 4096, "kernel argument size");

static __global__ __launch_bounds__(256) void noalloc_items_kernel(ItemPieces a,
                                                                   unsigned char* base) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int nitems = a.start[a.n];
  BatchItem* items = reinterpret_cast<BatchItem*>(base + NA_ITEMS);
  if (i == 0) {
    BatchCtl* ctl = reinterpret_cast<BatchCtl*>(base + NA_CTL);
    ctl->items = items;
    ctl->nitems = nitems;
    ctl->nq = NQUEUE;
    for (int q = 0; q <= NQUEUE; q++) ctl->qstart[q] = a.qstart[q];
    unsigned* head = reinterpret_cast<unsigned*>(base + NA_HEAD);
    for (int q = 0; q < NQUEUE; q++) head[q * HEAD_STRIDE] = head[q * HEAD_STRIDE + 1] = 0u;
  }
  if (i >= nitems) return;
  int lo = 0, hi = a.n - 1;   // last p with start[p] <= i
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (a.start[mid] <= i) lo = mid; else hi = mid - 1;
  }
  items[i] = BatchItem{a.grid[lo], (int32_t)(a.first[lo] + i - a.start[lo])};
}

struct GridTiles {
  int j, cost;       // the grid, the cost of a tile
  int64_t tiles;
};

// Grids (the largest first) whole to the least loaded queue each, if no queue gets
// more blocks than an XCD has compute units: the tiles' shared rows and columns
// stay in one L2, and every block runs at once (see make_pieces).
bool whole_grids(const GridTiles* g, int n, int* queue_of) {
  int64_t load[NQUEUE] = {};
  for (int k = 0; k < n; k++) {
    const int q = (int)(std::min_element(load, load + NQUEUE) - load);
    queue_of[k] = q;
    if ((load[q] += g[k].tiles) > 32) return false;
  }
  return true;
}

// The work list of n grids in block tiles of `tile` rows, or (0) in marching
// tiles of each plan's many_rows.  The grids' tiles, those of the most marched
// rows first and each grid's segment by segment, are laid end to end and cut at
// NQUEUE equal shares (of tiles, or of marched rows), so that every XCD has the
// same work, however few or uneven the grids: a block of the tile kernel takes
// tiles of its XCD's queue only, and a marching wavefront tries one other.  Within
// a queue the taller tiles come first, so that the short ones fill the tail.
// us per step with every grid whole in one queue / now: one FP64 grid of 1000^2
// 326 / 57, of 2048^2 410 / 181, one corrected FP32 grid of 512^2 71 / 20, 1024^2
// with 63 of 32-512 136 / 112.  Grids whose blocks fit an XCD at once do stay
// whole: one 33^2 grid 9.7 / 10.8 (FP64 8.3 / 9.0), four of 64^2 10.6 / 11.1.
void make_pieces(const dugks_plan* const* plans, int n, int tile, ItemPieces* out) {
  GridTiles g[NOALLOC_GRIDS];
  int64_t total = 0;
  for (int j = 0; j < n; j++) {
    const dugks_plan* P = plans[j];
    const int segs = tile ? (P->p.ny + tile - 1) / tile : P->many_segs;
    g[j] = {j, tile ? 1 : P->many_rows + 5, (int64_t)P->nstrips * segs};
    total += g[j].tiles * g[j].cost;
  }
  std::stable_sort(g, g + n, [](const GridTiles& a, const GridTiles& b) {
    return a.tiles * a.cost > b.tiles * b.cost;
  });
  struct Piece {
    int32_t grid, first, count, cost;
  };
  Piece p[NOALLOC_PIECES];
  int np = 0, k = 0;
  int64_t items = 0, done = 0, taken = 0;   // taken: tiles of g[k] so far
  int queue_of[NOALLOC_GRIDS];
  const bool whole = tile && whole_grids(g, n, queue_of);
  for (int q = 0; q < NQUEUE; q++) {
    const int from = np;
    out->qstart[q] = (int32_t)items;
    for (int j = 0; whole && j < n; j++)
      if (queue_of[j] == q) {
        p[np++] = {g[j].j, 0, (int32_t)g[j].tiles, g[j].cost};
        items += g[j].tiles;
      }
    // up to the queue's share of the work (the last queue takes the rest)
    const int64_t upto = total * (q + 1) / NQUEUE;
    while (!whole && k < n) {
      const int64_t left = g[k].tiles - taken;
      const int64_t m = q == NQUEUE - 1 ? left : std::min(left, (upto - done) / g[k].cost);
      if (m > 0) {
        p[np++] = {g[k].j, (int32_t)taken, (int32_t)m, g[k].cost};
        items += m;
        done += m * g[k].cost;
        taken += m;
      }
      if (m < left) break;
      taken = 0;
      k++;
    }
    std::stable_sort(p + from, p + np,
                     [](const Piece& a, const Piece& b) { return a.cost > b.cost; });
  }
  out->qstart[NQUEUE] = (int32_t)items;
  out->n = np;
  out->start[0] = 0;
  for (int i = 0; i < np; i++) {
    out->grid[i] = p[i].grid;
    out->first[i] = p[i].first;
    out->start[i + 1] = out->start[i] + p[i].count;
  }
}

}  // namespace

// The array itself: one copy per GPU, held until the process ends.  Host code
// never passes its name to a kernel (that would be a host-side stand-in, not a
// device address); it uses the address hipGetSymbolAddress returns on each
// device.
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

namespace {

// the device address of `scratch` on each GPU (each holds its own copy),
// looked up once per device with that device current
constexpr int NOALLOC_MAX_DEVICES = 64;
std::once_flag g_scratch_once[NOALLOC_MAX_DEVICES];
unsigned char* g_scratch_ptr[NOALLOC_MAX_DEVICES];
int g_scratch_rc[NOALLOC_MAX_DEVICES];

int scratch_of_current_device(unsigned char** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return DUGKS_EDEVICE;
  if (dev >= NOALLOC_MAX_DEVICES) return DUGKS_EUNSUPPORTED;
  std::call_once(g_scratch_once[dev], [dev] {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
    g_scratch_rc[dev] = (e == hipSuccess && ptr) ? DUGKS_OK : DUGKS_EDEVICE;
  });
  *out = g_scratch_ptr[dev];
  return g_scratch_rc[dev];
}

template <typename T>
int noalloc_setup(const dugks_plan* const* plans, void* const* states, const int64_t* steps,
                  int n, int64_t nsteps, int tile, const ItemPieces& pieces,
                  unsigned char* base, hipStream_t s) {
  DescChunk<T> c;
  for (int first = 0; first < n; first += DESC_CHUNK) {
    memset(&c, 0, sizeof(c));
    c.first = first;
    c.count = std::min(DESC_CHUNK, n - first);
    for (int k = 0; k < c.count; k++) {
      const dugks_plan* P = plans[first + k];
      c.d[k] = make_grid_desc<T>(P, states[first + k], tile ? tile : P->many_rows);
      c.st[k].n = steps[first + k];
      c.st[k].target = steps[first + k] + nsteps;
    }
    hipLaunchKernelGGL((noalloc_desc_kernel<T>), dim3(1), dim3(64), 0, s, c, base);
  }
  const int nitems = pieces.qstart[NQUEUE];
  hipLaunchKernelGGL(noalloc_items_kernel, dim3((unsigned)((nitems + 255) / 256)), dim3(256),
                     0, s, pieces, base);
  return hip_status(hipGetLastError());
}

}  // namespace

extern "C" {

int dugks_step_many_noalloc(const dugks_plan* const* plans, void* const* states,
                            const int64_t* steps, int32_t n, int64_t nsteps, void* stream) {
  if (!plans || !states || !steps || n < 1 || n > NOALLOC_GRIDS || nsteps < 0)
    return DUGKS_EINVAL;
  const dugks_plan* p0 = plans[0];
  if (!p0) return DUGKS_EINVAL;
  const int precision = p0->p.precision, recon = p0->p.recon, scheme = p0->p.scheme;
  const bool mfix = (p0->p.flags & DUGKS_FLAG_MASS_FIX) != 0;
  for (int j = 0; j < n; j++) {
    const dugks_plan* P = plans[j];
    if (!P || !states[j] || !aligned(states[j]) || steps[j] < 0) return DUGKS_EINVAL;
    if (P->p.precision != precision || P->p.recon != recon || P->p.scheme != scheme ||
        ((P->p.flags & DUGKS_FLAG_MASS_FIX) != 0) != mfix)
      return DUGKS_EINVAL;
    if (P->p.vel_kind == DUGKS_VEL_ARRAYS || P->p.recon == DUGKS_UPWIND5)
      return DUGKS_EUNSUPPORTED;
  }
  // block tiles where the grids together are too few to fill the chip with
  // marching wavefronts (as a batch chooses them), else each plan's own height
  int64_t n16 = 0, n4 = 0;
  for (int j = 0; j < n; j++) {
    n16 += (int64_t)plans[j]->nstrips * ((plans[j]->p.ny + 15) / 16);
    n4 += (int64_t)plans[j]->nstrips * ((plans[j]->p.ny + 3) / 4);
  }
  const int tile = n16 <= batch_tile_limit(precision, recon, scheme)
                       ? block_tile_rows(precision == DUGKS_F64 ? 8 : 4, recon, scheme, mfix, n4)
                       : 0;
  int64_t total = 0, items = 0;
  for (int j = 0; j < n; j++) {
    const dugks_plan* P = plans[j];
    total += (int64_t)P->nstrips * P->many_limit_segs;
    items += (int64_t)P->nstrips * (tile ? (P->p.ny + tile - 1) / tile : P->many_segs);
    if (std::max(total, items) > NOALLOC_ITEMS) return DUGKS_EINVAL;   // beyond the work list
  }
  if (nsteps == 0) return DUGKS_OK;
  unsigned char* base = nullptr;
  int rc = scratch_of_current_device(&base);
  if (rc) return rc;
  int dev = 0, ncu = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return DUGKS_EDEVICE;
  if ((rc = batch_occupancy(precision, recon, mfix, scheme, &per_cu)) != DUGKS_OK) return rc;
  if (per_cu < 1 || ncu < 1) return DUGKS_EDEVICE;
  ItemPieces pieces;
  memset(&pieces, 0, sizeof(pieces));
  make_pieces(plans, n, tile, &pieces);
  int longest = 1;
  for (int k = 0; k < NQUEUE; k++)
    longest = std::max(longest, pieces.qstart[k + 1] - pieces.qstart[k]);
  hipStream_t s = static_cast<hipStream_t>(stream);
  rc = precision == DUGKS_F64
           ? noalloc_setup<double>(plans, states, steps, n, nsteps, tile, pieces, base, s)
           : noalloc_setup<float>(plans, states, steps, n, nsteps, tile, pieces, base, s);
  if (rc) return rc;
  const BatchDev D{base + NA_DESC,
                   reinterpret_cast<SlotStep*>(base + NA_STEPS),
                   reinterpret_cast<int32_t*>(base + NA_STATUS),
                   reinterpret_cast<BatchCtl*>(base + NA_CTL),
                   reinterpret_cast<unsigned*>(base + NA_HEAD),
                   n,
                   per_cu * ncu,
                   tile,
                   NQUEUE * longest};
  for (int64_t k = 0; k < nsteps; k++)
    if ((rc = launch_batch(D, precision, recon, mfix, scheme, s, true))) return rc;
  return DUGKS_OK;
}

}  // extern "C"
