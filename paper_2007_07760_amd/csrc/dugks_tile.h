// dugks_tile.h -- the step of a small grid: one block of wavefronts per tile,
// one wavefront per cell row (arXiv 2007.07760, Sec. II).
//
// A grid that cannot fill the chip with marching wavefronts (step_kernel) is
// bound by the march's serial chain: a 16-row tile takes 21 rows in turn, ~35
// us in FP64, whatever the grid's size.  Here the rows of a tile run side by
// side: wavefront w of a block forms phi, the cell terms and fbar+ of cell row
// y0 - LAG + w, then the faces of that row and its update, with four block
// barriers between (differences of phi; fbar+ rows; faces; the faces' values
// below each row).  What bounds it is that chain of latencies: 5.2-6.7 us per
// step for grids of up to 256 tiles (64^2 FP64: 36 us with the march, 6.0 now;
// 256^2 8.6; FP32 corrected 256^2 with its reduction 37.7, 9.2; upwind-5 64^2
// 79, 8.7): a wavefront issues for a quarter of its life there and waits for
// loads, LDS and barriers for most of the rest.  On larger grids VALU (a third
// of it lane shifts) is busy half the time, and TR rows take the cell terms of
// TR + 4 (6), so the march wins from ~800^2 on, upwind-5 from ~1400^2 (corrected
// FP64 from ~500^2; see tile_kernel_default; the rows of a tile: block_tile_rows).
//
// Two stages in one launch (two T2 steps, or both of T3S3's) were slower: per
// step 64^2 6.2 us against 6.0, 200^2 7.8 against 6.7, T3S3 200^2 15.8 against
// 14.0.  A step waits for its own chain, not for the launch.
//
// The arithmetic is the march's, expression by expression, so the results are
// bitwise the same.  The face values take their neighbour columns from lane
// shifts of one LDS read per row: reading every tap from LDS needed 224
// registers in FP64, this 80, which leaves room for 24 wavefronts per compute
// unit (three blocks of 4-row tiles or two of 8).  For that, values that are
// needed again only after the faces are re-read then (s from LDS, the face
// velocities from their table), and the north faces' values go to rows of fbar+
// that no update needs (768^2 FP64 38.9 -> 33.0 us with 8-row tiles; T3S3
// 104 -> 89).
#pragma once

#include "dugks_common.h"
#include "dugks_kernels.h"

namespace dugks {

// the face values of row k, velocity by velocity from I on: pn of the north
// faces, de of the east less the west ones, and their sums over the velocities
template <bool EAST, int I = 0, typename M, typename T>
__device__ __forceinline__ void faces(const M& m, int k, T (&pn)[9], T (&de)[9], T& phN, T& phE) {
  T pe;
  m.template recon_pair<I, EAST>(k, pn[I], pe);
  phN += pn[I];
  if constexpr (EAST) {
    phE += pe;
    if constexpr (ex(I) != 0) de[I] = pe - from_left(pe);
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (I < 8) faces<EAST, I + 1>(m, k, pn, de, phN, phE);
}

template <typename T, int R, bool MFIX, int TR>
struct TileShared {
  static constexpr int CR = tile_cell_rows(R, TR);
  static_assert(!MFIX || TR == MASS_GROUP, "a tile of a corrected plan is one mass group");
  T bfp[CR][9][LANES];          // fbar+ of the cell rows; then the north faces
  // one buffer, in turn: the row differences phi(x+1) - phi(x-1) and
  // phi(x-1) + 4 phi + phi(x+1); s of the cell rows; the mass sums of the rows
  union {
    T da[CR + 2][2][LANES];
    T s[CR][2][LANES];
    struct {
      double sum[MFIX ? TR : 1][LANES];
      int fit[MFIX ? TR : 1][LANES];
    } mass;
  };
  double red[MFIX ? 2 * CR + 2 : 1];   // sums of the strips, the correction (see fix_inline)
};

// The mass correction from the partials of the last step, by every block: strip
// w by wavefront w, then the strips by the first, in the order of
// mass_fix_strips_kernel (the same bits).  Its loads are in flight with those of
// the rows, so a step pays the sums (~1 us) and not another launch (5.2 us):
// FP32 corrected 256^2 12.4 -> 9.2 us, 64^2 11.9 -> 8.0.  For up to CR strips and 64 groups each
// (fix_inline): the sums are done by every block again.
template <int CR>
__device__ __forceinline__ void block_fix(const double* __restrict__ prev, int nstrips,
                                          int ngroups, double ncells, bool first,
                                          StateHeader* __restrict__ hdr, double* red,
                                          double& pend, double& fitmax) {
  const int lane = threadIdx.x & (LANES - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
  const double mass0 = hdr->mass0;
  double m, c;
  if (w < nstrips) {
    wave_pair_sum(prev + 2 * (int64_t)w * ngroups, ngroups, m, c);
    if (lane == 0) {
      red[2 * w] = m;
      red[2 * w + 1] = c;
    }
  }
  __syncthreads();
  if (w == 0) {
    wave_pair_sum(red, nstrips, m, c);
    if (lane == 0) {
      mass_fix_values(mass0, m, c, ncells, red[2 * CR], red[2 * CR + 1]);
      if (first && !isfinite(m)) hdr->status = DUGKS_ENUMERIC;
    }
  }
  __syncthreads();
  pend = red[2 * CR];
  fitmax = red[2 * CR + 1];
}

// One tile by the whole block: rows [seg * TR, seg * TR + TR) of `strip`, step
// n; the arguments are march_tile's, and prev: the partials of the last step, if
// the correction is still to be formed from them (see block_fix).
template <typename T, int R, bool MFIX, int STAGE, bool VARR, int TR, typename Args>
__device__ __forceinline__ void tile_step(Args& a, int64_t n,
                                          const T* __restrict__ src, T* __restrict__ dst,
                                          T* __restrict__ dst2, const T* __restrict__ aux,
                                          const T* __restrict__ cf, const T* __restrict__ tabx,
                                          const T* __restrict__ taby, const T* __restrict__ uv,
                                          double* __restrict__ part, double pend, double fitmax,
                                          int strip, int seg, const double* __restrict__ prev,
                                          StateHeader* __restrict__ hdr,
                                          TileShared<T, R, MFIX, TR>& u) {
  constexpr int CR = tile_cell_rows(R, TR);
  using M = Marcher<T, R, MFIX, STAGE, VARR, CR, Args&>;
  constexpr int LAG = M::LAG;
  const int lane = threadIdx.x & (LANES - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);

  M m{a, src, as_const(cf), tabx, as_const(taby), uv, u.bfp};
  m.place(lane, strip, seg * TR, TR, dst, dst2, aux, part, pend, fitmax);
  m.base = m.y0 - LAG;
  // the cell row of this wavefront; the last tile may hold fewer rows, the
  // wavefronts beyond what it needs load its top row and write nothing
  const int top = m.y1 + LAG - 1;
  const int r = m.y0 - LAG + w;
  const bool cells = r <= top;
  const int k = r;                                  // its face row
  const bool upd = k >= m.y0 && k < m.y1;
  RowRegs<T> d, o;
  // touch the stencil table's scalar-cache lines (64 bytes) and the row's
  // velocity factors now: the cache is cold at every launch, and their first
  // misses would otherwise come one by one in the face stage
  constexpr int LINES = (4 * cclass(R) * (int)sizeof(T) + 63) / 64;
  T warm[LINES + 2];
#pragma unroll
  for (int j = 0; j < LINES; j++) warm[j] = m.cf[j * (64 / (int)sizeof(T))];
  if (!VARR) {
    warm[LINES] = m.taby[2 * wrapi(min(r, top), a.ny) + 1];
    warm[LINES + 1] = m.taby[(2 * a.ny + 2) + 2 * wrapi(min(r, top), a.ny) + 1];
  } else {
    warm[LINES] = warm[LINES + 1] = T(0);
  }
  __builtin_amdgcn_sched_barrier(0);
  m.load_raw(d, min(r, top + 1));
  const bool outer = w == 0 || w == CR - 1;
  if (outer) m.load_raw(o, w == 0 ? m.y0 - LAG - 1 : min(r + 1, top + 1));
  T qv[10];
  if (STAGE == STAGE_B && upd) m.load_q(k, qv);
  m.flow(n);
  constexpr bool LEAN = sizeof(T) == 8;
  if (!LEAN) m.flow_east();
  if (M::FIX_LOAD) {
    if (prev) {
      block_fix<CR>(prev, a.nstrips, a.ngroups, (double)a.nx * (double)a.ny,
                    strip == 0 && seg == 0, hdr, u.red, pend, fitmax);
      m.set_fix(pend, fitmax);
    }
    m.fix_row(d);
    if (outer) m.fix_row(o);
  }

  T p, D, A;
  m.phi_row(d, p, D, A);
  u.da[w + 1][0][lane] = D;
  u.da[w + 1][1][lane] = A;
  if (outer) {
    T po, Do, Ao;
    m.phi_row(o, po, Do, Ao);
    u.da[w == 0 ? 0 : CR + 1][0][lane] = Do;
    u.da[w == 0 ? 0 : CR + 1][1][lane] = Ao;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < LINES + 2; j++) asm volatile("" ::"s"(warm[j]));
  if (cells) {
    m.D0 = u.da[w][0][lane];
    m.A0 = u.da[w][1][lane];
    m.D1 = D;
    m.A1 = A;
    m.D2 = u.da[w + 2][0][lane];
    m.A2 = u.da[w + 2][1][lane];
    m.ph[LAG] = p;
    m.cell_stage(d, r);
  }
  __syncthreads();
  if (cells) {
    u.s[w][0][lane] = m.sxp[LAG];
    u.s[w][1][lane] = m.syp[LAG];
  }
  // faces: north ones of the rows y0 - 1 .. y1 - 1, east ones of the tile's rows
  const bool north = k >= m.y0 - 1 && k < m.y1;
  T pn[9], de[9], phN = T(0), phE = T(0);
  if (upd)
    faces<true>(m, k, pn, de, phN, phE);
  else if (north)
    faces<false>(m, k, pn, de, phN, phE);
  // no wavefront reads another's fbar+ row from here on: each leaves its north
  // faces (dt*alpha*fbar of the six crossing velocities, P, Q) in a row for the
  // row above -- of 4-row tiles one that no update needs, else its own, kept
  // in registers
  __syncthreads();
  const int kk = wrapi(k, a.ny);
  constexpr bool SPARE = 2 * LAG >= TR;
  auto face_row = [](int v) {   // of the wavefront v, LAG - 1 <= v < LAG - 1 + TR
    return !SPARE ? v : (v - (LAG - 1) < LAG ? v - (LAG - 1) : v - (LAG - 1) + TR);
  };
  T eP, eQx, eQy, PN, QNx, QNy;
  T bp[9];
  if (north) {
    // FP64: read again here, not held across the faces (6 wavefronts per SIMD)
    const T sx = LEAN ? u.s[w][0][lane] : m.sxp[LAG], sy = LEAN ? u.s[w][1][lane] : m.syp[LAG];
    if (LEAN) m.flow_east();
    T uk, vk;
    m.uv_row(kk, uk, vk);
    m.north_moments(kk, uk, vk, phN, sx, sy, u.s[w + 1][0][lane], u.s[w + 1][1][lane],
                    PN, QNx, QNy);
    if (!SPARE) {
#pragma unroll
      for (int i = 0; i < 9; i++) bp[i] = u.bfp[w][i][lane];
    }
    if (!SPARE || w < LAG - 1 + TR) {
      const int v = face_row(w);
#pragma unroll
      for (int i = 0; i < 9; i++)
        if (ey(i) != 0) u.bfp[v][i][lane] = pn[i];
      u.bfp[v][0][lane] = PN;
      u.bfp[v][1][lane] = QNx;
      u.bfp[v][5][lane] = QNy;
    }
    if (upd) m.east_moments(kk, uk, vk, phE, sx, sy, eP, eQx, eQy);
  }
  __syncthreads();
  if (upd) {
    T out[9];
    const int v = face_row(w - 1);
#pragma unroll
    for (int i = 0; i < 9; i++) {
      out[i] = T(0);
      if (ey(i) != 0) {
        const T dn = pn[i] - u.bfp[v][i][lane];
        out[i] = ey(i) > 0 ? -dn : dn;
      }
      if (ex(i) != 0) out[i] = ex(i) > 0 ? out[i] - de[i] : out[i] + de[i];
    }
    if (SPARE) {
#pragma unroll
      for (int i = 0; i < 9; i++) bp[i] = u.bfp[w][i][lane];
    }
    double cs = 0.0, cf0 = 0.0;
    m.update_cells(kk, bp, out, PN - u.bfp[v][0][lane], QNx - u.bfp[v][1][lane],
                   QNy - u.bfp[v][5][lane], eP, eQx, eQy, m.cp[LAG], m.cx[LAG], m.cy[LAG],
                   p, qv, cs, cf0);
    if (M::FIX_SUM) {
      u.mass.sum[MFIX ? k - m.y0 : 0][lane] = m.owned ? cs : 0.0;
      u.mass.fit[MFIX ? k - m.y0 : 0][lane] = cf0 != 0.0;
    }
  }
  if (M::FIX_SUM) {
    // the group's totals as the march forms them: each lane's rows in order,
    // then the lanes
    __syncthreads();
    if (w == 0) {
      double v = 0.0, c = 0.0;
      for (int j = 0; j < m.y1 - m.y0; j++) {
        v += u.mass.sum[MFIX ? j : 0][lane];
        c += u.mass.fit[MFIX ? j : 0][lane];
      }
      M::lane_totals(v, c);
      if (lane == 0) {
        m.part_row[2 * seg] = v;
        m.part_row[2 * seg + 1] = c;
      }
    }
  }
}

template <typename T, int R, bool MFIX, int STAGE, bool VARR, int TR>
__global__ __launch_bounds__(LANES* tile_cell_rows(R, TR), tile_waves(sizeof(T), R, TR, STAGE == STAGE_B)) void
tile_kernel(StepArgs<T> a, int64_t n, const T* __restrict__ src, T* __restrict__ dst,
            T* __restrict__ dst2, const T* __restrict__ aux, const T* __restrict__ cf,
            const T* __restrict__ tabx, const T* __restrict__ taby, const T* __restrict__ uv,
            double* __restrict__ part, const double* __restrict__ prev,
            StateHeader* __restrict__ hdr) {
  __shared__ TileShared<T, R, MFIX, TR> u;
  // bands of tiles per XCD, as in step_kernel, cut so that the launch has exactly
  // a block per tile: without an exit on the way, all arguments are fetched at
  // once (each fetch that waits for another costs a cold scalar-cache miss)
  const int x = blockIdx.x & 7;
  const int logical = x * (a.nlogical >> 3) + min(x, a.nlogical & 7) + (int)(blockIdx.x >> 3);
  const StepArgs<T>& args = a;
  tile_step<T, R, MFIX, STAGE, VARR, TR>(args, n, src, dst, dst2, aux, cf, tabx, taby, uv, part,
                                         MFIX ? hdr->pending : 0.0, MFIX ? hdr->fit_max : 0.0,
                                         logical % a.nstrips, logical / a.nstrips, prev, hdr, u);
}

// One batch step (or one stage of a T3S3 batch step) over a work list of
// TR-row tiles, a block per item: the launch holds 8 blocks for every item of
// the longest queue (or more), block b taking item b / 8 of queue b % 8, its
// XCD's.  (A loop over items, for a fixed number of resident blocks, kept
// constants of the arithmetic in registers: 27 spilled in FP64.)
template <typename T, int R, bool MFIX, int STAGE, int TR>
__global__ __launch_bounds__(LANES* tile_cell_rows(R, TR),
                             tile_waves(sizeof(T), R, TR, STAGE == STAGE_B)) void
batch_tile_kernel(const GridDesc<T>* __restrict__ desc, const SlotStep* __restrict__ steps,
                  const BatchCtl* __restrict__ ctl) {
  __shared__ TileShared<T, R, MFIX, TR> u;
  const cptr<BatchCtl> c = as_const(ctl);
  const cptr<SlotStep> st = as_const(steps);
  const int q = (int)(blockIdx.x % NQUEUE);
  if (q >= c->nq) return;
  const int it = c->qstart[q] + (int)(blockIdx.x / NQUEUE);
  if (it >= c->qstart[q + 1]) return;
  const BatchItem w = load_const(as_const(c->items) + it);
  const int64_t n = st[w.slot].n;
  if (n >= st[w.slot].target) return;
  const cptr<GridDesc<T>> d = as_const(desc) + w.slot;
  const auto& a = STAGE == STAGE_B ? d->b : d->a;
  const int b = (int)(n & 1);
  // T2 f~^n -> f~^{n+1}; stage A f^^n -> f~(t'), Q; stage B f~(t'), Q -> f^^{n+1}
  tile_step<T, R, MFIX, STAGE, false, TR>(
      a, n, STAGE == STAGE_B ? d->mid : d->buf[b], STAGE == STAGE_A ? d->mid : d->buf[b ^ 1],
      STAGE == STAGE_A ? d->q : nullptr, STAGE == STAGE_B ? d->q : nullptr,
      STAGE == STAGE_B ? d->cf2 : d->cf, d->tabx, d->taby, nullptr, d->part,
      MFIX ? d->hdr->pending : 0.0, MFIX ? d->hdr->fit_max : 0.0, w.tile % a.nstrips,
      w.tile / a.nstrips, nullptr, d->hdr, u);
}

}  // namespace dugks
