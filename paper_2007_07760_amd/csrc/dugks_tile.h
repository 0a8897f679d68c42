// dugks_tile.h -- the step of a small grid: one block of wavefronts per tile,
// one wavefront per cell row (arXiv 2007.07760, Sec. II).
//
// A grid that cannot fill the chip with marching wavefronts (step_kernel) is
// bound by the march's serial chain: a 16-row tile takes 21 rows in turn, ~35
// us in FP64, whatever the grid's size.  Here the rows of a tile run side by
// side: wavefront w of a block forms phi, the cell terms and fbar+ of cell row
// y0 - LAG + w, then the faces of that row and its update, with four block
// barriers between (differences of phi; fbar+ rows; faces; the faces' values
// below each row).  What bounds it is that chain of latencies: 5.8-6.6 us per
// step for grids of up to 256 tiles (64^2 FP64: 36 us with the march, 6.7 now;
// 256^2 8.7; FP32 corrected 256^2 with its reduction 37.7, 12.3; upwind-5 64^2
// 79, 9.4).  On larger grids it is bound by VALU and LDS: TR rows take the
// cell terms of TR + 4 (6), so 4-row tiles do twice the march's cell work, and
// the march wins from ~800^2 (FP64) or ~1100^2 (FP32) on (plan creation holds
// the rule).  4 rows against 8: a tile's faces wait for fewer rows, and its
// blocks spread over more compute units (FP64 upwind-3 64^2 6.7 against 8.2
// us, 1024^2 59.9 against 64.0).
//
// The arithmetic is the march's, expression by expression, so the results are
// bitwise the same.  The face values take their neighbour columns from lane
// shifts of one LDS read per row, which needs 80-100 registers in FP64 where
// reading every tap from LDS needed 224 (spilled at the 5 wavefronts per SIMD
// it is built for).
#pragma once

#include "dugks_common.h"
#include "dugks_kernels.h"

namespace dugks {

// cell rows of a tile of TR rows: the faces of its rows and of the row below
// reach LAG rows down and up
__host__ __device__ constexpr int tile_cell_rows(int recon, int TR) {
  return TR + 2 * (wide(recon) ? 3 : 2);
}

// the face values of row k, velocity by velocity: pn of the north faces, de of
// the east less the west ones, and their sums over the velocities
template <bool EAST, typename M, typename T>
__device__ __forceinline__ void faces(const M& m, int k, T (&pn)[9], T (&de)[9], T& phN, T& phE) {
  unroll<9>([&](auto I) {
    constexpr int i = decltype(I)::value;
    T pe;
    m.template recon_pair<i, EAST>(k, pn[i], pe);
    phN += pn[i];
    if constexpr (EAST) {
      phE += pe;
      if constexpr (ex(i) != 0) de[i] = pe - from_left(pe);
    }
    __builtin_amdgcn_sched_barrier(0);
  });
}

template <typename T, int R, bool MFIX, int STAGE, bool VARR, int TR>
__global__ __launch_bounds__(LANES* tile_cell_rows(R, TR), tile_waves(sizeof(T), R, TR)) void
tile_kernel(StepArgs<T> a, int64_t n, const T* __restrict__ src, T* __restrict__ dst,
            T* __restrict__ dst2, const T* __restrict__ aux, const T* __restrict__ cf,
            const T* __restrict__ tabx, const T* __restrict__ taby, const T* __restrict__ uv,
            double* __restrict__ part, const StateHeader* __restrict__ hdr) {
  constexpr int CR = tile_cell_rows(R, TR);
  using M = Marcher<T, R, MFIX, STAGE, VARR, CR>;
  constexpr int LAG = M::LAG;
  static_assert(!MFIX || TR == MASS_GROUP, "a tile of a corrected plan is one mass group");
  // one buffer, in turn: the row differences phi(x+1) - phi(x-1) and
  // phi(x-1) + 4 phi + phi(x+1); s of the cell rows; the mass sums of the rows
  union Shared {
    T da[CR + 2][2][LANES];
    T s[CR][2][LANES];
    struct {
      double sum[MFIX ? TR : 1][LANES];
      int fit[MFIX ? TR : 1][LANES];
    } mass;
  };
  __shared__ T s_bfp[CR][9][LANES];
  __shared__ Shared u;

  const int lane = threadIdx.x & (LANES - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
  // bands of tiles per XCD, as in step_kernel
  const int per = (a.nlogical + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || logical >= a.nlogical) return;
  const int strip = logical % a.nstrips;
  const int seg = logical / a.nstrips;

  M m{a, src, as_const(cf), tabx, as_const(taby), uv, s_bfp};
  m.place(lane, strip, seg * TR, TR, dst, dst2, aux, part, MFIX ? hdr->pending : 0.0,
          MFIX ? hdr->fit_max : 0.0);
  m.base = m.y0 - LAG;
  // the cell row of this wavefront; the last tile may hold fewer rows, the
  // wavefronts beyond what it needs load its top row and write nothing
  const int top = m.y1 + LAG - 1;
  const int r = m.y0 - LAG + w;
  const bool cells = r <= top;
  const int k = r;                                  // its face row
  const bool upd = k >= m.y0 && k < m.y1;
  RowRegs<T> d, o;
  m.load_row(d, min(r, top + 1));
  const bool outer = w == 0 || w == CR - 1;
  if (outer) m.load_row(o, w == 0 ? m.y0 - LAG - 1 : min(r + 1, top + 1));
  T qv[10];
  if (STAGE == STAGE_B && upd) m.load_q(k, qv);
  m.flow(n);

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
  // no wavefront reads another's fbar+ row from here on: each keeps its own in
  // registers and leaves its north faces (dt*alpha*fbar of the six crossing
  // velocities, P, Q) in its place for the row above
  __syncthreads();
  const int kk = wrapi(k, a.ny);
  T eP, eQx, eQy, PN, QNx, QNy;
  T bp[9];
  if (north) {
    m.north_moments(kk, phN, m.sxp[LAG], m.syp[LAG], u.s[w + 1][0][lane], u.s[w + 1][1][lane],
                    PN, QNx, QNy);
#pragma unroll
    for (int i = 0; i < 9; i++) bp[i] = s_bfp[w][i][lane];
#pragma unroll
    for (int i = 0; i < 9; i++)
      if (ey(i) != 0) s_bfp[w][i][lane] = pn[i];
    s_bfp[w][0][lane] = PN;
    s_bfp[w][1][lane] = QNx;
    s_bfp[w][5][lane] = QNy;
    if (upd) m.east_moments(kk, phE, m.sxp[LAG], m.syp[LAG], eP, eQx, eQy);
  }
  __syncthreads();
  if (upd) {
    T out[9];
#pragma unroll
    for (int i = 0; i < 9; i++) {
      out[i] = T(0);
      if (ey(i) != 0) {
        const T dn = pn[i] - s_bfp[w - 1][i][lane];
        out[i] = ey(i) > 0 ? -dn : dn;
      }
      if (ex(i) != 0) out[i] = ex(i) > 0 ? out[i] - de[i] : out[i] + de[i];
    }
    double cs = 0.0, cf0 = 0.0;
    m.update_cells(kk, bp, out, PN - s_bfp[w - 1][0][lane], QNx - s_bfp[w - 1][1][lane],
                   QNy - s_bfp[w - 1][5][lane], eP, eQx, eQy, m.cp[LAG], m.cx[LAG], m.cy[LAG],
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

}  // namespace dugks
