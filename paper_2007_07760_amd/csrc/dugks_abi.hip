// dugks_abi.hip -- C ABI of the DUGKS library (include/dugks.h): plan
// validation and set-up on the host, launches of the device kernels.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "dugks_common.h"
#include "dugks_kernels.h"
#include "dugks_plan.h"

using namespace dugks;

namespace {

constexpr double RT = 1.0 / 3.0;

bool finite(double v) { return isfinite(v); }

// ------------------------------------------------------------ stencils
// bf = sum over the patch of c * fbar+, for face orientation o and velocity i.
void add_tap(int recon, double (&c)[NTAP], int o, int s, int q, double v) {
  int dx = o == 0 ? s : q;
  int dy = o == 0 ? q : s;
  c[tap_index(recon, o, dx, dy)] += v;
}

// Lagrange weight of node j among the unit-spaced nodes m0..m1 for the value
// at coordinate x
double lagrange_weight(int m0, int m1, int j, double x) {
  double w = 1.0;
  for (int k = m0; k <= m1; k++)
    if (k != j) w *= (x - k) / (double)(j - k);
  return w;
}

void make_coefficients(int recon, double h, double (&coef)[2][9][NTAP]) {
  memset(coef, 0, sizeof(coef));
  for (int o = 0; o < 2; o++)
    for (int i = 0; i < 9; i++) {
      double(&c)[NTAP] = coef[o][i];
      // velocity components along the face normal (n) and tangent (t)
      const int en = o == 0 ? ex(i) : ey(i);
      const int et = o == 0 ? ey(i) : ex(i);
      auto add = [&](int s, int q, double v) { add_tap(recon, c, o, s, q, v); };
      if (recon == DUGKS_UPWIND5) {
        // fbar+ at the foot x_b - xi h: along the normal at 1/2 - en h from
        // the centre of L, through the five cells centred on the upstream
        // cell (six centred on the face when en = 0); along the tangent at
        // -et h, through five cells (one when et = 0)
        const int n0 = en < 0 ? -1 : -2, n1 = en > 0 ? 2 : 3;
        const int t0 = et != 0 ? -2 : 0, t1 = et != 0 ? 2 : 0;
        for (int sn = n0; sn <= n1; sn++)
          for (int q = t0; q <= t1; q++)
            add(sn, q, lagrange_weight(n0, n1, sn, 0.5 - en * h) *
                           lagrange_weight(t0, t1, q, -et * h));
      } else if (recon == DUGKS_UPWIND3) {
        // foot of the characteristic relative to the centre of L, (n, t)
        const double pn = 0.5 - en * h, pt = -et * h;
        auto side = [&](int ks, double wgt) {
          // f(k) + d.G + (1/2) d.H.d with G = 3 sum w_m e_m f_m and
          // H = 9 sum w_m (e_m e_m - I/3) f_m over the 3x3 patch about k
          const double dn = pn - ks, dq = pt;
          const double d2 = dn * dn + dq * dq;
          add(ks, 0, wgt);
          for (int m = 0; m < 9; m++) {
            // the lattice is symmetric under x <-> y, so e_m in (n, t) axes
            const int mn = o == 0 ? ex(m) : ey(m);
            const int mt = o == 0 ? ey(m) : ex(m);
            const double de = dn * mn + dq * mt;
            const double v = 3.0 * wq(m) * de + 4.5 * wq(m) * (de * de - d2 / 3.0);
            add(ks + mn, mt, wgt * v);
          }
        };
        if (en > 0)
          side(0, 1.0);
        else if (en < 0)
          side(1, 1.0);
        else {
          side(0, 0.5);
          side(1, 0.5);
        }
      } else if (recon == DUGKS_CENTRAL2) {
        // F = (fL + fR)/2, dn = fR - fL, dt = (fL+t + fR+t - fL-t - fR-t)/4,
        // bf = F - h (en dn + et dt)
        add(0, 0, 0.5);
        add(1, 0, 0.5);
        add(1, 0, -h * en);
        add(0, 0, h * en);
        const double q = -h * et * 0.25;
        add(0, 1, q);
        add(1, 1, q);
        add(0, -1, -q);
        add(1, -1, -q);
      } else {
        // fourth order on LL, L, R, RR (s = -1..2):
        // F = (-1, 9, 9, -1)/16, dn = (1, -27, 27, -1)/24,
        // dt = sum_s F_s D_s with D = (1, -8, 0, 8, -1)/12 across the tangent
        const double wF[4] = {-1.0 / 16, 9.0 / 16, 9.0 / 16, -1.0 / 16};
        const double wN[4] = {1.0 / 24, -27.0 / 24, 27.0 / 24, -1.0 / 24};
        const double wD[5] = {1.0 / 12, -8.0 / 12, 0.0, 8.0 / 12, -1.0 / 12};
        for (int s = -1; s <= 2; s++) {
          add(s, 0, wF[s + 1]);
          add(s, 0, -h * en * wN[s + 1]);
          if (et != 0)
            for (int q = -2; q <= 2; q++)
              if (q != 0) add(s, q, -h * et * wF[s + 1] * wD[q + 2]);
        }
      }
    }
}

// Fold the full table into the compact one (see compact_index): each entry is
// taken from the east face (o = 0) of the velocity with e = (|en|, |et|), and
// every (o, i, tap) used by the scheme must map onto it with the right sign.
// Returns false if some coefficient is not reproduced (a broken symmetry).
bool make_compact(int recon, const double (&coef)[2][9][NTAP], double (&cp)[NCOMPACT]) {
  for (int k = 0; k < NCOMPACT; k++) cp[k] = 0.0;
  const int rep[4] = {0, 3, 1, 2};   // class 2|en|+|et| -> velocity (|en|, |et|)
  for (int c = 0; c < 4; c++)
    for (int t = 0; t < ntap(recon); t++)
      if (tap_used(recon, 0, rep[c], t))
        cp[compact_index(recon, 0, rep[c], t)] = coef[0][rep[c]][t];
  for (int o = 0; o < 2; o++)
    for (int i = 0; i < 9; i++)
      for (int t = 0; t < ntap(recon); t++) {
        const double want = coef[o][i][t];
        if (!tap_used(recon, o, i, t)) {
          if (want != 0.0) return false;
          continue;
        }
        const double got = cp[compact_index(recon, o, i, t)];
        if (fabs(got - want) > 1e-14 * (1.0 + fabs(want))) return false;
      }
  return true;
}

// ------------------------------------------------------ velocity tables
// u(x, y, t) = g(t) UX(x) UY(y), v = g(t) VX(x) VY(y), tables at x = k/2.
void make_tables(dugks_plan* P) {
  const dugks_params& p = P->p;
  const int nx = p.nx, ny = p.ny;
  const double* q = p.vel_param;
  P->tabx.assign(2 * (2 * (size_t)nx + 2), 0.0);
  P->taby.assign(2 * (2 * (size_t)ny + 2), 0.0);
  double* UX = P->tabx.data();
  double* VX = UX + (2 * nx + 2);
  double* UY = P->taby.data();
  double* VY = UY + (2 * ny + 2);
  P->period = 0.0;
  for (int k = 0; k < 2 * nx + 2; k++) {
    const double x = 0.5 * k;
    switch (p.vel_kind) {
      case DUGKS_VEL_UNIFORM: UX[k] = 1.0; VX[k] = 1.0; break;
      case DUGKS_VEL_ROTATION: UX[k] = 1.0; VX[k] = q[0] * (x - q[1]); break;
      case DUGKS_VEL_SINGLE_VORTEX: {
        const double s = sin(M_PI * (x / nx));
        UX[k] = -q[0] * s * s;
        VX[k] = q[0] * sin(2.0 * M_PI * (x / nx));
        break;
      }
      case DUGKS_VEL_DEFORMATION: {
        const double ax = 4.0 * M_PI * x / nx;
        UX[k] = -q[0] * sin(ax);
        VX[k] = -q[0] * cos(ax);
        break;
      }
    }
  }
  for (int k = 0; k < 2 * ny + 2; k++) {
    const double y = 0.5 * k;
    switch (p.vel_kind) {
      case DUGKS_VEL_UNIFORM: UY[k] = q[0]; VY[k] = q[1]; break;
      case DUGKS_VEL_ROTATION: UY[k] = -q[0] * (y - q[2]); VY[k] = 1.0; break;
      case DUGKS_VEL_SINGLE_VORTEX: {
        const double s = sin(M_PI * (y / ny));
        UY[k] = sin(2.0 * M_PI * (y / ny));
        VY[k] = s * s;
        break;
      }
      case DUGKS_VEL_DEFORMATION: {
        const double ay = 4.0 * M_PI * y / ny;
        UY[k] = sin(ay);
        VY[k] = cos(ay);
        break;
      }
    }
  }
  if (p.vel_kind == DUGKS_VEL_SINGLE_VORTEX || p.vel_kind == DUGKS_VEL_DEFORMATION)
    P->period = q[1];
  if (p.vel_kind == DUGKS_VEL_ROTATION) {
    // the rotation is u = -w (y - yc): UX = 1 and the sign sits in UY
  }
}

int validate(const dugks_params* p) {
  if (!p) return DUGKS_EINVAL;
  if (p->nx < 8 || p->ny < 8 || p->nx > 65536 || p->ny > 65536) return DUGKS_EINVAL;
  if (!finite(p->mobility) || !(p->mobility > 0.0)) return DUGKS_EINVAL;
  if (isnan(p->width) || !(p->width > 0.0)) return DUGKS_EINVAL;
  if (!finite(p->cfl) || !(p->cfl > 0.0) || p->cfl > 1.0) return DUGKS_EINVAL;
  if (p->recon < 0 || p->recon > 3) return DUGKS_EINVAL;
  if (p->precision < 0 || p->precision > 1) return DUGKS_EINVAL;
  if (p->vel_kind < 0 || p->vel_kind > 4) return DUGKS_EINVAL;
  if (p->flags & ~(DUGKS_FLAG_DTPHIU_ZERO | DUGKS_FLAG_MASS_FIX)) return DUGKS_EINVAL;
  if (p->tile_rows < 0 || p->tile_rows > 65536) return DUGKS_EINVAL;
  if (p->scheme != DUGKS_T2 && p->scheme != DUGKS_T3S3) return DUGKS_EINVAL;
  // T3S3: the coefficient (12 tau - dt) of f^ in Eq. 31 must stay positive
  if (p->scheme == DUGKS_T3S3 && !(p->cfl < 12.0 * (p->mobility / RT))) return DUGKS_EINVAL;
  for (int k = 0; k < 6; k++)
    if (!finite(p->vel_param[k])) return DUGKS_EINVAL;
  if ((p->vel_kind == DUGKS_VEL_SINGLE_VORTEX || p->vel_kind == DUGKS_VEL_DEFORMATION) &&
      !(p->vel_param[1] > 0.0))
    return DUGKS_EINVAL;
  // the fifth-order reconstruction (DUGKS-T2S5) runs with the T2 time scheme
  // and the analytic velocity kinds only
  if (p->recon == DUGKS_UPWIND5 &&
      (p->scheme != DUGKS_T2 || p->vel_kind == DUGKS_VEL_ARRAYS))
    return DUGKS_EUNSUPPORTED;
  return DUGKS_OK;
}

// Wavefronts of the step kernel resident on one MI355X: 256 CUs, each 4 SIMDs x
// step_waves (the register budget of the kernel variant), as many as their
// fbar+ rings leave room for in 160 KB of LDS.
long resident_wavefronts(const dugks_params& p) {
  const size_t esize = p.precision == DUGKS_F64 ? 8 : 4;
  const int waves = 4 * step_waves((int)esize, p.recon, (p.flags & DUGKS_FLAG_MASS_FIX) != 0);
  return 256L * std::min(waves, (int)(160 * 1024 / (ring_rows(p.recon) * 9 * lrow(p.recon) * esize)));
}

// The height that minimises rounds * (seg + 4), a launch running in
// ceil(tiles / resident) rounds of seg + 4 rows of work: whole rounds, little
// halo.  Segments are whole mass groups (multiples of MASS_GROUP rows).
int whole_round_rows(const dugks_params& p, int nstrips) {
  const long resident = 256L * 4 * step_waves(p.precision == DUGKS_F64 ? 8 : 4, p.recon,
                                              (p.flags & DUGKS_FLAG_MASS_FIX) != 0);
  int best = 64;
  long best_cost = -1;
  for (int seg = 16; seg <= 256; seg += MASS_GROUP) {
    const long tiles = (long)nstrips * ((p.ny + seg - 1) / seg);
    const long rounds = (tiles + resident - 1) / resident;
    const long cost = rounds * (long)(std::min(seg, p.ny) + 4);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = seg;
    }
  }
  return best;
}

// Default rows per marching wavefront: the height with the least estimated time.
// An XCD takes a band of whole segments (or of tiles, see step_args), so with t
// tiles in the largest band and c wavefronts resident on an XCD it works
// n = t / c rounds.  A full round takes seg + 5 rows' time, a part f of one
// 0.5 + 0.5 f of that (few wavefronts run faster, to half the time), and a row
// costs 0.6 % more for every row of height beyond 16 (the wavefronts of
// neighbouring strips fall out of step, and lines they share leave the caches; 1 %
// in FP32 with velocity arrays).
// FP32 without the correction has 3 or 4 wavefronts per SIMD but is bound by VALU
// from 2 on, with velocity arrays from 3 on; there and in central-4 a part of a
// round steps with its wavefronts per SIMD, 0.5 + 0.4 f + 0.1 from the first to the
// last of them.  The estimate orders the heights as measured within 3-5 %; us per step at
// its choice / at the lowest multiple of 8 that makes whole rounds of the chip:
// FP64 upwind-3 1024^2 51.7 (10 rows) / 54.9, 1400^2 83 (18) / 92, 1900^2 139
// (16) / 187 (32 rows: 8 segments in some bands, and a second round there),
// 4096^2 602 (16) / 692 (72); central-4 1900^2 203 (14) / 216; FP32 corrected
// 2000^2 105 (32) / 125 (24), 4096^2 358 (32) / 469 (96); T3S3 1900^2 400 / 509;
// FP32 arrays, against the choice for 2 wavefronts per SIMD, central-4 1900^2 110
// (22) / 129 (34), 1024 x 8192 245 (16) / 294 (40), upwind-3 1900^2 101 (22) / 114 (34);
// 3000^2 246 (16) / 262 (32 at 0.6 %).
// Upwind-5, one wavefront per SIMD in FP64, keeps whole rounds (2048^2 377
// against 432 at 16); in FP32 also that of 8-row tiles (900^2 42 against 57 at 16,
// corrected 51 against 73).
int default_tile_rows(const dugks_params& p, int nstrips) {
  if (p.recon == DUGKS_UPWIND5) {
    const bool one = p.precision == DUGKS_F32 && (long)nstrips * ((p.ny + 7) / 8) <= 2048;
    return one ? 8 : whole_round_rows(p, nstrips);
  }
  const bool fix = (p.flags & DUGKS_FLAG_MASS_FIX) != 0;
  long resident = resident_wavefronts(p);
  const bool arrays = p.vel_kind == DUGKS_VEL_ARRAYS;
  double step = 0.0, drift = 0.006;
  if (p.precision == DUGKS_F32 && !fix) {
    resident = std::min(resident, arrays ? 3072L : 2048L);
    if (arrays || p.recon == DUGKS_CENTRAL4) step = 0.1;
    if (arrays) drift = 0.01;
  }
  const double c = resident / 8.0, simds = 128.0;   // of an XCD
  auto cost = [&](int seg) {
    const int nsegs = (p.ny + seg - 1) / seg;
    const double t = segment_bands(nsegs, p.recon) ? (double)((nsegs + 7) / 8) * nstrips
                                                   : (double)(((long)nstrips * nsegs + 7) / 8);
    const double n = t / c, whole = floor(n), f = n - whole;
    double part = 0.5 + (0.5 - step) * f;
    if (step > 0.0) part += step * (ceil((t - whole * c) / simds) - 1.0) / (ceil(c / simds) - 1.0);
    return (whole + (f > 0.0 ? part : 0.0)) * (seg + 5) * (1.0 + drift * (seg - 16));
  };
  // every height where there are few rounds, else the multiples of 8 from 16 on
  const long tiles16 = (long)nstrips * ((p.ny + 15) / 16);
  const bool few = tiles16 < (fix ? 4 * resident : std::min(4 * resident, 8192L));
  int best = 16;
  for (int seg = few ? 8 : 16; seg <= 40; seg += few && !fix ? 1 : MASS_GROUP)
    if (cost(seg) < cost(best)) best = seg;
  return best;
}

// Rows of the tiles the tile kernel takes of such a grid.
int tile_rows_of(const dugks_params& p, int nstrips) {
  const bool mfix = (p.flags & DUGKS_FLAG_MASS_FIX) != 0;
  const int rows = block_tile_rows(p.precision == DUGKS_F64 ? 8 : 4, p.recon, p.scheme, mfix,
                                   (int64_t)nstrips * ((p.ny + 3) / 4));
  if (!wide(p.recon) || mfix || rows != 8) return rows;
  // An upwind-5 block of 8 rows is 14 wavefronts and has a compute unit for
  // itself, so a step takes whole rounds of 256 blocks (~11 us each in FP64, ~7.5
  // in FP32, also for a last round of a few).  10 rows, 16 wavefronts, take ~12.5
  // (8.5) but may take fewer rounds: 512^2 FP64 3 rounds 32.6 us, 2 of 10 rows
  // 26.4 (FP32 22.2, 17.0); 832^2 7 rounds 76.1, 5 64.1; 384^2 2 rounds either
  // way, 21.7 and 23.8; 1024^2 9 and 8, 101.5 and 99.9.
  const int r8 = (nstrips * ((p.ny + 7) / 8) + 255) / 256;
  const int r10 = (nstrips * ((p.ny + 9) / 10) + 255) / 256;
  return 10 * r10 < 9 * r8 ? 10 : 8;
}

// Whether a grid is too small to fill the chip with marching wavefronts, so that
// the tile kernel is its default.  A marching wavefront needs ~25 us (FP64
// upwind-3) for an 8-row tile however few there are, the tile kernel 6.0 us for
// a grid of up to 256 tiles, but it forms the cell terms of 12 rows for every 8
// (8 for every 4).  The line lies at the number of 16-row marching tiles where
// the two meet, measured on square grids (us per step, tile / march): FP64
// upwind-3 768^2 33.0 / 35.2, 896^2 43.0 / 40.2; central-4 768^2 43.3 / 45.8,
// 896^2 56.0 / 54.5; central-2 900^2 38.4 / 40.9, 1000^2 45.1 / 44.3; velocity
// arrays 768^2 34.5 / 38.4, 896^2 45.2 / 43.7; T3S3 640^2 66.3 / 60.9; FP32 corrected 768^2 29.0 / 30.8, 896^2 34.9 / 32.3, central-4
// 896^2 37.6 / 37.6, upwind-5 704^2 35 / 40, 768^2 43 / 40, corrected 576^2 37 / 42,
// 704^2 57 / 48.  The corrected FP64
// kernels of the 3-point patches have room for one round of 512 blocks: upwind-3
// 448^2 27 / 33, 512^2 38 / 34; central-2 26 / 27, 37 / 27; T3S3 46 / 62, 69 / 65;
// with arrays upwind-3 576^2 36 / 38, 640^2 42 / 40.
// FP64 upwind-5 runs whole rounds either way, of 256 blocks or of 1024 marching
// wavefronts (one per SIMD): ~11.3 us a round of 8-row blocks, 12.7 of 10-row
// ones, 4.45 a row of a marching round (corrected 13.8 and 5.35): 1040^2 105 /
// 124, 1000 x 1300 129 / 125, 1400^2 178 / 195; corrected 832^2 97 / 106, 940^2
// 114 / 108, 1000^2 128 / 149, 1150^2 162 / 152.
bool tile_kernel_default(const dugks_params& p, int nstrips, int rows) {
  const bool f64 = p.precision == DUGKS_F64, mfix = (p.flags & DUGKS_FLAG_MASS_FIX) != 0;
  const bool arrays = p.vel_kind == DUGKS_VEL_ARRAYS;
  if (f64 && wide(p.recon)) {
    const int h = std::min(whole_round_rows(p, nstrips), p.ny);
    const long blocks = (long)nstrips * ((p.ny + rows - 1) / rows);
    const long tiles = (long)nstrips * ((p.ny + h - 1) / h);
    const double block_us = mfix ? 13.8 : (rows == 10 ? 12.7 : 11.3);
    return (double)((blocks + 255) / 256) * block_us <
           (double)((tiles + 1023) / 1024) * (h + 4) * (mfix ? 5.35 : 4.45);
  }
  const long n16 = (long)nstrips * ((p.ny + 15) / 16);
  const long limit = wide(p.recon)                ? (mfix ? 450 : 620)
                     : p.recon == DUGKS_CENTRAL4  ? (f64 ? 840 : 900)
                     : f64 && mfix                ? (arrays ? 400 : 256)
                     : f64 && p.scheme == DUGKS_T3S3 ? 400
                     : f64 && p.recon == DUGKS_CENTRAL2 ? 930
                     : f64 && arrays              ? 840
                                                  : 760;
  return n16 <= limit;
}

// Rows of the tile kernel's tiles, or 0 where the march runs.  Heights up to
// TILE_MAX_ROWS ask for the kernel.  They get it wherever it is the default, and on
// larger grids where it beats a march of that height (us per step, tile / march):
// always in FP64 upwind-5 (8 rows: 2500^2 corrected 712 / 770) and uncorrected FP64
// central-4 (361 / 451), and for up to 3 rows uncorrected (2500^2: FP64 upwind-3 297 /
// 335, FP32 195 / 203); up to some way beyond the default's line in the other FP64 T2
// forms (8 rows: upwind-3 1024^2 54 / 62, 1448^2 103 / 103, 2500^2 298 / 273;
// corrected central-4 1200^2 120 / 129, 1448^2 167 / 149) and in uncorrected FP32 (6
// rows: upwind-3 1200^2 47.0 / 49.3, 2500^2 199 / 165, T3S3 900^2 67 / 63; 8 rows:
// central-4 1200^2 51.4 / 58.2, 1448^2 71.2 / 68.5).  Elsewhere they are marched (8
// rows: 2500^2 FP32 upwind-3
// 199 / 159, corrected 224 / 183, upwind-5 363 / 268; T3S3 1448^2 285 / 259).  Where the
// march's default is 8 rows too, asking for 8 gives the default.
int tile_kernel_rows(const dugks_params& p, int nstrips) {
  if (p.tile_rows > TILE_MAX_ROWS) return 0;
  const int rows = tile_rows_of(p, nstrips);
  bool take = tile_kernel_default(p, nstrips, rows);
  if (p.tile_rows > 0) {
    const bool f64 = p.precision == DUGKS_F64, mfix = (p.flags & DUGKS_FLAG_MASS_FIX) != 0;
    const bool c4 = p.recon == DUGKS_CENTRAL4;
    const long n16 = (long)nstrips * ((p.ny + 15) / 16);
    if (!take && p.tile_rows == 8 && default_tile_rows(p, nstrips) == 8) return 0;
    long line = 0;
    if (f64 && p.scheme == DUGKS_T2) {
      line = !mfix ? 2280 : (c4 ? 1680 : 0);
    } else if (!f64 && !mfix) {
      const int most = p.scheme == DUGKS_T3S3 ? 4 : 6;
      line = p.tile_rows <= most ? (wide(p.recon) ? 1000 : 2280) : (c4 ? 1575 : 0);
    }
    take = take || n16 <= line || (f64 && (wide(p.recon) || (c4 && !mfix))) ||
           (!mfix && p.tile_rows <= 3);
  }
  // a launch holds fewer than 2^32 threads
  const int64_t blocks = (int64_t)nstrips * ((p.ny + rows - 1) / rows);
  if (blocks * LANES * tile_cell_rows(p.recon, rows) >= INT64_C(1) << 32) return 0;
  return take ? rows : 0;
}

// ------------------------------------------------------------ launches
template <typename T, bool MFIX, int STAGE>
void launch_march(const dugks_plan* P, const StageBufs<T>& q, int64_t n, hipStream_t s) {
  StepArgs<T> a = step_args<T>(P, STAGE);
  // blocks per XCD (see step_kernel's tile order)
  const int per = a.ileave > 1 ? a.ileave * a.clen * a.nstrips : (a.nlogical + 7) / 8;
  dim3 grid(per * 8), block(LANES);
  const bool varr = P->p.vel_kind == DUGKS_VEL_ARRAYS;
#define DUGKS_LAUNCH(RR, VA)                                                                   \
  hipLaunchKernelGGL((step_kernel<T, RR, MFIX, STAGE, VA>), grid, block, 0, s, a, n, q.src,    \
                     q.dst, q.dst2, q.aux, q.cf, q.tabx, q.taby, q.uv, q.part, q.hdr)
  switch (P->p.recon) {
    case DUGKS_CENTRAL2:
      if (varr) DUGKS_LAUNCH(DUGKS_CENTRAL2, true); else DUGKS_LAUNCH(DUGKS_CENTRAL2, false);
      break;
    case DUGKS_UPWIND3:
      if (varr) DUGKS_LAUNCH(DUGKS_UPWIND3, true); else DUGKS_LAUNCH(DUGKS_UPWIND3, false);
      break;
    case DUGKS_CENTRAL4:
      if (varr) DUGKS_LAUNCH(DUGKS_CENTRAL4, true); else DUGKS_LAUNCH(DUGKS_CENTRAL4, false);
      break;
    default:   // upwind-5: T2, analytic velocities (validate)
      if constexpr (STAGE == STAGE_T2) DUGKS_LAUNCH(DUGKS_UPWIND5, false);
      break;
  }
#undef DUGKS_LAUNCH
}

template <typename T, bool MFIX, int STAGE>
int launch_stage(const dugks_plan* P, void* state, int64_t n, hipStream_t s, FixUse fix) {
  const Layout& L = P->L;
  StageBufs<T> q = stage_bufs<T>(P, state, n, STAGE);
  if (fix.prev && STAGE != STAGE_B)
    q.prev = at<double>(state, fix.prev_spare ? L.off_scratch : L.off_groups);
  if (fix.spare) q.part = at<double>(state, L.off_scratch);
  if (P->tile)
    launch_tile<T, STAGE>(P, q, n, s);
  else
    launch_march<T, MFIX, STAGE>(P, q, n, s);
  if (MFIX && fix.reduce && STAGE != STAGE_A)
    hipLaunchKernelGGL(mass_fix_strips_kernel, dim3(L.tl.nstrips), dim3(LANES), 0, s,
                       q.part, L.ngroups, L.tl.nstrips, at<double>(state, L.off_strips), q.hdr,
                       (double)P->p.nx * (double)P->p.ny);
  return hip_status(hipGetLastError());
}

template <typename T>
int launch_step(const dugks_plan* P, void* state, int64_t n, hipStream_t s, FixUse fix) {
  if (P->p.scheme == DUGKS_T3S3) {
    // with the fused correction, stage A applies the pending one as it reads
    // f^^n and stage B gives the partials of f^^{n+1}: one reduction per step
    if (P->p.flags & DUGKS_FLAG_MASS_FIX) {
      int rc = launch_stage<T, true, STAGE_A>(P, state, n, s, fix);
      return rc ? rc : launch_stage<T, true, STAGE_B>(P, state, n, s, fix);
    }
    int rc = launch_stage<T, false, STAGE_A>(P, state, n, s, fix);
    return rc ? rc : launch_stage<T, false, STAGE_B>(P, state, n, s, fix);
  }
  return (P->p.flags & DUGKS_FLAG_MASS_FIX)
             ? launch_stage<T, true, STAGE_T2>(P, state, n, s, fix)
             : launch_stage<T, false, STAGE_T2>(P, state, n, s, fix);
}

template <typename T>
int stage_head(const dugks_plan* P) {
  const Layout& L = P->L;
  void* h = nullptr;
  if (hipHostMalloc(&h, L.off_buf[0], hipHostMallocDefault) != hipSuccess) return DUGKS_EDEVICE;
  memset(h, 0, L.off_buf[0]);
  StateHeader* hd = static_cast<StateHeader*>(h);
  hd->magic = STATE_MAGIC;
  hd->nx = P->p.nx;
  hd->ny = P->p.ny;
  hd->precision = P->p.precision;
  hd->recon = P->p.recon;
  hd->fit_max = INFINITY;
  // the device tables carry dt * alpha (Eq. 27 with the stage's half step)
  // times the stencil
  const int s0 = P->p.scheme == DUGKS_T3S3 ? STAGE_A : STAGE_T2;
  T* cf = at<T>(h, L.off_coef);
  for (int k = 0; k < NCOMPACT; k++) cf[k] = T(P->dt * P->st[s0].alpha * P->compact[k]);
  T* cf2 = at<T>(h, L.off_coef2);
  for (int k = 0; k < NCOMPACT; k++)
    cf2[k] = T(P->dt * P->st[STAGE_B].alpha * P->compact2[k]);
  T* tx = at<T>(h, L.off_tabx);
  for (size_t k = 0; k < P->tabx.size(); k++) tx[k] = T(P->tabx[k]);
  T* ty = at<T>(h, L.off_taby);
  for (size_t k = 0; k < P->taby.size(); k++) ty[k] = T(P->taby[k]);
  P->head = h;
  return DUGKS_OK;
}

template <typename T>
int do_init(const dugks_plan* P, void* state, const double* phi0, const double* uv,
            hipStream_t s) {
  const Layout& L = P->L;
  const int nx = P->p.nx, ny = P->p.ny;
  std::call_once(P->staged, [P] { P->head_rc = stage_head<T>(P); });
  if (P->head_rc) return P->head_rc;
  hipError_t e;
  if ((e = hipMemcpyAsync(state, P->head, L.off_buf[0], hipMemcpyHostToDevice, s)))
    return hip_status(e);
  InitArgs<T> a;
  a.uv = nullptr;
  if (P->p.vel_kind == DUGKS_VEL_ARRAYS) {
    const int64_t n2 = 2 * (int64_t)nx * ny;
    T* dst = at<T>(state, L.off_vel);
    hipLaunchKernelGGL((velocity_store_kernel<T>), dim3((unsigned)((n2 + 255) / 256)), dim3(256),
                       0, s, uv, dst, n2);
    a.uv = dst;
  }
  a.phi0 = phi0;
  a.buf = at<T>(state, L.off_buf[0]);
  a.tabx = at<T>(state, L.off_tabx);
  a.taby = at<T>(state, L.off_taby);
  a.tl = L.tl;
  a.shift = P->p.scheme == DUGKS_T3S3 ? 0.25 * P->dt : 0.5 * P->dt;
  a.kth = isfinite(P->p.width) ? 4.0 / P->p.width : 0.0;
  dim3 grid((nx + 255) / 256, ny), block(256);
  hipLaunchKernelGGL((init_kernel<T>), grid, block, 0, s, a);
  if ((e = hipGetLastError())) return hip_status(e);
  // M0: FP64 total of phi0 itself (not of its rounded f~)
  double* part = at<double>(state, L.off_scratch);
  StateHeader* hd = at<StateHeader>(state, 0);
  hipLaunchKernelGGL((mass_partial_kernel<double, false>), dim3(MASS_BLOCKS), dim3(MASS_THREADS),
                     0, s, phi0, L.tl, nullptr, part);
  hipLaunchKernelGGL(mass_final_kernel, dim3(1), dim3(64), 0, s, part, &hd->mass0,
                     &hd->mass_now, hd);
  return hip_status(hipGetLastError());
}

template <typename T>
int do_phi(const dugks_plan* P, const void* state, int64_t n, void* out, hipStream_t s) {
  const Layout& L = P->L;
  hipLaunchKernelGGL((phi_kernel<T>), read_grid<T>(P->p.nx, P->p.ny), dim3(READ_THREADS), 0, s,
                     at<T>(state, L.off_buf[n & 1]), L.tl, at<StateHeader>(state, 0),
                     static_cast<T*>(out));
  return hip_status(hipGetLastError());
}

template <typename T>
int do_export(const dugks_plan* P, const void* state, int64_t n, void* out, hipStream_t s) {
  const Layout& L = P->L;
  hipLaunchKernelGGL((export_kernel<T>), read_grid<T>(P->p.nx, P->p.ny), dim3(READ_THREADS), 0, s,
                     at<T>(state, L.off_buf[n & 1]), L.tl, at<StateHeader>(state, 0),
                     static_cast<T*>(out));
  return hip_status(hipGetLastError());
}

template <typename T>
int do_history(const dugks_plan* P, const void* state, int64_t n, void* out, hipStream_t s) {
  const Layout& L = P->L;
  hipLaunchKernelGGL((history_kernel<T>), read_grid<T>(P->p.nx, P->p.ny), dim3(READ_THREADS), 0, s,
                     at<T>(state, L.off_buf[n & 1]), L.tl, static_cast<T*>(out));
  return hip_status(hipGetLastError());
}

template <typename T>
int do_mass(const dugks_plan* P, void* state, int64_t n, double* out, hipStream_t s) {
  const Layout& L = P->L;
  double* part = at<double>(state, L.off_scratch);
  StateHeader* hd = at<StateHeader>(state, 0);
  hipLaunchKernelGGL((mass_partial_kernel<T, true>), dim3(MASS_BLOCKS), dim3(MASS_THREADS), 0, s,
                     at<T>(state, L.off_buf[n & 1]), L.tl, hd, part);
  hipLaunchKernelGGL(mass_final_kernel, dim3(1), dim3(64), 0, s, part, &hd->mass_now, out, hd);
  return hip_status(hipGetLastError());
}

template <typename T>
int do_correct(const dugks_plan* P, void* state, int64_t n, hipStream_t s) {
  const Layout& L = P->L;
  const int nx = P->p.nx, ny = P->p.ny;
  const StateHeader* hd = at<StateHeader>(state, 0);
  dim3 grid((nx + 255) / 256, ny), block(256);
  for (int pass = 0; pass < 2; pass++) {
    int rc = do_mass<T>(P, state, n, nullptr, s);
    if (rc) return rc;
    hipLaunchKernelGGL((mass_correct_kernel<T>), grid, block, 0, s,
                       at<T>(state, L.off_buf[n & 1]), L.tl, hd);
    if (hipGetLastError() != hipSuccess) return DUGKS_EDEVICE;
  }
  return DUGKS_OK;
}

}  // namespace

// ================================================================== C ABI
extern "C" {

int dugks_plan_create(const dugks_params* p, dugks_plan** out) {
  if (!out) return DUGKS_EINVAL;
  *out = nullptr;
  int rc = validate(p);
  if (rc) return rc;
  dugks_plan* P = new (std::nothrow) dugks_plan();
  if (!P) return DUGKS_ENOMEM;
  P->p = *p;
  P->L = make_layout(p->nx, p->ny, p->precision, p->scheme, p->vel_kind);
  P->dt = p->cfl;                 // Eq. (39), dx = sqrt(3RT) = 1
  P->h = 0.5 * P->dt;
  P->tau = p->mobility / RT;      // M_phi = tau RT
  const double tau = P->tau, dt = P->dt, h = P->h;
  // g+ = (tau - b)/(tau + a) g + (a + b)/(tau + a) (feq + tau S) for
  // g = f - a (Omega + S), g+ = f + b (Omega + S)
  P->cA = (2 * tau - dt) / (2 * tau + dt);     // (a, b) = (dt/2, dt/2): f~+
  P->cB = 2 * dt / (2 * tau + dt);
  P->cA2 = (2 * tau - h) / (2 * tau + dt);     // (a, b) = (dt/2, h/2): fbar+
  P->cB2 = 3 * h / (2 * tau + dt);
  P->alpha = 2 * tau / (2 * tau + h);          // Eq. (27)
  P->beta = h / (2 * tau + h);
  P->gamma = tau * h / (2 * tau + h);
  // launch kinds: T2 (f~ in, half step h), T3S3 stage A (f^ in, dt/6), stage B
  // (f~ at t + dt/3 in, 5 dt/12); the shift identity above gives cbar with
  // a = the input's shift and b = half of the stage's half step
  auto stage = [&](int k, double hs, double a_in, double kap, double wo1, double wo2,
                   double toff, double troff, double jdt, int jfirst) {
    dugks_plan::StageCoef& c = P->st[k];
    c.h = hs;
    c.cbar = (a_in + 0.5 * hs) / (tau + a_in);
    c.kap = kap;
    c.wo1 = wo1;
    c.wo2 = wo2;
    c.alpha = 2 * tau / (2 * tau + hs);
    c.beta = hs / (2 * tau + hs);
    c.gamma = tau * hs / (2 * tau + hs);
    c.toff = toff;
    c.troff = troff;
    c.jdt = jdt;
    c.jfirst = jfirst;
  };
  // T2: f~+ = fbar+ + kap (X - fbar+), kap = cbar / (3 (1 - cbar))
  stage(STAGE_T2, h, 0.5 * dt, P->cB2 / (3.0 * (1.0 - P->cB2)), 1.0, 0.0, 0.0, -dt, dt, 1);
  P->st[STAGE_T2].cbar = P->cB2;   // the same value, rounded as Eq. 23's 3h / (2 tau + dt)
  {
    // stage A: cbar = 4 dt / (12 tau + 3 dt) (Eq. 31); f~+ (Eq. 33) and f^n
    // (Eq. 32) are fbar+ -/+ (cbar / (4 (1 - cbar))) (X - fbar+)
    const double c1 = (0.25 * dt + dt / 12.0) / (tau + 0.25 * dt);
    stage(STAGE_A, dt / 6.0, 0.25 * dt, c1 / (4.0 * (1.0 - c1)), 1.0 / 3.0, 3.0 / 7.0, 0.0, -dt,
          dt, 1);
    // stage B: cbar = 9 dt / (24 tau + 4 dt) (Eq. 34); (3/4) dt (Omega + S)(t')
    // = (3/4) dt 6 / ((6 tau + dt)(1 - cbar)) (X' - fbar+) (Eq. 29)
    const double c2 = (dt / 6.0 + 5.0 * dt / 24.0) / (tau + dt / 6.0);
    stage(STAGE_B, 5.0 * dt / 12.0, dt / 6.0,
          0.75 * dt * 6.0 / ((6.0 * tau + dt) * (1.0 - c2)), 4.0 / 7.0, 0.0, dt / 3.0, 0.0,
          dt / 3.0, 0);
  }
  const bool t3 = p->scheme == DUGKS_T3S3;
  make_coefficients(p->recon, t3 ? P->st[STAGE_A].h : h, P->coef);
  if (!make_compact(p->recon, P->coef, P->compact)) {
    delete P;
    return DUGKS_EINVAL;   // cannot happen for the schemes built in
  }
  if (t3) {
    double coef2[2][9][NTAP];
    make_coefficients(p->recon, P->st[STAGE_B].h, coef2);
    if (!make_compact(p->recon, coef2, P->compact2)) {
      delete P;
      return DUGKS_EINVAL;
    }
  }
  make_tables(P);
  P->nstrips = (p->nx + OWN - 1) / OWN;
  P->tile = tile_kernel_rows(*p, P->nstrips);
  auto rows = [p](int r) {
    if (p->flags & DUGKS_FLAG_MASS_FIX)   // whole mass groups per segment
      r = (r + MASS_GROUP - 1) / MASS_GROUP * MASS_GROUP;
    return std::min(r, p->ny);
  };
  P->seg_rows = rows(p->tile_rows > 0 ? p->tile_rows : default_tile_rows(*p, P->nstrips));
  P->nsegs = (p->ny + P->seg_rows - 1) / P->seg_rows;
  // dugks_step_many_noalloc: its work list is of a fixed length, so large
  // grids keep the taller tiles of whole rounds, and short ones are not shorter
  // than 16 rows; its limit counts the height asked for
  const int asked = p->tile_rows > 0 ? p->tile_rows : whole_round_rows(*p, P->nstrips);
  P->many_rows = rows(std::max(16, asked));
  P->many_segs = (p->ny + P->many_rows - 1) / P->many_rows;
  P->many_limit_segs = (p->ny + rows(asked) - 1) / rows(asked);
  *out = P;
  return DUGKS_OK;
}

void dugks_plan_destroy(dugks_plan* plan) {
  if (!plan) return;
  if (plan->head) (void)hipHostFree(plan->head);
  delete plan;
}

size_t dugks_state_bytes(const dugks_plan* plan) { return plan ? plan->L.total : 0; }

int dugks_init(const dugks_plan* plan, void* state, const double* phi0_dev,
               const double* uv_dev, void* stream) {
  if (!plan || !state || !phi0_dev || !aligned(state)) return DUGKS_EINVAL;
  if (plan->p.vel_kind == DUGKS_VEL_ARRAYS && !uv_dev) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return plan->p.precision == DUGKS_F64 ? do_init<double>(plan, state, phi0_dev, uv_dev, s)
                                        : do_init<float>(plan, state, phi0_dev, uv_dev, s);
}

int dugks_step(const dugks_plan* plan, void* state, int64_t step, int64_t nsteps,
               void* stream) {
  if (!plan || !state || !aligned(state) || step < 0 || nsteps < 0) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool inl = fix_inline(plan);
  const bool two = plan->p.scheme == DUGKS_T2;   // alternate sets of partials
  for (int64_t k = 0; k < nsteps; k++) {
    // the last step's partials are the regular ones, reduced into the header
    FixUse fix;
    fix.reduce = !inl || k == nsteps - 1;
    fix.prev = inl && k > 0;
    fix.spare = inl && two && ((nsteps - 1 - k) & 1);
    fix.prev_spare = two && ((nsteps - k) & 1);
    int rc = plan->p.precision == DUGKS_F64 ? launch_step<double>(plan, state, step + k, s, fix)
                                            : launch_step<float>(plan, state, step + k, s, fix);
    if (rc) return rc;
  }
  return DUGKS_OK;
}

int dugks_tune(const dugks_params* params, void* state, int64_t step, int32_t reps,
               int32_t* rows_out, void* stream) {
  if (!params || !state || !rows_out || !aligned(state) || step < 0 || reps < 1 || reps > 1000)
    return DUGKS_EINVAL;
  const int rc0 = validate(params);
  if (rc0) return rc0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // candidates: the default height, then 16..256 rows in steps of MASS_GROUP
  // (as the plans round them: duplicates dropped)
  std::vector<dugks_plan*> plans;
  int rc = DUGKS_OK;
  for (int c = 0; c <= std::min(256, params->ny) && !rc; c = (c == 0 ? 16 : c + MASS_GROUP)) {
    dugks_params q = *params;
    q.tile_rows = c;
    dugks_plan* P = nullptr;
    if ((rc = dugks_plan_create(&q, &P))) break;
    bool dup = false;
    for (dugks_plan* o : plans)
      dup = dup || (o->tile == P->tile && (P->tile || o->seg_rows == P->seg_rows));
    if (dup)
      dugks_plan_destroy(P);
    else
      plans.push_back(P);
  }
  // without the correction's reduction: the header keeps the correction the next
  // real step applies
  FixUse keep;
  keep.reduce = false;
  auto launch = [&](const dugks_plan* P) {
    return P->p.precision == DUGKS_F64 ? launch_step<double>(P, state, step, s, keep)
                                       : launch_step<float>(P, state, step, s, keep);
  };
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (!rc && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
    rc = DUGKS_EDEVICE;
  // the clocks ramp up over the first launches after idle: warm up first, then
  // time every candidate twice (forward, then backward) and keep its best
  for (int k = 0; k < 20 && !rc; k++) rc = launch(plans[0]);
  std::vector<float> best(plans.size(), 0.0f);
  for (int pass = 0; pass < 2 && !rc; pass++) {
    for (size_t j = 0; j < plans.size() && !rc; j++) {
      const size_t i = pass == 0 ? j : plans.size() - 1 - j;
      rc = launch(plans[i]);   // one untimed launch at this shape
      if (!rc && hipEventRecord(e0, s) != hipSuccess) rc = DUGKS_EDEVICE;
      for (int k = 0; k < reps && !rc; k++) rc = launch(plans[i]);
      if (!rc && hipEventRecord(e1, s) != hipSuccess) rc = DUGKS_EDEVICE;
      float ms = 0.0f;
      if (!rc && (hipEventSynchronize(e1) != hipSuccess ||
                  hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
        rc = DUGKS_EDEVICE;
      if (!rc && (pass == 0 || ms < best[i])) best[i] = ms;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (!rc) {
    size_t b = 0;
    for (size_t i = 1; i < plans.size(); i++)
      if (best[i] < best[b]) b = i;
    *rows_out = plans[b]->tile ? TILE_MAX_ROWS : plans[b]->seg_rows;
  }
  for (dugks_plan* P : plans) dugks_plan_destroy(P);
  return rc;
}

int dugks_phi(const dugks_plan* plan, const void* state, int64_t step, void* phi_out_dev,
              void* stream) {
  if (!plan || !state || !phi_out_dev || !aligned(state) || step < 0) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return plan->p.precision == DUGKS_F64 ? do_phi<double>(plan, state, step, phi_out_dev, s)
                                        : do_phi<float>(plan, state, step, phi_out_dev, s);
}

int dugks_distributions(const dugks_plan* plan, const void* state, int64_t step,
                        void* out_dev, void* stream) {
  if (!plan || !state || !out_dev || !aligned(state) || step < 0) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return plan->p.precision == DUGKS_F64 ? do_export<double>(plan, state, step, out_dev, s)
                                        : do_export<float>(plan, state, step, out_dev, s);
}

int dugks_history(const dugks_plan* plan, const void* state, int64_t step, void* out_dev,
                  void* stream) {
  if (!plan || !state || !out_dev || !aligned(state) || step < 0) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return plan->p.precision == DUGKS_F64 ? do_history<double>(plan, state, step, out_dev, s)
                                        : do_history<float>(plan, state, step, out_dev, s);
}

int dugks_state_status(const dugks_plan* plan, const void* state, int32_t* status_out,
                 void* stream) {
  if (!plan || !state || !status_out || !aligned(state)) return DUGKS_EINVAL;
  const StateHeader* hd = at<StateHeader>(state, 0);
  return hip_status(hipMemcpyAsync(status_out, &hd->status, sizeof(int32_t), hipMemcpyDefault,
                                   static_cast<hipStream_t>(stream)));
}

int dugks_mass(const dugks_plan* plan, void* state, int64_t step, double* mass_out_dev,
               void* stream) {
  if (!plan || !state || !mass_out_dev || !aligned(state) || step < 0) return DUGKS_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return plan->p.precision == DUGKS_F64 ? do_mass<double>(plan, state, step, mass_out_dev, s)
                                        : do_mass<float>(plan, state, step, mass_out_dev, s);
}

int dugks_mass_correct(const dugks_plan* plan, void* state, int64_t step, void* stream) {
  if (!plan || !state || !aligned(state) || step < 0) return DUGKS_EINVAL;
  if (plan->p.precision == DUGKS_F64 || (plan->p.flags & DUGKS_FLAG_MASS_FIX)) return DUGKS_OK;
  return do_correct<float>(plan, state, step, static_cast<hipStream_t>(stream));
}

int dugks_mass0(const dugks_plan* plan, const void* state, double* out_dev, void* stream) {
  if (!plan || !state || !out_dev || !aligned(state)) return DUGKS_EINVAL;
  const StateHeader* hd = at<StateHeader>(state, 0);
  return hip_status(hipMemcpyAsync(out_dev, &hd->mass0, sizeof(double),
                                   hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream)));
}

const char* dugks_strerror(int status) {
  switch (status) {
    case DUGKS_OK: return "ok";
    case DUGKS_EINVAL: return "invalid argument";
    case DUGKS_ENOMEM: return "out of host memory";
    case DUGKS_EDEVICE: return "HIP launch or runtime call failed";
    case DUGKS_ENUMERIC: return "non-finite total mass";
    case DUGKS_EUNSUPPORTED: return "not supported by this library";
    default: return "unknown status";
  }
}

const char* dugks_version(void) { return "dugks-gfx950 0.1"; }

}  // extern "C"
