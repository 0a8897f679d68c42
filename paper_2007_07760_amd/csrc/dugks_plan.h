// dugks_plan.h -- the plan object and the launch helpers shared by the
// single-grid and batch entry points (private to the library).
#pragma once

#include <math.h>

#include <mutex>
#include <vector>

#include "dugks_common.h"
#include "dugks_kernels.h"

struct dugks_plan {
  dugks_params p;
  dugks::Layout L;
  double coef[2][9][dugks::NTAP];   // face stencils (Eqs. 25-26)
  double compact[dugks::NCOMPACT];  // the same, folded by the lattice symmetries
  double dt, h, tau;
  double cA, cB, cA2, cB2, alpha, beta, gamma;
  double period;             // cos(pi t / period) modulation; 0 = steady
  // coefficients of each launch kind (dugks::Stage): the face stencil is built
  // with the stage's half step h; fbar+ = g + cbar (X - g) from the stage's
  // input g; the outputs take kap (X - fbar+) and wo1 / wo2 dt L; d(phi u)/dt
  // uses phi at n dt + toff and at n dt + troff
  struct StageCoef {
    double h, cbar, kap, wo1, wo2, alpha, beta, gamma, toff, troff, jdt;
    int jfirst;
  } st[3];
  double compact2[dugks::NCOMPACT];  // T3S3 stage B stencil (compact: stage A)
  int seg_rows, nstrips, nsegs;   // of the march
  int many_rows, many_segs;       // of dugks_step_many_noalloc
  int many_limit_segs;            // segments its limit counts
  int tile;                  // rows of the tile kernel's tiles (4, 8 or 10); 0: the march
  std::vector<double> tabx, taby;
  // the constant head of every state of this plan (header, coefficient and
  // velocity tables in the plan's precision), staged once in pinned host memory
  // so that dugks_init can copy it asynchronously
  mutable std::once_flag staged;
  mutable void* head = nullptr;
  mutable int head_rc = DUGKS_OK;
};

namespace dugks {

// How a launch of the step deals with the fused mass correction: `reduce` runs
// the reduction kernel after it, which leaves the correction in the header;
// `prev` forms the correction from the last step's partials in the step kernel
// itself; `spare`, `prev_spare`: the partials written, read are in the state's
// mass scratch.
struct FixUse {
  bool reduce = true, prev = false, spare = false, prev_spare = false;
};

// Plans whose steps may form the correction themselves: the tile kernel sums the
// partials again in every block, so few of them (one strip per wavefront, one
// group per lane), and a second set of them has to fit the mass scratch (T3S3
// writes them a launch after it has read them).
inline bool fix_inline(const dugks_plan* P) {
  if (!(P->p.flags & DUGKS_FLAG_MASS_FIX) || !P->tile) return false;
  if (P->nstrips > MASS_GROUP + 4 || P->L.ngroups > LANES) return false;
  return P->p.scheme == DUGKS_T3S3 || P->nstrips * P->L.ngroups <= MASS_BLOCKS;
}

inline int hip_status(hipError_t e) { return e == hipSuccess ? DUGKS_OK : DUGKS_EDEVICE; }

template <typename T>
inline T* at(void* state, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(state) + off);
}
template <typename T>
inline const T* at(const void* state, size_t off) {
  return reinterpret_cast<const T*>(static_cast<const char*>(state) + off);
}

inline bool aligned(const void* ptr) { return ((uintptr_t)ptr & 255u) == 0; }


// the buffers of one launch (see Stage)
template <typename T>
struct StageBufs {
  const T* src;
  T* dst;
  T* dst2;
  const T* aux;
  const T* cf;
  const T* tabx;
  const T* taby;
  const T* uv;
  double* part;              // mass partials this launch writes
  const double* prev;        // those its correction is to be formed from, or nullptr
  StateHeader* hdr;
};

template <typename T>
inline StageBufs<T> stage_bufs(const dugks_plan* P, void* state, int64_t n, int stage) {
  const Layout& L = P->L;
  const int b = (int)(n & 1);
  StageBufs<T> q;
  q.src = at<T>(state, L.off_buf[b]);
  q.dst = at<T>(state, L.off_buf[b ^ 1]);
  q.dst2 = nullptr;
  q.aux = nullptr;
  q.cf = at<T>(state, L.off_coef);
  if (stage == STAGE_A) {           // f^^n -> f~(t'), Q
    q.dst = at<T>(state, L.off_mid);
    q.dst2 = at<T>(state, L.off_q);
  } else if (stage == STAGE_B) {    // f~(t'), Q -> f^^{n+1}
    q.src = at<T>(state, L.off_mid);
    q.aux = at<T>(state, L.off_q);
    q.cf = at<T>(state, L.off_coef2);
  }
  q.tabx = at<T>(state, L.off_tabx);
  q.taby = at<T>(state, L.off_taby);
  q.uv = P->p.vel_kind == DUGKS_VEL_ARRAYS ? at<T>(state, L.off_vel) : nullptr;
  q.part = at<double>(state, L.off_groups);
  q.prev = nullptr;
  q.hdr = at<StateHeader>(state, 0);
  return q;
}

// One launch of the tile kernel (plans with P->tile != 0).
template <typename T, int STAGE>
void launch_tile(const dugks_plan* P, const StageBufs<T>& q, int64_t n, hipStream_t s);

// Whether an XCD's band of the march is whole segments, its two halves in turn:
// once it holds 4 segments or more (not for the wide patch: one wavefront per
// SIMD, and it measured slower).
inline bool segment_bands(int nsegs, int recon) { return nsegs >= 32 && !wide(recon); }

template <typename T>
inline StepArgs<T> step_args(const dugks_plan* P, int stage = STAGE_T2) {
  const Layout& L = P->L;
  StepArgs<T> a;
  a.CH = L.tl.CH;
  a.nx = P->p.nx;
  a.ny = P->p.ny;
  a.seg_rows = P->seg_rows;
  a.nstrips = P->nstrips;
  a.nsegs = P->nsegs;
  a.nlogical = P->nstrips * P->nsegs;
  a.ileave = segment_bands(P->nsegs, P->p.recon) ? 2 : 1;
  a.clen = ((P->nsegs + 7) / 8 + a.ileave - 1) / a.ileave;
  a.ngroups = L.ngroups;
  const dugks_plan::StageCoef& c = P->st[stage];
  a.cB2 = T(c.cbar);
  a.kap = T(c.kap);
  a.wo1 = T(c.wo1);
  a.wo2 = T(c.wo2);
  a.pscale = T(c.beta / c.alpha);
  a.gdt = T(0.5 * P->dt * c.gamma);
  a.dt = T(P->dt);
  a.jinv = T(1) / T(c.jdt);
  a.toff = c.toff;
  a.troff = c.troff;
  a.jfirst = c.jfirst;
  a.tau = T(P->tau);
  a.kth = isfinite(P->p.width) ? T(4.0 / P->p.width) : T(0);
  a.period = P->period;
  a.dtd = P->dt;
  a.hd = c.h;
  a.jzero = (P->p.flags & DUGKS_FLAG_DTPHIU_ZERO) ? 1 : 0;
  return a;
}

}  // namespace dugks
