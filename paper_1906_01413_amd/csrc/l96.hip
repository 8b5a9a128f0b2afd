// Lorenz-96 nonlinear, tangent-linear and adjoint integrations for gfx950.
//
// Model: Section 3.1.1 (Lorenz-96, periodic), integrated with classical RK4.
// Hessian-probe product (Alg. 3, y_i = A w_i with A = L^T G^T R^{-1} G L):
// one TL sweep over the window collecting R^{-1}-weighted observation values,
// one AD sweep injecting them at the observed steps. Each member (probe) runs
// in one workgroup (or one wave) with its state in registers.

#include <type_traits>

#include "l96_common.h"
#include "riot_internal.h"

namespace riot {
namespace {

// LDS elements per wave of the batched launches: halo buffer of a one-strip member (2 parities,
// at most 199 each) and a staging row of up to 17 positions per lane
constexpr int kWaveLds = 400 + 64 * 17;

// ---------------------------------------------------------------------------
// Strips. A member's state of n elements is cut into NW strips of `own` consecutive elements,
// one wave each; lane i of a wave holds the E consecutive positions i E .. i E + E - 1 of a
// window of 64 E elements that starts HL elements before the strip. A wave so recomputes HL
// elements of its left and HR of its right neighbour: inside the window the periodic halo of a
// stage comes from the adjacent lanes (DPP moves), with no LDS and no barrier, and what goes
// wrong at the window's ends creeps inwards by at most two positions per stage. Only after
// mv.K RK4 steps do the waves refresh their halos through LDS, one barrier each time.
//
// How far it creeps (positions invalid after s stages, from the left / right): the nonlinear
// stage and the TL use i-2 .. i+1: 2 s / s. A trajectory whose stages are stored refreshes every
// step, so the stored stage s = 0..3 of a step is wrong on 2 s / s positions; one whose stages are
// not (a forecast, observed values only) every mv.K steps. The AD uses i-1 .. i+2 of
// its own state and i-2 .. i+2 of stages 3, 2, 1, 0 of the base: the first stage leaves
// 8 / 5 wrong, each further one 1 / 2 more. After K steps: TL 8 K / 4 K, AD 4 K + 7 / 8 K + 3.
// The layout (strip_layout, in the API layer) leaves HL = max(8 K, 4 K + 7), HR = 8 K + 3.
//
// Before, a member's lanes exchanged their halo through LDS with a workgroup barrier in every
// stage, and the stage was the latency of that. A block product (TL and AD over the window) took
// then and takes now: n = 40, m = 30, T = 20: 131 and 54 us; n = 2048, m = 128, T = 50: 217 and
// 135 us; n = 4096, T = 100: m = 16 758 and 405 us, m = 256 783 and 424 us, m = 272 790 and
// 580 us. What bounds it now: FP64 issue (about 390 instructions per 9 positions and step in the
// TL, two waves on a SIMD), then the base loads (37 KB a stage and compute unit at 64 bytes a
// clock).
// ---------------------------------------------------------------------------

// place of position j of lane i in its wave's part of a stage block: rows in pairs, each lane's
// two values adjacent (16-byte loads: a product of n = 4096, m = 256, T = 100 takes 424 us, with
// one row per load 564), an odd last row by itself
__device__ __forceinline__ int base_index(int E, int j, int i) {
  return (j | 1) < E ? (j >> 1) * 128 + 2 * i + (j & 1) : j * 64 + i;
}

// value of the lane one below or above (the end lanes get zero)
template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_shift(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)dpp_int<CTRL>((int)b);
  const unsigned hi = (unsigned)dpp_int<CTRL>((int)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double from_below(double v) { return dpp_shift<0x138>(v); }  // wave_shr:1
__device__ __forceinline__ double from_above(double v) { return dpp_shift<0x130>(v); }  // wave_shl:1

// d = J(x) e : (J e)_i = (e_{i+1} - e_{i-2}) x_{i-1} + (x_{i+1} - x_{i-2}) e_{i-1} - e_i
template <int E>
__device__ __forceinline__ void tl_jac(const double (&xe)[E + 4], const double (&e)[E], double hl2,
                                       double hl1, double hr1, double (&d)[E]) {
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const double em2 = (j >= 2) ? e[j - 2] : (j == 0 ? hl2 : hl1);
    const double em1 = (j >= 1) ? e[j - 1] : hl1;
    const double ep1 = (j + 1 < E) ? e[j + 1] : hr1;
    d[j] = fma(ep1 - em2, xe[j + 1], fma(xe[j + 3] - xe[j], em1, -e[j]));
  }
}

// s = J(x)^T w : (J^T w)_i = x_{i-2} w_{i-1} - x_{i+1} w_{i+2} + (x_{i+2} - x_{i-1}) w_{i+1} - w_i
template <int E>
__device__ __forceinline__ void ad_jac(const double (&xe)[E + 4], const double (&w)[E], double hl1,
                                       double hr1, double hr2, double (&s)[E]) {
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const double wm1 = (j >= 1) ? w[j - 1] : hl1;
    const double wp1 = (j + 1 < E) ? w[j + 1] : hr1;
    const double wp2 = (j + 2 < E) ? w[j + 2] : (j + 2 == E ? hr1 : hr2);
    s[j] = fma(xe[j + 4] - xe[j + 1], wp1, fma(-xe[j + 3], wp2, fma(xe[j], wm1, -w[j])));
  }
}

// Nonlinear tendency on the extended state: f_i = (x_{i+1} - x_{i-2}) x_{i-1} - x_i + F
template <int E>
__device__ __forceinline__ void tendency(const double (&xe)[E + 4], double F, double (&f)[E]) {
#pragma unroll
  for (int j = 0; j < E; ++j) f[j] = (xe[j + 3] - xe[j]) * xe[j + 1] - xe[j + 2] + F;
}

// A wave's strip: positions, halo refresh, base loads, TL and AD sweeps.
template <int E, int MB = 1>
struct Strip {
  typedef double d2 __attribute__((ext_vector_type(2)));
  const ModelView &mv;
  double *lds;               // halo buffer of the member(s), 2 parities
  double *stg;               // this wave's staging row of observed steps (64 E)
  int lane, w, parity;
  int el0;                 // element of this lane's first position
  unsigned own, pub, sub;  // bit j: position j is owned / read by another strip / a halo position
  int pb, sb;              // its buffer index as published / read is pb + j / sb + j (unless
                           // the buffer holds the whole state, element by element)
  bool whole;              // the buffer holds the whole state (shorter than two halos)
  int nbuf;                // elements per parity

  __device__ Strip(const ModelView &m, double *lds_, int tid)
      : mv(m), lds(lds_), lane(tid & 63), w(__builtin_amdgcn_readfirstlane(tid >> 6)), parity(0) {
    const int n = mv.n, HL = mv.HL, HR = mv.HR, ew = HL + HR;
    const int ow = min(mv.own, n - w * mv.own);
    const int q0 = lane * E - HL;  // strip-relative position of j = 0
    el0 = (w * mv.own + q0) % n;
    el0 = el0 < 0 ? el0 + n : el0;
    whole = n < ew + E;
    const int nslot = ew + 4 * E;
    nbuf = whole ? n : mv.NW * nslot;
    stg = lds + 2 * MB * nbuf + w * 64 * E;
    own = pub = sub = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int q = q0 + j;
      if (q >= 0 && q < ow) {
        own |= 1u << j;
        if (whole || q < HR || q >= ow - HL) pub |= 1u << j;
      } else if (q >= -HL && q < ow + HR) {
        sub |= 1u << j;
      }
    }
    pb = sb = 0;
    if (!whole) {
      // a strip's slot: its first HR elements (its left neighbour's right halo), then its last
      // HL (its right neighbour's left halo), each with E spare places at both ends, so that
      // a lane writes and reads all its E positions (no lane holds positions of both ends)
      pb = w * nslot + (q0 < HR ? E + q0 : HR + 3 * E + q0 - (ow - HL));
      const int wl = w == 0 ? mv.NW - 1 : w - 1, wr = w == mv.NW - 1 ? 0 : w + 1;
      sb = q0 < 0 ? wl * nslot + HR + 3 * E + q0 + HL : wr * nslot + E + q0 - ow;
    }
  }

  // element of position j from el0 (opaque(el0) where the E elements must not stay in
  // registers from an earlier use)
  __device__ __forceinline__ int element(int e0, int j) const {
    const int e = e0 + j;
    return e >= mv.n ? e - mv.n : e;
  }
  __device__ __forceinline__ static int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
  }

  // The halo positions of v from the strips that own them. Two buffers in turn, so that one
  // barrier per refresh is enough.
  template <int M>
  __device__ __forceinline__ void refresh(double (&v)[M][E]) {
    double *b = lds + parity * nbuf * M;
    parity ^= 1;
    auto sync = [&]() {
      if (mv.NW == 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      } else {
        // (not __syncthreads: its fence would also wait for the base loads in flight)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      }
    };
    const unsigned pub_ = TIGHT ? opaque(pub) : pub, sub_ = TIGHT ? opaque(sub) : sub;
    if (whole) {
      const int e0 = opaque(el0);
#pragma unroll
      for (int q = 0; q < M; ++q)
#pragma unroll
        for (int j = 0; j < E; ++j)
          if (pub_ >> j & 1) b[q * nbuf + element(e0, j)] = v[q][j];
      sync();
#pragma unroll
      for (int q = 0; q < M; ++q)
#pragma unroll
        for (int j = 0; j < E; ++j)
          if (sub_ >> j & 1) v[q][j] = b[q * nbuf + element(e0, j)];
      return;
    }
    if (pub_) {
#pragma unroll
      for (int q = 0; q < M; ++q)
#pragma unroll
        for (int j = 0; j < E; ++j) b[q * nbuf + pb + j] = v[q][j];
    }
    sync();
    if (sub_) {
#pragma unroll
      for (int q = 0; q < M; ++q) {
        double r[E];
#pragma unroll
        for (int j = 0; j < E; ++j) r[j] = b[q * nbuf + sb + j];
#pragma unroll
        for (int j = 0; j < E; ++j) v[q][j] = sub_ >> j & 1 ? r[j] : v[q][j];
      }
    }
  }

  // neighbours' values at the ends of this lane's positions
  __device__ __forceinline__ void halo(const double (&v)[E], double &hl2, double &hl1, double &hr1,
                                       double &hr2) const {
    hl1 = from_below(v[E - 1]);
    hl2 = from_below(v[E - 2]);
    hr1 = from_above(v[0]);
    hr2 = from_above(v[1]);
  }

  // Stage block b = 4 t + s of this wave (layout: base_index).
  __device__ __forceinline__ void load_base(int b, double (&x)[E]) const {
    const double *p = reinterpret_cast<const double *>(mv.xs) +
                    ((size_t)b * mv.NW + w) * (size_t)(64 * E);
#pragma unroll
    for (int j = 0; j + 1 < E; j += 2) {
      const d2 v = *reinterpret_cast<const gmem<d2> *>(gptr(p) + j * 64 + 2 * lane);
      x[j] = v.x, x[j + 1] = v.y;
    }
    if (E & 1) x[E - 1] = gptr(p)[(E - 1) * 64 + lane];
  }
  // TIGHT: the members' states alone fill the registers, so one stage block is in flight (else
  // two, or a whole step's), an observed step's tables are loaded when it is reached, and the
  // halo masks are taken apart anew at each refresh.
  static constexpr bool TIGHT = E * MB > 17;
  static constexpr int D = E * MB <= 5 ? 4 : TIGHT ? 1 : 2;
  __device__ __forceinline__ void extend(const double (&x)[E], double (&xe)[E + 4]) const {
#pragma unroll
    for (int j = 0; j < E; ++j) xe[2 + j] = x[j];
    halo(x, xe[0], xe[1], xe[E + 2], xe[E + 3]);
  }

  // natural-layout vector <-> the window's positions
  __device__ __forceinline__ void load_vec(const double *x, double (&v)[E]) const {
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = gptr(x)[element(el0, j)];
  }
  __device__ __forceinline__ void store_vec(double *x, const double (&v)[E]) const {
    const int e0 = opaque(el0), own_ = opaque(own);
#pragma unroll
    for (int j = 0; j < E; ++j)
      if (own_ >> j & 1) gptr(x)[element(e0, j)] = (double)v[j];
  }

  // Observed steps. The unique observations of a step's strip are consecutive, so they are
  // read and written coalesced, 64 at a time, and meet the positions in the wave's staging
  // row. (Each lane taking its own positions' values, E predicated accesses per member, cost
  // 0.3 of 0.87 ms at n = 4096, m = 272, T = 100.) ObsAhead holds what the next observed step needs first, loaded before it is reached:
  // the strip's range, and the window positions (and values of a table) of its first 128.
  static constexpr int kPre = TIGHT ? 1 : 2;
  struct ObsAhead {
    int u0 = 0, u1 = 0, pos[kPre];
    double val[MB][kPre];
  };
  __device__ __forceinline__ int obs_step(int t) const {
    return __builtin_amdgcn_readfirstlane(gptr(mv.stepk)[t]);
  }
  // nsrc tables src + q stride, q < nsrc (0: positions only)
  __device__ __forceinline__ void obs_ahead(int k, const double *src, int nsrc, size_t stride,
                                            ObsAhead &o) const {
    o.u0 = __builtin_amdgcn_readfirstlane(gptr(mv.wstart)[k * mv.NW + w]);
    o.u1 = __builtin_amdgcn_readfirstlane(gptr(mv.wstart)[k * mv.NW + w + 1]);
#pragma unroll
    for (int c = 0; c < kPre; ++c) {
      const int u = min(o.u0 + c * 64 + lane, mv.U - 1);
      o.pos[c] = gptr(mv.upos)[u];
#pragma unroll
      for (int q = 0; q < MB; ++q)
        if (q < nsrc) o.val[q][c] = gptr(src + q * stride)[u];
    }
  }
  __device__ __forceinline__ void wave_fence() const {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  // f[u] = wgt[u] v_i, or v_i (wgt null); o holds wgt's values
  __device__ __forceinline__ void obs_store(const ObsAhead &o, const double (&v)[E], const double *wgt,
                                            double *f) const {
#pragma unroll
    for (int j = 0; j < E; ++j) stg[lane * E + j] = v[j];
    wave_fence();
#pragma unroll
    for (int c = 0; c < kPre; ++c) {
      const int u = o.u0 + c * 64 + lane;
      if (u < o.u1) gptr(f)[u] = wgt ? o.val[0][c] * stg[o.pos[c]] : stg[o.pos[c]];
    }
    for (int u = o.u0 + kPre * 64 + lane; u < o.u1; u += 64) {
      const double x = stg[gptr(mv.upos)[u]];
      gptr(f)[u] = wgt ? gptr(wgt)[u] * x : x;
    }
    wave_fence();
  }
  // v_i += f[u]; o holds f's values as table q
  __device__ __forceinline__ void obs_add(const ObsAhead &o, int q, const double *f,
                                          double (&v)[E]) const {
#pragma unroll
    for (int j = 0; j < E; ++j) stg[lane * E + j] = 0;
    wave_fence();
#pragma unroll
    for (int c = 0; c < kPre; ++c)
      if (o.u0 + c * 64 + lane < o.u1) stg[o.pos[c]] = o.val[q][c];
    for (int u = o.u0 + kPre * 64 + lane; u < o.u1; u += 64) stg[gptr(mv.upos)[u]] = gptr(f)[u];
    wave_fence();
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] += stg[lane * E + j];
    wave_fence();
  }

  // Tangent-linear sweep over the window from dl (valid on the whole window of positions); at
  // an observed step f[u] = wgt[u] dl_i (weighted) or dl_i. The base of each stage is loaded D
  // stages ahead, what an observed step needs one stage ahead.
  __device__ __forceinline__ void tl_sweep(double (&dl)[MB][E], double *f, bool weighted, bool skip0, int live) {
    const double h = mv.h, h2 = 0.5 * mv.h, h6 = mv.h / 6.0;
    const double *wgt = reinterpret_cast<const double *>(mv.wgt);
    double xb[D][E], xe[E + 4], e[MB][E], d[E], acc[MB][E];
    double hl2, hl1, hr1, hr2;
    ObsAhead oa;
    int since = 0, kn = obs_step(0), kl = gptr(mv.stepk)[min(1, mv.T)];
    auto fetch = [&](int k) {
      obs_ahead(k, wgt, weighted ? 1 : 0, 0, oa);
    };
#pragma unroll
    for (int i = 0; i < D; ++i) load_base(i, xb[i]);
    if (kn >= 0) fetch(kn);
    for (int t = 0; t <= mv.T; ++t) {
      const int k = kn;
      kn = __builtin_amdgcn_readfirstlane(kl);
      kl = gptr(mv.stepk)[min(t + 2, mv.T)];
      if (k >= 0 && !(skip0 && t == 0)) {
        if (TIGHT) fetch(k);
#pragma unroll
        for (int q = 0; q < MB; ++q)
          if (q < live) obs_store(oa, dl[q], weighted ? wgt : nullptr, f + (size_t)q * mv.U);
      }
      if (t == mv.T) break;
      if (since == mv.K) {
        refresh(dl);
        since = 0;
      }
      ++since;
      // (loads past the last step: block 4 T and the three after it, whose contents are not
      // used, lie in the buffer)
      // stage 1
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[0 % D], xe);
      if (TIGHT) load_base(4 * t + 0 + D, xb[0 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(dl[q], hl2, hl1, hr1, hr2);
        tl_jac<E>(xe, dl[q], hl2, hl1, hr1, d);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(4 * t + 0 + D, xb[0 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          acc[q][j] = d[j];
          e[q][j] = dl[q][j] + h2 * d[j];
        }
      }
      // stage 2
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[1 % D], xe);
      if (TIGHT) load_base(4 * t + 1 + D, xb[1 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(e[q], hl2, hl1, hr1, hr2);
        tl_jac<E>(xe, e[q], hl2, hl1, hr1, d);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(4 * t + 1 + D, xb[1 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          acc[q][j] = fma(2, d[j], acc[q][j]);
          e[q][j] = dl[q][j] + h2 * d[j];
        }
      }
      // stage 3
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[2 % D], xe);
      if (TIGHT) load_base(4 * t + 2 + D, xb[2 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(e[q], hl2, hl1, hr1, hr2);
        tl_jac<E>(xe, e[q], hl2, hl1, hr1, d);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(4 * t + 2 + D, xb[2 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          acc[q][j] = fma(2, d[j], acc[q][j]);
          e[q][j] = dl[q][j] + h * d[j];
        }
      }
      // stage 4
      if (!TIGHT && kn >= 0) fetch(kn);
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[3 % D], xe);
      if (TIGHT) load_base(4 * t + 3 + D, xb[3 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(e[q], hl2, hl1, hr1, hr2);
        tl_jac<E>(xe, e[q], hl2, hl1, hr1, d);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(4 * t + 3 + D, xb[3 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          acc[q][j] += d[j];
          dl[q][j] = dl[q][j] + h6 * acc[q][j];
        }
      }
    }
  }

  // Adjoint sweep over the window with forcing f injected at observed steps, from lam (valid
  // on the whole window of positions); loads ahead as in the TL.
  __device__ __forceinline__ void ad_sweep(double (&lam)[MB][E], const double *f, size_t fstride, bool skip0) {
    const double h = mv.h, h2 = 0.5 * mv.h, h3 = mv.h / 3.0, h6 = mv.h / 6.0;
    double xb[D][E], xe[E + 4], lp[MB][E], a[MB][E], s[E];
    double hl2, hl1, hr1, hr2;
    ObsAhead oa;
    int since = 0, kn = obs_step(mv.T), kl = gptr(mv.stepk)[max(mv.T - 1, 0)];
    auto fetch = [&](int k) {
      obs_ahead(k, f, MB, fstride, oa);
    };
    const int bl = max(4 * mv.T - 1, 3);
#pragma unroll
    for (int i = 0; i < D; ++i) load_base(bl - i, xb[(3 - i) % D]);
    if (kn >= 0) fetch(kn);
    for (int t = mv.T; t >= 0; --t) {
      const int k = kn;
      kn = __builtin_amdgcn_readfirstlane(kl);
      kl = gptr(mv.stepk)[max(t - 2, 0)];
      if (k >= 0 && !(skip0 && t == 0)) {
        if (TIGHT) fetch(k);
#pragma unroll
        for (int q = 0; q < MB; ++q) obs_add(oa, q, f + q * fstride, lam[q]);
        since = mv.K;  // forced on the owned positions only
      }
      if (t == 0) break;
      if (since == mv.K) {
        refresh(lam);
        since = 0;
      }
      ++since;
      const int b0 = 4 * (t - 1);
      // adjoint of stage 4 input
#pragma unroll
      for (int q = 0; q < MB; ++q)
#pragma unroll
        for (int j = 0; j < E; ++j) {
          lp[q][j] = lam[q][j];
          a[q][j] = h6 * lp[q][j];
        }
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[3 % D], xe);
      if (TIGHT) load_base(max(b0 + 3 - D, 0), xb[3 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(a[q], hl2, hl1, hr1, hr2);
        ad_jac<E>(xe, a[q], hl1, hr1, hr2, s);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(max(b0 + 3 - D, 0), xb[3 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          lam[q][j] = lp[q][j] + s[j];
          a[q][j] = fma(h, s[j], h3 * lp[q][j]);
        }
      }
      // stage 3
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[2 % D], xe);
      if (TIGHT) load_base(max(b0 + 2 - D, 0), xb[2 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(a[q], hl2, hl1, hr1, hr2);
        ad_jac<E>(xe, a[q], hl1, hr1, hr2, s);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(max(b0 + 2 - D, 0), xb[2 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          lam[q][j] += s[j];
          a[q][j] = fma(h2, s[j], h3 * lp[q][j]);
        }
      }
      // stage 2
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[1 % D], xe);
      if (TIGHT) load_base(max(b0 + 1 - D, 0), xb[1 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(a[q], hl2, hl1, hr1, hr2);
        ad_jac<E>(xe, a[q], hl1, hr1, hr2, s);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(max(b0 + 1 - D, 0), xb[1 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) {
          lam[q][j] += s[j];
          a[q][j] = fma(h2, s[j], h6 * lp[q][j]);
        }
      }
      // stage 1
      if (!TIGHT && kn >= 0) fetch(kn);
      __builtin_amdgcn_sched_barrier(0);
      extend(xb[0 % D], xe);
      if (TIGHT) load_base(max(b0 + 0 - D, 0), xb[0 % D]);
#pragma unroll
      for (int q = 0; q < MB; ++q) {
        if (MB > 1) __builtin_amdgcn_sched_barrier(0);
        halo(a[q], hl2, hl1, hr1, hr2);
        ad_jac<E>(xe, a[q], hl1, hr1, hr2, s);
        if (!TIGHT && q == MB - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_base(max(b0 + 0 - D, 0), xb[0 % D]);
        }
#pragma unroll
        for (int j = 0; j < E; ++j) lam[q][j] += s[j];
      }
    }
  }

  // One member. Base mode (mode & 7): 0 = TL (R^{-1}-weighted store) then AD -> lam0;
  // 1 = AD forced by the shared fsrc -> lam0; 2 = TL only, raw observed values into f;
  // 3 = AD forced by this member's own f -> lam0. Flags: kTladSkip0 = no store or injection
  // at the window's step 0 (a checkpoint segment after the first, whose step 0 is the
  // previous segment's last step); kTladInitLam = the AD starts from dx0 instead of zero;
  // kTladOutState = mode 2 writes the final tangent state into lam0. dx0 and lam0 use the
  // natural layout (double).
  // MB members from dx0, lam0 and f on, n and U apart, the first `live` of which are stored
  // (the others repeat the last of those).
  __device__ __forceinline__ void run(int mode, const double *dx0, double *lam0, double *f,
                                      const double *fsrc, int live = MB) {
    const int base = mode & 7;
    const bool skip0 = (mode & kTladSkip0) != 0;
    double v[MB][E];
    auto load = [&]() {
#pragma unroll
      for (int q = 0; q < MB; ++q) load_vec(dx0 + (size_t)min(q, live - 1) * mv.n, v[q]);
    };
    auto store = [&]() {
#pragma unroll
      for (int q = 0; q < MB; ++q)
        if (q < live) store_vec(lam0 + (size_t)q * mv.n, v[q]);
    };
    if (base == 0 || base == 2) {
      load();
      tl_sweep(v, f, base == 0, skip0, live);
      if (base == 2) {
        if (mode & kTladOutState) store();
        return;
      }
      // each forcing value is re-read by the lane that stored it
    }
    if (mode & kTladInitLam) {
      load();
    } else {
#pragma unroll
      for (int q = 0; q < MB; ++q)
#pragma unroll
        for (int j = 0; j < E; ++j) v[q][j] = 0;
    }
    // (a member beyond the live ones takes the first one's forcing)
    ad_sweep(v, base == 1 ? fsrc : f, base == 1 || live < MB ? 0 : (size_t)mv.U, skip0);
    store();
  }
};

// ---------------------------------------------------------------------------
// Nonlinear trajectory, one workgroup per window.
// ---------------------------------------------------------------------------

// Stage block (t, s) of the window's positions (and its FP32 copy).
template <int E>
__device__ __forceinline__ void store_block(const ModelView &mv, double *xs64, int t,
                                            int s, int w, int lane, const double (&v)[E]) {
  const size_t base = ((size_t)(t * 4 + s) * mv.NW + w) * (size_t)(64 * E);
  typedef double d2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int j = 0; j + 1 < E; j += 2)
    *reinterpret_cast<gmem<d2> *>(gptr(xs64 + base) + j * 64 + 2 * lane) = d2{v[j], v[j + 1]};
  if (E & 1) gptr(xs64 + base)[(E - 1) * 64 + lane] = v[E - 1];
}

// xu != nullptr: no stage blocks; the state at every observed (step, variable) pair u is
// written to xu[u].
template <int E>
__device__ __forceinline__ void trajectory_window(const ModelView &mv, int nsteps,
                                                  const double *x0, double *xout, double *xs64,
                                                  double *xu, double *lds,
                                                  int shard = -1) {
  Strip<E> S(mv, lds, threadIdx.x);
  if (S.w >= mv.NW) return;
  const int every = xs64 ? 1 : mv.K;  // steps between refreshes
  if (shard >= 0 && S.w != shard) xs64 = nullptr;
  if (shard > 0) xout = nullptr;
  const double h = mv.h, F = mv.F;
  double xw[1][E], xs[E], acc[E], k[E], xe[E + 4];
  double(&x)[E] = xw[0];
  S.load_vec(x0, x);
  auto sample = [&](int t) {
    const int ks = S.obs_step(t);
    if (ks >= 0) {
      typename Strip<E>::ObsAhead o;
      S.obs_ahead(ks, nullptr, 0, 0, o);
      S.obs_store(o, x, nullptr, xu);
    }
  };
  int since = 0;
  for (int t = 0; t < nsteps; ++t) {
    if (xu) sample(t);
    S.extend(x, xe);
    if (xs64) store_block<E>(mv, xs64, t, 0, S.w, S.lane, x);
    tendency<E>(xe, F, k);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      acc[j] = k[j];
      xs[j] = x[j] + (0.5 * h) * k[j];
    }
    S.extend(xs, xe);
    if (xs64) store_block<E>(mv, xs64, t, 1, S.w, S.lane, xs);
    tendency<E>(xe, F, k);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      acc[j] += 2.0 * k[j];
      xs[j] = x[j] + (0.5 * h) * k[j];
    }
    S.extend(xs, xe);
    if (xs64) store_block<E>(mv, xs64, t, 2, S.w, S.lane, xs);
    tendency<E>(xe, F, k);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      acc[j] += 2.0 * k[j];
      xs[j] = x[j] + h * k[j];
    }
    S.extend(xs, xe);
    if (xs64) store_block<E>(mv, xs64, t, 3, S.w, S.lane, xs);
    tendency<E>(xe, F, k);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      acc[j] += k[j];
      x[j] = x[j] + (h / 6.0) * acc[j];
    }
    if (++since == every) {
      S.refresh(xw);
      since = 0;
    }
  }
  if (xu) sample(nsteps);
  if (xs64) store_block<E>(mv, xs64, nsteps, 0, S.w, S.lane, x);
  if (xout) {
    if (mv.NW > 1) __syncthreads();  // (xout may be x0: every wave has taken its window from it)
    S.store_vec(xout, x);
  }
}

template <int E, int TH>
__global__ void __launch_bounds__(TH)
    trajectory_kernel(ModelView mv, int nsteps, const double *__restrict__ x0,
                      double *__restrict__ xout, double *__restrict__ xs64,
                      double *__restrict__ xu) {
  extern __shared__ double lds_d[];
  if (xu) {  // one workgroup per initial state
    x0 += (size_t)blockIdx.x * mv.n;
    xu += (size_t)blockIdx.x * mv.U;
  }
  trajectory_window<E>(mv, nsteps, x0, xout, xs64, xu, lds_d, xs64 ? blockIdx.x : -1);
}

// One workgroup per problem of a batch (waves beyond a problem's strips leave at once; a
// problem of one strip needs no barrier).
__global__ void __launch_bounds__(256)
    trajectory_batched_kernel(const TrajJob *__restrict__ jobs) {
  extern __shared__ double lds_d[];
  const TrajJob J = jobs[blockIdx.x];
  switch (J.mv.E) {
    case 3: trajectory_window<3>(J.mv, J.mv.T, J.x0, nullptr, J.xs64, nullptr, lds_d); break;
    case 5: trajectory_window<5>(J.mv, J.mv.T, J.x0, nullptr, J.xs64, nullptr, lds_d); break;
    case 9: trajectory_window<9>(J.mv, J.mv.T, J.x0, nullptr, J.xs64, nullptr, lds_d); break;
    default: trajectory_window<17>(J.mv, J.mv.T, J.x0, nullptr, J.xs64, nullptr, lds_d);
  }
}

// ---------------------------------------------------------------------------
// TL/AD sweeps of a block of members, one workgroup each.
// ---------------------------------------------------------------------------
template <int E, int TH, int MB>
__global__ void __launch_bounds__(TH)
    tlad_kernel(ModelView mv, int m, int mode, const double *__restrict__ dx0,
                double *__restrict__ lam0, double *__restrict__ f, const double *__restrict__ fsrc) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int mem = blockIdx.x * MB;
  Strip<E, MB> S(mv, reinterpret_cast<double *>(lds_raw), threadIdx.x);
  S.run(mode, dx0 + (size_t)mem * mv.n, lam0 + (size_t)mem * mv.n,
        f + (size_t)mem * (size_t)mv.U, fsrc, min(MB, m - mem));
}

// ---------------------------------------------------------------------------
// Persistent TL/AD over a batch of independent problems. Phase 1: each workgroup takes
// whole-workgroup tiles (members of several strips) from an atomic counter; phase 2: each
// wave takes tiles of members of one strip from a second counter. The tile lists are in
// decreasing cost order, so the longest integrations start first and the short ones fill the
// tail. Every wave leaves once both lists are exhausted.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void run_tile(int mode, const TladProb &P, int mem, double *lds, int tid) {
  const ModelView mv = P.mv;
  const size_t n = (size_t)mv.n, U = (size_t)mv.U;
  const double *dx0 = P.dx0 ? P.dx0 + (size_t)mem * n : nullptr;
  double *lam0 = P.lam0 ? P.lam0 + (size_t)mem * n : nullptr;
  double *f = P.f ? reinterpret_cast<double *>(P.f) + (size_t)mem * U : nullptr;
  const double *fsrc = reinterpret_cast<const double *>(P.fsrc);
  auto go = [&](auto e) {
    Strip<decltype(e)::value> S(mv, lds, tid);
    if (S.w < mv.NW) S.run(mode, dx0, lam0, f, fsrc);
  };
  switch (mv.E) {
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 9: go(std::integral_constant<int, 9>{}); break;
    default: go(std::integral_constant<int, 17>{});
  }
}

__global__ void __launch_bounds__(256)
    tlad_persistent_kernel(int mode, const TladProb *__restrict__ probs,
                           const TladTile *__restrict__ wg_tiles, int n_wg,
                           const TladTile *__restrict__ wave_tiles, int n_wave,
                           int *__restrict__ counters, long long *__restrict__ clk) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double *lds = reinterpret_cast<double *>(lds_raw);
  __shared__ int tile_sh;
  for (;;) {
    if (threadIdx.x == 0) tile_sh = atomicAdd(&counters[0], 1);
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(tile_sh);
    __syncthreads();  // every thread has its tile before thread 0 fetches the next
    if (t >= n_wg) break;
    const TladTile tile = wg_tiles[t];
    const long long c0 = clk ? wall_clock64() : 0;
    run_tile(mode, probs[tile.prob], tile.mem, lds, threadIdx.x);
    __syncthreads();  // the tile's LDS traffic is over before the next tile starts
    if (clk && threadIdx.x == 0) {
      clk[2 * t] = c0;
      clk[2 * t + 1] = wall_clock64();
    }
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double *wlds = lds + (size_t)wave * kWaveLds;
  for (;;) {
    int t = 0;
    if (lane == 0) t = atomicAdd(&counters[1], 1);
    t = __builtin_amdgcn_readfirstlane(t);
    if (t >= n_wave) break;
    const TladTile tile = wave_tiles[t];
    const long long c0 = clk ? wall_clock64() : 0;
    run_tile(mode, probs[tile.prob], tile.mem, wlds, lane);
    if (clk && lane == 0) {
      clk[2 * (n_wg + t)] = c0;
      clk[2 * (n_wg + t) + 1] = wall_clock64();
    }
  }
}

// ---------------------------------------------------------------------------
// Innovation, gradient forcing and cost.
// ---------------------------------------------------------------------------

// Place of element i's own copy in stage block (t, 0).
__device__ __forceinline__ size_t stage_index(const ModelView &mv, int t, int i) {
  const int w = i / mv.own, q = i - w * mv.own + mv.HL, l = q / mv.E;
  return ((size_t)(t * 4) * mv.NW + w) * (size_t)(64 * mv.E) + base_index(mv.E, q - l * mv.E, l);
}

__global__ void innovation_kernel(ModelView mv, const double *__restrict__ xs64, int U,
                                  const int *__restrict__ obs_step, const int *__restrict__ obs_idx,
                                  const double *__restrict__ y, const double *__restrict__ rinv,
                                  const int *__restrict__ u_optr, const int *__restrict__ u_olist,
                                  double *__restrict__ d, double *__restrict__ fgrad,
                                  const InnovJob *__restrict__ jobs) {
  if (jobs) {  // batched: blockIdx.y selects the problem
    const InnovJob &J = jobs[blockIdx.y];
    mv = J.mv, xs64 = J.xs64, U = J.mv.U, obs_step = J.obs_step, obs_idx = J.obs_idx, y = J.y;
    rinv = J.rinv, u_optr = J.u_optr, u_olist = J.u_olist, d = J.d;
    fgrad = reinterpret_cast<double *>(J.fgrad);
  }
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= U) return;
  double acc = 0.0;
  for (int q = u_optr[u]; q < u_optr[u + 1]; ++q) {
    const int o = u_olist[q];
    const int t = obs_step[o];
    const int i = obs_idx[o];
    const double xv = xs64[stage_index(mv, t, i)];
    const double dv = y[o] - xv;
    d[o] = dv;
    acc += rinv[o] * dv;
  }
  fgrad[u] = acc;
}

// Observed values of a stored window segment: out[o] = x_t[i] for the observations whose
// step t lies in (lo, lo + T] (and t = lo when include_lo), read from block (t - lo, 0).
__global__ void obs_value_kernel(ModelView mv, const double *__restrict__ xs64, int nobs,
                                 const int *__restrict__ obs_step, const int *__restrict__ obs_idx,
                                 int lo, int include_lo, double *__restrict__ out) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= nobs) return;
  const int t = obs_step[o];
  if (t < lo || t > lo + mv.T || (t == lo && !include_lo)) return;
  const int i = obs_idx[o];
  out[o] = xs64[stage_index(mv, t - lo, i)];
}

// Z[o, j] = f_j[u(o)] : raw TL values back in the caller's observation order, multiplied by
// sqrt(rinv[o]) when rinv is given (the R^{-1/2} factor of the dual operator).
template <typename Real>
__global__ void obs_gather_kernel(int nobs, int U, int m, const int *__restrict__ u_of_o,
                                  const Real *__restrict__ f, double *__restrict__ Z,
                                  const double *__restrict__ rinv) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)nobs * m) return;
  const int o = (int)(idx % nobs), j = (int)(idx / nobs);
  const double z = (double)f[(size_t)j * U + u_of_o[o]];
  Z[idx] = rinv ? sqrt(rinv[o]) * z : z;
}

// f_j[u] = sum_{o in u} F[o, j] : observation-space forcing folded onto unique pairs (each
// F[o, j] first multiplied by sqrt(rinv[o]) when rinv is given).
template <typename Real>
__global__ void obs_scatter_kernel(int nobs, int U, int m, const int *__restrict__ u_optr,
                                   const int *__restrict__ u_olist, const double *__restrict__ Fo,
                                   Real *__restrict__ f, const double *__restrict__ rinv) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)U * m) return;
  const int u = (int)(idx % U), j = (int)(idx / U);
  double s = 0.0;
  for (int q = u_optr[u]; q < u_optr[u + 1]; ++q) {
    const int o = u_olist[q];
    const double v = Fo[(size_t)j * nobs + o];
    s += rinv ? sqrt(rinv[o]) * v : v;
  }
  f[idx] = (Real)s;
}

// Dual right-hand side and increment scaling: out[o] = sqrt(rinv[o]) (d[o] - bp[o]) (bp may be
// nullptr), and dw[o] = -sqrt(rinv[o]) t[o] (t from the negated low-rank combination).
__global__ void psas_rhs_kernel(int nobs, const double *__restrict__ rinv,
                                const double *__restrict__ d, const double *__restrict__ bp,
                                double *__restrict__ out) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= nobs) return;
  out[o] = sqrt(rinv[o]) * (bp ? d[o] - bp[o] : d[o]);
}

// Perturbed observations of one gradient sample: out[o] = y[o] - eps[o] / sqrt(rinv[o]).
__global__ void obs_perturb_kernel(int nobs, const double *__restrict__ y,
                                   const double *__restrict__ rinv, const double *__restrict__ eps,
                                   double *__restrict__ out) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= nobs) return;
  out[o] = y[o] - eps[o] / sqrt(rinv[o]);
}

__global__ void psas_scale_kernel(int nobs, const double *__restrict__ rinv,
                                  const double *__restrict__ t, double *__restrict__ dw) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= nobs) return;
  dw[o] = -sqrt(rinv[o]) * t[o];
}

__global__ void __launch_bounds__(1024)
    cost_kernel(int n, const double *__restrict__ v, int nobs, const double *__restrict__ d,
                const double *__restrict__ rinv, double *__restrict__ out) {
  __shared__ double red[16];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    if (v) a += v[i] * v[i];
  for (int o = threadIdx.x; o < nobs; o += blockDim.x) b += rinv[o] * d[o] * d[o];
  const double sa = block_sum(a, red);
  const double sb = block_sum(b, red);
  if (threadIdx.x == 0) out[0] = 0.5 * sa + 0.5 * sb;
}

// ---------------------------------------------------------------------------
// L (symmetric circulant, half-kernel taps) applied to columns.
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(256)
    apply_L_kernel(int n, int w, const double *__restrict__ taps, const double *__restrict__ X,
                   double *__restrict__ Y, const double *__restrict__ Z, int mode, int use_lds,
                   const ApplyLJobE *__restrict__ jobs) {
  extern __shared__ double ext[];
  const size_t c = blockIdx.x;
  if (jobs) {  // batched: blockIdx.y selects the problem, blockIdx.x the column
    const ApplyLJobE &J = jobs[blockIdx.y];
    if ((int)c >= J.m) return;
    n = J.n, w = J.w, taps = J.taps, X = J.X, Y = J.Y, Z = J.Z, mode = J.mode;
  }
  apply_L_column(n, w, taps, X + c * n, Y + c * n, Z ? Z + c * n : nullptr, mode,
                 use_lds ? ext : nullptr);
}

// The same product for one segment of kLSeg rows of one column per workgroup (grid: column,
// segment): the segment with its w-row halo on each side is staged in LDS, and the sums run
// in the order of apply_L_column, so results are identical. A column split into segments
// gives a block of m columns n / kLSeg times as many workgroups to hide the LDS latency.
constexpr int kLSeg = 1024;

__global__ void __launch_bounds__(256)
    apply_L_seg_kernel(int n, int w, const double *__restrict__ taps, const double *__restrict__ X,
                       double *__restrict__ Y, const double *__restrict__ Z, int mode) {
  extern __shared__ double ext[];
  const size_t c = blockIdx.x;
  const int r0 = blockIdx.y * kLSeg, len = min(kLSeg, n - r0);
  const double *x = X + c * n;
  const int tot = len + 2 * w;
  auto src_of = [&](int k) {
    int src = (r0 + k - w) % n;
    return src < 0 ? src + n : src;
  };
  if (tot <= 6 * 256 && blockDim.x == 256) {
    // the segment's loads all issued before the first wait (one memory latency, not one per
    // round of 256)
    double v[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int k = threadIdx.x + 256 * t;
      v[t] = x[src_of(k < tot ? k : 0)];
    }
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int k = threadIdx.x + 256 * t;
      if (k < tot) ext[k] = v[t];
    }
  } else {
    for (int k = threadIdx.x; k < tot; k += blockDim.x) ext[k] = x[src_of(k)];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < len; i += blockDim.x) {
    double acc = taps[0] * ext[i + w];
    for (int dd = 1; dd <= w; ++dd) acc += taps[dd] * (ext[i + w + dd] + ext[i + w - dd]);
    const size_t o = c * n + r0 + i;
    if (mode == 1)
      acc += Z[o];
    else if (mode == 2)
      acc = (Z ? Z[o] : 0.0) - acc;
    Y[o] = acc;
  }
}

// ---------------------------------------------------------------------------
// Conjugate gradients: one workgroup, all iterations in one launch.
// ---------------------------------------------------------------------------

template <int E, int TH>
__global__ void __launch_bounds__(TH)
    cg_kernel(ModelView mv, int w, const double *__restrict__ taps, const double *__restrict__ g,
              int iters, double rtol, double *__restrict__ x, double *__restrict__ iterates,
              double *__restrict__ vs, double *__restrict__ f, int *__restrict__ used,
              int ext_off_bytes, int use_lds_ext) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ double red[16];
  double *lds = reinterpret_cast<double *>(lds_raw);
  double *ext = use_lds_ext ? reinterpret_cast<double *>(lds_raw + ext_off_bytes) : nullptr;
  const int n = mv.n;
  double *r = vs, *p = vs + n, *q = vs + 2 * n, *tmp = vs + 3 * n, *lam = vs + 4 * n;
  Strip<E> M(mv, lds, threadIdx.x);

  double rr_part = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double ri = -g[i];
    x[i] = 0.0;
    r[i] = ri;
    p[i] = ri;
    rr_part += ri * ri;
  }
  double rr = block_sum(rr_part, red);
  const double r0 = sqrt(rr);
  int it = 0;
  for (; it < iters; ++it) {
    // q = (I + A) p = p + L^T G^T R^{-1} G L p
    apply_L_column(n, w, taps, p, tmp, nullptr, 0, ext);
    M.run(0, tmp, lam, f, nullptr);
    __syncthreads();
    apply_L_column(n, w, taps, lam, q, p, 1, ext);
    double pq_part = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) pq_part += p[i] * q[i];
    const double pq = block_sum(pq_part, red);
    const double alpha = rr / pq;
    double rn_part = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      x[i] += alpha * p[i];
      const double ri = r[i] - alpha * q[i];
      r[i] = ri;
      rn_part += ri * ri;
      if (iterates) iterates[(size_t)it * n + i] = x[i];
    }
    const double rr_new = block_sum(rn_part, red);
    if (rtol > 0.0 && sqrt(rr_new) <= rtol * r0) {
      ++it;
      break;
    }
    const double beta = rr_new / rr;
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = r[i] + beta * p[i];
    rr = rr_new;
    __syncthreads();
  }
  if (threadIdx.x == 0) used[0] = it;
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC 2011) and Box-Muller normals.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += W0;
      k1 += W1;
    }
    const uint64_t p0 = (uint64_t)M0 * c[0];
    const uint64_t p1 = (uint64_t)M1 * c[2];
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

__global__ void philox_normal_kernel(long long total, uint64_t seed, uint64_t stream,
                                     double *__restrict__ out, const PhiloxJob *__restrict__ jobs) {
  if (jobs) {  // batched: blockIdx.y selects the problem (its own stream)
    const PhiloxJob &J = jobs[blockIdx.y];
    total = J.total, stream = J.stream, out = J.out;
  }
  const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long pairs = (total + 1) / 2;
  if (j >= pairs) return;
  uint32_t c[4] = {(uint32_t)j, (uint32_t)((unsigned long long)j >> 32), (uint32_t)stream,
                   (uint32_t)(stream >> 32)};
  philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
  const uint64_t v1 = (((uint64_t)c[1] << 32) | c[0]) >> 11;
  const uint64_t v2 = (((uint64_t)c[3] << 32) | c[2]) >> 11;
  const double u1 = ((double)v1 + 0.5) * 0x1.0p-53;
  const double u2 = ((double)v2 + 0.5) * 0x1.0p-53;
  const double r = sqrt(-2.0 * log(u1));
  const double th = 2.0 * 3.14159265358979323846 * u2;
  out[2 * j] = r * cos(th);
  if (2 * j + 1 < total) out[2 * j + 1] = r * sin(th);
}

// ---------------------------------------------------------------------------
// Deterministic LRA/LRU choice: candidate states, non-quadratic costs, selection.
// ---------------------------------------------------------------------------

// xc[c] = x + dx[c], vc[c] = v + dz[c] (v = nullptr: zero), c = 0 .. nc-1, n-vectors.
__global__ void cand_state_kernel(int n, int nc, const double *__restrict__ x,
                                  const double *__restrict__ v, const double *__restrict__ dz,
                                  const double *__restrict__ dx, double *__restrict__ xc,
                                  double *__restrict__ vc) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)n * nc) return;
  const int i = (int)(e % n);
  xc[e] = x[i] + dx[e];
  vc[e] = (v ? v[i] : 0.0) + dz[e];
}

// J[c] = 1/2 vc^T vc + 1/2 sum_o rinv_o (y_o - x_c at o)^2 (eq. 2 in control variables), one
// workgroup per candidate, sums in a fixed order.
__global__ void __launch_bounds__(1024)
    cand_cost_kernel(int n, const double *__restrict__ vc, int nobs, int U,
                     const double *__restrict__ y, const double *__restrict__ rinv,
                     const int *__restrict__ u_of_o, const double *__restrict__ xu,
                     double *__restrict__ J) {
  __shared__ double red[16];
  const int c = blockIdx.x;
  const double *v = vc + (size_t)c * n;
  const double *xo = xu + (size_t)c * U;
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) a += v[i] * v[i];
  for (int o = threadIdx.x; o < nobs; o += blockDim.x) {
    const double d = y[o] - xo[u_of_o[o]];
    b += rinv[o] * d * d;
  }
  const double sa = block_sum(a, red);
  const double sb = block_sum(b, red);
  if (threadIdx.x == 0) J[c] = 0.5 * sa + 0.5 * sb;
}

// The candidate with the lowest cost (the first on a tie; a non-finite cost never beats a
// finite one) is copied to dz, dx; its index is written to mode_out (candidate 0 = LRA,
// 1 = LRU: RIOT_LRA or RIOT_LRU).
__global__ void cand_select_kernel(int n, int nc, const double *__restrict__ J,
                                   const double *__restrict__ dzc, const double *__restrict__ dxc,
                                   double *__restrict__ dz, double *__restrict__ dx,
                                   int *__restrict__ mode_out) {
  int best = 0;
  for (int c = 1; c < nc; ++c)
    if (isfinite(J[c]) && (!isfinite(J[best]) || J[c] < J[best])) best = c;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    dz[i] = dzc[(size_t)best * n + i];
    dx[i] = dxc[(size_t)best * n + i];
  }
  if (i == 0 && mode_out) mode_out[0] = best == 0 ? RIOT_LRA : RIOT_LRU;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------


// Strip widths and the largest workgroups that strip_layout uses them with.
#define RIOT_DISPATCH_E(MV, CALL)                  \
  switch ((MV).E) {                                \
    case 2: {                                      \
      constexpr int EE = 2, TH = 256;              \
      CALL;                                        \
    } break;                                       \
    case 3: {                                      \
      constexpr int EE = 3, TH = 256;              \
      CALL;                                        \
    } break;                                       \
    case 5: {                                      \
      constexpr int EE = 5, TH = 512;              \
      CALL;                                        \
    } break;                                       \
    case 9: {                                      \
      constexpr int EE = 9, TH = 512;              \
      CALL;                                        \
    } break;                                       \
    case 17: { /* a problem of a batch */          \
      constexpr int EE = 17, TH = 256;             \
      CALL;                                        \
    } break;                                       \
    default: return hipErrorInvalidValue;          \
  }

// LDS elements of a workgroup of mb members: halo buffers (both parities) and staging rows
static size_t strip_lds(const ModelView &mv, int mb) {
  const int ew = mv.HL + mv.HR;
  const size_t halo = mv.n < ew + mv.E ? mv.n : mv.NW * (ew + 4 * mv.E);
  return 2 * mb * halo + (size_t)mv.NW * 64 * mv.E;
}

hipError_t launch_trajectory(const ModelView &mv, int nsteps, const double *x0, double *xout,
                             double *xs64, float *xs32, hipStream_t st) {
  if (mv.NT) return lanes_trajectory(mv, nsteps, x0, xout, xs64, xs32, st);
  const size_t lds = strip_lds(mv, 1) * sizeof(double);
  // One compute unit stores 64 bytes a clock, less than a trajectory of many strips produces, so
  // NW workgroups each run the whole trajectory and store one strip's stage blocks.
  const dim3 grid(xs64 ? mv.NW : 1);
  RIOT_DISPATCH_E(mv, hipLaunchKernelGGL((trajectory_kernel<EE, TH>), grid, dim3(64 * mv.NW), lds,
                                         st, mv, nsteps, x0, xout, xs64, nullptr));
  return hipGetLastError();
}

hipError_t launch_window_obs(const ModelView &mv, int nstates, const double *x0, double *xu,
                             hipStream_t st) {
  if (nstates <= 0) return hipSuccess;
  if (mv.NT) return lanes_window_obs(mv, nstates, x0, xu, st);
  const size_t lds = strip_lds(mv, 1) * sizeof(double);
  RIOT_DISPATCH_E(mv, hipLaunchKernelGGL((trajectory_kernel<EE, TH>), dim3(nstates),
                                         dim3(64 * mv.NW), lds, st, mv, mv.T, x0, nullptr, nullptr, xu));
  return hipGetLastError();
}

hipError_t launch_cand_state(int n, int nc, const double *x, const double *v, const double *dz,
                             const double *dx, double *xc, double *vc, hipStream_t st) {
  const long long tot = (long long)n * nc;
  hipLaunchKernelGGL(cand_state_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n,
                     nc, x, v, dz, dx, xc, vc);
  return hipGetLastError();
}

hipError_t launch_cand_cost(int n, int nc, const double *vc, int nobs, int U, const double *y,
                            const double *rinv, const int *u_of_o, const double *xu, double *J,
                            hipStream_t st) {
  hipLaunchKernelGGL(cand_cost_kernel, dim3(nc), dim3(1024), 0, st, n, vc, nobs, U, y, rinv,
                     u_of_o, xu, J);
  return hipGetLastError();
}

hipError_t launch_cand_select(int n, int nc, const double *J, const double *dzc, const double *dxc,
                              double *dz, double *dx, int *mode_out, hipStream_t st) {
  hipLaunchKernelGGL(cand_select_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, nc, J, dzc,
                     dxc, dz, dx, mode_out);
  return hipGetLastError();
}

hipError_t launch_innovation(const ModelView &mv, const double *xs64, int nobs, const int *obs_step,
                             const int *obs_idx, const double *y, const double *rinv,
                             const int *u_optr, const int *u_olist, double *d, void *fgrad,
                             bool fp32, hipStream_t st) {
  (void)nobs;
  if (mv.U == 0) return hipSuccess;
  if (mv.NT)
    return lanes_innovation(mv, xs64, obs_step, obs_idx, y, rinv, u_optr, u_olist, d, fgrad, fp32,
                            st);
  const int bs = 256;
  const int grid = (mv.U + bs - 1) / bs;
  hipLaunchKernelGGL(innovation_kernel, dim3(grid), dim3(bs), 0, st, mv, xs64, mv.U, obs_step,
                     obs_idx, y, rinv, u_optr, u_olist, d, reinterpret_cast<double *>(fgrad),
                     nullptr);
  return hipGetLastError();
}

hipError_t launch_cost(int n, const double *v, int nobs, const double *d, const double *rinv,
                       double *out, hipStream_t st) {
  hipLaunchKernelGGL(cost_kernel, dim3(1), dim3(1024), 0, st, n, v, nobs, d, rinv, out);
  return hipGetLastError();
}

hipError_t launch_tlad(const ModelView &mv, int m, int mode, const double *dx0, double *lam0,
                       void *f, const void *fsrc, bool fp32, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  if (mv.NT) return lanes_tlad(mv, m, mode, dx0, lam0, f, fsrc, fp32, st);
  // Two members per workgroup where each compute unit would otherwise run its workgroups one
  // after the other (a workgroup of 9 positions per lane fills one: eight waves of 256
  // registers): they share the base loads and hide each other's latencies. n = 4096, T = 100:
  // m = 272 at two each 0.58 ms, one each 2 x 0.43 ms.
  if (mv.E == 9 && m > mv.cus) {
    hipLaunchKernelGGL((tlad_kernel<9, 512, 2>), dim3((m + 1) / 2), dim3(64 * mv.NW),
                       strip_lds(mv, 2) * sizeof(double), st, mv, m, mode, dx0, lam0,
                       reinterpret_cast<double *>(f), reinterpret_cast<const double *>(fsrc));
    return hipGetLastError();
  }
  RIOT_DISPATCH_E(mv, hipLaunchKernelGGL((tlad_kernel<EE, TH, 1>), dim3(m), dim3(64 * mv.NW),
                                         strip_lds(mv, 1) * sizeof(double), st, mv, m, mode, dx0,
                                         lam0, reinterpret_cast<double *>(f),
                                         reinterpret_cast<const double *>(fsrc)));
  return hipGetLastError();
}

hipError_t launch_obs_value(const ModelView &mv, const double *xs64, int nobs, const int *obs_step,
                            const int *obs_idx, int lo, bool include_lo, double *out,
                            hipStream_t st) {
  if (nobs <= 0) return hipSuccess;
  if (mv.NT)
    return lanes_obs_value(mv, xs64, nobs, obs_step, obs_idx, lo, include_lo, out, st);
  hipLaunchKernelGGL(obs_value_kernel, dim3((nobs + 255) / 256), dim3(256), 0, st, mv, xs64, nobs,
                     obs_step, obs_idx, lo, include_lo ? 1 : 0, out);
  return hipGetLastError();
}

hipError_t launch_obs_gather(int nobs, int U, int m, const int *u_of_o, const void *f, double *Z,
                             bool fp32, hipStream_t st, const double *rinv) {
  const size_t tot = (size_t)nobs * m;
  if (tot == 0) return hipSuccess;
  const unsigned grid = (unsigned)((tot + 255) / 256);
  if (fp32)
    hipLaunchKernelGGL(obs_gather_kernel<float>, dim3(grid), dim3(256), 0, st, nobs, U, m, u_of_o,
                       reinterpret_cast<const float *>(f), Z, rinv);
  else
    hipLaunchKernelGGL(obs_gather_kernel<double>, dim3(grid), dim3(256), 0, st, nobs, U, m, u_of_o,
                       reinterpret_cast<const double *>(f), Z, rinv);
  return hipGetLastError();
}

hipError_t launch_obs_scatter(int nobs, int U, int m, const int *u_optr, const int *u_olist,
                              const double *Fo, void *f, bool fp32, hipStream_t st,
                              const double *rinv) {
  const size_t tot = (size_t)U * m;
  if (tot == 0) return hipSuccess;
  const unsigned grid = (unsigned)((tot + 255) / 256);
  if (fp32)
    hipLaunchKernelGGL(obs_scatter_kernel<float>, dim3(grid), dim3(256), 0, st, nobs, U, m, u_optr,
                       u_olist, Fo, reinterpret_cast<float *>(f), rinv);
  else
    hipLaunchKernelGGL(obs_scatter_kernel<double>, dim3(grid), dim3(256), 0, st, nobs, U, m, u_optr,
                       u_olist, Fo, reinterpret_cast<double *>(f), rinv);
  return hipGetLastError();
}

hipError_t launch_psas_rhs(int nobs, const double *rinv, const double *d, const double *bp,
                           double *out, hipStream_t st) {
  if (nobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(psas_rhs_kernel, dim3((nobs + 255) / 256), dim3(256), 0, st, nobs, rinv, d, bp,
                     out);
  return hipGetLastError();
}

hipError_t launch_obs_perturb(int nobs, const double *y, const double *rinv, const double *eps,
                              double *out, hipStream_t st) {
  if (nobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(obs_perturb_kernel, dim3((nobs + 255) / 256), dim3(256), 0, st, nobs, y, rinv,
                     eps, out);
  return hipGetLastError();
}

hipError_t launch_psas_scale(int nobs, const double *rinv, const double *t, double *dw,
                             hipStream_t st) {
  if (nobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(psas_scale_kernel, dim3((nobs + 255) / 256), dim3(256), 0, st, nobs, rinv, t,
                     dw);
  return hipGetLastError();
}

hipError_t launch_apply_L(int n, int w, const double *taps, int m, const double *X, double *Y,
                          const double *Z, int mode, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  const size_t seg_lds = (size_t)(kLSeg + 2 * w) * sizeof(double);
  if (seg_lds <= 60 * 1024) {
    const unsigned nseg = (unsigned)((n + kLSeg - 1) / kLSeg);
    hipLaunchKernelGGL(apply_L_seg_kernel, dim3(m, nseg), dim3(256), seg_lds, st, n, w, taps, X, Y,
                       Z, mode);
    return hipGetLastError();
  }
  const size_t lds = (size_t)(n + 2 * w) * sizeof(double);
  const int use_lds = lds <= 60 * 1024 ? 1 : 0;
  hipLaunchKernelGGL(apply_L_kernel, dim3(m), dim3(256), use_lds ? lds : 0, st, n, w, taps, X, Y,
                     Z, mode, use_lds, nullptr);
  return hipGetLastError();
}

hipError_t launch_cg(const ModelView &mv, int w, const double *taps, const double *g, int iters,
                     double rtol, double *x, double *iterates, double *vec_scratch, void *f,
                     int *used, bool fp32, hipStream_t st) {
  if (mv.NT)
    return lanes_cg(mv, w, taps, g, iters, rtol, x, iterates, vec_scratch, f, used, fp32, st);
  const size_t xb = strip_lds(mv, 1) * sizeof(double);
  const size_t ext_off = (xb + 255) / 256 * 256;
  const size_t ext_bytes = (size_t)(mv.n + 2 * w) * sizeof(double);
  const int use_ext = (ext_off + ext_bytes) <= 60 * 1024 ? 1 : 0;
  const size_t lds = use_ext ? ext_off + ext_bytes : xb;
  RIOT_DISPATCH_E(mv, hipLaunchKernelGGL((cg_kernel<EE, TH>), dim3(1), dim3(64 * mv.NW), lds, st,
                                         mv, w, taps, g, iters, rtol, x, iterates, vec_scratch,
                                         reinterpret_cast<double *>(f), used, (int)ext_off,
                                         use_ext));
  return hipGetLastError();
}

hipError_t launch_philox_normal(long long total, uint64_t seed, uint64_t stream, double *out,
                                hipStream_t st) {
  if (total <= 0) return hipSuccess;
  const long long pairs = (total + 1) / 2;
  const int bs = 256;
  const long long grid = (pairs + bs - 1) / bs;
  hipLaunchKernelGGL(philox_normal_kernel, dim3((unsigned)grid), dim3(bs), 0, st, total, seed,
                     stream, out, nullptr);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// Batched launchers (workgroups of 256 threads, one or four strips per problem)
// ---------------------------------------------------------------------------

constexpr int kBatchThreads = 256;

hipError_t launch_trajectory_batched(int nprob, const TrajJob *jobs, bool fp32, hipStream_t st) {
  if (nprob <= 0) return hipSuccess;
  if (fp32) return lanes_trajectory_batched(nprob, jobs, st);
  hipLaunchKernelGGL(trajectory_batched_kernel, dim3(nprob), dim3(kBatchThreads),
                     (kBatchThreads / 64) * kWaveLds * sizeof(double), st, jobs);
  return hipGetLastError();
}

hipError_t launch_innovation_batched(int nprob, int maxU, const InnovJob *jobs, bool fp32,
                                     hipStream_t st) {
  if (nprob <= 0 || maxU <= 0) return hipSuccess;
  if (fp32) return lanes_innovation_batched(nprob, maxU, jobs, st);
  hipLaunchKernelGGL(innovation_kernel, dim3((maxU + 255) / 256, nprob), dim3(256), 0, st,
                     ModelView{}, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                     nullptr, nullptr, jobs);
  return hipGetLastError();
}

constexpr size_t kPersistentLds = (size_t)(kBatchThreads / 64) * kWaveLds * sizeof(double);

hipError_t launch_tlad_persistent(int nwg, int mode, const TladProb *probs, const TladTile *wg_tiles,
                                  int n_wg, const TladTile *wave_tiles, int n_wave, int *counters,
                                  bool fp32, hipStream_t st, long long *clk) {
  if (nwg <= 0 || (n_wg <= 0 && n_wave <= 0)) return hipSuccess;
  hipError_t e = launch_zero_ints(counters, 2, st);
  if (e != hipSuccess) return e;
  if (fp32)
    return lanes_tlad_persistent(nwg, mode, probs, wg_tiles, n_wg, wave_tiles, n_wave, counters, st,
                                 clk);
  hipLaunchKernelGGL(tlad_persistent_kernel, dim3(nwg), dim3(kBatchThreads), kPersistentLds, st,
                     mode, probs, wg_tiles, n_wg, wave_tiles, n_wave, counters, clk);
  return hipGetLastError();
}

int tlad_persistent_resident_per_cu(bool fp32) {
  if (fp32) return lanes_persistent_resident_per_cu();
  int nb = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &nb, tlad_persistent_kernel, kBatchThreads, kPersistentLds);
  return e == hipSuccess ? nb : 0;
}

hipError_t launch_apply_L_batched(int nprob, int maxm, int maxext, const ApplyLJobE *jobs,
                                  hipStream_t st) {
  if (nprob <= 0 || maxm <= 0) return hipSuccess;
  const size_t lds = (size_t)maxext * sizeof(double);
  if (lds > 60 * 1024) return hipErrorInvalidValue;
  hipLaunchKernelGGL(apply_L_kernel, dim3(maxm, nprob), dim3(256), lds, st, 0, 0, nullptr, nullptr,
                     nullptr, nullptr, 0, 1, jobs);
  return hipGetLastError();
}

hipError_t launch_philox_batched(int nprob, long long maxtotal, uint64_t seed,
                                 const PhiloxJob *jobs, hipStream_t st) {
  if (nprob <= 0 || maxtotal <= 0) return hipSuccess;
  const long long pairs = (maxtotal + 1) / 2;
  hipLaunchKernelGGL(philox_normal_kernel, dim3((unsigned)((pairs + 255) / 256), nprob), dim3(256),
                     0, st, 0LL, seed, 0ULL, nullptr, jobs);
  return hipGetLastError();
}

}  // namespace riot
