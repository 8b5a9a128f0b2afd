// Tracer source inversion on a periodic 2-D grid: forward model, tangent-linear and adjoint
// sweeps over a batch of members, the square root of B, and the prior-preconditioned
// Hessian product of Alg. 3 for this model.
//
// Model (a synthetic stand-in for the transport model of the paper's black-carbon
// inversion, Sec. 3.2): explicit upwind advection by a positive wind (u(y) along x, v
// along y) and 5-point diffusion on an N x N periodic grid, emissions E * exp(s) on
// coarse space-time blocks of controls s (the lognormal transform of Sec. 3.2), point
// observations. The transport is linear in the concentration, so the tangent and the
// adjoint need the base emissions only, never a stored trajectory.
//
// Layout: fields [member][y][x] (x fastest); controls [member][time block][by][bx].
// A sweep runs up to eight steps per launch: a wave marches down the rows of a strip of
// columns with all the group's steps in flight at once, one row apart, in registers.

#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "riot_internal.h"

namespace riot {
namespace {

struct TracerView {
  int N, T, block, bshift, ntb, Nb, spb;  // block = 1 << bshift; spb: steps per time block
  double dt, aS, aE, aN;
  const double *a0, *aW;          // [N] row coefficients
};

// ---------------------------------------------------------------------------
// Marching sweeps. A wave owns `width` columns (two adjacent cells per lane, 128 with a halo
// of kHalo cells on each side) and the rows [ys, ye) of one member's field, and advances the
// field S <= kMaxS steps in one pass over its rows: at iteration i it takes row r = ys - S + i
// of the input (level 0), and level s finishes row r - s of the field after s steps. The
// five-point stencil is applied in scatter form, so a level keeps one row of partial sums
// (everything but the next row's term) and one row of its input, and the chain through the
// levels of an iteration is one multiply-add per level. East and west neighbours come from
// the adjacent lanes by DPP moves; lanes at the strip's ends go wrong by one cell per level,
// which the halo absorbs, and so do the rows beyond [ys, ye) at the ends of the march.
// No LDS and no barrier: nothing is exchanged between waves.
//
// All steps of a launch lie in one time block, so the emission term of a cell is the same at
// every level: it is formed once per row and kept for the S - 1 rows until the last level
// has used it. Likewise the adjoint adds the levels' lam of a cell first and multiplies by
// dt W once. TWO: time blocks of one step each; a launch takes the steps of two blocks, with the
// weights, controls and gradients of both. (512 x 512, 24 blocks, 64 members: product 2.74 ms;
// one step per launch moves every field twice as often, 4.39 ms.)
//
// Bound: the fields' traffic, one read and one write per S steps (0.44 ms per launch at a
// copy's 4.9 TB/s for 512 members on 512 x 512 cells), and vector issue, about 300
// instructions per row of 8 levels at two waves per SIMD. Measured there, 96 steps: 0.60 ms
// (forward) and 0.70 ms (adjoint) per 8 steps, the Hessian product of 512 probes 62.4 ms (two
// steps per launch through LDS tiles, 3.1 TB/s) -> 16.8 ms; S = 6: 18.9 ms, S = 4: 26.6 ms.
// Held to three waves per SIMD the registers spill (71 ms). One member, where a launch lasts
// as long as one march: value and gradient 810 -> 520 us.
// ---------------------------------------------------------------------------
constexpr int kMaxS = 8;    // steps per launch; the register rings below have kMaxS rows
constexpr int kHalo = 8;    // >= kMaxS, a multiple of 4 (the largest control block side)
constexpr int kCells = 128; // cells per wave row
constexpr int kAhead = 4;   // rows loaded ahead; divides kMaxS
constexpr int kAheadG = 2;  // the same for what stays in L2: cell lists; adjoint: weights, old gS
constexpr int kLevShift = 27;  // level 8 stays positive

typedef double d2 __attribute__((ext_vector_type(2)));

struct MarchArgs {
  int ns, width;              // strips across x, columns per strip (a multiple of 4)
  int nch, rows;              // chunks down y, rows per chunk (a multiple of 4)
  int m;                      // members
  const double *in;           // input fields, or null: zero
  double *out;                // fields after S steps, or null: not needed
  const double *W;            // [N*N] emission weights of the time block
  const double *bv;           // forward: [mem][Nb*Nb] control values of the time block
  long long bv_stride;
  double *gS;                 // adjoint: [mem][Nb*Nb] control gradient of the time block
  long long gS_stride;
  // where the launch's two steps lie in two time blocks: the second one's
  const double *W2, *bv2;
  double *gS2;
  int gS_add;                 // 0: gS is written, 1: added to
  // cells sampled (forward: observations) or forced (adjoint: unique cells) in this group, in
  // the order of the march: entries [ptr[r], ptr[r + 1]) lie in rows (r - lev) mod N, which
  // level lev finishes when row r is taken in; ent holds x + (lev << kLevShift)
  const int *ptr, *ent;
  const int *orig;            // forward: caller's index of each entry
  int nobs;
  double *obs;                // forward: [mem][nobs] out, or null
  const double *fu;           // adjoint: [mem][nuniq] forcing of each entry's cell
  int nuniq;
};

// value of the lane one below (shr) or above (shl); the end lane gets zero
template <int CTRL>
__device__ __forceinline__ double dpp_shift(double v) {
  union { double d; int i[2]; } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, 0xf, 0xf, true);
  return b.d;
}
__device__ __forceinline__ double from_below(double v) { return dpp_shift<0x138>(v); }  // wave_shr:1
__device__ __forceinline__ double from_above(double v) { return dpp_shift<0x130>(v); }  // wave_shl:1

// element of a row (wave-uniform address) at a lane's byte offset
template <typename T>
__device__ __forceinline__ gmem<T> *row_at(double *row, unsigned off) {
  return (gmem<T> *)((gmem<char> *)row + off);
}
template <typename T>
__device__ __forceinline__ const gmem<T> *row_at(const double *row, unsigned off) {
  return (const gmem<T> *)((const gmem<char> *)row + off);
}

// LDS written by other lanes of this wave may be read after it (a wave's LDS accesses stay in
// order; this keeps the compiler from reordering or forwarding them)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ d2 own_copy(d2 v) {
  d2 r;
  asm("v_mov_b64 %0, %1" : "=v"(r.x) : "v"(v.x));
  asm("v_mov_b64 %0, %1" : "=v"(r.y) : "v"(v.y));
  return r;
}

__device__ __forceinline__ int wrap(int i, int N) { return i < 0 ? i + N : (i >= N ? i - N : i); }

template <bool ADJ, int S, bool TWO = false>
__global__ void __launch_bounds__(64, S > 4 ? 2 : 3)
    tracer_march_kernel(TracerView tv, MarchArgs a, const double *__restrict__ ca0,
                        const double *__restrict__ caW, const int *__restrict__ ptr) {
  constexpr int R = S <= 4 ? 4 : kMaxS;  // rows of the rings below, unrolled iterations
  static_assert(S >= 1 && S <= kMaxS && kHalo >= kMaxS && R % kAhead == 0 && (!TWO || S == 2), "");
  __shared__ double rows[S][kCells];  // levels' rows sampled, or their forcing, at one iteration
  const int N = tv.N, lane = threadIdx.x;
  // Workgroups are dealt round-robin to the 8 XCDs: the strips of one chunk go to one XCD,
  // one after the other, so that their overlapping columns are read into one L2.
  const int units = a.m * a.nch;
  int unit, strip;
  if ((units & 7) == 0) {
    const int q = blockIdx.x >> 3;
    strip = q % a.ns;
    unit = (q / a.ns) * 8 + (blockIdx.x & 7);
  } else {
    strip = blockIdx.x % a.ns;
    unit = blockIdx.x / a.ns;
  }
  const int mem = unit / a.nch, ch = unit - mem * a.nch;
  const int xs = strip * a.width, xe = min(xs + a.width, N);
  const int ys = ch * a.rows, ye = min(ys + a.rows, N);
  if (xs >= N || ys >= N) return;
  int x = xs - kHalo + 2 * lane;  // this lane's first cell, wrapped (N >= 64)
  const bool own = x >= xs && x < xe;
  x = x < 0 ? x + N : x;
  while (x >= N) x -= N;
  const size_t NN = (size_t)N * N;
  const bool has_in = a.in != nullptr;  // else any field is loaded and its values dropped
  const double *src = has_in ? a.in + mem * NN : a.W;
  const int sh = tv.bshift;
  const unsigned xo8 = 8u * x, xb8 = 8u * (x >> sh),
                 xc8 = 8u * ((x + 1) >> sh);  // byte offsets of this lane in a row
  const double *bvm = ADJ ? nullptr : a.bv + mem * a.bv_stride;
  const double *bvm2 = !ADJ && TWO ? a.bv2 + mem * a.bv_stride : nullptr;
  double *gSm = ADJ ? a.gS + mem * a.gS_stride : nullptr;
  double *gSm2 = ADJ && TWO ? a.gS2 + mem * a.gS_stride : nullptr;
  const int iters = ye - ys + 2 * S;

  d2 q[S], cold[S], ring[R];  // ring: emission terms (forward) or sums of lam (adjoint)
  d2 ring2[2];  // TWO: the second block's term of this row and of the one before (forward)
#pragma unroll
  for (int s = 0; s < S; ++s) q[s] = cold[s] = d2{0.0, 0.0};
#pragma unroll
  for (int s = 0; s < R; ++s) ring[s] = d2{0.0, 0.0};
  ring2[0] = ring2[1] = d2{0.0, 0.0};
  double r0[R], rW[R];  // a0 and aW of the last R rows
#pragma unroll
  for (int s = 0; s < R; ++s) r0[s] = rW[s] = 0.0;

  // rows in flight: input field and (forward: emission weights and controls of the same row;
  // adjoint: weights of the row whose sums complete at that iteration)
  constexpr int kAW = ADJ || TWO ? kAheadG : kAhead;  // (TWO: four rows of both blocks would spill)
  d2 fb[kAhead], wb[kAW], eb[kAW];  // eb: controls (forward), old gS of that row (adjoint)
  d2 wb2[kAW], eb2[kAW];            // TWO: the second block's
  int rl = wrap(ys - S, N), rw = ADJ ? wrap(wrap(ys - S - (S - 1), N), N) : rl;  // next rows to load
  auto issue_f = [&](int k) {
    fb[k] = *row_at<d2>(src + (size_t)rl * N, xo8);
    rl = rl + 1 == N ? 0 : rl + 1;
  };
  auto issue_w = [&](int k) {
    wb[k] = *row_at<d2>(a.W + (size_t)rw * N, xo8);
    const double *bp = (ADJ ? gSm : bvm) + (size_t)(rw >> sh) * tv.Nb;
    eb[k].x = *row_at<double>(bp, xb8);
    eb[k].y = *row_at<double>(bp, xc8);
    if constexpr (TWO) {
      wb2[k] = *row_at<d2>(a.W2 + (size_t)rw * N, xo8);
      if constexpr (!ADJ) {
        const double *bp2 = bvm2 + (size_t)(rw >> sh) * tv.Nb;
        eb2[k].x = *row_at<double>(bp2, xb8);
        eb2[k].y = *row_at<double>(bp2, xc8);
      }
    }
    rw = rw + 1 == N ? 0 : rw + 1;
  };
  int rc = wrap(ys - S, N);            // row taken in by this iteration
  // cell list of the rows in flight, one entry per lane (beyond 64: loaded when needed); the
  // row pointers are read one row ahead of the entries
  int eb0[kAheadG], eb1[kAheadG], ee[kAheadG], eo[kAheadG];
  double ef[kAheadG];
  int rp = rc, np0 = ptr[rp], np1 = ptr[rp + 1];
  const double *fum = ADJ ? a.fu + (size_t)mem * a.nuniq : nullptr;
  auto issue_e = [&](int k) {
    eb0[k] = np0;
    eb1[k] = np1;
    const int e = min(np0 + lane, max(np1 - 1, 0));  // (the lists hold at least one element)
    ee[k] = a.ent[e];
    if constexpr (ADJ) ef[k] = fum[e];
    else eo[k] = a.orig[e];
    rp = rp + 1 == N ? 0 : rp + 1;
    np0 = ptr[rp];
    np1 = ptr[rp + 1];
  };
#pragma unroll
  for (int k = 0; k < kAhead; ++k) {
    issue_f(k);
    if (k < kAW) issue_w(k);
    if (k < kAheadG) issue_e(k);
  }
  double na0 = ca0[rc], naW = caW[rc];
  d2 bsum = {0.0, 0.0}, bsum2 = {0.0, 0.0};

  for (int i0 = 0; i0 < iters; i0 += R) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = i0 + u;
      // (a copy, so that the next load into this slot needs no copy at the end of the loop,
      // which would wait for it)
      d2 cin = own_copy(fb[u % kAhead]);
      if (!has_in) cin = d2{0.0, 0.0};
      const d2 wrow = wb[u % kAW];
      const d2 ev = eb[u % kAW];
      d2 wrow2 = wrow, ev2 = ev, lam2 = {0.0, 0.0};
      if constexpr (TWO) wrow2 = wb2[u % kAW];
      if constexpr (TWO && !ADJ) ev2 = eb2[u % kAW];
      issue_f(u % kAhead);
      if constexpr (!ADJ) issue_w(u % kAW);
      r0[u] = na0;
      rW[u] = naW;
      const int beg = eb0[u % kAheadG], end = eb1[u % kAheadG];
      const int en = ee[u % kAheadG], eno = ADJ ? 0 : eo[u % kAheadG];
      const double enf = ADJ ? ef[u % kAheadG] : 0.0;
      issue_e(u % kAheadG);
      const int rn = rc + 1 == N ? 0 : rc + 1;
      na0 = ca0[rn];
      naW = caW[rn];
      // does the strip hold any of this iteration's cells?
      auto column = [&](int e) { return e & ((1 << kLevShift) - 1); };
      bool some = false;
      if (end > beg) {
        const int xe0 = column(en);
        const bool in = ADJ ? wrap(xe0 - (xs - kHalo), N) < kCells : xe0 >= xs && xe0 < xe;
        some = __any(in && beg + lane < end) || end - beg > 64;
      }
      if constexpr (!ADJ) {
        ring[u] = d2{tv.dt * wrow.x * ev.x, tv.dt * wrow.y * ev.y};
        if constexpr (TWO) ring2[u & 1] = d2{tv.dt * wrow2.x * ev2.x, tv.dt * wrow2.y * ev2.y};
      } else if (some) {
        // forcing of the levels' rows, scattered in LDS (a cell may sit at several places of
        // the strip when the strip is wider than the period)
#pragma unroll
        for (int s = 0; s < S; ++s) rows[s][2 * lane] = rows[s][2 * lane + 1] = 0.0;
        wave_lds_fence();
        auto scatter = [&](int e, double f) {
          for (int pos = wrap(column(e) - (xs - kHalo), N); pos < kCells; pos += N)
            rows[e >> kLevShift][pos] = f;
        };
        if (beg + lane < end) scatter(en, enf);
        for (int k = beg + 64 + lane; k < end; k += 64) scatter(a.ent[k], fum[k]);
        wave_lds_fence();
        cin += d2{rows[0][2 * lane], rows[0][2 * lane + 1]};
      }
#pragma unroll
      for (int s = 1; s <= S; ++s) {
        const int d = (u - (s - 1)) & (R - 1);  // ring slot of the row this level takes in
        const double xm = from_below(cin.y), xp = from_above(cin.x);
        const double cm = ADJ ? tv.aE : rW[d], cp = ADJ ? rW[d] : tv.aE;
        const double cym = ADJ ? tv.aN : tv.aS, cyp = ADJ ? tv.aS : tv.aN;
        d2 o;
        o.x = fma(cyp, cin.x, q[s - 1].x);
        o.y = fma(cyp, cin.y, q[s - 1].y);
        d2 t;
        t.x = fma(cm, xm, r0[d] * cin.x);
        t.y = fma(cm, cin.x, r0[d] * cin.y);
        t.x = fma(cym, cold[s - 1].x, t.x);
        t.y = fma(cym, cold[s - 1].y, t.y);
        t.x = fma(cp, cin.y, t.x);
        t.y = fma(cp, xp, t.y);
        if constexpr (ADJ) {
          if (TWO && s == 2)
            lam2 = cin;
          else
            ring[d] = s == 1 ? cin : d2{ring[d].x + cin.x, ring[d].y + cin.y};
        } else {
          const d2 em = TWO && s == 2 ? ring2[(u - 1) & 1] : ring[d];
          t.x += em.x;
          t.y += em.y;
        }
        q[s - 1] = t;
        cold[s - 1] = cin;
        cin = o;
        if constexpr (ADJ) {
          const int k = s < S ? s : 0;
          if (s < S && some) cin += d2{rows[k][2 * lane], rows[k][2 * lane + 1]};
        }
      }
      if constexpr (!ADJ) {
        if (some) {
#pragma unroll
          for (int s = 1; s <= S; ++s) {
            const d2 v = s < S ? cold[s < S ? s : 0] : cin;  // level s + 1 took it in
            rows[s - 1][2 * lane] = v.x;
            rows[s - 1][2 * lane + 1] = v.y;
          }
          wave_lds_fence();
          auto sample = [&](int e, int o) {
            const int lv = e >> kLevShift, xo = column(e), yu = ys - S + i - lv;
            if (yu >= ys && yu < ye && xo >= xs && xo < xe && a.obs)
              a.obs[(size_t)mem * a.nobs + o] = rows[lv - 1][xo - xs + kHalo];
          };
          if (beg + lane < end) sample(en, eno);
          for (int k = beg + 64 + lane; k < end; k += 64) sample(a.ent[k], a.orig[k]);
          wave_lds_fence();
        }
      }
      const int yo = ys - 2 * S + i;  // row of the last level
      if (a.out && yo >= ys && yo < ye && own)
        *row_at<d2>(a.out + mem * NN + (size_t)yo * N, xo8) = cin;
      if constexpr (ADJ) {
        const int yg = yo + 1;  // row whose sums of lam are complete
        issue_w(u % kAW);
        if (yg >= ys && yg < ye) {
          const int bm = (1 << sh) - 1;
          auto add = [&](double *gm, d2 old, d2 wr, d2 sl, d2 &bs) {
            const d2 w = {tv.dt * wr.x * sl.x, tv.dt * wr.y * sl.y};
            bs = (yg & bm) == 0 ? w : bs + w;
            if ((yg & bm) != bm) return;  // not the last row of its control blocks
            gmem<double> *g = row_at<double>(gm + (size_t)(yg >> sh) * tv.Nb, xb8);
            if (sh == 0) {
              if (own) {
                g[0] = old.x + bs.x;
                g[1] = old.y + bs.y;
              }
            } else {
              double t = bs.x + bs.y;
              if (sh == 2) t += dpp_shift<0xB1>(t);  // the other lane of the pair
              if (own && (sh < 2 || (lane & 1) == 0)) g[0] = old.x + t;
            }
          };
          // TWO: level 1 is the later step (its gradient needs no old value: one step per block)
          const d2 old = !TWO && a.gS_add ? ev : d2{0.0, 0.0};
          add(gSm, old, wrow, TWO ? lam2 : ring[(u - (S - 1)) & (R - 1)], bsum);
          if constexpr (TWO) add(gSm2, old, wrow2, ring[(u - 1) & (R - 1)], bsum2);
        }
      }
      rc = rn;
    }
  }
}

// Observation forcing gathered per unique cell: fu[mem nuniq + u] = sum of f over the
// observations of u (all steps at once, before an adjoint sweep).
__global__ void tracer_gather_kernel(int nuniq, const int *__restrict__ uptr,
                                     const int *__restrict__ orig, const double *__restrict__ f,
                                     int nobs, double *__restrict__ fu) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= nuniq) return;
  const int mem = blockIdx.y;
  double s = 0.0;
  for (int k = uptr[u]; k < uptr[u + 1]; ++k) s += f[(size_t)mem * nobs + orig[k]];
  fu[(size_t)mem * nuniq + u] = s;
}

// Elementwise helpers.
__global__ void exp_kernel(long long n, const double *__restrict__ a, double *__restrict__ b) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = exp(a[i]);
}

// W_tau[y, x] = E[y, x] exp(s_b[tau, y / block, x / block]) for every time block.
__global__ void base_emission_kernel(TracerView tv, const double *__restrict__ E,
                                     const double *__restrict__ sb, double *__restrict__ W) {
  const size_t NN = (size_t)tv.N * tv.N;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= NN * tv.ntb) return;
  const int tau = (int)(i / NN);
  const size_t c = i - (size_t)tau * NN;
  const int y = (int)(c / tv.N), x = (int)(c - (size_t)y * tv.N);
  W[i] = E[c] * exp(sb[(size_t)tau * tv.Nb * tv.Nb + (size_t)(y >> tv.bshift) * tv.Nb + (x >> tv.bshift)]);
}

// d = y - hx; f = rinv d (observation space, one column)
__global__ void innov_kernel(int nobs, const double *__restrict__ y, const double *__restrict__ hx,
                             const double *__restrict__ rinv, double *__restrict__ d,
                             double *__restrict__ f) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= nobs) return;
  const double dv = y[o] - hx[o];
  d[o] = dv;
  f[o] = rinv[o] * dv;
}

// out = v - a (v nullable); out = rinv * in row by row (scale_rows) for m columns
__global__ void axpy_rows_kernel(long long n, const double *__restrict__ v,
                                 const double *__restrict__ a, double *__restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (v ? v[i] : 0.0) - a[i];
}

__global__ void scale_rows_kernel(int nobs, int m, const double *__restrict__ rinv,
                                  const double *in, double *out) {  // in may alias out
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)nobs * m) return;
  out[i] = rinv[i % nobs] * in[i];
}

__global__ void cost_terms_kernel(int n, const double *__restrict__ v, int nobs,
                                  const double *__restrict__ d, const double *__restrict__ rinv,
                                  double *__restrict__ out) {
  __shared__ double red[1024];
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    if (v) a += v[i] * v[i];
  for (int o = threadIdx.x; o < nobs; o += blockDim.x) a += rinv[o] * d[o] * d[o];
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = 0.5 * red[0];
}

unsigned blocks_for(long long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace
}  // namespace riot

using riot::TracerView;

struct riot_tracer {
  riot_tracer_desc d{};
  hipStream_t st = nullptr;
  int Nb = 0, ncontrol = 0, nuniq = 0;
  TracerView tv{};
  // device regions
  double *a0 = nullptr, *aW = nullptr, *E = nullptr, *Wb = nullptr, *sb = nullptr,
         *expS = nullptr;
  double *y = nullptr, *rinv = nullptr, *L1 = nullptr;
  int *orig = nullptr, *uptr = nullptr;
  int *ent = nullptr, *forig = nullptr, *uent = nullptr;  // see MarchArgs
  int *optr = nullptr, *gptr = nullptr;  // [group][N + 1] entries of observations and unique cells
  double *F0 = nullptr, *F1 = nullptr;           // m_max fields each (ping-pong)
  double *CA = nullptr, *CB = nullptr, *CC = nullptr;  // m_max control blocks each
  double *OA = nullptr;                          // m_max observation columns
  double *FU = nullptr;                          // m_max forcing columns per unique cell
  double *hx = nullptr, *dvec = nullptr, *fvec = nullptr, *scal = nullptr;
  std::vector<int> gstep;  // first step of each group of steps, then nsteps
  bool has_base = false;
};

namespace {

size_t a256(size_t b) { return (b + 255) / 256 * 256; }

struct TCarve {
  char *base;
  size_t off = 0;
  explicit TCarve(void *b) : base(static_cast<char *>(b)) {}
  template <typename T>
  T *take(size_t n) {
    off = a256(off);
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += std::max<size_t>(n, 1) * sizeof(T);
    return p;
  }
};

bool tracer_desc_ok(const riot_tracer_desc *d) {
  if (!d || d->N < 4 || d->N % 64 || d->nsteps < 1 || d->nobs < 0 || d->m_max < 1) return false;
  if (!(d->block == 1 || d->block == 2 || d->block == 4) || d->N % d->block) return false;
  if (d->ntb < 1 || d->nsteps % d->ntb) return false;
  if (!(d->dt > 0) || d->u0 - std::fabs(d->u1) < 0 || d->v < 0 || d->K < 0) return false;
  const double cmax = d->dt * (d->u0 + std::fabs(d->u1) + d->v) + 4.0 * d->dt * d->K;
  if (cmax > 1.0) return false;  // the explicit upwind step needs a Courant number <= 1
  if (!d->E || !d->L1 || !(d->sigma > 0)) return false;
  if (d->nobs > 0 && (!d->obs_t || !d->obs_y || !d->obs_x || !d->y || !d->rinv)) return false;
  for (int o = 0; o < d->nobs; ++o)
    if (d->obs_t[o] < 1 || d->obs_t[o] > d->nsteps || d->obs_y[o] < 0 || d->obs_y[o] >= d->N ||
        d->obs_x[o] < 0 || d->obs_x[o] >= d->N)
      return false;
  return true;
}

// The launches of a sweep: each time block's steps in equal groups of at most kMaxS (a group
// does not cross a time block: one emission field per launch), time blocks of one step in pairs.
int block_groups(const riot_tracer_desc &d) {  // launches per time block (pair)
  return (d.nsteps / d.ntb - 1) / riot::kMaxS + 1;
}
size_t step_group_count(const riot_tracer_desc &d) {
  return d.nsteps == d.ntb ? (size_t)(d.ntb / 2) + d.ntb % 2 : (size_t)d.ntb * block_groups(d);
}
// First steps, then nsteps.
std::vector<int> step_groups(const riot_tracer_desc &d) {
  std::vector<int> g;
  g.reserve(step_group_count(d) + 1);
  const int spb = d.nsteps / d.ntb, ng = block_groups(d);
  for (long long b = 0; b < d.ntb; b += spb == 1 ? 2 : 1)
    for (int k = 0; k < ng; ++k) g.push_back((int)(b * spb + (long long)spb * k / ng));
  g.push_back(d.nsteps);
  return g;
}

size_t tracer_carve(riot_tracer &h, void *base) {
  TCarve c(base);
  const riot_tracer_desc &d = h.d;
  const size_t NN = (size_t)d.N * d.N, m = d.m_max;
  const int Nb = d.N / d.block;
  const size_t nc = (size_t)d.ntb * Nb * Nb;
  h.a0 = c.take<double>(d.N);
  h.aW = c.take<double>(d.N);
  h.E = c.take<double>(NN);
  h.Wb = c.take<double>(NN * d.ntb);
  h.sb = c.take<double>(nc);
  h.expS = c.take<double>(nc);
  h.y = c.take<double>(d.nobs);
  h.rinv = c.take<double>(d.nobs);
  h.L1 = c.take<double>((size_t)Nb * Nb);
  h.orig = c.take<int>(d.nobs);
  h.uptr = c.take<int>(d.nobs + 1);
  h.ent = c.take<int>(d.nobs);
  h.forig = c.take<int>(d.nobs);
  h.uent = c.take<int>(d.nobs);
  h.optr = c.take<int>((step_group_count(d) + 1) * (d.N + 1));
  h.gptr = c.take<int>((step_group_count(d) + 1) * (d.N + 1));
  h.F0 = c.take<double>(NN * m);
  h.F1 = c.take<double>(NN * m);
  h.CA = c.take<double>(nc * m);
  h.CB = c.take<double>(nc * m);
  h.CC = c.take<double>(nc * m);
  h.OA = c.take<double>((size_t)std::max(d.nobs, 1) * m);
  h.FU = c.take<double>((size_t)std::max(d.nobs, 1) * m);
  h.hx = c.take<double>(d.nobs);
  h.dvec = c.take<double>(d.nobs);
  h.fvec = c.take<double>(d.nobs);
  h.scal = c.take<double>(16);
  return a256(c.off) + 256;
}

#define TR_HIP(call)                            \
  do {                                          \
    if ((call) != hipSuccess) return RIOT_E_HIP; \
  } while (0)

// Strips and chunks of a sweep over m members. Strips: as few as hold the width with the
// halo. Chunks: a wave's march costs 2 S rows on top of its own, so a chunk is as tall as
// leaves kWaves waves in the launch (two per SIMD, twice over so that the last ones even
// out: 512 members at 512 x 512 take 16.8 ms per product with 4096, 19.2 with 2048, 16.9
// with 8192), and at least kMinRows rows (value and gradient of one member at 512 x 512:
// 16 rows 15 % slower than 8; 4 rows gain 2 % there and lose 25 % at 64 x 64). The two rows of halo
// a side of a launch of two steps cost less: 4 rows where 8 leave a SIMD without a wave (64 x 64, 48
// blocks of one step, one member: product 404 -> 324 us; 64 members of 256 x 256 would lose 10 %).
constexpr long long kWaves = 4096;
constexpr int kMinRows = 8;

void march_geometry(const riot_tracer *h, int m, riot::MarchArgs &a) {
  const int N = h->d.N, use = riot::kCells - 2 * riot::kHalo;
  a.m = m;
  a.ns = (N + use - 1) / use;
  a.width = ((N + a.ns - 1) / a.ns + 3) / 4 * 4;
  const long long per = (long long)m * a.ns;  // waves per chunk row
  const bool few = h->tv.spb == 1 && per * (N / kMinRows) <= 1024;
  const int lo = few ? kMinRows / 2 : kMinRows;
  const int want = (int)std::min<long long>((kWaves + per - 1) / per, N / lo);
  a.rows = ((N + want - 1) / want + lo - 1) / lo * lo;
  a.nch = (N + a.rows - 1) / a.rows;
}

template <bool ADJ>
riot_status launch_march(const riot_tracer *h, int S, const riot::MarchArgs &a) {
  const dim3 grid((unsigned)((long long)a.m * a.nch * a.ns));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64), 0, h->st, h->tv, a, h->tv.a0, h->tv.aW, a.ptr);
  };
  if (S == 2 && h->tv.spb == 1) {  // two time blocks
    go(riot::tracer_march_kernel<ADJ, 2, true>);
    TR_HIP(hipGetLastError());
    return RIOT_OK;
  }
  switch (S) {
    case 1: go(riot::tracer_march_kernel<ADJ, 1>); break;
    case 2: go(riot::tracer_march_kernel<ADJ, 2>); break;
    case 3: go(riot::tracer_march_kernel<ADJ, 3>); break;
    case 4: go(riot::tracer_march_kernel<ADJ, 4>); break;
    case 5: go(riot::tracer_march_kernel<ADJ, 5>); break;
    case 6: go(riot::tracer_march_kernel<ADJ, 6>); break;
    case 7: go(riot::tracer_march_kernel<ADJ, 7>); break;
    default: go(riot::tracer_march_kernel<ADJ, 8>); break;
  }
  TR_HIP(hipGetLastError());
  return RIOT_OK;
}

// One sweep of the forward or tangent model over all members: fields start at zero,
// step t uses control block tau(t); observation samples into obs [nobs x m].
riot_status tracer_forward_sweep(riot_tracer *h, int m, const double *Wfield, long long Wstride,
                                 const double *bv, long long bv_stride, double *obs) {
  const riot_tracer_desc &d = h->d;
  const int Nbb = h->Nb * h->Nb, ng = (int)h->gstep.size() - 1;
  riot::MarchArgs a{};
  march_geometry(h, m, a);
  a.bv_stride = bv_stride;
  a.ent = h->ent, a.orig = h->forig, a.nobs = d.nobs;
  a.obs = d.nobs > 0 ? obs : nullptr;
  double *bufs[2] = {h->F0, h->F1};
  for (int g = 0; g < ng; ++g) {
    const int t = h->gstep[g], tau = t / h->tv.spb;
    a.in = g ? bufs[(g - 1) & 1] : nullptr;
    a.out = g + 1 < ng ? bufs[g & 1] : nullptr;
    a.W = Wfield + Wstride * tau;
    a.bv = bv + (size_t)tau * Nbb;
    a.W2 = a.W + Wstride, a.bv2 = a.bv + Nbb;
    a.ptr = h->optr + (size_t)g * (d.N + 1);
    riot_status rs = launch_march<false>(h, h->gstep[g + 1] - t, a);
    if (rs != RIOT_OK) return rs;
  }
  return RIOT_OK;
}

// Adjoint sweep: gS [ncontrol x m] = G^T f for observation-space f [nobs x m].
riot_status tracer_adjoint_sweep(riot_tracer *h, int m, const double *f, double *gS) {
  const riot_tracer_desc &d = h->d;
  const size_t NN = (size_t)d.N * d.N;
  const int Nbb = h->Nb * h->Nb, ng = (int)h->gstep.size() - 1;
  if (h->nuniq > 0) {
    hipLaunchKernelGGL(riot::tracer_gather_kernel, dim3(riot::blocks_for(h->nuniq), m), dim3(256),
                       0, h->st, h->nuniq, h->uptr, h->orig, f, d.nobs, h->FU);
    TR_HIP(hipGetLastError());
  }
  riot::MarchArgs a{};
  march_geometry(h, m, a);
  a.gS_stride = h->ncontrol;
  a.ent = h->uent, a.fu = h->FU, a.nuniq = h->nuniq;
  double *bufs[2] = {h->F0, h->F1};
  for (int g = ng - 1, k = 0; g >= 0; --g, ++k) {  // states gstep[g + 1] -> gstep[g]
    const int t = h->gstep[g], tau = t / h->tv.spb;
    a.in = k ? bufs[(k - 1) & 1] : nullptr;
    a.out = g ? bufs[k & 1] : nullptr;
    a.W = h->Wb + NN * tau;
    a.gS = gS + (size_t)tau * Nbb;
    a.W2 = a.W + NN, a.gS2 = a.gS + Nbb;
    a.gS_add = g + 1 < ng && h->gstep[g + 1] / h->tv.spb == tau;  // not the block's first launch
    a.ptr = h->gptr + (size_t)g * (d.N + 1);
    riot_status rs = launch_march<true>(h, h->gstep[g + 1] - t, a);
    if (rs != RIOT_OK) return rs;
  }
  return RIOT_OK;
}

// S = L Z = sigma (L1 kron L1) Z per time-block image: with an image Z stored [by][bx]
// read as the column-major matrix M = Z^T, L1 Z L1 corresponds to L1 M L1 (L1 symmetric).
riot_status tracer_apply_L(riot_tracer *h, int m, const double *Z, double *S, double *tmp) {
  const int Nb = h->Nb;
  const long long img = (long long)Nb * Nb;
  const int nimg = m * h->d.ntb;
  TR_HIP(riot::gemm_f64_strided(0, 0, Nb, Nb, Nb, 1.0, Z, Nb, img, h->L1, Nb, 0, 0.0, tmp, Nb, img,
                                nimg, h->st));
  TR_HIP(riot::gemm_f64_strided(0, 0, Nb, Nb, Nb, h->d.sigma, h->L1, Nb, 0, tmp, Nb, img, 0.0, S,
                                Nb, img, nimg, h->st));
  return RIOT_OK;
}

}  // namespace

extern "C" {

size_t riot_tracer_workspace_bytes(const riot_tracer_desc *desc) {
  if (!tracer_desc_ok(desc)) return 0;
  riot_tracer h;
  h.d = *desc;
  return tracer_carve(h, nullptr);
}

riot_status riot_tracer_init(const riot_tracer_desc *desc, void *workspace, size_t bytes,
                             void *hip_stream, riot_tracer **out) {
  if (!out) return RIOT_E_ARG;
  *out = nullptr;
  if (!tracer_desc_ok(desc) || !workspace) return RIOT_E_ARG;
  if (reinterpret_cast<uintptr_t>(workspace) % 256) return RIOT_E_WORKSPACE;
  if (bytes < riot_tracer_workspace_bytes(desc)) return RIOT_E_WORKSPACE;
  riot_tracer *h = new (std::nothrow) riot_tracer();
  if (!h) return RIOT_E_ARG;
  h->d = *desc;
  h->st = static_cast<hipStream_t>(hip_stream);
  tracer_carve(*h, workspace);
  const riot_tracer_desc &d = h->d;
  h->Nb = d.N / d.block;
  h->ncontrol = d.ntb * h->Nb * h->Nb;
  // stencil coefficients of the upwind / diffusion step
  std::vector<double> a0(d.N), aW(d.N);
  for (int yy = 0; yy < d.N; ++yy) {
    const double u = d.u0 + d.u1 * std::sin(2.0 * 3.14159265358979323846 * yy / d.N);
    a0[yy] = 1.0 - d.dt * (u + d.v) - 4.0 * d.dt * d.K;
    aW[yy] = d.dt * (u + d.K);
  }
  TracerView &tv = h->tv;
  tv.N = d.N, tv.T = d.nsteps, tv.block = d.block, tv.ntb = d.ntb, tv.Nb = h->Nb;
  tv.bshift = d.block == 4 ? 2 : (d.block == 2 ? 1 : 0);
  tv.spb = d.nsteps / d.ntb;
  tv.dt = d.dt, tv.aS = d.dt * (d.v + d.K), tv.aE = d.dt * d.K, tv.aN = d.dt * d.K;
  tv.a0 = h->a0, tv.aW = h->aW;
  // Observations in the order of the march: by group of steps, by the row taken in when their
  // level finishes theirs, by level and column. Forward: state t + lev of the group's first
  // state t, lev = 1 .. S; adjoint: state t + S - lev, lev = 0 .. S - 1. Both put an
  // observation of state t + k in the same group for 1 <= k <= S.
  h->gstep = step_groups(d);
  const int ng = (int)h->gstep.size() - 1;
  struct Entry {
    int g, r, lev, cell, o;
  };
  std::vector<Entry> fe(d.nobs), ae(d.nobs);
  for (int o = 0; o < d.nobs; ++o) {
    const int g = (int)(std::lower_bound(h->gstep.begin(), h->gstep.end(), d.obs_t[o]) -
                        h->gstep.begin()) - 1;
    const int c = d.obs_y[o] * d.N + d.obs_x[o];
    const int lf = d.obs_t[o] - h->gstep[g], la = h->gstep[g + 1] - d.obs_t[o];
    fe[o] = {g, (d.obs_y[o] + lf) % d.N, lf, c, o};
    ae[o] = {g, (d.obs_y[o] + la) % d.N, la, c, o};
  }
  auto before = [](const Entry &a, const Entry &b) {
    if (a.g != b.g) return a.g < b.g;
    if (a.r != b.r) return a.r < b.r;
    if (a.lev != b.lev) return a.lev < b.lev;
    return a.cell != b.cell ? a.cell < b.cell : a.o < b.o;
  };
  std::sort(fe.begin(), fe.end(), before);
  std::sort(ae.begin(), ae.end(), before);
  const size_t n1 = (size_t)d.N + 1;
  std::vector<int> ent(d.nobs), forig(d.nobs), ord(d.nobs), uent, uptr{0};
  auto pack = [&](const Entry &e) { return e.cell % d.N + (e.lev << riot::kLevShift); };
  std::vector<int> optr((ng + 1) * n1, 0), gptr((ng + 1) * n1, 0);
  for (int k = 0; k < d.nobs; ++k) {
    ent[k] = pack(fe[k]);
    forig[k] = fe[k].o;
    optr[fe[k].g * n1 + fe[k].r + 1]++;
    ord[k] = ae[k].o;
    if (k == 0 || before({ae[k - 1].g, ae[k - 1].r, ae[k - 1].lev, ae[k - 1].cell, 0},
                         {ae[k].g, ae[k].r, ae[k].lev, ae[k].cell, 0})) {
      uent.push_back(pack(ae[k]));
      uptr.push_back(uptr.back());
      gptr[ae[k].g * n1 + ae[k].r + 1]++;
    }
    uptr.back()++;
  }
  for (size_t k = 1; k < optr.size(); ++k) optr[k] += optr[k - 1], gptr[k] += gptr[k - 1];
  h->nuniq = (int)uent.size();
  riot_status rs = RIOT_OK;
  auto cp = [&](void *dst, const void *src, size_t b) {
    if (b && hipMemcpyAsync(dst, src, b, hipMemcpyHostToDevice, h->st) != hipSuccess)
      rs = RIOT_E_HIP;
  };
  const size_t NN = (size_t)d.N * d.N;
  cp(h->a0, a0.data(), d.N * sizeof(double));
  cp(h->aW, aW.data(), d.N * sizeof(double));
  cp(h->E, d.E, NN * sizeof(double));
  cp(h->L1, d.L1, (size_t)h->Nb * h->Nb * sizeof(double));
  cp(h->orig, ord.data(), ord.size() * sizeof(int));
  cp(h->uptr, uptr.data(), uptr.size() * sizeof(int));
  cp(h->ent, ent.data(), ent.size() * sizeof(int));
  cp(h->forig, forig.data(), forig.size() * sizeof(int));
  cp(h->uent, uent.data(), uent.size() * sizeof(int));
  cp(h->optr, optr.data(), optr.size() * sizeof(int));
  cp(h->gptr, gptr.data(), gptr.size() * sizeof(int));
  cp(h->y, d.y, (size_t)d.nobs * sizeof(double));
  cp(h->rinv, d.rinv, (size_t)d.nobs * sizeof(double));
  if (hipStreamSynchronize(h->st) != hipSuccess) rs = RIOT_E_HIP;
  h->d.E = nullptr, h->d.L1 = nullptr, h->d.obs_t = nullptr, h->d.obs_y = nullptr;
  h->d.obs_x = nullptr, h->d.y = nullptr, h->d.rinv = nullptr;
  if (rs != RIOT_OK) {
    delete h;
    return rs;
  }
  *out = h;
  return RIOT_OK;
}

void riot_tracer_free(riot_tracer *h) { delete h; }

riot_status riot_tracer_forward(riot_tracer *h, const double *s, double *obs) {
  if (!h || !s || (h->d.nobs > 0 && !obs)) return RIOT_E_ARG;
  const riot_tracer_desc &d = h->d;
  hipStream_t st = h->st;
  // base state for the derivatives: s_b = s, W_tau = E exp(up(s_tau))
  TR_HIP(hipMemcpyAsync(h->sb, s, (size_t)h->ncontrol * sizeof(double), hipMemcpyDeviceToDevice,
                        st));
  const size_t NN = (size_t)d.N * d.N;
  hipLaunchKernelGGL(riot::base_emission_kernel, dim3(riot::blocks_for((long long)NN * d.ntb)),
                     dim3(256), 0, st, h->tv, h->E, h->sb, h->Wb);
  TR_HIP(hipGetLastError());
  hipLaunchKernelGGL(riot::exp_kernel, dim3(riot::blocks_for(h->ncontrol)), dim3(256), 0, st,
                     (long long)h->ncontrol, s, h->expS);
  TR_HIP(hipGetLastError());
  h->has_base = true;
  return tracer_forward_sweep(h, 1, h->E, 0, h->expS, h->ncontrol, obs);
}

riot_status riot_tracer_tangent(riot_tracer *h, int32_t m, const double *dS, double *dObs) {
  if (!h || !dS || m < 1 || m > h->d.m_max || (h->d.nobs > 0 && !dObs)) return RIOT_E_ARG;
  if (!h->has_base) return RIOT_E_STATE;
  return tracer_forward_sweep(h, m, h->Wb, (long long)h->d.N * h->d.N, dS, h->ncontrol, dObs);
}

riot_status riot_tracer_adjoint(riot_tracer *h, int32_t m, const double *gObs, double *gS) {
  if (!h || !gS || m < 1 || m > h->d.m_max || (h->d.nobs > 0 && !gObs)) return RIOT_E_ARG;
  if (!h->has_base) return RIOT_E_STATE;
  return tracer_adjoint_sweep(h, m, gObs, gS);
}

riot_status riot_tracer_apply_L(riot_tracer *h, int32_t m, const double *Z, double *S) {
  if (!h || !Z || !S || Z == S || m < 1 || m > h->d.m_max) return RIOT_E_ARG;
  return tracer_apply_L(h, m, Z, S, h->CC);
}

riot_status riot_tracer_hess_apply(riot_tracer *h, int32_t m, const double *W, double *Y) {
  if (!h || !W || !Y || W == Y || m < 1 || m > h->d.m_max) return RIOT_E_ARG;
  if (!h->has_base) return RIOT_E_STATE;
  const riot_tracer_desc &d = h->d;
  riot_status rs;
  if ((rs = tracer_apply_L(h, m, W, h->CA, h->CC)) != RIOT_OK) return rs;
  if ((rs = tracer_forward_sweep(h, m, h->Wb, (long long)d.N * d.N, h->CA, h->ncontrol, h->OA)) !=
      RIOT_OK)
    return rs;
  if (d.nobs > 0) {
    hipLaunchKernelGGL(riot::scale_rows_kernel, dim3(riot::blocks_for((long long)d.nobs * m)),
                       dim3(256), 0, h->st, d.nobs, m, h->rinv, h->OA, h->OA);
    TR_HIP(hipGetLastError());
  }
  if ((rs = tracer_adjoint_sweep(h, m, h->OA, h->CB)) != RIOT_OK) return rs;
  return tracer_apply_L(h, m, h->CB, Y, h->CC);
}

riot_status riot_tracer_gradient(riot_tracer *h, const double *v, double *grad, double *d_out,
                                 double *J_host) {
  if (!h || !grad) return RIOT_E_ARG;
  if (!h->has_base) return RIOT_E_STATE;
  const riot_tracer_desc &d = h->d;
  hipStream_t st = h->st;
  riot_status rs;
  // d = y - H(M(s_b)) from a fresh forward sweep at the base, f = R^{-1} d
  if ((rs = tracer_forward_sweep(h, 1, h->E, 0, h->expS, h->ncontrol, h->hx)) != RIOT_OK) return rs;
  if (d.nobs > 0) {
    hipLaunchKernelGGL(riot::innov_kernel, dim3(riot::blocks_for(d.nobs)), dim3(256), 0, st,
                       d.nobs, h->y, h->hx, h->rinv, h->dvec, h->fvec);
    TR_HIP(hipGetLastError());
    if (d_out)
      TR_HIP(hipMemcpyAsync(d_out, h->dvec, (size_t)d.nobs * sizeof(double),
                            hipMemcpyDeviceToDevice, st));
  }
  if ((rs = tracer_adjoint_sweep(h, 1, h->fvec, h->CB)) != RIOT_OK) return rs;
  if ((rs = tracer_apply_L(h, 1, h->CB, h->CA, h->CC)) != RIOT_OK) return rs;
  hipLaunchKernelGGL(riot::axpy_rows_kernel, dim3(riot::blocks_for(h->ncontrol)), dim3(256), 0, st,
                     (long long)h->ncontrol, v, h->CA, grad);
  TR_HIP(hipGetLastError());
  if (J_host) {
    hipLaunchKernelGGL(riot::cost_terms_kernel, dim3(1), dim3(1024), 0, st, h->ncontrol, v, d.nobs,
                       h->dvec, h->rinv, h->scal);
    TR_HIP(hipGetLastError());
    TR_HIP(hipMemcpyAsync(J_host, h->scal, sizeof(double), hipMemcpyDeviceToHost, st));
    TR_HIP(hipStreamSynchronize(st));
  }
  return RIOT_OK;
}

}  // extern "C"
