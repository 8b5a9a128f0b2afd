// Learned sketch proposal: a 1-D periodic convolutional network (FP32) that maps a
// background state to k probe vectors, its backward pass, Adam, and the subspace-capture
// loss of the leading Hessian eigenvectors with its gradient (FP64 on the MFMA GEMMs).
//
// Network: input = the standardized state (one channel); L layers of periodic conv1d of
// odd width 2r+1, ReLU after all but the last; output channel c is probe vector c.
// Layout: activations [sample][channel][grid point]; parameters flat, per layer the
// weights [cout][cin][width] then the biases [cout].

#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "riot_internal.h"

namespace riot {
namespace {

constexpr int kMaxWidth = 11;
typedef float f4 __attribute__((ext_vector_type(4)));

// Sum over a workgroup of 256 threads as a binary tree (thread t adds t + 128, t + 64, ...).
__device__ __forceinline__ double tree_sum(double v, double *red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  if (t < 128) red[t] += red[t + 128];
  __syncthreads();
  double s = 0.0;
  if (t < 64) {
    s = red[t] + red[t + 64];
    for (int k = 32; k > 0; k >>= 1) s += __shfl_down(s, k, 64);
    if (t == 0) red[0] = s;
  }
  __syncthreads();
  s = red[0];
  __syncthreads();
  return s;
}

// Per-row standardization (x - mean) / std of FP64 input rows (one workgroup per sample and
// input channel) into FP32.
__global__ void __launch_bounds__(256)
    standardize_kernel(int n, const double *__restrict__ x, float *__restrict__ out) {
  __shared__ double red[256];
  const double *xs = x + (size_t)blockIdx.x * n;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += xs[i];
  const double mean = tree_sum(s, red) / n;
  double q = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) q += (xs[i] - mean) * (xs[i] - mean);
  const double inv = 1.0 / sqrt(tree_sum(q, red) / n);
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    out[(size_t)blockIdx.x * n + i] = (float)((xs[i] - mean) * inv);
}

// Weights in operand order. The contraction index of a convolution is k = c' W + j; step k / 4
// takes lanes l / 16 = k % 4; groups of four steps are stored lane by lane, so element k of
// output channel c is float (step % 4) of lane 16 (k % 4) + c % 16 of group step / 4 of the 16
// channels c / 16. Zeros fill up to whole groups and 16 channels. fwd: the layer's own weights;
// bwd: those of its backward-data pass (none for the first layer).
struct Frag {
  int layers, width;
  int cin[16], cout[16];
  long long woff[16], fwd[16], bwd[16];  // offsets of the layer's weights in the three arrays
};
__host__ __device__ __forceinline__ int frag_groups(int cin, int width) {
  return ((cin + 3) / 4 * width + 3) / 4;
}
__host__ __device__ __forceinline__ long long frag_floats(int cin, int cout, int width) {
  return (long long)((cout + 15) / 16) * frag_groups(cin, width) * 256;
}
__device__ __forceinline__ long long frag_at(int cin, int width, int c, int k) {
  const int step = k / 4;
  return (((long long)(c / 16) * frag_groups(cin, width) + step / 4) * 64 + 16 * (k % 4) + c % 16) *
             4 + step % 4;
}
// parameter i (of the flat parameters) is v
__device__ __forceinline__ void frag_put(const Frag &f, long long i, float v,
                                         float *__restrict__ frag) {
  int l = f.layers - 1;
  while (l > 0 && i < f.woff[l]) --l;
  const int e = (int)(i - f.woff[l]), cin = f.cin[l], cout = f.cout[l], W = f.width;
  if (e >= cout * cin * W) return;  // a bias
  const int co = e / (cin * W), k = e - co * cin * W, ci = k / W, j = k - ci * W;
  frag[f.fwd[l] + frag_at(cin, W, co, k)] = v;
  if (l > 0) frag[f.bwd[l] + frag_at(cout, W, ci, co * W + W - 1 - j)] = v;
}

// New parameters: the flat copy and the operand order in one launch (6 us; a copy and a
// launch after it 7.8, the copy alone 4.7).
__global__ void set_params_kernel(long long count, Frag f, const float *__restrict__ in,
                                  float *__restrict__ p, float *__restrict__ frag) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float v = in[i];
  p[i] = v;
  frag_put(f, i, v, frag);
}

// z[c, i] = b[c] + sum_{c', j} W[c, c', j] h[c', (i + j - r) mod n], ReLU when relu != 0, on
// the FP32 matrix cores: the contraction over (c', j) in that order, four values per
// v_mfma_f32_16x16x4_f32, which adds its four products one after the other, each with one
// rounding, so that an output value is the same chain of fused multiply-adds as before.
// Operand lanes: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; result register r of
// lane l is C[4 (l / 16) + r][l % 16].
// A workgroup takes all output channels, wave by wave 16 of them, and 16 NT grid points per wave
// (waves that have no channels of their own take the next points: cgs waves along the
// channels); the input rows (all cin, with the halo) are staged in LDS once. The weights come
// in the order of the operands (Frag), 16 bytes per lane for four matrix instructions, 16 input
// channels ahead.
// FLIP: the backward-data pass, weights W[c'][c][W - 1 - j] of a forward layer cin <- cout, and
// the result zeroed where act <= 0 (the ReLU derivative of the layer below).
// n = 2048, 64 -> 64 channels, width 9: 16 samples (2.4 GFLOP) 31 us (16 us at the rate of a
// large FP32 product), one sample 12 us, bound by staging and the chain of 144 matrix
// instructions. One fused multiply-add per lane and LDS value took 91 and 23 us; weights in
// parameter order, 16 rows of 16 bytes per load, 55 and 23 us.
template <int W, int NT, bool FLIP>
__global__ void __launch_bounds__(256)
    conv_kernel(int n, int cin, int cout, int cgs, const float *__restrict__ h,
                const float *__restrict__ wf, const float *__restrict__ b,
                const float *__restrict__ act, float *__restrict__ z, int relu) {
  extern __shared__ float Xs[];  // [cin rounded up to 4][span]
  constexpr int r = W / 2;
  const int XT = 16 * NT * (4 / cgs), span = XT + W - 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int x0 = blockIdx.x * XT, s = blockIdx.y;
  const int c0 = 16 * (wave % cgs), xw = 16 * NT * (wave / cgs);
  const int cin4 = (cin + 3) / 4 * 4, groups = frag_groups(cin, W);
  // (a wave without channels of its own repeats the last ones')
  const f4 *wl = reinterpret_cast<const f4 *>(wf) +
                 (size_t)min(c0 / 16, (cout - 1) / 16) * groups * 64 + lane;
  f4 a[W], an[W];
  auto load_a = [&](int cb, f4 (&av)[W]) {  // W groups: 16 input channels from cb
#pragma unroll
    for (int q = 0; q < W; ++q) av[q] = wl[(size_t)min(cb / 16 * W + q, groups - 1) * 64];
  };
  load_a(0, a);
  const float *hs = h + (size_t)s * cin * n;
  for (int cb = wave; cb < cin4; cb += 16) {  // four rows of this wave at a time
    float v[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int ci = cb + 4 * q, xx = lane + 64 * p;
        int g = x0 + xx - r;
        g = g < 0 ? g + n : (g >= n ? g - n : g);
        v[q][p] = (ci < cin && xx < span) ? hs[(size_t)ci * n + g] : 0.f;
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int ci = cb + 4 * q, xx = lane + 64 * p;
        if (ci < cin4 && xx < span) Xs[ci * span + xx] = v[q][p];
      }
  }
  f4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = c0 + 4 * lg + q;
      acc[t][q] = (!FLIP && c < cout) ? b[c] : 0.f;
    }
  int off[W];
#pragma unroll
  for (int q = 0; q < W; ++q) off[q] = (4 * q + lg) / W * span + (4 * q + lg) % W + xw + li;
  __syncthreads();
  for (int cb = 0; cb < cin4; cb += 16) {
    load_a(cb + 16, an);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (cb + 4 * u >= cin4) break;
      const float *xr = Xs + (cb + 4 * u) * span;
#pragma unroll
      for (int q = 0; q < W; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(u * W + q) / 4][(u * W + q) % 4],
                                                        xr[off[q] + 16 * t], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < W; ++q) a[q] = an[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = c0 + 4 * lg + q;
    if (c >= cout) continue;
    const size_t o = ((size_t)s * cout + c) * n + x0 + xw + li;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float v = acc[t][q];
      if (FLIP)
        v = act[o + 16 * t] > 0.f ? v : 0.f;
      else if (relu)
        v = fmaxf(v, 0.f);
      z[o + 16 * t] = v;
    }
  }
}

// Localized output head: N[s][c S + q][i] = z[s][c][i] for grid points i of segment q
// (n / S consecutive points), 0 elsewhere; z has k / S channels. To FP32 (N) and / or, with
// columns ld64 apart, FP64 (N64).
__global__ void segment_out_kernel(int n, int kch, int S, long long total,
                                   const float *__restrict__ z, float *__restrict__ N,
                                   double *__restrict__ N64, int ld64) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int k = kch * S;
  const long long gcol = e / n;
  const int i = (int)(e - gcol * n);
  const long long s = gcol / k;
  const int col = (int)(gcol - s * k), c = col / S, q = col - c * S;
  const float v = (i / (n / S) == q) ? z[(s * kch + c) * n + i] : 0.f;
  if (N) N[e] = v;
  if (N64) N64[gcol * ld64 + i] = (double)v;
}

// Its transpose: gz[s][c][i] = gN[s][c S + (segment of i)][i].
__global__ void segment_grad_kernel(int n, int kch, int S, long long total,
                                    const float *__restrict__ gN, float *__restrict__ gz) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int i = (int)(e % n), c = (int)((e / n) % kch);
  const long long s = e / ((long long)n * kch);
  const int q = i / (n / S);
  gz[e] = gN[(s * kch * S + (long long)c * S + q) * n + i];
}

// Weight gradient gW[co][ci][j] = sum_s sum_i g[s][co][i] h[s][ci][(i + j - r) mod n] and bias
// gradient gb[co] = sum_s sum_i g[s][co][i], in two passes with a fixed summation order. Pass 1,
// on the FP32 matrix cores: a workgroup takes the chunks of kCP grid points [z per, z per + per)
// of all samples, 16 WC output and 16 WI input channels, a wave 16 x 16 of them with all W taps:
// four points of g are one operand of W products with h shifted by j, and the bias gradient is
// the product with ones. The chunk's rows of g and h (with the halo) are staged in LDS, the next
// chunk's in registers meanwhile. FP32 sums run over fl chunks (256, 128 or 64 points of one
// sample, as they divide n; fl divides per) and then go to FP64. Pass 2 adds the workgroups'
// sums in FP64.
// n = 2048, 64 x 64 channels, width 9, 16 samples (2.4 GFLOP): 43 us and 5 us; one fused
// multiply-add per lane and register window took 37 us, and the second pass, one chain of 128
// partial sums per weight, 28 us.
constexpr int kCP = 64;

template <int W, int WC, int WI>
__global__ void __launch_bounds__(256)
    conv_wgrad_kernel(int n, int cin, int cout, int chunks, int per, int fl, const float *__restrict__ g,
                      const float *__restrict__ h, double *__restrict__ part) {
  constexpr int r = W / 2, span = kCP + W - 1;
  // row strides of 4 mod 8 words: the 16 rows x 4 points of an operand fall into distinct banks
  constexpr int ldg = kCP + 4, ldh = (span + 3) / 8 * 8 + 4;
  __shared__ float Gs[16 * WC * ldg], Hs[16 * WI * ldh];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int ci0 = blockIdx.y * 16 * WI, co0 = blockIdx.z * 16 * WC;
  const int wc = wave % WC, wi = wave / WC;
  const int cps = n / kCP, cbeg = blockIdx.x * per, cend = min(cbeg + per, chunks);
  float vg[4 * WC], vh[4 * WI][2];
  auto fetch = [&](int c) {
    const int s = c / cps, i0 = (c - s * cps) * kCP;
#pragma unroll
    for (int q = 0; q < 4 * WC; ++q) {
      const int co = co0 + wave + 4 * q;
      const float v = g[((size_t)s * cout + min(co, cout - 1)) * n + i0 + lane];
      vg[q] = co < cout ? v : 0.f;
    }
    int p0 = i0 + lane - r, p1 = i0 + 64 + lane - r;
    p0 = p0 < 0 ? p0 + n : p0;
    p1 = p1 >= n ? p1 - n : p1;
#pragma unroll
    for (int q = 0; q < 4 * WI; ++q) {
      const int ci = ci0 + wave + 4 * q;
      const float *hr = h + ((size_t)s * cin + min(ci, cin - 1)) * n;
      const float a = hr[p0], b = lane < W - 1 ? hr[p1] : 0.f;
      vh[q][0] = ci < cin ? a : 0.f;
      vh[q][1] = ci < cin ? b : 0.f;
    }
  };
  const bool bias = blockIdx.y == 0 && wi == 0;
  f4 acc[W + 1];
  double sum[W + 1][4];
#pragma unroll
  for (int j = 0; j <= W; ++j) {
    acc[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[j][q] = 0.0;
  }
  auto flush = [&]() {
#pragma unroll
    for (int j = 0; j <= W; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[j][q] += (double)acc[j][q];
      acc[j] = f4{0.f, 0.f, 0.f, 0.f};
    }
  };
  if (cbeg < cend) fetch(cbeg);
  for (int c = cbeg; c < cend; ++c) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4 * WC; ++q) Gs[(wave + 4 * q) * ldg + lane] = vg[q];
#pragma unroll
    for (int q = 0; q < 4 * WI; ++q) {
      Hs[(wave + 4 * q) * ldh + lane] = vh[q][0];
      if (lane < W - 1) Hs[(wave + 4 * q) * ldh + 64 + lane] = vh[q][1];
    }
    __syncthreads();
    if (c + 1 < cend) fetch(c + 1);
    const float *gr = Gs + (16 * wc + li) * ldg + lg, *hr = Hs + (16 * wi + li) * ldh + lg;
#pragma unroll 4
    for (int p = 0; p < kCP; p += 4) {
      const float av = gr[p];
#pragma unroll
      for (int j = 0; j < W; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, hr[p + j], acc[j], 0, 0, 0);
      if (bias) acc[W] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, 1.f, acc[W], 0, 0, 0);
    }
    if ((c + 1) % fl == 0) flush();
  }
  const long long cw = (long long)cout * cin * W;
  double *o = part + (size_t)blockIdx.x * (cw + cout);
  const int ci = ci0 + 16 * wi + li;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int co = co0 + 16 * wc + 4 * lg + q;
    if (co < cout && ci < cin) {
#pragma unroll
      for (int j = 0; j < W; ++j) o[((size_t)co * cin + ci) * W + j] = sum[j][q];
    }
    if (co < cout && bias && li == 0) o[cw + co] = sum[W][q];
  }
}

// out[e] = sum over z < parts of part[z * count + e] (FP64): thread group q of a workgroup adds
// z = q, q + 8, ..., then the groups are added in order. (One chain of loads per element would
// be bound by their latency.)
__global__ void __launch_bounds__(256)
    part_sum_kernel(long long count, int parts, const double *__restrict__ part,
                    float *__restrict__ out) {
  __shared__ double red[256];
  const int q = threadIdx.x >> 5;
  const long long e = (long long)blockIdx.x * 32 + (threadIdx.x & 31);
  double acc = 0.0;
  if (e < count) {
#pragma unroll 8
    for (int z = q; z < parts; z += 8) acc += part[(size_t)z * count + e];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (q == 0 && e < count) {
    for (int g = 1; g < 8; ++g) acc += red[32 * g + threadIdx.x];
    out[e] = (float)acc;
  }
}

__global__ void adam_kernel(long long count, float *__restrict__ p, const float *__restrict__ g,
                            float *__restrict__ m, float *__restrict__ v, float lr, float b1,
                            float b2, float eps, float c1, float c2, Frag fm,
                            float *__restrict__ frag) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  frag_put(fm, i, pi, frag);
}

__global__ void f2d_kernel(long long count, const float *__restrict__ a, double *__restrict__ b) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) b[i] = (double)a[i];
}

// identity blocks (k x k per sample)
__global__ void eye_kernel(int k, int batch, double *__restrict__ I) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)k * k * batch) return;
  const int e = (int)(i % ((long long)k * k));
  I[i] = (e % k == e / k) ? 1.0 : 0.0;
}

// WA[s][i][j] = w[s][i] A[s][i][j] (A column-major k x k per sample)
__global__ void scale_rows_kernel(int k, int batch, const double *__restrict__ w,
                                  const double *__restrict__ A, double *__restrict__ WA) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)k * k * batch) return;
  const int s = (int)(i / ((long long)k * k));
  const int row = (int)(i % k);
  WA[i] = w[(size_t)s * k + row] * A[i];
}

// gN[s] = -(2 / sum w) (X - PX) as FP32
__global__ void capture_grad_kernel(int n, int k, const double *__restrict__ w,
                                    const double *__restrict__ X, const double *__restrict__ PX,
                                    float *__restrict__ gN) {
  const int s = blockIdx.y;
  double sw = 0.0;
  for (int i = 0; i < k; ++i) sw += w[(size_t)s * k + i];
  const size_t nk = (size_t)n * k;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < nk;
       e += (size_t)gridDim.x * blockDim.x)
    gN[s * nk + e] = (float)(-(2.0 / sw) * (X[s * nk + e] - PX[s * nk + e]));
}

// loss[s] = -(1 / sum w) sum_i w_i sum_j C_ij A_ij (C, A column-major k x k per sample);
// one workgroup per sample, fixed-order tree reduction.
__global__ void __launch_bounds__(256)
    capture_value_kernel(int k, const double *__restrict__ w, const double *__restrict__ C,
                         const double *__restrict__ A, double *__restrict__ loss) {
  __shared__ double red[256];
  const int s = blockIdx.x;
  const size_t kk = (size_t)k * k;
  double acc = 0.0;
  for (size_t e = threadIdx.x; e < kk; e += blockDim.x)
    acc += w[(size_t)s * k + e % k] * C[s * kk + e] * A[s * kk + e];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double sw = 0.0;
    for (int i = 0; i < k; ++i) sw += w[(size_t)s * k + i];
    loss[s] = -red[0] / sw;
  }
}

unsigned nblocks(long long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace
}  // namespace riot

struct riot_net {
  riot_net_desc d{};
  hipStream_t st = nullptr;
  long long nparams = 0;
  std::vector<long long> woff, boff;  // per layer offsets into the flat parameters
  std::vector<int> cin, cout;
  riot::Frag fm{};                    // the weights in operand order: follow params
  float *frag = nullptr;
  size_t nfrag = 0;
  float *params = nullptr, *grads = nullptr, *am = nullptr, *av = nullptr;
  float *x0 = nullptr;               // standardized inputs [batch][in_channels][n]
  std::vector<float *> acts;         // per layer outputs [batch][cout][n]
  float *g0 = nullptr, *g1 = nullptr, *gN = nullptr;
  float *Nout = nullptr;             // network output after the head [batch][k][n]
  double *wpart = nullptr;           // partial weight and bias gradients
  // loss workspace (FP64)
  double *Nd = nullptr, *G = nullptr, *Lc = nullptr, *Z = nullptr, *Gi = nullptr, *A = nullptr,
         *WA = nullptr, *C = nullptr, *Y1 = nullptr, *Y2 = nullptr, *MN = nullptr, *X = nullptr,
         *PX = nullptr, *loss = nullptr;
  int *flags = nullptr;
  riot::CholJob *chol_jobs = nullptr;
  riot::TrsmJob *trsm_jobs = nullptr;
};

namespace {

size_t n256(size_t b) { return (b + 255) / 256 * 256; }

// Split of a layer's weight gradient: channel tiles per workgroup (16 wc output, 16 wi input
// channels: four waves, along the side that has them), and as many workgroups along the grid
// points as give one per compute unit (256) with the tiles.
struct WgradPlan {
  int wc, wi, chunks, per, parts, fl;
  int most;  // parts beside the tiles that fill the compute units
};
WgradPlan wgrad_plan(int batch, int n, int cin, int cout) {
  WgradPlan p;
  p.wc = cin <= 16 ? 4 : (cout <= 16 ? 1 : 2);
  p.wi = 4 / p.wc;
  const int tiles = ((cin + 16 * p.wi - 1) / (16 * p.wi)) * ((cout + 16 * p.wc - 1) / (16 * p.wc));
  p.most = 256 / tiles;
  p.chunks = batch * (n / riot::kCP);
  p.fl = n % 256 == 0 ? 4 : (n % 128 == 0 ? 2 : 1);
  p.per = (p.chunks / p.fl + p.most - 1) / p.most * p.fl;
  p.parts = (p.chunks + p.per - 1) / p.per;
  return p;
}

// As many parts as any batch up to batch_max can have: one per fl chunks, and no more than `most`.
long long wgrad_max_parts(int batch_max, int n, int cin, int cout) {
  const WgradPlan p = wgrad_plan(1, n, cin, cout);
  return std::min((long long)batch_max * (p.chunks / p.fl), (long long)p.most);
}

struct NCarve {
  char *base;
  size_t off = 0;
  explicit NCarve(void *b) : base(static_cast<char *>(b)) {}
  template <typename T>
  T *take(size_t n) {
    off = n256(off);
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += std::max<size_t>(n, 1) * sizeof(T);
    return p;
  }
};

bool net_desc_ok(const riot_net_desc *d) {
  return d && d->n >= 64 && d->n % 64 == 0 && d->layers >= 1 && d->layers <= 16 &&
         d->channels >= 1 && d->channels <= 64 && d->k >= 1 && d->k <= 64 && d->k <= d->n &&
         d->width >= 1 && d->width % 2 == 1 && d->width <= riot::kMaxWidth &&
         d->batch_max >= 1 && d->segments >= 1 && d->n % d->segments == 0 &&
         d->k % d->segments == 0 && d->in_channels >= 1 && d->in_channels <= 64;
}

size_t net_carve(riot_net &h, void *base) {
  NCarve c(base);
  const riot_net_desc &d = h.d;
  h.woff.clear(), h.boff.clear(), h.cin.clear(), h.cout.clear();
  long long np = 0;
  int ci = d.in_channels;
  int maxc = 1;
  for (int l = 0; l < d.layers; ++l) {
    const int co = (l == d.layers - 1) ? d.k / d.segments : d.channels;
    h.cin.push_back(ci), h.cout.push_back(co);
    h.woff.push_back(np);
    np += (long long)co * ci * d.width;
    h.boff.push_back(np);
    np += co;
    maxc = std::max(maxc, co);
    ci = co;
  }
  h.nparams = np;
  const size_t B = d.batch_max, n = d.n, k = d.k, kk = (size_t)k * k;
  h.params = c.take<float>(np);
  h.grads = c.take<float>(np);
  h.fm.layers = d.layers, h.fm.width = d.width;
  long long nf = 0;
  for (int l = 0; l < d.layers; ++l) {
    h.fm.cin[l] = h.cin[l], h.fm.cout[l] = h.cout[l], h.fm.woff[l] = h.woff[l];
    h.fm.fwd[l] = nf;
    nf += riot::frag_floats(h.cin[l], h.cout[l], d.width);
    h.fm.bwd[l] = nf;
    if (l > 0) nf += riot::frag_floats(h.cout[l], h.cin[l], d.width);
  }
  h.nfrag = nf;
  h.frag = c.take<float>(nf);
  h.am = c.take<float>(np);
  h.av = c.take<float>(np);
  h.x0 = c.take<float>(B * d.in_channels * n);
  h.acts.assign(d.layers, nullptr);
  for (int l = 0; l < d.layers; ++l) h.acts[l] = c.take<float>(B * h.cout[l] * n);
  h.g0 = c.take<float>(B * maxc * n);
  h.g1 = c.take<float>(B * maxc * n);
  h.gN = c.take<float>(B * k * n);
  h.Nout = c.take<float>(B * k * n);
  {
    size_t mx = 0;
    for (int l = 0; l < d.layers; ++l)
      mx = std::max(mx, (size_t)wgrad_max_parts(d.batch_max, (int)n, h.cin[l], h.cout[l]) *
                            ((size_t)h.cout[l] * h.cin[l] * d.width + h.cout[l]));
    h.wpart = c.take<double>(mx);
  }
  h.Nd = c.take<double>(B * n * k);
  h.G = c.take<double>(B * kk);
  h.Lc = c.take<double>(B * kk);
  h.Z = c.take<double>(B * kk);
  h.Gi = c.take<double>(B * kk);
  h.A = c.take<double>(B * kk);
  h.WA = c.take<double>(B * kk);
  h.C = c.take<double>(B * kk);
  h.Y1 = c.take<double>(B * kk);
  h.Y2 = c.take<double>(B * kk);
  h.MN = c.take<double>(B * n * k);
  h.X = c.take<double>(B * n * k);
  h.PX = c.take<double>(B * n * k);
  h.loss = c.take<double>(B);
  h.flags = c.take<int>(2 * B);
  h.chol_jobs = c.take<riot::CholJob>(B);
  h.trsm_jobs = c.take<riot::TrsmJob>(B);
  return n256(c.off) + 256;
}

#define NET_HIP(call)                           \
  do {                                          \
    if ((call) != hipSuccess) return RIOT_E_HIP; \
  } while (0)

// Convolution of `batch` samples: the forward layer (weights in operand order, b; ReLU when relu), or with act the
// backward-data pass of a layer cout -> cin. Grid points per wave: the most (64, 32, 16) that
// leave two workgroups per compute unit, since the weights are read once per workgroup.
template <int W, bool FLIP>
void launch_conv(riot_net *h, int batch, const float *in, int cin, int cout, const float *wf,
                 const float *b, const float *act, float *out, bool relu) {
  const int n = h->d.n, cgs = cout > 32 ? 4 : (cout > 16 ? 2 : 1), xw = 4 / cgs;
  int nt = std::min(4, 4 / xw);
  while (nt > 1 && (long long)batch * (n / (16 * nt * xw)) < 512) nt /= 2;
  const int XT = 16 * nt * xw;
  const size_t lds = (size_t)((cin + 3) / 4 * 4) * (XT + W - 1) * sizeof(float);
  const dim3 grid(n / XT, batch);
#define RIOT_CONV(NT_)                                                                          \
  hipLaunchKernelGGL((riot::conv_kernel<W, NT_, FLIP>), grid, dim3(256), lds, h->st, n, cin, cout, \
                     cgs, in, wf, b, act, out, relu ? 1 : 0)
  if (nt == 4)
    RIOT_CONV(4);
  else if (nt == 2)
    RIOT_CONV(2);
  else
    RIOT_CONV(1);
#undef RIOT_CONV
}

template <int W, int WC, int WI>
void launch_wgrad(riot_net *h, const WgradPlan &p, int cin, int cout, const float *g,
                  const float *hin) {
  const dim3 grid(p.parts, (cin + 16 * WI - 1) / (16 * WI), (cout + 16 * WC - 1) / (16 * WC));
  hipLaunchKernelGGL((riot::conv_wgrad_kernel<W, WC, WI>), grid, dim3(256), 0, h->st, h->d.n, cin,
                     cout, p.chunks, p.per, p.fl, g, hin, h->wpart);
}

#define RIOT_WIDTH(W_, CALL)                  \
  switch (W_) {                               \
    case 1: { constexpr int WW = 1; CALL; } break;   \
    case 3: { constexpr int WW = 3; CALL; } break;   \
    case 5: { constexpr int WW = 5; CALL; } break;   \
    case 7: { constexpr int WW = 7; CALL; } break;   \
    case 9: { constexpr int WW = 9; CALL; } break;   \
    case 11: { constexpr int WW = 11; CALL; } break; \
    default: return RIOT_E_ARG;               \
  }

riot_status conv_forward(riot_net *h, int batch, const float *in, int cin, int cout,
                         const float *W, const float *b, float *out, bool relu) {
  RIOT_WIDTH(h->d.width, (launch_conv<WW, false>(h, batch, in, cin, cout, W, b, nullptr, out, relu)));
  NET_HIP(hipGetLastError());
  return RIOT_OK;
}

// out = the gradient of the layer's input, zeroed where act <= 0 (layer: cout -> cin channels)
riot_status conv_backward_data(riot_net *h, int batch, const float *g, int cin, int cout,
                               const float *W, const float *act, float *out) {
  RIOT_WIDTH(h->d.width, (launch_conv<WW, true>(h, batch, g, cin, cout, W, nullptr, act, out, false)));
  NET_HIP(hipGetLastError());
  return RIOT_OK;
}

// grads: the layer's weights, then its biases
riot_status weight_grad(riot_net *h, int batch, int cin, int cout, const float *g,
                        const float *hin, float *grads) {
  const WgradPlan p = wgrad_plan(batch, h->d.n, cin, cout);
  if (p.wc == 4) {
    RIOT_WIDTH(h->d.width, (launch_wgrad<WW, 4, 1>(h, p, cin, cout, g, hin)));
  } else if (p.wc == 2) {
    RIOT_WIDTH(h->d.width, (launch_wgrad<WW, 2, 2>(h, p, cin, cout, g, hin)));
  } else {
    RIOT_WIDTH(h->d.width, (launch_wgrad<WW, 1, 4>(h, p, cin, cout, g, hin)));
  }
  NET_HIP(hipGetLastError());
  const long long count = (long long)cout * cin * h->d.width + cout;
  hipLaunchKernelGGL(riot::part_sum_kernel, dim3((unsigned)((count + 31) / 32)), dim3(256), 0,
                     h->st, count, p.parts, h->wpart, grads);
  NET_HIP(hipGetLastError());
  return RIOT_OK;
}

}  // namespace

extern "C" {

size_t riot_net_workspace_bytes(const riot_net_desc *desc) {
  if (!net_desc_ok(desc)) return 0;
  riot_net h;
  h.d = *desc;
  return net_carve(h, nullptr);
}

riot_status riot_net_init(const riot_net_desc *desc, void *workspace, size_t bytes,
                          void *hip_stream, riot_net **out) {
  if (!out) return RIOT_E_ARG;
  *out = nullptr;
  if (!net_desc_ok(desc) || !workspace) return RIOT_E_ARG;
  if (reinterpret_cast<uintptr_t>(workspace) % 256) return RIOT_E_WORKSPACE;
  if (bytes < riot_net_workspace_bytes(desc)) return RIOT_E_WORKSPACE;
  riot_net *h = new (std::nothrow) riot_net();
  if (!h) return RIOT_E_ARG;
  h->d = *desc;
  h->st = static_cast<hipStream_t>(hip_stream);
  net_carve(*h, workspace);
  // batched Cholesky / triangular-solve jobs of the loss (k x k per sample)
  const int k = desc->k, B = desc->batch_max;
  const size_t kk = (size_t)k * k;
  std::vector<riot::CholJob> cj(B);
  std::vector<riot::TrsmJob> tj(B);
  for (int s = 0; s < B; ++s) {
    cj[s] = {k, h->G + s * kk, h->Lc + s * kk, 0.0, h->flags + 2 * s, h->flags + 2 * s + 1,
             nullptr, nullptr};
    tj[s] = {k, k, h->Z + s * kk, k, h->Lc + s * kk, nullptr, nullptr};
  }
  riot_status rs = RIOT_OK;
  if (hipMemcpyAsync(h->chol_jobs, cj.data(), B * sizeof(riot::CholJob), hipMemcpyHostToDevice,
                     h->st) != hipSuccess ||
      hipMemcpyAsync(h->trsm_jobs, tj.data(), B * sizeof(riot::TrsmJob), hipMemcpyHostToDevice,
                     h->st) != hipSuccess ||
      hipMemsetAsync(h->frag, 0, h->nfrag * sizeof(float), h->st) != hipSuccess ||
      hipStreamSynchronize(h->st) != hipSuccess)
    rs = RIOT_E_HIP;
  if (rs != RIOT_OK) {
    delete h;
    return rs;
  }
  *out = h;
  return RIOT_OK;
}

void riot_net_free(riot_net *h) { delete h; }

int64_t riot_net_param_count(const riot_net *h) { return h ? h->nparams : 0; }

riot_status riot_net_set_params(riot_net *h, const float *params, const float *grads) {
  if (!h) return RIOT_E_ARG;
  if (params) {
    hipLaunchKernelGGL(riot::set_params_kernel, dim3(riot::nblocks(h->nparams)), dim3(256), 0, h->st,
                       (long long)h->nparams, h->fm, params, h->params, h->frag);
    NET_HIP(hipGetLastError());
  }
  if (grads)
    NET_HIP(hipMemcpyAsync(h->grads, grads, h->nparams * sizeof(float), hipMemcpyDeviceToDevice,
                           h->st));
  return RIOT_OK;
}

riot_status riot_net_get_params(riot_net *h, float *params, float *grads) {
  if (!h) return RIOT_E_ARG;
  if (params)
    NET_HIP(hipMemcpyAsync(params, h->params, h->nparams * sizeof(float),
                           hipMemcpyDeviceToDevice, h->st));
  if (grads)
    NET_HIP(hipMemcpyAsync(grads, h->grads, h->nparams * sizeof(float), hipMemcpyDeviceToDevice,
                           h->st));
  return RIOT_OK;
}

riot_status riot_net_forward(riot_net *h, int32_t batch, const double *x, float *N,
                             double *N64, int32_t ld64) {
  if (!h || !x || batch < 1 || batch > h->d.batch_max) return RIOT_E_ARG;
  const int n = h->d.n, k = h->d.k;
  if (N64 && ld64 < n) return RIOT_E_ARG;
  hipLaunchKernelGGL(riot::standardize_kernel, dim3(batch * h->d.in_channels), dim3(256), 0, h->st,
                     n, x, h->x0);
  NET_HIP(hipGetLastError());
  const float *in = h->x0;
  for (int l = 0; l < h->d.layers; ++l) {
    const bool last = l == h->d.layers - 1;
    float *out = h->acts[l];
    riot_status rs = conv_forward(h, batch, in, h->cin[l], h->cout[l], h->frag + h->fm.fwd[l],
                                  h->params + h->boff[l], out, !last);
    if (rs != RIOT_OK) return rs;
    in = out;
  }
  const int S = h->d.segments;
  const long long tot = (long long)batch * k * n;
  hipLaunchKernelGGL(riot::segment_out_kernel, dim3(riot::nblocks(tot)), dim3(256), 0, h->st, n,
                     k / S, S, tot, h->acts[h->d.layers - 1], N || N64 ? N : h->Nout, N64, ld64);
  NET_HIP(hipGetLastError());
  return RIOT_OK;
}

riot_status riot_net_backward(riot_net *h, int32_t batch, const float *gN) {
  if (!h || !gN || batch < 1 || batch > h->d.batch_max) return RIOT_E_ARG;
  const int n = h->d.n, L = h->d.layers;
  const int S = h->d.segments, kch = h->d.k / S;
  const long long tot = (long long)batch * kch * n;
  hipLaunchKernelGGL(riot::segment_grad_kernel, dim3(riot::nblocks(tot)), dim3(256), 0, h->st, n,
                     kch, S, tot, gN, h->g0);
  NET_HIP(hipGetLastError());
  float *g = h->g0, *gnext = h->g1;
  for (int l = L - 1; l >= 0; --l) {
    const int ci = h->cin[l], co = h->cout[l];
    const float *hin = l == 0 ? h->x0 : h->acts[l - 1];
    riot_status rs = weight_grad(h, batch, ci, co, g, hin, h->grads + h->woff[l]);
    if (rs != RIOT_OK) return rs;
    if (l > 0) {
      rs = conv_backward_data(h, batch, g, co, ci, h->frag + h->fm.bwd[l], h->acts[l - 1], gnext);
      if (rs != RIOT_OK) return rs;
      std::swap(g, gnext);
    }
  }
  return RIOT_OK;
}

riot_status riot_net_adam(riot_net *h, float lr, float beta1, float beta2, float eps, int32_t step) {
  if (!h || step < 1) return RIOT_E_ARG;
  const float c1 = 1.f - std::pow(beta1, (float)step), c2 = 1.f - std::pow(beta2, (float)step);
  if (step == 1) {
    NET_HIP(hipMemsetAsync(h->am, 0, h->nparams * sizeof(float), h->st));
    NET_HIP(hipMemsetAsync(h->av, 0, h->nparams * sizeof(float), h->st));
  }
  hipLaunchKernelGGL(riot::adam_kernel, dim3(riot::nblocks(h->nparams)), dim3(256), 0, h->st,
                     (long long)h->nparams, h->params, h->grads, h->am, h->av, lr, beta1, beta2,
                     eps, c1, c2, h->fm, h->frag);
  NET_HIP(hipGetLastError());
  return RIOT_OK;
}

riot_status riot_net_capture_loss(riot_net *h, int32_t batch, const float *N, const double *V,
                                  const double *w, double *loss_host, float *gN) {
  if (!h || !N || !V || !w || !gN || batch < 1 || batch > h->d.batch_max) return RIOT_E_ARG;
  const int n = h->d.n, k = h->d.k;
  const long long nk = (long long)n * k, kk = (long long)k * k;
  hipStream_t st = h->st;
  hipLaunchKernelGGL(riot::f2d_kernel, dim3(riot::nblocks(nk * batch)), dim3(256), 0, st,
                     nk * batch, N, h->Nd);
  NET_HIP(hipGetLastError());
  // G = N^T N = L L^T, Gi = L^{-T} L^{-1}
  NET_HIP(riot::gemm_f64_strided(1, 0, k, k, n, 1.0, h->Nd, n, nk, h->Nd, n, nk, 0.0, h->G, k, kk,
                                 batch, st));
  NET_HIP(riot::launch_chol_batched(batch, 0, h->chol_jobs, st));
  hipLaunchKernelGGL(riot::eye_kernel, dim3(riot::nblocks(kk * batch)), dim3(256), 0, st, k, batch,
                     h->Z);
  NET_HIP(hipGetLastError());
  NET_HIP(riot::launch_trsm_batched(batch, k, h->trsm_jobs, st));  // Z = L^{-T}
  NET_HIP(riot::gemm_f64_strided(0, 1, k, k, k, 1.0, h->Z, k, kk, h->Z, k, kk, 0.0, h->Gi, k, kk,
                                 batch, st));
  // A = V^T N, M N = V diag(w) A, X = M N Gi, P X = N Gi N^T X, C = A Gi
  NET_HIP(riot::gemm_f64_strided(1, 0, k, k, n, 1.0, V, n, nk, h->Nd, n, nk, 0.0, h->A, k, kk,
                                 batch, st));
  hipLaunchKernelGGL(riot::scale_rows_kernel, dim3(riot::nblocks(kk * batch)), dim3(256), 0, st, k,
                     batch, w, h->A, h->WA);
  NET_HIP(hipGetLastError());
  NET_HIP(riot::gemm_f64_strided(0, 0, n, k, k, 1.0, V, n, nk, h->WA, k, kk, 0.0, h->MN, n, nk,
                                 batch, st));
  NET_HIP(riot::gemm_f64_strided(0, 0, n, k, k, 1.0, h->MN, n, nk, h->Gi, k, kk, 0.0, h->X, n, nk,
                                 batch, st));
  NET_HIP(riot::gemm_f64_strided(1, 0, k, k, n, 1.0, h->Nd, n, nk, h->X, n, nk, 0.0, h->Y1, k, kk,
                                 batch, st));
  NET_HIP(riot::gemm_f64_strided(0, 0, k, k, k, 1.0, h->Gi, k, kk, h->Y1, k, kk, 0.0, h->Y2, k, kk,
                                 batch, st));
  NET_HIP(riot::gemm_f64_strided(0, 0, n, k, k, 1.0, h->Nd, n, nk, h->Y2, k, kk, 0.0, h->PX, n, nk,
                                 batch, st));
  NET_HIP(riot::gemm_f64_strided(0, 0, k, k, k, 1.0, h->A, k, kk, h->Gi, k, kk, 0.0, h->C, k, kk,
                                 batch, st));
  hipLaunchKernelGGL(riot::capture_grad_kernel, dim3(64, batch), dim3(256), 0, st, n, k, w, h->X,
                     h->PX, gN);
  NET_HIP(hipGetLastError());
  hipLaunchKernelGGL(riot::capture_value_kernel, dim3(batch), dim3(256), 0, st, k, w, h->C, h->A,
                     h->loss);
  NET_HIP(hipGetLastError());
  if (loss_host) {
    NET_HIP(hipMemcpyAsync(loss_host, h->loss, batch * sizeof(double), hipMemcpyDeviceToHost, st));
    NET_HIP(hipStreamSynchronize(st));
  }
  return RIOT_OK;
}

riot_status riot_net_train_step(riot_net *h, int32_t batch, const double *x, const double *V,
                                const double *w, float lr, int32_t step, double *loss_host) {
  if (!h || !x || !V || !w || batch < 1 || batch > h->d.batch_max || step < 1) return RIOT_E_ARG;
  riot_status rs = riot_net_forward(h, batch, x, nullptr, nullptr, 0);
  if (rs != RIOT_OK) return rs;
  rs = riot_net_capture_loss(h, batch, h->Nout, V, w, loss_host, h->gN);
  if (rs != RIOT_OK) return rs;
  rs = riot_net_backward(h, batch, h->gN);
  if (rs != RIOT_OK) return rs;
  return riot_net_adam(h, lr, 0.9f, 0.999f, 1e-8f, step);
}

}  // extern "C"
