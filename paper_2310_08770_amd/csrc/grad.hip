// Adjoint of the refined displacement and the Fisher information.
//
// At the Newton maximiser d of the band-limited correlation C(s) the
// gradient of C vanishes, so for L = g_d . d + g_c C(d) the implicit function
// theorem gives, with lam = -H^-1 g_d (H the Hessian of C at d),
//
//   dL/dA(x) = sum_k conj(F[B](k)) Psi(k) exp(-2 pi i k.x / N)
//   dL/dB(x) = sum_k F[A](k)       Psi(k) exp(+2 pi i k.x / N)
//   Psi(k)   = (lam_y d/ds_y + lam_x d/ds_x + g_c) phi_k(s) / N^2  at s = d,
//
// phi_k(s) = phi_ky(s_y) phi_kx(s_x) as in the forward pass (cos(pi s) for a
// Nyquist bin).  Both sums are real inverse transforms of Hermitian half
// spectra: Q_A = conj(R Psi) with R = conj F[B] (the resident reference
// spectrum) and Q_B = F[A] Psi.  CC-SN chains through A = (I+eps)^2 and
// B = -1/(E+eps).  The reference gradient is summed over frames in the
// frequency domain (fixed order, no float atomics) and transformed once.
//
// Fisher information of the displacement for an expected image mu under
// Poisson noise: F_jl = sum_r (d_j mu)(d_l mu) / mu, where d_j mu is the
// derivative of the band-limited translate mu(r - d) at d = 0.
#include <hip/hip_runtime.h>

#include <math.h>

#include "common.h"
#include "lds_frame.h"

namespace ccpt {

constexpr int kGThreads = 256;

__device__ __forceinline__ void phi2(int k, int n, double s, double2& p0, double2& p1) {
  const double pi = 3.14159265358979323846;
  if (2 * k == n) {
    double sn, cs;
    sincospi(s, &sn, &cs);
    p0 = make_double2(cs, 0.0);
    p1 = make_double2(-pi * sn, 0.0);
    return;
  }
  const int kt = 2 * k < n ? k : k - n;
  double sn, cs;
  sincospi(2.0 * (double)kt * s / (double)n, &sn, &cs);
  const double w = 2.0 * pi * (double)kt / (double)n;
  p0 = make_double2(cs, sn);
  p1 = make_double2(-w * sn, w * cs);
}

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ bool grad_usable(unsigned status) {
  return (status & (CCPT_ST_NONFINITE | CCPT_ST_FLAT | CCPT_ST_NEWTON_FALLBACK |
                    CCPT_ST_WINDOW_EXIT)) == 0;
}

// Psi of one frame: lam, the cotangent of C(d), and the phases of d.  With
// u = (g_c phi_kx + lam_x phi'_kx) / N^2 and v = lam_y phi_kx / N^2,
// Psi(ky, kx) = phi_ky u + phi'_ky v.
struct Adjoint {
  double lam_y, lam_x, gc;
  bool ok;
};

__device__ __forceinline__ Adjoint adjoint_of(const ccpt_result& r, int out_idx, const double* __restrict__ g_d,
                                              const double* __restrict__ g_peak) {
  Adjoint a{0.0, 0.0, 0.0, grad_usable(r.status)};
  if (a.ok) {
    const double gy = g_d[2 * out_idx], gx = g_d[2 * out_idx + 1];
    const double hyy = r.hess[0], hyx = r.hess[1], hxx = r.hess[2];
    const double det = hyy * hxx - hyx * hyx;
    // lam = -H^-1 g
    a.lam_y = -(hxx * gy - hyx * gx) / det;
    a.lam_x = -(hyy * gx - hyx * gy) / det;
    a.gc = g_peak ? g_peak[out_idx] : 0.0;
  }
  return a;
}

__device__ __forceinline__ void col_factors(int k, int n, double s, const Adjoint& a, double2& u, double2& v) {
  double2 p, dp;
  phi2(k, n, s, p, dp);
  const double inv = 1.0 / ((double)n * (double)n);
  u = make_double2((a.gc * p.x + a.lam_x * dp.x) * inv, (a.gc * p.y + a.lam_x * dp.y) * inv);
  v = make_double2(a.lam_y * p.x * inv, a.lam_y * p.y * inv);
}

__device__ __forceinline__ double2 psi_of(double2 py, double2 dpy, double2 u, double2 v) {
  const double2 a = zmul(py, u), b = zmul(dpy, v);
  return make_double2(a.x + b.x, a.y + b.y);
}

// One block per (ky block, frame): builds Psi on the half spectrum and writes
// QA = conj(R Psi) (frame gradient) and QB = F[A] Psi (reference gradient).
constexpr int kPsiRows = 16;

template <int N>
__global__ void __launch_bounds__(kGThreads) k_grad_psi(const FrameDesc* __restrict__ desc, int first,
                                                        const ccpt_result* __restrict__ fwd,
                                                        const double* __restrict__ g_d,
                                                        const double* __restrict__ g_peak,
                                                        const float2* __restrict__ FA,
                                                        float2* __restrict__ QA,
                                                        float2* __restrict__ QB) {
  constexpr int H = N / 2 + 1;
  __shared__ double2 ey0[kPsiRows], ey1[kPsiRows];
  __shared__ double2 ux[H], vx[H];
  const int tid = threadIdx.x;
  const int f = blockIdx.y;
  const int y0 = blockIdx.x * kPsiRows;
  const int rows = min(kPsiRows, N - y0);
  const FrameDesc d = desc[first + f];
  const ccpt_result r = fwd[d.out_idx];
  const Adjoint ad = adjoint_of(r, d.out_idx, g_d, g_peak);
  for (int k = tid; k < rows; k += kGThreads) phi2(y0 + k, N, r.d[0], ey0[k], ey1[k]);
  for (int k = tid; k < H; k += kGThreads) col_factors(k, N, r.d[1], ad, ux[k], vx[k]);
  __syncthreads();
  const size_t base = (size_t)f * N * H;
  const float2* R = (const float2*)d.rspec;
  for (int i = tid; i < rows * H; i += kGThreads) {
    const int ry = i / H, kx = i % H;
    const size_t e = (size_t)(y0 + ry) * H + kx;
    float2 qa = make_float2(0.f, 0.f), qb = qa;
    if (ad.ok) {
      const double2 psi = psi_of(ey0[ry], ey1[ry], ux[kx], vx[kx]);
      const float2 rr = R[e];
      const double2 ra = zmul(make_double2(rr.x, rr.y), psi);
      qa = make_float2((float)ra.x, (float)-ra.y);
      if (QB) {
        const float2 fa = FA[base + e];
        const double2 rb = zmul(make_double2(fa.x, fa.y), psi);
        qb = make_float2((float)rb.x, (float)rb.y);
      }
    }
    QA[base + e] = qa;
    if (QB) QB[base + e] = qb;
  }
}

// The whole adjoint of a frame that fits LDS, one block per frame: F[A], the
// product with Psi (QB to memory for the reference gradient, QA back into
// LDS), and the inverse transform times the chain factor to the caller's
// gradient array.  Memory sees the frame, the reference spectrum, QB and the
// gradient once; the passes (spectra, k_grad_psi, inverse, k_grad_frames) move
// eight spectra more per frame.  Bound as k_xcorr_lds by VALU issue and LDS.
// 1024 frames of 128 x 128: 233 us -> 110.  Larger frames than kLdsSmall have a
// CU each, so a last round of few goes to the passes: whole adjoint at 192 x
// 192, passes / one kernel, 8 frames 57 / 78 us, 64 frames 80 / 86, 128 frames
// 106 / 90; at 144 x 144 58 / 60, 76 / 65, 90 / 69 (kGradMinFrames lies
// between); at 128 x 128 one frame takes 52 / 50.
template <int N>
__global__ void __launch_bounds__(lds::lds_threads(N, N)) k_grad_lds(GradParams g) {
  using namespace lds;
  constexpr int THR = lds_threads(N, N), L = N / 2, H = L + 1, S = Col<N>::S;
  __shared__ float2 m[H * S];
  __shared__ float2 tw[N];
  __shared__ double2 ey0[N], ey1[N];
  __shared__ double2 ux[H], vx[H];
  const int f = blockIdx.x;
  const FrameDesc d = g.desc[g.first + f];
  const ccpt_result& r = g.fwd[d.out_idx];
  const Adjoint ad = adjoint_of(r, d.out_idx, g.g_d, g.g_peak);
  const bool sn = g.mode == CCPT_MODE_CCSN;
  for (int i = threadIdx.x; i < N; i += THR) tw[i] = g.tw[i];
  unsigned kmin, kmax, bad;
  load_frame<N, N, THR>(d, sn, g.eps, false, m, kmin, kmax, bad);
  for (int k = threadIdx.x; k < N + H; k += THR) {
    if (k < N)
      phi2(k, N, r.d[0], ey0[k], ey1[k]);
    else
      col_factors(k - N, N, r.d[1], ad, ux[k - N], vx[k - N]);
  }
  __syncthreads();
  if (g.QB) {
    rows_forward<N, N, THR>(m, tw, g.tw);
    stages<N, -1, H, N, N, false, THR, false, 0, 1>(m, tw, g.tw, NoUse());
  }
  {
    const float2* R = (const float2*)d.rspec;
    constexpr int BT = 4;  // reference values in flight per thread
    for (unsigned i0 = fresh_tid(); i0 < N * H; i0 += BT * THR) {
      float2 rr[BT];
#pragma unroll
      for (int e = 0; e < BT; ++e) rr[e] = R[min(i0 + e * THR, (unsigned)(N * H - 1))];
#pragma unroll
      for (int e = 0; e < BT; ++e) {
        const unsigned i = i0 + e * THR;
        if (i < N * H) {
          const unsigned y = i / H, kx = i % H, a = at<N, false>(kx, y);
          float2 qa = make_float2(0.f, 0.f), qb = qa;
          if (ad.ok) {
            const double2 psi = psi_of(ey0[y], ey1[y], ux[kx], vx[kx]);
            const double2 ra = zmul(make_double2(rr[e].x, rr[e].y), psi);
            qa = make_float2((float)ra.x, (float)-ra.y);
            const float2 fa = m[a];
            const double2 rb = zmul(make_double2(fa.x, fa.y), psi);
            qb = make_float2((float)rb.x, (float)rb.y);
          }
          m[a] = qa;
          if (g.QB) g.QB[(size_t)f * N * H + i] = qb;
        }
      }
    }
  }
  if (!g.g_frames) return;
  __syncthreads();
  stages<N, +1, H, N, N, false, THR, false, 0, 1>(m, tw, g.tw, NoUse());
  pack_rows<N, N, THR>(m, tw);
  stages<L, +1, N, N, N, true, THR, false, 0, 1>(m, tw, g.tw, NoUse());
  float* out = g.g_frames + g.goff[d.out_idx];
  for (unsigned i = fresh_tid(); i < N * L; i += THR) {
    const unsigned y = i / L, n = i % L;
    float2 v = m[at<N, true>(y, n)];
    v = make_float2(2.0f * v.x, 2.0f * v.y);  // the scale of the packed inverse
    if (sn) {
      const long idx = (long)y * d.pitch + 2 * n;
      v.x *= 2.0f * (lds::load_px(d.data, d.dtype, idx) + g.eps);
      v.y *= 2.0f * (lds::load_px(d.data, d.dtype, idx + 1) + g.eps);
    }
    out[2 * i] = v.x;
    out[2 * i + 1] = v.y;
  }
}

// Frame gradient: c2r output (already scaled) times the CC-SN chain factor
// 2 (I + eps), scattered to the caller's packed gradient array.
template <int N>
__global__ void k_grad_frames(const FrameDesc* __restrict__ desc, int first,
                              const float* __restrict__ img, const long* __restrict__ goff,
                              float* __restrict__ g_frames, int mode, float eps) {
  const int f = blockIdx.y;
  const FrameDesc d = desc[first + f];
  float* out = g_frames + goff[d.out_idx];
  const float* src = img + (size_t)f * N * N;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N * N; i += gridDim.x * blockDim.x) {
    float v = src[i];
    if (mode == CCPT_MODE_CCSN) {
      const int y = i / N, x = i - y * N;
      const long idx = (long)y * d.pitch + x;
      const float px = d.dtype == CCPT_U16   ? (float)((const unsigned short*)d.data)[idx]
                       : d.dtype == CCPT_F64 ? (float)((const double*)d.data)[idx]
                                             : ((const float*)d.data)[idx];
      v *= 2.0f * (px + eps);
    }
    out[i] = v;
  }
}

// acc[ref][k] += sum over the chunk's frames of that reference of QB[f][k], in
// two levels of fixed order: each run of at most kSumRun frames of one
// reference (order[run.x .. run.x + run.y)) is summed into its first frame's
// QB, then each reference's runs are summed into acc.  A thread has a run's
// loads in flight together; one thread per element over all frames waited for
// each in turn (795 frames of 128 x 128: 338 us -> 26).
template <int N>
__global__ void k_sum_runs(float2* __restrict__ QB, const int* __restrict__ order,
                           const int2* __restrict__ runs) {
  constexpr int NH = N * (N / 2 + 1);
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int2 run = runs[blockIdx.y];
  if (e >= NH || run.y < 2) return;
  float2 v[kSumRun];
#pragma unroll
  for (int j = 0; j < kSumRun; ++j) v[j] = QB[(size_t)order[run.x + min(j, run.y - 1)] * NH + e];
  float2 sum = v[0];
#pragma unroll
  for (int j = 1; j < kSumRun; ++j)
    if (j < run.y) sum = cadd(sum, v[j]);
  QB[(size_t)order[run.x] * NH + e] = sum;
}

template <int N>
__global__ void k_sum_refs(const float2* __restrict__ QB, const int* __restrict__ order,
                           const int2* __restrict__ runs, const int4* __restrict__ heads,
                           float2* const* __restrict__ acc) {
  constexpr int NH = N * (N / 2 + 1), BT = 8;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= NH) return;
  const int4 h = heads[blockIdx.y];  // reference, first run, runs
  float2 sum = make_float2(0.f, 0.f);
  for (int r0 = 0; r0 < h.z; r0 += BT) {
    float2 v[BT];
#pragma unroll
    for (int j = 0; j < BT; ++j)
      v[j] = QB[(size_t)order[runs[h.y + min(r0 + j, h.z - 1)].x] * NH + e];
#pragma unroll
    for (int j = 0; j < BT; ++j)
      if (r0 + j < h.z) sum = cadd(sum, v[j]);
  }
  float2* a = acc[h.x];
  a[e] = cadd(a[e], sum);
}

// Reference gradient image: chain factor of B = -1/(E+eps) is 1/(E+eps)^2.
__global__ void k_grad_ref_chain(const float* __restrict__ img, const float* __restrict__ E, int nn,
                                 int mode, float eps, float* __restrict__ out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nn; i += gridDim.x * blockDim.x) {
    float v = img[i];
    if (mode == CCPT_MODE_CCSN) {
      const float e = E[i] + eps;
      v /= e * e;
    }
    out[i] = v;
  }
}

// Derivative spectra of the band-limited translate at d = 0:
// d mu / d d_j = -sum_k F(k) (i w_kj) e^{2 pi i k.r/N} / N^2, Nyquist term 0.
template <int N>
__global__ void k_fisher_deriv(const float2* __restrict__ F, float2* __restrict__ Dy,
                               float2* __restrict__ Dx) {
  constexpr int H = N / 2 + 1;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N * H) return;
  const int ky = e / H, kx = e % H;
  const double pi = 3.14159265358979323846;
  const int kty = 2 * ky < N ? ky : ky - N;
  const double wy = (2 * ky == N) ? 0.0 : 2.0 * pi * kty / N;
  const double wx = (2 * kx == N) ? 0.0 : 2.0 * pi * kx / N;
  const double inv = 1.0 / ((double)N * (double)N);
  const float2 v = F[e];
  // -(i w) v = (w v.y, -w v.x)
  Dy[e] = make_float2((float)(wy * v.y * inv), (float)(-wy * v.x * inv));
  Dx[e] = make_float2((float)(wx * v.y * inv), (float)(-wx * v.x * inv));
}

// Per-block partial sums of (dy^2/mu, dy dx/mu, dx^2/mu) in FP64.
__global__ void k_fisher_partial(const float* __restrict__ dy, const float* __restrict__ dx,
                                 const void* __restrict__ mu, int dtype, int pitch, int n,
                                 double* __restrict__ part) {
  __shared__ double red[3][kGThreads / 64];
  double a = 0, b = 0, c = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n * n; i += gridDim.x * blockDim.x) {
    const int y = i / n, x = i - y * n;
    const long idx = (long)y * pitch + x;
    const double m = dtype == CCPT_U16   ? (double)((const unsigned short*)mu)[idx]
                     : dtype == CCPT_F64 ? ((const double*)mu)[idx]
                                         : (double)((const float*)mu)[idx];
    const double p = dy[i], q = dx[i];
    a += p * p / m;
    b += p * q / m;
    c += q * q / m;
  }
  double v[3] = {a, b, c};
  for (int t = 0; t < 3; ++t) {
    double s = v[t];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[t][threadIdx.x >> 6] = s;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0;
    for (int w = 0; w < kGThreads / 64; ++w) s += red[threadIdx.x][w];
    part[blockIdx.x * 3 + threadIdx.x] = s;
  }
}

__global__ void k_fisher_final(const double* __restrict__ part, int nblocks, double* __restrict__ out) {
  if (threadIdx.x < 3) {
    double s = 0;
    for (int b = 0; b < nblocks; ++b) s += part[b * 3 + threadIdx.x];
    out[threadIdx.x] = s;
  }
}

// ------------------------------------------------------------ launchers

template <int N>
static int grad_psi_n(const GradParams& g, const float2* FA, float2* QA, hipStream_t s) {
  hipLaunchKernelGGL((k_grad_psi<N>), dim3((N + kPsiRows - 1) / kPsiRows, g.count), dim3(kGThreads), 0, s,
                     g.desc, g.first, g.fwd, g.g_d, g.g_peak, FA, QA, g.QB);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int N>
static int grad_frames_n(const FrameDesc* desc, int first, int count, const float* img,
                         const long* goff, float* g_frames, int mode, float eps, hipStream_t s) {
  hipLaunchKernelGGL((k_grad_frames<N>), dim3((N * N + 255) / 256 < 64 ? (N * N + 255) / 256 : 64, count),
                     dim3(256), 0, s, desc, first, img, goff, g_frames, mode, eps);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int N>
static int ref_accum_n(float2* QB, const RefSums& t, float2* const* acc, hipStream_t s) {
  constexpr int blocks = (N * (N / 2 + 1) + 255) / 256;
  hipLaunchKernelGGL((k_sum_runs<N>), dim3(blocks, t.nruns), dim3(256), 0, s, QB, t.order, t.runs);
  hipLaunchKernelGGL((k_sum_refs<N>), dim3(blocks, t.nheads), dim3(256), 0, s, (const float2*)QB, t.order,
                     t.runs, t.heads, acc);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int N>
static int fisher_deriv_n(const float2* F, float2* Dy, float2* Dx, hipStream_t s) {
  constexpr int H = N / 2 + 1;
  hipLaunchKernelGGL((k_fisher_deriv<N>), dim3((N * H + 255) / 256), dim3(256), 0, s, F, Dy, Dx);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_grad_psi(int N, const GradParams& g, const float2* FA, float2* QA, hipStream_t s) {
  switch (N) {
#define CASE(n) \
  case n:       \
    return grad_psi_n<n>(g, FA, QA, s);
    CCPT_FOR_SIZES(CASE)
#undef CASE
  }
  return -2;
}

int launch_grad_lds(int N, const GradParams& g, hipStream_t s) {
#define CASE(n, n2)                                                                                   \
  if (N == n) {                                                                                       \
    hipLaunchKernelGGL((k_grad_lds<n>), dim3(g.count), dim3(lds::lds_threads(n, n)), 0, s, g);         \
    return hipGetLastError() == hipSuccess ? 0 : -1;                                                  \
  }
  CCPT_FOR_LDS_SQUARE(CASE)
#undef CASE
  return -2;
}

int launch_grad_frames(int N, const FrameDesc* desc, int first, int count, const float* img,
                       const long* goff, float* g_frames, int mode, float eps, hipStream_t s) {
  switch (N) {
#define CASE(n) \
  case n:       \
    return grad_frames_n<n>(desc, first, count, img, goff, g_frames, mode, eps, s);
    CCPT_FOR_SIZES(CASE)
#undef CASE
  }
  return -2;
}

int launch_ref_accum(int N, float2* QB, const RefSums& t, float2* const* acc, hipStream_t s) {
  switch (N) {
#define CASE(n) \
  case n:       \
    return ref_accum_n<n>(QB, t, acc, s);
    CCPT_FOR_SIZES(CASE)
#undef CASE
  }
  return -2;
}

int launch_grad_ref_chain(const float* img, const float* E, int nn, int mode, float eps,
                          float* out, hipStream_t s) {
  int blocks = (nn + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_grad_ref_chain, dim3(blocks), dim3(256), 0, s, img, E, nn, mode, eps, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_fisher_deriv(int N, const float2* F, float2* Dy, float2* Dx, hipStream_t s) {
  switch (N) {
#define CASE(n) \
  case n:       \
    return fisher_deriv_n<n>(F, Dy, Dx, s);
    CCPT_FOR_SIZES(CASE)
#undef CASE
  }
  return -2;
}

int launch_fisher_reduce(const float* dy, const float* dx, const void* mu, int dtype, int pitch,
                         int n, double* part, int nblocks, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fisher_partial, dim3(nblocks), dim3(kGThreads), 0, s, dy, dx, mu, dtype,
                     pitch, n, part);
  hipLaunchKernelGGL(k_fisher_final, dim3(1), dim3(64), 0, s, part, nblocks, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ccpt
