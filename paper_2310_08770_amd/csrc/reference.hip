// Reference images from aligned frames: the offline reference of Sec. III.A
// (Eq. 8), the mean of all frames shifted back by their measured
// displacements, and the real-time low-pass of Sec. III.B (Eq. 9), both
// taken in Fourier space.
//
// A frame I tracked at displacement d (frame(r) ~ ref(r - d)) shifted back
// is I(r + d), the paper's I(r - r0) with r0 = -d; its spectrum is
// F[I](k) phi_ky(d_y) phi_kx(d_x) with phi_k(s) = exp(2 pi i k~ s / N) and
// phi = cos(pi s) for a Nyquist bin (the band-limited shift, the same
// interpolant the tracker maximises).  Frames whose tracking was non-finite
// or flat are left out of the mean.
#include <hip/hip_runtime.h>

#include <math.h>

#include "common.h"
#include "lds_frame.h"
#include "shift.h"

namespace ccpt {

constexpr int kRefThreads = 256;
constexpr int kAlignRows = 8;  // spectrum rows per block of k_align_spectra

// F[f] (row-major N x (N/2+1)) *= phi_ky(d_y) phi_kx(d_x) for frame f's
// displacement; frames that did not track are zeroed, the others counted.
template <int N>
__global__ void __launch_bounds__(kRefThreads) k_align_spectra(const FrameDesc* __restrict__ desc,
                                                               int first,
                                                               const ccpt_result* __restrict__ fwd,
                                                               float2* __restrict__ F,
                                                               unsigned* __restrict__ cnt) {
  constexpr int H = N / 2 + 1;
  __shared__ float2 px[H];
  __shared__ float2 py[kAlignRows];
  const int f = blockIdx.y, y0 = blockIdx.x * kAlignRows, tid = threadIdx.x;
  const ccpt_result r = fwd[desc[first + f].out_idx];
  const bool ok = tracked(r);
  if (ok && blockIdx.x == 0 && tid == 0) atomicAdd(cnt, 1u);
  for (int k = tid; k < H; k += kRefThreads) px[k] = ok ? shift_phase(k, N, r.d[1]) : make_float2(0.f, 0.f);
  for (int k = tid; k < kAlignRows; k += kRefThreads)
    py[k] = (ok && y0 + k < N) ? shift_phase(y0 + k, N, r.d[0]) : make_float2(0.f, 0.f);
  __syncthreads();
  float2* Ff = F + (size_t)f * N * H;
  const int rows = min(kAlignRows, N - y0);
  for (int i = tid; i < rows * H; i += kRefThreads) {
    const int ry = i / H, kx = i - ry * H;
    const size_t e = (size_t)(y0 + ry) * H + kx;
    // (a frame that did not track may hold NaN: written as zeros, not scaled)
    Ff[e] = ok ? cmul(Ff[e], cmul(py[ry], px[kx])) : make_float2(0.f, 0.f);
  }
}

// The same from the frame itself, for frames that fit LDS: one block per frame
// transforms it there and writes the aligned spectrum, where the passes write
// and read two spectra more (256 frames of 192 x 192: 58 us -> 33).  The bits
// are those of the passes; launches split between the two as the correlation
// does (whole mean at 192 x 192, passes / LDS: 64 frames 46 / 47 us, 128 frames
// 60 / 54; at 128 x 128 one frame takes 28 / 28).
template <int N>
__global__ void __launch_bounds__(lds::lds_threads(N, N)) k_align_lds(const FrameDesc* __restrict__ desc, int first,
                                                                      const ccpt_result* __restrict__ fwd,
                                                                      const float2* __restrict__ gtw,
                                                                      float2* __restrict__ F,
                                                                      unsigned* __restrict__ cnt) {
  using namespace lds;
  constexpr int THR = lds_threads(N, N), H = N / 2 + 1, S = Col<N>::S;
  __shared__ float2 m[H * S];
  __shared__ float2 tw[N];
  __shared__ float2 px[H], py[N];
  const int f = blockIdx.x;
  const FrameDesc d = desc[first + f];
  const ccpt_result& r = fwd[d.out_idx];
  float2* Ff = F + (size_t)f * N * H;
  if (!tracked(r)) {  // (it may hold NaN: zeros, not a scaled spectrum)
    for (unsigned i = threadIdx.x; i < N * H; i += THR) Ff[i] = make_float2(0.f, 0.f);
    return;
  }
  if (threadIdx.x == 0) atomicAdd(cnt, 1u);
  for (int i = threadIdx.x; i < N; i += THR) tw[i] = gtw[i];
  unsigned kmin, kmax, bad;
  load_frame<N, N, THR>(d, false, 0.f, false, m, kmin, kmax, bad);
  for (int k = threadIdx.x; k < N + H; k += THR) {
    if (k < N)
      py[k] = shift_phase(k, N, r.d[0]);
    else
      px[k - N] = shift_phase(k - N, N, r.d[1]);
  }
  __syncthreads();
  rows_forward<N, N, THR>(m, tw, gtw);
  stages<N, -1, H, N, N, false, THR, false, 0, 1>(m, tw, gtw, NoUse());
  for (unsigned i = fresh_tid(); i < N * H; i += THR) {
    const unsigned y = i / H, kx = i % H;
    Ff[i] = cmul(m[at<N, false>(kx, y)], cmul(py[y], px[kx]));
  }
}

// acc[k] += sum over the chunk's frames of F[f][k], frames in order: one chain
// of additions per element, so it is the loads that have to overlap.  kSumLoads
// of them are in flight per thread (256 frames of 192 x 192: 64 us with one,
// 13 with them), and small blocks spread a frame's elements over the CUs.
constexpr int kSumThreads = 64, kSumLoads = 32;

template <int N>
__global__ void __launch_bounds__(kSumThreads) k_sum_spectra(int count, const float2* __restrict__ F,
                                                             float2* __restrict__ acc) {
  constexpr int NH = N * (N / 2 + 1);
  const int e = blockIdx.x * kSumThreads + threadIdx.x;
  if (e >= NH) return;
  float2 sum = make_float2(0.f, 0.f);
  for (int f0 = 0; f0 < count; f0 += kSumLoads) {
    float2 v[kSumLoads];
#pragma unroll
    for (int j = 0; j < kSumLoads; ++j) v[j] = F[(size_t)min(f0 + j, count - 1) * NH + e];
#pragma unroll
    for (int j = 0; j < kSumLoads; ++j)
      if (f0 + j < count) sum = cadd(sum, v[j]);
  }
  acc[e] = cadd(acc[e], sum);
}

// img *= scale / count (count >= 1; an empty mean is left as zeros)
__global__ void k_scale_by_count(float* __restrict__ img, int nn, float scale,
                                 const unsigned* __restrict__ cnt) {
  const unsigned c = *cnt;
  const float s = c ? scale / (float)c : 0.f;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nn; i += gridDim.x * blockDim.x)
    img[i] *= s;
}

template <int N>
static int align_n(const FrameDesc* desc, int first, int count, const ccpt_result* fwd, float2* F, unsigned* cnt,
                   hipStream_t s) {
  hipLaunchKernelGGL((k_align_spectra<N>), dim3((N + kAlignRows - 1) / kAlignRows, count), dim3(kRefThreads), 0, s,
                     desc, first, fwd, F, cnt);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_align(int N, const FrameDesc* desc, int first, int count, const ccpt_result* fwd, float2* F, unsigned* cnt,
                 hipStream_t s) {
  switch (N) {
#define CASE(n) \
  case n:       \
    return align_n<n>(desc, first, count, fwd, F, cnt, s);
    CCPT_FOR_SIZES(CASE)
#undef CASE
  }
  return -2;
}

int launch_align_lds(int N, const FrameDesc* desc, int first, int count, const ccpt_result* fwd, const float2* tw,
                     float2* F, unsigned* cnt, hipStream_t s) {
#define CASE(n, n2)                                                                                              \
  if (N == n) {                                                                                                  \
    hipLaunchKernelGGL((k_align_lds<n>), dim3(count), dim3(lds::lds_threads(n, n)), 0, s, desc, first, fwd, tw, F, cnt); \
    return hipGetLastError() == hipSuccess ? 0 : -1;                                                             \
  }
  CCPT_FOR_LDS_SQUARE(CASE)
#undef CASE
  return -2;
}

int launch_sum_spectra(int N, int count, const float2* F, float2* acc, hipStream_t s) {
  switch (N) {
#define CASE(n)                                                                                                \
  case n:                                                                                                      \
    hipLaunchKernelGGL((k_sum_spectra<n>), dim3((n * (n / 2 + 1) + kSumThreads - 1) / kSumThreads), dim3(kSumThreads), \
                       0, s, count, F, acc);                                                                   \
    return hipGetLastError() == hipSuccess ? 0 : -1;
    CCPT_FOR_SIZES(CASE)
#undef CASE
  }
  return -2;
}

int launch_scale_by_count(float* img, int nn, float scale, const unsigned* cnt, hipStream_t s) {
  int blocks = (nn + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_scale_by_count, dim3(blocks), dim3(256), 0, s, img, nn, scale, cnt);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ------------------------------------------------------------ references
__device__ __forceinline__ double ref_px(const void* p, int dtype, size_t idx) {
  if (dtype == CCPT_U16) return (double)((const unsigned short*)p)[idx];
  if (dtype == CCPT_F64) return ((const double*)p)[idx];
  return (double)((const float*)p)[idx];
}

__global__ void k_ref_check(const void* __restrict__ data, int dtype, int pitch, int ny, int nx, int mode,
                            double eps, unsigned* __restrict__ flag) {
  bool bad = false;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ny * nx; i += gridDim.x * blockDim.x) {
    const double v = ref_px(data, dtype, (size_t)(i / nx) * pitch + i % nx);
    bad |= !isfinite(v) || (mode == CCPT_MODE_CCSN && !(v + eps > 0.0));
  }
  if (bad) *flag = 1u;  // (every writer stores the same value)
}

__global__ void k_ref_copy(const void* __restrict__ data, int dtype, int pitch, int ny, int nx,
                           float* __restrict__ img) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ny * nx; i += gridDim.x * blockDim.x)
    img[i] = (float)ref_px(data, dtype, (size_t)(i / nx) * pitch + i % nx);
}

int launch_ref_check(const void* data, int dtype, int pitch, int ny, int nx, int mode, double eps,
                     unsigned* flag, hipStream_t s) {
  const int blocks = (ny * nx + 1023) / 1024;  // four pixels per thread
  hipLaunchKernelGGL(k_ref_check, dim3(blocks), dim3(256), 0, s, data, dtype, pitch, ny, nx, mode, eps, flag);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_ref_copy(const void* data, int dtype, int pitch, int ny, int nx, float* img, hipStream_t s) {
  const int blocks = (ny * nx + 1023) / 1024;
  hipLaunchKernelGGL(k_ref_copy, dim3(blocks), dim3(256), 0, s, data, dtype, pitch, ny, nx, img);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ccpt
