// Correlation stage of frames whose half spectrum fits a CU's LDS (up to
// 192 x 192, and 256 x 128) in one kernel: prologue, forward 2-D r2c FFT,
// product with the resident conj F[B], inverse 2-D c2r FFT and the integer-lag
// maximum (Sec. II Eq. 4 / Eq. 7, Sec. III first paragraph), one block per
// frame.
//
// The three passes of xcorr.hip move the half spectrum through memory four
// times (T written and read twice) and wait on it in each of three launches;
// here it stays in LDS (lds_frame.h) from the first row stage to the last, so
// memory sees the frame, the reference spectrum and X once.  X and the
// correlation have the same bits on either path; which one a frame takes
// (lds_frames) is a matter of time only.
//
// Bound by VALU issue (address arithmetic and butterflies, about 3100
// instructions per wave at 128 x 128, which take 0.65 to 0.8 of the issue slots)
// and the waits on the LDS passes.  us for the stage,
// three passes -> one kernel: 1024 frames of 64 x 64 63 -> 21, 96 x 96 114 -> 52, 128 x 128
// 143 -> 65, 192 x 192 323 -> 254, 256 x 128 306 -> 182; one frame of 64 x 64
// 22 -> 10, of 128 x 128 24 -> 22.
#include <hip/hip_runtime.h>

#include "lds_frame.h"

namespace ccpt {

using namespace lds;

namespace {

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const T w = __shfl_xor(v, o, 64);
    v = w > v ? w : v;
  }
  return v;
}

}  // namespace

template <int NY, int NX>
__global__ void __launch_bounds__(lds_threads(NY, NX)) k_xcorr_lds(GroupParams g) {
  constexpr int THR = lds_threads(NY, NX), NW = THR / 64;
  constexpr int L = NX / 2, H = L + 1, S = Col<NY>::S, RX = NY / NX;
  __shared__ float2 m[H * S];
  __shared__ float2 tw[NY];
  __shared__ float2 twx[RX > 1 ? NX : 1];
  __shared__ float redf[2][NW];
  __shared__ unsigned redu[4][NW];
  const int tid = threadIdx.x, f = blockIdx.x;
  const FrameDesc d = g.desc[g.first + f];
  for (int i = tid; i < NY; i += THR) tw[i] = g.tw[i];
  const float2* twr = tw;
  if constexpr (RX > 1) {
    for (int i = tid; i < NX; i += THR) twx[i] = g.tw[i * RX];
    twr = twx;
  }
  unsigned kmin, kmax, bad;
  const bool trans = transposed<NY, NX>(g.trans);
  load_frame<NY, NX, THR>(d, g.mode == CCPT_MODE_CCSN, g.eps, trans, m, kmin, kmax, bad);
  __syncthreads();
  rows_forward<NY, NX, THR>(m, twr, g.tw);
  // ---- columns forward, X = F[A] conj F[B], columns inverse
  stages<NY, -1, H, NY, NY, false, THR, false, 0, 1>(m, tw, g.tw, NoUse());
  {
    const float2* R = (const float2*)d.rspec;
    float2* Xf = g.X + (size_t)f * NY * H;
    constexpr int BT = 8;  // reference values in flight per thread
    for (unsigned i0 = fresh_tid(); i0 < NY * H; i0 += BT * THR) {
      float2 r[BT];
#pragma unroll
      for (int e = 0; e < BT; ++e) r[e] = R[min(i0 + e * THR, (unsigned)(NY * H - 1))];
#pragma unroll
      for (int e = 0; e < BT; ++e) {
        const unsigned i = i0 + e * THR;
        if (i < NY * H) {
          const unsigned y = i / H, kx = i % H;
          const float2 v = cmul_fixed(m[at<NY, false>(kx, y)], r[e]);
          Xf[i] = v;
          m[at<NY, false>(kx, y)] = v;
        }
      }
    }
    __syncthreads();
  }
  stages<NY, +1, H, NY, NY, false, THR, false, 0, 1>(m, tw, g.tw, NoUse());
  pack_rows<NY, NX, THR>(m, twr);
  // ---- the two largest values (equal ones count twice), then the lowest
  // frame row-major index that holds the largest
  constexpr int RL = fft_radix(L, fft_stages(L) - 1);
  constexpr int NV = (NY * (L / RL) + THR - 1) / THR * RL;  // pairs per thread
  float2 z[NV];
  float t1 = -__builtin_inff(), t2 = t1;
#pragma unroll
  for (int e = 0; e < NV; ++e) z[e] = make_float2(t1, t1);
  stages<L, +1, NY, NX, NY, true, THR, true, 0, 1>(m, twr, g.tw, [&](int e, float2 v) {
    z[e] = v;
    float lo = fminf(t1, v.x);
    t1 = fmaxf(t1, v.x);
    t2 = fmaxf(t2, lo);
    lo = fminf(t1, v.y);
    t1 = fmaxf(t1, v.y);
    t2 = fmaxf(t2, lo);
  });
  auto merge2 = [](float& a1, float& a2, float b1, float b2) {
    const float lo = fminf(a1, b1);
    a1 = fmaxf(a1, b1);
    a2 = fmaxf(fmaxf(a2, b2), lo);
  };
  const float mine = t1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) merge2(t1, t2, __shfl_xor(t1, o, 64), __shfl_xor(t2, o, 64));
  kmin = ~wave_max(~kmin);
  kmax = wave_max(kmax);
  bad = wave_max(bad);
  if ((tid & 63) == 0) {
    redf[0][tid >> 6] = t1;
    redf[1][tid >> 6] = t2;
    redu[0][tid >> 6] = kmin;
    redu[1][tid >> 6] = kmax;
    redu[2][tid >> 6] = bad;
  }
  __syncthreads();
  t1 = redf[0][0];
  t2 = redf[1][0];
  for (int w = 1; w < NW; ++w) merge2(t1, t2, redf[0][w], redf[1][w]);
  unsigned idx = 0xFFFFFFFFu;
  if (mine == t1) {  // (few threads hold the maximum)
    constexpr unsigned B = L / RL, TOTAL = NY * B;
    const unsigned tf = fresh_tid();
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      const unsigned b = tf + e / RL * THR;
      if (TOTAL % THR == 0 || b < TOTAL) {
        // the last stage's outputs: sequence y = b mod NY, n = b / NY + t L / RL
        const unsigned y = b % NY, n = b / NY + e % RL * B;
        const unsigned flat = trans ? (unsigned)(2 * n * NY + y) : (unsigned)(y * NX + 2 * n);
        if (__float_as_uint(z[e].x) == __float_as_uint(t1)) idx = min(idx, flat);
        if (__float_as_uint(z[e].y) == __float_as_uint(t1)) idx = min(idx, flat + (trans ? (unsigned)NY : 1u));
      }
    }
  }
  idx = ~wave_max(~idx);
  if ((tid & 63) == 0) redu[3][tid >> 6] = idx;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < NW; ++w) {
      idx = min(idx, redu[3][w]);
      kmin = min(kmin, redu[0][w]);
      kmax = max(kmax, redu[1][w]);
      bad |= redu[2][w];
    }
    FrameState& st = g.st[f];
    st.peak_key = peak_key(t1, idx);
    st.second_key = peak_key(t2, 0u);
    st.amin = kmin;
    st.amax = kmax;
    if (bad) st.flags |= CCPT_ST_NONFINITE;
  }
}

int lds_frames(int ny, int nx, int count, int min_frames) {
  bool fits = false;
#define CASE(a, b) \
  if (ny == a && nx == b) fits = true;
  CCPT_FOR_LDS(CASE)
#undef CASE
  if (!fits) return 0;
  if (ny * (nx / 2 + 1) <= kLdsSmall) return count;
  const int rest = count % kLdsRound;
  return rest >= min_frames ? count : count - rest;
}

int launch_xcorr_lds(int ny, int nx, const GroupParams& g, hipStream_t s) {
#define CASE(a, b)                                                                                  \
  if (ny == a && nx == b) {                                                                         \
    hipLaunchKernelGGL((k_xcorr_lds<a, b>), dim3(g.count), dim3(lds_threads(a, b)), 0, s, g);        \
    return hipGetLastError() == hipSuccess ? 0 : -1;                                                \
  }
  CCPT_FOR_LDS(CASE)
#undef CASE
  return -2;
}

}  // namespace ccpt
