// Correlation stage of frames whose half spectrum fits a CU's LDS (up to
// 192 x 192, and 256 x 128) in one kernel: prologue, forward 2-D r2c FFT,
// product with the resident conj F[B], inverse 2-D c2r FFT and the integer-lag
// maximum (Sec. II Eq. 4 / Eq. 7, Sec. III first paragraph), one block per
// frame.
//
// The three passes of xcorr.hip move the half spectrum through memory four
// times (T written and read twice) and wait on it in each of three launches;
// here it stays in LDS as m[kx][y] (columns contiguous, padded) from the first
// row stage to the last, so memory sees the frame, the reference spectrum and
// X once.  Both directions work on that one layout without a transpose: the
// row transforms take lanes along y (consecutive LDS words, and one twiddle
// per wave), the column transforms lanes along the column.  Every Stockham
// stage runs in place: a thread holds its butterflies in registers across the
// barrier between the reads and the writes (16 or so complex values per
// thread), so one buffer is enough.
//
// Radices, twiddles and formulas are those of xcorr.hip in the same order, so
// X and the correlation have the same bits on either path; which one a frame
// takes (xcorr_lds_frames) is a matter of time only.
//
// Bound by VALU issue (address arithmetic and butterflies, about 3400
// instructions per wave at 128 x 128) and the LDS passes.  us for the stage,
// three passes -> one kernel: 1024 frames of 64 x 64 63 -> 21, 96 x 96 114 -> 52, 128 x 128
// 143 -> 65, 192 x 192 323 -> 254, 256 x 128 306 -> 182; one frame of 64 x 64
// 22 -> 10, of 128 x 128 24 -> 22.
#include <hip/hip_runtime.h>

#include "common.h"
#include "fft.h"

namespace ccpt {

namespace {

// Threads per block: one radix-8 butterfly (eight complex values) per thread
// and stage for small frames, whose blocks are many to a CU; from 128 x 128 on
// 512 or 1024, so that one or two blocks fill a CU's four SIMDs evenly.
constexpr int lds_threads(int ny, int nx) {
  const int b8 = ny * (nx / 2 + 1) / 8;
  if (b8 > 1040) return 1024;
  if (b8 > 800) return 512;
  return (b8 + 63) / 64 * 64;
}

// A column of m: y sits at pad(y), columns `col_stride` apart.  The strided
// writes of the early stages of a power-of-two length want a slot after every
// 16; with a factor 3 in the length the strides are odd or spread anyway.
template <int NY>
struct Col {
  static constexpr bool PAD = (NY & (NY - 1)) == 0;
  static constexpr int S = PAD ? NY + NY / 16 + 1 : NY + 1;
  static __device__ __forceinline__ unsigned pad(unsigned y) { return PAD ? y + (y >> 4) : y; }
};

__device__ __forceinline__ float load_px(const void* p, int dtype, long idx) {
  if (dtype == CCPT_U16) return (float)((const unsigned short*)p)[idx];
  if (dtype == CCPT_F64) return (float)((const double*)p)[idx];
  return ((const float*)p)[idx];
}

// The thread index anew for each phase: the phases index LDS with the same
// expressions, and values kept from one to the next would fill the registers.
__device__ __forceinline__ unsigned fresh_tid() {
  unsigned t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Place of element i of sequence q: rows (q = y, i = column) or columns (q =
// column, i = y) of m[column][y].
template <int NY, bool ROW>
__device__ __forceinline__ unsigned at(unsigned q, unsigned i) {
  return ROW ? i * Col<NY>::S + Col<NY>::pad(q) : q * Col<NY>::S + Col<NY>::pad(i);
}

// Places of elements i0 + t STEP, t = 0, 1, ..: a constant step from the first
// for rows and unpadded columns.  In padded columns (powers of two) STEP is a
// multiple of 16, or a power of two below 16 with i0 mod 16 < STEP (the
// Stockham write order; pad() then adds as for i0 = 0).
template <int NY, bool ROW, int STEP>
__device__ __forceinline__ constexpr unsigned step_to(unsigned t) {
  return ROW ? t * STEP * Col<NY>::S : Col<NY>::PAD ? t * STEP + ((t * STEP) >> 4) : t * STEP;
}

// One Stockham stage of radix R (NS: product of the radices before it) of
// NSEQ sequences of length L in place; twiddle exp(SIGN 2 pi i t k / (NS R)) =
// tw[t k NTW / (NS R)], conjugated for SIGN > 0.  LAST: the results stay in
// registers and go to use(register, value) instead.
// gtw: where the twiddles of rows are read by scalar loads (every lane of a
// wave has the same column j when a wave's rows are of one column), the table
// in memory; tw: the table in LDS.
template <int L, int R, int SIGN, int NS, int NSEQ, int NTW, int NY, bool ROW, int THR, bool LAST, typename F>
__device__ __forceinline__ void stage(float2* m, const float2* tw, const float2* __restrict__ gtw, F&& use) {
  constexpr unsigned B = L / R, TOTAL = NSEQ * B;
  constexpr int IT = (TOTAL + THR - 1) / THR;
  constexpr bool SCALAR_TW = ROW && NSEQ % 64 == 0;
  // (a padded column read of step B < 16 is general: j need not be below B's block)
  constexpr bool READ_STEP = ROW || !Col<NY>::PAD || B % 16 == 0;
  float2 v[IT][R];
  const unsigned tid = fresh_tid();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const unsigned b = tid + it * THR;
    if (TOTAL % THR == 0 || b < TOTAL) {
      const unsigned q = ROW ? b % NSEQ : b / B, j = ROW ? b / NSEQ : b % B;
      const unsigned a = at<NY, ROW>(q, j);
#pragma unroll
      for (int t = 0; t < R; ++t)
        v[it][t] = m[READ_STEP ? a + step_to<NY, ROW, B>(t) : at<NY, ROW>(q, j + t * B)];
      if (NS > 1) {
        constexpr unsigned step = NTW / (NS * R);
        const unsigned k = SCALAR_TW ? (unsigned)__builtin_amdgcn_readfirstlane((int)(j % NS)) : j % NS;
#pragma unroll
        for (int t = 1; t < R; ++t) {
          float2 w = SCALAR_TW ? gtw[t * k * (step * (NY / NTW))] : tw[t * k * step];
          if (SIGN > 0) w.y = -w.y;
          v[it][t] = cmul(v[it][t], w);
        }
      }
      dft<R, SIGN>(v[it]);
    }
  }
  if constexpr (!LAST) __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const unsigned b = tid + it * THR;
    if (TOTAL % THR == 0 || b < TOTAL) {
      const unsigned q = ROW ? b % NSEQ : b / B, j = ROW ? b / NSEQ : b % B;
      const unsigned a = at<NY, ROW>(q, j / NS * (NS * R) + j % NS);
#pragma unroll
      for (int t = 0; t < R; ++t) {
        if constexpr (LAST)
          use(it * R + t, v[it][t]);
        else
          m[a + step_to<NY, ROW, NS>(t)] = v[it][t];
      }
    }
  }
  if constexpr (!LAST) __syncthreads();
}

struct NoUse {
  __device__ void operator()(int, float2) const {}
};

// All stages; KEEP: the last one's results go to use().
template <int L, int SIGN, int NSEQ, int NTW, int NY, bool ROW, int THR, bool KEEP, int ST, int NS, typename F>
__device__ __forceinline__ void stages(float2* m, const float2* tw, const float2* __restrict__ gtw, F&& use) {
  if constexpr (ST < fft_stages(L)) {
    constexpr int R = fft_radix(L, ST);
    constexpr bool last = KEEP && ST + 1 == fft_stages(L);
    if constexpr (last)
      stage<L, R, SIGN, NS, NSEQ, NTW, NY, ROW, THR, true>(m, tw, gtw, use);
    else
      stage<L, R, SIGN, NS, NSEQ, NTW, NY, ROW, THR, false>(m, tw, gtw, NoUse());
    stages<L, SIGN, NSEQ, NTW, NY, ROW, THR, KEEP, ST + 1, NS * R>(m, tw, gtw, use);
  }
}

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
  // ---- frame -> m[n][y], z[y][n] = A[y][2n] + i A[y][2n+1]
  const bool sn = g.mode == CCPT_MODE_CCSN;
  const float eps = g.eps;
  unsigned kmin = 0xFFFFFFFFu, kmax = 0, bad = 0;
  auto pro = [&](float a) {
    if (sn) a = (a + eps) * (a + eps);
    if (!isfinite(a)) bad = 1;
    kmin = min(kmin, f2key(a));
    kmax = max(kmax, f2key(a));
    return a;
  };
  const bool trans = transposed<NY, NX>(g.trans);
  const void* data = d.data;
  const long pitch = d.pitch;
  // uint16: A >= 0, whose float bits order as unsigned integers
  auto pro16 = [&](unsigned p) {
    float a = (float)p;
    if (sn) a = (a + eps) * (a + eps);
    kmin = min(kmin, __float_as_uint(a));
    kmax = max(kmax, __float_as_uint(a));
    return a;
  };
  auto keys16 = [&]() {
    bad = kmax >= 0x7F800000u ? 1u : 0u;
    kmin |= 0x80000000u;
    kmax |= 0x80000000u;
  };
  if (!trans && d.dtype == CCPT_U16 && NX % 8 == 0 && pitch % 8 == 0 && ((uintptr_t)data & 15) == 0) {
    for (unsigned i = tid; i < NY * (NX / 8); i += THR) {
      const unsigned r = i / (NX / 8), q = i % (NX / 8);
      const uint4 v = *(const uint4*)((const unsigned short*)data + r * pitch + 8 * q);
      const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        m[at<NY, true>(r, 4 * q + e)] = make_float2(pro16(w[e] & 0xFFFFu), pro16(w[e] >> 16));
    }
    keys16();
  } else if (!trans && d.dtype == CCPT_F32 && NX % 4 == 0 && pitch % 4 == 0 && ((uintptr_t)data & 15) == 0) {
    for (unsigned i = tid; i < NY * (NX / 4); i += THR) {
      const unsigned r = i / (NX / 4), q = i % (NX / 4);
      const float4 v = *(const float4*)((const float*)data + r * pitch + 4 * q);
      m[at<NY, true>(r, 2 * q)] = make_float2(pro(v.x), pro(v.y));
      m[at<NY, true>(r, 2 * q + 1)] = make_float2(pro(v.z), pro(v.w));
    }
  } else if (trans && d.dtype == CCPT_U16 && pitch % 8 == 0 && ((uintptr_t)data & 15) == 0) {
    // row y of the tall image is column y of the wide frame: eight columns of
    // two frame rows per thread
    for (unsigned i = tid; i < L * (NY / 8); i += THR) {
      const unsigned c = i / (NY / 8), q = i % (NY / 8);
      const unsigned short* p = (const unsigned short*)data + 2 * c * pitch + 8 * q;
      const uint4 v0 = *(const uint4*)p, v1 = *(const uint4*)(p + pitch);
      const unsigned a[4] = {v0.x, v0.y, v0.z, v0.w}, b[4] = {v1.x, v1.y, v1.z, v1.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        m[at<NY, true>(8 * q + 2 * e, c)] = make_float2(pro16(a[e] & 0xFFFFu), pro16(b[e] & 0xFFFFu));
        m[at<NY, true>(8 * q + 2 * e + 1, c)] = make_float2(pro16(a[e] >> 16), pro16(b[e] >> 16));
      }
    }
    keys16();
  } else if (trans) {
    for (unsigned i = tid; i < NY * L; i += THR) {
      const unsigned c = i / NY, r = i % NY;
      const long idx = 2 * c * pitch + r;
      const float a0 = pro(load_px(data, d.dtype, idx));
      const float a1 = pro(load_px(data, d.dtype, idx + pitch));
      m[at<NY, true>(r, c)] = make_float2(a0, a1);
    }
  } else {
    for (unsigned i = tid; i < NY * L; i += THR) {
      const unsigned r = i / L, c = i % L;
      const long idx = r * pitch + 2 * c;
      const float a0 = pro(load_px(data, d.dtype, idx));
      const float a1 = pro(load_px(data, d.dtype, idx + 1));
      m[at<NY, true>(r, c)] = make_float2(a0, a1);
    }
  }
  __syncthreads();
  // ---- rows forward, unpack X[k] = E[k] + W^k O[k] (as k_rows_fwd)
  stages<L, -1, NY, NX, NY, true, THR, false, 0, 1>(m, twr, g.tw, NoUse());
  {
    constexpr int IT = (H * NY + THR - 1) / THR;
    float2 o[IT];
    unsigned tp = fresh_tid();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const unsigned i = tp + it * THR;
      if ((H * NY) % THR == 0 || i < H * NY) {
        const unsigned k = i / NY, y = i % NY;
        const float2 zk = m[at<NY, true>(y, k == L ? 0 : k)];
        const float2 zc = cconj(m[at<NY, true>(y, k == 0 ? 0 : L - k)]);
        const float2 e = cscale(cadd(zk, zc), 0.5f);
        const float2 dd = csub(zk, zc);
        const float2 od = make_float2(0.5f * dd.y, -0.5f * dd.x);
        o[it] = cadd(e, cmul(twr[k], od));
      }
      if (it % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    tp = fresh_tid();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const unsigned i = tp + it * THR;
      if ((H * NY) % THR == 0 || i < H * NY) {
        const unsigned k = i / NY, y = i % NY;
        m[at<NY, true>(y, k)] = o[it];
      }
    }
    __syncthreads();
  }
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
          const float2 v = cmul(m[at<NY, false>(kx, y)], r[e]);
          Xf[i] = v;
          m[at<NY, false>(kx, y)] = v;
        }
      }
    }
    __syncthreads();
  }
  stages<NY, +1, H, NY, NY, false, THR, false, 0, 1>(m, tw, g.tw, NoUse());
  // ---- pack Z = E + i O (as k_rows_inv), rows inverse
  {
    constexpr int IT = (L * NY + THR - 1) / THR;
    float2 o[IT];
    unsigned tp = fresh_tid();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const unsigned i = tp + it * THR;
      if ((L * NY) % THR == 0 || i < L * NY) {
        const unsigned k = i / NY, y = i % NY;
        const float2 xk = m[at<NY, true>(y, k)];
        const float2 xc = cconj(m[at<NY, true>(y, L - k)]);
        const float2 e = cscale(cadd(xk, xc), 0.5f);
        const float2 od = cmul(cscale(csub(xk, xc), 0.5f), cconj(twr[k]));
        o[it] = make_float2(e.x - od.y, e.y + od.x);
      }
      if (it % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    tp = fresh_tid();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const unsigned i = tp + it * THR;
      if ((L * NY) % THR == 0 || i < L * NY) {
        const unsigned k = i / NY, y = i % NY;
        m[at<NY, true>(y, k)] = o[it];
      }
    }
    __syncthreads();
  }
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

// Shapes whose m[kx][y] (with the tables) fits 160 KB.
#define CCPT_FOR_LDS(X)                                                                       \
  X(16, 16) X(18, 18) X(24, 24) X(32, 32) X(36, 36) X(48, 48) X(54, 54) X(64, 64) X(72, 72)    \
      X(96, 96) X(108, 108) X(128, 128) X(144, 144) X(162, 162) X(192, 192) X(256, 128)

int xcorr_lds_frames(int ny, int nx, int count) {
  bool fits = false;
#define CASE(a, b) \
  if (ny == a && nx == b) fits = true;
  CCPT_FOR_LDS(CASE)
#undef CASE
  if (!fits) return 0;
  if (ny * (nx / 2 + 1) <= kLdsSmall) return count;
  const int rest = count % kLdsRound;
  return rest >= kLdsMinFrames ? count : count - rest;
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
