// Building blocks of the kernels that hold one frame's half spectrum in a CU's
// LDS (one block per frame) as m[kx][y], columns contiguous and padded.  Both
// directions of the transform work on that one layout without a transpose: the
// row transforms take lanes along y (consecutive LDS words, and one twiddle
// per wave), the column transforms lanes along the column.  Every Stockham
// stage runs in place: a thread holds its butterflies in registers across the
// barrier between the reads and the writes (16 or so complex values per
// thread), so one buffer is enough.
//
// Radices, twiddles and formulas are those of xcorr.hip in the same order, so
// spectra and images have the same bits on either path.
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"
#include "fft.h"

namespace ccpt {
namespace lds {

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
// multiple of 16, or (the Stockham write order, i0 = k + a BLOCK with k < STEP) a
// power of two below 16 whose BLOCK, STEP times the radix, divides 16 or is a
// multiple of it; pad() then adds as for i0 = 0.
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

// Frame d -> m[n][y], z[y][n] = A[y][2n] + i A[y][2n+1], A = I or (sn) (I + eps)^2;
// the extremes of A as ordered keys and whether a value is not finite.
// (Callers __syncthreads() before they use m.)
template <int NY, int NX, int THR>
__device__ __forceinline__ void load_frame(const FrameDesc& d, bool sn, float eps, bool trans, float2* m,
                                           unsigned& kmin_out, unsigned& kmax_out, unsigned& bad_out) {
  constexpr int L = NX / 2;
  const int tid = threadIdx.x;
  unsigned kmin = 0xFFFFFFFFu, kmax = 0, bad = 0;
  auto pro = [&](float a) {
    if (sn) a = (a + eps) * (a + eps);
    if (!isfinite(a)) bad = 1;
    kmin = min(kmin, f2key(a));
    kmax = max(kmax, f2key(a));
    return a;
  };
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
  kmin_out = kmin;
  kmax_out = kmax;
  bad_out = bad;
}

// Rows forward and their unpacking X[k] = E[k] + W^k O[k] (as k_rows_fwd).
// twr: exp(-2 pi i m / NX) in LDS; gtw: the shape's table in memory.
template <int NY, int NX, int THR>
__device__ __forceinline__ void rows_forward(float2* m, const float2* twr, const float2* __restrict__ gtw) {
  constexpr int L = NX / 2, H = L + 1;
  stages<L, -1, NY, NX, NY, true, THR, false, 0, 1>(m, twr, gtw, NoUse());
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
}

// Packs the bins of each row for its inverse, Z = E + i O (as k_rows_inv).
template <int NY, int NX, int THR>
__device__ __forceinline__ void pack_rows(float2* m, const float2* twr) {
  constexpr int L = NX / 2;
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
}

// Shapes whose m[kx][y] (with the tables) fits 160 KB.
#define CCPT_FOR_LDS_SQUARE(X)                                                                   \
  X(16, 16) X(18, 18) X(24, 24) X(32, 32) X(36, 36) X(48, 48) X(54, 54) X(64, 64) X(72, 72)      \
      X(96, 96) X(108, 108) X(128, 128) X(144, 144) X(162, 162) X(192, 192)
#define CCPT_FOR_LDS(X) CCPT_FOR_LDS_SQUARE(X) X(256, 128)

}  // namespace lds
}  // namespace ccpt
