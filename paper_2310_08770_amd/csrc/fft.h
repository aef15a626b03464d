// Batched complex FFTs of length L = 2^a 3^b held in LDS, in Stockham
// (self-sorting) form: each stage reads its inputs with unit stride across
// butterflies and writes them back already in order, so no bit reversal
// pass is needed.  Radix 3 for the factors of 3, then radix 8, closing with
// radix 4 or 2.  Twiddles come from an LDS table of exp(-2 pi i m / N) for
// the transform size N of the kernel (L divides N).
#pragma once

#include <hip/hip_runtime.h>

namespace ccpt {

// Complex arithmetic on float2 (FP32 path) and double2 (FP64 path).
template <typename C>
struct cplx;
template <>
struct cplx<float2> {
  using real = float;
  static constexpr float sin60 = 0.86602540378443864676f;
  static constexpr float sqrt_half = 0.70710678118654752440f;
};
template <>
struct cplx<double2> {
  using real = double;
  static constexpr double sin60 = 0.86602540378443864676;
  static constexpr double sqrt_half = 0.70710678118654752440;
};
template <typename C>
using real_t = typename cplx<C>::real;

template <typename C>
__device__ __forceinline__ C mkc(real_t<C> x, real_t<C> y) {
  if constexpr (sizeof(C) == sizeof(float2))
    return make_float2(x, y);
  else
    return make_double2(x, y);
}
template <typename C>
__device__ __forceinline__ C cadd(C a, C b) { return mkc<C>(a.x + b.x, a.y + b.y); }
template <typename C>
__device__ __forceinline__ C csub(C a, C b) { return mkc<C>(a.x - b.x, a.y - b.y); }
template <typename C>
__device__ __forceinline__ C cmul(C a, C b) {
  return mkc<C>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// The same with its roundings fixed: left to the compiler, which product of a sum
// is fused depends on the code around it, and the kernels that form the
// cross-power spectrum have to agree (blocks of one value a thread, 16 x 16 to 24 x
// 24, had the products of y the other way round in the column pass).
template <typename C>
__device__ __forceinline__ C cmul_fixed(C a, C b) {
  return mkc<C>(fma(a.x, b.x, -(a.y * b.y)), fma(a.y, b.x, a.x * b.y));
}
template <typename C>
__device__ __forceinline__ C cconj(C a) { return mkc<C>(a.x, -a.y); }
template <typename C>
__device__ __forceinline__ C cscale(C a, real_t<C> s) { return mkc<C>(a.x * s, a.y * s); }
// multiply by i * SIGN
template <int SIGN, typename C>
__device__ __forceinline__ C mul_i(C a) {
  return SIGN > 0 ? mkc<C>(-a.y, a.x) : mkc<C>(a.y, -a.x);
}

// LDS layout of an FFT sequence: element i sits at lds_idx(i), with one
// unused slot after every 2^kLdsPadShift elements when the shift is nonzero,
// so the strided writes of the early Stockham stages spread over the LDS
// banks.  lds_len(n) slots hold a sequence of n elements.
constexpr int kLdsPadShift = 4;
__host__ __device__ constexpr unsigned lds_idx(unsigned i) {
  return kLdsPadShift ? i + (i >> kLdsPadShift) : i;
}
// Whether lds_idx(i0 + t STEP) = lds_idx(i0) + lds_idx(t STEP) for every t of a
// stage: STEP a multiple of the pad period, or (the Stockham write order, i0 =
// k + a BLOCK with k < STEP) a divisor of it with BLOCK dividing or divided by
// it.  The places of a butterfly's values are then constants apart.
constexpr bool lds_step(unsigned step, unsigned block) {
  constexpr unsigned p = 1u << kLdsPadShift;
  return step % p == 0 || (block && p % step == 0 && (block % p == 0 || p % block == 0));
}
__host__ __device__ constexpr int lds_len(int n) {
  return kLdsPadShift ? n + (n >> kLdsPadShift) : n;
}

constexpr int fft_radix(int L, int stage) {
  int i = 0;
  while (L % 3 == 0) {
    if (i == stage) return 3;
    L /= 3;
    ++i;
  }
  while (L % 8 == 0) {
    if (i == stage) return 8;
    L /= 8;
    ++i;
  }
  if (L % 4 == 0) {
    if (i == stage) return 4;
    L /= 4;
    ++i;
  }
  if (L % 2 == 0) {
    if (i == stage) return 2;
    L /= 2;
    ++i;
  }
  return 1;
}

constexpr int fft_stages(int L) {
  int s = 0;
  while (fft_radix(L, s) > 1) ++s;
  return s;
}

// In-register DFT of size R with exponent sign SIGN (-1 forward, +1 inverse).
template <int R, int SIGN, typename C>
__device__ __forceinline__ void dft(C* v) {
  using Rt = real_t<C>;
  if constexpr (R == 2) {
    C a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 3) {
    const Rt c = Rt(-0.5);
    const Rt s = SIGN * cplx<C>::sin60;
    C a = v[0], b = v[1], d = v[2];
    C t = cadd(b, d);
    C u = csub(b, d);
    v[0] = cadd(a, t);
    C m = mkc<C>(a.x + c * t.x, a.y + c * t.y);
    // i * s * u
    C r = mkc<C>(-s * u.y, s * u.x);
    v[1] = cadd(m, r);
    v[2] = csub(m, r);
  } else if constexpr (R == 4) {
    C a0 = v[0], a1 = v[1], a2 = v[2], a3 = v[3];
    C s02 = cadd(a0, a2), d02 = csub(a0, a2);
    C s13 = cadd(a1, a3), d13 = mul_i<SIGN>(csub(a1, a3));
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, d13);
    v[3] = csub(d02, d13);
  } else if constexpr (R == 8) {
    C e[4] = {v[0], v[2], v[4], v[6]};
    C o[4] = {v[1], v[3], v[5], v[7]};
    dft<4, SIGN>(e);
    dft<4, SIGN>(o);
    const Rt h = cplx<C>::sqrt_half;
    // w8^k = exp(SIGN * 2 pi i k / 8)
    C o1 = mkc<C>(h * (o[1].x - SIGN * o[1].y), h * (o[1].y + SIGN * o[1].x));
    C o2 = mul_i<SIGN>(o[2]);
    C o3 = mkc<C>(h * (-o[3].x - SIGN * o[3].y), h * (-o[3].y + SIGN * o[3].x));
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
  }
}

// One Stockham stage of radix R, in place, on `nseq` (at most MAXSEQ) sequences
// of length L (sequence q at buf + q*stride) by THR threads: a thread's
// butterflies stay in registers between the reads and, after a barrier, the
// writes, so no second buffer is needed and more blocks fit a CU (the passes
// wait on memory and LDS: 512 x 512 with 512 frames takes 1408 us against 1522
// with two buffers, 64 frames of 384 x 384 86 us against 93; a single frame is
// as fast either way).  NS = product of the radices already applied.  tw: exp(-2 pi i m / NTW), m < NTW, with L |
// NTW.  (Unsigned throughout: the divisions are by constants, and shifts for
// powers of two.)
template <int L, int R, int SIGN, int NTW, int NS, int MAXSEQ, int THR, typename C>
__device__ __forceinline__ void fft_stage(C* buf, unsigned nseq, unsigned stride, const C* tw, unsigned tid) {
  constexpr unsigned B = L / R;
  constexpr int IT = (MAXSEQ * B + THR - 1) / THR;
  constexpr bool RD = lds_step(B, 0), WR = lds_step(NS, NS * R);
  const unsigned total = nseq * B;
  C v[IT][R];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const unsigned b = tid + it * THR;
    if (b < total) {
      const unsigned q = b / B, j = b % B;
      const C* in = buf + q * stride;
      const unsigned j0 = lds_idx(j);
#pragma unroll
      for (unsigned t = 0; t < R; ++t) v[it][t] = in[RD ? j0 + lds_idx(t * B) : lds_idx(j + t * B)];
      if (NS > 1) {
        // twiddle exp(SIGN * 2 pi i t k / (NS R)) = tw[t k NTW / (NS R)] (conj for SIGN > 0)
        constexpr unsigned step = NTW / (NS * R);
        const unsigned k = j % NS;
#pragma unroll
        for (unsigned t = 1; t < R; ++t) {
          C w = tw[t * k * step];
          if (SIGN > 0) w.y = -w.y;
          v[it][t] = cmul(v[it][t], w);
        }
      }
      dft<R, SIGN>(v[it]);
      // the results are complete here: sums that the compiler moves past the
      // barrier are no longer fused with their products and round differently
      // from the same transform elsewhere
#pragma unroll
      for (unsigned t = 0; t < R; ++t) asm volatile("" : "+v"(v[it][t].x), "+v"(v[it][t].y));
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const unsigned b = tid + it * THR;
    if (b < total) {
      const unsigned q = b / B, j = b % B;
      C* out = buf + q * stride;
      const unsigned base = j / NS * (NS * R) + j % NS, base0 = lds_idx(base);
#pragma unroll
      for (unsigned t = 0; t < R; ++t) out[WR ? base0 + lds_idx(t * NS) : lds_idx(base + t * NS)] = v[it][t];
    }
  }
  __syncthreads();
}

template <int L, int SIGN, int NTW, int MAXSEQ, int THR, int ST, int NS, typename C>
__device__ __forceinline__ void fft_run(C* buf, unsigned nseq, unsigned stride, const C* tw, unsigned tid) {
  if constexpr (ST < fft_stages(L)) {
    constexpr int R = fft_radix(L, ST);
    fft_stage<L, R, SIGN, NTW, NS, MAXSEQ, THR>(buf, nseq, stride, tw, tid);
    fft_run<L, SIGN, NTW, MAXSEQ, THR, ST + 1, NS * R>(buf, nseq, stride, tw, tid);
  }
}

// Transforms nseq sequences in place, with a block of THR threads.  Callers
// must __syncthreads() before; the results are ready for every thread.
template <int L, int SIGN, int NTW, int MAXSEQ, int THR, typename C>
__device__ __forceinline__ void fft_lds(C* buf, unsigned nseq, unsigned stride, const C* tw) {
  fft_run<L, SIGN, NTW, MAXSEQ, THR, 0, 1>(buf, nseq, stride, tw, threadIdx.x);
}

}  // namespace ccpt
