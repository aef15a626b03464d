// The correlation on the 1.5-px window around the integer peak: the upsampled
// grid and its maximum (Sec. III, first paragraph) and the FP64 refinement of
// that maximum, both from one FP64 pass over the cross-power spectrum X.
//
// With phi_k(s) = exp(2 pi i k~ s / N) (cos(pi s) for a Nyquist bin), p the
// integer peak and e = s - p, the band-limited correlation is
//
//   C(p + e) = 1/(NY NX) sum_kx w_kx Re[ phi_kx(px) phi_kx(ex)
//                sum_ky X[ky, kx] phi_ky(py) phi_ky(ey) ],  w = 1, 2, .., 2, 1.
//
// On |e| <= B (B about 0.8 px) the phases 2 pi k~ e / N stay below pi B, so
// each exponential is a short Chebyshev series
//
//   exp(i z x) = sum_n (2 - [n = 0]) i^n J_n(z) T_n(x),  x = e / B, z = 2 pi k~ B / N,
//
// whose terms fall as (z/2)^n / n!: 24 of them leave about 2 J_24(pi B),
// 5e-19 at B = 1.05 (the widest window) and 7e-22 at the paper's 1.5 px.  So
//
//   C(p + e) = sum_{n, m < 24} c[n][m] T_n(ey / B) T_m(ex / B)
//
// to FP64 rounding everywhere in the window, and 24 x 24 numbers stand for the
// whole spectrum: the M x M grid is T c T^T, and Newton's C, gradient and
// Hessian are sums over c.  The matrix-multiply DFT of the window
// (8 M N H + 4 M^2 H operations: 51 MFLOP for 256 x 256 at u = 100) becomes
// 24-row contractions (2 x 12 x N/2 x 2H products: 0.8 M) plus the grid's own
// 16 M^2 products.
//
// k_window_coef  sums the coefficients (FP64 matrix instructions);
// k_window_max   the grid maximum (FP32 matrix instructions; FP64 in the FP64
//                mode), the Newton iterations and the result record.
//
// Parity.  Rows q and NY - q have opposite frequencies, so with
// P_q, D_q = X[q] phi_q(py) +- X[NY-q] conj(phi_q(py)), q = 0 .. NY/2, even n
// take sum_q G_n[q] P_q and odd n take i sum_q G_n[q] D_q, with real tables
// G_n[q] = +-(2 - [n = 0]) J_n(z_q) (halved at q = 0 and NY/2, which pair with
// themselves; the Nyquist row's D vanishes since phi(py) = +-1): half the
// products of the plain sum, all real.  The same holds along x, where the
// real output needs Re for even m and Im for odd m.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "common.h"

namespace ccpt {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kNC2 = kChebN * kChebN;  // coefficients of a frame
static_assert(kChebN == 24 && kGridN == 16, "operand layouts below");
constexpr int kCThreads = 256;         // k_window_coef: four waves

__device__ __forceinline__ bool frame_skipped(const FrameState& s) {
  return (s.flags & CCPT_ST_NONFINITE) || s.amin == s.amax;
}

// Tall-image coordinates of a frame's integer peak, in [0, NY) x [0, NX).
__device__ __forceinline__ void peak_at(unsigned q, int ny, int nx, int trans, int& y, int& x) {
  if (q >= (unsigned)(ny * nx)) q = 0;
  const unsigned w = trans ? (unsigned)ny : (unsigned)nx;  // frame row length
  const int a = (int)(q / w), b = (int)(q % w);
  y = trans ? b : a;
  x = trans ? a : b;
}

// FP64 mode: the frame's integer peak from its row blocks' candidates, in
// fixed order (ties to the lower row-major index); tie: the runner-up (the
// largest block runner-up or a block maximum that lost) is a near tie.
__device__ unsigned peak_of_cands(const PeakCand* cd, int nb, bool& tie) {
  double bv = -__builtin_inf(), sv = -__builtin_inf();
  unsigned bi = 0xFFFFFFFFu;
  for (int j = 0; j < nb; ++j) {
    const double v = cd[j].v;
    const unsigned i = cd[j].idx;
    if (v > bv || (v == bv && i < bi)) {
      sv = bv > sv ? bv : sv;
      bv = v;
      bi = i;
    } else if (v > sv) {
      sv = v;
    }
    sv = cd[j].v2 > sv ? cd[j].v2 : sv;
  }
  tie = near_tie(bv, sv);
  return bi;
}

// ------------------------------------------------------------ coefficients
// One block of four waves per (frame, part).  The NX/2 columns kx < NX/2 are
// taken in tiles of 16, TPW tiles at a time by one wave (a "group"), and the
// row pairs q = 0 .. NY/2 in k steps of 4; QS waves of a block share a group,
// each over its own range of k steps, the others take other groups.  With
// nparts > 1 (few frames) the groups are spread over nparts blocks, whose
// coefficients k_window_max adds in block order.
//
// Per k step a lane holds column kx = lane mod 16 of the tile and row pair
// q = 4 ks + lane / 16: it loads X[q][kx] and X[NY-q][kx], forms P and D in
// FP64 and passes them as the A operands of four 16x16x4 matrix instructions
// against G (B operand: n = lane mod 16).  The products come out as
// D[kx = 4 v + lane/16][n = lane mod 16], register v, which is the B operand
// layout of the second contraction's k step v (kx = 4 v + lane / 16), so the
// sums over kx run on the registers, after the kx phase phi_kx(px), without a
// pass through LDS.
//
// The pass is meant to be bound by reading X once (264 KB per 256 x 256
// frame): the next kDepth - 1 k steps' loads are in flight while one is
// summed.  10,000 frames of 256 x 256 in launches of 768 take 0.83 ms
// (3.2 TB/s of the 5.2 that a copy reaches, matrix cores busy 0.39); other
// depths, three blocks per CU and one tile per wave were within 3 %.  With
// k_window_max it replaces the matrix DFT (1.6 ms on 16-bit operands, 7.3 ms in
// FP32) and Newton's own passes over X (0.8 ms).
template <typename CX, int TPW>
struct CoefStep {
  CX a[TPW], b[TPW];
  double2 g;
  CX na, nb;  // the Nyquist column (one wave of a frame)
};

template <typename CX, int TPW>
__global__ void __launch_bounds__(kCThreads, 2)
    k_window_coef(GroupParams g, WindowTables t, int ny, int nx, int qs) {
  constexpr int kDepth = 4;
  const int H = nx / 2 + 1, NC = nx / 2, NQ = ny / 2;
  __shared__ double2 phy[kMaxSide / 2 + 1];    // phi_q(py)
  __shared__ double2 phx[kMaxCols / 2];        // phi_kx(px)
  __shared__ double red[kCThreads / 64][kNC2];
  __shared__ double nyq[kCThreads / 64][kChebN];
  __shared__ int pk[2];
  // (the wave index is made scalar: the branches on it below are uniform)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f = blockIdx.y, part = blockIdx.x, nparts = gridDim.x;
  const FrameState st = g.st[f];
  if (frame_skipped(st)) return;
  int py, px;
  if constexpr (sizeof(CX) == sizeof(float2)) {
    peak_at(key_index(st.peak_key), ny, nx, g.trans, py, px);
  } else {
    if (tid == 0) {
      bool tie;
      peak_at(peak_of_cands(g.cand + (size_t)f * g.ncand, g.ncand, tie), ny, nx, 0, pk[0], pk[1]);
    }
    __syncthreads();
    py = pk[0];
    px = pk[1];
  }
  // (k p mod N) / N turns: exact at multiples of a quarter turn
  for (int q = tid; q <= NQ; q += kCThreads) {
    double sn, cs;
    sincospi(2.0 * (double)((unsigned)(q * py) % (unsigned)ny) / (double)ny, &sn, &cs);
    phy[q] = make_double2(cs, sn);
  }
  for (int k = tid; k < NC; k += kCThreads) {
    double sn, cs;
    sincospi(2.0 * (double)((unsigned)(k * px) % (unsigned)nx) / (double)nx, &sn, &cs);
    phx[k] = make_double2(cs, sn);
  }
  __syncthreads();

  const CX* Xf = (sizeof(CX) == sizeof(float2) ? (const CX*)g.X : (const CX*)g.X64) +
                 (size_t)f * ny * H;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int ntile = (NC + 15) / 16;
  const int ngrp = (ntile + TPW - 1) / TPW;
  const int qseg = wave % qs, slots = (kCThreads / 64 / qs) * nparts;
  const int slot = part * (kCThreads / 64 / qs) + wave / qs;
  const int ks0 = qseg * t.ksteps / qs, ks1 = (qseg + 1) * t.ksteps / qs;
  const bool nyq_wave = slot == (ngrp - 1) % slots;

  const f64x4 zero4 = {0.0, 0.0, 0.0, 0.0};
  f64x4 cee = zero4, coe = zero4, ceo = zero4, coo = zero4;  // c[m][n]: m parity, n parity
  double ne = 0.0, no = 0.0;                                 // Nyquist column: even n, odd n

  for (int grp = slot; grp < ngrp; grp += slots) {
    const bool nyq_here = nyq_wave && grp == slot;
    f64x4 er[TPW], ei[TPW], dr[TPW], di[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) er[i] = ei[i] = dr[i] = di[i] = zero4;
    unsigned kx[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) kx[i] = (unsigned)min((grp * TPW + i) * 16 + l16, NC - 1);
    CoefStep<CX, TPW> buf[kDepth];
    // (row pairs past NY/2 read the last one; their table entries are zero)
    auto load = [&](CoefStep<CX, TPW>& s, int ks) {
      const int q = min(4 * ks + l4, NQ);
      const unsigned o1 = (unsigned)(q * H), o2 = (unsigned)((q ? ny - q : 0) * H);
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        s.a[i] = Xf[o1 + kx[i]];
        s.b[i] = Xf[o2 + kx[i]];
      }
      s.g = t.gy[ks * 64 + lane];
      if (nyq_here) {
        s.na = Xf[o1 + NC];
        s.nb = Xf[o2 + NC];
      }
    };
    auto sum = [&](const CoefStep<CX, TPW>& s, int ks) {
      const double2 ph = phy[min(4 * ks + l4, NQ)];
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        const double ax = (double)s.a[i].x, ay = (double)s.a[i].y;
        const double bx = (double)s.b[i].x, by = (double)s.b[i].y;
        const double s1 = ax + bx, s2 = ay - by, s3 = ay + by, s4 = ax - bx;
        er[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(s1 * ph.x - s2 * ph.y, s.g.x, er[i], 0, 0, 0);
        ei[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(s3 * ph.x + s4 * ph.y, s.g.x, ei[i], 0, 0, 0);
        dr[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(s4 * ph.x - s3 * ph.y, s.g.y, dr[i], 0, 0, 0);
        di[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(s2 * ph.x + s1 * ph.y, s.g.y, di[i], 0, 0, 0);
      }
      if (nyq_here) {  // real parts only: Re P (even n) and Re(i D) = -Im D (odd n)
        const double ax = (double)s.na.x, ay = (double)s.na.y;
        const double bx = (double)s.nb.x, by = (double)s.nb.y;
        ne += s.g.x * ((ax + bx) * ph.x - (ay - by) * ph.y);
        no -= s.g.y * ((ay - by) * ph.x + (ax + bx) * ph.y);
      }
    };
#pragma unroll
    for (int d = 0; d < kDepth; ++d) load(buf[d], min(ks0 + d, t.ksteps - 1));
    for (int ks = ks0; ks < ks1; ks += kDepth) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {
        if (ks + d < ks1) sum(buf[d], ks + d);
        if (ks + d + kDepth < ks1) load(buf[d], ks + d + kDepth);
      }
    }
    // kx phase, then c[m][n] += sum_kx Gx_m[kx] (Re A_n for even m, Im A_n for odd m)
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int tile = grp * TPW + i;
      if (tile < ntile) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double2 ph = phx[min(tile * 16 + 4 * v + l4, NC - 1)];
          const double2 gx = t.gx[(tile * 4 + v) * 64 + lane];
          const double re = er[i][v] * ph.x - ei[i][v] * ph.y;
          const double ie = er[i][v] * ph.y + ei[i][v] * ph.x;
          // odd n: A = i (dr + i di)
          const double ro = -di[i][v] * ph.x - dr[i][v] * ph.y;
          const double io = -di[i][v] * ph.y + dr[i][v] * ph.x;
          cee = __builtin_amdgcn_mfma_f64_16x16x4f64(gx.x, re, cee, 0, 0, 0);
          coe = __builtin_amdgcn_mfma_f64_16x16x4f64(gx.y, ie, coe, 0, 0, 0);
          ceo = __builtin_amdgcn_mfma_f64_16x16x4f64(gx.x, ro, ceo, 0, 0, 0);
          coo = __builtin_amdgcn_mfma_f64_16x16x4f64(gx.y, io, coo, 0, 0, 0);
        }
      }
    }
  }
  // this wave's coefficients (m index 4 v + lane/16, n index lane mod 16)
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int mi = 4 * v + l4;
    if (mi < kChebN / 2 && l16 < kChebN / 2) {
      double* r = &red[wave][2 * l16 * kChebN + 2 * mi];
      r[0] = cee[v];
      r[1] = coe[v];
      r[kChebN] = ceo[v];
      r[kChebN + 1] = coo[v];
    }
  }
  ne += __shfl_xor(ne, 16, 64);
  ne += __shfl_xor(ne, 32, 64);
  no += __shfl_xor(no, 16, 64);
  no += __shfl_xor(no, 32, 64);
  if (lane < kChebN / 2) {
    nyq[wave][2 * lane] = ne;
    nyq[wave][2 * lane + 1] = no;
  }
  __syncthreads();
  // waves in order; the Nyquist column adds phi(px) = +-1 times its real
  // moments to the even m
  const double sgn = (px & 1) ? -1.0 : 1.0;
  double* out = g.coef + ((size_t)f * nparts + part) * kNC2;
  for (int i = tid; i < kNC2; i += kCThreads) {
    const int n = i / kChebN, m = i - n * kChebN;
    double v = red[0][i], w = nyq[0][n];
#pragma unroll
    for (int k = 1; k < kCThreads / 64; ++k) {
      v += red[k][i];
      w += nyq[k][n];
    }
    out[i] = v + ((m & 1) ? 0.0 : sgn * w * t.gxn[m >> 1]);
  }
}

// -------------------------------------------------- grid maximum and Newton
struct Deriv {
  double c, gy, gx, hyy, hxy, hxx;
};

// Lane moves of doubles by DPP (operand modifiers of VALU moves: no LDS
// traffic).  Every lane of the wave is active in the callers; lanes outside
// ROWS (or without a source lane) receive 0.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// A lane's value for the whole wave, in scalar registers.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Sum over the 64 lanes of a wave, fixed order: quads, half rows and rows of
// 16 by quad permutations and mirrors, then rows into the next (row_bcast),
// the total in lane 63.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1>(v);        // quad [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);        // quad [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);       // half-row mirror
  v += dpp_f64<0x140>(v);       // row mirror
  v += dpp_f64<0x142, 0xA>(v);  // lane 15 of each row to the next: rows 1 and 3
  v += dpp_f64<0x143, 0xC>(v);  // lane 31 to rows 2 and 3
  return lane_value(v, 63);
}

// C and its first and second derivatives (per px) at offset (ey, ex) from the
// integer peak, by one whole wave from the coefficients in LDS: lane m (mod
// 32) sums column m over the n of one parity (lanes 0-31 even, 32-63 odd),
// then over the columns.  T_{n+2} = w T_n - T_{n-2}, w = 2 T_2 = 4 x^2 - 2,
// and its derivatives.
__device__ Deriv window_eval(const double* c, double ey, double ex, double inv_b) {
  const int lane = threadIdx.x & 63, m = lane & 31, h = lane >> 5;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, tx0 = 0.0, tx1 = 0.0, tx2 = 0.0;
  auto chain = [](double x, int par, auto&& use) {
    const double w = 4.0 * x * x - 2.0, w1 = 8.0 * x;
    double t = par ? x : 1.0, u = par ? 1.0 : 0.0, v = 0.0;                     // T_n, T_n', T_n''
    double tp = par ? x : 0.5 * w, up = par ? 1.0 : 0.5 * w1, vp = par ? 0.0 : 4.0;  // at |n - 2|
#pragma unroll
    for (int k = 0; k < kChebN / 2; ++k) {
      use(k, t, u, v);
      const double tn = w * t - tp, un = w * u + (w1 * t - up);
      const double vn = w * v + (2.0 * w1 * u + (8.0 * t - vp));
      tp = t; up = u; vp = v;
      t = tn; u = un; v = vn;
    }
  };
  const int mc = m < kChebN ? m : 0;
  chain(ey * inv_b, h, [&](int k, double t, double u, double v) {
    const double cv = c[(2 * k + h) * kChebN + mc];
    s0 += cv * t;
    s1 += cv * u;
    s2 += cv * v;
  });
  chain(ex * inv_b, m & 1, [&](int k, double t, double u, double v) {
    const bool mine = 2 * k + (m & 1) == m;
    tx0 = mine ? t : tx0;
    tx1 = mine ? u : tx1;
    tx2 = mine ? v : tx2;
  });
  Deriv d;  // (lanes m >= 24 hold zero T)
  d.c = wave_sum(s0 * tx0);
  d.gy = wave_sum(s1 * tx0) * inv_b;
  d.gx = wave_sum(s0 * tx1) * inv_b;
  d.hyy = wave_sum(s2 * tx0) * inv_b * inv_b;
  d.hxy = wave_sum(s1 * tx1) * inv_b * inv_b;
  d.hxx = wave_sum(s0 * tx2) * inv_b * inv_b;
  return d;
}

// phi_k(s) and its first two derivatives (k~ signed; Nyquist cos(pi s)).
__device__ void phi_derivs(int k, int n, double s, double2* v) {
  double sn, cs;
  if (2 * k == n) {
    const double pi = 3.14159265358979323846;
    sincospi(s, &sn, &cs);
    v[0] = make_double2(cs, 0.0);
    v[1] = make_double2(-pi * sn, 0.0);
    v[2] = make_double2(-pi * pi * cs, 0.0);
    return;
  }
  const int kt = 2 * k < n ? k : k - n;
  const double a = 2.0 * 3.14159265358979323846 * kt / n;
  sincospi(2.0 * (double)kt * s / (double)n, &sn, &cs);
  v[0] = make_double2(cs, sn);
  v[1] = make_double2(-a * sn, a * cs);
  v[2] = make_double2(-a * a * cs, -a * a * sn);
}

// The same derivatives at any position s by the whole block, straight from
// the spectrum: for an iterate that has left the window of the series (a
// rejected or wandering Newton step; rare, so plain code).
template <typename CX>
__device__ __noinline__ Deriv direct_eval(const CX* __restrict__ Xf, int ny, int nx, double sy, double sx,
                             double (*red)[6]) {
  const int H = nx / 2 + 1;
  double a[6] = {0, 0, 0, 0, 0, 0};
  for (int i = threadIdx.x; i < ny * H; i += blockDim.x) {
    const int ky = i / H, kx = i - ky * H;
    double2 p[3], q[3];
    phi_derivs(ky, ny, sy, p);
    phi_derivs(kx, nx, sx, q);
    const double w = (kx == 0 || 2 * kx == nx) ? 1.0 : 2.0;
    const double xr = w * (double)Xf[i].x, xi = w * (double)Xf[i].y;
    auto term = [&](int o, int b) {  // Re[X phi_y^(o) phi_x^(b)]
      const double r = p[o].x * q[b].x - p[o].y * q[b].y, m = p[o].x * q[b].y + p[o].y * q[b].x;
      return xr * r - xi * m;
    };
    a[0] += term(0, 0);
    a[1] += term(1, 0);
    a[2] += term(0, 1);
    a[3] += term(2, 0);
    a[4] += term(1, 1);
    a[5] += term(0, 2);
  }
  const double inv = 1.0 / ((double)ny * (double)nx);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const double s = wave_sum(a[j]);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][j] = s;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    a[j] = 0.0;
    for (int w = 0; w < (int)blockDim.x / 64; ++w) a[j] += red[w][j];
  }
  return Deriv{a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv, a[4] * inv, a[5] * inv};
}

__device__ void write_special(ccpt_result* out, unsigned status) {
  ccpt_result r;
  r.reserved = 0;
  const double v = status == CCPT_ST_NONFINITE ? __builtin_nan("") : 0.0;
  r.d[0] = r.d[1] = v;
  r.peak = v;
  r.hess[0] = r.hess[1] = r.hess[2] = v;
  r.d_grid[0] = r.d_grid[1] = (float)v;
  r.p[0] = r.p[1] = 0;
  r.status = status;
  *out = r;
}

// The state a frame slot has between chunks (xcorr.hip sets it up).
__device__ void reset_state(FrameState* st) {
  FrameState z;
  z.peak_key = 0;
  z.grid_key = 0;
  z.second_key = 0;
  z.amin = 0xFFFFFFFFu;
  z.amax = 0;
  z.flags = 0;
  z.done = 0;
  *st = z;
}

constexpr int kMThreads = 256;

// 32 x 32 product over the grid's 16 terms, the lane's eight per operand in
// two float4 (terms 4 h .. 4 h + 3 and 8 + 4 h .. 8 + 4 h + 3, h = lane / 32);
// the high, small terms first.
__device__ __forceinline__ f32x16 grid_mma(float4 a0, float4 a1, float4 b0, float4 b1) {
  f32x16 u;
#pragma unroll
  for (int v = 0; v < 16; ++v) u[v] = 0.f;
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, b1.w, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, b1.z, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, b1.y, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, b1.x, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, b0.w, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, b0.z, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, b0.y, u, 0, 0, 0);
  u = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, b0.x, u, 0, 0, 0);
  return u;
}

// Rebuild radius and passes of the iteration (as the refinement is defined:
// an iterate farther than kModelRadius from the last centre starts another
// pass; steps are taken in the first kMaxPasses passes).
constexpr double kModelRadius = 0.02;  // px
constexpr int kMaxPasses = 3;

// Grid: one block of four waves per frame, or (few frames) nb blocks, each
// over its share of the 32-column strips of the grid, the last of them to
// finish going on to Newton.  A wave takes a strip: V[n][mx] =
// sum_m c[n][m] T_m(x_mx) in registers (16 terms: what they leave out is about
// 2 J_16(pi B) of the sum of |X|, 3e-12 at the paper's 1.5 px and 2.4e-10 at the
// widest window, below FP32), then U = T V row tile by row tile on 32x32x2 FP32
// matrix instructions (8 per 1024 grid points) with the running maximum per
// lane.  c is scaled by a power of two and its constant
// (the largest term, which moves no maximum) is dropped before the rounding
// to FP32.  The FP64 mode does the same with 24 terms on 16x16x4 FP64.
// The FP32 instance has 84 bytes of scratch a lane: one spilled register and the
// call of direct_eval.
// Bound by the serial chain of a frame (coefficients, grid, maximum, Newton's
// FP64 steps), not by the grid's matrix work (busy 0.24): 10,000 frames of 256 x
// 256, u = 100, in launches of 768 take 0.32 ms; one frame takes 14 us, against 26 us for the second half of
// the DFT and Newton before.
template <typename CX>
__global__ void __launch_bounds__(kMThreads, sizeof(CX) == sizeof(float2) ? 3 : 2)
    k_window_max(GroupParams g, WindowTables t, int ny, int nx, int nparts, int nb, double step_limit) {
  constexpr bool FP64 = sizeof(CX) != sizeof(float2);
  constexpr int NW = kMThreads / 64;
  __shared__ double c[kNC2];
  __shared__ double redd[NW][6];
  __shared__ unsigned long long redk[NW];
  __shared__ unsigned redi[NW];
  __shared__ double ctl[2];
  __shared__ int go;
  __shared__ unsigned cpk[2];  // FP64: integer peak, near tie
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f = blockIdx.y, part = blockIdx.x;
  const FrameState st = g.st[f];
  const FrameDesc d = g.desc[g.first + f];
  // the coefficients are requested with the state (a skipped frame's are
  // whatever the buffer holds, and unused), the parts in groups of up to
  // eight at a time, added in order
  constexpr int kPer = (kNC2 + kMThreads - 1) / kMThreads;
  double cv[kPer];
  {
    const double* src = g.coef + (size_t)f * nparts * kNC2;
#pragma unroll
    for (int e = 0; e < kPer; ++e) cv[e] = src[min(tid + e * kMThreads, kNC2 - 1)];
    for (int p0 = 1; p0 < nparts; p0 += 8) {
      double a[8][kPer];
#pragma unroll
      for (int p = 0; p < 8; ++p)
#pragma unroll
        for (int e = 0; e < kPer; ++e)
          a[p][e] = src[(size_t)min(p0 + p, nparts - 1) * kNC2 + min(tid + e * kMThreads, kNC2 - 1)];
#pragma unroll
      for (int p = 0; p < 8; ++p)
#pragma unroll
        for (int e = 0; e < kPer; ++e) cv[e] += p0 + p < nparts ? a[p][e] : 0.0;
    }
  }
  ccpt_result* out = g.out + d.out_idx;
  const int M = g.M;
  const bool tr = ny != nx && g.trans;
  if (frame_skipped(st)) {
    __syncthreads();  // every thread of the block has read the state
    if (tid == 0) {
      bool last = true;
      if (nb > 1) last = atomicAdd(&g.st[f].done, 1u) == (unsigned)nb - 1;
      if (last) {
        write_special(out, (st.flags & CCPT_ST_NONFINITE) ? CCPT_ST_NONFINITE : CCPT_ST_FLAT);
        reset_state(&g.st[f]);
      }
    }
    return;
  }
  // ---- coefficients into LDS, the parts in order
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int i = tid + e * kMThreads;
    if (i < kNC2) c[i] = cv[e];
  }
  if constexpr (FP64) {
    if (tid == 0) {
      bool tie;
      cpk[0] = peak_of_cands(g.cand + (size_t)f * g.ncand, g.ncand, tie);
      cpk[1] = tie ? CCPT_ST_NEAR_TIE : 0u;
    }
  }
  __syncthreads();
  unsigned best_idx;
  if constexpr (!FP64) {
    const int l32 = lane & 31, h = lane >> 5;
    // ---- scale: the largest coefficient but the constant to [0.5, 1) (every
    // wave finds it for itself)
    float4 c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0;
    {
      double big = 0.0;
#pragma unroll
      for (int e = 0; e < kNC2 / 64; ++e) {
        const int i = lane + 64 * e;
        big = fmax(big, i ? fabs(c[i]) : 0.0);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
      int ex = 0;
      if (big > 0.0 && big < __builtin_inf()) (void)frexp(big, &ex);
      // A operand of V: row n of c (rows 16.. of the 32-row product are zero)
      if (l32 < kGridN) {
        const double* r = c + l32 * kChebN + 4 * h;
        c0 = make_float4((float)ldexp(r[0], -ex), (float)ldexp(r[1], -ex), (float)ldexp(r[2], -ex),
                         (float)ldexp(r[3], -ex));
        c1 = make_float4((float)ldexp(r[8], -ex), (float)ldexp(r[9], -ex), (float)ldexp(r[10], -ex),
                         (float)ldexp(r[11], -ex));
        if (lane == 0) c0.x = 0.f;  // the constant
      }
    }
    // ---- 32 x 32 tiles of the grid, column strip by column strip; each wave
    // of the frame's blocks takes an equal run of them
    const int nt = (M + 31) / 32;
    const int nw = nb * NW, w0 = part * NW + wave;
    const int k1 = (int)((long)(w0 + 1) * nt * nt / nw);
    unsigned long long best = 0;
    float bv = -__builtin_inff();
    int br = 0;
    f32x16 vb;
    int k = (int)((long)w0 * nt * nt / nw), s = k / nt, r = k - s * nt;
    bool fresh = true;  // the strip's V is due
    // k step j of both products takes terms 8 (j / 4) + 4 h + j mod 4, which
    // is the row that register j of a 32x32 product holds in lane half h: V
    // comes out of the first product as the second's B operand
    const float* ta = t.tf + (size_t)l32 * kGridN + 4 * h;
    float4 t0, t1;  // A operand of the next tile: T(y) of rows 32 r + lane mod 32
    if (k < k1) {
      t0 = *(const float4*)(ta + (size_t)r * 32 * kGridN);
      t1 = *(const float4*)(ta + (size_t)r * 32 * kGridN + 8);
    }
    for (; k < k1; ++k) {
      if (fresh) {
        const float4 x0 = *(const float4*)(ta + (size_t)s * 32 * kGridN);
        const float4 x1 = *(const float4*)(ta + (size_t)s * 32 * kGridN + 8);
        vb = grid_mma(c0, c1, x0, x1);
        fresh = false;
      }
      const f32x16 u = grid_mma(t0, t1, make_float4(vb[0], vb[1], vb[2], vb[3]),
                                make_float4(vb[4], vb[5], vb[6], vb[7]));
      const int row0 = r * 32 + 4 * h, mx0 = s * 32 + l32;
      const bool whole = r * 32 + 32 <= M;
      if (++r == nt) {
        r = 0;
        ++s;
        fresh = true;
      }
      t0 = *(const float4*)(ta + (size_t)r * 32 * kGridN);
      t1 = *(const float4*)(ta + (size_t)r * 32 * kGridN + 8);
      // rows in increasing order within a lane: a strict compare keeps the
      // lowest of equal values, in either orientation of the frame
      if (whole) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const bool gt = u[v] > bv;
          bv = gt ? u[v] : bv;
          br = gt ? row0 + (v >> 2) * 8 + (v & 3) : br;
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int my = row0 + (v >> 2) * 8 + (v & 3);
          const bool gt = u[v] > bv && my < M;
          bv = gt ? u[v] : bv;
          br = gt ? my : br;
        }
      }
      if (fresh || k + 1 == k1) {  // the lane's column is done
        const unsigned long long key = peak_key(bv, grid_index(br, mx0, M, tr));
        if (mx0 < M && bv > -__builtin_inff()) best = key > best ? key : best;
        bv = -__builtin_inff();
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const unsigned long long w = __shfl_xor(best, o, 64);
      best = w > best ? w : best;
    }
    if (lane == 0) redk[wave] = best;
    __syncthreads();
    best = redk[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) best = redk[w] > best ? redk[w] : best;
    if (nb > 1) {
      // the blocks of a frame meet in its state; the last to arrive goes on
      if (tid == 0) {
        atomicMax(&g.st[f].grid_key, best);
        __threadfence();
        const bool last = atomicAdd(&g.st[f].done, 1u) == (unsigned)nb - 1;
        if (last) {
          __threadfence();
          redk[0] = atomicMax(&g.st[f].grid_key, 0ull);
        }
        go = last ? 1 : 0;
      }
      __syncthreads();
      if (!go) return;
      best = redk[0];
    }
    best_idx = best ? key_index(best) : 0xFFFFFFFFu;
  } else {
    const int l16 = lane & 15, l4 = lane >> 4;
    const int nt = (M + 15) / 16;
    double bv = -__builtin_inf();
    unsigned bi = 0xFFFFFFFFu;
    for (int s = wave; s < nt; s += NW) {
      const int mx0 = s * 16 + l16;
      const double* tx = t.td + (size_t)mx0 * kChebN;
      // V = c T(x): register v of the product's row tile h is its row n = 16 h
      // + 4 v + lane / 16, the B operand of k step 4 h + v below
      f64x4 va = {0.0, 0.0, 0.0, 0.0}, vc = va;
#pragma unroll
      for (int j = kChebN / 4 - 1; j >= 0; --j) {
        const int m = 4 * j + l4;
        const double b = tx[m];
        double a = c[l16 * kChebN + m];
        if (l16 == 0 && m == 0) a = 0.0;  // the constant dropped
        va = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, va, 0, 0, 0);
        a = l16 < kChebN - 16 ? c[min(16 + l16, kChebN - 1) * kChebN + m] : 0.0;
        vc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, vc, 0, 0, 0);
      }
      const double vb[kChebN / 4] = {va[0], va[1], va[2], va[3], vc[0], vc[1]};
      for (int r = 0; r < nt; ++r) {
        const double* ty = t.td + (size_t)(r * 16 + l16) * kChebN + l4;
        f64x4 u = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = kChebN / 4 - 1; j >= 0; --j)
          u = __builtin_amdgcn_mfma_f64_16x16x4f64(ty[4 * j], vb[j], u, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int my = r * 16 + 4 * v + l4;
          if (my < M && mx0 < M) {
            const unsigned i = (unsigned)(my * M + mx0);
            if (u[v] > bv || (u[v] == bv && i < bi)) {
              bv = u[v];
              bi = i;
            }
          }
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ov = __shfl_xor(bv, o, 64);
      const unsigned oi = (unsigned)__shfl_xor((int)bi, o, 64);
      if (ov > bv || (ov == bv && oi < bi)) {
        bv = ov;
        bi = oi;
      }
    }
    if (lane == 0) {
      redd[wave][0] = bv;
      redi[wave] = bi;
    }
    __syncthreads();
    bv = redd[0][0];
    bi = redi[0];
#pragma unroll
    for (int w = 1; w < NW; ++w)
      if (redd[w][0] > bv || (redd[w][0] == bv && redi[w] < bi)) {
        bv = redd[w][0];
        bi = redi[w];
      }
    best_idx = bi;
  }
  // every block of the frame has read the state: back to its initial value
  if (tid == 0) reset_state(&g.st[f]);

  // ---- seed
  int py, px;
  peak_at(FP64 ? cpk[0] : key_index(st.peak_key), ny, nx, g.trans && ny != nx, py, px);
  if (2 * py >= ny) py -= ny;
  if (2 * px >= nx) px -= nx;
  if (best_idx >= (unsigned)(M * M)) best_idx = (unsigned)(g.c * M + g.c);
  const int my = tr ? best_idx % M : best_idx / M, mx = tr ? best_idx / M : best_idx % M;
  const double dgy = py + (double)(my - g.c) / g.u, dgx = px + (double)(mx - g.c) / g.u;
  // near tie of the integer peak: from the FP64 reduction, or the two largest
  // FP32 keys
  unsigned status = FP64 ? cpk[1] : 0u;
  if (st.second_key && near_tie((double)key_value(st.peak_key), (double)key_value(st.second_key)))
    status |= CCPT_ST_NEAR_TIE;
  const CX* Xf = (FP64 ? (const CX*)g.X64 : (const CX*)g.X) + (size_t)f * ny * (nx / 2 + 1);

  // ---- Newton, by wave 0 (all its lanes hold the same values): one
  // evaluation per turn, each followed by a step or, when the position is
  // final, by the result.  The other waves wait, and help where an iterate
  // outside the series' window asks for a direct evaluation.
  double sy = dgy, sx = dgx, cy = dgy, cx = dgx;
  Deriv e{0, 0, 0, 0, 0, 0};
  bool have = false;  // e holds the direct evaluation at (sy, sx)
  int it_left = g.newton_iters, pass = 0;
  // the iterate is final: the window test applies to it whether or not it converged
  auto finish = [&]() {
    if (fmax(fabs(sy - py), fabs(sx - px)) > g.half_window) {
      status |= CCPT_ST_WINDOW_EXIT;
      sy = dgy;
      sx = dgx;
    }
  };
  bool last = it_left == 0;
  if (last) finish();
  __syncthreads();
  for (;;) {
    int ask = 0;
    if (wave == 0) {
      for (;;) {
        if (!have) {
          if (!(fmax(fabs(sy - py), fabs(sx - px)) <= t.half)) {
            ask = 1;
            break;
          }
          e = window_eval(c, sy - py, sx - px, 1.0 / t.half);
        }
        have = false;
        if (last) break;
        const double det = e.hyy * e.hxx - e.hxy * e.hxy;
        const double ty = -(e.hxx * e.gy - e.hxy * e.gx) / det;
        const double tx = -(e.hyy * e.gx - e.hxy * e.gy) / det;
        if (!(e.hyy < 0.0 && det > 0.0) || fmax(fabs(ty), fabs(tx)) > step_limit) {
          status |= CCPT_ST_NEWTON_FALLBACK;
          sy = dgy;
          sx = dgx;
          last = true;
        } else {
          sy += ty;
          sx += tx;
          --it_left;
          last = it_left == 0;
          if (!last && fmax(fabs(sy - cy), fabs(sx - cx)) > kModelRadius) {
            // another pass around this iterate, or out of passes
            last = pass >= kMaxPasses - 1;
            ++pass;
            cy = sy;
            cx = sx;
          }
        }
        if (last) finish();
      }
      if (lane == 0) {
        ctl[0] = sy;
        ctl[1] = sx;
        go = ask;
      }
    }
    __syncthreads();
    ask = go;
    const double ay = ctl[0], ax = ctl[1];
    __syncthreads();
    if (!ask) break;
    e = direct_eval<CX>(Xf, ny, nx, ay, ax, redd);
    have = true;
  }
  if (tid == 0) {
    // in the frame's own axes (a wide frame was processed transposed)
    const int a = tr ? 1 : 0, b = 1 - a;
    ccpt_result r;
    r.reserved = 0;
    r.d[a] = sy;
    r.d[b] = sx;
    r.peak = e.c;
    r.hess[2 * a] = e.hyy;
    r.hess[1] = e.hxy;
    r.hess[2 * b] = e.hxx;
    r.d_grid[a] = (float)dgy;
    r.d_grid[b] = (float)dgx;
    r.p[a] = py;
    r.p[b] = px;
    r.status = status;
    *out = r;
  }
}

// ------------------------------------------------------------------ launch
template <typename CX>
static int coef_x(int ny, int nx, const GroupParams& g, const WindowTables& t, int nparts, hipStream_t s) {
  const int ntile = (nx / 2 + 15) / 16;
  // (in FP64 two tiles a wave need 27 registers more than there are, 112 bytes of
  // scratch a lane; one tile needs none)
  // tiles per wave and waves per group: the split whose busiest wave has the
  // fewest k steps (the second contraction counts as four for each tile);
  // among equals two tiles at a time, which share the table values of a k step
  int tpw = 2, qs = 1, cost = 1 << 30;
  for (int p = 2; p >= 1; --p)
    for (int q = 1; q <= kCThreads / 64; q *= 2) {
      const int grp = (ntile + p - 1) / p, slots = kCThreads / 64 / q * nparts;
      const int c = (grp + slots - 1) / slots * p * ((t.ksteps + q - 1) / q + 4);
      if (c < cost) {
        cost = c;
        tpw = p;
        qs = q;
      }
    }
  const dim3 grid(nparts, g.count), block(kCThreads);
  if (tpw == 2)
    hipLaunchKernelGGL((k_window_coef<CX, 2>), grid, block, 0, s, g, t, ny, nx, qs);
  else
    hipLaunchKernelGGL((k_window_coef<CX, 1>), grid, block, 0, s, g, t, ny, nx, qs);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_window_coef(int ny, int nx, const GroupParams& g, const WindowTables& t, int nparts, hipStream_t s) {
  return g.X64 ? coef_x<double2>(ny, nx, g, t, nparts, s) : coef_x<float2>(ny, nx, g, t, nparts, s);
}

int launch_window_max(int ny, int nx, const GroupParams& g, const WindowTables& t, int nparts,
                      double step_limit, hipStream_t s) {
  // few frames: a frame's grid is spread over blocks (three tiles a wave) as
  // long as there are CUs without one
  const int strips = (g.M + 31) / 32;
  int nb = 1;
  if (!g.X64) nb = std::max(1, std::min((strips * strips + 11) / 12, 256 / std::max(1, g.count)));
  if (g.X64)
    hipLaunchKernelGGL((k_window_max<double2>), dim3(1, g.count), dim3(kMThreads), 0, s, g, t, ny, nx, nparts, 1,
                       step_limit);
  else
    hipLaunchKernelGGL((k_window_max<float2>), dim3(nb, g.count), dim3(kMThreads), 0, s, g, t, ny, nx, nparts, nb,
                       step_limit);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ccpt
