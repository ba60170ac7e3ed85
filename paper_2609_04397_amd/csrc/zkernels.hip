// gfx950 kernels of the reciprocal-space operator O(k) = sum_R e^{-2 pi i k.R} O(R)
// (paper, section 3.3, equation 4) and its complex products (section 3.2 and
// equation 1 with the conjugate transpose).
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "zkernels.hpp"

namespace vbcsr {
namespace {

template <typename T> struct C2;
template <> struct C2<double> { using type = double2; };
template <> struct C2<float> { using type = float2; };

__global__ void __launch_bounds__(kThreads) k_zphase(ZPhaseParams P) {
  const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (c >= P.n) return;
  const int32_t *R = P.shifts + 3 * (int64_t)P.image[c];
  double d0 = R[0], d1 = R[1], d2 = R[2];
  if (P.tau) {
    const double *tj = P.tau + 3 * (int64_t)P.col_idx[c];
    const double *ti = P.tau + 3 * (int64_t)P.blk_row[c];
    d0 += tj[0] - ti[0];
    d1 += tj[1] - ti[1];
    d2 += tj[2] - ti[2];
  }
  const double th = -2.0 * M_PI * (P.k[0] * d0 + P.k[1] * d1 + P.k[2] * d2);
  double sn, cs;
  sincos(th, &sn, &cs);
  P.ph[2 * c] = cs;
  P.ph[2 * c + 1] = sn;
}

// Values in flight per lane in the sampling kernel.
constexpr int kSampleBatch = 8;

// The wave's blocks are kb0 .. kb0 + nb - 1, their values numbered 0 .. T-1
// in graph order; lane l takes values l, l + 64, ... in batches whose value
// and phase loads are all issued before the first use.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_zsample(ZSampleParams P, T *fwd, T *tr) {
  using V2 = typename C2<T>::type;
  const int64_t kb0 = ((int64_t)blockIdx.x * kWaves + wave_id()) * kSampleBlocks;
  if (kb0 >= P.nkb) return;
  const int lane = threadIdx.x & 63;
  const int nb = (int)min((int64_t)kSampleBlocks, P.nkb - kb0);
  // lane j < nb holds block kb0 + j; lane nb reads the end of the last block
  int d = 0, cnt = 0;
  int64_t base = 0, vb = 0, c0 = 0, fp = 0, tp = 0;
  if (lane <= nb) base = P.kbase[kb0 + lane];
  if (lane < nb) {
    const int64_t kb = kb0 + lane;
    d = P.kdim[kb];
    c0 = P.cptr[kb];
    cnt = (int)(P.cptr[kb + 1] - c0);
    vb = P.kvbase[kb];
    fp = P.fwd_pos[kb];
    tp = P.tr_pos[kb];
  }
  const int rel = (int)(base - __shfl(base, 0));  // value offset of lane j's block
  const int total = __builtin_amdgcn_readlane(rel, nb);
  int start[kSampleBlocks];
#pragma unroll
  for (int k = 0; k < kSampleBlocks; ++k)
    start[k] = k <= nb ? __builtin_amdgcn_readlane(rel, k) : total;
  const double2 *ph = reinterpret_cast<const double2 *>(P.ph);
  for (int v0 = 0; v0 < total; v0 += 64 * kSampleBatch) {
    double x[kSampleBatch];
    double2 w[kSampleBatch];
    int jv[kSampleBatch], ev[kSampleBatch];
#pragma unroll
    for (int u = 0; u < kSampleBatch; ++u) {
      const int v = v0 + 64 * u + lane;
      int j = 0;
#pragma unroll
      for (int k = 1; k < kSampleBlocks; ++k) j += start[k] <= v ? 1 : 0;
      jv[u] = j;
      ev[u] = v - __shfl(rel, j);
      const int64_t vbj = __shfl(vb, j), c0j = __shfl(c0, j);
      x[u] = 0.0;
      w[u] = make_double2(0.0, 0.0);
      if (v < total) {
        x[u] = P.values[vbj + ev[u]];
        w[u] = ph[c0j];
      }
    }
#pragma unroll
    for (int u = 0; u < kSampleBatch; ++u) {
      const int v = v0 + 64 * u + lane, j = jv[u], e = ev[u];
      const int dj = __shfl(d, j), cj = __shfl(cnt, j);
      const int64_t c0j = __shfl(c0, j), fj = __shfl(fp, j), tj = __shfl(tp, j);
      if (v >= total) continue;
      double re = x[u] * w[u].x, im = x[u] * w[u].y;
      for (int64_t c = c0j + 1; c < c0j + cj; ++c) {  // further images of the block
        const double y = P.values[P.cgbase[c] + e];
        const double2 z = ph[c];
        re = fma(y, z.x, re);
        im = fma(y, z.y, im);
      }
      const int bi = dj & 0xffff, bj = dj >> 16;
      const int p = e / bj, q = e - p * bj;
      V2 o;
      o.x = (T)re;
      o.y = (T)im;
      *reinterpret_cast<V2 *>(fwd + 2 * (fj + (int64_t)q * bi + p)) = o;  // column-major
      o.y = (T)(-im);
      *reinterpret_cast<V2 *>(tr + 2 * (tj + (int64_t)e)) = o;  // row-major (= A^H column-major)
    }
  }
}

// One wave per panel (block row of op(O)): lane (g, p) takes panel row p and
// the panel columns k = g, g + G, ... (G = floor(64 / b) groups), NR
// right-hand sides per pass; groups are reduced by shuffles.  Every complex
// product is four FMAs in T.
template <typename T, int NR>
__global__ void __launch_bounds__(kThreads) k_zspmm(ZSpmmParams<T> P) {
  using V = typename C2<T>::type;
  const int row = xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (row >= P.nrows) return;
  const int lane = threadIdx.x & 63;
  const RowDesc rd = P.rows[row];
  const int b = rd.b, K = rd.K;
  const int G = 64 / b;
  const int g = lane / b, p = lane - g * b;
  const bool act = g < G;
  const V *__restrict__ A = reinterpret_cast<const V *>(P.pages) + rd.vbase;
  const int32_t *__restrict__ cx = P.colx + rd.cbase;
  const V *__restrict__ X = reinterpret_cast<const V *>(P.X);
  V *__restrict__ Y = reinterpret_cast<V *>(P.Y);
  for (int c0 = 0; c0 < P.nrhs; c0 += NR) {
    T re[NR], im[NR];
#pragma unroll
    for (int c = 0; c < NR; ++c) re[c] = im[c] = T(0);
    if (act && g < K) {
      // the operands of column k + G are in flight while column k
      // multiplies; the index is clamped to the last column (no branch
      // around the loads), the clamped copy is never multiplied
      const int nc = min(NR, P.nrhs - c0);
      V a = A[(int64_t)g * b + p];
      V x[NR];
      {
        const V *xr = X + (int64_t)cx[g] * P.ldx + c0;
#pragma unroll
        for (int c = 0; c < NR; ++c) x[c] = xr[min(c, nc - 1)];
      }
      for (int k = g; k < K; k += G) {
        const int kn = min(k + G, K - 1);
        const V an = A[(int64_t)kn * b + p];
        const V *xn = X + (int64_t)cx[kn] * P.ldx + c0;
        V xv[NR];
#pragma unroll
        for (int c = 0; c < NR; ++c) xv[c] = xn[min(c, nc - 1)];
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          re[c] = fma(a.x, x[c].x, re[c]);
          re[c] = fma(-a.y, x[c].y, re[c]);
          im[c] = fma(a.x, x[c].y, im[c]);
          im[c] = fma(a.y, x[c].x, im[c]);
        }
        a = an;
#pragma unroll
        for (int c = 0; c < NR; ++c) x[c] = xv[c];
      }
    }
    for (int st = 1; st < G; st <<= 1) {
#pragma unroll
      for (int c = 0; c < NR; ++c) {
        const T orr = __shfl_down(re[c], st * b, 64);
        const T oi = __shfl_down(im[c], st * b, 64);
        if (act && (g & (2 * st - 1)) == 0 && g + st < G) {
          re[c] += orr;
          im[c] += oi;
        }
      }
    }
    if (lane < b) {
      V *yr = Y + (int64_t)(rd.yrow + p) * P.ldy + c0;
#pragma unroll
      for (int c = 0; c < NR; ++c) {
        if (c0 + c < P.nrhs) {
          const double sr = re[c], si = im[c];
          double yr_ = P.ar * sr - P.ai * si, yi_ = P.ar * si + P.ai * sr;
          if (P.br != 0.0 || P.bi != 0.0) {
            const V y = yr[c];
            yr_ += P.br * (double)y.x - P.bi * (double)y.y;
            yi_ += P.br * (double)y.y + P.bi * (double)y.x;
          }
          V o;
          o.x = (T)yr_;
          o.y = (T)yi_;
          yr[c] = o;
        }
      }
    }
  }
}

typedef double v4d __attribute__((ext_vector_type(4)));

// One complex value in one load, widened to FP64.
template <typename T> __device__ __forceinline__ double2 zload(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <> __device__ __forceinline__ double2 zload<double>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
template <> __device__ __forceinline__ double2 zload<float>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  return double2{(double)v.x, (double)v.y};
}

// y = alpha s + beta y for one complex element (y unread when beta is 0).
template <typename T>
__device__ __forceinline__ void zstore(const ZSpmmParams<T> &P, int64_t r, int c, double sr, double si) {
  using V = typename C2<T>::type;
  V *yp = reinterpret_cast<V *>(P.Y) + r * P.ldy + c;
  double yr = P.ar * sr - P.ai * si, yi = P.ar * si + P.ai * sr;
  if (P.br != 0.0 || P.bi != 0.0) {
    const V y = *yp;
    yr += P.br * (double)y.x - P.bi * (double)y.y;
    yi += P.br * (double)y.y + P.bi * (double)y.x;
  }
  V o;
  o.x = (T)yr;
  o.y = (T)yi;
  *yp = o;
}

// Complex product on small FP64 matrix-core tiles, 4 NG right-hand sides per
// pass: the four 4x4 blocks of v_mfma_f64_4x4x4 take 4 panel rows x 4 panel
// columns each (a step is 16 columns), so rows pad to 4 only.  Lane
// 16 k + 4 q + i works on column 4 k + q and on row i of a row group (values)
// or right-hand side i of a group (X); one load brings one complex value.
// Four real products per complex one go to two accumulators (the imaginary
// part of the value enters the real one negated); FP32 pages and vectors are
// widened on load and accumulate in FP64.  PARTS (FP64 below 16 right-hand
// sides): each step is summed from zero and added to the total once.  With one
// chain per block the rounding error was 1.4 times that of the vector kernel,
// which splits a row over up to 64 lanes (b = 1/4/9: 4.4e-16 of the result
// against 3.2e-16, now 2.0e-16), and from 16 on it is below that of 16-row
// tiles without (4.4e-16 against 6.2e-16).  A ring of R register sets: the
// next R - 1 steps are in flight, their indices R further ahead; an index is
// compared with the panel's end where it is used (at the load it would be
// waited for).  The blocks' partial sums meet once per panel.
// Bound by the load path (16 cycles of a compute unit per load): O(k) of the
// b = 1/4/9 cube of 20 000 atoms, 16 right-hand sides, 103 us against 163 us
// with 16-row tiles, whose matrix work was mostly padding; R = 3 110 us.
template <typename T, int RG, int NG, int R, bool PARTS>
__device__ __forceinline__ void zsmall_rows(const ZSpmmParams<T> &P, const RowDesc &rd, int m0, int c0,
                                            uint32_t xbytes) {
  constexpr uint32_t ES = 2 * sizeof(T);
  const int lane = threadIdx.x & 63;
  const int ij = lane & 3;
  const int col = 4 * (lane >> 4) + ((lane >> 2) & 3);
  const int b = rd.b, K = rd.K;
  const __amdgpu_buffer_rsrc_t ra = panel_rsrc(P.pages + 2 * rd.vbase, (uint32_t)K * (uint32_t)b * ES);
  const __amdgpu_buffer_rsrc_t rc = panel_rsrc(P.colx + rd.cbase, (uint32_t)K * 4u);
  const __amdgpu_buffer_rsrc_t rx = panel_rsrc(P.X, xbytes);
  double re[RG][NG], im[RG][NG];
#pragma unroll
  for (int g = 0; g < RG; ++g)
#pragma unroll
    for (int t = 0; t < NG; ++t) re[g][t] = im[g][t] = 0.0;
  const uint32_t vo = (uint32_t)(col * b + m0 + ij) * ES, vstep = (uint32_t)(16 * b) * ES;
  uint32_t xcol[NG];
#pragma unroll
  for (int t = 0; t < NG; ++t) {
    const int c = c0 + 4 * t + ij;
    xcol[t] = c < P.nrhs ? (uint32_t)c * ES : kOutCol;
  }
  auto ld_idx = [&](int s) {
    return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(16 * s + col) * 4, 0, 0);
  };
  auto ld = [&](int s, int32_t xi, double2 (&a)[RG], double2 (&x)[NG]) {
    const uint32_t ro =
        16 * s + col < K ? (uint32_t)((int64_t)xi * P.ldx * (int64_t)ES) : kOutRow;
#pragma unroll
    for (int t = 0; t < NG; ++t) x[t] = zload<T>(rx, ro + xcol[t]);
    // rows past the panel read the next column's values into sums that are
    // never stored
#pragma unroll
    for (int g = 0; g < RG; ++g) a[g] = zload<T>(ra, vo + (uint32_t)s * vstep + 4u * ES * g);
  };
  auto mma = [&](const double2 (&a)[RG], const double2 (&x)[NG]) {
    if constexpr (PARTS) {
      // added one row group behind the matrix instructions that form them
      double pr[2][NG], pi[2][NG];
#pragma unroll
      for (int g = 0; g <= RG; ++g) {
        if (g < RG) {
          const double n = -a[g % RG].y;
#pragma unroll
          for (int t = 0; t < NG; ++t) {
            pr[g & 1][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g % RG].x, x[t].x, 0.0, 0, 0, 0);
            pi[g & 1][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g % RG].x, x[t].y, 0.0, 0, 0, 0);
          }
#pragma unroll
          for (int t = 0; t < NG; ++t) {
            pr[g & 1][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(n, x[t].y, pr[g & 1][t], 0, 0, 0);
            pi[g & 1][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g % RG].y, x[t].x, pi[g & 1][t], 0, 0, 0);
          }
        }
        if (g > 0) {
#pragma unroll
          for (int t = 0; t < NG; ++t) {
            re[g - 1][t] += pr[(g - 1) & 1][t];
            im[g - 1][t] += pi[(g - 1) & 1][t];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int t = 0; t < NG; ++t) {
        re[g][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g].x, x[t].x, re[g][t], 0, 0, 0);
        im[g][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g].x, x[t].y, im[g][t], 0, 0, 0);
      }
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      const double n = -a[g].y;
#pragma unroll
      for (int t = 0; t < NG; ++t) {
        re[g][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(n, x[t].y, re[g][t], 0, 0, 0);
        im[g][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g].y, x[t].x, im[g][t], 0, 0, 0);
      }
    }
  };
  const int ns = (K + 15) >> 4;
  double2 av[R][RG], xv[R][NG];
  int32_t xi[R];
#pragma unroll
  for (int r = 0; r < R; ++r) xi[r] = ld_idx(r);
#pragma unroll
  for (int r = 0; r + 1 < R; ++r) {
    ld(r, xi[r], av[r], xv[r]);
    xi[r] = ld_idx(r + R);
  }
  __builtin_amdgcn_sched_barrier(0);
  int s = 0;
  for (; s + R <= ns; s += R) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int q = (r + R - 1) % R;
      ld(s + r + R - 1, xi[q], av[q], xv[q]);
      xi[q] = ld_idx(s + r + 2 * R - 1);
      __builtin_amdgcn_sched_barrier(0);
      mma(av[r], xv[r]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int r = 0; r + 1 < R; ++r)
    if (s + r < ns) mma(av[r], xv[r]);
  // lane 16 i + 4 g + j writes row 4 g + i, right-hand sides j of each group
  const int gl = (lane >> 2) & 3;
  const int prow = m0 + 4 * gl + (lane >> 4);
#pragma unroll
  for (int t = 0; t < NG; ++t) {
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      double u = re[g][t], v = im[g][t];
      u += __shfl_xor(u, 4, 64);
      u += __shfl_xor(u, 8, 64);
      v += __shfl_xor(v, 4, 64);
      v += __shfl_xor(v, 8, 64);
      sr = gl == g ? u : sr;
      si = gl == g ? v : si;
    }
    const int c = c0 + 4 * t + ij;
    if (gl < RG && prow < b && c < P.nrhs) zstore(P, (int64_t)rd.yrow + prow, c, sr, si);
  }
}

template <typename T, int NG, int R, bool PARTS>
__global__ void __launch_bounds__(kThreads) k_zspmm_small(ZSpmmParams<T> P, uint32_t xbytes) {
  const int row = xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (row >= P.nrows) return;
  const RowDesc rd = P.rows[row];
  for (int c0 = 0; c0 < P.nrhs; c0 += 4 * NG)
    for (int m0 = 0; m0 < rd.b; m0 += 16) {
      switch ((min(rd.b - m0, 16) + 3) >> 2) {
        case 1: zsmall_rows<T, 1, NG, R, PARTS>(P, rd, m0, c0, xbytes); break;
        case 2: zsmall_rows<T, 2, NG, R, PARTS>(P, rd, m0, c0, xbytes); break;
        case 3: zsmall_rows<T, 3, NG, R, PARTS>(P, rd, m0, c0, xbytes); break;
        default: zsmall_rows<T, 4, NG, R, PARTS>(P, rd, m0, c0, xbytes); break;
      }
    }
}

// Complex product on 16x16x4 FP64 matrix cores, for more than 16 right-hand
// sides: one wave per panel, M = panel rows in tiles of 16, K = panel columns
// in slices of 4, N = 16 right-hand sides per tile, NT tiles per pass.  Lane
// (m, kq) loads 16 bytes of A (row m, column 4s + kq: one complex value) and,
// per tile, 16 bytes of X; ring and padding as above.  Each of the four real
// products has an accumulator of its own: with two, whose chains are twice as
// long, the rounding error was 1.4 times larger (b = 9..20: 1.41e-15 against
// 0.99e-15 of the result) at the same speed (b = 13, 32 right-hand sides 297
// us with two, 298 with four; b = 9..20 493 and 472).
template <int NT, int R>
__global__ void __launch_bounds__(kThreads) k_zspmm_mfma(ZSpmmParams<double> P, uint32_t xbytes) {
  const int row = xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (row >= P.nrows) return;
  const int lane = threadIdx.x & 63;
  const int m = lane & 15, kq = lane >> 4;
  const RowDesc rd = P.rows[row];
  const int b = rd.b, K = rd.K;
  const __amdgpu_buffer_rsrc_t ra = panel_rsrc(P.pages + 2 * rd.vbase, (uint32_t)K * (uint32_t)b * 16u);
  const __amdgpu_buffer_rsrc_t rc = panel_rsrc(P.colx + rd.cbase, (uint32_t)K * 4u);
  const __amdgpu_buffer_rsrc_t rx = panel_rsrc(P.X, xbytes);
  const int nsl = (K + 3) >> 2;
  for (int mt = 0; mt * 16 < b; ++mt) {
    const uint32_t vo = (uint32_t)(kq * b + mt * 16 + m) * 16u, vstep = (uint32_t)(4 * b) * 16u;
    for (int c0 = 0; c0 < P.nrhs; c0 += 16 * NT) {
      v4d re[NT], im[NT], ii[NT], ir[NT];
      uint32_t xcol[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        re[t] = im[t] = ii[t] = ir[t] = v4d{0.0, 0.0, 0.0, 0.0};
        const int c = c0 + 16 * t + m;
        xcol[t] = c < P.nrhs ? (uint32_t)c * 16u : kOutCol;
      }
      auto ld_idx = [&](int s) {
        return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(4 * s + kq) * 4, 0, 0);
      };
      auto ld = [&](int s, int32_t xi, double2 &a, double2 (&x)[NT]) {
        const uint32_t ro = 4 * s + kq < K ? (uint32_t)((int64_t)xi * P.ldx * 16) : kOutRow;
#pragma unroll
        for (int t = 0; t < NT; ++t) x[t] = zload<double>(rx, ro + xcol[t]);
        a = zload<double>(ra, vo + (uint32_t)s * vstep);
      };
      auto mma = [&](const double2 &a, const double2 (&x)[NT]) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          re[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, x[t].x, re[t], 0, 0, 0);
          ii[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, x[t].y, ii[t], 0, 0, 0);
          im[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, x[t].y, im[t], 0, 0, 0);
          ir[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, x[t].x, ir[t], 0, 0, 0);
        }
      };
      double2 av[R], xv[R][NT];
      int32_t xi[R];
#pragma unroll
      for (int r = 0; r < R; ++r) xi[r] = ld_idx(r);
#pragma unroll
      for (int r = 0; r + 1 < R; ++r) {
        ld(r, xi[r], av[r], xv[r]);
        xi[r] = ld_idx(r + R);
      }
      __builtin_amdgcn_sched_barrier(0);
      int s = 0;
      for (; s + R <= nsl; s += R) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int q = (r + R - 1) % R;
          ld(s + r + R - 1, xi[q], av[q], xv[q]);
          xi[q] = ld_idx(s + r + 2 * R - 1);
          __builtin_amdgcn_sched_barrier(0);
          mma(av[r], xv[r]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int r = 0; r + 1 < R; ++r)
        if (s + r < nsl) mma(av[r], xv[r]);
      // accumulator element e of quarter-wave kq: tile row kq + 4e, column m
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int c = c0 + t * 16 + m;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = mt * 16 + kq + 4 * e;
          if (r < b && c < P.nrhs) zstore(P, (int64_t)rd.yrow + r, c, re[t][e] - ii[t][e], im[t][e] + ir[t][e]);
        }
      }
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_zunpack(const T *fwd, const int64_t *pos,
                                                      const int32_t *krow, const int32_t *kcol,
                                                      const int32_t *b, const int64_t *kbase,
                                                      int64_t nkb, T *dst) {
  const int64_t kb = (int64_t)blockIdx.x * kWaves + wave_id();
  if (kb >= nkb) return;
  const int lane = threadIdx.x & 63;
  const int bi = b[krow[kb]], bj = b[kcol[kb]];
  const T *f = fwd + 2 * pos[kb];
  T *d = dst + 2 * kbase[kb];
  for (int e = lane; e < bi * bj; e += 64) {
    const int p = e / bj, q = e - p * bj;
    d[2 * e] = f[2 * ((int64_t)q * bi + p)];
    d[2 * e + 1] = f[2 * ((int64_t)q * bi + p) + 1];
  }
}

template <typename T>
hipError_t launch_zspmm_t(const ZSpmmParams<T> &p, hipStream_t s) {
  if (p.nrows == 0) return hipSuccess;
  const dim3 grid((unsigned)((p.nrows + kWaves - 1) / kWaves));
  // right-hand sides per pass: every pass streams the pages once more
  if (p.nrhs == 1)
    hipLaunchKernelGGL((k_zspmm<T, 1>), grid, dim3(kThreads), 0, s, p);
  else if (p.nrhs == 2)
    hipLaunchKernelGGL((k_zspmm<T, 2>), grid, dim3(kThreads), 0, s, p);
  else if (p.nrhs <= 4)
    hipLaunchKernelGGL((k_zspmm<T, 4>), grid, dim3(kThreads), 0, s, p);
  else if (p.nrhs <= 8)
    hipLaunchKernelGGL((k_zspmm<T, 8>), grid, dim3(kThreads), 0, s, p);
  else
    hipLaunchKernelGGL((k_zspmm<T, 16>), grid, dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_zphase(const ZPhaseParams &p, hipStream_t s) {
  if (p.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zphase, dim3((unsigned)((p.n + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_zsample(const ZSampleParams &p, void *fwd, void *tr, int elem_bytes,
                          hipStream_t s) {
  if (p.nkb == 0) return hipSuccess;
  const int64_t waves = (p.nkb + kSampleBlocks - 1) / kSampleBlocks;
  const dim3 grid((unsigned)((waves + kWaves - 1) / kWaves));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_zsample<double>, grid, dim3(kThreads), 0, s, p,
                       static_cast<double *>(fwd), static_cast<double *>(tr));
  else
    hipLaunchKernelGGL(k_zsample<float>, grid, dim3(kThreads), 0, s, p,
                       static_cast<float *>(fwd), static_cast<float *>(tr));
  return hipGetLastError();
}

// Matrix cores when X spans less than one buffer descriptor (kXSpan), else
// the vector kernel with 64-bit addresses.  Small tiles for operators of any but
// the smallest blocks up to 16 right-hand sides and in FP32 (vector kernel
// against small tiles, O(k) of the b = 1/4/9 cube of 20 000 atoms, FP64: 53
// against 43 us at 1, 78/49 at 4, 195/70 at 8; FP32 42/38 at 1, 99/57 at 8,
// 197/98 at 16, 387/182 at 32; 16-row tiles against small tiles, FP64 at 16:
// 163/103).  FP64 beyond 16: small
// tiles where 16-row tiles pad much (b = 1/4/9, ratio 1.9: 204 us against 162
// at 24, 386/239 at 40, 388/330 at 64), 16-row tiles where they pad less
// (b = 9/20, ratio 1.4: 316 against 331 at 20, 331/364 at 32, 591/787 at 64).
template <typename T>
hipError_t launch_zspmm_any(const ZSpmmParams<T> &p, hipStream_t s) {
  const int64_t xbytes = (((int64_t)p.xrows - 1) * p.ldx + p.nrhs) * 2 * (int64_t)sizeof(T);
  // The vector kernel too where a small tile of 4 rows is mostly padding (mean
  // panel height of 2 or 3) and few right-hand sides leave it the value stream
  // alone; us on it and on small tiles, operators of one size: FP32, 1
  // right-hand side, b = 1 39/68, b = 3 47/60; 2, b = 1 45/67, b = 3 52/59; 4,
  // b = 1 63/66, b = 2 59/63, b = 3 74/59; FP64, 1, b = 1 44/57, b = 3 80/83;
  // 2, b = 2 55/62, b = 3 91/87; 4, b = 1 105/56.
  constexpr bool kF64 = sizeof(T) == 8;
  const double flat = p.nrhs == 1   ? 3.0
                      : p.nrhs == 2 ? (kF64 ? 2.0 : 3.0)
                      : p.nrhs <= 4 ? (kF64 ? 0.0 : 2.0)
                                    : 0.0;
  if (p.nrows == 0 || xbytes >= kXSpan || p.height <= flat) return launch_zspmm_t(p, s);
  const dim3 grid((unsigned)((p.nrows + kWaves - 1) / kWaves));
  const uint32_t xb = (uint32_t)xbytes;
  if constexpr (sizeof(T) == 8) {
    if (p.nrhs > 16 && p.pad16 <= 1.6) {
      if (p.nrhs <= 32)
        hipLaunchKernelGGL((k_zspmm_mfma<2, 4>), grid, dim3(kThreads), 0, s, p, xb);
      else
        hipLaunchKernelGGL((k_zspmm_mfma<4, 2>), grid, dim3(kThreads), 0, s, p, xb);
      return hipGetLastError();
    }
  }
  if (p.nrhs <= 4)
    hipLaunchKernelGGL((k_zspmm_small<T, 1, 2, kF64>), grid, dim3(kThreads), 0, s, p, xb);
  else if (p.nrhs <= 8)
    hipLaunchKernelGGL((k_zspmm_small<T, 2, 2, kF64>), grid, dim3(kThreads), 0, s, p, xb);
  else if (kF64 && p.nrhs <= 12)
    hipLaunchKernelGGL((k_zspmm_small<T, 3, 2, kF64>), grid, dim3(kThreads), 0, s, p, xb);
  else if (kF64 && p.nrhs < 16)
    hipLaunchKernelGGL((k_zspmm_small<T, 4, 2, kF64>), grid, dim3(kThreads), 0, s, p, xb);
  else
    hipLaunchKernelGGL((k_zspmm_small<T, 4, 2, false>), grid, dim3(kThreads), 0, s, p, xb);
  return hipGetLastError();
}

hipError_t launch_zspmm_f64(const ZSpmmParams<double> &p, hipStream_t s) {
  return launch_zspmm_any(p, s);
}
hipError_t launch_zspmm_f32(const ZSpmmParams<float> &p, hipStream_t s) {
  return launch_zspmm_any(p, s);
}

hipError_t launch_zunpack(const void *fwd, int elem_bytes, const int64_t *pos,
                          const int32_t *krow, const int32_t *kcol, const int32_t *b,
                          const int64_t *kbase, int64_t nkb, void *dst, hipStream_t s) {
  if (nkb == 0) return hipSuccess;
  const dim3 grid((unsigned)((nkb + kWaves - 1) / kWaves));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_zunpack<double>, grid, dim3(kThreads), 0, s,
                       static_cast<const double *>(fwd), pos, krow, kcol, b, kbase, nkb,
                       static_cast<double *>(dst));
  else
    hipLaunchKernelGGL(k_zunpack<float>, grid, dim3(kThreads), 0, s,
                       static_cast<const float *>(fwd), pos, krow, kcol, b, kbase, nkb,
                       static_cast<float *>(dst));
  return hipGetLastError();
}

}  // namespace vbcsr
