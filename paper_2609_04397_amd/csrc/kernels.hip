// gfx950 (CDNA4) kernels of the variable-block sparse library.
//
// Products run one 64-lane wave per panel (block row of A, or of A^T for the
// adjoint).  Panels are column-major b x K, so a run of consecutive panel
// values is a sequence of whole columns.  Two kernel families cover the
// forward product Y_i = sum_j A_ij X_j (paper, section 3.2):
//
//  * vector FMA (few right-hand sides): lane (g, p) owns panel row p of
//    column group g; with G = 64 / b groups, load step s reads the G*b
//    consecutive values [s*G*b, (s+1)*G*b) -- one contiguous wave access for
//    any block size -- and multiplies each by the X row of its column.
//    Partial sums of one panel row meet by a tree of cross-lane shuffles.
//  * matrix cores (many right-hand sides): the panel is the A operand of
//    16x16x4 FP64/FP32 MFMA (M = panel rows padded to 16 in registers only,
//    K = panel columns, N = 16 right-hand sides per tile); its 4-column slices
//    are again contiguous in memory.  FP64 products of few right-hand sides or
//    much row padding use 4x4x4 tiles.  The BF16x3 form uses 16x16x32 BF16 MFMA
//    on pages stored in 8-column groups (8 consecutive columns of one panel
//    row are 16 contiguous bytes, the per-lane A fragment).
//
// Every output element has exactly one writer (no atomics), so results are
// bitwise reproducible run to run.
#include <mutex>
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace vbcsr {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short v8u __attribute__((ext_vector_type(8)));
typedef unsigned int v4u32 __attribute__((ext_vector_type(4)));
typedef unsigned int v2u32 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma_bf16(v8u a, v8u b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                 __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

template <typename T> struct Frag;
template <> struct Frag<double> { using type = v4d; };
template <> struct Frag<float> { using type = v4f; };

// Output row (within the 16x16 tile) of accumulator element i of the lanes
// in quarter-wave kq.  The FP32 and BF16 16x16 tiles give each quarter-wave
// four consecutive rows; the FP64 16x16x4 tile interleaves them with stride 4
// (lane layout measured on gfx950).
template <typename T> __device__ __forceinline__ int dst_row(int kq, int i);
template <> __device__ __forceinline__ int dst_row<double>(int kq, int i) { return kq + 4 * i; }
template <> __device__ __forceinline__ int dst_row<float>(int kq, int i) { return 4 * kq + i; }

// Round-to-nearest-even FP32 -> BF16 (finite inputs) and back.
__device__ __forceinline__ unsigned short bf16_rne(float f) {
  unsigned int u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(unsigned short h) {
  return __uint_as_float(((unsigned int)h) << 16);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <bool MOM>
__device__ __forceinline__ void mom_init(double *s_mom, int nrhs) {
  if (MOM) {
    for (int c = threadIdx.x; c < kWaves * nrhs; c += kThreads) s_mom[c] = 0.0;
    __syncthreads();
  }
}

template <bool MOM>
__device__ __forceinline__ void mom_flush(const double *s_mom, int nrhs, int wg, double *out) {
  if (MOM) {
    __syncthreads();
    for (int c = threadIdx.x; c < nrhs; c += kThreads) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) t += s_mom[w * nrhs + c];
      out[(int64_t)wg * nrhs + c] = t;
    }
  }
}

// Wave-private LDS hand-off (LDS writes of a wave become visible to its
// own later LDS reads; no workgroup barrier needed).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Panel values are read exactly once per product: stream them past the
// caches (non-temporal) so the gathered X rows stay resident.
template <typename T>
__device__ __forceinline__ T stream_load(const T *p) {
  return __builtin_nontemporal_load(p);
}

template <typename T> __device__ __forceinline__ T buf_load_nt(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <> __device__ __forceinline__ double buf_load_nt<double>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 2));
}
template <> __device__ __forceinline__ float buf_load_nt<float>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2));
}
template <typename T> __device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <> __device__ __forceinline__ double buf_load<double>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <> __device__ __forceinline__ float buf_load<float>(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// Bytes from X's first element to its last (XB kernels: below kXSpan).
template <typename T> __device__ __forceinline__ uint32_t x_span(const FwdParams<T> &P) {
  return P.xrows > 0
             ? (uint32_t)(((P.xrows - 1) * P.ldx + P.nrhs) * (int64_t)sizeof(T))
             : 0u;
}

// Value of lane 16 q + U of the caller's 16-lane row q, to the whole row.
template <int U>
__device__ __forceinline__ int32_t row_bcast(int32_t v) {
  // 0x150 + n: row_newbcast of the gfx9 data-parallel primitives
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + U, 0xF, 0xF, false);
}

// Value of lane 4 q + u of the caller's four lanes q to all of them (u constant).
__device__ __forceinline__ int32_t quad_bcast(int32_t v, int u) {
  switch (u) {
    case 0: return __builtin_amdgcn_update_dpp(0, v, 0x00, 0xF, 0xF, false);
    case 1: return __builtin_amdgcn_update_dpp(0, v, 0x55, 0xF, 0xF, false);
    case 2: return __builtin_amdgcn_update_dpp(0, v, 0xAA, 0xF, 0xF, false);
    default: return __builtin_amdgcn_update_dpp(0, v, 0xFF, 0xF, 0xF, false);
  }
}

// 64 zeros, read in place of an X row where a lane has none (padding slices,
// columns past a staged chunk, right-hand sides past nrhs); any T of <= 8 bytes
__device__ __align__(16) double kZeroRow[64] = {};  // never written
template <typename T> __device__ __forceinline__ const T *zero_row() {
  return reinterpret_cast<const T *>(kZeroRow);
}

// Gather the X rows of panel columns [kc, kc + kn) into a wave-private LDS
// tile xs[col * NRP + c] (NRP >= nc values per row, zero-padded).  Each lane
// owns whole columns: the column indices of up to CPL columns per lane are
// loaded first, then every X load, then the LDS writes, so a chunk costs two
// memory round trips however many columns it holds.  The loads carry no
// branches: indices past the chunk read zero from the buffer and columns
// past the chunk (or right-hand sides past nc) read the row of zeros.
template <typename T, int NRP, int CPL>
__device__ __forceinline__ void stage_x(T *xs, const int32_t *__restrict__ cx, const T *__restrict__ X,
                                        int64_t ldx, int c0, int nc, int kc, int kn, int lane) {
  const __amdgpu_buffer_rsrc_t rc = panel_rsrc(cx + kc, (uint32_t)kn * 4);
  for (int k0 = 0; k0 < kn; k0 += 64 * CPL) {
    int32_t xr[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j)
      xr[j] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(k0 + j * 64 + lane) * 4, 0, 0);
    T v[CPL][NRP];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int k = k0 + j * 64 + lane;
      const T *xp = k < kn ? X + (int64_t)xr[j] * ldx + c0 : zero_row<T>();
#pragma unroll
      for (int c = 0; c < NRP; ++c) v[j][c] = (c < nc ? xp : zero_row<T>())[c];
    }
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int k = k0 + j * 64 + lane;
      if (k < kn) {
#pragma unroll
        for (int c = 0; c < NRP; ++c) xs[k * NRP + c] = v[j][c];
      }
    }
  }
}

// Same tile from whole pieces of X rows, for full passes (nc = NRP) whose
// rows start on 16-byte boundaries: LPR lanes share a row and each loads up
// to 16 bytes of it, so one load instruction brings 64/LPR rows instead of
// one element of 64 rows.  A lane loads the indices of 64 columns, the
// others receive theirs through a lane permute, and CB blocks of 64 columns
// are in flight at a time.
template <int B> struct Bytes;
template <> struct Bytes<4> { using type = unsigned int; };
template <> struct Bytes<8> { using type = unsigned long long; };
template <> struct Bytes<16> { using type = v4u32; };

template <typename T, int NRP>
__device__ __forceinline__ void stage_x_rows(T *xs, const int32_t *__restrict__ cx,
                                             const T *__restrict__ X, int64_t ldx, int c0, int kc,
                                             int kn, int lane) {
  constexpr int RB = NRP * (int)sizeof(T);  // bytes of a staged row
  constexpr int LB = RB >= 16 ? 16 : RB;    // bytes per lane
  constexpr int LPR = RB / LB;              // lanes per row
  constexpr int RPI = 64 / LPR;             // rows per load instruction
  constexpr int EPL = LB / (int)sizeof(T);  // elements per lane
  constexpr int CB = LPR >= 4 ? 1 : 4 / LPR;
  using L = typename Bytes<LB>::type;
  const __amdgpu_buffer_rsrc_t rc = panel_rsrc(cx + kc, (uint32_t)kn * 4);
  const int sub = (lane % LPR) * EPL;
  for (int k0 = 0; k0 < kn; k0 += 64 * CB) {
    int32_t idx[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      idx[cb] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(k0 + cb * 64 + lane) * 4, 0, 0);
    L v[CB][LPR];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int q = 0; q < LPR; ++q) {
        const int rl = q * RPI + lane / LPR;
        const int32_t r = __shfl(idx[cb], rl, 64);
        const int k = k0 + cb * 64 + rl;
        const T *xp = (k < kn ? X + (int64_t)r * ldx + c0 : zero_row<T>()) + sub;
        v[cb][q] = *reinterpret_cast<const L *>(xp);
      }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int q = 0; q < LPR; ++q) {
        const int k = k0 + cb * 64 + q * RPI + lane / LPR;
        if (k < kn) *reinterpret_cast<L *>(xs + k * NRP + sub) = v[cb][q];
      }
  }
}

// ---------------------------------------------------------------------------
// vector-FMA product, NR right-hand sides per pass
// ---------------------------------------------------------------------------
// The X rows of a chunk of panel columns are first gathered into a
// wave-private LDS buffer, so the value stream never waits on a dependent
// index -> X load chain.  The values of the next U steps are in flight while
// the current U steps are multiplied.
// Tuning of the two vector kernels, measured on the 32^3 lattice (b = 13),
// the zincblende particle and the three-species random operator: which pass
// widths use 16-byte value loads (the kernel after this one), the value
// loads in flight per lane (steps of look-ahead) and the LDS staging per
// wave in bytes.
template <typename T, int NR> constexpr bool use_vp() { return sizeof(T) == 8 ? NR <= 4 : NR == 1; }
template <typename T, int NR> constexpr int vec_depth() { return 8; }
template <typename T, int NR> constexpr int vec_xs_bytes() { return sizeof(T) == 8 && NR >= 4 ? 8192 : 4096; }
template <typename T, int NR> constexpr int vp_depth() { return sizeof(T) == 8 && NR >= 2 ? 8 : 4; }
template <typename T, int NR> constexpr int vp_xs_bytes() { return sizeof(T) == 8 && NR >= 2 ? 8192 : 4096; }

template <typename T, int NR, bool MOM>
__global__ void __launch_bounds__(kThreads) k_spmm_vec(FwdParams<T> P) {
  extern __shared__ double s_mom[];
  constexpr int XCAP = vec_xs_bytes<T, NR>() / sizeof(T);
  constexpr int U = vec_depth<T, NR>();
  __shared__ __align__(16) T xs_all[kWaves * XCAP];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int w = wave_id();
  const int lane = threadIdx.x & 63;
  const int row = wg * kWaves + w;
  T *xs = xs_all + w * XCAP;
  mom_init<MOM>(s_mom, P.nrhs);
  if (row < P.nrows) {
    const RowDesc rd = P.rows[row];
    const int b = rd.b, K = rd.K;
    // G column groups of b lanes; capped so that one staged chunk holds at
    // least G*U columns of NR values (otherwise ccap below would be 0 and the
    // chunk loop would not advance: b = 1 gives 64 groups)
    constexpr int GMAX = XCAP / (NR * U);
    static_assert(GMAX >= 1, "LDS staging buffer too small");
    const int G = min(64 / b, GMAX);
    const int g = lane / b;
    const int p = lane - g * b;
    const int GB = G * b;
    // panel columns per staged chunk: a positive multiple of G*U that fits
    const int ccap = (XCAP / NR) / (G * U) * (G * U);
    const int32_t *__restrict__ cxrow = P.colx + rd.cbase;
    for (int c0 = 0; c0 < P.nrhs; c0 += NR) {
      const int nc = min(NR, P.nrhs - c0);
      T acc[NR];
#pragma unroll
      for (int c = 0; c < NR; ++c) acc[c] = T(0);
      for (int kc = 0; kc < K; kc += ccap) {
        const int kn = min(ccap, K - kc);
        // steps over the chunk, rounded up to whole groups of U; values past
        // the chunk read as zero and meet zero-padded staged X rows
        const int ngrp = (kn + G * U - 1) / (G * U);
        const __amdgpu_buffer_rsrc_t vr =
            panel_rsrc(P.vals + rd.vbase + (int64_t)kc * b, (uint32_t)(kn * b * sizeof(T)));
        const uint32_t lo = (uint32_t)lane * sizeof(T);
        const uint32_t stepb = (uint32_t)GB * sizeof(T);
        T a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = buf_load_nt<T>(vr, lo + u * stepb);
        wave_lds_sync();  // previous chunk fully consumed
        if (NR > 1 && nc == NR && P.xrow16)
          stage_x_rows<T, NR>(xs, cxrow, P.X, P.ldx, c0, kc, kn, lane);
        else
          stage_x<T, NR, (NR <= 2 ? 4 : 2)>(xs, cxrow, P.X, P.ldx, c0, nc, kc, kn, lane);
        for (int e = kn * NR + lane; e < ngrp * G * U * NR; e += 64) xs[e] = T(0);
        wave_lds_sync();
        if (g < G) {
          for (int q = 0; q < ngrp; ++q) {
            const int s = q * U;
            T an[U];
#pragma unroll
            for (int u = 0; u < U; ++u) an[u] = buf_load_nt<T>(vr, lo + (s + U + u) * stepb);
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const T *xp = xs + ((s + u) * G + g) * NR;
#pragma unroll
              for (int c = 0; c < NR; ++c) acc[c] = fma(a[u], xp[c], acc[c]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = an[u];
          }
        }
      }
      // groups g and g + st hold partial sums of the same panel row
      for (int st = 1; st < G; st <<= 1) {
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          const T o = __shfl_down(acc[c], st * b, 64);
          if ((g & (2 * st - 1)) == 0 && g + st < G) acc[c] += o;
        }
      }
      double mom[NR];
#pragma unroll
      for (int c = 0; c < NR; ++c) mom[c] = 0.0;
      if (lane < b) {
        const int64_t r = (int64_t)rd.yrow + p;
        T *yo = P.Yout + r * P.ldy + c0;
        const T *yi = P.Yin + r * P.ldyin + c0;
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          if (c < nc) {
            T y = T(P.alpha) * acc[c];
            if (P.beta != 0.0) y = fma(T(P.beta), yi[c], y);
            yo[c] = y;
            if (MOM) mom[c] = (double)P.R[r * P.ldr + c0 + c] * (double)y;
          }
        }
      }
      if (MOM) {
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          const double t = wave_sum(mom[c]);
          if (lane == 0 && c < nc) s_mom[w * P.nrhs + c0 + c] += t;
        }
      }
    }
  }
  mom_flush<MOM>(s_mom, P.nrhs, wg, P.mom);
}

// ---------------------------------------------------------------------------
// vector-FMA product with 16-byte value loads
// ---------------------------------------------------------------------------
// A step covers C panel columns (C*b values, contiguous in the column-major
// panel); lane l loads the E = 16/sizeof(T) consecutive values E*l .. E*l+E-1
// of the step with one 16-byte load.  C is the largest multiple of E with
// C*b <= 64*E, so the step length is a multiple of b and every lane keeps
// the same E panel rows in every step; lanes l and l + b hold the same rows.
// X rows are staged in LDS as in the kernel above.
template <typename T, int NR, bool MOM>
__global__ void __launch_bounds__(kThreads) k_spmm_vp(FwdParams<T> P) {
  extern __shared__ double s_mom[];
  constexpr int E = 16 / (int)sizeof(T);
  constexpr int XCAP = vp_xs_bytes<T, NR>() / sizeof(T);
  constexpr int U = vp_depth<T, NR>();
  __shared__ __align__(16) T xs_all[kWaves * XCAP];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int w = wave_id();
  const int lane = threadIdx.x & 63;
  const int row = wg * kWaves + w;
  T *xs = xs_all + w * XCAP;
  mom_init<MOM>(s_mom, P.nrhs);
  if (row < P.nrows) {
    const RowDesc rd = P.rows[row];
    const int b = rd.b, K = rd.K;
    // columns per step (a multiple of E), capped so a staged chunk holds U steps
    constexpr int CMAX = XCAP / (NR * U) / E * E;
    static_assert(CMAX >= E, "LDS staging buffer too small");
    const int C = min((64 * E / b) / E * E, CMAX);
    const int NL = C * b / E;  // active lanes
    int cj[E], rj[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int e = E * lane + j;
      cj[j] = e / b;
      rj[j] = e - cj[j] * b;
    }
    const int ccap = (XCAP / NR) / (C * U) * (C * U);
    const int32_t *__restrict__ cxrow = P.colx + rd.cbase;
    for (int c0 = 0; c0 < P.nrhs; c0 += NR) {
      const int nc = min(NR, P.nrhs - c0);
      T acc[E][NR];
#pragma unroll
      for (int j = 0; j < E; ++j)
#pragma unroll
        for (int c = 0; c < NR; ++c) acc[j][c] = T(0);
      for (int kc = 0; kc < K; kc += ccap) {
        const int kn = min(ccap, K - kc);
        const int ngrp = (kn + C * U - 1) / (C * U);
        // the chunk's values rounded up to whole 16-byte loads: the pages
        // pad every panel with zeros to a multiple of 4 values
        const __amdgpu_buffer_rsrc_t vr = panel_rsrc(P.vals + rd.vbase + (int64_t)kc * b,
                                                     (uint32_t)((kn * b + E - 1) / E * E * sizeof(T)));
        const uint32_t lo = (uint32_t)lane * 16;
        const uint32_t stepb = (uint32_t)(C * b) * sizeof(T);
        v4u32 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          a[u] = __builtin_bit_cast(v4u32, __builtin_amdgcn_raw_buffer_load_b128(vr, lo + u * stepb, 0, 2));
        wave_lds_sync();
        if (NR > 1 && nc == NR && P.xrow16)
          stage_x_rows<T, NR>(xs, cxrow, P.X, P.ldx, c0, kc, kn, lane);
        else
          stage_x<T, NR, (NR <= 2 ? 4 : 2)>(xs, cxrow, P.X, P.ldx, c0, nc, kc, kn, lane);
        for (int e = kn * NR + lane; e < ngrp * C * U * NR; e += 64) xs[e] = T(0);
        wave_lds_sync();
        if (lane < NL) {
          for (int q = 0; q < ngrp; ++q) {
            const int s = q * U;
            v4u32 an[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
              an[u] = __builtin_bit_cast(
                  v4u32, __builtin_amdgcn_raw_buffer_load_b128(vr, lo + (s + U + u) * stepb, 0, 2));
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const T *av = reinterpret_cast<const T *>(&a[u]);
#pragma unroll
              for (int j = 0; j < E; ++j) {
                const T *xp = xs + ((s + u) * C + cj[j]) * NR;
#pragma unroll
                for (int c = 0; c < NR; ++c) acc[j][c] = fma(av[j], xp[c], acc[j][c]);
              }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = an[u];
          }
        }
      }
      // lanes l and l + b hold the same rows: tree over the C/E groups
      const int ng = C / E;
      const int g = lane / b;
      for (int st = 1; st < ng; st <<= 1) {
#pragma unroll
        for (int j = 0; j < E; ++j)
#pragma unroll
          for (int c = 0; c < NR; ++c) {
            const T o = __shfl_down(acc[j][c], st * b, 64);
            if ((g & (2 * st - 1)) == 0 && g + st < ng) acc[j][c] += o;
          }
      }
      // lanes < b now hold values E*l + j of the first E*b; row p collects
      // values p + t*b, t < E (lane (p + t*b) / E, slot (p + t*b) % E)
      T ysum[NR];
#pragma unroll
      for (int c = 0; c < NR; ++c) ysum[c] = T(0);
#pragma unroll
      for (int t = 0; t < E; ++t) {
        const int e = (lane < b ? lane : 0) + t * b;
        const int sl = e / E, sj = e - sl * E;
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          T v = T(0);
#pragma unroll
          for (int j = 0; j < E; ++j) {
            const T o = __shfl(acc[j][c], sl, 64);
            v = sj == j ? o : v;
          }
          ysum[c] += v;
        }
      }
      double mom[NR];
#pragma unroll
      for (int c = 0; c < NR; ++c) mom[c] = 0.0;
      if (lane < b) {
        const int64_t r = (int64_t)rd.yrow + lane;
        T *yo = P.Yout + r * P.ldy + c0;
        const T *yi = P.Yin + r * P.ldyin + c0;
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          if (c < nc) {
            T y = T(P.alpha) * ysum[c];
            if (P.beta != 0.0) y = fma(T(P.beta), yi[c], y);
            yo[c] = y;
            if (MOM) mom[c] = (double)P.R[r * P.ldr + c0 + c] * (double)y;
          }
        }
      }
      if (MOM) {
#pragma unroll
        for (int c = 0; c < NR; ++c) {
          const double t = wave_sum(mom[c]);
          if (lane == 0 && c < nc) s_mom[w * P.nrhs + c0 + c] += t;
        }
      }
    }
  }
  mom_flush<MOM>(s_mom, P.nrhs, wg, P.mom);
}

// ---------------------------------------------------------------------------
// FP64 product on small matrix-core tiles, few right-hand sides
// ---------------------------------------------------------------------------
// The four 4x4 blocks of v_mfma_f64_4x4x4 (which runs at the rate of the
// 16x16x4 one: 75 of 78 TFLOP/s measured) take 4 panel rows x 4 panel columns
// each against the X rows of those columns and 4 right-hand sides: a step is
// 16 panel columns, the blocks' partial sums meet once per panel.  Rows pad
// to 4 and right-hand sides to 4 or 8 instead of 16.  Lane 16 k + 4 q + i
// works on column 4 k + q of the step and on row i of a row group (values) or
// on right-hand sides LW i .. LW i + LW - 1 of every 4 LW (X).
//
// Bound by the load path like the kernel below, so both operands come 16
// bytes a lane, straight into the operand registers: two rows of a column
// (row groups g = 0, 1 are its even and odd rows; 5 to 8 rows one load, 9 to
// 12 one of 16 and one of 8 bytes, 13 to 16 two) and two right-hand sides of
// an X row, 16 rows a load.  The vector kernel needs 8-byte value loads and a
// round trip through LDS per chunk, the 16x16 tiles waste half their columns
// on 8 right-hand sides and take 4 + 4 loads per 16 columns where these take
// 2 + 2.  A ring of R register sets as in the kernel below.  Values are read
// through the caches: two loads share each line (streamed past them, nrhs 16
// on b = 9..20 took 203 us instead of 162).  Up to 32 rows go in one pass (162
// -> 141).  The kernels in their place (vector up to 8 right-hand sides, 16x16
// tiles with 8-byte loads beyond) and these, us: 40,000-atom particle nrhs 6
// 267 -> 228, 8 256 -> 236, 12 323 -> 259; b = 13 lattice nrhs 8 212 -> 195;
// 50,000 atoms of b = 1/4/9 nrhs 4 132 -> 88, 8 144 -> 98, 16 189 -> 139, 32
// 214 -> 197; b = 9..20 nrhs 8 138 -> 122, 16 212 -> 141, 32 234 -> 218.
template <typename T, int RG, int NG, int LW, bool MOM, int R>
__device__ __forceinline__ void small_rows(const FwdParams<T> &P, const RowDesc &rd, int m0, int c0,
                                           double *s_mom) {
  static_assert(sizeof(T) == 8, "FP64 tiles");
  constexpr int NL = NG / LW;            // X loads per step
  constexpr int NV = (RG + 1) / 2;       // value loads per step
  const int lane = threadIdx.x & 63;
  const int ij = lane & 3;
  const int col = 4 * (lane >> 4) + ((lane >> 2) & 3);
  const int b = rd.b, K = rd.K;
  const __amdgpu_buffer_rsrc_t rv =
      panel_rsrc(P.vals + rd.vbase, (uint32_t)((int64_t)K * b * sizeof(T)));
  const __amdgpu_buffer_rsrc_t rc = panel_rsrc(P.colx + rd.cbase, (uint32_t)(K * 4));
  const __amdgpu_buffer_rsrc_t rx = panel_rsrc(P.X, x_span(P));
  double acc[RG][NG];
#pragma unroll
  for (int g = 0; g < RG; ++g)
#pragma unroll
    for (int t = 0; t < NG; ++t) acc[g][t] = 0.0;
  // load v covers row groups 2v and 2v + 1, or with RG odd the last one alone
  auto single = [](int v) { return 2 * v + 1 == RG; };
  uint32_t vo[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v)
    vo[v] = (uint32_t)(col * b + m0 + 8 * v + (single(v) ? ij : 2 * ij)) * 8u;
  const uint32_t vstep = (uint32_t)(16 * b) * 8u;
  uint32_t xcol[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int c = c0 + 4 * LW * l + LW * ij;
    xcol[l] = c < P.nrhs ? (uint32_t)c * 8u : kOutCol;
  }
  auto ld_idx = [&](int s) {
    return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(16 * s + col) * 4, 0, 0);
  };
  auto ld_val = [&](int s, double (&av)[RG]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const uint32_t off = vo[v] + (uint32_t)s * vstep;
      if (single(v)) {
        av[2 * v] = buf_load<double>(rv, off);
      } else {
        const double2 q =
            __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0));
        av[2 * v] = q.x;
        av[(2 * v + 1) % RG] = q.y;
      }
    }
  };
  auto ld_x = [&](int s, int32_t xi, double (&xv)[NG]) {
    const uint32_t ro =
        16 * s + col < K ? (uint32_t)((int64_t)xi * P.ldx * (int64_t)sizeof(T)) : kOutRow;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      if constexpr (LW == 2) {
        const double2 q =
            __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rx, ro + xcol[l], 0, 0));
        xv[2 * l] = q.x;
        xv[2 * l + 1] = q.y;
      } else {
        xv[l] = buf_load<double>(rx, ro + xcol[l]);
      }
    }
  };
  auto mma = [&](const double (&av)[RG], const double (&xv)[NG], double (&sum)[RG][NG]) {
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int t = 0; t < NG; ++t)
        sum[g][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[g], xv[t], sum[g][t], 0, 0, 0);
  };
  // Up to 8 right-hand sides: the R steps of one turn of the ring are summed
  // from zero and added to the total once, 4 R terms at a time.  The vector
  // kernel splits a row over up to 128 lanes; with one chain per block the
  // rounding error was up to 1.76 times its (relative, b = 8: 3.8e-16 against
  // 2.2e-16 at 3 right-hand sides, now 1.8e-16; 3.8e-16 against 2.8e-16 at 8,
  // now 1.9e-16).
  constexpr bool kParts = NG <= 2;
  double part[kParts ? RG : 1][kParts ? NG : 1];
  auto begin_part = [&] {
    if constexpr (kParts) {
#pragma unroll
      for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int t = 0; t < NG; ++t) part[g][t] = 0.0;
    }
  };
  auto add = [&](const double (&av)[RG], const double (&xv)[NG]) {
    if constexpr (kParts)
      mma(av, xv, part);
    else
      mma(av, xv, acc);
  };
  auto end_part = [&] {
    if constexpr (kParts) {
#pragma unroll
      for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int t = 0; t < NG; ++t) acc[g][t] += part[g][t];
    }
  };
  const int ns = (K + 15) >> 4;
  double av[R][RG], xv[R][NG];
  int32_t xi[R];
#pragma unroll
  for (int r = 0; r < R; ++r) xi[r] = ld_idx(r);
#pragma unroll
  for (int r = 0; r + 1 < R; ++r) {
    ld_x(r, xi[r], xv[r]);
    ld_val(r, av[r]);
    xi[r] = ld_idx(r + R);
  }
  __builtin_amdgcn_sched_barrier(0);
  int s = 0;
  for (; s + R <= ns; s += R) {
    begin_part();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int q = (r + R - 1) % R;
      ld_x(s + r + R - 1, xi[q], xv[q]);
      ld_val(s + r + R - 1, av[q]);
      xi[q] = ld_idx(s + r + 2 * R - 1);
      __builtin_amdgcn_sched_barrier(0);
      add(av[r], xv[r]);
      __builtin_amdgcn_sched_barrier(0);
    }
    end_part();
  }
  begin_part();
#pragma unroll
  for (int r = 0; r + 1 < R; ++r)
    if (s + r < ns) add(av[r], xv[r]);
  end_part();
  // sum over the four blocks; then, four row groups at a time, lane
  // 16 i + 4 g + j writes the row that row group g holds at i, right-hand
  // sides j of each tile
  const int gl = (lane >> 2) & 3, il = lane >> 4;
  double mm[NG];
#pragma unroll
  for (int t = 0; t < NG; ++t) mm[t] = 0.0;
#pragma unroll
  for (int h = 0; h < RG; h += 4) {
    double y[NG];
#pragma unroll
    for (int t = 0; t < NG; ++t) y[t] = 0.0;
#pragma unroll
    for (int g = h; g < h + 4 && g < RG; ++g)
#pragma unroll
      for (int t = 0; t < NG; ++t) {
        double a = acc[g][t];
        a += __shfl_xor(a, 4, 64);
        a += __shfl_xor(a, 8, 64);
        y[t] = gl == g - h ? a : y[t];
      }
    const int gr = h + gl;   // this lane's row group
    const int prow = 8 * (gr >> 1) + (single(gr >> 1) ? il : 2 * il + (gr & 1));
    const bool ok = gr < RG && m0 + prow < b;
    const int64_t r = (int64_t)rd.yrow + m0 + prow;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const int cc = c0 + 4 * LW * l + LW * ij;
      if (ok && LW == 2 && P.yrow16 && cc + 2 <= P.nrhs) {
        double2 v = {P.alpha * y[LW * l], P.alpha * y[LW * l + LW - 1]};
        if (P.beta != 0.0) {
          const double2 q = *reinterpret_cast<const double2 *>(P.Yin + r * P.ldyin + cc);
          v.x = fma(P.beta, q.x, v.x);
          v.y = fma(P.beta, q.y, v.y);
        }
        *reinterpret_cast<double2 *>(P.Yout + r * P.ldy + cc) = v;
        if (MOM) {
          const double2 q = *reinterpret_cast<const double2 *>(P.R + r * P.ldr + cc);
          mm[LW * l] += q.x * v.x;
          mm[LW * l + LW - 1] += q.y * v.y;
        }
      } else if (ok) {
#pragma unroll
        for (int e = 0; e < LW; ++e) {
          if (cc + e < P.nrhs) {
            double v = P.alpha * y[LW * l + e];
            if (P.beta != 0.0) v = fma(P.beta, P.Yin[r * P.ldyin + cc + e], v);
            P.Yout[r * P.ldy + cc + e] = v;
            if (MOM) mm[LW * l + e] += P.R[r * P.ldr + cc + e] * v;
          }
        }
      }
    }
  }
  if (MOM) {
#pragma unroll
    for (int t = 0; t < NG; ++t) {
      double v = mm[t];
#pragma unroll
      for (int o = 4; o <= 32; o <<= 1) v += __shfl_xor(v, o, 64);
      const int n = c0 + 4 * LW * (t / LW) + LW * ij + t % LW;
      if (lane < 4 && n < P.nrhs) s_mom[wave_id() * P.nrhs + n] += v;
    }
  }
}

// NG groups of 4 right-hand sides and MR panel rows per pass; LW right-hand
// sides per X load.
template <int NG, int LW, bool MOM, int R, int MR>
__global__ void __launch_bounds__(kThreads) k_spmm_small(FwdParams<double> P) {
  extern __shared__ double s_mom[];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int row = wg * kWaves + wave_id();
  mom_init<MOM>(s_mom, P.nrhs);
  if (row < P.nrows) {
    const RowDesc rd = P.rows[row];
    for (int c0 = 0; c0 < P.nrhs; c0 += 4 * NG)
      for (int m0 = 0; m0 < rd.b; m0 += MR) {
        // 29 to 32 rows and 25 to 28 share a case; those past MR are not reached
        switch ((min(rd.b - m0, MR) + 3) >> 2) {
          case 1: small_rows<double, 1, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
          case 2: small_rows<double, 2, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
          case 3: small_rows<double, 3, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
          case 4: small_rows<double, 4, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
          case 5: small_rows<double, MR >= 20 ? 5 : 4, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
          case 6: small_rows<double, MR >= 24 ? 6 : 4, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
          default: small_rows<double, MR >= 32 ? 8 : 4, NG, LW, MOM, R>(P, rd, m0, c0, s_mom); break;
        }
      }
  }
  mom_flush<MOM>(s_mom, P.nrhs, wg, P.mom);
}

// ---------------------------------------------------------------------------
// FP64 / FP32 matrix-core product
// ---------------------------------------------------------------------------
// A operand: the panel's 4-column slice (contiguous, 4*b values, panel row m
// in lane m, slice column kq in lane group kq); B operand: the X rows of
// those 4 columns.  Slices are taken in groups of U.  A ring of R register
// sets: while one group multiplies, the values and X rows of the next R - 1
// groups are in flight, and the column indices of the R after those.  The
// ring loop has no branch (one around a load, or a way out of the loop other
// than its end, makes the compiler copy the sets and wait for every load in
// flight); the last groups are multiplied after it.  Values and indices are
// buffer loads that read zero past the panel, and padding slices point at a
// row of zeros instead of a row of X.  An index is compared with the panel's
// end where it is used, not where it is loaded: done at the load, it makes
// every group wait for the index just requested and, since loads return in
// order, for all the X rows requested before it.  Scheduling barriers keep
// each group's loads ahead of the matrix instructions.
//
// What bounds it: the compute unit's load path.  A load instruction of 8 or
// 16 bytes a lane takes 16 cycles of it; one of 4 bytes takes 4.7 when every
// four neighbouring lanes read consecutive or equal addresses, and 16 too
// when they don't or only some of them are in range.  The value stream from
// HBM and the gathered rows from L2 return through it in order, so their
// times add up (5 KiB of L2 hits alone take 102 cycles of a unit, 1 KiB of
// stream alone 95, together 221, at any occupancy).  Measured against two
// alternating sets with the index tested at the load, masked rows and
// right-hand sides and, in FP64, one row a value load: FP32 100,000 atoms of b
// = 1/4/9, nrhs 16 208 -> 156 us, 32 260 -> 216; FP32 40,000-atom particle,
// nrhs 13 276 -> 154, 33 369 -> 266, 64 314 -> 294; FP64 on it, nrhs 20 429 ->
// 305, 50 656 -> 491, 64 557 -> 540; FP64 32^3 lattice b = 13, nrhs 16 241 ->
// 215; FP64 Chebyshev step on the 24^3 one, nrhs 64: 206 -> 200.  Longer rings
// (R = 4) gain 2 % on the lattice and lose 4 % on the small blocks, groups of
// one slice lose on the lattice.
//
// VX: the N index of the 16x16 tiles is permuted so that lane m of tile t
// holds right-hand side c0 + l*16*VEC + VEC*m + e, with t = l*VEC + e and VEC
// elements per 16 bytes: one 16-byte load per lane and X row fetches VEC
// tiles, and outputs leave 16 bytes at a time where the vectors' alignment
// allows (yrow16).  A buffer load needs no more than 4-byte alignment, so with
// XB this serves every nrhs and leading dimension that fill VEC tiles (a
// lane's elements past nrhs go to columns that are not stored); with one
// 8-byte load per tile FP64 nrhs 20 and 50 took 367 and 600 us on the
// 40,000-atom particle, with these 305 and 491.
// Without XB it needs 16-byte aligned rows and whole passes.  The other
// form (VX = false) loads one element per lane and tile.
template <typename T> struct Vec16;
template <> struct Vec16<double> { using type = double2; static constexpr int n = 2; };
template <> struct Vec16<float> { using type = float4; static constexpr int n = 4; };

// Lane m < 8 of a 16-lane row holds rows 2m (x) and 2m + 1 (y) of one panel
// column, lane m >= 8 rows 2 (m - 8) and 2 (m - 8) + 1 of the next: a gets
// the first column, even rows in lanes 0-7 and odd rows in lanes 8-15, b the
// second (two data-parallel moves per half, no memory).
__device__ __forceinline__ int tile_row(int m) { return m < 8 ? 2 * m : 2 * m - 15; }
template <typename T> __device__ __forceinline__ void fill_pair(T x, T y, T &a, T &b) {
  static_assert(sizeof(T) == 8, "two 32-bit halves");
  const v2u32 xi = __builtin_bit_cast(v2u32, x), yi = __builtin_bit_cast(v2u32, y);
  v2u32 ai, bi;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // 0x128: row_ror:8; bank masks 0xC / 0x3: lanes 8-15 / 0-7 of each row
    ai[h] = (uint32_t)__builtin_amdgcn_update_dpp((int)xi[h], (int)yi[h], 0x128, 0xF, 0xC, false);
    bi[h] = (uint32_t)__builtin_amdgcn_update_dpp((int)yi[h], (int)xi[h], 0x128, 0xF, 0x3, false);
  }
  a = __builtin_bit_cast(T, ai);
  b = __builtin_bit_cast(T, bi);
}

template <typename T, int NT, bool MOM, bool VX, bool XB>
__global__ void __launch_bounds__(kThreads) k_spmm_mfma(FwdParams<T> P) {
  extern __shared__ double s_mom[];
  using V = typename Frag<T>::type;
  using L16 = typename Vec16<T>::type;
  constexpr int VEC = Vec16<T>::n;
  constexpr int NL = VX ? NT / VEC : 0;  // 16-byte loads per lane and X row
  constexpr int U = 2;                    // slices per group
  constexpr bool PAIR = sizeof(T) == 8;   // values two rows at a time
  constexpr int R = NT * sizeof(T) <= 8 ? 4 : 3;  // groups in the ring
  static_assert(!VX || NT % VEC == 0, "tile count must fill whole 16-byte loads");
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int w = wave_id();
  const int lane = threadIdx.x & 63;
  const int row = wg * kWaves + w;
  const int m = lane & 15;   // A: panel row in the tile; B and D: column in the tile
  const int kq = lane >> 4;  // A and B: column of the 4-column slice; D: row group
  mom_init<MOM>(s_mom, P.nrhs);
  if (row < P.nrows) {
    const RowDesc rd = P.rows[row];
    const int b = rd.b, K = rd.K;
    const int nsteps = (K + 3) >> 2;
    const T *__restrict__ vals = P.vals + rd.vbase;
    const int32_t *__restrict__ cx = P.colx + rd.cbase;
    // column of (tile t, lane m) relative to c0
    auto col = [&](int t) {
      return VX ? (t / VEC) * 16 * VEC + VEC * m + (t % VEC) : t * 16 + m;
    };
    for (int mt = 0; mt * 16 < b; ++mt) {
      const int p = mt * 16 + m;
      for (int c0 = 0; c0 < P.nrhs; c0 += 16 * NT) {
        V acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = V{};
        const __amdgpu_buffer_rsrc_t rv = panel_rsrc(vals, (uint32_t)((int64_t)K * b * sizeof(T)));
        const __amdgpu_buffer_rsrc_t rc = panel_rsrc(cx, (uint32_t)(K * 4));
        // FP32: lane (m, kq) loads row m of column kq of a slice.  Four
        // neighbouring lanes are in range together, or they take the slow path
        // of the load unit: rows past the panel, to the next multiple of four,
        // read the next column's values into tile rows that are never stored.
        // Those beyond load nothing (b = 8, nrhs 64: 167 us; reading on 178).
        // FP64: an 8-byte load costs the unit as much as one of 16, so lane
        // (m, kq) loads rows 2 (m % 8) and 2 (m % 8) + 1 of column 2 kq + m / 8
        // of the group's 8 columns in one, and lanes m and m + 8 then exchange
        // halves (fill_pair below): slice u of a group holds its columns
        // 2 kq + u, tile row m the panel row tile_row(m).
        const uint32_t vlane = PAIR ? (uint32_t)((2 * kq + (m >> 3)) * b + mt * 16 + 2 * (m & 7)) * 8u
                               : (p & ~3) < b ? (uint32_t)(kq * b + p) * (uint32_t)sizeof(T)
                                              : kOutRow;
        // XB: all of X lies within 2^31 bytes and is read through one buffer
        // descriptor (cheaper addressing); otherwise through 64-bit pointers
        const __amdgpu_buffer_rsrc_t rx =
            panel_rsrc(P.X, XB ? x_span(P) : 0u);
        // column part of the lane's offsets, per 16-byte load (VX) or tile.
        // 4-byte loads: four neighbouring lanes are in range together (see
        // the values above); those past nrhs read what follows inside X's
        // span into output columns that are never stored.
        uint32_t xcol[VX ? NL : NT];
#pragma unroll
        for (int l = 0; l < (VX ? NL : NT); ++l) {
          const int c = VX ? c0 + l * 16 * VEC + VEC * m : c0 + l * 16 + m;
          const int cq = !VX && sizeof(T) == 4 ? c & ~3 : c;
          xcol[l] = cq < P.nrhs ? (uint32_t)c * (uint32_t)sizeof(T) : kOutCol;
        }
        // lane (m, kq) loads the index of column kq of slice m / 8 (equal
        // addresses in every group of four lanes); the lanes of a row (equal
        // kq) then read slice u's from lane 8 u
        static_assert(U == 2, "one index register serves two slices");
        auto col_of = [&](int g, int u) {   // panel column of slice u, lane row kq
          return PAIR ? g * 8 + 2 * kq + u : (g * U + u) * 4 + kq;
        };
        auto ld_idx = [&](int g) {
          const int k = col_of(g, m >> 3);
          return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)k * 4, 0, 0);
        };
        // AUX 2: streamed past the caches; 0: kept, for the panel's next tile
        // of rows (b > 16: FP64 b = 9..20 nrhs 16 200 -> 177 us; on b <= 16
        // streaming is 2-5 % faster)
        auto ld_val = [&](auto aux, int g, T(&av)[U]) {
          constexpr int AUX = decltype(aux)::value;
          if constexpr (PAIR) {
            const double2 q = __builtin_bit_cast(
                double2,
                __builtin_amdgcn_raw_buffer_load_b128(rv, vlane + (uint32_t)(g * 8 * b) * 8u, 0, AUX));
            av[0] = q.x;
            av[1] = q.y;
          } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const uint32_t off = vlane + (uint32_t)((g * U + u) * 4 * b) * (uint32_t)sizeof(T);
              av[u] = AUX ? buf_load_nt<T>(rv, off) : buf_load<T>(rv, off);
            }
          }
        };
        auto ld_x = [&](int g, int32_t xg, T(&xv)[U][NT]) {
          // XB: byte offset of the lane's own column, past the descriptor for
          // a padding column (reads zeros).  The product is formed before the
          // broadcast: after it the compiler fuses it with the addition of
          // the column part into a 64-bit one whose unused upper half can be a register
          // with a load in flight, and waits for that load.
          const int32_t xo =
              XB ? (col_of(g, m >> 3) < K
                        ? (int32_t)(uint32_t)((int64_t)xg * P.ldx * (int64_t)sizeof(T))
                        : (int32_t)kOutRow)
                 : xg;
          const int32_t xi[U] = {row_bcast<0>(xo), row_bcast<8>(xo)};
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if constexpr (XB) {
              const uint32_t ro = (uint32_t)xi[u];
              if constexpr (VX) {
#pragma unroll
                for (int l = 0; l < (VX ? NL : 1); ++l) {
                  const L16 q = __builtin_bit_cast(
                      L16, __builtin_amdgcn_raw_buffer_load_b128(rx, ro + xcol[l], 0, 0));
                  const T *qe = reinterpret_cast<const T *>(&q);
#pragma unroll
                  for (int e = 0; e < VEC; ++e) xv[u][l * VEC + e] = qe[e];
                }
              } else {
#pragma unroll
                for (int t = 0; t < NT; ++t)
                  xv[u][t] = buf_load<T>(rx, ro + xcol[t]);
              }
            } else {
              // padding slices read a row of zeros instead of a row of X
              const T *xp = col_of(g, u) < K ? P.X + (int64_t)xi[u] * P.ldx + c0 : zero_row<T>();
              if constexpr (VX) {
#pragma unroll
                for (int l = 0; l < (VX ? NL : 1); ++l) {
                  const L16 q = *reinterpret_cast<const L16 *>(xp + l * 16 * VEC + VEC * m);
                  const T *qe = reinterpret_cast<const T *>(&q);
#pragma unroll
                  for (int e = 0; e < VEC; ++e) xv[u][l * VEC + e] = qe[e];
                }
              } else {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                  const int n = t * 16 + m;
                  xv[u][t] = (c0 + n < P.nrhs ? xp : zero_row<T>())[n];
                }
              }
            }
          }
        };
        auto mma = [&](const T(&lv)[U], const T(&xv)[U][NT]) {
          T av[U];
          if constexpr (PAIR) {
            fill_pair(lv[0], lv[1], av[0], av[1]);
          } else {
#pragma unroll
            for (int u = 0; u < U; ++u) av[u] = lv[u];
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = mfma(av[u], xv[u][t], acc[t]);
        };
        const int ngroups = (nsteps + U - 1) / U;
        auto panel = [&](auto aux) {
          T av[R][U], xv[R][U][NT];
          int32_t xi[R];
#pragma unroll
          for (int r = 0; r < R; ++r) xi[r] = ld_idx(r);
#pragma unroll
          for (int r = 0; r + 1 < R; ++r) {
            ld_x(r, xi[r], xv[r]);
            ld_val(aux, r, av[r]);
            xi[r] = ld_idx(r + R);
          }
          __builtin_amdgcn_sched_barrier(0);
          int g = 0;
          for (; g + R <= ngroups; g += R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const int q = (r + R - 1) % R;
              ld_x(g + r + R - 1, xi[q], xv[q]);
              ld_val(aux, g + r + R - 1, av[q]);
              xi[q] = ld_idx(g + r + 2 * R - 1);
              __builtin_amdgcn_sched_barrier(0);
              mma(av[r], xv[r]);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
#pragma unroll
          for (int r = 0; r + 1 < R; ++r)
            if (g + r < ngroups) mma(av[r], xv[r]);
        };
        if (b > 16)
          panel(std::integral_constant<int, 0>{});
        else
          panel(std::integral_constant<int, 2>{});
        // epilogue: row pr of the tile, columns col(t)
        double mmv[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) mmv[t] = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int pr = mt * 16 + (PAIR ? tile_row(dst_row<T>(kq, i)) : dst_row<T>(kq, i));
          if (pr < b) {
            const int64_t r = (int64_t)rd.yrow + pr;
            T y[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) y[t] = T(P.alpha) * acc[t][i];
            if constexpr (VX) {
#pragma unroll
              for (int l = 0; l < (VX ? NL : 1); ++l) {
                const int64_t cc = c0 + l * 16 * VEC + VEC * m;
                if (!P.yrow16 || cc + VEC > P.nrhs) {   // element by element
#pragma unroll
                  for (int e = 0; e < VEC; ++e) {
                    if (cc + e < P.nrhs) {
                      T &ye = y[l * VEC + e];
                      if (P.beta != 0.0) ye = fma(T(P.beta), P.Yin[r * P.ldyin + cc + e], ye);
                      P.Yout[r * P.ldy + cc + e] = ye;
                      if (MOM) mmv[l * VEC + e] += (double)P.R[r * P.ldr + cc + e] * (double)ye;
                    }
                  }
                  continue;
                }
                if (P.beta != 0.0) {
                  const L16 q = *reinterpret_cast<const L16 *>(P.Yin + r * P.ldyin + cc);
                  const T *qe = reinterpret_cast<const T *>(&q);
#pragma unroll
                  for (int e = 0; e < VEC; ++e) y[l * VEC + e] = fma(T(P.beta), qe[e], y[l * VEC + e]);
                }
                L16 o;
                T *oe = reinterpret_cast<T *>(&o);
#pragma unroll
                for (int e = 0; e < VEC; ++e) oe[e] = y[l * VEC + e];
                *reinterpret_cast<L16 *>(P.Yout + r * P.ldy + cc) = o;
                if (MOM) {
                  const L16 q = *reinterpret_cast<const L16 *>(P.R + r * P.ldr + cc);
                  const T *qe = reinterpret_cast<const T *>(&q);
#pragma unroll
                  for (int e = 0; e < VEC; ++e) mmv[l * VEC + e] += (double)qe[e] * (double)oe[e];
                }
              }
            } else {
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                const int n = c0 + t * 16 + m;
                if (n < P.nrhs) {
                  if (P.beta != 0.0) y[t] = fma(T(P.beta), P.Yin[r * P.ldyin + n], y[t]);
                  P.Yout[r * P.ldy + n] = y[t];
                  if (MOM) mmv[t] += (double)P.R[r * P.ldr + n] * (double)y[t];
                }
              }
            }
          }
        }
        if (MOM) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            double mm = mmv[t];
            mm += __shfl_xor(mm, 16, 64);
            mm += __shfl_xor(mm, 32, 64);
            const int n = c0 + col(t);
            if (kq == 0 && n < P.nrhs) s_mom[w * P.nrhs + n] += mm;
          }
        }
      }
    }
  }
  mom_flush<MOM>(s_mom, P.nrhs, wg, P.mom);
}

// ---------------------------------------------------------------------------
// BF16x3 matrix-core product: a*x ~ ah*xh + ah*xl + al*xh, FP32 accumulation
// ---------------------------------------------------------------------------
// 32-column slices; lane (m, kg) owns 8 consecutive panel columns of row m
// (one 16-byte load per page) and, for the B operand, the same 8 columns of
// X in column m of the tile.  X is split into bf16 hi/lo on the fly with the
// hardware round-to-nearest-even conversion (two values per instruction).
// Loads are branch-free and the next slice's values and X rows are in flight
// while the current slice multiplies, its column indices two slices ahead.
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned int pack_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned int, v2bf{(__bf16)a, (__bf16)b});
}

// Split of 8 consecutive panel columns' X values into hi and lo fragments.
__device__ __forceinline__ void split_bf16(const float (&x)[8], v8u &xh, v8u &xl) {
  v4u32 hi, lo;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const unsigned int h = pack_bf16(x[2 * q], x[2 * q + 1]);
    hi[q] = h;
    lo[q] = pack_bf16(x[2 * q] - __uint_as_float(h << 16),
                      x[2 * q + 1] - __uint_as_float(h & 0xFFFF0000u));
  }
  xh = __builtin_bit_cast(v8u, hi);
  xl = __builtin_bit_cast(v8u, lo);
}

// Any nrhs and leading dimension, NT tiles of 16 right-hand sides per pass,
// one 4-byte load per lane, X row and tile.  (With clamped pointer loads and
// a software rounding, waiting for each slice's X rows: nrhs 32 on 100,000
// atoms of b = 1/4/9 788 us, now 208; nrhs 50 on the 40,000-atom particle
// 1186 -> 300, nrhs 20 550 -> 163.)
template <int NT, bool MOM, bool XB>
__global__ void __launch_bounds__(kThreads) k_spmm_bf16x3(FwdParams<float> P) {
  extern __shared__ double s_mom[];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int w = wave_id();
  const int lane = threadIdx.x & 63;
  const int row = wg * kWaves + w;
  const int m = lane & 15;
  const int kg = lane >> 4;  // 8-column group of the 32-column slice
  mom_init<MOM>(s_mom, P.nrhs);
  if (row < P.nrows) {
    const RowDesc rd = P.rows[row];
    const int b = rd.b, K = rd.K;
    const int ngroups = (K + 7) >> 3;
    const int nsteps = (K + 31) >> 5;
    const int64_t vb16 = P.vbase16[row];
    constexpr uint32_t kOut = 0x80000000u;
    const uint32_t pbytes = (uint32_t)((int64_t)ngroups * 8 * b * sizeof(uint16_t));
    const __amdgpu_buffer_rsrc_t rh = panel_rsrc(P.hi + vb16, pbytes);
    const __amdgpu_buffer_rsrc_t rl = panel_rsrc(P.lo + vb16, pbytes);
    const __amdgpu_buffer_rsrc_t rc = panel_rsrc(P.colx + rd.cbase, (uint32_t)(K * 4));
    const __amdgpu_buffer_rsrc_t rx =
        panel_rsrc(P.X, XB ? x_span(P) : 0u);
    for (int mt = 0; mt * 16 < b; ++mt) {
      const int p = mt * 16 + m;
      const uint32_t vlane = p < b ? (uint32_t)(kg * 8 * b + p * 8) * sizeof(uint16_t) : kOut;
      for (int c0 = 0; c0 < P.nrhs; c0 += 16 * NT) {
        v4f acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = v4f{};
        // four neighbouring lanes are in range together (as in the FP32 kernel)
        uint32_t xcol[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int c = c0 + t * 16 + m;
          xcol[t] = (c & ~3) < P.nrhs ? (uint32_t)c * 4u : kOutCol;
        }
        auto ld_idx = [&](int s) {
          // lane (m, kg) loads column m % 8 of its group; the lanes of a row
          // (equal kg) then read column u's from lane u
          const int k = (s * 4 + kg) * 8 + (m & 7);
          return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)k * 4, 0, 0);
        };
        auto ld_val = [&](int s, v8u &h, v8u &l) {
          const uint32_t off = vlane + (uint32_t)(s * 32 * b) * sizeof(uint16_t);
          h = __builtin_bit_cast(v8u, __builtin_amdgcn_raw_buffer_load_b128(rh, off, 0, 2));
          l = __builtin_bit_cast(v8u, __builtin_amdgcn_raw_buffer_load_b128(rl, off, 0, 2));
        };
        auto ld_x = [&](int s, int32_t xg, float(&xv)[NT][8]) {
          const int k0 = (s * 4 + kg) * 8;
          const int32_t xo =
              XB ? (k0 + (m & 7) < K
                        ? (int32_t)(uint32_t)((int64_t)xg * P.ldx * (int64_t)sizeof(float))
                        : (int32_t)kOutRow)
                 : xg;
          const int32_t xi[8] = {row_bcast<0>(xo), row_bcast<1>(xo), row_bcast<2>(xo),
                                 row_bcast<3>(xo), row_bcast<4>(xo), row_bcast<5>(xo),
                                 row_bcast<6>(xo), row_bcast<7>(xo)};
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              if constexpr (XB) {
                xv[t][u] = buf_load<float>(rx, (uint32_t)xi[u] + xcol[t]);
              } else {
                const int n = c0 + t * 16 + m;
                const float *xp = k0 + u < K && n < P.nrhs ? P.X + (int64_t)xi[u] * P.ldx + n
                                                           : zero_row<float>();
                xv[t][u] = *xp;
              }
            }
        };
        auto mma = [&](const v8u &ah, const v8u &al, const float(&xv)[NT][8]) {
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            v8u xh, xl;
            split_bf16(xv[t], xh, xl);
            acc[t] = mfma_bf16(ah, xh, acc[t]);
            acc[t] = mfma_bf16(ah, xl, acc[t]);
            acc[t] = mfma_bf16(al, xh, acc[t]);
          }
        };
        v8u vh[2], vl[2];
        float xv[2][NT][8];
        int32_t xi[2] = {ld_idx(0), ld_idx(1)};
        ld_x(0, xi[0], xv[0]);
        ld_val(0, vh[0], vl[0]);
        xi[0] = ld_idx(2);
        __builtin_amdgcn_sched_barrier(0);
        int s = 0;
        for (; s + 2 <= nsteps; s += 2) {
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const int q = r ^ 1;
            ld_x(s + r + 1, xi[q], xv[q]);
            ld_val(s + r + 1, vh[q], vl[q]);
            xi[q] = ld_idx(s + r + 3);
            __builtin_amdgcn_sched_barrier(0);
            mma(vh[r], vl[r], xv[r]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (s < nsteps) mma(vh[0], vl[0], xv[0]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int n = c0 + t * 16 + m;
          double mm = 0.0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int pr = mt * 16 + dst_row<float>(kg, i);
            if (pr < b && n < P.nrhs) {
              const int64_t r = (int64_t)rd.yrow + pr;
              float y = float(P.alpha) * acc[t][i];
              if (P.beta != 0.0) y = fmaf(float(P.beta), P.Yin[r * P.ldyin + n], y);
              P.Yout[r * P.ldy + n] = y;
              if (MOM) mm += (double)P.R[r * P.ldr + n] * (double)y;
            }
          }
          if (MOM) {
            mm += __shfl_xor(mm, 16, 64);
            mm += __shfl_xor(mm, 32, 64);
            if (kg == 0 && n < P.nrhs) s_mom[w * P.nrhs + n] += mm;
          }
        }
      }
    }
  }
  mom_flush<MOM>(s_mom, P.nrhs, wg, P.mom);
}

// BF16x3 fast path: 64 right-hand sides per pass, tile t of lane m holds
// column c0 + 4m + t, so the 8 X rows of a lane's 8-column group arrive as
// eight 16-byte loads.  With one index register a lane, broadcast along the
// row, instead of two 16-byte index loads that were compared with the panel's
// end at once (and so waited for): Chebyshev step on the 32^3 lattice b = 13,
// nrhs 64: 240 -> 199 us (184 -> 158 registers).

template <bool MOM, bool XB>
__global__ void __launch_bounds__(kThreads) k_spmm_bf16x3_vx(FwdParams<float> P) {
  extern __shared__ double s_mom[];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int w = wave_id();
  const int lane = threadIdx.x & 63;
  const int row = wg * kWaves + w;
  const int m = lane & 15;
  const int kg = lane >> 4;
  mom_init<MOM>(s_mom, P.nrhs);
  if (row < P.nrows) {
    const RowDesc rd = P.rows[row];
    const int b = rd.b, K = rd.K;
    const int ngroups = (K + 7) >> 3;
    const int nsteps = (K + 31) >> 5;
    const int64_t vb16 = P.vbase16[row];
    constexpr uint32_t kOut = 0x80000000u;
    // the row's BF16 pages, its column table and (XB) all of X, each read
    // through one buffer descriptor; offsets past the end read zero
    const uint32_t pbytes = (uint32_t)((int64_t)ngroups * 8 * b * sizeof(uint16_t));
    const __amdgpu_buffer_rsrc_t rh = panel_rsrc(P.hi + vb16, pbytes);
    const __amdgpu_buffer_rsrc_t rl = panel_rsrc(P.lo + vb16, pbytes);
    const __amdgpu_buffer_rsrc_t rc = panel_rsrc(P.colx + rd.cbase, (uint32_t)(K * 4));
    const __amdgpu_buffer_rsrc_t rx =
        panel_rsrc(P.X, XB ? (uint32_t)(P.xrows * P.ldx * (int64_t)sizeof(float)) : 0u);
    for (int mt = 0; mt * 16 < b; ++mt) {
      const int p = mt * 16 + m;
      const bool prow = p < b;
      const uint32_t vlane = prow ? (uint32_t)(kg * 8 * b + p * 8) * sizeof(uint16_t) : kOut;
      for (int c0 = 0; c0 < P.nrhs; c0 += 64) {
        v4f acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = v4f{};
        const uint32_t xcol = (uint32_t)(c0 + 4 * m) * sizeof(float);
        // step s covers panel columns [32 s, 32 s + 32); lane group kg holds
        // the 8 columns 32 s + 8 kg + u.  Two register sets alternate as in
        // the FP64/FP32 kernel: indices run two steps ahead, values and X
        // rows one step ahead.
        auto ld_idx = [&](int s) {
          // lane (m, kg) loads column m % 8 of its group; the lanes of a row
          // (equal kg) then read column u's from lane u
          const int k = (s * 4 + kg) * 8 + (m & 7);
          return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)k * 4, 0, 0);
        };
        auto ld_val = [&](int s, v8u &h, v8u &l) {
          const uint32_t off = vlane + (uint32_t)(s * 32 * b) * sizeof(uint16_t);
          h = __builtin_bit_cast(v8u, __builtin_amdgcn_raw_buffer_load_b128(rh, off, 0, 2));
          l = __builtin_bit_cast(v8u, __builtin_amdgcn_raw_buffer_load_b128(rl, off, 0, 2));
        };
        auto ld_x = [&](int s, int32_t xg, float4(&xv)[8]) {
          const int k0 = (s * 4 + kg) * 8;
          // XB: byte offset of the lane's own column, past the descriptor for
          // a padding column (reads zeros)
          const int32_t xo =
              XB ? (k0 + (m & 7) < K
                        ? (int32_t)(uint32_t)((int64_t)xg * P.ldx * (int64_t)sizeof(float))
                        : (int32_t)kOut)
                 : xg;
          const int32_t xi[8] = {row_bcast<0>(xo), row_bcast<1>(xo), row_bcast<2>(xo),
                                 row_bcast<3>(xo), row_bcast<4>(xo), row_bcast<5>(xo),
                                 row_bcast<6>(xo), row_bcast<7>(xo)};
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if constexpr (XB) {
              xv[u] = __builtin_bit_cast(
                  float4, __builtin_amdgcn_raw_buffer_load_b128(rx, (uint32_t)xi[u] + xcol, 0, 0));
            } else {
              const float *xp = k0 + u < K ? P.X + (int64_t)xi[u] * P.ldx + c0 : zero_row<float>();
              xv[u] = *reinterpret_cast<const float4 *>(xp + 4 * m);
            }
          }
        };
        auto mma = [&](const v8u &ah, const v8u &al, const float4(&xv)[8]) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = reinterpret_cast<const float *>(&xv[u])[t];
            v8u xh, xl;
            split_bf16(x, xh, xl);
            acc[t] = mfma_bf16(ah, xh, acc[t]);
            acc[t] = mfma_bf16(ah, xl, acc[t]);
            acc[t] = mfma_bf16(al, xh, acc[t]);
          }
        };
        v8u vh[2], vl[2];
        float4 xv[2][8];
        int32_t xi[2] = {ld_idx(0), ld_idx(1)};
        ld_x(0, xi[0], xv[0]);
        ld_val(0, vh[0], vl[0]);
        xi[0] = ld_idx(2);
        __builtin_amdgcn_sched_barrier(0);
        int s = 0;
        for (; s + 2 <= nsteps; s += 2) {
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const int q = r ^ 1;
            ld_x(s + r + 1, xi[q], xv[q]);
            ld_val(s + r + 1, vh[q], vl[q]);
            xi[q] = ld_idx(s + r + 3);
            __builtin_amdgcn_sched_barrier(0);
            mma(vh[r], vl[r], xv[r]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (s < nsteps) mma(vh[0], vl[0], xv[0]);
        double mmv[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int pr = mt * 16 + dst_row<float>(kg, i);
          if (pr < b) {
            const int64_t r = (int64_t)rd.yrow + pr;
            const int64_t cc = c0 + 4 * m;
            float4 y = {float(P.alpha) * acc[0][i], float(P.alpha) * acc[1][i],
                        float(P.alpha) * acc[2][i], float(P.alpha) * acc[3][i]};
            if (P.beta != 0.0) {
              const float4 q = *reinterpret_cast<const float4 *>(P.Yin + r * P.ldyin + cc);
              const float be = float(P.beta);
              y.x = fmaf(be, q.x, y.x);
              y.y = fmaf(be, q.y, y.y);
              y.z = fmaf(be, q.z, y.z);
              y.w = fmaf(be, q.w, y.w);
            }
            *reinterpret_cast<float4 *>(P.Yout + r * P.ldy + cc) = y;
            if (MOM) {
              const float4 q = *reinterpret_cast<const float4 *>(P.R + r * P.ldr + cc);
              mmv[0] += (double)q.x * (double)y.x;
              mmv[1] += (double)q.y * (double)y.y;
              mmv[2] += (double)q.z * (double)y.z;
              mmv[3] += (double)q.w * (double)y.w;
            }
          }
        }
        if (MOM) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            double mm = mmv[t];
            mm += __shfl_xor(mm, 16, 64);
            mm += __shfl_xor(mm, 32, 64);
            if (kg == 0) s_mom[w * P.nrhs + c0 + 4 * m + t] += mm;
          }
        }
      }
    }
  }
  mom_flush<MOM>(s_mom, P.nrhs, wg, P.mom);
}

// ---------------------------------------------------------------------------
// value packing: graph order (row-major blocks) -> pages
// ---------------------------------------------------------------------------
// One wave per run of kPackRun consecutive graph blocks (their values are
// contiguous in graph order): lane l takes elements l, l + 64, ... of the
// run, so every lane is busy whatever the block sizes and the loads of
// different elements are independent (the loop is unrolled four times to keep
// four in flight per lane).  A lane finds its block by comparing the element
// with the run's block starts (wave-uniform, in scalar registers) and reads
// the block's map from a wave-private LDS table.  For the FP64/FP32 pages one
// sweep in row-major order (the order of the source) writes the transposed
// pages as a contiguous copy and the forward pages (each block transposed)
// inside each block's own contiguous range.  BF16 pages (8-column groups)
// take one sweep per direction, each in the order in which its writes are
// contiguous.  Row and column of an element come from a reciprocal of the
// block width, corrected by one step (exact for offsets below 2^12 and
// widths up to 64).
constexpr int kPackRun = 8;
constexpr int kPackChunk = 4;

// Output map of panel column kk for the block-sampled product written in the
// forward pages' layout: column kk of the panel starts at vbase + kk * b and
// its rows are consecutive (stride 1).
__device__ __forceinline__ int64_t page_map(const RowDesc &rd, int kk) {
  return ((rd.vbase + (int64_t)kk * rd.b) << 7) | 1;
}

__device__ __forceinline__ void pack_store(const PackDir &D, int kind, int64_t pos, int k0,
                                           int64_t vb16, int h, int r, int c, double v) {
  if (kind == 2) {
    const int col = k0 + c;
    const int64_t a = vb16 + (int64_t)(col >> 3) * 8 * h + r * 8 + (col & 7);
    const float f = (float)v;
    const unsigned short hb = bf16_rne(f);
    static_cast<uint16_t *>(D.dst)[a] = hb;
    D.dst_lo[a] = bf16_rne(f - bf16_to_f32(hb));
  } else {
    const int64_t a = pos + (int64_t)c * h + r;
    if (kind == 0)
      static_cast<double *>(D.dst)[a] = v;
    else
      static_cast<float *>(D.dst)[a] = (float)v;
  }
}

struct PackRec {       // one block of a run, in LDS
  int32_t start;       // run-relative first value (graph order)
  int32_t bi, bj;
  int32_t kf, kt;      // BF16: first panel column, forward / transposed
  int32_t pad[3];
  int64_t pf, pt;      // page offset, forward / transposed
  int64_t vf, vt;      // BF16: panel base in the BF16 pages, forward / transposed
};
static_assert(sizeof(PackRec) == 64, "PackRec layout");

template <int SRC, int KIND>  // SRC 0/1: double/float source; KIND: dst_kind
__global__ void __launch_bounds__(kThreads) k_pack(PackParams P, const void *src) {
  __shared__ PackRec tab_all[kWaves * kPackRun];
  const int64_t k0 = ((int64_t)blockIdx.x * kWaves + wave_id()) * kPackRun;
  if (k0 >= P.nnzb) return;
  const int lane = threadIdx.x & 63;
  const int nb = (int)min((int64_t)kPackRun, P.nnzb - k0);
  PackRec *tab = tab_all + wave_id() * kPackRun;
  // lanes 0 .. nb-1 read one block's map each into the table
  int64_t g = 0;
  int n = 0;
  PackRec r{};
  if (lane < nb) {
    const int64_t k = k0 + lane;
    r.bi = P.b[P.blk_row[k]];
    r.bj = P.b[P.col_idx[k]];
    g = P.gbase[k];
    r.pf = P.dir[0].pos[k];
    r.pt = P.dir[1].pos[k];
    if (KIND == 2) {
      r.kf = P.dir[0].k0[k];
      r.kt = P.dir[1].k0[k];
      r.vf = P.dir[0].vbase16[P.dir[0].prow[k]];
      r.vt = P.dir[1].vbase16[P.dir[1].prow[k]];
    }
    n = r.bi * r.bj;
  }
  const int64_t g0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(g >> 32), 0) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)g, 0));
  const int start = (int)(g - g0);   // run-relative first value (lanes < nb)
  if (lane < nb) {
    r.start = start;
    tab[lane] = r;
  }
  wave_lds_sync();
  int st[kPackRun];   // block starts (wave-uniform; past nb: beyond the run)
  const int len = __builtin_amdgcn_readlane(start + n, nb - 1);
#pragma unroll
  for (int u = 0; u < kPackRun; ++u) st[u] = u < nb ? __builtin_amdgcn_readlane(start, u) : len;
  auto load = [&](int64_t at) {
    if constexpr (SRC == 0)
      return static_cast<const double *>(src)[at];
    else
      return (double)static_cast<const float *>(src)[at];
  };
  // sweep 0 in row-major order, sweep 1 (BF16 only) in column-major order.
  // Elements go in chunks of kPackChunk per lane: every load of a chunk is
  // issued before its first store, so a lane waits once per chunk (a lane
  // has only a few elements when blocks are small).
  for (int sweep = 0; sweep < (KIND == 2 ? 2 : 1); ++sweep) {
    for (int e0 = lane; e0 < len; e0 += 64 * kPackChunk) {
      double v[kPackChunk];
      int tt[kPackChunk], pp[kPackChunk], qq[kPackChunk];
#pragma unroll
      for (int c = 0; c < kPackChunk; ++c) {
        const int e = e0 + 64 * c;
        const int ec = e < len ? e : len - 1;
        int t = 0;
#pragma unroll
        for (int u = 1; u < kPackRun; ++u) t += ec >= st[u] ? 1 : 0;
        const PackRec &rt = tab[t];
        const int b1 = rt.bi, b2 = rt.bj;
        const int loc = ec - rt.start;
        int p, q;
        if (sweep == 0) {   // row-major: p = loc / b2
          p = (int)((float)loc * __builtin_amdgcn_rcpf((float)b2));
          q = loc - p * b2;
          if (q >= b2) { ++p; q -= b2; }
        } else {            // column-major: q = loc / b1
          q = (int)((float)loc * __builtin_amdgcn_rcpf((float)b1));
          p = loc - q * b1;
          if (p >= b1) { ++q; p -= b1; }
        }
        tt[c] = t;
        pp[c] = p;
        qq[c] = q;
        // row-major sweep: the source is read in its own order (the load
        // does not wait on the block lookup)
        v[c] = load(g0 + (sweep == 0 ? (int64_t)ec : (int64_t)rt.start + (int64_t)p * b2 + q));
      }
#pragma unroll
      for (int c = 0; c < kPackChunk; ++c) {
        if (e0 + 64 * c >= len) break;
        const PackRec &rt = tab[tt[c]];
        const int b1 = rt.bi, b2 = rt.bj, p = pp[c], q = qq[c];
        if (KIND != 2) {
          // transposed panel of atom j: height b_j, row q, column k0 + p
          pack_store(P.dir[1], KIND, rt.pt, 0, 0, b2, q, p, v[c]);
          // forward panel of atom i: height b_i, row p, column k0 + q
          pack_store(P.dir[0], KIND, rt.pf, 0, 0, b1, p, q, v[c]);
        } else if (sweep == 0) {
          pack_store(P.dir[0], KIND, rt.pf, rt.kf, rt.vf, b1, p, q, v[c]);
        } else {
          pack_store(P.dir[1], KIND, rt.pt, rt.kt, rt.vt, b2, q, p, v[c]);
        }
      }
    }
  }
}

// Rebuild of the transposed pages from the forward pages, walking the
// transposed pages: rec[u] describes the block at transposed-page position u
// (its forward-page and transposed-page offsets and its shape), so a wave
// reads its run's maps with one load per lane before its element loads.
__global__ void __launch_bounds__(kThreads) k_refresh_records(PackParams P, const int32_t *order,
                                                              PageRec *rec) {
  const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (u >= P.nnzb) return;
  const int32_t k = order[u];
  PageRec r;
  r.src = P.dir[0].pos[k];
  r.dst = P.dir[1].pos[k];
  r.bi = P.b[P.blk_row[k]];
  r.bj = P.b[P.col_idx[k]];
  r.pad[0] = r.pad[1] = 0;
  rec[u] = r;
}

// Blocks lane u < nb (record r) of a wave, column-major at the source, row-major
// at the destination; the records go through `tab` (the wave's LDS).
template <typename T>
__device__ __forceinline__ void transpose_run(const PageRec &r, PageRec *tab, int nb, int lane,
                                              int part, int parts, const T *src, T *dst) {
  int n = 0;
  if (lane < nb) {
    n = r.bi * r.bj;
    tab[lane] = r;
  }
  int incl = n;
#pragma unroll
  for (int o = 1; o < kPackRun; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  const int start = incl - n;
  wave_lds_sync();
  int st[kPackRun];
  const int len = __builtin_amdgcn_readlane(incl, nb - 1);
#pragma unroll
  for (int u = 0; u < kPackRun; ++u) st[u] = u < nb ? __builtin_amdgcn_readlane(start, u) : len;
  for (int e0 = 64 * kPackChunk * part + lane; e0 < len; e0 += 64 * kPackChunk * parts) {
    T v[kPackChunk];
    int64_t d[kPackChunk];
#pragma unroll
    for (int c = 0; c < kPackChunk; ++c) {
      const int e = min(e0 + 64 * c, len - 1);
      int t = 0, stt = 0;
#pragma unroll
      for (int u = 1; u < kPackRun; ++u)
        if (e >= st[u]) {
          t = u;
          stt = st[u];
        }
      const PageRec &q0 = tab[t];
      const int b1 = q0.bi, b2 = q0.bj, l = e - stt;
      // element (p, q): row-major at the destination, column-major at the source
      int p = (int)((float)l * __builtin_amdgcn_rcpf((float)b2));
      int q = l - p * b2;
      if (q >= b2) { ++p; q -= b2; }
      v[c] = src[q0.src + (int64_t)q * b1 + p];
      d[c] = q0.dst + l;
    }
#pragma unroll
    for (int c = 0; c < kPackChunk; ++c) {
      if (e0 + 64 * c >= len) break;
      dst[d[c]] = v[c];
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_refresh(const PageRec *rec, int64_t nnzb,
                                                      const T *src, T *dst) {
  __shared__ PageRec tab_all[kWaves * kPackRun];
  const int64_t u0 = ((int64_t)blockIdx.x * kWaves + wave_id()) * kPackRun;
  if (u0 >= nnzb) return;
  const int lane = threadIdx.x & 63;
  const int nb = (int)min((int64_t)kPackRun, nnzb - u0);
  // every lane holds a record: one filled in part of the lanes goes through LDS,
  // whose address then needs the dispatch packet in host memory (13 us a call)
  const PageRec r = rec[u0 + min(lane, nb - 1)];
  transpose_run<T>(r, tab_all + wave_id() * kPackRun, nb, lane, 0, 1, src, dst);
}

// ---------------------------------------------------------------------------
// block-sampled dY X^T on matrix cores, one wave per forward panel
// ---------------------------------------------------------------------------
// For block row i the result is the b_i x K_i panel dY_i Xg_i^T, Xg_i the X
// rows of the panel's columns: a 16 x 16 output tile per MFMA chain with
// M = panel rows, N = 16 panel columns, K = right-hand sides.  Lane (m, kq)
// holds 8 of the right-hand sides of each 32-wide chunk, the same ones for
// both operands (the contraction order inside a chunk is permuted, the sum
// is the same).  Each output goes to graph order through colg = (graph
// offset of the column's block + q) << 7 | b_j.
template <typename T, int NCH>
__global__ void __launch_bounds__(kThreads) k_sddmm_mfma(SddmmParams<T> P) {
  using V = typename Frag<T>::type;
  const int row = xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (row >= P.nrows) return;
  const int lane = threadIdx.x & 63;
  const int m = lane & 15;
  const int kq = lane >> 4;
  const RowDesc rd = P.rows[row];
  const int b = rd.b, K = rd.K;
  if (K == 0) return;
  const int nch = (P.nrhs + 31) >> 5;
  const int ntiles = (K + 15) >> 4;
  const int32_t *__restrict__ cx = P.colx + rd.cbase;
  const int64_t *__restrict__ cg = P.colg + rd.cbase;
  for (int mt = 0; mt * 16 < b; ++mt) {
    const int p = mt * 16 + m;
    const T *dyrow = P.dY + ((int64_t)rd.yrow + (p < b ? p : b - 1)) * P.lddy;
    // lane group kq holds 8 right-hand sides of each 32-wide chunk, the same
    // ones for both operands: FP64 takes c = 32 ch + 8 l + 2 kq + e (l < 4,
    // e < 2), so the four lane groups of one 16-byte load read 64 contiguous
    // bytes of a row; FP32 takes c = 32 ch + 8 kq + s (two 16-byte loads)
    constexpr bool PAIR = sizeof(T) == 8;
    const int kofs = PAIR ? 2 * kq : 8 * kq;
    auto ldrun = [&](const T *src, int ch, bool ok, T *dst) {
      const int cb = ch * 32 + kofs;
      auto rhs = [&](int s) { return PAIR ? cb + 8 * (s >> 1) + (s & 1) : cb + s; };
      if (ch * 32 + 32 <= P.nrhs) {
#pragma unroll
        for (int s = 0; s < 8; ++s) dst[s] = src[rhs(s)];
#pragma unroll
        for (int s = 0; s < 8; ++s) dst[s] = ok ? dst[s] : T(0);
      } else {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const int c = rhs(s);
          const T v = src[min(c, P.nrhs - 1)];
          dst[s] = (ok && c < P.nrhs) ? v : T(0);
        }
      }
    };
    // A fragments (dY rows) of the first NCH 32-wide chunks stay in registers
    T af[NCH][8];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) ldrun(dyrow, ch, p < b && ch < nch, af[ch]);
    // one 16-column tile: B fragments of chunk 0/1 and the output map
    struct Tile {
      T bv[NCH][8];
      const T *xrow;
      int64_t g;
      bool kin;
    };
    auto load_tile = [&](int j, Tile &tl) {
      const int kc = j * 16 + m;
      tl.kin = kc < K;
      const int kk = tl.kin ? kc : K - 1;
      tl.xrow = P.X + (int64_t)cx[kk] * P.ldx;
      tl.g = P.page_out ? page_map(rd, kk) : cg[kk];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) ldrun(tl.xrow, ch, tl.kin && ch < nch, tl.bv[ch]);
    };
    // one tile's products, split over two independent accumulator chains
    auto do_tile = [&](const Tile &tl) {
      V acc0 = V{}, acc1 = V{};
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
        for (int s = 0; s < 8; s += 2) {
          acc0 = mfma(af[ch][s], tl.bv[ch][s], acc0);
          acc1 = mfma(af[ch][s + 1], tl.bv[ch][s + 1], acc1);
        }
      for (int ch = NCH; ch < nch; ++ch) {
        T av[8], bv[8];
        ldrun(dyrow, ch, p < b, av);
        ldrun(tl.xrow, ch, tl.kin, bv);
#pragma unroll
        for (int s = 0; s < 8; s += 2) {
          acc0 = mfma(av[s], bv[s], acc0);
          acc1 = mfma(av[s + 1], bv[s + 1], acc1);
        }
      }
      if (tl.kin) {
        const int64_t base = tl.g >> 7;
        const int bj = (int)(tl.g & 127);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int pr = mt * 16 + dst_row<T>(kq, i);
          if (pr < b) P.dA[base + (int64_t)pr * bj] = acc0[i] + acc1[i];
        }
      }
    };
    // one tile at a time: other waves hide the load latency (a prefetched
    // second tile raised register use enough to cost more than it hid)
    for (int j = 0; j < ntiles; ++j) {
      Tile t0;
      load_tile(j, t0);
      do_tile(t0);
    }
  }
}

// ---------------------------------------------------------------------------
// block-sampled dY X^T with the X rows of each tile staged in LDS
// ---------------------------------------------------------------------------
// Same products, accumulation order and output map as k_sddmm_mfma; only the
// way X reaches the B operand differs.  A tile's 16 X rows (CW right-hand
// sides each) are loaded with whole-row pieces -- 64 / (CW / EPL) rows per
// load instruction, EPL elements (16 bytes) per lane -- instead of 16 rows
// per instruction, written to a wave-private LDS tile (rows padded by EPL
// elements, so the fragment reads of the 16 rows hit distinct banks) and read
// back in the MFMA fragment order.  For more than 64 right-hand sides, in
// passes of CW (and for 33 to 64 with a leading dimension of dY of 2^22 or
// more, which the kernel below does not address).  X is addressed through one
// buffer descriptor (all of X within 2^31 bytes): reads past its end return
// zero.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_sddmm_lds(SddmmParams<T> P) {
  using V = typename Frag<T>::type;
  constexpr int CW = 64;                       // right-hand sides per pass
  constexpr int NCH = CW / 32;                 // 32-wide chunks per pass
  constexpr int EPL = 16 / (int)sizeof(T);     // elements per 16-byte piece
  constexpr int LPR = CW / EPL;                // lanes per staged row
  constexpr int RPI = 64 / LPR;                // rows per staging load
  constexpr int RS = CW + EPL;                 // LDS row stride (elements)
  __shared__ __align__(16) T xs_all[kWaves * 16 * RS];
  const int row = xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (row >= P.nrows) return;
  const int lane = threadIdx.x & 63;
  const int m = lane & 15;
  const int kq = lane >> 4;
  T *xs = xs_all + wave_id() * 16 * RS;
  const RowDesc rd = P.rows[row];
  const int b = rd.b, K = rd.K;
  if (K == 0) return;
  const int ntiles = (K + 15) >> 4;
  const int npass = (P.nrhs + CW - 1) / CW;
  const int32_t *__restrict__ cx = P.colx + rd.cbase;
  const int64_t *__restrict__ cg = P.colg + rd.cbase;
  const __amdgpu_buffer_rsrc_t rx =
      panel_rsrc(P.X, (uint32_t)(((P.xrows - 1) * P.ldx + P.nrhs) * (int64_t)sizeof(T)));
  // contraction order inside a 32-wide chunk (the same for both operands):
  // FP64 c = 8 l + 2 kq + e (l < 4, e < 2), FP32 c = 8 kq + s
  constexpr bool PAIR = sizeof(T) == 8;
  const int kofs = PAIR ? 2 * kq : 8 * kq;
  auto rhs = [&](int ch, int s) { return ch * 32 + kofs + (PAIR ? 8 * (s >> 1) + (s & 1) : s); };
  const int sr = lane / LPR;            // staging: row within a load
  const int se = (lane % LPR) * EPL;    // staging: first element of the piece
  for (int mt = 0; mt * 16 < b; ++mt) {
    const int p = mt * 16 + m;
    const T *dyrow = P.dY + ((int64_t)rd.yrow + (p < b ? p : b - 1)) * P.lddy;
    T af[NCH][8];
    auto load_af = [&](int c0) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const int c = c0 + rhs(ch, s);
          const T v = dyrow[min(c, P.nrhs - 1)];
          af[ch][s] = (p < b && c < P.nrhs) ? v : T(0);
        }
    };
    if (npass == 1) load_af(0);
    for (int j = 0; j < ntiles; ++j) {
      // lane r (and r + 16, r + 32, r + 48) holds tile column r
      const int kc = j * 16 + m;
      const int kk = kc < K ? kc : K - 1;
      const int32_t xr = cx[kk];
      const int64_t g = P.page_out ? page_map(rd, kk) : cg[kk];
      V acc0 = V{}, acc1 = V{};
      for (int pass = 0; pass < npass; ++pass) {
        const int c0 = pass * CW;
        if (npass > 1) load_af(c0);
        // stage the tile's 16 rows x CW right-hand sides
        typename Vec16<T>::type v[16 / RPI];
#pragma unroll
        for (int it = 0; it < 16 / RPI; ++it) {
          const int r = it * RPI + sr;
          const int32_t xrow = __shfl(xr, r, 64);
          const int c = c0 + se;
          const uint32_t off = (j * 16 + r < K && c < P.nrhs)
                                   ? (uint32_t)(((int64_t)xrow * P.ldx + c) * (int64_t)sizeof(T))
                                   : 0x80000000u;
          v[it] = __builtin_bit_cast(typename Vec16<T>::type,
                                     __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
        }
#pragma unroll
        for (int it = 0; it < 16 / RPI; ++it) {
          const int r = it * RPI + sr;
          const int c = c0 + se;
          T *e = reinterpret_cast<T *>(&v[it]);
#pragma unroll
          for (int q = 0; q < EPL; ++q) e[q] = c + q < P.nrhs ? e[q] : T(0);
          *reinterpret_cast<typename Vec16<T>::type *>(xs + r * RS + se) = v[it];
        }
        wave_lds_sync();
        T bv[NCH][8];
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
          for (int s = 0; s < 8; ++s) bv[ch][s] = xs[m * RS + rhs(ch, s)];
        wave_lds_sync();  // every read done before the next staging
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
          for (int s = 0; s < 8; s += 2) {
            acc0 = mfma(af[ch][s], bv[ch][s], acc0);
            acc1 = mfma(af[ch][s + 1], bv[ch][s + 1], acc1);
          }
      }
      if (kc < K) {
        const int64_t base = g >> 7;
        const int bj = (int)(g & 127);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int pr = mt * 16 + dst_row<T>(kq, i);
          if (pr < b) P.dA[base + (int64_t)pr * bj] = acc0[i] + acc1[i];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// block-sampled dY X^T, X rows loaded straight into LDS, outputs through LDS
// ---------------------------------------------------------------------------
// One wave per panel, up to 64 right-hand sides: 16 panel rows x 16 panel
// columns per tile on matrix cores.  A step is one tile and one chunk of PR
// 16-byte pieces of right-hand sides (NCH chunks); its 16 X row pieces go to a
// wave-private LDS buffer by buffer-to-LDS loads, which hold no registers
// while in flight, adjacent lanes reading adjacent pieces of a row (a load
// whose neighbouring lanes read different rows costs four times the tag
// lookups: X straight to registers in fragment order took 324 us where this
// takes 299).  The next step's loads are issued as soon as the fragments are
// in registers.  Lane (m, kq) holds pieces kq + 4 h of row m for both operands.
//
// How the outputs leave, NS > 0 through LDS, NS < 0 straight from the
// accumulators in -NS stores:
//   * PAGE (the forward pages' layout), b <= 16: a tile's outputs are one run,
//     stored 16 bytes a lane.
//   * PAGE, taller panels, 16 rows at a time: X is the row operand, so that a
//     lane's column of the tile is a panel row and a store writes 16
//     consecutive rows of 4 columns (b = 64, 32 right-hand sides, FP32: 281 ->
//     194 us; b = 33 199 -> 149); the rows left over as in graph order.
//   * Graph order: 16 columns of 4 rows a store, or through a ring of RS
//     outputs in panel order (block by block, each row-major) with their graph
//     offsets; whole blocks are stored, 64 NS outputs a tile, a block that runs
//     on into the next tile waits for its end.  At most (bj - 1) b wait as a
//     block's first columns and as many for their turn, and a tile spans up to
//     16 + 2 (bj - 1) columns' outputs: b (3 bj + 13) < RS keeps them apart and
//     one entry free, bj the panel's widest block.
//   * NS = kHold (FP64, graph order, b = 11 to 47, outputs that go to
//     memory): the columns of a block that runs on into the next tile wait for
//     it in registers, so that a block's lines are written at once (b = 13, 64
//     right-hand sides, 32,768 rows: 638 -> 603 us; 13,824 rows 273 -> 258).
//   * NS = kWide: by 64-bit addresses (panels of 1 GiB and more).
// The ring's turn through LDS takes as long as a tile's matrix instructions, so
// it is for outputs that go to memory: see the launcher.
//
// Against kernels for 32 and 64 right-hand sides with scattered stores, and one
// that staged X through registers for the other counts: b = 1/4/9, K about 150,
// 32 right-hand sides, FP32, 100,000 panels, graph order 357 -> 309 us, pages
// 287 -> 235; FP64, 50,000 panels 297 -> 264 and 235 -> 221; 40 right-hand sides
// FP64 544 -> 385; b = 4/9, 8,000 panels, 7 right-hand sides, FP64, 89 -> 38,
// pages 86 -> 33; b = 13 lattice, 64, FP64 pages 633 -> 524.
// Values of NS: the form that holds outputs back, and that with 64-bit addresses.
constexpr int kHold = -8, kWide = 0;
// Outputs of this size and more go to memory, not to the 256 MB Infinity Cache.
constexpr int64_t kMemoryBytes = 192 << 20;

template <typename T, int PR, int NCH, bool PAGE, int RS, int NS>
__device__ __forceinline__ void sddmm_panel(const SddmmParams<T> &P, const RowDesc &rd, int m0,
                                            uint32_t xbytes, T *xs, T *ring, int32_t *aring) {
  using LdsPtr = __attribute__((address_space(3))) void *;
  using V = typename Frag<T>::type;
  using L16 = typename Vec16<T>::type;
  constexpr int EPL = 16 / (int)sizeof(T);   // elements of a piece
  constexpr uint32_t ES = sizeof(T);
  constexpr int NIT = PR / 4;                // load instructions of a step
  const int lane = threadIdx.x & 63;
  const int m = lane & 15, kq = lane >> 4;
  const int b = rd.b, K = rd.K;
  const __amdgpu_buffer_rsrc_t rc = panel_rsrc(P.colx + rd.cbase, (uint32_t)K * 4u);
  const __amdgpu_buffer_rsrc_t rg = panel_rsrc(PAGE ? nullptr : P.colg + rd.cbase, (uint32_t)K * 8u);
  const __amdgpu_buffer_rsrc_t rx = panel_rsrc(P.X, xbytes);
  // graph offset of the panel's first column; outputs lie within b K of it
  const int64_t g0 = PAGE ? 0 : P.colg[rd.cbase] >> 7;
  const uint32_t bk = (uint32_t)b * (uint32_t)K;
  const __amdgpu_buffer_rsrc_t ro =
      PAGE ? panel_rsrc(P.dA + rd.vbase, ((bk + 3) & ~3u) * ES)
           : panel_rsrc(P.dA + (g0 - (int64_t)bk), NS == kWide ? 0 : 2 * bk * ES);
  // the 64 / PR lane groups (group = lane / PR) stage rows NIT group + it of a
  // tile with load it; lane i of every four loads the index of row NIT group + i
  const int grp = lane / PR;
  auto rows_of = [&](int j) {
    return __builtin_amdgcn_raw_buffer_load_b32(rc, (uint32_t)(16 * j + NIT * grp + (lane & 3)) * 4u, 0, 0);
  };
  auto gmap_of = [&](int j) {
    if constexpr (PAGE)
      return v2u32{0u, 0u};
    else
      return __builtin_bit_cast(v2u32, __builtin_amdgcn_raw_buffer_load_b64(rg, (uint32_t)(16 * j + m) * 8u, 0, 0));
  };
  // pieces sit permuted in their LDS row, so that one piece index of the 16
  // rows covers all banks
  auto perm = [](int r) { return PR == 16 ? r : PR == 8 ? ((r >> 2) << 1 | (r & 1)) : r >> 2; };
  uint32_t xcol[NCH][NIT];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int c = EPL * (PR * ch + ((lane % PR) ^ perm(NIT * grp + it)));
      xcol[ch][it] = c < P.nrhs ? (uint32_t)c * ES : kOutCol;
    }
  auto issue = [&](int j, int ch, int32_t xi) {
    const int32_t xo = 16 * j + NIT * grp + (lane & 3) < K
                           ? (int32_t)(uint32_t)((int64_t)xi * P.ldx * (int64_t)ES)
                           : (int32_t)kOutRow;
#pragma unroll
    for (int it = 0; it < NIT; ++it)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (LdsPtr)(xs + it * 64 * EPL), 16,
                                               (uint32_t)quad_bcast(xo, it) + xcol[ch][it], 0, 0, 0);
  };
  // dY: rows past the panel and right-hand sides past nrhs are zero
  T af[NCH][NIT][EPL];
  {
    const __amdgpu_buffer_rsrc_t rdy =
        panel_rsrc(P.dY + (int64_t)rd.yrow * P.lddy, (uint32_t)((b - 1) * P.lddy + P.nrhs) * ES);
    const uint32_t yo = m0 + m < b ? (uint32_t)((m0 + m) * P.lddy) * ES : kOutRow;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
      for (int h = 0; h < NIT; ++h) {
        const int c = EPL * (PR * ch + 4 * h + kq);
        const L16 v = __builtin_bit_cast(
            L16, __builtin_amdgcn_raw_buffer_load_b128(rdy, yo + (c < P.nrhs ? (uint32_t)c * ES : kOutCol), 0, 0));
#pragma unroll
        for (int e = 0; e < EPL; ++e)
          af[ch][h][e] = c + e < P.nrhs ? reinterpret_cast<const T *>(&v)[e] : T(0);
      }
  }
  const bool ragged = P.nrhs % EPL != 0;
  constexpr bool kSwap = PAGE && NS == -4;   // X is the row operand
  // two chunks a tile: its outputs leave during the next tile's first chunk,
  // behind that chunk's loads (b = 8, 64 right-hand sides 131 -> 120 us)
  constexpr bool kLate = PAGE && NS > 0 && NCH == 2;
  const int nt = (K + 15) >> 4;
  int sprev = 0, F = 0;        // first column of the block at a tile's start; outputs flushed
  int32_t uprev = -1;
  // graph offset of a column relative to g0 (at most a panel's size: 32 bits)
  auto rel = [&](const v2u32 &g) {
    return (int32_t)(__builtin_amdgcn_alignbit(g.y, g.x, 7) - (uint32_t)g0);
  };
  // every lane issues its stores, those without an output past the range
  // (no store): the number of stores in flight is then known at each wait
  auto put = [&](T v, uint32_t e, bool ok) {
    const uint32_t off = e * ES | (ok ? 0u : 0xF0000000u);
    if constexpr (sizeof(T) == 8)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u32, v), ro, off, 0, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), ro, off, 0, 0);
  };
  // kHold: sums of the tile before whose block runs on, in lanes m >= csplit
  V carry = V{};
  bool held = false;
  uint32_t ca = 0;
  int cbj = 0, csplit = 16;
  auto flush = [&](int e, int E) {
    const T v = ring[e & (RS - 1)];
    put(v, (uint32_t)aring[e & (RS - 1)], e < E);
  };
  auto out = [&](int j, const V &acc, const v2u32 &g, const v2u32 &gn) {
    const int k = 16 * j + m;
    if constexpr (PAGE && NS > 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = dst_row<T>(kq, i);
        if (p < b) ring[m * b + p] = acc[i];
      }
      wave_lds_sync();
      const uint32_t nst = j < 0 ? 0u : (uint32_t)(min(K - 16 * j, 16) * b);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const uint32_t e = (uint32_t)EPL * (64 * i + lane);
        L16 v = *reinterpret_cast<const L16 *>(ring + (e & (RS - 1)));
        T *ve = reinterpret_cast<T *>(&v);
#pragma unroll
        for (int q = 0; q < EPL; ++q) ve[q] = e + q < nst ? ve[q] : T(0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u32, v), ro,
                                               e < nst ? (16u * j * b + e) * ES : 0xF0000000u, 0, 0);
      }
      wave_lds_sync();
    } else if constexpr (NS > 0) {
      const int32_t u = rel(g);
      const int bj = (int)(g.x & 127);
      const int32_t up = __builtin_amdgcn_update_dpp(uprev, u, 0x111, 0xF, 0xF, false);  // row_shr:1
      const uint32_t brk = (uint32_t)__ballot(k < K && u != up + 1) & 0xFFFFu;
      const uint32_t below = brk & ((2u << m) - 1u);
      const int sc = below ? 16 * j + 31 - __builtin_clz(below) : sprev;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = dst_row<T>(kq, i);
        // lanes without an output write to the entry before the oldest one
        const int at = (p < b && k < K ? b * sc + p * bj + k - sc : F - 1) & (RS - 1);
        ring[at] = acc[i];
        aring[at] = u + p * bj + (int32_t)bk;
      }
      wave_lds_sync();
      sprev = __builtin_amdgcn_readlane(sc, 15);
      uprev = __builtin_amdgcn_readlane(u, 15);
      const bool cont = j + 1 < nt && __builtin_amdgcn_readlane(rel(gn), 0) == uprev + 1 && b > 1;
      const int E = cont ? b * sprev : b * min(16 * (j + 1), K);
#pragma unroll
      for (int i = 0; i < NS; ++i) flush(F + 64 * i + lane, E);
      F = min(E, F + 64 * NS);
      wave_lds_sync();
    } else if constexpr (kSwap) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 16 * j + dst_row<T>(kq, i);
        put(acc[i], (uint32_t)(c * b + m0 + m), m0 + m < b && c < K);
      }
    } else if constexpr (NS == kHold) {
      const int32_t u = rel(g);
      const int bj = (int)(g.x & 127);
      const uint32_t a = (uint32_t)u + bk;
      const int32_t up = __builtin_amdgcn_update_dpp(u, u, 0x111, 0xF, 0xF, false);  // row_shr:1
      const uint32_t brk = ((uint32_t)__ballot(u != up + 1) & 0xFFFFu) | 1u;
      const bool cont = j + 1 < nt && __builtin_amdgcn_readlane(rel(gn), 0) ==
                                          __builtin_amdgcn_readlane(u, 15) + 1;
      const int split = cont ? 31 - __builtin_clz(brk) : 16;
      if (csplit < 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int p = m0 + dst_row<T>(kq, i);
          put(carry[i], ca + (uint32_t)(p * cbj), p < b && m >= csplit);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = m0 + dst_row<T>(kq, i);
        put(acc[i], a + (uint32_t)(p * bj), p < b && k < K && m < split);
      }
      held = csplit < 16;
      carry = acc;
      ca = a;
      cbj = bj;
      csplit = split;
    } else if constexpr (NS < 0) {
      const uint32_t a = PAGE ? (uint32_t)(k * b) : (uint32_t)rel(g) + bk;
      const int bj = PAGE ? 1 : (int)(g.x & 127);
#pragma unroll
      for (int i = 0; i < -NS; ++i) {
        const int p = m0 + dst_row<T>(kq, i);
        put(acc[i], a + (uint32_t)(p * bj), p < b && k < K);
      }
    } else {
      if (k < K) {
        const int64_t a = PAGE ? rd.vbase + (int64_t)k * b : g0 + rel(g);
        const int bj = PAGE ? 1 : (int)(g.x & 127);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int p = m0 + dst_row<T>(kq, i);
          if (p < b) P.dA[a + (int64_t)p * bj] = acc[i];
        }
      }
    }
  };
  const T *xm = xs + ((m % NIT) * 64 + (m / NIT) * PR) * EPL;   // row m in LDS
  // indices and maps of tile j + 1 are loaded ahead of tile j's X rows: they
  // have arrived when the rows have, and move along then.  The fragments of a
  // step are read at the end of the step before, after its stores: there the
  // number of stores behind the rows' loads is known, and the wait for the
  // rows leaves them in flight.
  L16 bv[NIT];
  auto fragments = [&](auto behind) {   // stores issued since the rows' loads
    // vmcnt(behind): the rows are in LDS; expcnt, lgkmcnt unchanged
    if constexpr (NS == kHold && decltype(behind)::value != 0) {
      if (held)
        __builtin_amdgcn_s_waitcnt(0x0F78);
      else
        __builtin_amdgcn_s_waitcnt(0x0F74);
    } else {
      __builtin_amdgcn_s_waitcnt(0x0F70 | decltype(behind)::value);
    }
#pragma unroll
    for (int h = 0; h < NIT; ++h)
      bv[h] = *reinterpret_cast<const L16 *>(xm + EPL * ((kq + 4 * h) ^ perm(m)));
    // the fragments are in registers before the buffer is refilled
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt, expcnt unchanged
  };
  int32_t xn = rows_of(0), xc = xn;
  v2u32 gp{}, gc = v2u32{0u, 0u}, gx = gmap_of(0);
  V done = V{};   // kLate: sums of the tile before
  int32_t xl = rows_of(1);
  v2u32 gl = gmap_of(1);
  issue(0, 0, xn);
  fragments(std::integral_constant<int, 0>{});
  for (int j = 0; j < nt; ++j) {
    V acc0 = V{}, acc1 = V{};
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      if (ch == 0) {
        gp = gc;
        gc = gx;
        gx = gl;
        xc = xn;
        xn = xl;
      }
      if (ch + 1 < NCH) {
        issue(j, ch + 1, xc);
      } else {
        xl = rows_of(j + 2);
        gl = gmap_of(j + 2);
        issue(j + 1, 0, xn);
      }
      // only arithmetic and LDS accesses may move across: the wait for these
      // loads counts the stores behind them
      __builtin_amdgcn_sched_barrier(0x8F);
      // right-hand sides past nrhs within a piece: what follows in X's row (a
      // branch: selecting in every step cost 5 % at 64 right-hand sides)
      if (ragged) {
#pragma unroll
        for (int h = 0; h < NIT; ++h) {
          T *xe = reinterpret_cast<T *>(&bv[h]);
#pragma unroll
          for (int e = 0; e < EPL; ++e)
            xe[e] = EPL * (PR * ch + 4 * h + kq) + e < P.nrhs ? xe[e] : T(0);
        }
      }
#pragma unroll
      for (int h = 0; h < NIT; ++h) {
        const T *xe = reinterpret_cast<const T *>(&bv[h]);
#pragma unroll
        for (int e = 0; e < EPL; e += 2) {
          const T a0 = af[ch][h][e], a1 = af[ch][h][e + 1];
          acc0 = kSwap ? mfma(xe[e], a0, acc0) : mfma(a0, xe[e], acc0);
          acc1 = kSwap ? mfma(xe[e + 1], a1, acc1) : mfma(a1, xe[e + 1], acc1);
        }
      }
      constexpr auto stores = std::integral_constant<int, (NS < 0 ? -NS : NS)>{};
      if constexpr (!kLate) {
        if (ch + 1 < NCH) {
          fragments(std::integral_constant<int, 0>{});
          continue;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc0[i] += acc1[i];
        out(j, acc0, gc, gx);
        fragments(stores);
      } else if (ch == 0) {
        out(j - 1, done, gp, gc);
        fragments(stores);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) done[i] = acc0[i] + acc1[i];
        fragments(std::integral_constant<int, 0>{});
      }
    }
  }
  if constexpr (kLate) out(nt - 1, done, gc, gx);
  if constexpr (!PAGE && NS > 0)
    for (; F < (int)bk; F += 64) flush(F + lane, (int)bk);
}

template <typename T, int PR, int NCH, bool PAGE, int RS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NCH == 2 ? 4 : 1)))
k_sddmm(SddmmParams<T> P, uint32_t xbytes) {
  constexpr int XE = 16 * PR * (16 / (int)sizeof(T));
  __shared__ __align__(16) T xs_all[kWaves * XE];
  __shared__ __align__(16) T ring_all[kWaves * RS];
  __shared__ int32_t aring_all[PAGE ? 1 : kWaves * RS];
  const int row = xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (row >= P.nrows) return;
  const RowDesc rd = P.rows[row];
  if (rd.K == 0) return;
  T *xs = xs_all + wave_id() * XE, *ring = ring_all + wave_id() * RS;
  int32_t *ra = aring_all + (PAGE ? 0 : wave_id() * RS);
  const int b = rd.b;
  if ((int64_t)b * rd.K * (int64_t)sizeof(T) >= (int64_t(1) << 30)) {
    for (int m0 = 0; m0 < b; m0 += 16)
      sddmm_panel<T, PR, NCH, PAGE, RS, kWide>(P, rd, m0, xbytes, xs, ring, ra);
    return;
  }
  if constexpr (PAGE) {
    if (b <= 16) {
      if (sizeof(T) == 4 || b <= 8)
        sddmm_panel<T, PR, NCH, PAGE, RS, 1>(P, rd, 0, xbytes, xs, ring, ra);
      else
        sddmm_panel<T, PR, NCH, PAGE, RS, 2>(P, rd, 0, xbytes, xs, ring, ra);
      return;
    }
  } else if constexpr (RS > 1) {
    // the panel's columns are in ascending order of their blocks' widths
    const int bj = (int)(P.colg[rd.cbase + rd.K - 1] & 127);
    if (b <= 12 && b * (3 * bj + 13) < RS) {
      if (b <= 4)
        sddmm_panel<T, PR, NCH, PAGE, RS, 1>(P, rd, 0, xbytes, xs, ring, ra);
      else
        sddmm_panel<T, PR, NCH, PAGE, RS, 3>(P, rd, 0, xbytes, xs, ring, ra);
      return;
    }
  }
  // straight from the accumulators: element i of a lane holds row kq + 4 i in
  // FP64 and 4 kq + i in FP32
  int m0 = 0;
  if constexpr (!PAGE && sizeof(T) == 8) {
    if (b > 10 && b < 48 && P.nnz * 8 >= kMemoryBytes)
      for (; m0 + 8 < b; m0 += 16)
        sddmm_panel<T, PR, NCH, PAGE, RS, kHold>(P, rd, m0, xbytes, xs, ring, ra);
  }
  for (; m0 < b; m0 += 16) {
    const int n = sizeof(T) == 8 ? (b - m0 + 3) / 4 : b - m0;
    if (n == 1)
      sddmm_panel<T, PR, NCH, PAGE, RS, -1>(P, rd, m0, xbytes, xs, ring, ra);
    else if (n == 2)
      sddmm_panel<T, PR, NCH, PAGE, RS, -2>(P, rd, m0, xbytes, xs, ring, ra);
    else
      sddmm_panel<T, PR, NCH, PAGE, RS, -4>(P, rd, m0, xbytes, xs, ring, ra);
  }
}

// ---------------------------------------------------------------------------
// column dot products in FP64 and their fixed-order reduction
// ---------------------------------------------------------------------------
constexpr int kDotRows = 256;

// One workgroup per kDotRows rows.  The threads form CL columns (the power of
// two at or above nrhs, at most 64) by kThreads / CL rows, so that every lane
// has work and every load of a wave is one run of row pieces; the row lanes'
// sums meet in LDS in a fixed order.  SAME: B is A, read once.  (With one
// thread per column three waves of four idled: <A, A> of 425,984 rows x 64
// floats 77 us, now 17.6, 6.2 TB/s.)
template <typename T, bool SAME>
__global__ void __launch_bounds__(kThreads) k_coldot(const T *A, int64_t lda, const T *B, int64_t ldb,
                                                     int64_t nrows, int32_t nrhs, int cl,
                                                     double *partial) {
  __shared__ double s[kThreads];
  const int64_t r0 = (int64_t)blockIdx.x * kDotRows;
  const int64_t r1 = min(r0 + kDotRows, nrows);
  const int tc = threadIdx.x & (cl - 1), tr = threadIdx.x / cl, nr = kThreads / cl;
  for (int c0 = 0; c0 < nrhs; c0 += cl) {
    const int c = c0 + tc;
    double t = 0.0;
    if (c < nrhs) {
#pragma unroll 8
      for (int64_t r = r0 + tr; r < r1; r += nr) {
        const double a = (double)A[r * lda + c];
        t += a * (SAME ? a : (double)B[r * ldb + c]);
      }
    }
    s[threadIdx.x] = t;
    __syncthreads();
    if (tr == 0 && c < nrhs) {
      for (int q = 1; q < nr; ++q) t += s[q * cl + tc];
      partial[(int64_t)blockIdx.x * nrhs + c] = t;
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kThreads) k_reduce(const double *partial, int64_t nparts,
                                                     int32_t nrhs, double *out) {
  __shared__ double s[kThreads];
  const int c = blockIdx.x;
  double t = 0.0;
  for (int64_t w = threadIdx.x; w < nparts; w += kThreads) t += partial[w * nrhs + c];
  s[threadIdx.x] = t;
  __syncthreads();
  for (int st = kThreads / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[c] = s[0];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int NR>
hipError_t launch_vec_nr(const FwdParams<T> &p0, hipStream_t s, dim3 grid, size_t shm) {
  FwdParams<T> p = p0;
  p.xrow16 = (reinterpret_cast<uintptr_t>(p.X) % 16 == 0 && (p.ldx * sizeof(T)) % 16 == 0) ? 1 : 0;
  if constexpr (use_vp<T, NR>()) {
    if (p.mom)
      hipLaunchKernelGGL((k_spmm_vp<T, NR, true>), grid, dim3(kThreads), shm, s, p);
    else
      hipLaunchKernelGGL((k_spmm_vp<T, NR, false>), grid, dim3(kThreads), 0, s, p);
  } else {
    if (p.mom)
      hipLaunchKernelGGL((k_spmm_vec<T, NR, true>), grid, dim3(kThreads), shm, s, p);
    else
      hipLaunchKernelGGL((k_spmm_vec<T, NR, false>), grid, dim3(kThreads), 0, s, p);
  }
  return hipGetLastError();
}

template <typename T, int NT, bool VX, bool XB>
hipError_t launch_mfma_xb(const FwdParams<T> &p, hipStream_t s, dim3 grid, size_t shm) {
  if (p.mom)
    hipLaunchKernelGGL((k_spmm_mfma<T, NT, true, VX, XB>), grid, dim3(kThreads), shm, s, p);
  else
    hipLaunchKernelGGL((k_spmm_mfma<T, NT, false, VX, XB>), grid, dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

// Whether the rows that the epilogue reads and writes start on 16-byte
// boundaries, and (vectorizable) the rows of X too, with the right-hand sides
// filling whole passes.
template <typename T>
bool out_rows16(const FwdParams<T> &p) {
  constexpr int VEC = 16 / sizeof(T);
  auto al = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  return al(p.Yout) && p.ldy % VEC == 0 && (p.beta == 0.0 || (al(p.Yin) && p.ldyin % VEC == 0)) &&
         (!p.mom || (al(p.R) && p.ldr % VEC == 0));
}
template <typename T>
bool vectorizable(const FwdParams<T> &p, int nt) {
  constexpr int VEC = 16 / sizeof(T);
  return p.nrhs % (16 * nt) == 0 && (reinterpret_cast<uintptr_t>(p.X) & 15) == 0 &&
         p.ldx % VEC == 0 && out_rows16(p);
}

template <typename T, int NT>
hipError_t launch_mfma_nt(const FwdParams<T> &p0, hipStream_t s, dim3 grid, size_t shm) {
  FwdParams<T> p = p0;
  p.yrow16 = out_rows16(p) ? 1 : 0;
  constexpr bool V = NT % (16 / (int)sizeof(T)) == 0;   // tiles fill 16-byte loads
  if (p.xrows * p.ldx * (int64_t)sizeof(T) < kXSpan)
    return launch_mfma_xb<T, NT, V, true>(p, s, grid, shm);
  if constexpr (V) {
    if (vectorizable(p, NT)) return launch_mfma_xb<T, NT, true, false>(p, s, grid, shm);
  }
  return launch_mfma_xb<T, NT, false, false>(p, s, grid, shm);
}

template <int NT>
hipError_t launch_bf16_nt(const FwdParams<float> &p, hipStream_t s, dim3 grid, size_t shm) {
  const bool xb = p.xrows * p.ldx * (int64_t)sizeof(float) < kXSpan;
  if (p.mom) {
    if (xb)
      hipLaunchKernelGGL((k_spmm_bf16x3<NT, true, true>), grid, dim3(kThreads), shm, s, p);
    else
      hipLaunchKernelGGL((k_spmm_bf16x3<NT, true, false>), grid, dim3(kThreads), shm, s, p);
  } else {
    if (xb)
      hipLaunchKernelGGL((k_spmm_bf16x3<NT, false, true>), grid, dim3(kThreads), 0, s, p);
    else
      hipLaunchKernelGGL((k_spmm_bf16x3<NT, false, false>), grid, dim3(kThreads), 0, s, p);
  }
  return hipGetLastError();
}

template <int NG, int LW, int R, int MR>
hipError_t launch_small_nr(const FwdParams<double> &p, hipStream_t s, dim3 grid, size_t shm) {
  if (p.mom)
    hipLaunchKernelGGL((k_spmm_small<NG, LW, true, R, MR>), grid, dim3(kThreads), shm, s, p);
  else
    hipLaunchKernelGGL((k_spmm_small<NG, LW, false, R, MR>), grid, dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_small(const FwdParams<double> &p0, hipStream_t s, dim3 grid, size_t shm) {
  FwdParams<double> p = p0;
  p.yrow16 = out_rows16(p) ? 1 : 0;
  // registers allow deeper rings only where a step is narrow: R = 3 against 2
  // is 4 % better on b = 8 at 3 right-hand sides and 14 % worse on b = 1/4/9
  // at 16
  if (p.nrhs <= 8) {
    // operators without a block above 16: the form for 16 rows a pass, whose
    // registers leave room for 5 waves a SIMD instead of 3 (b = 1/4/9, nrhs 4:
    // 76 us with 32 rows a pass, 72 with 16; b = 5 54 and 46, b = 1 74 and 49)
    if (p.bmax <= 16)
      return p.nrhs <= 4 ? launch_small_nr<1, 1, 3, 16>(p, s, grid, shm)
                         : launch_small_nr<2, 2, 2, 16>(p, s, grid, shm);
    return p.nrhs <= 4 ? launch_small_nr<1, 1, 3, 32>(p, s, grid, shm)
                       : launch_small_nr<2, 2, 2, 32>(p, s, grid, shm);
  }
  if (p.nrhs <= 16) return launch_small_nr<4, 2, 2, 32>(p, s, grid, shm);
  return launch_small_nr<8, 2, 2, 16>(p, s, grid, shm);
}

template <typename T>
hipError_t launch_spmm_t(const FwdParams<T> &p, Kind kind, int tile, hipStream_t s) {
  const int64_t nwg = product_workgroups(p.nrows);
  if (nwg == 0) return hipSuccess;
  const dim3 grid((unsigned)nwg);
  const size_t shm = p.mom ? sizeof(double) * kWaves * (size_t)p.nrhs : 0;
  if constexpr (std::is_same<T, double>::value) {
    if (kind == Kind::Small) {
      if (p.xrows * p.ldx * (int64_t)sizeof(T) < kXSpan) return launch_small(p, s, grid, shm);
      // X beyond one buffer descriptor: the kernels with 64-bit addresses
      if (p.nrhs <= 8) {
        kind = Kind::Vec;
        tile = p.nrhs <= 2 ? 2 : p.nrhs <= 4 ? 4 : 8;
      } else {
        kind = Kind::Mfma;
        tile = p.nrhs <= 16 ? 1 : 2;
      }
    }
  }
  if (kind == Kind::Vec) {
    switch (tile) {
      case 1: return launch_vec_nr<T, 1>(p, s, grid, shm);
      case 2: return launch_vec_nr<T, 2>(p, s, grid, shm);
      case 4: return launch_vec_nr<T, 4>(p, s, grid, shm);
      default: return launch_vec_nr<T, 8>(p, s, grid, shm);
    }
  }
  if constexpr (std::is_same<T, float>::value) {
    if (kind == Kind::Bf16x3) {
      if (vectorizable(p, 4)) {
        const bool xb = p.xrows * p.ldx * (int64_t)sizeof(float) < (int64_t(1) << 31);
        if (p.mom) {
          if (xb)
            hipLaunchKernelGGL((k_spmm_bf16x3_vx<true, true>), grid, dim3(kThreads), shm, s, p);
          else
            hipLaunchKernelGGL((k_spmm_bf16x3_vx<true, false>), grid, dim3(kThreads), shm, s, p);
        } else {
          if (xb)
            hipLaunchKernelGGL((k_spmm_bf16x3_vx<false, true>), grid, dim3(kThreads), 0, s, p);
          else
            hipLaunchKernelGGL((k_spmm_bf16x3_vx<false, false>), grid, dim3(kThreads), 0, s, p);
        }
        return hipGetLastError();
      }
      switch (tile) {
        case 1: return launch_bf16_nt<1>(p, s, grid, shm);
        case 2: return launch_bf16_nt<2>(p, s, grid, shm);
        default: return launch_bf16_nt<4>(p, s, grid, shm);
      }
    }
  }
  // matrix cores: tile = right-hand-side tiles of 16 per pass
  switch (tile) {
    case 1: return launch_mfma_nt<T, 1>(p, s, grid, shm);
    case 2: return launch_mfma_nt<T, 2>(p, s, grid, shm);
    default: return launch_mfma_nt<T, 4>(p, s, grid, shm);
  }
}

// ---------------------------------------------------------------------------
// thresholded block product C = A B: numeric stage, block norms, unpacking
// ---------------------------------------------------------------------------
// One wave per output block C_ij (b_i x b_j, 16 x 16 output tiles): a
// matrix-core chain over all products A_ik B_kj of the block, every tile of
// the block accumulated in the same pass so that each operand load serves
// all tiles it belongs to.  The vector-memory instruction count bounds this
// kernel (as the products), so each lane loads 16 bytes: two consecutive
// inner indices k0 = 8t + 2kq and k0 + 1 of its row of A_ik (row-major, from
// A's transposed pages, which hold every block row-major) and of its column
// of B_kj (column-major, from B's forward pages).  Step pair t then feeds two
// matrix instructions, the first over k = 8t + {0, 2, 4, 6}, the second over
// 8t + {1, 3, 5, 7}; both operands use the same k per lane, so the sum is the
// same.  Lanes past the block (row, column or k0 >= b_k) read zeros through
// the buffer bounds; when k0 + 1 == b_k the second value belongs to the next
// row or column (or the slack after the pages) and is replaced by zero.
// Matrix instructions whose k are all past b_k are skipped.
__device__ __forceinline__ double2 pair_load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                             bool second) {
  double2 v = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  v.y = second ? v.y : 0.0;
  return v;
}

// Tiles [ti0, ti0 + TI) x [tj0, tj0 + TJ) of output block c.
template <int KS2, int TI, int TJ>
__device__ __forceinline__ void spgemm_tiles(const SpgemmParams &P, int64_t c, int bi, int bj,
                                             int ti0, int tj0, double &ss) {
  const int lane = threadIdx.x & 63;
  const int m = lane & 15, kq = lane >> 4;
  const int64_t p0 = P.pptr[c];
  const int np = (int)(P.pptr[c + 1] - p0);
  const int64_t *__restrict__ pa = P.pa + p0;
  const int64_t *__restrict__ pb = P.pb + p0;
  constexpr uint32_t kOut = 0x80000000u;
  v4d acc[TI][TJ];
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj) acc[ti][tj] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int q = 0; q < np; ++q) {
    const int64_t ak = pa[q];
    const int bk = (int)(ak & 255);
    // one value of slack past each block: the pair load of k0 = b_k - 1 on
    // the last row reads it (and discards it)
    const __amdgpu_buffer_rsrc_t ra =
        panel_rsrc(P.avals + (ak >> 8), (uint32_t)(bi * bk + 1) * 8u);
    const __amdgpu_buffer_rsrc_t rb = panel_rsrc(P.bvals + pb[q], (uint32_t)(bk * bj + 1) * 8u);
    double2 av[TI][KS2], bv[TJ][KS2];
#pragma unroll
    for (int t = 0; t < KS2; ++t) {
      const int k0 = 8 * t + 2 * kq;
      const bool kin = k0 < bk, k2 = k0 + 1 < bk;
#pragma unroll
      for (int ti = 0; ti < TI; ++ti) {
        const int row = (ti0 + ti) * 16 + m;
        av[ti][t] = pair_load(ra, row < bi && kin ? (uint32_t)(row * bk + k0) * 8u : kOut, k2);
      }
#pragma unroll
      for (int tj = 0; tj < TJ; ++tj) {
        const int col = (tj0 + tj) * 16 + m;
        bv[tj][t] = pair_load(rb, col < bj && kin ? (uint32_t)(col * bk + k0) * 8u : kOut, k2);
      }
    }
#pragma unroll
    for (int t = 0; t < KS2; ++t) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (8 * t + h < bk) {
#pragma unroll
          for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
              acc[ti][tj] = mfma(h ? av[ti][t].y : av[ti][t].x, h ? bv[tj][t].y : bv[tj][t].x,
                                 acc[ti][tj]);
        }
      }
    }
  }
  if (P.fpages) {   // straight into C's pages: forward column-major, transposed row-major
    // the forward (column-major) stores go through a wave-private LDS copy
    // of the tile, so that 8 lanes write one whole column of 16 rows with
    // 16-byte stores (a lane's own values are rows 4 apart of one column)
    __shared__ __align__(16) double tl_all[kWaves * 16 * 18];
    double *tl = tl_all + wave_id() * 16 * 18;   // column-major, 18 per column
    double *ot = P.tpages + P.tpos[c];
    // the block's forward values: columns past b_j fall outside and are dropped
    const __amdgpu_buffer_rsrc_t rf =
        panel_rsrc(P.fpages + P.fpos[c], (uint32_t)(bi * bj) * 8u);
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
      for (int tj = 0; tj < TJ; ++tj) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = (ti0 + ti) * 16 + dst_row<double>(kq, e), col = (tj0 + tj) * 16 + m;
          if (r < bi && col < bj) {
            ot[(int64_t)r * bj + col] = acc[ti][tj][e];
            ss = fma(acc[ti][tj][e], acc[ti][tj][e], ss);
          }
          tl[m * 18 + dst_row<double>(kq, e)] = acc[ti][tj][e];
        }
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int cl = 8 * h + (lane >> 3), rl = 2 * (lane & 7);
          const int col = (tj0 + tj) * 16 + cl, r = (ti0 + ti) * 16 + rl;
          const double2 v = *reinterpret_cast<const double2 *>(tl + cl * 18 + rl);
          const uint32_t off = (uint32_t)(col * bi + r) * 8u;
          if (r + 1 < bi)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u32, v), rf, off, 0, 0);
          else if (r < bi)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u32, v.x), rf, off, 0, 0);
        }
        wave_lds_sync();   // read before the next tile is written
      }
    return;
  }
  double *out = P.cvals + P.obase[c];
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = (ti0 + ti) * 16 + dst_row<double>(kq, e), col = (tj0 + tj) * 16 + m;
        if (r < bi && col < bj) {
          out[(int64_t)r * bj + col] = acc[ti][tj][e];
          ss = fma(acc[ti][tj][e], acc[ti][tj][e], ss);
        }
      }
}

// Output blocks P.order[0 .. P.count) of one tile class: TI x TJ tiles of
// 16 x 16, or (TI = TJ = 0) any size, one tile at a time.
template <int KS2, int TI, int TJ>
__global__ void __launch_bounds__(kThreads) k_spgemm(SpgemmParams P) {
  const int64_t w = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * kWaves + wave_id();
  if (w >= P.count) return;
  const int64_t c = P.order[w];
  const int bi = P.b[P.oi[c]], bj = P.b[P.oj[c]];
  double ss = 0.0;
  if constexpr (TI > 0) {
    spgemm_tiles<KS2, TI, TJ>(P, c, bi, bj, 0, 0, ss);
  } else {
    for (int ti = 0; ti * 16 < bi; ++ti)
      for (int tj = 0; tj * 16 < bj; ++tj) spgemm_tiles<KS2, 1, 1>(P, c, bi, bj, ti, tj, ss);
  }
  if (P.cnorm) {
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) P.cnorm[c] = sqrt(ss);
  }
}

// Frobenius norm of every stored block from the forward pages (a block is a
// contiguous run of b_i*b_j values there); one wave per block.
__global__ void __launch_bounds__(kThreads) k_block_norms(const double *pages, const int64_t *pos,
                                                          const int32_t *blk_row,
                                                          const int32_t *col_idx,
                                                          const int32_t *b, int64_t nnzb,
                                                          double *out) {
  const int64_t k = (int64_t)blockIdx.x * kWaves + wave_id();
  if (k >= nnzb) return;
  const int lane = threadIdx.x & 63;
  const int sz = b[blk_row[k]] * b[col_idx[k]];
  const double *v = pages + pos[k];
  double s = 0.0;
  for (int e = lane; e < sz; e += 64) s = fma(v[e], v[e], s);
  s = wave_sum(s);
  if (lane == 0) out[k] = sqrt(s);
}

// Zero the alignment gap after every panel and the slack after the last
// (the values themselves are written by the packing): one thread per panel.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_zero_gaps(const RowDesc *rows, int32_t np,
                                                        int64_t n_values, T *vals) {
  const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (p >= np && !(p == 0 && np == 0)) return;
  const int64_t s = np ? rows[p].vbase + (int64_t)rows[p].b * rows[p].K : 0;
  const int64_t e = p + 1 < np ? rows[p + 1].vbase : n_values + kPageSlack;
  for (int64_t x = s; x < e; ++x) vals[x] = T(0);
}

// dst[dbase[t] + e] = src[sbase[t] + e] for e < size[t]; one wave per block.
__global__ void __launch_bounds__(kThreads) k_gather_blocks(const double *src,
                                                            const int64_t *sbase,
                                                            const int64_t *dbase,
                                                            const int32_t *size, int64_t nblk,
                                                            double *dst) {
  const int64_t t = (int64_t)blockIdx.x * kWaves + wave_id();
  if (t >= nblk) return;
  const int lane = threadIdx.x & 63;
  const double *sp = src + sbase[t];
  double *dp = dst + dbase[t];
  for (int e = lane; e < size[t]; e += 64) dp[e] = sp[e];
}

// Forward pages -> graph order (each block row-major at gbase): `parts` waves take
// kPackRun blocks, whose values are one run of the destination (a million
// blocks of 1, 4 and 9: 112 us, 374 with one block a wave; 775,000 blocks of
// 9 to 20, 1.3 GB each way: 645 both ways, 4 TB/s, columns read 8 bytes a lane).
template <typename T>
__global__ void __launch_bounds__(kThreads) k_unpack(const T *pages, const int64_t *pos,
                                                     const int32_t *blk_row,
                                                     const int32_t *col_idx, const int32_t *b,
                                                     const int64_t *gbase, int64_t nnzb, int parts, T *dst) {
  __shared__ PageRec tab_all[kWaves * kPackRun];
  const int64_t w = (int64_t)blockIdx.x * kWaves + wave_id();
  const int part = (int)(w % parts);
  const int64_t k0 = w / parts * kPackRun;
  if (k0 >= nnzb) return;
  const int lane = threadIdx.x & 63;
  const int nb = (int)min((int64_t)kPackRun, nnzb - k0);
  PageRec *tab = tab_all + wave_id() * kPackRun;
  PageRec r{};
  if (lane < nb) {
    const int64_t k = k0 + lane;
    r.src = pos[k];
    r.dst = gbase[k];
    r.bi = b[blk_row[k]];
    r.bj = b[col_idx[k]];
  }
  transpose_run<T>(r, tab, nb, lane, part, parts, pages, dst);
}

// ---------------------------------------------------------------------------
// kernel polynomial method: damped coefficients and the density of states
// ---------------------------------------------------------------------------
// c_0 = g_0 mu_0, c_k = 2 g_k mu_k (k >= 1): the coefficients of the series
// sum_k c_k T_k(x); g_k = 1 (no damping) or the Jackson factors
// [(M-k+1) cos(q k) + sin(q k) cot(q)] / (M+1), q = pi / (M+1).
__global__ void __launch_bounds__(kThreads) k_kpm_coef(const double *mu, int M, int damping,
                                                       double *c) {
  const int k = blockIdx.x * kThreads + threadIdx.x;
  if (k >= M) return;
  double g = 1.0;
  if (damping == 1) {
    const double q = M_PI / (M + 1);
    g = ((double)(M - k + 1) * cos(q * k) + sin(q * k) * cos(q) / sin(q)) / (M + 1);
  }
  c[k] = (k == 0 ? 1.0 : 2.0) * g * mu[k];
}

// rho(x) = sum_k c_k T_k(x) / (pi sqrt(1 - x^2)) at every point, one lane per
// point, the series summed by Clenshaw's recurrence from the highest degree
// (b_k = c_k + 2x b_{k+1} - b_{k+2}; sum = c_0 + x b_1 - b_2).  All lanes read
// the same c_k: the coefficients come through the scalar cache, 16 per
// unrolled step.
__global__ void __launch_bounds__(kThreads) k_kpm_dos(const double *c, int M, const double *x,
                                                      int64_t np, double *rho) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const double xi = i < np ? x[i] : 0.0;
  const double tx = 2.0 * xi;
  double b1 = 0.0, b2 = 0.0;
  int k = M - 1;
  for (; k >= 16; k -= 16) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const double b0 = fma(tx, b1, c[k - u] - b2);
      b2 = b1;
      b1 = b0;
    }
  }
  for (; k >= 1; --k) {
    const double b0 = fma(tx, b1, c[k] - b2);
    b2 = b1;
    b1 = b0;
  }
  const double s = fma(xi, b1, c[0] - b2);
  if (i < np) rho[i] = s / (M_PI * sqrt(1.0 - xi * xi));
}

// 16 lanes per graph block write the column-table entries of its panel columns
// (set-up, once per structure): runs of b entries instead of one lane's
// entries b apart (775,000 blocks of 9 to 20, both directions: 39 us
// a call against 147).
__global__ void __launch_bounds__(kThreads) k_columns(ColumnParams P) {
  for (int64_t k = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 4; k < P.nnzb;
       k += (int64_t)gridDim.x * (kThreads / 16)) {
    const int32_t c = P.catom[k];
    const int bc = P.b[c];
    const int64_t base = P.rows[P.prow[k]].cbase + P.k0[k];
    const int32_t o = P.off[c];
    const int64_t g = P.colg ? P.gbase[k] : 0;
    for (int q = threadIdx.x & 15; q < bc; q += 16) {
      P.colx[base + q] = o + q;
      if (P.colg) P.colg[base + q] = ((g + q) << 7) | bc;
    }
  }
}

}  // namespace

int64_t product_workgroups(int64_t nrows) { return (nrows + kWaves - 1) / kWaves; }

hipError_t launch_spmm_f64(const FwdParams<double> &p, Kind kind, int tile, hipStream_t s) {
  return launch_spmm_t<double>(p, kind == Kind::Bf16x3 ? Kind::Mfma : kind, tile, s);
}
hipError_t launch_spmm_f32(const FwdParams<float> &p, Kind kind, int tile, hipStream_t s) {
  return launch_spmm_t<float>(p, kind, tile, s);
}

hipError_t launch_pack(const PackParams &p, const void *src, int src_dtype, hipStream_t s) {
  if (p.nnzb == 0) return hipSuccess;
  const int64_t waves = (p.nnzb + kPackRun - 1) / kPackRun;
  const dim3 grid((unsigned)((waves + kWaves - 1) / kWaves));
  const int sel = src_dtype * 3 + p.dst_kind;
  switch (sel) {
    case 0: hipLaunchKernelGGL((k_pack<0, 0>), grid, dim3(kThreads), 0, s, p, src); break;
    case 1: hipLaunchKernelGGL((k_pack<0, 1>), grid, dim3(kThreads), 0, s, p, src); break;
    case 2: hipLaunchKernelGGL((k_pack<0, 2>), grid, dim3(kThreads), 0, s, p, src); break;
    case 3: hipLaunchKernelGGL((k_pack<1, 0>), grid, dim3(kThreads), 0, s, p, src); break;
    case 4: hipLaunchKernelGGL((k_pack<1, 1>), grid, dim3(kThreads), 0, s, p, src); break;
    case 5: hipLaunchKernelGGL((k_pack<1, 2>), grid, dim3(kThreads), 0, s, p, src); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Outputs in graph order take the ring where they go to memory; us straight
// from the accumulators and through the ring: FP32, 32 right-hand sides, b = 8
// (250 MB) 196/174, b = 4/9 (205 MB) 217/188, b = 1/4/9 (142 MB) 114/133, b = 5
// (122 MB) 99/124; FP64, 16, b = 4/9 (410 MB) 268/256, b = 1/4/9 (283 MB)
// 201/194, b = 8 (150 MB) 49/70, 1,000 rows of b = 5 12/19.  FP64 beyond 32
// right-hand sides never: b = 8, 48, 500 MB 367/403; 64, b = 1/4/9, 640 MB
// 774/819, b = 4/9, 660 MB 786/803 (its LDS, held until a workgroup's last wave
// ends, costs the panels that do not use it as much).  Only 9 rows beside
// blocks of 13 gain there (b = 9/13, 490 MB 404/389; b = 13/9/1, 950 MB 772/748).
template <typename T, int PR, int NCH>
void launch_sddmm_tiles(const SddmmParams<T> &p, dim3 grid, uint32_t xbytes, hipStream_t s) {
  if (p.page_out)
    hipLaunchKernelGGL((k_sddmm<T, PR, NCH, true, 256>), grid, dim3(kThreads), 0, s, p, xbytes);
  else if (NCH == 1 && p.nnz * (int64_t)sizeof(T) >= kMemoryBytes)
    hipLaunchKernelGGL((k_sddmm<T, PR, NCH, false, NCH == 1 ? 512 : 1>), grid, dim3(kThreads), 0, s, p, xbytes);
  else
    hipLaunchKernelGGL((k_sddmm<T, PR, NCH, false, 1>), grid, dim3(kThreads), 0, s, p, xbytes);
}

template <typename T>
hipError_t launch_sddmm_t(const SddmmParams<T> &p, hipStream_t s) {
  if (p.nrows == 0) return hipSuccess;
  const dim3 grid((unsigned)product_workgroups(p.nrows));
  // X rows through LDS when X spans less than one buffer descriptor; up to 64
  // right-hand sides in one pass (a panel's dY rows are addressed by 32 bits)
  const int64_t xb = ((p.xrows - 1) * p.ldx + p.nrhs) * (int64_t)sizeof(T);
  if (xb < kXSpan && p.nrhs <= 64 && p.lddy < (1 << 22)) {
    const int pieces = (p.nrhs * (int)sizeof(T) + 15) / 16;
    if (pieces <= 4)
      launch_sddmm_tiles<T, 4, 1>(p, grid, (uint32_t)xb, s);
    else if (pieces <= 8)
      launch_sddmm_tiles<T, 8, 1>(p, grid, (uint32_t)xb, s);
    else if (pieces <= 16)
      launch_sddmm_tiles<T, 16, 1>(p, grid, (uint32_t)xb, s);
    else if constexpr (sizeof(T) == 8)
      launch_sddmm_tiles<T, 16, 2>(p, grid, (uint32_t)xb, s);
    return hipGetLastError();
  }
  if (p.nrhs > 32 && p.xrows * p.ldx * (int64_t)sizeof(T) < (int64_t(1) << 31)) {
    hipLaunchKernelGGL((k_sddmm_lds<T>), grid, dim3(kThreads), 0, s, p);
    return hipGetLastError();
  }
  // right-hand sides beyond the register-resident chunks are loaded per tile
  if (p.nrhs <= 32)
    hipLaunchKernelGGL((k_sddmm_mfma<T, 1>), grid, dim3(kThreads), 0, s, p);
  else
    hipLaunchKernelGGL((k_sddmm_mfma<T, 2>), grid, dim3(kThreads), 0, s, p);
  return hipGetLastError();
}
hipError_t launch_sddmm_f64(const SddmmParams<double> &p, hipStream_t s) {
  return launch_sddmm_t(p, s);
}
hipError_t launch_sddmm_f32(const SddmmParams<float> &p, hipStream_t s) {
  return launch_sddmm_t(p, s);
}

static int dot_columns(int32_t nrhs) {
  int cl = 1;
  while (cl < 64 && cl < nrhs) cl *= 2;
  return cl;
}
int64_t coldot_chunks(int64_t nrows) { return (nrows + kDotRows - 1) / kDotRows; }

template <typename T>
hipError_t launch_coldot_t(const T *A, int64_t lda, const T *B, int64_t ldb, int64_t nrows,
                           int32_t nrhs, double *partial, int64_t *nchunks, hipStream_t s) {
  *nchunks = coldot_chunks(nrows);
  if (*nchunks == 0) return hipSuccess;
  const dim3 grid((unsigned)*nchunks);
  if (A == B && lda == ldb)
    hipLaunchKernelGGL((k_coldot<T, true>), grid, dim3(kThreads), 0, s, A, lda, B, ldb, nrows, nrhs,
                       dot_columns(nrhs), partial);
  else
    hipLaunchKernelGGL((k_coldot<T, false>), grid, dim3(kThreads), 0, s, A, lda, B, ldb, nrows,
                       nrhs, dot_columns(nrhs), partial);
  return hipGetLastError();
}
hipError_t launch_coldot_f64(const double *A, int64_t lda, const double *B, int64_t ldb,
                             int64_t nrows, int32_t nrhs, double *partial, int64_t *nchunks,
                             hipStream_t s) {
  return launch_coldot_t(A, lda, B, ldb, nrows, nrhs, partial, nchunks, s);
}
hipError_t launch_coldot_f32(const float *A, int64_t lda, const float *B, int64_t ldb,
                             int64_t nrows, int32_t nrhs, double *partial, int64_t *nchunks,
                             hipStream_t s) {
  return launch_coldot_t(A, lda, B, ldb, nrows, nrhs, partial, nchunks, s);
}

hipError_t launch_reduce_partials(const double *partial, int64_t nparts, int32_t nrhs, double *out,
                                  hipStream_t s) {
  if (nrhs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce, dim3((unsigned)nrhs), dim3(kThreads), 0, s, partial, nparts, nrhs, out);
  return hipGetLastError();
}

template <int KS2>
hipError_t launch_spgemm_ks(const SpgemmParams &p, int cls, dim3 grid, hipStream_t s) {
  switch (cls) {
    case 0: hipLaunchKernelGGL((k_spgemm<KS2, 1, 1>), grid, dim3(kThreads), 0, s, p); break;
    case 1: hipLaunchKernelGGL((k_spgemm<KS2, 1, 2>), grid, dim3(kThreads), 0, s, p); break;
    case 2: hipLaunchKernelGGL((k_spgemm<KS2, 2, 1>), grid, dim3(kThreads), 0, s, p); break;
    case 3: hipLaunchKernelGGL((k_spgemm<KS2, 2, 2>), grid, dim3(kThreads), 0, s, p); break;
    default: hipLaunchKernelGGL((k_spgemm<KS2, 0, 0>), grid, dim3(kThreads), 0, s, p); break;
  }
  return hipGetLastError();
}

hipError_t launch_spgemm_numeric(const SpgemmParams &p, int cls, int max_b, hipStream_t s) {
  if (p.count == 0) return hipSuccess;
  const dim3 grid((unsigned)((p.count + kWaves - 1) / kWaves));
  // pairs of inner indices held per product: ceil(max_b / 8)
  if (max_b <= 8) return launch_spgemm_ks<1>(p, cls, grid, s);
  if (max_b <= 16) return launch_spgemm_ks<2>(p, cls, grid, s);
  if (max_b <= 24) return launch_spgemm_ks<3>(p, cls, grid, s);
  if (max_b <= 32) return launch_spgemm_ks<4>(p, cls, grid, s);
  return launch_spgemm_ks<8>(p, cls, grid, s);
}

hipError_t launch_block_norms(const double *pages, const int64_t *pos, const int32_t *blk_row,
                              const int32_t *col_idx, const int32_t *b, int64_t nnzb, double *out,
                              hipStream_t s) {
  if (nnzb == 0) return hipSuccess;
  const dim3 grid((unsigned)((nnzb + kWaves - 1) / kWaves));
  hipLaunchKernelGGL(k_block_norms, grid, dim3(kThreads), 0, s, pages, pos, blk_row, col_idx, b,
                     nnzb, out);
  return hipGetLastError();
}

hipError_t launch_refresh_records(const PackParams &p, const int32_t *order, PageRec *rec,
                                  hipStream_t s) {
  if (p.nnzb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_refresh_records, dim3((unsigned)((p.nnzb + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, p, order, rec);
  return hipGetLastError();
}

hipError_t launch_refresh(const PageRec *rec, int64_t nnzb, int elem_bytes, const void *src,
                          void *dst, hipStream_t s) {
  if (nnzb == 0) return hipSuccess;
  const int64_t waves = (nnzb + kPackRun - 1) / kPackRun;
  const dim3 grid((unsigned)((waves + kWaves - 1) / kWaves));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_refresh<double>, grid, dim3(kThreads), 0, s, rec, nnzb,
                       static_cast<const double *>(src), static_cast<double *>(dst));
  else
    hipLaunchKernelGGL(k_refresh<float>, grid, dim3(kThreads), 0, s, rec, nnzb,
                       static_cast<const float *>(src), static_cast<float *>(dst));
  return hipGetLastError();
}

hipError_t launch_zero_gaps(const RowDesc *rows, int32_t np, int64_t n_values, int elem_bytes,
                            void *vals, hipStream_t s) {
  const dim3 grid((unsigned)((std::max<int64_t>(np, 1) + kThreads - 1) / kThreads));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_zero_gaps<double>, grid, dim3(kThreads), 0, s, rows, np, n_values,
                       static_cast<double *>(vals));
  else
    hipLaunchKernelGGL(k_zero_gaps<float>, grid, dim3(kThreads), 0, s, rows, np, n_values,
                       static_cast<float *>(vals));
  return hipGetLastError();
}

hipError_t launch_gather_blocks(const double *src, const int64_t *sbase, const int64_t *dbase,
                                const int32_t *size, int64_t nblk, double *dst, hipStream_t s) {
  if (nblk == 0) return hipSuccess;
  const dim3 grid((unsigned)((nblk + kWaves - 1) / kWaves));
  hipLaunchKernelGGL(k_gather_blocks, grid, dim3(kThreads), 0, s, src, sbase, dbase, size, nblk,
                     dst);
  return hipGetLastError();
}

hipError_t launch_unpack(const void *pages, int elem_bytes, const int64_t *pos,
                         const int32_t *blk_row, const int32_t *col_idx, const int32_t *b,
                         const int64_t *gbase, int64_t nnzb, int64_t nnz, int bmax, void *dst,
                         hipStream_t s) {
  if (nnzb == 0) return hipSuccess;
  const int64_t runs = (nnzb + kPackRun - 1) / kPackRun;
  // Waves of a run: each about 1024 values, and where the runs are too few to
  // fill the chip enough for 8192 waves, as long as the longest run can use
  // them (30 atoms of b = 64: 20 us with one wave a block, 96 with one a run,
  // now 13; 1,000 atoms of b = 1/4/9 with one of 64: 22, 27 and 18; 10,000 of
  // b = 13: 210, 190 and 180).
  const int64_t avg = (nnz / runs + 1023) / 1024;
  const int64_t most = ((int64_t)kPackRun * bmax * bmax + 64 * kPackChunk - 1) / (64 * kPackChunk);
  const int parts = (int)std::max(avg, std::min((8191 + runs) / runs, most));
  const int64_t waves = runs * parts;
  const dim3 grid((unsigned)((waves + kWaves - 1) / kWaves));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_unpack<double>, grid, dim3(kThreads), 0, s,
                       static_cast<const double *>(pages), pos, blk_row, col_idx, b, gbase, nnzb, parts,
                       static_cast<double *>(dst));
  else
    hipLaunchKernelGGL(k_unpack<float>, grid, dim3(kThreads), 0, s,
                       static_cast<const float *>(pages), pos, blk_row, col_idx, b, gbase, nnzb, parts,
                       static_cast<float *>(dst));
  return hipGetLastError();
}

hipError_t launch_kpm_dos(const double *mu, int M, int damping, const double *x, int64_t np,
                          double *coef, double *rho, hipStream_t s) {
  hipLaunchKernelGGL(k_kpm_coef, dim3((unsigned)((M + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     s, mu, M, damping, coef);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || np == 0) return e;
  hipLaunchKernelGGL(k_kpm_dos, dim3((unsigned)((np + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     s, coef, M, x, np, rho);
  return hipGetLastError();
}

hipError_t launch_columns(const ColumnParams &p, hipStream_t s) {
  if (p.nnzb == 0) return hipSuccess;
  const int64_t lanes = std::min<int64_t>(16 * p.nnzb, int64_t(1) << 30);
  hipLaunchKernelGGL(k_columns, dim3((unsigned)((lanes + kThreads - 1) / kThreads)), dim3(kThreads),
                     0, s, p);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// halo exchange buffers of a rank-local operator
// ---------------------------------------------------------------------------
// buf[t, c] = X[rows[t], c]: one thread per element, consecutive threads
// along c (coalesced row pieces).  Rows outside [0, xrows) are skipped.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_rows_pack(const T *__restrict__ X, int64_t xrows,
                                                        int64_t ldx, const int32_t *__restrict__ rows,
                                                        int64_t nrows, int32_t nrhs,
                                                        T *__restrict__ buf, int64_t ldb) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= nrows * nrhs) return;
  const int64_t t = e / nrhs, c = e - t * nrhs;
  const int64_t r = rows[t];
  if (r < 0 || r >= xrows) return;
  buf[t * ldb + c] = X[r * ldx + c];
}

// Y[red_rows[u], c] += sum over e in [red_ptr[u], red_ptr[u+1]) of
// buf[red_pos[e], c], in e order: one thread per (u, c), so every output
// element has one writer.  Indices outside Y or the buffer are skipped.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_rows_reduce(T *__restrict__ Y, int64_t yrows,
                                                          int64_t ldy,
                                                          const int32_t *__restrict__ red_rows,
                                                          const int64_t *__restrict__ red_ptr,
                                                          const int64_t *__restrict__ red_pos,
                                                          int64_t n_red, int64_t brows,
                                                          const T *__restrict__ buf, int64_t ldb,
                                                          int32_t nrhs) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= n_red * nrhs) return;
  const int64_t u = e / nrhs, c = e - u * nrhs;
  const int64_t r = red_rows[u];
  if (r < 0 || r >= yrows) return;
  T acc = Y[r * ldy + c];
  for (int64_t q = red_ptr[u]; q < red_ptr[u + 1]; ++q) {
    const int64_t s = red_pos[q];
    if (s >= 0 && s < brows) acc += buf[s * ldb + c];
  }
  Y[r * ldy + c] = acc;
}

// ---------------------------------------------------------------------------
// scratch of the allocation-free entry points
// ---------------------------------------------------------------------------
// One copy per GPU, resident from the module's load to the end of the
// process.  In host code `scratch` names only the host-side stand-in of the
// array: its device address is looked up below, once per device, and only
// that address is ever passed to kernels.
static __device__ __align__(256) double scratch[kNoAllocScratchBytes / sizeof(double)];

hipError_t noalloc_scratch(void **ptr, size_t *bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = kNoAllocScratchBytes;
  return hipSuccess;
}


hipError_t launch_rows_pack(const void *X, int64_t xrows, int64_t ldx, const int32_t *rows,
                            int64_t nrows, int32_t nrhs, int elem_bytes, void *buf, int64_t ldb,
                            hipStream_t s) {
  const int64_t n = nrows * nrhs;
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_rows_pack<double>, grid, dim3(kThreads), 0, s,
                       static_cast<const double *>(X), xrows, ldx, rows, nrows, nrhs,
                       static_cast<double *>(buf), ldb);
  else
    hipLaunchKernelGGL(k_rows_pack<float>, grid, dim3(kThreads), 0, s,
                       static_cast<const float *>(X), xrows, ldx, rows, nrows, nrhs,
                       static_cast<float *>(buf), ldb);
  return hipGetLastError();
}

hipError_t launch_rows_reduce(void *Y, int64_t yrows, int64_t ldy, const int32_t *red_rows,
                              const int64_t *red_ptr, const int64_t *red_pos, int64_t n_red,
                              int64_t brows, const void *buf, int64_t ldb, int32_t nrhs,
                              int elem_bytes, hipStream_t s) {
  const int64_t n = n_red * nrhs;
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
  if (elem_bytes == 8)
    hipLaunchKernelGGL(k_rows_reduce<double>, grid, dim3(kThreads), 0, s, static_cast<double *>(Y),
                       yrows, ldy, red_rows, red_ptr, red_pos, n_red, brows,
                       static_cast<const double *>(buf), ldb, nrhs);
  else
    hipLaunchKernelGGL(k_rows_reduce<float>, grid, dim3(kThreads), 0, s, static_cast<float *>(Y),
                       yrows, ldy, red_rows, red_ptr, red_pos, n_red, brows,
                       static_cast<const float *>(buf), ldb, nrhs);
  return hipGetLastError();
}

}  // namespace vbcsr
