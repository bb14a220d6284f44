// gcp_backward.hip -- adjoint of the purification (reverse mode), gfx950.
//
// Given Gbar_p = dL/dD_p of the returned matrix, every update
// D' = a D + b D^2 + e D^3, with (a, b, e) functions of
// c = (T2 - T3)/(T1 - T2) (eq. (hpcp3): 1 - 2c, 2 + 2c, -2; eqs.
// (pm1a)/(pm1b) for PMCP; update_coefs), is differentiated by hand for
// symmetric D and Gbar' (= dL/dD'):
//
//   Gbar = a Gbar' + b (D Gbar' + Gbar' D) + e (D^2 Gbar' + Gbar' D^2 + D Gbar' D)
//          + kappa [(2 D - 3 D^2) - c (I - 2 D)] / (T1 - T2),
//   kappa = <Gbar', dD'/dc> = a' <Gbar', D> + b' <Gbar', D^2> + e' <Gbar', D^3>
//
// (Frobenius products; a', b', e' from update_coef_derivs; <Gbar', D^3> =
// <D^2, D Gbar'>, needed only when e' != 0, i.e. for PMCP).
//
// One adjoint step is three launches of 64 x 64 MFMA tile products, all of
// the A * B^T row-panel form of the forward (every operand is symmetric
// except AT and CT, which are only ever read along their rows):
//   mode 0 (upper tiles)  X2 = D D           epilogue: per-tile sums of
//                                            w_ij Gbar'_ij X2_ij and w_ij Gbar'_ij D_ij
//   mode 1 (all tiles)    AT = D Gbar'  and  CT = X2 Gbar'   (one launch;
//                                            PMCP: per-tile sums of X2 o AT)
//   mode 2 (upper tiles)  E  = D (Gbar' D)   epilogue: Gbar_n from Gbar', AT,
//                                            AT^T, CT, CT^T, E, D and X2
// with AT + AT^T = D Gbar' + Gbar' D and CT + CT^T = D^2 Gbar' + Gbar' D^2.
// Algorithmic cost per step: two symmetric products (M^3 each, upper-triangle
// output) and two general ones (2 M^3 each).  kappa is reduced on the device
// in a fixed order, so the whole backward is bitwise reproducible.
//
// The initial guess D_0 = theta I + beta (mu I - H), mu = Tr(H)/M.  With a
// fixed slope rule (eqs. (dmguess),(pmcpguess), or eq. (hpcpguess) with a
// fixed alpha) and the spectral bounds held fixed,
//   dL/dH = -beta Gbar_0 + (I/M) [beta Tr Gbar_0 + beta'(mu) <Gbar_0, mu I - H>],
// where <Gbar_0, mu I - H> = (<Gbar_0, D_0> - theta Tr Gbar_0) / beta, so H is
// not needed again, and beta' belongs to the active branch of the min.  The
// alpha search of eq. (hpcpguessalpha) sets beta = sqrt((target - N theta)/S)
// with S = ||mu I - H||_F^2 (alpha strictly inside (0, 1)); then beta' = 0
// and d beta = (beta / S) <mu I - H, dH> adds
//   (<Gbar_0, mu I - H> / S) (D_0 - theta I)     (= (beta <Gbar_0, g>/S) g).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcp_encode.h"
#include "gcp_kernels.h"
#include "gcp_mma.h"

namespace gcp {

// All tiles of the nt x nt grid, in groups of TILE_GROUP tile rows,
// column-major inside a group: consecutive blocks share the right-hand
// (column) panel and cycle over the group's row panels.
__device__ __forceinline__ void full_tile_of_block(int L, int nt, int &ti, int &tj) {
  const int gr = L / (TILE_GROUP * nt);
  const int r0 = gr * TILE_GROUP, rows = min(TILE_GROUP, nt - r0);
  const int rem = L - gr * TILE_GROUP * nt;
  ti = r0 + rem % rows;
  tj = rem / rows;
}

// Contiguous run of [0, total) for the XCD that block b is dispatched to.
__device__ __forceinline__ int xcd_linear(int b, int total) {
  const int xcd = b & 7, loc = b >> 3, q = total >> 3, r = total & 7;
  return xcd * q + (xcd < r ? xcd : r) + loc;
}

template <int P> struct BwdCfg {
  static constexpr int W = T64 * VP * 8;     // FP64 staging of a tile
  static constexpr int MM = TileCfg<P>::SMEM > W ? TileCfg<P>::SMEM : W;
  static constexpr int SMEM = MM + 8 * 8;    // and two sums per wave
  static constexpr int BLOCKS = Enc<P>::KIND == 0 ? 3 : 2;   // per CU, as k_tile
};

// 64 x 64 tiles, one per block; thread tid works on columns 4 (tid % 16) .. +3
// of rows 16 q + tid / 16 of the tile, so that the inputs are read, and the
// result and its mirror (through LDS) written, as rows of 64 elements.
template <int P, int MODE>
__global__ __launch_bounds__(NTH, BwdCfg<P>::BLOCKS) void k_bgemm(BwdArgs a) {
  using E = Enc<P>;
  using T = typename E::T;
  typedef T v4t __attribute__((ext_vector_type(4)));
  using S = typename TileCfg<P>::S;
  static_assert(E::NP == 1, "the adjoint uses single-plane FP64 / FP32 storage");

  __shared__ __attribute__((aligned(16))) char smem[BwdCfg<P>::SMEM];
  double *W = (double *)smem, *red = (double *)(smem + BwdCfg<P>::MM);

  const int64_t Mp = a.Mp;
  int ti, tj, lin = 0, which = 0;
  if constexpr (MODE == 1) {
    const int nfull = a.nt * a.nt;
    int L = xcd_linear(blockIdx.x, 2 * nfull);
    which = L >= nfull;
    full_tile_of_block(L - which * nfull, a.nt, ti, tj);
  } else {
    tile_of_block(blockIdx.x, a.nt, ti, tj, lin);
  }
  const int64_t arow0 = (int64_t)ti * T64, brow0 = (int64_t)tj * T64;
  const T *__restrict__ D = (const T *)a.D;
  const T *__restrict__ X2 = (const T *)a.X2;
  const T *__restrict__ G = (const T *)a.G;
  const T *__restrict__ AT = (const T *)a.AT;
  const T *__restrict__ CT = (const T *)a.CT;
  const T *Al, *Bl;
  if constexpr (MODE == 0) {
    Al = D;
    Bl = D;
  } else if constexpr (MODE == 1) {
    Al = which ? X2 : D;
    Bl = G;
  } else {
    Al = D;
    Bl = AT;
  }

  tile_product<P>(Al, Bl, arow0, brow0, Mp, smem, fp32_fold(Mp), 0,
                  (int)(Mp / TileCfg<P>::KT));

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c4 = (tid & 15) * 4, r0 = tid >> 4;
  const S *V = (const S *)smem + r0 * VP + c4;   // this thread's elements
  const int64_t o0 = (arow0 + r0) * Mp + brow0 + c4;
  const int64_t m0 = (brow0 + r0) * Mp + arow0 + c4;   // in the mirrored tile

  if constexpr (MODE == 1) {
    T *__restrict__ O = (T *)(which ? a.out1 : a.out0);
    const bool x3 = a.need_x3 && !which;   // block-uniform
    double xsum = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t o = o0 + q * 16 * Mp;
      v4t ov;
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = V[q * 16 * VP + e];
      if (x3) {
        const v4t xv = *(const v4t *)(X2 + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) xsum += (double)xv[e] * (double)ov[e];
      }
      *(v4t *)(O + o) = ov;
    }
    if (x3) {
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) xsum += shfl_xor_d(xsum, m);
      if (lane == 0) red[wave] = xsum;
      __syncthreads();
      if (tid == 0) {
        const int ntri = a.nt * (a.nt + 1) / 2;
        a.tpart[2 * ntri + ti * a.nt + tj] = ((red[0] + red[1]) + red[2]) + red[3];
      }
    }
    return;
  }

  const bool dtile = (ti == tj);
  T *__restrict__ O = (T *)a.out0;
  double tsum = 0.0, dsum = 0.0;
  const double kappa = MODE == 2 ? *a.kappa : 0.0;
  double v[4][4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[q][e] = (double)V[q * 16 * VP + e];
  if constexpr (MODE == 2) {
    // b AT^T + e CT^T + e E: the transposes from rows of the mirrored tile
    double t[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const v4t at = *(const v4t *)(AT + m0 + q * 16 * Mp), ct = *(const v4t *)(CT + m0 + q * 16 * Mp);
#pragma unroll
      for (int e = 0; e < 4; ++e) t[q][e] = a.b * (double)at[e] + a.e * (double)ct[e];
    }
    __syncthreads();   // V read by all
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) W[(q * 16 + r0) * VP + c4 + e] = t[q][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q][e] = W[(c4 + e) * VP + q * 16 + r0] + a.e * v[q][e];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = q * 16 + r0;
    const int64_t o = o0 + q * 16 * Mp;
    const v4t dv = *(const v4t *)(D + o), gv = *(const v4t *)(G + o);
    v4t ov;
    if constexpr (MODE == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = c4 + e;
        const T x = (T)v[q][e];
        ov[e] = x;
        if (dtile && row > c) continue;   // covered by the mirror of (j, i)
        const double wg = ((dtile && row == c) ? 1.0 : 2.0) * (double)gv[e];
        tsum += wg * (double)x;
        dsum += wg * (double)dv[e];
      }
    } else {
      const v4t xv = *(const v4t *)(X2 + o), av = *(const v4t *)(AT + o), cv = *(const v4t *)(CT + o);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double d = (double)dv[e], x2 = (double)xv[e];
        const double one = (dtile && row == c4 + e) ? 1.0 : 0.0;
        const double gc = ((2.0 * d - 3.0 * x2) - a.c * (one - 2.0 * d)) * a.inv_t12;
        ov[e] = (T)(a.a * (double)gv[e] + a.b * (double)av[e] + a.e * (double)cv[e] + v[q][e] +
                    kappa * gc);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) ((T *)smem)[row * VP + c4 + e] = ov[e];
    if (!dtile) *(v4t *)(O + o) = ov;
  }
  __syncthreads();
  // mirrored tile, from LDS; a diagonal tile is written whole from here, its
  // lower half from the upper one
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = q * 16 + r0;
    v4t ov;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = c4 + e;
      const bool up = dtile && row < c;
      ov[e] = ((const T *)smem)[(up ? row : c) * VP + (up ? c : row)];
    }
    *(v4t *)(O + m0 + q * 16 * Mp) = ov;
  }

  if constexpr (MODE == 0) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      tsum += shfl_xor_d(tsum, m);
      dsum += shfl_xor_d(dsum, m);
    }
    if (lane == 0) {
      red[wave] = tsum;
      red[4 + wave] = dsum;
    }
    __syncthreads();
    if (tid == 0) {
      const int ntri = a.nt * (a.nt + 1) / 2;
      a.tpart[lin] = ((red[0] + red[1]) + red[2]) + red[3];
      a.tpart[ntri + lin] = ((red[4] + red[5]) + red[6]) + red[7];
    }
  }
}

// Sum of tpart[t0 .. t1) in a fixed order by the 256 threads of one block.
__device__ double block_sum(const double *tpart, int t0, int t1, double *s) {
  double v = 0.0;
  for (int t = t0 + (int)threadIdx.x; t < t1; t += 256) v += tpart[t];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  const double r = s[0];
  __syncthreads();
  return r;
}

// kappa = da <G, D> + db <G, D^2> + de <G, D^3> from the per-tile sums, in a
// fixed order (one block).
__global__ __launch_bounds__(256) void k_bkappa(const double *tpart, int ntri, int nfull,
                                                double da, double db, double de, double *kappa) {
  __shared__ double s[256];
  const double sx2 = block_sum(tpart, 0, ntri, s);
  const double sd = block_sum(tpart, ntri, 2 * ntri, s);
  const double sx3 = de != 0.0 ? block_sum(tpart, 2 * ntri, 2 * ntri + nfull, s) : 0.0;
  if (threadIdx.x == 0) *kappa = da * sd + db * sx2 + de * sx3;
}

// Iterate D_n of the forward (operand planes of encoding PF plus the exact
// FP64 diagonal) as a plain Mp x Mp matrix in the adjoint's storage type.
template <int PF, int PB>
__global__ __launch_bounds__(256) void k_bstore(const void *planes, const double *dg, int64_t Mp,
                                                void *out) {
  using EF = Enc<PF>;
  using TF = typename EF::T;
  using TB = typename Enc<PB>::T;
  // rows on the x dimension of the grid (no 64K limit), 256 columns per block on y
  const int64_t i = blockIdx.x;
  const int64_t j = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (j >= Mp) return;
  double x;
  if (i == j) {
    x = dg[i];
  } else {
    TF p[EF::NP];
#pragma unroll
    for (int q = 0; q < EF::NP; ++q) p[q] = ((const TF *)planes)[eoff<PF>(i, j, q, Mp)];
    x = EF::dec(p);
  }
  ((TB *)out)[i * Mp + j] = (TB)x;
}

// G = (g + g^T)/2 of the caller's M x M gradient over 64 x 64 tiles of the
// padded matrix (zero outside M x M).
template <int PB>
__global__ __launch_bounds__(256) void k_bload(const void *g, int64_t ldg, int dtype, int64_t M,
                                               int64_t Mp, void *G) {
  using TB = typename Enc<PB>::T;
  __shared__ double hs[64][65], ht[64][65];
  const int64_t I = (int64_t)blockIdx.y * 64, J = (int64_t)blockIdx.x * 64;
  const int tid = threadIdx.x, row = tid >> 2, c0 = (tid & 3) * 16;
  auto ld = [&](int64_t r, int64_t c) -> double {
    if (r >= M || c >= M) return 0.0;
    return dtype == GCP_DTYPE_F64 ? ((const double *)g)[r * ldg + c]
                                  : (double)((const float *)g)[r * ldg + c];
  };
  for (int c = 0; c < 16; ++c) {
    hs[row][c0 + c] = ld(I + row, J + c0 + c);
    ht[row][c0 + c] = ld(J + row, I + c0 + c);
  }
  __syncthreads();
  for (int c = 0; c < 16; ++c) {
    const int64_t i = I + row, j = J + c0 + c;
    ((TB *)G)[i * Mp + j] = (TB)(0.5 * (hs[row][c0 + c] + ht[c0 + c][row]));
  }
}

// Row sums of G0 o D0 and the diagonal of G0 (one block per row).
template <int PB>
__global__ __launch_bounds__(256) void k_bdot(BwdInitArgs a) {
  using TB = typename Enc<PB>::T;
  __shared__ double s[256];
  const int64_t i = blockIdx.x;
  const TB *G0 = (const TB *)a.G0, *D0 = (const TB *)a.D0;
  double v = 0.0;
  for (int64_t j = threadIdx.x; j < a.Mp; j += 256)
    v += (double)G0[i * a.Mp + j] * (double)D0[i * a.Mp + j];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.rows[i] = s[0];
    a.rows[a.Mp + i] = (double)G0[i * a.Mp + i];
  }
}

// sums[0] = <G0, D0>, sums[1] = Tr G0 (fixed order, one block).
__global__ __launch_bounds__(256) void k_bsum(BwdInitArgs a) {
  __shared__ double s0[256], s1[256];
  double v0 = 0.0, v1 = 0.0;
  for (int64_t i = threadIdx.x; i < a.Mp; i += 256) {
    v0 += a.rows[i];
    v1 += a.rows[a.Mp + i];
  }
  s0[threadIdx.x] = v0;
  s1[threadIdx.x] = v1;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      s0[threadIdx.x] += s0[threadIdx.x + w];
      s1[threadIdx.x] += s1[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.sums[0] = s0[0];
    a.sums[1] = s1[0];
  }
}

// dL/dH = sign (-beta G0 + s I) (M x M, leading dimension ldh).
template <int PB>
__global__ __launch_bounds__(256) void k_bdh(BwdInitArgs a) {
  using TB = typename Enc<PB>::T;
  // rows on the x dimension of the grid (no 64K limit), 256 columns per block on y
  const int64_t i = blockIdx.x;
  const int64_t j = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (j >= a.M) return;
  double s = 0.0, k = 0.0;
  if (a.beta != 0.0) {
    const double gd = a.sums[0], tr = a.sums[1];
    const double g_muh = (gd - a.theta * tr) / a.beta;   // <G0, mu I - H>
    s = (a.beta * tr + a.dbeta * g_muh) / (double)a.M;
    if (a.hdev > 0.0) k = g_muh / a.hdev;               // alpha-searched slope
  }
  double x = -a.beta * (double)((const TB *)a.G0)[i * a.Mp + j];
  if (k != 0.0) x += k * (double)((const TB *)a.D0)[i * a.Mp + j];
  if (i == j) x += s - k * a.theta;
  x *= a.sign;
  if (a.dtype == GCP_DTYPE_F64)
    ((double *)a.dH)[i * a.ldh + j] = x;
  else
    ((float *)a.dH)[i * a.ldh + j] = (float)x;
}

// ---------------------------------------------------------------- dispatch
template <int PF>
static hipError_t store_pf(int bprec, const void *planes, const double *dg, int64_t Mp, void *out,
                           hipStream_t st) {
  const dim3 grid((unsigned)Mp, (unsigned)((Mp + 255) / 256));
  if (bprec == GCP_FP64)
    k_bstore<PF, GCP_FP64><<<grid, 256, 0, st>>>(planes, dg, Mp, out);
  else
    k_bstore<PF, GCP_FP32><<<grid, 256, 0, st>>>(planes, dg, Mp, out);
  return hipGetLastError();
}

hipError_t launch_bwd_store(int fprec, int bprec, const void *planes, const double *dg, int64_t Mp,
                            void *out, hipStream_t st) {
  if (bprec != GCP_FP64 && bprec != GCP_FP32) return hipErrorInvalidValue;
  switch (fprec) {
    case GCP_FP64: return store_pf<GCP_FP64>(bprec, planes, dg, Mp, out, st);
    case GCP_FP32: return store_pf<GCP_FP32>(bprec, planes, dg, Mp, out, st);
    case GCP_BF16: return store_pf<GCP_BF16>(bprec, planes, dg, Mp, out, st);
    case GCP_FP16: return store_pf<GCP_FP16>(bprec, planes, dg, Mp, out, st);
    case GCP_BF16X3: return store_pf<GCP_BF16X3>(bprec, planes, dg, Mp, out, st);
    case GCP_FP16X3: return store_pf<GCP_FP16X3>(bprec, planes, dg, Mp, out, st);
    case GCP_BF16X6: return store_pf<GCP_BF16X6>(bprec, planes, dg, Mp, out, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_bwd_load(int bprec, const void *g, int64_t ldg, int dtype, int64_t M,
                           int64_t Mp, void *G, hipStream_t st) {
  const dim3 grid((unsigned)(Mp / 64), (unsigned)(Mp / 64));
  if (bprec == GCP_FP64)
    k_bload<GCP_FP64><<<grid, 256, 0, st>>>(g, ldg, dtype, M, Mp, G);
  else if (bprec == GCP_FP32)
    k_bload<GCP_FP32><<<grid, 256, 0, st>>>(g, ldg, dtype, M, Mp, G);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int P>
static hipError_t bgemm_p(const BwdArgs &a, hipStream_t st) {
  const unsigned ntri = (unsigned)(a.nt * (a.nt + 1) / 2);
  switch (a.mode) {
    case 0: k_bgemm<P, 0><<<ntri, NTH, 0, st>>>(a); break;
    case 1: k_bgemm<P, 1><<<(unsigned)(2 * a.nt * a.nt), NTH, 0, st>>>(a); break;
    case 2: k_bgemm<P, 2><<<ntri, NTH, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_bwd_gemm(int bprec, const BwdArgs &a, hipStream_t st) {
  if (bprec == GCP_FP64) return bgemm_p<GCP_FP64>(a, st);
  if (bprec == GCP_FP32) return bgemm_p<GCP_FP32>(a, st);
  return hipErrorInvalidValue;
}

hipError_t launch_bwd_kappa(const double *tpart, int ntri, int nfull, double da, double db,
                            double de, double *kappa, hipStream_t st) {
  k_bkappa<<<1, 256, 0, st>>>(tpart, ntri, nfull, da, db, de, kappa);
  return hipGetLastError();
}

hipError_t launch_bwd_init(int bprec, const BwdInitArgs &a, hipStream_t st) {
  const dim3 gout((unsigned)a.M, (unsigned)((a.M + 255) / 256));
  if (bprec == GCP_FP64) {
    k_bdot<GCP_FP64><<<(unsigned)a.Mp, 256, 0, st>>>(a);
    k_bsum<<<1, 256, 0, st>>>(a);
    k_bdh<GCP_FP64><<<gout, 256, 0, st>>>(a);
  } else if (bprec == GCP_FP32) {
    k_bdot<GCP_FP32><<<(unsigned)a.Mp, 256, 0, st>>>(a);
    k_bsum<<<1, 256, 0, st>>>(a);
    k_bdh<GCP_FP32><<<gout, 256, 0, st>>>(a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gcp
