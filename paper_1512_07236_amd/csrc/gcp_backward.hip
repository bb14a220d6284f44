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
// One adjoint step is two launches of 64 x 64 MFMA tile products over upper
// tiles, two products per tile, all of the A * B^T row-panel form of the
// forward:
//   k_bpair   D_i G_j and D_j G_i, i.e. both tiles of A = D Gbar' of a mirrored
//             pair: stores S = A + A^T and T = A^T, and sums <A, D> = <Gbar', D^2>
//             and <Gbar', D> (both = 1/2 <S, .> by symmetry)
//   k_bstep   D_i T_j + S_i D_j = D^2 Gbar' + (D Gbar' D + Gbar' D^2), the two
//             added in FP64; epilogue: Gbar_n from Gbar', S, D and their sum
// with S = D Gbar' + Gbar' D.  The term -3 kappa D^2 / (T1 - T2) is linear in
// a third product D D, which k_badd folds into the first one by adding a
// multiple of D to T once kappa is known (T is then rounded once more in the
// adjoint's type).  That is 4 M^3 flops per step; with
// D^2 formed for itself, D Gbar' and D^2 Gbar' as general products and D
// Gbar' D it was 6 M^3.  PMCP alone needs D^2: k_bx2 forms its tiles for the
// sum <Gbar', D^3> = 1/2 <S, D^2> and does not store them.
// kappa is reduced on the device in a fixed order, so the whole backward is
// bitwise reproducible.
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

template <int P> struct BwdCfg {
  using S = typename TileCfg<P>::S;
  static constexpr int V = T64 * VP * (int)sizeof(S);
  static constexpr int MM = TileCfg<P>::SMEM > V ? TileCfg<P>::SMEM : V;
  static constexpr int SMEM = MM + 8 * 8;    // and two sums per wave
  // per CU, as k_tile; in FP64 k_bpair spills 29 registers and k_bstep 6
  static constexpr int BLOCKS = Enc<P>::KIND == 0 ? 4 : 2;
};

// Tile of this block, and for a tile of the last partial round its split: the
// two products of such a tile are nsplit/2 blocks each (nsplit even).
struct BwdTile {
  int ti, tj, lin, split;
};
__device__ __forceinline__ BwdTile bwd_tile(const BwdArgs &a) {
  BwdTile t{0, 0, 0, -1};
  const int u = (int)blockIdx.x - a.nfull;
  if (u < 0) {
    tile_of_block(blockIdx.x, a.nfull, a.nt, t.ti, t.tj, t.lin);
  } else {
    const int ntail = ((int)gridDim.x - a.nfull) / a.nsplit;
    t.split = u / ntail;
    t.lin = a.nfull + u % ntail;
    tile_of_index(t.lin, a.nt, t.ti, t.tj);
  }
  return t;
}

// Thread tid works on columns 4 (tid % 16) .. +3 of rows 16 q + tid / 16 of
// the tile, so that inputs are read and results written as rows of 64
// elements; mirrored tiles go through LDS.
template <int P> struct BwdThread {
  using T = typename Enc<P>::T;
  using S = typename TileCfg<P>::S;
  typedef T v4t __attribute__((ext_vector_type(4)));
  int c4, r0;
  char *smem;
  __device__ explicit BwdThread(char *s) : c4((threadIdx.x & 15) * 4), r0(threadIdx.x >> 4), smem(s) {}
  __device__ __forceinline__ void take(S (&v)[4][4]) const {   // own elements of the tile in LDS
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q][e] = ((const S *)smem)[(q * 16 + r0) * VP + c4 + e];
  }
  __device__ __forceinline__ void put(const S (&v)[4][4]) const {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) ((S *)smem)[(q * 16 + r0) * VP + c4 + e] = v[q][e];
    __syncthreads();
  }
  __device__ __forceinline__ void take_mirror(S (&v)[4][4]) const {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q][e] = ((const S *)smem)[(c4 + e) * VP + q * 16 + r0];
  }
  __device__ __forceinline__ void store(T *O, int64_t i0, int64_t j0, int64_t Mp,
                                        const S (&v)[4][4]) const {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(v4t *)(O + (i0 + q * 16 + r0) * Mp + j0 + c4) = v4t{v[q][0], v[q][1], v[q][2], v[q][3]};
  }
};

// Sums of x and y over the tile into tpart[lin] and tpart[ntri + lin].
__device__ __forceinline__ void tile_sums(const BwdArgs &a, int lin, double x, double y, double *red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ntri = a.nt * (a.nt + 1) / 2;
  x = wave_sum(x);
  y = wave_sum(y);
  if (lane == 0) {
    red[wave] = x;
    red[4 + wave] = y;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.tpart[lin] = ((red[0] + red[1]) + red[2]) + red[3];
    a.tpart[ntri + lin] = ((red[4] + red[5]) + red[6]) + red[7];
  }
}

template <int P>
__global__ __launch_bounds__(NTH, BwdCfg<P>::BLOCKS) void k_bpair(BwdArgs a) {
  using B = BwdCfg<P>;
  using T = typename Enc<P>::T;
  using S = typename B::S;
  typedef T v4t __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) char smem[B::SMEM];
  const int64_t Mp = a.Mp;
  const BwdTile t = bwd_tile(a);
  const int64_t i0 = (int64_t)t.ti * T64, j0 = (int64_t)t.tj * T64;
  const int nk = (int)(Mp / TileCfg<P>::KT), half = a.nsplit / 2;
  const bool dtile = t.ti == t.tj;
  const BwdThread<P> me(smem);
  S p[4][4], m[4][4];   // A(i, j), and A(j, i) read as its transpose
  if (t.split < 0) {
    tile_product<P>(a.D, a.G, i0, j0, Mp, smem, a.fold, 0, nk);
    me.take(p);
    if (!dtile) {
      __syncthreads();   // read by all before the next product's stages land in it
      tile_product<P>(a.D, a.G, j0, i0, Mp, smem, a.fold, 0, nk);
    }
  } else {
    const int which = t.split >= half, s = t.split - which * half;
    tile_product<P>(a.D, a.G, which ? j0 : i0, which ? i0 : j0, Mp, smem, a.fold, s * nk / half,
                    (s + 1) * nk / half);
    const int64_t ps = (int64_t)((int)gridDim.x - a.nfull) / a.nsplit * (T64 * T64);
    S *w = (S *)a.ws + (int64_t)(t.lin - a.nfull) * (T64 * T64) + me.r0 * T64 + me.c4;
    if (!publish_split((const S *)smem + me.r0 * VP + me.c4, w + t.split * ps,
                       a.cnt + (t.lin - a.nfull), a.nsplit, smem))
      return;
    double v[4][4];
    add_partials(w + half * ps, ps, half, v);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) p[q][e] = (S)v[q][e];
    me.put(p);   // A(j, i), as a whole product leaves it
    add_partials(w, ps, half, v);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) p[q][e] = (S)v[q][e];
  }
  me.take_mirror(m);
  S s[4][4];
  double sd = 0.0, gd = 0.0;
  const T *__restrict__ D = (const T *)a.D;
  const T *__restrict__ G = (const T *)a.G;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t o = (i0 + q * 16 + me.r0) * Mp + j0 + me.c4;
    const v4t dv = *(const v4t *)(D + o), gv = *(const v4t *)(G + o);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double x = (double)p[q][e] + (double)m[q][e];
      s[q][e] = (S)x;
      sd += x * (double)dv[e];
      gd += (double)gv[e] * (double)dv[e];
    }
  }
  T *To = (T *)a.T, *So = (T *)a.S;
  me.store(To, i0, j0, Mp, m);
  me.store(So, i0, j0, Mp, s);
  if (!dtile) {
    S x[4][4];
    me.put(p);
    me.take_mirror(x);
    me.store(To, j0, i0, Mp, x);
    me.put(s);
    me.take_mirror(x);
    me.store(So, j0, i0, Mp, x);
  }
  tile_sums(a, t.lin, dtile ? 0.5 * sd : sd, dtile ? gd : 2.0 * gd, (double *)(smem + B::MM));
}

// T += *kappa w D (the D^2 term of the update's kappa part).
template <int P>
__global__ __launch_bounds__(256) void k_badd(const void *D, void *T, const double *kappa, double w,
                                              int64_t n4) {
  using TB = typename Enc<P>::T;
  typedef TB v4t __attribute__((ext_vector_type(4)));
  const double f = *kappa * w;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    const v4t d = ((const v4t *)D)[i];
    v4t t = ((const v4t *)T)[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = (TB)((double)t[e] + f * (double)d[e]);
    ((v4t *)T)[i] = t;
  }
}

template <int P>
__global__ __launch_bounds__(NTH, BwdCfg<P>::BLOCKS) void k_bstep(BwdArgs a) {
  using B = BwdCfg<P>;
  using T = typename Enc<P>::T;
  using S = typename B::S;
  typedef T v4t __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) char smem[B::SMEM];
  const int64_t Mp = a.Mp;
  const BwdTile t = bwd_tile(a);
  const int64_t i0 = (int64_t)t.ti * T64, j0 = (int64_t)t.tj * T64;
  const int nk = (int)(Mp / TileCfg<P>::KT), half = a.nsplit / 2;
  const bool dtile = t.ti == t.tj;
  const BwdThread<P> me(smem);
  double v[4][4];
  S p[4][4];
  if (t.split < 0) {
    tile_product<P>(a.D, a.T, i0, j0, Mp, smem, a.fold, 0, nk);
    me.take(p);
    __syncthreads();   // read by all before the next product's stages land in it
    tile_product<P>(a.S, a.D, i0, j0, Mp, smem, a.fold, 0, nk);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[q][e] = (double)p[q][e] + (double)((const S *)smem)[(q * 16 + me.r0) * VP + me.c4 + e];
  } else {
    const int which = t.split >= half, s = t.split - which * half;
    tile_product<P>(which ? a.S : a.D, which ? a.D : a.T, i0, j0, Mp, smem, a.fold, s * nk / half,
                    (s + 1) * nk / half);
    const int64_t ps = (int64_t)((int)gridDim.x - a.nfull) / a.nsplit * (T64 * T64);
    S *w = (S *)a.ws + (int64_t)(t.lin - a.nfull) * (T64 * T64) + me.r0 * T64 + me.c4;
    if (!publish_split((const S *)smem + me.r0 * VP + me.c4, w + t.split * ps,
                       a.cnt + (t.lin - a.nfull), a.nsplit, smem))
      return;
    add_partials(w, ps, a.nsplit, v);
  }
  const T *__restrict__ D = (const T *)a.D;
  const T *__restrict__ G = (const T *)a.G;
  const T *__restrict__ Sm = (const T *)a.S;
  const double k = *a.kappa * a.inv_t12, kd = k * (2.0 + 2.0 * a.c), ki = -k * a.c;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = q * 16 + me.r0;
    const int64_t o = (i0 + row) * Mp + j0 + me.c4;
    const v4t dv = *(const v4t *)(D + o), gv = *(const v4t *)(G + o), sv = *(const v4t *)(Sm + o);
    // the I of c (I - 2D) is that of the M x M problem: the padding of Gbar
    // stays zero, as Tr Gbar_0 and <Gbar_0, D_0> take it to be
    const bool drow = dtile && i0 + row < a.M;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      p[q][e] = (S)(a.a * (double)gv[e] + a.b * (double)sv[e] + a.e * v[q][e] + kd * (double)dv[e] +
                    (drow && row == me.c4 + e ? ki : 0.0));
  }
  T *O = (T *)a.out;
  if (!dtile) me.store(O, i0, j0, Mp, p);
  me.put(p);
  // mirrored tile; a diagonal tile is written whole, its lower half from the
  // upper one
  S x[4][4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = q * 16 + me.r0, c = me.c4 + e;
      const bool up = dtile && row < c;
      x[q][e] = ((const S *)smem)[(up ? row : c) * VP + (up ? c : row)];
    }
  me.store(O, j0, i0, Mp, x);
}

// PMCP: tiles of X2 = D D, not stored, for 1/2 <S, D^2> into tpart[2 ntri ..).
template <int P>
__global__ __launch_bounds__(NTH, BwdCfg<P>::BLOCKS) void k_bx2(BwdArgs a) {
  using B = BwdCfg<P>;
  using T = typename Enc<P>::T;
  using S = typename B::S;
  typedef T v4t __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) char smem[B::SMEM];
  const int64_t Mp = a.Mp;
  int ti, tj, lin;
  tile_of_block(blockIdx.x, a.nt, ti, tj, lin);
  const int64_t i0 = (int64_t)ti * T64, j0 = (int64_t)tj * T64;
  tile_product<P>(a.D, a.D, i0, j0, Mp, smem, a.fold, 0, (int)(Mp / TileCfg<P>::KT));
  const BwdThread<P> me(smem);
  S v[4][4];
  me.take(v);
  double x = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const v4t sv = *(const v4t *)((const T *)a.S + (i0 + q * 16 + me.r0) * Mp + j0 + me.c4);
#pragma unroll
    for (int e = 0; e < 4; ++e) x += (double)sv[e] * (double)v[q][e];
  }
  x = wave_sum(ti == tj ? 0.5 * x : x);
  double *red = (double *)(smem + B::MM);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0)
    a.tpart[a.nt * (a.nt + 1) + lin] = ((red[0] + red[1]) + red[2]) + red[3];
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
__global__ __launch_bounds__(256) void k_bkappa(const double *tpart, int ntri, double da,
                                                double db, double de, double *kappa) {
  __shared__ double s[256];
  const double sx2 = block_sum(tpart, 0, ntri, s);
  const double sd = block_sum(tpart, ntri, 2 * ntri, s);
  const double sx3 = de != 0.0 ? block_sum(tpart, 2 * ntri, 3 * ntri, s) : 0.0;
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

// G = (g + g^T)/2 of the caller's M x M matrix over the padded matrix (zero
// outside M x M).  Bound by HBM; M = 3000, FP64: 137 -> 31 us against reading
// 16 consecutive elements per thread of every tile and its mirror.
template <int PB>
__global__ __launch_bounds__(256) void k_bload(const void *g, int64_t ldg, int dtype, int64_t M,
                                               int64_t Mp, void *G) {
  using TB = typename Enc<PB>::T;
  __shared__ double ta[64][65], tb[64][65];
  double ha[16], hb[16];
  const SymPair p =
      dtype == GCP_DTYPE_F64
          ? sym_pair(blockIdx.x, M,
                     [&](int64_t r, int64_t c) { return ((const double *)g)[r * ldg + c]; }, ha, hb,
                     ta, tb)
          : sym_pair(blockIdx.x, M,
                     [&](int64_t r, int64_t c) { return (double)((const float *)g)[r * ldg + c]; },
                     ha, hb, ta, tb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  TB *__restrict__ O = (TB *)G;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + wave;
    O[(p.I + r) * Mp + p.J + lane] = (TB)(0.5 * (ha[q] + tb[lane][r]));
    if (!p.diag) O[(p.J + r) * Mp + p.I + lane] = (TB)(0.5 * (hb[q] + ta[lane][r]));
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
  const int64_t nt = Mp / 64;
  const unsigned grid = (unsigned)(nt * (nt + 1) / 2);
  if (bprec == GCP_FP64)
    k_bload<GCP_FP64><<<grid, 256, 0, st>>>(g, ldg, dtype, M, Mp, G);
  else if (bprec == GCP_FP32)
    k_bload<GCP_FP32><<<grid, 256, 0, st>>>(g, ldg, dtype, M, Mp, G);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int P>
static hipError_t bwd_step(const BwdArgs &a, int mode, hipStream_t st) {
  const int ntri = a.nt * (a.nt + 1) / 2;
  const unsigned grid = (unsigned)(a.nfull + (ntri - a.nfull) * a.nsplit);
  const int64_t n4 = a.Mp * a.Mp / 4;
  switch (mode) {
    case BWD_PAIR: k_bpair<P><<<grid, NTH, 0, st>>>(a); break;
    case BWD_X2: k_bx2<P><<<(unsigned)ntri, NTH, 0, st>>>(a); break;
    case BWD_STEP:
      k_badd<P><<<(unsigned)(n4 / 1024 + 1 > 4096 ? 4096 : n4 / 1024 + 1), 256, 0, st>>>(
          a.D, a.T, a.kappa, -3.0 * a.inv_t12 / a.e, n4);
      k_bstep<P><<<grid, NTH, 0, st>>>(a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_bwd(int bprec, const BwdArgs &a, int mode, hipStream_t st) {
  if (bprec == GCP_FP64) return bwd_step<GCP_FP64>(a, mode, st);
  if (bprec == GCP_FP32) return bwd_step<GCP_FP32>(a, mode, st);
  return hipErrorInvalidValue;
}

hipError_t launch_bwd_kappa(const double *tpart, int ntri, double da, double db, double de,
                            double *kappa, hipStream_t st) {
  k_bkappa<<<1, 256, 0, st>>>(tpart, ntri, da, db, de, kappa);
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
