// gcp_kernels.hip -- device kernels of the purification path (gfx950 / CDNA4).
//
// One purification iteration (eq. (hpcp3) expanded with Dbar = I - D):
//   D_{n+1} = (1 - 2c) D + (2 + 2c) D^2 - 2 D^3,   c = (T2 - T3) / (T1 - T2),
//   T_k = Tr D^k.
// It is two symmetric matrix products over the upper triangle of output tiles
// (results mirrored), 32 x 32 (k_small), 64 x 64 (k_tile) or, for 16-bit
// encodings above M = 3008, pairs of 128 x 128 (k_gemm16):
//   K1 (mode 0):  X2 = D D        epilogue: store X2, row sums of X2 o D
//                                 (diag of D^3) and ||X2 - D||_F^2
//   K2 (mode 1):  X3 = X2 D       epilogue: D_{n+1} from D, X2 and X3 (X3 never
//                                 stored), row sums of D_{n+1} o D_{n+1} (diag
//                                 of D_{n+1}^2) and ||D_{n+1} - D_n||_F^2
// Both are A * B^T products of row panels (all iterates are symmetric), so
// both operands are read along contiguous K.  Row sums go to a [slot][row]
// FP64 buffer (one writer per slot).  The last block of a tile kernel, or
// k_reduce after pairs, adds them in a fixed order and runs the scalar step:
// every trace, and therefore c_n, is bitwise reproducible.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gcp_encode.h"
#include "gcp_kernels.h"
#include "gcp_mma.h"

namespace gcp {

// ------------------------------------------------------- scalar step
__device__ __forceinline__ double ld_agent(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The scalar step at this point of the iteration (one thread); returns the
// solve's status.
__device__ int take_step(const RedArgs &a, double sum_out, double sum_extra, double sum_tiles) {
  Scalars *sc = a.sc;
  if (a.mode == 0) {            // after the initial guess
    sc->t2 = sum_out;
    sc->t1 = sum_extra;
  } else if (a.mode == 1) {     // after D^2: decide and form c
    const double t1 = sc->t1, t2 = sc->t2, t3 = sum_out, om = sum_tiles;
    const double ddbar = t1 - t2;
    int status = 0;
    double c = NAN;
    if (!isfinite(t1) || !isfinite(t2) || !isfinite(om)) {
      status = 3;
    } else if (fabs(ddbar) <= a.tol_ddbar || sqrt(om) <= a.tol_idem) {
      status = 1;
    } else if (a.iter >= a.max_iter) {
      status = 2;
    } else {
      if (ddbar > 0.0) c = (t2 - t3) / ddbar;
      // Tr(D Dbar) <= 0 or c outside [0, 1] is a runaway, unless |Tr(D Dbar)|
      // is already within the encoding's rounding floor, where it (and c)
      // is rounding noise and stops decreasing: the iterate is then as
      // idempotent as the encoding allows and the solve stops there.
      const bool bad = !(ddbar > 0.0) || !isfinite(c) || c < 0.0 || c > 1.0;
      const bool stalled = !a.recheck && fabs(ddbar) >= sc->prev_ddbar;
      if ((bad || stalled) && fabs(ddbar) <= a.floor_ddbar) status = 4;
      else if (bad) status = 3;
    }
    if (!a.recheck) sc->prev_ddbar = fabs(ddbar);
    if (status != 0) sc->iter = a.iter;
    sc->t3 = t3;
    sc->omega = om;
    sc->c = c;
    sc->status = status;
    double *h = a.hist + (int64_t)a.iter * 9;
    const double gamma = 1.0 / 3.0 - 2.0 / 3.0 * c;
    h[0] = a.iter; h[1] = t1; h[2] = t2; h[5] = om;
    if (status == 0) {
      h[3] = t3; h[4] = c; h[6] = gamma;
      h[7] = om - gamma * (3.0 * t2 - 2.0 * t3 - a.N);
    } else {
      h[3] = h[4] = h[6] = h[7] = NAN;
    }
    h[8] = NAN;
    return status;
  } else {                      // after the update: traces of D_{n+1}
    sc->t2 = sum_out;
    sc->t1 = sum_extra;
    sc->step = sum_tiles;
    a.hist[(int64_t)a.iter * 9 + 8] = sqrt(sum_tiles);
    if (!a.early_stop) return 0;
    // The stops of the mode-1 decision that need only T1 and T2 of D_{n+1},
    // taken here so that the square of the last iterate is never formed:
    // |Tr(D Dbar)| within tol_ddbar, or within the rounding floor while not
    // decreasing or not positive (below max_iter, where mode 1 would report
    // max_iter first).  Everything else (non-finite traces, c outside
    // [0, 1], max_iter) is left to mode 1, which would take the same
    // decision on the same traces.
    const double t1 = sum_extra, t2 = sum_out, ddbar = t1 - t2;
    const int nx = a.iter + 1;
    int status = 0;
    if (isfinite(t1) && isfinite(t2)) {
      if (fabs(ddbar) <= a.tol_ddbar) status = 1;
      else if (nx < a.max_iter && (!(ddbar > 0.0) || fabs(ddbar) >= sc->prev_ddbar) &&
               fabs(ddbar) <= a.floor_ddbar)
        status = 4;
    }
    if (status == 0) return 0;
    sc->status = status;
    sc->iter = nx;
    sc->on_traces = 1;
    sc->omega = NAN;
    double *h = a.hist + (int64_t)nx * 9;
    h[0] = nx; h[1] = t1; h[2] = t2;
    h[3] = h[4] = h[5] = h[6] = h[7] = h[8] = NAN;
    return status;
  }
  return 0;
}

// Stores to pinned host memory, which the host polls: the values are out
// before the word that announces them.
template <class T>
__device__ __forceinline__ void st_host(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void host_order() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ void scalar_step(const RedArgs &a, double sum_out, double sum_extra,
                            double sum_tiles) {
  const int status = take_step(a, sum_out, sum_extra, sum_tiles);
  if (!a.post || (status == 0 && a.what == POST_NONE)) return;
  Scalars *p = a.post;
  if (status != 0 || a.what == POST_ALL) {
    const Scalars *sc = a.sc;
    st_host(&p->t1, sc->t1);
    st_host(&p->t2, sc->t2);
    st_host(&p->t3, sc->t3);
    st_host(&p->omega, sc->omega);
    st_host(&p->iter, sc->iter);
    st_host(&p->on_traces, sc->on_traces);
    host_order();
    st_host(&p->status, status);
    host_order();
  }
  st_host(&p->seq, a.seq);
}

// ------------------------------------------------- epilogue of one tile
// The epilogues work on TE x TE tiles (64 or 32; ti <= tj) of the output with
// 256 threads: TE/4 lanes take a row, 4 columns each, so that it is one
// contiguous access; thread tid holds the rows RP q + tid / (TE/4), q < NQ.
// The encoded results also go to LDS, from which the mirrored tile is written
// as rows.
template <int P, int TE> struct FinCfg {
  using T = typename Enc<P>::T;
  static constexpr int RP = 1024 / TE, NQ = TE / RP;
  static constexpr int QC = sizeof(T) == 8 && NQ > 2 ? 2 : NQ;   // rows of a thread taken together
  static constexpr int VP = TE + 1;                   // LDS row pitch (elements)
  static constexpr int V = Enc<P>::NP * TE * VP * (int)sizeof(T);   // encoded results
  static constexpr int SUMS = (V + 15) / 16 * 16;                   // then FP64 sums
  static constexpr int SMEM_FIN = SUMS + (TE + 4 * TE + 4) * 8;
  static constexpr int SMEM_RED = 8 * 64 * 8;                       // finish_rows
  static constexpr int SMEM = SMEM_FIN > SMEM_RED ? SMEM_FIN : SMEM_RED;
};

// Row block R (TE rows) is complete when all nt tiles that touch it have
// stored their row sums.  The block that completes it adds the slots (the
// q-th of its 256/TE groups of threads the slots s = q (mod 256/TE) in
// ascending order, then the group sums in order), and
// the block that completes the last row block adds the block sums and the
// tile sums in a fixed order and runs the scalar step: the sums do not depend
// on the order in which blocks finish.  Sums that cross blocks inside the
// launch are stored and loaded at agent scope (the XCDs' L2s are not coherent
// for plain accesses) and are out before the counters move.
template <int TE>
__device__ __forceinline__ void finish_rows(const RedArgs &a, int ti, int tj, int nt,
                                            double *sm) {
  constexpr int NG = 256 / TE;
  const int tid = threadIdx.x, lane = tid & 63, row = tid % TE, q = tid / TE;
  int *flag = (int *)sm;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    int f = atomicAdd(a.rcnt + ti, 1u) == (unsigned)nt - 1 ? 1 : 0;
    if (tj != ti && atomicAdd(a.rcnt + tj, 1u) == (unsigned)nt - 1) f |= 2;
    *flag = f;
  }
  __syncthreads();
  const int f = *flag;
  if (f == 0) return;
  bool last = false;
  for (int h = 0; h < 2; ++h) {
    if (!((f >> h) & 1)) continue;   // block-uniform
    const int R = h ? tj : ti;
    const int64_t i = (int64_t)R * TE + row;
    double w = 0.0;
#pragma unroll 8
    for (int s = q; s < nt; s += NG) w += ld_agent(a.part + (int64_t)s * a.Mp + i);
    __syncthreads();
    sm[tid] = w;
    __syncthreads();
    if (tid < 64) {   // whole wave; lanes past the block's rows add nothing
      double v = 0.0, x = 0.0;
      if (tid < TE) {
#pragma unroll
        for (int k = 0; k < NG; ++k) v += sm[k * TE + tid];
        a.out[i] = v;
        if (a.extra) x = ld_agent(a.extra + i);
      }
      v = wave_sum(v);
      x = wave_sum(x);
      if (tid == 0) {
        st_agent(a.bpart + 2 * R, v);
        st_agent(a.bpart + 2 * R + 1, x);
        a.rcnt[R] = 0u;   // ready for the next launch
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        flag[2 * 256] = atomicAdd(a.counter, 1u) == (unsigned)nt - 1;
      }
    }
    __syncthreads();
    last = last || flag[2 * 256];
  }
  if (!last) return;
  double b1 = 0.0, b2 = 0.0, b3 = 0.0;
  for (int b = tid; b < nt; b += 256) {
    b1 += ld_agent(a.bpart + 2 * b);
    b2 += ld_agent(a.bpart + 2 * b + 1);
  }
#pragma unroll 4
  for (int t = tid; t < a.ntiles; t += 256) b3 += ld_agent(a.tpart + t);
  b1 = wave_sum(b1);
  b2 = wave_sum(b2);
  b3 = wave_sum(b3);
  __syncthreads();
  if (lane == 0) {
    const int wave = tid >> 6;
    sm[wave] = b1;
    sm[4 + wave] = b2;
    sm[8 + wave] = b3;
  }
  __syncthreads();
  if (tid != 0) return;
  *a.counter = 0u;
  scalar_step(a, ((sm[0] + sm[1]) + sm[2]) + sm[3], ((sm[4] + sm[5]) + sm[6]) + sm[7],
              ((sm[8] + sm[9]) + sm[10]) + sm[11]);
}

// Epilogue of tile (ti, tj): the update from the products of this thread's
// elements (vload(q0, v) gives rows q0 .., SC^2 times the product), stored at (i, j) and
// mirrored, with its row sums, column sums and tile sum.  lin: the tile's
// index among all upper tiles.  DT: a diagonal tile, whose elements below
// the diagonal are the mirror of those above and whose diagonal comes from
// the FP64 vectors; the other tiles are compiled without those cases.
// Elements are kept in the stored units SC x, whose scaling is exact.
//
// Bound by the chain of memory round trips, and for many tiles by vector
// instructions (about 100 per element before the diagonal cases and the
// scalings went, 40 now).
template <int P, int TE, int MODE, bool DT, class V>
__device__ __forceinline__ void finish_tile(const GemmArgs &g, int ti, int tj, int lin, V &&vload,
                                            char *smem) {
  using E = Enc<P>;
  using T = typename E::T;
  typedef T v4t __attribute__((ext_vector_type(4)));
  using F = FinCfg<P, TE>;
  constexpr int NP = E::NP, RP = F::RP, NQ = F::NQ, QC = F::QC, VP = F::VP, LR = TE / 4;
  constexpr double SC = E::SC, INV = 1.0 / SC;
  const int64_t Mp = g.Mp, i0 = (int64_t)ti * TE, j0 = (int64_t)tj * TE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c4 = tid % LR * 4, r0 = tid / LR;
  const T *__restrict__ Ag = (const T *)g.A;
  const T *__restrict__ Bg = (const T *)g.B;
  T *__restrict__ Og = (T *)g.out;
  T *Vt = (T *)smem;
  double rDj[4], colacc[4] = {}, rowacc[NQ], tacc = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) rDj[e] = g.rD[j0 + c4 + e];
  double a_coef = 0.0, b_coef = 0.0, e_coef = 0.0;
  if constexpr (MODE == 1) update_coefs(g.method, g.coef[0], a_coef, b_coef, e_coef);
  // the inputs of QC rows are loaded together, before any of their stores (the
  // compiler cannot tell the output from the inputs); four FP64 rows would
  // not fit the registers of four blocks per CU
#pragma unroll
  for (int q0 = 0; q0 < NQ; q0 += QC) {
    v4t dv[QC][NP], xv[QC][NP];
    double ri[QC], dgi[QC], d2i[QC], d3i[QC];   // (the last three: the diagonal, DT)
#pragma unroll
    for (int u = 0; u < QC; ++u) {
      const int64_t i = i0 + (q0 + u) * RP + r0;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        dv[u][p] = *(const v4t *)(Bg + eoff<P>(i, j0 + c4, p, Mp));
        if constexpr (MODE == 1) xv[u][p] = *(const v4t *)(Ag + eoff<P>(i, j0 + c4, p, Mp));
      }
      ri[u] = MODE == 0 ? g.rD[i] : g.s2[i];
      if constexpr (DT) {
        dgi[u] = g.dg[i];
        d2i[u] = g.d2[i];
        if constexpr (MODE == 1) d3i[u] = g.d3[i];
      }
    }
    double v[QC][4];
    vload(q0, v);
#pragma unroll
    for (int u = 0; u < QC; ++u) {
      const int q = q0 + u, row = q * RP + r0;
      const int64_t i = i0 + row;
      v4t ov[NP];
      double rs = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool diag = DT && row == c4 + e, lower = DT && row > c4 + e;
        T dp[NP], op[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) dp[p] = dv[u][p][e];
        const double pv = v[u][e] * INV;   // SC times the product
        double Dm = E::dec_s(dp), prod, diff;
        if constexpr (MODE == 0) {
          // X2 = (D_enc + diag(rD))^2: exact diagonal-residual correction
          double x2 = pv + Dm * (ri[u] + rDj[e]);
          if (diag) {
            Dm = SC * dgi[u];
            x2 = SC * d2i[u];
          }
          E::enc_s(x2, op);
          double x2m = E::dec_s(op);
          if (diag) {
            g.s2[i] = INV * (x2 - x2m);
            x2m = x2;
          }
          prod = x2m * Dm;
          diff = x2m - Dm;
        } else {
          T xp[NP];
#pragma unroll
          for (int p = 0; p < NP; ++p) xp[p] = xv[u][p][e];
          const double X2m = E::dec_s(xp);
          // X3 = (X2_enc + diag(s2)) (D_enc + diag(rD))
          const double x3 = pv + X2m * rDj[e] + ri[u] * Dm;
          double dn = a_coef * Dm + b_coef * X2m + e_coef * x3;
          if (diag) {
            const double d = dgi[u], x = a_coef * d + b_coef * d2i[u] + e_coef * d3i[u];
            st_agent(g.dg_new + i, x);   // summed inside this launch
            Dm = SC * d;
            dn = SC * x;
          }
          E::enc_s(dn, op);
          double dnm = E::dec_s(op);
          if (diag) {
            g.rD_new[i] = INV * (dn - dnm);
            dnm = dn;
          }
          prod = dnm * dnm;
          diff = dnm - Dm;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          ov[p][e] = op[p];
          Vt[(p * TE + row) * VP + c4 + e] = op[p];
        }
        if (lower) continue;   // covered by the mirror of (j, i)
        rs += prod;
        if (!diag) {
          colacc[e] += prod;
          tacc += diff * diff;
        } else {
          tacc += 0.5 * diff * diff;
        }
      }
      rowacc[q] = rs;
      if constexpr (!DT) {
#pragma unroll
        for (int p = 0; p < NP; ++p) *(v4t *)(Og + eoff<P>(i, j0 + c4, p, Mp)) = ov[p];
      }
    }
  }
  double *rp = (double *)(smem + F::SUMS);   // [TE] row sums
  double *cp = rp + TE;                      // [4 waves][TE] column sums
  double *tp = cp + 4 * TE;                  // [4 waves]
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double x = TE == 64 ? row_sum(rowacc[q]) : sum8(rowacc[q]);
    if (lane % LR == 0) rp[q * RP + r0] = x;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    double x = colacc[e];
    if (TE == 32) x += dpp_d<0x128>(x);   // row_ror:8
    x = swap32_sum(swap16_sum(x));
    if (lane < LR) cp[wave * TE + c4 + e] = x;
  }
  tacc = wave_sum(tacc);
  if (lane == 0) tp[wave] = tacc;
  __syncthreads();
  // mirrored tile: row j0 + row, columns i0 + c4 .. +3.  A diagonal tile is
  // written whole from here, its lower half from the upper one.
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int row = q * RP + r0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      v4t w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = c4 + e;
        const bool up = DT && row < c;
        w[e] = Vt[(p * TE + (up ? row : c)) * VP + (up ? c : row)];
      }
      *(v4t *)(Og + eoff<P>(j0 + row, i0 + c4, p, Mp)) = w;
    }
  }
  if (tid < TE) {
    constexpr double I2 = INV * INV;
    const double rs = I2 * rp[tid];
    const double cs = I2 * (((cp[tid] + cp[TE + tid]) + cp[2 * TE + tid]) + cp[3 * TE + tid]);
    if constexpr (!DT) {
      st_agent(g.part + (int64_t)tj * Mp + i0 + tid, rs);
      st_agent(g.part + (int64_t)ti * Mp + j0 + tid, cs);
    } else {
      st_agent(g.part + (int64_t)ti * Mp + i0 + tid, rs + cs);
    }
    // every off-diagonal element counts twice
    if (tid == 0) st_agent(g.tpart + lin, (2.0 * I2) * (((tp[0] + tp[1]) + tp[2]) + tp[3]));
  }
}

template <int P, int TE, class V>
__device__ __forceinline__ void finish_any(const GemmArgs &g, int ti, int tj, int lin, V &&vload,
                                           char *smem) {
  if (g.mode == 0) {
    if (ti != tj) finish_tile<P, TE, 0, false>(g, ti, tj, lin, vload, smem);
    else finish_tile<P, TE, 0, true>(g, ti, tj, lin, vload, smem);
  } else {
    if (ti != tj) finish_tile<P, TE, 1, false>(g, ti, tj, lin, vload, smem);
    else finish_tile<P, TE, 1, true>(g, ti, tj, lin, vload, smem);
  }
  finish_rows<TE>(g.red, ti, tj, (int)(g.Mp / TE), (double *)smem);
}

// ---------------------------------------------------- tile product kernel
// One 64 x 64 upper tile per block, with its epilogue and the reduction that
// follows the product.  Blocks [0, nfull) compute whole tiles; each remaining
// tile is split along K over nsplit blocks, which publish their partial
// tiles, and the last of them to finish adds all of them in FP64, in split
// order (the sum does not depend on the order of arrival), and runs the
// epilogue.
//
// Small tiles keep several blocks on a CU, so that the epilogue of one runs
// under the products of the others, and fill the chip at small M.  Per
// product, against 128 x 128 tiles of one block's 64 x 64 waves (16-bit:
// pairs) followed by a reduction launch, in us: FP64 M = 2048 310 -> 152,
// M = 4096 1360 -> 997; FP32 M = 4096 670 -> 575; FP16X3 M = 1000 80 -> 28,
// M = 2048 145 -> 50.
template <int P> struct TileKernel {
  using C = TileCfg<P>;
  static constexpr int VS = T64 * VP * (int)sizeof(typename C::S);
  static constexpr int MM = C::SMEM > VS ? C::SMEM : VS;
  static constexpr int SMEM = FinCfg<P, T64>::SMEM > MM ? FinCfg<P, T64>::SMEM : MM;
  // per CU; at four, FP64 has 128 registers and its epilogue spills 26
  static constexpr int BLOCKS = C::KIND == 0 ? 4 : C::KIND == 1 ? 2 : 3;
};

template <int P>
__global__ __launch_bounds__(NTH, (TileKernel<P>::BLOCKS)) void k_tile(GemmArgs g) {
  using C = TileCfg<P>;
  using S = typename C::S;
  __shared__ __attribute__((aligned(16))) char smem[TileKernel<P>::SMEM];
  if (g.status && *g.status != 0) return;   // the solve has stopped

  const int nk_all = (int)(g.Mp / C::KT), nt = (int)(g.Mp / T64);
  int ti, tj, lin, split = -1, kb = 0, ke = nk_all;
  const int u = (int)blockIdx.x - g.nfull, ntail = ((int)gridDim.x - g.nfull) / g.nsplit;
  if (u < 0) {
    tile_of_block(blockIdx.x, g.nfull, nt, ti, tj, lin);
  } else {
    // split-major: the blocks in flight together cover the same K range of
    // consecutive tiles
    split = u / ntail;
    lin = g.nfull + u % ntail;
    tile_of_index(lin, nt, ti, tj);
    kb = (int)((int64_t)split * nk_all / g.nsplit);
    ke = (int)((int64_t)(split + 1) * nk_all / g.nsplit);
  }
  tile_product<P>(g.A, g.B, (int64_t)ti * T64, (int64_t)tj * T64, g.Mp, smem, g.fold, kb, ke);
  const int tid = threadIdx.x, c4 = (tid & 15) * 4, r0 = tid >> 4;
  const S *V = (const S *)smem + r0 * VP + c4;
  const int64_t ps = (int64_t)ntail * (T64 * T64);
  const S *w0 = (const S *)g.ws + (int64_t)(lin - g.nfull) * (T64 * T64) + r0 * T64 + c4;
  if (split >= 0 &&
      !publish_split(V, (S *)w0 + split * ps, g.cnt + (lin - g.nfull), g.nsplit, smem))
    return;
  constexpr int QC = FinCfg<P, T64>::QC;
  finish_any<P, T64>(g, ti, tj, lin, [&](int q0, double (&v)[QC][4]) {
    if (split >= 0) {
      add_partials(w0 + q0 * 16 * T64, ps, g.nsplit, v);
      return;
    }
#pragma unroll
    for (int u = 0; u < QC; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[u][e] = (double)V[(q0 + u) * 16 * VP + e];
    // FP64 / FP32 results replace the products element by element; 16-bit
    // ones lie elsewhere in the same LDS, so all products are read first
    if constexpr (C::ES == 2) {
      static_assert(QC == 4, "all rows at once");
      __syncthreads();
    }
  }, smem);
}

// One 32 x 32 upper tile per block (small_product), for products whose 64 x
// 64 tiles would leave most CUs idle behind the K loops of few blocks: at
// M = 256 the ten 64 x 64 tiles of an FP64 product spend 10 of their 19 us
// there; with 36 tiles, each on four independent waves, the product takes 14
// us instead of 23.
template <int P, int NB>
__global__ __launch_bounds__(NTH) void k_small(GemmArgs g) {
  constexpr int TE = 32;
  __shared__ __attribute__((aligned(16))) char smem[SmallCfg<P, NB>::SMEM];
  static_assert(SmallCfg<P, NB>::SMEM >= FinCfg<P, TE>::SMEM, "the epilogue fits");
  if (g.status && *g.status != 0) return;   // the solve has stopped
  int ti, tj, lin;
  tile_of_block(blockIdx.x, (int)gridDim.x, (int)(g.Mp / TE), ti, tj, lin);
  double x[4];
  small_product<P, NB>(g.A, g.B, (int64_t)ti * TE, (int64_t)tj * TE, g.Mp, smem, g.fold, x);
  finish_any<P, TE>(g, ti, tj, lin, [&](int, double (&v)[1][4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[0][e] = x[e];
  }, smem);
}

// ------------------------------------------------ 16-bit product kernel
// Pairs of horizontally adjacent 128 x 128 tiles, (ti, 2c) and (ti, 2c+1),
// share one row panel of the left operand: a 128 x 256 output per block of
// 8 waves (2 per SIMD), each wave 64 rows x 64 columns of one tile (4 x 4
// MFMA blocks).  The panels stream through a 3-stage LDS ring (2 stages for
// three planes), one K stage of 32 per step.  All split products of a K step
// go into one FP32 chunk accumulator, which is added into a running FP32
// total every `fold` K steps.  With r products per step and n = K/32 steps
// the rounding error then grows like sqrt(r*fold + n/fold) instead of
// sqrt(r*n): fold = sqrt(n/r) (the default) minimises it.  This accumulation
// error, not the operand encoding, bounds the accuracy of the split
// encodings at large M.  A pair may be split along K over several blocks
// (the pairs of a last partial round, or every pair with the ksplit option):
// each split folds its own K range, and the last to finish adds the splits'
// FP32 totals in FP64, in split order.
constexpr int PAIR_COLS = 2;

// Pair (ti, c) of block b, c >= ti/2, in column-major order of the pair
// triangle: consecutive blocks share the column pair (the 256-row B panel)
// and walk down the row panels.  Blocks go round-robin to the 8 XCDs, so at
// any time all XCDs stream the same B panel (served once from the Infinity
// Cache) while each keeps a few A panels in flight.  Measured on the load
// path alone, this order moves 1.3x the data per unit time of an 8 x 8
// grouped order with per-XCD contiguous ranges.
__device__ __forceinline__ void pair_of_block(int b, int nt, int &ti, int &cp, int &lin) {
  const int npc = nt / PAIR_COLS;
  int L = b;
  lin = b;
  for (int c = 0; c < npc; ++c) {
    const int len = min(nt, PAIR_COLS * c + PAIR_COLS);   // rows ti <= 2c + 1
    if (L < len) {
      ti = L;
      cp = c;
      return;
    }
    L -= len;
  }
  ti = cp = 0;
}

constexpr int NW16 = 8;              // waves per block of the 16-bit kernel (2 per SIMD)
constexpr int NTH16 = 64 * NW16;

// Eight waves of 64 x 64 with 16x16x32 products (any plane count; the
// three-plane BF16X6 uses 64-byte plane segments per stage).
template <int P>
__global__ __launch_bounds__(NTH16, 1) void k_gemm16(GemmArgs g) {
  using E = Enc<P>;
  using T = uint16_t;
  constexpr int NP = E::NP, KIND = E::KIND;
  constexpr int KT = 32;                         // K per stage: one MFMA step
  constexpr int AR = TILE, BR = PAIR_COLS * TILE;
  constexpr int WCOLS = BR / (NW16 / 2);         // columns per wave (64)
  constexpr int NBJ = WCOLS / 16;                // MFMA blocks per wave row (4)
  // One- and two-plane encodings: a stage is one 128-byte segment of every
  // panel row (64 halves: 64 K values of one plane, or 32 K values of both
  // planes, which the interleaved storage keeps together).  Three-plane
  // encodings: 64-byte segments of each plane (32 K values).
  constexpr bool R128 = NP <= 2;
  constexpr int RH = R128 ? 64 : NP * KT;        // halves per panel row per stage
  constexpr int STAGE = (AR + BR) * RH;          // halves per stage
  // ring of NBUF stages, NBUF - 1 of them in flight while one is consumed
  constexpr int NBUF_FIT = (150 * 1024) / (STAGE * 2);
  constexpr int NBUF = NBUF_FIT > 4 ? 4 : (NBUF_FIT < 2 ? 2 : NBUF_FIT);
  constexpr int PD = NBUF - 1;                   // prefetch distance (stages)
  constexpr int ROWS_PER_LOAD = R128 ? 8 : 16;   // rows filled by one wave instruction
  constexpr int BLK = (R128 ? 1 : NP) * (AR + BR) / ROWS_PER_LOAD;
  static_assert(BLK % NW16 == 0, "whole blocks per wave");
  constexpr int LPS = BLK / NW16;                // loads per stage per wave
  // s_waitcnt immediate: vmcnt <= n, expcnt/lgkmcnt not waited on
  constexpr int WAIT_STEADY = ((PD - 1) * LPS & 0xF) | ((((PD - 1) * LPS) >> 4) << 14) | (0x7 << 4) | (0xF << 8);
  static_assert((PD - 1) * LPS <= 63, "vmcnt range");
  constexpr int EPLD = TILE + 4;                 // epilogue row pitch (floats)
  constexpr int WPT = NW16 / 2;                  // waves per tile in the epilogue
  constexpr int EVEC = 5 * TILE + BR;            // FP64 side vectors staged for the epilogue
  constexpr int EPI =
      (2 * TILE * EPLD * 4 + (2 + 2 * WPT) * TILE * 8 + 2 * WPT * 8 + EVEC * 8) / 2;   // halves
  constexpr int SMEM = NBUF * STAGE > EPI ? NBUF * STAGE : EPI;
  __shared__ __attribute__((aligned(16))) T smem[SMEM];
  if (g.status && *g.status != 0) return;   // the solve has stopped

  // whole pair, or split s of a tail pair over K stages [kbase, kbase + nk)
  const int nk_all = (int)(R128 ? g.Mp * NP / 64 : g.Mp / KT);
  int ti, cpair, lin, split = -1, kbase = 0, nk = nk_all;
  if ((int)blockIdx.x < g.nfull) {
    pair_of_block(blockIdx.x, g.nt, ti, cpair, lin);
  } else {
    const int u = (int)blockIdx.x - g.nfull;
    // split-major: the blocks in flight together work on the same K range
    // of consecutive pairs, which share their panels as whole pairs do
    const int ntail = ((int)gridDim.x - g.nfull) / g.nsplit;
    split = u / ntail;
    pair_of_block(g.nfull + u % ntail, g.nt, ti, cpair, lin);
    kbase = split * nk_all / g.nsplit;
    nk = (split + 1) * nk_all / g.nsplit - kbase;
  }
  const int64_t Mp = g.Mp;
  const int64_t arow0 = (int64_t)ti * TILE, brow0 = (int64_t)cpair * BR;
  const T *__restrict__ Ag = (const T *)g.A;
  const T *__restrict__ Bg = (const T *)g.B;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  // wave (rh, wc): rows rh*64 .. +63 of the panel, pair columns wc*64 .. +63
  const int rh = wave & 1, wc = wave >> 1;
  const int h = (wc * WCOLS) / TILE;             // which tile of the pair
  const int tcol0 = wc * WCOLS - h * TILE;       // first column inside that tile
  const int tj = cpair * PAIR_COLS + h;
  const bool valid = tj >= ti;

  // 128-byte rows: the 8 chunks of stage row R sit at slots c ^ (R % 8), so
  // the 16 rows an MFMA fragment read touches cover every slot twice, with
  // the two rows of a slot of opposite parity.  Measured on gfx950 with the
  // fragment pattern alone: no LDS bank conflicts (SQ_LDS_BANK_CONFLICT = 0)
  // and 176 B/clk per CU, against 2-way conflicts and 117 B/clk for the slot
  // c ^ ((R ^ (R >> 3)) % 8).  64-byte rows (three planes): 4 chunks at slots
  // c ^ ((R >> 1) ^ (R >> 3)) % 4.  Global data goes straight to LDS
  // (global_load_lds, 16 B per lane; one wave instruction fills 8 or 16
  // contiguous rows).
  auto swz = [](int R) { return R128 ? (R & 7) : (((R >> 1) ^ (R >> 3)) & 3); };
  auto issue = [&](int kt, int buf) {
    T *st = smem + buf * STAGE;
#pragma unroll
    for (int q = 0; q < LPS; ++q) {
      const int blk = wave + NW16 * q;
      if constexpr (R128) {
        const int R = blk * 8 + (lane >> 3);
        const int c = (lane & 7) ^ swz(R);
        const T *src = (R < AR ? Ag + (arow0 + R) * (NP * Mp) : Bg + (brow0 + R - AR) * (NP * Mp)) +
                       (int64_t)(kbase + kt) * 64 + c * 8;
        __builtin_amdgcn_global_load_lds((const void *)src, (lds_void *)(st + blk * 8 * 64), 16, 0, 0);
      } else {
        const int p = blk / ((AR + BR) / 16), gq = blk % ((AR + BR) / 16);
        const int R = gq * 16 + (lane >> 2);
        const int c = (lane & 3) ^ swz(R);
        const T *src = (R < AR ? Ag + (arow0 + R) * (NP * Mp) : Bg + (brow0 + R - AR) * (NP * Mp)) +
                       (int64_t)(kbase + kt) * (NP * KT) + p * KT + c * 8;
        __builtin_amdgcn_global_load_lds((const void *)src,
                                         (lds_void *)(st + (p * (AR + BR) + gq * 16) * KT), 16, 0, 0);
      }
    }
  };
  // fragment x (chunk group) of stage row R: 128-byte rows hold two groups
  // of 4 chunks (two planes, or two K halves of one plane)
  auto frag = [&](const T *st, int R, int x) -> v4u {
    if constexpr (R128)
      return *(const v4u *)(st + R * 64 + ((x * 4 + lg) ^ swz(R)) * 8);
    else
      return *(const v4u *)(st + (x * (AR + BR) + R) * KT + (lg ^ swz(R)) * 8);
  };
  constexpr int NX = R128 ? 2 : NP;              // fragment groups per stage row
  // two wave groups half a stage apart (below); the three-plane encodings
  // keep the plain loop (their fragments would not fit in the registers)
  constexpr bool PING = R128;

  v4f acc[4][NBJ], tot[4][NBJ];
#pragma unroll
  for (int bi = 0; bi < 4; ++bi)
#pragma unroll
    for (int bj = 0; bj < NBJ; ++bj) {
      acc[bi][bj] = v4f{};
      tot[bi][bj] = v4f{};
    }

  // products per stage (group of A, group of B), largest first: split
  // encodings pair the planes; one plane pairs the two K halves
  constexpr int NPR = NP == 1 ? 2 : E::NPROD;
  constexpr int PA[6] = {0, 0, 1, 1, 0, 2};
  constexpr int PB[6] = {0, 1, 0, 1, 2, 0};
  constexpr int QA[2] = {0, 1};

  const int fold = g.fold;   // >= 1 (resolved on the host)
  v4u af[4][NX], bf[NBJ][NX];
  auto read_frags = [&](int kt) {
    const T *st = smem + (kt % NBUF) * STAGE;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int x = 0; x < NX; ++x) af[bi][x] = frag(st, rh * 64 + bi * 16 + l16, x);
#pragma unroll
    for (int bj = 0; bj < NBJ; ++bj)
#pragma unroll
      for (int x = 0; x < NX; ++x) bf[bj][x] = frag(st, AR + wc * WCOLS + bj * 16 + l16, x);
  };
  // the products of stage kt; the chunk accumulator goes into the running
  // total after the last stage of each chunk of `fold` stages
  auto compute = [&](int kt) {
#pragma unroll
    for (int pr = 0; pr < NPR; ++pr)
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int bj = 0; bj < NBJ; ++bj) {
          const int xa = NP == 1 ? QA[pr] : PA[pr], xb = NP == 1 ? QA[pr] : PB[pr];
          acc[bi][bj] = mfma16<KIND>(af[bi][xa], bf[bj][xb], acc[bi][bj]);
        }
    if ((kt + 1) % fold == 0 || kt == nk - 1) {
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int bj = 0; bj < NBJ; ++bj) {
          tot[bi][bj] += acc[bi][bj];
          acc[bi][bj] = v4f{};
        }
    }
  };
  // Bare s_barrier: __syncthreads() would add a workgroup release fence,
  // which waits for every outstanding LDS-DMA load and so drains the
  // pipeline.  The empty asm statements keep the compiler from moving LDS
  // accesses across it, the scheduling barriers keep the matrix products on
  // their side of it; the waits before it provide the hardware ordering.
  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };
  // this wave's loads of stage kt have landed (later stages may still fly)
  // and its fragment reads are complete
  auto wait_stage = [&](int kt) {
    if (kt + PD - 1 < nk)
      __builtin_amdgcn_s_waitcnt(WAIT_STEADY & ~(0xF << 8));
    else
      __builtin_amdgcn_s_waitcnt(0);
  };
  // Waves of a tile below the diagonal run the same instruction stream (their
  // results are discarded).
#pragma unroll
  for (int s0 = 0; s0 < PD; ++s0)
    if (s0 < nk) issue(s0, s0);
  if constexpr (PING) {
    // Two wave groups, waves 0-3 (A) and 4-7 (B), one of each per SIMD, half
    // a stage apart: in the first half of stage kt A reads its fragments of
    // stage kt while B runs its products of stage kt-1; in the second half A
    // runs the products of stage kt while B reads its fragments of it.  Each
    // SIMD's matrix core is fed by one group while the other waits on LDS.
    // Each wave's products and their order are those of the plain loop.
    // A wave whose load cannot issue stalls its whole instruction stream, so
    // each group issues its share of the loads of stage kt+PD (into the
    // buffer freed at the first barrier) in its fragment-read half only.
    const bool grp_b = wave >= NW16 / 2;
    for (int kt = 0; kt <= nk; ++kt) {
      wait_stage(kt);
      barrier();   // stage kt has landed; the buffer of stage kt-1 is free
      if (!grp_b) {
        if (kt + PD < nk) issue(kt + PD, (kt + PD) % NBUF);
        if (kt < nk) read_frags(kt);
      } else if (kt > 0) {
        compute(kt - 1);
      }
      barrier();
      if (kt < nk) {
        if (!grp_b) {
          compute(kt);
        } else {
          if (kt + PD < nk) issue(kt + PD, (kt + PD) % NBUF);
          read_frags(kt);
        }
      }
    }
  } else {
    for (int kt = 0; kt < nk; ++kt) {
      wait_stage(kt);
      barrier();   // ... and everyone's; the buffer of stage kt-1 is free
      if (kt + PD < nk) issue(kt + PD, (kt + PD) % NBUF);
      read_frags(kt);
      compute(kt);
    }
  }
  __syncthreads();   // all waves done with the stage buffers (reused below)

  if (split >= 0) {
    // K-split tail pair: publish this split's FP32 totals; the last split to
    // arrive adds all of them in split order (so the sum does not depend on
    // the arrival order) and runs the epilogue.
    constexpr int NV = 4 * NBJ;   // float4 per thread
    const int pair = lin - g.nfull;  // index among the split pairs
    float4 *wsp = (float4 *)g.ws + ((int64_t)pair * g.nsplit + split) * NV * NTH16;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int bj = 0; bj < NBJ; ++bj) {
        const v4f t = tot[bi][bj];
        wsp[(bi * NBJ + bj) * NTH16 + tid] = make_float4(t[0], t[1], t[2], t[3]);
      }
    __threadfence();
    // The arrival flag lives in the (now idle) stage buffers: a second
    // __shared__ object would make the compiler wait for every LDS-DMA load
    // before each LDS read of the main loop (it cannot tell them apart).
    unsigned *last = (unsigned *)smem;
    __syncthreads();
    if (tid == 0) *last = (atomicAdd(g.cnt + pair, 1u) == (unsigned)g.nsplit - 1);
    __syncthreads();
    if (!*last) return;
    __syncthreads();   // flag read by all before the epilogue reuses smem
    __threadfence();
    const float4 *w0 = (const float4 *)g.ws + (int64_t)pair * g.nsplit * NV * NTH16;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int bj = 0; bj < NBJ; ++bj) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
#pragma unroll 4
        for (int s = 0; s < g.nsplit; ++s) {
          const float4 v = w0[((int64_t)s * NV + bi * NBJ + bj) * NTH16 + tid];
          a0 += v.x;
          a1 += v.y;
          a2 += v.z;
          a3 += v.w;
        }
        tot[bi][bj] = v4f{(float)a0, (float)a1, (float)a2, (float)a3};
      }
    if (tid == 0) g.cnt[pair] = 0u;   // ready for the next launch
  }

  // ------------------------------------------------------------ epilogue
  // Phase 0: every wave dumps its FP32 results into LDS, V[tile][row][col]
  // with a row pitch of 132 floats.
  float *V = (float *)smem;
  double *rp = (double *)(V + 2 * TILE * EPLD);   // [2 tiles][128] row sums
  double *cpart = rp + 2 * TILE;                  // [2 tiles][WPT waves][128] column sums
  double *tp = cpart + 2 * WPT * TILE;            // [2 tiles][WPT waves] tile sums
  // The FP64 side vectors of the block's rows (rD, s2, dg, d2, d3) and
  // columns (rD) are staged in LDS: read per element from global memory they
  // would each wait for the stores before them (the compiler cannot tell
  // them from the output), one memory round trip per element.
  double *vrow = tp + 2 * WPT;                    // [5][128]
  double *vcol = vrow + 5 * TILE;                 // [256]
  for (int q = tid; q < EVEC; q += NTH16) {
    if (q < 5 * TILE) {
      const int k = q / TILE;
      const int64_t i = arow0 + q % TILE;
      double v = 0.0;
      if (k == 0) v = g.rD[i];
      else if (k == 1) v = g.mode == 1 ? g.s2[i] : 0.0;
      else if (k == 2) v = g.dg[i];
      else if (k == 3) v = g.d2[i];
      else v = g.mode == 1 ? g.d3[i] : 0.0;
      vrow[q] = v;
    } else {
      vcol[q - 5 * TILE] = g.rD[brow0 + q - 5 * TILE];
    }
  }
  if (valid) {
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int bj = 0; bj < NBJ; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          V[(h * TILE + rh * 64 + bi * 16 + lg * 4 + r) * EPLD + tcol0 + bj * 16 + l16] =
              tot[bi][bj][r];
  }
  __syncthreads();
  // Phase 1: 256 threads per tile, each owning one 8 x 8 block (block row br,
  // block column bc).  Row-contiguous 16-byte loads of D (and X2) and stores
  // of the result; the mirrored store writes the transposed block, again as
  // 16-byte rows.
  const int th = tid >> 8, x = tid & 255;
  const int tjj = cpair * PAIR_COLS + th;
  const bool tvalid = tjj >= ti, dtile = tjj == ti;
  const int br = x >> 4, bc = x & 15;
  const int64_t i0 = arow0 + br * 8;
  // elements are kept in the stored units SC x (SC a power of two)
  constexpr double SC = E::SC, INV = 1.0 / SC;
  T *__restrict__ Og = (T *)g.out;
  double a_coef = 0.0, b_coef = 0.0, e_coef = 0.0;
  if (g.mode == 1) update_coefs(g.method, g.coef[0], a_coef, b_coef, e_coef);
  double rsum[8], csum[8], tsum = 0.0;
#pragma unroll
  for (int r = 0; r < 8; ++r) rsum[r] = csum[r] = 0.0;
  // The 8 x 8 blocks on a tile's diagonal hold the diagonal elements, formed
  // from the FP64 side vectors, and are their own mirrors.  DK = 1 compiles
  // such a block, DK = 0 every other block (the lean path), DK = 2 decides at
  // run time.  Both update modes are compiled separately.
  auto element_block = [&](auto dk_t, auto mode_t) {
    constexpr int DK = decltype(dk_t)::value;
    constexpr int MODE = decltype(mode_t)::value;
    const bool dblk = DK == 1 || (DK == 2 && dtile && br == bc);
    const int64_t j0 = (int64_t)tjj * TILE + bc * 8;
    // Encoded results, row r of the block, 8 halves per plane, kept for the
    // mirrored store.  Planes p < NPARK are parked in this thread's own 8 x 8
    // block of V (32 bytes per row, already consumed when row r is encoded),
    // which keeps them out of the registers; a third plane stays in them.
    constexpr int NPARK = NP < 2 ? NP : 2;
    v4u ob[NP > NPARK ? NP - NPARK : 1][8];
    uint32_t *park = (uint32_t *)(V + (th * TILE + br * 8) * EPLD + bc * 8);   // row r at park + r * EPLD
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int64_t i = i0 + r;
      v4u dv[NP], xv[NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        dv[p] = *(const v4u *)(Bg + eoff<P>(i, j0, p, Mp));
        if constexpr (MODE == 1) xv[p] = *(const v4u *)(Ag + eoff<P>(i, j0, p, Mp));
      }
      const float *vr = V + (th * TILE + br * 8 + r) * EPLD + bc * 8;
      uint16_t o[NP][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t j = j0 + e;
        T dp[NP], op[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) dp[p] = (uint16_t)(dv[p][e >> 1] >> (16 * (e & 1)));
        const double v = (double)vr[e] * INV;   // SC times the product
        double prod, diff;
        if constexpr (MODE == 0) {
          double Dm, x2;
          if (DK != 0 && i == j) {
            Dm = SC * vrow[2 * TILE + br * 8 + r];
            x2 = SC * vrow[3 * TILE + br * 8 + r];
          } else {
            Dm = E::dec_s(dp);
            x2 = v + Dm * (vrow[br * 8 + r] + vcol[th * TILE + bc * 8 + e]);
          }
          E::enc_s(x2, op);
          const double x2m = (DK != 0 && i == j) ? x2 : E::dec_s(op);
          if (DK != 0 && i == j) g.s2[i] = INV * (x2 - E::dec_s(op));
          prod = x2m * Dm;
          diff = x2m - Dm;
        } else {
          double Dm, dn, dx = 0.0;
          if (DK != 0 && i == j) {
            const double d = vrow[2 * TILE + br * 8 + r];
            dx = a_coef * d + b_coef * vrow[3 * TILE + br * 8 + r] + e_coef * vrow[4 * TILE + br * 8 + r];
            Dm = SC * d;
            dn = SC * dx;
          } else {
            T xp[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) xp[p] = (uint16_t)(xv[p][e >> 1] >> (16 * (e & 1)));
            Dm = E::dec_s(dp);
            const double X2m = E::dec_s(xp);
            const double x3 = v + X2m * vcol[th * TILE + bc * 8 + e] + vrow[TILE + br * 8 + r] * Dm;
            dn = a_coef * Dm + b_coef * X2m + e_coef * x3;
          }
          E::enc_s(dn, op);
          const double dnm = (DK != 0 && i == j) ? dn : E::dec_s(op);
          if (DK != 0 && i == j) {
            g.dg_new[i] = dx;
            g.rD_new[i] = INV * (dn - E::dec_s(op));
          }
          prod = dnm * dnm;
          diff = dnm - Dm;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) o[p][e] = op[p];
        if (dblk && i > j) continue;   // lower half of a diagonal block
        rsum[r] += prod;
        if (DK == 0 || i != j) {
          csum[e] += prod;
          tsum += diff * diff;
        } else {
          tsum += 0.5 * diff * diff;   // off-diagonal elements count twice, below
        }
      }
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        v4u w;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = (uint32_t)o[p][2 * q] | ((uint32_t)o[p][2 * q + 1] << 16);
        if (p < NPARK)
          *(v4u *)(park + r * EPLD + 4 * p) = w;
        else
          ob[p - NPARK][r] = w;
        if (!dblk) {
          *(v4u *)(Og + eoff<P>(i, j0, p, Mp)) = w;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (e >= r) Og[eoff<P>(i, j0 + e, p, Mp)] = o[p][e];
        }
      }
    }
    // mirrored (transposed) block: row j0+e gets column e of the block
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      v4u obp[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (p < NPARK)
          obp[r] = *(const v4u *)(park + r * EPLD + 4 * p);
        else
          obp[r] = ob[p - NPARK][r];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (!dblk) {
          v4u w;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t lo = (obp[2 * q][e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
            const uint32_t hi = (obp[2 * q + 1][e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
            w[q] = lo | (hi << 16);
          }
          *(v4u *)(Og + eoff<P>(j0 + e, i0, p, Mp)) = w;
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r)
            if (r < e)
              Og[eoff<P>(j0 + e, i0 + r, p, Mp)] =
                  (uint16_t)((obp[r][e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
        }
      }
    }
  };
  if (tvalid && !(dtile && br > bc)) {   // blocks below the diagonal are mirrors
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    // (three planes: one body for both kinds of block; the split one measured
    // slower there, its main loop scheduled worse)
    if constexpr (NP == 3) {
      if (g.mode == 0) element_block(I2{}, I0{});
      else element_block(I2{}, I1{});
    } else if (dtile && br == bc) {
      if (g.mode == 0) element_block(I1{}, I0{});
      else element_block(I1{}, I1{});
    } else {
      if (g.mode == 0) element_block(I0{}, I0{});
      else element_block(I0{}, I1{});
    }
  }
  // row sums: the 16 threads of a block row (lanes differing in bits 0..3)
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    rsum[r] = row_sum(rsum[r]);
  }
  // column sums: the 4 block rows of a wave (bits 4..5), then the tile's waves
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    csum[e] = swap32_sum(swap16_sum(csum[e]));
  }
  tsum = wave_sum(tsum);
  const int wt = x >> 6;   // wave within the tile
  if ((x & 15) == 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) rp[th * TILE + br * 8 + r] = rsum[r];
  }
  if (lg == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) cpart[(th * WPT + wt) * TILE + bc * 8 + e] = csum[e];
  }
  if (lane == 0) tp[th * WPT + wt] = tsum;
  __syncthreads();
  if (x < TILE && tvalid) {
    const double rs = INV * INV * rp[th * TILE + x];
    double cs = 0.0;
#pragma unroll
    for (int w = 0; w < WPT; ++w) cs += cpart[(th * WPT + w) * TILE + x];
    cs *= INV * INV;
    if (!dtile) {
      g.part[(int64_t)tjj * Mp + arow0 + x] = rs;
      g.part[(int64_t)ti * Mp + (int64_t)tjj * TILE + x] = cs;
    } else {
      g.part[(int64_t)ti * Mp + arow0 + x] = rs + cs;
    }
  }
  if (tid < 2) {   // 0 for a skipped tile
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < WPT; ++w) t += tp[tid * WPT + w];
    g.tpart[2 * lin + tid] = 2.0 * INV * INV * t;
  }
}

int pair_count(int nt) {
  int n = 0;
  for (int t = 0; t < nt; ++t) n += nt / PAIR_COLS - t / PAIR_COLS;
  return n;
}

int gemm16_blocks(const GemmArgs &g) {
  const int np = pair_count(g.nt);
  return g.nfull + (np - g.nfull) * g.nsplit;
}

// ------------------------------------------------------------------ H stats
// Per row: H_ii and the Gershgorin radius r_i = sum_{j != i} |H_ij|.
__global__ __launch_bounds__(256) void k_hstats(const double *__restrict__ H, int64_t ldh,
                                                int64_t M, double *lo, double *hi,
                                                double *hd) {
  __shared__ double red[256];
  const int64_t i = blockIdx.x;
  double s = 0.0;
  for (int64_t j = threadIdx.x; j < M; j += 256)
    if (j != i) s += fabs(H[i * ldh + j]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double d = H[i * ldh + i];
    lo[i] = d - red[0];
    hi[i] = d + red[0];
    hd[i] = d;
  }
}

// Single block: min of lo, max of hi and the (fixed-order) sum of hd.
__global__ __launch_bounds__(256) void k_hfinal(const double *lo, const double *hi,
                                                const double *hd, int64_t M, double *out,
                                                Scalars *post, uint32_t seq) {
  __shared__ double smin[256], smax[256], ssum[256];
  double mn = INFINITY, mx = -INFINITY, sm = 0.0;
  for (int64_t i = threadIdx.x; i < M; i += 256) {
    mn = fmin(mn, lo[i]);
    mx = fmax(mx, hi[i]);
    sm += hd[i];
  }
  smin[threadIdx.x] = mn;
  smax[threadIdx.x] = mx;
  ssum[threadIdx.x] = sm;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + w]);
      smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + w]);
      ssum[threadIdx.x] += ssum[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = smin[0];
    out[1] = smax[0];
    out[2] = ssum[0];
    if (post) {
      st_host(&post->hstat[0], smin[0]);
      st_host(&post->hstat[1], smax[0]);
      st_host(&post->hstat[2], ssum[0]);
      host_order();
      st_host(&post->seq, seq);
    }
  }
}

// ||(H + H^T)/2 - mu I||_F^2 (the alpha search of the hole-particle guess):
// one partial per mirrored pair of 64 x 64 tiles, then a fixed-order sum.
// M = 1500: 35 -> 7 us against uncoalesced reads of every tile and its mirror.
__global__ __launch_bounds__(256) void k_hdev(const double *__restrict__ H, int64_t ldh, int64_t M,
                                              double mu, double *part) {
  __shared__ double ta[64][65], tb[64][65], red[4];
  double ha[16], hb[16];
  const SymPair p = sym_pair(
      blockIdx.x, M, [&](int64_t r, int64_t c) { return H[r * ldh + c]; }, ha, hb, ta, tb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + wave;
    const int64_t i = p.I + r, j = p.J + lane;
    if (i < M && j < M) {
      const double x = 0.5 * (ha[q] + tb[lane][r]) - (i == j ? mu : 0.0);
      s += x * x;
    }
  }
  s = wave_sum(p.diag ? s : 2.0 * s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ __launch_bounds__(256) void k_hdev_sum(const double *part, int n, double *out,
                                                  Scalars *post, uint32_t seq) {
  __shared__ double red[256];
  double s = 0.0;
  for (int t = threadIdx.x; t < n; t += 256) s += part[t];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *out = red[0];
    if (post) {
      st_host(&post->hstat[3], red[0]);
      host_order();
      st_host(&post->seq, seq);
    }
  }
}

// ------------------------------------------------------------ initial guess
// D0 = theta I + beta (mu I - (H + H^T)/2) over 64 x 64 tiles of the padded
// matrix; writes the operand planes, the FP64 diagonal (dg, rD) and row sums
// of D0 o D0 into part[tile column][row] (the diagonal of D0^2).  One block
// per mirrored tile pair (I, J), (J, I) with I <= J: each tile of H is read
// once, and (H_ij + H_ji)/2 is the same sum in both output tiles, so D0 is
// exactly symmetric.

// Output tile (I, J) of the pair: hv[q] = H[I + r][J + lane] from the
// block's own load (r = 4q + wave), tr[c][r] = H[J + c][I + r] from LDS.
template <int P>
__device__ __forceinline__ void init_tile(const InitArgs &a, int64_t I, int64_t J,
                                          const double (&hv)[16],
                                          const double (*tr)[65], int wave, int lane) {
  using E = Enc<P>;
  using T = typename E::T;
  constexpr int NP = E::NP;
  T *__restrict__ Og = (T *)a.out;
#pragma unroll 2
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + wave;
    const int64_t i = I + r, j = J + lane;
    double x = 0.0;
    if (i < a.M && j < a.M) {
      const double h = 0.5 * (hv[q] + tr[lane][r]);
      x = -a.beta * h;
      if (i == j) x += a.theta + a.beta * a.mu;
    }
    T op[NP];
    E::enc(x, op);
#pragma unroll
    for (int p = 0; p < NP; ++p) Og[eoff<P>(i, j, p, a.Mp)] = op[p];
    const double xm = (i == j) ? x : E::dec(op);
    if (i == j) {
      a.dg[i] = x;
      a.rD[i] = x - E::dec(op);
    }
    // row sum of D0 o D0 over the tile's 64 columns (fixed order)
    const double rs = wave_sum(xm * xm);
    if (lane == 0) a.part[(J >> 6) * a.Mp + i] = rs;
  }
}

template <int P>
__global__ __launch_bounds__(256) void k_init(InitArgs a) {
  __shared__ double ta[64][65], tb[64][65];
  double ha[16], hb[16];
  const SymPair p = sym_pair(
      blockIdx.x, a.M, [&](int64_t r, int64_t c) { return a.H[r * a.ldh + c]; }, ha, hb, ta, tb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  init_tile<P>(a, p.I, p.J, ha, tb, wave, lane);
  if (!p.diag) init_tile<P>(a, p.J, p.I, hb, ta, wave, lane);
}

// -------------------------------------------------------------- reductions
// out[i] = sum_s part[s][i]: a block covers 64 rows, wave q of it sums the
// slots s = q (mod 4) in ascending order, and the four wave sums are added in
// wave order.  Per-block sums of out and of extra; the last block to finish
// adds the block sums and the tile partials in a fixed order and runs the
// scalar step for this point of the iteration.
__global__ __launch_bounds__(256) void k_reduce(RedArgs a) {
  __shared__ double rq[4][64], s1[256], s2[256], s3[256];
  __shared__ int is_last;
  // a batch enqueued ahead of the host's check: nothing to do once stopped
  // (the status is written by the last block of a mode-1 launch, after
  // every block of that launch has read it here)
  if (a.skip_if_stopped && a.sc->status != 0) return;
  const int tid = threadIdx.x, lane = tid & 63, q = tid >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  double w = 0.0;
  if (i < a.Mp) {
    // unrolled so that the loads are in flight together; the adds keep
    // their order
#pragma unroll 8
    for (int s = q; s < a.nslots; s += 4) w += a.part[(int64_t)s * a.Mp + i];
  }
  rq[q][lane] = w;
  __syncthreads();
  double v = 0.0, e = 0.0;
  if (q == 0 && i < a.Mp) {
    v = ((rq[0][lane] + rq[1][lane]) + rq[2][lane]) + rq[3][lane];
    a.out[i] = v;
    if (a.extra) e = a.extra[i];
  }
  s1[tid] = v;
  s2[tid] = e;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) {
      s1[tid] += s1[tid + w];
      s2[tid] += s2[tid + w];
    }
    __syncthreads();
  }
  if (tid == 0) {
    a.bpart[2 * blockIdx.x] = s1[0];
    a.bpart[2 * blockIdx.x + 1] = s2[0];
    __threadfence();
    const unsigned ticket = atomicAdd(a.counter, 1u);
    is_last = (ticket == gridDim.x - 1);
  }
  __syncthreads();
  if (!is_last) return;
  __threadfence();
  double b1 = 0.0, b2 = 0.0, b3 = 0.0;
  for (int b = tid; b < (int)gridDim.x; b += 256) {
    b1 += ld_agent(a.bpart + 2 * b);
    b2 += ld_agent(a.bpart + 2 * b + 1);
  }
  if (a.tpart)
    for (int t = tid; t < a.ntiles; t += 256) b3 += a.tpart[t];
  s1[tid] = b1;
  s2[tid] = b2;
  s3[tid] = b3;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) {
      s1[tid] += s1[tid + w];
      s2[tid] += s2[tid + w];
      s3[tid] += s3[tid + w];
    }
    __syncthreads();
  }
  if (tid != 0) return;
  *a.counter = 0u;
  scalar_step(a, s1[0], s2[0], s3[0]);
}

// ------------------------------------------------------------------ output
template <int P>
__global__ __launch_bounds__(256) void k_output(OutArgs a) {
  using E = Enc<P>;
  using T = typename E::T;
  constexpr int NP = E::NP;
  // rows on the x dimension of the grid (no 64K limit), 256 columns per block on y
  const int64_t i = blockIdx.x;
  const int64_t j = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (i >= a.M || j >= a.M) return;
  double x;
  if (i == j) {
    x = a.dg[i];
  } else {
    T p[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) p[q] = ((const T *)a.planes)[eoff<P>(i, j, q, a.Mp)];
    x = E::dec(p);
  }
  if (a.hole) x = (i == j ? 1.0 : 0.0) - x;
  if (a.dtype == GCP_DTYPE_F64)
    ((double *)a.D)[i * a.ldd + j] = x;
  else
    ((float *)a.D)[i * a.ldd + j] = (float)x;
}

// -------------------------------------------------- encoding conversion
// Re-encodes an iterate from encoding PA to PB (precision schedule): the
// off-diagonal master values dec_A(planes) are encoded in B; the diagonal
// is the exact FP64 vector diag, encoded in B with its residual
// diag - dec_B(enc_B(diag)) written to resid.
template <int P>
__device__ __forceinline__ double dec_at(const void *b, int64_t i, int64_t j, int64_t Mp) {
  using E = Enc<P>;
  typename E::T p[E::NP];
#pragma unroll
  for (int q = 0; q < E::NP; ++q) p[q] = ((const typename E::T *)b)[eoff<P>(i, j, q, Mp)];
  return E::dec(p);
}
template <int P>
__device__ __forceinline__ double enc_at(void *b, int64_t i, int64_t j, int64_t Mp, double x) {
  using E = Enc<P>;
  typename E::T p[E::NP];
  E::enc(x, p);
#pragma unroll
  for (int q = 0; q < E::NP; ++q) ((typename E::T *)b)[eoff<P>(i, j, q, Mp)] = p[q];
  return E::dec(p);
}

__device__ __forceinline__ double enc_any(int pb, void *out, int64_t i, int64_t j, int64_t Mp,
                                            double x) {
  switch (pb) {
    case GCP_FP64: return enc_at<GCP_FP64>(out, i, j, Mp, x);
    case GCP_FP32: return enc_at<GCP_FP32>(out, i, j, Mp, x);
    case GCP_BF16: return enc_at<GCP_BF16>(out, i, j, Mp, x);
    case GCP_FP16: return enc_at<GCP_FP16>(out, i, j, Mp, x);
    case GCP_BF16X3: return enc_at<GCP_BF16X3>(out, i, j, Mp, x);
    case GCP_FP16X3: return enc_at<GCP_FP16X3>(out, i, j, Mp, x);
    default: return enc_at<GCP_BF16X6>(out, i, j, Mp, x);
  }
}

template <int PA>
__global__ __launch_bounds__(256) void k_convert(int pb, const void *in, const double *diag, void *out,
                                                 double *resid, int64_t Mp) {
  // rows on the x dimension of the grid (no 64K limit), 256 columns per block on y
  const int64_t i = blockIdx.x;
  const int64_t j = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (j >= Mp) return;
  const double x = (i == j) ? diag[i] : dec_at<PA>(in, i, j, Mp);
  const double xe = enc_any(pb, out, i, j, Mp, x);
  if (i == j) resid[i] = x - xe;
}

hipError_t launch_convert(int pa, int pb, const void *in, const double *diag, void *out,
                          double *resid, int64_t Mp, hipStream_t st) {
  const dim3 grid((unsigned)Mp, (unsigned)((Mp + 255) / 256));
  switch (pa) {
    case GCP_FP64: k_convert<GCP_FP64><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    case GCP_FP32: k_convert<GCP_FP32><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    case GCP_BF16: k_convert<GCP_BF16><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    case GCP_FP16: k_convert<GCP_FP16><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    case GCP_BF16X3: k_convert<GCP_BF16X3><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    case GCP_FP16X3: k_convert<GCP_FP16X3><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    case GCP_BF16X6: k_convert<GCP_BF16X6><<<grid, 256, 0, st>>>(pb, in, diag, out, resid, Mp); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- dispatch
template <int P>
static hipError_t launch_gemm_p(const GemmArgs &g, hipStream_t st) {
  if (g.path == PATH_T32) {
    const int nt = (int)(g.Mp / 32);
    const unsigned n = (unsigned)(nt * (nt + 1) / 2);
    // deep rings (one block per CU) while there is one tile per CU
    if ((int)n <= g.cus) k_small<P, Enc<P>::NP == 3 ? 3 : 4><<<n, NTH, 0, st>>>(g);
    else k_small<P, 2><<<n, NTH, 0, st>>>(g);
    return hipGetLastError();
  }
  const int nt = (int)(g.Mp / T64), ntail = nt * (nt + 1) / 2 - g.nfull;
  if constexpr (Enc<P>::KIND >= 2) {
    if (g.path == PATH_PAIR) {
      k_gemm16<P><<<gemm16_blocks(g), NTH16, 0, st>>>(g);
      return hipGetLastError();
    }
  }
  k_tile<P><<<g.nfull + ntail * g.nsplit, NTH, 0, st>>>(g);
  return hipGetLastError();
}

hipError_t launch_gemm(int prec, const GemmArgs &g, hipStream_t st) {
  switch (prec) {
    case GCP_FP64: return launch_gemm_p<GCP_FP64>(g, st);
    case GCP_FP32: return launch_gemm_p<GCP_FP32>(g, st);
    case GCP_BF16: return launch_gemm_p<GCP_BF16>(g, st);
    case GCP_FP16: return launch_gemm_p<GCP_FP16>(g, st);
    case GCP_BF16X3: return launch_gemm_p<GCP_BF16X3>(g, st);
    case GCP_FP16X3: return launch_gemm_p<GCP_FP16X3>(g, st);
    case GCP_BF16X6: return launch_gemm_p<GCP_BF16X6>(g, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_init(int prec, const InitArgs &a, hipStream_t st) {
  const int64_t nt = a.Mp / 64;
  const dim3 grid((unsigned)(nt * (nt + 1) / 2));
  switch (prec) {
    case GCP_FP64: k_init<GCP_FP64><<<grid, 256, 0, st>>>(a); break;
    case GCP_FP32: k_init<GCP_FP32><<<grid, 256, 0, st>>>(a); break;
    case GCP_BF16: k_init<GCP_BF16><<<grid, 256, 0, st>>>(a); break;
    case GCP_FP16: k_init<GCP_FP16><<<grid, 256, 0, st>>>(a); break;
    case GCP_BF16X3: k_init<GCP_BF16X3><<<grid, 256, 0, st>>>(a); break;
    case GCP_FP16X3: k_init<GCP_FP16X3><<<grid, 256, 0, st>>>(a); break;
    case GCP_BF16X6: k_init<GCP_BF16X6><<<grid, 256, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_output(int prec, const OutArgs &a, hipStream_t st) {
  const dim3 grid((unsigned)a.M, (unsigned)((a.M + 255) / 256));
  switch (prec) {
    case GCP_FP64: k_output<GCP_FP64><<<grid, 256, 0, st>>>(a); break;
    case GCP_FP32: k_output<GCP_FP32><<<grid, 256, 0, st>>>(a); break;
    case GCP_BF16: k_output<GCP_BF16><<<grid, 256, 0, st>>>(a); break;
    case GCP_FP16: k_output<GCP_FP16><<<grid, 256, 0, st>>>(a); break;
    case GCP_BF16X3: k_output<GCP_BF16X3><<<grid, 256, 0, st>>>(a); break;
    case GCP_FP16X3: k_output<GCP_FP16X3><<<grid, 256, 0, st>>>(a); break;
    case GCP_BF16X6: k_output<GCP_BF16X6><<<grid, 256, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_hstats(const double *H, int64_t ldh, int64_t M, double *lo, double *hi,
                         double *hd, double *out, Scalars *post, uint32_t seq, hipStream_t st) {
  k_hstats<<<(unsigned)M, 256, 0, st>>>(H, ldh, M, lo, hi, hd);
  k_hfinal<<<1, 256, 0, st>>>(lo, hi, hd, M, out, post, seq);
  return hipGetLastError();
}

hipError_t launch_hdev(const double *H, int64_t ldh, int64_t M, int64_t Mp, double mu,
                       double *scratch, double *out, Scalars *post, uint32_t seq,
                       hipStream_t st) {
  const int64_t nt = Mp / 64, np = nt * (nt + 1) / 2;
  k_hdev<<<(unsigned)np, 256, 0, st>>>(H, ldh, M, mu, scratch);
  k_hdev_sum<<<1, 256, 0, st>>>(scratch, (int)np, out, post, seq);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_zero(uint32_t *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    p[i] = 0u;
}

hipError_t launch_zero(void *p, int64_t nwords, hipStream_t st) {
  if (!p || nwords <= 0) return hipSuccess;
  int64_t nb = (nwords + 255) / 256;
  if (nb > 1024) nb = 1024;
  k_zero<<<(unsigned)nb, 256, 0, st>>>((uint32_t *)p, nwords);
  return hipGetLastError();
}

// Traffic yardstick: 64 KiB per block, each wave loading 16 KiB as sixteen
// contiguous wave instructions of 1 KiB (16 bytes per lane) straight into
// LDS, the load type of the 16-bit product kernel's panels.
__global__ __launch_bounds__(256) void k_stream_lds(const uint16_t *buf) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[32768];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint16_t *src = buf + (int64_t)blockIdx.x * 32768 + wave * 8192 + lane * 8;
#pragma unroll
  for (int q = 0; q < 16; ++q)
    __builtin_amdgcn_global_load_lds((const void *)(src + q * 512),
                                     (lds_void *)(lds + wave * 8192 + q * 512), 16, 0, 0);
  __builtin_amdgcn_s_waitcnt(0);
}

hipError_t launch_stream_lds(const void *buf, int64_t bytes, hipStream_t st) {
  k_stream_lds<<<(unsigned)(bytes / 65536), 256, 0, st>>>((const uint16_t *)buf);
  return hipGetLastError();
}

hipError_t launch_reduce(const RedArgs &a, hipStream_t st) {
  k_reduce<<<(unsigned)((a.Mp + 63) / 64), 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace gcp
