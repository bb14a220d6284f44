// gcp_mma.h -- MFMA building blocks shared by the forward and adjoint kernels.
//
// A 64 x 64 output tile of an A * B^T product of row panels (A rows arow0..,
// B rows brow0.., both Mp x Mp row-major, K contiguous) computed by 4 waves
// in 16 x 16 MFMA blocks.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gcp_encode.h"
#include "gcp_kernels.h"

namespace gcp {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int TILE = 128;   // output tile edge of the 16-bit pair kernel
constexpr int T64 = 64;     // edge of the tiles that the epilogues work on
constexpr int NTH = 256;    // threads per tile: 4 waves

template <int KIND> struct AccType { using type = v4f; };
template <> struct AccType<0> { using type = v4d; };

// 16x16 output block per MFMA; lane l holds column l%16 and four rows r = 0..3:
// rows 4*(l/16)+r for the FP32-accumulating instructions, rows (l/16)+4r for
// the FP64 one.  A/B fragments: lane l supplies row l%16 of its operand at K
// offsets determined by l/16 (the same for A and B, so the K order inside an
// instruction never matters).
template <int KIND>
__device__ __forceinline__ int acc_row(int lg, int r) {
  return KIND == 0 ? lg + 4 * r : 4 * lg + r;
}
__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <int KIND>
__device__ __forceinline__ v4f mfma16(v4u a, v4u b, v4f c) {
  if constexpr (KIND == 2)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a),
                                                   __builtin_bit_cast(v8b, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a),
                                                  __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}

// Sums over lanes in a fixed order, by rotations inside the rows of 16 lanes
// (DPP) and swaps of rows and half waves: no LDS round trip per step, as a
// general shuffle takes.  row_sum leaves the sum of its row of 16 lanes in
// every lane, wave_sum that of the wave.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_d<0x128>(v);   // row_ror:8
  v += dpp_d<0x124>(v);
  v += dpp_d<0x122>(v);
  v += dpp_d<0x121>(v);
  return v;
}
// v + v of the lane 16 (32) away, by the row and half-wave swaps.
__device__ __forceinline__ double swap16_sum(double v) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double swap32_sum(double v) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// sum of the aligned group of 8 lanes, in every lane of it
__device__ __forceinline__ double sum8(double v) {
  v += dpp_d<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_d<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_d<0x141>(v);   // row_half_mirror
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
  return swap32_sum(swap16_sum(row_sum(v)));
}

typedef double v2d __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

// A symmetrised matrix (A + A^T)/2 is formed by one block of 256 threads per
// mirrored pair (I, J), (J, I), I <= J, of 64 x 64 tiles: each tile of A is
// read once, a wave taking 64 consecutive elements of a row per load, and the
// transposed operand comes from LDS.  Block L of the nt (nt + 1)/2 pairs.
// ha[q] = A[I + r][J + lane] and hb[q] = A[J + r][I + lane] with r = 4q +
// wave; ta and tb hold the two tiles ([r][lane]).
// ld(r, c) is called with r and c clamped to the M x M matrix and its value
// dropped outside it, so that all 32 loads of a thread are in flight
// together (loads under a condition go out one by one).
struct SymPair {
  int64_t I, J;
  bool diag;
};
template <class LD>
__device__ __forceinline__ SymPair sym_pair(int64_t L, int64_t M, LD &&ld, double (&ha)[16],
                                            double (&hb)[16], double (*ta)[T64 + 1],
                                            double (*tb)[T64 + 1]) {
  int64_t u = (int64_t)((sqrt(8.0 * (double)L + 1.0) - 1.0) * 0.5);
  while (u * (u + 1) / 2 > L) --u;
  while ((u + 1) * (u + 2) / 2 <= L) ++u;
  const int64_t v = L - u * (u + 1) / 2;
  const SymPair p{v * 64, u * 64, u == v};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t cJ = p.J + lane, cI = p.I + lane, last = M - 1;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + wave;
    ha[q] = ld(p.I + r < M ? p.I + r : last, cJ < M ? cJ : last);
    hb[q] = ld(p.J + r < M ? p.J + r : last, cI < M ? cI : last);
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + wave;
    if (p.I + r >= M || cJ >= M) ha[q] = 0.0;
    if (p.J + r >= M || cI >= M) hb[q] = 0.0;
    ta[r][lane] = ha[q];
    tb[r][lane] = hb[q];
  }
  __syncthreads();
  return p;
}

// Upper-triangle tiles are ordered in G x G groups of the tile grid (the
// diagonal groups are triangular), row-major inside a group; tile_of_index
// gives tile L of that order in closed form (a search over the groups took
// up to a thousand scalar steps per block).
constexpr int TILE_GROUP = 8;

__device__ __forceinline__ void tile_of_index(int L, int nt, int &ti, int &tj) {
  constexpr int G = TILE_GROUP;
  // group row gr: rows gr G .. ; the rows before row s hold s nt - s (s - 1)/2 tiles
  auto before = [&](int gr) {
    const int s = gr * G;
    return s * nt - s * (s - 1) / 2;
  };
  const float q = 2.0f * nt + 1.0f;
  int gr = (int)((q - sqrtf(fmaxf(q * q - 8.0f * L, 0.0f))) * (0.5f / G));
  while (gr > 0 && before(gr) > L) --gr;
  while ((gr + 1) * G < nt && before(gr + 1) <= L) ++gr;
  int rem = L - before(gr);
  const int r0 = gr * G, rows = min(G, nt - r0), diag = rows * (rows + 1) / 2;
  if (rem < diag) {
    int t = 0;
    while (rem >= rows - t) {
      rem -= rows - t;
      ++t;
    }
    ti = r0 + t;
    tj = ti + rem;
    return;
  }
  rem -= diag;   // full groups of G rows (the last may have fewer columns)
  const int k = rem / (G * G), c0 = (gr + 1 + k) * G, w = min(G, nt - c0);
  rem -= k * G * G;
  ti = r0 + rem / w;
  tj = c0 + rem % w;
}

// Tile of block b of the first nblk blocks, which cover tiles 0 .. nblk-1 of
// that order.  Blocks are dispatched round-robin over the 8 XCDs; each XCD
// gets a contiguous run of the order, so the tiles resident on one XCD at a
// time fall in few groups and read few row panels, which its L2 serves.
__device__ __forceinline__ void tile_of_block(int b, int nblk, int nt, int &ti, int &tj, int &lin) {
  const int xcd = b & 7, loc = b >> 3, q = nblk >> 3, r = nblk & 7;
  lin = xcd * q + (xcd < r ? xcd : r) + loc;
  tile_of_index(lin, nt, ti, tj);
}

__device__ __forceinline__ void tile_of_block(int b, int nt, int &ti, int &tj, int &lin) {
  tile_of_block(b, nt * (nt + 1) / 2, nt, ti, tj, lin);
}

// Geometry of the tile product.  A K stage is one 128-byte segment of every
// panel row (16 FP64, 32 FP32, 64 values of one 16-bit plane, or 32 of two
// interleaved planes); three planes take a 64-byte segment of each (32
// values).
//
// Wave layout.  16-bit: 2 x 2 waves of 2 x 2 MFMA blocks.  FP64 / FP32: waves
// 0 and 1 take the upper and lower 32 rows, 2 x 4 blocks each, of the first
// half of every stage's K values, waves 2 and 3 of the second half.  With
// 2 x 2 blocks per wave (four accumulators) FP64 products alone reach 67
// TFLOP/s, however many waves there are; with eight accumulators 78.
//
// Stages in LDS: FP64 runs best with four blocks per CU, FP32 with two (the
// product loop alone, in TFLOP/s: FP32 139 with two blocks, 89 with three;
// FP64 71.6 and 72.5); FP32 uses the LDS of the other two for a deeper ring.
template <int P> struct TileCfg {
  using T = typename Enc<P>::T;
  static constexpr int NP = Enc<P>::NP, KIND = Enc<P>::KIND, ES = (int)sizeof(T);
  static constexpr int TE = T64;                           // tile edge
  static constexpr int KS = KIND <= 1 ? 2 : 1;             // wave groups along K
  static constexpr int WA = TE / 32, WB = WA * KS;         // MFMA blocks per wave
  static constexpr bool R128 = NP <= 2;
  static constexpr int KT = R128 ? 128 / ES / NP : 32;     // K values per stage
  static constexpr int ROWB = R128 ? 128 : 64 * NP;        // bytes per panel row per stage
  static constexpr int STAGE = 2 * TE * ROWB;              // bytes per stage
  static constexpr int NBUF = KIND == 1 ? 4 : KIND >= 2 && NP <= 2 ? 3 : 2;   // stages in LDS
  static constexpr int SMEM = NBUF * STAGE;
  static constexpr int LPS = STAGE / 1024 / 4;             // 1 KiB loads per stage per wave
  static constexpr int NX = R128 ? 2 : NP;                 // 16-byte fragments per row
  static constexpr int NXW = NX / KS;                      // ... that a wave reads
  static_assert(KS == 1 || NP == 1, "K halves of one-plane stages");
  using Acc = typename AccType<KIND>::type;
  using S = std::conditional_t<KIND == 0, double, float>;
};

// Bare s_barrier: __syncthreads() would add a workgroup release fence, which
// waits for every outstanding LDS-DMA load.  The empty asm statements keep
// the compiler from moving LDS accesses across it, the scheduling barriers
// keep the matrix products on their side of it; the waits before it provide
// the hardware ordering.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// acc[bi][bj] = rows of A x rows of B over the K stages [kb, ke).  Lane l of a
// wave holds row wrow + bi*16 + l%16 and the four columns wcol + bj*16 +
// acc_row<KIND>(l/16, r) of the tile, with (wrow, wcol) from tile_origin.
//
// FP32 and the 16-bit encodings add all products of `fold` stages into a
// chunk accumulator and that into a running total; FP64 keeps one
// accumulator.  Ends with a barrier: smem is free.
//
// Panels go from global memory straight to LDS (16 bytes per lane, one wave
// instruction fills 1 KiB).  In 128-byte rows chunk c sits at slot c ^ (R % 8)
// and a lane reads whole 16-byte chunks (two FP64 or four FP32 values of K,
// the same ones of A and B, so their order inside the stage does not
// matter), which reads LDS without bank conflicts; 64-byte rows use slot
// c ^ ((R >> 1) ^ (R >> 3)) % 4.
template <class C>
__device__ __forceinline__ void tile_origin(int wave, int &wrow, int &wcol) {
  wrow = (C::KS == 1 ? wave >> 1 : wave & 1) * 16 * C::WA;
  wcol = C::KS == 1 ? (wave & 1) * 16 * C::WB : 0;
}

template <class C, int P>
__device__ __forceinline__ void tile_mma(const void *A, const void *B, int64_t arow0,
                                         int64_t brow0, int64_t Mp, char *smem, int fold, int kb,
                                         int ke, typename C::Acc (&acc)[C::WA][C::WB]) {
  using Acc = typename C::Acc;
  constexpr int TE = C::TE, LPS = C::LPS, NX = C::NXW, KIND = C::KIND, WA = C::WA, WB = C::WB;
  constexpr bool R128 = C::R128;
  // The loop keeps its vector instructions to the products, the fragment
  // reads and the loads: FP64 products and vector instructions do not overlap
  // on a SIMD, so every address instruction costs product time.  Loads take a
  // scalar base that advances and a fixed 32-bit lane offset; fragments a
  // fixed LDS base with immediate offsets (two stages are unrolled).
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4, kg = C::KS == 1 ? 0 : wave >> 1;
  int wrow, wcol;
  tile_origin<C>(wave, wrow, wcol);
  const int64_t rowb = Mp * C::NP * C::ES;       // bytes per panel row
  const char *Ab = (const char *)A + arow0 * rowb, *Bb = (const char *)B + brow0 * rowb;

  // load q of a stage: rows of one panel (R128: the first half of the loads
  // fills A), swizzled chunk
  constexpr int PB = R128 ? 1 : 2 * TE / 16;   // loads per plane (three planes)
  uint32_t voff[LPS];
#pragma unroll
  for (int q = 0; q < LPS; ++q) {
    const int blk = wave + 4 * q;
    if constexpr (R128) {
      const int R = (q < LPS / 2 ? blk : blk - TE / 8) * 8 + (lane >> 3);   // row in its panel
      voff[q] = (uint32_t)(R * rowb) + ((lane & 7) ^ (R & 7)) * 16;
    } else {
      const int p = blk / PB, Rl = blk % PB * 16 + (lane >> 2), R = Rl & (TE - 1);
      voff[q] = (uint32_t)(R * rowb) + p * 64 + ((lane & 3) ^ (((Rl >> 1) ^ (Rl >> 3)) & 3)) * 16;
    }
  }
  auto issue = [&](int kt, char *st) {
    const char *pa = Ab + (int64_t)kt * C::ROWB, *pb = Bb + (int64_t)kt * C::ROWB;
#pragma unroll
    for (int q = 0; q < LPS; ++q) {
      const int blk = wave + 4 * q;
      const bool isA = R128 ? q < LPS / 2 : blk % PB < TE / 16;
      const char *src = (isA ? pa : pb) + voff[q];
      char *dst = st + (R128 ? blk * 1024 : (blk / PB * 2 * TE + blk % PB * 16) * 64);
      __builtin_amdgcn_global_load_lds((const void *)src, (lds_void *)dst, 16, 0, 0);
    }
  };
  // fragment x of MFMA row block b of this wave (panel rows rb ..)
  auto frag = [&](const char *st, int rb, int b, int x) -> v4u {
    const int R = rb + b * 16 + l16;
    if constexpr (R128)   // R % 8 does not depend on b
      return *(const v4u *)(st + ((rb + l16) * 128 + (((kg + x) * 4 + lg) ^ (l16 & 7)) * 16) + b * 2048);
    else
      return *(const v4u *)(st + (x * 2 * TE + R) * 64 + (lg ^ (((R >> 1) ^ (R >> 3)) & 3)) * 16);
  };

  // 16-bit: every GF folds the FP32 totals move on into FP64 ones, so that a
  // term's roundings do not grow with K.  The registers are free here (the
  // epilogue needs more), the conversions take 0 to 2 % of a product.  Error of
  // a solve, FP16X3, without -> with (and folds every second stage): M = 1500
  // 4.3e-7 -> 3.3e-7, M = 2500 4.7e-7 -> 3.3e-7; BF16X6 at 2500 5.3e-7 -> 3.8e-7.
  // GF = 8 takes the same time and errs 5 % more.
  constexpr bool FOLD = KIND != 0, RUN64 = KIND >= 2;
  constexpr int GF = 4;
  Acc tot[WA][WB];
  double run[RUN64 ? WA : 1][RUN64 ? WB : 1][4] = {};
  int to_drain = GF;   // folds until then
#pragma unroll
  for (int bi = 0; bi < WA; ++bi)
#pragma unroll
    for (int bj = 0; bj < WB; ++bj) acc[bi][bj] = tot[bi][bj] = Acc{};

  // Products of a stage, largest first: split encodings pair the planes.
  constexpr int NPR = C::NP == 1 ? 2 : Enc<P>::NPROD;
  constexpr int PA[6] = {0, 0, 1, 1, 0, 2};
  constexpr int PB2[6] = {0, 1, 0, 1, 2, 0};

  int left = fold;   // stages until the next fold
  // s_waitcnt immediate: vmcnt <= the loads of the PD - 1 stages after the one
  // waited for, lgkmcnt 0, expcnt not waited on
  constexpr int PD = C::NBUF - 1, AHEAD = (PD - 1) * LPS;
  static_assert(AHEAD <= 63, "vmcnt range");
  constexpr int WAIT = (AHEAD & 0xF) | ((AHEAD >> 4) << 14) | (0x7 << 4);
  auto drain = [&] {
    if constexpr (RUN64) {
#pragma unroll
      for (int bi = 0; bi < WA; ++bi)
#pragma unroll
        for (int bj = 0; bj < WB; ++bj)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            run[bi][bj][r] += (double)tot[bi][bj][r];
            tot[bi][bj][r] = 0.0f;
          }
    }
  };
  auto stage = [&](int kt, int buf) {
    const char *st = smem + buf * C::STAGE;
    if (PD > 1 && kt + PD - 1 < ke)
      __builtin_amdgcn_s_waitcnt(WAIT);
    else
      __builtin_amdgcn_s_waitcnt(0);
    // this wave's loads of stage kt have landed; after the barrier everyone's
    // have, and the buffer of stage kt - 1 is free
    bare_barrier();
    v4u af[WA][NX], bf[WB][NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
#pragma unroll
      for (int b = 0; b < WA; ++b) af[b][x] = frag(st, wrow, b, x);
#pragma unroll
      for (int b = 0; b < WB; ++b) bf[b][x] = frag(st, TE + wcol, b, x);
    }
    // the fragment reads go out before the loads (which take long to issue),
    // and those before the first product
    __builtin_amdgcn_sched_barrier(0);
    if (kt + PD < ke) issue(kt + PD, smem + (buf + PD) % C::NBUF * C::STAGE);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (KIND == 0) {
#pragma unroll
      for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int bi = 0; bi < WA; ++bi)
#pragma unroll
            for (int bj = 0; bj < WB; ++bj)
              acc[bi][bj] = mfma(__builtin_bit_cast(v2d, bf[bj][x])[e],
                                 __builtin_bit_cast(v2d, af[bi][x])[e], acc[bi][bj]);
    } else if constexpr (KIND == 1) {
#pragma unroll
      for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int bi = 0; bi < WA; ++bi)
#pragma unroll
            for (int bj = 0; bj < WB; ++bj)
              acc[bi][bj] = mfma(__builtin_bit_cast(v4f, bf[bj][x])[e],
                                 __builtin_bit_cast(v4f, af[bi][x])[e], acc[bi][bj]);
    } else {
#pragma unroll
      for (int pr = 0; pr < NPR; ++pr)
#pragma unroll
        for (int bi = 0; bi < WA; ++bi)
#pragma unroll
          for (int bj = 0; bj < WB; ++bj) {
            const int xa = C::NP == 1 ? pr : PA[pr], xb = C::NP == 1 ? pr : PB2[pr];
            acc[bi][bj] = mfma16<KIND>(bf[bj][xb], af[bi][xa], acc[bi][bj]);
          }
    }
    if constexpr (FOLD) {
      if (--left == 0 || kt + 1 == ke) {
        left = fold;
#pragma unroll
        for (int bi = 0; bi < WA; ++bi)
#pragma unroll
          for (int bj = 0; bj < WB; ++bj) {
            tot[bi][bj] += acc[bi][bj];
            acc[bi][bj] = Acc{};
          }
        if constexpr (RUN64)
          if (--to_drain == 0) {
            to_drain = GF;
            drain();
          }
      }
    }
  };
#pragma unroll
  for (int s = 0; s < PD; ++s)
    if (kb + s < ke) issue(kb + s, smem + s * C::STAGE);
  for (int kt = kb; kt < ke; kt += C::NBUF) {
#pragma unroll
    for (int s = 0; s < C::NBUF; ++s)
      if (kt + s < ke) stage(kt + s, s);
  }
  if constexpr (FOLD) {
#pragma unroll
    for (int bi = 0; bi < WA; ++bi)
#pragma unroll
      for (int bj = 0; bj < WB; ++bj)
        if constexpr (RUN64) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[bi][bj][r] = (float)(run[bi][bj][r] + (double)tot[bi][bj][r]);
        } else {
          acc[bi][bj] = tot[bi][bj];
        }
  }
  __syncthreads();
}

// The same with the whole 64 x 64 tile as the result, in LDS: V[row][col] with
// a row pitch of VP elements (a product of the K halves adds the second
// half's totals to the first's).  Ends with a barrier.
constexpr int VP = T64 + 1;

template <int P>
__device__ __forceinline__ void tile_product(const void *A, const void *B, int64_t arow0,
                                             int64_t brow0, int64_t Mp, char *smem, int fold,
                                             int kb, int ke) {
  using C = TileCfg<P>;
  typename C::Acc acc[C::WA][C::WB];
  tile_mma<C, P>(A, B, arow0, brow0, Mp, smem, fold, kb, ke, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lg = lane >> 4;
  int wrow, wcol;
  tile_origin<C>(wave, wrow, wcol);
  typename C::S *V = (typename C::S *)smem + (wrow + l16) * VP + wcol;
  auto each = [&](auto &&f) {
#pragma unroll
    for (int bi = 0; bi < C::WA; ++bi)
#pragma unroll
      for (int bj = 0; bj < C::WB; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          f(V[bi * 16 * VP + bj * 16 + acc_row<C::KIND>(lg, r)], acc[bi][bj][r]);
  };
  using S = typename C::S;
  if (C::KS == 1 || wave >= 2) each([](S &v, S x) { v = x; });
  __syncthreads();
  if constexpr (C::KS == 2) {
    if (wave < 2) each([](S &v, S x) { v = x + v; });
    __syncthreads();
  }
}

// v[u][e] = the sum of the n partial tiles w, w + ps, .. at QC rows of this
// thread, which blocks on other XCDs have written in this launch: stored and
// loaded at agent scope, 8 bytes at a time.  (Plain accesses between
// __threadfence() calls write back and invalidate a whole L2 per block:
// measured 65 us instead of 30 per FP16X3 product at M = 1000.)
template <class S, int QC>
__device__ __forceinline__ void add_partials(const S *w, int64_t ps, int n, double (&v)[QC][4]) {
  typedef S v4s __attribute__((ext_vector_type(4)));
  constexpr int NW = (int)sizeof(v4s) / 8;
  union Pack {
    uint64_t u[NW];
    v4s x;
  };
#pragma unroll
  for (int q = 0; q < QC; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[q][e] = 0.0;
#pragma unroll 2
  for (int s = 0; s < n; ++s)
#pragma unroll
    for (int q = 0; q < QC; ++q) {
      const S *p = w + s * ps + q * 16 * T64;
      Pack t;
#pragma unroll
      for (int k = 0; k < NW; ++k)
        t.u[k] = __hip_atomic_load((const uint64_t *)p + k, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[q][e] += (double)t.x[e];
    }
}

template <class S>
__device__ __forceinline__ void publish4(S *p, S a, S b, S c, S d) {
  typedef S v4s __attribute__((ext_vector_type(4)));
  constexpr int NW = (int)sizeof(v4s) / 8;
  union Pack {
    uint64_t u[NW];
    v4s x;
  } t;
  t.x = v4s{a, b, c, d};
#pragma unroll
  for (int k = 0; k < NW; ++k)
    __hip_atomic_store((uint64_t *)p + k, t.u[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One split of a tile: publishes this thread's elements of V (its own base in
// a 64 x 64 LDS tile) to w (its own base in the split's partial tile) and
// counts the split.  True in the block that completes the tile, where all
// partials may be read and smem is free.
template <class S>
__device__ __forceinline__ bool publish_split(const S *V, S *w, unsigned *cnt, int nsplit,
                                              char *smem) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const S *v = V + q * 16 * VP;
    publish4(w + q * 16 * T64, v[0], v[1], v[2], v[3]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // out before the counter moves
  __syncthreads();
  unsigned *last = (unsigned *)smem;
  if (threadIdx.x == 0) *last = atomicAdd(cnt, 1u) == (unsigned)nsplit - 1;
  __syncthreads();
  if (!*last) return false;
  __syncthreads();   // flag read by all before smem is used again
  if (threadIdx.x == 0) *cnt = 0u;   // ready for the next launch
  return true;
}

// ------------------------------------------------------ 32 x 32 tiles
// For products of few tiles: a 32 x 32 tile per block, whose four waves take
// every fourth K stage of the whole tile (2 x 2 MFMA blocks each) through LDS
// rings of their own, without barriers; their totals are added in FP64.
template <int P, int NB_> struct SmallCfg {
  using C = TileCfg<P>;
  using Acc = typename C::Acc;
  using S = typename C::S;
  static constexpr int TE = 32, NB = NB_, PD = NB - 1;   // stages in a wave's ring, ahead
  static constexpr int STAGE = 2 * TE * C::ROWB;         // bytes
  static constexpr int LPS = STAGE / 1024;               // loads per stage
  static constexpr int RING = NB * STAGE;
  static constexpr int SMEM = 4 * RING;
  static_assert(PD * LPS <= 63 && RING >= TE * (TE + 1) * (int)sizeof(S), "vmcnt range, result fits");
};

// v[e] = element (row, c4 + e) of the tile at (arow0, brow0) for row = tid / 8
// and c4 = 4 (tid % 8).  Ends with a barrier: smem is free.
template <int P, int NB>
__device__ __forceinline__ void small_product(const void *A, const void *B, int64_t arow0,
                                              int64_t brow0, int64_t Mp, char *smem, int fold,
                                              double (&v)[4]) {
  using C = TileCfg<P>;
  using Z = SmallCfg<P, NB>;
  using Acc = typename C::Acc;
  using S = typename C::S;
  constexpr int KIND = C::KIND, NX = C::NX, LPS = Z::LPS, PD = Z::PD, TE = Z::TE;
  constexpr bool R128 = C::R128;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4, nk = (int)(Mp / C::KT);
  const int64_t rowb = Mp * C::NP * C::ES;
  const char *Ab = (const char *)A + arow0 * rowb, *Bb = (const char *)B + brow0 * rowb;
  char *ring = smem + wave * Z::RING;
  // 128-byte rows: 8 rows per load; 64-byte rows of a plane: 16
  constexpr int RPL = R128 ? 8 : 16, LPA = TE / RPL;   // rows per load, loads per panel (and plane)
  uint32_t voff[LPS];
#pragma unroll
  for (int q = 0; q < LPS; ++q) {
    const int p = q / (2 * LPA), R = q % LPA * RPL + (R128 ? lane >> 3 : lane >> 2);
    voff[q] = (uint32_t)(R * rowb) +
              (R128 ? ((lane & 7) ^ (R & 7)) * 16
                    : p * 64 + ((lane & 3) ^ (((R >> 1) ^ (R >> 3)) & 3)) * 16);
  }
  auto issue = [&](int kt, char *st) {
    const char *pa = Ab + (int64_t)kt * C::ROWB, *pb = Bb + (int64_t)kt * C::ROWB;
#pragma unroll
    for (int q = 0; q < LPS; ++q)
      __builtin_amdgcn_global_load_lds((const void *)((q % (2 * LPA) < LPA ? pa : pb) + voff[q]),
                                       (lds_void *)(st + q * 1024), 16, 0, 0);
  };
  auto frag = [&](const char *st, int pan, int b, int x) -> v4u {   // panel 0: A, 1: B
    const int R = b * 16 + l16;
    if constexpr (R128)
      return *(const v4u *)(st + (pan * TE + R) * 128 + ((x * 4 + lg) ^ (R & 7)) * 16);
    else
      return *(const v4u *)(st + ((x * 2 + pan) * TE + R) * 64 +
                            (lg ^ (((R >> 1) ^ (R >> 3)) & 3)) * 16);
  };
  Acc acc[2][2], tot[2][2];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = tot[bi][bj] = Acc{};
  constexpr int NPR = C::NP == 1 ? 2 : Enc<P>::NPROD;
  constexpr int PA[6] = {0, 0, 1, 1, 0, 2};
  constexpr int PB2[6] = {0, 1, 0, 1, 2, 0};
  constexpr int AHEAD = (PD - 1) * LPS;
  constexpr int WAIT = (AHEAD & 0xF) | ((AHEAD >> 4) << 14) | (0x7 << 4);
  int left = fold;
#pragma unroll
  for (int s = 0; s < PD; ++s)
    if (wave + 4 * s < nk) issue(wave + 4 * s, ring + s * Z::STAGE);
  int buf = 0;
  for (int kt = wave; kt < nk; kt += 4) {
    if (PD > 1 && kt + 4 * (PD - 1) < nk)
      __builtin_amdgcn_s_waitcnt(WAIT);
    else
      __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const char *st = ring + buf * Z::STAGE;
    v4u af[2][NX], bf[2][NX];
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        af[b][x] = frag(st, 0, b, x);
        bf[b][x] = frag(st, 1, b, x);
      }
    __builtin_amdgcn_sched_barrier(0);
    // the buffer of the previous stage: its fragments have been used
    if (kt + 4 * PD < nk) issue(kt + 4 * PD, ring + (buf + PD) % NB * Z::STAGE);
    __builtin_amdgcn_sched_barrier(0);
    buf = buf + 1 == NB ? 0 : buf + 1;
    if constexpr (KIND <= 1) {
      constexpr int NE = KIND == 0 ? 2 : 4;
      typedef S vs __attribute__((ext_vector_type(NE)));
#pragma unroll
      for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
          for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
              acc[bi][bj] = mfma(__builtin_bit_cast(vs, bf[bj][x])[e],
                                 __builtin_bit_cast(vs, af[bi][x])[e], acc[bi][bj]);
    } else {
#pragma unroll
      for (int pr = 0; pr < NPR; ++pr)
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) {
            const int xa = C::NP == 1 ? pr : PA[pr], xb = C::NP == 1 ? pr : PB2[pr];
            acc[bi][bj] = mfma16<KIND>(bf[bj][xb], af[bi][xa], acc[bi][bj]);
          }
    }
    if constexpr (KIND != 0) {
      if (--left == 0 || kt + 4 >= nk) {
        left = fold;
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) {
            tot[bi][bj] += acc[bi][bj];
            acc[bi][bj] = Acc{};
          }
      }
    }
  }
  // every wave leaves its totals in its own ring
  S *V = (S *)ring + l16 * (TE + 1);
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        V[bi * 16 * (TE + 1) + bj * 16 + acc_row<KIND>(lg, r)] =
            KIND == 0 ? acc[bi][bj][r] : tot[bi][bj][r];
  __syncthreads();
  const int o = (tid >> 3) * (TE + 1) + (tid & 7) * 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) v[e] += (double)((const S *)(smem + w * Z::RING))[o + e];
  }
  __syncthreads();
}

}  // namespace gcp
