// gcp_verify.hip -- FP64 checks of a density matrix against H (gfx950).
//
// For a symmetric D and H (both read as their symmetric parts):
//   Tr D and ||D||_F^2      -- a projector has both equal to N (the trace and
//                              Frobenius tests that follow the convergence
//                              discussion; ||D||_F^2 is read as the square)
//   ||D^2 - D||_F           -- idempotency, from an FP64 MFMA product D D
//   Tr(D H) = sum D o H     -- the energy, equal to the sum of the N lowest
//                              eigenvalues of H for the ground-state projector
//   ||H D - D H||_F         -- the commutator, from an FP64 MFMA product H D
//                              (D H = (H D)^T for symmetric H and D)
// Every sum is FP64 and reduced in a fixed order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcp_encode.h"
#include "gcp_kernels.h"
#include "gcp_mma.h"

namespace gcp {

// One 64 x 64 upper tile (ti <= tj) of one product per block, sums over the
// tile's elements with the mirrored ones (w_ij = 2 off the diagonal).
//   MODE 0: X = D D.  Sums of w (X - D)^2, w D H, w D^2 and the trace of D.
//   MODE 1: H D - D H, both products over the same panels, (D H)_ij being
//           (H D)_ji: the sum of w ((H D)_ij - (H D)_ji)^2.  Neither product
//           is stored.
// The tile sums go to tpart[5][ntri].
template <int MODE>
__device__ __forceinline__ void verify_tile(const VerifyArgs &a, int L, char *smem, double *red) {
  const int64_t Mp = a.Mp;
  const int nk = (int)(Mp / TileCfg<GCP_FP64>::KT);
  int ti, tj, lin;
  tile_of_block(L, a.ntri, a.nt, ti, tj, lin);
  const int64_t arow0 = (int64_t)ti * T64, brow0 = (int64_t)tj * T64;
  const double *__restrict__ D = a.D;
  const double *__restrict__ H = a.H;
  constexpr int NS = MODE == 0 ? 4 : 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c4 = (tid & 15) * 4, r0 = tid >> 4;
  const double *V = (const double *)smem + r0 * VP + c4;   // this thread's elements
  double p[4][4], v[NS] = {};
  tile_product<GCP_FP64>(MODE == 0 ? D : H, D, arow0, brow0, Mp, smem, 0, 0, nk);
  if constexpr (MODE == 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) p[q][e] = V[q * 16 * VP + e];
    __syncthreads();   // V read before the next product's stages land in it
    tile_product<GCP_FP64>(D, H, arow0, brow0, Mp, smem, 0, 0, nk);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t i = arow0 + q * 16 + r0, j = brow0 + c4 + e;
      if (i > j) continue;
      const double w = i == j ? 1.0 : 2.0;
      const double m = V[q * 16 * VP + e];
      if constexpr (MODE == 1) {
        const double x = p[q][e] - m;
        v[0] += w * x * x;
      } else {
        const double d = D[i * Mp + j], x = m - d;
        v[0] += w * x * x;
        v[1] += w * d * H[i * Mp + j];
        v[2] += w * d * d;
        if (i == j) v[3] += d;
      }
    }
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    v[k] = wave_sum(v[k]);
    if (lane == 0) red[k * 4 + wave] = v[k];
  }
  __syncthreads();
  if (tid < NS)
    a.tpart[(MODE == 1 ? 4 : tid) * a.ntri + lin] =
        ((red[tid * 4] + red[tid * 4 + 1]) + red[tid * 4 + 2]) + red[tid * 4 + 3];
}

// The commutator's tiles (twice the work) come first.
__global__ __launch_bounds__(NTH, 3) void k_vgemm(VerifyArgs a) {
  constexpr int MM = T64 * VP * 8;
  static_assert(MM >= TileCfg<GCP_FP64>::SMEM, "the product's stages fit");
  __shared__ __attribute__((aligned(16))) char smem[MM + 16 * 8];
  const int b = (int)blockIdx.x;
  if (b < a.ntri) verify_tile<1>(a, b, smem, (double *)(smem + MM));
  else verify_tile<0>(a, b - a.ntri, smem, (double *)(smem + MM));
}

// out[k] = sum of tpart[k][..] in a fixed order, one block per sum.
__global__ __launch_bounds__(256) void k_vsum(VerifyArgs a) {
  __shared__ double s[256];
  const int k = (int)blockIdx.x;
  double v = 0.0;
#pragma unroll 4
  for (int t = threadIdx.x; t < a.ntri; t += 256) v += a.tpart[(int64_t)k * a.ntri + t];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.out[k] = s[0];
}

hipError_t launch_verify(const VerifyArgs &a, hipStream_t st) {
  k_vgemm<<<(unsigned)(2 * a.ntri), NTH, 0, st>>>(a);
  k_vsum<<<5, 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace gcp
