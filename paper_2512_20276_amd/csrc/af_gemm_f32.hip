// fp32 projection GEMM for small models: many small tiles, the K range split over the waves.
#include "af_device.h"
#include "af_epilogue.h"

namespace af {

// One workgroup = 16 rows x 32 columns (two weight blocks); its four waves take the 32-wide k
// steps in turn and their sums meet in LDS.  Such a step is bound by latency: the projections of
// a model of d 256 have 0.2 to 0.7 MB of weights and K of 256 or 688, so what counts is how many
// loads are outstanding at once and how long the serial chain is.  Every wave requests UN steps
// (its whole share at K = 256 and K = 768) before it uses any, nothing is staged through LDS on the way
// in, and 34 rows make 24 to 129 workgroups.  Measured per launch at 34 rows, d 256, against the
// 96 x 128 tile of gemm_kernel (2 to 11 workgroups, most of their rows padding, one k step of
// fragments after the other): qkv 25.5 -> 4.2 us, output 21.0 -> 4.0, gate/up 20.3 -> 4.2, down
// 18.4 -> 5.8, LM head of 3 rows 7.9 -> 3.4; the whole step 224 -> 74 us.
template <int EPI, int UN>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(GemmArgs a) {
  typedef Mma<float>::frag frag;
  __shared__ __attribute__((aligned(16))) float T_[4][2][64][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
  const int n_mt = (a.M + 15) / 16;
  const int mt = blockIdx.x % n_mt, nt = blockIdx.x / n_mt;
  const int n_blocks = a.N >> 4, ksteps = a.Kp >> 5;
  // rows past M repeat the last one and are never stored; k past K meets zero weights
  const float* arow = (const float*)a.A + (size_t)min(mt * 16 + lr, a.M - 1) * a.lda;
  const float* brow[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) brow[n] = (const float*)a.B + (size_t)min(2 * nt + n, n_blocks - 1) * a.bstride + lane * 8;
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  for (int k0 = wave; k0 < ksteps; k0 += 4 * UN) {
    frag x[UN], w[UN][2];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int ks = min(k0 + 4 * u, ksteps - 1), k = ks * 32 + lg * 8;
      ((f32x4*)&x[u])[0] = *(const f32x4*)(arow + min(k, a.K - 4));
      ((f32x4*)&x[u])[1] = *(const f32x4*)(arow + min(k + 4, a.K - 4));
#pragma unroll
      for (int n = 0; n < 2; ++n) w[u][n] = *(const frag*)(brow[n] + (size_t)ks * 512);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      // a step past the last one has loaded that one again: it adds nothing (not a product with
      // zeros, which an infinite weight would make NaN); the same for every lane of the wave
      if (UN > 2 && __builtin_amdgcn_readfirstlane(k0 + 4 * u) >= ksteps) break;
      // weights first: lane l then holds columns 4 lg .. 4 lg + 3 of row lr
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[n] = Mma<float>::mma(w[u][n], x[u], acc[n]);
    }
  }
#pragma unroll
  for (int n = 0; n < 2; ++n) *(f32x4*)T_[wave][n][lane] = acc[n];
  __syncthreads();
  if (threadIdx.x >= 32) return;
  // one thread per row and 16-column block: the waves' sums are added in wave order
  const int row = threadIdx.x & 15, blk = threadIdx.x >> 4;
  const int m = mt * 16 + row, nc = (2 * nt + blk) * 16;
  if (m >= a.M || nc >= a.N) return;
  float v[16];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 s = *(const f32x4*)T_[0][blk][16 * q + row];
#pragma unroll
    for (int w = 1; w < 4; ++w) s += *(const f32x4*)T_[w][blk][16 * q + row];
    *(f32x4*)&v[4 * q] = s;
  }
  if constexpr (EPI == EPI_SWIGLU || EPI == EPI_QKV) {
    epi_group16<float, EPI>(a, m, nc, v, v + 8);
  } else {
    epi_group8<float, EPI>(a, m, nc, v);
    epi_group8<float, EPI>(a, m, nc + 8, v + 8);
  }
}

template <int UN>
static hipError_t f32_small_launch(int epi, const GemmArgs& a, hipStream_t s) {
  const dim3 grid(((a.M + 15) / 16) * ((a.N + 31) / 32)), block(256);
  switch (epi) {
    case EPI_STORE:
    case EPI_STORE_F32: hipLaunchKernelGGL((gemm_f32_small_kernel<EPI_STORE_F32, UN>), grid, block, 0, s, a); break;
    case EPI_RESID: hipLaunchKernelGGL((gemm_f32_small_kernel<EPI_RESID, UN>), grid, block, 0, s, a); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((gemm_f32_small_kernel<EPI_SWIGLU, UN>), grid, block, 0, s, a); break;
    case EPI_QKV: hipLaunchKernelGGL((gemm_f32_small_kernel<EPI_QKV, UN>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm_f32_small(int epi, const GemmArgs& a, hipStream_t s) {
  if (a.splits != 1 || a.col0 != 0 || a.N % 16 || a.K % 4 || a.K < 4 || a.Kp % 256 || a.Kp < a.K) return hipErrorInvalidValue;
  return a.Kp == 256 ? f32_small_launch<2>(epi, a, s) : f32_small_launch<6>(epi, a, s);
}

}  // namespace af
