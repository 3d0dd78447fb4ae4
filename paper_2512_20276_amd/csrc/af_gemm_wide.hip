// bf16 projection GEMMs on 288 x 256 and 288 x 128 tiles, for many packed rows.
#include "af_device.h"
#include "af_epilogue.h"

namespace af {

// 16 bytes per lane from p + voff; counted by vmcnt.  (The register is an in-out operand, so that a
// refill stays in the registers of its ring slot.)
__device__ __forceinline__ void load16(bf16x8& v, const void* p, unsigned voff) {
  asm volatile("global_load_dwordx4 %0, %1, %2" : "+v"(v) : "v"(voff), "s"(p) : "memory");
}

// Wide tile for many rows: 288 rows x 256 columns on eight waves, as two row groups (five and four
// 32-row blocks) x four column groups of 64 columns.  Waves 0..3 and 4..7 sit on the same four
// SIMDs, so every SIMD runs one wave of each row group: 18 MFMAs per 16-wide k step and SIMD.
// Every activation fragment read from LDS feeds two MFMAs: the LDS moves 45 KB a k step, 61 % of
// what it can in the time of the step's MFMAs, where eight waves of one column block each over
// all nine row blocks read 72 KB and were bound by them (54 KB of fragments per k step of 16 more
// than its MFMAs took).  Weights come straight from L2 into a register ring four k steps deep (a
// fragment is requested by both row groups, the second time from L1); the activations' DMAs run
// three stages ahead, one a k step per wave, so that no wait ever counts a burst of them.
//
// KG = 2: a 288 x 128 tile for the projections that need 256 workgroups of it to fill the GPU.
// Waves of one column block each would be LDS-bound again, so the waves keep 64 columns and form
// two k groups instead, which take the k steps of a stage in turn; their sums are added in the
// epilogue (group 0 first).  Against four waves of 64 columns, one per SIMD (gemm32x2_kernel), a
// SIMD has a second wave to run while one waits, and the two row groups' five and four blocks are
// balanced over the SIMDs.  2264 rows: 4096 columns 79.1 -> 72.9 us at K = 4096 and 194.7 -> 184.8 at
// K = 11008, 12288 columns 227.8 -> 209.5; 527 rows, 4096 columns, K = 11008 in four splits 61.2 ->
// 57.7.  It sums k in another order than the other tiles, so it is not taken with fixed_order.
//
// Measured for KG = 1 at K = 4096, 2264 rows, against waves of one column block: 12288 columns 225.6 ->
// 215.6 us, 22016 columns 358.8 -> 345.0.  In the packed step of that size the matrix cores are busy 60 %
// of the gate/up launch's cycles (54 % before), with the last of its three passes 69 % full, and 48 %
// in the output and down projections on KG = 2 (42 %); the clock gives part of it back (1.96 -> 1.87
// and 2.17 -> 2.07 GHz): the chip is at its power limit.
template <int KG, int EPI>
__global__ __launch_bounds__(512, 1) void gemm32w_kernel(GemmArgs a) {
  constexpr int FM = 9, KS = 4, NBUF = 4, PFB = 4, BLK = 512, TN = 256 / KG, PB = 3;
  constexpr int WPS = KS / KG;  // k steps of a stage taken by one k group
  constexpr int CBT = TN / 32;  // column blocks of the tile
  constexpr int SB = FM * KS;  // fragment blocks per stage
  constexpr int NPASS = (FM + PB - 1) / PB;
  __shared__ __attribute__((aligned(1024))) bf16 As[NBUF][SB * BLK];
  static_assert(32 * PB * TN * KG * 4 <= (int)sizeof(As), "an epilogue pass must fit the stage buffers");

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cg = wave & (4 / KG - 1), kg = (wave & 3) / (4 / KG);  // column group and k group
  const int n_blocks = (a.N + 31) >> 5, n_nt = (n_blocks + CBT - 1) / CBT;
  const int m_blocks = (a.M + 31) >> 5, n_mt = (m_blocks + FM - 1) / FM;
  const int S = a.splits;
  const int t = xcd_remap(blockIdx.x, n_mt * n_nt * S);
  const int mt = t % n_mt, rest = t / n_mt;
  const int sp = rest % S, nt = rest / S;
  const int ks16 = a.Kp >> 4;
  const int units = ks16 / (KS * NBUF), per = (units + S - 1) / S;
  const int kb = min(units, sp * per) * (KS * NBUF), ke = min(units, sp * per + per) * (KS * NBUF);
  const int n_st = (ke - kb) / KS;  // a multiple of NBUF
  // this wave's two weight blocks (past N: a valid block whose columns are never stored)
  const bf16* bp0 = (const bf16*)a.B + (size_t)min(nt * CBT + cg * 2, n_blocks - 1) * a.bstride;
  const bf16* bp1 = (const bf16*)a.B + (size_t)min(nt * CBT + cg * 2 + 1, n_blocks - 1) * a.bstride;
  const unsigned voff = lane * 16;
  const unsigned as0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) bf16*)&As[0][0]);
  const bf16* __restrict__ Ab = (const bf16*)a.A;
  float* T_ = (float*)&As[0][0];
  const int m0 = mt * FM * 32, n0 = nt * TN;

  // MB row blocks from MOFF on; D DMAs per stage issued by this wave
  auto body = [&](auto mb_c, auto moff_c, auto d_c) {
    constexpr int MB = decltype(mb_c)::value, MOFF = decltype(moff_c)::value, D = decltype(d_c)::value;
    // block q of a stage (row block q / KS, k step q % KS) lands at As[buf][q * BLK]; the first
    // DMA of k step 0 is the extra one of the waves that have D = KS + 1
    auto dma1 = [&](auto buf, int st, int i) {
      const int q = i < 4 ? wave + 8 * i : 28 + wave;  // i = 4: blocks 32..35 by waves 4..7
      const int mb = q / KS, j = q % KS;
      const int k = min(kb + st * KS + j, ks16 - 1);
      const int blk = min(mt * FM + mb, m_blocks - 1);  // rows past M: a valid block, never stored
      dma16((const char*)(Ab + (size_t)blk * a.astride + (size_t)k * BLK), voff, as0 + ((int)decltype(buf)::value * SB + q) * (BLK * 2));
    };
    bf16x8 rb[PFB][2] = {};
    // the group's k step i (counted over stages): step KG (i % WPS) + kg of stage i / WPS
    auto load_b = [&](auto slot, int st, int i) {
      const int k = min(kb + (st + i / WPS) * KS + KG * (i % WPS) + kg, ks16 - 1);
      const bf16* s0 = bp0 + (size_t)k * BLK;
      const bf16* s1 = bp1 + (size_t)k * BLK;
      load16(rb[slot][0], s0, voff);
      load16(rb[slot][1], s1, voff);
    };
    f32x16 acc[MB][2];
    static_for<0, MB>([&](auto i) {
      acc[i][0] = f32x16{};
      acc[i][1] = f32x16{};
    });
    static_for<0, NBUF - 1>([&](auto b) { static_for<0, D>([&](auto i) { dma1(b, b, decltype(i)::value); }); });
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, PFB>([&](auto j) { load_b(j, 0, decltype(j)::value); });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loop's waits count from a full ring
    __builtin_amdgcn_sched_barrier(0);
    for (int st0 = 0; st0 < n_st; st0 += NBUF) {
      static_for<0, NBUF>([&](auto u) {
        constexpr int U = decltype(u)::value;
        const int st = st0 + U;
        // Stage st's activations were issued NBUF - 1 stages ago, before the weights of every k
        // step that has been waited for since, and loads complete in order: the barrier alone
        // makes them visible to all waves (and frees buffer (st - 1) % NBUF).
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        bf16x8 af[2][MB];
        static_for<0, MB>([&](auto i) {
          af[0][i] = *(const bf16x8*)(&As[U][((MOFF + decltype(i)::value) * KS + kg) * BLK + lane * 8]);
        });
        static_for<0, WPS>([&](auto j) {
          constexpr int J = decltype(j)::value;
          constexpr int slot = (U * WPS + J) % PFB;
          if constexpr (J + 1 < WPS) {
            static_for<0, MB>([&](auto i) {
              af[(J + 1) & 1][i] = *(const bf16x8*)(&As[U][((MOFF + decltype(i)::value) * KS + KG * (J + 1) + kg) * BLK + lane * 8]);
            });
          }
          // k step j's weights were issued PFB of the group's steps ago; the PFB - 1 steps since then
          // have issued two weight loads and KG DMAs each, and the first of a stage one DMA more with
          // D = KS + 1
          constexpr int FIRST = (PFB - 1 - J) / WPS + (J > 0 ? 1 : 0);  // of the last PFB - 1 steps
          constexpr int WAIT = (2 + KG) * (PFB - 1) + (D > KS ? FIRST : 0);
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(WAIT) : "memory");
          __builtin_amdgcn_sched_barrier(0);
          static_for<0, MB>([&](auto i) {
            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[J & 1][i], rb[slot][0], acc[i][0], 0, 0, 0);
            acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[J & 1][i], rb[slot][1], acc[i][1], 0, 0, 0);
          });
          __builtin_amdgcn_sched_barrier(0);
          constexpr std::integral_constant<int, (U + NBUF - 1) % NBUF> nb{};
          if constexpr (D > KS && J == 0) dma1(nb, st + NBUF - 1, 4);
          static_for<0, KG>([&](auto q) { dma1(nb, st + NBUF - 1, KG * J + decltype(q)::value); });
          load_b(std::integral_constant<int, slot>{}, st, J + PFB);
          __builtin_amdgcn_sched_barrier(0);
        });
      });
    }
    // the ring's last (unused) loads land before any of its registers can be reused
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int p = 0; p < PFB; ++p) {
      asm volatile("" : "+v"(rb[p][0]));
      asm volatile("" : "+v"(rb[p][1]));
    }

    // ---- epilogue, PB row blocks per pass through the stage buffers
    constexpr bool paired = EPI == EPI_SWIGLU || EPI == EPI_QKV;
    constexpr int W = paired ? 16 : 8;
    static_for<0, NPASS>([&](auto p_c) {
      constexpr int PS = decltype(p_c)::value;
      constexpr int NB = PS * PB + PB <= FM ? PB : FM - PS * PB;  // row blocks in this pass
      __syncthreads();  // every wave's DMAs have landed and the buffers' last readers are done
      static_for<0, NB>([&](auto i) {
        constexpr int blk = PS * PB + decltype(i)::value;
        if constexpr (blk >= MOFF && blk < MOFF + MB) {
          static_for<0, 2>([&](auto c) {
            static_for<0, 16>([&](auto r) {
              constexpr int R = decltype(r)::value;
              const int row = (int)decltype(i)::value * 32 + 8 * (R / 4) + 4 * (lane >> 5) + (R % 4);
              T_[kg * (32 * PB * TN) + row * TN + (cg * 2 + (int)decltype(c)::value) * 32 + (lane & 31)] = acc[blk - MOFF][decltype(c)::value][R];
            });
          });
        }
      });
      __syncthreads();
      constexpr int ITEMS = 32 * NB * (TN / W);
      for (int it = tid; it < ITEMS; it += 512) {
        const int row = it / (TN / W), col = (it % (TN / W)) * W;
        const int m = m0 + PS * PB * 32 + row, nc = n0 + col;
        if (m >= a.M || nc >= a.N) continue;  // N % 16 == 0: a group is wholly inside or outside
        float v[W];
#pragma unroll
        for (int e = 0; e < W; e += 4) {
          f32x4 u = *(const f32x4*)&T_[row * TN + col + e];
          if constexpr (KG == 2) u += *(const f32x4*)&T_[32 * PB * TN + row * TN + col + e];
          *(f32x4*)&v[e] = u;
        }
        if (S > 1) {
          float* dst = a.partial + ((size_t)sp * a.M + m) * a.N + nc;
#pragma unroll
          for (int e = 0; e < W; e += 4) *(f32x4*)(dst + e) = *(const f32x4*)&v[e];
        } else if constexpr (paired) {
          epi_group16<bf16, EPI>(a, m, nc, v, v + 8);
        } else {
          epi_group8<bf16, EPI>(a, m, nc, v);
        }
      }
    });
  };
  if (wave < 4)
    body(std::integral_constant<int, 5>{}, std::integral_constant<int, 0>{}, std::integral_constant<int, 4>{});
  else
    body(std::integral_constant<int, 4>{}, std::integral_constant<int, 5>{}, std::integral_constant<int, 5>{});
}

template <int KG>
static hipError_t wide_launch(int epi, const GemmArgs& a, hipStream_t s) {
  constexpr int CBT = 8 / KG;  // column blocks of a tile
  const int mb = (a.M + 31) / 32, nb = (a.N + 31) / 32;
  const dim3 grid(((mb + 8) / 9) * ((nb + CBT - 1) / CBT) * a.splits), block(512);
  if (a.splits > 1) epi = EPI_STORE;  // partial sums only: one instance serves every epilogue
  switch (epi) {
    case EPI_STORE: hipLaunchKernelGGL((gemm32w_kernel<KG, EPI_STORE>), grid, block, 0, s, a); break;
    case EPI_RESID: hipLaunchKernelGGL((gemm32w_kernel<KG, EPI_RESID>), grid, block, 0, s, a); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((gemm32w_kernel<KG, EPI_SWIGLU>), grid, block, 0, s, a); break;
    case EPI_QKV: hipLaunchKernelGGL((gemm32w_kernel<KG, EPI_QKV>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm_wide(int epi, const GemmArgs& a, hipStream_t s) { return wide_launch<1>(epi, a, s); }

hipError_t launch_gemm_ksplit(int epi, const GemmArgs& a, hipStream_t s) {
  return a.fixed_order ? hipErrorInvalidValue : wide_launch<2>(epi, a, s);
}

}  // namespace af
