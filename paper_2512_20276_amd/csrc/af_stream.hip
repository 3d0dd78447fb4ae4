// bf16 projection GEMM for up to 192 rows: every row in one tile, K split over the waves.
#include "af_device.h"
#include "af_epilogue.h"

namespace af {

// acc += w . x over 16 k with the accumulator held in AGPRs (AG) or VGPRs.
template <bool AG>
__device__ __forceinline__ void mma(f32x16& acc, bf16x8 w, bf16x8 x) {
  if constexpr (AG)
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
  else
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(x));
}
template <bool AG>
__device__ __forceinline__ void pin(f32x16& acc) {
  if constexpr (AG)
    asm volatile("" : "+a"(acc));
  else
    asm volatile("" : "+v"(acc));
}

// A step of few packed rows is bound by the weights' way from HBM.  One workgroup = all 32 FM rows
// x 32 CB columns x one K split, so every weight is loaded by one CU only, and its four waves take
// the 16-wide k steps in turn: no fragment, of weights or activations, is used by two waves, so
// each wave streams both through an LDS ring of its own (up to 40 KB, R steps, filled by
// global_load_lds) without a barrier: up to 160 KB per CU are requested ahead.  The accumulators of
// the whole tile sit in every wave (FM CB x 16 registers, one wave per SIMD) and are summed through
// LDS at the end, RB row blocks at a time.  The product is taken with the weights as first operand,
// so that a lane holds four consecutive columns of a row and the sums are parked and read back
// with 16-byte accesses.
//
// What bounds it is the reads of 128 bytes that a CU keeps on their way, however many are requested
// (counters of layers of 1 to 15 and of 129 to 143 rows): with one row block 81 to 99, at 1130 to
// 1310 cycles each, since nearly all come from HBM; with five 62 to 66, at 550 to 610, as in the
// tiles that split K over workgroups only; the matrix cores are busy 6 and 16 to 20 % of the time.
// So a tile's cost is its (FM + CB) fragments a step, and with six row blocks two row tiles that
// share the weights through L2 (gemm32c_kernel) move no more bytes per CU and are as fast where K is
// split (192 rows, QKV of the 7B shape: 44.4 against 44.5 us here).
//
// FM <= 5: the step's fragments are read, then its ring slot is refilled, then the MFMAs run.
// FM = 6: there the MFMAs matter (18 per step and wave), so fragment reads run two row blocks
// ahead of them and each fragment's slot is refilled as soon as its MFMAs are issued.
//
// Measured for one 7B layer against the tiles of 128 columns split over K (gemm32_kernel,
// gemm32x2_kernel): 1 row 113.9 -> 103.3 us, 15 rows 125.3 -> 114.7, 103 rows 178.7 -> 161.3, 135 rows
// 183.7 -> 173.9; gate/up at 160 rows 60.7 -> 56.0 us, at 64 rows 48.0 -> 38.1, at 16 rows 36.0 ->
// 34.0 (5.3 TB/s of weights).
template <int FM, int CB, int R>
__global__ __launch_bounds__(256, 1) void gemm_stream_kernel(GemmArgs a, int epi) {
  constexpr int E = FM + CB;          // 1 KB fragments per k step: CB of weights, then FM of activations
  constexpr int RING = R * E * 1024;  // bytes per wave
  constexpr int NAG = 16;             // accumulator blocks kept in AGPRs, the rest in VGPRs
  constexpr int QS = 260;             // floats per quad of the staged tile (256 and a pad of 4)
  constexpr int RB = FM < 9 / CB ? FM : 9 / CB;  // row blocks per round of the final sum
  constexpr int WS = RB * CB * 4 * QS;           // floats parked by a wave in a round
  constexpr int T_BYTES = 4 * WS * 4;
  static_assert(4 * RING <= 160 * 1024 && T_BYTES <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char smem[4 * RING > T_BYTES ? 4 * RING : T_BYTES];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_blocks = (a.N + 31) >> 5, n_nt = (n_blocks + CB - 1) / CB;
  const int S = a.splits;
  const int t = xcd_remap(blockIdx.x, n_nt * S);
  const int nt = t % n_nt, sp = t / n_nt;
  const int units = a.Kp >> 6;  // of four k steps, one per wave
  const int ub = (int)((long)units * sp / S), n = (int)((long)units * (sp + 1) / S) - ub;

  // scalar base of every fragment stream, at this wave's first k step
  const char* src[E];
  static_for<0, E>([&](auto e) {
    constexpr int X = decltype(e)::value;
    if constexpr (X < CB)
      src[X] = (const char*)a.B + ((size_t)min(nt * CB + X, n_blocks - 1) * a.bstride + (size_t)(4 * ub + wave) * 512) * 2;
    else
      src[X] = (const char*)a.A + ((size_t)(X - CB) * a.astride + (size_t)(4 * ub + wave) * 512) * 2;
  });
  const unsigned voff = lane * 16;
  // activation rows past M repeat the last row: they feed output rows that are never stored, and
  // a step of a few rows then touches only the lines that hold them
  const unsigned avoff = FM == 1 ? (min(lane & 31, a.M - 1) + (lane & 32)) * 16 : voff;
  const unsigned ring0 = __builtin_amdgcn_readfirstlane(
      (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * RING);
  const char* ring = smem + wave * RING + lane * 16;
  auto dma = [&](auto e, int step, int slot) {
    const char* p = src[decltype(e)::value] + (size_t)step * 4096;
    const unsigned dst = ring0 + slot * (E * 1024) + decltype(e)::value * 1024;
    dma16(p, decltype(e)::value < CB ? voff : avoff, dst);
  };
  f32x16 acc[FM * CB];
  static_for<0, FM * CB>([&](auto b) { acc[b] = f32x16{}; });
  static_for<0, FM * CB>([&](auto b) { pin<(decltype(b)::value < NAG)>(acc[b]); });
  asm volatile("s_nop 7" ::: "memory");
  static_for<0, R>([&](auto s) {
    static_for<0, E>([&](auto e) { dma(e, min((int)decltype(s)::value, n - 1), s); });
  });
  auto frag = [&](int slot, int e) { return *(const bf16x8*)(ring + slot * (E * 1024) + e * 1024); };

  if constexpr (FM <= 5) {
    auto step = [&](auto wait_c, int i, int slot, auto more_c) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(wait_c)::value) : "memory");
      bf16x8 f[E];
      static_for<0, E>([&](auto e) { f[e] = frag(slot, e); });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(more_c)::value != 0) static_for<0, E>([&](auto e) { dma(e, i + R, slot); });
      static_for<0, FM>([&](auto r) {
        static_for<0, CB>([&](auto c) {
          constexpr int b = decltype(r)::value * CB + decltype(c)::value;
          mma<(b < NAG)>(acc[b], f[c], f[CB + decltype(r)::value]);
        });
      });
      __builtin_amdgcn_sched_barrier(0);
    };
    int i = 0, slot = 0;
    for (; i + R < n; ++i) {
      step(std::integral_constant<int, (R - 1) * E>{}, i, slot, std::integral_constant<int, 1>{});
      slot = slot + 1 == R ? 0 : slot + 1;
    }
    static_for<0, R>([&](auto u) {
      if (i < n) {
        step(std::integral_constant<int, (R - 1 - decltype(u)::value) * E>{}, i, slot, std::integral_constant<int, 0>{});
        slot = slot + 1 == R ? 0 : slot + 1;
        ++i;
      }
    });
  } else {
    constexpr int NA = FM % 3 == 0 ? 3 : FM % 4 == 0 ? 4 : FM;
    bf16x8 af[NA], bf[2][CB];
    // Reads run two row blocks ahead of the MFMAs.  DMAs are issued in ring order, so a fragment
    // has landed once at most as many are outstanding as were issued after it.  LEFT: steps in
    // flight after this one (R - 1 while DMAs go on, fewer in the tail).
    auto body = [&](auto par_c, int i, int slot, int nslot, auto more_c, auto left_c) {
      constexpr int PAR = decltype(par_c)::value;
      constexpr bool MORE = decltype(more_c)::value != 0;
      constexpr int LEFT = decltype(left_c)::value;
      static_for<0, FM>([&](auto r_c) {
        constexpr int r = decltype(r_c)::value;
        constexpr int done = MORE && r > 0 ? CB + r : 0;  // of step i + R, issued in this body so far
        if constexpr (r + 2 < FM) {
          constexpr int W = (FM - r - 3) + LEFT * E + done;
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(W < 63 ? W : 63) : "memory");
          af[(r + 2) % NA] = frag(slot, CB + r + 2);
        } else if constexpr (LEFT > 0) {
          constexpr int q = r + 2 - FM;  // row block q of the next step; its weights with q = 0
          constexpr int W = (FM - q - 1) + (LEFT - 1) * E + done;
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(W < 63 ? W : 63) : "memory");
          if constexpr (q == 0) static_for<0, CB>([&](auto c) { bf[PAR ^ 1][c] = frag(nslot, c); });
          af[q % NA] = frag(nslot, CB + q);
        }
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, CB>([&](auto c) {
          constexpr int b = r * CB + decltype(c)::value;
          mma<(b < NAG)>(acc[b], bf[PAR][c], af[r % NA]);
        });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE) {
          if constexpr (r == 0) static_for<0, CB>([&](auto c) { dma(c, i + R, slot); });
          dma(std::integral_constant<int, CB + r>{}, i + R, slot);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    // first fragments of step 0; an odd number of steps before the tail starts with one on the
    // second set of weight fragments, so that the loop and the tail start on the first
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, R - 1> left{};
    int slot = 0, i = 0;
    auto nxt = [&](int s) { return s + 1 == R ? 0 : s + 1; };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 1) * E + FM - 2) : "memory");
    af[0] = frag(0, CB);
    af[1] = frag(0, CB + 1);
    if ((n - R) & 1) {
      static_for<0, CB>([&](auto c) { bf[1][c] = frag(0, c); });
      body(c1, 0, 0, nxt(0), c1, left);
      slot = nxt(0);
      i = 1;
    } else {
      static_for<0, CB>([&](auto c) { bf[0][c] = frag(0, c); });
    }
    for (; i + R < n; i += 2) {
      const int s1 = nxt(slot), s2 = nxt(s1);
      body(c0, i, slot, s1, c1, left);
      body(c1, i + 1, s1, s2, c1, left);
      slot = s2;
    }
    static_for<0, R>([&](auto u) {
      const int ns = nxt(slot);
      body(std::integral_constant<int, decltype(u)::value & 1>{}, 0, slot, ns, c0,
           std::integral_constant<int, R - 1 - decltype(u)::value>{});
      slot = ns;
    });
  }

  // no load is in flight when the ring is reused, and the last MFMAs have written their
  // accumulators before anything else reads them
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  static_for<0, FM * CB>([&](auto b) { pin<(decltype(b)::value < NAG)>(acc[b]); });

  // ---- RB row blocks per round: every wave parks its sums (quad j of block b of the round at
  // [wave][b * 4 + j], lane-major), then each item adds the four waves' sums in wave order
  const int n0 = nt * CB * 32;
  float* T_ = (float*)smem;
  static_for<0, (FM + RB - 1) / RB>([&](auto p_c) {
    constexpr int R0 = decltype(p_c)::value * RB, NR = R0 + RB <= FM ? RB : FM - R0;
    __syncthreads();
    static_for<0, NR * CB>([&](auto b_c) {
      constexpr int b = decltype(b_c)::value;
      static_for<0, 4>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        f32x4 v;
        static_for<0, 4>([&](auto x) { v[decltype(x)::value] = acc[R0 * CB + b][4 * j + decltype(x)::value]; });
        *(f32x4*)(T_ + wave * WS + (b * 4 + j) * QS + lane * 4) = v;
      });
    });
    __syncthreads();
    // one item: 16 columns of a row (a pair group of the paired epilogues)
    for (int it = tid; it < NR * 32 * CB * 2; it += 256) {
      const int row = it / (CB * 2), g = it % (CB * 2);
      const int m = R0 * 32 + row, nc = n0 + g * 16;
      if (m >= a.M || nc >= a.N) continue;
      const float* q = T_ + (((row >> 5) * CB + (g >> 1)) * 4 + (g & 1) * 2) * QS + (row & 31) * 4;
      f32x4 u[4];
      u[0] = *(const f32x4*)q;
      u[1] = *(const f32x4*)(q + 128);
      u[2] = *(const f32x4*)(q + QS);
      u[3] = *(const f32x4*)(q + QS + 128);
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        u[0] += *(const f32x4*)(q + w * WS);
        u[1] += *(const f32x4*)(q + w * WS + 128);
        u[2] += *(const f32x4*)(q + w * WS + QS);
        u[3] += *(const f32x4*)(q + w * WS + QS + 128);
      }
      float v[16];
      __builtin_memcpy(v, u, sizeof(v));
      if (S > 1) {
        float* dst = a.partial + ((size_t)sp * a.M + m) * a.N + nc;
#pragma unroll
        for (int e = 0; e < 4; ++e) *(f32x4*)(dst + 4 * e) = u[e];
      } else if (epi == EPI_SWIGLU) {
        epi_group16<bf16, EPI_SWIGLU>(a, m, nc, v, v + 8);
      } else if (epi == EPI_QKV) {
        epi_group16<bf16, EPI_QKV>(a, m, nc, v, v + 8);
      } else if (epi == EPI_RESID) {
        epi_group8<bf16, EPI_RESID>(a, m, nc, v);
        epi_group8<bf16, EPI_RESID>(a, m, nc + 8, v + 8);
      } else if (epi == EPI_STORE) {
        epi_group8<bf16, EPI_STORE>(a, m, nc, v);
        epi_group8<bf16, EPI_STORE>(a, m, nc + 8, v + 8);
      } else {
        epi_group8<bf16, EPI_STORE_F32>(a, m, nc, v);
        epi_group8<bf16, EPI_STORE_F32>(a, m, nc + 8, v + 8);
      }
    }
  });
}

// Ring depth in k steps: 40 KB per wave.
constexpr int stream_ring(int fm, int cb) { return 40 / (fm + cb); }
// Column blocks of a tile: the accumulators of six row blocks leave registers for three.
constexpr int stream_max_cb(int fm) { return fm <= 5 ? 4 : 3; }

template <int FM, int CB>
static hipError_t stream_launch(int epi, const GemmArgs& a, hipStream_t s) {
  const dim3 grid((((a.N + 31) / 32 + CB - 1) / CB) * a.splits);
  hipLaunchKernelGGL((gemm_stream_kernel<FM, CB, stream_ring(FM, CB)>), grid, dim3(256), 0, s, a, epi);
  return hipGetLastError();
}

template <int FM>
static hipError_t stream_launch_cb(int cb, int epi, const GemmArgs& a, hipStream_t s) {
  switch (cb) {
    case 1: return stream_launch<FM, 1>(epi, a, s);
    case 2: return stream_launch<FM, 2>(epi, a, s);
    case 3: return stream_launch<FM, 3>(epi, a, s);
    default: return stream_launch<FM, stream_max_cb(FM)>(epi, a, s);
  }
}

// Whether the streaming plan p (wg workgroups) is taken, against the tiles that split K over
// workgroups only.  Both were timed over every plan of ten model shapes (d 512 to 8192) and of LM
// heads of 4096 to 128256 columns, these with cached weights and with weights that others had
// displaced; where the lines lie, us tiles -> streamed:
//  - It pays where the tiles' workgroups are few or their splits many: 64 rows, gate/up of the 7B
//    shape 48.0 -> 38.1; 192 rows, N 5632, K 1024 24.9 -> 11.8.
//  - An LM head of which the tiles fill the GPU unsplit: 96 rows, N 32000, 13.2 -> 15.9 at K 512 and
//    26.9 -> 29.8 at K 2048 (cached), 90.5 -> 93.4 at K 4096 (displaced).  Storing a tile's fp32
//    logits and adding the waves' sums cost the same at any K, so only long K pays, the longer the
//    more row blocks (64 rows, K 4096, with norm and argmax 61.7 -> 60.8; 128 rows, K 8192
//    149.3 -> 146.2), and with one row block none.  Where the tiles leave a third of the GPU idle, on
//    96-column tiles, from K 1024 on (N 22016: 64 rows, K 1024, with norm and argmax 28.2 -> 26.2;
//    96 rows, K 5120 83.2 -> 80.1).
//    Split heads on 128-column tiles: 128 rows, N 8192, K 4096 35.7 -> 39.5.
//  - 128-column streamed tiles share less than the tiles of that width do.  Split more than two ways
//    they pay over long K only (96 rows, N 8192: K 28672 97.8 -> 91.7, K 8192 42.0 -> 46.9), and with
//    fewer workgroups than the tiles not at all (160 rows, N 5120, K 13824 51.0 -> 53.6).
//  - Six row blocks: a tile of at most 96 columns.  Two passes of it for one of the tiles': N 27648,
//    K 5120 84.6 -> 103.6, LM head N 32000, K 4096 71.6 -> 89.4.  Split ones are no faster than the
//    160-row tiles (a layer of d 3072 with O streamed 128.1 -> 129.8); narrow ones are (N 11008, K 2048
//    30.4 -> 26.2), wide ones over long K (a 7B layer of 192 rows with gate/up streamed 179.5 -> 177.5,
//    N 24576, K 8192 123.5 -> 117.4), and split ones against the 224-row tiles unless their workgroups
//    are fewer (N 6144, K 2048 29.3 -> 26.6; d 6144, 192 rows, down 70.1 -> 66.8; d 5120 53.7 -> 56.5)
//    or two column blocks go over long K (K 8192 56.5 -> 58.9).
//  - Short K: the waves' sums outweigh it.  Tiles that fill the GPU unsplit: 160 rows, N 27648, K 512
//    16.6 -> 20.3, K 2048 36.1 -> 37.5; N 22016, K 512 15.4 -> 17.5 (64 rows 12.5 -> 11.6).  One row
//    block at K 256, where a wave has four steps of a ring of up to twenty: N 768 6.3 -> 6.9; before a
//    residual also at K up to 1536, where the tiles' split sums are added in the norm that follows (a
//    layer of d 1024, 16 rows, with O streamed 37.9 -> 38.6; of d 512, one row, with down 31.0 -> 32.1).
static bool stream_pays(const StreamPlan& p, int wg, int Kp, int epi, const TilePlan& tiles) {
  const bool full = tiles.splits == 1 && tiles.wg >= 160;  // the tiles fill the GPU unsplit
  if (p.fm == 1 && Kp <= (epi == EPI_RESID ? 1536 : 256)) return false;
  if (epi == EPI_STORE_F32) {
    if (full && p.cb == 3 && p.fm < 6 && tiles.wg < 180) return Kp >= (p.fm <= 3 ? 1024 : 2048);
    if (full) return p.fm > 1 && p.fm < 6 && Kp >= (p.cb == 3 || p.fm == 3 ? 5120 : p.fm == 2 ? 4096 : 8192);
    if (p.cb == 4) return false;
  }
  if (p.fm == 6) {
    if (wg > 256) return false;
    if (p.splits == 1) return p.cb == 1 || (p.cb == 2 ? Kp <= 6144 : Kp >= 4096);
    return p.cb == 1 || (tiles.fm == 7 && (p.cb == 2 ? Kp <= 3072 : wg >= tiles.wg));
  }
  // one row block, 128 columns, unsplit: the tile's waves share the activations and it is 1 % faster
  // (61.5 against 62.1 us for the LM head of 7 rows with its norm and argmax)
  if (p.fm == 1 && p.cb == 4 && p.splits == 1) return false;
  if (full && Kp < (p.cb == 4 ? 3072 : p.fm > 3 ? 1536 : 512)) return false;
  if (p.cb >= 3 && p.splits > 2 && wg < tiles.wg) return false;
  return !(p.cb == 4 && p.splits > 2 && Kp / p.splits < 4096);
}

// Tile width and K splits for up to STREAM_MAX_M rows: the plan of the least estimate (us) of 4 per
// pass of 256 workgroups, the fragments a workgroup loads at 55 GB/s per CU, not less than the
// weights at 6.2 TB/s, and for a split the fp32 sums written at 4 TB/s and the reduction that
// follows (2 more than the norm it is fused with after the residual projections, else 5).  The
// estimate only ranks streaming plans: 55 GB/s is what weights and activations reach at best, with
// both in flight a CU loads 37 to 46, so gate/up of the 7B shape at 135 rows is put at 42 us and
// takes 55.  Against the best of all plans the ranking loses 1 to 2 % over the ten shapes.
// Equal costs go to the plan with more workgroups, then to the wider tile.  The tiles' splits bound
// the fp32 sums: a caller's fixed scratch then holds every step that it held with those tiles.  No
// plan of the 7B shape is held back by it.
bool stream_plan(int M, int N, int Kp, int epi, const TilePlan& tiles, StreamPlan* p) {
  if (M > STREAM_MAX_M) return false;
  const int fm = (M + 31) / 32, nb = (N + 31) / 32, units = Kp / 64;
  double best = 0;
  int best_wg = 0;
  p->fm = 0;
  for (int cb = 1; cb <= stream_max_cb(fm); ++cb)
    for (int S : {1, 2, 3, 4, 6, 8}) {
      if (S > tiles.splits) break;
      if (S > 4 && cb > 1) continue;  // short K ranges: a tile's prologue and sum weigh too much
      if (units / S < (S > 1 ? 8 : fm > 5 ? stream_ring(fm, cb) : 1)) continue;
      const int wg = (nb + cb - 1) / cb * S, passes = (wg + 255) / 256;
      double us = std::max(passes * (fm + cb) * (Kp * 64.0 / S) / 55e3, (double)N * Kp * 2 / 6.2e6) + 4 * passes;
      if (S > 1) us += (double)S * M * N / 1e6 + (epi == EPI_RESID ? 2 : 5) + 0.25 * S;
      if (!p->fm || us < best - 1e-6 || (us < best + 1e-6 && wg >= best_wg)) {
        *p = {fm, cb, S};
        best = us;
        best_wg = wg;
      }
    }
  return p->fm > 0 && stream_pays(*p, best_wg, Kp, epi, tiles);
}

hipError_t launch_gemm_stream(const StreamPlan& p, int epi, const GemmArgs& a, hipStream_t s) {
  // the kernel reads exactly fm row blocks, and from six on at least a full ring of k steps
  if (p.fm != (a.M + 31) / 32 || p.cb < 1 || p.cb > stream_max_cb(p.fm) || p.splits != a.splits || a.col0 != 0 ||
      a.Kp / 64 / a.splits < (p.fm > 5 ? stream_ring(p.fm, p.cb) : 1))
    return hipErrorInvalidValue;
  switch (p.fm) {
    case 1: return stream_launch_cb<1>(p.cb, epi, a, s);
    case 2: return stream_launch_cb<2>(p.cb, epi, a, s);
    case 3: return stream_launch_cb<3>(p.cb, epi, a, s);
    case 4: return stream_launch_cb<4>(p.cb, epi, a, s);
    case 5: return stream_launch_cb<5>(p.cb, epi, a, s);
    case 6: return stream_launch_cb<6>(p.cb, epi, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace af
