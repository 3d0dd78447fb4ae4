// The step that follows a projection's sums, fused into the GEMM that makes them: plain stores,
// residual add, SwiGLU, and rotary embedding with the ring write.  Shared by every GEMM kernel.
#pragma once

#include "af_device.h"

namespace af {

template <typename T, int EPI>
__device__ __forceinline__ void epi_single(const GemmArgs& a, int m, int n, float v) {
  n += a.col0;
  if constexpr (EPI == EPI_STORE) {
    ((T*)a.out)[(size_t)m * a.ldo + n] = from_f<T>(v);
  } else if constexpr (EPI == EPI_STORE_F32) {
    ((float*)a.out)[(size_t)m * a.ldo + n] = v;
  } else {  // EPI_RESID (out may alias resid: each element is read and written by one thread)
    const float r = to_f(((const T*)a.resid)[(size_t)m * a.ldr + n]);
    ((T*)a.out)[(size_t)m * a.ldo + n] = from_f<T>(r + v);
  }
}

// Paired epilogues: each 16-column block holds 8 a-columns followed by their 8 partners
// (weights repacked that way); c is the a-column, va/vb the pair.
template <typename T, int EPI>
__device__ __forceinline__ void epi_pair(const GemmArgs& a, int m, int c, float va, float vb) {
  c += a.col0;
  if constexpr (EPI == EPI_SWIGLU) {
    const int f = (c >> 4) * 8 + (c & 7);
    const float s = va / (1.0f + __expf(-va));
    const size_t o = a.ostride > 0 ? frag_off(m, f, a.ostride) : (size_t)m * a.ldo + f;
    ((T*)a.out)[o] = from_f<T>(s * vb);
  } else {  // EPI_QKV
    const int D = a.d_model, hd = a.head_dim, half = hd >> 1;
    const int region = c / D, cr = c - region * D;
    const int h = cr / hd, jj = cr - h * hd;
    const int dj = (jj >> 4) * 8 + (jj & 7);  // rotary pair (dj, dj + hd/2)
    const int slot = a.row_sp[2 * m], pos = a.row_sp[2 * m + 1];
    if (region == 2) {
      T* dst = (T*)a.ring_v + (((size_t)slot * a.n_heads + h) * a.max_pos + pos) * hd;
      dst[dj] = from_f<T>(va);
      dst[dj + half] = from_f<T>(vb);
    } else {
      const float cs = a.rope_cs[((size_t)pos * half + dj) * 2];
      const float sn = a.rope_cs[((size_t)pos * half + dj) * 2 + 1];
      const float ra = fmaf(va, cs, -(vb * sn)), rb = fmaf(vb, cs, va * sn);  // as epi_group16
      T* dst = region == 0 ? (T*)a.out + (size_t)m * a.ldo + h * hd
                           : (T*)a.ring_k + (((size_t)slot * a.n_heads + h) * a.max_pos + pos) * hd;
      dst[dj] = from_f<T>(ra);
      dst[dj + half] = from_f<T>(rb);
    }
  }
}

// Columns nc .. nc+7 (nc % 8 == 0) of row m.
template <typename T, int EPI>
__device__ __forceinline__ void epi_group8(const GemmArgs& a, int m, int nc, const float* v) {
  nc += a.col0;
  if constexpr (EPI == EPI_STORE_F32) {
    store8<float>((float*)a.out + (size_t)m * a.ldo + nc, v);
  } else {
    T r[8];
    if constexpr (EPI == EPI_RESID) {  // out may alias resid: each element is read, then written, by one thread
      T res[8];
      load8<T>((const T*)a.resid + (size_t)m * a.ldr + nc, res);
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = from_f<T>(to_f(res[e]) + v[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = from_f<T>(v[e]);
    }
    store8<T>((T*)a.out + (size_t)m * a.ldo + nc, r);
  }
}

// What the QKV epilogue needs besides the sums for one 16-column group of row m: the region
// (queries, keys, values), head, rotary offset, the row's ring slot and position, and the
// rotary (cos, sin) pairs; loaded ahead of the sums where the sums come from memory.
struct QkvRow {
  int region, h, dj, slot, pos;
  float cs[16];
  __device__ __forceinline__ void load(const GemmArgs& a, int m, int c) {
    const int D = a.d_model, hd = a.head_dim, half = hd >> 1;
    c += a.col0;
    region = c / D;
    const int cr = c - region * D;
    h = cr / hd;
    dj = ((cr - h * hd) >> 4) * 8;
    slot = a.row_sp[2 * m];
    pos = a.row_sp[2 * m + 1];
    if (region != 2) {
      load8<float>(a.rope_cs + ((size_t)pos * half + dj) * 2, cs);
      load8<float>(a.rope_cs + ((size_t)pos * half + dj) * 2 + 8, cs + 8);
    }
  }
};

// The 16-column group starting at c (c % 16 == 0): a-columns c .. c+7, partners c+8 .. c+15.
template <typename T, int EPI>
__device__ __forceinline__ void epi_group16(const GemmArgs& a, int m, int c, const float* va, const float* vb,
                                            const QkvRow* pre = nullptr) {
  T r0[8], r1[8];
  if constexpr (EPI == EPI_SWIGLU) {
    const int f = ((c + a.col0) >> 4) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) r0[e] = from_f<T>(va[e] / (1.0f + __expf(-va[e])) * vb[e]);
    store8<T>((T*)a.out + (a.ostride > 0 ? frag_off(m, f, a.ostride) : (size_t)m * a.ldo + f), r0);
  } else {  // EPI_QKV: rotary pairs (dj + e, dj + e + hd/2), e < 8
    QkvRow q;
    if (pre) q = *pre;
    else q.load(a, m, c);
    const int hd = a.head_dim, half = hd >> 1;
    T* dst;
    if (q.region == 2) {
      dst = (T*)a.ring_v + (((size_t)q.slot * a.n_heads + q.h) * a.max_pos + q.pos) * hd;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        r0[e] = from_f<T>(va[e]);
        r1[e] = from_f<T>(vb[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // explicit fused multiply-adds: every kernel that applies this epilogue rounds alike
        r0[e] = from_f<T>(fmaf(va[e], q.cs[2 * e], -(vb[e] * q.cs[2 * e + 1])));
        r1[e] = from_f<T>(fmaf(vb[e], q.cs[2 * e], va[e] * q.cs[2 * e + 1]));
      }
      dst = q.region == 0 ? (T*)a.out + (size_t)m * a.ldo + q.h * hd
                          : (T*)a.ring_k + (((size_t)q.slot * a.n_heads + q.h) * a.max_pos + q.pos) * hd;
    }
    store8<T>(dst + q.dj, r0);
    store8<T>(dst + q.dj + half, r1);
  }
}

}  // namespace af
