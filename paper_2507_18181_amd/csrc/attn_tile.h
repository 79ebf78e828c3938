// One wavefront's part of tree attention: a tile of 32 keys x 32 queries on bf16 MFMA (kernels_attn.hip says why it is like this).
#pragma once
#include "common.h"

namespace specasr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

// The K operands of a tile (16-byte LDS reads) with their wait, and transposing LDS reads with theirs.  As assembly, because for ordinary LDS reads the compiler waits for every direct-to-LDS load in
// flight, those of the other buffer among them.  Transposing read: 16 lanes give the addresses of 4 rows x 16 columns (8 bytes
// each) and get 4 rows of one column each.
template <int N>
__device__ __forceinline__ void read_k(u32x4 (&k)[N], const uint32_t (&a)[N]) {
  if constexpr (N == 8)
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                 "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3]), "=&v"(k[4]), "=&v"(k[5]), "=&v"(k[6]), "=&v"(k[7])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]) : "memory");
  else
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3]) : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]) : "memory");
}
// V^T quads of (cb, part) = 0 .. N-1 for the keys OFF / row size .. +15 of the tile
template <int N, int OFF>
__device__ __forceinline__ void read_v(u32x2 (&v)[N], const uint32_t (&a)[N]) {
  if constexpr (N == 8)
    asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%16\n\tds_read_b64_tr_b16 %1, %9 offset:%16\n\tds_read_b64_tr_b16 %2, %10 offset:%16\n\tds_read_b64_tr_b16 %3, %11 offset:%16\n\t"
                 "ds_read_b64_tr_b16 %4, %12 offset:%16\n\tds_read_b64_tr_b16 %5, %13 offset:%16\n\tds_read_b64_tr_b16 %6, %14 offset:%16\n\tds_read_b64_tr_b16 %7, %15 offset:%16\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "i"(OFF) : "memory");
  else
    asm volatile("ds_read_b64_tr_b16 %0, %4 offset:%8\n\tds_read_b64_tr_b16 %1, %5 offset:%8\n\tds_read_b64_tr_b16 %2, %6 offset:%8\n\tds_read_b64_tr_b16 %3, %7 offset:%8\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "i"(OFF) : "memory");
}

// a / b with inv = 1 / b: the residual of the product corrects it, 3 instructions for the 10 of a division (one tile
// per wavefront, 1.1B: 6.5 -> 6.4 us)
__device__ __forceinline__ float div_by(float a, float b, float inv) {
  const float q = a * inv;
  return fmaf(fmaf(-b, q, a), inv, q);
}
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
// maximum / sum of a value over lanes l and l ^ 32
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// 16 bytes per lane to 64 consecutive places.  Direct copies are only defined for aligned addresses; a cache that is not
// on 16 bytes (a caller's slice of a larger tensor) goes through registers.
template <bool DIRECT>
__device__ __forceinline__ void load_16_to_lds(const char *src_lane, u32x4 *dst_64, int lane) {
  if constexpr (!DIRECT) {
    u32x4 v;
    __builtin_memcpy(&v, src_lane, 16);
    dst_64[lane] = v;
    return;
  }
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src_lane, (void __attribute__((address_space(3))) *)dst_64, 16, 0, 0);
}

// Chunk (16 bytes) c of row r of a tile sits at chunk c ^ swizzle(r) of that row.
template <int HD>
__device__ __forceinline__ int swizzle(int r) {
  return HD == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}

// A 32 x 32 tile of scores and outputs of one wavefront: query ql = lane % 32 in the columns, keys (rows) split over the two halves.
template <int HD>
struct TileState {
  static constexpr int KK = HD / 16;  // MFMA k-steps across the head dimension
  static constexpr int CB = HD / 32;  // 32-wide output column blocks
  static constexpr int CR = HD / 8;   // 16-byte chunks of a row
  float m_run, l_run;                 // l_run: this lane's keys only, the halves are added at the end
  f32x16 o[CB], sT;
  uint32_t ka[KK], va[2 * CB];        // LDS addresses of the operands
  u32x4 pb[2], pl[2];

  // K and V tiles of the wavefront in LDS.  K: row ql, chunk 2 kk + h.  V^T of (mm, part, cb): lane i of a group of
  // 16 addresses row 16 mm + 8 part + 4 h + i/4, columns 32 cb + 16 (group & 1) + 4 (i%4).
  __device__ __forceinline__ void init(u32x4 *kb, u32x4 *vb, int lane) {
    const int h = lane >> 5, ql = lane & 31;
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[cb][j] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) ka[kk] = (uint32_t)(uintptr_t)(lds_u32x4 *)(kb + ql * CR + (h ^ swizzle<HD>(ql) ^ (2 * kk)));
    const int vi = lane & 15, vrow = 4 * h + (vi >> 2);
    const int vx = (2 * ((lane >> 4) & 1) + ((vi & 3) >> 1)) ^ swizzle<HD>(vrow);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int part = 0; part < 2; ++part)  // LDS byte address of (cb, part); mm adds 16 rows
        va[2 * cb + part] = (uint32_t)(uintptr_t)(lds_u32x4 *)(vb + (vrow + 8 * part) * CR + (vx ^ (4 * cb) ^ (2 * part))) + (vi & 1) * 8;
  }
  // S^T of the tile whose K is in LDS (the reads have returned where this ends: the buffer is free then)
  __device__ __forceinline__ void scores(const u32x4 (&qh)[KK], const u32x4 (&qlo)[KK]) {
#pragma unroll
    for (int j = 0; j < 16; ++j) sT[j] = 0.f;
    u32x4 kreg[KK];
    read_k(kreg, ka);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      sT = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kreg[kk]), __builtin_bit_cast(bf16x8, qlo[kk]), sT, 0, 0, 0);
      sT = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kreg[kk]), __builtin_bit_cast(bf16x8, qh[kk]), sT, 0, 0, 0);
    }
  }
  // bit i of w: key i of the tile is visible.  A lane holds, for query ql, the keys 8*(j/4) + 4*h + j%4
  __device__ __forceinline__ void mask(uint32_t w, int h) {
    w >>= 4 * h;
#pragma unroll
    for (int j = 0; j < 16; ++j) sT[j] = (w >> (8 * (j >> 2) + (j & 3))) & 1u ? sT[j] : -INFINITY;
  }
  __device__ __forceinline__ void softmax() {
    float mx = sT[0];
#pragma unroll
    for (int j = 1; j < 16; ++j) mx = fmaxf(mx, sT[j]);
    mx = max_halves(mx);
    // The running maximum itself is subtracted: the largest probability is 1, exact in two bf16 planes.  (A
    // reference that may lag by 2^8 saves rescaling but rounds that probability as well: attention output 2 .. 5 %
    // further from the 64-bit result over 1 .. 1024 rows of the 1.1B, 7B and 13B shapes, at the same times: 7B 64
    // nodes 4.74 / 4.75 ms, prefill of 810 23.84 / 23.89 ms.)
    const bool grow = mx > m_run;  // also at the first visible key (m_run = -inf)
    if (__ballot(grow) != 0ull) {
      const float m_new = grow ? mx : m_run;
      const float alpha = grow ? exp2_fast(m_run - m_new) : 1.f;
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[cb][j] *= alpha;
    }
    // a query that has seen no key yet subtracts 0: its scores stay -inf and give probability 0
    const float m_sub = m_run == -INFINITY ? 0.f : m_run;
    float p[16], ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      p[j] = exp2_fast(sT[j] - m_sub);
      ps[j & 3] += p[j];
    }
    l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
    // P^T as B operand: MFMA mm covers keys 16*mm .. 16*mm+15 of the tile; this lane's k-slots
    // i = 0..7 are keys 16*mm + 8*(i/4) + 4*h + i%4, i.e. its own p[8*mm + i]
#pragma unroll
    for (int mm = 0; mm < 2; ++mm)
#pragma unroll
      for (int i2 = 0; i2 < 4; ++i2) {
        uint32_t hi2, lo2;
        split_bf16_pair(p[8 * mm + 2 * i2], p[8 * mm + 2 * i2 + 1], hi2, lo2);
        pb[mm][i2] = hi2;
        pl[mm][i2] = lo2;
      }
  }
  // O^T += V^T * P^T of the tile whose V is in LDS
  __device__ __forceinline__ void values() {
    auto pv = [&](const u32x2 (&v)[2 * CB], int mm) {
#pragma unroll
      for (int pass = 0; pass < 2; ++pass)  // lo products, then hi: CB independent accumulators in between
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const u32x4 vv = (u32x4){v[2 * cb][0], v[2 * cb][1], v[2 * cb + 1][0], v[2 * cb + 1][1]};
          o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv), __builtin_bit_cast(bf16x8, pass ? pb[mm] : pl[mm]), o[cb], 0, 0, 0);
        }
    };
    u32x2 v0[2 * CB], v1[2 * CB];
    read_v<2 * CB, 0>(v0, va);
    pv(v0, 0);
    read_v<2 * CB, 16 * HD * 2>(v1, va);
    pv(v1, 1);
  }
};

}  // namespace specasr
