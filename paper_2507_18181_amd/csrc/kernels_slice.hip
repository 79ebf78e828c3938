// Unsplit skinny GEMMs that finish their own output (rows <= 64), for gfx950.
//
// The split-k skinny GEMM (kernels_mfma.hip) spreads k over workgroups and leaves fp32 partial sums
// that a finishing kernel adds up; per projection that is 4 .. 8 output-sized buffers written and
// read again plus a dependent launch of about 4 us.  Here a workgroup owns WHOLE k for a few output
// features, so its epilogue is the finishing kernel:
//   * One workgroup = HB half-bands of 16 output features x all rows (NC groups of 16), 8 wavefronts,
//     each with an eighth of k.  A half-band is what makes this balance: 7B gate|up has 1376 of
//     them, 5.4 per compute unit (whole bands: 2.7, i.e. 3), q|k|v exactly 3.
//   * v_mfma_f32_16x16x32_bf16; both operands are read in the layouts the split kernel uses (a pair
//     of its k-step tiles is one operand: lane l takes k-step l/32, k-half (l/16)%2, row l%16), so
//     nothing is stored twice.  Weights and activations stream together through a ring of D
//     register stages: no LDS, no barrier before the epilogue, 128 .. 320 KB in flight per compute unit.
//   * What bounds it: the weight stream while HB >= NC, the bytes one compute unit can pull out of
//     its L2 beside that stream (about 60 bytes/ns together; activations alone come at 110 .. 134) where activations outweigh
//     weights (few features per workgroup).
//   * The 8 slices are summed through LDS; the summing thread applies the finishing step.
// Measured (us per launch under the tracer, split kernel + its finishing kernel against this one): 7B, 32 rows
// gate|up 33.6 + 5.4 -> 33.4, q|k|v 18.9 + 4.7 -> 23.2; 13B gate|up 51.6 + 6.2 -> 48.5, q|k|v 32.8 + 5.7 -> 33.2; 1.1B,
// 16 rows gate|up 11.6 + 4.3 -> 11.5 .. 11.9, q|k|v 5.8 + 4.0 -> 7.1, o 4.9 + 3.9 -> 6.1 .. 6.5.
#include <hip/hip_ext.h>

#include "kernels.h"
#include "kernels_mfma.h"
#include "kernels_slice.h"

namespace specasr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kSliceWaves = 8;

// Register stages of the ring: 8, 4 or 2, as many as fit
// 250 registers next to the accumulators (a spill costs more than a stage gives: 7B gate|up 33.3 us
// with 2 .. 3 stages, 41 with 4 and 80 bytes spilled).  Powers of two, because a wavefront's slice is 8 k-step
// pairs on a 2048-wide model and 16 on a 4096-wide one: with 6 stages the last, partial block cost
// 2 us (1.1B gate|up 10.3 us with 4, 11.9 with 6, 9.9 with 8).
template <int EPI, int HB, int NC>
constexpr int slice_regs(int stages, int accs) {
  constexpr int xo = NC ? 2 * NC : 1, tc = NC ? NC : 1;  // operands of a stage, tiles per half-band
  return stages * 4 * (HB + xo) + 4 * HB * tc * accs + 2 * HB + (EPI == kSliceQkv ? 60 : 48);
}
template <int EPI, int HB, int NC>
constexpr int slice_depth() {
  // Both planes in one operand (NC = 0): the ring of 16 rows, though a deeper one would fit, so that two accumulators always
  // do and the chains get no longer (below).
  if (NC == 0 && EPI != kSliceQkv) return slice_depth<EPI, HB, 1>();
  constexpr int accs = EPI == kSliceQkv ? 3 : 1;
  return slice_regs<EPI, HB, NC>(8, accs) <= 250 ? 8 : slice_regs<EPI, HB, NC>(4, accs) <= 250 ? 4 : 2;
}
// Accumulators per tile: what rounds is mostly the fp32 addition chain, one step per 8 products, so it is
// cut: 2 = the running products of a few stages, then added to the sum; 3 = lo products apart as well.
// Always 3 for q|k|v: its rounding flips K and V elements, and what is wrong in the first layer's travels through
// all layers (bf16 elements of layer 0's K and V rows that differ from the 64-bit result, 7B / 13B with 32 rows, mean of
// 64 seeds: 35.2 / 48.3 with one chain of half the length for hi, 30.6 / 39.2 now, 30.9 / 39.6 with the split kernel).
// Elsewhere as many as fit without giving up a stage.
template <int EPI, int HB, int NC>
constexpr int slice_accs() {
  constexpr int D = slice_depth<EPI, HB, NC>();
  // Both planes in one operand: lo products have columns of their own; q|k|v with a ring of 8: both halves of a block and the sum.
  // With the ring as deep as it fits, gate|up of 16384 features ran in one chain and the 13B down projection in two of half a
  // slice: rms errors of the sums 2.04 / 2.04 units of 2^-24, with 16 rows' instances 1.30 / 1.65, now 1.24 / 1.64; times equal
  // (10 layers, 8 rows: 13B 1442 us / 1425, 16384 features 1236 / 1222).
  if constexpr (NC == 0) {
    static_assert(EPI == kSliceQkv || slice_regs<EPI, HB, NC>(D, 2) <= 250, "blocks of D steps and their sum");
    return EPI == kSliceQkv && D == 8 ? 3 : 2;
  }
  return EPI == kSliceQkv || slice_regs<EPI, HB, NC>(D, 3) <= 250 ? 3 : slice_regs<EPI, HB, NC>(D, 2) <= 250 ? 2 : 1;
}
// Output tiles summed through LDS at a time (1 KB per tile and wavefront, at most 128 KB).
template <int HB, int NC>
constexpr int slice_chunk() { constexpr int n = HB * (NC ? NC : 1); return n <= 16 ? n : (n + 1) / 2; }

// grid = 8 * ceil(tiles * S / 8): an XCD (workgroup index mod 8) owns a contiguous run of tiles, so
// its L2 sees every k-range of them.  block = 512.
template <int EPI, int HB, int NCP>
__global__ __launch_bounds__(kSliceWaves * 64, 2) void gemm_slice_kernel(SliceArgs p) {
  extern __shared__ float4 lds_slice[];
  __shared__ float rms[64];
  constexpr bool BOTH = NCP == 0;  // both planes of 8 rows in one operand
  constexpr int NC = BOTH ? 1 : NCP, NP = BOTH ? 1 : 2, RW = BOTH ? 1 : 2 * NC;  // row groups, operands per group, rows per wavefront in the norm
  constexpr int NW = kSliceWaves, D = slice_depth<EPI, HB, NCP>(), nb = NC <= 2 ? 1 : 2, NT = HB * NC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int slot = blockIdx.x >> 3, id = (blockIdx.x & 7) * p.per_xcd + slot;
  if (slot >= p.per_xcd || id >= p.total) return;
  // tile and k-chunk (only the partial-sum epilogue may be split: integer divisions are long code here)
  const uint32_t S = EPI == kSlicePartial ? p.S : 1, s = EPI == kSlicePartial ? (uint32_t)id % S : 0, nt = EPI == kSlicePartial ? (uint32_t)id / S : id;
  const uint32_t kp = (uint32_t)p.ksteps / 2, c0 = kp * s / S, c1 = kp * (s + 1) / S;
  const int w0 = c0 + (c1 - c0) * wave / NW, len = (int)(c0 + (c1 - c0) * (wave + 1) / NW) - w0;

  // What the epilogue needs besides the sums is requested first: it arrives while the ring fills.
  float ss[8];  // this wavefront's rows wave, wave + 8, ...: one lane's share of the slab sums of squares
  if (EPI == kSliceSwiglu || EPI == kSliceQkv) {
#pragma unroll
    for (int i = 0; i < RW; ++i) ss[i] = row_ssq_lane(p.nrm, min(wave + 8 * i, p.rows - 1));
  }
  // item of this thread in the residual epilogue (one per thread: HB * NC <= 8)
  const int rt = threadIdx.x >> 6;
  const int r_row = (rt % NC) * 16 + (lane & 15), r_hb = nt * HB + rt / NC, r_col = r_hb * 16 + (lane >> 4) * 4;
  const bool r_ok = rt < NT && r_row < p.rows && r_hb < p.n_half && r_col < p.d;
  float4 r_x = make_float4(0.f, 0.f, 0.f, 0.f);
  uint2 r_g = make_uint2(0u, 0u);
  if (EPI == kSliceResid && r_ok) {
    r_x = *reinterpret_cast<const float4 *>(p.x + (int64_t)r_row * p.d + r_col);
    r_g = *reinterpret_cast<const uint2 *>(p.gain + r_col);
  }
  // item of this thread in the q|k|v epilogue: node, 4 rotary pairs (first halves in quad q_qd, second
  // halves in quad q_qd + 2 of the half-band)
  const int q_t = threadIdx.x >> 5, q_qd = (threadIdx.x >> 4) & 1;
  const int q_row = (q_t % NC) * 16 + (threadIdx.x & 15), q_hb = nt * HB + q_t / NC;
  int q_kind = -1, q_head = 0, q_j = 0;  // 0 query, 1 key, 2 value
  float4 q_cs01 = make_float4(1.f, 0.f, 1.f, 0.f), q_cs23 = q_cs01;
  int64_t q_cache = 0;
  if (EPI == kSliceQkv && q_t < NT && q_row < p.rows && q_hb < p.n_half) {
    const int col = q_hb * 16, dq = p.H * p.hd, dkv = p.Hkv * p.hd;
    int c = col;
    if (col < dq) q_kind = 0;
    else if (col >= p.col_k && col - p.col_k < dkv) { q_kind = 1; c = col - p.col_k; }
    else if (col >= p.col_v && col - p.col_v < dkv) { q_kind = 2; c = col - p.col_v; }
    if (q_kind >= 0) {
      q_head = c >> p.hd_shift;
      const int in_head = c - (q_head << p.hd_shift);
      q_j = (q_kind == 2 ? in_head : in_head / 2) + 4 * q_qd;
      if (q_kind < 2) {
        const float4 *csp = reinterpret_cast<const float4 *>(p.cs + (int64_t)q_row * (p.hd / 2) + q_j);
        q_cs01 = csp[0];
        q_cs23 = csp[1];
      }
      if (q_kind > 0) q_cache = p.g.row(p.m.seq_of_row(q_row), p.layer, q_head, p.m.slot[q_row]);
    }
  }

  const int in_tile = 32 * ((lane >> 4) & 1) + (lane & 15);
  const u32x4 *wp[HB];
#pragma unroll
  for (int a = 0; a < HB; ++a) {
    const int hb = min(nt * HB + a, p.n_half - 1);  // half-bands past the matrix edge repeat the last one, unused
    wp[a] = (const u32x4 *)p.W + ((int64_t)(hb >> 1) * p.ksteps + 2 * w0 + (lane >> 5)) * 64 + in_tile + 16 * (hb & 1);
  }
  const int64_t plane = (int64_t)p.ksteps * nb * 64;
  const u32x4 *xp = (const u32x4 *)p.X + (int64_t)(2 * w0 + (lane >> 5)) * nb * 64 + in_tile;
  if (BOTH && (lane & 8)) xp += plane - 8;  // operand rows 8 .. 15 are the lo plane of rows 0 .. 7
  // accumulators: 0 running products, 1 what they were after earlier blocks of D stages (D = 8: the products of the
  // block's second half instead, no additions in the loop), 2 lo products (with NA < 3 they go with the hi ones).
  // BOTH: lo products have columns of their own in all of them; 2 (q|k|v, D = 8) is the sum of both halves of earlier blocks.
  constexpr int NA = slice_accs<EPI, HB, NCP>();
  f32x4 acc[HB][NC][NA];
#pragma unroll
  for (int a = 0; a < HB; ++a)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = 0; i < NA; ++i) acc[a][c][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  u32x4 wa[D][HB], xb[D][NP][NC];
  auto load = [&](int j, int k) {
#pragma unroll
    for (int a = 0; a < HB; ++a) wa[j][a] = __builtin_nontemporal_load(wp[a] + (int64_t)k * 128);
#pragma unroll
    for (int h = 0; h < NP; ++h)
#pragma unroll
      for (int c = 0; c < NC; ++c) xb[j][h][c] = xp[h * plane + (int64_t)k * nb * 128 + (c >> 1) * 64 + (c & 1) * 16];
  };
  auto mul = [&](int j) {
#pragma unroll
    for (int h = 0; h < NP; ++h)
#pragma unroll
      for (int a = 0; a < HB; ++a)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          f32x4 &z = acc[a][c][!BOTH && NA == 3 && h ? 2 : NA > 1 && D == 8 ? j >> 2 : 0];
          z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[j][a]), __builtin_bit_cast(bf16x8, xb[j][h][c]), z, 0, 0, 0);
        }
    constexpr bool sum_of_halves = BOTH && NA == 3 && D == 8;
    if (NA > 1 && (D < 8 || sum_of_halves) && j == D - 1)
#pragma unroll
      for (int a = 0; a < HB; ++a)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if constexpr (sum_of_halves) {
            acc[a][c][2] += acc[a][c][0] + acc[a][c][1];
            acc[a][c][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
          } else {
            acc[a][c][1] += acc[a][c][0];
          }
          acc[a][c][0] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
  };
  if (len > 0) {
    // ring: stage j of a block of D steps is multiplied, then requested again for the step D later.
    // The scheduling fences keep that order (the compiler otherwise gathers all products behind one
    // wait for every load in flight).
#pragma unroll
    for (int j = 0; j < D; ++j) {
      load(j, min(j, len - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (EPI == kSliceSwiglu || EPI == kSliceQkv) {  // 1 / rms per row, while the ring fills
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      const float rs = row_rms_finish(p.nrm, ss[i]);
      if (lane == 0) rms[wave + 8 * i] = rs;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (len > 0) {
    int base = 0;
    for (; base + 2 * D <= len; base += D) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        mul(j);
        __builtin_amdgcn_sched_barrier(0);
        load(j, base + D + j);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (base + D < len) {  // the last refills, fewer than D
#pragma unroll
      for (int j = 0; j < D; ++j) {
        mul(j);
        __builtin_amdgcn_sched_barrier(0);
        if (base + D + j < len) load(j, base + D + j);
        __builtin_amdgcn_sched_barrier(0);
      }
      base += D;
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (base + j < len) mul(j);
  }

  // sum of the 8 slices through LDS, CH tiles at a time (C layout: lane l = row l%16 of the column
  // group, output features 4*(l/16) .. +3 of the half-band)
  constexpr int CH = slice_chunk<HB, NCP>();
#pragma unroll
  for (int t0 = 0; t0 < NT; t0 += CH) {
    if (t0) __syncthreads();
#pragma unroll
    for (int t = t0; t < NT && t < t0 + CH; ++t) {
      f32x4 z = acc[t / NC][t % NC][0];
      if (NA > 1) z += acc[t / NC][t % NC][1];
      if (NA == 3) z += acc[t / NC][t % NC][2];
      lds_slice[((t - t0) * NW + wave) * 64 + lane] = make_float4(z[0], z[1], z[2], z[3]);
    }
    __syncthreads();
    const int n_here = CH < NT - t0 ? CH : NT - t0;
    auto sum = [&](int t, int l) {  // tile t (within the matrix tile), lane slot l
      const float4 *src = lds_slice + (t - t0) * NW * 64 + l;
      auto add = [](const float4 &a, const float4 &b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
      static_assert(NW == 8, "tree of 8 slices");
      auto slices = [&](const float4 *q) { return add(add(add(q[0], q[64]), add(q[128], q[192])), add(add(q[256], q[320]), add(q[384], q[448]))); };
      if constexpr (BOTH) {  // hi products in rows 0 .. 7, lo products in rows 8 .. 15 (surplus rows repeat them, unused)
        const float4 *hi = src - (l & 8);
        return add(slices(hi), slices(hi + 8));
      }
      return slices(src);
    };
    if (EPI == kSlicePartial) {
      for (int u = threadIdx.x; u < n_here * 64; u += NW * 64) {
        const int t = t0 + (u >> 6), l = u & 63, hb = nt * HB + t / NC, row = (t % NC) * 16 + (l & 15);
        const float4 v = sum(t, l);
        if (row < p.rows && hb < p.n_half)
          *reinterpret_cast<float4 *>(p.part + part_offset(s, row, hb * 16 + (l >> 4) * 4, (p.n_half + 1) / 2, 32 * nb)) = v;
      }
    } else if (EPI == kSliceSwiglu) {
      // half-band = gate features 8*hb .. +7, then the up features of the same index
      for (int u = threadIdx.x; u < n_here * 32; u += NW * 64) {
        const int t = t0 + (u >> 5), qd = (u >> 4) & 1, hb = nt * HB + t / NC, row = (t % NC) * 16 + (u & 15);
        const float4 gt = sum(t, qd * 16 + (u & 15)), up = sum(t, (qd + 2) * 16 + (u & 15));
        if (row >= p.rows || hb >= p.n_half) continue;
        const float rs = rms[row];
        const float y[4] = {swiglu_act(gt.x, up.x, rs), swiglu_act(gt.y, up.y, rs), swiglu_act(gt.z, up.z, rs), swiglu_act(gt.w, up.w, rs)};
        store_planes4(y, p.t, p.t_lo, packed_act_offset(row, 8 * hb + 4 * qd, nb));
      }
    } else if (EPI == kSliceQkv) {
      if (q_kind >= 0 && q_t >= t0 && q_t < t0 + n_here) {
        const int l = q_qd * 16 + (threadIdx.x & 15);
        float4 a = sum(q_t, l), b = sum(q_t, l + 32);
        const float rs = rms[q_row];
        const float x0[4] = {a.x * rs, a.y * rs, a.z * rs, a.w * rs}, x1[4] = {b.x * rs, b.y * rs, b.z * rs, b.w * rs};
        const float co[4] = {q_cs01.x, q_cs01.z, q_cs23.x, q_cs23.z}, si[4] = {q_cs01.y, q_cs01.w, q_cs23.y, q_cs23.w};
        float y0[4], y1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          y0[i] = rotated_first(x0[i], x1[i], co[i], si[i]);
          y1[i] = rotated_second(x0[i], x1[i], co[i], si[i]);
        }
        if (q_kind == 0) {
          const int64_t o = ((int64_t)q_row * p.H + q_head) * p.hd + q_j;
#pragma unroll
          for (int i = 0; i < 4; ++i) { y0[i] *= p.qscale; y1[i] *= p.qscale; }
          store_planes4(y0, p.qb, p.qb_lo, o);
          store_planes4(y1, p.qb, p.qb_lo, o + p.hd / 2);
        } else if (q_kind == 1) {
          store_bf16x4(y0, p.kc + q_cache + q_j);
          store_bf16x4(y1, p.kc + q_cache + q_j + p.hd / 2);
        } else {  // values: natural order, quads q_qd and q_qd + 2
          store_bf16x4(x0, p.vc + q_cache + q_j);
          store_bf16x4(x1, p.vc + q_cache + q_j + 8);
        }
      }
    } else {  // kSliceResid: x += sum; planes of x * gain; sum of squares per row and half-band
      float sq = 0.f;
      if (rt < NT) {
        const float4 v = sum(rt, lane);
        const float y[4] = {r_x.x + v.x, r_x.y + v.y, r_x.z + v.z, r_x.w + v.w};
        if (r_ok) {
          *reinterpret_cast<float4 *>(p.x + (int64_t)r_row * p.d + r_col) = make_float4(y[0], y[1], y[2], y[3]);
          const float z[4] = {y[0] * bf16_bits_to_f32(r_g.x & 0xffffu), y[1] * bf16_bits_to_f32(r_g.x >> 16),
                              y[2] * bf16_bits_to_f32(r_g.y & 0xffffu), y[3] * bf16_bits_to_f32(r_g.y >> 16)};
          store_planes4(z, p.t, p.t_lo, packed_act_offset(r_row, r_col, nb));
          sq = sum_squares4(y[0], y[1], y[2], y[3]);
        }
        sq += __shfl_xor(sq, 16, 64);
        sq += __shfl_xor(sq, 32, 64);
        if (r_ok && lane < 16) p.ssq_out[(int64_t)r_row * p.n_slab_out + r_hb] = sq;
      }
    }
  }
}

// --------------------------------------------------------------------------- plans and launch
namespace {

constexpr int kMaxLds = 128 * 1024;

template <int EPI, int HB, int NC>
void launch_one(const SliceArgs &args, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  SliceArgs a = args;
  a.total = (a.n_half + HB - 1) / HB * a.S;
  a.per_xcd = (a.total + 7) / 8;
  const unsigned grid = 8u * a.per_xcd;
  constexpr unsigned lds = slice_chunk<HB, NC>() * kSliceWaves * 1024;
  static_assert(lds <= kMaxLds, "LDS of the slice sums");
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL((gemm_slice_kernel<EPI, HB, NC>), dim3(grid), dim3(kSliceWaves * 64), lds, st, ev0, ev1, 0u, a);
  else
    gemm_slice_kernel<EPI, HB, NC><<<grid, kSliceWaves * 64, lds, st>>>(a);
}

template <int EPI, int HB, int NC>
hipError_t set_lds_one() {
  return hipFuncSetAttribute((const void *)gemm_slice_kernel<EPI, HB, NC>, hipFuncAttributeMaxDynamicSharedMemorySize, slice_chunk<HB, NC>() * kSliceWaves * 1024);
}

// The instantiated (half-bands, row groups) per epilogue; F is called with the two as types.
template <int V> struct Int { static constexpr int value = V; };
template <int EPI, int NC, class F>
bool with_hb(int hb, F f) {
  constexpr bool qkv = EPI == kSliceQkv, sw = EPI == kSliceSwiglu, part = EPI == kSlicePartial;
  // (partial sums of two row groups: the split kernel is faster)
  if constexpr ((part && NC == 2) || (!part && NC > 3) || ((qkv || EPI == kSliceResid) && NC > 2)) return false;
  else switch (hb) {
    case 1: if constexpr (!part) { f(Int<1>{}, Int<NC>{}); return true; } break;
    case 2: if constexpr (EPI != kSliceResid) { f(Int<2>{}, Int<NC>{}); return true; } break;
    case 3: if constexpr (sw || qkv) { f(Int<3>{}, Int<NC>{}); return true; } break;
    case 4: if constexpr (EPI != kSliceResid) { f(Int<4>{}, Int<NC>{}); return true; } break;
    case 5: if constexpr (sw && NC <= 3) { f(Int<5>{}, Int<NC>{}); return true; } break;
    case 6: if constexpr (sw && NC <= 3) { f(Int<6>{}, Int<NC>{}); return true; } break;
    case 7: if constexpr (sw && NC <= 2) { f(Int<7>{}, Int<NC>{}); return true; } break;
    case 8: if constexpr ((sw || part) && NC <= 2) { f(Int<8>{}, Int<NC>{}); return true; } break;
  }
  return false;
}
template <int EPI, class F>
bool with_shape(int hb, int nc, F f) {
  switch (nc) {
    case 1: return with_hb<EPI, 1>(hb, f);
    case 2: return with_hb<EPI, 2>(hb, f);
    case 3: return with_hb<EPI, 3>(hb, f);
    case 4: return with_hb<EPI, 4>(hb, f);
  }
  return false;
}

template <int EPI>
hipError_t set_lds_epi() {
  hipError_t e = hipSuccess;
  for (int nc = 1; nc <= 4; ++nc)
    for (int hb = 1; hb <= 8; ++hb)
      with_shape<EPI>(hb, nc, [&](auto h, auto c) {
        constexpr int HB = decltype(h)::value, NC = decltype(c)::value;
        if (e == hipSuccess) e = set_lds_one<EPI, HB, NC>();
        if constexpr (NC == 1)
          if (e == hipSuccess) e = set_lds_one<EPI, HB, 0>();
      });
  return e;
}

template <int EPI>
bool launch_epi(const SliceArgs &a, const SlicePlan &pl, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  return with_shape<EPI>(pl.hb, pl.nc, [&](auto h, auto c) {
    constexpr int HB = decltype(h)::value, NC = decltype(c)::value;
    if constexpr (NC == 1) {
      // up to 8 rows one operand holds both planes: half the activation loads and products (1.1B, 1 row: gate|up 12.5 ->
      // 11.8 us, q|k|v 7.0 -> 6.2, down 7.1 -> 6.6, o 6.3 -> 5.6)
      if (slice_groups_launched(NC, a.rows) == 0) return launch_one<EPI, HB, 0>(a, st, ev0, ev1);
    }
    launch_one<EPI, HB, NC>(a, st, ev0, ev1);
  });
}

}  // namespace

bool slice_shape_built(int epi, int hb, int nc) {
  auto nop = [](auto, auto) {};
  switch (epi) {
    case kSlicePartial: return with_shape<kSlicePartial>(hb, nc, nop);
    case kSliceSwiglu: return with_shape<kSliceSwiglu>(hb, nc, nop);
    case kSliceQkv: return with_shape<kSliceQkv>(hb, nc, nop);
    case kSliceResid: return with_shape<kSliceResid>(hb, nc, nop);
  }
  return false;
}

hipError_t gemm_slice_set_lds_limit() {
  hipError_t e = set_lds_epi<kSlicePartial>();
  if (e == hipSuccess) e = set_lds_epi<kSliceSwiglu>();
  if (e == hipSuccess) e = set_lds_epi<kSliceQkv>();
  if (e == hipSuccess) e = set_lds_epi<kSliceResid>();
  return e;
}

bool launch_gemm_slice(int epi, const SliceArgs &a, const SlicePlan &pl, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  switch (epi) {
    case kSlicePartial: return launch_epi<kSlicePartial>(a, pl, st, ev0, ev1);
    case kSliceSwiglu: return launch_epi<kSliceSwiglu>(a, pl, st, ev0, ev1);
    case kSliceQkv: return launch_epi<kSliceQkv>(a, pl, st, ev0, ev1);
    case kSliceResid: return launch_epi<kSliceResid>(a, pl, st, ev0, ev1);
  }
  return false;
}

}  // namespace specasr
