// GEMMs for a few hundred activation rows at most (a small batch of trees, a short prefill), gfx950.
//
// Between the skinny kernels (<= 64 rows, bound by the weight stream) and the tiled kernel of
// kernels_mfma.hip (256 features x 128 rows per workgroup, bound by the matrix cores) the tiled kernel
// runs out of workgroups: it has to cut k into 5 .. 13 splits to fill the chip, each an output-sized
// fp32 buffer that the consumer reads again.  Here the output tile is small (2 .. 3 bands of 32
// features x 2 .. 3 groups of 32 rows) and k is cut INSIDE the workgroup: every wavefront takes a slice
// of k for the whole tile and streams its operands straight into registers (a ring of D stages; both
// operands are stored in MFMA operand order), without LDS or barriers in the loop; the slices are
// summed through LDS at the end.  One wavefront multiplies A x B tiles from A + 2B loads; up to 7 x 3 tiles fit the registers
// of a lone wavefront per SIMD (plan_mid_tall).
// What bounds it: the bytes a compute unit can pull out of its L2, about 58 per ns.
// Measured (us under the tracer, tiled kernel and its splits at 96 rows -> this at 87, 7B): gate|up 53.7 + its finishing
// kernel -> 52.2 with SwiGLU, q|k|v 37.9 (5 splits) -> 28.8 (2), o 17.4 (8) -> 14.6 (5), down 31.5 (13) -> 30.1 (5); 384
// rows of the 1.1B model q|k|v 19.8 (5) -> 14.6 (2), o 17.1 (5) -> 13.3 (2).  At 33 .. 64 rows it also replaces the split
// skinny kernel (not for q|k|v) where one round of workgroups covers the output: 7B, 64 rows gate|up 39.3 + 6.4 -> 40.7,
// down 26.8 -> 26.7 with 5 splits instead of 16, which the next kernel reads.
#include <hip/hip_ext.h>

#include <algorithm>

#include "kernels.h"
#include "kernels_mfma.h"

namespace specasr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kMidTile = 8 * 33;  // float4 of one 32 x 32 tile in LDS: [feature quad][row], one pad per quad row

// Tiles of a workgroup summed through LDS at a time (at most 152 KB).
template <int A, int B, int NW>
constexpr int mid_chunk() {
  constexpr int fit = 152 * 1024 / (NW * kMidTile * 16);
  return fit < A * B ? fit : A * B;
}

struct MidArgs {
  const void *W;
  const uint16_t *X;
  float *part;
  int rows, rows_pad, n_bands, ksteps, nb, S;  // nb: row groups in the planes
  int n_mt, total, per_xcd;                    // row tiles, workgroups, workgroups per XCD
  RowNorm nrm;                                 // SwiGLU epilogue
  uint16_t *t, *t_lo;
};

// ONCE: one row tile, every weight is used once and need not stay in the L2.
// grid 8 * per_xcd, block 64 * NW.  An XCD (workgroup index mod 8) owns a contiguous run of tiles, row tiles of
// one feature tile next to each other.
template <int A, int B, int D, int NW, bool SWIGLU, bool ONCE = false>
__global__ __launch_bounds__(NW * 64, NW / 4) void gemm_mid_kernel(MidArgs p) {
  extern __shared__ float4 lds_mid[];
  __shared__ float rms[SWIGLU ? 32 * B : 1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t slot = blockIdx.x >> 3, id = (blockIdx.x & 7) * p.per_xcd + slot;
  if (slot >= (uint32_t)p.per_xcd || id >= (uint32_t)p.total) return;
  const uint32_t mt = id % (uint32_t)p.n_mt, rest = id / (uint32_t)p.n_mt, s = rest % (uint32_t)p.S, nt = rest / (uint32_t)p.S;
  const uint32_t ks = p.ksteps, c0 = ks * s / p.S, c1 = ks * (s + 1) / p.S;
  const int w0 = c0 + (c1 - c0) * wave / NW, len = (int)(c0 + (c1 - c0) * (wave + 1) / NW) - w0;
  const int n_groups = (p.rows + 31) >> 5;
  const u32x4 *wp[A], *xp[2][B];
#pragma unroll
  for (int a = 0; a < A; ++a) wp[a] = (const u32x4 *)p.W + ((int64_t)min((int)nt * A + a, p.n_bands - 1) * p.ksteps + w0) * 64 + lane;
  const int64_t plane = (int64_t)p.ksteps * p.nb * 64;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int b = 0; b < B; ++b) xp[h][b] = (const u32x4 *)p.X + h * plane + ((int64_t)w0 * p.nb + min((int)mt * B + b, n_groups - 1)) * 64 + lane;
  const uint32_t xs = p.nb * 64;
  f32x16 acc[A][B];
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[a][b][j] = 0.f;
  u32x4 wa[D][A], xb[D][2][B];
  auto load = [&](int j, uint32_t k) {
#pragma unroll
    for (int a = 0; a < A; ++a) wa[j][a] = ONCE ? __builtin_nontemporal_load(wp[a] + k * 64) : wp[a][k * 64];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int b = 0; b < B; ++b) xb[j][h][b] = xp[h][b][k * xs];
  };
  // hi products first, then lo: A * B independent accumulators in between.  Beyond 16 tiles the accumulators outgrow the
  // 256 accumulation registers that the compiler keeps them in, so those tiles are named as vector registers by hand (it
  // spills otherwise: 6 x 3 tiles 940 bytes, no gain).  It puts no wait states around what it does not know to be MFMAs, so
  // their order is held by fences: in each plane they come first and 16 other MFMAs behind them, more than the wait states of a
  // result, before the other plane, the end of the step or anything else may touch them.
  auto mul = [&](int j) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int t = 16; t < A * B; ++t)
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc[t / B][t % B]) : "v"(wa[j][t / B]), "v"(xb[j][h][t % B]));
      if (A * B > 16) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 16 && t < A * B; ++t)
        acc[t / B][t % B] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wa[j][t / B]), __builtin_bit_cast(bf16x8, xb[j][h][t % B]), acc[t / B][t % B], 0, 0, 0);
      if (A * B > 16) __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (len > 0) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      load(j, min(j, len - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (SWIGLU) {  // 1 / rms of the tile's rows, 8 threads per row, while the ring fills
#pragma unroll
    for (int r0 = 0; r0 < 32 * B; r0 += NW * 8) {
      const int rl = r0 + (threadIdx.x >> 3);
      const float *sq = p.nrm.ssq + (int64_t)min((int)mt * B * 32 + rl, p.rows - 1) * p.nrm.n_slab;
      float ss = 0.f;
#pragma unroll 4
      for (int i = threadIdx.x & 7; i < p.nrm.n_slab; i += 8) ss += sq[i];
      ss += __shfl_xor(ss, 1, 64);
      ss += __shfl_xor(ss, 2, 64);
      ss += __shfl_xor(ss, 4, 64);
      if ((threadIdx.x & 7) == 0 && rl < 32 * B) rms[rl] = 1.0f / sqrtf(ss / (float)p.nrm.d + p.nrm.eps);
    }
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
  // The sums read those results behind this wait, whatever stands in front of it (20 wait states).
  if (A * B > 16) asm volatile("s_nop 15\n\ts_nop 3");
#pragma unroll
  for (int t = 16; t < A * B; ++t) asm volatile("" : "+v"(acc[t / B][t % B]));
  // sum of the NW slices through LDS, CH tiles at a time.  C layout: register 4q + e of lane l = row l%32,
  // feature 8q + 4(l/32) + e, i.e. feature quad 2q + l/32
  constexpr int NT = A * B, CH = mid_chunk<A, B, NW>();
#pragma unroll
  for (int t0 = 0; t0 < NT; t0 += CH) {
    if (t0) __syncthreads();
#pragma unroll
    for (int t = t0; t < NT && t < t0 + CH; ++t) {
      const f32x16 &z = acc[t / B][t % B];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        lds_mid[((t - t0) * NW + wave) * kMidTile + (2 * q + (lane >> 5)) * 33 + (lane & 31)] = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
    }
    __syncthreads();
    const int n_here = CH < NT - t0 ? CH : NT - t0;
    auto sum = [&](int t, int quad, int rl) {
      const float4 *src = lds_mid + (t - t0) * NW * kMidTile + quad * 33 + rl;
      auto add = [](const float4 &a, const float4 &b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
      float4 v = add(add(src[0], src[kMidTile]), add(src[2 * kMidTile], src[3 * kMidTile]));
      if constexpr (NW == 8) v = add(v, add(add(src[4 * kMidTile], src[5 * kMidTile]), add(src[6 * kMidTile], src[7 * kMidTile])));
      return v;
    };
    if (SWIGLU) {
      // quads 0, 1 (4, 5) are gate, 2, 3 (6, 7) up of the same 8 features; item = (tile, quad pair, row)
      for (int u = threadIdx.x; u < n_here * 128; u += NW * 64) {
        const int t = t0 + (u >> 7), gq = (u >> 5) & 3, rl = u & 31, quad = (gq & 1) + 4 * (gq >> 1);
        const int row = ((int)mt * B + t % B) * 32 + rl, band = (int)nt * A + t / B;
        const float4 g = sum(t, quad, rl), up = sum(t, quad + 2, rl);
        if (row >= p.rows || band >= p.n_bands) continue;
        const float rs = rms[(t % B) * 32 + rl];
        const float y[4] = {swiglu_act(g.x, up.x, rs), swiglu_act(g.y, up.y, rs), swiglu_act(g.z, up.z, rs), swiglu_act(g.w, up.w, rs)};
        store_planes4(y, p.t, p.t_lo, packed_act_offset(row, band * 16 + 8 * (gq >> 1) + 4 * (gq & 1), p.nb));
      }
    } else {
      for (int u = threadIdx.x; u < n_here * 256; u += NW * 64) {  // item = (tile, row, quad): 128 bytes per row
        const int t = t0 + (u >> 8), rl = (u >> 3) & 31, quad = u & 7;
        const int row = ((int)mt * B + t % B) * 32 + rl, band = (int)nt * A + t / B;
        const float4 v = sum(t, quad, rl);
        if (row < p.rows && band < p.n_bands)
          *reinterpret_cast<float4 *>(p.part + part_offset(s, row, band * 32 + quad * 4, p.n_bands, p.rows_pad)) = v;
      }
    }
  }
}

namespace {

template <int A, int B, int D, int NW, bool SWIGLU, bool ONCE = false>
void launch_mid_t(MidArgs a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  a.n_mt = ((a.rows + 31) / 32 + B - 1) / B;
  a.total = a.n_mt * ((a.n_bands + A - 1) / A) * a.S;
  a.per_xcd = (a.total + 7) / 8;
  constexpr unsigned lds = mid_chunk<A, B, NW>() * NW * kMidTile * 16;
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL((gemm_mid_kernel<A, B, D, NW, SWIGLU, ONCE>), dim3(8u * a.per_xcd), dim3(NW * 64), lds, st, ev0, ev1, 0u, a);
  else
    gemm_mid_kernel<A, B, D, NW, SWIGLU, ONCE><<<8u * a.per_xcd, NW * 64, lds, st>>>(a);
}

template <int A, int B, int D, int NW, bool SWIGLU, bool ONCE = false>
hipError_t set_lds_mid() {
  return hipFuncSetAttribute((const void *)gemm_mid_kernel<A, B, D, NW, SWIGLU, ONCE>, hipFuncAttributeMaxDynamicSharedMemorySize, mid_chunk<A, B, NW>() * NW * kMidTile * 16);
}

}  // namespace

// The built tiles; ring and wavefronts as many as their registers allow.
hipError_t gemm_mid_set_lds_limit() {
  hipError_t e = set_lds_mid<2, 2, 4, 8, false>();
  if (e == hipSuccess) e = set_lds_mid<2, 3, 3, 8, false>();
  if (e == hipSuccess) e = set_lds_mid<3, 3, 4, 4, false>();
  if (e == hipSuccess) e = set_lds_mid<2, 3, 3, 8, true>();
  if (e == hipSuccess) e = set_lds_mid<3, 3, 4, 4, true>();
  if (e == hipSuccess) e = set_lds_mid<3, 3, 4, 4, false, true>();
  if (e == hipSuccess) e = set_lds_mid<3, 3, 4, 4, true, true>();
  if (e == hipSuccess) e = set_lds_mid<6, 3, 3, 4, false>();
  if (e == hipSuccess) e = set_lds_mid<6, 3, 3, 4, true>();
  if (e == hipSuccess) e = set_lds_mid<7, 3, 2, 4, false>();
  if (e == hipSuccess) e = set_lds_mid<7, 3, 2, 4, true>();
  if (e == hipSuccess) e = set_lds_mid<2, 2, 4, 8, false, true>();
  if (e == hipSuccess) e = set_lds_mid<2, 2, 4, 8, true, true>();
  if (e == hipSuccess) e = set_lds_mid<3, 2, 3, 8, false, true>();
  if (e == hipSuccess) e = set_lds_mid<3, 2, 3, 8, true, true>();
  return e;
}

// Tile and split of a GEMM over `rows` (> 32) rows, or a = 0 where the other kernel, estimated at `other_us`, is
// faster.  Costs in us, fitted to the measurements above: launch, ring fill and sums 3.5, per round of
// workgroups the bytes of one at 58 per ns (47 up to 64 rows: 13B q|k|v + o, 40 rows, 59.4 here against 55.3) or its MFMAs, at least the weight stream, 0.1 per MB of partial
// sums written and 0.12 per MB read again (none with the SwiGLU epilogue).
MidPlan plan_mid(int n_bands, int ksteps, int rows, double other_us, bool swiglu, int n_cu) {
  MidPlan best;
  double best_cost = other_us;
  const int nb = (rows + 31) / 32;
  const double out_mb = (double)n_bands * 32 * rows * 4e-6, w_mb = (double)n_bands * ksteps * 1.024e-3;
  const int tiles[4][2] = {{2, 2}, {2, 3}, {3, 3}, {3, 2}};
  for (const auto &t : tiles) {
    const int a = t[0], b = t[1];
    if (rows <= 64 ? b == 3 : (a == 3 && b == 2) || (swiglu && b == 2)) continue;  // not built or never better
    const int64_t n = (int64_t)((n_bands + a - 1) / a) * ((nb + b - 1) / b);
    for (int S = 1; S <= (swiglu ? 1 : 8) && ksteps / S >= 32; ++S) {
      const double len = (double)ksteps / S, rounds = (double)((n * S + n_cu - 1) / n_cu);
      // a second, part-filled round loses to the split kernel, which spreads bands evenly (13B gate|up, 40 rows: 78.6
      // against 67.8 + 9.0)
      if (rows <= 64 && rounds > 1) break;
      const double wg = std::max((a + 2 * b) * len * 1.024 / (rows <= 64 ? 47.0 : 58.0), a * b * 2 * len * 8.0 / 2100.0);
      const double cost = 3.5 + std::max(rounds * wg, w_mb / 5.9) + (swiglu ? out_mb * 0.1 : S * out_mb * 0.22);
      if (cost < best_cost) {
        best_cost = cost;
        best.a = a;
        best.b = b;
        best.S = S;
      }
    }
  }
  best.cost_us = best_cost;
  return best;
}

// Six or seven bands per workgroup instead of the plan's kernel (`slices`: its parts of k, `other_us`: its estimate), or a = 0.
// A wavefront with 6 x 3 tiles loads 12 KB per 36 MFMAs where one with 3 x 3 loads 9 per 18, and there is half the number of
// workgroups, in one round where it took two.  More than 64 rows, where the rows fill three groups.
// Measured, us: 1.1B gate|up, 384 rows 51.8 (3 x 3, two rounds) -> 38.7, 192 rows 31.0 (one round) against 36.8 here; 7B q|k|v, 300
// rows 94 (tiled, split) -> 64, 810 rows 163 + 8 for the second partial sum -> 147 (7 bands: 495 workgroups where 6 have 576);
// 13B down, 192 rows 65 -> 58.  In the model, ms: 1.1B 16 x 24 nodes 3.55 -> 3.27, prefill of 330 2.89 -> 2.69, of 900 6.18 ->
// 5.67; 7B prefill of 192 7.80 -> 6.93, of 384 11.27 -> 10.62, of 810 22.17 -> 21.48.  Costs fitted to these: 5, and per round 5
// and 0.215 per k-step (7 bands 0.24); 0.12 per MB of partial sums for the reader.  The other kernels' estimates are less exact,
// so 10 % is asked for.  k is cut into 4 slices per split, and the sums' chains may not get longer than they were: no fewer
// slices than the other plan's.
MidPlan plan_mid_tall(int n_bands, int ksteps, int rows, int slices, double other_us, bool swiglu, int n_cu) {
  MidPlan best;
  double limit = 0.9 * other_us;
  const int64_t n_mt = (rows + 95) / 96;
  const double out_mb = (double)n_bands * 32 * rows * 4e-6;
  for (int a = 6; a <= 7; ++a)
    for (int S = 1; S <= (swiglu ? 1 : 8) && ksteps / S >= 32; ++S) {
      if (4 * S < slices) continue;
      const double rounds = (double)((n_mt * ((n_bands + a - 1) / a) * S + n_cu - 1) / n_cu);
      const double cost = 5.0 + rounds * ((double)ksteps / S * (a == 7 ? 0.24 : 0.215) + 5.0) + (swiglu ? 0.0 : S * out_mb * 0.12);
      if (cost >= limit) continue;
      limit = cost;
      best.a = a;
      best.b = 3;
      best.S = S;
      best.cost_us = cost;
    }
  return best;
}

// What the tiled kernel takes by the same measure: 10 plus its k-loop (its own planner's constants), and the finishing
// kernel of a split gate|up about 4.  This is fitted for the comparison with the small tiles at 65 .. 400 rows, by
// kernel times and with the reading of the partial sums; wide_gemm_cost, which picks the split count, counts 18 and
// 0.3 per MB, fitted to the tiled kernel alone at 256 .. 512 rows.  Above that range this one is low (7B down at 810 rows:
// 112, measured 141), but the small tiles are further behind there than that.
double wide_gemm_estimate(int n_bands, int ksteps, int rows, int splits, bool swiglu, int n_cu) {
  const double out_mb = (double)n_bands * 32 * rows * 4e-6;
  const int64_t wgs = (int64_t)((n_bands + 7) / 8) * (wide_row_groups(rows) / 4) * splits, per_cu = (wgs + n_cu - 1) / n_cu;
  const double t = 10.0 + per_cu * ((double)ksteps / splits) * (wgs >= n_cu ? 0.33 : 0.28) + (per_cu - 1) * 6.0;
  return t + (swiglu && splits == 1 ? out_mb * 0.1 : splits * out_mb * 0.22 + (swiglu ? 4.0 : 0.0));
}

void launch_gemm_mid(const PackedMatrix &W, const uint16_t *Xp, int rows, float *part, const MidPlan &pl, const RowNorm *nrm,
                     uint16_t *t, uint16_t *t_lo, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  MidArgs a{};
  a.W = W.data; a.X = Xp; a.part = part;
  a.rows = rows; a.rows_pad = part_rows_pad(rows); a.n_bands = W.n_bands; a.ksteps = W.ksteps; a.nb = rows <= 64 ? 2 : wide_row_groups(rows); a.S = pl.S;
  if (nrm != nullptr) {  // SwiGLU epilogue
    a.nrm = *nrm; a.t = t; a.t_lo = t_lo;
    if (pl.a == 7) launch_mid_t<7, 3, 2, 4, true>(a, st, ev0, ev1);
    else if (pl.a == 6) launch_mid_t<6, 3, 3, 4, true>(a, st, ev0, ev1);
    else if (rows <= 64 && pl.a == 2) launch_mid_t<2, 2, 4, 8, true, true>(a, st, ev0, ev1);
    else if (rows <= 64) launch_mid_t<3, 2, 3, 8, true, true>(a, st, ev0, ev1);
    else if (pl.a == 2) launch_mid_t<2, 3, 3, 8, true>(a, st, ev0, ev1);
    else if (rows <= 96) launch_mid_t<3, 3, 4, 4, true, true>(a, st, ev0, ev1);
    else launch_mid_t<3, 3, 4, 4, true>(a, st, ev0, ev1);
  } else if (pl.a == 7) {
    launch_mid_t<7, 3, 2, 4, false>(a, st, ev0, ev1);
  } else if (pl.a == 6) {
    launch_mid_t<6, 3, 3, 4, false>(a, st, ev0, ev1);
  } else if (rows <= 64 && pl.a == 2) {
    launch_mid_t<2, 2, 4, 8, false, true>(a, st, ev0, ev1);
  } else if (rows <= 64) {
    launch_mid_t<3, 2, 3, 8, false, true>(a, st, ev0, ev1);
  } else if (pl.a == 3 && rows <= 96) {
    launch_mid_t<3, 3, 4, 4, false, true>(a, st, ev0, ev1);
  } else if (pl.a == 3) {
    launch_mid_t<3, 3, 4, 4, false>(a, st, ev0, ev1);
  } else if (pl.b == 3) {
    launch_mid_t<2, 3, 3, 8, false>(a, st, ev0, ev1);
  } else {
    launch_mid_t<2, 2, 4, 8, false>(a, st, ev0, ev1);
  }
}

}  // namespace specasr
