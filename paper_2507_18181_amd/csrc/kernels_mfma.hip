// bf16 MFMA stages of the tree-verification path for gfx950 (CDNA4, wave64).
//
// The projections of the decoder are skinny GEMMs: at most 64 tree-node rows against every
// weight of the model, so each weight byte is used once per call and the stage is bound by HBM
// bandwidth.  Design:
//   * Weights are repacked once (specasr_create) into MFMA-operand order: the matrix is cut into
//     tiles of 32 output features x 16 input features; one tile is 1 KB laid out exactly as the A
//     operand of v_mfma_f32_32x32x16_bf16 (lane l holds row l%32, k = 8*(l/32)..+7), and the tiles
//     of one 32-row band are contiguous along k.  A wavefront streams its tiles with one fully
//     coalesced 16-byte non-temporal load per lane per tile, straight into the matrix core.
//   * The activations (the B operand, <= 64 rows) are kept by their producers in the matching
//     B-operand order, as TWO bf16 planes hi = bf16(v) and lo = bf16(v - hi).  Every weight tile is
//     multiplied with both (products exact in fp32), so the projections see the activations to
//     16 mantissa bits; the matrix cores have >10x headroom on this stage, and the extra MFMA is
//     what keeps 22-32 layers inside the 2e-2 logit tolerance.
//   * One workgroup of 8 wavefronts per compute unit.  The k range is cut into S chunks across
//     workgroups and each chunk into 8 slices across the wavefronts of a workgroup; a wavefront
//     keeps the activations of ITS slice in registers for the whole kernel (no LDS traffic in the
//     inner loop) and walks over the bands of its workgroup.  Slot k of its weight ring always
//     holds tile k of the slice and is refilled, right after use, with the same tile of the next
//     band: a whole band-slice of loads stays in flight, across band boundaries, branch-free.
//   * The 8 slice results of a band are summed through LDS and written as one partial sum per
//     k-chunk; the consumer stage adds the S partials in fixed order (deterministic, no atomics).
#include <hip/hip_ext.h>

#include "kernels.h"
#include "kernels_mfma.h"
#include <type_traits>

namespace specasr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ u32x4 load_stream(const u32x4 *p) { return __builtin_nontemporal_load(p); }

// --------------------------------------------------------------------------- weight repack
// dst tile (band, kt), lane l, element i  <-  src[band*32 + l%32][kt*16 + 8*(l/32) + i]
// Rows >= n_out (padding of the last band) are zero.  `band0` is the first packed band written,
// so several source matrices can be concatenated band-aligned into one packed matrix.
__global__ void repack_kernel(const uint16_t *src, int n_out, int K, uint16_t *dst, int band0) {
  const int ksteps = K / 16;
  const int64_t tile = blockIdx.x;  // over bands * ksteps
  const int band = (int)(tile / ksteps), kt = (int)(tile - (int64_t)band * ksteps);
  const int l = threadIdx.x;  // 64 lanes
  const int row = band * 32 + (l & 31);
  u32x4 v = (u32x4){0u, 0u, 0u, 0u};
  if (row < n_out) v = *reinterpret_cast<const u32x4 *>(src + (int64_t)row * K + kt * 16 + 8 * (l >> 5));
  reinterpret_cast<u32x4 *>(dst)[((int64_t)(band0 + band) * ksteps + kt) * 64 + l] = v;
}

// The same with permuted rows, so that every group of 16 packed rows (a half-band) holds what an
// epilogue combines: packed rows 16i .. 16i+7 are rows 8i .. 8i+7 of `a` and rows 16i+8 .. +15 rows
// 8i .. 8i+7 of `b` (both [n][K]).  gate|up: a = w_gate, b = w_up.  Rotary heads: per head of hd
// rows, a = its first half and b = its second half (n = hd/2, one call per head's row range:
// group = hd/16 half-bands, a and b advance by hd rows from head to head).
__global__ void repack_pairs_kernel(const uint16_t *a, const uint16_t *b, int group, int64_t head_rows, int K, uint16_t *dst, int band0, int n_rows) {
  const int ksteps = K / 16;
  const int64_t tile = blockIdx.x;
  const int band = (int)(tile / ksteps), kt = (int)(tile - (int64_t)band * ksteps);
  const int l = threadIdx.x, prow = band * 32 + (l & 31);
  u32x4 v = (u32x4){0u, 0u, 0u, 0u};
  if (prow < n_rows) {
    const int hb = prow >> 4, in = prow & 15, head = hb / group, j = (hb - head * group) * 8 + (in & 7);
    const uint16_t *src = (in < 8 ? a : b) + (head * head_rows + j) * K;
    v = *reinterpret_cast<const u32x4 *>(src + kt * 16 + 8 * (l >> 5));
  }
  reinterpret_cast<u32x4 *>(dst)[((int64_t)(band0 + band) * ksteps + kt) * 64 + l] = v;
}

void launch_repack_gate_up(const void *gate, const void *up, int F, int K, void *dst, hipStream_t st) {
  const int64_t tiles = (int64_t)((2 * F + 31) / 32) * (K / 16);
  repack_pairs_kernel<<<(unsigned)tiles, 64, 0, st>>>((const uint16_t *)gate, (const uint16_t *)up, F / 8, 0, K, (uint16_t *)dst, 0, 2 * F);
}

void launch_repack_rope(const void *src, int heads, int hd, int K, void *dst, int band0, hipStream_t st) {
  const int64_t tiles = (int64_t)((heads * hd + 31) / 32) * (K / 16);
  repack_pairs_kernel<<<(unsigned)tiles, 64, 0, st>>>((const uint16_t *)src, (const uint16_t *)src + (int64_t)(hd / 2) * K, hd / 16, hd, K, (uint16_t *)dst, band0, heads * hd);
}

void launch_repack(const void *src, int n_out, int K, void *dst, int band0, hipStream_t st) {
  const int bands = (n_out + 31) / 32;
  const int64_t tiles = (int64_t)bands * (K / 16);
  repack_kernel<<<(unsigned)tiles, 64, 0, st>>>((const uint16_t *)src, n_out, K, (uint16_t *)dst, band0);
}

// --------------------------------------------------------------------------- read-bandwidth probe
// Streams `n_vec` 16-byte words with the skinny GEMM's access pattern (one workgroup of 512 threads
// per compute unit, each wavefront 8 non-temporal loads of 1 KB in flight) and does nothing with
// them: the ceiling any weight stream on this part can reach, for benchmarks to quote next to the
// nominal HBM figure.
__global__ __launch_bounds__(512) void read_probe_kernel(const u32x4 *__restrict__ p, int64_t n_vec, uint32_t *sink) {
  const int64_t per_wg = (n_vec + gridDim.x - 1) / gridDim.x;
  const int64_t b0 = per_wg * blockIdx.x, b1 = min(b0 + per_wg, n_vec);
  u32x4 acc = (u32x4){0u, 0u, 0u, 0u};
  int64_t i = b0 + threadIdx.x;
  for (; i + 7 * 512 < b1; i += 8 * 512) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = load_stream(p + i + u * 512);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u];
  }
  for (; i < b1; i += 512) acc ^= load_stream(p + i);
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9e3779b9u && n_vec < 0) sink[0] = acc[0];  // never true; keeps the loads
}

void launch_read_probe(const void *buf, size_t bytes, int grid, uint32_t *sink, hipStream_t st) {
  read_probe_kernel<<<grid, 512, 0, st>>>((const u32x4 *)buf, (int64_t)(bytes / 16), sink);
}

// --------------------------------------------------------------------------- skinny GEMM
// part[s][band][row][o % 32] = sum over k in chunk s of X[row][k] * W[o][k]   (see part_offset)
// grid.x = P (a multiple of S), block = 512.  Workgroup g: chunk s, bands bg + j*(P/S) (mapping of g below).
// Xp: packed activations [plane hi|lo][kstep][NB][64 lanes] x 16 bytes.
// STAGE only names the projection (0 qkv, 1 o, 2 gate|up, 3 down, 4 LM head) so that a profiler
// lists each of them as its own kernel; the code is identical.
constexpr int kRedStride = 66;                  // floats between accumulator registers in LDS
constexpr int kRedFloats = 16 * kRedStride;     // one wavefront's 32x32 tile
template <int NB>
constexpr size_t gemm_lds_bytes() { return (size_t)2 * 8 * NB * kRedFloats * 4; }

// Wavefronts 8.. of a workgroup (NR of them; where the register budget allows any: 12 wavefronts
// are three per SIMD, 170 registers each -- the ring of 12 fits with one accumulator for both
// activation planes) do nothing but the summation and the stores, so the 8 streaming wavefronts
// never fall behind one another.
template <int NB, int LW>
constexpr int gemm_reducers() { return (NB == 1 && LW <= 12) ? 4 : 0; }

template <int NB, int LW, int STAGE>
__global__ __launch_bounds__((512 + 64 * gemm_reducers<NB, LW>())) void gemm_skinny_kernel(const u32x4 *__restrict__ Wp,
                                                          const u32x4 *__restrict__ Xp,
                                                          float *__restrict__ part,
                                                          int rows, int n_bands, int ksteps, int S) {
  extern __shared__ float red[];  // [2][8 wavefronts][NB][kRedFloats]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int P = gridDim.x, bstride = P / S;
  // Workgroup -> (k-chunk s, band group bg).  Workgroups reach the 8 XCDs round-robin by index;
  // where the grid allows it, XCD x owns the band groups x * bstride/8 .. and ALL k-chunks of them,
  // so that the addresses one XCD's L2 sees at any time vary in every bit (the plain mapping
  // s = index % S pins the chunk bits per XCD: measured 7 % less bandwidth on the 180 MB stream).
  int s = blockIdx.x % S, bg = blockIdx.x / S;
  if (P % (8 * S) == 0) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    s = slot % S;
    bg = xcd * (bstride >> 3) + slot / S;
  }
  // k-chunk of the workgroup and slice of the wavefront, balanced to within one k-step
  const int c0 = (int)((int64_t)ksteps * s / S), c1 = (int)((int64_t)ksteps * (s + 1) / S);
  const int w0 = c0 + (int)((int64_t)(c1 - c0) * wave / 8), w1 = c0 + (int)((int64_t)(c1 - c0) * (wave + 1) / 8);
  const int len = w1 - w0;  // 0 <= len <= LW
  const int n_units = bg < n_bands ? (n_bands - bg + bstride - 1) / bstride : 0;
  if (n_units == 0) return;
  constexpr int NR = gemm_reducers<NB, LW>();
  const int rows_pad = NB * 32;
  // thread rt of the summing threads: (node group, node, seg) sums output rows 4*seg .. 4*seg+3 of
  // its node over the 8 streaming wavefronts; the 256 threads of a node group write one
  // contiguous 4 KB block [node][32 outputs].  C layout: register j of lane l = node column l%32,
  // output row 8*(j/4) + 4*(l/32) + j%4.
  auto sum_and_store = [&](int rt, int unit) {
    const float *all = red + (unit & 1) * 8 * (NB * kRedFloats);
    const int band = bg + unit * bstride;
    const int n = rt >> 8, node = (rt >> 3) & 31, seg = rt & 7;
    const int q = seg >> 1, h = seg & 1;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const float *src = all + w * (NB * kRedFloats) + n * kRedFloats + (4 * q) * kRedStride + node + 32 * h;
      v.x += src[0]; v.y += src[kRedStride]; v.z += src[2 * kRedStride]; v.w += src[3 * kRedStride];
    }
    const int row = n * 32 + node;
    if (row < rows)
      *reinterpret_cast<float4 *>(part + part_offset(s, row, band * 32 + seg * 4, n_bands, rows_pad)) = v;
  };
  if (NR > 0 && wave >= 8) {
    // One barrier per band on both sides: the streaming wavefronts arrive after writing buffer
    // unit%2, this side after reading buffer (unit-1)%2 -- which is therefore free again before
    // band unit+1 is written into it.
    for (int unit = 0; unit < n_units; ++unit) {
      __syncthreads();
      sum_and_store((int)threadIdx.x - 512, unit);
    }
    return;
  }
  const int64_t band_stride = (int64_t)ksteps * 64;
  const u32x4 *wbase = Wp + (int64_t)min(w0, ksteps - 1) * 64 + lane;
  // slot k reads tile min(k, len-1) of the slice (a duplicate beyond the slice: multiplied by zero)
  int toff[LW];
#pragma unroll
  for (int k = 0; k < LW; ++k) toff[k] = max(min(k, len - 1), 0) * 64;

  u32x4 buf[LW];
  {
    const u32x4 *p = wbase + (int64_t)bg * band_stride;
#pragma unroll
    for (int k = 0; k < LW; ++k) buf[k] = load_stream(p + toff[k]);
  }
  // activations of the slice, both planes, into registers
  u32x4 xh[LW][NB], xl[LW][NB];
  const int64_t plane = (int64_t)ksteps * NB * 64;
#pragma unroll
  for (int k = 0; k < LW; ++k)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const bool ok = k < len;
      const int64_t off = ((int64_t)(w0 + k) * NB + n) * 64 + lane;
      xh[k][n] = ok ? Xp[off] : (u32x4){0u, 0u, 0u, 0u};
      xl[k][n] = ok ? Xp[plane + off] : (u32x4){0u, 0u, 0u, 0u};
    }

  // One band: multiply the ring with the activations while (refill) slot k is reloaded with the
  // same tile of the next band, then sum the 8 wavefronts' tiles through LDS and store the block.
  // The last band is a copy of the code without the reloads, so the steady state has no branch.
  auto do_band = [&](int unit, auto refill) {
    const int band = bg + unit * bstride;
    const u32x4 *pn = wbase + (int64_t)(band + bstride) * band_stride;
    // hi and lo plane on separate accumulators (independent MFMA chains) where the registers
    // allow; the ring of 12 with summing wavefronts has one accumulator per row group
    constexpr int NA = (NB == 1 && LW == 12) ? 1 : 2;
    f32x16 acc[NB][NA];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int h = 0; h < NA; ++h)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[n][h][j] = 0.f;
#pragma unroll
    for (int k = 0; k < LW; ++k) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, buf[k]);
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        acc[n][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, xh[k][n]), acc[n][0], 0, 0, 0);
        acc[n][NA - 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, xl[k][n]), acc[n][NA - 1], 0, 0, 0);
      }
      if (decltype(refill)::value) buf[k] = load_stream(pn + toff[k]);
      // keep this order in the instruction stream: without the fence the scheduler gathers all
      // MFMAs of the band behind one wait for ALL its tiles and issues the refills afterwards,
      // so nothing is in flight while the band is multiplied, reduced and synchronised
      __builtin_amdgcn_sched_barrier(0);
    }
    float *mine = red + ((unit & 1) * 8 + wave) * (NB * kRedFloats);
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) mine[n * kRedFloats + j * kRedStride + lane] = NA == 2 ? acc[n][0][j] + acc[n][NA - 1][j] : acc[n][0][j];
    __syncthreads();
    if (NR == 0 && (int)threadIdx.x < NB * 256) sum_and_store(threadIdx.x, unit);
  };
  // Everything requested so far (first band, activations) has to be there before the first MFMA
  // anyway.  Stating it here lets the compiler see that inside the loop only the refills are
  // outstanding, in slot order: it then waits for slot k with "at most LW - 1 younger loads in
  // flight" instead of draining the whole ring at the top of every band.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  int unit = 0;
  for (; unit + 1 < n_units; ++unit) do_band(unit, std::true_type{});
  do_band(unit, std::false_type{});
}

template <int NB, int LW, int STAGE>
static void launch_gemm_t(const PackedMatrix &W, const uint16_t *Xp, int rows, float *part,
                          const GemmPlan &plan, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const size_t lds = gemm_lds_bytes<NB>();
  constexpr int block = 512 + 64 * gemm_reducers<NB, LW>();
  if (ev0 != nullptr)  // the events take the start and stop time of this dispatch itself
    hipExtLaunchKernelGGL((gemm_skinny_kernel<NB, LW, STAGE>), dim3(plan.grid), dim3(block), (uint32_t)lds, st, ev0, ev1, 0u,
                          (const u32x4 *)W.data, (const u32x4 *)Xp, part, rows, W.n_bands, W.ksteps, plan.n_splits);
  else
    gemm_skinny_kernel<NB, LW, STAGE><<<plan.grid, block, lds, st>>>((const u32x4 *)W.data, (const u32x4 *)Xp, part, rows, W.n_bands, W.ksteps, plan.n_splits);
}

template <int STAGE>
static void launch_gemm_s(const PackedMatrix &W, const uint16_t *Xp, int rows, float *part,
                          const GemmPlan &plan, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (rows <= 32) {
    switch (plan.lw) {
      case 4: launch_gemm_t<1, 4, STAGE>(W, Xp, rows, part, plan, st, ev0, ev1); break;
      case 8: launch_gemm_t<1, 8, STAGE>(W, Xp, rows, part, plan, st, ev0, ev1); break;
      case 12: launch_gemm_t<1, 12, STAGE>(W, Xp, rows, part, plan, st, ev0, ev1); break;
      default: launch_gemm_t<1, 16, STAGE>(W, Xp, rows, part, plan, st, ev0, ev1); break;
    }
  } else {
    if (plan.lw <= 4) launch_gemm_t<2, 4, STAGE>(W, Xp, rows, part, plan, st, ev0, ev1);
    else launch_gemm_t<2, 8, STAGE>(W, Xp, rows, part, plan, st, ev0, ev1);
  }
}

void launch_gemm_skinny(const PackedMatrix &W, const uint16_t *Xp, int rows, float *part,
                        const GemmPlan &plan, int stage, hipStream_t st, hipEvent_t ev0,
                        hipEvent_t ev1) {
  switch (stage) {
    case 0: launch_gemm_s<0>(W, Xp, rows, part, plan, st, ev0, ev1); break;
    case 1: launch_gemm_s<1>(W, Xp, rows, part, plan, st, ev0, ev1); break;
    case 2: launch_gemm_s<2>(W, Xp, rows, part, plan, st, ev0, ev1); break;
    case 3: launch_gemm_s<3>(W, Xp, rows, part, plan, st, ev0, ev1); break;
    default: launch_gemm_s<4>(W, Xp, rows, part, plan, st, ev0, ev1); break;
  }
}

template <int NB, int LW, int STAGE>
static hipError_t set_lds_t() {
  return hipFuncSetAttribute((const void *)gemm_skinny_kernel<NB, LW, STAGE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)gemm_lds_bytes<NB>());
}

template <int STAGE>
static hipError_t set_lds_s() {
  hipError_t e = set_lds_t<1, 4, STAGE>();
  if (e == hipSuccess) e = set_lds_t<1, 8, STAGE>();
  if (e == hipSuccess) e = set_lds_t<1, 12, STAGE>();
  if (e == hipSuccess) e = set_lds_t<1, 16, STAGE>();
  if (e == hipSuccess) e = set_lds_t<2, 4, STAGE>();
  if (e == hipSuccess) e = set_lds_t<2, 8, STAGE>();
  return e;
}

hipError_t gemm_skinny_set_lds_limit() {
  hipError_t e = set_lds_s<0>();
  if (e == hipSuccess) e = set_lds_s<1>();
  if (e == hipSuccess) e = set_lds_s<2>();
  if (e == hipSuccess) e = set_lds_s<3>();
  if (e == hipSuccess) e = set_lds_s<4>();
  return e;
}

// --------------------------------------------------------------------------- wide GEMM (prefill, large batches)
// The same product for hundreds of activation rows (a prefill pass over many positions at once,
// or the trees of a large batch): now every weight tile is used by all rows, the stage is bound
// by the matrix cores, and the classical tiling applies.  One workgroup of 4 wavefronts computes
// 256 output features x 128 rows.  Both operands already are in MFMA operand order in memory, one
// 1 KB tile per (band or row group, k-step), so a tile is copied with ONE direct-to-LDS load per
// wavefront (global_load_lds_dwordx4: lane l's 16 bytes land at base + 16 l -- no staging
// registers, no LDS store instructions) and read back with conflict-free 16-byte LDS loads.
// LDS holds a ring of 4 stages of one k-step each (8 weight tiles + 2 planes x 4 activation
// tiles = 16 KB); wide_loop below says how it turns.  A wavefront owns 128 features x 64 rows: 4 + 2 x 2 operand tiles
// feed 16 MFMAs per k-step into 8 accumulator tiles (hi products first, then lo: 8 independent accumulators between two
// uses of one).  With that loop, us before -> now: 7B 810 rows down 157 -> 143, o 63.5 -> 59, q|k|v 182 -> 175; 300 rows q|k|v
// 105 -> 94; 400 rows down 86 -> 79; 1.1B 384 rows down 28.9 -> 27.4; two full rounds (7B gate|up, 640 rows) the same.
// 64 KB LDS and < 256 registers let two workgroups share a compute unit.  Workgroups that share
// a weight tile (the row tiles of one feature tile) get consecutive slots of one XCD.
//   part[s][band][row][o % 32] as for the skinny kernel; nb = row groups of 32 in Xp, a multiple
//   of 4 (the buffer is allocated to that size; rows >= `rows` hold anything and are not stored).
// grid.x = (nb / 4) * ceil(n_bands / 8) * S rounded up to 8, block 256.
constexpr int kWideTileBands = 8;   // 256 output features per workgroup
constexpr int kWideTileGroups = 4;  // 128 rows per workgroup
constexpr int kWideStageTiles = kWideTileBands + 2 * kWideTileGroups;  // 1 KB tiles per stage (one k-step)

__device__ __forceinline__ void copy_tile_to_lds(const u32x4 *src_lane, u32x4 *dst_tile) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src_lane,
                                   (void __attribute__((address_space(3))) *)dst_tile, 16, 0, 0);
}

// The k loop of the two tiled kernels below: wavefront tile of a bands x b row groups, a ring of D LDS stages (s0 ..) of
// one k-step.  src: what this wavefront copies per stage, 1 KB tiles [lane][16 bytes] at scalar bases, to tile slots dst; the
// k-step adds a multiple of 1 KB (weights) or nb KB (activations).  The copies of the
// D stages have been started for k-steps k0 .. k0 + D-1 before (wide_copy), this runs k-steps k0 .. k0 + n_steps - 1, of which
// the last ones may lie past k1 (multiplied by zero, so that several wavefronts do the same number of steps).  Copies past
// the end of k are clamped to valid tiles, so the number in flight is the same in every step.
//
// Between the hi and the lo products of a k-step stands the barrier that says: everybody's copies of the next stage have
// landed (vmcnt: those of the younger stages may stay in flight), nobody reads this stage any more (lgkmcnt).  Behind it
// this stage's buffer is filled for k-step + D, and w and xh are reloaded from the next stage one by one behind their
// last use: LDS reads, copies and address arithmetic run under the products, without registers for prefetched operands.
// (With wait, barrier, copies and all reads in front of the products of a step, 7B gate|up of 810 rows took 318 us, with
// this order and 64-bit address products in vector registers 275, now 254.)  The barrier is the bare s_barrier:
// __syncthreads would add a fence that waits for ALL copies in flight.
struct WideCopy {
  uint32_t ksteps, nb, lane16;
};
template <int C>
__device__ __forceinline__ void wide_copy(const WideCopy &wc, const char *const (&src)[C], const bool (&weight)[C], const int (&dst)[C], u32x4 *buf, int i, uint32_t ks) {
  const char *base = src[i] + ((uint64_t)ks * (weight[i] ? 1u : wc.nb) << 10);
  copy_tile_to_lds(reinterpret_cast<const u32x4 *>(base + wc.lane16), buf + dst[i] * 64);
}
template <int a, int b, int C, int D, class S, class S3>
__device__ __forceinline__ void wide_loop(f32x16 (&acc)[a][b], S &s0, S &s1, S &s2, S3 &s3, const WideCopy &wc, const char *const (&src)[C], const bool (&weight)[C],
                                          const int (&dst)[C], int at_w, int at_h, int at_l, int k0, int k1, int n_full, int n_steps) {
  static_assert(D == 3 || D == 4, "ring");
  // s_waitcnt immediates of gfx9-class parts: vmcnt in bits 3:0 and 15:14, expcnt 6:4 (7: not waited for), lgkmcnt 11:8 (15: not)
  constexpr int V = (D - 2) * C, V0 = (D - 1) * C;
  constexpr int kNext = (V & 15) | ((V >> 4) << 14) | 0x0070, kFirst = (V0 & 15) | ((V0 >> 4) << 14) | 0x0F70;
  bf16x8 w[a], xh[b], xl[b];
  __builtin_amdgcn_s_waitcnt(kFirst);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");  // no LDS access may be scheduled above the barrier
#pragma unroll
  for (int i = 0; i < a; ++i) w[i] = __builtin_bit_cast(bf16x8, s0[at_w + i * 64]);
#pragma unroll
  for (int g = 0; g < b; ++g) xh[g] = __builtin_bit_cast(bf16x8, s0[at_h + g * 64]);
  auto step = [&](u32x4 *cur, const u32x4 *next, int kt, auto live) {
    const bool dead = !decltype(live)::value && kt >= k1;
    const bf16x8 zero = __builtin_bit_cast(bf16x8, (u32x4){0u, 0u, 0u, 0u});
    const uint32_t ks = min((uint32_t)(kt + D), wc.ksteps - 1);
#pragma unroll
    for (int i = 0; i < a; ++i) {
#pragma unroll
      for (int g = 0; g < b; ++g) acc[i][g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i], dead ? zero : xh[g], acc[i][g], 0, 0, 0);
      if (i == 0) {
#pragma unroll
        for (int g = 0; g < b; ++g) xl[g] = __builtin_bit_cast(bf16x8, cur[at_l + g * 64]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kNext);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < a; ++i) {
#pragma unroll
      for (int g = 0; g < b; ++g) acc[i][g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i], dead ? zero : xl[g], acc[i][g], 0, 0, 0);
      if (i == 0)
#pragma unroll
        for (int g = 0; g < b; ++g) xh[g] = __builtin_bit_cast(bf16x8, next[at_h + g * 64]);
      w[i] = __builtin_bit_cast(bf16x8, next[at_w + i * 64]);
      if (i < C) wide_copy(wc, src, weight, dst, cur, i, ks);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = a; i < C; ++i) wide_copy(wc, src, weight, dst, cur, i, ks);
  };
  int t = 0;
  for (; t + D <= n_full; t += D) {
    step(s0, s1, k0 + t, std::true_type{});
    step(s1, s2, k0 + t + 1, std::true_type{});
    if constexpr (D == 3) {
      step(s2, s0, k0 + t + 2, std::true_type{});
    } else {
      step(s2, s3, k0 + t + 2, std::true_type{});
      step(s3, s0, k0 + t + 3, std::true_type{});
    }
  }
  if (t < n_steps) step(s0, s1, k0 + t, std::false_type{});
  if (t + 1 < n_steps) step(s1, s2, k0 + t + 1, std::false_type{});
  if constexpr (D == 3) {
    if (t + 2 < n_steps) step(s2, s0, k0 + t + 2, std::false_type{});
  } else {
    if (t + 2 < n_steps) step(s2, s3, k0 + t + 2, std::false_type{});
    if (t + 3 < n_steps) step(s3, s0, k0 + t + 3, std::false_type{});
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // all copies and LDS reads: the LDS may be reused or handed to another workgroup
}

// SWIGLU (gate|up, unsplit): the epilogue is the finishing step instead.  gate and up rows are interleaved
// by 8, so a lane's accumulator quads 0 and 1 (2 and 3) are gate and up of the same 4 features: SwiGLU
// happens in registers and the planes of the down projection leave as 512-byte runs.  Saves the
// finishing kernel and the fp32 output (1.1B, 384 rows: 17 MB written and read again for 8.6 MB of planes).
struct WideSwiglu {
  RowNorm nrm;
  uint16_t *t, *t_lo;
};

template <int STAGE, bool SWIGLU = false>
__global__ __launch_bounds__(256, 2) void gemm_wide_kernel(const u32x4 *__restrict__ Wp,
                                                           const u32x4 *__restrict__ Xp,
                                                           float *__restrict__ part, int rows,
                                                           int rows_pad, int n_bands, int ksteps,
                                                           int nb, int S, WideSwiglu sw) {
  // four separate arrays: the compiler can tell a copy into one from the reads of another
  __shared__ u32x4 s0[kWideStageTiles * 64], s1[kWideStageTiles * 64], s2[kWideStageTiles * 64], s3[kWideStageTiles * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // An XCD (workgroup index mod 8) takes an eighth of all (split, feature tile, row tile)s in this order.  (Feature tiles
  // dealt to XCDs by number leave some with one more, and its splits and row tiles as a second round, where 8 does not divide
  // them: 13B down with 20 tiles, 192 rows 108.5 us against 65, 384 rows 160 / 96, o 66 / 41.5; 1.1B q|k|v with 10, 1024 rows
  // 42.5 / 27.7; equal where it does.  In the model, ms: 13B prefill of 384 22.7 / 19.4, 4 x 24 nodes 10.5 / 9.64, 1.1B prefill
  // of 1024 6.55 / 6.05.)
  const uint32_t n_mt = nb / kWideTileGroups, n_nt = (n_bands + kWideTileBands - 1) / kWideTileBands, total = n_mt * n_nt * S;
  const uint32_t id = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (id >= total) return;
  const uint32_t rest = id / n_mt;
  const int mt = id % n_mt, nt = rest % n_nt, s = rest / n_nt;
  const int k0 = (int)((int64_t)ksteps * s / S), k1 = (int)((int64_t)ksteps * (s + 1) / S);
  const int wn = wave & 1, wm = wave >> 1;
  // the 4 tiles this wavefront copies per stage: wavefronts 0, 1 the weight bands 4w .. 4w+3 (bands
  // past the matrix edge are clamped to the last one; their products are never stored), wavefronts
  // 2, 3 the activation tiles [plane][row group]
  const char *src[4];
  bool weight[4];
  int dst[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ti = wave * 4 + i, tb = ti - kWideTileBands;
    weight[i] = ti < kWideTileBands;
    dst[i] = ti;
    src[i] = weight[i] ? (const char *)(Wp + (int64_t)min(nt * kWideTileBands + ti, n_bands - 1) * ksteps * 64)
                       : (const char *)(Xp + (tb >> 2) * ((int64_t)ksteps * nb * 64) + (int64_t)(mt * kWideTileGroups + (tb & 3)) * 64);
  }
  const WideCopy wc{(uint32_t)ksteps, (uint32_t)nb, (uint32_t)lane * 16};
  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][g][j] = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) wide_copy(wc, src, weight, dst, j == 0 ? s0 : j == 1 ? s1 : j == 2 ? s2 : s3, i, min(k0 + j, ksteps - 1));
  __shared__ float rms[SWIGLU ? 32 * kWideTileGroups : 1];
  if (SWIGLU) {  // 1 / rms of the tile's rows, two threads per row, while the first stages arrive
    const int rl = threadIdx.x >> 1;
    const float *sq = sw.nrm.ssq + (int64_t)min(mt * 32 * kWideTileGroups + rl, rows - 1) * sw.nrm.n_slab;
    float ss = 0.f;
    for (int i = threadIdx.x & 1; i < sw.nrm.n_slab; i += 2) ss += sq[i];
    ss += __shfl_xor(ss, 1, 64);
    if ((threadIdx.x & 1) == 0) rms[rl] = 1.0f / sqrtf(ss / (float)sw.nrm.d + sw.nrm.eps);
  }
  wide_loop<4, 2, 4, 4>(acc, s0, s1, s2, s3, wc, src, weight, dst, 4 * wn * 64 + lane, (kWideTileBands + 2 * wm) * 64 + lane,
                        (kWideTileBands + kWideTileGroups + 2 * wm) * 64 + lane, k0, k1, k1 - k0, k1 - k0);
  // C layout: register j of lane l = row l%32 of the group, output feature 8*(j/4) + 4*(l/32) + j%4
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int band = nt * kWideTileBands + 4 * wn + i;
    if (band >= n_bands) continue;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int row = (mt * kWideTileGroups + 2 * wm + g) * 32 + (lane & 31);
      if (row >= rows) continue;
      if (SWIGLU) {
        const float rs = rms[(2 * wm + g) * 32 + (lane & 31)];
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = swiglu_act(acc[i][g][4 * q + e], acc[i][g][4 * q + 4 + e], rs);
          store_planes4(y, sw.t, sw.t_lo, packed_act_offset(row, band * 16 + 4 * q + 4 * (lane >> 5), nb));
        }
        continue;
      }
      float *dst = part + part_offset(s, row, band * 32 + 4 * (lane >> 5), n_bands, rows_pad);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4 *>(dst + 8 * q) =
            make_float4(acc[i][g][4 * q], acc[i][g][4 * q + 1], acc[i][g][4 * q + 2], acc[i][g][4 * q + 3]);
    }
  }
}

int wide_row_groups(int rows) { return (rows + 32 * kWideTileGroups - 1) / (32 * kWideTileGroups) * kWideTileGroups; }

// k-split S of a wide GEMM (any integer, each split >= 8 k-steps), from a cost model fitted to
// measurements on MI355X (7B shapes at 256 and 512 rows), in microseconds.  One workgroup keeps
// the matrix cores of its compute unit almost busy by itself, so a compute unit works its
// workgroups off one after the other in effect: 18 us for launch, pipeline fill and the last
// epilogue, 0.33 us per k-step (0.28 while fewer workgroups than compute units run), 6 us per
// further workgroup on the same compute unit, and every split writes the output once as fp32
// partial sums that the consumer reads again (0.3 us per MB + 0.5 us per split).  What this mostly decides is how
// many rounds of workgroups a launch takes: gate|up at 512 rows of the 7B model has 344 tiles on
// 256 compute units: S = 1 187 us, S = 2 162 us, S = 4 183 us.
static double wide_gemm_cost(int n_bands, int ksteps, int rows, int n_cu, int S) {
  const int64_t tiles = (int64_t)((n_bands + kWideTileBands - 1) / kWideTileBands) * (wide_row_groups(rows) / kWideTileGroups);
  const double out_mb = (double)n_bands * 32 * part_rows_pad(rows) * 4 / 1e6;
  const int64_t wgs = tiles * S, per_cu = (wgs + n_cu - 1) / n_cu;
  const double len = (double)ksteps / S, tk = wgs >= n_cu ? 0.33 : 0.28;
  return 18.0 + per_cu * len * tk + (per_cu - 1) * 6.0 + S * (out_mb * 0.3 + 0.5);
}

int wide_gemm_splits(int n_bands, int ksteps, int rows, int n_cu) {
  int best = 1;
  double best_cost = 1e300;
  for (int S = 1; S <= 16 && ksteps / S >= 8; ++S) {
    const double cost = wide_gemm_cost(n_bands, ksteps, rows, n_cu, S);
    if (cost < best_cost) { best_cost = cost; best = S; }
  }
  return best;
}

template <int STAGE, bool SWIGLU = false>
static void launch_gemm_wide_s(const PackedMatrix &W, const uint16_t *Xp, int rows, float *part,
                               int n_splits, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1,
                               const WideSwiglu &sw = WideSwiglu{}) {
  const int nb = wide_row_groups(rows);
  const int n_nt = (W.n_bands + kWideTileBands - 1) / kWideTileBands;
  const unsigned grid = ((unsigned)(nb / kWideTileGroups) * n_nt * n_splits + 7u) / 8u * 8u;
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL((gemm_wide_kernel<STAGE, SWIGLU>), dim3(grid), dim3(256), 0u, st, ev0, ev1, 0u, (const u32x4 *)W.data,
                          (const u32x4 *)Xp, part, rows, part_rows_pad(rows), W.n_bands, W.ksteps, nb, n_splits, sw);
  else
    gemm_wide_kernel<STAGE, SWIGLU><<<grid, 256, 0, st>>>((const u32x4 *)W.data, (const u32x4 *)Xp, part, rows, part_rows_pad(rows), W.n_bands, W.ksteps, nb, n_splits, sw);
}

// gate|up with the SwiGLU epilogue (unsplit): planes t / t_lo of silu(gate) * up
void launch_gemm_wide_swiglu(const PackedMatrix &W, const uint16_t *Xp, int rows, const RowNorm &nrm, uint16_t *t,
                             uint16_t *t_lo, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  launch_gemm_wide_s<2, true>(W, Xp, rows, nullptr, 1, st, ev0, ev1, WideSwiglu{nrm, t, t_lo});
}

void launch_gemm_wide(const PackedMatrix &W, const uint16_t *Xp, int rows, float *part, int n_splits,
                      int stage, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  switch (stage) {
    case 0: launch_gemm_wide_s<0>(W, Xp, rows, part, n_splits, st, ev0, ev1); break;
    case 1: launch_gemm_wide_s<1>(W, Xp, rows, part, n_splits, st, ev0, ev1); break;
    case 2: launch_gemm_wide_s<2>(W, Xp, rows, part, n_splits, st, ev0, ev1); break;
    case 3: launch_gemm_wide_s<3>(W, Xp, rows, part, n_splits, st, ev0, ev1); break;
    default: launch_gemm_wide_s<4>(W, Xp, rows, part, n_splits, st, ev0, ev1); break;
  }
}

// --------------------------------------------------------------------------- wide gate|up, k halved inside the workgroup
// gate|up for hundreds of rows where the tiled kernel above needs two k-splits to fill its rounds of workgroups: there the
// fp32 partial sums of both (7B, 810 rows: 146 MB) are written, read again by a SwiGLU kernel, and cost as much as a
// fifth of the products.  Here one workgroup of 8 wavefronts takes A bands x 4 row groups and ALL of k: wavefronts 0 .. 3
// the first half, 4 .. 7 the second, each half with its own ring in LDS, so the addition chains are those of two
// splits.  At the end the halves exchange half of their tiles through LDS, every wavefront finishes the tiles it
// keeps, and SwiGLU happens in registers as in the tiled kernel.
// What bounds it: MFMAs with random data run at a throttled 0.020 us each per SIMD (1.6 GHz; 10 bands 0.80 us per
// step of both halves) and share power and L2 with the copies; measured 0.9.  10 bands: 5 x 2 tiles per wavefront, 160
// accumulators, ring of 3 (of 4: 4 % slower); 8 bands: 4 x 2, ring of 4.
// Measured, GEMM + SwiGLU kernel before -> this, us: 7B 320 rows 150 + 16 -> 125, 768 rows 258 + 29 -> 238, 810 rows 287 + 31 ->
// 254; 13B 640 rows 325 + 36 -> 300, 810 rows 484 -> 396, 1024 rows 477 + 59 -> 457; 1.1B 810 rows 88 + 18 -> 72.  Prefill of
// 810 positions, 7B: 23.8 -> 22.3 ms.
constexpr int kPairGroups = 4;  // row groups per workgroup

template <int A> struct PairShape {
  static constexpr int D = A == 10 ? 3 : 4;                // ring stages of one k-step per half
  static constexpr int tiles = A + 2 * kPairGroups;        // 1 KB tiles per stage and half
  static constexpr int copies = (tiles + 3) / 4;           // per wavefront; surplus ones repeat the last tile
};

// grid 8 * per_xcd, block 512.  An XCD (workgroup index mod 8) owns a contiguous run of tiles, the row tiles of one
// feature tile next to each other.
template <int A>
__global__ __launch_bounds__(512, 2) void gemm_wide_pair_kernel(const u32x4 *__restrict__ Wp, const u32x4 *__restrict__ Xp, int rows, int n_bands,
                                                                int ksteps, int nb, int n_mt, int total, int per_xcd, WideSwiglu sw) {
  constexpr int D = PairShape<A>::D, T = PairShape<A>::tiles, C = PairShape<A>::copies, B = kPairGroups, a = A / 2, b = B / 2;
  static_assert(A % 2 == 0 && T % 2 == 0 && (D == 3 || D == 4), "wavefront grid 2 x 2, ring");
  // separate arrays: the compiler can tell a copy into one from the reads of another
  __shared__ u32x4 s0[2 * T * 64], s1[2 * T * 64], s2[2 * T * 64], s3[D > 3 ? 2 * T * 64 : 1];
  __shared__ float rms[32 * B];
  const int wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int half = wave8 >> 2, wave = wave8 & 3, wn = wave & 1, wm = wave >> 1;
  const int slot = blockIdx.x >> 3, id = (blockIdx.x & 7) * per_xcd + slot;
  if (slot >= per_xcd || id >= total) return;
  const int mt = (uint32_t)id % (uint32_t)n_mt, nt = (uint32_t)id / (uint32_t)n_mt;
  const int n_groups = (rows + 31) >> 5;
  const int len = (ksteps + 1) / 2;                            // steps of the first half; the second has as many or one less
  const int k0 = half * len, k1 = half ? ksteps : len;
  // the tiles this wavefront copies per stage (bands and row groups past the edge repeat the last one, unused)
  const char *src[C];
  bool weight[C];
  int dst[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int ti = min(wave * C + i, T - 1), plane = ti - A >= B, g = ti - A - plane * B;
    weight[i] = ti < A;
    dst[i] = half * T + ti;
    src[i] = ti < A ? (const char *)(Wp + (int64_t)min(nt * A + ti, n_bands - 1) * ksteps * 64)
                    : (const char *)(Xp + plane * ((int64_t)ksteps * nb * 64) + (int64_t)min(mt * B + g, n_groups - 1) * 64);
  }
  const WideCopy wc{(uint32_t)ksteps, (uint32_t)nb, (uint32_t)lane * 16};
  f32x16 acc[a][b];
#pragma unroll
  for (int i = 0; i < a; ++i)
#pragma unroll
    for (int g = 0; g < b; ++g)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][g][j] = 0.f;
#pragma unroll
  for (int j = 0; j < D; ++j)
#pragma unroll
    for (int i = 0; i < C; ++i) wide_copy(wc, src, weight, dst, j == 0 ? s0 : j == 1 ? s1 : j == 2 ? s2 : s3, i, min(k0 + j, ksteps - 1));
#pragma unroll
  for (int r0 = 0; r0 < 32 * B; r0 += 64) {  // 1 / rms of the tile's rows, 8 threads per row, while the first stages arrive
    const int rl = r0 + (threadIdx.x >> 3);
    const float *sq = sw.nrm.ssq + (int64_t)min(mt * B * 32 + rl, rows - 1) * sw.nrm.n_slab;
    float ss = 0.f;
    for (int i = threadIdx.x & 7; i < sw.nrm.n_slab; i += 8) ss += sq[i];
    ss += __shfl_xor(ss, 1, 64);
    ss += __shfl_xor(ss, 2, 64);
    ss += __shfl_xor(ss, 4, 64);
    if ((threadIdx.x & 7) == 0) rms[rl] = 1.0f / sqrtf(ss / (float)sw.nrm.d + sw.nrm.eps);
  }
  const int at = half * T * 64 + lane;
  wide_loop<a, b, C, D>(acc, s0, s1, s2, s3, wc, src, weight, dst, at + a * wn * 64, at + (A + b * wm) * 64, at + (A + B + b * wm) * 64, k0, k1, ksteps / 2, len);
  __syncthreads();
  // Tiles 0 .. H-1 of a wavefront's tile are finished by the first half, the others by the second: each gives the partner
  // what it does not keep, HC tiles at a time (4 KB each in the ring's arrays).
  constexpr int H = a * b / 2, TA = T / 2, FIT = TA * D / 8, HC = H < FIT ? H : FIT;
  static_assert(HC > 0, "room for the exchange");
  auto slot_of = [&](int w8, int i) -> float4 * {
    const int q = w8 * HC + i, arr = q / TA, o = q - arr * TA;
    return reinterpret_cast<float4 *>((arr == 0 ? s0 : arr == 1 ? s1 : arr == 2 ? s2 : s3) + o * 256);
  };
#pragma unroll
  for (int t0 = 0; t0 < H; t0 += HC) {
    if (t0) __syncthreads();
#pragma unroll
    for (int i = t0; i < H && i < t0 + HC; ++i) {
      const f32x16 &lo = acc[i / b][i % b], &up = acc[(i + H) / b][(i + H) % b];
      float4 *dst = slot_of(wave8, i - t0) + lane;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        dst[q * 64] = half ? make_float4(lo[4 * q], lo[4 * q + 1], lo[4 * q + 2], lo[4 * q + 3]) : make_float4(up[4 * q], up[4 * q + 1], up[4 * q + 2], up[4 * q + 3]);
    }
    __syncthreads();
#pragma unroll
    for (int i = t0; i < H && i < t0 + HC; ++i) {
      const f32x16 &lo = acc[i / b][i % b], &up = acc[(i + H) / b][(i + H) % b];
      const float4 *other = slot_of(wave8 ^ 4, i - t0) + lane;
      float z[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 o = other[q * 64];
        z[4 * q] = (half ? up[4 * q] : lo[4 * q]) + o.x;
        z[4 * q + 1] = (half ? up[4 * q + 1] : lo[4 * q + 1]) + o.y;
        z[4 * q + 2] = (half ? up[4 * q + 2] : lo[4 * q + 2]) + o.z;
        z[4 * q + 3] = (half ? up[4 * q + 3] : lo[4 * q + 3]) + o.w;
      }
      // C layout: register j of lane l = row l%32 of the group, output feature 8*(j/4) + 4*(l/32) + j%4
      const int ti = half ? i + H : i, band = nt * A + a * wn + ti / b, rl = (b * wm + ti % b) * 32 + (lane & 31), row = mt * B * 32 + rl;
      if (band >= n_bands || row >= rows) continue;
      const float rs = rms[rl];
#pragma unroll
      for (int q = 0; q < 4; q += 2) {
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = swiglu_act(z[4 * q + e], z[4 * q + 4 + e], rs);
        store_planes4(y, sw.t, sw.t_lo, packed_act_offset(row, band * 16 + 4 * q + 4 * (lane >> 5), nb));
      }
    }
  }
}

// Bands per workgroup of the kernel above, or 0 where the tiled kernel (with `splits` k-splits and, if more than one, its
// SwiGLU kernel) is estimated faster.  All in us, fitted to 7B, 13B and 1.1B at 128 ..
// 1024 rows: 12 per launch; rounds of workgroups (one per compute unit) times half of the k-steps at 0.91 (10 bands) or 0.74
// (8 bands); the tiled kernel 0.38 per k-step of the workgroups that follow one another on a compute unit, its SwiGLU
// kernel 6 and 0.17 per MB of partial sums.  Measured, tiled kernel against this: 7B 256 rows 101 / 97, 512 rows 185 / 196,
// 640 rows 240 / 220, 810 rows 297 / 254; 13B 810 rows 470 / 395; 1.1B 640 rows 57 / 55.  More than two splits stay with the
// tiled kernel: their addition chains are shorter.
int plan_wide_pair(int n_bands, int ksteps, int rows, int splits, int n_cu, double *cost_us) {
  const int64_t mt = wide_row_groups(rows) / kWideTileGroups;
  auto rounds = [n_cu](int64_t wgs) { return (double)((wgs + n_cu - 1) / n_cu); };
  const double out_mb = (double)n_bands * 32 * rows * 4e-6;
  double limit = 12.0 + rounds((n_bands + kWideTileBands - 1) / kWideTileBands * mt * splits) * ksteps / splits * 0.38 + (splits > 1 ? 6.0 + 0.17 * splits * out_mb : 0.0);
  limit *= 0.98;
  if (splits > 2) return 0;
  int best = 0;
  for (const int a : {8, 10}) {
    const double cost = 12.0 + rounds((n_bands + a - 1) / a * mt) * (ksteps / 2.0) * (a == 10 ? 0.91 : 0.74);
    if (cost >= limit) continue;
    *cost_us = limit = cost;
    best = a;
  }
  return best;
}

void launch_gemm_wide_pair(const PackedMatrix &W, const uint16_t *Xp, int rows, int bands, const RowNorm &nrm, uint16_t *t, uint16_t *t_lo,
                           hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const int nb = wide_row_groups(rows), n_mt = nb / kPairGroups, total = n_mt * ((W.n_bands + bands - 1) / bands), per_xcd = (total + 7) / 8;
  const WideSwiglu sw{nrm, t, t_lo};
  const auto kernel = bands == 10 ? gemm_wide_pair_kernel<10> : gemm_wide_pair_kernel<8>;
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL(kernel, dim3(8u * per_xcd), dim3(512), 0u, st, ev0, ev1, 0u, (const u32x4 *)W.data, (const u32x4 *)Xp, rows, W.n_bands, W.ksteps, nb, n_mt, total, per_xcd, sw);
  else
    kernel<<<8u * per_xcd, 512, 0, st>>>((const u32x4 *)W.data, (const u32x4 *)Xp, rows, W.n_bands, W.ksteps, nb, n_mt, total, per_xcd, sw);
}

// --------------------------------------------------------------------------- consumers of partial sums
// RMSNorm is applied in two halves so that no kernel has to see a whole row: this kernel adds the
// pending partial sums to the residual stream, multiplies by the norm's gain and records the sum
// of squares of its 32-column slab; the consumer of the following GEMM multiplies that GEMM's
// output by 1/rms(row) (the GEMM is linear in its input, so W (g * x / rms) = (W (g * x)) / rms).
//   x[r][:]   += sum_s part[s][r][:]            (n_splits may be 0)
//   hb[r][:]   = hi/lo bf16 planes of x[r][:] * gain[:]
//   ssq[r][slab] = sum over the slab of x[r][c]^2
// Block = 8 threads per row (4 columns each, <= 64 rows), grid = (slabs of 32 columns, row blocks).
// Bound by one trip to memory and the launch: gain, x and all splits up to 3 are requested together (us per launch, with the last splits one
// by one and the gain behind the store of x -> now: 1.1B, 37 rows 3.6 -> 3.5, 13B, 160 rows 7.6 -> 7.2; 7B the same).
constexpr int kSlabCols = 32;
__global__ __launch_bounds__(512) void residual_gain_kernel(float *x, const float *part, int n_splits,
                                                            int rows, int ldp, const uint16_t *gain,
                                                            int d, uint16_t *hb, uint16_t *hb_lo,
                                                            int nb, float *ssq, int n_slab, int rows_pad) {
  const int r = blockIdx.y * 64 + (threadIdx.x >> 3), c = blockIdx.x * kSlabCols + (threadIdx.x & 7) * 4;
  const bool ok = r < rows && c < d;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  uint2 g = make_uint2(0u, 0u);
  float *xr = x + (int64_t)r * d + c;
  if (ok) {
    g = *reinterpret_cast<const uint2 *>(gain + c);
    v = *reinterpret_cast<const float4 *>(xr);
    const float *pp = part + part_offset(0, r, c, ldp >> 5, rows_pad);
    const int64_t sstride = (int64_t)ldp * rows_pad;
    add_splits4(v, pp, sstride, n_splits);
  }
  float ss = sum_squares4(v.x, v.y, v.z, v.w);
  ss += __shfl_xor(ss, 1, 64);
  ss += __shfl_xor(ss, 2, 64);
  ss += __shfl_xor(ss, 4, 64);
  if (ok) {  // all stores behind the sums: in front of them a wait for loads would be one for the store of x as well
    if (n_splits > 0) *reinterpret_cast<float4 *>(xr) = v;
    if ((threadIdx.x & 7) == 0) ssq[(int64_t)r * n_slab + blockIdx.x] = ss;
    const float y[4] = {v.x * bf16_bits_to_f32(g.x & 0xffffu), v.y * bf16_bits_to_f32(g.x >> 16),
                        v.z * bf16_bits_to_f32(g.y & 0xffffu), v.w * bf16_bits_to_f32(g.y >> 16)};
    store_planes4(y, hb, hb_lo, packed_act_offset(r, c, nb));
  }
}

int residual_slabs(int d) { return (d + kSlabCols - 1) / kSlabCols; }

// `rows_pad` = row padding of the partial-sum blocks; 0: that of `rows` (differs when x, part and
// ssq are views that start at a later row of a larger call).
void launch_residual_gain(float *x, const float *part, int n_splits, int rows, int ldp,
                          const void *gain, int d, uint16_t *hb, uint16_t *hb_lo, int nb, float *ssq,
                          hipStream_t st, int rows_pad) {
  const int n_slab = residual_slabs(d);
  if (rows_pad <= 0) rows_pad = part_rows_pad(rows);
  const int per_block = rows < 64 ? rows : 64;
  dim3 grid(n_slab, (rows + 63) / 64);
  residual_gain_kernel<<<grid, ((per_block + 7) / 8) * 64, 0, st>>>(x, part, n_splits, rows, ldp, (const uint16_t *)gain, d, hb, hb_lo, nb, ssq, n_slab, rows_pad);
}

// q, k, v = sum of partials; rotary embedding at the node's depth position (Sec. II-B: each
// branch is verified as its own sequence, so position = kv_len + depth).  Outputs: q either as
// fp32 [rows][H*hd] (generic attention) or as bf16 pre-multiplied by log2(e)/sqrt(hd) (MFMA
// attention); k, v -> bf16 cache slot kv_len + node.  Packed columns: [q | pad | k | pad | v]; with
// `paired` the rows of a query or key head are stored as launch_repack_rope leaves them.
__device__ __forceinline__ int rope_col(int j, int paired) { return paired ? ((j >> 3) << 4) + (j & 7) : j; }
__device__ __forceinline__ int rope_step(int half, int paired) { return paired ? 8 : half; }
__global__ __launch_bounds__(256) void qkv_finish_kernel(StepMeta m, KvGeom g, int layer, int H, int Hkv,
                                                         int hd, const float *part, int n_splits,
                                                         int ldp, RowNorm nrm, int col_k, int col_v,
                                                         const float2 *cs, float *q, uint16_t *qb,
                                                         uint16_t *qb_lo, float qscale, uint16_t *kc,
                                                         uint16_t *vc, int paired) {
  const int r = blockIdx.y, half = hd / 2, rows = m.rows;
  const int idx0 = blockIdx.x * 256 + threadIdx.x, n_items = (H + Hkv) * half;
  const bool live = idx0 < n_items;
  const int idx = live ? idx0 : n_items - 1;  // surplus threads of the last block repeat its last item, without stores
  const float lane_ssq = row_ssq_lane(nrm, r);
  const int a = idx / half, j = idx - a * half;
  const float2 c = cs[(int64_t)r * half + j];
  const int rows_pad = part_rows_pad(rows);
  const float *pr = part + part_offset(0, r, 0, ldp >> 5, rows_pad);  // column c at (c/32)*rows_pad*32 + c%32
  const int64_t sstride = (int64_t)ldp * rows_pad;
  auto at = [rows_pad](int col) { return (col >> 5) * (rows_pad << 5) + (col & 31); };
  // sums of the split-k partials of up to four columns, loads of one split issued together
  auto val4 = [&](int c0, int c1, int c2, int c3, float (&out)[4]) {
    out[0] = out[1] = out[2] = out[3] = 0.f;
#pragma unroll 4
    for (int s = 0; s < n_splits; ++s) {
      const float *q = pr + s * sstride;
      const float v0 = q[at(c0)], v1 = q[at(c1)], v2 = q[at(c2)], v3 = q[at(c3)];
      out[0] += v0; out[1] += v1; out[2] += v2; out[3] += v3;
    }
  };
  float t[4];
  const int jc = rope_col(j, paired), j2 = jc + rope_step(half, paired);
  if (a < H)
    val4(a * hd + jc, a * hd + j2, a * hd + jc, a * hd + j2, t);
  else
    val4(col_k + (a - H) * hd + jc, col_k + (a - H) * hd + j2, col_v + (a - H) * hd + j, col_v + (a - H) * hd + j + half, t);
  const float rs = row_rms_finish(nrm, lane_ssq);
  if (!live) return;
  t[0] *= rs; t[1] *= rs; t[2] *= rs; t[3] *= rs;
  if (a < H) {
    const float x0 = t[0], x1 = t[1];
    const float y0 = rotated_first(x0, x1, c.x, c.y), y1 = rotated_second(x0, x1, c.x, c.y);
    const int64_t o = ((int64_t)r * H + a) * hd + j;
    if (qb) {
      split_bf16(y0 * qscale, qb[o], qb_lo[o]);
      split_bf16(y1 * qscale, qb[o + half], qb_lo[o + half]);
    } else {
      q[o] = y0;
      q[o + half] = y1;
    }
  } else {
    const int b = a - H;
    const float x0 = t[0], x1 = t[1];
    const int64_t base = g.row(m.seq[r], layer, b, m.slot[r]);
    kc[base + j] = f32_to_bf16_bits(rotated_first(x0, x1, c.x, c.y));
    kc[base + j + half] = f32_to_bf16_bits(rotated_second(x0, x1, c.x, c.y));
    vc[base + j] = f32_to_bf16_bits(t[2]);
    vc[base + j + half] = f32_to_bf16_bits(t[3]);
  }
}

// The same for many rows (a wide pass, bf16 queries for the MFMA attention): one workgroup per
// (head, group of 32 rows); thread t takes row t/8 and the rotary pairs j = 4*(t%8)..+3 (+32 per
// further band of the half head), so that every load is 16 bytes per thread out of a contiguous
// 4 KB band block and every store 8 bytes of 4 consecutive bf16.
// Bound by its trips to memory, one after the other: statistics, then the splits of each half.  Cache slots travel with the first splits, and up to 3
// splits together (us per launch, slots behind the sums and the last n % 4 splits one by one -> now: 7B, 4 x 24 rows 8.9 -> 7.3, 2 x 64 11.8 -> 11.1;
// 1.1B, 330 rows 6.3 -> 5.7, 384 6.5 -> 5.9, 1024 16.9 -> 15.7; 13B, 4 x 40 11.3 -> 10.0, 2 x 40, 4 splits, 9.35 -> 9.5).
__global__ __launch_bounds__(256) void qkv_finish_wide_kernel(StepMeta m, KvGeom g, int layer, int H, int Hkv,
                                                              int hd, const float *part, int n_splits,
                                                              int ldp, RowNorm nrm, int col_k, int col_v,
                                                              const float2 *cs, uint16_t *qb,
                                                              uint16_t *qb_lo, float qscale, uint16_t *kc,
                                                              uint16_t *vc, int paired) {
  const int rows = m.rows, half = hd / 2;
  const int a = blockIdx.x, r = blockIdx.y * 32 + (threadIdx.x >> 3), sub = threadIdx.x & 7;
  const int rr = r < rows ? r : rows - 1;
  float ss = 0.f;
  {
    const float *sq = nrm.ssq + (int64_t)rr * nrm.n_slab;
    int i = sub;
    for (; i + 56 < nrm.n_slab; i += 64) {  // 8 independent loads in flight
      const float a0 = sq[i], a1 = sq[i + 8], a2 = sq[i + 16], a3 = sq[i + 24];
      const float a4 = sq[i + 32], a5 = sq[i + 40], a6 = sq[i + 48], a7 = sq[i + 56];
      ss += ((a0 + a1) + (a2 + a3)) + ((a4 + a5) + (a6 + a7));
    }
    for (; i < nrm.n_slab; i += 8) ss += sq[i];
  }
  ss += __shfl_xor(ss, 1, 64);
  ss += __shfl_xor(ss, 2, 64);
  ss += __shfl_xor(ss, 4, 64);
  const float rs = 1.0f / sqrtf(ss / (float)nrm.d + nrm.eps);
  if (r >= rows) return;
  const int rows_pad = part_rows_pad(rows), n_bands = ldp >> 5;
  int seq = m.seq[r], slot = m.slot[r];  // in flight together with the partial sums
  auto sum4 = [&](int col) {  // sum over the splits of 4 consecutive columns of row r, times 1/rms
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    add_splits4(v, part + part_offset(0, r, col, n_bands, rows_pad), (int64_t)ldp * rows_pad, n_splits);
    v.x *= rs; v.y *= rs; v.z *= rs; v.w *= rs;
    return v;
  };
  const bool is_q = a < H;
  const int b = a - H;
  const int c0 = is_q ? a * hd : col_k + b * hd;
  for (int j = sub * 4; j < half; j += 32) {
    const int jc = rope_col(j, paired);
    const float4 x0 = sum4(c0 + jc), x1 = sum4(c0 + jc + rope_step(half, paired));
    const float4 cs01 = *reinterpret_cast<const float4 *>(cs + (int64_t)r * half + j);       // (cos, sin) of j, j+1
    const float4 cs23 = *reinterpret_cast<const float4 *>(cs + (int64_t)r * half + j + 2);   // ... of j+2, j+3
    const float co[4] = {cs01.x, cs01.z, cs23.x, cs23.z}, si[4] = {cs01.y, cs01.w, cs23.y, cs23.w};
    const float a0[4] = {x0.x, x0.y, x0.z, x0.w}, a1[4] = {x1.x, x1.y, x1.z, x1.w};
    float y0[4], y1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      y0[i] = rotated_first(a0[i], a1[i], co[i], si[i]);
      y1[i] = rotated_second(a0[i], a1[i], co[i], si[i]);
    }
    if (is_q) {
      const int64_t o = ((int64_t)r * H + a) * hd + j;
#pragma unroll
      for (int i = 0; i < 4; ++i) { y0[i] *= qscale; y1[i] *= qscale; }
      store_planes4(y0, qb, qb_lo, o);
      store_planes4(y1, qb, qb_lo, o + half);
    } else {
      const float4 v0 = sum4(col_v + b * hd + j), v1 = sum4(col_v + b * hd + j + half);
      asm volatile("" : "+v"(seq), "+v"(slot));  // waited for here, not in front of the sums
      const int64_t base = g.row(seq, layer, b, slot);
      store_bf16x4(y0, kc + base + j);
      store_bf16x4(y1, kc + base + j + half);
      const float w0[4] = {v0.x, v0.y, v0.z, v0.w}, w1[4] = {v1.x, v1.y, v1.z, v1.w};
      store_bf16x4(w0, vc + base + j);
      store_bf16x4(w1, vc + base + j + half);
    }
  }
}

void launch_qkv_finish(const StepMeta &m, const ModelDims &md, const KvGeom &g, int layer,
                       const float *part, int n_splits, int ldp, const RowNorm &nrm, int col_k,
                       int col_v, const float2 *cs, float *q, uint16_t *qb, uint16_t *qb_lo, void *kc,
                       void *vc, bool paired, hipStream_t st) {
  if (m.rows > 64 && qb != nullptr && md.head_dim % 64 == 0) {
    dim3 wgrid(md.n_heads + md.n_kv_heads, (m.rows + 31) / 32);
    qkv_finish_wide_kernel<<<wgrid, 256, 0, st>>>(m, g, layer, md.n_heads, md.n_kv_heads, md.head_dim, part, n_splits, ldp, nrm, col_k, col_v, cs, qb, qb_lo, tree_attention_qscale(md.head_dim), (uint16_t *)kc, (uint16_t *)vc, paired ? 1 : 0);
    return;
  }
  const int items = (md.n_heads + md.n_kv_heads) * (md.head_dim / 2);
  dim3 grid((items + 255) / 256, m.rows);
  qkv_finish_kernel<<<grid, 256, 0, st>>>(m, g, layer, md.n_heads, md.n_kv_heads, md.head_dim, part, n_splits, ldp, nrm, col_k, col_v, cs, q, qb, qb_lo, tree_attention_qscale(md.head_dim), (uint16_t *)kc, (uint16_t *)vc, paired ? 1 : 0);
}

// t[r][f] = bf16 planes of silu(sum_s gate) * (sum_s up); gate at column 16*(f/8) + f%8, up 8 columns
// further (launch_repack_gate_up).
__device__ __forceinline__ int gate_col(int f) { return ((f >> 3) << 4) + (f & 7); }
// One workgroup per (band of 32 features, group of 32 rows): in the partial-sum layout that is one
// contiguous 4 KB block of gate and one of up per split, read with 16 bytes per thread (thread t:
// row t/8, features 4*(t%8)..+3), and one contiguous 1 KB block per k-step and plane on the way
// out.  The 8 threads of a row also share the sum over its norm slabs.
__global__ __launch_bounds__(256) void swiglu_finish_kernel(const float *part, int n_splits, int rows,
                                                            int ldp, RowNorm nrm, int F,
                                                            uint16_t *t, uint16_t *t_lo, int nb) {
  const int r = blockIdx.y * 32 + (threadIdx.x >> 3), sub = threadIdx.x & 7;
  const int f = blockIdx.x * 32 + sub * 4;
  const bool ok = r < rows && f < F;
  const int rr = r < rows ? r : rows - 1;
  // 1 / rms of the row: the 8 threads of a row add up its slab sums of squares
  float ss = 0.f;
  {
    const float *sq = nrm.ssq + (int64_t)rr * nrm.n_slab;
    int i = sub;
    for (; i + 56 < nrm.n_slab; i += 64) {  // 8 independent loads in flight
      const float a0 = sq[i], a1 = sq[i + 8], a2 = sq[i + 16], a3 = sq[i + 24];
      const float a4 = sq[i + 32], a5 = sq[i + 40], a6 = sq[i + 48], a7 = sq[i + 56];
      ss += ((a0 + a1) + (a2 + a3)) + ((a4 + a5) + (a6 + a7));
    }
    for (; i < nrm.n_slab; i += 8) ss += sq[i];
  }
  ss += __shfl_xor(ss, 1, 64);
  ss += __shfl_xor(ss, 2, 64);
  ss += __shfl_xor(ss, 4, 64);
  const float rs = 1.0f / sqrtf(ss / (float)nrm.d + nrm.eps);
  if (!ok) return;
  float4 gt = make_float4(0.f, 0.f, 0.f, 0.f), up = gt;
  const int rows_pad = part_rows_pad(rows), n_bands = ldp >> 5;
#pragma unroll 4
  for (int s = 0; s < n_splits; ++s) {
    const float4 a = *reinterpret_cast<const float4 *>(part + part_offset(s, r, gate_col(f), n_bands, rows_pad));
    const float4 b = *reinterpret_cast<const float4 *>(part + part_offset(s, r, gate_col(f) + 8, n_bands, rows_pad));
    gt.x += a.x; gt.y += a.y; gt.z += a.z; gt.w += a.w;
    up.x += b.x; up.y += b.y; up.z += b.z; up.w += b.w;
  }
  const float y[4] = {swiglu_act(gt.x, up.x, rs), swiglu_act(gt.y, up.y, rs), swiglu_act(gt.z, up.z, rs), swiglu_act(gt.w, up.w, rs)};
  store_planes4(y, t, t_lo, packed_act_offset(r, f, nb));
}

// The same for one row group (<= 32 rows): one workgroup per (1024 features, row), one sum over the
// norm slabs per wavefront -- with so few rows the band-block mapping above re-reads the slab sums
// too often (7B, 32 rows: 5.5 against 6.8 us; from 33 rows on the band-block mapping wins: 7B, 64
// rows 5.17 -> 5.11 ms per step).
__global__ __launch_bounds__(256) void swiglu_finish_rows_kernel(const float *part, int n_splits, int rows,
                                                            int ldp, RowNorm nrm, int F,
                                                            uint16_t *t, uint16_t *t_lo, int nb) {
  const int r = blockIdx.y;
  const int f = (blockIdx.x * 256 + threadIdx.x) * 4;
  const float lane_ssq = row_ssq_lane(nrm, r);
  float4 gt = make_float4(0.f, 0.f, 0.f, 0.f), up = gt;
  const int rows_pad = part_rows_pad(rows), n_bands = ldp >> 5;
  if (f < F) {
#pragma unroll 4
    for (int s = 0; s < n_splits; ++s) {
      const float4 a = *reinterpret_cast<const float4 *>(part + part_offset(s, r, gate_col(f), n_bands, rows_pad));
      const float4 b = *reinterpret_cast<const float4 *>(part + part_offset(s, r, gate_col(f) + 8, n_bands, rows_pad));
      gt.x += a.x; gt.y += a.y; gt.z += a.z; gt.w += a.w;
      up.x += b.x; up.y += b.y; up.z += b.z; up.w += b.w;
    }
  }
  const float rs = row_rms_finish(nrm, lane_ssq);
  if (f >= F) return;
  const float y[4] = {swiglu_act(gt.x, up.x, rs), swiglu_act(gt.y, up.y, rs), swiglu_act(gt.z, up.z, rs), swiglu_act(gt.w, up.w, rs)};
  store_planes4(y, t, t_lo, packed_act_offset(r, f, nb));
}

void launch_swiglu_finish(const float *part, int n_splits, int rows, int ldp, const RowNorm &nrm,
                          int F, uint16_t *t, uint16_t *t_lo, int nb, hipStream_t st) {
  if (rows <= 32) {
    dim3 grid((F / 4 + 255) / 256, rows);
    swiglu_finish_rows_kernel<<<grid, 256, 0, st>>>(part, n_splits, rows, ldp, nrm, F, t, t_lo, nb);
    return;
  }
  dim3 grid((F + 31) / 32, (rows + 31) / 32);
  swiglu_finish_kernel<<<grid, 256, 0, st>>>(part, n_splits, rows, ldp, nrm, F, t, t_lo, nb);
}

// fp32 -> bf16 row conversion (attention output feeding the output projection)
__global__ void to_bf16_kernel(const float *src, int64_t n, int K, int nb, uint16_t *dst, uint16_t *dst_lo) {
  int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= n) return;
  const float4 v = *reinterpret_cast<const float4 *>(src + i);
  const float y[4] = {v.x, v.y, v.z, v.w};
  uint16_t hi[4], lo[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) split_bf16(y[k], hi[k], lo[k]);
  const int64_t po = packed_act_offset((int)(i / K), (int)(i % K), nb);
  *reinterpret_cast<uint2 *>(dst + po) =
      make_uint2((uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16));
  *reinterpret_cast<uint2 *>(dst_lo + po) =
      make_uint2((uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16));
}

// row-major fp32 [rows][K] -> packed hi/lo planes
void launch_to_bf16(const float *src, int rows, int K, uint16_t *dst, uint16_t *dst_lo, hipStream_t st) {
  const int64_t n = (int64_t)rows * K;
  to_bf16_kernel<<<(unsigned)((n / 4 + 255) / 256), 256, 0, st>>>(src, n, K, rows <= 32 ? 1 : 2, dst, dst_lo);
}

// logits[r][v] = sum_s part[s][r][v]; per-(row, block) best (value, lowest index); optional
// store of the logits into the caller's padded array.  The acceptance kernel, or a second tiny one, merges the blocks.
__global__ __launch_bounds__(256) void logits_argmax_kernel(StepMeta m, const float *part, int n_splits,
                                                            int ldp, RowNorm nrm, int V,
                                                            int max_nodes, float *logits_out,
                                                            float2 *rec) {
  __shared__ float bv[4];
  __shared__ int bi[4];
  const int r = blockIdx.y, rows = m.rows;
  const int v0 = (blockIdx.x * 256 + threadIdx.x) * 4;
  const float rs = row_rms_scale(nrm, r);
  float best = -INFINITY;
  int besti = 0x7fffffff;
  if (v0 < V) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < n_splits; ++s) {
      const float4 p = *reinterpret_cast<const float4 *>(part + part_offset(s, r, v0, ldp >> 5, part_rows_pad(rows)));
      a.x += p.x; a.y += p.y; a.z += p.z; a.w += p.w;
    }
    const float vals[4] = {a.x * rs, a.y * rs, a.z * rs, a.w * rs};
    if (logits_out) {
      float *dst = logits_out + ((int64_t)m.seq[r] * max_nodes + m.node[r]) * V + v0;
      for (int i = 0; i < 4; ++i)
        if (v0 + i < V) dst[i] = vals[i];
    }
    for (int i = 0; i < 4; ++i)
      if (v0 + i < V && vals[i] > best) { best = vals[i]; besti = v0 + i; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(besti, o, 64);
    if (ov > best || (ov == best && oi < besti)) { best = ov; besti = oi; }
  }
  if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = besti; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (bv[w] > best || (bv[w] == best && bi[w] < besti)) { best = bv[w]; besti = bi[w]; }
    rec[(int64_t)r * gridDim.x + blockIdx.x] = make_float2(best, __int_as_float(besti));
  }
}

__global__ __launch_bounds__(64) void argmax_merge_kernel(StepMeta m, const float2 *rec, int n_blk, int max_nodes, int32_t *argmax) {
  const int r = blockIdx.x;
  float best = -INFINITY;
  int besti = 0x7fffffff;
  for (int b = threadIdx.x; b < n_blk; b += 64) {
    const float2 q = rec[(int64_t)r * n_blk + b];
    const float v = q.x;
    const int i = __float_as_int(q.y);
    if (v > best || (v == best && i < besti)) { best = v; besti = i; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(besti, o, 64);
    if (ov > best || (ov == best && oi < besti)) { best = ov; besti = oi; }
  }
  if (threadIdx.x == 0) argmax[m.seq[r] * max_nodes + m.node[r]] = besti == 0x7fffffff ? 0 : besti;
}

int logits_argmax_blocks(int V) { return ((V + 3) / 4 + 255) / 256; }

void launch_logits_argmax(const StepMeta &m, const float *part, int n_splits, int ldp,
                          const RowNorm &nrm, int V, int max_nodes, float *logits_out, float2 *rec,
                          int32_t *argmax, hipStream_t st) {
  const int n_blk = logits_argmax_blocks(V);
  dim3 grid(n_blk, m.rows);
  logits_argmax_kernel<<<grid, 256, 0, st>>>(m, part, n_splits, ldp, nrm, V, max_nodes, logits_out, rec);
  if (argmax != nullptr) argmax_merge_kernel<<<m.rows, 64, 0, st>>>(m, rec, n_blk, max_nodes, argmax);
}

}  // namespace specasr
