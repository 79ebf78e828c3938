// All decoder layers of a forward with at most 16 rows of one sequence in one launch, gfx950 (models up to the 1.1B class).
//
// As a chain of kernels such a forward is 6 dependent launches per layer, each 1.3 us of boundary plus the way of its first
// bytes: weights that could have been on their way are only asked for when the kernel before has drained.  Here workgroups
// stay: a workgroup takes an item (q|k|v, attention, o, gate|up or down of a layer, for a few output features or query
// rows), asks for ALL its weights and only then looks for its input.  They wait in registers: 1.1B, gate|up 256 KB, down 180, q|k|v 128, o 128
// up to 8 rows and 64 beyond, which is half of a workgroup's registers at most.
//
// Hand-over.  Between the workgroups of one launch nothing orders plain stores and loads, and fences cost more than a launch
// (15 us when every workgroup invalidates its caches).  So every datum carries its own readiness: the regions below are
// filled with ones before the launch, are written once, by stores of whole words that go through to memory, and a reader loads
// them past its caches until none of its words is all ones.  There is no flag, no counter, no order between two stores or between the
// words of one to rely on: every 4 bytes that have been read are checked themselves.  A word that would be all ones (NaN) is stored with
// its last bit cleared (ready_word).
//
// Progress.  Items are numbered in the order of their dependencies and handed out by one counter, so a workgroup only ever waits
// for items that running workgroups have taken before: any number of resident workgroups, also one, finishes the forward,
// whatever else runs on the chip.  Each wait is bounded all the same, at 2^21 looks, two to four seconds; a wait that is given up ends all
// others, what was computed without its data is NaN, and the library reports it.
//
// What bounds it: a layer is 5 phases that wait for each other, 24 us together with one row and 29 with 16 where its weights need 14 (each the store to
// memory, 0.7, the look that finds it, 1, products, sums through LDS and epilogue, 1.5, and the latest workgroup), and at the last of them the
// weights that 48 workgroups could not ask for earlier.
// Measured (us per draft forward, chain of kernels -> this): 1.1B, 330 keys, 1 row 940 -> 609, 8 rows 946 -> 640, 16 rows 1014 -> 718; 3200 keys,
// 1 row 1017 -> 700, 8 rows 1072 -> 744, 16 rows 1115 -> 876; 12 layers of d 1024, 1 row 466 -> 310; 2 layers of d 256, 8 rows, 1160 keys 80 -> 62.  No
// combination of 1 .. 32 KV heads, d 64 .. 2048, 1 .. 16 rows and 0 .. 4000 keys is slower than the chain.  The variants named below are of the same
// state and unit.
#include "kernels.h"
#include "kernels_mfma.h"
#include "kernels_one.h"
#include "attn_tile.h"

namespace specasr {

typedef __attribute__((ext_vector_type(4))) float f32x4;

typedef __attribute__((address_space(1))) u32x4 global_u32x4;  // (a pointer out of the table is generic otherwise, and its loads flat)

constexpr int kOneWaves = 8, kOneThreads = kOneWaves * 64;
// Half-bands of an item.  Two phases that follow each other should fit the 256 workgroups, so that the weights of the second are on
// their way before its input exists: 1.1B 80 + 4 items, 64 (9 .. 16 rows 128), 176 and 128.  With half as many features per item
// (160, 128, 235, 128) late workgroups ask for 180 KB when everything else waits for them: 330 keys, 1 row 609 -> 671, 16 rows 718 -> 768.
constexpr int kHbQkv = 2, kHbGu = 4, kHbDn = 1;
constexpr int one_hb_o(int np) { return np == 1 ? 2 : 1; }  // 1 row 609 (2), 638 (1); 16 rows 330 keys 699, 718, 3200 keys 915, 876
constexpr int kOneSums = 4 * kOneWaves * 64;  // float4 of the sums of up to 4 half-bands
constexpr int kOneHd = 64;
constexpr int kTU = 32 * kOneHd / 8;          // 16-byte units of a key tile
constexpr int kOneKeys = 4096, kChunkTiles = 16;  // cached keys of a call at most; tiles of a chunk at least, where there are several
constexpr int kMaxChunks = 8;                     // so many chunks are in flight in one_merge, and have room in the scratch
static_assert((kOneKeys / 32 + kChunkTiles - 1) / kChunkTiles <= kMaxChunks, "every prefix that is taken fits");

typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kThrough = 17;  // cache policy sc0 sc1: past the caches (sc1 alone is as fast)

__device__ __forceinline__ u32x4 ll_load16(rsrc_t r, uint32_t off) { return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kThrough)); }
__device__ __forceinline__ uint32_t ll_load4(rsrc_t r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kThrough); }
__device__ __forceinline__ bool missing16(const u32x4 &v) { return max(max(v[0], v[1]), max(v[2], v[3])) == ~0u; }  // any word
__device__ __forceinline__ void ll_store8(rsrc_t r, uint32_t off, uint32_t a, uint32_t b) {
  typedef __attribute__((ext_vector_type(2))) uint32_t u2;
  __builtin_amdgcn_raw_buffer_store_b64((u2){ready_word(a), ready_word(b)}, r, off, 0, kThrough);
}
__device__ __forceinline__ void ll_store4(rsrc_t r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(ready_word(__float_as_uint(v)), r, off, 0, kThrough);
}
__device__ __forceinline__ void ll_store_f4(rsrc_t r, uint32_t off, const float (&y)[4]) {
  ll_store8(r, off, __float_as_uint(y[0]), __float_as_uint(y[1]));
  ll_store8(r, off + 8, __float_as_uint(y[2]), __float_as_uint(y[3]));
}
// planes of 4 values, `plane` bytes apart
__device__ __forceinline__ void ll_store_planes(rsrc_t r, uint32_t off, uint32_t plane, const float (&y)[4]) {
  uint32_t h0, h1, l0, l1;
  split_bf16_pair(y[0], y[1], h0, l0);
  split_bf16_pair(y[2], y[3], h1, l1);
  ll_store8(r, off, h0, h1);
  ll_store8(r, off + plane, l0, l1);
}
// byte offset of columns col .. col+3 of a row in planes of rp rows: [k / 8][row][8]
__device__ __forceinline__ uint32_t act_off(int row, int col, int rp) { return ((uint32_t)(col >> 3) * rp + row) * 16 + (col & 4) * 2; }

// true: stop waiting.  The first to give up tells the others, and the host.
__device__ __forceinline__ bool give_up(const OneArgs &p, int it) {
  asm volatile("" ::: "memory");
  if (it >= p.polls) {
    __hip_atomic_store(p.ctl + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p.gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return true;
  }
  return (it & 255) == 255 && __hip_atomic_load(p.ctl + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

__device__ __forceinline__ void barrier_only() {  // loads in flight stay in flight
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

enum OneEpi { kOneQkv, kOneSwiglu, kOneResid };

struct OneShared {
  float4 sums[2][kOneSums];
  float rms[2][16];
  uint32_t next[2];
  float2 ml[kOneWaves * 32];
};

// What a wavefront knows of the item behind the current one.
struct Next {
  uint32_t ticket;
  __device__ __forceinline__ void ask(const OneArgs &p) {  // one thread; the answer is needed at the end of the item
    if (threadIdx.x == 0) ticket = __hip_atomic_fetch_add(p.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void publish(OneShared &sh, int par) {
    if (threadIdx.x == 0) sh.next[par] = ticket;
  }
};

// Item nt of a product with K inputs (k pairs of 32 per wavefront: at most LW): HB half-bands of 16 features, all rows.
// NP = 1: up to 8 rows, both planes in the 16 columns of one operand; 2: up to 16 rows.  Weights as the half-band GEMM reads them.
template <int EPI, int HB, int LW, int NP>
__device__ __forceinline__ void one_gemm(const OneArgs &p, OneShared &sh, int par, const void *W, int K, int n_half, int nt, int layer, rsrc_t rs,
                                         uint32_t x_off, uint32_t s_off, int n_slab, uint32_t res_in, rsrc_t ro, uint32_t out_hb, uint32_t out_x,
                                         uint32_t out_s, const uint16_t *gain, bool last) {
  constexpr int DX = HB > 2 && NP == 2 ? 4 : 8;                        // stages of activations asked for together
  constexpr int NA = NP == 2 ? 3 : LW > 8 ? 4 : 2;                     // accumulators: hi products in NA (- 1) chains, lo ones apart
  constexpr int NH = NP == 2 ? NA - 1 : NA;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t kp = (uint32_t)K >> 5;
  const int w0 = kp * wave / kOneWaves, len = (int)(kp * (wave + 1) / kOneWaves) - w0;
  const uint32_t ksteps = 2 * kp;
  const int end = max(len, 1) - 1;  // stages past the slice repeat its last one, unused
  const int in_tile = 32 * ((lane >> 4) & 1) + (lane & 15);
  // The o projection is taken two phases early, while the 180 KB that the last workgroups of down need are on their way: its weights
  // wait until the first queries are there (1 row 634 -> 609, 8 rows 669 -> 640, 16 rows 749 -> 718; the same for other phases only costs).
  // Up to 8 rows one wavefront looks for all (1 row 616 -> 609, 8 rows 647 -> 640; 16 rows the same either way).
  if (EPI == kOneResid && LW == 8) {
    if (NP == 2 || wave == 0)
      for (int it = 0; __ballot(!missing16(ll_load16(rs, p.lay.q + (uint32_t)(lane * 16) % (uint32_t)(p.dq * 2)))) == 0ull && !give_up(p, it); ++it)
        __builtin_amdgcn_s_sleep(NP == 2 ? 8 : 16);
    if (NP == 1) barrier_only();
  }
  u32x4 wa[LW][HB];
#pragma unroll
  for (int a = 0; a < HB; ++a) {
    const int hb = min(nt * HB + a, n_half - 1);
    const global_u32x4 *wp = (const global_u32x4 *)W + ((int64_t)(hb >> 1) * ksteps + 2 * w0 + (lane >> 5)) * 64 + in_tile + 16 * (hb & 1);
#pragma unroll
    for (int k = 0; k < LW; ++k) wa[k][a] = __builtin_nontemporal_load(wp + min(k, end) * 128);
  }
  __builtin_amdgcn_sched_barrier(0);

  // residual rows of the epilogue (wavefront a: half-band a, row lane % 16, columns 4 (lane / 16) .. +3); written two phases ago
  const int e_row = lane & 15, e_hb = nt * HB + wave, e_col = e_hb * 16 + (lane >> 4) * 4;
  const bool e_ok = EPI == kOneResid && wave < HB && e_row < p.rows && e_hb < n_half;
  u32x4 e_x = (u32x4){0, 0, 0, 0};
  uint2 e_g = make_uint2(0u, 0u);
  const uint32_t e_off = res_in + ((uint32_t)e_row * p.d + e_col) * 4;
  if (e_ok) {
    e_x = ll_load16(rs, e_off);
    e_g = *reinterpret_cast<const uint2 *>(gain + e_col);
  }

  // q|k|v epilogue: 32 threads per half-band take row q_r and 4 rotary pairs, first halves in quad q_qd, second halves in quad q_qd + 2
  const int q_qd = (threadIdx.x >> 4) & 1, q_r = threadIdx.x & 15;
  int q_kind = -1, q_j = 0;  // 0 query, 1 key, 2 value
  uint32_t q_off = 0;        // where the first 4 go in this layer's region ...
  uint16_t *q_cache = nullptr;  // ... and in the cache
  float4 q_c01 = make_float4(1.f, 0.f, 1.f, 0.f), q_c23 = q_c01;
  const int q_t = threadIdx.x >> 5;
  if (EPI == kOneQkv && q_t < HB && q_r < p.rows && nt * HB + q_t < n_half) {
    const int col = (nt * HB + q_t) * 16;
    int c = col;
    if (col < p.dq) q_kind = 0;
    else if (col >= p.col_k && col - p.col_k < p.Hkv * kOneHd) { q_kind = 1; c = col - p.col_k; }
    else if (col >= p.col_v && col - p.col_v < p.Hkv * kOneHd) { q_kind = 2; c = col - p.col_v; }
    const int in_head = c % kOneHd, q_head = c / kOneHd;
    q_j = (q_kind == 2 ? in_head : in_head / 2) + 4 * q_qd;
    if (q_kind == 0 || q_kind == 1) {
      const float4 *csp = reinterpret_cast<const float4 *>(p.cs + q_r * (kOneHd / 2) + q_j);
      q_c01 = csp[0];
      q_c23 = csp[1];
    }
    if (q_kind == 0) {
      q_off = p.lay.q + ((uint32_t)(q_r * p.H + q_head) * kOneHd + q_j) * 2;
    } else {
      q_off = (q_kind == 1 ? p.lay.kt : p.lay.vt) + ((uint32_t)(q_head * p.rp + q_r) * kOneHd + q_j) * 2;
      if (q_kind > 0) q_cache = (q_kind == 1 ? p.kc : p.vc) + p.g.row(0, layer, q_head, p.L + q_r) + q_j;
    }
  }
  float q_scale = p.qscale;
  const uint32_t dq_plane = (uint32_t)p.dq * 2 * p.rp, out_plane = (uint32_t)(EPI == kOneSwiglu ? p.F : p.d) * 2 * p.rp;
  uint32_t out_off = out_hb + (EPI == kOneSwiglu ? act_off(q_r, 8 * (nt * HB + q_t) + 4 * q_qd, p.rp) : act_off(e_row, e_col, p.rp));
  // computed here, not on the way out of the sums
  if (EPI == kOneQkv) asm volatile("" : "+v"(q_off), "+v"(q_cache), "+v"(q_kind), "+s"(q_scale));
  else asm volatile("" : "+v"(out_off));
  __builtin_amdgcn_sched_barrier(0);

  const int row = min(NP == 1 ? lane & 7 : lane & 15, p.rows - 1);
  const uint32_t plane = (uint32_t)K * 2 * p.rp, x_step = 64u * p.rp;
  const uint32_t x0 = x_off + ((uint32_t)(4 * w0 + (lane >> 4)) * p.rp + row) * 16 + (NP == 1 && (lane & 8) ? plane : 0);
  f32x4 acc[HB][NA];
#pragma unroll
  for (int a = 0; a < HB; ++a)
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[a][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  constexpr int RW = NP;  // rows of a wavefront in the norm: wave, wave + 8
  float ssum[RW];
  Next next;
  // A workgroup that is a phase ahead looks at one stage now and then, until that is there, and one wavefront looks for all of it:
  // the looks of 256 workgroups past the caches get in the way of the data (1 / 8 / 16 rows: each wavefront looks at a stage of its
  // own 634 / 659 / 763, one of them 609 / 640 / 718).
  if (wave == 0)
    for (int it = 0; __ballot(missing16(ll_load16(rs, x0))) != 0ull && !give_up(p, it); ++it) __builtin_amdgcn_s_sleep(24);
  barrier_only();
#pragma unroll
  for (int c0 = 0; c0 < LW; c0 += DX) {
    u32x4 xb[DX][NP];
    uint32_t sq[RW][4];
    const bool norm = EPI != kOneResid && c0 == 0;
    auto load_x = [&](int k) {
#pragma unroll
      for (int h = 0; h < NP; ++h) xb[k][h] = ll_load16(rs, x0 + min(c0 + k, end) * x_step + h * plane);
    };
    auto load_s = [&] {
#pragma unroll
      for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) sq[r][i] = wave + 8 * r < p.rows && lane + 64 * i < n_slab ? ll_load4(rs, s_off + ((wave + 8 * r) * n_slab + lane + 64 * i) * 4) : 0u;
    };
#pragma unroll
    for (int k = 0; k < DX; ++k)
      if (c0 + k < LW) load_x(k);
    if (norm) load_s();
    for (int it = 0;; ++it) {  // (all of them again: asking only for what is missing was slower)
      bool bad = false;
#pragma unroll
      for (int k = 0; k < DX; ++k)
        if (c0 + k < LW)
#pragma unroll
          for (int h = 0; h < NP; ++h) bad |= missing16(xb[k][h]);
      if (norm) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) bad |= sq[r][i] == ~0u;
      }
      if (__ballot(bad) == 0ull || give_up(p, it)) break;
#pragma unroll
      for (int k = 0; k < DX; ++k)
        if (c0 + k < LW) load_x(k);
      if (norm) load_s();
    }
    if (c0 == 0) next.ask(p);
    if (norm) {
#pragma unroll
      for (int r = 0; r < RW; ++r) ssum[r] = (__uint_as_float(sq[r][0]) + __uint_as_float(sq[r][1])) + (__uint_as_float(sq[r][2]) + __uint_as_float(sq[r][3]));
    }
#pragma unroll
    for (int k = 0; k < DX; ++k)
      if (c0 + k < LW && c0 + k < len)
#pragma unroll
        for (int h = 0; h < NP; ++h)
#pragma unroll
          for (int a = 0; a < HB; ++a) {
            f32x4 &z = acc[a][NP == 2 && h ? NA - 1 : (c0 + k) * NH / LW];
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[c0 + k][a]), __builtin_bit_cast(bf16x8, xb[k][h]), z, 0, 0, 0);
          }
  }
  if (EPI != kOneResid) {
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const float v = 1.0f / sqrtf(wave_sum(ssum[r]) / (float)p.d + p.eps);
      if (lane == 0) sh.rms[par][wave + 8 * r] = v;
    }
  }
  float4 *sums = sh.sums[par];
#pragma unroll
  for (int a = 0; a < HB; ++a) {
    f32x4 z = acc[a][0];
#pragma unroll
    for (int i = 1; i < NA; ++i) z += acc[a][i];
    sums[(a * kOneWaves + wave) * 64 + lane] = make_float4(z[0], z[1], z[2], z[3]);
  }
  next.publish(sh, par);
  __syncthreads();
  auto sum = [&](int t, int l) {
    auto add = [](const float4 &a, const float4 &b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
    auto slices = [&](const float4 *q) { return add(add(add(q[0], q[64]), add(q[128], q[192])), add(add(q[256], q[320]), add(q[384], q[448]))); };
    const float4 *src = sums + t * kOneWaves * 64 + l;
    if constexpr (NP == 1) {
      const float4 *hi = src - (l & 8);
      return add(slices(hi), slices(hi + 8));
    }
    return slices(src);
  };
  if (EPI == kOneSwiglu) {
    // half-band = gate features 8 hb .. +7, then the up features of the same index
    const int t = threadIdx.x >> 5, qd = (threadIdx.x >> 4) & 1, r = threadIdx.x & 15, hb = nt * HB + t;
    if (t < HB && r < p.rows && hb < n_half) {
      const float4 g = sum(t, qd * 16 + r), u = sum(t, (qd + 2) * 16 + r);
      const float v = sh.rms[par][r];
      const float y[4] = {swiglu_act(g.x, u.x, v), swiglu_act(g.y, u.y, v), swiglu_act(g.z, u.z, v), swiglu_act(g.w, u.w, v)};
      ll_store_planes(ro, out_off, out_plane, y);
    }
  } else if (EPI == kOneQkv) {
    if (q_kind >= 0) {
      const int r = q_r;
      const float4 a = sum(q_t, q_qd * 16 + r), b = sum(q_t, (q_qd + 2) * 16 + r);
      const float v = sh.rms[par][r];
      const float v0[4] = {a.x * v, a.y * v, a.z * v, a.w * v}, v1[4] = {b.x * v, b.y * v, b.z * v, b.w * v};
      const float co[4] = {q_c01.x, q_c01.z, q_c23.x, q_c23.z}, si[4] = {q_c01.y, q_c01.w, q_c23.y, q_c23.w};
      float y0[4], y1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        y0[i] = rotated_first(v0[i], v1[i], co[i], si[i]);
        y1[i] = rotated_second(v0[i], v1[i], co[i], si[i]);
      }
      if (q_kind == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { y0[i] *= q_scale; y1[i] *= q_scale; }
        ll_store_planes(rs, q_off, dq_plane, y0);
        ll_store_planes(rs, q_off + kOneHd, dq_plane, y1);
      } else {
        // this forward reads them from its own region, later ones from the cache
        auto put = [&](const float(&y)[4], uint32_t off, uint16_t *dst) {
          const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){y[0], y[1]}, bf16x2_t));
          const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){y[2], y[3]}, bf16x2_t));
          ll_store8(rs, off, lo, hi);
          *reinterpret_cast<uint2 *>(dst) = make_uint2(lo, hi);
        };
        const bool key = q_kind == 1;
        const int step = key ? kOneHd / 2 : 8;
        put(key ? y0 : v0, q_off, q_cache);
        put(key ? y1 : v1, q_off + step * 2, q_cache + step);
      }
    }
  } else if (wave < HB) {
    const float4 v = sum(wave, lane);
    for (int it = 0; __ballot(e_ok && missing16(e_x)) != 0ull && !give_up(p, it); ++it)
      if (e_ok) e_x = ll_load16(rs, e_off);
    const float y[4] = {__uint_as_float(e_x[0]) + v.x, __uint_as_float(e_x[1]) + v.y, __uint_as_float(e_x[2]) + v.z, __uint_as_float(e_x[3]) + v.w};
    const float z[4] = {y[0] * bf16_bits_to_f32(e_g.x & 0xffffu), y[1] * bf16_bits_to_f32(e_g.x >> 16),
                        y[2] * bf16_bits_to_f32(e_g.y & 0xffffu), y[3] * bf16_bits_to_f32(e_g.y >> 16)};
    float sq = e_ok ? sum_squares4(y[0], y[1], y[2], y[3]) : 0.f;
    if (e_ok) {
      if (last) {
        store_planes4(z, p.hb, p.hb_lo, packed_act_offset(e_row, e_col, 1));
      } else {
        ll_store_planes(ro, out_off, out_plane, z);
        ll_store_f4(ro, out_x + ((uint32_t)e_row * p.d + e_col) * 4, y);
      }
    }
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    if (e_ok && lane < 16) {
      if (last) p.ssq[e_row * (p.d / 16) + e_hb] = sq;
      else ll_store4(ro, out_s + (e_row * (p.d / 16) + e_hb) * 4, sq);
    }
  }
}

// Attention of one KV head: 32 query rows, one chunk of the prefix keys, and in the last chunk this forward's own rows.
// The wavefronts take tiles of 32 keys in turn and are merged through LDS, as in the attention kernel; the first tile of each is on its
// way to LDS before the queries are looked for.
template <bool DIRECT>
__device__ __forceinline__ void one_attention(const OneArgs &p, OneShared &sh, int par, u32x4 *kv_lds, int item, int layer, rsrc_t rs) {
  constexpr int HD = kOneHd, KK = HD / 16, CB = HD / 32, CR = HD / 8, NI = kTU / 64, RI = 64 / CR, NW = kOneWaves;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, h = lane >> 5, ql = lane & 31;
  __syncthreads();  // the tile buffers may still be read for the item before
  const int rg = item % p.n_rg, rest = item / p.n_rg, chunk = rest % p.n_chunks, kvh = rest / p.n_chunks;
  const int G = p.H / p.Hkv, n = p.rows, QR = G * n, L = p.L;
  const int n_tiles = (L + 31) / 32, c_begin = chunk * p.chunk_tiles, c_end = min(n_tiles, c_begin + p.chunk_tiles);
  const bool own = chunk == p.n_chunks - 1 && wave == (c_end - c_begin) % NW;  // this wavefront takes the forward's own rows
  u32x4 *kb = kv_lds + wave * kTU, *vb = kv_lds + (NW + wave) * kTU;
  const char *kbase = reinterpret_cast<const char *>(p.kc + p.g.row(0, layer, kvh, 0));
  const char *vbase = reinterpret_cast<const char *>(p.vc + p.g.row(0, layer, kvh, 0));
  const int lr = lane / CR;
  auto issue = [&](const char *src, u32x4 *dst, int tile) {
    const char *base = src + (int64_t)tile * (32 * HD * 2);
    const int last = L - 1 - tile * 32;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = RI * i + lr, c = (lane & (CR - 1)) ^ swizzle<HD>(r);
      load_16_to_lds<DIRECT>(base + (uint32_t)(min(r, last) * (HD * 2) + c * 16), dst + i * 64, lane);
    }
  };
  int tile = c_begin + wave;
  if (tile < c_end) {
    issue(kbase, kb, tile);
    issue(vbase, vb, tile);
  }
  const int qrow = rg * 32 + ql;
  const bool valid = qrow < QR;
  const int gi = valid ? qrow / n : 0, node = valid ? qrow - gi * n : 0, head = kvh * G + gi;
  const uint32_t anc = (uint32_t)p.anc[node];
  u32x4 qh[KK], qlo[KK];
  {
    const uint32_t qoff = p.lay.q + ((uint32_t)(node * p.H + head) * HD + 8 * h) * 2, plane = (uint32_t)p.dq * 2 * p.rp;
    if (wave == 0)  // (as in one_gemm: 3200 keys, 8 rows 769 -> 743, 16 rows 895 -> 876; 330 keys 635 -> 640, 708 -> 718)
      for (int it = 0; __ballot(missing16(ll_load16(rs, qoff))) != 0ull && !give_up(p, it); ++it) __builtin_amdgcn_s_sleep(8);
    barrier_only();
    for (int it = 0;; ++it) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        qh[kk] = ll_load16(rs, qoff + 32 * kk);
        qlo[kk] = ll_load16(rs, qoff + plane + 32 * kk);
      }
      bool bad = false;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) bad |= missing16(qh[kk]) || missing16(qlo[kk]);
      if (__ballot(bad) == 0ull || give_up(p, it)) break;
    }
  }
  Next next;
  next.ask(p);
  TileState<HD> s;
  s.init(kb, vb, lane);
  constexpr int kVm = 0x0F70 | NI, kVm0 = 0x0F70;
  for (; tile < c_end; tile += NW) {
    const bool more = tile + NW < c_end;
    __builtin_amdgcn_s_waitcnt(kVm);
    asm volatile("" ::: "memory");
    s.scores(qh, qlo);
    if (more) issue(kbase, kb, tile + NW);
    const int left = L - tile * 32;
    if (left < 32) s.mask(((1u << left) - 1u), h);
    s.softmax();
    if (more) __builtin_amdgcn_s_waitcnt(kVm);
    else __builtin_amdgcn_s_waitcnt(kVm0);
    asm volatile("" ::: "memory");
    s.values();
    if (more) issue(vbase, vb, tile + NW);
  }
  if (own) {
    u32x4 kr[NI], vr[NI];
    uint32_t at[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = RI * i + lr, c = (lane & (CR - 1)) ^ swizzle<HD>(r);
      at[i] = ((uint32_t)(kvh * p.rp + min(r, n - 1)) * HD + c * 8) * 2;
    }
    for (int it = 0;; ++it) {
      bool bad = false;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        kr[i] = ll_load16(rs, p.lay.kt + at[i]);
        vr[i] = ll_load16(rs, p.lay.vt + at[i]);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) bad |= missing16(kr[i]) || missing16(vr[i]);
      if (__ballot(bad) == 0ull || give_up(p, it)) break;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      kb[i * 64 + lane] = kr[i];
      vb[i * 64 + lane] = vr[i];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    s.scores(qh, qlo);
    s.mask(anc, h);
    s.softmax();
    s.values();
  }
  // merge of the wavefronts
  s.l_run = sum_halves(s.l_run);
  float4 *ko = reinterpret_cast<float4 *>(kv_lds), *vo = reinterpret_cast<float4 *>(kv_lds + NW * kTU);
  constexpr int HBK = CB / 2;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    float4 *dst = (cb < HBK ? ko : vo) + wave * kTU + (cb % HBK) * 256 + lane;
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[q * 64] = make_float4(s.o[cb][4 * q], s.o[cb][4 * q + 1], s.o[cb][4 * q + 2], s.o[cb][4 * q + 3]);
  }
  if (h == 0) sh.ml[wave * 32 + ql] = make_float2(s.m_run, s.l_run);
  next.publish(sh, par);
  __syncthreads();
  if (!valid) return;
  float wgt[NW], M = -INFINITY, Lsum = 0.f;
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    wgt[v] = sh.ml[v * 32 + ql].x;
    M = fmaxf(M, wgt[v]);
  }
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    wgt[v] = wgt[v] == -INFINITY ? 0.f : exp2_fast(wgt[v] - M);
    Lsum += wgt[v] * sh.ml[v * 32 + ql].y;
  }
  const float inv = 1.f / Lsum;
  const uint32_t part = (uint32_t)(chunk * n + node) * p.H + head;
  if (p.n_chunks > 1 && wave == 0 && h == 0) ll_store8(rs, p.lay.ml + part * 8, __float_as_uint(M), __float_as_uint(Lsum));
  static_assert(CB * 4 == NW, "one column quad per wavefront");
  {
    const int cb = wave >> 2, q = wave & 3;
    const float4 *src = (cb < HBK ? ko : vo) + (cb % HBK) * 256 + q * 64 + lane;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      const float4 z = src[v * kTU];
      acc[0] += wgt[v] * z.x; acc[1] += wgt[v] * z.y; acc[2] += wgt[v] * z.z; acc[3] += wgt[v] * z.w;
    }
    const int col = 32 * cb + 8 * q + 4 * h;
    if (p.n_chunks == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = div_by(acc[i], Lsum, inv);
      ll_store_planes(rs, p.lay.att + act_off(node, head * HD + col, p.rp), (uint32_t)p.dq * 2 * p.rp, acc);
    } else {
      ll_store_f4(rs, p.lay.po + (part * HD + col) * 4, acc);
    }
  }
}

// Merge of the key chunks: a thread takes 4 columns of a (row, head).
__device__ __forceinline__ void one_merge(const OneArgs &p, OneShared &sh, int par, int item, rsrc_t rs) {
  Next next;
  next.ask(p);
  constexpr int TPR = kOneHd / 4, MC = kMaxChunks;
  const uint32_t rh = (item * kOneThreads + threadIdx.x) / TPR;
  const int c = (threadIdx.x % TPR) * 4;
  const bool ok = rh < (uint32_t)(p.rows * p.H);
  if (ok) {
    const int row = rh / (uint32_t)p.H, head = rh - row * p.H;
    u32x4 o[MC];
    uint32_t m[MC], l[MC];
    float M = -INFINITY, den = 0.f, num[4] = {0.f, 0.f, 0.f, 0.f};
    for (int it = 0;; ++it) {
      bool bad = false;
#pragma unroll
      for (int i = 0; i < MC; ++i)
        if (i < p.n_chunks) {
          const uint32_t part = (uint32_t)(i * p.rows + row) * p.H + head;
          o[i] = ll_load16(rs, p.lay.po + (part * kOneHd + c) * 4);
          m[i] = ll_load4(rs, p.lay.ml + part * 8);
          l[i] = ll_load4(rs, p.lay.ml + part * 8 + 4);
        }
#pragma unroll
      for (int i = 0; i < MC; ++i)
        if (i < p.n_chunks) bad |= missing16(o[i]) || m[i] == ~0u || l[i] == ~0u;
      if (__ballot(bad) == 0ull || give_up(p, it)) break;
    }
#pragma unroll
    for (int i = 0; i < MC; ++i)
      if (i < p.n_chunks) M = fmaxf(M, __uint_as_float(m[i]));
#pragma unroll
    for (int i = 0; i < MC; ++i)
      if (i < p.n_chunks) {
        const float w = __uint_as_float(m[i]) == -INFINITY ? 0.f : exp2_fast(__uint_as_float(m[i]) - M);
        den += w * __uint_as_float(l[i]);
#pragma unroll
        for (int k = 0; k < 4; ++k) num[k] += w * __uint_as_float(o[i][k]);
      }
    const float inv = 1.f / den;
#pragma unroll
    for (int k = 0; k < 4; ++k) num[k] = div_by(num[k], den, inv);
    ll_store_planes(rs, p.lay.att + act_off(row, head * kOneHd + c, p.rp), (uint32_t)p.dq * 2 * p.rp, num);
  }
  next.publish(sh, par);
  __syncthreads();
}

// grid: one workgroup per compute unit (or fewer items), block 512.  DIRECT: the cache is on 16 bytes.  All 256 registers; NP = 2 spills 6
// constants of a thread (20 bytes of scratch), one of which q|k|v reads back while its weights are on their way, and so waits for those.
template <int NP, bool DIRECT>
__global__ __launch_bounds__(kOneThreads, 2) void one_launch_kernel(OneArgs args) {
  extern __shared__ u32x4 kv_lds[];
  __shared__ OneShared sh;
  if (threadIdx.x == 0) sh.next[1] = __hip_atomic_fetch_add(args.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  for (int par = 0;; par ^= 1) {
    // The arguments are read again for every item: kept over the loop they outgrow the scalar registers (1000 lane reads).
    auto pa = (const __attribute__((address_space(4))) OneArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(pa));
    const OneArgs &p = *(const OneArgs *)pa;
    const int t = __builtin_amdgcn_readfirstlane(sh.next[par ^ 1]);
    if (t >= p.total) return;
    const int layer = (uint32_t)t / (uint32_t)p.per_layer, i = t - layer * p.per_layer;
    const OneLayer lw = p.layers[layer];
    char *base = p.ll + (size_t)layer * p.lay.bytes;
    const bool last = layer == p.n_layers - 1;
    const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, p.lay.bytes, 0x00020000);
    if (i < p.i_att) {
      one_gemm<kOneQkv, kHbQkv, 8, NP>(p, sh, par, lw.qkv, p.d, p.n_half_qkv, i, layer, rs, p.lay.hb0, p.lay.s0, layer ? p.d / 16 : p.d / 32, 0, rs, 0, 0, 0, nullptr, false);
    } else if (i < p.i_mrg) {
      one_attention<DIRECT>(p, sh, par, kv_lds, i - p.i_att, layer, rs);
    } else if (i < p.i_o) {
      one_merge(p, sh, par, i - p.i_mrg, rs);
    } else if (i < p.i_gu) {
      one_gemm<kOneResid, one_hb_o(NP), 8, NP>(p, sh, par, lw.o, p.dq, p.d / 16, i - p.i_o, layer, rs, p.lay.att, 0, 0, p.lay.x0, rs, p.lay.hb1, p.lay.x1, p.lay.s1, lw.gain_ffn, false);
    } else if (i < p.i_dn) {
      one_gemm<kOneSwiglu, kHbGu, 8, NP>(p, sh, par, lw.gu, p.d, p.n_half_gu, i - p.i_gu, layer, rs, p.lay.hb1, p.lay.s1, p.d / 16, 0, rs, p.lay.t, 0, 0, nullptr, false);
    } else {
      const rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc(base + (last ? 0 : p.lay.bytes), 0, p.lay.bytes, 0x00020000);
      one_gemm<kOneResid, kHbDn, 22, NP>(p, sh, par, lw.down, p.F, p.d / 16, i - p.i_dn, layer, rs, p.lay.t, 0, 0, p.lay.x1, rn, p.lay.hb0, p.lay.x0, p.lay.s0, lw.gain_next, last);
    }
  }
}

// --------------------------------------------------------------------------- plan and launch
namespace {
constexpr unsigned kOneLds = 2 * kOneWaves * kTU * 16;

OneLayout one_layout(const ModelDims &md, int rp, int n_chunks) {
  OneLayout y{};
  const uint32_t d = md.d_model, dq = md.n_heads * md.head_dim, dkv = md.n_kv_heads * md.head_dim, F = md.d_ffn;
  uint32_t off = 0;
  auto take = [&](uint32_t bytes) { const uint32_t o = off; off = (off + bytes + 127) / 128 * 128; return o; };
  y.hb0 = take(d * 4 * rp); y.x0 = take(d * 4 * rp); y.s0 = take(d / 16 * 4 * rp);
  y.q = take(dq * 4 * rp); y.kt = take(dkv * 2 * rp); y.vt = take(dkv * 2 * rp);
  if (n_chunks > 1) { y.po = take(n_chunks * dq * 4 * rp); y.ml = take(n_chunks * md.n_heads * 8 * rp); }
  y.att = take(dq * 4 * rp);
  y.hb1 = take(d * 4 * rp); y.x1 = take(d * 4 * rp); y.s1 = take(d / 16 * 4 * rp);
  y.t = take(F * 4 * rp);
  y.bytes = off;
  return y;
}
}  // namespace

bool one_launch_model(const ModelDims &md, int n_cu) {
  const int dq = md.n_heads * md.head_dim;
  return md.head_dim == kOneHd && md.n_layers >= 2 && md.d_model % 32 == 0 && dq % 32 == 0 && md.d_ffn % 32 == 0 && md.d_model <= 2048 &&
         dq <= 2048 && md.d_ffn <= 5632 && n_cu >= 8;
}

OnePlan plan_one_launch(const ModelDims &md, int rows, int kv_len) {
  OnePlan pl;
  if (rows > 16 || kv_len > kOneKeys) return pl;
  pl.rows = rows;
  for (pl.rp = 1; pl.rp < rows;) pl.rp *= 2;
  pl.n_rg = (md.n_heads / md.n_kv_heads * rows + 31) / 32;
  const int tiles = (kv_len + 31) / 32;
  // One chunk per KV head: 0.9 us per layer for every 8 tiles, against another hand-over and the partial outputs, 1.5 us where these are few (2 layers
  // of 1 head: 8 rows, 2000 keys 69 us per call in one chunk, 59 in chunks) and 6 with 8 rows of 32 heads (1.1B, us per call, one chunk / chunks of 16
  // tiles: 1 row, 800 keys 648 / 690, 1600 714 / 685, 3200 872 / 700; 8 rows, 1600 750 / 800, 3200 908 / 743; 16 rows, 3200 992 / 876).
  pl.n_chunks = tiles <= (rows * md.n_heads <= 64 ? 36 : 64) ? 1 : (tiles + kChunkTiles - 1) / kChunkTiles;
  pl.chunk_tiles = (tiles + pl.n_chunks - 1) / pl.n_chunks;
  if (pl.chunk_tiles > 0) pl.n_chunks = (tiles + pl.chunk_tiles - 1) / pl.chunk_tiles;
  pl.lay = one_layout(md, pl.rp, pl.n_chunks);
  return pl;
}

size_t one_launch_bytes(const ModelDims &md) { return kOneCtl + (size_t)md.n_layers * one_layout(md, 16, kMaxChunks).bytes; }

hipError_t one_launch_set_lds_limit() {
  const void *kernels[] = {(const void *)one_launch_kernel<1, true>, (const void *)one_launch_kernel<1, false>, (const void *)one_launch_kernel<2, true>,
                           (const void *)one_launch_kernel<2, false>};
  for (const void *k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kOneLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

void launch_one(OneArgs a, int n_cu, hipStream_t st) {
  const int n_att = a.Hkv * a.n_rg * a.n_chunks;
  const int hb_o = one_hb_o(a.rows <= 8 ? 1 : 2);
  const int n_mrg = a.n_chunks > 1 ? (a.rows * a.H * (kOneHd / 4) + kOneThreads - 1) / kOneThreads : 0;
  a.i_att = (a.n_half_qkv + kHbQkv - 1) / kHbQkv;
  a.i_mrg = a.i_att + n_att;
  a.i_o = a.i_mrg + n_mrg;
  a.i_gu = a.i_o + (a.d / 16 + hb_o - 1) / hb_o;
  a.i_dn = a.i_gu + (a.n_half_gu + kHbGu - 1) / kHbGu;
  a.per_layer = a.i_dn + (a.d / 16 + kHbDn - 1) / kHbDn;
  a.total = a.per_layer * a.n_layers;
  const unsigned grid = a.total < n_cu ? a.total : n_cu;
  const bool aligned = (((uintptr_t)a.kc | (uintptr_t)a.vc) & 15) == 0;
  const auto kernel = a.rows <= 8 ? aligned ? one_launch_kernel<1, true> : one_launch_kernel<1, false>
                                  : aligned ? one_launch_kernel<2, true> : one_launch_kernel<2, false>;
  kernel<<<grid, kOneThreads, kOneLds, st>>>(a);
}

}  // namespace specasr
