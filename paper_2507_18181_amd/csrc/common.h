// Shared device helpers and internal layouts of the tree-verification library (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace specasr {

constexpr int kWave = 64;

// ---- storage types -------------------------------------------------------
struct bf16_t {
  uint16_t bits;
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v.bits) << 16); }
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// float -> bf16, round to nearest even (finite inputs; NaN keeps a quiet-NaN pattern)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// v = hi + lo with both parts bf16: the pair carries 16 mantissa bits of v
__device__ __forceinline__ void split_bf16(float v, uint16_t &hi, uint16_t &lo) {
  hi = f32_to_bf16_bits(v);
  lo = f32_to_bf16_bits(v - __uint_as_float(((uint32_t)hi) << 16));
}

// Two floats -> their hi planes packed (a in the low half) and their lo planes packed, with the
// hardware's round-to-nearest-even conversion (one v_cvt_pk_bf16_f32 per pair and plane; the same
// values as split_bf16).
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
__device__ __forceinline__ void split_bf16_pair(float a, float b, uint32_t &hi, uint32_t &lo) {
  const bf16x2_t h = __builtin_convertvector((f32x2_t){a, b}, bf16x2_t);
  hi = __builtin_bit_cast(uint32_t, h);
  const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){ra, rb}, bf16x2_t));
}
// 4 consecutive values of both planes (8 bytes each) at element offset o.
__device__ __forceinline__ void store_planes4(const float (&y)[4], uint16_t *hi_p, uint16_t *lo_p, int64_t o) {
  uint2 hi, lo;
  split_bf16_pair(y[0], y[1], hi.x, lo.x);
  split_bf16_pair(y[2], y[3], hi.y, lo.y);
  *reinterpret_cast<uint2 *>(hi_p + o) = hi;
  *reinterpret_cast<uint2 *>(lo_p + o) = lo;
}
__device__ __forceinline__ void store_bf16x4(const float (&y)[4], uint16_t *p) {
  *reinterpret_cast<uint2 *>(p) = make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){y[0], y[1]}, bf16x2_t)),
                                            __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){y[2], y[3]}, bf16x2_t)));
}

// A word as it goes into the hand-over regions of a forward in one launch, where all ones means "not there yet": a NaN of just those bits
// loses the last one and stays a NaN, as a float and as two bf16.
__device__ __forceinline__ uint32_t ready_word(uint32_t u) { return u < ~1u ? u : ~1u; }

// Sum of four squares and the rotation of a pair, with what is fused written out: left to the compiler it is another product after every
// change around it, and the results move by an ulp, which turns single K and V elements.
__device__ __forceinline__ float sum_squares4(float x, float y, float z, float w) { return fmaf(w, w, fmaf(z, z, fmaf(x, x, y * y))); }
__device__ __forceinline__ float rotated_first(float x0, float x1, float c, float s) { return fmaf(x0, c, -(x1 * s)); }
__device__ __forceinline__ float rotated_second(float x0, float x1, float c, float s) { return fmaf(x1, c, x0 * s); }

// SwiGLU of one feature with the row's 1/rms: silu(g * rs) * (u * rs), the quotient g / (1 + exp(-g)) from the hardware's
// reciprocal and one residual step.  The hardware flushes reciprocals below 2^-126, and 1 + exp(-g) reaches 2^128: it is
// taken of a 16th.  exp(-g) = inf (g < -88.7) leaves no residual; there the quotient is -0 already.  7B prefill of 810,
// gate|up: 299.0 us with the bare reciprocal (which gave 0 for g < -87.3), 299.9, 300.9 with a division.
__device__ __forceinline__ float swiglu_act(float g, float u, float rs) {
  g *= rs;
  const float d = 1.0f + __expf(-g), r = __builtin_amdgcn_rcpf(d * 0.0625f) * 0.0625f, q = g * r;
  return (d == INFINITY ? q : fmaf(fmaf(-d, q, g), r, q)) * (u * rs);
}

template <class T> __device__ __forceinline__ T from_f32(float f);
template <> __device__ __forceinline__ float from_f32<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float f) {
  bf16_t r;
  r.bits = f32_to_bf16_bits(f);
  return r;
}

// Element offset of activation (row, col) inside one plane of a B-operand-packed buffer:
// [kstep = col/16][node group = row/32][lane = row%32 + 32*((col%16)/8)][col%8]
__host__ __device__ __forceinline__ int64_t packed_act_offset(int row, int col, int nb) {
  return ((((int64_t)(col >> 4) * nb + (row >> 5)) * 64 + (row & 31) + 32 * ((col >> 3) & 1)) << 3) + (col & 7);
}

// Element offset of split-k partial sum (split s, activation row, output column) in the partial-sum
// buffer: [split][band = col/32][row, padded to rows_pad = 32 or a multiple of 64][col%32].  One (split, band)
// block is contiguous, so the GEMM writes it with full-line stores and a consumer thread reads
// 4 consecutive columns as one float4 (col a multiple of 4).
__host__ __device__ __forceinline__ int64_t part_offset(int s, int row, int col, int n_bands, int rows_pad) {
  return ((((int64_t)s * n_bands + (col >> 5)) * rows_pad + row) << 5) + (col & 31);
}
__host__ __device__ __forceinline__ int part_rows_pad(int rows) { return rows <= 32 ? 32 : (rows + 63) / 64 * 64; }

// v += partial sums of 4 columns, `stride` floats apart, in the order of the splits: rounds of 4 that are requested together, and so are the last
// n_splits % 4 (the compiler's own unrolling by 4 waits for each of those by itself).
__device__ __forceinline__ void add_splits4(float4 &v, const float *p, int64_t stride, int n_splits) {
  auto add = [&](const float4 &t) { v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w; };
  int s = 0;
  for (; s + 4 <= n_splits; s += 4, p += 4 * stride) {
    float4 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = *reinterpret_cast<const float4 *>(p + i * stride);
#pragma unroll
    for (int i = 0; i < 4; ++i) add(t[i]);
  }
  float4 t[3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (s + i < n_splits) t[i] = *reinterpret_cast<const float4 *>(p + i * stride);
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (s + i < n_splits) add(t[i]);
}

// ---- per-call tree metadata as the kernels see it ------------------------
// Rows are the tree nodes of all sequences of the call, flattened without
// padding: row = row_start[seq] + node.
struct StepMeta {
  const int32_t *token;      // [rows] token id (ignored where use_embed)
  const int32_t *seq;        // [rows] sequence of the row
  const int32_t *node;       // [rows] node index inside its tree
  const int32_t *depth;      // [rows]
  const int32_t *pos;        // [rows] kv_len[seq] + depth  (rotary position)
  const int32_t *slot;       // [rows] kv_len[seq] + node   (cache slot)
  const int32_t *parent;     // [rows] parent node index inside the tree, -1 for the root
  const int32_t *use_embed;  // [rows]
  const uint64_t *anc;       // [rows] bit j set iff node j is on the row's root path (self included)
  const int32_t *kv_len;     // [batch]
  const int32_t *row_start;  // [batch]
  const int32_t *n_nodes;    // [batch]
  int32_t rows, batch;
  // Copies of kv_len[0] and n_nodes[0] that travel with the kernel arguments: a single-sequence
  // call (the common case) needs no dependent global load to find its key range.
  int32_t kv_len0, n_nodes0;
  __device__ __forceinline__ int seq_of_row(int r) const { return batch == 1 ? 0 : seq[r]; }
  __device__ __forceinline__ int seq_kv_len(int s) const { return batch == 1 ? kv_len0 : kv_len[s]; }
  __device__ __forceinline__ int seq_n_nodes(int s) const { return batch == 1 ? n_nodes0 : n_nodes[s]; }
  __device__ __forceinline__ int seq_row_start(int s) const { return batch == 1 ? 0 : row_start[s]; }
};

// KV cache geometry: element index of (seq, layer, kv head, slot, 0)
struct KvGeom {
  int64_t capacity;
  int32_t n_layers, n_kv_heads, head_dim;
  // 1: every sequence of the call is a window onto the cache of sequence 0 (a long chain cut into
  // pieces that are processed together: piece j is "sequence" j with its own kv_len)
  int32_t shared_cache = 0;
  __host__ __device__ int64_t row(int32_t seq, int32_t layer, int32_t h, int64_t slot) const {
    return ((((int64_t)(shared_cache ? 0 : seq) * n_layers + layer) * n_kv_heads + h) * capacity + slot) * head_dim;
  }
};

// ---- wavefront / block reductions ---------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Sums 16 values over the 64 lanes; every lane returns the sum of value 8*b5 + 4*b4 + 2*b3 + b2 (bits of its
// index).  Lanes 32 and 16 apart exchange by swaps of register halves, nearer ones inside a row of 16.  (Written as
// selects between elements of v, the compiler made them selects of an index, and each of those a chain of 15 compares:
// tiny fp32 verify of 8 nodes 137 us with them, 113 now.)
template <int CTRL> __device__ __forceinline__ float lane_move(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_sum16(const float (&v)[16], int lane) {
  auto add32 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  auto add16 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  const float a0 = add32(v[0], v[8]), a1 = add32(v[1], v[9]), a2 = add32(v[2], v[10]), a3 = add32(v[3], v[11]);
  const float a4 = add32(v[4], v[12]), a5 = add32(v[5], v[13]), a6 = add32(v[6], v[14]), a7 = add32(v[7], v[15]);
  const float b0 = add16(a0, a4), b1 = add16(a1, a5), b2 = add16(a2, a6), b3 = add16(a3, a7);
  const bool up8 = lane & 8, up4 = lane & 4;
  const float c0 = (up8 ? b2 : b0) + lane_move<0x128>(up8 ? b0 : b2);  // rotated by 8
  const float c1 = (up8 ? b3 : b1) + lane_move<0x128>(up8 ? b1 : b3);
  float d = (up4 ? c1 : c0) + __shfl_xor(up4 ? c0 : c1, 4, 64);
  d += lane_move<0x4e>(d);  // pairs 2 apart, then neighbours
  return d + lane_move<0xb1>(d);
}

// Block-wide reductions for blockDim.x a multiple of 64 and <= 1024. `red` holds >= 16 floats.
__device__ __forceinline__ float block_sum(float v, float *red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];
  return t;
}
__device__ __forceinline__ float block_max(float v, float *red) {
  v = wave_max(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = red[0];
  for (int i = 1; i < nw; ++i) t = fmaxf(t, red[i]);
  return t;
}

// Per-row RMSNorm statistics left by launch_residual_gain for the consumer of the next GEMM.
struct RowNorm {
  const float *ssq;  // [rows][n_slab] sums of squares of the residual row, one per column slab
  int n_slab;
  int d;      // row length
  float eps;  // added to the mean square inside the root
};
// 1 / rms of residual row r from the slab sums of squares (eps inside the root, Sec. II-A's decoder
// block), in two steps: row_ssq_lane issues the loads of this lane's share (up to 4 at once) and adds
// them up, which waits for them, so that loads that follow it in a kernel are a trip of their own;
// row_rms_finish sums over the wavefront.  Every lane of the calling wavefront must be active in
// row_rms_finish; all lanes get the same value.
__device__ __forceinline__ float row_ssq_lane(const RowNorm &nrm, int r) {
  const float *p = nrm.ssq + (int64_t)r * nrm.n_slab;
  const int i = threadIdx.x & 63, n = nrm.n_slab;
  const float v0 = i < n ? p[i] : 0.f, v1 = i + 64 < n ? p[i + 64] : 0.f;
  const float v2 = i + 128 < n ? p[i + 128] : 0.f, v3 = i + 192 < n ? p[i + 192] : 0.f;
  float s = (v0 + v1) + (v2 + v3);
  for (int k = i + 256; k < n; k += 64) s += p[k];
  return s;
}
__device__ __forceinline__ float row_rms_finish(const RowNorm &nrm, float lane_ssq) {
  return 1.0f / sqrtf(wave_sum(lane_ssq) / (float)nrm.d + nrm.eps);
}
__device__ __forceinline__ float row_rms_scale(const RowNorm &nrm, int r) {
  return row_rms_finish(nrm, row_ssq_lane(nrm, r));
}

}  // namespace specasr
