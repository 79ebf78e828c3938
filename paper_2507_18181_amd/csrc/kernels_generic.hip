// Dtype-generic stages of the tree-verification path: fp32 arithmetic on fp32 activations,
// weights and KV cache read in their storage type.  They serve fp32 models and are the
// fallback for shapes the MFMA kernels do not cover.  Also the integer stages (acceptance,
// KV compaction), which are shared by every path.
#include "kernels.h"

namespace specasr {

// 4 consecutive elements
template <class T> struct Vec4;
template <> struct Vec4<float> {
  static __device__ __forceinline__ void load(const float *p, float w[4]) {
    float4 v = *reinterpret_cast<const float4 *>(p);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  }
};
template <> struct Vec4<bf16_t> {
  static __device__ __forceinline__ void load(const bf16_t *p, float w[4]) {
    uint2 v = *reinterpret_cast<const uint2 *>(p);
    w[0] = __uint_as_float(v.x << 16); w[1] = __uint_as_float(v.x & 0xffff0000u);
    w[2] = __uint_as_float(v.y << 16); w[3] = __uint_as_float(v.y & 0xffff0000u);
  }
};

// --------------------------------------------------------------------------- the start of a forward
// One launch for what depends on nothing but the call's metadata, which it reads in pinned host memory (`m` points there):
// the first blocks fill the rope table (64-bit functions: the longest), the next ones copy the metadata block to the device
// for all later kernels, the others fetch the embedding rows.  PLANES (MFMA path): an embedding row leaves as residual_gain_kernel would
// leave it, x * gain in two planes and one sum of squares per 32 columns.  Bound by one read across PCIe and one of
// the table: 7B, 32 rows copy 4.5 + embed 9.9 + rope 3.5 + residual_gain 4.9 us before.
// Sec. II-B: a tree node is verified as if decoded after its own branch, so its rotary
// position is kv_len + depth, shared by siblings.  Angles are formed in fp64 once per call.
template <class T, bool PLANES>
__global__ __launch_bounds__(256) void begin_kernel(StepMeta m, const T *E, const T *in_emb, int vec, int max_nodes, int d, float *x, int half, int hd,
                                                    double theta, float2 *cs, int rope_blocks, BeginPlanes pl, const int32_t *words, int32_t *dst, int n_words) {
  int blk = blockIdx.x;
  if (blk < rope_blocks) {
    const int idx = blk * 256 + threadIdx.x;
    if (idx >= m.rows * half) return;
    const int row = idx / half, j = idx - row * half;
    const double ang = (double)m.pos[row] * pow(theta, -2.0 * (double)j / (double)hd);
    cs[idx] = make_float2((float)cos(ang), (float)sin(ang));
    return;
  }
  blk -= rope_blocks;
  const int copy_blocks = (n_words + 1023) / 1024;
  if (blk < copy_blocks) {
    const int i0 = blk * 1024 + threadIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i0 + i * 256 < n_words) dst[i0 + i * 256] = words[i0 + i * 256];
    return;
  }
  blk -= copy_blocks;
  if (PLANES && blk < pl.fill_blocks) {  // regions whose data carry their own readiness start as all ones
    if (blk == 0 && threadIdx.x < 2) pl.ctl[threadIdx.x] = 0;
    for (uint32_t i = blk * 256 + threadIdx.x; i < pl.fill_units; i += pl.fill_blocks * 256) pl.fill[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    return;
  }
  if (PLANES) blk -= pl.fill_blocks;
  const int row_blocks = (m.rows + 31) >> 5;
  // 32 rows x 128 columns: 8 threads per row take 4 columns each, 4 times; whole lines of both planes leave a block
  const int cols = (uint32_t)blk / (uint32_t)row_blocks, row = (blk - cols * row_blocks) * 32 + (threadIdx.x >> 3);
  const bool live = row < m.rows;
  const int r = live ? row : m.rows - 1;
  const T *src;
  if (in_emb != nullptr && m.use_embed[r])
    src = in_emb + ((int64_t)m.seq[r] * max_nodes + m.node[r]) * d;
  else
    src = E + (int64_t)m.token[r] * d;
  float v[4][4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = cols * 128 + t * 32 + (threadIdx.x & 7) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[t][i] = 0.f;
    if (live && c < d) {  // d is a multiple of 8
      if (vec) {
        Vec4<T>::load(src + c, v[t]);
      } else {  // a table that is not on 4 elements (a caller's slice)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[t][i] = to_f32(src[c + i]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = cols * 128 + t * 32 + (threadIdx.x & 7) * 4;
    const bool ok = live && c < d;
    if (ok) *reinterpret_cast<float4 *>(x + (int64_t)r * d + c) = make_float4(v[t][0], v[t][1], v[t][2], v[t][3]);  // (widened bf16 is never all ones)
    if (PLANES) {
      float ss = v[t][0] * v[t][0] + v[t][1] * v[t][1] + v[t][2] * v[t][2] + v[t][3] * v[t][3];
      ss += __shfl_xor(ss, 1, 64);
      ss += __shfl_xor(ss, 2, 64);
      ss += __shfl_xor(ss, 4, 64);
      if (ok) {
        if ((threadIdx.x & 7) == 0) pl.ssq[(int64_t)r * pl.n_slab + (c >> 5)] = pl.rp ? __uint_as_float(ready_word(__float_as_uint(ss))) : ss;
        const uint2 g = *reinterpret_cast<const uint2 *>(pl.gain + c);
        const float y[4] = {v[t][0] * bf16_bits_to_f32(g.x & 0xffffu), v[t][1] * bf16_bits_to_f32(g.x >> 16),
                            v[t][2] * bf16_bits_to_f32(g.y & 0xffffu), v[t][3] * bf16_bits_to_f32(g.y >> 16)};
        if (pl.rp) {
          uint2 hi, lo;
          split_bf16_pair(y[0], y[1], hi.x, lo.x);
          split_bf16_pair(y[2], y[3], hi.y, lo.y);
          const int64_t o = ((int64_t)(c >> 3) * pl.rp + r) * 8 + (c & 4);
          *reinterpret_cast<uint2 *>(pl.hb + o) = make_uint2(ready_word(hi.x), ready_word(hi.y));
          *reinterpret_cast<uint2 *>(pl.hb_lo + o) = make_uint2(ready_word(lo.x), ready_word(lo.y));
        } else {
          store_planes4(y, pl.hb, pl.hb_lo, packed_act_offset(r, c, pl.nb));
        }
      }
    }
  }
}

void launch_begin(const StepMeta &hm, int dtype, const void *E, const void *in_emb, int max_nodes, int d, float *x, int hd, float theta,
                  float2 *cs, const BeginPlanes *pl, const int32_t *words, int32_t *dst, int n_words, hipStream_t st) {
  const int half = hd / 2, rope_blocks = (hm.rows * half + 255) / 256;
  const int blocks = rope_blocks + (n_words + 1023) / 1024 + (hm.rows + 31) / 32 * ((d + 127) / 128) + (pl ? pl->fill_blocks : 0);
  const size_t esz = dtype == 1 ? 2 : 4;
  const int vec = (((uintptr_t)E | (uintptr_t)in_emb) & (4 * esz - 1)) == 0;
  const BeginPlanes none{};
  if (pl != nullptr)
    begin_kernel<bf16_t, true><<<blocks, 256, 0, st>>>(hm, (const bf16_t *)E, (const bf16_t *)in_emb, vec, max_nodes, d, x, half, hd, (double)theta, cs, rope_blocks, *pl, words, dst, n_words);
  else if (dtype == 1)
    begin_kernel<bf16_t, false><<<blocks, 256, 0, st>>>(hm, (const bf16_t *)E, (const bf16_t *)in_emb, vec, max_nodes, d, x, half, hd, (double)theta, cs, rope_blocks, none, words, dst, n_words);
  else
    begin_kernel<float, false><<<blocks, 256, 0, st>>>(hm, (const float *)E, (const float *)in_emb, vec, max_nodes, d, x, half, hd, (double)theta, cs, rope_blocks, none, words, dst, n_words);
}

// --------------------------------------------------------------------------- RMSNorm
template <class T>
__global__ void rmsnorm_kernel(const float *x, const T *g, int d, float eps, float *y) {
  __shared__ float red[16];
  const float *xr = x + (int64_t)blockIdx.x * d;
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += blockDim.x) ss += xr[c] * xr[c];
  ss = block_sum(ss, red);
  float rs = 1.0f / sqrtf(ss / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += blockDim.x)
    y[(int64_t)blockIdx.x * d + c] = xr[c] * rs * to_f32(g[c]);
}

// --------------------------------------------------------------------------- linear
// One wavefront owns OW output features and RB activation rows; lanes stride over k in 4-element vectors; the
// OW * RB dot products are finished together by a halving exchange (17 steps for 16 sums instead of 96).  n_in % 4 == 0.  On a tiny model a launch costs more than its work, so what stands between two products is
// done by them: gate and up of one feature belong to one wavefront, which applies SwiGLU; q, k and v are one launch
// whose wavefronts own the two halves of a rotary pair, rotate it and write k and v to the cache; the logits go to the
// caller's array; and up to kNormWidth input features and a few hundred rows a workgroup normalises its 8 rows itself, in
// LDS.  Bound by the chain of launches, about 5 us each: tiny fp32 verify of 8 nodes 170 us with a kernel for each of these
// (24 launches), 138 with 15 (the first and last kernels of a call merged as well), 116 since the exchange is one of registers, 111 with
// everything that a product needs requested at once.

// The matrices of one launch: blocks [first[i], first[i+1]) work on matrix i.
template <class T>
struct LinearSet {
  const T *W[3];
  float *y[3];
  int n_out[3], ldy[3], first[3];
};

// What the modes below need besides.
template <class T>
struct LinearMore {
  const T *gain;                  // NORM
  float eps;
  const int32_t *seq, *slot, *node;  // QKV: seq, slot; LOGITS: seq, node
  int max_nodes;
  KvGeom g;                       // QKV
  int layer, hd;
  const float2 *cs;
  T *kc, *vc;
};

constexpr int kLinRows = 8, kLinOut = 2;  // RB, OW
// Widest input that a workgroup normalises itself: 8 rows of it are 32 KB of LDS and every workgroup repeats them.  An
// 8-layer fp32 model, 16 rows, with the norm in the linear / as a kernel of its own: 532 / 617 us at d_model 512, 735 /
// 866 at 1024 (64 rows 1311 / 1491); wider was not built, it would need more LDS or a second pass.
constexpr int kNormWidth = 1024;

enum LinearMode {
  kLinPlain = 0,   // y = W a, or y += W a
  kLinSwiglu = 1,  // W[0] = gate, W[1] = up, one feature per wavefront, y[0] = silu(gate) * up
  kLinQkv = 2,     // W = q, k, v; y[0] = rotated queries, rotated k and v go to their cache slots
  kLinLogits = 3,  // row r goes to row seq * max_nodes + node of y
};

// NORM: a holds residual rows; the product takes a * gain / rms(a), as rmsnorm_kernel leaves it.
// KB: blocks of 256 inputs that a wavefront asks for at once (not NORM, which asks for all of them).
template <class T, int MODE, bool NORM, int KB>
__global__ __launch_bounds__(256) void linear_kernel(LinearSet<T> ls, LinearMore<T> mo, int n_in, const float *a, int lda, int rows, int accumulate) {
  constexpr int RB = kLinRows, OW = kLinOut, NIT = kNormWidth / 256;
  __shared__ float4 as[NORM ? RB * (kNormWidth / 4) : 1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // selected by value: an index into the arguments would be a second, dependent load of them
  const bool is1 = MODE != kLinSwiglu && (int)blockIdx.x >= ls.first[1], is2 = MODE != kLinSwiglu && (int)blockIdx.x >= ls.first[2];
  const T *W = is2 ? ls.W[2] : is1 ? ls.W[1] : ls.W[0];
  float *y = is2 ? ls.y[2] : is1 ? ls.y[1] : ls.y[0];
  const int n_out = is2 ? ls.n_out[2] : is1 ? ls.n_out[1] : ls.n_out[0], ldy = is2 ? ls.ldy[2] : is1 ? ls.ldy[1] : ls.ldy[0];
  const int u = ((int)blockIdx.x - (is2 ? ls.first[2] : is1 ? ls.first[1] : 0)) * 4 + wave, r0 = blockIdx.y * RB;
  // this wavefront's outputs o0 and o1
  int o0, o1, head = 0, j0 = 0;
  const int half = mo.hd >> 1;
  if (MODE == kLinQkv) {
    head = (uint32_t)u / (uint32_t)half;
    j0 = u - head * half;
    o0 = head * mo.hd + j0;
    o1 = o0 + half;
  } else {
    o0 = u * (MODE == kLinSwiglu ? 1 : OW);
    o1 = o0 + 1;
  }
  const bool live = o0 < n_out;
  if (!NORM && !live) return;
  const T *w0 = W + (int64_t)min(o0, n_out - 1) * n_in;
  const T *w1 = MODE == kLinSwiglu ? ls.W[1] + (int64_t)min(o0, n_out - 1) * n_in : W + (int64_t)min(o1, n_out - 1) * n_in;
  // what the sums are added to, requested before them
  const int e_o = lane < 32 ? o0 : o1, e_r = r0 + ((lane >> 2) & 7);
  float before = 0.f;
  if (MODE == kLinPlain && accumulate && (lane & 3) == 0 && e_r < rows && e_o < n_out) before = y[(int64_t)e_r * ldy + e_o];
  float acc[OW * RB];
#pragma unroll
  for (int i = 0; i < OW * RB; ++i) acc[i] = 0.f;
  if constexpr (NORM) {
    // all weights of the wavefront and its 2 rows are requested at once
    float w[NIT][OW][4];
    float4 x[2][NIT];
    float gn[NIT][4];
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
      const int k = lane * 4 + t * 256;
      if (k < n_in) {
        Vec4<T>::load(w0 + k, w[t][0]);
        Vec4<T>::load(w1 + k, w[t][1]);
        Vec4<T>::load(mo.gain + k, gn[t]);
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i][t] = *reinterpret_cast<const float4 *>(a + (int64_t)min(r0 + 2 * wave + i, rows - 1) * lda + k);
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float ss = 0.f;
#pragma unroll
      for (int t = 0; t < NIT; ++t)
        if (lane * 4 + t * 256 < n_in) ss += (x[i][t].x * x[i][t].x + x[i][t].y * x[i][t].y) + (x[i][t].z * x[i][t].z + x[i][t].w * x[i][t].w);
      const float rs = 1.0f / sqrtf(wave_sum(ss) / (float)n_in + mo.eps);
#pragma unroll
      for (int t = 0; t < NIT; ++t)
        if (lane * 4 + t * 256 < n_in)
          as[(2 * wave + i) * (kNormWidth / 4) + lane + t * 64] =
              make_float4(x[i][t].x * rs * gn[t][0], x[i][t].y * rs * gn[t][1], x[i][t].z * rs * gn[t][2], x[i][t].w * rs * gn[t][3]);
    }
    __syncthreads();
    if (!live) return;
#pragma unroll
    for (int t = 0; t < NIT; ++t)
      if (lane * 4 + t * 256 < n_in)
#pragma unroll
        for (int j = 0; j < RB; ++j) {
          const float4 av = as[j * (kNormWidth / 4) + lane + t * 64];
#pragma unroll
          for (int i = 0; i < OW; ++i)
            acc[i * RB + j] += w[t][i][0] * av.x + w[t][i][1] * av.y + w[t][i][2] * av.z + w[t][i][3] * av.w;
        }
  } else {
    for (int k0 = lane * 4; k0 < n_in; k0 += 256 * KB) {
      float w[KB][OW][4];
      float4 av[KB][RB];
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        const int k = k0 + t * 256;
        if (k < n_in) {
          Vec4<T>::load(w0 + k, w[t][0]);
          Vec4<T>::load(w1 + k, w[t][1]);
#pragma unroll
          for (int j = 0; j < RB; ++j) av[t][j] = *reinterpret_cast<const float4 *>(a + (int64_t)min(r0 + j, rows - 1) * lda + k);
        }
      }
#pragma unroll
      for (int t = 0; t < KB; ++t)
        if (k0 + t * 256 < n_in)
#pragma unroll
          for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int i = 0; i < OW; ++i)
              acc[i * RB + j] += w[t][i][0] * av[t][j].x + w[t][i][1] * av[t][j].y + w[t][i][2] * av[t][j].z + w[t][i][3] * av[t][j].w;
    }
  }
  const float s = wave_sum16(acc, lane);  // of output (lane < 32 ? o0 : o1), row r0 + (lane/4)%8
  const int o = e_o, r = e_r;
  const bool mine = (lane & 3) == 0 && r < rows;
  if (MODE == kLinSwiglu) {
    const float up = __shfl_xor(s, 32, 64);
    if (lane < 32 && mine) y[(int64_t)r * ldy + o0] = s / (1.0f + __expf(-s)) * up;
  } else if (MODE == kLinQkv) {
    const float other = __shfl_xor(s, 32, 64);
    if (!mine) return;
    float v = s;
    if (!is2) {  // rotary pair: x0 cos - x1 sin, x1 cos + x0 sin
      const float2 c = mo.cs[(int64_t)r * half + j0];
      v = lane < 32 ? s * c.x - other * c.y : s * c.x + other * c.y;
    }
    if (!is1 && !is2) {
      y[(int64_t)r * ldy + o] = v;
    } else {
      T *cache = is2 ? mo.vc : mo.kc;
      cache[mo.g.row(mo.seq[r], mo.layer, head, mo.slot[r]) + (o - head * mo.hd)] = from_f32<T>(v);
    }
  } else if (mine && o < n_out) {
    const int64_t yr = MODE == kLinLogits ? (int64_t)mo.seq[r] * mo.max_nodes + mo.node[r] : r;
    float *dst = y + yr * ldy + o;
    *dst = MODE == kLinPlain && accumulate ? before + s : s;
  }
}

template <class T, int MODE, bool NORM>
static void launch_linear_t(const LinearJob *jobs, int n, const LinearMore<T> &mo, int n_in, const float *a, int lda, int rows, bool accumulate, hipStream_t st) {
  LinearSet<T> ls{};
  int blocks = 0;
  for (int i = 0; i < 3; ++i) {
    const LinearJob &j = jobs[i < n ? i : n - 1];
    ls.W[i] = (const T *)j.W;
    ls.y[i] = j.y;
    ls.n_out[i] = j.n_out;
    ls.ldy[i] = j.ldy;
    ls.first[i] = i < n ? blocks : 0x7fffffff;
    if (MODE == kLinSwiglu) blocks = (j.n_out + 3) / 4;
    else if (i < n) blocks += (j.n_out + 4 * kLinOut - 1) / (4 * kLinOut);
  }
  dim3 grid(blocks, (rows + kLinRows - 1) / kLinRows);
  // All 4 blocks of 1024 inputs at once take 200 registers, 2 wavefronts per SIMD: where no more than that are there, they wait once instead of
  // twice or three times; with more, 2 blocks and twice the wavefronts (us per verify, fp32, 2 / 4: d_model 256, 8 rows 116 / 111, 64 rows
  // 127 / 123; 512, 8 rows 344 / 290; 1024, 16 rows 392 / 347, 64 rows (1024 workgroups) 637 / 642).
  if (NORM || (int64_t)grid.x * grid.y > 512) linear_kernel<T, MODE, NORM, 2><<<grid, 256, 0, st>>>(ls, mo, n_in, a, lda, rows, accumulate ? 1 : 0);
  else linear_kernel<T, MODE, NORM, NORM ? 2 : 4><<<grid, 256, 0, st>>>(ls, mo, n_in, a, lda, rows, accumulate ? 1 : 0);
}

// With many rows the launch that is saved is small against the norm that every workgroup repeats.  Norm in the linear / as a
// kernel, us per verify, fp32 (bf16 alike): d_model 256, 2 layers, 256 rows 282 / 285, 384 376 / 371, 1024 838 / 778; 512, 4
// layers, 256 rows 870 / 866, 384 1220 / 1178, 1024 2934 / 2685; 1024, 4 layers, 512 rows 3296 / 3330, 768 4841 / 4800.
// The linear reads the gain 4 elements at a time, rmsnorm_kernel one by one: it takes a gain that is a caller's slice off that grid.
bool linear_normalises(int d, const void *gain, int elem_bytes, int rows) {
  return d <= kNormWidth && rows <= (d / 2 > 256 ? d / 2 : 256) && ((uintptr_t)gain & (4 * elem_bytes - 1)) == 0;
}

template <class T, int MODE>
static void launch_linear_norm(const LinearJob *jobs, int n, LinearMore<T> mo, const NormIn &nx, hipStream_t st) {
  if (linear_normalises(nx.d, nx.gain, sizeof(T), nx.rows)) {
    mo.gain = (const T *)nx.gain;
    mo.eps = nx.eps;
    launch_linear_t<T, MODE, true>(jobs, n, mo, nx.d, nx.x, nx.d, nx.rows, false, st);
    return;
  }
  rmsnorm_kernel<T><<<nx.rows, 256, 0, st>>>(nx.x, (const T *)nx.gain, nx.d, nx.eps, nx.h);
  launch_linear_t<T, MODE, false>(jobs, n, mo, nx.d, nx.h, nx.d, nx.rows, false, st);
}

void launch_linear_add(int dtype, const void *W, int n_out, int n_in, const float *a, float *y, int rows, hipStream_t st) {
  const LinearJob j{W, n_out, y, n_out};
  if (dtype == 1) launch_linear_t<bf16_t, kLinPlain, false>(&j, 1, LinearMore<bf16_t>{}, n_in, a, n_in, rows, true, st);
  else launch_linear_t<float, kLinPlain, false>(&j, 1, LinearMore<float>{}, n_in, a, n_in, rows, true, st);
}

void launch_linear_swiglu(int dtype, const NormIn &nx, const void *gate, const void *up, int F, float *t, hipStream_t st) {
  const LinearJob j[2] = {{gate, F, t, F}, {up, F, t, F}};
  if (dtype == 1) launch_linear_norm<bf16_t, kLinSwiglu>(j, 2, LinearMore<bf16_t>{}, nx, st);
  else launch_linear_norm<float, kLinSwiglu>(j, 2, LinearMore<float>{}, nx, st);
}

template <class T>
static void launch_linear_qkv_t(const NormIn &nx, const LinearJob *jobs, const StepMeta &m, const KvGeom &g, int layer, const float2 *cs,
                                void *kc, void *vc, hipStream_t st) {
  LinearMore<T> mo{};
  mo.seq = m.seq; mo.slot = m.slot; mo.g = g; mo.layer = layer; mo.hd = g.head_dim; mo.cs = cs; mo.kc = (T *)kc; mo.vc = (T *)vc;
  launch_linear_norm<T, kLinQkv>(jobs, 3, mo, nx, st);
}

void launch_linear_qkv(const StepMeta &m, const ModelDims &md, const KvGeom &g, int layer, const NormIn &nx, const void *wq, const void *wk,
                       const void *wv, const float2 *cs, float *q, void *kc, void *vc, hipStream_t st) {
  const int dq = md.n_heads * md.head_dim, dkv = md.n_kv_heads * md.head_dim;
  const LinearJob jobs[3] = {{wq, dq, q, dq}, {wk, dkv, nullptr, 0}, {wv, dkv, nullptr, 0}};
  if (md.dtype == 1) launch_linear_qkv_t<bf16_t>(nx, jobs, m, g, layer, cs, kc, vc, st);
  else launch_linear_qkv_t<float>(nx, jobs, m, g, layer, cs, kc, vc, st);
}

template <class T>
static void launch_linear_logits_t(const StepMeta &m, const NormIn &nx, const LinearJob &j, int max_nodes, bool padded, hipStream_t st) {
  LinearMore<T> mo{};
  mo.seq = m.seq; mo.node = m.node; mo.max_nodes = max_nodes;
  if (padded) launch_linear_norm<T, kLinLogits>(&j, 1, mo, nx, st);
  else launch_linear_norm<T, kLinPlain>(&j, 1, mo, nx, st);
}

void launch_linear_logits(const StepMeta &m, int dtype, const NormIn &nx, const void *W, int V, int max_nodes, float *logits, bool padded, hipStream_t st) {
  const LinearJob j{W, V, logits, V};
  if (dtype == 1) launch_linear_logits_t<bf16_t>(m, nx, j, max_nodes, padded, st);
  else launch_linear_logits_t<float>(m, nx, j, max_nodes, padded, st);
}

// --------------------------------------------------------------------------- attention
// One block per (row, query head).  Keys are the cache slots [0, kv_len) plus the slots of
// the row's own root path (Sec. II-B: the 2D tree mask).  Online softmax over chunks of 256
// keys; scores, running maximum and sums in fp32.  hd <= 256 and 256 % hd == 0.
template <class T>
__global__ __launch_bounds__(256) void attention_generic_kernel(StepMeta m, KvGeom g, int layer,
                                                                int H, int Hkv, int hd,
                                                                const float *q, const T *kc,
                                                                const T *vc, float *out) {
  __shared__ float qs[256];
  __shared__ float sc[256];
  __shared__ float red[16];
  __shared__ float osum[256];
  const int r = blockIdx.x, a = blockIdx.y, tid = threadIdx.x;
  const int seq = m.seq[r], b = a / (H / Hkv);
  const int L = m.kv_len[seq], n = m.n_nodes[seq], T_all = L + n;
  const uint64_t anc = m.anc[r];
  const float scale = 1.0f / sqrtf((float)hd);
  if (tid < hd) qs[tid] = q[((int64_t)r * H + a) * hd + tid] * scale;
  __syncthreads();
  const T *kbase = kc + g.row(seq, layer, b, 0);
  const T *vbase = vc + g.row(seq, layer, b, 0);
  const int groups = 256 / hd, grp = tid / hd, c = tid - grp * hd;
  float m_run = -INFINITY, l_run = 0.f, o = 0.f;
  for (int t0 = 0; t0 < T_all; t0 += 256) {
    const int t = t0 + tid;
    const bool valid = t < T_all && (t < L || ((anc >> (t - L)) & 1ull));
    float s = -INFINITY;
    if (valid) {
      const T *kr = kbase + (int64_t)t * hd;
      float acc = 0.f;
#pragma unroll 16
      for (int e = 0; e < hd; e += 4) {  // hd is a multiple of 8
        float k4[4];
        Vec4<T>::load(kr + e, k4);
        acc += qs[e] * k4[0];
        acc += qs[e + 1] * k4[1];
        acc += qs[e + 2] * k4[2];
        acc += qs[e + 3] * k4[3];
      }
      s = acc;
    }
    const float cm = block_max(s, red);
    const float m_new = fmaxf(m_run, cm);
    if (m_new == -INFINITY) continue;  // a chunk with no visible key (uniform across the block)
    const float p = valid ? __expf(s - m_new) : 0.f;
    __syncthreads();
    sc[tid] = p;
    const float ls = block_sum(p, red);  // contains the barriers that publish sc[]
    const float alpha = (m_run == -INFINITY) ? 0.f : __expf(m_run - m_new);
    l_run = l_run * alpha + ls;
    o *= alpha;
    const int cnt = min(256, T_all - t0);
    int j = grp;
    for (; j + 7 * groups < cnt; j += 8 * groups) {  // 8 rows in flight
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = to_f32(vbase[(int64_t)(t0 + j + u * groups) * hd + c]);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float pj = sc[j + u * groups];
        if (pj != 0.f) o += pj * v[u];  // a masked row may hold anything
      }
    }
    for (; j < cnt; j += groups) {
      const float pj = sc[j];
      if (pj != 0.f) o += pj * to_f32(vbase[(int64_t)(t0 + j) * hd + c]);
    }
    m_run = m_new;
    __syncthreads();
  }
  osum[tid] = o;
  __syncthreads();
  if (tid < hd) {
    float tot = 0.f;
    for (int gi = 0; gi < groups; ++gi) tot += osum[gi * hd + tid];
    out[((int64_t)r * H + a) * hd + tid] = tot / l_run;
  }
}

void launch_attention_generic(const StepMeta &m, const ModelDims &md, const KvGeom &g, int layer,
                              const float *q, const void *kc, const void *vc, float *out,
                              hipStream_t st) {
  dim3 grid(m.rows, md.n_heads);
  if (md.dtype == 1)
    attention_generic_kernel<bf16_t><<<grid, 256, 0, st>>>(m, g, layer, md.n_heads, md.n_kv_heads, md.head_dim, q, (const bf16_t *)kc, (const bf16_t *)vc, out);
  else
    attention_generic_kernel<float><<<grid, 256, 0, st>>>(m, g, layer, md.n_heads, md.n_kv_heads, md.head_dim, q, (const float *)kc, (const float *)vc, out);
}

// --------------------------------------------------------------------------- argmax
__global__ __launch_bounds__(256) void argmax_kernel(StepMeta m, const float *logits, int padded,
                                                     int max_nodes, int V, int32_t *argmax) {
  __shared__ float bv[4];
  __shared__ int bi[4];
  const int r = blockIdx.x;
  const int orow = m.seq[r] * max_nodes + m.node[r];
  const float *row = logits + (int64_t)(padded ? orow : r) * V;
  float best = -INFINITY;
  int besti = 0x7fffffff;
  for (int t0 = threadIdx.x; t0 < V; t0 += 256 * 8) {  // 8 loads in flight
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (t0 + i * 256 < V) v[i] = row[t0 + i * 256];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int t = t0 + i * 256;
      if (t < V && (v[i] > best || (v[i] == best && t < besti))) { best = v[i]; besti = t; }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(best, o, 64);
    int oi = __shfl_xor(besti, o, 64);
    if (ov > best || (ov == best && oi < besti)) { best = ov; besti = oi; }
  }
  if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = besti; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (bv[w] > best || (bv[w] == best && bi[w] < besti)) { best = bv[w]; besti = bi[w]; }
    argmax[orow] = besti == 0x7fffffff ? 0 : besti;
  }
}

void launch_argmax(const StepMeta &m, const float *logits, bool padded_in, int max_nodes, int V,
                   int32_t *argmax, hipStream_t st) {
  argmax_kernel<<<m.rows, 256, 0, st>>>(m, logits, padded_in ? 1 : 0, max_nodes, V, argmax);
}

// The same for the caller's padded logits, the vocabulary of a row cut into pieces of kArgmaxPiece ids so
// that a 64-node tree fills the chip (64 rows x 32000: one workgroup per row 23.4 us, 8 per row 4.5):
// record (value, lowest id) per (row, piece); accept_kernel merges them.
constexpr int kArgmaxPiece = 4096;
int argmax_pieces(int V) { return (V + kArgmaxPiece - 1) / kArgmaxPiece; }

// grid rows * pieces: rows alone may exceed the 65535 workgroups of the second dimension.
__global__ __launch_bounds__(256) void argmax_pieces_kernel(StepMeta m, const float *logits, int max_nodes, int V, int pieces, float2 *rec) {
  __shared__ float bv[4];
  __shared__ int bi[4];
  const int r = blockIdx.x / (uint32_t)pieces, t0 = (blockIdx.x - r * pieces) * kArgmaxPiece;
  const float *row = logits + (int64_t)(m.batch == 1 ? r : m.seq[r] * max_nodes + m.node[r]) * V;
  float best = -INFINITY;
  int besti = 0x7fffffff;
  auto take = [&](float v, int t) {
    if (v > best || (v == best && t < besti)) { best = v; besti = t; }
  };
  const int t1 = min(t0 + kArgmaxPiece, V);
  if ((V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0) {  // every row starts on 16 bytes
    float4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + (i * 256 + (int)threadIdx.x) * 4;
      v[i] = t < t1 ? *reinterpret_cast<const float4 *>(row + t) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + (i * 256 + (int)threadIdx.x) * 4;
      if (t < t1) { take(v[i].x, t); take(v[i].y, t + 1); take(v[i].z, t + 2); take(v[i].w, t + 3); }
    }
  } else {
    for (int t = t0 + threadIdx.x; t < t1; t += 256) take(row[t], t);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(besti, o, 64);
    take(ov, oi);
  }
  if ((threadIdx.x & 63) == 0) { bv[threadIdx.x >> 6] = best; bi[threadIdx.x >> 6] = besti; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) take(bv[w], bi[w]);
    rec[blockIdx.x] = make_float2(best, __int_as_float(besti));
  }
}

// --------------------------------------------------------------------------- draft-side read-out
// Per row: the ids of the largest and the second largest logit and the softmax probability of
// the largest -- the draft model's normalised logit that is compared with a threshold, and the
// candidate of second highest probability that a sparse tree expands (Sec. IV-A, Sec. IV-C).
// Order: value descending, id ascending among equal values.
struct Top2 {
  float v1, v2;
  int i1, i2;
};
__device__ __forceinline__ bool top2_before(float a, int ia, float b, int ib) {
  return a > b || (a == b && ia < ib);
}
__device__ __forceinline__ void top2_push(Top2 &t, float v, int i) {
  if (top2_before(v, i, t.v1, t.i1)) {
    t.v2 = t.v1; t.i2 = t.i1; t.v1 = v; t.i1 = i;
  } else if (top2_before(v, i, t.v2, t.i2)) {
    t.v2 = v; t.i2 = i;
  }
}
__device__ __forceinline__ Top2 top2_merge(const Top2 &a, const Top2 &b) {
  Top2 r = a;
  top2_push(r, b.v1, b.i1);
  top2_push(r, b.v2, b.i2);
  return r;
}
__device__ __forceinline__ Top2 top2_wave(Top2 t) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    Top2 u;
    u.v1 = __shfl_xor(t.v1, o, 64); u.v2 = __shfl_xor(t.v2, o, 64);
    u.i1 = __shfl_xor(t.i1, o, 64); u.i2 = __shfl_xor(t.i2, o, 64);
    t = top2_merge(t, u);
  }
  return t;
}
constexpr int kNoId = 0x7fffffff;

// Stage 1, grid (blocks of 1024 ids, rows), block 256, 4 consecutive ids per thread.  SRC = 0: the
// logits are compact rows [rows][V]; SRC = 1: they are split-k partial sums (part_offset) that
// are summed here, multiplied by 1/rms of the row when nrm.ssq is set (second half of the final
// RMSNorm), and optionally stored into the caller's padded [batch][max_nodes][V] array.
// Record per (row, block): (v1, v2, sum of exp(v - v1) over the block), (i1, i2).
template <int SRC>
__global__ __launch_bounds__(256) void top2_blocks_kernel(StepMeta m, const float *src, int n_splits,
                                                          int ldp, RowNorm nrm, int V,
                                                          int max_nodes, float *logits_out,
                                                          float *rec_v, int *rec_i) {
  __shared__ Top2 wt[4];
  __shared__ float ws[4];
  const int r = blockIdx.y, rows = m.rows;
  const float rs = (SRC == 1 && nrm.ssq != nullptr) ? row_rms_scale(nrm, r) : 1.0f;
  const int v0 = (blockIdx.x * 256 + threadIdx.x) * 4;
  float vals[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (v0 < V) {
    if (SRC == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (v0 + i < V) vals[i] = src[(int64_t)r * V + v0 + i];
    } else {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int s = 0; s < n_splits; ++s) {
        const float4 p = *reinterpret_cast<const float4 *>(src + part_offset(s, r, v0, ldp >> 5, part_rows_pad(rows)));
        a.x += p.x; a.y += p.y; a.z += p.z; a.w += p.w;
      }
      const float t[4] = {a.x * rs, a.y * rs, a.z * rs, a.w * rs};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (v0 + i < V) vals[i] = t[i];
    }
    if (logits_out) {
      float *dst = logits_out + ((int64_t)m.seq[r] * max_nodes + m.node[r]) * V + v0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (v0 + i < V) dst[i] = vals[i];
    }
  }
  Top2 t{-INFINITY, -INFINITY, kNoId, kNoId};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (v0 + i < V) top2_push(t, vals[i], v0 + i);
  t = top2_wave(t);
  if ((threadIdx.x & 63) == 0) wt[threadIdx.x >> 6] = t;
  __syncthreads();
  t = top2_merge(top2_merge(wt[0], wt[1]), top2_merge(wt[2], wt[3]));
  float e = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (v0 + i < V) e += __expf(vals[i] - t.v1);
  e = wave_sum(e);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t o = (int64_t)r * gridDim.x + blockIdx.x;
    rec_v[o * 3] = t.v1;
    rec_v[o * 3 + 1] = t.v2;
    rec_v[o * 3 + 2] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
    rec_i[o * 2] = t.i1;
    rec_i[o * 2 + 1] = t.i2;
  }
}

// Stage 2, one wavefront per row: merge the block records.  p1 = 1 / sum_b s_b * exp(v1_b - v1).
__global__ __launch_bounds__(64) void top2_merge_kernel(StepMeta m, const float *rec_v,
                                                        const int *rec_i, int n_blk, int max_nodes,
                                                        int32_t *top2, float *prob, int32_t *argmax) {
  const int r = blockIdx.x;
  Top2 t{-INFINITY, -INFINITY, kNoId, kNoId};
  for (int b = threadIdx.x; b < n_blk; b += 64) {
    const int64_t o = (int64_t)r * n_blk + b;
    const Top2 u{rec_v[o * 3], rec_v[o * 3 + 1], rec_i[o * 2], rec_i[o * 2 + 1]};
    t = top2_merge(t, u);
  }
  t = top2_wave(t);
  float sum = 0.f;
  for (int b = threadIdx.x; b < n_blk; b += 64) {
    const int64_t o = (int64_t)r * n_blk + b;
    sum += rec_v[o * 3 + 2] * __expf(rec_v[o * 3] - t.v1);
  }
  sum = wave_sum(sum);
  if (threadIdx.x == 0) {
    const int64_t orow = (int64_t)m.seq[r] * max_nodes + m.node[r];
    top2[orow * 2] = t.i1 == kNoId ? 0 : t.i1;
    top2[orow * 2 + 1] = t.i2 == kNoId ? -1 : t.i2;
    prob[orow] = 1.0f / sum;
    if (argmax) argmax[orow] = t.i1 == kNoId ? 0 : t.i1;
  }
}

int top2_blocks(int V) { return ((V + 3) / 4 + 255) / 256; }

void launch_top2(const StepMeta &m, const float *src, bool from_partials, int n_splits, int ldp,
                 const RowNorm &nrm, int V, int max_nodes, float *logits_out, float *rec_v, int *rec_i, int32_t *top2,
                 float *prob, int32_t *argmax, hipStream_t st) {
  const int n_blk = top2_blocks(V);
  dim3 grid(n_blk, m.rows);
  if (from_partials)
    top2_blocks_kernel<1><<<grid, 256, 0, st>>>(m, src, n_splits, ldp, nrm, V, max_nodes, logits_out, rec_v, rec_i);
  else
    top2_blocks_kernel<0><<<grid, 256, 0, st>>>(m, src, 0, 0, nrm, V, max_nodes, logits_out, rec_v, rec_i);
  top2_merge_kernel<<<m.rows, 64, 0, st>>>(m, rec_v, rec_i, n_blk, max_nodes, top2, prob, argmax);
}

// --------------------------------------------------------------------------- acceptance
// One wavefront per sequence, lane i = tree node i (trees have at most 64 nodes).
// Sec. II-B: draft tokens are accepted while they match the target's output and
// verification stops at the first failure.  A node matches when its token equals the
// target's greedy token at its parent; ballot gathers the match flags into one mask; a node is
// acceptable when its ancestor mask has no unmatched bit; the deepest acceptable node wins
// (lowest index among equals).
// PER > 0: the argmax of a node is first merged from its piece records (argmax_pieces_kernel, logits_argmax_kernel) by PER
// threads and written to argmax_out; otherwise it is read from argmax.
template <int PER>
__global__ __launch_bounds__(64 * (PER ? PER : 1)) void accept_kernel(StepMeta m, int max_nodes, const int32_t *argmax,
                                                                      int32_t *argmax_out, const float2 *rec, int pieces, int32_t *path,
                                                                      int32_t *accept_len, int32_t *next_token, AcceptMirror host) {
  const int s = blockIdx.x, lane = threadIdx.x;
  const int n = m.seq_n_nodes(s), r0 = m.seq_row_start(s);
  bool matched = false;
  uint64_t anc = 0;
  int depth = 0, par = 0, tok = 0, mine = 0;
  __shared__ int merged[PER > 1 ? 64 : 1];
  if (lane < n) {
    par = max(m.parent[r0 + lane], 0);
    tok = m.token[r0 + lane];
    anc = m.anc[r0 + lane];
    depth = m.depth[r0 + lane];
    if (PER == 0) mine = argmax[(int64_t)s * max_nodes + lane];
  }
  if constexpr (PER > 0) {
    const int node = threadIdx.x / PER, part = threadIdx.x % PER;
    float best = -INFINITY;
    int besti = 0x7fffffff;
    auto take = [&](float v, int i) {
      if (v > best || (v == best && i < besti)) { best = v; besti = i; }
    };
    if (node < n) {
      const float2 *p = rec + (int64_t)(r0 + node) * pieces;
#pragma unroll PER > 1 ? 4 : 16
      for (int i = part; i < pieces; i += PER) {
        const float2 q = p[i];
        take(q.x, __float_as_int(q.y));
      }
    }
#pragma unroll
    for (int o = PER / 2; o > 0; o >>= 1) {
      const float ov = __shfl_xor(best, o, 64);
      take(ov, __shfl_xor(besti, o, 64));
    }
    mine = besti == 0x7fffffff ? 0 : besti;
    if (PER > 1) {
      if (part == 0) merged[node] = mine;
      __syncthreads();
      if (threadIdx.x >= 64) return;
      mine = merged[lane];
    }
    if (lane < n) argmax_out[(int64_t)s * max_nodes + lane] = mine;
  }
  const int want = __shfl(mine, par, 64);  // the target's token after the parent
  if (lane < n) matched = lane == 0 || tok == want;
  const uint64_t mm = __ballot(matched);
  const bool ok = lane < n && (anc & ~mm) == 0ull;
  int key = ok ? (depth * 64 + (63 - lane)) : -1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) key = max(key, __shfl_xor(key, o, 64));
  const int win = 63 - (key & 63);
  const uint64_t wanc = __shfl(anc, win, 64);
  const int wdepth = key >> 6;
  const int next = __shfl(mine, win, 64);
  auto write = [&](int32_t *path_, int32_t *len_, int32_t *next_) {
    int32_t *p = path_ + (int64_t)s * max_nodes;
    if (lane < max_nodes && lane > wdepth) p[lane] = -1;
    if (lane < n && ((wanc >> lane) & 1ull)) p[depth] = lane;
    if (lane == 0) {
      len_[s] = wdepth + 1;
      next_[s] = next;
    }
  };
  write(path, accept_len, next_token);
  if (host.path != nullptr) {
    write(host.path, host.accept_len, host.next_token);
    if (lane < n) host.argmax[(int64_t)s * max_nodes + lane] = mine;
  }
}

void launch_accept(const StepMeta &m, int max_nodes, const int32_t *argmax, int32_t *path,
                   int32_t *accept_len, int32_t *next_token, hipStream_t st, const AcceptMirror &host) {
  accept_kernel<0><<<m.batch, 64, 0, st>>>(m, max_nodes, argmax, nullptr, nullptr, 0, path, accept_len, next_token, host);
}

void launch_accept_records(const StepMeta &m, int max_nodes, const float2 *rec, int pieces, int32_t *argmax, int32_t *path,
                           int32_t *accept_len, int32_t *next_token, hipStream_t st, const AcceptMirror &host) {
  // A thread of its own reads a node's records one by one, a line each, but needs no barrier.  Verify of a one-layer model, us,
  // one thread / 16 per node: 4000 ids (4 records), 64 nodes equal, 32000 ids (32) 106 / 103, 100352 ids (98) 144 / 127,
  // 152064 ids (149) 185 / 142, 8 nodes 129 / 104; accept_from_logits of 32000 ids (8), 64 nodes 30.3 / 31.4.
  if (pieces > 16)
    accept_kernel<16><<<m.batch, 1024, 0, st>>>(m, max_nodes, nullptr, argmax, rec, pieces, path, accept_len, next_token, host);
  else
    accept_kernel<1><<<m.batch, 64, 0, st>>>(m, max_nodes, nullptr, argmax, rec, pieces, path, accept_len, next_token, host);
}

void launch_argmax_accept(const StepMeta &m, const float *logits, int max_nodes, int V, float *rec, int32_t *argmax,
                          int32_t *path, int32_t *accept_len, int32_t *next_token, hipStream_t st) {
  const int pieces = argmax_pieces(V);
  argmax_pieces_kernel<<<(unsigned)m.rows * pieces, 256, 0, st>>>(m, logits, max_nodes, V, pieces, (float2 *)rec);
  launch_accept_records(m, max_nodes, (const float2 *)rec, pieces, argmax, path, accept_len, next_token, st);
}

// --------------------------------------------------------------------------- KV compaction
// Moves cache slot kv_len + path[k] to slot kv_len + k (k < accept_len) for one (sequence, layer, K|V) and up to
// kCompactHeads KV heads per block.  Since path is strictly increasing with path[k] >= k, a destination slot may be another
// move's source: every source row of a head is read into registers, the block synchronises, and only then is anything
// written.  Usually the accepted path is the front of the trunk and nothing moves (path[len - 1] == len - 1 says so):
// then the launch is bound by its number of blocks.  7B class, one block per head -> this: 4 sequences, nothing moves 22.2
// -> 2.3 us, 19 of 64 rows move 45 -> 16; one sequence 7.5 -> 1.9, 12.4 -> 8.3.  (Where few heads are left to few blocks, moving
// takes a little longer: 1.1B class, one sequence 4.6 -> 4.9, 62 rows 5.0 -> 6.4.)
constexpr int kCompactHeads = 8;
typedef __attribute__((ext_vector_type(4))) uint32_t mv16_t;  // one 16-byte unit of a cache row

template <int UNITS>
__global__ __launch_bounds__(256) void compact_kernel(KvGeom g, int max_nodes, int row_bytes,
                                                      const int32_t *kv_len, const int32_t *path,
                                                      const int32_t *accept_len, char *kc, char *vc,
                                                      int elem_bytes) {
  uint32_t idx = blockIdx.x;
  const uint32_t hg = (uint32_t)(g.n_kv_heads + kCompactHeads - 1) / kCompactHeads;
  const int which = idx & 1; idx >>= 1;
  const int h_first = (int)(idx % hg) * kCompactHeads; idx /= hg;
  const int layer = (int)(idx % (uint32_t)g.n_layers), seq = (int)(idx / (uint32_t)g.n_layers);
  const int len = accept_len[seq];
  const int32_t *p = path + (int64_t)seq * max_nodes;
  if (p[len - 1] == len - 1) return;
  const int h_end = min(h_first + kCompactHeads, g.n_kv_heads);
  const int upr = row_bytes / 16;  // 16-byte units per row
  const int total = len * upr;     // units of one head
  const int64_t head_bytes = g.capacity * row_bytes;
  char *base = (which ? vc : kc) + g.row(seq, layer, h_first, kv_len[seq]) * elem_bytes;
  if (total <= 256 * UNITS) {
    const int heads = min(256 * UNITS / total, h_end - h_first);  // at a time
    for (int h = h_first; h < h_end; h += heads, base += heads * head_bytes) {
      const int n = min(heads, h_end - h) * total;
      mv16_t regs[UNITS];
#pragma unroll
      for (int i = 0; i < UNITS; ++i) {
        const int u = threadIdx.x + i * 256;
        if (u < n) {
          const int hh = u / total, v = u - hh * total, k = v / upr, w = v - k * upr, src = p[k];
          regs[i] = (mv16_t){0u, 0u, 0u, 0u};
          if (src != k) regs[i] = *reinterpret_cast<const mv16_t *>(base + hh * head_bytes + (int64_t)src * row_bytes + w * 16);
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < UNITS; ++i) {
        const int u = threadIdx.x + i * 256;
        if (u < n) {
          const int hh = u / total, v = u - hh * total, k = v / upr, w = v - k * upr;
          if (p[k] != k) *reinterpret_cast<mv16_t *>(base + hh * head_bytes + (int64_t)k * row_bytes + w * 16) = regs[i];
        }
      }
    }
  } else {
    // rows too large to stage at once: ascending order is safe because the source of move k'
    // (> k) lies beyond every destination written so far.
    for (int h = h_first; h < h_end; ++h, base += head_bytes)
      for (int k = 0; k < len; ++k) {
        const int src = p[k];
        if (src == k) continue;
        // one row is at most 1 KB = 64 units: every thread moves at most one
        mv16_t v = (mv16_t){0u, 0u, 0u, 0u};
        if ((int)threadIdx.x < upr)
          v = *reinterpret_cast<const mv16_t *>(base + (int64_t)src * row_bytes + threadIdx.x * 16);
        __syncthreads();
        if ((int)threadIdx.x < upr)
          *reinterpret_cast<mv16_t *>(base + (int64_t)k * row_bytes + threadIdx.x * 16) = v;
        __syncthreads();
      }
  }
}

void launch_compact(int dtype, const KvGeom &g, int batch, int max_nodes, const int32_t *kv_len,
                    const int32_t *path, const int32_t *accept_len, void *kc, void *vc,
                    hipStream_t st) {
  const int eb = dtype == 1 ? 2 : 4;
  const int row_bytes = g.head_dim * eb;  // multiple of 16: head_dim % 8 == 0
  const int blocks = batch * g.n_layers * ((g.n_kv_heads + kCompactHeads - 1) / kCompactHeads) * 2;
  compact_kernel<8><<<blocks, 256, 0, st>>>(g, max_nodes, row_bytes, kv_len, path, accept_len,
                                           (char *)kc, (char *)vc, eb);
}

}  // namespace specasr
