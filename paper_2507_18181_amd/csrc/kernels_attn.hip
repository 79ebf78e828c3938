// Tree-masked attention for gfx950 with bf16 MFMA (Sec. II-B: 2D attention mask over the draft
// token tree; Sec. IV-C: used to verify the two-pass sparse tree).
//
// Every tree node attends to the cached prefix [0, kv_len) and to the cache slots of the nodes
// on its own root path.  A workgroup takes (sequence, KV head, 32 query rows, chunk of keys); the
// query rows that share the head are the grouped-query heads times the tree nodes.  Its wavefronts
// take the chunk's 32-key tiles round-robin, each with its own online softmax, and are merged
// through LDS at the end.
//
//   S^T[key][query] = K[key][:] . Q[query][:]      A = K tile, B = Q^T
//   online softmax per query column (fp32, base 2: log2(e) is part of the query scale)
//   Q and P enter the matrix cores as hi + lo bf16 planes (two MFMAs), so only the bf16 storage
//   of the cache itself limits the precision.
//   O^T[c][query]  += V^T[c][key] * P^T[key][query] A = V^T, B = P^T, which is exactly how the lanes
//                                                   already hold P
//
// K and V tiles go into LDS row by row with direct-to-LDS loads (whole 128-byte lines per request, no
// staging registers), 16-byte chunks of a row XOR-permuted by its row number so that both kinds of
// read are free of bank conflicts beyond the minimum: K as 16-byte rows of the A operand, V^T through the
// transposing LDS read (ds_read_b64_tr_b16: 16 lanes give 4 rows x 16 columns and get 4 keys of one
// column each).  Each wavefront has one buffer for K and one for V and requests the next tile of
// either as soon as the current one has been consumed: K flies during softmax and PV, V during the
// next QK^T and softmax.  The first tile overlaps nothing: the queries are requested behind its K and V,
// and the compiler waits for every load in front of the loop.  So a wavefront with one tile (7B, 842 keys: 7 chunks
// of 128) waits for K, V and queries once and then computes.
//
// What bounds it: per 32 x 32 tile 32 MFMAs (head_dim 128; 1024 cycles) and about 170 vector
// instructions; two wavefronts per SIMD overlap the two.
#include "kernels.h"
#include "attn_tile.h"
#include "kernels_mfma.h"

namespace specasr {

constexpr int kAttnWaves = 4;  // 8 were measured: 5 .. 30 % slower everywhere (more outputs to merge per workgroup)

// grid (8 * n_rg * ceil(n_chunks * Hkv / 8), 1, batch), block 256.  Workgroups go to the 8 XCDs
// round-robin by their linear index, so the n_rg workgroups that stream the SAME keys for
// different query row groups are placed 8 apart: they run on one XCD and share its L2.
// Sequences of a batched call in the kernel arguments (up to 16), in dispatch order, longest first: all
// of a workgroup's metadata is one scalar load (the arrays in memory are a cold load each), and the
// workgroups that start last are short (16 utterances on the 1.1B model 23.2 -> 21.0 us).
struct AttnSeqs {
  int4 e[16];     // kv_len, n_nodes, first row, sequence
  int32_t count;  // 0: one sequence (StepMeta has it) or more than 16 (metadata arrays)
};

template <int HD, bool DIRECT>
__global__ __launch_bounds__(64 * kAttnWaves, HD == 64 ? 3 : 2) void tree_attention_kernel(StepMeta m, AttnSeqs sq, KvGeom g, int layer, int H,
                                                                    int Hkv, int n_rg,
                                                                    const uint16_t *__restrict__ qb,
                                                                    const uint16_t *__restrict__ qb_lo,
                                                                    const uint16_t *__restrict__ kc,
                                                                    const uint16_t *__restrict__ vc,
                                                                    int chunk_keys, int n_chunks,
                                                                    float *__restrict__ o_part,
                                                                    float *__restrict__ ml_part,
                                                                    uint16_t *__restrict__ out,
                                                                    uint16_t *__restrict__ out_lo, int nb) {
  constexpr int KK = HD / 16;         // MFMA k-steps across the head dimension
  constexpr int CB = HD / 32;         // 32-wide output column blocks
  constexpr int CR = HD / 8;          // 16-byte chunks of a row
  constexpr int TU = 32 * CR;         // 16-byte units of a tile
  constexpr int NI = TU / 64;         // direct-to-LDS loads of a tile
  constexpr int RI = 64 / CR;         // rows per such load
  constexpr int NW = kAttnWaves;
  __shared__ u32x4 kbuf[NW * TU], vbuf[NW * TU];  // afterwards: the wavefronts' outputs, for the merge
  __shared__ float2 ml[NW * 32];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 5, ql = lane & 31;
  const uint32_t bx = blockIdx.x >> 3, rg = bx % (uint32_t)n_rg, base = bx / (uint32_t)n_rg * 8 + (blockIdx.x & 7);
  if (base >= (uint32_t)(n_chunks * Hkv)) return;
  const int chunk = base % (uint32_t)n_chunks, kvh = base / (uint32_t)n_chunks;
  int seq = gridDim.z - 1 - blockIdx.z, L, n, r0;
  if (sq.count) {
    const int4 e = sq.e[blockIdx.z];
    L = e.x; n = e.y; r0 = e.z; seq = e.w;
  } else {
    L = m.seq_kv_len(seq); n = m.seq_n_nodes(seq); r0 = m.seq_row_start(seq);
  }
  const int G = (uint32_t)H / (uint32_t)Hkv, rows = m.rows;
  const int T = L + n, QR = G * n;
  const int t_begin = chunk * chunk_keys;
  if (t_begin >= T || (int)rg * 32 >= QR) return;
  const int t_end = min(T, t_begin + chunk_keys);

  const char *kbase = reinterpret_cast<const char *>(kc + g.row(seq, layer, kvh, 0));
  const char *vbase = reinterpret_cast<const char *>(vc + g.row(seq, layer, kvh, 0));
  u32x4 *kb = kbuf + wave * TU, *vb = vbuf + wave * TU;
  // load i of a tile: lane l brings chunk c of row r = RI*i + l/CR to position l of the 1 KB block i.  The
  // tile's first row is part of the 64-bit scalar base: one head's rows may exceed 4 GiB (2^24 keys of 128).
  const int lr = lane / CR;
  auto issue = [&](const char *src, u32x4 *dst, int t0) {
    const char *tile = src + (int64_t)t0 * (HD * 2);
    const int last = T - 1 - t0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = RI * i + lr, c = (lane & (CR - 1)) ^ swizzle<HD>(r);
      load_16_to_lds<DIRECT>(tile + (uint32_t)(min(r, last) * (HD * 2) + c * 16), dst + i * 64, lane);
    }
  };
  const int t_first = t_begin + 32 * wave;  // this wavefront's tiles: t_first, + 32 NW, ...
  if (t_first < t_end) {
    issue(kbase, kb, t_first);
    issue(vbase, vb, t_first);
  }

  // queries of this wavefront (the same 32 for all of them)
  const int qrow = rg * 32 + ql;
  const bool valid = qrow < QR;
  const int gi = valid ? (uint32_t)qrow / (uint32_t)n : 0, node = valid ? qrow - gi * n : 0;
  const int out_row = r0 + node, out_head = kvh * G + gi;
  const uint64_t anc = valid ? m.anc[out_row] : 0ull;
  u32x4 qh[KK], qlo[KK];  // queries as hi + lo bf16 planes; surplus columns repeat node 0, without stores
  {
    const int64_t qoff = ((int64_t)out_row * H + out_head) * HD + 8 * h;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qh[kk] = *reinterpret_cast<const u32x4 *>(qb + qoff + 16 * kk);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qlo[kk] = *reinterpret_cast<const u32x4 *>(qb_lo + qoff + 16 * kk);
  }
  TileState<HD> ts;
  ts.init(kb, vb, lane);

  // s_waitcnt immediates: vmcnt in bits 3:0 and 15:14; lgkmcnt and expcnt not waited for
  constexpr int kVm = 0x0F70 | NI, kVm0 = 0x0F70;
  for (int t0 = t_first; t0 < t_end; t0 += 32 * NW) {
    const bool more = t0 + 32 * NW < t_end;
    // K of this tile has landed; the NI loads of its V may still be in flight
    __builtin_amdgcn_s_waitcnt(kVm);
    asm volatile("" ::: "memory");
    ts.scores(qh, qlo);
    if (more) issue(kbase, kb, t0 + 32 * NW);
    if (t0 + 32 > L) {  // a tile with tree slots: bit i of w = key t0 + i is visible
      const int d = t0 - L;
      uint32_t w = d >= 0 ? (uint32_t)(anc >> d) : ((uint32_t)(anc << -d) | ((1u << -d) - 1u));
      ts.mask(w, h);
    }
    ts.softmax();
    // V of this tile has landed; the NI loads of the next K may still be in flight
    if (more) __builtin_amdgcn_s_waitcnt(kVm);
    else __builtin_amdgcn_s_waitcnt(kVm0);
    asm volatile("" ::: "memory");
    ts.values();
    if (more) issue(vbase, vb, t0 + 32 * NW);
  }

  // Merge: every wavefront leaves its output in its own two tile buffers (column blocks of the lower half of
  // the head in kbuf, of the upper half in vbuf), C layout [cb][q][lane] x 4 columns, then all threads
  // reduce: item = (cb, q, lane) = query lane%32, columns 32 cb + 8 q + 4 (lane/32) .. +3
  constexpr int HB = CB / 2;
  ts.l_run = sum_halves(ts.l_run);
  float4 *ko = reinterpret_cast<float4 *>(kbuf), *vo = reinterpret_cast<float4 *>(vbuf);
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    float4 *dst = (cb < HB ? ko : vo) + wave * TU + (cb % HB) * 256 + lane;
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[q * 64] = make_float4(ts.o[cb][4 * q], ts.o[cb][4 * q + 1], ts.o[cb][4 * q + 2], ts.o[cb][4 * q + 3]);
  }
  if (h == 0) ml[wave * 32 + ql] = make_float2(ts.m_run, ts.l_run);
  __syncthreads();
  if (!valid) return;
  float wgt[NW], M = -INFINITY, Lsum = 0.f;
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    wgt[v] = ml[v * 32 + ql].x;
    M = fmaxf(M, wgt[v]);
  }
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    wgt[v] = wgt[v] == -INFINITY ? 0.f : exp2_fast(wgt[v] - M);
    Lsum += wgt[v] * ml[v * 32 + ql].y;
  }
  const float inv = 1.f / Lsum;
  const int64_t pbase = ((int64_t)chunk * rows + out_row) * H + out_head;
  if (out == nullptr && wave == 0 && h == 0) *reinterpret_cast<float2 *>(ml_part + pbase * 2) = make_float2(M, Lsum);
#pragma unroll
  for (int u = wave; u < CB * 4; u += NW) {
    const int cb = u >> 2, q = u & 3;
    const float4 *src = (cb < HB ? ko : vo) + (cb % HB) * 256 + q * 64 + lane;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      const float4 z = src[v * TU];
      acc[0] += wgt[v] * z.x; acc[1] += wgt[v] * z.y; acc[2] += wgt[v] * z.z; acc[3] += wgt[v] * z.w;
    }
    const int col = 32 * cb + 8 * q + 4 * h;
    if (out != nullptr) {
      // every sequence is a single chunk: this IS the result -- normalise and write the packed hi/lo
      // planes the output projection reads (what the merge kernel would do with one chunk)
      uint32_t hi2[2], lo2[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) split_bf16_pair(div_by(acc[2 * i], Lsum, inv), div_by(acc[2 * i + 1], Lsum, inv), hi2[i], lo2[i]);
      const int64_t po = packed_act_offset(out_row, out_head * HD + col, nb);
      *reinterpret_cast<uint2 *>(out + po) = make_uint2(hi2[0], hi2[1]);
      *reinterpret_cast<uint2 *>(out_lo + po) = make_uint2(lo2[0], lo2[1]);
    } else {
      *reinterpret_cast<float4 *>(o_part + pbase * HD + col) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    }
  }
}

// Merge the key chunks: out = sum_c 2^(m_c - M) o_c / sum_c 2^(m_c - M) l_c, as hi/lo planes.  One thread
// per 4 columns of a (row, head): 16-byte loads, 8 chunks of them in flight (7B, 32 rows, 7 chunks: 4.9 us with
// one column per thread).  grid ceil(rows * H * HD / 1024), block 256.
template <int HD>
__global__ __launch_bounds__(256) void tree_attention_merge_kernel(StepMeta m, int H, int chunk_keys,
                                                                   const float *__restrict__ o_part,
                                                                   const float *__restrict__ ml_part,
                                                                   uint16_t *__restrict__ out, uint16_t *__restrict__ out_lo,
                                                                   int nb) {
  constexpr int TPR = HD / 4;  // threads per (row, head)
  const int rows = m.rows;
  const uint32_t rh = (blockIdx.x * 256 + threadIdx.x) / TPR;  // row * H + head
  if (rh >= (uint32_t)(rows * H)) return;
  const int c = (threadIdx.x & (TPR - 1)) * 4, r = rh / (uint32_t)H, a = rh - r * H;
  const int seq = m.seq_of_row(r);
  const int T = m.seq_kv_len(seq) + m.seq_n_nodes(seq);
  const int n_chunks = (uint32_t)(T + chunk_keys - 1) / (uint32_t)chunk_keys;
  // batches of 8 chunks with all loads issued together; running (max, numerator, denominator)
  float M = -INFINITY, den = 0.f, num[4] = {0.f, 0.f, 0.f, 0.f};
  const int64_t cstride = (int64_t)rows * H;
  for (int c0 = 0; c0 < n_chunks; c0 += 8) {
    float2 ml[8];
    float4 oc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t base = rh + min(c0 + i, n_chunks - 1) * cstride;
      ml[i] = *reinterpret_cast<const float2 *>(ml_part + base * 2);
      oc[i] = *reinterpret_cast<const float4 *>(o_part + base * HD + c);
    }
    float Mb = M;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (c0 + i >= n_chunks) ml[i].x = -INFINITY;
      Mb = fmaxf(Mb, ml[i].x);
    }
    if (Mb == -INFINITY) continue;
    const float scale = (M == -INFINITY) ? 0.f : exp2_fast(M - Mb);
    den *= scale;
#pragma unroll
    for (int k = 0; k < 4; ++k) num[k] *= scale;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float wgt = (ml[i].x == -INFINITY) ? 0.f : exp2_fast(ml[i].x - Mb);
      num[0] += wgt * oc[i].x; num[1] += wgt * oc[i].y; num[2] += wgt * oc[i].z; num[3] += wgt * oc[i].w;
      den += wgt * ml[i].y;
    }
    M = Mb;
  }
  const float inv = 1.f / den;
  uint32_t hi2[2], lo2[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) split_bf16_pair(div_by(num[2 * i], den, inv), div_by(num[2 * i + 1], den, inv), hi2[i], lo2[i]);
  const int64_t po = packed_act_offset(r, a * HD + c, nb);  // B-operand order of the output projection
  *reinterpret_cast<uint2 *>(out + po) = make_uint2(hi2[0], hi2[1]);
  *reinterpret_cast<uint2 *>(out_lo + po) = make_uint2(lo2[0], lo2[1]);
}

template <int HD>
static void launch_attn_hd(const StepMeta &m, const AttnSeqs &sq, const ModelDims &md, const KvGeom &g, int layer,
                           int max_seq_nodes, int chunk_keys, int n_chunks,
                           const uint16_t *qb, const uint16_t *qb_lo, const void *kc, const void *vc,
                           float *o_part, float *ml_part, uint16_t *out, uint16_t *out_lo, int nb,
                           hipStream_t st) {
  const int G = md.n_heads / md.n_kv_heads;
  const int row_groups = (G * max_seq_nodes + 31) / 32;
  const bool direct = n_chunks == 1;  // nothing to merge: the attention kernel writes the final planes
  dim3 grid((n_chunks * md.n_kv_heads + 7) / 8 * 8 * row_groups, 1, m.batch);
  const bool aligned = (((uintptr_t)kc | (uintptr_t)vc) & 15) == 0;
  const auto kernel = aligned ? tree_attention_kernel<HD, true> : tree_attention_kernel<HD, false>;
  kernel<<<grid, 64 * kAttnWaves, 0, st>>>(m, sq, g, layer, md.n_heads, md.n_kv_heads, row_groups, qb, qb_lo, (const uint16_t *)kc, (const uint16_t *)vc, chunk_keys, n_chunks, o_part, ml_part, direct ? out : nullptr, direct ? out_lo : nullptr, nb);
  if (direct) return;
  const unsigned mgrid = (unsigned)(((int64_t)m.rows * md.n_heads * HD + 1023) / 1024);
  tree_attention_merge_kernel<HD><<<mgrid, 256, 0, st>>>(m, md.n_heads, chunk_keys, o_part, ml_part, out, out_lo, nb);
}

float tree_attention_qscale(int head_dim) { return 1.44269504088896340736f / sqrtf((float)head_dim); }

bool tree_attention_supported(int head_dim) { return head_dim == 64 || head_dim == 128; }

int tree_attention_max_chunks(int n_kv_heads) { return 256 / n_kv_heads + 2; }

// Key-chunk size (a multiple of 32).  One sequence: ~256 workgroups (one per compute unit) over
// its keys.  Several sequences (a batch, or the pieces of a wide prefill pass): if (KV heads x
// sequences x row-group blocks) already gives half a workgroup per compute unit, every sequence is one
// chunk and no merge runs (4 utterances of 200 .. 1500 keys on the 7B model, 128 workgroups: 23.2 us against
// 19.0 + 6.0 in chunks of 320 keys) -- below one workgroup per compute unit only up to 2048 keys, beyond that the idle
// half of the chip costs more than the merge (7B, 4 utterances of 200 .. 2000 / 4000 / 12000 keys: a call 1.00 / 0.93 /
// 0.84 times as fast in one chunk; 1.1B, 8 of up to 2000 / 4000 / 8000: 1.02 / 0.95 / 0.79); otherwise the sequences differ in length and there are few heads to
// spread them, so the chunks are made smaller -- ~1024 workgroups if all were as long as the longest, at
// least 128 keys (one tile per wavefront) -- and the short ones simply need fewer of them; the number of
// chunks stays within what the wide workspace holds (128 / n_kv_heads + 1).
int tree_attention_chunk_keys(int max_total_keys, int n_kv_heads, int batch, int row_group_blocks, int min_chunk_keys) {
  const long target = batch > 1 ? 1024 : 256;
  long want = ((long)max_total_keys * n_kv_heads * batch * row_group_blocks + target - 1) / target;
  long ck = (want + 31) / 32 * 32;
  // at least one tile per wavefront; more chunks only make the merge longer (1.1B, one row, 1600 keys: attention +
  // merge 8.5 us with chunks of 256 keys, 9.0 with 128)
  if (ck < 128) ck = batch == 1 && max_total_keys > 1280 ? 256 : 128;
  // a short single sequence: one chunk, the attention kernel writes the result itself and no merge
  // kernel runs.  1.1B: 0.7 us per further round of 4 tiles against 3.1 for the merge (one chunk: 5.9 us at 331 keys,
  // about 8 at 700; 128-key chunks + merge 7.9 at 800); 7B, 32 nodes: 1.1 us against 4.5 (842 keys: 14.7
  // against 13.5)
  if (batch == 1 && max_total_keys <= 704) ck = 704;
  if (batch > 1) {
    const long wgs = (long)n_kv_heads * batch * row_group_blocks;
    if (wgs >= 256 || (wgs >= 128 && max_total_keys <= 2048)) ck = ((long)max_total_keys + 31) / 32 * 32;
    const long max_chunks = 128 / n_kv_heads + 1;
    const long ck_min = ((max_total_keys + max_chunks - 1) / max_chunks + 31) / 32 * 32;
    if (ck < ck_min) ck = ck_min;
  }
  if (min_chunk_keys / 32 * 32 > ck) ck = min_chunk_keys / 32 * 32;  // development aid: never below the automatic size
  return (int)ck;
}

void launch_tree_attention(const StepMeta &m, const ModelDims &md, const KvGeom &g, int layer,
                           int max_total_keys, int max_seq_nodes, const uint16_t *qb,
                           const uint16_t *qb_lo, const void *kc, const void *vc, float *o_part,
                           float *ml_part, uint16_t *out, uint16_t *out_lo, int nb, int min_chunk_keys,
                           const int32_t *seq_kv_len, const int32_t *seq_row_start, const int32_t *seq_n_nodes, hipStream_t st) {
  AttnSeqs sq{};
  if (m.batch > 1 && m.batch <= 16) {
    sq.count = m.batch;
    for (int b = 0; b < m.batch; ++b) {
      const int4 e = make_int4(seq_kv_len[b], seq_n_nodes[b], seq_row_start[b], b);
      int at = b;  // insertion by falling key count
      for (; at > 0 && sq.e[at - 1].x + sq.e[at - 1].y < e.x + e.y; --at) sq.e[at] = sq.e[at - 1];
      sq.e[at] = e;
    }
  }
  const int G = md.n_heads / md.n_kv_heads;
  // One query row group (32 rows) per workgroup.  Two per workgroup would halve the key traffic
  // (head_dim 64: the accumulators would fit), but the keys of a head are L2 hits after their
  // first use and the kernel is bound by its softmax arithmetic: measured slower wherever it was
  // tried (16 utterances on the 1.1B model: 43 against 38 us).
  const int row_groups = (G * max_seq_nodes + 31) / 32;
  const int ck = tree_attention_chunk_keys(max_total_keys, md.n_kv_heads, m.batch, row_groups, min_chunk_keys);
  const int n_chunks = (max_total_keys + ck - 1) / ck;
  if (md.head_dim == 64)
    launch_attn_hd<64>(m, sq, md, g, layer, max_seq_nodes, ck, n_chunks, qb, qb_lo, kc, vc, o_part, ml_part, out, out_lo, nb, st);
  else
    launch_attn_hd<128>(m, sq, md, g, layer, max_seq_nodes, ck, n_chunks, qb, qb_lo, kc, vc, o_part, ml_part, out, out_lo, nb, st);
}

}  // namespace specasr
