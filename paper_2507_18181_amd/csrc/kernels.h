// Host-callable launchers of the device stages.  Every launcher only enqueues work on
// `st`; none synchronises or allocates.
#pragma once
#include "common.h"

namespace specasr {

struct ModelDims {
  int32_t n_layers, d_model, n_heads, n_kv_heads, head_dim, d_ffn, vocab;
  float rms_eps, rope_theta;
  int32_t dtype;  // 0 = fp32, 1 = bf16 storage
};

// ---- dtype-generic stages (fp32 arithmetic on fp32 activations) ----------
// Start of a forward: x[row][:] = tok_embed[token[row]][:] (or the caller's embedding row); the rope table
// cs[row][j] = (cos, sin)(pos[row] * theta^(-2j/hd)), computed in fp64; the metadata block words -> dst; and with pl (bf16
// models) the planes of x * gain with the sums of squares per 32 columns.  hm: the metadata in pinned host memory, as
// the device sees it.
struct BeginPlanes {
  const uint16_t *gain;
  uint16_t *hb, *hb_lo;
  int nb;
  float *ssq;
  int n_slab;
  // for a forward in one launch (kernels_one.hip): rows of its planes (0: packed as above), and what is filled with ones
  int rp = 0;
  uint4 *fill = nullptr;
  uint32_t fill_units = 0;
  int fill_blocks = 0;
  uint32_t *ctl = nullptr;
};
void launch_begin(const StepMeta &hm, int dtype, const void *tok_embed, const void *input_embeds, int max_nodes, int d, float *x, int hd,
                  float theta, float2 *cs, const BeginPlanes *pl, const int32_t *words, int32_t *dst, int n_words, hipStream_t st);
// Input of the linears below: residual rows x [rows][d] that are normalised first, x * rsqrt(mean(x^2)+eps) * gain, either
// by the linear itself or (wide rows, many rows, a gain that is not on 4 elements) into the scratch rows h
struct NormIn {
  const float *x;
  const void *gain;
  int rows, d;
  float eps;
  float *h;
};
bool linear_normalises(int d, const void *gain, int elem_bytes, int rows);
// y[row][o] += sum_k W[o][k] * a[row][k]
void launch_linear_add(int dtype, const void *W, int n_out, int n_in, const float *a, float *y, int rows, hipStream_t st);
struct LinearJob {
  const void *W;
  int n_out;
  float *y;
  int ldy;
};
// t[row][f] = silu(gate[f] . h[row]) * (up[f] . h[row])
void launch_linear_swiglu(int dtype, const NormIn &nx, const void *gate, const void *up, int F, float *t, hipStream_t st);
// q rotated, k rotated and written with v to their cache slots
void launch_linear_qkv(const StepMeta &m, const ModelDims &md, const KvGeom &g, int layer, const NormIn &nx, const void *wq, const void *wk,
                       const void *wv, const float2 *cs, float *q, void *kc, void *vc, hipStream_t st);
// logits as compact rows [rows][V], or (padded) in the caller's [batch][max_nodes][V] array
void launch_linear_logits(const StepMeta &m, int dtype, const NormIn &nx, const void *W, int V, int max_nodes, float *logits, bool padded, hipStream_t st);
// tree-masked attention of every (row, head) over cache slots [0, kv_len + n_nodes)
void launch_attention_generic(const StepMeta &m, const ModelDims &md, const KvGeom &g, int layer,
                              const float *q, const void *kcache, const void *vcache, float *out,
                              hipStream_t st);
// argmax[seq][node] = lowest index of the maximum of the row's logits.  The logits are
// either compact ([rows][V], padded_in = false) or padded ([batch][max_nodes][V]).
void launch_argmax(const StepMeta &m, const float *logits, bool padded_in, int max_nodes, int V,
                   int32_t *argmax, hipStream_t st);
// Draft-side read-out (Sec. IV-A, Sec. IV-C): top2[seq][node] = ids of the largest and second
// largest logit (value descending, id ascending; second = -1 if V == 1), prob[seq][node] = softmax
// probability of the first, argmax (optional) = the first id.  The logits are compact rows
// [rows][V], or (from_partials) split-k partial sums, times 1/rms of the row if nrm.ssq is set;
// they are also stored into logits_out ([batch][max_nodes][V], optional).  rec_v / rec_i: rows * top2_blocks(V) * 3 floats / 2 ints.
int top2_blocks(int V);
void launch_top2(const StepMeta &m, const float *src, bool from_partials, int n_splits, int ldp,
                 const RowNorm &nrm, int V, int max_nodes, float *logits_out, float *rec_v, int *rec_i, int32_t *top2,
                 float *prob, int32_t *argmax, hipStream_t st);

// ---- integer stages --------------------------------------------------------
// greedy acceptance, one wavefront per sequence; argmax in [batch][max_nodes] layout.  The results also go to `host`
// (pinned memory, as the device sees it), if given, so that no copy has to bring them there.
struct AcceptMirror {
  int32_t *argmax = nullptr, *path = nullptr, *accept_len = nullptr, *next_token = nullptr;
};
void launch_accept(const StepMeta &m, int max_nodes, const int32_t *argmax, int32_t *path,
                   int32_t *accept_len, int32_t *next_token, hipStream_t st, const AcceptMirror &host = AcceptMirror());
// the same from records (value, lowest id) of `pieces` parts of each row's vocabulary; also writes argmax
void launch_accept_records(const StepMeta &m, int max_nodes, const float2 *rec, int pieces, int32_t *argmax, int32_t *path,
                           int32_t *accept_len, int32_t *next_token, hipStream_t st, const AcceptMirror &host = AcceptMirror());
// argmax of the caller's padded logits ([batch][max_nodes][V]), then the acceptance above.  rec: rows *
// argmax_pieces(V) pairs of floats.
int argmax_pieces(int V);
void launch_argmax_accept(const StepMeta &m, const float *logits, int max_nodes, int V, float *rec, int32_t *argmax,
                          int32_t *path, int32_t *accept_len, int32_t *next_token, hipStream_t st);
// in-place compaction of the accepted path's cache rows (path/accept_len on the device)
void launch_compact(int dtype, const KvGeom &g, int batch, int max_nodes, const int32_t *kv_len,
                    const int32_t *path, const int32_t *accept_len, void *kcache, void *vcache,
                    hipStream_t st);

}  // namespace specasr
