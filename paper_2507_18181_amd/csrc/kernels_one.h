// All decoder layers of a small forward in one launch (kernels_one.hip).
#pragma once
#include "kernels.h"

namespace specasr {

// Weights of a layer as the kernel reads them; a table of them lives in device memory.
struct OneLayer {
  const void *qkv, *o, *gu, *down;  // packed
  const uint16_t *gain_ffn;         // norm in front of this layer's feed-forward part
  const uint16_t *gain_next;        // norm behind the layer: the next layer's, or the final one
};

// Bytes from the start of a layer's region, and its size.
struct OneLayout {
  uint32_t hb0, x0, s0;  // in front of the attention part: planes of x * gain, x, sums of squares
  uint32_t q, kt, vt;    // rotated queries (planes), this forward's own K and V rows
  uint32_t po, ml;       // attention outputs per key chunk, with their maxima and sums
  uint32_t att;          // attention output (planes)
  uint32_t hb1, x1, s1;  // in front of the feed-forward part
  uint32_t t;            // SwiGLU output (planes)
  uint32_t bytes;
};

// A forward of one sequence: rows, keys, and how the work is cut.
struct OnePlan {
  int rows = 0;                  // 0: not this kernel
  int rp = 0;                    // rows that the planes have room for: 1, 2, 4, 8 or 16
  int n_rg = 0;                  // groups of 32 query rows per KV head
  int n_chunks = 0, chunk_tiles = 0;  // key chunks, tiles of 32 prefix keys in each
  OneLayout lay;
};

struct OneArgs {
  const OneLayer *layers;
  int n_layers, d, dq, F, H, Hkv, col_k, col_v;
  int rows, rp, L, n_rg, n_chunks, chunk_tiles;
  int n_half_qkv, n_half_gu;
  int i_att, i_mrg, i_o, i_gu, i_dn, per_layer, total;  // first item of each phase of a layer; items of a layer, of the call
  float eps, qscale;
  const uint64_t *anc;
  const float2 *cs;
  uint16_t *kc, *vc;
  KvGeom g;
  char *ll;
  OneLayout lay;
  uint32_t *ctl;        // [0] next item, [1] set when a wait was given up
  uint32_t *gave_up;    // the same for the host (pinned)
  int polls;            // bound of a wait
  uint16_t *hb, *hb_lo; // after the last layer, as the LM head reads them
  float *ssq;
};

// Words in front of the regions: the counters that the first kernel of the call clears.
constexpr size_t kOneCtl = 256;
constexpr int kOnePolls = 1 << 21;  // looks of a wait at most: two to four seconds

bool one_launch_model(const ModelDims &md, int n_cu);
OnePlan plan_one_launch(const ModelDims &md, int rows, int kv_len);
size_t one_launch_bytes(const ModelDims &md);  // scratch of the largest plan
hipError_t one_launch_set_lds_limit();
void launch_one(OneArgs a, int n_cu, hipStream_t st);

}  // namespace specasr
