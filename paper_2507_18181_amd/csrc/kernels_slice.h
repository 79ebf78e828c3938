// Unsplit skinny GEMMs with finishing epilogues (kernels_slice.hip).
#pragma once
#include "kernels_mfma.h"

namespace specasr {

// What the workgroup does with its finished output.
enum SliceEpi {
  kSlicePartial = 0,  // store it as split-k partial sums (S may be > 1)
  kSliceSwiglu = 1,   // gate|up: planes of silu(gate) * up
  kSliceQkv = 2,      // q|k|v: rotary embedding, query planes, K and V rows into the cache
  kSliceResid = 3,    // o: residual update, planes of x * gain, sums of squares per 16 columns
};

struct SliceArgs {
  const void *W;      // packed weights (PackedMatrix::data)
  const uint16_t *X;  // packed activation planes, hi then lo
  int rows, n_half, ksteps, S;
  int total, per_xcd; // workgroups, and workgroups per XCD (set by the launcher)
  float *part;        // kSlicePartial
  RowNorm nrm;        // kSliceSwiglu, kSliceQkv: statistics of the input rows
  uint16_t *t, *t_lo; // kSliceSwiglu, kSliceResid: output planes
  // kSliceResid
  float *x;
  const uint16_t *gain;
  int d, n_slab_out;
  float *ssq_out;
  // kSliceQkv
  StepMeta m;
  KvGeom g;
  int layer, H, Hkv, hd, hd_shift, col_k, col_v;
  const float2 *cs;
  uint16_t *qb, *qb_lo, *kc, *vc;
  float qscale;
};

struct SlicePlan {
  int hb = 0;  // half-bands per workgroup; 0: this projection takes the split kernel
  int nc = 1;  // groups of 16 rows
  int S = 1;
};

// Row groups of the instance that is launched for a plan's nc: 0 stands for 8 rows with both planes in one operand.
inline int slice_groups_launched(int nc, int rows) { return nc == 1 && rows <= 8 ? 0 : nc; }
bool slice_shape_built(int epi, int hb, int nc);
hipError_t gemm_slice_set_lds_limit();
// false (nothing launched) if the plan's shape is not built
bool launch_gemm_slice(int epi, const SliceArgs &a, const SlicePlan &pl, hipStream_t st, hipEvent_t ev0 = nullptr,
                       hipEvent_t ev1 = nullptr);

}  // namespace specasr
