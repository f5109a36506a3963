// The attention by per-query projected vectors (attn_proj.hip): sizes, buffers and entry points.
//
// A head's score is q_h . (W_k,h x_j) / sqrt(dh) = (W_k,h^T q_h) . x_j / sqrt(dh), plus a share of b_k
// that is the same for all of a query's slots and leaves the softmax; its weighted sum of values is
// W_v,h (sum_j p_j x_j) + b_v,h.  So the key/value weights meet one row per query and head instead of
// one per neighbour slot, and a slot costs two dot-length passes over its input row
// x_j = [M[n_j] || x[e_j] || phi(tau - t_j)].
#pragma once

#include "ops.h"

namespace mtgnn {

// Widths inside: heads are padded to dhp = 4 ceil(dh / 4) columns (dap = H dhp), the edge features to
// dep = 4 ceil(de / 4), so a slot's row is [dm | dep | dt] (kvp columns), every group of four aligned.
struct ProjShape {
  int64_t Q, P, N;
  int dm, dt, de, dep, da, H, dh, dhp, dap, k, kvp, Dq, Dkv;
  int us, uu, as;   // LDS row strides (multiples of 4, odd in 16-byte groups): a row of H kvp (or da + dm), of
                    // H (dm + dt), of dap
  int esz;      // bytes of a stored slot-row element
  ProjShape(const mtgnn_dims* d, int64_t max_q);
};

// Whether these dims take this path (the general path of attention.hip covers the rest).
bool proj_ok(const mtgnn_dims* d);

// Packed weights (MFMA fragment order), then the arrays the backward reads.
struct ProjSave {
  float *w[13];   // see ProjPack
  float* qc;      // [dap] the query projection's constant b_q + W_q[:, dm:] phi(0)
  float *qv, *c, *p, *attn, *m_in, *a1;
  void* xs;       // [Q k, dm + dep] the slots' memory and edge columns as stored (float32 or bfloat16)
  size_t total;
};
enum ProjPack { PK_WQ, PK_WKT, PK_WV, PK_WO, PK_W1, PK_W2, PK_W2T, PK_W1OT, PK_W1HT, PK_WOT, PK_WVT, PK_WK, PK_WQT };
ProjSave carve_proj_save(void* base, const ProjShape& s);

struct ProjBwd {   // the backward's workspace regions
  float *dz, *dm1, *dout, *dattn, *dqv, *du, *dhq, *dx, *tg, *tg2;
  char* dw;
  size_t dw_bytes, total;
};
ProjBwd carve_proj_bwd(void* base, const ProjShape& s);

mtgnn_status proj_prepare_weights(const mtgnn_attn_params* p, const float* tw, const float* tb, const mtgnn_dims* d,
                                  void* save, hipStream_t s, const PadCopy* more, int n_more);
mtgnn_status proj_fwd(const int32_t* q_node, const float* q_t, const int32_t* n_q, int64_t max_q, const int32_t* nbr,
                      const float* nt, const int32_t* neid, const void* memory, const float* edge_feat,
                      const float* tw, const float* tb, const mtgnn_attn_params* p, const mtgnn_dims* d, float* z,
                      void* save, hipStream_t s);
// Data gradients: everything the weight gradients and the d M' sums read, and the time encoder's partials.
mtgnn_status proj_bwd(const float* q_t, const int32_t* n_q, int64_t max_q, const int32_t* nbr, const float* nt,
                      const float* dz, const float* tw, const float* tb, const mtgnn_dims* d, const void* save,
                      const ProjBwd& b, hipStream_t s);
// Weight and time-encoder gradients from proj_bwd's outputs.
mtgnn_status proj_params(const int32_t* n_q, int64_t max_q, const float* dz, const float* tw, const float* tb,
                         const mtgnn_attn_params* p, const mtgnn_dims* d, const void* save, const ProjBwd& b,
                         mtgnn_attn_grads* g, float* d_time_w, float* d_time_b, hipStream_t s);

}  // namespace mtgnn
