// Kernel launch interfaces shared by the API layer and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "treetrain.h"

namespace tt {

// Brackets one kernel launch with HIP events on its stream when kernel timing is enabled
// (tt_kernel_timing_enable); does nothing otherwise.
class KernelTimer {
 public:
  KernelTimer(int id, hipStream_t st);
  ~KernelTimer();
  KernelTimer(const KernelTimer&) = delete;
  KernelTimer& operator=(const KernelTimer&) = delete;
 private:
  int id_;
  hipStream_t st_;
  bool active_;
  hipEvent_t start_, stop_;
};

// Arguments of one attention call, after validation; strides are in elements.
struct RefArgs {
  int n_q, n_prefix, hq, hkv, d;
  float scale;
  int64_t q_stride, k_stride, v_stride;
  const void *q, *k_own, *v_own, *k_prefix, *v_prefix;
  const int32_t *kend, *kt_min, *kt_max;
  void* o;
  float* lse;
  // backward only
  const void* d_o;
  float* delta;                 // [hq][n_q] workspace: rowsum(dO o O); the MFMA path stores its negation here
  float* neg_lse2;              // [hq][n_q] MFMA path only: -lse * log2(e)
  void *dq, *dk_own, *dv_own;
  float *dk_prefix_acc, *dv_prefix_acc;
  void* workspace;              // remaining workspace after delta (MFMA path scratch)
  size_t workspace_bytes;
};
typedef RefArgs AttnArgs;

// fp32-arithmetic reference-grade kernels (tt_attn_ref.hip)
hipError_t ref_attn_fwd(const RefArgs& a, bool bf16, hipStream_t st);
hipError_t ref_attn_bwd(const RefArgs& a, bool bf16, hipStream_t st);

// fp32 kernels on the fp32 matrix instruction, d = 64 and 128 (tt_attn_f32.hip)
bool f32_attn_supported(const RefArgs& a);
hipError_t f32_attn_fwd(const RefArgs& a, hipStream_t st);
hipError_t f32_attn_bwd(const RefArgs& a, hipStream_t st);

// bf16 MFMA kernels, d = 128 (tt_attn_fwd.hip / tt_attn_bwd.hip)
hipError_t mfma_attn_fwd(const AttnArgs& a, hipStream_t st);
hipError_t mfma_attn_bwd(const AttnArgs& a, hipStream_t st);
bool attn_two_groups(const AttnArgs& a, int64_t blocks, int min_tiles);      // whether forward or dQ run two groups of waves
int attn_lg_heads(const AttnArgs& a);                                            // log2 of the query heads per workgroup of both
size_t mfma_attn_workspace(int n_q, int n_prefix, int hq, int hkv, int d, bool backward);
// dK/dV pass of the backward (tt_attn_dkdv.hip); a.workspace must hold mfma_attn_dkdv_workspace bytes and the plan that the dQ launch wrote there
hipError_t mfma_attn_dkdv(const AttnArgs& a, hipStream_t st);
size_t mfma_attn_dkdv_workspace(int n_q, int n_prefix, int hkv);

// fused log-softmax / gather / weighting (tt_loss.hip)
hipError_t weighted_logprob(int64_t n_rows, int vocab, bool bf16, const void* logits, int64_t row_stride,
                            const int32_t* target, const float* weight, float* logp, float* lse,
                            float* loss_acc, hipStream_t st);
hipError_t weighted_logprob_bwd(int64_t n_rows, int vocab, bool bf16, const void* logits, int64_t row_stride,
                                const int32_t* target, const float* weight, const float* lse, float grad_scale,
                                void* dlogits, int64_t out_stride, hipStream_t st);

// both in one pass over the logits; weighted_logprob_fused_ok tells whether the pointers and strides allow it (every row
// of the logits and of the gradient the same distance from a 16-byte boundary), the rows fit one launch and it is the faster way
bool weighted_logprob_fused_ok(int64_t n_rows, int vocab, bool bf16, const void* logits, int64_t row_stride, const void* dlogits,
                               int64_t out_stride);
hipError_t weighted_logprob_fused(int64_t n_rows, int vocab, bool bf16, const void* logits, int64_t row_stride,
                                  const int32_t* target, const float* weight, float grad_scale, float* logp, float* lse,
                                  float* loss_acc, void* dlogits, int64_t out_stride, hipStream_t st);

// rotary position embedding (tt_rope.hip); strides in elements
hipError_t rope(int64_t n_tokens, int n_heads, int d, bool bf16, const void* x, int64_t x_stride, const int32_t* pos,
                float theta_base, bool inverse, void* y, int64_t y_stride, hipStream_t st);

// tree-correct causal convolution (tt_conv.hip); strides in bytes
hipError_t conv_fwd(int64_t n_tokens, int channels, int kernel_size, bool bf16, bool silu, const void* x, int64_t x_stride_bytes,
                    const float* weight, const float* bias, const int32_t* tok_pred, void* y, int64_t y_stride_bytes,
                    hipStream_t st);
hipError_t conv_bwd(int64_t n_tokens, int channels, int kernel_size, bool bf16, bool silu, const void* x, int64_t x_stride_bytes,
                    const float* weight, const float* bias, const int32_t* tok_pred, const void* dy, int64_t dy_stride_bytes,
                    int n_fix, const int32_t* fix_tok, const int32_t* fix_off, const int32_t* fix_t, const int32_t* fix_r,
                    void* dx, int64_t dx_stride_bytes, float* dweight, float* dbias, void* workspace, hipStream_t st);
size_t conv_bwd_workspace(int64_t n_tokens, int channels, int kernel_size, bool bf16);

// gated delta rule with tree state routing, forward (tt_gdn.hip); dk = dv = 128, bf16
// `sched` (nullable): the segments of the chunk program by dependency level; see tt_gdn_schedule
hipError_t gdn_fwd(int64_t n_tokens, int hk, int hv, float scale, const void* q, const void* k, const void* v, const float* g,
                   const float* beta, int n_chunks, const int32_t* chunk_tok0, const int32_t* chunk_len, const int32_t* chunk_src,
                   const int32_t* chunk_dst, int n_slots, const int32_t* chunk_cap, const tt_gdn_schedule* sched,
                   const float* initial_state, float* state_out, void* o, void* workspace, hipStream_t st);
size_t gdn_workspace(int n_chunks, int n_slots, int hv);

// Backward of the gated delta rule.  Every per-chunk array is indexed by (head * n_chunks + chunk).
constexpr int GDN_REC_ELEMS = 19 * 512;      // bf16 elements of a chunk's record (tt_gdn.hip)
constexpr int GDN_REC_ROW = 12 * 512;        // its rows of 64 fp32 factors: beta, beta exp(gamma), exp(gamma_last - gamma), exp(gamma)
// What the walks leave for the finish kernel, rounded to bf16, as the 1 KB fragments their waves hold (four blocks of 32 value
// columns; lane = column, at position gdn_saved_lane):
struct GdnBwdSaved {
  void* rec;         // records
  float* gam;        // [64] running sum of the log-decays inside the chunk
  void* s0;          // [4][8][64][8]: state entering the chunk; fragment ks, half hf, element e = key dim 16 ks + 8 hf + e
  void* ds1;         // gradient of the state leaving the chunk, same layout
  void* vns;         // [4][4][64][8]: Vn; fragment js, half hf, element e = token 16 js + 4 hf + 8 (e / 4) + e % 4
  void* drs;         // dR, same layout
  // states and gradients of states, 128 x 128 floats each, in the order in which the walks' lanes hold them:
  float* slots;      // [n_slots][hv] saved node-end states
  float* slot_grad;  // [n_slots][hv] their gradients (zeroed by the caller); walk in sequence order only
  float* seg_grad;   // [n_segments][hv] gradient of the state every segment starts from; scheduled walk only
  void* sync;        // [n_slots + n_segments][value heads of the pass] of 16 bytes: what the walks synchronise with
};
// Position of a lane's 16 bytes in a saved fragment: the two halves of the wave lie 512 bytes apart, where the transposing reads of
// the finish kernel would meet in the same banks; the upper half is shifted by 64 bytes.
__host__ __device__ inline int gdn_saved_lane(int lane) { return lane ^ ((lane >> 5) << 2); }

// backward of the gated delta rule (tt_gdn_bwd.hip)
struct GdnBwdArgs {
  int64_t n_tokens;
  int hk, hv, n_chunks, n_slots;
  int hv_n;                          // value heads this pass works on (set by gdn_bwd: a batch of whole key-head groups;
                                     // the tensor pointers are moved to the batch's first head, hk / hv stay the strides)
  float scale;
  const void *q, *k, *v, *d_o;       // bf16
  const float *g, *beta;
  const int32_t *chunk_tok0, *chunk_len, *chunk_src, *chunk_dst, *chunk_cap;
  const tt_gdn_schedule* sched;      // nullptr: all chunks in one sequence
  const float* initial_state;        // nullptr or [hv][128][128]
  const float* d_state_out;          // nullptr or [n_capture][hv][128][128]: upstream gradient of the captured states
  void *dq, *dk, *dv;                // bf16
  float *dg, *dbeta;                 // [N][hv]
  float* d_initial_state;            // nullptr or [hv][128][128], overwritten
  void* workspace;
  size_t workspace_bytes;            // decides how many key-head groups one pass takes
};
// prepare kernel (backward form) + forward walk + reverse walk (tt_gdn.hip)
hipError_t gdn_bwd_prepare_and_walks(const GdnBwdArgs& b, const GdnBwdSaved& sv, hipStream_t st);
hipError_t gdn_bwd(const GdnBwdArgs& a, hipStream_t st);
// workspace for passes of key_heads_per_pass key heads (with their hv / hk value heads) at a time
size_t gdn_bwd_workspace(int64_t n_tokens, int n_chunks, int n_slots, int n_segments, int hk, int hv, int key_heads_per_pass);

}  // namespace tt
