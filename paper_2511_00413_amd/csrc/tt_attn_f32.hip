// Tree attention in fp32 on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32), head dims 64 and 128: products,
// sums, softmax and results in fp32 throughout (the paper verifies its gradients in float32, Appendix "Numerical
// Verification").  Other head dims take the kernels of tt_attn_ref.hip.
//
// Mask (Section "Attention Mask"): key j is visible to query i  <=>  j <= i + P < kend[j].
//
// A workgroup of 8 waves takes 16 queries of a head (forward, dQ) or 16 keys of a kv head (dK / dV); the waves go
// through the 16-wide blocks of the other side in turn, each with its own running softmax or gradients, and are
// combined in a fixed order at the end.  The work is small (verification trees of some hundred tokens) and bound by
// latency, so the split is the finest that fills the matrix instruction: 240 tokens x 4 heads make 60 workgroups of two
// steps a wave instead of one wave per row with serial dot products, and the backward is one launch (dK / dV workgroups
// first, longest ranges first; they form the row terms <dO, O> themselves).  At large sizes the fp32 matrix rate bounds
// it.  Operands go from memory to registers: no two waves of a workgroup share a row.
// Forward + backward, worked tree of 240 tokens, 4 heads of 64: 27 us (the row kernels: 198 us);  agentic tree of
// 2048 tokens, 4 / 2 heads of 128: 0.28 ms (5.2 ms);  8192 tokens, 32 / 8 heads: 6.9 ms, 37 TFLOP/s (196 ms, 1.3).
//
// Layouts of the instruction (lane l: l16 = l % 16, g = l / 16): A [16 x 4] row l16, k = g;  B [4 x 16] k = g, column
// l16;  C [16 x 16] column l16, rows 4 g + r.  A contraction over the head dim takes d = 16 m + 4 g + e in step (m, e), so
// that a lane reads its row in 16-byte pieces.  A 16 x 16 result is the B operand of the following product as it stands
// (step r contracts the rows 4 g + r); that product's A operand reads row 4 g + r at d = 64 m + 4 l16 .. + 3, and its
// result's tile (m, e) holds d = 64 m + 16 g + 4 r + e.
#include <hip/hip_runtime.h>
#include "tt_kernels.h"
#include "tt_mfma.h"

namespace tt {
namespace {

constexpr int NW = 8;                // waves per workgroup
constexpr int BLK = 16;              // queries / keys per block

template <int D> using Rows = f32x4[D / 16];        // a lane's pieces of one row
template <int D> using Cols = f32x4[4][D / 64];     // a lane's pieces of the rows 4 g + r
template <int D> using Acc = f32x4[D / 16];         // tiles (m, e) at 4 m + e

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int D>
__device__ __forceinline__ void load_rows(const float* row, int g, Rows<D>& x) {
#pragma unroll
  for (int m = 0; m < D / 16; m++) x[m] = *(const f32x4*)(row + 16 * m + 4 * g);
}
// [16 rows of a] x [16 rows of b]^T
template <int D>
__device__ __forceinline__ f32x4 dot_rows(const Rows<D>& a, const Rows<D>& b) {
  f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int m = 0; m < D / 16; m++)
#pragma unroll
    for (int e = 0; e < 4; e++) c = mfma4(a[m][e], b[m][e], c);
  return c;
}
// acc[d][column] += sum over the 16 rows i of x[i][d] w[i][column];  row(i) is the address of row i (0 .. 15).  `vis` bit r:
// the pair (row 4 g + r, column l16) is visible.  A row that only some columns see adds nothing to the others even where
// it holds an infinity or NaN (0 times it is NaN): such a block is added element by element.
template <int D, class RowFn>
__device__ __forceinline__ void add_outer(const RowFn& row, const float (&w)[4], unsigned vis, Acc<D>& acc, int lane) {
  const int l16 = lane & 15, g = lane >> 4;
  Cols<D> x;
#pragma unroll
  for (int r = 0; r < 4; r++)
#pragma unroll
    for (int m = 0; m < D / 64; m++) x[r][m] = *(const f32x4*)(row(4 * g + r) + 64 * m + 4 * l16);
  if (__ballot(vis != 15u) != 0) {
    float t = 0.f;                                   // stays zero if everything is finite
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
      for (int m = 0; m < D / 64; m++)
#pragma unroll
        for (int e = 0; e < 4; e++) t = fmaf(x[r][m][e], 0.f, t);
    if (__ballot(!(t == 0.f)) != 0) {
#pragma unroll 1
      for (int i = 0; i < BLK; i++) {
        const int src = (i >> 2) * 16 + l16;
        const float wi = __shfl(i & 2 ? (i & 1 ? w[3] : w[2]) : (i & 1 ? w[1] : w[0]), src);
        if (!(((unsigned)__shfl((int)vis, src) >> (i & 3)) & 1u)) continue;
        const float* p = row(i);
#pragma unroll
        for (int m = 0; m < D / 64; m++)
#pragma unroll
          for (int e = 0; e < 4; e++)
#pragma unroll
            for (int r = 0; r < 4; r++) acc[4 * m + e][r] = fmaf(wi, p[64 * m + 16 * g + 4 * r + e], acc[4 * m + e][r]);
      }
      return;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; r++)
#pragma unroll
    for (int m = 0; m < D / 64; m++)
#pragma unroll
      for (int e = 0; e < 4; e++) acc[4 * m + e] = mfma4(x[r][m][e], w[r], acc[4 * m + e]);
}
// value of the four lanes that share l16, combined
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}
// wave 0's acc = sum over the waves, in a fixed order
template <int N>
__device__ __forceinline__ void sum_waves(f32x4* lds, f32x4 (&acc)[N], int w, int lane) {
#pragma unroll
  for (int step = NW / 2; step > 0; step >>= 1) {
    if (w >= step && w < 2 * step)
#pragma unroll
      for (int i = 0; i < N; i++) lds[((w - step) * N + i) * 64 + lane] = acc[i];
    __syncthreads();
    if (w < step)
#pragma unroll
      for (int i = 0; i < N; i++) acc[i] += lds[(w * N + i) * 64 + lane];
    __syncthreads();
  }
}
template <int D>
__device__ __forceinline__ void store_row(float* p, const Acc<D>& acc, float f, int g) {
#pragma unroll
  for (int m = 0; m < D / 64; m++)
#pragma unroll
    for (int r = 0; r < 4; r++)
      *(f32x4*)(p + 64 * m + 16 * g + 4 * r) = f32x4{f * acc[4 * m][r], f * acc[4 * m + 1][r], f * acc[4 * m + 2][r], f * acc[4 * m + 3][r]};
}

__device__ __forceinline__ const float* key_row(const void* own, const void* prefix, int64_t own_stride, int hkv, int d, int P, int j, int kvh) {
  return j < P ? (const float*)prefix + ((int64_t)j * hkv + kvh) * d : (const float*)own + (int64_t)(j - P) * own_stride + (int64_t)kvh * d;
}

// Calls block(j0) for every 16-key block that holds a key some query of [gi_first, gi_last] sees and that belongs to wave w
// (the blocks are dealt out in turn; four of a wave's blocks are looked at with one load).
template <class F>
__device__ __forceinline__ void for_key_blocks(const RefArgs& a, int gi_first, int gi_last, int w, int lane, const F& block) {
  for (int b0 = w; b0 * BLK <= gi_last; b0 += 4 * NW) {
    const int j = (b0 + (lane >> 4) * NW) * BLK + (lane & 15);
    const uint64_t any = __ballot(j <= gi_last && a.kend[min(j, gi_last)] > gi_first);
#pragma unroll 1
    for (int t = 0; t < 4; t++)
      if ((any >> (16 * t)) & 0xffff) block((b0 + t * NW) * BLK);
  }
}
// visibility of the keys j0 + 4 g + r to the query gi
__device__ __forceinline__ unsigned key_bits(const RefArgs& a, int j0, int g, int gi) {
  unsigned vis = 0;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int j = j0 + 4 * g + r;
    vis |= (j <= gi && gi < a.kend[min(j, gi)] ? 1u : 0u) << r;
  }
  return vis;
}

template <int D>
__global__ void __launch_bounds__(64 * NW, 2) f32_fwd_kernel(RefArgs a, int n_qt) {
  __shared__ f32x4 lds[NW / 2 * (D / 16) * 64];
  __shared__ float m_s[NW][BLK], l_s[NW][BLK];
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = blockIdx.x % a.hq, qt = n_qt - 1 - blockIdx.x / a.hq, kvh = h / (a.hq / a.hkv);      // longest rows first
  const int P = a.n_prefix, n_k = P + a.n_q;
  const int qi = min(qt * BLK + l16, a.n_q - 1), gi = P + qi;           // rows past the last one repeat it and are not stored
  Rows<D> q;
  load_rows<D>((const float*)a.q + (int64_t)qi * a.q_stride + (int64_t)h * D, g, q);
  Acc<D> o;
#pragma unroll
  for (int i = 0; i < D / 16; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;                                         // l: this lane's keys
  for_key_blocks(a, P + qt * BLK, P + min(qt * BLK + BLK, a.n_q) - 1, w, lane, [&](int j0) {
    Rows<D> k;
    load_rows<D>(key_row(a.k_own, a.k_prefix, a.k_stride, a.hkv, D, P, min(j0 + l16, n_k - 1), kvh), g, k);
    const unsigned vis = key_bits(a, j0, g, gi);
    const f32x4 s = dot_rows<D>(k, q);
    float sv[4], p[4], top = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      sv[r] = vis >> r & 1 ? a.scale * s[r] : -INFINITY;
      top = fmaxf(top, sv[r]);
    }
    const float m_new = fmaxf(m, group_max(top)), ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m - ref);
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      p[r] = vis >> r & 1 ? expf(sv[r] - ref) : 0.f;
      l += p[r];
    }
    m = m_new;
#pragma unroll
    for (int i = 0; i < D / 16; i++) o[i] *= alpha;
    add_outer<D>([&](int i) { return key_row(a.v_own, a.v_prefix, a.v_stride, a.hkv, D, P, min(j0 + i, n_k - 1), kvh); }, p, vis, o, lane);
  });
  l = group_sum(l);
  if (g == 0) { m_s[w][l16] = m; l_s[w][l16] = l; }
  __syncthreads();
  float top = -INFINITY, total = 0.f;
#pragma unroll
  for (int v = 0; v < NW; v++) top = fmaxf(top, m_s[v][l16]);
  // (a wave without a reference has a sum of zero if it saw no key, and of NaN if every score it saw was NaN, which the
  // maximum passes over)
#pragma unroll
  for (int v = 0; v < NW; v++) total += m_s[v][l16] == -INFINITY ? l_s[v][l16] : l_s[v][l16] * expf(m_s[v][l16] - top);
  const float f = m == -INFINITY ? 0.f : expf(m - top);
#pragma unroll
  for (int i = 0; i < D / 16; i++) o[i] *= f;
  sum_waves<D / 16>(lds, o, w, lane);
  if (w == 0 && qt * BLK + l16 < a.n_q) {
#pragma unroll
    for (int i = 0; i < D / 16; i++) o[i] /= total;
    store_row<D>((float*)a.o + ((int64_t)qi * a.hq + h) * D, o, 1.f, g);
    // (every score -inf: no distribution, NaN like the row)
    if (g == 0) a.lse[(int64_t)h * a.n_q + qi] = top == -INFINITY ? NAN : top + logf(total);
  }
}

// <dO, O> of the row whose pieces of dO a lane group holds
template <int D>
__device__ __forceinline__ float row_delta(const Rows<D>& d_o, const float* o_row, int g) {
  Rows<D> o;
  load_rows<D>(o_row, g, o);
  float s = 0.f;
#pragma unroll
  for (int m = 0; m < D / 16; m++)
#pragma unroll
    for (int e = 0; e < 4; e++) s = fmaf(d_o[m][e], o[m][e], s);
  return group_sum(s);
}

template <int D>
__device__ __forceinline__ void dq_tile(const RefArgs& a, f32x4* lds, int h, int qt, int w, int lane) {
  const int l16 = lane & 15, g = lane >> 4, kvh = h / (a.hq / a.hkv);
  const int P = a.n_prefix, n_k = P + a.n_q;
  const int qi = min(qt * BLK + l16, a.n_q - 1), gi = P + qi;
  const int64_t orow = ((int64_t)qi * a.hq + h) * D;
  Rows<D> q, d_o;
  load_rows<D>((const float*)a.q + (int64_t)qi * a.q_stride + (int64_t)h * D, g, q);
  load_rows<D>((const float*)a.d_o + orow, g, d_o);
  const float delta = row_delta<D>(d_o, (const float*)a.o + orow, g);
  const float lse = a.lse[(int64_t)h * a.n_q + qi];
  Acc<D> dq;
#pragma unroll
  for (int i = 0; i < D / 16; i++) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for_key_blocks(a, P + qt * BLK, P + min(qt * BLK + BLK, a.n_q) - 1, w, lane, [&](int j0) {
    Rows<D> k, v;
    const int j = min(j0 + l16, n_k - 1);
    load_rows<D>(key_row(a.k_own, a.k_prefix, a.k_stride, a.hkv, D, P, j, kvh), g, k);
    load_rows<D>(key_row(a.v_own, a.v_prefix, a.v_stride, a.hkv, D, P, j, kvh), g, v);
    const unsigned vis = key_bits(a, j0, g, gi);
    const f32x4 s = dot_rows<D>(k, q), dp = dot_rows<D>(v, d_o);
    float ds[4];
#pragma unroll
    for (int r = 0; r < 4; r++) ds[r] = vis >> r & 1 ? expf(a.scale * s[r] - lse) * (dp[r] - delta) : 0.f;
    add_outer<D>([&](int i) { return key_row(a.k_own, a.k_prefix, a.k_stride, a.hkv, D, P, min(j0 + i, n_k - 1), kvh); }, ds, vis, dq, lane);
  });
  sum_waves<D / 16>(lds, dq, w, lane);
  if (w == 0 && qt * BLK + l16 < a.n_q) store_row<D>((float*)a.dq + orow, dq, a.scale, g);
}

// The visible queries of key j form the contiguous range [max(j - P, 0), kend[j] - P).
template <int D>
__device__ __forceinline__ void dkv_tile(const RefArgs& a, f32x4* lds, int kvh, int jt, int w, int lane) {
  const int l16 = lane & 15, g = lane >> 4, G = a.hq / a.hkv;
  const int P = a.n_prefix, n_k = P + a.n_q, j = jt * BLK + l16, jc = min(j, n_k - 1);
  Rows<D> k, v;
  load_rows<D>(key_row(a.k_own, a.k_prefix, a.k_stride, a.hkv, D, P, jc, kvh), g, k);
  load_rows<D>(key_row(a.v_own, a.v_prefix, a.v_stride, a.hkv, D, P, jc, kvh), g, v);
  const int lo = max(j - P, 0), hi = j < n_k ? min(max(a.kend[jc], P) - P, a.n_q) : 0;       // (kend = INT32_MAX or 0 for prefix keys)
  int lo_t = max(jt * BLK - P, 0), hi_t = hi;
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) hi_t = max(hi_t, __shfl_xor(hi_t, d));
  hi_t = __builtin_amdgcn_readfirstlane(hi_t);
  const int n_blk = hi_t > lo_t ? (hi_t - lo_t + BLK - 1) / BLK : 0;
  f32x4 dkv[2 * (D / 16)];
  Acc<D>&dk = *(Acc<D>*)dkv, &dv = *(Acc<D>*)(dkv + D / 16);
#pragma unroll
  for (int i = 0; i < 2 * (D / 16); i++) dkv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int it = w; it < n_blk * G; it += NW) {
    const int h = kvh * G + it / n_blk, i0 = lo_t + it % n_blk * BLK;
    unsigned vis = 0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = i0 + 4 * g + r;
      vis |= (i >= lo && i < hi ? 1u : 0u) << r;
    }
    if (__ballot(vis != 0) == 0) continue;
    auto q_row = [&](int i) { return (const float*)a.q + (int64_t)min(i0 + i, a.n_q - 1) * a.q_stride + (int64_t)h * D; };
    auto o_off = [&](int i) { return ((int64_t)min(i0 + i, a.n_q - 1) * a.hq + h) * D; };
    Rows<D> q, d_o;
    load_rows<D>(q_row(l16), g, q);
    load_rows<D>((const float*)a.d_o + o_off(l16), g, d_o);
    float lse[4];
#pragma unroll
    for (int r = 0; r < 4; r++) lse[r] = a.lse[(int64_t)h * a.n_q + min(i0 + 4 * g + r, a.n_q - 1)];
    const float delta = row_delta<D>(d_o, (const float*)a.o + o_off(l16), g);
    const f32x4 s = dot_rows<D>(q, k), dp = dot_rows<D>(d_o, v);
    float p[4], ds[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const float dr = __shfl(delta, 4 * g + r);
      p[r] = vis >> r & 1 ? expf(a.scale * s[r] - lse[r]) : 0.f;
      ds[r] = vis >> r & 1 ? p[r] * (dp[r] - dr) : 0.f;
    }
    add_outer<D>([&](int i) { return (const float*)a.d_o + o_off(i); }, p, vis, dv, lane);
    add_outer<D>(q_row, ds, vis, dk, lane);
  }
  sum_waves<2 * (D / 16)>(lds, dkv, w, lane);
  if (w != 0 || j >= n_k) return;
  if (j >= P) {
    store_row<D>((float*)a.dk_own + ((int64_t)(j - P) * a.hkv + kvh) * D, dk, a.scale, g);
    store_row<D>((float*)a.dv_own + ((int64_t)(j - P) * a.hkv + kvh) * D, dv, 1.f, g);
  } else if (hi > lo) {
    float* kp = a.dk_prefix_acc + ((int64_t)j * a.hkv + kvh) * D;
    float* vp = a.dv_prefix_acc + ((int64_t)j * a.hkv + kvh) * D;
#pragma unroll
    for (int m = 0; m < D / 64; m++)
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int at = 64 * m + 16 * g + 4 * r + e;
          kp[at] += a.scale * dk[4 * m + e][r];
          vp[at] += dv[4 * m + e][r];
        }
  }
}

template <int D>
__global__ void __launch_bounds__(64 * NW, 2) f32_bwd_kernel(RefArgs a, int n_qt, unsigned n_dkv) {
  __shared__ f32x4 lds[NW / 2 * 2 * (D / 16) * 64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x < n_dkv) {
    dkv_tile<D>(a, lds, blockIdx.x % a.hkv, blockIdx.x / a.hkv, w, lane);
  } else {
    const unsigned b = blockIdx.x - n_dkv;
    dq_tile<D>(a, lds, b % a.hq, n_qt - 1 - b / a.hq, w, lane);
  }
}

}  // namespace

// Workgroups of a launch.  All of them lie along one grid dimension, and a dimension of a launch holds less than 2^32
// work-items: calls beyond that (more than 8388607 workgroups) stay with the row kernels, whose grids are two-dimensional.
static constexpr int64_t f32_workgroups(int64_t n_keys, int64_t heads) { return (n_keys + BLK - 1) / BLK * heads; }
static constexpr bool f32_grid_fits(int64_t n_keys, int64_t heads) { return f32_workgroups(n_keys, heads) * 64 * NW < (int64_t)1 << 32; }
static_assert(f32_grid_fits(8388607 * (int64_t)BLK, 1) && !f32_grid_fits(8388607 * (int64_t)BLK + 1, 1), "work-items of a launch");
static_assert(!f32_grid_fits(1 << 20, 128) && f32_grid_fits(1 << 20, 127), "work-items of a launch");

bool f32_attn_supported(const RefArgs& a) {
  return (a.d == 64 || a.d == 128) && f32_grid_fits((int64_t)a.n_prefix + a.n_q, (int64_t)a.hq + a.hkv);
}

hipError_t f32_attn_fwd(const RefArgs& a, hipStream_t st) {
  if (a.n_q == 0) return hipSuccess;
  const int n_qt = (a.n_q + BLK - 1) / BLK;
  KernelTimer timer(TT_KERNEL_REF_FWD, st);
  if (a.d == 64) f32_fwd_kernel<64><<<(unsigned)n_qt * a.hq, 64 * NW, 0, st>>>(a, n_qt);
  else f32_fwd_kernel<128><<<(unsigned)n_qt * a.hq, 64 * NW, 0, st>>>(a, n_qt);
  return hipGetLastError();
}

hipError_t f32_attn_bwd(const RefArgs& a, hipStream_t st) {
  if (a.n_q == 0) return hipSuccess;
  const int n_qt = (a.n_q + BLK - 1) / BLK;
  const unsigned n_dkv = (unsigned)((a.n_prefix + a.n_q + BLK - 1) / BLK) * a.hkv, blocks = n_dkv + (unsigned)n_qt * a.hq;
  KernelTimer timer(TT_KERNEL_REF_BWD, st);
  if (a.d == 64) f32_bwd_kernel<64><<<blocks, 64 * NW, 0, st>>>(a, n_qt, n_dkv);
  else f32_bwd_kernel<128><<<blocks, 64 * NW, 0, st>>>(a, n_qt, n_dkv);
  return hipGetLastError();
}

}  // namespace tt
