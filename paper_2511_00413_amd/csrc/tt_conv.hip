// Tree-correct depthwise causal convolution (Section "Implementation", paragraph "SSM Layers (GDN)",
// item (ii); Appendix "Tree-Correct Causal Convolution"): every token's window holds the K-1 tokens
// that precede it on its own root-to-token sequence, found through tok_pred, not the K-1 tokens that
// precede it in DFS order.  HBM-bound: one lane owns four channels and walks a tile of
// consecutive tokens with the window in registers; the window is rebuilt from the predecessor chain
// only where the sequence jumps (first token of a node that does not directly follow its parent's
// last token) and at the start of a tile.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>
#include "tt_internal.h"
#include "tt_kernels.h"

namespace tt {
namespace {

constexpr int CONV_THREADS = 256;
constexpr int CONV_BWD_TILE = 256;       // (512 measured the same)
constexpr int CONV_SUM_RUN = 24;         // tokens; a multiple of two batches of every kernel size (48 and 96 take the same time)
constexpr int conv_bwd_wgs(bool bf16) { return bf16 ? 3 : 2; }      // workgroups of the backward walk per compute unit (registers)

// Channels per lane: four of either type, so 8 bytes of bf16 or 16 of fp32 per access.  The walks are bound by HBM and the
// arithmetic together (sigmoid, K taps twice over and the weight sums per element), and what hides one under the
// other is waves: with eight bf16 channels per lane the forward took 133 registers and the backward 247 (3 and 2 waves per
// SIMD), with four 90 and 162 (5 and 3).  16406 tokens x 8192 channels, K = 4: forward 106 -> 97 us (5.5 TB/s), backward walk
// 181 -> 170 us (4.7 TB/s).
typedef unsigned int u32x4c __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2c __attribute__((ext_vector_type(2)));
template <bool BF16> struct Chan { static constexpr int NV = 4; using Raw = u32x4c; };
template <> struct Chan<true> { static constexpr int NV = 4; using Raw = u32x2c; };

// one channel vector of a row, as loaded; STREAM: a non-temporal access, for rows that this kernel touches once
template <bool BF16, bool STREAM = false>
__device__ __forceinline__ typename Chan<BF16>::Raw load_raw(const void* base, int64_t row, int64_t stride_bytes, int cv) {
  using Raw = typename Chan<BF16>::Raw;
  const Raw* p = (const Raw*)((const char*)base + row * stride_bytes) + cv;
  return STREAM ? __builtin_nontemporal_load(p) : *p;
}
template <bool BF16>
__device__ __forceinline__ void unpack_raw(const typename Chan<BF16>::Raw& u, float (&v)[Chan<BF16>::NV]) {
  if constexpr (BF16) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      v[2 * i] = __uint_as_float(u[i] << 16);
      v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; i++) v[i] = __uint_as_float(u[i]);
  }
}
template <bool BF16>
__device__ __forceinline__ void load_row(const void* base, int64_t row, int64_t stride_bytes, int cv, float (&v)[Chan<BF16>::NV]) {
  unpack_raw<BF16>(load_raw<BF16>(base, row, stride_bytes, cv), v);
}

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));

template <bool BF16, bool STREAM = false>
__device__ __forceinline__ void store_row(void* base, int64_t row, int64_t stride_bytes, int cv, const float (&v)[Chan<BF16>::NV]) {
  using Raw = typename Chan<BF16>::Raw;
  Raw* p = (Raw*)((char*)base + row * stride_bytes) + cv;
  f32x4v f;
#pragma unroll
  for (int i = 0; i < 4; i++) f[i] = v[i];
  Raw out;
  if constexpr (BF16) out = __builtin_bit_cast(Raw, __builtin_convertvector(f, bf16x4v));       // round to nearest even
  else out = __builtin_bit_cast(Raw, f);
  if (STREAM) __builtin_nontemporal_store(out, p);
  else *p = out;
}

struct ConvArgs {
  int n_tokens, channels, tok_tile, n_tiles;
  int silu;
  const void* x; int64_t x_stride;       // strides in bytes
  const float* weight;                   // [C][K]
  const float* bias;                     // [C] or nullptr
  const int32_t* tok_pred;
  void* y; int64_t y_stride;             // forward output / backward: dx
  const void* dy; int64_t dy_stride;
  float* partial;                        // [n_tiles][K+1][C]: per-tile dweight (K rows) and dbias
  int n_fix;
  const int32_t *fix_tok, *fix_off, *fix_t, *fix_r;
};

// sigmoid through the bare exp2 / reciprocal instructions (1 ulp each; the results are rounded to
// bf16 or meet fp32 sums of comparable error)
__device__ __forceinline__ float sigmoid_f(float z) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * z));
}
__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_f(z); }
__device__ __forceinline__ float dsilu_f(float z) {
  const float s = sigmoid_f(z);
  return s * (1.f + z * (1.f - s));
}

template <bool BF16, int K>
struct Weights {
  static constexpr int NV = Chan<BF16>::NV;
  float w[K][NV], b[NV];
  __device__ __forceinline__ void load(const ConvArgs& a, int c0) {
#pragma unroll
    for (int i = 0; i < NV; i++) {
#pragma unroll
      for (int j = 0; j < K; j++) w[j][i] = a.weight[(int64_t)(c0 + i) * K + j];
      b[i] = a.bias ? a.bias[c0 + i] : 0.f;
    }
  }
};

// win[m-1] = x[pred^m(t)] for m = 1..K-1, zero past the start of the branch
template <bool BF16, int K>
__device__ __forceinline__ void rebuild_window(const ConvArgs& a, int pred, int cv, float (&win)[K > 1 ? K - 1 : 1][Chan<BF16>::NV]) {
  constexpr int NV = Chan<BF16>::NV;
  int q = pred;
#pragma unroll
  for (int m = 1; m < K; m++) {
    if (q >= 0) {
      load_row<BF16>(a.x, q, a.x_stride, cv, win[m - 1]);
      q = a.tok_pred[q];
    } else {
#pragma unroll
      for (int i = 0; i < NV; i++) win[m - 1][i] = 0.f;
    }
  }
}

// Tokens whose loads are issued together.  A multiple of K: the kernels keep the last K inputs (and, backward,
// the last K gradients) in rings of K register slots, token t0 + i in slot i % K, and with batches that are
// multiples of K every slot index is a compile-time constant after unrolling -- the rings never move.
template <int K> struct ConvBatch { static constexpr int U = K == 3 ? 3 : 4; };

// ring slot m places before slot `slot`
template <int K> __device__ __forceinline__ constexpr int ring_back(int slot, int m) { return (slot - m + 2 * K) % K; }

// xr[ring_back(slot, m)] = x[pred^m(t)] for m = 1..K-1, zero past the start of the branch
template <bool BF16, int K>
__device__ __forceinline__ void rebuild_ring(const ConvArgs& a, int pred, int cv, int slot, float (&xr)[K][Chan<BF16>::NV]) {
  constexpr int NV = Chan<BF16>::NV;
  int q = pred;
#pragma unroll
  for (int m = 1; m < K; m++) {
    if (q >= 0) {
      load_row<BF16>(a.x, q, a.x_stride, cv, xr[ring_back<K>(slot, m)]);
      q = a.tok_pred[q];
    } else {
#pragma unroll
      for (int i = 0; i < NV; i++) xr[ring_back<K>(slot, m)][i] = 0.f;
    }
  }
}

template <bool BF16, int K>
__global__ __launch_bounds__(CONV_THREADS) void tree_conv_fwd_kernel(ConvArgs a) {
  constexpr int NV = Chan<BF16>::NV;
  constexpr int U = ConvBatch<K>::U;
  // consecutive workgroups cover one token tile's channel vectors (a row is read in full by neighbours)
  const int64_t gid = (int64_t)blockIdx.x * CONV_THREADS + threadIdx.x;
  const int vpr = a.channels / NV;
  const int tile = (int)(gid / vpr);
  const int cv = (int)(gid - (int64_t)tile * vpr);
  if (tile >= a.n_tiles) return;
  Weights<BF16, K> wt;
  wt.load(a, cv * NV);
  float xr[K][NV];                                  // ring of the last K inputs
  const int t0 = (int)tile * a.tok_tile;
  const int t1 = min(t0 + a.tok_tile, a.n_tokens);
  // Two batches of U tokens are in flight: the loads of the next batch are issued before the current one is
  // worked on, so the memory round trip of a batch runs under the arithmetic of the one before.
  struct Batch { int p[U]; typename Chan<BF16>::Raw x[U]; };
  auto load_batch = [&](int tb, Batch& b) {
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int t = min(tb + u, t1 - 1);
      b.p[u] = a.tok_pred[t];
      b.x[u] = load_raw<BF16, true>(a.x, t, a.x_stride, cv);
    }
  };
  auto work_batch = [&](int tb, const Batch& b) {       // (tb - t0) is a multiple of U, hence of K
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int t = tb + u;
      const int slot = u % K;
      if (t < t1) {
        unpack_raw<BF16>(b.x[u], xr[slot]);
        if (t == t0 || b.p[u] != t - 1) rebuild_ring<BF16, K>(a, b.p[u], cv, slot, xr);
        float pre[NV];
#pragma unroll
        for (int i = 0; i < NV; i++) {
          float acc = wt.b[i] + wt.w[K - 1][i] * xr[slot][i];
#pragma unroll
          for (int m = 1; m < K; m++) acc += wt.w[K - 1 - m][i] * xr[ring_back<K>(slot, m)][i];
          pre[i] = a.silu ? silu_f(acc) : acc;
        }
        store_row<BF16>(a.y, t, a.y_stride, cv, pre);
      }
    }
  };
  Batch ba, bb;
  load_batch(t0, ba);
  for (int tb = t0; tb < t1; tb += 2 * U) {
    load_batch(tb + U, bb);
    work_batch(tb, ba);
    load_batch(tb + 2 * U, ba);
    work_batch(tb + U, bb);
  }
}

// Backward, fast path.  Walks the tile plus K-1 tokens of look-ahead; g of the last K tokens and
// their "directly follows its predecessor" flags stay in registers.  dx[s] takes the successors
// s+1 .. s+K-1 for as long as each directly follows the one before (successors that sit elsewhere
// in DFS order -- later children of a branch point -- are added by the fix-up kernel, which
// recomputes those few dx rows completely).  dweight / dbias partial sums per tile go to `partial`.
template <bool BF16, int K>
__global__ __launch_bounds__(CONV_THREADS, conv_bwd_wgs(BF16)) void tree_conv_bwd_kernel(ConvArgs a) {
  constexpr int NV = Chan<BF16>::NV;
  constexpr int U = ConvBatch<K>::U;
  const int64_t gid = (int64_t)blockIdx.x * CONV_THREADS + threadIdx.x;
  const int vpr = a.channels / NV;
  const int tile = (int)(gid / vpr);
  const int cv = (int)(gid - (int64_t)tile * vpr);
  if (tile >= a.n_tiles) return;
  Weights<BF16, K> wt;
  wt.load(a, cv * NV);
  // rings of K slots, token t0 + i in slot i % K: inputs, g = dy * act'(pre), and the "directly follows its
  // predecessor" flags
  float xr[K][NV], gq[K][NV];
  bool lk[K];
  // dweight, dbias: the running sums of at most CONV_SUM_RUN tokens, and the sum of the runs that are complete.  A tile is longer
  // than a single fp32 chain of additions should be: dweight of 16406 x 8192, K = 4, is 2.6e-7 from the exact one (bf16; fp32
  // 3.1e-7) with one chain per tile, 1.7e-7 with runs of 48, 1.5e-7 with 24 (both types), all three at 280 us (bf16, both
  // directions); at 300 - 2500 tokens 1.35 - 1.49e-7 with 48 and 1.19 - 1.39e-7 with 24
  float dw[K][NV], db[NV], dw_runs[K][NV], db_runs[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) {
    db[i] = db_runs[i] = 0.f;
#pragma unroll
    for (int j = 0; j < K; j++) { dw[j][i] = dw_runs[j][i] = 0.f; gq[j][i] = 0.f; xr[j][i] = 0.f; }
  }
  auto end_run = [&]() {
#pragma unroll
    for (int i = 0; i < NV; i++) {
      db_runs[i] += db[i];
      db[i] = 0.f;
#pragma unroll
      for (int j = 0; j < K; j++) { dw_runs[j][i] += dw[j][i]; dw[j][i] = 0.f; }
    }
  };
#pragma unroll
  for (int j = 0; j < K; j++) lk[j] = false;
  const int t0 = (int)tile * a.tok_tile;
  const int t1 = min(t0 + a.tok_tile, a.n_tokens);
  const int t_end = t1 + K - 1;                     // look-ahead: g of the K-1 tokens after the tile
  // two batches of U tokens in flight, as in the forward
  struct Batch { int p[U]; typename Chan<BF16>::Raw x[U], dy[U]; };
  auto load_batch = [&](int tb, Batch& b) {
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int t = min(tb + u, a.n_tokens - 1);
      b.p[u] = a.tok_pred[t];
      b.x[u] = load_raw<BF16, true>(a.x, t, a.x_stride, cv);
      b.dy[u] = load_raw<BF16, true>(a.dy, t, a.dy_stride, cv);
    }
  };
  auto work_batch = [&](int tb, const Batch& b) {       // (tb - t0) is a multiple of U, hence of K
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int t = tb + u;
      const int slot = u % K;
      if (t < t_end) {
        if (t < a.n_tokens) {
          float dyt[NV];
          unpack_raw<BF16>(b.x[u], xr[slot]);
          unpack_raw<BF16>(b.dy[u], dyt);
          if (t == t0 || b.p[u] != t - 1) rebuild_ring<BF16, K>(a, b.p[u], cv, slot, xr);
#pragma unroll
          for (int i = 0; i < NV; i++) {
            float pre = wt.b[i] + wt.w[K - 1][i] * xr[slot][i];
#pragma unroll
            for (int m = 1; m < K; m++) pre += wt.w[K - 1 - m][i] * xr[ring_back<K>(slot, m)][i];
            gq[slot][i] = a.silu ? dyt[i] * dsilu_f(pre) : dyt[i];
          }
          lk[slot] = b.p[u] == t - 1;
          if (t < t1) {
#pragma unroll
            for (int i = 0; i < NV; i++) {
              db[i] += gq[slot][i];
#pragma unroll
              for (int m = 0; m < K; m++) dw[K - 1 - m][i] += gq[slot][i] * xr[ring_back<K>(slot, m)][i];
            }
          }
        } else {
          lk[slot] = false;
#pragma unroll
          for (int i = 0; i < NV; i++) gq[slot][i] = 0.f;
        }
        const int s = t - (K - 1);                // its g sits K-1 slots back; successor m one slot further on each
        if (s >= t0) {                            // s < t1 by the loop bound
          float dx[NV];
#pragma unroll
          for (int i = 0; i < NV; i++) dx[i] = wt.w[K - 1][i] * gq[ring_back<K>(slot, K - 1)][i];
          bool valid = true;
#pragma unroll
          for (int m = 1; m < K; m++) {
            valid = valid && lk[ring_back<K>(slot, K - 1 - m)];
            if (valid) {
#pragma unroll
              for (int i = 0; i < NV; i++) dx[i] += wt.w[K - 1 - m][i] * gq[ring_back<K>(slot, K - 1 - m)][i];
            }
          }
          store_row<BF16, true>(a.y, s, a.y_stride, cv, dx);
        }
      }
    }
  };
  Batch ba, bb;
  load_batch(t0, ba);
  static_assert(CONV_SUM_RUN % (2 * U) == 0);
  int turns = 0;
  for (int tb = t0; tb < t_end; tb += 2 * U) {
    load_batch(tb + U, bb);
    work_batch(tb, ba);
    load_batch(tb + 2 * U, ba);
    work_batch(tb + U, bb);
    if (++turns == CONV_SUM_RUN / (2 * U)) {
      turns = 0;
      end_run();
    }
  }
  end_run();
  float* part = a.partial + (int64_t)tile * (K + 1) * a.channels + cv * NV;
#pragma unroll
  for (int j = 0; j < K; j++)
#pragma unroll
    for (int i = 0; i < NV; i++) part[(int64_t)j * a.channels + i] = dw_runs[j][i];
#pragma unroll
  for (int i = 0; i < NV; i++) part[(int64_t)K * a.channels + i] = db_runs[i];
}

// Backward, fix-up: dx of the tokens that have a successor outside the "directly follows" chain.
// Each listed token is recomputed completely (chain part + listed extra successors) and overwrites
// what the fast path stored, so every dx row has one writer last and one rounding.
template <bool BF16, int K>
__device__ __forceinline__ void conv_fix_block(const ConvArgs& a, int64_t block) {
  constexpr int NV = Chan<BF16>::NV;
  const int64_t gid = block * CONV_THREADS + threadIdx.x;
  const int vpr = a.channels / NV;
  const int64_t f = gid / vpr;
  const int cv = (int)(gid - f * vpr);
  if (f >= a.n_fix) return;
  Weights<BF16, K> wt;
  wt.load(a, cv * NV);
  const int s = a.fix_tok[f];
  float dx[NV];
#pragma unroll
  for (int i = 0; i < NV; i++) dx[i] = 0.f;
  // Successors along a run of directly-following tokens that starts at `first`, whose distance from s is `r`.  A few rows
  // of work, so it is the chain of loads that counts: what does not hang on the predecessor chain of `first` (the rows
  // of up to K tokens of the run) is requested beside it, and the window moves along the run instead of being looked
  // up again for every token.  (The finish launch at 16406 x 8192: 31 us, with the reduce below in 16 segments 23, with
  // this 11; it is the larger part of a small call: 700 x 2048 61 -> 39 us.)
  // (N tokens at most: K from s itself, K - 1 from a listed successor, which is at least one place away.)
  auto add_run = [&](auto n_tok, int first, int r) {
    constexpr int N = decltype(n_tok)::value;
    int pr[N];
    typename Chan<BF16>::Raw xq[N], dyq[N];
#pragma unroll
    for (int u = 0; u < N; u++) {
      const int t = min(first + u, a.n_tokens - 1);
      pr[u] = a.tok_pred[t];
      xq[u] = load_raw<BF16>(a.x, t, a.x_stride, cv);
      dyq[u] = load_raw<BF16>(a.dy, t, a.dy_stride, cv);
    }
    float win[K][NV];                                        // x of the token, of its predecessor, ...
    {
      float before[K - 1][NV];
      rebuild_window<BF16, K>(a, pr[0], cv, before);
#pragma unroll
      for (int m = 1; m < K; m++)
#pragma unroll
        for (int i = 0; i < NV; i++) win[m][i] = before[m - 1][i];
    }
    bool in_run = true;
#pragma unroll
    for (int u = 0; u < N; u++) {
      in_run = in_run && r + u < K && (u == 0 || (first + u < a.n_tokens && pr[u] == first + u - 1));
      if (u > 0) {
#pragma unroll
        for (int m = K - 1; m > 0; m--)
#pragma unroll
          for (int i = 0; i < NV; i++) win[m][i] = win[m - 1][i];
      }
      unpack_raw<BF16>(xq[u], win[0]);
      float g[NV];
      unpack_raw<BF16>(dyq[u], g);
      if (in_run) {
        const int j = K - 1 - (r + u);
#pragma unroll
        for (int i = 0; i < NV; i++) {
          float pre = wt.b[i];
#pragma unroll
          for (int m = 0; m < K; m++) pre += wt.w[K - 1 - m][i] * win[m][i];
          if (a.silu) g[i] *= dsilu_f(pre);
          // weight row j selected without dynamic register indexing
          float wj = wt.w[0][i];
#pragma unroll
          for (int jj = 1; jj < K; jj++) wj = jj == j ? wt.w[jj][i] : wj;
          dx[i] += wj * g[i];
        }
      }
    }
  };
  add_run(std::integral_constant<int, K>{}, s, 0);
  for (int e = a.fix_off[f]; e < a.fix_off[f + 1]; e++) add_run(std::integral_constant<int, K - 1>{}, a.fix_t[e], a.fix_r[e]);
  store_row<BF16>(a.y, s, a.y_stride, cv, dx);
}

// dweight[c][j] = sum over tiles of partial[tile][j][c]; dbias[c] = same for j = K.  Fixed order: the tiles are
// cut into RED_SEG consecutive segments, one thread sums one segment of four outputs in tile order (8 loads in
// flight), and the segment sums are added in segment order -- the same association on every run.  A workgroup
// covers RED_OUT consecutive outputs x RED_SEG segments, so a segment's threads read 256 contiguous bytes per tile.
constexpr int RED_SEG = 16, RED_OUT = 4 * CONV_THREADS / RED_SEG;
__device__ __forceinline__ void conv_reduce_block(const float* __restrict__ partial, int n_tiles, int K, int channels,
                                                  float* __restrict__ dweight, float* __restrict__ dbias, int64_t block) {
  __shared__ f32x4v seg_sum[RED_SEG][RED_OUT / 4];
  const int o = threadIdx.x % (RED_OUT / 4), sg = threadIdx.x / (RED_OUT / 4);
  const int64_t n_out = (int64_t)(K + 1) * channels;        // a multiple of 4, as channels is
  const int64_t gid = block * RED_OUT + 4 * o;
  const int per = (n_tiles + RED_SEG - 1) / RED_SEG;
  const int t_lo = min(sg * per, n_tiles), t_hi = min(t_lo + per, n_tiles);
  f32x4v acc = {0.f, 0.f, 0.f, 0.f};
  if (gid < n_out) {
    const float* src = partial + gid;
    int t = t_lo;
    for (; t + 8 <= t_hi; t += 8) {
      f32x4v v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = *(const f32x4v*)(src + (int64_t)(t + u) * n_out);
#pragma unroll
      for (int u = 0; u < 8; u++) acc += v[u];
    }
    for (; t < t_hi; t++) acc += *(const f32x4v*)(src + (int64_t)t * n_out);
  }
  seg_sum[sg][o] = acc;
  __syncthreads();
  if (threadIdx.x < RED_OUT && block * RED_OUT + threadIdx.x < n_out) {
    const int64_t out = block * RED_OUT + threadIdx.x;
    const float* col = (const float*)seg_sum + threadIdx.x;
    float tot = col[0];
#pragma unroll
    for (int q = 1; q < RED_SEG; q++) tot += col[q * RED_OUT];
    const int j = (int)(out / channels), c = (int)(out - (int64_t)j * channels);
    if (j < K) dweight[(int64_t)c * K + j] = tot;
    else if (dbias) dbias[c] = tot;
  }
}

// What follows the fast path of the backward, in one launch: the first n_reduce_blocks workgroups sum the
// weight-gradient partials, the others recompute the dx rows of the listed branch-point tokens (the two jobs touch
// different outputs and both only need the fast path to have finished).
template <bool BF16, int K>
__global__ __launch_bounds__(CONV_THREADS) void tree_conv_finish_kernel(ConvArgs a, float* dweight, float* dbias, int n_reduce_blocks) {
  if ((int)blockIdx.x < n_reduce_blocks) conv_reduce_block(a.partial, a.n_tiles, K, a.channels, dweight, dbias, blockIdx.x);
  else conv_fix_block<BF16, K>(a, (int64_t)blockIdx.x - n_reduce_blocks);
}

int pick_tile(int64_t n_tokens, int vpr, int lo, int hi) {
  // enough lanes for the chip (about 1024 workgroups) without making tiles shorter than `lo` tokens
  int tile = hi;
  while (tile > lo && tt::ceil_div(n_tokens, tile) * vpr < (int64_t)1024 * CONV_THREADS) tile >>= 1;
  return tile;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + CONV_THREADS - 1) / CONV_THREADS); }

template <bool BF16, int K>
hipError_t launch_fwd(const ConvArgs& a, hipStream_t st) {
  tree_conv_fwd_kernel<BF16, K><<<blocks_for((int64_t)a.n_tiles * (a.channels / Chan<BF16>::NV)), CONV_THREADS, 0, st>>>(a);
  return hipGetLastError();
}

template <bool BF16, int K>
hipError_t launch_bwd(const ConvArgs& a, float* dweight, float* dbias, hipStream_t st) {
  const int vpr = a.channels / Chan<BF16>::NV;
  if (a.n_tiles > 0) {
    KernelTimer t(TT_KERNEL_CONV_BWD, st);
    tree_conv_bwd_kernel<BF16, K><<<blocks_for((int64_t)a.n_tiles * vpr), CONV_THREADS, 0, st>>>(a);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  {
    KernelTimer t(TT_KERNEL_CONV_FIX, st);
    const int64_t n_out = (int64_t)(K + 1) * a.channels;
    const int n_reduce_blocks = (int)((n_out + RED_OUT - 1) / RED_OUT);
    const unsigned n_fix_blocks = a.n_fix > 0 ? blocks_for((int64_t)a.n_fix * vpr) : 0;
    tree_conv_finish_kernel<BF16, K><<<(unsigned)n_reduce_blocks + n_fix_blocks, CONV_THREADS, 0, st>>>(a, dweight, dbias, n_reduce_blocks);
  }
  return hipGetLastError();
}

#define TT_CONV_DISPATCH(FN, ...)                                            \
  switch (kernel_size) {                                                     \
    case 2: return bf16 ? FN<true, 2>(__VA_ARGS__) : FN<false, 2>(__VA_ARGS__); \
    case 3: return bf16 ? FN<true, 3>(__VA_ARGS__) : FN<false, 3>(__VA_ARGS__); \
    case 4: return bf16 ? FN<true, 4>(__VA_ARGS__) : FN<false, 4>(__VA_ARGS__); \
    default: return hipErrorInvalidValue;                                    \
  }

}  // namespace

// Tokens per tile of the backward walk: long tiles (each walks K - 1 tokens of look-ahead and writes a row of partial sums)
// that still make one workgroup for every one of the chip's conv_bwd_wgs * 256 places, 32 to CONV_BWD_TILE tokens; never
// shorter than the power of two that makes 1024 workgroups of 16-byte lanes, which bounds the partial sums.  In fp32, where
// a row takes twice the lanes, the longest tile is reached from 16384 tokens x 6144 channels on; from 8 tokens beyond it on
// the tokens are cut into equal rounds of all places (a second round of more than a few workgroups costs as much as a full one), and
// from 128 tokens on a tile is a multiple of the 8 tokens that a turn of the loop takes.
// Whole backward and forward at 16406 x 8192 bf16, K = 4: tiles of 64 tokens 314 us, 128 294, 171 (this rule) 291; 32000 x
// 8192: 167 tokens 616 us, 256 (this rule) 591;  fp32, tiles of a power of two for 1024 workgroups / one round without the two rules
// / this: 9000 x 4096 196 / 170 / 170, 16406 x 4096 276 / 292 / 273, 16406 x 6144 450 / 474 / 435, 24000 x 6144 663 / 727 / 620, 20000 x 8192
// 680 / 729 / 660, 16406 x 8192 642 / 542 / 542.
int conv_bwd_tile(int64_t n_tokens, int channels, bool bf16) {
  const int64_t vpr = channels / (bf16 ? Chan<true>::NV : Chan<false>::NV);
  const int64_t tiles = std::max<int64_t>(1, (int64_t)conv_bwd_wgs(bf16) * 256 * CONV_THREADS / vpr);      // of one round
  int64_t tile = tt::ceil_div(n_tokens, tiles);
  if (!bf16) {
    const int64_t rounds = std::max<int64_t>(1, tt::ceil_div(tile, CONV_BWD_TILE + 8));
    tile = tt::ceil_div(n_tokens, tiles * rounds);
    if (tile >= 128) tile = tt::ceil_div(tile, 8) * 8;
  }
  return (int)std::max<int64_t>(pick_tile(n_tokens, channels / (bf16 ? 8 : 4), 32, 256), std::min<int64_t>(tile, CONV_BWD_TILE));
}

size_t conv_bwd_workspace(int64_t n_tokens, int channels, int kernel_size, bool bf16) {
  const int tile = conv_bwd_tile(n_tokens, channels, bf16);
  return (size_t)tt::ceil_div(n_tokens, tile) * (size_t)(kernel_size + 1) * (size_t)channels * sizeof(float) + 256;
}

hipError_t conv_fwd(int64_t n_tokens, int channels, int kernel_size, bool bf16, bool silu, const void* x, int64_t x_stride_bytes,
                    const float* weight, const float* bias, const int32_t* tok_pred, void* y, int64_t y_stride_bytes,
                    hipStream_t st) {
  if (n_tokens == 0) return hipSuccess;
  ConvArgs a{};
  a.n_tokens = (int)n_tokens; a.channels = channels; a.silu = silu ? 1 : 0;
  a.tok_tile = pick_tile(n_tokens, channels / Chan<true>::NV, 16, 64);
  a.n_tiles = (int)tt::ceil_div(n_tokens, a.tok_tile);
  a.x = x; a.x_stride = x_stride_bytes; a.weight = weight; a.bias = bias; a.tok_pred = tok_pred;
  a.y = y; a.y_stride = y_stride_bytes;
  KernelTimer t(TT_KERNEL_CONV_FWD, st);
  TT_CONV_DISPATCH(launch_fwd, a, st)
}

hipError_t conv_bwd(int64_t n_tokens, int channels, int kernel_size, bool bf16, bool silu, const void* x, int64_t x_stride_bytes,
                    const float* weight, const float* bias, const int32_t* tok_pred, const void* dy, int64_t dy_stride_bytes,
                    int n_fix, const int32_t* fix_tok, const int32_t* fix_off, const int32_t* fix_t, const int32_t* fix_r,
                    void* dx, int64_t dx_stride_bytes, float* dweight, float* dbias, void* workspace, hipStream_t st) {
  ConvArgs a{};
  a.n_tokens = (int)n_tokens; a.channels = channels; a.silu = silu ? 1 : 0;
  a.tok_tile = conv_bwd_tile(n_tokens, channels, bf16);
  a.n_tiles = (int)tt::ceil_div(n_tokens, a.tok_tile);
  a.x = x; a.x_stride = x_stride_bytes; a.weight = weight; a.bias = bias; a.tok_pred = tok_pred;
  a.y = dx; a.y_stride = dx_stride_bytes; a.dy = dy; a.dy_stride = dy_stride_bytes;
  a.partial = (float*)workspace;
  a.n_fix = n_fix; a.fix_tok = fix_tok; a.fix_off = fix_off; a.fix_t = fix_t; a.fix_r = fix_r;
  TT_CONV_DISPATCH(launch_bwd, a, dweight, dbias, st)
}

}  // namespace tt
