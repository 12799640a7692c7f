// Gated delta rule with tree state routing, backward (Section "Implementation", paragraph "SSM Layers
// (GDN)" (i): gradients accumulate at the shared parent state; Appendix "Tree-Aware SSM State
// Routing").  Chunked like the forward (64 tokens, chunks never cross a node boundary).  With
//     Vn = U - W S0,   O = Qg S0 + P Vn,   S1 = EL S0 + Kd^T Vn
// (Qg = scale exp(gamma) Q, Kd = exp(gamma_last - gamma) K, EL = exp(gamma_last), U = (I+A)^-1 beta V,
// W = (I+A)^-1 beta exp(gamma) K, A = beta_i A0_ij, A0 = strictly-lower((k_i.k_j) D_ij),
// P = scale tril((q_i.k_j) D_ij), D_ij = exp(gamma_i - gamma_j)) the chain rule gives, per chunk,
//     dVn = P^T dO + Kd dS1                      dS0 = EL dS1 + Qg^T dO - W^T dVn          (serial part)
//     dQg = dO S0^T    dKd = Vn dS1^T    dW = -dVn S0^T    dP = tril(dO Vn^T)
//     [dVb | dKb] = (I+A)^-T [dVn | dW]          dA = strictly-lower(-dVb U^T - dKb W^T)
// and from there dq, dk, dv, dbeta and dgamma by the product rule; dg is the reverse running sum of
// dgamma inside the chunk.  State routing backwards: dS1 of a chunk is the dS0 of the chunk that
// continued from it on chip plus the gradient collected in its saved-state slot (every chunk that
// started from the slot added its dS0 there; they all come later in DFS order, so a reverse walk over
// the chunks has seen them), plus the upstream gradient of a captured state.
//
// Kernels (the first three live in tt_gdn.hip with the forward's):
//   gdn_prepare_kernel<true>   per (chunk, head): the bf16 record of both walks, what the reverse walk needs besides
//                              (P^T, dO^T), and gamma and (I + A)^-1 unrounded
//   gdn_scan_kernel<true>      (32 value columns, head): the forward scan without its output; saves S0 and Vn
//                              of every chunk (bf16)
//   gdn_rscan_kernel           (32 value columns, head): reverse walk in the forward scan's form (bf16 matrix
//                              instruction, fp32 state gradient in accumulators); saves dS1 and dVn (bf16)
//   gdn_bwd_finish_kernel      per (chunk, key head): everything else: products on the bf16 matrix instruction (fp32
//                              accumulation), the transposed solve as a product with the inverse and all element-wise
//                              work in fp32; dq / dk summed over the key head's value heads in registers
//   gdn_bwd_group_sum_kernel   calls with few chunks: sums fp32 dq / dk over the value heads, rounds to bf16
#include <hip/hip_runtime.h>
#include <algorithm>
#include "tt_internal.h"
#include "tt_kernels.h"
#include "tt_mfma.h"

namespace tt {
namespace {

constexpr int GC = TT_GDN_CHUNK;     // 64
constexpr int GD = 128;
constexpr int BT = 256;

struct BwdWs {
  GdnChunkOps ops;
  GdnBwdSaved sv;
  float* dqh;        // split calls only: [N][hv_n][128] per-value-head dq, dk (the heads of the pass)
  float* dkh;
};
struct KArgs {
  GdnBwdArgs b;
  BwdWs w;
};

__device__ __forceinline__ float4 ld4(const float* p) { return *(const float4*)p; }

// Register r of a 32 x 32 accumulator tile holds row (r / 4) * 8 + 4 hf + r % 4 of column lane % 32.
__device__ __forceinline__ int tile_row(int r, int hf) { return (r >> 2) * 8 + 4 * hf + (r & 3); }

// ---- per-chunk finish ----------------------------------------------------------------------------------
// One workgroup of four waves per (chunk, key head); it goes through the value heads of the key head one after the
// other and keeps dq and dk, which are sums over them, in accumulator registers (SPLIT: one value head per workgroup, dq /
// dk of every head in fp32 to memory, summed by gdn_bwd_group_sum_kernel).  What bounds it is memory: about 190 KB of
// operands per (chunk, value head), of which every byte is read once.  To that end everything that shares an operand is
// done while that operand is on chip:
//   1. one pass over the four blocks of 32 value columns with S0, dS1, dO, Vn and dVn of the block in LDS:
//      dW = -dVn S0^T, dQg = dO S0^T, dKd = Vn dS1^T, dP = dO Vn^T and <dS1, S0>
//   2. [dVb | dKb]^T = [dVn | dW]^T T on both halves of the split T; the result stays in LDS.  A wave's dW
//      accumulators are, as bf16, the A fragments of its own column block
//   3. dA = -[dVb | dKb] [U | W]^T, dv and dbeta's part from dVb
//   4. K K^T and Q K^T again (K and Q stay in LDS for all heads; cheaper than 32 KB of A0 and P per head out and in):
//      row and column sums of dP o P + dA o A in registers, dP scale D and dA beta D as bf16 to LDS
//   5. dq += (dP scale D) K;  dk += (dP scale D)^T Q + (dA beta D) K + (dA beta D)^T K + beta eg dKb
// LDS 80 KB: two workgroups per compute unit, one's loads beside the other's products.  16406 tokens, 16 / 32 heads: 0.50
// ms at 2.3 GB (4.6 TB/s; a large copy reaches 4.8).  The loop over the heads spills 24 registers (76 bytes per lane and
// head out and in again): 0.18 of the 0.46 GB that the kernel writes at that size, 8 % of its traffic.  With one value head
// per workgroup, fp32 dq / dk through memory, A0 and P from memory and S0, dS1, dO, Vn read once per product it was 0.86 ms
// at 4.9 GB and 0.12 ms for the sum.
// Register r of a wave's tile (row block t, column block w) of a 64 x 128 result: row 32 t + tile_row(r), column
// 32 w + lane % 32; of a 64 x 64 result: row block w & 1, column block w >> 1.
constexpr int PG = GD + 8;                               // LDS pitches (elements): rows 16-byte aligned, 8 elements of
constexpr int PK = GC + 8;                               // padding against bank conflicts

struct FinishSmem {
  __bf16 k[GC * PG], q[GC * PG];                         // rows of K and Q, zero past the chunk's length
  // step 1: slabs S0^T, dS1^T [32 columns][128], Vn, dVn [32 columns][64 tokens];  step 2: T as hi and lo halves;  from
  // there on dVb and dKb [token][128];  after step 3 dP scale D in dVb's place, and the closing sums behind it
  __bf16 x[2 * GC * PG];
  __bf16 r2[GC * PK];                                    // dO, 64 columns; U^T, 64 rows, then -W, 64 columns; dA beta D
  float gam[GC], bet[GC], eg[GC], el[GC], db_v[GC];
  float dg_row[2][GC], dg_col[2][GC], db_a[2][GC];       // per column / row block
};
static_assert(sizeof(FinishSmem) <= 80 * 1024, "two workgroups per compute unit");
constexpr int SLAB = 32;                                 // value columns per slab of step 1
constexpr int X_S0 = 0, X_DS1 = SLAB * PG, X_VN = 2 * SLAB * PG, X_DVN = 2 * SLAB * PG + SLAB * PK;
constexpr int X_TLO = GC * PK;
constexpr int X_KB = GC * PG;                            // dKb
constexpr int X_SUMS = GC * PK;                          // 9 x 64 floats
static_assert(X_DVN + SLAB * PK <= 2 * GC * PG && X_SUMS % 8 == 0 && X_SUMS + 2 * 9 * GC <= X_KB && GC * PK <= X_SUMS, "LDS areas");

// Barrier that waits for this wave's LDS traffic only (a __syncthreads also waits for every global load in flight,
// i.e. for what was requested ahead).  Not for global data written by other threads of the workgroup.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sums 16 values over the 32 lanes of a half wave (the lanes that hold one row of an accumulator tile in register r): every
// step folds the lane positions on each other and hands half of the values to either side, so that 16 sums take 16
// additions instead of 80.  Lane c of the half gets the total of v[c % 16].
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float half_wave_sums(float (&v)[16], int c) {
  const bool b3 = c & 8, b2 = c & 4, b1 = c & 2, b0 = c & 1;
#pragma unroll
  for (int r = 0; r < 8; r++) v[r] = (b3 ? v[r + 8] : v[r]) + dpp_move<0x140>(b3 ? v[r] : v[r + 8]);     // row_mirror: lane ^ 15
#pragma unroll
  for (int r = 0; r < 4; r++) v[r] = (b2 ? v[r + 4] : v[r]) + dpp_move<0x141>(b2 ? v[r] : v[r + 4]);     // row_half_mirror: lane ^ 7
#pragma unroll
  for (int r = 0; r < 2; r++) v[r] = (b1 ? v[r + 2] : v[r]) + dpp_move<0x4e>(b1 ? v[r] : v[r + 2]);      // quad_perm: lane ^ 2
  const float x = (b0 ? v[1] : v[0]) + dpp_move<0xb1>(b0 ? v[0] : v[1]);                                   // quad_perm: lane ^ 1
  const auto o = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);   // lane ^ 16
  return __uint_as_float(o[0]) + __uint_as_float(o[1]);
}

// The value is formed at this point of the program.  (The compiler moves additions to their use two steps later and keeps
// both operands in registers until then: 94 spilled registers, 1.3 GB of scratch traffic and 0.82 ms at 16 K tokens.)
template <class T> __device__ __forceinline__ void form_here(T& x) { asm volatile("" : "+v"(x)); }

template <bool SPLIT>
__global__ __launch_bounds__(BT, 2) void gdn_bwd_finish_kernel(KArgs a) {
  __shared__ __attribute__((aligned(16))) FinishSmem sm;
  const int nc = a.b.n_chunks, hv = a.b.hv, rep = hv / a.b.hk;
  int chunk, unit;                                       // unit: key head (SPLIT: value head) inside this pass
  if (!gdn_group_order(blockIdx.x, nc, SPLIT ? a.b.hv_n : a.b.hv_n / rep, SPLIT ? rep : 1, chunk, unit)) return;
  const int kh = SPLIT ? unit / rep : unit;
  const int tok0 = a.b.chunk_tok0[chunk], len = a.b.chunk_len[chunk];
  const float scale = a.b.scale;
  const size_t qrow = (size_t)a.b.hk * GD, vrow = (size_t)hv * GD;
  bf16x8 zero8;
#pragma unroll
  for (int e = 0; e < 8; e++) zero8[e] = (__bf16)0.f;

  // Thread positions (ib, jb: this wave's tile of a 64 x 64 result).  LDS and memory offsets are functions of these alone:
  // taken from an opaque copy per step, they are formed where they are used; otherwise the compiler forms those of all
  // steps in front of the loop over the heads and keeps them.
  int tid, lane, c, hf, c16, w, ib, jb;
  auto place = [&]() {
    int t = threadIdx.x & (BT - 1);
    asm volatile("" : "+v"(t)::"memory");
    tid = t; lane = t & 63; c = lane & 31; hf = lane >> 5; c16 = 16 * (c >> 4);
    w = __builtin_amdgcn_readfirstlane(t >> 6);
    ib = w & 1; jb = w >> 1;
  };
  // The pieces of a slab, and what a head starts with (slab 0 and the chunk's scalars): requested one slab ahead, a head's
  // first ones during the last step of the head in front of it.
  bf16x8 s0r[2], ds1r[2], vnr, dvnr, dor[2];
  float glast, gv, bv;
  auto load_slab = [&](int h, int cb) {
    // saved by the walks (bf16): S0 and dS1 transposed [value col][key dim], Vn and dVn in fragment order
    const size_t op = (size_t)h * nc + chunk;
    const __bf16* s0t = (const __bf16*)a.w.sv.s0t + op * (GD * GD) + cb * (SLAB * GD);
    const __bf16* ds1t = (const __bf16*)a.w.sv.ds1t + op * (GD * GD) + cb * (SLAB * GD);
#pragma unroll
    for (int p = 0; p < 2; p++) {
      s0r[p] = *(const bf16x8*)(s0t + 8 * (tid + p * BT));
      ds1r[p] = *(const bf16x8*)(ds1t + 8 * (tid + p * BT));
    }
    vnr = *(const bf16x8*)((const __bf16*)a.w.sv.vns + op * (GC * GD) + cb * (SLAB * GC) + 8 * tid);
    dvnr = *(const bf16x8*)((const __bf16*)a.w.sv.dvns + op * (GC * GD) + cb * (SLAB * GC) + 8 * tid);
    if ((cb & 1) == 0) {
      const __bf16* dob = (const __bf16*)a.b.d_o + (size_t)tok0 * vrow + (size_t)h * GD + cb * SLAB;
#pragma unroll
      for (int p = 0; p < 2; p++) {
        const int piece = tid + p * BT, i = piece >> 3, k8 = (piece & 7) * 8;
        dor[p] = *(const bf16x8*)(dob + (size_t)min(i, len - 1) * vrow + k8);
      }
    }
  };
  auto load_head = [&](int h) {
    const float* gam = a.w.ops.gam + ((size_t)h * nc + chunk) * GC;
    glast = gam[GC - 1];
    gv = gam[lane];
    bv = a.b.beta[(size_t)(tok0 + min(lane, len - 1)) * hv + h];
    load_slab(h, 0);
  };
  {
    place();
    const __bf16* qb = (const __bf16*)a.b.q + (size_t)tok0 * qrow + (size_t)kh * GD;
    const __bf16* kb = (const __bf16*)a.b.k + (size_t)tok0 * qrow + (size_t)kh * GD;
    bf16x8 kr[4], qr[4];
#pragma unroll
    for (int p = 0; p < 4; p++) {
      const int piece = tid + p * BT, i = piece >> 4, c8 = (piece & 15) * 8;
      const size_t at = (size_t)min(i, len - 1) * qrow + c8;
      kr[p] = *(const bf16x8*)(kb + at);
      qr[p] = *(const bf16x8*)(qb + at);
    }
    load_head(SPLIT ? unit : kh * rep);
#pragma unroll
    for (int p = 0; p < 4; p++) {
      const int piece = tid + p * BT, i = piece >> 4, c8 = (piece & 15) * 8;
      *(bf16x8*)(sm.k + i * PG + c8) = i < len ? kr[p] : zero8;
      *(bf16x8*)(sm.q + i * PG + c8) = i < len ? qr[p] : zero8;
    }
  }

  f32x16 dq[2] = {zero16(), zero16()}, dk[2] = {zero16(), zero16()};
#pragma unroll 1
  for (int r_h = 0; r_h < (SPLIT ? 1 : rep); r_h++) {
    const int h = SPLIT ? unit : kh * rep + r_h;
    const size_t op = (size_t)h * nc + chunk;
    const __bf16* dvns = (const __bf16*)a.w.sv.dvns + op * (GC * GD);
    const __bf16* ut = (const __bf16*)a.w.sv.fwd_rec + op * GDN_REC_ELEMS + GDN_REC_UT;
    const __bf16* wn = (const __bf16*)a.w.sv.fwd_rec + op * GDN_REC_ELEMS + GDN_REC_WN;
    const __bf16* vb = (const __bf16*)a.b.v + (size_t)tok0 * vrow + (size_t)h * GD;

    // ---- 1. everything that contracts over value columns ----
    place();
    const float el_last = __expf(glast);
    if (tid < GC) {
      sm.gam[tid] = gv;
      sm.bet[tid] = tid < len ? bv : 0.f;
      sm.eg[tid] = __expf(gv);
      sm.el[tid] = __expf(glast - gv);
    }
    float s_dot = 0.f;                                   // this thread's part of <dS1, S0>
    bf16x8 xf[2][GC / 16];                               // A fragments of the right-hand sides of step 2
    float4 t_in[3];
    f32x16 dp = zero16();
    float row_qk[2], s_kd = 0.f;                         // row sums of dQg o Qg - dKd o Kd;  this thread's part of <dKd, Kd>
    {
      f32x16 dw[2] = {zero16(), zero16()}, dqg[2] = {zero16(), zero16()}, dkd[2] = {zero16(), zero16()};
#pragma unroll
      for (int cb = 0; cb < GD / SLAB; cb++) {
        place();
        lds_barrier();                                   // the previous slab (or whatever was here before) has been read
#pragma unroll
        for (int p = 0; p < 2; p++) {
          const int piece = tid + p * BT, at = (piece >> 4) * PG + (piece & 15) * 8;
          *(bf16x8*)(sm.x + X_S0 + at) = s0r[p];
          *(bf16x8*)(sm.x + X_DS1 + at) = ds1r[p];
#pragma unroll
          for (int e = 0; e < 8; e++) s_dot += (float)s0r[p][e] * (float)ds1r[p][e];
        }
        form_here(s_dot);
        {
          // one piece of a fragment-ordered array = 8 tokens of one column: base .. base + 3 and base + 8 .. base + 11
          const int f = tid >> 6, at = c * PK + 16 * f + 4 * hf;
          *(bf16x4*)(sm.x + X_VN + at) = __builtin_shufflevector(vnr, vnr, 0, 1, 2, 3);
          *(bf16x4*)(sm.x + X_VN + at + 8) = __builtin_shufflevector(vnr, vnr, 4, 5, 6, 7);
          *(bf16x4*)(sm.x + X_DVN + at) = __builtin_shufflevector(dvnr, dvnr, 0, 1, 2, 3);
          *(bf16x4*)(sm.x + X_DVN + at + 8) = __builtin_shufflevector(dvnr, dvnr, 4, 5, 6, 7);
        }
        if ((cb & 1) == 0) {
#pragma unroll
          for (int p = 0; p < 2; p++) {
            const int piece = tid + p * BT, i = piece >> 3, k8 = (piece & 7) * 8;
            *(bf16x8*)(sm.r2 + i * PK + k8) = i < len ? dor[p] : zero8;
          }
        }
        lds_barrier();
        if (cb + 1 < GD / SLAB) {
          load_slab(h, cb + 1);
        } else {
          // for step 2: T (three 32 x 32 blocks, the fourth is zero) and the dVn fragments of this wave's column block
          const float* tg = a.w.ops.t + op * GDN_T_ELEMS;
#pragma unroll
          for (int p = 0; p < 3; p++) t_in[p] = ld4(tg + 4 * (tid + p * BT));
#pragma unroll
          for (int s = 0; s < GC / 16; s++) xf[0][s] = ((const bf16x8*)dvns)[(w * 4 + s) * 64 + lane];
        }
#pragma unroll
        for (int s = 0; s < SLAB / 16; s++) {
          const int k0 = 16 * s + 8 * hf;
          const bf16x8 b_s0 = kmajor_frag(sm.x + X_S0, PG, k0, 32 * w + c16, lane);
          const bf16x8 b_ds1 = kmajor_frag(sm.x + X_DS1, PG, k0, 32 * w + c16, lane);
#pragma unroll
          for (int t = 0; t < 2; t++) {
            dw[t] = mfma32(kmajor_frag(sm.x + X_DVN, PK, k0, 32 * t + c16, lane), b_s0, dw[t]);
            dqg[t] = mfma32(*(const bf16x8*)(sm.r2 + (32 * t + c) * PK + (cb & 1) * SLAB + k0), b_s0, dqg[t]);
            dkd[t] = mfma32(kmajor_frag(sm.x + X_VN, PK, k0, 32 * t + c16, lane), b_ds1, dkd[t]);
          }
          dp = mfma32(*(const bf16x8*)(sm.r2 + (32 * ib + c) * PK + (cb & 1) * SLAB + k0),
                      kmajor_frag(sm.x + X_VN, PK, k0, 32 * jb + c16, lane), dp);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 2; t++) {
        place();
#pragma unroll
        for (int u = 0; u < 2; u++)
          xf[1][2 * t + u] = cvt8(-dw[t][8 * u], -dw[t][8 * u + 1], -dw[t][8 * u + 2], -dw[t][8 * u + 3], -dw[t][8 * u + 4],
                                  -dw[t][8 * u + 5], -dw[t][8 * u + 6], -dw[t][8 * u + 7]);
        // dq_i = scale exp(gamma_i) dQg_i + ...;  dk_j = exp(gamma_last - gamma_j) dKd_j + ...;  their dot products with
        // q_i and k_j go into dgamma.  (A k-major fragment in accumulator order holds the rows of 8 registers.)
        float dot[16];
#pragma unroll
        for (int u = 0; u < 2; u++) {
          const bf16x8 qf = kmajor_frag_acc_order(sm.q, PG, 32 * t + 16 * u + 4 * hf, 32 * w + c16, lane);
          const bf16x8 kf = kmajor_frag_acc_order(sm.k, PG, 32 * t + 16 * u + 4 * hf, 32 * w + c16, lane);
#pragma unroll
          for (int v4 = 0; v4 < 2; v4++) {
            const int i4 = 32 * t + 16 * u + 8 * v4 + 4 * hf;
            const f32x4 eg4 = *(const f32x4*)(sm.eg + i4), el4 = *(const f32x4*)(sm.el + i4);
#pragma unroll
            for (int e = 0; e < 4; e++) {
              const int r = 8 * u + 4 * v4 + e;
              const float vq = scale * eg4[e] * dqg[t][r], vk = el4[e] * dkd[t][r], vkk = vk * (float)kf[4 * v4 + e];
              dot[r] = vq * (float)qf[4 * v4 + e] - vkk;
              s_kd += vkk;
              dq[t][r] += vq;
              dk[t][r] += vk;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        row_qk[t] = half_wave_sums(dot, c);
        form_here(dq[t]);
        form_here(dk[t]);
      }
    }

    place();
    // ---- 2. (I + A)^T [dVb | dKb] = [dVn | dW]: X^T = rhs^T T ----
    bf16x8 ur[2][2], vv[4];
    // two slabs ahead: 64 rows of U^T (value columns), or 64 columns (key dims) of the rows of -W
    auto load_uw = [&](int s) {
#pragma unroll
      for (int p = 0; p < 2; p++) {
        const int piece = tid + p * BT;
        ur[s & 1][p] = *(const bf16x8*)(s < 2 ? ut + s * (GC * GC) + 8 * piece
                                              : wn + (s - 2) * GC + (piece >> 3) * GD + (piece & 7) * 8);
      }
    };
    const int v_i = tid >> 2, v_c0 = (tid & 3) * 32;     // step 3: this thread's row and columns of dVb
    lds_barrier();                                       // the last slab has been read
#pragma unroll
    for (int p = 0; p < 3; p++) {
      const int k = (p > 0 ? 32 : 0) + (tid >> 3), i4 = (p == 2 ? 32 : 0) + (tid & 7) * 4;
      const float4 v = t_in[p];
      const bf16x4 h4 = cvt4(v.x, v.y, v.z, v.w);
      *(bf16x4*)(sm.x + k * PK + i4) = h4;
      *(bf16x4*)(sm.x + X_TLO + k * PK + i4) = cvt4(v.x - (float)h4[0], v.y - (float)h4[1], v.z - (float)h4[2], v.w - (float)h4[3]);
    }
    lds_barrier();
    load_uw(0);
    load_uw(1);
#pragma unroll
    for (int q = 0; q < 4; q++) vv[q] = *(const bf16x8*)(vb + (size_t)min(v_i, len - 1) * vrow + v_c0 + 8 * q);
    {
      bf16x4 xo[2][2][4];                                // the result as bf16, one column block of T at a time (registers)
#pragma unroll
      for (int cb = 0; cb < 2; cb++) {
        f32x16 xa[2] = {zero16(), zero16()};
#pragma unroll
        for (int s = 2 * cb; s < GC / 16; s++) {         // (rows 0 .. 31 of T are zero from column 32 on)
          const bf16x8 th = kmajor_frag_acc_order(sm.x, PK, 16 * s + 4 * hf, 32 * cb + c16, lane);
          const bf16x8 tl = kmajor_frag_acc_order(sm.x + X_TLO, PK, 16 * s + 4 * hf, 32 * cb + c16, lane);
#pragma unroll
          for (int m = 0; m < 2; m++) {
            xa[m] = mfma32(xf[m][s], th, xa[m]);
            xa[m] = mfma32(xf[m][s], tl, xa[m]);
          }
        }
#pragma unroll
        for (int m = 0; m < 2; m++)
#pragma unroll
          for (int r4 = 0; r4 < 4; r4++)
            xo[m][cb][r4] = cvt4(xa[m][4 * r4], xa[m][4 * r4 + 1], xa[m][4 * r4 + 2], xa[m][4 * r4 + 3]);
        __builtin_amdgcn_sched_barrier(0);
      }
      lds_barrier();                                     // T has been read
      // a lane holds row i = 32 cb + c and, per register group, 4 consecutive columns
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
          for (int r4 = 0; r4 < 4; r4++)
            *(bf16x4*)(sm.x + m * X_KB + (32 * cb + c) * PG + 32 * w + 8 * r4 + 4 * hf) = xo[m][cb][r4];
    }

    // ---- 3. dA = strictly-lower(-[dVb | dKb] [U | W]^T);  dv_i = beta_i dVb_i,  dbeta_i += dVb_i . v_i ----
    f32x16 da = zero16();
#pragma unroll
    for (int s = 0; s < 4; s++) {
      place();
      lds_barrier();                                     // the previous slab has been read (first time: dVb, dKb are there)
#pragma unroll
      for (int p = 0; p < 2; p++) {
        const int piece = tid + p * BT;
        *(bf16x8*)(sm.r2 + (piece >> 3) * PK + (piece & 7) * 8) = ur[s & 1][p];
      }
      lds_barrier();
      if (s < 2) load_uw(s + 2);
      if (s == 2) {                                      // from the second half on the records hold -W
#pragma unroll
        for (int r = 0; r < 16; r++) da[r] = -da[r];
      }
#pragma unroll
      for (int ss = 0; ss < 4; ss++) {
        const bf16x8 uw = s < 2 ? kmajor_frag(sm.r2, PK, 16 * ss + 8 * hf, 32 * jb + c16, lane)
                                : *(const bf16x8*)(sm.r2 + (32 * jb + c) * PK + 16 * ss + 8 * hf);
        da = mfma32(*(const bf16x8*)(sm.x + (s >> 1) * X_KB + (32 * ib + c) * PG + (s & 1) * 64 + 16 * ss + 8 * hf), uw, da);
      }
      if (s == 0) {
        float dot = 0.f;
        const float b = sm.bet[v_i];
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const bf16x8 xb = *(const bf16x8*)(sm.x + v_i * PG + v_c0 + 8 * q);
          float xv[8];
#pragma unroll
          for (int e = 0; e < 8; e++) {
            xv[e] = (float)xb[e];
            dot += xv[e] * (float)vv[q][e];
          }
          if (v_i < len)
            *(bf16x8*)((__bf16*)a.b.dv + ((size_t)(tok0 + v_i) * hv + h) * GD + v_c0 + 8 * q) =
                cvt8(b * xv[0], b * xv[1], b * xv[2], b * xv[3], b * xv[4], b * xv[5], b * xv[6], b * xv[7]);
        }
        dot += __shfl_xor(dot, 1);
        dot += __shfl_xor(dot, 2);
        if ((tid & 3) == 0) sm.db_v[v_i] = v_i < len ? dot : 0.f;
      }
    }

    // ---- 4. G = dP o P + dA o A: its row sums minus its column sums are the part of dgamma that comes through D ----
    {
      place();
      f32x16 kk = zero16(), qk = zero16();
#pragma unroll
      for (int s = 0; s < GD / 16; s++) {
        const bf16x8 kj = *(const bf16x8*)(sm.k + (32 * jb + c) * PG + 16 * s + 8 * hf);
        kk = mfma32(*(const bf16x8*)(sm.k + (32 * ib + c) * PG + 16 * s + 8 * hf), kj, kk);
        qk = mfma32(*(const bf16x8*)(sm.q + (32 * ib + c) * PG + 16 * s + 8 * hf), kj, qk);
      }
      const int j = 32 * jb + c;
      const float gj = sm.gam[j];
      float col = 0.f;
      lds_barrier();                                     // dVb and the last slab have been read: dP scale D, dA beta D go there
      float g[16], ga[16];
#pragma unroll
      for (int r4 = 0; r4 < 4; r4++) {
        const int i4 = 32 * ib + 8 * r4 + 4 * hf;
        const f32x4 gi4 = *(const f32x4*)(sm.gam + i4), b4 = *(const f32x4*)(sm.bet + i4);
        f32x4 mp, ma;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int r = 4 * r4 + e, i = i4 + e;
          const float dec = j <= i ? __expf(gi4[e] - gj) : 0.f;
          const float vp = j <= i ? dp[r] : 0.f, va = j < i ? da[r] : 0.f;
          mp[e] = vp * (scale * dec);
          ma[e] = va * dec;
          ga[r] = ma[e] * (j < i ? kk[r] : 0.f);         // its row sums are the part of dbeta that comes through A
          ma[e] *= b4[e];
          g[r] = mp[e] * (j <= i ? qk[r] : 0.f) + b4[e] * ga[r];
          col += g[r];
        }
        *(bf16x4*)(sm.x + j * PK + i4) = cvt4(mp[0], mp[1], mp[2], mp[3]);
        *(bf16x4*)(sm.r2 + j * PK + i4) = cvt4(ma[0], ma[1], ma[2], ma[3]);
        __builtin_amdgcn_sched_barrier(0);
      }
      const float row_g = half_wave_sums(g, c), row_a = half_wave_sums(ga, c);
      if (c < 16) {
        sm.dg_row[jb][32 * ib + tile_row(c, hf)] = row_g;
        sm.db_a[jb][32 * ib + tile_row(c, hf)] = row_a;
      }
      col = half_swap_sum(col);
      if (hf == 0) sm.dg_col[ib][j] = col;
    }
    lds_barrier();

    // ---- 5. what is left of dq and dk (the 64 x 64 matrices are lower triangular) ----
    place();
    if (!SPLIT && r_h + 1 < rep) load_head(h + 1);
    float row_kb[2];
#pragma unroll
    for (int s = 0; s < GC / 16; s++) {
      const int k0 = 16 * s + 8 * hf;
      const bf16x8 b_k = kmajor_frag(sm.k, PG, k0, 32 * w + c16, lane);
      const bf16x8 b_q = kmajor_frag(sm.q, PG, k0, 32 * w + c16, lane);
#pragma unroll
      for (int t = 0; t < 2; t++) {
        if (s < 2 * t + 2) {                             // rows of block t: columns up to its diagonal
          dq[t] = mfma32(kmajor_frag(sm.x, PK, k0, 32 * t + c16, lane), b_k, dq[t]);
          dk[t] = mfma32(kmajor_frag(sm.r2, PK, k0, 32 * t + c16, lane), b_k, dk[t]);
        }
        if (s >= 2 * t) {                                // transposed
          dk[t] = mfma32(*(const bf16x8*)(sm.x + (32 * t + c) * PK + k0), b_q, dk[t]);
          dk[t] = mfma32(*(const bf16x8*)(sm.r2 + (32 * t + c) * PK + k0), b_k, dk[t]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    place();
#pragma unroll
    for (int t = 0; t < 2; t++) {
      float dot[16];
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const bf16x8 xf = kmajor_frag_acc_order(sm.x + X_KB, PG, 32 * t + 16 * u + 4 * hf, 32 * w + c16, lane);
        const bf16x8 kf = kmajor_frag_acc_order(sm.k, PG, 32 * t + 16 * u + 4 * hf, 32 * w + c16, lane);
#pragma unroll
        for (int v4 = 0; v4 < 2; v4++) {
          const int i4 = 32 * t + 16 * u + 8 * v4 + 4 * hf;
          const f32x4 b4 = *(const f32x4*)(sm.bet + i4), eg4 = *(const f32x4*)(sm.eg + i4);
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const float dkb = (float)xf[4 * v4 + e];
            dot[8 * u + 4 * v4 + e] = dkb * (float)kf[4 * v4 + e];
            dk[t][8 * u + 4 * v4 + e] += b4[e] * eg4[e] * dkb;
          }
        }
      }
      row_kb[t] = half_wave_sums(dot, c);
      __builtin_amdgcn_sched_barrier(0);
    }

    // ---- dg, dbeta ----
    float(*sum_qk)[GC] = (float(*)[GC])(sm.x + X_SUMS);  // per-wave parts of the row sums (a quarter of the columns each)
    float(*sum_kb)[GC] = sum_qk + 4, *part = &sum_qk[8][0];
    if (c < 16) {
#pragma unroll
      for (int t = 0; t < 2; t++) {
        sum_qk[w][32 * t + tile_row(c, hf)] = row_qk[t];
        sum_kb[w][32 * t + tile_row(c, hf)] = row_kb[t];
      }
    }
    // what goes through gamma_last: <dKd, Kd>, and exp(gamma_last) <dS1, S0> (it also scales the state that is carried over)
    float s_last = s_kd + el_last * s_dot;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s_last += __shfl_xor(s_last, d);
    if (lane == 0) part[w] = s_last;
    lds_barrier();
    if (tid < GC) {
      const float dkb = sm.eg[tid] * ((sum_kb[0][tid] + sum_kb[1][tid]) + (sum_kb[2][tid] + sum_kb[3][tid]));       // eg dKb_i . k_i
      float s = (sm.dg_row[0][tid] + sm.dg_row[1][tid]) - (sm.dg_col[0][tid] + sm.dg_col[1][tid]) +
                ((sum_qk[0][tid] + sum_qk[1][tid]) + (sum_qk[2][tid] + sum_qk[3][tid])) + sm.bet[tid] * dkb;
      // gamma_i = sum of g_j over j <= i: a sum over the rows from this one on; gamma_last reaches every g
#pragma unroll
      for (int d = 1; d < GC; d <<= 1) {
        const float down = __shfl_down(s, d);
        s += tid + d < GC ? down : 0.f;
      }
      const float last = (part[0] + part[1]) + (part[2] + part[3]);
      if (tid < len) {
        a.b.dg[(size_t)(tok0 + tid) * hv + h] = s + last;
        a.b.dbeta[(size_t)(tok0 + tid) * hv + h] = sm.db_a[0][tid] + sm.db_a[1][tid] + dkb + sm.db_v[tid];
      }
    }
  }

  place();
  if constexpr (SPLIT) {
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int i = 32 * t + tile_row(r, hf);
        const size_t at = ((size_t)(tok0 + i) * a.b.hv_n + unit) * GD + 32 * w + c;
        if (i < len) {
          a.w.dqh[at] = dq[t][r];
          a.w.dkh[at] = dk[t][r];
        }
      }
  } else {
    // through LDS, so that rows leave in 16-byte pieces
    lds_barrier();                                       // K and Q have been read
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int at = (32 * t + tile_row(r, hf)) * PG + 32 * w + c;
        sm.q[at] = (__bf16)dq[t][r];
        sm.k[at] = (__bf16)dk[t][r];
      }
    lds_barrier();
#pragma unroll
    for (int p = 0; p < 4; p++) {
      const int piece = tid + p * BT, i = piece >> 4, c8 = (piece & 15) * 8;
      const size_t at = (size_t)(tok0 + i) * qrow + (size_t)kh * GD + c8;
      if (i < len) {
        *(bf16x8*)((__bf16*)a.b.dq + at) = *(const bf16x8*)(sm.q + i * PG + c8);
        *(bf16x8*)((__bf16*)a.b.dk + at) = *(const bf16x8*)(sm.k + i * PG + c8);
      }
    }
  }
}

// dq, dk [N][hk][128] bf16 = sum over the value heads of a group of the per-head fp32 gradients
__global__ __launch_bounds__(BT) void gdn_bwd_group_sum_kernel(KArgs a) {
  const int rep = a.b.hv / a.b.hk, hk_n = a.b.hv_n / rep;          // key heads of this pass
  const size_t n4 = (size_t)a.b.n_tokens * hk_n * (GD / 4);
  for (size_t e = (size_t)blockIdx.x * BT + threadIdx.x; e < n4; e += (size_t)gridDim.x * BT) {
    const size_t t = e / ((size_t)hk_n * (GD / 4));
    const int rem = (int)(e % ((size_t)hk_n * (GD / 4))), kh = rem / (GD / 4), d4 = (rem % (GD / 4)) * 4;
    float4 sq = make_float4(0.f, 0.f, 0.f, 0.f), sk = sq;
    for (int r = 0; r < rep; r++) {
      const size_t src = ((size_t)t * a.b.hv_n + kh * rep + r) * GD + d4;
      const float4 x = ld4(a.w.dqh + src), y = ld4(a.w.dkh + src);
      sq.x += x.x; sq.y += x.y; sq.z += x.z; sq.w += x.w;
      sk.x += y.x; sk.y += y.y; sk.z += y.z; sk.w += y.w;
    }
    const size_t dst = ((size_t)t * a.b.hk + kh) * GD + d4;
    *(bf16x4*)((__bf16*)a.b.dq + dst) = cvt4(sq.x, sq.y, sq.z, sq.w);
    *(bf16x4*)((__bf16*)a.b.dk + dst) = cvt4(sk.x, sk.y, sk.z, sk.w);
  }
}

__global__ __launch_bounds__(BT) void gdn_bwd_fill_zero_kernel(float4* p, size_t n4) {
  for (size_t e = (size_t)blockIdx.x * BT + threadIdx.x; e < n4; e += (size_t)gridDim.x * BT) p[e] = make_float4(0.f, 0.f, 0.f, 0.f);
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// carves the workspace; returns the total size (with p == nullptr: only the size)
// (hv_n: value heads of one pass; the saved states and their gradients keep the tensors' head stride hv)
size_t carve(char* p, int64_t n_tokens, int n_chunks, int n_slots, int n_segments, int hv, int hv_n, bool split, BwdWs* w) {
  const size_t per = (size_t)n_chunks * hv_n;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* r = p ? p + off : nullptr;
    off += align256(bytes);
    return r;
  };
  BwdWs t{};
  t.ops.gam = (float*)take(per * GC * 4);
  t.ops.t = (float*)take(per * GDN_T_ELEMS * 4);
  t.sv.fwd_rec = take(per * GDN_REC_ELEMS * 2);
  t.sv.rev_rec = take(per * GDN_REV_ELEMS * 2);
  t.sv.glast = (float*)take(per * 4);
  t.sv.s0t = take(per * GD * GD * 2);
  t.sv.ds1t = take(per * GD * GD * 2);
  t.sv.vns = take(per * GC * GD * 2);
  t.sv.dvns = take(per * GC * GD * 2);
  t.sv.slots = (float*)take((size_t)n_slots * hv * GD * GD * 4);
  t.sv.slot_grad = (float*)take((size_t)n_slots * hv * GD * GD * 4);
  t.sv.seg_grad = (float*)take((size_t)n_segments * hv * GD * GD * 4);
  if (split) {
    t.dqh = (float*)take((size_t)n_tokens * hv_n * GD * 4);
    t.dkh = (float*)take((size_t)n_tokens * hv_n * GD * 4);
  }
  if (w) *w = t;
  return off + 256;
}

// One value head per workgroup of the finish kernel where a call has few (chunk, key head) pairs (the chip holds 512
// workgroups): there the value heads side by side are worth more than the fp32 dq / dk saved.  Whole backward, two value
// heads per key head, one by one / in one workgroup: 164 pairs 200 / 208 us, 328 pairs 221 / 225, 332 pairs (longer walk)
// 317 / 316, 408 pairs 279 / 265, 664 pairs 443 / 430, 1328 pairs 636 / 610.  The whole call decides, not the pass: results do not depend on how much workspace there is.
constexpr int64_t FINISH_SPLIT_BELOW = 384;
bool finish_split(int n_chunks, int hk, int hv) { return hv > hk && (int64_t)n_chunks * hk < FINISH_SPLIT_BELOW; }

}  // namespace

size_t gdn_bwd_workspace(int64_t n_tokens, int n_chunks, int n_slots, int n_segments, int hk, int hv, int key_heads_per_pass) {
  return carve(nullptr, n_tokens, n_chunks, n_slots, n_segments, hv, key_heads_per_pass * (hv / hk),
               finish_split(n_chunks, hk, hv), nullptr);
}

// The value heads are independent of each other up to the final sum over the value heads of a key head, so the
// pass can be cut into batches of whole key-head groups: as many per batch as the workspace holds.  A batch sees
// the tensors through pointers moved to its first head (the head counts stay the strides).
hipError_t gdn_bwd(const GdnBwdArgs& b0, hipStream_t st) {
  if (b0.n_chunks == 0 || b0.n_tokens == 0) return hipSuccess;
  const int rep = b0.hv / b0.hk, n_seg = b0.sched ? b0.sched->n_segments : 0;
  int per_pass = b0.hk;
  while (per_pass > 1 && gdn_bwd_workspace(b0.n_tokens, b0.n_chunks, b0.n_slots, n_seg, b0.hk, b0.hv, per_pass) > b0.workspace_bytes)
    per_pass--;
  if (gdn_bwd_workspace(b0.n_tokens, b0.n_chunks, b0.n_slots, n_seg, b0.hk, b0.hv, per_pass) > b0.workspace_bytes)
    return hipErrorInvalidValue;
  const bool split = finish_split(b0.n_chunks, b0.hk, b0.hv);
  auto zero = [&](float* p, size_t floats) {
    if (floats == 0) return;
    const size_t n4 = floats / 4;
    gdn_bwd_fill_zero_kernel<<<dim3((unsigned)std::min<size_t>((n4 + BT - 1) / BT, 4096)), BT, 0, st>>>((float4*)p, n4);
  };
  for (int kh0 = 0; kh0 < b0.hk; kh0 += per_pass) {
    const int hk_n = std::min(per_pass, b0.hk - kh0), h0 = kh0 * rep;
    GdnBwdArgs b = b0;
    b.hv_n = hk_n * rep;
    const size_t ko = (size_t)kh0 * GD, vo = (size_t)h0 * GD, so = (size_t)h0 * GD * GD;
    b.q = (const __bf16*)b0.q + ko; b.k = (const __bf16*)b0.k + ko; b.v = (const __bf16*)b0.v + vo; b.d_o = (const __bf16*)b0.d_o + vo;
    b.g = b0.g + h0; b.beta = b0.beta + h0;
    b.dq = (__bf16*)b0.dq + ko; b.dk = (__bf16*)b0.dk + ko; b.dv = (__bf16*)b0.dv + vo;
    b.dg = b0.dg + h0; b.dbeta = b0.dbeta + h0;
    if (b0.initial_state) b.initial_state = b0.initial_state + so;
    if (b0.d_state_out) b.d_state_out = b0.d_state_out + so;
    if (b0.d_initial_state) b.d_initial_state = b0.d_initial_state + so;
    KArgs a{};
    a.b = b;
    carve((char*)b.workspace, b.n_tokens, b.n_chunks, b.n_slots, n_seg, b.hv, b.hv_n, split, &a.w);
    // walking all chunks in sequence order, readers add into the slot gradients and into d_initial_state; with a
    // schedule every segment stores its own gradient and nothing has to start from zero
    if (!b.sched) {
      zero(a.w.sv.slot_grad, (size_t)b.n_slots * b.hv * GD * GD);
      if (b.d_initial_state) {
        // the rows of this pass's heads (one contiguous piece: heads are the outer index)
        zero(b.d_initial_state, (size_t)b.hv_n * GD * GD);
      }
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (hipError_t e = gdn_bwd_prepare_and_walks(b, a.w.ops, a.w.sv, st); e != hipSuccess) return e;
    {
      KernelTimer t(TT_KERNEL_GDN_BWD_FINISH, st);
      if (split) gdn_bwd_finish_kernel<true><<<gdn_group_order_grid(b.n_chunks, b.hv_n, rep), BT, 0, st>>>(a);
      else gdn_bwd_finish_kernel<false><<<gdn_group_order_grid(b.n_chunks, hk_n, 1), BT, 0, st>>>(a);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (split) {
      const size_t n4 = (size_t)b.n_tokens * hk_n * (GD / 4);
      gdn_bwd_group_sum_kernel<<<dim3((unsigned)std::min<size_t>((n4 + BT - 1) / BT, 8192)), BT, 0, st>>>(a);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tt
