// Gated delta rule with tree state routing, backward (Section "Implementation", paragraph "SSM Layers
// (GDN)" (i): gradients accumulate at the shared parent state; Appendix "Tree-Aware SSM State
// Routing").  Chunked like the forward (64 tokens, chunks never cross a node boundary).  With
//     R = beta V - beta eg (K S0),   Vn = T R,   O = scale eg (Q S0) + P Vn,   S1 = EL S0 + K^T (el Vn)
// (eg = exp(gamma), el = exp(gamma_last - gamma), EL = exp(gamma_last), row factors; T = (I + A)^-1, A = beta_i A0_ij,
// A0 = strictly-lower((k_i.k_j) D_ij), P = scale tril((q_i.k_j) D_ij), D_ij = exp(gamma_i - gamma_j)) the chain rule gives, per chunk,
//     dVn = P^T dO + el (K dS1)     dR = T^T dVn     dS0 = EL dS1 + Q^T (scale eg dO) - K^T (beta eg dR)          (serial part)
//     dQg = dO S0^T      dKd = Vn dS1^T      dKb = -dR S0^T      dP = tril(dO Vn^T)      dA = strictly-lower(-dR Vn^T)
// (the triangular solve's own gradient: dA = -T^T dVn Vn^T).  From there dq, dk, dv = beta dR, dbeta and dgamma by the product
// rule; dg is the reverse running sum of
// dgamma inside the chunk.  State routing backwards: dS1 of a chunk is the dS0 of the chunk that
// continued from it on chip plus the gradient collected in its saved-state slot (every chunk that
// started from the slot added its dS0 there; they all come later in DFS order, so a reverse walk over
// the chunks has seen them), plus the upstream gradient of a captured state.
//
// Kernels (the first three live in tt_gdn.hip with the forward's):
//   gdn_prepare_kernel<true>   per (chunk, key head): T, P transposed, row factors
//   gdn_fwalk_kernel           (value head, segment): the forward scan without its output; saves S0 and Vn of every chunk (bf16)
//   gdn_rwalk_kernel           (value head, segment): reverse walk in the forward scan's form; saves dS1 and dR (bf16)
//   gdn_bwd_finish_kernel      per (chunk, key head): everything else: products on the bf16 matrix instruction (fp32
//                              accumulation), element-wise work in fp32; dq / dk summed over the key head's value heads in registers
//   gdn_bwd_group_sum_kernel   calls with few chunks: sums fp32 dq / dk over the value heads, rounds to bf16
#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>
#include "tt_internal.h"
#include "tt_kernels.h"
#include "tt_mfma.h"

namespace tt {
namespace {

constexpr int GC = TT_GDN_CHUNK;     // 64
constexpr int GD = 128;
constexpr int BT = 256;              // threads of the small kernels
constexpr int FT = 512;              // of the finish kernel

struct BwdWs {
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
// One workgroup of eight waves per compute unit; it goes through its (chunk, key head) pairs, the value heads of a key head one after
// the other, and keeps dq and dk, which are sums over them, in accumulator registers (SPLIT: one value head each, dq /
// dk of every head in fp32 to memory, summed by gdn_bwd_group_sum_kernel).  What bounds it is memory: 128 KB of
// operands per (chunk, value head), each byte read once.  To that end
//   - everything that contracts over value columns is done while a slab of 32 of them is on chip: S0, dS1, Vn, dR, dO, V, 32 KB, copied
//     straight to LDS as the walks stored it; transposing reads give the operands
//         dQg = dO S0^T, dKb = -dR S0^T, dKd = Vn dS1^T, dP = dO Vn^T, dA = -dR Vn^T and <dS1, S0>
//   - three slabs are on chip: two on their way while one is worked on, across heads and pairs
// Then, per head: K K^T and Q K^T again (K and Q stay in LDS for all heads): row and column sums of dP o P + dA o A in
// registers, dP scale D and dA beta D as bf16 to LDS, and
//         dq += (dP scale D) K;  dk += (dP scale D)^T Q + (dA beta D) K + (dA beta D)^T K + beta eg dKb
// A wave's tile (tb, kb) of a 64 x 128 result: rows 32 tb .., columns 32 kb ..
// 16406 tokens, 16 / 32 heads: 0.40 ms at 1.45 GB (0.50 ms at 2.3 GB before, when dW went through the transposed solve and U, W and T
// were read for it).  A slab takes 2600 cycles of which 1000 are waits for memory, what follows the slabs of a head 9000.
constexpr int PK = GC + 8;                               // LDS pitch (elements) of the 64 x 64 matrices
constexpr int SLAB_B = 32 * 1024, N_SLOTS = 3;
constexpr int F_S0 = 0, F_DS1 = 8 * 1024, F_VN = 16 * 1024, F_DR = 20 * 1024, F_DO = 24 * 1024, F_V = 28 * 1024;
struct FinishSmem {
  unsigned char slab[N_SLOTS][SLAB_B];
  __bf16 k[GC * GD], q[GC * GD];                         // swizzled tiles; at a pair's end dk and dq on their way to memory
  __bf16 m1[GC * PK], m2[GC * PK];                       // dP scale D, dA beta D, column by column
  float row[2][5][GC];                                   // beta, beta eg, el, eg, gamma of this head and the next
  float dg_row[2][2][GC], dg_col[2][2][GC], db_a[2][GC]; // [dP / dA part][column / row block]
  float sum_qk[4][GC], sum_kb[4][GC], db_v[4][GC], part[8];
};
static_assert(sizeof(FinishSmem) <= 160 * 1024, "LDS of one compute unit");

// Barriers that wait for this wave's LDS traffic, and for its copies except the last n requests.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ __forceinline__ void copies_barrier() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory"); }

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

// a value that is the same for all lanes, by a scalar load (a vector load would be waited for with the copies in flight)
__device__ __forceinline__ int ld_uniform(const int32_t* p) { return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p; }
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

template <bool SPLIT>
__global__ __launch_bounds__(FT, 2) void gdn_bwd_finish_kernel(KArgs a) {
  __shared__ __attribute__((aligned(1024))) FinishSmem sm;
  const int nc = a.b.n_chunks, hv = a.b.hv, rep = hv / a.b.hk, n_r = SPLIT ? 1 : rep;
  const int items = nc * (SPLIT ? a.b.hv_n : a.b.hv_n / rep);
  const float scale = a.b.scale;
  const uint32_t qrow = (uint32_t)a.b.hk * (GD * 2), vrow = (uint32_t)hv * (GD * 2);      // bytes per token
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tb = w & 1, kb = w >> 1;
  // waves 0 .. 2: the lower tiles (0, 0), (1, 0), (1, 1) of dP;  3 .. 5: of dA
  const int part = w / 3, ib = (w % 3 + 1) >> 1, jb = (w % 3) >> 1;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&sm);

  // ---- copies ----
  // 32 pieces of a slab: wave w takes fragment w of S0 and of dS1, one of Vn or dR, one of dO or V (16 rows of 64 bytes, the
  // 16-byte chunks of a row permuted so that 16 rows read at the same chunk meet all banks).  Pointers move on by a slab; a new head's
  // are formed with its first one.
  int n_item = blockIdx.x, n_rh = 0, n_cb = 0, n_slot = 0, n_par = 0;      // the slab to request next
  if (n_item >= items) return;
  int n_chunk = n_item % nc, n_unit = n_item / nc, n_tok0 = ld_uniform(a.b.chunk_tok0 + n_chunk), n_len = ld_uniform(a.b.chunk_len + n_chunk);
  const char *p_s0 = nullptr, *p_ds1 = nullptr, *p_vn = nullptr, *p_do = nullptr;
  uint32_t do_at = 0;
  auto request = [&]() {
    if (n_item >= items) return;
    if (n_cb == 0) {
      const int h = SPLIT ? n_unit : n_unit * rep + n_rh;
      const size_t op = (size_t)h * nc + n_chunk;
      p_s0 = (const char*)a.w.sv.s0 + op * (GD * GD * 2) + 1024 * w;
      p_ds1 = (const char*)a.w.sv.ds1 + op * (GD * GD * 2) + 1024 * w;
      p_vn = (const char*)(w < 4 ? a.w.sv.vns : a.w.sv.drs) + op * (GC * GD * 2) + 1024 * (w & 3);
      p_do = (const char*)(w < 4 ? a.b.d_o : a.b.v) + (uint64_t)(uint32_t)n_tok0 * vrow + (size_t)h * (GD * 2);
      do_at = (uint32_t)min(16 * (w & 3) + (lane >> 2), n_len - 1) * vrow + 16u * (uint32_t)((lane & 3) ^ ((lane >> 4) & 3));
      const uint32_t rows = lds0 + (uint32_t)offsetof(FinishSmem, row) + 5 * GC * 4 * n_par;
      if (w == 0) dma16((const char*)a.w.sv.rec + (op * GDN_REC_ELEMS + GDN_REC_ROW) * 2, 16u * lane, rows);
      if (w == 1) dma4(a.w.sv.gam + op * GC, 4u * lane, rows + 4 * GC * 4);
    }
    const uint32_t dst = lds0 + (uint32_t)offsetof(FinishSmem, slab) + SLAB_B * n_slot + 1024 * w;
    dma16(p_s0, 16u * lane, dst + F_S0);
    dma16(p_ds1, 16u * lane, dst + F_DS1);
  };
  auto request_rest = [&]() {           // (between the products: a compute unit takes 64 bytes a cycle, and a wave waits for its turn)
    if (n_item >= items) return;
    const uint32_t dst = lds0 + (uint32_t)offsetof(FinishSmem, slab) + SLAB_B * n_slot + 1024 * w;
    dma16(p_vn, 16u * lane, dst + F_VN);
    dma16(p_do, do_at, dst + F_DO);
    p_s0 += 8192; p_ds1 += 8192; p_vn += 4096; p_do += 64;
    n_slot = n_slot == N_SLOTS - 1 ? 0 : n_slot + 1;
    if (++n_cb == 4) {
      n_cb = 0; n_par ^= 1;
      if (++n_rh == n_r) {
        n_rh = 0;
        n_item += gridDim.x;
        if (n_item < items) {
          n_chunk = n_item % nc; n_unit = n_item / nc;
          n_tok0 = ld_uniform(a.b.chunk_tok0 + n_chunk); n_len = ld_uniform(a.b.chunk_len + n_chunk);
        }
      }
    }
  };
  auto request_kq = [&](int kh, int tok0, int len) {
    const uint64_t at = (uint64_t)(uint32_t)tok0 * qrow + (size_t)kh * (GD * 2);
    int ln = lane;
    asm volatile("" : "+v"(ln));
    dma_tile64<8>((const char*)a.b.k + at, qrow, len, sm.k, w, ln);
    dma_tile64<8>((const char*)a.b.q + at, qrow, len, sm.q, w, ln);
  };

  // ---- LDS addresses ----
  const int c = lane & 31, hf = lane >> 5, i16 = lane & 15, gidx = (lane >> 4) & 1, q2 = i16 >> 2, qd = i16 & 3;
  const uint32_t slab0 = lds0 + (uint32_t)offsetof(FinishSmem, slab);
  // rows of dO / V as operands: token 32 blk + c, columns 16 s + 8 hf .. of the slab
  uint32_t a_row[2];
#pragma unroll
  for (int s = 0; s < 2; s++) a_row[s] = (uint32_t)(64 * c + 16 * ((2 * s + hf) ^ ((c >> 2) & 3)));
  // tokens as lanes, 8 value columns 16 s + 8 hf .. each, out of the column-wise fragments of Vn / dR (two reads x of 4)
  uint32_t a_tr[2], b_tr[2];
#pragma unroll
  for (int x = 0; x < 2; x++) {
    a_tr[x] = (uint32_t)(1024 * gidx + 512 * (qd & 1) + 16 * ((8 * hf + 4 * x + q2) ^ (4 * (qd & 1))) + 8 * (qd >> 1));
    // key dims as lanes, 8 value columns each, out of the fragments of S0 / dS1
    b_tr[x] = (uint32_t)(1024 * gidx + 512 * (qd >> 1) + 16 * ((8 * hf + 4 * x + q2) ^ (4 * (qd >> 1))) + 8 * (qd & 1)) + 2048u * kb;
  }
  int item = blockIdx.x, slot = 0, par = 0;
  request_kq(SPLIT ? n_unit / rep : n_unit, n_tok0, n_len);
  request(); request_rest();
  request(); request_rest();
  for (; item < items; item += gridDim.x) {
    const int chunk = item % nc, unit = item / nc, kh = SPLIT ? unit / rep : unit;
    const int tok0 = ld_uniform(a.b.chunk_tok0 + chunk), len = ld_uniform(a.b.chunk_len + chunk);
    f32x16 dq = zero16(), dk = zero16(), x = zero16();    // x: this wave's tile of Q K^T or K K^T
#pragma unroll 1
    for (int r_h = 0; r_h < n_r; r_h++) {
      const int h = SPLIT ? unit : kh * rep + r_h;
      const float(*row)[GC] = sm.row[par];
      // ---- 1. everything that contracts over value columns ----
      f32x16 dqg = zero16(), dkb = zero16(), dkd = zero16(), dm = zero16();      // dm: this wave's tile of dP or -dA
      float s_dot = 0.f, db = 0.f;      // this thread's part of <dS1, S0>;  of dR_i . v_i (token 32 tb + c)
#pragma unroll 1
      for (int cb = 0; cb < 4; cb++) {
        // this slab has landed (what was requested behind it may still be on its way), and every wave has left the one before
        // requested behind it: 4 pieces of the next slab, and 4 of K and Q behind a pair's third slab
        const bool kq = r_h == 0 && item != (int)blockIdx.x;
        if (kq && (cb == 1 || cb == 2)) copies_barrier<8>();
        else if (cb < 3 || r_h + 1 < n_r || item + (int)gridDim.x < items) copies_barrier<4>();
        else copies_barrier<0>();
        request();
        const uint32_t sl = slab0 + SLAB_B * slot;
        slot = slot == N_SLOTS - 1 ? 0 : slot + 1;
        const uint32_t at0 = sl + a_tr[0], at1 = sl + a_tr[1], bt0 = sl + b_tr[0], bt1 = sl + b_tr[1];
        bf16x8 d_o[2], dr[2], vn[2], s0[2], ds1[2], left[2], right[2];
#pragma unroll
        for (int s = 0; s < 2; s++) {
          d_o[s] = lds_b128(sl + a_row[s] + 2048 * tb, F_DO);
          s0[s] = lds_tr2(bt0, bt1, F_S0 + 256 * s);
          dr[s] = lds_tr2(at0 + 2048 * tb, at1 + 2048 * tb, F_DR + 256 * s);
          vn[s] = lds_tr2(at0 + 2048 * tb, at1 + 2048 * tb, F_VN + 256 * s);
          ds1[s] = lds_tr2(bt0, bt1, F_DS1 + 256 * s);
          left[s] = part == 0 ? lds_b128(sl + a_row[s] + 2048 * ib, F_DO) : lds_tr2(at0 + 2048 * ib, at1 + 2048 * ib, F_DR + 256 * s);
          right[s] = lds_tr2(at0 + 2048 * jb, at1 + 2048 * jb, F_VN + 256 * s);     // (waves 6, 7: not used)
        }
        fence();
#pragma unroll
        for (int s = 0; s < 2; s++) {
          dqg = mfma32(d_o[s], s0[s], dqg);
          dkb = mfma32(dr[s], s0[s], dkb);
          dkd = mfma32(vn[s], ds1[s], dkd);
          dm = mfma32(left[s], right[s], dm);
          if (s == 0) {
            request_rest();
            if (kq && cb == 0) request_kq(kh, tok0, len);     // (the previous pair's dq and dk have left their place)
          }
          fence();
        }
        {
          const uint32_t at = sl + 16u * threadIdx.x;
          const bf16x8 x = lds_b128(at, F_S0), y = lds_b128(at, F_DS1);
#pragma unroll
          for (int e = 0; e < 8; e++) s_dot += (float)x[e] * (float)y[e];
        }
        if ((kb >> 1) == (cb & 1)) {    // dv_i = beta_i dR_i of 16 columns
          const int s = kb & 1, i = 32 * tb + c;
          const bf16x8 dr_s = s ? dr[1] : dr[0], v = lds_b128(sl + (s ? a_row[1] : a_row[0]) + 2048 * tb, F_V);
          const float b = row[0][i];
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; e++) {
            x[e] = b * (float)dr_s[e];
            db += (float)dr_s[e] * (float)v[e];
          }
          if (i < len)
            *(bf16x8*)((char*)a.b.dv + (uint64_t)(uint32_t)tok0 * vrow + (size_t)h * (GD * 2) + (uint32_t)i * vrow + 64 * cb + 32 * s + 16 * hf) =
                cvt8(x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]);
        }
      }

      // Lane positions of the steps per head, from an opaque copy of the lane: their LDS and memory offsets are formed where they
      // are used; otherwise the compiler forms those of all steps in front of the loops and keeps them (72 spilled registers).
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const int c = ln & 31, hf = ln >> 5;
      // ---- 2. dq_i = scale eg_i dQg_i + ..;  dk_j = el_j dKd_j + beta eg_j dKb_j + ..;  their dot products with q_i and k_j go into dgamma ----
      float row_qk, row_kb, s_kd = 0.f;
      {
        float dot[16], dot_kb[16];
        const TrBase tr = tr_frag_base(ln);
        auto acc_frag = [&](const __bf16* tile, int r0) {       // 16 tokens in the order of accumulator registers, this wave's key dims
          return cat4(lds_read_tr(tile + r0 * GD + (tr.x0 ^ (kb << 5))), lds_read_tr(tile + r0 * GD + (tr.x1 ^ (kb << 5))));
        };
        bf16x8 qf[2], kf[2];
        f32x4 eg4[4], el4[4], beg4[4];
#pragma unroll
        for (int u = 0; u < 2; u++) { qf[u] = acc_frag(sm.q, 32 * tb + 16 * u); kf[u] = acc_frag(sm.k, 32 * tb + 16 * u); }
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++) {
          const int i4 = 32 * tb + 8 * r4 + 4 * hf;
          eg4[r4] = *(const f32x4*)&row[3][i4];
          el4[r4] = *(const f32x4*)&row[2][i4];
          beg4[r4] = *(const f32x4*)&row[1][i4];
        }
        fence();
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const float kv = (float)kf[r >> 3][r & 7], vq = scale * eg4[r >> 2][r & 3] * dqg[r], vk = el4[r >> 2][r & 3] * dkd[r], vkk = vk * kv;
          dot[r] = vq * (float)qf[r >> 3][r & 7] - vkk;
          dot_kb[r] = -dkb[r] * kv;
          s_kd += vkk;
          dq[r] += vq;
          dk[r] += vk - beg4[r >> 2][r & 3] * dkb[r];
        }
        row_qk = half_wave_sums(dot, c);
        row_kb = half_wave_sums(dot_kb, c);
      }
      // ---- 3. G = dP o P + dA o A: its row sums minus its column sums are the part of dgamma that comes through D ----
      auto through_d = [&](auto part_, auto diag_) {
        constexpr int part = decltype(part_)::value;
        constexpr bool DIAG = decltype(diag_)::value;
        if (r_h == 0) {
          const __bf16* left = part == 0 ? sm.q : sm.k;
          const int rd = row_frag_base(ln);
          bf16x8 fa[4], fb[4];
#pragma unroll
          for (int s = 0; s < 4; s++) { fa[s] = lds_row_frag(left, rd, ib, s); fb[s] = lds_row_frag(sm.k, rd, jb, s); }
          fence();
#pragma unroll
          for (int s = 0; s < GD / 16; s++) {
            x = mfma32(fa[s & 3], fb[s & 3], x);
            if (s + 4 < GD / 16) { fa[s & 3] = lds_row_frag(left, rd, ib, s + 4); fb[s & 3] = lds_row_frag(sm.k, rd, jb, s + 4); }
            fence();
          }
        }
        const int j = 32 * jb + c;
        const float gj = row[4][j];
        if (part == 0 && len < GC) {    // rows of dO past the chunk's length are copies of its last row
#pragma unroll
          for (int r = 0; r < 16; r++) dm[r] = 32 * ib + tile_row(r, hf) < len ? dm[r] : 0.f;
        }
        float col = 0.f, g[16], ga[16];
        __bf16* const m = part == 0 ? sm.m1 : sm.m2;
        f32x4 gi[2], bi[2];
        auto read = [&](int r4) {
          gi[r4 & 1] = *(const f32x4*)&row[4][32 * ib + 8 * r4 + 4 * hf];
          bi[r4 & 1] = *(const f32x4*)&row[0][32 * ib + 8 * r4 + 4 * hf];
        };
        read(0);
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++) {
          const int i4 = 32 * ib + 8 * r4 + 4 * hf;
          const f32x4 gi4 = gi[r4 & 1], b4 = bi[r4 & 1];
          if (r4 < 3) read(r4 + 1);
          const int below = 8 * r4 + 4 * hf - c;      // i - j of the group's first row, inside a diagonal tile
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const int r = 4 * r4 + e;
            float dec = fast_exp2((gi4[e] - gj) * LOG2E_F);
            if (DIAG) dec = below + e >= part ? dec : 0.f;       // dP: j <= i, dA: j < i
            if (part == 0) {
              v[e] = dm[r] * (scale * dec);
              g[r] = v[e] * x[r];
            } else {
              const float ma = -dm[r] * dec;
              ga[r] = ma * x[r];        // its row sums are the part of dbeta that comes through A
              v[e] = ma * b4[e];
              g[r] = b4[e] * ga[r];
            }
            col += g[r];
          }
          *(bf16x4*)(m + j * PK + i4) = cvt4(v[0], v[1], v[2], v[3]);
          fence();
        }
        const float row_g = half_wave_sums(g, c);
        if (c < 16) sm.dg_row[part][jb][32 * ib + tile_row(c, hf)] = row_g;
        if (part == 1) {
          const float row_a = half_wave_sums(ga, c);
          if (c < 16) sm.db_a[jb][32 * ib + tile_row(c, hf)] = row_a;
        }
        col = half_swap_sum(col);
        if (hf == 0) sm.dg_col[part][ib][j] = col;
        if (DIAG && ib == 0) {          // the upper right tile is zero: nobody forms its sums
          if (hf == 0) sm.dg_row[part][1][c] = 0.f;
          if (hf == 1) sm.dg_col[part][0][32 + c] = 0.f;
          if (part == 1 && hf == 0) sm.db_a[1][c] = 0.f;
        }
      };
      if (w == 1) through_d(std::integral_constant<int, 0>{}, std::false_type{});
      else if (w < 3) through_d(std::integral_constant<int, 0>{}, std::true_type{});
      else if (w == 4) through_d(std::integral_constant<int, 1>{}, std::false_type{});
      else if (w < 6) through_d(std::integral_constant<int, 1>{}, std::true_type{});
      if (c < 16) {
        sm.sum_qk[kb][32 * tb + tile_row(c, hf)] = row_qk;
        sm.sum_kb[kb][32 * tb + tile_row(c, hf)] = row_kb;
      }
      db = half_swap_sum(db);
      if (hf == 0) sm.db_v[kb][32 * tb + c] = db;
      // what goes through gamma_last: <dKd, Kd>, and exp(gamma_last) <dS1, S0> (it also scales the state that is carried over)
      float s_last = s_kd + row[3][GC - 1] * s_dot;
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) s_last += __shfl_xor(s_last, d);
      if (ln == 0) sm.part[w] = s_last;
      lds_barrier();

      // ---- 4. what is left of dq and dk (the 64 x 64 matrices are lower triangular) ----
      // K / Q: 8 consecutive tokens per half of the wave, this wave's key dims as lanes
      const int l16 = ln & 15, chunk16 = 4 * kb + 2 * ((ln >> 4) & 1) + ((l16 & 3) >> 1);
      int nat[2];
#pragma unroll
      for (int x = 0; x < 2; x++)
        nat[x] = (8 * hf + 4 * x + (l16 >> 2)) * GD + ((chunk16 ^ (((l16 >> 2) << 2) | ((2 * hf + x) & 3))) << 3) + 4 * (l16 & 1);
      auto nat_frag = [&](const __bf16* tile, int s) { return cat4(lds_read_tr(tile + 16 * s * GD + nat[0]), lds_read_tr(tile + 16 * s * GD + nat[1])); };
      // rows of block tb: columns up to its diagonal (s < 2 tb + 2), and transposed (s >= 2 tb)
      auto below = [&](const __bf16* m, int s) { return kmajor_frag(m, PK, 16 * s + 8 * hf, 32 * tb + 16 * (c >> 4), ln); };
      auto across = [&](const __bf16* m, int s) { return *(const bf16x8*)(m + (32 * tb + c) * PK + 16 * s + 8 * hf); };
      auto rest = [&](auto tb_) {
        constexpr int TB = decltype(tb_)::value;
        bf16x8 fk[2], fq[2], f1[2], f2[2], t1[2], t2[2];
        auto read = [&](int s) {
          const int u = s & 1;
          fk[u] = nat_frag(sm.k, s);
          if (s < 2 * TB + 2) { f1[u] = below(sm.m1, s); f2[u] = below(sm.m2, s); }
          if (s >= 2 * TB) { fq[u] = nat_frag(sm.q, s); t1[u] = across(sm.m1, s); t2[u] = across(sm.m2, s); }
        };
        read(0);
#pragma unroll
        for (int s = 0; s < GC / 16; s++) {
          const int u = s & 1;
          if (s + 1 < GC / 16) read(s + 1);
          fence();
          if (s < 2 * TB + 2) { dq = mfma32(f1[u], fk[u], dq); dk = mfma32(f2[u], fk[u], dk); }
          if (s >= 2 * TB) { dk = mfma32(t1[u], fq[u], dk); dk = mfma32(t2[u], fk[u], dk); }
          fence();
        }
      };
      if (tb == 0) rest(std::integral_constant<int, 0>{});
      else rest(std::integral_constant<int, 1>{});
      // ---- dg, dbeta ----
      if (w == 7) {
        const int t = ln;
        const float dkb_k = row[3][t] * ((sm.sum_kb[0][t] + sm.sum_kb[1][t]) + (sm.sum_kb[2][t] + sm.sum_kb[3][t]));       // eg dKb_i . k_i
        float s = (sm.dg_row[0][0][t] + sm.dg_row[0][1][t]) + (sm.dg_row[1][0][t] + sm.dg_row[1][1][t]) -
                  ((sm.dg_col[0][0][t] + sm.dg_col[0][1][t]) + (sm.dg_col[1][0][t] + sm.dg_col[1][1][t])) +
                  ((sm.sum_qk[0][t] + sm.sum_qk[1][t]) + (sm.sum_qk[2][t] + sm.sum_qk[3][t])) + row[0][t] * dkb_k;
        s = t < len ? s : 0.f;
        // gamma_i = sum of g_j over j <= i: a sum over the rows from this one on; gamma_last reaches every g
#pragma unroll
        for (int d = 1; d < GC; d <<= 1) {
          const float down = __shfl_down(s, d);
          s += t + d < GC ? down : 0.f;
        }
        const float last = ((sm.part[0] + sm.part[1]) + (sm.part[2] + sm.part[3])) + ((sm.part[4] + sm.part[5]) + (sm.part[6] + sm.part[7]));
        if (t < len) {
          a.b.dg[(size_t)(tok0 + t) * hv + h] = s + last;
          a.b.dbeta[(size_t)(tok0 + t) * hv + h] =
              sm.db_a[0][t] + sm.db_a[1][t] + dkb_k + ((sm.db_v[0][t] + sm.db_v[1][t]) + (sm.db_v[2][t] + sm.db_v[3][t]));
        }
      }
      par ^= 1;
    }

    // ---- the pair's dq and dk ----
    int ln = lane;                      // (opaque, as above)
    asm volatile("" : "+v"(ln));
    const int c = ln & 31, hf = ln >> 5;
    if constexpr (SPLIT) {
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int i = 32 * tb + tile_row(r, hf);
        const size_t at = ((size_t)(tok0 + i) * a.b.hv_n + unit) * GD + 32 * kb + c;
        if (i < len) {
          a.w.dqh[at] = dq[r];
          a.w.dkh[at] = dk[r];
        }
      }
    } else {
      // through LDS, so that rows leave in 16-byte pieces
      lds_barrier();                    // K and Q have been read
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int at = (32 * tb + tile_row(r, hf)) * GD + 32 * kb + c;
        sm.q[at] = (__bf16)dq[r];
        sm.k[at] = (__bf16)dk[r];
      }
      lds_barrier();
#pragma unroll
      for (int p = 0; p < 2; p++) {
        const int piece = 64 * w + ln + p * FT, i = piece >> 4, c8 = (piece & 15) * 8;
        const uint64_t at = (uint64_t)(uint32_t)(tok0 + i) * qrow + (size_t)kh * (GD * 2) + c8 * 2;
        if (i < len) {
          *(bf16x8*)((char*)a.b.dq + at) = *(const bf16x8*)(sm.q + i * GD + c8);
          *(bf16x8*)((char*)a.b.dk + at) = *(const bf16x8*)(sm.k + i * GD + c8);
        }
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
  t.sv.gam = (float*)take(per * GC * 4);
  t.sv.rec = take(per * GDN_REC_ELEMS * 2);
  t.sv.s0 = take(per * GD * GD * 2);
  t.sv.ds1 = take(per * GD * GD * 2);
  t.sv.vns = take(per * GC * GD * 2);
  t.sv.drs = take(per * GC * GD * 2);
  t.sv.slots = (float*)take((size_t)n_slots * hv * GD * GD * 4);
  t.sv.slot_grad = (float*)take((size_t)n_slots * hv * GD * GD * 4);
  t.sv.seg_grad = (float*)take((size_t)n_segments * hv * GD * GD * 4);
  t.sv.sync = take((size_t)(n_slots + n_segments) * hv_n * 16);
  if (split) {
    t.dqh = (float*)take((size_t)n_tokens * hv_n * GD * 4);
    t.dkh = (float*)take((size_t)n_tokens * hv_n * GD * 4);
  }
  if (w) *w = t;
  return off + 256;
}

// One value head per workgroup of the finish kernel where a call has so few (chunk, key head) pairs that two value heads each have a
// compute unit of their own (the kernel holds one): beyond that the fp32 dq / dk, written and read again, cost more than a shorter last round
// saves.  Whole backward, value heads one by one / in one workgroup, two value heads per key head: 74 pairs 99 / 103 us, 115 125 / 127, 140
// 148 / 141, 237 211 / 200, 280 157.5 / 154.5, 366 202 / 193, 504 195 / 170, 1076 411 / 355;  three: 180 149 / 136, 280 195 / 193;  four: 74
// 121 / 128, 115 148 / 153, 140 173 / 167, 345 258 / 227.  The whole call decides, not the pass: results do not depend on how much
// workspace there is.
constexpr int64_t FINISH_SPLIT_BELOW = 128;
bool finish_split(int n_chunks, int hk, int hv) { return hv > hk && (int64_t)n_chunks * hk < FINISH_SPLIT_BELOW; }

}  // namespace

// What carve takes, at most: 118 KB per (chunk, value head), the states, and the words that the walks synchronise with counted for as
// many slots and segments as there are chunks (a program has no more), so that a segment adds its gradient and nothing else.
// (It was 209156 bytes per chunk and head, what the call took when the walks' operands were stored in full: 0.8 GB of 1.9 at 16406
// tokens of 16 / 32 heads were never touched.)
size_t gdn_bwd_workspace(int64_t n_tokens, int n_chunks, int n_slots, int n_segments, int hk, int hv, int key_heads_per_pass) {
  constexpr size_t PER_CHUNK = GC * 4 + GDN_REC_ELEMS * 2 + 4 * GD * GD + 4 * GC * GD;
  const int hv_n = key_heads_per_pass * (hv / hk);
  const size_t arrays = 16 * 256;
  const size_t sync = ((size_t)n_chunks + std::max(n_chunks, n_slots)) * hv_n * 16;
  const size_t states = (size_t)(2 * (size_t)n_slots + n_segments) * hv * GD * GD * 4;
  return align256((size_t)n_chunks * hv_n * PER_CHUNK + sync) + states + (finish_split(n_chunks, hk, hv) ? 2 * align256((size_t)n_tokens * hv_n * GD * 4) : 0) + arrays;
}

// The value heads are independent of each other up to the final sum over the value heads of a key head, so the
// pass can be cut into batches of whole key-head groups: as many per batch as the workspace holds.  A batch sees
// the tensors through pointers moved to its first head (the head counts stay the strides).
hipError_t gdn_bwd(const GdnBwdArgs& b0, hipStream_t st) {
  if (b0.n_chunks == 0 || b0.n_tokens == 0) return hipSuccess;
  const int rep = b0.hv / b0.hk, n_seg = b0.sched ? b0.sched->n_segments : 0;
  const bool split = finish_split(b0.n_chunks, b0.hk, b0.hv);
  auto used = [&](int key_heads) { return carve(nullptr, b0.n_tokens, b0.n_chunks, b0.n_slots, n_seg, b0.hv, key_heads * rep, split, nullptr); };
  int per_pass = b0.hk;
  while (per_pass > 1 && used(per_pass) > b0.workspace_bytes) per_pass--;
  if (used(per_pass) > b0.workspace_bytes) return hipErrorInvalidValue;
  int dev = 0, n_cu = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
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
    if (hipError_t e = gdn_bwd_prepare_and_walks(b, a.w.sv, st); e != hipSuccess) return e;
    {
      KernelTimer t(TT_KERNEL_GDN_BWD_FINISH, st);
      const int64_t items = (int64_t)b.n_chunks * (split ? b.hv_n : hk_n);
      const unsigned grid = (unsigned)std::min<int64_t>(items, n_cu);
      if (split) gdn_bwd_finish_kernel<true><<<grid, FT, 0, st>>>(a);
      else gdn_bwd_finish_kernel<false><<<grid, FT, 0, st>>>(a);
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
