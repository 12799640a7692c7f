// Gated delta rule with tree state routing: the forward, and the walks of the backward (Section "Implementation",
// paragraph "SSM Layers (GDN)" (i); Appendix "Tree-Aware SSM State Routing"): the recurrent state at a node's first token
// is the end state of its parent node, not of the previous node in DFS order.
//
// Chunked form, 64 tokens per chunk, chunks never cross a node boundary.  With gamma_i the running
// sum of the log-decays inside a chunk, beta the write strengths and S0 the state entering the chunk:
//     A  = strictly-lower( beta_i (k_i . k_j) exp(gamma_i - gamma_j) ),      T = (I + A)^-1
//     P  = scale tril( (q_i . k_j) exp(gamma_i - gamma_j) )
//     R  = beta * V - (beta exp(gamma)) * (K S0)                             (rows scaled)
//     Vn = T R
//     O  = (scale exp(gamma)) * (Q S0) + P Vn
//     S1 = exp(gamma_last) S0 + K^T (exp(gamma_last - gamma) * Vn)
// which is the token recurrence  S <- e^g S + beta k (v - (e^g S)^T k)^T,  o = scale S^T q  written
// per chunk.  The raw rows of Q, K and V are the operands; all that is formed in advance per chunk and value head are two
// lower triangular 64 x 64 matrices and the row factors, 19 KB.  Two kernels:
//   gdn_prepare_kernel  (chunk, key head): K K^T and Q K^T on MFMA once for all value heads of the key head; per value head
//       the inverse T by blocks (one wave, one lane per row, no synchronisation inside) and the decayed Q K^T, written
//       as the fragments the scan's matrix instructions take
//   gdn_scan_kernel  (value head, segment of the chunk program): walks the chunks with the state in MFMA accumulators; the
//       columns of S evolve independently, so a wave holds 32 value columns of the whole state and depends on no other wave;
//       state routing = where a chunk takes S0 from (registers when it continues the previous chunk's sequence, a saved
//       node-end state, or the initial state)
// The backward (tt_gdn_bwd.hip) uses the prepare kernel with P transposed, gdn_fwalk_kernel, the scan without its output that saves
// S0 and Vn of every chunk, and gdn_rwalk_kernel, the reverse walk:
//     dVn = P^T dO + exp(gamma_last - gamma) * (K dS1),      dR = T^T dVn
//     dS0 = exp(gamma_last) dS1 + Q^T (scale exp(gamma) * dO) - K^T (beta exp(gamma) * dR)
#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>
#include "tt_gdn_order.h"
#include "tt_internal.h"
#include "tt_kernels.h"
#include "tt_mfma.h"

namespace tt {
namespace {

constexpr int GC = TT_GDN_CHUNK;     // tokens per chunk (64)
constexpr int GD = 128;              // head dim of keys and values
constexpr int G_THREADS = 256;

// Record of one (value head, chunk), records ordered head-major: a walk streams through memory front to back.  A 64 x 64 lower
// triangular matrix is six fragments of 32 rows x 16 columns (1 KB, 16 bytes per lane: lane = row, half hf and element e
// = column 4 hf + 8 (e / 4) + e % 4), row block 0 first: (0, 0), (0, 1), (1, 0) .. (1, 3).  P is stored transposed in the backward:
// (0, 0) .. (0, 3), (1, 2), (1, 3).  The pieces of T's fragments are permuted (t_piece), so that the reverse walk's transposing reads, which
// take 4 rows of both column halves of two fragments at once, meet every LDS bank once (as they stood, four times).
constexpr int FRAG = 512;                                        // bf16 elements of a fragment
constexpr int REC_THI = 0, REC_TLO = 6 * FRAG;                   // T - I as two bf16 halves (relative error 2^-17)
constexpr int REC_ROW = 12 * FRAG;                               // fp32 rows of 64: beta, beta exp(gamma), exp(gamma_last - gamma), exp(gamma)
constexpr int REC_P = REC_ROW + 2 * 4 * GC;
constexpr int REC_ELEMS = REC_P + 6 * FRAG;                      // 19 KB
__device__ __forceinline__ int t_piece(int lane, int f) { return lane ^ (lane >> 5 << 2) ^ ((f & 1) << 3); }
static_assert(REC_ELEMS == GDN_REC_ELEMS && REC_ROW == GDN_REC_ROW && REC_ELEMS * 2 == 19 * 1024, "whole 1 KB pieces; shared with the finish kernel");

// What scheduled walks synchronise with, per value head and saved state, or gradient of a segment: whether the waves that hold its four
// blocks of columns have stored it; and, in those of state 0 and segment 0, how many workgroups of a column of the grid have started
// (a head has one column, or two).  16 bytes each: hundreds of waves look at the flags of one state, and with 4 bytes for a head, all
// heads in one line of memory, the forward walks took 6 us longer (16406 tokens of 16 / 32 heads).
struct WalkSync {
  uint8_t stored[4];
  int started[2], unused;
};
static_assert(sizeof(WalkSync) == 16, "as the workspaces count them");

constexpr int WALK_LEVELS = 32;
struct GdnArgs {
  int hk, hv, n_chunks;              // hk, hv: heads of the tensors (their strides)
  int hk_n;                          // key heads this launch works on, with their value heads (0 .. relative to the pointers below)
  float scale;
  const __bf16 *q, *k, *v;           // [N][hk][128], [N][hk][128], [N][hv][128]
  const float *g, *beta;             // [N][hv]
  const int32_t *chunk_tok0, *chunk_len, *chunk_src, *chunk_dst;
  const int32_t* chunk_cap;          // nullptr, or per chunk: -1 / index into state_out
  const int32_t *seg_chunk0, *seg_chunk1;   // nullptr (one segment: all chunks), or the chunk ranges of the segments
  int seg_base, n_segments;          // place of this launch's first workgroups (blockIdx.y counts from it), segments in all
  int n_levels, level_off[WALK_LEVELS + 1];       // reverse walk: the levels' first segments, or n_levels = 0 (more than WALK_LEVELS)
  int hv_n;                          // value heads of this launch
  WalkSync *slot_sync, *seg_sync;    // scheduled walks: [n_slots][hv_n], [n_segments][hv_n] behind it
  int n_sync;                        // cleared by the prepare kernel, from slot_sync on
  WalkSync* tickets;                 // nullptr (no segment waits for another), or whose `started` this walk counts in
  int max_polls;                     // after which a wait gives up
  const float* initial_state;        // nullptr (zero) or [hv][128][128]: the state roots start from
  float* state_out;                  // [n_capture][hv][128][128]
  __bf16* o;                         // [N][hv][128]
  __bf16* rec;                       // [hv][n_chunks][REC_ELEMS]
  float* slots;                      // [n_slots][hv][128][128] saved node-end states
  // backward only
  GdnBwdSaved sv;
  const __bf16* d_o;                 // [N][hv][128]
  const int32_t *slot_cons_off, *slot_cons;   // scheduled walk: the segments that start from every slot
  const float* d_state_out;          // nullptr or [n_capture][hv][128][128]
  float* d_initial_state;            // nullptr or [hv][128][128]
};
__device__ __forceinline__ size_t op_index(const GdnArgs& a, int chunk, int h) { return (size_t)h * a.n_chunks + chunk; }

// register pair (x, y) of two half-waves -> (x.lo, y.lo), (x.hi, y.hi)
__device__ __forceinline__ void swap32(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

// ---- prepare kernel ------------------------------------------------------------------------------------
constexpr int AT_PITCH = GC + 4;     // LDS row (floats) of A^T: rows 16-byte aligned
constexpr int PREP_HEADS = 2;        // value heads worked on side by side (one wave each forms its inverse)
struct PrepSmem {
  union {
    struct { __bf16 k[GC * GD], q[GC * GD]; };                   // swizzled tiles; free once the products are in registers
    float at[PREP_HEADS][GC][AT_PITCH];                          // A^T (row = column of A)
  };
  float gam[PREP_HEADS][GC], bet[PREP_HEADS][GC];
};

// What bounds it: the chain tile copy -> products -> A -> inverse (31 dependent steps of one wave) of a workgroup, three
// workgroups per compute unit, and 0.3 GB of traffic at 16406 tokens of 16 / 32 heads: 92 us.  (It was 230 us with one workgroup per
// value head that also formed the products of the inverse with V and K and wrote them, and the decayed Q and K, 72 KB per
// chunk and head instead of 19.)
// BWD: P transposed, and gamma itself for the finish kernel.
template <bool BWD>
__global__ __launch_bounds__(G_THREADS, 3) void gdn_prepare_kernel(GdnArgs a) {
  __shared__ __attribute__((aligned(1024))) PrepSmem sm;
  for (int i = (int)blockIdx.x * G_THREADS + (int)threadIdx.x; i < a.n_sync; i += (int)gridDim.x * G_THREADS) a.slot_sync[i] = WalkSync{};
  const int rep = a.hv / a.hk;
  const int chunk = (int)blockIdx.x % a.n_chunks, kh = (int)blockIdx.x / a.n_chunks;
  const int lane = threadIdx.x & 63, c = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tok0 = a.chunk_tok0[chunk], len = a.chunk_len[chunk];

  // rows past the chunk's length repeat its last row: their beta is 0, so their rows of A are 0 and those of T are unit rows
  const size_t krow = (size_t)tok0 * a.hk + kh;
  dma_tile64(a.k + krow * GD, (uint32_t)a.hk * GD * 2, len, sm.k, w, lane);
  dma_tile64(a.q + krow * GD, (uint32_t)a.hk * GD * 2, len, sm.q, w, lane);

  // waves 2 and 3: the row factors of one value head each (lane = token; gamma by a scan over the lanes)
  auto row_factors = [&](int r0) {
    const int hh = w - 2, h = kh * rep + r0 + hh;
    if (w < 2 || r0 + hh >= rep) return;
    const bool in = lane < len;
    const size_t at = (size_t)(tok0 + min(lane, len - 1)) * a.hv + h;
    float run = a.g[at], b = a.beta[at];
    run = in ? run : 0.f;
    b = in ? b : 0.f;
#pragma unroll
    for (int d = 1; d < GC; d <<= 1) {
      const float up = __shfl_up(run, d);
      if (lane >= d) run += up;
    }
    sm.gam[hh][lane] = run;
    sm.bet[hh][lane] = b;
    const float eg = __expf(run);
    float* row = (float*)(a.rec + op_index(a, chunk, h) * REC_ELEMS + REC_ROW) + lane;
    row[0] = b;
    row[GC] = b * eg;
    row[2 * GC] = __expf(__shfl(run, GC - 1) - run);
    row[3 * GC] = eg;
    if constexpr (BWD) a.sv.gam[op_index(a, chunk, h) * GC + lane] = run;
  };
  row_factors(0);
  dma_wait_all();
  __syncthreads();

  // K K^T and Q K^T, one 32 x 32 tile of the lower triangle per wave (wave 3: none): rows = j, columns (lanes) = i; Q K^T in the
  // backward: rows = i, columns = j
  const int ib = (w + 1) >> 1, jb = w >> 1;
  f32x16 kk = zero16(), qk = zero16();
  if (w < 3) {
    const int base = row_frag_base(lane);
#pragma unroll
    for (int ks = 0; ks < GD / 16; ks++) {
      const bf16x8 kj = lds_row_frag(sm.k, base, jb, ks);
      kk = mfma32(kj, lds_row_frag(sm.k, base, ib, ks), kk);
      const bf16x8 qi = lds_row_frag(sm.q, base, ib, ks);
      qk = BWD ? mfma32(qi, kj, qk) : mfma32(kj, qi, qk);
    }
  }
  for (int r0 = 0; r0 < rep; r0 += PREP_HEADS) {
    __syncthreads();                    // K and Q (or the previous heads' A) have been read, the row factors are there
    if (w < 3) {
      const int i = 32 * ib + c;
#pragma unroll
      for (int hh = 0; hh < PREP_HEADS; hh++) {
        if (r0 + hh >= rep) break;
        const float gi = sm.gam[hh][i], bi = sm.bet[hh][i];
        [[maybe_unused]] const float gc = sm.gam[hh][32 * jb + c];
        float p[16];
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++) {
          const int j4 = 32 * jb + 8 * r4 + 4 * hf;
          const f32x4 gj = *(const f32x4*)&sm.gam[hh][j4];
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const int j = j4 + e, r = 4 * r4 + e;
            const float dec = j <= i ? __expf(gi - gj[e]) : 0.f;
            sm.at[hh][j][i] = j < i ? bi * (kk[r] * dec) : 0.f;
            if constexpr (!BWD) p[r] = j <= i ? a.scale * qk[r] * dec : 0.f;
          }
          if constexpr (BWD) {
            const int i4 = 32 * ib + 8 * r4 + 4 * hf;
            const f32x4 gr = *(const f32x4*)&sm.gam[hh][i4];
#pragma unroll
            for (int e = 0; e < 4; e++) p[4 * r4 + e] = 32 * jb + c <= i4 + e ? a.scale * qk[4 * r4 + e] * __expf(gr[e] - gc) : 0.f;
          }
        }
        // fragments (ib, 2 jb), (ib, 2 jb + 1) of P, or (jb, 2 ib), (jb, 2 ib + 1) of its transpose: the accumulator's registers as they stand
        const int f = BWD ? (jb == 0 ? 2 * ib : 4) : 2 * ib + 2 * jb;
        __bf16* out = a.rec + op_index(a, chunk, kh * rep + r0 + hh) * REC_ELEMS + REC_P + f * FRAG + 8 * lane;
        *(bf16x8*)out = cvt8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
        *(bf16x8*)(out + FRAG) = cvt8(p[8], p[9], p[10], p[11], p[12], p[13], p[14], p[15]);
      }
    }
    __syncthreads();
    // T = (I + A)^-1 by 32 x 32 blocks, T = [T11 0; T21 T22]: the diagonal blocks by substitution on T (I + A) = I, one lane
    // per row (column j from columns j + 1 .. on), both blocks at once in the two halves of the wave; then
    // T21 = -T22 A21 T11 as two products on the fp32 matrix instruction.  One wave per value head; which wave it is differs
    // from workgroup to workgroup (the waves of a workgroup sit on different SIMDs).
    const int hh = (w - (int)(blockIdx.x >> 3) * PREP_HEADS) & 3;
    if (hh < PREP_HEADS && r0 + hh < rep) {
      float(*at)[AT_PITCH] = sm.at[hh];
      const float* ablk = &at[32 * hf][32 * hf];
      float x[32];
#pragma unroll
      for (int j = 0; j < 32; j++) x[j] = j == c ? 1.f : 0.f;
#pragma unroll
      for (int j = 30; j >= 0; j--) {
        // four partial sums (the chain of one sum would leave the wave waiting); A^T is zero at k <= j
        float s0 = x[j], s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
        for (int k4 = (j + 1) / 4; k4 < 8; k4++) {
          const float4 av = *(const float4*)(ablk + j * AT_PITCH + k4 * 4);
          s0 -= av.x * x[4 * k4];
          s1 -= av.y * x[4 * k4 + 1];
          s2 -= av.z * x[4 * k4 + 2];
          s3 -= av.w * x[4 * k4 + 3];
        }
        x[j] = (s0 + s1) + (s2 + s3);
      }
      // T11 for the second product, into the lower left block of A^T, which nothing reads
      if (!hf) {
#pragma unroll
        for (int j4 = 0; j4 < 8; j4++) *(float4*)&at[32 + c][4 * j4] = make_float4(x[4 * j4], x[4 * j4 + 1], x[4 * j4 + 2], x[4 * j4 + 3]);
      }
      // Y^T = (T22 A21)^T: step s contracts m = 2 s (lower half of the wave) and 2 s + 1 (upper half)
      f32x16 y = zero16();
#pragma unroll
      for (int s = 0; s < 16; s++) {
        float t0 = x[2 * s], t1 = x[2 * s + 1];
        swap32(t0, t1);                                           // t1: row c of T22, column 2 s + hf
        y = __builtin_amdgcn_mfma_f32_32x32x2f32(at[c][32 + 2 * s + hf], t1, y, 0, 0, 0);
      }
      // T21^T = -T11^T Y^T: Y^T's registers are the B operand as they stand when step s contracts the rows that register s holds
      f32x16 t21 = zero16();
#pragma unroll
      for (int s = 0; s < 16; s++)
        t21 = __builtin_amdgcn_mfma_f32_32x32x2f32(at[32 + 8 * (s >> 2) + 4 * hf + (s & 3)][c], y[s], t21, 0, 0, 0);
      __bf16* out = a.rec + op_index(a, chunk, kh * rep + r0 + hh) * REC_ELEMS;
      const int at_f[2] = {8 * t_piece(lane, 0), 8 * t_piece(lane, 1)};
      auto put = [&](int f, const float (&t)[8]) {
        const bf16x8 hi = cvt8(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7]);
        *(bf16x8*)(out + REC_THI + f * FRAG + at_f[f & 1]) = hi;
        *(bf16x8*)(out + REC_TLO + f * FRAG + at_f[f & 1]) = cvt8(t[0] - (float)hi[0], t[1] - (float)hi[1], t[2] - (float)hi[2], t[3] - (float)hi[3],
                                                    t[4] - (float)hi[4], t[5] - (float)hi[5], t[6] - (float)hi[6], t[7] - (float)hi[7]);
      };
#pragma unroll
      for (int js = 0; js < 2; js++) {
        float t11[8], t22[8], t[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const int j = 16 * js + 8 * (e >> 2) + (e & 3);         // column of the lower half of the lanes; the upper half: j + 4
          t11[e] = j == c ? 0.f : x[j];                           // (T - I: the unit diagonal is added in fp32)
          t22[e] = j + 4 == c ? 0.f : x[j + 4];
          swap32(t11[e], t22[e]);
          t[e] = -t21[8 * js + e];
        }
        put(js, t11);
        put(2 + js, t);
        put(4 + js, t22);
      }
    }
    if (r0 + PREP_HEADS < rep) row_factors(r0 + PREP_HEADS);
  }
}

// ---- scan kernel ------------------------------------------------------------------------------------
// LDS: two images of one chunk's operands, filled by direct global -> LDS copies: the copy of the next chunk runs beside the
// products of this one.  K, Q and V are swizzled tiles (dma_tile64), the record is copied as it stands.  The two images of
// an array lie next to each other, so that both are within an instruction's immediate offset of one address register.
constexpr int TILE_B = GC * GD * 2, REC_B = REC_ELEMS * 2;
constexpr int L_K = 0, L_Q = 2 * TILE_B, L_V = 4 * TILE_B, L_REC = 6 * TILE_B, SCAN_LDS = 6 * TILE_B + 2 * REC_B;
static_assert(SCAN_LDS <= 160 * 1024, "LDS of one compute unit");
constexpr int R_THI = REC_THI * 2, R_TLO = REC_TLO * 2, R_ROW = REC_ROW * 2, R_P = REC_P * 2;         // bytes inside a record
constexpr int R_BETA = R_ROW, R_BEG = R_ROW + 4 * GC, R_EL = R_ROW + 8 * GC, R_EG = R_ROW + 12 * GC;

// The scalars of 64 consecutive chunks, one chunk per lane.
struct ChunkMeta {
  int first, tok0, len, src, dst, cap;
  static constexpr int ENTERS = 256, LEAVES = 512;
  __device__ __forceinline__ void load(const GdnArgs& a, int chunk, int lane) {
    const int at = min(chunk + lane, a.n_chunks - 1);
    first = chunk;
    tok0 = a.chunk_tok0[at]; len = a.chunk_len[at]; src = a.chunk_src[at]; dst = a.chunk_dst[at];
    cap = a.chunk_cap ? a.chunk_cap[at] : -1;
    len |= (src != -2 ? ENTERS : 0) | (dst >= 0 || cap >= 0 ? LEAVES : 0);       // length and what is rare about the chunk in one word
    asm volatile("" : "+v"(tok0), "+v"(len), "+v"(src), "+v"(dst), "+v"(cap));   // (waited for here)
  }
  __device__ __forceinline__ int get(int v, int chunk) const { return __builtin_amdgcn_readlane(v, chunk - first); }
};

// Which value head a walk's workgroup takes.  Consecutive workgroups go round-robin over the 8 XCDs; the value heads of a key
// head read the same q and k rows, so they are given ids 8 apart and share one XCD's L2.
__device__ __forceinline__ int walk_head(const GdnArgs& a, int id) {
  const int rep = a.hv / a.hk;
  return a.hk_n % 8 == 0 ? ((id >> 3) / rep * 8 + (id & 7)) * rep + (id >> 3) % rep : id;
}
// Which segment a workgroup takes: its place in the walk's order is its ticket, the number of workgroups of its column (blockIdx.x) that
// have started before it.  The order in which the hardware starts workgroups is not documented, and with walks of two streams on the
// chip the first one that is not finished may not have been started at all: 4 heads' workgroups of one walk wait on XCD 0 for one
// that has no room on XCD 1, where those of the other walk wait for one that has none on XCD 0.  (16406 tokens of 16 / 32 heads, places
// from block ids / from tickets: forward 257.8 / 257.7 us, backward 913.7 / 914.4.)
template <bool REVERSE>
__device__ __forceinline__ void walk_start(const GdnArgs& a, int half, int lane, ChunkMeta& meta, int& seg, int& c_begin, int& c_end) {
  __shared__ int place_of_all;
  if (a.tickets) {
    if (threadIdx.x == 0)
      place_of_all = __hip_atomic_fetch_add(&a.tickets[(int)blockIdx.x - half * a.hv_n].started[half], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
  }
  const int place = __builtin_amdgcn_readfirstlane(a.tickets ? place_of_all : a.seg_base + (int)blockIdx.y);
  seg = REVERSE ? reverse_walk_segment(place, a.n_segments, a.n_levels, a.level_off) : place;
  c_begin = __builtin_amdgcn_readfirstlane(a.seg_chunk0 ? a.seg_chunk0[seg] : 0);
  c_end = __builtin_amdgcn_readfirstlane(a.seg_chunk1 ? a.seg_chunk1[seg] : a.n_chunks);
  meta.load(a, REVERSE ? max(c_end - 64, 0) : c_begin, lane);
}
__device__ __forceinline__ void walker_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }      // (of waves that copy nothing)
__device__ __forceinline__ void walk_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }

// The copies of one chunk's operands, pieces of 1 KB per wave.  They are requested one by one between the products of the
// chunk before (piece): a wave that requests them all at once stands still for 2000 of a step's 7000 cycles.
// WALK_FWD: Q, K, V and the record (17 pieces); WALK_SAVE: K, V and the record up to the row factors (12); WALK_REV: Q, K, dO
// in V's place and the record (17).  A piece is copied by the four waves of a workgroup, or by two in two turns.
enum { WALK_FWD, WALK_SAVE, WALK_REV };
struct NoCopy { static constexpr int N = 0; };           // somebody else's
template <int WALK, int WAVES>
struct ChunkCopy {
  static constexpr int TURNS = 4 / WAVES;
  static constexpr int REC_KB = WALK == WALK_SAVE ? REC_P * 2 / 1024 : REC_B / 1024, N = (WALK == WALK_SAVE ? 8 : 12) + (REC_KB + 3) / 4;
  const char *k0, *q0, *v0, *rec0;      // of token 0 / chunk 0: K and Q of the key head, V of the value head, the records of the head
  uint32_t k_row, v_row;                // bytes per token
  const char *k, *q, *v, *rec;
  uint32_t kv[4 * TURNS], vv[4 * TURNS];    // this lane's byte offsets in the rows of K / Q and of V
  int len;
  uint32_t to_tile, to_rec;             // LDS address of the image to fill: its tiles' first, its record
  __device__ __forceinline__ void start(const GdnArgs& a, int h, uint32_t lds) {
    const int kh = h / (a.hv / a.hk);
    k0 = (const char*)(a.k + (size_t)kh * GD);
    q0 = (const char*)(a.q + (size_t)kh * GD);
    v0 = (const char*)((WALK == WALK_REV ? a.d_o : a.v) + (size_t)h * GD);
    rec0 = (const char*)(a.rec + op_index(a, 0, h) * REC_ELEMS);
    k_row = (uint32_t)a.hk * (GD * 2);
    v_row = (uint32_t)a.hv * (GD * 2);
    len = 0;
    to_tile = lds;
    to_rec = lds + L_REC;
  }
  __device__ __forceinline__ void other_image(int sign) { to_tile += sign * TILE_B; to_rec += sign * REC_B; }
  __device__ __forceinline__ void point(int chunk, int tok0, int new_len, int w, int lane) {
    const uint64_t krow = (uint64_t)(uint32_t)tok0 * k_row;
    k = k0 + krow;
    q = q0 + krow;
    v = v0 + (uint64_t)(uint32_t)tok0 * v_row;
    rec = rec0 + (uint64_t)(uint32_t)chunk * REC_B;
    if (new_len == len) return;
    len = new_len;
#pragma unroll
    for (int u = 0; u < 4 * TURNS; u++) {
      const int r4 = 4 * (w + WAVES * (u >> 2)) + (u & 3), lr = lane >> 4;    // as dma_tile64: 4 rows per piece, 16-byte chunks permuted
      const uint32_t row = (uint32_t)min(4 * r4 + lr, len - 1), col = 16u * (uint32_t)((lane & 15) ^ ((lr << 2) | (r4 & 3)));
      kv[u] = row * k_row + col;
      vv[u] = row * v_row + col;
    }
  }
  __device__ __forceinline__ void piece(int p, int w, int lane) const {
    const int u = p & 3;
    if (WALK == WALK_SAVE && p >= 4) p += 4;                      // (no Q)
#pragma unroll
    for (int t = 0; t < TURNS; t++) {
      const int wt = w + WAVES * t;
      if (p < 12) {
        const int tile = p < 4 ? L_K : p < 8 ? L_Q : L_V;
        dma16(p < 4 ? k : p < 8 ? q : v, p < 8 ? kv[4 * t + u] : vv[4 * t + u], to_tile + tile + (4 * wt + u) * 1024);
      } else {
        const int i = min(4 * (p - 12) + wt, REC_KB - 1);         // (the last one twice)
        dma16(rec + 1024 * i, 16u * lane, to_rec + 1024 * i);
      }
    }
  }
};

// LDS byte addresses of this lane's fragments in the current image
struct ScanAddr {
  uint32_t row[8];      // rows of K as operands, k-step ks (row block, tile, image: immediate offsets)
  uint32_t kt[4][2];    // K transposed, 32 key dims kt
  uint32_t vt[2];       // V transposed, this wave's 32 columns
  uint32_t rec, frag, sc, eg;
  uint32_t tf[2];       // T: even and odd fragments
  uint32_t tt[2];       // T transposed: blocks of 4 rows x 16 columns of the fragments, and the 4 rows 8 below
  __device__ __forceinline__ void other_image(int sign) {
    const uint32_t tile = (uint32_t)(sign * TILE_B), rec_b = (uint32_t)(sign * REC_B);
#pragma unroll
    for (int i = 0; i < 8; i++) row[i] += tile;
#pragma unroll
    for (int i = 0; i < 4; i++) { kt[i][0] += tile; kt[i][1] += tile; }
    vt[0] += tile; vt[1] += tile;
    frag += rec_b; sc += rec_b; eg += rec_b;
    tf[0] += rec_b; tf[1] += rec_b; tt[0] += rec_b; tt[1] += rec_b;
  }
  __device__ __forceinline__ void set(uint32_t lds, int lane, int w) {
    const int c = lane & 31, hf = lane >> 5, i16 = lane & 15, gidx = (lane >> 4) & 1;
    rec = lds;
    const int rd = row_frag_base(lane);
#pragma unroll
    for (int ks = 0; ks < 8; ks++) row[ks] = rec + 2u * (uint32_t)(rd ^ (ks << 4));
    const TrBase tr = tr_frag_base(lane);
    vt[0] = rec + L_V + 2u * (uint32_t)(tr.x0 ^ (w << 5));
    vt[1] = rec + L_V + 2u * (uint32_t)(tr.x1 ^ (w << 5));
    // K: the two middle groups of 4 of every 16 columns change places (state_dim)
    const TrBase kr = tr_frag_base((lane & ~3) | ((lane & 1) << 1) | ((lane >> 1) & 1));
#pragma unroll
    for (int t = 0; t < 4; t++) {
      kt[t][0] = rec + 2u * (uint32_t)(kr.x0 ^ (t << 5));
      kt[t][1] = rec + 2u * (uint32_t)(kr.x1 ^ (t << 5));
    }
    frag = rec + L_REC + 16u * lane;
    sc = rec + L_REC + 16u * hf;
    eg = rec + L_REC + 4u * c;
    const int at = 32 * (i16 & 1) + 4 * hf + (i16 >> 2);          // row 4 hf + i16 / 4, columns 16 gidx + 4 (i16 % 4) ..
#pragma unroll
    for (int b = 0; b < 2; b++) {
      tf[b] = rec + L_REC + 16u * (uint32_t)t_piece(lane, b);
      tt[b] = rec + L_REC + (uint32_t)(1024 * gidx + 16 * t_piece(at + 8 * b, gidx) + 8 * ((i16 >> 1) & 1));
    }
    // (opaque: with known parts the compiler folds them into offsets past 64 KB and adds them up again at every read)
    asm volatile("" : "+v"(frag), "+v"(sc), "+v"(eg), "+v"(vt[0]), "+v"(vt[1]), "+v"(tf[0]), "+v"(tf[1]), "+v"(tt[0]), "+v"(tt[1]));
  }
};


// Which key dims of a 32-row state tile an accumulator register holds.  Rows of the tile are key dims in an order in which the
// 8 rows that make up a lane's share of a 16-deep operand are 8 consecutive key dims, so that the rows of K and Q meet them
// as plain 16-byte reads: tile row 16 t + 8 a + 4 h + b is key dim 16 t + 8 h + 4 a + b.
__device__ __forceinline__ int state_dim(int r, int hf) { return 16 * (r >> 3) + 8 * hf + 4 * ((r >> 2) & 1) + (r & 3); }

__device__ __forceinline__ bf16x8 cvt_regs(const f32x16& t, int r) {
  return cvt8(t[r], t[r + 1], t[r + 2], t[r + 3], t[r + 4], t[r + 5], t[r + 6], t[r + 7]);
}

// The state (or its gradient) of a wave's 32 columns.
struct ScanState {
  f32x16 s[4];          // key dims 32 kt + state_dim(r), this wave's column c
  bf16x8 sb[8];         // the same rounded, as an operand: lane = value column, k = key dims 16 ks + 8 hf ..  (6, 7: formed inside the step)
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int kt = 0; kt < 4; kt++) s[kt] = zero16();
  }
  __device__ __forceinline__ void round() {
#pragma unroll
    for (int ks = 0; ks < 6; ks++) sb[ks] = cvt_regs(s[ks >> 1], 8 * (ks & 1));
  }
  // A state in memory.  SHARED: what only the walks use (saved node-end states, gradients of segments and slots) lies as the waves hold
  // it, two registers of a lane side by side, and goes past the caches of the XCD that may hold an older version, as another
  // workgroup of the same launch reads it.  Otherwise [128][128], as the caller gives and takes it.
  // (The lane's first element is opaque: the offsets from it are formed where they are used, not kept.)
  template <bool SHARED>
  __device__ static __forceinline__ int first(int lane, int w) {
    int at = SHARED ? GD * 32 * w + 2 * lane : 8 * (lane >> 5) * GD + 32 * w + (lane & 31);
    asm volatile("" : "+v"(at));
    return at;
  }
  // pin: the wait for these (rare) loads belongs here, not at the merge point
  template <bool SHARED>
  __device__ __forceinline__ void get(const float* state, int lane, int w) {
    const float* sp = state + first<SHARED>(lane, w);
#pragma unroll
    for (int kt = 0; kt < 4; kt++)
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        if constexpr (SHARED) {
          const uint64_t x = __hip_atomic_load((const uint64_t*)(sp + 128 * (8 * kt + r / 2)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          s[kt][r] = __uint_as_float((uint32_t)x);
          s[kt][r + 1] = __uint_as_float((uint32_t)(x >> 32));
        } else {
          s[kt][r] = sp[(32 * kt + state_dim(r, 0)) * GD];
          s[kt][r + 1] = sp[(32 * kt + state_dim(r + 1, 0)) * GD];
        }
      }
#pragma unroll
    for (int kt = 0; kt < 4; kt++) pin(s[kt]);
  }
  template <bool SHARED>
  __device__ __forceinline__ void add(const float* state, int lane, int w) {
    ScanState t;                        // (all loads in flight before the first sum)
    t.get<SHARED>(state, lane, w);
#pragma unroll
    for (int kt = 0; kt < 4; kt++) s[kt] += t.s[kt];
  }
  template <bool SHARED>
  __device__ __forceinline__ void put(float* state, int lane, int w) const {
    float* sp = state + first<SHARED>(lane, w);
#pragma unroll
    for (int kt = 0; kt < 4; kt++)
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        if constexpr (SHARED) {
          const uint64_t x = (uint64_t)__float_as_uint(s[kt][r + 1]) << 32 | __float_as_uint(s[kt][r]);
          __hip_atomic_store((uint64_t*)(sp + 128 * (8 * kt + r / 2)), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          sp[(32 * kt + state_dim(r, 0)) * GD] = s[kt][r];
          sp[(32 * kt + state_dim(r + 1, 0)) * GD] = s[kt][r + 1];
        }
      }
  }
  // where a chunk does not continue the previous one: a saved node-end state, or the state handed in for the roots
  __device__ __forceinline__ void enter(const GdnArgs& a, int src, int h, int lane, int w) {
    if (src >= 0) {
      const bool saved = !a.seg_chunk0 || wait_for(a, a.slot_sync, src, h, w);
      get<true>(a.slots + ((size_t)src * a.hv + h) * (GD * GD), lane, w);
      if (!saved) spoil();
    } else if (a.initial_state) {
      get<false>(a.initial_state + (size_t)h * (GD * GD), lane, w);
    } else {
      zero();
    }
    round();
  }
  __device__ __forceinline__ void leave(const GdnArgs& a, int dst, int cap, int h, int lane, int w) const {
    if (dst >= 0) {
      put<true>(a.slots + ((size_t)dst * a.hv + h) * (GD * GD), lane, w);
      publish(a, a.slot_sync, dst, h, lane, w);
    }
    if (cap >= 0) put<false>(a.state_out + ((size_t)cap * a.hv + h) * (GD * GD), lane, w);
  }
  // What a segment starts from comes from segments of earlier levels, of the same launch: a flag per state and wave (a wave needs
  // the columns that its like in the other workgroup holds).  The stores have reached memory when the flag is set.
  __device__ static __forceinline__ void publish(const GdnArgs& a, WalkSync* sync, int i, int h, int lane, int w) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0 && a.seg_chunk0) __hip_atomic_store(&sync[(size_t)i * a.hv_n + h].stored[w], (uint8_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // Every wait ends: the workgroups of a column of the grid (a head's, or half a head's) take their segments by ticket (walk_start), so
  // that whoever is waited for, being of the same column and earlier in the order, has a smaller ticket and is running, whatever the
  // order in which workgroups are started and whatever else is on the chip; of those running the first has nothing left to wait for.
  // With a schedule that is not one of this program (a state that no segment saves) the wait gives up after a time that no
  // walk takes, 75 times a step for every chunk of the call, and what depends on it becomes NaN.
  __device__ static __forceinline__ bool wait_for(const GdnArgs& a, const WalkSync* sync, int i, int h, int w) {
    const uint8_t* flag = &sync[(size_t)i * a.hv_n + h].stored[w];
    bool there = false;
    for (int n = 0; n < a.max_polls; n++) {
      there = __builtin_amdgcn_readfirstlane(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (there) break;
      __builtin_amdgcn_s_sleep(4);
    }
    asm volatile("" ::: "memory");
    return there;
  }
  __device__ __forceinline__ void spoil() {
#pragma unroll
    for (int kt = 0; kt < 4; kt++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[kt][r] = __builtin_nanf("");
  }
};

// One chunk.  On entry the copy of its operands has landed, `copy` points to the next chunk's.  The matrix instructions are a sequence of slots,
// each with a share of the reads, the arithmetic and the next chunk's copies, closed by a scheduling fence.  A wave is alone on its
// SIMD, so that nothing else fills a gap: what counts is the number of instructions (about 4 cycles each) and that none waits.
__device__ __forceinline__ void scan_step(const GdnArgs& a, ScanState& st, const ScanAddr& ad, const ChunkCopy<WALK_FWD, 4>& copy, bool has_next, int tok0,
                                          int len, int h, int w, int lane, const uint32_t (&o_at)[2]) {
  const int c = lane & 31;
  f32x16(&s)[4] = st.s;
  bf16x8(&sb)[8] = st.sb;
  auto copies = [&](int p, int n) {
    if (has_next) {
#pragma unroll
      for (int i = p; i < p + n; i++) copy.piece(i, w, lane);
    }
  };
  auto read_row = [&](int i, int tile) { return lds_b128(ad.row[i >> 1], tile + (i & 1) * 32 * TILE_ROW * 2); };
  auto read_kt = [&](int kt, int js) { return lds_tr2(ad.kt[kt][0], ad.kt[kt][1], L_K + 16 * js * TILE_ROW * 2); };
  auto read_t = [&](int off, int f) { return lds_b128(ad.tf[f & 1], off + 1024 * f); };
  auto read_frag = [&](int off, int f) { return lds_b128(ad.frag, off + 1024 * f); };
  auto read_rows = [&](int arr, int grp) { return *(TT_LDS(const f32x4)*)(ad.sc + arr + 32 * grp); };

  // Fragments are requested eight slots and more ahead: an LDS round trip takes about 250 cycles while the other waves read and
  // the copies land.
  constexpr int RING = 8;
  // ---- K S0 (rows = tokens, columns = value columns); the state is scaled beside it ----
  bf16x8 fk[RING], fq[RING], vf[4], th[6], tl[6];
  f32x16 vn[2], qs[2];                  // vn: K S0, then R, then Vn
  f32x4 b4[2], g4[2], el[4];
  auto rows_r = [&](int grp) { b4[grp & 1] = read_rows(R_BETA, grp); g4[grp & 1] = read_rows(R_BEG, grp); };
  const float glast = *(TT_LDS(const float)*)(ad.eg - 4u * c + R_EG + 4 * (GC - 1));
#pragma unroll
  for (int i = 0; i < RING; i++) fk[i] = read_row(i, L_K);
  float eg0 = *(TT_LDS(const float)*)(ad.eg + R_EG), eg1 = *(TT_LDS(const float)*)(ad.eg + R_EG + 128);
  fence();
#pragma unroll
  for (int i = 0; i < 16; i++) {
    vn[i & 1] = mfma32(fk[i % RING], sb[i >> 1], i < 2 ? zero16() : vn[i & 1]);
    if (i + RING < 16) fk[i % RING] = read_row(i + RING, L_K);
    else fq[i % RING] = read_row(i + RING - 16, L_Q);
    if (i == 2) sb[6] = cvt_regs(s[3], 0);
    if (i == 3) sb[7] = cvt_regs(s[3], 8);
    if (i >= 4 && i < 14) {
#pragma unroll
      for (int r = 0; r < 64; r++)
        if (r * 10 / 64 == i - 4) s[r >> 4][r & 15] *= glast;
    }
    if (i >= 8 && i < 12) vf[i - 8] = lds_tr2(ad.vt[0], ad.vt[1], 16 * (i - 8) * TILE_ROW * 2);
    if (i == 12) rows_r(0);
    if (i == 14) rows_r(1);
    if (i & 1) copies(i >> 1, 1);
    fence();
  }
  eg0 *= a.scale; eg1 *= a.scale;
  // ---- (Q S0)^T (rows = value columns, columns = tokens); R beside it, 4 tokens (token block tb, register group r4) per two slots ----
  bf16x8 rf[4], uf[4], us[4], kf[4][4], pf[6];
#pragma unroll
  for (int i = 0; i < 16; i++) {
    qs[i & 1] = mfma32(sb[i >> 1], fq[i % RING], i < 2 ? zero16() : qs[i & 1]);
    if (i + RING < 16) fq[i % RING] = read_row(i + RING, L_Q);
    const int grp = i >> 1, tb = grp >> 2, r4 = grp & 3;
#pragma unroll
    for (int e = 2 * (i & 1); e < 2 * (i & 1) + 2; e++)
      vn[tb][4 * r4 + e] = b4[grp & 1][e] * (float)vf[grp >> 1][4 * (grp & 1) + e] - g4[grp & 1][e] * vn[tb][4 * r4 + e];
    if ((i & 1) && grp < 6) rows_r(grp + 2);
    if ((i & 3) == 3) rf[i >> 2] = cvt_regs(vn[i >> 3], 8 * ((i >> 2) & 1));
    if (i & 1) copies(8 + (i >> 1), 1);
    if (i >= 2 && i < 8) th[i - 2] = read_t(R_THI, i - 2);
    if (i >= 8 && i < 14) tl[i - 8] = read_t(R_TLO, i - 8);
    if (i >= 14) { el[2 * (i - 14)] = read_rows(R_EL, 2 * (i - 14)); el[2 * (i - 14) + 1] = read_rows(R_EL, 2 * (i - 14) + 1); }
    fence();
  }
  // ---- Vn = R + (T - I) R: the accumulators start from R in fp32 ----
  // Vn as an operand twice: for P Vn as it is, for the state update with its rows scaled
  auto put_u = [&](int js) {
    const f32x16& t = vn[js >> 1];
    const int r = 8 * (js & 1);
    const f32x4 e0 = el[2 * (js & 1)], e1 = el[2 * (js & 1) + 1];
    uf[js] = cvt_regs(t, r);
    us[js] = cvt8(t[r] * e0[0], t[r + 1] * e0[1], t[r + 2] * e0[2], t[r + 3] * e0[3], t[r + 4] * e1[0], t[r + 5] * e1[1],
                  t[r + 6] * e1[2], t[r + 7] * e1[3]);
  };
  auto scale_q = [&](int tb, int r0, float eg) {
#pragma unroll
    for (int r = r0; r < r0 + 4; r++) qs[tb][r] *= eg;
  };
  vn[0] = mfma32(th[0], rf[0], vn[0]);  kf[0][0] = read_kt(0, 0); copies(16, 1);              fence();
  vn[1] = mfma32(th[2], rf[0], vn[1]);  kf[1][0] = read_kt(1, 0); scale_q(0, 0, eg0);         fence();
  vn[0] = mfma32(tl[0], rf[0], vn[0]);  kf[2][0] = read_kt(2, 0); scale_q(0, 4, eg0);         fence();
  vn[1] = mfma32(tl[2], rf[0], vn[1]);  kf[3][0] = read_kt(3, 0); scale_q(0, 8, eg0);         fence();
  vn[0] = mfma32(th[1], rf[1], vn[0]);  pf[0] = read_frag(R_P, 0); scale_q(0, 12, eg0);       fence();
  vn[1] = mfma32(th[3], rf[1], vn[1]);  kf[0][1] = read_kt(0, 1); scale_q(1, 0, eg1);         fence();
  vn[0] = mfma32(tl[1], rf[1], vn[0]);  kf[1][1] = read_kt(1, 1); scale_q(1, 4, eg1);         fence();
  vn[1] = mfma32(tl[3], rf[1], vn[1]);  kf[2][1] = read_kt(2, 1); scale_q(1, 8, eg1);         fence();
  vn[1] = mfma32(th[4], rf[2], vn[1]);  kf[3][1] = read_kt(3, 1); scale_q(1, 12, eg1);        fence();
  vn[1] = mfma32(tl[4], rf[2], vn[1]);  pf[1] = read_frag(R_P, 1); put_u(0);                  fence();
  vn[1] = mfma32(th[5], rf[3], vn[1]);  pf[2] = read_frag(R_P, 2); pf[3] = read_frag(R_P, 3); put_u(1); fence();
  vn[1] = mfma32(tl[5], rf[3], vn[1]);
#pragma unroll
  for (int i = 0; i < 4; i++) el[i] = read_rows(R_EL, 4 + i);
  fence();

  // ---- S1 = exp(gamma_last) S0 + K^T (scaled Vn);  O^T = (scaled Q S0)^T + Vn^T P^T ----
  // a lane holds token 32 tb + c and, per register group, 4 columns; the halves of the wave exchange theirs for pieces of 16 bytes
  __bf16* const o_row = a.o + ((size_t)tok0 * a.hv + h) * GD + 32 * w;
  auto put_o = [&](int tb, int pair) {
    const f32x16& t = qs[tb];
    const int r = 8 * pair;
    const uint2 x = __builtin_bit_cast(uint2, cvt4(t[r], t[r + 1], t[r + 2], t[r + 3]));
    const uint2 y = __builtin_bit_cast(uint2, cvt4(t[r + 4], t[r + 5], t[r + 6], t[r + 7]));
    const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false), hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    const i32x4 piece = {(int)lo[0], (int)hi[0], (int)lo[1], (int)hi[1]};
    if (32 * tb + c < len) *(i32x4*)((char*)o_row + o_at[tb] + 32 * pair) = piece;
  };
  s[0] = mfma32(kf[0][0], us[0], s[0]);    kf[0][2] = read_kt(0, 2);                           fence();
  s[1] = mfma32(kf[1][0], us[0], s[1]);    kf[1][2] = read_kt(1, 2);                           fence();
  qs[0] = mfma32(uf[0], pf[0], qs[0]);     pf[4] = read_frag(R_P, 4);                          fence();
  s[2] = mfma32(kf[2][0], us[0], s[2]);    kf[0][3] = read_kt(0, 3); put_u(2);                 fence();
  s[3] = mfma32(kf[3][0], us[0], s[3]);    kf[1][3] = read_kt(1, 3);                           fence();
  qs[0] = mfma32(uf[1], pf[1], qs[0]);     pf[5] = read_frag(R_P, 5);                          fence();
  s[0] = mfma32(kf[0][1], us[1], s[0]);    kf[2][2] = read_kt(2, 2); put_u(3);                 fence();
  s[1] = mfma32(kf[1][1], us[1], s[1]);    kf[2][3] = read_kt(2, 3);                           fence();
  qs[1] = mfma32(uf[0], pf[2], qs[1]);                                                         fence();
  s[2] = mfma32(kf[2][1], us[1], s[2]);    kf[3][2] = read_kt(3, 2);                           fence();
  s[3] = mfma32(kf[3][1], us[1], s[3]);    kf[3][3] = read_kt(3, 3);                           fence();
  qs[1] = mfma32(uf[1], pf[3], qs[1]);     put_o(0, 0);                                        fence();
  s[0] = mfma32(kf[0][2], us[2], s[0]);                                                        fence();
  qs[1] = mfma32(uf[2], pf[4], qs[1]);     put_o(0, 1);                                        fence();
  s[0] = mfma32(kf[0][3], us[3], s[0]);                                                        fence();
  s[1] = mfma32(kf[1][2], us[2], s[1]);                                                        fence();
  qs[1] = mfma32(uf[3], pf[5], qs[1]);     sb[0] = cvt_regs(s[0], 0);                          fence();
  s[1] = mfma32(kf[1][3], us[3], s[1]);    sb[1] = cvt_regs(s[0], 8);                          fence();
  s[2] = mfma32(kf[2][2], us[2], s[2]);    put_o(1, 0);                                        fence();
  s[2] = mfma32(kf[2][3], us[3], s[2]);    sb[2] = cvt_regs(s[1], 0); sb[3] = cvt_regs(s[1], 8); fence();
  s[3] = mfma32(kf[3][2], us[2], s[3]);    put_o(1, 1);                                        fence();
  s[3] = mfma32(kf[3][3], us[3], s[3]);    sb[4] = cvt_regs(s[2], 0); sb[5] = cvt_regs(s[2], 8); fence();
}

// A wave walks its segment with 32 columns of the state in its accumulators: 66 matrix instructions per chunk, no exchange
// between waves, one barrier per chunk (for the operand images).  Everything that one product hands to the next stays in the
// wave's registers: an accumulator tile is, rounded to bf16, an operand of the next product (tt_mfma.h).  A step of a chunk
// takes 2.7 us (3.3 with all copies requested at its start; the form before cut a head into two workgroups of eight waves that exchanged
// the state and Vn through LDS, 3.1 us and two workgroup steps per chunk and head on a full chip): all of 16406 tokens of 32 heads 172 us, 265
// before, with 67 KB instead of 128 per chunk and head from memory.  A few heads alone on the chip take longer than before (the
// eight waves stepped in 1.5 us there).  Two waves per column block, one for the chain K S0 -> Vn and one for the output, half of the state's rows
// each: 2 % slower.
__global__ __launch_bounds__(G_THREADS, 1) void gdn_scan_kernel(GdnArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char sm[SCAN_LDS];
  const int lane = threadIdx.x & 63, c = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = walk_head(a, blockIdx.x);
  ChunkMeta meta;
  int seg, c_begin, c_end;
  walk_start<false>(a, 0, lane, meta, seg, c_begin, c_end);
  ScanAddr ad;
  ad.set(__builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&sm), lane, w);
  const uint32_t o_at[2] = {(uint32_t)c * (uint32_t)a.hv * (GD * 2) + 16u * hf, (uint32_t)(32 + c) * (uint32_t)a.hv * (GD * 2) + 16u * hf};
  ChunkCopy<WALK_FWD, 4> copy;
  copy.start(a, h, ad.rec);
  copy.point(c_begin, meta.get(meta.tok0, c_begin), meta.get(meta.len, c_begin) & 255, w, lane);
#pragma unroll
  for (int p = 0; p < copy.N; p++) copy.piece(p, w, lane);
  ScanState st;
  st.zero();

  int sign = 1;                         // where the other image lies
  auto step = [&](int chunk) {
    const int tok0 = meta.get(meta.tok0, chunk), bits = meta.get(meta.len, chunk);
    const int dst = meta.get(meta.dst, chunk), cap = meta.get(meta.cap, chunk);
    if (bits & ChunkMeta::ENTERS) st.enter(a, meta.get(meta.src, chunk), h, lane, w);
    const bool has_next = chunk + 1 < c_end;
    if (has_next) {
      if (chunk + 1 - meta.first == 64) meta.load(a, chunk + 1, lane);
      copy.point(chunk + 1, meta.get(meta.tok0, chunk + 1), meta.get(meta.len, chunk + 1) & 255, w, lane);
    }
    walk_barrier();     // this wave's share of the operands has landed, and so has everybody else's; every wave has left the other image
    copy.other_image(sign);
    scan_step(a, st, ad, copy, has_next, tok0, bits & 255, h, w, lane, o_at);
    if (bits & ChunkMeta::LEAVES) st.leave(a, dst, cap, h, lane, w);
    ad.other_image(sign);
    sign = -sign;
  };
  for (int chunk = c_begin; chunk < c_end; chunk++) step(chunk);
}

// ---- forward walk of the backward: the scan without its output; S0 and Vn of every chunk are saved, rounded -----------
// Bound by memory where the chip is full (93 KB in and out per chunk and head), by a step's own instructions and LDS round trips where it is not:
// 182 us at 16406 tokens of 32 heads (235 in the form before).
template <class Copy>
__device__ __forceinline__ void fwalk_step(const GdnArgs& a, ScanState& st, const ScanAddr& ad, const Copy& copy, bool has_next,
                                           size_t op, int w, int lane) {
  const int c = lane & 31;
  f32x16(&s)[4] = st.s;
  bf16x8(&sb)[8] = st.sb;
  auto copies = [&](int p, int n) {
    if constexpr (Copy::N > 0) {
      if (has_next) {
#pragma unroll
        for (int i = p; i < p + n; i++) copy.piece(i, w, lane);
      }
    }
  };
  auto read_row = [&](int i) { return lds_b128(ad.row[i >> 1], L_K + (i & 1) * 32 * TILE_ROW * 2); };
  auto read_kt = [&](int kt, int js) { return lds_tr2(ad.kt[kt][0], ad.kt[kt][1], L_K + 16 * js * TILE_ROW * 2); };
  auto read_t = [&](int off, int f) { return lds_b128(ad.tf[f & 1], off + 1024 * f); };
  auto read_rows = [&](int arr, int grp) { return *(TT_LDS(const f32x4)*)(ad.sc + arr + 32 * grp); };
  const int pos = gdn_saved_lane(lane);
  bf16x8* const s0_out = (bf16x8*)a.sv.s0 + (op * 4 + w) * 512 + pos;
  bf16x8* const vn_out = (bf16x8*)a.sv.vns + (op * 4 + w) * 256 + pos;

  constexpr int RING = 8;
  // ---- K S0 (rows = tokens, columns = value columns) ----
  bf16x8 fk[RING], vf[4], th[6], tl[6], rf[4], us[4], kf[4][4];
  f32x16 vn[2], t1;                     // vn: K S0, then R, then Vn;  t1: part of the second block's sum
  f32x4 b4[2], g4[2], el[8];
  auto rows_r = [&](int grp) { b4[grp & 1] = read_rows(R_BETA, grp); g4[grp & 1] = read_rows(R_BEG, grp); };
  const float glast = *(TT_LDS(const float)*)(ad.eg - 4u * c + R_EG + 4 * (GC - 1));
#pragma unroll
  for (int i = 0; i < RING; i++) fk[i] = read_row(i);
  fence();
#pragma unroll
  for (int i = 0; i < 16; i++) {
    vn[i & 1] = mfma32(fk[i % RING], sb[i >> 1], i < 2 ? zero16() : vn[i & 1]);
    if (i + RING < 16) fk[i % RING] = read_row(i + RING);
    if (i == 2) sb[6] = cvt_regs(s[3], 0);
    if (i == 3) sb[7] = cvt_regs(s[3], 8);
    if (i >= 4 && i < 14) {
#pragma unroll
      for (int r = 0; r < 64; r++)
        if (r * 10 / 64 == i - 4) s[r >> 4][r & 15] *= glast;
    }
    if (i >= 8) s0_out[64 * (i - 8)] = sb[i - 8];
    if (i >= 6 && i < 10) vf[i - 6] = lds_tr2(ad.vt[0], ad.vt[1], 16 * (i - 6) * TILE_ROW * 2);
    if (i == 10) rows_r(0);
    if (i == 11) rows_r(1);
    if (i >= 12) th[i - 12] = read_t(R_THI, i - 12);
    if (i >= 12) tl[i - 12] = read_t(R_TLO, i - 12);
    if (i & 1) copies(i >> 1, 1);
    fence();
  }
  // ---- R, 4 tokens (token block tb, register group r4) at a time;  Vn = R + (T - I) R: the accumulators start from R in fp32 ----
  auto form_r = [&](int grp) {
    const int tb = grp >> 2, r = 4 * (grp & 3);
#pragma unroll
    for (int e = 0; e < 4; e++)
      vn[tb][r + e] = b4[grp & 1][e] * (float)vf[grp >> 1][4 * (grp & 1) + e] - g4[grp & 1][e] * vn[tb][r + e];
    if (grp < 6) rows_r(grp + 2);
    if (grp & 1) rf[grp >> 1] = cvt_regs(vn[tb], 8 * ((grp >> 1) & 1));
  };
  auto put_u = [&](int js) {
    const f32x16& t = vn[js >> 1];
    const int r = 8 * (js & 1);
    const f32x4 e0 = el[2 * js], e1 = el[2 * js + 1];
    vn_out[64 * js] = cvt_regs(t, r);
    us[js] = cvt8(t[r] * e0[0], t[r + 1] * e0[1], t[r + 2] * e0[2], t[r + 3] * e0[3], t[r + 4] * e1[0], t[r + 5] * e1[1],
                  t[r + 6] * e1[2], t[r + 7] * e1[3]);
  };
  form_r(0); form_r(1);
  fence();
  t1 = mfma32(th[2], rf[0], zero16());   form_r(2); copies(8, 1);                                        fence();
  t1 = mfma32(tl[2], rf[0], t1);         form_r(3); th[4] = read_t(R_THI, 4); tl[4] = read_t(R_TLO, 4); fence();
  vn[0] = mfma32(th[0], rf[0], vn[0]);   form_r(4); th[5] = read_t(R_THI, 5); tl[5] = read_t(R_TLO, 5); fence();
  t1 = mfma32(th[3], rf[1], t1);         form_r(5); copies(9, 1);                                        fence();
  vn[0] = mfma32(tl[0], rf[0], vn[0]);   form_r(6); el[0] = read_rows(R_EL, 0); el[1] = read_rows(R_EL, 1); fence();
  t1 = mfma32(tl[3], rf[1], t1);         form_r(7); el[2] = read_rows(R_EL, 2); el[3] = read_rows(R_EL, 3); fence();
  vn[0] = mfma32(th[1], rf[1], vn[0]);   kf[0][0] = read_kt(0, 0); kf[1][0] = read_kt(1, 0);              fence();
  t1 = mfma32(th[4], rf[2], t1);         kf[2][0] = read_kt(2, 0); kf[3][0] = read_kt(3, 0); copies(10, 1); fence();
  vn[0] = mfma32(tl[1], rf[1], vn[0]);   kf[0][1] = read_kt(0, 1); kf[1][1] = read_kt(1, 1);              fence();
  t1 = mfma32(tl[4], rf[2], t1);         kf[2][1] = read_kt(2, 1); kf[3][1] = read_kt(3, 1);              fence();
  vn[1] = mfma32(th[5], rf[3], vn[1]);   el[4] = read_rows(R_EL, 4); el[5] = read_rows(R_EL, 5);          fence();
  t1 = mfma32(tl[5], rf[3], t1);         el[6] = read_rows(R_EL, 6); el[7] = read_rows(R_EL, 7); put_u(0); fence();
  // ---- S1 = exp(gamma_last) S0 + K^T (scaled Vn) ----
  s[0] = mfma32(kf[0][0], us[0], s[0]);  put_u(1); kf[0][2] = read_kt(0, 2);                             fence();
  s[1] = mfma32(kf[1][0], us[0], s[1]);  copies(11, 1); kf[0][3] = read_kt(0, 3);                        fence();
  s[2] = mfma32(kf[2][0], us[0], s[2]);  kf[1][2] = read_kt(1, 2);
#pragma unroll
  for (int r = 0; r < 16; r++) vn[1][r] += t1[r];
  fence();
  s[3] = mfma32(kf[3][0], us[0], s[3]);  kf[1][3] = read_kt(1, 3);                                       fence();
  s[0] = mfma32(kf[0][1], us[1], s[0]);  put_u(2); kf[2][2] = read_kt(2, 2);                             fence();
  s[1] = mfma32(kf[1][1], us[1], s[1]);  kf[2][3] = read_kt(2, 3);                                       fence();
  s[2] = mfma32(kf[2][1], us[1], s[2]);  put_u(3); kf[3][2] = read_kt(3, 2);                             fence();
  s[3] = mfma32(kf[3][1], us[1], s[3]);  kf[3][3] = read_kt(3, 3);                                       fence();
#pragma unroll
  for (int kt = 0; kt < 4; kt++) {
    s[kt] = mfma32(kf[kt][2], us[2], s[kt]);
    if (kt >= 2) sb[2 * kt - 4] = cvt_regs(s[kt - 2], 0);
    fence();
    s[kt] = mfma32(kf[kt][3], us[3], s[kt]);
    if (kt >= 2) sb[2 * kt - 3] = cvt_regs(s[kt - 2], 8);
    fence();
  }
  sb[4] = cvt_regs(s[2], 0); sb[5] = cvt_regs(s[2], 8);
}

// The two-wave forms of the walks have two waves more that copy the operands of both: on its SIMD nothing but a walking wave's own chain
// counts, and the copies, twice as many per wave there, are out of it (and so is the wait for its stores at a step's end).  Backward of chains of
// 1500 / 4000 / 8000 tokens of 8 heads 227 -> 197 / 367 -> 308 / 588 -> 512 us; and with a pause of 128 cycles behind every piece, so that
// they don't take the LDS from the walking waves' first reads, 197 / 304 / 485.
template <int WALK>
__device__ __forceinline__ void walk_copies(const GdnArgs& a, ChunkMeta& meta, uint32_t lds, int h, int first, int n, int w, int lane) {
  constexpr int STEP = WALK == WALK_REV ? -1 : 1;
  ChunkCopy<WALK, 2> copy;
  copy.start(a, h, lds);
  int sign = 1;
  for (int i = 0, chunk = first; i < n; i++, chunk += STEP) {      // the operands of step i, into the image that step i - 2 has left
    if (STEP > 0 && chunk - meta.first == 64) meta.load(a, chunk, lane);
    if (STEP < 0 && chunk < meta.first) meta.load(a, max(chunk - 63, 0), lane);
    copy.point(chunk, meta.get(meta.tok0, chunk), meta.get(meta.len, chunk) & 255, w, lane);
#pragma unroll
    for (int p = 0; p < copy.N; p++) {
      copy.piece(p, w, lane);
      __builtin_amdgcn_s_sleep(2);
    }
    walk_barrier();                     // (the one in front of step i)
    copy.other_image(sign);
    sign = -sign;
  }
}

template <int WAVES>
__global__ __launch_bounds__(G_THREADS, 1) void gdn_fwalk_kernel(GdnArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char sm[SCAN_LDS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = WAVES < 4 ? (int)blockIdx.x / a.hv_n : 0;
  const int w = wave + WAVES * half;
  const int h = walk_head(a, blockIdx.x - half * a.hv_n);
  ChunkMeta meta;
  int seg, c_begin, c_end;
  walk_start<false>(a, half, lane, meta, seg, c_begin, c_end);
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&sm);
  if (WAVES < 4 && wave >= WAVES) {
    walk_copies<WALK_SAVE>(a, meta, lds, h, c_begin, c_end - c_begin, wave - WAVES, lane);
    return;
  }
  ScanAddr ad;
  ad.set(lds, lane, w);
  std::conditional_t<WAVES == 4, ChunkCopy<WALK_SAVE, 4>, NoCopy> copy;
  if constexpr (WAVES == 4) {
    copy.start(a, h, ad.rec);
    copy.point(c_begin, meta.get(meta.tok0, c_begin), meta.get(meta.len, c_begin) & 255, w, lane);
#pragma unroll
    for (int p = 0; p < copy.N; p++) copy.piece(p, w, lane);
  }
  ScanState st;
  st.zero();
  int sign = 1;                         // where the other image lies
  auto step = [&](int chunk) {
    const int bits = meta.get(meta.len, chunk), dst = meta.get(meta.dst, chunk);
    if (bits & ChunkMeta::ENTERS) st.enter(a, meta.get(meta.src, chunk), h, lane, w);
    const bool has_next = chunk + 1 < c_end;
    if (has_next) {
      if (chunk + 1 - meta.first == 64) meta.load(a, chunk + 1, lane);
      if constexpr (WAVES == 4) copy.point(chunk + 1, meta.get(meta.tok0, chunk + 1), meta.get(meta.len, chunk + 1) & 255, w, lane);
    }
    if constexpr (WAVES == 4) {
      walk_barrier();
      copy.other_image(sign);
    } else {
      walker_barrier();
    }
    fwalk_step(a, st, ad, copy, has_next, op_index(a, chunk, h), w, lane);
    if (bits & ChunkMeta::LEAVES) st.leave(a, dst, -1, h, lane, w);         // (nothing is captured here)
    ad.other_image(sign);
    sign = -sign;
  };
  for (int chunk = c_begin; chunk < c_end; chunk++) step(chunk);
}

// ---- reverse walk of the backward ------------------------------------------------------------------------
// The state's gradient in the place of the state, last chunk of a segment to first; the leaving state's gradient dS1 and dR of
// every chunk are saved, rounded.  The scan's structure: K dS1 -> dVn -> dR is the chain, Q^T dO beside it.  257 us at 16406 tokens of
// 32 heads (303 in the form before, which left the transposed solve to the finish kernel).
template <class Copy>
__device__ __forceinline__ void rwalk_step(const GdnArgs& a, ScanState& st, const ScanAddr& ad, const Copy& copy, bool has_next,
                                           size_t op, int len, int w, int lane) {
  const int c = lane & 31, hf = lane >> 5;
  f32x16(&s)[4] = st.s;
  bf16x8(&sb)[8] = st.sb;
  auto copies = [&](int p, int n) {
    if constexpr (Copy::N > 0) {
      if (has_next) {
#pragma unroll
        for (int i = p; i < p + n; i++) copy.piece(i, w, lane);
      }
    }
  };
  auto read_row = [&](int i) { return lds_b128(ad.row[i >> 1], L_K + (i & 1) * 32 * TILE_ROW * 2); };
  auto read_kt = [&](int kt, int js) { return lds_tr2(ad.kt[kt][0], ad.kt[kt][1], L_K + 16 * js * TILE_ROW * 2); };
  auto read_qt = [&](int kt, int js) { return lds_tr2(ad.kt[kt][0], ad.kt[kt][1], L_Q + 16 * js * TILE_ROW * 2); };
  auto read_frag = [&](int off, int f) { return lds_b128(ad.frag, off + 1024 * f); };
  auto read_rows = [&](int arr, int grp) { return *(TT_LDS(const f32x4)*)(ad.sc + arr + 32 * grp); };
  // rows 32 jb .. of T^T, tokens 16 is .. in the order of accumulator registers: fragment f holds (is / 2, 2 jb) of T
  auto read_tt = [&](int off, int f, int is) { return lds_tr2(ad.tt[0], ad.tt[1], off + 1024 * f + 256 * (is & 1)); };
  const int pos = gdn_saved_lane(lane);
  bf16x8* const ds1_out = (bf16x8*)a.sv.ds1 + (op * 4 + w) * 512 + pos;
  bf16x8* const dr_out = (bf16x8*)a.sv.drs + (op * 4 + w) * 256 + pos;

  constexpr int RING = 8;
  // ---- K dS1 (rows = tokens, columns = value columns); dO as an operand, as it is and with its rows scaled ----
  bf16x8 fk[RING], of[4], os[4], pf[6], qf[4][4];
  f32x16 dv[2];                         // K dS1, then dVn, then dR
  f32x4 el[8];
  const float glast = *(TT_LDS(const float)*)(ad.eg - 4u * c + R_EG + 4 * (GC - 1));
#pragma unroll
  for (int js = 0; js < 4; js++) of[js] = lds_tr2(ad.vt[0], ad.vt[1], 16 * js * TILE_ROW * 2);
#pragma unroll
  for (int i = 0; i < RING; i++) fk[i] = read_row(i);
  if (len < GC) {                       // rows of dO past the chunk's length (copies of its last row) count as zero
#pragma unroll
    for (int js = 0; js < 4; js++)
#pragma unroll
      for (int e = 0; e < 8; e++)
        if (16 * js + 8 * (e >> 2) + 4 * hf + (e & 3) >= len) of[js][e] = (__bf16)0.f;
  }
  fence();
#pragma unroll
  for (int i = 0; i < 16; i++) {
    dv[i & 1] = mfma32(fk[i % RING], sb[i >> 1], i < 2 ? zero16() : dv[i & 1]);
    if (i + RING < 16) fk[i % RING] = read_row(i + RING);
    if (i == 2) sb[6] = cvt_regs(s[3], 0);
    if (i == 3) sb[7] = cvt_regs(s[3], 8);
    if (i >= 4 && i < 14) {
#pragma unroll
      for (int r = 0; r < 64; r++)
        if (r * 10 / 64 == i - 4) s[r >> 4][r & 15] *= glast;
    }
    if (i >= 8) ds1_out[64 * (i - 8)] = sb[i - 8];
    if (i < 8) el[i] = read_rows(R_EG, i);
    if (i >= 4 && i < 12 && i % 2 == 1) {
      const int js = (i - 4) >> 1;
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; e++) x[e] = (a.scale * el[2 * js + (e >> 2)][e & 3]) * (float)of[js][e];
      os[js] = cvt8(x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]);
    }
    if (i >= 8 && i < 14) pf[i - 8] = read_frag(R_P, i - 8);
    if (i >= 12) qf[i - 12][0] = read_qt(i - 12, 0);
    if (i & 1) copies(i >> 1, 1);
    fence();
  }
  // ---- dS0 = exp(gamma_last) dS1 + Q^T (scaled dO) ..; beside it dVn = exp(gamma_last - gamma) * (K dS1) + P^T dO ----
#pragma unroll
  for (int i = 0; i < 4; i++) el[i] = read_rows(R_EL, i);
  bf16x8 df[4], th[6], tl[6], kf[4][4];
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const int js = i >> 2, kt = i & 3;
    s[kt] = mfma32(qf[kt][js], os[js], s[kt]);
    if (js < 3) qf[kt][js + 1] = read_qt(kt, js + 1);
    if (i < 4) el[4 + i] = read_rows(R_EL, 4 + i);
    if (i >= 2 && i < 10) {
#pragma unroll
      for (int e = 0; e < 4; e++) dv[(i - 2) >> 2][4 * ((i - 2) & 3) + e] *= el[i - 2][e];
    }
    if (i == 6) dv[0] = mfma32(pf[0], of[0], dv[0]);
    if (i == 7) dv[0] = mfma32(pf[1], of[1], dv[0]);
    if (i == 8) dv[0] = mfma32(pf[2], of[2], dv[0]);
    if (i == 9) dv[0] = mfma32(pf[3], of[3], dv[0]);
    if (i == 10) dv[1] = mfma32(pf[4], of[2], dv[1]);
    if (i == 11) dv[1] = mfma32(pf[5], of[3], dv[1]);
    if (i == 12) df[0] = cvt_regs(dv[0], 0);
    if (i == 13) df[1] = cvt_regs(dv[0], 8);
    if (i == 14) df[2] = cvt_regs(dv[1], 0);
    if (i == 15) df[3] = cvt_regs(dv[1], 8);
    if (i & 1) copies(8 + (i >> 1), 1);
    if (i >= 10) { th[i - 10] = read_tt(R_THI, i < 12 ? 0 : i < 14 ? 2 : 4, i & 1); tl[i - 10] = read_tt(R_TLO, i < 12 ? 0 : i < 14 ? 2 : 4, i & 1); }
    fence();
  }
  // ---- dR = dVn + (T - I)^T dVn: fragments 0 .. 3 of T^T are (0, 0) .. (0, 3), 4 and 5 are (1, 2) and (1, 3) ----
  dv[1] = mfma32(th[4], df[2], dv[1]);   kf[0][0] = read_kt(0, 0); copies(16, 1);                 fence();
  dv[0] = mfma32(th[0], df[0], dv[0]);   kf[1][0] = read_kt(1, 0);                                fence();
  dv[1] = mfma32(th[5], df[3], dv[1]);   kf[2][0] = read_kt(2, 0);                                fence();
  dv[0] = mfma32(th[1], df[1], dv[0]);   kf[3][0] = read_kt(3, 0);                                fence();
  dv[1] = mfma32(tl[4], df[2], dv[1]);   kf[0][1] = read_kt(0, 1);                                fence();
  dv[0] = mfma32(th[2], df[2], dv[0]);   kf[1][1] = read_kt(1, 1);                                fence();
  dv[1] = mfma32(tl[5], df[3], dv[1]);   kf[2][1] = read_kt(2, 1);                                fence();
  dv[0] = mfma32(th[3], df[3], dv[0]);   kf[3][1] = read_kt(3, 1); el[4] = read_rows(R_BEG, 4); el[5] = read_rows(R_BEG, 5); fence();
  dv[0] = mfma32(tl[0], df[0], dv[0]);   el[6] = read_rows(R_BEG, 6); el[7] = read_rows(R_BEG, 7); fence();
  dv[0] = mfma32(tl[1], df[1], dv[0]);   el[0] = read_rows(R_BEG, 0); el[1] = read_rows(R_BEG, 1); fence();
  dv[0] = mfma32(tl[2], df[2], dv[0]);   el[2] = read_rows(R_BEG, 2); el[3] = read_rows(R_BEG, 3); fence();
  bf16x8 ds[4];
  auto put_r = [&](int js) {
    const f32x16& t = dv[js >> 1];
    const int r = 8 * (js & 1);
    const f32x4 e0 = el[2 * js], e1 = el[2 * js + 1];
    dr_out[64 * js] = cvt_regs(t, r);
    ds[js] = cvt8(-e0[0] * t[r], -e0[1] * t[r + 1], -e0[2] * t[r + 2], -e0[3] * t[r + 3], -e1[0] * t[r + 4], -e1[1] * t[r + 5],
                  -e1[2] * t[r + 6], -e1[3] * t[r + 7]);
  };
  dv[0] = mfma32(tl[3], df[3], dv[0]);   put_r(2);                                                fence();
  // ---- .. - K^T (scaled dR) ----
  put_r(3);
#pragma unroll
  for (int kt = 0; kt < 4; kt++) { kf[kt][2] = read_kt(kt, 2); kf[kt][3] = read_kt(kt, 3); }
  fence();
#pragma unroll
  for (int kt = 0; kt < 4; kt++) {
    s[kt] = mfma32(kf[kt][2], ds[2], s[kt]);
    if (kt == 0) put_r(0);
    if (kt == 2) put_r(1);
    fence();
  }
#pragma unroll
  for (int kt = 0; kt < 4; kt++) { s[kt] = mfma32(kf[kt][3], ds[3], s[kt]); fence(); }
#pragma unroll
  for (int kt = 0; kt < 4; kt++) {
    s[kt] = mfma32(kf[kt][0], ds[0], s[kt]);
    if (kt >= 2) sb[2 * kt - 4] = cvt_regs(s[kt - 2], 0);
    fence();
    s[kt] = mfma32(kf[kt][1], ds[1], s[kt]);
    if (kt >= 2) sb[2 * kt - 3] = cvt_regs(s[kt - 2], 8);
    fence();
  }
  sb[4] = cvt_regs(s[2], 0); sb[5] = cvt_regs(s[2], 8);
}

template <int WAVES>
__global__ __launch_bounds__(G_THREADS, 1) void gdn_rwalk_kernel(GdnArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char sm[SCAN_LDS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = WAVES < 4 ? (int)blockIdx.x / a.hv_n : 0;
  const int w = wave + WAVES * half;
  const int h = walk_head(a, blockIdx.x - half * a.hv_n);
  ChunkMeta meta;
  int seg, c_begin, c_end;
  walk_start<true>(a, half, lane, meta, seg, c_begin, c_end);
  const int last = c_end - 1;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&sm);
  if (WAVES < 4 && wave >= WAVES) {
    walk_copies<WALK_REV>(a, meta, lds, h, last, c_end - c_begin, wave - WAVES, lane);
    return;
  }
  ScanAddr ad;
  ad.set(lds, lane, w);
  std::conditional_t<WAVES == 4, ChunkCopy<WALK_REV, 4>, NoCopy> copy;
  if constexpr (WAVES == 4) {
    copy.start(a, h, ad.rec);
    copy.point(last, meta.get(meta.tok0, last), meta.get(meta.len, last) & 255, w, lane);
#pragma unroll
    for (int p = 0; p < copy.N; p++) copy.piece(p, w, lane);
  }
  // The gradient of the state a segment's last chunk leaves starts from zero; so does, walking all chunks in sequence, that of a
  // chunk whose successor in the sequence did not continue from it.
  ScanState st;
  st.zero();
  st.round();
  bool fresh = false;
  int sign = 1;                         // where the other image lies
  auto step = [&](int chunk) {
    const int bits = meta.get(meta.len, chunk);
    const int src = meta.get(meta.src, chunk);
    if (fresh || (bits & ChunkMeta::LEAVES)) {
      if (fresh) st.zero();
      const int dst = meta.get(meta.dst, chunk), cap = meta.get(meta.cap, chunk);
      if (dst >= 0) {
        if (a.seg_chunk0) {
          // scheduled walk: every segment that started from this slot (all of later levels) stores the gradient of its
          // entering state; they are added in the order of the slot's reader list
          const int k1 = a.slot_cons_off[dst + 1];
          for (int k = a.slot_cons_off[dst]; k < k1; k++) {
            const int reader = a.slot_cons[k];
            const bool stored = ScanState::wait_for(a, a.seg_sync, reader, h, w);
            st.add<true>(a.sv.seg_grad + ((size_t)reader * a.hv + h) * (GD * GD), lane, w);
            if (!stored) st.spoil();
          }
        } else {
          st.add<true>(a.sv.slot_grad + ((size_t)dst * a.hv + h) * (GD * GD), lane, w);
        }
      }
      if (cap >= 0 && a.d_state_out) st.add<false>(a.d_state_out + ((size_t)cap * a.hv + h) * (GD * GD), lane, w);
      st.round();
    }
    const bool has_next = chunk > c_begin;
    if (has_next) {
      if (chunk == meta.first) meta.load(a, max(chunk - 64, 0), lane);
      if constexpr (WAVES == 4) copy.point(chunk - 1, meta.get(meta.tok0, chunk - 1), meta.get(meta.len, chunk - 1) & 255, w, lane);
    }
    if constexpr (WAVES == 4) {
      walk_barrier();
      copy.other_image(sign);
    } else {
      walker_barrier();
    }
    rwalk_step(a, st, ad, copy, has_next, op_index(a, chunk, h), bits & 255, w, lane);
    fresh = src != -2;
    if (src >= 0 || (src == -1 && a.d_initial_state)) {
      if (a.seg_chunk0) {
        // scheduled walk: this is the first chunk of segment `seg`; its entering state's gradient is stored in the
        // segment's own array -- the slot's saver, or the sum over the roots, picks it up
        st.put<true>(a.sv.seg_grad + ((size_t)seg * a.hv + h) * (GD * GD), lane, w);
        ScanState::publish(a, a.seg_sync, seg, h, lane, w);
      } else if (src >= 0) {
        float* g = a.sv.slot_grad + ((size_t)src * a.hv + h) * (GD * GD);
        st.add<true>(g, lane, w);
        st.put<true>(g, lane, w);
      } else {
        float* g = a.d_initial_state + (size_t)h * (GD * GD);
        st.add<false>(g, lane, w);
        st.put<false>(g, lane, w);
      }
    }
    ad.other_image(sign);
    sign = -sign;
  };
  for (int chunk = last; chunk >= c_begin; chunk--) step(chunk);
}

// d_initial_state = sum over the root segments (level 0, in order) of the gradients they stored, 2 registers of a lane at a time
__global__ __launch_bounds__(G_THREADS) void gdn_root_grad_kernel(const float* __restrict__ seg_grad, int n_roots, int hv, int hv_n,
                                                                  float* __restrict__ d_initial_state) {
  const size_t n2 = (size_t)hv_n * (GD * GD / 2), seg_stride = (size_t)hv * GD * GD;
  for (size_t i = (size_t)blockIdx.x * G_THREADS + threadIdx.x; i < n2; i += (size_t)gridDim.x * G_THREADS) {
    float x = 0.f, y = 0.f;
    for (int r = 0; r < n_roots; r++) {
      const float2 v = *(const float2*)(seg_grad + (size_t)r * seg_stride + 2 * i);
      x += v.x; y += v.y;
    }
    const int e = (int)(i % (GD * GD / 2)), lane = e & 63, r = 2 * ((e >> 6) & 7), kt = (e >> 9) & 3, w = e >> 11;
    float* out = d_initial_state + (i / (GD * GD / 2)) * (GD * GD) + (8 * (lane >> 5)) * GD + 32 * w + (lane & 31);
    out[(32 * kt + state_dim(r, 0)) * GD] = x;
    out[(32 * kt + state_dim(r + 1, 0)) * GD] = y;
  }
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t gdn_workspace(int n_chunks, int n_slots, int hv) {
  return align256((size_t)n_chunks * hv * REC_ELEMS * 2) + align256((size_t)n_slots * hv * GD * GD * 4) + align256((size_t)n_slots * hv * 16) + 256;
}

// Walks the chunk program: one workgroup per head and segment, segments in level order (without a schedule one segment).  The
// levels are kept by the flags and tickets, not by launches: a launch per level cost 3 to 5 us each, and short segments stood still for the
// longest of their level (16406 tokens of 16 / 32 heads, 4 levels: forward 286 -> 254 us, backward 959 -> 918; 1500 tokens in 8
// levels, 4 / 8 heads: backward 280 -> 256).
//
// The backward's walks put a head on two workgroups of two waves, and two that copy for them (walk_copies), as long as the walks of the
// widest level all run side by side like that: a wave shares the LDS with one other instead of three.  Against the form before (a head on two
// workgroups of eight waves that exchange the state through LDS) / two waves that copy for themselves / this: chains of 1500, 4000, 8000 tokens of
// 8 heads 198 / 227 / 197, 314 / 367 / 304, 508 / 588 / 485 us; 16384 tokens of 32 heads 1752 / 1485 / 1441.  Four waves / this in levels of
// 104 walks 224 / 197, of 128 371 / 337 and 203 / 186.  (Levels of 256 walks were 2 to 3 % slower with two waves, and so is the
// scan everywhere.)
constexpr int NARROW_WALKS = 128;      // widest level, in walks (segments x heads)
template <class Kernel>
static hipError_t launch_walk(Kernel kernel4, Kernel kernel2, GdnArgs& a, const tt_gdn_schedule* sched, hipStream_t st) {
  int widest = 1;
  for (int l = 0; sched && l < sched->n_levels; l++) widest = std::max(widest, sched->level_off[l + 1] - sched->level_off[l]);
  const int waves = kernel2 && (int64_t)widest * a.hv_n <= NARROW_WALKS ? 2 : 4;
  const Kernel kernel = waves == 4 ? kernel4 : kernel2;
  const unsigned heads = (unsigned)(a.hv_n * (4 / waves));      // x: heads, or heads of the lower and then of the upper columns
  a.seg_base = 0;
  if (!sched) {
    a.seg_chunk0 = a.seg_chunk1 = nullptr; a.n_segments = 1; a.n_levels = 0;
    kernel<<<dim3(heads, 1), G_THREADS, 0, st>>>(a);
    return hipGetLastError();
  }
  a.seg_chunk0 = sched->seg_chunk0; a.seg_chunk1 = sched->seg_chunk1; a.n_segments = sched->n_segments;
  a.n_levels = sched->n_levels <= WALK_LEVELS ? sched->n_levels : 0;
  for (int l = 0; a.n_levels > 0 && l <= a.n_levels; l++) a.level_off[l] = sched->level_off[l];
  constexpr int MAX_Y = 65535;          // blocks of a launch along y
  for (; a.seg_base < a.n_segments; a.seg_base += MAX_Y) {
    const int n = a.n_segments - a.seg_base;
    kernel<<<dim3(heads, (unsigned)(n < MAX_Y ? n : MAX_Y)), G_THREADS, 0, st>>>(a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// (Without saved states nobody waits, and no places are counted.)
static void set_sync(GdnArgs& a, void* sync, int n_slots, int n_segments, const tt_gdn_schedule* sched) {
  a.slot_sync = (WalkSync*)sync;
  a.seg_sync = a.slot_sync + (size_t)n_slots * a.hv_n;
  a.n_sync = sched ? (n_slots + n_segments) * a.hv_n : 0;
  a.tickets = sched && n_slots > 0 ? a.slot_sync : nullptr;
  a.max_polls = (1 << 18) + 256 * a.n_chunks;       // (a poll takes 1 us and more)
}

hipError_t gdn_fwd(int64_t n_tokens, int hk, int hv, float scale, const void* q, const void* k, const void* v, const float* g,
                   const float* beta, int n_chunks, const int32_t* chunk_tok0, const int32_t* chunk_len, const int32_t* chunk_src,
                   const int32_t* chunk_dst, int n_slots, const int32_t* chunk_cap, const tt_gdn_schedule* sched,
                   const float* initial_state, float* state_out, void* o, void* workspace, hipStream_t st) {
  if (n_chunks == 0) return hipSuccess;
  GdnArgs a{};
  a.hk = hk; a.hv = hv; a.hk_n = hk; a.n_chunks = n_chunks; a.scale = scale;
  a.q = (const __bf16*)q; a.k = (const __bf16*)k; a.v = (const __bf16*)v; a.g = g; a.beta = beta;
  a.chunk_tok0 = chunk_tok0; a.chunk_len = chunk_len; a.chunk_src = chunk_src; a.chunk_dst = chunk_dst;
  a.chunk_cap = chunk_cap; a.initial_state = initial_state; a.state_out = state_out;
  a.o = (__bf16*)o;
  a.rec = (__bf16*)workspace;
  a.slots = (float*)((char*)workspace + align256((size_t)n_chunks * hv * REC_ELEMS * 2));
  a.hv_n = hv;
  set_sync(a, (char*)a.slots + align256((size_t)n_slots * hv * GD * GD * 4), n_slots, 0, sched);
  {
    KernelTimer t(TT_KERNEL_GDN_PREPARE, st);
    gdn_prepare_kernel<false><<<(unsigned)n_chunks * (unsigned)hk, G_THREADS, 0, st>>>(a);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  KernelTimer t(TT_KERNEL_GDN_SCAN, st);
  return launch_walk<void (*)(GdnArgs)>(gdn_scan_kernel, nullptr, a, sched, st);
}

hipError_t gdn_bwd_prepare_and_walks(const GdnBwdArgs& b, const GdnBwdSaved& sv, hipStream_t st) {
  if (b.n_chunks == 0) return hipSuccess;
  GdnArgs a{};
  a.hk = b.hk; a.hv = b.hv; a.hk_n = b.hv_n / (b.hv / b.hk); a.n_chunks = b.n_chunks; a.scale = b.scale;
  a.q = (const __bf16*)b.q; a.k = (const __bf16*)b.k; a.v = (const __bf16*)b.v; a.g = b.g; a.beta = b.beta;
  a.chunk_tok0 = b.chunk_tok0; a.chunk_len = b.chunk_len; a.chunk_src = b.chunk_src; a.chunk_dst = b.chunk_dst;
  a.initial_state = b.initial_state;
  a.rec = (__bf16*)sv.rec; a.slots = sv.slots; a.sv = sv; a.d_o = (const __bf16*)b.d_o;
  a.d_state_out = b.d_state_out; a.d_initial_state = b.d_initial_state;
  a.hv_n = b.hv_n;
  set_sync(a, sv.sync, b.n_slots, b.sched ? b.sched->n_segments : 0, b.sched);
  {
    KernelTimer t(TT_KERNEL_GDN_PREPARE, st);
    gdn_prepare_kernel<true><<<(unsigned)b.n_chunks * (unsigned)a.hk_n, G_THREADS, 0, st>>>(a);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  {
    KernelTimer t(TT_KERNEL_GDN_BWD_FSCAN, st);
    if (hipError_t e = launch_walk(gdn_fwalk_kernel<4>, gdn_fwalk_kernel<2>, a, b.sched, st); e != hipSuccess) return e;
  }
  a.chunk_cap = b.d_state_out ? b.chunk_cap : nullptr;
  if (a.tickets) a.tickets = a.seg_sync;
  KernelTimer t(TT_KERNEL_GDN_BWD_RSCAN, st);
  if (b.sched) { a.slot_cons_off = b.sched->slot_cons_off; a.slot_cons = b.sched->slot_cons; }
  if (hipError_t e = launch_walk(gdn_rwalk_kernel<4>, gdn_rwalk_kernel<2>, a, b.sched, st); e != hipSuccess) return e;
  if (b.sched && b.d_initial_state && b.sched->n_levels > 0)
    gdn_root_grad_kernel<<<256, G_THREADS, 0, st>>>(sv.seg_grad, b.sched->level_off[1], b.hv, b.hv_n, b.d_initial_state);
  return hipGetLastError();
}

}  // namespace tt
