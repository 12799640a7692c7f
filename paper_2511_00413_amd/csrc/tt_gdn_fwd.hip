// Gated delta rule with tree state routing, forward (Section "Implementation", paragraph "SSM Layers
// (GDN)" (i); Appendix "Tree-Aware SSM State Routing"): the recurrent state at a node's first token
// is the end state of its parent node, not of the previous node in DFS order.
//
// Chunked form, 64 tokens per chunk, chunks never cross a node boundary.  With gamma_i the running
// sum of the log-decays inside a chunk, beta the write strengths and S0 the state entering the chunk:
//     A  = strictly-lower( beta_i (k_i . k_j) exp(gamma_i - gamma_j) ),      T = (I + A)^-1
//     R  = beta * V - (beta exp(gamma)) * (K S0)                             (rows scaled)
//     Vn = T R
//     O  = (scale exp(gamma)) * (Q S0) + scale tril( (Q K^T) * exp(gamma_i - gamma_j) ) Vn
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
#include <hip/hip_runtime.h>
#include <type_traits>
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
// = column 4 hf + 8 (e / 4) + e % 4), row block 0 first: (0, 0), (0, 1), (1, 0) .. (1, 3).
constexpr int FRAG = 512;                                        // bf16 elements of a fragment
constexpr int REC_THI = 0, REC_TLO = 6 * FRAG;                   // T - I as two bf16 halves (relative error 2^-17)
constexpr int REC_ROW = 12 * FRAG;                               // fp32 rows of 64: beta, beta exp(gamma), exp(gamma_last - gamma), exp(gamma)
constexpr int REC_P = REC_ROW + 2 * 4 * GC;                      // tril((q_i . k_j) scale exp(gamma_i - gamma_j))
constexpr int REC_ELEMS = REC_P + 6 * FRAG;                      // 19 KB
static_assert(REC_ELEMS * 2 == 19 * 1024, "whole 1 KB pieces");

struct GdnArgs {
  int n_tokens, hk, hv, n_chunks;    // hk, hv: heads of the tensors (their strides)
  float scale;
  const __bf16 *q, *k, *v;           // [N][hk][128], [N][hk][128], [N][hv][128]
  const float *g, *beta;             // [N][hv]
  const int32_t *chunk_tok0, *chunk_len, *chunk_src, *chunk_dst;
  const int32_t* chunk_cap;          // nullptr, or per chunk: -1 / index into state_out
  const int32_t *seg_chunk0, *seg_chunk1;   // nullptr (one segment: all chunks), or the chunk ranges of the segments
  int seg_base;                      // first segment of the level this launch walks (blockIdx.y counts from it)
  const float* initial_state;        // nullptr (zero) or [hv][128][128]: the state roots start from
  float* state_out;                  // [n_capture][hv][128][128]
  __bf16* o;                         // [N][hv][128]
  __bf16* rec;                       // [hv][n_chunks][REC_ELEMS]
  float* slots;                      // [n_slots][hv][128][128] saved node-end states
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
__global__ __launch_bounds__(G_THREADS, 3) void gdn_prepare_kernel(GdnArgs a) {
  __shared__ __attribute__((aligned(1024))) PrepSmem sm;
  const int rep = a.hv / a.hk;
  int chunk, kh;
  if (!gdn_group_order(blockIdx.x, a.n_chunks, a.hk, 1, chunk, kh)) return;
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
  };
  row_factors(0);
  dma_wait_all();
  __syncthreads();

  // K K^T and Q K^T, one 32 x 32 tile of the lower triangle per wave (wave 3: none): rows = j, columns (lanes) = i
  const int ib = (w + 1) >> 1, jb = w >> 1;
  f32x16 kk = zero16(), qk = zero16();
  if (w < 3) {
    const int base = row_frag_base(lane);
#pragma unroll
    for (int ks = 0; ks < GD / 16; ks++) {
      const bf16x8 kj = lds_row_frag(sm.k, base, jb, ks);
      kk = mfma32(kj, lds_row_frag(sm.k, base, ib, ks), kk);
      qk = mfma32(kj, lds_row_frag(sm.q, base, ib, ks), qk);
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
            p[r] = j <= i ? a.scale * qk[r] * dec : 0.f;
          }
        }
        // fragments (ib, 2 jb) and (ib, 2 jb + 1): the accumulator's registers as they stand
        __bf16* out = a.rec + op_index(a, chunk, kh * rep + r0 + hh) * REC_ELEMS + REC_P + (2 * ib + 2 * jb) * FRAG + 8 * lane;
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
      __bf16* out = a.rec + op_index(a, chunk, kh * rep + r0 + hh) * REC_ELEMS + 8 * lane;
      auto put = [&](int f, const float (&t)[8]) {
        const bf16x8 hi = cvt8(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7]);
        *(bf16x8*)(out + REC_THI + f * FRAG) = hi;
        *(bf16x8*)(out + REC_TLO + f * FRAG) = cvt8(t[0] - (float)hi[0], t[1] - (float)hi[1], t[2] - (float)hi[2], t[3] - (float)hi[3],
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

// The copies of one chunk's operands, 17 pieces of 1 KB per wave.  They are requested one by one between the products of the
// chunk before (dma_piece): a compute unit takes them at about 30 cycles each, and a wave that requests them all at once stands
// still for 2000 of a step's 7000 cycles.
constexpr int N_PIECES = 17;
struct ChunkCopy {
  const char *k0, *q0, *v0, *rec0;      // of token 0 / chunk 0: K and Q of the key head, V of the value head, the records of the head
  uint32_t k_row, v_row;                // bytes per token
  const char *k, *q, *v, *rec;
  uint32_t kv[4], vv[4];                // this lane's byte offsets in the rows of K / Q and of V
  int len;
  __device__ __forceinline__ void point(int chunk, int tok0, int new_len, int w, int lane) {
    const uint64_t krow = (uint64_t)(uint32_t)tok0 * k_row;
    k = k0 + krow;
    q = q0 + krow;
    v = v0 + (uint64_t)(uint32_t)tok0 * v_row;
    rec = rec0 + (uint64_t)(uint32_t)chunk * REC_B;
    if (new_len == len) return;
    len = new_len;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int r4 = 4 * w + u, lr = lane >> 4;                   // as dma_tile64: 4 rows per piece, 16-byte chunks permuted
      const uint32_t row = (uint32_t)min(4 * r4 + lr, len - 1), col = 16u * (uint32_t)((lane & 15) ^ ((lr << 2) | (r4 & 3)));
      kv[u] = row * k_row + col;
      vv[u] = row * v_row + col;
    }
  }
  __device__ __forceinline__ void piece(int p, int buf, uint32_t lds, int w, int lane) const {
    const int u = p & 3;
    if (p < 12) {
      const int tile = p < 4 ? L_K : p < 8 ? L_Q : L_V;
      dma16(p < 4 ? k : p < 8 ? q : v, p < 8 ? kv[u] : vv[u], lds + tile + buf * TILE_B + (4 * w + u) * 1024);
    } else {
      const int i = min(4 * (p - 12) + w, REC_B / 1024 - 1);      // (the last one twice)
      dma16(rec + 1024 * i, 16u * lane, lds + L_REC + buf * REC_B + 1024 * i);
    }
  }
};

// LDS byte addresses of this lane's fragments in the first image
struct ScanAddr {
  uint32_t row[8];      // rows of K as operands, k-step ks (row block, tile, image: immediate offsets)
  uint32_t kt[4][2];    // K transposed, 32 key dims kt
  uint32_t vt[2];       // V transposed, this wave's 32 columns
  uint32_t rec, frag, sc, eg;
};

// Which key dims of a 32-row state tile an accumulator register holds.  Rows of the tile are key dims in an order in which the
// 8 rows that make up a lane's share of a 16-deep operand are 8 consecutive key dims, so that the rows of K and Q meet them
// as plain 16-byte reads: tile row 16 t + 8 a + 4 h + b is key dim 16 t + 8 h + 4 a + b.
__device__ __forceinline__ int state_dim(int r, int hf) { return 16 * (r >> 3) + 8 * hf + 4 * ((r >> 2) & 1) + (r & 3); }

__device__ __forceinline__ bf16x8 cvt_regs(const f32x16& t, int r) {
  return cvt8(t[r], t[r + 1], t[r + 2], t[r + 3], t[r + 4], t[r + 5], t[r + 6], t[r + 7]);
}

struct ScanState {
  f32x16 s[4];          // key dims 32 kt + state_dim(r), this wave's column c
  bf16x8 sb[8];         // the same rounded, as an operand: lane = value column, k = key dims 16 ks + 8 hf ..  (6, 7: formed inside the step)
};

// One chunk.  On entry the copy of its operands into image BUF is in flight.  The matrix instructions are a sequence of slots,
// each with a share of the reads, the arithmetic and the next chunk's copies, closed by a scheduling fence.  A wave is alone on its
// SIMD, so that nothing else fills a gap: what counts is the number of instructions (about 4 cycles each) and that none waits.
template <int BUF>
__device__ __forceinline__ void scan_step(const GdnArgs& a, ScanState& st, const ScanAddr& ad, const ChunkCopy& copy, bool has_next, int tok0,
                                          int len, int h, int w, int lane, const uint32_t (&o_at)[2]) {
  const int c = lane & 31;
  f32x16(&s)[4] = st.s;
  bf16x8(&sb)[8] = st.sb;
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  auto copies = [&](int p, int n) {
    if (has_next) {
#pragma unroll
      for (int i = p; i < p + n; i++) copy.piece(i, BUF ^ 1, ad.rec, w, lane);
    }
  };
  auto read_row = [&](int i, int tile) { return lds_b128(ad.row[i >> 1], tile + BUF * TILE_B + (i & 1) * 32 * TILE_ROW * 2); };
  auto read_kt = [&](int kt, int js) { return lds_tr2(ad.kt[kt][0], ad.kt[kt][1], L_K + BUF * TILE_B + 16 * js * TILE_ROW * 2); };
  auto read_frag = [&](int off, int f) { return lds_b128(ad.frag, BUF * REC_B + off + 1024 * f); };
  auto read_rows = [&](int arr, int grp) { return *(TT_LDS(const f32x4)*)(ad.sc + BUF * REC_B + arr + 32 * grp); };

  // Fragments are requested eight slots and more ahead: an LDS round trip takes about 250 cycles while the other waves read and
  // the copies land.
  constexpr int RING = 8;
  // ---- K S0 (rows = tokens, columns = value columns); the state is scaled beside it ----
  bf16x8 fk[RING], fq[RING], vf[4], th[6], tl[6];
  f32x16 vn[2], qs[2];                  // vn: K S0, then R, then Vn
  f32x4 b4[2], g4[2], el[4];
  auto rows_r = [&](int grp) { b4[grp & 1] = read_rows(R_BETA, grp); g4[grp & 1] = read_rows(R_BEG, grp); };
  const float glast = *(TT_LDS(const float)*)(ad.eg - 4u * c + BUF * REC_B + R_EG + 4 * (GC - 1));
#pragma unroll
  for (int i = 0; i < RING; i++) fk[i] = read_row(i, L_K);
  float eg0 = *(TT_LDS(const float)*)(ad.eg + BUF * REC_B + R_EG), eg1 = *(TT_LDS(const float)*)(ad.eg + BUF * REC_B + R_EG + 128);
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
    if (i >= 8 && i < 12) vf[i - 8] = lds_tr2(ad.vt[0], ad.vt[1], BUF * TILE_B + 16 * (i - 8) * TILE_ROW * 2);
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
    if (i >= 2 && i < 8) th[i - 2] = read_frag(R_THI, i - 2);
    if (i >= 8 && i < 14) tl[i - 8] = read_frag(R_TLO, i - 8);
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
// takes 2.7 us (3.1 with the operands of all heads requested at its start, 3.3 in the form before, which cut a head into two
// workgroups of eight waves that exchanged the state and Vn through LDS, and needed two workgroup steps per chunk and head for it): all levels of
// 16406 tokens of 32 heads 200 us, 265 before, with 67 KB instead of 128 per chunk and head from memory.  Two waves per column block, one for the chain
// K S0 -> Vn and one for the output, half of the state's rows each: 204 us.
__global__ __launch_bounds__(G_THREADS, 1) void gdn_scan_kernel(GdnArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char sm[SCAN_LDS];
  const int lane = threadIdx.x & 63, c = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rep = a.hv / a.hk;
  // Consecutive workgroups go round-robin over the 8 XCDs; the value heads of a key head read the same q and k rows, so
  // they are given ids 8 apart and share one XCD's L2.
  const int id = blockIdx.x;
  const int h = a.hk % 8 == 0 ? ((id >> 3) / rep * 8 + (id & 7)) * rep + (id >> 3) % rep : id;
  const int kh = h / rep;
  const int seg = a.seg_base + blockIdx.y;
  const int c_begin = a.seg_chunk0 ? a.seg_chunk0[seg] : 0;
  const int c_end = a.seg_chunk1 ? a.seg_chunk1[seg] : a.n_chunks;

  ScanAddr ad;
  ad.rec = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&sm);
  {
    const int rd = row_frag_base(lane);
#pragma unroll
    for (int ks = 0; ks < 8; ks++) ad.row[ks] = ad.rec + 2u * (uint32_t)(rd ^ (ks << 4));
    const TrBase tr = tr_frag_base(lane);
    ad.vt[0] = ad.rec + L_V + 2u * (uint32_t)(tr.x0 ^ (w << 5));
    ad.vt[1] = ad.rec + L_V + 2u * (uint32_t)(tr.x1 ^ (w << 5));
    // K: the two middle groups of 4 of every 16 columns change places (state_dim)
    const TrBase kr = tr_frag_base((lane & ~3) | ((lane & 1) << 1) | ((lane >> 1) & 1));
#pragma unroll
    for (int t = 0; t < 4; t++) {
      ad.kt[t][0] = ad.rec + 2u * (uint32_t)(kr.x0 ^ (t << 5));
      ad.kt[t][1] = ad.rec + 2u * (uint32_t)(kr.x1 ^ (t << 5));
    }
    ad.frag = ad.rec + L_REC + 16u * lane;
    ad.sc = ad.rec + L_REC + 16u * hf;
    ad.eg = ad.rec + L_REC + 4u * c;
    // (opaque: with known parts the compiler folds them into offsets past 64 KB and adds them up again at every read)
    asm volatile("" : "+v"(ad.frag), "+v"(ad.sc), "+v"(ad.eg), "+v"(ad.vt[0]), "+v"(ad.vt[1]));
  }
  const uint32_t o_at[2] = {(uint32_t)c * (uint32_t)a.hv * (GD * 2) + 16u * hf, (uint32_t)(32 + c) * (uint32_t)a.hv * (GD * 2) + 16u * hf};
  ChunkMeta meta;
  meta.load(a, c_begin, lane);
  ChunkCopy copy;
  copy.k0 = (const char*)(a.k + (size_t)kh * GD);
  copy.q0 = (const char*)(a.q + (size_t)kh * GD);
  copy.v0 = (const char*)(a.v + (size_t)h * GD);
  copy.rec0 = (const char*)(a.rec + op_index(a, 0, h) * REC_ELEMS);
  copy.k_row = (uint32_t)a.hk * (GD * 2);
  copy.v_row = (uint32_t)a.hv * (GD * 2);
  copy.len = 0;
  copy.point(c_begin, meta.get(meta.tok0, c_begin), meta.get(meta.len, c_begin) & 255, w, lane);
#pragma unroll
  for (int p = 0; p < N_PIECES; p++) copy.piece(p, 0, ad.rec, w, lane);
  // this lane's first element of a [128][128] state (opaque: the 64 offsets from it are formed where they are used, not kept)
  auto state_at = [&]() {
    int at = 8 * hf * GD + 32 * w + c;
    asm volatile("" : "+v"(at));
    return at;
  };
  ScanState st;
#pragma unroll
  for (int kt = 0; kt < 4; kt++) st.s[kt] = zero16();

  auto step = [&](auto buf, int chunk) {
    const int tok0 = meta.get(meta.tok0, chunk), bits = meta.get(meta.len, chunk), len = bits & 255;
    const int dst = meta.get(meta.dst, chunk), cap = meta.get(meta.cap, chunk);
    if (bits & ChunkMeta::ENTERS) {
      const int src = meta.get(meta.src, chunk);
      if (src == -1 && !a.initial_state) {
#pragma unroll
        for (int kt = 0; kt < 4; kt++) st.s[kt] = zero16();
      } else {
        // a saved node-end state, or the state handed in for the roots
        const float* sp = (src >= 0 ? a.slots + ((size_t)src * a.hv + h) * (GD * GD) : a.initial_state + (size_t)h * (GD * GD)) + state_at();
#pragma unroll
        for (int kt = 0; kt < 4; kt++)
#pragma unroll
          for (int r = 0; r < 16; r++) st.s[kt][r] = sp[(32 * kt + state_dim(r, 0)) * GD];
#pragma unroll
        for (int kt = 0; kt < 4; kt++) pin(st.s[kt]);     // the wait for these loads belongs inside this (rare) branch, not at the merge point
      }
#pragma unroll
      for (int ks = 0; ks < 6; ks++) st.sb[ks] = cvt_regs(st.s[ks >> 1], 8 * (ks & 1));
    }
    const bool has_next = chunk + 1 < c_end;
    if (has_next) {
      if (chunk + 1 - meta.first == 64) meta.load(a, chunk + 1, lane);
      copy.point(chunk + 1, meta.get(meta.tok0, chunk + 1), meta.get(meta.len, chunk + 1) & 255, w, lane);
    }
    // this wave's share of the operands has landed, and so has everybody else's; every wave has left the other image
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    scan_step<decltype(buf)::value>(a, st, ad, copy, has_next, tok0, len, h, w, lane, o_at);
    if (bits & ChunkMeta::LEAVES) {
      auto save = [&](float* state) {
        float* sp = state + (size_t)h * (GD * GD) + state_at();
#pragma unroll
        for (int kt = 0; kt < 4; kt++)
#pragma unroll
          for (int r = 0; r < 16; r++) sp[(32 * kt + state_dim(r, 0)) * GD] = st.s[kt][r];
      };
      if (dst >= 0) save(a.slots + (size_t)dst * a.hv * (GD * GD));
      if (cap >= 0) save(a.state_out + (size_t)cap * a.hv * (GD * GD));
    }
  };
  for (int chunk = c_begin; chunk < c_end; chunk += 2) {
    step(std::integral_constant<int, 0>{}, chunk);
    if (chunk + 1 < c_end) step(std::integral_constant<int, 1>{}, chunk + 1);
  }
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t gdn_workspace(int n_chunks, int n_slots, int hv) {
  return align256((size_t)n_chunks * hv * REC_ELEMS * 2) + align256((size_t)n_slots * hv * GD * GD * 4) + 256;
}

hipError_t gdn_fwd(int64_t n_tokens, int hk, int hv, float scale, const void* q, const void* k, const void* v, const float* g,
                   const float* beta, int n_chunks, const int32_t* chunk_tok0, const int32_t* chunk_len, const int32_t* chunk_src,
                   const int32_t* chunk_dst, int n_slots, const int32_t* chunk_cap, const tt_gdn_schedule* sched,
                   const float* initial_state, float* state_out, void* o, void* workspace, hipStream_t st) {
  if (n_chunks == 0) return hipSuccess;
  GdnArgs a{};
  a.n_tokens = (int)n_tokens; a.hk = hk; a.hv = hv; a.n_chunks = n_chunks; a.scale = scale;
  a.q = (const __bf16*)q; a.k = (const __bf16*)k; a.v = (const __bf16*)v; a.g = g; a.beta = beta;
  a.chunk_tok0 = chunk_tok0; a.chunk_len = chunk_len; a.chunk_src = chunk_src; a.chunk_dst = chunk_dst;
  a.chunk_cap = chunk_cap; a.initial_state = initial_state; a.state_out = state_out;
  a.o = (__bf16*)o;
  a.rec = (__bf16*)workspace;
  a.slots = (float*)((char*)workspace + align256((size_t)n_chunks * hv * REC_ELEMS * 2));
  {
    KernelTimer t(TT_KERNEL_GDN_PREPARE, st);
    gdn_prepare_kernel<<<gdn_group_order_grid(n_chunks, hk, 1), G_THREADS, 0, st>>>(a);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  KernelTimer t(TT_KERNEL_GDN_SCAN, st);
  if (!sched) {
    gdn_scan_kernel<<<dim3((unsigned)hv, 1), G_THREADS, 0, st>>>(a);
    return hipGetLastError();
  }
  // one launch per dependency level with the level's segments side by side (blockIdx.y)
  a.seg_chunk0 = sched->seg_chunk0; a.seg_chunk1 = sched->seg_chunk1;
  for (int l = 0; l < sched->n_levels; l++) {
    a.seg_base = sched->level_off[l];
    gdn_scan_kernel<<<dim3((unsigned)hv, (unsigned)(sched->level_off[l + 1] - sched->level_off[l])), G_THREADS, 0, st>>>(a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tt
