// Work decomposition of the dK/dV pass (tt_attn_dkdv.hip), computed beside the dQ pass (tt_attn_bwd.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <algorithm>
#include "tt_kernels.h"

namespace tt {
namespace {

constexpr int KV_D = 128;
constexpr int KV_BN = 256;         // keys per workgroup of the dK/dV pass
constexpr int KV_BM = 64;          // queries per staged tile (one pipeline step)

// ---- work decomposition -------------------------------------------------------------------------
// Key tiles.  A workgroup works on up to KV_BN consecutive keys and walks the (query head, query
// tile) steps of every query tile that can see one of them, so keys with different visibility ranges
// in one tile leave wavefronts idle.  In DFS order the keys of a tree node are consecutive and share
// their range; the planner therefore forms tiles from runs of consecutive 64-key summary entries with
// the same largest bound (kt_max), at most KV_BN / 64 entries per tile, instead of cutting the key
// axis at fixed multiples of KV_BN.
//
// Work items.  A tile's work is its list of steps.  Tiles near the root of the tree are seen by
// almost every query while leaf tiles are seen by few, so a tile's steps are cut into chunks of at
// most `chunk` steps; the planner sizes the chunks so that the launch has about KV_ITEMS_PER_WG work
// items per resident workgroup, workgroups pull items from a counter (longest items first), and tiles that were cut have their fp32 partial
// results summed in chunk order by a reduce kernel (bit-reproducible).
constexpr int KV_TARGET_WORK = 768;      // work items (tile chunk x kv head) aimed for, at most (sizes the plan tables)
constexpr int KV_ITEMS_PER_WG = 2;       // ... and per resident workgroup: with the longest items handed out first two
                                         // per workgroup balance as well as three did in plain order, with 40 % fewer
                                         // partial slots to write and reduce
// Chunks of small trees, in steps.  There a chunk is what gives every workgroup one item, KV_MIN_CHUNK to KV_MAX_SHORT steps, and
// only what is longer is cut for two items per workgroup (an item costs about 10 steps' time to start and finish, and its
// partial slot is written and summed).  Two corrections to that:
//   - below KV_MID_CHUNK steps the chunks come out uneven, and if more of them than workgroups are longer than half a chunk, some
//     workgroups take two: KV_MID_CHUNK it is then;
//   - if no tile can have more than KV_UNCUT steps, none is cut: the second item and the sum cost more than they save.
// Forward + backward, us, at a least chunk of 32 / 16 / 8:  200 tokens of 64 / 8 heads, a random tree 103 / 88 / 79;  800 142 / 119 / 137
// (here 119);  800, 32 / 8 129 / 104 / 96;  2100, 8 / 8 131 / 108 / 98;  600, 8 / 8, at most 10 steps 75 / 75 / 84 (here 75).  Largest
// short chunk 16 / 32: 3650 tokens of 32 / 8 heads, a random tree 249 / 226;  5000, 16 / 4, a shared prefix with branches 267 / 233.
constexpr int KV_MIN_CHUNK = 8, KV_MID_CHUNK = 16, KV_MAX_SHORT = 32, KV_UNCUT = 12;
constexpr int KV_SORT_BELOW = 16;        // items per workgroup below which the items are handed out longest first
constexpr int KV_EPT = KV_BN / 64;       // summary entries per key tile, at most

constexpr int KV_MAX_QUEUES = 64;
struct KvPlanHeader {
  int n_work;        // work items = n_items * hkv
  // Work queues.  With hkv <= KV_MAX_QUEUES there is one queue per kv head (entry w of queue q = item
  // item_order[w] for kv head q) and a workgroup starts on the queue of its XCD: the workgroups of one XCD then
  // work on neighbouring key tiles of one kv head, which stream the same Q / dO tiles at about the same time, so
  // the XCD's L2 serves part of those reads (at a 131 K-token tree: 348 GB fetched per launch with one shared
  // queue, 229 GB with one per head, the pass 5 % faster).  A workgroup whose queue is empty moves on to the next
  // one.  Used when every workgroup gets many items (the plain hand-out order); with few items per workgroup (the
  // longest-first order) one shared queue balances better and is what the planner sets up.
  int n_queues, per_queue;
  int counter[KV_MAX_QUEUES];   // next entry of every queue
  int chunk;         // steps per chunk
  int n_split_items; // items [0, n_split_items) write partial slots (slot index = item index)
  int n_tiles;       // key tiles formed
  int n_split_tiles; // tiles cut into more than one chunk (listed in split_tile)
};

struct KvPlan {                // device pointers into the workspace
  KvPlanHeader* hdr;
  int *tile_e0, *tile_ne;                                 // [max_tiles] first summary entry, entries (64 keys each)
  int *tile_nq, *tile_qtlo, *tile_nchunks, *tile_item0;   // [max_tiles]
  int *item_tile, *item_chunk;                            // [max_items]
  int* item_order;                                        // [max_items] items in the order they are handed out (longest first)
  int* split_tile;                                        // [max_split_tiles]
  float* slots;                                           // [max_slots][hkv][2][KV_BN][D]
  int np64, no64;                                         // summary entries of the prefix / own region
  int max_tiles, max_items, max_slots, max_split_tiles;
};

inline int kv_target_items(int hkv) { return (KV_TARGET_WORK + hkv - 1) / hkv; }

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Carves the plan out of `base`; with base == nullptr only the size is computed.
// Bounds: every tile holds at least one summary entry, so there are at most np64 + no64 tiles; a
// tile that is cut has more than `chunk` steps and the steps of one kv head sum to at most
// chunk * kv_target_items, so at most kv_target_items tiles are cut, into at most
// 2 * kv_target_items chunks.
inline size_t kv_plan_layout(void* base, int n_q, int n_prefix, int hkv, KvPlan* out) {
  const int np64 = (n_prefix + 63) / 64, no64 = (n_q + 63) / 64;
  const int max_tiles = np64 + no64;
  const int max_items = max_tiles + kv_target_items(hkv);
  const int max_slots = 2 * kv_target_items(hkv);
  const int max_split_tiles = kv_target_items(hkv);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return base ? (char*)base + o : (char*)nullptr; };
  char* hdr = take(sizeof(KvPlanHeader));
  char* t[6];
  for (int i = 0; i < 6; i++) t[i] = take(sizeof(int) * max_tiles);
  char* i0 = take(sizeof(int) * max_items);
  char* i1 = take(sizeof(int) * max_items);
  char* i2 = take(sizeof(int) * max_items);
  char* st = take(sizeof(int) * max_split_tiles);
  char* sl = take(sizeof(float) * (size_t)max_slots * hkv * 2 * KV_BN * KV_D);
  if (out) {
    out->hdr = (KvPlanHeader*)hdr;
    out->tile_e0 = (int*)t[0]; out->tile_ne = (int*)t[1];
    out->tile_nq = (int*)t[2]; out->tile_qtlo = (int*)t[3]; out->tile_nchunks = (int*)t[4]; out->tile_item0 = (int*)t[5];
    out->item_tile = (int*)i0; out->item_chunk = (int*)i1; out->item_order = (int*)i2; out->split_tile = (int*)st; out->slots = (float*)sl;
    out->np64 = np64; out->no64 = no64;
    out->max_tiles = max_tiles; out->max_items = max_items; out->max_slots = max_slots; out->max_split_tiles = max_split_tiles;
  }
  return off;
}

// exclusive prefix sum / prefix maximum of one int per thread over the workgroup; the reduction over
// all threads is returned through *total.  Inside a wavefront by lane shifts, then over the wavefronts' totals.
template <bool MAX, int THREADS>
__device__ inline int block_exclusive_scan(int v, int* scratch /*[THREADS / 64]*/, int* total, int identity = 0) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  auto add = [](int x, int y) { return MAX ? max(x, y) : x + y; };
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int other = __shfl_up(v, off);
    if (lane >= off) v = add(v, other);
  }
  if (lane == 63) scratch[wv] = v;
  __syncthreads();
  int before = identity, all = identity;
#pragma unroll
  for (int i = 0; i < THREADS / 64; i++) {
    const int t = scratch[i];
    if (i < wv) before = add(before, t);
    all = add(all, t);
  }
  *total = all;
  __syncthreads();                        // scratch is free again (and what the callers wrote before the call is visible)
  const int up = __shfl_up(v, 1);
  return lane > 0 ? add(before, up) : before;
}

// What bounds this kernel is its chain of dependent steps on one workgroup, so the two tables that are read again and
// again (kt_max, the tiles' query steps) are kept in LDS for up to PLAN_LDS summary entries (262144 keys), and the scans
// go by lane shifts instead of by 20 barriers each.  (Forward + backward of 256 .. 4000 tokens: 5 us less.)
//
// The planner runs as one more workgroup of the dQ kernel, the first: dQ does not need the plan, dK/dV comes after both.  (As a launch of its
// own between the two it was 9 to 11 us of one busy workgroup.  Forward + backward: trees of 300 tokens of 32 / 8 heads 87.6 -> 79.0 us, 1024 of
// 64 / 8 145 -> 137, 3000 of 8 / 8 131 -> 119; 16406 tokens in five partitions 2924 -> 2864.)
constexpr int PLAN_LDS = 4096;
struct PlanSmem {
  int scratch[16], cls_base[64], wave_cnt[16][64];
  int kt[PLAN_LDS], nq[PLAN_LDS];
};

template <int THREADS>
__device__ __forceinline__ void kv_plan(PlanSmem& sm, const KvPlan& pl, const int32_t* __restrict__ kt_max, int n_q, int n_prefix, int G, int hkv,
                                        int n_workgroups) {
  int* const scratch = sm.scratch;
  int *const kt_lds = sm.kt, *const nq_lds = sm.nq;
  const int t = threadIdx.x;
  const int np64 = pl.np64, n_ent = pl.np64 + pl.no64;
  const bool in_lds = n_ent <= PLAN_LDS;      // (there are at most as many tiles as entries)
  if (in_lds) {
    for (int e = t; e < n_ent; e += THREADS) kt_lds[e] = kt_max[e];
    __syncthreads();
  }
  auto kt = [&](int e) { return in_lds ? kt_lds[e] : kt_max[e]; };
  auto tile_nq = [&](int i) { return in_lds ? nq_lds[i] : pl.tile_nq[i]; };
  // a run starts at the first entry of a region and wherever the largest bound changes
  auto run_break = [&](int e) { return e == 0 || e == np64 || kt(e) != kt(e - 1); };

  // ---- pass 1: tiles = runs cut every KV_EPT entries; each thread owns consecutive entries ----
  const int per = (n_ent + THREADS - 1) / THREADS;
  const int lo = min(t * per, n_ent), hi = min(lo + per, n_ent);
  int last_break = -1;
  for (int e = lo; e < hi; e++)
    if (run_break(e)) last_break = e;
  int unused;
  const int carry = block_exclusive_scan<true, THREADS>(last_break, scratch, &unused, -1);    // start of the run my first entry is in
  int my_tiles = 0;
  {
    int run_start = carry;
    for (int e = lo; e < hi; e++) {
      if (run_break(e)) run_start = e;
      if (((e - run_start) % KV_EPT) == 0) my_tiles++;
    }
  }
  int n_tiles;
  int tl = block_exclusive_scan<false, THREADS>(my_tiles, scratch, &n_tiles);
  int my_steps = 0;
  {
    int run_start = carry;
    for (int e = lo; e < hi; e++) {
      if (run_break(e)) run_start = e;
      if (((e - run_start) % KV_EPT) != 0) continue;
      // the tile runs to the next break, region end or KV_EPT entries
      const int e_end = e < np64 ? np64 : n_ent;
      int ne = 1;
      const int kmax = kt(e);
      while (ne < KV_EPT && e + ne < e_end && kt(e + ne) == kmax) ne++;
      const int i_lo = e < np64 ? 0 : (e - np64) * 64;                 // first query that can see a key of the tile
      const int i_hi = (int)min((int64_t)n_q, (int64_t)kmax - n_prefix);
      const int qt_lo = i_lo / KV_BM;
      const int nq = i_hi > i_lo ? (i_hi + KV_BM - 1) / KV_BM - qt_lo : 0;
      pl.tile_e0[tl] = e;
      pl.tile_ne[tl] = ne;
      pl.tile_nq[tl] = nq;
      if (in_lds) nq_lds[tl] = nq;
      pl.tile_qtlo[tl] = qt_lo;
      my_steps += nq * G;
      tl++;
    }
  }
  int total_steps;
  block_exclusive_scan<false, THREADS>(my_steps, scratch, &total_steps);       // (its barriers also publish the tile tables)
  const int64_t all = (int64_t)total_steps * hkv;
  const int target = max(1, min(KV_TARGET_WORK, KV_ITEMS_PER_WG * n_workgroups));
  const int64_t one_each = (all + n_workgroups - 1) / n_workgroups;
  const int64_t longest = (int64_t)G * ((n_q + KV_BM - 1) / KV_BM);       // no tile has more steps than this
  const int per_t = (n_tiles + THREADS - 1) / THREADS;          // each thread owns consecutive tiles
  const int tlo = min(t * per_t, n_tiles), thi = min(tlo + per_t, n_tiles);
  int chunk = (int)min((int64_t)KV_MAX_SHORT, max((int64_t)KV_MIN_CHUNK, one_each));
  if (longest <= KV_UNCUT) {
    chunk = KV_UNCUT;
  } else if (chunk < KV_MID_CHUNK) {
    int my_long = 0, n_long;
    for (int i = tlo; i < thi; i++) {
      const int steps = tile_nq(i) * G;
      my_long += steps / chunk + (steps % chunk > chunk / 2 ? 1 : 0);
    }
    block_exclusive_scan<false, THREADS>(my_long, scratch, &n_long);
    if ((int64_t)n_long * hkv > n_workgroups) chunk = KV_MID_CHUNK;
  }
  chunk = (int)max((int64_t)chunk, (all + target - 1) / target);

  // ---- pass 2: chunks per tile; cut tiles are numbered first (their item index is also their slot) ----
  int my_split = 0, my_whole = 0, my_split_tiles = 0;
  for (int i = tlo; i < thi; i++) {
    const int steps = tile_nq(i) * G;
    const int nc = (steps + chunk - 1) / chunk;
    pl.tile_nchunks[i] = nc;
    if (nc > 1) { my_split += nc; my_split_tiles++; } else my_whole += nc;
  }
  int n_split, n_whole, n_split_tiles;
  int split0 = block_exclusive_scan<false, THREADS>(my_split, scratch, &n_split);
  int whole0 = block_exclusive_scan<false, THREADS>(my_whole, scratch, &n_whole) + n_split;
  int st0 = block_exclusive_scan<false, THREADS>(my_split_tiles, scratch, &n_split_tiles);
  for (int i = tlo; i < thi; i++) {
    const int nc = pl.tile_nchunks[i];
    int& cursor = nc > 1 ? split0 : whole0;
    pl.tile_item0[i] = cursor;
    for (int c = 0; c < nc; c++) { pl.item_tile[cursor + c] = i; pl.item_chunk[cursor + c] = c; }
    cursor += nc;
    if (nc > 1) pl.split_tile[st0++] = i;
  }
  // ---- pass 3: hand-out order.  Workgroups pull items from a counter, so the launch ends when the item that
  //      was started last finishes: long items go first and short ones fill the end.  A stable counting sort
  //      of the items by their number of steps into 64 classes: inside a class the items keep their order
  //      (neighbouring key tiles stream the same query tiles at about the same time, which the L2 likes).
  //      Results do not depend on the order: every item has its own output rows or partial slot.
  //      With many items per workgroup the end effect is small and the plain order (key tiles in sequence order)
  //      measured 1-2 % faster, so the sort is applied only below KV_SORT_BELOW items per workgroup. ----
  constexpr int NCLS = 64, WAVES = THREADS / 64;      // NCLS = wavefront size (see the placement loop)
  static_assert(WAVES <= 16, "PlanSmem");
  int* const cls_base = sm.cls_base;
  int(*const wave_cnt)[NCLS] = sm.wave_cnt;
  const int n_items = n_split + n_whole;
  if ((int64_t)n_items * hkv >= (int64_t)KV_SORT_BELOW * n_workgroups) {
    for (int i = t; i < n_items; i += THREADS) pl.item_order[i] = i;
    if (t == 0) {
      pl.hdr->n_work = (n_split + n_whole) * hkv;
      pl.hdr->n_queues = hkv <= KV_MAX_QUEUES ? hkv : 1;
      pl.hdr->per_queue = hkv <= KV_MAX_QUEUES ? n_split + n_whole : (n_split + n_whole) * hkv;
      for (int q = 0; q < KV_MAX_QUEUES; q++) pl.hdr->counter[q] = 0;
      pl.hdr->chunk = chunk;
      pl.hdr->n_split_items = n_split;
      pl.hdr->n_tiles = n_tiles;
      pl.hdr->n_split_tiles = n_split_tiles;
    }
    return;
  }
  auto item_class = [&](int i) {
    const int tile = pl.item_tile[i];
    const int steps = min(chunk, tile_nq(tile) * G - pl.item_chunk[i] * chunk);
    return NCLS - 1 - min(NCLS - 1, (int)(((int64_t)steps * NCLS) / (chunk + 1)));       // class 0 = longest
  };
  const int lane = t & 63, wv = t >> 6;
  if (t < NCLS) cls_base[t] = 0;
  __syncthreads();                       // (also publishes the item tables written above)
  // class sizes -> first position of every class
  for (int i = t; i < n_items; i += THREADS) atomicAdd(&cls_base[item_class(i)], 1);      // integer counts: order-independent
  __syncthreads();
  if (t == 0) {
    int run = 0;
    for (int c = 0; c < NCLS; c++) { const int n = cls_base[c]; cls_base[c] = run; run += n; }
  }
  __syncthreads();
  // placement, THREADS items at a time in item order.  Inside a wavefront the rank of an item among the items of
  // its class comes from one ballot per class that actually occurs in the wavefront (a few: neighbouring
  // items are chunks of the same tile).
  for (int i0 = 0; i0 < n_items; i0 += THREADS) {
    const int i = i0 + t;
    const int c = i < n_items ? item_class(i) : -1;
    wave_cnt[wv][lane] = 0;                            // NCLS == wavefront size: one class count per lane
    int rank_in_wave = 0;
    uint64_t todo = __ballot(c >= 0);
    while (todo) {
      const int leader = __builtin_ctzll(todo);
      const int lc = __builtin_amdgcn_readlane(c, leader);
      const uint64_t m = __ballot(c == lc);
      if (c == lc) rank_in_wave = __popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) wave_cnt[wv][lc] = __popcll(m);
      todo &= ~m;
    }
    __syncthreads();
    if (c >= 0) {
      int before = 0;
      for (int ww = 0; ww < wv; ww++) before += wave_cnt[ww][c];
      pl.item_order[cls_base[c] + before + rank_in_wave] = i;
    }
    __syncthreads();
    if (t < NCLS) {
      int n = 0;
      for (int ww = 0; ww < WAVES; ww++) n += wave_cnt[ww][t];
      cls_base[t] += n;
    }
    __syncthreads();
  }
  if (t == 0) {
    pl.hdr->n_work = (n_split + n_whole) * hkv;
    pl.hdr->n_queues = 1;                      // few items per workgroup: one shared queue balances best (measured)
    pl.hdr->per_queue = (n_split + n_whole) * hkv;
    for (int q = 0; q < KV_MAX_QUEUES; q++) pl.hdr->counter[q] = 0;
    pl.hdr->chunk = chunk;
    pl.hdr->n_split_items = n_split;
    pl.hdr->n_tiles = n_tiles;
    pl.hdr->n_split_tiles = n_split_tiles;
  }
}

// workgroups of the dK/dV pass: one resident workgroup per compute unit pulls work items until the counter runs out
inline int kv_workgroups(const KvPlan& pl, int hkv) {
  int dev = 0, n_cu = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  return (int)std::min<int64_t>(n_cu, (int64_t)pl.max_items * hkv);
}

}  // namespace
}  // namespace tt
