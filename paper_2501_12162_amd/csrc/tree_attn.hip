// Paged tree attention for batched tree verification on gfx950.
//
// Every node i of request r attends to the request's cached prefix (paged
// KV) followed by the nodes of its own root-to-node path, so one pass scores
// every candidate continuation of every draft token tree (section 2, draft
// token tree; section 4.3 step 4, verification of all trees in parallel).
//
// bf16 kernel, one workgroup (4 waves) per work unit (see plan.h):
//  * rows of a unit are (node, q-head-in-group) pairs of one kv-head, so the
//    G query heads that share a kv-head read each K/V byte once (GQA);
//  * K/V blocks of 32 keys go straight from HBM to LDS with 16-byte
//    global_load_lds (no staging registers) into a 5-stage ring: four
//    stages are in flight while one is multiplied, one barrier per block,
//    waits counted by hand (vmcnt) so the ring really overlaps; steps that
//    fetch whole prefix blocks run branch-free, five to a loop iteration,
//    so their LDS addresses are constants; when every request is one row
//    tile (no K/V byte is read twice) the loads carry the non-temporal hint;
//  * LDS rows are XOR-swizzled in 16-byte chunks so that both the K
//    fragment reads (16 keys x 16 B per quarter-wave) and the transposed V
//    reads (ds_read_b64_tr_b16, 4 keys x 64 B per half-wave) hit distinct
//    banks;
//  * S^T = K Q^T and O^T = V^T P^T run on v_mfma_f32_32x32x16_bf16.  In this
//    orientation a lane holds half the keys of one query row, so the online
//    softmax needs no cross-lane traffic except one exchange of the two
//    halves' maxima.  16x16x32 instructions at the same rate needed twice as
//    many, two rows per lane and two exchanges for each (one request of 7
//    nodes over 1500 keys 18.4 -> 17.5 us, 24 requests at D = 64 28.3 ->
//    25.6, a rank of the 70B shape 135.8 -> 131.1, larger batches 0-2%);
//  * a row's denominator is summed from the bf16-rounded P (the numerator's
//    own weights) with v_dot2_f32_bf16: two P per instruction;
//  * the softmax folds the scale into one FMA per score (exp2 of
//    s*c - m*c) and only rescales a row's running state when its block max
//    rises more than 2^8 above the reference;
//  * the tree block (the request's own N_r nodes) is masked by 128-bit
//    ancestor sets built in LDS from parent[];
//  * prefixes longer than one chunk are split across workgroups; each writes
//    its partial (its own normalised output in bf16, reference max and
//    denominator in fp32) and a second, fully parallel kernel merges them
//    (the kernel boundary makes the partials of every XCD visible without
//    per-workgroup cache flushes).
#include <float.h>

#include <mutex>
#include <type_traits>

#include "accept_wave.h"
#include "adaserve.h"
#include "argmax_row.h"
#include "device_common.h"
#include "kernels.h"
#include "plan.h"

namespace adaserve {

namespace {

constexpr int kThreads = 256;
constexpr int kWavesF32 = 8;   // of an F32 workgroup

// 16 bytes of zeros: the source of every DMA lane whose key is out of range,
// so no NaN from an unused page slot reaches LDS.  Its device address is
// passed in the kernel arguments (resolved once per device on the host).
__device__ __align__(16) uint32_t g_zero16[4];

typedef __attribute__((address_space(3))) char lds_char;

// LDS byte address of a __shared__ object (what M0 takes).
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const lds_char *)p;
}

// 16-byte loads from global memory straight into LDS (global_load_lds):
// lane l writes LDS bytes [lds + 16 l, +16).  Written as asm so that the
// compiler does not try to track these loads itself (it cannot follow a
// ring of stages across the loop and would wait for every load in flight
// before each LDS read); the "memory" clobber keeps every LDS access in
// program order around them, and the waits below are counted by hand.
// Setting M0 needs one wait state before the load that reads it.  The
// compiler reserves M0 and warns about the clobber; nothing else in this
// library uses M0 (LDS instructions on gfx950 do not read it).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// With NT the loads carry the non-temporal hint: used when every K/V byte of
// the launch is read by one workgroup only (single-tile requests), so the
// lines are not kept for a reuse that never comes (measured 3-6% faster on
// a 1 GB long-context batch, 6% slower where row tiles share a chunk).
template <bool NT>
__device__ __forceinline__ void dma16(const void *src, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :: "v"(src), "s"(lds) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(src), "s"(lds) : "memory", "m0");
}
// Same with a wave-uniform base address and a 32-bit per-lane offset.
template <bool NT>
__device__ __forceinline__ void dma16_off(const void *base, uint32_t off, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop

// s_waitcnt vmcnt(N) with the other counters left open (for loads the
// compiler issued itself).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 16, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt(0xF70 | N);
}

// Waits until at most N of this wave's loads are in flight and its LDS
// operations are done, then the workgroup barrier.  No memory access moves
// across it.
template <int N>
__device__ __forceinline__ void wait_loads_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt immediate");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// Index of the first plan entry whose unit_end (or group_end) exceeds `key`,
// or -1: every lane reads one entry per 64, so the whole table costs one
// round of loads instead of a chain of dependent ones.  Uniform result.
__device__ __forceinline__ int find_plan_entry(const TreeAttnArgs &a, int64_t key, bool groups) {
  static_assert(kPlanMax <= 3 * 64, "three rounds of 64 lanes cover the plan table");
  const int lane = threadIdx.x & 63;
  int32_t end[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int i = k * 64 + lane;
    end[k] = i < a.plan_count ? (groups ? a.plan[i].group_end : a.plan[i].unit_end) : INT32_MAX;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const unsigned long long hit = __ballot((int64_t)end[k] > key);
    if (hit) return k * 64 + __ffsll(hit) - 1;
  }
  return -1;
}

// Finds the request that owns logical index `idx`, counting either work units
// or (kv-head, row tile) groups per request.  Every lane of the wave ends with
// the same answer.  Returns false when idx is past the end.
__device__ bool locate_request(int64_t idx, bool count_groups, const TreeAttnArgs &a,
                               int32_t &r_out, int64_t &unit_base, int64_t &group_base) {
  const int lane = threadIdx.x & 63;
  int64_t cum_u = 0, cum_g = 0;
  for (int r0 = 0; r0 < a.num_requests; r0 += 64) {
    const int r = r0 + lane;
    int64_t nu = 0, ng = 0;
    if (r < a.num_requests) {
      int32_t n = a.node_indptr[r + 1] - a.node_indptr[r];
      n = min(max(n, 0), kMaxTreeNodes);
      const int32_t L = max(a.prefix_len[r], 0);
      ng = (int64_t)a.num_kv_heads * row_tiles(n, a.group, a.rows_per_tile);
      nu = ng * prefix_chunks(L, chunk_keys(n, a.group, a.rows_per_tile, a.chunk_target, a.chunk_floor));
    }
    const int64_t iu = wave_inclusive_scan(nu);
    const int64_t ig = wave_inclusive_scan(ng);
    const int64_t key = count_groups ? ig : iu;
    const int64_t base = count_groups ? cum_g : cum_u;
    const int64_t total = __shfl(key, 63, 64);
    if (idx < base + total) {
      const unsigned long long hit = __ballot(base + key > idx);
      const int first = __ffsll(hit) - 1;
      r_out = r0 + first;
      unit_base = cum_u + __shfl(iu - nu, first, 64);
      group_base = cum_g + __shfl(ig - ng, first, 64);
      return true;
    }
    cum_u += __shfl(iu, 63, 64);
    cum_g += __shfl(ig, 63, 64);
  }
  return false;
}

// The work unit with logical id `uid`: its request, that request's sizes, the
// prefix keys per unit (F32: of no meaning, always the whole prefix) and the
// request's first unit id.  From the plan table in the kernel arguments, or,
// without one, by the scan.  Every field is uniform; false when there is no
// such unit or its request does not fit the batch.
struct Unit {
  int32_t r, node_base, n, L, chunk_len;
  int64_t ubase;
};
__device__ __forceinline__ bool find_unit(const TreeAttnArgs &a, int64_t uid, Unit &u) {
  int32_t r, node_base, n, L, chunk_len;
  int64_t ubase;
  if (a.plan_count > 0) {
    // the dispatch-ordered plan in the kernel arguments
    const int lo = __builtin_amdgcn_readfirstlane(find_plan_entry(a, uid, false));
    if (lo < 0) return false;
    r = plan_request(a.plan[lo].request_and_chunk);
    chunk_len = plan_chunk_keys(a.plan[lo].request_and_chunk);
    ubase = lo > 0 ? a.plan[lo - 1].unit_end : 0;
    node_base = a.plan[lo].node_base;
    n = plan_nodes(a.plan[lo].n_and_len);
    L = plan_prefix_len(a.plan[lo].n_and_len);
  } else {
    int64_t gbase;
    if (!locate_request(uid, false, a, r, ubase, gbase)) return false;
    node_base = a.node_indptr[r];
    n = min(max(a.node_indptr[r + 1] - node_base, 0), kMaxTreeNodes);
    L = max(a.prefix_len[r], 0);
    chunk_len = chunk_keys(n, a.group, a.rows_per_tile, a.chunk_target, a.chunk_floor);
  }
  // Request values are uniform; make that visible so branches on them stay scalar.
  u.r = __builtin_amdgcn_readfirstlane(r);
  u.node_base = __builtin_amdgcn_readfirstlane(node_base);
  u.n = __builtin_amdgcn_readfirstlane(n);
  u.L = __builtin_amdgcn_readfirstlane(L);
  u.chunk_len = __builtin_amdgcn_readfirstlane(chunk_len);
  u.ubase = ((int64_t)__builtin_amdgcn_readfirstlane((int32_t)(ubase >> 32)) << 32) |
            (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)ubase);
  return u.n > 0 && u.node_base >= 0 && u.node_base + u.n <= a.total_nodes;
}

__device__ __forceinline__ uint32_t set_bit_in(uint32_t w, int word, int v) {
  return ((v >> 5) == word) ? (w | (1u << (v & 31))) : w;
}

// Ancestor sets of a request's n nodes from its parents in LDS: bit j of
// node i's 128-bit set is 1 when j is on i's root-to-node path, i included.
// The walk stops at anything that is not a parent strictly before its child,
// so malformed trees stay in bounds.  Called by all of the workgroup's
// `threads` threads.
__device__ __forceinline__ void build_ancestors(const int32_t *par, uint32_t *anc, int n, int threads) {
  for (int i = threadIdx.x; i < kMaxTreeNodes; i += threads) {
    uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
    if (i < n) {
      int v = i;
      for (int step = 0; step < kMaxTreeNodes; ++step) {
        w0 = set_bit_in(w0, 0, v);
        w1 = set_bit_in(w1, 1, v);
        w2 = set_bit_in(w2, 2, v);
        w3 = set_bit_in(w3, 3, v);
        if (v == 0) break;
        const int p = par[v];
        if (p < 0 || p >= v) break;
        v = p;
      }
    }
    anc[i * 4 + 0] = w0;
    anc[i * 4 + 1] = w1;
    anc[i * 4 + 2] = w2;
    anc[i * 4 + 3] = w3;
  }
}

// 16-byte chunk permutation of LDS row `row`: chunk c of the row is stored in
// slot c ^ swizzle(row).  Any 16 consecutive rows keep one chunk in 16
// distinct places (K reads); rows 4k .. 4k+3 keep four neighbouring chunks in
// 16 distinct places (V reads).
template <int NCH>
__device__ __forceinline__ int swizzle(int row) {
  if (NCH == 16) return ((row & 3) << 2) | ((row >> 2) & 3);
  return ((row & 2) << 1) | ((row >> 2) & 3);
}

template <int D, bool NT>
__global__ __launch_bounds__(kThreads, 2) void tree_attn_bf16_kernel(TreeAttnArgs a) {
  constexpr int KS = D / 16;                 // MFMA k-steps over the head dim
  constexpr int DT = D / 32;                 // 32-wide output tiles over the head dim
  constexpr int KB = kKeysPerBlock;          // 32 keys per pipeline stage
  constexpr int ROWB = D * 2;                // bytes per key row
  constexpr int NCH = D / 8;                 // 16-byte chunks per key row
  constexpr int BLK = KB * ROWB;             // bytes of K (or V) per block
  constexpr int WI = BLK / 1024 / 4;         // DMA wave-instructions per wave per tensor block
  constexpr int RPI = 1024 / ROWB;           // key rows covered by one wave-instruction
  constexpr float kRescaleLog2 = 8.f;

  // Scores run one block ahead of the PV product: step j multiplies K of
  // block j+1 and V of block j, and fetches K block j+5 and V block j+4.
  // Stage t of the five-stage ring holds [K block t+1 | V block t] (mod 5),
  // so a step reads one stage and refills another, and four of the five
  // stages are in flight while one is multiplied.  The ring is all the LDS
  // this kernel has (80 KB at D = 128, two workgroups per CU): page ids are
  // read from the block table with scalar loads, and the parents and
  // ancestor sets live in the V half of stage 4 until the first step
  // refills it (each lane keeps its own rows' ancestor sets in registers).
  constexpr int NST = 5;
  __shared__ __align__(1024) char ring[NST * 2 * BLK];
  int32_t *const par = (int32_t *)(ring + (NST - 1) * 2 * BLK + BLK);
  uint32_t *const anc = (uint32_t *)(ring + (NST - 1) * 2 * BLK + BLK + kMaxTreeNodes * 4);
  static_assert(kMaxTreeNodes * 4 * 5 <= BLK, "parents and ancestor sets fit in a V half-stage");

  if ((int64_t)blockIdx.x >= a.padded_grid) {
    // fused verification step: argmax workgroups follow the attention units,
    // taking CUs that no attention unit occupies
    const int64_t row = (int64_t)blockIdx.x - a.padded_grid;
    if (row < a.argmax_rows)
      argmax_row<true, kThreads>(a.logits, a.logit_stride, a.vocab, (int32_t)row, a.argmax_out, (float *)ring,
                                 (int *)(ring + 64));
    return;
  }
  const int64_t uid = xcd_swizzle(blockIdx.x, a.padded_grid);
  if (uid >= a.units) return;
  Unit unit;
  if (!find_unit(a, uid, unit)) return;
  const int32_t r = unit.r, node_base = unit.node_base, n = unit.n, L = unit.L, chunk_len = unit.chunk_len;
  // a chunk is whole 32-key blocks and its page ids fit the page-id registers
  if (chunk_len <= 0 || chunk_len > kMaxChunk || chunk_len % kKeysPerBlock != 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.group;
  const int RT = a.rows_per_tile;
  const int32_t tiles = row_tiles(n, G, RT);
  const int32_t chunks = prefix_chunks(L, chunk_len);
  const int64_t u = uid - unit.ubase;
  const int32_t tile = (int32_t)(u % tiles);
  const int64_t rest = u / tiles;
  const int32_t g = (int32_t)(rest % a.num_kv_heads);
  const int32_t chunk = (int32_t)(rest / a.num_kv_heads);
  const int32_t M = n * G;
  const int32_t row0 = tile * RT;
  const int32_t row_end = min(M, row0 + RT);
  const bool last_chunk = chunk == chunks - 1;
  const int32_t k0 = chunk * chunk_len;
  const int32_t k1 = min(L, k0 + chunk_len);
  const int32_t n_prefix_blocks = k1 > k0 ? ceil_div(k1 - k0, KB) : 0;
  const int32_t n_full = k1 > k0 ? (k1 - k0) / KB : 0;   // prefix blocks that need no mask
  const int32_t n_tree_blocks = last_chunk ? ceil_div(n, KB) : 0;
  const int32_t nb = n_prefix_blocks + n_tree_blocks;
  const int32_t page0 = k0 / kPageSize;
  const int32_t npages = k1 > k0 ? ceil_div(k1, kPageSize) - page0 : 0;

  // ---- start-up: page ids, parents and queries, all loads in flight together.
  // The DMA rows of a wave lie in one 16-key page of each 32-key block (page
  // wave_page of the two); lane l of pgv[i] holds that page's id in prefix
  // block i*64 + l, or -1.
  const int wave_page = (wave * WI * RPI) / kPageSize;
  static_assert(kMaxChunk / KB <= 4 * 64, "page ids of a chunk fit in four lanes-wide registers");
  int32_t pgv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t blk = i * 64 + lane;
    const int32_t e = page0 + blk * (KB / kPageSize) + wave_page;
    int32_t p = -1;
    if (blk < n_prefix_blocks && e < a.bt_stride) {
      p = a.block_table[(int64_t)r * a.bt_stride + e];
      if (p < 0 || p >= a.num_pages) p = -1;
    }
    pgv[i] = p;
  }
  (void)npages;
  if (last_chunk)
    for (int i = tid; i < n; i += kThreads) par[i] = a.parent[node_base + i];

  // Query fragments (B operand of S^T = K Q^T): lane holds row (lane & 31) of
  // the wave's 32, head-dim elements ks*16 + (lane >> 5)*8 .. +7.
  const int wrow0 = row0 + wave * 32;
  const bool wave_live = wrow0 < row_end;
  const int row = wrow0 + (lane & 31);
  const bool row_valid = row < row_end;
  const int row_node = row_valid ? row / G : 0;
  const int row_head = g * G + (row_valid ? row - row_node * G : 0);
  bf16x8 qf[KS];
  {
    const __bf16 *qp =
        (const __bf16 *)a.q + ((int64_t)(node_base + row_node) * a.num_q_heads + row_head) * D + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 v = {};
      if (row_valid) v = *(const bf16x8 *)(qp + ks * 16);
      qf[ks] = v;
    }
  }
  // Let the start-up loads land before the first DMA, so the waits counted
  // by hand below only ever cover K/V blocks.
  wait_vmcnt<0>();

  // ---- DMA addressing: wave-instruction i of this wave fills LDS bytes
  // [(wave*WI + i)*1024, +1024) of a stage; lane `lane` lands on key row
  // dma_row[i], slot `slot`, so it fetches chunk slot ^ swizzle(row).  A
  // wave's rows lie in one 16-key page (wave_page of the two in a block), so
  // the page and its base address are wave-uniform; lanes add a 32-bit byte
  // offset inside the (page, kv-head) chunk or inside the tree block.
  const int slot = ((lane * 16) % ROWB) / 16;
  int dma_row[WI];
  uint32_t page_off[WI];   // bytes inside the (page, kv-head) chunk
  uint32_t tree_off[WI];   // bytes from the first key row of the tree block
  const int64_t tree_stride = (int64_t)a.num_kv_heads * D;   // elements between node rows
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    dma_row[i] = (wave * WI + i) * RPI + (lane * 16) / ROWB;
    const int chunk_el = (slot ^ swizzle<NCH>(dma_row[i])) * 8;
    page_off[i] = (uint32_t)(((dma_row[i] % kPageSize) * D + chunk_el) * 2);
    tree_off[i] = (uint32_t)((dma_row[i] * tree_stride + chunk_el) * 2);
  }
  const int64_t page_stride_b = (int64_t)a.num_kv_heads * kPageSize * D * 2;   // bytes per page
  const int64_t head_off_b = (int64_t)g * kPageSize * D * 2;
  const int64_t tree_off_b = ((int64_t)node_base * a.num_kv_heads + g) * D * 2;
  // Fetches block blk of K (pool = k_pages, tree = k_tree) or of V into
  // `dst`.  Rows past the end of the block's keys, pages outside the pool and
  // blocks past the last one come from the zero line: every step issues the
  // same number of loads, so the waits below are constants.
  // `page` is this wave's physical page of block blk, or -1 (tree block,
  // entry past the block table row, or a page id outside the pool), read from
  // the page-id registers with lane reads (blk is uniform).
  auto page_of = [&](int blk) -> int32_t {
    if (blk >= n_prefix_blocks) return -1;
    const int l = blk & 63, hi = blk >> 6;
    const int32_t p0 = __builtin_amdgcn_readlane(pgv[0], l), p1 = __builtin_amdgcn_readlane(pgv[1], l);
    const int32_t p2 = __builtin_amdgcn_readlane(pgv[2], l), p3 = __builtin_amdgcn_readlane(pgv[3], l);
    return hi == 0 ? p0 : hi == 1 ? p1 : hi == 2 ? p2 : p3;
  };
  auto issue = [&](const void *pool, const void *tree, char *dst, int blk, int32_t page) {
    const char *base;
    int rows_left;
    const bool pre = blk < n_prefix_blocks;
    if (blk >= nb) {
      rows_left = 0;
      base = (const char *)tree;
    } else if (pre) {
      const int32_t p = __builtin_amdgcn_readfirstlane(page);
      rows_left = p >= 0 ? k1 - k0 - blk * KB : 0;
      base = (const char *)pool + head_off_b + (int64_t)max(p, 0) * page_stride_b;
    } else {
      const int tb = blk - n_prefix_blocks;
      rows_left = n - tb * KB;
      base = (const char *)tree + tree_off_b + (int64_t)tb * KB * tree_stride * 2;
    }
    const uint32_t lds = lds_addr(dst) + wave * WI * 1024;
    if (rows_left >= KB) {
#pragma unroll
      for (int i = 0; i < WI; ++i) dma16_off<NT>(base, pre ? page_off[i] : tree_off[i], lds + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < WI; ++i) {
        const bool ok = dma_row[i] < rows_left;
        dma16<NT>(ok ? (const void *)(base + (pre ? page_off[i] : tree_off[i])) : a.zero16, lds + i * 1024);
      }
    }
  };
  auto issue_k = [&](char *stage, int blk, int32_t page) { issue(a.k_pages, a.k_tree, stage, blk, page); };
  auto issue_v = [&](char *stage, int blk, int32_t page) {
    issue(a.v_pages, a.v_tree, stage + BLK, blk, page);
  };

  __syncthreads();  // par[] visible
  // Prologue issue order: K0 (stage 4), then (K1, V0), (K2, V1), (K3, V2),
  // (K4, V3) into stages 0 .. 3.
  int32_t pg4 = -1, pg5 = -1;   // pages of blocks j+4 and j+5 at step j
  if (nb > 0) {
    const int32_t pg0 = page_of(0), pg1 = page_of(1), pg2 = page_of(2), pg3 = page_of(3);
    pg4 = page_of(4);
    pg5 = page_of(5);
    issue_k(ring + 4 * 2 * BLK, 0, pg0);
    issue_k(ring + 0 * 2 * BLK, 1, pg1);
    issue_v(ring + 0 * 2 * BLK, 0, pg0);
    issue_k(ring + 1 * 2 * BLK, 2, pg2);
    issue_v(ring + 1 * 2 * BLK, 1, pg1);
    issue_k(ring + 2 * 2 * BLK, 3, pg3);
    issue_v(ring + 2 * 2 * BLK, 2, pg2);
    issue_k(ring + 3 * 2 * BLK, 4, pg4);
    issue_v(ring + 3 * 2 * BLK, 3, pg3);
  }

  // Ancestor sets, while the first blocks are in flight.
  if (last_chunk) build_ancestors(par, anc, n, kThreads);

  // Per-lane LDS offsets of the MFMA operand fragments inside a stage.
  const int half = lane >> 5;

  // The ancestor set of this lane's row's node, in registers.
  uint32_t an0 = 0, an1 = 0, an2 = 0, an3 = 0;
  if (last_chunk) {
    __syncthreads();  // anc[] complete
    an0 = anc[row_node * 4 + 0], an1 = anc[row_node * 4 + 1], an2 = anc[row_node * 4 + 2], an3 = anc[row_node * 4 + 3];
  }
  int koff[KS];  // K fragment: key row lane & 31, chunk ks*2 + half
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    koff[ks] = (lane & 31) * ROWB + (((ks * 2 + half) ^ swizzle<NCH>(lane & 31)) * 16);
  // Transposed V reads: a 16-lane group takes 4 key rows x 16 columns; lane
  // (half, c) of a fragment holds column dt*32 + c of key rows half*4 + 0..3
  // (+ 8 for its upper four elements, + 16 for the second k-step).
  int voff[DT], voff8[DT];
  {
    const int j16 = lane & 15;
    const int vrow = half * 4 + (j16 >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int ch = dt * 4 + ((lane >> 4) & 1) * 2 + ((j16 & 3) >> 1);
      voff[dt] = vrow * ROWB + ((ch ^ swizzle<NCH>(vrow)) * 16) + (j16 & 1) * 8;
      voff8[dt] = (vrow + 8) * ROWB + ((ch ^ swizzle<NCH>(vrow + 8)) * 16) + (j16 & 1) * 8;
    }
  }

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x16{};
  float lsum = 0.f;                                  // sum of this lane's (rounded) P
  const float c = a.scale_log2;                      // raw score -> log2 units
  const float up_raw = kRescaleLog2 / c;             // rescale threshold in raw units
  float m_ref = -1e30f;                              // reference max of this lane's row (raw units)

  // S^T tile of one block: s[i] holds key (i >> 2)*8 + half*4 + (i & 3) of
  // the lane's row.
  auto scores = [&](const char *kst, f32x16 &s) {
    s = f32x16{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 kf = *(const bf16x8 *)(kst + koff[ks]);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s, 0, 0, 0);
    }
  };
  // Masks the partial prefix block and the tree blocks (ancestor sets).
  auto mask = [&](f32x16 &s, int blk) {
    const bool tree_blk = blk >= n_prefix_blocks;
    const int tb = blk - n_prefix_blocks;
    const int valid = tree_blk ? min(KB, n - tb * KB) : min(KB, k1 - k0 - blk * KB);
    uint32_t aw = 0xffffffffu;
    if (tree_blk) {
      const uint32_t w0 = an0, w1 = an1, w2 = an2, w3 = an3;
      aw = (tb & 2) ? ((tb & 1) ? w3 : w2) : ((tb & 1) ? w1 : w0);
    }
    if (valid < KB) aw &= (1u << valid) - 1u;
    aw >>= half * 4;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = ((aw >> ((i >> 2) * 8 + (i & 3))) & 1u) ? s[i] : -INFINITY;
  };
  // The row's block max.
  auto rowmax = [&](const f32x16 &s) {
    float m0 = s[0], m1 = s[1];
#pragma unroll
    for (int i = 2; i < 14; i += 4) {
      m0 = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m0, s[i]), s[i + 2]);
      m1 = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m1, s[i + 1]), s[i + 3]);
    }
    m0 = __builtin_elementwise_maximum(m0, s[14]);
    return max_over_halves(__builtin_elementwise_maximum(__builtin_elementwise_maximum(m0, m1), s[15]));
  };
  // Raises the reference max of the rows whose block max went more than
  // 2^8 above it, rescaling their running numerator and denominator.
  auto rescale = [&](float bm) {
    const bool up = bm > m_ref + up_raw;
    if (__any(up)) {
      const float mn = up ? bm : m_ref;
      const float al = up ? __builtin_amdgcn_exp2f((m_ref - mn) * c) : 1.f;
      m_ref = mn;
      lsum *= al;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= al;
    }
  };
  // P = 2^(s c - m c) in bf16, packed as the B operand of the PV product:
  // slot e of k-step h is score register h*8 + e.
  auto probs = [&](const f32x16 &s, bf16x8 (&pk)[2]) {
    const float mc = m_ref * c;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h * 8 + 2 * e], c, -mc));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h * 8 + 2 * e + 1], c, -mc));
        const bf16x2 pp = __builtin_convertvector((f32x2{p0, p1}), bf16x2);
        lsum = __builtin_amdgcn_fdot2_f32_bf16(pp, ones, lsum, false);
        w[e] = __builtin_bit_cast(uint32_t, pp);
      }
      pk[h] = __builtin_bit_cast(bf16x8, w);
    }
  };
  // O^T += V^T P^T.
  auto pv = [&](const char *vst, const bf16x8 (&pk)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(vst + voff[dt] + h * 16 * ROWB));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(vst + voff8[dt] + h * 16 * ROWB));
        const bf16x8 vf = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pk[h], o[dt], 0, 0, 0);
      }
  };

  f32x16 s;        // scores of the block whose PV product comes next
  float bm = 0.f;  // its row maximum
  // Prologue: wait for K0 (the eight later prologue loads may still fly),
  // then the scores of block 0.
  if (nb > 0) {
    wait_loads_barrier<8 * WI>();
    if (wave_live) {
      scores(ring + 4 * 2 * BLK, s);
      if (n_full == 0) mask(s, 0);
      bm = rowmax(s);
    }
  }

  // Step j (its stage is cs = j mod 5): wait until K block j+1 and V block j
  // have landed (the loads of the three following steps may still fly),
  // barrier (every wave is done with K block j and V block j-1, whose stage
  // is refilled now), fetch K block j+5 and V block j+4, then P of block j,
  // scores of block j+1 and the PV product of block j; the scores of block
  // j+1 are masked (when they need it) and reduced last, while the PV
  // products run on the matrix cores.
  // `issue` for a block known to be a whole prefix block: no block-kind or
  // row-count branches, and a page outside the pool sends every lane to the
  // zero line (base = zero line, offset 0) without a branch.  Steps whose two
  // fetches are such blocks (most of a long chunk) take this form; it cuts
  // the scalar work of a step by about a third.
  auto issue_full = [&](const void *pool, char *dst, int32_t page) {
    const int32_t p = __builtin_amdgcn_readfirstlane(page);
    const uint32_t lds = lds_addr(dst) + wave * WI * 1024;
    const bool ok = p >= 0;
    const char *base = ok ? (const char *)pool + head_off_b + (int64_t)p * page_stride_b : (const char *)a.zero16;
#pragma unroll
    for (int i = 0; i < WI; ++i) dma16_off<NT>(base, ok ? page_off[i] : 0u, lds + i * 1024);
  };
  auto step = [&](int j, int cs, auto masked, auto has_next, auto full_fetch) {
    constexpr bool kMasked = decltype(masked)::value;
    constexpr bool kNext = decltype(has_next)::value;
    constexpr bool kFull = decltype(full_fetch)::value;
    const char *cur = ring + cs * (2 * BLK);
    if constexpr (kNext) {
      wait_loads_barrier<6 * WI>();
      char *fill = ring + (cs == 0 ? NST - 1 : cs - 1) * (2 * BLK);
      if constexpr (kFull) {
        issue_full(a.k_pages, fill, pg5);
        issue_full(a.v_pages, fill + BLK, pg4);
      } else {
        issue_k(fill, j + 5, pg5);
        issue_v(fill, j + 4, pg4);
      }
      pg4 = pg5;
      pg5 = page_of(j + 6);
    } else {
      wait_loads_barrier<0>();  // also drains the zero-line loads past the last block
    }
    if (wave_live) {
      rescale(bm);
      bf16x8 pk[2];
      probs(s, pk);
      if constexpr (kNext) {
        f32x16 sn;
        scores(cur, sn);
        pv(cur + BLK, pk);
        if constexpr (kMasked) mask(sn, j + 1);
        bm = rowmax(sn);
        s = sn;
      } else {
        pv(cur + BLK, pk);
      }
    }
  };
  using Yes = std::true_type;
  using No = std::false_type;
  int j = 0, cs = 0;
  auto next_stage = [](int c) { return c == NST - 1 ? 0 : c + 1; };
  // Blocks j+4 and j+5 whole prefix blocks: five steps per iteration (one
  // per ring stage, starting at stage 0), so every LDS address of a step is
  // a constant and folds into the instruction's offset.
  for (; j + 9 < n_full; j += 5) {
    step(j, 0, No{}, Yes{}, Yes{});
    step(j + 1, 1, No{}, Yes{}, Yes{});
    step(j + 2, 2, No{}, Yes{}, Yes{});
    step(j + 3, 3, No{}, Yes{}, Yes{});
    step(j + 4, 4, No{}, Yes{}, Yes{});
  }
  for (; j + 5 < n_full; ++j, cs = next_stage(cs)) step(j, cs, No{}, Yes{}, Yes{});
  for (; j + 1 < n_full; ++j, cs = next_stage(cs)) step(j, cs, No{}, Yes{}, No{});  // block j+1: full prefix block
  for (; j + 1 < nb; ++j, cs = next_stage(cs)) step(j, cs, Yes{}, Yes{}, No{});     // block j+1 needs the mask
  if (nb > 0) step(nb - 1, cs, No{}, No{}, No{});

  if (!wave_live) return;
  const float l_tot = sum_over_halves(lsum);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  // The row's normalised output in bf16: into `out`, or, when the prefix is
  // split, as this chunk's partial (a weighted mean of V rows, so bf16 keeps
  // 2^-9 relative precision) with its reference max and denominator in fp32;
  // tree_attn_combine_kernel merges the chunks after this kernel.
  const int64_t pslot = uid * kMaxRowsPerTile + (row - row0);
  __bf16 *dst = chunks == 1 ? (__bf16 *)a.out + ((int64_t)(node_base + row_node) * a.num_q_heads + row_head) * D
                            : a.ws_o + pslot * D;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; i += 8) {
      // registers i .. i+3 / i+4 .. i+7 are columns i*2 + half*4 .. +3 and 8
      // further; the halves swap so that each lane stores 16 contiguous bytes
      const uint32_t x0 = pack_bf16x2(o[dt][i] * inv, o[dt][i + 1] * inv);
      const uint32_t x1 = pack_bf16x2(o[dt][i + 2] * inv, o[dt][i + 3] * inv);
      const uint32_t y0 = pack_bf16x2(o[dt][i + 4] * inv, o[dt][i + 5] * inv);
      const uint32_t y1 = pack_bf16x2(o[dt][i + 6] * inv, o[dt][i + 7] * inv);
      const auto r0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
      const auto r1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
      if (row_valid) *(u32x4 *)(dst + dt * 32 + i * 2 + half * 8) = u32x4{r0[0], r1[0], r0[1], r1[1]};
    }
  if (chunks > 1 && row_valid && half == 0) *(f32x2 *)(a.ws_ml + pslot * 2) = f32x2{m_ref, l_tot};
}

// Merges the chunk partials of every split (request, kv-head, row tile):
// with w_c = l_c 2^((m_c - m) c), out = sum_c w_c o_c / sum_c w_c, o_c being
// chunk c's own normalised output.  One workgroup per 16 rows of one
// kv-head; each thread owns D/16 columns of one row.  With a plan table the
// grid holds the split requests' rows only (group_end counts 16-row merge
// blocks); without one, workgroup b takes rows (b % 8) * 16 .. +15 of
// (kv-head, row tile) group b / 8 in the scan order, and the workgroups of
// unsplit requests or past a tile's rows return at once.
template <int D>
__global__ __launch_bounds__(kThreads) void tree_attn_combine_kernel(TreeAttnArgs a) {
  constexpr int kRowsPerWg = 16;
  constexpr int TPR = kThreads / kRowsPerWg;  // threads per row
  constexpr int CPT = D / TPR;                // columns per thread (8 or 4)
  if ((int64_t)blockIdx.x >= a.merge_blocks) {
    // fused verification step: one acceptance wave per request after the
    // merge workgroups (the argmax finished in the previous launch)
    __shared__ int32_t acc_lds[kThreads / 64][3][kMaxTreeNodes];
    const int w = threadIdx.x >> 6;
    const int64_t r = ((int64_t)blockIdx.x - a.merge_blocks) * (kThreads / 64) + w;
    if (r < a.accept_requests)
      accept_request((int)r, a.total_nodes, a.node_indptr, a.parent, a.draft_tokens, a.argmax_out, a.max_accept,
                     a.accept_len, a.accept_tokens, a.accept_nodes, acc_lds[w][0], acc_lds[w][1], acc_lds[w][2]);
    return;
  }
  int32_t node_base, n, L, chunk_len, tile, g, rl;
  int64_t ubase;
  const int G = a.group, RT = a.rows_per_tile;
  if (a.plan_count > 0) {
    const int lo = __builtin_amdgcn_readfirstlane(find_plan_entry(a, blockIdx.x, true));
    if (lo < 0) return;
    const int64_t mbase = lo > 0 ? a.plan[lo - 1].group_end : 0;
    ubase = lo > 0 ? a.plan[lo - 1].unit_end : 0;
    node_base = a.plan[lo].node_base;
    n = plan_nodes(a.plan[lo].n_and_len);
    L = plan_prefix_len(a.plan[lo].n_and_len);
    chunk_len = plan_chunk_keys(a.plan[lo].request_and_chunk);
    const int32_t per_head = ceil_div(n * G, kRowsPerWg);
    if (per_head <= 0) return;
    const int32_t local = (int32_t)(blockIdx.x - mbase);
    g = local / per_head;
    const int32_t row = (local - g * per_head) * kRowsPerWg + (int)threadIdx.x / TPR;
    if (g >= a.num_kv_heads || row >= n * G) return;
    tile = row / RT;
    rl = row - tile * RT;
  } else {
    const int64_t gid = blockIdx.x / (kMaxRowsPerTile / kRowsPerWg);
    const int rblk = blockIdx.x % (kMaxRowsPerTile / kRowsPerWg);
    if (gid >= a.row_groups) return;
    int32_t r;
    int64_t gbase;
    if (!locate_request(gid, true, a, r, ubase, gbase)) return;
    node_base = a.node_indptr[r];
    n = min(max(a.node_indptr[r + 1] - node_base, 0), kMaxTreeNodes);
    L = max(a.prefix_len[r], 0);
    chunk_len = chunk_keys(n, G, RT, a.chunk_target, a.chunk_floor);
    if (n == 0) return;
    const int32_t tiles_r = row_tiles(n, G, RT);
    const int64_t u = gid - gbase;
    tile = (int32_t)(u % tiles_r);
    g = (int32_t)(u / tiles_r);
    rl = rblk * kRowsPerWg + (int)threadIdx.x / TPR;
    if (rl >= min(RT, n * G - tile * RT)) return;
  }
  if (n == 0 || node_base < 0 || node_base + n > a.total_nodes) return;
  if (chunk_len <= 0 || chunk_len > kMaxChunk || chunk_len % kKeysPerBlock != 0) return;
  const int32_t tiles = row_tiles(n, G, RT);
  const int32_t chunks = prefix_chunks(L, chunk_len);
  if (chunks == 1) return;
  const int col = ((int)threadIdx.x % TPR) * CPT;
  const float c = a.scale_log2;
  float mm = -1e30f, ll = 0.f;
  f32x4 acc[CPT / 4];
#pragma unroll
  for (int k = 0; k < CPT / 4; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int cc = 0; cc < chunks; ++cc) {
    const int64_t slot = (ubase + ((int64_t)cc * a.num_kv_heads + g) * tiles + tile) * kMaxRowsPerTile + rl;
    const f32x2 ml = *(const f32x2 *)(a.ws_ml + slot * 2);
    u32x4 raw = {0u, 0u, 0u, 0u};  // CPT bf16 values
    if (CPT == 8) raw = *(const u32x4 *)(a.ws_o + slot * D + col);
    else { const u32x2 h = *(const u32x2 *)(a.ws_o + slot * D + col); raw[0] = h[0]; raw[1] = h[1]; }
    const float m_new = fmaxf(mm, ml[0]);
    const float sa = __builtin_amdgcn_exp2f((mm - m_new) * c);
    const float wb = ml[1] * __builtin_amdgcn_exp2f((ml[0] - m_new) * c);
    mm = m_new;
    ll = ll * sa + wb;
#pragma unroll
    for (int k = 0; k < CPT / 4; ++k) {
      const f32x4 v = {bf16_bits_to_float(raw[2 * k] & 0xffffu), bf16_bits_to_float(raw[2 * k] >> 16),
                       bf16_bits_to_float(raw[2 * k + 1] & 0xffffu), bf16_bits_to_float(raw[2 * k + 1] >> 16)};
      acc[k] = acc[k] * sa + v * wb;
    }
  }
  const float inv = ll > 0.f ? 1.f / ll : 0.f;
  const int row = tile * RT + rl;
  const int node = row / G, hh = row - (row / G) * G;
  __bf16 *op = (__bf16 *)a.out + ((int64_t)(node_base + node) * a.num_q_heads + g * G + hh) * D + col;
#pragma unroll
  for (int k = 0; k < CPT / 4; ++k) {
    u32x2 w;
    w[0] = pack_bf16x2(acc[k][0] * inv, acc[k][1] * inv);
    w[1] = pack_bf16x2(acc[k][2] * inv, acc[k][3] * inv);
    *(u32x2 *)(op + 4 * k) = w;
  }
}

// fp32 path: one workgroup of 8 waves per (request, kv-head, tile of 16 RB
// rows), rows as in the bf16 kernel.  The unit's keys -- the prefix's 16-key
// pages, then the tree in 16-node blocks -- are cut into 8 contiguous runs,
// one per wave, and the waves' online softmaxes are joined through LDS at the
// end.  S^T = K Q^T and O^T = V^T P^T run on v_mfma_f32_16x16x4_f32 (fp32
// inputs, products and sums).  Both contractions may take their slots in any
// order, so they are ordered such that every lane loads 16 contiguous bytes
// of K and of V straight into the operand registers and P needs no exchange:
// contraction slot q of QK step (c, e) is head-dim element 16 c + 4 q + e,
// slot q of PV step e is key 4 q + e, and O^T tile (h, k) holds the head-dim
// columns 64 h + 4 j + k, j = 0 .. 15.
// What bounds it: the matrix cores of the CUs that hold the longest requests
// (a unit's keys stay on one CU: F32 calls have no workspace for partial
// results).  So small batches take 16-row tiles (RB = 1), which put more CUs
// to work, and batches that fill the chip with 32-row tiles (RB = 2) take
// those, which read each K/V byte half as often.  4 requests of 15-55 nodes
// over 147-1254 keys (16 / 4 heads, D = 128): 41 us, of which the longest
// units' matrix instructions are 19 and launch, start and merge 13; a
// workgroup per (node, q-head) with the products on the vector ALUs read the
// whole prefix once for each and took 266.  One request of 16 nodes over 256
// keys (8 / 8 heads, D = 64): 14.8 -> 10 us.  A second set of K and V registers
// (loads two blocks ahead) and 12 or 16 waves with one set measured no faster.
template <int D, int RB>
__global__ __launch_bounds__(kWavesF32 * 64) void tree_attn_f32_kernel(TreeAttnArgs a) {
  constexpr int NW = kWavesF32, kT = NW * 64;
  constexpr int RT = 16 * RB;
  constexpr int NC = D / 16;      // 16-byte K loads per lane and block
  constexpr int NH = D / 64;      // 16-byte V loads per lane and key
  constexpr int LDO = D + 4;      // row stride of the waves' outputs in LDS (spreads a column over the banks)
  __shared__ __align__(16) float mo[NW * RT * LDO];
  __shared__ float mw[NW][RT], lw[NW][RT];
  static_assert(kMaxTreeNodes <= RT * LDO, "a wave's parents fit in its part of mo");

  if ((int64_t)blockIdx.x >= a.padded_grid) {
    // fused verification step: argmax workgroups follow the attention units
    const int64_t row = (int64_t)blockIdx.x - a.padded_grid;
    if (row < a.argmax_rows)
      argmax_row<false, kT>(a.logits, a.logit_stride, a.vocab, (int32_t)row, a.argmax_out, mo, (int *)(mo + 64));
    return;
  }
  const int64_t uid = xcd_swizzle(blockIdx.x, a.padded_grid);
  if (uid >= a.units) return;
  Unit unit;
  if (!find_unit(a, uid, unit)) return;
  const int32_t r = unit.r, node_base = unit.node_base, n = unit.n, L = unit.L;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, j = lane & 15;
  const int G = a.group;
  const int32_t tiles = row_tiles(n, G, RT);
  const int64_t u = uid - unit.ubase;
  const int32_t row0 = (int32_t)(u % tiles) * RT;
  const int32_t g = (int32_t)(u / tiles);
  const int32_t M = n * G;
  if (g >= a.num_kv_heads) return;

  // this wave's blocks of 16 keys
  const int32_t n_prefix_blocks = ceil_div(L, kPageSize);
  const int32_t nb = n_prefix_blocks + ceil_div(n, 16);
  const int32_t b0 = (int32_t)((int64_t)nb * wave / NW), b1 = (int32_t)((int64_t)nb * (wave + 1) / NW);

  // The waves that have tree blocks fetch the parents (each into its part of
  // mo, which holds nothing else before the merge).
  const bool has_tree = b1 > n_prefix_blocks && b1 > b0;
  int32_t *const par = (int32_t *)(mo + wave * RT * LDO);
  if (has_tree)
    for (int i = lane; i < n; i += 64) par[i] = a.parent[node_base + i];

  // query fragments: lane holds row j of each 16-row block
  f32x4 qf[RB][NC];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = row0 + rb * 16 + j;
    const int node = row < M ? row / G : 0, hh = row < M ? row - node * G : 0;
    const float *qp = (const float *)a.q + ((int64_t)(node_base + node) * a.num_q_heads + g * G + hh) * D + q * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) qf[rb][c] = *(const f32x4 *)(qp + c * 16);
  }

  // Block b's page (-1: the tree, an entry past the block-table row, or a page
  // id outside the pool) and the addresses of its rows.  Lane i holds the page
  // of block page_base + i; blocks are asked for in ascending order.  (A load
  // per block would be waited for, and every K and V load in flight with it.)
  int32_t page_base = b0, pages = -1;
  auto load_pages = [&]() {
    const int b = page_base + lane;
    pages = -1;
    if (b < n_prefix_blocks && b < a.bt_stride) {
      const int32_t p = a.block_table[(int64_t)r * a.bt_stride + b];
      if (p >= 0 && p < a.num_pages) pages = p;
    }
  };
  load_pages();
  auto page_of = [&](int b) -> int32_t {
    if (b >= page_base + 64) {
      page_base = b;
      load_pages();
    }
    return __builtin_amdgcn_readlane(pages, b - page_base);
  };
  const int64_t tree_stride = (int64_t)a.num_kv_heads * D;
  auto rows_at = [&](const void *pool, const void *tree, int b, int32_t page, int64_t &stride, int &rows) {
    if (b < n_prefix_blocks && page >= 0) {
      stride = D;
      rows = min(kPageSize, L - b * kPageSize);
      return (const float *)pool + ((int64_t)page * a.num_kv_heads + g) * kPageSize * D;
    }
    // a page outside the pool reads tree rows, whose values are not used
    const int tb = b < n_prefix_blocks ? 0 : b - n_prefix_blocks;
    stride = tree_stride;
    rows = min(16, n - tb * 16);
    return (const float *)tree + ((int64_t)(node_base + tb * 16) * a.num_kv_heads + g) * D;
  };
  // Rows past the block's keys repeat its last one (their scores are masked,
  // their V is zeroed), so every block loads without branches.
  f32x4 kr[NC], vr[4][NH];
  auto load_k = [&](int b, int32_t page) {
    int64_t stride;
    int rows;
    const float *base = rows_at(a.k_pages, a.k_tree, b, page, stride, rows);
    const float *p = base + min(j, rows - 1) * stride + q * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) kr[c] = *(const f32x4 *)(p + c * 16);
  };
  auto load_v = [&](int b, int32_t page) {
    int64_t stride;
    int rows;
    const float *base = rows_at(a.v_pages, a.v_tree, b, page, stride, rows);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < NH; ++h)
        vr[e][h] = *(const f32x4 *)(base + min(q * 4 + e, rows - 1) * stride + h * 64 + j * 4);
  };

  f32x4 o[RB][NH][4];
  float m[RB], l[RB];
  int32_t page = -1;   // of the block in kr / vr
  auto start = [&]() {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      m[rb] = -FLT_MAX;
      l[rb] = 0.f;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) o[rb][h][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (b0 < b1) {
      page = page_of(b0);
      load_k(b0, page);
      load_v(b0, page);
    }
  };
  start();
  // The ancestor sets of the lane's rows' nodes, while the first block's loads
  // are in flight: bit i is 1 when node i is on the root-to-node path.  The
  // walk stops at anything that is not a parent strictly before its child.
  uint32_t an[RB][4];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) an[rb][0] = an[rb][1] = an[rb][2] = an[rb][3] = 0;
  if (has_tree) {
    wave_lds_sync();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      int v = min((row0 + rb * 16 + j) / G, n - 1);
      for (int step = 0; step < kMaxTreeNodes; ++step) {
#pragma unroll
        for (int w = 0; w < 4; ++w) an[rb][w] = set_bit_in(an[rb][w], w, v);
        if (v == 0) break;
        const int p = par[v];
        if (p < 0 || p >= v) break;
        v = p;
      }
    }
  }

  // The values of block b that are not finite, taken out of vr and added to the
  // rows that weigh them.
  auto add_not_finite = [&](const f32x4 (&s)[RB], int b) {
    bool finite = true;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) finite = finite && fabsf(vr[e][h][i]) < INFINITY;
    if (__all(finite)) return;
    int64_t stride;
    int rows;
    const float *vb = rows_at(a.v_pages, a.v_tree, b, page, stride, rows);
    if (page < 0 && b < n_prefix_blocks) rows = 0;   // a zero page
#pragma unroll 1
    for (int key = 0; key < rows; ++key) {
      const float *vp = vb + key * stride + q * 16;
      float p[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float p01 = (key & 1) ? s[rb][1] : s[rb][0], p23 = (key & 1) ? s[rb][3] : s[rb][2];
        p[rb] = __shfl((key & 2) ? p23 : p01, (key >> 2) * 16 + j, 64);
      }
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 v = *(const f32x4 *)(vp + h * 64 + i * 4);   // o[.][h][k][i] is column 64 h + 16 q + 4 i + k
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              if (p[rb] != 0.f && !(fabsf(v[k]) < INFINITY)) o[rb][h][k][i] = fmaf(p[rb], v[k], o[rb][h][k][i]);
          __builtin_amdgcn_sched_barrier(0);   // one load's values at a time: no registers are left for more
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) vr[e][h][i] = fabsf(vr[e][h][i]) < INFINITY ? vr[e][h][i] : 0.f;
  };
  // The next block's K and V replace this one's as soon as they are used
  // (past the last block the last one is loaded again).
  auto blocks = [&](auto careful) {
    constexpr bool kCareful = decltype(careful)::value;
    // Puts the loop's matrix instructions where they start in the first half of
    // a 32-byte line: in the second half the loop is 2.5% slower (the 4 requests
    // above 39.1 | 40.1 us, 2 of 64 nodes over 2000 keys 55.7 | 57.4).
    if constexpr (!kCareful) asm volatile(".p2align 6\ns_nop 0\ns_nop 0\ns_nop 0\ns_nop 0");
    for (int b = b0; b < b1; ++b) {
      const int bn = min(b + 1, b1 - 1);
      const int32_t page_next = page_of(bn);
      f32x4 s[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) s[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            s[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[c][e], qf[rb][c][e], s[rb], 0, 0, 0);
      load_k(bn, page_next);

      // s[rb][e]: key 4 q + e of the block, row j
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[rb][e] *= a.sm_scale;
      const bool prefix = b < n_prefix_blocks;
      const int tb = b - n_prefix_blocks;
      const int valid = prefix ? min(kPageSize, L - b * kPageSize) : min(16, n - tb * 16);
      const bool zero_page = prefix && page < 0;
      if (!prefix || valid < 16 || zero_page) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          uint32_t seen = 0xffffu;
          if (!prefix) {
            const uint32_t w0 = an[rb][0], w1 = an[rb][1], w2 = an[rb][2], w3 = an[rb][3];
            const uint32_t w = (tb & 4) ? ((tb & 2) ? w3 : w2) : ((tb & 2) ? w1 : w0);
            seen = (tb & 1) ? w >> 16 : w;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = q * 4 + e;
            const float x = zero_page ? 0.f : s[rb][e];
            s[rb][e] = key < valid && ((seen >> key) & 1u) ? x : -INFINITY;
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int h = 0; h < NH; ++h)
            if (zero_page || q * 4 + e >= valid) vr[e][h] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      float mn[RB];
      bool up = false;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float bm = max_over_lane_rows(__builtin_elementwise_maximum(__builtin_elementwise_maximum(s[rb][0], s[rb][1]),
                                                                          __builtin_elementwise_maximum(s[rb][2], s[rb][3])));
        mn[rb] = bm > m[rb] ? bm : m[rb];
        up |= bm > m[rb];
      }
      if (__any(up)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const float al = expf(m[rb] - mn[rb]);
          m[rb] = mn[rb];
          l[rb] *= al;
#pragma unroll
          for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[rb][h][i] *= al;
        }
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[rb][e] = expf(s[rb][e] - m[rb]);
          l[rb] += s[rb][e];
        }
      if constexpr (kCareful) add_not_finite(s, b);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              o[rb][h][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[e][h][i], s[rb][e], o[rb][h][i], 0, 0, 0);
      load_v(bn, page_next);
      page = page_next;
    }
  };
  blocks(std::false_type{});
  // A key of weight 0 (a node off the row's path above all) adds nothing,
  // whatever its V, but 0 * Inf is NaN on the matrix cores.  A wave whose output
  // holds a NaN goes over its keys again with the values that are not finite
  // kept out of the products.  (Testing every block's V as it is used instead
  // cost 10% at D = 128, 40.0 -> 43.9 us for the 4 requests above; testing the
  // merged rows, which takes a barrier more, 9% for many short units, 128
  // requests of 16 nodes over 100 keys, 8 / 8 heads, D = 64: 34.1 -> 37.3.)
  float nan[2] = {0.f, 0.f};   // maxima, which a NaN passes through
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          nan[i] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(nan[i], o[rb][h][k][i]), o[rb][h][k][i + 2]);
  nan[0] = __builtin_elementwise_maximum(nan[0], nan[1]);
  if (__builtin_expect(__any(nan[0] != nan[0]), 0)) {
    page_base = b0;
    load_pages();
    start();
    blocks(std::true_type{});
  }

  // The waves' (max, sum, output) to LDS, then the merge.
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int rl = rb * 16 + j;
    const float ls = sum_over_lane_rows(l[rb]);
    if (q == 0) {
      mw[wave][rl] = m[rb];
      lw[wave][rl] = ls;
    }
    float *dst = mo + (wave * RT + rl) * LDO;
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(f32x4 *)(dst + h * 64 + q * 16 + i * 4) =
            f32x4{o[rb][h][0][i], o[rb][h][1][i], o[rb][h][2][i], o[rb][h][3][i]};
  }
  __syncthreads();
  for (int it = tid; it < RT * (D / 4); it += kT) {
    const int rl = it / (D / 4), col = it % (D / 4) * 4;
    const int row = row0 + rl;
    if (row >= M) continue;
    float mm = mw[0][rl];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, mw[w][rl]);
    float den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wt = expf(mw[w][rl] - mm);
      den += wt * lw[w][rl];
      acc += *(const f32x4 *)(mo + (w * RT + rl) * LDO + col) * wt;
    }
    const int node = row / G, hh = row - node * G;
    f32x4 res = {0.f, 0.f, 0.f, 0.f};
    if (den > 0.f) res = acc / den;
    *(f32x4 *)((float *)a.out + ((int64_t)(node_base + node) * a.num_q_heads + g * G + hh) * D + col) = res;
  }
}

}  // namespace

// Split-KV partial results of adaserve_tree_attn_verify_noalloc, for callers
// that cannot allocate: every call on a device shares that device's copy.
// The kernels take its device address (from hipGetSymbolAddress, below) as
// their workspace pointer, exactly like a caller's workspace; the array's
// name is only a host-side stand-in and is never passed to a kernel.
static __device__ __align__(256) unsigned char scratch[ADASERVE_TREE_ATTN_SCRATCH_BYTES];

hipError_t tree_attn_scratch(void **out) {
  static std::mutex mu;
  static void *addr[256];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 256) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || (uintptr_t)p % 256 != 0) return hipErrorInvalidValue;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

// Device address of g_zero16 on the current device, looked up once per device.
static hipError_t zero16_address(const void **out) {
  static std::mutex mu;
  static const void *addr[256];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 256) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_zero16));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

// The attention grid (and, in the one-call step, the argmax workgroups after
// it) with the K/V load hint the plan chose.
static void launch_attention(const TreeAttnArgs &a, int head_dim, int64_t blocks, hipStream_t stream) {
  const dim3 grid((unsigned)blocks), block(kThreads);
  if (head_dim == 128) {
    if (a.stream_kv)
      hipLaunchKernelGGL((tree_attn_bf16_kernel<128, true>), grid, block, 0, stream, a);
    else
      hipLaunchKernelGGL((tree_attn_bf16_kernel<128, false>), grid, block, 0, stream, a);
  } else {
    if (a.stream_kv)
      hipLaunchKernelGGL((tree_attn_bf16_kernel<64, true>), grid, block, 0, stream, a);
    else
      hipLaunchKernelGGL((tree_attn_bf16_kernel<64, false>), grid, block, 0, stream, a);
  }
}

hipError_t launch_tree_attn_bf16(TreeAttnArgs &a, int head_dim, bool needs_combine, hipStream_t stream) {
  if (a.units == 0) return hipSuccess;
  hipError_t e = zero16_address(&a.zero16);
  if (e != hipSuccess) return e;
  const dim3 block(kThreads);
  launch_attention(a, head_dim, a.padded_grid, stream);
  e = hipGetLastError();
  if (e != hipSuccess || !needs_combine) return e;
  const dim3 cgrid((unsigned)a.merge_blocks);
  if (head_dim == 128)
    hipLaunchKernelGGL(tree_attn_combine_kernel<128>, cgrid, block, 0, stream, a);
  else
    hipLaunchKernelGGL(tree_attn_combine_kernel<64>, cgrid, block, 0, stream, a);
  return hipGetLastError();
}

template <int D, int RB>
static void launch_f32_tile(const TreeAttnArgs &a, int64_t blocks, hipStream_t stream) {
  hipLaunchKernelGGL((tree_attn_f32_kernel<D, RB>), dim3((unsigned)blocks), dim3(kWavesF32 * 64), 0, stream, a);
}

hipError_t launch_tree_attn_f32(const TreeAttnArgs &a, int head_dim, int64_t blocks, hipStream_t stream) {
  if (blocks == 0) return hipSuccess;
  const bool wide = a.rows_per_tile == 32;
  if (head_dim == 128)
    wide ? launch_f32_tile<128, 2>(a, blocks, stream) : launch_f32_tile<128, 1>(a, blocks, stream);
  else
    wide ? launch_f32_tile<64, 2>(a, blocks, stream) : launch_f32_tile<64, 1>(a, blocks, stream);
  return hipGetLastError();
}

// An F32 argmax workgroup in the attention's grid takes the LDS and registers
// of an F32 attention workgroup, so a CU holds one: many short rows wait for
// their turn, and go into a launch of their own (full step, beside | apart:
// 16 / 4 heads, D = 128, 32-node trees over 400 keys, vocabulary 4096: 256 rows
// 27.0 | 30.0 us, 512 41.8 | 40.8, 1024 75.7 | 70.7, 4096 282 | 252; 4 / 4
// heads 512 rows 24.2 | 28.8, 1024 34.2 | 30.8, 4096 112 | 81).  Long rows stream
// as fast either way (65536 columns: 1024 rows 107 | 109, 2048 201 | 204;
// 16384: 1024 78.1 | 77.7, 4096 292 | 282).
constexpr int kF32RowsBeside = 768, kF32LongRow = 32768;

hipError_t launch_verify_step(TreeAttnArgs &a, int head_dim, bool bf16, bool needs_combine, hipStream_t stream) {
  hipError_t e = zero16_address(&a.zero16);
  if (e != hipSuccess) return e;
  const dim3 block(kThreads);
  const bool apart = !bf16 && a.argmax_rows > kF32RowsBeside && a.vocab <= kF32LongRow;
  const int64_t g1 = (a.units > 0 ? a.padded_grid : 0) + (apart ? 0 : a.argmax_rows);
  if (a.units == 0) a.padded_grid = 0;
  if (g1 > 0) {
    if (bf16) {
      launch_attention(a, head_dim, g1, stream);
      e = hipGetLastError();
    } else {
      e = launch_tree_attn_f32(a, head_dim, g1, stream);
    }
    if (e != hipSuccess) return e;
  }
  if (apart) {
    e = launch_node_argmax(a.logits, a.logit_stride, a.argmax_rows, a.vocab, bf16, a.argmax_out, stream);
    if (e != hipSuccess) return e;
  }
  if (!needs_combine) a.merge_blocks = 0;
  const int64_t g2 = a.merge_blocks + (a.accept_requests + kThreads / 64 - 1) / (kThreads / 64);
  if (g2 == 0) return hipSuccess;
  if (head_dim == 128)
    hipLaunchKernelGGL(tree_attn_combine_kernel<128>, dim3((unsigned)g2), block, 0, stream, a);
  else
    hipLaunchKernelGGL(tree_attn_combine_kernel<64>, dim3((unsigned)g2), block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace adaserve
