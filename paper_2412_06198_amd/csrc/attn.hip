// Sparse causal prefill attention for gfx950 (Alg. 2 / Alg. 3 "Compute Sparse
// Attention": softmax over the kept keys only, then the product with V).
//
// One workgroup = 128 query rows of one head (4 waves x 32 rows), two workgroups
// per compute unit, fed from work queues.  A (head, row block) item has two phases:
//   * tiles of 64 keys through LDS, shared by the four waves:
//       range tiles  - aligned key tiles of the key blocks the CSR keeps;
//       gather tiles - 64 selected key columns, gathered once per call into
//                      contiguous buffers, so that they are read like any tile;
//   * selected diagonals, one 32-key tile per wave and offset, without barriers.
// A key is counted once: selected columns are masked out of range tiles and
// diagonal entries whose key is a selected column or lies in a kept block are
// dropped.  Per tile each wave computes S^T = K Q^T (keys x queries) with
// v_mfma_f32_32x32x16_bf16, so that one lane owns one query: the online softmax
// needs a single cross-lane exchange, and the probabilities are already laid out
// as the B operand of O^T += V^T P^T.
#include "sa_internal.h"

namespace sa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int BQ = 128;           // query rows per workgroup
constexpr int BK = 64;            // keys per tile
// Consecutive row blocks that a queue takes before it passes over those of the queues that share its KV
// head: what an XCD has in progress together (64 workgroups), so that the diagonals of its row blocks
// read one stretch of keys per offset, not every second row block's of one twice as long (128K tokens,
// 32 heads: 4.07 -> 3.98 ms).
constexpr int kRunBits = 6, kRun = 1 << kRunBits;
constexpr int NWORDS = kMaxSeq / BK / 32;
constexpr int kPlanWaves = 4;     // items per workgroup of index_prepare_kernel
constexpr unsigned kNoItem = ~0u;
static_assert(kMaxHeads == 128 && kMaxSeq / BQ <= 2048, "an item's heads and row block fill a word");
// Diagonals whose scores are taken before their products with V: as many as leave two workgroups a compute
// unit's LDS.
constexpr int kDiagBatch = 28;

struct AttnArgs {
  const uint16_t *Q, *K, *V;
  uint16_t *O;
  const int32_t *n_cols, *cols, *n_offs, *offs, *rowptr, *blkcols;
  const uint32_t *colbits;   // [Hq][N/32] membership bitmap of the selected columns
  const int32_t *colprefix;  // [Hq][N/32] selected columns before each word of colbits
  uint16_t *Kg, *Vg;  // [Hq][kvg_rows][kv_rs] selected key columns, gathered once per call
  int kvg_rows;
  int Hq, Hkv, g, gq, N, b, nb, nT, k_v, k_s, cap_b;
  int64_t q_hs, q_rs, kv_hs, kv_rs, o_hs, o_rs;
  float c;  // softmax scale * log2(e)
  unsigned int *queue;           // [8] work-queue heads, zeroed by index_prepare_kernel
  int n_items;  // (head, row block) items in all
  int share;    // log2 of the queues (XCDs) that share one KV head at a time (1, 2, 4 or 8), and from bit 4 on
                // log2 of the consecutive row blocks a queue takes in a row (kRun or 1)
  int qcap;     // tickets per queue, holes of the id space included
  int side_by_side;  // also the heads with diagonals take a row block together, see plan_item
  unsigned long long *counters;  // instrumentation only: {32x32 sub-tiles computed (a diagonal is one, and an eighth of
                                 // its products), kept (query,key) pairs}
  // Written by index_prepare_kernel.  items[queue + 8 * ticket] = {head | its query head << 7 | its KV head << 14 |
  // row block << 21, key tiles in the list (kNoItem: a hole of the id space), list start inside the head's share
  // of tiles, first two entries}; tiles [Hq][tile_cap] list entries: key tile (bits 0..11), kept by waves 0, 1
  // (bit 14) / by waves 2, 3 (bit 15).
  uint4 *items;
  uint16_t *tiles;
  unsigned tile_cap;
  int grid;     // workgroups of the attention kernel
};

// Tickets per queue and query head, holes included: whole runs of every queue that shares the KV head.
__host__ __device__ inline int tickets_per_head(int nT, int share) {
  const int bits = (share & 15) + (share >> 4);
  return ((nT + (1 << bits) - 1) >> bits) << (share >> 4);
}

// Read-only words at a wave-uniform address: through the constant address space these become
// scalar loads, which neither occupy the vector memory path nor count in vmcnt.
typedef const uint32_t __attribute__((address_space(4))) *const_u32p;
__device__ inline uint32_t uload(const void *p, int idx) { return ((const_u32p)(uintptr_t)p)[idx]; }

// Item id = queue + 8 * ticket: which head and row block it is, and the list of its key tiles.
// Ticket k of queue qn: k / per_q selects the KV head, the rest walks the row blocks from the last
// (longest) one down, in runs of which the queues that share take one each in turn, back and forth:
// first for the query heads of the group that have no selected diagonals, side by side per row block
// (their tiles overlap: the band of Triangular heads is the same for all of them), then for each head
// with diagonals by itself (their diagonal phase re-reads nothing, and one head's gathered columns
// stay in L2).  With up to four items per workgroup (side_by_side) it is the order of lengths that counts, and
// the heads with diagonals take a row block side by side too: 8 heads of one KV head, all with diagonals, 42 -> 34 us at
// 8K tokens, 81 -> 71 at 16K, 146 -> 145 at 32K (four items each), 32 heads at 8K 99 -> 97; with five and more it
// costs: 10K 177 -> 182, 32 heads at 32K 529 -> 536.  Here and not at the head of every item of the attention kernel, where the same steps
// were four barriers and three round trips to memory one after the other while the matrix cores idled:
// a whole layer of 4K, 10K, 16K, 32K and 128K tokens 59.8, 355, 432, 733 and 4543 us, now 57.0, 343, 414,
// 718 and 4499 (plain causal attention at 16K 1986 and 1961).  One wave per item.
__device__ inline void plan_item(const AttnArgs &p, int id, uint32_t *k0, uint32_t *k1, uint16_t *first2) {
  const int lane = threadIdx.x & 63;
  const int qn = id & 7, k = id >> 3;
  const int xb = p.share & 15, rb = p.share >> 4;
  const int nslots = 8 >> xb, slot = qn >> xb, sub = qn & ((1 << xb) - 1);
  const int rows_q = tickets_per_head(p.nT, p.share), per_q = rows_q * p.g;
  // This wave's item: row `trow` of the queue's rows and head j of the group.  The ticket it gets follows from the heads
  // before j and their kinds, which are needed last: the reads below do not wait for them.
  const int kvh = k / per_q * nslots + slot, j = k % per_q / rows_q, trow = k % per_q % rows_q;
  const bool head_ok = kvh < p.Hkv;
  int n_offs[2];  // a group has at most kMaxHeads = 128 heads
#pragma unroll
  for (int i = 0; i < 2; ++i) n_offs[i] = head_ok && 64 * i + lane < p.g ? p.n_offs[kvh * p.g + 64 * i + lane] : 1;
  const int h = kvh * p.g + j, rn = trow >> rb;
  const int tidx = (((rn << xb) + ((rn & 1) ? (1 << xb) - 1 - sub : sub)) << rb) + (trow & ((1 << rb) - 1));
  auto ticket_id = [&]() {
    unsigned long long w[2];  // heads without diagonals
#pragma unroll
    for (int i = 0; i < 2; ++i) w[i] = __ballot(n_offs[i] <= 0);
    const int c = __popcll(w[0]) + __popcll(w[1]);
    const bool plain = ((j < 64 ? w[0] >> j : w[1] >> (j - 64)) & 1ull) != 0ull;
    const int plain_before = j < 64 ? __popcll(w[0] & ((1ull << j) - 1ull)) : __popcll(w[0]) + __popcll(w[1] & ((1ull << (j - 64)) - 1ull));
    const int nth = plain ? plain_before : j - plain_before;  // heads of its kind before it
    const int r = plain               ? trow * c + nth
                  : p.side_by_side ? c * rows_q + trow * (p.g - c) + nth
                                   : (c + nth) * rows_q + trow;
    return qn + 8 * (k / per_q * per_q + r);
  };
  if (!head_ok || tidx >= p.nT) {  // a hole (without a KV head all heads count as having diagonals: any order)
    const int at = ticket_id();
    if (lane == 0) p.items[at] = make_uint4(0u, kNoItem, 0u, 0u);
    return;
  }
  const int t128 = p.nT - 1 - tidx;
  const int ilast = min((t128 + 1) * BQ, p.N) - 1;
  const int nwords = (ilast / BK + 1 + 31) / 32;
  for (int i = lane; i < nwords; i += 64) { k0[i] = 0u; k1[i] = 0u; }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // CSR entry ranges of the row blocks of this item: one at block 128, two (2*t128 for waves 0,1
  // and 2*t128+1 for waves 2,3) at block 64
  const int32_t *rp = p.rowptr + (size_t)h * (p.nb + 1);
  const int Ra = p.b == BQ ? t128 : 2 * t128;
  const bool two = p.b != BQ && Ra + 1 < p.nb;
  const int ea0 = max(rp[Ra], 0), ea1 = min(rp[Ra + 1], p.cap_b);
  const int eb0 = max(rp[min(Ra + 1, p.nb)], 0), eb1 = min(rp[min(Ra + 2, p.nb)], p.cap_b);
  const int na = max(ea1 - ea0, 0), nbk = two ? max(eb1 - eb0, 0) : 0;
  const int32_t *bc = p.blkcols + (size_t)h * p.cap_b;
  const int tpb = p.b / BK;  // key tiles per key block: their bits are adjacent in one word
  const uint32_t tbits = tpb == 2 ? 3u : 1u;
  for (int e0 = lane; e0 < na + nbk; e0 += 256) {
    int C[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // four reads in flight
      const int e = e0 + 64 * u;
      C[u] = e < na + nbk ? bc[e >= na ? eb0 + (e - na) : ea0 + e] : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool second = e0 + 64 * u >= na;
      if (C[u] >= 0 && C[u] <= Ra + (second ? 1 : 0)) {
        const int kt = C[u] * tpb;
        if (!second) atomicOr(&k0[kt >> 5], tbits << (kt & 31));
        if (second || p.b == BQ) atomicOr(&k1[kt >> 5], tbits << (kt & 31));
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // One tile per lane, 64 at a time: the kept ones in ascending order.  Stretches that keep none are passed
  // over by a mask of the others (a row of a long sequence has thousands of tiles and keeps some thirty:
  // without it this launch took 46 us at 128K tokens and 32 heads, 34 with it).  Scattered
  // ones, up to three in a stretch, are taken by the lanes beside each other, each its own: with that, and the heads' kinds
  // read beside the row pointers and not before them, 29.6 us (64K tokens 19.6 -> 16.8, 32K 12.2 -> 11.0).
  const unsigned start = (unsigned)min(ea0, p.cap_b) * tpb;
  const unsigned room = p.tile_cap - start;
  uint16_t *out = p.tiles + (size_t)h * p.tile_cap + start;
  unsigned base = 0;
  static_assert(NWORDS <= 128, "one lane per pair of words");
  uint32_t mine[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) mine[i] = 2 * lane + i < nwords ? k0[2 * lane + i] | k1[2 * lane + i] : 0u;
  unsigned long long pairs = __ballot((mine[0] | mine[1]) != 0u);
  const unsigned count = __popc(mine[0]) + __popc(mine[1]), upto = wave_inclusive_sum(count);
  const unsigned total = __builtin_amdgcn_readlane(upto, 63);
  if (total <= 3u * __popcll(pairs)) {  // scattered tiles: each lane those of its own words
    unsigned pos = upto - count;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int w = 2 * lane + i;
      for (uint32_t m = mine[i]; m != 0u; m &= m - 1u, ++pos) {
        const int bit = __ffs(m) - 1;
        const uint16_t ent = (uint16_t)((w * 32 + bit) | ((k0[w] >> bit) & 1u) << 14 | ((k1[w] >> bit) & 1u) << 15);
        if (pos < room) {
          out[pos] = ent;
          if (pos < 2) first2[pos] = ent;
        }
      }
    }
    base = total;
    pairs = 0ull;
  }
  for (; pairs != 0ull; pairs &= pairs - 1ull) {
    const int w0 = 2 * (__ffsll(pairs) - 1), w = w0 + (lane >> 5);
    const uint32_t a = w < nwords ? (k0[w] >> (lane & 31)) & 1u : 0u, b = w < nwords ? (k1[w] >> (lane & 31)) & 1u : 0u;
    const unsigned long long m = __ballot((a | b) != 0u);
    const unsigned pos = base + (unsigned)__popcll(m & ((1ull << lane) - 1ull));
    if ((a | b) != 0u && pos < room) {
      const uint16_t ent = (uint16_t)((w0 * 32 + lane) | (a << 14) | (b << 15));
      out[pos] = ent;
      if (pos < 2) first2[pos] = ent;
    }
    base += (unsigned)__popcll(m);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const unsigned n = min(base, room);
  const int at = ticket_id();
  if (lane == 0)
    p.items[at] = make_uint4((unsigned)h | (unsigned)query_head(h, p.g, p.gq) << 7 | (unsigned)kvh << 14 | (unsigned)t128 << 21, n, start,
                             (n > 0 ? first2[0] : 0u) | (n > 1 ? (unsigned)first2[1] << 16 : 0u));
}

// What the attention kernel needs from the index before it starts, in one launch of 256-thread
// blocks.  Blocks 0 .. Hq-1: membership bitmap of a head's selected columns and the running count
// of selected columns before each bitmap word (built in LDS, written out once); block 0 also
// resets the work-queue heads (a workgroup's first ticket is its own number, so they start behind
// those).  The next blocks: one wave per item, plan_item.  The rest, (gather tile g, head h):
// the selected key columns of every head are copied once into contiguous [k][d] buffers so that
// the attention kernel reads gather tiles like any other tile.
__global__ __launch_bounds__(256) void index_prepare_kernel(AttnArgs p, unsigned int *queue, int n_bitmap_words) {
  extern __shared__ uint32_t bm[];  // the bitmap of a head, or two key-tile bitmaps per wave
  __shared__ int wsum[4];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < p.Hq) {
    const int h = blockIdx.x, nw = p.N / 32, lane = tid & 63, wv = tid >> 6;
    if (h == 0 && tid < 8) queue[tid] = (unsigned)(p.grid + 7 - tid) >> 3;
    for (int i = tid; i < nw; i += 256) bm[i] = 0u;
    __syncthreads();
    const int nc = min(max(p.n_cols[h], 0), p.k_v);
    for (int i = tid; i < nc; i += 256) {
      const int c = p.cols[(size_t)h * p.k_v + i];
      if (c >= 0 && c < p.N) atomicOr(&bm[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    // exclusive prefix popcount: thread t owns a contiguous run of words
    const int per = (nw + 255) / 256;
    const int w0 = min(tid * per, nw), w1 = min(w0 + per, nw);
    int mine = 0;
    for (int w = w0; w < w1; ++w) mine += __popc(bm[w]);
    int incl = mine;
    for (int dd = 1; dd < 64; dd <<= 1) {
      const int o = __shfl_up(incl, dd);
      if (lane >= dd) incl += o;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int run = incl - mine;
    for (int k = 0; k < wv; ++k) run += wsum[k];
    uint32_t *cb = const_cast<uint32_t *>(p.colbits) + (size_t)h * nw;
    int32_t *cp = const_cast<int32_t *>(p.colprefix) + (size_t)h * nw;
    for (int w = w0; w < w1; ++w) {
      const uint32_t word = bm[w];
      cb[w] = word;
      cp[w] = run;
      run += __popc(word);
    }
    return;
  }
  const int n_plan = (8 * p.qcap + kPlanWaves - 1) / kPlanWaves;
  if ((int)blockIdx.x < p.Hq + n_plan) {
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int id = ((int)blockIdx.x - p.Hq) * kPlanWaves + wv;
    const int words = n_bitmap_words / (2 * kPlanWaves);
    uint32_t *k0 = bm + 2 * words * wv;
    if (id < 8 * p.qcap) plan_item(p, id, k0, k0 + words, (uint16_t *)&wsum[wv]);
    return;
  }
  const int ntile = p.kvg_rows / BK, gb = (int)blockIdx.x - p.Hq - n_plan;
  const int h = gb / ntile, g = gb % ntile;
  const int kvh = h / p.g;
  const int lrow = tid >> 4, lcc = tid & 15;
  int col[4];  // on their way before their number is known
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int ci = g * BK + lrow + 16 * n;
    col[n] = ci < p.k_v ? p.cols[(size_t)h * p.k_v + ci] : 0;
  }
  const int nc = min(max(p.n_cols[h], 0), p.k_v);
  if (g * BK >= nc) return;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int ci = g * BK + lrow + 16 * n;
    const int src = min(max(ci < nc ? col[n] : 0, 0), p.N - 1);
    const size_t so = (size_t)kvh * p.kv_hs + (size_t)src * p.kv_rs + lcc * 8;
    const size_t dofs = ((size_t)h * p.kvg_rows + ci) * p.kv_rs + lcc * 8;  // same row stride as K / V
    *(uint4 *)(p.Kg + dofs) = *(const uint4 *)(p.K + so);
    *(uint4 *)(p.Vg + dofs) = *(const uint4 *)(p.V + so);
  }
}

// LDS tiles are 64 rows x 256 B with the 16-byte chunks of a row XOR-swizzled (no padding):
//   K: chunk c of row r sits at chunk c ^ (r & 15)      -> b128 reads of 16 rows hit 64 banks
//   V: chunk c of row r sits at chunk c ^ ((r & 3) << 2) -> the transposing b64 reads do

// The larger of a lane's value and that of the lane 32 away, in both.  A shuffle through LDS queues behind
// the operand reads of eight waves and every tile waits for it: with the half-wave swap and the order of
// the K products plain causal attention at 16K tokens takes 1860 us instead of 1905, a layer of 32K 695
// instead of 711.
__device__ inline float max_pair(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The sum of a lane's value and that of the lane 32 away, in both.
__device__ inline float sum_pair(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// G groups of four waves share an item: group j takes every G-th tile and diagonal from the j-th on, with buffers of
// its own, and the groups' sums are merged at the end.  With G = 1 two workgroups live on a compute unit, with G = 2
// one: see split_items for where that pays.
template <bool STATS, int G>
__global__ __launch_bounds__(256 * G, 2) void sparse_prefill_kernel(AttnArgs p) {
  __shared__ __attribute__((aligned(16))) uint16_t Ks[G][2][BK * 128];
  __shared__ __attribute__((aligned(16))) uint16_t Vs[G][2][BK * 128];
  __shared__ uint32_t kept0[NWORDS], kept1[NWORDS];
  // the item's list of key tiles; later the scores of a batch of diagonals, [offset][query]
  __shared__ __attribute__((aligned(16))) float dscore[G][kDiagBatch * BQ];
  static_assert(sizeof(dscore[0]) >= kMaxSeq / BK * 2, "holds the list");
  uint16_t *const tlist = (uint16_t *)dscore[0];

  // wave-uniform for the compiler too; the wave inside its group
  const int grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) - 4 * grp;

  // Persistent workgroups pull (head, row block) items from eight queues, one per XCD
  // (consecutive workgroup ids land on consecutive XCDs).  1, 2, 4 or 8 queues share one KV head at a
  // time: alone, a queue keeps its KV head in a single L2; with more of them fewer KV heads are live at
  // once, so that the rows the diagonal phase fetches (little reuse inside an L2) are in the
  // memory-side cache rather than in HBM.  plan_item has written down what every ticket stands for.  A
  // workgroup whose own queue is empty takes from the others, then exits.  The first ticket is the
  // workgroup's number; the one for the next item of the home queue is drawn while the current item
  // finishes, so its round trip is off the critical path.
  __shared__ int s_item;
  const int home = blockIdx.x & 7;
  int ticket = blockIdx.x >> 3;  // thread 0: position drawn from the home queue, not used yet; past its end: closed
  for (;;) {
  // Lane-derived constants are recomputed per item from an opaque copy of the thread id:
  // hoisted out of this loop they would stay live across every phase and spill.
  int tid = threadIdx.x;  // inside its group
  asm volatile("" : "+v"(tid));
  if (G > 1) tid &= 255;
  const int lane = tid & 63, q = lane & 31, gg = lane >> 5;
  __syncthreads();  // previous item fully retired: LDS work lists and tiles may be reused
  if (wv == 0 && grp == 0) {
    const int drawn = __builtin_amdgcn_readfirstlane(ticket);
    int item = drawn < p.qcap ? home + 8 * drawn : -1;
    if (item < 0) {
      // All queue heads in one read.  Every workgroup passes here at the end, and the reads go past the
      // L2: one after the other they kept it for several us from the work other queues still had (a layer
      // of 10K tokens 345 -> 335 us, 16K 405 -> 395, 4K 57.3 -> 56.1; from 64K on no difference).
      const int head = lane < 8 ? (int)__hip_atomic_load(&p.queue[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : p.qcap;
      unsigned open = (unsigned)__ballot(head < p.qcap) & ~(1u << home);
      while (open != 0u && item < 0) {
        const int qn = (home + __ffs((open | open << 8) >> home) - 1) & 7;  // the next one after home
        open &= ~(1u << qn);
        int k = 0;
        if (lane == 0) k = (int)atomicAdd(&p.queue[qn], 1u);
        k = __builtin_amdgcn_readfirstlane(k);
        if (k < p.qcap) item = qn + 8 * k;
      }
    }
    if (lane == 0) s_item = item;
  }
  if (tid < NWORDS) { kept0[tid] = 0u; kept1[tid] = 0u; }
  __syncthreads();
  const int id = __builtin_amdgcn_readfirstlane(s_item);
  if (id < 0) break;
  const uint32_t it_w = uload(p.items, 4 * id), it_n = uload(p.items, 4 * id + 1);
  const uint32_t it_at = uload(p.items, 4 * id + 2), it_e = uload(p.items, 4 * id + 3);
  if (it_n == kNoItem) {  // a hole of the id space
    if (tid == 0 && grp == 0 && ticket < p.qcap) ticket = (int)atomicAdd(&p.queue[home], 1u);
    continue;
  }
  const int h = (int)(it_w & 127u), qh = (int)(it_w >> 7 & 127u), kvh = (int)(it_w >> 14 & 127u), t128 = (int)(it_w >> 21);
  const int ntr = (int)it_n;
  const int i0 = t128 * BQ;
  const int r0 = i0 + 32 * wv;
  const int iq = r0 + q;  // this lane's query row
  const int N = p.N;
  const int ilast = min(i0 + BQ, N) - 1;

  // ---- operands ------------------------------------------------------------------------------
  const uint16_t *__restrict__ Kh = p.K + (size_t)kvh * p.kv_hs;
  const uint16_t *__restrict__ Vh = p.V + (size_t)kvh * p.kv_hs;
  const uint16_t *__restrict__ Kgh = p.Kg + (size_t)h * p.kvg_rows * p.kv_rs;
  const uint16_t *__restrict__ Vgh = p.Vg + (size_t)h * p.kvg_rows * p.kv_rs;
  const uint32_t *__restrict__ colbm = p.colbits + (size_t)h * (N / 32);

  f32x16 oacc[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 lacc[2] = {};  // the tile loop's share of the normaliser (every register of a lane holds the same sum)
  unsigned st_kept = 0u, st_tiles = 0u;  // counted variant: this lane's kept pairs, this wave's sub-tiles

  // ---- global -> LDS pipeline -----------------------------------------------------------------
  // K and V tiles go straight from global memory into LDS (global_load_lds_dwordx4: 16 bytes per
  // lane, LDS address = M0 + 16*lane, so one instruction fills four 256-byte rows).  The XOR
  // swizzle is applied on the global side: the lane that owns physical chunk pc of row r fetches
  // logical chunk pc ^ swz(r).  Wave w moves rows 4w..4w+3 (+16n, n = 0..3) of both tiles.
  const int rl = 4 * wv + (lane >> 4);  // (row & 15) of the rows this lane moves; (row & 3) = lane >> 4
  const unsigned dmaK = (unsigned)(rl * (int)p.kv_rs * 2 + (((lane & 15) ^ rl) << 4));
  const unsigned dmaV = (unsigned)(rl * (int)p.kv_rs * 2 + (((lane & 15) ^ ((lane >> 4) << 2)) << 4));
  const unsigned ldsK0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)&Ks[grp][0][0] + 4 * wv * 256;
  const unsigned ldsV0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)&Vs[grp][0][0] + 4 * wv * 256;
  const size_t row16 = 16 * (size_t)p.kv_rs;  // elements between the rows of consecutive instructions
#define SA_DMA16(gptr, voff, ldsb)                                                                    \
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(gptr), \
               "s"(ldsb)                                                                              \
               : "memory")
#define SA_ISSUE_TILE(t, buf, ent)                                                                  \
  {                                                                                              \
    const uint16_t *kb, *vb;                                                                     \
    if ((t) < ntr) {                                                                             \
      const size_t j0_ = (size_t)((ent) & 0xFFF) * BK * p.kv_rs;                                 \
      kb = Kh + j0_; vb = Vh + j0_;                                                              \
    } else {                                                                                     \
      const size_t g0_ = (size_t)((t) - ntr) * BK * p.kv_rs;                                     \
      kb = Kgh + g0_; vb = Vgh + g0_;                                                            \
    }                                                                                            \
    const unsigned lk = ldsK0 + (buf) * (BK * 256), lv = ldsV0 + (buf) * (BK * 256);             \
    SA_DMA16(kb, dmaK, lk); SA_DMA16(kb + row16, dmaK, lk + 16 * 256);                           \
    SA_DMA16(kb + 2 * row16, dmaK, lk + 32 * 256); SA_DMA16(kb + 3 * row16, dmaK, lk + 48 * 256); \
    SA_DMA16(vb, dmaV, lv); SA_DMA16(vb + row16, dmaV, lv + 16 * 256);                           \
    SA_DMA16(vb + 2 * row16, dmaV, lv + 32 * 256); SA_DMA16(vb + 3 * row16, dmaV, lv + 48 * 256); \
  }

  // per-lane LDS byte offsets of the operand reads.  The swizzles only touch address bits 4..7,
  // so every access is (one per-lane base) XOR (a compile-time constant):
  //   K (A of S^T): row 32hf + q, chunk 2ks + gg -> b128 at kbase ^ ((2ks + gg) << 4) + 32hf*256
  //   V (A of O^T, transposing read): within 16 lanes, source lane r supplies the 8-byte piece
  //   (key r/4, d 4(r%4)..+3) and receives (keys 0..3, d r); lanes 16..31 take d 16..31:
  //   row 4gg + r/4 (+ multiples of 4), chunk 4db + 2grp + (r%4)/2 -> b64 at vbase ^ (db << 6)
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const unsigned kbase = (unsigned)(q * 256) | (unsigned)((q & 15) << 4);
  unsigned vbase;
  {
    const int r = lane & 15, grp = (lane >> 4) & 1;
    const int row = 4 * gg + (r >> 2);
    vbase = (unsigned)(row * 256) | (unsigned)(((2 * grp + ((r & 3) >> 1)) ^ ((row & 3) << 2)) << 4) |
            (unsigned)((r & 1) << 3);
  }
#define SA_KFRAG(tile, hf, ks) \
  (*(const bf16x8 *)((const char *)(tile) + ((kbase ^ (unsigned)((2 * (ks) + gg) << 4)) + (hf) * 32 * 256)))
#define SA_VTR(tile, db, key0) \
  __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)((const char *)(tile) + ((vbase ^ (unsigned)((db) << 6)) + (key0) * 256)))

  // list entries travel one tile ahead in scalar registers, so that neither the copy of the next
  // tile nor this tile's keep test waits for an LDS read behind the barrier
  int e_cur = (int)((grp ? it_e >> 16 : it_e) & 0xFFFFu);
  int r_nxt = (int)(it_e >> 16);  // from LDS later on: made scalar only where it is used, a tile later
  if (grp < ntr) SA_ISSUE_TILE(grp, 0, e_cur);

  // the item's other reads, all in flight together with the first tile's copies
  bf16x8 qf[8];  // Q^T fragments: B operand, lane = query, 8 consecutive d per k-step half
  {
    const uint16_t *qrow = p.Q + (size_t)qh * p.q_hs + (size_t)min(iq, N - 1) * p.q_rs;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = *(const bf16x8 *)(qrow + 16 * ks + 8 * gg);
  }
  const bool has_offs = (int)uload(p.n_offs, h) > 0;
  const int nc = min(max((int)uload(p.n_cols, h), 0), p.k_v);
  const bool has_cols = nc > 0;
  // Selected columns visible to a query = those up to its own position: the running count before its
  // bitmap word plus the bits of that word up to the position (the list is ascending and without
  // repeats, so this is also the query's cut in the gathered list).  The 32 queries of a wave share a
  // word, the last of the row block ends one.
  int cle, cwave, cwmin, call;  // this lane's query; the wave's last and first; the row block's last
  {
    const int32_t *cp = p.colprefix + (size_t)h * (N / 32);
    const int wi = min(r0, N - 1) >> 5, wl = ilast >> 5;
    const int before = (int)uload(cp, wi);
    const uint32_t word = uload(colbm, wi);
    cle = has_cols ? before + __popc(word & (0xFFFFFFFFu >> (31 - q))) : 0;
    cwave = has_cols ? before + __popc(word) : 0;
    cwmin = has_cols ? before + (int)(word & 1u) : 0;
    call = has_cols ? (int)uload(cp, wl) + __popc(uload(colbm, wl)) : 0;
  }
  const int ng = (call + BK - 1) / BK;
  const int ntot = ntr + ng;
  if (grp >= ntr && grp < ntot) SA_ISSUE_TILE(grp, 0, e_cur);
  {
    // the list, for the tile loop (read behind its first barrier), and the kept tiles as bitmaps, for the diagonals
    const uint16_t *tl = p.tiles + (size_t)h * p.tile_cap + it_at;
    if (G > 1) r_nxt = G + grp < ntr ? tl[G + grp] : 0;
    for (int i = tid + 256 * grp; i < ntr; i += 256 * G) {
      const int ent = tl[i];
      tlist[i] = (uint16_t)ent;
      if (has_offs) {
        const int kt = ent & 0xFFF;
        if (ent & 0x4000) atomicOr(&kept0[kt >> 5], 1u << (kt & 31));
        if (ent & 0x8000) atomicOr(&kept1[kt >> 5], 1u << (kt & 31));
      }
    }
  }

  const int n_step = (ntot + G - 1) / G;
  for (int step = 0; step < n_step; ++step) {
    const int t = G * step + grp, cur = step & 1;
    // this wave's share of tile t has landed (nothing else is in flight); after the barrier the
    // whole tile is in LDS[cur] and every wave has finished reading LDS[cur^1] (tile t-1)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    const int e_nxt = __builtin_amdgcn_readfirstlane(r_nxt);
    if (t + G < ntot) SA_ISSUE_TILE(t + G, cur ^ 1, e_nxt);
    const int e_this = e_cur;
    e_cur = e_nxt;
    r_nxt = (int)tlist[min(t + 2 * G, kMaxSeq / BK - 1)];

    // ---- what this wave keeps of the tile: a 64-bit mask per lane over the key slots ---------
    // slot c (0..59 used) stands for key_local = c + 4*gg; see the accumulator layout below.
    // Without selected columns inside the tile the mask is a threshold (slot c kept iff c <= lim),
    // applied with one compare per element; km is then only needed by the counted variant.
    bool active, needmask, bits = false;
    uint64_t km;
    int lim = 63;
    if (t < ntr) {
      const int kt = e_this & 0xFFF;
      const int j0 = kt * BK;
      const bool bk = ((e_this >> (wv < 2 ? 14 : 15)) & 1) != 0;
      const bool beyond = j0 > min(r0 + 31, N - 1);
      active = !beyond && bk;
      const uint64_t vm = has_cols ? ((uint64_t)uload(colbm, 2 * kt) | ((uint64_t)uload(colbm, 2 * kt + 1) << 32)) : 0ull;
      needmask = !(vm == 0 && j0 + 63 <= r0);
      km = ~0ull;
      bits = vm != 0;
      if (active && needmask) {
        lim = iq - j0 - 4 * gg;  // causal: slot c kept iff c <= lim
        const uint64_t cm = lim < 0 ? 0ull : (lim >= 63 ? ~0ull : ((2ull << lim) - 1ull));
        km = cm & ~(vm >> (4 * gg));  // selected columns are served by the gather tiles
      }
    } else {
      const int gi = t - ntr;
      active = cwave > gi * BK;
      needmask = cwmin < (gi + 1) * BK;  // some query of the wave sees only a part of this tile
      km = ~0ull;
      if (needmask) {
        lim = cle - gi * BK - 1 - 4 * gg;  // visible columns of this tile for this query, as a slot limit
        km = lim < 0 ? 0ull : (lim >= 63 ? ~0ull : ((2ull << lim) - 1ull));
      }
    }
    if (!active) continue;
    if constexpr (STATS) {
      // slots this lane owns: c = 32hf + 8(r/4) + r%4
      st_kept += iq < N ? (unsigned)__popcll(km & 0x0F0F0F0F0F0F0F0Full) : 0u;
      st_tiles += 2u;
    }

    // ---- S^T = K Q^T : lane = query (q), accumulator r of half hf <-> key 32hf + 8(r/4) + 4gg + r%4
    const uint16_t *Kt = Ks[grp][cur];
    f32x16 sacc[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[hf][r] = 0.f;
    {
      // The 16 K fragments go through a ring of four registers: the LDS read of fragment i+4 is
      // issued right after the MFMA that consumed fragment i, so reads stay 3-4 deep in flight.  Fenced
      // in this order: left to itself the compiler let the second product wait for the read just issued.
      // The two key halves take turns, so that a product does not follow the one whose sums it adds to.
      bf16x8 kf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) kf[i] = SA_KFRAG(Kt, i & 1, i >> 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int hf = i & 1, ks = i >> 1;
        sacc[hf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i & 3], qf[ks], sacc[hf], 0, 0, 0);
        if (i + 4 < 16) kf[i & 3] = SA_KFRAG(Kt, (i + 4) & 1, (i + 4) >> 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (needmask) {
      if (bits) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = 32 * hf + 8 * (r / 4) + (r % 4);
            if (!((km >> c) & 1ull)) sacc[hf][r] = -INFINITY;
          }
      } else {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = 32 * hf + 8 * (r / 4) + (r % 4);
            if (c > lim) sacc[hf][r] = -INFINITY;
          }
      }
    }
    // ---- online softmax (log2 domain) -----------------------------------------------------------
    // a wave in its matrix phases (from here on: P V, the wait for the next tile, K Q^T) is issued ahead of
    // the other wave of the SIMD while that one does softmax arithmetic: measured 1-2 % on the tile loop
    __builtin_amdgcn_s_setprio(0);
    float tmax = -INFINITY;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sacc[hf][r]);
    tmax = max_pair(tmax);
    const float m_new = fmaxf(m_run, tmax * p.c);
    // The reference maximum moves only when some row's maximum grew by more than 2^8: until
    // then probabilities may exceed 1 (by at most 256x), which fp32 sums and bf16 P hold easily,
    // and the 64 accumulator registers are not rescaled.
    if (__any(m_new - m_run > 8.f)) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
      m_run = m_new;
      lacc[0] *= alpha;
      lacc[1] *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    }
    const float m_ref = (m_run == -INFINITY) ? 0.f : m_run;
    // Probabilities of key step g (8 of this lane's 32 entries, the B operand of that step's four
    // MFMAs), one pair at a time: exp2 of the pair j of step g, and its conversion to packed bf16.
    auto soft2 = [&](int g, int j) {
#pragma unroll
      for (int e = 2 * j; e < 2 * j + 2; ++e)
        sacc[g >> 1][8 * (g & 1) + e] =
            __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[g >> 1][8 * (g & 1) + e], p.c, -m_ref));
    };
    u32x4 pbuf[2];  // packed bf16 pairs of two consecutive steps
    auto cvt2 = [&](int g, int j) {
      const bf16x2 pr = {(__bf16)sacc[g >> 1][8 * (g & 1) + 2 * j], (__bf16)sacc[g >> 1][8 * (g & 1) + 2 * j + 1]};
      pbuf[g & 1][j] = __builtin_bit_cast(uint32_t, pr);
    };
    // The normaliser sums the probabilities as the matrix pipe sees them, rounded to bf16: the weights
    // p~ / sum p~ then add up to one exactly and a row's output stays a convex combination of its V
    // rows whatever the rounding of the individual p (with an fp32 sum of the unrounded p, a row with
    // a handful of kept keys shows the rounding of its dominant weight at full size).
    // v_mfma_f32_4x4x4_16b_bf16 with an all-ones A operand leaves, in every output register of a
    // lane, the sum of the four bf16 values the lane passed as B: two of them per key step
    // (2 passes each) replace eight additions on the vector ALU.
    const s16x4 ones4 = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
    // ---- O^T += V^T P^T : k-slot (gg,e) of step (hf,u) <-> key 32hf + 16u + 8(e/4) + 4gg + e%4 ----
    const uint16_t *Vt = Vs[grp][cur];
    {
      // 16 V^T fragments (4 key steps x 4 d blocks), each two transposing reads; same ring of four
      s16x4 vlo[4], vhi[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) soft2(0, j);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        vlo[i] = SA_VTR(Vt, i & 3, 16 * (i >> 2));
        vhi[i] = SA_VTR(Vt, i & 3, 16 * (i >> 2) + 8);
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) cvt2(0, j);
      __builtin_amdgcn_s_setprio(1);
      // One slot per MFMA, in program order and fenced: the product, the two LDS reads that refill
      // its V fragment, a quarter of the next step's exponentials and the conversion of the quarter
      // before.  Vector-ALU and matrix instructions of one wave overlap only when they alternate
      // in its instruction stream.
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int g = i >> 2, db = i & 3;  // key step g = 2*hf + u covers keys 16g .. 16g+15
        if (db == 0) {
          cvt2(g, 3);
          asm("" : "+v"(pbuf[g & 1]));  // opaque from here on: halves are sub-registers, not new conversions
        }
        const bf16x8 pb = __builtin_bit_cast(bf16x8, pbuf[g & 1]);
        const s16x8 av = __builtin_shufflevector(vlo[i & 3], vhi[i & 3], 0, 1, 2, 3, 4, 5, 6, 7);
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), pb, oacc[db], 0, 0, 0);
        {  // the step's row sums: low half in the first slot, high half in the last (placement swept: flat)
          const s16x8 ps = __builtin_bit_cast(s16x8, pb);
          if (db == 0)
            lacc[0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, __builtin_shufflevector(ps, ps, 0, 1, 2, 3), lacc[0], 0, 0, 0);
          if (db == 3)
            lacc[1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, __builtin_shufflevector(ps, ps, 4, 5, 6, 7), lacc[1], 0, 0, 0);
        }
        if (i + 4 < 16) {
          vlo[i & 3] = SA_VTR(Vt, (i + 4) & 3, 16 * ((i + 4) >> 2));
          vhi[i & 3] = SA_VTR(Vt, (i + 4) & 3, 16 * ((i + 4) >> 2) + 8);
        }
        if (g + 1 < 4) {
          soft2(g + 1, db);
          if (db > 0) cvt2(g + 1, db - 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  l_run = lacc[0][0] + lacc[1][0];

  // ---- selected diagonals: one 32-key tile per (wave, offset), no workgroup barriers -----------
  // For offset o the 32 queries of this wave need the 32 keys r0-o .. r0-o+31, row q for query q.  A lane holds half of
  // a key's row and of its query, which is what v_mfma_f32_4x4x4_16b takes of each of its 16 blocks: it multiplies four
  // neighbours with each other and three of four results are not used, where a product of 32x32x16 used one of 32 and the
  // diagonals were 17 % of the matrix work of a launch that runs at the card's power limit (layers of 128K tokens 4378
  // -> 4290 us, 64K 1595 -> 1556, 32K 684 -> 673, 16K 376 -> 372; of 8 heads at 4K this launch 19.5 -> 19.2, but the
  // layer 56.5 -> 56.8, since two others of it take longer).  K and V tiles are
  // copied by the LDS DMA into two wave-private 8 KB buffers in turn (swizzled like the shared tiles)
  // and read from there like any tile, the copies of one running while the one before is multiplied.
  // An entry is dropped when its key block is kept by the CSR or its key is a selected column: those
  // tiles already counted it.
  // The phase waits for its rows, and these for the path from the L2s to the fabric: copies of such tiles, two a wave in
  // flight as here, run at 35 TB/s out of an L2 and at 6.8 to 7.2 where they miss it, whatever the rows span beyond
  // 128 MiB.  Little of what a row block reads is in its XCD's L2 (nearby row blocks reach the same keys at
  // another offset and another time): an index of diagonals alone, 32 heads at 128K tokens, reads 35 GB of rows
  // in 3.38 ms, 22.4 GB of it past the L2s, which is 6.6 TB/s.  In a mix of heads the tile loops of other workgroups
  // run meanwhile: 14.7 GB cost 0.99 ms more than no diagonals, not the 2.1 they would take alone.
  // So the chain between two copies is kept short: which
  // queries take an entry is worked out for 64 offsets at once, one per lane, and the scores of a batch of offsets
  // are taken from K before their products with V, so that the row maximum is exchanged and compared once a
  // batch and either copy has a whole step of the other buffer to land.  Against K and V of one offset after the
  // other, the bitmaps read at each: 32 heads, 128K tokens 1025 -> 995 us of diagonals, 32K 98 -> 93, a layer of
  // 16K 430 -> 421, 4K 55.8 -> 54.9.
  __builtin_amdgcn_s_setprio(0);
  if (tid == 0 && grp == 0 && ticket < p.qcap) ticket = (int)atomicAdd(&p.queue[home], 1u);  // used at the next item
  if (has_offs) __syncthreads();  // all waves are done with the shared tiles and the list: reuse them
  if (has_offs && r0 < N) {
    const int32_t *__restrict__ offp = p.offs + (size_t)h * p.k_s;
    const int no = min(max(p.n_offs[h], 0), p.k_s);
    int dl = lane;
    asm volatile("" : "+v"(dl));  // this phase's lane constants are born here, not before the tile loop
    const int q = dl & 31, gg = dl >> 5, lane = dl;
    // two 8 KB tiles per wave: waves 0, 1 in the V buffers, waves 2, 3 in the K buffers
    uint16_t *const tile0 = (wv < 2 ? &Vs[grp][0][0] : &Ks[grp][0][0]) + (wv & 1) * (2 * 32 * 128);
    const unsigned ldsT = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)tile0;
    const int vrow = lane >> 4;                      // copies: one instruction moves rows 4n + vrow
    // rows are swizzled by (row & 15) = (4n & 15) ^ vrow, on the global side: four per-lane offsets serve the eight copies
    const unsigned kchunk = (unsigned)(((lane & 15) ^ vrow) << 4);
    // V (A operand of the 4x4 products, transposing read): the 16 lanes of a read supply four pieces of each of four blocks
    // of four keys, lane s the piece of key 4 (s % 4) + s / 4, and lane r receives keys 4 (r / 4) .. + 3 of element r % 4
    const int dvrow = (lane & 16) + 4 * (lane & 3) + ((lane >> 2) & 3);
    const unsigned dvbase = (unsigned)(dvrow * 256) | (unsigned)((dvrow & 15) << 4) | (unsigned)(8 * gg);
    const unsigned krow = (unsigned)(vrow * (int)p.kv_rs * 2);
    const uint32_t *kw = wv < 2 ? kept0 : kept1;
    float *const dsc = dscore[grp] + 32 * wv + q;
#define SA_DIAG_COPY(src, jb_, ldsb)                                                             \
  {                                                                                              \
    if ((jb_) >= 0) {                                                                            \
      const uint16_t *b_ = (src) + (size_t)(jb_) * p.kv_rs;                                      \
      _Pragma("unroll") for (int n_ = 0; n_ < 8; ++n_)                                           \
        SA_DMA16(b_ + (size_t)(4 * n_) * p.kv_rs, krow + (kchunk ^ (unsigned)(((4 * n_) & 15) << 4)), (ldsb) + n_ * 1024); \
    } else { /* rows before the sequence: clamped copies, masked out by the validity test */     \
      _Pragma("unroll") for (int n_ = 0; n_ < 8; ++n_) {                                         \
        const int rb_ = max((jb_) + 4 * n_, 0);                                                  \
        const int dr_ = max((jb_) + 4 * n_ + vrow, 0) - rb_; /* >= 0 */                          \
        SA_DMA16((src) + (size_t)rb_ * p.kv_rs,                                                  \
                 (unsigned)(dr_ * (int)p.kv_rs * 2) + (kchunk ^ (unsigned)(((4 * n_) & 15) << 4)), (ldsb) + n_ * 1024); \
      }                                                                                          \
    }                                                                                            \
  }
    for (int base = 0; base < no; base += 64) {
      // One offset per lane: which of the wave's queries (bit q) take its entry.  Offsets are ascending:
      // the usable ones (0 <= o <= last row of the wave) come first.
      const int ov = base + lane < no ? offp[base + lane] : -1;
      const unsigned long long bad = ~__ballot(ov >= 0 && ov <= r0 + 31);
      const int run = bad ? __ffsll(bad) - 1 : 64;
      uint32_t take = 0u;
      if (lane < run) {
        const int jb = r0 - ov;
        const int kta = max(jb, 0) >> 6, ktb = (jb + 31) >> 6;  // the (at most two) key tiles touched
        const int cut = 64 * (kta + 1) - jb;                    // queries below it take a key of the first
        const uint32_t first = cut >= 32 ? ~0u : (1u << cut) - 1u;
        take = jb >= 0 ? ~0u : ~0u << -jb;
        if ((kw[kta >> 5] >> (kta & 31)) & 1u) take &= ~first;
        if ((kw[ktb >> 5] >> (ktb & 31)) & 1u) take &= kta == ktb ? 0u : first;
        if (has_cols) {
          const int wi = jb >> 5;
          const uint32_t lo = wi >= 0 ? colbm[wi] : 0u, hi = (jb & 31) ? colbm[wi + 1] : 0u;
          take &= ~(uint32_t)(((uint64_t)lo | ((uint64_t)hi << 32)) >> (jb & 31));
        }
      }
      // An offset that no query takes is passed over.  The others in even batches; of the batch whose
      // copies are issued: its offsets (i_all), those still to be issued in this pass (i_left), which pass.
      unsigned long long rest = __ballot(take != 0u);
      if (G > 1) rest = __ballot(((rest >> lane) & 1ull) && __popcll(rest & ((1ull << lane) - 1ull)) % G == grp);
      const int n_live = __popcll(rest), n_batch = (n_live + kDiagBatch - 1) / kDiagBatch;
      const int per_batch = n_batch ? (n_live + n_batch - 1) / n_batch : 0;
      auto next_batch = [&]() {
        const bool mine = (rest >> lane) & 1ull;
        const unsigned long long b = __ballot(mine && __popcll(rest & ((1ull << lane) - 1ull)) < per_batch);
        rest &= ~b;
        return b;
      };
      unsigned long long i_all = next_batch(), i_left = i_all;
      bool i_v = false;
      int n_out = 0, ibuf = 0, cbuf = 0;  // tiles in flight; buffers of the next copy and of the next product
      auto issue = [&]() {
        if (i_left == 0ull) {
          if (!i_v) {
            i_v = true;
          } else {
            i_all = next_batch();
            i_v = false;
          }
          i_left = i_all;
          if (i_left == 0ull) return;
        }
        const int jb = r0 - __builtin_amdgcn_readlane(ov, __ffsll(i_left) - 1);
        i_left &= i_left - 1ull;
        const unsigned ldsb = ldsT + ibuf * (32 * 256);
        const uint16_t *const src = i_v ? Vh : Kh;
        SA_DIAG_COPY(src, jb, ldsb)
        ibuf ^= 1;
        ++n_out;
      };
      auto landed = [&]() {  // the oldest tile in flight has arrived
        if (n_out > 1) __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8)
        else __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
        asm volatile("" ::: "memory");
        --n_out;
      };
      if (i_all != 0ull) {
        issue();
        issue();
      }
      while (n_out > 0) {
        const unsigned long long batch = i_all;  // copies run two tiles ahead, never past the batch after this one
        float smax = -INFINITY;
        int slot = 0;
        for (unsigned long long left = batch; left != 0ull; left &= left - 1ull, ++slot) {
          const uint32_t tk = (uint32_t)__builtin_amdgcn_readlane((int)take, __ffsll(left) - 1);
          landed();
          const uint16_t *Kw = tile0 + cbuf * (32 * 128);
          bf16x8 kf[8];
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) kf[ks] = SA_KFRAG(Kw, 0, ks);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the tile is in registers: its buffer is free
          __builtin_amdgcn_sched_barrier(0);
          cbuf ^= 1;
          issue();
          // a lane's key row times its query and those of its three neighbours, 8 of 16 elements of a k-step per lane
          f32x4 sd[4] = {};
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) {
            const s16x8 k8 = __builtin_bit_cast(s16x8, kf[ks]), q8 = __builtin_bit_cast(s16x8, qf[ks]);
            sd[2 * (ks & 1)] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_shufflevector(k8, k8, 0, 1, 2, 3),
                                                          __builtin_shufflevector(q8, q8, 0, 1, 2, 3), sd[2 * (ks & 1)], 0, 0, 0);
            sd[2 * (ks & 1) + 1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_shufflevector(k8, k8, 4, 5, 6, 7),
                                                          __builtin_shufflevector(q8, q8, 4, 5, 6, 7), sd[2 * (ks & 1) + 1], 0, 0, 0);
          }
          float sv = (sd[0][0] + sd[2][0]) + (sd[1][0] + sd[3][0]);
#pragma unroll
          for (int r = 1; r < 4; ++r) sv = r == (q & 3) ? (sd[0][r] + sd[2][r]) + (sd[1][r] + sd[3][r]) : sv;
          sv = sum_pair(sv);
          smax = fmaxf(smax, (tk >> q) & 1u ? sv : -INFINITY);
          dsc[slot * BQ] = sv;  // as it is: a maximum would drop a NaN
          if constexpr (STATS) {
            st_kept += gg == 0 && ((tk >> q) & 1u) ? 1u : 0u;
            st_tiles += 1u;
          }
        }
        const float m_new = fmaxf(m_run, max_pair(smax) * p.c);
        if (__any(m_new - m_run > 8.f)) {
          const float alpha = __builtin_amdgcn_exp2f(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
          m_run = m_new;
          l_run *= alpha;
#pragma unroll
          for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
        }
        const float m_ref = (m_run == -INFINITY) ? 0.f : m_run;
        slot = 0;
        for (unsigned long long left = batch; left != 0ull; left &= left - 1ull, ++slot) {
          const uint32_t tk = (uint32_t)__builtin_amdgcn_readlane((int)take, __ffsll(left) - 1);
          const float sv = dsc[slot * BQ];
          const float pv = (tk >> q) & 1u ? __builtin_amdgcn_exp2f(__builtin_fmaf(sv, p.c, -m_ref)) : 0.f;
          const __bf16 pvb = (__bf16)pv;
          l_run += gg == 0 ? (float)pvb : 0.f;  // the weight as the matrix pipe sees it (see the tile loop's normaliser)
          const uint32_t pw = (uint32_t)__builtin_bit_cast(uint16_t, pvb) << (16 * (q & 1));
          const s16x4 pb = __builtin_bit_cast(s16x4, make_uint2(q & 2 ? 0u : pw, q & 2 ? pw : 0u));
          landed();
          const uint16_t *Vw = tile0 + cbuf * (32 * 128);
          s16x4 vf[16];
#pragma unroll
          for (int i = 0; i < 16; ++i)
            vf[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)((const char *)Vw + (dvbase ^ (unsigned)(i << 4))));
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
          cbuf ^= 1;
          issue();
          // P^T is diagonal: slot q % 4 of the block of four queries; elements 8 i + 4 gg .. + 3 are registers 4 (i % 4) .. + 3
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            f32x16 &o = oacc[i >> 2];
            const int r = 4 * (i & 3);
            const f32x4 s4 = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(vf[i], pb, f32x4{o[r], o[r + 1], o[r + 2], o[r + 3]}, 0, 0, 0);
            o[r] = s4[0];
            o[r + 1] = s4[1];
            o[r + 2] = s4[2];
            o[r + 3] = s4[3];
          }
        }
      }
    }
#undef SA_DIAG_COPY
  }

  if constexpr (STATS) {  // one pair of atomics per wave and item
    unsigned long long kept_n = st_kept;
    for (int d = 32; d >= 1; d >>= 1) kept_n += __shfl_xor(kept_n, d);
    if (lane == 0) {
      atomicAdd(&p.counters[0], (unsigned long long)st_tiles);
      atomicAdd(&p.counters[1], kept_n);
    }
  }
  // ---- epilogue: O[iq][32db + 8(r/4) + 4gg + r%4] = oacc / l -------------------------------------
  // A lane holds 16 separate 8-byte pieces of its row.  They go through an 8 KB LDS tile of the
  // wave's own (swizzled like a K tile) and leave as whole 256-byte rows, 16 bytes per lane: 64
  // cache lines per wave instead of 1024 partial writes.
  if constexpr (G == 2) {
    // The second group hands its sums to the first: 16 KB a wave through its own tiles.
    f32x4 *const xo = (f32x4 *)((wv < 2 ? &Vs[1][0][0] : &Ks[1][0][0]) + (wv & 1) * (64 * 128)) + lane;
    float *const xml = dscore[1] + tid;
    __syncthreads();
    if (grp == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        xo[64 * i] = f32x4{oacc[i >> 2][4 * (i & 3)], oacc[i >> 2][4 * (i & 3) + 1], oacc[i >> 2][4 * (i & 3) + 2], oacc[i >> 2][4 * (i & 3) + 3]};
      xml[0] = m_run;
      xml[256] = l_run;
    }
    __syncthreads();
    if (grp == 1) continue;
    const float m1 = xml[0], l1 = xml[256], m = fmaxf(m_run, m1), m_ref = m == -INFINITY ? 0.f : m;
    const float a0 = __builtin_amdgcn_exp2f(m_run - m_ref), a1 = __builtin_amdgcn_exp2f(m1 - m_ref);
    l_run = l_run * a0 + l1 * a1;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const f32x4 o = xo[64 * i];
#pragma unroll
      for (int e = 0; e < 4; ++e) oacc[i >> 2][4 * (i & 3) + e] = oacc[i >> 2][4 * (i & 3) + e] * a0 + o[e] * a1;
    }
  }
  const float ltot = l_run + __shfl_xor(l_run, 32);
  const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
  if (G == 1 && !has_offs) __syncthreads();  // the shared tiles are free (else such a barrier has been passed)
  {
    char *ow = (char *)((wv < 2 ? &Vs[0][0][0] : &Ks[0][0][0]) + (wv & 1) * (2 * 32 * 128));
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        union { __bf16 b[4]; uint2 u; } o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o.b[e] = (__bf16)(oacc[db][4 * rb + e] * inv);
        *(uint2 *)(ow + q * 256 + (((4 * db + rb) ^ (q & 15)) << 4) + 8 * gg) = o.u;
      }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int rr = lane >> 4, pc = lane & 15;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int r = 4 * n + rr;
      const uint4 v = *(const uint4 *)(ow + r * 256 + (pc << 4));
      if (r0 + r < N)
        *(uint4 *)(p.O + (size_t)h * p.o_hs + (size_t)(r0 + r) * p.o_rs + ((pc ^ (r & 15)) << 3)) = v;
    }
  }
  }  // work-queue loop
}

#undef SA_KFRAG
#undef SA_VTR
#undef SA_ISSUE_TILE
#undef SA_DMA16

// log2 of the queues that share a KV head, and from bit 4 on log2 of the row blocks a queue takes in a row
int queue_share(const Shape &sh) {
  const int nT = (sh.N + BQ - 1) / BQ;
  // KV heads in progress together: as many as there are queues, unless their K and V rows
  // (what the diagonal phase streams) exceed the 256 MiB memory-side cache.  32 heads at 128K tokens, a queue to itself
  // against two: a mix of heads 4.04 ms and 3.84, all Interval-Slash 3.73 and 3.66.  Not by fewer L2 misses (19.2 and 20.2
  // GB), nor by the rate of misses, which 128 MiB and 1 GiB of rows share; diagonals alone 3.30 and 3.39.  The cause is
  // not known.
  int xb = 0;
  while (xb < 3 && (8 >> xb) > sh.Hkv) ++xb;  // fewer than 8 KV heads: no idle queues
  while (xb < 3 && (size_t)(8 >> xb) * sh.N * kHeadDim * 2 * 2 > ((size_t)256 << 20)) ++xb;
  // sequences of a few runs per queue would not share out evenly
  return xb | (xb > 0 && nT >= (4 << xb) * kRun ? kRunBits << 4 : 0);
}

// Whether two groups of waves share an item.  A launch is at least as long as its longest item, whose tiles follow each
// other at 1.4 us with a compute unit to itself; with two groups, two tiles take 1.9.  Where the items
// are no more than the compute units, it is faster for every kind of head: layers of 4 to 8 heads at 1K to
// 4K tokens 19.7 -> 18.8 us, 28.9 -> 25.3, 45.2 -> 36.9, 56 -> 45 at 8K, slash heads only 22.9 -> 22.9 to 57 -> 47.
// With up to twice as many it depends on what the items hold, since two workgroups would share the unit anyway; the host
// knows the budgets.  Where the band of Triangular heads covers the sequence they gain (plain causal attention of 2K
// to 16K tokens 56 -> 50, 97 -> 81, 180 -> 141, 352 -> 263 us; at 2.25 items per unit 81 -> 90), and so do
// Block-Cluster heads that keep every block.  Interval-Slash heads gain if their items are long too, which asks for a
// quarter of the keys as columns, what sa_default_budgets gives for keep = 1: whole layers under the run-time rule, 8 heads
// at 5120 and 8192 tokens (slash, and seven slash heads of eight) 121 -> 98, 173 -> 152, 145 -> 120, 214 -> 188, 32 heads
// at 1280 and 2048 70.2 -> 71.6, 87.3 -> 86.7, 72.3 -> 73.3, 95.5 -> 95.0, 64 heads at 1024 71.5 -> 75.8 (all
// Block-Cluster 75 -> 69).  With few columns under such a band they lose (a tenth of the keys kept, 8 heads at 5120
// tokens 62 -> 69.5, 32 at 2048 60.8 -> 67, 24 at 2048 58 -> 64.5), so these stay whole, as do those without such a band
// (slash heads 34 -> 41, a mix 62 -> 46, which cannot be told apart here).  To ask the index on the device instead, with
// both kernels launched and one of them returning at once, cost 2 to 3 us a call.
// Heads taken with several indices (the offline search) stay whole: their results must not
// depend on how many heads are taken together.
bool split_items(const Shape &sh) {
  const int n_items = (sh.N + BQ - 1) / BQ * sh.Hq;
  // rounded to 64, a quarter of the keys can be half a tile short
  const bool long_items = sh.local >= sh.nb && 4 * ((long long)sh.k_v + BK / 2) >= sh.N;
  return sh.gq == sh.g && n_items <= (long_items ? 2 : 1) * sh.n_cu;
}

int queue_capacity(const Shape &sh) {
  const int share = queue_share(sh), slots = 8 >> (share & 15);
  return tickets_per_head((sh.N + BQ - 1) / BQ, share) * sh.g * ((sh.Hkv + slots - 1) / slots);
}

}  // namespace

size_t attn_item_bytes(const Shape &sh) { return (size_t)8 * queue_capacity(sh) * sizeof(uint4); }
size_t attn_tile_bytes(const Shape &sh) { return (size_t)sh.Hq * sh.cap_b * (sh.b / BK) * 2; }

hipError_t launch_sparse_prefill(const Shape &sh, const Workspace &ws, const uint16_t *Q,
                                 const uint16_t *K, const uint16_t *V, sa_index idx, uint16_t *O,
                                 unsigned long long *counters, hipStream_t st) {
  AttnArgs a = {};
  a.Q = Q; a.K = K; a.V = V; a.O = O;
  a.n_cols = idx.n_cols; a.cols = idx.cols; a.n_offs = idx.n_offs; a.offs = idx.offs;
  a.rowptr = idx.rowptr; a.blkcols = idx.blkcols;
  a.colbits = ws.colbits; a.colprefix = ws.colprefix;
  a.Hq = sh.Hq; a.Hkv = sh.Hkv; a.g = sh.g; a.gq = sh.gq; a.N = sh.N; a.b = sh.b; a.nb = sh.nb;
  a.nT = (sh.N + BQ - 1) / BQ;
  a.k_v = sh.k_v; a.k_s = sh.k_s; a.cap_b = sh.cap_b;
  a.q_hs = sh.q_hs; a.q_rs = sh.q_rs; a.kv_hs = sh.kv_hs; a.kv_rs = sh.kv_rs;
  a.o_hs = sh.o_hs; a.o_rs = sh.o_rs;
  a.c = sh.scale * 1.4426950408889634f;
  a.counters = counters;
  a.Kg = ws.kg; a.Vg = ws.vg; a.kvg_rows = (sh.k_v + BK - 1) / BK * BK;
  a.queue = ws.queue;
  a.n_items = a.nT * sh.Hq;
  a.share = queue_share(sh);
  a.qcap = queue_capacity(sh);
  a.side_by_side = a.n_items <= 8 * sh.n_cu;
  a.items = (uint4 *)ws.attn_items;
  a.tiles = ws.attn_tiles;
  a.tile_cap = (unsigned)sh.cap_b * (unsigned)(sh.b / BK);
  const bool split = split_items(sh);
  const int resident = (split ? 1 : 2) * sh.n_cu;  // workgroups
  a.grid = a.n_items < resident ? a.n_items : resident;
  const int n_plan = (8 * a.qcap + kPlanWaves - 1) / kPlanWaves;
  // LDS for the larger of a head's column bitmap and the key-tile bitmaps of four items: this bound also
  // limits the workgroups of a CU, so it follows the sequence
  const int tile_words = (sh.N / BK + 31) / 32 + 1;
  int words = 2 * kPlanWaves * tile_words;
  if (words < sh.N / 32) words = (sh.N / 32 + 2 * kPlanWaves - 1) / (2 * kPlanWaves) * (2 * kPlanWaves);
  index_prepare_kernel<<<sh.Hq + n_plan + a.kvg_rows / BK * sh.Hq, 256, words * 4, st>>>(a, ws.queue, words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int grid = a.grid;
  if (counters && split)
    sparse_prefill_kernel<true, 2><<<grid, 512, 0, st>>>(a);
  else if (counters)
    sparse_prefill_kernel<true, 1><<<grid, 256, 0, st>>>(a);
  else if (split)
    sparse_prefill_kernel<false, 2><<<grid, 512, 0, st>>>(a);
  else
    sparse_prefill_kernel<false, 1><<<grid, 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace sa
