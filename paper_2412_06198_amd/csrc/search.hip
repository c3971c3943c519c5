// Offline pattern search (Kernel-Aware Sparse Pattern Search Algorithm, Alg. 1):
//   Initialize Search Space - each candidate pattern has one integer size (Triangular: band
//     blocks; Interval-Slash: diagonals, with 32 columns per diagonal; Block-Cluster: blocks);
//     RefineSearchSpace is a bisection on it until the kept (query, key) pairs - FLOPs / (4 d) -
//     meet the target within the tolerance, or the two sizes around the target are adjacent;
//   Evaluate Patterns - the head's dense causal output against the sparse output of every
//     refined candidate, Frobenius norm of the difference, smallest wins (ties: lowest id).
// All heads of a batch go through every step together, with budgets of their own each, and the host
// waits once per batch.  A head is taken with several indices at a time: index and attention launches see
// kSets times as many heads as the batch has (Shape::gq), so that the dense reference and the three candidates are
// one index build and one attention launch.  The pairs of a Triangular or Block-Cluster candidate follow from
// its number of blocks alone; those of an Interval-Slash candidate are counted from the selected columns and
// offsets, and no attention runs before the sizes are known.  A head of a short sequence goes through its whole refinement
// in one workgroup (slash_refine_kernel).  Of a longer one a step evaluates three sizes with an index build, the one
// that the bisection asks for and the two it can ask for next, and slash_step_kernel counts their pairs and
// takes the head's next steps.
// (With one head at a time, an attention call per probe to count its pairs and a wait after each, 8 heads of 4096
// tokens took 35 ms; with one index at a time, 13 index builds and four attention launches as long as their longest
// row block each, 661 us; with index builds for every step of the refinement 333, now 273.)
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>

#include "sa_internal.h"

namespace {

constexpr int kNormBlocks = 1024;
constexpr int kSets = 4;    // indices of a head in the last launches: dense, then the candidates
constexpr int kProbes = 3;  // indices of a head in a refinement step
constexpr size_t kBatchBytes = (size_t)2 << 30;  // scratch that a batch of heads may take (one head always may)

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Virtual head of index `set` of head i, gb heads per KV head: a KV head's heads with their first index, with their
// second, ...
__host__ __device__ inline int virtual_head(int i, int set, int gb, int sets) { return (i / gb * sets + set) * gb + i % gb; }

// partial[set - 1][head][block] = sum over the block's rows of (output with index set - output with index 0)^2,
// O [virtual heads][N][128] bf16; fp64 accumulation, fixed order: bit-reproducible.
// grid (blocks, heads, kSets - 1)
__global__ __launch_bounds__(256) void sq_diff_kernel(const uint16_t *__restrict__ O, int gb, int N,
                                                      double *__restrict__ partial) {
  const size_t hs = (size_t)N * sa::kHeadDim;
  __shared__ double red[256];
  const int cc = threadIdx.x & 15, rg = threadIdx.x >> 4;
  const uint16_t *A = O + (size_t)virtual_head(blockIdx.y, blockIdx.z + 1, gb, kSets) * hs;
  const uint16_t *B = O + (size_t)virtual_head(blockIdx.y, 0, gb, kSets) * hs;
  double acc = 0.0;
  // the rows of a block: kNormBlocks blocks' worth apart, whatever the grid (the sums of the blocks that
  // a short sequence leaves without rows are zero)
  for (int64_t i = (int64_t)blockIdx.x * 16 + rg; i < N; i += (int64_t)kNormBlocks * 16) {
    const size_t o = (size_t)i * sa::kHeadDim + cc * 8;
    const uint4 a = *(const uint4 *)(A + o), b = *(const uint4 *)(B + o);
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float d0 = __uint_as_float(aw[e] << 16) - __uint_as_float(bw[e] << 16);
      const float d1 = __uint_as_float(aw[e] & 0xFFFF0000u) - __uint_as_float(bw[e] & 0xFFFF0000u);
      acc += (double)d0 * (double)d0 + (double)d1 * (double)d1;
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = red[0];
}

// RefineSearchSpace of one candidate, a step per evaluated size: the smallest size, the largest, then
// bisection between sizes whose pairs lie on either side of the target.
struct Refine {
  int64_t lo, hi, p_lo, p_hi;  // sizes around the target and their pairs
  int64_t x, px;               // size to evaluate next, or (done) the answer and its pairs
  int32_t stage, done;
  uint32_t arrived, unused;    // probes of this step whose pairs are counted
  int64_t pairs[kProbes];
  __host__ __device__ void start(int64_t x_lo, int64_t x_hi) {
    lo = x = x_lo; hi = x_hi;
    p_lo = p_hi = px = 0;
    stage = done = 0;
    arrived = unused = 0;
    for (int i = 0; i < kProbes; ++i) pairs[i] = 0;
  }
  // Sizes of a step's probes: x, and what can follow it (x again where nothing can).
  __host__ __device__ int64_t probe(int i) const {
    if (i == 0 || done) return x;
    if (stage == 0) return i == 1 ? hi : hi - lo > 1 ? (lo + hi) / 2 : x;
    const int64_t l = i == 1 ? lo : x, h = i == 1 ? x : hi;
    return h - l > 1 ? (l + h) / 2 : x;
  }
  __host__ __device__ void step(int64_t pairs, int64_t target, int64_t eps) {
    if (done) return;
    const int64_t off = pairs < target ? target - pairs : pairs - target;
    const bool hit = off <= eps;
    px = pairs;
    if (stage == 0) {
      p_lo = pairs;
      if (pairs >= target || hit || lo == hi) { done = 1; return; }
      x = hi;
      stage = 1;
      return;
    }
    if (stage == 1) {
      p_hi = pairs;
      if (pairs <= target || hit) { done = 1; return; }
      stage = 2;
    } else {
      if (hit) { done = 1; return; }
      if (pairs < target) { lo = x; p_lo = pairs; } else { hi = x; p_hi = pairs; }
    }
    if (hi - lo > 1) { x = (lo + hi) / 2; return; }
    done = 1;  // adjacent sizes: the closer one, the smaller on a tie
    if (target - p_lo <= p_hi - target) { x = lo; px = p_lo; } else { x = hi; px = p_hi; }
  }
};

__host__ __device__ inline sa::HeadBudget slash_budget(int64_t x, int N, int nb) {
  sa::HeadBudget b;
  b.k_s = (int32_t)x;
  b.k_v = (int32_t)(32 * x < N ? 32 * x : N);
  b.k_b = nb;
  b.local = 1;
  return b;
}

// Sizes of a head's indices in the last launches, those known beforehand: the smallest Interval-Slash size, the refined
// Triangular and Block-Cluster sizes.
struct Sizes { int64_t slash, triangular, cluster; };

// Budget of index `set` (0: dense, then the candidates) of a head.
__host__ __device__ inline sa::HeadBudget set_budget(int set, const Sizes &x, int N, int nb) {
  sa::HeadBudget b = slash_budget(x.slash, N, nb);
  if (set == 0) b.local = nb;
  if (set == 1 + SA_TRIANGULAR) b.local = (int32_t)x.triangular;
  if (set == 1 + SA_BLOCK_CLUSTER) b.k_b = (int32_t)x.cluster;
  return b;
}

// One workgroup per virtual head of a refinement step: the kept pairs of its Interval-Slash index (its diagonal blocks,
// the selected columns, the selected diagonals; each pair once).  The workgroup that counts a head's last
// probe takes the steps of its bisection that the probes answer.
//   diagonal blocks: nb b (b + 1) / 2
//   column c: the queries behind its key block
//   offset o: the pairs (i, i - o) in different blocks, less those whose key is a selected column,
//     i.e. the columns c < N - o with c % b >= b - o
constexpr int kStepThreads = 512, kStepCols = 8192;  // columns that are searched in LDS

__global__ __launch_bounds__(kStepThreads) void slash_step_kernel(const int32_t *cols, const int32_t *offs, int k_v, int k_s,
                                                                  int N, int b, int gb, Refine *state, sa::HeadBudget *probes,
                                                                  sa::HeadBudget *last, int64_t target, int64_t eps) {
  __shared__ int by_pos[128];            // columns outside the last key block by their position in the block
  __shared__ int from[129];              // ... at position p or behind
  __shared__ long long red[kStepThreads / 64];
  __shared__ int32_t c_lds[kStepCols];
  const int i0 = blockIdx.x, pr = blockIdx.y, h = virtual_head(i0, pr, gb, kProbes), tid = threadIdx.x, nb = N / b;
  Refine *st = state + i0;
  if (st->done) return;
  const int nc = min(probes[h].k_v, N), no = min(probes[h].k_s, N);
  const int32_t *c = cols + (size_t)h * k_v, *o = offs + (size_t)h * k_s;
  const bool in_lds = nc <= kStepCols;
  if (tid < b) by_pos[tid] = 0;
  __syncthreads();
  long long sum = 0;
  for (int i = tid; i < nc; i += kStepThreads) {
    const int key = c[i], blk = key / b;
    if (in_lds) c_lds[i] = key;
    sum += N - (blk + 1) * b;
    if (blk < nb - 1) atomicAdd(&by_pos[key - blk * b], 1);
  }
  __syncthreads();
  if (tid < 64) {  // b is 64 or 128: a wave sums from the end, b / 64 positions per lane
    const int per = b >> 6, p0 = b - per * (tid + 1);
    const int x0 = by_pos[p0], x1 = per > 1 ? by_pos[p0 + 1] : 0;
    int incl = x0 + x1;
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(incl, d);
      if (tid >= d) incl += y;
    }
    from[p0] = incl;
    if (per > 1) from[p0 + 1] = incl - x0;
    if (tid == 0) from[b] = 0;
  }
  __syncthreads();
  for (int i = tid; i < no; i += kStepThreads) {
    const int off = o[i];
    if (off >= b) {
      int lo = 0, hi = nc;  // the first column that is not below N - off
      while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if ((in_lds ? c_lds[m] : c[m]) < N - off) lo = m + 1;
        else hi = m;
      }
      sum += N - off - lo;
    } else {
      sum += (long long)(N - off) - (long long)nb * (b - off) - from[b - off];
    }
  }
  for (int d = 32; d >= 1; d >>= 1) sum += __shfl_down(sum, d);
  if ((tid & 63) == 0) red[tid >> 6] = sum;
  __syncthreads();
  if (tid != 0) return;
  for (int i = 1; i < kStepThreads / 64; ++i) sum += red[i];
  // Agent-scope accesses, the pairs performed (vmcnt(0)) before the arrival is counted: the last one reads them all.
  __hip_atomic_store(&st->pairs[pr], (int64_t)(sum + (long long)nb * b * (b + 1) / 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::: "memory");
  if (atomicAdd(&st->arrived, 1u) != kProbes - 1) return;
  Refine r = *st;
  int64_t size[kProbes], pairs[kProbes];
#pragma unroll
  for (int i = 0; i < kProbes; ++i) {
    size[i] = r.probe(i);
    pairs[i] = __hip_atomic_load(&st->pairs[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (bool known = true; known && !r.done;) {
    known = false;
    for (int i = 0; i < kProbes && !known; ++i)
      if (size[i] == r.x) { r.step(pairs[i], target, eps); known = true; }
  }
  r.arrived = 0;
  *st = r;
#pragma unroll
  for (int i = 0; i < kProbes; ++i) probes[virtual_head(i0, i, gb, kProbes)] = slash_budget(r.probe(i), N, nb);
  last[virtual_head(i0, 1 + SA_INTERVAL_SLASH, gb, kSets)] = slash_budget(r.x, N, nb);
}

// RefineSearchSpace of the Interval-Slash candidate of short sequences, a workgroup per head.  The selections of all
// sizes are prefixes of one ranking, so columns and offsets are ranked once and a size is evaluated from the ranks: its
// columns as a bitmap, with the counts before each word, answer how many of them lie below N - o.
// The ranking is a bitonic sort in LDS, by half of the waves for each array, four strides a pass in registers
// (one at a time it is bound by LDS).  A key is a score and its index in the mantissa of a double
// between 1 and 2, so that a comparison is v_max_f64 and v_min_f64, and a change of sign turns the order.
// What bounds it is one compute unit: 28 us of 45 at 4096 are the sorts, 1.9 each evaluation.  Four steps of
// an index build and a count each took 108 (a whole search of 1, 4, 8 and 24 heads of 4096 tokens 249, 289, 333
// and 515 us, now 190, 224, 273 and 447; 8 heads of 8192 tokens 629 and 556, of 1024 172 and 130).  As far as both
// arrays fit LDS; beyond, the attention is what a search waits for.
constexpr int kRankThreads = 1024, kRankHalf = kRankThreads / 2, kRankMaxSeq = 8192;
constexpr unsigned long long kRankOne = 0x3FF0000000000000ull, kRankSign = 1ull << 63;
__device__ inline unsigned long long rank_key(uint32_t score, int i) {
  return kRankOne | (unsigned long long)score << 13 | (unsigned)(kRankMaxSeq - 1 - i);
}
__device__ inline int rank_index(unsigned long long key) { return kRankMaxSeq - 1 - (int)(key & (kRankMaxSeq - 1)); }

// Where key i of a sort sits: keys 8, 64 or 1 apart, which the lanes of a wave take, spread over the banks.
__device__ inline int rank_slot(int i) { return i ^ (i >> 3 & 31); }

__device__ __forceinline__ void rank_pair(double &larger, double &smaller) {
  double hi, lo;
  asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(larger), "v"(smaller));
  asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(larger), "v"(smaller));
  larger = hi;
  smaller = lo;
}

// S strides of a bitonic merge of k keys, j and below, largest first: 2^S keys per thread and chunk.  FIRST: all merges
// of up to 2^S neighbours.
template <int S, bool FIRST = false>
__device__ __forceinline__ void rank_pass(unsigned long long *key, int P, int k, int j, int ht) {
  const int jl = j >> (S - 1);
  __syncthreads();
  for (int t = ht; t < P >> S; t += kRankHalf) {
    const int at = (t & ~(jl - 1)) << S | (t & (jl - 1));
    const unsigned long long turn = (at & k) ? kRankSign : 0ull;
    double e[1 << S];
    int slot[1 << S];
#pragma unroll
    for (int i = 0; i < 1 << S; ++i) slot[i] = rank_slot(at + i * jl);
#pragma unroll
    for (int i = 0; i < 1 << S; ++i) e[i] = __longlong_as_double((long long)(key[slot[i]] ^ turn));
    if (FIRST) {
#pragma unroll
      for (int m = 1; m < S; ++m)
#pragma unroll
        for (int s = m - 1; s >= 0; --s)
#pragma unroll
          for (int i = 0; i < 1 << S; ++i)
            if (!((i >> s) & 1)) {
              if ((i >> m) & 1) rank_pair(e[i | 1 << s], e[i]);
              else rank_pair(e[i], e[i | 1 << s]);
            }
    }
#pragma unroll
    for (int s = S - 1; s >= 0; --s)
#pragma unroll
      for (int i = 0; i < 1 << S; ++i)
        if (!((i >> s) & 1)) rank_pair(e[i], e[i | 1 << s]);
#pragma unroll
    for (int i = 0; i < 1 << S; ++i) key[slot[i]] = (unsigned long long)__double_as_longlong(e[i]) ^ turn;
  }
}

__global__ __launch_bounds__(kRankThreads) void slash_refine_kernel(const uint32_t *v, const uint32_t *s, int N, int b, int gb,
                                                                    Sizes known, int64_t x_hi, Refine *state, sa::HeadBudget *last,
                                                                    int64_t target, int64_t eps) {
  typedef unsigned long long u64;
  __shared__ u64 key[2][kRankMaxSeq];
  __shared__ uint16_t group[kRankMaxSeq];         // a column's rank / 32
  __shared__ uint16_t offset[kRankMaxSeq / 32];   // offsets by rank
  __shared__ u64 word[kRankMaxSeq / 64];          // the columns of a size ...
  __shared__ int before[kRankMaxSeq / 64];        // ... and how many lie before each word
  __shared__ int by_pos[2][128], from[129];       // as in slash_step_kernel, of this size and of the next
  __shared__ long long red[2][kRankThreads / 64];
  const int i0 = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = N / b, bl = b == 64 ? 6 : 7, half = tid / kRankHalf, ht = tid % kRankHalf;
  int P = 64;
  while (P < N) P *= 2;
  const uint32_t *src = (half ? s : v) + (size_t)i0 * N;
  for (int i = ht; i < P; i += kRankHalf) key[half][rank_slot(i)] = i < N ? rank_key(src[i], i) : kRankOne;  // fillers last
  rank_pass<4, true>(key[half], P, 16, 8, ht);
  for (int k = 32; k <= P; k *= 2) {
    int j = k / 2;
    const int steps = 31 - __clz(k);
    if (steps % 4 == 1) { rank_pass<1>(key[half], P, k, j, ht); j >>= 1; }
    if (steps % 4 == 2) { rank_pass<2>(key[half], P, k, j, ht); j >>= 2; }
    if (steps % 4 == 3) { rank_pass<3>(key[half], P, k, j, ht); j >>= 3; }
    for (; j > 0; j >>= 4) rank_pass<4>(key[half], P, k, j, ht);
  }
  __syncthreads();
  for (int i = tid; i < N; i += kRankThreads) group[rank_index(key[0][rank_slot(i)])] = (uint16_t)(i >> 5);
  for (int i = tid; i < N / 32; i += kRankThreads) offset[i] = (uint16_t)rank_index(key[1][rank_slot(i)]);

  Refine r;
  r.start(known.slash, x_hi);
  if (tid < 256) by_pos[tid >> 7][tid & 127] = 0;
  __syncthreads();
  for (int cur = 0; !r.done; cur ^= 1) {
    const int x = (int)r.x;  // so many offsets, and the columns of the first x groups
    long long sum = 0;
    for (int c = tid; c < N; c += kRankThreads) {  // whole waves: N is a multiple of 64
      const bool in = (int)group[c] < x;
      const u64 m = __ballot(in);
      if (lane == 0) word[c >> 6] = m;
      if (in) {
        const int blk = c >> bl;
        sum += N - ((blk + 1) << bl);
        if (blk < nb - 1) atomicAdd(&by_pos[cur][c - (blk << bl)], 1);
      }
    }
    __syncthreads();
    if (wv == 0) {  // two words per lane
      const int w = 2 * lane, nw = N >> 6;
      const int n0 = w < nw ? __popcll(word[w]) : 0, n1 = w + 1 < nw ? __popcll(word[w + 1]) : 0;
      const int incl = (int)sa::wave_inclusive_sum((unsigned)(n0 + n1));
      if (w < nw) before[w] = incl - n0 - n1;
      if (w + 1 < nw) before[w + 1] = incl - n1;
    } else if (wv == 1) {  // sums from the end, b / 64 positions per lane
      const int per = b >> 6, p0 = b - per * (lane + 1);
      const int n0 = by_pos[cur][p0], n1 = per > 1 ? by_pos[cur][p0 + 1] : 0;
      const int incl = (int)sa::wave_inclusive_sum((unsigned)(n0 + n1));
      from[p0] = incl;
      if (per > 1) from[p0 + 1] = incl - n0;
      if (lane == 0) from[b] = 0;
    } else if (wv < 4) {
      by_pos[cur ^ 1][64 * (wv - 2) + lane] = 0;
    }
    __syncthreads();
    if (tid < x) {
      const int off = offset[tid], m = N - off;  // its keys lie below m
      if (off >= b) sum += m - before[m >> 6] - __popcll(word[m >> 6] & ((1ull << (m & 63)) - 1ull));
      else sum += (long long)m - (long long)nb * (b - off) - from[b - off];
    }
    sum = (long long)sa::wave_sum63((u64)sum);
    if (lane == 63) red[cur][wv] = sum;
    __syncthreads();
    long long pairs = (long long)nb * b * (b + 1) / 2;
#pragma unroll
    for (int i = 0; i < kRankThreads / 64; ++i) pairs += red[cur][i];
    r.step(pairs, target, eps);  // every thread the same
  }
  // The budgets of all of the head's indices, from here: a copy from the host's pageable memory before this launch held the
  // host for its staging (8 heads of 4096 tokens 273 us a search with it, 243 without, 4 of 2048 153 and 128, 8 of 1024
  // 131 and 110).
  if (tid < kSets) last[virtual_head(i0, tid, gb, kSets)] = tid == 1 + SA_INTERVAL_SLASH ? slash_budget(r.x, N, nb) : set_budget(tid, known, N, nb);
  if (tid == 0) state[i0] = r;
}

// Heads that go through the search together, and the scratch they take.
struct Batch {
  int heads, kv_heads;  // query heads (whole KV groups, or a part of one), their KV heads
  sa_config cfg;        // of the virtual heads: budgets as large as any candidate's
  int64_t x_lo[3], x_hi[3];
  size_t off[11], total;
};

sa_status plan_batch(const sa_ctx *ctx, int heads, Batch *z) {
  const sa_config &p = ctx->cfg;
  const int N = p.seq_len, nb = N / p.block, g = ctx->sh.g;
  z->heads = heads;
  z->kv_heads = heads > g ? heads / g : 1;
  z->x_lo[0] = 1; z->x_hi[0] = nb;
  z->x_lo[1] = 1; z->x_hi[1] = N / 32 > 1 ? N / 32 : 1;
  z->x_lo[2] = nb; z->x_hi[2] = (int64_t)nb * (nb + 1) / 2;
  if (z->x_hi[2] > 0x7FFFFFFFll) return SA_ERR_UNSUPPORTED;
  sa_config &c = z->cfg;
  c = p;
  c.n_q_heads = kSets * heads; c.n_kv_heads = z->kv_heads;
  const sa::HeadBudget most = slash_budget(z->x_hi[1], N, nb);
  c.k_vertical = most.k_v; c.k_slash = most.k_s;
  c.local_blocks = nb; c.k_blocks = (int32_t)z->x_hi[2];
  c.block_select = SA_BLOCKS_GLOBAL;        // the search's Block-Cluster candidate is the one-top-k rule,
  c.diagonal_select = SA_DIAGONALS_EXACT;   // its Interval-Slash candidate the element-exact one
  c.lazy_block_map = 0;
  if (!c.q_head_stride) c.q_head_stride = ctx->sh.q_hs;
  if (!c.kv_head_stride) c.kv_head_stride = ctx->sh.kv_hs;
  sa_ctx *child = nullptr;
  sa_status st = sa_create(&c, &child);
  if (st != SA_OK) return st;
  size_t ws = 0, ix[7];
  st = sa_workspace_bytes(child, &ws);
  if (st == SA_OK) st = sa_index_bytes(child, ix);
  sa_destroy(child);
  if (st != SA_OK) return st;
  const size_t o_bytes = (size_t)kSets * heads * N * sa::kHeadDim * 2;
  const size_t parts[11] = {ws, o_bytes, (size_t)heads * (kSets + kProbes) * sizeof(sa::HeadBudget),
                            (size_t)heads * (sizeof(Refine) + 3 * kNormBlocks * 8), ix[0], ix[1], ix[2], ix[3], ix[4], ix[5], ix[6]};
  size_t o = 0;
  for (int i = 0; i < 11; ++i) { z->off[i] = o; o += align256(parts[i]); }
  z->total = o;
  return SA_OK;
}

// The batches of a search: all of one size, but the last one (of every group, where they are parts of one).
struct Plan {
  Batch full, last;  // last.heads = 0: every batch is full
  int period;        // heads that are shared out: all, or a KV group's
  size_t total;
  int heads_from(int h0) const { return period - h0 % period < full.heads ? last.heads : full.heads; }
};

sa_status plan_batches(const sa_ctx *ctx, int heads, int period, Plan *z) {
  z->period = period;
  z->last.heads = 0;
  sa_status st = plan_batch(ctx, heads, &z->full);
  if (st == SA_OK && period % heads) st = plan_batch(ctx, period % heads, &z->last);
  z->total = z->last.heads && z->last.total > z->full.total ? z->last.total : z->full.total;
  return st;
}

// As few batches as the head limit and kBatchBytes allow, of equal sizes as far as that goes: of whole KV groups, else of
// parts of one.  Equal parts alone are not enough: 37 heads on one KV head, a prime number above the 32 that four
// indices each leave, would go head by head with a wait of the host after each (at 192, 1024 and 4096
// tokens 3215, 3965 and 7072 us, in two batches 238, 339 and 909; 39 heads on 13 KV heads at 2048 tokens 1810 and 442).
sa_status plan(const sa_ctx *ctx, Plan *z) {
  const int g = ctx->sh.g, Hkv = ctx->sh.Hkv;
  sa_status st = SA_OK;
  for (int n = 1; n <= Hkv; ++n) {
    const int kv = (Hkv + n - 1) / n;
    if ((n > 1 && kv == (Hkv + n - 2) / (n - 1)) || kSets * kv * g > sa::kMaxHeads) continue;
    if ((st = plan_batches(ctx, kv * g, Hkv * g, z)) != SA_OK) return st;
    if (z->total <= kBatchBytes) return SA_OK;
  }
  for (int n = 2; n <= g; ++n) {
    const int heads = (g + n - 1) / n;
    if (heads == (g + n - 2) / (n - 1) || kSets * heads > sa::kMaxHeads) continue;
    if ((st = plan_batches(ctx, heads, g, z)) != SA_OK) return st;
    if (z->total <= kBatchBytes) return SA_OK;
  }
  return SA_OK;  // one head at a time
}

// Where a batch's buffers lie in the scratch, and its shapes.
struct Layout {
  sa::Shape cs, ps;  // of the dense reference and the candidates; of a refinement step
  sa::Workspace ws;
  uint16_t *outputs;
  sa::HeadBudget *budgets, *probes;  // of the virtual heads: dense and candidates, probes
  Refine *state;                     // and the sums behind it: the results
  double *partial;
  sa_index ix;
};

sa_status lay_out(const Batch &z, char *base, Layout *l) {
  const int B = z.heads, gb = B / z.kv_heads;
  l->outputs = (uint16_t *)(base + z.off[1]);
  l->budgets = (sa::HeadBudget *)(base + z.off[2]);
  l->probes = l->budgets + (size_t)kSets * B;
  l->state = (Refine *)(base + z.off[3]);
  l->partial = (double *)(l->state + B);
  int32_t **part[7] = {&l->ix.pattern, &l->ix.n_cols, &l->ix.cols, &l->ix.n_offs, &l->ix.offs, &l->ix.rowptr, &l->ix.blkcols};
  for (int i = 0; i < 7; ++i) *part[i] = (int32_t *)(base + z.off[4 + i]);
  sa_ctx *child = nullptr;
  sa_status st = sa_create(&z.cfg, &child);
  if (st != SA_OK) return st;
  st = sa_set_workspace(child, base + z.off[0], child->ws_bytes);
  l->cs = child->sh;
  l->cs.gq = gb;
  l->cs.o_rs = sa::kHeadDim;
  l->cs.o_hs = (int64_t)l->cs.N * sa::kHeadDim;
  l->ps = l->cs;
  l->ps.Hq = kProbes * B; l->ps.g = kProbes * gb;
  l->ws = child->ws;
  sa_destroy(child);
  return st;
}

sa_status failp(sa_ctx *c, sa_status st, const char *msg) {
  snprintf(c->err, sizeof(c->err), "%s", msg);
  return st;
}

}  // namespace

extern "C" {

sa_status sa_search_scratch_bytes(const sa_ctx *ctx, size_t *bytes) {
  if (!ctx || !bytes) return SA_ERR_INVALID_ARG;
  Plan z;
  const sa_status st = plan(ctx, &z);
  if (st == SA_OK) *bytes = z.total;
  return st;
}

sa_status sa_search_patterns(sa_ctx *ctx, const void *Q, const void *K, const void *V, sa_scores scores,
                             int64_t target_pairs, int64_t eps_pairs, void *scratch, size_t scratch_bytes,
                             sa_search_head *out_host, void *hip_stream) {
  if (!ctx) return SA_ERR_INVALID_ARG;
  if (!Q || !K || !V || !scores.v || !scores.s || !scores.blk || !scratch || !out_host)
    return failp(ctx, SA_ERR_INVALID_ARG, "null pointer");
  if (target_pairs < 0 || eps_pairs < 0) return failp(ctx, SA_ERR_INVALID_ARG, "negative target or tolerance");
  if ((uintptr_t)scratch & 255) return failp(ctx, SA_ERR_INVALID_ARG, "scratch must be 256-byte aligned");
  if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)scores.v | (uintptr_t)scores.s) & 15)
    return failp(ctx, SA_ERR_INVALID_ARG, "search: Q, K, V, v, s must be 16-byte aligned");
  Plan z;
  sa_status st = plan(ctx, &z);
  if (st != SA_OK) return failp(ctx, st, "search: sizes not supported");
  if (scratch_bytes < z.total) return failp(ctx, SA_ERR_BUFFER_TOO_SMALL, "scratch smaller than sa_search_scratch_bytes");
  hipStream_t stream = (hipStream_t)hip_stream;
  const sa::Shape &sh = ctx->sh;
  const int N = sh.N, nb = sh.nb, b = sh.b;
  Layout l;

  // pairs of an index made of whole blocks, the nb diagonal ones among them
  auto block_pairs = [&](int64_t blocks) { return (blocks - nb) * b * b + (int64_t)nb * b * (b + 1) / 2; };
  // The sizes of the candidates whose pairs are known without an index are the same for every head.
  Refine tri, clu;
  tri.start(z.full.x_lo[0], z.full.x_hi[0]);
  while (!tri.done) tri.step(block_pairs(sa::triangular_count(nb, sh.sink, (int)tri.x)), target_pairs, eps_pairs);
  clu.start(z.full.x_lo[2], z.full.x_hi[2]);
  while (!clu.done) clu.step(block_pairs(clu.x), target_pairs, eps_pairs);
  // A bisection evaluates the ends and a size per halving; the first step takes both ends and the middle, every
  // other one two sizes in a row.
  const int64_t x_lo = z.full.x_lo[1], x_hi = z.full.x_hi[1];
  const Sizes known = {x_lo, tri.x, clu.x};
  int halvings = 0;
  for (int64_t w = x_hi - x_lo; w > 1; w = (w + 1) / 2) ++halvings;
  const int rounds = 1 + halvings / 2;
  const bool ranked = N <= kRankMaxSeq;  // all steps in one launch

  // host memory of the call: what goes to the device (nothing where one launch takes all steps), what comes back
  const int nblocks = (N + 15) / 16 < kNormBlocks ? (N + 15) / 16 : kNormBlocks;
  static_assert(sizeof(Refine) % sizeof(double) == 0, "the sums follow the states");
  const int most = z.full.heads;
  const std::unique_ptr<sa::HeadBudget[]> head(ranked ? nullptr : new (std::nothrow) sa::HeadBudget[(size_t)most * (kSets + kProbes)]);
  const std::unique_ptr<Refine[]> begin(ranked ? nullptr : new (std::nothrow) Refine[most]);
  const std::unique_ptr<double[]> back(new (std::nothrow) double[most * (sizeof(Refine) / sizeof(double) + 3 * (size_t)nblocks)]);
  if (!back || (!ranked && (!head || !begin))) return failp(ctx, SA_ERR_INVALID_ARG, "search: out of host memory");
  sa::HeadBudget *hb = head.get();
  Refine *hr = begin.get();
  for (int i = 0; !ranked && i < most; ++i) hr[i].start(x_lo, x_hi);
  hipError_t he = hipSuccess;
  auto ok = [&](hipError_t e) {
    if (e != hipSuccess && he == hipSuccess) he = e;
    return he == hipSuccess;
  };
  int B = 0, gb = 0;  // heads of the batch, and of a KV head in it
  for (int h0 = 0; h0 < sh.Hq && he == hipSuccess; h0 += B) {
    if (B != z.heads_from(h0)) {  // the device and the host are done with the batch before
      B = z.heads_from(h0);
      const Batch &batch = B == z.full.heads ? z.full : z.last;
      gb = B / batch.kv_heads;
      if ((st = lay_out(batch, (char *)scratch, &l)) != SA_OK) return failp(ctx, st, "search: batch rejected");
      for (int i = 0; !ranked && i < B; ++i) {
        for (int p = 0; p < kProbes; ++p) hb[kSets * B + virtual_head(i, p, gb, kProbes)] = slash_budget(hr[i].probe(p), N, nb);
        for (int k = 0; k < kSets; ++k) hb[virtual_head(i, k, gb, kSets)] = set_budget(k, known, N, nb);
      }
    }
    const size_t norms = (size_t)B * 3 * nblocks;
    const double *hp = back.get() + B * (sizeof(Refine) / sizeof(double));
    const sa::Shape &cs = l.cs, &ps = l.ps;
    const sa::Workspace &ws = l.ws;
    const sa_index &ix = l.ix;
    uint16_t *outputs = l.outputs;
    sa::HeadBudget *budgets = l.budgets, *probes = l.probes;
    Refine *state = l.state;
    double *partial = l.partial;
    const uint16_t *Qh = (const uint16_t *)Q + (size_t)h0 * sh.q_hs;
    const uint16_t *Kh = (const uint16_t *)K + (size_t)(h0 / sh.g) * sh.kv_hs;
    const uint16_t *Vh = (const uint16_t *)V + (size_t)(h0 / sh.g) * sh.kv_hs;
    const sa_scores sc{scores.v + (size_t)h0 * N, scores.s + (size_t)h0 * N, scores.blk + (size_t)h0 * nb * nb};
    if (!ranked) {
      ok(hipMemcpyAsync(budgets, hb, (size_t)B * (kSets + kProbes) * sizeof(sa::HeadBudget), hipMemcpyHostToDevice, stream));
      ok(hipMemcpyAsync(state, hr, (size_t)B * sizeof(Refine), hipMemcpyHostToDevice, stream));
    }
    // RefineSearchSpace of the Interval-Slash candidate, all heads a step per round (a head that is done
    // repeats its last index)
    sa::Override ov;
    for (int h = 0; h < sa::kMaxHeads; ++h) ov.pat[h] = SA_INTERVAL_SLASH;
    if (ranked && he == hipSuccess) {
      slash_refine_kernel<<<B, kRankThreads, 0, stream>>>((const uint32_t *)sc.v, (const uint32_t *)sc.s, N, b, gb, known, x_hi,
                                                          state, budgets, target_pairs, eps_pairs);
      ok(hipGetLastError());
    }
    for (int r = 0; !ranked && r < rounds && he == hipSuccess; ++r) {
      if (!ok(sa::launch_build_index(ps, ws, sc, ov, ix, stream, probes))) break;
      slash_step_kernel<<<dim3(B, kProbes), kStepThreads, 0, stream>>>(ix.cols, ix.offs, cs.k_v, cs.k_s, N, b, gb, state, probes,
                                                                       budgets, target_pairs, eps_pairs);
      ok(hipGetLastError());
    }
    // dense reference (the band as wide as the sequence) and every refined candidate, and the candidates against it
    for (int i = 0; i < B; ++i)
      for (int k = 0; k < kSets; ++k)
        ov.pat[virtual_head(i, k, gb, kSets)] = (int8_t)(k == 0 ? SA_TRIANGULAR : k - 1);
    if (he == hipSuccess && ok(sa::launch_build_index(cs, ws, sc, ov, ix, stream, budgets)) &&
        ok(sa::launch_sparse_prefill(cs, ws, Qh, Kh, Vh, ix, outputs, nullptr, stream))) {
      sq_diff_kernel<<<dim3(nblocks, B, kSets - 1), 256, 0, stream>>>(outputs, gb, N, partial);
      ok(hipGetLastError());
    }
    ok(hipMemcpyAsync(back.get(), state, (size_t)B * sizeof(Refine) + norms * 8, hipMemcpyDeviceToHost, stream));
    // also after an error: nothing of this call is in flight when it returns
    const hipError_t last = hipStreamSynchronize(stream);
    if (!ok(last)) break;
    for (int i = 0; i < B; ++i) {
      sa_search_head &r = out_host[h0 + i];
      Refine slash;
      memcpy(&slash, back.get() + i * (sizeof(Refine) / sizeof(double)), sizeof(Refine));
      const Refine *c[3] = {&tri, &slash, &clu};
      for (int p = 0; p < 3; ++p) {
        double sum = 0.0;
        for (int k = 0; k < nblocks; ++k) sum += hp[((size_t)p * B + i) * nblocks + k];
        r.param[p] = (int32_t)c[p]->x;
        r.pairs[p] = c[p]->px;
        r.err[p] = std::sqrt(sum);
      }
      r.pattern = 0;
      for (int p = 1; p < 3; ++p)
        if (r.err[p] < r.err[r.pattern]) r.pattern = p;
    }
  }
  if (he == hipSuccess) return SA_OK;
  snprintf(ctx->err, sizeof(ctx->err), "HIP: %s", hipGetErrorString(he));
  return SA_ERR_HIP;
}

}  // extern "C"
