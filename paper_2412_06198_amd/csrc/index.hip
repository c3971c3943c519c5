// Index builder for gfx950: per-head pattern choice and top-k selection
// (Main Idea "Categorization of Attention Heads"; Alg. 2 TopK / CombineIndices;
// Alg. 3 TopKBlocks).
//
// Integer work only: scores are compared through their fp32 bit patterns (all
// scores are >= +0, so the unsigned order is the numeric order), ties go to the
// lower index, and the pattern rule sums floor(score * 2^30) in 64-bit integers.
//
// Five selections run side by side for every head, so that nothing waits on the
// pattern decision: the probe_v / probe_s best of v and s (pattern rule), the
// k_v best columns, the k_s best diagonals, the k_b - nb best blocks.  Where workgroups can hold the arrays in
// segments and what those select (see idx_top_kernel and held_arrays), two launches; else five:
//   zero    clears the head's counters;
//   hist    one pass over the scores: 2048 logarithmic bins (64 per octave);
//   refine  a second pass that splits a bin in 1024, only for selections whose boundary bin holds
//           more keys than a list can take (it returns at once otherwise, which is the rule);
//   count   a pass that counts, per wave, the keys above the boundary bin and appends the few
//           inside it to a list, from which the exact threshold follows (or, where long runs of equal
//           scores leave more of them than a list takes, counts them per wave);
//   emit    a pass that writes the selected entries in index order (wave ballots), so the result
//           is sorted without any sort; only the pattern's own arrays are read.
// Small steps between the passes (finding a bin, resolving a list, prefixes, the pattern decision)
// are done by the workgroup of a head and array that arrives last, not by launches of their own:
// an integer ticket says who that is, nobody waits.  What it reads from the others travels in
// atomic operations and agent-scope loads and stores (which pass the L2 caches by), each completed
// before the ticket is drawn (vmcnt(0) in every wave, then the workgroup's barrier), so that no cache has to
// be written back or invalidated on the way.  The order rests on gfx950 there: a memory operation that
// the counter reports as done has been performed at its scope.  The language promises nothing of the kind
// for relaxed atomics, and the fences that would cost an L2 write-back per workgroup.
// Every launch costs 3 to 8 us whatever it does, and a pass over the scores of 32 heads 10 to 40 us.  Five
// launches take 30 us at 10K tokens, 40 at 16K, 55 at 32K, 60 at 64K and 103 at 128K; two, where they are taken,
// 21, 30, 44, 41 and none (4 heads at 4K: 14).
//
// With the per-row block rule (every row block of a Block-Cluster head keeps the
// same fraction of its causal blocks) the fifth selection is switched off and
// the emission selects inside each row instead: one wave per row, keys in
// registers, the threshold found by halving the range of the row's keys.
//
// With block-granular diagonals the selected offsets of the Interval-Slash heads become rows of
// the block CSR, in the second launch of the held form or in one after the emission (diag_rows).
#include <algorithm>
#include <cstddef>

#include "sa_internal.h"

namespace sa {
namespace {

constexpr int BT = 256;            // threads per workgroup
constexpr int WPB = BT / 64;       // waves per workgroup
constexpr int kUnit = 256;         // keys a wave takes with one load: 16 bytes per lane
constexpr int kVsUnits = 4;        // units of v or s per wave
constexpr int kMaxVsParts = kMaxSeq / (kVsUnits * kUnit);
constexpr int kMaxBlkParts = 512;  // waves that share the block map of a head
constexpr int kMaxNb = kMaxSeq / 64;
constexpr int NSEL = 5;            // 0: v probe, 1: s probe, 2: v top k_v, 3: s top k_s, 4: blk top k_b - nb
constexpr int kBins = 2048, kSubBins = 1024;
constexpr int kBinShift = 17;      // key bits below a bin: 6 mantissa bits count
// Bin 0 takes everything up to 2^-25 (2^-19), the last bin everything from 2^7 (2^13) on: window
// sums stay below 64 and block weights below 1, or below the row length where they are scaled by it.
constexpr int kBase = ((127 + 7) << 6) - kBins, kBaseRowNorm = ((127 + 13) << 6) - kBins;
constexpr int kListVs = 4096, kListBlk = 16384;  // boundary keys that are listed without splitting their bin first
// Keys of a range that does not fit its list are counted one by one, per wave part, while there are no more
// different ones than this: what the refine pass leaves of a bin.
constexpr int kDense = 1 << (kBinShift - 10);
constexpr int kMaxSegs = 8, kMaxMapSegs = 16;  // of arrays that workgroups hold

typedef unsigned long long u64;
typedef unsigned u32x4a __attribute__((ext_vector_type(4), aligned(4)));

// per-head scratch in the workspace
struct IdxScratch {
  alignas(16) unsigned hist1[3][kBins];   // per array: v, s, blk
  alignas(16) unsigned hist2[NSEL][kSubBins];
  u64 vtot, ct, topsum[2];
  unsigned nlist[NSEL];                   // boundary keys appended so far
  unsigned ticket[3][3];                  // per launch (hist, refine, count) and array
  unsigned ticket_vs;                     // v and s resolved (where their launch writes the patterns)
  unsigned dense_max[NSEL], dense_inv[NSEL];  // of a range with more keys than a list takes: largest key, largest ~key
  // everything above is zeroed at the start of a call
  alignas(16) u64 psum[2];                // sums of the probe best of v and s
  // arrays that workgroups hold whole or in segments: sums of v per segment, best keys per segment of v and s
  u64 seg_vtot[kMaxSegs], seg_ct[kMaxSegs];
  unsigned seg_best[2][64], seg_thr[3][kMaxMapSegs];
  unsigned lo[NSEL], last[NSEL];          // key range that holds the k-th key of a selection ...
  unsigned rem[NSEL], pop[NSEL];          // ... its rank inside, and the keys in the range
  unsigned thr[NSEL], need[NSEL];
  unsigned wgt[2][kMaxVsParts], weq[2][kMaxVsParts];  // v / s: counts per wave part, then exclusive prefixes
  unsigned bgt[kMaxBlkParts], beq[kMaxBlkParts];      // blk: likewise
};
constexpr size_t kZeroBytes = offsetof(IdxScratch, psum);
static_assert(kZeroBytes % 16 == 0, "cleared 16 bytes at a time");

struct IdxArgs {
  const unsigned *v, *s, *blk;     // fp32 scores as bit patterns
  IdxScratch *scratch;
  u64 *list_vs, *list_blk;         // [Hq][4][cap_vs], [Hq][cap_blk]: boundary keys, (key << 32) | wave part
  int32_t *doffs;                  // [Hq][k_s] selected offsets when they are kept as blocks
  int cap_vs, cap_blk;
  Shape sh;
  Override ov;
  sa_index out;
  int Pv, Pb;                      // workgroups per head for v (and for s), and for the block map
  int refine_vs, refine_blk;       // likewise, in the refine launch
  int vpart, bpart;                // entries of v and s, and of the block map (row-major, upper half included) per wave
  int first;                       // array v of a launch starts at workgroup -first (see Role)
  int decide_here;                 // 1: the launches before the emission write the patterns, 0: it decides by itself
  int ksel[NSEL];                  // clamped k of every selection
  u64 nb_magic;                    // ceil(2^40 / nb)
  unsigned wrap_magic;             // ceil(2^20 / nb)
  u64 share_magic;                 // floor(2^64 / (nb (nb + 1) / 2)) + 1
  u64 E, ET;                       // causal window entries; those in the sink + band region
  // Heads (bit h) whose pattern override makes the v/s selections, or the block selection, unnecessary.
  uint32_t skip_vs[kMaxHeads / 32], skip_blk[kMaxHeads / 32];
  // Not null: the patterns an earlier launch decided ([Hq], device); the block-map part of the work
  // is then done for the Block-Cluster heads only (the block map of the others was never computed).
  const int32_t *decided;
  const HeadBudget *hb;            // not null: budgets per head instead of the configuration's
  // Arrays that workgroups hold (see idx_top_kernel): segments of v (and of s) and of the block map's lower triangle,
  // keys of a segment; the best of a segment, indices ([Hq][2][segments][cap], [Hq][segments][cap]) and, where
  // there are several segments, keys in the same order.
  int held, seg_vs, seg_blk, per_vs, per_blk, cap_top_vs, cap_top_blk, place_vs;
  unsigned *top_vs, *top_blk, *top_vs_key, *top_blk_key;
};

// What crosses workgroups inside a launch: agent-scope accesses, see the top of the file.
__device__ inline unsigned agent_load(const unsigned *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline u64 agent_load(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void agent_store(unsigned *p, unsigned x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void agent_store(u64 *p, u64 x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// True in the workgroup that draws ticket n - 1: every access of the others has completed by then.
// Called by all threads.
__device__ inline bool arrives_last(unsigned *ticket, unsigned n) {
  __shared__ unsigned s_last;
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this thread's stores and atomics have been performed
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(ticket, 1u) == n - 1;
  __syncthreads();
  asm volatile("" ::: "memory");
  return s_last != 0;
}

__device__ inline HeadBudget head_budget(const IdxArgs &a, int h) {
  if (a.hb) return a.hb[h];
  HeadBudget b;
  b.k_v = a.ksel[2]; b.k_s = a.ksel[3]; b.k_b = a.sh.k_b; b.local = a.sh.local;
  return b;
}

// k of selection q, never more than there are candidates
__device__ inline int ksel(const IdxArgs &a, int h, int q) {
  if (!a.hb || q < 2) return a.ksel[q];
  const HeadBudget b = a.hb[h];
  if (q < 4) return min(q == 2 ? b.k_v : b.k_s, a.sh.N);
  const long long ncand = (long long)a.sh.nb * (a.sh.nb - 1) / 2, k = (long long)b.k_b - a.sh.nb;
  return (int)(k < 0 ? 0 : k < ncand ? k : ncand);
}

// Whether a launch has to touch one part of a head's work (the selections on v and s, or the one on
// the block map): with a pattern override only the overridden pattern's own selection is needed,
// none for Triangular.
__device__ inline bool head_wants(const IdxArgs &a, int h, bool blk_part) {
  const int w = h >> 5;  // four words: selected without indexing the argument block dynamically
  const uint32_t *m = blk_part ? a.skip_blk : a.skip_vs;
  const uint32_t bits = w == 0 ? m[0] : w == 1 ? m[1] : w == 2 ? m[2] : m[3];
  if ((bits >> (h & 31)) & 1u) return false;
  if (!blk_part) return true;
  if (a.decided && a.decided[h] != SA_BLOCK_CLUSTER) return false;
  return !a.sh.row_select && ksel(a, h, 4) > 0;
}

// A workgroup's array and its number among the workgroups of that array.
struct Role { int arr, p, n; };
__device__ inline Role role_of(const IdxArgs &a) {
  const int x = (int)blockIdx.x + a.first;
  if (x < a.Pv) return {0, x, a.Pv};
  if (x < 2 * a.Pv) return {1, x - a.Pv, a.Pv};
  return {2, x - 2 * a.Pv, a.Pb};
}
// Selections of an array: 0 and 2 on v, 1 and 3 on s, 4 on the block map.
__device__ inline int n_sel(int arr) { return arr < 2 ? 2 : 1; }
__device__ inline int sel_of(int arr, int k) { return arr < 2 ? arr + 2 * k : 4; }

// floor(x * 2^30) of a finite fp32 x >= 0 given by its bits: the scaling is exact, the conversion
// truncates, and from 2^32 on the value is a multiple of 2^9.
__device__ inline u64 fx30(unsigned bits) {
  const float f = __uint_as_float(bits) * 1073741824.f;
  const bool big = f >= 4294967296.f;
  const u64 u = (unsigned)(big ? f * 0.00390625f : f);
  return big ? u << 8 : u;
}

// Pattern of a head by the integer lift tests, from the sums of v (all, and in the Triangular region) and the
// sums sv, ss of the probe best of v and s.
__device__ inline int decide_pattern(const IdxArgs &a, u64 vtot, u64 ct, u64 sv, u64 ss) {
  const Shape &sh = a.sh;
  typedef unsigned __int128 u128;
  if ((u128)sh.lift_den * ct * a.E >= (u128)sh.lift_num * vtot * a.ET) return SA_TRIANGULAR;
  if ((u128)sh.lift_den * (sv + ss) * a.E >=
      (u128)sh.lift_num * vtot * (u64)(sh.probe_v + sh.probe_s) * (u64)sh.w)
    return SA_INTERVAL_SLASH;
  return SA_BLOCK_CLUSTER;
}

// Blocks that row block R keeps under the per-row rule: the same fraction k_b / (nb (nb+1) / 2) of
// its R + 1 causal blocks, rounded up (the diagonal block is one of them).  The quotient by a product
// with the reciprocal: exact, dividends stay below 2^36 and the divisor below 2^23.
__device__ inline int row_share(const IdxArgs &a, int R) {
  const u64 all = (u64)a.sh.nb * (a.sh.nb + 1) / 2;
  const u64 k = all == 1 ? 1 : __umul64hi((u64)min((u64)a.sh.k_b, all) * (R + 1) + all - 1, a.share_magic);
  return (int)(k < (u64)R + 1 ? k : R + 1);
}

// Triangular rows: row R keeps the blocks C < min(sink, band start) and the band of `local` blocks.
__device__ inline int tri_prefix(int sink, int local, int R) {  // blocks in the rows above R
  if (R <= local) return R * (R + 1) / 2;
  const int m = R - local;  // rows whose band starts at 1 .. m
  const int s = m <= sink ? m * (m + 1) / 2 : sink * (sink + 1) / 2 + (m - sink) * sink;
  return local * (local + 1) / 2 + m * local + s;
}

// ---- candidate walks ---------------------------------------------------------------------------
// Four entries of an array per lane: keys, their place (v and s: R = 0 and C = the index), which of
// them lie in the array (bit j of `in`) and which are candidates (`ok`).
struct Four {
  unsigned k[4];
  int R[4], C[4];
  unsigned in, ok;
};

// One wave part of an array, a unit of 256 entries at a time, two units' loads ahead.  v and s are
// plain; the block map is walked as a run of the row-major map, of which the entries C < R are the
// candidates and units above the diagonal are passed over unread.  Most units of long rows are all
// candidates, which is wave-uniform and carries no tests per entry.  fn is called by all 64 lanes
// (and compiled in once: in the short launches of this file the cold fetch of the code itself
// counts).  With row_norm the key of an entry of row R is its value times R + 1 (one fp32
// multiplication; all values are >= +0, so the products order like their bit patterns too).
// part: wave-uniform.
template <class Fn>
__device__ __forceinline__ void visit(const IdxArgs &a, int arr, const unsigned *src, int part, Fn fn) {
  const int lane = threadIdx.x & 63, nb = a.sh.nb;
  const unsigned total = arr == 2 ? (unsigned)nb * (unsigned)nb : (unsigned)a.sh.N;
  const unsigned len = (unsigned)(arr == 2 ? a.bpart : a.vpart);
  const unsigned begin = (unsigned)part * len, end = min(begin + len, total);
  struct Unit { u32x4a x; int R0, C0, kind; };  // kind 0: nothing to see, 1: mixed, 2: all candidates
  auto fetch = [&](unsigned u0, Unit &u) {
    u.kind = u.R0 = 0;
    u.C0 = (int)u0;
    if (u0 >= end) return;
    if (arr == 2) {
      u.R0 = (int)(((u64)u0 * a.nb_magic) >> 40);
      u.C0 = (int)u0 - u.R0 * nb;
      u.kind = u.C0 + kUnit > nb ? 1 : u.C0 + kUnit <= u.R0 ? 2 : u.C0 > u.R0 ? 0 : 1;
      if (u.kind == 0) return;
    } else {
      u.kind = u0 + kUnit <= total ? 2 : 1;
    }
    const unsigned e = u0 + 4 * lane;
    if (e + 3 < total) {
      u.x = *(const u32x4a *)(src + e);
    } else {
      u.x.x = e < total ? src[e] : 0u;
      u.x.y = e + 1 < total ? src[e + 1] : 0u;
      u.x.z = e + 2 < total ? src[e + 2] : 0u;
      u.x.w = 0u;
    }
  };
  Unit cur, n1, n2;
  fetch(begin, n1);
  fetch(begin + kUnit, n2);
#pragma unroll 1
  for (unsigned u0 = begin; u0 < end; u0 += kUnit) {
    cur = n1;
    n1 = n2;
    fetch(u0 + 2 * kUnit, n2);
    if (cur.kind == 0) continue;
    Four f;
    f.k[0] = cur.x.x; f.k[1] = cur.x.y; f.k[2] = cur.x.z; f.k[3] = cur.x.w;
    int c = cur.C0 + 4 * lane, r = cur.R0;
    if (cur.kind == 2) {
      f.in = f.ok = 15u;
#pragma unroll
      for (int j = 0; j < 4; ++j) { f.R[j] = r; f.C[j] = c + j; }
    } else if (arr != 2) {
      f.in = f.ok = c < (int)total ? 15u : 0u;  // N is a multiple of 4
#pragma unroll
      for (int j = 0; j < 4; ++j) { f.R[j] = r; f.C[j] = c + j; }
    } else {
      // rows passed: one at most where a unit is no longer than a row, else by c / nb (c < nb + 256)
      const int w = nb >= kUnit ? (c >= nb ? 1 : 0) : (int)(((unsigned)c * a.wrap_magic) >> 20);
      r += w;
      c -= w * nb;
      if ((nb & 3) == 0) {  // the four entries share their row
        f.in = u0 + 4 * lane < total ? 15u : 0u;
        f.ok = f.in & ((1u << min(max(r - c, 0), 4)) - 1u);
#pragma unroll
        for (int j = 0; j < 4; ++j) { f.R[j] = r; f.C[j] = c + j; }
      } else {
        f.in = f.ok = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f.R[j] = r; f.C[j] = c;
          if (u0 + 4 * lane + j < total) {
            f.in |= 1u << j;
            if (c < r) f.ok |= 1u << j;
          }
          const bool wrap = c + 1 >= nb;
          r += wrap ? 1 : 0;
          c = wrap ? 0 : c + 1;
        }
      }
    }
    if (arr == 2 && a.sh.row_norm) {
#pragma unroll
      for (int j = 0; j < 4; ++j) f.k[j] = __float_as_uint(__uint_as_float(f.k[j]) * (float)(f.R[j] + 1));
    }
    fn(f);
  }
}

// The largest (smallest) of the wave's values.
__device__ inline unsigned wave_max(unsigned x) {
  x = max(x, lane_move<0x111, 0xF>(x));
  x = max(x, lane_move<0x112, 0xF>(x));
  x = max(x, lane_move<0x114, 0xF>(x));
  x = max(x, lane_move<0x118, 0xF>(x));
  x = max(x, lane_move<0x142, 0xA>(x));
  x = max(x, lane_move<0x143, 0xC>(x));
  return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ inline unsigned wave_min(unsigned x) { return ~wave_max(~x); }
// Exclusive prefixes of two values per thread over the 64 * NW threads of a workgroup: lane moves inside
// the waves, the wave totals through LDS (wsum: 2 * NW words).  Called by all threads.
template <int NW>
__device__ inline void block_exclusive_scan2(unsigned &a, unsigned &b, unsigned *wsum) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const unsigned ia = wave_inclusive_sum(a), ib = wave_inclusive_sum(b);
  if (lane == 63) { wsum[wv] = ia; wsum[NW + wv] = ib; }
  __syncthreads();
  const unsigned ta = wave_inclusive_sum(lane < NW ? wsum[lane] : 0u);
  const unsigned tb = wave_inclusive_sum(lane < NW ? wsum[NW + lane] : 0u);
  const unsigned ba = wv ? __builtin_amdgcn_readlane(ta, wv - 1) : 0u, bb = wv ? __builtin_amdgcn_readlane(tb, wv - 1) : 0u;
  __syncthreads();
  a = ba + ia - a;
  b = bb + ib - b;
}

// The bins of a workgroup's histogram (NB bins of COPIES interleaved counters: the weights of a map's
// row are nearly equal, so a wave's additions meet in a few bins, and lanes of different copies at least
// do not wait for each other) that hold the k-th keys counted from the top bin down, for ns values of k
// (1 <= k <= total), with the rank of that key inside the bin and the bin's count.  All threads; pick is
// valid after the call.
struct Pick { unsigned bin, rank, count; };

template <int NT, int NB, int COPIES>
__device__ __forceinline__ void block_find_kth(const unsigned *hist, int ns, unsigned k0, unsigned k1, Pick *pick, unsigned *wsum) {
  constexpr int PER = NB / NT;  // thread t owns PER bins, the first threads the top ones
  const int top = NB - 1 - (int)threadIdx.x * PER;
  unsigned c[PER], tot = 0, unused = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    c[i] = hist[(top - i) * COPIES];
#pragma unroll
    for (int y = 1; y < COPIES; ++y) c[i] += hist[(top - i) * COPIES + y];
    tot += c[i];
  }
  unsigned above = tot;
  block_exclusive_scan2<NT / 64>(above, unused, wsum);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (above < k0 && k0 <= above + c[i]) pick[0] = {(unsigned)(top - i), k0 - above, c[i]};
    if (ns > 1 && above < k1 && k1 <= above + c[i]) pick[1] = {(unsigned)(top - i), k1 - above, c[i]};
    above += c[i];
  }
  __syncthreads();
}

// grid (Hq, parts): clears the counters of a head
__global__ __launch_bounds__(BT) void idx_zero_kernel(IdxScratch *scratch) {
  uint4 *p = (uint4 *)(scratch + blockIdx.x);
  for (unsigned i = blockIdx.y * BT + threadIdx.x; i < kZeroBytes / 16; i += gridDim.y * BT)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Shift that brings the offsets of a key range into kSubBins digits.
__device__ inline int digit_shift(unsigned width_minus_1) {
  const int bits = 32 - __clz((int)width_minus_1);  // __clz(0) = 32
  return bits > 10 ? bits - 10 : 0;
}

// ---- building blocks of the passes -----------------------------------------------------------------
constexpr int kCopies = 2;
constexpr int kL1Words = kBins * kCopies, kSubWords = kSubBins;
constexpr int kList = 512;        // boundary keys of a selection that a workgroup holds in LDS

__device__ inline int first_bin(const IdxArgs &a, int arr) { return arr == 2 && a.sh.row_norm ? kBaseRowNorm : kBase; }
__device__ inline const unsigned *array_of(const IdxArgs &a, int arr, int h) {
  const size_t q = (size_t)query_head(h, a.sh.g, a.sh.gq);
  return arr == 2 ? a.blk + q * a.sh.nb * a.sh.nb : (arr ? a.s : a.v) + q * a.sh.N;
}

// One wave part into the level-1 histogram; of v also the fixed-point sums over all keys and over
// those of the Triangular region.
__device__ inline void hist_part(const IdxArgs &a, int arr, const unsigned *src, int part, unsigned *hist,
                                 u64 &vt, u64 &ct) {
  const Shape &sh = a.sh;
  const int base = first_bin(a, arr), copy = threadIdx.x & (kCopies - 1);
  int sbnd = (int)min((long long)sh.sink * sh.b, (long long)sh.N);
  int lb0 = max((sh.nb - sh.local) * sh.b, sbnd);
  visit(a, arr, src, part, [&](const Four &f) {
    int bin[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) bin[j] = min(max((int)(f.k[j] >> kBinShift) - base, 0), kBins - 1);
    // the neighbours of a lane often share their bin
    if (f.ok == 15u && bin[0] == bin[1] && bin[0] == bin[2] && bin[0] == bin[3]) {
      atomicAdd(&hist[bin[0] * kCopies + copy], 4u);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((f.ok >> j) & 1u) atomicAdd(&hist[bin[j] * kCopies + copy], 1u);
    }
    if (arr == 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((f.ok >> j) & 1u) {
          const u64 x = fx30(f.k[j]);
          vt += x;
          if (f.C[j] < sbnd || f.C[j] >= lb0) ct += x;
        }
    }
  });
}

// The range of keys that bin `bin` of the level-1 histogram stands for (of one that is 2^FINE times as fine).
template <int FINE = 0>
__device__ inline void bin_range(unsigned bin, int base, unsigned &lo, unsigned &last) {
  lo = bin == 0 ? 0u : (bin + (base << FINE)) << (kBinShift - FINE);
  last = bin == (kBins << FINE) - 1 ? 0xFFFFFFFFu : ((bin + 1 + (base << FINE)) << (kBinShift - FINE)) - 1u;
}

// The selections of one array on their way to a threshold: the k-th key lies in lo .. last, has rank
// `rank` from the top there, and n keys lie in that range.
struct Ranges {
  unsigned lo[2], last[2], rank[2], n[2];
  __device__ inline bool open(int k, unsigned most) const { return n[k] > most && lo[k] != last[k]; }
};
// The digit of every wanted selection from its histogram of digits, and the narrower ranges.
template <int NT>
__device__ inline void narrow_step(int ns, unsigned (*hist)[kSubWords], Pick *pick, unsigned *wsum,
                                   const bool (&want)[2], Ranges &r) {
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (want[k]) {
      block_find_kth<NT, kSubBins, 1>(hist[k], 1, r.rank[k], 0u, &pick[k], wsum);
      const int shift = digit_shift(r.last[k] - r.lo[k]);
      r.lo[k] += pick[k].bin << shift;
      r.last[k] = min(r.last[k], r.lo[k] + ((1u << shift) - 1u));
      r.rank[k] = pick[k].rank;
      r.n[k] = pick[k].count;
    }
}

// Counts the keys of `bits` (bit j: entry j of the lane) by their offset from lo, shifted: hist[(key - lo) >> shift].
// For ranges that hold runs of equal keys: a wave that meets a single value adds once, a lane likewise; additions
// of a wave to one counter take their turns otherwise, 64 of them for each entry of a lane.
__device__ inline void count_keys(const Four &f, unsigned bits, unsigned lo, int shift, unsigned *hist) {
  const u64 any = __ballot(bits != 0u);
  if (any == 0ull) return;
  unsigned d[4], mine = 0u;
  bool same = true;
#pragma unroll
  for (int j = 3; j >= 0; --j) {
    d[j] = (f.k[j] - lo) >> shift;
    if ((bits >> j) & 1u) mine = d[j];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) same = same && (!((bits >> j) & 1u) || d[j] == mine);
  const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)mine, __builtin_ctzll(any));
  if (__all(bits == 0u || (same && mine == first))) {
    unsigned n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) n += __popcll(__ballot((bits >> j) & 1u));
    if ((threadIdx.x & 63) == 0) atomicAdd(&hist[first], n);
  } else if (same) {
    if (bits) atomicAdd(&hist[mine], (unsigned)__popc(bits));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if ((bits >> j) & 1u) atomicAdd(&hist[d[j]], 1u);
  }
}

// One workgroup narrows the ranges by walks over the whole array until at most kList keys are left or
// a single one, ...
__device__ inline void narrow(const IdxArgs &a, int arr, const unsigned *src, int nparts, int ns,
                              unsigned (*hist)[kSubWords], Pick *pick, unsigned *wsum, Ranges &r) {
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  while (r.open(0, kList) || r.open(1, kList)) {
    const bool want[2] = {r.open(0, kList), r.open(1, kList)};
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * kSubWords; i += BT) (&hist[0][0])[i] = 0u;
    __syncthreads();
    for (int pt = wv; pt < nparts; pt += BT / 64)
      visit(a, arr, src, pt, [&](const Four &f) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
          if (want[k]) {
            unsigned bits = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (((f.ok >> j) & 1u) && f.k[j] >= r.lo[k] && f.k[j] <= r.last[k]) bits |= 1u << j;
            count_keys(f, bits, r.lo[k], digit_shift(r.last[k] - r.lo[k]), hist[k]);
          }
      });
    narrow_step<BT>(ns, hist, pick, wsum, want, r);
  }
  __syncthreads();
}

// ... and then, per part, counts the keys above them (up to `top`) and puts the keys inside them on
// the lists.  A range of a single key needs no list, its keys are counted.  Selection ns - 1 is the
// one whose entries are emitted; of the other, a probe, only the sum of the keys matters.
__device__ inline void collect(const IdxArgs &a, int arr, const unsigned *src, int nparts, int ns, const Ranges &r,
                               const unsigned (&top)[2], u64 (*list)[kList], unsigned *n_list, unsigned *pgt,
                               unsigned *peq, u64 &ts) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), km = ns - 1;
  const unsigned lom = km ? r.lo[1] : r.lo[0], lastm = km ? r.last[1] : r.last[0], topm = km ? top[1] : top[0];
  for (int pt = wv; pt < nparts; pt += BT / 64) {
    unsigned gt = 0, eq = 0;
    visit(a, arr, src, pt, [&](const Four &f) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((f.ok >> j) & 1u) {
          const unsigned key = f.k[j];
          if (key > lastm) {
            gt += key <= topm;
          } else if (key >= lom) {
            if (lom == lastm) ++eq;
            else list[km][atomicAdd(&n_list[km], 1u)] = ((u64)key << 32) | (unsigned)pt;
          }
          if (arr < 2 && key >= r.lo[0] && key <= top[0]) {
            if (key > r.last[0]) ts += fx30(key);
            else if (r.lo[0] != r.last[0]) list[0][atomicAdd(&n_list[0], 1u)] = ((u64)key << 32) | (unsigned)pt;
          }
        }
    });
    gt = wave_inclusive_sum(gt);
    eq = wave_inclusive_sum(eq);
    if (lane == 63) { pgt[pt] = gt; peq[pt] = eq; }
  }
  __syncthreads();
}

// Last steps of one array, by one workgroup: thresholds from the lists (each(k, fn) calls fn(key,
// part) for every key of list k on some thread), per-part prefixes of the counts (own: parts 2 tid and
// 2 tid + 1 counted elsewhere), and of v and s the sum of the probe best (ts: this thread's share of
// the keys above the probe's list, above: the workgroup's).  Both selections step together: a step
// is a chain of barriers and LDS round trips.
template <class Each>
__device__ inline u64 finish_array(const IdxArgs &a, IdxScratch *G, int arr, int nparts, int ns,
                                   const u64 (*list)[kList], Each each,
                                   unsigned (*hist)[kSubWords], Pick *pick, Ranges &r, const unsigned (&own)[2],
                                   unsigned *pgt, unsigned *peq, unsigned *wsum, u64 *red, u64 ts) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // A list of up to 64 keys, the usual case, by one wave: each lane counts the keys above its own.
  if (wv < ns) {
    const unsigned n = wv ? r.n[1] : r.n[0], rank = wv ? r.rank[1] : r.rank[0];
    if (n <= 64 && (wv ? r.lo[1] != r.last[1] : r.lo[0] != r.last[0])) {
      const unsigned key = lane < (int)n ? (unsigned)(list[wv][lane] >> 32) : 0u;
      unsigned g = 0, e = 0;
      for (unsigned i = 0; i < n; ++i) {
        const unsigned o = __builtin_amdgcn_readlane(key, i);
        g += o > key;
        e += o == key;
      }
      if (lane < (int)n && g < rank && rank <= g + e) pick[wv] = {key, rank - g, e};  // equal lanes write the same
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (k < ns && r.n[k] <= 64 && r.lo[k] != r.last[k]) {
      r.lo[k] = r.last[k] = pick[k].bin;
      r.rank[k] = pick[k].rank;
    }
  while (r.lo[0] != r.last[0] || r.lo[1] != r.last[1]) {
    const bool want[2] = {r.lo[0] != r.last[0], r.lo[1] != r.last[1]};
    __syncthreads();
    for (int i = tid; i < ns * kSubWords; i += BT) (&hist[0][0])[i] = 0u;
    __syncthreads();
    for (int k = 0; k < ns; ++k) {
      const unsigned l = k ? r.lo[1] : r.lo[0], e = k ? r.last[1] : r.last[0];
      const int shift = digit_shift(e - l);
      if (l != e)
        each(k, [&](unsigned key, int) {
          if (key >= l && key <= e) atomicAdd(&hist[k][(key - l) >> shift], 1u);
        });
    }
    narrow_step<BT>(ns, hist, pick, wsum, want, r);
  }
  const unsigned thr_p = r.lo[0], thr = ns > 1 ? r.lo[1] : r.lo[0], need = ns > 1 ? r.rank[1] : r.rank[0];
  for (int k = 0; k < ns; ++k) {
    const bool probe = k < ns - 1;
    each(k, [&](unsigned key, int pt) {
      if (probe) {
        if (key > thr_p) ts += fx30(key);
      } else {
        if (key > thr) atomicAdd(&pgt[pt], 1u);
        else if (key == thr) atomicAdd(&peq[pt], 1u);
      }
    });
  }
  if (arr < 2) {
    ts = wave_sum63(ts);
    if (lane == 63) red[wv] = ts;
  }
  __syncthreads();
  unsigned *wg = arr == 2 ? G->bgt : G->wgt[arr], *we = arr == 2 ? G->beq : G->weq[arr];
  unsigned g[2], e[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const bool in = 2 * tid + j < nparts;
    g[j] = own[j] + (in ? pgt[2 * tid + j] : 0u);
    e[j] = in ? peq[2 * tid + j] : 0u;
  }
  unsigned xg = g[0] + g[1], xe = e[0] + e[1];
  block_exclusive_scan2<BT / 64>(xg, xe, wsum);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (2 * tid + j < nparts) { wg[2 * tid + j] = xg; we[2 * tid + j] = xe; }
    xg += g[j]; xe += e[j];
  }
  if (tid == 0) {
    G->thr[sel_of(arr, ns - 1)] = thr;
    G->need[sel_of(arr, ns - 1)] = need;
  }
  u64 sum = 0;
  if (arr < 2 && tid == 0) {
    sum = (u64)r.rank[0] * fx30(thr_p);  // ties at the threshold
    for (int w = 0; w < BT / 64; ++w) sum += red[w];
  }
  return sum;
}

// Thread 0 of the workgroup that has finished v or s: the second of the two decides the pattern.
__device__ inline void finish_vs(const IdxArgs &a, IdxScratch *G, int arr, int h) {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  asm volatile("" ::: "memory");
  if (atomicAdd(&G->ticket_vs, 1u) == 1u && a.ov.pat[h] < 0)
    a.out.pattern[h] = decide_pattern(a, agent_load(&G->vtot), agent_load(&G->ct), agent_load(&G->psum[0]), agent_load(&G->psum[1]));
}

// ---- pass 1: histograms ------------------------------------------------------------------------
// grid (workgroups of v, s and the block map, Hq)
__global__ __launch_bounds__(BT) void idx_hist_kernel(IdxArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned hist[kL1Words];
  __shared__ u64 red[2][WPB];
  __shared__ Pick pick[2];
  __shared__ unsigned wsum[2 * WPB];
  const Role ro = role_of(a);
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (!head_wants(a, h, ro.arr == 2)) return;
  IdxScratch *G = a.scratch + h;
  for (int i = tid; i < kL1Words / 4; i += BT) ((uint4 *)hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  u64 vt = 0, ct = 0;
  hist_part(a, ro.arr, array_of(a, ro.arr, h), ro.p * WPB + wv, hist, vt, ct);
  if (ro.arr == 0) {
    vt = wave_sum63(vt);
    ct = wave_sum63(ct);
    if (lane == 63) { red[0][wv] = vt; red[1][wv] = ct; }
  }
  __syncthreads();
  unsigned *gh = G->hist1[ro.arr];
  static_assert(kCopies == 2, "copies of a bin are read as one uint2");
  for (int i = tid; i < kBins; i += BT) {
    const uint2 c = ((const uint2 *)hist)[i];
    const unsigned n = c.x + c.y;
    if (n) atomicAdd(&gh[i], n);
  }
  if (ro.arr == 0 && tid < 2) {
    u64 t = 0;
    for (int w = 0; w < WPB; ++w) t += red[tid][w];
    atomicAdd(tid ? &G->ct : &G->vtot, t);
  }
  if (!arrives_last(&G->ticket[0][ro.arr], ro.n)) return;
  // the merged histogram: the bin of every selection on this array
  for (int i = tid; i < kBins; i += BT) hist[i] = agent_load(&gh[i]);
  __syncthreads();
  const int ns = n_sel(ro.arr);
  block_find_kth<BT, kBins, 1>(hist, ns, (unsigned)ksel(a, h, sel_of(ro.arr, 0)), (unsigned)ksel(a, h, sel_of(ro.arr, ns - 1)),
                               pick, wsum);
  if (tid < ns) {
    const int q = sel_of(ro.arr, tid);
    bin_range(pick[tid].bin, first_bin(a, ro.arr), G->lo[q], G->last[q]);
    G->rem[q] = pick[tid].rank;
    G->pop[q] = pick[tid].count;
  }
}

// ---- pass 2, where it is needed: a boundary bin with more keys than its list takes is split --------
// grid (refine_vs + refine_vs + refine_blk, Hq): few workgroups, since most have nothing to do (see index_args)
constexpr int kRefineVs = 4, kRefineBlk = 24;

__global__ __launch_bounds__(BT) void idx_refine_kernel(IdxArgs a) {
  __shared__ unsigned hist[2][kSubWords];
  __shared__ Pick pick[2];
  __shared__ unsigned wsum[2 * WPB];
  const int h = blockIdx.y, tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  int x = (int)blockIdx.x, arr = 2, nwg = a.refine_blk;
  if (a.first == 0) {
    if (x < 2 * a.refine_vs) { arr = x >= a.refine_vs; x -= arr ? a.refine_vs : 0; nwg = a.refine_vs; }
    else x -= 2 * a.refine_vs;
  }
  if (!head_wants(a, h, arr == 2)) return;
  IdxScratch *G = a.scratch + h;
  const int ns = n_sel(arr);
  const unsigned most = arr == 2 ? kListBlk : kListVs;
  unsigned lo[2], last[2];
  int shift[2];
  bool want[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int q = sel_of(arr, k < ns ? k : 0);
    want[k] = k < ns && G->pop[q] > most;
    lo[k] = G->lo[q]; last[k] = G->last[q];
    shift[k] = digit_shift(last[k] - lo[k]);
  }
  if (!want[0] && !want[1]) return;
  for (int i = tid; i < 2 * kSubWords; i += BT) (&hist[0][0])[i] = 0u;
  __syncthreads();
  const int nparts = (arr == 2 ? a.Pb : a.Pv) * WPB;
  for (int part = x * WPB + wv; part < nparts; part += nwg * WPB)
    visit(a, arr, array_of(a, arr, h), part, [&](const Four &f) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (want[k]) {
          unsigned bits = 0u;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (((f.ok >> j) & 1u) && f.k[j] >= lo[k] && f.k[j] <= last[k]) bits |= 1u << j;
          count_keys(f, bits, lo[k], shift[k], hist[k]);
        }
    });
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (want[k])
      for (int i = tid; i < kSubBins; i += BT) {
        const unsigned c = hist[k][i];
        if (c) atomicAdd(&G->hist2[sel_of(arr, k)][i], c);
      }
  if (!arrives_last(&G->ticket[1][arr], nwg)) return;
  Ranges r;
#pragma unroll
  for (int k = 0; k < 2; ++k) { r.lo[k] = lo[k]; r.last[k] = last[k]; r.rank[k] = G->rem[sel_of(arr, k < ns ? k : 0)]; }
  for (int k = 0; k < ns; ++k)
    for (int i = tid; i < kSubBins; i += BT) hist[k][i] = agent_load(&G->hist2[sel_of(arr, k)][i]);
  narrow_step<BT>(ns, hist, pick, wsum, want, r);
  if (tid == 0) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (want[k]) {
        const int q = sel_of(arr, k);
        G->lo[q] = r.lo[k]; G->last[q] = r.last[k]; G->rem[q] = r.rank[k]; G->pop[q] = r.n[k];
      }
  }
}

// ---- pass 3: counts, thresholds, pattern ---------------------------------------------------------
__global__ __launch_bounds__(BT) void idx_count_kernel(IdxArgs a) {
  __shared__ __attribute__((aligned(16))) u64 list[2][kList];  // the workgroup's boundary keys; later the head's
  __shared__ unsigned n_list[2], s_base[2], s_ext[2][2];
  __shared__ u64 red[WPB];
  __shared__ unsigned hist[2][kSubWords];
  __shared__ Pick pick[2];
  __shared__ unsigned pgt[kMaxBlkParts], peq[kMaxBlkParts];
  __shared__ unsigned wsum[2 * WPB];
  const Role ro = role_of(a);
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, arr = ro.arr;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (arr == 0 && ro.p == 0 && tid == 0 && a.ov.pat[h] >= 0) a.out.pattern[h] = a.ov.pat[h];
  if (!head_wants(a, h, arr == 2)) return;
  IdxScratch *G = a.scratch + h;
  const int ns = n_sel(arr), km = ns - 1;
  const unsigned cap = arr == 2 ? (unsigned)a.cap_blk : (unsigned)a.cap_vs;
  const unsigned *src = array_of(a, arr, h);
  auto list_of = [&](int k) { return arr == 2 ? a.list_blk + (size_t)h * cap : a.list_vs + ((size_t)h * 4 + arr + 2 * k) * cap; };
  if (tid < 2) n_list[tid] = 0u;
  if (tid < 4) (&s_ext[0][0])[tid] = 0u;
  Ranges r;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int q = sel_of(arr, k < ns ? k : 0);
    r.lo[k] = G->lo[q]; r.last[k] = G->last[q]; r.rank[k] = G->rem[q]; r.n[k] = G->pop[q];
  }
  // A range with more keys than its list takes holds stretches of equal scores, or nearly equal ones.  Its keys
  // are counted instead: each of them per wave part where the range has no more than kDense (what is left of a bin
  // after the refine pass), else all together with their smallest and largest.  32 heads, 128K tokens, the index
  // alone (scores without ties 108 us): v and s constant 192 us, block map constant 173, 99 of 100 blocks 0 185.
  // (One workgroup per array that walks it for them takes 1.73, 3.15 and 5.97 ms.)
  const bool dense[2] = {r.n[0] > cap, ns > 1 && r.n[1] > cap}, any_dense = dense[0] || dense[1];
  typedef unsigned __attribute__((may_alias)) word;
  word *counts[2] = {(word *)list[0], (word *)list[1]};  // [2][WPB][kDense], where the list would be
  static_assert(2 * WPB * kDense * sizeof(unsigned) <= sizeof(list[0]), "counts in place of a list");
  if (any_dense)
    for (int i = tid; i < (int)(sizeof(list) / 16); i += BT) ((uint4 *)&list[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();

  const int part = ro.p * WPB + wv;
  {
    const unsigned lom = km ? r.lo[1] : r.lo[0], lastm = km ? r.last[1] : r.last[0];
    // of a dense range; a wide one: number of keys, largest key and largest ~key, a counter of each lane's own
    auto count = [&](int k, const Four &f, unsigned bits) {
      const unsigned lo = k ? r.lo[1] : r.lo[0], last = k ? r.last[1] : r.last[0];
      word *c = (k ? counts[1] : counts[0]) + wv * kDense;
      if (last - lo < kDense) {
        count_keys(f, bits, lo, 0, c);
      } else {
        word *up = c + WPB * kDense + lane, *down = up + 64;
        c[lane] += (unsigned)__popc(bits);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if ((bits >> j) & 1u) { *up = max((unsigned)*up, f.k[j]); *down = max((unsigned)*down, ~f.k[j]); }
      }
    };
    unsigned gt = 0;
    u64 ts = 0;
    visit(a, arr, src, part, [&](const Four &f) {
      unsigned inm = 0u, inp = 0u;  // keys for the lists
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool ok = (f.ok >> j) & 1u;
        const unsigned key = f.k[j];
        gt += ok && key > lastm;
        if (ok && key >= lom && key <= lastm) inm |= 1u << j;
        if (arr < 2 && ok && key >= r.lo[0]) {
          if (key > r.last[0]) ts += fx30(key);
          else inp |= 1u << j;
        }
      }
      if (any_dense) {
        if (dense[km]) { count(km, f, inm); inm = 0u; }
        if (arr < 2 && dense[0]) { count(0, f, inp); inp = 0u; }
      }
      unsigned k0 = f.k[0], k1 = f.k[1], k2 = f.k[2], k3 = f.k[3];
      while (inm | inp) {
#pragma unroll 1
        for (int s2 = 0; s2 < 2; ++s2) {
          const int k = s2 ? 0 : km;
          if (!((s2 ? inp : inm) & 1u)) continue;
          const u64 item = ((u64)k0 << 32) | (unsigned)part;
          const unsigned n = atomicAdd(&n_list[k], 1u);
          if (n < kList) list[k][n] = item;
          else agent_store(&list_of(k)[atomicAdd(&G->nlist[sel_of(arr, k)], 1u)], item);
        }
        inm >>= 1; inp >>= 1;
        k0 = k1; k1 = k2; k2 = k3;
      }
    });
    gt = wave_inclusive_sum(gt);
    if (lane == 63) agent_store(arr == 2 ? &G->bgt[part] : &G->wgt[arr][part], gt);
    if (arr < 2) {
      ts = wave_sum63(ts);
      if (lane == 63) red[wv] = ts;
    }
  }
  __syncthreads();
  if (tid < ns) s_base[tid] = n_list[tid] ? atomicAdd(&G->nlist[sel_of(arr, tid)], min(n_list[tid], (unsigned)kList)) : 0u;
  if (arr < 2 && tid == 64) {
    u64 t = 0;
    for (int w = 0; w < WPB; ++w) t += red[w];
    if (t) atomicAdd(&G->topsum[arr], t);
  }
  __syncthreads();
  for (int k = 0; k < ns; ++k) {
    const unsigned n = min(n_list[k], (unsigned)kList), b = s_base[k];
    u64 *to = list_of(k);
    for (unsigned i = tid; i < n; i += BT) agent_store(&to[b + i], list[k][i]);
  }
  if (any_dense) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (dense[k]) {  // 16 bits each: a part has 32768 entries at most
        const word *c = counts[k] + wv * kDense, *ext = c + WPB * kDense;
        unsigned *to = (unsigned *)list_of(k) + part * (kDense / 2);
        if (r.last[k] - r.lo[k] < kDense) {
          agent_store(to + lane, c[2 * lane] | c[2 * lane + 1] << 16);
        } else {
          const unsigned n = wave_inclusive_sum(c[lane]);
          agent_store(to + 63 - lane, lane == 63 ? n : 0u);  // the last lane has the sum, word 0 takes it
          if (ext[lane]) atomicMax(&s_ext[k][0], ext[lane]);
          if (ext[64 + lane]) atomicMax(&s_ext[k][1], ext[64 + lane]);
        }
      }
    __syncthreads();
    if (tid < 4 && s_ext[tid >> 1][tid & 1])
      atomicMax((tid & 1 ? G->dense_inv : G->dense_max) + sel_of(arr, tid >> 1), s_ext[tid >> 1][tid & 1]);
  }
  static_assert(kDense == 128, "two counts per lane");
  static_assert((long long)kMaxNb * kMaxNb / kMaxBlkParts < 65536, "counts of 16 bits");
  if (!arrives_last(&G->ticket[2][arr], ro.n)) return;

  // ---- one workgroup: the exact threshold of every selection on this array.  All reads that pass the
  // L2 caches by are issued together.
  const int nparts = ro.n * WPB;
  unsigned own[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    own[j] = 2 * tid + j < nparts ? agent_load(arr == 2 ? &G->bgt[2 * tid + j] : &G->wgt[arr][2 * tid + j]) : 0u;
  u64 ts = tid == 0 && arr < 2 ? agent_load(&G->topsum[arr]) : 0ull;
  unsigned m[2] = {dense[0] ? 0u : r.n[0], ns > 1 && !dense[1] ? r.n[1] : 0u};  // on the lists
  for (int k = 0; k < ns; ++k)
    for (unsigned i = tid; i < min(m[k], (unsigned)kList); i += BT) list[k][i] = agent_load(&list_of(k)[i]);
  for (int i = tid; i < nparts; i += BT) { pgt[i] = 0u; peq[i] = 0u; }
  if (tid < 2) n_list[tid] = 0u;
  if (ns == 1) r.lo[1] = r.last[1] = r.n[1] = 0u;
  __syncthreads();
  bool counted = true;  // every dense range has kDense different keys at most, or a single one
  if (any_dense) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (dense[k] && r.last[k] - r.lo[k] >= kDense) {
        const unsigned key = agent_load(&G->dense_max[sel_of(arr, k)]);
        counted = counted && key == ~agent_load(&G->dense_inv[sel_of(arr, k)]);
      }
  }
  if (any_dense && !counted) {
    // A wide range of different keys, more than a list takes: below the lowest bin (or above the highest) only.
    const unsigned top[2] = {r.last[0], r.last[1]};
    narrow(a, arr, src, nparts, ns, hist, pick, wsum, r);
    collect(a, arr, src, nparts, ns, r, top, list, n_list, pgt, peq, ts);
    m[0] = n_list[0]; m[1] = n_list[1];
  } else if (any_dense) {
#pragma unroll 1
    for (int k = 0; k < ns; ++k) {
      if (!(k ? dense[1] : dense[0])) continue;
      const unsigned *c = (const unsigned *)list_of(k) + lane;
      unsigned lo = k ? r.lo[1] : r.lo[0];
      if ((k ? r.last[1] : r.last[0]) - lo >= kDense) lo = agent_load(&G->dense_max[sel_of(arr, k)]);
      for (int i = tid; i < kSubWords; i += BT) hist[k][i] = 0u;
      __syncthreads();
      unsigned n0 = 0, n1 = 0;
#pragma unroll 8
      for (int pt = wv; pt < nparts; pt += WPB) {
        const unsigned x = agent_load(c + pt * (kDense / 2));
        n0 += x & 0xFFFFu; n1 += x >> 16;
      }
      atomicAdd(&hist[k][2 * lane], n0);
      atomicAdd(&hist[k][2 * lane + 1], n1);
      __syncthreads();
      block_find_kth<BT, kSubBins, 1>(hist[k], 1, k ? r.rank[1] : r.rank[0], 0u, &pick[k], wsum);
      const unsigned d = pick[k].bin;
      if (k == km) {
#pragma unroll 4
        for (int pt = wv; pt < nparts; pt += WPB) {
          const unsigned x = agent_load(c + pt * (kDense / 2));
          const unsigned lo16 = x & 0xFFFFu, hi16 = x >> 16;
          const unsigned g = wave_inclusive_sum((2 * lane > (int)d ? lo16 : 0u) + (2 * lane + 1 > (int)d ? hi16 : 0u));
          if (lane == 63) pgt[pt] = g;
          if (lane == (int)(d >> 1)) peq[pt] = d & 1u ? hi16 : lo16;
        }
      } else if (tid > (int)d && tid < kDense) {
        ts += (u64)hist[k][tid] * fx30(lo + (unsigned)tid);
      }
      if (k) { r.lo[1] = r.last[1] = lo + d; r.rank[1] = pick[1].rank; }
      else { r.lo[0] = r.last[0] = lo + d; r.rank[0] = pick[0].rank; }
    }
    __syncthreads();
  }
  auto each = [&](int k, auto fn) {
    for (unsigned i = tid; i < (k ? m[1] : m[0]); i += BT) {
      const u64 it = i < kList ? list[k][i] : agent_load(&list_of(k)[i]);
      fn((unsigned)(it >> 32), (int)(unsigned)it);
    }
  };
  const u64 sum = finish_array(a, G, arr, nparts, ns, list, each, hist, pick, r, own, pgt, peq, wsum, red, ts);
  if (arr == 2 || tid != 0) return;
  agent_store(&G->psum[arr], sum);
  finish_vs(a, G, arr, h);
}

// ---- pass 4: emission ------------------------------------------------------------------------------
// One 256-key group of a wave: an element is selected if its key is above the threshold, or equal to
// it and among the first `need` such elements in index order.  visit(j, pos, sel) receives every
// element with the number of selected elements before it; grun / erun count the greater / equal
// elements seen so far.
template <class Visit>
__device__ inline void emit_group(const Four &f, unsigned thr, unsigned need,
                                  unsigned &grun, unsigned &erun, Visit visit) {
  const int lane = threadIdx.x & 63;
  const u64 below = (1ull << lane) - 1ull;
  unsigned gl = 0, el = 0, gtot = 0, etot = 0;
  bool isgt[4], iseq[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    isgt[j] = ((f.ok >> j) & 1u) && f.k[j] > thr;
    iseq[j] = ((f.ok >> j) & 1u) && f.k[j] == thr;
    const u64 bg = __ballot(isgt[j]), be = __ballot(iseq[j]);
    gl += __popcll(bg & below); el += __popcll(be & below);
    gtot += __popcll(bg); etot += __popcll(be);
  }
  unsigned G = grun + gl, E = erun + el;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    visit(j, G + min(E, need), isgt[j] || (iseq[j] && E < need));
    G += isgt[j];
    E += iseq[j];
  }
  grun += gtot;
  erun += etot;
}

// Keys raised by one: 0 stands for no key.
__device__ inline unsigned raised(unsigned key) { return max(key, key + 1u); }  // (the largest word stays: no score)

// Per-row block rule, one wave per row: out[0..kr) = the kr candidates C < R with the largest keys
// (ties to the lower C) in ascending order, out[kr] = R (the forced diagonal block).  Lane l holds four neighbours of
// every 256 keys in registers (U times, R <= 256 U), raised by one: slots past the row hold 0.
// What bounds it is its own instructions: a step of the search compares, counts and adds per 64 keys.  With 32
// steps, one per bit, and a key per lane and load the index of 32 heads took 28.8 us at 161 blocks, 61 at 512, 89 at
// 1024 and 695 at 2048; like this 25.4, 48, 57 and 126.
template <int U>
__device__ __forceinline__ void emit_row_select(const unsigned *row, int R, int kr, int32_t *out) {
  const int lane = threadIdx.x & 63;
  if (kr > 0) {
    u32x4a x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x[u] = u32x4a{0u, 0u, 0u, 0u};
      const int i = kUnit * u + 4 * lane;
      if (i + 3 < R) {
        x[u] = *(const u32x4a *)(row + i);
      } else if (i < R) {  // nothing is read behind the row: the last one ends the map
        x[u].x = row[i];
        if (i + 1 < R) x[u].y = row[i + 1];
        if (i + 2 < R) x[u].z = row[i + 2];
      }
    }
    unsigned most = 0u, least = 0xFFFFFFFFu;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = kUnit * u + 4 * lane;
      if (kUnit * u >= R) continue;
      x[u] = u32x4a{i < R ? raised(x[u].x) : 0u, i + 1 < R ? raised(x[u].y) : 0u, i + 2 < R ? raised(x[u].z) : 0u,
                    i + 3 < R ? raised(x[u].w) : 0u};
      most = max(most, max(max(x[u].x, x[u].y), max(x[u].z, x[u].w)));
      least = min(least, min(min(x[u].x - 1u, x[u].y - 1u), min(x[u].z - 1u, x[u].w - 1u)));
    }
    auto reach = [&](unsigned c) {  // keys >= c, c >= 1
      int n = 0;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (kUnit * u < R)
          n += __popcll(__ballot(x[u].x >= c)) + __popcll(__ballot(x[u].y >= c)) + __popcll(__ballot(x[u].z >= c)) +
               __popcll(__ballot(x[u].w >= c));
      return n;
    };
    // The kr-th largest key, between the smallest and the largest, in halves.  The search is over as soon as kr keys
    // reach the middle: after 12 of up to 31 steps in a row of 1000 softmax weights, the gaps between which are
    // wide against their last bits.
    unsigned lo = wave_min(least) + 1u, hi = wave_max(most), need = 0xFFFFFFFFu;  // need: ties taken, in index order
    while (kr < R) {
      if (lo == hi) {
        need = (unsigned)kr - (hi == 0xFFFFFFFFu ? 0u : (unsigned)reach(hi + 1u));
        break;
      }
      const unsigned c = lo + (hi - lo + 1u) / 2u;
      const int n = reach(c);
      if (n >= kr) lo = c;
      else hi = c - 1u;
      if (n == kr) break;
    }
    unsigned run = 0u, erun = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kUnit * u >= R) continue;
      const unsigned y[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
      u64 in[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) in[j] = __ballot(y[j] >= lo);
      if (need != 0xFFFFFFFFu) {
        u64 eq[4];
        unsigned before = erun;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          eq[j] = __ballot(y[j] == lo);
          before += __builtin_amdgcn_mbcnt_hi((unsigned)(eq[j] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)eq[j], 0u));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          in[j] &= ~__ballot(y[j] == lo && before >= need);
          before += (unsigned)((eq[j] >> lane) & 1ull);
          erun += (unsigned)__popcll(eq[j]);
        }
      }
      unsigned pos = run;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        pos = __builtin_amdgcn_mbcnt_hi((unsigned)(in[j] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in[j], pos));
        run += (unsigned)__popcll(in[j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((in[j] >> lane) & 1ull) out[pos++] = kUnit * u + 4 * lane + j;
    }
  }
  if (lane == 0) out[kr] = R;
}

// Block CSR of a Block-Cluster head under the per-row rule, by workgroups of 64 NW threads: a wave takes whole rows
// (part of nparts).  Every workgroup finds its rows' pointers for itself: thread t sums the shares of `per` rows.
template <int T, int NW>
__device__ __forceinline__ int emit_rows(const IdxArgs &a, const unsigned *hb, int part, int nparts, int32_t *rp, int32_t *bc,
                                int *s_at, unsigned *wsum) {
  const int tid = threadIdx.x, lane = tid & 63, nb = a.sh.nb;
  const int per = (nb + 64 * NW - 1) / (64 * NW);
  unsigned sum = 0, unused = 0;
  for (int j = 0; j < per; ++j)
    if (per * tid + j < nb) sum += (unsigned)row_share(a, per * tid + j);
  unsigned run = sum;
  block_exclusive_scan2<NW>(run, unused, wsum);
  for (int j = 0; j < per; ++j) {
    const int R = per * tid + j;
    if (R < nb) {
      s_at[R] = (int)run;
      run += (unsigned)row_share(a, R);
      if (R == nb - 1) s_at[nb] = (int)run;
    }
  }
  __syncthreads();
  for (int R = part; R < nb; R += nparts) {
    const int at = __builtin_amdgcn_readfirstlane(s_at[R]), end = __builtin_amdgcn_readfirstlane(s_at[R + 1]);
    if (lane == 0) rp[R] = at;
    emit_row_select<T / 4>(hb + (size_t)R * nb, R, end - at - 1, bc + at);
  }
  return s_at[nb];
}

// ---- diagonals at block granularity -----------------------------------------------------------------
// An offset o leads from row block R to the key blocks R - floor(o / b) and R - ceil(o / b): the same distances in every
// row.  So the kept blocks of row R are R - d for the distances d <= R of one set, 0 among them, and row pointers
// are sums of the counts up to each R.  Every workgroup of 64 NW threads forms the set for itself; a wave takes whole
// rows (part of nparts).  (A bitmap per row from all offsets, in a launch that counted and one that wrote, took 10 us of a layer of
// 10K tokens and 32 heads, like this nothing beside the columns' part of the placing launch.  32K, all 32 heads
// diagonals, blocks of 128: 4.7 + 2 x 5.6 before, 9.4 now in one launch; 128K, in a launch of their own: 2 x 11.6 and 9.3.)
template <int NB>
struct DiagRows {
  unsigned word[NB / 32];  // the set
  int before[NB / 32];     // distances before each word
  uint16_t dist[NB];       // in ascending order
  int at[NB + 1];          // row pointers
};
template <int NW, int NB>
__device__ __forceinline__ int diag_rows(const IdxArgs &a, const unsigned *offs, int n_offs, int part, int nparts, int32_t *rp,
                                         int32_t *bc, DiagRows<NB> &l, unsigned *wsum) {
  const int tid = threadIdx.x, lane = tid & 63, nb = a.sh.nb, words = (nb + 31) / 32, shift = a.sh.b == 128 ? 7 : 6;
  static_assert(NB / 32 <= 64 * NW, "a word per thread");
  if (tid < words) l.word[tid] = tid == 0 ? 1u : 0u;
  __syncthreads();
  for (int t = tid; t < n_offs; t += 64 * NW) {
    const unsigned o = offs[t], near = o >> shift, far = (o + a.sh.b - 1) >> shift;
    atomicOr(&l.word[near >> 5], 1u << (near & 31));
    if (far != near && far < (unsigned)nb) atomicOr(&l.word[far >> 5], 1u << (far & 31));
  }
  __syncthreads();
  unsigned bits = tid < words ? l.word[tid] : 0u, run = __popc(bits), unused = 0;
  block_exclusive_scan2<NW>(run, unused, wsum);
  if (tid < words) {
    l.before[tid] = (int)run;
    for (; bits; bits &= bits - 1u) l.dist[run++] = (uint16_t)(32 * tid + __ffs(bits) - 1);
  }
  __syncthreads();
  auto count = [&](int R) { return l.before[R >> 5] + __popc(l.word[R >> 5] & (0xFFFFFFFFu >> (31 - (R & 31)))); };
  const int per = (nb + 64 * NW - 1) / (64 * NW);
  unsigned sum = 0;
  for (int j = 0; j < per; ++j)
    if (per * tid + j < nb) sum += (unsigned)count(per * tid + j);
  run = sum;
  block_exclusive_scan2<NW>(run, unused, wsum);
  for (int j = 0; j < per; ++j) {
    const int R = per * tid + j;
    if (R < nb) {
      l.at[R] = (int)run;
      run += (unsigned)count(R);
      if (R == nb - 1) l.at[nb] = (int)run;
    }
  }
  __syncthreads();
  for (int R = part; R < nb; R += nparts) {
    const int at = l.at[R], n = l.at[R + 1] - at;
    if (lane == 0) rp[R] = at;
    for (int i = lane; i < n; i += 64) bc[at + i] = R - (int)l.dist[n - 1 - i];
  }
  return l.at[nb];
}

// Block CSR of a Triangular head (a wave takes whole rows) or an Interval-Slash head: the blocks of all rows.
__device__ inline int emit_fixed(const IdxArgs &a, int h, int pat, int part, int nparts, int gtid, int gthreads,
                                 int32_t *rp, int32_t *bc) {
  const Shape &sh = a.sh;
  const int lane = threadIdx.x & 63, nb = sh.nb;
  if (pat == SA_TRIANGULAR) {
    const int local = head_budget(a, h).local;
    for (int R = part; R < nb; R += nparts) {
      const int at = tri_prefix(sh.sink, local, R);
      const int bs = max(R - local + 1, 0), ns = min(sh.sink, bs), n = ns + R - bs + 1;
      if (lane == 0) rp[R] = at;
      for (int i = lane; i < n; i += 64) bc[at + i] = i < ns ? i : bs + i - ns;
    }
    return tri_prefix(sh.sink, local, nb);
  }
  for (int R = gtid; R < nb; R += gthreads) { rp[R] = R; bc[R] = R; }
  return nb;
}

// grid as in the passes above.  T: 64-key slices of a row under the per-row rule (nb <= 64 T), 0 for
// the rules with one selection per head.
template <int T>
__global__ __launch_bounds__(BT) void idx_emit_kernel(IdxArgs a) {
  __shared__ unsigned s_wsum[2 * WPB];
  const Shape &sh = a.sh;
  const Role ro = role_of(a);
  const int h = blockIdx.y, tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = sh.nb;
  IdxScratch *G = a.scratch + h;
  int pat = a.ov.pat[h];
  if (pat < 0) pat = a.out.pattern[h];
  pat = __builtin_amdgcn_readfirstlane(pat);
  const int part = ro.p * WPB + wv, nparts = ro.n * WPB;
  const int gtid = ro.p * BT + tid, gthreads = ro.n * BT;
  if (ro.arr < 2) {  // columns and diagonals: Interval-Slash only
    const int q = ro.arr + 2, width = ro.arr ? sh.k_s : sh.k_v;
    const int k = pat == SA_INTERVAL_SLASH ? ksel(a, h, q) : 0;
    int32_t *idx = (ro.arr ? a.out.offs : a.out.cols) + (size_t)h * width;
    const bool aside = ro.arr == 1 && sh.diag_blocks;  // the offsets become blocks: the list stays empty
    if (k > 0) {
      int32_t *dst = aside ? a.doffs + (size_t)h * width : idx;
      const unsigned thr = G->thr[q], need = G->need[q];
      unsigned grun = G->wgt[ro.arr][part], erun = G->weq[ro.arr][part];
      visit(a, ro.arr, array_of(a, ro.arr, h), part, [&](const Four &f) {
        emit_group(f, thr, need, grun, erun, [&](int j, unsigned pos, bool sel) {
          if (sel) dst[pos] = f.C[j];
        });
      });
    }
    const int shown = aside ? 0 : k;
    for (int i = shown + gtid; i < width; i += gthreads) idx[i] = -1;
    if (gtid == 0) {
      (ro.arr ? a.out.n_offs : a.out.n_cols)[h] = shown;
    }
    return;
  }
  // block CSR
  int32_t *rp = a.out.rowptr + (size_t)h * (nb + 1);
  int32_t *bc = a.out.blkcols + (size_t)h * sh.cap_b;
  const unsigned *hb = array_of(a, 2, h);
  int total;
  if (pat == SA_BLOCK_CLUSTER && T > 0) {
    __shared__ int s_at[kMaxNb + 1];
    total = emit_rows<T == 0 ? 4 : T, WPB>(a, hb, part, nparts, rp, bc, s_at, s_wsum);
  } else if (pat == SA_BLOCK_CLUSTER) {
    const int k = ksel(a, h, 4);
    // no block below the diagonal is selected: no key is above this threshold, and no tie is taken
    const unsigned thr = k > 0 ? G->thr[4] : 0xFFFFFFFFu, need = k > 0 ? G->need[4] : 0u;
    unsigned grun = k > 0 ? G->bgt[part] : 0u, erun = k > 0 ? G->beq[part] : 0u;
    // An entry of row R lands after the R diagonal blocks of the rows above; the first column of a
    // row knows the row pointer, the diagonal entry the end of the row.
    visit(a, 2, hb, part, [&](const Four &f) {
      emit_group(f, thr, need, grun, erun, [&](int j, unsigned pos, bool sel) {
        if (!((f.in >> j) & 1u)) return;
        if (f.C[j] == 0) rp[f.R[j]] = (int)pos + f.R[j];
        if (sel || f.C[j] == f.R[j]) bc[pos + f.R[j]] = f.C[j];
      });
    });
    total = k + nb;
  } else {
    total = emit_fixed(a, h, pat, part, nparts, gtid, gthreads, rp, bc);
  }
  if (gtid == 0) rp[nb] = total;
  for (int i = total + gtid; i < sh.cap_b; i += gthreads) bc[i] = -1;
}

// ---- arrays that workgroups hold --------------------------------------------------------------------
// Two launches instead of the five above: idx_top_kernel, in which a workgroup reads a segment of an array once, into
// registers, and finds the best k of its keys, and idx_place_kernel, which decides the pattern, takes the best
// of the segments' best where an array has several, and writes the index.  Nothing is merged between workgroups
// of a launch, so there are no counters to clear and no tickets.  Taken where the segments' best fit a
// workgroup again (see held_arrays).
// What such a workgroup waits for is its own instructions: one on each of 32768 keys takes a compute unit
// 0.25 us.  So few are spent on all keys: of the four keys of a lane the largest goes into a histogram
// (all four where they are alike); the k-th of those is a bound that k keys reach; the keys that reach it, a
// tenth more than k as a rule, go to a list in LDS, in order, and everything else is done on that list.  (With all
// keys in LDS and the walks over them 37 us a launch of 32 heads at 64K tokens, with 64 keys a step in
// registers 46, 25 like this.)
constexpr int ST = 1024, SW = ST / 64;
constexpr int kHeldUnits = 8;                          // units of a wave at most
constexpr int kSeg = SW * kHeldUnits * kUnit;          // keys of a workgroup
constexpr int kCap = 16384;                            // keys of its list
constexpr int kDirect = SW * kUnit;                    // keys that go to the list all
constexpr int kFew = 64;                               // keys that a wave ranks one against the other

struct TopShared {
  __attribute__((aligned(16))) unsigned hist[kL1Words];
  u64 red[2][SW];
  unsigned few[2][kFew], n_few[2];
  Pick pick[2];
  unsigned wsum[2 * SW], wgt[SW], weq[SW];
};
template <int CAP>
struct List {
  __attribute__((aligned(16))) unsigned key[CAP];
  uint16_t at[CAP];  // place in the segment
};

// Keys of a wave, four per lane and unit in index order, raised by one: 0 stands for no key.
template <int UNITS>
struct Held { u32x4a k[UNITS]; int units; };
// Units per wave and the first key of a wave for n keys.
__device__ inline int wave_units(int n) { return (n + SW * kUnit - 1) / (SW * kUnit); }

__device__ inline int bin_of(unsigned key, int base) { return min(max((int)(key >> kBinShift) - base, 0), kBins - 1); }
// Of keys that are alike: four bins in the place of one, so that fewer additions meet in one (those of a wave to one
// counter take their turns) and fewer keys share that of the k-th.
constexpr int kFine = 2, kFineBins = kBins << kFine;
__device__ inline int fine_bin_of(unsigned key, int base) {
  return min(max((int)(key >> (kBinShift - kFine)) - (base << kFine), 0), kFineBins - 1);
}
__device__ inline void zero_hist(TopShared &s) {
  for (int i = threadIdx.x; i < kL1Words / 4; i += ST) ((uint4 *)s.hist)[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Walk of a list of n keys, one per thread and step; fn is called by whole waves.
template <int CAP, class Fn>
__device__ __forceinline__ void list_visit(const List<CAP> &l, int n, Fn fn) {
#pragma unroll 1
  for (int i = threadIdx.x; i < ((n + 63) & ~63); i += ST) fn(i, i < n ? l.key[i] : 0u);
}

// Keys into a histogram of `bins`, in which a wave that meets one bin adds once: equal scores come in runs.
__device__ inline void count_key(bool mine, unsigned bin, unsigned *hist, int copies) {
  const u64 in = __ballot(mine);
  if (in == 0ull) return;
  const int first = __builtin_ctzll(in);
  if ((__ballot(bin == (unsigned)__builtin_amdgcn_readlane((int)bin, first)) & in) == in) {
    if ((int)(threadIdx.x & 63) == first) atomicAdd(&hist[bin * copies], (unsigned)__popcll(in));
  } else if (mine) {
    atomicAdd(&hist[bin * copies + (threadIdx.x & (copies - 1))], 1u);
  }
}

// The list of the keys that reach a bound which at least the larger k (>= 1) of the workgroup's n keys reach, or, where
// too many are equal, of exactly the k best; returns its length.  alike: the keys of a lane
// are much alike (neighbours in a row of the block map), so that the largest of them says little.  hist is zero.
// r: the ranges that hold the k-th keys, where all keys were counted (else left alone).
template <int UNITS, int CAP>
__device__ __forceinline__ int held_list(const Held<UNITS> &x, int n, const int (&ks)[2], bool alike, int base,
                                         TopShared &s, List<CAP> &l, Ranges &r) {
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), k = max(ks[0], ks[1]);
  // Keys of a unit into the histogram; all of them, or the largest of every four.
  auto count = [&](const u32x4a &y, bool all, unsigned *hist, int copies) {
    const unsigned m = max(max(y.x, y.y), max(y.z, y.w));
    if (m == 0u) return;
    const int b3 = bin_of(m, base), copy = lane & (copies - 1);
    if (!all) {
      atomicAdd(&hist[b3 * copies + copy], 1u);
      return;
    }
    const unsigned f = min(min(y.x, y.y), min(y.z, y.w));
    if (f != 0u && bin_of(f, base) == b3) {  // the four share their bin
      atomicAdd(&hist[b3 * copies + copy], 4u);
    } else {
      atomicAdd(&hist[bin_of(y.x, base) * copies + copy], 1u);
      if (y.y) atomicAdd(&hist[bin_of(y.y, base) * copies + copy], 1u);
      if (y.z) atomicAdd(&hist[bin_of(y.z, base) * copies + copy], 1u);
      if (y.w) atomicAdd(&hist[bin_of(y.w, base) * copies + copy], 1u);
    }
  };
  auto ranges = [&](bool fine) {  // of the k-th keys, from the bins picked
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (ks[q] > 0) {
        if (fine) bin_range<kFine>(s.pick[q].bin, base, r.lo[q], r.last[q]);
        else bin_range(s.pick[q].bin, base, r.lo[q], r.last[q]);
        r.lo[q] = max(r.lo[q], 1u);
        r.rank[q] = s.pick[q].rank; r.n[q] = s.pick[q].count;
      }
  };
  if (UNITS == 1 || n <= kDirect) {
    if (x.units > 0) {
      const int i = wv * kUnit + 4 * lane;
      if (i < n) *(u32x4a *)(l.key + i) = x.k[0];
#pragma unroll
      for (int j = 0; j < 4; ++j) l.at[i + j] = (uint16_t)(i + j);
      if (k < n) count(x.k[0], true, s.hist, kCopies);
    }
    __syncthreads();
    if (k < n) {
      block_find_kth<ST, kBins, kCopies>(s.hist, 2, (unsigned)max(ks[0], 0), (unsigned)max(ks[1], 0), s.pick, s.wsum);
      ranges(false);
    }
    return n;
  }
  if constexpr (UNITS > 1) {
    unsigned floor = 1u;
    auto reach = [&]() {  // keys that reach the bound, in the waves up to each
      int c = 0;
#pragma unroll
      for (int u = 0; u < UNITS; ++u)
        if (u < x.units)
          c += __popcll(__ballot(x.k[u].x >= floor)) + __popcll(__ballot(x.k[u].y >= floor)) +
               __popcll(__ballot(x.k[u].z >= floor)) + __popcll(__ballot(x.k[u].w >= floor));
      __syncthreads();
      if (lane == 0) s.wgt[wv] = (unsigned)c;
      __syncthreads();
      return wave_inclusive_sum(lane < SW ? s.wgt[lane] : 0u);
    };
    if (k < n) {
      const bool all = alike || 8 * k > n || n <= 2 * SW * kUnit;
      if (alike) {  // in the list's memory
        static_assert(kFineBins * kCopies <= CAP, "the histogram fits the list");
        for (int i = tid; i < kFineBins * kCopies / 4; i += ST) ((uint4 *)l.key)[i] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < UNITS; ++u)
          if (u < x.units) {
            const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (y[j]) atomicAdd(&l.key[fine_bin_of(y[j], base) * kCopies + (lane & (kCopies - 1))], 1u);
          }
        __syncthreads();
        block_find_kth<ST, kFineBins, kCopies>(l.key, 2, (unsigned)max(ks[0], 0), (unsigned)max(ks[1], 0), s.pick, s.wsum);
      } else {
#pragma unroll
        for (int u = 0; u < UNITS; ++u)
          if (u < x.units) count(x.k[u], all, s.hist, kCopies);
        __syncthreads();
        if (all) block_find_kth<ST, kBins, kCopies>(s.hist, 2, (unsigned)max(ks[0], 0), (unsigned)max(ks[1], 0), s.pick, s.wsum);
        else block_find_kth<ST, kBins, kCopies>(s.hist, 1, (unsigned)k, 0u, s.pick, s.wsum);
        zero_hist(s);
      }
      if (all) {
        ranges(alike);
        floor = ks[0] > 0 ? r.lo[0] : r.lo[1];
        if (ks[1] > 0) floor = min(floor, r.lo[1]);
      } else {
        unsigned last;
        bin_range(s.pick[0].bin, base, floor, last);
        floor = max(floor, 1u);
      }
    }
    unsigned sums = reach();
    int total = (int)__builtin_amdgcn_readlane(sums, SW - 1);
    unsigned need = 0u;  // not 0: of the keys equal to the bound only the first ones
    if (total > CAP) {
      r.n[0] = r.n[1] = 0u;
      // Runs of nearly equal scores: the range of the k-th key, ten bits at a time.
      unsigned lo = floor, last = 0xFFFFFFFFu, rank = (unsigned)k;
      do {
        const int shift = digit_shift(last - lo);
  #pragma unroll
        for (int u = 0; u < UNITS; ++u)
          if (u < x.units) {
            const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
  #pragma unroll 1
            for (int j = 0; j < 4; ++j) {
              const unsigned key = j == 0 ? y[0] : j == 1 ? y[1] : j == 2 ? y[2] : y[3];
              count_key(key >= lo && key <= last, (key - lo) >> shift, s.hist, 1);
            }
          }
        __syncthreads();
        block_find_kth<ST, kSubBins, 1>(s.hist, 1, rank, 0u, s.pick, s.wsum);
        lo += s.pick[0].bin << shift;
        last = min(last, lo + ((1u << shift) - 1u));
        rank = s.pick[0].rank;
        total = k - (int)rank + (int)s.pick[0].count;
        for (int i = tid; i < kSubBins; i += ST) s.hist[i] = 0u;
        __syncthreads();
      } while (total > CAP && lo != last);
      floor = lo;
      if (total > CAP) need = rank;
      sums = reach();
      total = need ? k : (int)__builtin_amdgcn_readlane(sums, SW - 1);
    }
    unsigned run = wv ? __builtin_amdgcn_readlane(sums, wv - 1) : 0u, erun = 0u;
    if (need) {  // keys above the bound and equal to it, before this wave
      int e = 0;
#pragma unroll
      for (int u = 0; u < UNITS; ++u)
        if (u < x.units)
          e += __popcll(__ballot(x.k[u].x == floor)) + __popcll(__ballot(x.k[u].y == floor)) +
               __popcll(__ballot(x.k[u].z == floor)) + __popcll(__ballot(x.k[u].w == floor));
      if (lane == 0) s.weq[wv] = (unsigned)e;
      __syncthreads();
      const unsigned es = wave_inclusive_sum(lane < SW ? s.weq[lane] : 0u);
      erun = wv ? __builtin_amdgcn_readlane(es, wv - 1) : 0u;
      run = run - erun + min(erun, need);
    }
    const int at0 = wv * wave_units(n) * kUnit + 4 * lane;
  #pragma unroll
    for (int u = 0; u < UNITS; ++u)
      if (u < x.units) {
        const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
        u64 in[4];
  #pragma unroll
        for (int j = 0; j < 4; ++j) in[j] = __ballot(y[j] >= floor);
        if (need) {  // uniform: cut the ties, in index order
          u64 eq[4];
          unsigned before = erun;
  #pragma unroll
          for (int j = 0; j < 4; ++j) {
            eq[j] = __ballot(y[j] == floor);
            before += __builtin_amdgcn_mbcnt_hi((unsigned)(eq[j] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)eq[j], 0u));
          }
  #pragma unroll
          for (int j = 0; j < 4; ++j) {
            in[j] &= ~__ballot(y[j] == floor && before >= need);
            before += (unsigned)((eq[j] >> lane) & 1ull);
            erun += (unsigned)__popcll(eq[j]);
          }
        }
        if ((in[0] | in[1] | in[2] | in[3]) == 0ull) continue;
        unsigned pos = run;
  #pragma unroll
        for (int j = 0; j < 4; ++j) {
          pos = __builtin_amdgcn_mbcnt_hi((unsigned)(in[j] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in[j], pos));
          run += (unsigned)__popcll(in[j]);
        }
  #pragma unroll
        for (int j = 0; j < 4; ++j)
          if ((in[j] >> lane) & 1ull) {
            l.key[pos] = y[j];
            l.at[pos] = (uint16_t)(at0 + kUnit * u + j);
            ++pos;
          }
      }
    __syncthreads();
    return total;
  }
}

// Of n <= kFew keys the one of rank `rank` from the top, its rank among its equals, and those: a wave, each lane counts the
// keys above its own.
__device__ inline void few_rank(TopShared &s, int q, unsigned n, unsigned rank) {
  const unsigned lane = threadIdx.x & 63, key = lane < n ? s.few[q][lane] : 0u;
  unsigned g = 0u, e = 0u;
  for (unsigned i = 0; i < n; ++i) {
    const unsigned o = (unsigned)__builtin_amdgcn_readlane((int)key, (int)i);
    g += o > key;
    e += o == key;
  }
  if (lane < n && g < rank && rank <= g + e) s.pick[q] = {key, rank - g, e};  // equal keys write the same
}

// The k-th largest of a list's n keys for two values of k, and how many of the keys equal to it are among the k.  A key
// is among the k best if it lies above thr, or is one of the first `need` that equal it.  k <= 0: none is; k >= n: all
// are.  hist is zero.  r.n[q] != 0: the range that holds the k[q]-th key is known.
struct Top { unsigned thr[2], need[2]; };
template <int CAP>
__device__ __forceinline__ Top list_top(const List<CAP> &l, int n, const int (&k)[2], int base, TopShared &s, Ranges &r) {
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  Top t;
  bool open[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    open[q] = k[q] > 0 && k[q] < n;
    t.thr[q] = k[q] > 0 ? 0u : 0xFFFFFFFFu;
    t.need[q] = 0u;
  }
  if (!open[0] && !open[1]) return t;
  if (tid < 2) s.n_few[tid] = 0u;
  if ((open[0] && r.n[0] == 0u) || (open[1] && r.n[1] == 0u)) {
    list_visit(l, n, [&](int, unsigned key) { count_key(key != 0u, (unsigned)bin_of(key, base), s.hist, kCopies); });
    __syncthreads();
    block_find_kth<ST, kBins, kCopies>(s.hist, 2, open[0] ? (unsigned)k[0] : 0u, open[1] ? (unsigned)k[1] : 0u, s.pick, s.wsum);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (open[q]) {
        bin_range(s.pick[q].bin, base, r.lo[q], r.last[q]);
        r.lo[q] = max(r.lo[q], 1u);
        r.rank[q] = s.pick[q].rank; r.n[q] = s.pick[q].count;
      }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (!open[q]) r.lo[q] = r.last[q] = r.n[q] = 0u;
  __syncthreads();
  while (r.open(0, kFew) || r.open(1, kFew)) {  // too many to rank them: ten bits at a time
    const bool want[2] = {r.open(0, kFew), r.open(1, kFew)};
    unsigned (*sub)[kSubWords] = (unsigned (*)[kSubWords])s.hist;
    __syncthreads();
    for (int i = tid; i < 2 * kSubWords; i += ST) s.hist[i] = 0u;
    __syncthreads();
    list_visit(l, n, [&](int, unsigned key) {
#pragma unroll 1
      for (int q = 0; q < 2; ++q) {
        const unsigned lo = q ? r.lo[1] : r.lo[0], last = q ? r.last[1] : r.last[0];
        if (q ? want[1] : want[0]) count_key(key >= lo && key <= last, (key - lo) >> digit_shift(last - lo), s.hist + q * kSubWords, 1);
      }
    });
    narrow_step<ST>(2, sub, s.pick, s.wsum, want, r);
  }
  const bool few[2] = {r.lo[0] != r.last[0], r.lo[1] != r.last[1]};
  if (few[0] || few[1]) {
    list_visit(l, n, [&](int, unsigned key) {
      if (few[0] && key - r.lo[0] <= r.last[0] - r.lo[0]) s.few[0][atomicAdd(&s.n_few[0], 1u)] = key;
      if (few[1] && key - r.lo[1] <= r.last[1] - r.lo[1]) s.few[1][atomicAdd(&s.n_few[1], 1u)] = key;
    });
    __syncthreads();
    if (wv == 0 && few[0]) few_rank(s, 0, r.n[0], r.rank[0]);
    if (wv == 1 && few[1]) few_rank(s, 1, r.n[1], r.rank[1]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (few[q]) { r.lo[q] = s.pick[q].bin; r.rank[q] = s.pick[q].rank; }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (open[q]) { t.thr[q] = r.lo[q]; t.need[q] = r.rank[q]; }
  return t;
}

// every(key): all keys.  place(key, value(entry of the list), position): the selected keys in order.  A wave takes a
// stretch of the list, four times 64 keys at a time, whose values are read together.
template <int CAP, class Every, class Value, class Place>
__device__ __forceinline__ void list_place(const List<CAP> &l, int n, unsigned thr, unsigned need, TopShared &s, Every every, Value value,
                                           Place place) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int len = (n + 64 * SW - 1) / (64 * SW) * 64, begin = wv * len, end = min(begin + len, n);
  int g = 0, e = 0;
#pragma unroll 1
  for (int i = begin + lane; i - lane < end; i += 64) {
    const unsigned key = i < end ? l.key[i] : 0u;
    every(key);
    g += __popcll(__ballot(key > thr));
    e += __popcll(__ballot(key == thr && key != 0u));
  }
  if (lane == 0) { s.wgt[wv] = (unsigned)g; s.weq[wv] = (unsigned)e; }
  __syncthreads();
  const unsigned gs = wave_inclusive_sum(lane < SW ? s.wgt[lane] : 0u), es = wave_inclusive_sum(lane < SW ? s.weq[lane] : 0u);
  unsigned erun = wv ? __builtin_amdgcn_readlane(es, wv - 1) : 0u;
  unsigned run = (wv ? __builtin_amdgcn_readlane(gs, wv - 1) : 0u) + min(erun, need);
#pragma unroll 1
  for (int i0 = begin + lane; i0 - lane < end; i0 += 256) {
    unsigned val[4], key[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + 64 * j;
      key[j] = i < end ? l.key[i] : 0u;
      val[j] = i < end ? value(i) : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool tie = key[j] == thr && key[j] != 0u;
      const u64 eq = __ballot(tie);
      const unsigned before = erun + __builtin_amdgcn_mbcnt_hi((unsigned)(eq >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)eq, 0u));
      const u64 sel = __ballot(key[j] > thr || (tie && before < need));
      erun += (unsigned)__popcll(eq);
      if ((sel >> lane) & 1ull)
        place(key[j], val[j], (int)__builtin_amdgcn_mbcnt_hi((unsigned)(sel >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)sel, run)));
      run += (unsigned)__popcll(sel);
    }
  }
}

// Row and column of candidate i of the block map's lower triangle, row by row: i = R (R - 1) / 2 + C, C < R.
__device__ inline void map_entry(unsigned i, int &R, int &C) {
  int r = (int)((1.f + sqrtf(8.f * (float)i + 1.f)) * 0.5f);  // i < 2^23: off by one at most
  if ((unsigned)r * (unsigned)(r - 1) / 2 > i) --r;
  if ((unsigned)r * (unsigned)(r + 1) / 2 <= i) ++r;
  R = r;
  C = (int)(i - (unsigned)r * (unsigned)(r - 1) / 2);
}

__device__ inline int held_total(const IdxArgs &a, int arr) { return arr == 2 ? a.sh.nb * (a.sh.nb - 1) / 2 : a.sh.N; }
// The best of an array's segments, one segment after the other: indices, or keys (key = true).
__device__ inline unsigned *top_of(const IdxArgs &a, int h, int arr, bool key) {
  unsigned *p = arr == 2 ? (key ? a.top_blk_key : a.top_blk) : (key ? a.top_vs_key : a.top_vs);
  return arr == 2 ? p + (size_t)h * a.seg_blk * a.cap_top_blk : p + ((size_t)h * 2 + arr) * a.seg_vs * a.cap_top_vs;
}

// Sum of the best of v or s over its segments; whole wave, the result in every lane.  BEFORE: the segments' results
// are those of a launch before, not of this one.
template <bool BEFORE, class X>
__device__ inline X result_load(const X *p) { return BEFORE ? *p : agent_load(p); }
template <bool BEFORE>
__device__ inline u64 held_best_sum(const IdxArgs &a, const IdxScratch *G, int arr) {
  if (a.seg_vs == 1) return result_load<BEFORE>(&G->psum[arr]);
  const int lane = threadIdx.x & 63, n = a.seg_vs * a.ksel[arr];
  const unsigned key = lane < n ? result_load<BEFORE>(&G->seg_best[arr][lane]) : 0u;
  int before = 0;  // keys of higher rank, the lower lane of equal ones first
  for (int i = 0; i < n; ++i) {
    const unsigned o = __builtin_amdgcn_readlane(key, i);
    before += o > key || (o == key && i < lane);
  }
  const u64 sum = wave_sum63(before < a.ksel[arr] ? fx30(key) : 0ull);
  return (u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)sum, 63) |
         (u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(sum >> 32), 63) << 32;
}
template <bool BEFORE>
__device__ inline int held_pattern(const IdxArgs &a, const IdxScratch *G) {
  u64 vt = 0, ct = 0;
  for (int i = 0; i < a.seg_vs; ++i) { vt += result_load<BEFORE>(&G->seg_vtot[i]); ct += result_load<BEFORE>(&G->seg_ct[i]); }
  return decide_pattern(a, vt, ct, held_best_sum<BEFORE>(a, G, 0), held_best_sum<BEFORE>(a, G, 1));
}

// grid (segments of v, of s and of the block map, from segment `first` on, Hq).
template <int UNITS>
__global__ __launch_bounds__(ST) void idx_top_kernel(IdxArgs a, int first) {
  __shared__ TopShared s;
  __shared__ List<(UNITS == 1 ? kDirect : kCap)> l;
  const int x0 = (int)blockIdx.x + first, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int arr = x0 < a.seg_vs ? 0 : x0 < 2 * a.seg_vs ? 1 : 2, seg = x0 - arr * a.seg_vs;
  const Shape &sh = a.sh;
  if (arr == 0 && seg == 0 && tid == 0 && a.ov.pat[h] >= 0) a.out.pattern[h] = a.ov.pat[h];
  if (!head_wants(a, h, arr == 2)) return;
  IdxScratch *G = a.scratch + h;
  const unsigned *src = array_of(a, arr, h);
  const int ns = n_sel(arr), nsegs = arr == 2 ? a.seg_blk : a.seg_vs, per = arr == 2 ? a.per_blk : a.per_vs;
  const int start = seg * per, n = min(held_total(a, arr) - start, per);
  const int units = wave_units(n), w0 = wv * units * kUnit;
  Held<UNITS> x;
  x.units = max(0, min(units, (n - w0 + kUnit - 1) / kUnit));
  // every key is on its way before the first is looked at
  if (arr < 2) {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      x.k[u] = u32x4a{0u, 0u, 0u, 0u};
      const int i = w0 + kUnit * u + 4 * lane;
      if (u < x.units && i < n) x.k[u] = *(const u32x4a *)(src + start + i);  // n is a multiple of 4
    }
  } else {
    // Four candidates of a lane lie in one row, or in the end of one and the start of the next: `skip` entries further on.
    int R, C;
    map_entry((unsigned)min(start + w0 + 4 * lane, held_total(a, 2) - 1), R, C);
    unsigned at = (unsigned)R * sh.nb + C;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      x.k[u] = u32x4a{0u, 0u, 0u, 0u};
      const int i = w0 + kUnit * u + 4 * lane;
      if (u >= x.units) continue;
      if (u > 0) {  // kUnit candidates on
        C += kUnit;
        at += kUnit;
        while (__any(C >= R)) {
          const bool next = C >= R;
          C -= next ? R : 0;
          at += next ? sh.nb - R : 0;
          R += next ? 1 : 0;
        }
      }
      if (i + 3 < n && R >= 4) {
        const int wrap = R - C, skip = sh.nb - R;
        const unsigned *q = src + at;
        if (wrap >= 4) {
          x.k[u] = *(const u32x4a *)q;
        } else {
          x.k[u].x = q[0];
          x.k[u].y = q[1 + (wrap > 1 ? 0 : skip)];
          x.k[u].z = q[2 + (wrap > 2 ? 0 : skip)];
          x.k[u].w = q[3 + skip];
        }
      } else if (i < n) {  // the first rows, and the end of the segment
        unsigned y[4] = {0u, 0u, 0u, 0u};
        int r = R, c = C;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (i + j < n) y[j] = src[(size_t)r * sh.nb + c];
          if (++c == r) { ++r; c = 0; }
        }
        x.k[u] = u32x4a{y[0], y[1], y[2], y[3]};
      }
    }
  }
  zero_hist(s);
  __syncthreads();
  u64 vt = 0, ct = 0;
  {
    const int sbnd = (int)min((long long)sh.sink * sh.b, (long long)sh.N), lb0 = max((sh.nb - sh.local) * sh.b, sbnd);
#pragma unroll
    for (int u = 0; u < UNITS; ++u)
      if (u < x.units) {
        const int i = w0 + kUnit * u + 4 * lane;
        unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
        if (arr == 2 && sh.row_norm) {
          int R, C;
          map_entry((unsigned)(start + i), R, C);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            y[j] = __float_as_uint(__uint_as_float(y[j]) * (float)(R + 1));
            if (++C == R) { ++R; C = 0; }
          }
        }
        if (arr == 0) {
          u64 z = 0;
          if (__any(max(max(y[0], y[1]), max(y[2], y[3])) >= 0x40800000u)) {  // 4 and more: beyond 32 bits
#pragma unroll
            for (int j = 0; j < 4; ++j) z += fx30(y[j]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) z += (u64)(unsigned)(__uint_as_float(y[j]) * 1073741824.f);
          }
          vt += z;  // nothing where there is no key
          const int c = start + i;  // the boundaries are multiples of a block
          if (c < sbnd || c >= lb0) ct += z;
        }
        x.k[u] = u32x4a{i < n ? raised(y[0]) : 0u, i + 1 < n ? raised(y[1]) : 0u, i + 2 < n ? raised(y[2]) : 0u, i + 3 < n ? raised(y[3]) : 0u};
      }
  }
  if (arr == 0) {
    vt = wave_sum63(vt);
    ct = wave_sum63(ct);
    if (lane == 63) { s.red[0][wv] = vt; s.red[1][wv] = ct; }
  }
  const int k[2] = {min(ksel(a, h, sel_of(arr, 0)), n), ns > 1 ? min(ksel(a, h, sel_of(arr, 1)), n) : 0};
  const int base = first_bin(a, arr), most = max(k[0], k[1]);
  if (most <= 0) return;  // the block map's selection only, and then nobody else waits
  Ranges r;
#pragma unroll
  for (int q = 0; q < 2; ++q) r.lo[q] = r.last[q] = r.n[q] = r.rank[q] = 0u;
  const int m = held_list(x, n, k, arr == 2, base, s, l, r);
  if (arr == 0 && tid < 2) {  // behind a barrier of the list
    u64 t = 0;
    for (int w = 0; w < SW; ++w) t += s.red[tid][w];
    agent_store(tid ? &G->seg_ct[seg] : &G->seg_vtot[seg], t);
  }
  const Top t = list_top(l, m, k, base, s, r);
  u64 ts = 0;  // of the probe: the keys above its threshold
  const unsigned thr_p = t.thr[0], ties = arr < 2 && k[0] < m ? thr_p - 1u : 0u;
  if (arr < 2) {
    __syncthreads();
    if (nsegs > 1) {  // its keys, for the sum over all segments
      unsigned *to = G->seg_best[arr] + seg * a.ksel[arr];
      if (tid == 0) s.n_few[0] = 0u;
      __syncthreads();
      list_visit(l, m, [&](int, unsigned key) {
        if (key > thr_p) agent_store(&to[atomicAdd(&s.n_few[0], 1u)], key - 1u);
      });
      __syncthreads();
      // the ties, and nothing behind the end of a short segment
      if (tid >= (int)s.n_few[0] && tid < a.ksel[arr]) agent_store(&to[tid], tid < k[0] ? ties : 0u);
    }
  }
  const int km = ns > 1 ? k[1] : k[0];
  const unsigned thr = km <= 0 ? ~0u : ns > 1 ? t.thr[1] : t.thr[0], need = km <= 0 ? 0u : ns > 1 ? t.need[1] : t.need[0];
  {
    const size_t at = (size_t)seg * min(ksel(a, h, sel_of(arr, ns - 1)), per);  // of every segment before: k, or all its keys
    unsigned *to = top_of(a, h, arr, false) + at, *to_key = nsegs > 1 ? top_of(a, h, arr, true) + at : nullptr;
    if (nsegs > 1 && km > 0 && tid == 0) G->seg_thr[arr][seg] = max(thr, 1u);
    list_place(l, m, thr, need, s,
               [&](unsigned key) {
                 if (arr < 2 && nsegs == 1 && key > thr_p) ts += fx30(key - 1u);
               },
               [&](int i) { return (unsigned)(start + l.at[i]); },
               [&](unsigned key, unsigned idx, int pos) {
                 to[pos] = idx;
                 if (to_key) to_key[pos] = key;
               });
  }
  if (arr < 2 && nsegs == 1) {
    ts = wave_sum63(ts);
    if (lane == 63) s.red[1][wv] = ts;
    __syncthreads();
    if (tid == 0) {
      u64 sum = (u64)t.need[0] * fx30(ties);
      for (int w = 0; w < SW; ++w) sum += s.red[1][w];
      agent_store(&G->psum[arr], sum);
    }
  }
  if (arr == 2 || !a.decide_here) return;
  // the block map waits for the patterns: the workgroup of v and s that arrives last decides
  if (!arrives_last(&G->ticket_vs, 2 * a.seg_vs)) return;
  if (a.ov.pat[h] < 0 && wv == 0) {
    const int pat = held_pattern<false>(a, G);
    if (lane == 0) a.out.pattern[h] = pat;
  }
}

constexpr int kSlice = 4 * ST;    // selected entries' candidates that a workgroup of the second launch writes
constexpr int kMapCopies = 4;     // copies of a bin in its histogram

// The k best of an array's segments' best, of which every thread holds four neighbours per slice: threshold, and how many
// of the keys equal to it are among them (all: 0).  floor: a bound that k keys reach.  hist and n_few are zero.
// The range of the k-th key is cut into 2048, and on into 1024, until a wave can compare the keys in it.
__device__ __forceinline__ void best_of_segments(const Held<kHeldUnits> &x, unsigned k, unsigned floor, unsigned *hist,
                                                 TopShared &s, unsigned &thr, unsigned &need) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  unsigned most = 0u;
#pragma unroll
  for (int u = 0; u < kHeldUnits; ++u)
    if (u < x.units) most = max(max(most, max(x.k[u].x, x.k[u].y)), max(x.k[u].z, x.k[u].w));
  most = wave_max(most);
  if (lane == 0) s.wgt[wv] = most;
  __syncthreads();
  unsigned lo = floor, last = wave_max(lane < SW ? s.wgt[lane] : 0u), rank = k, n;
  {
    const unsigned bits = 32 - __clz((int)(last - lo));  // __clz(0) = 32
    const int shift = bits > 11 ? (int)bits - 11 : 0;
#pragma unroll
    for (int u = 0; u < kHeldUnits; ++u)
      if (u < x.units) {
        const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (y[j] >= lo) atomicAdd(&hist[((y[j] - lo) >> shift) * kMapCopies + (lane & (kMapCopies - 1))], 1u);
      }
    __syncthreads();
    block_find_kth<ST, kBins, kMapCopies>(hist, 1, rank, 0u, s.pick, s.wsum);
    lo += s.pick[0].bin << shift;
    last = min(last, lo + ((1u << shift) - 1u));
    rank = s.pick[0].rank;
    n = s.pick[0].count;
  }
  while (n > (unsigned)kFew && lo != last) {
    const int shift = digit_shift(last - lo);
    __syncthreads();
    for (int i = threadIdx.x; i < kSubBins; i += ST) hist[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kHeldUnits; ++u)
      if (u < x.units) {
        const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) count_key(y[j] >= lo && y[j] <= last, (y[j] - lo) >> shift, hist, 1);
      }
    __syncthreads();
    block_find_kth<ST, kSubBins, 1>(hist, 1, rank, 0u, s.pick, s.wsum);
    lo += s.pick[0].bin << shift;
    last = min(last, lo + ((1u << shift) - 1u));
    rank = s.pick[0].rank;
    n = s.pick[0].count;
  }
  if (lo != last) {
#pragma unroll
    for (int u = 0; u < kHeldUnits; ++u)
      if (u < x.units) {
        const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
        if (min(min(y[0] - lo, y[1] - lo), min(y[2] - lo, y[3] - lo)) > last - lo) continue;  // as a rule
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (y[j] - lo <= last - lo) s.few[0][atomicAdd(&s.n_few[0], 1u)] = y[j];
      }
    __syncthreads();
    if (wv == 0) few_rank(s, 0, n, rank);
    __syncthreads();
    lo = s.pick[0].bin; rank = s.pick[0].rank; n = s.pick[0].count;
  }
  thr = lo;
  need = rank < n ? rank : 0u;
}

// grid (slices of the columns, of the diagonals, workgroups of the block CSR, Hq).  ROWS as T in idx_emit_kernel; SEGS: an
// array has several segments, the best of whose best every workgroup finds for itself; then it writes the selected entries of
// its slice.  What bounds it is the instructions that a workgroup spends on all segments' best, some 12 on each, and before
// them the time until the pattern is known and the keys are there (5 of 18 us).  With one workgroup per array and head,
// which made a list of the keys that reach the bound, 32 heads at 32K tokens (29500 best of four segments) took 28 us,
// like this 18; at 64K (19000 of four) 21 and 15.
//
// Diagonals at block granularity are written here where v and s are one segment, so that the selection has left the
// offsets in their final order.  Every workgroup that takes part forms their set first, so few do: at 32K tokens and 32
// heads with the per-row rule (64 workgroups a head, blocks of 64) 4, 8 and 16 of them take 11.0, 11.2 and 12.3 us, all 20.
constexpr int kDiagWgs = 8;
template <int ROWS, bool SEGS>
__global__ __launch_bounds__(ST) void idx_place_kernel(IdxArgs a) {
  __shared__ TopShared s;
  __shared__ int s_pat, s_at[ROWS > 0 ? kMaxNb + 1 : 1];
  __shared__ __attribute__((aligned(16))) unsigned s_hist[SEGS ? kBins * kMapCopies : 4];
  __shared__ uint16_t s_row[ROWS > 0 ? 1 : kSlice];  // rows of the selected entries of the slice
  __shared__ DiagRows<kSeg / 64> s_diag;             // v and s of one segment: up to kSeg / 64 row blocks
  const Shape &sh = a.sh;
  const int x0 = (int)blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, nb = sh.nb;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int place_vs = SEGS ? a.place_vs : 1;
  const int arr = x0 < place_vs ? 0 : x0 < 2 * place_vs ? 1 : 2, wg = x0 - arr * place_vs;
  const int nwg = arr == 2 ? (int)gridDim.x - 2 * place_vs : place_vs;
  const bool rows = arr == 2 && ROWS > 0;
  IdxScratch *G = a.scratch + h;
  const int nsegs = arr == 2 ? a.seg_blk : a.seg_vs, kq = ksel(a, h, arr == 2 ? 4 : arr + 2);
  const unsigned *from = top_of(a, h, arr, false);
  const int i0 = wg * kSlice + (SEGS ? 4 * tid : tid);  // the first of this thread's four entries of the slice
  int n = kq;
  if (SEGS && nsegs > 1) {  // the segments' best one after the other: of a segment kq, or all its keys
    const int per = arr == 2 ? a.per_blk : a.per_vs;
    n = (nsegs - 1) * min(kq, per) + min(kq, held_total(a, arr) - (nsegs - 1) * per);
  }
  int pat = a.ov.pat[h];
  if (pat < 0) {
    if (wv == 0) {
      const int p = a.decide_here ? a.out.pattern[h] : held_pattern<true>(a, G);
      if (tid == 0) {
        s_pat = p;
        if (x0 == 0) a.out.pattern[h] = p;
      }
    }
    __syncthreads();
    pat = s_pat;
  }
  pat = __builtin_amdgcn_readfirstlane(pat);
  const bool wanted = pat == (arr == 2 ? SA_BLOCK_CLUSTER : SA_INTERVAL_SLASH) && !rows;
  const int k = wanted ? kq : 0;
  Held<SEGS ? kHeldUnits : 1> x;
  unsigned floor = 1u;            // k keys of one segment reach its threshold
  unsigned begin = 0u, end = 0u;  // the first candidates of this slice and of the next
  if (wanted && arr == 2) {
    if (wg > 0 && wg * kSlice < n) begin = from[wg * kSlice];
    if ((wg + 1) * kSlice < n) end = from[(wg + 1) * kSlice];
  }
  // Up to three words behind the end are read: there is room (see index_scratch_bytes).
  unsigned own[4] = {0u, 0u, 0u, 0u};
  if (!SEGS && arr == 2) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (i0 + ST * j < k) own[j] = from[i0 + ST * j];
  } else if (SEGS && k > 0 && i0 < n) {
    const u32x4a y = *(const u32x4a *)(from + i0);
    own[0] = y.x; own[1] = y.y; own[2] = y.z; own[3] = y.w;
  }
  if constexpr (SEGS)
    if (k > 0 && nsegs > 1) {  // only now: all heads' keys to all their workgroups are more than the pattern takes to decide
      const unsigned *from_key = top_of(a, h, arr, true);
      x.units = (n + kSlice - 1) / kSlice;
#pragma unroll
      for (int u = 0; u < kHeldUnits; ++u) {
        x.k[u] = u32x4a{0u, 0u, 0u, 0u};
        const int i = kSlice * u + 4 * tid;
        if (i < n) x.k[u] = *(const u32x4a *)(from_key + i);
      }
      for (int i = 0; i < nsegs; ++i) floor = max(floor, G->seg_thr[arr][i]);
      for (int i = tid; i < kBins * kMapCopies / 4; i += ST) ((uint4 *)s_hist)[i] = make_uint4(0u, 0u, 0u, 0u);
      if (tid == 0) s.n_few[0] = 0u;
    }

  // This thread's entries: places in the index (-1: not selected); of the slice: selected entries before it and in it.
  int pos[4] = {-1, -1, -1, -1}, before = 0, count = 0;
  if (k > 0 && (!SEGS || nsegs <= 1)) {
    count = max(0, min(k - wg * kSlice, kSlice));
    before = min(wg * kSlice, k);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + (SEGS ? j : ST * j);
      pos[j] = i < k ? i : -1;
    }
  }
  if constexpr (SEGS)
    if (k > 0 && nsegs > 1) {
#pragma unroll
      for (int u = 0; u < kHeldUnits; ++u) {
        const int i = kSlice * u + 4 * tid;
        x.k[u].y = i + 1 < n ? x.k[u].y : 0u;
        x.k[u].z = i + 2 < n ? x.k[u].z : 0u;
        x.k[u].w = i + 3 < n ? x.k[u].w : 0u;
      }
      __syncthreads();
      unsigned thr, need;
      best_of_segments(x, (unsigned)k, floor, s_hist, s, thr, need);
      // In the order of the index: slice by slice, wave by wave.  Above the threshold (or, where all ties are taken, from it
      // on) and equal to it, in the slices before and in this one.
      const unsigned below = need ? thr : thr - 1u;
      int gt = 0, eq = 0, gt_own = 0, eq_own = 0;
      unsigned in = 0u, tie = 0u;
#pragma unroll
      for (int u = 0; u < kHeldUnits; ++u)
        if (u < x.units && u <= wg) {
          const unsigned y[4] = {x.k[u].x, x.k[u].y, x.k[u].z, x.k[u].w};
          int g = 0, e = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            g += __popcll(__ballot(y[j] > below));
            if (need) e += __popcll(__ballot(y[j] == thr));
          }
          if (u < wg) {
            gt += g; eq += e;
          } else {
            gt_own = g; eq_own = e;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              in |= (unsigned)(y[j] > below) << j;
              tie |= (unsigned)(need && y[j] == thr) << j;
            }
          }
        }
      if (lane == 0) { s.wgt[wv] = (unsigned)(gt + (gt_own << 16)); s.weq[wv] = (unsigned)(eq + (eq_own << 16)); }
      __syncthreads();
      const unsigned sg = lane < SW ? s.wgt[lane] : 0u, se = lane < SW ? s.weq[lane] : 0u;
      const unsigned g0 = wave_inclusive_sum(sg & 0xFFFFu), g1 = wave_inclusive_sum(sg >> 16);
      const unsigned e0 = wave_inclusive_sum(se & 0xFFFFu), e1 = wave_inclusive_sum(se >> 16);
      const unsigned ties0 = __builtin_amdgcn_readlane(e0, SW - 1), ties1 = ties0 + __builtin_amdgcn_readlane(e1, SW - 1);
      before = (int)(__builtin_amdgcn_readlane(g0, SW - 1) + min(ties0, need));
      count = (int)(__builtin_amdgcn_readlane(g0, SW - 1) + __builtin_amdgcn_readlane(g1, SW - 1) + min(ties1, need)) - before;
      unsigned gr = __builtin_amdgcn_readlane(g0, SW - 1) + (wv ? __builtin_amdgcn_readlane(g1, wv - 1) : 0u);
      unsigned er = ties0 + (wv ? __builtin_amdgcn_readlane(e1, wv - 1) : 0u);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u64 bg = __ballot((in >> j) & 1u), be = __ballot((tie >> j) & 1u);
        gr = __builtin_amdgcn_mbcnt_hi((unsigned)(bg >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bg, gr));
        er = __builtin_amdgcn_mbcnt_hi((unsigned)(be >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)be, er));
      }
      int at = (int)(gr + min(er, need));
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (((in >> j) & 1u) || (((tie >> j) & 1u) && er++ < need)) pos[j] = at++;
    }

  if (arr < 2) {
    const int width = arr ? sh.k_s : sh.k_v;
    int32_t *idx = (arr ? a.out.offs : a.out.cols) + (size_t)h * width;
    const bool aside = arr == 1 && sh.diag_blocks;  // the offsets become blocks: the list stays empty
    int32_t *dst = aside ? a.doffs + (size_t)h * width : idx;
    if constexpr (SEGS) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (pos[j] >= 0) dst[pos[j]] = (int)own[j];
    } else {
      for (int i = tid; i < k; i += ST) dst[i] = (int)from[i];
    }
    const int shown = aside ? 0 : k;
    for (int i = shown + wg * ST + tid; i < width; i += nwg * ST) idx[i] = -1;
    if (wg == 0 && tid == 0) {
      (arr ? a.out.n_offs : a.out.n_cols)[h] = shown;
    }
    return;
  }
  const bool diags = pat == SA_INTERVAL_SLASH && sh.diag_blocks && a.seg_vs == 1;  // the offsets are in order already
  const int wgs = diags ? min(nwg, kDiagWgs) : nwg;
  if (wg >= wgs) return;
  const int part = wg * SW + wv, nparts = wgs * SW, gtid = wg * ST + tid, gthreads = wgs * ST;
  int32_t *rp = a.out.rowptr + (size_t)h * (nb + 1);
  int32_t *bc = a.out.blkcols + (size_t)h * sh.cap_b;
  int total;
  if (pat == SA_BLOCK_CLUSTER && ROWS > 0) {
    total = emit_rows<ROWS == 0 ? 4 : ROWS, SW>(a, array_of(a, 2, h), part, nparts, rp, bc, s_at, s.wsum);
  } else if (pat == SA_BLOCK_CLUSTER) {
    // an entry of row R lands after the R diagonal blocks of the rows above
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (pos[j] >= 0) {
        int R, C;
        map_entry(own[j], R, C);
        bc[pos[j] + R] = C;
        s_row[pos[j] - before] = (uint16_t)R;
      }
    __syncthreads();
    // The rows behind that of the slice's first candidate, up to that of the next slice's first: no entry of another slice
    // decides where they start.
    int r0 = 0, r1 = nb, C;
    if (wg > 0) {
      if (wg * kSlice < n) map_entry(begin, r0, C);
      else r0 = nb;
    }
    if ((wg + 1) * kSlice < n) map_entry(end, r1, C);
    for (int r = r0 + 1 + tid; r <= r1; r += ST) {
      int lo = 0, hi = count;  // the first entry of the slice in row r or behind
      while (lo < hi) {
        const int m = (lo + hi) / 2;
        if ((int)s_row[m] < r) lo = m + 1;
        else hi = m;
      }
      const int at = before + lo + r;
      if (r < nb) rp[r] = at;
      bc[at - 1] = r - 1;
    }
    if (gtid == 0) rp[0] = 0;
    total = k + nb;
  } else if (diags) {
    total = diag_rows<SW>(a, top_of(a, h, 1, false), ksel(a, h, 3), part, nparts, rp, bc, s_diag, s.wsum);
  } else {
    total = emit_fixed(a, h, pat, part, nparts, gtid, gthreads, rp, bc);
  }
  if (gtid == 0) rp[nb] = total;
  for (int i = total + gtid; i < sh.cap_b; i += gthreads) bc[i] = -1;
}

// Interval-Slash heads when the selected diagonals are kept as whole blocks, where the launch before does not write
// them itself: the emission has left the offsets in doffs.  grid (workgroups, Hq)
__global__ __launch_bounds__(BT) void idx_diag_rows_kernel(IdxArgs a) {
  __shared__ DiagRows<kMaxNb> l;
  __shared__ unsigned s_wsum[2 * WPB];
  const Shape &sh = a.sh;
  const int h = blockIdx.y, nb = sh.nb;
  if (a.out.pattern[h] != SA_INTERVAL_SLASH) return;
  int32_t *rp = a.out.rowptr + (size_t)h * (nb + 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int total = diag_rows<WPB>(a, (const unsigned *)a.doffs + (size_t)h * sh.k_s, ksel(a, h, 3), (int)blockIdx.x * WPB + wv,
                                   (int)gridDim.x * WPB, rp, a.out.blkcols + (size_t)h * sh.cap_b, l, s_wsum);
  if (blockIdx.x == 0 && threadIdx.x == 0) rp[nb] = total;
}

// Boundary keys a list takes (8 bytes each).  The same memory holds the counts of a range whose keys are counted
// instead, kDense of 2 bytes per wave part; and a 128th of a large map, so that a range of many different keys fits
// where it holds no more (an eighth of an octave below the lowest bin does, unless the map is nearly flat there).
int list_cap_vs(const Shape &sh) {
  const int counts = (sh.N + WPB * kVsUnits * kUnit - 1) / (WPB * kVsUnits * kUnit) * WPB * (kDense * 2 / 8);
  return sh.N < kListVs ? sh.N : counts > kListVs ? counts : kListVs;
}
static_assert(kMaxBlkParts * (kDense * 2 / 8) <= kListBlk, "counts of all wave parts");
int list_cap_blk(const Shape &sh) {
  const long long all = (long long)sh.nb * (sh.nb - 1) / 2 + 1;
  return all < kListBlk ? (int)all : all / 128 > kListBlk ? (int)(all / 128) : kListBlk;
}
size_t round16(size_t x) { return (x + 15) & ~(size_t)15; }

// What idx_top_kernel leaves of every array.
struct HeldPlan { bool held; int seg_vs, seg_blk, per_vs, per_blk, cap_vs, cap_blk; };

// Arrays that workgroups hold: where a segment's best fit its list, and the best of all segments of an array, which a
// workgroup of the second launch takes again, are no more than it holds (and the best of all segments by the
// pattern rule no more than a wave).  Two launches against five, 32 heads: 18 us and 22 at 8K tokens, 30 and 40 at 16K,
// 44 and 55 at 32K with 7400 blocks selected below the diagonal, 32 and 53 with 2100, 41 and 60 at 64K.  A list
// of more than 8192 blocks loses: 38.6 and 39.3 with 9400 at 16K tokens, 43.4 and 40.4 with 12600, 47 and 41 with 15300,
// 42.5 and 36.8 with 8 heads.  The five launches follow the number of heads, the two hardly: with up to 8 heads, Block-
// Cluster ones among them, long lists of several segments already lose below that (4 heads at 32K tokens with 7368
// blocks 40.1 and 34.6, with 3428 33.3 and 34.5; at 64K with 4741 37.6 and 35.2), while without such heads, which the host
// cannot know, the two stay ahead (29.5 and 32.4, 28.5 and 33.2 with 5398).  So the line is not drawn by the heads.
HeldPlan held_arrays(const Shape &sh) {
  HeldPlan p;
  const long long ncand = sh.row_select ? 0 : (long long)sh.nb * (sh.nb - 1) / 2;
  auto split = [](long long n, int &segs, int &per) {  // even segments, in units
    segs = (int)((n + kSeg - 1) / kSeg);
    per = segs ? (int)(((n + segs - 1) / segs + kUnit - 1) / kUnit * kUnit) : 0;
  };
  split(sh.N, p.seg_vs, p.per_vs);
  split(ncand, p.seg_blk, p.per_blk);
  // the best k of a segment, or all its keys
  auto best = [](long long k, long long n, int per) { return (int)std::min<long long>(k < 1 ? 1 : k, std::min<long long>(n, per)); };
  const int kv = std::max(std::max(sh.k_v, sh.k_s), std::max(sh.probe_v, sh.probe_s));
  p.cap_vs = best(kv, sh.N, p.per_vs);
  p.cap_blk = ncand ? best((long long)sh.k_b - sh.nb, ncand, p.per_blk) : 0;
  p.held = p.cap_vs <= kCap && p.cap_blk <= kCap / 2 &&
           (p.seg_vs == 1 || (p.seg_vs <= kMaxSegs && (long long)p.seg_vs * p.cap_vs <= kSeg &&
                              (long long)p.seg_vs * std::max(sh.probe_v, sh.probe_s) <= 64)) &&
           (p.seg_blk <= 1 || (p.seg_blk <= kMaxMapSegs && (long long)p.seg_blk * p.cap_blk <= kSeg));
  return p;
}

// Words of idx_top_kernel's results: indices, and keys where there are several segments.
size_t top_words_vs(const Shape &sh, const HeldPlan &p) { return (size_t)sh.Hq * 2 * p.seg_vs * p.cap_vs; }
size_t top_words_blk(const Shape &sh, const HeldPlan &p) { return (size_t)sh.Hq * p.seg_blk * p.cap_blk; }

}  // namespace

size_t index_scratch_bytes(const Shape &sh) {
  const size_t H = (size_t)sh.Hq;
  const HeldPlan p = held_arrays(sh);
  const size_t keys = p.held ? ((p.seg_vs > 1 ? 2 : 1) * top_words_vs(sh, p) + (p.seg_blk > 1 ? 2 : 1) * top_words_blk(sh, p)) * 4
                             : H * 4 * list_cap_vs(sh) * 8 + H * list_cap_blk(sh) * 8;
  return H * sizeof(IdxScratch) + round16(keys) + 16 + (sh.diag_blocks ? round16(H * (size_t)sh.k_s * 4) : 0);
}

namespace {

IdxArgs index_args(const Shape &sh, const Workspace &ws, sa_scores in, const Override &ov, sa_index out,
                   const HeadBudget *hb, bool lazy) {
  IdxArgs a;
  a.v = (const unsigned *)in.v; a.s = (const unsigned *)in.s; a.blk = (const unsigned *)in.blk;
  a.scratch = (IdxScratch *)ws.idx;
  a.cap_vs = list_cap_vs(sh); a.cap_blk = list_cap_blk(sh);
  a.list_vs = (u64 *)(a.scratch + sh.Hq);
  a.list_blk = a.list_vs + (size_t)sh.Hq * 4 * a.cap_vs;
  a.doffs = (int32_t *)(a.list_blk + (size_t)sh.Hq * a.cap_blk);
  const HeldPlan held = held_arrays(sh);
  a.held = held.held;
  a.seg_vs = held.seg_vs; a.seg_blk = held.seg_blk; a.per_vs = held.per_vs; a.per_blk = held.per_blk;
  a.cap_top_vs = held.cap_vs; a.cap_top_blk = held.cap_blk;
  a.place_vs = (held.seg_vs * held.cap_vs + kSlice - 1) / kSlice;
  a.top_vs = a.top_vs_key = a.top_blk = a.top_blk_key = nullptr;
  if (held.held) {
    const size_t nv = top_words_vs(sh, held), nk = top_words_blk(sh, held);
    a.top_vs = (unsigned *)(a.scratch + sh.Hq);
    a.top_vs_key = a.top_vs + nv;
    a.top_blk = a.top_vs + (held.seg_vs > 1 ? 2 : 1) * nv;
    a.top_blk_key = a.top_blk + nk;
    a.doffs = (int32_t *)((char *)a.top_vs + round16(((held.seg_vs > 1 ? 2 : 1) * nv + (held.seg_blk > 1 ? 2 : 1) * nk) * 4));
  }
  a.sh = sh; a.ov = ov; a.out = out;
  // A wave takes 1024 keys of v or s; of the block map it takes 1024 entries or a 512th of the map,
  // whichever is more (a 256th at 128K tokens: 119 us for the index, a 512th 103; more, shorter waves
  // hide more latency until merging their histograms takes over).
  a.vpart = kVsUnits * kUnit;
  a.Pv = (sh.N + WPB * a.vpart - 1) / (WPB * a.vpart);
  const long long entries = (long long)sh.nb * sh.nb, units = (entries + kUnit - 1) / kUnit;
  long long per = (units + kMaxBlkParts - 1) / kMaxBlkParts;
  if (per < 4) per = 4;
  a.bpart = (int)per * kUnit;
  a.Pb = (int)(((units + per - 1) / per + WPB - 1) / WPB);
  // under the per-row rule a wave of the emission takes whole rows
  if (sh.row_select) a.Pb = (sh.nb + WPB - 1) / WPB < 128 ? (sh.nb + WPB - 1) / WPB : 128;
  // 1024 workgroups for up to 32 heads: where the launch has something to do, one or two heads need the chip too
  a.refine_vs = min(a.Pv, max(kRefineVs, 32 * kRefineVs / sh.Hq));
  a.refine_blk = min(a.Pb, max(kRefineBlk, 32 * kRefineBlk / sh.Hq));
  a.first = 0;
  a.decide_here = lazy || !held.held;
  a.nb_magic = ((1ull << 40) + sh.nb - 1) / sh.nb;
  a.wrap_magic = ((1u << 20) + sh.nb - 1) / sh.nb;
  const u64 all = (u64)sh.nb * (sh.nb + 1) / 2;
  a.share_magic = all == 1 ? 0 : ~0ull / all + 1;
  const long long ncand = (long long)sh.nb * (sh.nb - 1) / 2;
  long long kb = (long long)sh.k_b - sh.nb;
  if (kb < 0) kb = 0;
  if (kb > ncand) kb = ncand;
  a.ksel[0] = sh.probe_v < sh.N ? sh.probe_v : sh.N;
  a.ksel[1] = sh.probe_s < sh.N ? sh.probe_s : sh.N;
  a.ksel[2] = sh.k_v < sh.N ? sh.k_v : sh.N;
  a.ksel[3] = sh.k_s < sh.N ? sh.k_s : sh.N;
  a.ksel[4] = sh.row_select ? 0 : (int)kb;   // per-row rule: selected row by row while emitting
  a.decided = nullptr;
  a.hb = hb;
  // causal window entries, and those inside the Triangular region (sinks and band)
  long long sbnd = (long long)sh.sink * sh.b;
  if (sbnd > sh.N) sbnd = sh.N;
  long long lb0 = (long long)(sh.nb - sh.local) * sh.b;
  if (lb0 < sbnd) lb0 = sbnd;
  a.E = a.ET = 0;
  for (int i = 0; i < sh.w; ++i) {
    const long long qi1 = (long long)sh.N - sh.w + i + 1;
    a.E += (u64)qi1;
    a.ET += (u64)(qi1 < sbnd ? qi1 : sbnd);
    if (qi1 > lb0) a.ET += (u64)(qi1 - lb0);
  }
  static_assert(kMaxHeads == 128, "four mask words");
  for (int w = 0; w < kMaxHeads / 32; ++w) a.skip_vs[w] = a.skip_blk[w] = 0u;
  for (int h = 0; h < sh.Hq; ++h) {
    const int p = ov.pat[h];
    if (p >= 0 && p != SA_INTERVAL_SLASH) a.skip_vs[h >> 5] |= 1u << (h & 31);
    if (p >= 0 && p != SA_BLOCK_CLUSTER) a.skip_blk[h >> 5] |= 1u << (h & 31);
  }
  return a;
}

void launch_zero(const IdxArgs &a, hipStream_t st) {
  if (a.decide_here) idx_zero_kernel<<<dim3(a.sh.Hq, 3), BT, 0, st>>>(a.scratch);
}

// The passes before the emission, for the selections on v and s, the one on the block map, or both.
void launch_levels(IdxArgs a, bool vs, bool blk, hipStream_t st) {
  if (a.sh.row_select || (a.ksel[4] <= 0 && !a.hb)) blk = false;
  if (!vs && !blk) return;
  if (a.held) {
    const dim3 grid((vs ? 2 * a.seg_vs : 0) + (blk ? a.seg_blk : 0), a.sh.Hq);
    const int first = vs ? 0 : 2 * a.seg_vs;
    // a unit per wave and nothing to bound: a third of the code, which every call of a prompt's layers fetches anew
    // (4 heads at 4K tokens, in a layer: 1.2 us less)
    if (max(a.per_vs, a.per_blk) <= kDirect) idx_top_kernel<1><<<grid, ST, 0, st>>>(a, first);
    else idx_top_kernel<kHeldUnits><<<grid, ST, 0, st>>>(a, first);
    return;
  }
  a.first = vs ? 0 : 2 * a.Pv;
  const dim3 grid((vs ? 2 * a.Pv : 0) + (blk ? a.Pb : 0), a.sh.Hq);
  idx_hist_kernel<<<grid, BT, 0, st>>>(a);
  idx_refine_kernel<<<dim3((vs ? 2 * a.refine_vs : 0) + (blk ? a.refine_blk : 0), a.sh.Hq), BT, 0, st>>>(a);
  idx_count_kernel<<<grid, BT, 0, st>>>(a);
}

void launch_finish(const IdxArgs &a, hipStream_t st) {
  const dim3 grid(2 * a.Pv + a.Pb, a.sh.Hq);
  const bool one = a.seg_vs == 1 && a.seg_blk <= 1;
  const int place_blk = a.sh.row_select ? (a.sh.nb + SW - 1) / SW : max(1, (a.seg_blk * a.cap_top_blk + kSlice - 1) / kSlice);
  const dim3 place(2 * (one ? 1 : a.place_vs) + place_blk, a.sh.Hq);
  if (a.held && !a.sh.row_select) {
    if (one) idx_place_kernel<0, false><<<place, ST, 0, st>>>(a);
    else idx_place_kernel<0, true><<<place, ST, 0, st>>>(a);
  } else if (a.held && one) {
    static_assert(kSeg / 64 <= 1024, "rows of a map beside arrays of one segment");
    if (a.sh.nb <= 256) idx_place_kernel<4, false><<<place, ST, 0, st>>>(a);
    else idx_place_kernel<16, false><<<place, ST, 0, st>>>(a);
  } else if (a.held) {
    // the rows by themselves, in workgroups without a list's memory
    idx_place_kernel<0, true><<<dim3(2 * a.place_vs, a.sh.Hq), ST, 0, st>>>(a);
    IdxArgs b = a;
    b.first = 2 * a.Pv;
    const dim3 rows(a.Pb, a.sh.Hq);
    if (a.sh.nb <= 1024) idx_emit_kernel<16><<<rows, BT, 0, st>>>(b);
    else idx_emit_kernel<kMaxNb / 64><<<rows, BT, 0, st>>>(b);
  }
  else if (!a.sh.row_select) idx_emit_kernel<0><<<grid, BT, 0, st>>>(a);
  else if (a.sh.nb <= 256) idx_emit_kernel<4><<<grid, BT, 0, st>>>(a);
  else if (a.sh.nb <= 1024) idx_emit_kernel<16><<<grid, BT, 0, st>>>(a);
  else idx_emit_kernel<kMaxNb / 64><<<grid, BT, 0, st>>>(a);
  if (a.sh.diag_blocks && !(a.held && a.seg_vs == 1 && (one || !a.sh.row_select))) {  // not by the placing launch
    // a row per wave, up to 64 workgroups per head
    int P = (a.sh.nb + WPB - 1) / WPB;
    if (P > 64) P = 64;
    idx_diag_rows_kernel<<<dim3(P, a.sh.Hq), BT, 0, st>>>(a);
  }
}

}  // namespace

hipError_t launch_build_index(const Shape &sh, const Workspace &ws, sa_scores in, const Override &ov,
                              sa_index out, hipStream_t st, const HeadBudget *budgets) {
  const IdxArgs a = index_args(sh, ws, in, ov, out, budgets, false);
  launch_zero(a, st);
  launch_levels(a, true, true, st);
  launch_finish(a, st);
  return hipGetLastError();
}

// The same work in parts, for a caller that computes the block map only where it is needed: the
// selections on v and s, which write the patterns, then the selection on the block map and the
// emission.
hipError_t launch_index_stage(const Shape &sh, const Workspace &ws, sa_scores in, const Override &ov,
                              sa_index out, IndexStage stage, hipStream_t st) {
  IdxArgs a = index_args(sh, ws, in, ov, out, nullptr, true);
  a.decided = out.pattern;
  switch (stage) {
    case IndexStage::Zero: launch_zero(a, st); break;
    case IndexStage::ColumnsDiagonals: launch_levels(a, true, false, st); break;
    case IndexStage::Blocks: launch_levels(a, false, true, st); break;
    case IndexStage::Emit: launch_finish(a, st); break;
  }
  return hipGetLastError();
}

}  // namespace sa
