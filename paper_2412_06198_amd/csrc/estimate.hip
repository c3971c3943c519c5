// Pattern estimator for gfx950: two launches.
//
//  * window scores (Alg. 2 "Compute Dense Attention Scores" on the last w query
//    rows only, then SumRows -> v and SumDiagonals -> s).  The softmax of a
//    window row needs its maximum and normaliser over ALL keys before any
//    column can be summed, so K is streamed twice:
//      pass 1  S^T = K Qwin^T  (lane = query)  -> per-chunk (max, sum) partials,
//                                                 and the block means of K on the way
//      pass 2  S   = Qwin K^T  (lane = key)    -> normalised weights, column sums in
//                                                 the lane, diagonal sums by lane shifts
//    The 4 query heads of a GQA group ride on one K stream: wave w = head w.
//    K tiles go global -> LDS directly (global_load_lds_dwordx4).
//  * block map (Alg. 3 "Compute Blocked Representation"): a workgroup streams the
//    queries of 16 row blocks of a head, keeps their fp32 means in LDS, forms the
//    16-row strip of block logits on the matrix pipe, keeps it in registers, and
//    writes its causal row softmax once.
// The first launch is pass 1; the second holds the workgroups of pass 2 (bound by exp and vector
// ALU) spread among those of the block map (bound by the HBM stream of Q), which needs the K means of
// pass 1.  One stream, no events: with five launches on two streams 4 heads of 4096 tokens took 55 us,
// now 18; 32 heads at 10K, 16K, 32K, 64K and 128K tokens 59, 78, 122, 189 and 394, now 55, 65, 114, 183 and 364.
#include <algorithm>

#include "sa_internal.h"

namespace sa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr float kLog2e = 1.4426950408889634f;

__device__ inline float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// Block means are kept as two bf16 numbers, head + remainder (x = hi + lo to about 2^-17 |x|), so
// that the block map can form their products on the bf16 matrix pipe: hi.hi + hi.lo + lo.hi with
// fp32 accumulation differs from the fp32 product by about 2^-16 of it.
// A means array is laid out in the order in which the block map's matrix instruction wants its
// operands: per head ceil(nb/16) tiles of 16 rows, 8 KB each = [part: heads, remainders][k-step
// st = d/32][g = d%32/8][row n = R%16][8 elements], so that lane n + 16 g of a wave reads 16
// contiguous bytes of a contiguous 1 KB per instruction.  (With plain rows every quarter-wave
// touched 16 different cache lines, and the block map spent half its time in the L1's tag
// lookups.)  Rows past nb in the last tile are never written; nothing that is kept depends on them.
__device__ inline size_t means_tiles(int nb) { return (size_t)((nb + 15) / 16); }

__device__ inline void store_split(float *means_head, int R, int d, float x) {
  const __bf16 hi = (__bf16)x;
  const __bf16 lo = (__bf16)(x - (float)hi);
  uint16_t *tile = (uint16_t *)means_head + (size_t)(R >> 4) * 4096;
  const int o = (d >> 5) * 512 + ((d >> 3) & 3) * 128 + (R & 15) * 8 + (d & 7);
  tile[o] = __builtin_bit_cast(uint16_t, hi);
  tile[2048 + o] = __builtin_bit_cast(uint16_t, lo);
}

// ------------------------------------------------------------------ Q block means
constexpr int kMapWaves = 4;

// The means of the queries of a strip's row blocks first, first + step, ... (up to rows), split, into the
// strip's operand tile (LDS, laid out like the K means).  One wave.
__device__ __forceinline__ void strip_means(const uint16_t *__restrict__ src, const Shape &sh, uint16_t *tile, int first,
                                            int step, int rows) {
  const int lane = threadIdx.x & 63, cc = lane & 15, rg = lane >> 4;
  typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
  const int64_t q_rs = sh.q_rs;
  const uint16_t *lane_src = src + (size_t)rg * q_rs + cc * 8;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  // A batch is eight loads of four query rows; a row block has two or four.  The next batch is always
  // under way while one is summed, across the row blocks too: 8 to 16 KB in flight per wave.  Read once:
  // streaming (non-temporal) loads leave the caches to K, which the second window pass reads again, and
  // to the K means.
  const int per = sh.b >> 5, total = ((rows - first + step - 1) / step) * per;
  u32x4_t x0[8], x1[8];
  auto fetch = [&](u32x4_t (&x)[8], int it) {
    const int blk = first + step * (it / per), bt = it % per;
    const uint16_t *p = lane_src + ((size_t)blk * sh.b + 32 * bt) * q_rs;
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = __builtin_nontemporal_load((const u32x4_t *)(p + (size_t)(4 * k) * q_rs));
  };
  auto add = [&](const u32x4_t (&x)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t wds[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += bf16_bits_to_f32(wds[e]);
        acc[2 * e + 1] += __uint_as_float(wds[e] & 0xFFFF0000u);
      }
    }
  };
  if (total > 0) fetch(x0, 0);
#pragma unroll 1
  for (int it = 0; it < total; it += 2) {
    fetch(x1, it + 1);
    add(x0);
    if (it + 2 < total) fetch(x0, it + 2);
    add(x1);
    if ((it + 2) % per) continue;
    bf16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float s = acc[e];
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      s *= 1.0f / (float)sh.b;
      hi[e] = (__bf16)s;
      lo[e] = (__bf16)(s - (float)hi[e]);
      acc[e] = 0.f;
    }
    // elements 8 cc .. 8 cc + 7: k-step cc / 4, g = cc % 4
    uint16_t *dst = tile + (cc >> 2) * 512 + (cc & 3) * 128 + (first + step * (it / per)) * 8;
    if (rg == 0) *(bf16x8 *)dst = hi;
    if (rg == 1) *(bf16x8 *)(dst + 2048) = lo;
  }
}

// The L-th strip to be taken, the longest ones first.  Consecutive workgroup ids land on consecutive XCDs.
// While Hkv is a multiple of 8, KV head k is served by XCD k % 8 only, so that the L2 of an XCD holds the
// K means of one KV head at a time instead of all of them.
__device__ inline void strip_of(int L, const Shape &sh, int &strip, int &h) {
  const int nstrips = (sh.nb + 15) / 16;
  if (sh.Hkv % 8 == 0) {
    const int x = L & 7, s = L >> 3, hx = sh.Hq / 8;  // hx heads per XCD
    const int hl = s % hx;
    strip = nstrips - 1 - s / hx;
    h = (x + 8 * (hl / sh.g)) * sh.g + hl % sh.g;
  } else {
    strip = nstrips - 1 - L % nstrips;
    h = L / nstrips;
  }
}

// ------------------------------------------------------------------ window passes
// Q window fragments of one head: lane (q = lane%32, gg = lane/32) holds window row
// 32*qh + q, elements d = 16*ks + 8*gg .. +7.  The same registers serve as the B operand
// of K Q^T (pass 1) and as the A operand of Q K^T (pass 2).
__device__ inline void load_qwin(const uint16_t *__restrict__ Q, const Shape &sh, int hq, int lane,
                                 bf16x8 (&qf)[2][8]) {
  const int q = lane & 31, gg = lane >> 5;
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    int i = 32 * qh + q;
    if (i >= sh.w) i = sh.w - 1;  // rows past the window are computed and ignored
    const uint16_t *row = Q + (size_t)hq * sh.q_hs + (size_t)(sh.N - sh.w + i) * sh.q_rs;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[qh][ks] = *(const bf16x8 *)(row + 16 * ks + 8 * gg);
  }
}

// A K tile is 64 keys x 256 B in LDS, the 16-byte chunks of a row XOR-swizzled with the row
// number (chunk c of row r sits at chunk c ^ (r & 15)): the b128 fragment reads of 32 rows are
// conflict-free without padding.  The swizzle is applied on the global side of the copy: the
// lane that owns physical chunk pc of row r fetches logical chunk pc ^ (r & 15).  One
// instruction moves four rows (16 bytes per lane, LDS address = M0 + 16*lane); wave w moves rows
// 4w..4w+3 (+16n, n = 0..3).
#define SA_DMA16(gptr, voff, ldsb)                                                                    \
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(gptr), \
               "s"(ldsb)                                                                              \
               : "memory")

// The window passes keep kStages K tiles in LDS: tile t is multiplied while the copies of the
// next kStages - 2 tiles are in flight (one tile of lead per workgroup left the passes waiting for
// memory latency most of the time: a workgroup only had 16 KB on its way).
constexpr int kStages = 3;

// Wait until this wave's copies of tile t have landed while up to `ahead` younger tiles (four copy
// instructions each) may still be in flight.  Vector memory operations of a kind retire in issue
// order, so at most 4 * ahead outstanding operations means the older copies are complete.
__device__ inline void wait_tile(int ahead) {
  if (ahead >= 2) __builtin_amdgcn_s_waitcnt(0x0F78);       // vmcnt(8)
  else if (ahead == 1) __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4)
  else __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
}

struct KTileCopy {
  unsigned voff;   // per-lane byte offset inside a 16-row slab of K
  unsigned lds0;   // LDS byte address of this wave's first row in buffer 0
  size_t row16;    // elements between the rows of consecutive instructions
  __device__ inline void init(const uint16_t *ks0, int wv, int lane, int64_t kv_rs) {
    const int rl = 4 * wv + (lane >> 4);
    voff = (unsigned)(rl * (int)kv_rs * 2 + (((lane & 15) ^ rl) << 4));
    lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const uint16_t *)ks0 + 4 * wv * 256;
    row16 = 16 * (size_t)kv_rs;
  }
  __device__ inline void issue(const uint16_t *kb, int buf) const {
    const unsigned l = lds0 + buf * (64 * 256);
    SA_DMA16(kb, voff, l);
    SA_DMA16(kb + row16, voff, l + 16 * 256);
    SA_DMA16(kb + 2 * row16, voff, l + 32 * 256);
    SA_DMA16(kb + 3 * row16, voff, l + 48 * 256);
  }
};

// Fragment addresses of a swizzled tile: rows 32 kh + q, logical chunk 2 ks + gg.  One per-lane address
// per ks, shared by both halves of the tile and, with the tile's buffer added, by all buffers.
typedef const __attribute__((address_space(3))) bf16x8 lds_frag;
struct KFrags {
  unsigned at[8];
  __device__ inline void init(const uint16_t *ks0, int lane) {
    const int q = lane & 31, gg = lane >> 5;
    const unsigned base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const uint16_t *)ks0 + (unsigned)(q * 256);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) at[ks] = base + (unsigned)((((2 * ks + gg) ^ (q & 15)) & 15) << 4);
  }
};

// Products of one 32-key half of a tile with the two halves of the window (pass 1: K is the A operand).  The
// fragments go through a ring of four registers: the read of fragment i + 4 follows the products with
// fragment i.
__device__ inline void half_tile(const unsigned (&at)[8], int kh, const bf16x8 (&qf)[2][8], f32x16 (&acc)[2]) {
#pragma unroll
  for (int qh = 0; qh < 2; ++qh)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[qh][r] = 0.f;
  bf16x8 kf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) kf[ks] = *(lds_frag *)(uintptr_t)(at[ks] + kh * 32 * 256);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
    for (int qh = 0; qh < 2; ++qh)
      acc[qh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks & 3], qf[qh][ks], acc[qh], 0, 0, 0);
    if (ks + 4 < 8) kf[ks & 3] = *(lds_frag *)(uintptr_t)(at[ks + 4] + kh * 32 * 256);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
}

// Products of 32 window rows with both halves of a tile (pass 2: K is the B operand), likewise.
__device__ inline void rows_tile(const unsigned (&at)[8], const bf16x8 (&qf)[8], f32x16 (&acc)[2]) {
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[kh][r] = 0.f;
  bf16x8 kf[4];
  auto frag = [&](int i) { return *(lds_frag *)(uintptr_t)(at[i >> 1] + (i & 1) * 32 * 256); };
#pragma unroll
  for (int i = 0; i < 4; ++i) kf[i] = frag(i);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[i >> 1], kf[i & 3], acc[i & 1], 0, 0, 0);
    if (i + 4 < 16) kf[i & 3] = frag(i + 4);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
}

// The head of a workgroup's four that wave wv takes.  Where there are fewer (g < 4, or the last ones of a group), the waves
// without one only copy; workgroups that share a compute unit (256 apart) leave others without, since the wave's
// number decides on its SIMD.  With those waves repeating the first head's work, 8 heads without groups took 215 us at 128K
// tokens, 71.6 at 32K and 45.7 at 16K, like this 184, 69.2 and 42.6; 4 heads 122.6, 51.4 and (4K) 18.1, now 115.3,
// 49.2 and 18.1.
__device__ inline int head_wave(int L, int wv) { return (wv + (L >> 8)) & 3; }

// pass 1, workgroup L of nchunks * Hkv * ceil(g/4), 256 threads.
__device__ inline void window_stats(int L, uint16_t (*Ks)[64 * 128], const uint16_t *__restrict__ Q,
                                    const uint16_t *__restrict__ K, const Shape &sh, float c,
                                    float2 *__restrict__ part, float *__restrict__ s_out,
                                    float *__restrict__ kblk) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 31, gg = lane >> 5;
  const int chunk = L % sh.nchunks, kvh = L / sh.nchunks % sh.Hkv, z0 = L / (sh.nchunks * sh.Hkv);
  const int hsub = 4 * z0 + head_wave(L, wv);
  const bool head_ok = hsub < sh.g;
  const int hq = kvh * sh.g + (head_ok ? hsub : 0);
  const int jc0 = chunk * sh.chunk;
  const int jc1 = min(jc0 + sh.chunk, sh.N);
  const int nt = (jc1 - jc0) >> 6;  // N is a multiple of 64: whole tiles only
  const uint16_t *Kh = K + (size_t)kvh * sh.kv_hs + (size_t)jc0 * sh.kv_rs;
  const bool do_means = z0 == 0;

  KTileCopy cp;
  cp.init(&Ks[0][0], wv, lane, sh.kv_rs);
  cp.issue(Kh, 0);

  // the slash scores are accumulated with atomics in pass 2: clear this chunk's share now
  if (head_ok)
    for (int j = jc0 + lane; j < jc1; j += 64) s_out[(size_t)hq * sh.N + j] = 0.f;

  bf16x8 qf[2][8];
  load_qwin(Q, sh, hq, lane, qf);
#pragma unroll
  for (int s2 = 1; s2 < kStages - 1; ++s2)
    if (s2 < nt) cp.issue(Kh + (size_t)s2 * 64 * sh.kv_rs, s2);
  float m[2] = {-INFINITY, -INFINITY}, z[2] = {0.f, 0.f};
  KFrags kfr;
  kfr.init(&Ks[0][0], lane);

  // Block sums of K on the matrix pipe: ones (16 x 32 keys) times K (32 keys x 16 elements) in
  // v_mfma_f32_16x16x32_bf16 leaves the sum of the 32 keys in every row; wave w takes elements 32 w ..
  // 32 w + 31.  Its B operand, lane (n = element, group lane/16) = keys 8 group .. + 7, is K transposed,
  // which two transposing reads of four keys each deliver.  Their source lane r = lane % 16 supplies
  // the 8-byte piece (key r/4, elements 4(r%4)..+3); the piece of key row y sits in chunk
  // (2 blk16 + (r%4)/2) ^ (y & 15).  (Adding the rows on the vector ALU took a fifth of this pass, which
  // is bound there.)
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const int tpb = sh.b >> 6;  // tiles per block: 1 or 2
  f32x4 ksum[2] = {};
  unsigned tr[2];             // byte offsets of the two reads of element block 2 wv, key step 0
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int r = lane & 15, y = 8 * (lane >> 4) + 4 * p + (r >> 2);
    tr[p] = (unsigned)(y * 256 + (((4 * wv + ((r & 3) >> 1)) ^ (y & 15)) << 4) + ((r & 1) << 3));
  }
  const __bf16 one = (__bf16)1.f;
  const bf16x8 ones = {one, one, one, one, one, one, one, one};

  for (int t = 0; t < nt; ++t) {
    const int cur = t % kStages;
    wait_tile(min(nt - 1 - t, kStages - 2));  // this wave's share of tile t has landed
    __syncthreads();                          // ... and everybody's; tile t-1 has been read by all
    if (t + kStages - 1 < nt)
      cp.issue(Kh + (size_t)(t + kStages - 1) * 64 * sh.kv_rs, (t + kStages - 1) % kStages);
    const uint16_t *Kt = Ks[cur];
    const int j0 = jc0 + 64 * t;

    if (do_means) {
#pragma unroll
      for (int eb = 0; eb < 2; ++eb)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const char *base = (const char *)Kt + ks * 32 * 256;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(base + (tr[0] ^ (unsigned)(eb << 5))));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(base + (tr[1] ^ (unsigned)(eb << 5))));
          const s16x8 kt = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          ksum[eb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, kt), ksum[eb], 0, 0, 0);
        }
      if ((t + 1) % tpb == 0) {  // every lane of a column holds its sum: lanes 0..15 write one block, 16..31 the other
        if (lane < 32)
          store_split(kblk + (size_t)kvh * means_tiles(sh.nb) * 2048, j0 / sh.b, 32 * wv + lane,
                      (lane < 16 ? ksum[0][0] : ksum[1][0]) * (1.0f / (float)sh.b));
        ksum[0] = ksum[1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }

    if (!head_ok) continue;
    // One 32-key half of the tile at a time: its scores are reduced to (max, sum) before the next
    // half is multiplied, so only 32 accumulator registers are live (three waves per SIMD fit).
    // lane = query 32qh+q ; acc[qh][r] <-> key j0 + 32kh + 8(r/4) + 4gg + r%4
    const bool tail = j0 + 63 > sh.N - sh.w;  // causal masking only in the last tile of the sequence
    unsigned at[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) at[ks] = kfr.at[ks] + cur * (64 * 256);
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {
      f32x16 acc[2];  // [query half]
      half_tile(at, kh, qf, acc);
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        if (tail) {
          // last visible key of this window row, relative to the lane's first key of the half
          const int lim = sh.N - sh.w + 32 * qh + q - (j0 + 32 * kh + 4 * gg);
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (8 * (r / 4) + (r % 4) > lim) acc[qh][r] = -INFINITY;
        }
        // The reference of a row moves when a logit lies 8 octaves or more above it.  A sum below 2^8 shows
        // that none does, so the sum is taken without looking for a maximum, and only a larger one (or a row
        // without a reference yet) has the half tile reduced again.  A bound at the end of the fp32 range
        // would serve as well against overflow but not for precision: the exponents and log2(sum) would
        // carry the distance to the first keys, and its rounding (a row 29 octaves above them: weights off by
        // 1.2e-6 instead of 1e-7).  It is not faster either: 32K tokens, 32 heads 109.9 us with 2^60, 110.1 with 2^8.
        auto sum_with = [&](float m_ref) {
          float sum = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[qh][r], c, -m_ref));
          return sum;
        };
        float sum = sum_with(m[qh]);
        if (__any(!(sum < 0x1p8f))) {  // also m = -inf (no key seen yet): the sum is then inf or nan
          float tmax = -INFINITY;
#pragma unroll
          for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, acc[qh][r]);
          const float m_new = fmaxf(m[qh], tmax * c);
          if (m_new != -INFINITY) z[qh] *= __builtin_amdgcn_exp2f(m[qh] - m_new);
          m[qh] = m_new;
          sum = sum_with(m_new == -INFINITY ? 0.f : m_new);
        }
        z[qh] += sum;
      }
    }
  }
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const float mp = __shfl_xor(m[qh], 32), zp = __shfl_xor(z[qh], 32);
    const float M = fmaxf(m[qh], mp);
    float Z = 0.f;
    if (M != -INFINITY) {
      if (m[qh] != -INFINITY) Z += z[qh] * __builtin_amdgcn_exp2f(m[qh] - M);
      if (mp != -INFINITY) Z += zp * __builtin_amdgcn_exp2f(mp - M);
    }
    const int i = 32 * qh + q;
    if (head_ok && gg == 0 && i < sh.w)
      part[((size_t)hq * sh.nchunks + chunk) * kWin + i] = make_float2(M, Z);
  }
}

// combine the per-chunk partials into bias[i] = max_i + log2(sum_i) (log2 domain), so that a
// window weight is exp2(logit * scale * log2e - bias).  Rows past the window get +inf (weight 0).
// grid (Hq, 4), 1024 threads = 64 chunk slices x 16 window rows.
__global__ __launch_bounds__(1024) void window_stats_reduce_kernel(const float2 *__restrict__ part,
                                                                  int nchunks, int w,
                                                                  float *__restrict__ bias) {
  __shared__ float red[64][17];
  const int hq = blockIdx.x, il = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int i = 16 * blockIdx.y + il;
  const float2 *p = part + (size_t)hq * nchunks * kWin + i;
  float M = -INFINITY;
  if (i < w)
    for (int cidx = sl; cidx < nchunks; cidx += 64) M = fmaxf(M, p[(size_t)cidx * kWin].x);
  red[sl][il] = M;
  __syncthreads();
  float Mt = -INFINITY;
#pragma unroll 16
  for (int k = 0; k < 64; ++k) Mt = fmaxf(Mt, red[k][il]);
  __syncthreads();
  float Z = 0.f;
  if (i < w)
    for (int cidx = sl; cidx < nchunks; cidx += 64) {
      const float2 e = p[(size_t)cidx * kWin];
      if (e.x != -INFINITY) Z += e.y * __builtin_amdgcn_exp2f(e.x - Mt);
    }
  red[sl][il] = Z;
  __syncthreads();
  if (sl == 0) {
    float Zt = 0.f;
#pragma unroll 16
    for (int k = 0; k < 64; ++k) Zt += red[k][il];
    bias[(size_t)hq * kWin + i] = i < w ? Mt + __builtin_amdgcn_logf(Zt) : INFINITY;  // v_log_f32 = log2
  }
}

// Lane shifts of a whole wavefront (DPP wave_shl:1 / wave_shr:1): lane l takes lane l+1, the last one 0.
__device__ inline float wave_shl1(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, true));
}
// Lane l takes x of lane l - 1; lane 0 keeps `old`.
__device__ inline float wave_shr1_into(float old, float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x138, 0xF, 0xF, false));
}

// Weights of one 64-key tile for 32 window rows (pass 2).  After the MFMAs lane l holds key 32kh + l%32
// and register r of acc[kh] window row 32qh + 8(r/4) + 4(l/32) + r%4.  v_permlane32_swap of
// the two key halves turns that into "register = one window row, lane = key 0..63": the row
// constants are wave-uniform and the column sum stays in the lane.
//
// Diagonal sums without LDS: the rows are taken in DESCENDING order, step tau = 64*tile + 63 - i,
// so that the offset of element (i, lane l) is A - (tau + l) for a chunk constant A.  `run`
// shifts one lane down per step (run[l] <- run[l+1] + weight): a slot then collects exactly one
// offset over 64 consecutive steps, is complete when it reaches lane 0, and `done` picks it up
// there while shifting the other way, so that after the 64 rows of a tile done[l] is the finished
// sum of offset (N - w - j0) + l.  Sums that straddle a chunk boundary are the only partial ones.
template <bool TAIL>
__device__ inline float scores_rows(const f32x16 (&acc)[2], int qh, const float (&bias)[kWin], float c,
                                    int lim0, float &run, float &done) {
  float colsum = 0.f;
  // `done` trails `run` by one step: by then the previous `run` is dead, and its register can become the
  // shifted `done` (lane 0, which the shift leaves alone, holds the finished sum) in one instruction
  bool first = true;
#pragma unroll
  for (int rq = 3; rq >= 0; --rq) {
    float x[2][4];
#pragma unroll
    for (int rm = 0; rm < 4; ++rm) {
      const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[0][4 * rq + rm]),
                                                       __float_as_uint(acc[1][4 * rq + rm]), false, false);
      x[0][rm] = __uint_as_float(pr[0]);
      x[1][rm] = __uint_as_float(pr[1]);
    }
#pragma unroll
    for (int u = 1; u >= 0; --u)
#pragma unroll
      for (int rm = 3; rm >= 0; --rm) {
        const int i = 32 * qh + 8 * rq + 4 * u + rm;
        float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x[u][rm], c, -bias[i]));
        if (TAIL) e = (lim0 + i >= 0) ? e : 0.f;  // key j0 + lane visible to row i iff j <= N-w+i
        colsum += e;
        const float next = wave_shl1(run) + e;
        if (!first) done = wave_shr1_into(run, done);
        first = false;
        run = next;
      }
  }
  done = wave_shr1_into(run, done);
  return colsum;
}

// The row constants of a window from the per-chunk partials, one row per lane: max + log2(sum), in the
// log2 domain, so that a window weight is exp2(logit * scale * log2e - bias).  Rows past the window
// get +inf (weight 0).
__device__ inline float window_bias(const float2 *__restrict__ part, int nchunks, int w, int lane) {
  float M = -INFINITY, Z = 0.f;
  for (int c0 = 0; c0 < nchunks; c0 += 16) {
    float2 e[16];
#pragma unroll
    for (int k = 0; k < 16; ++k)  // past the end: the last chunk again, its sum dropped
      e[k] = part[(size_t)min(c0 + k, nchunks - 1) * kWin + min(lane, w - 1)];
    float Mn = M;
#pragma unroll
    for (int k = 0; k < 16; ++k) Mn = fmaxf(Mn, e[k].x);
    const float ref = Mn == -INFINITY ? 0.f : Mn;
    Z *= __builtin_amdgcn_exp2f(M - ref);
#pragma unroll
    for (int k = 0; k < 16; ++k)
      Z = __builtin_fmaf(c0 + k < nchunks ? e[k].y : 0.f, __builtin_amdgcn_exp2f(e[k].x - ref), Z);
    M = Mn;
  }
  return lane < w ? M + __builtin_amdgcn_logf(Z) : INFINITY;  // v_log_f32 = log2
}

// pass 2, workgroup L of nchunks * Hkv * ceil(g/4), 256 threads.  Chunks are walked in the reverse order
// of pass 1, so that the most recently streamed part of K is re-read first.  bias_g: the row constants
// if a launch before has formed them, else nullptr.
__device__ inline void window_scores(int L, uint16_t (*Ks)[64 * 128], const uint16_t *__restrict__ Q,
                                     const uint16_t *__restrict__ K, const Shape &sh, float c,
                                     const float2 *__restrict__ part, const float *__restrict__ bias_g,
                                     float *__restrict__ v_out, float *__restrict__ s_out) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 31, gg = lane >> 5;
  const int chunk = sh.nchunks - 1 - L % sh.nchunks, rest = L / sh.nchunks;
  const int kvh = sh.Hkv - 1 - rest % sh.Hkv;
  const int hsub = 4 * (rest / sh.Hkv) + head_wave(L, wv);
  const bool head_ok = hsub < sh.g;
  const int hq = kvh * sh.g + (head_ok ? hsub : 0);
  const int jc0 = chunk * sh.chunk;
  const int jc1 = min(jc0 + sh.chunk, sh.N);
  const int nt = (jc1 - jc0) >> 6;
  const uint16_t *Kh = K + (size_t)kvh * sh.kv_hs + (size_t)jc0 * sh.kv_rs;

  KTileCopy cp;
  cp.init(&Ks[0][0], wv, lane, sh.kv_rs);
  cp.issue(Kh, 0);

  bf16x8 qf[2][8];
  load_qwin(Q, sh, hq, lane, qf);
  const float row_bias = bias_g ? bias_g[(size_t)hq * kWin + lane]
                                : window_bias(part + (size_t)hq * sh.nchunks * kWin, sh.nchunks, sh.w, lane);
  float bias[kWin];  // wave-uniform: lives in scalar registers
#pragma unroll
  for (int i = 0; i < kWin; ++i)
    bias[i] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(row_bias), i));
#pragma unroll
  for (int s2 = 1; s2 < kStages - 1; ++s2)
    if (s2 < nt) cp.issue(Kh + (size_t)s2 * 64 * sh.kv_rs, s2);
  KFrags kfr;
  kfr.init(&Ks[0][0], lane);
  float *srow = s_out + (size_t)hq * sh.N;
  float run = 0.f, done = 0.f;
  float cv = c;  // in a vector register: an FMA takes only one scalar operand, and that is the row's bias
  asm volatile("" : "+v"(cv));

  for (int t = 0; t < nt; ++t) {
    const int cur = t % kStages;
    // the stores of the previous tiles count like the copies: they only make the wait longer
    wait_tile(min(nt - 1 - t, kStages - 2));
    __syncthreads();
    if (t + kStages - 1 < nt)
      cp.issue(Kh + (size_t)(t + kStages - 1) * 64 * sh.kv_rs, (t + kStages - 1) % kStages);
    if (!head_ok) continue;
    const int j0 = jc0 + 64 * t;

    unsigned at[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) at[ks] = kfr.at[ks] + cur * (64 * 256);
    // the upper 32 window rows first (the diagonal sums take the rows in descending order), by themselves:
    // reading the K fragments twice costs less than the registers of all 64 rows, with which only two
    // workgroups fit a compute unit
    float colsum = 0.f;
#pragma unroll
    for (int qh = 1; qh >= 0; --qh) {
      f32x16 acc[2];  // [key half]
      rows_tile(at, qf[qh], acc);
      if (j0 + 63 > sh.N - sh.w)
        colsum += scores_rows<true>(acc, qh, bias, cv, sh.N - sh.w - j0 - lane, run, done);
      else
        colsum += scores_rows<false>(acc, qh, bias, cv, 0, run, done);
    }
    {
      v_out[(size_t)hq * sh.N + j0 + lane] = colsum;
      // The first tile's sums lack the previous chunk's rows (all but lane 0): they are added to
      // the zeroed slot, as is that chunk's remainder below.  Every offset so receives at most
      // two partial sums, so the result does not depend on the order of the atomics.
      const int o = sh.N - sh.w - j0 + lane;
      if (o < sh.N) {
        if (t == 0) atomicAdd(&srow[o], done);
        else srow[o] = done;
      }
    }
  }
  // what is left in `run` belongs to the next chunk's first tile: lane l holds offset
  // (N - w - jc1) + 64 - l, l = 1..63
  if (head_ok && lane > 0) {
    const int o = sh.N - sh.w - jc1 + 64 - lane;
    if (o >= 0 && o < sh.N) atomicAdd(&srow[o], run);
  }
}

// ------------------------------------------------------------------ block map
// blk[h][R][C] = softmax over C <= R of scale * Qblk[R].Kblk[C]; entries C > R are 0.
// One workgroup = a strip of 16 rows of one head, or rows_wg = 8 or 4 of them where the strips are few: the other rows
// of its matrix tiles are then left alone.  It first streams its rows_wg b query rows (a row
// block per wave at a time, its loads one batch of eight ahead of the sums) and keeps their means in
// LDS.  The means are split into bf16 head + remainder (see store_split), and
// v_mfma_f32_16x16x32_bf16 forms the 16x16 logit tiles from head x head and the
// two cross products: fp32-grade logits (a bf16 product alone would break the 1e-3 tolerance of
// blk) at a fifth of the cycles of the fp32 matrix instruction.  Lane l of a tile: column l%16,
// rows 4(l/16) + r.  The column tiles of the strip go round-robin to the four waves and stay in
// registers (MT tiles per wave) until the row maxima and sums are known, so blk is written exactly
// once.  Strips are taken longest first.  Bound by the HBM stream of Q, which runs at 5 TB/s with the
// workgroups of pass 2 beside it (281 us at 128K tokens and 32 heads).
template <int MT>
__device__ inline void block_map_strip(int L, int rows_wg, char *lds, const uint16_t *__restrict__ Q,
                                       const float *__restrict__ kblk, const Shape &sh, float c2,
                                       float *__restrict__ blk, const int32_t *__restrict__ only_bc) {
  uint16_t *tile = (uint16_t *)lds;                            // 8 KB
  float (*red)[kMapWaves][16] = (float (*)[kMapWaves][16])(lds + 8192);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int nb = sh.nb;
  const int nst = (nb + 15) / 16 * sh.Hq;
  if (L * rows_wg >= 16 * nst) return;
  int sub = 0;
  while (L - sub * nst >= nst) ++sub;
  int strip, h;
  strip_of(L - sub * nst, sh, strip, h);
  if (only_bc && only_bc[h] != SA_BLOCK_CLUSTER) return;  // uniform over the workgroup, before any barrier
  const int R0 = 16 * strip + sub * rows_wg, rows = min(rows_wg, nb - R0);
  if (rows <= 0) return;
  const int T = strip + 1;  // column tiles 0..strip hold every C <= R of this strip
  // other rows of the matrix tile are never formed; nothing that is kept depends on them
  strip_means(Q + (size_t)h * sh.q_hs + (size_t)R0 * sh.b * sh.q_rs, sh, tile, wv, kMapWaves, rows);
  __syncthreads();
  // tile t of a means array: 8 KB = [part][st][lane][16 bytes]
  const uint16_t *ksrc = (const uint16_t *)(kblk + (size_t)(h / sh.g) * means_tiles(nb) * 2048) + 8 * lane;

  // operands of v_mfma_f32_16x16x32_bf16: lane (n = row of A / column of B, g) holds elements
  // 32 st + 8 g .. + 7 of its mean, st = 0..3: 16 bytes of heads and 16 bytes of remainders per step,
  // which is the order the means are stored in
  bf16x8 ah[4], al[4];
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    ah[st] = *(const bf16x8 *)(tile + 512 * st + 8 * lane);
    al[st] = *(const bf16x8 *)(tile + 2048 + 512 * st + 8 * lane);
  }
  f32x4 acc[MT];
  bf16x8 bh[4], bl[4];
#pragma unroll
  for (int k = 0; k < MT; ++k) {
    const int tc = kMapWaves * k + wv;
    if (tc < T) {
      {
        const uint16_t *bp = ksrc + (size_t)tc * 4096;
#pragma unroll
        for (int st = 0; st < 4; ++st) {
          bh[st] = *(const bf16x8 *)(bp + 512 * st);
          bl[st] = *(const bf16x8 *)(bp + 2048 + 512 * st);
        }
      }
      // three independent chains: heads x heads, and the two cross terms (remainder x remainder,
      // about 2^-18 of the product, is dropped)
      f32x4 dhh = {0.f, 0.f, 0.f, 0.f}, dhl = dhh, dlh = dhh;
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        dhh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[st], bh[st], dhh, 0, 0, 0);
        dhl = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[st], bl[st], dhl, 0, 0, 0);
        dlh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[st], bh[st], dlh, 0, 0, 0);
      }
      const f32x4 d = dhh + (dhl + dlh);
      const int C = 16 * tc + n;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[k][r] = (C <= R0 + 4 * g + r) ? d[r] * c2 : -INFINITY;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[k][r] = -INFINITY;
    }
  }
  // row maxima: over this lane's tiles, the 16 lanes of a group, the four waves
  float mx[4], sm[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float v = -INFINITY;
#pragma unroll
    for (int k = 0; k < MT; ++k) v = fmaxf(v, acc[k][r]);
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d));
    mx[r] = v;
  }
  if (n == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[0][wv][4 * g + r] = mx[r];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float v = red[0][0][4 * g + r];
#pragma unroll
    for (int k = 1; k < kMapWaves; ++k) v = fmaxf(v, red[0][k][4 * g + r]);
    mx[r] = v;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < MT; ++k) {
      acc[k][r] = __builtin_amdgcn_exp2f(acc[k][r] - mx[r]);  // column 0 is kept in every row: mx is finite
      v += acc[k][r];
    }
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    sm[r] = v;
  }
  if (n == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[1][wv][4 * g + r] = sm[r];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float v = red[1][0][4 * g + r];
#pragma unroll
    for (int k = 1; k < kMapWaves; ++k) v += red[1][k][4 * g + r];
    sm[r] = 1.0f / v;
  }
  float *dst = blk + (size_t)h * nb * nb;
#pragma unroll
  for (int k = 0; k < MT; ++k) {
    const int tc = kMapWaves * k + wv;
    if (tc < T) {
      const int C = 16 * tc + n;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int R = R0 + 4 * g + r;
        if (4 * g + r < rows && C < nb) dst[(size_t)R * nb + C] = acc[k][r] * sm[r];
      }
    }
  }
  // zeros right of the strip's last tile (16 bytes per lane where the rows allow it)
  const int c0 = 16 * T;
  if ((nb & 3) == 0) {
    const int n4 = (nb - c0) >> 2;
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = tid; i < rows * n4; i += 64 * kMapWaves) {
      const int r = i / n4, c4 = i - r * n4;
      *(float4 *)(dst + (size_t)(R0 + r) * nb + c0 + 4 * c4) = z4;
    }
  } else {
    for (int r = 0; r < rows; ++r) {
      const int R = R0 + r;
      for (int C = c0 + tid; C < nb; C += 64 * kMapWaves) dst[(size_t)R * nb + C] = 0.f;
    }
  }
}

// ------------------------------------------------------------------ the two launches
// The second launch in units of eight consecutive workgroups (one per XCD): window_units of them belong
// to pass 2, spread evenly over the first `spread` units, the others to the block map.  True for a unit
// of pass 2; k: its number among the units of its kind.
__device__ inline bool window_unit(int u, int window_units, int spread, int &k) {
  const int v = min(u, spread);
  const int before = (int)((long long)v * window_units / spread);
  const bool window = v < spread && (int)((long long)(v + 1) * window_units / spread) != before;
  k = window ? before : u - before;
  return window;
}

constexpr int kWindowLds = kStages * 64 * 128 * 2;

// First: pass 1.
__global__ __launch_bounds__(256, 3) void estimate_first_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, Shape sh, float c, float2 *__restrict__ part,
    float *__restrict__ kblk, float *__restrict__ s_out) {
  __shared__ __attribute__((aligned(16))) char lds[kWindowLds];
  window_stats((int)blockIdx.x, (uint16_t (*)[64 * 128])lds, Q, K, sh, c, part, s_out, kblk);
}

// Second: pass 2, and the block map.
template <int MT>
__global__ __launch_bounds__(256, (MT <= 16 ? 3 : MT <= 32 ? 2 : 1)) void estimate_second_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, Shape sh, float c, const float2 *__restrict__ part,
    const float *__restrict__ bias, const float *__restrict__ kblk, sa_scores out, int window_units, int spread,
    int rows_wg, const int32_t *__restrict__ only_bc) {
  __shared__ __attribute__((aligned(16))) char lds[kWindowLds];
  int k;
  const bool window = window_unit((int)blockIdx.x >> 3, window_units, spread, k);
  const int L = 8 * k + ((int)blockIdx.x & 7);
  if (!window)
    block_map_strip<MT>(L, rows_wg, lds, Q, kblk, sh, c, out.blk, only_bc);
  else if (L < sh.nchunks * sh.Hkv * ((sh.g + 3) / 4))
    window_scores(L, (uint16_t (*)[64 * 128])lds, Q, K, sh, c, part, bias, out.v, out.s);
}

// Chunks up to which every pass-2 workgroup forms its rows' constants itself; beyond, a launch does.
constexpr int kBiasChunks = 128;

}  // namespace

hipError_t launch_estimate_part(const Shape &sh, const Workspace &ws, const uint16_t *Q, const uint16_t *K,
                                sa_scores out, EstimatePart what, const int32_t *only_block_cluster,
                                hipStream_t st) {
  const float c = sh.scale * kLog2e;
  const int nstrips = (sh.nb + 15) / 16, windows = sh.nchunks * sh.Hkv * ((sh.g + 3) / 4);
  float *bias = sh.nchunks > kBiasChunks ? (float *)ws.stats : nullptr;
  if (what != EstimatePart::BlockMap) {
    estimate_first_kernel<<<windows, 256, 0, st>>>(Q, K, sh, c, ws.part, ws.kblk, out.s);
    if (bias) window_stats_reduce_kernel<<<dim3(sh.Hq, kWin / 16), 1024, 0, st>>>(ws.part, sh.nchunks, sh.w, bias);
  }
  const int wu = what == EstimatePart::BlockMap ? 0 : (windows + 7) / 8;
  // Row blocks per workgroup of the block map: a strip's 16, or where those workgroups leave compute units without one, 8
  // or 4, each with all column tiles of the strip.  A workgroup waits for the stream of its queries, which
  // is twice as long with 128-row blocks: there up to two workgroups per compute unit.  4 heads at 1K and 4K tokens 17.5 ->
  // 16.4 and 18.7 -> 17.2 us, with 128-row blocks 23.9 -> 17.1 at 4K and 73.5 -> 66.5 at 64K, 8 heads of one KV head at
  // 8K 23.9 -> 18.9; beyond the line it costs (one workgroup more per unit: 16 heads at 16K 42.7 -> 45.9).  Over 568 sizes
  // of 2 to 32 heads 9 % in the mean; 39 of them are up to 17 % slower than with whole strips, most where the map's
  // workgroups and the windows' come to one more per unit (6 heads at 10K 21.2 -> 24.7, 4 at 14K 30.5 -> 34.6), but not
  // halving there would give away as many gains as losses (8 heads at 24K, b = 128, 36.9 -> 31.9).
  int rows_wg = 16;
  while (rows_wg > 4 && nstrips * sh.Hq * (16 / rows_wg) * 2 * 64 <= sh.n_cu * sh.b) rows_wg /= 2;
  // A single strip of less than 16 row blocks needs no workgroups for those it lacks: empty as they are, they push the
  // windows' workgroups on to units that have one (128 heads on 8 KV heads at 384 and 512 tokens 21.4 and 19.8 us with
  // them, 17.2 and 17.1 without, with 128-row blocks 19.1 and 21.1, 17.0 and 16.8; 64 at 1024 19.6, 16.9).
  const int per_strip = (std::min(sh.nb, 16) + rows_wg - 1) / rows_wg;
  const int units = wu + (what == EstimatePart::Windows ? 0 : (nstrips * sh.Hq * per_strip + 7) / 8);
  // 4/5: 364 us for the estimator at 128K tokens, 114 at 32K; all units 388 and 119 (pass 2 is left for the end), the
  // first ones 388 and 121 (it does not run beside the stream any more); 65, 65 and 62 at 16K
  int spread = units * 4 / 5;
  if (spread < wu) spread = wu;
  if (spread < 1) spread = 1;
  const int tiles_per_wave = (nstrips + kMapWaves - 1) / kMapWaves;
#define SA_SECOND(MT)                                                                                         \
  estimate_second_kernel<MT><<<8 * units, 256, 0, st>>>(Q, K, sh, c, ws.part, bias, ws.kblk, out, wu, spread, \
                                                        rows_wg, only_block_cluster)
  if (tiles_per_wave <= 8) SA_SECOND(8);
  else if (tiles_per_wave <= 16) SA_SECOND(16);
  else if (tiles_per_wave <= 32) SA_SECOND(32);
  else SA_SECOND(64);
#undef SA_SECOND
  return hipGetLastError();
}

}  // namespace sa
