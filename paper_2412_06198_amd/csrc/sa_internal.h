// Internal declarations shared by the host API and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sa.h"

namespace sa {

constexpr int kHeadDim = 128;
constexpr int kMaxHeads = 128;
constexpr int kWin = 64;          // rows of the last-query window the estimator tiles for
constexpr int kMaxSeq = 262144;   // key-tile bitmaps of the attention kernel cover this many keys

struct Override { int8_t pat[kMaxHeads]; };

// Budgets of one head, for index builds whose heads differ in them (device arrays of these).
struct HeadBudget { int32_t k_v, k_s, k_b, local; };

// Prefix sums and sums over a wave on the data-parallel lane moves (row shifts inside 16 lanes, then
// two broadcasts): a shuffle through LDS per step is a round trip of some 60 cycles.
template <int CTRL, int ROWS>
__device__ inline unsigned lane_move(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
__device__ inline unsigned wave_inclusive_sum(unsigned x) {
  x += lane_move<0x111, 0xF>(x);  // row_shr:1
  x += lane_move<0x112, 0xF>(x);  // row_shr:2
  x += lane_move<0x114, 0xF>(x);  // row_shr:4
  x += lane_move<0x118, 0xF>(x);  // row_shr:8
  x += lane_move<0x142, 0xA>(x);  // row_bcast:15 into rows 1 and 3
  x += lane_move<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}
template <int CTRL, int ROWS>
__device__ inline unsigned long long lane_move64(unsigned long long x) {
  return (unsigned long long)lane_move<CTRL, ROWS>((unsigned)x) | ((unsigned long long)lane_move<CTRL, ROWS>((unsigned)(x >> 32)) << 32);
}
// The sum over the wave, in lane 63.
__device__ inline unsigned long long wave_sum63(unsigned long long x) {
  x += lane_move64<0x111, 0xF>(x);
  x += lane_move64<0x112, 0xF>(x);
  x += lane_move64<0x114, 0xF>(x);
  x += lane_move64<0x118, 0xF>(x);
  x += lane_move64<0x142, 0xA>(x);
  x += lane_move64<0x143, 0xC>(x);
  return x;
}

// Everything the kernels need, resolved from sa_config at sa_create time.
struct Shape {
  int Hq, Hkv, g, N, b, nb, w;
  int gq;                         // query heads of a KV head in Q and the scores: g, or a part of it where every one
                                  // of them is taken with several indices (head h is then query head h % gq of its group)
  int k_v, k_s, k_b, cap_b, sink, local;
  int probe_v, probe_s, lift_num, lift_den;
  int row_select;                 // Block-Cluster heads: 1 = every row keeps its own share of k_b
  int row_norm;                   // Block-Cluster heads: 1 = global top-k on blk[R][C] * (R + 1)
  int diag_blocks;                // Interval-Slash heads: 1 = selected diagonals kept as whole blocks
  int lazy_blk;                   // one-call form: 1 = block map only for the heads decided Block-Cluster
  int chunk, nchunks;             // keys per estimator workgroup (window passes), ceil(N / chunk)
  int n_cu;                       // compute units of the device the context was created on
  int64_t q_hs, q_rs, kv_hs, kv_rs;
  int64_t o_hs, o_rs;             // of the attention output: Q's
  float scale;
};

struct Workspace {
  float *kblk;                    // [Hkv][ceil(nb/16)] tiles (8 KB) of K block means
  float2 *part;                   // [Hq][nchunks][64] partial (max, sum) of the window rows
  float2 *stats;                  // [Hq][64] row constants, where a launch of their own forms them
  uint32_t *colbits;              // [Hq][N/32] membership bitmap of the selected columns
  int32_t *colprefix;             // [Hq][N/32] number of selected columns before each word of colbits
  float *dec_part;                // [Hq][splits][132] partial (max, sum, output) of the decode step
  unsigned int *queue;            // [8] work-queue heads of the attention kernel
  void *idx;                      // per-head scratch of the index builder
  uint16_t *kg, *vg;              // [Hq][roundup64(k_v)][kv_rs] gathered K / V rows of the selected columns
  void *attn_items;               // what each ticket of the attention kernel's queues stands for (16 bytes)
  uint16_t *attn_tiles;           // [Hq][cap_b * block / 64] key-tile lists of the row blocks
};

// Head of Q and of the scores that head h stands for.
__host__ __device__ inline int query_head(int h, int g, int gq) { return g == gq ? h : h / g * gq + h % gq; }

size_t index_scratch_bytes(const Shape &sh);

// Parts of the index builder when they run between the parts of the estimator.
enum class IndexStage { Zero, ColumnsDiagonals, Blocks, Emit };

// Which of the estimator's outputs a call computes: v and s (the window passes), blk, or all.
enum class EstimatePart { All, Windows, BlockMap };

}  // namespace sa

// The context behind the opaque handle of the C ABI (host memory).
struct sa_ctx {
  sa_config cfg;
  sa::Shape sh;
  sa::Workspace ws;
  bool have_ws;
  size_t ws_bytes;
  size_t off[13];
  char err[256];
};

namespace sa {

// key blocks of a Triangular index
long long triangular_count(int nb, int sink, int local);
// All: windows and block map.  BlockMap needs the K block means that Windows leaves in the workspace;
// only_block_cluster (device, [Hq] patterns, or nullptr = every head) restricts it to the heads
// whose entry is SA_BLOCK_CLUSTER.
hipError_t launch_estimate_part(const Shape &sh, const Workspace &ws, const uint16_t *Q, const uint16_t *K,
                                sa_scores out, EstimatePart part, const int32_t *only_block_cluster,
                                hipStream_t st);
hipError_t launch_build_index(const Shape &sh, const Workspace &ws, sa_scores in,
                              const Override &ov, sa_index out, hipStream_t st,
                              const HeadBudget *budgets = nullptr);
// The block-map part of the work is done only for the heads whose out.pattern (written by the
// ColumnsDiagonals stage) is SA_BLOCK_CLUSTER.
hipError_t launch_index_stage(const Shape &sh, const Workspace &ws, sa_scores in, const Override &ov,
                              sa_index out, IndexStage stage, hipStream_t st);
size_t decode_partial_bytes(const Shape &sh);
size_t attn_item_bytes(const Shape &sh);
size_t attn_tile_bytes(const Shape &sh);
// partials: decode_partial_bytes(sh) bytes of device memory (the context's workspace, or the static array)
hipError_t launch_sparse_decode(const Shape &sh, float *partials, const uint16_t *q, const uint16_t *K,
                                const uint16_t *V, sa_index idx, int pos, uint16_t *o, hipStream_t st);
size_t decode_static_bytes();                       // size of the library's static decode scratch
hipError_t decode_static_scratch(float **out);      // its address on the current device
hipError_t launch_sparse_prefill(const Shape &sh, const Workspace &ws, const uint16_t *Q,
                                 const uint16_t *K, const uint16_t *V, sa_index idx, uint16_t *O,
                                 unsigned long long *counters, hipStream_t st);

}  // namespace sa
