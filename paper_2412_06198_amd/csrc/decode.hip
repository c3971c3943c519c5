// One decode step over the prefill index (the paper names gains in the decoding phase without a
// method; problem statement: decode queries are [B, 1, H]).  The query at position pos >= N
// attends, per query head, the union of the generated keys N..pos, the selected key columns, the
// keys pos - o of the selected diagonal offsets and the keys of the key blocks kept for the last
// row block of the prompt, each key once.  A pure gather: 512 bytes of K and V per kept key and
// head, nothing reused, so the kernel is laid out for HBM: every key is read by 16 lanes as one
// 256-byte row of K and one of V, the rows of a step of 16 keys per wave in flight while the step before is
// computed, and the key list of a head split over several workgroups.  A short list leaves a chain of
// memory round trips (list lengths, list, rows, partial (max, sum, output) triple, arrival counter, all
// triples of the head) and what a single wave issues in between: the workgroup that arrives last merges
// instead of a second launch, and a list place is resolved by one lane, not by the 16 that read its row.
// 8 heads, 4096-token prompt: 10.9 -> 6.8 us (an empty launch is 2.2); 32 heads, 128K-token prompt, 29 MB
// of rows out of the memory-side cache: 16.3 -> 10.8 us, and 26.7 -> 15.0 (the kernels alone) where K and V
// have been pushed out of it, as they are where a step reads other layers in between.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "sa_internal.h"

namespace sa {
namespace {

constexpr int kPartStride = 132;  // floats per partial: max, sum, 2 (first one: arrival counter, others: 0), 128 outputs

// Partials of the variant that allocates nothing (sa_sparse_decode_static): room for the largest
// head count x split count the launcher ever picks (Hq * splits <= 512), 270336 bytes on every GPU
// the library runs on, held until the process ends.  In host code this name is only a stand-in for
// the symbol: the device address comes from hipGetSymbolAddress, once per device.
constexpr int kStaticPartials = 512;
static __device__ __align__(256) float scratch[kStaticPartials * kPartStride];
constexpr int kMaxDevices = 64;

// A head's arrival counter lives in floats 2 and 3 of its first partial: the step's token in the upper 48
// bits, in the lower 16 the number of workgroups that have arrived.  The memory may hold anything: what the
// caller's workspace was used for before, or the count of a step that overlapped another one or never ended.
// A step takes only its own token for a count: a head's first workgroup puts the token there while its rows are
// on their way, one that arrives before that does it itself, and nothing is read from what was left.  Each
// launch has a token of its own, so that no clearing launch is needed; a recorded one repeats its token with
// every replay, so there the counters are cleared by a launch before it (8 heads, 4096 tokens: 8.4 us a
// recorded step instead of 6.6; a count that the last one to arrive put back to 0 cost 0.1 us less, and what an
// overlapping step left there stayed for good).
constexpr int kCountBits = 16;

struct DecArgs {
  const uint16_t *q, *K, *V;
  uint16_t *o;
  const int32_t *n_cols, *cols, *n_offs, *offs, *rowptr, *blkcols;
  float *part;
  int Hq, g, N, b, nb, k_v, k_s, cap_b, S, pos;
  int64_t kv_hs, kv_rs;
  float c;  // softmax scale * log2(e)
  uint64_t token;  // of this launch, counted 0; never 0 itself
};

constexpr int kThreads = 256, kWaves = kThreads / 64;  // 512: 3 % faster for 128K, 10 % slower for short prompts
constexpr int U = 4;          // rows of K and of V that a lane has in flight per step
constexpr int kStep = 4 * U;  // keys of a wave per step: four slots of 16 lanes
constexpr int kRing = 128;    // keys of a wave that are resolved and not yet read: 15 + 64 at most
constexpr int kMinChunk = kWaves * kStep;  // keys of a workgroup: one step of each wave; 128 was 0.7 us slower

// A reduction over the four 16-lane slots of a wave, on each lane.
template <typename F>
__device__ inline float over_slots(float x, F f) {
  const unsigned a = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  const unsigned c = __float_as_uint(f(__uint_as_float(r0), __uint_as_float(r1)));
  const auto s = __builtin_amdgcn_permlane32_swap(c, c, false, false);
  const unsigned s0 = s[0], s1 = s[1];
  return f(__uint_as_float(s0), __uint_as_float(s1));
}

__device__ inline void unpack8(const uint4 x, float (&f)[8]) {
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(w[e] << 16);
    f[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
  }
}

// Sum over 16 lanes, on each of them: partners at distance 8, 7, 2 and 1.
template <int CTRL>
__device__ inline float row_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ inline float sum16(float x) {
  x += row_move<0x128>(x);
  x += row_move<0x141>(x);
  x += row_move<0x4E>(x);
  x += row_move<0xB1>(x);
  return x;
}

// Partial results cross workgroups inside the launch by agent-scope accesses, which pass the L2 caches
// by: nothing has to be written back or invalidated on the way (fences at that scope cost 40 us here).  They
// are ordered before the arrival by vmcnt(0) and the workgroup's barrier, see the top of index.hip.
__device__ inline void put(float *p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline float get(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Merge n <= 64 partials of a head, normalise, round to bf16: 256 threads, thread (k0, d) takes the outputs d
// of partials k0, k0 + 2, ...  All reads are on their way before the first is needed.
__device__ inline void merge(const float *src, int n, float *wgt, float *s_L, float *half, uint16_t *o) {
  const int tid = threadIdx.x, d = tid & 127, k0 = tid >> 7;
  float mk = -INFINITY, lk = 0.f;
  if (tid < n) {
    mk = get(src + (size_t)tid * kPartStride);
    lk = get(src + (size_t)tid * kPartStride + 1);
  }
  float x[32];
  // Places past the end weigh 0 and read the 0 that the last partial holds for them: anything else could be
  // infinite.  (Masks on x after the reads cost 0.3 us.)
  const int none = (n - 1) * kPartStride + 2;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    if (8 * (i / 8) * 2 < n) x[i] = get(src + (k0 + 2 * i < n ? (k0 + 2 * i) * kPartStride + 4 + d : none));  // by eights
    else x[i] = 0.f;
  }
  if (tid < 64) {
    float M = mk;
    for (int e = 32; e >= 1; e >>= 1) M = fmaxf(M, __shfl_xor(M, e));
    const float w = mk == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk - M);
    float L = lk * w;
    for (int e = 32; e >= 1; e >>= 1) L += __shfl_xor(L, e);
    wgt[tid] = w;  // 0 from n on
    if (tid == 0) *s_L = L;
  }
  __syncthreads();
  float O = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i)
    O = __builtin_fmaf(x[i], wgt[k0 + 2 * i], O);
  if (k0) half[d] = O;
  __syncthreads();
  if (k0) return;
  O += half[d];
  const float L = *s_L;
  const __bf16 r = (__bf16)(L > 0.f ? O / L : 0.f);
  o[d] = __builtin_bit_cast(uint16_t, r);
}

// A head's key list, in this order: keys of the kept blocks, columns, diagonal keys, generated keys; and how
// it is shared out: workgroups 0 .. n - 1 take `chunk` keys each.
struct KeyList {
  int e0, nblk, nc, no, n0, n1, n2, total, chunk, n;
};
__device__ inline KeyList key_list(const DecArgs &p, int h) {
  KeyList k;
  const int32_t *rp = p.rowptr + (size_t)h * (p.nb + 1);
  k.e0 = min(max(rp[p.nb - 1], 0), p.cap_b);
  k.nblk = min(max(rp[p.nb], k.e0), p.cap_b) - k.e0;
  k.nc = min(max(p.n_cols[h], 0), p.k_v);
  k.no = min(max(p.n_offs[h], 0), p.k_s);
  k.n0 = k.nblk * p.b;
  k.n1 = k.n0 + k.nc;
  k.n2 = k.n1 + k.no;
  k.total = k.n2 + p.pos - p.N + 1;
  k.chunk = max(((k.total + p.S - 1) / p.S + 15) / 16 * 16, kMinChunk);
  k.n = (k.total + k.chunk - 1) / k.chunk;  // <= S, and at least 1: the query's own key is in the list
  return k;
}

// What one lane has written to LDS before is read by the others of its wave after it, and the other way round.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// grid (S, Hq), 256 threads.  Each wave walks a quarter of the workgroup's keys by itself: 64 lanes resolve 64
// list places (which key, does it count here), the keys that count queue up in the wave's ring, and a step
// reads the rows of 16 of them, slot s of 16 lanes every fourth one, lane ln elements 8 ln .. 8 ln + 7.
__global__ __launch_bounds__(kThreads) void decode_kernel(DecArgs p) {
  __shared__ __attribute__((aligned(16))) uint32_t blkbm[kMaxSeq / 64 / 32];  // key blocks kept for the last row block
  __shared__ __attribute__((aligned(16))) uint32_t colbm[kMaxSeq / 32];       // selected key columns
  __shared__ int64_t ring[kWaves][kRing];                                     // element offsets of key rows
  __shared__ float sm[kWaves], sl[kWaves];
  __shared__ __attribute__((aligned(16))) float so[kWaves][kHeadDim];
  __shared__ float wgt[64], s_L;
  __shared__ unsigned s_last;
  const int sp = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const int N = p.N, nb = p.nb, b = p.b, shift = b == 128 ? 7 : 6;
  const int lane = tid & 63, ln = tid & 15, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint4 qx = *(const uint4 *)(p.q + (size_t)h * kHeadDim + ln * 8);
  const KeyList L = key_list(p, h);
  if (sp >= L.n) return;
  float *part = p.part + (size_t)h * p.S * kPartStride;
  uint64_t *arrived = (uint64_t *)(part + 2);
  // the thread that counts the arrival, in the wave with the fewest keys (0.07 us less than in the first one)
  const bool counts = tid == kThreads - 1, claims = counts && sp == 0;
  uint64_t seen = 0;
  if (claims) seen = __hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int32_t *bc = p.blkcols + (size_t)h * p.cap_b + L.e0;
  const int32_t *colp = p.cols + (size_t)h * p.k_v;
  const int32_t *offp = p.offs + (size_t)h * p.k_s;
  const int t_begin = sp * L.chunk, t_end = min(t_begin + L.chunk, L.total);
  const int share = ((t_end - t_begin + kWaves - 1) / kWaves + kStep - 1) / kStep * kStep;
  int t_next = min(t_begin + wave * share, t_end);
  const int t_stop = min(t_next + share, t_end);
  auto entry = [&](int t) {  // what the list says at a place; generated keys stand in no list
    const int32_t *src = t < L.n0 ? bc + (t >> shift) : t < L.n1 ? colp + (t - L.n0) : offp + (t - L.n1);
    return t < t_stop && t < L.n2 ? *src : -1;
  };
  int ent = entry(t_next + lane);
  // A key counts where it first appears in the list: columns and diagonal keys are screened by the kept
  // blocks, diagonal keys by the columns too.  Only workgroups with such keys build the bitmaps.
  const bool need_blk = t_begin < L.n2 && t_end > L.n0, need_cols = t_begin < L.n2 && t_end > L.n1 && L.nc > 0 && L.no > 0;
  if (need_blk) {
    for (int i = tid; i < (nb + 127) / 128; i += kThreads) ((uint4 *)blkbm)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (need_cols)
      for (int i = tid; i < (N + 127) / 128; i += kThreads) ((uint4 *)colbm)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    for (int e = tid; e < L.nblk; e += kThreads) {
      const int C = bc[e];
      if (C >= 0 && C < nb) atomicOr(&blkbm[C >> 5], 1u << (C & 31));
    }
    if (need_cols)
      for (int i = tid; i < L.nc; i += kThreads) {
        const int c = colp[i];
        if (c >= 0 && c < N) atomicOr(&colbm[c >> 5], 1u << (c & 31));
      }
    __syncthreads();
  }
  auto kept_block = [&](int key) { const int C = key >> shift; return ((blkbm[C >> 5] >> (C & 31)) & 1u) != 0u; };
  const uint16_t *Kh = p.K + (size_t)(h / p.g) * p.kv_hs + ln * 8;
  const uint16_t *Vh = p.V + (size_t)(h / p.g) * p.kv_hs + ln * 8;
  int put_at = 0, get_at = 0;  // of the ring, uniform
  auto resolve = [&] {         // until a step is full or the list at its end
    while (put_at - get_at < kStep && t_next < t_stop) {
      const int t = t_next + lane;
      int j = -1;
      if (t < L.n0) {
        if (ent >= 0 && ent < nb) j = (ent << shift) + (t & (b - 1));
      } else if (t < L.n1) {
        if (ent >= 0 && ent < N && !kept_block(ent)) j = ent;
      } else if (t < L.n2) {
        const int jj = p.pos - ent;
        if (ent >= 0 && jj >= 0 && jj < N && !kept_block(jj) && !(need_cols && ((colbm[jj >> 5] >> (jj & 31)) & 1u)))
          j = jj;
      } else if (t < t_stop) {
        j = N + (t - L.n2);
      }
      t_next += 64;
      ent = entry(t_next + lane);
      const uint64_t live = __ballot(j >= 0);
      const int at = put_at + __builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));
      if (j >= 0) ring[wave][at & (kRing - 1)] = (int64_t)j * p.kv_rs;
      put_at += __popcll(live);
    }
    return put_at > get_at;
  };
  const int slot = lane >> 4;
  uint4 kx[2][U], vx[2][U];
  int cnt[2];
  auto fetch = [&](uint4 (&kr)[U], uint4 (&vr)[U], int &n) {
    n = min(put_at - get_at, kStep);
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < U; ++u) {  // a place without a key reads the last key again
      const int64_t row = ring[wave][(get_at + min(4 * u + slot, n - 1)) & (kRing - 1)];
      kr[u] = *(const uint4 *)(Kh + row);
      vr[u] = *(const uint4 *)(Vh + row);
    }
    wave_lds_sync();
    get_at += n;
  };
  float qv[8], m = -INFINITY, l = 0.f, acc[8];
  unpack8(qx, qv);
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  auto attend = [&](const uint4 (&kr)[U], uint4 (&vr)[U], int n) {
    if (n < kStep) {  // the last step: a place without a key weighs 0, and 0 x inf is not 0
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (4 * u + slot >= n) vr[u] = make_uint4(0u, 0u, 0u, 0u);
    }
    float s[U], m_new = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[8], dot = 0.f;
      unpack8(kr[u], kf);
#pragma unroll
      for (int e = 0; e < 8; ++e) dot = __builtin_fmaf(kf[e], qv[e], dot);
      s[u] = 4 * u + slot < n ? sum16(dot) * p.c : -INFINITY;
      m_new = fmaxf(m_new, s[u]);
    }
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m - m_ref);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float pv = __builtin_amdgcn_exp2f(s[u] - m_ref);
      float vf[8];
      unpack8(vr[u], vf);
      l += pv;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(pv, vf[e], acc[e]);
    }
  };
  // the rows of a step are read while the step before is computed
  if (resolve()) {
    fetch(kx[0], vx[0], cnt[0]);
    // the token into the counter, unless a workgroup of this step has been there
    if (claims && (seen ^ p.token) >> kCountBits)
      (void)__hip_atomic_compare_exchange_strong(arrived, &seen, p.token, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
      const bool more = resolve();
      if (more) fetch(kx[1], vx[1], cnt[1]);
      attend(kx[0], vx[0], cnt[0]);
      if (!more) break;
      const bool again = resolve();
      if (again) fetch(kx[0], vx[0], cnt[0]);
      attend(kx[1], vx[1], cnt[1]);
      if (!again) break;
    }
  }
  // the four slots of a wave, then the waves
  const float Mw = over_slots(m, [](float x, float y) { return fmaxf(x, y); });
  const float ww = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - Mw);
  const auto add = [](float x, float y) { return x + y; };
  l = over_slots(l * ww, add);
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = over_slots(acc[e] * ww, add);
  if (lane < 16) {
    if (lane == 0) { sm[wave] = Mw; sl[wave] = l; }
    *(float4 *)&so[wave][ln * 8] = make_float4(acc[0], acc[1], acc[2], acc[3]);
    *(float4 *)&so[wave][ln * 8 + 4] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
  __syncthreads();
  if (tid < kHeadDim) {
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) M = fmaxf(M, sm[k]);
    float lsum = 0.f, O = 0.f;
    if (M > -INFINITY) {
#pragma unroll
      for (int k = 0; k < kWaves; ++k) {
        const float w = __builtin_amdgcn_exp2f(sm[k] - M);  // 0 for an empty one
        lsum += sl[k] * w;
        O += so[k][tid] * w;
      }
    }
    if (L.n == 1) {  // the only workgroup of the head
      const __bf16 r = (__bf16)(lsum > 0.f ? O / lsum : 0.f);
      p.o[(size_t)h * kHeadDim + tid] = __builtin_bit_cast(uint16_t, r);
    } else {
      float *dst = part + (size_t)sp * kPartStride;
      if (tid == 0) { put(dst, M); put(dst + 1, lsum); }
      if (tid == 1 && sp > 0) put(dst + 2, 0.f);  // see merge; dst[2], dst[3] of the first one: the counter
      put(dst + 4 + tid, O);
    }
  }
  if (L.n == 1) return;
  // ---- the last one to arrive merges; nobody waits
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this thread's partials have been performed
  __syncthreads();
  if (counts) {
    uint64_t before = __hip_atomic_fetch_add(arrived, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while ((before ^ p.token) >> kCountBits) {  // added to a value that is not this step's: nobody has been here yet
      uint64_t cur = before + 1;                // ends: an exchange only fails where a workgroup has changed the counter
      if (__hip_atomic_compare_exchange_strong(arrived, &cur, p.token + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT))
        before = p.token;  // this one put the token there, and itself
      else if ((cur ^ p.token) >> kCountBits)
        before = cur - 1;
      else
        before = __hip_atomic_fetch_add(arrived, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    s_last = before == p.token + (uint64_t)(L.n - 1);
  }
  __syncthreads();
  asm volatile("" ::: "memory");
  if (s_last) merge(part, L.n, wgt, &s_L, so[0], p.o + (size_t)h * kHeadDim);
}

// The arrival counters of all heads, before a recorded step.
__global__ void clear_arrivals_kernel(float *part, int Hq, int S) {
  if ((int)threadIdx.x < Hq) *(uint64_t *)(part + (size_t)threadIdx.x * S * kPartStride + 2) = 0;
}

// 48 bits that no launch of the process has had before: a count times an odd number, so that they are neither a
// neighbour of an earlier token nor a value that other data is likely to hold.  (2^48 launches come around
// after 28 years at one every 3 us.)
uint64_t next_token() {
  static std::atomic<uint64_t> launches{0};
  for (;;) {
    const uint64_t t = (launches.fetch_add(1, std::memory_order_relaxed) + 1) * 0x9D37C1E5A86B4F01ull << kCountBits;
    if (t) return t;
  }
}

}  // namespace

int decode_splits(const Shape &sh) {
  const int s = 512 / (sh.Hq > 0 ? sh.Hq : 1);  // about two workgroups per compute unit in all
  return s < 1 ? 1 : (s > 64 ? 64 : s);
}

namespace {

// Workgroups per head of one step: decode_splits, but no more than have a step's 64 keys in the longest list that the
// budgets allow.  Those without keys only read how long the list is, but 512 of them are still 0.4 us of a step of 7 (8
// heads at 1.2K tokens with 744 generated ones 6.97 -> 6.67 us, 6.74 -> 6.19 with few blocks).  What a list does hold is
// known on the device alone, and k_blocks >= nb lets any head keep every block of the last row.  The line is not drawn by
// what the budgets give on average: 256 workgroups wherever such lists fit them took 0.4 us from those, but rows of twice
// the mean lost (24 heads at 3K 6.6 -> 7.9 us, 8 at 64K 7.1 -> 8.2) and whole rows more (8 heads at 64K 23 -> 31, at 128K 38 -> 54).
int splits_of_step(const Shape &sh, int pos) {
  const int64_t longest = (int64_t)pos + 1 + sh.k_v + sh.k_s;  // every key, and the columns and offsets beside them
  return (int)std::min<int64_t>(decode_splits(sh), (longest + kMinChunk - 1) / kMinChunk);
}

}  // namespace

size_t decode_partial_bytes(const Shape &sh) { return (size_t)sh.Hq * decode_splits(sh) * kPartStride * 4; }

size_t decode_static_bytes() { return sizeof(float) * kStaticPartials * kPartStride; }

// Device address of `scratch` on the current device: asked for once per device (each GPU holds its
// own copy of the array at its own address) and kept.
hipError_t decode_static_scratch(float **out) {
  static std::mutex mu;
  static float *ptr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    float *d = nullptr;
    e = hipGetSymbolAddress((void **)&d, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!d) return hipErrorInvalidSymbol;
    ptr[dev] = d;
  }
  *out = ptr[dev];
  return hipSuccess;
}

hipError_t launch_sparse_decode(const Shape &sh, float *partials, const uint16_t *q, const uint16_t *K,
                                const uint16_t *V, sa_index idx, int pos, uint16_t *o, hipStream_t st) {
  DecArgs a;
  a.q = q; a.K = K; a.V = V; a.o = o;
  a.n_cols = idx.n_cols; a.cols = idx.cols; a.n_offs = idx.n_offs; a.offs = idx.offs;
  a.rowptr = idx.rowptr; a.blkcols = idx.blkcols;
  a.part = partials;
  a.Hq = sh.Hq; a.g = sh.g; a.N = sh.N; a.b = sh.b; a.nb = sh.nb; a.k_v = sh.k_v; a.k_s = sh.k_s;
  a.cap_b = sh.cap_b; a.S = splits_of_step(sh, pos); a.pos = pos;
  a.kv_hs = sh.kv_hs; a.kv_rs = sh.kv_rs;
  a.c = sh.scale * 1.4426950408889634f;
  a.token = next_token();
  hipStreamCaptureStatus recording = hipStreamCaptureStatusNone;
  // if the stream cannot say, the step is launched as a recorded one: right in either case
  if (hipStreamIsCapturing(st, &recording) != hipSuccess) {
    (void)hipGetLastError();
    recording = hipStreamCaptureStatusActive;
  }
  if (recording != hipStreamCaptureStatusNone) clear_arrivals_kernel<<<1, kMaxHeads, 0, st>>>(partials, sh.Hq, a.S);
  decode_kernel<<<dim3(a.S, sh.Hq), kThreads, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace sa
