// Decoding-time update of the running scores (KVCrush Sec. 1: the cache grows
// by one entry per generated token; the H2O importance the method builds on,
// Sec. 2.3, keeps accumulating the attention every cached token receives).
//
// One call = one new token per sequence: its query of every head attends to
// the S cached keys and the resulting probability row is added to the scores.
// A matrix-vector product per head: HBM-bound on reading K once
// (B*Hkv*S*D*sizeof bytes); the exponentials and the fp32 dot products are far
// below the VALU's rate at that pace.
//
//   append_logits_mfma_kernel  (bf16 / fp16) workgroup = 256 keys of one KV head
//                          (dense cache or paged pool), 32 a wave: they go
//                          global -> LDS asynchronously and are multiplied with
//                          the query vectors of the KV group's heads (the 32
//                          columns of a 32x32x16 MFMA; unused columns are zero),
//                          so K is read once for the whole group and the dot
//                          products cost the VALU nothing.  Leaves base-2 logits in the workspace and
//                          one (max, sum) pair per workgroup and head.
//   append_logits_kernel   (fp32 inputs) the same on the VALU: a key row is read
//                          as 16-byte vectors by neighbouring lanes, the queries
//                          of up to 8 heads sit in registers.
//   append_update_kernel   merges the pairs into the row normaliser, turns
//                          logits into probabilities, sums the group's heads in
//                          ascending order and updates the score row.
#include <cmath>

#include "common.h"
#include "tiles.h"

namespace {

using namespace kvc::tiles;  // kThreads = 256, kWaves = 4, kNegBig, tile helpers

typedef uint32_t vec16 __attribute__((ext_vector_type(4)));

constexpr int kKeysPerWg = 256;
constexpr int kHeadChunk = 8;  // VALU path: query heads whose vectors are held in registers at once

struct AppendParams {
  const char* q_new;   // [B,Hq,D]
  const char* k;       // [B,Hkv,capacity,D]
  float* scores;       // [B,Hs,capacity]
  float* logits;       // workspace [B,Hq,S]
  float2* part;        // workspace [B,Hq,n_kb]
  const int* lengths;  // null, or [B]: valid tokens of each sequence (<= S), read on the device
  const int* block_table;  // null: k is dense [B,Hkv,capacity,D]; else k is a pool
                           // [n_blocks,block_size,Hkv,D] and block_table [B,capacity/block_size]
  int block_size;
  const char* k_new;   // null, or [B,Hkv,D]: the key of token S - 1 (and its value), not yet in the cache: the
  const char* v_new;   // workgroup that has this token reads it from here and puts it into k_slot and v_slot,
  char* k_slot;        // which are k and v (dense caches without lengths)
  char* v_slot;
  int B, Hq, Hkv, S, capacity, G, reduce_groups;  // S: valid tokens, or their upper bound with lengths
  int n_kb;            // kKeysPerWg-key blocks of S
  float scale_log2;    // log2(e) x softmax scale (1 / sqrt(D) unless the caller set one)
};

// First byte of key row `key` of sequence b, KV head g (bg = b * Hkv + g).
__device__ __forceinline__ const char* key_row(const AppendParams& p, int b, int g, int bg, int key,
                                               int row_bytes) {
  if (!p.block_table) return p.k + ((size_t)bg * p.capacity + key) * row_bytes;
  const int blk = p.block_table[(size_t)b * (p.capacity / p.block_size) + key / p.block_size];
  return p.k + (((size_t)blk * p.block_size + key % p.block_size) * p.Hkv + g) * row_bytes;
}

// The new token's rows go to their place in the cache: `lane` of the 2 * row_bytes / 16 lanes of one wave that do it.
__device__ __forceinline__ void store_new_token(const AppendParams& p, int bg, int S, int lane, int row_bytes) {
  const int chunks = row_bytes / 16;
  if (lane >= 2 * chunks) return;
  const bool key = lane < chunks;
  const size_t off = (size_t)(lane % chunks) * 16, src = (size_t)bg * row_bytes + off;
  const size_t dst = ((size_t)bg * p.capacity + S - 1) * row_bytes + off;
  *(vec16*)((key ? p.k_slot : p.v_slot) + dst) = *(const vec16*)((key ? p.k_new : p.v_new) + src);
}

template <bool BF16>
__device__ __forceinline__ void unpack(const vec16& x, float (&f)[BF16 ? 8 : 4]) {
  if constexpr (BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(x[i] << 16);
      f[2 * i + 1] = __uint_as_float(x[i] & 0xFFFF0000u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(x[i]);
  }
}

__device__ __forceinline__ float block_max(float v, float* red) {
  v = kvc::wave_max(v);
  __syncthreads();  // `red` may still be read from the previous use
  if (kvc::lane_id() == 0) red[threadIdx.x / KVC_WAVE] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) r = fmaxf(r, red[w]);
  return r;
}

__device__ __forceinline__ float block_sum(float v, float* red) {
  v = kvc::wave_sum(v);
  __syncthreads();
  if (kvc::lane_id() == 0) red[threadIdx.x / KVC_WAVE] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) r += red[w];
  return r;
}

// FRESH: the new token is not in the cache yet (an instantiation of its own: the test costs the loop 3 %).
template <bool BF16, int D, bool FRESH>
__global__ __launch_bounds__(kThreads) void append_logits_kernel(AppendParams p) {
  constexpr int kRowBytes = D * (BF16 ? 2 : 4);
  constexpr int kLanesPerRow = kRowBytes / 16;          // 8, 16 or 32
  constexpr int kRowsPerWave = KVC_WAVE / kLanesPerRow;  // rows covered by one wave load
  constexpr int kElems = BF16 ? 8 : 4;                   // values per 16-byte vector
  constexpr int kIters = (kKeysPerWg / kWaves) / kRowsPerWave;
  constexpr int kUnroll = 4;
  static_assert(kIters % kUnroll == 0, "unroll must divide the trip count");

  __shared__ float lds_logit[kHeadChunk][kKeysPerWg];
  __shared__ float red[kWaves];

  const int tid = threadIdx.x, lane = kvc::lane_id(), wave = tid / KVC_WAVE;
  const int kb = blockIdx.x, bg = blockIdx.y;  // bg = b * Hkv + kv head
  const int b = bg / p.Hkv, g = bg % p.Hkv;
  const int S = p.lengths ? min(max(p.lengths[b], 1), p.S) : p.S;
  const int k0 = kb * kKeysPerWg;
  if (k0 >= S) return;  // this sequence is shorter than the launch's upper bound (uniform exit)
  const int col = lane % kLanesPerRow, sub = lane / kLanesPerRow;

  for (int h0 = 0; h0 < p.G; h0 += kHeadChunk) {
    const int nh = min(kHeadChunk, p.G - h0);
    // this lane's slice of every query vector of the chunk
    float qv[kHeadChunk][kElems];
#pragma unroll
    for (int i = 0; i < kHeadChunk; ++i) {
      const int h = g * p.G + h0 + min(i, nh - 1);
      const vec16 x = *(const vec16*)(p.q_new + ((size_t)b * p.Hq + h) * kRowBytes + col * 16);
      unpack<BF16>(x, qv[i]);
    }
    for (int it0 = 0; it0 < kIters; it0 += kUnroll) {
      vec16 kx[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int key = k0 + wave * (kKeysPerWg / kWaves) + (it0 + u) * kRowsPerWave + sub;
        const bool fresh = FRESH && key >= S - 1;
        kx[u] = *(const vec16*)((fresh ? p.k_new + (size_t)bg * kRowBytes : key_row(p, b, g, bg, min(key, S - 1), kRowBytes)) +
                                col * 16);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        float kf[kElems];
        unpack<BF16>(kx[u], kf);
        const int lk = wave * (kKeysPerWg / kWaves) + (it0 + u) * kRowsPerWave + sub;
#pragma unroll
        for (int i = 0; i < kHeadChunk; ++i) {
          if (i < nh) {  // uniform
            float d = 0.0f;
#pragma unroll
            for (int e = 0; e < kElems; ++e) d = __builtin_fmaf(kf[e], qv[i][e], d);
#pragma unroll
            for (int off = kLanesPerRow / 2; off > 0; off >>= 1) d += __shfl_xor(d, off);
            if (col == 0) lds_logit[i][lk] = d * p.scale_log2;
          }
        }
      }
    }
    __syncthreads();
    // one key per thread: logits out (coalesced), block (max, sum of 2^(x - max)) per head
    const int key = k0 + tid;
    for (int i = 0; i < nh; ++i) {
      const int h = g * p.G + h0 + i;
      const float x = key < S ? lds_logit[i][tid] : kNegBig;
      if (key < S) p.logits[((size_t)b * p.Hq + h) * p.S + key] = x;
      const float m = block_max(x, red);
      const float l = block_sum(key < S ? __builtin_amdgcn_exp2f(x - m) : 0.0f, red);
      if (tid == 0) p.part[((size_t)b * p.Hq + h) * p.n_kb + kb] = make_float2(m, l);
    }
    __syncthreads();  // lds_logit is rewritten by the next chunk of heads
  }
  if (FRESH && S - 1 < k0 + kKeysPerWg && wave == 0) store_new_token(p, bg, S, lane, kRowBytes);
}

// bf16 / fp16: logits of kKeysPerWg keys x up to 32 heads per pass on the matrix cores.
// Bound by reading K.  Each of the eight waves copies its own 32 keys into LDS, multiplies, reduces and stores
// them by itself, so that it waits for nobody's loads but its own; the waves meet once per 32 heads, at the
// end, when their pairs are merged into one per workgroup.  Measured with D = 128, four waves sharing four
// 64-row tiles -> this: 8 sequences of 2048 keys, 8 KV heads 11.4 -> 9.8 us; 4 sequences of up to 32768 keys,
// 218 MB of K in scattered 16-token blocks 55.9 -> 48.2 (4.5 TB/s).  The KV heads run along the grid's y
// dimension: side by side, the last call takes 1 us more and dense fp32 caches up to 17 % more.
constexpr int kMfmaWaves = kKeysPerWg / 32;
template <int D, bool F16>
__global__ __launch_bounds__(kMfmaWaves * KVC_WAVE, 4) void append_logits_mfma_kernel(AppendParams p) {
  using C = Cfg<true, D>;
  constexpr int kLoads = C::kSubBytes / 1024;  // 1 KiB per wave instruction
  __shared__ __attribute__((aligned(1024))) char lds[kMfmaWaves][C::kSubBytes];
  __shared__ float2 red[2][kMfmaWaves][32];    // (two chunks of heads in turn)

  const int tid = threadIdx.x, lane = kvc::lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / KVC_WAVE);
  const int kb = blockIdx.x, bg = blockIdx.y;  // bg = b * Hkv + kv head
  const int b = bg / p.Hkv, g = bg % p.Hkv;
  const int S = p.lengths ? min(max(p.lengths[b], 1), p.S) : p.S;
  const int k0 = kb * kKeysPerWg;
  if (k0 >= S) return;  // this sequence is shorter than the launch's upper bound (uniform exit)
  const int row0 = k0 + 32 * wave;             // this wave's first key
  const bool live = row0 < S;                  // (rows past the end repeat the last one and are masked below)

  if (live) {
    // the 16-byte chunk that this lane copies with instruction j: the image of one 32-row sub-tile (tiles.h)
    int row[kLoads];
    uint32_t in_row[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int q = j * 64 + lane, line = q >> 4, logical = line * 16 + ((q & 15) ^ (line & 15));
      row[j] = min(logical / C::kChunksPerRow, S - 1 - row0);
      in_row[j] = (uint32_t)(logical % C::kChunksPerRow) * 16;
    }
    auto copy = [&](const char* base, size_t off, int j) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + off),
                                       (__attribute__((address_space(3))) void*)(lds[wave] + j * 1024), 16, 0, 0);
    };
    if (p.block_table) {
      const int* table = p.block_table + (size_t)b * (p.capacity / p.block_size);
      const char* pool = p.k + (size_t)g * C::kRowBytes;
      int blk[kLoads];  // (all entries on their way before the first is used)
#pragma unroll
      for (int j = 0; j < kLoads; ++j) blk[j] = table[(row0 + row[j]) / p.block_size];
#pragma unroll
      for (int j = 0; j < kLoads; ++j)
        copy(pool, ((size_t)blk[j] * p.block_size + (row0 + row[j]) % p.block_size) * p.Hkv * C::kRowBytes + in_row[j], j);
    } else {
      const char* rows = p.k + ((size_t)bg * p.capacity + row0) * C::kRowBytes;  // uniform
#pragma unroll
      for (int j = 0; j < kLoads; ++j) copy(rows, (uint32_t)row[j] * C::kRowBytes + in_row[j], j);
    }
  }
  const int n = lane & 31;  // result column of this lane = head inside the chunk
  // query vectors of a chunk of up to 32 heads, as the MFMA's column operand (issued before the
  // wait for the keys, so that the two latencies overlap)
  u32x4 qf[C::kSteps];
  auto load_q = [&](int h0) {
    const int nh = min(32, p.G - h0);
    const size_t bh = (size_t)b * p.Hq + g * p.G + h0 + min(n, nh - 1);
#pragma unroll
    for (int s = 0; s < C::kSteps; ++s) {
      u32x4 v = *(const u32x4*)(p.q_new + bh * C::kRowBytes + (s + (lane >> 5) * C::kSteps) * 16);
      if (n >= nh) v = u32x4{0u, 0u, 0u, 0u};
      qf[s] = v;
    }
  };
  load_q(0);
  wait_async_loads();  // (a wave reads only what it copied itself)
  if (p.k_new && live && S - 1 - row0 < 32) {  // the wave with the new token: its row in place of what the cache held
    if (lane < C::kChunksPerRow)
      *(vec16*)(lds[wave] + lds_chunk_offset<C>(S - 1 - row0, lane)) =
          *(const vec16*)(p.k_new + (size_t)bg * C::kRowBytes + lane * 16);
    kvc::wave_fence();
    store_new_token(p, bg, S, lane, C::kRowBytes);
  }

  const int off0 = lds_frag_offset0<C>(lane);
  const int key_base = row0 + 4 * (lane >> 5);  // + 8 * (r / 4) + r % 4
  for (int h0 = 0, turn = 0; h0 < p.G; h0 += 32, turn ^= 1) {
    const int nh = min(32, p.G - h0);
    const size_t bh = (size_t)b * p.Hq + g * p.G + h0 + min(n, nh - 1);
    if (h0 > 0) load_q(h0);
    float m = kNegBig, l = 0.0f;
    if (live) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
      for (int s = 0; s < C::kSteps; ++s) mma_step<true, F16>(acc, lds_frag<C>(lds[wave], off0, 0, s), qf[s]);
      // this lane: 16 keys of head n, those past the end masked
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = key_base + 8 * (r >> 2) + (r & 3);
        acc[r] = key < S ? acc[r] * p.scale_log2 : kNegBig;
        m = fmaxf(m, acc[r]);
      }
      m = fmaxf(m, __shfl_xor(m, 32));
#pragma unroll
      for (int r = 0; r < 16; ++r) l += __builtin_amdgcn_exp2f(acc[r] - m);  // masked keys: 2^-huge = 0
      l += __shfl_xor(l, 32);
      if (n < nh) {
        float* dst = p.logits + bh * p.S;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = key_base + 8 * (r >> 2) + (r & 3);
          if (key < S) dst[key] = acc[r];
        }
      }
    }
    if (lane < 32) red[turn][wave][n] = make_float2(m, l);
    __syncthreads();
    if (tid < nh) {
      float mt = red[turn][0][tid].x;  // (the first wave always has keys)
#pragma unroll
      for (int w = 1; w < kMfmaWaves; ++w) mt = fmaxf(mt, red[turn][w][tid].x);
      float lt = 0.0f;
#pragma unroll
      for (int w = 0; w < kMfmaWaves; ++w) lt += red[turn][w][tid].y * __builtin_amdgcn_exp2f(red[turn][w][tid].x - mt);
      p.part[((size_t)b * p.Hq + g * p.G + h0 + tid) * p.n_kb + kb] = make_float2(mt, lt);
    }
  }
}

// Bound by the logits and scores it moves, 4 * (G + 2) bytes a key and score row, and by the chain
// pairs -> normalisers -> probabilities in front of them: a wave merges one head's pairs by itself
// (no barrier per head), and the logits of KPT keys per thread, 256 apart, are in flight together, those of the
// row's first kFirst heads while the pairs are merged (four, or one where a row is one head: the registers of four
// would cost waves there, 4 to 8 % of the whole call).  A lane has four pairs on their way at a time: at 131072 keys and
// one head a row, the chain of pair loads one by one took 5 us of the call's 26.  Measured, whole calls, without and
// with the logits ahead: 4 sequences of up to 32768 keys, 32 heads in 8 groups (27 MB here) 67.3 -> 62.9 us, of
// which this kernel had 9.6; a decoding step of 8 sequences of 2048 keys 14.9 -> 13.6, of which it had 4.3.
template <int KPT, int kFirst>
__global__ __launch_bounds__(kThreads) void append_update_kernel(AppendParams p) {
  constexpr int kHeads = 32;  // heads whose normalisers are held at once
  __shared__ float lse2[kHeads];
  const int tid = threadIdx.x, lane = kvc::lane_id(), wave = tid / KVC_WAVE;
  const int row = blockIdx.y;  // row = b * Hs + r
  const int Hs = p.reduce_groups ? p.Hkv : p.Hq;
  const int b = row / Hs, r = row % Hs;
  const int h_first = p.reduce_groups ? r * p.G : r, n_heads = p.reduce_groups ? p.G : 1;
  const int S = p.lengths ? min(max(p.lengths[b], 1), p.S) : p.S;
  const int key0 = blockIdx.x * (kThreads * KPT);
  if (key0 >= S) return;
  const int n_kb = (S + kKeysPerWg - 1) / kKeysPerWg;  // blocks that wrote a pair for this sequence
  const float2* __restrict__ part = p.part;
  const float* __restrict__ logits = p.logits;
  float* __restrict__ dst = p.scores + (size_t)row * p.capacity;
  float acc[KPT], old[KPT];
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const int key = key0 + u * kThreads + tid;
    acc[u] = 0.0f;
    old[u] = key < S - 1 ? dst[key] : 0.0f;  // the new token's slot starts from nothing
  }
  // the first heads' logits are on their way while the pairs are merged
  float x[kFirst][KPT];
#pragma unroll
  for (int i = 0; i < kFirst; ++i)
    if (i < n_heads) {  // uniform
      const float* src = logits + ((size_t)b * p.Hq + h_first + i) * p.S;
#pragma unroll
      for (int u = 0; u < KPT; ++u) x[i][u] = src[min(key0 + u * kThreads + tid, S - 1)];
    }
  for (int h0 = 0; h0 < n_heads; h0 += kHeads) {
    const int nh = min(kHeads, n_heads - h0);
    if (h0 > 0) __syncthreads();
    for (int i = wave; i < nh; i += kWaves) {
      // row normaliser from the per-workgroup pairs
      const float2* src = part + ((size_t)b * p.Hq + h_first + h0 + i) * p.n_kb;
      float m = kNegBig, l = 0.0f;
      constexpr int kAhead = 4;  // pairs of a lane in flight together
      for (int j0 = lane; j0 < n_kb; j0 += kAhead * KVC_WAVE) {
        float2 ml[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int j = j0 + u * KVC_WAVE;
          ml[u] = src[min(j, n_kb - 1)];
          if (j >= n_kb) ml[u] = make_float2(kNegBig, 0.0f);
        }
        const float mn = fmaxf(fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x)), m);
        l *= __builtin_amdgcn_exp2f(m - mn);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) l += ml[u].y * __builtin_amdgcn_exp2f(ml[u].x - mn);
        m = mn;
      }
      const float mt = kvc::wave_max(m);
      l = kvc::wave_sum(l * __builtin_amdgcn_exp2f(m - mt));
      if (lane == 0) lse2[i] = mt + __builtin_amdgcn_logf(l);
    }
    __syncthreads();
    int done = 0;
    if (h0 == 0) {
#pragma unroll
      for (int i = 0; i < kFirst; ++i)
        if (i < nh) {  // uniform
#pragma unroll
          for (int u = 0; u < KPT; ++u) acc[u] += __builtin_amdgcn_exp2f(x[i][u] - lse2[i]);
        }
      done = kFirst;
    }
    for (int i = done; i < nh; ++i) {  // heads ascending
      const float* src = logits + ((size_t)b * p.Hq + h_first + h0 + i) * p.S;
      const float ref = lse2[i];
#pragma unroll
      for (int u = 0; u < KPT; ++u) {
        const int key = key0 + u * kThreads + tid;
        if (key < S) acc[u] += __builtin_amdgcn_exp2f(src[key] - ref);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const int key = key0 + u * kThreads + tid;
    if (key < S) dst[key] = old[u] + acc[u];
  }
}

size_t logits_bytes(const kvcrush_shape* s) {
  return kvc::align_up((size_t)s->B * s->Hq * s->S * sizeof(float), 256);
}

int key_blocks(const kvcrush_shape* s) { return (s->S + kKeysPerWg - 1) / kKeysPerWg; }

size_t part_bytes(const kvcrush_shape* s) {
  return kvc::align_up((size_t)s->B * s->Hq * key_blocks(s) * sizeof(float2), 256);
}

bool append_shape_ok(const kvcrush_shape* s, int capacity) {
  if (!s) return false;
  if (s->B < 1 || s->Hq < 1 || s->Hkv < 1 || s->S < 1 || s->D < 1 || capacity < s->S) return false;
  if (s->Hq % s->Hkv != 0) return false;
  if (s->dtype != KVCRUSH_F32 && s->dtype != KVCRUSH_BF16 && s->dtype != KVCRUSH_F16) return false;
  if (s->reduce_groups != 0 && s->reduce_groups != 1) return false;
  if (s->obs_window != 0) return false;
  if (!(s->softmax_scale >= 0.0f) || s->softmax_scale > 1.0e6f) return false;  // also rejects NaN
  return true;
}

// Keys per thread of the update: four where that still leaves four workgroups to a compute unit.
constexpr int kUpdateKeys = 4;
constexpr long long kUpdateWorkgroups = 1024;
template <int FIRST>
kvcrush_status launch_update(const AppendParams& p, hipStream_t stream) {
  const int rows = p.B * (p.reduce_groups ? p.Hkv : p.Hq);
  const int wide = (p.S + kThreads * kUpdateKeys - 1) / (kThreads * kUpdateKeys);
  if ((long long)wide * rows >= kUpdateWorkgroups)
    return kvc::launch(append_update_kernel<kUpdateKeys, FIRST>, dim3(wide, rows), dim3(kThreads), 0, stream, p);
  return kvc::launch(append_update_kernel<1, FIRST>, dim3((p.S + kThreads - 1) / kThreads, rows), dim3(kThreads), 0, stream, p);
}

template <bool BF16, int D, bool F16 = false>
kvcrush_status launch_append(const AppendParams& p, hipStream_t stream) {
  const dim3 grid(p.n_kb, p.B * p.Hkv);
  kvcrush_status st;
  if constexpr (BF16) {
    st = kvc::launch(append_logits_mfma_kernel<D, F16>, grid, dim3(kMfmaWaves * KVC_WAVE), 0, stream, p);
  } else {
    st = p.k_new ? kvc::launch(append_logits_kernel<BF16, D, true>, grid, dim3(kThreads), 0, stream, p)
                 : kvc::launch(append_logits_kernel<BF16, D, false>, grid, dim3(kThreads), 0, stream, p);
  }
  if (st != KVCRUSH_OK) return st;
  return p.reduce_groups && p.G > 1 ? launch_update<4>(p, stream) : launch_update<1>(p, stream);
}

}  // namespace

extern "C" size_t kvcrush_scores_append_workspace(const kvcrush_shape* shape, int32_t capacity) {
  if (!append_shape_ok(shape, capacity)) return 0;
  return logits_bytes(shape) + part_bytes(shape);
}

namespace {
kvcrush_status append_entry(const kvcrush_shape* shape, int32_t capacity, const int32_t* lengths, const void* q_new,
                            const void* k, const int32_t* block_table, int32_t block_size, const void* k_new,
                            const void* v_new, void* v, float* scores, void* workspace, size_t workspace_bytes,
                            void* hip_stream) {
  if (!append_shape_ok(shape, capacity)) return KVCRUSH_ERR_INVALID_ARG;
  if (block_table && (block_size < 1 || capacity % block_size != 0)) return KVCRUSH_ERR_INVALID_ARG;
  if (shape->D != 64 && shape->D != 128) return KVCRUSH_ERR_UNSUPPORTED;
  if ((long long)shape->B * shape->Hq > 65535) return KVCRUSH_ERR_UNSUPPORTED;
  if (!q_new || !k || !scores) return KVCRUSH_ERR_INVALID_ARG;
  if (!kvc::aligned16(q_new) || !kvc::aligned16(k) || !kvc::aligned16(scores))
    return KVCRUSH_ERR_INVALID_ARG;
  if (!workspace || !kvc::aligned16(workspace) ||
      workspace_bytes < logits_bytes(shape) + part_bytes(shape))
    return KVCRUSH_ERR_WORKSPACE;
  AppendParams p;
  p.q_new = (const char*)q_new;
  p.k = (const char*)k;
  p.scores = scores;
  p.logits = (float*)workspace;
  p.part = (float2*)((char*)workspace + logits_bytes(shape));
  p.lengths = lengths;
  p.block_table = block_table;
  p.block_size = block_table ? block_size : 1;
  p.k_new = (const char*)k_new;
  p.v_new = (const char*)v_new;
  p.k_slot = (char*)k;
  p.v_slot = (char*)v;
  p.B = shape->B;
  p.Hq = shape->Hq;
  p.Hkv = shape->Hkv;
  p.S = shape->S;
  p.capacity = capacity;
  p.G = shape->Hq / shape->Hkv;
  p.reduce_groups = shape->reduce_groups;
  p.n_kb = key_blocks(shape);
  p.scale_log2 = (float)(1.4426950408889634 *
                         (shape->softmax_scale != 0.0f ? (double)shape->softmax_scale : 1.0 / sqrt((double)shape->D)));
  hipStream_t stream = (hipStream_t)hip_stream;
  if (shape->dtype == KVCRUSH_F16)
    return shape->D == 128 ? launch_append<true, 128, true>(p, stream) : launch_append<true, 64, true>(p, stream);
  const bool bf16 = shape->dtype == KVCRUSH_BF16;
  if (bf16 && shape->D == 128) return launch_append<true, 128>(p, stream);
  if (bf16 && shape->D == 64) return launch_append<true, 64>(p, stream);
  if (!bf16 && shape->D == 128) return launch_append<false, 128>(p, stream);
  return launch_append<false, 64>(p, stream);
}
}  // namespace

extern "C" kvcrush_status kvcrush_scores_append(const kvcrush_shape* shape, int32_t capacity,
                                                const int32_t* lengths, const void* q_new,
                                                const void* k, const int32_t* block_table,
                                                int32_t block_size, float* scores, void* workspace,
                                                size_t workspace_bytes, void* hip_stream) {
  return append_entry(shape, capacity, lengths, q_new, k, block_table, block_size, nullptr, nullptr, nullptr, scores,
                      workspace, workspace_bytes, hip_stream);
}

extern "C" kvcrush_status kvcrush_decode_step(const kvcrush_shape* shape, int32_t capacity, const void* q_new,
                                              const void* k_new, const void* v_new, void* k, void* v, float* scores,
                                              void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!k_new || !v_new || !v) return KVCRUSH_ERR_INVALID_ARG;
  if (!kvc::aligned16(k_new) || !kvc::aligned16(v_new) || !kvc::aligned16(v)) return KVCRUSH_ERR_INVALID_ARG;
  return append_entry(shape, capacity, nullptr, q_new, k, nullptr, 0, k_new, v_new, v, scores, workspace, workspace_bytes,
                      hip_stream);
}
