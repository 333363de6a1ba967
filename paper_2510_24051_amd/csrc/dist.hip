// Next-token distribution: softmax over the whole vocabulary and exact top-k.  Two pairs of kernels, so that a handful of
// rows still fills the chip; group_threads says which takes a call:
//   topk_groups + topk_select : where the vocabulary has 2 k groups of 16 logits, which is nearly every call (described
//                there).
//   topk_chunk + topk_merge : the rest, at most four chunks of 8192 logits (k above a 32nd of the vocabulary, or a
//                vocabulary below one chunk).
//     topk_chunk : grid (rows, chunks).  A workgroup takes one chunk (<= 8192 logits) of a row, keeps its
//                order-preserving 32-bit keys in registers, reduces the chunk max and sum of exponentials with
//                wavefront reductions, finds the chunk's k-th largest key by radix select and writes the
//                chunk's top-k candidates as 64-bit (key, ~id) composites.
//     topk_merge : grid (rows).  Combines the chunk maxima/sums into the row's softmax normaliser, radix-selects
//                the k largest composites among chunks*k candidates (composites are unique, so ties on the
//                logit resolve to the lower id), sorts those k with a bitonic network and writes ids and
//                probabilities of the full distribution.
//
// Radix select, 8 bits per pass.  Logits share a handful of sign/exponent values, so a histogram of the top
// byte would hammer a few LDS addresses with atomics; instead the top byte is found by walking the byte values
// downward from the maximum's and counting matches in registers (a few steps for any realistic distribution).
// The lower bytes only concern the few keys that share the selected top byte: LDS histogram with atomics.
#include <type_traits>

#include "internal.h"

#define TC_THREADS 512
// keys per thread of the chunk kernel: 16 (chunks of at most 8192 logits) or, when there are enough rows to fill
// the chip with half as many workgroups, 32 (16384 logits): half the block-wide synchronisation per logit
#define TC_LIST 2048  // composites the chunk kernel's short-list selection holds (4 per thread)
#define TM_THREADS 1024
#define TM_PER 4  // composites per thread: at most 4096 candidates per row, four chunks of 1024 (see the head of this file)

__device__ __forceinline__ uint32_t order_key(float z) {
  uint32_t u = __float_as_uint(z);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Sum of one unsigned per thread over the workgroup (all threads get the result).  red: [THREADS / 64] words.
template <int THREADS>
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();  // previous use of red is over
  if (lane == 0) red[wave] = v;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) t += red[w];
  return t;
}

// Top byte of the need-th largest key.  On return *out_b is that byte, *out_need what is still needed among the keys
// that carry it and *out_cnt how many keys carry it (need - *out_need keys have a larger top byte).
// The byte values are walked downward from the maximum's, counting matches in registers: logits of one row share a
// handful of sign/exponent values, so the k-th largest is almost always found within a step or two.  When it is not
// after WALK_STEPS values (a positive maximum over a negative k-th largest lies 128 byte values apart, all the
// exponents of tiny magnitudes in between being empty), the rest of the range is bisected instead: at most eight
// more counts, whatever the distribution.  Every count is uniform over the workgroup, so the control flow is too.
#define WALK_STEPS 4
template <typename KeyT, int PER, int THREADS>
__device__ __forceinline__ void walk_top_byte(const KeyT (&keys)[PER], uint32_t need, int top_byte_max, uint32_t* red,
                                              int* out_b, uint32_t* out_need, uint32_t* out_cnt) {
  constexpr int TOP = sizeof(KeyT) * 8 - 8;
  auto count_in = [&](int lo, int hi) {  // keys whose top byte lies in [lo, hi]
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int tb = (int)(keys[i] >> TOP);
      c += (tb >= lo && tb <= hi && keys[i] != 0) ? 1u : 0u;
    }
    return block_sum<THREADS>(c, red);
  };
  int b = top_byte_max;
  uint32_t cnt = 0;
  bool found = false;
  for (int step = 0; step < WALK_STEPS; ++step, --b) {
    cnt = count_in(b, b);
    if (cnt >= need || b == 0) { found = true; break; }
    need -= cnt;
  }
  if (!found) {
    // the answer is the largest byte value t <= hi with count_in(t, hi) >= need (0 when there are fewer keys)
    const int hi = b;
    int lo = 0, up = hi;
    while (lo < up) {
      const int mid = (lo + up + 1) >> 1;
      if (count_in(mid, hi) >= need) lo = mid;
      else up = mid - 1;
    }
    b = lo;
    const uint32_t above = b < hi ? count_in(b + 1, hi) : 0u;
    need -= above;
    cnt = count_in(b, b);
  }
  *out_b = b;
  *out_need = need;
  *out_cnt = cnt;
}

// The lower bytes of the need-th largest among the keys whose top byte is b (eq of them), eight bits per pass with
// an LDS histogram; keys with another top byte take no part.  On return: *out_kth the selected value, *out_need
// how many keys equal to it belong to the top set, *out_eq how many keys equal it in total.  With
// stop_at_shift > 0 the search stops before the passes below that shift when every key sharing the bits decided
// so far is needed anyway (then the low bits of *out_kth are 0 and it is a lower bound of exactly the selected
// set).  hist: 2 x 256 words (the passes alternate between the halves: while the first wave scans one, other
// threads clear the other, so a pass costs two barriers), red: THREADS / 64 words of LDS.
template <typename KeyT, int PER, int THREADS>
__device__ __forceinline__ void select_lower_bytes(const KeyT (&keys)[PER], int b, uint32_t need, uint32_t eq,
                                                   int stop_at_shift, uint32_t* hist, KeyT* sh_prefix,
                                                   uint32_t* sh_need, uint32_t* sh_eq, KeyT* out_kth,
                                                   uint32_t* out_need, uint32_t* out_eq) {
  static_assert(THREADS >= 512, "threads 256..511 clear the idle histogram");
  constexpr int TOP = sizeof(KeyT) * 8 - 8;
  const int tid = threadIdx.x, lane = tid & 63;
  KeyT prefix = (KeyT)b << TOP;
  __syncthreads();  // earlier users of hist and of the shared results are done
  if (tid < 512) hist[tid] = 0u;
  __syncthreads();
  int pass = 0;
  for (int shift = TOP - 8; shift >= 0; shift -= 8, ++pass) {
    if (stop_at_shift > 0 && shift < stop_at_shift && eq == need) break;
    uint32_t* h = hist + (pass & 1) * 256;
    const KeyT hi_mask = ~(KeyT)0 << (shift + 8);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if ((keys[i] & hi_mask) == prefix && keys[i] != 0) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 0xFFu], 1u);
    __syncthreads();
    if (tid < 64) {
      // lane L owns bins 255-4L .. 252-4L (descending); a wave scan gives the number of keys in higher bins
      const int b0 = 255 - 4 * lane;
      const uint32_t h0 = h[b0], h1 = h[b0 - 1], h2 = h[b0 - 2], h3 = h[b0 - 3];
      const uint32_t tot = h0 + h1 + h2 + h3;
      uint32_t incl = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      const uint32_t excl = incl - tot;
      if (excl < need && need <= incl) {
        uint32_t acc = excl, hb = h0;
        int bb = b0;
        if (acc + h0 < need) { acc += h0; bb = b0 - 1; hb = h1;
          if (acc + h1 < need) { acc += h1; bb = b0 - 2; hb = h2;
            if (acc + h2 < need) { acc += h2; bb = b0 - 3; hb = h3; } } }
        *sh_need = need - acc;
        *sh_eq = hb;
        *sh_prefix = prefix | ((KeyT)bb << shift);
      }
    } else if (tid >= 256 && tid < 512) {
      hist[((pass + 1) & 1) * 256 + (tid - 256)] = 0u;  // scanned a pass ago; the next pass counts into it
    }
    __syncthreads();
    need = *sh_need;
    eq = *sh_eq;
    prefix = *sh_prefix;
  }
  *out_kth = prefix;
  *out_need = need;
  *out_eq = eq;
}

// k-th largest of the workgroup's keys (PER per thread in registers, key 0 = padding below every real key):
// the top byte by walking down from `top_byte_max` (the top byte of the largest key), the rest by
// select_lower_bytes.
template <typename KeyT, int PER, int THREADS>
__device__ __forceinline__ void select_kth(const KeyT (&keys)[PER], uint32_t need, int top_byte_max, int stop_at_shift,
                                           uint32_t* hist, uint32_t* red, KeyT* sh_prefix, uint32_t* sh_need,
                                           uint32_t* sh_eq, KeyT* out_kth, uint32_t* out_need, uint32_t* out_eq) {
  int b;
  uint32_t cnt;
  walk_top_byte<KeyT, PER, THREADS>(keys, need, top_byte_max, red, &b, &need, &cnt);
  select_lower_bytes<KeyT, PER, THREADS>(keys, b, need, cnt, stop_at_shift, hist, sh_prefix, sh_need, sh_eq, out_kth,
                                         out_need, out_eq);
}

template <int TC_PER>
__global__ __launch_bounds__(TC_THREADS) void topk_chunk_kernel(const float* __restrict__ logits, int V, int chunk_len,
                                                                int k, float inv_temp,
                                                                unsigned long long* __restrict__ cand,
                                                                float* __restrict__ stats) {
  __shared__ uint32_t hist[512];
  __shared__ uint32_t red[TC_THREADS / 64];
  __shared__ float fred[TC_THREADS / 64];
  __shared__ uint32_t sh_prefix, sh_need, sh_eq, sh_count, sh_count_eq, sh_wave_off[TC_THREADS / 64 + 1];
  __shared__ unsigned long long sh_prefix64;
  __shared__ unsigned long long list[TC_LIST];
  __shared__ float sh_max;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blockIdx.x, chunk = blockIdx.y, n_chunks = gridDim.y;
  const int start = chunk * chunk_len;
  const int n = min(chunk_len, V - start);
  const float* z = logits + (int64_t)row * V + start;

  // thread t holds logits t*4 + j*(4*THREADS) + e (e < 4, j < PER/4): 16-byte loads, ids recoverable from (j, e)
  uint32_t keys[TC_PER];
  float mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < TC_PER / 4; ++j) {
    const int i = tid * 4 + j * 4 * TC_THREADS;  // start, n and V are multiples of 4
    f32x4 v = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    const bool in = i < n;
    if (in) v = *reinterpret_cast<const f32x4*>(z + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      keys[j * 4 + e] = in ? order_key(v[e]) : 0u;
      mx = fmaxf(mx, v[e]);
    }
  }
  mx = wave_max(mx);
  if (lane == 0) fred[wave] = mx;
  __syncthreads();
  if (tid == 0) {
    float m = fred[0];
    for (int w = 1; w < TC_THREADS / 64; ++w) m = fmaxf(m, fred[w]);
    sh_max = m;
    sh_count = 0u;
    sh_count_eq = 0u;
  }
  __syncthreads();
  const float cmax = sh_max;
  // exponentials on the hardware's base-2 instruction (1 ulp): arguments are <= 0, nothing to guard
  const float c2 = inv_temp * 1.44269504088896340736f;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < TC_PER; ++i)
    if (keys[i] != 0u) sum += __builtin_amdgcn_exp2f((key_to_float(keys[i]) - cmax) * c2);
  sum = wave_sum(sum);
  __syncthreads();
  if (lane == 0) fred[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
    for (int w = 0; w < TC_THREADS / 64; ++w) t += fred[w];
    stats[((int64_t)row * n_chunks + chunk) * 2] = cmax;
    stats[((int64_t)row * n_chunks + chunk) * 2 + 1] = t;
  }
  const int kc = min(k, n);  // candidates this chunk contributes
  unsigned long long* out = cand + ((int64_t)row * n_chunks + chunk) * k;
  auto comp_of = [&](int i) {
    const int id = start + tid * 4 + (i >> 2) * 4 * TC_THREADS + (i & 3);
    return ((unsigned long long)keys[i] << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)id);
  };
  // Usually only a few per cent of the keys share the top byte of the k-th largest or lie above it.  Those are
  // collected as composites in LDS (per-thread counts, a wave scan, one atomic per wave), and the selection runs
  // on that short list, at most TC_LIST / TC_THREADS composites per thread; composites are unique, so equal
  // logits at the cut resolve to the lower ids without a separate pass.  Longer lists (e.g. many equal logits)
  // take the selection over all keys in registers below.
  const int top_byte = (int)(order_key(cmax) >> 24);
  int wb;
  uint32_t w_need, w_cnt;
  walk_top_byte<uint32_t, TC_PER, TC_THREADS>(keys, (uint32_t)kc, top_byte, red, &wb, &w_need, &w_cnt);
  const uint32_t n_list = (uint32_t)kc - w_need + w_cnt;  // keys whose top byte is wb or larger
  if (n_list <= TC_LIST) {
    uint32_t mine = 0u;
#pragma unroll
    for (int i = 0; i < TC_PER; ++i) mine += ((int)(keys[i] >> 24) >= wb && keys[i] != 0u) ? 1u : 0u;
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    uint32_t base = 0u;
    if (lane == 63 && incl) base = atomicAdd(&sh_count_eq, incl);  // sh_count_eq: entries of the list so far
    uint32_t pos = __shfl(base, 63) + incl - mine;
#pragma unroll
    for (int i = 0; i < TC_PER; ++i)
      if ((int)(keys[i] >> 24) >= wb && keys[i] != 0u) {
        if (pos < TC_LIST) list[pos] = comp_of(i);
        ++pos;
      }
    __syncthreads();
    unsigned long long c[TC_LIST / TC_THREADS];
#pragma unroll
    for (int j = 0; j < TC_LIST / TC_THREADS; ++j) {
      const uint32_t idx = tid + j * TC_THREADS;
      c[j] = idx < n_list ? list[idx] : 0ull;
    }
    unsigned long long kth64;
    uint32_t need64, eq64;
    // the walk above already found the top byte and what is still needed among the composites that carry it
    select_lower_bytes<unsigned long long, TC_LIST / TC_THREADS, TC_THREADS>(c, wb, w_need, w_cnt, 32, hist, &sh_prefix64,
                                                                             &sh_need, &sh_eq, &kth64, &need64, &eq64);
    // exactly kc composites are >= kth64
#pragma unroll
    for (int j = 0; j < TC_LIST / TC_THREADS; ++j)
      if (c[j] >= kth64 && c[j] != 0ull) {
        const uint32_t p2 = atomicAdd(&sh_count, 1u);
        if (p2 < (uint32_t)kc) out[p2] = c[j];
      }
    for (int i = kc + tid; i < k; i += TC_THREADS) out[i] = 0ull;  // short chunk: pad (a zero never wins)
    return;
  }
  uint32_t kth, need_eq, eq_total;
  select_kth<uint32_t, TC_PER, TC_THREADS>(keys, (uint32_t)kc, (int)(order_key(cmax) >> 24), 0, hist, red, &sh_prefix,
                                           &sh_need, &sh_eq, &kth, &need_eq, &eq_total);
  // keys above kth: any order, slots [need_eq, kc); keys equal to kth: slots [0, need_eq), lowest ids first when
  // only some of them are taken
  const bool split_tie = eq_total != need_eq;
#pragma unroll
  for (int i = 0; i < TC_PER; ++i) {
    if (keys[i] > kth) {
      const uint32_t pos = need_eq + atomicAdd(&sh_count, 1u);
      if (pos < (uint32_t)kc) out[pos] = comp_of(i);  // kc - need_eq keys by construction
    } else if (!split_tie && keys[i] == kth && keys[i] != 0u) {
      const uint32_t pos = atomicAdd(&sh_count_eq, 1u);
      if (pos < need_eq) out[pos] = comp_of(i);
    }
  }
  if (split_tie) {
    // ids ascend with (j, thread, e): walk j outermost; within a j the workgroup's ids are tid*4 + e
    uint32_t eq_seen = 0u;
#pragma unroll  // keys[] must only be indexed by constants, or the array is placed in scratch memory
    for (int j = 0; j < TC_PER / 4; ++j) {
      if (eq_seen >= need_eq) break;  // eq_seen is uniform across the workgroup
      uint32_t mine = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) mine += (keys[j * 4 + e] == kth && keys[j * 4 + e] != 0u) ? 1u : 0u;
      uint32_t incl = mine;  // inclusive prefix over the wave, then wave offsets through LDS
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      __syncthreads();
      if (lane == 63) sh_wave_off[wave + 1] = incl;
      __syncthreads();
      if (tid == 0) {
        sh_wave_off[0] = 0u;
        for (int w = 0; w < TC_THREADS / 64; ++w) sh_wave_off[w + 1] += sh_wave_off[w];
      }
      __syncthreads();
      uint32_t pos = eq_seen + sh_wave_off[wave] + incl - mine;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (keys[j * 4 + e] == kth && keys[j * 4 + e] != 0u) {
          if (pos < need_eq) out[pos] = comp_of(j * 4 + e);
          ++pos;
        }
      eq_seen += sh_wave_off[TC_THREADS / 64];
    }
  }
  for (int i = kc + tid; i < k; i += TC_THREADS) out[i] = 0ull;  // short chunk: pad (a zero never wins)
}

template <int PER>  // composites per thread: the smaller of 2 and 4 that holds the row's candidates
__global__ __launch_bounds__(TM_THREADS) void topk_merge_kernel(int n_chunks, int k, float inv_temp,
                                                                const unsigned long long* __restrict__ cand,
                                                                const float* __restrict__ stats, int n2,
                                                                int32_t* __restrict__ out_ids,
                                                                float* __restrict__ out_probs) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  unsigned long long* top = reinterpret_cast<unsigned long long*>(smem_raw);  // [n2 >= k]
  __shared__ uint32_t hist[512];
  __shared__ uint32_t red[TM_THREADS / 64];
  __shared__ unsigned long long sh_prefix;
  __shared__ uint32_t sh_need, sh_eq, sh_count;
  __shared__ uint32_t rank_s[256];
  __shared__ float sh_max, sh_sum;
  const int tid = threadIdx.x;
  const int row = blockIdx.x;
  const int n = n_chunks * k;
  unsigned long long c[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int idx = tid + i * TM_THREADS;
    c[i] = idx < n ? cand[(int64_t)row * n + idx] : 0ull;
  }
  if (tid == 0) {
    float gm = -INFINITY;
    for (int j = 0; j < n_chunks; ++j) gm = fmaxf(gm, stats[((int64_t)row * n_chunks + j) * 2]);
    float s = 0.f;
    for (int j = 0; j < n_chunks; ++j)
      s += stats[((int64_t)row * n_chunks + j) * 2 + 1] * expf((stats[((int64_t)row * n_chunks + j) * 2] - gm) * inv_temp);
    sh_max = gm;
    sh_sum = s;
    sh_count = 0u;
  }
  for (int i = tid; i < n2; i += TM_THREADS) top[i] = 0ull;
  __syncthreads();
  const int top_byte = (int)(order_key(sh_max) >> 24);  // the row maximum is among the candidates
  unsigned long long kth;
  uint32_t need_eq, eq_total;
  // the id half of a composite only matters when equal logits straddle the cut: stop after the key half when
  // every candidate sharing the selected key is needed
  select_kth<unsigned long long, PER, TM_THREADS>(c, (uint32_t)k, top_byte, 32, hist, red, &sh_prefix, &sh_need,
                                                     &sh_eq, &kth, &need_eq, &eq_total);
  // composites are unique: exactly k of them are >= kth
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (c[i] >= kth && c[i] != 0ull) {
      const uint32_t pos = atomicAdd(&sh_count, 1u);
      if (pos < (uint32_t)n2) top[pos] = c[i];  // exactly k by construction; never write past the buffer
    }
  __syncthreads();
  const float inv_sum = 1.0f / sh_sum, gmax = sh_max;
  auto emit = [&](int slot, unsigned long long v) {
    const int id = (int)(0xFFFFFFFFu - (uint32_t)(v & 0xFFFFFFFFull));
    out_ids[(int64_t)row * k + slot] = id;
    out_probs[(int64_t)row * k + slot] = expf((key_to_float((uint32_t)(v >> 32)) - gmax) * inv_temp) * inv_sum;
  };
  if (n2 <= 256) {
    // Few survivors: every composite finds its place by counting the larger ones (they are unique, so the counts
    // are a permutation).  TM_THREADS / n2 threads share the comparisons of one element; the threads of a wave
    // read the same composite in every step (an LDS broadcast).  Two barriers instead of one per bitonic stage.
    const int parts = TM_THREADS / n2, e = tid & (n2 - 1), part = tid / n2;
    if (tid < n2) rank_s[tid] = 0u;
    __syncthreads();
    if (e < k) {
      const unsigned long long mine = top[e];
      uint32_t larger = 0u;
      for (int j = part; j < k; j += parts) larger += top[j] > mine ? 1u : 0u;
      if (larger) atomicAdd(&rank_s[e], larger);
    }
    __syncthreads();
    if (tid < k) emit((int)rank_s[tid], top[tid]);
    return;
  }
  for (int size = 2; size <= n2; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < n2 / 2; i += TM_THREADS) {
        const int lo = ((i & ~(stride - 1)) << 1) | (i & (stride - 1));  // stride is a power of two
        const int hi = lo + stride;
        const bool desc = ((lo & size) == 0);
        const unsigned long long a = top[lo], b = top[hi];
        if ((a < b) == desc) {
          top[lo] = b;
          top[hi] = a;
        }
      }
      __syncthreads();
    }
  }
  for (int i = tid; i < k; i += TM_THREADS) emit(i, top[i]);
}

// ------------------------------------------------------------------------------------------------
// Top-k by group maxima (vocabularies of at least 2 k groups of 16): two kernels that sort nothing until few are left
//
//   topk_groups : grid (rows, chunks of 8192 logits).  Reads the logits once and leaves, per group of `16 m` of them (the 16
//                 of m neighbouring threads), the largest key and the sum of exponentials relative to it.  Bound by the
//                 read (64 x 128256: 32.8 MB).
//   topk_select : grid (rows).  At least k logits reach the k-th largest group maximum, so only groups whose maximum reaches
//                 it, and in them only the logits that do, can be among the top k.  A lower bound T of that maximum that
//                 hardly more than k groups reach comes from a histogram of the maxima between the smallest and the
//                 largest, refined where a bin holds too many.  Where it ends at one key that many maxima equal (rows with
//                 equal logits, a masked row with fewer than k groups left), the groups that exceed it, fewer than k, are
//                 taken, and of those that equal it the ones of the first chunks that hold enough: equal logits win by the
//                 lower id, and every id of a chunk lies below those of the next.  The groups taken are read again (k of
//                 them, 32 KiB of the row's 513 at k = 256) and the logits that reach T (1.2 to 1.4 k of them) go to a list as
//                 their distance from T in (key, ~id), which is unique, so equal logits come in the order of their ids.
//                 A list that overflows is cut by the same histogram over those distances.  Each entry finds its place
//                 by counts over ever finer bins, as many bins as entries in each crowded one.
// Measured against topk_chunk + topk_merge, which select each chunk's k first (both kernels between events, 128256 logits):
// 64 ordinary rows k = 256 41.7 -> 20.0 us, k = 512 47.5 -> 21.8, 256 rows k = 256 105 -> 43; of 32000, 64 rows k = 256 21.9 ->
// 14.8.  Rows of other kinds, 64 of them, k = 256: all logits equal 122 -> 30, a quarter tied at the top 62 -> 34, fewer than
// k unmasked 161 -> 50, one logit far above the rest 74 -> 35, ascending with the id 64 -> 34 (one such row, k = 50: 27 -> 32).
// (Selecting every group that reaches T, and counting the overflowing ones from the top of the key range, one atomic each:
// equal logits 650, a quarter tied 275.)  What is left of topk_select is latency: three dependent reads of memory and a dozen
// barriers with one workgroup per row.
// ------------------------------------------------------------------------------------------------
#define TG_THREADS 512
#define TG_CHUNK (TG_THREADS * 16)
#define TS_THREADS 1024
#define TS_LIST 2048
#define TS_PER (TS_LIST / TS_THREADS)
#define TS_COUNT 32

__global__ __launch_bounds__(TG_THREADS) void topk_groups_kernel(const float* __restrict__ logits, int V, int m, float inv_temp,
                                                                 uint2* __restrict__ groups) {
  __shared__ uint32_t kred[TG_THREADS / 64];
  __shared__ float sred[TG_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blockIdx.x, chunk = blockIdx.y;
  const int n = min(TG_CHUNK, V - chunk * TG_CHUNK);
  const float* z = logits + (int64_t)row * V + chunk * TG_CHUNK;
  f32x4 v[4];
  uint32_t best = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = tid * 4 + j * 4 * TG_THREADS;  // n and V are multiples of 4
    v[j] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (i < n) v[j] = *reinterpret_cast<const f32x4*>(z + i);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (tid * 4 + j * 4 * TG_THREADS < n)
#pragma unroll
      for (int e = 0; e < 4; ++e) best = max(best, order_key(v[j][e]));
  for (int o = 1; o < m && o < 64; o <<= 1) best = max(best, (uint32_t)__shfl_xor((int)best, o));
  const int w0 = m > 64 ? wave & ~(m / 64 - 1) : wave, w1 = m > 64 ? w0 + m / 64 : w0;  // the group's waves where it has several
  if (m > 64) {
    if (lane == 0) kred[wave] = best;
    __syncthreads();
    for (int w = w0; w < w1; ++w) best = max(best, kred[w]);
  }
  const float gm = best ? key_to_float(best) : -INFINITY;
  const float c2 = inv_temp * 1.44269504088896340736f;
  float sum = 0.f;
  if (gm != -INFINITY) {  // (padding, and a logit of -inf among others, add 2^-inf = 0)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) sum += __builtin_amdgcn_exp2f((v[j][e] - gm) * c2);
  }
  for (int o = 1; o < m && o < 64; o <<= 1) sum += __shfl_xor(sum, o);
  if (m > 64) {
    if (lane == 0) sred[wave] = sum;
    __syncthreads();
    sum = 0.f;
    for (int w = w0; w < w1; ++w) sum += sred[w];
  }
  if (tid % m == 0) groups[((int64_t)row * gridDim.y + chunk) * (TG_THREADS / m) + tid / m] = uint2{best, __float_as_uint(sum)};
}

// Where the bin of the `need`-th largest of 1024 histogram counts lies: *bin, and *above, how many lie in larger bins (bin 0
// and everything above it when there are fewer than `need`).  Every thread returns the same.  hist must be complete (a
// barrier behind its counts) and is cleared on return for the next count.
__device__ __forceinline__ void cut_bin(uint32_t* hist, uint32_t need, uint32_t* wtot, uint32_t* sh, uint32_t* bin, uint32_t* above,
                                        uint32_t* in_bin) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t c = hist[1023 - tid];  // descending bins
  uint32_t incl = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  uint32_t before = 0u;
#pragma unroll
  for (int w = 0; w < TS_THREADS / 64; ++w) before += w < wave ? wtot[w] : 0u;
  const uint32_t excl = before + incl - c;
  if ((excl < need && need <= excl + c) || (tid == 1023 && excl + c < need)) {
    sh[0] = 1023 - tid;
    sh[1] = excl;
    sh[2] = c;
  }
  hist[1023 - tid] = 0u;
  __syncthreads();
  *bin = sh[0];
  *above = sh[1];
  *in_bin = sh[2];
}

// A place behind *counter for every lane that takes one, one LDS atomic per wave.
__device__ __forceinline__ uint32_t wave_append(bool take, uint32_t* counter) {
  const unsigned long long mask = __builtin_amdgcn_ballot_w64(take);
  if (mask == 0ull) return 0u;
  const int leader = __ffsll(mask) - 1;
  uint32_t base = 0u;
  if ((int)(threadIdx.x & 63) == leader) base = atomicAdd(counter, (uint32_t)__popcll(mask));
  return (uint32_t)__builtin_amdgcn_readlane((int)base, leader) +
         __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// One more in hist[bin] for every lane that counts.  Lanes that share the first one's bin (many equal values) take one LDS
// atomic together instead of one each at one address.
__device__ __forceinline__ void wave_count(bool counts, uint32_t bin, uint32_t* hist) {
  const unsigned long long mask = __builtin_amdgcn_ballot_w64(counts);
  if (mask == 0ull) return;
  const int leader = __ffsll(mask) - 1;
  const bool same = counts && bin == (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
  const unsigned long long together = __builtin_amdgcn_ballot_w64(same);
  if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[bin], (uint32_t)__popcll(together));
  else if (counts && !same) atomicAdd(&hist[bin], 1u);
}

template <int PER>  // groups per thread
__global__ __launch_bounds__(TS_THREADS) void topk_select_kernel(const float* __restrict__ logits, int V, int n_groups, int m, int k,
                                                                 float inv_temp, const uint2* __restrict__ groups,
                                                                 int32_t* __restrict__ out_ids, float* __restrict__ out_probs) {
  __shared__ uint32_t hist[1024];
  __shared__ uint32_t kmax_s[TS_THREADS / 64], kmin_s[TS_THREADS / 64], wtot[TS_THREADS / 64], sh[3];
  __shared__ float sum_s[TS_THREADS / 64];
  __shared__ uint32_t n_list, n_sel, used_bits, in_chunk[16];
  __shared__ uint16_t sel[PER * TS_THREADS];
  __shared__ __align__(16) unsigned long long list[TS_LIST];
  __shared__ __align__(8) uint32_t cnt[2][TS_LIST], pos[TS_LIST];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blockIdx.x;
  const float* z = logits + (int64_t)row * V;
  uint32_t key[PER];
  float part[PER];
  uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int g = tid + i * TS_THREADS;
    const uint2 e = g < n_groups ? groups[(int64_t)row * n_groups + g] : uint2{0u, 0u};
    key[i] = e.x;
    part[i] = __uint_as_float(e.y);
    kmax = max(kmax, e.x);
    if (e.x != 0u) kmin = min(kmin, e.x);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o));
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o));
  }
  if (lane == 0) { kmax_s[wave] = kmax; kmin_s[wave] = kmin; }
  hist[tid] = 0u;
  if (tid < 16) in_chunk[tid] = 0u;
  if (tid == 0) { n_list = 0u; n_sel = 0u; used_bits = 0u; }
  *reinterpret_cast<uint2*>(cnt[0] + 2 * tid) = uint2{0u, 0u};
  __syncthreads();
#pragma unroll
  for (int w = 0; w < TS_THREADS / 64; ++w) { kmax = max(kmax, kmax_s[w]); kmin = min(kmin, kmin_s[w]); }
  const uint32_t kall = kmax;
  const float gmax = key_to_float(kmax);
  {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i)  // (expf as in topk_merge: a base-2 exponential of the scaled distance is off by up to 5e-7 at 7 to 14)
      if (part[i] != 0.f) s += part[i] * expf((key_to_float(key[i]) - gmax) * inv_temp);
    s = wave_sum(s);
    if (lane == 0) sum_s[wave] = s;
  }
  const int lm = __ffs(m) - 1, lp = 9 - lm;  // m and the groups per chunk are powers of two
  static_assert(TG_THREADS == 1 << 9, "lp");
  const uint32_t few = (uint32_t)(k + k / 4 + 32);
  // T: at least k group maxima reach it, and few more.  Bins of 2^shift keys from `base` up; `above` maxima lie past the last.
  uint32_t T = kmin, above = 0u;
  int chunks_eq = 16;  // groups whose maximum is T itself are taken in chunks below this
  {
    uint32_t base = kmin, span = kmax - kmin;
    int shift = 0;
    while ((span >> shift) > 1023u) ++shift;
    for (bool refined = false;; refined = true) {
      const uint32_t last = (uint32_t)min((uint64_t)kmax, (uint64_t)base + (((uint64_t)1024 << shift) - 1));
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const bool counts = key[i] >= base && key[i] <= last && key[i] != 0u;
        const uint32_t bin = min((key[i] - base) >> shift, 1023u);
        if (refined) wave_count(counts, bin, hist);  // (a bin that holds too many, often of one value)
        else if (counts) atomicAdd(&hist[bin], 1u);
      }
      __syncthreads();
      uint32_t bin, over, in_bin;
      cut_bin(hist, (uint32_t)k - above, wtot, sh, &bin, &over, &in_bin);
      T = base + (bin << shift);
      above += over;
      if (above + in_bin <= few) break;
      if (shift == 0) {  // (uniform) T is a key that many maxima equal: the first chunks that hold k - above of them
#pragma unroll
        for (int i = 0; i < PER; ++i) wave_count(key[i] == T && T != 0u, (uint32_t)(tid + i * TS_THREADS) >> lp, in_chunk);
        __syncthreads();
        uint32_t have = 0u;
        for (chunks_eq = 0; chunks_eq < 16 && have < (uint32_t)k - above; ++chunks_eq) have += in_chunk[chunks_eq];
        break;
      }
      base = T;
      kmax = (uint32_t)min((uint64_t)kmax, (uint64_t)T + (((uint64_t)1 << shift) - 1));  // the maxima past the bin are counted
      shift = max(0, shift - 10);
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int g = tid + i * TS_THREADS;
    const bool take = key[i] != 0u && (key[i] > T || (key[i] == T && (g >> lp) < chunks_eq));
    const uint32_t p = wave_append(take, &n_sel);
    if (take) sel[p] = (uint16_t)g;
  }
  __syncthreads();
  // Every 16-byte piece of the selected groups: f(id of the first logit, the four logits).
  const int n_pieces = (int)n_sel << (2 + lm);
  auto for_pieces = [&](auto f) {
    for (int q = tid; q < n_pieces; q += TS_THREADS) {
      const int g = sel[q >> (2 + lm)], idx = q & (4 * m - 1);
      const int id = (g >> lp) * TG_CHUNK + (idx >> lm) * (4 * TG_THREADS) + (((g & ((1 << lp) - 1)) << lm) + (idx & (m - 1))) * 4;
      if (id < V) f(id, *reinterpret_cast<const f32x4*>(z + id));
    }
  };
  // A logit that reaches T as one number, larger for larger logits and, among equal ones, for lower ids (of 17 bits): its key's
  // distance from T and ~id.  Where bins of these crowd, `trim` finds the low bits that no such distance has (16 of them where
  // logits are bf16 values), which are then left out.
  int tz = 0;
  auto trim = [&](uint32_t used) {  // used: the bits of this thread's distances
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) used |= (uint32_t)__shfl_xor((int)used, o);
    if (lane == 0) atomicOr(&used_bits, used);
    __syncthreads();
    tz = used_bits ? __ffs((int)used_bits) - 1 : 0;
  };
  auto spot_of = [&](uint32_t from_T, int id) { return ((unsigned long long)(from_T >> tz) << 17) | (uint32_t)(0x1FFFF - id); };
  unsigned long long least = 0ull;
  // To the list: all that reach T, or those of at least `least` (past the list they are only counted); one LDS atomic per
  // wave and piece.
  auto collect = [&](auto bounded_c) {
    for_pieces([&](int id, const f32x4& x) {
      bool take[4];
      unsigned long long mask[4];
      uint32_t total = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t kx = order_key(x[e]);
        take[e] = kx >= T;
        if constexpr (decltype(bounded_c)::value) take[e] = take[e] && spot_of(kx - T, id + e) >= least;
        mask[e] = __builtin_amdgcn_ballot_w64(take[e]);
        total += (uint32_t)__popcll(mask[e]);
      }
      if (total == 0u) return;
      const unsigned long long active = __builtin_amdgcn_ballot_w64(true);
      const int leader = __ffsll(active) - 1;
      uint32_t p = 0u;
      if (lane == leader) p = atomicAdd(&n_list, total);
      p = (uint32_t)__builtin_amdgcn_readlane((int)p, leader);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t at = p + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[e] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask[e], 0u));
        if (take[e] && at < TS_LIST) list[at] = spot_of(order_key(x[e]) - T, id + e);
        p += (uint32_t)__popcll(mask[e]);
      }
    });
    __syncthreads();
  };
  collect(std::false_type{});
  unsigned long long span = spot_of(kall - T, 0);  // (holds at least an id's 17 bits)
  const bool trimmed = n_list > TS_LIST;
  if (trimmed) {  // (uniform) too many: raise the bound until no more than the list holds reach it
    uint32_t used = 0u;
    for_pieces([&](int, const f32x4& x) {
#pragma unroll
      for (int e = 0; e < 4; ++e) used |= order_key(x[e]) >= T ? order_key(x[e]) - T : 0u;
    });
    trim(used);
    span = spot_of(kall - T, 0);
    uint32_t over_all = 0u;
    for (int shift = 54 - __clzll((long long)span);; shift -= 10) {
      for_pieces([&](int id, const f32x4& x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t kx = order_key(x[e]);
          const unsigned long long c = spot_of(kx - T, id + e) - least;
          wave_count(kx >= T && (c >> shift) < 1024ull, (uint32_t)(c >> shift), hist);  // (below `least` c is huge)
        }
      });
      __syncthreads();
      uint32_t bin, over, in_bin;
      cut_bin(hist, (uint32_t)k - over_all, wtot, sh, &bin, &over, &in_bin);
      least += (unsigned long long)bin << shift;
      over_all += over;
      if (shift <= 10 || over_all + in_bin <= TS_LIST) break;  // (over_all < k: a bin of up to 1024 numbers leaves few enough)
    }
    if (tid == 0) n_list = 0u;
    __syncthreads();
    collect(std::true_type{});
  }
  const int n = min((int)n_list, TS_LIST);
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < TS_THREADS / 64; ++w) sum += sum_s[w];
  const float inv_sum = 1.0f / sum;
  auto emit = [&](int slot, int id, float x) {
    if (slot >= k) return;
    out_ids[(int64_t)row * k + slot] = id;
    out_probs[(int64_t)row * k + slot] = expf((x - gmax) * inv_temp) * inv_sum;
  };
  // Each entry's place is the number of larger ones.  `in_seg` entries share the places from `start` on and differ in their
  // last `bits` bits; a crowded segment is split by its next bits into as many bins as it has places, its own counters, so one
  // scan over all counters renumbers every segment, until none holds more than TS_COUNT entries, which are compared.  One round
  // does unless values crowd in a part of the range (an outlier, equal logits): counting over the whole crowd instead took
  // 3.4 us of 18 at k = 256 and, with 700 logits far above the others, 30 of 48.
  unsigned long long mine[TS_PER];
  uint32_t start[TS_PER], in_seg[TS_PER], slot[TS_PER];
  int bits[TS_PER];
#pragma unroll
  for (int i = 0; i < TS_PER; ++i) {
    const int at = tid + i * TS_THREADS;
    mine[i] = at < n ? list[at] : 0ull;
    start[i] = 0u;
    in_seg[i] = at < n ? TS_LIST : 0u;  // (all counters are the first segment's)
    bits[i] = 64 - __clzll((long long)span);
  }
  int now = 0;
  for (bool first = !trimmed;; now ^= 1) {
#pragma unroll
    for (int i = 0; i < TS_PER; ++i) {
      slot[i] = start[i];
      if (in_seg[i] > TS_COUNT) {
        const int take = min(bits[i], 31 - __clz((int)in_seg[i]));
        bits[i] -= take;
        slot[i] += ((1u << take) - 1u) & ~(uint32_t)(mine[i] >> bits[i]);  // larger ones first
      }
      if (in_seg[i] > 0u) atomicAdd(&cnt[now][slot[i]], 1u);
    }
    __syncthreads();
    const uint2 c = *reinterpret_cast<const uint2*>(cnt[now] + 2 * tid);
    *reinterpret_cast<uint2*>(cnt[now ^ 1] + 2 * tid) = uint2{0u, 0u};
    const bool crowded = __builtin_amdgcn_ballot_w64(max(c.x, c.y) > TS_COUNT) != 0ull;
    uint32_t incl = c.x + c.y;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    if (lane == 63) wtot[wave] = incl | (crowded ? 0x80000000u : 0u);
    __syncthreads();
    uint32_t before = incl - c.x - c.y, any = 0u;
#pragma unroll
    for (int w = 0; w < TS_THREADS / 64; ++w) {
      before += w < wave ? wtot[w] & 0x7FFFFFFFu : 0u;
      any |= wtot[w];
    }
    *reinterpret_cast<uint2*>(pos + 2 * tid) = uint2{before | c.x << 16, (before + c.x) | c.y << 16};
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TS_PER; ++i)
      if (in_seg[i] > 0u) {
        start[i] = pos[slot[i]] & 0xFFFFu;
        in_seg[i] = pos[slot[i]] >> 16;
      }
    if (!(any & 0x80000000u)) break;  // (uniform; entries that agree in all bits would be one)
    if (first) {
      first = false;
      uint32_t used = 0u;
#pragma unroll
      for (int i = 0; i < TS_PER; ++i) used |= (uint32_t)(mine[i] >> 17);
      trim(used);
#pragma unroll
      for (int i = 0; i < TS_PER; ++i) {  // (of undecided bits, those above an id's are key bits)
        mine[i] = ((mine[i] >> (17 + tz)) << 17) | (mine[i] & 0x1FFFFull);
        if (bits[i] > 17) bits[i] = max(17, bits[i] - tz);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TS_PER; ++i)
    if (in_seg[i] > 0u) list[start[i] + atomicSub(&cnt[now][slot[i]], 1u) - 1u] = mine[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TS_PER; ++i)
    if (in_seg[i] > 0u) {
      uint32_t place = start[i];
      for (uint32_t j = start[i]; j < start[i] + in_seg[i]; ++j) place += list[j] > mine[i] ? 1u : 0u;
      emit((int)place, 0x1FFFF - (int)(mine[i] & 0x1FFFFull), key_to_float(T + ((uint32_t)(mine[i] >> 17) << tz)));
    }
  for (int i = n + tid; i < k; i += TS_THREADS) emit(i, -1, key_to_float(0u));  // (fewer than k comparable logits: only with NaNs)
}

// Threads per group of topk_groups for a vocabulary of V entries, 0 where the chunk kernels take the row: as many groups as the
// candidate buffer has room for (16 k), since that leaves the fewest logits to read again (64 rows of 128256, k = 256: 15.5 us
// with 16 k groups, 16.2 with 8 k, 18.4 with 4 k), but of 32 logits where that still gives 2 k of them, so that few more than k
// logits reach the k-th largest maximum (k = 512: 17.6 us, with groups of 16 20.3: their maxima span too much for one histogram).
static int group_threads(int V, int k) {
  const int chunks = (V + TG_CHUNK - 1) / TG_CHUNK;
  int m = V / 32 >= 2 * k ? 2 : 1;
  while (m < TG_THREADS && (int64_t)chunks * (TG_THREADS / m) > 16 * (int64_t)k) m <<= 1;
  if ((int64_t)chunks * (TG_THREADS / m) > 16 * (int64_t)k || chunks > 16 || V / (16 * m) < 2 * k) return 0;
  return m;
}

// chunks per row for a vocabulary of V entries; 0 when the combination is not supported
int topk_chunks(int V, int k) {
  int n_chunks = (V + 8191) / 8192;
  if (n_chunks < 1) n_chunks = 1;
  if (n_chunks > 16) return 0;
  return n_chunks;
}

hipError_t launch_topk(const float* logits, int n, int V, int k, float inv_temp, int32_t* out_ids, float* out_probs,
                       unsigned long long* cand_ws, float* stats_ws, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int n_chunks = topk_chunks(V, k);
  if (n_chunks == 0 || k > 1024 || k > V || k <= 0 || (V & 3)) return hipErrorInvalidValue;
  if (const int m = group_threads(V, k)) {
    const int chunks = (V + TG_CHUNK - 1) / TG_CHUNK, n_groups = chunks * (TG_THREADS / m);
    uint2* groups = reinterpret_cast<uint2*>(cand_ws);  // [n, n_groups], n_groups <= 16 k
    topk_groups_kernel<<<dim3(n, chunks), dim3(TG_THREADS), 0, s>>>(logits, V, m, inv_temp, groups);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto select = [&](auto per_c) {
      topk_select_kernel<decltype(per_c)::value><<<dim3(n), dim3(TS_THREADS), 0, s>>>(logits, V, n_groups, m, k, inv_temp, groups, out_ids, out_probs);
    };
    if (n_groups <= TS_THREADS) select(std::integral_constant<int, 1>{});
    else if (n_groups <= 2 * TS_THREADS) select(std::integral_constant<int, 2>{});
    else if (n_groups <= 4 * TS_THREADS) select(std::integral_constant<int, 4>{});
    else return hipErrorInvalidValue;  // (groups of 16 are for vocabularies below 64 k, at most eight chunks)
    return hipGetLastError();
  }
  // with many rows, chunks twice as long still give every CU several workgroups
  const bool wide = n_chunks > 1 && (int64_t)n * n_chunks >= 1024;
  if (wide) n_chunks = (n_chunks + 1) / 2;
  const int per = wide ? 32 : 16;
  int chunk_len = ((V + n_chunks - 1) / n_chunks + 3) / 4 * 4;
  if (chunk_len > TC_THREADS * per || n_chunks * k > TM_THREADS * TM_PER) return hipErrorInvalidValue;
  int n2 = 1;
  while (n2 < k) n2 <<= 1;
  size_t smem_b = (size_t)n2 * 8;
  if (wide)
    topk_chunk_kernel<32><<<dim3(n, n_chunks), dim3(TC_THREADS), 0, s>>>(logits, V, chunk_len, k, inv_temp, cand_ws, stats_ws);
  else
    topk_chunk_kernel<16><<<dim3(n, n_chunks), dim3(TC_THREADS), 0, s>>>(logits, V, chunk_len, k, inv_temp, cand_ws, stats_ws);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int n_cand = n_chunks * k;
  const dim3 mg(n), mb(TM_THREADS);
  if (n_cand <= 2 * TM_THREADS)
    topk_merge_kernel<2><<<mg, mb, smem_b, s>>>(n_chunks, k, inv_temp, cand_ws, stats_ws, n2, out_ids, out_probs);
  else
    topk_merge_kernel<TM_PER><<<mg, mb, smem_b, s>>>(n_chunks, k, inv_temp, cand_ws, stats_ws, n2, out_ids, out_probs);
  return hipGetLastError();
}
