// Products of 1 to 32 rows (single users, small decode batches): the weight stream and the launches around it.
//
// A workgroup of eight waves owns 16 output columns for the whole contraction; each wave takes an eighth of it on 16x16x32
// MFMAs and the eight sums meet through LDS in wave order.  So a 4096-column product is 256 workgroups, one per compute unit,
// with no partial sums in memory and nothing left for another kernel to add up, and the work of the small kernels around a
// product moves into it:
//   few_rows_kernel    each wave keeps its K slice of the rows in registers as MFMA operands (K = 256 * NS; MB blocks of 16 rows,
//                      two of them for q, k, v and logits of Embeds) and walks any number of column tiles; the rows may be
//                      normalised on the way in (RMSNorm of Embeds or of fp32 rows: every workgroup does it for itself while its
//                      first weights are in flight); a QKV tile is rotated and appended to its page, a gate/up tile becomes
//                      eight activations
//   few_stream_kernel  rows streamed beside the weights (long contractions; products that end in the residual)
// A wave of few_stream has 16 KiB of weights in flight (128 KiB per compute unit); one of few_rows a tile's k steps, K / 256 KiB
// up to K = 4096 and 7 to 10 KiB above, where the rows leave no registers for more.  They are requested non-temporally
// through buffer descriptors; requests past the end are sent out of the buffer's range, where they return without touching
// memory.
//
// Bound by HBM, and by launches: a layer of ten has six.  Kernel trace, one and 16 rows, before (norm + product + rotary
// step, product + second norm, product, product + epilogue) and now:
//                    6144 x 4096 q, k, v   4096 x 4096 output + norm   28672 x 4096 gate/up   4096 x 14336 down   layer, wall
//   1 row     us     18.0 -> 14.7          11.2 -> 8                   40.7 -> 40.5           25.3 -> 21.0        124 -> 110
//   16 rows          19.9 -> 15.8          13.8 -> 10.5                40.9 -> 42.8           26.1 -> 23.9
// (the norm of the third column is part of gate/up now); logits of 128256 x 4096 with their norm 169 -> 156 and 167 -> 163, of
// 32000 x 2048 30 -> 22.5 and 32 -> 24.  With 32 rows, norm and rotary step included: q, k, v 22.9 -> 21.3 (17 rows 20.1 and
// 20.2), 3072 x 2048 14.7 -> 10.8; logits of 128256 x 4096 179 -> 174, of 32000 x 2048 33.9 -> 27.4.  Why not more rows, and 16
// where rows are streamed: they come out of L2 beside the weights, in the same order of returns, 459 KiB per compute unit for 16
// rows of 14336 against 459 KiB of weights, and cost 3 us of 24; with 32 rows the split product and its epilogue are as fast.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace {

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr int FEW_RING = 16;  // weight requests of a wave in flight, 1 KiB each

// Columns of a tile.  Plain: 16 in a row.  Pairs: eight columns and the eight they belong with (gate and up of a 32-column
// block pair, or a rotary piece and its other half), in lanes 0-7 and 8-15 of each row of 16: 128-byte pieces of the
// tiled weights instead of 256.
__device__ __forceinline__ int64_t tile_base(int mode, int t, int KB, int D) {  // elements, at k = 0
  if (mode == EPI_SWIGLU) return (int64_t)(t >> 2) * 2 * KB * 512 + (t & 3) * 64;
  if (mode == EPI_STORE_BF16) {
    const int cpt = D / 16, n0 = (t / cpt) * D + (t % cpt) * 8;
    return (int64_t)(n0 >> 5) * KB * 512 + (n0 & 31) * 8;
  }
  return (int64_t)(t >> 1) * KB * 512 + (t & 1) * 128;
}
__device__ __forceinline__ int tile_lane(int mode, int lane, int KB, int D) {  // elements
  const int c = lane & 15, q = lane >> 4, at = (q >> 1) * 512 + (q & 1) * 256;
  if (mode == EPI_SWIGLU) return at + (c & 7) * 8 + (c >> 3) * KB * 512;
  if (mode == EPI_STORE_BF16) return at + (c & 7) * 8 + (c >> 3) * (D / 64) * KB * 512;
  return at + c * 8;
}
// Position of element k (of 64) of row r in a wave's LDS scratch: rows of 128 bytes, 16-byte chunks swizzled so that the 16
// rows' chunks of one k step (an operand read) fall on different banks.
__device__ __forceinline__ int turn_at(int r, int k) { return r * 64 + (((k >> 3) ^ ((r >> 1) & 7)) << 3) + (k & 7); }

constexpr int RSRC_FLAGS = 0x00020000;      // raw dword buffer, gfx9 family
constexpr uint32_t OUT_OF_RANGE = 0xFFFFFF00u;

// ------------------------------------------------------------------------------------------------
// MODE: EPI_STORE_BF16 (q, k, v rotated and stored), EPI_SWIGLU, EPI_STORE_F32.
// ------------------------------------------------------------------------------------------------
template <int MODE, int SRC, int NS, int MB>
__global__ __launch_bounds__(512, 2) void few_rows_kernel(FewSource src, FewIds arg_ids, int M, const bf16_t* __restrict__ Wp, int NB, int n_tiles,
                                                          void* __restrict__ out, int ldo, FewRope rope) {
  constexpr int K = NS * 256, KB = K / 16;
  static_assert(NS % 2 == 0 && NS <= 32, "pairs of k steps, held in registers");
  // weight requests in flight: a tile's k steps (R divides NS, so that the next tile's go on in the same registers)
  [[maybe_unused]] constexpr int R = NS <= FEW_RING ? NS : NS % 8 == 0 ? 8 : NS % 10 == 0 ? 10 : 7;
  static_assert(NS % R == 0, "the ring goes on from tile to tile");
  // requested ahead of the norm, as registers allow: the rows take 4 NS of them a block, twice that in fp32, and nothing may spill
  [[maybe_unused]] constexpr int EARLY = SRC == FEW_F32 ? (R < 12 ? R : 12) : MB == 2 && 35 - 2 * NS < R ? 35 - 2 * NS : R;
  constexpr bool ROPE = MODE == EPI_STORE_BF16;
  __shared__ __align__(16) float red[2][8][MB * 256];
  __shared__ __align__(16) bf16_t turn[8][MB * 16 * 64];
  constexpr int KEPT = (MODE == EPI_STORE_F32 ? 32 : 16) / MB;  // tiles whose sums are kept for the epilogue
  __shared__ __align__(16) float done[KEPT][MB * 256];
  __shared__ float row_ss[8][16 * MB];
  __shared__ __align__(16) bf16_t gain_s[K];
  __shared__ __align__(16) float ang[ROPE ? MB * 16 * 128 : 4];
  __shared__ int place[2][16 * MB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, q = lane >> 4, wgs = gridDim.x;
  const int D = rope.D;
  static_assert(MB == 1 || SRC != FEW_F32, "fp32 rows: 16");
  bf16x8 A[MB][NS];
  [[maybe_unused]] const int k0 = wave * (NS * 32);  // the wave's columns of the rows: k0 .. + NS * 32

  // what the norm and the epilogue read, into registers now and into LDS behind the weight requests
  // (bf16 rows: this lane loads from rows lane / 8, 8 + lane / 8 and so on, fp32 rows: from lane / 16, + 4, + 8, + 12)
  [[maybe_unused]] int ids[2 * MB];
  if constexpr (SRC != FEW_F32) {
#pragma unroll
    for (int h = 0; h < 2 * MB; ++h) {
      const int r = min(h * 8 + (lane >> 3), M - 1);
      ids[h] = SRC == FEW_EMBED ? src.ids[r] : arg_ids.v[r];
    }
  }
  constexpr int GP = (K + 4095) / 4096;
  u32x4 g_in[GP];
#pragma unroll
  for (int i = 0; i < GP; ++i) g_in[i] = *reinterpret_cast<const u32x4*>(src.gain + min(i * 4096 + tid * 8, K - 8));
  [[maybe_unused]] f32x4 ang_in[MB];
  [[maybe_unused]] int place_in;
  if constexpr (ROPE) {
#pragma unroll
    for (int b = 0; b < MB; ++b) ang_in[b] = *reinterpret_cast<const f32x4*>(rope.angles + min(b * 2048 + tid * 4, M * D - 4));
    place_in = ((tid & (16 * MB)) ? rope.tok_slot : rope.tok_page)[min(tid & (16 * MB - 1), M - 1)];
  }
  auto fill_lds = [&]() {
#pragma unroll
    for (int i = 0; i < GP; ++i)
      if (i * 4096 + tid * 8 < K) *reinterpret_cast<u32x4*>(gain_s + i * 4096 + tid * 8) = g_in[i];
    if constexpr (ROPE) {
#pragma unroll
      for (int b = 0; b < MB; ++b)
        if (b * 2048 + tid * 4 < M * D) *reinterpret_cast<f32x4*>(ang + b * 2048 + tid * 4) = ang_in[b];
      if (tid < 32 * MB) place[tid / (16 * MB)][tid & (16 * MB - 1)] = place_in;
    }
  };
#if __HIP_DEVICE_COMPILE__
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(Wp), 0, (int)((int64_t)NB * 32 * K * 2), RSRC_FLAGS);
  const uint32_t woff = (uint32_t)(tile_lane(MODE, lane, KB, D) + wave * NS * 1024) * 2;
  u32x4 W[R];
  int round = 0, t = blockIdx.x;
  uint32_t base = t < n_tiles ? (uint32_t)(tile_base(MODE, t, KB, D) * 2) : 0;
  auto load_w = [&](uint32_t from, bool real, const int step, const int slot) {
    W[slot] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, real ? woff : OUT_OF_RANGE, real ? from + step * 2048 : 0, 2);  // (2: non-temporal)
  };
  // The rows are requested before the weights: requests return in order, and the rows are needed first.  Lanes load 128 (256)
  // consecutive bytes of a row together and the wave turns two k steps at a time into operands through 2 KiB of LDS of
  // its own (LDS operations of a wave are carried out in order: no barrier).
  bf16_t* const my_turn = turn[wave];
  auto put = [&](int r, int k, auto v) { *reinterpret_cast<decltype(v)*>(my_turn + turn_at(r, k)) = v; };
  auto operands = [&](const int p) {
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h) A[b][2 * p + h] = *reinterpret_cast<const bf16x8*>(my_turn + turn_at(b * 16 + c, h * 32 + q * 8));
    __builtin_amdgcn_sched_barrier(0);
  };
  // 1 / rms of rows r0, r0 + step, ..: sums of this wave's columns in `ss`, one row each per LANES lanes
  [[maybe_unused]] auto inv_rms = [&](auto lanes_c, auto& ss) {
    constexpr int LANES = decltype(lanes_c)::value, ROWS = 64 / LANES, N = 16 * MB / ROWS;
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int o = 1; o < LANES; o <<= 1) ss[i] += __shfl_xor(ss[i], o);
      if ((lane & (LANES - 1)) == 0) row_ss[wave][i * ROWS + lane / LANES] = ss[i];
    }
    PIE_S_WAIT_LGKMCNT0();
    wg_barrier();
#pragma unroll
    for (int i = 0; i < N; ++i) {
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) tot += row_ss[w][i * ROWS + lane / LANES];
      ss[i] = 1.0f / sqrtf(tot / (float)K + src.eps);
    }
  };
  if constexpr (SRC == FEW_F32) {
    f32x4 x[NS / 2][4];
    const float* xp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      xp[i] = reinterpret_cast<const float*>(src.x) + (int64_t)min(i * 4 + (lane >> 4), M - 1) * src.ldx + k0 + (lane & 15) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i * 4 < M) {  // (operand rows past M may hold anything: they end in sums of rows that are not stored)
#pragma unroll
        for (int p = 0; p < NS / 2; ++p) x[p][i] = *reinterpret_cast<const f32x4*>(xp[i] + p * 64);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < EARLY; ++s) load_w(base, t < n_tiles, s, s);
    __builtin_amdgcn_sched_barrier(0);
    fill_lds();
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i * 4 < M) {
#pragma unroll
        for (int p = 0; p < NS / 2; ++p)
#pragma unroll
          for (int e = 0; e < 4; ++e) ss[i] += x[p][i][e] * x[p][i][e];
      }
    inv_rms(std::integral_constant<int, 16>{}, ss);
#pragma unroll
    for (int p = 0; p < NS / 2; ++p) {
      const bf16x4 g = *reinterpret_cast<const bf16x4*>(gain_s + k0 + p * 64 + (lane & 15) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(x[p][i][e] * ss[i] * bf16_to_f32(g[e]));
        put(i * 4 + (lane >> 4), (lane & 15) * 4, o);
      }
      operands(p);
    }
  } else {
    Pack16 x[NS / 2][2 * MB];
#pragma unroll
    for (int p = 0; p < NS / 2; ++p)
#pragma unroll
      for (int h = 0; h < 2 * MB; ++h)
        x[p][h].u = *reinterpret_cast<const u32x4*>(reinterpret_cast<const bf16_t*>(src.x) + (int64_t)ids[h] * src.ldx + k0 + (lane & 7) * 8 + p * 64);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < EARLY; ++s) load_w(base, t < n_tiles, s, s);
    __builtin_amdgcn_sched_barrier(0);
    fill_lds();
    float ss[2 * MB];
#pragma unroll
    for (int h = 0; h < 2 * MB; ++h) ss[h] = 0.f;
#pragma unroll
    for (int p = 0; p < NS / 2; ++p)
#pragma unroll
      for (int h = 0; h < 2 * MB; ++h) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = bf16_bits_to_f32(x[p][h].s[e]);
          ss[h] += v * v;
        }
        asm("" : "+v"(x[p][h].u));  // (widened again below, not kept widened: twice the registers)
        __builtin_amdgcn_sched_barrier(0);
      }
    inv_rms(std::integral_constant<int, 8>{}, ss);
#pragma unroll
    for (int p = 0; p < NS / 2; ++p) {
      Pack16 g;
      g.u = *reinterpret_cast<const u32x4*>(gain_s + k0 + p * 64 + (lane & 7) * 8);
#pragma unroll
      for (int h = 0; h < 2 * MB; ++h) {
        Pack16 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o.h[e] = f32_to_bf16(bf16_bits_to_f32(x[p][h].s[e]) * ss[h] * bf16_bits_to_f32(g.s[e]));
        put(h * 8 + (lane >> 3), (lane & 7) * 8, o.u);
      }
      operands(p);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = EARLY; s < R; ++s) load_w(base, t < n_tiles, s, s);

  while (t < n_tiles) {
    const int t_next = t + wgs;
    const bool more = t_next < n_tiles;
    const uint32_t base_next = more ? (uint32_t)(tile_base(MODE, t_next, KB, D) * 2) : 0;
    f32x4 acc[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      Pack16 w;
      w.u = W[s % R];
#pragma unroll
      for (int b = 0; b < MB; ++b) acc[b] = mfma16(A[b][s], w.h, acc[b]);
      if (s + R < NS) load_w(base, true, s + R, s % R);
      else load_w(base_next, more, s + R - NS, s % R);
      __builtin_amdgcn_sched_barrier(0);
    }
    float* mine = red[round & 1][wave];
#pragma unroll
    for (int b = 0; b < MB; ++b) *reinterpret_cast<f32x4*>(mine + b * 256 + lane * 4) = acc[b];
    PIE_S_WAIT_LGKMCNT0();
    wg_barrier();
    // One wave after the other adds a tile's sums up while the others go on with the next tile.  (red is written again two tiles
    // on, behind another barrier.)  What follows, the stores above all, waits for the last tile: a store holds up what its wave
    // requests behind it until memory has taken it (128256 x 4096 at 16 rows: 168 us with every tile stored when it was done).
    if (wave == (round & 7)) {
#pragma unroll
      for (int b = 0; b < MB; ++b) {
        const float* sums = &red[round & 1][0][b * 256 + lane * 4];
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 8; ++w) v += *reinterpret_cast<const f32x4*>(sums + w * (MB * 256));
        *reinterpret_cast<f32x4*>(&done[round % KEPT][b * 256 + lane * 4]) = v;
      }
    }
    if (!more || round % KEPT == KEPT - 1) {
      PIE_S_WAIT_LGKMCNT0();
      wg_barrier();
      for (int u = round / KEPT * KEPT * MB + wave; u < (round + 1) * MB; u += 8) {
        const int r = u / MB, m0 = u % MB * 16 + q * 4, tr = blockIdx.x + r * wgs;
        const f32x4 v = *reinterpret_cast<const f32x4*>(&done[r % KEPT][u % MB * 256 + lane * 4]);  // rows m0 .. + 3 of column c
        if constexpr (MODE == EPI_STORE_F32) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (m0 + i < M) store_nt(reinterpret_cast<float*>(out) + (int64_t)(m0 + i) * ldo + tr * 16 + c, v[i]);
        } else if constexpr (MODE == EPI_SWIGLU) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float up = __shfl_xor(v[i], 8);
            if (m0 + i < M && c < 8)
              reinterpret_cast<bf16_t*>(out)[(int64_t)(m0 + i) * ldo + tr * 8 + c] = f32_to_bf16(silu_f(v[i]) * up);
          }
        } else {
          const int cpt = D / 16, h = tr / cpt, f = (tr % cpt) * 8 + (c & 7), d = f + (c >> 3) * (D / 2);
          const int hk = h - rope.Hq, hv = hk - rope.Hkv;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int m = m0 + i;
            const float own = bf16_to_f32(f32_to_bf16(v[i])), other = __shfl_xor(own, 8);  // (rounded like a stored row)
            if (m >= M) continue;
            bf16_t* page = rope.kv_layer + ((int64_t)place[0][m] * rope.Hkv + (hv >= 0 ? hv : hk)) * (2 * PAGE * D);
            if (hv >= 0) {
              page[v_elem_offset(place[1][m], d, D)] = f32_to_bf16(own);
            } else {
              const float fc = ang[m * D + f], fs = ang[m * D + D / 2 + f];
              const bf16_t o = f32_to_bf16(c < 8 ? own * fc - other * fs : own * fc + other * fs);
              if (hk < 0) reinterpret_cast<bf16_t*>(out)[(int64_t)m * ldo + h * D + d] = o;
              else page[k_elem_offset(place[1][m], d)] = o;
            }
          }
        }
      }
    }
    base = base_next;
    t = t_next;
    ++round;
  }
#endif
}

// Workgroup ids go to the XCDs in turn; here the tiles go to them in ranges, so that the two tiles of a 32-column block, whose
// weights alternate in pieces of 256 bytes, are read through one L2 (4096 x 4096 at one row 7.9 us, 9.9 in launch order;
// the pair tiles above are as fast or faster in launch order).
__device__ __forceinline__ int xcd_order(int wgs, int wg) { return wgs % 8 == 0 ? (wg & 7) * (wgs >> 3) + (wg >> 3) : wg; }

// ------------------------------------------------------------------------------------------------
// NC: 16-column tiles of a workgroup, next to each other.  MODE: EPI_RESID_EMBED, EPI_RESID_OUT.  Any K that is a multiple of
// 32; wave w takes k steps [w n / 8, (w + 1) n / 8) of the n = K / 32.
// ------------------------------------------------------------------------------------------------
template <int MODE, int NC>
__global__ __launch_bounds__(512, 2) void few_stream_kernel(const bf16_t* __restrict__ A, int lda, int M, const bf16_t* __restrict__ Wp,
                                                            int NB, int K, EpiArgs epi) {
  constexpr int P = FEW_RING / 2 / NC;  // pairs of k steps in flight
  __shared__ __align__(16) float red[8][NC][256];
  __shared__ __align__(16) bf16_t turn[8][16 * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  [[maybe_unused]] const int c = lane & 15, q = lane >> 4;
  const int KB = K / 16, wg = xcd_order(gridDim.x, blockIdx.x);
  // the element of the tile(s) this thread finishes, and its residual
  const int em = (tid >> 4) & 15, ej = NC == 1 ? 0 : tid >> 8, en = (wg * NC + ej) * 16 + (tid & 15), er = min(em, M - 1);
  const bool by_id = MODE == EPI_RESID_EMBED ? epi.resid == nullptr : epi.out == nullptr;
  const int id = by_id ? epi.ids[er] : 0;
  float resid = 0.f;
#if __HIP_DEVICE_COMPILE__
  const __amdgpu_buffer_rsrc_t rsrc_w =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(Wp), 0, (int)((int64_t)NB * 32 * K * 2), RSRC_FLAGS);
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, (int)(((int64_t)(M - 1) * lda + K) * 2), RSRC_FLAGS);
  const int steps = K / 32, s0 = wave * steps / 8, n = (wave + 1) * steps / 8 - s0;
  const uint32_t woff = (uint32_t)(tile_lane(MODE, lane, KB, 0) * 2);
  uint32_t aoff[2];  // rows lane / 8 and 8 + lane / 8, 128 bytes (two k steps) of a row by eight lanes
#pragma unroll
  for (int h = 0; h < 2; ++h) aoff[h] = h * 8 < M ? (uint32_t)((min(h * 8 + (lane >> 3), M - 1) * lda + (lane & 7) * 8) * 2) : OUT_OF_RANGE;
  const uint32_t wbase = (uint32_t)(tile_base(MODE, wg * NC, KB, 0) * 2) + s0 * 2048, abase = s0 * 64;
  u32x4 W[P][2][NC], X[P][2];
  auto load_x = [&](int p, const int slot) {
    const bool real = 2 * p < n;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      X[slot][h] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, real ? aoff[h] : OUT_OF_RANGE, real ? abase + p * 128 : 0, 0);
  };
  auto load_w = [&](int p, const int slot) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int s = 2 * p + h;
#pragma unroll
      for (int j = 0; j < NC; ++j)
        W[slot][h][j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, s < n ? woff + j * 256 : OUT_OF_RANGE, s < n ? wbase + s * 2048 : 0, 2);
    }
  };
  f32x4 acc[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < P; ++p) {
    load_x(p, p);
    load_w(p, p);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (MODE == EPI_RESID_EMBED && by_id) resid = bf16_to_f32(epi.embeds[(int64_t)id * epi.H + en]);
  else resid = epi.resid[(int64_t)er * epi.H + en];
  __builtin_amdgcn_sched_barrier(0);
  bf16_t* const my_turn = turn[wave];
  for (int b = 0; 2 * b < n; b += P) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
      for (int h = 0; h < 2; ++h) *reinterpret_cast<u32x4*>(my_turn + turn_at(h * 8 + (lane >> 3), (lane & 7) * 8)) = X[p][h];
      load_x(b + p + P, p);
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 x[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) x[h] = *reinterpret_cast<const bf16x8*>(my_turn + turn_at(c, h * 32 + q * 8));
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (2 * (b + p) + h < n) {  // (uniform)
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            Pack16 w;
            w.u = W[p][h][j];
            acc[j] = mfma16(x[h], w.h, acc[j]);
          }
        }
      load_w(b + p + P, p);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) *reinterpret_cast<f32x4*>(&red[wave][j][lane * 4]) = acc[j];
#endif
  PIE_S_WAIT_LGKMCNT0();
  wg_barrier();
  if (tid >= 256 * NC || em >= M) return;
  const float* sums = &red[0][ej][((em >> 2) * 16 + (tid & 15)) * 4 + (em & 3)];
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) v += sums[w * (NC * 256)];
  v += resid;
  if (MODE == EPI_RESID_EMBED || !by_id) reinterpret_cast<float*>(epi.out)[(int64_t)em * epi.ldo + en] = v;
  else if (id >= 0) epi.embeds[(int64_t)id * epi.H + en] = f32_to_bf16(v);
}

bool fits(const PackedWeight& W) { return (int64_t)W.NB * 32 * W.K * 2 < ((int64_t)1 << 32) - (1 << 20); }

// Workgroups for n tiles with one workgroup per compute unit: as many rounds as it takes, evenly.
int even_wgs(int n, int n_cus) {
  const int rounds = (n + n_cus - 1) / n_cus, wgs = (n + rounds - 1) / rounds;
  return std::min((wgs + 7) / 8 * 8, n_cus);
}

template <int MODE, int SRC>
hipError_t run_rows(const FewSource& given, int M, const PackedWeight& W, int n_tiles, void* out, int ldo, const FewRope& rope, int n_cus,
                    hipStream_t s) {
  FewIds ids{};
  FewSource src = given;
  if (SRC == FEW_EMBED_ARGS) {  // (a host array)
    for (int i = 0; i < M; ++i) ids.v[i] = src.ids[i];
    src.ids = nullptr;
  }
  const dim3 grid(even_wgs(n_tiles, n_cus)), block(512);
  auto run = [&](auto ns_c) {
    constexpr int NS = decltype(ns_c)::value;
    if constexpr (SRC != FEW_F32 && NS <= 16)
      if (M > 16) {
        few_rows_kernel<MODE, SRC, NS, 2><<<grid, block, 0, s>>>(src, ids, M, W.data, W.NB, n_tiles, out, ldo, rope);
        return hipGetLastError();
      }
    few_rows_kernel<MODE, SRC, NS, 1><<<grid, block, 0, s>>>(src, ids, M, W.data, W.NB, n_tiles, out, ldo, rope);
    return hipGetLastError();
  };
  switch (W.K / 256) {
    case 2: return run(std::integral_constant<int, 2>{});
    case 4: return run(std::integral_constant<int, 4>{});
    case 6: return run(std::integral_constant<int, 6>{});
    case 8: return run(std::integral_constant<int, 8>{});
    case 10: return run(std::integral_constant<int, 10>{});
    case 12: return run(std::integral_constant<int, 12>{});
    case 14: return run(std::integral_constant<int, 14>{});
    case 16: return run(std::integral_constant<int, 16>{});
  }
  if constexpr (MODE == EPI_STORE_BF16 && SRC == FEW_EMBED) switch (W.K / 256) {
    case 20: return run(std::integral_constant<int, 20>{});
    case 24: return run(std::integral_constant<int, 24>{});
    case 28: return run(std::integral_constant<int, 28>{});
    case 32: return run(std::integral_constant<int, 32>{});
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Which rows: a wave's slice is pairs of k steps, so K goes in steps of 512; the rows of a slice stay in registers, fp32 rows
// twice over while they are normalised, which ends at 4096.  Embeds of q, k, v go on to 8192 in steps of 1024 (with a ring of at
// least seven).  Every length gains.  Whole layers, us a layer through several with weights from HBM, general path -> this one:
//   width x mlp       512 x 2048     1024 x 4096    1536 x 8960    2560 x 6912    3072 x 8192    4096 x 14336
//   1 row             36.5 -> 28.0   42.2 -> 31.6   60.6 -> 46.8   59.7 -> 51.9   72.8 -> 64.0   107.7 -> 95.5
//   16 rows           41.4 -> 34.3   45.7 -> 37.8   68.4 -> 57.4   67.0 -> 63.2   79.3 -> 73.0   113.1 -> 105.7
// q, k, v of Embeds alone, a layer at one row: 5120 137.1 -> 134.2, 6144 159.0 -> 156.0, 7168 214.1 -> 211.9, 8192 294.0 -> 291.1; 17 to
// 32 rows of 512 to 4096: 0 to 5.
// Logits of up to 16 rows gain 1.5 to 30 us at 512 to 131072 columns.  Of 17 to 32 rows those of up to 3072 gain 0 to 8; at 4096 the
// norm of two blocks in every workgroup has to be paid by the stream (32000 columns 69.4 -> 63.4, 100000 184.3 -> 163.5, but 2048
// columns 23.0 -> 24.4 and 16384 40.7 -> 41.9, top-k included), and 3584, 14 requests a wave, loses where it counts (131072 columns 175 -> 182).
bool few_rows_ok(int M, const PackedWeight& W, int mode, int source) {
  if (M < 1 || M > (source == FEW_F32 || W.K > 16 * 256 ? 16 : FEW_ROWS) || !fits(W)) return false;
  if (W.K < 512 || W.K % 512 != 0) return false;
  if (mode == EPI_STORE_F32 && M > 16 && W.K > 3072) return W.K == 4096 && W.N > 16384;
  return W.K <= 4096 || (W.K <= 8192 && W.K % 1024 == 0 && mode == EPI_STORE_BF16 && source == FEW_EMBED);
}

hipError_t launch_few_qkv(const FewSource& src, int M, const PackedWeight& W, bf16_t* qkv, const FewRope& rope, int n_cus, hipStream_t s) {
  const int heads = rope.Hq + 2 * rope.Hkv;
  if (!few_rows_ok(M, W, EPI_STORE_BF16, src.kind) || (rope.D != 64 && rope.D != 128) || W.N != heads * rope.D) return hipErrorInvalidValue;
  const int tiles = heads * (rope.D / 16);
  if (src.kind == FEW_EMBED) return run_rows<EPI_STORE_BF16, FEW_EMBED>(src, M, W, tiles, qkv, W.N, rope, n_cus, s);
  if (src.kind == FEW_F32) return run_rows<EPI_STORE_BF16, FEW_F32>(src, M, W, tiles, qkv, W.N, rope, n_cus, s);
  return hipErrorInvalidValue;
}

hipError_t launch_few_swiglu(const FewSource& src, int M, const PackedWeight& W, bf16_t* act, int n_cus, hipStream_t s) {
  if (!few_rows_ok(M, W, EPI_SWIGLU, src.kind) || W.N % 64 != 0 || src.kind != FEW_F32) return hipErrorInvalidValue;
  return run_rows<EPI_SWIGLU, FEW_F32>(src, M, W, W.N / 16, act, W.N / 2, FewRope{}, n_cus, s);
}

hipError_t launch_few_f32(const FewSource& src, int M, const PackedWeight& W, float* out, int n_cus, hipStream_t s) {
  if (!few_rows_ok(M, W, EPI_STORE_F32, src.kind) || W.N % 32 != 0 || src.kind != FEW_EMBED_ARGS) return hipErrorInvalidValue;
  return run_rows<EPI_STORE_F32, FEW_EMBED_ARGS>(src, M, W, W.N / 16, out, W.N, FewRope{}, n_cus, s);
}

bool few_resid_ok(int M, int lda, const PackedWeight& W) {
  return M >= 1 && M <= 16 && W.K % 32 == 0 && W.N % 32 == 0 && fits(W) && (int64_t)M * lda * 2 < ((int64_t)1 << 31);
}

namespace {
// Workgroups of an output or down product: 16 columns each, or 32 where that is more than one a compute unit.
int resid_wgs(int N, int n_cus, bool* two) {
  const int tiles = N / 16;
  *two = tiles > n_cus;  // (an even number of tiles: two next to each other are a whole 32-column block)
  return *two ? tiles / 2 : tiles;
}
}  // namespace

// Against the product split along K, whose partial sums the kernel behind it adds up at little cost where that is a norm of its own
// (SUMS_JOIN_NORM); where it is none they take a kernel (SUMS_KERNEL), and where the next product takes its norm in they keep it from
// doing so, which costs 4 to 5 us more (SUMS_KEEP_NORM).  Whole layers of forms that differ in this product alone, us that
// few_stream gains (256 compute units, weights from HBM, one and 16 rows):
//   N x K             1024 x 2048   1024 x 4096   2560 x 8192   3584 x 1024   3584 x 4096   4096 x 4096   5120 x 4096   8192 x 8192
//   SUMS_JOIN_NORM    -1.7  -1.5    0.0  -0.7     0.6  -2.4     -1.0  -1.1    1.4   0.6     1.5   1.7     2.7   2.8     8.8   5.1
//   SUMS_KERNEL                     1.1   0.8     2.1  -0.6      0.6   1.8    1.3   1.0     2.6   3.9     5.0   3.8     7.5   6.8
// So where the sums are free it takes three quarters of the compute units and 2048 of K to gain.  Where they cost something it always
// gains, but for many long rows in few workgroups: every workgroup reads all rows, and with 9 to 16 of them as many bytes as of 16
// columns' weights, at what one compute unit takes (sums free: 3072 x 6144 at 16 rows -1.5; a kernel: 2304 x 9216 -1.7, 3328 x 8960
// -1.4, 2048 x 8192 -0.3; a norm kept: 2048 x 16384 -1.3, 3072 x 24576 -0.7, 5120 x 13824 -2.8, but 2048 x 8192 2.5, 3584 x 18944 2.7,
// 4096 x 14336 2.5 and, two column tiles to the rows, 6144 x 16384 1.8).
bool few_resid_pays(int M, const PackedWeight& W, int n_cus, SplitSums sums) {
  bool two;
  const int wgs = resid_wgs(W.N, n_cus, &two);
  const bool busy = wgs * 8 >= n_cus * (two ? 6 : 7);
  if (M > 8 && !busy && W.K > (sums == SUMS_KEEP_NORM ? 12288 : sums == SUMS_KERNEL || two ? 8192 : 4096)) return false;
  return sums != SUMS_JOIN_NORM || (W.K >= 2048 && (two || wgs * 4 >= n_cus * 3));
}

hipError_t launch_few_resid(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, int n_cus, hipStream_t s) {
  if (!few_resid_ok(M, lda, W) || (epi.mode != EPI_RESID_EMBED && epi.mode != EPI_RESID_OUT)) return hipErrorInvalidValue;
  bool two;
  const dim3 grid(resid_wgs(W.N, n_cus, &two)), block(512);
  if (epi.mode == EPI_RESID_EMBED) {
    if (two) few_stream_kernel<EPI_RESID_EMBED, 2><<<grid, block, 0, s>>>(A, lda, M, W.data, W.NB, W.K, epi);
    else few_stream_kernel<EPI_RESID_EMBED, 1><<<grid, block, 0, s>>>(A, lda, M, W.data, W.NB, W.K, epi);
  } else {
    if (two) few_stream_kernel<EPI_RESID_OUT, 2><<<grid, block, 0, s>>>(A, lda, M, W.data, W.NB, W.K, epi);
    else few_stream_kernel<EPI_RESID_OUT, 1><<<grid, block, 0, s>>>(A, lda, M, W.data, W.NB, W.K, epi);
  }
  return hipGetLastError();
}
