// bf16 MFMA GEMMs  C[M, N] = A[M, K] x W[N, K]^T  with fused epilogues.
//
// (Products of 1 to 16 rows, logits and q, k, v of 17 to 32 as well, that also norm, rotate or finish their rows: few.hip,
// where its conditions hold.)
//   gemm_skinny : M <= 64 (decode batches, LM head).  HBM-bound on the weight stream: every wave owns one
//                 32-column block of W and reads its tiles straight from global memory into MFMA B operands
//                 (each load is 1 KiB contiguous thanks to the tiled weight layout); the activation tile is
//                 shared by the workgroup through LDS.  K is split across gridDim.y when N alone gives too
//                 few workgroups; partial sums go to a workspace and a second kernel applies the epilogue.
//   gemm_stream : up to 640 rows where its workgroups fill the chip; one workgroup per CU with a deep ring of weights in registers.
//   gemm_rows   : tiles of 96 or 128 rows by 256 columns, K split where the tiles alone leave CUs idle.
//   gemm_large  : large M (prefill).  MFMA-bound: 256x256x64 workgroup tile, 8 waves of 128x64.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "internal.h"

// ------------------------------------------------------------------------------------------------
// epilogue on one 32x32 accumulator tile (rows m0.., columns n0..), see mfma32 for the lane layout
// ------------------------------------------------------------------------------------------------
// Loads are batched ahead of the stores (ids, then residual values, then all stores) so that a tile costs
// three dependent memory round trips instead of one per element.
// FULL: all 32 rows of the tile exist (the caller's uniform test), so no per-row predicates are needed; with them
// every element is its own predicated block and the loads cannot be batched.
// NT: non-temporal stores (see gemm_skinny_kernel).
template <int MODE, bool FULL = false, bool NT = false>
__device__ __forceinline__ void epi_tile(const EpiArgs& e, const f32x16& acc, const f32x16& acc2, int m0, int n0,
                                         int M_rows, int N, int lane) {
  const int M = FULL ? 0x7fffffff : M_rows;
  const int n = n0 + (lane & 31);
  const int g = lane >> 5;
  if (n >= N) return;
  auto st = [](auto* p, auto v) {
    if (NT) store_nt(p, v);
    else *p = v;
  };
  int rows[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) rows[v] = m0 + (v >> 2) * 8 + g * 4 + (v & 3);
  if (MODE == EPI_STORE_BF16) {
    bf16_t* out = reinterpret_cast<bf16_t*>(e.out);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (rows[v] < M) st(out + (int64_t)rows[v] * e.ldo + n, f32_to_bf16(acc[v]));
  } else if (MODE == EPI_STORE_F32) {
    float* out = reinterpret_cast<float*>(e.out);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (rows[v] < M) st(out + (int64_t)rows[v] * e.ldo + n, acc[v]);
  } else if (MODE == EPI_SWIGLU) {  // acc = gate block, acc2 = up block; n0 is the gate block's packed column
    bf16_t* out = reinterpret_cast<bf16_t*>(e.out);
    const int nc = (n0 >> 1) + (lane & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (rows[v] < M) st(out + (int64_t)rows[v] * e.ldo + nc, f32_to_bf16(silu_f(acc[v]) * acc2[v]));
  } else if (MODE == EPI_RESID_EMBED) {
    float r[16];
    if (e.resid != nullptr) {  // wide residual stream of an inner layer
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v] = rows[v] < M ? e.resid[(int64_t)rows[v] * e.H + n] : 0.f;
    } else {
      int id[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) id[v] = rows[v] < M ? e.ids[rows[v]] : 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v] = bf16_to_f32(e.embeds[(int64_t)id[v] * e.H + n]);
    }
    float* out = reinterpret_cast<float*>(e.out);
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (rows[v] < M) st(out + (int64_t)rows[v] * e.ldo + n, r[v] + acc[v]);
  } else if (MODE == EPI_RESID_OUT) {
    float r[16];
    if (e.out != nullptr) {  // inner layer: the sum stays wide and feeds the next layer
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v] = rows[v] < M ? e.resid[(int64_t)rows[v] * e.H + n] : 0.f;
      float* out = reinterpret_cast<float*>(e.out);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (rows[v] < M) st(out + (int64_t)rows[v] * e.ldo + n, r[v] + acc[v]);
    } else {
      int id[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) id[v] = rows[v] < M ? e.ids[rows[v]] : -1;
#pragma unroll
      for (int v = 0; v < 16; ++v) r[v] = id[v] >= 0 ? e.resid[(int64_t)rows[v] * e.H + n] : 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (id[v] >= 0) st(e.embeds + (int64_t)id[v] * e.H + n, f32_to_bf16(r[v] + acc[v]));
    }
  }
}

// ------------------------------------------------------------------------------------------------
// gemm_skinny
// ------------------------------------------------------------------------------------------------
#define SK_BK 128  // contraction elements per main-loop iteration (8 MFMA steps)
#define SK_MAX_SPLITS 8

// WAVES: waves per workgroup.  KS: the contraction is split KS ways INSIDE the workgroup (where the widths give too few
// waves otherwise): waves w and w + WAVES / KS own the same column block and each takes a K-th of
// the contraction, with an activation tile of its own per iteration; the sums meet through LDS at the end, so twice
// as many waves stream weights and no more partial sums leave the workgroup.
template <int MB, int MODE, bool PARTIAL, int NBW, int WAVES = 4, int KS = 1>
__global__ __launch_bounds__(WAVES * 64) void gemm_skinny_kernel(const bf16_t* __restrict__ A, int lda, int M,
                                                          const bf16_t* __restrict__ Wp, int N, int NB, int K,
                                                          int iters_per_split, EpiArgs epi, float* __restrict__ part) {
  // Non-temporal stores for what is written just before a kernel that streams from HBM for a long time: the QKV sums
  // (a small rotary kernel, then decode attention) and the LM head's own logits (33 MB at 64 rows, which otherwise
  // compete with its weight stream: 205 -> 193 us).  The other products are followed by a small kernel that reads
  // what they wrote at once, and that one is a microsecond or two slower when the lines have left the caches.
  constexpr bool SK_NT = MODE == EPI_STORE_BF16 || MODE == EPI_STORE_F32 || (PARTIAL && MODE == EPI_RESID_OUT);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem_raw);  // [2][KS][MB*32][SK_BK], 16-byte chunks swizzled by row
  static_assert(WAVES % KS == 0, "every slice gets the same number of waves");
  constexpr int BM = MB * 32;
  constexpr int NT = WAVES * 64;
  constexpr int WPS = WAVES / KS;            // waves per K slice
  constexpr int A_SLICE = BM * SK_BK;        // elements of one slice's activation tile
  constexpr int A_ELEMS = KS * A_SLICE;      // elements of one stage
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ks = wave / WPS;                 // this wave's K slice
  const int KB = K / 16;
  const int total_iters = (K + SK_BK - 1) / SK_BK;
  // This workgroup covers iterations first .. of the contraction; with KS > 1 their number is a multiple of KS (the host
  // sees to it), slice s takes the s-th part of them and `it` below counts within the slice.
  const int first = PARTIAL || KS == 1 ? blockIdx.y * iters_per_split : 0;
  const int last = min(total_iters, first + iters_per_split);
  const int it0 = KS > 1 ? 0 : first;
  const int it1 = KS > 1 ? (last - first) / KS : last;
  const int slice_it0 = KS > 1 ? first + ks * it1 : 0;  // added to `it`: the global iteration of this wave's slice
  // a wave owns NBW adjacent 32-column blocks (SWIGLU: a gate/up pair)
  int nb0 = (blockIdx.x * WPS + wave % WPS) * NBW;
  const bool wave_active = nb0 < NB;
  if (!wave_active) nb0 = 0;  // keep loads in bounds; results are dropped

  f32x16 acc[NBW][MB];
#pragma unroll
  for (int j = 0; j < NBW; ++j)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;

  // A tile loader: BM rows x 16 chunks (16 B) per iteration; chunk c of row r is stored at chunk (c ^ (r & 15))
  constexpr int A_CHUNKS = KS * BM * 16;     // the tiles of all slices, slice by slice
  constexpr int A_PER_THREAD = (A_CHUNKS + NT - 1) / NT;
  // The activation chunks travel in the same ring of three register sets as the weights, requested two iterations
  // ahead and stored to LDS one iteration ahead: the memory counter completes in order, so waiting for the chunks
  // of iteration it + 1 also waits for every load requested before them; with the chunks requested in the
  // previous step, the weights of two iterations stay in flight across that wait instead of one.  Only for several
  // row blocks of one column block per wave (64-row layer products: 0.244 -> 0.239 ms per forward call): with one
  // row block the extra registers cost the third wave per SIMD, and with two column blocks per wave (LM head) the
  // kernel got 2-3% slower.
  constexpr bool A_RING = MB >= 2 && NBW == 1 && (KS == 1 || WAVES >= 8);  // (few chunks per thread: the ring still fits two waves per SIMD)
  constexpr int A_SETS = A_RING ? 3 : 1;
  u32x4 areg[A_SETS][A_PER_THREAD];
  // Loads always read an in-bounds address (row and k clamped); chunks outside the matrix are zeroed when the
  // registers are stored to LDS, so no register is written while an earlier load into it could be pending.
  auto load_a = [&](int it, const int slot_ring) {
    const int slot = A_RING ? slot_ring : 0;
#pragma unroll
    for (int j = 0; j < A_PER_THREAD; ++j) {
      const int c = min(tid + j * NT, A_CHUNKS - 1);
      const int sl = c / (BM * 16), cc = c % (BM * 16);
      const int r = min(cc >> 4, M - 1), kc = cc & 15;
      const int k = min(((KS > 1 ? first + sl * it1 : 0) + it) * SK_BK + kc * 8, K - 8);
      areg[slot][j] = *reinterpret_cast<const u32x4*>(A + (int64_t)r * lda + k);
    }
  };
  auto store_a = [&](int buf, int it, const int slot_ring) {
    const int slot = A_RING ? slot_ring : 0;
#pragma unroll
    for (int j = 0; j < A_PER_THREAD; ++j) {
      const int c = tid + j * NT;
      const int sl = c / (BM * 16), cc = c % (BM * 16);
      const int r = cc >> 4, kc = cc & 15;
      const bool inside = r < M && ((KS > 1 ? first + sl * it1 : 0) + it) * SK_BK + kc * 8 < K;
      if (c < A_CHUNKS)
        *reinterpret_cast<u32x4*>(As + buf * A_ELEMS + sl * A_SLICE + r * SK_BK + ((kc ^ (r & 15)) << 3)) =
            inside ? areg[slot][j] : u32x4{0, 0, 0, 0};
    }
  };
  bf16x8 breg[3][NBW][8];  // ring of three register sets: the weights of the next two iterations are in flight
  auto load_b = [&](int it, const int slot) {
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        int kb = (slice_it0 + it) * 8 + s;
        kb = kb < KB ? kb : KB - 1;  // tail steps read a valid tile; their A operand is zero
        const int nbj = nb0 + j < NB ? nb0 + j : NB - 1;  // a missing second block re-reads a valid one
        breg[slot][j][s] = load_nt(reinterpret_cast<const bf16x8*>(Wp + packed_tile_offset(nbj, kb, KB) + lane * 8));  // read once
      }
  };

  // One main-loop iteration; SLOT is the register set holding this iteration's W operands (compile-time so
  // the operand arrays stay in registers).  The barrier carries no memory fence (a fence would make the compiler
  // drain every outstanding load, i.e. the weights requested two iterations ahead): only the LDS stores of the
  // next activation tile have to be visible to the other waves, hence the explicit wait for LDS operations.
  auto step = [&](auto slot_c, int it) {
    constexpr int SLOT = decltype(slot_c)::value;
    const int cur = (it - it0) & 1;
    const bool more = it + 1 < it1;
    if (!A_RING && more) load_a(it + 1, 0);
    if (it + 2 < it1) {
      if (A_RING) load_a(it + 2, (SLOT + 2) % 3);
      load_b(it + 2, (SLOT + 2) % 3);
    }
    const bf16_t* Ab = As + cur * A_ELEMS + ks * A_SLICE;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int kc = s * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int r = i * 32 + (lane & 31);
        bf16x8 af = *reinterpret_cast<const bf16x8*>(Ab + r * SK_BK + ((kc ^ (r & 15)) << 3));
#pragma unroll
        for (int j = 0; j < NBW; ++j) acc[j][i] = mfma32(af, breg[SLOT][j][s], acc[j][i]);
      }
    }
    if (more) store_a(cur ^ 1, it + 1, (SLOT + 1) % 3);
    PIE_S_WAIT_LGKMCNT0();
    wg_barrier();
  };
  if (it0 < it1) {
    load_a(it0, 0);
    load_b(it0, 0);
    if (it0 + 1 < it1) {
      if (A_RING) load_a(it0 + 1, 1);
      load_b(it0 + 1, 1);
    }
    store_a(0, it0, 0);  // waits for the oldest loads only
  }
  PIE_S_WAIT_LGKMCNT0();
  wg_barrier();
  for (int it = it0; it < it1; it += 3) {
    step(std::integral_constant<int, 0>{}, it);
    if (it + 1 < it1) step(std::integral_constant<int, 1>{}, it + 1);
    if (it + 2 < it1) step(std::integral_constant<int, 2>{}, it + 2);
  }
  if constexpr (KS > 1) {
    // The slices' sums meet through LDS (the activation stages are free once the main loop has passed its last
    // barrier): slices 1.. leave theirs, slice 0 adds them in slice order.
    static_assert(NBW == 1, "one column block per wave");
    float* red = reinterpret_cast<float*>(smem_raw) + (MODE == EPI_SWIGLU ? (WPS / 2) * MB * 16 * 64 : 0);  // [KS - 1][WPS][MB][16][64]
    if (ks > 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[((((ks - 1) * WPS + wave % WPS) * MB + i) * 16 + v) * 64 + lane] = acc[0][i][v];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int sl = 1; sl < KS; ++sl)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[0][i][v] += red[((((sl - 1) * WPS + wave) * MB + i) * 16 + v) * 64 + lane];
    }
  }
  if constexpr (!PARTIAL && MODE == EPI_SWIGLU && NBW == 1) {
    // One block per wave: the gate block sits in the even waves, its up block in the wave after it, which hands
    // its sums over through LDS.
    float* xch = reinterpret_cast<float*>(smem_raw);  // [WPS / 2 pairs][MB][16][64]
    const int pair = (wave % WPS) >> 1;
    if ((wave & 1) && ks == 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) xch[((pair * MB + i) * 16 + v) * 64 + lane] = acc[0][i][v];
    }
    __syncthreads();
    if (!(wave & 1) && ks == 0 && wave_active) {
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        f32x16 up;
#pragma unroll
        for (int v = 0; v < 16; ++v) up[v] = xch[((pair * MB + i) * 16 + v) * 64 + lane];
        epi_tile<MODE, false, SK_NT>(epi, acc[0][i], up, i * 32, nb0 * 32, M, NB * 32, lane);
      }
    }
    return;
  }
  if (!wave_active || ks > 0) return;
  if (PARTIAL) {
    // raw partial sums: part[split][m][n_packed]
    float* P = part + (int64_t)blockIdx.y * M * (NB * 32);
#pragma unroll
    for (int j = 0; j < NBW; ++j)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          int m = i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
          if (m < M && nb0 + j < NB) {
            float* dst = P + (int64_t)m * (NB * 32) + (nb0 + j) * 32 + (lane & 31);
            if (SK_NT) store_nt(dst, acc[j][i][v]);
            else *dst = acc[j][i][v];
          }
        }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      if (MODE == EPI_SWIGLU) {
        epi_tile<MODE, false, SK_NT>(epi, acc[0][i], acc[NBW - 1][i], i * 32, nb0 * 32, M, NB * 32, lane);
      } else {
#pragma unroll
        for (int j = 0; j < NBW; ++j)
          if (nb0 + j < NB) epi_tile<MODE, false, SK_NT>(epi, acc[j][i], acc[j][i], i * 32, (nb0 + j) * 32, M, N, lane);
      }
    }
  }
}

// Sum split-K partials and apply the epilogue.  One thread per four consecutive output columns (SWIGLU: four
// gate/up pairs); all column counts are multiples of 32, so the four never straddle a 32-column block.
template <int MODE>
__global__ void splitk_epilogue_kernel(const float* __restrict__ part, int splits, int M, int N, int NP, EpiArgs e) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int cols = (MODE == EPI_SWIGLU) ? NP / 2 : N;
  const int cols4 = cols / 4;
  if (idx >= (int64_t)M * cols4) return;
  const int m = (int)(idx / cols4), c = (int)(idx % cols4) * 4;
  // partial sums are added in split order; eight loads are requested together so that the few threads of a
  // small batch still keep enough bytes in flight
  auto total = [&](int n) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    const float* p = part + (int64_t)m * NP + n;
    const int64_t stride = (int64_t)M * NP;
    int k = 0;
    for (; k + 8 <= splits; k += 8) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4*>(p + (k + u) * stride);
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < splits; ++k) s += *reinterpret_cast<const f32x4*>(p + k * stride);
    return s;
  };
  auto store_bf16x4 = [](bf16_t* dst, const f32x4& v) {
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = f32_to_bf16(v[i]);
    *reinterpret_cast<bf16x4*>(dst) = o;
  };
  if (MODE == EPI_SWIGLU) {
    const int ng = (c >> 5) * 64 + (c & 31);  // gate columns in packed order; the up columns are 32 further
    const f32x4 g = total(ng), u = total(ng + 32);
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = silu_f(g[i]) * u[i];
    store_bf16x4(reinterpret_cast<bf16_t*>(e.out) + (int64_t)m * e.ldo + c, r);
  } else if (MODE == EPI_STORE_BF16) {
    store_bf16x4(reinterpret_cast<bf16_t*>(e.out) + (int64_t)m * e.ldo + c, total(c));
  } else if (MODE == EPI_STORE_F32) {
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(e.out) + (int64_t)m * e.ldo + c) = total(c);
  } else {
    // The residual (and the id of the output Embed) is requested ahead of the partial sums, not behind them.
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
    int id = 0;
    if (MODE == EPI_RESID_OUT || e.resid != nullptr) {
      r = *reinterpret_cast<const f32x4*>(e.resid + (int64_t)m * e.H + c);
      if (MODE == EPI_RESID_OUT && e.out == nullptr) id = e.ids[m];
    } else {
      const bf16x4 v = *reinterpret_cast<const bf16x4*>(e.embeds + (int64_t)e.ids[m] * e.H + c);
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = bf16_to_f32(v[i]);
    }
    const f32x4 y = total(c) + r;
    if (MODE == EPI_RESID_EMBED || e.out != nullptr) {
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(e.out) + (int64_t)m * e.ldo + c) = y;
    } else if (id >= 0) {
      store_bf16x4(e.embeds + (int64_t)id * e.H + c, y);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// gemm_large
// ------------------------------------------------------------------------------------------------
#define LG_BM 256
#define LG_BN 256
#define LG_BK 64

template <int MODE>
__global__ __launch_bounds__(512) void gemm_large_kernel(const bf16_t* __restrict__ A, int lda, int M,
                                                         const bf16_t* __restrict__ Wp, int N, int NB, int K,
                                                         EpiArgs epi) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  bf16_t* As = reinterpret_cast<bf16_t*>(smem_raw);       // [2][256 rows][64], chunk c of row r at c ^ (r & 7)
  bf16_t* Bs = As + 2 * LG_BM * LG_BK;                    // [2][8 blocks][4 k-steps][512], operand order
  constexpr int TILE = LG_BM * LG_BK;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;  // wave tile: rows wm*128.., columns wn*64..
  const int KB = K / 16;
  const int m0 = blockIdx.y * LG_BM;
  const int nb0 = blockIdx.x * (LG_BN / 32);
  const int KT = (K + LG_BK - 1) / LG_BK;

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  u32x4 ra[4], rb[4];
  auto load_g = [&](int kt) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int c = tid + j * 512;
      int r = c >> 3, kc = c & 7;
      int gr = m0 + r;
      gr = gr < M ? gr : M - 1;  // rows past M read a valid row; their results are never stored
      int k = kt * LG_BK + kc * 8;
      u32x4 v = {0, 0, 0, 0};
      if (k < K) v = *reinterpret_cast<const u32x4*>(A + (int64_t)gr * lda + k);
      ra[j] = v;
      // W: chunk c -> block c / 256, 16-byte piece c % 256 of that block's 4 consecutive k-tiles
      int nbl = c >> 8, w = c & 255;
      int nb = nb0 + nbl;
      nb = nb < NB ? nb : NB - 1;
      int kb = kt * 4 + (w >> 6);
      u32x4 wv = {0, 0, 0, 0};
      if (kb < KB) wv = *reinterpret_cast<const u32x4*>(Wp + packed_tile_offset(nb, kb, KB) + (w & 63) * 8);
      rb[j] = wv;
    }
  };
  auto store_s = [&](int buf) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int c = tid + j * 512;
      int r = c >> 3, kc = c & 7;
      *reinterpret_cast<u32x4*>(As + buf * TILE + r * LG_BK + ((kc ^ (r & 7)) << 3)) = ra[j];
      *reinterpret_cast<u32x4*>(Bs + buf * TILE + c * 8) = rb[j];
    }
  };

  load_g(0);
  store_s(0);
  __syncthreads();
  for (int kt = 0; kt < KT; ++kt) {
    const int cur = kt & 1;
    const bool more = kt + 1 < KT;
    if (more) load_g(kt + 1);
    const bf16_t* Ab = As + cur * TILE;
    const bf16_t* Bb = Bs + cur * TILE;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      bf16x8 af[4], bfr[2];
      const int kc = s * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = wm * 128 + i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8*>(Ab + r * LG_BK + ((kc ^ (r & 7)) << 3));
      }
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bfr[j] = *reinterpret_cast<const bf16x8*>(Bb + ((wn * 2 + j) * 4 + s) * 512 + lane * 8);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(af[i], bfr[j], acc[i][j]);
    }
    if (more) store_s(cur ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int mt = m0 + wm * 128 + i * 32;
    if (MODE == EPI_SWIGLU) {
      int nb = nb0 + wn * 2;
      if (nb < NB) epi_tile<MODE>(epi, acc[i][0], acc[i][1], mt, nb * 32, M, NB * 32, lane);
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        int nb = nb0 + wn * 2 + j;
        if (nb < NB) epi_tile<MODE>(epi, acc[i][j], acc[i][j], mt, nb * 32, M, N, lane);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// gemm_large, asynchronous-copy version (K a multiple of 64)
//
// Same 256x256x64 tile and 8 waves of 128x64 as above.  The activation tile is copied global -> LDS by direct-to-LDS
// loads (no VGPR staging, no LDS store instructions): each wave instruction moves 1 KiB and the rows land
// pre-swizzled (16-byte chunk c of row r at position c ^ ((r >> 1) & 7), conflict-free for the 64-bank LDS when 16
// consecutive rows read the same chunk); three stages as separate arrays (the compiler's wait counters then know
// which copy a read may alias), copies two k steps ahead, one fence-free barrier per k step.
// The weight operands do not pass through LDS: a wave reads the tiles of its two column blocks straight from
// global memory into MFMA B operands (the tiled weight layout makes each a contiguous 1 KiB load; the two waves
// that share a column block meet in the vector cache), one k step ahead, refilling each register set right after
// the MFMAs that consumed it.  Why: with both operands in LDS a 128x64 wave tile issues and waits for 6 LDS reads
// per 8 MFMAs, without the weights 4, and every instruction issued beside the MFMAs takes matrix time (LDS bandwidth
// itself is not short: 240-250 bytes per clock and compute unit with many reads in flight, the kernel uses a fifth
// of it).  The matrix pipe went from 62% to 72% busy, of which the lower clock under the higher load gives back a
// part (8320 x 28672 x 4096: 1.70 -> 1.58 ms on one box).
// Workgroup ids are remapped so that each XCD (id % 8) works on a contiguous range of a grouped tile order (8 row
// tiles per group) and its L2 sees a few activation and weight panels at a time.
// ------------------------------------------------------------------------------------------------
// Position of workgroup `id` in that order: ids go to the XCDs in turn, XCD x has n / 8 of them and one more when
// x < n % 8.  A single row of tiles shares no weights between workgroups; where its length is not a multiple of 8 it is
// left in launch order (128256 x 4096 at 193 rows 257 us, in ranges 262).  With more rows the ranges are what makes the
// row tiles of a column meet in one L2, whatever the number of tiles: at 129 rows, 501 x 2 tiles of 96 rows, 299 us in
// launch order (the weights fetched twice), 244 in ranges.
__host__ __device__ __forceinline__ int xcd_range(int id, int tiles_m, int tiles_n) {
  const int n = tiles_m * tiles_n, x = id & 7;
  return tiles_m == 1 && n % 8 != 0 ? id : x * (n >> 3) + (x < (n & 7) ? x : n & 7) + (id >> 3);
}
// Row and column tile at a position of the grouped order.
__host__ __device__ __forceinline__ void tile_at(int pos, int tiles_m, int tiles_n, int& tm, int& tn) {
  constexpr int GROUP_M = 8;
  const int width = GROUP_M * tiles_n;
  const int first_m = (pos / width) * GROUP_M;
  const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
  tm = first_m + (pos % width) % gsz;
  tn = (pos % width) / gsz;
}

template <int MODE, bool PARTIAL>
__global__ __launch_bounds__(512) void gemm_large_async_kernel(const bf16_t* __restrict__ A, int lda, int M,
                                                               const bf16_t* __restrict__ Wp, int N, int NB, int K,
                                                               EpiArgs epi, int tiles_m, int tiles_n,
                                                               int kts_per_split, float* __restrict__ part) {
  constexpr int BM = LG_BM;
  constexpr int MI = BM / 64;  // 32-row accumulator blocks per wave, and activation copy instructions per wave
  __shared__ __align__(16) bf16_t As0[BM * LG_BK], As1[BM * LG_BK], As2[BM * LG_BK];  // three activation stages
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int KB = K / 16, KT = K / LG_BK;
  // split K: workgroup row blockIdx.y takes k tiles [kt0, kt1)
  // Non-temporal stores for the logits and for the partial sums of the down projection, the last product before the
  // LM head (see gemm_skinny_kernel; LM head at 256 rows 278 -> 262 us).  The partial sums
  // of the QKV product are stored plainly here: at 65 to 256 rows the rotary step that sums them loses what the
  // attention kernel gains.
  constexpr bool LG_NT = MODE == EPI_STORE_F32 || (PARTIAL && MODE == EPI_RESID_OUT) || (!PARTIAL && MODE == EPI_SWIGLU);
  const int kt0 = PARTIAL ? blockIdx.y * kts_per_split : 0;
  const int kt1 = PARTIAL ? min(KT, kt0 + kts_per_split) : KT;
  int tm, tn;
  tile_at(xcd_range(blockIdx.x, tiles_m, tiles_n), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, nb0 = tn * (LG_BN / 32);

  f32x16 acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  {
#if __HIP_DEVICE_COMPILE__  // (the buffer-descriptor builtins exist for the device target only)
    // Both operands are addressed through buffer descriptors (base in scalar registers, a 32-bit byte offset per
    // lane, the k step as a scalar offset): a request is one instruction without 64-bit address arithmetic, reads
    // past the end return zeros, and the direct-to-LDS copies are buffer loads, not global (flat-encoded) loads:
    // with those in flight the compiler waits for all outstanding vector memory operations before every use of a
    // register that a load returns, which would drain the weight loads requested ahead at every step.
    constexpr int RSRC_FLAGS = 0x00020000;  // raw dword buffer, gfx9 family
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(A), 0, (int)(((int64_t)(M - 1) * lda + K) * 2), RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(Wp), 0, (int)((int64_t)NB * 32 * K * 2), RSRC_FLAGS);
    // copy instruction j = wave * MI + jj of a stage covers LDS bytes [j KiB, (j + 1) KiB): rows j*8 .. j*8+7 of
    // the tile, lane -> row j*8 + lane/8, stored chunk lane%8
    int aoff[MI], woff[2];  // byte offsets of this lane's pieces at k step 0
#pragma unroll
    for (int jj = 0; jj < MI; ++jj) {
      const int r = (wave * MI + jj) * 8 + (lane >> 3);
      const int kc = (lane & 7) ^ ((r >> 1) & 7);
      int gr = m0 + r;
      gr = gr < M ? gr : M - 1;  // rows past M re-read a valid row; their results are never stored
      aoff[jj] = (int)(((int64_t)gr * lda + kc * 8) * 2);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int nb = nb0 + wn * 2 + j;
      nb = nb < NB ? nb : NB - 1;  // a column block past the matrix re-reads a valid one; its results are dropped
      woff[j] = (int)((packed_tile_offset(nb, 0, KB) + lane * 8) * 2);
    }
    u32x4 wreg[4][2];  // the weight operands of one k step: [16-wide contraction step][column block]
    auto issue_a = [&](bf16_t* As, int kt) {
      const int k = kt < kt1 ? kt : kt1 - 1;  // past the end: a copy nobody reads, so that the wait counts stay uniform
#pragma unroll
      for (int jj = 0; jj < MI; ++jj)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (__attribute__((address_space(3))) void*)(As + (wave * MI + jj) * 512),
                                                 16, aoff[jj], k * (LG_BK * 2), 0, 0);
    };
    auto load_w = [&](int kt, const int s) {
      const int k = kt < kt1 ? kt : kt1 - 1;
#pragma unroll
      for (int j = 0; j < 2; ++j) wreg[s][j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, woff[j], (k * 4 + s) * 1024, 0);
    };
    auto load_a = [&](const bf16_t* As, int s, bf16x8 (&af)[MI]) {
      const int kc = s * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = wm * (BM / 2) + i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8*>(As + r * LG_BK + ((kc ^ ((r >> 1) & 7)) << 3));
      }
    };
    // One k step on stage Acur; the copy of k step kt + 2 goes to Afill (read last in k step kt - 1, which every wave
    // has left).  The step's barrier sits before its last 16-wide contraction step instead of at its end: by then a
    // wave has read everything it needs from Acur, so after the barrier the first operands of the next k step can be
    // read from Anext while the last MFMAs of this one run, and no step starts with the matrix cores waiting for
    // LDS.  Vector memory operations complete in order: at the barrier the newest MI + 6 (the copy issued at the top
    // of the step and the weight loads of its first three contraction steps) may still be in flight, everything
    // older has arrived, in particular this wave's part of the activation tile of k step kt + 1.
    bf16x8 af[2][MI];
    auto step = [&](const bf16_t* Acur, const bf16_t* Anext, bf16_t* Afill, int kt) {
      issue_a(Afill, kt + 2);
      __builtin_amdgcn_sched_barrier(0);  // the copies go out first: the wait counts rely on the request order
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s + 1 < 4) {
          load_a(Acur, s + 1, af[(s + 1) & 1]);
        } else {
          PIE_S_WAIT_LGKMCNT0();  // this wave's last reads of Acur have returned
          PIE_S_WAIT_VMCNT(MI + 6);
          wg_barrier();
          load_a(Anext, 0, af[0]);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            Pack16 w;
            w.u = wreg[s][j];
            acc[i][j] = mfma32(af[s & 1][i], w.h, acc[i][j]);
          }
        load_w(kt + 1, s);  // refill the registers just consumed with the next k step's weights
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    issue_a(As0, kt0);
    issue_a(As1, kt0 + 1);
#pragma unroll
    for (int s = 0; s < 4; ++s) load_w(kt0, s);
    PIE_S_WAIT_VMCNT(MI + 8);  // the first activation tile has arrived
    wg_barrier();
    load_a(As0, 0, af[0]);
    int kt = kt0;
    for (; kt + 3 <= kt1; kt += 3) {  // whole revolutions of the three stages; the one or two steps left over follow
      step(As0, As1, As2, kt);
      step(As1, As2, As0, kt + 1);
      step(As2, As0, As1, kt + 2);
    }
    if (kt < kt1) {
      step(As0, As1, As2, kt);
      if (kt + 1 < kt1) step(As1, As2, As0, kt + 1);
    }
    PIE_S_WAIT_VMCNT(0);  // the surplus copies of the last steps land before the workgroup gives up its LDS
#endif
  }
  if (PARTIAL) {
    // raw partial sums: part[split][m][n_packed]
    const int NP = NB * 32;
    float* P = part + (int64_t)blockIdx.y * M * NP;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int nb = nb0 + wn * 2 + j;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = m0 + wm * (BM / 2) + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
          if (m < M && nb < NB) {
            float* dst = P + (int64_t)m * NP + nb * 32 + (lane & 31);
            if (LG_NT) store_nt(dst, acc[i][j][v]);
            else *dst = acc[i][j][v];
          }
        }
      }
    return;
  }
  // row tiles that lie wholly inside the matrix (all of them except in a ragged last row block) take the
  // epilogue without per-row predicates
  auto epilogue = [&](auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int mt = m0 + wm * (BM / 2) + i * 32;
      if (MODE == EPI_SWIGLU) {
        int nb = nb0 + wn * 2;
        if (nb < NB) epi_tile<MODE, FULL, LG_NT>(epi, acc[i][0], acc[i][1], mt, nb * 32, M, NB * 32, lane);
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          int nb = nb0 + wn * 2 + j;
          if (nb < NB) epi_tile<MODE, FULL, LG_NT>(epi, acc[i][j], acc[i][j], mt, nb * 32, M, N, lane);
        }
      }
    }
  };
  const bool rows_full = m0 + wm * (BM / 2) + MI * 32 <= M;
  if constexpr (MODE == EPI_RESID_EMBED || MODE == EPI_RESID_OUT) {
    // Residual epilogues of full row tiles, pipelined over the wave's 2 * MI accumulator tiles: the Embed ids of
    // all its rows are read first (one round trip), then the residual values of tile t + 1 are requested before
    // tile t is stored, so a tile no longer costs two or three dependent round trips of its own.
    if (rows_full && N % 32 == 0) {
      const bool by_id = MODE == EPI_RESID_EMBED ? epi.resid == nullptr : epi.out == nullptr;
      const int g = lane >> 5;
      const int mw = m0 + wm * (BM / 2) + g * 4;
      auto row_of = [&](int i, int v) { return mw + i * 32 + (v >> 2) * 8 + (v & 3); };
      auto run = [&](auto by_id_c) {
        constexpr bool BY_ID = decltype(by_id_c)::value;
        int id[MI][16];
        if (BY_ID) {
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) id[i][v] = epi.ids[row_of(i, v)];
        }
        float r[2][16];
        auto col_of = [&](int t) { return (nb0 + wn * 2 + (t & 1)) * 32 + (lane & 31); };
        auto fetch = [&](int t, float (&dst)[16]) {
          const int i = t >> 1, n = col_of(t);
          if (n >= N) return;  // uniform: a column block past the matrix
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            if (MODE == EPI_RESID_EMBED && BY_ID) dst[v] = bf16_to_f32(epi.embeds[(int64_t)id[i][v] * epi.H + n]);
            else dst[v] = epi.resid[(int64_t)row_of(i, v) * epi.H + n];
          }
        };
        auto put = [&](int t, const float (&src)[16]) {
          const int i = t >> 1, j = t & 1, n = col_of(t);
          if (n >= N) return;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float y = src[v] + acc[i][j][v];
            if (MODE == EPI_RESID_OUT && BY_ID) {
              // (non-temporal: the output Embeds are the last thing written before the LM head streams its weights:
              // 241 -> 219 us at 8320 rows; the fp32 sums of the output projection below lose 9 us that way)
              if (id[i][v] >= 0) store_nt(epi.embeds + (int64_t)id[i][v] * epi.H + n, f32_to_bf16(y));
            } else if (MODE == EPI_RESID_OUT) {
              store_nt(reinterpret_cast<float*>(epi.out) + (int64_t)row_of(i, v) * epi.ldo + n, y);
            } else {
              reinterpret_cast<float*>(epi.out)[(int64_t)row_of(i, v) * epi.ldo + n] = y;
            }
          }
        };
        fetch(0, r[0]);
#pragma unroll
        for (int t = 0; t < 2 * MI; ++t) {
          if (t + 1 < 2 * MI) fetch(t + 1, r[(t + 1) & 1]);
          put(t, r[t & 1]);
        }
      };
      if (by_id) run(std::true_type{});
      else run(std::false_type{});
      return;
    }
  }
  if (rows_full) epilogue(std::true_type{});
  else epilogue(std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// SwiGLU epilogue of a tile whose gate and up blocks (and KS slices of K) are in different waves.  CHUNK rows of accumulator
// blocks at a time go to LDS (`piece(p)`: 4 KiB pieces, room for 8 * CHUNK; block i of wave w is piece 8 i + w, 16 bytes per
// lane), and then all eight waves take quarters of the results in turn: a column per lane and four rows.  (With the up
// sums handed to the gate waves, one wave per SIMD waited out every exponential and store by itself: 28672 x 4096 within a layer at
// 64 rows 44.4 -> 43.3 us, at 84 44.6 -> 42.8, at 157 60.1 -> 58.7, at 256 the same, 75.7 and 76.3; 16384 x 2048 at 324 rows 32.1 and
// 32.0.)
// ------------------------------------------------------------------------------------------------
template <bool NT, int MB, int KS, int CHUNK, typename Piece>
__device__ __forceinline__ void swiglu_through_lds(const f32x16 (&acc)[MB], Piece piece, int wave, int lane, int m0, int nb0, int M, int NB,
                                                   const EpiArgs& e) {
  constexpr int WPS = 8 / KS, PAIRS = WPS / 2;  // column blocks and gate/up pairs of the tile
#pragma unroll
  for (int i0 = 0; i0 < MB; i0 += CHUNK) {
    constexpr int REST = MB % CHUNK;
    const int rows = REST != 0 && i0 + CHUNK > MB ? REST : CHUNK;
    // (barriers without the fence of __syncthreads, which would wait here for the stores of the rows before)
    PIE_S_WAIT_LGKMCNT0();
    wg_barrier();
#pragma unroll
    for (int i = i0; i < MB && i < i0 + CHUNK; ++i) {
      float* d = piece((i - i0) * 8 + wave) + lane * 4;
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const f32x4 x = {acc[i][v4 * 4], acc[i][v4 * 4 + 1], acc[i][v4 * 4 + 2], acc[i][v4 * 4 + 3]};
        *reinterpret_cast<f32x4*>(d + v4 * 256) = x;
      }
    }
    PIE_S_WAIT_LGKMCNT0();
    wg_barrier();
#pragma unroll 2
    for (int u = wave; u < rows * PAIRS * 4; u += 8) {
      const int v4 = u & 3, pair = (u >> 2) % PAIRS, i = (u >> 2) / PAIRS;
      auto sums = [&](int w) {  // of the column block that wave w of each slice holds, in slice order
        f32x4 x = *reinterpret_cast<const f32x4*>(piece(i * 8 + w) + v4 * 256 + lane * 4);
#pragma unroll
        for (int sl = 1; sl < KS; ++sl) x += *reinterpret_cast<const f32x4*>(piece(i * 8 + sl * WPS + w) + v4 * 256 + lane * 4);
        return x;
      };
      const int nb = nb0 + 2 * pair, m = m0 + (i0 + i) * 32 + v4 * 8 + (lane >> 5) * 4;
      if (nb >= NB) continue;
      const f32x4 gate = sums(2 * pair), up = sums(2 * pair + 1);
      bf16_t* out = reinterpret_cast<bf16_t*>(e.out) + (int64_t)m * e.ldo + nb * 16 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (m + r >= M) continue;
        const bf16_t y = f32_to_bf16(silu_f(gate[r]) * up[r]);
        if (NT) store_nt(out + (int64_t)r * e.ldo, y);
        else out[(int64_t)r * e.ldo] = y;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// gemm_rows (K a multiple of 64): 65 rows up to where whole rounds of 256x256 tiles fill the chip
//
// Tiles of 32 * MB rows (96 or 128) by 256 columns, K in steps of 64, eight waves side by side along the columns: a
// wave owns one 32-column block for all rows of the tile.  Against the 2 x 4 arrangement of the 256 x 256 tile no two
// waves read the same weights, which matters because the vector memory path of a compute unit moves 64 bytes per clock
// and its share of a step is as long as the MFMAs': 32 KiB of weights + 4 MB KiB of activations per step here, 64 KiB +
// 4 MB KiB with every weight tile read by two waves.  The price, one LDS read per MFMA instead of one per two, is half
// of what LDS delivers.  Registers are kept to 128 (one k step of weights, 16 MB accumulators, and for MB = 4 a single
// set of activation operands) so that two workgroups share a compute unit and one computes while the other waits at
// its barrier.  Measured, kernel plus epilogue, weights from HBM, against the 128-row form of the 256-column tile it
// replaces: 28672 x 4096 at 84 rows 59 -> 52 us, at 157 rows (256-row tile) 74 -> 61, 4096 x 14336 at 333 rows 69 ->
// 53, at 2000 rows 233 -> 189, 6144 x 4096 at 4096 rows 191 (256-row tile) -> 164.  Over many rounds of a full chip the
// 128-row tile equals the 256-row one and the 96-row tile loses (28672 x 4096 at 8192 rows 1473, 1432 and 1695 us).
// With one workgroup per compute unit (a few hundred rows) the bound is the weight bytes in flight, 32 KiB per compute
// unit: gate/up 28672 x 4096 at 157 rows takes 60 us with its weights in HBM and 42 with them in the last-level cache.
// The workgroup order is that of gemm_large_async_kernel.
// ------------------------------------------------------------------------------------------------
template <int MODE, bool PARTIAL, int MB>
__global__ __launch_bounds__(512, 4) void gemm_rows_kernel(const bf16_t* __restrict__ A, int lda, int M,
                                                           const bf16_t* __restrict__ Wp, int N, int NB, int K,
                                                           EpiArgs epi, int tiles_m, int tiles_n, int kts_per_split,
                                                           float* __restrict__ part) {
  static_assert(MB == 3 || MB == 4, "tile height");
  constexpr int BM = MB * 32;
  constexpr int PIECES = BM / 8;        // 1 KiB copy instructions per activation stage
  constexpr int CP = (PIECES + 7) / 8;  // per wave; past the last piece a wave copies that one again (same bytes)
  [[maybe_unused]] constexpr bool AHEAD = MB < 4;        // the next contraction step's activation operands are read under this one's MFMAs
  __shared__ __align__(16) bf16_t As0[BM * LG_BK], As1[BM * LG_BK], As2[BM * LG_BK], As3[BM * LG_BK];
  constexpr bool NT = MODE == EPI_STORE_F32 || (PARTIAL && MODE == EPI_RESID_OUT) || (!PARTIAL && MODE == EPI_SWIGLU);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  [[maybe_unused]] const int KB = K / 16;
  const int KT = K / LG_BK;
  const int kt0 = PARTIAL ? blockIdx.y * kts_per_split : 0;
  [[maybe_unused]] const int kt1 = PARTIAL ? min(KT, kt0 + kts_per_split) : KT;
  int tm, tn;
  tile_at(xcd_range(blockIdx.x, tiles_m, tiles_n), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, nb = tn * 8 + wave;

  f32x16 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

  {
#if __HIP_DEVICE_COMPILE__  // (buffer descriptors: see gemm_large_async_kernel)
    constexpr int RSRC_FLAGS = 0x00020000;
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(A), 0, (int)(((int64_t)(M - 1) * lda + K) * 2), RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(Wp), 0, (int)((int64_t)NB * 32 * K * 2), RSRC_FLAGS);
    // copy piece p of a stage covers rows p*8 .. p*8+7 of the tile: lane -> row p*8 + lane/8, stored chunk lane%8
    int piece[CP], aoff[CP];
#pragma unroll
    for (int jj = 0; jj < CP; ++jj) {
      piece[jj] = PIECES % 8 == 0 ? wave * CP + jj : min(wave * CP + jj, PIECES - 1);
      const int r = piece[jj] * 8 + (lane >> 3);
      const int kc = (lane & 7) ^ ((r >> 1) & 7);
      const int gr = min(m0 + r, M - 1);  // rows past M re-read a valid row; their results are never stored
      aoff[jj] = (int)(((int64_t)gr * lda + kc * 8) * 2);
    }
    // a column block past the matrix re-reads a valid one; its results are dropped
    const int woff = (int)((packed_tile_offset(min(nb, NB - 1), 0, KB) + lane * 8) * 2);
    u32x4 wreg[4];  // the weight operands of one k step
    auto issue_a = [&](bf16_t* As, int kt) {
      const int k = kt < kt1 ? kt : kt1 - 1;  // past the end: a copy nobody reads, so that the wait counts stay uniform
#pragma unroll
      for (int jj = 0; jj < CP; ++jj)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (__attribute__((address_space(3))) void*)(As + piece[jj] * 512),
                                                 16, aoff[jj], k * (LG_BK * 2), 0, 0);
    };
    auto load_w = [&](int kt, const int s) {
      const int k = kt < kt1 ? kt : kt1 - 1;
      wreg[s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, woff, (k * 4 + s) * 1024, 0);
    };
    auto load_a = [&](const bf16_t* As, int s, bf16x8 (&af)[MB]) {
      const int kc = s * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int r = i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8*>(As + r * LG_BK + ((kc ^ ((r >> 1) & 7)) << 3));
      }
    };
    // One k step on stage Acur; the copy of k step kt + 3 goes to Afill, read last in k step kt - 1, which every wave
    // has left.  At the barrier, before the last contraction step's MFMAs, this wave has read all of Acur and its part
    // of the tile of k step kt + 1 has to have arrived; requested after that one were the copies of two steps (2 CP)
    // and 4 + 4 + 3 weight loads.
    bf16x8 af[2][MB];
    auto step = [&](const bf16_t* Acur, const bf16_t* Anext, bf16_t* Afill, int kt) {
      issue_a(Afill, kt + 3);
      __builtin_amdgcn_sched_barrier(0);  // the copies go out first: the wait counts rely on the request order
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (!AHEAD) load_a(Acur, s, af[0]);
        else if (s < 3) load_a(Acur, s + 1, af[(s + 1) & 1]);
        if (s == 3) {
          PIE_S_WAIT_LGKMCNT0();  // this wave's last reads of Acur have returned
          PIE_S_WAIT_VMCNT(2 * CP + 11);
          wg_barrier();
          if (AHEAD) load_a(Anext, 0, af[0]);
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          Pack16 w;
          w.u = wreg[s];
          acc[i] = mfma32(af[AHEAD ? s & 1 : 0][i], w.h, acc[i]);
        }
        load_w(kt + 1, s);  // refill the register just consumed with the next k step's weights
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    issue_a(As0, kt0);
    issue_a(As1, kt0 + 1);
    issue_a(As2, kt0 + 2);
#pragma unroll
    for (int s = 0; s < 4; ++s) load_w(kt0, s);
    PIE_S_WAIT_VMCNT(2 * CP + 4);  // the first activation tile has arrived
    wg_barrier();
    if (AHEAD) load_a(As0, 0, af[0]);
    int kt = kt0;
    for (; kt + 4 <= kt1; kt += 4) {  // whole revolutions of the four stages, then up to three steps
      step(As0, As1, As3, kt);
      step(As1, As2, As0, kt + 1);
      step(As2, As3, As1, kt + 2);
      step(As3, As0, As2, kt + 3);
    }
    if (kt < kt1) step(As0, As1, As3, kt);
    if (kt + 1 < kt1) step(As1, As2, As0, kt + 1);
    if (kt + 2 < kt1) step(As2, As3, As1, kt + 2);
    PIE_S_WAIT_VMCNT(0);  // the surplus copies of the last steps land before the workgroup gives up its LDS
#endif
  }
  if (PARTIAL) {
    if (nb >= NB) return;
    const int NP = NB * 32;
    float* P = part + (int64_t)blockIdx.y * M * NP + nb * 32 + (lane & 31);  // raw sums: part[split][m][n_packed]
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = m0 + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        if (m < M) {
          if (NT) store_nt(P + (int64_t)m * NP, acc[i][v]);
          else P[(int64_t)m * NP] = acc[i][v];
        }
      }
    return;
  }
  const bool rows_full = m0 + BM <= M;
  if constexpr (MODE == EPI_SWIGLU) {
    // a gate block sits in an even wave, its up block in the wave after it
    constexpr int PER_STAGE = BM * LG_BK * 2 / 4096;
    auto piece = [&](int p) {
      const int st = p / PER_STAGE;
      return reinterpret_cast<float*>(st == 0 ? As0 : st == 1 ? As1 : st == 2 ? As2 : As3) + (p % PER_STAGE) * 1024;
    };
    swiglu_through_lds<NT, MB, 1, 4 * PER_STAGE / 8>(acc, piece, wave, lane, m0, tn * 8, M, NB, epi);
  } else {
    if (nb >= NB) return;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      if (rows_full) epi_tile<MODE, true, NT>(epi, acc[i], acc[i], m0 + i * 32, nb * 32, M, N, lane);
      else epi_tile<MODE, false, NT>(epi, acc[i], acc[i], m0 + i * 32, nb * 32, M, N, lane);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// gemm_stream (K a multiple of 64): 1 to 640 rows, where the weight stream, or its latency, is the bound
//
// What gemm_rows lacks with one workgroup per compute unit is weight bytes in flight (one k step, 32 KiB, and half of
// that with tiles of 96 rows read twice).  Here a compute unit holds one workgroup of eight waves on purpose and spends
// the registers that frees (256 per lane) on a ring of S = 3 or 4 k steps of weights, 96 to 128 KiB in flight, requested
// non-temporally (read once, or by all row tiles of a column at once, on one XCD).  KS: the contraction is
// split KS ways inside the workgroup: slice s (8 / KS waves, 32 columns each) takes the s-th part of the workgroup's k
// steps with an activation tile of its own, and the sums meet through LDS in slice order.  That is what keeps tiles
// narrow enough for a workgroup on (nearly) every compute unit without partial sums in memory: 28672 columns are 224
// tiles of 128 (KS = 2), 16384 are 256 tiles of 64 (KS = 4).  Activations go to LDS by direct copies as in gemm_rows, S
// stages, rows swizzled.
// Measured by itself, kernel plus epilogue, weights from HBM, against what ran before (gemm_skinny up to 64 rows, gemm_rows
// above): 28672 x 4096 at 84 rows 52 -> 44 us, 128 rows 59 -> 48, 157 rows 61 -> 54, 300 rows 100 -> 78; 4096 x 14336 at
// 84 rows 32 -> 29; 57344 x 8192 at 64 rows 152 -> 138 (6.8 TB/s), 157 rows 225 -> 158; 16384 x 2048 at 16 rows 23 -> 15;
// 128256 x 4096 at 157 rows 254 -> 183; 3072 x 2048 at 200 rows 15.9 -> 10.4, 8192 x 28672 at 520 rows 287 -> 260.  Within
// passes over several layers (kernel trace) 28672 x 4096 takes 45, 57, 64 and 86 us at 84, 128, 157 and 300 rows.  Without
// its copies, LDS reads and MFMAs (timing only) that stream takes 46 us by itself: at 157 rows 8 us are not hidden under it.
// ------------------------------------------------------------------------------------------------
// stages and weight ring: four where 128 KiB of LDS and the registers hold them
constexpr int stream_stages(int mb, int ks) { return ks == 1 && mb <= 5 ? 4 : ks == 2 && mb == 2 ? 4 : 3; }

template <int MODE, bool PARTIAL, int MB, int KS>
__global__ __launch_bounds__(512, 2) void gemm_stream_kernel(const bf16_t* __restrict__ A, int lda, int M,
                                                             const bf16_t* __restrict__ Wp, int N, int NB, int K,
                                                             EpiArgs epi, int tiles_m, int tiles_n, int kts_per_split,
                                                             float* __restrict__ part) {
  constexpr int BM = MB * 32;
  constexpr int S = stream_stages(MB, KS);
  constexpr int WPS = 8 / KS;                // column blocks of the tile
  constexpr int PIECES = KS * BM / 8;        // 1 KiB copy instructions per activation stage
  [[maybe_unused]] constexpr int CP = (PIECES + 7) / 8;  // per wave
  constexpr int STAGE = KS * BM * LG_BK;
  __shared__ __align__(16) bf16_t As0[STAGE], As1[STAGE], As2[STAGE], As3[S > 3 ? STAGE : 16];
  constexpr bool NT = MODE == EPI_STORE_F32 || (PARTIAL && MODE == EPI_RESID_OUT) || (!PARTIAL && MODE == EPI_SWIGLU);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / WPS;                 // this wave's K slice
  [[maybe_unused]] const int KB = K / 16;
  const int KT = K / LG_BK;
  const int first = PARTIAL ? blockIdx.y * kts_per_split : 0;
  const int last = PARTIAL ? min(KT, first + kts_per_split) : KT;
  [[maybe_unused]] const int n = (last - first) / KS;  // k steps of a slice (KS divides them, the host sees to it)
  int tm, tn;
  tile_at(xcd_range(blockIdx.x, tiles_m, tiles_n), tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, nb = tn * WPS + wave % WPS;

  f32x16 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  {
#if __HIP_DEVICE_COMPILE__  // (buffer descriptors: see gemm_large_async_kernel)
    constexpr int RSRC_FLAGS = 0x00020000;
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(A), 0, (int)(((int64_t)(M - 1) * lda + K) * 2), RSRC_FLAGS);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(Wp), 0, (int)((int64_t)NB * 32 * K * 2), RSRC_FLAGS);
    // copy piece p of a stage covers eight rows of one slice's tile: lane -> row lane / 8 of them, stored chunk lane % 8;
    // past the last piece a wave copies that one again (same bytes)
    int piece[CP], aoff[CP];
#pragma unroll
    for (int jj = 0; jj < CP; ++jj) {
      piece[jj] = PIECES % 8 == 0 ? wave * CP + jj : min(wave * CP + jj, PIECES - 1);
      const int sl = piece[jj] / (BM / 8), r = (piece[jj] % (BM / 8)) * 8 + (lane >> 3);
      const int kc = (lane & 7) ^ ((r >> 1) & 7);
      const int gr = min(m0 + r, M - 1);  // rows past M re-read a valid row; their results are never stored
      aoff[jj] = (int)(((int64_t)gr * lda + kc * 8 + (int64_t)(first + sl * n) * LG_BK) * 2);
    }
    const int woff = (int)((packed_tile_offset(min(nb, NB - 1), (first + ks * n) * 4, KB) + lane * 8) * 2);
    u32x4 wreg[S][4];  // ring: the weight operands of S k steps
    auto issue_a = [&](bf16_t* As, int kt) {
      const int k = kt < n ? kt : n - 1;  // past the end: a copy nobody reads, so that the wait counts stay uniform
#pragma unroll
      for (int jj = 0; jj < CP; ++jj)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (__attribute__((address_space(3))) void*)(As + piece[jj] * 512),
                                                 16, aoff[jj], k * (LG_BK * 2), 0, 0);
    };
    auto load_w = [&](int kt, const int slot, const int s) {
      const int k = kt < n ? kt : n - 1;
      wreg[slot][s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, woff, (k * 4 + s) * 1024, 2);  // (2: non-temporal)
    };
    auto load_a = [&](const bf16_t* As, int s, bf16x8 (&af)[MB]) {
      const int kc = s * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int r = i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8*>(As + ks * (BM * LG_BK) + r * LG_BK + ((kc ^ ((r >> 1) & 7)) << 3));
      }
    };
    bf16x8 af[2][MB];
    // Step kt on stage Acur: the copies of step kt + S - 1 go to Afill, read last in step kt - 1, which every wave has
    // left; each weight register set is refilled for step kt + S right behind its MFMAs.  At the barrier, before the last
    // contraction step's MFMAs, this wave has read all of Acur and its part of the tile of step kt + 1 has to have
    // arrived.  Requested after that one were the copies of S - 2 steps and, inside the loop, the weights of S - 2 steps
    // and three quarters.  TAIL: in the steps behind the loop the compiler drops the weight requests that no step uses,
    // so only the copies may be counted on there.
    auto step = [&](auto tail_c, auto slot_c, const bf16_t* Acur, const bf16_t* Anext, bf16_t* Afill, int kt) {
      constexpr int SLOT = decltype(slot_c)::value;
      constexpr bool TAIL = decltype(tail_c)::value;
      issue_a(Afill, kt + S - 1);
      __builtin_amdgcn_sched_barrier(0);  // the copies go out first: the wait counts rely on the request order
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        // the next contraction step's activation operands are read under this one's MFMAs
        if (s < 3) load_a(Acur, s + 1, af[(s + 1) & 1]);
        if (s == 3) {
          PIE_S_WAIT_LGKMCNT0();  // this wave's last reads of Acur have returned
          if constexpr (TAIL) PIE_S_WAIT_VMCNT((S - 2) * CP);
          else PIE_S_WAIT_VMCNT((S - 2) * CP + (S - 2) * 4 + 3);
          wg_barrier();
          load_a(Anext, 0, af[0]);
        }
        __builtin_amdgcn_sched_barrier(0);  // (else the compiler moves the reads behind the MFMAs, into the same registers)
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          Pack16 w;
          w.u = wreg[SLOT][s];
          acc[i] = mfma32(af[s & 1][i], w.h, acc[i]);
        }
        load_w(kt + S, SLOT, s);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // Prologue in the order of the main loop: copies of step j, weights of step j.  The loop below is entered
    // unconditionally (every slice has at least S steps, the host sees to it): a branch around it would let the compiler
    // move the weight requests that only the loop uses behind the wait that counts them.
    issue_a(As0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < S; ++j) {
#pragma unroll
      for (int s = 0; s < 4; ++s) load_w(j, j, s);
      __builtin_amdgcn_sched_barrier(0);
      if (j == 0) issue_a(As1, 1);
      if (j == 1 && S > 3) issue_a(As2, 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    PIE_S_WAIT_VMCNT((S - 2) * CP + S * 4);  // this wave's part of the first activation tile has arrived
    wg_barrier();
    load_a(As0, 0, af[0]);
    int kt = 0;
    using std::integral_constant;
    if constexpr (S == 3) {
      do {
        step(std::false_type{}, integral_constant<int, 0>{}, As0, As1, As2, kt);
        step(std::false_type{}, integral_constant<int, 1>{}, As1, As2, As0, kt + 1);
        step(std::false_type{}, integral_constant<int, 2>{}, As2, As0, As1, kt + 2);
        kt += 3;
      } while (kt + 3 <= n);
      if (kt < n) step(std::true_type{}, integral_constant<int, 0>{}, As0, As1, As2, kt);
      if (kt + 1 < n) step(std::true_type{}, integral_constant<int, 1>{}, As1, As2, As0, kt + 1);
    } else {
      do {
        step(std::false_type{}, integral_constant<int, 0>{}, As0, As1, As3, kt);
        step(std::false_type{}, integral_constant<int, 1>{}, As1, As2, As0, kt + 1);
        step(std::false_type{}, integral_constant<int, 2>{}, As2, As3, As1, kt + 2);
        step(std::false_type{}, integral_constant<int, 3>{}, As3, As0, As2, kt + 3);
        kt += 4;
      } while (kt + 4 <= n);
      if (kt < n) step(std::true_type{}, integral_constant<int, 0>{}, As0, As1, As3, kt);
      if (kt + 1 < n) step(std::true_type{}, integral_constant<int, 1>{}, As1, As2, As0, kt + 1);
      if (kt + 2 < n) step(std::true_type{}, integral_constant<int, 2>{}, As2, As3, As1, kt + 2);
    }
    PIE_S_WAIT_VMCNT(0);  // the surplus copies of the last steps land before the stages are used for anything else
#endif
  }
  // 4 KiB pieces of LDS (one accumulator block of one wave) for exchanges between waves: piece p of the stages laid end
  // to end
  constexpr int PER_STAGE = STAGE * 2 / 4096;
  auto lds_piece = [&](int p) {
    const int st = p / PER_STAGE;
    bf16_t* b = st == 0 ? As0 : st == 1 ? As1 : st == 2 ? As2 : As3;
    return reinterpret_cast<float*>(b) + (p % PER_STAGE) * 1024;
  };
  if constexpr (MODE == EPI_SWIGLU && !PARTIAL) {
    constexpr int FIT = S * PER_STAGE / 8;
    swiglu_through_lds<NT, MB, KS, (FIT < MB ? FIT : MB)>(acc, lds_piece, wave, lane, m0, tn * WPS, M, NB, epi);
    return;
  }
  __syncthreads();
  if constexpr (KS > 1) {
    static_assert((KS - 1) * WPS * MB <= S * PER_STAGE, "the slices' sums fit the stages");
    if (ks > 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        float* d = lds_piece(((ks - 1) * WPS + wave % WPS) * MB + i);
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v * 64 + lane] = acc[i][v];
      }
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int sl = 1; sl < KS; ++sl)
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const float* d = lds_piece(((sl - 1) * WPS + wave) * MB + i);
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][v] += d[v * 64 + lane];
        }
    }
    __syncthreads();
  }
  if (nb >= NB || ks > 0) return;
  if (PARTIAL) {
    const int NP = NB * 32;
    float* P = part + (int64_t)blockIdx.y * M * NP + nb * 32 + (lane & 31);  // raw sums: part[split][m][n_packed]
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = m0 + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        if (m < M) {
          if (NT) store_nt(P + (int64_t)m * NP, acc[i][v]);
          else P[(int64_t)m * NP] = acc[i][v];
        }
      }
    return;
  }
  const bool rows_full = m0 + BM <= M;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    if (rows_full) epi_tile<MODE, true, NT>(epi, acc[i], acc[i], m0 + i * 32, nb * 32, M, N, lane);
    else epi_tile<MODE, false, NT>(epi, acc[i], acc[i], m0 + i * 32, nb * 32, M, N, lane);
  }
}

// ------------------------------------------------------------------------------------------------
// dispatch
// ------------------------------------------------------------------------------------------------
// Raises a kernel's dynamic LDS limit once per process and device (done: one bit per device), not per launch.
static hipError_t set_lds_limit_once(const void* kern, size_t bytes, uint32_t& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < 32 && ((done >> dev) & 1u)) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && dev >= 0 && dev < 32) done |= 1u << dev;
  return e;
}

template <int MODE>
static hipError_t launch_splitk_epilogue(int splits, int M, const PackedWeight& W, const EpiArgs& epi, const float* ws, hipStream_t s) {
  const int NP = W.NB * 32, cols = (MODE == EPI_SWIGLU) ? NP / 2 : W.N;
  const int64_t total = (int64_t)M * (cols / 4);
  const int wg = total < 512 * 256 ? 64 : 256;  // (few threads: workgroups of one wave reach every compute unit)
  splitk_epilogue_kernel<MODE><<<dim3((unsigned)((total + wg - 1) / wg)), dim3(wg), 0, s>>>(ws, splits, M, W.N, NP, epi);
  return hipGetLastError();
}

template <int MB, int MODE, int NBW, int WAVES = 4, int KS = 1>
static hipError_t run_skinny_n(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, float* ws,
                               size_t ws_elems, int n_cus, hipStream_t s, int* defer, int max_splits = SK_MAX_SPLITS) {
  const int wg_n = (W.NB + (WAVES / KS) * NBW - 1) / ((WAVES / KS) * NBW);
  const int total_iters = (W.K + SK_BK - 1) / SK_BK;
  // Split K so that one round of workgroups fills the chip without spilling into a second, mostly empty round:
  // the kernel keeps `occ` workgroups per CU resident (register-limited).
  const int occ = (MB == 1 && NBW == 1) ? 3 : ((MB * NBW <= 2) ? 2 : 1);
  const int slots = n_cus * occ;
  int splits = slots / wg_n;
  if (splits > total_iters / 2) splits = total_iters / 2;
  // Every split writes an M x N fp32 partial that is read back once and then sits dirty in the caches until the
  // next weight stream pushes it out to HBM; beyond 8 splits that costs more than the extra workgroups gain
  // (c2 forward -2.5 us, c5 -8 us against 16 and 12 splits).
  if (splits > max_splits) splits = max_splits;
  // The QKV product does as well with half as many splits while three quarters of the CUs still get a workgroup
  // (8B shape at 64 rows: the same 18 us with 192 workgroups as with 384; 70B shape at 16 rows: 36 against 37 us),
  // and every split less is an M x N partial less for the rotary step to read and to be written out of the caches
  // underneath the attention kernel (8B: -1.5 and -1 us).  The output and down projections lose more than the
  // kernels after them gain (70B shape: +2 and +8 us), so they keep their splits.
  if (MODE == EPI_STORE_BF16)
    while (splits >= 4 && splits % 2 == 0 && wg_n * (splits / 2) * 4 >= n_cus * 3) splits /= 2;
  if (splits < 1) splits = 1;
  // At most one workgroup of four waves per CU: eight waves, each column block's share of K cut in two slices that meet
  // through LDS, put twice as many waves on the weight stream for the same partial sums (8B shape, one row: QKV 13.8 ->
  // 12.1 us, O 7.9 -> 7.4, down 23.7 -> 20.5).  With two row blocks, or with more workgroups, it gains nothing or loses
  // (70B shape, 16 rows: QKV 33 -> 40 us with 320 workgroups), and below 1024 inputs the extra barriers cost more.
  if constexpr (MB == 1 && NBW == 1 && WAVES == 4 && KS == 1 && MODE != EPI_SWIGLU)
    if (wg_n * splits <= n_cus && total_iters >= 8 && total_iters % 2 == 0 && W.K % SK_BK == 0)
      return run_skinny_n<MB, MODE, 1, 8, 2>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer, max_splits);
  const int NP = W.NB * 32;
  while (splits > 1 && (size_t)splits * M * NP > ws_elems) --splits;
  int ips = (total_iters + splits - 1) / splits;
  if (KS > 1) ips = (ips + KS - 1) / KS * KS;  // (the callers see to it that total_iters is a multiple of KS)
  splits = (total_iters + ips - 1) / ips;
  size_t smem = (size_t)2 * KS * MB * 32 * SK_BK * sizeof(bf16_t);
  dim3 grid(wg_n, splits), block(WAVES * 64);
  if (splits == 1) {
    auto kern = gemm_skinny_kernel<MB, MODE, false, NBW, WAVES, KS>;
    static uint32_t lds_set = 0;
    hipError_t e = set_lds_limit_once((const void*)kern, smem, lds_set);
    if (e != hipSuccess) return e;
    kern<<<grid, block, smem, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, ips, epi, nullptr);
    return hipGetLastError();
  }
  auto kern = gemm_skinny_kernel<MB, MODE, true, NBW, WAVES, KS>;
  static uint32_t lds_set_partial = 0;
  hipError_t e = set_lds_limit_once((const void*)kern, smem, lds_set_partial);
  if (e != hipSuccess) return e;
  kern<<<grid, block, smem, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, ips, epi, ws);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (defer) { *defer = splits; return hipSuccess; }  // the caller's next kernel sums the partials
  return launch_splitk_epilogue<MODE>(splits, M, W, epi, ws, s);
}

template <int MB, int MODE>
static hipError_t run_skinny(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, float* ws,
                             size_t ws_elems, int n_cus, hipStream_t s, int* defer) {
  if constexpr (MODE == EPI_SWIGLU) {
    // What the streaming kernel leaves (takes_stream): K not a multiple of 64, weights under 48 MB, outputs that would be its
    // widest.  Wide enough MLPs fill the chip with one block per wave and no split at all (gate and up meet through LDS): no
    // partial sums to write, read back and write out of the caches.  Whole layers of 32 rows, weights from HBM, against the
    // split version with a gate/up pair per wave: 49152 x 448 67 us and 76, 57344 x 4128 169 and 188.
    if constexpr (MB <= 2) {
      if ((W.NB + 3) / 4 >= n_cus + n_cus / 2)
        return run_skinny_n<MB, MODE, 1>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer, 1);
      // narrower ones get there with workgroups of one pair (two waves): layers of 32 rows, 28672 x 512 54 us and 59, 28672 x
      // 768 59 and 68, 28672 x 4128 119 and 129
      if ((W.NB + 1) / 2 >= n_cus + n_cus / 2) {
        // With two row blocks a two-wave workgroup fetches as many activation bytes (through the L2) as weight
        // bytes.  Eight waves, two pairs times two K slices, share each slice's activation tile between two pairs
        // and put twice as many waves on the weight stream (layers of 64 rows, 28672 x 512 64.3 -> 63.6 us, 28672 x 768
        // 70.0 -> 69.3).  With one row block the two-wave form stays ahead.
        if (MB == 2 && W.K % (2 * SK_BK) == 0)
          return run_skinny_n<MB, MODE, 1, 8, 2>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer, 1);
        return run_skinny_n<MB, MODE, 1, 2>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer, 1);
      }
    }
    return run_skinny_n<MB, MODE, 2>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer);
  } else {
    // wide outputs (LM head): two blocks per wave halve the workgroup count and the activation reads from LDS
    if constexpr (MB <= 2)
      if ((W.NB + 3) / 4 > n_cus * (MB == 1 ? 3 : 2))
        return run_skinny_n<MB, MODE, 2>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer);
    return run_skinny_n<MB, MODE, 1>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer);
  }
}

// The epilogue arguments of rows m0.. of the same product.
template <int MODE>
static EpiArgs offset_rows(EpiArgs e, int m0) {
  if (MODE == EPI_STORE_BF16 || MODE == EPI_SWIGLU) e.out = reinterpret_cast<bf16_t*>(e.out) + (int64_t)m0 * e.ldo;
  if (MODE == EPI_STORE_F32 || MODE == EPI_RESID_EMBED || (MODE == EPI_RESID_OUT && e.out != nullptr))
    e.out = reinterpret_cast<float*>(e.out) + (int64_t)m0 * e.ldo;
  if ((MODE == EPI_RESID_EMBED || MODE == EPI_RESID_OUT) && e.ids != nullptr) e.ids += m0;
  if ((MODE == EPI_RESID_EMBED || MODE == EPI_RESID_OUT) && e.resid != nullptr) e.resid += (int64_t)m0 * e.H;
  return e;
}

// Tile height and split of K for a tiled product (K a multiple of 64).
struct TiledPlan {
  int rows;        // tile height: 96 or 128 (gemm_rows), 256 (gemm_large_async)
  int splits, kts; // splits of K and k steps per split
  int full_rows;   // leading rows in whole rounds of 256-row tiles, the rest as a product of its own; 0 = one product
  double us;
};

// The estimate every choice is made by: workgroups are spread evenly over the CUs, a workgroup's k step takes
//   rows   one workgroup per CU   all CUs full (two workgroups of gemm_rows, one of gemm_large_async)
//    96        0.70 us               1.42 us for both
//   128        0.75 us               1.65 us for both
//   256        1.35 us               1.55 us
// the weights come from HBM at 5.4 TB/s at best (the two add up by their cubes: both matter where they are close), a
// launch costs 3 us besides, and the partial sums of a split are written and read once at 6 TB/s (+ 3 us).  Fitted to
// sweeps of every tile and 1..16 splits for N x K = 6144 x 4096, 4096 x 4096, 28672 x 4096, 4096 x 14336, 3072 x 2048,
// 2048 x 2048, 16384 x 2048, 2048 x 8192, 10240 x 8192, 8192 x 8192, 57344 x 8192, 8192 x 28672 and the LM heads
// (128256 x 4096 and x 8192, 32000 x 2048) at 65 to 8320 rows; the form it picks is within 2% of the fastest on average.
// (With 1.25 us for a full chip of 96-row tiles, which holds for one round of them only, long products went to those:
// 28672 x 4096 at 1024 rows 231 us instead of 202, 57344 x 8192 at 4100 rows 3500 instead of 3016.)  What it replaces: one row of tiles with as many splits
// as CUs up to 256 rows and unsplit 256-row tiles beyond, which left most of the chip idle at a few hundred rows
// (4096 x 14336 at 333 rows: 32 workgroups, 308 us; now 240 and 53 us).
static TiledPlan plan_tiled(int M, int NB, int K, size_t ws_elems, int n_cus) {
  const int tiles_n = (NB + 7) / 8, KT = K / LG_BK, NP = NB * 32;
  const double stream_us = (double)NP * K * 2 / 5.4e6;
  TiledPlan best{0, 1, KT, 0, 1e30};
  const double stream_cube = stream_us * stream_us * stream_us;
  auto main_us = [&](double compute) { return 3.0 + std::cbrt(compute * compute * compute + stream_cube); };
  auto steps_us = [&](int rows, int64_t wgs) {  // time of one k step of all workgroups
    const int slots = rows == 256 ? n_cus : 2 * n_cus;
    const double one = rows == 96 ? 0.70 : rows == 128 ? 0.75 : 1.35, full = rows == 96 ? 1.42 : rows == 128 ? 1.65 : 1.55;
    const int64_t rem = wgs % slots;
    const bool light = rows == 256 ? rem * 8 <= (int64_t)n_cus * 7 && wgs < slots : rem <= n_cus;
    return (double)(wgs / slots) * full + (rem == 0 ? 0.0 : light ? one : full);
  };
  for (int rows : {96, 128, 256}) {
    const int tiles_m = (M + rows - 1) / rows;
    for (int splits = 1, last = 0; splits <= 16; ++splits) {
      const int kts = (KT + splits - 1) / splits;
      if (kts == last || (splits > 1 && kts < 4)) continue;
      last = kts;
      const int n = (KT + kts - 1) / kts;
      if (n > 1 && (size_t)n * M * NP > ws_elems) break;
      const double compute = kts * steps_us(rows, (int64_t)tiles_m * tiles_n * n);
      const double parts_us = n > 1 ? 3.0 + (double)n * M * NP * 8 / 6e6 : 0.0, left = best.us - 3.0 - parts_us;
      if (left <= 0.0 || compute * compute * compute + stream_cube >= left * left * left) continue;
      best = TiledPlan{rows, n, kts, 0, main_us(compute) + parts_us};
    }
  }
  // whole 256-row tiles whose remainder would open one more round of them
  const int full = M / LG_BM, ragged = M % LG_BM;
  if (full > 0 && ragged > 0) {
    const double us = main_us(KT * steps_us(256, (int64_t)full * tiles_n));
    if (us < best.us) {
      const double rest = plan_tiled(ragged, NB, K, ws_elems, n_cus).us;
      if (us + rest < best.us) best = TiledPlan{256, 1, KT, full * LG_BM, us + rest};
    }
  }
  return best;
}

// the tiled kernels step 64 contraction elements at a time and address both operands with 32-bit byte offsets
static bool tiled_ok(int M, int lda, int NB, int K) {
  return K % LG_BK == 0 && (int64_t)M * lda * 2 < ((int64_t)1 << 32) && (int64_t)NB * 32 * K * 2 < ((int64_t)1 << 32);
}

// The forms of gemm_stream and what a k step of a slice takes with one workgroup on every compute unit: step_us, and
// once per workgroup (the ring's fill, the slices' sums, the epilogue) wg_us; above 64 rows, and up to 64.
struct StreamForm { int mb, ks; double step_us, wg_us, few_step_us, few_wg_us; };
static constexpr StreamForm STREAM_FORMS[] = {
    {2, 1, 0.67, 10.2, 0.57, 3.6}, {2, 2, 0.78, 10.1, 0.64, 4.0}, {2, 4, 1.02, 9.5, 0.75, 4.2}, {3, 2, 0.93, 10.6, 0, 0}, {3, 4, 1.24, 11.1, 0, 0},
    {4, 1, 0.86, 12.7, 0, 0}, {4, 2, 1.07, 12.2, 0, 0}, {5, 1, 0.99, 12.7, 0, 0}, {5, 2, 1.22, 13.1, 0, 0}, {6, 1, 1.16, 11.6, 0, 0}};
// A whole product that ends in the residual has at most 8192 columns: 32 tiles of 256, with which row tiles of 160 and 192 leave at
// least half of 256 compute units idle.  No plan picks those there (the sums of six blocks and the residual's rows would not fit
// the registers either), and they are not built.
constexpr bool stream_resid_whole(int mb, int ks) { return ks > 1 || mb < 5; }
struct StreamPlan {
  int form;         // index into STREAM_FORMS, -1: none fits
  int splits, kts;  // splits of K and k steps per split, a multiple of the form's ks
  double us;
};

// The estimate: rounds of one workgroup per compute unit, the weights at 6.36 TB/s, the two added by their cubes as in
// plan_tiled, the partial sums of a split written and read once.  Up to 64 rows (one row tile) 3 us for a launch.  Above,
// up to eight row tiles: a step takes 0.65 of its time on an empty chip, growing with the workgroups; several row tiles
// fetch the weights 1.38 times; the 5.4 us taken off the sum are those that the rings' fills overlap with the stream.  Fitted
// to sweeps of every form and 1..10 splits at 80 to 760 rows for N x K = 16384 x 2048, 2048 x 8192, 3072 x 2048, 2048 x 2048,
// 28672 x 4096, 4096 x 14336, 6144 x 4096, 4096 x 4096, 10240 x 8192, 8192 x 8192 and 8192 x 28672 (and at 1 to 64 rows).
static StreamPlan plan_stream(int M, int NB, int K, size_t ws_elems, int n_cus, bool resid) {
  const int KT = K / LG_BK, NP = NB * 32;
  const bool few = M <= 64;
  const double stream_us = (double)NP * K * 2 / 6.36e6;
  StreamPlan best{-1, 1, KT, 1e30};
  for (int f = 0; f < (int)(sizeof(STREAM_FORMS) / sizeof(STREAM_FORMS[0])); ++f) {
    const StreamForm& F = STREAM_FORMS[f];
    if (KT % F.ks != 0 || (few && F.mb > 2)) continue;
    const int tiles_m = (M + F.mb * 32 - 1) / (F.mb * 32), tiles_n = (NB + 8 / F.ks - 1) / (8 / F.ks);
    if (tiles_m > 8) continue;
    const double stream = tiles_m == 1 ? stream_us : 1.38 * stream_us;
    for (int splits = 1, last = 0; splits <= 16; ++splits) {
      const int kts = (KT / F.ks + splits - 1) / splits * F.ks;
      if (kts == last) continue;
      last = kts;
      const int n = (KT + kts - 1) / kts;
      if ((KT - (n - 1) * kts) / F.ks < 4) continue;  // the ring is three or four steps deep, and every slice fills it
      if (n > 1 && (size_t)n * M * NP > ws_elems) break;
      if (n == 1 && resid && !stream_resid_whole(F.mb, F.ks)) continue;
      const int64_t wgs = (int64_t)tiles_m * tiles_n * n;
      const double rounds = (double)((wgs + n_cus - 1) / n_cus), load = wgs < n_cus ? 0.65 + 0.35 * (double)wgs / n_cus : 1.0;
      const double compute = rounds * (few ? kts / F.ks * F.few_step_us + F.few_wg_us : kts / F.ks * F.step_us * load + F.wg_us);
      const double rest = (few ? 3.0 : -5.4) + (n > 1 ? 2.5 + (double)n * M * NP * 8 / (few ? 5.5e6 : 6.8e6) : 0.0), left = best.us - rest;
      const double cubes = compute * compute * compute + stream * stream * stream;
      if (left <= 0.0 || cubes >= left * left * left) continue;  // (no root for what cannot win: the plan is made per launch)
      best = StreamPlan{f, n, kts, rest + std::cbrt(cubes)};
    }
  }
  return best;
}

// Where gemm_stream takes a product (tiled_ok holds).  Up to 64 rows gemm_skinny does as well
// with what streams in under 8 us and with most split products (6144 x 4096 at 16 rows 15.4 us there and 16 here, 4096 x
// 14336 24.0 and 24.5), so there it has to be an unsplit product of 48 MB and more (28672 x 4096 at 16 rows 43 -> 40 us,
// 16384 x 2048 23 -> 15, 32000 x 2048 at 64 rows 36 -> 32) or weights of 128 MiB and more (10240 x 8192 at 33 rows 37 -> 33,
// 8192 x 28672 79 -> 76); the widest outputs, where gemm_skinny gives a wave two column blocks, stay with it (128256 x 4096
// at 33 rows 165 us there, 175 here).  Above 64 rows the two estimates decide,
// the tiled kernels' corrected by what they were off by in the sweeps (unsplit products 16%, split ones 3%), up to 640 rows:
// there a streamed product beats them where the chip is filled by one round of whole contractions, or nearly so (3072 x 2048
// at 200 rows 15.9 -> 10.4 us, at 600 21.6 -> 16.5; 2048 x 2048 at 324 rows 14.9 -> 10.7; 6144 x 4096 at 450 rows 37 -> 31;
// 8192 x 8192 at 600 rows 96 -> 87), beyond whole rounds of 256-row tiles (57344 x 8192 at 700 rows 598, 629 streamed).
// A split qkv or output product is summed by the kernel that follows, for 2 to 3 us less than the epilogue kernel that the
// sweeps timed with it: a whole one has to win by that much (without it a layer of 256 rows lost 3 us in a whole layer).
// Weights under 10 MiB are streamed unsplit and above 220 rows only (2048 x 2048 at 200 rows 10.7 us, in 8 parts of 96-row
// tiles 9.0; 1536 x 1024 at 324 rows 7.5 and 12.5).  Over the products of plan_stream's sweeps the choice gains 6% on
// average against the former rule (32 MiB and more, up to 384 rows and two row tiles), and is 2% off the fastest.
static bool takes_stream(int M, int NB, int K, size_t ws_elems, int n_cus, bool resid, const TiledPlan* tiled, StreamPlan& p) {
  const int64_t bytes = (int64_t)NB * 32 * K * 2;
  if (M > 64) {
    const bool small = bytes < (int64_t)10 << 20;
    if (M > 640 || (small && M <= 220)) return false;
    p = plan_stream(M, NB, K, small ? 0 : ws_elems, n_cus, resid);
    const double saved = p.splits == 1 && tiled->splits > 1 ? 2.5 : 0.0;  // what the next kernel saves of a split's epilogue
    return p.form >= 0 && p.us + 0.8 + saved < tiled->us * (tiled->splits == 1 ? 1.16 : 1.03);
  }
  if (bytes < 48000000 || (NB + 3) / 4 > n_cus * (M <= 32 ? 3 : 2)) return false;
  const bool unsplit = bytes < ((int64_t)1 << 27);
  p = plan_stream(M, NB, K, unsplit ? 0 : ws_elems, n_cus, resid);
  if (p.form < 0) return false;
  return !unsplit || ((int64_t)NB * STREAM_FORMS[p.form].ks + 7) / 8 * 4 >= n_cus * 3;
}

template <int MODE, bool PARTIAL>
static hipError_t run_tiles(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, const TiledPlan& p,
                            float* ws, hipStream_t s) {
  const int tiles_n = (W.NB + 7) / 8, tiles_m = (M + p.rows - 1) / p.rows;
  const dim3 grid(tiles_m * tiles_n, p.splits), block(512);
  if (p.rows == 96)
    gemm_rows_kernel<MODE, PARTIAL, 3><<<grid, block, 0, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, epi, tiles_m, tiles_n, p.kts, ws);
  else if (p.rows == 128)
    gemm_rows_kernel<MODE, PARTIAL, 4><<<grid, block, 0, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, epi, tiles_m, tiles_n, p.kts, ws);
  else
    gemm_large_async_kernel<MODE, PARTIAL><<<grid, block, 0, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, epi, tiles_m, tiles_n, p.kts, ws);
  return hipGetLastError();
}

template <int MODE, int MB, int KS>
static hipError_t run_stream_form(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, const StreamPlan& p,
                                  float* ws, hipStream_t s) {
  const int tiles_n = (W.NB + 8 / KS - 1) / (8 / KS), tiles_m = (M + MB * 32 - 1) / (MB * 32);
  const dim3 grid(tiles_m * tiles_n, p.splits), block(512);
  // (raw partial sums depend on the mode by how they are stored only)
  constexpr int PART_MODE = MODE == EPI_STORE_F32 || MODE == EPI_RESID_OUT ? EPI_RESID_OUT : EPI_RESID_EMBED;
  if (p.splits == 1) {
    if constexpr ((MODE != EPI_RESID_EMBED && MODE != EPI_RESID_OUT) || stream_resid_whole(MB, KS))
      gemm_stream_kernel<MODE, false, MB, KS><<<grid, block, 0, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, epi, tiles_m, tiles_n, p.kts, ws);
    else return hipErrorInvalidValue;  // (no plan says so)
  } else gemm_stream_kernel<PART_MODE, true, MB, KS><<<grid, block, 0, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, epi, tiles_m, tiles_n, p.kts, ws);
  return hipGetLastError();
}

template <int MODE>
static hipError_t run_stream(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, const StreamPlan& p, float* ws,
                             hipStream_t s) {
  const StreamForm& F = STREAM_FORMS[p.form];
  switch (F.mb * 8 + F.ks) {
    case 2 * 8 + 1: return run_stream_form<MODE, 2, 1>(A, lda, M, W, epi, p, ws, s);
    case 2 * 8 + 2: return run_stream_form<MODE, 2, 2>(A, lda, M, W, epi, p, ws, s);
    case 2 * 8 + 4: return run_stream_form<MODE, 2, 4>(A, lda, M, W, epi, p, ws, s);
    case 3 * 8 + 2: return run_stream_form<MODE, 3, 2>(A, lda, M, W, epi, p, ws, s);
    case 3 * 8 + 4: return run_stream_form<MODE, 3, 4>(A, lda, M, W, epi, p, ws, s);
    case 4 * 8 + 1: return run_stream_form<MODE, 4, 1>(A, lda, M, W, epi, p, ws, s);
    case 4 * 8 + 2: return run_stream_form<MODE, 4, 2>(A, lda, M, W, epi, p, ws, s);
    case 5 * 8 + 1: return run_stream_form<MODE, 5, 1>(A, lda, M, W, epi, p, ws, s);
    case 5 * 8 + 2: return run_stream_form<MODE, 5, 2>(A, lda, M, W, epi, p, ws, s);
    case 6 * 8 + 1: return run_stream_form<MODE, 6, 1>(A, lda, M, W, epi, p, ws, s);
  }
  return hipErrorInvalidValue;
}

// What follows a product split along K: the caller's next kernel sums the partials, or the epilogue kernel does.
template <int MODE>
static hipError_t finish_split(int splits, int M, const PackedWeight& W, const EpiArgs& epi, float* ws, hipStream_t s, int* defer) {
  if (defer) { *defer = splits; return hipSuccess; }
  return launch_splitk_epilogue<MODE>(splits, M, W, epi, ws, s);
}

template <int MODE>
static hipError_t run_mode(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, float* ws,
                           size_t ws_elems, int n_cus, hipStream_t s, int* defer) {
  if (M <= 0) return hipSuccess;
  const bool tiled = tiled_ok(M, lda, W.NB, W.K);
  constexpr bool RESID = MODE == EPI_RESID_EMBED || MODE == EPI_RESID_OUT;
  StreamPlan sp;
  if (M <= 64) {
    if (tiled && takes_stream(M, W.NB, W.K, ws_elems, n_cus, RESID, nullptr, sp)) {
      hipError_t e = run_stream<MODE>(A, lda, M, W, epi, sp, ws, s);
      return e != hipSuccess || sp.splits == 1 ? e : finish_split<MODE>(sp.splits, M, W, epi, ws, s, defer);
    }
    return M <= 32 ? run_skinny<1, MODE>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer)
                   : run_skinny<2, MODE>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer);
  }
  if (tiled) {
    const TiledPlan p = plan_tiled(M, W.NB, W.K, ws_elems, n_cus);
    if (takes_stream(M, W.NB, W.K, ws_elems, n_cus, RESID, &p, sp)) {
      hipError_t e = run_stream<MODE>(A, lda, M, W, epi, sp, ws, s);
      return e != hipSuccess || sp.splits == 1 ? e : finish_split<MODE>(sp.splits, M, W, epi, ws, s, defer);
    }
    if (p.full_rows > 0) {
      hipError_t e = run_tiles<MODE, false>(A, lda, p.full_rows, W, epi, p, nullptr, s);
      if (e != hipSuccess) return e;
      return run_mode<MODE>(A + (int64_t)p.full_rows * lda, lda, M - p.full_rows, W, offset_rows<MODE>(epi, p.full_rows), ws,
                            ws_elems, n_cus, s, nullptr);
    }
    if (p.splits == 1) return run_tiles<MODE, false>(A, lda, M, W, epi, p, nullptr, s);
    hipError_t e = run_tiles<MODE, true>(A, lda, M, W, epi, p, ws, s);
    return e != hipSuccess ? e : finish_split<MODE>(p.splits, M, W, epi, ws, s, defer);
  }
  if (M <= 128) return run_skinny<4, MODE>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer);
  if constexpr (MODE != EPI_SWIGLU) {  // (eight row blocks of gate/up pairs would not fit the register file)
    if (M <= 256) return run_skinny<8, MODE>(A, lda, M, W, epi, ws, ws_elems, n_cus, s, defer);
  }
  auto kern = gemm_large_kernel<MODE>;
  size_t smem = (size_t)4 * LG_BM * LG_BK * sizeof(bf16_t);
  static uint32_t lds_set_large = 0;
  hipError_t e = set_lds_limit_once((const void*)kern, smem, lds_set_large);
  if (e != hipSuccess) return e;
  dim3 grid((W.NB + 7) / 8, (M + LG_BM - 1) / LG_BM), block(512);
  kern<<<grid, block, smem, s>>>(A, lda, M, W.data, W.N, W.NB, W.K, epi);
  return hipGetLastError();
}

hipError_t launch_gemm(const bf16_t* A, int lda, int M, const PackedWeight& W, const EpiArgs& epi, float* splitk_ws,
                       size_t splitk_elems, int n_cus, hipStream_t s, int* deferred_splits) {
  int* defer = deferred_splits;  // used where the whole product goes through one split-K launch
  if (defer) *defer = 0;
  switch (epi.mode) {
    case EPI_STORE_BF16: return run_mode<EPI_STORE_BF16>(A, lda, M, W, epi, splitk_ws, splitk_elems, n_cus, s, defer);
    case EPI_RESID_EMBED: return run_mode<EPI_RESID_EMBED>(A, lda, M, W, epi, splitk_ws, splitk_elems, n_cus, s, defer);
    case EPI_SWIGLU: return run_mode<EPI_SWIGLU>(A, lda, M, W, epi, splitk_ws, splitk_elems, n_cus, s, defer);
    case EPI_RESID_OUT: return run_mode<EPI_RESID_OUT>(A, lda, M, W, epi, splitk_ws, splitk_elems, n_cus, s, defer);
    case EPI_STORE_F32: return run_mode<EPI_STORE_F32>(A, lda, M, W, epi, splitk_ws, splitk_elems, n_cus, s, defer);
  }
  return hipErrorInvalidValue;
}

void product_plan(int M, int N, int K, size_t ws_elems, int n_cus, int64_t out[4]) {
  out[0] = out[1] = out[2] = out[3] = 0;
  const int NB = (N + 31) / 32;
  if (M <= 64 || !tiled_ok(M, K, NB, K)) return;
  const TiledPlan p = plan_tiled(M, NB, K, ws_elems, n_cus);
  const int tiles_m = ((p.full_rows ? p.full_rows : M) + p.rows - 1) / p.rows, tiles_n = (NB + 7) / 8, n = tiles_m * tiles_n;
  out[0] = p.rows;
  out[1] = p.splits;
  out[2] = p.full_rows;
  std::vector<uint8_t> fetched((size_t)tiles_n * p.splits, 0);  // XCDs that work on a column tile (of a part of K)
  for (int split = 0; split < p.splits; ++split)
    for (int id = 0; id < n; ++id) {
      int tm, tn;
      tile_at(xcd_range(id, tiles_m, tiles_n), tiles_m, tiles_n, tm, tn);
      fetched[(size_t)split * tiles_n + tn] |= 1u << ((split * (int64_t)n + id) % 8);
    }
  for (uint8_t f : fetched) out[3] += __builtin_popcount(f);
}

void product_stream(int M, int N, int K, size_t ws_elems, int n_cus, int64_t out[3]) {
  out[0] = out[1] = out[2] = 0;
  const int NB = (N + 31) / 32;
  if (!tiled_ok(M, K, NB, K)) return;
  StreamPlan p;
  TiledPlan t{};
  if (M > 64) t = plan_tiled(M, NB, K, ws_elems, n_cus);
  if (!takes_stream(M, NB, K, ws_elems, n_cus, false, &t, p)) return;
  out[0] = STREAM_FORMS[p.form].mb * 32;
  out[1] = STREAM_FORMS[p.form].ks;
  out[2] = p.splits;
}
