// Memory-bound helper kernels: weight tiling, RMSNorm, rotary step + KV append into pages,
// Embed / KvPage pool copies.
#include <type_traits>

#include "internal.h"

// ---------------------------------------------------------------------------------------------
// Weight tiling: up to three [rows_i, K] matrices stacked (or two interleaved in 32-row blocks)
// into the tiled layout described in common.h.  One thread moves one 16-byte piece.
// ---------------------------------------------------------------------------------------------
__global__ void pack_weight_kernel(const bf16_t* __restrict__ s0, int r0, const bf16_t* __restrict__ s1, int r1,
                                   const bf16_t* __restrict__ s2, int r2, int K, int interleave,
                                   bf16_t* __restrict__ dst, int NB) {
  const int KB = K / 16;
  int64_t piece = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one per (nb, kb, lane)
  int64_t total = (int64_t)NB * KB * 64;
  if (piece >= total) return;
  int lane = (int)(piece & 63);
  int64_t tile = piece >> 6;
  int kb = (int)(tile % KB);
  int nb = (int)(tile / KB);
  int n = nb * 32 + (lane & 31);
  int k = kb * 16 + (lane >> 5) * 8;
  const bf16_t* src = nullptr;
  if (interleave) {  // block 2b <- s0 rows [32b, 32b+32), block 2b+1 <- s1 rows [32b, 32b+32)
    int row = (nb >> 1) * 32 + (lane & 31);
    if (row < r0) src = ((nb & 1) ? s1 : s0) + (int64_t)row * K + k;
  } else {
    if (n < r0) src = s0 + (int64_t)n * K + k;
    else if (n < r0 + r1) src = s1 + (int64_t)(n - r0) * K + k;
    else if (n < r0 + r1 + r2) src = s2 + (int64_t)(n - r0 - r1) * K + k;
  }
  u32x4 v = {0, 0, 0, 0};
  if (src) v = *reinterpret_cast<const u32x4*>(src);
  *reinterpret_cast<u32x4*>(dst + piece * 8) = v;
}

hipError_t launch_pack_weight(const bf16_t* s0, int r0, const bf16_t* s1, int r1, const bf16_t* s2, int r2, int K,
                              int interleave, bf16_t* dst, int NB, hipStream_t s) {
  int64_t total = (int64_t)NB * (K / 16) * 64;
  int64_t blocks = (total + 255) / 256;
  pack_weight_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(s0, r0, s1, r1, s2, r2, K, interleave, dst, NB);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// RMSNorm: one workgroup per row, values kept in registers.
// ---------------------------------------------------------------------------------------------
// The row comes from an Embed (NORM_EMBED), from a wide fp32 row (NORM_F32), or is first formed as residual +
// split-K partial sums of the projection before it (NORM_PARTIAL: partials added in split order, then the
// residual, exactly as the stand-alone split-K epilogue does, and the wide row is stored as well).
enum { NORM_EMBED = 0, NORM_F32 = 1, NORM_PARTIAL = 2 };
struct NormPartial {
  const float* part;    // [splits][rows][NP]
  int splits, NP, rows;
  const float* resid;   // [rows, H] fp32, or null: the residual is Embed ids[row]
  float* wide;          // [rows, H] fp32 destination of residual + sum
};

// id: the row's Embed, for the sources that read one.  A thread holds eight columns (THREADS * 8 >= H).  At decode sizes the
// kernel is a chain of latencies, so everything that does not depend on the row's sum is requested at once: gain, residual
// and eight partial sums at a time (one row of 256 threads that took two passes over 4096 columns and read the gain behind
// the reduction: 4.3 us for 64 Embed rows, 6.0 with eight partial sums; now 3.6 and 5.2).
template <int SRC, int THREADS>
__device__ __forceinline__ void rmsnorm_row(int row, int id, const void* __restrict__ xin, const bf16_t* __restrict__ gain,
                                            bf16_t* __restrict__ out, int H, float eps, const NormPartial& np) {
  __shared__ float red[THREADS / 64];
  const int tid = threadIdx.x, c = tid * 8;
  float vals[8];
  float ss = 0.f;
  Pack16 g;
  if (c < H) {
    g.u = *reinterpret_cast<const u32x4*>(gain + c);
    if (SRC == NORM_EMBED) {
      Pack16 pk;
      pk.u = *reinterpret_cast<const u32x4*>(reinterpret_cast<const bf16_t*>(xin) + (int64_t)id * H + c);
#pragma unroll
      for (int e = 0; e < 8; ++e) vals[e] = bf16_bits_to_f32(pk.s[e]);
    } else if (SRC == NORM_PARTIAL) {
      f32x4 ra, rb;
      Pack16 pk;
      if (np.resid != nullptr) {
        ra = *reinterpret_cast<const f32x4*>(np.resid + (int64_t)row * H + c);
        rb = *reinterpret_cast<const f32x4*>(np.resid + (int64_t)row * H + c + 4);
      } else {
        pk.u = *reinterpret_cast<const u32x4*>(reinterpret_cast<const bf16_t*>(xin) + (int64_t)id * H + c);
      }
      f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
      const float* pp = np.part + (int64_t)row * np.NP + c;
      const int64_t stride = (int64_t)np.rows * np.NP;
      int k = 0;
      for (; k + 8 <= np.splits; k += 8) {  // eight splits requested together, added in order
        f32x4 va[8], vb[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          va[u] = *reinterpret_cast<const f32x4*>(pp + (k + u) * stride);
          vb[u] = *reinterpret_cast<const f32x4*>(pp + (k + u) * stride + 4);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) { a += va[u]; b += vb[u]; }
      }
      if (k + 4 <= np.splits) {
        f32x4 va[4], vb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          va[u] = *reinterpret_cast<const f32x4*>(pp + (k + u) * stride);
          vb[u] = *reinterpret_cast<const f32x4*>(pp + (k + u) * stride + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { a += va[u]; b += vb[u]; }
        k += 4;
      }
      for (; k < np.splits; ++k) {
        a += *reinterpret_cast<const f32x4*>(pp + k * stride);
        b += *reinterpret_cast<const f32x4*>(pp + k * stride + 4);
      }
      if (np.resid == nullptr) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { ra[e] = bf16_bits_to_f32(pk.s[e]); rb[e] = bf16_bits_to_f32(pk.s[4 + e]); }
      }
      a += ra;
      b += rb;
      *reinterpret_cast<f32x4*>(np.wide + (int64_t)row * H + c) = a;
      *reinterpret_cast<f32x4*>(np.wide + (int64_t)row * H + c + 4) = b;
#pragma unroll
      for (int e = 0; e < 4; ++e) { vals[e] = a[e]; vals[4 + e] = b[e]; }
    } else {
      const float* x = reinterpret_cast<const float*>(xin) + (int64_t)row * H + c;
      const f32x4 a = *reinterpret_cast<const f32x4*>(x), b = *reinterpret_cast<const f32x4*>(x + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { vals[e] = a[e]; vals[4 + e] = b[e]; }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += vals[e] * vals[e];
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) tot += red[w];
  const float rstd = 1.0f / sqrtf(tot / (float)H + eps);
  if (c < H) {
    Pack16 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o.h[e] = f32_to_bf16(vals[e] * rstd * bf16_bits_to_f32(g.s[e]));
    *reinterpret_cast<u32x4*>(out + (int64_t)row * H + c) = o.u;
  }
}

template <int SRC, int THREADS>
__global__ __launch_bounds__(THREADS) void rmsnorm_kernel(const void* __restrict__ xin, const int32_t* __restrict__ ids,
                                                      const bf16_t* __restrict__ gain, bf16_t* __restrict__ out,
                                                      int H, float eps, NormPartial np) {
  const int row = blockIdx.x;
  const int id = SRC == NORM_EMBED || (SRC == NORM_PARTIAL && np.resid == nullptr) ? ids[row] : 0;
  rmsnorm_row<SRC, THREADS>(row, id, xin, gain, out, H, eps, np);
}

// The same over Embeds whose ids are kernel arguments: calls that take an id list from the host (distributions, reads and
// writes of Embeds) need no copy to the device in front of their first kernel, which was a launch of its own: 4.6 us of a
// pass that reads up to IDS_BY_VALUE output Embeds (one row through an 8B-shaped layer: 130 -> 124 us with the read).
// Longer lists go through a device buffer.  The smaller argument block is for the usual few rows.
template <int N>
struct IdArgs {
  int32_t v[N];
};
template <int N, int THREADS>
__global__ __launch_bounds__(THREADS) void rmsnorm_ids_kernel(const bf16_t* __restrict__ embeds, IdArgs<N> ids,
                                                          const bf16_t* __restrict__ gain, bf16_t* __restrict__ out,
                                                          int H, float eps) {
  rmsnorm_row<NORM_EMBED, THREADS>(blockIdx.x, ids.v[blockIdx.x], embeds, gain, out, H, eps, NormPartial{});
}

// Calls launch with the workgroup size a row of H columns takes.
template <typename F>
static hipError_t norm_threads(int H, F launch) {
  if (H <= 2048) launch(std::integral_constant<int, 256>{});
  else if (H <= 4096) launch(std::integral_constant<int, 512>{});
  else if (H <= 8192) launch(std::integral_constant<int, 1024>{});
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int N>
static IdArgs<N> id_args(const int32_t* ids, int n) {
  IdArgs<N> a;
  for (int i = 0; i < n; ++i) a.v[i] = ids[i];
  for (int i = n; i < N; ++i) a.v[i] = 0;
  return a;
}

hipError_t launch_rmsnorm_embed_ids(const bf16_t* embeds, const int32_t* host_ids, const bf16_t* gain, bf16_t* out, int rows,
                                    int H, float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (rows > IDS_BY_VALUE) return hipErrorInvalidValue;
  return norm_threads(H, [&](auto t_c) {
    constexpr int T = decltype(t_c)::value;
    if (rows <= 64) rmsnorm_ids_kernel<64, T><<<dim3(rows), dim3(T), 0, s>>>(embeds, id_args<64>(host_ids, rows), gain, out, H, eps);
    else rmsnorm_ids_kernel<IDS_BY_VALUE, T><<<dim3(rows), dim3(T), 0, s>>>(embeds, id_args<IDS_BY_VALUE>(host_ids, rows), gain, out, H, eps);
  });
}
hipError_t launch_rmsnorm_embed(const bf16_t* embeds, const int32_t* ids, const bf16_t* gain, bf16_t* out, int rows,
                                int H, float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  return norm_threads(H, [&](auto t_c) {
    constexpr int T = decltype(t_c)::value;
    rmsnorm_kernel<NORM_EMBED, T><<<dim3(rows), dim3(T), 0, s>>>(embeds, ids, gain, out, H, eps, NormPartial{});
  });
}
hipError_t launch_rmsnorm_f32(const float* x, const bf16_t* gain, bf16_t* out, int rows, int H, float eps,
                              hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  return norm_threads(H, [&](auto t_c) {
    constexpr int T = decltype(t_c)::value;
    rmsnorm_kernel<NORM_F32, T><<<dim3(rows), dim3(T), 0, s>>>(x, nullptr, gain, out, H, eps, NormPartial{});
  });
}
hipError_t launch_splitk_resid_norm(const float* part, int splits, int NP, const float* resid, const bf16_t* embeds,
                                    const int32_t* ids, float* wide, const bf16_t* gain, bf16_t* out, int rows, int H,
                                    float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (splits <= 0 || NP < H || (resid == nullptr && (embeds == nullptr || ids == nullptr))) return hipErrorInvalidValue;
  return norm_threads(H, [&](auto t_c) {
    constexpr int T = decltype(t_c)::value;
    rmsnorm_kernel<NORM_PARTIAL, T><<<dim3(rows), dim3(T), 0, s>>>(embeds, ids, gain, out, H, eps,
                                                                  NormPartial{part, splits, NP, rows, resid, wide});
  });
}

// ---------------------------------------------------------------------------------------------
// Rotary step + KV append.  qkv is [T, (Hq + 2 Hkv) * D] bf16.  A rotary thread handles the 8 pairs
// (c*8 + e, D/2 + c*8 + e) of `hpt` consecutive query/key heads of one token, so the 8 angles
// pos * theta^(-2i/D), evaluated in double (positions reach tens of thousands), are computed once for all of
// them; a value thread handles 16 consecutive elements of a token, or two of eight tokens.  Rotated queries are written back in place; rotated
// keys and values go to the token's page slot.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rope_append_kernel(bf16_t* __restrict__ qkv, int T, int Hq, int Hkv, int D,
                                                          const int32_t* __restrict__ pos,
                                                          const int32_t* __restrict__ tok_page,
                                                          const int32_t* __restrict__ tok_slot,
                                                          const float* __restrict__ angles,
                                                          bf16_t* __restrict__ kv_layer, int hpt, bool by_octet,
                                                          const float* __restrict__ part, int splits, int NP) {
  // Eight consecutive values each of token t from columns `col0` and `col1` of its qkv row: read as stored, or (splits > 0)
  // summed in split order from the partials of the QKV product and rounded to bf16 like the stored row would be.  Both
  // pieces' loads of up to four splits go out together.
  auto load_two = [&](int t, int col0, int col1, Pack16& r0, Pack16& r1) {
    if (splits > 0) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0, s2 = s0, s3 = s0;
      const float* pp = part + (int64_t)t * NP;
      const int64_t stride = (int64_t)T * NP;
      int k = 0;
      for (; k + 4 <= splits; k += 4) {
        f32x4 v0[4], v1[4], v2[4], v3[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float* q = pp + (k + u) * stride;
          v0[u] = *reinterpret_cast<const f32x4*>(q + col0);
          v1[u] = *reinterpret_cast<const f32x4*>(q + col0 + 4);
          v2[u] = *reinterpret_cast<const f32x4*>(q + col1);
          v3[u] = *reinterpret_cast<const f32x4*>(q + col1 + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { s0 += v0[u]; s1 += v1[u]; s2 += v2[u]; s3 += v3[u]; }
      }
      for (; k < splits; ++k) {
        const float* q = pp + k * stride;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(q + col0), v1 = *reinterpret_cast<const f32x4*>(q + col0 + 4);
        const f32x4 v2 = *reinterpret_cast<const f32x4*>(q + col1), v3 = *reinterpret_cast<const f32x4*>(q + col1 + 4);
        s0 += v0; s1 += v1; s2 += v2; s3 += v3;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r0.h[e] = f32_to_bf16(s0[e]); r0.h[4 + e] = f32_to_bf16(s1[e]);
        r1.h[e] = f32_to_bf16(s2[e]); r1.h[4 + e] = f32_to_bf16(s3[e]);
      }
    } else {
      r0.u = *reinterpret_cast<const u32x4*>(qkv + (int64_t)t * NP + col0);
      r1.u = *reinterpret_cast<const u32x4*>(qkv + (int64_t)t * NP + col1);
    }
  };
  const int cpt = D / 16;  // work pieces per head
  const int heads = Hq + 2 * Hkv, rot = Hq + Hkv;
  const int groups = (rot + hpt - 1) / hpt;
  const int64_t n_rot = (int64_t)T * groups * cpt, n_val = (int64_t)((T + 7) / 8 * 8) * Hkv * cpt;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_rot + n_val) return;
  if (idx < n_rot) {
    const int c = (int)(idx % cpt);
    const int g = (int)((idx / cpt) % groups);
    const int t = (int)(idx / ((int64_t)cpt * groups));
    const int page = tok_page[t], slot = tok_slot[t];
    float fc[8], fs[8];  // cos and sin of the token's 8 angles of this piece, from the batch's table
    {
      const float* ang = angles + (int64_t)t * D + c * 8;
      const f32x4 c0 = *reinterpret_cast<const f32x4*>(ang), c1 = *reinterpret_cast<const f32x4*>(ang + 4);
      const f32x4 s0 = *reinterpret_cast<const f32x4*>(ang + D / 2), s1 = *reinterpret_cast<const f32x4*>(ang + D / 2 + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { fc[e] = c0[e]; fc[4 + e] = c1[e]; fs[e] = s0[e]; fs[4 + e] = s1[e]; }
    }
    const int h1 = min(rot, (g + 1) * hpt);
    for (int h = g * hpt; h < h1; ++h) {
      bf16_t* row = qkv + (int64_t)t * heads * D + (int64_t)h * D;
      Pack16 olo, ohi;
      Pack16 lo, hi;
      load_two(t, h * D + c * 8, h * D + D / 2 + c * 8, lo, hi);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float a = bf16_bits_to_f32(lo.s[e]), b = bf16_bits_to_f32(hi.s[e]);
        olo.h[e] = f32_to_bf16(a * fc[e] - b * fs[e]);
        ohi.h[e] = f32_to_bf16(b * fc[e] + a * fs[e]);
      }
      if (h < Hq) {
        *reinterpret_cast<u32x4*>(row + c * 8) = olo.u;
        *reinterpret_cast<u32x4*>(row + D / 2 + c * 8) = ohi.u;
      } else {
        bf16_t* blk = kv_layer + ((int64_t)page * Hkv + (h - Hq)) * (2 * PAGE * D);
        *reinterpret_cast<u32x4*>(blk + k_elem_offset(slot, c * 8)) = olo.u;
        *reinterpret_cast<u32x4*>(blk + k_elem_offset(slot, D / 2 + c * 8)) = ohi.u;
      }
    }
  } else {
    // by_octet: eight consecutive tokens of one (head, piece) sit in neighbouring lanes; else the pieces of one token do
    idx -= n_rot;
    const int per8 = 8 * Hkv * cpt;
    const int in8 = (int)(idx % per8), piece = by_octet ? in8 >> 3 : in8 % (Hkv * cpt);
    const int t = (int)(idx / per8) * 8 + (by_octet ? in8 & 7 : in8 / (Hkv * cpt));
    if (t >= T) return;
    const int c = piece % cpt, hv = piece / cpt;
    const int page = tok_page[t], slot = tok_slot[t];
    bf16_t* blk = kv_layer + ((int64_t)page * Hkv + hv) * (2 * PAGE * D);
    // The V part keeps the 8 tokens of slots 8k .. 8k+7 next to each other for every d.  When the batch fills such an
    // octet with consecutive tokens (prefill), its eight threads share the work by d: the thread of slot 8k + i gathers
    // values 2i and 2i + 1 of the piece from all eight tokens (its neighbours read the bytes next to them) and stores 16
    // bytes per d; single tokens (decode) store their 2-byte values one by one.  (One thread per octet, the other seven
    // idle, left a long chain of loads at the end: 333 tokens over three split-K copies 20 -> 10 us,
    // 8320 tokens 51 -> 49.  For batches of single tokens that order of lanes costs 1.5 us at 157 tokens.)
    const int t0 = t - (slot & 7);
    bool octet = by_octet && t0 >= 0 && t0 + 7 < T;
    if (octet) {
#pragma unroll
      for (int i = 0; i < 8; ++i) octet = octet && tok_page[t0 + i] == page && tok_slot[t0 + i] == (slot & ~7) + i;
    }
    if (octet) {
      const int d = c * 16 + (slot & 7) * 2, col = (rot + hv) * D + d;
      Pack16 o0, o1;
      if (splits > 0) {
        float s0[8], s1[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) { s0[i] = 0.f; s1[i] = 0.f; }
        const int64_t stride = (int64_t)T * NP;
        for (int k = 0; k < splits; ++k) {
          f32x2 v[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const f32x2*>(part + k * stride + (int64_t)(t0 + i) * NP + col);
#pragma unroll
          for (int i = 0; i < 8; ++i) { s0[i] += v[i][0]; s1[i] += v[i][1]; }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) { o0.h[i] = f32_to_bf16(s0[i]); o1.h[i] = f32_to_bf16(s1[i]); }
      } else {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const uint32_t*>(qkv + (int64_t)(t0 + i) * NP + col);
#pragma unroll
        for (int i = 0; i < 8; ++i) { o0.s[i] = (uint16_t)v[i]; o1.s[i] = (uint16_t)(v[i] >> 16); }
      }
      *reinterpret_cast<u32x4*>(blk + v_elem_offset(slot & ~7, d, D)) = o0.u;
      *reinterpret_cast<u32x4*>(blk + v_elem_offset(slot & ~7, d + 1, D)) = o1.u;
      return;
    }
    Pack16 a, b;
    load_two(t, (rot + hv) * D + c * 16, (rot + hv) * D + c * 16 + 8, a, b);
    uint16_t* dst = reinterpret_cast<uint16_t*>(blk);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      dst[v_elem_offset(slot, c * 16 + e, D)] = a.s[e];
      dst[v_elem_offset(slot, c * 16 + 8 + e, D)] = b.s[e];
    }
  }
}

// cos and sin of every (token, frequency) of a batch: angles[t][0 .. D/2) = cos, [D/2 .. D) = sin of
// pos[t] * inv_freq[i], evaluated in double precision and rounded to float.  Positions do not change from layer to
// layer, so the table is made once per batch and every layer's rotary step reads it.
__global__ void rope_table_kernel(const int32_t* __restrict__ pos, const double* __restrict__ inv_freq, int T, int half,
                                  float* __restrict__ angles) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)T * half) return;
  const int t = (int)(idx / half), i = (int)(idx % half);
  double sn, cs;
  sincos((double)pos[t] * inv_freq[i], &sn, &cs);
  angles[(int64_t)t * 2 * half + i] = (float)cs;
  angles[(int64_t)t * 2 * half + half + i] = (float)sn;
}

hipError_t launch_rope_table(const int32_t* pos, const double* inv_freq, int T, int D, float* angles, hipStream_t s) {
  const int64_t total = (int64_t)T * (D / 2);
  if (total <= 0) return hipSuccess;
  rope_table_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(pos, inv_freq, T, D / 2, angles);
  return hipGetLastError();
}

hipError_t launch_rope_append(bf16_t* qkv, int T, int Hq, int Hkv, int D, const int32_t* pos, const int32_t* tok_page,
                              const int32_t* tok_slot, const float* angles, bf16_t* kv_layer, bool by_octet,
                              const float* part, int splits, int NP, hipStream_t s) {
  if (splits > 0 && (part == nullptr || NP < (Hq + 2 * Hkv) * D)) return hipErrorInvalidValue;
  if (splits <= 0) NP = (Hq + 2 * Hkv) * D;  // row length of the stored qkv
  // few tokens: one head per thread keeps enough threads in flight; many tokens: a thread walks several heads
  // with the same 8 angles
  const int hpt = T >= 1024 ? 8 : 1;
  const int groups = (Hq + Hkv + hpt - 1) / hpt;
  int64_t total = ((int64_t)T * groups + (int64_t)((T + 7) / 8 * 8) * Hkv) * (D / 16);
  if (total <= 0) return hipSuccess;
  // Few threads: workgroups of one wave, so that they reach every compute unit (64 tokens of the 8B shape are 96 workgroups
  // of four waves).
  const int wg = total < 512 * 256 ? 64 : 256;
  rope_append_kernel<<<dim3((unsigned)((total + wg - 1) / wg)), dim3(wg), 0, s>>>(qkv, T, Hq, Hkv, D, pos, tok_page, tok_slot,
                                                                                    angles, kv_layer, hpt, by_octet, part, splits, NP);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Pool copies for seeding and inspection.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void embed_copy_piece(bf16_t* __restrict__ embeds, int id, int64_t idx, int H,
                                                 bf16_t* __restrict__ buf, int to_pool) {
  bf16_t* p = embeds + (int64_t)id * H + (int)(idx % (H / 8)) * 8;
  bf16_t* b = buf + idx * 8;
  if (to_pool) *reinterpret_cast<u32x4*>(p) = *reinterpret_cast<const u32x4*>(b);
  else *reinterpret_cast<u32x4*>(b) = *reinterpret_cast<const u32x4*>(p);
}
__global__ void embed_copy_kernel(bf16_t* __restrict__ embeds, const int32_t* __restrict__ ids, int n, int H,
                                  bf16_t* __restrict__ buf, int to_pool) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one 16-byte piece
  if (idx >= (int64_t)n * (H / 8)) return;
  embed_copy_piece(embeds, ids[idx / (H / 8)], idx, H, buf, to_pool);
}
template <int N>
__global__ void embed_copy_ids_kernel(bf16_t* __restrict__ embeds, IdArgs<N> ids, int n, int H, bf16_t* __restrict__ buf,
                                      int to_pool) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * (H / 8)) return;
  embed_copy_piece(embeds, ids.v[idx / (H / 8)], idx, H, buf, to_pool);
}

// embed_txt: Embed ids[r] receives row tok[r] of the embedding table, 16 bytes per thread.
__global__ void embed_gather_kernel(bf16_t* __restrict__ embeds, const int32_t* __restrict__ ids,
                                    const int32_t* __restrict__ tok, int n, int H, const bf16_t* __restrict__ table) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int per_row = H / 8;
  if (idx >= (int64_t)n * per_row) return;
  int r = (int)(idx / per_row), c = (int)(idx % per_row) * 8;
  *reinterpret_cast<u32x4*>(embeds + (int64_t)ids[r] * H + c) =
      *reinterpret_cast<const u32x4*>(table + (int64_t)tok[r] * H + c);
}

hipError_t launch_embed_gather(bf16_t* embeds, const int32_t* ids, const int32_t* tok, int n, int H,
                               const bf16_t* table, hipStream_t s) {
  int64_t total = (int64_t)n * (H / 8);
  if (total <= 0) return hipSuccess;
  embed_gather_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(embeds, ids, tok, n, H, table);
  return hipGetLastError();
}

hipError_t launch_embed_copy(bf16_t* embeds, const int32_t* ids, int n, int H, bf16_t* buf, int to_pool,
                             hipStream_t s) {
  int64_t total = (int64_t)n * (H / 8);
  if (total <= 0) return hipSuccess;
  embed_copy_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(embeds, ids, n, H, buf, to_pool);
  return hipGetLastError();
}

hipError_t launch_embed_copy_ids(bf16_t* embeds, const int32_t* host_ids, int n, int H, bf16_t* buf, int to_pool, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n > IDS_BY_VALUE) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((n * (H / 8) + 255) / 256)), block(256);
  if (n <= 64) embed_copy_ids_kernel<64><<<grid, block, 0, s>>>(embeds, id_args<64>(host_ids, n), n, H, buf, to_pool);
  else embed_copy_ids_kernel<IDS_BY_VALUE><<<grid, block, 0, s>>>(embeds, id_args<IDS_BY_VALUE>(host_ids, n), n, H, buf, to_pool);
  return hipGetLastError();
}

__global__ void kv_copy_kernel(bf16_t* __restrict__ kv_layer, const int32_t* __restrict__ pages,
                               const int32_t* __restrict__ slots, int n, int Hkv, int D, bf16_t* __restrict__ k,
                               bf16_t* __restrict__ v, int to_pool) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one (token, head, d) element
  int64_t total = (int64_t)n * Hkv * D;
  if (idx >= total) return;
  int d = (int)(idx % D);
  int h = (int)((idx / D) % Hkv);
  int i = (int)(idx / ((int64_t)D * Hkv));
  uint16_t* blk = reinterpret_cast<uint16_t*>(kv_layer + ((int64_t)pages[i] * Hkv + h) * (2 * PAGE * D));
  uint16_t* kk = reinterpret_cast<uint16_t*>(k);
  uint16_t* vv = reinterpret_cast<uint16_t*>(v);
  int ko = k_elem_offset(slots[i], d), vo = v_elem_offset(slots[i], d, D);
  if (to_pool) {
    blk[ko] = kk[idx];
    blk[vo] = vv[idx];
  } else {
    kk[idx] = blk[ko];
    vv[idx] = blk[vo];
  }
}

hipError_t launch_kv_copy(bf16_t* kv_layer, const int32_t* pages, const int32_t* slots, int n, int Hkv, int D,
                          bf16_t* k, bf16_t* v, int to_pool, hipStream_t s) {
  int64_t total = (int64_t)n * Hkv * D;
  if (total <= 0) return hipSuccess;
  kv_copy_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(kv_layer, pages, slots, n, Hkv, D, k, v,
                                                                               to_pool);
  return hipGetLastError();
}

// copy_kvpage: token k of the call moves from (src page, src slot) to (dst page, dst slot), K and V, in every
// layer's pool (grid.y = layer); one thread per (token, kv head, element).
__global__ void kv_token_copy_kernel(bf16_t* __restrict__ kv, size_t layer_elems, const int32_t* __restrict__ sp,
                                     const int32_t* __restrict__ ss, const int32_t* __restrict__ dp,
                                     const int32_t* __restrict__ ds, int n, int Hkv, int D) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * Hkv * D) return;
  const int d = (int)(idx % D);
  const int h = (int)((idx / D) % Hkv);
  const int i = (int)(idx / ((int64_t)D * Hkv));
  uint16_t* pool = reinterpret_cast<uint16_t*>(kv + (size_t)blockIdx.y * layer_elems);
  const uint16_t* src = pool + ((int64_t)sp[i] * Hkv + h) * (2 * PAGE * D);
  uint16_t* dst = pool + ((int64_t)dp[i] * Hkv + h) * (2 * PAGE * D);
  dst[k_elem_offset(ds[i], d)] = src[k_elem_offset(ss[i], d)];
  dst[v_elem_offset(ds[i], d, D)] = src[v_elem_offset(ss[i], d, D)];
}

hipError_t launch_kv_token_copy(bf16_t* kv, size_t layer_elems, int n_layers, const int32_t* src_pages,
                                const int32_t* src_slots, const int32_t* dst_pages, const int32_t* dst_slots, int n,
                                int Hkv, int D, hipStream_t s) {
  int64_t total = (int64_t)n * Hkv * D;
  if (total <= 0 || n_layers <= 0) return hipSuccess;
  kv_token_copy_kernel<<<dim3((unsigned)((total + 255) / 256), (unsigned)n_layers), dim3(256), 0, s>>>(
      kv, layer_elems, src_pages, src_slots, dst_pages, dst_slots, n, Hkv, D);
  return hipGetLastError();
}
