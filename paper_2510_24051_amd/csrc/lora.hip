// LoRA adapters (forward_with_adapter): per-token low-rank updates  y += scale * B (A x)  of the layer's
// projections.  Tokens carry the adapter of their request (-1: none); the pairs of all adapters live in one
// device table indexed [adapter][layer][projection], A stored [rank_p, in] and B [out, rank_p] with the rank padded
// to a multiple of 16 by zeros.  The batch plan lists the adapted tokens grouped by adapter in tiles of 32 rows
// (row = token index, -1 = padding; one adapter per tile), so both steps are small grouped GEMMs on the matrix
// cores and A, B are read once per 32 tokens:
//   lora_down  z[row, slot, :] = A x            X rows gathered as the MFMA A operand, A's rows as the B operand,
//                                               the contraction split over the workgroup's sixteen waves
//   lora_up    y[token, n]    += scale * B z    z (fp32) enters as a bf16 pair hi + lo, so that its rounding does
//                                               not show; y is the bf16 qkv row, the fp32 residual stream, the
//                                               fp32 gate/up sums in the packed column order of the tiled weight, or
//                                               (qkv, o) the partial sums of a product split along K
// Where the qkv or output product is split along K, the update goes into the partial sums, and the rotary step or the
// second norm sums them as it does without adapters: no epilogue kernel in between (two of 4.4 us less per layer; 40
// tokens on four rank-16 adapters, a whole layer 192 -> 187 us).  For o, an fp32 sum, it is added to the first partial
// copy.  The qkv row is rounded to bf16 before the update and after it, so there the adapted elements are summed here,
// and the first copy takes the result, the others zeros.
// When gate or up carry an adapter the SwiGLU product cannot be fused into the GEMM epilogue; it is taken from the
// fp32 sums by `swiglu_f32`.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace {

constexpr int DOWN_WAVES = 16;  // waves of a lora_down workgroup, one for each accumulator register

__device__ __forceinline__ const LoraPair& pair_of(const LoraPair* table, int ad, int n_layers, int layer, int proj) {
  return table[((int64_t)ad * n_layers + layer) * PIE_N_PROJ + proj];
}

// grid (tiles, slots, rank blocks of 32 x ksplits); z is [ksplits][rows, 3, rmax_p] fp32.  What bounds it is the latency of
// its few loads: x and A rows of a decode batch are a few hundred KB.  So the contraction goes over the sixteen waves of a
// workgroup, and with few tiles also over workgroups (partial sums that lora_up adds while it loads z).  Four waves and
// up to 16 copies were as fast here (4.0 against 4.8 us at 40 tokens and 4096, 7.5 against 6.1 at 128 tokens and rank 64) but
// left every wave of lora_up 16 copies to read: 9.3 and 6.2 us there for qkv and o, 20.1 and 12.3 at rank 64.  With at most
// four copies, and with what the update is added to requested ahead of z, it takes 6.8 and 5.3, 12.5 and 9.2.
// Many tiles gain more, 2048 tokens of four prompts on rank-16 adapters: down 35.6 and 34.8 -> 17.1 and 17.0 us, up (one instance
// of 248 registers before, two of 108 and 152) 77 and 36 -> 23 and 21.
__global__ __launch_bounds__(64 * DOWN_WAVES) void lora_down_kernel(
    const bf16_t* __restrict__ x, int ldx, int in, const int32_t* __restrict__ rows, const int32_t* __restrict__ tile_ad,
    const LoraPair* __restrict__ table, int layer, int n_layers, int proj0, float* __restrict__ z, int rmax_p, int ksplits) {
  __shared__ float red[DOWN_WAVES][16][64];
  const int tile = blockIdx.x, slot = blockIdx.y, rb = blockIdx.z / ksplits, ks = blockIdx.z % ksplits;
  const LoraPair p = pair_of(table, tile_ad[tile], n_layers, layer, proj0 + slot);
  if (p.A == nullptr || rb * 32 >= p.rank_p) return;  // the same for the whole workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 31, g = lane >> 5;
  const int tok = max(rows[tile * 32 + m], 0);  // padding rows read token 0; their sums are never used
  const bf16_t* xr = x + (int64_t)tok * ldx + g * 8;
  const bf16_t* ar = p.A + (int64_t)min(rb * 32 + m, p.rank_p - 1) * in + g * 8;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int steps = in / 16;  // `in` is a multiple of 32
  const int per = (steps + ksplits - 1) / ksplits;
  const int s_end = min(steps, (ks + 1) * per);
#pragma unroll 4
  for (int s = ks * per + wave; s < s_end; s += DOWN_WAVES) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(xr + s * 16);
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(ar + s * 16);
    acc = mfma32(a, b, acc);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
  __syncthreads();
  // wave w finishes accumulator register w: row (w / 4) * 8 + g * 4 + (w % 4) of the tile, column m
  const int j = rb * 32 + m;
  if (j >= p.rank_p) return;
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < DOWN_WAVES; ++w) sum += red[w][wave][lane];
  const int row = (wave >> 2) * 8 + g * 4 + (wave & 3);
  z[(((int64_t)ks * gridDim.x + tile) * 32 + row) * 3 * rmax_p + slot * rmax_p + j] = sum;
}

// grid (tiles, blocks of 128 output columns); a wave owns 32 columns
//   kind 0: dst bf16, column = col0 + n       (q, k or v inside the qkv rows)
//   kind 1: dst fp32, column = col0 + n       (residual stream)
//   kind 2: dst fp32, column = (n / 32) * 64 + n % 32 + col0   (gate: col0 = 0, up: col0 = 32; packed order)
//   kind 3: dst bf16 qkv rows, all three projections in one launch: out = the row length, columns [0, col0) are
//           q (projection proj, slot 0), the next kd columns k (proj + 1, slot 1), the rest v (proj + 2, slot 2)
//   kind 4: dst the partial sums of the qkv product, [copies][copy elements], columns as in kind 3
template <bool PARTS>
__global__ __launch_bounds__(256) void lora_up_kernel(void* __restrict__ dst, int ld, int out, int kind, int col0,
                                                      int kd, const int32_t* __restrict__ rows,
                                                      const int32_t* __restrict__ tile_ad,
                                                      const LoraPair* __restrict__ table, int layer, int n_layers,
                                                      int proj, int slot, const float* __restrict__ z, int rmax_p,
                                                      int ksplits, int copies, int64_t copy_elems) {
  const int tile = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nb = blockIdx.y * 4 + wave;
  if (nb * 32 >= out) return;  // `out` is a multiple of 32; no barrier below
  const int m = lane & 31, g = lane >> 5;
  int n = nb * 32 + m, col_base = col0;
  if (kind >= 3) {  // which of q, k, v this block of 32 columns belongs to (their widths are multiples of 32)
    const int seg = nb * 32 < col0 ? 0 : (nb * 32 < col0 + kd ? 1 : 2);
    col_base = seg == 0 ? 0 : (seg == 1 ? col0 : col0 + kd);
    n -= col_base;
    proj += seg;
    slot = seg;
  }
  const LoraPair p = pair_of(table, tile_ad[tile], n_layers, layer, proj);
  if (p.B == nullptr) return;
  const int col = kind == 2 ? (n >> 5) * 64 + (n & 31) + col0 : col_base + n;
  int tok[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) tok[v] = rows[tile * 32 + (v >> 2) * 8 + g * 4 + (v & 3)];
  // What the update is added to is requested before z and B, on which it does not depend.  A padding row reads its
  // tile's first token, which always is one (no branch between the requests; the value is not used).
  constexpr int FIRST = PARTS ? 4 : 1;  // partial copies that are requested here; later ones follow below
  const int64_t row0 = rows[tile * 32];
  float old[FIRST][16];
  if (kind == 0 || kind == 3) {
    const bf16_t* d = reinterpret_cast<const bf16_t*>(dst) + col;
#pragma unroll
    for (int v = 0; v < 16; ++v) old[0][v] = bf16_to_f32(d[(tok[v] >= 0 ? tok[v] : row0) * ld]);
  } else {
    const float* d = reinterpret_cast<const float*>(dst) + col;
#pragma unroll
    for (int k = 0; k < FIRST; ++k) {
      const float* dk = k == 0 ? d : d + min(k, copies - 1) * copy_elems;
#pragma unroll
      for (int v = 0; v < 16; ++v) old[k][v] = dk[(tok[v] >= 0 ? tok[v] : row0) * ld];
    }
  }
  const float* zr = z + ((int64_t)(tile * 32 + m) * 3 + slot) * rmax_p + g * 8;
  const int64_t zsplit = (int64_t)gridDim.x * 32 * 3 * rmax_p;
  const bf16_t* br = p.B + (int64_t)n * p.rank_p + g * 8;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  for (int s = 0; s < p.rank_p / 16; ++s) {
    f32x4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    const auto add = [&](auto group) {  // partial copies requested together; the sum is in split order in any case
      constexpr int N = decltype(group)::value;
      for (; k + N <= ksplits; k += N) {
        f32x4 pa[N], pb[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
          pa[u] = *reinterpret_cast<const f32x4*>(zr + (k + u) * zsplit + s * 16);
          pb[u] = *reinterpret_cast<const f32x4*>(zr + (k + u) * zsplit + s * 16 + 4);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) { z0 += pa[u]; z1 += pb[u]; }
      }
    };
    add(std::integral_constant<int, 4>());
    add(std::integral_constant<int, 1>());
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(br + s * 16);
    bf16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float f = e < 4 ? z0[e] : z1[e - 4];
      hi[e] = f32_to_bf16(f);
      lo[e] = f32_to_bf16(f - bf16_to_f32(hi[e]));
    }
    acc = mfma32(hi, b, acc);
    acc = mfma32(lo, b, acc);
  }
  if (PARTS) {
    float* d = reinterpret_cast<float*>(dst) + col;
#pragma unroll
    for (int k = 1; k < FIRST; ++k)  // in split order, as the kernels that sum the copies do
#pragma unroll
      for (int v = 0; v < 16; ++v) old[0][v] += k < copies ? old[k][v] : 0.f;
    for (int k = FIRST; k < copies; ++k)
#pragma unroll
      for (int v = 0; v < 16; ++v) old[0][v] += d[k * copy_elems + (tok[v] >= 0 ? tok[v] : row0) * ld];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if (tok[v] < 0) continue;
      d[(int64_t)tok[v] * ld] = bf16_to_f32(f32_to_bf16(bf16_to_f32(f32_to_bf16(old[0][v])) + acc[v] * p.scale));
      for (int k = 1; k < copies; ++k) d[k * copy_elems + (int64_t)tok[v] * ld] = 0.f;
    }
  } else if (kind == 0 || kind == 3) {
    bf16_t* d = reinterpret_cast<bf16_t*>(dst) + col;
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (tok[v] >= 0) d[(int64_t)tok[v] * ld] = f32_to_bf16(old[0][v] + acc[v] * p.scale);
  } else {
    float* d = reinterpret_cast<float*>(dst) + col;
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (tok[v] >= 0) d[(int64_t)tok[v] * ld] = old[0][v] + acc[v] * p.scale;
  }
}

// act[t, i] = silu(gate) * up from fp32 sums in the packed column order (gate block, up block alternating)
__global__ __launch_bounds__(256) void swiglu_f32_kernel(const float* __restrict__ gu, int I, bf16_t* __restrict__ act,
                                                         int64_t total) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int i = (int)(idx % I);
  const int64_t t = idx / I;
  const float* row = gu + t * 2 * I;
  const int c = (i >> 5) * 64 + (i & 31);
  const float g = row[c], u = row[c + 32];
  act[idx] = f32_to_bf16(silu_f(g) * u);
}

}  // namespace

int lora_ksplits(int n_tiles, int n_slots, int in, int rmax_p, size_t z_rows) {
  // enough workgroups to cover half the chip, at least 4 contraction steps per wave, and room for the partial copies
  const int wgs = n_tiles * n_slots * ((rmax_p + 31) / 32);
  int ks = std::max(1, 256 / std::max(1, wgs));
  ks = std::min(ks, std::max(1, in / 16 / (4 * DOWN_WAVES)));
  ks = std::min<int>(ks, (int)std::max<size_t>(1, z_rows / ((size_t)n_tiles * 32)));
  return std::min(ks, 4);
}

hipError_t launch_lora_down(const bf16_t* x, int ldx, int in, int n_tiles, int n_slots, const int32_t* rows,
                            const int32_t* tile_ad, const LoraPair* table, int layer, int n_layers, int proj0, float* z,
                            int rmax_p, int ksplits, hipStream_t s) {
  if (n_tiles <= 0 || n_slots <= 0) return hipSuccess;
  if (n_slots > 3 || in % 32 != 0 || rmax_p % 16 != 0 || ksplits < 1) return hipErrorInvalidValue;
  lora_down_kernel<<<dim3(n_tiles, n_slots, ((rmax_p + 31) / 32) * ksplits), dim3(64 * DOWN_WAVES), 0, s>>>(
      x, ldx, in, rows, tile_ad, table, layer, n_layers, proj0, z, rmax_p, ksplits);
  return hipGetLastError();
}

hipError_t launch_lora_up(void* dst, int ld, int out, int kind, int col0, int kd, int n_tiles, const int32_t* rows,
                          const int32_t* tile_ad, const LoraPair* table, int layer, int n_layers, int proj, int slot,
                          const float* z, int rmax_p, int ksplits, hipStream_t s, int copies, int64_t copy_elems) {
  if (n_tiles <= 0 || out <= 0) return hipSuccess;
  if (out % 32 != 0 || slot < 0 || slot > 2 || ksplits < 1) return hipErrorInvalidValue;
  if (kind == 4 && copies < 1) return hipErrorInvalidValue;
  if (kind >= 3 && (col0 % 32 != 0 || kd % 32 != 0 || col0 + 2 * kd != out)) return hipErrorInvalidValue;
  const auto kernel = kind == 4 ? lora_up_kernel<true> : lora_up_kernel<false>;
  kernel<<<dim3(n_tiles, (out + 127) / 128), dim3(256), 0, s>>>(dst, ld, out, kind, col0, kd, rows, tile_ad, table,
                                                                       layer, n_layers, proj, slot, z, rmax_p, ksplits, copies, copy_elems);
  return hipGetLastError();
}

hipError_t launch_swiglu_f32(const float* gu, int I, bf16_t* act, int T, hipStream_t s) {
  const int64_t total = (int64_t)T * I;
  if (total <= 0) return hipSuccess;
  swiglu_f32_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s>>>(gu, I, act, total);
  return hipGetLastError();
}
