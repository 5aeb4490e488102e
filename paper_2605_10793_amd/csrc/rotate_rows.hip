// Y = X R_op for a few rows (token-by-token use): up to 32, per head, both activation dtypes.
//
// With so few rows the product is bound by reading the rotation once (32 MiB at d = 4096) and
// by latency, not by the matrix cores.  The tiled GEMM gives it one row of 64 x 64 tiles (64
// workgroups at d = 4096), each a serial chain of 64 K steps.  Here a workgroup owns 16 NT
// output columns (256 workgroups at d = 4096) and its 8 wavefronts share out K; operands go
// straight from memory to MFMA fragments (nothing is read twice by a workgroup, so LDS would
// only add a stage), four K chunks of every operand in flight per wavefront, and the partial
// sums meet in LDS in a fixed order.  16 x 4096 x 4096, bf16: 19.7 us with the tiled GEMM, 9.3
// here (one row 7.2: 4.7 TB/s).
//
// The statistics step of a few rows takes its corner signs from the same sums, so that a batch
// is rotated once whatever is asked of it, and with bf16 activations the same launch writes the
// accumulate GEMM's scaled transposed operand: 64 tokens of a column are 128 bytes of either
// array, put together in LDS from one value per thread.
#include "kernels.h"

namespace conqur {

namespace {

constexpr int NWAVES = 8;
constexpr int U = 4;         // K chunks of 32 per round: 256 contiguous bytes of a bf16 row

template <bool F32, bool STATS, int MT, int NT>
__global__ void __launch_bounds__(64 * NWAVES) k_rotate_rows(const void* __restrict__ X, int T, int64_t stride,
                                                             const bf16_bits* __restrict__ RopT, int64_t plane, int dh,
                                                             void* __restrict__ Y, int64_t ldy, const RotateRowsStats st) {
  constexpr int NP = F32 ? 3 : 1;    // planes of the rotate operand
  __shared__ float red[NWAVES][MT * NT * 4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, kg = lane >> 4;      // fragments: row (column of the product) col, K elements 8 kg .. 8 kg + 7 of 32
  const int n0 = blockIdx.x * 16 * NT, h = blockIdx.y;
  const int64_t hcol = (int64_t)h * dh;
  const bf16_bits* R = RopT + hcol * dh;
  const int nch = (dh + 31) / 32;

  f32x4 acc[MT][NT], low[F32 ? MT : 1][F32 ? NT : 1];   // fp32: the products of lower planes are summed on their own
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if constexpr (F32) low[i][j] = acc[i][j];
    }

  for (int g = wave; g * U < nch; g += NWAVES) {
    uint4 a[U][MT][F32 ? 2 : 1], b[U][NT][NP];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (g * U + u) * 32 + kg * 8;
      const bool k_in = k < dh;                          // dh is a multiple of 16: 8 elements are inside or outside together
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int n = n0 + 16 * j + col;
#pragma unroll
        for (int p = 0; p < NP; ++p)
          b[u][j][p] = (k_in && n < dh) ? *reinterpret_cast<const uint4*>(R + p * plane + (int64_t)n * dh + k) : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int t = 16 * i + col;
        const bool in = k_in && t < T;
        if constexpr (F32) {
          const float* x = reinterpret_cast<const float*>(X) + t * stride + hcol + k;
          a[u][i][0] = in ? *reinterpret_cast<const uint4*>(x) : make_uint4(0u, 0u, 0u, 0u);
          a[u][i][1] = in ? *reinterpret_cast<const uint4*>(x + 4) : make_uint4(0u, 0u, 0u, 0u);
        } else {
          a[u][i][0] = in ? *reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_bits*>(X) + t * stride + hcol + k)
                          : make_uint4(0u, 0u, 0u, 0u);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if constexpr (F32) {
          // the exact three-way bf16 split of the row's values, and all products down to 2^-24 (smallest first)
          float f[8] = {__uint_as_float(a[u][i][0].x), __uint_as_float(a[u][i][0].y), __uint_as_float(a[u][i][0].z), __uint_as_float(a[u][i][0].w),
                        __uint_as_float(a[u][i][1].x), __uint_as_float(a[u][i][1].y), __uint_as_float(a[u][i][1].z), __uint_as_float(a[u][i][1].w)};
          bf16x8 s[3];
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            uint4 t;
            uint32_t* tw = reinterpret_cast<uint32_t*>(&t);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              tw[e] = f32x2_to_bf16x2(f[2 * e], f[2 * e + 1]);
              f[2 * e] -= __uint_as_float(tw[e] << 16);
              f[2 * e + 1] -= __uint_as_float(tw[e] & 0xffff0000u);
            }
            s[p] = __builtin_bit_cast(bf16x8, t);
          }
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            bf16x8 r[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) r[p] = __builtin_bit_cast(bf16x8, b[u][j][p < NP ? p : 0]);
            low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s[2], r[0], low[i][j], 0, 0, 0);
            low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s[1], r[1], low[i][j], 0, 0, 0);
            low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s[0], r[2], low[i][j], 0, 0, 0);
            low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s[1], r[0], low[i][j], 0, 0, 0);
            low[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s[0], r[1], low[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s[0], r[0], acc[i][j], 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u][i][0]), __builtin_bit_cast(bf16x8, b[u][j][0]),
                                                                acc[i][j], 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(i * NT + j) * 4 + r][lane] = F32 ? acc[i][j][r] + low[F32 ? i : 0][F32 ? j : 0][r] : acc[i][j][r];
  __syncthreads();
  constexpr int PT = kRotateRowsTokens + 8;   // a column's 64 tokens, padded by 16 bytes: 16 columns spread over the banks
  __shared__ __attribute__((aligned(16))) bf16_bits tile[STATS ? 16 * NT : 1][PT];   // corner signs, then the scaled operand
  constexpr uint32_t one = F32 ? 0x3F80u : 0x3C00u;   // the accumulate GEMM takes bf16 planes for fp32 activations, else fp16
  if constexpr (STATS) {   // tokens past the batch: +1, as the sign of a sum of no terms
    for (int o = tid; o < 16 * NT * (PT / 2); o += 64 * NWAVES) reinterpret_cast<uint32_t*>(&tile[0][0])[o] = one | one << 16;
    __syncthreads();
  }
  // value (i, j, r) of lane l is row 16 i + 4 (l / 16) + r, column 16 j + l % 16
  for (int o = tid; o < MT * NT * 256; o += 64 * NWAVES) {
    const int q = o >> 6, l = o & 63;
    float y = 0.0f;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) y += red[w][q][l];
    const int t = 16 * (q / (NT * 4)) + 4 * (l >> 4) + (q & 3), n = n0 + 16 * ((q >> 2) % NT) + (l & 15);
    if (t < T && n < dh) {
      if constexpr (STATS) tile[n - n0][t] = (bf16_bits)(y >= 0.0f ? one : one | 0x8000u);   // sgn(+-0) = +1
      if (!STATS || Y) {
        if constexpr (F32) reinterpret_cast<float*>(Y)[t * ldy + hcol + n] = y;
        else reinterpret_cast<bf16_bits*>(Y)[t * ldy + hcol + n] = f32_to_bf16(y);
      }
    }
  }
  if constexpr (STATS) {
    // rows of either array: 8 threads store the 128 bytes of a column's 64 tokens
    auto store_tile = [&](bf16_bits* base) {
      __syncthreads();
      for (int o = tid; o < 16 * NT * 8; o += 64 * NWAVES) {
        const int c = o >> 3, n = n0 + c;
        if (n < dh) *reinterpret_cast<uint4*>(base + (hcol + n) * st.pitch + (o & 7) * 8) = *reinterpret_cast<const uint4*>(&tile[c][(o & 7) * 8]);
      }
    };
    store_tile(st.St);
    if constexpr (!F32) {
      __syncthreads();
      for (int o = tid; o < 16 * NT * kRotateRowsTokens; o += 64 * NWAVES) {
        const int c = o % (16 * NT), t = o / (16 * NT), n = n0 + c;
        const bool in = t < T && n < dh;
        const float w = in ? st.w[(int64_t)h * st.ldw + t] : 0.0f;
        // a skipped row has w = 0 and possibly Inf / NaN values: select, do not multiply
        const float x = w != 0.0f ? bf16_to_f32(reinterpret_cast<const bf16_bits*>(X)[t * stride + hcol + n]) * w : 0.0f;
        tile[c][t] = f32_to_f16(x);
      }
      store_tile(st.Xt);
      if (n0 == 0 && wave == 0) {   // the head's rows that entered M (w != 0) and those skipped
        const bool in = lane < T;
        const float w = in ? st.w[(int64_t)h * st.ldw + lane] : 0.0f;
        const unsigned long long entered = __ballot(in && w != 0.0f), skipped = __ballot(in && w == 0.0f);
        if (lane == 0) {
          unsigned long long* slot = st.cnt + (int64_t)h * st.cnt_slots * 2;
          if (entered) atomicAdd(slot, (unsigned long long)__popcll(entered));
          if (skipped) atomicAdd(slot + 1, (unsigned long long)__popcll(skipped));
        }
      }
    }
  }
}

template <bool F32, bool STATS>
hipError_t launch(const void* X, int T, int64_t stride, const bf16_bits* RopT, int64_t plane, int heads, int dh, void* Y, int64_t ldy,
                  const RotateRowsStats& st, hipStream_t s) {
  const dim3 grid((dh + 15) / 16, heads), block(64 * NWAVES);
  if (T <= 16) hipLaunchKernelGGL((k_rotate_rows<F32, STATS, 1, 1>), grid, block, 0, s, X, T, stride, RopT, plane, dh, Y, ldy, st);
  else hipLaunchKernelGGL((k_rotate_rows<F32, STATS, 2, 1>), grid, block, 0, s, X, T, stride, RopT, plane, dh, Y, ldy, st);
  return hipGetLastError();
}

}  // namespace

// Every workgroup reads all of X: more rows cost more than they bring.  Measured against the tiled GEMM (us): bf16, d = 4096,
// 16 rows 9.3 against 19.7, 32 rows 13.2 against 19.8, 64 rows 24.6 against 19.9; d = 8192, 16 rows 33.3 against 35.6, 32 rows
// 45.5 against 35.6; fp32, d = 4096 (three planes of the operand, six products) 32 rows 32 against 102.
bool rotate_rows_fits(int x_is_f32, int64_t T, int dh) { return T <= 16 || (T <= 32 && (x_is_f32 || dh <= 4096)); }

hipError_t launch_rotate_rows(const void* X, int x_is_f32, int64_t T, int64_t stride, const bf16_bits* RopT, int64_t plane, int heads,
                              int dh, void* Y, int64_t ldy, const RotateRowsStats* stats, hipStream_t s) {
  if (T < 1 || !rotate_rows_fits(x_is_f32, T, dh) || heads < 1 || heads > 65535 || dh < 16 || (dh & 15)) return hipErrorInvalidValue;
  if (!stats) {
    if (!Y) return hipErrorInvalidValue;
    return x_is_f32 ? launch<true, false>(X, (int)T, stride, RopT, plane, heads, dh, Y, ldy, RotateRowsStats{}, s)
                    : launch<false, false>(X, (int)T, stride, RopT, plane, heads, dh, Y, ldy, RotateRowsStats{}, s);
  }
  if (!stats->St || stats->pitch < kRotateRowsTokens || (stats->pitch & 7) || (!x_is_f32 && (!stats->Xt || !stats->w || !stats->cnt || stats->cnt_slots < 1)))
    return hipErrorInvalidValue;
  return x_is_f32 ? launch<true, true>(X, (int)T, stride, RopT, plane, heads, dh, Y, ldy, *stats, s)
                  : launch<false, true>(X, (int)T, stride, RopT, plane, heads, dh, Y, ldy, *stats, s);
}

}  // namespace conqur
