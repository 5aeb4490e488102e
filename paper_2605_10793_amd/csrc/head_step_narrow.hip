// Statistics step of the per-head rotations of several heads of width 16 .. 112 with bf16 activations, one launch: norms, Y = X R,
// corner signs and M_h += x^^T C (Sec. 3.3-3.4, per-head blocks as for the value / output projections of Alg. 1).
//
// M's rounding is part of the result (where nothing holds M's weak directions a last bit of it comes back as 1e-2 of a later
// rotation), and the general path adds every entry up in one chain of MFMAs over all tokens.  So does this kernel: a workgroup
// owns one tile column of one head's M (and one block of 32 channels, or all), and goes through all tokens, 256 at a time:
//   operands   Every wavefront takes 32 tokens, in registers.  Rows come by 16-byte loads straight into the MFMA A layout (lane: row
//              `col`, channels 8 kg .. + 7), 256 tokens ahead.  Norms: over a lane's chunks and the four lane groups of a row, in the order
//              of k_row_norms_narrow.  Y: this tile column's products, K ascending as in every product with R, so that the signs
//              are those of the rotated rows.  Two row tiles' signs, turned by lane swaps, are an operand whose K runs over the tokens;
//              the scaled rows (fp16) times an identity leave accumulators that hold them, exactly, in Y's layout, turned the same way.
//   M          The operands of the 256 tokens meet in LDS (two buffers, one barrier), and one wavefront per tile of M takes them in order.
// What bounds it: the arithmetic of the operands (some 330 VALU instructions per 32 tokens), half of which, the norms, every
// workgroup of a head repeats, in series over the tokens: 256 tokens take 0.8 us at width 16 and 2.2 to 2.9 at 112, whatever the number of
// heads up to a round of workgroups.  Statistics step, us, as norms, rotation with signs and operand,
// and accumulation in a launch each, and so: 32 heads of width 64, 2048 tokens 29.2 and 16.6; 24 of 64, 700 tokens 16.3 and 8.5; 32 of 16, 2048
// 22.5 and 10.2; 16 of 48, 3000 27.9 and 19.5; 32 of 96, 2048 30.9 and 24.1; 8 of 112, 2500 27.8 and 26.3.  Where the three launches are the
// faster ones (long batches of few heads 48 wide and more, a second round of workgroups) they stay: head_step_narrow_pays.  Not faster: 16
// wavefronts, rows fetched 512 tokens ahead (17.5 .. 19.2 for the first), wavefronts of their own for M (18.1).
#include "kernels.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace conqur {

namespace {

constexpr int NW = 8;                  // wavefronts of a workgroup
constexpr int kBlock = 32;             // tokens of a wavefront at a time
constexpr int kSuper = NW * kBlock;    // ... of a workgroup

// SPLIT: the workgroup has the two channel tiles of K block blockIdx.y, not all.
template <int DH, bool SPLIT>
__global__ void __launch_bounds__(64 * NW) k_head_step_narrow(const HeadStepNarrow g, const float out_scale) {
  constexpr int KB = (DH + 31) / 32, NT = DH / 16, CH = DH / 8;   // K blocks of a row, 16-wide tiles, 16-byte chunks
  constexpr int KA = SPLIT ? 1 : KB, NA = SPLIT ? (NT < 2 ? NT : 2) : NT;   // K blocks and tiles of the workgroup's channels
  static_assert(NA <= NW, "a wavefront per tile");
  __shared__ __attribute__((aligned(16))) f16x8 ops[2][NW][NA + 1][64];   // x^^T tiles, then the corners
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = lane >> 4, col = lane & 15;
  // the workgroups of a head follow one another on one XCD, whose L2 then fetches the head's rows once
  const int h = (blockIdx.x & 7) + 8 * ((blockIdx.x >> 3) / NT), tile = (blockIdx.x >> 3) % NT;
  const int part = SPLIT ? blockIdx.y : 0;
  if (h >= g.heads) return;
  const int T = (int)g.T;
  const bool reports = tile == 0 && part == 0;   // norms and row counts, once per head

  // Rows t0 + 16 i + col, chunks kg + 4 kk.  Rows past the end and chunks past the head lie past the range and read zero.
  constexpr uint32_t kOob = 0x80000000u;
  const uint32_t row_bytes = 2u * (uint32_t)g.stride;
  const auto rX = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_bits*>(g.X + (int64_t)h * DH), 0, (int)((uint32_t)(T - 1) * row_bytes + 2u * DH), 0x00020000);
  const uint32_t lane_off = (uint32_t)col * row_bytes + 16u * kg;
  auto fetch = [&](int t0, uint4 (&v)[2][KB]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t off = lane_off + (uint32_t)(t0 + 16 * i) * row_bytes;
#pragma unroll
      for (int kk = 0; kk < KB; ++kk)
        v[i][kk] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rX, CH % 4 == 0 || kk + 1 < KB || kg < CH % 4 ? off + 64u * kk : kOob, 0, 0));
    }
  };
  // Packed 16-bit values of two accumulator tiles of one column, rows 4 kg .. + 3 of each: lane group kg gets rows 8 kg .. + 7 of the 32.
  auto to_operand = [](const uint2& u0, const uint2& u1) {
    const auto a = __builtin_amdgcn_permlane32_swap(u0.x, u1.x, false, false), b = __builtin_amdgcn_permlane32_swap(u0.y, u1.y, false, false);
    const auto x = __builtin_amdgcn_permlane16_swap(a[0], a[1], false, false), y = __builtin_amdgcn_permlane16_swap(b[0], b[1], false, false);
    return make_uint4(x[0], y[0], x[1], y[1]);
  };

  uint4 next[2][KB];
  fetch(wave * kBlock, next);
  // R_h^T: row (output column) 16 tile + col, K elements 32 kk + 8 kg .. + 7
  bf16x8 rot[KB];
#pragma unroll
  for (int kk = 0; kk < KB; ++kk) {
    const bool in = 4 * kk + kg < CH;
    const uint4 v = *reinterpret_cast<const uint4*>(g.RopT + ((int64_t)h * DH + 16 * tile + col) * DH + 8 * (in ? 4 * kk + kg : 0));
    rot[kk] = __builtin_bit_cast(bf16x8, make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u));
  }
  // columns 16 p + col of a 32-wide identity, K elements 8 kg .. + 7
  f16x8 eye[2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int e = 0; e < 8; ++e) eye[p][e] = 8 * kg + e == 16 * p + col ? (_Float16)1.0f : (_Float16)0.0f;
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 acc = zero;                    // wavefront a: channels 16 a .. of the workgroup's, columns 16 tile ..
  unsigned entered = 0, skipped = 0;   // (uniform over the wavefront)

  const auto rS = __builtin_amdgcn_make_buffer_rsrc(g.St + (int64_t)h * DH * g.pitch, 0, (int)(2u * DH * (uint32_t)g.pitch), 0x00020000);
  const uint32_t sign_off = 2u * ((uint32_t)(16 * tile + col) * (uint32_t)g.pitch + 8u * kg);
  // the value of element e of a 16-byte chunk
  auto value = [](const uint4& v, int e) {
    const uint32_t u = e < 2 ? v.x : (e < 4 ? v.y : (e < 6 ? v.z : v.w));
    return __uint_as_float((e & 1) ? u & 0xffff0000u : u << 16);
  };
  auto tokens = [&](int s0, auto parity) {
    constexpr int buf = decltype(parity)::value;
    const int t0 = s0 + wave * kBlock;
    if (t0 < T) {
      uint4 x[2][KB];
      float s[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float ss[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
          x[i][kk] = next[i][kk];
#pragma unroll
          for (int e = 0; e < 8; ++e) ss[kk] += value(x[i][kk], e) * value(x[i][kk], e);
        }
        // chunk c meets c ^ 8, c ^ 4 (another K block), c ^ 2, c ^ 1 (another lane group)
        const uint32_t u = __float_as_uint((ss[0] + ss[2]) + (ss[1] + ss[3]));
        const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        const uint32_t v = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
        const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        s[i] = __uint_as_float(b[0]) + __uint_as_float(b[1]);
      }
      if (t0 + kSuper < T) fetch(t0 + kSuper, next);
      // The root and the quotient of both row tiles at once: odd lane groups have the second one's.
      const float mine = kg & 1 ? s[1] : s[0];
      const bool used = mine > 0.0f && mine < __builtin_inff();
      const float n = used ? sqrtf(mine) : 0.0f, wn = used ? kXhatScale / n : 0.0f;
      const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(wn), __float_as_uint(wn), false, false);   // of either row tile
      const bool all_used = __all(used);
      if (reports) {
        const int t = t0 + 16 * (kg & 1) + col;
        const bool one = t < T && kg < 2;
        if (one) {
          g.nrm[(int64_t)h * g.ldn + t] = n;
          if (!used && !isfinite(mine)) atomicOr(g.nonfinite, 1);
        }
        entered += __popcll(__ballot(one && used));
        skipped += __popcll(__ballot(one && !used));
      }
      f16x8 xs[2][KA];
      auto scale = [&](int i, const uint4& v, f16x8& out) {
        const float wi = __uint_as_float(w[i]);
        uint32_t u[4];
        if (all_used) {
#pragma unroll
          for (int e = 0; e < 4; ++e) u[e] = f32x2_to_f16x2(value(v, 2 * e) * wi, value(v, 2 * e + 1) * wi);
        } else {   // a skipped row has w = 0 and possibly Inf / NaN values: select, do not multiply
#pragma unroll
          for (int e = 0; e < 4; ++e) u[e] = f32x2_to_f16x2(wi != 0.0f ? value(v, 2 * e) * wi : 0.0f, wi != 0.0f ? value(v, 2 * e + 1) * wi : 0.0f);
        }
        out = __builtin_bit_cast(f16x8, make_uint4(u[0], u[1], u[2], u[3]));
      };
#pragma unroll
      for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int kk = 0; kk < KB; ++kk)
          if (!SPLIT || kk == part) scale(i, x[i][kk], xs[i][SPLIT ? 0 : kk]);
      }
      uint2 sign[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f32x4 y = zero;
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[i][kk]), rot[kk], y, 0, 0, 0);
        // +-1 with the sign bits of Y + 0 (sgn(-0) = +1), two to a register
        uint32_t sg[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) sg[r] = __float_as_uint(y[r] + 0.0f);
        sign[i].x = (__builtin_amdgcn_perm(sg[1], sg[0], 0x07060302u) & 0x80008000u) | 0x3C003C00u;
        sign[i].y = (__builtin_amdgcn_perm(sg[3], sg[2], 0x07060302u) & 0x80008000u) | 0x3C003C00u;
      }
      const uint4 c = to_operand(sign[0], sign[1]);
      ops[buf][wave][NA][lane] = __builtin_bit_cast(f16x8, c);
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      // (the rows of St are padded to whole blocks of 32)
      if (part == 0) __builtin_amdgcn_raw_buffer_store_b128(u32x4{c.x, c.y, c.z, c.w}, rS, sign_off + 2u * (uint32_t)t0, 0, 0);
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        uint2 v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4 u = __builtin_amdgcn_mfma_f32_16x16x32_f16(xs[i][SPLIT ? 0 : a / 2], eye[a & 1], zero, 0, 0, 0);
          v[i] = make_uint2(f32x2_to_f16x2(u[0], u[1]), f32x2_to_f16x2(u[2], u[3]));
        }
        ops[buf][wave][a][lane] = __builtin_bit_cast(f16x8, to_operand(v[0], v[1]));
      }
    }
    else {   // (a product of zeros: M's waves take all blocks alike)
      const f16x8 none = __builtin_bit_cast(f16x8, make_uint4(0u, 0u, 0u, 0u));
#pragma unroll
      for (int a = 0; a <= NA; ++a) ops[buf][wave][a][lane] = none;
    }
    __syncthreads();   // (the buffer written next was read before this one was full)
    if (wave < NA) {
      f16x8 xt[NW], c[NW];
#pragma unroll
      for (int q = 0; q < NW; ++q) { xt[q] = ops[buf][q][wave][lane]; c[q] = ops[buf][q][NA][lane]; }
#pragma unroll
      for (int q = 0; q < NW; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(xt[q], c[q], acc, 0, 0, 0);
    }
  };
  for (int s0 = 0; s0 < T; s0 += 2 * kSuper) {
    tokens(s0, std::integral_constant<int, 0>{});
    if (s0 + kSuper < T) tokens(s0 + kSuper, std::integral_constant<int, 1>{});
  }

  const int a = SPLIT ? 2 * part + wave : wave;
  if (wave < NA && a < NT) {
#pragma clang fp contract(off)   // the scaled product is rounded before the sum, as in the accumulate GEMM
    float* const m = g.M + ((int64_t)h * DH + 16 * a + 4 * kg) * DH + 16 * tile + col;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float v = out_scale * acc[r];
      if (g.accumulate) v = v + m[r * DH];
      m[r * DH] = v;
    }
  }
  if (reports && lane == 0) {
    unsigned long long* const slot = g.cnt + ((int64_t)h * g.cnt_slots + wave % g.cnt_slots) * 2;
    if (entered) atomicAdd(slot, (unsigned long long)entered);
    if (skipped) atomicAdd(slot + 1, (unsigned long long)skipped);
  }
}

// By channel blocks where that still gives every workgroup a compute unit of its own: 32 heads of width 64, 2048 tokens 16.6 us (18.0
// without), 8 of 112, 2500 tokens 26.3 (32.4); but 32 of 80, 2000 tokens, 480 workgroups 32.4 (22.8), 16 of 96, 400 tokens 11.7 (8.9).
bool by_channel_blocks(int dh, int heads) {
  const int kb = (dh + 31) / 32;
  return kb > 1 && heads * (dh / 16) * kb <= 256;
}

template <int DH>
hipError_t launch_one(const HeadStepNarrow& a, hipStream_t s) {
  constexpr int KB = (DH + 31) / 32, NT = DH / 16;
  const float out_scale = 1.0f / (kXhatScale * std::sqrt((float)DH));
  const dim3 grid(8 * NT * ((a.heads + 7) / 8));
  if constexpr (KB > 1) {
    if (by_channel_blocks(DH, a.heads)) {
      hipLaunchKernelGGL((k_head_step_narrow<DH, true>), dim3(grid.x, KB), dim3(64 * NW), 0, s, a, out_scale);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_head_step_narrow<DH, false>), grid, dim3(64 * NW), 0, s, a, out_scale);
  return hipGetLastError();
}

}  // namespace

// The expected times of this launch and of the general path's three, us.  Here: a fixed 3 and `per_block` for every 256 tokens, as many
// times over as the workgroups, of which a compute unit holds what its LDS does, are rounds.  There: 12 for the launches, the
// accumulate GEMM's chain over the tokens and the passes over the elements.  Fitted to 1140 steps, 2 to 256 heads, 33 to 65536
// tokens, both ways each: the way taken is 0.2 % slower than the faster one on average, at worst 1.18 times, and slower than the three
// launches by more than 2 % in 8 (1.09 at worst; without the rule in 154, 1.96 at worst).  One launch and three, us: 32 heads of
// width 64, 2048 tokens 16 and 27; 2 of 112, 1024 tokens 12 and 16, 4096 35 and 27, 65536 500 and 265; 16 of 96, 2048 23 and 27, 8192 77 and
// 66; 40 of 112, 512 17 and 19, 2048 52 and 42.  Heads up to 32 wide are faster in one launch throughout.
bool head_step_narrow_pays(int dh, int heads, int64_t T) {
  if (heads < 2 || dh < 16 || (dh & 15) || dh > kHeadStepNarrowMaxDh) return false;
  static constexpr double kWhole[] = {0.85, 0.95, 1.45, 1.7, 2.2, 2.3, 2.9}, kSplit[] = {0.85, 0.95, 1.3, 1.4, 1.7, 1.75, 2.2};
  const bool split = by_channel_blocks(dh, heads);
  const int nt = dh / 16, tiles = split ? 2 : nt;
  const int64_t workgroups = (int64_t)heads * nt * (split ? (dh + 31) / 32 : 1);
  const bool share = 160 / (2 * NW * (tiles + 1)) > 1;   // of 160 KiB of LDS (nt == 1 is never split)
  const double rounds = share ? std::max(1.0, (double)workgroups / 256) : (double)((workgroups + 255) / 256);
  const double per_block = (split ? kSplit : kWhole)[nt - 1];
  const double one = rounds * (3.0 + per_block * (double)T / 256);
  const double three = 12.0 + 0.9 * (double)T / 256 + 2.4e-6 * (double)T * dh * heads;
  return one < three;
}

// For tests (host code only).
extern "C" __attribute__((visibility("default"))) int conqur_head_step_narrow_for_tests(int dh, int heads, int64_t T) {
  return head_step_narrow_pays(dh, heads, T);
}

hipError_t launch_head_step_narrow(const HeadStepNarrow& a, int dh, hipStream_t s) {
  if (a.heads < 1 || a.T < 1 || a.cnt_slots < 1 || a.pitch < round_up(a.T, kBlock) || (a.pitch & 7)) return hipErrorInvalidValue;
  switch (dh) {
    case 16: return launch_one<16>(a, s);
    case 32: return launch_one<32>(a, s);
    case 48: return launch_one<48>(a, s);
    case 64: return launch_one<64>(a, s);
    case 80: return launch_one<80>(a, s);
    case 96: return launch_one<96>(a, s);
    case 112: return launch_one<112>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace conqur
