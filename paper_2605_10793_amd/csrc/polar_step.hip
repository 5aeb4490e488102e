// One step of the polar iteration's main phase, X <- X (a I + b X^T X) (Sec. 3.3), in one launch: heads of width
// kHeadPolarMaxDh + 16 .. kPolarStepMaxDh.
//
// Up to 128 the iterate and the products of a whole update fit one compute unit (head_polar.hip); here a step's products take
// one 5 us and more, so a head is spread over workgroups.  Column block p of the step needs, besides X, only columns p of
// W = a I + b G: a workgroup forms G[:, p] = X^T X[:, p], turns it into W[:, p] and takes X'[:, p] = X W[:, p].  Nothing passes
// between workgroups within a step, so Gram matrix and apply are one launch instead of two, W never leaves the compute unit, and
// one layout of the iterate, X^T, is all that is stored between steps: LDS holds all of it, read as rows (the Gram product) and
// by transposing reads (the apply).  Beyond kPolarStepMaxDh it does not fit and would be fetched twice.
//
// What bounds it: launch, one fetch of X^T (up to 128 KiB per workgroup, from memory: the step before wrote it on other XCDs)
// and a short chain of MFMAs behind it.  So a workgroup fetches the rows its columns are first, and every wavefront then takes the rows
// of G that it has fetched itself, as they land; all of a product's LDS reads are in flight before its MFMAs.  16 columns per
// workgroup while that gives at most one workgroup per compute unit, else 32.  A whole update by events, 23 iterations, us, with two
// launches a step; with one that waited for all of X^T and had 4 wavefronts; and so, with 8 (squares of 192: 12): one head of 256
// 276, 166 .. 173, 141 .. 145; 32 of 256 434, 211, 191; 24 of 208 422, 185, 166; 3 of 192 - , 139, 120; 8 of 176 - , 133, 117.
// (In 4, 6 wavefronts a square of 192 took 132 and 129 in the fourth case; 16 for 256 are no faster than 8.)
//
// Roundings are those of the two GEMM launches it stands for (K in ascending blocks of 32, W and X' once to fp16), bit for bit.
#include "gemm_nt.h"
#include "kernels.h"

#include <type_traits>

namespace conqur {

namespace {

constexpr int kRowB = 512;   // bytes of an LDS row, whatever the width: the rows' bank pattern is head_polar.hip's

// s_waitcnt's operand for vmcnt(n) only
constexpr int vmcnt(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// N: width of the square the head is taken as (zero beyond the head); P: columns of a workgroup; kNW: its wavefronts.
template <int N, int P, int kNW>
__global__ void __launch_bounds__(64 * kNW) k_polar_step(const bf16_bits* __restrict__ Xt, const int dh, const int panels, const float ci,
                                                           const float cg, bf16_bits* __restrict__ Xt_out, const int last,
                                                           float* __restrict__ X32, bf16_bits* __restrict__ Pn) {
  static_assert(N % (16 * kNW) == 0 && N <= kPolarStepMaxDh && P % 16 == 0, "whole row tiles per wavefront");
  constexpr int TM = N / (16 * kNW), TN = P / 16, KB = N / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* const sX = smem;                  // X^T: row c, K = row of X
  unsigned char* const sW = smem + N * kRowB;      // columns p of W: row = column, K = row of W; before that, rows p of X^T
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 4, col = lane & 15;
  // a head's workgroups on one XCD (bid % 8), where its L2 fetches X^T once
  const int total = gridDim.x, xcd = blockIdx.x & 7, rest = total & 7;
  const int at = xcd * (total >> 3) + (xcd < rest ? xcd : rest) + (blockIdx.x >> 3);
  const int h = at / panels, n0 = (at % panels) * P;
  const int64_t hoff = (int64_t)h * dh * dh;
  constexpr uint32_t kOob = 0x80000000u;           // an offset past every descriptor's range: loads give zero, stores nothing
  auto rsrc = [&](const void* p, int elem) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(p) + hoff * elem, 0, dh * dh * elem, 0x00020000);
  };

  // 16-byte chunk c of row r lies at chunk c ^ swz(r): see head_polar.hip
  auto swz = [](int r) { return ((r >> 2) & 1) | ((r & 1) << 1) | ((r & 2) << 1) | ((r ^ (r << 1)) & 8); };
  const int s = swz(col), t = 8 * kg + (col >> 2);
  const uint32_t l_row = col * kRowB + ((kg ^ s) << 4);                                              // row col, chunk kg
  const uint32_t l_tr = t * kRowB + ((((col >> 1) & 1) ^ swz(t)) << 4) + 8 * (col & 1);              // row 8 kg + col / 4, element 4 (col % 4)
  const uint32_t l_put = col * kRowB + (((kg >> 1) ^ s) << 4) + 8 * (kg & 1);                        // row col, element 4 kg

  // X^T to LDS, 2 rows per instruction; what lies beyond the head reads zero.  Rows p first, into the place of W: the right operand
  // of every wavefront's G.  Then each wavefront the row tiles it takes of G, which it can start on one by one as they land.
  const auto rx = rsrc(Xt, 2);
  const int half = lane >> 5, pc = lane & 31;
  auto fetch = [&](__amdgpu_buffer_rsrc_t r, unsigned char* to, int row0, int from) {
    const int row = from + half, chunk = pc ^ swz(row0 + half);
    const uint32_t off = row < dh && 8 * chunk < dh ? (uint32_t)(row * dh + 8 * chunk) * 2u : kOob;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(to + row0 * kRowB), 16, off, 0, 0, 0);
  };
#pragma unroll
  for (int q = 0; q < (P / 2 + kNW - 1) / kNW; ++q)
    if (q * kNW + wave < P / 2) fetch(rx, sW, 2 * (q * kNW + wave), n0 + 2 * (q * kNW + wave));
#pragma unroll
  for (int q = 0; q < 8 * TM; ++q) fetch(rx, sX, 16 * TM * wave + 2 * q, 16 * TM * wave + 2 * q);
  __builtin_amdgcn_s_waitcnt(vmcnt(8 * TM));
  asm volatile("s_barrier" ::: "memory");   // (without the fence of __syncthreads, which would wait for the rows as well)

  // rows row .. row + 15 of an LDS matrix, K elements 32 kk + 8 kg .. + 7
  auto frag = [&](const unsigned char* base, int row, int kk) {
    return *reinterpret_cast<const f16x8*>(base + row * kRowB + (l_row ^ (kk << 6)));
  };
  // rows 16 i + col of the matrix's transpose
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
  auto frag_tr = [&](int i, int kk) {
    unsigned char* const p = sX + 32 * kk * kRowB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + (l_tr ^ (i << 5))));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 4 * kRowB + (l_tr ^ (i << 5) ^ 144)));   // swz(r + 4) = swz(r) ^ 9
    return __builtin_bit_cast(f16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto pack_f16 = [](const f32x4& a) { return make_uint2(f32x2_to_f16x2(a[0], a[1]), f32x2_to_f16x2(a[2], a[3])); };

  // Element r of acc[i][j]: row 16 (TM wave + i) + 4 kg + r, column n0 + 16 j + col.
  const int i0 = TM * wave;
  f32x4 acc[TM][TN];
  auto zero = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  // G[:, p]
  zero();
  {
    f16x8 b[TN][KB];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int kk = 0; kk < KB; ++kk) b[j][kk] = frag(sW, 16 * j, kk);
    static_assert(TM <= 2, "row tiles of a wavefront");
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (TM - i == 2) __builtin_amdgcn_s_waitcnt(vmcnt(8));
      else __builtin_amdgcn_s_waitcnt(vmcnt(0));
      asm volatile("" ::: "memory");   // (the tile's reads stay behind the wait)
      f16x8 a[KB];
#pragma unroll
      for (int kk = 0; kk < KB; ++kk) a[kk] = frag(sX, 16 * (i0 + i), kk);
      __builtin_amdgcn_sched_barrier(0);   // (all reads in flight: left alone, the compiler waits for one at a time)
#pragma unroll
      for (int kk = 0; kk < KB; ++kk)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[kk], b[j][kk], acc[i][j], 0, 0, 0);
    }
  }
  __syncthreads();   // everyone has rows p, whose place W takes
  // W[:, p] (as the general path's epilogue rounds it)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const float on = 16 * (i0 + i) == n0 + 16 * j ? ci : 0.0f;
      f32x4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = fmaf(on, 4 * kg + r == col ? 1.0f : 0.0f, cg * acc[i][j][r]);
      *reinterpret_cast<uint2*>(sW + 16 * j * kRowB + (l_put ^ ((i0 + i) << 5))) = pack_f16(v);
    }
  __syncthreads();
  // X'[:, p]
  zero();
  {
    constexpr int KH = KB / 2;   // half of K at a time in registers, the other half's reads on the way
    f16x8 a[2][KH][TM], b[2][KH][TN];
    auto read = [&](int half) {
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        const int kk = half * KH + k;
#pragma unroll
        for (int j = 0; j < TN; ++j) b[half][k][j] = frag(sW, 16 * j, kk);
#pragma unroll
        for (int i = 0; i < TM; ++i) a[half][k][i] = frag_tr(i0 + i, kk);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int half) {
#pragma unroll
      for (int k = 0; k < KH; ++k)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[half][k][i], b[half][k][j], acc[i][j], 0, 0, 0);
    };
    read(0);
    read(1);
    multiply(0);
    multiply(1);
  }

  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const auto rt = rsrc(Xt_out, 2);
  auto put_tr = [&](int i, int j, const uint2& v) {   // rows n past the head lie past the range
    const uint32_t off = (uint32_t)((n0 + 16 * j + col) * dh + 16 * (i0 + i) + 4 * kg) * 2u;
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, rt, 16 * (i0 + i) < dh ? off : kOob, 0, 0);
  };
  if (!last) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) put_tr(i, j, pack_f16(acc[i][j]));
    return;
  }
  // The hand-over to the closing iterations: rounded to bf16, that value as fp32, transposed and natural plane.
  const auto r32 = rsrc(X32, 4), rn = rsrc(Pn, 2);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const uint2 v = make_uint2(f32x2_to_bf16x2(acc[i][j][0], acc[i][j][1]), f32x2_to_bf16x2(acc[i][j][2], acc[i][j][3]));
      put_tr(i, j, v);
      const int n = n0 + 16 * j + col;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t bits = (r & 2 ? v.y : v.x) >> (16 * (r & 1)) & 0xffffu;
        const uint32_t el = (uint32_t)((16 * (i0 + i) + 4 * kg + r) * dh + n);   // rows past the head: past the range
        __builtin_amdgcn_raw_buffer_store_b32(bits << 16, r32, n < dh ? el * 4u : kOob, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)bits, rn, n < dh ? el * 2u : kOob, 0, 0);
      }
    }
}

template <int N, int P>
hipError_t launch_one(const bf16_bits* Xt, int heads, int dh, float a, float b, bf16_bits* Xt_out, int last, float* X32, bf16_bits* Pn,
                      hipStream_t s) {
  constexpr int smem = (N + P) * kRowB;
  static PerDeviceOnce configured;
  constexpr int NW = N == 256 ? 8 : 12;   // whole row tiles each (see above)
  auto kern = k_polar_step<N, P, NW>;
  hipError_t e = configured.run([&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (e != hipSuccess) return e;
  const int panels = (dh + P - 1) / P;
  hipLaunchKernelGGL(kern, dim3(panels * heads), dim3(64 * NW), smem, s, Xt, dh, panels, a, b, Xt_out, last, X32, Pn);
  return hipGetLastError();
}

// 32 columns per workgroup from more than one workgroup per compute unit on.
int panel_width(int heads, int dh) { return (int64_t)heads * (dh / 16) <= 256 ? 16 : 32; }

int square_width(int dh) { return dh <= 192 ? 192 : 256; }

}  // namespace

double polar_step_flop(int heads, int dh) {
  const double n = square_width(dh), p = panel_width(heads, dh);
  return 4.0 * n * n * (double)round_up(dh, (int64_t)p) * heads;
}

hipError_t launch_polar_step(const bf16_bits* Xt, int heads, int dh, float a, float b, bf16_bits* Xt_out, int last, float* X32, bf16_bits* Pn,
                             hipStream_t s) {
  if (heads < 1 || dh < 16 || dh > kPolarStepMaxDh || (dh & 15) || !Xt || !Xt_out || Xt == Xt_out || (last && (!X32 || !Pn)))
    return hipErrorInvalidValue;
  using std::integral_constant;
  auto go = [&](auto n, auto p) {
    return launch_one<decltype(n)::value, decltype(p)::value>(Xt, heads, dh, a, b, Xt_out, last, X32, Pn, s);
  };
  const bool narrow = panel_width(heads, dh) == 16;
  if (square_width(dh) == 192)
    return narrow ? go(integral_constant<int, 192>{}, integral_constant<int, 16>{}) : go(integral_constant<int, 192>{}, integral_constant<int, 32>{});
  return narrow ? go(integral_constant<int, 256>{}, integral_constant<int, 16>{}) : go(integral_constant<int, 256>{}, integral_constant<int, 32>{});
}

// One step from the same start planes either way, for tests: launch_polar_step, or (two_launches) the two products it stands for,
// which also need the natural plane Xn and room for W and write the natural plane after every step.  DEVICE pointers, default
// stream.  Returns the hipError_t.
extern "C" __attribute__((visibility("default"))) int conqur_polar_step_for_tests(int two_launches, const bf16_bits* Xn, const bf16_bits* Xt, int heads,
                                                                                  int dh, float a, float b, int last, bf16_bits* Xt_out, float* X32,
                                                                                  bf16_bits* Xn_out, bf16_bits* W) {
  if (!two_launches) return launch_polar_step(Xt, heads, dh, a, b, Xt_out, last, X32, Xn_out, nullptr);
  GemmArgs g{};
  g.ab_f16 = 1;
  g.A = g.B = Xt; g.lda = g.ldb = g.ldc = dh; g.batchA = g.batchB = g.batchC = (int64_t)dh * dh;
  g.M = g.N = g.K = dh;
  g.nseg = 1;
  g.np_out = 1; g.plane_out = heads * g.batchC;
  GemmArgs x = g;
  g.Pn = W; g.symmetric = 1; g.coef_i = a; g.coef_g = b;
  const hipError_t e = launch_gemm_nt(g, EPI_GRAMW, heads, nullptr);
  if (e != hipSuccess) return e;
  x.A = Xn; x.B = W; x.Pn = Xn_out; x.Pt = Xt_out;
  if (last) x.C32 = X32;
  else x.np_out_n = 1;
  return launch_gemm_nt(x, last ? EPI_XLAST : EPI_XOUT, heads, nullptr);
}

}  // namespace conqur
