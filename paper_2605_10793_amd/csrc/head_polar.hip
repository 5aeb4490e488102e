// Main phase of the polar iteration for heads of width up to 128, one launch for all steps
// (the composed cubics X <- X (a_k I + b_k X^T X) of the Procrustes update, Sec. 3.3).
//
// At these widths the iterate (up to 34 KiB as fp16, natural and transposed) and the
// polynomial factor W live in the LDS of one compute unit, so a workgroup per head runs the
// whole schedule without touching HBM between steps; the general path needs two GEMM launches
// per step, which at 128 x 128 are launch latency only (32 heads of width 64: 41 launches of
// 4.3 us, the update 229 us; here one launch, the update 34).  Per step, with every product 16x16x32 fp16
// MFMAs on K-contiguous operands (the iterate and the factor are held as fp16: 11 significant
// bits at the rate of bf16's 8; every entry is at most a few units in magnitude):
//   G = X^T X            A = B = X^T                     -> W = a I + b G, fp16, to LDS
//   X' = X W             A = X,  B = W (symmetric)       -> accumulators hold X'
// An accumulator lane owns 4 consecutive rows of one column, i.e. 8 contiguous bytes of the transposed matrix:
// X'^T goes to LDS as packed 8-byte writes, X' itself as four 2-byte writes per such group.  Computing the product in
// the other orientation as well (X'^T = W X^T, packed stores for both layouts) costs a third of the step's MFMA and
// LDS-read time and is kept for the last step only, whose results leave for HBM.
// The last step writes what the closing iterations read: the iterate rounded to bf16, as
// fp32 and as one plane of each layout.  On request the same launch then takes the closing
// step itself (exact Gram matrix of that bf16 iterate, D, D^2, two-plane correction; bf16
// MFMAs) and leaves the rotation, the rotate operand and <R, M>: see HeadPolarClose.
//
// Widths between multiples of 32 run in the next larger square, zero outside the head: zero rows and columns of X stay
// zero through every step, and the identity of the closing step ends at the head's width.
#include "kernels.h"

#include <type_traits>

namespace conqur {

namespace {

// N: width of the square (a multiple of 32); WGM x WGN wavefronts own (N / WGM) x (N / WGN) blocks of every product.
// DH128: heads of width 128 themselves.  Their results keep the order of roundings they have always had; narrower heads, 112
// in the square of 128 among them, have the general path's, bit for bit.
template <int N, int WGM, int WGN, bool CLOSE, bool DH128>
__global__ void __launch_bounds__(64 * WGM * WGN) k_head_polar(const bf16_bits* __restrict__ Xn0, const bf16_bits* __restrict__ Xt0,
                                                               const int dh, const PolarSchedule sched, float* __restrict__ X32,
                                                               bf16_bits* __restrict__ Pn, bf16_bits* __restrict__ Pt,
                                                               const HeadPolarClose cl, const HeadPolarStart st) {
  constexpr int NT = 64 * WGM * WGN, WM = N / WGM, WN = N / WGN, TM = WM / 16, TN = WN / 16;
  static_assert(N % 32 == 0 && WM % 16 == 0 && WN % 16 == 0, "whole MFMA tiles");
  // bytes per LDS row: the 16-byte pad spreads 16 consecutive rows of one chunk (fragment reads), 16 columns x 4 row groups of
  // 8 bytes (transposed writes) and 4 rows x 16 values (natural writes) over the 64 banks
  constexpr int ROWB = N * 2 + 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* const sXn = smem;                  // X   : row r, K = column
  unsigned char* const sXt = smem + N * ROWB;       // X^T : row c, K = row of X
  unsigned char* const sW = smem + 2 * N * ROWB;    // W   : symmetric
  __shared__ double red[5][WGM * WGN];
  const int h = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kg = lane >> 4, col = lane & 15;
  const int wm = wave / WGN, wn = wave % WGN;
  const int mb = WM * wm, nb = WN * wn;             // this wavefront's block of every product
  const int64_t hoff = (int64_t)h * dh * dh;

  typedef f32x4 Acc[TM][TN];
  auto frag = [&](const unsigned char* base, int row, int kk) {
    return *reinterpret_cast<const f16x8*>(base + (row + col) * ROWB + kk * 64 + kg * 16);
  };
  auto zero = [](Acc& v) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) v[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  // acc[i][j] += sum_k A[mb + 16 i + .][k] B[nb + 16 j + .][k], fp16 or bf16 operands
  auto product = [&](auto f16, const unsigned char* A, const unsigned char* B, Acc& acc) {
#pragma unroll
    for (int kk = 0; kk < N / 32; ++kk) {
      f16x8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = frag(A, mb + 16 * i, kk);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = frag(B, nb + 16 * j, kk);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (decltype(f16)::value) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
          else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[i]), __builtin_bit_cast(bf16x8, fb[j]), acc[i][j], 0, 0, 0);
        }
    }
  };
  constexpr std::true_type kF16{};
  constexpr std::false_type kBF16{};
  // Element r of acc[i][j]: row m = mb + 16 i + 4 kg + r, column n = nb + 16 j + col.  fn(i, j, m of r = 0, n) over the block;
  // inside(i, j): whether the 16 x 16 tile lies in the head (dh is a multiple of 16: as a whole or not at all).
  auto each = [&](auto&& fn) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) fn(i, j, mb + 16 * i + 4 * kg, nb + 16 * j + col);
  };
  auto inside = [&](int i, int j) { return mb + 16 * i < dh && nb + 16 * j < dh; };
  auto tr_addr = [&](int m0, int n) { return n * ROWB + m0 * 2; };      // transposed: row n, K positions m0 .. m0 + 3 (8 bytes)
  // the transposed matrix into an LDS operand (fp16): W = ci I + cg acc, or the iterate itself
  auto store_transposed = [&](unsigned char* dst, const Acc& acc, float ci, float cg) {
    each([&](int i, int j, int m0, int n) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // (as the general path's epilogue rounds it, the product first; heads of width 128: the identity's part first)
        const float eye = m0 + r == n ? 1.0f : 0.0f;
        v[r] = DH128 ? fmaf(cg, acc[i][j][r], eye * ci) : fmaf(ci, eye, cg * acc[i][j][r]);
      }
      *reinterpret_cast<uint2*>(dst + tr_addr(m0, n)) = make_uint2(f32x2_to_f16x2(v[0], v[1]), f32x2_to_f16x2(v[2], v[3]));
    });
  };
  // the iterate in both layouts: packed rows of X^T, and row m, K position n of X one value at a time
  auto store_iterate = [&](const Acc& acc) {
    each([&](int i, int j, int m0, int n) {
      const uint32_t lo = f32x2_to_f16x2(acc[i][j][0], acc[i][j][1]), hi = f32x2_to_f16x2(acc[i][j][2], acc[i][j][3]);
      *reinterpret_cast<uint2*>(sXt + tr_addr(m0, n)) = make_uint2(lo, hi);
      unsigned char* d = sXn + m0 * ROWB + n * 2;
      *reinterpret_cast<unsigned short*>(d) = (unsigned short)lo;
      *reinterpret_cast<unsigned short*>(d + ROWB) = (unsigned short)(lo >> 16);
      *reinterpret_cast<unsigned short*>(d + 2 * ROWB) = (unsigned short)hi;
      *reinterpret_cast<unsigned short*>(d + 3 * ROWB) = (unsigned short)(hi >> 16);
    });
  };
  // sum of one double per lane over the workgroup, known to every thread afterwards (a slot is used once)
  auto block_sum = [&](double v, int slot) {
    v = wave_sum_d(v);
    if (lane == 0) red[slot][wave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < WGM * WGN; ++q) t += red[slot][q];
    return t;
  };

  Acc acc, accT;
  if (st.M) {
    // The start of the update in this launch as well (what the packing pass does on the general path):
    // X0 = (M + lambda tau R_prev) / alpha, tau = ||M||_F / sqrt(dh), alpha = ||M||_F (1 + lambda); lambda = 0 stands for the
    // limit at fp32 resolution, an empty M for R_prev itself.  ||M||_F^2 is the sum of the partial sums the reduction of the
    // token shares left, or is taken here.  Elements in the accumulators' layout, so that the two LDS operands are written
    // exactly as after a step.
    Acc prev;
    zero(acc);
    zero(prev);
    double f2 = 0.0, dot = 0.0;
    each([&](int i, int j, int m0, int n) {
      if (!inside(i, j)) return;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t off = hoff + (int64_t)(m0 + r) * dh + n;
        acc[i][j][r] = st.M[off];
        prev[i][j][r] = st.R[off];
        if (st.R_keep) st.R_keep[off] = prev[i][j][r];
      }
    });
    if (st.nparts > 0) {
      for (int p = 0; p < st.nparts; ++p) f2 += st.fro2_parts[(int64_t)h * st.nparts + p];
    } else {
      each([&](int i, int j, int, int) {
#pragma unroll
        for (int r = 0; r < 4; ++r) f2 += (double)acc[i][j][r] * acc[i][j][r];
      });
      f2 = block_sum(f2, 0);
    }
    if (st.rop_dot) {   // <R_op, M>: the l1 term of the rows this update consumes (see k_dot_rm)
      each([&](int i, int j, int, int) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          dot += (double)acc[i][j][r] * (st.round_bf16 ? bf16_to_f32(f32_to_bf16(prev[i][j][r])) : prev[i][j][r]);
      });
      dot = block_sum(dot, 1);
    }
    if (tid == 0) {
      st.fro2_out[h] = f2;
      if (st.ldot) st.ldot[h] = st.rop_dot ? dot : st.L[h];   // kept before the statistics restart
    }
    const double f = sqrt(f2);
    const bool empty = !(f > 0.0);
    const float lambda = fmaxf(st.lambda, 9.5367431640625e-07f);
    const float tau = (float)(f / sqrt((double)dh));
    const float inv_alpha = empty ? 1.0f : (float)(1.0 / (f * (1.0 + (double)lambda)));
    const float cm = empty ? 0.0f : inv_alpha, cr = empty ? 1.0f : lambda * tau * inv_alpha;
    each([&](int i, int j, int, int) {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = fmaf(cm, acc[i][j][r], cr * prev[i][j][r]);   // (as the packing pass rounds it)
    });
    store_iterate(acc);
  } else {   // the start iterate is given as planes
    for (int idx = tid; idx < N * (N / 8); idx += NT) {
      const int row = idx / (N / 8), chunk = idx % (N / 8);
      uint4 a = make_uint4(0u, 0u, 0u, 0u), b = a;
      if (row < dh && chunk * 8 < dh) {
        a = *reinterpret_cast<const uint4*>(Xn0 + hoff + (int64_t)row * dh + chunk * 8);
        b = *reinterpret_cast<const uint4*>(Xt0 + hoff + (int64_t)row * dh + chunk * 8);
      }
      *reinterpret_cast<uint4*>(sXn + row * ROWB + chunk * 16) = a;
      *reinterpret_cast<uint4*>(sXt + row * ROWB + chunk * 16) = b;
    }
  }
  __syncthreads();
  for (int k = 0; k < sched.nsteps; ++k) {
    const bool last = k + 1 == sched.nsteps;
    // G = X^T X;  W = a I + b G (G symmetric: storing the transpose stores W itself)
    zero(acc);
    product(kF16, sXt, sXt, acc);
    store_transposed(sW, acc, sched.a[k], sched.b[k]);
    __syncthreads();
    zero(acc);
    product(kF16, sXn, sW, acc);                  // X'   [r][c]
    if (last) {
      zero(accT);
      product(kF16, sW, sXn, accT);               // X'^T [c][r]: the natural-layout plane below as packed stores
      break;
    }
    __syncthreads();                              // every wavefront has read the old iterate
    store_iterate(acc);
    __syncthreads();
  }

  // Hand-over to the closing iterations: the result rounded to bf16 like every step's, and exactly that value as fp32 X,
  // as one transposed plane (from X') and as one natural plane (from X'^T; the two orientations issue the same products
  // in the same order, so they hold the same numbers): the closing Gram matrix is then exact with one plane product.
  auto rounded = [](f32x4& a) {   // the packed bf16 values; a becomes exactly those
    const uint2 t = make_uint2(f32x2_to_bf16x2(a[0], a[1]), f32x2_to_bf16x2(a[2], a[3]));
    a = f32x4{__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16), __uint_as_float(t.y & 0xffff0000u)};
    return t;
  };
  each([&](int i, int j, int m0, int n) {
    const uint2 hi = rounded(acc[i][j]), thi = rounded(accT[i][j]);
    if (!inside(i, j)) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) X32[hoff + (int64_t)(m0 + r) * dh + n] = acc[i][j][r];
    *reinterpret_cast<uint2*>(Pt + hoff + (int64_t)n * dh + m0) = hi;     // X^T[c = n][r = m0 ..]
    *reinterpret_cast<uint2*>(Pn + hoff + (int64_t)n * dh + m0) = thi;    // accT: X[r = n][c = m0 ..]
  });

  if constexpr (CLOSE) {
    // ---- the closing step of the update in the same launch (Sec. 3.3; the general path's sequence of Gram matrix, D^2,
    // correction product and finishing pass, with the same operand planes): D = (I - X^T X)/2 from the exact bf16 iterate,
    // X <- X + X (D + 1.5 D^2) with the correction as two bf16 planes, then R, the rotate operand R^T and <R, M>.
    // The step is taken only if this head's residual allows the quintic form (cl.res_max); otherwise the head reports
    // its residual, marks the step as not taken (sq_out < 0) and the host continues on the general path from the
    // hand-over state written above.
    unsigned char* const sD0 = sW;                    // first plane of D, then of the correction
    unsigned char* const sD1 = smem + 3 * N * ROWB;   // second plane
    // bf16 planes of a symmetric matrix given as accumulator blocks: the transposed store of block (wm, wn) is block
    // (wn, wm) of the matrix itself
    auto store_planes = [&](const Acc& v) {
      each([&](int i, int j, int m0, int n) {
        const f32x4 a = v[i][j];
        f32x4 hi = a;
        const uint2 h0 = rounded(hi);
        const f32x4 lo = a - hi;
        *reinterpret_cast<uint2*>(sD0 + tr_addr(m0, n)) = h0;
        *reinterpret_cast<uint2*>(sD1 + tr_addr(m0, n)) = make_uint2(f32x2_to_bf16x2(lo[0], lo[1]), f32x2_to_bf16x2(lo[2], lo[3]));
      });
    };
    __syncthreads();   // every wavefront has finished the last step's reads of the old iterate and of W
    // the rounded iterate as bf16 operands: X^T from X', X from X'^T (packed 8-byte writes both)
    each([&](int i, int j, int m0, int n) {
      *reinterpret_cast<uint2*>(sXt + tr_addr(m0, n)) = rounded(acc[i][j]);
    });
    // accT's block is (wm, wn) of X^T as a product of W's rows and X's rows: element (m, n) is X[n][m]
    each([&](int i, int j, int m0, int n) {
      *reinterpret_cast<uint2*>(sXn + tr_addr(m0, n)) = rounded(accT[i][j]);
    });
    __syncthreads();
    // G = X^T X (products of bf16 values are exact in fp32), D = (I - G) / 2, ||I - G||_F^2
    Acc dm;
    zero(dm);
    product(kBF16, sXt, sXt, dm);
    double part = 0.0;
    each([&](int i, int j, int m0, int n) {
      float p32 = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dlt = (m0 + r == n && n < dh ? 1.0f : 0.0f) - dm[i][j][r];
        p32 += dlt * dlt;
        dm[i][j][r] = 0.5f * dlt;
      }
      part += (double)p32;
    });
    const double res2 = block_sum(part, 2);
    if (!(res2 <= (double)cl.res_max * cl.res_max)) {   // (also a non-finite residual)
      if (tid == 0) { cl.res_out[h] = res2; cl.sq_out[h] = -1.0; }
      return;
    }
    store_planes(dm);
    __syncthreads();
    // D^2 from the first plane (second-order small: one plane is ample), ||D^2||_F^2, the correction D + 1.5 D^2
    Acc sq;
    zero(sq);
    product(kBF16, sD0, sD0, sq);
    part = 0.0;
    each([&](int i, int j, int, int) {
      float p32 = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p32 += sq[i][j][r] * sq[i][j][r];
      }
      part += (double)p32;
      if constexpr (DH128) {
        dm[i][j] += 1.5f * sq[i][j];
      } else {   // D as its two planes hold it: the rounding of the general path, bit for bit
        f32x4 d0 = dm[i][j];
        rounded(d0);
        f32x4 d1 = dm[i][j] - d0;
        rounded(d1);
#pragma unroll
        for (int r = 0; r < 4; ++r) dm[i][j][r] = fmaf(1.5f, sq[i][j][r], d0[r]) + d1[r];
      }
    });
    const double sq2 = block_sum(part, 3);   // (its barrier: every wavefront has read the planes of D)
    store_planes(dm);
    __syncthreads();
    // X <- X + X (W0 + W1).  The small correction is summed on its own and the iterate added once at the end: with the
    // iterate as the accumulators' start every MFMA would round at the iterate's magnitude, and the orthogonality of the
    // result was measured above the bound that holds for the general path's order.
    zero(sq);
    product(kBF16, sXn, DH128 ? sD0 : sD1, sq);   // (the general path's order: smaller plane first)
    product(kBF16, sXn, DH128 ? sD1 : sD0, sq);
    // R, the rotate operand R^T (bf16 planes, [n][m]: packed rows of the transposed matrix) and <R, M>
    part = 0.0;
    each([&](int i, int j, int m0, int n) {
      acc[i][j] += sq[i][j];
      if (!inside(i, j)) return;
      float p32 = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t off = hoff + (int64_t)(m0 + r) * dh + n;
        cl.R[off] = acc[i][j][r];
        p32 += acc[i][j][r] * cl.M[off];
      }
      part += (double)p32;
      f32x4 left = acc[i][j];
      for (int p = 0; p < cl.rop_planes; ++p) {
        f32x4 hi = left;
        *reinterpret_cast<uint2*>(cl.RopT + p * cl.rop_plane + hoff + (int64_t)n * dh + m0) = rounded(hi);
        left -= hi;
      }
    });
    const double inner = block_sum(part, 4);
    if (tid == 0) { cl.res_out[h] = res2; cl.sq_out[h] = sq2; cl.inner_out[h] = inner; }
  }
}

template <int N, int WGM, int WGN, bool CLOSE, bool DH128>
hipError_t launch_one(const bf16_bits* Xn0, const bf16_bits* Xt0, int heads, int dh, const PolarSchedule& sched, float* X32,
                      bf16_bits* Pn, bf16_bits* Pt, const HeadPolarClose& cl, const HeadPolarStart& st, hipStream_t s) {
  constexpr int smem = (CLOSE ? 4 : 3) * N * (N * 2 + 16);   // the closing step holds two planes of its correction beside the iterate
  static PerDeviceOnce configured;
  auto kern = k_head_polar<N, WGM, WGN, CLOSE, DH128>;
  hipError_t e = configured.run([&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(heads), dim3(64 * WGM * WGN), smem, s, Xn0, Xt0, dh, sched, X32, Pn, Pt, cl, st);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_head_polar(const bf16_bits* Xn0, const bf16_bits* Xt0, int heads, int dh, const PolarSchedule& sched, float* X32,
                             bf16_bits* Pn, bf16_bits* Pt, const HeadPolarClose* close, const HeadPolarStart* start, hipStream_t s) {
  if (heads < 1 || dh < 16 || dh > kHeadPolarMaxDh || (dh & 15) || sched.nsteps < 1 || sched.nsteps > kPolarScheduleMax) return hipErrorInvalidValue;
  if (close && (!close->R || !close->RopT || !close->M || !close->res_out || !close->sq_out || !close->inner_out || close->rop_planes < 1))
    return hipErrorInvalidValue;
  if (start && (!start->M || !start->R || (start->nparts > 0 && !start->fro2_parts) || !start->fro2_out ||
                (start->ldot && !start->rop_dot && !start->L)))
    return hipErrorInvalidValue;
  if (!start && (!Xn0 || !Xt0)) return hipErrorInvalidValue;
  const HeadPolarStart st = start ? *start : HeadPolarStart{};
  const HeadPolarClose cl = close ? *close : HeadPolarClose{};
  auto go = [&](auto n, auto wgm, auto wgn, auto own) {
    constexpr int N = decltype(n)::value, M_ = decltype(wgm)::value, N_ = decltype(wgn)::value;
    constexpr bool OWN = decltype(own)::value;
    return close ? launch_one<N, M_, N_, true, OWN>(Xn0, Xt0, heads, dh, sched, X32, Pn, Pt, cl, st, s)
                 : launch_one<N, M_, N_, false, OWN>(Xn0, Xt0, heads, dh, sched, X32, Pn, Pt, cl, st, s);
  };
  // 8 wavefronts (2 per SIMD, so that one's LDS writes and conversions run beside the other's MFMAs) read half as much LDS
  // again as 4 with square blocks and are still ahead: 32 heads of width 128, 22 steps, whole update 94 us with 2 x 2, 86 with
  // 4 x 2, 92 with 4 x 4 wavefronts; width 64: 35, 34, 37; width 96 (9 steps): 38, 36 with 3 x 2, 36 with 3 x 3.
  using std::integral_constant;
  constexpr integral_constant<int, 2> two{};
  constexpr integral_constant<int, 3> three{};
  constexpr integral_constant<int, 4> four{};
  constexpr std::false_type general{};
  if (dh <= 32) return go(integral_constant<int, 32>{}, two, two, general);
  if (dh <= 64) return go(integral_constant<int, 64>{}, four, two, general);
  if (dh <= 96) return go(integral_constant<int, 96>{}, three, two, general);
  if (dh < 128) return go(integral_constant<int, 128>{}, four, two, general);
  return go(integral_constant<int, 128>{}, four, two, std::true_type{});
}

}  // namespace conqur
