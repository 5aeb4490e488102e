// Main phase of the polar iteration for heads of width up to 128, one launch for all steps
// (the composed cubics X <- X (a_k I + b_k X^T X) of the Procrustes update, Sec. 3.3).
//
// At these widths the iterate (up to 32 KiB as fp16) lives in the LDS of one compute unit and the polynomial factor W in its
// registers, so a workgroup per head runs the whole schedule without touching HBM between steps; the general path needs two
// GEMM launches per step, which at 128 x 128 are launch latency only (32 heads of width 64: 41 launches of 4.3 us).  Per step,
// with every product 16x16x32 fp16 MFMAs (the iterate and the factor are held as fp16: 11 significant bits at the rate of
// bf16's 8; every entry is at most a few units in magnitude):
//   G = X^T X            rows of X^T from LDS            -> W = a I + b G, fp16
//   X' = X W             X by transposing reads of X^T   -> accumulators hold X'
// A wavefront computes whole columns of every product.  So the columns of W it needs are the ones it has computed: two lane
// swaps per pair of accumulator tiles make them the right operand of X' = X W, and W never leaves the registers.  LDS holds X^T
// alone, twice: a lane owns 4 consecutive rows of one column of X', i.e. 8 contiguous bytes of a row of X'^T, and a step that
// writes the buffer nobody reads has one barrier, at its end.
// What bounds it: a step is a chain (fragments, G, W, X', barrier) on one compute unit per head.  At width 128 its 128 MFMAs
// per wavefront take 0.85 us and its 288 KiB of LDS reads about as long; the step takes 1.6.  With W and X in LDS as well, in
// blocks of 32 x 64 per wavefront (392 KiB read at two-way bank conflicts, W and X written, three barriers) it took 2.5.  The
// whole update, 32 heads, by events, before and now: width 128, 22 steps 93.5 and 69 us; 64, 22 steps 36.3 and 29.4; 96, 9
// steps 42 and 34; 16 heads of width 32, 22 steps 24.3 and 22.
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

// N: width of the square (a multiple of 32); NW wavefronts of N / NW columns each.  Two wavefronts per SIMD are asked for not to
// have them (a workgroup has one) but to keep a wavefront within 256 registers: beyond, the compiler puts the accumulators in the
// other half and moves every one of them before use, 128 moves a step.
// DH128: heads of width 128 themselves.  Their results keep the order of roundings they have always had; narrower heads, 112
// in the square of 128 among them, have the general path's, bit for bit.
template <int N, int NW, bool CLOSE, bool DH128>
__global__ void __launch_bounds__(64 * NW, 2) k_head_polar(const bf16_bits* __restrict__ Xt0, const int dh, const PolarSchedule sched,
                                                        float* __restrict__ X32, bf16_bits* __restrict__ Pn, bf16_bits* __restrict__ Pt,
                                                        const HeadPolarClose cl, const HeadPolarStart st) {
  constexpr int NT = 64 * NW, WN = N / NW, TM = N / 16, TN = WN / 16, KB = N / 32;
  static_assert(N % 32 == 0 && N <= 128 && WN % 16 == 0, "whole MFMA tiles, rows of at most 256 bytes");
  constexpr int ROWB = 256;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* const buf0 = smem;                 // X^T : row c, K = row of X; a step reads one buffer and writes the other
  unsigned char* const buf1 = smem + N * ROWB;
  unsigned char* const start = sched.nsteps & 1 ? buf0 : buf1;   // (so that the last step reads buf0)
  __shared__ double red[5][NW];
  const int h = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 4, col = lane & 15;
  const int nb = WN * wave;                         // this wavefront's columns of every product
  const int64_t hoff = (int64_t)h * dh * dh;

  typedef f32x4 Acc[TM][TN];
  auto zero = [](auto& v) {
    for (auto& row : v)
      for (auto& e : row) e = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  // 16-byte chunk c of row r lies at chunk c ^ swz(r).  A 16-byte read of 16 rows x 4 chunks is served 16 lanes at a time, rows
  // 0-3 and 12-15 of one chunk with rows 4-11 of the next (measured: 272-byte rows without a swizzle conflict two ways); a
  // transposing read takes 32 bytes of 8 rows.  Both spread over all banks: bits 0 and 1 and the difference of bits 2 and 3 of
  // the row number the eight 32-byte places, bit 2 the half.
  auto swz = [](int r) { return ((r >> 2) & 1) | ((r & 1) << 1) | ((r & 2) << 1) | ((r ^ (r << 1)) & 8); };
  // Addresses: an offset of the lane, XORed with the chunk, on top of constants.  lanes() gives the lane offsets anew to each
  // step and product: addresses shared between them would stay live throughout, and the accumulators need the registers.
  struct Lanes { uint32_t row, own, tr, put; };
  auto lanes = [&]() {
    const int s = swz(col), t = 8 * kg + (col >> 2);
    Lanes l;
    l.row = col * ROWB + ((kg ^ s) << 4);                                         // row col, chunk kg
    l.own = l.row + nb * ROWB;                                                    // ... of this wavefront's columns
    l.tr = t * ROWB + ((((col >> 1) & 1) ^ swz(t)) << 4) + 8 * (col & 1);         // row 8 kg + col / 4, element 4 (col % 4)
    l.put = (nb + col) * ROWB + (((kg >> 1) ^ s) << 4) + 8 * (kg & 1);            // row nb + col, element 4 kg
    asm volatile("" : "+v"(l.row), "+v"(l.own), "+v"(l.tr), "+v"(l.put));
    return l;
  };
  // rows row + col of an LDS matrix (from l.row; nb + row + col from l.own), K elements 32 kk + 8 kg .. + 7
  auto frag = [&](const unsigned char* base, uint32_t at, int row, int kk) {
    return *reinterpret_cast<const f16x8*>(base + row * ROWB + (at ^ (kk << 6)));
  };
  // Rows 16 i + col of the matrix's transpose: K runs over the rows.  A transposing read gives lane l of 16 the element l of 4
  // rows, whose 16 elements lie under the addresses of 4 lanes each.
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
  auto frag_tr = [&](unsigned char* base, const Lanes& l, int i, int kk) {
    unsigned char* const p = base + 32 * kk * ROWB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + (l.tr ^ (i << 5))));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 4 * ROWB + (l.tr ^ (i << 5) ^ 144)));   // swz(r + 4) = swz(r) ^ 9
    return __builtin_bit_cast(f16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto mfma = [](auto f16, const f16x8& a, const f16x8& b, f32x4& c) {
    if constexpr (decltype(f16)::value) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  };
  // acc[i][j] += sum_k A[16 i + .][k] B[nb + 16 j + .][k], fp16 or bf16 operands
  auto product = [&](auto f16, const unsigned char* A, const unsigned char* B, Acc& acc) {
    const Lanes l = lanes();
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
      f16x8 fa[TM], fb[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = frag(B, l.own, 16 * j, kk);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = frag(A, l.row, 16 * i, kk);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) mfma(f16, fa[i], fb[j], acc[i][j]);
      if (N > 96) __builtin_amdgcn_sched_barrier(0);   // (bounds what the scheduler keeps live: without it width 128 spills)
    }
  };
  // The right operand of a product whose columns this wavefront holds itself, in registers: f[kk][j] is column nb + 16 j + col,
  // K elements 32 kk + 8 kg .. + 7.
  typedef f16x8 Cols[KB][TN];
  // acc[i][j] += sum_k X[16 i + .][k] W[k][nb + 16 j + .], X from its transpose At
  auto product_tr = [&](auto f16, unsigned char* At, const Cols& w, Acc& acc) {
    const Lanes l = lanes();
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
      f16x8 fa[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = frag_tr(At, l, i, kk);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) mfma(f16, fa[i], w[kk][j], acc[i][j]);
      if (N > 96) __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Packed 16-bit values of the accumulator tiles 2 kk and 2 kk + 1 of one column (rows 4 kg .. + 3 of each) as such an operand:
  // lane group kg needs rows 8 kg .. + 7 of the 32, which two swaps of lane groups bring it.
  auto to_cols = [](const uint2& t0, const uint2& t1) {
    const auto a = __builtin_amdgcn_permlane32_swap(t0.x, t1.x, false, false), b = __builtin_amdgcn_permlane32_swap(t0.y, t1.y, false, false);
    const auto x = __builtin_amdgcn_permlane16_swap(a[0], a[1], false, false), y = __builtin_amdgcn_permlane16_swap(b[0], b[1], false, false);
    return __builtin_bit_cast(f16x8, make_uint4(x[0], y[0], x[1], y[1]));
  };
  constexpr std::true_type kF16{};
  constexpr std::false_type kBF16{};
  // Element r of acc[i][j]: row m = 16 i + 4 kg + r, column n = nb + 16 j + col.  fn(i, j, m of r = 0, n) over the block.
  auto each = [&](auto&& fn) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) fn(i, j, 16 * i + 4 * kg, nb + 16 * j + col);
      if (TM * TN > 8) __builtin_amdgcn_sched_barrier(0);   // (bounds what the scheduler keeps live: without it width 128 spills)
    }
  };
  // The head's matrices in memory through buffer instructions with 32-bit offsets: rows past the head lie past the descriptor's
  // range, and lanes or tiles whose columns do not exist get an offset there; such a load returns zero and such a store does
  // nothing, so that the loads and stores of all tiles are in flight together (behind a branch per tile each waited for its
  // own).  The pitch comes from pitch() each time: offsets shared by all of these would have to stay live through the steps.
  constexpr uint32_t kOob = 0x80000000u;
  auto rsrc = [&](const void* p, int elem) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(p) + hoff * elem, 0, dh * dh * elem, 0x00020000);
  };
  auto pitch = [&]() {
    int p = dh;
    asm volatile("" : "+s"(p));
    return (uint32_t)p;
  };
  // fp32 blocks, natural layout: fn(i, j, r, offset) for row 16 i + 4 kg + r, column nb + 16 j + col
  auto each4 = [&](auto&& fn) {
    const uint32_t ld = 4u * pitch();
    uint32_t o[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) o[j] = nb + 16 * j < dh ? 4u * kg * ld + 4u * (uint32_t)(nb + 16 * j + col) : kOob;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) fn(i, j, r, o[j] + (uint32_t)(16 * i + r) * ld);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto load_block = [&](const float* p, Acc& v) {
    const auto b = rsrc(p, 4);
    each4([&](int i, int j, int r, uint32_t at) { v[i][j][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, at, 0, 0)); });
  };
  auto store_block = [&](float* p, const Acc& v) {
    const auto b = rsrc(p, 4);
    each4([&](int i, int j, int r, uint32_t at) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[i][j][r]), b, at, 0, 0); });
  };
  // a transposed 16-bit plane: value(i, j) gives the 4 packed values of row nb + 16 j + col, elements 16 i + 4 kg .. + 3
  auto store_plane = [&](bf16_bits* p, auto&& value) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const auto b = rsrc(p, 2);
    const uint32_t ld = 2u * pitch();
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const uint32_t k = 16 * i < dh ? 32u * i : kOob;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const uint2 t = value(i, j);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{t.x, t.y}, b, (uint32_t)(nb + 16 * j + col) * ld + 8u * kg + k, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // tile (i, j) transposed, packed: row n, K positions 16 i + 4 kg .. + 3 (8 bytes)
  auto store_tr = [&](unsigned char* dst, const Lanes& l, int i, int j, const uint2& t) {
    *reinterpret_cast<uint2*>(dst + 16 * j * ROWB + (l.put ^ (i << 5))) = t;
  };
  auto pack_f16 = [](const f32x4& a) { return make_uint2(f32x2_to_f16x2(a[0], a[1]), f32x2_to_f16x2(a[2], a[3])); };
  auto store_iterate = [&](unsigned char* dst, const Acc& acc) {
    const Lanes l = lanes();
    each([&](int i, int j, int, int) { store_tr(dst, l, i, j, pack_f16(acc[i][j])); });
  };
  // sum of one double per lane over the workgroup, known to every thread afterwards (a slot is used once)
  auto block_sum = [&](double v, int slot) {
    v = wave_sum_d(v);
    if (lane == 0) red[slot][wave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) t += red[slot][q];
    return t;
  };

  // word q of this head's batch statistics: L, rows, skipped, then its counters
  auto stat_at = [&](int q) { return q < 3 ? (int64_t)q * gridDim.x + h : (int64_t)(3 * gridDim.x) + (int64_t)h * (2 * kCountSlots) + q - 3; };
  Acc acc;
  if (st.stamp && h == 0 && tid == 0) store_for_host(st.stamp, (unsigned long long)wall_clock64());
  if (st.M) {
    // The start of the update in this launch as well (what the packing pass does on the general path):
    // X0 = (M + lambda tau R_prev) / alpha, tau = ||M||_F / sqrt(dh), alpha = ||M||_F (1 + lambda); lambda = 0 stands for the
    // limit at fp32 resolution, an empty M for R_prev itself.  ||M||_F^2 is the sum of the partial sums the reduction of the
    // token shares left, or is taken here.  Elements in the accumulators' layout, so that the two LDS operands are written
    // exactly as after a step.
    Acc prev;
    double f2 = 0.0, dot = 0.0;
    load_block(st.M, acc);
    load_block(st.R, prev);
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
        for (int r = 0; r < 4; ++r) {
          float m = acc[i][j][r];
          asm volatile("" : "+v"(m));   // (else its conversion above is kept: 64 doubles)
          dot += (double)m * (st.round_bf16 ? bf16_to_f32(f32_to_bf16(prev[i][j][r])) : prev[i][j][r]);
        }
      });
      dot = block_sum(dot, 1);
    }
    if (tid == 0) {
      const double l = st.rop_dot || !st.ldot ? dot : st.L[h];
      st.fro2_out[h] = f2;
      if (st.ldot) st.ldot[h] = l;   // kept before the statistics restart
      if constexpr (CLOSE) {         // (here, where the way to the host is covered by the steps)
        store_for_host(cl.host + 2 * gridDim.x + h, l);
        store_for_host(cl.host + 4 * gridDim.x + h, f2);
      }
    }
    if constexpr (CLOSE) {
      for (int q = tid; q < 3 + 2 * kCountSlots; q += NT) cl.stats_keep[stat_at(q)] = cl.stats[stat_at(q)];
    }
    if (st.R_keep) store_block(st.R_keep, prev);
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
    store_iterate(start, acc);
  } else {   // the start iterate is given as a plane
    for (int idx = tid; idx < N * (N / 8); idx += NT) {
      const int row = idx / (N / 8), chunk = idx % (N / 8);
      uint4 a = make_uint4(0u, 0u, 0u, 0u);
      if (row < dh && chunk * 8 < dh) a = *reinterpret_cast<const uint4*>(Xt0 + hoff + (int64_t)row * dh + chunk * 8);
      *reinterpret_cast<uint4*>(start + row * ROWB + ((chunk ^ swz(row)) << 4)) = a;
    }
  }
  __syncthreads();
  // One step in KB pairs of row tiles.  G(p): this wavefront's columns of G's tiles 2 p, 2 p + 1; conv(p): those as the fp16
  // operand W; A(p): what K block p adds to X'.  A wavefront has its SIMD to itself, so the latencies are covered here: the LDS
  // reads and conversions of one pair are dealt out over the MFMAs of another, one G ahead of the A they feed.  Fragments are
  // read into the registers that the MFMAs in front have finished with (two sets of each would not leave the accumulators their
  // half of the registers).
  f32x4 eye;   // the identity on a diagonal tile
#pragma unroll
  for (int r = 0; r < 4; ++r) eye[r] = 4 * kg + r == col ? 1.0f : 0.0f;
  auto step = [&](int k, auto last, unsigned char* from, unsigned char* to) {
    constexpr bool LAST = decltype(last)::value;
    constexpr int NG = 2 * TN * KB, NA = TM * TN;   // MFMAs of G(p) and of A(p)
    constexpr int NX = TM > 6 ? TM / 2 : TM;        // fragments of X held: row tile i in fx[i % NX]
    static_assert(TM % NX == 0, "the next block's fragments take the same places");
    const float ci = sched.a[k], cg = sched.b[k];
    f16x8 fb[KB][TN], fa[KB][2], fx[NX], w[2][TN];
    f32x4 g[2][2][TN];
    uint2 t[2][TN];
    const Lanes l = lanes();
    auto read_fa = [&](int p, int kk, int q) { fa[kk][q] = frag(from, l.row, 16 * (2 * p + q), kk); };
    auto read_fx = [&](int p, int i) { fx[i % NX] = frag_tr(from, l, i, p); };
    auto conv = [&](int p, int n) {   // n < 2 TN: one tile; then one column tile's operand each
      if (n < 2 * TN) {
        const int q = n / TN, j = n % TN, i = 2 * p + q;
        const float on = 16 * i == nb + 16 * j ? ci : 0.0f;   // (wave-uniform)
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          // (as the general path's epilogue rounds it, the product first; heads of width 128: the identity's part first)
          v[r] = DH128 ? fmaf(cg, g[p & 1][q][j][r], eye[r] * on) : fmaf(on, eye[r], cg * g[p & 1][q][j][r]);
        t[q][j] = pack_f16(v);
      } else {
        const int j = n - 2 * TN;
        w[p & 1][j] = to_cols(t[0][j], t[1][j]);
      }
    };
    auto G = [&](int p, auto&& side) {
#pragma unroll
      for (int m = 0; m < NG; ++m) {
        const int kk = m / (2 * TN), q = m / TN % 2, j = m % TN;
        if (kk == 0) g[p & 1][q][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        mfma(kF16, fa[kk][q], fb[kk][j], g[p & 1][q][j]);
        side(m);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto A = [&](int p, auto&& side) {
#pragma unroll
      for (int m = 0; m < NA; ++m) {
        const int i = m / TN, j = m % TN;
        if (p == 0) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        mfma(kF16, fx[i % NX], w[p & 1][j], acc[i][j]);
        side(m);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // conv(p), dealt out over `of` MFMAs behind the results' latency
    auto conv_over = [&](int p, int m, int of) {
#pragma unroll
      for (int n = 0; n < 3 * TN; ++n) {
        const int lead = of > 8 ? 3 : 1;
        if (lead + n * (of - lead) / (3 * TN) == m) conv(p, n);
      }
    };
#pragma unroll
    for (int kk = 0; kk < KB; ++kk) {
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[kk][j] = frag(from, l.own, 16 * j, kk);
      read_fa(0, kk, 0);
      read_fa(0, kk, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    G(0, [&](int m) {
      if (KB > 1 && m % TN == TN - 1) read_fa(1, m / (2 * TN), m / TN % 2);
      if (KB == 1 && m < NX) read_fx(0, m);
    });
    if (KB == 1) {
#pragma unroll
      for (int n = 0; n < 3 * TN; ++n) conv(0, n);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int p = 0; p < KB; ++p) {
      if (p + 1 < KB)
        G(p + 1, [&](int m) {
#pragma unroll
          for (int i = 0; i < NX; ++i)
            if (i * NG / NX == m) read_fx(p, i);
          conv_over(p, m, NG);
        });
      A(p, [&](int m) {
        if (p + 2 < KB) {
#pragma unroll
          for (int n = 0; n < 2 * KB; ++n)
            if (n * NA / (2 * KB) == m) read_fa(p + 2, n / 2, n % 2);
        }
        if (m % TN == TN - 1) {
          const int i = m / TN + NX;
          if (i < TM) read_fx(p, i);
          else if (p + 2 == KB && i - TM < NX) read_fx(p + 1, i - TM);
        }
        if (p + 2 == KB) conv_over(p + 1, m, NA);
        if (p + 1 == KB && !LAST) {   // finished tiles into the other buffer
          if (m >= 2 * TN) store_tr(to, l, m / TN - 2, m % TN, pack_f16(acc[m / TN - 2][m % TN]));
        }
      });
    }
    if constexpr (!LAST) {
#pragma unroll
      for (int m = NA - 2 * TN; m < NA; ++m) store_tr(to, l, m / TN, m % TN, pack_f16(acc[m / TN][m % TN]));
      __syncthreads();                              // the step's one barrier: it writes where nobody reads any more
    }
  };
  int k = 0;
  if (!(sched.nsteps & 1)) step(k++, std::false_type{}, buf1, buf0);
  for (; k + 1 < sched.nsteps; k += 2) {
    step(k, std::false_type{}, buf0, buf1);
    step(k + 1, std::false_type{}, buf1, buf0);
  }
  step(k, std::true_type{}, buf0, buf1);   // X' stays in the accumulators

  // Hand-over to the closing iterations: the result rounded to bf16 like every step's, and exactly that value as fp32 X, as one
  // transposed plane and as one natural plane: the closing Gram matrix is then exact with one plane product.
  auto rounded = [](f32x4& a) {   // the packed bf16 values; a becomes exactly those
    const uint2 t = make_uint2(f32x2_to_bf16x2(a[0], a[1]), f32x2_to_bf16x2(a[2], a[3]));
    a = f32x4{__uint_as_float(t.x << 16), __uint_as_float(t.x & 0xffff0000u), __uint_as_float(t.y << 16), __uint_as_float(t.y & 0xffff0000u)};
    return t;
  };
  unsigned char* const sX = buf1;    // X^T, bf16
  const Lanes lx = lanes();
  store_plane(Pt, [&](int i, int j) {
    const uint2 hi = rounded(acc[i][j]);
    store_tr(sX, lx, i, j, hi);
    return hi;
  });
  store_block(X32, acc);
  __syncthreads();   // X^T is there, and every wavefront has finished the last step's reads of the old iterate
  {   // the natural plane: a transposing read gives 8 values of a row
    const auto rn = rsrc(Pn, 2);
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    for (int q = wave; q < TM * KB; q += NW) {
      const int i = q / KB, kk = q % KB;
      const bool in = 16 * i < dh && 32 * kk + 8 * kg < dh;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, frag_tr(sX, lx, i, kk)), rn,
                                             in ? (uint32_t)((16 * i + col) * dh + 32 * kk + 8 * kg) * 2u : kOob, 0, 0);
    }
  }

  if constexpr (CLOSE) {
    // ---- the closing step of the update in the same launch (Sec. 3.3; the general path's sequence of Gram matrix, D^2,
    // correction product and finishing pass, with the same operand planes): D = (I - X^T X)/2 from the exact bf16 iterate,
    // X <- X + X (D + 1.5 D^2) with the correction as two bf16 planes, then R, the rotate operand R^T and <R, M>.
    // The step is taken only if this head's residual allows the quintic form (cl.res_max); otherwise the head reports
    // its residual and a negative ||D^2||_F^2, which says that it did not, and the host continues on the general path from the
    // hand-over state written above.
    unsigned char* const sD = buf0;    // first plane of D (symmetric)
    // G = X^T X (products of bf16 values are exact in fp32), D = (I - G) / 2, ||I - G||_F^2
    Acc dm;
    zero(dm);
    product(kBF16, sX, sX, dm);
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
    auto report = [&](double sq2) {
      if (isfinite(res2))
        for (int q = tid; q < 3 + 2 * kCountSlots; q += NT) cl.stats[stat_at(q)] = 0;
      if (tid == 0) {
        store_for_host(cl.host + h, res2);
        store_for_host(cl.host + gridDim.x + h, sq2);
        if (h == 0 && *cl.nonfinite) {
          store_for_host(cl.host_nonfinite, 1);
          if (isfinite(res2)) *cl.nonfinite = 0;
        }
        store_for_host(cl.host_stamps + h, (unsigned long long)wall_clock64());
      }
    };
    if (!(res2 <= (double)cl.res_max * cl.res_max)) {   // (also a non-finite residual)
      report(-1.0);
      return;
    }
    const Lanes ld = lanes();
    each([&](int i, int j, int, int) {
      f32x4 d0 = dm[i][j];
      store_tr(sD, ld, i, j, rounded(d0));
    });
    __syncthreads();
    // D^2 from the first plane (second-order small: one plane is ample), ||D^2||_F^2, the correction D + 1.5 D^2
    Acc sq;
    zero(sq);
    product(kBF16, sD, sD, sq);
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
    const double sq2 = block_sum(part, 3);
    // the two planes of the correction, this wavefront's columns (the matrix is symmetric)
    Cols c0, c1;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int kk = 0; kk < KB; ++kk) {
        uint2 t0[2], t1[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          f32x4 hi = dm[2 * kk + q][j];
          t0[q] = rounded(hi);
          f32x4 lo = dm[2 * kk + q][j] - hi;
          t1[q] = rounded(lo);
        }
        c0[kk][j] = to_cols(t0[0], t0[1]);
        c1[kk][j] = to_cols(t1[0], t1[1]);
      }
    // X <- X + X (W0 + W1).  The small correction is summed on its own and the iterate added once at the end: with the
    // iterate as the accumulators' start every MFMA would round at the iterate's magnitude, and the orthogonality of the
    // result was measured above the bound that holds for the general path's order.
    zero(sq);
    product_tr(kBF16, sX, DH128 ? c0 : c1, sq);   // (the general path's order: smaller plane first)
    product_tr(kBF16, sX, DH128 ? c1 : c0, sq);
    // R, the rotate operand R^T (bf16 planes, [n][m]: packed rows of the transposed matrix) and <R, M>
    load_block(cl.M, dm);
    const Lanes le = lanes();
    each([&](int i, int j, int, int) {
      const uint2 x = *reinterpret_cast<const uint2*>(sX + 16 * j * ROWB + (le.put ^ (i << 5)));
      sq[i][j] += f32x4{__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xffff0000u), __uint_as_float(x.y << 16), __uint_as_float(x.y & 0xffff0000u)};
    });
    store_block(cl.R, sq);
    part = 0.0;
    each([&](int i, int j, int, int) {
      float p32 = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) p32 += sq[i][j][r] * dm[i][j][r];
      part += (double)p32;
    });
    for (int p = 0; p < cl.rop_planes; ++p)   // sq: what the planes before leave over
      store_plane(cl.RopT + p * cl.rop_plane, [&](int i, int j) {
        f32x4 hi = sq[i][j];
        const uint2 t = rounded(hi);
        sq[i][j] -= hi;
        return t;
      });
    const double inner = block_sum(part, 4);
    if (tid == 0) store_for_host(cl.host + 3 * gridDim.x + h, inner);
    report(sq2);
  }
}

template <int N, int NW, bool CLOSE, bool DH128>
hipError_t launch_one(const bf16_bits* Xt0, int heads, int dh, const PolarSchedule& sched, float* X32, bf16_bits* Pn, bf16_bits* Pt,
                      const HeadPolarClose& cl, const HeadPolarStart& st, hipStream_t s) {
  constexpr int smem = 2 * N * 256;
  static PerDeviceOnce configured;
  auto kern = k_head_polar<N, NW, CLOSE, DH128>;
  hipError_t e = configured.run([&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(heads), dim3(64 * NW), smem, s, Xt0, dh, sched, X32, Pn, Pt, cl, st);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_head_polar(const bf16_bits* Xt0, int heads, int dh, const PolarSchedule& sched, float* X32, bf16_bits* Pn, bf16_bits* Pt,
                             const HeadPolarClose* close, const HeadPolarStart* start, hipStream_t s) {
  if (heads < 1 || dh < 16 || dh > kHeadPolarMaxDh || (dh & 15) || sched.nsteps < 1 || sched.nsteps > kPolarScheduleMax) return hipErrorInvalidValue;
  if (close && (!start || !close->R || !close->RopT || !close->M || !close->host || !close->host_stamps || !close->stats || !close->stats_keep ||
                !close->nonfinite || !close->host_nonfinite || close->rop_planes < 1))
    return hipErrorInvalidValue;
  if (start && (!start->M || !start->R || (start->nparts > 0 && !start->fro2_parts) || !start->fro2_out ||
                (start->ldot && !start->rop_dot && !start->L)))
    return hipErrorInvalidValue;
  if (!start && !Xt0) return hipErrorInvalidValue;
  const HeadPolarStart st = start ? *start : HeadPolarStart{};
  const HeadPolarClose cl = close ? *close : HeadPolarClose{};
  auto go = [&](auto n, auto nw, auto own) {
    constexpr int N = decltype(n)::value, NW = decltype(nw)::value;
    constexpr bool OWN = decltype(own)::value;
    return close ? launch_one<N, NW, true, OWN>(Xt0, heads, dh, sched, X32, Pn, Pt, cl, st, s)
                 : launch_one<N, NW, false, OWN>(Xt0, heads, dh, sched, X32, Pn, Pt, cl, st, s);
  };
  using std::integral_constant;
  constexpr std::false_type general{};
  if (dh <= 32) return go(integral_constant<int, 32>{}, integral_constant<int, 2>{}, general);
  if (dh <= 64) return go(integral_constant<int, 64>{}, integral_constant<int, 4>{}, general);
  if (dh <= 96) return go(integral_constant<int, 96>{}, integral_constant<int, 3>{}, general);
  if (dh < 128) return go(integral_constant<int, 128>{}, integral_constant<int, 4>{}, general);
  return go(integral_constant<int, 128>{}, integral_constant<int, 4>{}, std::true_type{});
}

}  // namespace conqur
