// bf16 MFMA "NT" GEMM with fused epilogues (see gemm_nt.h).
//
// Tiling: a workgroup of WGM x WGN wavefronts owns a BM x BN tile of the output; each
// 64-lane wavefront owns (BM/WGM) x (BN/WGN) as a grid of 16x16 MFMA tiles
// (v_mfma_f32_16x16x32_bf16 / _f16, fp32 accumulators).  4 wavefronts (1 per SIMD) in the
// tiles that run the polar products, 8 in 256 x 128, which mostly rotates: its launches are
// one round of short K loops, and the sign and row epilogues wait on memory and LDS as much
// as they work (2048 x 3072 x 3072 rotated 42.0 us with 4 wavefronts, 40.0 with 8; with corner
// signs and the transposed operand 45.7 and 40.8).
//
// These kernels are limited by power and by LDS reads, so both choices are about what a
// multiply-add costs besides the MFMA itself.  A 128 x 128 wavefront tile reads 128 KiB of
// LDS per K step of a 256 x 256 workgroup tile, 8 wavefronts of 128 x 64 read 192 KiB (1536
// of the 2048 cycles the MFMAs take); a 16x16x32 MFMA updates 4 accumulator registers per
// 8192 multiply-adds, a 32x32x16 one 16 per 16384.  Plain bf16 product, us (TFLOP/s), 8
// wavefronts and 32x32x16 -> 8 and 16x16x32 -> 4 and 16x16x32: 4096^3 107 (1280) -> 98 -> 96
// (1420); 8192^3 805 (1365) -> 784 -> 732 (1500); 4 wavefronts and 32x32x16: 110 and 820.
//
// Operand path: HBM/L2 -> LDS directly (buffer_load ... lds, 16 bytes per lane, no
// register staging), 2 or 3 LDS stages of 64 K-elements (what fits in 160 KiB), fragments
// double buffered in registers, one fence-free barrier per K step placed between MFMA groups.
//
// LDS layout: a tile row is 64 bf16 = 128 bytes = 8 chunks of 16 bytes; chunk c of row r
// sits at physical chunk c ^ ((r >> 1) & 7), which spreads any 16 consecutive rows of
// one logical chunk (what a ds_read_b128 quarter-wave touches) over all 64 banks:
// SQ_LDS_BANK_CONFLICT = 0 in the accumulate launch, whose epilogue leaves LDS alone (1.5 %
// of the LDS-active cycles where the staged sign epilogue is in the launch).
#include "gemm_nt.h"

#include <algorithm>
#include <type_traits>

namespace conqur {

namespace {

constexpr int BK = 64;      // K elements per pipeline stage (one LDS tile row = 128 bytes = 8 chunks of 16 bytes)

__device__ __forceinline__ int lds_off(int row, int chunk) {
  return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4);
}

// s_waitcnt vmcnt(N) only (gfx9 encoding: vmcnt = simm16[15:14]:[3:0], expcnt and lgkmcnt left at max).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// The same, and every LDS read this wavefront has issued has returned (lgkmcnt(0)).
template <int N>
__device__ __forceinline__ void wait_vmcnt_and_lds() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// Workgroup barrier without the release/acquire fence of __syncthreads(): the fence
// would drain every outstanding LDS-direct load (vmcnt(0)) and serialise the
// pipeline.  Ordering here is explicit: each wave waits for its own loads of the tile that
// is consumed next (vmcnt) and for its LDS reads of the current one (lgkmcnt).  The "memory" clobber keeps
// the compiler from moving LDS accesses across the barrier.
__device__ __forceinline__ void pipeline_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Forms of a conversion and of a constant that the compiler cannot merge with an earlier identical one.  The epilogues walk
// over up to 256 accumulators per lane several times (a plane in two layouts, several planes); merged, the walks' common
// values would have to stay live from one to the next, and the kernels spill hundreds of bytes per lane.
__device__ __forceinline__ uint32_t cvt_bf16x2_again(float lo, float hi) {
  uint32_t r;
  asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
  return r;
}
__device__ __forceinline__ float again(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

// K-tail / invalid-row loads are pointed past the end of the buffer descriptor, where
// the hardware returns zeros (also for loads whose destination is LDS).
constexpr uint32_t kOobOffset = 0x80000000u;

// a / b for 0 <= a < 2^30, by one multiplication: m = ceil(2^(31 + l) / b) with l = floor(log2 b), so that a m / 2^(31 + l) exceeds a / b by
// less than a / 2^(31 + l) < 1 / b.  (The division ahead of a kernel's first loads is the latency of the launch.)
struct Divisor { uint32_t b, m, l; };
inline Divisor divisor(int b) {
  uint32_t l = 0;
  while ((2u << l) <= (uint32_t)b) ++l;
  return Divisor{(uint32_t)b, (uint32_t)(((1ull << (31 + l)) + b - 1) / b), l};
}
__host__ __device__ inline int quotient(int a, const Divisor& d) { return (int)((uint32_t)(((uint64_t)(2u * (uint32_t)a) * d.m) >> 32) >> d.l); }

// The order of a launch's tiles.  Workgroups are dealt round-robin to the 8 XCDs (bid % 8), each with its own L2; every XCD
// takes a run of consecutive tiles (the first n % 8 of them one tile more), numbered
//   whole grids      in `bands` bands of tile rows of equal height (+- 1, the first ones higher), down the columns of one band after another;
//                    1: down the columns of the grid, tiles_m: along its rows
//   mirrored grids   (the tiles on and above the diagonal, tiles_m == tiles_n) the same in bands of `bands` rows; 0: tile rows r and T-1-r,
//                    which hold T + 1 tiles between them, after one another
// What the tiles that an XCD runs at a time read together is one panel per tile row and column they span: see order_of.
struct TileOrder {
  int tiles_m, tiles_n, bands;
  int high_tiles, high_rows;   // whole grids: tiles and rows of the higher bands
  Divisor high_band, high;     // ... tiles of such a band, its rows
  Divisor band, rows;          // ... of the others; mirrored grids, rows: `bands`, or T + 1
};

inline TileOrder tile_order(int tiles_m, int tiles_n, bool sym, int bands) {
  TileOrder o{tiles_m, tiles_n, bands, 0, 0, divisor(1), divisor(1), divisor(1), divisor(1)};
  if (sym) {
    o.rows = divisor(bands ? bands : tiles_m + 1);
  } else {
    const int h = tiles_m / bands, higher = tiles_m - h * bands;
    o.high_rows = higher * (h + 1);
    o.high_tiles = o.high_rows * tiles_n;
    o.high_band = divisor((h + 1) * tiles_n); o.high = divisor(h + 1);
    o.band = divisor(h * tiles_n); o.rows = divisor(h);
  }
  return o;
}

// The tile workgroup bid computes.
template <bool SYM>
__host__ __device__ inline void tile_of(int bid, const TileOrder& o, int* tm, int* tn) {
  const int T = o.tiles_m, n = SYM ? T * (T + 1) / 2 : T * o.tiles_n;
  const int x = bid & 7, rest = n & 7;
  int at = x * (n >> 3) + (x < rest ? x : rest) + (bid >> 3);
  if constexpr (!SYM) {
    const bool high = at < o.high_tiles;
    const Divisor in_band = high ? o.high_band : o.band, rows = high ? o.high : o.rows;
    if (!high) at -= o.high_tiles;
    const int band = quotient(at, in_band);
    at -= band * (int)in_band.b;
    *tn = quotient(at, rows);
    *tm = (high ? 0 : o.high_rows) + band * (int)rows.b + at - *tn * (int)rows.b;
  } else if (o.bands == 0) {
    const int pair = quotient(at, o.rows), within = at - pair * (T + 1);
    const bool first = within < T - pair;
    *tm = first ? pair : T - 1 - pair;
    *tn = first ? pair + within : within - 1;
  } else {
    int r0 = 0, h;
    for (;; r0 += h) {
      h = o.bands < T - r0 ? o.bands : T - r0;
      const int in_band = h * (T - r0) - h * (h - 1) / 2;
      if (at < in_band) break;
      at -= in_band;
    }
    int c = 0;   // the band's columns: 1, 2 .. h tiles (its triangle), then h each
    while (c < h && at > c) { at -= c + 1; ++c; }
    const int right = c < h ? 0 : quotient(at, o.rows);   // (h == bands: a lower band, the last one, is all triangle)
    *tm = r0 + at - right * h;
    *tn = r0 + c + right;
  }
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE, int EPI, bool F16, bool SYM>
__global__ void __launch_bounds__(64 * WGM * WGN) gemm_nt_kernel(const GemmArgs g, const TileOrder order) {
  static_assert(!SYM || (BM == BN && (EPI == EPI_GRAMW || EPI == EPI_SQUARE || EPI == EPI_FRO2)),
                "mirrored tiles: square tiles, symmetric results");
  constexpr int NW = WGM * WGN;                 // wavefronts per workgroup
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  constexpr int NLA = BM / 8, NLB = BN / 8;     // wave-wide 1 KiB loads per stage (8 tile rows each)
  constexpr int QA = NLA / NW, QB = NLB / NW;   // ... per wavefront
  static_assert(NLA % NW == 0 && NLB % NW == 0 && WM % 16 == 0 && WN % 16 == 0, "tile shape");
  constexpr int STAGE = (BM + BN) * 128;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // Optional clock probe (g.clk != null): wall-clock ticks (100 MHz) of the prologue, main loop and epilogue
  // of this workgroup and the shader-clock cycles of the main loop, from which the host derives the clock
  // frequency the chip sustained while the MFMAs ran.
  const unsigned long long pr_w0 = g.clk ? wall_clock64() : 0;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int kg = lane >> 4, col = lane & 15;    // operand fragments: row (or column) col, K elements 8 kg .. 8 kg + 7 of 32

  int tm, tn;
  tile_of<SYM>(blockIdx.x, order, &tm, &tn);
  [[maybe_unused]] const int tiles_m = order.tiles_m, ntiles = order.tiles_m * order.tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;
  const int bz = blockIdx.z;
  const bf16_bits* Ab = g.A + (int64_t)bz * g.batchA;
  const bf16_bits* Bb = g.B + (int64_t)bz * g.batchB;

  // Global -> LDS without passing through registers: each buffer_load ... lds moves
  // 64 lanes x 16 bytes = 8 tile rows into 1 KiB of LDS (lane L lands at L*16).
  // Lane L therefore fetches the chunk that the swizzled layout stores at row L/8,
  // physical chunk L%8.  Rows past M (N) lie past the descriptor's range and read 0.
  const int lrow = lane >> 3, lpc = lane & 7;
  uint32_t offA[QA], offB[QB];
  int chunkA[QA], chunkB[QB];
#pragma unroll
  for (int q = 0; q < QA; ++q) {
    const int row = (q * NW + wave) * 8 + lrow;
    chunkA[q] = lpc ^ ((row >> 1) & 7);
    offA[q] = (m0 + row < g.M) ? (uint32_t)(((int64_t)(m0 + row) * g.lda + chunkA[q] * 8) * 2) : kOobOffset;
  }
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int row = (q * NW + wave) * 8 + lrow;
    chunkB[q] = lpc ^ ((row >> 1) & 7);
    offB[q] = (n0 + row < g.N) ? (uint32_t)(((int64_t)(n0 + row) * g.ldb + chunkB[q] * 8) * 2) : kOobOffset;
  }
  const uint32_t recA = (uint32_t)((((int64_t)g.M - 1) * g.lda + BK) * 2);
  const uint32_t recB = (uint32_t)((((int64_t)g.N - 1) * g.ldb + BK) * 2);
  const int nkb = (g.K + BK - 1) / BK;
  const int nit = nkb * g.nseg;
  // Epilogues of the largest tile whose registers need help (see where the accumulators are pinned): a guard around the loop
  // costs them a second set of accumulators at its exit.  The others spill nothing either way, and the two that rotate or
  // accumulate lose up to 5 % without it (11008 x 4096 x 4096: 297 us instead of 282).
  constexpr bool TIGHT = (BM / WGM) * (BN / WGN) >= 128 * 128 && EPI != EPI_ACT && EPI != EPI_F32;
  if constexpr (TIGHT) __builtin_assume(nit > 0);
  const bool ktail = (g.K % BK) != 0;
  // offsets for the last, partial K step of a segment: chunks past K read zeros
  uint32_t offAt[QA], offBt[QB];
  {
    const int kleft = g.K - (nkb - 1) * BK;
#pragma unroll
    for (int q = 0; q < QA; ++q) offAt[q] = (chunkA[q] * 8 < kleft) ? offA[q] : kOobOffset;
#pragma unroll
    for (int q = 0; q < QB; ++q) offBt[q] = (chunkB[q] * 8 < kleft) ? offB[q] : kOobOffset;
  }

  // Issue state: the next tile to fetch is K step is_kb of segment is_s; its operand
  // pointers advance incrementally (wave-uniform, scalar registers).
  int is_s = 0, is_kb = 0;
  const bf16_bits* pa = Ab + g.a_seg[0];
  const bf16_bits* pb = Bb + g.b_seg[0];
  __amdgpu_buffer_rsrc_t ra, rb;
  bool tail = false;
  auto issue_prep = [&]() {
    // Past the last tile the pipeline keeps issuing (so that every step has the same
    // number of loads in flight and needs no branches); those loads get an empty
    // descriptor range, fetch nothing and write zeros to a stage nobody reads again.
    const bool real = is_s < g.nseg;
    ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_bits*>(pa), 0, real ? recA : 0u, 0x00020000);
    rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_bits*>(pb), 0, real ? recB : 0u, 0x00020000);
    tail = ktail && is_kb == nkb - 1;
    if (++is_kb == nkb) {
      is_kb = 0;
      ++is_s;
      const int sc = is_s < g.nseg ? is_s : g.nseg - 1;
      pa = Ab + g.a_seg[sc];
      pb = Bb + g.b_seg[sc];
    } else {
      pa += BK; pb += BK;
    }
  };
  auto issue_one = [&](int q, int stage) {   // load q of LPT of the prepared tile
    unsigned char* sa = smem + stage * STAGE;
    if (q < QA) {
      const uint32_t off = tail ? offAt[q] : offA[q];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(sa + (q * NW + wave) * 1024), 16,
                                               off, 0, 0, 0);
    } else {
      const int qb = q - QA;
      const uint32_t off = tail ? offBt[qb] : offB[qb];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (__attribute__((address_space(3))) void*)(sa + BM * 128 + (qb * NW + wave) * 1024),
                                               16, off, 0, 0, 0);
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;

  // Software pipeline.  LDS holds NSTAGE tiles; tile t lives in stage t % NSTAGE.
  // Operand fragments are double buffered in registers: while the MFMAs of K-substep
  // kk run, the fragments of substep kk+1 are read from LDS, spread over the substep (one
  // read per 4 MFMAs for the largest tile), so that they issue in the MFMAs' shadow.  The
  // step's only synchronisation sits in the middle of its last substep: wait for this
  // wave's loads of the next tile (vmcnt counts outstanding loads, which retire in order),
  // barrier (now every wave's part of the next tile is visible and every wave has finished
  // reading the current stage), refill the current stage with tile it+NSTAGE, read the
  // first fragments of the next tile, and cover that latency with the second half of the
  // substep's MFMAs.
  constexpr int LPT = QA + QB;   // loads per thread per tile
  constexpr int KS = BK / 32;    // MFMA K-substeps per tile
  constexpr int NMF = TM * TN, HALF = NMF / 2, NR = TM + TN;
  constexpr int RS = NMF / NR > 1 ? NMF / NR : 1;       // MFMAs between two fragment reads of a full substep
  constexpr int RH = HALF / NR > 1 ? HALF / NR : 1;     // ... of the half substep behind the barrier
  constexpr int R0 = NR > HALF ? NR - HALF : 0;         // reads issued ahead of that half (small tiles: more reads than MFMAs)
  constexpr int LQ2 = LPT / 2, LQ1 = LPT - LQ2;         // a tile's loads: LQ2 behind the barrier, LQ1 in the next step's first substep
  constexpr int S2 = HALF / LQ2 > 1 ? HALF / LQ2 : 1;   // ... S2 and S1 MFMAs apart (early in the step: what is issued late
  constexpr int S1 = NMF / LQ1 > 4 ? 4 : (NMF / LQ1 > 1 ? NMF / LQ1 : 1);   // has less time to land before the next barrier)
  static_assert(KS == 2, "fragment double buffering: the two substeps of a step take one buffer each");
  static_assert(LQ2 * S2 <= HALF + S2 - 1 && LQ1 * S1 <= NMF + S1 - 1 && NR <= NMF, "every load and read has its MFMA");
  bf16x8 fa[2][TM], fb[2][TN];

  auto read_frag = [&](int buf, int r, const unsigned char* sa, int kk) {
    // read number r of a substep, in the order the MFMAs need them: a0, b0..b(TN-1), a1..a(TM-1)
    const unsigned char* sb = sa + BM * 128;
    if (r == 0) fa[buf][0] = *reinterpret_cast<const bf16x8*>(sa + lds_off(wm * WM + col, kk * 4 + kg));
    else if (r <= TN) fb[buf][r - 1] = *reinterpret_cast<const bf16x8*>(sb + lds_off(wn * WN + (r - 1) * 16 + col, kk * 4 + kg));
    else fa[buf][r - TN] = *reinterpret_cast<const bf16x8*>(sa + lds_off(wm * WM + (r - TN) * 16 + col, kk * 4 + kg));
  };
  auto mfma = [&](int buf, int m) {
    const int i = m / TN, j = m % TN;
    if constexpr (F16)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, fa[buf][i]), __builtin_bit_cast(f16x8, fb[buf][j]),
                                                         acc[i][j], 0, 0, 0);
    else
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
  };

#pragma unroll
  for (int p = 0; p < NSTAGE; ++p) {
    issue_prep();
#pragma unroll
    for (int q = 0; q < LPT; ++q) issue_one(q, p);
  }
  wait_vmcnt<(NSTAGE - 1) * LPT>();   // tile 0 has landed
  pipeline_barrier();
#pragma unroll
  for (int r = 0; r < NR; ++r) read_frag(0, r, smem, 0);

  const unsigned long long pr_w1 = g.clk ? wall_clock64() : 0, pr_c1 = g.clk ? clock64() : 0;
  int stage = 0;   // it % NSTAGE
  for (int it = 0; it < nit; ++it) {
    const int prev_stage = stage == 0 ? NSTAGE - 1 : stage - 1, next_stage = stage == NSTAGE - 1 ? 0 : stage + 1;
    const unsigned char* sa = smem + stage * STAGE;
    // first substep
#pragma unroll
    for (int m = 0; m < NMF; ++m) {
      mfma(0, m);
      if (m % RS == 0 && m / RS < NR) read_frag(1, m / RS, sa, 1);
      // the loads of tile it-1+NSTAGE that were left over behind the previous step's barrier
      if (it > 0 && m % S1 == S1 / 2 && m / S1 < LQ1) issue_one(LQ2 + m / S1, prev_stage);
      __builtin_amdgcn_sched_barrier(0);
    }
    // last substep
    issue_prep();   // tile it+NSTAGE refills the stage being consumed; scalar work, hidden behind the MFMAs
#pragma unroll
    for (int m = 0; m < HALF; ++m) mfma(1, m);
    __builtin_amdgcn_sched_barrier(0);
    // tiles up to it+NSTAGE-1 have been issued; all but the newest NSTAGE-2 have landed => tile it+1 is in LDS.  And this
    // wavefront's last fragment reads of the current tile have returned: behind the barrier the other wavefronts refill its
    // stage, and a load that fetches nothing (padding steps, the K tail) writes its zeros within the time a read takes.  (The
    // small tiles issue their last read 2 MFMAs ahead of this point; the large ones wait for nothing here.)
    wait_vmcnt_and_lds<(NSTAGE - 2) * LPT>();
    pipeline_barrier();
    const unsigned char* sn = smem + next_stage * STAGE;
#pragma unroll
    for (int r = 0; r < R0; ++r) read_frag(0, r, sn, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = HALF; m < NMF; ++m) {
      mfma(1, m);
      if ((m - HALF) % RH == 0 && R0 + (m - HALF) / RH < NR) read_frag(0, R0 + (m - HALF) / RH, sn, 0);
      if ((m - HALF) % S2 == S2 / 2 && (m - HALF) / S2 < LQ2) issue_one((m - HALF) / S2, stage);
      __builtin_amdgcn_sched_barrier(0);
    }
    stage = next_stage;
  }
  const unsigned long long pr_w2 = g.clk ? wall_clock64() : 0, pr_c2 = g.clk ? clock64() : 0;
  wait_vmcnt<0>();   // drain the padding loads before the epilogue reuses nothing of LDS (keeps exit clean)
  // The epilogues read accumulators in inline asm (cvt_bf16x2_again), for which the compiler keeps no distance from the MFMA
  // that writes them: 20 wait states, more than any MFMA needs, stand here once.
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  // The 256 accumulators of the largest tile fill one half of the registers.  Left to itself the compiler moves them over to
  // the other half for the epilogue's arithmetic, all at once, and spills what that half held.  Pinned to their half here,
  // they are read from it where they are used.  (The two sign epilogues that store a second array spill with the pin and
  // not without.)
  if constexpr (TIGHT && EPI != EPI_SIGN_XT && EPI != EPI_SIGN_ACT) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
  }

  // Accumulator element r of tile (i, j) is output row
  //   m = m0 + wm*WM + 16*i + 4*kg + r,   column n = n0 + wn*WN + 16*j + col.
  const int mw = m0 + wm * WM, nw = n0 + wn * WN;

  // Addressing of the epilogues that write matrices [row][ldc]: buffer instructions with 32-bit byte offsets, so that
  // a store is one instruction (no 64-bit address arithmetic per element) and bounds need no branches.  An offset at
  // or beyond the range of its array (rows past the last one; kOobOffset for lanes whose column, or whose rows in the
  // transposed layout, do not exist) makes a store a no-op and a load return zero.  With the per-element pointer
  // arithmetic and branches these epilogues ran 4000-5000 instructions per wavefront for 128 values per lane, and
  // instruction issue, not memory, was what they waited for.
  //   natural layout     [m][n]: byte offset nat{2,4}[j] + row_off(rows below the lane's first) * element size
  //   transposed layout  [n][m]: byte offset tr_off(j, rows below the lane's first), 4 consecutive m = 8 bytes
  [[maybe_unused]] const uint32_t ldc_u = (uint32_t)g.ldc;
  [[maybe_unused]] const uint32_t nat_rows = (uint32_t)g.M * ldc_u, tr_rows = (uint32_t)g.N * ldc_u;   // elements
  [[maybe_unused]] const int mlim = g.M - (mw + 4 * kg);   // rows ml .. ml + 3 of this lane exist iff ml < mlim
  [[maybe_unused]] bool n_ok[TN];
  [[maybe_unused]] uint32_t nat2[TN], nat4[TN], tr2[TN];
  {
    const uint32_t lane_nat = (uint32_t)(mw + 4 * kg) * ldc_u + (uint32_t)(nw + col);
    const uint32_t lane_tr = (uint32_t)(nw + col) * ldc_u + (uint32_t)(mw + 4 * kg);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      n_ok[j] = nw + 16 * j + col < g.N;
      nat2[j] = n_ok[j] ? (lane_nat + 16u * j) * 2u : kOobOffset;
      nat4[j] = n_ok[j] ? (lane_nat + 16u * j) * 4u : kOobOffset;
      tr2[j] = (lane_tr + 16u * j * ldc_u) * 2u;   // columns n >= N are rows past the end of the transposed array
    }
  }
  [[maybe_unused]] auto row_off = [&](int ml) { return (uint32_t)ml * ldc_u; };
  [[maybe_unused]] auto tr_off = [&](int j, int ml) { return ml < mlim ? tr2[j] + 2u * (uint32_t)ml : kOobOffset; };
  [[maybe_unused]] auto out_rsrc = [](void* p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000); };
  [[maybe_unused]] auto in_rsrc = [](const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
  };
  [[maybe_unused]] auto ld32 = [](__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  };
  [[maybe_unused]] auto ld64 = [](__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  };
  [[maybe_unused]] auto st32 = [](__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, 0);
  };
  [[maybe_unused]] auto st64 = [](__amdgpu_buffer_rsrc_t r, uint32_t off, const uint2& t) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = {t.x, t.y};
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
  };
  // the 4 packed 16-bit values of t to rows 0 .. 3 below byte offset off of a natural-layout plane
  [[maybe_unused]] auto st_rows4 = [&](__amdgpu_buffer_rsrc_t r, uint32_t off, const uint2& t) {
    const uint32_t rb = 2u * ldc_u;
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)t.x, r, off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(t.x >> 16), r, off + rb, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)t.y, r, off + 2u * rb, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(t.y >> 16), r, off + 3u * rb, 0, 0);
  };
  // Large tiles write their matrices through LDS: each wavefront lays its block out in its own slice of the (now idle)
  // stage memory and stores whole rows of it, 16 bytes per lane.  Straight from the accumulators a natural-layout store
  // instruction writes four rows' segments of 16 values and the L2s see every 128-byte line in four pieces (two in a
  // transposed layout).  Both bf16 layouts of a 4096^3 product: 101 us straight, 97 staged; of an 8192^3 one 785 and 726.
  // A 64 x 64 tile, whose launches are bound by latency, has 4 accumulators per lane and layout and stores them directly.
  constexpr bool STAGED = BM >= 128;
  constexpr int SLICE = NSTAGE * STAGE / NW;
  [[maybe_unused]] unsigned char* const slice = smem + wave * SLICE;
  // Rows staged at a time: a row is padded by 16 bytes, which spreads the accumulators' 4 rows (2- and 4-byte writes) and 16
  // columns (8-byte writes) over the banks.
  [[maybe_unused]] constexpr auto pass_rows = [](int rows, int pitch) constexpr { while (rows * pitch > SLICE) rows /= 2; return rows; };
  [[maybe_unused]] auto st128 = [](__amdgpu_buffer_rsrc_t r, uint32_t off, const uint4& t) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = {t.x, t.y, t.z, t.w};
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
  };
  [[maybe_unused]] auto stage_begin = [&]() {
    if constexpr (STAGED) __syncthreads();   // every wavefront has finished reading operand tiles, its loads have landed
  };
  // 16-bit plane in the natural layout: row m of the block at byte offset origin + m * 2 pitch; quad(i, j) gives the 4 packed
  // values of accumulator (i, j).  (Column counts are multiples of 8: a chunk of 8 is inside or outside as a whole.)
  [[maybe_unused]] auto store_nat16 = [&](__amdgpu_buffer_rsrc_t r, uint32_t origin, uint32_t pitch, auto&& quad) {
    constexpr int ROWB = WN * 2 + 16, ROWS = pass_rows(WM, ROWB), CPR = WN / 8;
    static_assert(ROWS % 16 == 0, "whole accumulator rows per pass");
#pragma unroll
    for (int h = 0; h < WM / ROWS; ++h) {
#pragma unroll
      for (int i = 0; i < ROWS / 16; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const uint2 t = quad(h * (ROWS / 16) + i, j);
          unsigned char* d = slice + (16 * i + 4 * kg) * ROWB + (16 * j + col) * 2;
          *reinterpret_cast<unsigned short*>(d) = (unsigned short)t.x;
          *reinterpret_cast<unsigned short*>(d + ROWB) = (unsigned short)(t.x >> 16);
          *reinterpret_cast<unsigned short*>(d + 2 * ROWB) = (unsigned short)t.y;
          *reinterpret_cast<unsigned short*>(d + 3 * ROWB) = (unsigned short)(t.y >> 16);
        }
        __builtin_amdgcn_sched_barrier(0);   // (bounds what the scheduler keeps live: without these the kernels spill)
      }
#pragma unroll
      for (int q = 0; q < (ROWS * CPR + 63) / 64; ++q) {
        const int idx = q * 64 + lane, row = idx / CPR, c = idx % CPR;
        const uint4 v = *reinterpret_cast<const uint4*>(slice + row * ROWB + c * 16);   // (lanes past the last row read LDS nobody stores)
        st128(r, nw + 8 * c < g.N && ((ROWS * CPR) % 64 == 0 || row < ROWS) ? origin + ((uint32_t)(h * ROWS + row) * pitch + 8u * c) * 2u : kOobOffset, v);
        if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the same plane transposed, row n of the block at origin + n * 2 pitch
  [[maybe_unused]] auto store_tr16 = [&](__amdgpu_buffer_rsrc_t r, uint32_t origin, uint32_t pitch, auto&& quad) {
    constexpr int ROWB = WM * 2 + 16, ROWS = pass_rows(WN, ROWB), CPR = WM / 8;
    static_assert(ROWS % 16 == 0, "whole accumulator columns per pass");
#pragma unroll
    for (int h = 0; h < WN / ROWS; ++h) {
#pragma unroll
      for (int j = 0; j < ROWS / 16; ++j) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          *reinterpret_cast<uint2*>(slice + (16 * j + col) * ROWB + (16 * i + 4 * kg) * 2) = quad(i, h * (ROWS / 16) + j);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < (ROWS * CPR + 63) / 64; ++q) {
        const int idx = q * 64 + lane, row = idx / CPR, c = idx % CPR;
        const uint4 v = *reinterpret_cast<const uint4*>(slice + row * ROWB + c * 16);
        st128(r, mw + 8 * c < g.M && ((ROWS * CPR) % 64 == 0 || row < ROWS) ? origin + ((uint32_t)(h * ROWS + row) * pitch + 8u * c) * 2u : kOobOffset, v);
        if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // fp32 in the natural layout, straight from the accumulators (16 lanes write 64 contiguous bytes of a row; through LDS, which
  // holds a quarter of the block at a time, the 4096^2 M of the accumulate GEMM took 10 us instead of 6).  add: the array at
  // radd (same addressing) is added first, its loads one row of accumulators ahead of their use.
  [[maybe_unused]] auto store_f32 = [&](__amdgpu_buffer_rsrc_t r, auto add, __amdgpu_buffer_rsrc_t radd, auto&& val) {
#pragma clang fp contract(off)   // the scaled product is rounded before the sum, as a further batch always was
    constexpr bool ADD = decltype(add)::value;
    [[maybe_unused]] f32x4 more[2][ADD ? TN : 1];
    auto fetch = [&](int i) {
      if constexpr (ADD) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) more[i & 1][j][e] = ld32(radd, nat4[j] + row_off(16 * i + e) * 4u);
      }
    };
    fetch(0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i + 1 < TM) fetch(i + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f32x4 v = val(i, j);
        if constexpr (ADD) v += more[i & 1][j];
#pragma unroll
        for (int e = 0; e < 4; ++e) st32(r, nat4[j] + row_off(16 * i + e) * 4u, v[e]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // byte offsets of this wavefront's block in the [row][ldc] arrays, natural (2- and 4-byte elements) and transposed
  [[maybe_unused]] const uint32_t blk_nat = (uint32_t)mw * ldc_u + (uint32_t)nw, blk_tr = (uint32_t)nw * ldc_u + (uint32_t)mw;
  // Split plane p of the values val(i, j) (f32x4): fp16 or bf16 rounding for p = 0; what the planes before leave over, rounded
  // to bf16, for the next ones.
  [[maybe_unused]] auto split16 = [&](auto plane, f32x4 a) {
    constexpr int P = decltype(plane)::value;
    if constexpr (F16 && EPI != EPI_XLAST) {
      static_assert(P == 0, "fp16 operands: one plane");
      return make_uint2(f32x2_to_f16x2(a[0], a[1]), f32x2_to_f16x2(a[2], a[3]));
    } else {
      uint2 t = make_uint2(cvt_bf16x2_again(a[0], a[1]), cvt_bf16x2_again(a[2], a[3]));
#pragma unroll
      for (int p = 0; p < P; ++p) {
        a[0] -= __uint_as_float(t.x << 16); a[1] -= __uint_as_float(t.x & 0xffff0000u);
        a[2] -= __uint_as_float(t.y << 16); a[3] -= __uint_as_float(t.y & 0xffff0000u);
        t = make_uint2(cvt_bf16x2_again(a[0], a[1]), cvt_bf16x2_again(a[2], a[3]));
      }
      return t;
    }
  };
  [[maybe_unused]] auto acc_val = [&](int i, int j) { return acc[i][j]; };
  // split plane `plane` of val(i, j) in the natural layout (nat), the transposed one (tr), or both
  [[maybe_unused]] auto store_plane = [&](auto plane, auto&& val, __amdgpu_buffer_rsrc_t rn, bool nat, __amdgpu_buffer_rsrc_t rt, bool tr) {
    auto quad = [&](int i, int j) { return split16(plane, val(i, j)); };
    if constexpr (STAGED) {
      if (nat) store_nat16(rn, blk_nat * 2u, ldc_u, quad);
      if (tr) store_tr16(rt, blk_tr * 2u, ldc_u, quad);
    } else {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const uint2 t = quad(i, j);
          if (nat) st_rows4(rn, nat2[j] + row_off(16 * i) * 2u, t);
          if (tr) st64(rt, tr_off(j, 16 * i), t);
        }
    }
  };
  using Plane0 = std::integral_constant<int, 0>;
  using Plane1 = std::integral_constant<int, 1>;
  using Plane2 = std::integral_constant<int, 2>;

  // The accumulators as activations Y[m][n] (bf16 or fp32 by g.c_is_f32), row pitch `pitch`: the pitch is the caller's,
  // so the offsets are taken relative to the tile's first row (at most BM rows x pitch x 4 bytes, which the launcher
  // keeps below 2^31); rows past M lie beyond the range, columns past N are masked.  The staged form stores 16 bytes per
  // lane and needs rows aligned to them; a caller's Y need not be (conqur_rotate asks for its element size only).
  [[maybe_unused]] auto store_act = [&](void* base, int64_t pitch, int64_t batch_off) {
    const uint32_t pu = (uint32_t)pitch;
    const uint32_t rows = (uint32_t)(g.M - m0 < BM ? g.M - m0 : BM);
    const uint32_t lane_el = (uint32_t)(wm * WM + 4 * kg) * pu + (uint32_t)(nw + col);
    const uint32_t blk_el = (uint32_t)(wm * WM) * pu + (uint32_t)nw;
    const int64_t tile_el = (int64_t)bz * batch_off + (int64_t)m0 * pitch;
    if (g.c_is_f32) {
      float* const tile = reinterpret_cast<float*>(base) + tile_el;
      const auto r = out_rsrc(tile, rows * pu * 4u);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const uint32_t o = n_ok[j] ? (lane_el + 16u * j) * 4u : kOobOffset;
#pragma unroll
          for (int e = 0; e < 4; ++e) st32(r, o + (uint32_t)(16 * i + e) * pu * 4u, acc[i][j][e]);
        }
    } else {
      bf16_bits* const tile = reinterpret_cast<bf16_bits*>(base) + tile_el;
      const auto r = out_rsrc(tile, rows * pu * 2u);
      if (STAGED && (((uintptr_t)tile | (uintptr_t)(pu * 2u)) & 15) == 0) {
        if constexpr (STAGED) store_nat16(r, blk_el * 2u, pu, [&](int i, int j) { return split16(Plane0{}, acc[i][j]); });
        return;
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const uint32_t o = n_ok[j] ? (lane_el + 16u * j) * 2u : kOobOffset;
          const uint2 t = split16(Plane0{}, acc[i][j]);
          const uint32_t oq = o + (uint32_t)(16 * i) * pu * 2u, rb = 2u * pu;
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)t.x, r, oq, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(t.x >> 16), r, oq + rb, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)t.y, r, oq + 2u * rb, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(t.y >> 16), r, oq + 3u * rb, 0, 0);
        }
    }
  };

  if constexpr (EPI == EPI_SIGN || EPI == EPI_SIGN_ACT || EPI == EPI_SIGN_XT) {
    // (the accumulate product contracts over whole steps of BK tokens: every call writes them, none is left from another)
    static_assert(BM % BK == 0, "the tiles' rows cover St up to the next multiple of BK tokens");
    // St is the transpose of the accumulator tile.  Storing it straight from the registers gives every lane 8 bytes of
    // a different row (64 cache lines per store instruction); instead each wavefront transposes its WM x WN block
    // through its own slice of the (now idle) stage memory and stores whole 16-byte chunks, 8 or 16 lanes per row.
    bf16_bits* St = reinterpret_cast<bf16_bits*>(g.C) + (int64_t)bz * g.batchC;
    const uint32_t one = g.sign_f16 ? 0x3C00u : 0x3F80u;
    constexpr int CPR = WM / 8;                       // 16-byte chunks per staged row (one output column n, WM tokens)
    constexpr bool POW2 = (CPR & (CPR - 1)) == 0;     // ... XOR swizzled by the row, or rows padded by one chunk (WM = 96)
    constexpr int SROW = WM * 2 + (POW2 ? 0 : 16);
    static_assert(WN * SROW <= SLICE, "sign staging fits the wavefront's slice");
    auto sign_chunk = [](int r, int c) { return POW2 ? c ^ (r & (CPR - 1)) : c; };
    unsigned char* const stg = slice;
    // EPI_SIGN_XT: the block of A this wavefront transposes below, loaded now so that the sign staging covers the latency
    // (loaded ahead of the main loop instead, the prologue grows by what the epilogue saves)
    constexpr int XT_ITEMS = EPI == EPI_SIGN_XT ? (WM / 2) * (WN / 8) / 64 : 1;
    [[maybe_unused]] uint4 xt_a[XT_ITEMS], xt_b[XT_ITEMS];
    [[maybe_unused]] float xt_w0[XT_ITEMS], xt_w1[XT_ITEMS];
    if constexpr (EPI == EPI_SIGN_XT) {
      constexpr int CH = WN / 8;
      const bf16_bits* Xb = Ab + g.a_seg[0];
      const float* wrow = g.xt_w + (int64_t)bz * g.xt_ldw;
#pragma unroll
      for (int q = 0; q < XT_ITEMS; ++q) {
        const int item = q * 64 + lane, c = item % CH, p = item / CH;
        const int m = mw + 2 * p, k = nw + 8 * c;
        xt_a[q] = make_uint4(0u, 0u, 0u, 0u); xt_b[q] = xt_a[q];
        xt_w0[q] = 0.0f; xt_w1[q] = 0.0f;
        if (k < g.N) {
          if (m < g.M) { xt_a[q] = *reinterpret_cast<const uint4*>(Xb + (int64_t)m * g.lda + k); xt_w0[q] = wrow[m]; }
          if (m + 1 < g.M) { xt_b[q] = *reinterpret_cast<const uint4*>(Xb + (int64_t)(m + 1) * g.lda + k); xt_w1[q] = wrow[m + 1]; }
        }
      }
    }
    __syncthreads();                                  // every wavefront has finished reading operand tiles
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4& a = acc[i][j];
        uint2 v;  // +1 with the sign bit of each accumulator (sgn(+-0) = +1, so test >= 0)
        v.x = (a[0] >= 0.0f ? one : one | 0x8000u) | ((a[1] >= 0.0f ? one : one | 0x8000u) << 16);
        v.y = (a[2] >= 0.0f ? one : one | 0x8000u) | ((a[3] >= 0.0f ? one : one | 0x8000u) << 16);
        const int r = j * 16 + col, c = 2 * i + (kg >> 1);   // tokens 16 i + 4 kg .. + 3 of row r
        *reinterpret_cast<uint2*>(stg + r * SROW + (sign_chunk(r, c) << 4) + 8 * (kg & 1)) = v;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // the slice is private to the wavefront: its own LDS writes are visible to it after the wait the compiler inserts
#pragma unroll
    for (int it2 = 0; it2 < WN * CPR / 64; ++it2) {
      const int idx = it2 * 64 + lane, r = idx / CPR, c = idx % CPR;
      const int n = nw + r, m = mw + c * 8;
      const uint4 v = *reinterpret_cast<const uint4*>(stg + r * SROW + (sign_chunk(r, c) << 4));
      if (n < g.N && m < g.st_rows_valid) *reinterpret_cast<uint4*>(St + (int64_t)n * g.ldc + m) = v;
      if (it2 % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (EPI == EPI_SIGN_ACT) store_act(g.Yact, g.ldy, g.batchY);   // the rotated rows themselves, as EPI_ACT writes them
    if constexpr (EPI == EPI_SIGN_XT) {
      // The scaled, transposed fp16 copy of A's block under this wavefront's output block: tokens [mw, mw + WM) x
      // channels [nw, nw + WN).  A lane takes items (token pair p, 16-byte chunk c of 8 channels), chunk fastest so
      // that 8 lanes read 128 contiguous bytes of a row; the pair's two values of a channel go to the staging slice as
      // one 4-byte write (row = channel, position = token pair); 16-byte chunks of 8 tokens come back and are stored
      // like the signs.  The slice is this wavefront's own and LDS operations of one wavefront complete in order, so
      // no barrier separates this from the sign staging above.
      constexpr int PAIRS = WM / 2, CH = WN / 8;
      static_assert((PAIRS * CH) % 64 == 0, "whole wavefronts of items");
      const float* wrow = g.xt_w + (int64_t)bz * g.xt_ldw;
      bf16_bits* Xt = g.Xt + (int64_t)bz * g.batchC;
      auto phys = [](int r, int cc) { return POW2 ? cc ^ ((r ^ (r >> 3)) & (CPR - 1)) : cc; };
#pragma unroll
      for (int q = 0; q < PAIRS * CH / 64; ++q) {
        const int item = q * 64 + lane, c = item % CH, p = item / CH;
        const uint4 xa = xt_a[q], xb = xt_b[q];
        const float w0 = xt_w0[q], w1 = xt_w1[q];
        const uint32_t ua[4] = {xa.x, xa.y, xa.z, xa.w}, ub[4] = {xb.x, xb.y, xb.z, xb.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t ba = (e & 1) ? (ua[e >> 1] & 0xffff0000u) : (ua[e >> 1] << 16);
          const uint32_t bb = (e & 1) ? (ub[e >> 1] & 0xffff0000u) : (ub[e >> 1] << 16);
          // a skipped row has w = 0 and possibly Inf / NaN values: select, do not multiply
          const float fa = w0 != 0.0f ? __uint_as_float(ba) * w0 : 0.0f;
          const float fb = w1 != 0.0f ? __uint_as_float(bb) * w1 : 0.0f;
          const int r = c * 8 + e;
          *reinterpret_cast<uint32_t*>(stg + r * SROW + (phys(r, p >> 2) << 4) + (p & 3) * 4) = f32x2_to_f16x2(fa, fb);
        }
      }
#pragma unroll
      for (int it2 = 0; it2 < WN * CPR / 64; ++it2) {
        const int idx = it2 * 64 + lane, r = idx / CPR, cc = idx % CPR;
        const int n = nw + r, m = mw + cc * 8;
        const uint4 v = *reinterpret_cast<const uint4*>(stg + r * SROW + (phys(r, cc) << 4));
        if (n < g.N && m < g.st_rows_valid) *reinterpret_cast<uint4*>(Xt + (int64_t)n * g.ldc + m) = v;
      }
      if (tn == 0 && wn == 0) {   // one wavefront per 64 tokens of the tile row counts them
#pragma unroll
        for (int t0 = 0; t0 < WM; t0 += 64) {
          const int m = mw + t0 + lane;
          const bool in_block = t0 + lane < WM && m < g.M;
          const float wv = in_block ? wrow[m] : 0.0f;
          const unsigned long long in = __ballot(in_block && wv != 0.0f), out = __ballot(in_block && wv == 0.0f);
          if (lane == 0) {
            unsigned long long* slot = g.cnt + ((int64_t)bz * g.cnt_slots + (tm % g.cnt_slots)) * 2;
            if (in) atomicAdd(slot, (unsigned long long)__popcll(in));
            if (out) atomicAdd(slot + 1, (unsigned long long)__popcll(out));
          }
        }
      }
    }
  } else if constexpr (EPI == EPI_ACT) {
    stage_begin();
    store_act(g.C, g.ldc, g.batchC);
  } else if constexpr (EPI == EPI_F32) {
    const auto rC = out_rsrc(reinterpret_cast<float*>(g.C) + (int64_t)bz * g.batchC, nat_rows * 4u);
    auto val = [&](int i, int j) { return g.out_scale * acc[i][j]; };
    if (g.accumulate) store_f32(rC, std::true_type{}, rC, val);
    else store_f32(rC, std::false_type{}, rC, val);
  } else if constexpr (EPI == EPI_GRAMW) {
    const int64_t boff = (int64_t)bz * g.batchC;
    [[maybe_unused]] const bool mirror = SYM && tm != tn;   // this tile is also the transpose of tile (tn, tm)
    // The identity: of a 16 x 16 tile on the diagonal (a wave-uniform choice, `on`) the entries 4 kg + r == col.  One
    // multiply-add per entry whether the tile meets the diagonal or not: two versions of the walks cost more registers than
    // the largest tile has.
    auto on = [&](int i, int j) { return mw + 16 * i == nw + 16 * j ? 1.0f : 0.0f; };
    f32x4 eye;
#pragma unroll
    for (int r = 0; r < 4; ++r) eye[r] = 4 * kg + r == col ? 1.0f : 0.0f;
    auto val = [&](int i, int j) {
      const float cg = again(g.coef_g), ci = again(g.coef_i * on(i, j));
      f32x4 w;
#pragma unroll
      for (int r = 0; r < 4; ++r) w[r] = fmaf(ci, eye[r], cg * acc[i][j][r]);
      return w;
    };
    auto plane = [&](auto p) {
      const auto rP = out_rsrc(g.Pn + decltype(p)::value * g.plane_out + boff, nat_rows * 2u);
      const auto rM = out_rsrc(g.Pn + decltype(p)::value * g.plane_out + boff, mirror ? nat_rows * 2u : 0u);   // (a diagonal tile's mirror image: dropped)
      store_plane(p, val, rP, true, rM, SYM);
    };
    stage_begin();
    plane(Plane0{});
    if constexpr (!F16) {   // fp16 operands: the factor is one fp16 plane, and nobody asks for the residual
      if (g.np_out > 1) plane(Plane1{});
      if (g.np_out > 2) plane(Plane2{});
    }
    if (!F16 && g.resid_part) {
      double rsum = 0.0;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const float o = on(i, j);
          float part = 0.0f;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float d = fmaf(-o, eye[r], acc[i][j][r]);
            part += d * d;
          }
          rsum += (double)((n_ok[j] && 16 * i < mlim) ? part : 0.0f);   // rows 16 i .. + 3 of the lane's block (M is a multiple of 4)
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      rsum = wave_sum_d(rsum);
      if (lane == 0) {
        g.resid_part[((int64_t)bz * ntiles + tn * tiles_m + tm) * NW + wave] = rsum;
        if constexpr (SYM) {   // the mirrored tile's slot: the sum over all slots stays the sum over the whole matrix
          if (mirror) g.resid_part[((int64_t)bz * ntiles + tm * tiles_m + tn) * NW + wave] = rsum;
        }
      }
    }
  } else if constexpr (EPI == EPI_SQUARE) {
    const int64_t boff = (int64_t)bz * g.batchC;
    [[maybe_unused]] const bool mirror = SYM && tm != tn;
    const auto rA0 = in_rsrc(g.Padd + boff, nat_rows * 2u), rA1 = in_rsrc(g.Padd + g.plane_out + boff, nat_rows * 2u);
    double rsum = 0.0;   // sum of the squares of this wavefront's accumulators: ||D^2||_F^2 over the whole launch
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        float part = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) part += acc[i][j][r] * acc[i][j][r];
        rsum += (double)((n_ok[j] && 16 * i < mlim) ? part : 0.0f);
      }
    stage_begin();
    {   // D^2 itself
      const auto rSq = out_rsrc(g.Pacc + boff, nat_rows * 2u);
      store_plane(Plane0{}, acc_val, rSq, true, rSq, mirror);
    }
    // the accumulators become the entries of the correction; D is symmetric: its entries (m .. m + 3, n) are 4 consecutive ones
    // of row n
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const uint32_t off = tr_off(j, 16 * i);
        const uint2 d0 = ld64(rA0, off), d1 = ld64(rA1, off);
        acc[i][j][0] = fmaf(g.coef_g, acc[i][j][0], __uint_as_float(d0.x << 16)) + __uint_as_float(d1.x << 16);
        acc[i][j][1] = fmaf(g.coef_g, acc[i][j][1], __uint_as_float(d0.x & 0xffff0000u)) + __uint_as_float(d1.x & 0xffff0000u);
        acc[i][j][2] = fmaf(g.coef_g, acc[i][j][2], __uint_as_float(d0.y << 16)) + __uint_as_float(d1.y << 16);
        acc[i][j][3] = fmaf(g.coef_g, acc[i][j][3], __uint_as_float(d0.y & 0xffff0000u)) + __uint_as_float(d1.y & 0xffff0000u);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      const auto r0 = out_rsrc(g.Pn + boff, nat_rows * 2u), r1 = out_rsrc(g.Pn + g.plane_out + boff, nat_rows * 2u);
      store_plane(Plane0{}, acc_val, r0, true, r0, mirror);
      store_plane(Plane1{}, acc_val, r1, true, r1, mirror);
    }
    if (g.resid_part) {
      rsum = wave_sum_d(rsum);
      if (lane == 0) {
        g.resid_part[((int64_t)bz * ntiles + tn * tiles_m + tm) * NW + wave] = rsum;
        if constexpr (SYM) {   // a tile above the diagonal stands for its mirror image as well
          if (mirror) g.resid_part[((int64_t)bz * ntiles + tm * tiles_m + tn) * NW + wave] = rsum;
        }
      }
    }
  } else if constexpr (EPI == EPI_FRO2) {
    double rsum = 0.0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        float part = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = n_ok[j] && 16 * i + e < mlim;
          part += in ? acc[i][j][e] * acc[i][j][e] : 0.0f;
        }
        rsum += (double)part;
      }
    rsum = wave_sum_d(rsum);
    if (lane == 0) {
      g.resid_part[((int64_t)bz * ntiles + tn * tiles_m + tm) * NW + wave] = rsum;
      if constexpr (SYM) {   // a tile above the diagonal stands for its mirror image as well
        if (tm != tn) g.resid_part[((int64_t)bz * ntiles + tm * tiles_m + tn) * NW + wave] = rsum;
      }
    }
  } else if constexpr (EPI == EPI_XLAST) {
    const int64_t boff = (int64_t)bz * g.batchC;
    const bool two = g.np_out == 2;
    const auto rC = out_rsrc(g.C32 + boff, nat_rows * 4u);
    // the value the planes hold: hi, or hi + lo (at most 17 significant bits: the fp32 sums are exact)
    auto rounded = [&](int i, int j) {
      const uint2 hi = split16(Plane0{}, acc[i][j]);
      f32x4 v = {__uint_as_float(hi.x << 16), __uint_as_float(hi.x & 0xffff0000u), __uint_as_float(hi.y << 16), __uint_as_float(hi.y & 0xffff0000u)};
      if (two) {
        const uint2 lo = split16(Plane1{}, acc[i][j]);
        v[0] += __uint_as_float(lo.x << 16); v[1] += __uint_as_float(lo.x & 0xffff0000u);
        v[2] += __uint_as_float(lo.y << 16); v[3] += __uint_as_float(lo.y & 0xffff0000u);
      }
      return v;
    };
    stage_begin();
    store_f32(rC, std::false_type{}, rC, rounded);
    store_plane(Plane0{}, acc_val, out_rsrc(g.Pn + boff, nat_rows * 2u), true, out_rsrc(g.Pt + boff, tr_rows * 2u), true);
    if (two)
      store_plane(Plane1{}, acc_val, out_rsrc(g.Pn + g.plane_out + boff, nat_rows * 2u), true,
                  out_rsrc(g.Pt + g.plane_out + boff, tr_rows * 2u), true);
  } else if constexpr (EPI == EPI_XADD) {
    const int64_t boff = (int64_t)bz * g.batchC;
    const auto rX = in_rsrc(g.Xadd + boff, nat_rows * 4u);
    const auto rC = out_rsrc(g.C32 + boff, nat_rows * 4u);
    store_f32(rC, std::true_type{}, rX, acc_val);
  } else {  // EPI_XOUT
    const int64_t boff = (int64_t)bz * g.batchC;
    const int np_max = F16 ? 1 : (g.np_out > g.np_out_n ? g.np_out : g.np_out_n);
    stage_begin();
    if constexpr (!F16) {
      const auto rX = in_rsrc(g.Xadd ? g.Xadd + boff : nullptr, g.Xadd ? nat_rows * 4u : 0u);
      const auto rC = out_rsrc(g.C32 ? g.C32 + boff : nullptr, g.C32 ? nat_rows * 4u : 0u);
      if (g.Xadd) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] += ld32(rX, nat4[j] + row_off(16 * i + e) * 4u);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (g.C32) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) st32(rC, nat4[j] + row_off(16 * i + e) * 4u, acc[i][j][e]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    auto plane = [&](auto p) {
      constexpr int P = decltype(p)::value;
      const bool nat = F16 || P < g.np_out_n, tr = F16 || P < g.np_out;
      store_plane(p, acc_val, out_rsrc(g.Pn + P * g.plane_out + boff, nat_rows * 2u), nat, out_rsrc(g.Pt + P * g.plane_out + boff, tr_rows * 2u), tr);
    };
    if (F16 || np_max > 0) plane(Plane0{});   // fp16 operands: the iterate is one fp16 plane of each layout
    if constexpr (!F16) {
      if (np_max > 1) plane(Plane1{});
      if (np_max > 2) plane(Plane2{});
    }
  }
  if (g.clk) {
    wait_vmcnt<0>();   // the epilogue's stores have left the wavefront
    if (tid == 0) {
      unsigned long long* o = g.clk + 4 * ((int64_t)blockIdx.z * gridDim.x + blockIdx.x);
      o[0] = pr_c2 - pr_c1;
      o[1] = pr_w2 - pr_w1;
      o[2] = pr_w1 - pr_w0;
      o[3] = wall_clock64() - pr_w2;
    }
  }
}

// Tiles, with what a workgroup that has its CU to itself takes: t0 us outside the main loop and ts per K step of 64 (fits to
// rotate, accumulate and polar launches at 16 .. 10500 tokens and widths 64 .. 8192).  192: fills the chip exactly at 3072.
// The second form of the largest tile is the one in 8 wavefronts, for the launches fits_largest_8 names; the last five are for
// the launches special_tile names.
struct Tile { int bm, bn, wgm, wgn; float t0, ts; };
constexpr Tile kTiles[] = {{256, 256, 2, 2, 10.0f, 1.30f}, {256, 128, 4, 2, 6.5f, 0.72f}, {128, 128, 2, 2, 6.5f, 0.42f}, {64, 64, 2, 2, 4.5f, 0.26f},
                           {192, 192, 2, 2, 8.5f, 0.75f}, {256, 256, 2, 4, 8.5f, 1.34f},
                           {96, 96, 2, 2, 4.5f, 0.38f}, {160, 160, 2, 2, 5.5f, 0.69f}, {96, 64, 2, 2, 4.7f, 0.29f}, {128, 64, 2, 2, 6.2f, 0.45f},
                           {128, 192, 2, 2, 6.5f, 0.62f}};
constexpr int kNumTiles = 11;

// Whether an epilogue's registers fit beside the 256 accumulators per lane of the 256 x 256 tile.  Those that change the
// accumulators in place or walk over them for a varying number of planes do not (64 .. 970 bytes per lane of scratch): they
// take the next best tile, in most cases 192 x 192.  None of them runs more than twice in an update.
constexpr bool fits_largest(int epi, bool f16) {
  return !(epi == EPI_SQUARE || (!f16 && (epi == EPI_GRAMW || epi == EPI_XOUT)));
}

// The largest tile in 8 wavefronts: a dearer K step (half as much LDS again is read), but less time outside the main loop,
// where 4 wavefronts have little to cover a latency with.  For the launches whose epilogue weighs against a short K: 6713 x
// 1584 rotated for the statistics 57.5 us in 4, 53.1 in 8; 432 tokens accumulated at d = 3280 30.8 and 28.6; but 8192 x 8192
// rotated 354 and 374.  The polar products have K = width.
constexpr bool fits_largest_8(int epi) {
  return epi == EPI_ACT || epi == EPI_SIGN || epi == EPI_SIGN_ACT || epi == EPI_SIGN_XT || epi == EPI_F32;
}

// Tiles between the others' sizes, each for launches whose count of the others' tiles just misses the 256 compute units:
//  96 x 96, 160 x 160   mirrored symmetric products: X^T X at 2048 253 tiles, 15.9 us (128 x 128 20.0), at 1792 14.2 (18.1); at
//                       3072 210 tiles, 35.2 us (192 x 192 42.2), at 2832 33.2 (39.5), at 3328 38.9 (45.3)
//  96 x 64              polar and accumulate products: 1104^3 216 tiles, 9.2 us (64 x 64, some sharing a compute unit, 10.0); among an
//                       update's other launches 11.3 and 13.2, the correction 18.3 (128 x 128 24.0)
//  128 x 64             signs and operand of heads up to 64 wide: 32 x 2048 x 64 8.4 us (256 x 128, half of it empty, 10.6).  What is
//                       left to it are long batches of one head or a few (the other steps are one launch, head_step_narrow.hip): step of
//                       4 heads of 64, 16384 tokens 80.4 and 77.3 us, of 8, 60000 285 and 266, of one, 65536 56.4 and 54.5
//  128 x 192            rotations of at most 256 such tiles (4 wavefronts of 64 x 96 read 80 KiB of LDS a K step, 8 of 64 x 48 would 112)
//                       and applies: 2048 x 3072 rotated 36.0 us (192 tiles of 256 x 128 39.3), 1842 x 2576 34.8 (40.0), 978 x 4464
//                       50.4 (59.5), with signs and operand 2.5 to 10 us less a step; update at 2304 727 (746).  Two rounds lose:
//                       2165 x 4240 104 and 92.  From 20 K steps to 100 (700 x 6400), the range it was measured over; the lower line is no
//                       crossing (4600 x 1072, 17 steps: 17.1 us, 256 x 128 19.3).  Accumulating at 2304 it was no faster than 192 x 192.
// (One launch after another on the same operands; the constants above are dearer, as operands just written by other units are.)
constexpr bool special_tile(int t, int epi, bool sym) {
  switch (t) {
    case 6: case 7: return sym;
    case 8: return epi == EPI_F32 || epi == EPI_XOUT || epi == EPI_XLAST || epi == EPI_XADD;
    case 9: return epi == EPI_SIGN_XT;
    default: return epi == EPI_ACT || epi == EPI_SIGN || epi == EPI_SIGN_ACT || epi == EPI_SIGN_XT || epi == EPI_XOUT || epi == EPI_XLAST;
  }
}

// Expected time of `tiles` workgroups of tile t with `steps` K steps each, all segments counted.  The large tiles fill a CU's
// LDS: whole rounds of 256.  Three 64 x 64 workgroups share one: up to 768 start at once, and a step of two or three sharing a
// CU takes 0.48 or 0.75 us, three also 1 us more outside the loop.  (Constants chosen over 170 random shapes, rotate, accumulate and update launches of both dtypes,
// every tile timed.)  The lines between 64 and 128 wide, us: 393 rows of 16 heads of width 384 rotated 13.2 (672 small tiles) and
// 8.6; fp32, six segments, 815 rows of 8 x 384 50.7 (624) and 36.2, 663 x 1488 59.9 (264) and 76.5; 1500 x 1104 with signs 17.3 (432)
// and 19.4; 2316 tokens of 32 heads of width 256 accumulated 38.0 (512, 37 steps) and 29.5.
double tile_time(int t, int64_t tiles, double steps) {
  const int64_t rounds = (tiles + 255) / 256;
  if (t == 3) {
    const double step = rounds <= 1 ? kTiles[t].ts : (rounds == 2 ? 0.48 : 0.75);
    return (kTiles[t].t0 + (rounds > 2 ? 1.0 : 0.0) + steps * step) * (tiles > 768 ? tiles / 768.0 : 1.0);
  }
  if (t == 10 && (rounds > 1 || steps < 20 || steps > 100)) return 1e300;   // (see special_tile)
  if (t == 9 && rounds > 1) return (double)((tiles + 511) / 512) * (kTiles[t].t0 + steps * 0.60);   // two share a compute unit
  return (double)rounds * (kTiles[t].t0 + steps * kTiles[t].ts);
}

constexpr int kSymMinTiles = 8;   // tiles per side from which the mirrored form of a symmetric product is used

struct Choice { int tile; bool sym; int64_t tiles; };   // tiles: workgroups per batch entry

// The tile of the least expected time.  A symmetric product whose square tiles give at least kSymMinTiles per side runs the
// t (t + 1) / 2 of them on and above the diagonal only, and is compared by the count that really runs: at 4096 the
// 256 x 256 tile leaves 136 workgroups on 256 compute units, the 192 x 192 tile 253.
Choice choose(const GemmArgs& a, GemmEpilogue epi, int batch) {
  const double steps = (double)((a.K + BK - 1) / BK) * a.nseg;
  const bool sym_epi = a.symmetric && (epi == EPI_GRAMW || epi == EPI_SQUARE || epi == EPI_FRO2);
  Choice best{-1, false, 0};
  for (int sym = sym_epi ? 1 : 0; sym >= 0 && best.tile < 0; --sym) {
    double best_time = 1e300;
    for (int t = 0; t < kNumTiles; ++t) {
      if ((t == 0 && !fits_largest(epi, a.ab_f16)) || (t == 5 && !fits_largest_8(epi)) || (t > 5 && !special_tile(t, epi, sym))) continue;
      const int64_t tm = (a.M + kTiles[t].bm - 1) / kTiles[t].bm, tn = (a.N + kTiles[t].bn - 1) / kTiles[t].bn;
      if (sym && (kTiles[t].bm != kTiles[t].bn || tm < kSymMinTiles)) continue;
      const int64_t tiles = sym ? tm * (tm + 1) / 2 : tm * tn;
      const double time = tile_time(t, tiles * batch, steps);
      if (time < best_time) { best_time = time; best = Choice{t, sym != 0, tiles}; }
    }
  }
  return best;
}

// The order of the tiles (`bands` of tile_of).  In bands, what an XCD runs at a time (32 tiles, or its whole share; tiles that share a
// compute unit are counted alike) is about square and reads the fewest operand rows; along lines its whole share is one run
// of whole tile rows or columns.  Which one wins was measured, us along lines and in bands:
//   rotations of several rounds    bands where they read at most 0.6 of the rows (and K is long enough for that to count): 9190 x 4096 280
//                                  and 264, 12000 x 5120 490 and 456, 4045 x 4480 166 and 161 (0.35 .. 0.5 of the rows); but 9190 x
//                                  3344 171 and 181 (0.63), 9190 rows of 8 x 304, 5 steps, 34.0 and 35.8
//   rotations of one round         lines: fp32, six segments, 1936 x 1040 55.1 and 60.4, 1100 x 480 17.7 and 19.4, 1500 x 800 40.2 and
//                                  43.4; 603 x 2096 (64 x 64, some sharing a compute unit) 15.7 and 18.7, 6000 x 2096 50.8 and 55.6.
//                                  But 64 x 64 tiles of many steps: 777 x 1040 34.8 and 33.5, 872 x 944 31.8 and 29.8; of 125
//                                  such from 84 steps on bands took 0.94 to 1.01 of the time, from 72 to 78 0.95 to 1.06
//   other products                 bands from two rounds on (a step of 4045 tokens at d = 5120 434 and 407).  A polar product of one round
//                                  reads what the same XCD has just written, and whole lines keep more of that in its L2: update at
//                                  d = 1104 360 us along the columns, 371 in bands.
// (Of 758 rotations timed, 24 are more than 3 % slower than along lines or in whole 4 x 8 blocks, in two library builds; 19 such are
// noise of the comparison.  Bands for every rotation of 32 steps or several rounds were slower for 130, by up to 21 %.)
int order_of(int tiles_m, int tiles_n, int bm, int bn, bool sym, int epi, int batch, int steps) {
  const int n = sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int share = (n + 7) / 8, run = std::min(share, 32);
  const bool one_round = (int64_t)n * batch <= 256;
  if (sym) {
    int h = 0;
    if (!one_round)
      for (h = 1; (h + 1) * (h + 1) <= run;) ++h;
    return h;
  }
  const bool square = (tiles_m & 3) == 0 && (tiles_n & 7) == 0 && (((tiles_m >> 2) * (tiles_n >> 3)) & 7) == 0;   // whole 4 x 8 blocks
  const bool rotates = epi == EPI_ACT || epi == EPI_SIGN || epi == EPI_SIGN_ACT || epi == EPI_SIGN_XT;
  // along the columns or the rows, whichever reads fewer operand rows
  const int64_t down = (int64_t)std::min(share, tiles_m) * bm + (int64_t)(share / tiles_m + 1) * bn;
  const int64_t across = (int64_t)std::min(share, tiles_n) * bn + (int64_t)(share / tiles_n + 1) * bm;
  const int line = across < down ? tiles_m : 1;
  const bool short_k = rotates && steps < (one_round ? 80 : 16), large = rotates && one_round && bm * bn > 64 * 64;
  if (!square && (short_k || large || (one_round && !rotates))) return line;
  // Of two blocks that read the same, accumulating and 256 x 256 tiles of whole blocks take the wider one, whose rows of the result are
  // longer: 4 x 8 tiles instead of 8 x 4.  A step of 512 tokens at d = 4096 66.3 us in 4 x 8, 69.9 in 8 x 4, of 2048 124 and 128, of
  // 512 at 8192 258 and 270, 8192 x 8192 rotated 717 and 730.  The others are the other way round: 11008 x 4096 (43 x 16 tiles of
  // 256 x 256) 292 and 288, 1024 x 2048 in 64 x 64 14.4 and 13.5.
  const bool wide = epi == EPI_F32 || (square && bm == 256 && bn == 256);
  int best = 1;
  int64_t best_rows = INT64_MAX;
  for (int h = std::min(tiles_m, run); h >= 1; --h) {
    const int64_t rows = (int64_t)h * bm + (int64_t)((run + h - 1) / h) * bn;
    if (rows < best_rows || (wide && rows == best_rows)) { best_rows = rows; best = (tiles_m + h - 1) / h; }
  }
  if (!square && rotates && !one_round && 5 * best_rows > 3 * std::min(down, across)) return line;
  return best;
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE, int EPI, bool F16, bool SYM = false>
hipError_t launch_one(const GemmArgs& a, int batch, hipStream_t stream) {
  constexpr int smem = NSTAGE * (BM + BN) * BK * 2;
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  static PerDeviceOnce configured;
  auto kern = gemm_nt_kernel<BM, BN, WGM, WGN, NSTAGE, EPI, F16, SYM>;
  hipError_t e = configured.run([&] {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (e != hipSuccess) return e;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  dim3 grid(SYM ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n, 1, batch);
  const int bands = order_of(tiles_m, tiles_n, BM, BN, SYM, EPI, batch, (a.K + BK - 1) / BK * a.nseg);
  hipLaunchKernelGGL(kern, grid, dim3(64 * WGM * WGN), smem, stream, a, tile_order(tiles_m, tiles_n, SYM, bands));
  return hipGetLastError();
}

template <int EPI, bool F16 = false>
hipError_t launch_epi(const GemmArgs& a, int batch, hipStream_t stream) {
  const Choice c = choose(a, (GemmEpilogue)EPI, batch);
  constexpr bool LARGEST = fits_largest(EPI, F16);
  if constexpr (EPI == EPI_GRAMW || EPI == EPI_SQUARE || EPI == EPI_FRO2) {
    if (c.sym) {   // tiles on and above the diagonal only
      switch (c.tile) {
        case 0: if constexpr (LARGEST) return launch_one<256, 256, 2, 2, 2, EPI, F16, true>(a, batch, stream); break;
        case 2: return launch_one<128, 128, 2, 2, 3, EPI, F16, true>(a, batch, stream);
        case 4: return launch_one<192, 192, 2, 2, 3, EPI, F16, true>(a, batch, stream);
        case 6: return launch_one<96, 96, 2, 2, 3, EPI, F16, true>(a, batch, stream);
        case 7: return launch_one<160, 160, 2, 2, 3, EPI, F16, true>(a, batch, stream);
        default: return launch_one<64, 64, 2, 2, 3, EPI, F16, true>(a, batch, stream);
      }
    }
  }
  switch (c.tile) {
    // LDS stages: as many 64-deep tiles as fit (two of 64 KiB for 256 x 256; smaller tiles take a third, which
    // puts two K steps instead of one between a load's issue and its use)
    case 0: if constexpr (LARGEST) return launch_one<256, 256, 2, 2, 2, EPI, F16>(a, batch, stream); break;
    case 1: return launch_one<256, 128, 4, 2, 3, EPI, F16>(a, batch, stream);
    case 2: return launch_one<128, 128, 2, 2, 3, EPI, F16>(a, batch, stream);
    case 4: return launch_one<192, 192, 2, 2, 3, EPI, F16>(a, batch, stream);
    case 5: if constexpr (fits_largest_8(EPI)) return launch_one<256, 256, 2, 4, 2, EPI, F16>(a, batch, stream); break;
    case 8: if constexpr (special_tile(8, EPI, false)) return launch_one<96, 64, 2, 2, 3, EPI, F16>(a, batch, stream); break;
    case 9: if constexpr (special_tile(9, EPI, false)) return launch_one<128, 64, 2, 2, 3, EPI, F16>(a, batch, stream); break;
    case 10: if constexpr (special_tile(10, EPI, false)) return launch_one<128, 192, 2, 2, 3, EPI, F16>(a, batch, stream); break;
    default: return launch_one<64, 64, 2, 2, 3, EPI, F16>(a, batch, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// For tests (host code only): the tile launch_gemm_nt takes for such a launch, as { rows, columns, wavefronts, workgroups per
// batch entry, 1 if mirrored }.
extern "C" __attribute__((visibility("default"))) void conqur_gemm_tile_for_tests(int epi, int f16, int symmetric, int M, int N, int K, int nseg,
                                                                                  int batch, int* out) {
  GemmArgs a{};
  a.M = M; a.N = N; a.K = K; a.nseg = nseg; a.ab_f16 = f16; a.symmetric = symmetric;
  const Choice c = choose(a, (GemmEpilogue)epi, batch);
  const Tile& u = kTiles[c.tile];
  out[0] = u.bm; out[1] = u.bn; out[2] = u.wgm * u.wgn; out[3] = (int)c.tiles; out[4] = c.sym;
}

// For tests (host code only): the tile of every workgroup of such a grid, in the order the launcher takes for it, and that order's `bands`.
extern "C" __attribute__((visibility("default"))) int conqur_gemm_order_for_tests(int epi, int symmetric, int tiles_m, int tiles_n, int bm, int bn,
                                                                                  int batch, int steps, int* tm, int* tn) {
  const int bands = order_of(tiles_m, tiles_n, bm, bn, symmetric != 0, epi, batch, steps);
  const int n = symmetric ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const TileOrder o = tile_order(tiles_m, tiles_n, symmetric != 0, bands);
  for (int i = 0; i < n; ++i) symmetric ? tile_of<true>(i, o, tm + i, tn + i) : tile_of<false>(i, o, tm + i, tn + i);
  return bands;
}

int gemm_num_workgroups(const GemmArgs& a, GemmEpilogue epi, int batch) { return (int)(choose(a, epi, batch).tiles * batch); }

int gemm_num_partials(const GemmArgs& a, GemmEpilogue epi, int batch) {
  const Tile& u = kTiles[choose(a, epi, batch).tile];   // (a mirrored tile has slots of its own)
  return ((a.M + u.bm - 1) / u.bm) * ((a.N + u.bn - 1) / u.bn) * u.wgm * u.wgn;
}

int gemm_max_partials(int M) {
  const Tile& u = kTiles[3];
  return ((M + u.bm - 1) / u.bm) * ((M + u.bn - 1) / u.bn) * u.wgm * u.wgn;
}

double gemm_issued_flop(const GemmArgs& a, GemmEpilogue epi, int batch) {
  const Choice c = choose(a, epi, batch);
  return 2.0 * (double)c.tiles * kTiles[c.tile].bm * kTiles[c.tile].bn * (double)a.K * a.nseg * batch;
}

hipError_t launch_gemm_nt(const GemmArgs& a, GemmEpilogue epi, int batch, hipStream_t stream) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0 || (a.K & 7) || (a.lda & 7) || (a.ldb & 7) || a.nseg < 1 || a.nseg > kMaxSegments ||
      batch < 1 || (a.ab_f16 && epi != EPI_F32 && epi != EPI_GRAMW && epi != EPI_XOUT && epi != EPI_XLAST) ||
      (a.ab_f16 && ((epi == EPI_GRAMW && (a.np_out != 1 || a.resid_part)) ||
                    (epi == EPI_XOUT && (a.np_out != 1 || a.np_out_n != 1 || a.Xadd || a.C32)))) || (int64_t)a.M * a.lda >= (1ll << 30) || (int64_t)a.N * a.ldb >= (1ll << 30))
    return hipErrorInvalidValue;
  if (a.symmetric && ((epi != EPI_GRAMW && epi != EPI_SQUARE && epi != EPI_FRO2) || (epi != EPI_FRO2 && a.A != a.B) ||
                      a.M != a.N || a.lda != a.ldb || (a.M & 3)))
    return hipErrorInvalidValue;
  // the matrix-writing epilogues address their arrays [M or N rows][ldc] through 32-bit byte offsets
  if ((epi == EPI_F32 || epi == EPI_GRAMW || epi == EPI_SQUARE || epi == EPI_XLAST || epi == EPI_XOUT || epi == EPI_XADD) &&
      ((a.M & 7) || (a.N & 7) || (a.ldc & 7) || a.ldc < a.N || (epi != EPI_F32 && a.ldc < a.M) || (int64_t)((a.M > a.N ? a.M : a.N) + 256) * a.ldc >= (1ll << 29)))
    return hipErrorInvalidValue;
  // EPI_ACT / EPI_SIGN_ACT address Y relative to a tile's first row: 256 rows x pitch x 4 bytes below 2^31
  if ((epi == EPI_ACT && (a.ldc < a.N || a.ldc >= (1ll << 21))) || (epi == EPI_SIGN_ACT && (a.ldy < a.N || a.ldy >= (1ll << 21))))
    return hipErrorInvalidValue;
  if ((epi == EPI_ACT || epi == EPI_SIGN_ACT) && (a.N & 7)) return hipErrorInvalidValue;   // the staged stores take whole chunks of columns
  if (epi == EPI_XADD && (!a.Xadd || !a.C32)) return hipErrorInvalidValue;
  if (epi == EPI_XLAST && (!a.C32 || !a.Pn || !a.Pt || (a.M & 3) || a.np_out < 1 || a.np_out > 2)) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_SIGN: return launch_epi<EPI_SIGN>(a, batch, stream);
    case EPI_SIGN_XT:
      if (!a.xt_w || !a.Xt || !a.cnt || a.cnt_slots < 1 || a.N != a.K || a.nseg != 1) return hipErrorInvalidValue;
      return launch_epi<EPI_SIGN_XT>(a, batch, stream);
    case EPI_SIGN_ACT: return a.Yact ? launch_epi<EPI_SIGN_ACT>(a, batch, stream) : hipErrorInvalidValue;
    case EPI_ACT: return launch_epi<EPI_ACT>(a, batch, stream);
    case EPI_F32: return a.ab_f16 ? launch_epi<EPI_F32, true>(a, batch, stream) : launch_epi<EPI_F32>(a, batch, stream);
    case EPI_GRAMW: return a.ab_f16 ? launch_epi<EPI_GRAMW, true>(a, batch, stream) : launch_epi<EPI_GRAMW>(a, batch, stream);
    case EPI_XLAST: return a.ab_f16 ? launch_epi<EPI_XLAST, true>(a, batch, stream) : launch_epi<EPI_XLAST>(a, batch, stream);
    case EPI_XOUT: return a.ab_f16 ? launch_epi<EPI_XOUT, true>(a, batch, stream) : launch_epi<EPI_XOUT>(a, batch, stream);
    case EPI_XADD: return launch_epi<EPI_XADD>(a, batch, stream);
    case EPI_SQUARE: return launch_epi<EPI_SQUARE>(a, batch, stream);
    case EPI_FRO2: return launch_epi<EPI_FRO2>(a, batch, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace conqur
