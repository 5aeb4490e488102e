// Non-GEMM kernels of the calibration path: row norms, scaled/transposed operand
// preparation, bf16 split packing, statistics reductions, polar start/finish and
// the bandwidth-bound fake-quantisation error kernel.  Launch wrappers only; each
// returns the launch status.
#pragma once
#include "common.h"

namespace conqur {

// n_i = ||x_i||_2 over each head slice; w_i = kXhatScale / n_i, or 0 for a row that is
// all zero or holds a non-finite value (then nrm = 0 and *nonfinite is raised for NaN/Inf).
hipError_t launch_row_norms(const void* X, int x_is_f32, int64_t T, int64_t stride, int heads, int dh,
                            float* nrm, float* w, int64_t ldn, int* nonfinite, hipStream_t s);

// Xt[p][k][i] = x_ik * w_{head(k), i} for i < T, 0 for T <= i < Tk.  np = 1 (bf16 activations):
// one fp16 plane; np = 3 (fp32 activations): three bf16 split planes (exact).
// Also counts the rows (w != 0: entered M, w == 0: skipped) into cnt [heads][kCountSlots][2], the token block b
// into slot b % kCountSlots.
constexpr int kCountSlots = 64;
hipError_t launch_transpose_scale(const void* X, int x_is_f32, int64_t T, int64_t Tk, int64_t stride, int d, int dh,
                                  const float* w, int64_t ldn, bf16_bits* Xt, int64_t pitch, int64_t plane, int np,
                                  unsigned long long* cnt, hipStream_t s);

// Xs[p][i][k] = split_p(x_ik), fp32 activations only (3 planes).
hipError_t launch_split_rows(const float* X, int64_t T, int64_t stride, int d, bf16_bits* Xs, int64_t plane,
                             hipStream_t s);

// Y = X R_op per head for the few rows rotate_rows_fits() admits (rotate_rows.hip): X [T][stride] and Y [T][ldy] in bf16 or fp32,
// RopT the rotate operand [heads][dh][dh] (R^T; three split planes, `plane` elements apart, for fp32).  stats non-null: a
// statistics step, whose operands the launch leaves in the first kRotateRowsTokens tokens of St and (bf16) Xt, both
// [heads * dh][pitch]: the corner signs (+1 beyond T; fp16 for bf16 activations, bf16 for fp32) and the rows of X times w
// ([heads][ldw]), fp16 (0 beyond T); the rows entered and skipped are added to cnt (bf16).  Y may be null then.
constexpr int kRotateRowsTokens = 64;
struct RotateRowsStats {
  bf16_bits* St;
  bf16_bits* Xt;
  int64_t pitch;
  const float* w;
  int64_t ldw;
  unsigned long long* cnt;   // [heads][cnt_slots][2]
  int cnt_slots;
};
bool rotate_rows_fits(int x_is_f32, int64_t T, int dh);
hipError_t launch_rotate_rows(const void* X, int x_is_f32, int64_t T, int64_t stride, const bf16_bits* RopT, int64_t plane, int heads,
                              int dh, void* Y, int64_t ldy, const RotateRowsStats* stats, hipStream_t s);

// Split an fp32 matrix batch [batch][rows][cols] into np bf16 planes, in natural
// layout (outN[p][b][r][c]) and/or transposed (outT[p][b][c][r]); either may be null.
// out_f16 (np = 1 only): the plane holds the values rounded to fp16 instead of bf16.
hipError_t launch_pack(const float* src, int batch, int rows, int cols, int np, bf16_bits* outN, bf16_bits* outT,
                       int64_t plane, hipStream_t s, int out_f16 = 0);

// out[h] = <R_op,h , M_h> over n elements per head, R_op = R rounded to bf16 if round_bf16 else R (the l1 term of
// the accumulated rows is sqrt(dh) times this).  part: heads * dot_rm_partials(n) doubles of scratch.
int dot_rm_partials(int64_t n);
hipError_t launch_dot_rm(const float* R, const float* M, int heads, int64_t n, int round_bf16, double* part, double* out,
                         hipStream_t s);

// part[h][dot_rm_partials(n)]: partial sums of M_h^2.  stamp: receives the device's wall clock at the start of the launch.
hipError_t launch_fro2(const float* M, int heads, int64_t n, double* part, unsigned long long* stamp, hipStream_t s);

// Start of the polar iteration, fused with the operand packing: X0 = (M + lambda*tau*R) / alpha with
// tau = ||M||_F/sqrt(dh), alpha = ||M||_F (1 + lambda) (a head with M = 0 starts from R itself), written as np bf16
// split planes in natural (outN) and transposed (outT) layout.  ||M_h||_F^2 is the sum of nparts partial sums per head
// (fro2_parts[h * nparts + p]), which every workgroup adds up for itself, and goes to fro2_out[h].
// If dot_part is not null, also pack_dot_partials(dh) partial sums per head of <R_op,h , M_h> (R_op = R rounded to bf16 if
// round_bf16), the quantity of launch_dot_rm, from the same pass.
hipError_t launch_polar_start_pack(const float* M, const float* R, int heads, int dh, float lambda, const double* fro2_parts, int nparts,
                                   double* fro2_out, int np, bf16_bits* outN, bf16_bits* outT, int64_t plane, int round_bf16,
                                   double* dot_part, hipStream_t s, int out_f16 = 0);

// X += kappa * R over n elements (all heads).
hipError_t launch_axpy(float* X, const float* R, int64_t n, float kappa, hipStream_t s);

// End of the polar iteration, one pass over X: pack_dot_partials(dh) partial sums per head of <X_h, M_h>, the rotate operand
// outT = np bf16 split planes of X^T, and, if R32 is not null, R32 = X.
int pack_dot_partials(int dh);
hipError_t launch_polar_finish_pack(const float* X, const float* M, int heads, int dh, int np, float* R32, bf16_bits* outT,
                                    int64_t plane, double* dot_part, hipStream_t s);

// The last launch of an update that is not one launch: its scalar results to the host, the batch statistics and the non-finite flag cleared.
struct UpdateEnd {
  int heads;
  // <R_op, M> and <R, M> per head: sums of nparts partial sums each; ldot_parts null: <R_op, M> as it lies at scalars
  const double* ldot_parts;
  const double* inner_parts;
  int nparts;
  const double* scalars;       // device: [ldot heads | fro2 heads]
  int* nonfinite;
  void* stats;                 // stats_bytes, a multiple of 8
  size_t stats_bytes;
  // in host memory the device can write
  double* host;                // [ldot | inner | fro2]
  int* host_nonfinite;         // set if the flag is (never cleared here)
  unsigned long long* stamp;   // the device's wall clock (100 MHz) near the end
};
hipError_t launch_update_end(const UpdateEnd& u, hipStream_t s);

// Fused statistics step for heads of width 128 with bf16 activations (head_step.hip): one kernel rotates, normalises,
// takes the corners and accumulates; every workgroup (head, share of the tokens) stores a partial M_h into
// Mpart [nsplit][heads][128][128], adds its share of L / rows / skipped, writes the row norms and, if St is not null,
// the corner signs (+-1 as fp16, transposed [heads*128][pitch]).  launch_head_reduce then sets or adds the shares to M.
// The partial M_h already carry the factor 1 / (kXhatScale sqrt(128)).
int head_step_splits(int heads, int64_t T);
hipError_t launch_head_step128(const bf16_bits* X, int64_t T, int64_t stride, int heads, const bf16_bits* RopT, float* Mpart,
                               int nsplit, float* nrm, int64_t ldn, double* L, unsigned long long* rows,
                               unsigned long long* skipped, int* nonfinite, bf16_bits* St, int64_t pitch, hipStream_t s);
// fro2_part non-null: also 16 partial sums of squares per head of the resulting M (kHeadReduceParts doubles per head, in
// head order), whose sum per head is ||M_h||_F^2.
// The same sum for any matrix of n_total floats (a multiple of 1024) held as nsplit shares [nsplit][n_total], fixed order.
hipError_t launch_sum_shares(const float* part, int nsplit, int64_t n_total, float* M, int accumulate, hipStream_t s);
constexpr int kHeadReduceParts = 16;
// stamp non-null: receives the device's wall clock at the start of the launch.
hipError_t launch_head_reduce(const float* Mpart, int nsplit, int heads, float* M, int accumulate, double* fro2_part, hipStream_t s,
                              unsigned long long* stamp = nullptr);

// The statistics step of heads of width 16 .. 112 with bf16 activations in one launch (head_step_narrow.hip), bit for bit what the row
// norms, the rotate GEMM's signs and operand and the accumulate GEMM leave: the row norms, the corner signs St (fp16 +-1,
// transposed [heads * dh][pitch], pitch at least T rounded up to 32), the row counters cnt [heads][cnt_slots][2], and M
// [heads][dh][dh], set or added to.
constexpr int kHeadStepNarrowMaxDh = 112;
struct HeadStepNarrow {
  const bf16_bits* X;
  int64_t T, stride;
  int heads;
  const bf16_bits* RopT;
  float* M;
  int accumulate;
  float* nrm;
  int64_t ldn;
  unsigned long long* cnt;
  int cnt_slots;
  int* nonfinite;
  bf16_bits* St;
  int64_t pitch;
};
hipError_t launch_head_step_narrow(const HeadStepNarrow& a, int dh, hipStream_t s);
// Whether that is the faster way for these sizes (several heads of a width it takes; T tokens of a batch).
bool head_step_narrow_pays(int dh, int heads, int64_t T);

// Main phase of the polar iteration for heads of width up to kHeadPolarMaxDh (a multiple of 16) in one launch
// (head_polar.hip): runs the composed cubics X <- X (a_k I + b_k X^T X), k < nsteps, on single fp16 operand planes held in
// LDS (11 significant bits).  Xt0: the start iterate as one transposed fp16 plane [heads][dh][dh].
// Outputs, as the last step of the general path writes them: the result rounded to bf16, as X32 (fp32), Pt (one transposed
// bf16 plane) and Pn (one natural bf16 plane).
constexpr int kHeadPolarMaxDh = 128;
constexpr int kPolarScheduleMax = 64;
struct PolarSchedule {
  int nsteps;
  float a[kPolarScheduleMax], b[kPolarScheduleMax];
};
// close non-null (start as well): each head whose residual ||I - X^T X||_F at the hand-over is at most res_max also takes the closing
// step X <- X + X (D + 1.5 D^2), D = (I - X^T X)/2, in the same launch and writes R (fp32) and RopT (bf16 plane of R^T).  Of a head that
// did not take the step R and RopT are untouched and ||D^2||_F^2 is reported < 0.  The hand-over outputs are written either way.
struct HeadPolarClose {
  float* R;
  bf16_bits* RopT;     // rop_planes split planes of R^T, rop_plane elements apart
  int rop_planes;
  int64_t rop_plane;
  const float* M;
  float res_max;
  // The update's report, by each head for itself: its results to host memory the device can write, [||I - X^T X||_F^2 | ||D^2||_F^2 |
  // <R_op, M> | <R, M> | ||M||_F^2] of `heads` values each (<R, M>: if the step was taken), and the device's wall clock behind them to
  // host_stamps[h]; its batch statistics copied to stats_keep and, if its residual is finite, cleared (both [L | rows | skipped |
  // counters [kCountSlots][2]] of 8 bytes per value, `heads` of each); by head 0 the non-finite flag, likewise.
  double* host;
  unsigned long long* host_stamps;
  unsigned long long* stats;
  unsigned long long* stats_keep;
  int* nonfinite;
  int* host_nonfinite;
};
// start non-null: the launch forms the start iterate itself, X0 = (M + lambda tau R) / alpha per head (Xt0 unused, may
// be null), from M and R (fp32 [heads][dh][dh]).  ||M_h||_F^2 is the sum of nparts partial sums per head
// (fro2_parts[h * nparts + p]), or taken from M in the launch (nparts = 0); it also goes to fro2_out[h].  ldot non-null:
// ldot[h] = <R_op, M_h> (rop_dot; R_op = R rounded to bf16 if round_bf16, else R), or a copy of L[h].
struct HeadPolarStart {
  const float* M;
  const float* R;
  const double* fro2_parts;
  int nparts;
  double* fro2_out;
  float lambda;
  const double* L;
  double* ldot;
  int rop_dot;
  int round_bf16;
  float* R_keep;       // non-null: a copy of R, which the closing step may replace in the same launch
  unsigned long long* stamp;   // non-null: receives the device's wall clock at the start of the launch
};
hipError_t launch_head_polar(const bf16_bits* Xt0, int heads, int dh, const PolarSchedule& sched, float* X32, bf16_bits* Pn, bf16_bits* Pt,
                             const HeadPolarClose* close, const HeadPolarStart* start, hipStream_t s);

// One step X <- X (a I + b X^T X) of that phase for wider heads, up to kPolarStepMaxDh (a multiple of 16), in one launch
// (polar_step.hip): reads the iterate as one transposed fp16 plane [heads][dh][dh] and writes the next one the same way into another.
// last: the hand-over outputs of launch_head_polar instead (Xt_out the transposed bf16 plane).
constexpr int kPolarStepMaxDh = 256;
hipError_t launch_polar_step(const bf16_bits* Xt, int heads, int dh, float a, float b, bf16_bits* Xt_out, int last, float* X32, bf16_bits* Pn,
                             hipStream_t s);
double polar_step_flop(int heads, int dh);   // multiply-add work of such a launch

// Per-row fake-quantisation error of Y [T][ld] (bf16 or fp32) into row_sse / row_en, then their sums over rows:
// out[0] = SSE, out[1] = energy (skipped if out is null).  zero_point = 0: symmetric quantiser; 1: zero-point quantiser on [clip*min, clip*max].
// Q non-null: the quantised rows are also written to Q [T][ldq] in Y's element type (Q must not overlap Y).
hipError_t launch_quant_error(const void* Y, int y_is_f32, int64_t T, int64_t ld, int d, int bits, int zero_point, float clip,
                              float* row_sse, float* row_en, double* out, void* Q, int64_t ldq, hipStream_t s);

// Per-row diagnostics of Y [T][ld] (bf16 or fp32): row_pr = ||y||_2^4 / (d ||y||_4^4), row_rho = ||y||_inf^2 / ||y||_2^2
// (0, 0 for a row with zero or non-finite energy).
hipError_t launch_row_diag(const void* Y, int y_is_f32, int64_t T, int64_t ld, int d, float* row_pr, float* row_rho,
                           hipStream_t s);

// out[h] = sum of part[h][0..n) for h < heads, fixed order.  out may be host memory the device can write.
hipError_t launch_sum_partials(const double* part, int n, int heads, double* out, hipStream_t s);

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);

// Device address, on the current device, of the static array conqur_score_rows_static keeps its per-row results in
// (static_score.hip); looked up once per device.
hipError_t static_scratch_for_current_device(float** out);

}  // namespace conqur
