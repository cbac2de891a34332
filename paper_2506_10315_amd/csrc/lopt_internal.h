// Internal declarations shared by the host planner and the gfx950 kernels of the
// learned-optimizer step library. Not part of the public boundary (see include/lopt.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lopt.h"

namespace lopt {

constexpr int kBlock = 256;       // threads per workgroup (4 wavefronts of 64)
constexpr int kWave = 64;
constexpr int kTileCols = 256;    // one wavefront row-segment: 64 lanes x float4
constexpr int kRowUnit = 64;      // standard tile height (taller for tall tensors, shorter for small lists)
constexpr int kMaxRowTiles = 256; // tile height grows so that a large tensor has at most this many row tiles ...
constexpr int kMaxTileRows = 1024; // ... up to this height (bounds the length of the per-lane fp32 partial sums)
constexpr int kShortRows = 64;    // short lists: rows of a statistics tile at most
// Short lists: rows per tile of the row/column sums (16 wavefronts, four or eight rows each). Their column sums are doubles, of
// which every workgroup of the statistics pass reads all for its columns: fewer and taller tiles where there would be many. us a step
// with fp32 sums of 64 rows / doubles of 64 / doubles of 128: 2000x2000 103.2 / 106.2 / 104.3, 3000x3000 under VeLO 139.6 / 144.7 /
// 140.2, 1000x1000 41.5 / 41.7 / 42.5, under VeLO, whose recurrent product rides along, 37.0 / 37.8 / 37.2, 512x512 there no difference.
__host__ __device__ inline int short_rows(int m, bool velo) { return m <= (velo ? 512 : 1024) ? 64 : 128; }
constexpr int kStatStride = 20;   // floats per tile in the per-tile statistics partials (17 used)
constexpr int kRcStride = 12;     // floats per entry of the row/column partials (9 used)
constexpr int kNStat = 17;        // per-element statistics accumulated per tile
constexpr int kStatsPerTensor = 32;
constexpr int kLstmInPad = 48;    // LOPT_VELO_LSTM_IN rounded up to a multiple of 4
constexpr int kMaxGroups = 16;    // tensor groups of the two-stream pipeline, tile counters in the workspace
constexpr int kMixSlices = 64;    // at most this many slices of the tensor list in the cross-tensor mean
// Tensor lists up to this length form the LSTM's recurrent product ahead, beside the row/column sums. us, row/column sums + LSTM,
// in one launch / ahead: one tensor 4.4 + 9.7 / 5.4 + 4.1, 66 tensors 4.4 + 10.7 / 9.2 + 4.2, 152 tensors 58 + 14 / 66 + 5.5, 502
// tensors 25 + 26 / 68 + 7.
constexpr int kLstmAheadMax = 96;
// Its workgroups, kRecurTensors tensors x 8 units each, must leave room for those of the sums: the chip holds 512 of sixteen
// wavefronts. Tensors of 64x64, us a step in one launch / ahead, H_L 1024 32 tensors (256 workgroups) 48.2 / 42.4, 48 (384) 50.3 / 51.8, 64
// (512) 54.2 / 56.6, 80 60.9 / 67.0, 96 61.6 / 68.7; H_L 768 64 tensors (384) 49.8 / 49.7, 80 (480) 55.0 / 52.8, 96 (576) 55.7 / 59.3; H_L 512
// 96 tensors (384) 45.8 / 46.0.
constexpr int kRecurTensors = 16, kRecurBlocks = 512;
inline bool lstm_ahead(size_t n, int HL) {
  return n <= (size_t)kLstmAheadMax && ((int)n + kRecurTensors - 1) / kRecurTensors * ((HL + 7) / 8) < kRecurBlocks;
}
constexpr int kFinTensorsMax = 8;    // tensor lists up to this length may form the LSTM's inputs in its own launch (Plan::fold_finalize)
constexpr int kHeadSplitMax = 96;    // tensor lists up to this length cut the hypernetwork head's product into column blocks
constexpr int kHeadBatchMin = 1024;  // tensor lists from this length on take the batched form of the hypernetwork head
constexpr int kMixJSplit = 4;     // the LSTM units are cut into this many ranges when hbar Wg is formed
#ifndef LOPT_APPLY_ROWS
#define LOPT_APPLY_ROWS 128
#endif
constexpr int kApplyRows = LOPT_APPLY_ROWS;   // tile of the strip-form apply kernel: up to this many rows x 128 columns
constexpr int kApplyCols = 128;
// small_fc_lopt of padded width 4, 8 or 16 (k_apply_fc4x): rows of loads in flight per wavefront, wavefronts per SIMD (which is
// workgroups per CU). Width 16 is bound by its instructions: occupancy is worth more than prefetch there (four rows and three
// wavefronts 198 us a step, two and four 196, one and four 192, one and five 191 with 14 spilled registers; 9.5 M elements).
constexpr int narrow_trip_rows(int HP) { return HP == 16 ? 1 : 4; }
constexpr int narrow_waves_per_simd(int HP) { return HP == 8 ? 3 : 4; }

// Per-tensor record in device memory. Offsets o* are in floats from the workspace base.
struct TensorDev {
  float* p;
  const float* g;
  float* st;
  int m, n;
  uint32_t padN, padm, padn, padH;  // state section strides in floats
  uint32_t ndim;
  int vec;                          // 0: rows are not 16-byte aligned, 1: they are (n % 4 == 0), 2: 128-byte aligned (n % 32 == 0)
  int TR, nrt, nct, tile0;          // tile height, tile grid, first global tile id
  int rc0, nrpart, ncpart;          // first row/col block id, number of row and column partials: one a block, short lists two
  uint64_t oRowPart;                // [nct][m]   sum over the tile's columns of g^2
  uint64_t oColPart;                // [nrt][n]   sum over the tile's rows of g^2 (short lists: [ceil(m / short_rows)][n], double)
  uint64_t oRR;                     // [3][padm]  rsqrt(r_k + eps_acc); short lists: then r_k [3][padm] as the step found them
  uint64_t oRC;                     // [3][padn]  rsqrt(c_k + eps_acc); short lists: then c_k [3][padn] as the step found them
  uint64_t oRcPart;                 // [nrpart + ncpart][kRcStride]
  uint64_t oStatPart;               // [nrt*nct][kStatStride]
  uint64_t oStats;                  // [kStatsPerTensor] s_f
  uint64_t oScale;                  // [kStatsPerTensor] factor applied to the raw feature
  uint64_t oPrep;                   // prepared first layer: W1s[F][HP] then b1'[HP]
};

struct TileDev { int tensor, ti, tj, pad; };
struct RcItemDev { int tensor, is_col, blk, pad; };
struct ApplyTileDev { int tensor, r0, c0, rows; };   // rows <= kApplyRows

// Scalars of one step, passed by value to the kernels.
struct StepArgs {
  float mom_decay[3];
  float rms_decay;
  float fac_decay[3];
  float eps_acc, eps_norm;
  float exp_mult, step_mult;
  float lr, wd;
  int kind, H, HP, F;         // F = number of normalized per-element features (28 or 29)
  int HL, K, P;               // VeLO: LSTM width, bank rows, floats per per-tensor MLP
  int n_tensors;
};

// Time features tanh(step / x) and VeLO's loss features tanh(psi / x), psi = sign(loss) ln(1 + |loss|), formed in double by the host: on the
// device fourteen tanh in double held up the sums of k_finalize (0.3 to 0.5 us of it).
struct StepFeats { float time[LOPT_N_TIME], loss[LOPT_N_LOSS]; };

// Device weights of the optimizer, owned by the context.
struct WeightsDev {
  // small_fc_lopt (original layout, as uploaded)
  const float* mlp;    // W1[39,H] b1[H] W2[H,H] b2[H] W3[H,2] b3[2]
  const float* mlp_tail;  // W2[HP,HP] b2[HP] W3[HP,2] b3[2] pad[2] W1[28,HP]: zero-padded to the padded width HP
  // VeLO
  const float* Wx; const float* Wh; const float* Wg; const float* b; const float* Wa; const float* ba;
  const float* ws; const float* bs; const float* B;
  const float* lstm;   // [Wx ; Wh] repacked for k_velo_lstm: [ceil(H_L / 8)][lstm_k_pad(H_L)][4 gates x 8 units]
  const float* head;   // W_a, b_a, B and the step-size head folded into one matrix (null: two products, see head_folds)
};

// Input slots of the LSTM rounded up to whole octets; row length of the folded head (P columns and the step size's).
__host__ __device__ inline int lstm_k_pad(int HL) { return kLstmInPad + (HL + 7) / 8 * 8; }
__host__ __device__ inline int head_ld(int P) { return (P + 1 + 3) / 4 * 4; }
// The folded head reads (H_L + 1) (P + 1) weights per tensor, the two products H_L K + K P. (K >= 4: the folded form's scratch
// row, P + 1 rounded up, is then never longer than the K + P floats of the other.)
inline bool head_folds(int HL, int K, int P) { return K >= 4 && (size_t)HL * P <= (size_t)HL * K + (size_t)K * P; }

struct Launch {
  const TensorDev* tensors;
  const TileDev* tiles;
  const RcItemDev* rcitems;   // row and column blocks: workgroups of k_rc_update, on short lists of the statistics pass
  float* ws;
  int n_tensors, n_tiles, n_rcitems;
  const ApplyTileDev* atiles;
  int n_atiles;
  int tensor0;   // first tensor of the sub-list this launch covers (the per-tensor kernels index from it)
  int* apply_counter;     // tile counter of the apply kernel for this sub-list (cleared by k_finalize)
  int resident_wgs;       // workgroups of the strip-form apply kernel that are resident at once (2 per CU)
  int beside_apply;       // this sub-list's passes run beside the apply pass of another one
  const TileDev* rctiles; // short lists: tiles of short_rows x kTileCols of the row/column sums
  int n_rctiles;
  bool short_list;        // the statistics pass finishes the row and column means itself (Plan::short_list)
  int keep, keep_off;     // tiles below these numbers are read by the statistics pass with ordinary loads: rows on the 128-byte grid,
                          // rows off the 16-byte grid (Plan::keep)
  bool keep_line;         // short lists: rows on the 16-byte but off the 128-byte grid are read as rows off the 16-byte grid
  bool backwards;         // the statistics pass takes its tiles from the last to the first
  bool strip_ordinary;    // the strip kernel reads with ordinary loads (Plan; never where it folds the finalize)
  bool off_grid_nt;       // the narrow and the VeLO kernel access rows off the 16-byte grid nontemporally (Plan)
};

// kernels (lopt_kernels.hip / lopt_apply_mfma.hip)
void launch_fill_zero(const Launch&, const StepArgs&, hipStream_t);
// VeLO: the two stages of the cross-tensor term (hbar = mean of the tensors' LSTM outputs of the previous step,
// b_eff = b + hbar Wg) ride along as extra workgroups of these two launches, which always cover the WHOLE list and
// come before any tensor's LSTM state is rewritten
// (lstm_z: room for the LSTM's recurrent product, which then rides along in the first of them; null: not formed ahead)
void launch_rowcol_sums(const Launch&, const StepArgs&, const WeightsDev&, float* hbar_part, float* b_eff, float* lstm_z, hipStream_t);
void launch_rc_update(const Launch&, const StepArgs&, const WeightsDev&, float* hbar_part, float* b_eff, hipStream_t);
// short lists: the row/column sums on taller tiles, copying r_k and c_k aside
void launch_rowcol_short(const Launch&, const StepArgs&, const WeightsDev&, float* hbar_part, float* b_eff, float* lstm_z, hipStream_t);
// write_state = false: M_1..3 and V stay as they are (the strip-form apply pass updates them, see launch_apply_f16s). Short
// lists: the second stage of VeLO's cross-tensor term rides along here (there is no launch_rc_update)
void launch_accum_stats(const Launch&, const StepArgs&, const WeightsDev&, bool write_state, float* hbar_part, float* b_eff, hipStream_t);
void launch_finalize(const Launch&, const StepArgs&, const WeightsDev&, const StepFeats&, float* lstm_u, hipStream_t);
// lopt_create: fills WeightsDev::lstm and, if `head` is not null, WeightsDev::head
void launch_velo_pack(const WeightsDev&, int HL, int K, int P, float* lstm, float* head, hipStream_t);
// lstm_z: the recurrent product formed ahead (null: this launch forms it); feats not null: no k_finalize has run
void launch_velo_lstm(const Launch&, const StepArgs&, const WeightsDev&, const float* lstm_u, const float* b_eff,
                      const float* lstm_z, const StepFeats* feats, float* h_new, hipStream_t);
void launch_velo_head(const Launch&, const StepArgs&, const WeightsDev&, const float* h_new, float* alpha,
                      float* theta, hipStream_t);
void launch_apply_small_fc(const Launch&, const StepArgs&, const WeightsDev&, hipStream_t);
void launch_apply_velo(const Launch&, const StepArgs&, const WeightsDev&, hipStream_t);
bool apply_mfma_available(const StepArgs&);
void launch_apply_mfma(const Launch&, const StepArgs&, const WeightsDev&, hipStream_t);
bool apply_fc4x_available(const StepArgs&);
void launch_apply_fc4x(const Launch&, const StepArgs&, const WeightsDev&, bool update_state, hipStream_t);
bool apply_velo4_available(const StepArgs&);
void launch_apply_velo4(const Launch&, const StepArgs&, bool update_state, hipStream_t);
// feats not null: no k_finalize has run, every workgroup forms its tensor's scales and first layer (Plan::fold_finalize)
void launch_apply_f16s(const Launch&, const StepArgs&, const WeightsDev&, const StepFeats* feats, bool update_state, hipStream_t);

}  // namespace lopt
