// gfx950 kernels of the learned-optimizer step (paper: section "Optimized Kernel Design").
//
// The paper's two CUDA kernels (feature statistics; fused apply) are re-cut here into a
// fixed sequence of launches that each cover ALL tensors of the step through a table of
// work items (one workgroup = one tile of one tensor):
//   rowcol_sums  : per tile, sum of g^2 over the tile's columns (per row) and rows (per column)
//                  (+ VeLO: extra workgroups sum the tensors' previous LSTM outputs, slice by slice)
//   rc_update    : per row / per column: finish the means, update r_k, c_k, keep rsqrt(r_k+eps),
//                  rsqrt(c_k+eps), and partial sums for the row/column-constant features
//                  (+ VeLO: extra workgroups finish the cross-tensor mean and its gate contribution)
//   accum_stats  : M_i, V update + per-tile sums of squares of the per-element features
//   finalize     : per tensor, fixed-order reduction of all partials -> s_f, scale factors,
//                  first MLP layer with the normalization folded in (small_fc_lopt), LSTM input incl. time and
//                  loss features (VeLO)
//   velo_lstm, velo_head : the per-tensor hypernetwork (VeLO only)
//   apply        : rebuild features, MLP, exponentiated update (lopt_apply_mfma.hip has the
//                  matrix-core variant for hidden width 32)
// Short lists do without rc_update (k_rowcol_short leaves fewer partials, accum_stats finishes the means: fuse_means), the shortest
// also without finalize (the apply or LSTM launch reduces its partials itself: lopt_finalize.h).
// A tile is TR rows x 256 columns, and row indices are wave-uniform everywhere. Lane l holds the four consecutive columns
// 4l..4l+3 and a wavefront takes whole rows of the tile, in the statistics and VeLO apply passes in the order of row_walk; the
// sums and the statistics read rows off the 16-byte grid the same way (load_quad).
#include <stddef.h>

#include <type_traits>

#include "lopt_internal.h"
#include "lopt_device.h"
#include "lopt_finalize.h"

namespace lopt {

// ----------------------------------------------------------------------------- fill

__global__ void __launch_bounds__(kBlock) k_fill_zero(const TensorDev* __restrict__ tensors, int H2) {
  const TensorDev T = tensors[blockIdx.y];
  size_t total = 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn + (size_t)H2 * T.padH;
  size_t n4 = total / 4;  // every section is a multiple of 4 floats
  float4* dst = reinterpret_cast<float4*>(T.st);
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock)
    dst[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

void launch_fill_zero(const Launch& L, const StepArgs& A, hipStream_t s) {
  if (L.n_tensors == 0) return;
  // grid.y is limited to 65535: loop over slabs of tensors
  for (int t0 = 0; t0 < L.n_tensors; t0 += 32768) {
    int nt = L.n_tensors - t0 < 32768 ? L.n_tensors - t0 : 32768;
    hipLaunchKernelGGL(k_fill_zero, dim3(64, nt), dim3(kBlock), 0, s, L.tensors + t0,
                       A.kind == LOPT_VELO ? 2 : 0);
  }
}

// ----------------------------------------------------------------------------- VeLO cross-tensor term

// The cross-tensor input of VeLO's LSTM depends on nothing this step computes (it reads the LSTM outputs h the previous
// step left in the state blobs), so its two stages ride along as extra workgroups of the first two launches of the
// step instead of taking launches of their own: slice sums of h behind the tiles of k_rowcol_sums, the final mean and
// the gate bias b_eff = b + hbar Wg behind the row/column blocks of k_rc_update. Both have a fixed summation order.
struct MixArgs {
  const float* Wg;        // [HL][4 HL]
  const float* b;         // [4 HL]
  float* part;            // [n_slices][HL] slice sums of h
  float* b_eff;           // [kMixJSplit][4 HL]: hbar Wg summed over a quarter of the units j each
  int HL, n_tensors, per_slice, n_slices;   // n_slices == 0: not VeLO, no extra workgroups
  const float* lstm;      // WeightsDev::lstm
  float* z;               // the LSTM's recurrent product (null: not formed ahead)
};

// Workgroup (chunk of 64 units, slice of the tensor list): lane = unit j, the four wavefronts take every fourth tensor
// of the slice, four tensors in flight each, and meet in LDS.
__device__ __forceinline__ void mix_hbar_block(const TensorDev* __restrict__ tensors, const MixArgs& M, int blk,
                                               float (*red)[kWave]) {
  const int n_chunks = (M.HL + kWave - 1) / kWave;
  const int chunk = blk % n_chunks, slice = blk / n_chunks;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = min(chunk * kWave + lane, M.HL - 1);   // lanes past the end repeat the last unit (dropped below)
  const int t0 = slice * M.per_slice, t1 = min(t0 + M.per_slice, M.n_tensors);
  float a = 0.f;
  for (int t = t0 + wave; wave < 4 && t < t1; t += 16) {   // (k_rowcol_short has sixteen wavefronts)
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int tt = min(t + 4 * k, t1 - 1);
      const TensorDev& T = tensors[tt];
      v[k] = T.st[4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn + j];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) a += t + 4 * k < t1 ? v[k] : 0.f;
  }
  if (wave < 4) red[wave][lane] = a;
  __syncthreads();
  if (wave == 0 && chunk * kWave + lane < M.HL)
    M.part[(size_t)slice * M.HL + j] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Workgroup = 64 gate columns (lane = column: coalesced rows of Wg) x one quarter of the units j; its wavefronts
// take the units of the quarter in turn, eight rows in flight each, and meet in LDS in a fixed order. The quarters
// are added up (with the bias b) by k_velo_lstm, again in a fixed order.
__device__ __forceinline__ void mix_bias_block(const MixArgs& M, int blk, float* hbar, float (*red)[kWave]) {
  const int HL = M.HL, G = 4 * HL;
  const int n_colblk = (G + kWave - 1) / kWave;
  const int colblk = blk % n_colblk, quarter = blk / n_colblk;
  const int jq = (HL + kMixJSplit - 1) / kMixJSplit;
  const int j0 = quarter * jq, j1 = min(j0 + jq, HL);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int col = min(colblk * kWave + lane, G - 1);
  const float* __restrict__ wg = M.Wg + col;
  for (int j = j0 + (int)threadIdx.x; j < j1; j += (int)blockDim.x)
    hbar[j - j0] = (float)(strided_sum(M.part + j, M.n_slices, (size_t)HL) / (double)M.n_tensors);
  __syncthreads();
  float a = 0.f;
  for (int j = j0 + wave; j < j1; j += 8 * nw) {
    float w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = wg[(size_t)min(j + nw * k, j1 - 1) * G];
#pragma unroll
    for (int k = 0; k < 8; ++k) a += j + nw * k < j1 ? hbar[j + nw * k - j0] * w[k] : 0.f;
  }
  red[wave][lane] = a;
  __syncthreads();
  if (wave == 0 && colblk * kWave + lane < G) {
    float s = 0.f;
    for (int w = 0; w < nw; ++w) s += red[w][lane];
    M.b_eff[(size_t)quarter * G + col] = s;
  }
}

// The LSTM's recurrent product h W_h of the step before, formed here because it depends on nothing this step computes: what is
// left behind the statistics is the product of the 48 inputs (k_velo_lstm_tail). Workgroup = 16 tensors x 8 units x 4 gates, in
// front of the tiles of the row/column sums; its wavefronts share the octets of h slots and meet in LDS in a fixed order.
// v_mfma_f32_16x16x4_f32 (exact products) on two column tiles; 32 tensors at a time would double the chain of a short list. As
// extra workgroups of the statistics pass of a short list it is the longer side there (layer of 2000x2000 32 us instead of 26).
// Out: z[tensor][unit block][gate, unit].
constexpr int kRecurOctets = 4;   // octets in flight per wavefront
typedef float f32x16_l __attribute__((ext_vector_type(16)));
typedef float f32x4_l __attribute__((ext_vector_type(4)));

template <int WAVES>
__device__ __forceinline__ void lstm_recur_block(const TensorDev* __restrict__ tensors, const MixArgs& M, int blk,
                                                 float (*part)[kRecurTensors][32]) {
  const int HL = M.HL, n_ub = (HL + 7) / 8, ub = blk % n_ub, t0 = blk / n_ub * kRecurTensors;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int quarter = lane >> 4, l16 = lane & 15;   // A: tensor l16, slot of the quad; B: column l16, slot
  const int n_oct = lstm_k_pad(HL) / 8, first = kLstmInPad / 8;
  const float* __restrict__ wcol = M.lstm + ((size_t)ub * (8 * n_oct) + quarter) * 32 + l16;
  const TensorDev& T = tensors[min(t0 + l16, M.n_tensors - 1)];   // rows past the list compute on the last tensor and are dropped
  const float* __restrict__ h = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn;
  f32x4_l acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  const int per_wave = (n_oct - first + WAVES - 1) / WAVES;
  const int o_begin = first + wave * per_wave, o_end = min(o_begin + per_wave, n_oct);
  for (int ob = o_begin; ob < o_end; ob += kRecurOctets) {
    float a[kRecurOctets][2], b[kRecurOctets][2][2];
#pragma unroll
    for (int j = 0; j < kRecurOctets; ++j) {
      const int o = min(ob + j, o_end - 1);   // octets past the wavefront's share repeat its last one (dropped below)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        a[j][q] = h[min(8 * o + 4 * q + quarter - kLstmInPad, HL - 1)];   // slots past H_L: their weights are zero
#pragma unroll
        for (int c = 0; c < 2; ++c) b[j][q][c] = wcol[((size_t)o * 8 + 4 * q) * 32 + 16 * c];
      }
    }
#pragma unroll
    for (int j = 0; j < kRecurOctets; ++j) {
      if (ob + j >= o_end) break;   // wavefront-uniform
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][q], b[j][q][c], acc[c], 0, 0, 0);
    }
  }
  // accumulator register v of lane (quarter, column) is row 4 quarter + v
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][4 * quarter + v][16 * c + l16] = acc[c][v];
  __syncthreads();
  for (int i = threadIdx.x; i < kRecurTensors * 32; i += 64 * WAVES) {
    const int r = i >> 5, c = i & 31;
    float s[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) s[w] = part[w][r][c];
#pragma unroll
    for (int step = 1; step < WAVES; step *= 2)
#pragma unroll
      for (int w = 0; w < WAVES; w += 2 * step) s[w] += s[w + step];
    if (t0 + r < M.n_tensors) M.z[((size_t)(t0 + r) * n_ub + ub) * 32 + c] = s[0];
  }
}

// Extra workgroups of the row/column sums (slices of the mean; the recurrent product, if it is formed ahead) and of the launch
// that forms the gate bias.
inline int mix_hbar_blocks(const MixArgs& M) { return M.n_slices * ((M.HL + kWave - 1) / kWave); }
inline int mix_bias_blocks(const MixArgs& M) { return M.n_slices ? kMixJSplit * ((4 * M.HL + kWave - 1) / kWave) : 0; }
inline int recur_blocks(const MixArgs& M) {
  return M.n_slices && M.z ? (M.n_tensors + kRecurTensors - 1) / kRecurTensors * ((M.HL + 7) / 8) : 0;
}

static MixArgs make_mix(const Launch& L, const StepArgs& A, const WeightsDev& W, float* hbar_part, float* b_eff, float* lstm_z = nullptr) {
  MixArgs M{};
  if (A.kind != LOPT_VELO || L.n_tensors == 0) return M;
  M.Wg = W.Wg; M.b = W.b; M.part = hbar_part; M.b_eff = b_eff;
  M.lstm = W.lstm; M.z = lstm_z;
  M.HL = A.HL; M.n_tensors = L.n_tensors;
  int per_slice = (L.n_tensors + kMixSlices - 1) / kMixSlices;
  if (per_slice < 16) per_slice = 16;   // four tensors in flight on each of four wavefronts
  M.per_slice = per_slice;
  M.n_slices = (L.n_tensors + per_slice - 1) / per_slice;
  return M;
}

// ----------------------------------------------------------------------------- rowcol_sums

// NT: nontemporal loads. R: rows in flight per wavefront.
template <bool NT, int R>
__device__ __forceinline__ void rowcol_tile(const TensorDev& T, const TileDev& tile, float* __restrict__ ws,
                                            float (*colred)[kTileCols]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = T.n, m = T.m;
  const int c0 = tile.tj * kTileCols;
  const unsigned bytes = segment_bytes(n, c0);
  auto row4 = [&](unsigned r) __attribute__((always_inline)) {   // past the last column: zeros
    return load_quad<NT>(T.g + ((size_t)r * (unsigned)n + c0), 16u * lane, bytes);
  };
  const auto [r0, r1] = tile_rows(T, tile);
  float* __restrict__ rowpart = ws + T.oRowPart + (size_t)tile.tj * m;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  for (unsigned r = r0 + wave; r < r1; r += 4 * R) {
    f32x4v v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = row4(min(r + 4 * i, r1 - 1));   // rows past the tile: its last row, counted as 0
    float sum[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const float ax = v[i].x * v[i].x, ay = v[i].y * v[i].y, az = v[i].z * v[i].z, aw = v[i].w * v[i].w;
      const bool in = r + 4 * i < r1;   // wavefront-uniform
      s0 += in ? ax : 0.f; s1 += in ? ay : 0.f; s2 += in ? az : 0.f; s3 += in ? aw : 0.f;
      sum[i] = wave_sum((ax + ay) + (az + aw));
    }
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (r + 4 * i < r1) rowpart[r + 4 * i] = sum[i];
    }
  }
  *reinterpret_cast<float4*>(&colred[wave][4 * lane]) = make_float4(s0, s1, s2, s3);
  __syncthreads();
  const int c = tile.tj * kTileCols + threadIdx.x;
  if (c < n) {
    float s = (colred[0][threadIdx.x] + colred[1][threadIdx.x]) + (colred[2][threadIdx.x] + colred[3][threadIdx.x]);
    ws[T.oColPart + (size_t)tile.ti * n + c] = s;
  }
}

__global__ void __launch_bounds__(kBlock) k_rowcol_sums(const TensorDev* __restrict__ tensors,
                                                        const TileDev* __restrict__ tiles, float* __restrict__ ws,
                                                        int n_tiles, MixArgs M, int n_recur) {
  __shared__ union alignas(16) { float col[4][kTileCols], hbar[4][kWave], z[4][kRecurTensors][32]; } red;
  const int blk = (int)blockIdx.x - n_recur;
  if (blk < 0) {   // the extra workgroups of a VeLO step: recurrent product, slice sums of the LSTM outputs
    lstm_recur_block<4>(tensors, M, (int)blockIdx.x, red.z);
    return;
  }
  if (blk >= n_tiles) {
    mix_hbar_block(tensors, M, blk - n_tiles, red.hbar);
    return;
  }
  float (*colred)[kTileCols] = red.col;
  const TileDev tile = tiles[blk];
  const TensorDev& T = tensors[tile.tensor];
  if (T.n <= kNarrowCols) rowcol_tile<false, 8>(T, tile, ws, colred);
  else if (T.vec) rowcol_tile<true, 2>(T, tile, ws, colred);
  else rowcol_tile<false, 2>(T, tile, ws, colred);   // off the grid neighbours share lines
}

void launch_rowcol_sums(const Launch& L, const StepArgs& A, const WeightsDev& W, float* hbar_part, float* b_eff, float* lstm_z,
                        hipStream_t s) {
  if (L.n_tiles == 0) return;
  const MixArgs M = make_mix(L, A, W, hbar_part, b_eff, lstm_z);
  const int n_recur = recur_blocks(M);
  hipLaunchKernelGGL(k_rowcol_sums, dim3(n_recur + L.n_tiles + mix_hbar_blocks(M)), dim3(kBlock), 0, s, L.tensors, L.tiles, L.ws,
                     L.n_tiles, M, n_recur);
}

// Short lists: tiles of short_rows rows, sixteen wavefronts with four or eight rows in flight each, so that a column has few partial sums
// and every workgroup of the statistics pass can add them up itself (fuse_means). r_k and c_k are copied aside for it: the
// statistics pass writes the new ones while other workgroups still need the old.
constexpr int kShortWaves = 16;

// [ceil(m / short_rows)][n] sums of g^2 over a tile's rows, added up over the wavefronts and kept in double: there are few of them, and
// rounded to fp32 they would make the column means less exact than the sums over tiles of eight rows that lists of this length had
// before (rms error of a mean of 128 rows 4.3e-8 with fp32 sums of 64 rows, 2.9e-8 of eight).
template <typename F>
__device__ __forceinline__ auto short_colpart(const TensorDev& T, F* ws) {
  return reinterpret_cast<std::conditional_t<std::is_const_v<F>, const double, double>*>(ws + T.oColPart);
}

// R: rows per wavefront.
template <int R>
__device__ __forceinline__ void rowcol_short_tile(const TensorDev& T, const TileDev& tile, float* __restrict__ ws,
                                                  float (*colred)[kTileCols]) {
  constexpr int kRows = R * kShortWaves;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = T.n, m = T.m, c0 = tile.tj * kTileCols;
  const int r0 = tile.ti * kRows, r1 = min(r0 + kRows, m);
  f32x4v v[R];
  const unsigned bytes = segment_bytes(n, c0);
#pragma unroll
  for (int i = 0; i < R; ++i)   // rows past the tile: its last row, counted as 0
    v[i] = load_quad<false>(T.g + ((size_t)min(r0 + wave + kShortWaves * i, r1 - 1) * (unsigned)n + c0), 16u * lane, bytes);
  const float* rst = T.st + 4 * (size_t)T.padN;   // r_k[3][padm], c_k[3][padn]
  const int t = threadIdx.x;
  if (tile.tj == 0 && t < 3 * kRows) {
    const size_t at = (size_t)(t / kRows) * T.padm + r0 + t % kRows;
    if (r0 + t % kRows < m) ws[T.oRR + 3 * (size_t)T.padm + at] = rst[at];
  }
  if (tile.ti == 0 && t >= kTileCols) {
    const int k = t / kTileCols - 1, c = c0 + t % kTileCols;
    if (c < n) ws[T.oRC + (size_t)(3 + k) * T.padn + c] = rst[3 * (size_t)T.padm + (size_t)k * T.padn + c];
  }
  float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int r = r0 + wave + kShortWaves * i;   // wavefront-uniform
    if (r < r1) {
      const float ax = v[i].x * v[i].x, ay = v[i].y * v[i].y, az = v[i].z * v[i].z, aw = v[i].w * v[i].w;
      s[0] += ax; s[1] += ay; s[2] += az; s[3] += aw;
      const float sum = wave_sum((ax + ay) + (az + aw));
      if (lane == 0) ws[T.oRowPart + (size_t)tile.tj * m + r] = sum;
    }
  }
  *reinterpret_cast<float4*>(&colred[wave][4 * lane]) = make_float4(s[0], s[1], s[2], s[3]);
  __syncthreads();
  const int c = c0 + t;
  if (t < kTileCols && c < n) {
    double x[kShortWaves];
#pragma unroll
    for (int w = 0; w < kShortWaves; ++w) x[w] = (double)colred[w][t];
#pragma unroll
    for (int step = 1; step < kShortWaves; step *= 2)
#pragma unroll
      for (int w = 0; w < kShortWaves; w += 2 * step) x[w] += x[w + step];
    short_colpart(T, ws)[(size_t)tile.ti * n + c] = x[0];
  }
}

__global__ void __launch_bounds__(kWave * kShortWaves) k_rowcol_short(const TensorDev* __restrict__ tensors,
                                                                      const TileDev* __restrict__ tiles, float* __restrict__ ws,
                                                                      int n_tiles, MixArgs M, int n_recur, int* __restrict__ counters) {
  if (blockIdx.x == 0 && threadIdx.x < kMaxGroups) counters[threadIdx.x] = 0;   // k_finalize does it on other lists
  __shared__ union alignas(16) { float col[kShortWaves][kTileCols], hbar[4][kWave], z[kShortWaves][kRecurTensors][32]; } red;
  const int blk = (int)blockIdx.x - n_recur;
  if (blk < 0) {
    lstm_recur_block<kShortWaves>(tensors, M, (int)blockIdx.x, red.z);
    return;
  }
  if (blk >= n_tiles) {
    mix_hbar_block(tensors, M, blk - n_tiles, red.hbar);
    return;
  }
  float (*colred)[kTileCols] = red.col;
  const TileDev tile = tiles[blk];
  const TensorDev& T = tensors[tile.tensor];
  constexpr int R = 64 / kShortWaves;
  if (short_rows(T.m, M.n_slices > 0) == 64) rowcol_short_tile<R>(T, tile, ws, colred);
  else rowcol_short_tile<2 * R>(T, tile, ws, colred);
}

void launch_rowcol_short(const Launch& L, const StepArgs& A, const WeightsDev& W, float* hbar_part, float* b_eff, float* lstm_z,
                         hipStream_t s) {
  if (L.n_rctiles == 0) return;
  const MixArgs M = make_mix(L, A, W, hbar_part, b_eff, lstm_z);
  const int n_recur = recur_blocks(M);
  hipLaunchKernelGGL(k_rowcol_short, dim3(n_recur + L.n_rctiles + mix_hbar_blocks(M)), dim3(kWave * kShortWaves), 0, s, L.tensors,
                     L.rctiles, L.ws, L.n_rctiles, M, n_recur, L.apply_counter);
}

// ----------------------------------------------------------------------------- rc_update

// Sums over the workgroup's first four wavefronts (256 threads) of NV values per thread, to out[0..NV). A tree throughout: four values
// are folded into one register while the four lanes of a quad are added up (lane l ends with value l & 3), the quads of a row
// of 16 lanes by rotations, the sixteen rows in LDS. A tree per value over the whole wavefront takes three times the instructions, and
// on a short list they are a fifth of the statistics pass (toy list of three tensors: 1.1 of 6.8 us, now 0.5).
constexpr int kRedStride = 20;   // floats: sixteen rows, and two lanes at most on a bank
template <int NV>
__device__ __forceinline__ void block_sum(const float (&v)[NV], float (*red)[kRedStride], float* out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int N16 = NV < 16 ? NV : 16, Q = (N16 + 3) / 4;
  if (wave < 4) {
    const int row = 4 * wave + (lane >> 4), q = lane & 15;
    const bool b0 = lane & 1, b1 = lane & 2;
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i >= Q) { s[i] = 0.f; continue; }
      const float x0 = v[4 * i], x1 = 4 * i + 1 < N16 ? v[4 * i + 1] : 0.f;
      const float x2 = 4 * i + 2 < N16 ? v[4 * i + 2] : 0.f, x3 = 4 * i + 3 < N16 ? v[4 * i + 3] : 0.f;
      const float y0 = (b0 ? x1 : x0) + dpp_f<0xB1>(b0 ? x0 : x1);   // lane ^ 1
      const float y1 = (b0 ? x3 : x2) + dpp_f<0xB1>(b0 ? x2 : x3);
      float t = (b1 ? y1 : y0) + dpp_f<0x4E>(b1 ? y0 : y1);          // lane ^ 2
      t += dpp_f<0x124>(t);                                          // rotations by 4 and 8 within the row
      s[i] = t + dpp_f<0x128>(t);
    }
    const float lo = lane & 4 ? s[1] : s[0], hi = lane & 4 ? s[3] : s[2];
    if (q < N16) red[q][row] = lane & 8 ? hi : lo;
#pragma unroll
    for (int j = 16; j < NV; ++j) {
      float t = v[j];
      t += dpp_f<0xB1>(t);
      t += dpp_f<0x4E>(t);
      t += dpp_f<0x124>(t);
      t += dpp_f<0x128>(t);
      if (q == 0) red[j][row] = t;
    }
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const float4* r = reinterpret_cast<const float4*>(red[threadIdx.x]);
    float4 a = r[0], b = r[1], c = r[2], d = r[3];
    out[threadIdx.x] = (((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w))) +
                       (((c.x + c.y) + (c.z + c.w)) + ((d.x + d.y) + (d.z + d.w)));
  }
}

// The same sum formed by the whole workgroup (for one row or column at a time): thread t adds every blockDim-th term from t on
// in index order, then a fixed tree over the threads. Every thread gets the result. For tensors of extreme aspect
// ratio (a 1 x 2^28 vector has a million column tiles): one lane summing them all would take milliseconds.
__device__ __forceinline__ double strided_sum_coop(const float* __restrict__ part, int count, size_t stride, double* tree) {
  double a = 0.0;
  const int nt = blockDim.x;
  int j = threadIdx.x;
  for (; j + 7 * nt < count; j += 8 * nt) {
    float t[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = part[(size_t)(j + k * nt) * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) a += (double)t[k];
  }
  for (; j < count; j += nt) a += (double)part[(size_t)j * stride];
  __syncthreads();   // the previous use of the tree is over
  tree[threadIdx.x] = a;
  __syncthreads();
  for (int w = nt / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) tree[threadIdx.x] += tree[threadIdx.x + w];
    __syncthreads();
  }
  return tree[0];
}

// A block of rows (or columns) takes the cooperative sum when there are at least 64 partials per row of the block and
// more than 512 in all (decided by the shapes alone, so a given tensor list always takes the same path).
__device__ __forceinline__ bool rc_sum_coop(int count, int valid) { return count > 512 && count >= 64 * valid; }

__device__ __forceinline__ float new_factor(const StepArgs& A, int k, float old, float mean) {
  return A.fac_decay[k] * old + (1.0f - A.fac_decay[k]) * mean;
}

// One row or column: writes its three accumulators and their reciprocal roots, and leaves the nine values that its block sums.
template <typename V>
__device__ __forceinline__ void finish_factors(const StepArgs& A, const float (&old)[3], float mean, float* acc3, float* inv3, size_t pd,
                                               V (&v)[9]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float r = new_factor(A, k, old[k], mean), rr = rsqrtf(r + A.eps_acc);
    acc3[(size_t)k * pd] = r;
    inv3[(size_t)k * pd] = rr;
    v[k] = r;   // (the columns' plain sum is not used)
    v[3 + k] = (V)r * r;
    v[6 + k] = (V)rr * rr;
  }
}

// Workgroup = a block of 256 rows (or columns) of one tensor; the first 256 threads finish one row each. On short lists it
// has 1024 threads, which sum each row's partials as four interleaved quarters that meet in LDS in a fixed order: the
// kernel is a chain of load latencies (125 partials a column, 1000x1000: 7.2 -> 5.5 us with one batch of loads, not eight).
constexpr int kRcMaxThreads = 4 * kBlock;
__global__ void __launch_bounds__(kRcMaxThreads) k_rc_update(const TensorDev* __restrict__ tensors,
                                                      const RcItemDev* __restrict__ items, float* __restrict__ ws,
                                                      StepArgs A, int n_items, MixArgs M) {
  __shared__ __align__(16) float red[9][kRedStride];
  __shared__ double tree[kRcMaxThreads];
  if ((int)blockIdx.x >= n_items) {   // the extra workgroups of a VeLO step: mean of the LSTM outputs, gate bias
    __shared__ float hbar[1024];
    __shared__ float mred[kRcMaxThreads / kWave][kWave];
    mix_bias_block(M, (int)blockIdx.x - n_items, hbar, mred);
    return;
  }
  const RcItemDev it = items[blockIdx.x];
  const TensorDev& T = tensors[it.tensor];
  const int i = threadIdx.x & (kBlock - 1), quarter = threadIdx.x / kBlock, nq = blockDim.x / kBlock;
  const int idx = it.blk * kBlock + i;
  float v[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) v[q] = 0.f;
  float* st = T.st;
  const int dim = it.is_col ? T.n : T.m, count = it.is_col ? T.nrt : T.nct;
  const int valid = min(kBlock, dim - it.blk * kBlock);
  const float* __restrict__ pbase = ws + (it.is_col ? T.oColPart : T.oRowPart) + (size_t)it.blk * kBlock;
  // the three accumulators of this row or column, ahead of the sums
  const size_t pd = it.is_col ? T.padn : T.padm;
  float* acc3 = st + 4 * (size_t)T.padN + (it.is_col ? 3 * (size_t)T.padm : 0) + idx;
  float* inv3 = ws + (it.is_col ? T.oRC : T.oRR) + idx;
  const bool mine = quarter == 0 && idx < dim;
  float old[3] = {0.f, 0.f, 0.f};
  if (mine)
#pragma unroll
    for (int k = 0; k < 3; ++k) old[k] = acc3[(size_t)k * pd];
  double acc = 0.0;
  if (rc_sum_coop(count, valid)) {   // workgroup-uniform
    for (int r = 0; r < valid; ++r) {
      const double v1 = strided_sum_coop(pbase + r, count, (size_t)dim, tree);
      if (i == r) acc = v1;
    }
  } else {
    if (idx < dim && quarter < count)
      acc = strided_sum(pbase + i + (size_t)quarter * dim, (count - quarter + nq - 1) / nq, (size_t)nq * dim);
    if (count > 1 && nq > 1) {   // workgroup-uniform
      tree[threadIdx.x] = acc;
      __syncthreads();
      if (quarter == 0) acc = (tree[i] + tree[kBlock + i]) + (tree[2 * kBlock + i] + tree[3 * kBlock + i]);
    }
  }
  if (mine) finish_factors(A, old, (float)(acc / (double)(it.is_col ? T.m : T.n)), acc3, inv3, pd, v);
  const int slot = it.is_col ? T.nrpart + it.blk : it.blk;
  block_sum<9>(v, red, ws + T.oRcPart + (size_t)slot * kRcStride);
}

void launch_rc_update(const Launch& L, const StepArgs& A, const WeightsDev& W, float* hbar_part, float* b_eff,
                      hipStream_t s) {
  if (L.n_rcitems == 0) return;
  const MixArgs M = make_mix(L, A, W, hbar_part, b_eff);
  const int extra = mix_bias_blocks(M);
  // The wide form shortens the chain of loads; on longer lists its workgroups no longer all fit on the chip at once and its
  // idle wavefronts cost more than that (2219 tensors: 46 us narrow, 154 us wide).
  const int threads = L.n_rcitems + extra <= 512 ? kRcMaxThreads : kBlock;
  hipLaunchKernelGGL(k_rc_update, dim3(L.n_rcitems + extra), dim3(threads), 0, s, L.tensors, L.rcitems, L.ws, A,
                     L.n_rcitems, M);
}

// ----------------------------------------------------------------------------- accum_stats

// Short lists: the row and column means that k_rc_update finishes on others, formed by every statistics workgroup for its own
// rows and columns (the sums in double, in index order). The new r_k and c_k and their partial sums are written by workgroups of
// their own (short_rc_block): at the end of the tiles of the first row and column they made the launch 1.1 to 2.2 us longer. They
// come behind the tiles where the chip holds those at once, and in front where it does not and they would be its last round (us a
// step under VeLO, in front / behind, 6 tensors of 0.33 M elements 33.8 / 33.2, 66 of 2.4 M, 1180 tiles, 59.0 / 55.8, 4 M, 2000 tiles,
// 75.1 / 75.1; 17 M, 4200 tiles, 191 / 196).
struct alignas(16) FuseLds {
  float rr[3][kShortRows];   // rsqrt(r_k + eps) of the tile's rows
  float rc[3][kTileCols];
};

// Sums of the partials of a row and of a column.
__device__ __forceinline__ double short_row_sum(const TensorDev& T, const float* __restrict__ ws, int r) {
  return strided_sum(ws + T.oRowPart + r, T.nct, (size_t)T.m);
}
__device__ __forceinline__ double short_col_sum(const TensorDev& T, const float* __restrict__ ws, const StepArgs& A, int c) {
  const int sr = short_rows(T.m, A.kind == LOPT_VELO);
  return strided_sum(short_colpart(T, ws) + c, (T.m + sr - 1) / sr, (size_t)T.n);
}

union ShortLds {
  FuseLds means;
  double rc[9][kBlock / kWave];
  struct { float hbar[1024 / kMixJSplit], red[kBlock / kWave][kWave]; } mix;   // a quarter of at most 1024 units
};

__device__ __forceinline__ void fuse_means(const TensorDev& T, const TileDev& tile, const float* __restrict__ ws, const StepArgs& A,
                                           FuseLds& L) {
  const int t = threadIdx.x, n = T.n, m = T.m;
  const int c = tile.tj * kTileCols + t, r = tile.ti * T.TR + t;
  const bool cin = c < n, rin = t < T.TR && r < m;
  float co[3] = {0.f, 0.f, 0.f}, ro[3] = {0.f, 0.f, 0.f};
  if (rin)
#pragma unroll
    for (int k = 0; k < 3; ++k) ro[k] = ws[T.oRR + (size_t)(3 + k) * T.padm + r];
  if (cin)
#pragma unroll
    for (int k = 0; k < 3; ++k) co[k] = ws[T.oRC + (size_t)(3 + k) * T.padn + c];
  double rs = 0.0, cs = 0.0;
  if (rin) rs = short_row_sum(T, ws, r);
  if (cin) {
    cs = short_col_sum(T, ws, A, c);
    const float mean = (float)(cs / (double)m);
#pragma unroll
    for (int k = 0; k < 3; ++k) L.rc[k][t] = rsqrtf(new_factor(A, k, co[k], mean) + A.eps_acc);
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) L.rc[k][t] = 0.f;   // columns past the last one of a ragged row
  }
  if (rin) {
    const float mean = (float)(rs / (double)n);
#pragma unroll
    for (int k = 0; k < 3; ++k) L.rr[k][t] = rsqrtf(new_factor(A, k, ro[k], mean) + A.eps_acc);
  }
  __syncthreads();
}

// 256 rows or columns of a tensor: what k_rc_update does on longer lists, from the partial sums of short ones. Their nine sums are
// doubles, handed on as two floats: few blocks make up a tensor here, so that the rounding of each would be as large as that of the
// statistic (256 rows in fp32 4.6e-8, 1000 rows 2.4e-8; partials of 8 rows each, which these blocks replace, 3.6e-9).
__device__ __forceinline__ void short_rc_block(const TensorDev& T, const RcItemDev& it, float* __restrict__ ws, const StepArgs& A,
                                               double (*red)[kBlock / kWave]) {
  const int idx = it.blk * kBlock + (int)threadIdx.x, dim = it.is_col ? T.n : T.m;
  const size_t pd = it.is_col ? T.padn : T.padm;
  float* acc3 = T.st + 4 * (size_t)T.padN + (it.is_col ? 3 * (size_t)T.padm : 0) + idx;
  float* inv3 = ws + (it.is_col ? T.oRC : T.oRR) + idx;
  double v[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) v[q] = 0.0;
  if (idx < dim) {
    float old[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) old[k] = acc3[(size_t)k * pd];
    const double sum = it.is_col ? short_col_sum(T, ws, A, idx) : short_row_sum(T, ws, idx);
    finish_factors(A, old, (float)(sum / (double)(it.is_col ? T.m : T.n)), acc3, inv3, pd, v);
  }
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const double s = wave_sum(v[q]);
    if (t % kWave == 0) red[q][t / kWave] = s;
  }
  __syncthreads();
  if (t < 9) {
    const double s = (red[t][0] + red[t][1]) + (red[t][2] + red[t][3]);
    const float hi = (float)s, lo = isinf(hi) ? 0.f : (float)(s - (double)hi);   // beyond fp32 the sum is infinite, as on longer lists
    float* part = ws + T.oRcPart + (size_t)((it.is_col ? T.nrpart : 0) + 2 * it.blk) * kRcStride + t;
    part[0] = hi;
    part[kRcStride] = lo;
  }
}

// The per-element features that need a statistic of their own (the row/column-constant ones
// follow from r_k, c_k alone). rrc[k] = rsqrt(r_k[i]+eps) * rsqrt(c_k[j]+eps); the common
// factor sqrt(mean(r_k)+eps) of the factored features is applied per tensor in k_finalize.
// Streaming accesses of this pass on long lists: nontemporal loads, ordinary stores (measured: 0.649 ms on the ViT-B/16 set
// against 0.670 plain/plain, 0.670 plain/nontemporal, 0.680 nontemporal/nontemporal); what is worth keeping in the cache for
// the apply pass is read with ordinary loads (choose_loads in lopt_plan.h).

// What one element adds to the sums. Every feature is formed before it is squared: the squares of its factors leave the fp32
// range long before the feature does ((g a_i b_j)^2 taken as g^2 (a_i^2 b_j^2) and M_i^2 / (V+eps): 0.3 % off for gradients of 1e-19, wrong
// altogether below 1e-21 and above 1e11, NaN for a gradient of zeros where eps_acc is below 5e-20). Products of squares save nine of some
// fifty vector instructions an element, but these streams wait for memory. us a step, squares / this way: 1000x1000 35.3 / 34.5,
// 8.2 M elements of 1531 columns 180 / 179, 54 M of 2731 under VeLO 779 / 778, ViT-B/16 shapes under VeLO 1130 / 1130; beside the apply pass
// of another tensor group, which wants the vector units too, ViT-B/16 shapes 1480 / 1483.5, 355 M elements 5865 / 5881.
__device__ __forceinline__ void add_squares(float (&acc)[kNStat], float g, float g2, float p, const float (&m)[3], float v, float rs,
                                            const float (&f)[3]) {
  const float clip2 = 0.1f * 0.1f;   // clip(g, +-0.1)^2 = min(g^2, 0.01)
  acc[0] += g2;
  acc[1] += p * p;
  acc[5] += v * v;
  acc[9] += rs * rs;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float mn = m[k] * rs, gf = g * f[k], mf = m[k] * f[k];
    acc[2 + k] += m[k] * m[k];
    acc[6 + k] += mn * mn;
    acc[10 + k] += gf * gf;
    acc[13 + k] += mf * mf;
  }
  acc[16] += fminf(g2, clip2);
}

// A lane holds four consecutive columns of a row; lanes past the last column sit the tile out and nothing in the loop is
// predicated. RAW_RSQ: the bare v_rsq_f32 (it treats inputs below the smallest normal float as zero, so the launcher asks for it
// only when eps_acc >= 1e-30).
// In the last lane of a ragged row the columns past the end hold zeros, which add nothing to any sum but that of 1/(V+eps), which is set
// to zero there. Rows off the 16-byte grid, four columns a lane against one column a lane in 64-column segments, us a step: 8.3 M
// elements of 1531 columns 189 -> 183, width 16 143 -> 135.5, VeLO 153 -> 147.5; 54 M of 2731 columns under VeLO 838 -> 811 (with the
// sums); 0.4 M under VeLO 37 -> 34.3. NT: nontemporal loads (Plan::keep).
template <bool RAW_RSQ, bool WRITE, bool FUSE, bool NT>
__device__ __forceinline__ void accum_tile(const TensorDev& T, const TileDev& tile, float* __restrict__ ws,
                                               const StepArgs& A, float (&acc)[kNStat], FuseLds* L) {
  const int lane = threadIdx.x & 63;
  const int n = T.n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowWalk w = FUSE ? plain_walk(T, tile, wave) : row_walk(T, tile, wave);   // FUSE: the means in LDS are the tile's own
  const int c0 = w.tj * kTileCols, col = c0 + 4 * lane, ncol = n - col;   // ncol: 4 or more but in a ragged row's last lane and beyond it
  const unsigned bytes = segment_bytes(n, c0);
  const bool mine = ncol > 0 && w.cnt > 0;
  if (!FUSE && !mine) return;
  // The first row's loads leave before the column factors are waited for: a short list's tile is one or two rows a wavefront
  // (toy list of three tensors 30.3 -> 29.6 us a step, 1000x1000 46.5 -> 45.6). The read-only form also needs 63 registers
  // this way instead of 66: eight wavefronts per SIMD (ViT-B/16 shapes beside the apply pass 1.488 -> 1.472 ms a step).
  struct Row { f32x4v g4, p4, m1, m2, m3, v4; size_t ro; int r; };
  const size_t pN = T.padN;
  auto load = [&](int i, Row& x) __attribute__((always_inline)) {
    x.r = walk_row(w, i);
    const size_t ro = x.ro = (size_t)x.r * n + c0;   // rows on the grid: a multiple of 4, and every section starts 16-byte aligned
    x.g4 = load_quad<NT>(T.g + ro, 16u * lane, bytes);
    x.p4 = load_quad<NT>(T.p + ro, 16u * lane, bytes);
    x.m1 = load_quad<NT>(T.st + ro, 16u * lane, bytes);
    x.m2 = load_quad<NT>(T.st + pN + ro, 16u * lane, bytes);
    x.m3 = load_quad<NT>(T.st + 2 * pN + ro, 16u * lane, bytes);
    x.v4 = load_quad<NT>(T.st + 3 * pN + ro, 16u * lane, bytes);
  };
  Row row;
  float4 c3[3];
  if (FUSE) {
    if (mine) load(0, row);
    fuse_means(T, tile, ws, A, *L);
    if (!mine) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) c3[k] = *reinterpret_cast<const float4*>(&L->rc[k][4 * lane]);
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) c3[k] = *reinterpret_cast<const float4*>(ws + T.oRC + (size_t)k * T.padn + col);
    load(0, row);
  }
  float rc[3][4];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float4 c = c3[k];
    rc[k][0] = c.x; rc[k][1] = c.y; rc[k][2] = c.z; rc[k][3] = c.w;
    if (!FUSE)   // (LDS holds zeros there)
#pragma unroll
      for (int e = 1; e < 4; ++e) rc[k][e] = e < ncol ? rc[k][e] : 0.f;
  }
  const float b1 = A.mom_decay[0], b2 = A.mom_decay[1], b3 = A.mom_decay[2], b4 = A.rms_decay;
  const float a1 = 1.0f - b1, a2 = 1.0f - b2, a3 = 1.0f - b3, a4 = 1.0f - b4;
  const float eps = A.eps_acc;
  auto add = [&](const Row& x) __attribute__((always_inline)) {
    const auto& [g4, p4, m1, m2, m3, v4, ro, r] = x;
    float rr[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) rr[k] = FUSE ? L->rr[k][r - tile.ti * T.TR] : ws[T.oRR + (size_t)k * T.padm + r];
    f32x4v o1, o2, o3, ov;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float g = g4[e], p = p4[e];
      const float g2 = g * g;
      // explicit fused multiply-adds: the apply pass may form the same values again (lopt_state_pass), bit for bit
      const float nm1 = __builtin_fmaf(b1, m1[e], a1 * g);
      const float nm2 = __builtin_fmaf(b2, m2[e], a2 * g);
      const float nm3 = __builtin_fmaf(b3, m3[e], a3 * g);
      const float nv = __builtin_fmaf(b4, v4[e], a4 * g2);
      o1[e] = nm1; o2[e] = nm2; o3[e] = nm3; ov[e] = nv;
      float rs = RAW_RSQ ? __builtin_amdgcn_rsqf(nv + eps) : rsqrtf(nv + eps);
      if (e > 0) rs = e < ncol ? rs : 0.f;
      add_squares(acc, g, g2, p, {nm1, nm2, nm3}, nv, rs, {rr[0] * rc[0][e], rr[1] * rc[1][e], rr[2] * rc[2][e]});
    }
    if (WRITE) {
      store_quad<false>(T.st + ro, 16u * lane, bytes, o1);
      store_quad<false>(T.st + pN + ro, 16u * lane, bytes, o2);
      store_quad<false>(T.st + 2 * pN + ro, 16u * lane, bytes, o3);
      store_quad<false>(T.st + 3 * pN + ro, 16u * lane, bytes, ov);
    }
  };
  for (int i = 0;;) {
    add(row);
    // Beside the apply pass of another tensor group there is room for 64 registers: the sums are pinned here, or the compiler
    // moves the next row's loads in front of them (95 registers, ViT-B/16 shapes 1.472 -> 1.547 ms a step). Without such a
    // neighbour that order is as good or 1 % better.
    if (!FUSE)
      asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]),
                   "+v"(acc[7]), "+v"(acc[8]), "+v"(acc[9]), "+v"(acc[10]), "+v"(acc[11]), "+v"(acc[12]), "+v"(acc[13]),
                   "+v"(acc[14]), "+v"(acc[15]), "+v"(acc[16]) :: "memory");
    if (++i >= w.cnt) break;
    load(i, row);
  }
}

// Narrow tensors: one column a lane (NarrowWalk), the same sums. A row past the tile adds nothing: its values read as 0.
constexpr int kNarrowTrip = 2;   // accesses in flight
template <bool RAW_RSQ, bool WRITE, bool FUSE>
__device__ __forceinline__ void accum_narrow(const TensorDev& T, const TileDev& tile, float* __restrict__ ws, const StepArgs& A,
                                             float (&acc)[kNStat], FuseLds* L) {
  if (FUSE) fuse_means(T, tile, ws, A, *L);
  const int n = T.n;
  const NarrowWalk w(n, kNarrowTrip);
  if (!w.col_ok) return;
  const auto [r0, r1] = tile_rows(T, tile);
  const size_t pN = T.padN;
  const float b1 = A.mom_decay[0], b2 = A.mom_decay[1], b3 = A.mom_decay[2], b4 = A.rms_decay;
  const float a1 = 1.0f - b1, a2 = 1.0f - b2, a3 = 1.0f - b3, a4 = 1.0f - b4;
  const float eps = A.eps_acc;
  float rc[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) rc[k] = FUSE ? L->rc[k][w.col] : ws[T.oRC + (size_t)k * T.padn + w.col];
  for (unsigned r = r0 + w.first; r < r1; r += w.step) {
    float in[kNarrowTrip][6], rr[kNarrowTrip][3];
    const size_t ro = (size_t)r * (unsigned)n;
    const unsigned bytes = 4u * (unsigned)n * min(r1 - r, (unsigned)(kNarrowTrip * w.rows));   // of the rows this trip takes
#pragma unroll
    for (int e = 0; e < kNarrowTrip; ++e) {
      const unsigned off = w.off + 4u * (unsigned)(e * w.rows * n);
      in[e][0] = load_one(T.g + ro, off, bytes);
      in[e][1] = load_one(T.p + ro, off, bytes);
#pragma unroll
      for (int k = 0; k < 4; ++k) in[e][2 + k] = load_one(T.st + k * pN + ro, off, bytes);
      const unsigned row = min(r + e * w.rows + w.sub, r1 - 1);
#pragma unroll
      for (int k = 0; k < 3; ++k) rr[e][k] = FUSE ? L->rr[k][row - r0] : ws[T.oRR + (size_t)k * T.padm + row];
    }
#pragma unroll
    for (int e = 0; e < kNarrowTrip; ++e) {
      const float g = in[e][0], p = in[e][1], g2 = g * g;
      const float nm1 = __builtin_fmaf(b1, in[e][2], a1 * g);
      const float nm2 = __builtin_fmaf(b2, in[e][3], a2 * g);
      const float nm3 = __builtin_fmaf(b3, in[e][4], a3 * g);
      const float nv = __builtin_fmaf(b4, in[e][5], a4 * g2);
      float rs = RAW_RSQ ? __builtin_amdgcn_rsqf(nv + eps) : rsqrtf(nv + eps);
      rs = r + e * w.rows + w.sub < r1 ? rs : 0.f;
      add_squares(acc, g, g2, p, {nm1, nm2, nm3}, nv, rs, {rr[e][0] * rc[0], rr[e][1] * rc[1], rr[e][2] * rc[2]});
      if (WRITE) {
        const unsigned off = w.off + 4u * (unsigned)(e * w.rows * n);
        store_one(T.st + ro, off, bytes, nm1);
        store_one(T.st + pN + ro, off, bytes, nm2);
        store_one(T.st + 2 * pN + ro, off, bytes, nm3);
        store_one(T.st + 3 * pN + ro, off, bytes, nv);
      }
    }
  }
}

// WRITE = false: the accumulators are only read (their new values are formed for the statistics and dropped); the apply
// pass of the same step forms them again and writes them (the two default apply kernels can; a read-only stream
// sustains a higher share of the HBM rate than a read-write one, and 16 of this pass's 40 bytes per element move there).
// Registers: where nothing is fused in, 64 are asked for (eight wavefronts a SIMD), with the stores 72. With 65 the reading form
// no longer fits beside the apply kernel of another tensor group (ViT-B/16 shapes 1510 -> 1567 us a step, 355 M elements 5939 -> 6278).
template <bool RAW_RSQ, bool WRITE, bool FUSE>
__global__ void __launch_bounds__(kBlock, FUSE ? 1 : WRITE ? 7 : 8) k_accum_stats(const TensorDev* __restrict__ tensors,
                                                        const TileDev* __restrict__ tiles, float* __restrict__ ws,
                                                        StepArgs A, int n_tiles, MixArgs M, int keep, bool keep_line, int keep_off,
                                                        bool backwards, const RcItemDev* __restrict__ rcitems, int n_rcitems,
                                                        bool rc_first) {
  __shared__ __align__(16) float red[kNStat][kRedStride];
  __shared__ std::conditional_t<FUSE, ShortLds, int> sh;
  FuseLds* L = nullptr;
  int idx = (int)blockIdx.x;
  if constexpr (FUSE) {
    const int n_mix = (int)gridDim.x - n_tiles - n_rcitems;
    if (idx < n_mix) {   // the extra workgroups of a VeLO step: mean of the LSTM outputs, gate bias
      mix_bias_block(M, idx, sh.mix.hbar, sh.mix.red);
      return;
    }
    idx -= n_mix;
    const int rc = rc_first ? idx : idx - n_tiles;
    if (rc >= 0 && rc < n_rcitems) {
      const RcItemDev it = rcitems[rc];
      short_rc_block(tensors[it.tensor], it, ws, A, sh.rc);
      return;
    }
    if (rc_first) idx -= n_rcitems;
    L = &sh.means;
  }
  if (backwards) idx = n_tiles - 1 - idx;
  const TileDev tile = tiles[idx];
  const TensorDev& T = tensors[tile.tensor];
  float acc[kNStat];
#pragma unroll
  for (int q = 0; q < kNStat; ++q) acc[q] = 0.f;
  if (T.n <= kNarrowCols) accum_narrow<RAW_RSQ, WRITE, FUSE>(T, tile, ws, A, acc, L);
  // (written so that it costs no register: one more and the pass no longer fits beside the apply kernel)
  else if (T.vec == 2 ? idx < keep : (T.vec == 0 || (FUSE && keep_line)) && idx < keep_off) accum_tile<RAW_RSQ, WRITE, FUSE, false>(T, tile, ws, A, acc, L);
  else accum_tile<RAW_RSQ, WRITE, FUSE, true>(T, tile, ws, A, acc, L);
  const int lt = tile.ti * T.nct + tile.tj;
  block_sum<kNStat>(acc, red, ws + T.oStatPart + (size_t)lt * kStatStride);
}

void launch_accum_stats(const Launch& L, const StepArgs& A, const WeightsDev& W, bool write_state, float* hbar_part, float* b_eff,
                        hipStream_t s) {
  if (L.n_tiles == 0) return;
  const bool raw = A.eps_acc >= 1e-30f;
  MixArgs M{};
  if (L.short_list) M = make_mix(L, A, W, hbar_part, b_eff);   // on other lists launch_rc_update has formed the cross-tensor term
  const int n_rc = L.short_list ? L.n_rcitems : 0, extra = n_rc + mix_bias_blocks(M);
  const bool rc_first = L.n_tiles > 4 * L.resident_wgs;   // eight workgroups a CU
#define LOPT_LAUNCH_ACC(R, Wr, F) \
  hipLaunchKernelGGL((k_accum_stats<R, Wr, F>), dim3(L.n_tiles + extra), dim3(kBlock), 0, s, L.tensors, L.tiles, L.ws, A, L.n_tiles, M, \
                     L.keep, L.keep_line, L.keep_off, L.backwards, L.rcitems, n_rc, rc_first)
#define LOPT_LAUNCH_ACC2(R, Wr) do { if (L.short_list) LOPT_LAUNCH_ACC(R, Wr, true); else LOPT_LAUNCH_ACC(R, Wr, false); } while (0)
  if (raw && write_state) LOPT_LAUNCH_ACC2(true, true);
  else if (raw) LOPT_LAUNCH_ACC2(true, false);
  else if (write_state) LOPT_LAUNCH_ACC2(false, true);
  else LOPT_LAUNCH_ACC2(false, false);
#undef LOPT_LAUNCH_ACC2
#undef LOPT_LAUNCH_ACC
}

// ----------------------------------------------------------------------------- finalize

// One workgroup per tensor: s_f and the per-feature scale factors (finalize_scales), then the prepared first layer or the LSTM's
// input. (Lists whose apply launch forms the scales itself do without: Plan::fold_finalize.)
__global__ void __launch_bounds__(32 * kFinSegs) k_finalize(const TensorDev* __restrict__ tensors, float* __restrict__ ws,
                                                     StepArgs A, WeightsDev W, float* __restrict__ lstm_u, int tensor0,
                                                     int* __restrict__ apply_counter, StepFeats F) {
  __shared__ FinLds L;
  const int ti = tensor0 + (int)blockIdx.x;
  const TensorDev& T = tensors[ti];
  if (blockIdx.x == 0 && threadIdx.x == 0) *apply_counter = 0;   // the apply pass of this sub-list starts at its first tile
  finalize_scales(T, ws, A, L, true);
  if (A.kind == LOPT_SMALL_FC) {
    // first layer with the normalization folded in, hidden width padded with zeros to HP;
    // the un-normalized time features only shift the bias.
    const int H = A.H, HP = A.HP;
    float* prep = ws + T.oPrep;
    for (int i = threadIdx.x; i < LOPT_N_ELEM_FEATS * HP; i += (int)blockDim.x) {
      const int f = i / HP, u = i - f * HP;
      prep[i] = u < H ? W.mlp[f * H + u] * L.scale[f] : 0.f;
    }
    for (int u = threadIdx.x; u < HP; u += (int)blockDim.x) {
      float b = 0.f;
      if (u < H) {
        b = W.mlp[LOPT_D_SMALL_FC * H + u];
        for (int i = 0; i < LOPT_N_TIME; ++i) b += F.time[i] * W.mlp[(LOPT_N_ELEM_FEATS + i) * H + u];
      }
      prep[LOPT_N_ELEM_FEATS * HP + u] = b;
    }
  } else {
    // LSTM input: 0.05*ln(s_f + 1e-30), time features, one-hot of min(ndim, 4), loss features
    float* u = lstm_u + (size_t)ti * kLstmInPad;
    const int t = threadIdx.x;
    if (t < LOPT_D_VELO) u[t] = 0.05f * logf(L.stats[t] + 1e-30f);
    else if (t < LOPT_D_VELO + LOPT_N_TIME) u[t] = F.time[t - LOPT_D_VELO];
    else if (t < LOPT_D_VELO + LOPT_N_TIME + 5) {
      const int nd = T.ndim < 4u ? (int)T.ndim : 4;
      u[t] = (t - (LOPT_D_VELO + LOPT_N_TIME)) == nd ? 1.f : 0.f;
    } else if (t < LOPT_VELO_LSTM_IN) u[t] = F.loss[t - (LOPT_D_VELO + LOPT_N_TIME + 5)];
    else if (t < kLstmInPad) u[t] = 0.f;
  }
}

void launch_finalize(const Launch& L, const StepArgs& A, const WeightsDev& W, const StepFeats& F, float* lstm_u, hipStream_t s) {
  if (L.n_tensors == 0) return;
  // long lists have more workgroups than the chip holds at once: there small ones win; beside the apply pass of another
  // tensor group only small ones find room (eight groups of 388 tensors: 18 us a launch, 53 us with 1024 threads)
  const int threads = L.n_tensors <= 512 && !L.beside_apply ? 32 * kFinSegs : kBlock;
  hipLaunchKernelGGL(k_finalize, dim3(L.n_tensors), dim3(threads), 0, s, L.tensors, L.ws, A, W, lstm_u, L.tensor0,
                     L.apply_counter, F);
}

// ----------------------------------------------------------------------------- VeLO hypernetwork

// One LSTM-cell step for all tensors: Z[T, 4 H_L] = [u | h_prev] [Wx ; Wh] is a dense contraction and runs on the
// matrix cores in fp32 (v_mfma_f32_32x32x2_f32: exact fp32 products, fp32 accumulation). A workgroup owns 32 tensors x
// 8 hidden units (one 32-column MFMA tile of 4 gates x 8 units); its eight wavefronts split the 48 + H_L input slots
// and meet in LDS in a fixed order; one thread per (tensor, unit) then applies the cell equations.
// The kernel is bound by the latency of its loads (4.6 MB of weights, a few hundred KB of inputs), so every wavefront
// issues all of them before its first product: the weights are repacked at lopt_create into the order of the tiles,
// [unit block][input slot][gate, unit], where a slot is one 128-byte line, and eight consecutive slots ("octet") are one
// float4 of the lane's tensor (its k-half's four slots) and four lines of weights. Default widths: nine octets a wavefront,
// one trip. One 1000x1000 layer 15.6 -> 9.9 us, 66 tensors 24 -> 11 us, 152 tensors 26 -> 15 us, 2219 tensors 185 -> 91 us
// (from four wavefronts over 16 units and four gathered 32-byte segments a slot).
constexpr int kLstmTensors = 32;
constexpr int kLstmWaves = 8;
constexpr int kLstmOctets = 9;   // octets in flight per wavefront

// Weights in the order k_velo_lstm reads them: out[ub][k][8 gate + u] for unit 8 ub + u, zero past H_L in units and slots.
__global__ void __launch_bounds__(kBlock) k_pack_lstm(WeightsDev W, int HL, int k_pad, float* __restrict__ out) {
  const int ub = blockIdx.x, G = 4 * HL;
#pragma unroll 8
  for (int i = threadIdx.x; i < k_pad * 32; i += kBlock) {
    const int k = i >> 5, gate = (i >> 3) & 3, unit = 8 * ub + (i & 7);
    float v = 0.f;
    if (unit < HL) {
      const size_t col = (size_t)gate * HL + unit;
      if (k < kLstmInPad) v = W.Wx[(size_t)k * G + col];
      else if (k - kLstmInPad < HL) v = W.Wh[(size_t)(k - kLstmInPad) * G + col];
    }
    out[((size_t)ub * k_pad + k) * 32 + (i & 31)] = v;
  }
}

__global__ void __launch_bounds__(64 * kLstmWaves) k_velo_lstm(const TensorDev* __restrict__ tensors, StepArgs A, WeightsDev W,
                                                      const float* __restrict__ lstm_u, const float* __restrict__ b_eff,
                                                      float* __restrict__ h_new) {
  __shared__ float part[kLstmWaves][32][32];   // [wavefront][tensor][column]: 32 KB
  const int HL = A.HL, G = 4 * HL;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int khalf = lane >> 5, l32 = lane & 31;
  const int t0 = blockIdx.x * kLstmTensors, u0 = blockIdx.y * 8;
  const int n_oct = lstm_k_pad(HL) / 8;
  // A side: the tensor of this lane (clamped: rows past the list compute on the last tensor and are dropped)
  const int tA = min(t0 + l32, A.n_tensors - 1);
  const TensorDev& T = tensors[tA];
  const float* __restrict__ hsrc = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn;
  const float* __restrict__ usrc = lstm_u + (size_t)tA * kLstmInPad;
  // B side: this lane's column of the packed weights, its k-half's four slots of an octet
  const float* __restrict__ wcol = W.lstm + ((size_t)blockIdx.y * (8 * n_oct) + 4 * khalf) * 32 + l32;
  // bias, cross-tensor term and cell state of this thread's (tensor, unit), ahead of the products
  const int tt = threadIdx.x >> 3, unit = u0 + (threadIdx.x & 7);
  const bool cell_ok = tt < kLstmTensors && t0 + tt < A.n_tensors && unit < HL;
  float be[4] = {0.f, 0.f, 0.f, 0.f}, c_old = 0.f;
  float* cl = nullptr;
  if (cell_ok) {
    const TensorDev& Tt = tensors[t0 + tt];
    cl = Tt.st + 4 * (size_t)Tt.padN + 3 * (size_t)Tt.padm + 3 * (size_t)Tt.padn + Tt.padH;
    c_old = cl[unit];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int gc = g * HL + unit;   // bias + cross-tensor term (its four partial sums, in order)
      be[g] = W.b[gc] + ((b_eff[gc] + b_eff[G + gc]) + (b_eff[2 * G + gc] + b_eff[3 * G + gc]));
    }
  }
  f32x16_l acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int per_wave = (n_oct + kLstmWaves - 1) / kLstmWaves;
  const int o_begin = wave * per_wave, o_end = min(o_begin + per_wave, n_oct);
  for (int ob = o_begin; ob < o_end; ob += kLstmOctets) {
    float4 a[kLstmOctets];
    float b[kLstmOctets][4];
#pragma unroll
    for (int j = 0; j < kLstmOctets; ++j) {
      const int o = min(ob + j, o_end - 1);   // octets past the wavefront's share repeat its last one (dropped below)
      const float4* src = 8 * o < kLstmInPad ? reinterpret_cast<const float4*>(usrc + 8 * o)
                                             : reinterpret_cast<const float4*>(hsrc + (8 * o - kLstmInPad));
      // the last octet's upper quad may start at or past H_L: the lower quad is read instead (its weights are zero)
      const int up = 8 * o - kLstmInPad + 4 < HL ? khalf : 0;
      a[j] = src[up];
#pragma unroll
      for (int i = 0; i < 4; ++i) b[j][i] = wcol[((size_t)o * 8 + i) * 32];
    }
#pragma unroll
    for (int j = 0; j < kLstmOctets; ++j) {
      if (ob + j >= o_end) break;   // wavefront-uniform
      float x[4] = {a[j].x, a[j].y, a[j].z, a[j].w};
      const int kh = 8 * (ob + j) + 4 * khalf - kLstmInPad;   // slots of h past H_L (the section's padding to four) count as 0
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = kh + i < HL ? x[i] : 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], b[j][i], acc, 0, 0, 0);
      }
    }
  }
  // accumulator register v of lane (k-half, c) is row 8 (v / 4) + 4 k-half + v % 4, column c
#pragma unroll
  for (int v = 0; v < 16; ++v) part[wave][8 * (v >> 2) + 4 * khalf + (v & 3)][l32] = acc[v];
  __syncthreads();
  if (cell_ok) {
    float zz[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float s[kLstmWaves];
#pragma unroll
      for (int w = 0; w < kLstmWaves; ++w) s[w] = part[w][tt][8 * g + (threadIdx.x & 7)];
      zz[g] = be[g] + (((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])));
    }
    const float ig = 1.f / (1.f + expf(-zz[0]));
    const float fg = 1.f / (1.f + expf(-zz[1]));
    const float gg = tanhf(zz[2]);
    const float og = 1.f / (1.f + expf(-zz[3]));
    const float c = fg * c_old + ig * gg;
    cl[unit] = c;
    h_new[(size_t)(t0 + tt) * HL + unit] = og * tanhf(c);
  }
}

// What is left of the step where the recurrent product was formed ahead (lstm_recur_block): the 48 inputs' product, two
// octets each by three wavefronts, and the cell equations, one thread per (tensor, unit).
// FIN: k_finalize has not run; every workgroup forms the inputs of the list's tensors (at most eight) from the partials first. Its
// eight half wavefronts share the tensors, one, two, four or eight to a tensor; lane = sum. The segments and their order are
// those of finalize_scales, whatever the number of tensors in the launch.
constexpr int kTailWaves = 3;
static_assert(kLstmInPad == 16 * kTailWaves, "two octets a wavefront");
struct TailFin {
  double part[4][kFinSegs][32], tot[kFinTensorsMax][32];
  alignas(16) float u[kFinTensorsMax][kLstmInPad];   // read as float4
};
static_assert(alignof(TailFin) == 16 && offsetof(TailFin, u) % 16 == 0 && kLstmInPad % 4 == 0, "rows of u on the 16-byte grid");

template <int NS>
__device__ __forceinline__ void tail_sums(const FinTerms& t, int tn, int slot, TailFin& L) {
  constexpr int HW = kFinSegs / NS;   // half wavefronts of this tensor: this one has segments slot, slot + HW, ...
  const int q = threadIdx.x & 31;
  double a[NS];
  strided_sums(t.base + (size_t)slot * t.stride, slot < t.count ? (t.count - slot + HW - 1) / HW : 0, (size_t)HW * t.stride, a);
  if (NS == kFinSegs) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};   // as segment_sum
#pragma unroll
    for (int k = 0; k < NS; ++k) s[k % 4] += a[k];
    L.tot[tn][q] = (s[0] + s[1]) + (s[2] + s[3]);
  } else {
#pragma unroll
    for (int k = 0; k < NS; ++k) L.part[tn][slot + HW * k][q] = a[k];
  }
}

__device__ __forceinline__ void tail_inputs(const TensorDev* __restrict__ tensors, float* __restrict__ ws, const StepArgs& A,
                                            const StepFeats& F, TailFin& L, bool store) {
  const int nT = A.n_tensors, w = threadIdx.x >> 5, q = threadIdx.x & 31;
  const int hw = nT <= 1 ? 8 : nT <= 2 ? 4 : nT <= 4 ? 2 : 1;
  const int tn = w / hw, slot = w % hw;
  if (tn < nT) {
    const FinTerms t = fin_terms(tensors[tn], ws, q);
    if (hw == 8) tail_sums<4>(t, tn, slot, L);
    else if (hw == 4) tail_sums<8>(t, tn, slot, L);
    else if (hw == 2) tail_sums<16>(t, tn, slot, L);
    else tail_sums<32>(t, tn, slot, L);
  }
  __syncthreads();
  if (w < nT) {
    const TensorDev& T = tensors[w];
    if (hw > 1) L.tot[w][q] = segment_sum(&L.part[w][0][q]);
    __builtin_amdgcn_wave_barrier();   // the tensor's 32 sums are this half wavefront's own
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float sf, scale;
    feature_scale(T, A, L.tot[w], q, sf, scale);
    if (store) {
      ws[T.oStats + q] = q < A.F ? sf : 0.f;
      ws[T.oScale + q] = q < A.F ? scale : 0.f;
    }
    if (q < LOPT_D_VELO) L.u[w][q] = 0.05f * logf(sf + 1e-30f);
    const int nd = T.ndim < 4u ? (int)T.ndim : 4;
    if (q < LOPT_N_TIME) L.u[w][LOPT_D_VELO + q] = F.time[q];
    if (q < 5) L.u[w][LOPT_D_VELO + LOPT_N_TIME + q] = q == nd ? 1.f : 0.f;
    if (q < kLstmInPad - (LOPT_D_VELO + LOPT_N_TIME + 5)) L.u[w][LOPT_D_VELO + LOPT_N_TIME + 5 + q] = q < LOPT_N_LOSS ? F.loss[q] : 0.f;
  }
  __syncthreads();
}

template <bool FIN>
__global__ void __launch_bounds__(kBlock) k_velo_lstm_tail(const TensorDev* __restrict__ tensors, StepArgs A, WeightsDev W,
                                                           const float* __restrict__ lstm_u, const float* __restrict__ b_eff,
                                                           const float* __restrict__ z, float* __restrict__ h_new,
                                                           float* __restrict__ ws, StepFeats F) {
  __shared__ float part[kTailWaves][32][32];   // [wavefront][tensor][column]
  __shared__ std::conditional_t<FIN, TailFin, int> fin;
  const int HL = A.HL, G = 4 * HL;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int khalf = lane >> 5, l32 = lane & 31;
  const int t0 = blockIdx.x * kLstmTensors, u0 = blockIdx.y * 8;
  const int tt = threadIdx.x >> 3, j = threadIdx.x & 7, unit = u0 + j;
  const bool cell_ok = t0 + tt < A.n_tensors && unit < HL;
  float be[4] = {0.f, 0.f, 0.f, 0.f}, zr[4] = {0.f, 0.f, 0.f, 0.f}, c_old = 0.f;
  float* cl = nullptr;
  if (cell_ok) {
    const TensorDev& Tt = tensors[t0 + tt];
    cl = Tt.st + 4 * (size_t)Tt.padN + 3 * (size_t)Tt.padm + 3 * (size_t)Tt.padn + Tt.padH;
    c_old = cl[unit];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int gc = g * HL + unit;   // bias + cross-tensor term (its four partial sums, in order)
      be[g] = W.b[gc] + ((b_eff[gc] + b_eff[G + gc]) + (b_eff[2 * G + gc] + b_eff[3 * G + gc]));
      zr[g] = z[((size_t)(t0 + tt) * gridDim.y + blockIdx.y) * 32 + 8 * g + j];
    }
  }
  if constexpr (FIN) tail_inputs(tensors, ws, A, F, fin, blockIdx.y == 0);
  if (wave < kTailWaves) {
    const float* usrc = lstm_u;
    if constexpr (FIN) usrc = fin.u[min(l32, A.n_tensors - 1)];
    else usrc += (size_t)min(t0 + l32, A.n_tensors - 1) * kLstmInPad;
    const float* __restrict__ wcol = W.lstm + ((size_t)blockIdx.y * lstm_k_pad(HL) + 4 * khalf) * 32 + l32;
    f32x16_l acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    float4 a[2];
    float b[2][4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int o = 2 * wave + q;
      a[q] = *reinterpret_cast<const float4*>(usrc + 8 * o + 4 * khalf);
#pragma unroll
      for (int i = 0; i < 4; ++i) b[q][i] = wcol[(size_t)(8 * o + i) * 32];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float x[4] = {a[q].x, a[q].y, a[q].z, a[q].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], b[q][i], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) part[wave][8 * (v >> 2) + 4 * khalf + (v & 3)][l32] = acc[v];
  }
  __syncthreads();
  if (cell_ok) {
    float zz[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) zz[g] = be[g] + ((zr[g] + part[0][tt][8 * g + j]) + (part[1][tt][8 * g + j] + part[2][tt][8 * g + j]));
    const float ig = 1.f / (1.f + expf(-zz[0]));
    const float fg = 1.f / (1.f + expf(-zz[1]));
    const float gg = tanhf(zz[2]);
    const float og = 1.f / (1.f + expf(-zz[3]));
    const float c = fg * c_old + ig * gg;
    cl[unit] = c;
    h_new[(size_t)(t0 + tt) * HL + unit] = og * tanhf(c);
  }
}

void launch_velo_lstm(const Launch& L, const StepArgs& A, const WeightsDev& W, const float* lstm_u, const float* b_eff,
                      const float* lstm_z, const StepFeats* feats, float* h_new, hipStream_t s) {
  if (L.n_tensors == 0) return;
  dim3 grid((L.n_tensors + kLstmTensors - 1) / kLstmTensors, (A.HL + 7) / 8);
  // a sub-list starts at tensor L.tensor0: the kernel indexes tensors, inputs and outputs from there
  StepArgs As = A;
  As.n_tensors = L.n_tensors;
  const TensorDev* T0 = L.tensors + L.tensor0;
  const float* u0 = lstm_u + (size_t)L.tensor0 * kLstmInPad;
  float* h0 = h_new + (size_t)L.tensor0 * A.HL;
  const float* z0 = lstm_z ? lstm_z + (size_t)L.tensor0 * grid.y * 32 : nullptr;
  if (lstm_z && feats)
    hipLaunchKernelGGL((k_velo_lstm_tail<true>), grid, dim3(kBlock), 0, s, T0, As, W, u0, b_eff, z0, h0, L.ws, *feats);
  else if (lstm_z)
    hipLaunchKernelGGL((k_velo_lstm_tail<false>), grid, dim3(kBlock), 0, s, T0, As, W, u0, b_eff, z0, h0, L.ws, StepFeats{});
  else
    hipLaunchKernelGGL(k_velo_lstm, grid, dim3(64 * kLstmWaves), 0, s, T0, As, W, u0, b_eff, h0);
}

// ---- the head with its two products folded into one at lopt_create (WeightsDev::head): theta = h (W_a B) + b_a B, with the
// step-size row (ws, bs) as one more column, [H_L + 1][head_ld(P)], row H_L the constant. Formed in double, stored in fp32.
__global__ void __launch_bounds__(kBlock) k_pack_head(WeightsDev W, int HL, int K, int P, int ld, float* __restrict__ out) {
  __shared__ float row[1024];   // this unit's coefficients of the bank's K <= 1024 rows
  const int u = blockIdx.x;     // 0 .. H_L
  for (int q = threadIdx.x; q < K; q += kBlock) row[q] = u < HL ? W.Wa[(size_t)u * K + q] : W.ba[q];
  __syncthreads();
  for (int p = threadIdx.x; p < ld; p += kBlock) {
    double a = 0.0;
    if (p < P) {
      for (int q0 = 0; q0 < K; q0 += 32) {   // 32 loads in flight
        float t[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) t[k] = W.B[(size_t)min(q0 + k, K - 1) * P + p];
#pragma unroll
        for (int k = 0; k < 32; ++k) a += q0 + k < K ? (double)row[q0 + k] * (double)t[k] : 0.0;
      }
    } else if (p == P) a = u < HL ? W.ws[u] : W.bs[0];
    out[(size_t)u * ld + p] = (float)a;
  }
}

void launch_velo_pack(const WeightsDev& W, int HL, int K, int P, float* lstm, float* head, hipStream_t s) {
  hipLaunchKernelGGL(k_pack_lstm, dim3((HL + 7) / 8), dim3(kBlock), 0, s, W, HL, lstm_k_pad(HL), lstm);
  if (head) hipLaunchKernelGGL(k_pack_head, dim3(HL + 1), dim3(kBlock), 0, s, W, HL, K, P, head_ld(P), head);
}

// theta[i] of the compact per-tensor MLP (W1[F,H] b1[H] W2[H,H] b2[H] W3[H,2] b3[2]) goes to prep[head_slot(i, ...)], the layout
// padded to HP; the first layer takes the tensor's feature scales and the direction column of the last layer the step size.
__device__ __forceinline__ int head_slot(int i, int H, int HP, const float* __restrict__ scale, float lam, float& th) {
  constexpr int F = LOPT_D_VELO;
  int o = i;
  if (o < F * H) { const int f = o / H, u = o - f * H; th *= scale[f]; return f * HP + u; }
  if ((o -= F * H) < H) return F * HP + o;
  if ((o -= H) < H * H) { const int a = o / H, u = o - a * H; return (F + 1) * HP + a * HP + u; }
  if ((o -= H * H) < H) return (F + 1) * HP + HP * HP + o;
  if ((o -= H) < 2 * H) { if (!(o & 1)) th *= lam; return (F + 1) * HP + HP * HP + HP + o; }   // W3[a][0]: direction
  o -= 2 * H;
  if (o == 0) th *= lam;                                                                         // b3[0]
  return (F + 1) * HP + HP * HP + HP + 2 * HP + o;
}

// One workgroup per tensor, 16 wavefronts. Wavefront w reduces rows w, w + 16, ... of the folded matrix, a lane four columns
// as one float4, sixteen rows in flight (bound by their latency: 309 KB at the default widths); partials meet in LDS in a
// fixed order. Replaces two dependent products (660 KB): 10.3 -> 6.5 us; 152 tensors 14.7 -> 8.4 us. Eight sums per lane
// and column and a tree behind them, not one chain: the step size's logarithm is a column too, and its absolute error is the
// relative error of the whole update (rms error of 512 random terms: 8.9e-8 in chains of 32 and 16, 5.9e-8 as 64 chains of
// eight and a tree, 5.7e-8 this way).
constexpr int kHeadWaves = 16;
__global__ void __launch_bounds__(64 * kHeadWaves) k_velo_head_folded(const TensorDev* __restrict__ tensors,
                                                                      float* __restrict__ ws, StepArgs A, WeightsDev W,
                                                                      const float* __restrict__ h_new) {
  extern __shared__ float4 sh4[];   // part[16][256] | h[HL]
  const TensorDev& T = tensors[blockIdx.x];
  const int HL = A.HL, H = A.H, HP = A.HP, P = A.P, ld = head_ld(P);
  float* part = reinterpret_cast<float*>(sh4);
  float* sh_h = part + kHeadWaves * 256;
  __shared__ float s_lam;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* hstate = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn;
  for (int i = threadIdx.x; i < HL; i += 64 * kHeadWaves) {
    const float v = h_new[(size_t)blockIdx.x * HL + i];
    sh_h[i] = v;
    hstate[i] = v;
  }
  float* prep = ws + T.oPrep;
  const float* scale = ws + T.oScale;
  if (H != HP) {   // the padding must be zero; written before the values by the barriers below
    const int prep_n = (LOPT_D_VELO + 1) * HP + HP * HP + HP + 2 * HP + 2;
    for (int i = threadIdx.x; i < prep_n; i += 64 * kHeadWaves) prep[i] = 0.f;
  }
  __syncthreads();
  // the block with the step-size column comes first: every other block needs its value
  const int last = P / 256 * 256;
  for (int blk = 0; blk <= last / 256; ++blk) {
    const int c0 = blk == 0 ? last : (blk - 1) * 256;
    const int col = c0 + 4 * lane;
    const float4* __restrict__ m = reinterpret_cast<const float4*>(W.head + min(col, ld - 4));
    float4 acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = wave; k0 < HL; k0 += 16 * kHeadWaves) {
      float4 w[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = m[(size_t)min(k0 + j * kHeadWaves, HL) * (ld / 4)];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int k = k0 + j * kHeadWaves;
        const float x = k < HL ? sh_h[min(k, HL - 1)] : 0.f;
        float4& a = acc[j & 7];
        a.x += x * w[j].x; a.y += x * w[j].y; a.z += x * w[j].z; a.w += x * w[j].w;
      }
    }
#pragma unroll
    for (int step = 1; step < 8; step *= 2)
#pragma unroll
      for (int q = 0; q < 8; q += 2 * step) {
        acc[q].x += acc[q + step].x; acc[q].y += acc[q + step].y; acc[q].z += acc[q + step].z; acc[q].w += acc[q + step].w;
      }
    *reinterpret_cast<float4*>(part + wave * 256 + 4 * lane) = acc[0];
    __syncthreads();
    const int i = c0 + (int)threadIdx.x;
    float th = 0.f;
    if (threadIdx.x < 256 && i <= P) {
      float s[kHeadWaves];
#pragma unroll
      for (int w = 0; w < kHeadWaves; ++w) s[w] = part[w * 256 + threadIdx.x];
#pragma unroll
      for (int step = 1; step < kHeadWaves; step *= 2)
#pragma unroll
        for (int w = 0; w < kHeadWaves; w += 2 * step) s[w] += s[w + step];
      th = W.head[(size_t)HL * ld + i] + s[0];
      if (i == P) s_lam = expf(th);
    }
    __syncthreads();   // s_lam; the partials may be overwritten
    if (threadIdx.x < 256 && i < P) {
      const int dst = head_slot(i, H, HP, scale, s_lam, th);
      prep[dst] = th;
    }
  }
}

// Slot i of the prepared layout is one of the zeros that pad the width H to HP.
__device__ __forceinline__ bool head_pad(int i, int H, int HP) {
  constexpr int F = LOPT_D_VELO;
  int o = i;
  if (o < (F + 1) * HP) return o % HP >= H;
  if ((o -= (F + 1) * HP) < HP * HP) return o / HP >= H || o % HP >= H;
  if ((o -= HP * HP) < HP) return o >= H;
  return (o -= HP) < 2 * HP && o / 2 >= H;
}

// The same product cut into workgroups of 32 columns, so that a tensor's 309 KB of weights come in over several compute units. A
// lane holds four columns of every 128th row, all its loads (weights and h, nothing depends on anything) leave at once; four
// terms a lane, eight lanes by shuffles, sixteen wavefronts by a tree in LDS. ln lambda is formed by every workgroup, one term
// a thread, in double: its absolute error is the relative error of the whole update (rms error of 512 random terms 2.5e-8; 8.3e-8 as
// fp32 products and trees, 7.9e-8 in k_velo_head_folded). One tensor 6.9 -> 4.6 us, 66 tensors 7.1 -> 5.9, 152 tensors 7.6 -> 8.2 (five workgroups of 1024 threads each
// are then more than the chip holds at once): kHeadSplitMax.
constexpr int kSplitCols = 32, kSplitRows = 128, kSplitTrips = 1024 / kSplitRows;   // H_L <= 1024
template <int TRIPS>
__global__ void __launch_bounds__(64 * kHeadWaves) k_velo_head_split(const TensorDev* __restrict__ tensors,
                                                                     float* __restrict__ ws, StepArgs A, WeightsDev W,
                                                                     const float* __restrict__ h_new) {
  __shared__ __align__(16) float part[kHeadWaves][kSplitCols];   // written as float4
  __shared__ double lam_part[kHeadWaves];
  const int HL = A.HL, H = A.H, HP = A.HP, P = A.P, ld = head_ld(P);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int c0 = blockIdx.x * kSplitCols, row0 = 8 * wave + (lane >> 3);
  const float* __restrict__ h = h_new + (size_t)blockIdx.y * HL;
  const float4* __restrict__ m = reinterpret_cast<const float4*>(W.head + min(c0 + 4 * (lane & 7), ld - 4));
  float4 w[TRIPS];
  float x[TRIPS];
#pragma unroll
  for (int j = 0; j < TRIPS; ++j) {
    const int k = row0 + kSplitRows * j, kc = min(k, HL - 1);
    w[j] = m[(size_t)kc * (ld / 4)];
    x[j] = h[kc];
  }
  const int kl = min(t, HL - 1);
  const float hl = h[kl], wl = W.head[(size_t)kl * ld + P], b_lam = W.head[(size_t)HL * ld + P];
  const int i = c0 + t;   // threads 0..31: column
  const float bias = t < kSplitCols && i < P ? W.head[(size_t)HL * ld + i] : 0.f;
  const TensorDev& T = tensors[blockIdx.y];
  float* prep = ws + T.oPrep;
  if (blockIdx.x == 0) {
    float* hstate = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn;
    if (t < HL) hstate[t] = hl;
    if (H != HP) {   // the padding must be zero; no workgroup writes values there
      const int prep_n = (LOPT_D_VELO + 1) * HP + HP * HP + HP + 2 * HP + 2;
      for (int s = t; s < prep_n; s += 64 * kHeadWaves)
        if (head_pad(s, H, HP)) prep[s] = 0.f;
    }
  }
  float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < TRIPS; ++j) {
    const float xv = row0 + kSplitRows * j < HL ? x[j] : 0.f;
    a[0] += xv * w[j].x; a[1] += xv * w[j].y; a[2] += xv * w[j].z; a[3] += xv * w[j].w;
  }
#pragma unroll
  for (int d = 8; d < 64; d *= 2)
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] += __shfl_xor(a[e], d);
  const double lsum = wave_sum(t < HL ? (double)hl * (double)wl : 0.0);
  if (lane < 8) *reinterpret_cast<float4*>(&part[wave][4 * lane]) = make_float4(a[0], a[1], a[2], a[3]);
  if (lane == 0) lam_part[wave] = lsum;
  __syncthreads();
  if (t < kSplitCols && i < P) {
    float s[kHeadWaves];
    double l[kHeadWaves];
#pragma unroll
    for (int q = 0; q < kHeadWaves; ++q) { s[q] = part[q][t]; l[q] = lam_part[q]; }
#pragma unroll
    for (int step = 1; step < kHeadWaves; step *= 2)
#pragma unroll
      for (int q = 0; q < kHeadWaves; q += 2 * step) { s[q] += s[q + step]; l[q] += l[q + step]; }
    float th = bias + s[0];
    const int dst = head_slot(i, H, HP, ws + T.oScale, expf((float)((double)b_lam + l[0])), th);
    prep[dst] = th;
  }
}

// Partial matrix-vector product for the hypernetwork head: out[w][c0 + 64 c + lane] = sum over rows
// k = w, w+nw, ... of x[k] * M[k][col], for the four columns c = 0..3 of this lane. Columns past the
// end are clamped for the loads (their results are never read); four rows per trip keep sixteen
// independent coalesced loads in flight (the kernel is bound by their latency).
__device__ __forceinline__ void matvec4(const float* __restrict__ x, int n_in, const float* __restrict__ M, int ld,
                                        int c0, int wave, int nw, int lane, float* __restrict__ part, int W64) {
  const float* wp[4];
  float acc[4][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int col = c0 + 64 * c + lane;
    wp[c] = M + (col < ld ? col : ld - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r][c] = 0.f;
  }
  int k = wave;
  for (; k + 3 * nw < n_in; k += 4 * nw) {
    float xv[4], w[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      xv[r] = x[k + r * nw];
#pragma unroll
      for (int c = 0; c < 4; ++c) w[r][c] = wp[c][(size_t)(k + r * nw) * ld];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[r][c] += xv[r] * w[r][c];
  }
  for (int r = 0; k < n_in; k += nw, ++r) {   // at most three rows left
    const float x0 = x[k];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float wv = wp[c][(size_t)k * ld];
      if (r == 0) acc[0][c] += x0 * wv; else if (r == 1) acc[1][c] += x0 * wv; else acc[2][c] += x0 * wv;
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (c0 + 64 * c < W64) part[wave * W64 + c0 + 64 * c + lane] = (acc[0][c] + acc[1][c]) + (acc[2][c] + acc[3][c]);
}

// Head of the hypernetwork for one tensor: alpha = h W_a + b_a, theta = alpha B, written as the
// prepared (zero-padded, first layer scaled) per-tensor MLP; the step-size multiplier lam = exp(h . ws + bs)
// is folded into the direction column of the last layer (W3[:, 0], b3[0]), so the apply pass does not see it.
// Also stores the new h into the state.
// Both products split their reduction across the workgroup's wavefronts (combined through LDS in a
// fixed order); lanes own output columns, so weight reads are coalesced.
__global__ void __launch_bounds__(1024) k_velo_head(const TensorDev* __restrict__ tensors, float* __restrict__ ws,
                                                      StepArgs A, WeightsDev W, const float* __restrict__ h_new) {
  extern __shared__ float sh[];  // h[HL] | alpha[K] | part[nw][max(K, P) rounded up to 64]
  __shared__ float s_lam;
  const TensorDev& T = tensors[blockIdx.x];
  const int HL = A.HL, K = A.K, H = A.H, HP = A.HP, F = LOPT_D_VELO, P = A.P;
  const int W64 = ((K > P ? K : P) + 63) & ~63;
  float* sh_h = sh;
  float* sh_a = sh + HL;
  float* part = sh_a + K;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  float* hstate = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn;
  for (int i = threadIdx.x; i < HL; i += blockDim.x) {
    const float v = h_new[(size_t)blockIdx.x * HL + i];
    sh_h[i] = v;
    hstate[i] = v;
  }
  // zero the padded layout (padding must be zero); disjoint from everything read below
  float* prep = ws + T.oPrep;
  const int prep_n = (F + 1) * HP + HP * HP + HP + 2 * HP + 2;
  for (int i = threadIdx.x; i < prep_n; i += blockDim.x) prep[i] = 0.f;
  __syncthreads();
  if (wave == 0) {
    float a = 0.f;
    for (int i = lane; i < HL; i += kWave) a += sh_h[i] * W.ws[i];
    a = wave_sum(a);
    if (lane == 0) s_lam = expf(a + W.bs[0]);
  }
  // alpha = h W_a: wavefront w reduces rows w, w+nw, ...; a lane owns four output columns 64 apart
  for (int q0 = 0; q0 < K; q0 += 256) matvec4(sh_h, HL, W.Wa, K, q0, wave, nw, lane, part, W64);
  __syncthreads();
  for (int q = threadIdx.x; q < K; q += blockDim.x)
  {
    float a = W.ba[q];
    for (int w = 0; w < nw; ++w) a += part[w * W64 + q];
    sh_a[q] = a;
  }
  __syncthreads();
  // theta = alpha B, same scheme
  for (int i0 = 0; i0 < P; i0 += 256) matvec4(sh_a, K, W.B, P, i0, wave, nw, lane, part, W64);
  __syncthreads();
  const float* scale = ws + T.oScale;
  for (int i = threadIdx.x; i < P; i += blockDim.x) {
    float th = 0.f;
    for (int w = 0; w < nw; ++w) th += part[w * W64 + i];
    const int dst = head_slot(i, H, HP, scale, s_lam, th);   // from the compact layout to the padded one
    prep[dst] = th;
  }
}

// ---- the head for long tensor lists as batched products on the matrix cores (fp32), then one small workgroup per tensor
// that scatters theta into the prepared layout: one product with the folded matrix, or alpha = H' W_a + b_a, theta = alpha B.

// Y[r][c] = bias[c] + sum_k X[r][k] Wm[k][c] with exact fp32 products (v_mfma_f32_32x32x2_f32), 
// a workgroup owns 32 rows x 64 columns (two 32-column tiles), its four wavefronts split the k range and
// meet in LDS in a fixed order. Lane (k-half, i) holds X[row i][2p + k-half] (A operand) and Wm[2p + k-half][column i] (B
// operand); loads are unconditional (rows, columns and k clamped, surplus k multiplied by 0).
constexpr int kMatPairsPerTrip = 16;
__global__ void __launch_bounds__(kBlock) k_rows_matmul(const float* __restrict__ X, int ldx, int n_rows, int n_in,
                                                        const float* __restrict__ Wm, int ldw, int n_cols,
                                                        const float* __restrict__ bias, float* __restrict__ Y, int ldy) {
  __shared__ float part[4][2][32][32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int khalf = lane >> 5, l32 = lane & 31;
  const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 64;
  const float* __restrict__ xrow = X + (size_t)min(r0 + l32, n_rows - 1) * ldx;
  const int ca = min(c0 + l32, n_cols - 1), cb = min(c0 + 32 + l32, n_cols - 1);
  f32x16_l acc0, acc1;
#pragma unroll
  for (int v = 0; v < 16; ++v) { acc0[v] = 0.f; acc1[v] = 0.f; }
  const int n_pairs = (n_in + 1) / 2;
  const int per_wave = (n_pairs + 3) / 4;
  const int p_begin = wave * per_wave, p_end = min(p_begin + per_wave, n_pairs);
  for (int pb = p_begin; pb < p_end; pb += kMatPairsPerTrip) {
    float a[kMatPairsPerTrip], b0[kMatPairsPerTrip], b1[kMatPairsPerTrip];
#pragma unroll
    for (int j = 0; j < kMatPairsPerTrip; ++j) {
      const int pp = pb + j < p_end ? pb + j : p_end - 1;   // a repeated pair is multiplied by 0 below
      const int k = 2 * pp + khalf;
      const int kc = k < n_in ? k : n_in - 1;
      const float keep = (pb + j < p_end && k < n_in) ? 1.f : 0.f;
      a[j] = xrow[kc] * keep;
      b0[j] = Wm[(size_t)kc * ldw + ca];
      b1[j] = Wm[(size_t)kc * ldw + cb];
    }
#pragma unroll
    for (int j = 0; j < kMatPairsPerTrip; ++j) {
      acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b0[j], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b1[j], acc1, 0, 0, 0);
    }
  }
  // accumulator register v of lane (k-half, c) is row 8 (v / 4) + 4 k-half + v % 4, column c
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = 8 * (v >> 2) + 4 * khalf + (v & 3);
    part[wave][0][row][l32] = acc0[v];
    part[wave][1][row][l32] = acc1[v];
  }
  __syncthreads();
  const int rr = threadIdx.x >> 3, cc = threadIdx.x & 7;
  if (r0 + rr < n_rows) {
#pragma unroll
    for (int tile = 0; tile < 2; ++tile)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cl = 8 * q + cc, col = c0 + 32 * tile + cl;
        if (col < n_cols)
          Y[(size_t)(r0 + rr) * ldy + col] = (bias ? bias[col] : 0.f) + ((part[0][tile][rr][cl] + part[1][tile][rr][cl]) +
                                                                          (part[2][tile][rr][cl] + part[3][tile][rr][cl]));
      }
  }
}

// One workgroup per tensor: new h into the state, step-size multiplier, theta[P] (rows of ld) scattered into the prepared layout.
// The step size's logarithm is formed here (eight terms a lane and a tree): as a column of the product it would be chains of 128.
__global__ void __launch_bounds__(kBlock) k_velo_head_scatter(const TensorDev* __restrict__ tensors, float* __restrict__ ws,
                                                              StepArgs A, WeightsDev W, const float* __restrict__ h_new,
                                                              const float* __restrict__ theta, int ld) {
  __shared__ float s_lam;
  const TensorDev& T = tensors[blockIdx.x];
  const int HL = A.HL, H = A.H, HP = A.HP, F = LOPT_D_VELO, P = A.P;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* hstate = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm + 3 * (size_t)T.padn;
  const float* __restrict__ hn = h_new + (size_t)blockIdx.x * HL;
  const float* __restrict__ th_row = theta + (size_t)blockIdx.x * ld;
  for (int i = threadIdx.x; i < HL; i += kBlock) hstate[i] = hn[i];
  float* prep = ws + T.oPrep;
  const int prep_n = (F + 1) * HP + HP * HP + HP + 2 * HP + 2;
  for (int i = threadIdx.x; i < prep_n; i += kBlock) prep[i] = 0.f;   // the padding must be zero
  if (wave == 0) {
    float a = 0.f;
    for (int i = lane; i < HL; i += kWave) a += hn[i] * W.ws[i];
    a = wave_sum(a);
    if (lane == 0) s_lam = expf(a + W.bs[0]);
  }
  __syncthreads();
  const float* scale = ws + T.oScale;
  for (int i = threadIdx.x; i < P; i += kBlock) {
    float th = th_row[i];
    const int dst = head_slot(i, H, HP, scale, s_lam, th);
    prep[dst] = th;
  }
}

// theta (and alpha, if the head is not folded): scratch of n_tensors rows for the batched form, null for lists below
// kHeadBatchMin tensors (one workgroup per tensor then does everything; cheaper in launches, dearer in weight reads). The
// form is the whole list's, also for a sub-list of it: the forms round differently.
void launch_velo_head(const Launch& L, const StepArgs& A, const WeightsDev& W, const float* h_new, float* alpha,
                      float* theta, hipStream_t s) {
  if (L.n_tensors == 0) return;
  const int T = L.n_tensors;
  const float* hn = h_new + (size_t)L.tensor0 * A.HL;
  const bool batched = theta != nullptr;
  if (W.head) {
    const int ld = head_ld(A.P);
    if (batched) {
      float* th = theta + (size_t)L.tensor0 * ld;
      hipLaunchKernelGGL(k_rows_matmul, dim3((T + 31) / 32, (A.P + 63) / 64), dim3(kBlock), 0, s, hn, A.HL, T, A.HL, W.head,
                         ld, A.P, W.head + (size_t)A.HL * ld, th, ld);
      hipLaunchKernelGGL(k_velo_head_scatter, dim3(T), dim3(kBlock), 0, s, L.tensors + L.tensor0, L.ws, A, W, hn, th, ld);
    } else if (A.n_tensors <= kHeadSplitMax) {   // of the whole list, see above
      const dim3 grid((A.P + kSplitCols - 1) / kSplitCols, T);
#define LOPT_LAUNCH_SPLIT(N) \
  hipLaunchKernelGGL((k_velo_head_split<N>), grid, dim3(64 * kHeadWaves), 0, s, L.tensors + L.tensor0, L.ws, A, W, hn)
      if (A.HL <= 4 * kSplitRows) LOPT_LAUNCH_SPLIT(4);
      else LOPT_LAUNCH_SPLIT(kSplitTrips);
#undef LOPT_LAUNCH_SPLIT
    } else {
      const size_t shmem = (size_t)(((A.HL + 3) & ~3) + kHeadWaves * 256) * sizeof(float);
      hipLaunchKernelGGL(k_velo_head_folded, dim3(T), dim3(64 * kHeadWaves), shmem, s, L.tensors + L.tensor0, L.ws, A, W, hn);
    }
    return;
  }
  if (batched) {
    float* al = alpha + (size_t)L.tensor0 * A.K;
    float* th = theta + (size_t)L.tensor0 * A.P;
    hipLaunchKernelGGL(k_rows_matmul, dim3((T + 31) / 32, (A.K + 63) / 64), dim3(kBlock), 0, s, hn, A.HL, T, A.HL, W.Wa, A.K,
                       A.K, W.ba, al, A.K);
    hipLaunchKernelGGL(k_rows_matmul, dim3((T + 31) / 32, (A.P + 63) / 64), dim3(kBlock), 0, s, al, A.K, T, A.K, W.B, A.P,
                       A.P, (const float*)nullptr, th, A.P);
    hipLaunchKernelGGL(k_velo_head_scatter, dim3(T), dim3(kBlock), 0, s, L.tensors + L.tensor0, L.ws, A, W, hn, th, A.P);
    return;
  }
  const int W64 = ((A.K > A.P ? A.K : A.P) + 63) & ~63;
  int nw = 16;  // wavefronts per workgroup = ways the reductions are split; bounded by 48 KB of partials
  while (nw > 1 && (size_t)nw * W64 * sizeof(float) > 48 * 1024) nw >>= 1;
  size_t shmem = (size_t)(A.HL + A.K + nw * W64) * sizeof(float);
  hipLaunchKernelGGL(k_velo_head, dim3(L.n_tensors), dim3(64 * nw), shmem, s, L.tensors + L.tensor0, L.ws, A, W,
                     h_new + (size_t)L.tensor0 * A.HL);
}

}  // namespace lopt
