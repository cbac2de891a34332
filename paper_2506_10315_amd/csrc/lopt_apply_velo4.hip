// Fused apply pass for VeLO with per-element MLP width 4 (paper: "Kernel 2"; per-tensor weights from
// the hypernetwork). The three tiny layers run on v_mfma_f32_4x4x1_16B_f32: the instruction performs
// 16 independent 4x4 outer-product accumulations, D_b[i][j] += A_b[i] * B_b[j], one per group of four
// lanes. With A = W[k][i] (i = lane & 3, the same in every group) and B = feature k of the lane's OWN
// element, lane l ends up with all four hidden pre-activations of its own element in the four
// accumulator registers: no cross-lane traffic at all, exact fp32, and twice the FMA rate of the
// vector ALU (which is what bounds this pass once the weights are per tensor and only 28 to 44 bytes per
// element move). The 12 row/column-constant features enter through the C operand (4 values per row
// and 4 per column), so layer 1 is 17 MFMAs per element instead of 29.
#include "lopt_internal.h"
#include "lopt_device.h"

namespace lopt {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kVF = LOPT_D_VELO;  // 29
constexpr int kVH = 4;
constexpr unsigned kNoColumn = 0xFFFFF000u;   // byte offset beyond every descriptor: reads as 0, is not written
constexpr int kVE = 17;           // features that vary per element: 0..12, 25..27, 28

__device__ __forceinline__ constexpr int velo_elem_feat(int i) { return i < 13 ? i : 12 + i; }   // 0..12, 25..28
__device__ __forceinline__ constexpr int velo_row_feat(int i) { return i < 3 ? 13 + i : 16 + i; }  // 13..15, 19..21
__device__ __forceinline__ constexpr int velo_col_feat(int i) { return i < 3 ? 16 + i : 19 + i; }  // 16..18, 22..24

__device__ __forceinline__ float relu1(float x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, i > 0 ? i : 0);
}

// UPDATE_STATE: the statistics pass left M_1..3 and V as they were; this pass forms the new values (the statistics
// pass's operations, in its order: the same bits), builds the features from them and writes them back.
// NT: nontemporal accesses, for rows on the 128-byte grid (each line is touched by one wavefront only). Rows off the grid
// share their first and last line with the neighbouring tiles, which nontemporal accesses fetch and write twice: there
// ordinary ones are faster (18 matrices of 2732 columns: 0.587 -> 0.496 ms; on the grid, ViT-B/16 shapes, they cost the
// next step's statistics pass more than this pass gains).
// MASK: lanes past the last column take no part in the accesses, instead of leaving it to the range check. Rows on the 16-byte but off the
// 128-byte grid are faster with it (two of 4096x4100 508 -> 500 us a step, twelve of 4000x132 127 -> 122), rows off the 16-byte grid without
// (16001x9001 2139 -> 2085, 54 M elements of 2731 columns 782 -> 777; 4000x191 the other way, 132 / 134), rows on the 128-byte grid are
// the same either way to 0.3 %.
// Rows off the 16-byte grid, four columns a lane against one column a lane: 54 M of 2731 columns 808 -> 777 us a step, 16001x9001 2137 ->
// 2085, 8.2 M of 2731 columns 144 -> 138, five layers of 777 61 -> 57.
template <bool NT, bool MASK, bool RAW_RSQ, bool UPDATE_STATE>
__device__ __forceinline__ void apply_velo4_tile(const TensorDev& T, const RowWalk& w, const float* __restrict__ ws,
                                                 const StepArgs& A) {
  const int lane = threadIdx.x & 63;
  const int i4 = lane & 3;
  // prepared per-tensor MLP: W1s[29][4] (normalization folded in) b1[4] W2[4][4] b2[4] W3[4][2] b3[2]
  const float* __restrict__ prep = ws + T.oPrep;
  const float* __restrict__ W2 = prep + (kVF + 1) * kVH;
  const float* __restrict__ B2 = W2 + kVH * kVH;
  const float* __restrict__ W3 = B2 + kVH;
  const float* __restrict__ B3 = W3 + 2 * kVH;
  float a1[kVE], a2[kVH], a3[kVH];
#pragma unroll
  for (int k = 0; k < kVE; ++k) a1[k] = prep[velo_elem_feat(k) * kVH + i4];
#pragma unroll
  for (int k = 0; k < kVH; ++k) {
    a2[k] = W2[k * kVH + i4];
    a3[k] = i4 < 2 ? W3[2 * k + i4] : 0.f;
  }
  const f32x4 c2 = {B2[0], B2[1], B2[2], B2[3]};
  const f32x4 c3 = {B3[0], B3[1], 0.f, 0.f};

  const int n = T.n;
  // columns past the row's end (load_quad) and rows' pad columns of r_k and c_k: computed on, never stored
  const int c0 = w.tj * kTileCols, col = c0 + 4 * lane;
  const unsigned off = 16u * lane, bytes = segment_bytes(n, c0);
  float4 rc[3];
  f32x4 colv[4];   // per column of this lane: sum over the 6 column-constant features, for the 4 hidden units
  {
    float4 cc[3];
    const float* cst = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      rc[k] = load4<true>(ws + T.oRC + (size_t)k * T.padn, col, n);
      cc[k] = load4<true>(cst + (size_t)k * T.padn, col, n);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int u = 0; u < kVH; ++u) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          a += get(cc[k], e) * prep[velo_col_feat(k) * kVH + u];
          a += get(rc[k], e) * prep[velo_col_feat(3 + k) * kVH + u];
        }
        colv[e][u] = a;
      }
    }
  }
  float* __restrict__ M1 = T.st;
  float* __restrict__ M2 = T.st + (size_t)T.padN;
  float* __restrict__ M3 = T.st + 2 * (size_t)T.padN;
  float* __restrict__ Vp = T.st + 3 * (size_t)T.padN;
  const float* rst = T.st + 4 * (size_t)T.padN;
  const float eps = A.eps_acc, lr = A.lr, wd = A.wd;
  const float bm1 = A.mom_decay[0], bm2 = A.mom_decay[1], bm3 = A.mom_decay[2], bv = A.rms_decay;
  const float am1 = 1.0f - bm1, am2 = 1.0f - bm2, am3 = 1.0f - bm3, av = 1.0f - bv;

  for (int i = 0; i < w.cnt; ++i) {
    const int r = walk_row(w, i);
    const size_t ro = (size_t)r * n + c0;
    f32x4v g4 = {0.f, 0.f, 0.f, 0.f}, p4 = g4, m1 = g4, m2 = g4, m3 = g4, v4 = g4;
    if (!MASK || col < n) {
      g4 = load_quad<NT>(T.g + ro, off, bytes);
      p4 = load_quad<NT>(T.p + ro, off, bytes);
      m1 = load_quad<NT>(M1 + ro, off, bytes);
      m2 = load_quad<NT>(M2 + ro, off, bytes);
      m3 = load_quad<NT>(M3 + ro, off, bytes);
      v4 = load_quad<NT>(Vp + ro, off, bytes);
    }
    float rr[3], rv[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      rr[k] = ws[T.oRR + (size_t)k * T.padm + r];
      rv[k] = rst[(size_t)k * T.padm + r];
    }
    // bias + row-constant features (wave-uniform)
    f32x4 rowv;
#pragma unroll
    for (int u = 0; u < kVH; ++u) {
      float a = prep[kVF * kVH + u];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        a += rv[k] * prep[velo_row_feat(k) * kVH + u];
        a += rr[k] * prep[velo_row_feat(3 + k) * kVH + u];
      }
      rowv[u] = a;
    }
    float x[4][kVE];
    f32x4 h[4];
    f32x4v n1, n2, n3, nv;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float g = g4[e];
      float q1 = m1[e], q2 = m2[e], q3 = m3[e], v = v4[e];
      if (UPDATE_STATE) {
        q1 = __builtin_fmaf(bm1, q1, am1 * g);
        q2 = __builtin_fmaf(bm2, q2, am2 * g);
        q3 = __builtin_fmaf(bm3, q3, am3 * g);
        v = __builtin_fmaf(bv, v, av * (g * g));
        n1[e] = q1; n2[e] = q2; n3[e] = q3; nv[e] = v;
      }
      const float rs = RAW_RSQ ? __builtin_amdgcn_rsqf(v + eps) : rsqrtf(v + eps);
      const float f0 = rr[0] * get(rc[0], e), f1 = rr[1] * get(rc[1], e), f2 = rr[2] * get(rc[2], e);
      x[e][0] = g; x[e][1] = p4[e]; x[e][2] = q1; x[e][3] = q2; x[e][4] = q3; x[e][5] = v;
      x[e][6] = q1 * rs; x[e][7] = q2 * rs; x[e][8] = q3 * rs; x[e][9] = rs;
      x[e][10] = g * f0; x[e][11] = g * f1; x[e][12] = g * f2;
      x[e][13] = q1 * f0; x[e][14] = q2 * f1; x[e][15] = q3 * f2;
      x[e][16] = fminf(fmaxf(g, -0.1f), 0.1f);
      h[e] = rowv + colv[e];
    }
    if (UPDATE_STATE && (!MASK || col < n)) {   // stored while the values are live as features anyway
      store_quad<NT>(M1 + ro, off, bytes, n1);
      store_quad<NT>(M2 + ro, off, bytes, n2);
      store_quad<NT>(M3 + ro, off, bytes, n3);
      store_quad<NT>(Vp + ro, off, bytes, nv);
    }
    // layer 1: the four elements of the lane are four independent accumulation chains
#pragma unroll
    for (int k = 0; k < kVE; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(a1[k], x[e][k], h[e], 0, 0, 0);
    }
    f32x4 h2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h2[e] = c2;
#pragma unroll
    for (int k = 0; k < kVH; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) h2[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(a2[k], relu1(h[e][k]), h2[e], 0, 0, 0);
    }
    f32x4 o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = c3;
#pragma unroll
    for (int k = 0; k < kVH; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(a3[k], relu1(h2[e][k]), o[e], 0, 0, 0);
    }
    f32x4v pn;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float delta = o[e][0] * __expf(o[e][1] * A.exp_mult) * A.step_mult;
      const float p = p4[e];
      pn[e] = p - lr * (delta + wd * p);
    }
    if (!MASK || col < n) store_quad<NT>(T.p + ro, off, bytes, pn);
  }
}

// Narrow tensors: one column a lane (NarrowWalk), four accesses per trip (the four elements of the MFMA chains are rows instead of
// columns). Ordinary accesses: neighbouring wavefronts share their boundary lines.
template <bool RAW_RSQ, bool UPDATE_STATE>
__device__ __forceinline__ void apply_velo4_narrow(const TensorDev& T, const TileDev& tile, const float* __restrict__ ws,
                                                      const StepArgs& A) {
  const int i4 = threadIdx.x & 3;
  const int n = T.n;
  const NarrowWalk w(n, 4);
  const unsigned cc = (unsigned)min(w.col, n - 1);   // lanes without a column compute on the last one and store nothing
  const float* __restrict__ prep = ws + T.oPrep;
  const float* __restrict__ W2 = prep + (kVF + 1) * kVH;
  const float* __restrict__ B2 = W2 + kVH * kVH;
  const float* __restrict__ W3 = B2 + kVH;
  const float* __restrict__ B3 = W3 + 2 * kVH;
  float a1[kVE], a2[kVH], a3[kVH];
#pragma unroll
  for (int k = 0; k < kVE; ++k) a1[k] = prep[velo_elem_feat(k) * kVH + i4];
#pragma unroll
  for (int k = 0; k < kVH; ++k) {
    a2[k] = W2[k * kVH + i4];
    a3[k] = i4 < 2 ? W3[2 * k + i4] : 0.f;
  }
  const f32x4 c2 = {B2[0], B2[1], B2[2], B2[3]};
  const f32x4 c3 = {B3[0], B3[1], 0.f, 0.f};
  float rc[3];
  f32x4 colv;
  {
    float cv[3];
    const float* cst = T.st + 4 * (size_t)T.padN + 3 * (size_t)T.padm;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      rc[k] = ws[T.oRC + (size_t)k * T.padn + cc];
      cv[k] = cst[(size_t)k * T.padn + cc];
    }
#pragma unroll
    for (int u = 0; u < kVH; ++u) {
      float a = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        a += cv[k] * prep[velo_col_feat(k) * kVH + u];
        a += rc[k] * prep[velo_col_feat(3 + k) * kVH + u];
      }
      colv[u] = a;
    }
  }
  const size_t pN = T.padN;
  const float* rst = T.st + 4 * pN;
  const float eps = A.eps_acc, lr = A.lr, wd = A.wd;
  const float bm1 = A.mom_decay[0], bm2 = A.mom_decay[1], bm3 = A.mom_decay[2], bv = A.rms_decay;
  const float am1 = 1.0f - bm1, am2 = 1.0f - bm2, am3 = 1.0f - bm3, av = 1.0f - bv;
  const auto [r0, r1] = tile_rows(T, tile);
  for (unsigned r = r0 + w.first; r < r1; r += w.step) {
    const size_t ro = (size_t)r * (unsigned)n;
    const unsigned bytes = 4u * (unsigned)n * min(r1 - r, (unsigned)(4 * w.rows));   // of the rows this trip takes: others read as 0
    float e_in[4][6];
    unsigned off[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      off[e] = w.col_ok ? w.off + 4u * (unsigned)(e * w.rows * n) : kNoColumn;
      e_in[e][0] = load_one(T.g + ro, off[e], bytes);
      e_in[e][1] = load_one(T.p + ro, off[e], bytes);
#pragma unroll
      for (int k = 0; k < 4; ++k) e_in[e][2 + k] = load_one(T.st + k * pN + ro, off[e], bytes);
    }
    float x[4][kVE];
    f32x4 h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned row = min(r + e * w.rows + w.sub, r1 - 1);
      float rr[3], rv[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        rr[k] = ws[T.oRR + (size_t)k * T.padm + row];
        rv[k] = rst[(size_t)k * T.padm + row];
      }
      f32x4 rowv;   // bias + row-constant features of this lane's row
#pragma unroll
      for (int u = 0; u < kVH; ++u) {
        float a = prep[kVF * kVH + u];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          a += rv[k] * prep[velo_row_feat(k) * kVH + u];
          a += rr[k] * prep[velo_row_feat(3 + k) * kVH + u];
        }
        rowv[u] = a;
      }
      const float g = e_in[e][0];
      float q1 = e_in[e][2], q2 = e_in[e][3], q3 = e_in[e][4], v = e_in[e][5];
      if (UPDATE_STATE) {
        q1 = __builtin_fmaf(bm1, q1, am1 * g);
        q2 = __builtin_fmaf(bm2, q2, am2 * g);
        q3 = __builtin_fmaf(bm3, q3, am3 * g);
        v = __builtin_fmaf(bv, v, av * (g * g));
        store_one(T.st + ro, off[e], bytes, q1);
        store_one(T.st + pN + ro, off[e], bytes, q2);
        store_one(T.st + 2 * pN + ro, off[e], bytes, q3);
        store_one(T.st + 3 * pN + ro, off[e], bytes, v);
      }
      const float rs = RAW_RSQ ? __builtin_amdgcn_rsqf(v + eps) : rsqrtf(v + eps);
      const float f0 = rr[0] * rc[0], f1 = rr[1] * rc[1], f2 = rr[2] * rc[2];
      x[e][0] = g; x[e][1] = e_in[e][1]; x[e][2] = q1; x[e][3] = q2; x[e][4] = q3; x[e][5] = v;
      x[e][6] = q1 * rs; x[e][7] = q2 * rs; x[e][8] = q3 * rs; x[e][9] = rs;
      x[e][10] = g * f0; x[e][11] = g * f1; x[e][12] = g * f2;
      x[e][13] = q1 * f0; x[e][14] = q2 * f1; x[e][15] = q3 * f2;
      x[e][16] = fminf(fmaxf(g, -0.1f), 0.1f);
      h[e] = rowv + colv;
    }
#pragma unroll
    for (int k = 0; k < kVE; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(a1[k], x[e][k], h[e], 0, 0, 0);
    }
    f32x4 h2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h2[e] = c2;
#pragma unroll
    for (int k = 0; k < kVH; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) h2[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(a2[k], relu1(h[e][k]), h2[e], 0, 0, 0);
    }
    f32x4 o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = c3;
#pragma unroll
    for (int k = 0; k < kVH; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(a3[k], relu1(h2[e][k]), o[e], 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float delta = o[e][0] * __expf(o[e][1] * A.exp_mult) * A.step_mult;
      const float p = e_in[e][1];
      store_one(T.p + ro, off[e], bytes, p - lr * (delta + wd * p));
    }
  }
}

template <bool RAW_RSQ, bool UPDATE_STATE>
__global__ void __launch_bounds__(kBlock, 4) k_apply_velo4(const TensorDev* __restrict__ tensors,
                                                        const TileDev* __restrict__ tiles, float* __restrict__ ws,
                                                        StepArgs A, bool off_grid_nt) {
  const TileDev tile = tiles[blockIdx.x];
  const TensorDev& T = tensors[tile.tensor];
  if (T.n <= kNarrowCols) apply_velo4_narrow<RAW_RSQ, UPDATE_STATE>(T, tile, ws, A);
  else {
    const RowWalk w = row_walk(T, tile, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
    if (T.vec == 2 || (T.vec == 0 && off_grid_nt)) apply_velo4_tile<true, false, RAW_RSQ, UPDATE_STATE>(T, w, ws, A);
    else if (T.vec) apply_velo4_tile<false, true, RAW_RSQ, UPDATE_STATE>(T, w, ws, A);
    else apply_velo4_tile<false, false, RAW_RSQ, UPDATE_STATE>(T, w, ws, A);
  }
}

bool apply_velo4_available(const StepArgs& A) { return A.kind == LOPT_VELO && A.H == kVH && A.HP == kVH; }

void launch_apply_velo4(const Launch& L, const StepArgs& A, bool update_state, hipStream_t s) {
  if (L.n_tiles == 0) return;
  // v_rsq_f32 treats inputs below the smallest normal float as zero; with eps_acc that small the kernel takes the
  // library reciprocal square root (which rescales such inputs) instead of the bare instruction
  const bool raw = A.eps_acc >= 1e-30f;
#define LOPT_LAUNCH_V4(R, U) \
  hipLaunchKernelGGL((k_apply_velo4<R, U>), dim3(L.n_tiles), dim3(kBlock), 0, s, L.tensors, L.tiles, L.ws, A, L.off_grid_nt)
  if (raw && update_state) LOPT_LAUNCH_V4(true, true);
  else if (raw) LOPT_LAUNCH_V4(true, false);
  else if (update_state) LOPT_LAUNCH_V4(false, true);
  else LOPT_LAUNCH_V4(false, false);
#undef LOPT_LAUNCH_V4
}

}  // namespace lopt
