// Fused apply pass for small_fc_lopt with (padded) hidden width 4, 8 or 16 (paper: "Kernel 2: fused feature construction
// and network application"), on the fp32 matrix instructions (exact fp32 products and sums). The 12 row- or column-constant
// features enter as a vector per row (LDS, once per tile) and per column (registers), so layer 1 takes 16
// products per unit instead of 28. A lane owns one column and takes its rows one after the other, with the next
// rows' loads ahead, so that any row length and alignment is a coalesced dword access.
//
// Widths 4 and 8: v_mfma_f32_4x4x1_16B_f32, 16 independent 4x4 outer products, one per group of four lanes. With
// A = W[k][4 g + i] (i = lane & 3) and B = feature k of the lane's OWN element, lane l ends up with hidden units
// 4 g .. 4 g + 3 of its own element, with no cross-lane traffic. Both are close to the memory bound.
//
// Width 16: the 4x4x1 form sustains a third of the fp32 matrix rate there (144 instructions per 64 elements, 217 us for
// 9.5 M elements), so the products run on v_mfma_f32_16x16x4_f32, transposed, D[unit, element] = W^T X^T, as four tiles of
// 16 columns: v_permlane32_swap and v_permlane16_swap transpose each four features of the four lane quarters into the B
// operands of the four tiles; a lane then holds four units of one element of every tile, which (after the ReLU) are
// layer 2's B operands as they stand; layer 3 is 32 vector FMAs and a transposing sum over the quarters.
// Against the vector-ALU kernel these replace by default (9.5 M elements, 1024 columns): width 16 388 -> 158 us, accumulators
// written here included; rows off the 16-byte grid, where that kernel spills: 2.0 M elements, 1001 columns, width 12, whole
// step 1.27 ms -> 62 us. Widths 4 and 8, 14.7 M elements, whole step 230 -> 211 and 382 -> 225 us.
#include "lopt_apply_common.h"

namespace lopt {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int HP>
struct Fc4Lds {
  f32x4 rowv[kApplyRows][HP / 4];         // bias (time features folded in) + row-constant features, first layer
  alignas(16) float rr[kApplyRows][4];    // rsqrt(r_k + eps) of the row
};

// fmax(x, 0), a NaN giving 0 like the vector-ALU kernel's: one instruction, where fmaxf (and a median whose third operand the
// compiler knows to be infinity) takes two
__device__ __forceinline__ float relu_max(float x) {
  float inf = __builtin_inff();
  asm("" : "+s"(inf));
  return __builtin_amdgcn_fmed3f(x, 0.f, inf);
}

template <bool NT>
__device__ __forceinline__ float ld1(const float* p) { return NT ? __builtin_nontemporal_load(p) : *p; }
template <bool NT>
__device__ __forceinline__ void st1(float v, float* p) {
  if (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// The per-element MLP: weights of this lane and of its column.
template <int HP>
struct Mlp {   // widths 4 and 8
  static constexpr int G = HP / 4;
  float a1[kNE][G], a2[HP][G], a3[HP];
  f32x4 b2[G], c3, colv[G];
  __device__ __forceinline__ void load(const float* __restrict__ prep, const float* __restrict__ tail) {
    const int i4 = threadIdx.x & 3;
    const float* __restrict__ W3 = tail + HP * HP + HP;
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int k = 0; k < kNE; ++k) a1[k][g] = prep[elem_feat(k) * HP + 4 * g + i4];
#pragma unroll
      for (int k = 0; k < HP; ++k) a2[k][g] = tail[k * HP + 4 * g + i4];
#pragma unroll
      for (int j = 0; j < 4; ++j) b2[g][j] = tail[HP * HP + 4 * g + j];
    }
#pragma unroll
    for (int k = 0; k < HP; ++k) a3[k] = i4 < 2 ? W3[2 * k + i4] : 0.f;
    c3 = f32x4{W3[2 * HP], W3[2 * HP + 1], 0.f, 0.f};
  }
  // c: the column accumulators c_k [3][padn], rcp: rsqrt(c_k + eps) [3][padn]; cc: this lane's column (clamped)
  __device__ __forceinline__ void load_col(const float* __restrict__ prep, const float* __restrict__ c,
                                           const float* __restrict__ rcp, size_t padn, int /*first*/, int /*n*/, size_t cc) {
    float cv[3], rv[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) { cv[k] = c[k * padn + cc]; rv[k] = rcp[k * padn + cc]; }
#pragma unroll
    for (int u = 0; u < HP; ++u) {
      float a = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) a += cv[k] * prep[col_feat(k) * HP + u];
#pragma unroll
      for (int k = 0; k < 3; ++k) a += rv[k] * prep[col_feat(3 + k) * HP + u];
      colv[u >> 2][u & 3] = a;
    }
  }
  __device__ __forceinline__ void operator()(const float (&x)[kNE], const f32x4* rowv, float& d, float& mg) const {
    f32x4 h[G], h2[G];
#pragma unroll
    for (int u = 0; u < G; ++u) { h[u] = rowv[u] + colv[u]; h2[u] = b2[u]; }
#pragma unroll
    for (int k = 0; k < kNE; ++k)
#pragma unroll
      for (int u = 0; u < G; ++u) h[u] = __builtin_amdgcn_mfma_f32_4x4x1f32(a1[k][u], x[k], h[u], 0, 0, 0);
#pragma unroll
    for (int k = 0; k < HP; ++k) {
      const float hk = relu_max(h[k >> 2][k & 3]);
#pragma unroll
      for (int u = 0; u < G; ++u) h2[u] = __builtin_amdgcn_mfma_f32_4x4x1f32(a2[k][u], hk, h2[u], 0, 0, 0);
    }
    // two half chains: the last layer has one group of outputs and would otherwise be one serial chain
    f32x4 o = c3, o2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < HP; k += 2) {
      o = __builtin_amdgcn_mfma_f32_4x4x1f32(a3[k], relu_max(h2[k >> 2][k & 3]), o, 0, 0, 0);
      o2 = __builtin_amdgcn_mfma_f32_4x4x1f32(a3[k + 1], relu_max(h2[(k + 1) >> 2][(k + 1) & 3]), o2, 0, 0, 0);
    }
    d = o[0] + o2[0];
    mg = o[1] + o2[1];
  }
};

// Swaps in assembly (the compiler's builtin of the 32-lane one returns its first result twice, checked on ROCm 7.2), with
// the wait states around vector instructions that the compiler cannot see inside the block. v_permlane32_swap a, b exchanges
// a's upper half with b's lower half, v_permlane16_swap a's odd quarters with b's even ones.
// x[4 s + i] of lane quarter q -> x[4 s + t] = feature 4 s + q of quarter t's element, for s = 0..3.
__device__ __forceinline__ void transpose_quarters(float (&x)[kNE]) {
  asm("s_nop 1\n\t"
      "v_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3\n\t"
      "v_permlane32_swap_b32 %4, %6\n\tv_permlane32_swap_b32 %5, %7\n\t"
      "v_permlane32_swap_b32 %8, %10\n\tv_permlane32_swap_b32 %9, %11\n\t"
      "v_permlane32_swap_b32 %12, %14\n\tv_permlane32_swap_b32 %13, %15\n\t"
      "s_nop 1\n\t"
      "v_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\t"
      "v_permlane16_swap_b32 %4, %5\n\tv_permlane16_swap_b32 %6, %7\n\t"
      "v_permlane16_swap_b32 %8, %9\n\tv_permlane16_swap_b32 %10, %11\n\t"
      "v_permlane16_swap_b32 %12, %13\n\tv_permlane16_swap_b32 %14, %15\n\t"
      "s_nop 1"
      : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]),
        "+v"(x[8]), "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]), "+v"(x[15]));
}

// d[t], m[t]: partial sums of tile t in the four lane quarters -> the totals of the lane's own tile (its quarter's).
__device__ __forceinline__ void sum_quarters(float (&d)[4], float (&m)[4], float& dt, float& mt) {
  asm("s_nop 1\n\t"
      "v_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3\n\t"
      "v_permlane32_swap_b32 %4, %6\n\tv_permlane32_swap_b32 %5, %7\n\t"
      "s_nop 1"
      : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]), "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]));
  float d02 = d[0] + d[2], d13 = d[1] + d[3], m02 = m[0] + m[2], m13 = m[1] + m[3];
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\ts_nop 1"
      : "+v"(d02), "+v"(d13), "+v"(m02), "+v"(m13));
  dt = d02 + d13;
  mt = m02 + m13;
}

template <>
struct Mlp<16> {
  float a1[4], a2[4];   // A operands: [step]: W1[feature 4 s + quarter][unit], W2[unit 4 quarter + s][unit]
  f32x4 b2, colc[4];    // units 4 quarter + j: second bias; column part of the first layer of tile t's column
  float w3d[4], w3m[4], b3d, b3m;
  __device__ __forceinline__ void load(const float* __restrict__ prep, const float* __restrict__ tail) {
    const int q = (threadIdx.x & 63) >> 4, u = threadIdx.x & 15;
    const float* __restrict__ W3 = tail + 16 * 16 + 16;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int f = 4 * s + q;
      a1[s] = prep[(f < 13 ? f : 12 + f) * 16 + u];   // elem_feat(f)
      a2[s] = tail[(4 * q + s) * 16 + u];
      b2[s] = tail[16 * 16 + 4 * q + s];
      w3d[s] = W3[2 * (4 * q + s)];
      w3m[s] = W3[2 * (4 * q + s) + 1];
    }
    b3d = W3[32];
    b3m = W3[33];
  }
  // first: the wavefront's first column
  __device__ __forceinline__ void load_col(const float* __restrict__ prep, const float* __restrict__ c,
                                           const float* __restrict__ rcp, size_t padn, int first, int n, size_t /*cc*/) {
    const int q = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const size_t col = (size_t)min(first + 16 * t + (int)(threadIdx.x & 15), n - 1);
      float cv[3], rv[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) { cv[k] = c[k * padn + col]; rv[k] = rcp[k * padn + col]; }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) a += cv[k] * prep[col_feat(k) * 16 + 4 * q + j];
#pragma unroll
        for (int k = 0; k < 3; ++k) a += rv[k] * prep[col_feat(3 + k) * 16 + 4 * q + j];
        colc[t][j] = a;
      }
    }
  }
  __device__ __forceinline__ void operator()(float (&x)[kNE], const f32x4* rowv, float& d, float& mg) const {
    const f32x4 row = rowv[(threadIdx.x & 63) >> 4];
    transpose_quarters(x);
    f32x4 h[4], h2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) { h[t] = colc[t] + row; h2[t] = b2; }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) h[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[s], x[4 * s + t], h[t], 0, 0, 0);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) h2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[s], relu_max(h[t][s]), h2[t], 0, 0, 0);
    float dp[4], mp[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      dp[t] = 0.f; mp[t] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = relu_max(h2[t][j]);
        dp[t] += v * w3d[j];
        mp[t] += v * w3m[j];
      }
    }
    sum_quarters(dp, mp, d, mg);
    d += b3d;
    mg += b3m;
  }
};

template <int HP, bool NT, bool RAW_RSQ, bool UPDATE_STATE>
__device__ __forceinline__ void apply_fc4x_tile(const TensorDev& T, const ApplyTileDev& tile, const float* __restrict__ ws,
                                                const StepArgs& A, const float* __restrict__ tail, Fc4Lds<HP>& L) {
  constexpr int kTrip = narrow_trip_rows(HP);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = T.n;
  const int rsplit = n - tile.c0 > kWave ? 2 : 4;          // wavefronts that share a 64-column segment's rows
  const int seg = wave / rsplit;
  const int c_first = tile.c0 + seg * kWave, col = c_first + lane;
  const bool col_ok = col < n;
  const size_t cc = (size_t)min(col, n - 1);   // lanes past the end compute on the last column and store nothing
  const float* __restrict__ prep = ws + T.oPrep;          // W1s[28][HP] (normalization folded in), b1'[HP]
  const float* rst = T.st + 4 * (size_t)T.padN;   // r_k[3][padm], c_k[3][padn]
  const int rb = tile.r0, r1 = tile.r0 + tile.rows;
  const size_t pN = T.padN;
  struct In { float g, p, m1, m2, m3, v; };
  auto fetch = [&](int r) __attribute__((always_inline)) {   // rows past the tile read its last row
    const size_t ro = (size_t)min(r, r1 - 1) * n + cc;
    In x;
    x.g = ld1<NT>(T.g + ro); x.p = ld1<NT>(T.p + ro);
    x.m1 = ld1<NT>(T.st + ro); x.m2 = ld1<NT>(T.st + pN + ro); x.m3 = ld1<NT>(T.st + 2 * pN + ro); x.v = ld1<NT>(T.st + 3 * pN + ro);
    return x;
  };
  const int r_first = rb + kTrip * (wave % rsplit);
  In cur[kTrip];
#pragma unroll
  for (int e = 0; e < kTrip; ++e) cur[e] = fetch(r_first + e);
  for (int i = threadIdx.x; i < tile.rows * HP; i += kBlock) {
    const int lrow = i / HP, u = i - lrow * HP, row = rb + lrow;
    float a = prep[kNF * HP + u];
#pragma unroll
    for (int k = 0; k < 3; ++k) a += rst[(size_t)k * T.padm + row] * prep[row_feat(k) * HP + u];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float rr = ws[T.oRR + (size_t)k * T.padm + row];
      a += rr * prep[row_feat(3 + k) * HP + u];
      if (u == 0) L.rr[lrow][k] = rr;
    }
    reinterpret_cast<float*>(&L.rowv[lrow][0])[u] = a;
  }
  Mlp<HP> mlp;
  mlp.load(prep, tail);
  float rc[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) rc[k] = ws[T.oRC + (size_t)k * T.padn + cc];
  mlp.load_col(prep, rst + 3 * (size_t)T.padm, ws + T.oRC, T.padn, min(c_first, n - 1), n, cc);
  const float eps = A.eps_acc, lr = A.lr, wd = A.wd;
  const float bm1 = A.mom_decay[0], bm2 = A.mom_decay[1], bm3 = A.mom_decay[2], bv = A.rms_decay;
  const float am1 = 1.0f - bm1, am2 = 1.0f - bm2, am3 = 1.0f - bm3, av = 1.0f - bv;
  __syncthreads();
  if (c_first < n) {   // wavefront-uniform
    for (int r = r_first; r < r1; r += kTrip * rsplit) {
      In nxt[kTrip];
#pragma unroll
      for (int e = 0; e < kTrip; ++e) nxt[e] = fetch(r + kTrip * rsplit + e);
#pragma unroll
      for (int e = 0; e < kTrip; ++e) {
        if (r + e >= r1) break;   // wavefront-uniform
        const int lrow = r + e - rb;
        const size_t ro = (size_t)(r + e) * n + cc;
        const float g = cur[e].g, p = cur[e].p;
        float q1 = cur[e].m1, q2 = cur[e].m2, q3 = cur[e].m3, v = cur[e].v;
        if (UPDATE_STATE) {   // the statistics pass's operations, in its order: the same bits
          q1 = __builtin_fmaf(bm1, q1, am1 * g);
          q2 = __builtin_fmaf(bm2, q2, am2 * g);
          q3 = __builtin_fmaf(bm3, q3, am3 * g);
          v = __builtin_fmaf(bv, v, av * (g * g));
          if (col_ok) {
            st1<NT>(q1, T.st + ro); st1<NT>(q2, T.st + pN + ro); st1<NT>(q3, T.st + 2 * pN + ro); st1<NT>(v, T.st + 3 * pN + ro);
          }
        }
        const float rs = RAW_RSQ ? __builtin_amdgcn_rsqf(v + eps) : rsqrtf(v + eps);
        const float4 rr = *reinterpret_cast<const float4*>(L.rr[lrow]);
        const float f0 = rr.x * rc[0], f1 = rr.y * rc[1], f2 = rr.z * rc[2];
        float x[kNE] = {g, p, q1, q2, q3, v, q1 * rs, q2 * rs, q3 * rs, rs, g * f0, g * f1, g * f2, q1 * f0, q2 * f1, q3 * f2};
        float d, mg;
        mlp(x, L.rowv[lrow], d, mg);
        const float delta = d * expf(mg * A.exp_mult) * A.step_mult;
        if (col_ok) st1<NT>(p - lr * (delta + wd * p), T.p + ro);
        __builtin_amdgcn_sched_barrier(0);   // one row at a time: bounds the registers
      }
#pragma unroll
      for (int e = 0; e < kTrip; ++e) cur[e] = nxt[e];
    }
  }
}

}  // namespace

// Persistent workgroups: the first tile is the workgroup's number, the next ones come from a counter (k_finalize cleared
// it); the table's last tiles are shorter, so that a launch does not end on a nearly empty last round.
template <int HP, bool RAW_RSQ, bool UPDATE_STATE>
__global__ void __launch_bounds__(kBlock, narrow_waves_per_simd(HP)) k_apply_fc4x(const TensorDev* __restrict__ tensors,
                                                                               const ApplyTileDev* __restrict__ atiles, int n_atiles,
                                                                               int* __restrict__ next_tile, float* __restrict__ ws,
                                                                               StepArgs A, const float* __restrict__ tail, bool off_grid_nt) {
  __shared__ Fc4Lds<HP> L;
  __shared__ int s_tile;
  for (int tile_id = blockIdx.x; tile_id < n_atiles; tile_id = s_tile) {   // workgroup-uniform
    const ApplyTileDev tile = atiles[tile_id];
    const TensorDev& T = tensors[tile.tensor];
    // nontemporal accesses where no line is shared between wavefronts (rows on the 128-byte grid), and by choose_loads
    if (T.vec == 2 || (T.vec == 0 && off_grid_nt)) apply_fc4x_tile<HP, true, RAW_RSQ, UPDATE_STATE>(T, tile, ws, A, tail, L);
    else apply_fc4x_tile<HP, false, RAW_RSQ, UPDATE_STATE>(T, tile, ws, A, tail, L);
    __syncthreads();   // every wavefront is done with this tile's tables and has read s_tile
    if (n_atiles <= (int)gridDim.x) break;   // one tile each: nobody asks (see k_apply_f16s)
    if (threadIdx.x == 0) s_tile = (int)gridDim.x + atomicAdd(next_tile, 1);
    __syncthreads();
  }
}

bool apply_fc4x_available(const StepArgs& A) { return A.kind == LOPT_SMALL_FC && A.HP <= 16; }

void launch_apply_fc4x(const Launch& L, const StepArgs& A, const WeightsDev& W, bool update_state, hipStream_t s) {
  if (L.n_atiles == 0) return;
  // v_rsq_f32 treats inputs below the smallest normal float as zero; with eps_acc that small the kernel takes the library
  // reciprocal square root (which rescales such inputs) instead of the bare instruction
  const bool raw = A.eps_acc >= 1e-30f;
  const int resident = L.resident_wgs / 2 * narrow_waves_per_simd(A.HP);   // (resident_wgs counts two workgroups per CU)
  const int grid = L.n_atiles < resident ? L.n_atiles : resident;
#define LOPT_LAUNCH_FC4X(HP, R, U)                                                                                    \
  hipLaunchKernelGGL((k_apply_fc4x<HP, R, U>), dim3(grid), dim3(kBlock), 0, s, L.tensors, L.atiles, L.n_atiles,       \
                     L.apply_counter, L.ws, A, W.mlp_tail, L.off_grid_nt)
#define LOPT_LAUNCH_FC4X_W(HP)                          \
  do {                                                  \
    if (raw && update_state) LOPT_LAUNCH_FC4X(HP, true, true);  \
    else if (raw) LOPT_LAUNCH_FC4X(HP, true, false);    \
    else if (update_state) LOPT_LAUNCH_FC4X(HP, false, true);   \
    else LOPT_LAUNCH_FC4X(HP, false, false);            \
  } while (0)
  if (A.HP == 4) LOPT_LAUNCH_FC4X_W(4);
  else if (A.HP == 8) LOPT_LAUNCH_FC4X_W(8);
  else LOPT_LAUNCH_FC4X_W(16);
#undef LOPT_LAUNCH_FC4X_W
#undef LOPT_LAUNCH_FC4X
}

}  // namespace lopt
