// Device-side helpers shared by the kernels: wavefront reductions and masked float4 access.
#pragma once

#include "lopt_internal.h"

namespace lopt {

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// Sum over the 64 lanes of a wavefront; every lane gets the result. Fixed order.
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f<0x141>(v);  // row_half_mirror
  v += dpp_f<0x140>(v);  // row_mirror: every lane of a row of 16 holds the row's sum
  float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  float b = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
  float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
  return (a + b) + (c + d);
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xF, 0xF, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double readlane_d(double v, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// The same in double.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_d<0xB1>(v);
  v += dpp_d<0x4E>(v);
  v += dpp_d<0x141>(v);
  v += dpp_d<0x140>(v);
  return (readlane_d(v, 0) + readlane_d(v, 16)) + (readlane_d(v, 32) + readlane_d(v, 48));
}

typedef float f32x4n __attribute__((ext_vector_type(4)));

// Four columns of a row segment of a streamed array. `seg`: the segment's first element, wave-uniform; `off`: this lane's offset in
// BYTES. The access goes through a buffer descriptor of `bytes` bytes, what is left of the row: scalar base + 32-bit vector offset, and
// the hardware checks every dword by itself, so that columns past the row's end read as 0 and are not written. Rows may start
// anywhere: a four-dword access needs only the dword's alignment. Off the grid a wavefront's access touches nine 128-byte lines, on it
// eight; one dword per lane and column touches three lines for every two.
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));

// Bytes of a row from column c0 on, as far as a 256-column segment reaches.
__device__ __forceinline__ unsigned segment_bytes(int n, int c0) { return 4u * (unsigned)min(n - c0, kTileCols); }

template <bool NT>
constexpr int kBufferAux = NT ? 2 : 0;   // nontemporal
__device__ __forceinline__ __amdgpu_buffer_rsrc_t segment_rsrc(const float* seg, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)seg, 0, (int)bytes, 0x00020000);   // raw buffer, 32-bit data
}
template <bool NT>
__device__ __forceinline__ f32x4v load_quad(const float* seg, unsigned off, unsigned bytes) {
  return __builtin_bit_cast(f32x4v, __builtin_amdgcn_raw_buffer_load_b128(segment_rsrc(seg, bytes), (int)off, 0, kBufferAux<NT>));
}
__device__ __forceinline__ float load_one(const float* seg, unsigned off, unsigned bytes) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(segment_rsrc(seg, bytes), (int)off, 0, kBufferAux<false>));
}
__device__ __forceinline__ void store_one(float* seg, unsigned off, unsigned bytes, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), segment_rsrc(seg, bytes), (int)off, 0, kBufferAux<false>);
}
template <bool NT>
__device__ __forceinline__ void store_quad(float* seg, unsigned off, unsigned bytes, f32x4v v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4v, v), segment_rsrc(seg, bytes), (int)off, 0, kBufferAux<NT>);
}

// Narrow tensors, up to kNarrowCols columns: with four columns a lane most lanes of a row access would idle. A lane owns ONE column of a
// 64-column segment, and where several rows fit into the 64 lanes the wavefront takes that many at a time: consecutive rows of a tensor are
// consecutive in memory, so the access is one contiguous run of dwords. The wavefronts of the tile share out its rows (two segments:
// two wavefronts each). us a step with four columns and one row an access / this way: 4.2 M elements in 9, 3, 33 and 65 columns, width 32 858 / 588, VeLO
// 911 / 134; in 8, 4, 32 and 64 columns 907 / 579 and 990 / 115; twenty of 6000x27 under VeLO 181 / 78; twelve of 4000x101 102 / 88, of 4000x127 120 /
// 109, of 4000x128 109.7 / 106. From 129 columns on a lane in two works with four columns: 4000x133, four columns / one (64-column
// segments) 126 / 131, 4000x161 138 / 143.
constexpr int kNarrowCols = 128;
struct NarrowWalk {
  int col;             // this lane's column (col_ok: it is one)
  bool col_ok;
  int rows, sub;       // rows of one access, this lane's among them
  unsigned off;        // offset of the lane's element from the first row's first, in bytes
  int first, step;     // the wavefront's first row, from the tile's first, and the distance to its next for `per_trip` accesses a trip
  __device__ __forceinline__ NarrowWalk(int n, int per_trip) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int two = n > kWave ? 1 : 0, seg = two ? wave >> 1 : 0, share = two ? wave & 1 : wave;
    rows = n > kWave ? 1 : kWave / n;
    sub = n > kWave ? 0 : lane / n;
    col = seg * kWave + lane - sub * n;
    col_ok = sub < rows && col < n;
    off = 4u * (unsigned)(sub * n + col);
    first = share * per_trip * rows;
    step = (two ? 2 : 4) * per_trip * rows;
  }
};

// Load four consecutive floats starting at column `col` of a row of length n whose first
// element is at `row`. VEC: the address is 16-byte aligned and n % 4 == 0.
template <bool VEC>
__device__ __forceinline__ float4 load4(const float* __restrict__ row, int col, int n) {
  if (VEC) {
    if (col < n) return *reinterpret_cast<const float4*>(row + col);
    return make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col < n) v.x = row[col];
  if (col + 1 < n) v.y = row[col + 1];
  if (col + 2 < n) v.z = row[col + 2];
  if (col + 3 < n) v.w = row[col + 3];
  return v;
}

// The same for the big streamed arrays (g, p, M, V): every element is touched once per pass and the
// working set is far larger than the caches, so the accesses are marked nontemporal (measured +5 % on a
// 6-read/4-write stream).
template <bool VEC>
__device__ __forceinline__ float4 load4s(const float* __restrict__ row, int col, int n) {
  if (VEC) {
    if (col < n) {
      const f32x4n v = __builtin_nontemporal_load(reinterpret_cast<const f32x4n*>(row + col));
      return make_float4(v.x, v.y, v.z, v.w);
    }
    return make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col < n) v.x = __builtin_nontemporal_load(row + col);
  if (col + 1 < n) v.y = __builtin_nontemporal_load(row + col + 1);
  if (col + 2 < n) v.z = __builtin_nontemporal_load(row + col + 2);
  if (col + 3 < n) v.w = __builtin_nontemporal_load(row + col + 3);
  return v;
}

template <bool VEC>
__device__ __forceinline__ void store4s(float* __restrict__ row, int col, int n, float4 v) {
  if (VEC) {
    if (col < n) {
      const f32x4n w = {v.x, v.y, v.z, v.w};
      __builtin_nontemporal_store(w, reinterpret_cast<f32x4n*>(row + col));
    }
    return;
  }
  if (col < n) __builtin_nontemporal_store(v.x, row + col);
  if (col + 1 < n) __builtin_nontemporal_store(v.y, row + col + 1);
  if (col + 2 < n) __builtin_nontemporal_store(v.z, row + col + 2);
  if (col + 3 < n) __builtin_nontemporal_store(v.w, row + col + 3);
}

// Rows [r0, r1) of a statistics tile. Row counters are unsigned wherever a loop steps past its end or clamps a row ahead of it:
// a tensor may have 2^31 - 1 rows, and such a counter runs up to TR + 16 further.
struct TileRows { unsigned r0, r1; };
__device__ __forceinline__ TileRows tile_rows(const TensorDev& T, const TileDev& tile) {
  const unsigned r0 = (unsigned)tile.ti * (unsigned)T.TR;
  return TileRows{r0, min(r0 + (unsigned)T.TR, (unsigned)T.m)};
}

// The rows and the 256-column segment of a tile that one of the workgroup's four wavefronts streams (for passes that may cut
// the elements in any way). Workgroups advance through their rows more or less in step, and tiles of power-of-two pitch
// then keep meeting on the same few of the 128 memory channels (4 KB interleave: rows 512 KB apart share one). Where the
// row is a multiple of 4 KB the walk is changed, by what measured best (VeLO step, four tensors of 16.8 M elements):
//   up to 12 KB  the four workgroups of a group of four adjacent tiles cut their common rows into quarters and every wavefront
//                takes a segment of its own, so that a row access of the workgroup is 4 KB contiguous
//                (1024 columns 1.009 -> 0.907 ms, 2048 1.161 -> 0.894, 3072 0.915 -> 0.890)
//   longer       every fourth row, as for other rows, but starting at a place that differs from tile to tile
//                (4096 columns 0.932 -> 0.887 ms, 6144 0.934 -> 0.882, 8192 0.875 -> 0.867; the first form: 0.945, 0.928, 1.10)
// Other rows measured the same or up to 4 % slower with either. Their wavefronts take a quarter of the tile's rows each, one after the
// other (against every fourth row: 4352 columns 957 -> 949 us, 4128 1027 -> 997, 4100 967 -> 957, 3840 848 -> 842, ViT-B/16 shapes
// the same, 4224 918 -> 927).
struct RowWalk { int tj, base, cnt, rot, step; };
__device__ __forceinline__ RowWalk plain_walk(const TensorDev& T, const TileDev& tile, int wave) {   // rows r0 + wave + 4 i
  const int r0 = tile.ti * T.TR;
  return RowWalk{tile.tj, r0 + wave, (min(T.TR, T.m - r0) - wave + 3) >> 2, 0, 4};
}
__device__ __forceinline__ RowWalk row_walk(const TensorDev& T, const TileDev& tile, int wave) {
  const int r0 = tile.ti * T.TR;
  const bool pitch = (T.n & 1023) == 0;
  if (pitch && T.n <= 3072) {   // n % 1024 == 0: every group of four tiles is complete
    const int quarter = T.TR / 4, b = r0 + (tile.tj & 3) * quarter;   // TR is a multiple of 8
    return RowWalk{(tile.tj & ~3) + wave, b, min(quarter, T.m - b), 0, 1};
  }
  const int rows = min(T.TR, T.m - r0);
  if (!pitch) {
    const int per = (rows + 3) >> 2, b = wave * per;
    return RowWalk{tile.tj, r0 + b, min(per, rows - b), 0, 1};
  }
  const int cnt = (rows - wave + 3) >> 2;   // rows r0 + wave + 4 i
  return RowWalk{tile.tj, r0 + wave, cnt, cnt > 0 ? tile.ti * 7 % cnt : 0, 4};
}
__device__ __forceinline__ int walk_row(const RowWalk& w, int i) {   // 0 <= i < cnt (cnt <= 0: no rows)
  int k = i + w.rot;
  k = k >= w.cnt ? k - w.cnt : k;
  return w.base + w.step * k;
}

__device__ __forceinline__ float get(const float4& v, int i) {
  return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}


}  // namespace lopt
