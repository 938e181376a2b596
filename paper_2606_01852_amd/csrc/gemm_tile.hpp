// What the MFMA GEMM kernels share (device, internal): vector types, the
// order in which workgroups take the tiles of a GEMM, and the stores of a
// wave's accumulators.
#pragma once

#include "gemm_common.hpp"

namespace tnc {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef short s8v __attribute__((ext_vector_type(8)));

constexpr int GROUP_M = 8;

struct TileCoord {
  int64_t b, row0, col0;
};

// Tile of workgroup index `wg` (already in XCD order) within one GEMM:
// batch entry, then groups of GROUP_M M-tiles swept along N.
template <int BM, int BNC>
__device__ __forceinline__ TileCoord tile_of(int64_t wg, int64_t tiles_m, int64_t tiles_n) {
  const int64_t tpb = tiles_m * tiles_n;
  const int64_t b = wg / tpb;
  const int64_t r = wg - b * tpb;
  const int64_t gw = static_cast<int64_t>(GROUP_M) * tiles_n;
  const int64_t grp = r / gw;
  const int64_t first_m = grp * GROUP_M;
  const int64_t rem_m = tiles_m - first_m;
  const int64_t gsz = rem_m < GROUP_M ? rem_m : GROUP_M;
  const int64_t rr = r - grp * gw;
  TileCoord tc;
  tc.b = b;
  tc.row0 = (first_m + rr % gsz) * BM;
  tc.col0 = (rr / gsz) * BNC;
  return tc;
}

template <int BM, int BNC>
__device__ __forceinline__ TileCoord map_tile(int64_t tiles_m, int64_t tiles_n, int64_t total) {
  int64_t wg = blockIdx.x;
  const int64_t per = total >> 3;
  if (wg < (per << 3)) wg = (wg & 7) * per + (wg >> 3);
  return tile_of<BM, BNC>(wg, tiles_m, tiles_n);
}

// The same 8 x 4 blocks of tiles per XCD, but the eight XCDs work on the
// same eight M-tiles at once (XCD x takes N-tiles x, x + 8, ...): the A
// panels every XCD reads from its own L2 are then shared in the memory-side
// cache, so HBM serves each once instead of once per XCD.  Needs whole
// groups of 64 tiles (tiles_n a multiple of 8, GROUP_M M-tiles per group);
// other shapes keep map_tile's order.
template <int BM, int BNC>
__device__ __forceinline__ TileCoord map_tile_shared(int64_t tiles_m, int64_t tiles_n, int64_t total) {
  const int64_t wg = blockIdx.x;
  if (tiles_n % 8 != 0 || tiles_m % GROUP_M != 0) return map_tile<BM, BNC>(tiles_m, tiles_n, total);
  const int64_t g = wg >> 3, x = wg & 7;
  return tile_of<BM, BNC>(64 * (g >> 3) + 8 * x + (g & 7), tiles_m, tiles_n);
}

// Output offsets within one batch entry of C, in complex elements: a row's
// (offM[row], or row * n) plus a column's (offN[col], or col); -1 marks a
// row or column outside C.  Permuted-store epilogues read them into
// registers before issuing any store: C and the store tables are different
// arrays, but the compiler cannot know it, so a table read between two
// stores would wait for each read in turn.  (Row-major stores compute their
// addresses inline: that keeps the main loop's register allocation, and so
// its schedule, as it is without tables.)
__device__ __forceinline__ int64_t col_offset(const GemmDesc& d, bool perm, int64_t col) {
  return col < d.n ? (perm ? d.offN[col] : col) : -1;
}

// Rows 8*(v>>2) + 4*h + (v&3) of a 32-row MFMA block starting at row0, for
// v = v0 .. v0+7 (the accumulator layout of a 32x32 MFMA).
__device__ __forceinline__ void row_offsets8(const GemmDesc& d, bool perm, int64_t row0, int h, int v0,
                                             int64_t (&o)[8]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int v = v0 + u;
    const int64_t row = row0 + 8 * (v >> 2) + 4 * h + (v & 3);
    o[u] = row < d.m ? (perm ? d.offM[row] : row * d.n) : -1;
  }
}

// Permuted store of a wave's 64 x 32 complex block held in the 4M layout
// (MFMA 32x32 accumulators over real columns: even lanes hold the real and
// odd lanes the imaginary part of one complex column, for rows v and v+1 of
// each register pair).  One lane swap lets the even lane store row v's
// complex value and the odd lane row v+1's, as 8-byte stores (half the
// store instructions of a 4-byte store per part); each lane reads only the
// row offsets of the rows it stores.  The swap runs in both lanes of a pair
// whatever their row bounds (the column bound is shared by the pair).
// val(i, j, v) is the lane's accumulated value of MFMA block (i, j), entry v.
template <int PW = 1, class Val>
__device__ __forceinline__ void store_perm_pairs(const GemmDesc& d, const TileCoord& tc, int wm, int wn, int lane,
                                                 Val val) {
  constexpr int NJ = 2 * PW;  // 32-real-column blocks per wave
  const int h = lane >> 5, l32 = lane & 31;
  const bool odd = l32 & 1;
  float2* Cz = d.C + tc.b * d.m * d.n;
  int64_t co[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) co[j] = col_offset(d, true, (tc.col0 * 2 + wn * 64 * PW + j * 32 + l32) >> 1);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v0 = 0; v0 < 16; v0 += 8) {
      // this lane stores rows v = v0 + 2t + odd of the 32-row block
      int64_t ro[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int v = v0 + 2 * t + (odd ? 1 : 0);
        const int64_t row = tc.row0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        ro[t] = row < d.m ? d.offM[row] : -1;
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (co[j] < 0) continue;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float a0 = val(i, j, v0 + 2 * t), a1 = val(i, j, v0 + 2 * t + 1);
          const int sent = __builtin_bit_cast(int, odd ? a0 : a1);
          // quad_perm [1,0,3,2]: exchange with the neighbouring lane
          const float got = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, sent, 0xB1, 0xF, 0xF, false));
          if (ro[t] >= 0) Cz[ro[t] + co[j]] = odd ? make_float2(got, a1) : make_float2(a0, got);
        }
      }
    }
}

// Store of a wave's 64 x 32 PW complex block held in the 4M layout, row-major
// or through the offset tables; val as for store_perm_pairs.
template <int PW, class Val>
__device__ __forceinline__ void store_4m(const GemmDesc& d, bool perm, const TileCoord& tc, int wm, int wn, int lane,
                                         Val val) {
  if (perm) {
    store_perm_pairs<PW>(d, tc, wm, wn, lane, val);
    return;
  }
  const int h = lane >> 5, l32 = lane & 31;
  // real column tc.col0 * 2 + 64 PW wn + 32 j + l32: complex column >> 1, re/im by parity
  float* C = reinterpret_cast<float*>(d.C + tc.b * d.m * d.n) + (l32 & 1);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2 * PW; ++j) {
      const int64_t col = (tc.col0 * 2 + wn * 64 * PW + j * 32 + l32) >> 1;
      if (col >= d.n) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = tc.row0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (row < d.m) C[2 * (row * d.n + col)] = val(i, j, v);
      }
    }
}

// Store of a wave's 64 x 32 complex block from the 3M products (one 32x32
// accumulator block per 32 rows: T1 = Ar Br, T2 = Ai Bi, T3 = (Ar+Ai)(Br+Bi);
// Re = T1 - T2, Im = T3 - T1 - T2), row-major or through the offset tables.
__device__ __forceinline__ void store_3m(const GemmDesc& d, bool perm, const TileCoord& tc, int wm, int wn, int lane,
                                         const f16v (&t1)[2], const f16v (&t2)[2], const f16v (&t3)[2]) {
  const int h = lane >> 5, l32 = lane & 31;
  if (!perm) {  // row-major [M|N]: addresses from the indices alone
    const int64_t col = tc.col0 + wn * 32 + l32;
    if (col >= d.n) return;
    float2* C = d.C + tc.b * d.m * d.n + col;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = tc.row0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (row < d.m) {
          float2 o;
          o.x = t1[i][v] - t2[i][v];
          o.y = t3[i][v] - t1[i][v] - t2[i][v];
          C[row * d.n] = o;
        }
      }
    return;
  }
  const int64_t co = col_offset(d, perm, tc.col0 + wn * 32 + l32);
  if (co < 0) return;
  float2* C = d.C + tc.b * d.m * d.n + co;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v0 = 0; v0 < 16; v0 += 8) {
      int64_t ro[8];
      row_offsets8(d, perm, tc.row0 + wm * 64 + i * 32, h, v0, ro);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int v = v0 + u;
        if (ro[u] >= 0) {
          float2 o;
          o.x = t1[i][v] - t2[i][v];
          o.y = t3[i][v] - t1[i][v] - t2[i][v];
          C[ro[u]] = o;
        }
      }
    }
}

}  // namespace tnc
