// Complex GEMM in the 4M form on the bf16 matrix pipe,
// C[b,i,j] = sum_l A[b,i,l] B[b,j,l]:  complex64 at float32 precision (three
// bf16 parts an operand), and split precision (two).
//
// complex64.  A float32 has 24 significant bits, a bf16 eight, so x = hi + mid + lo with
// hi = rne(x), mid = rne(x - hi), lo = x - hi - mid, every difference and lo
// itself exact: the operands keep all their bits.  Of the nine products of
// two such sums six are formed (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi;
// the others are below 2^-24 of the product, about 2^-26 rms), each exact in
// float32, and added up by the bf16 MFMA in float32: one rounding per 16
// products, where the FP32 MFMA is a chain of FMAs.  A stage's six products of
// a block are summed from zero and the VALU adds the sum to the accumulator:
// one rounding at the accumulator's size per 16 terms instead of 16.  Error
// against the FP32 MFMA's, k = 16 .. 16384: 0.42 .. 0.26 of it for CN(0,1)
// operands, 0.55 .. 0.36 for real ones, 0.79 .. 0.44 for magnitudes over 2^30.
// Sums of few terms pay for the products left out and for the MFMA's cutting
// bits off where an FMA rounds: rms, in units of 2^-24 of the terms' size, FP32
// MFMA and here, one real term that is not zero 0.42 and 0.58 (largest 1.0 and
// 2.7), two 0.44 and 0.63, four 0.45 and 0.49, six 0.46 and 0.42, 64 0.47 and 0.23.
// (With the six products accumulated in place: 0.64 .. 1.05, 0.9 .. 1.3 and
// 1.0 .. 1.6, at 3 % less time: not kept.)
//
// What bounds it: power.  8192 x 8192 x 4096 on random values runs at 225-232
// complex TFLOP/s (the FP32 MFMA kernel before it: 139-140, its pipe's rate),
// 1350-1390 executed bf16 TFLOP/s, while the library's own bf16 matrix
// product sustains 1200; on zeros, where the clock stays up, the same code
// runs at 320.  So the order of the products counts: with one operand kept
// from each MFMA to the next 220 -> 225-232.  64 x 1024 x 256 x 1024: 135 ->
// 210-214; 2048 x 512 x 512 x 512: 136 -> 201; 6 x 1000 x 500 x 777: 82 ->
// 149 (odd k: rows are read 16 bytes at a time on 8-byte boundaries).
//
// The stage's code is dealt out by hand: after every MFMA (32 cycles) a few
// VALU operations of the next stage's split or of the last block's sum, so
// that one wave alone keeps the pipe busy (without: 206 instead of 218).
//
// Every input that a float32 can hold means what it means to float32
// arithmetic.  Both operands are scaled by 2^24 on their way in, so the split
// is exact for all of them, subnormals included; an operand with values of
// 2^30 or more is left as it is, and there a remainder that is a subnormal
// float32 (|x| below about 2^-102: bf16 has no bits there) is noticed while it
// is staged.  Such tiles, and those whose sums are not finite (infinities,
// NaNs, and sums past 2^80 where both operands were scaled), are computed
// again on the FP32 pipe.  2048^3, ms: 0.330 whatever small values there are
// (1.67 when one value below 2^-102 sent its tile to the FP32 pass, which
// then waited for every read), 0.343 with operands of 2^43, 0.914 with an
// infinity in every tile (1.67; all on the FP32 pipe: 0.544).  The scaling
// takes two operations for two values and the test for subnormal remainders,
// which the scaled copy of the loop does without, three: 6 x 1000 x 500 x 777
// 113.3 -> 112.7 us, 8192 x 4096 x 4096 4.83 -> 4.84 ms, 30 x 300 x 300 x 64 18.5
// -> 18.8 us.
//
// complex64 in the 3M form runs here as well: 16 x 1024 x 512 x 768 312 us
// on the FP32 pipe with three products, 243 here, at 0.3 of the error.
//
// Split precision (hi and lo, three products hi lo, lo hi, hi hi, the first two
// added to an accumulator of their own, in the 256 x 128 tile all to one)
// is the same tile with a part less and no FP32 pass: what the operands lose
// is the format's own.  Bound by power too, 1275 executed bf16 TFLOP/s: 64 x
// 1024 x 256 x 1024 0.390 -> 0.369 ms against tiles whose staging the
// compiler dealt out, 2048 x 512 x 512 x 512 6.35 -> 5.95, 6 x 1000 x 500 x
// 776 82.5 -> 70.9 us; shapes for few tiles as for complex64 (4 x 256 x 4096
// x 1024 as a planned pair 219 -> 150 us).
//
// 4M form as one real GEMM of m x 2n x 2k: a complex row of A read as 2k
// floats, times (br, -bi, ...) for Re C and (bi, br, ...) for Im C; both real
// rows of B' are laid out at staging (a sign flip and a swap of packed
// halves).
#include <atomic>
#include <type_traits>

#include "gemm_tile.hpp"

namespace tnc {

namespace {

constexpr int XK = 8;  // complex k per LDS stage: 16 real, one bf16 MFMA step

// The next part of x and y, packed [x | y << 16], which it is taken off.
__device__ __forceinline__ uint32_t take_part(float& x, float& y) {
#pragma clang fp contract(off)
  typedef float fv2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bv2 __attribute__((ext_vector_type(2)));
  const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector((fv2){x, y}, bv2));
  x -= __uint_as_float(w << 16);
  y -= __uint_as_float(w & 0xFFFF0000u);
  return w;
}

// The last part.  It is what is left of x and y, exactly, unless that is a
// subnormal float32: `tiny` keeps the smallest (bits << 1) - 1 seen, where
// zero wraps to the top and a subnormal value ends up below 0x00ffffff.
__device__ __forceinline__ uint32_t last_part(float x, float y, uint32_t& tiny) {
  typedef float fv2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bv2 __attribute__((ext_vector_type(2)));
  const uint32_t tx = (__float_as_uint(x) << 1) - 1, ty = (__float_as_uint(y) << 1) - 1;
  const uint32_t t = tx < ty ? tx : ty;
  tiny = tiny < t ? tiny : t;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((fv2){x, y}, bv2));
}

// Scaled by 2^24 every float32's last bit is 2^-125 or more, so the three parts
// of every value are normal; operands that are scaled hold values below 2^30,
// as far as they were looked at.
constexpr int kScale = 24;
constexpr float kScaleBelow = 1073741824.f;
__device__ __forceinline__ float pow2(int e) { return __int_as_float((127 + e) << 23); }
// Whether a wave's lanes all have values that may be scaled (uniform).
__device__ __forceinline__ bool scalable(float largest) {
  return __builtin_amdgcn_ballot_w64(!(largest < kScaleBelow)) == 0;
}
__device__ __forceinline__ float largest_of(const f4& v) {
  return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)));
}

// f(integral_constant 0), ..., f(N - 1): loops whose counters index registers
template <int N, int I = 0, class F>
__device__ __forceinline__ void each(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    each<N, I + 1>(f);
  }
}

// A tile's coordinates in scalar registers (every lane has the same).
__device__ __forceinline__ int64_t uniform(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
  return static_cast<int64_t>((uint64_t{hi} << 32) | lo);
}
__device__ __forceinline__ TileCoord uniform(const TileCoord& t) {
  return {uniform(t.b), uniform(t.row0), uniform(t.col0)};
}

typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));  // rows of odd length start on 8 bytes

// BI x BJ blocks of 32 x 16 complex of C again, by one wave on the FP32 pipe,
// straight from global memory and back: right for every float32.  Stages of
// four complex k, the next one's values on their way: with 2 x 2 blocks 16
// MFMAs of 64 cycles, and the same of the other wave on the SIMD, cover a read.
template <int BI, int BJ>
__device__ __forceinline__ void fp32_blocks(const GemmDesc& d, int64_t b, int64_t row0, int64_t col0, int lane) {
  if (row0 >= d.m || col0 >= d.n) return;
  int64_t oa, ob;
  batch_offsets(d, b, oa, ob);
  const int64_t ld = row_stride(d), k = d.k, n = (k + 3) / 4;
  const int h = lane >> 5, l32 = lane & 31;
  const bool odd = lane & 1;
  const float2 *pa[BI], *pb[BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int64_t r = row0 + 32 * i + l32;
    pa[i] = d.A + uniform(oa) + (r < d.m ? r : d.m - 1) * ld;
  }
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    const int64_t r = col0 + 16 * j + (l32 >> 1);
    pb[j] = d.B + uniform(ob) + (r < d.n ? r : d.n - 1) * ld;
  }
  f4 x[2][BI], y[2][BJ];  // two complex values of each row: k 4 st + 2 h and the next
  auto fetch = [&](const float2* row, int64_t l) {
    if (l + 2 <= k) return static_cast<f4>(*reinterpret_cast<const f4u*>(row + l));
    f4 v = {0.f, 0.f, 0.f, 0.f};
    if (l < k) {
      v.x = row[l].x;
      v.y = row[l].y;
    }
    return v;
  };
  auto load = [&](auto set, int64_t st) {
    const int64_t l = 4 * st + 2 * h;
#pragma unroll
    for (int i = 0; i < BI; ++i) x[set][i] = fetch(pa[i], l);
#pragma unroll
    for (int j = 0; j < BJ; ++j) y[set][j] = fetch(pb[j], l);
  };
  f16v c[BI][BJ] = {};
  auto multiply = [&](auto set) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int j = 0; j < BJ; ++j) {
        const float br = y[set][j][2 * e], bi = y[set][j][2 * e + 1];
        const float first = odd ? bi : br, second = odd ? br : -bi;
#pragma unroll
        for (int i = 0; i < BI; ++i) {
          c[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[set][i][2 * e], first, c[i][j], 0, 0, 0);
          c[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[set][i][2 * e + 1], second, c[i][j], 0, 0, 0);
        }
      }
  };
  constexpr std::integral_constant<int, 0> s0{};
  constexpr std::integral_constant<int, 1> s1{};
  load(s0, 0);
  int64_t st = 0;
#pragma unroll 1
  for (; st + 1 < n; st += 2) {
    load(s1, st + 1);
    multiply(s0);
    if (st + 2 < n) load(s0, st + 2);
    multiply(s1);
  }
  if (st < n) multiply(s0);
  // opaque, so that the stores' addresses are not made before the loop
  int at = lane;
  asm volatile("" : "+v"(at));
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    const int64_t col = col0 + 16 * j + (at >> 1 & 15);
    if (col >= d.n) continue;
    float* C = reinterpret_cast<float*>(d.C + b * d.m * d.n) + (at & 1);
    const int64_t co = d.offM ? d.offN[col] : col;
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = row0 + 32 * i + 8 * (v >> 2) + 4 * (at >> 5) + (v & 3);
        if (row < d.m) C[2 * ((d.offM ? d.offM[row] : row * d.n) + co)] = c[i][j][v];
      }
  }
}

// packed parts -> one MFMA operand's product with another
__device__ __forceinline__ f16v mm(const s8v& a, const s8v& b, const f16v& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}
// The six products: parts of A and of B, hi hi last; each shares an operand
// with the one before.
constexpr int kPartA[6] = {0, 0, 1, 1, 2, 0}, kPartB[6] = {2, 1, 1, 0, 0, 0};
// Split precision's three: a_hi b_lo, a_lo b_hi, a_hi b_hi.
constexpr int kSplitA[3] = {0, 1, 0}, kSplitB[3] = {1, 0, 0};

// What the scale of an operand is chosen by, the same in every wave: the first
// two values of 64 of its rows, which the first stage reads as well.
__device__ __forceinline__ f4 sample(const float2* X, int64_t row0, int64_t rows, int64_t ld, int64_t k, int lane) {
  const float2* p = X + (row0 + lane < rows ? row0 + lane : rows - 1) * ld;
  if (k > 1) return *reinterpret_cast<const f4u*>(p);
  return (f4){p->x, p->y, 0.f, 0.f};
}

// PARTS = 3: complex64, 2: split precision.  In complex64 the code from the
// first stage on is there twice, SCALED: both operands are scaled, otherwise
// each as its sample says, with an eye on remainders that bf16 loses (which
// costs three operations for every two values).
template <int PARTS, int WM, int WN, int PW>
struct XTile {
  static constexpr bool EXACT = PARTS == 3;
  static constexpr int BM = 64 * WM, BNC = 32 * WN * PW, NT = 64 * WM * WN;
  static constexpr int NJ = 2 * PW;                      // 32-column blocks of the real view per wave
  static constexpr int PA = BM * 32, PB = 2 * BNC * 32;  // bytes of one part's plane: 16 bf16 per row
  static constexpr int STAGE = PARTS * (PA + PB);
  // LDS holds BUFS stages and is staged AHEAD of the products, with a barrier
  // every AHEAD stages, and the AHEAD stages behind those are on their way to
  // registers: two parts make half the MFMAs of three, so their stages go in
  // pairs (one stage on its way: 20 x 130 x 260 x 900 48.3 us, two 46.2; 40 x 700 x
  // 190 x 300 with its operands in HBM 73.9, 70.7; 1 x 2437 x 2113 x 1999 334, 287).
  static constexpr int BUFS = EXACT ? 2 : 4, AHEAD = BUFS / 2;
  static constexpr size_t kLds = BUFS * STAGE;
  static constexpr int PRODUCTS = EXACT ? 6 : 3;
  static constexpr int AL = BM * 4 / NT, BL = BNC * 4 / NT;  // 16-byte loads per thread and stage
  static_assert(AL >= 1 && AL * NT == BM * 4 && BL >= 1 && BL * NT == BNC * 4, "staging must tile evenly");

  f16v acc[2][NJ];
  // three parts: sums of one stage, of the block at hand and of the one
  // before; two parts: the cross products' sums, except in the 256 x 128 tile,
  // whose eight wide waves have no registers for them (256 x 64 has four, one
  // per SIMD)
  static constexpr bool CROSS = !EXACT && !(PW == 2 && WM * WN > 4);
  static constexpr int WAVES = CROSS && PW == 2 ? 1 : 2;  // per SIMD, at least
  f16v t[2][CROSS ? NJ : 1];
  f4 ra[AHEAD][AL], rb[AHEAD][BL];  // the next AHEAD stages, on their way
  const float2 *pa[AL], *pb[BL];
  uint32_t tiny;
  float sa, sb, un;  // complex64: the operands' scales and what takes them off again

  // rows past the edge repeat the last one: their products are not stored
  __device__ __forceinline__ void init(const float2* A, const float2* B, const GemmDesc& d, const TileCoord& tc,
                                       int tid) {
    const int64_t ld = row_stride(d);
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      int64_t r = tc.row0 + ((tid + NT * i) >> 2);
      r = r < d.m ? r : d.m - 1;
      pa[i] = A + r * ld + 2 * (tid & 3);
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      int64_t r = tc.col0 + ((tid + NT * i) >> 2);
      r = r < d.n ? r : d.n - 1;
      pb[i] = B + r * ld + 2 * (tid & 3);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < (CROSS ? NJ : 1); ++j) t[i][j] = f16v{};
    tiny = 0xFFFFFFFFu;
  }

  // The stage at the pointers, which move on.  CHECK: the row ends `left`
  // complex k (1 .. XK) into it; what would lie behind reads as zero (its
  // last element is loaded instead, so no lane branches).
  template <bool CHECK>
  __device__ __forceinline__ static f4 fetch(const float2*& p, int left, int tid) {
    f4 v;
    if constexpr (CHECK) {
      const int c = 2 * (tid & 3), last = left - 1 - c;
      const float2 x = p[last < 0 ? last : 0], y = p[last < 1 ? last : 1];
      v.x = last >= 0 ? x.x : 0.f;
      v.y = last >= 0 ? x.y : 0.f;
      v.z = last >= 1 ? y.x : 0.f;
      v.w = last >= 1 ? y.y : 0.f;
    } else {
      v = *reinterpret_cast<const f4u*>(p);
    }
    p += XK;
    return v;
  }
  // Staging of a stage, in units of one 16-byte load (the first AL of A, the
  // others of B) and PIECES pieces each, so that it can be dealt out between
  // MFMAs.  LDS rows are 32 bytes, their two 16-byte halves swapped every 8
  // rows (half ^ ((row >> 3) & 1)): the fragment reads of 16 lanes (16 rows,
  // one half) and the 8-byte stores of 32 lanes (8 rows) touch every bank
  // once.  Within 16 rows of B' the even rows come first (row r at ((r & 1) <<
  // 3) | (r >> 1 & 7)), so that the rows that one store instruction writes
  // are neighbours.
  static constexpr int U = AL + BL, PIECES = 2 * PARTS + 2;
  uint32_t w[2][PARTS];  // the unit's parts: of its first and second complex value

  template <int set, int u>
  __device__ __forceinline__ f4& staged() {
    if constexpr (u < AL)
      return ra[set][u];
    else
      return rb[set][u - AL];
  }
  template <bool SCALED, int set, int u, int q>
  __device__ __forceinline__ void piece(char* lds, int tid) {
    const int r = tid >> 2, c = tid & 3;
    f4& v = staged<set, u>();
    if constexpr (q < 2 * PARTS) {
#pragma clang fp contract(off)
      constexpr int e = q / PARTS, part = q % PARTS;
      float x = v[2 * e], y = v[2 * e + 1];
      if constexpr (EXACT && part == 0) {
        x *= u < AL ? sa : sb;
        y *= u < AL ? sa : sb;
      }
      if constexpr (part < 2) {  // (what the second of two parts leaves is not read)
        w[e][part] = take_part(x, y);
        v[2 * e] = x;
        v[2 * e + 1] = y;
      } else {
        w[e][part] = SCALED ? take_part(x, y) : last_part(x, y, tiny);
      }
    } else if constexpr (u < AL) {
      if (q % 2 == 1) return;
      char* p = lds + r * 32 + ((8 * c) ^ (((r >> 3) & 1) << 4)) + u * (NT / 4) * 32;
#pragma unroll
      for (int t = 0; t < PARTS; ++t) *reinterpret_cast<uint2*>(p + t * PA) = make_uint2(w[0][t], w[1][t]);
    } else {
      char* p = lds + PARTS * PA + (((2 * r) & ~15) | (r & 7)) * 32 + (u - AL) * (NT / 4) * 64;
      if constexpr (q % 2 == 0) {
        constexpr uint32_t NEG_IM = 0x80000000u;
#pragma unroll
        for (int t = 0; t < PARTS; ++t)
          *reinterpret_cast<uint2*>(p + t * PB + 8 * c) = make_uint2(w[0][t] ^ NEG_IM, w[1][t] ^ NEG_IM);
      } else {
        auto swap = [](uint32_t x) { return (x >> 16) | (x << 16); };
#pragma unroll
        for (int t = 0; t < PARTS; ++t)
          *reinterpret_cast<uint2*>(p + t * PB + 256 + ((8 * c) ^ 16)) = make_uint2(swap(w[0][t]), swap(w[1][t]));
      }
    }
  }
  template <bool CHECK, int set, int u>
  __device__ __forceinline__ void load_unit(int left, int tid) {
    if constexpr (u < AL)
      ra[set][u] = fetch<CHECK>(pa[u], left, tid);
    else
      rb[set][u - AL] = fetch<CHECK>(pb[u - AL], left, tid);
  }
  // `left` complex k are left of the rows
  template <int set>
  __device__ __forceinline__ void load(int64_t left, int tid) {
    if (left >= XK)
      each<U>([&](auto u) { load_unit<false, set, u>(0, tid); });
    else
      each<U>([&](auto u) { load_unit<true, set, u>(static_cast<int>(left), tid); });
  }
  template <bool SCALED, int set>
  __device__ __forceinline__ void stage(char* lds, int tid) {
    each<U * PIECES>([&](auto q) { piece<SCALED, set, q / PIECES, q % PIECES>(lds, tid); });
  }

  // One stage: the products of `cur`; with NEXT the staged registers are
  // split into `nxt` and loaded again (whole stages).  Three parts: each 32 x
  // 32 block's six products of the stage are summed from zero and then added
  // to its accumulator by the VALU.
  template <bool SCALED, bool NEXT, int set>
  __device__ __forceinline__ void step(const char* cur, char* nxt, int tid, int wm, int wn, int lane) {
    const int h = lane >> 5, r = lane & 31;
    const char* a = cur + (wm * 64 + r) * 32 + ((h ^ ((r >> 3) & 1)) << 4);
    const char* b = cur + PARTS * PA + (wn * 64 * PW + ((r & 16) | ((r & 1) << 3) | ((r >> 1) & 7))) * 32 +
                    ((h ^ (r & 1)) << 4);
    constexpr int SLOTS = 2 * PRODUCTS * NJ, Q = U * PIECES;
    s8v fa[2][PARTS], fb[2][PARTS];
    auto read_a = [&](int i, int q) { fa[i][q] = *reinterpret_cast<const s8v*>(a + q * PA + i * 1024); };
    auto read_b = [&](int j, int q) { fb[j & 1][q] = *reinterpret_cast<const s8v*>(b + q * PB + j * 1024); };
    each<PARTS>([&](auto q) {
      read_a(0, q);
      read_b(0, PARTS - 1 - q);
    });
    __builtin_amdgcn_sched_barrier(0);
    each<SLOTS>([&](auto slot) {
      constexpr int s = slot, c = s / PRODUCTS, kp = s % PRODUCTS, i = c & 1, j = c >> 1;
      if constexpr (EXACT) {
        f16v& sum = t[i][0];
        if constexpr (kp == 0) sum = f16v{};
        sum = mm(fa[i][kPartA[kp]], fb[j & 1][kPartB[kp]], sum);
      } else {
        f16v& sum = CROSS && kp < 2 ? t[i][CROSS ? j : 0] : acc[i][j];
        sum = mm(fa[i][kSplitA[kp]], fb[j & 1][kSplitB[kp]], sum);
      }
      if constexpr (c == 0 && kp < PARTS) read_a(1, kp);
      if constexpr (i == 1 && j + 1 < NJ) {  // the next block's, once this one's part is done with
        if constexpr (kp == 0) read_b(j + 1, 0);
        if constexpr (kp == 1) read_b(j + 1, PARTS - 1);
        if constexpr (EXACT && kp == 3) read_b(j + 1, 1);
      }
      if constexpr (EXACT && kp >= 2) {  // four of the sums of the block before
        f16v& d = acc[i ^ 1][c == 0 ? NJ - 1 : (c - 1) >> 1];
        each<4>([&](auto v) { d[4 * (kp - 2) + v] += t[i ^ 1][0][4 * (kp - 2) + v]; });
      }
      if constexpr (NEXT)
        each<(s + 1) * Q / SLOTS - s * Q / SLOTS>([&](auto n) {
          constexpr int q = s * Q / SLOTS + n;
          piece<SCALED, set, q / PIECES, q % PIECES>(nxt, tid);
          if constexpr (q % PIECES == PIECES - 1) load_unit<false, set, q / PIECES>(0, tid);
        });
      __builtin_amdgcn_sched_barrier(0);
    });
  }

  // The tile's sums; false if they have to come from the FP32 pipe (never with
  // two parts).
  __device__ __forceinline__ bool run(const GemmDesc& d, const TileCoord& tc, char* lds, int tid, int wm, int wn,
                                      int lane) {
    int64_t oa, ob;
    batch_offsets(d, tc.b, oa, ob);
    const float2* A = d.A + uniform(oa);
    const float2* B = d.B + uniform(ob);
    f4 xa, xb;
    if constexpr (EXACT) {
      xa = sample(A, tc.row0, d.m, row_stride(d), d.k, lane);
      xb = sample(B, tc.col0, d.n, row_stride(d), d.k, lane);
    }
    init(A, B, d, tc, tid);
    each<AHEAD>([&](auto q) {
      if (!q || q < (d.k + XK - 1) / XK) load<q>(d.k - q * XK, tid);
    });
    if constexpr (EXACT) {
      const int ea = scalable(largest_of(xa)) ? kScale : 0, eb = scalable(largest_of(xb)) ? kScale : 0;
      sa = pow2(ea);
      sb = pow2(eb);
      un = pow2(-ea - eb);
      if (ea & eb) return add_up<true>(d.k, true, lds, tid, wm, wn, lane);
    }
    const bool busy = tc.row0 + wm * 64 < d.m && tc.col0 + wn * 32 * PW < d.n;
    return add_up<false>(d.k, busy, lds, tid, wm, wn, lane);
  }
  // A stage's staging alone.
  template <bool SCALED, int set>
  __device__ __forceinline__ void pass(char* nxt, int tid) {
    each<U>([&](auto u) {
      each<PIECES>([&](auto q) { piece<SCALED, set, u, q>(nxt, tid); });
      load_unit<false, set, u>(0, tid);
    });
  }
  template <bool SCALED>
  __device__ __forceinline__ bool add_up(int64_t k, bool busy, char* lds, int tid, int wm, int wn, int lane) {
    const int64_t nk = (k + XK - 1) / XK, full = k / XK;
    // stage st goes through register set st % AHEAD
    each<AHEAD>([&](auto q) {
      if (!q || q < nk) stage<SCALED, q>(lds + q * STAGE, tid);
      if (q + AHEAD < nk) load<q>(k - (q + AHEAD) * XK, tid);
    });
    __syncthreads();
    auto buf = [&](int64_t st) { return lds + (st & (BUFS - 1)) * STAGE; };
    // products: a wave with nothing of C only stages (its barriers are the
    // others', one for one)
    auto loop = [&](auto products) {
      int64_t kt = 0;
      for (; kt + 3 * AHEAD - 1 < full; kt += AHEAD) {
        each<AHEAD>([&](auto q) {
          if constexpr (decltype(products)::value)
            step<SCALED, true, q>(buf(kt + q), buf(kt + q + AHEAD), tid, wm, wn, lane);
          else
            pass<SCALED, q>(buf(kt + q + AHEAD), tid);
        });
        __syncthreads();
      }
      for (; kt < nk; kt += AHEAD)
        each<AHEAD>([&](auto q) {
          const int64_t st = kt + q;
          if (q && st >= nk) return;
          if (st + AHEAD < nk) stage<SCALED, q>(buf(st + AHEAD), tid);
          if (st + 2 * AHEAD < nk) load<q>(k - (st + 2 * AHEAD) * XK, tid);
          if constexpr (decltype(products)::value) step<SCALED, false, q>(buf(st), nullptr, tid, wm, wn, lane);
          __syncthreads();
        });
    };
    if (EXACT || busy)
      loop(std::true_type{});
    else
      loop(std::false_type{});
    if constexpr (!EXACT) return true;
    acc[1][NJ - 1] += t[1][0];
    float s = 0.f;  // NaN if any sum is not finite
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) s = fmaf(acc[i][j][v], 0.f, s);
    return !__syncthreads_or((!SCALED && tiny < 0x00FFFFFFu) || !(s == 0.f));
  }

  __device__ __forceinline__ float value(int i, int j, int v) const {
    if constexpr (CROSS)
      return acc[i][j][v] + t[i][j][v];
    else if constexpr (EXACT)
      return acc[i][j][v] * un;
    else
      return acc[i][j][v];
  }

  __device__ __forceinline__ void store(const GemmDesc& d, bool perm, const TileCoord& tc, int wm, int wn,
                                        int lane) const {
    store_4m<PW>(d, perm, tc, wm, wn, lane, [&](int i, int j, int v) { return value(i, j, v); });
  }
};

// A tile of C.
template <int PARTS, int WM, int WN, int PW>
__device__ __forceinline__ void tile(const GemmDesc& d, bool perm, const TileCoord& tc, char* lds, int tid, int wm,
                                     int wn, int lane) {
  XTile<PARTS, WM, WN, PW> t;
  if (t.run(d, tc, lds, tid, wm, wn, lane)) {
    t.store(d, perm, tc, wm, wn, lane);
    return;
  }
#pragma unroll 1
  for (int p = 0; p < PW; ++p)
    fp32_blocks<2, 2>(d, tc.b, tc.row0 + wm * 64, tc.col0 + wn * 32 * PW + 32 * p, lane);
}

template <int PARTS, int WM, int WN, int PW, bool PERM>
__global__ __launch_bounds__(64 * WM * WN, (XTile<PARTS, WM, WN, PW>::WAVES)) void cgemm_4m(GemmDesc d, int64_t tiles_m,
                                                                                  int64_t tiles_n, int64_t total) {
  using T = XTile<PARTS, WM, WN, PW>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TileCoord tc = uniform(map_tile_shared<T::BM, T::BNC>(tiles_m, tiles_n, total));
  tile<PARTS, WM, WN, PW>(d, PERM, tc, lds, tid, wave / WN, wave % WN, lane);
}

// Persistent grouped form: see GroupedEntry.  Tiles are dealt to the 8 XCDs
// in contiguous ranges (tiles of one entry stay on few XCDs, whose L2 they
// share) and each workgroup of an XCD takes every nb-th tile of its range.
template <int PARTS, int WM, int WN, int PW>
__global__ __launch_bounds__(64 * WM * WN, (WM * WN == 4 ? XTile<PARTS, WM, WN, PW>::WAVES : 1)) void cgemm_4m_grouped(
    const GroupedEntry* __restrict__ tab, int n, int64_t total) {
  using T = XTile<PARTS, WM, WN, PW>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int64_t per = (total + 7) >> 3;  // tiles per XCD
  const int64_t xcd = blockIdx.x & 7, nb = gridDim.x >> 3;
  for (int64_t q = blockIdx.x >> 3; q < per; q += nb) {
    const int64_t x = xcd * per + q;
    if (x >= total) break;
    int e = 0;
    while (e + 1 < n && tab[e + 1].tile0 <= x) ++e;
    const GemmDesc& d = tab[e].d;
    const TileCoord tc = uniform(tile_of<T::BM, T::BNC>(x - tab[e].tile0, tab[e].tiles_m, tab[e].tiles_n));
    // opaque, so that what depends on the lane is worked out again for each
    // tile instead of kept in registers across the main loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    tile<PARTS, WM, WN, PW>(d, d.offM != nullptr, tc, lds, tid, wave / WN, wave % WN, lane);
  }
}

// ---------------------------------------------------------- few tiles
// Launches with few tiles do not fill the chip and are bound by latency: a
// stage of the kernel above costs a wave or two on a CU of their own 0.6 us
// and more.  Here a workgroup is one tile of BI x BJ MFMA blocks (32 x 16
// complex each) and its W waves share out K: wave w takes the stages w, w + W,
// ..., reads its fragments straight from global memory (lane (h, r) needs
// four consecutive complex values of row r), splits them in registers, and
// meets the others only to add the W sums up, in LDS, in order.  No staging,
// no barrier in the loop.  complex64 is scaled first and goes again, unscaled,
// where sums come out too large for that (256 x 256 x 256 with operands of 2^43
// 10.7 us).  It splits every value once per wave that reads it,
// so it loses where tiles are many.  256 x 256 x 256 26.6 -> 7.0 us, 1024 x
// 128 x 128 16.5 -> 5.5, 16 x 256 x 256 25.8 -> 6.7 (launches back to back, 4.6
// of it the launch).
template <int PARTS, int W, int BI, int BJ>
struct XDirect {
  static constexpr int BM = 32 * BI, BNC = 16 * BJ, NT = 64 * W;
  static constexpr int REGS = 16 * BI * BJ;                  // sums per lane
  static constexpr size_t kLds = size_t{W} * REGS * 64 * 4;  // one wave's sums after the other's
  static constexpr int N = REGS / W;                         // of them, added up and stored by one wave
  static_assert(W <= 8, "sums below 2^124 add up to a finite one");
  static_assert(N >= 1 && N <= 16 && 16 % N == 0, "a wave stores part of one block");

  f4 x[BI][2], y[BJ][2];  // this lane's four complex values of its rows of A and columns of B

  template <bool CHECK>
  __device__ __forceinline__ static void fetch(f4 (&v)[2], const float2* row, int64_t l, int64_t k) {
    if constexpr (CHECK) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 z = row[l + e < k ? l + e : k - 1];
        const bool in = l + e < k;
        v[e >> 1][2 * (e & 1)] = in ? z.x : 0.f;
        v[e >> 1][2 * (e & 1) + 1] = in ? z.y : 0.f;
      }
    } else {
      v[0] = *reinterpret_cast<const f4u*>(row + l);
      v[1] = *reinterpret_cast<const f4u*>(row + l + 2);
    }
  }

  template <bool SCALED>
  __device__ __forceinline__ static void split(const f4 (&v)[2], s8v (&part)[PARTS], uint32_t& tiny) {
    uint32_t w[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float a = v[e >> 1][2 * (e & 1)], b = v[e >> 1][2 * (e & 1) + 1];
      if constexpr (SCALED) {
        a *= pow2(kScale);
        b *= pow2(kScale);
      }
      w[0][e] = take_part(a, b);
      w[1][e] = take_part(a, b);
      if constexpr (PARTS == 3) w[2][e] = SCALED ? take_part(a, b) : last_part(a, b, tiny);
    }
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < PARTS; ++q) part[q] = __builtin_bit_cast(s8v, (u4){w[q][0], w[q][1], w[q][2], w[q][3]});
  }

  template <bool CHECK>
  __device__ __forceinline__ void load(const float2* const (&pa)[BI], const float2* const (&pb)[BJ], int64_t l,
                                       int64_t k) {
#pragma unroll
    for (int i = 0; i < BI; ++i) fetch<CHECK>(x[i], pa[i], l, k);
#pragma unroll
    for (int j = 0; j < BJ; ++j) fetch<CHECK>(y[j], pb[j], l, k);
  }

  __device__ __forceinline__ void run(const GemmDesc& d, const TileCoord& tc, char* lds, int wave, int lane) {
    int64_t oa, ob;
    batch_offsets(d, tc.b, oa, ob);
    const int64_t ld = row_stride(d), k = d.k;
    const int h = lane >> 5, r = lane & 31;
    const bool odd = r & 1;
    const float2 *pa[BI], *pb[BJ];
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const int64_t row = tc.row0 + 32 * i + r;
      pa[i] = d.A + uniform(oa) + (row < d.m ? row : d.m - 1) * ld;
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int64_t col = tc.col0 + 16 * j + (r >> 1);
      pb[j] = d.B + uniform(ob) + (col < d.n ? col : d.n - 1) * ld;
    }
    f16v acc[BI][BJ];
    auto load_stage = [&](int64_t st) {
      const int64_t l = st * XK + 4 * h;
      if ((st + 1) * XK <= k)
        load<false>(pa, pb, l, k);
      else
        load<true>(pa, pb, l, k);
    };
    const int64_t nk = (k + XK - 1) / XK;
    uint32_t tiny = 0xFFFFFFFFu;
    // the sum of the stages first, first + stride, ...
    auto add_up = [&](auto scaled, int64_t first, auto stride) {
      constexpr bool SCALED = decltype(scaled)::value;
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j) acc[i][j] = f16v{};
      if (first < nk) load_stage(first);
      for (int64_t st = first; st < nk; st += stride) {
        s8v fa[BI][PARTS], fb[BJ][PARTS];
#pragma unroll
        for (int i = 0; i < BI; ++i) split<SCALED>(x[i], fa[i], tiny);
#pragma unroll
        for (int j = 0; j < BJ; ++j) {
          f4 z[2];  // B': (br, -bi) for even real columns, (bi, br) for odd ones
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            z[e].x = odd ? y[j][e].y : y[j][e].x;
            z[e].y = odd ? y[j][e].x : -y[j][e].y;
            z[e].z = odd ? y[j][e].w : y[j][e].z;
            z[e].w = odd ? y[j][e].z : -y[j][e].w;
          }
          split<SCALED>(z, fb[j], tiny);
        }
        if (st + stride < nk) load_stage(st + stride);
        f16v c[BI][BJ] = {};
#pragma unroll
        for (int q = 0; q < (PARTS == 3 ? 6 : 3); ++q)
#pragma unroll
          for (int j = 0; j < BJ; ++j)
#pragma unroll
            for (int i = 0; i < BI; ++i)
              c[i][j] = PARTS == 3 ? mm(fa[i][kPartA[q]], fb[j][kPartB[q]], c[i][j])
                                   : mm(fa[i][kSplitA[q]], fb[j][kSplitB[q]], c[i][j]);
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
          for (int j = 0; j < BJ; ++j) acc[i][j] += c[i][j];
      }
    };
    // the wave's sums to LDS; true if one of them is 2^124 or above: not
    // finite, or so large that the waves' sums, which follow K's order only
    // inside a wave, might not add up to one that is
    auto put = [&]() {
      uint32_t top[4] = {0, 0, 0, 0};  // twice the bits of the largest (a NaN's are above any other)
      float* mine = reinterpret_cast<float*>(lds) + wave * REGS * 64 + lane;
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const uint32_t t = __float_as_uint(acc[i][j][v]) << 1;
            top[v & 3] = top[v & 3] < t ? t : top[v & 3];
            mine[(16 * (i * BJ + j) + v) * 64] = acc[i][j][v];
          }
#pragma unroll
      for (int q = 1; q < 4; ++q) top[0] = top[0] < top[q] ? top[q] : top[0];
      return top[0] >= (uint32_t{127 + 124} << 24);
    };
    float un = PARTS == 3 ? pow2(-2 * kScale) : 1.f;
    add_up(std::bool_constant<PARTS == 3>{}, wave, std::integral_constant<int, W>{});
    // (the vote is a barrier: every wave's sums are in LDS behind it)
    if (__syncthreads_or(put())) {
      if constexpr (PARTS == 3) {
        un = 1.f;
        add_up(std::false_type{}, wave, std::integral_constant<int, W>{});
        if (__syncthreads_or(put() || tiny < 0x00FFFFFFu)) {
          if (wave < BI * BJ) fp32_blocks<1, 1>(d, tc.b, tc.row0 + 32 * (wave / BJ), tc.col0 + 16 * (wave % BJ), lane);
          return;
        }
      } else {
        add_up(std::false_type{}, wave ? nk : 0, std::integral_constant<int, 1>{});  // all of K in order, in one wave
        (void)put();
        __syncthreads();
      }
    }
    const float* part = reinterpret_cast<const float*>(lds) + wave * N * 64 + lane;
    const int ij = wave * N / 16, v0 = wave * N & 15;
    const int64_t row0 = tc.row0 + 32 * (ij / BJ), col = tc.col0 + 16 * (ij % BJ) + (r >> 1);
    float* C = reinterpret_cast<float*>(d.C + tc.b * d.m * d.n) + (r & 1);
    const int64_t co = col < d.n ? (d.offM ? d.offN[col] : col) : -1;
    float sum[N];
    int64_t ro[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int v = v0 + u;
      const int64_t row = row0 + 8 * (v >> 2) + 4 * h + (v & 3);
      ro[u] = row < d.m ? (d.offM ? d.offM[row] : row * d.n) : -1;
      sum[u] = part[u * 64];
#pragma unroll
      for (int w = 1; w < W; ++w) sum[u] += part[u * 64 + w * REGS * 64];
    }
    if (co >= 0)
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (ro[u] >= 0) C[2 * (ro[u] + co)] = PARTS == 3 ? sum[u] * un : sum[u];
  }
};

template <int PARTS, int W, int BI, int BJ>
__global__ __launch_bounds__(64 * W) void cgemm_4m_direct(GemmDesc d, int64_t tiles_m, int64_t tiles_n,
                                                           int64_t total) {
  using T = XDirect<PARTS, W, BI, BJ>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  const TileCoord tc = uniform(map_tile_shared<T::BM, T::BNC>(tiles_m, tiles_n, total));
  T t;
  t.run(d, tc, lds, __builtin_amdgcn_readfirstlane(tid >> 6), tid & 63);
}

// one workgroup per tile of the launch's entries
template <int PARTS, int W, int BI, int BJ>
__global__ __launch_bounds__(64 * W) void cgemm_4m_direct_grouped(const GroupedEntry* __restrict__ tab, int n) {
  using T = XDirect<PARTS, W, BI, BJ>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  int e = 0;
  while (e + 1 < n && tab[e + 1].tile0 <= blockIdx.x) ++e;
  const TileCoord tc = uniform(tile_of<T::BM, T::BNC>(blockIdx.x - tab[e].tile0, tab[e].tiles_m, tab[e].tiles_n));
  T t;
  t.run(tab[e].d, tc, lds, __builtin_amdgcn_readfirstlane(tid >> 6), tid & 63);
}

// LDS above 64 KiB must be allowed per kernel, once per device.
template <class F>
hipError_t allow_lds(F* kernel, size_t lds, std::atomic<uint64_t>& done) {
  if (lds <= 65536) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = uint64_t{1} << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                          static_cast<int>(lds));
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_acq_rel);
  return e;
}

template <int PARTS, int WM, int WN, int PW, bool PERM>
hipError_t ready_one() {
  static std::atomic<uint64_t> done{0};
  return allow_lds(cgemm_4m<PARTS, WM, WN, PW, PERM>, XTile<PARTS, WM, WN, PW>::kLds, done);
}
template <int PARTS, int WM, int WN, int PW>
hipError_t ready_grouped() {
  static std::atomic<uint64_t> done{0};
  return allow_lds(cgemm_4m_grouped<PARTS, WM, WN, PW>, XTile<PARTS, WM, WN, PW>::kLds, done);
}

template <int PARTS, int WM, int WN, int PW, bool PERM>
hipError_t launch_one(const GemmDesc& d, hipStream_t s) {
  using T = XTile<PARTS, WM, WN, PW>;
  const int64_t tiles_m = (d.m + T::BM - 1) / T::BM;
  const int64_t tiles_n = (d.n + T::BNC - 1) / T::BNC;
  const int64_t total = tiles_m * tiles_n * d.h;
  // one workgroup per tile; the grid's work-items must fit 32 bits
  if (total * T::NT > 0xFFFFFFFFLL) return hipErrorInvalidValue;
  const hipError_t e = ready_one<PARTS, WM, WN, PW, PERM>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((cgemm_4m<PARTS, WM, WN, PW, PERM>), dim3(static_cast<unsigned>(total)), dim3(T::NT), T::kLds, s, d,
                     tiles_m, tiles_n, total);
  return hipGetLastError();
}
template <int PARTS, int WM, int WN, int PW>
hipError_t launch_shape(const GemmDesc& d, hipStream_t s) {
  return d.offM ? launch_one<PARTS, WM, WN, PW, true>(d, s) : launch_one<PARTS, WM, WN, PW, false>(d, s);
}

// Persistent grid: a multiple of 8 (one range of tiles per XCD), never more
// than the tiles; at most 512 workgroups (two per compute unit), or 2048
// waves for the shapes of fewer than four waves.
template <int PARTS, int WM, int WN, int PW>
hipError_t launch_grouped_shape(const GroupedEntry* tab, int n, int64_t total, hipStream_t s) {
  using T = XTile<PARTS, WM, WN, PW>;
  const hipError_t e = ready_grouped<PARTS, WM, WN, PW>();
  if (e != hipSuccess) return e;
  constexpr int64_t cap = WM * WN < 4 ? 2048 / (WM * WN) : 512;
  int64_t grid = (total + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  hipLaunchKernelGGL((cgemm_4m_grouped<PARTS, WM, WN, PW>), dim3(static_cast<unsigned>(grid)), dim3(T::NT), T::kLds, s, tab, n,
                     total);
  return hipGetLastError();
}

template <int PARTS, int W, int BI, int BJ>
hipError_t ready_direct() {
  static std::atomic<uint64_t> done{0}, done_grouped{0};
  const size_t lds = XDirect<PARTS, W, BI, BJ>::kLds;
  const hipError_t e = allow_lds(cgemm_4m_direct<PARTS, W, BI, BJ>, lds, done);
  return e != hipSuccess ? e : allow_lds(cgemm_4m_direct_grouped<PARTS, W, BI, BJ>, lds, done_grouped);
}
template <int PARTS, int W, int BI, int BJ>
hipError_t launch_direct(const GemmDesc& d, hipStream_t s) {
  using T = XDirect<PARTS, W, BI, BJ>;
  const int64_t tiles_m = (d.m + T::BM - 1) / T::BM, tiles_n = (d.n + T::BNC - 1) / T::BNC;
  const int64_t total = tiles_m * tiles_n * d.h;
  if (total * T::NT > 0xFFFFFFFFLL) return hipErrorInvalidValue;
  const hipError_t e = ready_direct<PARTS, W, BI, BJ>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((cgemm_4m_direct<PARTS, W, BI, BJ>), dim3(static_cast<unsigned>(total)), dim3(T::NT), T::kLds, s, d,
                     tiles_m, tiles_n, total);
  return hipGetLastError();
}

template <int PARTS, int W, int BI, int BJ>
hipError_t launch_direct_grouped(const GroupedEntry* tab, int n, int64_t total, hipStream_t s) {
  using T = XDirect<PARTS, W, BI, BJ>;
  if (total * T::NT > 0xFFFFFFFFLL) return hipErrorInvalidValue;
  const hipError_t e = ready_direct<PARTS, W, BI, BJ>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((cgemm_4m_direct_grouped<PARTS, W, BI, BJ>), dim3(static_cast<unsigned>(total)), dim3(T::NT), T::kLds, s,
                     tab, n);
  return hipGetLastError();
}

template <int PARTS, int WM, int WN, int PW>
void prepare_shape() {
  (void)ready_one<PARTS, WM, WN, PW, false>();
  (void)ready_one<PARTS, WM, WN, PW, true>();
  (void)ready_grouped<PARTS, WM, WN, PW>();
}


template <int PARTS>
void prepare_tiles() {
  prepare_shape<PARTS, 2, 2, 1>();
  prepare_shape<PARTS, 4, 1, 2>();
  if constexpr (PARTS == 3) prepare_shape<PARTS, 2, 2, 2>();
  prepare_shape<PARTS, 4, 2, 2>();
  prepare_shape<PARTS, 1, 2, 1>();
  prepare_shape<PARTS, 2, 1, 1>();
  prepare_shape<PARTS, 1, 1, 1>();
  prepare_shape<PARTS, 2, 4, 1>();
  (void)ready_direct<PARTS, 8, 1, 1>();
  (void)ready_direct<PARTS, 8, 1, 2>();
  (void)ready_direct<PARTS, 8, 2, 2>();
}

// complex64's 128 x 128 tile runs as four wide waves (each A fragment feeds
// four column blocks: fewer LDS reads), or as eight narrow ones where a launch
// has no more tiles than compute units: a CU then has two waves per SIMD
// from its one workgroup instead of one (6 x 1000 x 500 x 777, 192 tiles:
// 0.141 -> 0.125 ms; 8192 x 8192 x 4096, 4096 tiles: 10.3 -> 9.8 ms the
// other way); an element's sums do not depend on which of them ran.  Split
// precision's always runs as eight, which have registers for the cross sums.
bool wide_128(int64_t tiles) { return tiles > 256; }

template <int PARTS>
hipError_t launch_tiles(const GemmDesc& d, int variant, hipStream_t s) {
  switch (variant) {
    case 0: return launch_shape<PARTS, 2, 2, 1>(d, s);
    case 1: return launch_shape<PARTS, 4, 1, 2>(d, s);
    case 2:
      if constexpr (PARTS == 3)
        if (wide_128(d.h * ((d.m + 127) / 128) * ((d.n + 127) / 128))) return launch_shape<PARTS, 2, 2, 2>(d, s);
      return launch_shape<PARTS, 2, 4, 1>(d, s);
    case 3: return launch_shape<PARTS, 4, 2, 2>(d, s);
    case 4: return launch_shape<PARTS, 1, 2, 1>(d, s);
    case 5: return launch_shape<PARTS, 2, 1, 1>(d, s);
    case 6: return launch_shape<PARTS, 1, 1, 1>(d, s);
    case kDirect32x16: return launch_direct<PARTS, 8, 1, 1>(d, s);
    case kDirect32x32: return launch_direct<PARTS, 8, 1, 2>(d, s);
    case kDirect64x32: return launch_direct<PARTS, 8, 2, 2>(d, s);
    default: return hipErrorInvalidValue;
  }
}

template <int PARTS>
hipError_t launch_tiles_grouped(const GroupedEntry* tab, int n, int64_t total, int variant, hipStream_t s) {
  switch (variant) {
    case 0: return launch_grouped_shape<PARTS, 2, 2, 1>(tab, n, total, s);
    case 1: return launch_grouped_shape<PARTS, 4, 1, 2>(tab, n, total, s);
    case 2:
      if constexpr (PARTS == 3)
        if (wide_128(total)) return launch_grouped_shape<PARTS, 2, 2, 2>(tab, n, total, s);
      return launch_grouped_shape<PARTS, 2, 4, 1>(tab, n, total, s);
    case 3: return launch_grouped_shape<PARTS, 4, 2, 2>(tab, n, total, s);
    case 4: return launch_grouped_shape<PARTS, 1, 2, 1>(tab, n, total, s);
    case 5: return launch_grouped_shape<PARTS, 2, 1, 1>(tab, n, total, s);
    case 6: return launch_grouped_shape<PARTS, 1, 1, 1>(tab, n, total, s);
    case kDirect32x16: return launch_direct_grouped<PARTS, 8, 1, 1>(tab, n, total, s);
    case kDirect32x32: return launch_direct_grouped<PARTS, 8, 1, 2>(tab, n, total, s);
    case kDirect64x32: return launch_direct_grouped<PARTS, 8, 2, 2>(tab, n, total, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

void prepare_gemm_4m() {
  prepare_tiles<3>();
  prepare_tiles<2>();
}

hipError_t launch_gemm_4m(const GemmDesc& d, int variant, Prec prec, hipStream_t s) {
  return prec == Prec::BF16X3 ? launch_tiles<2>(d, variant, s) : launch_tiles<3>(d, variant, s);
}

hipError_t launch_gemm_4m_grouped(const GroupedEntry* tab, int n, int64_t total, int variant, Prec prec,
                                  hipStream_t s) {
  return prec == Prec::BF16X3 ? launch_tiles_grouped<2>(tab, n, total, variant, s)
                              : launch_tiles_grouped<3>(tab, n, total, variant, s);
}

}  // namespace tnc
