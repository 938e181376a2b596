// Batched complex GEMM on MFMA for gfx950:  C[b,i,j] = sum_l A[b,i,l] B[b,j,l].
//
// Every contraction step of the path is one such GEMM once the operands are
// in [retained || reduced] order (paper Sec. II-B: A_MK x B_KN -> C_MN;
// Sec. IV-A: the canonical operand layout maps directly to a GEMM).  Both
// operands are K-contiguous, so the product is A * B^T per batch entry.
//
// Here are split precision's 3M form, its pre-split planes (both forms) and
// the choice between kernels; the 4M kernels have a file of their own
// (kern_cgemm_4m.hip).
//
// 4M form.  A complex row of A, read as 2k floats (ar0, ai0, ar1, ai1, ...),
// times the real 2k-vector
//   (br0, -bi0, br1, -bi1, ...)  gives Re C,
//   (bi0,  br0, bi1,  br1, ...)  gives Im C,
// so C, viewed as an m x 2n float matrix, is a single real GEMM of
// m x 2n x 2k.  The MFMA output columns then alternate re/im: exactly the
// interleaved complex64 layout, with no de-interleaving anywhere.  8 real
// FLOPs per complex MAC (the paper's counting convention, Sec. II-B).
//
// 3M form: T1 = Ar Br, T2 = Ai Bi, T3 = (Ar+Ai)(Br+Bi), Re = T1 - T2,
// Im = T3 - T1 - T2: three real GEMMs, 6 executed FLOPs per complex MAC.
//
// BF16x3: each float32 plane is split into bf16 hi/lo (round to nearest
// even) while it is staged into LDS; every real product becomes
// a_hi b_hi + (a_hi b_lo + a_lo b_hi) on bf16 MFMA with FP32 accumulation.
// 12 bf16 products per complex product in the 4M form, 9 in the 3M form (the
// sum planes Ar+Ai, Br+Bi formed in float32, then split).  Large single
// GEMMs split their operands once into bf16 planes in global memory instead
// and stage them straight into LDS (the pre-split section below); in the 3M
// form as three real GEMMs plus a combining pass.
//
// Tiling of the 3M form.  A wave64 owns a 64 x 32 complex tile of C (2x1
// complex blocks of 32 x 32); a workgroup is WM x WN waves.  K advances 16
// complex per stage through double-buffered LDS.  Interior tiles run a copy
// of the main loop without bounds checks.  Tiles sweep N in groups of 8
// M-tiles, and workgroups are remapped (the hardware deals them round-robin
// over the 8 XCDs, each with its own L2) so that the tiles one XCD runs at
// once form 8 x 4 blocks: 12 operand panels per 32 tiles through its L2.
// Where the tile counts allow, the eight XCDs' blocks share their 8 M-tiles,
// so the memory-side cache serves each A panel to all of them from one HBM
// read (pre-split kernel on pair30's shape: 316.7 -> 314.5 ms).
#include <atomic>
#include <cstring>

#include "bf16_split.hpp"
#include "gemm_common.hpp"
#include "gemm_tile.hpp"

namespace tnc {

namespace {

constexpr int BKC = 16;  // complex k per LDS stage

template <int WM, int WN>
struct Shape {
  static constexpr int BM = 64 * WM;   // rows of C per workgroup
  static constexpr int BNC = 32 * WN;  // complex columns of C per workgroup
  static constexpr int NT = 64 * WM * WN;
};

// Global -> register staging of one K stage (VW complex per load).
template <int WM, int WN, int VW>
struct Stage {
  using S = Shape<WM, WN>;
  static constexpr int PER_ROW = BKC / VW;
  static constexpr int A_LOADS = S::BM * PER_ROW / S::NT;
  static constexpr int B_LOADS = S::BNC * PER_ROW / S::NT;
  static_assert(A_LOADS >= 1 && A_LOADS * S::NT == S::BM * PER_ROW, "A staging must tile evenly");
  static_assert(B_LOADS >= 1 && B_LOADS * S::NT == S::BNC * PER_ROW, "B staging must tile evenly");
  f4 a[A_LOADS];
  f4 b[B_LOADS];

  template <bool CHECK>
  __device__ __forceinline__ static f4 fetch(const float2* __restrict__ X, int64_t gr, int64_t gk, int64_t rows,
                                             int64_t k, int64_t ld) {
    f4 v = {0.f, 0.f, 0.f, 0.f};
    if (!CHECK || (gr < rows && gk < k)) {
      const float2* p = X + gr * ld + gk;
      if constexpr (VW == 2) {
        v = *reinterpret_cast<const f4*>(p);
      } else {
        const float2 x = *p;
        v.x = x.x;
        v.y = x.y;
      }
    }
    return v;
  }

  template <bool CHECK>
  __device__ __forceinline__ void load(const float2* __restrict__ A, const float2* __restrict__ B, int64_t m,
                                       int64_t n, int64_t k, int64_t ld, int64_t row0, int64_t col0, int64_t kk,
                                       int tid) {
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
      const int idx = tid + S::NT * i;
      a[i] = fetch<CHECK>(A, row0 + (idx / PER_ROW), kk + (idx % PER_ROW) * VW, m, k, ld);
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) {
      const int idx = tid + S::NT * i;
      b[i] = fetch<CHECK>(B, col0 + (idx / PER_ROW), kk + (idx % PER_ROW) * VW, n, k, ld);
    }
  }
};

// ------------------------------------------------------------------ split BF16x3, 3M form
// The 3M form's three real products T1 = Ar Br, T2 = Ai Bi, T3 = (Ar+Ai)
// (Br+Bi), each as a_hi b_lo + a_lo b_hi + a_hi b_hi on bf16 MFMA
// 32x32x16 into one FP32 accumulator per product: 9 bf16 products per
// complex product instead of the 4M form's 12.  The sum planes are formed
// in float32 at staging, then split like the others.  A stage (16 complex
// k) holds six unpadded bf16 planes per operand (r, i, s, each hi and lo),
// a row of 16 k in 32 bytes; the row's two 16-byte halves swap places
// every 8 rows (slot = half ^ ((row >> 3) & 1)), so the fragment reads of
// 16 lanes (16 rows, one half) and the 4-byte staging stores of a wave (8
// rows x 8 pairs) hit distinct banks.  The wave tile and the store are the
// complex64 3M form's.
template <int WM, int WN, int VW>
struct Ops3MBF16 {
  using S = Shape<WM, WN>;
  static constexpr int ROWB = 32;  // bytes per plane row
  static constexpr int PLANE_A = S::BM * ROWB, PLANE_B = S::BNC * ROWB;
  static constexpr int STAGE = 6 * (PLANE_A + PLANE_B);
  static constexpr size_t kLds = 2 * STAGE;
  f16v t1[2], t2[2], t3[2];

  // byte offset of k (0..15) in plane row `row`
  __device__ __forceinline__ static int at(int row, int k) {
    return row * ROWB + ((((k >> 3) ^ ((row >> 3) & 1)) << 4) | ((k & 7) << 1));
  }

  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) t1[i][v] = t2[i][v] = t3[i][v] = 0.f;
  }

  // planes p = 0..5 (r hi, r lo, i hi, i lo, s hi, s lo) at base + p * plane
  template <class St>
  __device__ __forceinline__ static void put(char* base, int plane, int row, int idx, const f4& v) {
    const int off = at(row, (idx % St::PER_ROW) * VW);
    if constexpr (VW == 2) {  // complex k, k + 1: (re k, im k, re k+1, im k+1)
      uint32_t rh, rl, ih, il, sh, sl;
      bf16_split2(v.x, v.z, rh, rl);
      bf16_split2(v.y, v.w, ih, il);
      bf16_split2(v.x + v.y, v.z + v.w, sh, sl);
      *reinterpret_cast<uint32_t*>(base + off) = rh;
      *reinterpret_cast<uint32_t*>(base + plane + off) = rl;
      *reinterpret_cast<uint32_t*>(base + 2 * plane + off) = ih;
      *reinterpret_cast<uint32_t*>(base + 3 * plane + off) = il;
      *reinterpret_cast<uint32_t*>(base + 4 * plane + off) = sh;
      *reinterpret_cast<uint32_t*>(base + 5 * plane + off) = sl;
    } else {  // one complex value: (re, im) split as a pair, the sum alone
      uint32_t h, l, sh, sl;
      bf16_split2(v.x, v.y, h, l);
      bf16_split2(v.x + v.y, 0.f, sh, sl);
      *reinterpret_cast<uint16_t*>(base + off) = static_cast<uint16_t>(h);
      *reinterpret_cast<uint16_t*>(base + plane + off) = static_cast<uint16_t>(l);
      *reinterpret_cast<uint16_t*>(base + 2 * plane + off) = static_cast<uint16_t>(h >> 16);
      *reinterpret_cast<uint16_t*>(base + 3 * plane + off) = static_cast<uint16_t>(l >> 16);
      *reinterpret_cast<uint16_t*>(base + 4 * plane + off) = static_cast<uint16_t>(sh);
      *reinterpret_cast<uint16_t*>(base + 5 * plane + off) = static_cast<uint16_t>(sl);
    }
  }

  template <class St>
  __device__ __forceinline__ void stage(const St& st, char* lds, int buf, int tid) const {
    char* As = lds + buf * STAGE;
    char* Bs = As + 6 * PLANE_A;
#pragma unroll
    for (int i = 0; i < St::A_LOADS; ++i) put<St>(As, PLANE_A, (tid + S::NT * i) / St::PER_ROW, tid + S::NT * i, st.a[i]);
#pragma unroll
    for (int i = 0; i < St::B_LOADS; ++i) put<St>(Bs, PLANE_B, (tid + S::NT * i) / St::PER_ROW, tid + S::NT * i, st.b[i]);
  }

  __device__ __forceinline__ static void mm(f16v& t, const s8v& ah, const s8v& al, const s8v& bh, const s8v& bl) {
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, ah), __builtin_bit_cast(bf8, bl), t, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, al), __builtin_bit_cast(bf8, bh), t, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, ah), __builtin_bit_cast(bf8, bh), t, 0, 0, 0);
  }

  // product p (planes 2p, 2p + 1) of the stage into t
  __device__ __forceinline__ static void product(f16v (&t)[2], const char* ah, const char* bh, int oa0, int oa1,
                                                 int ob) {
    const s8v a0h = *reinterpret_cast<const s8v*>(ah + oa0);
    const s8v a0l = *reinterpret_cast<const s8v*>(ah + PLANE_A + oa0);
    const s8v a1h = *reinterpret_cast<const s8v*>(ah + oa1);
    const s8v a1l = *reinterpret_cast<const s8v*>(ah + PLANE_A + oa1);
    const s8v b_h = *reinterpret_cast<const s8v*>(bh + ob);
    const s8v b_l = *reinterpret_cast<const s8v*>(bh + PLANE_B + ob);
    mm(t[0], a0h, a0l, b_h, b_l);
    mm(t[1], a1h, a1l, b_h, b_l);
  }

  // lane (h, r) supplies k = 8h .. 8h + 7 of row r (A) or column r (B);
  // one product at a time keeps a third of the fragments live
  __device__ __forceinline__ void compute(const char* lds, int buf, int wm, int wn, int lane) {
    const char* As = lds + buf * STAGE;
    const char* Bs = As + 6 * PLANE_A;
    const int h = lane >> 5, l32 = lane & 31;
    const int oa0 = at(wm * 64 + l32, 8 * h), oa1 = at(wm * 64 + 32 + l32, 8 * h);
    const int ob = at(wn * 32 + l32, 8 * h);
    product(t1, As, Bs, oa0, oa1, ob);
    product(t2, As + 2 * PLANE_A, Bs + 2 * PLANE_B, oa0, oa1, ob);
    product(t3, As + 4 * PLANE_A, Bs + 4 * PLANE_B, oa0, oa1, ob);
  }

  __device__ __forceinline__ void store(const GemmDesc& d, bool perm, const TileCoord& tc, int wm, int wn,
                                        int lane) const {
    store_3m(d, perm, tc, wm, wn, lane, t1, t2, t3);
  }
};

// ------------------------------------------------------------------ driver
template <int WM, int WN, int VW, bool CHECK>
__device__ __forceinline__ void main_loop(const GemmDesc& d, const float2* A, const float2* B, const TileCoord& tc,
                                          char* lds, Ops3MBF16<WM, WN, VW>& ops, int tid, int wm, int wn, int lane) {
  const int64_t nk = (d.k + BKC - 1) / BKC;
  const int64_t ld = row_stride(d);
  Stage<WM, WN, VW> st;
  st.template load<CHECK>(A, B, d.m, d.n, d.k, ld, tc.row0, tc.col0, 0, tid);
  ops.stage(st, lds, 0, tid);
  __syncthreads();
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) st.template load<CHECK>(A, B, d.m, d.n, d.k, ld, tc.row0, tc.col0, (kt + 1) * BKC, tid);
    ops.compute(lds, buf, wm, wn, lane);
    if (kt + 1 < nk) ops.stage(st, lds, buf ^ 1, tid);
    __syncthreads();
  }
}

template <int WM, int WN, int VW, bool PERM>
__global__ __launch_bounds__(64 * WM * WN, WM * WN <= 4 ? 2 : 1) void cgemm_mfma(GemmDesc d, int64_t tiles_m,
                                                                                 int64_t tiles_n, int64_t total) {
  using S = Shape<WM, WN>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const TileCoord tc = map_tile_shared<S::BM, S::BNC>(tiles_m, tiles_n, total);
  int64_t oa, ob;
  batch_offsets(d, tc.b, oa, ob);
  const float2* __restrict__ A = d.A + oa;
  const float2* __restrict__ B = d.B + ob;
  Ops3MBF16<WM, WN, VW> ops;
  ops.init();
  const bool interior = tc.row0 + S::BM <= d.m && tc.col0 + S::BNC <= d.n && d.k % BKC == 0;
  if (interior)
    main_loop<WM, WN, VW, false>(d, A, B, tc, lds, ops, tid, wm, wn, lane);
  else
    main_loop<WM, WN, VW, true>(d, A, B, tc, lds, ops, tid, wm, wn, lane);
  ops.store(d, PERM, tc, wm, wn, lane);
}

// Persistent grouped form: workgroups loop over the tiles of every entry of
// the table.  Tiles are dealt to the 8 XCDs in contiguous ranges (tiles of
// one entry stay on few XCDs, whose L2 they share) and each workgroup of an
// XCD takes every nb-th tile of its range.  The tile's work is the
// single-GEMM kernel's, line for line.  The tile loop keeps more values
// live than one tile does, so most instances are built for one workgroup
// per CU, which lets the compiler keep accumulators in AGPRs instead of
// spilling (the persistent grid runs a fixed number of workgroups anyway).
template <int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN, WM * WN == 4 ? 2 : 1) void cgemm_mfma_grouped(
    const GroupedEntry* __restrict__ tab, int n, int64_t total) {
  using S = Shape<WM, WN>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int64_t per = (total + 7) >> 3;  // tiles per XCD
  const int64_t xcd = blockIdx.x & 7, nb = gridDim.x >> 3;
  for (int64_t q = blockIdx.x >> 3; q < per; q += nb) {
    const int64_t t = xcd * per + q;
    if (t >= total) break;
    int e = 0;
    while (e + 1 < n && tab[e + 1].tile0 <= t) ++e;
    const GemmDesc& d = tab[e].d;
    const TileCoord tc = tile_of<S::BM, S::BNC>(t - tab[e].tile0, tab[e].tiles_m, tab[e].tiles_n);
    int64_t oa, ob;
    batch_offsets(d, tc.b, oa, ob);
    const float2* __restrict__ A = d.A + oa;
    const float2* __restrict__ B = d.B + ob;
    Ops3MBF16<WM, WN, 2> ops;
    ops.init();
    const bool interior = tc.row0 + S::BM <= d.m && tc.col0 + S::BNC <= d.n && d.k % BKC == 0;
    if (interior)
      main_loop<WM, WN, 2, false>(d, A, B, tc, lds, ops, tid, wm, wn, lane);
    else
      main_loop<WM, WN, 2, true>(d, A, B, tc, lds, ops, tid, wm, wn, lane);
    ops.store(d, d.offM != nullptr, tc, wm, wn, lane);
  }
}

// ------------------------------------------ split-bf16x3 on pre-split planes
// Large split-precision steps split each operand once, into bf16 planes in
// global memory, instead of in the staging of every workgroup that reads
// it.  A row of A (or of the 4M real operand B': row 2c = (br, -bi, ...),
// row 2c + 1 = (bi, br, ...)) is stored in blocks of 16 complex k, 128
// bytes = [32 bf16 hi | 32 bf16 lo] of its 32 floats; rows are padded to
// the tile and k to 16 with zeros, so staging needs no bounds tests and
// moves blocks straight from global memory into LDS (16 bytes per lane,
// global_load_lds_dwordx4: no registers and no VALU on the way).  The split
// is the staging kernels' (round to nearest even, lo = rne(x - hi)) and the
// tile's products and accumulation order are those of the 4M kernels' 256 x
// 128 tile, so the result is bitwise that tile's.
//
// LDS: two stages of four unpadded planes (256 rows x 64 bytes each); the
// four 16-byte slots of a row are permuted by row (slot = chunk ^ ((row >> 2)
// & 3)), so that the fragment reads of 16 lanes (16 rows, one chunk) hit 16
// distinct 4-bank groups.  Each stage has one barrier, in its middle: the
// waves issue the first half's MFMAs (whose fragments they read during the
// previous half) and read the second half's fragments, then meet; after the
// barrier the stage's loads two stages ahead go out into the buffer just
// released, the next stage's first fragments are read, and the second
// half's MFMAs run, their issue interleaved with those reads.
constexpr int PS_PLANE = 256 * 64;        // bytes of one LDS plane
constexpr int PS_STAGE = 4 * PS_PLANE;    // A hi, A lo, B' hi, B' lo
constexpr size_t PS_LDS = 2 * PS_STAGE;   // 128 KiB

// uint32 (bf16 pair) index of the hi half of complex element (row, kc) in
// planes of kp complex columns; the lo half is 16 further
__device__ __forceinline__ int64_t ps_index(int64_t row, int64_t kc, int64_t kp) {
  return row * 2 * kp + 32 * (kc >> 4) + (kc & 15);
}

__device__ __forceinline__ void ps_split(float x, float y, uint32_t& hi, uint32_t& lo) { bf16_split2(x, y, hi, lo); }

// One thread per complex element of the padded planes; 16 consecutive
// threads cover one 128-byte block (their loads 128 contiguous bytes of
// the row, their stores the block).
__global__ __launch_bounds__(256) void split_planes_a(const float2* __restrict__ X, int64_t rows, int64_t k,
                                                     int64_t ld, uint32_t nkb, uint32_t blocks, int64_t kp,
                                                     uint32_t* __restrict__ out) {
  for (uint32_t t = blockIdx.x * 256u + threadIdx.x; t < blocks * 16u; t += gridDim.x * 256u) {
    const uint32_t b = t >> 4, e = t & 15;
    const int64_t row = b / nkb, kc = int64_t{b % nkb} * 16 + e;
    uint64_t v = 0;
    if (row < rows && kc < k) v = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(X + row * ld + kc));
    uint32_t hi, lo;
    ps_split(__uint_as_float(static_cast<uint32_t>(v)), __uint_as_float(static_cast<uint32_t>(v >> 32)), hi, lo);
    const int64_t p = ps_index(row, kc, kp);
    __builtin_nontemporal_store(hi, out + p);
    __builtin_nontemporal_store(lo, out + p + 16);
  }
}

// B -> the planes of B' (two real rows per complex row of B; negating a
// bf16 flips its sign bit, swapping re/im rotates the packed pair).
__global__ __launch_bounds__(256) void split_planes_b(const float2* __restrict__ X, int64_t rows, int64_t k,
                                                     int64_t ld, uint32_t nkb, uint32_t blocks, int64_t kp,
                                                     uint32_t* __restrict__ out) {
  for (uint32_t t = blockIdx.x * 256u + threadIdx.x; t < blocks * 16u; t += gridDim.x * 256u) {
    const uint32_t b = t >> 4, e = t & 15;
    const int64_t row = b / nkb, kc = int64_t{b % nkb} * 16 + e;
    uint64_t v = 0;
    if (row < rows && kc < k) v = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(X + row * ld + kc));
    uint32_t hi, lo;
    ps_split(__uint_as_float(static_cast<uint32_t>(v)), __uint_as_float(static_cast<uint32_t>(v >> 32)), hi, lo);
    const int64_t p0 = ps_index(2 * row, kc, kp), p1 = p0 + 2 * kp;
    __builtin_nontemporal_store(hi ^ 0x80000000u, out + p0);
    __builtin_nontemporal_store(lo ^ 0x80000000u, out + p0 + 16);
    __builtin_nontemporal_store((hi >> 16) | (hi << 16), out + p1);
    __builtin_nontemporal_store((lo >> 16) | (lo << 16), out + p1 + 16);
  }
}

// 3M form: the real parts X_r, X_i and X_s = X_r + X_i (float32 sums) of
// a complex operand as three real matrices of `rows` x k, each in the
// planes layout of a real GEMM (blocks of 32 real k, [32 bf16 hi | 32 bf16
// lo], kp real k pairs per row; padding rows and k zero).  One thread per
// pair of real k (two complex elements) of a padded row; P points at the
// r planes, the i and s planes follow at `plane` uint32 apart.
__global__ __launch_bounds__(256) void split_planes_3m(const float2* __restrict__ X, int64_t rows, int64_t k,
                                                      int64_t ld, uint32_t kp, uint32_t pairs, int64_t plane,
                                                      uint32_t* __restrict__ P) {
  for (uint32_t t = blockIdx.x * 256u + threadIdx.x; t < pairs; t += gridDim.x * 256u) {
    const int64_t row = t / kp, q = t - row * kp;  // real k 2q, 2q + 1
    float2 x0 = make_float2(0.f, 0.f), x1 = x0;
    if (row < rows) {
      const float2* src = X + row * ld + 2 * q;
      if (2 * q < k) x0 = src[0];
      if (2 * q + 1 < k) x1 = src[1];
    }
    uint32_t rh, rl, ih, il, sh, sl;
    ps_split(x0.x, x1.x, rh, rl);
    ps_split(x0.y, x1.y, ih, il);
    ps_split(x0.x + x0.y, x1.x + x1.y, sh, sl);
    const int64_t o = ps_index(row, q, kp);
    __builtin_nontemporal_store(rh, P + o);
    __builtin_nontemporal_store(rl, P + o + 16);
    __builtin_nontemporal_store(ih, P + plane + o);
    __builtin_nontemporal_store(il, P + plane + o + 16);
    __builtin_nontemporal_store(sh, P + 2 * plane + o);
    __builtin_nontemporal_store(sl, P + 2 * plane + o + 16);
  }
}

// C from the three real products (rows of `ldt` floats, T2 and T3 `tplane`
// floats after T1): re = T1 - T2, im = T3 - T1 - T2 in float32, the same
// expressions as the 3M store; row-major or through the offset tables.
__global__ __launch_bounds__(256) void combine_3m(const float* __restrict__ T, int64_t tplane, int64_t ldt,
                                                 GemmDesc d) {
  const int64_t total = d.m * d.n;
  const double inv_n = 1.0 / static_cast<double>(d.n);
  for (int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; e < total;
       e += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t row = plane_row(e, d.n, inv_n), col = e - row * d.n;
    const int64_t o = row * ldt + col;
    const float t1 = T[o], t2 = T[tplane + o], t3 = T[2 * tplane + o];
    float2 v;
    v.x = t1 - t2;
    v.y = t3 - t1 - t2;
    const int64_t c = d.offM ? d.offM[row] + d.offN[col] : e;
    d.C[c] = v;
  }
}

struct PsFrag {
  s8v ah[2], al[2], bh[4], bl[4];
};

// Fragments of sub-step s (16 real k) for wave (wm, wn): lane (h, r) takes 8
// consecutive k of row r (A) or real column r (B').
__device__ __forceinline__ void ps_read(const char* stage, int wm, int wn, int h, int l32, int s, PsFrag& f) {
  const int ch = 2 * s + h;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = wm * 64 + i * 32 + l32;
    const int off = row * 64 + 16 * (ch ^ ((row >> 2) & 3));
    f.ah[i] = *reinterpret_cast<const s8v*>(stage + off);
    f.al[i] = *reinterpret_cast<const s8v*>(stage + PS_PLANE + off);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 128 * wn + 32 * j + l32;
    const int off = row * 64 + 16 * (ch ^ ((row >> 2) & 3));
    f.bh[j] = *reinterpret_cast<const s8v*>(stage + 2 * PS_PLANE + off);
    f.bl[j] = *reinterpret_cast<const s8v*>(stage + 3 * PS_PLANE + off);
  }
}

// Per block a_hi b_lo, a_lo b_hi, a_hi b_hi, into one accumulator.  The two
// blocks of a column take turns so that five of six neighbours share an
// operand, which the chip's power budget feels (block by block two of six: 16384
// x 8192 x 8192 20.45 -> 20.29 ms, in the 3M form 15.78 -> 15.65).
__device__ __forceinline__ void ps_mfma(f16v (&acc)[2][4], const PsFrag& f) {
  auto mm = [&](int i, int j, const s8v& a, const s8v& b) {
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b),
                                                        acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = j & 1, q = p ^ 1;
    mm(p, j, f.ah[p], f.bl[j]);
    mm(q, j, f.ah[q], f.bl[j]);
    mm(q, j, f.al[q], f.bh[j]);
    mm(p, j, f.al[p], f.bh[j]);
    mm(p, j, f.ah[p], f.bh[j]);
    mm(q, j, f.ah[q], f.bh[j]);
  }
}

// Stage kk's blocks of the tile into LDS buffer `buf`: 64 wave-loads of 1
// KiB (16 rows x 4 slots of one plane), 8 per wave.  `wave` is uniform.
__device__ __forceinline__ void ps_issue(char* lds, int buf, int64_t kk, const uint32_t* gA, const uint32_t* gB,
                                         int64_t kp, int wave, int lane) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int bid = wave * 8 + q;
    const int plane = bid >> 4, rb = bid & 15;
    const int row = rb * 16 + (lane >> 2), slot = lane & 3;
    const int c = slot ^ ((row >> 2) & 3);
    const uint32_t* g = (plane < 2 ? gA : gB) + row * 2 * kp + 2 * kk + 16 * (plane & 1) + 4 * c;
    char* dst = lds + buf * PS_STAGE + plane * PS_PLANE + rb * 1024;
    __builtin_amdgcn_global_load_lds(static_cast<const void*>(g), (__attribute__((address_space(3))) void*)dst, 16, 0,
                                     0);
  }
}

// One K stage (16 complex k).  ISSUE: load stage kt + 2 after the barrier;
// READ: read the next stage's first fragments into f0.
template <bool ISSUE, bool READ>
__device__ __forceinline__ void ps_stage(f16v (&acc)[2][4], PsFrag& f0, PsFrag& f1, char* lds, int64_t kt,
                                         const uint32_t* gA, const uint32_t* gB, int64_t kp, int wave, int lane,
                                         int wm, int wn, int h, int l32) {
  const int buf = kt & 1;
  ps_read(lds + buf * PS_STAGE, wm, wn, h, l32, 1, f1);
  ps_mfma(acc, f0);
#pragma unroll
  for (int r = 0; r < 12; ++r) {  // one fragment read per two MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
  }
  __builtin_amdgcn_s_waitcnt(0);  // this wave's reads done, stage kt + 1 landed
  __syncthreads();
  if constexpr (ISSUE) ps_issue(lds, buf, (kt + 2) * BKC, gA, gB, kp, wave, lane);
  if constexpr (READ) ps_read(lds + (buf ^ 1) * PS_STAGE, wm, wn, h, l32, 0, f0);
  ps_mfma(acc, f1);
  if constexpr (ISSUE) __builtin_amdgcn_sched_group_barrier(0x020, 8, 0);
  if constexpr (READ) {
#pragma unroll
    for (int r = 0; r < 12; ++r) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
  }
}

// gfx9 s_waitcnt immediate: vmcnt <= 8, expcnt and lgkmcnt not waited for
constexpr int kWaitVm8 = 0x0F78;

template <bool PERM>
__global__ __launch_bounds__(512, 1) void cgemm_bf16x3_presplit(GemmDesc d, const uint32_t* __restrict__ Ap,
                                                                const uint32_t* __restrict__ Bp, int64_t kp,
                                                                int64_t tiles_m, int64_t tiles_n, int64_t total) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int h = lane >> 5, l32 = lane & 31;
  const TileCoord tc = map_tile_shared<kPresplitBM, kPresplitBNC>(tiles_m, tiles_n, total);
  const uint32_t* gA = Ap + tc.row0 * 2 * kp;
  const uint32_t* gB = Bp + 2 * tc.col0 * 2 * kp;
  const int64_t nk = kp / BKC;
  f16v acc[2][4] = {};
  PsFrag f0, f1;
  ps_issue(lds, 0, 0, gA, gB, kp, wave, lane);
  if (nk > 1) {
    ps_issue(lds, 1, BKC, gA, gB, kp, wave, lane);
    __builtin_amdgcn_s_waitcnt(kWaitVm8);  // stage 0 landed (loads complete in order)
  } else {
    __builtin_amdgcn_s_waitcnt(0);
  }
  __syncthreads();
  ps_read(lds, wm, wn, h, l32, 0, f0);
  if (nk > 1) {
    for (int64_t kt = 0; kt + 2 < nk; ++kt)
      ps_stage<true, true>(acc, f0, f1, lds, kt, gA, gB, kp, wave, lane, wm, wn, h, l32);
    ps_stage<false, true>(acc, f0, f1, lds, nk - 2, gA, gB, kp, wave, lane, wm, wn, h, l32);
  }
  ps_stage<false, false>(acc, f0, f1, lds, nk - 1, gA, gB, kp, wave, lane, wm, wn, h, l32);
  store_4m<2>(d, PERM, tc, wm, wn, lane, [&](int i, int j, int v) { return acc[i][j][v]; });
}

// LDS above 64 KiB for the pre-split kernel, once per device.
hipError_t ensure_lds_presplit() {
  static std::atomic<uint64_t> attr_set{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = uint64_t{1} << (dev & 63);
  if (attr_set.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(cgemm_bf16x3_presplit<false>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(PS_LDS));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(cgemm_bf16x3_presplit<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(PS_LDS));
  if (e == hipSuccess) attr_set.fetch_or(bit, std::memory_order_acq_rel);
  return e;
}

// LDS above 64 KiB must be allowed per kernel, once per device (done for
// every instance when a context is created, so that no first launch inside
// a graph capture has to do it).
template <int WM, int WN, int VW, bool PERM>
hipError_t ensure_lds(size_t lds) {
  static std::atomic<uint64_t> attr_set{0};
  if (lds <= 65536) return hipSuccess;
  int dev = 0;
  const hipError_t ge = hipGetDevice(&dev);
  if (ge != hipSuccess) return ge;
  const uint64_t bit = uint64_t{1} << (dev & 63);
  if (attr_set.load(std::memory_order_acquire) & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(cgemm_mfma<WM, WN, VW, PERM>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e == hipSuccess) attr_set.fetch_or(bit, std::memory_order_acq_rel);
  return e;
}

template <int WM, int WN, int VW, bool PERM>
hipError_t launch_one(const GemmDesc& d, size_t lds, hipStream_t s) {
  using S = Shape<WM, WN>;
  const int64_t tiles_m = (d.m + S::BM - 1) / S::BM;
  const int64_t tiles_n = (d.n + S::BNC - 1) / S::BNC;
  const int64_t total = tiles_m * tiles_n * d.h;
  // one workgroup per tile; the grid's work-items must fit 32 bits
  if (total * S::NT > 0xFFFFFFFFLL) return hipErrorInvalidValue;
  const hipError_t e = ensure_lds<WM, WN, VW, PERM>(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((cgemm_mfma<WM, WN, VW, PERM>), dim3(static_cast<unsigned>(total)), dim3(S::NT), lds, s, d,
                     tiles_m, tiles_n, total);
  return hipGetLastError();
}

template <int WM, int WN>
hipError_t ensure_lds_grouped(size_t lds) {
  static std::atomic<uint64_t> attr_set{0};
  if (lds <= 65536) return hipSuccess;
  int dev = 0;
  const hipError_t ge = hipGetDevice(&dev);
  if (ge != hipSuccess) return ge;
  const uint64_t bit = uint64_t{1} << (dev & 63);
  if (attr_set.load(std::memory_order_acquire) & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(cgemm_mfma_grouped<WM, WN>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e == hipSuccess) attr_set.fetch_or(bit, std::memory_order_acq_rel);
  return e;
}

template <int WM, int WN>
void prepare_shape() {
  const size_t lds = Ops3MBF16<WM, WN, 2>::kLds;
  (void)ensure_lds<WM, WN, 2, false>(lds);
  (void)ensure_lds<WM, WN, 2, true>(lds);
  (void)ensure_lds_grouped<WM, WN>(lds);
}

// Persistent grid: a multiple of 8 (one range of tiles per XCD), never more
// than the tiles; at most 512 workgroups (two per compute unit), or 2048
// waves for the shapes of fewer than four waves.
template <int WM, int WN>
hipError_t launch_grouped_shape(const GroupedEntry* tab, int n, int64_t total, hipStream_t s) {
  using S = Shape<WM, WN>;
  const size_t lds = Ops3MBF16<WM, WN, 2>::kLds;
  const hipError_t e = ensure_lds_grouped<WM, WN>(lds);
  if (e != hipSuccess) return e;
  constexpr int64_t cap = WM * WN < 4 ? 2048 / (WM * WN) : 512;
  int64_t grid = (total + 7) / 8 * 8;
  if (grid > cap) grid = cap;
  hipLaunchKernelGGL((cgemm_mfma_grouped<WM, WN>), dim3(static_cast<unsigned>(grid)), dim3(S::NT), lds, s, tab,
                     n, total);
  return hipGetLastError();
}

// The 3M split form has no (4,4) instance: its three accumulator sets spill
// at sixteen waves per workgroup (compiler resource report), so a forced
// variant 3 runs its (4,2) tile, and has no grouped form (those fail with
// hipErrorInvalidValue; callers run such GEMMs one launch each).
constexpr bool grouped_ok_3m(int variant) { return variant >= 0 && variant < kGemmVariants && variant != 3; }

hipError_t launch_grouped_3m(const GroupedEntry* tab, int n, int64_t total, int variant, hipStream_t s) {
  switch (variant) {
    case 0: return launch_grouped_shape<2, 2>(tab, n, total, s);
    case 1: return launch_grouped_shape<4, 2>(tab, n, total, s);
    case 2: return launch_grouped_shape<2, 4>(tab, n, total, s);
    case 4: return launch_grouped_shape<1, 2>(tab, n, total, s);
    case 5: return launch_grouped_shape<2, 1>(tab, n, total, s);
    case 6: return launch_grouped_shape<1, 1>(tab, n, total, s);
    default: return hipErrorInvalidValue;
  }
}

template <int WM, int WN>
hipError_t launch_shape(const GemmDesc& d, hipStream_t s) {
  const size_t lds = Ops3MBF16<WM, WN, 2>::kLds;
  return d.offM ? launch_one<WM, WN, 2, true>(d, lds, s) : launch_one<WM, WN, 2, false>(d, lds, s);
}

hipError_t launch_split_3m(const GemmDesc& d, int variant, hipStream_t s) {
  if ((d.k | row_stride(d)) % 2 != 0) {  // odd k or row stride: 8-byte loads, default shape only
    const size_t lds = Ops3MBF16<2, 2, 1>::kLds;
    return d.offM ? launch_one<2, 2, 1, true>(d, lds, s) : launch_one<2, 2, 1, false>(d, lds, s);
  }
  switch (variant) {
    case 0: return launch_shape<2, 2>(d, s);
    case 1:
    case 3: return launch_shape<4, 2>(d, s);
    case 2: return launch_shape<2, 4>(d, s);
    case 4: return launch_shape<1, 2>(d, s);
    case 5: return launch_shape<2, 1>(d, s);
    case 6: return launch_shape<1, 1>(d, s);
    default: return hipErrorInvalidValue;
  }
}

// Which kernels run a form: split precision has both; complex64 runs the 4M
// kernels in either (8 x 1024 x 512 x 768 in float32 3M 163 complex TFLOP/s,
// 178 at best on large shapes, against 205-230 here, and with an imaginary
// part that is not a difference of three sums).
bool three_m(Form form, Prec prec) { return form == Form::M3 && prec == Prec::BF16X3; }

}  // namespace

void prepare_gemm_kernels() {
  prepare_gemm_4m();
  prepare_shape<2, 2>();
  prepare_shape<4, 2>();
  prepare_shape<2, 4>();
  prepare_shape<1, 2>();
  prepare_shape<2, 1>();
  prepare_shape<1, 1>();
  const size_t lds = Ops3MBF16<2, 2, 1>::kLds;  // odd-k path
  (void)ensure_lds<2, 2, 1, false>(lds);
  (void)ensure_lds<2, 2, 1, true>(lds);
  (void)ensure_lds_presplit();
}

void gemm_variant_tile(int variant, int* bm, int* bnc) {
  static const int rows[kAllVariants] = {128, 256, 128, 256, 64, 128, 64, 32, 32, 64};
  static const int cols[kAllVariants] = {64, 64, 128, 128, 64, 32, 32, 16, 32, 32};
  if (variant < 0 || variant >= kAllVariants) variant = 0;
  *bm = rows[variant];
  *bnc = cols[variant];
}

int64_t grouped_layout(GroupedEntry* e, int n, int variant) {
  int bm = 0, bnc = 0;
  gemm_variant_tile(variant, &bm, &bnc);
  int64_t total = 0;
  for (int i = 0; i < n; ++i) {
    const GemmDesc& d = e[i].d;
    if (d.h <= 0 || d.m <= 0 || d.n <= 0 || d.k <= 0 || (d.k | row_stride(d)) % 2 != 0) return 0;
    e[i].tiles_m = (d.m + bm - 1) / bm;
    e[i].tiles_n = (d.n + bnc - 1) / bnc;
    e[i].tile0 = total;
    total += e[i].tiles_m * e[i].tiles_n * d.h;
  }
  return total;
}

bool grouped_variant_ok(Form form, Prec prec, int variant) {
  if (three_m(form, prec)) return grouped_ok_3m(variant);
  return variant >= 0 && variant < kAllVariants;
}

hipError_t launch_gemm_grouped(const GroupedEntry* dev, int n, int64_t total, int variant, Form form, Prec prec,
                               hipStream_t s) {
  if (n <= 0 || total <= 0) return hipSuccess;
  if (three_m(form, prec)) return launch_grouped_3m(dev, n, total, variant, s);
  return launch_gemm_4m_grouped(dev, n, total, variant, prec, s);
}

hipError_t launch_gemm_presplit(const GemmDesc& d, void* planes, bool have_a, bool have_b, hipStream_t s) {
  if (d.h <= 0 || d.m <= 0 || d.n <= 0) return hipSuccess;
  if (d.k <= 0 || d.h != 1 || d.rowA || d.kA || d.rowB || d.kB || !planes ||
      reinterpret_cast<uintptr_t>(planes) % 256 != 0)
    return hipErrorInvalidValue;
  const int64_t mp = presplit_rows_a(d.m), np2 = presplit_rows_b(d.n), kp = presplit_k(d.k);
  const int64_t nkb = kp / 16;
  // one thread per padded element, counted in 32 bits
  if ((mp > np2 / 2 ? mp : np2 / 2) * kp >= (int64_t{1} << 31)) return hipErrorInvalidValue;
  const hipError_t e = ensure_lds_presplit();
  if (e != hipSuccess) return e;
  uint32_t* Ap = static_cast<uint32_t*>(planes);
  uint32_t* Bp = Ap + mp * 2 * kp;
  const int64_t ld = row_stride(d);
  auto grid = [](int64_t threads) {
    const int64_t g = (threads + 255) / 256;
    return static_cast<unsigned>(g < 131072 ? g : 131072);
  };
  const uint32_t blocks_a = static_cast<uint32_t>(mp * nkb), blocks_b = static_cast<uint32_t>(np2 / 2 * nkb);
  if (!have_a)
    hipLaunchKernelGGL(split_planes_a, dim3(grid(int64_t{blocks_a} * 16)), dim3(256), 0, s, d.A, d.m, d.k, ld,
                       static_cast<uint32_t>(nkb), blocks_a, kp, Ap);
  if (!have_b)
    hipLaunchKernelGGL(split_planes_b, dim3(grid(int64_t{blocks_b} * 16)), dim3(256), 0, s, d.B, d.n, d.k, ld,
                       static_cast<uint32_t>(nkb), blocks_b, kp, Bp);
  const int64_t tiles_m = mp / kPresplitBM, tiles_n = np2 / 2 / kPresplitBNC, total = tiles_m * tiles_n;
  if (d.offM)
    hipLaunchKernelGGL(cgemm_bf16x3_presplit<true>, dim3(static_cast<unsigned>(total)), dim3(512), PS_LDS, s, d, Ap,
                       Bp, kp, tiles_m, tiles_n, total);
  else
    hipLaunchKernelGGL(cgemm_bf16x3_presplit<false>, dim3(static_cast<unsigned>(total)), dim3(512), PS_LDS, s, d, Ap,
                       Bp, kp, tiles_m, tiles_n, total);
  return hipGetLastError();
}

hipError_t launch_gemm_presplit_3m(const GemmDesc& d, void* buf, bool have_a, bool have_b, hipStream_t s) {
  if (d.h <= 0 || d.m <= 0 || d.n <= 0) return hipSuccess;
  if (d.k <= 0 || d.h != 1 || d.rowA || d.kA || d.rowB || d.kB || !buf || reinterpret_cast<uintptr_t>(buf) % 256 != 0)
    return hipErrorInvalidValue;
  const Presplit3M g = presplit_3m_layout(d.m, d.n, d.k);
  // one thread per real k pair of a padded row, counted in 32 bits
  if ((g.mp > g.np ? g.mp : g.np) * g.kp >= (int64_t{1} << 31)) return hipErrorInvalidValue;
  hipError_t e = ensure_lds_presplit();
  if (e != hipSuccess) return e;
  char* base = static_cast<char*>(buf);
  uint32_t* Ap = reinterpret_cast<uint32_t*>(base);
  uint32_t* Bp = reinterpret_cast<uint32_t*>(base + g.off_b);
  float* T = reinterpret_cast<float*>(base + g.off_t);
  const int64_t ld = row_stride(d);
  auto grid = [](int64_t threads) {
    const int64_t q = (threads + 255) / 256;
    return static_cast<unsigned>(q < 131072 ? q : 131072);
  };
  const int64_t plane_a = g.mp * 2 * g.kp, plane_b = g.np * 2 * g.kp;  // uint32 per plane
  if (!have_a)
    hipLaunchKernelGGL(split_planes_3m, dim3(grid(g.mp * g.kp)), dim3(256), 0, s, d.A, d.m, d.k, ld,
                       static_cast<uint32_t>(g.kp), static_cast<uint32_t>(g.mp * g.kp), plane_a, Ap);
  if (!have_b)
    hipLaunchKernelGGL(split_planes_3m, dim3(grid(g.np * g.kp)), dim3(256), 0, s, d.B, d.n, d.k, ld,
                       static_cast<uint32_t>(g.kp), static_cast<uint32_t>(g.np * g.kp), plane_b, Bp);
  // T_p = X_p Y_p^T as the pre-split kernel's real GEMM: m rows, np real
  // columns (nh column pairs), 2 kp real k; stored row-major in pairs
  const int64_t tiles_m = g.mp / kPresplitBM, tiles_n = g.np / 2 / kPresplitBNC, total = tiles_m * tiles_n;
  for (int p = 0; p < 3; ++p) {
    GemmDesc dp;
    std::memset(&dp, 0, sizeof(dp));
    dp.C = reinterpret_cast<float2*>(T + p * g.tplane);
    dp.m = d.m;
    dp.n = g.nh;
    dp.k = g.kp;
    dp.h = 1;
    hipLaunchKernelGGL(cgemm_bf16x3_presplit<false>, dim3(static_cast<unsigned>(total)), dim3(512), PS_LDS, s, dp,
                       Ap + p * plane_a, Bp + p * plane_b, g.kp, tiles_m, tiles_n, total);
  }
  hipLaunchKernelGGL(combine_3m, dim3(grid(d.m * d.n)), dim3(256), 0, s, T, g.tplane, 2 * g.nh, d);
  return hipGetLastError();
}

hipError_t launch_gemm(const GemmDesc& d, GemmKernel kind, int variant, Form form, Prec prec, hipStream_t s) {
  if (d.h <= 0 || d.m <= 0 || d.n <= 0) return hipSuccess;
  if (d.k <= 0) return hipErrorInvalidValue;
  if (kind != GemmKernel::MFMA) return launch_gemm_valu(d, kind, prec, s);
  if (three_m(form, prec)) return launch_split_3m(d, variant, s);
  return launch_gemm_4m(d, variant, prec, s);
}

}  // namespace tnc
