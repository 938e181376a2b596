// Complex GEMM kernels for shapes that do not fill MFMA tiles (VALU): the
// same pairwise-contraction-as-GEMM of Sec. II-B for steps with few
// outputs or tiny extents.
//
// cgemm_small: one thread per output element, k looped in order; used for
// the many tiny steps of circuit networks (m, n or k of a few elements).
// cgemm_dot:   one wave64 per output element for long reductions with few
// outputs (k large, m*n tiny); 4 x 64 partial sums are combined by a fixed
// tree, so the summation error grows like k/256 + 8 roundings, not k
// (cgemm_dot_few: one workgroup per output where there are few of them;
// cgemm_dot_tile: one per block of outputs that share rows of A and B).
// Both honour the split-bf16 precision with the same products as the MFMA
// kernel (hi*hi and the two cross products accumulated separately).
#include "gemm_common.hpp"

namespace tnc {

namespace {

template <bool SPLIT>
__device__ __forceinline__ void small_body(const GemmDesc& d) {
  const int64_t mn = d.m * d.n;
  const int64_t total = d.h * mn;
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < total;
       idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t b = idx / mn;
    const int64_t r = idx - b * mn;
    const int64_t i = r / d.n;
    const int64_t j = r - i * d.n;
    int64_t oa, ob;
    batch_offsets(d, b, oa, ob);
    float cr = 0.f, ci = 0.f, crx = 0.f, cix = 0.f;
    if (d.kA || d.kB) {
      const float2* a = d.A + oa + (d.baseA ? *d.baseA : 0) + (d.rowA ? d.rowA[i] : i * row_stride(d));
      const float2* bb = d.B + ob + (d.baseB ? *d.baseB : 0) + (d.rowB ? d.rowB[j] : j * row_stride(d));
      cdot_tables<SPLIT>(a, d.kA, bb, d.kB, d.k, cr, ci, crx, cix);
    } else {
      cdot_serial<SPLIT>(d.A + oa + i * row_stride(d), d.B + ob + j * row_stride(d), d.k, cr, ci, crx, cix);
    }
    const int64_t c = b * mn + (d.offM ? d.offM[i] + d.offN[j] : r);
    if constexpr (SPLIT)
      d.C[c] = make_float2(cr + crx, ci + cix);
    else
      d.C[c] = make_float2(cr, ci);
  }
}

// Long reductions with few outputs (k large, m*n tiny): one wave64 per output
// element; lanes stride over k with coalesced reads, each lane keeping four
// independent partial sums (four loads per operand in flight), and the
// 64 x 4 partial sums are combined by a fixed tree, so the summation error
// grows like (k/256 + 8) roundings instead of k.
constexpr int64_t kDotFewOutputs = 1024;  // four waves each fill the chip at most twice

template <bool SPLIT>
struct DotAcc {
  float cr = 0.f, ci = 0.f, crx = 0.f, cix = 0.f;
  __device__ __forceinline__ void add(float2 x, float2 y) { cmac<SPLIT>(x, y, cr, ci, crx, cix); }
};

template <bool SPLIT>
__device__ __forceinline__ void dot_body(const GemmDesc& d) {
  const int lane = threadIdx.x & 63;
  const int64_t mn = d.m * d.n;
  const int64_t total = d.h * mn;
  const int64_t out = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (out >= total) return;  // uniform per wave
  const int64_t b = out / mn;
  const int64_t r = out - b * mn;
  const int64_t i = r / d.n;
  const int64_t j = r - i * d.n;
  int64_t oa, ob;
  batch_offsets(d, b, oa, ob);
  const float2* a = d.A + oa + i * row_stride(d);
  const float2* bb = d.B + ob + j * row_stride(d);
  DotAcc<SPLIT> acc[4];
  int64_t l = lane;
  for (; l + 192 < d.k; l += 256) {
    float2 x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = a[l + 64 * u];
      y[u] = bb[l + 64 * u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u].add(x[u], y[u]);
  }
#pragma unroll
  for (int u = 0; u < 3; ++u)  // the last < 256 elements
    if (l + 64 * u < d.k) acc[u].add(a[l + 64 * u], bb[l + 64 * u]);
  float cr[4], ci[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    cr[u] = acc[u].cr + acc[u].crx;
    ci[u] = acc[u].ci + acc[u].cix;
  }
  float sr = (cr[0] + cr[1]) + (cr[2] + cr[3]);
  float si = (ci[0] + ci[1]) + (ci[2] + ci[3]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sr += __shfl_xor(sr, off, 64);
    si += __shfl_xor(si, off, 64);
  }
  if (lane == 0) {
    const int64_t c = b * mn + (d.offM ? d.offM[i] + d.offN[j] : r);
    d.C[c] = make_float2(sr, si);
  }
}

// The same for a launch with few outputs: one workgroup per output (as a
// wave per output, k = 4096 took 7.4 us for 16 outputs on four CUs, now
// 3.9).  The four waves' sums are added in order.
template <bool SPLIT>
__device__ __forceinline__ void dot_few_body(const GemmDesc& d) {
  __shared__ float2 part[4];
  const int tid = threadIdx.x;
  const int64_t mn = d.m * d.n, out = blockIdx.x;
  const int64_t b = out / mn, r = out - b * mn, i = r / d.n, j = r - i * d.n;
  int64_t oa, ob;
  batch_offsets(d, b, oa, ob);
  const float2* a = d.A + oa + i * row_stride(d);
  const float2* bb = d.B + ob + j * row_stride(d);
  DotAcc<SPLIT> acc[4];
  int64_t l = tid;
  for (; l + 768 < d.k; l += 1024) {
    float2 x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = a[l + 256 * u];
      y[u] = bb[l + 256 * u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u].add(x[u], y[u]);
  }
#pragma unroll
  for (int u = 0; u < 3; ++u)  // the last < 1024 elements
    if (l + 256 * u < d.k) acc[u].add(a[l + 256 * u], bb[l + 256 * u]);
  float sr = 0.f, si = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    sr += acc[u].cr + acc[u].crx;
    si += acc[u].ci + acc[u].cix;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sr += __shfl_xor(sr, off, 64);
    si += __shfl_xor(si, off, 64);
  }
  if ((tid & 63) == 0) part[tid >> 6] = make_float2(sr, si);
  __syncthreads();
  if (tid == 0) {
    const int64_t c = b * mn + (d.offM ? d.offM[i] + d.offN[j] : r);
    d.C[c] = make_float2((part[0].x + part[1].x) + (part[2].x + part[3].x),
                         (part[0].y + part[1].y) + (part[2].y + part[3].y));
  }
}

// Many long reductions over shared operands: one workgroup per R x N outputs,
// R rows of A that meet the same N rows of B.  A row axis is m, or a batch dim
// that B does not have; a column axis n, or a batch dim that A does not have.
// What bounds the one-output kernels there is the path from the caches: every
// output reads two rows.  Here 32 outputs read 12 (the last step of 256
// slices of a 40-qubit circuit, 16384 outputs of k = 32768 over 0.8 GB of
// operands: 8.6 GB through the L1s and 613 us, now 189; 64 x 32 x 2 x 32768
// 201 -> 124; 256 x 8 x 8 x 2048 37 -> 16).  Each thread keeps one running sum
// per output (k / 256 terms, as above); the 256 are combined by a fixed tree,
// a level of which halves the sums that a lane carries.
struct DotTile {
  int32_t rd, cd;        // the axes' batch dims; -1: m, n
  int32_t rows, cols;    // their extents
  int32_t rb, cb;        // blocks along them
  int32_t r, n;          // R, N
  int8_t order[kMaxBatchDims];  // the other batch dims, fastest first
};

template <bool SPLIT, int R, int N>
__device__ __forceinline__ void dot_tile_body(const GemmDesc& d, const DotTile& t) {
  constexpr int V = 2 * R * N;
  __shared__ float part[4][V];
  const int tid = threadIdx.x, lane = tid & 63;
  // block -> axes' blocks (fastest), batch digits, the axes not taken
  const uint32_t per = (gridDim.x + 7) >> 3;  // neighbours share operands: keep them on one XCD
  const uint32_t full = gridDim.x & 7;        // XCDs with `per` blocks (0: all)
  const uint32_t x = blockIdx.x & 7;
  int64_t q = int64_t{x} * per - (full && x > full ? x - full : 0) + (blockIdx.x >> 3);
  const int cblk = static_cast<int>(q % t.cb);
  q /= t.cb;
  const int rblk = static_cast<int>(q % t.rb);
  q /= t.rb;
  int64_t i = 0, j = 0, oa = 0, ob = 0, b = 0;
  for (int e = 0; e < d.nbd; ++e) {
    const int dim = t.order[e];
    if (dim < 0) break;
    const int64_t dig = q % d.bext[dim];
    q /= d.bext[dim];
    int64_t w = 1;  // the dim's weight in b
    for (int f = dim + 1; f < d.nbd; ++f) w *= d.bext[f];
    oa += dig * d.bsA[dim];
    ob += dig * d.bsB[dim];
    b += dig * w;
  }
  auto weight = [&](int dim) {
    int64_t w = 1;
    for (int f = dim + 1; f < d.nbd; ++f) w *= d.bext[f];
    return w;
  };
  if (t.cd >= 0) {
    j = q % d.n;
    q /= d.n;
  }
  if (t.rd >= 0) i = q % d.m;
  const int64_t ld = row_stride(d);
  const int64_t sr = t.rd >= 0 ? d.bsA[t.rd] : ld, sc = t.cd >= 0 ? d.bsB[t.cd] : ld;
  const float2 *pa[R], *pb[N];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int g = rblk * R + r;
    pa[r] = d.A + oa + i * ld + (g < t.rows ? g : t.rows - 1) * sr;
  }
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const int g = cblk * N + c;
    pb[c] = d.B + ob + j * ld + (g < t.cols ? g : t.cols - 1) * sc;
  }
  DotAcc<SPLIT> acc[R][N];
  auto step = [&](const float2 (&u)[R], const float2 (&v)[N]) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < N; ++c) acc[r][c].add(u[r], v[c]);
  };
  const int k = static_cast<int>(d.k);
  int l = tid;
  if (l < k) {
    float2 u[R], v[N];
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = pa[r][l];
#pragma unroll
    for (int c = 0; c < N; ++c) v[c] = pb[c][l];
    for (; l + 256 < k; l += 256) {  // the next step's elements are on their way
      float2 u1[R], v1[N];
#pragma unroll
      for (int r = 0; r < R; ++r) u1[r] = pa[r][l + 256];
#pragma unroll
      for (int c = 0; c < N; ++c) v1[c] = pb[c][l + 256];
      step(u, v);
#pragma unroll
      for (int r = 0; r < R; ++r) u[r] = u1[r];
#pragma unroll
      for (int c = 0; c < N; ++c) v[c] = v1[c];
    }
    step(u, v);
  }
  float s[V];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < N; ++c) {
      s[2 * (r * N + c)] = acc[r][c].cr + acc[r][c].crx;
      s[2 * (r * N + c) + 1] = acc[r][c].ci + acc[r][c].cix;
    }
  // sum over the wave: lane bits 5, 4, ... each pick the half that a lane
  // goes on with, so lane ends up with sum lane / (64 / V)
  int off = 32;
#pragma unroll
  for (int w = V / 2; w > 0; w >>= 1, off >>= 1) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int e = 0; e < w; ++e) {
      const float mine = up ? s[e + w] : s[e], other = up ? s[e] : s[e + w];
      s[e] = mine + __shfl_xor(other, off, 64);
    }
  }
  for (; off > 0; off >>= 1) s[0] += __shfl_xor(s[0], off, 64);
  constexpr int G = 64 / V;
  if (lane % G == 0) part[tid >> 6][lane / G] = s[0];
  __syncthreads();
  if (tid >= V) return;
  const int o = tid >> 1, gr = rblk * R + o / N, gc = cblk * N + o % N;
  if (gr >= t.rows || gc >= t.cols) return;
  if (t.rd >= 0)
    b += gr * weight(t.rd);
  else
    i = gr;
  if (t.cd >= 0)
    b += gc * weight(t.cd);
  else
    j = gc;
  const int64_t c = b * d.m * d.n + (d.offM ? d.offM[i] + d.offN[j] : i * d.n + j);
  reinterpret_cast<float*>(d.C + c)[tid & 1] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
}

template <bool SPLIT, int R, int N>
__global__ __launch_bounds__(256) void cgemm_dot_tile(GemmDesc d, DotTile t) {
  dot_tile_body<SPLIT, R, N>(d, t);
}
template <bool SPLIT, int R, int N>
__global__ __launch_bounds__(256) void cgemm_dot_tile_runs(const GemmDesc* __restrict__ runs, DotTile t) {
  dot_tile_body<SPLIT, R, N>(runs[blockIdx.y], t);
}

// The block of outputs for a step, or none (r = 0): the axes with the longest
// extents (a batch dim only where m or n is 1), the largest block that leaves
// 512 workgroups and no quarter of itself empty.  None where the rows are
// read at most three times anyway (512 x 1 x 32 x 1024 is at 6.2 TB/s one
// output at a time, 21.8 us, and 26.0 in blocks) and none below 2^25 complex
// MACs, where the blocks' longer prologue shows (100 x 16 x 4 x 600: 7.6 us,
// and 12.4).
DotTile dot_tile(const GemmDesc& d) {
  DotTile t{};
  t.rd = t.cd = -1;
  t.rows = static_cast<int32_t>(d.m);
  t.cols = static_cast<int32_t>(d.n);
  for (int e = 0; e < d.nbd; ++e) {
    if (d.m == 1 && d.bsB[e] == 0 && d.bsA[e] != 0 && d.bext[e] > t.rows) t.rows = d.bext[t.rd = e];
    if (d.n == 1 && d.bsA[e] == 0 && d.bsB[e] != 0 && d.bext[e] > t.cols) t.cols = d.bext[t.cd = e];
  }
  const int64_t total = d.h * d.m * d.n;
  if (d.k > 0x3FFFFFFF || total * d.k < (int64_t{1} << 25)) return t;
  int64_t ha = 1, hb = 1;
  for (int e = 0; e < d.nbd; ++e) {
    if (d.bsA[e] != 0) ha *= d.bext[e];
    if (d.bsB[e] != 0) hb *= d.bext[e];
  }
  if (2 * total < 3 * (ha * d.m + hb * d.n)) return t;
  static const int shapes[][2] = {{4, 8}, {8, 4}, {4, 4}, {2, 8}, {8, 2}, {2, 4}, {4, 2}};
  for (auto& s : shapes) {
    const int64_t rb = (t.rows + s[0] - 1) / s[0], cb = (t.cols + s[1] - 1) / s[1];
    const int64_t blocks = total / (int64_t{t.rows} * t.cols) * rb * cb;
    if (blocks < 512 || blocks > 0x7FFFFF || blocks * s[0] * s[1] * 3 > total * 4) continue;
    t.r = s[0];
    t.n = s[1];
    t.rb = static_cast<int32_t>(rb);
    t.cb = static_cast<int32_t>(cb);
    break;
  }
  // blocks that share B first, then those that share A, so that neighbours do
  int q = 0;
  for (int pass = 0; pass < 3; ++pass)
    for (int e = d.nbd - 1; e >= 0; --e)
      if (e != t.rd && e != t.cd && (d.bsB[e] == 0 ? 0 : d.bsA[e] == 0 ? 1 : 2) == pass) t.order[q++] = static_cast<int8_t>(e);
  if (q < kMaxBatchDims) t.order[q] = -1;
  return t;
}

// One launch for the step, or for the same step of several runs (grid row y
// is run y, its descriptor in the table): eight requests of a fused job that
// end in a small step each, a reduction and a copy took 24 launches there,
// 13 us apart while the workers contend for the runtime.
template <bool SPLIT>
__global__ __launch_bounds__(256) void cgemm_small(GemmDesc d) {
  small_body<SPLIT>(d);
}
template <bool SPLIT>
__global__ __launch_bounds__(256) void cgemm_small_runs(const GemmDesc* __restrict__ runs) {
  small_body<SPLIT>(runs[blockIdx.y]);
}
template <bool SPLIT>
__global__ __launch_bounds__(256) void cgemm_dot(GemmDesc d) {
  dot_body<SPLIT>(d);
}
template <bool SPLIT>
__global__ __launch_bounds__(256) void cgemm_dot_runs(const GemmDesc* __restrict__ runs) {
  dot_body<SPLIT>(runs[blockIdx.y]);
}
template <bool SPLIT>
__global__ __launch_bounds__(256) void cgemm_dot_few(GemmDesc d) {
  dot_few_body<SPLIT>(d);
}
template <bool SPLIT>
__global__ __launch_bounds__(256) void cgemm_dot_few_runs(const GemmDesc* __restrict__ runs) {
  dot_few_body<SPLIT>(runs[blockIdx.y]);
}

__device__ __forceinline__ void splitk_body(const float2* __restrict__ P, float2* __restrict__ C, int64_t h, int64_t m,
                                            int64_t n, int64_t S, const int64_t* __restrict__ offM,
                                            const int64_t* __restrict__ offN) {
  const int64_t mn = m * n;
  const int64_t total = h * mn;
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < total;
       idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    int64_t b, r, i;
    if (total <= 0xFFFFFFFFll) {  // 32-bit divisions
      const uint32_t x = static_cast<uint32_t>(idx), xm = static_cast<uint32_t>(mn);
      b = x / xm;
      r = x - static_cast<uint32_t>(b) * xm;
      i = static_cast<uint32_t>(r) / static_cast<uint32_t>(n);
    } else {
      b = idx / mn;
      r = idx - b * mn;
      i = r / n;
    }
    const float2* p = P + b * S * mn + r;
    float cr = 0.f, ci = 0.f;
    int64_t q = 0;
    for (; q + 8 <= S; q += 8) {  // eight reads in flight, added in order
      float2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(q + u) * mn];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        cr += v[u].x;
        ci += v[u].y;
      }
    }
    for (; q < S; ++q) {
      const float2 v = p[q * mn];
      cr += v.x;
      ci += v.y;
    }
    const int64_t j = r - i * n;
    C[b * mn + (offM ? offM[i] + offN[j] : r)] = make_float2(cr, ci);
  }
}

__global__ __launch_bounds__(256) void splitk_reduce(const float2* __restrict__ P, float2* __restrict__ C,
                                                     int64_t h, int64_t m, int64_t n, int64_t S,
                                                     const int64_t* __restrict__ offM,
                                                     const int64_t* __restrict__ offN) {
  splitk_body(P, C, h, m, n, S, offM, offN);
}
__global__ __launch_bounds__(256) void splitk_reduce_runs(const SplitkRun* __restrict__ runs, int64_t h, int64_t m,
                                                          int64_t n, int64_t S) {
  const SplitkRun q = runs[blockIdx.y];
  splitk_body(q.P, q.C, h, m, n, S, q.offM, q.offN);
}

int64_t elements_grid(int64_t total) {
  const int64_t grid = (total + 255) / 256;
  return grid > 1048576 ? 1048576 : grid;
}

template <bool SPLIT, int R, int N>
hipError_t launch_dot_block(const GemmDesc& d, const GemmDesc* runs, int n_runs, const DotTile& t, hipStream_t s) {
  const int64_t blocks = d.h * d.m * d.n / (int64_t{t.rows} * t.cols) * t.rb * t.cb;
  const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(n_runs));
  if (runs)
    hipLaunchKernelGGL((cgemm_dot_tile_runs<SPLIT, R, N>), grid, dim3(256), 0, s, runs, t);
  else
    hipLaunchKernelGGL((cgemm_dot_tile<SPLIT, R, N>), grid, dim3(256), 0, s, d, t);
  return hipGetLastError();
}

template <bool SPLIT>
hipError_t launch_dot_tile(const GemmDesc& d, const GemmDesc* runs, int n_runs, const DotTile& t, hipStream_t s) {
  switch (16 * t.r + t.n) {
#define TNC_DOT_CASE(R, N) \
  case 16 * R + N: return launch_dot_block<SPLIT, R, N>(d, runs, n_runs, t, s);
    TNC_DOT_CASE(4, 8)
    TNC_DOT_CASE(8, 4)
    TNC_DOT_CASE(4, 4)
    TNC_DOT_CASE(2, 8)
    TNC_DOT_CASE(8, 2)
    TNC_DOT_CASE(2, 4)
    TNC_DOT_CASE(4, 2)
#undef TNC_DOT_CASE
    default: return hipErrorInvalidValue;
  }
}

template <bool SPLIT>
hipError_t launch_valu(const GemmDesc& d, const GemmDesc* runs, int n_runs, GemmKernel kind, hipStream_t s) {
  const int64_t total = d.h * d.m * d.n;
  if (kind == GemmKernel::DOT) {
    const DotTile t = dot_tile(d);
    if (t.r) return launch_dot_tile<SPLIT>(d, runs, n_runs, t, s);
  }
  const bool few = total <= kDotFewOutputs;
  const int64_t gx = kind == GemmKernel::SMALL ? elements_grid(total) : few ? total : (total + 3) / 4;
  if (gx > 0x7FFFFFLL) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(n_runs));
  if (kind == GemmKernel::SMALL) {
    if (runs)
      hipLaunchKernelGGL(cgemm_small_runs<SPLIT>, grid, dim3(256), 0, s, runs);
    else
      hipLaunchKernelGGL(cgemm_small<SPLIT>, grid, dim3(256), 0, s, d);
  } else if (few) {
    if (runs)
      hipLaunchKernelGGL(cgemm_dot_few_runs<SPLIT>, grid, dim3(256), 0, s, runs);
    else
      hipLaunchKernelGGL(cgemm_dot_few<SPLIT>, grid, dim3(256), 0, s, d);
  } else {
    if (runs)
      hipLaunchKernelGGL(cgemm_dot_runs<SPLIT>, grid, dim3(256), 0, s, runs);
    else
      hipLaunchKernelGGL(cgemm_dot<SPLIT>, grid, dim3(256), 0, s, d);
  }
  return hipGetLastError();
}

hipError_t launch_valu(const GemmDesc& d, const GemmDesc* runs, int n_runs, GemmKernel kind, Prec prec, hipStream_t s) {
  if (d.h <= 0 || d.m <= 0 || d.n <= 0) return hipSuccess;
  if (d.k <= 0 || n_runs < 1 || n_runs > 65535 || (kind != GemmKernel::SMALL && kind != GemmKernel::DOT))
    return hipErrorInvalidValue;
  return prec == Prec::BF16X3 ? launch_valu<true>(d, runs, n_runs, kind, s) : launch_valu<false>(d, runs, n_runs, kind, s);
}

}  // namespace

hipError_t launch_splitk_reduce(const float2* P, float2* C, int64_t h, int64_t m, int64_t n, int64_t S,
                                const int64_t* offM, const int64_t* offN, hipStream_t s) {
  const int64_t total = h * m * n;
  if (total <= 0) return hipSuccess;
  if (S <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(splitk_reduce, dim3(static_cast<unsigned>(elements_grid(total))), dim3(256), 0, s, P, C, h, m, n, S,
                     offM, offN);
  return hipGetLastError();
}

hipError_t launch_splitk_reduce_runs(const SplitkRun* runs, int n_runs, int64_t h, int64_t m, int64_t n, int64_t S,
                                     hipStream_t s) {
  const int64_t total = h * m * n;
  if (total <= 0) return hipSuccess;
  if (S <= 0 || n_runs < 1 || n_runs > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(splitk_reduce_runs, dim3(static_cast<unsigned>(elements_grid(total)), static_cast<unsigned>(n_runs)),
                     dim3(256), 0, s, runs, h, m, n, S);
  return hipGetLastError();
}

hipError_t launch_gemm_valu(const GemmDesc& d, GemmKernel kind, Prec prec, hipStream_t s) {
  return launch_valu(d, nullptr, 1, kind, prec, s);
}

hipError_t launch_gemm_valu_runs(const GemmDesc& shape, const GemmDesc* runs, int n_runs, GemmKernel kind, Prec prec,
                                 hipStream_t s) {
  return runs ? launch_valu(shape, runs, n_runs, kind, prec, s) : hipErrorInvalidValue;
}

}  // namespace tnc
