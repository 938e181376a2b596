// Complex GEMM kernels for shapes that do not fill MFMA tiles (VALU): the
// same pairwise-contraction-as-GEMM of Sec. II-B for steps with few
// outputs or tiny extents.
//
// cgemm_small: one thread per output element, k looped in order; used for
// the many tiny steps of circuit networks (m, n or k of a few elements).
// cgemm_dot:   one wave64 per output element for long reductions with few
// outputs (k large, m*n tiny); 4 x 64 partial sums are combined by a fixed
// tree, so the summation error grows like k/256 + 8 roundings, not k
// (cgemm_dot_few: one workgroup per output where there are few of them).
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

template <bool SPLIT>
hipError_t launch_valu(const GemmDesc& d, const GemmDesc* runs, int n_runs, GemmKernel kind, hipStream_t s) {
  const int64_t total = d.h * d.m * d.n;
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
