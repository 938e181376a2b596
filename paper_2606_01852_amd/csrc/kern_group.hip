// Grouped launches: every small step (or leaf gather) of one level of the
// contraction tree (the SSA path of Sec. II-B) in a single kernel.
//
// Steps of one level depend only on lower levels, so they can run together.
// Circuit and grid networks have hundreds of tiny steps but trees only
// 10-20 levels deep; one launch per level instead of per step removes most
// of the launch chain that otherwise bounds their latency, and consecutive
// levels with next to no work share a launch of one workgroup.  A GEMM
// launch gives each workgroup elements of one step (a table made with the
// plan says which), a gather finds its leaf by binary search over the level's
// prefix sums; each thread then does exactly what the one-step kernel does
// for that element, so results are bitwise those of the per-step launches.
// The "runs" forms do the same over the levels of several runs of one
// structure (a fused serving job): a workgroup first finds its run.
#include "gemm_common.hpp"

namespace tnc {

namespace {

__device__ __forceinline__ int find_item(const int64_t* prefix, int n, int64_t gt) {
  int lo = 0, hi = n - 1;  // largest i with prefix[i] <= gt
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= gt)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

template <typename T>
__device__ __forceinline__ T* reloc(const void* p, int flag, char* arena) {
  return flag ? reinterpret_cast<T*>(arena + reinterpret_cast<intptr_t>(p)) : (T*)p;
}

// x / (uniform divisor): a shift where that is a power of two
__device__ __forceinline__ uint32_t udiv(uint32_t x, uint32_t by, int32_t shift) {
  return shift >= 0 ? x >> shift : x / by;
}

// One workgroup's share of a level's grouped small GEMMs: `per` output
// elements of one entry, so that the entry and everything read from it is
// uniform (scalar loads, scalar branches).  What bounds these launches is the
// chain of dependent reads before the first product (with a search over the
// level's prefix sums and 64-bit divisions per element the 8 x 8 lattice's
// seven levels took 9.4 us each, now 8.3) and, on the wide ones, 64 lanes
// reading as many rows of B at a time.
template <bool SPLIT>
__device__ __forceinline__ void small_gemm_block(const GroupGemm* __restrict__ g, const GroupBlock& bl, int per,
                                                 char* arena, const int64_t* bases) {
  const GroupGemm& e = g[bl.entry];
  const GemmDesc& d = e.d;
  const int64_t mn = d.m * d.n, ld = row_stride(d);
  const float2* A0 = reloc<const float2>(d.A, e.rel_a, arena);
  const float2* B0 = reloc<const float2>(d.B, e.rel_b, arena);
  float2* C = reloc<float2>(d.C, e.rel_c, arena);
  const bool vec = e.vec && reinterpret_cast<uintptr_t>(arena) % 16 == 0;
  for (int t = threadIdx.x; t < per; t += 256) {
    const int64_t idx = bl.first + t;
    if (idx >= e.total) return;
    int64_t b, i, j;
    if (e.total <= 0xFFFFFFFFll) {
      const uint32_t x = static_cast<uint32_t>(idx), n = static_cast<uint32_t>(d.n);
      const uint32_t xb = udiv(x, static_cast<uint32_t>(mn), e.shift_mn), xr = x - xb * static_cast<uint32_t>(mn);
      const uint32_t xi = udiv(xr, n, e.shift_n);
      b = xb;
      i = xi;
      j = xr - xi * n;
    } else {
      b = idx / mn;
      i = (idx - b * mn) / d.n;
      j = idx - b * mn - i * d.n;
    }
    int64_t oa, ob;
    batch_offsets(d, b, oa, ob);
    const float2* A = A0 + oa;
    const float2* B = B0 + ob;
    float cr = 0.f, ci = 0.f, crx = 0.f, cix = 0.f;
    if (d.kA || d.kB) {  // in-place leaf operands (tables, per-chunk base offsets)
      A += (e.slot_a >= 0 ? bases[e.slot_a] : 0) + (d.rowA ? d.rowA[i] : i * ld);
      B += (e.slot_b >= 0 ? bases[e.slot_b] : 0) + (d.rowB ? d.rowB[j] : j * ld);
      cdot_tables<SPLIT>(A, d.kA, B, d.kB, d.k, cr, ci, crx, cix);
    } else if (vec) {
      cdot_pairs<SPLIT>(A + i * ld, B + j * ld, d.k, cr, ci, crx, cix);
    } else {
      cdot_serial<SPLIT>(A + i * ld, B + j * ld, d.k, cr, ci, crx, cix);
    }
    const int64_t c = b * mn + (d.offM ? d.offM[i] + d.offN[j] : i * d.n + j);
    if constexpr (SPLIT)
      C[c] = make_float2(cr + crx, ci + cix);
    else
      C[c] = make_float2(cr, ci);
  }
}

// Consecutive levels of few outputs in one workgroup.  Each would take a
// launch of its own (about 3.5 us in a replayed graph) for a fraction of a
// microsecond of work; here a level is a barrier and one round of operand
// reads, its item read before the barrier: the first eleven levels of the
// 12-qubit circuit take 11 us, and its 4096 amplitudes 34 instead of 60.
template <bool SPLIT>
__device__ __forceinline__ void run_chain(const ChainItem* __restrict__ items, const int32_t* __restrict__ bounds,
                                          int levels, char* arena) {
  const bool aligned = reinterpret_cast<uintptr_t>(arena) % 16 == 0;
  const int tid = threadIdx.x;
  ChainItem it{};
  if (bounds[0] + tid < bounds[1]) it = items[bounds[0] + tid];
  for (int l = 0; l < levels; ++l) {
    const int end = bounds[l + 1];
    for (int t = bounds[l] + tid; t < end; t += kChainThreads) {
      const float2* A = reinterpret_cast<const float2*>(it.flags & 1 ? arena + it.a : reinterpret_cast<char*>(it.a));
      const float2* B = reinterpret_cast<const float2*>(it.flags & 2 ? arena + it.b : reinterpret_cast<char*>(it.b));
      float cr = 0.f, ci = 0.f, crx = 0.f, cix = 0.f;
      if ((it.flags & 4) && aligned)
        cdot_pairs<SPLIT>(A, B, it.k, cr, ci, crx, cix);
      else
        cdot_serial<SPLIT>(A, B, it.k, cr, ci, crx, cix);
      float2* c = reinterpret_cast<float2*>(arena + it.c);
      if constexpr (SPLIT)
        *c = make_float2(cr + crx, ci + cix);
      else
        *c = make_float2(cr, ci);
      if (t + kChainThreads < end) it = items[t + kChainThreads];
    }
    if (l + 1 < levels && end + tid < bounds[l + 2]) it = items[end + tid];
    __syncthreads();
  }
}

template <bool SPLIT>
__global__ __launch_bounds__(kChainThreads) void level_chain(const ChainItem* __restrict__ items,
                                                             const int32_t* __restrict__ bounds, int levels,
                                                             char* arena) {
  run_chain<SPLIT>(items, bounds, levels, arena);
}

template <bool SPLIT>
__global__ __launch_bounds__(kChainThreads) void level_chain_runs(const GroupRun* __restrict__ runs) {
  const GroupRun& q = runs[blockIdx.x];
  run_chain<SPLIT>(static_cast<const ChainItem*>(q.table), static_cast<const int32_t*>(q.index), q.n, q.arena);
}

// Work item gt of a level's grouped leaf gathers: one output element.
__device__ __forceinline__ void gather_item(const GroupGather* __restrict__ g, const int64_t* __restrict__ prefix,
                                            int n, int64_t gt, char* arena, const int64_t* bases) {
  const int s = find_item(prefix, n, gt);
  const GroupGather& e = g[s];
  int64_t rest = gt - prefix[s];
  int64_t off = e.base_slot >= 0 ? bases[e.base_slot] : 0;
  for (int j = e.rank - 1; j >= 0; --j) {
    const int64_t x = e.ext[j];
    const int64_t q = rest / x;
    off += (rest - q * x) * e.in_stride[j];
    rest = q;
  }
  reinterpret_cast<float2*>(arena + e.out_off)[gt - prefix[s]] = e.in[off];
}

// the run holding work item gt (runs in launch order, a few dozen at most)
__device__ __forceinline__ int find_run(const GroupRun* runs, int n_runs, int64_t gt) {
  int r = 0;
  while (r + 1 < n_runs && runs[r + 1].first <= gt) ++r;
  return r;
}

template <bool SPLIT>
__global__ __launch_bounds__(256) void group_small_gemm(const GroupGemm* __restrict__ g,
                                                        const GroupBlock* __restrict__ blocks, int per, char* arena,
                                                        const int64_t* bases) {
  small_gemm_block<SPLIT>(g, blocks[blockIdx.x], per, arena, bases);
}

template <bool SPLIT>
__global__ __launch_bounds__(256) void group_small_gemm_runs(const GroupRun* __restrict__ runs, int n_runs) {
  const GroupRun& q = runs[find_run(runs, n_runs, blockIdx.x)];
  small_gemm_block<SPLIT>(static_cast<const GroupGemm*>(q.table),
                          static_cast<const GroupBlock*>(q.index)[blockIdx.x - q.first], q.per, q.arena, q.bases);
}

__global__ __launch_bounds__(256) void group_gather(const GroupGather* __restrict__ g, const int64_t* __restrict__ prefix,
                                                    int n, int64_t total, char* arena, const int64_t* bases) {
  for (int64_t gt = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; gt < total;
       gt += static_cast<int64_t>(gridDim.x) * blockDim.x)
    gather_item(g, prefix, n, gt, arena, bases);
}

__global__ __launch_bounds__(256) void group_gather_runs(const GroupRun* __restrict__ runs, int n_runs, int64_t total) {
  for (int64_t gt = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; gt < total;
       gt += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const GroupRun& q = runs[find_run(runs, n_runs, gt)];
    gather_item(static_cast<const GroupGather*>(q.table), static_cast<const int64_t*>(q.index), q.n, gt - q.first,
                q.arena, q.bases);
  }
}

int64_t grid_for(int64_t total) {
  int64_t g = (total + 255) / 256;
  if (g < 1) g = 1;
  return g > 1048576 ? 1048576 : g;
}

}  // namespace

hipError_t launch_group_gemm(const GroupGemm* table, const GroupBlock* blocks, int64_t n_blocks, int32_t per,
                             char* arena, const int64_t* bases, Prec prec, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  if (n_blocks > 0xFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(n_blocks));
  if (prec == Prec::BF16X3)
    hipLaunchKernelGGL(group_small_gemm<true>, grid, dim3(256), 0, s, table, blocks, per, arena, bases);
  else
    hipLaunchKernelGGL(group_small_gemm<false>, grid, dim3(256), 0, s, table, blocks, per, arena, bases);
  return hipGetLastError();
}

hipError_t launch_level_chain(const ChainItem* items, const int32_t* bounds, int levels, char* arena, Prec prec,
                              hipStream_t s) {
  if (levels <= 0) return hipSuccess;
  if (prec == Prec::BF16X3)
    hipLaunchKernelGGL(level_chain<true>, dim3(1), dim3(kChainThreads), 0, s, items, bounds, levels, arena);
  else
    hipLaunchKernelGGL(level_chain<false>, dim3(1), dim3(kChainThreads), 0, s, items, bounds, levels, arena);
  return hipGetLastError();
}

hipError_t launch_level_chain_runs(const GroupRun* runs, int n_runs, Prec prec, hipStream_t s) {
  if (n_runs <= 0) return hipSuccess;
  if (prec == Prec::BF16X3)
    hipLaunchKernelGGL(level_chain_runs<true>, dim3(n_runs), dim3(kChainThreads), 0, s, runs);
  else
    hipLaunchKernelGGL(level_chain_runs<false>, dim3(n_runs), dim3(kChainThreads), 0, s, runs);
  return hipGetLastError();
}

hipError_t launch_group_gather(const GroupGather* table, const int64_t* prefix, int n, int64_t total, char* arena,
                               const int64_t* bases, hipStream_t s) {
  if (n <= 0 || total <= 0) return hipSuccess;
  hipLaunchKernelGGL(group_gather, dim3(grid_for(total)), dim3(256), 0, s, table, prefix, n, total, arena, bases);
  return hipGetLastError();
}

hipError_t launch_group_gemm_runs(const GroupRun* runs, int n_runs, int64_t n_blocks, Prec prec, hipStream_t s) {
  if (n_runs <= 0 || n_blocks <= 0) return hipSuccess;
  if (n_blocks > 0xFFFFFF) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(n_blocks));
  if (prec == Prec::BF16X3)
    hipLaunchKernelGGL(group_small_gemm_runs<true>, grid, dim3(256), 0, s, runs, n_runs);
  else
    hipLaunchKernelGGL(group_small_gemm_runs<false>, grid, dim3(256), 0, s, runs, n_runs);
  return hipGetLastError();
}

hipError_t launch_group_gather_runs(const GroupRun* runs, int n_runs, int64_t total, hipStream_t s) {
  if (n_runs <= 0 || total <= 0) return hipSuccess;
  hipLaunchKernelGGL(group_gather_runs, dim3(grid_for(total)), dim3(256), 0, s, runs, n_runs, total);
  return hipGetLastError();
}

}  // namespace tnc
