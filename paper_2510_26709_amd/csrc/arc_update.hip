// Gather + worker sum + error-feedback update of the compressor step (Eq. (5),
// Alg. 1's payload All-Reduce, Eq. (11b)).  With a non-null G the summed
// payload is also added into the node-summed tracker, G = fl(G + agg), at the
// same coordinates (the model step's view of the payload, Eq. (11c)).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "arc_device.h"
#include "arc_internal.h"

namespace arc {
namespace {

// Work item = one selected row x 4 columns (a row's last item may have
// fewer): for each worker in ascending order Delta = h - g, agg += Delta,
// g = g + Delta.  Bound by memory where many rows are kept and by the chain of
// dependent reads (bucket, row, values) where few are, so the values of up to
// kMaxUnrolledWorkers workers are requested together (8 at a time instead of
// 4 were no faster with 8 workers, and slower with 1: 68 against 56 us on
// per-tensor TinyLlama-1.1B, whose one worker's reads then held more
// registers than it used).  16-byte accesses need only whole words, so rows,
// payload and G are taken as they lie; one value a lane where they were off
// 16 bytes, and one worker at a time, took 46.5 us on per-tensor CIFAR
// ResNet-18 (1.1e6 values kept, 4 workers), now 19.0.
constexpr int kMaxUnrolledWorkers = 4;

// The item's ncols columns at coordinate e of every worker's vector; returns
// their worker sum, +0 in columns at or past ncols.
__device__ __forceinline__ float4 move_columns(const float* __restrict__ h, float* __restrict__ g,
                                               float* __restrict__ G, int64_t e, int ncols,
                                               int64_t d, int32_t N) {
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (ncols == 4) {
    for (int32_t i0 = 0; i0 < N; i0 += kMaxUnrolledWorkers) {
      const int32_t cnt = N - i0 < kMaxUnrolledWorkers ? N - i0 : kMaxUnrolledWorkers;
      float4 hv[kMaxUnrolledWorkers], gv[kMaxUnrolledWorkers];
#pragma unroll
      for (int u = 0; u < kMaxUnrolledWorkers; ++u) {
        if (u < cnt) {
          const int64_t at = (int64_t)(i0 + u) * d + e;
          hv[u] = load_f4_words(h + at);
          gv[u] = load_f4_words(g + at);
        }
      }
#pragma unroll
      for (int u = 0; u < kMaxUnrolledWorkers; ++u) {
        if (u < cnt) {
          const float4 dl = make_float4(hv[u].x - gv[u].x, hv[u].y - gv[u].y,
                                        hv[u].z - gv[u].z, hv[u].w - gv[u].w);
          if (i0 + u == 0) {
            acc = dl;
          } else {
            acc.x = acc.x + dl.x;
            acc.y = acc.y + dl.y;
            acc.z = acc.z + dl.z;
            acc.w = acc.w + dl.w;
          }
          store_f4_words(g + (int64_t)(i0 + u) * d + e,
                         make_float4(gv[u].x + dl.x, gv[u].y + dl.y, gv[u].z + dl.z,
                                     gv[u].w + dl.w));
        }
      }
    }
    if (G) {
      const float4 Gv = load_f4_words(G + e);
      store_f4_words(G + e, make_float4(Gv.x + acc.x, Gv.y + acc.y, Gv.z + acc.z, Gv.w + acc.w));
    }
  } else {
    float a4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jj = 0; jj < 3; ++jj) {
      if (jj < ncols) {
        for (int32_t i = 0; i < N; ++i) {
          const int64_t at = (int64_t)i * d + e + jj;
          const float dl = h[at] - g[at];
          a4[jj] = (i == 0) ? dl : a4[jj] + dl;
          g[at] = g[at] + dl;
        }
        if (G) G[e + jj] = G[e + jj] + a4[jj];
      }
    }
    acc = make_float4(a4[0], a4[1], a4[2], 0.f);
  }
  return acc;
}

// The first ncols of v at out.
__device__ __forceinline__ void store_columns(float* out, float4 v, int ncols) {
  if (ncols == 4) {
    store_f4_words(out, v);
  } else {
    const float a4[3] = {v.x, v.y, v.z};
#pragma unroll
    for (int jj = 0; jj < 3; ++jj)
      if (jj < ncols) out[jj] = a4[jj];
  }
}

// Single view: rows of n values, columns past d give agg = +0.
__global__ void __launch_bounds__(256)
gather_update_rows_kernel(const float* __restrict__ h, float* __restrict__ g,
                          const int32_t* __restrict__ idx, float* __restrict__ agg,
                          float* __restrict__ G, int64_t K_total, int64_t d, int64_t n,
                          int64_t m, int32_t N) {
  const int64_t per_row = (n + 3) / 4;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= K_total * per_row) return;
  const int64_t q = tid / per_row;
  const int64_t col = (tid - q * per_row) * 4;
  const int64_t p = idx[q];
  const int width = (int)(n - col < 4 ? n - col : 4);
  const int64_t e = p * n + col;
  int live = 0;  // columns that exist (none where idx holds no row: the state stays alone)
  if (p >= 0 && p < m && e < d) live = (int)(d - e < width ? d - e : width);
  const float4 acc = move_columns(h, g, G, e, live, d, N);
  store_columns(agg + q * n + col, acc, width);
}

// ---------------------------------------------------------------------------
// Per-tensor mode: items are numbered tensor after tensor
// (GatherBucket::work_off); a thread finds its tensor by binary search, over
// an LDS copy of the offsets where they fit, so that the search is one read
// of global memory deep.
// ---------------------------------------------------------------------------
constexpr int kSearchBuckets = 1024;

__global__ void __launch_bounds__(256)
gather_update_tensors_kernel(const float* __restrict__ h, float* __restrict__ g,
                             const int32_t* __restrict__ idx,
                             float* __restrict__ agg, float* __restrict__ G,
                             const GatherBucket* __restrict__ buckets,
                             int32_t nb, int64_t total_work, int64_t d,
                             int32_t N) {
  __shared__ int64_t first[kSearchBuckets];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool in_lds = nb <= kSearchBuckets;
  if (in_lds) {
    for (int32_t b = threadIdx.x; b < nb; b += blockDim.x) first[b] = buckets[b].work_off;
    __syncthreads();
  }
  if (w >= total_work) return;
  int32_t lo = 0, hi = nb;  // last bucket whose work_off <= w
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if ((in_lds ? first[mid] : buckets[mid].work_off) <= w) lo = mid; else hi = mid;
  }
  const GatherBucket bk = buckets[lo];
  const int64_t per_row = (bk.cols + 3) / 4;
  const int64_t item = w - bk.work_off;
  const int64_t q = item / per_row;
  const int64_t col = (item - q * per_row) * 4;
  const int64_t p = (int64_t)idx[bk.out_off + q] - bk.row0;
  const int ncols = (int)(bk.cols - col < 4 ? bk.cols - col : 4);
  const int64_t e = bk.elem_off + p * bk.cols + col;
  // Only rows of this tensor; the bounds keep a broken index from touching
  // memory outside the vectors.
  if (p < 0 || p >= bk.rows || q >= bk.k || e + ncols > d) return;
  const float4 acc = move_columns(h, g, G, e, ncols, d, N);
  store_columns(agg + bk.agg_off + q * bk.cols + col, acc, ncols);
}

}  // namespace

hipError_t launch_gather_update(const float* h, float* g,
                                const int32_t* idx, float* agg, float* G, int64_t K_total,
                                int64_t d, int64_t n, int64_t m, int32_t N,
                                hipStream_t stream) {
  if (K_total <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_update_rows_kernel, dim3(blocks_for(K_total * ((n + 3) / 4), 256)),
                     dim3(256), 0, stream, h, g, idx, agg, G, K_total, d, n, m, N);
  return hipGetLastError();
}

hipError_t launch_gather_update_tensors(const float* h, float* g,
                                        const int32_t* idx, float* agg, float* G,
                                        const GatherBucket* buckets, int32_t nb,
                                        int64_t total_work, int64_t d, int32_t N,
                                        hipStream_t stream) {
  if (total_work <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_update_tensors_kernel, dim3(blocks_for(total_work, 256)),
                     dim3(256), 0, stream, h, g, idx, agg, G, buckets, nb, total_work, d, N);
  return hipGetLastError();
}

}  // namespace arc
