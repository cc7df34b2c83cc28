// Gather + worker sum + error-feedback update of the compressor step (Eq. (5),
// Alg. 1's payload All-Reduce, Eq. (11b)).  With a non-null G the summed
// payload is also added into the node-summed tracker, G = fl(G + agg), at the
// same coordinates (the model step's view of the payload, Eq. (11c)).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "arc_device.h"
#include "arc_internal.h"

namespace arc {
namespace {

// Work item = one selected row x 4 columns (a row's last item may have
// fewer): for each worker in ascending order Delta = h - g, agg += Delta,
// g = g + Delta.  Bound by memory where many rows are kept and by the chain of
// dependent reads (bucket, row, values) where few are, so the values of WORKERS
// workers are requested together: 4 up to 8 workers (8 at a time were no faster
// with 8, and slower with 1: 68 against 56 us on per-tensor TinyLlama-1.1B,
// whose one worker's reads then held more registers than it used), 8 beyond
// (Rand-K steps, 256 workers, 45 rows of 1024 values kept: 182 us with 4, 144;
// 64 workers 116, 106).  Single columns go the same way: worker after worker and
// column after column, 256 workers' 1512 rows of 31 values took 521 us, now
// 135, 64 workers' 6048 rows 236 and 133.  16-byte accesses need only whole
// words, so rows, payload and G are taken as they lie; one value a lane where
// they were off 16 bytes, and one worker at a time, took 46.5 us on per-tensor
// CIFAR ResNet-18 (1.1e6 values kept, 4 workers), now 19.0.
constexpr int kFewWorkers = 8;

// COLS values from p (four or one), or, COLS = 0, its first ncols < 4 and the
// last of them again (loads without a branch, so that all of a batch are in
// flight together).
template <int COLS>
__device__ __forceinline__ float4 load_columns(const float* p, int ncols) {
  if constexpr (COLS == 4) return load_f4_words(p);
  if constexpr (COLS == 1) return make_float4(p[0], 0.f, 0.f, 0.f);
  return make_float4(p[0], p[ncols > 1 ? 1 : 0], p[ncols - 1], 0.f);
}

// The same values of v at out.
template <int COLS>
__device__ __forceinline__ void store_columns(float* out, float4 v, int ncols) {
  if constexpr (COLS == 4) {
    store_f4_words(out, v);
  } else {
    out[0] = v.x;
    if (COLS == 0 && ncols > 1) out[1] = v.y;
    if (COLS == 0 && ncols > 2) out[2] = v.z;
  }
}

// The item's columns at coordinate e of every worker's vector (COLS of them, or
// ncols of a row's end); returns their worker sum, +0 in columns past them.
template <int WORKERS, int COLS>
__device__ __forceinline__ float4 move_some(const float* __restrict__ h, float* __restrict__ g,
                                            float* __restrict__ G, int64_t e, int ncols,
                                            int64_t d, int32_t N) {
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto batch = [&](int32_t i0, auto full) __attribute__((always_inline)) {
    float4 hv[WORKERS], gv[WORKERS];
#pragma unroll
    for (int u = 0; u < WORKERS; ++u) {
      if (full.value || i0 + u < N) {
        const int64_t at = (int64_t)(i0 + u) * d + e;
        hv[u] = load_columns<COLS>(h + at, ncols);
        gv[u] = load_columns<COLS>(g + at, ncols);
      }
    }
#pragma unroll
    for (int u = 0; u < WORKERS; ++u) {
      if (full.value || i0 + u < N) {
        const float4 dl = make_float4(hv[u].x - gv[u].x, hv[u].y - gv[u].y, hv[u].z - gv[u].z,
                                      hv[u].w - gv[u].w);
        if (i0 + u == 0) {
          acc = dl;
        } else {
          acc.x = acc.x + dl.x;
          acc.y = acc.y + dl.y;
          acc.z = acc.z + dl.z;
          acc.w = acc.w + dl.w;
        }
        store_columns<COLS>(g + (int64_t)(i0 + u) * d + e,
                             make_float4(gv[u].x + dl.x, gv[u].y + dl.y, gv[u].z + dl.z,
                                         gv[u].w + dl.w),
                             ncols);
      }
    }
  };
  int32_t i0 = 0;
  for (; i0 + WORKERS <= N; i0 += WORKERS) batch(i0, std::true_type{});
  if (i0 < N) batch(i0, std::false_type{});
  if (G) {
    const float4 Gv = load_columns<COLS>(G + e, ncols);
    store_columns<COLS>(
        G + e, make_float4(Gv.x + acc.x, Gv.y + acc.y, Gv.z + acc.z, Gv.w + acc.w), ncols);
  }
  if constexpr (COLS == 0)
    acc = make_float4(acc.x, ncols > 1 ? acc.y : 0.f, ncols > 2 ? acc.z : 0.f, 0.f);
  return acc;
}

// As above for 0 to 4 columns (none: +0, nothing moved).
template <int WORKERS>
__device__ __forceinline__ float4 move_columns(const float* __restrict__ h, float* __restrict__ g,
                                               float* __restrict__ G, int64_t e, int ncols,
                                               int64_t d, int32_t N) {
  if (ncols == 4) return move_some<WORKERS, 4>(h, g, G, e, ncols, d, N);
  if (ncols == 1) return move_some<WORKERS, 1>(h, g, G, e, ncols, d, N);
  if (ncols > 1) return move_some<WORKERS, 0>(h, g, G, e, ncols, d, N);
  return make_float4(0.f, 0.f, 0.f, 0.f);
}

// The first ncols (1 to 4) of v at out.
__device__ __forceinline__ void store_item(float* out, float4 v, int ncols) {
  if (ncols == 4)
    store_columns<4>(out, v, ncols);
  else
    store_columns<0>(out, v, ncols);
}

// Single view: rows of n values, columns past d give agg = +0.  A row's items
// are its first `quads` groups of four columns and its other columns one by one:
// all of them where a width that is not a multiple of four is narrow, as quads
// and single columns take turns in every wave.  Step us of Rand-K, 4.0e7
// binary32 values, 30% kept, quads / single columns: one worker 19 values 187 /
// 195, 33 156 / 174, 257 139 / 165; 4 workers 19 164 / 150, 33 151 / 143, 130
// 134 / 136, 257 132 / 135; 8 workers 7 213 / 168, 63 145 / 137, 257 122 / 121.
// (A row's last columns as one item: 4 workers 7 values 309, 19 225.)
template <int WORKERS>
__global__ void __launch_bounds__(256)
gather_update_rows_kernel(const float* __restrict__ h, float* __restrict__ g,
                          const int32_t* __restrict__ idx, float* __restrict__ agg,
                          float* __restrict__ G, int64_t K_total, int64_t d, int64_t n,
                          int64_t quads, int64_t m, int32_t N) {
  const int64_t per_row = n - 3 * quads;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= K_total * per_row) return;
  const int64_t q = tid / per_row;
  const int64_t item = tid - q * per_row;
  const int64_t col = item < quads ? item * 4 : item + 3 * quads;
  const int64_t p = idx[q];
  const int width = item < quads ? 4 : 1;
  const int64_t e = p * n + col;
  int live = 0;  // columns that exist (none where idx holds no row: the state stays alone)
  if (p >= 0 && p < m && e < d) live = (int)(d - e < width ? d - e : width);
  const float4 acc = move_columns<WORKERS>(h, g, G, e, live, d, N);
  store_item(agg + q * n + col, acc, width);
}

// ---------------------------------------------------------------------------
// Per-tensor mode: items are numbered tensor after tensor
// (GatherBucket::work_off); a thread finds its tensor by binary search, over
// an LDS copy of the offsets where they fit, so that the search is one read
// of global memory deep.
// ---------------------------------------------------------------------------
constexpr int kSearchBuckets = 1024;

template <int WORKERS>
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
  const float4 acc = move_columns<WORKERS>(h, g, G, e, ncols, d, N);
  store_item(agg + bk.agg_off + q * bk.cols + col, acc, ncols);
}

}  // namespace

namespace {
bool aligned16(const void* a, const void* b, const void* c, const void* d) {
  return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) |
           reinterpret_cast<uintptr_t>(c) | reinterpret_cast<uintptr_t>(d)) & 15u) == 0;
}
}  // namespace

hipError_t launch_gather_update(const float* h, float* g,
                                const int32_t* idx, float* agg, float* G, int64_t K_total,
                                int64_t d, int64_t n, int64_t m, int32_t N,
                                hipStream_t stream) {
  if (K_total <= 0) return hipSuccess;
  // (Quads off 16 bytes pay from two a row on: 3124 rows of 4 values, 16 workers,
  // 88 us a step, single columns 74.)
  const bool whole = n % 4 == 0 && (n > 4 || (d % 4 == 0 && aligned16(h, g, agg, G)));
  const int64_t quads = whole || n >= (N == 1 ? 12 : 128) ? n / 4 : 0;
  const auto kernel = N <= kFewWorkers ? gather_update_rows_kernel<4>
                      : gather_update_rows_kernel<8>;
  hipLaunchKernelGGL(kernel, dim3(blocks_for(K_total * (n - 3 * quads), 256)), dim3(256), 0,
                     stream, h, g, idx, agg, G, K_total, d, n, quads, m, N);
  return hipGetLastError();
}

hipError_t launch_gather_update_tensors(const float* h, float* g,
                                        const int32_t* idx, float* agg, float* G,
                                        const GatherBucket* buckets, int32_t nb,
                                        int64_t total_work, int64_t d, int32_t N,
                                        hipStream_t stream) {
  if (total_work <= 0) return hipSuccess;
  const auto kernel =
      N <= kFewWorkers ? gather_update_tensors_kernel<4> : gather_update_tensors_kernel<8>;
  hipLaunchKernelGGL(kernel, dim3(blocks_for(total_work, 256)), dim3(256), 0, stream, h, g, idx,
                     agg, G, buckets, nb, total_work, d, N);
  return hipGetLastError();
}

}  // namespace arc
