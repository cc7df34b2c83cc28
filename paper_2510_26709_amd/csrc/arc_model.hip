// Model step around the compressor: the dense (identity-compressor) step of
// the warm-up iterations, and the x update of Eq. (11c) with the optimisers of
// the experiments (SGD, heavy-ball momentum SGD, Adam).
//
// The nodes keep G = sum_i g^(i) by adding each step's summed payload (the
// gather kernels do that at the selected coordinates; the dense step here at
// all of them).  Every operation is binary32 and correctly rounded, in the
// order documented in libarctopk.h, so that the result is bit-exact against a
// sequential evaluation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "arc_device.h"
#include "arc_internal.h"

namespace arc {
namespace {

// ---------------------------------------------------------------------------
// x update of one coordinate (division and sqrtf correctly rounded: the
// library is built with -fhip-fp32-correctly-rounded-divide-sqrt; the
// __fdiv_rn / __fsqrt_rn intrinsics are not used, as __fsqrt_rn maps to the
// native approximate square root): dir = fmaf(wd, x, G / N), then
//   SGD:  x = fmaf(-lr, dir, x)
//   MSGD: m = fmaf(beta, m, dir);  x = fmaf(-lr, m, x)
//   Adam: m = fmaf(beta1, m, fl((1-beta1) dir));  v = fmaf(beta2, v, fl((1-beta2) fl(dir dir)));
//         x = fmaf(-lr, fl(fl(m / c1) / fl(sqrt(fl(v / c2)) + eps)), x)
// HBM per coordinate: SGD 12 bytes, MSGD 20, Adam 28.
// ---------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ void update_one(const OptimizerArgs& o, float Gi, float& x, float& m,
                                           float& v) {
  const float dir = fmaf(o.weight_decay, x, Gi / o.fN);
  if constexpr (KIND == 0) {
    x = fmaf(o.neg_lr, dir, x);
  } else if constexpr (KIND == 1) {
    m = fmaf(o.momentum, m, dir);
    x = fmaf(o.neg_lr, m, x);
  } else {
    m = fmaf(o.beta1, m, o.one_minus_beta1 * dir);
    v = fmaf(o.beta2, v, o.one_minus_beta2 * (dir * dir));
    const float mh = m / o.c1, vh = v / o.c2;
    const float step = mh / (sqrtf(vh) + o.eps);
    x = fmaf(o.neg_lr, step, x);
  }
}

// ---------------------------------------------------------------------------
// Dense step, per coordinate e: for each worker in ascending order
//   h_i = fmaf(eta, grad_i, fl(a * h_i)),  Delta_i = h_i - g_i,
//   acc = Delta_0 + Delta_1 + ...,  g_i = g_i + Delta_i;
// then G = G + acc, and in the vectorised kernel the x update from that G.
// HBM per coordinate: N * (b_g + 16) + 8 bytes, and the update's without its
// read of G.  Bound by HBM.  Four workers' values are requested together, and
// at most two workgroups run per compute unit: with 3N + 4 arrays streamed
// side by side, fewer waves keep fewer DRAM rows open.  GPT-2 small, 4 bf16
// workers, Adam, step ms: dense step and update as two passes, one worker at a
// time, 2.45-2.53; one pass at the hardware's occupancy 2.44-2.48, at 4 / 3 /
// 2 workgroups per compute unit 2.38 / 2.32 / 2.27.  2.0e8 bf16 coordinates of
// one worker, Adam, 1.87 -> 1.74; 4.0e7 binary32 of 8 workers, heavy ball,
// 1.40 -> 1.38.
// ---------------------------------------------------------------------------
// Four values on 16 bytes, or (W) at any word.
template <bool W>
__device__ __forceinline__ float4 load4(const float* p) {
  if constexpr (W) return load_f4_words(p);
  return stream_load(reinterpret_cast<const float4*>(p));
}
template <bool W>
__device__ __forceinline__ void store4(float* p, float4 v) {
  if constexpr (W)
    store_f4_words(p, v);
  else
    stream_store(reinterpret_cast<float4*>(p), v);
}
template <bool BF16>
__device__ __forceinline__ float4 load_grad4(const void* grad, int64_t at) {
  if constexpr (BF16) {
    const uint2 w = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(grad) + at);
    return make_float4(bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y));
  } else {
    return stream_load(reinterpret_cast<const float4*>(static_cast<const float*>(grad) + at));
  }
}

constexpr int kDenseWorkers = 4;

template <bool BF16, int KIND, bool W>
__global__ void __launch_bounds__(256)
dense_model_vec_kernel(const void* __restrict__ grad, float* __restrict__ h,
                       float* __restrict__ g, float* __restrict__ G, OptimizerArgs o,
                       float* __restrict__ x, float* __restrict__ m, float* __restrict__ v,
                       int64_t d, int32_t N, float eta, float a) {
  const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (e >= d) return;
  float4 Gv = load4<W>(G + e);
  float4 xv = load4<W>(x + e);
  float4 mv = make_float4(0.f, 0.f, 0.f, 0.f), vv = mv, acc = mv;
  if constexpr (KIND >= 1) mv = load4<W>(m + e);
  if constexpr (KIND == 2) vv = load4<W>(v + e);
  for (int32_t i0 = 0; i0 < N; i0 += kDenseWorkers) {
    float4 gr[kDenseWorkers], hv[kDenseWorkers], gv[kDenseWorkers];
#pragma unroll
    for (int u = 0; u < kDenseWorkers; ++u) {
      if (i0 + u < N) {
        const int64_t at = (int64_t)(i0 + u) * d + e;
        gr[u] = load_grad4<BF16>(grad, at);
        hv[u] = load4<false>(h + at);
        gv[u] = load4<false>(g + at);
      }
    }
#pragma unroll
    for (int u = 0; u < kDenseWorkers; ++u) {
      if (i0 + u < N) {
        const int64_t at = (int64_t)(i0 + u) * d + e;
        hv[u].x = fmaf(eta, gr[u].x, a * hv[u].x);
        hv[u].y = fmaf(eta, gr[u].y, a * hv[u].y);
        hv[u].z = fmaf(eta, gr[u].z, a * hv[u].z);
        hv[u].w = fmaf(eta, gr[u].w, a * hv[u].w);
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
        store4<false>(h + at, hv[u]);
        store4<false>(g + at, make_float4(gv[u].x + dl.x, gv[u].y + dl.y, gv[u].z + dl.z,
                                 gv[u].w + dl.w));
      }
    }
  }
  Gv.x = Gv.x + acc.x;
  Gv.y = Gv.y + acc.y;
  Gv.z = Gv.z + acc.z;
  Gv.w = Gv.w + acc.w;
  update_one<KIND>(o, Gv.x, xv.x, mv.x, vv.x);
  update_one<KIND>(o, Gv.y, xv.y, mv.y, vv.y);
  update_one<KIND>(o, Gv.z, xv.z, mv.z, vv.z);
  update_one<KIND>(o, Gv.w, xv.w, mv.w, vv.w);
  store4<W>(G + e, Gv);
  store4<W>(x + e, xv);
  if constexpr (KIND >= 1) store4<W>(m + e, mv);
  if constexpr (KIND == 2) store4<W>(v + e, vv);
}

__global__ void __launch_bounds__(256)
dense_step_scalar_kernel(const void* __restrict__ grad, int32_t grad_bf16,
                         float* __restrict__ h, float* __restrict__ g, float* __restrict__ G,
                         int64_t d, int32_t N, float eta, float a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= d) return;
  float acc = 0.0f;
  for (int32_t i = 0; i < N; ++i) {
    const int64_t at = (int64_t)i * d + e;
    const float x =
        grad_bf16 ? __uint_as_float((uint32_t)static_cast<const uint16_t*>(grad)[at] << 16)
                  : static_cast<const float*>(grad)[at];
    const float hn = fmaf(eta, x, a * h[at]);
    const float dl = hn - g[at];
    acc = (i == 0) ? dl : acc + dl;
    h[at] = hn;
    g[at] = g[at] + dl;
  }
  G[e] = G[e] + acc;
}

// Vectorised x update: one workgroup of 256 threads per tile of kOptTile
// coordinates, each thread kOptUnroll float4 of every array (all loads of a
// thread in flight together), through buffer resources that end with
// d's last whole quad: the hardware returns zero for loads past the end and
// drops those stores, so the last, partial tile needs no branch; the last
// d % 4 coordinates go one a thread.  Loads are non-temporal (every value is
// read once), stores non-temporal at device scope (read again only by later
// launches).  5.0e7 + 1 coordinates, against one a thread: SGD 245 -> 203 us a
// step, heavy ball 289 -> 271.  Adam over 1.1e9 coordinates (28 bytes each), three MI355X
// boxes, every variant in one process per box: one float4 per thread
// through plain pointers 5.66 / 4.91-4.93 / 5.37-5.39 ms; this tile (four
// float4 per thread, at most four workgroups per compute unit through the
// launch's LDS reservation) - / 4.83 / 5.44-5.46 ms; two float4 per thread
// through buffer resources 5.49 / 4.87 / 5.61-5.63 ms.  The spread between
// boxes (up to 12%) is larger than between shapes on one box (2-3%).
// Default-policy stores were 3-4% slower, default-policy loads 3-7%, and
// grid-stride loops over tiles 7-30%.
constexpr int kOptUnroll = 4;
constexpr int kOptTile = 256 * 4 * kOptUnroll;

template <int KIND>
__global__ void __launch_bounds__(256)
optimizer_vec_kernel(OptimizerArgs o, const float* __restrict__ G, float* __restrict__ x,
                     float* __restrict__ m, float* __restrict__ v, int64_t d) {
  const int64_t b0 = (int64_t)blockIdx.x * kOptTile;
  const int64_t left = d - b0;
  if (left <= kOptTile && (int64_t)threadIdx.x < (d & 3)) {
    const int64_t e = d - (d & 3) + threadIdx.x;
    float xe = x[e], me = 0.0f, ve = 0.0f;
    if constexpr (KIND >= 1) me = m[e];
    if constexpr (KIND == 2) ve = v[e];
    update_one<KIND>(o, G[e], xe, me, ve);
    x[e] = xe;
    if constexpr (KIND >= 1) m[e] = me;
    if constexpr (KIND == 2) v[e] = ve;
  }
  const uint32_t bytes = (uint32_t)(left < kOptTile ? left / 4 * 4 : kOptTile) * 4u;
  const buffer_rsrc rG = make_buffer(G + b0, bytes);
  const buffer_rsrc rx = make_buffer(x + b0, bytes);
  const buffer_rsrc rm = make_buffer(KIND >= 1 ? m + b0 : x + b0, bytes);
  const buffer_rsrc rv = make_buffer(KIND == 2 ? v + b0 : x + b0, bytes);
  float4 Gv[kOptUnroll], xv[kOptUnroll], mv[kOptUnroll], vv[kOptUnroll];
#pragma unroll
  for (int u = 0; u < kOptUnroll; ++u) {
    const uint32_t off = (uint32_t)(u * 1024 + threadIdx.x * 4) * 4u;
    Gv[u] = buffer_load_f4<kCacheNonTemporal>(rG, off);
    xv[u] = buffer_load_f4<kCacheNonTemporal>(rx, off);
    mv[u] = vv[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (KIND >= 1) mv[u] = buffer_load_f4<kCacheNonTemporal>(rm, off);
    if constexpr (KIND == 2) vv[u] = buffer_load_f4<kCacheNonTemporal>(rv, off);
  }
#pragma unroll
  for (int u = 0; u < kOptUnroll; ++u) {
    const uint32_t off = (uint32_t)(u * 1024 + threadIdx.x * 4) * 4u;
    update_one<KIND>(o, Gv[u].x, xv[u].x, mv[u].x, vv[u].x);
    update_one<KIND>(o, Gv[u].y, xv[u].y, mv[u].y, vv[u].y);
    update_one<KIND>(o, Gv[u].z, xv[u].z, mv[u].z, vv[u].z);
    update_one<KIND>(o, Gv[u].w, xv[u].w, mv[u].w, vv[u].w);
    buffer_store_f4<kCacheStreamDevice>(rx, off, xv[u]);
    if constexpr (KIND >= 1) buffer_store_f4<kCacheStreamDevice>(rm, off, mv[u]);
    if constexpr (KIND == 2) buffer_store_f4<kCacheStreamDevice>(rv, off, vv[u]);
  }
}

// One coordinate a thread, where an array is off 16 bytes (heavy ball, 2.0e7
// coordinates, 4 workers 327 us a step, in tiles 342; SGD 24e6 120 / 124) or d %
// 4 != 0.  Adam at such a d: the tiles above take as long at 5.0e7 coordinates
// (bf16 step 417 / 418 us) and 0.7 us longer at 3.0e5.  SGD and heavy ball: steps
// whose arrays fit the Infinity Cache, whose bandwidth the tiles' four
// workgroups a compute unit do not reach.  Step us, one a thread / tiles, binary32, steps on the same arrays:
// dense, one bf16 worker, 6.0e6 coordinates, heavy ball 46 / 54, SGD 39 / 46;
// 1.1e7 80 / 95 and 70 / 82; 2.4e7 (beyond the cache) 214 / 208 and 196 / 178;
// dense, 4 workers, 3.0e6 53 / 56, 6.0e6 (beyond) 116 / 106.
template <int KIND>
__global__ void __launch_bounds__(256)
optimizer_scalar_kernel(OptimizerArgs o, const float* __restrict__ G, float* __restrict__ x,
                        float* __restrict__ m, float* __restrict__ v, int64_t d) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= d) return;
  float xe = x[e], me = 0.0f, ve = 0.0f;
  if constexpr (KIND >= 1) me = m[e];
  if constexpr (KIND == 2) ve = v[e];
  update_one<KIND>(o, G[e], xe, me, ve);
  x[e] = xe;
  if constexpr (KIND >= 1) m[e] = me;
  if constexpr (KIND == 2) v[e] = ve;
}

}  // namespace

hipError_t launch_dense_step(const void* grad, int32_t grad_bf16, float* h, float* g, float* G,
                             int64_t d, int32_t N, float eta, float a, hipStream_t stream) {
  if (d <= 0) return hipSuccess;
  hipLaunchKernelGGL(dense_step_scalar_kernel, dim3(blocks_for(d, 256)), dim3(256), 0, stream,
                     grad, grad_bf16, h, g, G, d, N, eta, a);
  return hipGetLastError();
}

hipError_t launch_dense_model(bool aligned, bool cap, const OptimizerArgs& o, const void* grad,
                              int32_t grad_bf16, float* h, float* g, float* G, float* x, float* m,
                              float* v, int64_t d, int32_t N, float eta, float a,
                              hipStream_t stream) {
  if (d <= 0) return hipSuccess;
  const dim3 grid(blocks_for(d / 4, 256));
  const size_t lds = cap ? kDenseLdsCap : 0;
#define ARC_DENSE_W(BB, KK, WW)                                                                \
  hipLaunchKernelGGL((dense_model_vec_kernel<BB, KK, WW>), grid, dim3(256), lds, stream, grad, \
                     h, g, G, o, x, m, v, d, N, eta, a)
#define ARC_DENSE(KK)                     \
  if (grad_bf16) {                        \
    if (aligned)                          \
      ARC_DENSE_W(true, KK, false);       \
    else                                  \
      ARC_DENSE_W(true, KK, true);        \
  } else {                                \
    if (aligned)                          \
      ARC_DENSE_W(false, KK, false);      \
    else                                  \
      ARC_DENSE_W(false, KK, true);       \
  }                                       \
  break
  switch (o.kind) {
    case 0: ARC_DENSE(0);
    case 1: ARC_DENSE(1);
    case 2: ARC_DENSE(2);
    default: return hipErrorInvalidValue;
  }
#undef ARC_DENSE
#undef ARC_DENSE_W
  return hipGetLastError();
}

hipError_t launch_optimizer(bool aligned, bool cached, bool cap, const OptimizerArgs& o,
                            const float* G, float* x, float* m, float* v, int64_t d,
                            hipStream_t stream) {
  if (d <= 0) return hipSuccess;
  if (d > INT64_MAX - kOptTile) return hipErrorInvalidValue;
  const bool tiles = aligned && (d % 4 == 0 || (!cached && o.kind != 2));
  const dim3 grid(blocks_for(d, tiles ? kOptTile : 256));
  const size_t lds = tiles && cap ? kOptLdsCap : 0;
#define ARC_OPT(KK)                                                                     \
  hipLaunchKernelGGL(tiles ? optimizer_vec_kernel<KK> : optimizer_scalar_kernel<KK>, grid, \
                     dim3(256), lds, stream, o, G, x, m, v, d)
  switch (o.kind) {
    case 0: ARC_OPT(0); break;
    case 1: ARC_OPT(1); break;
    case 2: ARC_OPT(2); break;
    default: return hipErrorInvalidValue;
  }
#undef ARC_OPT
  return hipGetLastError();
}

}  // namespace arc
