// Streaming stage for narrow rows: EF21M momentum (11a), residual Delta = h_t
// - g_{t-1} and per-worker sketch of Alg. 1 (or Top-K's squared row norms), as
// the column-window kernels of arc_sketch.hip compute them, with the same
// bits, for groups of consecutive rows that one wave takes whole.
//
// A wave reads its rows as one span of memory, whatever their width: all of
// the span's loads are in flight together, every one of them covers whole
// 128-byte lines of h, and only the span's two ends are taken one value a
// lane.  Delta goes to LDS row by row, and each lane then runs its row's
// chains from there, in ascending column order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "arc_device.h"
#include "arc_internal.h"

namespace arc {
namespace {

constexpr uint32_t kDropOffset = 0x80000000u;  // beyond every resource here
// One wave per workgroup and (row group, worker), at the occupancy its LDS
// allows (6 per compute unit for rows of 512 values at r = 4).  Bound by HBM:
// a wave streams once and ends, so what hides its latency is other waves.
// Workgroups of 2 or 4 waves were 4% and 19% slower on ResNet-18 (a
// workgroup's LDS is held until its last wave ends), reservations that leave
// 3 to 5 waves per compute unit 0.5-12%, spans of half the size 3%.  Registers
// stay under half a SIMD's (two waves): at 258 instead of 233 the rows of 333
// values took 330 us instead of 303.  Short spans hold fewer loads and run more
// waves (LOADS, see span_loads).
// Step times (us), r = 4, the window kernels / this one.  4 workers of 2.0e7 + x
// binary32 values, so that each worker's base lies x values further past a line
// than the one before: rows of 100 values (x = 4) 413 / 267, 300 (8) 337 / 268,
// 512 (8) 280 / 270, 600 (4) 315 / 273, 640 (8) 281 / 265, 704 (8) 392 / 267; bf16
// 100 (8) 334 / 217, 512 (8) 236 / 220, 640 (8) 230 / 215.  ResNet-18 (8 workers
// of 1.2e7, 512-wide rows, x = 8) 322 / 301.  On the lines (x = 0) 512 258 / 269,
// 768 262 / 266, which keep the windows, as do the widths at odd multiples of 32
// and 64 that are slower there (704 273 / 262, 800 304 / 265).
template <int R, bool BF16, bool NORM, int LOADS>
__global__ void __launch_bounds__(kWave, LOADS == kMaxSpanLoads ? 2 : 4)
sketch_span_kernel(const void* __restrict__ grad, float* __restrict__ h,
                   const float* __restrict__ g, const float* __restrict__ V,
                   const RowGroup* __restrict__ groups, int64_t ngroups, float* __restrict__ S,
                   int64_t d, int64_t m, float eta, float a, int32_t flat, int32_t wave_floats) {
  extern __shared__ float4 lds[];
  const int lane = threadIdx.x;
  int32_t i;   // worker
  int64_t gi;  // row group within the worker's list
  if (flat) {
    const int64_t f = xcd_contiguous_block(blockIdx.x, gridDim.x);
    i = (int32_t)(f / ngroups);
    gi = f - (int64_t)i * ngroups;
  } else {
    i = blockIdx.y;
    gi = xcd_contiguous_block(blockIdx.x, gridDim.x);
  }
  const RowGroup grp = groups[gi];
  const int n = grp.cols, rows = grp.rows;
  const int E = rows * n;  // the span's values, at most kSpanValues
  const int pitch = span_pitch(n);
  float* tile = reinterpret_cast<float*>(lds);
  float* vt = tile + rows * pitch;

  // This width's V (n x R) straight to LDS, first of all, so that it is there
  // when the span's own loads have come.
  if constexpr (!NORM) {
    const buffer_rsrc rv = make_buffer(V + grp.v_off, (uint32_t)(n * R + 3) / 4u * 16u);
    for (int f0 = 0; f0 < n * R; f0 += 4 * kWave)
      buffer_load_lds_f4(rv, (uint32_t)(f0 + lane * 4) * 4u, vt + f0);
  }

  const int64_t wbase = (int64_t)i * d + grp.elem_off;
  // Values between the line's start and the span's, and the span's values
  // before the first whole 16 bytes of h and after the last.
  const int shift = (int)((reinterpret_cast<uintptr_t>(h + wbase) & 127u) / 4u);
  const int head = min((4 - (shift & 3)) & 3, E);
  const int tail = (E - head) & 3;
  const uint32_t quads_end = (uint32_t)(E - tail);
  // The resources of h and g end with the last whole quad and every quad's
  // offset is a 32-bit number, so the quads before the span (whose offsets
  // wrap) and past its last whole one lie outside: the hardware drops their
  // accesses without a select.
  const buffer_rsrc rh = make_buffer(h + wbase, quads_end * 4u);
  const buffer_rsrc rg = make_buffer(g + wbase, quads_end * 4u);
  // bf16: the resource starts and ends on whole words.
  const uint16_t* xb = static_cast<const uint16_t*>(grad) + wbase;
  const uint32_t x_odd = BF16 ? (uint32_t)(reinterpret_cast<uintptr_t>(xb) & 2u) / 2u : 0u;
  const buffer_rsrc rx =
      BF16 ? make_buffer(xb - x_odd, ((uint32_t)E * 2u + 2u * x_odd + 3u) & ~3u)
           : make_buffer(static_cast<const float*>(grad) + wbase, quads_end * 4u);
  // Every quad starts head values past a multiple of 4 in the span, so all of
  // them start in the same half of a bf16 word.
  const bool half = BF16 && ((head + x_odd) & 1u) != 0;

  float4 xv[LOADS], hv[LOADS], gv[LOADS];
  // Load u's quad starts at span position at0 + u * 4 * kWave.
  int at0 = lane * 4 - shift;
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int at = at0 + u * 4 * kWave;
    const uint32_t o = (uint32_t)at * 4u;
    if constexpr (BF16) {
      const uint32_t b = (uint32_t)(at + (int)x_odd) * 2u;
      const uint2 w = buffer_load_u2<kCacheDefault>(rx, b & ~3u);
      const uint32_t w2 =
          buffer_load_u1<kCacheDefault>(rx, half ? (b & ~3u) + 8u : kDropOffset);
      xv[u] = make_float4(__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w2), 0.f);
    } else {
      xv[u] = buffer_load_f4<kCacheNonTemporal>(rx, o);
    }
    hv[u] = buffer_load_f4<kCacheNonTemporal>(rh, o);
    gv[u] = buffer_load_f4<kCacheNonTemporal>(rg, o);
  }
  // The ends, one value a lane: lanes 0-3 the head, 4-7 the tail.
  int end_at = lane < 4 ? lane : E - tail + lane - 4;
  const bool end_ok = lane < 4 ? lane < head : lane - 4 < tail;
  float end_x = 0.f, end_h = 0.f, end_g = 0.f;
  const buffer_rsrc rh_all = make_buffer(h + wbase, (uint32_t)E * 4u);
  if (head + tail > 0) {
    const uint32_t o = end_ok ? (uint32_t)end_at * 4u : kDropOffset;
    if constexpr (BF16)
      end_x = __uint_as_float(buffer_load_u16<kCacheDefault>(rx, o / 2 + 2 * x_odd) << 16);
    else
      end_x = buffer_load_f1<kCacheDefault>(
          make_buffer(static_cast<const float*>(grad) + wbase, (uint32_t)E * 4u), o);
    end_h = buffer_load_f1<kCacheDefault>(rh_all, o);
    end_g = buffer_load_f1<kCacheDefault>(make_buffer(g + wbase, (uint32_t)E * 4u), o);
  }

  // LDS word of span position p: row p / n, padded rows.  The product is
  // within 2^-11 / n of (p + 1/2) / n (p < 2^12), which lies at least
  // 1 / (2n) from a whole number.
  const float inv_n = 1.0f / (float)n;
  const int pad = pitch - n;
  auto row_of = [&](int p) { return (int)(((float)p + 0.5f) * inv_n); };
  // No branch per load: lanes without a whole quad park their Delta past V.
  const int trash = wave_floats - 4;
  asm("" : "+v"(at0));  // the loads' offsets are not kept for the stores
  auto consume = [&](int u, auto quads) __attribute__((always_inline)) {
    const int at = at0 + u * 4 * kWave;
    const bool whole = (uint32_t)at < quads_end;
    float4 x4 = xv[u];
    if constexpr (BF16) {
      const uint32_t w0 = __float_as_uint(xv[u].x), w1 = __float_as_uint(xv[u].y);
      const uint32_t bits = half ? 16u : 0u;
      const uint32_t v0 = __builtin_amdgcn_alignbit(w1, w0, bits);
      const uint32_t v1 = __builtin_amdgcn_alignbit(__float_as_uint(xv[u].z), w1, bits);
      x4 = make_float4(bf16_lo(v0), bf16_hi(v0), bf16_lo(v1), bf16_hi(v1));
    }
    float4 hn;
    hn.x = fmaf(eta, x4.x, a * hv[u].x);
    hn.y = fmaf(eta, x4.y, a * hv[u].y);
    hn.z = fmaf(eta, x4.z, a * hv[u].z);
    hn.w = fmaf(eta, x4.w, a * hv[u].w);
    buffer_store_f4<kCacheStreamDevice>(rh, (uint32_t)at * 4u, hn);
    const float4 dl =
        make_float4(hn.x - gv[u].x, hn.y - gv[u].y, hn.z - gv[u].z, hn.w - gv[u].w);
    const int row = row_of(at);
    const int w = at + __mul24(row, pad);
    if constexpr (decltype(quads)::value) {
      *reinterpret_cast<float4*>(tile + (whole ? w : trash)) = dl;
    } else {
      // The quad's values from the row's end on lie in the next row (rows
      // have at least 4 values).
      const int left = whole ? __mul24(row, n) + n - at : 4;
      float* to = tile + (whole ? w : trash);
      to[0] = dl.x;
      to[left > 1 ? 1 : 1 + pad] = dl.y;
      to[left > 2 ? 2 : 2 + pad] = dl.z;
      to[left > 3 ? 3 : 3 + pad] = dl.w;
    }
  };
  if (head == 0 && n % 4 == 0) {  // no quad crosses a row's end
#pragma unroll
    for (int u = 0; u < LOADS; ++u) consume(u, std::true_type{});
  } else {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) consume(u, std::false_type{});
  }
  if (head + tail > 0 && end_ok && lane < 8) {
    const float hn = fmaf(eta, end_x, a * end_h);
    buffer_store_f1<kCacheDefault>(rh_all, (uint32_t)end_at * 4u, hn);
    tile[end_at + row_of(end_at) * pad] = hn - end_g;
  }
  wave_vmem_fence();  // V's loads to LDS
  wave_lds_fence();

  // Chains: lane row + q * rows runs row `row` against columns [q * KPL,
  // (q + 1) * KPL) of V (or its squares, NORM).
  auto chains = [&](auto per_lane) __attribute__((always_inline)) {
    constexpr int KPL = decltype(per_lane)::value;
    int row = lane, q = 0;
#pragma unroll
    for (int u = 1; u < R / KPL; ++u)
      if (row >= rows) {
        row -= rows;
        ++q;
      }
    const bool live = row < rows;
    const float* my_row = tile + (live ? row : 0) * pitch;
    const float* my_v = vt + q * KPL;
    float s[KPL];
#pragma unroll
    for (int k = 0; k < KPL; ++k) s[k] = 0.0f;
    auto term = [&](float dv, int j) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < KPL; ++k) s[k] = fmaf(dv, NORM ? dv : my_v[j * R + k], s[k]);
    };
    int j = 0;
    auto quad = [&](int at) __attribute__((always_inline)) {
      const float4 dv = *reinterpret_cast<const float4*>(my_row + at);
      term(dv.x, at);
      term(dv.y, at + 1);
      term(dv.z, at + 2);
      term(dv.w, at + 3);
    };
    if constexpr (KPL == 1 && !NORM) {
#pragma unroll 8
      for (; j + 4 <= n; j += 4) quad(j);
    } else if constexpr (KPL < R) {
#pragma unroll 4
      for (; j + 4 <= n; j += 4) quad(j);
    } else {
#pragma unroll 2
      for (; j + 4 <= n; j += 4) quad(j);
    }
    for (; j < n; ++j) term(my_row[j], j);
    if (live) {
      float* out = S + ((int64_t)i * m + grp.row0 + row) * R + q * KPL;
#pragma unroll
      for (int k = 0; k < KPL; ++k) out[k] = s[k];
    }
  };
  // As few columns a lane as the rows leave lanes for: with all eight chains of
  // nine rows on nine lanes, rows of 416 values took 362 us a step (r = 8,
  // 8.0e7 binary32 values; the window kernel 289), with two a lane 280.  Short
  // spans have all 64 rows.
  if (!NORM && rows * R <= kWave)
    chains(std::integral_constant<int, 1>{});
  else if (LOADS == kMaxSpanLoads && R >= 4 && rows * (R / 2) <= kWave)
    chains(std::integral_constant<int, R >= 4 ? 2 : R>{});
  else if (LOADS == kMaxSpanLoads && R >= 8 && rows * (R / 4) <= kWave)
    chains(std::integral_constant<int, R >= 8 ? 4 : R>{});
  else
    chains(std::integral_constant<int, R>{});
}

template <int R, bool BF16, bool NORM, int LOADS>
void launch_span_loads(const void* grad, float* h, const float* g, const float* V,
                       const RowGroup* groups, int64_t ngroups, float* S, int64_t d, int64_t m,
                       int32_t N, float eta, float a, int32_t wave_floats, hipStream_t stream) {
  // The grid is one-dimensional for multiples of 8 workers, as the window
  // kernels' is.
  const bool flat = N % 8 == 0 && ngroups * N <= INT32_MAX;
  const unsigned n = (unsigned)ngroups;
  hipLaunchKernelGGL((sketch_span_kernel<R, BF16, NORM, LOADS>),
                     flat ? dim3(n * (unsigned)N) : dim3(n, (unsigned)N), dim3(kWave),
                     (size_t)wave_floats * sizeof(float), stream, grad, h, g, V, groups, ngroups,
                     S, d, m, eta, a, flat ? 1 : 0, wave_floats);
}

template <int R, bool BF16, bool NORM, typename... Args>
void launch_span(int32_t wave_values, Args... args) {
  switch (span_loads(wave_values)) {
    case 3: launch_span_loads<R, BF16, NORM, 3>(args...); break;
    case 5: launch_span_loads<R, BF16, NORM, 5>(args...); break;
    case 7: launch_span_loads<R, BF16, NORM, 7>(args...); break;
    default: launch_span_loads<R, BF16, NORM, kMaxSpanLoads>(args...);
  }
}

}  // namespace

hipError_t launch_sketch_span(const void* grad, int32_t grad_bf16, float* h, const float* g,
                              const float* V, const RowGroup* groups, int64_t ngroups, float* S,
                              int64_t d, int64_t m, int32_t N, int32_t r, float eta, float a,
                              bool norm, int32_t wave_floats, int32_t wave_values,
                              hipStream_t stream) {
  if (ngroups <= 0) return hipSuccess;
#define ARC_SPAN(RR, NN)                                                                      \
  if (grad_bf16)                                                                              \
    launch_span<RR, true, NN>(wave_values, grad, h, g, V, groups, ngroups, S, d, m, N, eta,   \
                              a, wave_floats, stream);                                        \
  else                                                                                        \
    launch_span<RR, false, NN>(wave_values, grad, h, g, V, groups, ngroups, S, d, m, N, eta,  \
                               a, wave_floats, stream)
  if (norm) {
    ARC_SPAN(1, true);
    return hipGetLastError();
  }
  switch (r) {
    case 1: ARC_SPAN(1, false); break;
    case 2: ARC_SPAN(2, false); break;
    case 4: ARC_SPAN(4, false); break;
    case 8: ARC_SPAN(8, false); break;
    default: return hipErrorInvalidValue;
  }
#undef ARC_SPAN
  return hipGetLastError();
}

}  // namespace arc
