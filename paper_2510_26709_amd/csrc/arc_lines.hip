// Streaming stage for wide rows off the 128-byte lines: EF21M momentum (11a),
// residual Delta = h_t - g_{t-1} and per-worker sketch of Alg. 1 (or Top-K's
// squared row norms), as the column-window kernels of arc_sketch.hip compute
// them, with the same bits.
//
// A wave streams groups of kLineRows rows a chunk of 256 columns at a time,
// one row per load instruction, and every row's windows start on that row's
// own 128-byte lines, wherever it lies: a load or store never shares a line
// with another one, and only a row's first and last values (fewer than four
// at either end) are taken one value a lane.  Delta is parked in LDS by
// column, so the chains run over the same columns of every row, kLineLag
// columns (one line) behind the windows; the columns a chunk's chains have
// not reached are carried to the front of the next one.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "arc_device.h"
#include "arc_internal.h"

namespace arc {
namespace {

constexpr uint32_t kDropOffset = 0x80000000u;  // beyond every resource here
constexpr int kCols = 4 * kWave;               // columns of a chunk
constexpr int kLineLag = 32;                   // values of a line
// LDS floats from one row to the next: a chunk and the lag, and one float4 to
// spread the rows over the banks.
constexpr int kPitch = kCols + kLineLag + 4;

// V's columns of a chunk in LDS, transposed ([k][column]) with a pitch that
// puts the R columns in distinct banks where the lanes take one chain each
// (8 rows x R chains on 64 lanes: always, for R <= 8).
template <int R, bool NORM>
constexpr int slice_floats() { return NORM ? 0 : R * (kCols + 4); }
template <int R, bool NORM>
constexpr int wave_f4() { return (kLineRows * kPitch + slice_floats<R, NORM>()) / 4; }

// Workgroups of four waves, one (row group, worker) each, at the hardware's
// occupancy.  Bound by HBM.  Step times (us), 4 workers of 2.0e7 values, the
// window kernels on the rows as they lie / this one: rows of 1001 values
// binary32 314 / 281, bf16 267 / 229; 1000 308 / 274; 3001 316 / 286, bf16
// 273 / 231; 2048 at an odd base 298 / 278, bf16 249 / 222; per-tensor CIFAR
// ResNet-18 (rows of 576 to 4608 values, bases 8 bytes off 16) 256 / 242.  One
// workgroup per compute unit: equal on binary32, 3-6% slower on bf16 rows
// and on that network (249); two-wave workgroups, one per compute unit: 5%
// faster on rows of 8101 binary32 values, 2-40% slower elsewhere.  Where all
// rows start the same distance past a line, on 16 bytes, the window kernels'
// common shift does as well or better (2048 values: 252 / 271) and they
// keep them.
constexpr int kLineWaves = 4;

template <int R, bool BF16, bool NORM>
__global__ void __launch_bounds__(kLineWaves * kWave)
sketch_lines_kernel(const void* __restrict__ grad, float* __restrict__ h,
                    const float* __restrict__ g, const float* __restrict__ V,
                    const RowGroup* __restrict__ groups, int64_t ngroups, float* __restrict__ S,
                    int64_t d, int64_t m, float eta, float a, int32_t flat) {
  static_assert(kLineRows * R <= kWave, "one chain per lane");
  __shared__ float4 lds[kLineWaves][wave_f4<R, NORM>()];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int32_t i;   // worker
  int64_t gb;  // block of row groups within the worker's list
  if (flat) {
    const int64_t nbx = (ngroups + kLineWaves - 1) / kLineWaves;
    const int64_t f = xcd_contiguous_block(blockIdx.x, gridDim.x);
    i = (int32_t)(f / nbx);
    gb = f - (int64_t)i * nbx;
  } else {
    i = blockIdx.y;
    gb = xcd_contiguous_block(blockIdx.x, gridDim.x);
  }
  const int64_t gi = gb * kLineWaves + wave;
  if (gi >= ngroups) return;  // whole wave; no block barrier follows
  const RowGroup grp = groups[gi];
  const int n = grp.cols, rows = grp.rows;
  const uint32_t row_step = (uint32_t)grp.stride * (uint32_t)n;  // values from row to row
  float* tile = reinterpret_cast<float*>(lds[wave]);
  float* vt = tile + kLineRows * kPitch;
  V += grp.v_off;

  const int64_t wbase = (int64_t)i * d + grp.elem_off;
  const uint32_t bytes = ((uint32_t)(rows - 1) * row_step + (uint32_t)n) * 4u;
  const buffer_rsrc rh = make_buffer(h + wbase, bytes);
  const buffer_rsrc rg = make_buffer(g + wbase, bytes);
  // bf16: the resource starts and ends on whole words.
  const uint16_t* xb = static_cast<const uint16_t*>(grad) + wbase;
  const uint32_t x_odd = BF16 ? (uint32_t)(reinterpret_cast<uintptr_t>(xb) & 2u) / 2u : 0u;
  const buffer_rsrc rx =
      BF16 ? make_buffer(xb - x_odd, (bytes / 2 + 2u * x_odd + 3u) & ~3u)
           : make_buffer(static_cast<const float*>(grad) + wbase, bytes);

  // Row u starts shift_of(u) values past a line of h, has its first whole
  // quad at column first_of(u) and its last one before column end_of(u)
  // (nothing for rows the group lacks).
  const uint32_t base_shift = (uint32_t)((reinterpret_cast<uintptr_t>(h + wbase) & 127u) / 4u);
  auto shift_of = [&](int u) { return (int)((base_shift + (uint32_t)u * row_step) & 31u); };
  auto first_of = [&](int u) { return (4 - (shift_of(u) & 3)) & 3; };
  auto end_of = [&](int u) { return u < rows ? n - ((n - min(first_of(u), n)) & 3) : 0; };
  // Every quad starts on 16 bytes of h, so all of them start in the same half
  // of a bf16 word.
  const bool half =
      BF16 && ((((4u - (base_shift & 3u)) & 3u) + x_odd) & 1u) != 0;

  float4 xv[kLineRows], hv[kLineRows], gv[kLineRows];
  constexpr int kSliceF4 = NORM ? 1 : (kCols * R / 4 + kWave - 1) / kWave;
  using VRegs = float __attribute__((ext_vector_type(4 * kSliceF4)));
  VRegs vreg;  // this lane's share of the chunk's V rows
  const int v_last = (n * R + 3) / 4 - 1;
  auto slice_at = [&](int q) { return lane + q * kWave; };
  // Offset of this lane's quad of row u in window c.
  auto quad_off = [&](int u, int c) {
    const int col = c * kCols + lane * 4 - shift_of(u);
    const uint32_t o = ((uint32_t)u * row_step + (uint32_t)col) * 4u;
    return (uint32_t)col < (uint32_t)end_of(u) ? o : kDropOffset;
  };
  auto issue = [&](int c) __attribute__((always_inline)) {
    if constexpr (!NORM) {
      // The chains of chunk c take columns [c * kCols - kLineLag, ...): the
      // positions before column 0 and past the last hold V's first and last
      // values, which no chain reads.
      const float4* src = reinterpret_cast<const float4*>(V);
      const int first = (c * kCols - kLineLag) * R / 4;
#pragma unroll
      for (int q = 0; q < kSliceF4; ++q) {
        const float4 t = src[min(max(first + min(slice_at(q), kCols * R / 4 - 1), 0), v_last)];
        vreg[4 * q] = t.x;
        vreg[4 * q + 1] = t.y;
        vreg[4 * q + 2] = t.z;
        vreg[4 * q + 3] = t.w;
      }
    }
#pragma unroll
    for (int u = 0; u < kLineRows; ++u) {
      const uint32_t o = quad_off(u, c);
      if constexpr (BF16) {
        const uint32_t b = o / 2 + 2 * x_odd;
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
  };

  // The rows' ends, one value a lane: lane 8 * e + u is value e of row u's
  // head (e < 3) or value e - 3 of its tail (e < 6).
  const int end_row = lane & (kLineRows - 1), end_e = lane / kLineRows;
  const int head =
      min((int)((4u - ((base_shift + (uint32_t)end_row * row_step) & 3u)) & 3u), n);
  const int tail = (n - head) & 3;
  const bool end_ok = end_row < rows && (end_e < 3 ? end_e < head : end_e - 3 < tail);
  const int end_col = end_e < 3 ? end_e : n - tail + end_e - 3;
  const uint32_t end_off =
      end_ok ? ((uint32_t)end_row * row_step + (uint32_t)end_col) * 4u : kDropOffset;
  float end_x;
  if constexpr (BF16)
    end_x = __uint_as_float(buffer_load_u16<kCacheDefault>(rx, end_off / 2 + 2 * x_odd) << 16);
  else
    end_x = buffer_load_f1<kCacheDefault>(rx, end_off);
  const float end_h = buffer_load_f1<kCacheDefault>(rh, end_off);
  const float end_g = buffer_load_f1<kCacheDefault>(rg, end_off);
  issue(0);
  const float end_hn = fmaf(eta, end_x, a * end_h);
  const float end_delta = end_hn - end_g;
  buffer_store_f1<kCacheDefault>(rh, end_off, end_hn);

  const int nchunks = (n + kLineLag + kCols - 1) / kCols;
  float s = 0.0f;
  for (int c = 0; c < nchunks; ++c) {
#pragma unroll
    for (int u = 0; u < kLineRows; ++u) {
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
      buffer_store_f4<kCacheStreamDevice>(rh, quad_off(u, c), hn);
      // Column col of the row goes to word col - c * kCols + kLineLag.
      // Lanes without a whole quad write values no chain reads, or that the
      // row's ends replace below.
      store_f4_words(tile + u * kPitch + kLineLag + lane * 4 - shift_of(u),
                     make_float4(hn.x - gv[u].x, hn.y - gv[u].y, hn.z - gv[u].z,
                                 hn.w - gv[u].w));
    }
    {
      // (A row's tail can lie in the last window but one and in the last.)
      const int at = end_col - c * kCols + kLineLag;
      if (end_ok && at >= 0 && at < kCols + kLineLag) tile[end_row * kPitch + at] = end_delta;
    }
    if constexpr (!NORM) {
#pragma unroll
      for (int q = 0; q < kSliceF4; ++q) {
        const int f = min(slice_at(q), kCols * R / 4 - 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int idx = 4 * f + e;  // V[idx / R][idx % R] of the chunk
          vt[(idx % R) * (kCols + 4) + idx / R] = vreg[4 * q + e];
        }
      }
    }
    // The next chunk's loads go out before this chunk's chains run.
    if (c + 1 < nchunks) issue(c + 1);
    __builtin_amdgcn_sched_barrier(0);
    wave_lds_fence();
    // Chains over words [w0, w1): lane row + 8 k runs row `row` against
    // column k of V (lanes past 8 R repeat others' chains).
    const float* my_row = tile + (lane & (kLineRows - 1)) * kPitch;
    const float* my_v = vt + ((lane / kLineRows) % R) * (kCols + 4);
    auto chain4 = [&](int w) __attribute__((always_inline)) {
      const float4 dv = *reinterpret_cast<const float4*>(my_row + w);
      float4 v4 = dv;
      if constexpr (!NORM) v4 = *reinterpret_cast<const float4*>(my_v + w);
      s = fmaf(dv.x, v4.x, s);
      s = fmaf(dv.y, v4.y, s);
      s = fmaf(dv.z, v4.z, s);
      s = fmaf(dv.w, v4.w, s);
    };
    const int w0 = c == 0 ? kLineLag : 0;
    const int left = n - c * kCols + kLineLag;  // words to the row's end
    if (w0 == 0 && left >= kCols) {
#pragma unroll
      for (int w = 0; w < kCols; w += 4) chain4(w);
    } else {
      const int w1 = left < kCols ? left : kCols;
      int w = w0;
      for (; w + 4 <= w1; w += 4) chain4(w);
      for (; w < w1; ++w) s = fmaf(my_row[w], NORM ? my_row[w] : my_v[w], s);
    }
    // Carry the columns past this chunk's chains to the front.
    if (c + 1 < nchunks) {
      static_assert(kLineRows * kLineLag == 4 * kWave, "one float4 a lane");
      float* row = tile + (lane / (kLineLag / 4)) * kPitch + (lane % (kLineLag / 4)) * 4;
      *reinterpret_cast<float4*>(row) = *reinterpret_cast<const float4*>(row + kCols);
    }
    wave_lds_fence();
  }
  if (lane < kLineRows * R && (lane & (kLineRows - 1)) < rows)
    S[((int64_t)i * m + grp.row0 + (int64_t)(lane & (kLineRows - 1)) * grp.stride) * R +
      lane / kLineRows] = s;
}

template <int R, bool BF16, bool NORM>
void launch_lines(const void* grad, float* h, const float* g, const float* V,
                  const RowGroup* groups, int64_t ngroups, float* S, int64_t d, int64_t m,
                  int32_t N, float eta, float a, hipStream_t stream) {
  // The grid is one-dimensional for multiples of 8 workers, as the window
  // kernels' is.
  const unsigned nbx = blocks_for(ngroups, kLineWaves);
  const bool flat = N % 8 == 0 && (int64_t)nbx * N <= INT32_MAX;
  hipLaunchKernelGGL((sketch_lines_kernel<R, BF16, NORM>),
                     flat ? dim3(nbx * (unsigned)N) : dim3(nbx, (unsigned)N),
                     dim3(kLineWaves * kWave), 0, stream, grad, h, g, V, groups, ngroups, S, d,
                     m, eta, a, flat ? 1 : 0);
}

}  // namespace

hipError_t launch_sketch_lines(const void* grad, int32_t grad_bf16, float* h, const float* g,
                               const float* V, const RowGroup* groups, int64_t ngroups, float* S,
                               int64_t d, int64_t m, int32_t N, int32_t r, float eta, float a,
                               bool norm, hipStream_t stream) {
  if (ngroups <= 0) return hipSuccess;
#define ARC_LINES(RR, NN)                                                                     \
  if (grad_bf16)                                                                              \
    launch_lines<RR, true, NN>(grad, h, g, V, groups, ngroups, S, d, m, N, eta, a,       \
                               stream);                                                       \
  else                                                                                        \
    launch_lines<RR, false, NN>(grad, h, g, V, groups, ngroups, S, d, m, N, eta, a, stream)
  if (norm) {
    ARC_LINES(1, true);
    return hipGetLastError();
  }
  switch (r) {
    case 1: ARC_LINES(1, false); break;
    case 2: ARC_LINES(2, false); break;
    case 4: ARC_LINES(4, false); break;
    case 8: ARC_LINES(8, false); break;
    default: return hipErrorInvalidValue;
  }
#undef ARC_LINES
  return hipGetLastError();
}

}  // namespace arc
