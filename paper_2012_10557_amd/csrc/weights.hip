// Weight layouts: the caller's canonical array (convolutions [K][C][RS]) to
// and from the internal fp32 master ([K][RS][C]), and the low-precision
// copies the convolutions read ([K][RS][Cp] and [C][RS][K]).
//
// All of it is copying, bound by memory: 11.2 M parameters read once and each
// layout written once.  A row k of a convolution is C * RS contiguous floats
// in both fp32 layouts (at most 18 KB in ResNet18), so a block takes one row,
// reads it in order into LDS, and writes it in the other order from there:
// every global access is coalesced, and with RS odd (9, 49) the strided LDS
// side meets no bank conflict.  The same pass leaves the low-precision copy.
// Measured (MI355X, the whole network, bf16): to the [K][RS][C] copies 24 us
// (45 MB read, 22 written) where permuting element by element took 81-100 us
// and a pass of its own for the copies 31 us; back to canonical 22 us (90 MB);
// the [C][RS][K] copies of layer4 16 us.
#include "kernels.hpp"

namespace ekya {
namespace {

constexpr int ROW_MAX = 4608;   // floats of a row (or part of one) staged in LDS
constexpr int CRSK_MAX = 128;   // floats of an output channel per transposing tile

// The table row a block works on: row blockIdx.y of tab, or `one`.
__device__ __forceinline__ LayoutRow layout_row(const LayoutRow* tab, const LayoutRow& one) {
  return tab ? tab[blockIdx.y] : one;
}

template <typename T> __device__ __forceinline__ T low(float v) { return (T)v; }

// blockIdx.y: table row; blocks along x share its output channels.
// TO_INTERNAL: src canonical, dst master (null: only the rows without a
// low-precision copy are written, to `rest`), shadow (null: none).
// Otherwise src master, dst canonical.
template <typename T, bool TO_INTERNAL>
__global__ __launch_bounds__(256) void layout_kernel(const float* src, float* dst, float* rest,
                                                     const LayoutRow* tab, LayoutRow one,
                                                     T* shadow) {
  __shared__ float buf[ROW_MAX];
  const LayoutRow row = layout_row(tab, one);
  const long long off = row.off;
  const int C = (int)row.C, RS = (int)row.RS, Cp = (int)row.Cp, t = threadIdx.x;
  const bool packed = TO_INTERNAL && shadow && row.krsc >= 0;
  if constexpr (TO_INTERNAL)
    if (row.krsc < 0) dst = rest;
  // (host: RS <= ROW_MAX, so rs * C + c below stays under 2^31)
  if (RS == 1 && (!packed || Cp == C)) {  // same order: a straight copy
    const long long n = row.K * C;
    for (long long i = blockIdx.x * 1024LL + t; i < n; i += gridDim.x * 1024LL) {
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = i + 256 * j < n ? src[off + i + 256 * j] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i + 256 * j < n) {
          if (dst) dst[off + i + 256 * j] = v[j];
          if (packed) shadow[row.krsc + i + 256 * j] = low<T>(v[j]);
        }
    }
    return;
  }
  const int part = min(C, ROW_MAX / RS);  // channels per staged part (host: RS <= ROW_MAX)
  const int parts = cdiv(C, part);
  const long long items = row.K * parts;
  for (long long it = blockIdx.x; it < items; it += gridDim.x) {
    const long long k = it / parts;
    const int c0 = (int)(it % parts) * part, cn = min(part, C - c0), n = cn * RS;
    const long long canon = off + (k * C + c0) * RS;  // [c][rs] from here
    const long long inner = off + k * RS * C + c0;    // [rs][c], rows C apart
    // (rs, c) of element i = t in [rs][c] order, stepped by 256
    int rs = t / cn, c = t - rs * cn;
    const int drs = 256 / cn, dc = 256 - drs * cn;
    if constexpr (TO_INTERNAL) {
      for (int i0 = t; i0 < n; i0 += 256 * 9) {
        float v[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) v[j] = i0 + 256 * j < n ? src[canon + i0 + 256 * j] : 0.f;
#pragma unroll
        for (int j = 0; j < 9; ++j)
          if (i0 + 256 * j < n) buf[i0 + 256 * j] = v[j];
      }
      __syncthreads();
      T* low_row = packed ? shadow + row.krsc + k * RS * Cp + c0 : nullptr;
      for (int i0 = t; i0 < n; i0 += 256 * 9) {
        float v[9];
        int at[9], al[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) {
          const bool in = i0 + 256 * j < n;
          v[j] = in ? buf[c * RS + rs] : 0.f;
          at[j] = in ? rs * C + c : -1;
          al[j] = rs * Cp + c;
          rs += drs;
          c += dc;
          if (c >= cn) {
            c -= cn;
            ++rs;
          }
        }
        if (dst) {
#pragma unroll
          for (int j = 0; j < 9; ++j)
            if (at[j] >= 0) dst[inner + at[j]] = v[j];
        }
        if (packed) {
#pragma unroll
          for (int j = 0; j < 9; ++j)
            if (at[j] >= 0) low_row[al[j]] = low<T>(v[j]);
        }
      }
      if (packed && c0 + cn == C)  // channels padded to the 16-byte unit
        for (int i = t; i < RS * (Cp - C); i += 256)
          shadow[row.krsc + (k * RS + i / (Cp - C)) * Cp + C + i % (Cp - C)] = low<T>(0.f);
    } else {
      for (int i0 = t; i0 < n; i0 += 256 * 9) {
        float v[9];
        int at[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) {
          const bool in = i0 + 256 * j < n;
          v[j] = in ? src[inner + (long long)rs * C + c] : 0.f;
          at[j] = in ? c * RS + rs : -1;
          rs += drs;
          c += dc;
          if (c >= cn) {
            c -= cn;
            ++rs;
          }
        }
#pragma unroll
        for (int j = 0; j < 9; ++j)
          if (at[j] >= 0) buf[at[j]] = v[j];
      }
      __syncthreads();
      for (int i = t; i < n; i += 256) dst[canon + i] = buf[i];
    }
    __syncthreads();
  }
}

// Filters of more than ROW_MAX taps: element by element.
template <typename T>
__global__ __launch_bounds__(256) void layout_any_kernel(const float* src, float* dst,
                                                         const LayoutRow* tab, LayoutRow one,
                                                         T* shadow, int to_internal) {
  const LayoutRow row = layout_row(tab, one);
  const long long off = row.off, C = row.C, RS = row.RS, Cp = row.Cp, n = row.K * RS * Cp;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += gridDim.x * 256LL) {
    const long long c = i % Cp, rs = i / Cp % RS, k = i / (Cp * RS);  // [k][rs][padded c]
    const long long a = off + (k * C + c) * RS + rs, b = off + (k * RS + rs) * C + c;
    const float v = c < C ? src[to_internal ? a : b] : 0.f;
    if (c < C && dst) dst[to_internal ? b : a] = v;
    if (shadow && row.krsc >= 0) shadow[row.krsc + i] = low<T>(v);
  }
}

// [C][RS][K] copy straight from the canonical [K][C][RS]: a tile is 64 output
// channels x `part` input channels, read in runs of part * RS floats and
// written in runs of 64 elements.
template <typename T>
__global__ __launch_bounds__(256) void pack_crsk_kernel(const float* src, const LayoutRow* tab,
                                                        LayoutRow one, T* shadow) {
  __shared__ float tile[64][CRSK_MAX + 1];
  const LayoutRow row = layout_row(tab, one);
  if (row.crsk < 0) return;
  const int K = (int)row.K, C = (int)row.C, RS = (int)row.RS, t = threadIdx.x;
  const int part = max(1, 72 / RS);  // 8 channels x 9 taps (host: RS <= CRSK_MAX)
  const int tk = cdiv(K, 64), tc = cdiv(C, part);
  const int kk = t & 63, w = t >> 6;
  for (long long it = blockIdx.x; it < (long long)tk * tc; it += gridDim.x) {
    const int k0 = (int)(it / tc) * 64, c0 = (int)(it % tc) * part;
    const int n = min(part, C - c0) * RS, kn = min(64, K - k0);
    const float* from = src + row.off + ((long long)k0 * C + c0) * RS;
    int r = t / n, e = t - r * n;
    const int dr = 256 / n, de = 256 - dr * n;
    for (int i0 = t; i0 < kn * n; i0 += 256 * 9) {
      float v[9];
      int at[9];
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const bool in = i0 + 256 * j < kn * n;
        v[j] = in ? from[(long long)r * C * RS + e] : 0.f;
        at[j] = in ? r * (CRSK_MAX + 1) + e : -1;
        r += dr;
        e += de;
        if (e >= n) {
          e -= n;
          ++r;
        }
      }
#pragma unroll
      for (int j = 0; j < 9; ++j)
        if (at[j] >= 0) (&tile[0][0])[at[j]] = v[j];
    }
    __syncthreads();
    if (kk < kn) {
      T* to = shadow + row.crsk + (long long)c0 * RS * K + k0 + kk;
#pragma unroll 6
      for (int u = w; u < n; u += 4)  // u: (channel, tap)
        to[(long long)u * K] = low<T>(tile[kk][u]);
    }
    __syncthreads();
  }
}

template <typename F> hipError_t with_type(int dt, F&& f) {
  if (dt == DT_F32) f((float*)nullptr); else f((bf16*)nullptr);
  return hipGetLastError();
}

// Blocks per table row: ResNet18's largest convolutions have 512 rows.
constexpr int LAYOUT_BLOCKS = 256;

}  // namespace

hipError_t weights_to_internal(int dt, const float* canonical, float* master, float* rest,
                               const LayoutTable& tab, void* shadow, hipStream_t stream) {
  if (tab.n == 0) return hipSuccess;
  return with_type(dt, [&](auto* tp) {
    using T = std::remove_pointer_t<decltype(tp)>;
    if (tab.max_taps > ROW_MAX)
      hipLaunchKernelGGL(layout_any_kernel<T>, dim3(1024, tab.n), dim3(256), 0, stream, canonical,
                         master, tab.rows, tab.one, (T*)shadow, 1);
    else
      hipLaunchKernelGGL((layout_kernel<T, true>), dim3(LAYOUT_BLOCKS, tab.n), dim3(256), 0, stream,
                         canonical, master, rest, tab.rows, tab.one, (T*)shadow);
  });
}

hipError_t weights_to_canonical(const float* master, float* canonical, const LayoutTable& tab,
                                hipStream_t stream) {
  if (tab.n == 0) return hipSuccess;
  if (tab.max_taps > ROW_MAX)
    hipLaunchKernelGGL(layout_any_kernel<float>, dim3(1024, tab.n), dim3(256), 0, stream, master,
                       canonical, tab.rows, tab.one, (float*)nullptr, 0);
  else
    hipLaunchKernelGGL((layout_kernel<float, false>), dim3(LAYOUT_BLOCKS, tab.n), dim3(256), 0,
                       stream, master, canonical, (float*)nullptr, tab.rows, tab.one,
                       (float*)nullptr);
  return hipGetLastError();
}

bool pack_crsk_ok(int taps) { return taps <= CRSK_MAX; }

hipError_t pack_crsk(int dt, const float* canonical, const LayoutTable& tab, void* shadow,
                     hipStream_t stream) {
  if (tab.n == 0) return hipSuccess;
  return with_type(dt, [&](auto* tp) {
    using T = std::remove_pointer_t<decltype(tp)>;
    hipLaunchKernelGGL(pack_crsk_kernel<T>, dim3(LAYOUT_BLOCKS, tab.n), dim3(256), 0, stream,
                       canonical, tab.rows, tab.one, (T*)shadow);
  });
}

}  // namespace ekya
