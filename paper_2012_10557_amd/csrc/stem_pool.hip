// The eval-mode stem in one kernel: 7x7 / stride 2 / pad 3 convolution of
// 3-channel bf16 frames into 64 channels, folded BatchNorm, ReLU and the 3x3 /
// stride 2 / pad 1 max pool.
//
// Its floor is memory (a 224 px frame: 301 KB read, 401 KB written); what
// bounds it is the vector work of pooling beside 28 MFMAs per 16 columns, and
// phases that follow one another in a block.  So:
//  - a block of four waves owns 4 pool rows of one image; a wave has 32
//    channels and two pool rows and walks its 5 stem rows downwards, keeping
//    its filter operands (7 filter rows) and the running vertical maximum in
//    registers: no LDS exchange and no barrier after the input is staged;
//  - the maximum is taken over raw sums, two rotations and one three-way
//    maximum a value, a column tile ahead of whose maxima the next tile's MFMAs
//    are issued, and scale, shift and ReLU are applied to pooled rows only.
//    With a finite, nonzero scale and a finite shift they are monotone in the
//    sum once the filter rows of channels with a negative scale are negated
//    (exact), so the result equals pooling the rounded stem output.  Any other
//    coefficient can turn an infinite (or, times infinity, a zero) sum into a
//    NaN, which a maximum has to skip: a wave with such a channel applies them
//    before the maximum (in a copy of the code, as a branch in it would keep
//    the maxima from running beside the MFMAs).  Maxima skip NaNs; a window of
//    nothing but NaNs gives -inf;
//  - input rows are staged in LDS once (channels 0..2 and a zero, 8 bytes a
//    pixel), two pixels per 12-byte load where frames are 4-byte aligned and
//    of even width (2-byte loads otherwise);
//  - blocks are persistent, two per CU, one staging while the other computes.
// One MFMA k-step is one filter row: 8 taps (the 8th zero) x 4 channels, a
// lane's operand 2 adjacent pixels of the staged row.
// Measured (MI355X): 500 frames at 224 px 656 -> 276 us (430 TFLOP/s of useful
// products, 1.3 TB/s; before, a wave per stem row finished every stem value
// and exchanged rows through LDS, one block per CU; without the waves' choice
// of path 267), 500 at 112 px 200 -> 81, 4 at 224 px 26.0 -> 17.8.
#include <type_traits>

#include "kernels.hpp"

namespace ekya {
namespace {

constexpr int SP_NT = 256;
constexpr int SP_IN_ROWS = 23;  // input rows behind 9 stem rows
constexpr int SP_BLOCKS = 512;  // two per CU
constexpr int SP_QMAX = 112;

struct StemPoolArgs {
  const bf16* x;       // [.][H][W][3]
  const int32_t* idx;  // image n at idx[n] (null: n)
  const bf16* wk;      // [64][7][7][8]
  bf16* y;             // [N][PP][PQ][64]
  ConvEpilogue epi;
  int N, H, W, P, Q;
};

__device__ __forceinline__ float max3_skip_nan(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float max_skip_nan(float a, float b) {
  float d;
  asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
// DPP on rows of 16 lanes: x of the lane one place higher (wrapping); x of the
// lane one place lower, lane 0 taking lane 15 of `before`.
__device__ __forceinline__ float lane_right(float x) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x12F, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_left(float x, float before) {
  const int wrapped =
      __builtin_amdgcn_update_dpp(0, __float_as_int(before), 0x121, 0xF, 0xF, false);
  return __int_as_float(
      __builtin_amdgcn_update_dpp(wrapped, __float_as_int(x), 0x111, 0xF, 0xF, false));
}

// Scale and shift are two roundings, as in the other convolutions' epilogues.
__device__ __forceinline__ float affine(float v, float scale, float shift) {
#pragma clang fp contract(off)
  v = v * scale;
  return v + shift;
}
// The epilogue of one pooled sum; NaN (nothing but NaNs in the window) gives
// -inf.
__device__ __forceinline__ float finish(float m, float scale, float shift, float floor) {
  const float v = affine(m, scale, shift), c = max_skip_nan(v, floor);
  return v == v ? c : -INFINITY;
}
// Coefficients with which the affine map is monotone and keeps NaNs apart.
__device__ __forceinline__ bool monotone(float scale, float shift) {
  return scale != 0.f && __builtin_isfinite(scale) && __builtin_isfinite(shift);
}

// ODD: Q is odd, so the last window lacks its right column.
template <int TQ, bool WIDE, bool ODD>
__global__ __launch_bounds__(SP_NT, 2) void stem_pool_kernel(StemPoolArgs a) {
  constexpr int PW = 32 * TQ + 6;  // staged pixels per row: columns -3 .. 32 TQ + 2
  __shared__ __align__(16) uint2 patch[SP_IN_ROWS * PW];
  const int lane = threadIdx.x & 63, lr = lane & 15, kc = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave & 1, rg = wave >> 1;  // channels 32 half .., pool rows 2 rg, 2 rg + 1
  const int H = a.H, W = a.W, P = a.P, Q = a.Q;
  const int PP = (P - 1) / 2 + 1, PQ = (Q - 1) / 2 + 1, per_img = cdiv(PP, 4);
  const float nan = __builtin_nanf(""), floor = a.epi.relu ? 0.f : -INFINITY;

  // filter operands: MFMA row lr of tile i is channel 32 half + 16 i + lr,
  // taps 2 kc, 2 kc + 1 of filter row r, channels 0..3; negated where the
  // channel's scale is negative
  uint4 fa[2][7];
  float sa[2][4], sb[2][4];  // |scale|, shift of the lane's outputs
  bool plain = true;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = 32 * half + 16 * i + lr, ko = 32 * half + 16 * i + 4 * kc;
    const uint32_t flip = a.epi.scale && a.epi.scale[k] < 0.f ? 0x80008000u : 0u;
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      const bf16* w = a.wk + ((k * 7 + r) * 7 + 2 * kc) * 8;
      const uint2 t0 = *reinterpret_cast<const uint2*>(w);
      const uint2 t1 = kc < 3 ? *reinterpret_cast<const uint2*>(w + 8) : make_uint2(0u, 0u);
      fa[i][r] = make_uint4(t0.x ^ flip, t0.y ^ flip, t1.x ^ flip, t1.y ^ flip);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sa[i][e] = a.epi.scale ? __builtin_fabsf(a.epi.scale[ko + e]) : 1.f;
      sb[i][e] = a.epi.shift ? a.epi.shift[ko + e] : 0.f;
      plain = plain && monotone(sa[i][e], sb[i][e]);
    }
  }

  for (int item = blockIdx.x; item < a.N * per_img; item += gridDim.x) {
    const int n = item / per_img, bq = item - n * per_img;
    const int p0 = 8 * bq - 1;  // first of the block's 9 stem rows
    const bf16* img = a.x + (a.idx ? a.idx[n] : n) * ((long long)H * W * 3);
    // wave v stages input rows 2 p0 - 3 + v, + 4, ..
    if constexpr (WIDE) {
      constexpr int RR = (SP_IN_ROWS + 3) / 4, UU = (16 * TQ + 63) / 64;
      uint3 v[RR][UU];
#pragma unroll
      for (int rr = 0; rr < RR; ++rr)
#pragma unroll
        for (int u = 0; u < UU; ++u) {
          const int pr = wave + 4 * rr, h = 2 * p0 - 3 + pr, j = lane + 64 * u;
          v[rr][u] = make_uint3(0u, 0u, 0u);
          if (pr < SP_IN_ROWS && (unsigned)h < (unsigned)H && 2 * j < W)
            v[rr][u] = *reinterpret_cast<const uint3*>(img + ((long long)h * W + 2 * j) * 3);
        }
      __syncthreads();  // the previous item's rows are done with
#pragma unroll
      for (int rr = 0; rr < RR; ++rr)
#pragma unroll
        for (int u = 0; u < UU; ++u) {
          const int pr = wave + 4 * rr, j = lane + 64 * u;
          if (pr < SP_IN_ROWS && 2 * j < W) {
            uint2* d = patch + pr * PW + 2 * j + 3;
            d[0] = make_uint2(v[rr][u].x, v[rr][u].y & 0xFFFFu);
            d[1] = make_uint2((v[rr][u].y >> 16) | (v[rr][u].z << 16), v[rr][u].z >> 16);
          }
        }
    } else {
      __syncthreads();
      for (int pr = wave; pr < SP_IN_ROWS; pr += 4) {
        const int h = 2 * p0 - 3 + pr;
        for (int w = lane; w < W; w += 64) {
          uint2 v = make_uint2(0u, 0u);
          if ((unsigned)h < (unsigned)H) {
            const unsigned short* px =
                reinterpret_cast<const unsigned short*>(img + ((long long)h * W + w) * 3);
            v = make_uint2((unsigned)px[0] | ((unsigned)px[1] << 16), (unsigned)px[2]);
          }
          patch[pr * PW + w + 3] = v;
        }
      }
    }
    // columns outside the image
    const int right = W + 3, pads = 3 + PW - right;
    for (int pr = wave; pr < SP_IN_ROWS; pr += 4)
      for (int c = lane; c < pads; c += 64)
        patch[pr * PW + (c < 3 ? c : right + c - 3)] = make_uint2(0u, 0u);
    __syncthreads();

    // EACH: scale and shift apply to every sum, not to the pooled ones (no
    // barrier in here: the waves of a block may differ)
    auto rows = [&](auto EACH) {
      float keep[TQ][2][4];  // vertical maximum so far of each column, lane's channels
      const int l0 = 4 * rg, pr0 = 4 * bq + 2 * rg;
      // one stem row: f(t, i, m) gets the window maxima of tile t along the row
      auto stem_row = [&](int l, auto&& f) {
        const uint2* prow = patch + 2 * l * PW + 2 * lr + 2 * kc;
        f32x4 acc[2][2];
        auto sums = [&](int t, f32x4 (&d)[2]) {
          uint4 fb[7];
#pragma unroll
          for (int r = 0; r < 7; ++r)
            fb[r] = *reinterpret_cast<const uint4*>(prow + r * PW + 32 * t);
#pragma unroll
          for (int i = 0; i < 2; ++i) d[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int r = 0; r < 7; ++r)
#pragma unroll
            for (int i = 0; i < 2; ++i) mma_unit(d[i], fa[i][r], fb[r], (bf16*)nullptr);
          if constexpr (EACH.value) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int e = 0; e < 4; ++e) d[i][e] = affine(d[i][e], sa[i][e], sb[i][e]);
          }
        };
        sums(0, acc[0]);
        float before[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) before[i][e] = nan;
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
          if (t + 1 < TQ) sums(t + 1, acc[(t + 1) & 1]);  // its MFMAs run beside this tile's maxima
          const int q = 16 * t + lr;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            float m[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float v = acc[t & 1][i][e];
              const float left = lane_left(v, before[i][e]);
              float right = lane_right(v);  // every lane rotates, then selects
              if (ODD) right = q + 1 < Q ? right : nan;
              m[e] = max3_skip_nan(left, v, right);
              before[i][e] = v;
            }
            f(t, i, m);
          }
        }
      };
      auto emit = [&](int pr, int t, int i, const float (&o)[4]) {
        const int q = 16 * t + lr;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = finish(o[e], EACH.value ? 1.f : sa[i][e], EACH.value ? 0.f : sb[i][e], floor);
        if (pr < PP && (lr & 1) == 0 && q < Q)
          store4<bf16>(a.y + (((long long)n * PP + pr) * PQ + (q >> 1)) * 64 + 32 * half + 16 * i +
                           4 * kc,
                       v);
      };
      // stem rows 2 m - 1, 2 m, 2 m + 1 of pool rows m = pr0, pr0 + 1; the last
      // row of a window is the first of the next.  Rows outside the image count
      // as NaNs.
      auto clear = [&] {
#pragma unroll
        for (int t = 0; t < TQ; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) keep[t][i][e] = nan;
      };
      if (p0 + l0 >= 0 && p0 + l0 < P)
        stem_row(l0, [&](int t, int i, const float (&m)[4]) {
#pragma unroll
          for (int e = 0; e < 4; ++e) keep[t][i][e] = m[e];
        });
      else
        clear();
#pragma unroll 1
      for (int j = 0; j < 2; ++j) {
        const int l = l0 + 2 * j, pr = pr0 + j;
        if (p0 + l + 1 < P)
          stem_row(l + 1, [&](int t, int i, const float (&m)[4]) {
#pragma unroll
            for (int e = 0; e < 4; ++e) keep[t][i][e] = max_skip_nan(keep[t][i][e], m[e]);
          });
        if (p0 + l + 2 < P) {
          stem_row(l + 2, [&](int t, int i, const float (&m)[4]) {
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              o[e] = max_skip_nan(keep[t][i][e], m[e]);
              keep[t][i][e] = m[e];
            }
            emit(pr, t, i, o);
          });
        } else {
#pragma unroll
          for (int t = 0; t < TQ; ++t)
#pragma unroll
            for (int i = 0; i < 2; ++i) emit(pr, t, i, keep[t][i]);
          clear();
        }
      }
    };
    if (__builtin_expect(__all(plain), 1))
      rows(std::false_type{});
    else
      rows(std::true_type{});
  }
}

template <int TQ>
void launch_stem_pool(const StemPoolArgs& a, bool wide, int blocks, hipStream_t stream) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(SP_NT), 0, stream, a);
  };
  if (wide)
    a.Q % 2 ? go(stem_pool_kernel<TQ, true, true>) : go(stem_pool_kernel<TQ, true, false>);
  else
    a.Q % 2 ? go(stem_pool_kernel<TQ, false, true>) : go(stem_pool_kernel<TQ, false, false>);
}

}  // namespace

bool stem_pool_ok(int dt, const ConvGeom& g) {
  return dt == DT_BF16 && g.C == 8 && (g.C0 == 0 || g.C0 == 3) && g.K == 64 && g.R == 7 &&
         g.S == 7 && g.stride == 2 && g.pad == 3 && g.Q <= SP_QMAX && g.Q >= 1 && g.P >= 1;
}

hipError_t stem_pool_fwd(int dt, const ConvGeom& g, const void* frames, const int32_t* idx,
                         const void* w, void* y, const ConvEpilogue& epi, hipStream_t stream) {
  if (!stem_pool_ok(dt, g) || epi.res) return hipErrorInvalidValue;
  if (g.N == 0) return hipSuccess;
  const StemPoolArgs a{(const bf16*)frames, idx, (const bf16*)w, (bf16*)y, epi,
                       g.N, g.H, g.W, g.P, g.Q};
  const int items = g.N * cdiv((g.P - 1) / 2 + 1, 4), blocks = items < SP_BLOCKS ? items : SP_BLOCKS;
  // 12-byte loads of two pixels: every row starts on a 4-byte boundary
  const bool wide = g.W % 2 == 0 && reinterpret_cast<uintptr_t>(frames) % 4 == 0;
  KernelTimer* t = thread_timer();
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (t) {
    e0 = t->take();
    e1 = t->take();
    EKYA_HIP(hipEventRecord(e0, stream));
  }
  // The running maxima are registers, by number of 16-column tiles: exact at the
  // frame sizes in use (64, 112, 160 and 224 px: 2, 4, 5, 7); widths in between
  // take the next and compute up to a third more than they store (500 frames at
  // 96 px, 3 tiles in 4, 144 -> 67 us; at 192 px, 6 in 7, 492 -> 222).
  switch (cdiv(g.Q, 16)) {
    case 1: case 2: launch_stem_pool<2>(a, wide, blocks, stream); break;
    case 3: case 4: launch_stem_pool<4>(a, wide, blocks, stream); break;
    case 5: launch_stem_pool<5>(a, wide, blocks, stream); break;
    default: launch_stem_pool<7>(a, wide, blocks, stream); break;
  }
  EKYA_HIP(hipGetLastError());
  if (t) {
    const double m = (double)g.N * g.P * g.Q;
    EKYA_HIP(hipEventRecord(e1, stream));
    t->recs.push_back({"conv_fwd<bf16,stem7x7+pool,frames>", 2.0 * m * 64 * 147,
                       ((double)g.N * g.H * g.W * g.C + m * 64 + 64.0 * 49 * g.C) * 2, e0, e1});
  }
  return hipSuccess;
}

}  // namespace ekya
