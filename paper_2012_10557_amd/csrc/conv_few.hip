// Forward convolutions with few output pixels (a handful of frames, or the
// late stages of a few dozen): D[k][pix] = sum_(r,s,c) w[k][r][s][c] x(pix; r,s,c)
// in one launch.
//
// With a few thousand outputs the big LDS tiles do not fill the chip, and
// splitting their reduction over blocks costs a round trip of fp32 partials
// and a second launch.  What bounds such a convolution is how fast one CU can
// fetch its operands (at best about 50 B per clock).  So here a block owns a
// small tile (16 to 64 channels x 32 to 64 pixels) and the whole reduction;
// its waves take equal shares of the reduction, each streaming its operands
// through a private LDS ring without barriers (direct copies: 8 lanes read a
// whole 128-byte line; loading the MFMA operands straight into registers, 16
// rows per instruction, measured a quarter of that rate), and the partial
// tiles are added in wave order through LDS, where the epilogue (scale, shift,
// residual, ReLU) also runs.  In the two larger tiles several waves share a
// ring (four waves with private rings, one per SIMD, could not overlap their
// copies, LDS reads and MFMAs: 7.4 against 5.9 us for 128 channels at 28 x 28,
// 4 frames).  Blocks of an XCD cover a contiguous range of
// channel tiles, so that its L2 fetches only those rows of the weights.
// Measured (MI355X, bf16, 224 px, split tiles + reduction before): 512
// channels at 7 x 7, 4 frames 18.9 -> 7.0 us, 16 frames 22.1 -> 13.6;
// 256 at 14 x 14, 4 frames 17.2 -> 5.9, 36 frames 33.2 -> 22.3; 128 at
// 28 x 28, 4 frames 15.2 -> 5.9, 16 frames 22.1 -> 14.0.  fp32: 64 channels at
// 16 x 16, 48 frames 23.0 -> 15.0 us; 256 at 14 x 14, 16 frames 60.8 -> 48.6.
// fp32 sums are kept in runs (RunSum), which costs 1 to 2.5% (16 fp32 frames
// at 224 px 920 -> 930 us per call).
#include "kernels.hpp"

namespace ekya {
namespace {

__device__ __align__(16) uint4 g_few_zero[1];

template <int N> __device__ __forceinline__ void few_wait() {
  wait_vmcnt<N>();
  asm volatile("" ::: "memory");
}

struct FewArgs {
  ConvGeom g;
  const void *x, *w;
  void* y;
  ConvEpilogue epi;
  int tiles_m, tiles_n;
};

// Sum of the partial tiles in order, then the epilogue.
template <typename T, int TM, int TN, int PARTS, int THREADS>
__device__ __forceinline__ void few_epilogue(const FewArgs& a, const float* red, int m0, int n0,
                                             int npix) {
  constexpr int PITCH = TM + 4;
  const ConvGeom& g = a.g;
  const ConvEpilogue& e = a.epi;
  for (int o = threadIdx.x; o < TN * (TM / 4); o += THREADS) {
    const int pl = o / (TM / 4), cl = (o % (TM / 4)) * 4, k = m0 + cl;
    const long long pix = n0 + pl;
    if (pix >= npix || k >= g.K) continue;
    f32x4 s = *reinterpret_cast<const f32x4*>(red + pl * PITCH + cl);
#pragma unroll
    for (int w = 1; w < PARTS; ++w)
      s += *reinterpret_cast<const f32x4*>(red + (w * TN + pl) * PITCH + cl);
    float v[4] = {s[0], s[1], s[2], s[3]};
    const long long at = pix * g.K + k;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (e.scale) v[u] *= e.scale[k + u];
      if (e.shift) v[u] += e.shift[k + u];
    }
    if (e.res) {
      float r[4];
      load4<T>(reinterpret_cast<const T*>(e.res) + at, r);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += r[u];
    }
    if (e.relu) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = relu_nan(v[u]);
    }
    store4<T>(reinterpret_cast<T*>(a.y) + at, v);
  }
}

// Position of output pixel `pix`: its first input row and column (a row that
// is never inside the image for a pixel past the last), and its element offset
// in the image at *px.
template <typename T>
__device__ __forceinline__ void few_pixel(const ConvGeom& g, int pix, int npix, int* h0, int* w0,
                                          int* row, const T** px, const T* x) {
  const int pp = pix < npix ? pix : 0, n = pp / (g.P * g.Q), rem = pp - n * (g.P * g.Q);
  const int p = rem / g.Q;
  *h0 = pix < npix ? p * g.stride - g.pad : -(1 << 30);
  *w0 = (rem - p * g.Q) * g.stride - g.pad;
  *row = ((p * g.stride - g.pad) * g.W + *w0) * g.C;  // used inside the image only
  *px = x + (long long)n * g.H * g.W * g.C;
}

// A stage is 8 units (128 bytes) of every tile row: 64 bf16 or 32 fp32
// reduction elements, never straddling a filter tap.  NW waves, each with a
// private ring of NB stages: TM weight rows, then TN input-pixel rows, unit u
// of row r at u ^ (r mod 8), so that one copy fills 8 whole rows (8 lanes read
// one 128-byte line) and the fragment reads meet no bank conflict.
template <typename T, int TM, int TN, int NW, int NB>
__global__ __launch_bounds__(NW * 64) void conv_few_kernel(FewArgs a) {
  constexpr int E = Elt<T>::E, SE = 8 * E, TI = TM / 16, TJ = TN / 16;
  constexpr int CA = TM / 8, CB = TN / 8, CP = CA + CB;  // copies per stage
  constexpr int SU = CP * 64, PITCH = TM + 4;            // units per stage; floats per partial row
  constexpr int RING = NW * NB * SU, RED = NW * TN * PITCH / 4;
  __shared__ uint4 smem[RING > RED ? RING : RED];
  const ConvGeom& g = a.g;
  const int lane = threadIdx.x & 63, fr = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // contiguous range of tiles per XCD, pixels fastest
  const int total = a.tiles_m * a.tiles_n, xcd = blockIdx.x & 7;
  const int item = xcd * (total >> 3) + min(xcd, total & 7) + (blockIdx.x >> 3);
  const int m0 = (item / a.tiles_n) * TM, n0 = (item % a.tiles_n) * TN;
  const int npix = g.N * g.P * g.Q, Ktot = g.R * g.S * g.C, ns = Ktot / SE;
  const int s0 = ns * wave / NW, s1 = ns * (wave + 1) / NW;

  const int r8 = lane >> 3, unit = ((lane & 7) ^ r8) * E;
  const T *pa[CA], *pb[CB];
  int h0[CB], w0[CB], row[CB];
#pragma unroll
  for (int i = 0; i < CA; ++i)  // rows past the last re-read it and are not stored
    pa[i] = (const T*)a.w + (long long)min(m0 + 8 * i + r8, g.K - 1) * Ktot + unit;
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    few_pixel(g, n0 + 8 * j + r8, npix, &h0[j], &w0[j], &row[j], &pb[j], (const T*)a.x + unit);
  }
  int rs = s0 * SE / g.C, tc = s0 * SE - rs * g.C, tr = rs / g.S, ts = rs - tr * g.S;
  const void* zero = g_few_zero;
  asm volatile("" : "+s"(zero));
  uint4* ring = smem + wave * (NB * SU);
  auto issue = [&](int st, uint4* slot) {
    const int k0 = st * SE, tap = (tr * g.W + ts) * g.C + tc;
#pragma unroll
    for (int i = 0; i < CA; ++i) dma16(pa[i] + k0, slot + i * 64);
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const bool in = (unsigned)(h0[j] + tr) < (unsigned)g.H && (unsigned)(w0[j] + ts) < (unsigned)g.W;
      dma16(in ? (const void*)(pb[j] + (row[j] + tap)) : zero, slot + (CA + j) * 64);
    }
    tc += SE;
    if (tc >= g.C) {
      tc = 0;
      if (++ts == g.S) {
        ts = 0;
        ++tr;
      }
    }
  };

  f32x4 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < NB; ++p)
    if (s0 + p < s1) issue(s0 + p, ring + p * SU);
  const int off[2] = {fr * 8 + (q ^ (fr & 7)), fr * 8 + ((4 + q) ^ (fr & 7))};
  uint4* slot = ring;
  RunSum<T, TI, TJ, FP32_RUN> sum(acc);
  for (int st = s0; st < s1; ++st) {
    // stages st + 1 .. st + NB - 1 may still be in flight
    if (st + NB - 1 < s1)
      few_wait<CP * (NB - 1)>();
    else
      few_wait<0>();
    uint4 fa[2][TI], fb[2][TJ];
#pragma unroll
    for (int kf = 0; kf < 2; ++kf) {
#pragma unroll
      for (int i = 0; i < TI; ++i) fa[kf][i] = slot[i * 128 + off[kf]];
#pragma unroll
      for (int j = 0; j < TJ; ++j) fb[kf][j] = slot[CA * 64 + j * 128 + off[kf]];
    }
    // the wave's reads of the slot are complete before its refill is issued
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (st + NB < s1) issue(st + NB, slot);
#pragma unroll
    for (int kf = 0; kf < 2; ++kf) sum.add(fa[kf], fb[kf]);
    sum.end_stage();
    slot += SU;
    if (slot == ring + NB * SU) slot = ring;
  }
  sum.flush();
  __syncthreads();  // every ring is done with: its memory takes the partial tiles
  // lane: channels 16 i + 4 q .. + 3 of pixel 16 j + fr
  float* red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      *reinterpret_cast<f32x4*>(red + (wave * TN + 16 * j + fr) * PITCH + 16 * i + 4 * q) = acc[i][j];
  __syncthreads();
  few_epilogue<T, TM, TN, NW, NW * 64>(a, red, m0, n0, npix);
}

// The same for the larger tiles, whose operands several waves share: NG groups
// of waves split the reduction, a group's (TM / 32) (TN / 32) waves each
// compute a 32 x 32 quadrant of the tile and copy an equal part of the group's
// stages.  One barrier per stage (all groups), NB - 1 stages in flight.
template <typename T, int TM, int TN, int NG, int NB>
__global__ __launch_bounds__(NG * (TM / 32) * (TN / 32) * 64) void conv_few_shared_kernel(
    FewArgs a) {
  constexpr int E = Elt<T>::E, SE = 8 * E, WN = TN / 32, WG = (TM / 32) * WN;
  constexpr int CA = TM / 8 / WG, CB = TN / 8 / WG, CP = CA + CB;  // a wave's copies per stage
  constexpr int SU = (TM + TN) * 8, PITCH = TM + 4;  // units per stage; floats per partial row
  constexpr int RING = NG * NB * SU, RED = NG * TN * PITCH / 4;
  static_assert(CA * WG * 8 == TM && CB * WG * 8 == TN, "whole copies per wave");
  __shared__ uint4 smem[RING > RED ? RING : RED];
  const ConvGeom& g = a.g;
  const int lane = threadIdx.x & 63, fr = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave / WG, wl = wave % WG;
  const int total = a.tiles_m * a.tiles_n, xcd = blockIdx.x & 7;
  const int item = xcd * (total >> 3) + min(xcd, total & 7) + (blockIdx.x >> 3);
  const int m0 = (item / a.tiles_n) * TM, n0 = (item % a.tiles_n) * TN;
  const int npix = g.N * g.P * g.Q, Ktot = g.R * g.S * g.C, ns = Ktot / SE;
  const int s0 = ns * grp / NG, count = ns * (grp + 1) / NG - s0, rounds = cdiv(ns, NG);

  const int r8 = lane >> 3, unit = ((lane & 7) ^ r8) * E;
  const T *pa[CA], *pb[CB];
  int h0[CB], w0[CB], row[CB];
#pragma unroll
  for (int i = 0; i < CA; ++i)
    pa[i] = (const T*)a.w + (long long)min(m0 + 8 * (wl + WG * i) + r8, g.K - 1) * Ktot + unit;
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    few_pixel(g, n0 + 8 * (wl + WG * j) + r8, npix, &h0[j], &w0[j], &row[j], &pb[j],
              (const T*)a.x + unit);
  }
  int rs = s0 * SE / g.C, tc = s0 * SE - rs * g.C, tr = rs / g.S, ts = rs - tr * g.S;
  const void* zero = g_few_zero;
  asm volatile("" : "+s"(zero));
  uint4* ring = smem + grp * (NB * SU);
  auto issue = [&](int st, uint4* slot) {
    const int k0 = st * SE, tap = (tr * g.W + ts) * g.C + tc;
#pragma unroll
    for (int i = 0; i < CA; ++i) dma16(pa[i] + k0, slot + (wl + WG * i) * 64);
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const bool in = (unsigned)(h0[j] + tr) < (unsigned)g.H && (unsigned)(w0[j] + ts) < (unsigned)g.W;
      dma16(in ? (const void*)(pb[j] + (row[j] + tap)) : zero, slot + (TM / 8 + wl + WG * j) * 64);
    }
    tc += SE;
    if (tc >= g.C) {
      tc = 0;
      if (++ts == g.S) {
        ts = 0;
        ++tr;
      }
    }
  };

  const int wm = wl / WN, wn = wl % WN;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < NB - 1; ++p)
    if (p < count) issue(s0 + p, ring + p * SU);
  const int off[2] = {fr * 8 + (q ^ (fr & 7)), fr * 8 + ((4 + q) ^ (fr & 7))};
  int slot = 0;
  RunSum<T, 2, 2, FP32_RUN> sum(acc);
  for (int it = 0; it < rounds; ++it) {
    // the wave's copies of stage `it` have landed (later ones may be in flight)
    if (it + NB - 2 < count)
      few_wait<CP * (NB - 2)>();
    else
      few_wait<0>();
    // every wave's copies are visible, and stage it - 1 has been read
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (it + NB - 1 < count) issue(s0 + it + NB - 1, ring + (slot == 0 ? NB - 1 : slot - 1) * SU);
    if (it < count) {
      const uint4* As = ring + slot * SU + wm * 256;
      const uint4* Bs = ring + slot * SU + TM * 8 + wn * 256;
#pragma unroll
      for (int kf = 0; kf < 2; ++kf) {
        uint4 fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[i] = As[i * 128 + off[kf]];
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j] = Bs[j * 128 + off[kf]];
        sum.add(fa, fb);
      }
      sum.end_stage();
    }
    if (++slot == NB) slot = 0;
  }
  sum.flush();
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      *reinterpret_cast<f32x4*>(red + (grp * TN + 32 * wn + 16 * j + fr) * PITCH + 32 * wm + 16 * i +
                                4 * q) = acc[i][j];
  __syncthreads();
  few_epilogue<T, TM, TN, NG, NG * WG * 64>(a, red, m0, n0, npix);
}

template <typename T, int TM, int TN, int NW, int NB, bool SHARED>
hipError_t launch_few(FewArgs a, hipStream_t stream) {
  a.tiles_m = cdiv(a.g.K, TM);
  a.tiles_n = cdiv(a.g.N * a.g.P * a.g.Q, TN);
  const dim3 grid(a.tiles_m * a.tiles_n);
  if constexpr (SHARED)
    hipLaunchKernelGGL((conv_few_shared_kernel<T, TM, TN, NW, NB>), grid,
                       dim3(NW * (TM / 32) * (TN / 32) * 64), 0, stream, a);
  else
    hipLaunchKernelGGL((conv_few_kernel<T, TM, TN, NW, NB>), grid, dim3(NW * 64), 0, stream, a);
  return hipGetLastError();
}

template <typename T> hipError_t dispatch_few(const FewArgs& a, hipStream_t stream) {
  // the tile whose busiest CU fetches the fewest operand rows
  constexpr int cand[4][2] = {{64, 64}, {32, 64}, {32, 32}, {16, 32}};
  const long long npix = (long long)a.g.N * a.g.P * a.g.Q;
  int best = 0;
  long long least = 0;
  for (int i = 0; i < 4; ++i) {
    const long long blocks = cdiv(a.g.K, cand[i][0]) * cdivl(npix, cand[i][1]);
    const long long rows = cdivl(blocks, 256) * (cand[i][0] + cand[i][1]);
    if (i == 0 || rows < least) {
      best = i;
      least = rows;
    }
  }
  switch (best) {
    case 0: return launch_few<T, 64, 64, 2, 4, true>(a, stream);
    case 1: return launch_few<T, 32, 64, 4, 3, true>(a, stream);
    case 2: return launch_few<T, 32, 32, 8, 2, false>(a, stream);
    default: return launch_few<T, 16, 32, 8, 3, false>(a, stream);
  }
}

}  // namespace

bool conv_few_ok(int dt, const ConvGeom& g) {
  const int se = 8 * dtype_vec(dt);
  const long long npix = (long long)g.N * g.P * g.Q, red = (long long)g.R * g.S * g.C;
  // At most two 64 x 64 tiles per CU: at 512 tiles (256 channels x 8192 pixels)
  // it is a third faster than split or half-filled large tiles, at 784 (12544
  // pixels) 42.6 against 31.4 us.  fp32, bound by the MFMAs there, meets 64 x 64
  // copied tiles with sums in runs as well: in inference at 224 px (layers 1 to
  // 4 of 10, 20, 40 and 80 frames, 490 tiles) 569, 928, 1653 and 3110 us per
  // call here, 559, 925, 1665 and 3150 there, so only long reductions go beyond
  // 448 tiles; at 512 (8192 pixels x 256) 94.6 against 90.9.  With fewer stages
  // than waves (1 x 1 filters) half a tile per CU: 64 -> 128 channels at 3136
  // pixels (98 tiles) 5.1 -> 4.4 us, at 14400 (450) 4.3 -> 6.6.
  const long long most = red < 8 * se ? 128 : dt == DT_BF16 ? 512 : red < 2048 ? 448 : 511;
  // Offsets within an image are 32-bit.
  return g.N > 0 && g.C % se == 0 && g.K % 4 == 0 && red < (1 << 24) &&
         ((long long)g.H + 2 * g.pad) * g.W * g.C < (1LL << 31) &&
         cdiv(g.K, 64) * cdivl(npix, 64) <= most;
}

hipError_t conv_few_fwd(int dt, const ConvGeom& g, const void* x, const void* w, void* y,
                        const ConvEpilogue& epi, hipStream_t stream) {
  if (!conv_few_ok(dt, g)) return hipErrorInvalidValue;
  const FewArgs a{g, x, w, y, epi, 0, 0};
  KernelTimer* t = thread_timer();
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (t) {
    e0 = t->take();
    e1 = t->take();
    EKYA_HIP(hipEventRecord(e0, stream));
  }
  EKYA_HIP(dt == DT_F32 ? dispatch_few<float>(a, stream) : dispatch_few<bf16>(a, stream));
  if (t) {
    const double m = (double)g.N * g.P * g.Q, taps = (double)g.R * g.S;
    EKYA_HIP(hipEventRecord(e1, stream));
    t->recs.push_back({dt == DT_F32 ? "conv_fwd<f32,few>" : "conv_fwd<bf16,few>",
                       2.0 * m * g.K * taps * (g.C0 ? g.C0 : g.C),
                       ((double)g.N * g.H * g.W * g.C + m * g.K + (double)g.K * taps * g.C) *
                           dtype_size(dt),
                       e0, e1});
  }
  return hipSuccess;
}

}  // namespace ekya
