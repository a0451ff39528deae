// Fully connected layers in fp32: forward, data gradient and weight gradient
// as one small matrix product on the fp32 matrix cores.
//
// The products of a classifier head are short (a hidden layer of 1024 neurons
// at batch 64: 64 x 1024 x 512, 67 MFLOP), so what bounds them is the latency
// of one pass over the operands, which L2 holds: a block owns one 16 x 16
// output tile (32 x 32 where there are many), its four waves take a quarter
// of the reduction each, a wave issues the loads of up to 128 reduction
// elements (16 of a short reduction) at once straight into the MFMA operand registers (no LDS staging:
// an operand is used by one wave only), and the four partial tiles are added
// in wave order through LDS.  Eight (four) accumulators per tile, folded
// after each round of loads, keep the rounding chains short and the MFMAs
// independent: against float64 the results are as close as the wave
// reductions this replaced (forward 8.4e-8, 8.3e-8 before) or closer (data
// gradient 1e-7, 5.8e-7 before).
//
// Measured (MI355X, the layer above): forward 445 -> 5.1 us, data gradient
// 98 -> 5.7, weight and bias gradient 16 -> 7.4; at 400 rows forward 455 ->
// 12.6 us.  Before, every sample's block read the whole weight matrix.
#include <climits>

#include "kernels.hpp"

namespace ekya {
namespace {

// C[m][n] = sum_k A(m, k) B(n, k) (+ bias[n]), then ReLU or a ReLU mask.
// An operand is k-contiguous (row * ld + k) or k-strided (k * ld + row).
struct LinArgs {
  const float *A, *B;
  long long lda, ldb;
  int avec, bvec;  // 16-byte loads along k allowed (k-contiguous operands)
  int M, N, K;
  const float* bias;   // [N] or null
  const float* mask;   // [M][N] or null: the result passes where mask > 0
  int relu;            // max(., 0)
  const int32_t* rows; // null, or row m of A (AK) / row k of B (BROWS) is at rows[.]
  float* C;            // [M][N]
  float* rowsum;       // [M] or null: sum_k A(m, k) (k-strided A)
};

// Elements k .. k + 3 of operand row `row`; zero from `end` on.  ROWS (k-strided
// operands): element k is at rows[k] * ld.
template <bool KC, bool ROWS = false>
__device__ __forceinline__ f32x4 lin_load(const float* P, long long ld, int row, int k, int end,
                                          int vec, const int32_t* rows = nullptr) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (KC) {
    const float* p = P + row * ld + k;
    if (vec) {  // end is a multiple of 4
      if (k < end) v = *reinterpret_cast<const f32x4*>(p);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + e < end) v[e] = p[e];
    }
  } else if constexpr (ROWS) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < end) v[e] = P[rows[k + e] * ld + row];
  } else {
    const float* p = P + (long long)k * ld + row;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < end) v[e] = p[e * ld];
  }
  return v;
}

// U: 16-element k-chunks in flight.
template <bool AK, bool BK, int T, bool BROWS, int U>
__global__ __launch_bounds__(256) void linear_kernel(LinArgs a) {
  constexpr int S = 16 * T;           // tile side
  constexpr int NA = T == 1 ? 8 : 4;  // accumulators per 16 x 16 tile
  __shared__ float red[4][S][S + 1];
  __shared__ float rs[4][S];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, q = lane >> 4, r = lane & 15;
  const int tn = cdiv(a.N, S);  // tiles per row of tiles
  const int m0 = (int)(blockIdx.x / tn) * S, n0 = (int)(blockIdx.x % tn) * S;
  int ra[T], rb[T];  // rows past the edge re-read the last one and are not stored
#pragma unroll
  for (int i = 0; i < T; ++i) {
    ra[i] = min(m0 + 16 * i + r, a.M - 1);
    if constexpr (AK && BK)
      if (a.rows) ra[i] = a.rows[ra[i]];
    rb[i] = min(n0 + 16 * i + r, a.N - 1);
  }
  const int chunks = cdiv(a.K, 16), per = cdiv(chunks, 4);
  const int c0 = min(chunks, wave * per), c1 = min(chunks, c0 + per);
  const int end = min(a.K, 16 * c1);
  f32x4 sum[T][T];
  float asum[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    asum[i] = 0.f;
#pragma unroll
    for (int j = 0; j < T; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int c = c0; c < c1; c += U) {
    f32x4 av[U][T], bv[U][T];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int k = 16 * (c + u) + 4 * q;
        av[u][i] = lin_load<AK>(a.A, a.lda, ra[i], k, end, a.avec);
        bv[u][i] = lin_load<BK, BROWS>(a.B, a.ldb, rb[i], k, end, a.bvec, a.rows);
      }
    f32x4 acc[T][T][NA];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int j = 0; j < T; ++j)
#pragma unroll
        for (int u = 0; u < NA; ++u) acc[i][j][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) {
            f32x4& d = acc[i][j][(4 * u + e) % NA];
            d = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][i][e], bv[u][j][e], d, 0, 0, 0);
          }
      if constexpr (!AK) {
#pragma unroll
        for (int i = 0; i < T; ++i)
          asum[i] += (av[u][i][0] + av[u][i][1]) + (av[u][i][2] + av[u][i][3]);
      }
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int j = 0; j < T; ++j) {
#pragma unroll
        for (int h = NA / 2; h > 0; h >>= 1)
#pragma unroll
          for (int u = 0; u < h; ++u) acc[i][j][u] += acc[i][j][u + h];
        sum[i][j] += acc[i][j][0];
      }
  }
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][16 * i + 4 * q + e][16 * j + r] = sum[i][j][e];
  if constexpr (!AK) {
#pragma unroll
    for (int i = 0; i < T; ++i) {
      float v = asum[i];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (q == 0) rs[wave][16 * i + r] = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < T * T; ++i) {
    const int x = t + 256 * i, row = x / S, col = x % S;
    const int m = m0 + row, n = n0 + col;
    if (m >= a.M || n >= a.N) continue;
    float v = (red[0][row][col] + red[1][row][col]) + (red[2][row][col] + red[3][row][col]);
    if (a.bias) v += a.bias[n];
    if (a.relu) v = fmaxf(v, 0.f);
    const long long o = (long long)m * a.N + n;
    if (a.mask) v = a.mask[o] > 0.f ? v : 0.f;
    a.C[o] = v;
  }
  if constexpr (!AK) {
    if (a.rowsum && n0 == 0 && t < S && m0 + t < a.M)
      a.rowsum[m0 + t] = (rs[0][t] + rs[1][t]) + (rs[2][t] + rs[3][t]);
  }
}

// At most JN outputs per row: a block takes a row, a strided slice per thread
// and then the wave and block reductions in one order.
template <int JN>
__global__ __launch_bounds__(256) void linear_rows_kernel(LinArgs a) {
  __shared__ float red[4][JN];
  const int m = blockIdx.x, t = threadIdx.x;
  const float* row = a.A + (a.rows ? a.rows[m] : m) * a.lda;
  float s[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j) s[j] = 0.f;
  for (int k = t; k < a.K; k += 256) {
    const float x = row[k];
#pragma unroll
    for (int j = 0; j < JN; ++j)
      if (j < a.N) s[j] += x * a.B[j * a.ldb + k];
  }
#pragma unroll
  for (int j = 0; j < JN; ++j) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[j] += __shfl_xor(s[j], o, 64);
    if ((t & 63) == 0) red[t >> 6][j] = s[j];
  }
  __syncthreads();
  if (t < a.N) {
    float v = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
    if (a.bias) v += a.bias[t];
    a.C[(long long)m * a.N + t] = a.relu ? fmaxf(v, 0.f) : v;
  }
}

int lin_vec(const float* p, long long ld, int K) {
  return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0 && K % 4 == 0;
}

template <bool AK, bool BK, bool BROWS = false>
hipError_t linear(LinArgs a, hipStream_t stream) {
  if (a.M < 1 || a.N < 1 || a.K < 1) return hipErrorInvalidValue;
  a.avec = AK && lin_vec(a.A, a.lda, a.K);
  a.bvec = BK && lin_vec(a.B, a.ldb, a.K);
  // 16 x 16 tiles up to two blocks per CU, then 32 x 32 (half the operand
  // reads per output): 64 x 1024 outputs (256 small tiles) over 512 5.1 us,
  // 400 x 1024 (1600) 16.7 us in small tiles and 12.6 in large ones,
  // 1024 x 512 (2048) over 64 13.0 and 7.4
  const long long t16 = (long long)cdiv(a.M, 16) * cdiv(a.N, 16);
  const long long t32 = (long long)cdiv(a.M, 32) * cdiv(a.N, 32);
  if (t32 > INT_MAX) return hipErrorInvalidValue;
  // up to 64 reduction elements are one chunk a wave: one in flight, for the
  // same sums from an eighth of the code, which such a call spends its time
  // fetching (both gradients of 512 -> 6, a synchronous call: 1 row 29.1 -> 25.9
  // us, 64 rows 28.7 -> 25.7)
  const dim3 grid((unsigned)(t16 <= 512 ? t16 : t32));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, a);
    return hipGetLastError();
  };
  if (t16 <= 512)
    return a.K <= 64 ? go(linear_kernel<AK, BK, 1, BROWS, 1>) : go(linear_kernel<AK, BK, 1, BROWS, 8>);
  return a.K <= 64 ? go(linear_kernel<AK, BK, 2, BROWS, 1>) : go(linear_kernel<AK, BK, 2, BROWS, 4>);
}

}  // namespace

hipError_t fc_fwd(const float* f, const float* W, const float* b, int N, int I, int J, float* z,
                  hipStream_t stream, bool relu, const int32_t* rows) {
  if (N == 0) return hipSuccess;
  LinArgs a{};
  a.A = f;
  a.lda = I;
  a.B = W;
  a.ldb = I;
  a.M = N;
  a.N = J;
  a.K = I;
  a.bias = b;
  a.relu = relu;
  a.rows = rows;
  a.C = z;
  // Few outputs leave most of a tile's columns unused; its waves make up for it
  // with 16-byte loads, or with many short rows to share the weights.  Without
  // either, and for one output, a block per row (synchronous calls, tiles and
  // rows: 39 rows of 1486 -> 2 30.8 and 22.4 us, 400 of 513 -> 6 25.3 and 22.5, 10 of
  // 4097 -> 8 53.1 and 34.3, 3000 of 2050 -> 3 46.1 and 31.4, but 3000 of 1486 -> 8
  // 32.7 and 37.2, 4096 of 513 -> 6 25.4 and 29.9; 39 of 1486 -> 1 29.6 and 20.2; up to
  // 16 outputs long rows only: 93 of 1503 -> 11 33.9 and 29.6, 1000 of 513 -> 16 25.2
  // and 27.8, 3000 of 2049 -> 16 45.6 and 59.7)
  const bool vec = lin_vec(f, I, I) && lin_vec(W, I, I);
  const bool few = J <= 8 ? N <= 1024 || I >= 2048 : J <= 16 && N <= 1024 && I >= 1024;
  // (a launch has fewer than 2^32 threads)
  if (N < (1 << 24) && (J == 1 || (J > 1 && !vec && few))) {
    if (I < 1) return hipErrorInvalidValue;
    if (J == 1)
      hipLaunchKernelGGL(linear_rows_kernel<1>, dim3(N), dim3(256), 0, stream, a);
    else if (J <= 8)
      hipLaunchKernelGGL(linear_rows_kernel<8>, dim3(N), dim3(256), 0, stream, a);
    else
      hipLaunchKernelGGL(linear_rows_kernel<16>, dim3(N), dim3(256), 0, stream, a);
    return hipGetLastError();
  }
  return linear<true, true>(a, stream);
}

hipError_t fc_bwd(const float* dz, const float* f, const float* W, int N, int I, int J, float* dW,
                  float* db, float* df, hipStream_t stream, const float* mask,
                  const int32_t* rows) {
  LinArgs w{};  // dW[j][i] = sum_n dz[n][j] f[n][i]
  w.A = dz;
  w.lda = J;
  w.B = f;
  w.ldb = I;
  w.M = J;
  w.N = I;
  w.K = N;
  w.C = dW;
  w.rowsum = db;
  w.rows = rows;
  if (rows)
    EKYA_HIP((linear<false, false, true>(w, stream)));
  else
    EKYA_HIP((linear<false, false>(w, stream)));
  if (!df) return hipSuccess;
  LinArgs x{};  // df[n][i] = sum_j dz[n][j] W[j][i]
  x.A = dz;
  x.lda = J;
  x.B = W;
  x.ldb = I;
  x.M = N;
  x.N = I;
  x.K = J;
  x.mask = mask;
  x.C = df;
  return linear<true, false>(x, stream);
}

}  // namespace ekya
