// fg_dense.hip -- the dense vertex transform Y = X W on the matrix cores
// (fp32 in and out).
#include "fg_device.h"

namespace fg {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Columns of K that a workgroup stages in LDS at a time.
constexpr int kDenseK = 16;

// Four floats of a row of `len` elements from column c on; 0 past its end.
__device__ __forceinline__ f32x4 row4(const float* row, int32_t c, int32_t len) {
  if (c + 4 <= len) {
    const float4_a4 t = *reinterpret_cast<const float4_a4*>(row + c);
    return f32x4{t.x, t.y, t.z, t.w};
  }
  f32x4 r = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int q = 0; q < 3; ++q)
    if (c + q < len) r[q] = row[c + q];
  return r;
}

// Y[n, M] = X[n, K] W[K, M]: one BM x BN tile of Y per workgroup, four
// wavefronts of 32x32 blocks (TM x TN each) of v_mfma_f32_32x32x2_f32.  Operand
// layout of the instruction: lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32] and receives D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32],
// r = 0..15.  Any two columns of K may form an instruction's pair as long as A
// and B agree: lane half h takes columns h * kDenseK / 2 + i, i = 0, 1, ..., so
// that its A values lie side by side in LDS and two 16-byte reads bring eight.
//
// Bound by the matrix cores at large K (602 -> 512: 118 TFLOP/s; without the
// loads from memory this loop reaches 133), at small K by the write of Y, which
// the tiles of one round do not hide.  X and W reach LDS through registers, one
// step of K ahead, in two buffers with one barrier a step.  The kernel before
// this one had no tiles: every lane loaded its operands, four bytes at a time,
// for each instruction.  232,965 rows, 256 -> 128: 403 -> 171 us (39 -> 89
// TFLOP/s); 602 -> 128: 1035 -> 350 us.  Steps of 32 columns (1.00-1.6x) and
// 128 x 128 tiles (1.10x at 256 -> 128, 0.96x at 602 -> 512) are not used.
template <int BM, int BN, int TM, int TN>
__global__ __launch_bounds__(kBlock) void dense_tile_kernel(const float* x, const float* w,
                                                            float* y, int64_t n, int32_t K,
                                                            int32_t M, int32_t col_tiles,
                                                            int64_t tiles) {
  static_assert((BM / (32 * TM)) * (BN / (32 * TN)) == kWavesPerBlock, "four wavefronts a tile");
  constexpr int AS = kDenseK + 4;  // LDS row strides: 16-byte rows, banks spread
  constexpr int BS = BN + 4;
  constexpr int NA = BM * kDenseK / 4 / kBlock;  // float4 per thread and step
  constexpr int NB = BN * kDenseK / 4 / kBlock;
  static_assert(NA >= 1 && NB >= 1, "every thread stages at least one float4 of each operand");
  __shared__ __align__(16) float as[2][BM * AS];
  __shared__ __align__(16) float bs[2][kDenseK * BS];
  // neighbouring tiles of a row of tiles read the same rows of X: keep them on
  // one die (workgroup i runs on die i mod 8)
  const int64_t per = (tiles + 7) / 8;
  const int64_t tile = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (tile >= tiles) return;
  const int64_t row0 = tile / col_tiles * BM;
  const int32_t col0 = (int32_t)(tile % col_tiles) * BN;
  const int t = threadIdx.x;
  const int lane = lane_id();
  const int wv = t >> 6;
  const int wm = wv / (BN / (32 * TN)) * (32 * TM), wn = wv % (BN / (32 * TN)) * (32 * TN);
  const int i = lane & 31, h = lane >> 5;

  // whole tiles and steps load without tests: a test per load would make the
  // compiler wait for each before it issues the next
  const bool full = row0 + BM <= n && col0 + BN <= M;
  f32x4 ra[NA], rb[NB];
  auto fetch = [&](int32_t k0) {
    if (full && k0 + kDenseK <= K) {
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        const int e = t + q * kBlock;
        const float* p = x + (row0 + e / (kDenseK / 4)) * K + k0 + e % (kDenseK / 4) * 4;
        ra[q] = *reinterpret_cast<const float4_a4*>(p);
      }
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int e = t + q * kBlock;
        const float* p = w + (int64_t)(k0 + e / (BN / 4)) * M + col0 + e % (BN / 4) * 4;
        rb[q] = *reinterpret_cast<const float4_a4*>(p);
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int e = t + q * kBlock;
      const int64_t r = row0 + e / (kDenseK / 4);
      ra[q] = r < n ? row4(x + r * K, k0 + e % (kDenseK / 4) * 4, K) : f32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int e = t + q * kBlock;
      const int32_t k = k0 + e / (BN / 4);
      rb[q] = k < K ? row4(w + (int64_t)k * M, col0 + e % (BN / 4) * 4, M) : f32x4{0, 0, 0, 0};
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int e = t + q * kBlock;
      *reinterpret_cast<f32x4*>(&as[buf][e / (kDenseK / 4) * AS + e % (kDenseK / 4) * 4]) = ra[q];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int e = t + q * kBlock;
      *reinterpret_cast<f32x4*>(&bs[buf][e / (BN / 4) * BS + e % (BN / 4) * 4]) = rb[q];
    }
  };

  f32x16 acc[TM][TN] = {};
  fetch(0);
  stage(0);
  __syncthreads();
  int buf = 0;
  for (int32_t k0 = 0; k0 < K; k0 += kDenseK, buf ^= 1) {
    const bool more = k0 + kDenseK < K;
    if (more) fetch(k0 + kDenseK);
    f32x4 a[TM][kDenseK / 8];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
      for (int q = 0; q < kDenseK / 8; ++q)
        a[m][q] = *reinterpret_cast<const f32x4*>(
            &as[buf][(wm + 32 * m + i) * AS + h * (kDenseK / 2) + 4 * q]);
#pragma unroll
    for (int s = 0; s < kDenseK / 2; ++s) {
      float b[TN];
#pragma unroll
      for (int c = 0; c < TN; ++c) b[c] = bs[buf][(h * (kDenseK / 2) + s) * BS + wn + 32 * c + i];
#pragma unroll
      for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int c = 0; c < TN; ++c)
          acc[m][c] =
              __builtin_amdgcn_mfma_f32_32x32x2f32(a[m][s / 4][s % 4], b[c], acc[m][c], 0, 0, 0);
    }
    if (more) stage(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < TM; ++m)
#pragma unroll
    for (int c = 0; c < TN; ++c) {
      const int32_t col = col0 + wn + 32 * c + i;
      if (col >= M) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = row0 + wm + 32 * m + 8 * (r / 4) + 4 * h + r % 4;
        if (row < n) y[row * M + col] = acc[m][c][r];
      }
    }
}

// Narrow X: one wavefront per 16-row x 64-column tile of Y, four 16 x 16 blocks of
// v_mfma_f32_16x16x4_f32, every lane loading its operands.  Lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[4 (l / 16) + r][l % 16].
// Without the staging and its barriers nothing delays the write of Y, and K is
// padded to 4, not 16.  300,000 rows, us, staged / direct: 8 -> 16: 14.0 / 9.9;
// 20 -> 7: 19.5 / 14.1; 33 -> 7: 27.9 / 21.8; 100,000 rows, 2 -> 128: 14.2 / 10.4.
constexpr int kDirectCols = 64;

__global__ __launch_bounds__(kBlock) void dense_direct_kernel(const float* x, const float* w,
                                                              float* y, int64_t n, int32_t K,
                                                              int32_t M, int64_t n_tiles) {
  const int64_t t = wave_item();
  if (t >= n_tiles) return;
  const int64_t col_tiles = (M + kDirectCols - 1) / kDirectCols;
  const int64_t rt = t / col_tiles, ct = t % col_tiles;
  const int lane = lane_id();
  const int i = lane & 15, q = lane >> 4;
  const int64_t arow = rt * 16 + i;
  f32x4 acc[4] = {};
  for (int k0 = 0; k0 < K; k0 += 4) {
    const int k = k0 + q;
    const float a = (arow < n && k < K) ? x[arow * K + k] : 0.0f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int64_t col = ct * kDirectCols + b * 16 + i;
      const float bv = (k < K && col < M) ? w[(int64_t)k * M + col] : 0.0f;
      acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv, acc[b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int64_t col = ct * kDirectCols + b * 16 + i;
    if (col >= M) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = rt * 16 + q * 4 + r;
      if (row < n) y[row * M + col] = acc[b][r];
    }
  }
}

template <int BM, int BN, int TM, int TN>
void dense_go(int64_t n, int64_t K, int64_t M, const float* x, const float* w, float* y,
              hipStream_t st) {
  const int64_t cols = (M + BN - 1) / BN, tiles = (n + BM - 1) / BM * cols;
  const int64_t grid = (tiles + 7) / 8 * 8;
  FG_LAUNCH((dense_tile_kernel<BM, BN, TM, TN>), dim3((unsigned)grid), st, x, w, y, n, (int32_t)K,
            (int32_t)M, (int32_t)cols, tiles);
}

}  // namespace

hipError_t launch_dense_matmul(int64_t n, int64_t K, int64_t M, const float* x, const float* w,
                               float* y, hipStream_t stream) {
  if (n == 0 || M == 0) return hipSuccess;
  // many rows, and up to 12 columns of X (unless much of the last block of 64
  // columns of Y is padding: 937,000 rows, 8 -> 68, lose 10 us) or a last step of
  // 16 that mostly is (17, 20, 33; any for Y of at most 16 columns); fewer rows
  // end together, staged or not
  const int64_t pad = (K + kDenseK - 1) / kDenseK * kDenseK - K;
  const int64_t cols = (M + kDirectCols - 1) / kDirectCols * kDirectCols;
  const bool narrow = K <= 12   ? M <= kDirectCols || 10 * cols <= 13 * M
                      : M <= 16 ? K < 64 && pad > 0
                                : K < 40 && pad >= 12;
  if (n >= 65536 && narrow) {
    const int64_t tiles = (n + 15) / 16 * ((M + kDirectCols - 1) / kDirectCols);
    FG_LAUNCH(dense_direct_kernel, grid_for(tiles, 1), stream, x, w, y, n, (int32_t)K, (int32_t)M,
              tiles);
    return hipGetLastError();
  }
  // 64 x 128 tiles read X half as often as 64 x 64 ones (232,965 rows, 256 ->
  // 128: 171 against 184 us) once they give each of the 256 compute units four
  // or more; below that (20,000 rows, 256 -> 256: 36 against 31 us), and for Y
  // of at most 64 columns (100,000 rows, 100 -> 64: 41 against 23 us), the
  // smaller tiles.
  if (M > 64 && (n + 63) / 64 * ((M + 127) / 128) >= 1024)
    dense_go<64, 128, 1, 2>(n, K, M, x, w, y, stream);
  else
    dense_go<64, 64, 1, 1>(n, K, M, x, w, y, stream);
  return hipGetLastError();
}

}  // namespace fg
