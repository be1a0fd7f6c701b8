// logits.hip -- the output projection of a batch: Y[m, n] = (X[m] . W[n]) *
// scale[n] in fp32 over a wide vocabulary (K = 64 KS up to 512, any M).
//
// Bound by its own output: 65.5 MB for 512 rows of 32,000 logits, 10.6 us at the
// 6.2 TB/s that a plain write kernel reaches, against 3.4 us of matrix-core time.  So a
// block does all of its loading at its start, and then only multiplies and
// stores: each of its 8 waves keeps the weights of 32 columns for the whole K
// in registers (two tiles of 16, 64 VGPRs at K = 512), the block's rows (up to
// 256) come into LDS 64 at a time, and no store is waited for (in the tiled
// GEMM each 64 columns of K cost a memory round trip and two barriers, and
// loads wait behind stores: one in-order counter).  X is the A operand, so 16
// lanes store 64 contiguous bytes of a row (with the weights there a lane
// stores 16 bytes of its own row, four times the store requests: 10.2 against
// 9.3 us at 256 x 256 x 32000).  Against the tiled kernels of the time, and the
// GEMV for 4 rows (row-major; in fragment order): 256 x 256 x 32000 12.6 -> 9.7
// us (9.1), 512 x 512 x 32000 27.5 -> 17.7 us (17.1), 4 x 256 x 32000 7.8 -> 4.0
// us (3.6).
//
// FRAG: W is in fragment order (launch_pack_fragments), each load one
// contiguous kilobyte.  Row-major, the block's weights come in as whole rows
// and pass through LDS into the matrix operand's order, before X takes the
// same LDS (gathered straight into that order, 64 bytes of 16 rows per load,
// they arrive at a quarter of the rate).
#include <algorithm>

#include "blocks.hpp"
#include "internal.h"

namespace mnmt {
namespace {

constexpr int kLgWaves = 8, kLgThreads = 64 * kLgWaves, kLgCols = 32 * kLgWaves, kLgRows = 256;

template <int KS, bool FRAG>
__global__ __launch_bounds__(kLgThreads) void k_logits_rows(const int8_t* __restrict__ X, int ldx,
                                                            const int8_t* __restrict__ W,
                                                            const float* __restrict__ scale, int M, int N, int ncol,
                                                            int rows_per_block, float* __restrict__ Y) {
  constexpr int K = 64 * KS, ROW = K + 16, CPR = K / 16;  // padded LDS row, 16-byte chunks per row
  constexpr int NX = kLgRows * CPR / kLgThreads, NW = kLgCols * CPR / kLgThreads;  // chunks per thread
  __shared__ __attribute__((aligned(16))) int8_t xl[kLgRows * ROW];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // blocks of one column range next to each other on one XCD (their weights
  // then come from its L2): the launcher pads the grid to whole groups of 8
  const int b = blockIdx.x, per = gridDim.x / 8, id = (b % 8) * per + b / 8;
  const int nr = (M + rows_per_block - 1) / rows_per_block;
  if (id >= ncol * nr) return;
  const int n0 = (id / nr) * kLgCols, row0 = (id % nr) * rows_per_block, rows = min(rows_per_block, M - row0);
  const int nw = n0 + 32 * wave, l16 = lane & 15, q4 = lane >> 4;
  v4i w[2][KS];
  v4i wr[FRAG ? 1 : NW];
  if constexpr (FRAG) {
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const size_t tile = min(nw / 16 + f, (N - 1) / 16);
#pragma unroll
      for (int k = 0; k < KS; ++k) w[f][k] = *(const v4i*)(W + (tile * KS + k) * 1024 + 16 * lane);
    }
  } else {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int c = tid + kLgThreads * i;
      wr[i] = *(const v4i*)(W + (size_t)min(n0 + c / CPR, N - 1) * K + 16 * (c % CPR));
    }
  }
  float sc[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) sc[f] = scale[min(nw + 16 * f + l16, N - 1)];
  v4i xr[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int c = tid + kLgThreads * i;
    xr[i] = *(const v4i*)(X + (size_t)(row0 + min(c / CPR, rows - 1)) * ldx + 16 * (c % CPR));
  }
  asm volatile("" ::: "memory");
  if constexpr (!FRAG) {
    static_assert(kLgCols <= kLgRows, "");
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int c = tid + kLgThreads * i;
      *(v4i*)(xl + (c / CPR) * ROW + 16 * (c % CPR)) = wr[i];
    }
    lds_barrier();
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int k = 0; k < KS; ++k) w[f][k] = *(const v4i*)(xl + (32 * wave + 16 * f + l16) * ROW + 64 * k + 16 * q4);
    lds_barrier();
  }
  const int8_t* xp = xl + l16 * ROW + 16 * q4;
  float* y = Y + (size_t)(row0 + 4 * q4) * N + nw + l16;
  const bool ok[2] = {nw + l16 < N, nw + 16 + l16 < N};
  // 64 rows at a time: X arrives in LDS while the rows before are multiplied
  // and stored (the stores come after every load, so no load waits for them)
#pragma unroll
  for (int g = 0; g < kLgRows / 64; ++g) {
    if (64 * g >= rows) break;
#pragma unroll
    for (int i = (64 * g * NX + kLgRows - 1) / kLgRows; i < (64 * (g + 1) * NX + kLgRows - 1) / kLgRows; ++i) {
      const int c = tid + kLgThreads * i;
      *(v4i*)(xl + (c / CPR) * ROW + 16 * (c % CPR)) = xr[i];
    }
    lds_barrier();
#pragma unroll 1
    for (int r = 64 * g; r < min(64 * g + 64, rows); r += 32) {
      v4i acc[2][2];
#pragma unroll
      for (int m = 0; m < 2; ++m) acc[m][0] = acc[m][1] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < KS; ++k) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const v4i x = *(const v4i*)(xp + 16 * m * ROW + 64 * k);
          acc[m][0] = mfma16(x, w[0][k], acc[m][0]);
          acc[m][1] = mfma16(x, w[1][k], acc[m][1]);
        }
      }
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int f = 0; f < 2; ++f)
            if (r + 16 * m + 4 * q4 + i < rows && ok[f])
              y[(size_t)(16 * m + i) * N + 16 * f] = (float)acc[m][f][i] * sc[f];
      xp += 32 * ROW;
      y += (size_t)32 * N;
    }
  }
}

template <int KS>
hipError_t launch_ks(const int8_t* X, int ldx, const int8_t* W, bool frag, const float* scale, int M, int N, float* Y,
                     hipStream_t s) {
  const int ncol = (N + kLgCols - 1) / kLgCols;
  // row ranges: at least what LDS holds, and enough for about one block per CU
  const int want = max((M + kLgRows - 1) / kLgRows, min((M + 15) / 16, 256 / ncol));
  const int rpb = ((M + want - 1) / want + 15) / 16 * 16, nr = (M + rpb - 1) / rpb;
  const dim3 grid((ncol * nr + 7) / 8 * 8), block(kLgThreads);
  if (frag)
    hipLaunchKernelGGL((k_logits_rows<KS, true>), grid, block, 0, s, X, ldx, W, scale, M, N, ncol, rpb, Y);
  else
    hipLaunchKernelGGL((k_logits_rows<KS, false>), grid, block, 0, s, X, ldx, W, scale, M, N, ncol, rpb, Y);
  return hipGetLastError();
}

}  // namespace

static bool logits_rows_fit(int K, int N) {
  return (K == 64 || K == 128 || K == 256 || K == 384 || K == 512) && N > 24 * kLgCols;
}

// Where it is used: the widths it is compiled for, vocabularies of more than 24
// column blocks, and outputs large enough.  A block's weights (256 columns for
// the whole K, 128 KB at K = 512) come in before its first product, so a small
// output waits for them longer than the tiles do (row-major, us, against the
// faster of the GEMV, fragment and chunk kernels): 3 x 384 x 8000 4.7 against
// 3.8, 16 x 384 x 8000 4.8 against 3.6, 64 x 512 x 16000 6.1 against 4.3, 256 x
// 512 x 12000 8.2 against 7.5, 256 x 256 x 16000 6.8 against 7.1, 512 x 512 x
// 8000 8.5 against 8.7, 1024 x 512 x 32000 31 against 39.  In fragment order
// they come in sooner: 64 x 256 x 16000 4.1 against 3.8, 128 x 256 x 12000 4.4
// against 4.5, 256 x 512 x 12000 7.3 against 7.5.  The GEMV of 5 to 8 rows is
// slower throughout (8 x 64 x 6200 4.6 against 3.1), that of 3 and 4 from 10,000
// columns on (3 x 384 x 12000 5.0 against 4.8); below 32 rows the tiles store
// cut-off fragments (16 x 256 x 32000 4.3 against 4.1, in fragment order 3.8).
bool logits_rows_wins(int M, int K, int N, bool frag) {
  if (!logits_rows_fit(K, N)) return false;
  if (M <= 8) return M > 4 || N >= 10000;
  if (M < 32 && (frag ? N >= (K <= 256 ? 12000 : 20000) : K <= 256 && N >= 20000)) return true;
  const long out = (long)M * N;
  return out >= (frag ? 6000L * K : std::min(10000L * K + 600000L, 3600000L));
}

hipError_t launch_logits_rows(const int8_t* X, int ldx, const int8_t* W, bool frag, const float* scale, int M, int K,
                              int N, float* Y, hipStream_t s) {
  if (M < 1 || !logits_rows_fit(K, N)) return hipErrorInvalidValue;
  switch (K) {
    case 64: return launch_ks<1>(X, ldx, W, frag, scale, M, N, Y, s);
    case 128: return launch_ks<2>(X, ldx, W, frag, scale, M, N, Y, s);
    case 256: return launch_ks<4>(X, ldx, W, frag, scale, M, N, Y, s);
    case 384: return launch_ks<6>(X, ldx, W, frag, scale, M, N, Y, s);
    default: return launch_ks<8>(X, ldx, W, frag, scale, M, N, Y, s);
  }
}

}  // namespace mnmt
