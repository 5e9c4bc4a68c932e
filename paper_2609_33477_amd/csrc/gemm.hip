// Plain bf16 GEMMs of a replayed transformer block (group replay chaining,
// Section 4.1), C = A B^T with A [M][K] row-major activations, B [N][K]
// row-major weights (nn.Linear layout), fp32 accumulation, and the block's
// element-wise work fused into the epilogue:
//   RESID   C[m][n] += acc          (fp32 residual stream, in place): the
//                                    output projection and the MLP's down
//                                    projection add into the hidden state
//   SWIGLU  H[m][j] = SiLU(gate) * up (bf16), gate = A W_gate^T,
//           up = A W_up^T: the wave's 16-column fragment blocks alternate gate
//           and up rows of the same hidden units, so a lane holds both factors
//           of each output in matching registers.
//
// Main loop: the 256 x 256 tile of sr_tile.hpp.  The weight rows of a wave's
// 128 columns are fed in the order that gives a lane 4 neighbouring columns of
// each 64 (RESID) or 4 neighbouring hidden units (SWIGLU), so the residual is
// accessed 16 bytes per lane (256 contiguous bytes per row) and hidden units
// are stored 8 bytes per lane.
#include "sr_tile.hpp"

#include <type_traits>

namespace sr {
namespace {

__device__ __forceinline__ float silu(float x) { return x * __builtin_amdgcn_rcpf(1.f + __expf(-x)); }

template <int MODE>
__global__ __launch_bounds__(kTileThreads<TileBig>, 1) void block_gemm_kernel(BlockGemmArgs a, int tiles_m, int tiles_n) {
  if (a.err && *a.err) return;   // the call's table check failed: write nothing
  __shared__ __attribute__((aligned(1024))) char smem[kTileLds<TileBig>];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid >> 1, wn = wid & 1;
  const int lc = lane & 15, g = lane >> 4;
  int mt, nt;
  tile_of(blockIdx.x, tiles_m, tiles_n, mt, nt);
  const int64_t row0 = (int64_t)mt * TileBig::ROWS;
  const int n0 = nt * TileBig::ROWS;
  const int K = a.K;
  const int64_t M = a.M;

  const char* a_base = static_cast<const char*>(a.A) + row0 * K * 2;
  uint32_t a_off[4];
  const char* b_ptr[TileRing<TileBig, bf16_t>::DB];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int row = tile_a_row(wid, i, lane);
    const int chunk = tile_a_chunk<TileBig>(row, lane);
    const int64_t last = M - 1 - row0;             // rows past M are never stored
    row = row < last ? row : (int)last;
    a_off[i] = (uint32_t)(row * (K * 2) + chunk * 16);
  }
#pragma unroll
  for (int i = 0; i < TileRing<TileBig, bf16_t>::DB; ++i) {
    const int row = tile_b_row<bf16_t>(wid, i, lane);
    const int h = row >> 7, j = (row >> 4) & 7, c = row & 15;   // column half, fragment block, lane
    const char* w;
    int64_t wr;
    if constexpr (MODE == kGemmSwiglu) {
      w = static_cast<const char*>((j & 1) ? a.B2 : a.B);
      wr = (int64_t)nt * 128 + h * 64 + 4 * c + (j >> 1);
    } else {
      w = static_cast<const char*>(a.B);
      wr = n0 + h * 128 + 64 * (j >> 2) + 4 * c + (j & 3);
    }
    b_ptr[i] = w + wr * K * 2 + tile_b_chunk<bf16_t>(row, lane) * 16;
  }
  f32x4 acc[4][8];
  tile_zero(acc);
  tile_main_loop<TileBig, bf16_t, 8>(acc, a_base, a_off, b_ptr, K / kTileK, smem, wid, lane);

  // ---- epilogue: acc[i][j][r] is tile row 64 wm + 16 g + 4 i + r of the
  // lane's block j
  const int64_t lrow = row0 + wm * 64 + 16 * g;
  if constexpr (MODE == kGemmSwiglu) {
    uint16_t* out = static_cast<uint16_t*>(a.C) + lrow * a.ldc + (int64_t)nt * 128 + wn * 64 + 4 * lc;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = tile_take(acc[i][j]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint2 v;
        v.x = pack_bf16x2(silu(x[0][r]) * x[1][r], silu(x[2][r]) * x[3][r]);
        v.y = pack_bf16x2(silu(x[4][r]) * x[5][r], silu(x[6][r]) * x[7][r]);
        if (lrow + 4 * i + r < M) *reinterpret_cast<uint2*>(out + (4 * i + r) * a.ldc) = v;
      }
    }
  } else {
    // 8 rows of the residual are read before the first of them is written:
    // read one by one, every row would wait for memory.  (With one K-step, K =
    // 64, the prologue's refetches may still be on their way to the LDS here;
    // loads return in order, so the wait for these rows covers them.)
    float* out = static_cast<float*>(a.C) + lrow * a.ldc + n0 + wn * 128 + 4 * lc;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f32x4 res[8][2];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool ok = lrow + 8 * h + u < M;       // past M the first row of C stands in
        const float* p = ok ? out + (8 * h + u) * a.ldc : static_cast<const float*>(a.C);
        res[u][0] = *reinterpret_cast<const f32x4*>(p);
        res[u][1] = *reinterpret_cast<const f32x4*>(p + 64);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        f32x4 x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = tile_take(acc[2 * h + q][j]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = 4 * q + r;
          float* p = out + (8 * h + u) * a.ldc;
          if (lrow + 8 * h + u < M) {
            *reinterpret_cast<f32x4*>(p) = res[u][0] + f32x4{x[0][r], x[1][r], x[2][r], x[3][r]};
            *reinterpret_cast<f32x4*>(p + 64) = res[u][1] + f32x4{x[4][r], x[5][r], x[6][r], x[7][r]};
          }
        }
      }
    }
  }
}

template <int MODE>
hipError_t run_gemm(const BlockGemmArgs& a, hipStream_t s) {
  if (a.M == 0) return hipSuccess;
  if (a.K < kTileK || a.K % kTileK || a.N % TileBig::ROWS) return hipErrorInvalidValue;
  const int tm = (int)((a.M + TileBig::ROWS - 1) / TileBig::ROWS), tn = a.N / TileBig::ROWS;
  hipLaunchKernelGGL((block_gemm_kernel<MODE>), dim3(tm * tn), dim3(kTileThreads<TileBig>), 0, s, a, tm, tn);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_block_gemm(int mode, const BlockGemmArgs& a, hipStream_t s) {
  if (mode == kGemmResid) return run_gemm<kGemmResid>(a, s);
  if (mode == kGemmSwiglu) return run_gemm<kGemmSwiglu>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace sr
