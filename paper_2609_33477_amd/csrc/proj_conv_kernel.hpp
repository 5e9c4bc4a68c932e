// Projection GEMM fused with the short causal conv, SiLU, key L2 norm, the
// decay / erase gates and the k | v conv tail (bf16 anchors; bf16 or fp8
// weights).
//
// What it computes (Section 2.1: the update's key, value and gates are linear
// maps of the layer input; Appendix A: a width-w depthwise conv over the q, k, v
// projections whose state is the last w-1 inputs):
//   P      = X [W_k; W_v; W_a; W_b]^T                       (fp32 accumulate)
//   k, v   = SiLU(sum_i cw[c][i] P[t-w+1+i][c])             (zero before the segment start)
//   k_hat  = k / sqrt(|k|^2 + eps)                           (per key head)
//   G      = log2 alpha = -exp(A_log) softplus(a + dt_bias) log2(e)
//   beta   = sigmoid(b)
// The projection never reaches HBM: each output tile (256 x 256 or 128 x 128) is
// finished in registers and only k_hat / v (bf16, head-major [H][T][d]), G and beta ([H_v][T],
// fp32) and the tail rows are written.
//
// Main loop: the tiles of sr_tile.hpp (8 waves of 64 x 128 or 4 of 32 x 128 on
// v_mfma_f32_16x16x32_bf16, K-steps of 64 through the LDS by DMA).  fp8 (E4M3)
// weights are staged as bytes and converted to bf16 after the fragment read
// (exact); the per-channel scale is folded into the conv taps (the conv is
// linear per column) and applied to the gate and tail values.  In a narrow
// last N-tile (the 2 H_v gate columns) waves skip the MFMAs and fragment reads
// of columns past N.
//
// Rectangular heads (RECT: OLMo-Hybrid's 96-wide keys and 192-wide values,
// Appendix A): each key head takes 128 output columns, its last 32 computed
// from a repeated weight row and zeroed before the conv, so the per-wave key
// norm is unchanged; keys stay in that padded layout, each value head is
// stored as two 96-column halves padded the same way (the scan runs them as
// two square units of 128), and every channel index into the caller's
// weights, scales, conv taps and tail goes through real_col.  The pad costs a tenth
// more MFMA work at OLMo's shape, against an unfused projection whose fp32
// rows went through HBM.
//
// Conv epilogue, in registers: M-tiles overlap by 3 rows (stride 253 or 125),
// so every output row's w-1 predecessors are in the tile (the first tile starts
// at row 0 and outputs all of its rows).  With MI = 4 (2 in the small tile)
// accumulator blocks of rows and WN = 2 (1) waves along N, lane l of wave w
// holds rows 16 MI (w / WN) + 4 MI (l / 16) + 0 .. 4 MI - 1 of 8 columns; the
// conv runs down those registers (the 3 rows above the lane's first come from the lane before it
// through a small LDS exchange), then SiLU.  The weight rows of a head are fed
// in the order that gives a lane 4 neighbouring columns of each 64 (2 of a
// 32-wide head), so 64 columns of a row leave as one 8-byte store per lane
// (128 contiguous bytes) and their taps arrive the same way.  A key's sum of
// squares is summed over the lane's columns and then across its 16 lanes by a
// DPP reduce-scatter; the inverse norms go back through the LDS.  Values need
// no norm and are stored as the conv produces them.  Waves with a row near a
// segment start or end (the conv tail) or past T take masked variants.  The
// segment info and conv taps are loaded when the main loop ends: held across
// it they would not fit beside the fragments in a wave's 128 VGPRs.
//
// Gate columns (no conv) keep their natural order and leave through a per-wave
// LDS transpose, so their head-major G and beta planes get stores of 64
// consecutive rows of a head.
//
// One launch covers up to kProjBatch layers of a call (same T and N): the
// grid holds the tiles of all of them, their m-tiles stacked for the walk
// above, and each block reads its layer's arguments from the kernel
// argument segment.  Blocks past the tiles compute the q part of the conv
// tail and the tail's leading zeros (tail_q.hpp): they need nothing the
// tiles write, so they run in the grid's last, partial round or on CUs the
// tiles leave idle.
#pragma once

#include "sr_tile.hpp"
#include "tail_q.hpp"

#include <algorithm>
#include <cstddef>
#include <type_traits>
#include <utility>

namespace sr {
namespace {

constexpr int HALO = 3;                          // rows M-tiles overlap by
// Epilogue areas in the drained stages: the last 3 rows of each lane's 8
// columns, the inverse norms of each group's rows (up to 4 heads per wave),
// and per wave a 16-column block of gate values.
template <typename C>
struct Epi {
  static constexpr int XB_BYTES = kTileThreads<C> * 24 * 4;
  static constexpr int INV_BYTES = C::WAVES * 4 * 4 * 4 * C::MI * 4;
  static constexpr int GATE_OFF = XB_BYTES + INV_BYTES, GATE_WAVE = 16 * 16 * C::MI * 4;
  static_assert(GATE_OFF + C::WAVES * GATE_WAVE <= kTileLds<C>, "epilogue areas");
};
constexpr float kLog2e = 1.4426950408889634f;

typedef __attribute__((address_space(3))) float lfloat;
typedef float nf32x4 __attribute__((ext_vector_type(4)));

// One step of a reduce-scatter over a group of 16 lanes: lanes whose bit BIT is
// b keep half b of the N values and add lane ^ 2^BIT's copy of it (DPP control
// CTRL, or ds_swizzle xor 4 when CTRL < 0).  Every partner is an exact xor, so
// a row's sum is the same tree whichever lane ends with it: its bits do not
// depend on the tile shape or the row's place in the tile.
template <int N, int BIT, int CTRL>
__device__ __forceinline__ void bfly_step(float* s, int lc) {
  const bool b = (lc >> BIT) & 1;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const float lo = s[i], hi = s[i + N / 2];
    const float send = b ? lo : hi, keep = b ? hi : lo;
    int r;
    if constexpr (CTRL < 0) r = __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, send), 0x101F);
    else r = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, send), CTRL, 0xF, 0xF, false);
    s[i] = keep + __builtin_bit_cast(float, r);
    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // bounds the scheduler's interleaving
  }
}

// OR of a 32-bit value over the 64 lanes (the result is wave-uniform)
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  auto op = [](uint32_t x, int y) { return x | (uint32_t)y; };
  v = op(v, __builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false));    // lane ^ 1
  v = op(v, __builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false));    // lane ^ 2
  v = op(v, __builtin_amdgcn_mov_dpp((int)v, 0x124, 0xF, 0xF, false));   // quad g -/+ 1
  v = op(v, __builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false));   // quads g -/+ 2, 3
  v = op(v, __builtin_amdgcn_ds_swizzle((int)v, 0x401F));                // lane ^ 16
  return op((uint32_t)__builtin_amdgcn_readlane((int)v, 0), __builtin_amdgcn_readlane((int)v, 32));
}

// f(integral_constant<int, i>) for i = 0 .. N-1, unrolled at compile time
// (register arrays indexed by i stay in registers)
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ void st_f4(lfloat* p, float x, float y, float z, float w) {
  *reinterpret_cast<__attribute__((address_space(3))) nf32x4*>(p) = nf32x4{x, y, z, w};
}

// bf16 scale of fp8 weight column n (selected without branches, one load)
__device__ __forceinline__ const uint16_t* col_scale_ptr(const ProjConvArgs& a, int n) {
  const uint16_t* p = static_cast<const uint16_t*>(a.seg[0].scale) + (n - a.seg[0].n0);
#pragma unroll
  for (int s = 1; s < 6; ++s)
    if (s < a.n_wseg && n >= a.seg[s].n0 && n < a.seg[s].n1) p = static_cast<const uint16_t*>(a.seg[s].scale) + (n - a.seg[s].n0);
  return p;
}
// Output column n -> the caller's channel order (weight rows, fp8 scales,
// conv taps, tail channels).  Square heads: n itself.  RECT: key head h's
// output columns h D + j map to channel h k_real + j (the pad columns
// j >= k_real to the head's last channel: their products are discarded),
// and the value and gate columns shift down by the keys' padding.
template <bool RECT, int D>
__device__ __forceinline__ int real_col(const ProjConvArgs& a, int n) {
  if constexpr (!RECT) return n;
  const int pad = (a.C_k / D) * (D - a.k_real);
  if (n >= a.C_k) return n - pad;
  const int h = n / D, j = n - h * D;
  return h * a.k_real + (j < a.k_real ? j : a.k_real - 1);
}
// per-output-column scale of fp8 weights (1 for bf16 weights)
template <typename TB>
__device__ __forceinline__ float col_scale(const ProjConvArgs& a, int n) {
  if constexpr (std::is_same<TB, fp8_t>::value) return bf16_bits_to_f32(*col_scale_ptr(a, n));
  return 1.f;
}

__device__ __forceinline__ float fast_sigmoid(float x) { return __builtin_amdgcn_rcpf(1.f + __expf(-x)); }
// max(x, 0) + ln(1 + e^-|x|) on the hardware exp and log: where e^-|x| is
// below half an ulp of 1 the second term drops out, an absolute error under
// 6e-8 in a value that then scales a log-decay
__device__ __forceinline__ float softplus(float x) { return fmaxf(x, 0.f) + __logf(1.f + __expf(-fabsf(x))); }

// N neighbouring bf16 (N = 2, 4) as one store
template <int N>
__device__ __forceinline__ void store_bf16(uint16_t* p, const uint32_t* v) {
  if constexpr (N == 4) *reinterpret_cast<uint2*>(p) = uint2{v[0], v[1]};
  else *reinterpret_cast<uint32_t*>(p) = v[0];
}

template <typename C, typename TB, int D, bool RECT>
__global__ __launch_bounds__(kTileThreads<C>, 1) void proj_conv_kernel(ProjConvBatch pb, int tiles_m, int tiles_n) {
  // The batch is the kernel's first argument: a layer's arguments are read
  // from the argument segment at a block-uniform offset.
  const char* kargs = (const char*)__builtin_amdgcn_kernarg_segment_ptr();
  auto layer_args = [&](int l) -> const ProjConvArgs& {
    return *reinterpret_cast<const ProjConvArgs*>(kargs + offsetof(ProjConvBatch, layer) + l * sizeof(ProjConvArgs));
  };
  if (pb.layer[0].err && *pb.layer[0].err) return;   // the call's table check failed: write nothing
  constexpr bool FP8 = std::is_same<TB, fp8_t>::value;
  __shared__ __attribute__((aligned(1024))) char smem_raw[kTileLds<C>];
  constexpr int MI = C::MI, U = 4 * MI;    // accumulator blocks and rows per lane
  const int n_tiles = pb.n_layers * tiles_m * tiles_n;
  if ((int)blockIdx.x >= n_tiles) {
    const int b = (int)blockIdx.x - n_tiles;
    int l = 0;
    while (l + 1 < pb.n_layers && b >= pb.tq_off[l + 1]) ++l;
    const TailArgs& tq = layer_args(l).tq;
    const int bl = b - pb.tq_off[l], gx = tail_q_grid_x(tq);
    tail_q_block<TB, C::WAVES, kTileLds<C>>(tq, bl % gx, bl / gx, smem_raw);
    return;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int wm = wid / C::WN, wn = wid % C::WN;                // 16 MI-row x 128-column sub-tile
  const int g = lane >> 4, lc = lane & 15;
  // m-tiles of the layers stacked: the XCD-aware walk runs over all of them
  int mt, nt;
  tile_of(blockIdx.x, pb.n_layers * tiles_m, tiles_n, mt, nt);
  const int layer = mt / tiles_m;
  mt -= layer * tiles_m;
  const ProjConvArgs& a = layer_args(layer);
  const int64_t row0 = (int64_t)mt * (C::ROWS - HALO);   // tile row 0
  const int hal = mt ? HALO : 0;                   // rows of the tile that are not output
  const int n0 = nt * C::ROWS;
  const int K = a.K;
  const int64_t T = a.T;

  // Output columns.  The wave's 128 are NG groups of GW (64, or a 32-wide
  // head); of a conv or z group a lane holds JG neighbouring columns, past
  // them (the gates) 16-column blocks in natural order.  Fragment block j,
  // lane c of column half h:
  constexpr int NH = 128 / D, JG = D >= 64 ? 4 : 2, GW = 16 * JG, GH = D / GW;
  auto group0 = [&](int h, int j) { return n0 + 128 * h + (j / JG) * GW; };   // first column of the block's group
  auto column = [&](int h, int j, int c) {
    const int nb = group0(h, j);
    return nb < a.C_z ? nb + JG * c + j % JG : nb + 16 * (j % JG) + c;
  };

  // ------------------------------------------------------------ main loop
  f32x4 acc[MI][8];
  tile_zero(acc);
  {
    const char* a_base = static_cast<const char*>(a.A) + row0 * K * 2;
    uint32_t a_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = tile_a_row(wid, i, lane);
      const int64_t last = T - 1 - row0;             // rows past T are never output
      a_off[i] = (uint32_t)((row < last ? row : (int)last) * (K * 2) + tile_a_chunk<C>(row, lane) * 16);
    }
    const char* b_ptr[TileRing<C, TB>::DB];
#pragma unroll
    for (int i = 0; i < TileRing<C, TB>::DB; ++i) {
      const int row = tile_b_row<TB>(wid, i, lane);
      const int n_out = column(row >> 7, (row >> 4) & 7, row & 15);
      const int n = real_col<RECT, D>(a, n_out < a.N ? n_out : a.N - 1);
      const char* p = static_cast<const char*>(a.seg[0].ptr);
#pragma unroll
      for (int s = 0; s < 6; ++s)
        if (s < a.n_wseg && n >= a.seg[s].n0 && n < a.seg[s].n1)
          p = static_cast<const char*>(a.seg[s].ptr) + (int64_t)(n - a.seg[s].n0) * K * Elem<TB>::bytes;
      b_ptr[i] = p + tile_b_chunk<TB>(row, lane) * 16;
    }
    const int n_wave = a.N - (n0 + wn * 128);        // valid columns of this wave's 128
    const int KT = K / kTileK;
    if (n_wave > 64) tile_main_loop<C, TB, 8>(acc, a_base, a_off, b_ptr, KT, smem_raw, wid, lane);
    else if (n_wave > 0) tile_main_loop<C, TB, 4>(acc, a_base, a_off, b_ptr, KT, smem_raw, wid, lane);
    else tile_main_loop<C, TB, 0>(acc, a_base, a_off, b_ptr, KT, smem_raw, wid, lane);
  }

  // ------------------------------------------------------------ epilogue
  // The share of this lane: tile rows rbase .. rbase + U - 1 of columns
  // column(wn, j, lc).  Its inputs: the segment position and rows left of the
  // first row, the raw conv taps of the columns and their fp8 scales.
  const int rbase = wm * 4 * U + U * g;
  const int64_t t0 = row0 + rbase;
  int pos0 = -1, rem0 = 0;
  if (t0 < T) {
    const int2 pr = *reinterpret_cast<const int2*>(a.info + t0);
    pos0 = pr.x;
    rem0 = pr.y;
  }
  // RECT: a key head's pad columns (from k_real on) hold products of a
  // repeated weight row; they enter neither the conv outputs, the tail, nor
  // the key's norm.  k_real is a multiple of JG: a lane's group is all pad or
  // none.
  const bool rect_k = RECT && n0 + 128 * wn < a.C_k;
  auto pad_lane = [&](int q) { return rect_k && GW * (q % GH) + JG * lc >= a.k_real; };
  // With w = 4 and an aligned table a column's conv taps, [row t-3, t-2, t-1,
  // t], are 8 (bf16) or 16 (fp32) bytes and the lane's JG columns of a group
  // neighbours; else they are read one by one.
  const int tap_mode = (a.w == 4 && (reinterpret_cast<uintptr_t>(a.conv_w) & 15) == 0) ? (a.conv_bf16 ? 1 : 2) : 0;
  // fp8: a q, k, v or z head's columns are one weight's, so one search, on the
  // wave's scalars, finds the scales of the head at column nb.  (A search per
  // fragment block and lane cost 4 us a tile: 2 layers of 14.8K rows, N = 7770,
  // D = 256, 372 us so and 340 as it is.)
  auto head_scales = [&](int nb) -> const uint16_t* {
    if constexpr (FP8) return col_scale_ptr(a, real_col<RECT, D>(a, nb));
    return nullptr;
  };
  auto scale = [&](const uint16_t* head, int c) {   // of the head's channel c
    if constexpr (FP8) return bf16_bits_to_f32(head[c]);
    return 1.f;
  };
  tile_drain();
  tile_pin(acc);

  // acc[i][j][r]: the raw projection of row rbase + 4 i + r, fragment block j.
  // The conv runs down a lane's registers; only the 3 rows before rbase come
  // from another lane (16 lanes down in this wave, or the last group of the
  // wave above), through the LDS.
  lfloat* XB = (lfloat*)smem_raw;
  lfloat* INV = (lfloat*)(smem_raw + Epi<C>::XB_BYTES);
  {
    lfloat* p = XB + (wid * 64 + lane) * 24;
    f32x4 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = tile_take(acc[MI - 1][j]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      st_f4(p + 8 * k, x[0][1 + k], x[1][1 + k], x[2][1 + k], x[3][1 + k]);
      st_f4(p + 8 * k + 4, x[4][1 + k], x[5][1 + k], x[6][1 + k], x[7][1 + k]);
    }
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  // rows rbase - 3 .. - 1 of the lane's columns, [3][8] (unused above the tile)
  const lfloat* above = XB + (g ? wid * 64 + lane - 16 : (wm ? (wid - C::WN) * 64 + lane + 48 : lane)) * 24;

  const int w1 = a.w - 1;
  // Fast case: all U rows lie inside one segment, at least w - 1 rows past
  // its start (or the first of them are halo rows) and more than w - 1 rows
  // before its end (no tail rows).  Otherwise the masks are built from the
  // rows' segment info.
  const bool fast = rem0 >= U + w1 && (pos0 >= w1 || (rbase == 0 && hal));
  const bool wave_fast = __builtin_amdgcn_ballot_w64(!fast) == 0;
  // bit u of m1 / m2 / m3: row u may use row u-1 / u-2 / u-3 (same segment);
  // outm: row u is an output; tailm: row u is one of its segment's last w-1
  // rows (the conv state)
  uint32_t m1 = ~0u, m2 = ~0u, m3 = ~0u, outm = rbase || !hal ? ~0u : ~7u, tailm = 0u;
  if (!wave_fast && !fast) {
    m1 = m2 = m3 = outm = 0u;
#pragma unroll
    for (int b = 0; b < U / 8; ++b) {
      int2 pr[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int64_t t = t0 + 8 * b + k;
        pr[k] = int2{-1, 0};
        if (t < T) pr[k] = *reinterpret_cast<const int2*>(a.info + t);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int u = 8 * b + k;
        const uint32_t bit = 1u << u;
        if (pr[k].x >= 1) m1 |= bit;
        if (pr[k].x >= 2) m2 |= bit;
        if (pr[k].x >= 3) m3 |= bit;
        if (pr[k].x >= 0 && rbase + u >= hal) {
          outm |= bit;
          if (pr[k].y <= w1) tailm |= bit;
        }
      }
    }
  }
  if (a.tail == nullptr) tailm = 0u;
  const bool tail_bf16 = a.tail_bf16 != 0;
  const uint32_t tail_rows = wave_fast ? 0u : wave_or(tailm);   // rows some lane keeps for the tail

  static_for<NH>([&](auto hd_c) {
    constexpr int hd = decltype(hd_c)::value;
    const int nb = n0 + 128 * wn + hd * D;   // first column of the head (wave-uniform)
    if (nb >= a.N) {
    } else if (nb < a.C_kv) {
      // ---- q, k or v head: conv, SiLU, (queries and keys) L2 norm
      const bool is_q = nb < a.C_q;
      const bool is_k = nb < a.C_k;   // q or k: normalised
      const uint16_t* const head_sc = head_scales(nb);
      const int rn = real_col<RECT, D>(a, nb);   // the head's first channel
      // destinations of the lane's JG columns of each group, row rbase
      const int hh = is_q ? nb / D : (is_k ? (nb - a.C_q) / D : (nb - a.C_k) / D);
      uint16_t* const head = static_cast<uint16_t*>(is_q ? a.Qbuf : (is_k ? a.Kbuf : a.Vbuf)) + ((int64_t)hh * T + t0) * D;
      uint16_t* dst[GH];
      bool vpad[GH];
#pragma unroll
      for (int gi = 0; gi < GH; ++gi) {
        dst[gi] = head + GW * gi + JG * lc;
        vpad[gi] = false;
        // RECT values: value head h (v_head = 2 k_real columns) is stored as
        // two halves 2 h + e of k_real columns, each padded to D like a key
        // head ([2 H_v][T][D]); the lanes of a half's last D - k_real columns
        // also write its pad columns (zeros).
        if (RECT && !is_k) {
          const int c = nb + GW * gi - a.C_k + JG * lc, h = c / a.v_head, c0 = c - h * a.v_head;
          const int e = c0 / a.k_real, col = c0 - e * a.k_real;
          dst[gi] = static_cast<uint16_t*>(a.Vbuf) + ((int64_t)(2 * h + e) * T + t0) * D + col;
          vpad[gi] = col + (D - a.k_real) >= a.k_real;
        }
      }
      auto put = [&](int gi, int u, const uint32_t* v) { store_bf16<JG>(dst[gi] + u * D, v); };
      // store of row u.  SIMPLE: only the tile's first rows may not be output
      auto row_out = [&](int gi, int u, const uint32_t* v, auto simple_tag) {
        constexpr bool SIMPLE = decltype(simple_tag)::value;
        if (SIMPLE && u >= HALO) put(gi, u, v);
        else if ((outm >> u) & 1u) put(gi, u, v);
      };
      float ss[U];
      // One group's columns.  Rows in descending order, so each x is
      // overwritten only after the three rows after it have read it; one row
      // per scheduling group (the scheduler would otherwise hoist every row's
      // exp and keep all conv results live at once).  NORM keeps y in place
      // of x and sums its squares; else y leaves at once.
      auto conv_rows = [&](auto gi_c, auto norm_tag) {
        constexpr bool NORM = decltype(norm_tag)::value;
        constexpr int gi = decltype(gi_c)::value, q = hd * GH + gi, j0 = q * JG;
        // conv taps (row t - d) with the fp8 column scale and -log2(e) folded
        // in: the conv yields z = -log2(e) c, so e^-c = 2^z and
        // SiLU(c) = z / (-log2(e) (1 + 2^z)).  Loaded per group: all of them
        // up front would spill.
        float tp[JG][4];
        const bool pad = pad_lane(q);
        {
          // first channel of the lane's JG (a pad lane: the head's last JG)
          const int ch0 = pad ? real_col<RECT, D>(a, nb) + a.k_real - JG : real_col<RECT, D>(a, nb + GW * gi + JG * lc);
          if (tap_mode == 1) {
            const uint4* p = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.conv_w) + (int64_t)ch0 * 4);
#pragma unroll
            for (int jj = 0; jj < JG; jj += 2) {
              const uint4 v = p[jj / 2];
              const uint32_t t[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
              for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  const uint32_t pair = t[2 * e + ((3 - d) >> 1)];
                  tp[jj + e][d] = __uint_as_float((d & 1) ? pair << 16 : pair & 0xffff0000u);
                }
            }
          } else if (tap_mode == 2) {
            const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(a.conv_w) + (int64_t)ch0 * 4);
#pragma unroll
            for (int jj = 0; jj < JG; ++jj) {
              const float4 v = p[jj];
              tp[jj][3] = v.x;
              tp[jj][2] = v.y;
              tp[jj][1] = v.z;
              tp[jj][0] = v.w;
            }
          } else {
#pragma unroll
            for (int jj = 0; jj < JG; ++jj)
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                tp[jj][d] = 0.f;
                if (d < a.w) {
                  const int64_t i = (int64_t)(ch0 + jj) * a.w + a.w - 1 - d;   // tap of row t - d
                  tp[jj][d] = a.conv_bf16 ? bf16_bits_to_f32(static_cast<const uint16_t*>(a.conv_w)[i])
                                          : static_cast<const float*>(a.conv_w)[i];
                }
              }
          }
#pragma unroll
          for (int jj = 0; jj < JG; ++jj) {
            const float sc = scale(head_sc, ch0 - rn + jj) * -kLog2e;
#pragma unroll
            for (int d = 0; d < 4; ++d) tp[jj][d] *= sc;
          }
        }
        f32x4 x[JG], up[JG];       // rows 4 i .. 4 i + 3, and the four above them
#pragma unroll
        for (int jj = 0; jj < JG; ++jj) up[jj] = tile_take(acc[MI - 1][j0 + jj]);
#pragma unroll
        for (int i = MI - 1; i >= 0; --i) {
#pragma unroll
          for (int jj = 0; jj < JG; ++jj) {
            x[jj] = up[jj];
            if (i > 0) {
              up[jj] = tile_take(acc[i > 0 ? i - 1 : 0][j0 + jj]);
            } else {
#pragma unroll
              for (int k = 0; k < 3; ++k) up[jj][1 + k] = rbase == 0 ? 0.f : above[8 * k + j0 + jj];
            }
          }
          f32x4 y[JG];
          auto four_rows = [&](auto mask_tag) {
            constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
            for (int r = 3; r >= 0; --r) {
              const int u = 4 * i + r;
              float sq = 0.f;
              static_for<JG>([&](auto jj_c) {
                constexpr int jj = decltype(jj_c)::value;
                const float x1 = r >= 1 ? x[jj][(r + 3) & 3] : up[jj][3];
                const float x2 = r >= 2 ? x[jj][(r + 2) & 3] : up[jj][(r + 2) & 3];
                const float x3 = r >= 3 ? x[jj][0] : up[jj][(r + 1) & 3];
                float z = tp[jj][0] * x[jj][r];
                z = fmaf(tp[jj][1], MASK && !((m1 >> u) & 1u) ? 0.f : x1, z);
                z = fmaf(tp[jj][2], MASK && !((m2 >> u) & 1u) ? 0.f : x2, z);
                z = fmaf(tp[jj][3], MASK && !((m3 >> u) & 1u) ? 0.f : x3, z);
                if (RECT && NORM) z = pad ? 0.f : z;
                float v = z * __builtin_amdgcn_rcpf(fmaf(__builtin_amdgcn_exp2f(z), -kLog2e, -kLog2e));
                if (NORM) asm volatile("" : "+v"(v));   // materialise y here, not at the stores
                y[jj][r] = v;
                sq = fmaf(v, v, sq);
              });
              if constexpr (NORM) {
                ss[u] = gi ? ss[u] + sq : sq;
              } else {
                uint32_t v[JG / 2];
#pragma unroll
                for (int h = 0; h < JG / 2; ++h) v[h] = pack_bf16x2(y[2 * h][r], y[2 * h + 1][r]);
                row_out(gi, u, v, std::integral_constant<bool, !MASK>{});
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          };
          if (wave_fast) four_rows(std::false_type{});
          else four_rows(std::true_type{});
          if constexpr (NORM) {
#pragma unroll
            for (int jj = 0; jj < JG; ++jj) tile_put(acc[i][j0 + jj], y[jj]);
          }
        }
      };
      if (tail_rows) {
        // the raw projection of the segment's last w-1 rows is the conv state
        static_for<GH>([&](auto gi_c) {
          constexpr int gi = decltype(gi_c)::value, q = hd * GH + gi, j0 = q * JG;
          const bool pad = pad_lane(q);
          const int ch0 = pad ? 0 : real_col<RECT, D>(a, nb + GW * gi + JG * lc);
          float sc[JG];
#pragma unroll
          for (int jj = 0; jj < JG; ++jj) sc[jj] = scale(head_sc, (pad ? 0 : ch0 - rn) + jj);
          static_for<U>([&](auto u_c) {
            constexpr int u = decltype(u_c)::value;
            if ((tail_rows >> u) & 1u) {
              float v[JG];
#pragma unroll
              for (int jj = 0; jj < JG; ++jj) v[jj] = tile_take(acc[u >> 2][j0 + jj])[u & 3] * sc[jj];
              if (((tailm >> u) & 1u) && !pad) {
                const RowInfo ri = a.info[t0 + u];
                if (ri.slot >= 0) {
                  const int64_t at = ((int64_t)ri.slot * a.c_tail + a.tail_kv_off + ch0) * w1 + (w1 - ri.rem);
                  if (tail_bf16) {
#pragma unroll
                    for (int jj = 0; jj < JG; ++jj) static_cast<uint16_t*>(a.tail)[at + jj * w1] = f32_to_bf16_bits(v[jj]);
                  } else {
#pragma unroll
                    for (int jj = 0; jj < JG; ++jj) static_cast<float*>(a.tail)[at + jj * w1] = v[jj];
                  }
                }
              }
            }
          });
        });
      }
      if (!is_k) {
        static_for<GH>([&](auto gi_c) { conv_rows(gi_c, std::false_type{}); });
        if constexpr (RECT) {
          const uint32_t z[2] = {0u, 0u};
#pragma unroll
          for (int gi = 0; gi < GH; ++gi)
            if (vpad[gi]) {
#pragma clang loop unroll(disable)
              for (int u = 0; u < U; ++u)
                if ((outm >> u) & 1u) store_bf16<JG>(dst[gi] + u * D + (D - a.k_real), z);
            }
        }
      } else {
        static_for<GH>([&](auto gi_c) { conv_rows(gi_c, std::true_type{}); });
        // sum of squares of each row over the head's D columns: over the
        // lane's columns above, then across the group's 16 lanes
        // (reduce-scatter: lane lc ends with row bitrev(lc) of U; with 8 rows
        // the last step leaves lanes lc and lc ^ 8 the same row)
        bfly_step<U, 0, 0xB1>(ss, lc);     // quad_perm 1,0,3,2: lane ^ 1
        bfly_step<U / 2, 1, 0x4E>(ss, lc); // quad_perm 2,3,0,1: lane ^ 2
        bfly_step<U / 4, 2, -1>(ss, lc);   // swizzle: lane ^ 4
        if constexpr (U == 16) bfly_step<2, 3, 0x128>(ss, lc);   // row_ror 8: lane ^ 8
        else ss[0] += __builtin_bit_cast(
            float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, ss[0]), 0x128, 0xF, 0xF, false));
        lfloat* ivp = INV + ((wid * 4 + g) * NH + hd) * U;
        ivp[__builtin_bitreverse32((uint32_t)lc) >> (U == 16 ? 28 : 29) & (U - 1)] =
            (is_q ? a.q_scale : 1.f) * __builtin_amdgcn_rsqf(ss[0] + a.eps);
        // LDS operations of one wave complete in order: the reads below see
        // every lane's writes
        static_for<GH>([&](auto gi_c) {
          constexpr int gi = decltype(gi_c)::value, j0 = (hd * GH + gi) * JG;
          auto out_rows = [&](auto simple_tag) {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
              const nf32x4 iv = *reinterpret_cast<const __attribute__((address_space(3))) nf32x4*>(ivp + 4 * i);
              f32x4 y[JG];
#pragma unroll
              for (int jj = 0; jj < JG; ++jj) y[jj] = tile_take(acc[i][j0 + jj]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                uint32_t v[JG / 2];
#pragma unroll
                for (int h = 0; h < JG / 2; ++h) v[h] = pack_bf16x2(y[2 * h][e] * iv[e], y[2 * h + 1][e] * iv[e]);
                row_out(gi, 4 * i + e, v, simple_tag);
              }
            }
          };
          if (wave_fast) out_rows(std::true_type{});
          else out_rows(std::false_type{});
        });
      }
    } else if (nb < a.C_z) {
      // ---- z head (output gate): the raw projection, bf16, head-major
      static_for<GH>([&](auto gi_c) {
        constexpr int gi = decltype(gi_c)::value, j0 = (hd * GH + gi) * JG;
        uint16_t* dst = static_cast<uint16_t*>(a.Zbuf) + ((int64_t)((nb - a.C_kv) / D) * T + t0) * D + GW * gi + JG * lc;
        float sc[JG];
#pragma unroll
        for (int jj = 0; jj < JG; ++jj) sc[jj] = scale(head_scales(nb), GW * gi + JG * lc + jj);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          f32x4 x[JG];
#pragma unroll
          for (int jj = 0; jj < JG; ++jj) x[jj] = tile_take(acc[i][j0 + jj]) * sc[jj];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            uint32_t v[JG / 2];
#pragma unroll
            for (int h = 0; h < JG / 2; ++h) v[h] = pack_bf16x2(x[2 * h][e], x[2 * h + 1][e]);
            if ((outm >> (4 * i + e)) & 1u) store_bf16<JG>(dst + (4 * i + e) * D, v);
          }
        }
      });
    } else {
      // ---- gate columns: G = log2 alpha from a, beta from b (no conv).  G
      // and beta are head-major ([H_v][T]): each 16-column block of raw
      // projections is transposed through the wave's LDS area (column pitch
      // 16 MI rows, 16-byte chunks XOR-swizzled by the column: writes of 16
      // columns and reads of one fall on distinct banks), then one column at
      // a time -- its gate wave-uniform -- is finished and stored, 16 MI
      // rows of one head per store.  Every row of the tile from hal on that lies
      // before T is an output (gates do not depend on the segments).
      lfloat* tw = (lfloat*)(smem_raw + Epi<C>::GATE_OFF + wid * Epi<C>::GATE_WAVE);
      const int r = wm * 16 * MI + lane;           // the tile row this lane stores
      const bool st_ok = lane < 16 * MI && r >= hal && row0 + r < T;
      static_for<D / 16>([&](auto jj_c) {
        constexpr int jj = decltype(jj_c)::value, j = hd * (D / 16) + jj;
        const int nb_j = nb + 16 * jj;             // first column of the block (wave-uniform)
        if (nb_j < a.N) {
#pragma unroll
          for (int i = 0; i < MI; ++i) {
            const f32x4 v = tile_take(acc[i][j]);
            st_f4(tw + lc * 16 * MI + (((MI * g + i) ^ (lc & (4 * MI - 1))) << 2), v[0], v[1], v[2], v[3]);
          }
          // LDS operations of one wave complete in order: the reads below
          // see every lane's writes
          const int nc = a.N - nb_j < 16 ? a.N - nb_j : 16;
          // lane c: the scale of column c (one load per block: a load per
          // column waits for the stores of the one before; the shape above
          // 340 us so, 301 as it is)
          const float sc_lane = col_scale<TB>(a, real_col<RECT, D>(a, nb_j + (lc < nc ? lc : nc - 1)));
#pragma clang loop unroll(disable)
          for (int c = 0; c < nc; ++c) {
            const int n = nb_j + c;
            const bool is_a = n < a.C_z + a.H_v;
            const int hv = is_a ? n - a.C_z : n - a.C_z - a.H_v;
            const float sc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sc_lane), c));
            const float x = tw[c * 16 * MI + ((((lane >> 2) ^ c) & (4 * MI - 1)) << 2) + (lane & 3)] * sc;
            const float v = is_a ? -__expf(a.a_log[hv]) * kLog2e * softplus(x + a.dt_bias[hv]) : fast_sigmoid(x);
            if (st_ok) ((is_a ? a.Gbuf : a.Bbuf) + (int64_t)hv * T)[row0 + r] = v;
          }
        }
      });
    }
  });
}

// tiles of rows along M: the first outputs all of its rows, every later one
// HALO fewer
int tiles_m(int64_t T, int rows) {
  const int step = rows - HALO;
  return T <= 0 ? 0 : 1 + (int)((std::max<int64_t>(T - rows, 0) + step - 1) / step);
}

template <typename C, typename TB, int D, bool RECT>
hipError_t run_tile(const ProjConvBatch& b, hipStream_t s) {
  const ProjConvArgs& a = b.layer[0];
  const int tm = tiles_m(a.T, C::ROWS), tn = (a.N + C::ROWS - 1) / C::ROWS;
  const int blocks = b.n_layers * tm * tn + b.tq_off[b.n_layers];
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((proj_conv_kernel<C, TB, D, RECT>), dim3(blocks), dim3(kTileThreads<C>), 0, s, b, tm, tn);
  return hipGetLastError();
}

template <typename TB, int D, bool RECT = false>
hipError_t run(const ProjConvBatch& b, hipStream_t s) {
  const ProjConvArgs& a = b.layer[0];
  if (a.K < kTileK || a.K % kTileK) return hipErrorInvalidValue;
  // Tile shape.  A 256 x 256 tile holds a CU alone, two 128 x 128 tiles share
  // one, so a round of the card is cus big or 2 cus small ones; a small round
  // takes 0.72 of a big one for half its work.  Measured on 256 CUs (us, big /
  // small): 75 / 147 tiles (D = 2560) 63 / 42, 125 / 441 70 / 52, 225 / 735
  // 82 / 83, 375 / 1323 143 / 136, 500 / 1764 165 / 182, 825 / 3234 284 / 297;
  // D = 2048: 153 / 561 62 / 66, 289 / 1089 118 / 103; D = 5120: 99 / 325
  // 112 / 80, 165 / 585 118 / 132, 297 / 1105 229 / 205.
  // So small tiles where one round holds them all, or where the big ones would
  // leave the last of two or more rounds mostly idle.  Those are kernels of bf16
  // square heads; for the other forms whole calls were timed with either tile
  // forced: of 268 shapes (bf16 and fp8; square heads, 96 x 192 ones, and 196 to
  // 516 columns with up to 120K rows) the rule's choice was within 1% of the
  // better one at 254 and 5% behind at worst (big / small, us): fp8, 16 key and
  // 48 value heads of 128: D = 5120, 1024 rows 150 / 164, 4096 rows 463 / 464; D
  // = 1024, 4096 rows 245 / 240 (big taken); 96 x 192: 30 heads, D = 3840, 1024
  // rows 136 / 148, 4096 rows 412 / 431; 8 heads, 4 layers, 2048 rows 155 / 148
  // (big taken, the worst); 196 columns, 20K rows 181 / 159, 120K rows 284 /
  // 320.
  const int64_t cus = device_cus();
  const int64_t big = (int64_t)b.n_layers * tiles_m(a.T, TileBig::ROWS) * ((a.N + 255) / 256);
  const int64_t small = (int64_t)b.n_layers * tiles_m(a.T, TileSmall::ROWS) * ((a.N + 127) / 128);
  const int64_t rounds = (big + cus - 1) / cus;
  if (small <= 2 * cus || (rounds > 1 && 72 * small < 100 * 2 * cus * rounds))
    return run_tile<TileSmall, TB, D, RECT>(b, s);
  return run_tile<TileBig, TB, D, RECT>(b, s);
}

template <typename TB>
hipError_t by_head(int d, const ProjConvBatch& a, hipStream_t s) {
  if (a.layer[0].k_real > 0) {
    // rectangular heads: key heads padded to 128 columns, no q or z columns
    for (int l = 0; l < a.n_layers; ++l) {
      const ProjConvArgs& x = a.layer[l];
      if (x.k_real != a.layer[0].k_real || x.v_head != a.layer[0].v_head || x.k_real % 32 || x.k_real >= 128 ||
          x.k_real + 32 != 128 || x.v_head != 2 * x.k_real || x.C_q != 0 || x.C_z != x.C_kv || x.C_k % 128 ||
          (x.C_kv - x.C_k) % 128)
        return hipErrorInvalidValue;
    }
    return d == 128 ? run<TB, 128, true>(a, s) : hipErrorInvalidValue;
  }
  switch (d) {
    case 32: return run<TB, 32>(a, s);
    case 64: return run<TB, 64>(a, s);
    case 128: return run<TB, 128>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace sr
