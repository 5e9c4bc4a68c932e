// The 256 x 256 bf16 tile main loop of the projection and the block GEMMs
// (C = A B^T, fp32 accumulation; A bf16, B bf16 or fp8 E4M3 rows).
//
// What bounds it: matrix issue and, at full load, the card's power limit, so
// the loop is shaped to move as few bits per product as it can.
//  - v_mfma_f32_16x16x32_bf16: it reads and writes half the accumulator bits
//    per multiply-add of the 32x32x16 form, which at the same issue rate
//    settled at a lower clock.
//  - K-steps of 64: every row a DMA fetches is a whole 128-byte line (bf16),
//    half the L2 requests of 64-byte rows.
//  - 8 waves of 64 x 128 (two per SIMD), accumulators in AGPRs.  4 waves of
//    128 x 128 read a third fewer fragments and run the plain loop 0 to 2%
//    faster, but leave one wave per SIMD for everything around it, and one
//    wave issues a VALU instruction every ~5 cycles: the projection's
//    epilogue took 25K cycles a tile that way, a fifth of its time.
// Plain GEMM of the varlen projection's shape (36864 x 6144 x 2560, normal
// inputs, one card): 32x32x16 with K-steps of 32 1029 us, with K-steps of 64
// (4 waves) 965 us, the same on 16x16x32 868 us; the hand-over moved into the
// first half step and the DMAs spread over the step 808 us (1.44 PFLOP/s; 4
// waves 807 us).
//
// LDS (160 KB).  bf16 B: a ring of five 32 KB half stages (A or B of one
// K-step), A(k) in slot 2k mod 5, B(k) in 2k + 1 mod 5.  fp8 B: three 32 KB A
// slots and four 16 KB B slots.  Rows keep their 16-byte chunks XOR-swizzled
// so that 16 lanes of a fragment read fall on 16 distinct bank groups.
//
// One hand-over (wait + barrier) per K-step, after MFMA kBarrierAt of the
// first half step: by then every wave has read its second-half fragments, so
// the step's slots are free, and the next step's rows have landed.  The
// refills follow it, one DMA per few MFMAs (issued closer together they cost
// up to 6%), until the step's end.
//
// The MFMAs are inline asm with AGPR accumulators: left to itself the
// compiler put part of the accumulators in VGPRs and copied them around the
// loop (180 to 500 moves per K-step, half the speed).  The asm hides them
// from its hazard bookkeeping, so the code keeps the distances itself: the
// fp8 conversions feeding an MFMA are issued at least four instructions before it,
// and the loop ends by letting the last products land before anyone reads them.
#pragma once

#include <type_traits>

#include "sr_device.hpp"

namespace sr {

constexpr int kTileM = 256, kTileN = 256, kTileK = 64;
constexpr int kTileThreads = 512, kTileWaves = 8;
constexpr int kTileLds = 160 * 1024;
constexpr int kTileHalf = 256 * 128;    // bytes of one K-step of A (and of bf16 B)
constexpr int kBarrierAt = 28;

typedef __attribute__((address_space(3))) char tile_lds;
typedef unsigned int tile_u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 tile_ld16(const tile_lds* p) {
  return __builtin_bit_cast(uint4, *reinterpret_cast<const __attribute__((address_space(3))) tile_u32x4*>(p));
}

// B storage: row bytes per K-step, 1 KB DMA blocks per wave, how many K-steps
// ahead B is fetched, DMA spacing in MFMAs, DMAs outstanding at a hand-over
// once the next step has landed, and before the first step
template <typename TB> struct TileB;
template <> struct TileB<bf16_t> {
  static constexpr int ROW = 128, DMAS = 4, AHEAD = 2, SPACING = 4, PENDING = 4, PENDING0 = 12;
};
template <> struct TileB<fp8_t> {
  static constexpr int ROW = 64, DMAS = 2, AHEAD = 4, SPACING = 5, PENDING = 6, PENDING0 = 14;
};
constexpr int kTileAheadA = 3;          // K-steps ahead of A

// Chunk swizzles: LDS row r keeps 16-byte chunk c of its K-step at c ^ swz(r).
// An A fragment reads rows 16 (m / 4) + 4 i + m % 4 (m = lane % 16), a B one 16
// consecutive rows.
__device__ __forceinline__ int tile_swz_a(int r) { return ((r >> 1) & 1) | ((r >> 3) & 6); }
template <typename TB>
__device__ __forceinline__ int tile_swz_b(int r) {
  return std::is_same<TB, bf16_t>::value ? (r >> 1) & 7 : (r >> 2) & 3;
}

// Tile row / chunk that lane `lane` of wave `wid` fetches with its DMA i (the
// LDS side is linear: A block wid * 4 + i, 16 bytes per lane)
__device__ __forceinline__ int tile_a_row(int wid, int i, int lane) { return (wid * 4 + i) * 8 + (lane >> 3); }
__device__ __forceinline__ int tile_a_chunk(int row, int lane) { return (lane & 7) ^ tile_swz_a(row); }
template <typename TB>
__device__ __forceinline__ int tile_b_row(int wid, int i, int lane) {
  return std::is_same<TB, bf16_t>::value ? (wid * 4 + i) * 8 + (lane >> 3) : (wid * 2 + i) * 16 + (lane >> 2);
}
template <typename TB>
__device__ __forceinline__ int tile_b_chunk(int row, int lane) {
  return std::is_same<TB, bf16_t>::value ? (lane & 7) ^ tile_swz_b<TB>(row) : (lane & 3) ^ tile_swz_b<TB>(row);
}

// Accumulators of wave (wm, wn) = (wid / 2, wid % 2): acc[i][j][r] of lane l
// is tile row 64 wm + 16 (l / 16) + 4 i + r -- 16 consecutive rows per lane
// over i and r -- and LDS row 128 wn + 16 j + l % 16 of B.
//
// hardware block id -> (m tile, n tile): contiguous runs per XCD (blocks are
// dealt round-robin to the 8 XCDs), walked in groups of 4 m-tiles, so the 32
// tiles an XCD runs at once span 4 A and 8 B panels (groups of 2, 4 and 8
// took 833, 817 and 817 us on the shape above; of 1 and 16 more)
__device__ __forceinline__ void tile_of(int b, int tm, int tn, int& mt, int& nt) {
  const int nb = tm * tn;
  const int per = nb / 8, rem = nb % 8;
  const int x = b % 8, loc = b / 8;
  const int t = x * per + (x < rem ? x : rem) + loc;
  constexpr int GM = 4;
  const int grp = t / (GM * tn);
  const int first = grp * GM;
  const int gs = (tm - first) < GM ? (tm - first) : GM;
  const int idx = t - grp * GM * tn;
  mt = first + idx % gs;
  nt = idx / gs;
}

// Accumulators stay in AGPRs across the epilogue too (moved to VGPRs as a
// whole they spill): tile_pin() ties them there, then four rows of a column
// block at a time are copied out by tile_take() and back by tile_put().
__device__ __forceinline__ void tile_pin(f32x4 (&acc)[4][8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) asm volatile("" : "+a"(acc[i][j]));
}
__device__ __forceinline__ f32x4 tile_take(const f32x4& a) {
  f32x4 t = a;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ void tile_put(f32x4& a, f32x4 v) {
  asm volatile("" : "+a"(v));
  a = v;
}

// The main loop.  a_base + a_off[i] and b_ptr[i]: this lane's source of DMA i
// at K = 0 (rows outside the operands clamped by the caller).  NJ: 16-column
// blocks of B this wave multiplies (8, or fewer where the rest lies past N: it
// keeps its DMA share and every barrier).  KT = K / 64 >= 1.
template <typename TB, int NJ>
__device__ __forceinline__ void tile_main_loop(f32x4 (&acc)[4][8], const char* a_base, const uint32_t (&a_off)[4],
                                               const char* (&b_ptr)[TileB<TB>::DMAS], int KT, char* smem_raw, int wid,
                                               int lane) {
  using B = TileB<TB>;
  constexpr bool FP8 = std::is_same<TB, fp8_t>::value;
  constexpr int BBYTES = 256 * B::ROW, NB = B::DMAS;
  constexpr int B0 = FP8 ? 3 * kTileHalf : 0;          // first byte of the B ring
  tile_lds* smem = (tile_lds*)smem_raw;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  const int wm = wid >> 1, wn = wid & 1, lc = lane & 15, g = lane >> 4;

  const int arow = wm * 64 + 16 * (lc >> 2) + (lc & 3), brow = wn * 128 + lc;
  // A chunk of half step s: 4 s + g; fp8: 2 g + s, so that one 16-byte read of
  // B holds the lane's bytes of both half steps
  int a_k[2], b_k[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    a_k[s] = arow * 128 + ((FP8 ? 2 * g + s : 4 * s + g) ^ tile_swz_a(arow)) * 16;
    b_k[s] = B0 + brow * B::ROW + ((FP8 ? g : 4 * s + g) ^ tile_swz_b<TB>(brow)) * 16;
  }

  bf16x8 fa[2][4];
  bf16x8 fb[2][8];               // B fragments by half step (bf16)
  uint4 raw[8];                  // fp8 fragments of the K-step
  uint32_t conv[4][4];           // fp8 fragments converted, [j % 4]
  auto read_a = [&](int slot, int s, int i) { fa[s][i] = as_bf16x8(tile_ld16(smem + slot + a_k[s] + i * 4 * 128)); };
  auto read_b = [&](int slot, int s, int j) {
    if (j >= NJ) return;
    const uint4 v = tile_ld16(smem + slot + b_k[s] + j * 16 * B::ROW);
    if constexpr (FP8) raw[j] = v;
    else fb[s][j] = as_bf16x8(v);
  };
  // one of the four conversions of fragment j of half step s
  auto cvt = [&](int s, int j, int c) {
    if constexpr (FP8) {
      if (j >= NJ) return;
      const uint32_t w = s ? (c < 2 ? raw[j].z : raw[j].w) : (c < 2 ? raw[j].x : raw[j].y);
      if (c & 1) conv[j & 3][c] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true));
      else conv[j & 3][c] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false));
    }
  };
  // MFMA q of a half step: fragment j = q / 4 of B against all of A
  auto mma = [&](int s, int q) {
    const int j = q >> 2, i = q & 3;
    if (j < NJ) {
      bf16x8 b;
      if constexpr (FP8) b = as_bf16x8(make_uint4(conv[j & 3][0], conv[j & 3][1], conv[j & 3][2], conv[j & 3][3]));
      else b = fb[s][j];
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fa[s][i]), "v"(b));
    }
  };
  auto dma_a = [&](int slot, int i) { dma16_s(a_base, a_off[i], lds0 + slot + (wid * 4 + i) * 1024); };
  auto dma_b = [&](int slot, int i) { dma16(b_ptr[i], lds0 + B0 + slot + (wid * NB + i) * 1024); };
  // sources advance one K-step after their last DMA of a step; not past the
  // last K-step (the prologue of a short K refetches it)
  auto next_a = [&](bool go) { a_base += go ? 128 : 0; };
  auto next_b = [&](bool go) {
#pragma unroll
    for (int i = 0; i < NB; ++i) b_ptr[i] += go ? B::ROW : 0;
  };

  // prologue: A 0..2, B 0..AHEAD-1, the first step's rows first
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < kTileAheadA) {
#pragma unroll
      for (int i = 0; i < 4; ++i) dma_a(FP8 ? k * kTileHalf : (2 * k % 5) * kTileHalf, i);
      next_a(k + 1 < KT);
    }
    if (k < B::AHEAD) {
#pragma unroll
      for (int i = 0; i < NB; ++i) dma_b(FP8 ? k * BBYTES : ((2 * k + 1) % 5) * kTileHalf, i);
      next_b(k + 1 < KT);
    }
  }
  wait_vm<B::PENDING0>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int sa = 0, sb = FP8 ? 0 : kTileHalf;     // slots of the current K-step
#pragma unroll
  for (int q = 0; q < 8; ++q) read_b(sb, 0, q);
#pragma unroll
  for (int q = 0; q < 4; ++q) read_a(sa, 0, q);
#pragma unroll
  for (int c = 0; c < 8; ++c) cvt(0, c >> 2, c & 3);
  __builtin_amdgcn_sched_barrier(0);

  // One K-step.  DB / DA: refill B (AHEAD steps on) and A; W: DMAs of this
  // wave that may still be in flight at the hand-over; LAST: nothing follows.
  auto step = [&](auto db_tag, auto da_tag, auto w_tag, auto last_tag) {
    constexpr bool DB = decltype(db_tag)::value, DA = decltype(da_tag)::value, LAST = decltype(last_tag)::value;
    constexpr int W = decltype(w_tag)::value;
    int na, nb;
    if constexpr (FP8) {
      na = sa == 2 * kTileHalf ? 0 : sa + kTileHalf;
      nb = sb == 3 * BBYTES ? 0 : sb + BBYTES;
    } else {
      na = sa >= 3 * kTileHalf ? sa - 3 * kTileHalf : sa + 2 * kTileHalf;
      nb = sb >= 3 * kTileHalf ? sb - 3 * kTileHalf : sb + 2 * kTileHalf;
    }
    // refill m MFMAs after the hand-over: B's DMAs, then A's.  bf16: B(k + 2)
    // takes A(k)'s slot and A(k + 3) B(k)'s; fp8: each its own ring.
    auto refill = [&](int m) {
      if (m % B::SPACING != B::SPACING - 1) return;
      const int d = m / B::SPACING;
      if (DB && d < NB) {
        dma_b(FP8 ? sb : sa, d);
        if (d == NB - 1) next_b(true);
      }
      if (DA && d >= NB && d < NB + 4) {
        dma_a(FP8 ? sa : sb, d - NB);
        if (d == NB + 3) next_a(true);
      }
    };
    static_assert((NB + 4) * B::SPACING <= 64 - kBarrierAt, "the refills fit behind the hand-over");
    // read r of a half step's fragments, in the order the MFMAs need them: B 0,
    // A 0..3, B 1..7 (fp8 B is read once a step, below)
    auto read_half = [&](int ra, int rb, int s, int r) {
      if (FP8) {
        if (r < 4) read_a(ra, s, r);
      } else if (r < 12) {
        if (r == 0) read_b(rb, s, 0);
        else if (r <= 4) read_a(ra, s, r - 1);
        else read_b(rb, s, r - 4);
      }
    };
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      mma(0, q);
      if (q % 2 == 0) read_half(sa, sb, 1, q / 2);      // second-half fragments of this step
      if (q < 24) cvt(0, (q >> 2) + 2, q & 3);          // two fragments ahead
      else cvt(1, (q >> 2) - 6, q & 3);
      __builtin_amdgcn_sched_barrier(0);
      if (q == kBarrierAt - 1 && !LAST) {
        // this wave's reads of the step's slots are complete and its DMAs of
        // the next step have landed; after the barrier so have every wave's
        wait_vm<W>();
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (q >= kBarrierAt) {
        refill(q - kBarrierAt);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      mma(1, q);
      if (!LAST) {                                      // first-half fragments of the next step
        if (q % 2 == 0) read_half(na, nb, 0, q / 2);
        if (FP8 && q % 4 == 0) read_b(nb, 0, q >> 2);   // raw[j] was converted for the last time in group j - 2
      }
      if (q < 24) cvt(1, (q >> 2) + 2, q & 3);
      else if (!LAST) cvt(0, (q >> 2) - 6, q & 3);
      refill(q + 32 - kBarrierAt);
      __builtin_amdgcn_sched_barrier(0);
    }
    sa = na;
    sb = nb;
  };
  using T = std::true_type;
  using F = std::false_type;
  constexpr int TAIL = FP8 ? 4 : 3;      // last steps, whose refills would lie past K
  for (int kt = 0; kt < KT - TAIL; ++kt) step(T{}, T{}, std::integral_constant<int, B::PENDING>{}, F{});
  if constexpr (FP8) {
    if (KT >= 4) step(F{}, T{}, std::integral_constant<int, 6>{}, F{});   // A(KT - 1)
    if (KT >= 3) step(F{}, F{}, std::integral_constant<int, 4>{}, F{});
  } else {
    if (KT >= 3) step(T{}, F{}, std::integral_constant<int, 4>{}, F{});    // B(KT - 1)
  }
  if (KT >= 2) step(F{}, F{}, std::integral_constant<int, 0>{}, F{});
  step(F{}, F{}, std::integral_constant<int, 0>{}, T{});
  // The last products must have reached the accumulators before anything
  // reads them -- the register moves the compiler may place at this variant's
  // end included -- so the wait (32 wait states; 11 are needed) stands here.
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  tile_pin(acc);
}

// After the main loop: no DMA may still land in LDS that is about to be
// reused, and every wave has read its last fragments.
__device__ __forceinline__ void tile_drain() {
  __builtin_amdgcn_sched_barrier(0);
  wait_vm<0>();
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void tile_zero(f32x4 (&acc)[4][8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

}  // namespace sr
