// The bf16 tile main loop of the projection and the block GEMMs
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
// LDS of the 256 x 256 tile (160 KB).  bf16 B: a ring of five 32 KB half stages
// (A or B of one K-step), A(k) in slot 2k mod 5, B(k) in 2k + 1 mod 5.  fp8 B:
// three 32 KB A slots and four 16 KB B slots.  Rows keep their 16-byte chunks
// XOR-swizzled so that the 16 lanes an LDS cycle serves fall on 16 distinct
// bank groups.
//
// A 128 x 128 tile (4 waves of 32 x 128, the same rings at half the size: two
// workgroups fit a CU) serves grids of few 256 x 256 tiles; the projection's
// dispatch says when.  One workgroup per CU with rings of five K-steps was 5
// to 10% faster still on grids of fewer tiles than CUs and slower on all
// others, and is not kept.
//
// One hand-over (wait + barrier) per K-step, after BARRIER MFMAs of the
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

constexpr int kTileK = 64;              // K per step: one 128-byte line of A

// Tile shapes.  ROWS x ROWS outputs on WAVES waves, WN of them along N, each
// 16 MI rows x 128 columns.  BARRIER: MFMAs of the first half step before the
// hand-over.  RD: MFMAs per fragment read.
struct TileBig { static constexpr int ROWS = 256, MI = 4, WN = 2, WAVES = 8, BARRIER = 28, RD = 2; };
struct TileSmall { static constexpr int ROWS = 128, MI = 2, WN = 1, WAVES = 4, BARRIER = 12, RD = 1; };
// bytes of one K-step of A (and of bf16 B), workgroup threads, LDS
template <typename C> constexpr int kTileHalf = C::ROWS * 128;
template <typename C> constexpr int kTileThreads = 64 * C::WAVES;
template <typename C> constexpr int kTileLds = 5 * kTileHalf<C>;

typedef __attribute__((address_space(3))) char tile_lds;
typedef unsigned int tile_u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 tile_ld16(const tile_lds* p) {
  return __builtin_bit_cast(uint4, *reinterpret_cast<const __attribute__((address_space(3))) tile_u32x4*>(p));
}

// Per tile shape and B storage.  ROW: bytes of a B row per K-step; DA, DB: 1 KB
// DMA blocks per wave and K-step; NA, NB: K-steps of A and B in flight or in
// use, refilled slot by slot (SHARED: one ring of five slots for both, A three
// and B two steps ahead); BARRIER, SPACING: MFMAs before the hand-over and per
// refill (fp8 has six refills a step against eight: 24 and 6 against 28 and 5
// 12958 against 13131 us for 12 layers of 16384 rows, D 5120, N 8288; 20 and 7
// 12980, 16 and 8 13151; bf16 takes 1% longer with 24); PENDING: DMAs that may
// still be in flight at a hand-over once the next step has landed (issue order
// of a step: B, then A); PENDING0: the same before the first step.
template <typename C, typename TB>
struct TileRing {
  static constexpr bool FP8 = std::is_same<TB, fp8_t>::value, SHARED = !FP8;
  static constexpr int ROW = FP8 ? 64 : 128, DA = 4, DB = FP8 ? 2 : 4;
  static constexpr int NA = 3, NB = FP8 ? 4 : 2;
  static constexpr int BARRIER = FP8 && C::MI == 4 ? 24 : C::BARRIER;
  static constexpr int SPACING = C::MI == 4 ? (FP8 ? 6 : 4) : (FP8 ? 3 : 2);
  static constexpr int PENDING = SHARED ? DA : (NA - 2) * (DA + DB);
  static constexpr int PENDING0 = (NA - 1) * DA + (NB - 1) * DB;
  static constexpr int TAIL = NA > NB ? NA : NB;   // last steps, whose refills would lie past K
  static constexpr int BSTEP = C::ROWS * ROW;      // bytes of one K-step of B
  static_assert(C::ROWS * 128 == DA * C::WAVES * 1024 && BSTEP == DB * C::WAVES * 1024, "DMA split");
  static_assert(NA * kTileHalf<C> + NB * BSTEP <= kTileLds<C>, "LDS");
  static_assert((DA + DB) * SPACING <= 16 * C::MI - BARRIER, "the refills fit behind the hand-over");
  // DMAs that may be in flight when `t` steps remain (t <= TAIL)
  static constexpr int pending(int t) {
    if (SHARED) return t >= 3 ? DA : 0;
    const int w = (t - 2) * DA + (t - 2 + NA - NB > 0 ? t - 2 + NA - NB : 0) * DB;
    return w < PENDING ? w : PENDING;
  }
};

// Chunk swizzles: LDS row r keeps 16-byte chunk c of its K-step at c ^ swz(r).
// An A fragment reads rows 4 MI (m / 4) + 4 i + m % 4 (m = lane % 16), a B one
// 16 consecutive rows.  An LDS cycle of a 16-byte read serves lanes 0-3,
// 12-15 and 20-27 (or 4-11, 16-19, 28-31; the same above 32): rows m / 4 = 0, 3
// of one chunk with rows 1, 2 of a chunk that differs in one bit, bit 0 for bf16
// and bit 1 (A) or 0 (B) for fp8.  quad() keeps those apart: it maps 0, 3 to 0, 1
// and 1, 2 to 2, 3.
__device__ __forceinline__ int tile_quad(int h) { return (((h ^ (h >> 1)) & 1) << 1) | ((h >> 1) & 1); }
template <typename C>
__device__ __forceinline__ int tile_swz_a(int r) { return ((r >> 1) & 1) | (tile_quad(r / (4 * C::MI)) << 1); }
template <typename TB>
__device__ __forceinline__ int tile_swz_b(int r) {
  return std::is_same<TB, bf16_t>::value ? (r >> 1) & 7 : tile_quad(r >> 2);
}

// Tile row / chunk that lane `lane` of wave `wid` fetches with its DMA i (the
// LDS side is linear: block wid * DA (DB) + i, 16 bytes per lane)
__device__ __forceinline__ int tile_a_row(int wid, int i, int lane) { return (wid * 4 + i) * 8 + (lane >> 3); }
template <typename C>
__device__ __forceinline__ int tile_a_chunk(int row, int lane) { return (lane & 7) ^ tile_swz_a<C>(row); }
template <typename TB>
__device__ __forceinline__ int tile_b_row(int wid, int i, int lane) {
  return std::is_same<TB, bf16_t>::value ? (wid * 4 + i) * 8 + (lane >> 3) : (wid * 2 + i) * 16 + (lane >> 2);
}
template <typename TB>
__device__ __forceinline__ int tile_b_chunk(int row, int lane) {
  return std::is_same<TB, bf16_t>::value ? (lane & 7) ^ tile_swz_b<TB>(row) : (lane & 3) ^ tile_swz_b<TB>(row);
}

// Accumulators of wave (wm, wn) = (wid / WN, wid % WN): acc[i][j][r] of lane l
// is tile row 16 MI wm + 4 MI (l / 16) + 4 i + r -- 4 MI consecutive rows per
// lane over i and r -- and LDS row 128 wn + 16 j + l % 16 of B.
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
template <int MI>
__device__ __forceinline__ void tile_pin(f32x4 (&acc)[MI][8]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
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
template <typename C, typename TB, int NJ>
__device__ __forceinline__ void tile_main_loop(f32x4 (&acc)[C::MI][8], const char* a_base, const uint32_t (&a_off)[4],
                                               const char* (&b_ptr)[TileRing<C, TB>::DB], int KT, char* smem_raw,
                                               int wid, int lane) {
  using R = TileRing<C, TB>;
  constexpr bool FP8 = R::FP8, SHARED = R::SHARED;
  constexpr int MI = C::MI, Q = 8 * MI, HALF = kTileHalf<C>, BSTEP = R::BSTEP, DA = R::DA, DB = R::DB;
  constexpr int B0 = SHARED ? 0 : R::NA * HALF;        // first byte of the B ring
  tile_lds* smem = (tile_lds*)smem_raw;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  const int wm = wid / C::WN, wn = wid % C::WN, lc = lane & 15, g = lane >> 4;

  const int arow = wm * 16 * MI + 4 * MI * (lc >> 2) + (lc & 3), brow = wn * 128 + lc;
  // A chunk of half step s: 4 s + g; fp8: 2 g + s, so that one 16-byte read of
  // B holds the lane's bytes of both half steps
  int a_k[2], b_k[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    a_k[s] = arow * 128 + ((FP8 ? 2 * g + s : 4 * s + g) ^ tile_swz_a<C>(arow)) * 16;
    b_k[s] = B0 + brow * R::ROW + ((FP8 ? g : 4 * s + g) ^ tile_swz_b<TB>(brow)) * 16;
  }

  bf16x8 fa[2][MI];
  bf16x8 fb[2][8];               // B fragments by half step (bf16)
  uint4 raw[8];                  // fp8 fragments of the K-step
  uint32_t conv[4][4];           // fp8 fragments converted, [j % 4]
  auto read_a = [&](int slot, int s, int i) { fa[s][i] = as_bf16x8(tile_ld16(smem + slot + a_k[s] + i * 4 * 128)); };
  auto read_b = [&](int slot, int s, int j) {
    if (j >= NJ) return;
    const uint4 v = tile_ld16(smem + slot + b_k[s] + j * 16 * R::ROW);
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
  // MFMA q of a half step: fragment j = q / MI of B against all of A
  auto mma = [&](int s, int q) {
    const int j = q / MI, i = q % MI;
    if (j < NJ) {
      bf16x8 b;
      if constexpr (FP8) b = as_bf16x8(make_uint4(conv[j & 3][0], conv[j & 3][1], conv[j & 3][2], conv[j & 3][3]));
      else b = fb[s][j];
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fa[s][i]), "v"(b));
    }
  };
  auto dma_a = [&](int slot, int i) { dma16_s(a_base, a_off[i], lds0 + slot + (wid * DA + i) * 1024); };
  auto dma_b = [&](int slot, int i) { dma16(b_ptr[i], lds0 + B0 + slot + (wid * DB + i) * 1024); };
  // sources advance one K-step after their last DMA of a step; not past the
  // last K-step (the prologue of a short K refetches it)
  auto next_a = [&](bool go) { a_base += go ? 128 : 0; };
  auto next_b = [&](bool go) {
#pragma unroll
    for (int i = 0; i < DB; ++i) b_ptr[i] += go ? R::ROW : 0;
  };

  // prologue: A 0 .. NA-1, B 0 .. NB-1, the first step's rows first
#pragma unroll
  for (int k = 0; k < R::TAIL; ++k) {
    if (k < R::NA) {
#pragma unroll
      for (int i = 0; i < DA; ++i) dma_a(SHARED ? (2 * k % 5) * HALF : k * HALF, i);
      next_a(k + 1 < KT);
    }
    if (k < R::NB) {
#pragma unroll
      for (int i = 0; i < DB; ++i) dma_b(SHARED ? ((2 * k + 1) % 5) * HALF : k * BSTEP, i);
      next_b(k + 1 < KT);
    }
  }
  wait_vm<R::PENDING0>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int sa = 0, sb = SHARED ? HALF : 0;       // slots of the current K-step
#pragma unroll
  for (int q = 0; q < 8; ++q) read_b(sb, 0, q);
#pragma unroll
  for (int q = 0; q < MI; ++q) read_a(sa, 0, q);
#pragma unroll
  for (int c = 0; c < 8; ++c) cvt(0, c >> 2, c & 3);
  __builtin_amdgcn_sched_barrier(0);

  // One K-step.  GB / GA: refill B and A; W: DMAs of this wave that may still
  // be in flight at the hand-over; LAST: nothing follows.
  auto step = [&](auto gb_tag, auto ga_tag, auto w_tag, auto last_tag) {
    constexpr bool GB = decltype(gb_tag)::value, GA = decltype(ga_tag)::value, LAST = decltype(last_tag)::value;
    constexpr int W = decltype(w_tag)::value;
    int na, nb;
    if constexpr (SHARED) {
      na = sa >= 3 * HALF ? sa - 3 * HALF : sa + 2 * HALF;
      nb = sb >= 3 * HALF ? sb - 3 * HALF : sb + 2 * HALF;
    } else {
      na = sa == (R::NA - 1) * HALF ? 0 : sa + HALF;
      nb = sb == (R::NB - 1) * BSTEP ? 0 : sb + BSTEP;
    }
    // refill m MFMAs after the hand-over: B's DMAs, then A's.  SHARED: B(k + 2)
    // takes A(k)'s slot and A(k + 3) B(k)'s; else each its own.
    auto refill = [&](int m) {
      if (m % R::SPACING != R::SPACING - 1) return;
      const int d = m / R::SPACING;
      if (GB && d < DB) {
        dma_b(SHARED ? sa : sb, d);
        if (d == DB - 1) next_b(true);
      }
      if (GA && d >= DB && d < DB + DA) {
        dma_a(SHARED ? sb : sa, d - DB);
        if (d == DB + DA - 1) next_a(true);
      }
    };
    // read r of a half step's fragments, in the order the MFMAs need them: B 0,
    // A, B 1..7 (fp8 B is read once a step, below)
    auto read_half = [&](int ra, int rb, int s, int r) {
      if (FP8) {
        if (r < MI) read_a(ra, s, r);
      } else if (r < 8 + MI) {
        if (r == 0) read_b(rb, s, 0);
        else if (r <= MI) read_a(ra, s, r - 1);
        else read_b(rb, s, r - MI);
      }
    };
    // fp8: the conversions after MFMA q of half s, two fragments ahead
    auto convert = [&](int s, int q) {
      constexpr int PER = 4 / MI;
      const int j = q / MI + 2;
#pragma unroll
      for (int c = 0; c < PER; ++c) {
        const int part = (q % MI) * PER + c;
        if (j < 8) cvt(s, j, part);
        else if (s == 0) cvt(1, j - 8, part);
        else if (!LAST) cvt(0, j - 8, part);
      }
    };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      mma(0, q);
      if (q % C::RD == 0) read_half(sa, sb, 1, q / C::RD);   // second-half fragments of this step
      convert(0, q);
      __builtin_amdgcn_sched_barrier(0);
      if (q == R::BARRIER - 1 && !LAST) {
        // this wave's reads of the step's slots are complete and its DMAs of
        // the next step have landed; after the barrier so have every wave's
        wait_vm<W>();
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (q >= R::BARRIER) {
        refill(q - R::BARRIER);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      mma(1, q);
      if (!LAST) {                                      // first-half fragments of the next step
        if (q % C::RD == 0) read_half(na, nb, 0, q / C::RD);
        if (FP8 && q % MI == 0) read_b(nb, 0, q / MI);  // raw[j] was converted for the last time in group j - 2
      }
      convert(1, q);
      refill(q + Q - R::BARRIER);
      __builtin_amdgcn_sched_barrier(0);
    }
    sa = na;
    sb = nb;
  };
  using T = std::true_type;
  using F = std::false_type;
  for (int kt = 0; kt < KT - R::TAIL; ++kt) step(T{}, T{}, std::integral_constant<int, R::PENDING>{}, F{});
  // `t` steps remain
  auto tail = [&](auto t_tag) {
    constexpr int t = decltype(t_tag)::value;
    if constexpr (t >= 2 && t <= R::TAIL) {
      if (KT >= t)
        step(std::integral_constant<bool, (t > R::NB)>{}, std::integral_constant<bool, (t > R::NA)>{},
             std::integral_constant<int, R::pending(t)>{}, F{});
    }
  };
  tail(std::integral_constant<int, 4>{});
  tail(std::integral_constant<int, 3>{});
  tail(std::integral_constant<int, 2>{});
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

template <int MI>
__device__ __forceinline__ void tile_zero(f32x4 (&acc)[MI][8]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

}  // namespace sr
