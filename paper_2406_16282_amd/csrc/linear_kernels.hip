// Linear layer with a fused ReGELU2 / ReSiLU2 forward epilogue, for gfx950.
//
// z = x W^T (+ b): x [M x K] and W [N x K] (the weight of a linear layer) are bf16
// and K-contiguous; products accumulate in fp32 on v_mfma_f32_16x16x32_bf16 and z is
// rounded once to bf16 (bias added in fp32 before the rounding). The epilogue then
// applies the activation to the rounded z and stores y = act(z) and the 2-bit codes
// of z (Sec. 4.2; 16 codes per word over the flattened [M x N] output), i.e. exactly
// what the activation kernels compute from a stored z. z itself is stored only when
// the caller asks for it: ReGELU2 / ReSiLU2 keep only the codes for the backward
// pass, so the pre-activation never has to reach HBM.
//
// What bounds it. Large products: the card's power. With random operands a loop of
// nothing but 32x32x16 MFMAs runs at 1840 TFLOP/s and of 16x16x32 ones at 2085 (2440 for
// both on zeros), so the smaller shape is used although it needs as many operand reads:
// the [8192 x 4096] x [4096 x 11008] SiLU layer took 641 us before and 606 us after that
// change alone, with the same bits. Then the delivery of operands: with one block
// barrier per K step and all of a step's loads issued behind it, the matrix cores were
// busy 70% of the cycles; the ring below (half steps, loads spread over the MFMAs, two
// to three half steps in flight) gave 597 us, the persistent blocks with the epilogue in
// registers 581 us; the gated [8192 x 4096] x 2 [4096 x 11008] layer went from 1213 to
// 1113 us (same card; others run 2 to 8% slower). No address spilled in the epilogue gave 1 to
// 2% more there and 4 to 8% at smaller sizes. Products with a short K (ViT-B: 768): the epilogue,
// about 22 VALU operations per element, is as long as the K loop; two blocks per CU let one
// block's epilogue run beside the other's MFMAs (77 us in 128 x 256 tiles, two to a CU, against
// 88 in 128 x 128 and 91 in 256 x 256, one to a CU).
//
// Tiling. A block computes a BM x BN tile of z with WM x WN waves, each BM/WM x 64 as
// 16 x 16 MFMA tiles, accumulators in registers. Four tiles are compiled, and a
// split-K form for few rows; the launcher picks one by a cost model of the measured times
// (below).
//
// K loop. K advances in steps of 64, each in two half steps. The LDS is a ring of slots
// of half a step's operands: slot 2t holds the first half of every wave's rows of x and
// of its rows of W (all 64 k), slot 2t + 1 the second halves. A half step h computes the
// products of fragments already in registers, reads the fragments that the next ones
// need from slot h + 1, and issues the loads of slot h + kRing into the place of slot h,
// whose last reader passed the barrier before. One barrier per half step, and a wait
// that leaves kRing - 2 slots of loads in flight (loads return in order; any other
// vector-memory operation in between only makes the wait stricter). The slots are filled
// straight from memory by raw buffer loads with an LDS destination. The buffer resources
// end at the tile's last valid row, so ragged tiles read zeros without branches, and
// chunks beyond K are pointed past the end to read zeros too. An LDS row is 64 bf16 =
// eight 16-byte units; unit u of row r holds k-chunk u ^ swz(r), with swz chosen so that
// the 16 rows of an operand read at one k-chunk fall into distinct banks: (r >> 1) % 8
// for x (rows 16 apart in a read: r = 16 i + 0 .. 15), bit 1 and bits 3..4 of r for W
// (rows 8 a + 4 j + 0 .. 3, a = 0 .. 3).
//
// Blocks are persistent (as many as fit the device) and the stream of loads runs on from
// one tile into the next: the first K steps of the next tile are under way while the
// epilogue of the current one runs. Tiles are dealt out XCD by XCD (consecutive blocks
// go to the 8 XCDs in turn) in groups of 8 row tiles, so that the blocks sharing an
// XCD's L2 also share their x and W tiles.
//
// Epilogue, in registers. The MFMA takes W rows as its first operand, so lane l holds
// row l % 16 of a 16-row block and, in register r of tile j, W index p = 4 (l / 16) + r.
// The rows of W are dealt to the tiles such that p of tile j is output column
// 16 (p / 4) + 4 j + p % 4 of the wave's 64: a lane holds 16 consecutive columns, one
// whole code word and 32 bytes of y. Gated form: the first half of a wave's W rows comes
// from the gate weight, the second from the up weight, for the same 32 output columns; a
// lane holds 8 consecutive columns of both, and two lanes make a code word. Lane layout
// of the MFMA (checked on the hardware): lane l supplies row l % 16 of the first operand
// and column l % 16 of the second at k = 8 (l / 16) .. + 7, and holds result rows
// 4 (l / 16) + 0 .. 3 of column l % 16.
//
// Norm in front (MS-RMSNorm, Sec. 5.2): the norm kernel writes z and rstd first, and this
// kernel multiplies each row's fp32 sums by its rstd (with the bias, one fused
// multiply-add). Letting the GEMM write z instead saved the norm kernel's stores but
// stretched the epilogue by more: [2048 x 4096] with two 11008-row weights, 415 us then.
#include "lmbp_device.hpp"
#include "act_codes.hpp"
#include "act_math.hpp"
#include "lmbp_launch.hpp"

#include <algorithm>
#include <atomic>
#include <cmath>

namespace lmbp {
namespace lin {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kGroupM = 8;
constexpr uint32_t kBufferGDword3 = 0x00020000;  // raw 32-bit buffer, gfx9 family
constexpr uint32_t kOutOfRange = 0x80000000u;    // beyond any resource's range: reads 0
constexpr int kBK = 64;                          // K step: an LDS row is 128 bytes

// MINW: waves per SIMD that the registers are budgeted for (blocks per CU follow from it).
template <int BM_, int BN_, int WM_, int WN_, int MINW_, int RING_ = 4>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, kMinWaves = MINW_;
  static constexpr int kWaves = WM * WN, kThreads = kWaves * kWave;
  static constexpr int HM = BM / WM / 2, HN = 32;       // half of a wave's rows, columns
  static constexpr int TMH = HM / 16, TNH = HN / 16;    // MFMA tiles per half
  static constexpr int TM = 2 * TMH, TN = 2 * TNH;
  static constexpr int kSlotElems = (BM + BN) / 2 * kBK;   // one ring slot: half of A and of B
  static constexpr int kRing = RING_;                   // slots in LDS
  static constexpr int kBlocksPerCu = kMinWaves * 4 / kWaves;
  static constexpr int kLA = BM / 16 / kWaves, kLB = BN / 16 / kWaves;   // 1 KiB loads per wave
  static constexpr int kSideBytes = 4 * (BN * 2 + BM * 4);   // bias and rstd of four tiles
  static constexpr int kLdsBytes = kRing * kSlotElems * 2 + kSideBytes;
  static_assert(BN / WN == 64 && HM % 16 == 0, "wave tile");
  static_assert(kLA >= 1 && kLB >= 1 && (BM / 16) % kWaves == 0 && (BN / 16) % kWaves == 0, "loads");
  static_assert(kLdsBytes * kBlocksPerCu <= 160 * 1024, "LDS per CU");
};

using BigTile = Tile<256, 256, 2, 4, 2>;      // one block of 8 waves per CU
using MidTile = Tile<128, 256, 1, 4, 2, 3>;   // two blocks of 4 waves
using SmallTile = Tile<128, 128, 4, 2, 4>;    // two blocks of 8 waves
using LowTile = Tile<64, 128, 2, 2, 3>;       // three blocks of 4 waves

// The grid of tiles: sizes, tiles per XCD, and floor(2^32 / tiles_n).
struct TileMap {
  uint32_t tiles_m, tiles_n, tiles, per_xcd, inv_n;
};

// The target builtins below are wrapped in device functions: used directly in the body of
// a kernel template, they make the host-side instantiation fail silently and the launch
// stub is never emitted.

// A raw buffer resource over `bytes` bytes at `base` (reads beyond return zeros).
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), kBufferGDword3);
}
// 16 or 4 bytes per lane from the buffer into LDS at `dst` + lane * 16 or 4 (dst wave-uniform).
// CPOL: cache policy bits of the instruction (nt = 2).
template <int CPOL = 0>
__device__ inline void load_lds16(__amdgpu_buffer_rsrc_t r, void* dst, uint32_t offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 16, offset, 0, 0, CPOL);
}
__device__ inline void load_lds4(__amdgpu_buffer_rsrc_t r, void* dst, uint32_t offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 4, offset, 0, 0, 0);
}

// Scheduling groups for MF MFMAs, with VM buffer loads and then DS LDS reads spread over
// the first half of them (so the reads have landed before the next wait).
template <int MF, int VM, int DS, int I = 0>
__device__ inline void spread() {
  if constexpr (I < MF) {
    constexpr int W = MF / 2 < 1 ? 1 : MF / 2;
    constexpr int T = VM + DS;
    constexpr int lo = I < W ? T * I / W : T, hi = I < W ? T * (I + 1) / W : T;
    constexpr int vm = (hi < VM ? hi : VM) - (lo < VM ? lo : VM);
    constexpr int ds = (hi - lo) - vm;
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // one MFMA
    if constexpr (vm > 0) __builtin_amdgcn_sched_group_barrier(0x020, vm, 0);  // buffer loads
    if constexpr (ds > 0) __builtin_amdgcn_sched_group_barrier(0x100, ds, 0);  // LDS reads
    spread<MF, VM, DS, I + 1>();
  }
}

// Tile coordinates of the t-th tile (see the file comment). tiles_n is divided by with a
// host-made reciprocal (floor(2^32 / tiles_n), at most one short of the quotient for
// t < 2^30) instead of an integer division.
__device__ inline void tile_of(uint32_t t, const TileMap& m, uint32_t& tm, uint32_t& tn) {
  const uint32_t id = (t < m.per_xcd * kXcds) ? (t % kXcds) * m.per_xcd + t / kXcds : t;
  const uint32_t id8 = id / kGroupM;
  uint32_t group = __umulhi(id8, m.inv_n);
  uint32_t in = id8 - group * m.tiles_n;
  while (in >= m.tiles_n) {
    in -= m.tiles_n;
    ++group;
  }
  const uint32_t first_m = group * kGroupM, r = in * kGroupM + id % kGroupM;
  const uint32_t left = m.tiles_m - first_m;
  if (left >= uint32_t(kGroupM)) {
    tm = first_m + r % kGroupM;
    tn = r / kGroupM;
  } else {   // the last, smaller group of row tiles
    tm = first_m + r % left;
    tn = r / left;
  }
}

// Arguments of the kernel (by value). Plain form: y = act(z), z = x w^T + bias.
// Gated form (GLU): g = x w^T and u = x w2^T (no bias), y = h = act(g) * u, s = act(g),
// u stored; z (optional) receives g; codes are those of g. Norm in front (NORM): x is the
// norm's input and rstd its per-row statistic.
struct LinArgs {
  const uint16_t* x;
  const uint16_t* w;
  const uint16_t* w2;
  const uint16_t* bias;
  uint16_t* y;
  uint16_t* s;
  uint16_t* u;
  uint32_t* codes;
  uint16_t* z;
  int64_t M, N, K;
  const float* rstd;
  TileMap map;
};

template <class C, int ACT, bool GLU, bool NORM>
__global__ __launch_bounds__(C::kThreads, C::kMinWaves) void linear_act_fwd_kernel(LinArgs a) {
  using A = ActOf<ACT>;
  constexpr int BM = C::BM, BN = C::BN, TM = C::TM, TN = C::TN, TMH = C::TMH, TNH = C::TNH;
  constexpr int HM = C::HM, HN = C::HN, kWaves = C::kWaves;
  constexpr int kLA = C::kLA, kLB = C::kLB, kL = kLA + kLB;
  constexpr int kOut = GLU ? BN / 2 : BN;
  constexpr int kSlot = C::kSlotElems;
  const int64_t M = a.M, N = a.N, K = a.K;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  uint16_t* const bias_lds = lds + C::kRing * kSlot;
  float* const rstd_lds = reinterpret_cast<float*>(bias_lds + 4 * BN);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_in_block();
  const int wm = wave / C::WN, wn = wave % C::WN;
  const uint32_t tiles = a.map.tiles;
  const int kt_count = K > 0 ? int((K + kBK - 1) / kBK) : 1;

  // The bias goes through LDS in 4-byte loads; one that starts between two words is read
  // in the epilogue instead.
  const bool bias_staged = a.bias != nullptr && (reinterpret_cast<uintptr_t>(a.bias) & 2) == 0;

  // ---- load side: byte offsets of this lane's chunks at K step 0, for both halves
  uint32_t ld_a[2][kLA], ld_b[GLU ? 1 : 2][kLB];
  int kc_a[kLA], kc_b[kLB];
  const int r_in = lane / 8, u_in = lane % 8;
#pragma unroll
  for (int q = 0; q < kLA; ++q) {
    const int lr = (wave + kWaves * q) * 8 + r_in;
    kc_a[q] = (u_in ^ ((lr >> 1) & 7)) * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      ld_a[h][q] = uint32_t(((lr / HM) * 2 * HM + h * HM + lr % HM) * K * 2 + kc_a[q] * 2);
  }
#pragma unroll
  for (int q = 0; q < kLB; ++q) {
    const int lr = (wave + kWaves * q) * 8 + r_in;
    kc_b[q] = (u_in ^ (((lr >> 1) & 1) | (((lr >> 3) & 3) << 1))) * 8;
    if constexpr (GLU) {
      ld_b[0][q] = uint32_t(lr * K * 2 + kc_b[q] * 2);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        ld_b[h][q] = uint32_t(((lr / 8) * 16 + h * 8 + lr % 8) * K * 2 + kc_b[q] * 2);
    }
  }
  // Load cursor: tile l_tile (l_seq-th of this block), K step l_k. Past the last tile the
  // resources are empty and the loads read zeros into slots that nothing reads.
  uint32_t l_tile = blockIdx.x;
  int l_seq = 0, l_k = 0;
  __amdgpu_buffer_rsrc_t rx, rw, rw2;
  auto enter_tile = [&]() {
    uint32_t tm = 0, tn = 0;
    const bool in = l_tile < tiles;
    if (in) tile_of(l_tile, a.map, tm, tn);
    const int64_t m0 = int64_t(tm) * BM, n0 = int64_t(tn) * kOut;
    const int64_t rows_x = !in ? 0 : (M - m0 < BM) ? M - m0 : BM;
    const int64_t rows_w = !in ? 0 : (N - n0 < kOut) ? N - n0 : kOut;
    rx = make_rsrc(a.x + m0 * K, rows_x * K * 2);
    rw = make_rsrc(a.w + n0 * K, rows_w * K * 2);
    if constexpr (GLU) rw2 = make_rsrc(a.w2 + n0 * K, rows_w * K * 2);
    // The tile's bias and rstd, into one of four places: the cursor runs at most two tiles
    // ahead of the tile being computed. Issued before the tile's first operands, they have
    // landed when those have.
    if constexpr (!GLU) {
      if (bias_staged)
        for (int v = wave; v < BN / 128; v += kWaves)
          load_lds4(make_rsrc(a.bias + n0, rows_w * 2), bias_lds + (l_seq & 3) * BN + v * 128,
                    uint32_t(v * 256 + lane * 4));
    }
    if constexpr (NORM) {
      for (int v = wave; v < BM / 64; v += kWaves)
        load_lds4(make_rsrc(a.rstd + m0, rows_x * 4), rstd_lds + (l_seq & 3) * BM + v * 64,
                  uint32_t(v * 256 + lane * 4));
    }
  };
  auto issue = [&](int h, uint16_t* S) {
    const uint32_t k0 = uint32_t(l_k) * kBK;
#pragma unroll
    for (int q = 0; q < kLA; ++q)
      load_lds16(rx, S + (wave + kWaves * q) * 512, k0 + kc_a[q] < K ? ld_a[h][q] + k0 * 2 : kOutOfRange);
#pragma unroll
    for (int q = 0; q < kLB; ++q)
      load_lds16((GLU && h == 1) ? rw2 : rw, S + BM / 2 * kBK + (wave + kWaves * q) * 512,
                 k0 + kc_b[q] < K ? ld_b[GLU ? 0 : h][q] + k0 * 2 : kOutOfRange);
  };
  auto advance = [&]() {
    if (++l_k == kt_count) {
      l_k = 0;
      l_tile += gridDim.x;
      ++l_seq;
      enter_tile();
    }
  };

  // ---- compute side
  const int a_off = (wm * HM + (lane & 15)) * kBK;
  const int b_off = BM / 2 * kBK + (wn * HN + ((lane & 15) >> 2) * 8 + (lane & 3)) * kBK;
  const int swa = (lane & 15) >> 1;
  const int swb = ((lane >> 1) & 1) | (((lane >> 2) & 3) << 1);
  const int ua[2] = {((lane >> 4) ^ swa) * 8, ((4 + (lane >> 4)) ^ swa) * 8};
  const int ub[2] = {((lane >> 4) ^ swb) * 8, ((4 + (lane >> 4)) ^ swb) * 8};
  bf16x8 fa[2][TMH][2], fb[2][TNH][2];
  auto read_a = [&](const uint16_t* S, int h) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < TMH; ++i)
        fa[h][i][kk] = *reinterpret_cast<const bf16x8*>(S + a_off + i * 16 * kBK + ua[kk]);
  };
  auto read_b = [&](const uint16_t* S, int h) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int j = 0; j < TNH; ++j)
        fb[h][j][kk] = *reinterpret_cast<const bf16x8*>(S + b_off + j * 4 * kBK + ub[kk]);
  };
  f32x4 acc[TM][TN];
  auto quad = [&](int ha, int hb) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < TMH; ++i)
#pragma unroll
        for (int j = 0; j < TNH; ++j)
          acc[ha * TMH + i][hb * TNH + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fb[hb][j][kk], fa[ha][i][kk], acc[ha * TMH + i][hb * TNH + j], 0, 0, 0);
  };
  constexpr int MF = TMH * TNH * 2, RA = TMH * 2, RB = TNH * 2;

  // An odd ring has its second-half slots loaded in first half steps and the other way round.
  enter_tile();
  constexpr int kRing = C::kRing;
  constexpr bool kOdd = kRing % 2 != 0;
#pragma unroll
  for (int d = 0; d < kRing; ++d) {
    issue(d & 1, lds + d * kSlot);
    if (d & 1) advance();
  }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 2) * kL) : "memory");
  asm volatile("s_barrier" ::: "memory");

  int slot = 0;   // of the half step's first data unit
  auto next = [&](int v, int d) { v += d; return v >= kRing ? v - kRing : v; };
  int seq = 0;
  for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x, ++seq) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;
    // The tile's first fragments; no wave may load over them before all have read them.
    read_a(lds + slot * kSlot, 0);
    read_b(lds + slot * kSlot, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");

    for (int kt = 0; kt < kt_count; ++kt) {
      uint16_t* S = lds + slot * kSlot;
      uint16_t* S1 = lds + next(slot, 1) * kSlot;
      slot = next(slot, 2);
      uint16_t* Sn = lds + slot * kSlot;
      issue(kOdd ? 1 : 0, S);
      read_b(S1, 1);
      read_a(S1, 1);
      quad(0, 0);
      quad(0, 1);
      spread<2 * MF, kL, RA + RB>();
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 2) * kL) : "memory");
      asm volatile("s_barrier" ::: "memory");
      if constexpr (kOdd) advance();
      issue(kOdd ? 0 : 1, S1);
      read_a(Sn, 0);
      quad(1, 0);
      spread<MF, kL, RA>();
      __builtin_amdgcn_sched_barrier(0);
      read_b(Sn, 0);
      quad(1, 1);
      spread<MF, 0, RB>();
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 2) * kL) : "memory");
      asm volatile("s_barrier" ::: "memory");
      if constexpr (!kOdd) advance();
    }

    // ---- epilogue (see the file comment); no LDS slot is touched, so the next tile's loads run on
    uint32_t tm, tn;
    tile_of(tile, a.map, tm, tn);
    const int64_t m0 = int64_t(tm) * BM, n0 = int64_t(tn) * kOut;
    // The lane as a value that is new in every tile: the addresses formed from it ahead of
    // the tile loop were 9 to 15 registers more than the two larger tiles have, and each reload
    // from scratch waited for every load and store in flight, the next tile's first K steps
    // among them. 12608 x 3072 x 768 (GELU) 86.4 us then and 79.8 now in 128 x 256 tiles; 2048 x
    // (4096 -> 2 x 11008) 341 and 321 in 256 x 256; 4 to 8% over all sizes of the two.
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int g = lane_e >> 4;
    const int64_t col = n0 + wn * (GLU ? 32 : 64) + g * (GLU ? 8 : 16);
    u32x4 b0 = {0u, 0u, 0u, 0u}, b1 = {0u, 0u, 0u, 0u};
    const bool in_col = col < N;   // N is a multiple of 16: a lane's columns are wholly in or out
    if constexpr (!GLU) {
      if (a.bias != nullptr && !bias_staged && in_col) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          b0[e] = a.bias[col + 2 * e] | uint32_t(a.bias[col + 2 * e + 1]) << 16;
          b1[e] = a.bias[col + 8 + 2 * e] | uint32_t(a.bias[col + 8 + 2 * e + 1]) << 16;
        }
      }
      if (bias_staged) {
        const uint16_t* bl = bias_lds + (seq & 3) * BN + wn * 64 + g * 16;
        b0 = *reinterpret_cast<const u32x4*>(bl);
        b1 = *reinterpret_cast<const u32x4*>(bl + 8);
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = wm * 2 * HM + i * 16 + (lane_e & 15);
      const float rs = NORM ? rstd_lds[(seq & 3) * BM + row] : 1.0f;
      float f0[8], f1[8], o0[8], o1[8];
      if constexpr (GLU) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { f0[e] = 0.0f; f1[e] = 0.0f; }
      } else {
        BF16::unpack(b0, f0);
        BF16::unpack(b1, f1);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v0 = acc[i][e / 4][e % 4], v1 = acc[i][2 + e / 4][e % 4];
        f0[e] = NORM ? __builtin_fmaf(v0, rs, f0[e]) : v0 + f0[e];
        f1[e] = NORM ? __builtin_fmaf(v1, rs, f1[e]) : v1 + f1[e];
      }
      const u32x4 z0 = BF16::pack(f0), z1 = BF16::pack(f1);
      BF16::unpack(z0, f0);
      BF16::unpack(z1, f1);
      const bool ok = in_col && m0 + row < M;
      const int64_t base = (m0 + row) * N + col;
      if constexpr (GLU) {
#pragma unroll
        for (int e = 0; e < 8; ++e) gated_value<ACT, false>(f0[e], f1[e], o0[e], o1[e]);
        const uint32_t part = codes_of<A>(f0);
        const uint32_t other = uint32_t(__shfl_xor(int(part), 16, kWave));
        if (ok) {
          *reinterpret_cast<u32x4*>(a.y + base) = BF16::pack(o1);
          *reinterpret_cast<u32x4*>(a.s + base) = BF16::pack(o0);
          *reinterpret_cast<u32x4*>(a.u + base) = z1;
          if ((g & 1) == 0) a.codes[base / 16] = part | (other << 16);
          if (a.z != nullptr) *reinterpret_cast<u32x4*>(a.z + base) = z0;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          o0[e] = act_value<ACT, false>(f0[e]);
          o1[e] = act_value<ACT, false>(f1[e]);
        }
        const uint32_t word = codes_of<A>(f0) | (codes_of<A>(f1) << 16);
        if (ok) {
          *reinterpret_cast<u32x4*>(a.y + base) = BF16::pack(o0);
          *reinterpret_cast<u32x4*>(a.y + base + 8) = BF16::pack(o1);
          a.codes[base / 16] = word;
          if (a.z != nullptr) {
            *reinterpret_cast<u32x4*>(a.z + base) = z0;
            *reinterpret_cast<u32x4*>(a.z + base + 8) = z1;
          }
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load into LDS outlives the block
}

// Few rows: the split-K form. What bounds it: for large weights the stream of W, each row
// of which serves at most 32 rows of x, so what counts is how many bytes are in flight
// over the whole device and that every lane quad asks for consecutive bytes; for small
// weights the latency of one chain of loads. A block of 4 waves takes MT x 16 rows of x
// and 32 rows of W (gated: 16 of each weight). Its waves take the K steps of 64 in turn,
// each through an LDS ring of its own with two steps in flight, so that the K loop has no
// barrier. The four partial sums of a result meet in LDS, are added in a fixed order, and
// go through the epilogue with 4 columns per lane, four lanes to a code word.
// Measured against the tiled kernel's best form: [16 x 768] x 3072 3.9 against 8.6 us;
// [16 x 4096] x two 11008 33 against 43-46 us (180 MB of weights, 5.5 TB/s). MFMA operands
// loaded straight into registers asked for 16 bytes per row and lane: 46 us; eight waves
// to a block 37.7, three steps in flight 35.8, two waves to a block 38 us, against 35.1
// (all before NT).
// NT: W by non-temporal loads, when it is read once and does not fit the caches
// (180 MB: 33 against 37 us; 4.7 MB, resident, 4.2 against 3.9 us).
constexpr int kRowsWaves = 4, kRowsDepth = 2;
template <int MT>
constexpr int kRowsLds = kRowsWaves * kRowsDepth * (32 + MT * 16) * kBK * 2;

template <int MT, bool NT, int ACT, bool GLU, bool NORM>
__global__ __launch_bounds__(kRowsWaves * kWave) void linear_act_fwd_rows_kernel(LinArgs a) {
  using A = ActOf<ACT>;
  constexpr int kWaves = kRowsWaves, D = kRowsDepth, kRows = MT * 16, kOut = GLU ? 16 : 32;
  static_assert(2 * MT <= kWaves && kRowsLds<MT> <= 64 * 1024, "one result tile per wave; LDS");
  const int64_t M = a.M, N = a.N, K = a.K;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_in_block();
  // Row blocks of one column block run on one XCD, next to each other.
  const uint32_t b = blockIdx.x;
  const uint32_t id = (b < a.map.per_xcd * kXcds) ? (b % kXcds) * a.map.per_xcd + b / kXcds : b;
  const int64_t m0 = int64_t(id % a.map.tiles_m) * kRows, n0 = int64_t(id / a.map.tiles_m) * kOut;
  const int64_t rows_x = (M - m0 < kRows) ? M - m0 : kRows;
  const int64_t rows_w = (N - n0 < kOut) ? N - n0 : kOut;
  const auto rx = make_rsrc(a.x + m0 * K, rows_x * K * 2);
  const auto rw = make_rsrc(a.w + n0 * K, rows_w * K * 2);
  const auto rw2 = make_rsrc((GLU ? a.w2 : a.w) + n0 * K, rows_w * K * 2);
  const int g = lane >> 4;
  // This wave's ring: D steps of 32 rows of W and kRows of x, 128 bytes a row, swizzled as
  // the x rows of the tiled kernel. No other wave touches it: no barrier in the K loop.
  constexpr int kStep = (32 + kRows) * kBK, kLoads = 4 + 2 * MT;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  uint16_t* const ring = lds + wave * D * kStep;
  const int r_in = lane / 8, kc = ((lane % 8) ^ (r_in >> 1)) * 8;   // rows 8 q + r_in: q even
  const int kc_odd = ((lane % 8) ^ (4 + (r_in >> 1))) * 8;          // q odd
  const uint32_t off_even = uint32_t(r_in * K * 2 + kc * 2), off_odd = uint32_t((8 + r_in) * K * 2 + kc_odd * 2);
  const uint32_t tile_off = uint32_t(16 * K * 2);
  auto load = [&](int step, int d) {
    uint16_t* S = ring + d * kStep;
    const uint32_t k0 = uint32_t(step) * kBK;
    const uint32_t even = k0 + kc < K ? off_even + k0 * 2 : kOutOfRange;
    const uint32_t odd = k0 + kc_odd < K ? off_odd + k0 * 2 : kOutOfRange;
    load_lds16<NT ? 2 : 0>(rw, S, even);
    load_lds16<NT ? 2 : 0>(rw, S + 512, odd);
    load_lds16<NT ? 2 : 0>(GLU ? rw2 : rw, S + 1024, (GLU || even == kOutOfRange) ? even : even + tile_off);
    load_lds16<NT ? 2 : 0>(GLU ? rw2 : rw, S + 1536, (GLU || odd == kOutOfRange) ? odd : odd + tile_off);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      load_lds16(rx, S + 2048 + i * 1024, even == kOutOfRange ? even : even + uint32_t(i) * tile_off);
      load_lds16(rx, S + 2048 + i * 1024 + 512, odd == kOutOfRange ? odd : odd + uint32_t(i) * tile_off);
    }
  };
  f32x4 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int steps = int((K + kBK - 1) / kBK);
#pragma unroll
  for (int d = 0; d < D; ++d) load(wave + d * kWaves, d);   // steps past the end read zeros
  const int frag = (lane & 15) * kBK, sw = (lane & 15) >> 1;
  const int u0 = (g ^ sw) * 8, u1 = ((4 + g) ^ sw) * 8;
  int d = 0;
  for (int st = wave; st < steps; st += kWaves) {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((D - 1) * kLoads) : "memory");
    const uint16_t* S = ring + d * kStep + frag;
    bf16x8 fw[2][2], fx[MT][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      fw[j][0] = *reinterpret_cast<const bf16x8*>(S + j * 1024 + u0);
      fw[j][1] = *reinterpret_cast<const bf16x8*>(S + j * 1024 + u1);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      fx[i][0] = *reinterpret_cast<const bf16x8*>(S + 2048 + i * 1024 + u0);
      fx[i][1] = *reinterpret_cast<const bf16x8*>(S + 2048 + i * 1024 + u1);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before it is loaded over
    load(st + D * kWaves, d);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j][kk], fx[i][kk], acc[i][j], 0, 0, 0);
    d = d + 1 == D ? 0 : d + 1;
  }
  // The rings' place holds the sums from here on: no load may still land there (a barrier
  // alone does not promise that), and every ring must have been read.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  auto part = reinterpret_cast<f32x4 (*)[MT][2][kWave]>(lds);
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) part[wave][i][j][lane] = acc[i][j];
  __syncthreads();

  auto total = [&](int i, int j) {
    f32x4 t = part[0][i][j][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      const f32x4 p = part[w][i][j][lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) t[r] += p[r];
    }
    return t;
  };
  // Gated: wave i takes row tile i; plain: wave 2 i + j takes row tile i, column tile j.
  constexpr int kParts = GLU ? MT : 2 * MT;
  if (wave >= kParts) return;
  const int i = GLU ? wave : wave / 2, j = GLU ? 0 : wave % 2;
  const int64_t row = m0 + i * 16 + (lane & 15), col = n0 + j * 16 + g * 4;
  const bool ok = row < M && col < N;
  const int64_t base = row * N + col;
  const float rs = (NORM && row < M) ? a.rstd[row] : 1.0f;
  f32x4 v = total(i, j);
  float f[4], o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float bj = (!GLU && a.bias != nullptr && ok) ? __uint_as_float(uint32_t(a.bias[col + e]) << 16) : 0.0f;
    f[e] = NORM ? __builtin_fmaf(v[e], rs, bj) : v[e] + bj;
  }
  const uint2 z = {pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])};
  auto unpack = [](const uint2& q, float (&t)[4]) {
    t[0] = __uint_as_float(q.x << 16);
    t[1] = __uint_as_float(q.x & 0xffff0000u);
    t[2] = __uint_as_float(q.y << 16);
    t[3] = __uint_as_float(q.y & 0xffff0000u);
  };
  unpack(z, f);
  uint32_t word = codes_of<A>(f) << (8 * g);
  word |= uint32_t(__shfl_xor(int(word), 16, kWave));
  word |= uint32_t(__shfl_xor(int(word), 32, kWave));
  if constexpr (GLU) {
    const f32x4 vu = total(i, 1);
    float fu[4], h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) fu[e] = NORM ? vu[e] * rs : vu[e];
    const uint2 u = {pack_bf16x2(fu[0], fu[1]), pack_bf16x2(fu[2], fu[3])};
    unpack(u, fu);
#pragma unroll
    for (int e = 0; e < 4; ++e) gated_value<ACT, false>(f[e], fu[e], o[e], h[e]);
    if (!ok) return;
    *reinterpret_cast<uint2*>(a.y + base) = uint2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
    *reinterpret_cast<uint2*>(a.s + base) = uint2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
    *reinterpret_cast<uint2*>(a.u + base) = u;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = act_value<ACT, false>(f[e]);
    if (!ok) return;
    *reinterpret_cast<uint2*>(a.y + base) = uint2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
  }
  if (g == 0) a.codes[base / 16] = word;
  if (a.z != nullptr) *reinterpret_cast<uint2*>(a.z + base) = z;
}

template <class C, bool GLU>
constexpr int kOutCols = GLU ? C::BN / 2 : C::BN;   // output columns per tile

template <class C, int ACT, bool GLU, bool NORM>
hipError_t launch_tile(LinArgs a, int dev, int cus, hipStream_t s) {
  const int64_t tiles_m = (a.M + C::BM - 1) / C::BM;
  const int64_t tiles_n = (a.N + kOutCols<C, GLU> - 1) / kOutCols<C, GLU>;
  const int64_t tiles = tiles_m * tiles_n;
  if (tiles > 0x3fffffff) return hipErrorInvalidValue;
  a.map = {uint32_t(tiles_m), uint32_t(tiles_n), uint32_t(tiles), uint32_t(tiles / kXcds),
           uint32_t((uint64_t(1) << 32) / uint64_t(tiles_n) - (tiles_n == 1))};
  // More than 64 KiB of dynamic LDS must be allowed explicitly, per kernel and device;
  // the attribute is set on the first launch on each device.
  static std::atomic<bool> attr_set[kMaxDevices];
  if (!attr_set[dev].load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(linear_act_fwd_kernel<C, ACT, GLU, NORM>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
    if (e != hipSuccess) return e;
    attr_set[dev].store(true, std::memory_order_release);
  }
  const int64_t slots = int64_t(cus) * C::kBlocksPerCu;
  hipLaunchKernelGGL((linear_act_fwd_kernel<C, ACT, GLU, NORM>), dim3(unsigned(tiles < slots ? tiles : slots)),
                     dim3(C::kThreads), C::kLdsBytes, s, a);
  return hipGetLastError();
}

// Estimated time of a tile configuration, in us: full rounds of the resident blocks and a
// partial one, in which a CU with one block (or two of three) is faster, the more so the fewer
// CUs have it; K steps that are longer where rows do not begin on 128-byte lines; the
// bytes of W, x and the outputs. The coefficients are non-negative least-squares fits of the
// relative error (one set per configuration, plain and gated) to the times on 256 CUs of
// M = 1 .. 16384 rows of 21 layers from 256 x 256 to 16384 x 4096 and 640 x 5120 with GELU, and of
// M = 1 .. 4096 rows of 11 gated ones from 1024 x 1024 to 14336 x 4096: 577 and 308 sizes, gated
// weights not in the caches, those near the size's best weighing more. The choice is 0.3%
// (gated 0.4%) slower than the fastest form on average, 8% (10%) at worst; with each layer's
// choices made by a fit to the other layers, 0.6% (0.8%), 21% (18%). A fit to fewer layers with
// fewer terms was 4% (2%) slower on average, 48% (24%) at worst: 4096 rows of 256 x 256 10.1 us
// against 7.7, 2500 of 4096 x 1024 41 against 32, 1500 of the gated 3072 x 768 34 against 26.
// kLinearCost.mid is 1.5% above its fit, which runs 2 to 8% short of the largest layers' times and
// took 128 x 256 tiles for the [8192 x 4096] x 11008 layer (607 against 593 us); the average is
// the same with it.
struct Cost {
  float base, step_full, step_any, step_second, step_third, step_load, full, any, second, w_mb, out_mb, x_mb, w_full_mb,
      step_ragged, load_second, load_third, load_first, third;
};
template <class C, bool GLU>
float cost(const LinArgs& a, int cus, const Cost& c) {
  const int64_t tiles = ((a.M + C::BM - 1) / C::BM) * ((a.N + kOutCols<C, GLU> - 1) / kOutCols<C, GLU>);
  const int64_t slots = int64_t(cus) * C::kBlocksPerCu, rest = tiles % slots;
  const float full = float(tiles / slots), any = rest > 0, second = rest > cus, third = rest > 2 * int64_t(cus);
  const float load = float(rest) / float(slots), ragged = a.K % 64 != 0;
  const float per_cu = float(rest) / float(cus);   // blocks of the partial round on a CU
  const float level = third > 0.0f    ? c.load_third * (per_cu - 2.0f)
                      : second > 0.0f ? c.load_second * (per_cu - 1.0f)
                                      : c.load_first * per_cu;
  const float w_mb = float(a.N) * float(a.K) * (GLU ? 4e-6f : 2e-6f);
  const float per_step = c.step_full * full + c.step_any * any + c.step_second * second + c.step_third * third +
                         c.step_load * load + level + c.step_ragged * ragged * (full + load);
  return c.base + float((a.K + kBK - 1) / kBK) * per_step + c.full * full + c.any * any + c.second * second +
         c.third * third + (c.w_mb + c.w_full_mb * full) * w_mb + c.out_mb * float(a.M) * float(a.N) * (GLU ? 6e-6f : 2e-6f) +
         c.x_mb * float(a.M) * float(a.K) * 2e-6f;
}
struct TileCosts {
  Cost big, mid, small, low;
};
constexpr TileCosts kLinearCost = {
    {6.259f, 1.45f, 0.9937f, 0, 0, 0.4028f, 8.674f, 7.53f, 0, 0, 0.1349f, 0.05882f, 0, 0.03813f, 0, 0, 0},
    {9.396f, 1.583f, 0.6624f, 0.5474f, 0, 0, 5.435f, 1.438f, 1.689f, 0, 0.138f, 0.05647f, 0, 0.2357f, 0.4247f, 0,
     0.1702f},
    {4.851f, 0.9643f, 0.4103f, 0.2916f, 0, 0, 1.463f, 0.5558f, 1.205f, 0, 0.2253f, 0.0656f, 0, 0.2431f, 0.2573f,
     0, 0.1185f},
    {4.64f, 0.8936f, 0.3183f, 0.1567f, 0.302f, 0, 1.294f, 0, 0.3331f, 0.006352f, 0.1777f, 0.0818f, 0, 0.3159f,
     0.1153f, 0.1076f, 0.04626f, 0.3873f}};
constexpr TileCosts kGatedCost = {
    {5.759f, 1.485f, 0.955f, 0, 0, 0.6037f, 7.985f, 4.71f, 0, 0, 0.07038f, 0, 0, 0, 0, 0, 0},
    {7.16f, 1.561f, 0.7105f, 0.4801f, 0, 0, 6.558f, 0.4042f, 1.888f, 0.06568f, 0.08794f, 0, 0, 0.0264f, 0.598f, 0,
     0.1684f},
    {4.17f, 0.8531f, 0.4276f, 0.3526f, 0, 0, 0.8689f, 0, 0, 0.07132f, 0.2383f, 0, 0.03413f, 0.04145f, 0.1557f, 0,
     0.0532f},
    {3.449f, 0.9078f, 0.3368f, 0.1544f, 0.332f, 0, 0.02381f, 0.08592f, 0, 0.1044f, 0.1717f, 0, 0.03171f, 0.2471f,
     0.1276f, 0.08594f, 0}};

// The same for the split-K form (in the same fit): a latency, the chain of a wave's K steps,
// longer from 1 .. 5 blocks on a CU on (`chain_more`) and with every 4 more, the bytes that all
// blocks take in, and those of W, x and the outputs.
struct RowsCost {
  float base, chain, mb, blocks, w_mb, out_mb, ragged_mb, chain_more[5], chain_round, round, x_mb;
};
struct RowsCosts {
  RowsCost rows16, rows32;
};
constexpr RowsCosts kLinearRowsCost = {
    {2.732f, 0.1367f, 0.01947f, 0.415f, 0, 1.289f, 0.002784f, {0.08641f, 0.09539f, 0.1303f, 0, 0.1894f}, 0.221f,
     0.7607f, 0.6995f},
    {2.903f, 0.1851f, 0.01669f, 0, 0, 1.12f, 0.002581f, {0.1102f, 0.3399f, 0.06528f, 0, 0.2304f}, 0.4299f, 1.404f,
     0.9115f}};
constexpr RowsCosts kGatedRowsCost = {
    {2.568f, 0.1036f, 0.0152f, 0.749f, 0.1047f, 0.3545f, 0, {0.1776f, 0.1262f, 0.124f, 0, 0.1921f}, 0.387f,
     0.1411f, 0},
    {2.686f, 0.1603f, 0.006446f, 0, 0.1014f, 1.025f, 0.0008366f, {0.2669f, 0.2736f, 0.1568f, 0, 0.2646f}, 0.5871f,
     0, 0}};
template <int MT, bool GLU>
float rows_cost(const LinArgs& a, int cus, const RowsCost& c) {
  constexpr int kOut = GLU ? 16 : 32;
  const float blocks = float((a.M + MT * 16 - 1) / (MT * 16)) * float((a.N + kOut - 1) / kOut);
  const int64_t steps = (a.K + kBK - 1) / kBK;
  const float per_cu = blocks / float(cus);
  float chain = c.chain;
  for (int i = 0; i < 5; ++i) chain += per_cu > float(i + 1) ? c.chain_more[i] : 0.0f;
  const float rounds = std::max(0.0f, std::ceil(per_cu / 4.0f) - 1.0f);
  const float mb = blocks * float(steps) * float((32 + MT * 16) * kBK * 2) * 1e-6f * 256.0f / float(cus);
  return c.base + (chain + c.chain_round * rounds) * float((steps + kRowsWaves - 1) / kRowsWaves) + c.round * rounds +
         (c.mb + c.ragged_mb * float(a.K % 64 != 0)) * mb + c.blocks * per_cu * 0.25f +
         c.w_mb * float(a.N) * float(a.K) * (GLU ? 4e-6f : 2e-6f) +
         c.out_mb * float(a.M) * float(a.N) * (GLU ? 6e-6f : 2e-6f) + c.x_mb * float(a.M) * float(a.K) * 2e-6f;
}

// The form that a layer runs in: the fastest by the estimates above.
enum Form { kRows16, kRows32, kBig, kMid, kSmall, kLow, kForms };
template <bool GLU>
Form choose_form(const LinArgs& a, int cus) {
  constexpr TileCosts c = GLU ? kGatedCost : kLinearCost;
  constexpr RowsCosts r = GLU ? kGatedRowsCost : kLinearRowsCost;
  const float t[kForms] = {rows_cost<1, GLU>(a, cus, r.rows16), rows_cost<2, GLU>(a, cus, r.rows32),
                           cost<BigTile, GLU>(a, cus, c.big),   cost<MidTile, GLU>(a, cus, c.mid),
                           cost<SmallTile, GLU>(a, cus, c.small), cost<LowTile, GLU>(a, cus, c.low)};
  return Form(std::min_element(t, t + kForms) - t);
}

template <int MT, int ACT, bool GLU, bool NORM>
hipError_t launch_rows(LinArgs a, hipStream_t s) {
  constexpr int kOut = GLU ? 16 : 32;
  const int64_t tiles_m = (a.M + MT * 16 - 1) / (MT * 16), tiles_n = (a.N + kOut - 1) / kOut;
  const int64_t blocks = tiles_m * tiles_n;
  if (blocks > 0x3fffffff) return hipErrorInvalidValue;
  a.map = {uint32_t(tiles_m), uint32_t(tiles_n), uint32_t(blocks), uint32_t(blocks / kXcds), 0u};
  // Non-temporal from 32 MiB of weights on, when one row block reads them (see the kernel).
  const bool nt = tiles_m == 1 && a.N * a.K * (GLU ? 4 : 2) > (int64_t(32) << 20);
  const auto kernel = nt ? linear_act_fwd_rows_kernel<MT, true, ACT, GLU, NORM>
                         : linear_act_fwd_rows_kernel<MT, false, ACT, GLU, NORM>;
  hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(kRowsWaves * kWave), kRowsLds<MT>, s, a);
  return hipGetLastError();
}

template <int ACT, bool GLU, bool NORM>
hipError_t launch_lin(const LinArgs& a, hipStream_t s) {
  int dev = 0, cus = 0;
  const hipError_t e = current_device(dev, cus);
  if (e != hipSuccess) return e;
  switch (choose_form<GLU>(a, cus)) {
    case kRows16: return launch_rows<1, ACT, GLU, NORM>(a, s);
    case kRows32: return launch_rows<2, ACT, GLU, NORM>(a, s);
    case kBig: return launch_tile<BigTile, ACT, GLU, NORM>(a, dev, cus, s);
    case kMid: return launch_tile<MidTile, ACT, GLU, NORM>(a, dev, cus, s);
    case kSmall: return launch_tile<SmallTile, ACT, GLU, NORM>(a, dev, cus, s);
    default: return launch_tile<LowTile, ACT, GLU, NORM>(a, dev, cus, s);
  }
}

}  // namespace lin

hipError_t current_device(int& dev, int& cus) {
  static std::atomic<int> known[kMaxDevices];
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  cus = known[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    known[dev].store(cus, std::memory_order_relaxed);
  }
  return hipSuccess;
}

LinearForm linear_form(bool gated, int64_t M, int64_t N, int64_t K) {
  int dev = 0, cus = 256;
  if (current_device(dev, cus) != hipSuccess) cus = 256;   // no device here
  lin::LinArgs a{};
  a.M = M;
  a.N = N;
  a.K = K;
  const lin::Form f = gated ? lin::choose_form<true>(a, cus) : lin::choose_form<false>(a, cus);
  auto of = [&](auto tile) -> LinearForm {
    using C = decltype(tile);
    const int64_t cols = gated ? C::BN / 2 : C::BN;
    const int64_t tiles = ((M + C::BM - 1) / C::BM) * ((N + cols - 1) / cols), slots = int64_t(cus) * C::kBlocksPerCu;
    return {int(f), (tiles + slots - 1) / slots};
  };
  switch (f) {
    case lin::kBig: return of(lin::BigTile{});
    case lin::kMid: return of(lin::MidTile{});
    case lin::kSmall: return of(lin::SmallTile{});
    case lin::kLow: return of(lin::LowTile{});
    default: return {int(f), 1};
  }
}

hipError_t launch_linear_act_fwd(int act, int64_t M, int64_t N, int64_t K, const void* x,
                                 const void* w, const void* bias, void* y, uint32_t* codes,
                                 void* z, hipStream_t s) {
  const lin::LinArgs a{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), nullptr,
                       static_cast<const uint16_t*>(bias), static_cast<uint16_t*>(y), nullptr,
                       nullptr, codes, static_cast<uint16_t*>(z), M, N, K, nullptr, {}};
  return act == kGelu ? lin::launch_lin<kGelu, false, false>(a, s) : lin::launch_lin<kSilu, false, false>(a, s);
}

hipError_t launch_linear_glu_fwd(int64_t M, int64_t N, int64_t K, const void* x, const void* w_gate,
                                 const void* w_up, void* h, void* s_out, void* u, uint32_t* codes,
                                 void* g, hipStream_t s) {
  const lin::LinArgs a{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w_gate),
                       static_cast<const uint16_t*>(w_up), nullptr, static_cast<uint16_t*>(h),
                       static_cast<uint16_t*>(s_out), static_cast<uint16_t*>(u), codes,
                       static_cast<uint16_t*>(g), M, N, K, nullptr, {}};
  return lin::launch_lin<kSilu, true, false>(a, s);
}

hipError_t launch_linear_rms_act_fwd(int act, int64_t M, int64_t N, int64_t K, float eps,
                                     const void* x, const void* w, const void* bias, void* y,
                                     uint32_t* codes, void* pre, void* z_norm, float* rstd,
                                     hipStream_t s) {
  hipError_t e = launch_norm_fwd(false, true, M, K, eps, x, z_norm, rstd, true, s);
  if (e != hipSuccess) return e;
  const lin::LinArgs a{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), nullptr,
                       static_cast<const uint16_t*>(bias), static_cast<uint16_t*>(y), nullptr,
                       nullptr, codes, static_cast<uint16_t*>(pre), M, N, K, rstd, {}};
  return act == kGelu ? lin::launch_lin<kGelu, false, true>(a, s) : lin::launch_lin<kSilu, false, true>(a, s);
}

hipError_t launch_linear_rms_glu_fwd(int64_t M, int64_t N, int64_t K, float eps, const void* x,
                                     const void* w_gate, const void* w_up, void* h, void* s_out,
                                     void* u, uint32_t* codes, void* g, void* z_norm, float* rstd,
                                     hipStream_t s) {
  hipError_t e = launch_norm_fwd(false, true, M, K, eps, x, z_norm, rstd, true, s);
  if (e != hipSuccess) return e;
  const lin::LinArgs a{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w_gate),
                       static_cast<const uint16_t*>(w_up), nullptr, static_cast<uint16_t*>(h),
                       static_cast<uint16_t*>(s_out), static_cast<uint16_t*>(u), codes,
                       static_cast<uint16_t*>(g), M, N, K, rstd, {}};
  return lin::launch_lin<kSilu, true, true>(a, s);
}

}  // namespace lmbp
