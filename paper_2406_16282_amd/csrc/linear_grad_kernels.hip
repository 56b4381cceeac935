// Backward of the fused linear layers' parameters, for gfx950: dW = dz^T x (fp32 sums over
// the rows, one rounding to bf16) and, for the layers with an activation, dz = dy *
// slope[code] together with db, the column sums of the rounded dz.
//
// grad_weight_kernel. dz [M x N] and x [M x K] are contracted over their rows, so both
// MFMA operands lie across memory. They are staged in LDS as they are (32 rows of BM
// columns of dz and BN of x per slot, whole row pieces of 256 to 512 bytes per load) and
// read with the transposing LDS read (ds_read_b64_tr_b16: of 16 lanes, lane q passes the
// address of columns 4 (q % 4) .. + 3 of row q / 4 and lane i gets the 4 rows of column i;
// checked on the hardware). Lane group g = l / 16 takes rows 4 g .. + 3 and 16 + 4 g ..
// + 3 of a slot in both operands, which is all that the product asks for. The rows of a
// slot start 256 or 512 bytes apart, on the same banks: the 32-byte units of row r are
// stored at unit ^ 2 (r % 4), so that the 16 lanes of a read fall on distinct banks.
// Column 4 a + c of operand tile j is output column 8 a + 4 (j % 2) + c + 32 (j / 2) of the
// wave's 64: a lane stores runs of 8 columns.
//
// The loop is that of the forward kernel: a ring of slots (one per 32 rows), the next
// fragments read while the present ones are multiplied, one barrier per slot with
// kRing - 2 slots of loads in flight, persistent blocks whose stream of loads runs on into
// the next unit of work. The loads are written as asm: of the builtin the compiler knows
// that it writes LDS, and it waits for all of them before every transposing read (634 us
// at most were 972 then, at 8192 rows of 11008 x 4096). They have no result register; the
// waits are the loop's own. The load cursor is stepped with additions only (its
// multiplications in every half step cost 581 against 634 us).
//
// A unit is a tile of dW over a share of the rows: small dW are split over the rows to fill
// the device, the shares' fp32 sums go to a workspace and are added in order by a second
// kernel. What bounds it: for large dW the card's power, as the forward; for split ones
// the partial sums' traffic besides. Measured against the library's product, operands not in
// the caches: 8192 rows of 11008 x 4096 581 against 785 us, 12608 of 3072 x 768 80 against 144,
// 2000 of 3072 x 768 22 against 32, 64 of 11008 x 4096 24 against 34 us.
#include "act_codes.hpp"
#include "lmbp_device.hpp"
#include "lmbp_launch.hpp"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace lmbp {
namespace lgrad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kRowsPerSlot = 32;

// A block computes BM rows (output features) x BN columns (input features) of dW with WM x
// WN waves, each BM/WM x 64. MINW: waves per SIMD that the registers are budgeted for.
template <int BM_, int BN_, int WM_, int WN_, int MINW_, int RING_ = 4>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, kMinWaves = MINW_;
  static constexpr int kWaves = WM * WN, kThreads = kWaves * kWave;
  static constexpr int TM = BM / WM / 16, TN = 4;
  static constexpr int kSlotElems = (BM + BN) * kRowsPerSlot;
  static constexpr int kRing = RING_;
  static constexpr int kBlocksPerCu = kMinWaves * 4 / kWaves;
  static constexpr int kLA = BM / 16 / kWaves, kLB = BN / 16 / kWaves;
  static constexpr int kLdsBytes = kRing * kSlotElems * 2;
  static_assert(BN / WN == 64, "wave tile");
  static_assert(kLA >= 1 && kLB >= 1 && (BM / 16) % kWaves == 0 && (BN / 16) % kWaves == 0, "loads");
  static_assert(kLdsBytes * kBlocksPerCu <= 160 * 1024, "LDS per CU");
};
using BigTile = Tile<256, 256, 2, 4, 2>;      // one block of 8 waves per CU
using MidTile = Tile<128, 256, 1, 4, 2, 3>;   // two blocks of 4 waves
using SmallTile = Tile<128, 128, 2, 2, 2>;    // two blocks of 4 waves

__device__ inline u32x4 rsrc(uint64_t base, uint32_t bytes) {
  return u32x4{uint32_t(base), uint32_t(base >> 32) & 0xffffu, bytes, 0x00020000u};
}
// 16 bytes per lane into LDS at `dst` + lane * 16 (see the file comment). The wait states
// cover a resource whose registers a VALU operation has just written (5, with the move).
// The compiler reserves m0 for itself and warns that it cannot keep a value there across
// the asm; the clobber is to say just that, so that it never counts on one.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void load_lds16(const u32x4& r, uint32_t dst, uint32_t offset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(dst), "v"(offset), "s"(r) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ inline uint32_t lds_addr(const uint16_t* p) { return uint32_t(uintptr_t((lds_void*)p)); }
__device__ inline s16x4 read_tr(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
}
// Scheduling groups: DS LDS reads spread over the first half of MF MFMAs.
template <int MF, int DS, int I = 0>
__device__ inline void spread() {
  if constexpr (I < MF) {
    constexpr int W = MF / 2 < 1 ? 1 : MF / 2;
    constexpr int ds = I < W ? DS * (I + 1) / W - DS * I / W : 0;
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (ds > 0) __builtin_amdgcn_sched_group_barrier(0x100, ds, 0);
    spread<MF, DS, I + 1>();
  }
}

struct GradArgs {
  const uint16_t* dz;   // [M x N]
  const uint16_t* x;    // [M x K]
  uint16_t* dw;         // [N x K]
  float* part;          // [splits][N x K]
  int64_t M, N, K;
  uint32_t tiles_n, tiles_k, tiles, units, per_xcd, steps_per_split, steps;   // steps of 64 rows
};

template <class C>
__global__ __launch_bounds__(C::kThreads, C::kMinWaves) void grad_weight_kernel(GradArgs a) {
  constexpr int BM = C::BM, BN = C::BN, TM = C::TM, TN = C::TN, kWaves = C::kWaves;
  constexpr int kLA = C::kLA, kLB = C::kLB, kL = kLA + kLB, kRing = C::kRing, kSlot = C::kSlotElems;
  const int64_t M = a.M, N = a.N, K = a.K;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_in_block();
  const int wm = wave / C::WN, wn = wave % C::WN;

  // Byte offsets of this lane's 16-byte chunks within a slot's rows. Columns beyond the
  // matrix read the next row's (in range, in results that are not stored) or zeros.
  uint32_t ld_a[kLA], ld_b[kLB];
#pragma unroll
  for (int q = 0; q < kLA; ++q) {
    const int p = (wave + kWaves * q) * 64 + lane;      // 16-byte position in the slot's A part
    const int row = p / (BM / 8), c = p % (BM / 8);
    ld_a[q] = uint32_t(row * N * 2 + (((c >> 1) ^ (2 * (row & 3))) * 2 + (c & 1)) * 16);
  }
#pragma unroll
  for (int q = 0; q < kLB; ++q) {
    const int p = (wave + kWaves * q) * 64 + lane;
    const int row = p / (BN / 8), c = p % (BN / 8);
    ld_b[q] = uint32_t(row * K * 2 + (((c >> 1) ^ (2 * (row & 3))) * 2 + (c & 1)) * 16);
  }

  auto tile_of = [&](uint32_t u, uint32_t& split, int64_t& n0, int64_t& k0) {
    const uint32_t id = (u < a.per_xcd * kXcds) ? (u % kXcds) * a.per_xcd + u / kXcds : u;
    split = id / a.tiles;
    const uint32_t t = id % a.tiles;
    // four tile columns at a time, so that the blocks of an XCD share rows of both operands
    const uint32_t group = 4 * a.tiles_n;
    const uint32_t first = t / group * 4;
    const uint32_t w = (a.tiles_k - first < 4) ? a.tiles_k - first : 4;
    const uint32_t r = t % group;
    n0 = int64_t(r / w) * BM;
    k0 = int64_t(first + r % w) * BN;
  };
  // Load cursor: slots of the current unit still to load, and how many of them are whole.
  uint32_t l_unit = blockIdx.x;
  int l_slots = 0, l_whole = 0;
  int64_t l_row = 0, l_n0 = 0, l_k0 = 0;
  uint64_t pa = 0, pb = 0;
  uint32_t na = 0, nb = 0;   // records: bytes in range
  auto ranges = [&]() {   // records of a slot whose rows end before the 32nd
    const int64_t rows = l_row >= M ? 0 : M - l_row;
    na = rows > 0 ? uint32_t((rows * N - l_n0) * 2) : 0u;
    nb = rows > 0 ? uint32_t((rows * K - l_k0) * 2) : 0u;
  };
  auto enter = [&]() {
    if (l_unit < a.units) {
      uint32_t split;
      tile_of(l_unit, split, l_n0, l_k0);
      const uint32_t left = a.steps - split * a.steps_per_split;
      l_slots = 2 * int(left < a.steps_per_split ? left : a.steps_per_split);
      l_row = int64_t(split) * a.steps_per_split * 64;
      const int64_t whole = (M - l_row) / kRowsPerSlot;
      l_whole = int(whole < l_slots ? whole : l_slots);
      pa = reinterpret_cast<uint64_t>(a.dz + l_row * N + l_n0);
      pb = reinterpret_cast<uint64_t>(a.x + l_row * K + l_k0);
      na = uint32_t((kRowsPerSlot * N - l_n0) * 2);
      nb = uint32_t((kRowsPerSlot * K - l_k0) * 2);
      if (l_whole == 0) ranges();
    } else {   // past the last unit: zeros
      l_slots = l_whole = 0x7fffffff;
      na = nb = 0u;
    }
  };
  auto load = [&](uint32_t S, int q) {
    if (q < kLA) load_lds16(rsrc(pa, na), S + (wave + kWaves * q) * 1024, ld_a[q < kLA ? q : 0]);
    else load_lds16(rsrc(pb, nb), S + BM * kRowsPerSlot * 2 + (wave + kWaves * (q - kLA)) * 1024, ld_b[q < kLA ? 0 : q - kLA]);
  };
  auto advance = [&]() {
    pa += uint64_t(kRowsPerSlot) * N * 2;
    pb += uint64_t(kRowsPerSlot) * K * 2;
    --l_whole;
    if (--l_slots == 0) {
      l_unit += gridDim.x;
      enter();
    } else if (l_whole <= 0) {
      l_row = (M / kRowsPerSlot - l_whole) * kRowsPerSlot;
      ranges();
    }
  };

  // fragment reads: piece q of lane group g: rows 4 g + q / 4 (and 16 more)
  const int g = lane >> 4, q4 = (lane & 15) >> 2, qc = lane & 3;
  const int row = 4 * g + q4, f = 2 * (row & 3);   // rows 16 apart have the same swizzle
  int a_un[TM], b_un[2];
#pragma unroll
  for (int i = 0; i < TM; ++i) a_un[i] = row * BM + ((wm * TM + i) ^ f) * 16 + qc * 4;
#pragma unroll
  for (int h = 0; h < 2; ++h)
    b_un[h] = BM * kRowsPerSlot + row * BN + ((wn * 4 + 2 * h + (qc >> 1)) ^ f) * 16 + (qc & 1) * 8;
  bf16x8 fa[2][TM], fb[2][TN];
  auto read_b = [&](const uint16_t* S, int buf, int j) {
    const uint16_t* p = S + b_un[j / 2] + (j & 1) * 4;
    const s16x4 lo = read_tr(p), hi = read_tr(p + 16 * BN);
    fb[buf][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read_a = [&](const uint16_t* S, int buf, int i) {
    const uint16_t* p = S + a_un[i];
    const s16x4 lo = read_tr(p), hi = read_tr(p + 16 * BM);
    fa[buf][i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  f32x4 acc[TM][TN];
  // One half step: 4 segments of MFMAs of the fragments in buf, with the loads into slot
  // `fill` and the reads of the next fragments from slot S spread over them.
  auto segment = [&](auto number, int buf, uint32_t fill, const uint16_t* S) {
    constexpr int sg = decltype(number)::value;
#pragma unroll
    for (int q = 0; q < kL; ++q)
      if (q * 4 / kL == sg) load(fill, q);
    if constexpr (sg == 0) {
#pragma unroll
      for (int j = 0; j < TN; ++j) read_b(S, buf ^ 1, j);
    } else if constexpr (sg < 3) {
#pragma unroll
      for (int i = (sg - 1) * TM / 2; i < sg * TM / 2; ++i) read_a(S, buf ^ 1, i);
    }
#pragma unroll
    for (int i = sg * TM / 4; i < (sg + 1) * TM / 4; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[buf][j], fa[buf][i], acc[i][j], 0, 0, 0);
    spread<TM * TN / 4, sg == 0 ? 2 * TN : sg < 3 ? TM : 0>();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto half = [&](int buf, uint32_t fill, const uint16_t* S) {
    segment(std::integral_constant<int, 0>{}, buf, fill, S);
    segment(std::integral_constant<int, 1>{}, buf, fill, S);
    segment(std::integral_constant<int, 2>{}, buf, fill, S);
    segment(std::integral_constant<int, 3>{}, buf, fill, S);
  };
  auto sync = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 2) * kL) : "memory");
    asm volatile("s_barrier" ::: "memory");
  };
  auto next = [&](int v, int d) { v += d; return v >= kRing ? v - kRing : v; };

  const uint32_t lds0 = lds_addr(lds);
  enter();
#pragma unroll
  for (int d = 0; d < kRing; ++d) {
#pragma unroll
    for (int q = 0; q < kL; ++q) load(lds0 + d * kSlot * 2, q);
    advance();
  }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kRing - 2) * kL) : "memory");
  asm volatile("s_barrier" ::: "memory");
  int slot = 0;
  for (uint32_t unit = blockIdx.x; unit < a.units; unit += gridDim.x) {
    uint32_t split;
    int64_t n0, k0;
    tile_of(unit, split, n0, k0);
    const uint32_t left = a.steps - split * a.steps_per_split;
    const int steps = int(left < a.steps_per_split ? left : a.steps_per_split);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < TN; ++j) read_b(lds + slot * kSlot, 0, j);
#pragma unroll
    for (int i = 0; i < TM; ++i) read_a(lds + slot * kSlot, 0, i);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
    for (int st = 0; st < steps; ++st) {
      const uint32_t f0 = lds0 + slot * kSlot * 2;
      const int one = next(slot, 1);
      const uint32_t f1 = lds0 + one * kSlot * 2;
      slot = next(slot, 2);
      half(0, f0, lds + one * kSlot);
      advance();
      sync();
      half(1, f1, lds + slot * kSlot);
      advance();
      sync();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t n = n0 + wm * TM * 16 + i * 16 + (lane & 15);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t k = k0 + wn * 64 + h * 32 + g * 8;
        if (n < N && k < K) {
          if (a.part != nullptr) {
            f32x4* p = reinterpret_cast<f32x4*>(a.part + (int64_t(split) * N + n) * K + k);
            p[0] = acc[i][2 * h];
            p[1] = acc[i][2 * h + 1];
          } else {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = acc[i][2 * h + e / 4][e % 4];
            *reinterpret_cast<u32x4*>(a.dw + n * K + k) = BF16::pack(v);
          }
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// dz = dy * slope[code] as the activation kernels compute it, and the sums of the rounded dz
// over a block's rows, per column (fp32): the read of dz that a separate sum would take is
// saved. 2^lanes_log lanes of a wave take a row's columns, 8 per lane, the others the rows
// after it (narrow rows); a wave has ROWS such pieces requested at once, the four waves of
// a block take consecutive ones, and a block goes on gridDim.y such groups further down. In
// the end the lanes and waves of a column add their sums. The blocks along the columns are
// neighbours, so that whole rows are in flight together: with those along the rows as
// neighbours, blocks next to each other were a power of two apart for the usual widths.
// Needs 16-byte aligned tensors and N % 16 == 0.
template <int ACT, int ROWS>
__global__ __launch_bounds__(256) void act_bwd_cols_kernel(const void* dy, const uint32_t* __restrict__ codes,
                                                           void* dz, float* __restrict__ sums, int64_t M,
                                                           int64_t N, int lanes_log) {
  using A = ActOf<ACT>;
  __shared__ float part[4][8][kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_in_block();
  const int lanes = 1 << lanes_log, piece = kWave >> lanes_log;   // rows of a piece
  const int64_t col = int64_t(blockIdx.x) * 512 + (lane & (lanes - 1)) * 8;
  const bool in_col = col < N;
  float sum[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t step = int64_t(gridDim.y) * (4 * ROWS * piece);
  for (int64_t base = (int64_t(blockIdx.y) * 4 + wave) * (ROWS * piece); base < M; base += step) {
    const int64_t row = base + (lane >> lanes_log);
    u32x4 v[ROWS];
    uint32_t w[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int64_t at = (row + r * piece) * N + col;
      const bool in = in_col && row + r * piece < M;
      v[r] = in ? ldg16<true>(dy, at / 8) : u32x4{0u, 0u, 0u, 0u};
      w[r] = in ? codes[at / 16] >> (16 * (lane & 1)) : 0u;
    }
    float group[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      float f[8];
      BF16::unpack(v[r], f);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = f[e] * seg_slope<A>((w[r] >> (2 * e)) & 3u);
      const u32x4 out = BF16::pack(f);
      if (in_col && row + r * piece < M) stg16(dz, ((row + r * piece) * N + col) / 8, out);
      BF16::unpack(out, f);
#pragma unroll
      for (int e = 0; e < 8; ++e) group[e] += f[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] += group[e];
  }
  for (int off = lanes; off < kWave; off *= 2) {
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] += __shfl_xor(sum[e], off, kWave);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[wave][e][lane] = sum[e];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int e = threadIdx.x / kWave + 4 * c;
    const float t = ((part[0][e][lane] + part[1][e][lane]) + part[2][e][lane]) + part[3][e][lane];
    if (in_col && lane < lanes) sums[int64_t(blockIdx.y) * N + col + e] = t;
  }
}

// The second passes, in one launch. The first dw_blocks blocks: dw = bf16(sum of the
// splits' partial sums, in split order), 8 values per thread. The others: db = bf16(sum of
// the row blocks' column sums, in a fixed order), 16 columns per block, 16 threads to a
// column, each with eight loads in flight (one thread to a column and a quarter of the rows
// was a chain of 50 loads: 23 us).
__global__ __launch_bounds__(256) void grad_reduce_kernel(const float* __restrict__ part, uint16_t* dw, int64_t n,
                                                          int splits, int64_t dw_blocks,
                                                          const float* __restrict__ sums, uint16_t* db,
                                                          int64_t cols, int64_t row_blocks) {
  __shared__ float red[16][16];
  if (int64_t(blockIdx.x) >= dw_blocks) {
    const int c = threadIdx.x % 16, q = threadIdx.x / 16;
    const int64_t col = (int64_t(blockIdx.x) - dw_blocks) * 16 + c;   // cols is a multiple of 16
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t b = q; b < row_blocks; b += 128) {
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u % 4] += b + 16 * u < row_blocks ? sums[(b + 16 * u) * cols + col] : 0.0f;
    }
    red[q][c] = (t[0] + t[1]) + (t[2] + t[3]);
    __syncthreads();
    if (q == 0) {
      float sum = red[0][c];
#pragma unroll
      for (int r = 1; r < 16; ++r) sum += red[r][c];
      BF16::store1(db, col, sum);
    }
    return;
  }
  const int64_t i = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  f32x4 s0 = *reinterpret_cast<const f32x4*>(part + i), s1 = *reinterpret_cast<const f32x4*>(part + i + 4);
  for (int s = 1; s < splits; ++s) {
    const f32x4* p = reinterpret_cast<const f32x4*>(part + s * n + i);
    const f32x4 a = p[0], b = p[1];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s0[e] += a[e];
      s1[e] += b[e];
    }
  }
  const float v[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
  *reinterpret_cast<u32x4*>(dw + i) = BF16::pack(v);
}

// Estimated time, in us, of a tile configuration with the rows split `splits` times: full
// rounds of the resident blocks and a partial one (in which a CU with one block, and few CUs
// with two, are faster), the partial sums' traffic and the second pass, the bytes of dW, dz and
// x, and the operands beyond what the memory-side cache keeps. Non-negative least-squares fit
// of the relative error, times near the size's best weighing more, to M = 1 .. 50000 rows of
// 20 layers from 16 x 8 to 13824 x 5120, 1 to 32 splits, on 256 CUs (356 sizes). The choice is 0.6%
// slower than the fastest plan on average and 13% at worst; with each layer's choices made
// by a fit to the others, 0.6% and 13%. A fit to five layers, fewer terms and at most 12 splits
// was 3.2% slower on average, 62% at worst: 6304 rows of 5120 x 1280 122 us against 99 (the
// library's product: 108), 50000 of 64 x 64 43 against 27.5 (88). The library's product is
// 1.47 times as slow on average; it is faster for the 16 x 8 layer from 197 to 4096 rows (by up
// to 1.3 us of 5 to 10) and by 2 to 4% at four other sizes (4096 rows of 2048 x 5632 98 us).
struct Cost {
  float base, step_full, step_any, step_second, full, any, part_mb, split, out_mb, beyond_mb, load_first, load_second,
      dz_mb, x_mb, per_split, second, step_load, load, split_mb;
};
constexpr Cost kBigCost = {4.484f, 1.553f, 1.078f, 0, 3.471f, 0.567f, 0.2069f, 1.242f, 0.0496f, 0, 0.3734f, 0,
                           0.03283f, 0.02745f, 0.2187f, 0, 0, 6.094f, 0.2307f};
constexpr Cost kMidCost = {3.969f, 1.565f, 0.8659f, 0.3437f, 0, 0, 0.2849f, 1.272f, 0.138f, 0.01897f, 0.001652f,
                           0.5249f, 0.03913f, 0.03597f, 0.2503f, 0.03601f, 0, 3.14f, 0.1684f};
constexpr Cost kSmallCost = {3.511f, 0.9227f, 0.526f, 0.1757f, 0, 0, 0.2531f, 1.199f, 0.1548f, 0.02875f, 0, 0.2816f,
                             0.08778f, 0.04232f, 0.2617f, 0, 0, 1.495f, 0.4445f};

// The partial sums take at most 256 MiB, which no size that was measured asks for: 7 shares of
// 3072 x 768 (12608 rows) are 66 MB, 4 of 5632 x 2048 (16384 rows) 185.
constexpr int64_t kMaxSplits = 32, kMaxPartial = int64_t(256) << 20;
using Plan = LinearGradPlan;

template <class C>
void consider(int tile, const Cost& c, int64_t M, int64_t N, int64_t K, int cus, float& best, Plan& plan) {
  const int64_t steps = std::max<int64_t>(1, (M + 63) / 64);
  const int64_t tiles = ((N + C::BM - 1) / C::BM) * ((K + C::BN - 1) / C::BN);
  const int64_t slots = int64_t(cus) * C::kBlocksPerCu;
  const float mb = float(N) * float(K) * 4e-6f;
  const float dz_mb = float(M) * float(N) * 2e-6f, x_mb = float(M) * float(K) * 2e-6f;
  const float beyond = std::max(0.0f, dz_mb + x_mb - 60.0f);
  for (int64_t want = 1; want <= kMaxSplits && want <= steps; want += want < 12 ? 1 : 4) {
    const int64_t per = (steps + want - 1) / want, splits = (steps + per - 1) / per;
    if (splits != want) continue;   // the same shares as a smaller number gives
    if (splits > 1 && splits * N * K * int64_t(sizeof(float)) > kMaxPartial) break;
    const int64_t rest = tiles * splits % slots;
    const float full = float(tiles * splits / slots), any = rest > 0, second = rest > cus;
    const float per_cu = float(rest) / float(cus), load = float(rest) / float(slots);
    const float per_step = c.step_full * full + c.step_any * any + c.step_second * second + c.step_load * load +
                           (second > 0.0f ? c.load_second * (per_cu - 1.0f) : c.load_first * per_cu);
    const float t = c.base + per_step * float(per) + c.full * full + c.any * any + c.second * second + c.load * load +
                    (splits > 1 ? (c.part_mb * mb + c.per_split) * float(splits) + c.split + c.split_mb * mb : 0.0f) +
                    c.out_mb * mb * 0.5f + c.beyond_mb * beyond + c.dz_mb * dz_mb + c.x_mb * x_mb;
    if (t < best) {
      best = t;
      plan = {tile, splits, per};
    }
  }
}

Plan make_plan(int64_t M, int64_t N, int64_t K, int cus) {
  Plan plan;
  float best = 3.0e38f;
  consider<BigTile>(0, kBigCost, M, N, K, cus, best, plan);
  consider<MidTile>(1, kMidCost, M, N, K, cus, best, plan);
  consider<SmallTile>(2, kSmallCost, M, N, K, cus, best, plan);
  return plan;
}

template <class C>
hipError_t launch_tile(GradArgs a, const Plan& plan, int dev, int cus, hipStream_t s) {
  const int64_t tiles_n = (a.N + C::BM - 1) / C::BM, tiles_k = (a.K + C::BN - 1) / C::BN;
  const int64_t units = tiles_n * tiles_k * plan.splits;
  if (units > 0x3fffffff) return hipErrorInvalidValue;
  a.tiles_n = uint32_t(tiles_n);
  a.tiles_k = uint32_t(tiles_k);
  a.tiles = uint32_t(tiles_n * tiles_k);
  a.units = uint32_t(units);
  a.per_xcd = a.units / kXcds;
  a.steps = uint32_t(std::max<int64_t>(1, (a.M + 63) / 64));
  a.steps_per_split = uint32_t(plan.per);
  // More than 64 KiB of dynamic LDS must be allowed explicitly, per kernel and device.
  static std::atomic<bool> attr_set[kMaxDevices];
  if (!attr_set[dev].load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(grad_weight_kernel<C>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
    if (e != hipSuccess) return e;
    attr_set[dev].store(true, std::memory_order_release);
  }
  const int64_t slots = int64_t(cus) * C::kBlocksPerCu;
  hipLaunchKernelGGL((grad_weight_kernel<C>), dim3(unsigned(units < slots ? units : slots)), dim3(C::kThreads),
                     C::kLdsBytes, s, a);
  return hipGetLastError();
}

// Launch of act_bwd_cols_kernel: pieces per wave at once, lanes to a row (log2), blocks along
// the columns and along the rows, the latter with the same number of groups each (one
// less in the last ones). Four pieces and at most 1280 blocks (5 per CU) up to 2^27 values,
// eight and at most 2048 beyond: 12608 x 4096 43.5 us with four, 51 with eight; 300000 x 768
// 228 with eight, 250 with four; 1024 blocks lose up to 13% (3152 x 5632), 1792 and more up to
// 15% (50000 x 768). Measured with the second pass, before (one block to 32 rows, any size,
// those along the rows as neighbours) and now: 700 x 3072 11.5 and 9.4 us, 12608 x 3072 42 and
// 35.5, 300000 x 4112 1690 and 1300 (a separate sum after the activation kernel: 1380),
// 300000 x 16 104 and 13.4 (25); of 200 sizes four are slower, by 5 to 8% (4096 x 4000: 20.2 and
// 21.9). The number of blocks also keeps the launch within 2^32 threads at any M.
struct ColPlan {
  int pieces, lanes_log;
  int64_t columns, rows;
};
ColPlan col_plan(int64_t M, int64_t N) {
  const bool large = M * N > (int64_t(1) << 27);
  ColPlan p{large ? 8 : 4, 6, (N + 511) / 512, 1};
  while (p.lanes_log > 1 && N <= (4 << p.lanes_log)) --p.lanes_log;
  const int64_t group = int64_t(4 * p.pieces) << (6 - p.lanes_log);
  const int64_t groups = std::max<int64_t>(1, (M + group - 1) / group);
  const int64_t most = large ? 2048 : 1280;
  const int64_t each = (groups * p.columns + most - 1) / most;
  p.rows = (groups + each - 1) / each;
  return p;
}

int64_t partial_floats(int64_t N, int64_t K, const Plan& p) { return p.splits > 1 ? p.splits * N * K : 0; }

}  // namespace lgrad

LinearGradPlan linear_grad_plan(int64_t M, int64_t N, int64_t K) {
  int dev = 0, cus = 256;
  if (current_device(dev, cus) != hipSuccess) cus = 256;   // a size to plan with, no device here
  return lgrad::make_plan(M, N, K, cus);
}

size_t linear_grad_workspace(int64_t M, int64_t N, int64_t K, bool bias, const LinearGradPlan& plan) {
  return size_t(lgrad::partial_floats(N, K, plan) + (bias ? lgrad::col_plan(M, N).rows * N : 0)) * sizeof(float);
}

LinearGradForm linear_grad_form(int64_t M, int64_t N, int64_t K) {
  int dev = 0, cus = 256;
  if (current_device(dev, cus) != hipSuccess) cus = 256;   // no device here
  const lgrad::Plan plan = lgrad::make_plan(M, N, K, cus);
  auto rounds = [&](auto tile) {
    using C = decltype(tile);
    const int64_t units = ((N + C::BM - 1) / C::BM) * ((K + C::BN - 1) / C::BN) * plan.splits;
    const int64_t slots = int64_t(cus) * C::kBlocksPerCu;
    return (units + slots - 1) / slots;
  };
  return {plan.tile, plan.splits, plan.tile == 0 ? rounds(lgrad::BigTile{}) : plan.tile == 1 ? rounds(lgrad::MidTile{})
                                                                                             : rounds(lgrad::SmallTile{})};
}

hipError_t launch_linear_grad(int act, int64_t M, int64_t N, int64_t K, const void* dy, const uint32_t* codes,
                              const void* x, void* dz, void* dw, void* db, void* workspace,
                              const LinearGradPlan& plan, hipStream_t s) {
  using namespace lgrad;
  int dev = 0, cus = 0;
  hipError_t e = current_device(dev, cus);
  if (e != hipSuccess) return e;
  float* const part = static_cast<float*>(workspace);
  float* const sums = part + (dw != nullptr ? partial_floats(N, K, plan) : 0);
  const ColPlan cols = col_plan(M, N);
  if (db != nullptr) {
    const auto kernel = act == kGelu ? (cols.pieces == 4 ? act_bwd_cols_kernel<kGelu, 4> : act_bwd_cols_kernel<kGelu, 8>)
                                     : (cols.pieces == 4 ? act_bwd_cols_kernel<kSilu, 4> : act_bwd_cols_kernel<kSilu, 8>);
    hipLaunchKernelGGL(kernel, dim3(unsigned(cols.columns), unsigned(cols.rows)), dim3(256), 0, s, dy, codes, dz, sums,
                       M, N, cols.lanes_log);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const bool split = dw != nullptr && plan.splits > 1;
  if (dw != nullptr) {
    GradArgs a{};
    a.dz = static_cast<const uint16_t*>(dz);
    a.x = static_cast<const uint16_t*>(x);
    a.dw = static_cast<uint16_t*>(dw);
    a.part = split ? part : nullptr;
    a.M = M;
    a.N = N;
    a.K = K;
    e = plan.tile == 0 ? launch_tile<BigTile>(a, plan, dev, cus, s)
        : plan.tile == 1 ? launch_tile<MidTile>(a, plan, dev, cus, s) : launch_tile<SmallTile>(a, plan, dev, cus, s);
    if (e != hipSuccess) return e;
  }
  const int64_t dw_blocks = split ? (N * K / 8 + 255) / 256 : 0, db_blocks = db != nullptr ? N / 16 : 0;
  if (dw_blocks + db_blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (dw_blocks + db_blocks > 0) {
    hipLaunchKernelGGL(grad_reduce_kernel, dim3(unsigned(dw_blocks + db_blocks)), dim3(256), 0, s, part,
                       static_cast<uint16_t*>(dw), N * K, int(plan.splits), dw_blocks, sums,
                       static_cast<uint16_t*>(db), N, cols.rows);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace lmbp
