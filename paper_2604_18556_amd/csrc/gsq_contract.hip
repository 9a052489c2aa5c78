// The dense contraction of the GSQ step: P = R H for every row of the residual R = W - W_hat,
// the gradient G = dL/dW_hat = -2 P (H symmetric) and, on request, per-tile partial sums of
// the loss tr(R H R^T) = sum(R * P) (Eq. 1 for a linear layer, H = X^T X).
//
// BF16 precision: R and H in bf16, products accumulated in fp32 on the matrix cores
// (v_mfma 16x16x32 bf16).  Because H is symmetric, column i of H is row i, so both operands
// are read along their contiguous dimension.
// FP32 precision: fp32 operands, fp64 accumulation on the fp64 matrix cores
// (v_mfma 16x16x4 f64).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gsq_device.hpp"
#include "gsq_internal.h"

namespace gsq {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = kTileM, BN = kTileN, BK = 64;
constexpr int ROW_BYTES = BK * 2;    // one 64-wide bf16 row: a full cache line
constexpr int GROUP_M = 8;           // tile rows swept together for L2 reuse
constexpr size_t LDS_BYTES = 160 * 1024;

// A workgroup's piece of a 256 x 256 tile: TM x TN outputs, and slabs loaded `AHEAD` ahead of the
// one in use.  LDS holds a ring of AHEAD + 1 slabs of R and AHEAD of H.
template <int TM_, int TN_, int AHEAD_>
struct Piece {
  static constexpr int TM = TM_, TN = TN_, AHEAD = AHEAD_;
  static constexpr int A_STAGES = AHEAD + 1, B_STAGES = AHEAD;
  static constexpr int A_SLAB = TM * ROW_BYTES, B_SLAB = TN * ROW_BYTES;
  static constexpr int B_BASE = A_STAGES * A_SLAB;
  static constexpr int A_LOADS = TM / 32, B_LOADS = TN / 32;   // 1 KB loads per wavefront and slab
  static constexpr int MI = TM / 32, NJ = TN / 32;             // 16 x 16 blocks per wavefront
  static_assert(B_BASE + B_STAGES * B_SLAB <= (int)LDS_BYTES, "the ring fits the LDS");
};
// The whole tile uses all the LDS; the smaller pieces, whose slabs last less long, load further
// ahead where there is room (the quarter's 3.5 slabs of time equal the whole tile's 1.5).
using Whole = Piece<256, 256, 2>;
using Half = Piece<256, 128, 2>;
using Quarter = Piece<128, 128, 4>;

// Sum over the workgroup into *out, through `red` (blockDim.x doubles of LDS, free to reuse).
__device__ __forceinline__ void block_sum_to(double x, double* out, double* red) {
  __syncthreads();
  red[threadIdx.x] = x;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// Position of block `bid` of nblk in the tile order.  Workgroups are handed to the 8 XCDs
// round-robin; renumbering so each XCD owns a contiguous range of the blocks keeps the R and H
// panels a group of tiles shares in the same XCD's L2.
__device__ __forceinline__ int lin_of(int bid, int nblk) {
  const int x = bid & 7, base = nblk >> 3, rem = nblk & 7;
  return x * base + min(x, rem) + (bid >> 3);
}

// Tile at position `lin`: GROUP_M tile rows are swept together, column by column.
__device__ __forceinline__ void tile_at(int lin, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int per_group = GROUP_M * tiles_n;
  const int first_m = (lin / per_group) * GROUP_M;
  const int gsz = min(tiles_m - first_m, GROUP_M);
  const int r = lin % per_group;
  tm = first_m + r % gsz;
  tn = r / gsz;
}

// Work of one launch: the tiles of every layer, of which the last round of the GPU may fill only
// some CUs.  Those tiles are cut into `parts` pieces (1, 2 or 4), one workgroup each.
//
// Without blocks, positions run over all layers' tiles; blocks 0 .. full - 1 take whole tiles and
// the rest one piece each.
//
// With blocks (batches of layers with many tiles, e.g. MoE experts): the tiles of each layer are
// grouped into blocks of bm x bn tiles (bm bn <= 32), one block per XCD at a time, so that the 32
// CUs of an XCD work on one layer's 32 tiles together and its L2 holds bm R panels and bn H
// panels for them.  Block q goes to XCD q mod 8 (workgroup w runs on XCD w mod 8); the XCD's
// workgroups take its blocks in turn, 32 per block.  `full` then counts blocks, and each block
// of the last round is spread over `parts` XCDs.
struct Plan {
  int tiles_m, tiles_n;
  int full, parts;
  int blocks;       // over all layers; 0: none
  int bm, bn;       // block shape in tiles
  int nbr, nbc;     // blocks per layer: rows, columns
  int slabs;        // K slabs that hold data
};

// The piece of this workgroup: layer b, tile (tm, tn), piece `part` of `parts`.  False: none
// (whole group).
__device__ __forceinline__ bool pick_piece(const Plan& pl, int& b, int& tm, int& tn, int& part,
                                           int& parts) {
  parts = 1;
  part = 0;
  if (pl.blocks) {
    const int x = blockIdx.x & 7, k = blockIdx.x >> 3;
    int q = (k >> 5) * 8 + x, j = k & 31;
    const int per_block = pl.bm * pl.bn;
    if (j >= per_block) return false;
    if (q >= pl.full) {
      parts = pl.parts;
      const int s = q - pl.full;
      q = pl.full + s / parts;
      j += (s % parts) * per_block;   // piece j of the block's parts bm bn
      part = j % parts;
      j /= parts;
    }
    if (q >= pl.blocks) return false;
    const int per_layer = pl.nbr * pl.nbc;
    b = q / per_layer;
    const int r = q - b * per_layer;
    tm = (r / pl.nbc) * pl.bm + j % pl.bm;
    tn = (r % pl.nbc) * pl.bn + j / pl.bm;
    return tm < pl.tiles_m && tn < pl.tiles_n;
  }
  int lin;
  if ((int)blockIdx.x < pl.full) {
    lin = lin_of(blockIdx.x, pl.full);
  } else {
    parts = pl.parts;
    const int q = lin_of(blockIdx.x - pl.full, (int)gridDim.x - pl.full);
    lin = pl.full + q / parts;
    part = q % parts;
  }
  const int tiles = pl.tiles_m * pl.tiles_n;
  b = lin / tiles;
  tile_at(lin - b * tiles, pl.tiles_m, pl.tiles_n, tm, tn);
  return true;
}

// LDS layout of a slab: row r occupies 128 bytes as eight 16-byte chunks, chunk c stored at
// position c ^ f(r), f(r) = (r / 2) & 7; two rows span the 64 banks.  A fragment read takes 16 rows,
// chunk c in one 16 lanes and c ^ 1 in the next, and the hardware serves lanes 0-3, 12-15 and 20-27
// together, then the others (measured: with f(r) = (r ^ (r / 8)) & 7, which is free of conflicts for
// 16 consecutive lanes, every read took 4 cycles more).  With this f both sets, and consecutive lanes
// too, fall on distinct banks.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Global->LDS copy of a wavefront's share of one operand slab: n instructions of eight rows, 16
// bytes per lane.  `src` is wave-uniform (the slab's first column); off[j] is the lane's element
// offset of instruction j, fixed for the whole K loop.
__device__ __forceinline__ void load_rows(const uint16_t* src, uint8_t* lds) {
  __builtin_amdgcn_global_load_lds(src, lds, 16, 0, 0);
}

// Lane offsets of those copies: row n 8 wave + 8 j + lane / 8, swizzled 16-byte chunk.
template <int n>
__device__ __forceinline__ void slab_offsets(uint32_t (&off)[n], int wave, int lane, int64_t Ipad) {
#pragma unroll
  for (int j = 0; j < n; ++j) {
    const int row = wave * (n * 8) + j * 8 + (lane >> 3);
    // < 256 Ipad + 64 <= 2^32 for the widest layer the library accepts (I <= 2^24)
    off[j] = (uint32_t)row * (uint32_t)Ipad + (uint32_t)(((lane & 7) ^ swz(row)) * 8);
  }
}

__device__ __forceinline__ bf16x8 read_frag(const uint8_t* lds, int row, int chunk) {
  return *reinterpret_cast<const bf16x8*>(lds + row * ROW_BYTES + ((chunk ^ swz(row)) << 4));
}

// Wait until at most n of this wavefront's vector-memory loads are outstanding (loads complete
// in issue order), leaving LDS and scalar counters alone.
template <int n>
__device__ __forceinline__ void wait_vm() {
  static_assert(n >= 0 && n < 64, "six bits");
  __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}

// Workgroup barrier for the slab ring: this wavefront's LDS reads are drained (its own
// global->LDS loads were waited for with wait_vm), then a plain s_barrier.  The signal fences
// keep the compiler from moving memory accesses across it; the waits are real instructions, so
// the compiler's own wait bookkeeping sees them.
__device__ __forceinline__ void slab_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt((15) | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// One block's product: G's columns are the instruction's rows, so that a lane's four results are
// four consecutive columns of a row.
//
// The instruction is written out because the builtin gives its result other registers than its
// accumulator input once there are 64 of these, and moves them around.  What the compiler then
// does not see is the time an accumulator takes to be readable by anything but another product:
// acc_settled() waits for it, before the first product and after the last.  The
// operands come from LDS reads, whose waits the compiler sets; no vector instruction writes them.
__device__ __forceinline__ void mfma_16x16x32(f32x4& acc, const bf16x8& h, const bf16x8& r) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(h), "v"(r));
}

template <int MI, int NJ>
__device__ __forceinline__ void acc_settled(f32x4 (&acc)[MI][NJ]) {
  // accumulators written before this are written before the wait, and read after it
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+a"(acc[i][j]));
  asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// One piece of G per workgroup; four wavefronts each own a quarter of it (128 x 128 of a whole
// tile) as MFMA 16x16x32 blocks.  K slabs 64 wide (whole 128-byte lines of R and H) move by direct
// global->LDS loads (16 bytes per lane, no staging registers) into the two rings.  R's extra
// buffer lets its slab k + AHEAD be loaded during the first half of slab k, H's during the second:
// the loads split evenly between the halves.  The steady-state loop has no branches, and the
// fragment reads and slab loads are spread between the matrix-core instructions instead of
// stalling them.
//
// Bound by the power that the matrix cores may draw.  With random operands in registers, the
// 16x16x32 form holds 2090 TFLOP/s on this chip and the 32x32x16 form 1824: half the accumulator
// traffic per product lets the clock stay higher.  From 32x32x16 to 16x16x32 with the order below
// and the swizzle above (one box): 4096 x 14336 1318 -> 1152 us (1.46 PFLOP/s), 8192 x 28672
// 10.0 -> 8.69 ms (1.55), 4096 x 4096 134 -> 118 us, 16 x 2048 x 7168 2.67 -> 2.33 ms.
template <class P>
__device__ __forceinline__ void contract_piece(const uint16_t* A, const uint16_t* Bt, float* Gp,
                                               const uint16_t* Rp, double* partial, int64_t Ipad,
                                               int nk, int want_loss, uint8_t* smem) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  f32x4 acc[P::MI][P::NJ];
#pragma unroll
  for (int i = 0; i < P::MI; ++i)
#pragma unroll
    for (int j = 0; j < P::NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  acc_settled(acc);

  uint32_t offa[P::A_LOADS], offb[P::B_LOADS];
  slab_offsets(offa, wave, lane, Ipad);
  slab_offsets(offb, wave, lane, Ipad);   // the same registers where the counts agree
  uint8_t* const a_wave = smem + wave * (P::TM / 4) * ROW_BYTES;
  uint8_t* const b_wave = smem + P::B_BASE + wave * (P::TN / 4) * ROW_BYTES;
  const int frow_a = wm * (P::TM / 2) + (lane & 15), frow_b = wn * (P::TN / 2) + (lane & 15);
  const int fchunk = lane >> 4;

  // load j of this wavefront's share of slab k
  const auto load_a = [&](int k, int j) {
    load_rows(A + (int64_t)k * BK + offa[j], a_wave + (k % P::A_STAGES) * P::A_SLAB + j * 8 * ROW_BYTES);
  };
  const auto load_b = [&](int k, int j) {
    load_rows(Bt + (int64_t)k * BK + offb[j], b_wave + (k % P::B_STAGES) * P::B_SLAB + j * 8 * ROW_BYTES);
  };
  // fragments of half a slab (32 of K): one read of each of R's and H's blocks in turn
  constexpr int kMfma = P::MI * P::NJ, kReads = P::MI + P::NJ;
  const auto read = [&](bf16x8 (&fa)[P::MI], bf16x8 (&fb)[P::NJ], int k, int half, int n) {
    const int i = n < 2 * P::NJ ? n / 2 : n - P::NJ;
    if (n < 2 * P::NJ && n % 2)
      fb[i] = read_frag(smem + P::B_BASE + (k % P::B_STAGES) * P::B_SLAB, frow_b + i * 16, half * 4 + fchunk);
    else
      fa[i] = read_frag(smem + (k % P::A_STAGES) * P::A_SLAB, frow_a + i * 16, half * 4 + fchunk);
  };
  static_assert(P::MI >= P::NJ, "the fragment reads walk R's blocks");
  // The products of one half, and between them, one at a time, the fragment reads of the next half
  // and the slab loads: a load after every two reads.  The products have side effects for the
  // compiler, so this order stays.  Blocks are walked back and forth: one operand of each product
  // is the last one's.  At 4096 x 14336, with a swizzle that cost each read four cycles: 1212 us so,
  // 1270 with all reads before the loads, 1229 with the loads first, 1228 spread evenly over the
  // half, 1351 one product apart instead of two; 1216 along R's blocks instead of H's.
  const auto half_slab = [&](const bf16x8 (&fa)[P::MI], const bf16x8 (&fb)[P::NJ], int n_loads,
                             auto&& next_read, auto&& next_load) {
    constexpr int kLoads = P::A_LOADS > P::B_LOADS ? P::A_LOADS : P::B_LOADS;
    constexpr int kOps = kReads + kReads / 2 > 3 * kLoads ? kReads + kReads / 2 : 3 * kLoads;
    constexpr int kStep = kMfma / kOps;
    static_assert(kStep >= 1, "every read and load has its product");
#pragma unroll
    for (int n = 0; n < kMfma; ++n) {
      const int i = n / P::NJ, j = i % 2 ? P::NJ - 1 - n % P::NJ : n % P::NJ;
      mfma_16x16x32(acc[i][j], fb[j], fa[i]);
      if (n % kStep == 0) {
        const int o = n / kStep;
        if (o % 3 == 2) { if (o / 3 < n_loads) next_load(o / 3); }
        else if (o - o / 3 < kReads) next_read(o - o / 3);
      }
    }
  };
  const auto none = [](int) {};

  // p: first half of the current slab; q: second half
  bf16x8 pa[P::MI], pb[P::NJ], qa[P::MI], qb[P::NJ];
#pragma unroll
  for (int k = 0; k < P::AHEAD; ++k) {
#pragma unroll
    for (int j = 0; j < P::A_LOADS; ++j) load_a(k, j);
#pragma unroll
    for (int j = 0; j < P::B_LOADS; ++j) load_b(k, j);
  }
  constexpr int kSlabLoads = P::A_LOADS + P::B_LOADS;
  wait_vm<(P::AHEAD - 1) * kSlabLoads>();
  slab_barrier();
#pragma unroll
  for (int n = 0; n < kReads; ++n) read(pa, pb, 0, 0, n);
  // steady state: R's slab kt + AHEAD is loaded during the first half of slab kt (its buffer last
  // held slab kt - 1), H's during the second half (its buffer held slab kt, read by then)
  for (int kt = 0; kt < nk - P::AHEAD; ++kt) {
    half_slab(pa, pb, P::A_LOADS, [&](int n) { read(qa, qb, kt, 1, n); },
              [&](int j) { load_a(kt + P::AHEAD, j); });
    __builtin_amdgcn_sched_barrier(0);   // every MFMA of this half is issued before the wait
    // slab kt + 1 has landed (later ones, of kt + AHEAD only R's, may be in flight), and every
    // wavefront has read slab kt
    wait_vm<(P::AHEAD - 2) * kSlabLoads + P::A_LOADS>();
    slab_barrier();
    half_slab(qa, qb, P::B_LOADS, [&](int n) { read(pa, pb, kt + 1, 0, n); },
              [&](int j) { load_b(kt + P::AHEAD, j); });
    __builtin_amdgcn_sched_barrier(0);
  }
  // the last slabs: nothing more to load
  for (int kt = nk - P::AHEAD; kt < nk - 1; ++kt) {
    half_slab(pa, pb, 0, [&](int n) { read(qa, qb, kt, 1, n); }, none);
    wait_vm<0>();
    slab_barrier();
    half_slab(qa, qb, 0, [&](int n) { read(pa, pb, kt + 1, 0, n); }, none);
  }
  half_slab(pa, pb, 0, [&](int n) { read(qa, qb, nk - 1, 1, n); }, none);
  half_slab(qa, qb, 0, none, none);
  acc_settled(acc);

  // G = -2 P and, on request, the piece's loss partial sum(R P).
  // 16 x 16 block: lane l holds row l % 16 and columns 4 (l / 16) .. + 3.
  double lsum = 0.0;
#pragma unroll
  for (int i = 0; i < P::MI; ++i)
#pragma unroll
    for (int j = 0; j < P::NJ; ++j) {
      const int64_t at = (int64_t)(frow_a + i * 16) * Ipad + wn * (P::TN / 2) + j * 16 + 4 * (lane >> 4);
      const f32x4 p = acc[i][j];
      *reinterpret_cast<f32x4*>(Gp + at) = -2.f * p;
      if (want_loss) {
        const uint2 r = *reinterpret_cast<const uint2*>(Rp + at);
        lsum += (double)bf16_to_f32((uint16_t)r.x) * (double)p[0];
        lsum += (double)bf16_to_f32((uint16_t)(r.x >> 16)) * (double)p[1];
        lsum += (double)bf16_to_f32((uint16_t)r.y) * (double)p[2];
        lsum += (double)bf16_to_f32((uint16_t)(r.y >> 16)) * (double)p[3];
      }
    }
  if (want_loss) block_sum_to(lsum, partial, reinterpret_cast<double*>(smem));
}

// Loss partials: four per tile, of which a whole tile writes the first and clears the others, and
// a piece writes its own (a half two, the second cleared).
constexpr int TILE_PARTIALS = 4;

__global__ __launch_bounds__(256, 1) void k_contract_bf16(const uint16_t* __restrict__ R,
                                                          const uint16_t* __restrict__ H,
                                                          float* __restrict__ G,
                                                          double* __restrict__ partials,
                                                          int64_t Opad, int64_t Ipad, int O, int I,
                                                          int want_loss, Plan pl) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  int b, tm, tn, part, parts;
  if (!pick_piece(pl, b, tm, tn, part, parts)) return;
  const int m0 = tm * BM + (parts == 4 ? (part >> 1) * Quarter::TM : 0);
  const int n0 = tn * BN + (parts == 4 ? (part & 1) : parts == 2 ? part : 0) * Half::TN;
  double* partial = partials + ((int64_t)b * pl.tiles_m * pl.tiles_n + tm * pl.tiles_n + tn) * TILE_PARTIALS + part;
  if (want_loss && threadIdx.x == 0)
    for (int k = part + parts; k < TILE_PARTIALS; k += parts) partial[k - part] = 0.0;
  if (m0 >= O || n0 >= I) {   // a piece of padding only
    if (want_loss && threadIdx.x == 0) *partial = 0.0;
    return;
  }
  const int64_t at = b * Opad * Ipad + (int64_t)m0 * Ipad;
  const uint16_t* A = R + at;
  const uint16_t* Bt = H + b * Ipad * Ipad + (int64_t)n0 * Ipad;
  float* Gp = G + at + n0;
  if (parts == 1)
    contract_piece<Whole>(A, Bt, Gp, A + n0, partial, Ipad, pl.slabs, want_loss, smem);
  else if (parts == 2)
    contract_piece<Half>(A, Bt, Gp, A + n0, partial, Ipad, pl.slabs, want_loss, smem);
  else
    contract_piece<Quarter>(A, Bt, Gp, A + n0, partial, Ipad, pl.slabs, want_loss, smem);
}

// The plan of a layer's contraction on a GPU of num_cu compute units.  Tiles beyond a whole number
// of rounds are cut where their pieces still fit one round: a piece per CU then takes about a half
// or a third of a whole tile's time, against whole tiles on half the CUs or fewer.
//   1024 x 4096 (64 tiles, as 256 quarters)              88 -> 45 us, 37 with the present MFMAs
//   14336 x 4096 (3.5 rounds, the half as 256 halves)   448 -> 410 us, 349
//   4096 x 14336 (3.5 rounds)                          1376 us, 1152, as with the K range of the
//     last tiles split over workgroups, which took a workspace and a second launch
// A quarter's K loop is bound by its loads: 32 KB per slab and CU at 64 B per clock take as long
// as its MFMAs.
//
// Blocks are taken where a layer's block about fills an XCD's 32 CUs and there is one for each XCD;
// else the tiles of all layers are numbered through.  Contraction, us, with blocks | without:
//   fewer than 24 tiles in a block: 8 x 256 x 1024 28.8 | 14.0, 16 x 512 x 1024 31.9 | 22.4,
//     32 x 1024 x 1280 130 | 119, 8 x 768 x 1792 46.0 | 45.9, 64 x 512 x 1024 72.5 | 74.5
//   fewer than 8 blocks: 3 x 2048 x 2048 56.0 | 50.2, 6 x 2048 x 1024 35.1 | 34.1
//   else: 3 x 4096 x 4096 286 | 311, 16 x 2048 x 7168 2280 | 2360, 64 x 768 x 2048 350 | 358, level at
//     4 x 2048 x 2048 and 12 x 2048 x 1008
// The line is not the best one everywhere: 64 x 1408 x 2048 817 | 661, 60 x 2048 x 1408 656 | 507,
// 8 x 1536 x 4096 378 | 308, 16 x 768 x 2048 104 | 92, 2 x 2048 x 7168 322 | 303.
Plan make_plan(const Layer& L) {
  Plan pl{};
  pl.tiles_m = (int)(L.Opad / BM);
  pl.tiles_n = (int)(L.Ipad / BN);
  pl.slabs = (int)std::max<int64_t>((L.I + BK - 1) / BK, Quarter::AHEAD);   // Ipad holds 4 or more
  pl.bm = std::min(pl.tiles_m, 8);
  pl.bn = std::min(pl.tiles_n, 32 / pl.bm);
  pl.nbr = (pl.tiles_m + pl.bm - 1) / pl.bm;
  pl.nbc = (pl.tiles_n + pl.bn - 1) / pl.bn;
  const bool blocks = L.B > 1 && pl.bm * pl.bn >= 24 && L.B * pl.nbr * pl.nbc >= 8;
  const int64_t units = blocks ? L.B * pl.nbr * pl.nbc : L.B * pl.tiles_m * pl.tiles_n;
  const int64_t round = blocks ? 8 : L.num_cu;
  const int64_t rest = units % round;
  pl.parts = rest == 0 ? 1 : rest * 4 <= round ? 4 : rest * 2 <= round ? 2 : 1;
  pl.full = (int)(pl.parts == 1 ? units : units - rest);
  pl.blocks = blocks ? (int)units : 0;
  return pl;
}

// Workgroups of a plan.
unsigned plan_grid(const Layer& L, const Plan& pl) {
  if (pl.blocks) {
    const int64_t slots = pl.full + (int64_t)(pl.blocks - pl.full) * pl.parts;
    return (unsigned)(8 * 32 * ((slots + 7) / 8));
  }
  const int64_t units = L.B * pl.tiles_m * pl.tiles_n;
  return (unsigned)(pl.full + (units - pl.full) * pl.parts);
}

// FP32 precision: products of fp32 values, exact in fp64 and summed in fp64, on the fp64 matrix
// cores (v_mfma 16x16x4 f64; their rate is the vector units', 78.6 TFLOP/s, but a fragment is
// read and converted once per 16 x 16 block instead of once per product).  A tile of 32 W x 32 W
// per workgroup, four wavefronts of 16 W x 16 W each; K slabs 32 wide go through registers into
// two LDS buffers while the other is used.  Rows of 36 floats keep the fragment reads (16 rows,
// 4 x 4 columns, 16 bytes per lane) on distinct banks.  1024 x 2048: 293 us with vector fmas (29
// TFLOP/s), 161 us here (53); 256 x 256: 24 -> 7.4 us.  The launch bound of two wavefronts per
// SIMD keeps the accumulators out of the AGPRs, whose copies cost a tenth of the loop.
//
// MFMA lane l holds row (column) l % 16 and one of four k.  A lane reads four consecutive floats
// at 4 (l / 16), one for each of four MFMAs: the same k on both sides, in another order than
// memory's.  Result: lane l, register r -> row 4 r + l / 16, column l % 16.
constexpr int SK = 32, SK_ROW = SK + 4;
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int W>
__global__ __launch_bounds__(256, 2) void k_contract_f32(const float* __restrict__ R,
                                                      const float* __restrict__ H,
                                                      float* __restrict__ G,
                                                      double* __restrict__ partials, int64_t Opad,
                                                      int64_t Ipad, int slabs, int want_loss) {
  constexpr int T = 32 * W;
  __shared__ __align__(16) float As[2][T * SK_ROW], Bs[2][T * SK_ROW];
  const int64_t b = blockIdx.z;
  const int64_t m0 = (int64_t)blockIdx.y * T, n0 = (int64_t)blockIdx.x * T;
  const float* A = R + b * Opad * Ipad + m0 * Ipad;
  const float* Bt = H + b * Ipad * Ipad + n0 * Ipad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 16 * W, wn = (wave & 1) * 16 * W;
  const int lrow = tid >> 3, lcol = (tid & 7) * 4;   // this thread's part of 32 rows of a slab

  f64x4 acc[W][W];
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};

  f32x4 ra[W], rb[W];
#define GSQ_FETCH(KT)                                                                    \
  _Pragma("unroll") for (int i = 0; i < W; ++i) {                                        \
    const int64_t at_ = (lrow + 32 * i) * Ipad + (int64_t)(KT) * SK + lcol;              \
    ra[i] = *reinterpret_cast<const f32x4*>(A + at_);                                    \
    rb[i] = *reinterpret_cast<const f32x4*>(Bt + at_);                                   \
  }
#define GSQ_STAGE(BUF)                                                                   \
  _Pragma("unroll") for (int i = 0; i < W; ++i) {                                        \
    *reinterpret_cast<f32x4*>(&As[BUF][(lrow + 32 * i) * SK_ROW + lcol]) = ra[i];        \
    *reinterpret_cast<f32x4*>(&Bs[BUF][(lrow + 32 * i) * SK_ROW + lcol]) = rb[i];        \
  }
  GSQ_FETCH(0);
  GSQ_STAGE(0);
  __syncthreads();
  for (int kt = 0; kt < slabs; ++kt) {
    const int cur = kt & 1;
    GSQ_FETCH(min(kt + 1, slabs - 1));   // the last slab again at the end: no branch
#pragma unroll
    for (int h = 0; h < SK / 16; ++h) {
      f32x4 a[W], c[W];
#pragma unroll
      for (int i = 0; i < W; ++i) {
        const int at = (lane & 15) * SK_ROW + 16 * h + 4 * (lane >> 4);
        a[i] = *reinterpret_cast<const f32x4*>(&As[cur][(wm + 16 * i) * SK_ROW + at]);
        c[i] = *reinterpret_cast<const f32x4*>(&Bs[cur][(wn + 16 * i) * SK_ROW + at]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
          for (int j = 0; j < W; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[i][k], (double)c[j][k],
                                                             acc[i][j], 0, 0, 0);
    }
    GSQ_STAGE(cur ^ 1);   // last read in the round before, whose barrier is past
    __syncthreads();
  }
#undef GSQ_FETCH
#undef GSQ_STAGE
  double lsum = 0.0;
  float* Gb = G + b * Opad * Ipad;
  const float* Rb = R + b * Opad * Ipad;
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = m0 + wm + 16 * i + 4 * r + (lane >> 4);
        const int64_t col = n0 + wn + 16 * j + (lane & 15);
        Gb[row * Ipad + col] = (float)(-2.0 * acc[i][j][r]);
        if (want_loss) lsum += (double)Rb[row * Ipad + col] * acc[i][j][r];
      }
  if (want_loss) {
    __shared__ double red[256];
    block_sum_to(lsum, partials + (b * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, red);
  }
}

// Tile of that kernel in units of 32: 64 x 64, or 32 x 32 where the larger tiles would not give
// every CU one (256 x 256: 7.4 us with 32 x 32 tiles, 14.0 with 64 x 64).
int f32_tile(const Layer& L) {
  const int64_t tiles = L.B * ((L.O + 63) / 64) * ((L.I + 63) / 64);
  return tiles >= L.num_cu ? 2 : 1;
}

// Loss of layer b = scale * the sum of its per_batch partials, in a fixed order, in one launch:
// block (c, b) sums chunk c (kChunk consecutive partials); where there are more chunks, into
// stage[b * nchunks + c], and the last block of layer b to finish (a ticket counter, reset by that
// block) sums the chunks in order.  Bound by latency: wavefront sums in registers and one exchange
// through LDS instead of a tree of eight barriers, chunks of 8192 instead of 2048, so that up to
// 8192 partials need no hand-over, and a hand-over without a fence (below, with what it rests on).
// 256 x 256: 4.1 -> 1.9 us, 1024 x 4096: 6.0 -> 5.3 (8.2 with the fence), 4096 x 4096: 7.2 -> 5.3.
constexpr int kPer = 8;                 // partials per thread, all loaded before summing
constexpr int kReduceBlock = 1024;
constexpr int kChunk = kReduceBlock * kPer;

// Sum over the workgroup, left in thread 0.
__device__ __forceinline__ double reduce_block_sum(double x) {
  __shared__ double red[kReduceBlock / 64];
  x = wave_sum_to_lane63(x);
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x < 64) {
    r = wave_sum_to_lane63(threadIdx.x < kReduceBlock / 64 ? red[threadIdx.x] : 0.0);
    r = __shfl(r, 63, 64);
  }
  __syncthreads();   // red may be used again
  return r;
}

__global__ __launch_bounds__(kReduceBlock) void k_reduce_loss(const double* partials,
                                                              int64_t per_batch, int nchunks,
                                                              double* stage, unsigned* tickets,
                                                              double scale, float* loss_out,
                                                              int* flag) {
  const int64_t b = blockIdx.y, c = blockIdx.x;
  const int64_t lo = c * kChunk, hi = min(per_batch, lo + kChunk);
  double v[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int64_t i = lo + threadIdx.x + kReduceBlock * j;
    v[j] = i < hi ? partials[b * per_batch + i] : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) s += v[j];
  double all = reduce_block_sum(s);
  if (nchunks > 1) {   // the same for the whole grid
    __shared__ unsigned ticket;
    if (threadIdx.x == 0) {
      // The chunk sum goes to where every XCD sees it, and the ticket is drawn once that has
      // answered: both are device-wide read-modify-writes, and the second needs the first's result.
      // A fence instead would write back the XCD's whole L2, full of the backward's output.
      // This rests on the hardware, not on the language's memory model, which orders relaxed
      // operations on two addresses by no dependence: gfx950 performs a device-scope
      // read-modify-write where all XCDs meet and returns its old value from there, so the sum is in
      // place before the ticket's request leaves the wavefront; and the reader's exchanges of the
      // sums leave only after the last ticket has returned (the barrier and the branch below).
      const uint64_t old = __hip_atomic_exchange(reinterpret_cast<uint64_t*>(stage) + b * nchunks + c,
                                                 (uint64_t)__double_as_longlong(all),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned one = 1u;
      asm volatile("" : "+v"(one) : "v"(old) : "memory");
      ticket = __hip_atomic_fetch_add(&tickets[b], one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (ticket != (unsigned)(nchunks - 1)) return;
    double t = 0.0;
    for (int i = threadIdx.x; i < nchunks; i += kReduceBlock)
      t += __longlong_as_double((long long)__hip_atomic_exchange(
          reinterpret_cast<uint64_t*>(stage) + b * nchunks + i, (uint64_t)0, __ATOMIC_RELAXED,
          __HIP_MEMORY_SCOPE_AGENT));   // read where it was written
    all = reduce_block_sum(t);
    if (threadIdx.x == 0) tickets[b] = 0u;
  }
  if (threadIdx.x == 0) {
    const float L = (float)(all * scale);
    loss_out[b] = L;
    if (!__builtin_isfinite(L)) *flag = 1;
  }
}

}  // namespace

hipError_t prepare_contract_kernel() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k_contract_bf16),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
}

int64_t contract_partials_per_batch(const Layer& L) {
  if (L.bf16) return (L.Opad / BM) * (L.Ipad / BN) * TILE_PARTIALS;
  const int t = 32 * f32_tile(L);
  return ((L.O + t - 1) / t) * ((L.I + t - 1) / t);
}

hipError_t launch_contract(const Layer& L, const void* R, bool want_loss, int slot, hipStream_t s) {
  float* G = L.G + (int64_t)slot * L.B * L.Opad * L.Ipad;
  double* partials = L.partials;
  if (L.bf16) {
    const Plan pl = make_plan(L);
    hipLaunchKernelGGL(k_contract_bf16, dim3(plan_grid(L, pl)), dim3(256), LDS_BYTES, s,
                       static_cast<const uint16_t*>(R), static_cast<const uint16_t*>(L.H), G,
                       partials, L.Opad, L.Ipad, (int)L.O, (int)L.I, want_loss ? 1 : 0, pl);
  } else {
    const int w = f32_tile(L), t = 32 * w, slabs = (int)((L.I + SK - 1) / SK);
    const dim3 grid((unsigned)((L.I + t - 1) / t), (unsigned)((L.O + t - 1) / t), (unsigned)L.B);
    const float* Rf = static_cast<const float*>(R);
    const float* Hf = static_cast<const float*>(L.H);
    if (w == 2)
      hipLaunchKernelGGL(k_contract_f32<2>, grid, dim3(256), 0, s, Rf, Hf, G, partials, L.Opad,
                         L.Ipad, slabs, want_loss ? 1 : 0);
    else
      hipLaunchKernelGGL(k_contract_f32<1>, grid, dim3(256), 0, s, Rf, Hf, G, partials, L.Opad,
                         L.Ipad, slabs, want_loss ? 1 : 0);
  }
  return hipGetLastError();
}

int64_t loss_stage_size(const Layer& L) {
  const int64_t most = std::max<int64_t>(L.O * L.loss_cols, contract_partials_per_batch(L));
  return L.B * ((most + kChunk - 1) / kChunk);
}

int64_t loss_row_partials(const Layer& L) { return L.B * L.O * L.loss_cols; }

int64_t loss_row_stage(const Layer& L) {
  return L.B * ((L.O * L.loss_cols + kChunk - 1) / kChunk);
}

hipError_t launch_reduce_loss(const Layer& L, float* loss_out, bool from_rows, double scale,
                              hipStream_t s) {
  return launch_reduce_loss(L, from_rows ? L.loss_part : L.partials, L.loss_stage, L.loss_tickets,
                            loss_out, from_rows, scale, s);
}

hipError_t launch_reduce_loss(const Layer& L, const double* part, double* stage, unsigned* tickets,
                              float* loss_out, bool from_rows, double scale, hipStream_t s) {
  const int64_t per_batch = from_rows ? L.O * L.loss_cols : contract_partials_per_batch(L);
  const int nchunks = (int)((per_batch + kChunk - 1) / kChunk);
  hipLaunchKernelGGL(k_reduce_loss, dim3((unsigned)nchunks, (unsigned)L.B), dim3(kReduceBlock), 0, s, part,
                     per_batch, nchunks, stage, tickets, scale, loss_out, L.flag);
  return hipGetLastError();
}

}  // namespace gsq
