// The QKV linear layer next to attention (Section 4.2: HelixPipe ships the layer's input and
// weights to the attention stage and runs the layer there) and its two backward products,
// as one bf16 MFMA GEMM kernel for gfx950:
//
//     C[i][j] = sum_r X(i, r) * Y(r, j),       fp32 accumulation
//
//   forward          qkv[M][N] = a[M][K]    * w[K][N]      X stored [i][r],  Y stored [r][j]
//   backward input   da[M][K]  = dqkv[M][N] * w[K][N]^T    X stored [i][r],  Y stored [r][j] after a transposing copy of w
//   backward weight  dw[K][N]  = a[M][K]^T  * dqkv[M][N]   X stored [r][i],  Y stored [r][j]
//
// A workgroup of 4 waves owns a 256 x 256, 128 x 128 or 64 x 64 tile of C (linear_tile and linear_gradient_tiles in dispatch.hpp say which: a
// large tile reads less per MFMA, a small one fills the chip when C is small); wave (wi, wj) owns a quarter of
// it as accumulator blocks of the 32x32x16 MFMA (256 accumulator registers and one wave per SIMD for the large
// tile), computed transposed (the MFMA's row index is j) so that a lane owns one row i of C and stores
// consecutive j.  The contraction runs in stages of 32 or 64: each stage's X and Y tiles are copied
// global -> LDS asynchronously AHEAD stages before their use (the scheme of the attention kernels, deeper
// because a stage is shorter).  An operand whose contraction index is contiguous in memory sits in LDS
// as [outer][STEP] and is read with ds_read_b128; one whose contraction index is the row of the
// stored matrix sits as [STEP][128] tiles and is read with the transposing LDS read.  Operand reads are issued
// one sub-step (16 contraction indices) ahead.
//
// What bounds it: at one GPU's share of a 7B layer (131072 x 4096 x 1536) the power limit, as in the attention
// kernels; with few tokens the latency of the copies and barriers.  The copies are spread behind the MFMAs, each one
// instruction with running scalar pointers; in front of the stage (as address arithmetic, an edge test and
// eight copies in a row, with no MFMA in flight) they cost 14 %: forward 1571 -> 1365 us (1050 -> 1208 TFLOP/s),
// da 1853 -> 1570, dw 1785 -> 1578.
#include "helix_common.hpp"
#include "kernels.hpp"
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace helix {
namespace {

constexpr int kWaves = 4;                     // 2 x 2 waves

// Geometry of a workgroup tile: TI x TJ elements of C, contraction in stages of STEP, NST stage buffers.
// A wave owns TI/2 x TJ/2 elements.
template <int TI_, int TJ_, int STEP_, int NST_>
struct Tile {
  static constexpr int TI = TI_, TJ = TJ_, STEP = STEP_, NST = NST_;
  static constexpr int BI = TI / 64, BJ = TJ / 64;   // 32-wide blocks per wave in i and in j
  static constexpr int XBYTES = TI * STEP * 2, YBYTES = TJ * STEP * 2;
  static constexpr int STAGE = XBYTES + YBYTES;
  static constexpr int AHEAD = NST - 1;              // a stage's copy is issued this many iterations before its use
  static constexpr int LDS = NST * STAGE;
  static constexpr int WORKGROUPS = LDS > 80 * 1024 ? 1 : 2;   // on a compute unit
};
using Tile256 = Tile<256, 256, 32, 5>;        // 160 KB of LDS: one workgroup per compute unit
using Tile128 = Tile<128, 128, 32, 5>;        // 80 KB: two
using Tile64ShortStages = Tile<64, 64, 32, 8>;
using Tile64 = Tile<64, 64, 64, 5>;           // 80 KB: two

__device__ __forceinline__ void copy_16_bytes_per_lane(uint32_t lane_byte_off, const __bf16* base, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(lane_byte_off), "s"(base), "s"(lds_dst) : "memory");
}

// Operand whose stored rows are the outer index (i or j) and whose contraction index is
// contiguous: LDS tile [OUTER][STEP].  Rows past the edge of the matrix are clamped to its last row once,
// here, because the outer index of a workgroup never changes: a stage's copy is nothing but its copy instructions.
template <int OUTER, int STEP>
struct ContiguousOperand {
  using Loader = TileLoader<STEP, OUTER, kWaves>;
  static constexpr int DMA = Loader::N;              // copy instructions per wave and stage
  uint32_t off[DMA];
  const __bf16* ptr;                                 // element (outer0, first contraction index of the next stage to copy)
  uint32_t piece0;                                   // this wave's first 1 KB piece of the LDS tile
  __device__ __forceinline__ ContiguousOperand(const __bf16* p, long long ld, int outer0, int outer_n, int r0, int lane, int wave)
      : piece0((uint32_t)wave * 1024) {
    const Loader loader(lane, wave, (int)ld);
    const int last = outer_n - 1 - outer0;
#pragma unroll
    for (int i = 0; i < DMA; i++) {
      const int row = (wave + kWaves * i) * Loader::ROWS_PER_KB + loader.lane_row;
      off[i] = loader.off[i] - (uint32_t)(row > last ? row - last : 0) * loader.row_bytes;
    }
    ptr = uniform_ptr(p + (size_t)outer0 * ld + r0);
  }
  // Copy instruction i of the next stage; `next` after the last one.
  __device__ __forceinline__ void copy(int i, uint32_t lds) const { copy_16_bytes_per_lane(off[i], ptr, lds + piece0 + i * kWaves * 1024); }
  __device__ __forceinline__ void next() { ptr += STEP; }
  // lane addresses of the operand of a 32-row block starting at tile row blk0, one per sub-step of 16
  static constexpr int NADDR = STEP / 16;
  __device__ __forceinline__ static void addresses(int lane, int blk0, uint32_t (&a)[NADDR]) {
    const int row = blk0 + (lane & 31), half = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < NADDR; ks++) a[ks] = lds_chunk_off<STEP>(row, 2 * ks + half);
  }
  __device__ __forceinline__ static bf16x8 read(const uint32_t (&a)[NADDR], int ks) { return lds_b128(a[ks], 0); }
};

// Operand whose stored rows are the contraction index: LDS holds [STEP][W] tiles side by side (W = 128, or 64
// for 64 outer indices), read with the transposing LDS read so that contraction slot e of lane half h is row 8h + e.
template <int OUTER, int STEP>
struct TransposedOperand {
  static constexpr int W = OUTER < 128 ? OUTER : 128, SUBS = OUTER / W;
  using Loader = TileLoader<W, STEP, kWaves>;
  static constexpr int DMA = SUBS * Loader::N;
  uint32_t off[Loader::N];
  const __bf16* ptr[SUBS];   // element (first contraction index of the next stage, first outer index of the sub-tile)
  uint32_t piece0;
  long long stage_elems;
  __device__ __forceinline__ TransposedOperand(const __bf16* p, long long ld, int outer0, int outer_n, int r0, int lane, int wave)
      : piece0((uint32_t)wave * 1024), stage_elems(STEP * ld) {
    const Loader loader(lane, wave, (int)ld);
#pragma unroll
    for (int i = 0; i < Loader::N; i++) off[i] = loader.off[i];
#pragma unroll
    for (int b = 0; b < SUBS; b++)   // a sub-tile past the edge falls back to the first one; its results are not stored
      ptr[b] = uniform_ptr(p + (size_t)r0 * ld + (outer0 + b * W < outer_n ? outer0 + b * W : outer0));
  }
  __device__ __forceinline__ void copy(int i, uint32_t lds) const {
    const int sub = i / Loader::N, piece = i % Loader::N;
    copy_16_bytes_per_lane(off[piece], ptr[sub], lds + sub * (W * STEP * 2) + piece0 + piece * kWaves * 1024);
  }
  __device__ __forceinline__ void next() {
#pragma unroll
    for (int b = 0; b < SUBS; b++) ptr[b] += stage_elems;
  }
  static constexpr int NADDR = 2;
  __device__ __forceinline__ static void addresses(int lane, int blk0, uint32_t (&a)[NADDR]) {
    const int i = lane & 15;
    const int c = (blk0 & (W - 1)) + ((lane >> 4) & 1) * 16 + (i & 3) * 4;
    const int r = (lane >> 5) * 8 + (i >> 2);
    const int sub = (blk0 / W) * (W * STEP * 2);
    a[0] = sub + lds_chunk_off<W>(r, c >> 3) + (c & 7) * 2;
    a[1] = sub + lds_chunk_off<W>(r + 4, c >> 3) + (c & 7) * 2;
  }
  // rows 16*ks + ...: the swizzle has period 16 in the row, so the sub-step is an immediate
  __device__ __forceinline__ static bf16x8 read(const uint32_t (&a)[NADDR], int ks) { return lds_tr_pair(a[0], a[1], ks * 16 * W * 2); }
};

// The fp32 counterparts of put_rows and store_rows in helix_common.hpp: 32 rows of W floats in this wave's own LDS, 16-byte
// chunks permuted by the row so that neither access has bank conflicts.
template <int W>
__device__ __forceinline__ int float_chunk_off(int row, int chunk) {
  return row * (W * 4) + ((chunk ^ (W == 32 ? (row >> 1) & 7 : row & 15)) << 4);
}
template <int W>
__device__ __forceinline__ void put_rows(char* tile, int lane, int block, const f32x16& acc, float) {
  pin(lane);
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const f32x4 x = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    *reinterpret_cast<f32x4*>(tile + float_chunk_off<W>(lane & 31, 8 * block + 2 * g + (lane >> 5))) = x;
  }
}
template <int W>
__device__ __forceinline__ void put_rows(char* tile, int lane, int block, const f32x16& acc, __bf16) { helix::put_rows<W>(tile, lane, block, acc); }
// One 32 x 32 block from the lanes, 16 bytes at a time.
__device__ __forceinline__ void store_block(float* row, int half, const f32x16& acc) {
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const f32x4 x = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    *reinterpret_cast<f32x4*>(row + 8 * g + 4 * half) = x;
  }
}
__device__ __forceinline__ void store_block(__bf16* row, int half, const f32x16& acc) {
  for_each_chunk(half, acc, [&](int chunk, const u32x4& x) __attribute__((always_inline)) { *reinterpret_cast<u32x4*>(row + 8 * chunk) = x; });
}
// Stores the tile; `rows` of its rows and `cols` of its columns (a multiple of 32) exist.
template <int W, typename T>
__device__ __forceinline__ void store_rows(const char* tile, int lane, T* row0, long long row_stride, int rows, int cols) {
  constexpr int PER_CHUNK = 16 / sizeof(T), CH = W / PER_CHUNK, PER = 64 / CH;   // elements of a chunk, chunks of a row, rows of a piece
  pin(lane);
  const int r0 = lane / CH, chunk = lane % CH;
  const uint32_t lane_off = (uint32_t)(r0 * (int)row_stride + chunk * PER_CHUNK) * (uint32_t)sizeof(T);   // below 2^30: the row pitch is bounded
#pragma unroll
  for (int i = 0; i < 32 / PER; i++) {
    const int r = i * PER + r0;
    const int off = sizeof(T) == 4 ? float_chunk_off<W>(r, chunk) : lds_chunk_off<W>(r, chunk);
    const u32x4 x = *reinterpret_cast<const u32x4*>(tile + off);
    char* const rows_i = const_cast<char*>(uniform_ptr(reinterpret_cast<const char*>(row0 + (size_t)(i * PER) * row_stride)));
    if (r < rows && chunk * PER_CHUNK < cols) *reinterpret_cast<u32x4*>(rows_i + lane_off) = x;
  }
}
// All but the N newest vector memory operations of this wave are done, and every wave of the workgroup has got here.
// LDS reads may stay in flight across it: the reads of a stage are consumed by MFMAs of that stage's own iteration, and
// its buffer is not copied into before the one after.
template <int N>
__device__ __forceinline__ void stage_barrier() {
  wait_tile_loads_except<N>();
  asm volatile("s_barrier" ::: "memory");
}

}  // namespace

// One product C = X Y, with its tiles and the parts its contraction is cut into.
template <typename OutT>
struct Gemm {
  const __bf16 *X, *Y;
  OutT* C;
  long long ldx, ldy, ldc, part_stride;   // a part's partial result goes to C + part * part_stride
  int I, J, R, tiles_i, tiles_j, parts, r_per_part;
  // Workgroups of a part: all tiles, rounded up so that the XCD of a workgroup is its number mod 8 in every part.
  __host__ __device__ int blocks_per_part() const { return (tiles_i * tiles_j + 7) & ~7; }
};

// The tile of workgroup `block`.
template <typename G, bool X_ROWS_ARE_R, bool Y_ROWS_ARE_R, typename OutT>
__device__ __forceinline__ void gemm_block(int block, const Gemm<OutT>& g) {
  using XOp = typename std::conditional<X_ROWS_ARE_R, TransposedOperand<G::TI, G::STEP>, ContiguousOperand<G::TI, G::STEP>>::type;
  using YOp = typename std::conditional<Y_ROWS_ARE_R, TransposedOperand<G::TJ, G::STEP>, ContiguousOperand<G::TJ, G::STEP>>::type;
  constexpr int BI = G::BI, BJ = G::BJ, NS = G::STEP / 16, AHEAD = G::AHEAD, NST = G::NST, STAGE = G::STAGE;
  extern __shared__ __align__(16) char smem[];

  // workgroup id mod 8 is the XCD: each XCD takes a contiguous run of tiles, all column tiles of a row tile
  // one after the other, so an X panel reaches one L2 only
  const int per_part = g.blocks_per_part();
  // (one part, as in every forward: no division in front of the first copies, 0.12 us of a short call's 2.6)
  const int part = g.parts == 1 ? 0 : block / per_part, n = block - part * per_part;
  const int t = (n & 7) * (per_part >> 3) + (n >> 3);
  if (t >= g.tiles_i * g.tiles_j) return;
  const int ti = t / g.tiles_j, tj = t - ti * g.tiles_j;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = w & 1, wj = w >> 1;
  const int i0 = ti * G::TI, j0 = tj * G::TJ;
  const uint32_t base = lds_base(smem);

  const int r_begin = part * g.r_per_part;
  const int nk = ((g.R - r_begin < g.r_per_part ? g.R - r_begin : g.r_per_part)) / G::STEP;
  XOp xsrc(g.X, g.ldx, i0, g.I, r_begin, lane, w);
  YOp ysrc(g.Y, g.ldy, j0, g.J, r_begin, lane, w);
  constexpr int NDMA = XOp::DMA + YOp::DMA;
  auto copy = [&](int n, uint32_t lds) __attribute__((always_inline)) {   // copy instruction n of the next stage
    if (n < XOp::DMA) xsrc.copy(n, lds);
    else ysrc.copy(n - XOp::DMA, lds + G::XBYTES);
  };
#pragma unroll
  for (int k = 0; k < AHEAD; k++)
    if (k < nk) {
#pragma unroll
      for (int n = 0; n < NDMA; n++) copy(n, base + k * STAGE);
      xsrc.next();
      ysrc.next();
    }
  // iteration k reads stages k and k+1: the first two must be complete, the others may still fly
  if (nk >= AHEAD) stage_barrier<(AHEAD - 2) * NDMA>();   // all AHEAD copies are out: the newest may fly
  else stage_barrier<0>();

  uint32_t xa[BI][XOp::NADDR], ya[BJ][YOp::NADDR];
#pragma unroll
  for (int b = 0; b < BI; b++) {
    XOp::addresses(lane, 32 * (BI * wi + b), xa[b]);
#pragma unroll
    for (int e = 0; e < XOp::NADDR; e++) xa[b][e] += base;
  }
#pragma unroll
  for (int b = 0; b < BJ; b++) {
    YOp::addresses(lane, 32 * (BJ * wj + b), ya[b]);
#pragma unroll
    for (int e = 0; e < YOp::NADDR; e++) ya[b][e] += base + G::XBYTES;
  }

  f32x16 acc[BJ][BI];
#pragma unroll
  for (int jb = 0; jb < BJ; jb++)
#pragma unroll
    for (int ib = 0; ib < BI; ib++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[jb][ib][e] = 0.f;

  // Operands are read a sub-step ahead into the other of two sets.  With a single MFMA to a sub-step (the 64 x 64 tile) that is not
  // ahead enough: there a set for every sub-step is refilled behind its MFMA, a whole stage ahead (64 tokens x 2048 x 768 forward
  // 8.8 -> 7.8 us; the larger tiles lose 5 to 10 % that way, by 14 registers more and reads in bursts).
  constexpr bool STAGE_AHEAD = BI * BJ == 1;
  constexpr int SETS = STAGE_AHEAD ? NS : 2;
  bf16x8 xo[SETS][BI], yo[SETS][BJ];
#pragma unroll
  for (int ks = 0; ks < (STAGE_AHEAD ? NS : 1); ks++) {
#pragma unroll
    for (int b = 0; b < BI; b++) xo[ks][b] = XOp::read(xa[b], ks);
#pragma unroll
    for (int b = 0; b < BJ; b++) yo[ks][b] = YOp::read(ya[b], ks);
  }

  // One stage: NS sub-steps of BI * BJ MFMAs; behind each MFMA its share of the operand reads (of the next sub-step, in the last one from
  // the next buffer; or of the same sub-step of the next stage) and of the copies of stage k + AHEAD, which replaces stage k - 1.
  int buf = 0;
  auto stage = [&](auto copying, auto reading) __attribute__((always_inline)) {
    constexpr bool COPY = decltype(copying)::value, READ = decltype(reading)::value;
    constexpr int MM = BI * BJ, SLOTS = NS * MM, READS = BI + BJ;
    const int step = (buf == NST - 1) ? -(NST - 1) * STAGE : STAGE;
    const uint32_t dst = base + (buf == 0 ? NST - 1 : buf - 1) * STAGE;
#pragma unroll
    for (int ks = 0; ks < NS; ks++) {
      if (ks == (STAGE_AHEAD ? 0 : NS - 1)) {
#pragma unroll
        for (int b = 0; b < BI; b++)
#pragma unroll
          for (int e = 0; e < XOp::NADDR; e++) xa[b][e] += step;
#pragma unroll
        for (int b = 0; b < BJ; b++)
#pragma unroll
          for (int e = 0; e < YOp::NADDR; e++) ya[b][e] += step;
      }
#pragma unroll
      for (int m = 0; m < MM; m++) {
        const int jb = m / BI, ib = m % BI, set = STAGE_AHEAD ? ks : ks & 1;
        acc[jb][ib] = mfma32(yo[set][jb], xo[set][ib], acc[jb][ib]);
        // reads go behind the first MFMAs of a sub-step, one each where there are enough of them
        const int to = STAGE_AHEAD ? ks : (ks & 1) ^ 1, next_ks = STAGE_AHEAD ? ks : (ks + 1) % NS;
#pragma unroll
        for (int q = 0; q < READS; q++) {
          if (!READ || (MM >= READS ? q : q * MM / READS) != m) continue;
          if (q < BI) xo[to][q] = XOp::read(xa[q], next_ks);
          else yo[to][q - BI] = YOp::read(ya[q - BI], next_ks);
        }
        if constexpr (COPY) {
#pragma unroll
          for (int n = 0; n < NDMA; n++)
            if (n * SLOTS / NDMA == ks * MM + m) copy(n, dst);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (COPY) {
      xsrc.next();
      ysrc.next();
    }
    buf = (buf == NST - 1) ? 0 : buf + 1;
  };
  int k = 0;
  // stages up to k+2 must have landed before the next iteration starts (it reads k+1 and k+2);
  // the copies of stages k+3 .. k+AHEAD may stay in flight
  for (; k + AHEAD < nk; k++) {
    stage(std::true_type{}, std::true_type{});
    stage_barrier<(AHEAD - 2) * NDMA>();
  }
  for (; k < (STAGE_AHEAD ? nk - 1 : nk); k++) {
    stage(std::false_type{}, std::true_type{});
    stage_barrier<0>();
  }
  // The last stage has nothing to read ahead and, as the tile leaves from the registers, nobody to wait for: its reads held up the workgroup beside this one (forward of
  // 12480 x 128 x 128 3.39 -> 3.27 us, 4256 x 512 x 256 4.91 -> 4.84).
  if constexpr (STAGE_AHEAD) stage(std::false_type{}, std::false_type{});

  // A lane owns row i of C: on the larger tiles 32 rows at a time go through LDS (free since the last barrier), this wave's part of it, and leave as whole
  // rows.  Stored from the lanes, 16 bytes of 32 or 64 rows an instruction, a 256 x 256 tile takes 4 to 5 us (fp32 7) in which the
  // compute unit has nothing else to do, of 21 us for a contraction of 768.
  if constexpr (BI * BJ == 16) {   // 256 sums stay in accumulator registers: moved to the others all at once, they push the lane's index out to memory
#pragma unroll
    for (int jb = 0; jb < BJ; jb++)
#pragma unroll
      for (int ib = 0; ib < BI; ib++) asm volatile("" : "+a"(acc[jb][ib]));
  }
  constexpr int W = 32 * BJ;
  const int i_wave = i0 + 32 * BI * wi, j_wave = j0 + W * wj;
  if constexpr (BI * BJ == 1) {   // one block to a wave: straight from the lanes is the shorter way (0.28 against 0.45 us at the end of a short call)
    const int half = lane >> 5, i = i_wave + (lane & 31);
    if (i < g.I && j_wave < g.J) store_block(g.C + (size_t)part * g.part_stride + (size_t)i * g.ldc + j_wave, half, acc[0][0]);
    return;
  }
  char* const out = smem + w * (32 * W * (int)sizeof(OutT));
#pragma unroll
  for (int ib = 0; ib < BI; ib++) {
#pragma unroll
    for (int jb = 0; jb < BJ; jb++) {
      put_rows<W>(out, lane, jb, acc[jb][ib], OutT());
      __builtin_amdgcn_sched_barrier(0);   // keeps the registers of one block in flight, not of all
    }
    store_rows<W>(out, lane, g.C + (size_t)part * g.part_stride + (size_t)(i_wave + 32 * ib) * g.ldc + j_wave, g.ldc,
                  g.I - i_wave - 32 * ib, g.J - j_wave);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <typename G, bool X_ROWS_ARE_R, bool Y_ROWS_ARE_R, typename OutT>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(G::WORKGROUPS, G::WORKGROUPS)))
gemm_kernel(Gemm<OutT> g) {
  gemm_block<G, X_ROWS_ARE_R, Y_ROWS_ARE_R, OutT>(blockIdx.x, g);
}

// Both gradients in one launch (see launch_linear_bwd): the first `weight_blocks` workgroups take the weight gradient.
template <typename GI, bool WT, typename GW>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(GI::WORKGROUPS, GI::WORKGROUPS)))
linear_bwd_kernel(Gemm<__bf16> input, Gemm<float> weight, int weight_blocks) {
  static_assert(GI::WORKGROUPS == GW::WORKGROUPS, "tiles that share a compute unit alike");
  const int block = (int)blockIdx.x;
  if (block < weight_blocks) gemm_block<GW, true, true, float>(block, weight);
  else gemm_block<GI, false, WT, __bf16>(block - weight_blocks, input);
}

// dst[e] = sum over `parts` slabs of src, `n` elements each (n a multiple of 4).
__global__ void __launch_bounds__(256) sum_parts_kernel(const float* __restrict__ src, float* __restrict__ dst, long long ld_dst,
                                                        int rows, int cols, int parts) {
  const long long quad = (long long)blockIdx.x * 256 + threadIdx.x;
  const int qpr = cols / 4;
  if (quad >= (long long)rows * qpr) return;
  const int r = (int)(quad / qpr), c = (int)(quad % qpr) * 4;
  const size_t slab = (size_t)rows * cols;
  f32x4 acc = *reinterpret_cast<const f32x4*>(src + (size_t)r * cols + c);
  for (int p = 1; p < parts; p++) acc += *reinterpret_cast<const f32x4*>(src + p * slab + (size_t)r * cols + c);
  *reinterpret_cast<f32x4*>(dst + (size_t)r * ld_dst + c) = acc;
}

template <typename G, typename OutT>
static long long set_tiles(Gemm<OutT>& g) {
  g.tiles_i = (g.I + G::TI - 1) / G::TI;
  g.tiles_j = (g.J + G::TJ - 1) / G::TJ;
  return (long long)g.blocks_per_part() * g.parts;
}
template <typename G, bool XR, bool YR, typename OutT>
static hipError_t launch_gemm_tile(Gemm<OutT> g, hipStream_t stream) {
  const unsigned grid = (unsigned)set_tiles<G>(g);
  auto kern = gemm_kernel<G, XR, YR, OutT>;
  static unsigned long long configured = 0;   // one static per template instantiation
  hipError_t e = allow_dynamic_lds(kern, G::LDS, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), G::LDS, stream, g);
  return hipGetLastError();
}
template <typename GI, bool WT, typename GW>
static hipError_t launch_gradients(Gemm<__bf16> input, Gemm<float> weight, hipStream_t stream) {
  const long long weight_blocks = set_tiles<GW>(weight), input_blocks = set_tiles<GI>(input);
  const size_t lds = GI::LDS > GW::LDS ? GI::LDS : GW::LDS;
  auto kern = linear_bwd_kernel<GI, WT, GW>;
  static unsigned long long configured = 0;   // one static per template instantiation
  hipError_t e = allow_dynamic_lds(kern, lds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(weight_blocks + input_blocks)), dim3(64 * kWaves), lds, stream, input, weight, (int)weight_blocks);
  return hipGetLastError();
}

hipError_t launch_linear_fwd(const void* a, long long lda, const void* w, long long ldw, void* out, long long ldo,
                             int M, int K, int N, hipStream_t stream) {
  const Gemm<__bf16> g = {(const __bf16*)a, (const __bf16*)w, (__bf16*)out, lda, ldw, ldo, 0, M, N, K, 0, 0, 1, K};
  switch (linear_tile(M, K, N)) {
    case TileKind::k256: return launch_gemm_tile<Tile256, false, true>(g, stream);
    case TileKind::k128: return launch_gemm_tile<Tile128, false, true>(g, stream);
    default: return launch_gemm_tile<Tile64, false, true>(g, stream);
  }
}
// out[c][r] = in[r][c] for a [rows][cols] bf16 matrix (both extents multiples of 64).
__global__ void __launch_bounds__(256) transpose_kernel(const __bf16* __restrict__ in, long long ld_in,
                                                        __bf16* __restrict__ out, long long ld_out) {
  __shared__ __bf16 tile[64][66];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const size_t r0 = (size_t)blockIdx.y * 64, c0 = (size_t)blockIdx.x * 64;
#pragma unroll
  for (int i = 0; i < 16; i++) tile[ty * 16 + i][tx] = in[(r0 + ty * 16 + i) * ld_in + c0 + tx];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; i++) out[(c0 + ty * 16 + i) * ld_out + r0 + tx] = tile[tx][ty * 16 + i];
}

// Workspace of the backward: w^T (bf16 [N][K], rounded up to 256 bytes), then the partial weight gradients.
size_t linear_bwd_wt_bytes(int K, int N) { return ((size_t)K * N * 2 + 255) & ~(size_t)255; }
size_t linear_bwd_workspace_bytes(int M, int K, int N) {
  const int parts = linear_bwd_weight_parts(M, K, N);
  return linear_bwd_wt_bytes(K, N) + (parts > 1 ? (size_t)parts * K * N * sizeof(float) : 0);
}

// Input gradient da = dout * w^T.  With w as stored ([K][N], contraction index n contiguous) both
// operands would reach LDS in 64-byte row pieces, the least efficient pattern of the copy path
// (measured 30 % slower than the forward product); on the large tile a transposed copy of the small weight matrix
// (w^T [N][K], in the workspace) turns it into the forward's operand combination.
// Weight gradient dw = a^T * dout, in parts.
//
// The two need nothing of each other, so they go in one launch where their tiles share a compute unit alike, the weight gradient's longer
// workgroups first: the last round of one is filled by the other, and a small layer pays for one start.
hipError_t launch_linear_bwd(const void* a, long long lda, const void* w, long long ldw, const void* dout, long long ldd, void* da,
                             long long ldda, float* dw, long long lddw, void* workspace, int M, int K, int N, hipStream_t stream) {
  __bf16* const wt = (__bf16*)workspace;
  float* const slabs = reinterpret_cast<float*>(static_cast<char*>(workspace) + linear_bwd_wt_bytes(K, N));
  const int parts = linear_bwd_weight_parts(M, K, N);
  const int per = parts == 1 ? M : ((M / 32 + parts - 1) / parts) * 32;    // tokens per part, a multiple of the stage length
  Gemm<__bf16> in = {(const __bf16*)dout, (const __bf16*)w, (__bf16*)da, ldd, ldw, ldda, 0, M, K, N, 0, 0, 1, N};
  const Gemm<float> grad_w = {(const __bf16*)a, (const __bf16*)dout, parts == 1 ? dw : slabs, lda, ldd, parts == 1 ? lddw : N,
                          (long long)K * N, K, N, M, 0, 0, parts, per};
  const TilePair kind = linear_gradient_tiles(M, K, N, parts);
  hipError_t e = hipSuccess;
  if (kind.input == TileKind::k256) {
    hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)(N / 64), (unsigned)(K / 64)), dim3(256), 0, stream, (const __bf16*)w, ldw, wt, (long long)K);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    in.Y = wt;
    in.ldy = K;
  }
  if (kind.input == TileKind::k256) {   // which the weight gradient then has too
    e = launch_gradients<Tile256, true, Tile256>(in, grad_w, stream);
  } else if (kind.weight == TileKind::k256) {   // tiles that do not share a compute unit alike: a launch each
    e = launch_gemm_tile<Tile256, true, true>(grad_w, stream);
    if (e != hipSuccess) return e;
    e = kind.input == TileKind::k128 ? launch_gemm_tile<Tile128, false, false>(in, stream) : launch_gemm_tile<Tile64, false, false>(in, stream);
  } else if (kind.input == TileKind::k128) {
    e = kind.weight == TileKind::k128 ? launch_gradients<Tile128, false, Tile128>(in, grad_w, stream)
                                      : launch_gradients<Tile128, false, Tile64ShortStages>(in, grad_w, stream);
  } else {
    e = kind.weight == TileKind::k128 ? launch_gradients<Tile64, false, Tile128>(in, grad_w, stream)
                                      : launch_gradients<Tile64, false, Tile64ShortStages>(in, grad_w, stream);
  }
  if (e != hipSuccess || parts == 1) return e;
  const long long quads = (long long)K * N / 4;
  hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, stream, slabs, dw, lddw, K, N, parts);
  return hipGetLastError();
}

}  // namespace helix
