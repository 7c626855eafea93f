// Backward attention for gfx950 (Table 1, Attention column, "Backward B"; attention has no
// parameters, so there is no "Backward W").  Works from q, k, v, o, lse only -- the
// activations the paper calls "saved by flash attention" (Section 4.4) -- in these passes:
//
//   preprocess : delta_i = sum_d dO_id * O_id                         (streams 2 tensors, HBM bound)
//   delta_head : causal attention only, the first rows of every head, which the preprocess pass then leaves out: a sweep
//                in the dQ layout that only produces delta_i = sum_j p_ij dp_ij
//   dkdv       : (bwd_dkdv_pair.hip for head dimension 128, bwd_dkdv.hip for 64) a workgroup owns
//                128 keys and sweeps the query blocks that see them: S = Q K^T,
//                P = exp(scale*S - LSE), dV^T += dO^T P, dP = dO V^T, dS = P o (dP - delta),
//                dK^T += Q^T dS
//   dq         : (bwd_dq.hpp) a workgroup owns 256 or 128 queries and sweeps the visible key tiles:
//                S^T = K Q^T, dP^T = V dO^T, dS^T = P^T o (dP^T - delta), dQ^T += K^T dS^T
// dkdv and dq share a launch on all but the largest grids (gradient_tiles in dispatch.hpp).  Between the kernels the row statistics travel as neg_delta = -delta and lse2 = LSE * log2(e).
//
// Every output element is produced by exactly one lane, so there are no atomics and the
// result is bit-reproducible.
#include "helix_common.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace helix {

constexpr int kPreprocessPasses = 4;   // rows in flight per lane group

// ------------------------------------------------------------------ preprocess
// One row of D bf16 is D/8 16-byte chunks; D/8 adjacent lanes own a row.  Besides the row
// sums the kernel rewrites LSE in the form the two gradient passes consume, so that neither
// spends a vector instruction per score element on it:
//   neg_delta_i = -sum_d dO_id * O_id      (becomes the initial accumulator of the dP product)
//   lse2_i      = LSE_i * log2(e)          (P = exp2(S * scale * log2(e) - lse2))
// Workgroup ids enumerate (slice, row block) in one dimension: no limit on B * H.
template <int D>
__global__ void __launch_bounds__(256)
bwd_preprocess_kernel(const __bf16* __restrict__ o, const __bf16* __restrict__ dO, const float* __restrict__ lse,
                      float* __restrict__ neg_delta, float* __restrict__ lse2, TensorMap mo, TensorMap mdo,
                      int H, int S, int first_row, int blocks_per_head) {
  constexpr int LPR = D / 8;            // lanes per row
  constexpr int RPB = 256 / LPR;        // rows per workgroup pass
  constexpr int PASSES = kPreprocessPasses;
  const int tid = threadIdx.x;
  const int sub = tid % LPR;
  const int bh = blockIdx.x / blocks_per_head;
  const int row0 = first_row + (blockIdx.x - bh * blocks_per_head) * (RPB * PASSES) + tid / LPR;
  const __bf16* oh = o + head_offset(mo, bh, H);
  const __bf16* gh = dO + head_offset(mdo, bh, H);
  bf16x8 a[PASSES], b[PASSES];
  float l[PASSES];   // requested with the rows: behind their sums it is one more round trip (27 heads x 777 x 64 3.48 -> 3.26 us)
#pragma unroll
  for (int p = 0; p < PASSES; p++) {
    const int r = row0 + p * RPB;
    if (r < S) {
      if (sub == 0) l[p] = lse[(size_t)bh * S + r];
      a[p] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(oh + (size_t)r * mo.row + sub * 8));
      b[p] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(gh + (size_t)r * mdo.row + sub * 8));
    }
  }
#pragma unroll
  for (int p = 0; p < PASSES; p++) {
    const int r = row0 + p * RPB;
    float s = 0.f;
    if (r < S) {
#pragma unroll
      for (int e = 0; e < 8; e++) s = fmaf((float)a[p][e], (float)b[p][e], s);
    }
#pragma unroll
    for (int off = LPR / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (sub == 0 && r < S) {
      neg_delta[(size_t)bh * S + r] = -s;
      lse2[(size_t)bh * S + r] = l[p] * kLog2e;
    }
  }
}

hipError_t launch_bwd_preprocess(const void* o, const void* dO, const float* lse, float* neg_delta, float* lse2,
                                 const BwdMaps& maps, int B, int H, int S, int D, int first_row, hipStream_t stream) {
  if (first_row >= S) return hipSuccess;
  const int per = (256 / (D / 8)) * kPreprocessPasses;
  const int bph = (S - first_row + per - 1) / per;
  const unsigned grid = (unsigned)((long long)bph * B * H);
  if (D == 128)
    hipLaunchKernelGGL(bwd_preprocess_kernel<128>, dim3(grid), dim3(256), 0, stream, (const __bf16*)o, (const __bf16*)dO, lse,
                       neg_delta, lse2, maps.o, maps.dO, H, S, first_row, bph);
  else
    hipLaunchKernelGGL(bwd_preprocess_kernel<64>, dim3(grid), dim3(256), 0, stream, (const __bf16*)o, (const __bf16*)dO, lse,
                       neg_delta, lse2, maps.o, maps.dO, H, S, first_row, bph);
  return hipGetLastError();
}

// ------------------------------------------------------------------ delta of the first rows
// A sweep in the dQ layout (a lane owns a query) that evaluates delta_i = sum_j p_ij dp_ij from its definition.
// It runs on the first rows of every head, where attention is concentrated on few keys and the bf16 rounding of O
// would otherwise dominate delta.
//
// The tiles are short (at most 2048 keys for causal attention) and few, so what counts is the length of one
// workgroup's chain: it owns 128 rows, wave (rg, kg) sweeps half kg of every 64-key tile for 32 of them (as in the split
// forward), one block of 2*D/16 hand-ordered slots per tile:
//     slots 0.. 7   dP^T(j)   = V(j) dO^T   | P^T(j) = exp2(S^T(j)*c - lse2)
//     slots 8..15   S^T(j+1)  = K(j+1) Q^T  | sum += P^T(j) o dP^T(j)
// with the tile copies asynchronous and four tiles ahead.  Against an unpipelined sweep of 256-row tiles through staging
// registers: 2 heads x 32k tokens 71 -> 32 us, 5 x 32k 72 -> 33, 16 x 16k at head dimension 64 56 -> 28, 4 x 16 x 2k
// (the time of the two products at 1230 TFLOP/s is 56) 107 -> 95, and about 82 with whole tiles (below).
template <int D>
struct DeltaHead {
  static constexpr int NST = 5, AHEAD = NST - 1;
  static constexpr int TILE = 64 * D * 2, STAGE = 2 * TILE;
  static constexpr int LDS = NST * STAGE;
};

// KG = 2: 128 rows per workgroup, key halves in two groups of waves, as above.  KG = 1, for the grids that fill the chip with
// 256-row tiles (delta_rows): every wave takes both halves of a tile for 32 rows of its own, one after the other, so an operand
// copied to LDS serves twice the rows; the halves keep sums of their own, and delta has the same bits.  Whole backward of 4 x 16
// heads x 2k tokens (512 tiles of 256 rows) with KG = 2 -> 1: 350.5 -> 336.7 us; 2 x 40 x 8000 forward + backward unchanged.
template <int D, bool CAUSAL, int KG, int RG>
__global__ void __launch_bounds__(64 * KG * RG) __attribute__((amdgpu_waves_per_eu(2)))
bwd_delta_head_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                      const __bf16* __restrict__ dO, const float* __restrict__ lse, float* __restrict__ neg_delta_out,
                      float* __restrict__ lse2_out, BwdMaps maps, int BH, int H, int S, int T, float scale) {
  using G = DeltaHead<D>;
  constexpr int BM = 32 * RG, BN = 64, KS = D / 16, R = 4;   // R: operands in flight
  constexpr int TILE = G::TILE, HALF = 32 * D * 2, STAGE = G::STAGE, NST = G::NST, AHEAD = G::AHEAD;
  extern __shared__ __align__(16) char smem[];   // tile j (K, V) in stage j % NST

  const TileCoord tc = map_block<CAUSAL, D>(blockIdx.x, BH, T, true);
  if (!tc.valid) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = w & (RG - 1), kg = w / RG;
  const int half = lane >> 5, n = lane & 31;
  const int q0 = tc.tile * BM;
  const int wave_qmin = q0 + 32 * rg, my_q = wave_qmin + n;
  const __bf16* qh = q + head_offset(maps.q, tc.bh, H);
  const __bf16* gh = dO + head_offset(maps.dO, tc.bh, H);
  const __bf16* kh = k + head_offset(maps.k, tc.bh, H);
  const __bf16* vh = v + head_offset(maps.v, tc.bh, H);
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale * kLog2e)));
  const uint32_t base = lds_base(smem);

  float dsum[3 - KG][2] = {};   // this lane's share of sum_j p_ij dp_ij, by key half

  const int q_end = (q0 + BM < S ? q0 + BM : S);
  const int n_tiles = CAUSAL ? (q_end + BN - 1) / BN : (S + BN - 1) / BN;
  // Key blocks of this wave and how many of them need no mask, as in fwd_split_kernel.
  const int k_end = CAUSAL ? (wave_qmin + 32 < S ? wave_qmin + 32 : S) : S;
  const int k_all = CAUSAL ? wave_qmin + 1 : S;
  const int n_w = wave_qmin < S ? (k_end - 32 * kg + BN - 1) / BN : 0;
  const int n_full = KG == 2 ? (k_all + 32 - 32 * kg) / BN : k_all / BN;

  const TileLoader<D, BN, KG * RG> kload(lane, w, maps.k.row), vload(lane, w, maps.v.row);
  constexpr int NDMA = decltype(kload)::N + decltype(vload)::N;
  int j = 0, st = 0;   // tile and its stage (j % NST)
  auto plus = [&](int d) __attribute__((always_inline)) { return st + d >= NST ? st + d - NST : st + d; };
  auto copy_tile = [&](int jj, int stage) __attribute__((always_inline)) {
    kload.issue(kh, jj * BN, S, base + stage * STAGE);
    vload.issue(vh, jj * BN, S, base + stage * STAGE + TILE);
  };
  auto copy_ahead = [&]() __attribute__((always_inline)) {
    if (j + AHEAD < n_tiles) copy_tile(j + AHEAD, plus(AHEAD));   // replaces tile j-1
  };
  auto finish_tile = [&]() __attribute__((always_inline)) {
    // tiles up to j+2 have landed before the next iteration (which reads j+1 and j+2) starts
    if (j + AHEAD < n_tiles) wait_tile_loads_except<(AHEAD - 2) * NDMA>();
    else wait_tile_loads();
    __syncthreads();
    st = plus(1);
  };
  // The Q and dO rows pass through the last stages: two of them for 128 rows, copied by one wave of a row group each, four for 256.
  // The tiles those stages are for follow when every wave has its fragments.
  constexpr int FIRST = KG == 2 ? 3 : 1;
  const uint32_t frag = base + FIRST * STAGE + rg * 2 * HALF;
  if (KG == 1 || kg == 0) issue_fragments<D>(qh, maps.q.row, wave_qmin, S, lane, 0, frag);
  if (KG == 1 || kg == 1) issue_fragments<D>(gh, maps.dO.row, wave_qmin, S, lane, 0, frag + HALF);
#pragma unroll
  for (int jj = 0; jj < FIRST; jj++)
    if (jj < n_tiles) copy_tile(jj, jj);
  float lse2 = lse[(size_t)tc.bh * S + (my_q < S ? my_q : S - 1)] * kLog2e;
  pin(lse2);
  if (n_tiles >= FIRST) wait_tile_loads_except<FIRST * NDMA>();
  else wait_tile_loads();
  if (KG == 2) __syncthreads();
  bf16x8 qf[KS], gf[KS];
  read_fragments<D>(frag, lane, qf);
  read_fragments<D>(frag + HALF, lane, gf);
  wait_tile_loads();
  __syncthreads();
#pragma unroll
  for (int jj = FIRST; jj < AHEAD; jj++)
    if (jj < n_tiles) copy_tile(jj, jj);

  uint32_t ab[KS];   // row n, contraction step ks of the K half tile (the V tile is TILE bytes further)
#pragma unroll
  for (int ks = 0; ks < KS; ks++) ab[ks] = base + kg * HALF + lds_chunk_off<D>(n, 2 * ks + half);
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 sa, sb;
  bf16x8 ring[R];
  if (n_w > 0) {
    sa = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(ab[ks], 0), qf[ks], sa);
#pragma unroll
    for (int i = 0; i < R; i++) ring[i] = lds_b128(ab[i], TILE);
  }
  if (KG == 1) {   // tile 1 has landed
    if (n_tiles >= AHEAD) wait_tile_loads_except<(AHEAD - 2) * NDMA>();
    else wait_tile_loads();
    __syncthreads();
  }

  // Block j: on entry s_cur = S^T(j) and ring = the first V operands of tile j; on exit the same for j + 1.
  // KG = 1: the first half of tile j ahead of the second, or the second half ahead of tile j + 1.
  auto step = [&](auto second, f32x16& s_cur, f32x16& s_next) __attribute__((always_inline)) {
    constexpr int H2 = decltype(second)::value;
    constexpr bool MOVES = KG == 2 || H2 == 1, COPIES = H2 == 0;
    constexpr int CUR = H2 * HALF, NEXT = MOVES ? 0 : HALF;
    const bool whole = COPIES && j + AHEAD < n_tiles && (j + AHEAD + 1) * BN <= S;
    if (COPIES && !whole) copy_ahead();
    const __bf16* kt = kload.tile_ptr(kh, (j + AHEAD) * BN);
    const __bf16* vt = vload.tile_ptr(vh, (j + AHEAD) * BN);
    const uint32_t dst = base + plus(AHEAD) * STAGE;
    const int stage_step = (st == NST - 1) ? -(NST - 1) * STAGE : STAGE;
    f32x16 dp;
#pragma unroll
    for (int s = 0; s < 2 * KS; s++) {
      if (s < KS) dp = mfma32(ring[s % R], gf[s], s == 0 ? zero : dp);
      else s_next = mfma32(ring[s % R], qf[s - KS], s == KS ? zero : s_next);
      if (s == 1 && whole) {
        kload.issue_whole(kt, dst);
        vload.issue_whole(vt, dst + TILE);
      }
      if (MOVES && s == KS - R) {   // the last read of this tile is out
#pragma unroll
        for (int ks = 0; ks < KS; ks++) ab[ks] += stage_step;
      }
      const int u = s + R;
      if (u < KS) ring[s % R] = lds_b128(ab[u], TILE + CUR);
      else if (u < 2 * KS) ring[s % R] = lds_b128(ab[u - KS], NEXT);
      else ring[s % R] = lds_b128(ab[u - 2 * KS], TILE + NEXT);
#pragma unroll
      for (int e = 0; e < 16; e++) {
        if (e * KS / 16 == s) s_cur[e] = __builtin_amdgcn_exp2f(fmaf(s_cur[e], c, -lse2));
        if (KS + e * KS / 16 == s) dsum[H2][e & 1] = fmaf(s_cur[e], dp[e], dsum[H2][e & 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (MOVES) {
      finish_tile();
      j++;
    }
  };
  const std::integral_constant<int, 0> first_half{};
  if constexpr (KG == 2) {
    while (j + 1 < n_w - 1) {
      step(first_half, sa, sb);
      step(first_half, sb, sa);
    }
    if (j < n_w - 1) {
      step(first_half, sa, sb);
      sa = sb;
    }
  } else {
    while (j < n_w - 1) {
      step(first_half, sa, sb);
      step(std::integral_constant<int, 1>{}, sb, sa);
    }
  }
  for (; j < n_tiles; j++) {
    copy_ahead();
    if (j == n_w - 1) {
      const bool masked = j >= n_full;
#pragma unroll
      for (int h = 0; h < 3 - KG; h++) {
        if (h == 1) {
          if (CAUSAL && j * BN + 32 > wave_qmin + 31) continue;   // above the diagonal: 0 * dP would be NaN for an infinite V there
          sa = zero;
#pragma unroll
          for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(ab[ks], HALF), qf[ks], sa);
        }
        f32x16 dp = zero;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) dp = mfma32(lds_b128(ab[ks], TILE + h * HALF), gf[ks], dp);
#pragma unroll
        for (int e = 0; e < 16; e++) {
          float p = __builtin_amdgcn_exp2f(fmaf(sa[e], c, -lse2));
          if (masked) {
            const int key = j * BN + 32 * (kg + h) + 8 * (e >> 2) + 4 * half + (e & 3);
            p = (CAUSAL ? key <= my_q : key < S) ? p : 0.f;
          }
          dsum[h][e & 1] = fmaf(p, dp[e], dsum[h][e & 1]);
        }
      }
    }
    finish_tile();
  }

  const float mine = half_sum(dsum[0][0] + dsum[0][1]);
  if constexpr (KG == 1) {
    const float other = half_sum(dsum[1][0] + dsum[1][1]);
    if (half == 0 && my_q < S) {
      neg_delta_out[(size_t)tc.bh * S + my_q] = -(mine + other);
      if (lse2_out) lse2_out[(size_t)tc.bh * S + my_q] = lse2;
    }
    return;
  }
  // the two key halves of a row meet in LDS (free by now)
  float* sums = reinterpret_cast<float*>(smem);
  if (kg == 1 && half == 0) sums[32 * rg + n] = mine;
  __syncthreads();
  if (kg == 0 && half == 0 && my_q < S) {
    neg_delta_out[(size_t)tc.bh * S + my_q] = -(mine + sums[32 * rg + n]);
    if (lse2_out) lse2_out[(size_t)tc.bh * S + my_q] = lse2;
  }
}

template <int D, bool CAUSAL>
static hipError_t launch_delta_head_t(const void* q, const void* k, const void* v, const void* dO, const float* lse,
                                      float* delta_out, float* lse2_out, const BwdMaps& maps, int B, int H, int S, int rows,
                                      float scale, hipStream_t stream) {
  const int BH = B * H;
  const Rows kind = delta_rows(D, BH, rows, CAUSAL);
  const int T = tiles(rows, kind);   // query tiles 0..T-1 of every head
  const unsigned grid = (unsigned)grid_blocks(BH, T);
  const size_t lds = DeltaHead<D>::LDS;
  auto kern = kind == Rows::k64 ? bwd_delta_head_kernel<D, CAUSAL, 2, 2> : bwd_delta_head_kernel<D, CAUSAL, 1, 8>;
  if constexpr (D == 128) {   // at head dimension 64 delta_rows knows the other two only
    if (kind == Rows::k128) kern = bwd_delta_head_kernel<D, CAUSAL, 2, 4>;
  }
  static unsigned long long configured[3] = {};   // per template instantiation and kernel
  hipError_t e = allow_dynamic_lds(kern, lds, configured[(int)kind]);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kind == Rows::k64 ? 256 : 512), lds, stream, (const __bf16*)q, (const __bf16*)k, (const __bf16*)v,
                     (const __bf16*)dO, lse, delta_out, lse2_out, maps, BH, H, S, T, scale);
  return hipGetLastError();
}

hipError_t launch_bwd_delta_head(const void* q, const void* k, const void* v, const void* dO,
                                 const float* lse, float* delta, float* lse2, const BwdMaps& maps, int B, int H, int S, int D,
                                 int rows, float scale, bool causal, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (rows > S) rows = S;
  rows = (rows + 255) / 256 * 256;   // whole groups of 256 rows
  if (rows > S) rows = S;
  if (D == 128) return causal ? launch_delta_head_t<128, true>(q, k, v, dO, lse, delta, lse2, maps, B, H, S, rows, scale, stream)
                              : launch_delta_head_t<128, false>(q, k, v, dO, lse, delta, lse2, maps, B, H, S, rows, scale, stream);
  return causal ? launch_delta_head_t<64, true>(q, k, v, dO, lse, delta, lse2, maps, B, H, S, rows, scale, stream)
                : launch_delta_head_t<64, false>(q, k, v, dO, lse, delta, lse2, maps, B, H, S, rows, scale, stream);
}

}  // namespace helix
