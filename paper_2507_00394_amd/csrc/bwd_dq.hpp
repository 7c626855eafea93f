// dQ pass of the attention backward for gfx950 (Table 1, Attention column, "Backward B"): the work of one workgroup,
// for the kernel that is nothing else (bwd_dq.hip) and for the ones that share a launch with the dK/dV pass.
//
// Work split (dq_whole_rows; dq_split_rows, for small grids, differs as its comment says): a workgroup of 8 waves owns
// 256 query rows of one (batch, head) slice, 32 per
// wave, and sweeps the 64-key tiles the causal mask leaves visible.  Everything is kept
// transposed so that a lane owns ONE query (column l%32): its LSE and delta are plain
// per-lane scalars.  Per 32-key half tile h a wave evaluates with the 32x32x16 bf16 MFMA
//     S^T(h)  = K(h) Q^T            P^T  = exp2(S^T*c - lse2)           (c = scale*log2e)
//     dP^T(h) = V(h) dO^T - delta   dS^T = P^T o dP^T
// (lse2 = LSE*log2e and -delta come from the preprocess kernel; -delta, replicated over an
// accumulator, is the initial value of the dP^T product)
//     dQ^T   += K(h)^T bf16(dS^T)                                        (dQ scaled at the end)
// Q and dO fragments of the wave's queries stay in registers (B operands); K and V rows come
// from LDS as A operands, K a second time through the transposing LDS read.
//
// Schedule (see fwd.hip for why): software pipelined over the half tiles, one basic block of
// 3*D/16 hand-ordered slots per half step, each slot with one MFMA, the LDS read of the A
// operand needed four slots later and a share of the vector work:
//     slots  0.. 7   dP^T(h)   = V(h) dO^T      | P^T(h), second half of the exponentials
//     slots  8..15   S^T(h+1)  = K(h+1) Q^T     | dS^T(h) = P^T o dP^T, bf16 packs
//     slots 16..23   dQ^T     += K(h)^T dS^T(h) | P^T(h+1), first half of the exponentials
// K / V tiles are copied global -> LDS asynchronously into four stages (tile j and j+1
// resident, j+2 landing, j+3 being issued); one workgroup barrier per 64-key tile.  The last
// tile of every wave (the only one the causal mask cuts, or the ragged end of the sequence)
// runs through a plain, masked path.
#pragma once
#include "helix_common.hpp"
#include "kernels.hpp"

namespace helix {

namespace {

constexpr int kDqRing = 4;   // A operands in flight

// One pipelined half step.  CUR: byte offset of h inside its tile; B_HALF: the block ahead
// (h+1) starts the next tile, so the lane addresses move on by stage_step as soon as their
// last read of the current tile is out.  On entry s_cur = S^T(h) with entries 0..7 already
// exponentiated and ring = first four V(h) operands; on exit the same holds for s_next.
template <int D, bool B_HALF, int CUR, typename Copy>
__device__ __forceinline__ void dq_half_step(const Copy& copy_tile, f32x16& s_cur, f32x16& s_next, bf16x8 (&ring)[kDqRing],
                                             const bf16x8 (&qf)[D / 16], const bf16x8 (&gf)[D / 16],
                                             f32x16 (&dqacc)[D / 32], uint32_t (&ab)[D / 16], uint32_t (&at)[D / 32][2],
                                             int stage_step, float c, float lse2, const f32x16& nd) {
  constexpr int KS = D / 16, DB = D / 32, NS = 3 * KS, R = kDqRing;
  constexpr int TILE = 64 * D * 2, HALF = 32 * D * 2;
  constexpr int V_CUR = TILE + CUR;                      // V rows of h, stage layout [K tile][V tile]
  constexpr int K_NEXT = B_HALF ? 0 : HALF;              // K rows of h+1 (after the move when B_HALF)
  constexpr int K_CUR_T = CUR;                           // K rows of h for the transposing reads
  constexpr int V_NEXT = TILE + (B_HALF ? 0 : HALF);     // V rows of h+1
  constexpr int EV = 8 / KS > 0 ? 8 / KS : 1;            // exponentials per slot in the first / last group
  constexpr int ED = 16 / KS;                            // dS elements per slot in the middle group
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dp;
  uint32_t sk[8];   // bf16 pairs of dS^T(h)

#pragma unroll
  for (int s = 0; s < NS; s++) {
    // ---- matrix work
    if (s < KS) {
      dp = mfma32(ring[s % R], gf[s], s == 0 ? nd : dp);
    } else if (s < 2 * KS) {
      s_next = mfma32(ring[s % R], qf[s - KS], s == KS ? zero : s_next);
    } else {
      const int i = s - 2 * KS;
      const u32x4 b = {sk[4 * (i / DB)], sk[4 * (i / DB) + 1], sk[4 * (i / DB) + 2], sk[4 * (i / DB) + 3]};
      dqacc[i % DB] = mfma32(ring[s % R], __builtin_bit_cast(bf16x8, b), dqacc[i % DB]);
    }
    if (s == 1) copy_tile();   // tile copies are issued under the first MFMAs, not in front of them
    // ---- lane addresses move to the next tile
    if (B_HALF && s == KS - R) {
#pragma unroll
      for (int ks = 0; ks < KS; ks++) ab[ks] += stage_step;
    }
    if (B_HALF && s == NS - R) {
#pragma unroll
      for (int db = 0; db < DB; db++) { at[db][0] += stage_step; at[db][1] += stage_step; }
    }
    // ---- A operand of slot s + R
    {
      const int u = s + R;
      if (u < KS) ring[s % R] = lds_b128(ab[u], V_CUR);
      else if (u < 2 * KS) ring[s % R] = lds_b128(ab[u - KS], K_NEXT);
      else if (u < 3 * KS) {
        const int i = u - 2 * KS;
        ring[s % R] = lds_tr_pair(at[i % DB][0], at[i % DB][1], K_CUR_T + 16 * (i / DB) * D * 2);
      } else {
        ring[s % R] = lds_b128(ab[u - NS], V_NEXT);
      }
    }
    // ---- vector work
    if (s < KS) {
#pragma unroll
      for (int e = 8 + s * EV; e < 8 + (s + 1) * EV && e < 16; e++)
        s_cur[e] = __builtin_amdgcn_exp2f(fmaf(s_cur[e], c, -lse2));
    } else if (s < 2 * KS) {
#pragma unroll
      for (int e = (s - KS) * ED; e < (s - KS + 1) * ED; e += 2) {
        const float d0 = s_cur[e] * dp[e];
        const float d1 = s_cur[e + 1] * dp[e + 1];
        sk[e / 2] = pack_bf16_pair(d0, d1);
      }
    } else {
#pragma unroll
      for (int e = (s - 2 * KS) * EV; e < (s - 2 * KS + 1) * EV && e < 8; e++)
        s_next[e] = __builtin_amdgcn_exp2f(fmaf(s_next[e], c, -lse2));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

}  // namespace

template <int D>
constexpr int kDqWholeLds = 5 * 2 * 64 * D * 2;   // four stages; the Q and dO rows of a workgroup take one more

template <int D, bool CAUSAL>
__device__ __forceinline__ void dq_whole_rows(int block, const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                                              const __bf16* __restrict__ dO, const float* __restrict__ lse2_all, const float* __restrict__ neg_delta,
                                              __bf16* __restrict__ dq, BwdMaps maps, int BH, int H, int S, int T, float scale) {
  constexpr int BM = 256, BN = 64;
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int TILE = BN * D * 2, HALF = 32 * D * 2;
  constexpr int STAGE = 2 * TILE;   // [K tile][V tile]; tile j lives in stage j % 4
  extern __shared__ __align__(16) char smem[];

  const TileCoord tc = map_block<CAUSAL, D>(block, BH, T, true);
  if (!tc.valid) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, n = lane & 31;
  const int q0 = tc.tile * BM;
  const int my_q = q0 + 32 * w + n;
  const __bf16* qh = q + head_offset(maps.q, tc.bh, H);
  const __bf16* gh = dO + head_offset(maps.dO, tc.bh, H);
  const __bf16* kh = k + head_offset(maps.k, tc.bh, H);
  const __bf16* vh = v + head_offset(maps.v, tc.bh, H);
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale * kLog2e)));
  const uint32_t base = lds_base(smem);

  f32x16 dqacc[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int e = 0; e < 16; e++) dqacc[db][e] = 0.f;

  const int q_end = (q0 + BM < S ? q0 + BM : S);
  const int n_tiles = CAUSAL ? (q_end + BN - 1) / BN : (S + BN - 1) / BN;
  const int wave_qmin = q0 + 32 * w, wave_qmax = wave_qmin + 31;
  // Tiles this wave works on (n_w) and how many of them need no mask (n_full >= n_w - 1).
  int n_w, n_full;
  if (wave_qmin >= S) { n_w = 0; n_full = 0; }
  else if (CAUSAL) { n_w = (wave_qmax < S ? wave_qmax : S - 1) / BN + 1; n_full = (wave_qmin + 1) / BN; }
  else { n_w = n_tiles; n_full = S / BN; }

  const TileLoader<D, BN, 8> kload(lane, w, maps.k.row), vload(lane, w, maps.v.row);
  constexpr int NDMA = decltype(kload)::N + decltype(vload)::N;   // copy instructions per wave and tile: what copy_tile() issues
  int j = 0, st = 0;   // tile and its stage (j % 4)
  auto copy_tile = [&](int jj, int stage) __attribute__((always_inline)) {
    kload.issue(kh, jj * BN, S, base + stage * STAGE);
    vload.issue(vh, jj * BN, S, base + stage * STAGE + TILE);
  };
  auto copy_ahead = [&]() __attribute__((always_inline)) {
    if (j + 3 < n_tiles) copy_tile(j + 3, (st + 3) & 3);   // replaces tile j-1
  };
  auto finish_tile = [&]() __attribute__((always_inline)) {
    // tiles up to j+2 have landed before the next iteration (which reads j+1 and j+2) starts
    if (j + 3 < n_tiles) wait_tile_loads_except<NDMA>();
    else wait_tile_loads();
    __syncthreads();
    st = (st + 1) & 3;
  };
  // the Q and dO rows of this wave pass through the stages behind the first; tiles 1 and 2 follow when every wave has them
  const uint32_t frag = base + STAGE + w * 2 * HALF;
  issue_fragments<D>(qh, maps.q.row, wave_qmin, S, lane, 0, frag);
  issue_fragments<D>(gh, maps.dO.row, wave_qmin, S, lane, 0, frag + HALF);
  copy_tile(0, 0);
  float lse2;
  f32x16 nd;     // -delta of this lane's query in every accumulator register
  {
    const int row = my_q < S ? my_q : S - 1;
    lse2 = lse2_all[(size_t)tc.bh * S + row];
    const float dl = neg_delta[(size_t)tc.bh * S + row];
#pragma unroll
    for (int e = 0; e < 16; e++) nd[e] = dl;
    pin(lse2); pin(nd);
  }
  wait_tile_loads();
  bf16x8 qf[KS], gf[KS];
  read_fragments<D>(frag, lane, qf);
  read_fragments<D>(frag + HALF, lane, gf);
  __syncthreads();
  if (n_tiles > 1) copy_tile(1, 1);
  if (n_tiles > 2) copy_tile(2, 2);

  // Lane addresses in stage 0: ab = row n, contraction step ks (K tile; the V tile is TILE
  // bytes further); at = transposing reads of the K tile.
  uint32_t ab[KS], at[DB][2];
#pragma unroll
  for (int ks = 0; ks < KS; ks++) ab[ks] = base + lds_chunk_off<D>(n, 2 * ks + half);
#pragma unroll
  for (int db = 0; db < DB; db++) {
    int o0, o1;
    tr_pair_offsets<D>(lane, db, o0, o1);
    at[db][0] = base + o0;
    at[db][1] = base + o1;
  }

  // Prime: S^T of the first half tile (entries 0..7 exponentiated) and its first V operands.
  f32x16 sa, sb;
  bf16x8 ring[kDqRing];
  if (n_w > 0) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sa = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(ab[ks], 0), qf[ks], sa);
#pragma unroll
    for (int e = 0; e < 8; e++) sa[e] = __builtin_amdgcn_exp2f(fmaf(sa[e], c, -lse2));
#pragma unroll
    for (int i = 0; i < kDqRing; i++) ring[i] = lds_b128(ab[i], TILE);
  }
  if (n_tiles > 2) wait_tile_loads_except<NDMA>();   // tile 1 has landed
  else wait_tile_loads();
  __syncthreads();

  const auto no_copy = []() {};
  for (; j < n_w - 1; j++) {
    // A complete tile j+3 is copied by a handful of instructions issued inside the half step; a
    // ragged one (the last of the sequence) takes the general path in front of it.
    const bool whole = j + 3 < n_tiles && (j + 4) * BN <= S;
    if (!whole) copy_ahead();
    const __bf16* kt = kload.tile_ptr(kh, (j + 3) * BN);
    const __bf16* vt = vload.tile_ptr(vh, (j + 3) * BN);
    const uint32_t dst = base + ((st + 3) & 3) * STAGE;
    const auto copy_whole = [&]() __attribute__((always_inline)) {
      if (whole) {
        kload.issue_whole(kt, dst);
        vload.issue_whole(vt, dst + TILE);
      }
    };
    const int stage_step = (st == 3) ? -3 * STAGE : STAGE;
    dq_half_step<D, false, 0>(copy_whole, sa, sb, ring, qf, gf, dqacc, ab, at, stage_step, c, lse2, nd);
    dq_half_step<D, true, HALF>(no_copy, sb, sa, ring, qf, gf, dqacc, ab, at, stage_step, c, lse2, nd);
    finish_tile();
  }

  for (; j < n_tiles; j++) {
    copy_ahead();
    if (j == n_w - 1) {
      // plain path: the last tile of this wave, masked unless the sequence ends on a tile
      // edge.  sa holds S^T of its first half with entries 0..7 already exponentiated; ab and
      // at point at this tile.
      const int k0 = j * BN;
      const bool masked = j >= n_full;
#pragma unroll
      for (int kb = 0; kb < 2; kb++) {
        f32x16 sacc, pacc;
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (kb == 0) {
          sacc = sa;
#pragma unroll
          for (int e = 8; e < 16; e++) sacc[e] = __builtin_amdgcn_exp2f(fmaf(sacc[e], c, -lse2));
        } else {
          sacc = zero;
#pragma unroll
          for (int ks = 0; ks < KS; ks++) sacc = mfma32(lds_b128(ab[ks], HALF), qf[ks], sacc);
#pragma unroll
          for (int e = 0; e < 16; e++) sacc[e] = __builtin_amdgcn_exp2f(fmaf(sacc[e], c, -lse2));
        }
        pacc = nd;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) pacc = mfma32(lds_b128(ab[ks], TILE + kb * HALF), gf[ks], pacc);
#pragma unroll
        for (int e = 0; e < 16; e++) {
          float p = sacc[e];
          if (masked) {
            const int key = k0 + 32 * kb + 8 * (e >> 2) + 4 * half + (e & 3);
            p = (CAUSAL ? key <= my_q : key < S) ? p : 0.f;
          }
          pacc[e] = p * pacc[e];
        }
#pragma unroll
        for (int t = 0; t < 2; t++) {
          const bf16x8 sbk = pack_half(pacc, t);
#pragma unroll
          for (int db = 0; db < DB; db++)
            dqacc[db] = mfma32(lds_tr_pair(at[db][0], at[db][1], kb * HALF + 16 * t * D * 2), sbk, dqacc[db]);
        }
      }
    }
    finish_tile();
  }

  char* const out = smem + w * HALF;
#pragma unroll
  for (int db = 0; db < DB; db++) {
    f32x16 x;
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = dqacc[db][e] * scale;
    put_rows<D>(out, lane, db, x);
  }
  store_rows<D>(out, lane, dq + head_offset(maps.dq, tc.bh, H) + (size_t)wave_qmin * maps.dq.row, maps.dq.row, S - wave_qmin);
}

// The dQ pass for grids that 256-row tiles cannot fill (dq_rows in dispatch.hpp): 32 RG = 128 query rows per
// workgroup, or 64 on the smallest grids, wave (rg, kg) on 32 rows and half kg of every 64-key tile, the two partial sums of a row added in LDS at
// the end (see fwd_split_kernel).  12 heads x 1500 tokens 49.1 -> 31.5 us, 2 heads x 32k 904 -> 693.
template <int D>
struct DqSplit {
  static constexpr int NST = 5, AHEAD = NST - 1;
  static constexpr int TILE = 64 * D * 2, STAGE = 2 * TILE;
  static constexpr int LDS = NST * STAGE;
};

template <int D, bool CAUSAL, int RG>
__device__ __forceinline__ void dq_split_rows(int block, const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                                              const __bf16* __restrict__ dO, const float* __restrict__ lse2_all, const float* __restrict__ neg_delta,
                                              __bf16* __restrict__ dq, BwdMaps maps, int BH, int H, int S, int T, float scale) {
  using G = DqSplit<D>;
  constexpr int BM = 32 * RG, BN = 64, KS = D / 16, DB = D / 32;
  constexpr int TILE = G::TILE, HALF = 32 * D * 2, STAGE = G::STAGE, NST = G::NST, AHEAD = G::AHEAD;
  extern __shared__ __align__(16) char smem[];   // tile j (K, V) in stage j % NST

  const TileCoord tc = map_block<CAUSAL, D>(block, BH, T, true);
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

  f32x16 dqacc[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int e = 0; e < 16; e++) dqacc[db][e] = 0.f;

  const int q_end = (q0 + BM < S ? q0 + BM : S);
  const int n_tiles = CAUSAL ? (q_end + BN - 1) / BN : (S + BN - 1) / BN;
  // Key blocks of this wave and how many of them need no mask, as in fwd_split_kernel.
  const int k_end = CAUSAL ? (wave_qmin + 32 < S ? wave_qmin + 32 : S) : S;
  const int k_all = CAUSAL ? wave_qmin + 1 : S;
  const int n_w = wave_qmin < S ? (k_end - 32 * kg + BN - 1) / BN : 0;
  const int n_full = (k_all + 32 - 32 * kg) / BN;

  const TileLoader<D, BN, 2 * RG> kload(lane, w, maps.k.row), vload(lane, w, maps.v.row);
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
  // the Q and dO rows pass through the last two stages, copied by one wave of a row group each; tile 3 follows when every
  // wave has them
  const uint32_t frag = base + 3 * STAGE + rg * 2 * HALF;
  if (kg == 0) issue_fragments<D>(qh, maps.q.row, wave_qmin, S, lane, 0, frag);
  else issue_fragments<D>(gh, maps.dO.row, wave_qmin, S, lane, 0, frag + HALF);
#pragma unroll
  for (int jj = 0; jj < 3; jj++)
    if (jj < n_tiles) copy_tile(jj, jj);
  float lse2;
  f32x16 nd;     // -delta of this lane's query in every accumulator register
  {
    const int row = my_q < S ? my_q : S - 1;
    lse2 = lse2_all[(size_t)tc.bh * S + row];
    const float dl = neg_delta[(size_t)tc.bh * S + row];
#pragma unroll
    for (int e = 0; e < 16; e++) nd[e] = dl;
    pin(lse2); pin(nd);
  }
  if (n_tiles > 2) wait_tile_loads_except<3 * NDMA>();
  else wait_tile_loads();
  __syncthreads();
  bf16x8 qf[KS], gf[KS];
  read_fragments<D>(frag, lane, qf);
  read_fragments<D>(frag + HALF, lane, gf);
  wait_tile_loads();
  __syncthreads();
  if (n_tiles > 3) copy_tile(3, 3);

  const uint32_t kbase = base + kg * HALF;
  uint32_t ab[KS], at[DB][2];
#pragma unroll
  for (int ks = 0; ks < KS; ks++) ab[ks] = kbase + lds_chunk_off<D>(n, 2 * ks + half);
#pragma unroll
  for (int db = 0; db < DB; db++) {
    int o0, o1;
    tr_pair_offsets<D>(lane, db, o0, o1);
    at[db][0] = kbase + o0;
    at[db][1] = kbase + o1;
  }
  f32x16 sa, sb;
  bf16x8 ring[kDqRing];
  if (n_w > 0) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sa = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(ab[ks], 0), qf[ks], sa);
#pragma unroll
    for (int e = 0; e < 8; e++) sa[e] = __builtin_amdgcn_exp2f(fmaf(sa[e], c, -lse2));
#pragma unroll
    for (int i = 0; i < kDqRing; i++) ring[i] = lds_b128(ab[i], TILE);
  }

  auto step = [&](f32x16& s_cur, f32x16& s_next) __attribute__((always_inline)) {
    const bool whole = j + AHEAD < n_tiles && (j + AHEAD + 1) * BN <= S;
    if (!whole) copy_ahead();
    const __bf16* kt = kload.tile_ptr(kh, (j + AHEAD) * BN);
    const __bf16* vt = vload.tile_ptr(vh, (j + AHEAD) * BN);
    const uint32_t dst = base + plus(AHEAD) * STAGE;
    const auto copy_whole = [&]() __attribute__((always_inline)) {
      if (whole) {
        kload.issue_whole(kt, dst);
        vload.issue_whole(vt, dst + TILE);
      }
    };
    const int stage_step = (st == NST - 1) ? -(NST - 1) * STAGE : STAGE;
    dq_half_step<D, true, 0>(copy_whole, s_cur, s_next, ring, qf, gf, dqacc, ab, at, stage_step, c, lse2, nd);
    finish_tile();
    j++;
  };
  while (j + 1 < n_w - 1) {
    step(sa, sb);
    step(sb, sa);
  }
  if (j < n_w - 1) {
    step(sa, sb);
    sa = sb;
  }
  for (; j < n_tiles; j++) {
    copy_ahead();
    if (j == n_w - 1) {
#pragma unroll
      for (int e = 8; e < 16; e++) sa[e] = __builtin_amdgcn_exp2f(fmaf(sa[e], c, -lse2));
      f32x16 pacc = nd;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) pacc = mfma32(lds_b128(ab[ks], TILE), gf[ks], pacc);
      const bool masked = j >= n_full;
#pragma unroll
      for (int e = 0; e < 16; e++) {
        float p = sa[e];
        if (masked) {
          const int key = j * BN + 32 * kg + 8 * (e >> 2) + 4 * half + (e & 3);
          p = (CAUSAL ? key <= my_q : key < S) ? p : 0.f;
        }
        pacc[e] = p * pacc[e];
      }
#pragma unroll
      for (int t = 0; t < 2; t++) {
        const bf16x8 sbk = pack_half(pacc, t);
#pragma unroll
        for (int db = 0; db < DB; db++)
          dqacc[db] = mfma32(lds_tr_pair(at[db][0], at[db][1], 16 * t * D * 2), sbk, dqacc[db]);
      }
    }
    finish_tile();
  }

  // wave kg finishes half of the head dimension and hands the other half over
  constexpr int HB = DB / 2;
#pragma unroll
  for (int b = 0; b < HB; b++) {
    const f32x16 give = kg == 0 ? dqacc[HB + b] : dqacc[b];
    lds_put_block(smem + ((kg * RG + rg) * HB + b) * 4096, lane, give);
  }
  __syncthreads();
  char* const in = smem + ((kg ^ 1) * RG + rg) * HB * 4096;   // what the other wave handed over; the results pass through it too
#pragma unroll
  for (int b = 0; b < HB; b++) {
    f32x16 x = kg == 0 ? dqacc[b] : dqacc[HB + b];
    const f32x16 got = lds_get_block(in + b * 4096, lane);
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = (x[e] + got[e]) * scale;
    put_rows<32 * HB>(in, lane, b, x);   // inside the blocks already taken
  }
  store_rows<32 * HB>(in, lane, dq + head_offset(maps.dq, tc.bh, H) + (size_t)wave_qmin * maps.dq.row + 32 * HB * kg, maps.dq.row, S - wave_qmin);
}

}  // namespace helix
