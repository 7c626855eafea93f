// Forward attention for gfx950: O = softmax(scale * Q K^T + causal mask) V and the
// log-sum-exp of every score row (Table 1, Attention column, "Forward").
//
// Work split (fwd_kernel; fwd_split_kernel, which serves small grids and head dimension 64, and fwd_quad_kernel, for
// smaller grids still, differ as their comments say): one workgroup of 8 waves owns 256 consecutive query rows of one (batch, head)
// slice, 32 rows per wave, and sweeps the key tiles (64 keys) that the causal mask leaves
// visible.  Each wave computes the TRANSPOSED score block S^T = K Q^T with the 32x32x16 bf16
// MFMA, so that a lane owns ONE query (column l%32) and 16 keys per 32-key block: the
// running maximum and sum of a row live in a single register per lane and need one
// exchange between the two wave halves, not a 32-lane reduction.  bf16(P^T) in its
// accumulator layout is directly the B operand of O^T += V^T P^T; V^T comes from the
// row-major V tile in LDS through the transposing LDS read.
//
// Schedule.  On this chip a second MFMA queued behind a running one stalls the vector-ALU
// port of the whole SIMD, so matrix and vector work only overlap when they alternate inside
// one instruction stream.  The sweep is therefore software pipelined over 32-key half tiles
// h = 0, 1, 2, ... and every half step is ONE basic block of 16 hand-ordered slots (D = 128):
//     slots 0..7   MFMA S(h+1) += K(h+1) Q^T   | VALU two elements of P(h) = exp2(S(h)*c - m*c),
//                                              | their row sum, bf16 packs | LDS: V operand i
//     slots 8..15  MFMA O^T += V(h)^T P(h)^T   | VALU row maximum of S(h+1) | LDS: K operand i of S(h+2)
// followed by the (rare) rescale of the accumulators when a row maximum outgrew its
// reference.  K and V tiles are copied global -> LDS asynchronously three tiles ahead into four
// buffers each (a step already reads the first operands of the tile after its own, so two
// tiles are in use, one is landing and one is being issued); one workgroup barrier per
// 64-key tile.  The last tile of every wave (the only
// one the causal mask cuts, or the ragged end of the sequence) runs unpipelined.
#include "helix_common.hpp"
#include "kernels.hpp"

#include <cfloat>

namespace helix {

// The running reference maximum may lag the true row maximum by up to 2^kSlack before the
// accumulators are rescaled (exact in real arithmetic; keeps the rescale off the hot path).
constexpr float kSlack = 8.f;

template <int D>
struct FwdLaneAddr {
  int k[D / 16];       // K operand, contraction step ks, key row n of a tile (+32 rows by immediate)
  int v[D / 32][2];    // V^T operand of head-dim block db: first / second group of 4 key rows
  __device__ __forceinline__ FwdLaneAddr(int lane) {
    const int half = lane >> 5, n = lane & 31;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) k[ks] = lds_chunk_off<D>(n, 2 * ks + half);
#pragma unroll
    for (int db = 0; db < D / 32; db++) tr_pair_offsets<D>(lane, db, v[db][0], v[db][1]);
  }
};

__device__ __forceinline__ float max16(const f32x16& s) {
  float a = fmaxf(fmaxf(s[0], s[1]), s[2]);
  float b = fmaxf(fmaxf(s[3], s[4]), s[5]);
  a = fmaxf(fmaxf(a, s[6]), s[7]);
  b = fmaxf(fmaxf(b, s[8]), s[9]);
  a = fmaxf(fmaxf(a, s[10]), s[11]);
  b = fmaxf(fmaxf(b, s[12]), s[13]);
  a = fmaxf(fmaxf(a, s[14]), s[15]);
  return fmaxf(a, b);
}

// Softmax state of a wave: reference maximum times c (the reference may lag the true row
// maximum by up to kSlack), the raw-score threshold that triggers a reference update, and
// two partial row sums per lane.
struct SoftmaxState {
  float mref_c = -INFINITY;
  float thr = -INFINITY;          // (mref_c + kSlack) / c
  float lsum[2] = {0.f, 0.f};
};

// Cheap per-block check: did any lane see a raw score above the threshold?  (Each lane holds
// 16 of the 32 keys of its query; the two halves share mref_c, so the union over all lanes
// is the test on the full rows.)  If so, move the reference of every row that grew and
// rescale the wave's accumulators.
template <int DB>
__device__ __forceinline__ void check_reference(float local_max, float c, SoftmaxState& st, f32x16 (&oacc)[DB]) {
  if (__any(local_max > st.thr)) {
    const float tc = half_max(local_max) * c;
    const float m_new = fmaxf(st.mref_c, tc);
    const float alpha = __builtin_amdgcn_exp2f(st.mref_c - m_new);   // 0 on the first block, 1 where nothing changed
    st.lsum[0] *= alpha;
    st.lsum[1] *= alpha;
#pragma unroll
    for (int db = 0; db < DB; db++)
#pragma unroll
      for (int e = 0; e < 16; e++) oacc[db][e] *= alpha;
    st.mref_c = m_new;
    st.thr = (m_new + kSlack) / c;
  }
}

// P = bf16(exp2(S*c - mref_c)) in two 16-key packs.  The row sum takes the unrounded fp32
// values: summing the bf16-rounded ones would put up to 2^-9 relative error into LSE on rows
// that see only a few keys.
__device__ __forceinline__ void exp_pack(const f32x16& s, float c, SoftmaxState& st, bf16x8 (&p)[2]) {
  f32x16 e;
#pragma unroll
  for (int i = 0; i < 16; i++) {
    e[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c, -st.mref_c));
    st.lsum[i & 1] += e[i];
  }
  p[0] = pack_half(e, 0);
  p[1] = pack_half(e, 1);
}

// O^T += V^T P^T over the 32 key rows at byte offset row_off of the V region (plain path).
template <int D>
__device__ __forceinline__ void pv_block(const uint32_t (&vaddr)[D / 32][2], int row_off,
                                         const bf16x8 (&p)[2], f32x16 (&oacc)[D / 32]) {
#pragma unroll
  for (int t = 0; t < 2; t++)
#pragma unroll
    for (int db = 0; db < D / 32; db++)
      oacc[db] = mfma32(lds_tr_pair(vaddr[db][0] + row_off, vaddr[db][1] + row_off, 16 * t * D * 2), p[t], oacc[db]);
}

// The vector work of a step on 32 keys, shared out over its 2 KS slots of one MFMA each.  P of the current block: elements
// 0..9 in the score slots, 10..15 in the first half of the P V slots (the second half of the P V MFMAs consume them).
constexpr int kExpInScoreSlots = 10;
template <int KS>
struct StepWeights {
  float ev[16];     // exp2 values, each alive until its pair is packed
  uint32_t pw[8];   // bf16 pairs of P
  __device__ __forceinline__ void element(int x, const f32x16& s, float c, SoftmaxState& st) {
    ev[x] = __builtin_amdgcn_exp2f(fmaf(s[x], c, -st.mref_c));
    st.lsum[x & 1] += ev[x];
    if (x & 1) pw[x / 2] = pack_bf16_pair(ev[x - 1], ev[x]);
  }
  __device__ __forceinline__ void in_score_slot(int i, const f32x16& s, float c, SoftmaxState& st) {
#pragma unroll
    for (int x = 0; x < kExpInScoreSlots; x++)
      if (x * KS / kExpInScoreSlots == i) element(x, s, c, st);
  }
  __device__ __forceinline__ void in_output_slot(int i, const f32x16& s, float c, SoftmaxState& st) {
#pragma unroll
    for (int x = kExpInScoreSlots; x < 16; x++)
      if ((x - kExpInScoreSlots) * (KS / 2) / (16 - kExpInScoreSlots) == i) element(x, s, c, st);
  }
  __device__ __forceinline__ bf16x8 packed(int half) const {
    const u32x4 pk = {pw[4 * half], pw[4 * half + 1], pw[4 * half + 2], pw[4 * half + 3]};
    return __builtin_bit_cast(bf16x8, pk);
  }
};

// This lane's maximum of the next block's 16 scores, in the last P V slots (the score MFMAs have drained by then).
template <int KS>
struct StepMaximum {
  float m0 = 0.f, m1 = 0.f, m2 = 0.f, m3 = 0.f, m4 = 0.f;
  __device__ __forceinline__ void in_output_slot(int i, const f32x16& s) {
    if (i == KS - 4) { m0 = fmaxf(fmaxf(s[0], s[1]), s[2]); m1 = fmaxf(fmaxf(s[3], s[4]), s[5]); pin(m0); pin(m1); }
    if (i == KS - 3) { m2 = fmaxf(fmaxf(s[6], s[7]), s[8]); m3 = fmaxf(fmaxf(s[9], s[10]), s[11]); pin(m2); pin(m3); }
    if (i == KS - 2) { m4 = fmaxf(fmaxf(s[12], s[13]), s[14]); m0 = fmaxf(fmaxf(m0, m1), s[15]); pin(m4); pin(m0); }
    if (i == KS - 1) { m2 = fmaxf(fmaxf(m2, m3), m4); m0 = fmaxf(m0, m2); pin(m0); }
  }
};

// One pipelined half step (see the header comment).  On entry s_cur is complete, kop holds
// the first KS/2 K operands of the block to be scored now and vop the first KS/2 V operands
// of this step; on exit s_next is complete, this lane's maximum over its 16 entries of
// s_next is returned, and kop / vop hold the first operands of the next step.  Every slot
// issues one MFMA and the LDS read of the operand needed KS/2 slots later:
//   score slots 0..KS/2-1   read K operand i + KS/2 of this block   (khi + K_CUR)
//   P V slots 0..KS/2-1     read V operand i + KS/2 of this step    (vaddr + V_IMM + 16 rows)
//   P V slots KS/2..KS-1    read K operand i - KS/2 of the next block (klo + K_NEXT) and
//                           V operand i - KS/2 of the next step
// The vector-ALU work is spread evenly: P(h) (fma, exp2, row sum, bf16 pack) by StepWeights, the
// row maximum of S(h+1) by StepMaximum.
// When LAST_OF_TILE the next step works on the next V tile: vaddr moves on by v_step once this
// tile's reads are issued.
template <int D, int K_CUR, int K_NEXT, int V_IMM, bool LAST_OF_TILE, typename Copy>
__device__ __forceinline__ float half_step(const Copy& copy_tile, const f32x16& s_cur, f32x16& s_next,
                                           bf16x8 (&kop)[D / 32], bf16x8 (&vop)[D / 32], const bf16x8 (&qf)[D / 16],
                                           const uint32_t (&klo)[D / 32], const uint32_t (&khi)[D / 32],
                                           uint32_t (&vaddr)[D / 32][2], int v_step,
                                           f32x16 (&oacc)[D / 32], float c, SoftmaxState& st) {
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int RING = KS / 2;                              // operands in flight (== DB)
  constexpr int HALF = 32 * D * 2;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  StepWeights<KS> w;
#pragma unroll
  for (int i = 0; i < KS; i++) {
    s_next = mfma32(kop[i % RING], qf[i], i == 0 ? zero : s_next);
    if (i < RING) kop[i] = lds_b128(khi[i], K_CUR);
    if (i == 1) copy_tile();   // tile copies are issued under the first MFMAs, not in front of them
    w.in_score_slot(i, s_cur, c, st);
    __builtin_amdgcn_sched_barrier(0);
  }
  StepMaximum<KS> m;
#pragma unroll
  for (int i = 0; i < KS; i++) {
    oacc[i % DB] = mfma32(vop[i % RING], w.packed(i / DB), oacc[i % DB]);
    if (i < RING) {
      vop[i] = lds_tr_pair(vaddr[i][0], vaddr[i][1], V_IMM + 16 * D * 2);
      w.in_output_slot(i, s_cur, c, st);
    } else {
      if (LAST_OF_TILE) { vaddr[i - RING][0] += v_step; vaddr[i - RING][1] += v_step; }
      vop[i - RING] = lds_tr_pair(vaddr[i - RING][0], vaddr[i - RING][1], LAST_OF_TILE ? 0 : V_IMM + HALF);
      kop[i - RING] = lds_b128(klo[i - RING], K_NEXT);
    }
    m.in_output_slot(i, s_next);
    __builtin_amdgcn_sched_barrier(0);
  }
  return m.m0;
}

template <int D, bool CAUSAL>
__global__ void __launch_bounds__(512, 1)
fwd_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
           __bf16* __restrict__ o, float* __restrict__ lse, FwdMaps maps, int BH, int H, int S, int T, float scale) {
  constexpr int BM = 256, BN = 64;
  constexpr int KS = D / 16;   // contraction steps of Q K^T
  constexpr int DB = D / 32;   // 32-wide blocks of the head dimension
  constexpr int TILE = BN * D * 2;
  constexpr int HALF = 32 * D * 2;   // bytes of 32 key rows
  constexpr int VREGION = 4 * TILE;
  extern __shared__ __align__(16) char smem[];   // K[4] then V[4]; tile j in buffer j % 4

  const TileCoord tc = map_block<CAUSAL, D>(blockIdx.x, BH, T, true);
  if (!tc.valid) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index, held in a scalar register
  const int half = lane >> 5, n = lane & 31;
  const int q0 = tc.tile * BM;
  const int my_q = q0 + 32 * w + n;
  const __bf16* qh = q + head_offset(maps.q, tc.bh, H);
  const __bf16* kh = k + head_offset(maps.k, tc.bh, H);
  const __bf16* vh = v + head_offset(maps.v, tc.bh, H);
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale * kLog2e)));
  const uint32_t base = lds_base(smem);

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int e = 0; e < 16; e++) oacc[db][e] = 0.f;
  SoftmaxState st;

  const int q_end = (q0 + BM < S ? q0 + BM : S);                 // one past the last real row
  const int n_tiles = CAUSAL ? (q_end + BN - 1) / BN : (S + BN - 1) / BN;
  const int wave_qmin = q0 + 32 * w, wave_qmax = wave_qmin + 31;
  // Tiles this wave works on (n_w) and how many of them need no mask (n_full).  All but the
  // last run through the pipelined path; n_full >= n_w - 1 always holds.
  int n_w, n_full;
  if (wave_qmin >= S) { n_w = 0; n_full = 0; }
  else if (CAUSAL) { n_w = (wave_qmax < S ? wave_qmax : S - 1) / BN + 1; n_full = (wave_qmin + 1) / BN; }
  else { n_w = n_tiles; n_full = S / BN; }

  const TileLoader<D, BN, 8> kload(lane, w, maps.k.row), vload(lane, w, maps.v.row);
  constexpr int NDMA = decltype(kload)::N + decltype(vload)::N;   // copy instructions per wave and tile: what copy_ahead() issues
  // the Q rows of this wave pass through the last two K or V buffers; tile 2 follows when every wave has them
  const uint32_t frag = base + (w < 4 ? 0 : VREGION) + 2 * TILE + (w & 3) * HALF;
  issue_fragments<D>(qh, maps.q.row, wave_qmin, S, lane, 0, frag);
  kload.issue(kh, 0, S, base);
  vload.issue(vh, 0, S, base + VREGION);
  if (n_tiles > 1) { kload.issue(kh, BN, S, base + TILE); vload.issue(vh, BN, S, base + VREGION + TILE); }
  if (n_tiles > 1) wait_tile_loads_except<2 * NDMA>();
  else wait_tile_loads();
  bf16x8 qf[KS];
  read_fragments<D>(frag, lane, qf);
  wait_tile_loads();
  __syncthreads();
  if (n_tiles > 2) { kload.issue(kh, 2 * BN, S, base + 2 * TILE); vload.issue(vh, 2 * BN, S, base + VREGION + 2 * TILE); }

  const FwdLaneAddr<D> la(lane);
  // Lane addresses: klo = contraction steps 0..KS/2-1 of the K tile the NEXT block comes from,
  // khi = steps KS/2..KS-1 of the tile the CURRENT block comes from, vaddr = current V tile.
  uint32_t klo[DB], khi[DB], vaddr[DB][2];
#pragma unroll
  for (int i = 0; i < DB; i++) { klo[i] = base + la.k[i] + TILE; khi[i] = base + la.k[i + DB]; }
#pragma unroll
  for (int db = 0; db < DB; db++) { vaddr[db][0] = base + VREGION + la.v[db][0]; vaddr[db][1] = base + VREGION + la.v[db][1]; }

  f32x16 sa, sb;                 // S^T of the two 32-key halves of a tile
  bf16x8 kop[DB];                // first K operands of the next block to be scored
  bf16x8 vop[DB];                // first V operands of the next P V block
#pragma unroll
  for (int db = 0; db < DB; db++) vop[db] = lds_tr_pair(vaddr[db][0], vaddr[db][1], 0);
  if (n_w > 0) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sa = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(base + la.k[ks]), qf[ks], sa);
#pragma unroll
    for (int i = 0; i < DB; i++) kop[i] = lds_b128(base + la.k[i], HALF);
    if (n_w > 1) check_reference<DB>(max16(sa), c, st, oacc);   // tile 0 goes through the pipelined path
  }

  // The tile sweep is split per wave into the pipelined tiles 0 .. n_w-2 and a second loop
  // with the wave's last tile (plain path) and the tiles it only helps to copy.  Every wave
  // of the workgroup runs n_tiles iterations in total and meets the others at the barriers.
  int rk = 0;   // j % 4
  int j = 0;
  auto copy_ahead = [&]() __attribute__((always_inline)) {
    // copies run three tiles ahead: K(j+3), V(j+3) replace K(j-1), V(j-1), last read in
    // iteration j-1.  Iteration j itself reads tile j and, ahead of its use, the first
    // operands of tile j+1 (K in both halves, V at the end of the second), so tiles up to j+1
    // must be complete when it starts.
    if (j + 3 < n_tiles) {
      kload.issue(kh, (j + 3) * BN, S, base + ((rk + 3) & 3) * TILE);
      vload.issue(vh, (j + 3) * BN, S, base + VREGION + ((rk + 3) & 3) * TILE);
    }
  };
  auto finish_tile = [&]() __attribute__((always_inline)) {
    // K(j+2) and V(j+2), issued one iteration ago, must have landed; this iteration's copies
    // (2 + 2 instructions per wave) may stay in flight.
    if (j + 3 < n_tiles) wait_tile_loads_except<NDMA>();
    else wait_tile_loads();
    __syncthreads();
    rk = (rk + 1) & 3;
  };

  const auto no_copy = []() {};
  for (; j < n_w - 1; j++) {
    const int khi_step = (rk == 3) ? -3 * TILE : TILE;   // K buffer of tile j   -> j+1
    const int klo_step = (rk == 2) ? -3 * TILE : TILE;   // K buffer of tile j+1 -> j+2
    const int v_step = khi_step;                         // V buffer of tile j   -> j+1
    // half a: score S_b(j) | P_a(j) | O += V_a(j) P_a(j) | read K_b(j) 4..7, K_a(j+1) 0..3
    // A complete tile j+3 is copied by a handful of instructions issued inside the half step; a
    // ragged one (the last of the sequence) takes the general path in front of it.
    const bool whole = j + 3 < n_tiles && (j + 4) * BN <= S;
    if (!whole) copy_ahead();
    const __bf16* kt = kload.tile_ptr(kh, (j + 3) * BN);
    const __bf16* vt = vload.tile_ptr(vh, (j + 3) * BN);
    const uint32_t dst = base + ((rk + 3) & 3) * TILE;
    const auto copy_whole = [&]() __attribute__((always_inline)) {
      if (whole) {
        kload.issue_whole(kt, dst);
        vload.issue_whole(vt, dst + VREGION);
      }
    };
    const float mb = half_step<D, HALF, 0, 0, false>(copy_whole, sa, sb, kop, vop, qf, klo, khi, vaddr, v_step, oacc, c, st);
    check_reference<DB>(mb, c, st, oacc);
#pragma unroll
    for (int i = 0; i < DB; i++) khi[i] += khi_step;
    // half b: score S_a(j+1) | P_b(j) | O += V_b(j) P_b(j) | read K_a(j+1) 4..7, K_b(j+1) 0..3;
    // vaddr moves to V(j+1)
    const float ma = half_step<D, 0, HALF, HALF, true>(no_copy, sb, sa, kop, vop, qf, klo, khi, vaddr, v_step, oacc, c, st);
    if (j + 1 < n_w - 1) check_reference<DB>(ma, c, st, oacc);   // the plain path masks first
#pragma unroll
    for (int i = 0; i < DB; i++) klo[i] += klo_step;
    finish_tile();
  }

  for (; j < n_tiles; j++) {
    copy_ahead();
    if (j == n_w - 1) {
      // plain path: the last tile of this wave (masked unless the sequence ends on a tile edge);
      // kop holds steps 0..KS/2-1 of K_b(j), khi points at K(j), vaddr at V(j)
      const int k0 = j * BN;
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      sb = zero;
#pragma unroll
      for (int i = 0; i < DB; i++) sb = mfma32(kop[i], qf[i], sb);
#pragma unroll
      for (int i = 0; i < DB; i++) sb = mfma32(lds_b128(khi[i], HALF), qf[i + DB], sb);
      if (j >= n_full) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int key = k0 + 8 * (e >> 2) + 4 * half + (e & 3);
          sa[e] = (CAUSAL ? (key <= my_q) : (key < S)) ? sa[e] : -INFINITY;
          sb[e] = (CAUSAL ? (key + 32 <= my_q) : (key + 32 < S)) ? sb[e] : -INFINITY;
        }
      }
      bf16x8 p[2];
      check_reference<DB>(max16(sa), c, st, oacc);
      exp_pack(sa, c, st, p);
      pv_block<D>(vaddr, 0, p, oacc);
      check_reference<DB>(max16(sb), c, st, oacc);
      exp_pack(sb, c, st, p);
      pv_block<D>(vaddr, HALF, p, oacc);
    }
    finish_tile();
  }

  // epilogue: normalise, store O (bf16) and LSE (natural log, scale included)
  const float ltot = half_sum(st.lsum[0] + st.lsum[1]);
  const float inv = 1.f / ltot;
  char* const out = smem + w * HALF;
#pragma unroll
  for (int db = 0; db < DB; db++) {
    f32x16 x;
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = oacc[db][e] * inv;
    put_rows<D>(out, lane, db, x);
  }
  if (half == 0 && my_q < S) lse[(size_t)tc.bh * S + my_q] = st.mref_c * kLn2 + __logf(ltot);
  store_rows<D>(out, lane, o + head_offset(maps.o, tc.bh, H) + (size_t)wave_qmin * maps.o.row, maps.o.row, S - wave_qmin);
}

// The forward for grids that 256-row tiles cannot fill (forward_rows in dispatch.hpp says which): a workgroup owns
// 128 query rows and its two groups of four waves share the keys.  Wave (rg, kg) works on 32 query rows and on
// half kg of every 64-key tile, through the same half steps as above, one per tile; at the end the two partial
// results of a row are merged in LDS.  Twice the workgroups, each of half the length, at two waves per SIMD;
// the price is that a tile's copy serves half the rows.  The step for tile j already reads K of tile j + 2, so
// five buffers (two in use beside the current one, one landing, one being issued) take the place of four.
// 12 heads x 1500 tokens 39.7 -> 25.9 us, 2 heads x 32k 710 -> 531.
template <int D, int RG>
struct FwdSplit {
  static constexpr int NST = 5, AHEAD = NST - 1;
  static constexpr int TILE = 64 * D * 2;
  static constexpr int LDS = 2 * NST * TILE;
  static constexpr int ROW_STATS = RG * (D / 32) * 4096;   // merge: after the accumulator blocks, (reference, sum) of every row and half
  static_assert(ROW_STATS + 2 * RG * 64 * 8 <= LDS, "the merge reuses the tile buffers");
};

template <int D, bool CAUSAL, int RG>
__global__ void __launch_bounds__(128 * RG) __attribute__((amdgpu_waves_per_eu(2)))
fwd_split_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                 __bf16* __restrict__ o, float* __restrict__ lse, FwdMaps maps, int BH, int H, int S, int T, float scale) {
  using G = FwdSplit<D, RG>;
  constexpr int BM = 32 * RG, BN = 64, KS = D / 16, DB = D / 32;
  constexpr int TILE = G::TILE, HALF = 32 * D * 2, NST = G::NST, AHEAD = G::AHEAD, VREGION = NST * TILE;
  extern __shared__ __align__(16) char smem[];   // K[NST] then V[NST]; tile j in buffer j % NST

  const TileCoord tc = map_block<CAUSAL, D>(blockIdx.x, BH, T, true);
  if (!tc.valid) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = w & (RG - 1), kg = w / RG;
  const int half = lane >> 5, n = lane & 31;
  const int q0 = tc.tile * BM;
  const int wave_qmin = q0 + 32 * rg, my_q = wave_qmin + n;
  const __bf16* qh = q + head_offset(maps.q, tc.bh, H);
  const __bf16* kh = k + head_offset(maps.k, tc.bh, H);
  const __bf16* vh = v + head_offset(maps.v, tc.bh, H);
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale * kLog2e)));
  const uint32_t base = lds_base(smem);

  const int q_end = (q0 + BM < S ? q0 + BM : S);
  const int n_tiles = CAUSAL ? (q_end + BN - 1) / BN : (S + BN - 1) / BN;
  const TileLoader<D, BN, 2 * RG> kload(lane, w, maps.k.row), vload(lane, w, maps.v.row);
  constexpr int NDMA = decltype(kload)::N + decltype(vload)::N;
  auto copy_tile = [&](int jj, int buf) __attribute__((always_inline)) {
    kload.issue(kh, jj * BN, S, base + buf * TILE);
    vload.issue(vh, jj * BN, S, base + VREGION + buf * TILE);
  };

  // the Q rows pass through the last buffer, K first, then V; a row group's two waves copy one half each
  const uint32_t frag = base + (rg < 2 ? 0 : VREGION) + AHEAD * TILE + (rg & 1) * HALF;
  issue_fragments<D, 2>(qh, maps.q.row, wave_qmin, S, lane, kg, frag);
#pragma unroll
  for (int jj = 0; jj < AHEAD; jj++)
    if (jj < n_tiles) copy_tile(jj, jj);
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int e = 0; e < 16; e++) oacc[db][e] = 0.f;
  SoftmaxState st;
  // A row need not see a key of the second half, nor one with a score above -inf: its reference starts at the lowest finite value
  // instead of -inf, where a score of -inf weighs 0 and NaN stays NaN.  Key 0 is in the first half, which starts as in fwd_kernel.
  if (kg == 1) st.mref_c = -FLT_MAX;

  // Key blocks (half kg of tiles 0, 1, ...) this wave works on and how many of them need no mask (n_full >= n_w - 1).
  const int k_end = CAUSAL ? (wave_qmin + 32 < S ? wave_qmin + 32 : S) : S;        // keys [0, k_end) are visible to some row,
  const int k_all = CAUSAL ? wave_qmin + 1 : S;                                     // [0, k_all) to every row
  const int n_w = wave_qmin < S ? (k_end - 32 * kg + BN - 1) / BN : 0;              // (numerators are >= 0: k_end >= 1, k_all >= 1)
  const int n_full = (k_all + 32 - 32 * kg) / BN;

  if (n_tiles >= AHEAD) wait_tile_loads_except<AHEAD * NDMA>();
  else wait_tile_loads();
  __syncthreads();
  bf16x8 qf[KS];
  read_fragments<D>(frag, lane, qf);
  wait_tile_loads();
  __syncthreads();

  const FwdLaneAddr<D> la(lane);
  const uint32_t kbase = base + kg * HALF;
  // klo = contraction steps 0..KS/2-1 of the tile after the one scored next, khi = steps KS/2..KS-1 of the tile
  // scored next, vaddr = current V tile
  uint32_t klo[DB], khi[DB], vaddr[DB][2];
#pragma unroll
  for (int i = 0; i < DB; i++) { klo[i] = kbase + la.k[i] + 2 * TILE; khi[i] = kbase + la.k[i + DB] + TILE; }
#pragma unroll
  for (int db = 0; db < DB; db++) { vaddr[db][0] = kbase + VREGION + la.v[db][0]; vaddr[db][1] = kbase + VREGION + la.v[db][1]; }

  f32x16 sa, sb;
  bf16x8 kop[DB], vop[DB];
#pragma unroll
  for (int db = 0; db < DB; db++) vop[db] = lds_tr_pair(vaddr[db][0], vaddr[db][1], 0);
  if (n_w > 0) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sa = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(kbase + la.k[ks]), qf[ks], sa);
#pragma unroll
    for (int i = 0; i < DB; i++) kop[i] = lds_b128(kbase + la.k[i], TILE);
    if (n_w > 1) check_reference<DB>(max16(sa), c, st, oacc);
  }

  int j = 0, buf = 0;   // tile and its buffer (j % NST)
  auto wrap_step = [&](int b) __attribute__((always_inline)) { return (b == NST - 1) ? -(NST - 1) * TILE : TILE; };   // buffer b -> next
  auto plus = [&](int d) __attribute__((always_inline)) { return buf + d >= NST ? buf + d - NST : buf + d; };
  auto copy_ahead = [&]() __attribute__((always_inline)) {
    if (j + AHEAD < n_tiles) copy_tile(j + AHEAD, plus(AHEAD));   // replaces tile j-1
  };
  auto finish_tile = [&]() __attribute__((always_inline)) {
    // tiles up to j+3 must have landed: the next iteration reads j+1, j+2 and the first operands of j+3
    if (j + AHEAD < n_tiles) wait_tile_loads_except<(AHEAD - 3) * NDMA>();
    else wait_tile_loads();
    __syncthreads();
    buf = plus(1);
  };
  auto step = [&](const f32x16& s_cur, f32x16& s_next) __attribute__((always_inline)) {
    const bool whole = j + AHEAD < n_tiles && (j + AHEAD + 1) * BN <= S;
    if (!whole) copy_ahead();
    const __bf16* kt = kload.tile_ptr(kh, (j + AHEAD) * BN);
    const __bf16* vt = vload.tile_ptr(vh, (j + AHEAD) * BN);
    const uint32_t dst = base + plus(AHEAD) * TILE;
    const auto copy_whole = [&]() __attribute__((always_inline)) {
      if (whole) {
        kload.issue_whole(kt, dst);
        vload.issue_whole(vt, dst + VREGION);
      }
    };
    const int khi_step = wrap_step(plus(1)), klo_step = wrap_step(plus(2));
    const float m = half_step<D, 0, 0, 0, true>(copy_whole, s_cur, s_next, kop, vop, qf, klo, khi, vaddr, wrap_step(buf), oacc, c, st);
    if (j + 1 < n_w - 1) check_reference<DB>(m, c, st, oacc);   // the plain path masks first
#pragma unroll
    for (int i = 0; i < DB; i++) { khi[i] += khi_step; klo[i] += klo_step; }
    finish_tile();
    j++;
  };
  // two tiles per trip, so that the scores alternate between sa and sb without moves
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
      if (j >= n_full) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int key = j * BN + 32 * kg + 8 * (e >> 2) + 4 * half + (e & 3);
          sa[e] = (CAUSAL ? (key <= my_q) : (key < S)) ? sa[e] : -INFINITY;
        }
      }
      bf16x8 p[2];
      check_reference<DB>(max16(sa), c, st, oacc);
      exp_pack(sa, c, st, p);
      pv_block<D>(vaddr, 0, p, oacc);
    }
    finish_tile();
  }

  // merge: O = a0 O0 + a1 O1 with a = 2^(own reference - common reference); wave kg finishes half of the head
  // dimension and hands the other half over.  The second half counts for the rows that see its first key, 32; which rows these
  // are is a matter of the indexes and not of the reference, which a NaN score does not move.
  constexpr int HB = DB / 2;
  const float l_own = half_sum(st.lsum[0] + st.lsum[1]);
  float* stats = reinterpret_cast<float*>(smem + G::ROW_STATS);
#pragma unroll
  for (int b = 0; b < HB; b++) {
    const f32x16 give = kg == 0 ? oacc[HB + b] : oacc[b];
    lds_put_block(smem + ((kg * RG + rg) * HB + b) * 4096, lane, give);
  }
  stats[(w * 64 + lane) * 2] = st.mref_c;
  stats[(w * 64 + lane) * 2 + 1] = l_own;
  __syncthreads();
  {
    const float m_other = stats[((w ^ RG) * 64 + lane) * 2], l_other = stats[((w ^ RG) * 64 + lane) * 2 + 1];
    const float m = fmaxf(st.mref_c, m_other);
    const bool second = (CAUSAL ? my_q : S - 1) >= 32;
    const bool own = kg == 0 || second, other = kg == 1 || second;
    const float a_own = own ? __builtin_amdgcn_exp2f(st.mref_c - m) : 0.f;
    const float a_other = other ? __builtin_amdgcn_exp2f(m_other - m) : 0.f;
    const float ltot = (own ? l_own * a_own : 0.f) + (other ? l_other * a_other : 0.f);
    const float inv = 1.f / ltot;
    char* const in = smem + ((kg ^ 1) * RG + rg) * HB * 4096;   // what the other wave handed over; the results pass through it too
#pragma unroll
    for (int b = 0; b < HB; b++) {
      const f32x16 mine = kg == 0 ? oacc[b] : oacc[HB + b];
      const f32x16 got = lds_get_block(in + b * 4096, lane);
      f32x16 x;
#pragma unroll
      for (int e = 0; e < 16; e++) x[e] = ((own ? mine[e] * a_own : 0.f) + (other ? got[e] * a_other : 0.f)) * inv;
      put_rows<32 * HB>(in, lane, b, x);   // block b takes no more than the first b + 1 blocks
    }
    if (half == 0 && kg == 0 && my_q < S) lse[(size_t)tc.bh * S + my_q] = m * kLn2 + __logf(ltot);
    store_rows<32 * HB>(in, lane, o + head_offset(maps.o, tc.bh, H) + (size_t)wave_qmin * maps.o.row + 32 * HB * kg, maps.o.row, S - wave_qmin);
  }
}

// The forward at head dimension 128 for small grids (forward_rows): a workgroup owns 64 query rows and its four pairs of waves share the keys, wave
// (rg, kg) on 32 rows and key block kg of every 128-key tile.  A quarter of the steps of a 256-row workgroup at two waves per SIMD; a
// tile's copy serves 64 rows.  A tile of K and V takes 64 KB, so LDS holds three of K and two of V, and a step reads nothing ahead of its own
// tiles: K(j+1), which it scores, and V(j).  K runs two tiles ahead, V(j+1) has the length of step j to land, which it does not always keep: a step
// takes 1.0 us where the split kernel's takes 0.79.  64 rows in two groups -> in four, us: 12 heads x 1500 22.3 -> 19.6, 4 x 2048 26.5 -> 22.1,
// 2 x 8192 91 -> 70, 3 x 300 8.25 -> 8.6 (the merge of four).
template <int D>
struct FwdQuad {
  static constexpr int KG = 4, RG = 2, NK = 3, NV = 2;
  static constexpr int TILE = 32 * KG * D * 2;
  static constexpr int LDS = (NK + NV) * TILE;
  static constexpr int STATS = 8 * (D / 32) * 4096;          // merge: after the accumulator blocks, (reference, sum) of every row and group
  static_assert(STATS + 8 * 64 * 8 <= LDS && D / 32 == KG, "the merge reuses the tile buffers; a wave finishes one block of the head dimension");
};

// One step: S of the next tile while P of this one is formed and multiplied, in 16 slots like half_step,
// with the same vector work in them; the operands come from the tile alone.
template <int D, typename Copy>
__device__ __forceinline__ float quad_step(const Copy& copy_tiles, const f32x16& s_cur, f32x16& s_next, const bf16x8 (&qf)[D / 16],
                                           const int (&kaddr)[D / 16], const int (&vaddr)[D / 32][2], uint32_t kbuf, uint32_t vbuf,
                                           f32x16 (&oacc)[D / 32], float c, SoftmaxState& st) {
  constexpr int KS = D / 16, DB = D / 32, RING = KS / 2;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 kop[RING], vop[RING];
  StepWeights<KS> w;
#pragma unroll
  for (int i = 0; i < RING; i++) kop[i] = lds_b128(kbuf + kaddr[i]);
#pragma unroll
  for (int i = 0; i < KS; i++) {
    s_next = mfma32(kop[i % RING], qf[i], i == 0 ? zero : s_next);
    if (i < RING) kop[i] = lds_b128(kbuf + kaddr[i + RING]);
    else vop[i - RING] = lds_tr_pair(vbuf + vaddr[i - RING][0], vbuf + vaddr[i - RING][1], 0);
    if (i == 1) copy_tiles();
    w.in_score_slot(i, s_cur, c, st);
    __builtin_amdgcn_sched_barrier(0);
  }
  StepMaximum<KS> m;
#pragma unroll
  for (int i = 0; i < KS; i++) {
    oacc[i % DB] = mfma32(vop[i % RING], w.packed(i / DB), oacc[i % DB]);
    if (i < RING) {
      vop[i] = lds_tr_pair(vbuf + vaddr[i][0], vbuf + vaddr[i][1], 16 * D * 2);
      w.in_output_slot(i, s_cur, c, st);
    }
    m.in_output_slot(i, s_next);
    __builtin_amdgcn_sched_barrier(0);
  }
  return m.m0;
}

template <int D, bool CAUSAL>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
fwd_quad_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                __bf16* __restrict__ o, float* __restrict__ lse, FwdMaps maps, int BH, int H, int S, int T, float scale) {
  using G = FwdQuad<D>;
  constexpr int RG = G::RG, KG = G::KG, BM = 32 * RG, BN = 32 * KG, KS = D / 16, DB = D / 32;
  constexpr int TILE = G::TILE, HALF = 32 * D * 2, VREGION = G::NK * TILE;
  extern __shared__ __align__(16) char smem[];   // K[3] then V[2]; tile j in buffers j % 3 and j % 2

  const TileCoord tc = map_block<CAUSAL, D>(blockIdx.x, BH, T, true);
  if (!tc.valid) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = w & (RG - 1), kg = w / RG;
  const int half = lane >> 5, n = lane & 31;
  const int q0 = tc.tile * BM;
  const int wave_qmin = q0 + 32 * rg, my_q = wave_qmin + n;
  const __bf16* qh = q + head_offset(maps.q, tc.bh, H);
  const __bf16* kh = k + head_offset(maps.k, tc.bh, H);
  const __bf16* vh = v + head_offset(maps.v, tc.bh, H);
  const float c = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale * kLog2e)));
  const uint32_t base = lds_base(smem);

  const int q_end = (q0 + BM < S ? q0 + BM : S);
  const int n_tiles = CAUSAL ? (q_end + BN - 1) / BN : (S + BN - 1) / BN;
  const TileLoader<D, BN, 8> kload(lane, w, maps.k.row), vload(lane, w, maps.v.row);
  constexpr int NDMA = decltype(kload)::N;   // copy instructions per wave and tile of K or V

  // the Q rows pass through the second V buffer; the four waves of a row group copy a quarter each
  const uint32_t frag = base + VREGION + TILE + rg * HALF;
  issue_fragments<D, KG>(qh, maps.q.row, wave_qmin, S, lane, kg, frag);
  kload.issue(kh, 0, S, base);
  vload.issue(vh, 0, S, base + VREGION);
  if (n_tiles > 1) kload.issue(kh, BN, S, base + TILE);
  if (n_tiles > 2) kload.issue(kh, 2 * BN, S, base + 2 * TILE);
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int e = 0; e < 16; e++) oacc[db][e] = 0.f;
  SoftmaxState st;
  if (kg > 0) st.mref_c = -FLT_MAX;   // as in fwd_split_kernel

  // Key blocks (block kg of tiles 0, 1, ...) this wave works on and how many of them need no mask (n_full >= n_w - 1).
  const int k_end = CAUSAL ? (wave_qmin + 32 < S ? wave_qmin + 32 : S) : S;
  const int k_all = CAUSAL ? wave_qmin + 1 : S;
  const int n_w = wave_qmin < S && k_end > 32 * kg ? (k_end - 32 * kg + BN - 1) / BN : 0;
  const int n_full = (k_all + BN - 32 - 32 * kg) / BN;

  if (n_tiles > 2) wait_tile_loads_except<4 * NDMA>();
  else wait_tile_loads();
  __syncthreads();
  bf16x8 qf[KS];
  read_fragments<D>(frag, lane, qf);
  if (n_tiles > 2) wait_tile_loads_except<NDMA>();   // K(0), V(0), K(1)
  else wait_tile_loads();
  __syncthreads();

  const FwdLaneAddr<D> la(lane);
  const uint32_t kbase = base + kg * HALF, vbase = kbase + VREGION;
  f32x16 sa, sb;
  if (n_w > 0) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sa = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sa = mfma32(lds_b128(kbase + la.k[ks]), qf[ks], sa);
    if (n_w > 1) check_reference<DB>(max16(sa), c, st, oacc);
  }
  __syncthreads();   // the first step copies K(3) over K(0)

  int j = 0, kb = 0;   // tile, j % 3
  auto next3 = [&](int b) __attribute__((always_inline)) { return b == 2 ? 0 : b + 1; };
  auto copy_ahead = [&]() __attribute__((always_inline)) {
    // V(j+1) replaces V(j-1), K(j+3) replaces K(j), scored in the step before this one
    if (j + 1 < n_tiles) vload.issue(vh, (j + 1) * BN, S, base + VREGION + ((j + 1) & 1) * TILE);
    if (j + 3 < n_tiles) kload.issue(kh, (j + 3) * BN, S, base + kb * TILE);
  };
  auto finish_tile = [&]() __attribute__((always_inline)) {
    if (j + 3 < n_tiles) wait_tile_loads_except<NDMA>();   // K(j+3) may fly; K(j+2) and V(j+1) have landed
    else wait_tile_loads();
    __syncthreads();
    kb = next3(kb);
  };
  auto step = [&](const f32x16& s_cur, f32x16& s_next) __attribute__((always_inline)) {
    const bool whole = j + 3 < n_tiles && (j + 4) * BN <= S;
    if (!whole) copy_ahead();
    const __bf16* kt = kload.tile_ptr(kh, (j + 3) * BN);
    const __bf16* vt = vload.tile_ptr(vh, (j + 1) * BN);
    const uint32_t vdst = base + VREGION + ((j + 1) & 1) * TILE, kdst = base + kb * TILE;
    const auto copy_whole = [&]() __attribute__((always_inline)) {
      if (whole) {
        vload.issue_whole(vt, vdst);
        kload.issue_whole(kt, kdst);
      }
    };
    const float m = quad_step<D>(copy_whole, s_cur, s_next, qf, la.k, la.v, kbase + next3(kb) * TILE, vbase + (j & 1) * TILE, oacc, c, st);
    if (j + 1 < n_w - 1) check_reference<DB>(m, c, st, oacc);   // the plain path masks first
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
      if (j >= n_full) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int key = j * BN + 32 * kg + 8 * (e >> 2) + 4 * half + (e & 3);
          sa[e] = (CAUSAL ? (key <= my_q) : (key < S)) ? sa[e] : -INFINITY;
        }
      }
      bf16x8 p[2];
      uint32_t vaddr[DB][2];
#pragma unroll
      for (int db = 0; db < DB; db++) {
        vaddr[db][0] = vbase + (j & 1) * TILE + la.v[db][0];
        vaddr[db][1] = vbase + (j & 1) * TILE + la.v[db][1];
      }
      check_reference<DB>(max16(sa), c, st, oacc);
      exp_pack(sa, c, st, p);
      pv_block<D>(vaddr, 0, p, oacc);
    }
    finish_tile();
  }

  // merge: O = sum over the groups of 2^(own reference - common reference) O_g; wave kg finishes block kg of the head dimension.  A
  // group counts for the rows that see its first key, 32 * kg.
  const float l_own = half_sum(st.lsum[0] + st.lsum[1]);
  float2* const stats = reinterpret_cast<float2*>(smem + G::STATS);
#pragma unroll
  for (int db = 0; db < DB; db++)
    if (db != kg) lds_put_block(smem + (w * DB + db) * 4096, lane, oacc[db]);
  stats[w * 64 + lane] = make_float2(st.mref_c, l_own);
  __syncthreads();
  const int seen = CAUSAL ? my_q : S - 1;
  float a[KG], m = -INFINITY, ltot = 0.f;
  float2 ml[KG];
#pragma unroll
  for (int g = 0; g < KG; g++) {
    ml[g] = stats[(rg + RG * g) * 64 + lane];
    if (seen >= 32 * g) m = fmaxf(m, ml[g].x);
  }
#pragma unroll
  for (int g = 0; g < KG; g++) {
    a[g] = seen >= 32 * g ? __builtin_amdgcn_exp2f(ml[g].x - m) : 0.f;
    ltot += seen >= 32 * g ? ml[g].y * a[g] : 0.f;
  }
  const float inv = 1.f / ltot;
  f32x16 x;
#pragma unroll
  for (int e = 0; e < 16; e++) x[e] = 0.f;
#pragma unroll
  for (int g = 0; g < KG; g++) {
    f32x16 part;
    if (g == kg) {
#pragma unroll
      for (int db = 0; db < DB; db++)
        if (db == g) part = oacc[db];
    } else {
      part = lds_get_block(smem + ((rg + RG * g) * DB + kg) * 4096, lane);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] += seen >= 32 * g ? part[e] * a[g] : 0.f;
  }
#pragma unroll
  for (int e = 0; e < 16; e++) x[e] *= inv;
  char* const out = smem + (w * DB + kg) * 4096;   // this wave's own block, which nobody put anything in
  put_rows<32>(out, lane, 0, x);
  if (half == 0 && kg == 0 && my_q < S) lse[(size_t)tc.bh * S + my_q] = m * kLn2 + __logf(ltot);
  store_rows<32>(out, lane, o + head_offset(maps.o, tc.bh, H) + (size_t)wave_qmin * maps.o.row + 32 * kg, maps.o.row, S - wave_qmin);
}

template <int D, bool CAUSAL>
static hipError_t launch_fwd_t(const void* q, const void* k, const void* v, void* o, float* lse,
                               const FwdMaps& maps, int B, int H, int S, float scale, hipStream_t stream) {
  const int BH = B * H;
  const Rows rows = forward_rows(D, BH, S, CAUSAL);
  const int T = tiles(S, rows);
  const unsigned grid = (unsigned)grid_blocks(BH, T);
  size_t lds = FwdSplit<D, 4>::LDS;
  auto kern = fwd_split_kernel<D, CAUSAL, 4>;
  if (rows == Rows::k64) {
    kern = fwd_split_kernel<D, CAUSAL, 2>;
    lds = FwdSplit<D, 2>::LDS;
  }
  if constexpr (D == 128) {   // at head dimension 64 forward_rows knows the two above only
    if (rows == Rows::k64Quad) {
      kern = fwd_quad_kernel<D, CAUSAL>;
      lds = FwdQuad<D>::LDS;
    } else if (rows == Rows::k256) {
      kern = fwd_kernel<D, CAUSAL>;
      lds = 8 * 64 * D * 2;
    }
  }
  static unsigned long long configured[4] = {};   // per template instantiation and kernel
  hipError_t e = allow_dynamic_lds(kern, lds, configured[(int)rows]);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(rows == Rows::k64 ? 256 : 512), lds, stream, (const __bf16*)q, (const __bf16*)k,
                     (const __bf16*)v, (__bf16*)o, lse, maps, BH, H, S, T, scale);
  return hipGetLastError();
}

hipError_t launch_fwd(const void* q, const void* k, const void* v, void* o, float* lse, const FwdMaps& maps,
                      int B, int H, int S, int D, float scale, bool causal, hipStream_t stream) {
  if (D == 128) return causal ? launch_fwd_t<128, true>(q, k, v, o, lse, maps, B, H, S, scale, stream)
                              : launch_fwd_t<128, false>(q, k, v, o, lse, maps, B, H, S, scale, stream);
  return causal ? launch_fwd_t<64, true>(q, k, v, o, lse, maps, B, H, S, scale, stream)
                : launch_fwd_t<64, false>(q, k, v, o, lse, maps, B, H, S, scale, stream);
}

}  // namespace helix
