// Causal window attention over the paged KV cache (grouped-query), bf16 MFMA
// with fp32 online softmax.
//
// Reduction schedule of one query row at absolute position p (it depends on p
// and on nothing else - not on the window, the row's index in it, the batch, or
// the context lengths of other sequences).  Keys are cut at absolute positions:
//   step   = 64 keys   [64 j, 64 j + 64)
//   chunk  = 256 keys  = 4 steps
//   super  = 2048 keys = 8 chunks
// * A chunk partial (m, l, acc) starts at (-inf, 0, 0) and is advanced by one
//   online-softmax step per 64 keys in ascending order; a step computes its
//   scores with head_dim/32 MFMA k-steps per 16-key block, takes max and sum
//   over its 64 keys in a fixed tree, rescales, and adds P V with two MFMA
//   k-steps of 32 keys.
// * The chunk partials of a super are folded left to right (fold() below), giving
//   the super partial; the super partials are folded left to right, giving the row.
// Keys beyond p contribute exact zeros (masked before the exponential); a step or
// a chunk in which every key of a row is masked leaves that row's state bit for
// bit unchanged, so rows of different positions can share a workgroup.
//
// Work distribution (free to change, does not touch the bits): a workgroup owns one unit of the keys
// of a (sequence, kv head) for 8 blocks of 16 query rows (attention_stream_kernel, 8 waves) or up to 4
// (attention_kernel, 4 waves).  Query rows are ordered by token (RowOrder): those that a partly filled window
// lacks come last, and blocks of 16 without any row are left out (27 sequences, 516 of 999 rows: 43.5 -> 28.4 us a launch against
// r = q_head_in_group * window + i, where every block has some).  A unit is
//   a chunk          - few sequences: most parallelism; chunk partials are written and the merge
//                      kernel does all folds;
//   a super          - more sequences: chunks are folded in registers, 8 times fewer partials;
//   a whole sequence - many sequences whose lengths deal out evenly (the plan kernel decides from the
//                      lengths): supers are folded in registers too and the workgroup writes the
//                      output rows itself, as it does whenever every context fits one super.
// K and V tiles go from global memory straight into a ring of LDS entries of 64 keys, three entries in
// flight, already in MFMA operand order (see the KV tile layouts in llm42.h), so nothing is transposed.
#include <algorithm>
#include <type_traits>

#include "llm42_dev.h"

namespace {

constexpr int STEP = 64, CHUNK = 256, SUPER_KEYS = 2048;
constexpr float kLazy = 8.0f;   // log2 units, see softmax_step

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

// state <- state (+) part, the only way two partials are ever combined:
//   mn = max(M, m2), a = exp2(M - mn), b = exp2(m2 - mn), L = fma(l2, b, L * a), A = fma(a2, b, A * a).
// One of a, b is exactly 1; where a is 1 for every lane of the wave (the running maximum stands,
// the usual case) the multiplication by it is left out, which cannot change a bit.
template <int NV>
__device__ inline void fold(float& M, float& L, f32x4 (&A)[NV], float m2, float l2, const f32x4 (&a2)[NV]) {
  const float mn = fmaxf(M, m2);
  const float mu = mn == -INFINITY ? 0.f : mn;
  const float a = __builtin_amdgcn_exp2f(M - mu), b = __builtin_amdgcn_exp2f(m2 - mu);
  if (__builtin_amdgcn_ballot_w64(a != 1.0f) != 0) {
    L *= a;
#pragma unroll
    for (int i = 0; i < NV; ++i) A[i] *= a;
  }
  L = __builtin_fmaf(l2, b, L);
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c) A[i][c] = __builtin_fmaf(a2[i][c], b, A[i][c]);
  M = mn;
}

// Copy one KV tile (TL KiB) from global memory to LDS without passing through registers: one
// instruction moves 1 KiB, lane i's 16 bytes landing at LDS byte address `dst` + 16 i (M0 holds the
// wave-uniform destination).  `src` already includes this lane's 16-byte offset.  Written as
// assembly on purpose: with the compiler's own form of this load every later LDS read waits for
// all earlier ones, which un-pipelines the operand reads of the steps.  The compiler therefore
// does not count these loads; fetch_landed() is the only wait that covers them.  Nothing else in
// this kernel uses M0.  STREAM marks the load non-temporal: K and V tiles are read once per (sequence,
// kv head) and launch, and the hint takes the fetch stream alone (no arithmetic) from 5.1 to 5.7 TB/s.
template <int TL, bool STREAM = false>
__device__ __forceinline__ void tile_to_lds(uint32_t dst, const uint4* src) {
#pragma unroll
  for (int i = 0; i < TL; ++i)
    if constexpr (STREAM)
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                   :
                   : "v"(src + i * 64), "s"(dst + i * 1024)
                   : "memory", "m0");
    else
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                   :
                   : "v"(src + i * 64), "s"(dst + i * 1024)
                   : "memory", "m0");
}
// At most N of the fetches this wave has issued are still on their way (they complete in order;
// the barrier that follows covers the other waves').
template <int N>
__device__ __forceinline__ void fetch_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// Every fetch this wave has issued is in LDS.
// (Both forms of the wait: the first tells the compiler that its own loads are complete as well.)
__device__ __forceinline__ void fetch_landed() {
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Butterflies over the four 16-lane rows of a wave (lane ^ 16, then lane ^ 32) without a trip
// through LDS: a swap leaves the two partners of every lane in the two results, and max / + are
// commutative, so each lane gets the same bits as from the shuffle form of the butterfly.
__device__ __forceinline__ float rows_max(float x) {
  u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ float rows_sum(float x) {
  u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r.x) + __uint_as_float(r.y);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r.x) + __uint_as_float(r.y);
}

// The output of query row r (of the sequence whose rows begin at `base`, kv head kvh): acc / l in bf16, into the tile layout of the
// O-projection's activation operand - exactly what the merge pass computes from a row's folded partials.
// The lane holds features d * 16 + g * 4 .. + 3 of the row; the lanes g and g ^ 1 of a row trade halves so that each
// writes 8 consecutive features of every second block d (16 bytes per lane and store, half as many stores).
// Called by all four lanes of a row or by none.
template <int HD>
__device__ __forceinline__ void store_output(uint16_t* __restrict__ out, int d_attn, int base, int kvh, RowOrder order,
                                             int r, int g, const f32x4 (&acc)[HD / 16], float l) {
  const int i = order.token(r), hq = kvh * order.group + order.head(r);
  const bool odd = g & 1;
#pragma unroll
  for (int d = 0; d < HD / 16; d += 2) {
    const uint32_t a0 = pack2_bf16(acc[d][0] / l, acc[d][1] / l), a1 = pack2_bf16(acc[d][2] / l, acc[d][3] / l);
    const uint32_t b0 = pack2_bf16(acc[d + 1][0] / l, acc[d + 1][1] / l), b1 = pack2_bf16(acc[d + 1][2] / l, acc[d + 1][3] / l);
    // even g keeps block d and takes its neighbour's four features of it; odd g keeps block d + 1
    const uint32_t t0 = __shfl_xor(odd ? a0 : b0, 16), t1 = __shfl_xor(odd ? a1 : b1, 16);
    const u32x4 o = odd ? (u32x4){t0, t1, b0, b1} : (u32x4){a0, a1, t0, t1};
    *(u32x4*)(out + pk_off(base + i, hq * HD + (d + (odd ? 1 : 0)) * 16 + (g & 2) * 4, d_attn)) = o;
  }
}

// What a step does between its two products, for one block of 16 query rows: masks the raw scores `sc` of the 64 keys
// from k0, advances (m, l) and rescales acc, and leaves P in bf16 in `pf`, as the operand of the P V product.
template <int DB, bool MASKED>
__device__ __forceinline__ void softmax_update(f32x4 (&sc)[4], int k0, int g, int qpos, float scale_log2, float& m, float& l,
                                               f32x4 (&acc)[DB], u32x4 (&pf)[2], const bool first) {
  if (MASKED) {
    // a select, not arithmetic: scores of keys past k_hi come from stale tiles and may be anything
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k0 + b * 16 + g * 4 + e > qpos) sc[b][e] = -INFINITY;
  }
  float mx = fmaxf(fmaxf(sc[0][0], sc[0][1]), sc[0][2]);
  mx = fmaxf(fmaxf(mx, sc[0][3]), sc[1][0]);
  mx = fmaxf(fmaxf(mx, sc[1][1]), sc[1][2]);
  mx = fmaxf(fmaxf(mx, sc[1][3]), sc[2][0]);
  mx = fmaxf(fmaxf(mx, sc[2][1]), sc[2][2]);
  mx = fmaxf(fmaxf(mx, sc[2][3]), sc[3][0]);
  mx = fmaxf(fmaxf(mx, sc[3][1]), sc[3][2]);
  mx = rows_max(fmaxf(mx, sc[3][3]));
  // scaling by a positive constant is monotonic: max(scaled) == scaled(max), bit for bit
  const float m_step = mx * scale_log2;
  // The partial's reference exponent m moves up to this step's maximum only when that exceeds it by more than
  // kLazy (then p = exp2(score - m) stays at or below 2^kLazy); otherwise it stands and alpha is exactly 1.
  // (An empty partial has m = -inf: +inf > kLazy takes the step's maximum; -inf - -inf is NaN and keeps -inf.)
  const float m_new = (m_step - m > kLazy) ? m_step : m;
  const float m_use = (MASKED && m_new == -INFINITY) ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(m - m_use);
  float rs = 0.f;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      sc[b][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[b][e], scale_log2, -m_use));
    rs += ((sc[b][0] + sc[b][1]) + sc[b][2]) + sc[b][3];
  }
  rs = rows_sum(rs);
  // Rescaling by alpha is skipped where it cannot change a bit: in the first step of a partial (l and acc are
  // zero, and zero times alpha is zero) and where alpha is exactly 1 for every row of the wave.
  if (!first && __builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
    l *= alpha;
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d] *= alpha;
  }
  l += rs;
  m = m_new;
  // k-slot e of lane group g is key g*4+e of the first block of a pair (e < 4) or of the
  // second (e >= 4); V uses the same assignment
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    pf[kk][0] = pack2_bf16(sc[2 * kk][0], sc[2 * kk][1]);
    pf[kk][1] = pack2_bf16(sc[2 * kk][2], sc[2 * kk][3]);
    pf[kk][2] = pack2_bf16(sc[2 * kk + 1][0], sc[2 * kk + 1][1]);
    pf[kk][3] = pack2_bf16(sc[2 * kk + 1][2], sc[2 * kk + 1][3]);
  }
}

// One online-softmax step over the 64 keys [k0, k0 + 64): `lk` / `lv` are the step's four K and
// four V tiles in LDS.  MASKED = false is the same arithmetic with the comparisons that cannot
// fail left out: every key of the step is at or below every position of this wave's rows (and
// hence below k_hi).  The operand reads are issued one ring ahead of the MFMAs that consume them
// and the order is pinned, so that an LDS round trip is never waited for in full.
template <int HD, int CB, bool MASKED>
__device__ __forceinline__ void softmax_step(const uint4* lk, const uint16_t* lv, int k0, int k_hi, int lane,
                                             float scale_log2, const bf16x8 (&qf)[CB][HD / 32], const int (&qpos)[CB],
                                             float (&m)[CB], float (&l)[CB], f32x4 (&acc)[CB][HD / 16], const bool first) {
  constexpr int DK = HD / 32, DB = HD / 16, TV4 = HD * 2;
  const int col = lane & 15, g = lane >> 4;
  constexpr int RV = 4;                                     // V operands in flight
  bf16x8 kb[DK];                                            // K operands in flight, one per head-dim k-step
  u32x4 vb[RV];
  auto load_k = [&](int b, int d) { kb[d] = ((const bf16x8*)lk)[b * TV4 + d * 64 + lane]; };
  auto load_v = [&](int idx) {                              // idx = key pair kk * DB + feature block d
    const uint16_t* vt0 = lv + (size_t)(2 * (idx / DB)) * TV4 * 8 + (((idx % DB) * 4 + g) * 16 + col) * 4;
    const u32x2 lo = *(const u32x2*)vt0, hi = *(const u32x2*)(vt0 + TV4 * 8);
    vb[idx % RV] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
  };
  // ---- raw scores of 4 blocks of 16 keys: S^T[key][query] ---------------------------------
  f32x4 sc[CB][4];
#pragma unroll
  for (int d = 0; d < DK; ++d) load_k(0, d);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
#pragma unroll
    for (int d = 0; d < DK; ++d) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        sc[cb][b] = mfma16(kb[d], qf[cb][d], d == 0 ? (f32x4){0.f, 0.f, 0.f, 0.f} : sc[cb][b]);
      if (b + 1 < 4) load_k(b + 1, d);
      else if (d < RV) load_v(d);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int i = DK; i < RV; ++i) load_v(i);
  // ---- mask, online softmax state (m in units of scaled scores), P in bf16 -----------------
  u32x4 pf[CB][2];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    softmax_update<DB, MASKED>(sc[cb], k0, g, qpos[cb], scale_log2, m[cb], l[cb], acc[cb], pf[cb], first);
  }
  // ---- acc^T[feature][query] += V^T P^T, 32 keys per MFMA ------------------------------
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int idx = 0; idx < 2 * DB; ++idx) {
    const int kk = idx / DB, d = idx % DB;
    if (MASKED) {
      // slots at or beyond k_hi hold stale, never-written or foreign data: force them to zero
      // so that 0 * garbage cannot produce a NaN
      const int kp0 = k0 + kk * 32 + g * 4, kp1 = kp0 + 16;
      if (kp1 + 3 >= k_hi) {
        u32x4& v = vb[idx % RV];
        if (kp0 + 0 >= k_hi) v[0] &= 0xFFFF0000u;
        if (kp0 + 1 >= k_hi) v[0] &= 0x0000FFFFu;
        if (kp0 + 2 >= k_hi) v[1] &= 0xFFFF0000u;
        if (kp0 + 3 >= k_hi) v[1] &= 0x0000FFFFu;
        if (kp1 + 0 >= k_hi) v[2] &= 0xFFFF0000u;
        if (kp1 + 1 >= k_hi) v[2] &= 0x0000FFFFu;
        if (kp1 + 2 >= k_hi) v[3] &= 0xFFFF0000u;
        if (kp1 + 3 >= k_hi) v[3] &= 0x0000FFFFu;
      }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      acc[cb][d] = mfma16(__builtin_bit_cast(bf16x8, vb[idx % RV]), __builtin_bit_cast(bf16x8, pf[cb][kk]),
                          acc[cb][d]);
    if (idx + RV < 2 * DB) load_v(idx + RV);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int HD, int CB, int NW, bool SUPER, int NBUF>
__device__ __forceinline__ void attention_items(
    const uint16_t* __restrict__ q, const uint4* __restrict__ k_plane, const uint4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int4* __restrict__ items, const int32_t* __restrict__ item_count,
    int32_t* __restrict__ queue, int n_kv_heads, RowOrder order, int r_pad, int y_blocks, int max_blocks_per_seq, int n_units,
    int part_rows, float scale_log2, float* __restrict__ part_acc, float* __restrict__ part_ml, uint16_t* __restrict__ attn_out,
    int d_attn) {
  constexpr int DK = HD / 32;        // MFMA k-steps over the head dimension (scores)
  constexpr int DB = HD / 16;        // 16-feature blocks of the output
  constexpr int TV4 = HD * 2;        // uint4 per KV tile (16 tokens x HD bf16)
  constexpr int TL = TV4 / 64;       // uint4 per lane per tile
  constexpr int UNIT = SUPER ? SUPER_KEYS : CHUNK;
  constexpr int AHEAD = NBUF - 1;       // ring of step buffers; steps in flight ahead of the one computed
  constexpr bool QUEUE = NBUF > 2;
  constexpr int FI = 8 * TL / NW;       // fetch instructions per wave per step (4 K and 4 V tiles in all)
  static_assert(NW == 4 || NW == 8, "a step's tiles are split over 4 or 8 waves");
  static_assert(TL % (NW / 4) == 0, "half a tile per wave needs an even number of pieces");
  __shared__ uint4 lds_k[NBUF][4 * TV4];   // per step: 4 K tiles
  __shared__ uint4 lds_v[NBUF][4 * TV4];   // and 4 V tiles
  __shared__ int wg_max[NW];
  __shared__ int next_work;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, g = lane >> 4;
  const uint32_t lds_k_addr = (uint32_t)(uintptr_t)(lds_ptr)&lds_k[0][0];
  const uint32_t lds_v_addr = (uint32_t)(uintptr_t)(lds_ptr)&lds_v[0][0];

  // One work item: unit `unit` of the keys of sequence `s`, kv head `kvh`, for the `yb`-th group of
  // NW * CB blocks of 16 query rows.  (A return leaves the item; every condition is workgroup-uniform.)
  auto run_item = [&](const int4 su, const int yb, const int kvh) {
  const int s = su.x, unit = su.y, L = su.z, tag = su.w, n = tag_rows(tag);
  if (yb * NW * CB * 16 >= n * order.group) return;                // whole workgroup: no live row
  const int k_lo = unit * UNIT;
  const int32_t* bt = block_table + (size_t)s * max_blocks_per_seq;
  // Requested before anything is known about the sequence, so that the three latencies (lengths,
  // block ids, query operands) overlap: the unit's block-table entries (clamped to the table, not
  // yet to the sequence) and the query operands of this wave's row blocks.
  const int first_blk = k_lo >> 4;
  const int raw0 = bt[min(first_blk + lane, max_blocks_per_seq - 1)];
  const int raw1 = SUPER ? bt[min(first_blk + 64 + lane, max_blocks_per_seq - 1)] : 0;
  bf16x8 qf[CB][DK];
  int row[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    row[cb] = ((yb * NW + wave) * CB + cb) * 16 + col;
    // row blocks past r_pad (grid padding) read the last real block instead; their rows are dead anyway
    const int rb = min(row[cb] >> 4, r_pad / 16 - 1);
    const uint16_t* qb = q + ((size_t)s * n_kv_heads + kvh) * r_pad * HD + (size_t)rb * DK * 512;
#pragma unroll
    for (int d = 0; d < DK; ++d) qf[cb][d] = *(const bf16x8*)(qb + d * 512 + lane * 8);
  }
  int qpos[CB];
  int wmax = -1, wmin = 0x7FFFFFFF;   // highest and lowest position among this wave's live rows
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int i = order.token(row[cb]);
    qpos[cb] = i < n ? L + i : -1;
    wmax = max(wmax, qpos[cb]);
    if (qpos[cb] >= 0) wmin = min(wmin, qpos[cb]);
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    wmax = max(wmax, __shfl_xor(wmax, off));
    wmin = min(wmin, __shfl_xor(wmin, off));
  }
  wmin = __builtin_amdgcn_readfirstlane(wmax) < 0 ? -1 : __builtin_amdgcn_readfirstlane(wmin);   // (-1: no live row, the wave only fetches)
  if (lane == 0) wg_max[wave] = wmax;
  __syncthreads();
  int gmax = wg_max[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) gmax = max(gmax, wg_max[w]);
  if (gmax < k_lo) return;                                   // whole workgroup: nobody looks into this unit
  const int k_hi = min(gmax + 1, k_lo + UNIT);               // exclusive; <= L + n
  const int n_steps = (k_hi - k_lo + STEP - 1) / STEP;
  const int last_blk = (k_hi - 1) >> 4;
  // table entries past the last needed block may hold anything: replace them by the last needed
  // block's id (its data is fetched in their place, and every key in those positions is masked)
  const int last_id = __shfl((last_blk - first_blk) < 64 ? raw0 : raw1, (last_blk - first_blk) & 63);
  const int ids0 = first_blk + lane <= last_blk ? raw0 : last_id;
  const int ids1 = first_blk + 64 + lane <= last_blk ? raw1 : last_id;

  // each wave fetches one (4 waves) or half (8 waves) of the four blocks of a step, its K and its V
  // tile, straight from global memory into LDS
  auto fetch = [&](int j) {
    constexpr int SPLIT = NW / 4, PIECES = TL / SPLIT;       // waves per block; 1 KiB pieces per wave and tile
    const int blk = wave / SPLIT, part = wave % SPLIT;
    const int bj = j * 4 + blk;                              // block index inside the unit (wave-uniform)
    const int id = bj < 64 ? __builtin_amdgcn_readlane(ids0, bj & 63) : __builtin_amdgcn_readlane(ids1, bj & 63);
    const uint32_t off = (uint32_t)(((j & (NBUF - 1)) * 4 + blk) * TV4 + part * PIECES * 64) * 16;
    const size_t src = ((size_t)id * n_kv_heads + kvh) * TV4 + part * PIECES * 64 + lane;
    tile_to_lds<PIECES, true>(lds_k_addr + off, k_plane + src);
    tile_to_lds<PIECES, true>(lds_v_addr + off, v_plane + src);
  };

  float m[CB], l[CB];
  f32x4 acc[CB][DB];
  float sm[CB], sl[CB];                                      // super mode: running fold of finished chunks
  f32x4 sacc[CB][DB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    m[cb] = -INFINITY;
    l[cb] = 0.f;
    sm[cb] = -INFINITY;
    sl[cb] = 0.f;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      acc[cb][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
      sacc[cb][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
  }

  // Steps j+1 .. j+AHEAD are in flight while step j is computed.  A buffer is refilled only after the
  // barrier that ends the step which read it; the wait before that barrier leaves the younger
  // fetches in flight (loads complete in order).
#pragma unroll
  for (int j = 0; j < AHEAD; ++j)
    if (j < n_steps) fetch(j);
  fetch_landed();
  __syncthreads();
  for (int j = 0; j < n_steps; ++j) {
    if (j + AHEAD < n_steps) fetch(j + AHEAD);                // into the buffer of step j - 1
    {
      const int k0 = k_lo + j * STEP;
      const uint4* sk = &lds_k[j & (NBUF - 1)][0];
      const uint16_t* sv = (const uint16_t*)&lds_v[j & (NBUF - 1)][0];
      const bool first = SUPER ? (j & 3) == 0 : j == 0;        // the chunk partial is empty
      if (k0 + STEP - 1 <= wmin)                               // wave-uniform
        softmax_step<HD, CB, false>(sk, sv, k0, k_hi, lane, scale_log2, qf, qpos, m, l, acc, first);
      else if (wmin >= 0)
        softmax_step<HD, CB, true>(sk, sv, k0, k_hi, lane, scale_log2, qf, qpos, m, l, acc, first);
    }
    if (SUPER && ((j & 3) == 3 || j + 1 == n_steps)) {
      // a chunk is complete: fold it into the running super partial and start the next one afresh
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        if (j < 4) {
          sm[cb] = m[cb];
          sl[cb] = l[cb];
#pragma unroll
          for (int d = 0; d < DB; ++d) sacc[cb][d] = acc[cb][d];
        } else {
          fold<DB>(sm[cb], sl[cb], sacc[cb], m[cb], l[cb], acc[cb]);
        }
        m[cb] = -INFINITY;
        l[cb] = 0.f;
#pragma unroll
        for (int d = 0; d < DB; ++d) acc[cb][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
    }
    // step j + 1 has landed once at most the fetches issued after it are outstanding
    const int younger = min(j + AHEAD, n_steps - 1) - (j + 1);
    if (younger >= 2) fetch_wait<2 * FI>();
    else if (younger == 1) fetch_wait<FI>();
    else fetch_wait<0>();
    __syncthreads();
  }

  // ---- partial of this unit for every row that reaches into it ---------------------------------
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    if (qpos[cb] < k_lo) continue;
    if (SUPER && attn_out) {   // (one unit per sequence: no partial, no merge pass)
      store_output<HD>(attn_out, d_attn, tag_base(tag), kvh, order, row[cb], g, sacc[cb], sl[cb]);
      continue;
    }
    const size_t prow = (((size_t)s * n_kv_heads + kvh) * n_units + unit) * part_rows + row[cb];
    float* pa = part_acc + prow * HD;
#pragma unroll
    for (int d = 0; d < DB; ++d) *(f32x4*)(pa + d * 16 + g * 4) = SUPER ? sacc[cb][d] : acc[cb][d];
    if (g == 0) *(float2*)(part_ml + prow * 2) = SUPER ? make_float2(sm[cb], sl[cb]) : make_float2(m[cb], l[cb]);
  }
  };  // run_item

  // Work distribution: the workgroups of the (CU-sized) grid take one item each to begin with and
  // pull further ones from a queue.  The list of (sequence, unit) pairs that hold keys is built once
  // per call (attention_plan_kernel), so no workgroup is spent on a unit past a sequence's end, and
  // the order in which workgroups finish does not matter: every item writes its own partial.
  const int per_item = n_kv_heads * y_blocks;
  const int total = *item_count * per_item;
  int4 su = items[blockIdx.x / per_item];                  // (in the list's room even if there is no such item)
  for (int t = blockIdx.x; t < total;) {
    const int rem = t % per_item;
    if constexpr (!QUEUE) {
      t += gridDim.x;
      const int4 next = items[min(t, total - 1) / per_item];
      run_item(su, rem % y_blocks, rem / y_blocks);
      su = next;
      if (t < total) __syncthreads();                      // every wave is done with the ring
    } else {
      run_item(su, rem % y_blocks, rem / y_blocks);
      __syncthreads();                                     // every wave is done with the ring
      if (threadIdx.x == 0) next_work = (int)gridDim.x + atomicAdd(queue, 1);
      __syncthreads();
      t = next_work;
      if (t < total) su = items[t / per_item];
    }
  }
}

template <int HD, int CB, int NW, bool SUPER, int NBUF>
__global__ __launch_bounds__(NW * 64, NBUF == 2 ? 2 : 1) void attention_kernel(
    const uint16_t* __restrict__ q, const uint4* __restrict__ k_plane, const uint4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int4* __restrict__ items, const int32_t* __restrict__ item_count,
    int32_t* __restrict__ queue, int n_kv_heads, RowOrder order, int r_pad, int y_blocks, int max_blocks_per_seq, int n_units,
    float scale_log2, float* __restrict__ part_acc, float* __restrict__ part_ml, uint16_t* __restrict__ attn_out,
    int d_attn) {
  attention_items<HD, CB, NW, SUPER, NBUF>(q, k_plane, v_plane, block_table, items, item_count, queue, n_kv_heads, order, r_pad, y_blocks,
                                           max_blocks_per_seq, n_units, r_pad, scale_log2, part_acc, part_ml, attn_out, d_attn);
}

// The same computation for 8 or more blocks of query rows per (sequence, kv head), as one stream per
// CU.  A workgroup of 8 waves (one block of 16 query rows each) walks its share of the work items
// (item t of round r goes to workgroup t mod G, rounds alternating direction, items sorted longest
// first: an even split without a queue).  Everything it needs from global memory arrives through one
// ring of LDS entries that never stops at an item boundary: per item first an entry with the eight
// row blocks' query operands, then one entry (4 K tiles + 4 V tiles) per 64-key step, AHEAD entries
// in flight.  A fetch cursor and a compute cursor walk the same item list independently; all item
// data they need is wave-uniform and comes through scalar loads, so nothing but the ring's own
// fetches is ever counted by vmcnt between the first and the last entry.  Past the last item the
// fetch cursor issues dummy fetches into slots nothing reads, which keeps the wait count constant.
// FOLD = false (measurement only): no chunk partials inside a super, one straight accumulation.
// FULL: every window of the call is full, a multiple of 128 query rows, and no item lacks keys that others have (see
// Workspace::full): nothing is tested for rows that are not there.  The loop is bound by instruction issue with every scalar register
// taken, and those tests' scalars cost 2 - 4 % of it: us a layer before there were any, with them for every call and now, 16 sequences x
// window 32 behind 1900 keys 56.7, 57.9, 56.5, 32 x 64 behind 1900 117.1, 121.4, 117.6, of 16 - 8000 316.7, 325.3, 315.2, 16 x 32
// behind 4500 85.2, 87.6, 85.0, 2 x 128 behind 3000 53.3, 54.7, 53.7; the same windows given as counts 0.5 - 2 % more, partly filled
// 10 - 15 % less than before.
// SEQ: an item is a whole sequence (all of its supers); the supers' partials are folded in registers, in the order
// of the merge pass, and the kernel writes the output rows itself.  The query operands then stay in LDS instead of
// registers (the third accumulator level needs theirs).
template <int HD, bool SUPER, bool FOLD, bool SEQ, bool FULL>
__global__ __launch_bounds__(512) void attention_stream_kernel(
    const uint16_t* __restrict__ q, const uint4* __restrict__ k_plane, const uint4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int4* __restrict__ items, const int32_t* __restrict__ item_count,
    int n_kv_heads, RowOrder order, int r_pad, int y_blocks, int max_blocks_per_seq, int n_units,
    float scale_log2, float* __restrict__ part_acc, float* __restrict__ part_ml, uint16_t* __restrict__ attn_out,
    int d_attn, const int32_t* __restrict__ seq_mode) {
  if (seq_mode && (*seq_mode != 0) != SEQ) return;   // the plan chose the other kind of item for this call (workgroup-uniform)
  constexpr int NW = 8, CB = 1;
  constexpr int DK = HD / 32, DB = HD / 16, TV4 = HD * 2, TL = TV4 / 64;
  constexpr int UNIT = SUPER ? SUPER_KEYS : CHUNK;
  constexpr int NBUF = 4, AHEAD = 3;
  constexpr int FI = TL;                // fetch instructions per wave per entry
  static_assert(TL % 2 == 0, "half a tile per wave");
  static_assert(!SEQ || (SUPER && FOLD), "whole sequences are folded like supers");
  __shared__ uint4 ring[NBUF][8 * TV4];
  __shared__ uint4 q_keep[SEQ ? 8 * TV4 : 1];   // SEQ: every wave's block of query operands for the current item

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, g = lane >> 4;
  const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_ptr)&ring[0][0];
  const int G = gridDim.x, w = blockIdx.x;
  const int per_item = n_kv_heads * y_blocks;
  const int total = *item_count * per_item;

  // a piece of work of this workgroup (wave-uniform; scalar loads)
  struct Work {
    bool valid;
    int s, kvh, yb, unit, L, n, base, k_lo, k_hi, n_steps;
  };
  const int item_tokens = (NW * 16 + order.group - 1) / order.group;   // (at least those that an item's rows span)
  // the list's entry of the ord-th piece; past the end: t = total, and a harmless stand-in, so that the dummy fetches read valid memory
  struct Entry {
    int t;
    int4 su;
  };
  auto entry_of = [&](int ord) {
    Entry e;
    e.t = min(ord * G + ((ord & 1) ? G - 1 - w : w), total);
    e.su = e.t < total ? items[e.t / per_item] : make_int4(0, 0, 0, seq_tag(1, 0));
    return e;
  };
  auto work_of = [&](const Entry e) {
    Work x;
    x.valid = e.t < total;
    const int rem = e.t % per_item;
    x.s = e.su.x, x.unit = e.su.y, x.L = e.su.z, x.n = tag_rows(e.su.w), x.base = tag_base(e.su.w);
    x.kvh = rem / y_blocks, x.yb = rem % y_blocks;
    x.k_lo = SEQ ? 0 : x.unit * UNIT;
    // Keys behind the last token of these rows are masked for all of them, and a masked step changes no state: left out (prefill of
    // 8 x 2048 tokens by 512: 0.995 -> 1.007 of the speed with rows by heads).
    const int end = x.L + (FULL ? x.n : min(x.n, (x.yb + 1) * item_tokens));
    x.k_hi = SEQ ? end : min(end, x.k_lo + UNIT);
    x.n_steps = (x.k_hi - x.k_lo + STEP - 1) / STEP;
    // (row blocks without a live row, or whose keys all lie before this unit: the query entry only)
    if (!FULL) x.n_steps = x.yb * NW * 16 < x.n * order.group ? max(0, x.n_steps) : 0;
    return x;
  };

  // ---- fetch cursor ----------------------------------------------------------------------------
  int f_ord = 0, f_entry = 0;           // entry 0 = query operands, entry e > 0 = step e - 1
  Work f = work_of(entry_of(0));
  int f_id = 0;                         // block id this wave needs for the entry at the cursor (steps only)
  const int blk = wave >> 1, part = wave & 1;
  auto id_for = [&](const Work& x, int e) {   // physical block of this wave's 16 keys of step e - 1
    const int b = min((x.k_lo >> 4) + (e - 1) * 4 + blk, (x.k_hi - 1) >> 4);   // never past the last block in use
    return block_table[(size_t)x.s * max_blocks_per_seq + b];
  };
  auto fetch_next = [&](int gidx) {
    const uint32_t slot = ring_addr + (uint32_t)((gidx & (NBUF - 1)) * 8 * TV4) * 16;
    if (!f.valid || f_entry == 0) {
      // this wave's block of 16 query rows (row blocks past r_pad read the last real one; past the
      // last item: the same fetch once more, into a slot nothing reads)
      const int rb = min(f.yb * NW + wave, r_pad / 16 - 1);
      const uint4* src = (const uint4*)(q + ((size_t)f.s * n_kv_heads + f.kvh) * r_pad * HD + (size_t)rb * DK * 512);
      tile_to_lds<TL>(slot + (uint32_t)(wave * TV4) * 16, src + lane);
    } else {
      const size_t src = ((size_t)f_id * n_kv_heads + f.kvh) * TV4 + part * (TL / 2) * 64 + lane;
      const uint32_t off = (uint32_t)(blk * TV4 + part * (TL / 2) * 64) * 16;
      tile_to_lds<TL / 2, true>(slot + off, k_plane + src);
      tile_to_lds<TL / 2, true>(slot + (uint32_t)(4 * TV4) * 16 + off, v_plane + src);
    }
    if (f.valid) {
      if (++f_entry > f.n_steps) {
        f = work_of(entry_of(++f_ord));
        f_entry = 0;
      } else {
        f_id = id_for(f, f_entry);      // requested one entry ahead of its use
      }
    }
  };

  // ---- compute cursor ---------------------------------------------------------------------------
#pragma unroll
  for (int e = 0; e < AHEAD; ++e) fetch_next(e);
  fetch_wait<(AHEAD - 1) * FI>();       // entry 0 has landed
  __syncthreads();
  int gidx = 0;                         // ring entry being consumed
  auto entry_done = [&]() {
    fetch_wait<(AHEAD - 1) * FI>();     // the next entry has landed: only the fetches issued after it may be outstanding
    __syncthreads();                    // ... for every wave, and every wave is done with this entry's slot
    ++gidx;
  };
  Work c = work_of(entry_of(0));
  for (int ord = 0; c.valid; ++ord) {
    const Entry next = entry_of(ord + 1);   // requested now, needed when this item is done (as a Work it took 6 registers more)
    // -- entry 0: query operands; per-lane row data
    fetch_next(gidx + AHEAD);
    bf16x8 qf[CB][DK];
#pragma unroll
    for (int d = 0; d < DK; ++d) qf[0][d] = ((const bf16x8*)ring[gidx & (NBUF - 1)])[wave * TV4 + d * 64 + lane];
    if (SEQ) {   // (each wave keeps and re-reads its own block only: no barrier needed for it)
#pragma unroll
      for (int d = 0; d < DK; ++d) ((bf16x8*)q_keep)[wave * TV4 + d * 64 + lane] = qf[0][d];
    }
    int row[CB], qpos[CB];
    row[0] = (c.yb * NW + wave) * 16 + col;
    {
      const int i = order.token(row[0]);
      qpos[0] = i < c.n ? c.L + i : -1;
    }
    int wmin = qpos[0] >= 0 ? qpos[0] : 0x7FFFFFFF;   // lowest position among this wave's live rows (-1: none, it only fetches)
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) wmin = min(wmin, __shfl_xor(wmin, off));
    wmin = FULL || (c.yb * NW + wave) * 16 < c.n * order.group ? __builtin_amdgcn_readfirstlane(wmin) : -1;
    float m[CB] = {-INFINITY}, l[CB] = {0.f}, sm[CB] = {-INFINITY}, sl[CB] = {0.f};
    f32x4 acc[CB][DB], sacc[CB][DB];
    float tm = -INFINITY, tl = 0.f;   // SEQ: running fold of finished supers
    f32x4 tacc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      acc[0][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
      sacc[0][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
      tacc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    entry_done();
    // -- one entry per step.  A wave without live rows only fetches, in a loop of its own: as a branch around the masked step it
    // changed the registers of the loop below (whole sequences 232 -> 216, others 200 -> 183).
    if (!FULL && wmin < 0) {
      for (int j = 0; j < c.n_steps; ++j) {
        fetch_next(gidx + AHEAD);
        entry_done();
      }
    } else for (int j = 0; j < c.n_steps; ++j) {
      fetch_next(gidx + AHEAD);
      const int k0 = c.k_lo + j * STEP;
      const uint4* sk = &ring[gidx & (NBUF - 1)][0];
      const uint16_t* sv = (const uint16_t*)&ring[gidx & (NBUF - 1)][4 * TV4];
      if (SEQ) {
#pragma unroll
        for (int d = 0; d < DK; ++d) qf[0][d] = ((const bf16x8*)q_keep)[wave * TV4 + d * 64 + lane];
      }
      const bool first = SUPER && FOLD ? (j & 3) == 0 : j == 0;   // the chunk partial is empty
      if (k0 + STEP - 1 <= wmin)                               // wave-uniform
        softmax_step<HD, CB, false>(sk, sv, k0, c.k_hi, lane, scale_log2, qf, qpos, m, l, acc, first);
      else
        softmax_step<HD, CB, true>(sk, sv, k0, c.k_hi, lane, scale_log2, qf, qpos, m, l, acc, first);
      if (SUPER && FOLD && ((j & 3) == 3 || j + 1 == c.n_steps)) {
        // a chunk is complete: fold it into the running super partial and start the next one afresh
        if ((SEQ ? (j & 31) : j) < 4) {
          sm[0] = m[0];
          sl[0] = l[0];
#pragma unroll
          for (int d = 0; d < DB; ++d) sacc[0][d] = acc[0][d];
        } else {
          fold<DB>(sm[0], sl[0], sacc[0], m[0], l[0], acc[0]);
        }
        m[0] = -INFINITY;
        l[0] = 0.f;
#pragma unroll
        for (int d = 0; d < DB; ++d) acc[0][d] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (SEQ && ((j & 31) == 31 || j + 1 == c.n_steps)) {
          // a super is complete as well: the same fold one level up
          if (j < 32) {
            tm = sm[0];
            tl = sl[0];
#pragma unroll
            for (int d = 0; d < DB; ++d) tacc[d] = sacc[0][d];
          } else {
            fold<DB>(tm, tl, tacc, sm[0], sl[0], sacc[0]);
          }
        }
      }
      entry_done();
    }
    // -- partial of this unit for every row that reaches into it
    if (SEQ) {
      if (qpos[0] >= 0) store_output<HD>(attn_out, d_attn, c.base, c.kvh, order, row[0], g, tacc, tl);
    } else if (SUPER && attn_out) {   // one unit per sequence: no partial, no merge pass
      if (qpos[0] >= 0)
        store_output<HD>(attn_out, d_attn, c.base, c.kvh, order, row[0], g, FOLD ? sacc[0] : acc[0], FOLD ? sl[0] : l[0]);
    } else if (qpos[0] >= c.k_lo) {
      const size_t prow = (((size_t)c.s * n_kv_heads + c.kvh) * n_units + c.unit) * r_pad + row[0];
      float* pa = part_acc + prow * HD;
#pragma unroll
      for (int d = 0; d < DB; ++d) *(f32x4*)(pa + d * 16 + g * 4) = SUPER && FOLD ? sacc[0][d] : acc[0][d];
      if (g == 0)
        *(float2*)(part_ml + prow * 2) = SUPER && FOLD ? make_float2(sm[0], sl[0]) : make_float2(m[0], l[0]);
    }
    c = work_of(next);
  }
  fetch_wait<0>();                      // the dummy fetches too
}

// One online-softmax step of a wave that has the 64 keys from k0 in registers, for one block of 16 query rows.  next_k and next_v
// request what follows into the same registers, each as soon as they are free.
// A lane takes V 16 bytes at a time: the keys of group g of TWO neighbouring features.  MFMA row c of product h of block
// pair p is then feature (2 p + c / 8) * 16 + 2 (c % 8) + h, and the lane ends up with 8 consecutive features of its row:
// (2 p + g / 2) * 16 + (g % 2) * 8 + 2 e + h for e = 0 .. 3.  Which row of the product a feature has does not touch its sum.
template <int HD, class NextK, class NextV>
__device__ __forceinline__ void register_step(bf16x8 (&kb)[4][HD / 32], u32x4 (&vb)[4][HD / 32], const bf16x8 (&qf)[HD / 32], int k0, int k_hi,
                                              int g, int qpos, int wmin, float scale_log2, float& m, float& l, f32x4 (&acc)[HD / 16],
                                              bool first, NextK next_k, NextV next_v) {
  constexpr int DK = HD / 32, DB = HD / 16;
  f32x4 sc[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int d = 0; d < DK; ++d)
      sc[b] = mfma16(kb[b][d], qf[d], d == 0 ? (f32x4){0.f, 0.f, 0.f, 0.f} : sc[b]);
  next_k();
  u32x4 pf[2];
  const bool inner = k0 + STEP - 1 <= wmin;                                // wave-uniform
  if (inner) softmax_update<DB, false>(sc, k0, g, qpos, scale_log2, m, l, acc, pf, first);
  else softmax_update<DB, true>(sc, k0, g, qpos, scale_log2, m, l, acc, pf, first);
  if (!inner) {
    // slots at or beyond k_hi hold stale, never-written or foreign data: zero, so that 0 * garbage is no NaN
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int kp = k0 + b * 16 + g * 4;
#pragma unroll
      for (int d = 0; d < DB / 2; ++d) {
        u32x4& v = vb[b][d];
        if (kp + 0 >= k_hi) v[0] &= 0xFFFF0000u, v[2] &= 0xFFFF0000u;
        if (kp + 1 >= k_hi) v[0] &= 0x0000FFFFu, v[2] &= 0x0000FFFFu;
        if (kp + 2 >= k_hi) v[1] &= 0xFFFF0000u, v[3] &= 0xFFFF0000u;
        if (kp + 3 >= k_hi) v[1] &= 0x0000FFFFu, v[3] &= 0x0000FFFFu;
      }
    }
  }
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const u32x4 x = vb[2 * kk][d / 2], y = vb[2 * kk + 1][d / 2];
      const u32x4 v = d % 2 == 0 ? (u32x4){x[0], x[1], y[0], y[1]} : (u32x4){x[2], x[3], y[2], y[3]};
      acc[d] = mfma16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pf[kk]), acc[d]);
    }
  next_v();
}

// 16 keys of K, or of V as register_step wants them: tile `tile` (in 16-byte units) of a plane.  NT: past the caches.
template <int DK, bool NT>
__device__ __forceinline__ void load_k_tile(bf16x8 (&kb)[DK], const bf16x8* __restrict__ plane, size_t tile, int lane) {
#pragma unroll
  for (int d = 0; d < DK; ++d) kb[d] = NT ? __builtin_nontemporal_load(plane + tile + lane + d * 64) : plane[tile + lane + d * 64];
}
template <int DK, bool NT>
__device__ __forceinline__ void load_v_tile(u32x4 (&vb)[DK], const u32x4* __restrict__ plane, size_t tile, int col, int g) {
  const u32x4* p = plane + tile + ((col >> 3) * 4 + g) * 8 + (col & 7);
#pragma unroll
  for (int d = 0; d < DK; ++d) vb[d] = NT ? __builtin_nontemporal_load(p + d * 64) : p[d * 64];
}

// Contexts within one super, for few sequences or few query rows per (sequence, kv head): a workgroup of 4 waves takes ONE
// block of 16 query rows, wave w walking chunks w and w + 4 on its own - K and V operands straight from global memory into registers, two
// steps ahead, no ring and no barrier - and the chunk partials are folded through LDS in the schedule's order.  What
// bounds such a call is the latency of one fetch after the other: four waves in a row of steps each put a whole super's
// first 512 keys in flight at once.  The K and V of a (sequence, kv head) are fetched once per row block (from L2 after
// the first), so it is used while the row blocks are few (see attention_mode).
// items == nullptr: item t is of sequence t / per_item (no list to wait for).
template <int HD>
__device__ __forceinline__ void attention_split(
    const uint16_t* __restrict__ q, const bf16x8* __restrict__ k_plane, const u32x4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_len, const int32_t* __restrict__ seq_n,
    const int4* __restrict__ items, const int32_t* __restrict__ item_count, int num_seqs, int n_kv_heads, RowOrder order,
    int r_pad, int max_blocks_per_seq, float scale_log2, uint16_t* __restrict__ attn_out, int d_attn) {
  constexpr int DK = HD / 32, DB = HD / 16, TV4 = HD * 2, PER = SUPER_KEYS / CHUNK, NW = 4, SPC = CHUNK / STEP;
  static_assert(PER == 2 * NW, "two chunks of a super per wave");
  __shared__ f32x4 fold_acc[PER][DB * 64];
  __shared__ float2 fold_ml[PER][16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, g = lane >> 4;
  const int row_blocks = r_pad / 16, per_item = n_kv_heads * row_blocks;
  const int total = (items ? *item_count : num_seqs) * per_item;
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    const int it = t / per_item, rem = t - it * per_item;
    const int s = items ? items[it].x : it;
    const int rb = rem % row_blocks, kvh = rem / row_blocks;
    // requested before the length is known (clamped to the table, not yet to the sequence): lanes 0 .. 15 the blocks of
    // the wave's first chunk, 16 .. 31 those of its second
    const int my_blk = (wave + (g & 1) * NW) * (CHUNK / 16) + col;
    const int raw = block_table[(size_t)s * max_blocks_per_seq + min(my_blk, max_blocks_per_seq - 1)];
    bf16x8 qf[DK];
    const uint16_t* qb = q + ((size_t)s * n_kv_heads + kvh) * r_pad * HD + (size_t)rb * DK * 512;
#pragma unroll
    for (int d = 0; d < DK; ++d) qf[d] = *(const bf16x8*)(qb + d * 512 + lane * 8);
    const int L = seq_len[s], tag = seq_n[s], n = tag_rows(tag);
    const int row = rb * 16 + col, i = order.token(row);
    const int qpos = L >= 0 && i < n ? L + i : -1;
    int wmax = qpos, wmin = qpos >= 0 ? qpos : 0x7FFFFFFF;   // highest and lowest position among the block's live rows
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      wmax = max(wmax, __shfl_xor(wmax, off));
      wmin = min(wmin, __shfl_xor(wmin, off));
    }
    wmax = __builtin_amdgcn_readfirstlane(wmax);
    wmin = __builtin_amdgcn_readfirstlane(wmin);
    const int k_hi = wmax + 1;                                             // exclusive; at most SUPER_KEYS
    const int chunks = (k_hi + CHUNK - 1) / CHUNK;                         // chunks any row looks into (0: no live row)
    if (wave < chunks) {
      // this wave's steps: those of chunk `wave`, then those of chunk `wave` + 4
      auto steps_of = [&](int c) { return c < chunks ? (min(k_hi - c * CHUNK, CHUNK) + STEP - 1) / STEP : 0; };
      const int steps = steps_of(wave) + steps_of(wave + NW);
      const int last_blk = (k_hi - 1) >> 4;
      // blocks past the last needed one: the table may hold anything there, and the steps' last blocks are masked; the
      // sequence's first block stands in for them
      const int safe_id = block_table[(size_t)s * max_blocks_per_seq];
      const int ids = my_blk <= last_blk ? raw : safe_id;
      bf16x8 ka[4][DK], kc[4][DK];
      u32x4 va[4][DK], vc[4][DK];
      auto tile_of = [&](int u, int b) {   // (a step past the wave's last one: the last one once more)
        const int id = __builtin_amdgcn_readlane(ids, min(u, steps - 1) * 4 + b);
        return ((size_t)id * n_kv_heads + kvh) * TV4;
      };
      auto load_k = [&](bf16x8(&kb)[4][DK], int u) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b) load_k_tile<DK, false>(kb[b], k_plane, tile_of(u, b), lane);
      };
      auto load_v = [&](u32x4(&vb)[4][DK], int u) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b) load_v_tile<DK, false>(vb[b], v_plane, tile_of(u, b), col, g);
      };
      float m = -INFINITY, l = 0.f;
      f32x4 acc[DB];
#pragma unroll
      for (int d = 0; d < DB; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
      auto step = [&](int u, bf16x8(&kb)[4][DK], u32x4(&vb)[4][DK]) __attribute__((always_inline)) {
        const int c = wave + (u / SPC) * NW, k0 = c * CHUNK + (u % SPC) * STEP;
        register_step<HD>(kb, vb, qf, k0, k_hi, g, qpos, wmin, scale_log2, m, l, acc, u % SPC == 0,
                          [&]() __attribute__((always_inline)) { load_k(kb, u + 2); }, [&]() __attribute__((always_inline)) { load_v(vb, u + 2); });
        if (u % SPC == SPC - 1 || u + 1 == steps) {                        // the chunk is complete
#pragma unroll
          for (int d = 0; d < DB; ++d) {
            fold_acc[c][d * 64 + lane] = acc[d];
            acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
          }
          if (g == 0) fold_ml[c][col] = make_float2(m, l);
          m = -INFINITY;
          l = 0.f;
        }
      };
      load_k(ka, 0);
      load_v(va, 0);
      load_k(kc, 1);
      load_v(vc, 1);
      for (int u = 0; u < steps; u += 2) {
        step(u, ka, va);
        if (u + 1 < steps) step(u + 1, kc, vc);
      }
    }
    __syncthreads();
    // every thread folds the chunks of eight features of one row: chunk 0, 1, 2, ... as in the other kernels
    if (wave < DB / 2 && qpos >= 0) {
      float2 ml = fold_ml[0][col];
      float M = ml.x, Ls = ml.y;
      f32x4 A[2] = {fold_acc[0][2 * wave * 64 + lane], fold_acc[0][(2 * wave + 1) * 64 + lane]};
      for (int c = 1; c < chunks; ++c) {
        ml = fold_ml[c][col];
        const f32x4 part[2] = {fold_acc[c][2 * wave * 64 + lane], fold_acc[c][(2 * wave + 1) * 64 + lane]};
        fold<2>(M, Ls, A, ml.x, ml.y, part);
      }
      const int f = (2 * wave + g / 2) * 16 + (g & 1) * 8;                 // the first of the lane's 8 features
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = pack2_bf16(A[0][e] / Ls, A[1][e] / Ls);
      *(u32x4*)(attn_out + pk_off(tag_base(tag) + i, (kvh * order.group + order.head(row)) * HD + f, d_attn)) = o;
    }
    __syncthreads();        // the partials are read before the next item's are written
  }
}

template <int HD>
__global__ __launch_bounds__(256) void attention_split_kernel(
    const uint16_t* __restrict__ q, const bf16x8* __restrict__ k_plane, const u32x4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_len, const int32_t* __restrict__ seq_n,
    const int4* __restrict__ items, const int32_t* __restrict__ item_count, int num_seqs, int n_kv_heads, RowOrder order,
    int r_pad, int max_blocks_per_seq, float scale_log2, uint16_t* __restrict__ attn_out, int d_attn) {
  attention_split<HD>(q, k_plane, v_plane, block_table, seq_len, seq_n, items, item_count, num_seqs, n_kv_heads, order, r_pad,
                      max_blocks_per_seq, scale_log2, attn_out, d_attn);
}

// One block of 16 query rows per (sequence, kv head), as in a decode step: a wave per chunk, and the merge pass for the sequences
// of several (the others' rows are written here).  The waves of the launch deal the plan's list among them, longest chunks first and
// neighbours on different CUs, and keep K and V of two steps on their way, straight to registers and across the end of an item: no
// ring, no barrier.  (attention_split_kernel, a workgroup per sequence and kv head, waits for its longest one; super items leave a
// launch's last round with few of them.  Where it is taken and what it takes against those: wave_use, in api.hip.)
// What bounds it is the memory where the waves walk several chunks each - 64 sequences of 1000 keys, 262 MB of K and V in 49 us, 5.4
// TB/s - and the way of a wave's first tiles where they have one or two: 8 x 1900, 62 MB in 15 us, 4.1 TB/s, 43 % of the waves' cycles
// waiting.
// (Folding by the wave that finishes a row's last chunk, partials through agent-scope stores and a counter, takes
// as long as the merge launch that it saves.  Requests past an item's last step repeat one tile: as whole steps they took 6 - 60 us.
// Within one super a workgroup of 8 waves, one per chunk, folded through LDS: 1.2 - 1.4 times the split kernel's time, for the
// registers of 8 waves hold one step of K and V each, not two.)
template <int HD>
__device__ __forceinline__ void attention_waves(
    const uint16_t* __restrict__ q, const bf16x8* __restrict__ k_plane, const u32x4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int4* __restrict__ items, const int32_t* __restrict__ item_count, int n_kv_heads,
    RowOrder order, int max_blocks_per_seq, int n_units, int part_rows, int max_items, float scale_log2,
    float* __restrict__ part_acc, float* __restrict__ part_ml, uint16_t* __restrict__ attn_out, int d_attn) {
  constexpr int DK = HD / 32, DB = HD / 16, TV4 = HD * 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, g = lane >> 4;
  const int stride = 4 * (int)gridDim.x;
  struct Item {
    int s, kvh, L, tag, k_lo, k_hi, steps, wmin, qpos, raw;
    bf16x8 qf[DK];
  };
  // An item's share of the list entry `su`; what it needs from memory is requested, not waited for.  steps = 0: nothing for
  // these rows in this chunk.
  auto open = [&](Item& x, int t, const int4 su) __attribute__((always_inline)) {
    x.kvh = t % n_kv_heads, x.s = su.x, x.L = su.z, x.tag = su.w, x.k_lo = su.y * CHUNK;
    x.raw = block_table[(size_t)x.s * max_blocks_per_seq + min(x.k_lo / 16 + col, max_blocks_per_seq - 1)];
    const uint16_t* qb = q + ((size_t)x.s * n_kv_heads + x.kvh) * 16 * HD;
#pragma unroll
    for (int d = 0; d < DK; ++d) x.qf[d] = *(const bf16x8*)(qb + d * 512 + lane * 8);
    const int i = order.token(col);
    x.qpos = i < tag_rows(x.tag) ? x.L + i : -1;
    int wmax = x.qpos, wmin = x.qpos >= 0 ? x.qpos : 0x7FFFFFFF;   // highest and lowest position among the block's live rows
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      wmax = max(wmax, __shfl_xor(wmax, off));
      wmin = min(wmin, __shfl_xor(wmin, off));
    }
    x.wmin = __builtin_amdgcn_readfirstlane(wmin);
    x.k_hi = min(__builtin_amdgcn_readfirstlane(wmax) + 1, x.k_lo + CHUNK);
    x.steps = max(0, (x.k_hi - x.k_lo + STEP - 1) / STEP);
  };
  // The tile of step u, block b of the item.  Blocks past the last needed one (the table may hold anything there): the chunk's
  // first; steps past the last one: the last tile, over and over.
  auto tile_of = [&](const Item& x, int u, int b) __attribute__((always_inline)) {
    const int at = u < x.steps ? u * 4 + b : x.steps * 4 - 1;
    return ((size_t)__builtin_amdgcn_readlane(x.raw, x.k_lo / 16 + at <= (x.k_hi - 1) / 16 ? at : 0) * n_kv_heads + x.kvh) * TV4;
  };
  int t = wave * (int)gridDim.x + (int)blockIdx.x;
  auto entry = [&](int at) { return items[min(at / n_kv_heads, max_items - 1)]; };   // (past the list: an entry that is not used)
  int4 su = entry(t);
  const int total = *item_count * n_kv_heads;
  // the next item that has steps, from t on (`su` is its entry, requested one item earlier)
  auto next = [&](Item& x) __attribute__((always_inline)) {
    x.steps = 0;
    while (t < total && x.steps == 0) {
      open(x, t, su);
      t += stride;
      su = entry(t);
    }
  };
  Item c, n;
  next(c);
  if (c.steps == 0) return;
  n.steps = 0;
  bf16x8 ka[4][DK], kc[4][DK];
  u32x4 va[4][DK], vc[4][DK];
  // (u counts from the current item's first step on; behind its last one come the next item's)
  auto tile_at = [&](int u, int b) __attribute__((always_inline)) {
    return u >= c.steps && n.steps > 0 ? tile_of(n, u - c.steps, b) : tile_of(c, u, b);
  };
  auto load_k = [&](bf16x8(&kb)[4][DK], int u) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 4; ++b) load_k_tile<DK, true>(kb[b], k_plane, tile_at(u, b), lane);
  };
  auto load_v = [&](u32x4(&vb)[4][DK], int u) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 4; ++b) load_v_tile<DK, true>(vb[b], v_plane, tile_at(u, b), col, g);
  };
  float m = -INFINITY, l = 0.f;
  f32x4 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
  int u = 0;
  // One step, and the end of the item behind its last one.  False: there is none left.
  auto step = [&](bf16x8(&kb)[4][DK], u32x4(&vb)[4][DK]) __attribute__((always_inline)) {
    register_step<HD>(kb, vb, c.qf, c.k_lo + u * STEP, c.k_hi, g, c.qpos, c.wmin, scale_log2, m, l, acc, u == 0,
                      [&]() __attribute__((always_inline)) { load_k(kb, u + 2); }, [&]() __attribute__((always_inline)) { load_v(vb, u + 2); });
    if (++u < c.steps) return true;
    const int f0 = (g / 2) * 16 + (g & 1) * 8;                             // the lane's 8 features of block pair p: f0 + 32 p
    if (c.L + tag_rows(c.tag) <= CHUNK) {                                  // the sequence's only chunk: no merge pass over its rows
      if (c.qpos >= 0) {
#pragma unroll
        for (int p = 0; p < DB / 2; ++p) {
          u32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = pack2_bf16(acc[2 * p][e] / l, acc[2 * p + 1][e] / l);
          const int feature = (c.kvh * order.group + order.head(col)) * HD + f0 + 32 * p;
          *(u32x4*)(attn_out + pk_off(tag_base(c.tag) + order.token(col), feature, d_attn)) = o;
        }
      }
    } else if (c.qpos >= c.k_lo) {
      const size_t prow = (((size_t)c.s * n_kv_heads + c.kvh) * n_units + c.k_lo / CHUNK) * part_rows + col;
      float* pa = part_acc + prow * HD + f0;
#pragma unroll
      for (int p = 0; p < DB / 2; ++p) {
        *(f32x4*)(pa + 32 * p) = (f32x4){acc[2 * p][0], acc[2 * p + 1][0], acc[2 * p][1], acc[2 * p + 1][1]};
        *(f32x4*)(pa + 32 * p + 4) = (f32x4){acc[2 * p][2], acc[2 * p + 1][2], acc[2 * p][3], acc[2 * p + 1][3]};
      }
      if (g == 0) *(float2*)(part_ml + prow * 2) = make_float2(m, l);
    }
    if (n.steps == 0) return false;
    c = n;
    next(n);
    u = 0;
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (c.steps == 1 && n.steps > 0) {     // two steps ahead was beyond an item of one step, into one not known then
      load_k(kb, 1);
      load_v(vb, 1);
    }
    return true;
  };
  load_k(ka, 0);
  load_v(va, 0);
  next(n);
  load_k(kc, 1);
  load_v(vc, 1);
  while (step(ka, va) && step(kc, vc)) {}
}

template <int HD>
__global__ __launch_bounds__(256) void attention_wave_kernel(
    const uint16_t* __restrict__ q, const bf16x8* __restrict__ k_plane, const u32x4* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int4* __restrict__ items, const int32_t* __restrict__ item_count, int n_kv_heads,
    RowOrder order, int max_blocks_per_seq, int n_units, int part_rows, int max_items, float scale_log2,
    float* __restrict__ part_acc, float* __restrict__ part_ml, uint16_t* __restrict__ attn_out, int d_attn) {
  attention_waves<HD>(q, k_plane, v_plane, block_table, items, item_count, n_kv_heads, order, max_blocks_per_seq, n_units, part_rows,
                      max_items, scale_log2, part_acc, part_ml, attn_out, d_attn);
}

// The same, or what the call runs otherwise - a workgroup per (sequence, kv head) where contexts are within one super, super items
// beyond - as the plan kernel has decided from the lengths (*by_waves): both in one launch, for one that leaves at once takes 4 us.
template <int HD, bool SPLIT>
__global__ __launch_bounds__(256) void attention_choice_kernel(
    const uint16_t* __restrict__ q, const void* __restrict__ k_plane, const void* __restrict__ v_plane,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ seq_len, const int32_t* __restrict__ seq_n,
    const int4* __restrict__ items, const int32_t* __restrict__ item_count, int32_t* __restrict__ queue, int num_seqs, int n_kv_heads,
    RowOrder order, int max_blocks_per_seq, int n_units, int part_rows, float scale_log2, float* __restrict__ part_acc,
    float* __restrict__ part_ml, uint16_t* __restrict__ attn_out, int d_attn, const int32_t* __restrict__ by_waves) {
  if (*by_waves)
    attention_waves<HD>(q, (const bf16x8*)k_plane, (const u32x4*)v_plane, block_table, items, item_count, n_kv_heads, order,
                        max_blocks_per_seq, n_units, part_rows, num_seqs * n_units, scale_log2, part_acc, part_ml, attn_out, d_attn);
  else if constexpr (SPLIT)
    attention_split<HD>(q, (const bf16x8*)k_plane, (const u32x4*)v_plane, block_table, seq_len, seq_n, nullptr, nullptr, num_seqs,
                        n_kv_heads, order, 16, max_blocks_per_seq, scale_log2, attn_out, d_attn);
  else
    attention_items<HD, 1, 4, true, 4>(q, (const uint4*)k_plane, (const uint4*)v_plane, block_table, items, item_count, queue, n_kv_heads,
                                       order, 16, 1, max_blocks_per_seq, n_units, part_rows, scale_log2, part_acc, part_ml, nullptr, d_attn);
}

// The work items of a call: every (sequence, unit) pair that holds keys, as (s, unit, L, seq_tag), sorted
// by the number of 64-key steps it takes, longest first (the attention kernels deal them out in that
// order, which keeps the tail of a launch short); and the per-layer queue counters.  The order
// inside a class of equal length is whatever the slot counter gives: it decides only which
// workgroup computes an item, never a bit of the result.  One workgroup; runs once per call.
//
// seq_unit_keys != 0: the call may run with whole sequences as items (one unit of seq_unit_keys keys
// per sequence) if they deal out evenly enough over seq_grid workgroups (seq_per_item workgroups per
// item, dealt as the stream kernel deals them); the kernel lists them, adds up every workgroup's
// entries, and keeps that list (*seq_mode = 1) if the busiest workgroup has at most 5 % more than the
// average - else (*seq_mode = 0) it lists the units of unit_keys keys as usual.  The choice moves
// work between kernels that compute the same bits.
//
// wave_rows != 0: the call may run a wave per chunk instead of what it runs otherwise (attention_choice_kernel on seq_grid
// workgroups, seq_per_item per item), with partials of wave_rows query rows; *seq_mode = 1 if it does.
// or_split: instead of the split kernel, if no wave gets a second chunk.  Else instead of supers: these take as long as the busiest
// workgroup, dealt as above (1.3 us per step of 64 keys), the waves as long as all steps at the rate of the memory (1.5 us per step
// and workgroup) or a wave's chunks one after the other (3.9 us a step), whichever is more, and their partials; both the starts and
// merge passes that were measured (8 kv heads, head dimension 128).  Over 223 calls of 8 - 48 sequences and 1 - 4 tokens, of 2100 - 16000
// keys, the one chosen took 0.3 % longer than the better one on average, 7 % at most; always the waves 3.5 %, always the supers 9.5 %.
__global__ __launch_bounds__(256) void attention_plan_kernel(const int32_t* __restrict__ seq_len,
                                                             const int32_t* __restrict__ seq_n, int num_seqs,
                                                             int unit_keys, int seq_unit_keys, int wave_rows,
                                                             bool or_split, int seq_per_item, int seq_grid, int4* __restrict__ items,
                                                             int32_t* __restrict__ item_count,
                                                             int32_t* __restrict__ queues, int n_layers,
                                                             int32_t* __restrict__ seq_mode) {
  // classes: an item's steps in units of class_steps, 1 .. nb <= MAXB (class_steps is 1 unless a unit is a whole sequence)
  constexpr int MAXB = SUPER_KEYS / STEP;
  __shared__ int count[MAXB + 1], cursor[MAXB + 1];
  __shared__ int n_items, n_chunks;
  __shared__ unsigned long long load_sum;
  __shared__ int load_max;
  for (int l = threadIdx.x; l < n_layers; l += 256) queues[l] = 0;
  auto list_items = [&](const int unit, const int class_steps) {
    const int nb = (unit / STEP + class_steps - 1) / class_steps;
    auto class_of = [&](int keys, int u) {
      return ((min(keys, (u + 1) * unit) - u * unit + STEP - 1) / STEP + class_steps - 1) / class_steps;
    };
    if (threadIdx.x <= MAXB) count[threadIdx.x] = 0;
    __syncthreads();
    for (int s = threadIdx.x; s < num_seqs; s += 256) {
      if (seq_len[s] < 0) continue;
      const int keys = seq_len[s] + tag_rows(seq_n[s]);      // positions 0 .. keys-1 are attended to
      const int full = keys / unit;
      if (full) atomicAdd(&count[nb], full);
      if (keys % unit) atomicAdd(&count[class_of(keys, full)], 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int at = 0;
      for (int c = nb; c >= 1; --c) {                        // longest class first
        cursor[c] = at;
        at += count[c];
      }
      n_items = at;
      *item_count = at;
    }
    __syncthreads();
    for (int s = threadIdx.x; s < num_seqs; s += 256) {
      if (seq_len[s] < 0) continue;
      const int L = seq_len[s], tag = seq_n[s], keys = L + tag_rows(tag);
      const int units = (keys + unit - 1) / unit;
      for (int u = 0; u < units; ++u) items[atomicAdd(&cursor[class_of(keys, u)], 1)] = make_int4(s, u, L, tag);
    }
    __syncthreads();                                         // the list is complete (and visible to this workgroup)
  };
  // load_sum and load_max: what the workgroups of a launch walk if the listed items of `unit` keys are dealt to them in turn, rounds
  // alternating direction - steps, and `extra` per item.  (A row group of a partly filled window may take fewer steps, or none.  With
  // those counted, units were taken more often and were no better: of 88 partly filled calls of 16 - 128 sequences, windows of 48 - 128, 42
  // slower, by up to 37 %, and 7 faster, by up to 9 %.)
  auto deal = [&](const int unit, const int extra) {
    if (threadIdx.x == 0) {
      load_sum = 0;
      load_max = 0;
    }
    __syncthreads();
    const int total = n_items * seq_per_item;
    for (int w = threadIdx.x; w < seq_grid; w += 256) {
      int load = 0;
      for (int ord = 0;; ++ord) {
        const int t = ord * seq_grid + ((ord & 1) ? seq_grid - 1 - w : w);
        if (t >= total) break;
        const int4 it = items[t / seq_per_item];
        load += (min(it.z + tag_rows(it.w) - it.y * unit, unit) + STEP - 1) / STEP + extra;
      }
      atomicAdd(&load_sum, (unsigned long long)load);
      atomicMax(&load_max, load);
    }
    __syncthreads();
  };
  int mode = 0;
  if (seq_unit_keys) {
    list_items(seq_unit_keys, (seq_unit_keys / STEP + MAXB - 1) / MAXB);
    deal(seq_unit_keys, 1);
    mode = (unsigned long long)load_max * seq_grid * 100ull <= load_sum * 105ull ? 1 : 0;
    __syncthreads();
  }
  if (!mode && !or_split) list_items(unit_keys, 1);
  if (wave_rows) {
    if (threadIdx.x == 0) n_chunks = 0;
    if (or_split) __syncthreads();
    else deal(unit_keys, 0);
    for (int s = threadIdx.x; s < num_seqs; s += 256)
      if (seq_len[s] >= 0) atomicAdd(&n_chunks, (seq_len[s] + tag_rows(seq_n[s]) + CHUNK - 1) / CHUNK);
    __syncthreads();
    const int chunks = n_chunks * seq_per_item, rounds = (chunks + 4 * seq_grid - 1) / (4 * seq_grid);
    const float supers_us = 4.f + 1.3f * (float)load_max;
    const float waves_us = 9.f + fmaxf(1.5f * (float)load_sum / (float)seq_grid, 3.9f * (CHUNK / STEP) * (float)rounds) +
                           2e-4f * (float)wave_rows * (float)chunks;
    mode = or_split ? rounds <= 1 : waves_us < supers_us;
    __syncthreads();
    if (mode) list_items(CHUNK, 1);
  }
  if (threadIdx.x == 0) *seq_mode = mode;
}

// Fold the partials of every query row (chunks inside a super left to right, then the supers
// left to right) and write the normalised output, bf16, into the tile layout of the
// O-projection's activation operand.  One thread per (row, 4 features).  Chunk partials: sequences of up to done_keys keys have
// their output already, and *seq_mode == 0 (where it is given) says that the call did not run a wave per chunk after all: all have
// it (SPLIT), or supers' partials.
template <int HD, bool SUPER, bool EARLY = false, bool SPLIT = false>
__global__ void attention_merge_kernel(const float* __restrict__ part_acc, const float* __restrict__ part_ml,
                                       const int32_t* __restrict__ seq_len, const int32_t* __restrict__ seq_n,
                                       int n_kv_heads, RowOrder order, int window, int r_pad, int n_units, int d_attn,
                                       uint16_t* __restrict__ out, const int32_t* __restrict__ seq_mode, int done_keys) {
  if (SUPER && seq_mode && *seq_mode) return;       // the attention kernel took whole sequences and wrote the output itself
  if (SPLIT && *seq_mode == 0) return;
  constexpr int QUADS = HD / 4;
  const int quad = threadIdx.x % QUADS;
  const int at = blockIdx.y * (blockDim.x / QUADS) + threadIdx.x / QUADS;   // (pairs can outnumber what grid.y allows)
  const int s = blockIdx.x / n_kv_heads, kvh = blockIdx.x % n_kv_heads;
  if (at >= order.group * window) return;
  // (neighbouring threads take neighbouring tokens of one head, as the output lies; the partials' rows are 512 bytes each anyway)
  const int i = at % window, hq = kvh * order.group + at / window, r = order.row(i, at / window);
  const size_t base = ((size_t)s * n_kv_heads + kvh) * n_units;
  auto slot_ml = [&](int u) { return *(const float2*)(part_ml + ((base + u) * r_pad + r) * 2); };
  auto slot_acc = [&](int u) { return *(const f32x4*)(part_acc + ((base + u) * r_pad + r) * HD + quad * 4); };
  // EARLY: the first partials are requested together with the length that says which of them there are (a round trip less, 1.4 us a
  // layer behind attention_wave_kernel; with 128 rows each the ones too many cost 1 us).
  constexpr int U = SUPER ? 1 : 4;
  float2 ml[U];
  f32x4 acc[U];
  if (EARLY) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ml[u] = slot_ml(min(u, n_units - 1));
      acc[u] = slot_acc(min(u, n_units - 1));
    }
  }
  const int L = seq_len[s], tag = seq_n[s];
  if (L < 0 || i >= tag_rows(tag)) return;   // no such row, or one that prepare_kernel has given zeros
  const bool by_super = SUPER || (EARLY && seq_mode && *seq_mode == 0);
  if (!by_super && L + tag_rows(tag) <= done_keys) return;
  uint2* dst = (uint2*)(out + pk_off(tag_base(tag) + i, hq * HD + quad * 4, d_attn));
  float M, Ls;
  f32x4 A[1];
  if (by_super) {
    const int last = (L + i) / SUPER_KEYS;
    float2 m2 = slot_ml(0);
    M = m2.x;
    Ls = m2.y;
    A[0] = slot_acc(0);
    for (int u = 1; u <= last; ++u) {
      m2 = slot_ml(u);
      const f32x4 B[1] = {slot_acc(u)};
      fold<1>(M, Ls, A, m2.x, m2.y, B);
    }
  } else {
    // The partials of half a super are requested together (those past the last one clamped to it): folding them as they
    // come is one dependent round trip after the other.
    constexpr int PER = SUPER_KEYS / CHUNK;
    const int last = (L + i) / CHUNK;
    M = 0.f;
    Ls = 0.f;
    A[0] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m2 = 0.f, l2 = 0.f;
    f32x4 a2[1] = {(f32x4){0.f, 0.f, 0.f, 0.f}};
    for (int c0 = 0; c0 <= last; c0 += U) {
      if (!EARLY || c0 > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ml[u] = slot_ml(min(c0 + u, last));
          acc[u] = slot_acc(min(c0 + u, last));
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const f32x4 B[1] = {acc[u]};
        if (u == 0 && c0 % PER == 0) m2 = ml[0].x, l2 = ml[0].y, a2[0] = acc[0];
        else if (c0 + u <= last) fold<1>(m2, l2, a2, ml[u].x, ml[u].y, B);
      }
      if (c0 % PER == PER - U || c0 + U > last) {   // the super is complete
        if (c0 < PER) M = m2, Ls = l2, A[0] = a2[0];
        else fold<1>(M, Ls, A, m2, l2, a2);
      }
    }
  }
  uint2 o;
  o.x = pack2_bf16(A[0][0] / Ls, A[0][1] / Ls);
  o.y = pack2_bf16(A[0][2] / Ls, A[0][3] / Ls);
  *dst = o;
}

// Entries of attention_kernel's ring for chunk items: two at head dimension 128, so that a CU holds two workgroups and one
// computes while the other waits for its item's first tiles, and the items dealt out in turn instead of by a counter whose answer is
// waited for.  us per layer less than with one workgroup, four entries and the counter: 2 row blocks, 2 sequences of up to 16000 keys
// 8.6; 4 row blocks, 8 x 1900 keys 7.8, 4 x 1900 2.1, 1 x 1900 0.9.
template <int HD>
constexpr int kChunkRing = HD == 128 ? 2 : 4;

template <int HD, int CB, int NW, bool SUPER, int NBUF = 4>
void launch_one(const llm42_model* m, int layer, const uint16_t* kp, const uint16_t* vp, const llm42_kv_cache* kv,
                int num_seqs, int window, const Workspace& ws, hipStream_t st) {
  const llm42_config& c = m->cfg;
  const float scale_log2 = (1.0f / sqrtf((float)c.head_dim)) * 1.44269504088896340736f;
  const int col_blocks = ws.r_pad / 16;
  const int y_blocks = (col_blocks + NW * CB - 1) / (NW * CB);
  // one workgroup per CU (the KV ring takes 128 KiB of LDS at head_dim 128), but no more than there can be items
  const long long max_items = (long long)num_seqs * ws.attn_units * c.n_kv_heads * y_blocks;
  const unsigned grid = (unsigned)std::min<long long>(m->num_cus * (HD == 128 ? 1 : 2) * (NBUF == 2 ? 2 : 1), max_items);
  attention_kernel<HD, CB, NW, SUPER, NBUF><<<grid, NW * 64, 0, st>>>(
      ws.q, (const uint4*)kp, (const uint4*)vp, kv->block_table, ws.attn_items, ws.attn_ctrl, ws.attn_ctrl + 1 + layer,
      c.n_kv_heads, row_order(m->group, window), ws.r_pad, y_blocks, kv->max_blocks_per_seq, ws.attn_units, scale_log2, ws.part_acc,
      ws.part_ml, SUPER && ws.attn_direct ? ws.attn : nullptr, m->d_attn);
  if (SUPER && ws.attn_direct) return;
  const int rows = m->group * window, rows_per_block = 256 / (HD / 4);
  attention_merge_kernel<HD, SUPER><<<dim3(num_seqs * c.n_kv_heads, (rows + rows_per_block - 1) / rows_per_block), 256,
                                      0, st>>>(ws.part_acc, ws.part_ml, ws.seq_len, ws.seq_n, c.n_kv_heads, row_order(m->group, window),
                                               window, ws.r_pad, ws.attn_units, m->d_attn, ws.attn,
                                               ws.attn_seq ? ws.attn_ctrl + 1 + c.n_layers : nullptr, 0);
}

// Workgroups of a stream-kernel launch: one per CU at head_dim 128 (two at 64), no more than there are items.
long long stream_grid(const llm42_model* m, int num_seqs, int units, int r_pad) {
  const long long max_items = (long long)num_seqs * units * m->cfg.n_kv_heads * ((r_pad / 16 + 7) / 8);
  return std::min<long long>(m->num_cus * (m->cfg.head_dim == 128 ? 1 : 2), max_items);
}

template <int HD, bool SUPER, bool FOLD, bool SEQ = false>
void launch_stream(const llm42_model* m, const uint16_t* kp, const uint16_t* vp, const llm42_kv_cache* kv, int num_seqs,
                   int window, const Workspace& ws, hipStream_t st) {
  const llm42_config& c = m->cfg;
  const float scale_log2 = (1.0f / sqrtf((float)c.head_dim)) * 1.44269504088896340736f;
  const int y_blocks = (ws.r_pad / 16 + 7) / 8;
  const unsigned grid = (unsigned)stream_grid(m, num_seqs, SEQ ? 1 : ws.attn_units, ws.r_pad);
  auto* const kernel = ws.full ? attention_stream_kernel<HD, SUPER, FOLD, SEQ, true> : attention_stream_kernel<HD, SUPER, FOLD, SEQ, false>;
  kernel<<<grid, 512, 0, st>>>(
      ws.q, (const uint4*)kp, (const uint4*)vp, kv->block_table, ws.attn_items, ws.attn_ctrl, c.n_kv_heads, row_order(m->group, window),
      ws.r_pad, y_blocks, kv->max_blocks_per_seq, ws.attn_units, scale_log2, ws.part_acc, ws.part_ml,
      SEQ || (SUPER && ws.attn_direct) ? ws.attn : nullptr, m->d_attn, ws.attn_seq ? ws.attn_ctrl + 1 + c.n_layers : nullptr);
  if (SEQ || (SUPER && ws.attn_direct)) return;
  const int rows = m->group * window, rows_per_block = 256 / (HD / 4);
  attention_merge_kernel<HD, SUPER><<<dim3(num_seqs * c.n_kv_heads, (rows + rows_per_block - 1) / rows_per_block), 256,
                                      0, st>>>(ws.part_acc, ws.part_ml, ws.seq_len, ws.seq_n, c.n_kv_heads, row_order(m->group, window),
                                               window, ws.r_pad, ws.attn_units, m->d_attn, ws.attn,
                                               ws.attn_seq ? ws.attn_ctrl + 1 + c.n_layers : nullptr, 0);
}

template <int HD>
void launch_split(const llm42_model* m, const uint16_t* kp, const uint16_t* vp, const llm42_kv_cache* kv, int num_seqs,
                  int window, const Workspace& ws, hipStream_t st) {
  const llm42_config& c = m->cfg;
  const float scale_log2 = (1.0f / sqrtf((float)c.head_dim)) * 1.44269504088896340736f;
  // As many workgroups as the device holds at once: one per CU at head dimension 128 (its 418 registers per wave), two at 64
  // (250 registers, 33 KiB of LDS).  One per CU there left half of each idle: 2048 workgroups' worth of work 62 us at 250
  // keys and 36 at 64, with two per CU 39 and 23.
  constexpr int kPerCu = HD == 64 ? 2 : 1;
  const unsigned grid = (unsigned)std::min<long long>((long long)kPerCu * m->num_cus, (long long)num_seqs * c.n_kv_heads * (ws.r_pad / 16));
  attention_split_kernel<HD><<<grid, 256, 0, st>>>(
      ws.q, (const bf16x8*)kp, (const u32x4*)vp, kv->block_table, ws.seq_len, ws.seq_n, ws.attn_list ? ws.attn_items : nullptr,
      ws.attn_ctrl, num_seqs, c.n_kv_heads, row_order(m->group, window), ws.r_pad, kv->max_blocks_per_seq, scale_log2, ws.attn, m->d_attn);
}

template <int HD>
void launch_waves(const llm42_model* m, int layer, const uint16_t* kp, const uint16_t* vp, const llm42_kv_cache* kv, int num_seqs,
                  int window, const Workspace& ws, hipStream_t st) {
  const llm42_config& c = m->cfg;
  const float scale_log2 = (1.0f / sqrtf((float)c.head_dim)) * 1.44269504088896340736f;
  const int rows = m->group * window, rows_per_block = 256 / (HD / 4);
  const unsigned grid = (unsigned)std::min<long long>(m->num_cus, (long long)num_seqs * ws.attn_units * c.n_kv_heads);
  const int32_t* by_waves = ws.attn_choice ? ws.attn_ctrl + 1 + c.n_layers : nullptr;
  if (by_waves) {
    auto* const kernel = ws.attn_split ? attention_choice_kernel<HD, true> : attention_choice_kernel<HD, false>;
    kernel<<<grid, 256, 0, st>>>(ws.q, kp, vp, kv->block_table, ws.seq_len, ws.seq_n, ws.attn_items, ws.attn_ctrl,
                                 ws.attn_ctrl + 1 + layer, num_seqs, c.n_kv_heads, row_order(m->group, window), kv->max_blocks_per_seq,
                                 ws.attn_units, ws.part_rows, scale_log2, ws.part_acc, ws.part_ml, ws.attn, m->d_attn, by_waves);
  } else {
    attention_wave_kernel<HD><<<grid, 256, 0, st>>>(
        ws.q, (const bf16x8*)kp, (const u32x4*)vp, kv->block_table, ws.attn_items, ws.attn_ctrl, c.n_kv_heads, row_order(m->group, window),
        kv->max_blocks_per_seq, ws.attn_units, ws.part_rows, num_seqs * ws.attn_units, scale_log2, ws.part_acc, ws.part_ml, ws.attn, m->d_attn);
  }
  auto* const merge = by_waves && ws.attn_split ? attention_merge_kernel<HD, false, true, true> : attention_merge_kernel<HD, false, true>;
  merge<<<dim3(num_seqs * c.n_kv_heads, (rows + rows_per_block - 1) / rows_per_block), 256, 0, st>>>(
      ws.part_acc, ws.part_ml, ws.seq_len, ws.seq_n, c.n_kv_heads, row_order(m->group, window), window, ws.part_rows, ws.attn_units,
      m->d_attn, ws.attn, by_waves, CHUNK);
}

template <int HD>
void launch_hd(const llm42_model* m, int layer, const uint16_t* kp, const uint16_t* vp, const llm42_kv_cache* kv,
               int num_seqs, int window, const Workspace& ws, hipStream_t st) {
  const bool wide = attention_streams(m, num_seqs, ws);
  // (a call that may take whole sequences as items launches that kernel too; the plan's choice, made on the device
  // from the lengths, leaves one of the two with nothing to do)
  if constexpr (HD == 128) {
    if (ws.attn_waves || ws.attn_choice) {
      launch_waves<HD>(m, layer, kp, vp, kv, num_seqs, window, ws, st);
      return;
    }
  }
  if (ws.attn_split) {
    launch_split<HD>(m, kp, vp, kv, num_seqs, window, ws, st);
    return;
  }
  if (ws.attn_seq) launch_stream<HD, true, true, true>(m, kp, vp, kv, num_seqs, window, ws, st);
  if (ws.attn_super) {
    if (wide && ws.batch_chosen) launch_stream<HD, true, false>(m, kp, vp, kv, num_seqs, window, ws, st);
    else if (wide) launch_stream<HD, true, true>(m, kp, vp, kv, num_seqs, window, ws, st);
    else launch_one<HD, 1, 4, true>(m, layer, kp, vp, kv, num_seqs, window, ws, st);
  } else {
    if (wide) launch_stream<HD, false, true>(m, kp, vp, kv, num_seqs, window, ws, st);
    else launch_one<HD, 1, 4, false, kChunkRing<HD>>(m, layer, kp, vp, kv, num_seqs, window, ws, st);
  }
}

}  // namespace

void launch_attention_plan(const llm42_model* m, int num_seqs, int max_context, const Workspace& ws, hipStream_t st) {
  // as a whole-sequence item a unit has as many keys as the longest sequence of the call may have
  const int seq_unit_keys = ws.attn_seq ? (max_context + STEP - 1) / STEP * STEP : 0;
  const int seq_per_item = m->cfg.n_kv_heads * ((ws.r_pad / 16 + 7) / 8);
  const int unit_keys = ws.attn_choice || (!ws.attn_waves && (ws.attn_super || ws.attn_split)) ? SUPER_KEYS : CHUNK;
  const int grid = ws.attn_choice ? m->num_cus : (int)stream_grid(m, num_seqs, 1, ws.r_pad);
  attention_plan_kernel<<<1, 256, 0, st>>>(ws.seq_len, ws.seq_n, num_seqs, unit_keys, seq_unit_keys, ws.attn_choice ? ws.part_rows : 0,
                                           ws.attn_choice && ws.attn_split, seq_per_item, grid, ws.attn_items, ws.attn_ctrl,
                                           ws.attn_ctrl + 1, m->cfg.n_layers,
                                           ws.attn_ctrl + 1 + m->cfg.n_layers);
}

// 8 row blocks or more per (sequence, kv head): 8 waves of one row block each, two per SIMD, so that one wave's MFMAs run under the
// other's softmax arithmetic, as one stream per CU; fewer: 4 waves.  So do chunks while there are few of them for two workgroups a CU,
// and few per sequence: four row blocks' worth of a chunk per workgroup, K and V are fetched twice.  us per layer, 4 waves / 8
// (sequences x window behind keys, 8 kv heads, 4 query heads each):
//   up to 5 chunks  8 x 32 / 300 18.6 / 20.8, 5 x 32 / 512 18.3 / 20.4, 4 x 32 / 1000 20.4 / 21.6, 2 x 64 / 1000 21.1 / 22.8,
//                   1 x 256 / 300 20.3 / 23.5, 1 x 256 / 512 22.8 / 23.6; 6 x 32 / 1000 23.1 / 23.4, 3 x 64 / 1000 24.0 / 23.9
//   6 - 8           1 x 32 / 1900 17.8 / 18.8, 1 x 64 / 1500 20.4 / 22.1; 2 x 32 / 1900 21.8 / 20.6, 4 x 32 / 1900 25.4 / 24.7, 1 x 128 / 1900 28.8 / 26.3
//   more            1 x 32 / 4500 24.9 / 22.0, 1 x 32 / 8000 31.8 / 26.8, 2 x 32 / 3000 27.1 / 23.3, 1 x 64 / 3000 27.1 / 26.2
// Where the 8 waves' last row group is at most half full, the 4 waves fetch less: 1 x 48 / 4500 28.8 / 34.6, 3 x 48 / 1500 24.0 / 30.7.
bool attention_streams(const llm42_model* m, int num_seqs, const Workspace& ws) {
  const int blocks = ws.r_pad / 16, groups = (blocks + 3) / 4, units = ws.attn_units;
  if (blocks < 8) return false;
  if (ws.attn_super || m->cfg.head_dim != 128) return true;
  const long long items = (long long)num_seqs * units * m->cfg.n_kv_heads * groups, cus = m->num_cus;
  return items > (groups % 2 ? 2 * cus : units <= 5 ? 7 * cus / 4 : units <= 8 ? cus - 1 : 0);
}

int attention_units(bool super_mode, int max_context) {
  const int keys = super_mode ? SUPER_KEYS : CHUNK;
  return (max_context + keys - 1) / keys;
}

void launch_attention(const llm42_model* m, int layer, const llm42_kv_cache* kv, int num_seqs, int window,
                      int max_context, const Workspace& ws, hipStream_t st) {
  const llm42_config& c = m->cfg;
  const size_t plane = (size_t)kv->num_blocks * c.n_kv_heads * 16 * c.head_dim;
  const uint16_t* kp = (const uint16_t*)kv->kv_base + ((size_t)layer * 2 + 0) * plane;
  const uint16_t* vp = (const uint16_t*)kv->kv_base + ((size_t)layer * 2 + 1) * plane;
  if (c.head_dim == 128) launch_hd<128>(m, layer, kp, vp, kv, num_seqs, window, ws, st);
  else launch_hd<64>(m, layer, kp, vp, kv, num_seqs, window, ws, st);
}
