// bf16 MFMA GEMMs of the verifier pass, D[feature][token] = sum_k W[feature][k] X[token][k],
// with the layer-specific epilogues fused (rotary embedding + KV-cache write,
// residual add, SwiGLU, logits + arg-max partials): the kernels for up to 64 rows and the choice among all.
//
// Reduction schedule (what fixes the bits of every output element): one fp32
// accumulator per element, started at zero, updated by v_mfma_f32_16x16x32_bf16
// over k-tiles 0, 1, 2, ... in ascending order; the two residual projections use two such
// accumulators, one per half of K, added once at the end (kSplit below), the other GEMMs one.  The
// schedule depends on K and on the kind of GEMM only.  How many token blocks a wave owns, how many waves share a
// workgroup and how the grid is shaped are work-distribution choices that do not
// touch it, so they may change with the number of rows.
#include "gemm_parts.h"

using namespace gemm;

namespace {

// Byte offset, in an activation operand, of what lane `lane` takes of a tile of token block `block` at k-tile 0: its row's 16 bytes, or
// those of the last row that there is.  Rows that only pad are not fetched then (a line holds 8 rows): every workgroup reads all
// activations, at 32 rows twice as many bytes as its share of the weights (8B, us a decode step: 1 row 3244 -> 3141, 24 rows
// 3854 -> 3721).
__device__ __forceinline__ uint32_t row_offset(int block, int lane, int last_row, int k_tiles) {
  const int row = min(block * 16 + (lane & 15), last_row);
  return (uint32_t)(row >> 4) * (uint32_t)k_tiles * 1024u + (uint32_t)((lane >> 4) * 16 + (row & 15)) * 16u;
}

// Small-batch kernel for narrow outputs (at most 64 tokens): bound by the weight stream, with one workgroup on every CU.  A
// workgroup owns NBW blocks of 16 features over one k range (a half of a split GEMM: blockIdx.y) and all MB token blocks.
// F waves do nothing but fetch: per k-tile the NBW weight and MB activation tiles go from global memory straight into a ring
// of R rounds of CH k-tiles in LDS; the other NBW * MB waves own one 16 x 16 block each and advance it through the round in
// ascending k.  One barrier per round: behind it round r has landed, and the slot of round r - 1 is refilled.
// Two feature blocks share their activation tiles, and the two halves of a split GEMM are workgroups of their own (their
// sum is taken by the RMSNorm that follows), so a launch of as many workgroups moves half the activation bytes of the
// kernel this replaces (one block per workgroup, both halves in it): down-projection 25.2 -> 20.5 us at 16 rows,
// 27.8 -> 22.0 at 32, 33.8 -> 28.7 at 64; O-projection 10.0 -> 7.7, 11.2 -> 8.6, 12.9 -> 10.7; QKV 13.6 -> 10.3,
// 16.4 -> 14.2, 20.0 -> 17.1 (a dependent read of the weights alone takes 22, 9 and 11 us).
template <int NBW, int MB, int CH, int R, int F, class Epi>
__global__ __launch_bounds__(64 * (NBW * MB + F)) void gemm_narrow_kernel(const bf16x8* __restrict__ w,
                                                                         const bf16x8* __restrict__ x, int n_blocks,
                                                                         int k_tiles, int split, int last_row, Epi epi) {
  constexpr int ST = NBW + MB;                       // operand tiles per k-tile
  constexpr int PW = CH * ST / F;                    // tiles a fetching wave requests per round
  static_assert(CH * ST % F == 0, "the fetching waves take equal shares");
  __shared__ bf16x8 ring[R][CH * ST * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n0 = blockIdx.x * NBW;
  const int k_begin = blockIdx.y ? split : 0, k_count = blockIdx.y ? k_tiles - split : split;
  const int rounds = (k_count + CH - 1) / CH;
  if constexpr (std::is_same<Epi, StorePartialEpi>::value) epi.partial += blockIdx.y * epi.plane;
  if (wave >= NBW * MB) {
    const int fw = wave - NBW * MB;
    const uint32_t dst = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0][0];
    const bf16x8* src[PW];
    int kt[PW];
    uint32_t at[PW];
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int q = fw * PW + i, op = q % ST;
      kt[i] = q / ST;
      src[i] = (op < NBW ? w + (size_t)min(n0 + op, n_blocks - 1) * k_tiles * 64 : x) + (size_t)k_begin * 64;
      at[i] = op < NBW ? lane * 16u : row_offset(op - NBW, lane, last_row, k_tiles);
    }
    auto fetch = [&](int r) {
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const uint32_t off = (uint32_t)min(r * CH + kt[i], k_count - 1) * 1024u + at[i];
        const uint32_t d = dst + (uint32_t)(((r % R) * CH * ST + fw * PW + i) * 1024);
        if ((fw * PW + i) % ST < NBW) lds_fetch_1k<true>(src[i], off, d);
        else lds_fetch_1k(src[i], off, d);
      }
    };
    for (int r = 0; r < min(R - 1, rounds); ++r) fetch(r);
    for (int r = 0; r < rounds; ++r) {
      wait_for_rounds<R, PW>(min(R - 2, rounds - 1 - r));
      __syncthreads();
      if (r + R - 1 < rounds) fetch(r + R - 1);
    }
    return;
  }
  const int bi = wave / MB, bm = wave % MB, nb = n0 + bi, row = bm * 16 + (lane & 15);
  const typename Epi::Pre pre = epi.pre(min(nb, n_blocks - 1), lane, row, epi.row_info(row));
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int full = k_count / CH;
  for (int r = 0; r < rounds; ++r) {
    __syncthreads();
    const bf16x8* p = ring[r % R] + lane;
    if (r < full) {
      bf16x8 a[CH], b[CH];
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        a[j] = p[(j * ST + bi) * 64];
        b[j] = p[(j * ST + NBW + bm) * 64];
      }
#pragma unroll
      for (int j = 0; j < CH; ++j) acc = mfma16(a[j], b[j], acc);
    } else {
      for (int j = 0; j < k_count - r * CH; ++j) acc = mfma16(p[(j * ST + bi) * 64], p[(j * ST + NBW + bm) * 64], acc);
    }
  }
  if (nb < n_blocks) epi(nb, lane, row, acc, pre);
}

// Small-batch kernel for narrow outputs that are NOT split although few workgroups share them (the residual projections of
// the fast path): one workgroup per block of 16 features.  F waves fetch the block's weight tiles into a ring of R rounds of
// CH k-tiles in LDS, MB waves own one token block each, with its activation tiles two rounds ahead in registers.  Down-
// projection 29.9 -> 26.9 us at 32 rows and 37.2 -> 34.1 at 64 against a ring through registers and two barriers a round;
// gemm_narrow_kernel, on half the CUs here, takes 37 and 45.
template <int MB, int CH, int R, int F, class Epi>
__global__ __launch_bounds__(64 * (MB + F)) void gemm_ring_kernel(const bf16x8* __restrict__ w,
                                                                  const bf16x8* __restrict__ x, int k_tiles, int last_row, Epi epi) {
  constexpr int PW = CH / F;                         // weight tiles a fetching wave requests per round
  static_assert(CH % F == 0, "the fetching waves take equal shares");
  __shared__ bf16x8 ring[R][CH * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const bool consumer = wave < MB;
  const int nb = blockIdx.x, rounds = k_tiles / CH;  // full rounds; the rest is the tail
  const bf16x8* wbase = w + (size_t)nb * k_tiles * 64;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  typename Epi::Pre pre{};
  if (!consumer) {
    const int fw = wave - MB;
    const uint32_t dst = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0][0];
    auto fetch = [&](int r) {
#pragma unroll
      for (int i = 0; i < PW; ++i)
        lds_fetch_1k<true>(wbase, (uint32_t)((r * CH + i * F + fw) * 1024 + lane * 16), dst + (uint32_t)(((r % R) * CH + i * F + fw) * 1024));
    };
    for (int r = 0; r < min(R - 1, rounds); ++r) fetch(r);
    for (int r = 0; r < rounds; ++r) {
      wait_for_rounds<R, PW>(min(R - 2, rounds - 1 - r));
      __syncthreads();                               // round r is in LDS; everyone is done with round r - 1
      if (r + R - 1 < rounds) fetch(r + R - 1);   // into the slot of round r - 1
    }
  } else {
    const bf16x8* xp = x + row_offset(wave, lane, last_row, k_tiles) / 16;
    const int row = wave * 16 + (lane & 15);
    bf16x8 xa[CH], xb[CH];
    auto load_x = [&](bf16x8(&dst)[CH], int r) __attribute__((always_inline)) {
      const bf16x8* p = xp + (size_t)min(r, rounds - 1) * CH * 64;   // (past the last round: the last one again)
#pragma unroll
      for (int j = 0; j < CH; ++j) dst[j] = p[(size_t)j * 64];
    };
    auto body = [&](bf16x8(&cur)[CH], int r) __attribute__((always_inline)) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < CH; ++j) acc = mfma16(ring[r % R][j * 64 + lane], cur[j], acc);
      load_x(cur, r + 2);
    };
    pre = epi.pre(nb, lane, row, epi.row_info(row));
    if (rounds > 0) {
      load_x(xa, 0);
      load_x(xb, 1);
    }
    for (int r = 0; r < rounds; r += 2) {
      body(xa, r);
      if (r + 1 < rounds) body(xb, r + 1);
    }
    const bf16x8* wp = wbase + lane;                 // tail of fewer than CH tiles: tile by tile
    for (int kt = rounds * CH; kt < k_tiles; ++kt) acc = mfma16(wp[(size_t)kt * 64], xp[(size_t)kt * 64], acc);
  }
  if (consumer) epi(nb, lane, wave * 16 + (lane & 15), acc, pre);
}

// Small-batch kernel for wide outputs (at most 64 tokens): 8 waves per workgroup, every wave owns
// its own block of 16 features and streams that block's weight tiles from HBM into registers, 16
// k-tiles ahead of their use.  The activation tiles, which all 8 waves need, are fetched
// once per workgroup and shared through LDS (double buffered), which cuts the L2 traffic for
// activations by 8.  Accumulation order per output element: as stated above.  A round is 16 k-tiles
// for one or two token blocks and 8 for four (three register sets of weights then), so that the
// registers hold the accumulators, the weights in flight and a few prefetched activation operands.
// (The same kernel with 8 and 16 token blocks is slower than gemm_direct_kernel at 128 and 256 rows: a round's
// arithmetic then outlasts neither the weight stream nor the latency of its own activation fetch.)
// NBW (7 or 8) of the 8 waves own a feature block; with NBW = 7 the eighth wave only helps fetching
// activations (this makes the grid of the 8B gate/up GEMM exactly one workgroup per CU).
template <int MB, int NBW, class Epi>
__global__ __launch_bounds__(512) void gemm_xshare_kernel(const bf16x8* __restrict__ w, const bf16x8* __restrict__ x,
                                                          int n_blocks, int k_tiles, int last_row, Epi epi) {
  // A round is CH k-tiles; NSET register sets of weights: one in use, NSET - 1 in flight (16 KiB per
  // wave whatever the round length).  The round's activation tiles go through LDS, double buffered.
  constexpr int CH = MB <= 2 ? 16 : 8, NSET = 16 / CH + 1, NW = 8;
  constexpr int XT = MB * CH / NW;                   // activation tiles each wave fetches per round
  static_assert(MB * CH % NW == 0, "a round's activation tiles are dealt evenly to the waves");
  __shared__ bf16x8 xlds[2][MB * CH * 64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool owner = wave < NBW && blockIdx.x * NBW + wave < n_blocks;   // other waves only fetch activations
  const int nb = owner ? blockIdx.x * NBW + wave : 0;
  const bf16x8* wp = w + (size_t)nb * k_tiles * 64 + lane;
  const bf16x8* xp[MB];                              // this lane's share of the token blocks' first tiles
#pragma unroll
  for (int b = 0; b < MB; ++b) xp[b] = x + row_offset(b, lane, last_row, k_tiles) / 16;
  f32x4 acc[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) acc[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  bf16x8 wr[NSET][CH], xg[XT];
  const int rounds = k_tiles / CH;                   // full rounds; the rest is the tail

  // none of these loads sits behind a per-load condition (the compiler would serialise them)
  // (a round past the last one re-reads the last round's first tile CH times: loads that keep the
  // loop free of branches but fetch next to nothing from HBM)
  auto load_w = [&](bf16x8(&dst)[CH], int r) {
    const int real = r < rounds ? 1 : 0, base = min(r, rounds - 1) * CH;
#pragma unroll
    for (int j = 0; j < CH; ++j) dst[j] = __builtin_nontemporal_load(wp + (size_t)(base + j * real) * 64);
  };
  auto load_x = [&](int r) {   // tile q of the round: token block q / CH, k-tile r * CH + q % CH
#pragma unroll
    for (int i = 0; i < XT; ++i) {
      const int q = i * NW + wave;
      xg[i] = xp[i * NW / CH][(size_t)(r * CH + q % CH) * 64];
    }
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int i = 0; i < XT; ++i) xlds[buf][(i * NW + wave) * 64 + lane] = xg[i];
  };
  auto compute = [&](const bf16x8(&cur)[CH], int buf) __attribute__((always_inline)) {
    if constexpr (MB <= 2) {
#pragma unroll
      for (int j = 0; j < CH; ++j)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[b] = mfma16(cur[j], xlds[buf][(b * CH + j) * 64 + lane], acc[b]);
    } else {
      // many token blocks: the activation operands are requested from LDS PD MFMAs ahead, by hand
      // (with the registers this full, the compiler reads each operand right before its MFMA)
      constexpr int PD = 6, N = CH * MB;
      bf16x8 xq[PD + 1];
      auto operand = [&](int idx) { return xlds[buf][((idx % MB) * CH + idx / MB) * 64 + lane]; };
#pragma unroll
      for (int t = 0; t < PD; ++t) xq[t] = operand(t);
#pragma unroll
      for (int idx = 0; idx < N; ++idx) {
        if (idx + PD < N) xq[(idx + PD) % (PD + 1)] = operand(idx + PD);
        __builtin_amdgcn_sched_barrier(0);
        acc[idx % MB] = mfma16(cur[idx / MB], xq[idx % (PD + 1)], acc[idx % MB]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // what the epilogue needs from memory: requested now (hidden behind the weight stream) while the
  // registers allow it, at the end with 4 token blocks and more
  constexpr bool kEarlyPre = MB < 4;
  typename Epi::Pre pre[kEarlyPre ? MB : 1];
  if (kEarlyPre && owner) {
#pragma unroll
    for (int b = 0; b < MB; ++b) pre[b] = epi.pre(nb, lane, b * 16 + (lane & 15), epi.row_info(b * 16 + (lane & 15)));
  }
  // A round's body is free of branches: past the last round the loads re-read the last round (into
  // registers and a buffer that nothing uses any more).  The activation loads of a round are issued
  // BEFORE its weight loads: loads return in order, so the wait for the activations (they go to LDS
  // within the round) then leaves the weight loads, which are needed NSET - 1 rounds later, in flight.
  // Rounds come in groups of NSET without an exit in between (with one, the compiler moves a round's
  // weight loads down to the round that uses them, which serialises fetch and arithmetic); the last
  // rounds % NSET rounds follow as straight code.
  auto run = [&](auto own) __attribute__((always_inline)) {
    constexpr bool OWN = decltype(own)::value;
    const int last = rounds - 1;
    load_x(0);
    if (OWN) {
#pragma unroll
      for (int u = 0; u < NSET - 1; ++u) load_w(wr[u], u);
    }
    store_x(0);
    __syncthreads();
    int flip = 0;                                    // activation buffer of the current round (NSET odd)
    auto body = [&](auto uc, int rr) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      const int buf = NSET % 2 == 0 ? (u & 1) : flip;
      load_x(min(rr + 1, last));
      // the set that the previous round used up takes the round NSET - 1 ahead
      if (OWN) load_w(wr[(u + NSET - 1) % NSET], rr + NSET - 1);
      __builtin_amdgcn_sched_barrier(0);             // (left alone the compiler sinks the loads behind the round's MFMAs)
      if (OWN) compute(wr[u], buf);
      store_x(buf ^ 1);
      __syncthreads();
      flip ^= 1;
    };
    int r = 0;
    for (; r + NSET <= rounds; r += NSET) {
      body(std::integral_constant<int, 0>{}, r);
      body(std::integral_constant<int, 1>{}, r + 1);
      if constexpr (NSET > 2) body(std::integral_constant<int, 2>{}, r + 2);
    }
    if (r < rounds) body(std::integral_constant<int, 0>{}, r);
    if (r + 1 < rounds) body(std::integral_constant<int, 1>{}, r + 1);
  };
  static_assert(NSET == 2 || NSET == 3, "the groups of rounds are written out for 2 and 3 register sets");
  if (rounds > 0) {
    if (owner) run(std::true_type{});
    else run(std::false_type{});
  }
  for (int kt = rounds * CH; owner && kt < k_tiles; ++kt) {   // tail of fewer than CH tiles: tile by tile
    const bf16x8 a = wp[(size_t)kt * 64];
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[b] = mfma16(a, xp[b][(size_t)kt * 64], acc[b]);
  }
  if (owner) {
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const int row = b * 16 + (lane & 15);
      if constexpr (kEarlyPre) epi(nb, lane, row, acc[b], pre[b]);
      else epi(nb, lane, row, acc[b], epi.pre(nb, lane, row, epi.row_info(row)));
    }
  }
}

// The split of each GEMM type (part of the reduction schedule, see above).
constexpr int kSplit[GEMM_KINDS] = {1, 2, 1, 2, 1};

template <int SPLIT, class Epi>
void launch_narrow(const bf16x8* wp, const bf16x8* xp, int n_blocks, int k_tiles, int n, const Workspace& ws, const Epi& epi,
                   hipStream_t st) {
  const int split = SPLIT == 2 ? split_point(k_tiles) : k_tiles;
  if constexpr (SPLIT == 1) {
    // Unsplit with no more blocks than CUs: a workgroup for each.  QKV by gemm_narrow_kernel (3072 x 1024 at 16, 32 and 64 rows:
    // 6.7, 7.0 and 8.7 us with two blocks each, 6.3, 6.6 and 7.7 with one; 3072 x 2048: 8.4, 9.2 and 11.5 -> 7.1, 8.2 and
    // 10.0), the residual projections by gemm_ring_kernel.  With more blocks two per workgroup are the faster ones: QKV of
    // 5120 x 3072 at 64 rows 15.4 us against 20.5; down-projection of 8192 x 28672 at 32 and 64 rows 83 and 102 against 106
    // and 121 by the ring, 5120 x 13824 42 and 48 against 49 and 58.
    if (n_blocks <= ws.num_cus) {
      if constexpr (std::is_same<Epi, ResidualEpi>::value) {
        if (ws.m_pad == 32) gemm_ring_kernel<2, 16, 5, 2, Epi><<<n_blocks, 64 * 4, 0, st>>>(wp, xp, k_tiles, ws.m_rows - 1, epi);
        else gemm_ring_kernel<4, 16, 5, 2, Epi><<<n_blocks, 64 * 6, 0, st>>>(wp, xp, k_tiles, ws.m_rows - 1, epi);
      } else {
        if (ws.m_pad == 16) gemm_narrow_kernel<1, 1, 8, 4, 4, Epi><<<n_blocks, 64 * 5, 0, st>>>(wp, xp, n_blocks, k_tiles, split, ws.m_rows - 1, epi);
        else if (ws.m_pad == 32) gemm_narrow_kernel<1, 2, 4, 5, 4, Epi><<<n_blocks, 64 * 6, 0, st>>>(wp, xp, n_blocks, k_tiles, split, ws.m_rows - 1, epi);
        else gemm_narrow_kernel<1, 4, 4, 6, 4, Epi><<<n_blocks, 64 * 8, 0, st>>>(wp, xp, n_blocks, k_tiles, split, ws.m_rows - 1, epi);
      }
      return;
    }
  }
  const dim3 grid((n_blocks + 1) / 2, SPLIT);
  auto go = [&](const auto& e) {
    using E = std::decay_t<decltype(e)>;
    // (ring depths within a few percent of each other: what counts is four fetching waves and few barriers)
    if (ws.m_pad == 16) gemm_narrow_kernel<2, 1, 8, 4, 4, E><<<grid, 64 * 6, 0, st>>>(wp, xp, n_blocks, k_tiles, split, ws.m_rows - 1, e);
    else if (ws.m_pad == 32) gemm_narrow_kernel<2, 2, 4, 5, 4, E><<<grid, 64 * 8, 0, st>>>(wp, xp, n_blocks, k_tiles, split, ws.m_rows - 1, e);
    else gemm_narrow_kernel<2, 4, 4, 6, 4, E><<<grid, 64 * 12, 0, st>>>(wp, xp, n_blocks, k_tiles, split, ws.m_rows - 1, e);
  };
  if constexpr (SPLIT == 2) go(StorePartialEpi{ws.split_part, ws.rl, n, (size_t)ws.m_pad * n});
  else go(epi);
}

// x + (p0 + p1) over the row blocks that hold rows: the halves of a split GEMM where the RMSNorm does not add them.
__global__ __launch_bounds__(256) void add_halves_kernel(float* __restrict__ x, const float* __restrict__ p0,
                                                         const float* __restrict__ p1, int n, const int32_t* __restrict__ live) {
  const size_t at = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;                 // (a workgroup lies within a row block: n % 128 == 0)
  if (live && (int)((size_t)blockIdx.x * 64 / n) * 16 >= live_rows(live)) return;
  *(f32x4*)(x + at) = *(const f32x4*)(x + at) + (*(const f32x4*)(p0 + at) + *(const f32x4*)(p1 + at));
}

// The halves in split_part: left to the RMSNorm that follows (true), or added here where that one runs a wave per row over
// interleaved rows (more than 512, d_model other than 1024, 2048, 4096 and 8192), whose pieces of 16 bytes cost more than this
// launch saves: the projections with their norms, us a pass of two layers, added here against left to that norm, taken on widths
// that ran so then: 2048 rows 298 against 338 (d_model 2048), 140 against 153 (1024), 1280 rows 1839 against 2037 (8192).
template <class Epi>
bool halves_pending(const Workspace& ws, int n, const Epi& epi, hipStream_t st) {
  if constexpr (std::is_same<Epi, ResidualEpi>::value) {
    if (norm_adds_halves(ws.m_pad, n)) return true;
    const size_t plane = (size_t)ws.m_pad * n;
    add_halves_kernel<<<(unsigned)(plane / 1024), 256, 0, st>>>(epi.resid, ws.split_part, ws.split_part + plane, n, ws.live);
  }
  return false;
}

// Up to 64 rows, wide outputs (gate/up, LM head).
template <class Epi>
void launch_wide(const bf16x8* wp, const bf16x8* xp, int n_blocks, int k_tiles, const Workspace& ws, const Epi& epi, hipStream_t st) {
  // 7 or 8 feature blocks per workgroup: whichever needs less (rounds of 256 workgroups) x (blocks each)
  const int g8 = (n_blocks + 7) / 8, g7 = (n_blocks + 6) / 7;
  const bool seven = ((g7 + 255) / 256) * 7 < ((g8 + 255) / 256) * 8;
  const unsigned gx = (unsigned)(seven ? g7 : g8);
  if (seven) {
    if (ws.m_pad == 16) gemm_xshare_kernel<1, 7, Epi><<<gx, 512, 0, st>>>(wp, xp, n_blocks, k_tiles, ws.m_rows - 1, epi);
    else if (ws.m_pad == 32) gemm_xshare_kernel<2, 7, Epi><<<gx, 512, 0, st>>>(wp, xp, n_blocks, k_tiles, ws.m_rows - 1, epi);
    else gemm_xshare_kernel<4, 7, Epi><<<gx, 512, 0, st>>>(wp, xp, n_blocks, k_tiles, ws.m_rows - 1, epi);
  } else {
    if (ws.m_pad == 16) gemm_xshare_kernel<1, 8, Epi><<<gx, 512, 0, st>>>(wp, xp, n_blocks, k_tiles, ws.m_rows - 1, epi);
    else if (ws.m_pad == 32) gemm_xshare_kernel<2, 8, Epi><<<gx, 512, 0, st>>>(wp, xp, n_blocks, k_tiles, ws.m_rows - 1, epi);
    else gemm_xshare_kernel<4, 8, Epi><<<gx, 512, 0, st>>>(wp, xp, n_blocks, k_tiles, ws.m_rows - 1, epi);
  }
}

// How a pass runs a GEMM of more than 64 rows; `split`: in two halves.
GemmPlan plan_gemm(Kind kind, int n_blocks, int k_tiles, bool split, const Workspace& ws) {
  const int h = split ? split_point(k_tiles) : k_tiles, m_pad = ws.m_pad;
  const Work one{kind, n_blocks, h, 1, ws.num_cus, ws.partly_filled}, both{kind, n_blocks, h, 2, ws.num_cus, ws.partly_filled};
  const Choice alone = pick_tile(one, m_pad), together = split ? pick_tile(both, m_pad) : alone;
  // The two halves in one launch, their sum left to what follows - or one after the other, the second adding the first one's
  // partial and the residual stream in its epilogue, where their workgroups take the same time either way: it saves the norms
  // the halves.  us for the projections and norms of one layer, one launch | two: 8B 1024 rows 199 | 205, 1280 210 | 237, 1536
  // 260 | 263, 2048 324 | 309, 4096 623 | 606; d_model 8192, 1024 rows 594 | 554, 4096 2246 | 2074; d_model 2048, 4096 rows
  // 174 | 162.  From 2048 rows on up to a third more is taken for it: the norms are a quarter of the layer there (d_model 2048,
  // 2048 rows: norms 38 | 26, but 95 | 106 in all; 127 before this kernel).
  // (The tile of short rounds has less than a launch's own time in its price: with it counted so here, d_model 512 at 2048 rows takes
  // 237 us a pass of two layers, in turn 244.)
  const long long apart = 2 * (alone.cost + (alone.tile == kShortRounds ? 1300 : 0));
  const bool in_turn = split && apart * 100 <= together.cost * (m_pad < 2048 ? 103 : 135);
  const Work& work = split && !in_turn ? both : one;
  const Choice all = split && !in_turn ? together : alone;
  const int fewer = ws.partly_filled && m_pad >= 768 ? rows_apart(work, m_pad, all) : 0;
  return GemmPlan{all.tile, fewer, fewer ? pick_tile(work, fewer).tile : 0, in_turn};
}

// QKV, gate/up and residual projections.  Returns whether a split GEMM left its two halves in split_part.
template <int SPLIT, class Epi>
bool launch_gemm(const uint16_t* w, const uint16_t* x, int n_blocks, int k_padded, int n, const Workspace& ws, const GemmPlan& plan,
                 const Epi& epi, hipStream_t st) {
  const int k_tiles = k_padded / 32, m_pad = ws.m_pad;
  const bf16x8* wp = (const bf16x8*)w;
  const bf16x8* xp = (const bf16x8*)x;
  if (m_pad <= 64) {
    if constexpr (std::is_same<Epi, SwigluEpi>::value) launch_wide(wp, xp, n_blocks, k_tiles, ws, epi, st);
    else launch_narrow<SPLIT>(wp, xp, n_blocks, k_tiles, n, ws, epi, st);
    return SPLIT == 2;
  }
  const auto launch = [&](int tile, int rows, int more_than) {
    if constexpr (SPLIT == 2) {
      const int h = split_point(k_tiles);
      const StorePartialEpi partial{ws.split_part, ws.rl, n, (size_t)m_pad * n};
      if (plan.in_turn) {
        launch_direct(tile, wp, xp, n_blocks, Range{k_tiles, h, 1, 1, rows, more_than}, ws, partial, st);
        launch_direct(tile, wp, xp, n_blocks, Range{k_tiles, h, 0, 1, rows, more_than}, ws, ResidualAddEpi{epi.resid, ws.split_part, ws.rl, n}, st);
      } else {
        launch_direct(tile, wp, xp, n_blocks, Range{k_tiles, h, 0, 2, rows, more_than}, ws, partial, st);
      }
    } else if constexpr (std::is_same<Epi, ResidualEpi>::value) {
      launch_direct(tile, wp, xp, n_blocks, Range{k_tiles, k_tiles, 0, 1, rows, more_than}, ws, ResidualAddEpi{epi.resid, nullptr, ws.rl, n}, st);
    } else {
      launch_direct(tile, wp, xp, n_blocks, Range{k_tiles, k_tiles, 0, 1, rows, more_than}, ws, epi, st);
    }
  };
  if (plan.fewer) launch(plan.fewer_tile, plan.fewer, -1);
  launch(plan.tile, m_pad, plan.fewer ? plan.fewer : -1);
  return SPLIT == 2 && !plan.in_turn && halves_pending(ws, n, epi, st);
}

// Off the fixed schedule (fast path, cost-of-determinism measurement) the split of the residual projections follows the batch, as
// in an ordinary engine: two halves while there are few rows to spread over the device, none beyond.
bool split_residual(const Workspace& ws) { return !(ws.batch_chosen && ws.m_rows > 16); }

}  // namespace

void plan_gemms(const llm42_model* m, Workspace& ws) {
  if (ws.m_pad <= 64) return;
  const int d_tiles = m->cfg.d_model / 32, d_blocks = m->cfg.d_model / 16;
  ws.gemm[GEMM_QKV] = plan_gemm(QKV, m->n_qkv / 16, d_tiles, false, ws);
  ws.gemm[GEMM_O] = plan_gemm(PLAIN, d_blocks, m->d_attn / 32, split_residual(ws), ws);
  ws.gemm[GEMM_GATE_UP] = plan_gemm(PLAIN, m->gu_blocks, d_tiles, false, ws);
  ws.gemm[GEMM_DOWN] = plan_gemm(PLAIN, d_blocks, m->ffn_k / 32, split_residual(ws), ws);
  const Work head{LM_HEAD, m->cfg.vocab / 16, d_tiles, 1, ws.num_cus, ws.partly_filled};
  ws.gemm[GEMM_LM_HEAD] = GemmPlan{ws.partly_filled ? pick_partly_filled(head, ws.m_pad) : pick_tile(head, ws.m_pad).tile, 0, 0, false};
}

void launch_gemm_qkv(const llm42_model* m, int layer, const llm42_kv_cache* kv, int window, const Workspace& ws,
                     hipStream_t st) {
  const llm42_config& c = m->cfg;
  const size_t plane = (size_t)kv->num_blocks * c.n_kv_heads * 16 * c.head_dim;
  QkvEpi e;
  e.row_rope = (const float4*)ws.row_rope;
  e.row_pos = ws.row_pos;
  e.row_seq = ws.row_seq;
  e.row_blk = ws.row_blk;
  e.q = ws.q;
  e.k_plane = (uint16_t*)kv->kv_base + ((size_t)layer * 2 + 0) * plane;
  e.v_plane = (uint16_t*)kv->kv_base + ((size_t)layer * 2 + 1) * plane;
  e.n_q_heads = c.n_q_heads;
  e.n_kv_heads = c.n_kv_heads;
  e.head_dim = c.head_dim;
  e.order = row_order(m->group, window);
  e.r_pad = ws.r_pad;
  launch_gemm<kSplit[GEMM_QKV]>(m->layers[layer].wqkv, ws.normed, m->n_qkv / 16, c.d_model, m->n_qkv, ws, ws.gemm[GEMM_QKV], e, st);
}

bool launch_gemm_residual(GemmKind kind, const uint16_t* w, const uint16_t* x, float* resid, int n, int k_padded,
                          const Workspace& ws, hipStream_t st) {
  ResidualEpi e{resid, ws.rl, n};
  if (!split_residual(ws)) return launch_gemm<1>(w, x, n / 16, k_padded, n, ws, ws.gemm[kind], e, st);
  return launch_gemm<kSplit[GEMM_O]>(w, x, n / 16, k_padded, n, ws, ws.gemm[kind], e, st);
}

void launch_gemm_swiglu(const llm42_model* m, int layer, const Workspace& ws, hipStream_t st) {
  SwigluEpi e{ws.hidden, m->ffn_k};
  launch_gemm<kSplit[GEMM_GATE_UP]>(m->layers[layer].wgu, ws.normed, m->gu_blocks, m->cfg.d_model, m->gu_blocks * 16, ws, ws.gemm[GEMM_GATE_UP], e, st);
}

// Returns the number of arg-max partials per row.
template <bool SAMPLED>
static int launch_logits(const llm42_model* m, int window, float* out_logits, const llm42_sampling* sampling, const Workspace& ws,
                         hipStream_t st) {
  LogitsEpi<SAMPLED> e;
  e.row_pos = ws.row_pos;
  e.row_seq = ws.row_seq;
  e.dump_slot = ws.dump_slot;
  e.out_logits = out_logits;
  e.amax = ws.amax;
  e.window = window;
  e.vocab = m->cfg.vocab;
  const int n_blocks = m->cfg.vocab / 16, k_tiles = m->cfg.d_model / 32;
  const bf16x8 *wp = (const bf16x8*)m->lm_head, *xp = (const bf16x8*)ws.normed;
  e.inv_temp = SAMPLED ? 1.0f / sampling->temperature : 0.f;
  e.seed = SAMPLED ? sampling->seed : 0;
  e.request_ids = SAMPLED ? sampling->request_ids : nullptr;
  if (ws.m_pad <= 64) {
    e.parts = n_blocks;
    launch_wide(wp, xp, n_blocks, k_tiles, ws, e, st);
  } else {
    const int tile = ws.gemm[GEMM_LM_HEAD].tile;
    e.parts = (n_blocks + kTiles[tile].bn() - 1) / kTiles[tile].bn();
    launch_direct(tile, wp, xp, n_blocks, Range{k_tiles, k_tiles, 0, 1, ws.m_pad, -1}, ws, e, st);
  }
  return e.parts;
}

int launch_gemm_logits(const llm42_model* m, int window, float* out_logits, const llm42_sampling* sampling,
                       const Workspace& ws, hipStream_t st) {
  return sampling && sampling->temperature > 0.f ? launch_logits<true>(m, window, out_logits, sampling, ws, st)
                                                 : launch_logits<false>(m, window, out_logits, sampling, ws, st);
}
