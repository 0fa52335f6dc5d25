// The GEMM of more than 64 rows: gemm_direct_kernel, its tiles and the rule that chooses among them.  A template of the
// epilogue; each gemm_direct_*.hip holds the kernels of one.
#pragma once
#include <utility>

#include "gemm_parts.h"

namespace gemm {

// A workgroup owns a tile of NW * FB feature blocks x TB token blocks.  Each of NW waves owns FB of the feature blocks and all
// the token blocks, and loads its weight tiles from memory straight into registers, NSET sets of CH k-tiles: one in use,
// NSET - 1 on their way.  F further waves do nothing but move the activation tiles, which all waves need, into a ring of R
// rounds of CH k-tiles in LDS.  One barrier per round: behind it round r of the activations has landed, and the slot of round
// r - 1 is refilled.
//
// What bounds it up to about 1000 rows is what one CU can fetch: it has 32 KiB of loads in flight, whatever a kernel issues
// (one CU reads 43 GB/s with 16 KiB outstanding, 68 with 32 KiB and 68 with 128 KiB), and they return in order, so weights from HBM
// and activations from L2 add up in a CU although neither the memory nor the L2 is busy (448 KiB of weights per CU 18 us, 1792 KiB
// of activations 18 us, both in one workgroup 35 us, in workgroups on different CUs 21 us).  Hence tiles that put every CU to work
// exactly once where there is one for the shape, and weights that do not pass through LDS, which leaves all of it to the
// activations, a barrier for every 2 - 8 k-tiles instead of one and runs of CH KiB per weight row (runs of 1 KiB stream
// at 4.4 TB/s, of 2 KiB and more at 6).  Beyond that it is the power of the matrix cores, as for any kernel here.
// us per launch within a pass (events, 8B shapes), operands through LDS with 64 x 64 ... 256 x 128 tiles before -> this:
//            QKV            O-projection   down-projection   gate/up          LM head
//    128     25.6 -> 22.0   16.6 -> 15.9    42.2 ->  39.4    57.8 ->  47.8     230 ->  211
//    256     30.4 -> 27.1   19.2 -> 18.4    48.9 ->  47.3    73.3 ->  63.8     316 ->  311
//    512     44.4 -> 36.6   26.4 -> 25.3    69.2 ->  64.1   114.1 ->  94.8     509 ->  508
//    768     64.0 -> 49.7   34.2 -> 30.1    96.0 ->  82.3   168.0 -> 135.8     761 ->  707
//   1024     66.1 -> 57.3   36.9 -> 34.9   104.8 ->  95.1   207.1 -> 181.3    1017 ->  911
//   1280     70.4 -> 66.6   58.4 -> 41.6   164.2 -> 117.7   262.8 -> 231.2    1270 -> 1196
//   1536     94.9 -> 78.7   62.2 -> 53.4   180.0 -> 152.3   302.9 -> 262.7    1505 -> 1385
//   2048    101.6 -> 100.6                                  366.6 -> 354.8    2102 -> 1796
//   3072    182.0 -> 152.5                                  552.9 -> 530      3145 -> 2747
//   4096    194.3 -> 184.0 157.1 -> 151.5  411.5 -> 394.6   717.5 ->  720    4379 -> 3687
// (gate/up at 4096 rows 1.30 - 1.35 PFLOP/s, level with the vendor library's GEMM of the shape: from 1 % below to 1.5 % above it
// in four runs that timed both.)
// Other widths (d_model 512 - 8192, 80 - 6144 rows), passes of two layers against the kernels before this one: 189 calls with full
// windows take 0.71 - 1.01 of their time, 0.88 on average, 532 with partly filled ones 0.71 - 1.05, 0.89 on average.  What takes
// longer: a quarter of 1280 - 3072 rows there (up to 1.05: the halves that follow each other, in tiles for 9/16 of the rows, leave CUs
// idle); and within calls that take less, gate/up of 32 k-tiles x 8192 features at 4096 rows (66 -> 76 us).
template <int NW, int FB, int TB, int CH, int R, int F, int NSET, int WGS, bool NT, class Epi>
__global__ __launch_bounds__(64 * (NW + F), (WGS * (NW + F) + 3) / 4) void gemm_direct_kernel(
    const bf16x8* __restrict__ w, const bf16x8* __restrict__ x, int n_blocks, int k_tiles, int split, int first_plane, int planes,
    int tiles_n, int tiles_m, const int32_t* __restrict__ live, int more_than, bool renumber, Epi epi) {
  constexpr int TBN = NW * FB;
  constexpr int PW = CH * TB / F;                    // activation tiles a fetching wave requests per round
  static_assert(CH * TB % F == 0, "the fetching waves take equal shares");
  static_assert(NSET >= 2 && NSET <= 4, "the rounds are written out for 2 .. 4 register sets");
  __shared__ bf16x8 ring[R][CH * TB * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // Packed rows: only the token blocks that hold any are fetched, and a workgroup without one leaves at once.  The others of its
  // tile are multiplied with whatever lies in LDS and stay apart, a column of the result each; what a CU fetches is what
  // these launches wait for.  (8B, ms per pass: 27 rows of 65 4.64 -> 4.32, 516 of 999 13.53 -> 12.90, draws up to 12 % less; the
  // count is a dependent read of 0.7 us that full windows pay for: prefill of 700 tokens by 256 as before.)  `renumber`: launches
  // of more workgroups than CUs also close the gaps.
  const int live_blocks = live ? (live_rows(live) + 15) / 16 : tiles_m * TB;
  if (live && (live_blocks <= more_than || live_blocks > tiles_m * TB)) return;
  if (renumber) tiles_m = max(1, (live_blocks + TB - 1) / TB);
  const int all = tiles_n * tiles_m, per_xcd = (all * planes + 7) / 8;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  const int nth = tile / all, plane = first_plane + nth, at = tile - nth * all;
  if ((int)(blockIdx.x >> 3) >= per_xcd || nth >= planes) return;
  // an XCD takes a contiguous run of the tiles, panel by panel of about 1024 tokens, token tiles fastest within a panel
  constexpr int PANEL = 64 / TB;
  const int panel = at / (tiles_n * PANEL), in = at - panel * tiles_n * PANEL, width = min(PANEL, tiles_m - panel * PANEL);
  const int n0 = in / width * TBN, m0 = (panel * PANEL + in % width) * TB;       // first feature / token block of the tile
  if (m0 >= live_blocks) return;
  const int k_begin = plane ? split : 0, k_count = plane ? k_tiles - split : split;
  const int rounds = (k_count + CH - 1) / CH;
  if constexpr (std::is_same<Epi, StorePartialEpi>::value) epi.partial += nth * epi.plane;
  if (wave >= NW) {
    const int fw = wave - NW;
    if (m0 + fw * PW / CH >= live_blocks) {          // nothing but padding: what the others find in LDS is of no account
      for (int r = 0; r < rounds; ++r) __syncthreads();
      return;
    }
    const uint32_t dst = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[0][0];
    const bf16x8* src[PW];                           // (a token block's CH k-tiles are neighbours, in memory and in the ring)
#pragma unroll
    for (int i = 0; i < PW; ++i) src[i] = x + ((size_t)(m0 + (fw * PW + i) / CH) * k_tiles + k_begin) * 64;
    auto fetch = [&](int r) {                        // (k-tiles past the range re-read the last one)
#pragma unroll
      for (int i = 0; i < PW; ++i)
        lds_fetch_1k(src[i], (uint32_t)min(r * CH + (fw * PW + i) % CH, k_count - 1) * 1024u + lane * 16u,
                     dst + (uint32_t)(((r % R) * CH * TB + fw * PW + i) * 1024));
    };
    for (int r = 0; r < min(R - 1, rounds); ++r) fetch(r);
    for (int r = 0; r < rounds; ++r) {
      wait_for_rounds<R, PW>(min(R - 2, rounds - 1 - r));
      __syncthreads();                               // round r is in LDS; everyone is done with round r - 1
      if (r + R - 1 < rounds) fetch(r + R - 1);      // into the slot of round r - 1
    }
    return;
  }
  const bf16x8* wp[FB];                              // (wave-uniform; feature blocks past the matrix re-read the last one)
#pragma unroll
  for (int i = 0; i < FB; ++i) wp[i] = w + ((size_t)min(n0 + wave * FB + i, n_blocks - 1) * k_tiles + k_begin) * 64;
  f32x4 acc[FB][TB];
#pragma unroll
  for (int i = 0; i < FB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  bf16x8 wr[NSET][CH][FB];
  auto load = [&](bf16x8(&d)[CH][FB], int r) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const size_t k = (size_t)min(r * CH + j, k_count - 1) * 64;
#pragma unroll
      for (int i = 0; i < FB; ++i) d[j][i] = NT ? __builtin_nontemporal_load(wp[i] + k + lane) : (wp[i] + k)[lane];
    }
  };
  // Round r on register set U.  The activation operands are requested PD MFMA groups ahead by hand (the scheduling barriers keep
  // the compiler from sinking the reads next to their uses); the weights of the round NSET - 1 ahead behind the first of them.
  // FULL: all CH k-tiles are in range (known at compile time: with a branch around it the loop spills).
  auto round = [&](auto set, auto is_full, int r) __attribute__((always_inline)) {
    constexpr int U = decltype(set)::value, PD = FB == 1 ? 6 : 4, N = CH * TB;
    constexpr bool FULL = decltype(is_full)::value;
    const bf16x8* p = ring[r % R] + lane;
    bf16x8 q[PD + 1];
    auto operand = [&](int idx) { return p[((idx % TB) * CH + idx / TB) * 64]; };
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PD; ++t) q[t] = operand(t);
    __builtin_amdgcn_sched_barrier(0);
    load(wr[(U + NSET - 1) % NSET], r + NSET - 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int idx = 0; idx < N; ++idx) {
      if (idx + PD < N) q[(idx + PD) % (PD + 1)] = operand(idx + PD);
      __builtin_amdgcn_sched_barrier(0);
      if (FULL || r * CH + idx / TB < k_count) {
#pragma unroll
        for (int i = 0; i < FB; ++i) acc[i][idx % TB] = mfma16(wr[U][idx / TB][i], q[idx % (PD + 1)], acc[i][idx % TB]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  using Set2 = std::integral_constant<int, NSET == 2 ? 0 : 2>;
  using Set3 = std::integral_constant<int, NSET == 4 ? 3 : 0>;
#pragma unroll
  for (int u = 0; u < NSET - 1; ++u) load(wr[u], u);
  int r = 0;
  for (; (r + NSET) * CH <= k_count; r += NSET) {    // groups of NSET rounds without an exit in between
    round(Set0{}, std::true_type{}, r);
    round(Set1{}, std::true_type{}, r + 1);
    if constexpr (NSET > 2) round(Set2{}, std::true_type{}, r + 2);
    if constexpr (NSET > 3) round(Set3{}, std::true_type{}, r + 3);
  }
  if (r < rounds) round(Set0{}, std::false_type{}, r);
  if (r + 1 < rounds) round(Set1{}, std::false_type{}, r + 1);
  if constexpr (NSET > 2) {
    if (r + 2 < rounds) round(Set2{}, std::false_type{}, r + 2);
  }
  if constexpr (NSET > 3) {
    if (r + 3 < rounds) round(Set3{}, std::false_type{}, r + 3);
  }
  // epilogue, EG token blocks at a time: what they need from memory is requested together.  kTight: beside 192 accumulators the 8
  // operands for each of four feature blocks have registers for one at a time, and offsets are not worked out ahead of the loop.
  constexpr bool kTight = FB * TB >= 48 && std::is_same<Epi, ResidualAddEpi>::value;
  constexpr int EG = kTight ? 1 : TB % 4 == 0 && FB <= 2 ? 4 : 2;
  int el = lane;
  if constexpr (kTight) asm volatile("" : "+v"(el));
  static_assert(TB % EG == 0, "whole groups of token blocks");
  constexpr bool kLogits = is_logits<Epi>::value;
  float2* best = (float2*)ring;                      // LM head: [NW][16 TB] best of a wave's features
  if constexpr (kLogits) __syncthreads();            // everyone is done with the ring (the fetching waves have left)
#pragma unroll
  for (int j0 = 0; j0 < TB; j0 += EG) {
    typename Epi::Row info[EG];
    typename Epi::Pre pre[EG][FB];
#pragma unroll
    for (int j = 0; j < EG; ++j) {
      const int row = (m0 + j0 + j) * 16 + (el & 15);
      info[j] = epi.row_info(row);
#pragma unroll
      for (int i = 0; i < FB; ++i) pre[j][i] = epi.pre(min(n0 + wave * FB + i, n_blocks - 1), el, row, info[j]);
    }
#pragma unroll
    for (int j = 0; j < EG; ++j) {
      if constexpr (kLogits) {
        typename Epi::Best b;
#pragma unroll
        for (int i = 0; i < FB; ++i) {
          const int nb = n0 + wave * FB + i;
          if (nb < n_blocks) epi.rank(nb, el, acc[i][j0 + j], info[j], b);
        }
        b = Epi::over_lanes(b);
        if (el < 16) best[wave * 16 * TB + (j0 + j) * 16 + el] = make_float2(b.v, __int_as_float(b.i));
      } else {
#pragma unroll
        for (int i = 0; i < FB; ++i) {
          const int nb = n0 + wave * FB + i;
          if (nb < n_blocks) epi(nb, el, (m0 + j0 + j) * 16 + (el & 15), acc[i][j0 + j], pre[j][i]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (kLogits) {
    // one partial per row and workgroup (with a partial per block of 16 features, each 8 bytes in a line of their own, the merge
    // took 77 us at 4096 rows of 128256 features and 14 at 512; now 12 and 7)
    __syncthreads();
    for (int t = threadIdx.x; t < 16 * TB; t += 64 * NW) {
      typename Epi::Best b;
#pragma unroll
      for (int v = 0; v < NW; ++v) {
        const float2 p = best[v * 16 * TB + t];
        b.take(p.x, __float_as_int(p.y));
      }
      epi.amax[(size_t)(m0 * 16 + t) * tiles_n + n0 / TBN] = make_float2(b.v, __int_as_float(b.i));
    }
  }
}

template <int T, bool NT, class Epi>
void launch_tile(const bf16x8* wp, const bf16x8* xp, int n_blocks, const Range& k, const Workspace& ws, const Epi& epi, hipStream_t st) {
  constexpr Tile q = kTiles[T];
  const int tiles_n = (n_blocks + q.bn() - 1) / q.bn(), tiles_m = k.rows / (16 * q.bm);
  const int per_xcd = (tiles_n * tiles_m * k.planes + 7) / 8;
  gemm_direct_kernel<q.nw, q.fb, q.bm, q.ch, q.r, q.f, q.nset, q.per_cu, NT, Epi><<<8 * per_xcd, 64 * (q.nw + q.f), 0, st>>>(
      wp, xp, n_blocks, k.k_tiles, k.split, k.first_plane, k.planes, tiles_n, tiles_m, ws.live, k.more_than / 16,
      ws.live && (long long)tiles_n * tiles_m * k.planes > ws.num_cus, epi);
}

// Tile::nt: with one token tile no other workgroup reads the weights, and they are marked to be streamed past the caches
// (gate/up at 128 rows 51.0 -> 48.8 us, at 256 66.7 -> 64.9, LM head at 128 230 -> 215; with several token tiles no gain)
template <int T, class Epi>
bool launch_if(int tile, const bf16x8* wp, const bf16x8* xp, int n_blocks, const Range& k, const Workspace& ws, const Epi& epi,
               hipStream_t st) {
  if (!serves<Epi>(T) || tile != T || k.rows % (16 * kTiles[T].bm)) return false;
  if constexpr (serves<Epi>(T)) {
    if (kTiles[T].nt && k.rows == 16 * kTiles[T].bm) launch_tile<T, kTiles[T].nt>(wp, xp, n_blocks, k, ws, epi, st);
    else launch_tile<T, false>(wp, xp, n_blocks, k, ws, epi, st);
  }
  return true;
}

template <int... T, class Epi>
bool launch_any(std::integer_sequence<int, T...>, int tile, const bf16x8* wp, const bf16x8* xp, int n_blocks, const Range& k,
                const Workspace& ws, const Epi& epi, hipStream_t st) {
  return (launch_if<T>(tile, wp, xp, n_blocks, k, ws, epi, st) || ...);
}

template <class Epi>
void launch_direct(int tile, const bf16x8* wp, const bf16x8* xp, int n_blocks, const Range& k, const Workspace& ws, const Epi& epi,
                   hipStream_t st) {
  if (!launch_any(std::make_integer_sequence<int, kTileCount>{}, tile, wp, xp, n_blocks, k, ws, epi, st))
    (void)hipLaunchKernel(nullptr, dim3(1), dim3(1), nullptr, 0, st);   // (fails: no such tile for this epilogue and number of rows)
}

}  // namespace gemm
