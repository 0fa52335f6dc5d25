// Parts shared by the GEMM kernels of the verifier pass: the layer-specific epilogues (rotary embedding + KV-cache write,
// residual add, SwiGLU, logits + arg-max partials) and the loads that go straight into LDS.
#pragma once
#include <type_traits>

#include "llm42_dev.h"

namespace gemm {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct QkvEpi {
  const float4* __restrict__ row_rope;    // [row][head_dim/4]: (cos, sin) of two consecutive rotary pairs at the row's position
  const int32_t* __restrict__ row_pos;
  const int32_t* __restrict__ row_seq;
  const int32_t* __restrict__ row_blk;    // physical KV block of the row's position
  uint16_t* q;               // [seq][kv head][r_pad][head_dim] tile layout, r: see RowOrder
  uint16_t* k_plane;         // this layer's K tiles [block][kv head][16*head_dim]
  uint16_t* v_plane;
  int n_q_heads, n_kv_heads, head_dim, r_pad;
  RowOrder order;

  // What the epilogue needs from memory besides the accumulators; requested when the kernel
  // starts so that its latency hides behind the weight stream.  Everything is indexed by the row
  // alone (the per-row block id and rotary factors are laid out once per call), so none of these
  // loads waits for another.
  struct Row {   // per token row
    int pos, tag, blk;
  };
  struct Pre {   // per (token row, feature block)
    int pos, tag, blk;
    float2 cs0, cs1;
  };
  __device__ Row row_info(int row) const {
    Row r;
    r.pos = row_pos[row];
    r.tag = row_seq[row];
    r.blk = row_blk[row];
    return r;
  }
  __device__ Pre pre(int nb, int lane, int row, const Row& r) const {
    Pre p;
    p.pos = r.pos;
    p.tag = r.tag;
    p.blk = r.blk;
    const int j0 = (nb % (head_dim >> 4)) * 8 + (lane >> 4) * 2;
    const float4 cs = row_rope[(size_t)row * (head_dim >> 2) + (j0 >> 1)];
    p.cs0 = make_float2(cs.x, cs.y);
    p.cs1 = make_float2(cs.z, cs.w);
    return p;
  }
  __device__ void operator()(int nb, int lane, int row, const f32x4 acc, const Pre& p) const {
    const int pos = p.pos;
    if (pos < 0) return;
    const int blocks_per_head = head_dim >> 4;
    const int head = nb / blocks_per_head, t = nb % blocks_per_head, g = lane >> 4;
    const int j0 = t * 8 + g * 2;           // features j0, j0+1 and their rotary partners j0 + hd/2, j0+1 + hd/2
    const int half = head_dim >> 1;
    const int s = tag_seq(p.tag);
    float lo0 = acc[0], lo1 = acc[1], hi0 = acc[2], hi1 = acc[3];
    if (head < n_q_heads + n_kv_heads) {
      const float2 cs0 = p.cs0, cs1 = p.cs1;
      const float a0 = lo0 * cs0.x - hi0 * cs0.y, b0 = hi0 * cs0.x + lo0 * cs0.y;
      const float a1 = lo1 * cs1.x - hi1 * cs1.y, b1 = hi1 * cs1.x + lo1 * cs1.y;
      lo0 = a0; hi0 = b0; lo1 = a1; hi1 = b1;
    }
    const uint32_t lo = pack2_bf16(lo0, lo1), hi = pack2_bf16(hi0, hi1);
    if (head < n_q_heads) {
      const int kvh = head / order.group, r = order.row(tag_index(p.tag), head % order.group);
      uint16_t* base = q + ((size_t)s * n_kv_heads + kvh) * r_pad * head_dim;
      *(uint32_t*)(base + pk_off(r, j0, head_dim)) = lo;
      *(uint32_t*)(base + pk_off(r, j0 + half, head_dim)) = hi;
      return;
    }
    const int blk = p.blk;
    const int tok = pos & 15;
    if (head < n_q_heads + n_kv_heads) {
      uint16_t* tile = k_plane + ((size_t)blk * n_kv_heads + (head - n_q_heads)) * 16 * head_dim;
      *(uint32_t*)(tile + ((j0 >> 3) * 16 + tok) * 8 + (j0 & 7)) = lo;
      *(uint32_t*)(tile + (((j0 + half) >> 3) * 16 + tok) * 8 + (j0 & 7)) = hi;
    } else {
      uint16_t* tile = v_plane + ((size_t)blk * n_kv_heads + (head - n_q_heads - n_kv_heads)) * 16 * head_dim;
      tile[v_tile_off(j0, tok)] = (uint16_t)lo;
      tile[v_tile_off(j0 + 1, tok)] = (uint16_t)(lo >> 16);
      tile[v_tile_off(j0 + half, tok)] = (uint16_t)hi;
      tile[v_tile_off(j0 + half + 1, tok)] = (uint16_t)(hi >> 16);
    }
  }
};

struct ResidualEpi {
  float* resid;   // fp32 residual stream [m_pad][n], updated in place (one lane owns each element)
  ResidLayout rl;
  int n;
  struct Row {};
  struct Pre {
    f32x4 old;
  };
  __device__ Row row_info(int) const { return Row{}; }
  __device__ Pre pre(int nb, int lane, int row, const Row&) const {
    return Pre{*(const f32x4*)(resid + rl.off(row, nb * 16 + (lane >> 4) * 4, n))};
  }
  __device__ void operator()(int nb, int lane, int row, const f32x4 acc, const Pre& p) const {
    *(f32x4*)(resid + rl.off(row, nb * 16 + (lane >> 4) * 4, n)) = p.old + acc;
  }
};

__device__ inline float silu_f32(float z) { return z / (1.0f + __expf(-z)); }

struct SwigluEpi {
  uint16_t* hidden;  // tile layout [m_pad][ffn_k]
  int ffn_k;
  struct Row {};
  struct Pre {};
  __device__ Row row_info(int) const { return Row{}; }
  __device__ Pre pre(int, int, int, const Row&) const { return Pre{}; }
  __device__ void operator()(int nb, int lane, int row, const f32x4 acc, const Pre&) const {
    // acc[0], acc[1]: gate of hidden features f, f+1;  acc[2], acc[3]: up of the same features
    const int f = nb * 8 + (lane >> 4) * 2;
    const float h0 = silu_f32(acc[0]) * acc[2], h1 = silu_f32(acc[1]) * acc[3];
    *(uint32_t*)(hidden + pk_off(row, f, ffn_k)) = pack2_bf16(h0, h1);
  }
};

// SAMPLED: temperature above zero.  (Kernels of their own: the noise is 10 times the code of the rest, and jumping over it
// misses the instruction cache for every block of an epilogue.)
template <bool SAMPLED>
struct LogitsEpi {
  const int32_t* row_pos;
  const int32_t* row_seq;
  const int32_t* dump_slot;
  float* out_logits;   // [n_dump][window][vocab] or null
  float2* amax;        // [m_pad][parts]: the best of a block of 16 features, or of a tile of gemm_direct_kernel
  int window, vocab, parts;
  // seeded sampling: 1 / temperature, seed, the caller's request ids (or null)
  float inv_temp;
  uint64_t seed;
  const int64_t* request_ids;
  struct Row {
    int pos, s, i, slot;
    uint64_t key;      // hash of (seed, request, position): the row's noise stream
  };
  typedef Row Pre;
  // output function of the splitmix64 generator
  static __device__ inline uint64_t mix(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  __device__ Row row_info(int row) const {
    Row p;
    p.pos = row_pos[row];
    const int tag = row_seq[row];
    p.s = tag_seq(tag);
    p.i = tag_index(tag);
    p.slot = out_logits ? dump_slot[p.s] : -1;
    p.key = 0;
    if constexpr (SAMPLED) {
      const uint64_t rid = request_ids ? (uint64_t)request_ids[p.s] : (uint64_t)p.s;
      p.key = mix(mix(seed ^ mix(rid)) ^ (uint64_t)(uint32_t)max(p.pos, 0));
    }
    return p;
  }
  __device__ Pre pre(int, int, int, const Row& r) const { return r; }
  // The best of what the sampler ranks and its feature so far: max, lowest index on ties, in any order.
  struct Best {
    float v = -INFINITY;
    int i = 0x7FFFFFFF;
    __device__ void take(float ov, int oi) {
      const bool other = ov > v || (ov == v && oi < i);
      v = other ? ov : v;
      i = other ? oi : i;
    }
  };
  // This lane's 4 logits of block nb: written out if asked for, ranked against `best`.
  __device__ void rank(int nb, int lane, const f32x4 acc, const Row& p, Best& best) const {
    const int n0 = nb * 16 + (lane >> 4) * 4;
    if (out_logits && p.pos >= 0) {
      const int slot = p.slot;
      if (slot >= 0)
        *(f32x4*)(out_logits + ((size_t)slot * window + p.i) * vocab + n0) = acc;
    }
    // what the sampler ranks: the logits, or (temperature > 0) logit / temperature + Gumbel noise
    f32x4 val = acc;
    if constexpr (SAMPLED) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t h = mix(p.key ^ (uint64_t)(n0 + e));
        const float u = (float)(2u * (uint32_t)(h >> 41) + 1u) * 0x1p-24f;   // exact: 24 significant bits, in (0, 1)
        val[e] = acc[e] * inv_temp - logf(-logf(u));
      }
    }
    // (ascending index, strict '>' keeps the lowest on ties)
    float bv = val[0];
    int bi = n0;
#pragma unroll
    for (int e = 1; e < 4; ++e)
      if (val[e] > bv) { bv = val[e]; bi = n0 + e; }
    best.take(bv, bi);
  }
  // ... and over the 4 lanes that hold the token's other features (lanes l ^ 16, l ^ 32).  A lane swap leaves a lane's own
  // pair and its partner's in the two results; `take` is symmetric in the two, so every lane ends up with the same winner.
  static __device__ Best over_lanes(Best b) {
    auto better_of = [](u32x2 v, u32x2 i) {
      Best r{__uint_as_float(v.x), (int)i.x};
      r.take(__uint_as_float(v.y), (int)i.y);
      return r;
    };
    b = better_of(__builtin_amdgcn_permlane16_swap(__float_as_uint(b.v), __float_as_uint(b.v), false, false),
                  __builtin_amdgcn_permlane16_swap((uint32_t)b.i, (uint32_t)b.i, false, false));
    return better_of(__builtin_amdgcn_permlane32_swap(__float_as_uint(b.v), __float_as_uint(b.v), false, false),
                     __builtin_amdgcn_permlane32_swap((uint32_t)b.i, (uint32_t)b.i, false, false));
  }
  // (the kernels of up to 64 rows: a partial per block)
  __device__ void operator()(int nb, int lane, int row, const f32x4 acc, const Pre& p) const {
    Best b;
    rank(nb, lane, acc, p, b);
    b = over_lanes(b);
    if (lane < 16) amax[(size_t)row * parts + nb] = make_float2(b.v, __int_as_float(b.i));
  }
};

template <class Epi>
struct is_logits : std::false_type {};
template <bool SAMPLED>
struct is_logits<LogitsEpi<SAMPLED>> : std::true_type {};

// ---------------------------------------------------------------------------------------------
// Split of the reduction dimension.  A GEMM with SPLIT == 2 has TWO accumulators per output
// element: p0 over k-tiles [0, h) and p1 over k-tiles [h, k_tiles), h = (k_tiles + 1) / 2, each
// started at zero and advanced in ascending k; the result is p0 + p1 (one fp32 add).  Which GEMMs
// are split is fixed per layer type below and never depends on the number of rows.
// ---------------------------------------------------------------------------------------------
__host__ __device__ inline int split_point(int k_tiles) { return (k_tiles + 1) / 2; }

// fp32 partial of one k-half of a split GEMM (the halves are workgroups of one launch, each with a buffer of its own, or two
// launches, the second of which adds the first one's).
struct StorePartialEpi {
  float* partial;   // [m_pad][n] in the residual-stream layout
  ResidLayout rl;
  int n;
  size_t plane;     // distance (floats) from the first half's buffer to the second's
  struct Row {};
  struct Pre {};
  __device__ Row row_info(int) const { return Row{}; }
  __device__ Pre pre(int, int, int, const Row&) const { return Pre{}; }
  __device__ void operator()(int nb, int lane, int row, const f32x4 acc, const Pre&) const {
    *(f32x4*)(partial + rl.off(row, nb * 16 + (lane >> 4) * 4, n)) = acc;
  }
};

// The residual stream with a projection added: x + p, or x + (p0 + p1) where `partial` holds the second half of a split one.
struct ResidualAddEpi {
  float* resid;
  const float* partial;   // p1, or null
  ResidLayout rl;
  int n;
  struct Row {};
  struct Pre {
    f32x4 old, other;
  };
  __device__ Row row_info(int) const { return Row{}; }
  __device__ Pre pre(int nb, int lane, int row, const Row&) const {
    const size_t at = rl.off(row, nb * 16 + (lane >> 4) * 4, n);
    return Pre{*(const f32x4*)(resid + at), *(const f32x4*)((partial ? partial : resid) + at)};
  }
  __device__ void operator()(int nb, int lane, int row, const f32x4 acc, const Pre& p) const {
    *(f32x4*)(resid + rl.off(row, nb * 16 + (lane >> 4) * 4, n)) = p.old + (partial ? acc + p.other : acc);
  }
};

// 1 KiB from global memory (wave-uniform `base` + per-lane byte offset `voff`) straight into LDS at
// byte address `dst` + 16 * lane (M0 holds the wave-uniform destination).  Written as assembly on
// purpose: with the compiler's own form of this load every later LDS read waits for all earlier
// ones, which un-pipelines the operand reads.  The compiler therefore does not count these loads;
// lds_fetch_wait() is the only wait that covers them.  Nothing else in these kernels uses M0.
// STREAM marks the load non-temporal (weights that no other workgroup reads).
template <bool STREAM = false>
__device__ __forceinline__ void lds_fetch_1k(const void* base, uint32_t voff, uint32_t dst) {
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(voff), "s"(base), "s"(dst) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base), "s"(dst) : "memory", "m0");
}
// At most N of the fetches this wave has issued are still on their way (they complete in order).
template <int N>
__device__ __forceinline__ void lds_fetch_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// The fetches of at most `ahead` rounds of PW each are still on their way.
template <int R, int PW>
__device__ __forceinline__ void wait_for_rounds(int ahead) {
  static_assert(R >= 3 && R <= 9 && (R - 2) * PW <= 63, "vmcnt counts up to 63");
  switch (ahead) {
    case 1: lds_fetch_wait<PW>(); break;
    case 2: lds_fetch_wait<(R > 3 ? 2 : 0) * PW>(); break;
    case 3: lds_fetch_wait<(R > 4 ? 3 : 0) * PW>(); break;
    case 4: lds_fetch_wait<(R > 5 ? 4 : 0) * PW>(); break;
    case 5: lds_fetch_wait<(R > 6 ? 5 : 0) * PW>(); break;
    case 6: lds_fetch_wait<(R > 7 ? 6 : 0) * PW>(); break;
    case 7: lds_fetch_wait<(R > 8 ? 7 : 0) * PW>(); break;
    default: lds_fetch_wait<0>();
  }
}

// Tiles of gemm_direct_kernel (gemm_direct.h), in blocks of 16, and what a round of one workgroup per CU takes: 1/1000 us per
// k-tile, fitted to launches within passes (8B shapes, 128 - 4096 rows) that fill one or more rounds, and 3 us + 24 ns per
// block of the tile that do not depend on K (O- and down-projection differ in K only: 16 x 10 blocks 41.7 and 117.7 us, 64 and
// 224 k-tiles).  Rounds of fewer workgroups take as long (half of the CUs 0.45 against 0.48 us per k-tile): a CU's own fetches
// and arithmetic are what a round waits for.  Of the last three the first is for split projections of partly filled windows,
// priced for half of the rows: every workgroup has all token blocks, fetches those that hold rows, and reads weights that no
// other does, where 4 x 4 blocks leave half of the CUs without rows (8B, us per pass with a quarter, half, three quarters and
// all of 120 rows there: 4442, 4667, 4607, 4643 -> 4034, 4433, 4692, 4735). The other two are for small K.  One is the 4 x 4
// blocks again in rounds of four k-tiles, two register sets: the others' rounds left over behind the last whole group of them
// take about 1 us more, in code of their own, and 900 ns where they have 3000 puts it ahead up to about 40 k-tiles (us for two
// launches, the tile at 2200 ns -> this: 128 rows of d_model 1024 O 16.6 -> 12.9 and gate/up 19.3 -> 16.6, at 512 rows down
// 25.8 -> 21.8; 128 rows of d_model 512 gate/up 17.0 -> 13.2; of the 34 launches that it now takes at d_model 512 - 4096 29 are
// faster, and QKV of 24 k-tiles at 128 - 192 rows is not, 16.5 - 17.0 -> 17.0 - 17.6).  The other is 8 x 8 blocks two to a CU,
// where neither's beginning nor end leaves it idle, for the LM head (32 k-tiles x 50304 features: 512 rows 58 us against 61 -
// 85 with the others, 4096 396 against 436; the heavier epilogue of gate/up gains nothing from it).
struct Tile {
  int nw, fb, bm;      // multiplying waves, feature blocks of each; token blocks
  int ch, r, f, nset;  // k-tiles of a round, rounds in LDS, fetching waves, register sets of weights
  int per_cu;          // workgroups per CU
  bool nt;             // with one token tile the weights are streamed past the caches (see launch_tile)
  int cost;
  constexpr int bn() const { return nw * fb; }
};
constexpr Tile kTiles[] = {
    {3, 1, 4, 8, 4, 4, 3, 1, false, 115}, {4, 1, 4, 8, 4, 4, 3, 1, false, 144}, {6, 1, 4, 8, 4, 4, 2, 1, false, 152},
    {3, 1, 6, 4, 5, 4, 3, 1, false, 140}, {4, 1, 6, 4, 5, 4, 3, 1, false, 160}, {4, 1, 8, 4, 4, 4, 2, 1, false, 180},
    {6, 1, 6, 4, 5, 4, 3, 1, false, 185}, {8, 1, 6, 4, 5, 4, 3, 1, false, 215}, {6, 1, 8, 4, 4, 4, 2, 1, false, 215},
    {7, 1, 8, 4, 4, 4, 2, 1, true, 230}, {8, 1, 8, 4, 4, 4, 2, 1, false, 242}, {8, 1, 10, 2, 5, 4, 3, 1, false, 285},
    {7, 1, 12, 2, 4, 4, 3, 1, true, 300}, {6, 1, 12, 2, 4, 2, 4, 1, false, 300}, {4, 2, 12, 2, 4, 4, 3, 1, false, 326},
    {7, 1, 16, 2, 4, 4, 2, 1, true, 365}, {6, 2, 8, 4, 4, 2, 2, 1, false, 330}, {8, 2, 8, 4, 4, 4, 2, 1, true, 376},
    {4, 2, 16, 2, 4, 4, 2, 1, false, 372}, {8, 2, 10, 2, 5, 4, 2, 1, false, 476}, {7, 2, 12, 2, 4, 1, 3, 1, false, 480},
    {7, 2, 14, 2, 4, 1, 3, 1, false, 545}, {6, 2, 16, 2, 3, 1, 3, 1, false, 570}, {7, 2, 16, 2, 3, 1, 3, 1, false, 605},
    {7, 4, 10, 1, 6, 1, 2, 1, false, 760}, {7, 4, 12, 1, 4, 1, 2, 1, false, 930}, {2, 1, 8, 4, 4, 4, 4, 1, false, 95},
    {4, 1, 4, 4, 4, 4, 2, 1, false, 170}, {4, 2, 8, 2, 4, 2, 2, 2, false, 477}};
constexpr int kTileCount = sizeof kTiles / sizeof kTiles[0], kShortRounds = kTileCount - 2, kPartly = kTileCount - 3;

// The epilogues that tile t has a kernel for; tile_cost offers it to no other work.
template <class Epi>
constexpr bool serves(int t) {
  return t == kPartly ? std::is_same<Epi, StorePartialEpi>::value : kTiles[t].per_cu == 1 || is_logits<Epi>::value;
}

struct Choice {
  int tile;
  long long cost;   // ns
};
// The cheapest tile for n_blocks x m_pad rows by k_tiles, `planes` times over.  A launch takes whole rounds however many there
// are: QKV of 12288 features x 4096 by 14 x 16 blocks 3.0 rounds 365 us, 3.4 368, 4.3 457, 5.2 557, 6.0 643, 6.9 661, gate/up
// of 8192 features x 4096 2.9 rounds 257, 3.5 329, 4.05 411, 4.6 414.  (Priced as their share and a quarter of a round beyond
// four rounds, the tile with a few workgroups too many won: that QKV at 6144 rows 557 us, 510 by 6.9 rounds of 14 x 12 blocks;
// at 5120 rows 457 -> 411; that gate/up at 7168 rows 411 -> 364; of 27 launches at d_model 768 - 8192 and 1152 - 8192 rows that
// take another tile now 25 are 1 - 13 % faster, two 0.4 and 1.9 % slower.) Two workgroups to a CU are never in step and take
// their share and a quarter (LM head of 50304 features x 1024 and x 768, 3.1 rounds at 512 rows: 59 and 51 us by 14 x 16
// blocks, 57 and 47 by 8 x 8; with half of the rows there 61 and 52 against 46 and 38).  With up to two rounds of them the
// other tiles are the better ones where all rows are there (32000 x 2048, 384 and 512 rows 58 and 65 us against 59 and 74), not
// where half are (50304 x 1024, 256 rows 33 against 25, with all of them 34 and 38). The epilogues of QKV and LM head do much
// per row, and with 16 token blocks to a wave and few features that counts (QKV at 1024 rows: 16 x 8 blocks 63.6 us, 8 x 16
// 67.0; LM head of 32000 features at 512 rows 114 and 119).  So it does for QKV with 12 x 16 blocks in more than one round
// (against 16 x 8, us: 8B 3328 rows 184 and 174, 4096 195 and 184, 5888 295 and 293, 8192 395 and 368; d_model 2048, 3072
// features, 6656 rows 118 and 107, 8192 120 and 114; d_model 8192, 12288 features, 3072 rows 533 and 538).
enum Kind { QKV, PLAIN, LM_HEAD };
struct Work {
  Kind kind;
  int n_blocks, k_tiles, planes;
  long long cus;
  bool partly;   // a verifier pass with partly filled windows
};
// What tile t takes for `rows` rows (negative: it is not for this work), in a launch for `of` rows.
inline long long tile_cost(int t, const Work& w, int rows, int of = 0) {
  const Tile& q = kTiles[t];
  const long long tiles_n = (w.n_blocks + q.bn() - 1) / q.bn(), tiles = tiles_n * ((rows + 16 * q.bm - 1) / (16 * q.bm)) * w.planes;
  const long long slots = w.cus * q.per_cu;
  const long long whole = (tiles + slots - 1) / slots * 64, share = tiles * 64 / slots + 16;   // rounds, in 1/64
  if (t == kPartly && !(w.partly && w.planes == 2)) return -1;
  const long long launched = of ? tiles_n * (of / (16 * q.bm)) : tiles;
  if (q.per_cu == 2 && (w.kind != LM_HEAD || launched <= (w.partly ? 1 : 2) * slots)) return -1;
  long long round = (long long)q.cost * w.k_tiles + (q.per_cu == 2 ? 500 : (t == kShortRounds ? 900 : 3000) + 24 * q.bn() * q.bm);
  if (w.kind != PLAIN && q.bm == 16 && q.bn() <= (w.kind == QKV ? 12 : 8)) round += round / 20;
  return (q.per_cu == 2 && share < whole ? share : whole) * round / 64;
}
inline Choice pick_tile(const Work& w, int m_pad) {
  Choice best{-1, 0};
  for (int t = 0; t < kTileCount; ++t) {
    if (m_pad % (16 * kTiles[t].bm)) continue;
    const long long cost = tile_cost(t, w, m_pad);
    if (cost >= 0 && (best.tile < 0 || cost < best.cost)) best = Choice{t, cost};
  }
  return best;
}
// The LM head of partly filled windows has one launch, for the merge reads its partials by the tile.  The best tile for all of the
// rows gives way to one that takes no more than 5 % longer there and a twentieth less on average over eight counts from 19/64 to 61/64
// of them: its workgroups may have nothing to leave out.  (us per launch with a quarter, half and all of the rows there, best for
// all -> this: 128256 features x 4096, 384 rows 246, 358, 359 -> 199, 271, 356; 32000 x 4096, 768 rows 82, 168, 170 -> 71, 114, 168.
// 88 launches at d_model 512 - 8192: 4 % less at a quarter and at half, as long where all rows are there; at 3 % seven more of them
// lose, at 10 % nine.)
inline int pick_partly_filled(const Work& w, int m_pad) {
  const Choice all = pick_tile(w, m_pad);
  auto average = [&](int t) {
    long long sum = 0;
    for (int q = 19; q < 64; q += 6) sum += tile_cost(t, w, m_pad * q / 64, m_pad);
    return sum;
  };
  Choice best{all.tile, average(all.tile) * 19 / 20};
  for (int t = 0; t < kTileCount; ++t) {
    if (m_pad % (16 * kTiles[t].bm)) continue;
    const long long full = tile_cost(t, w, m_pad);
    if (full < 0 || full * 100 > all.cost * 105) continue;
    const long long a = average(t);
    if (a < best.cost) best = Choice{t, a};
  }
  return best.tile;
}
// Partly filled windows: how many rows there are only the device knows, and the tile that fits all that there could be is not
// the one for the half of them that windows of random counts hold.  The number of rows, of 9/16 to 3/4 of all, that are to have
// a launch of their own beside the one for more (the one that does not apply ends at once, in 4 us): the largest whose tile
// takes no more than 5 % longer than the best of them, if that saves 15 % against the tile for all on as many rows; else 0.
// (8B, us per pass: 516 rows of 999 12682 -> 11126, 440 of 748 12141 -> 11153, 1735 of 3161 33318 -> 29146; with a tenth 1757
// of 3549 31191 -> 31444, with 5/8 of all whatever its tile -> 37841.  Windows that are all full, given as counts, take 0.97 -
// 1.02 of the time without counts at the 8B shape, 80 - 4096 rows, up to 1.03 at other widths and 1.06 at 128 - 256 rows there
// - the launch that ends at once, the read of the count, the tile for split projections of partly filled windows - and 0.75 -
// 1.01 of that before these kernels.)
inline int rows_apart(const Work& w, int m_pad, Choice all) {
  long long least = 0;
  for (int pass = 0; pass < 2; ++pass)
    for (int rows = m_pad * 3 / 4 / 128 * 128; rows * 16 >= m_pad * 9; rows -= 128) {
      const long long cost = pick_tile(w, rows).cost;
      if (pass == 0) least = least == 0 || cost < least ? cost : least;
      else if (cost * 100 <= least * 105) return (cost + 4000) * 100 <= tile_cost(all.tile, w, rows) * 85 ? rows : 0;
    }
  return 0;
}

// What a launch covers.  k-tiles: all of them (split == k_tiles), or `planes` halves from `first_plane` on, the second one from
// k-tile `split` on.  Rows: `rows` of the pass's; with packed rows it runs if more than `more_than` and no more than `rows` are
// there (counted in blocks of 16), else its workgroups leave at once.
struct Range {
  int k_tiles, split, first_plane, planes, rows, more_than;
};

// D = W X with the epilogue, by tile `tile` of kTiles.  Without such a tile nothing runs and the error is left for hipGetLastError.
template <class Epi>
void launch_direct(int tile, const bf16x8* wp, const bf16x8* xp, int n_blocks, const Range& k, const Workspace& ws, const Epi& epi,
                   hipStream_t st);
extern template void launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const QkvEpi&, hipStream_t);
extern template void launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const SwigluEpi&, hipStream_t);
extern template void launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const LogitsEpi<false>&, hipStream_t);
extern template void launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const LogitsEpi<true>&, hipStream_t);
extern template void launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const StorePartialEpi&, hipStream_t);
extern template void launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const ResidualAddEpi&, hipStream_t);

}  // namespace gemm
