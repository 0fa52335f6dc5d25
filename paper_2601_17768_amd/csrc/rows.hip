// Row-wise kernels of the verifier pass: input validation and row metadata,
// embedding gather, RMSNorm.
#include <type_traits>

#include "llm42_dev.h"

namespace {

// One workgroup per sequence.  Validates what only the device can see (lengths,
// block-table entries, token ids) and writes the row metadata every later kernel
// uses.  A sequence that fails a check is switched off as a whole: its rows get
// position -1, no KV slot of it is read or written and its outputs are -1.
__global__ void prepare_kernel(const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ candidates,
                               const int32_t* __restrict__ n_valid, const int32_t* __restrict__ block_table,
                               int max_blocks_per_seq, int64_t num_blocks, int window, int max_context, int vocab,
                               const int32_t* __restrict__ dump_seq_ids, int n_dump, int32_t* out_tokens,
                               int32_t* seq_status, int32_t* row_pos, int32_t* row_seq, int32_t* ws_len,
                               int32_t* ws_n, int32_t* dump_slot, const float2* __restrict__ rope, int half_dim,
                               int32_t* row_blk, float2* row_rope, int min_n, int status_or,
                               uint16_t* __restrict__ attn_zero, int d_attn, bool packed, int m_pad) {
  __shared__ int status, before;
  const int s = blockIdx.x;
  if (threadIdx.x == 0) status = 0, before = 0;
  __syncthreads();
  const int L = seq_lens[s];
  const int n = n_valid ? n_valid[s] : window;
  int bad = 0;
  // (min_n is 1; a prefill pass passes 0: a sequence whose prompt has ended takes no part in the pass)
  auto bad_length = [&](int len, int cnt) { return len < 0 || cnt < min_n || cnt > window || (int64_t)len + cnt > max_context; };
  if (bad_length(L, n)) bad = LLM42_SEQ_BAD_LENGTH;
  // Packed rows: what fails a check of its length has none, what fails a later one keeps dead rows.
  const int rows = !packed ? window : bad ? 0 : n;
  if (packed) {
    int sum = 0;
    for (int t = threadIdx.x; t < s; t += blockDim.x) sum += bad_length(seq_lens[t], n_valid[t]) ? 0 : n_valid[t];
    if (sum) atomicAdd(&before, sum);
  }
  if (!bad) {
    const int blocks = (L + n + LLM42_KV_BLOCK - 1) / LLM42_KV_BLOCK;   // <= max_blocks_per_seq (host checked)
    for (int b = threadIdx.x; b < blocks; b += blockDim.x) {
      const int id = block_table[(size_t)s * max_blocks_per_seq + b];
      if (id < 0 || id >= num_blocks) bad |= LLM42_SEQ_BAD_BLOCK;
    }
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const int t = candidates[(size_t)s * window + i];
      if (t < 0 || t >= vocab) bad |= LLM42_SEQ_BAD_TOKEN;
    }
  }
  if (bad) atomicOr(&status, bad);   // integer OR: order-free
  __syncthreads();
  const int st = status, base = packed ? before : s * window;
  for (int i = threadIdx.x; i < window; i += blockDim.x) {
    if (out_tokens) out_tokens[(size_t)s * window + i] = -1;   // overwritten by the arg-max merge for rows that take part
    if (i >= rows) continue;
    const int row = base + i;
    const bool part = st == 0 && i < n;
    row_pos[row] = part ? L + i : -1;
    row_seq[row] = row_tag(s, i);
    // where the row's K and V go (a block id that passed the check above), for the QKV epilogue
    row_blk[row] = part ? block_table[(size_t)s * max_blocks_per_seq + ((L + i) >> 4)] : 0;
  }
  // rows beyond those of the sequences, which only pad the GEMM grid: the last sequence's workgroup knows where they begin
  // (a launch of their own took 4 us of the smallest passes)
  if (s == (int)gridDim.x - 1) {
    for (int row = base + rows + (int)threadIdx.x; row < m_pad; row += blockDim.x) {
      row_pos[row] = -1;
      row_seq[row] = 0;
      row_blk[row] = 0;
    }
  }
  // the rotary factors of every live row, laid out by row so that the QKV epilogue finds them without
  // knowing the position first
  if (st == 0) {
    for (int e = threadIdx.x; e < n * half_dim; e += blockDim.x) {
      const int i = e / half_dim, j = e - i * half_dim;
      row_rope[(size_t)(base + i) * half_dim + j] = rope[(size_t)(L + i) * half_dim + j];
    }
  }
  // Nothing writes the attention output of rows that take no part: give them zeros once, so that everything downstream of
  // them stays finite.
  if (st != 0 || n < rows) {
    const int chunks = d_attn / 8;
    for (int e = threadIdx.x; e < rows * chunks; e += blockDim.x) {
      const int i = e / chunks, c8 = e - i * chunks;
      if (st != 0 || i >= n) *(uint4*)(attn_zero + pk_off(base + i, c8 * 8, d_attn)) = make_uint4(0, 0, 0, 0);
    }
  }
  if (threadIdx.x == 0) {
    ws_len[s] = st == 0 && n > 0 ? L : -1;
    ws_n[s] = seq_tag(st == 0 ? n : 0, base);
    if (seq_status) seq_status[s] = status_or ? (seq_status[s] | st) : st;
    int slot = -1;
    for (int j = 0; j < n_dump; ++j)
      if (dump_seq_ids[j] == s) slot = j;
    dump_slot[s] = slot;
  }
}

// Prefill, pass `chunk_index`: cuts the next `window` prompt tokens of every sequence into the
// candidate rows of one verifier pass.  One workgroup per sequence.
__global__ void prefill_window_kernel(const int32_t* __restrict__ prompt_tokens, const int32_t* __restrict__ prompt_offsets,
                                      const int32_t* __restrict__ seq_lens, int window, int chunk_index,
                                      int max_prompt_len, int32_t* __restrict__ cand, int32_t* __restrict__ n_valid,
                                      int32_t* __restrict__ lens_now, int32_t* __restrict__ seq_status,
                                      int32_t* __restrict__ out_next) {
  const int s = blockIdx.x;
  const int off = prompt_offsets[s], len = prompt_offsets[s + 1] - off;
  const int start = chunk_index * window;
  const bool bad = off < 0 || len < 0 || len > max_prompt_len;
  const int n = bad ? 0 : min(max(len - start, 0), window);
  for (int i = threadIdx.x; i < window; i += blockDim.x) cand[(size_t)s * window + i] = i < n ? prompt_tokens[off + start + i] : 0;
  if (threadIdx.x == 0) {
    n_valid[s] = n;
    lens_now[s] = seq_lens[s] + (n > 0 ? start : 0);
    if (chunk_index == 0) {
      if (seq_status) seq_status[s] = bad ? LLM42_SEQ_BAD_LENGTH : 0;
      out_next[s] = -1;
    }
  }
}

// The last prompt token of every sequence, carried from the pass that holds it to the one tail of the model that runs
// after all passes: its attention output and residual stream at the last layer move to row `s` of the tail's buffers.
// One workgroup per tail row; pass 0 clears every row that it does not fill (position -1: takes no part).  A sequence
// that failed a check in this pass or an earlier one keeps -1.
__global__ __launch_bounds__(256) void prefill_gather_kernel(const int32_t* __restrict__ prompt_offsets, int window,
                                                             int chunk_index, int num_seqs, int max_prompt_len,
                                                             const int32_t* __restrict__ seq_status,
                                                             const int32_t* __restrict__ seq_n,
                                                             const int32_t* __restrict__ row_pos,
                                                             const uint16_t* __restrict__ attn, int d_attn,
                                                             const float* __restrict__ resid, int d,
                                                             ResidLayout rl, ResidLayout tail_rl, int32_t* __restrict__ tail_pos, int32_t* __restrict__ tail_seq,
                                                             uint16_t* __restrict__ tail_attn, float* __restrict__ tail_resid) {
  const int s = blockIdx.x;
  int row = -1;
  if (s < num_seqs) {
    const int len = prompt_offsets[s + 1] - prompt_offsets[s];
    const int last = len - 1 - chunk_index * window;      // row of the last prompt token in this pass
    if (len > 0 && len <= max_prompt_len && last >= 0 && last < window && tag_rows(seq_n[s]) > last) row = tag_base(seq_n[s]) + last;
  }
  if (row < 0 && chunk_index > 0) return;                 // filled by another pass
  const bool live = row >= 0 && row_pos[row] >= 0 && seq_status[s] == 0;
  if (threadIdx.x == 0) {
    tail_pos[s] = live ? row_pos[row] : -1;
    tail_seq[s] = row_tag(s < num_seqs ? s : 0, 0);
  }
  for (int c = threadIdx.x * 8; c < d_attn; c += 256 * 8)
    *(uint4*)(tail_attn + pk_off(s, c, d_attn)) = live ? *(const uint4*)(attn + pk_off(row, c, d_attn)) : make_uint4(0, 0, 0, 0);
  for (int f = threadIdx.x * 4; f < d; f += 256 * 4)
    *(f32x4*)(tail_resid + tail_rl.off(s, f, d)) = live ? *(const f32x4*)(resid + rl.off(row, f, d)) : (f32x4){0.f, 0.f, 0.f, 0.f};
}

// One wave per 16 rows x 32 features of the residual stream: lane
// (row = lane % 16, g = lane / 16) converts 8 features of its row's embedding to
// fp32 (exact).  Dead rows get zeros so that everything downstream stays finite.
__global__ void embed_kernel(const uint16_t* __restrict__ table, const int32_t* __restrict__ candidates,
                             const int32_t* __restrict__ row_pos, const int32_t* __restrict__ row_seq, int window, int d,
                             float* __restrict__ resid,
                             ResidLayout rl) {
  const int col_tiles = d / 32;
  const size_t tile = (size_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  const int lane = threadIdx.x & 63;
  const int rb = (int)(tile / col_tiles), cb = (int)(tile % col_tiles);
  const int row = rb * 16 + (lane & 15);
  const int feat = cb * 32 + (lane >> 4) * 8;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row_pos[row] >= 0) {   // (also set for the rows that only pad)
    const int tag = row_seq[row], tok = candidates[(size_t)tag_seq(tag) * window + tag_index(tag)];
    v = *(const uint4*)(table + (size_t)tok * d + feat);
  }
  f32x4 lo = {bf16_bits_to_f32(v.x & 0xFFFFu), bf16_bits_to_f32(v.x >> 16), bf16_bits_to_f32(v.y & 0xFFFFu),
              bf16_bits_to_f32(v.y >> 16)};
  f32x4 hi = {bf16_bits_to_f32(v.z & 0xFFFFu), bf16_bits_to_f32(v.z >> 16), bf16_bits_to_f32(v.w & 0xFFFFu),
              bf16_bits_to_f32(v.w >> 16)};
  *(f32x4*)(resid + rl.off(row, feat, d)) = lo;
  *(f32x4*)(resid + rl.off(row, feat + 4, d)) = hi;
}

// Sum of the 64 per-lane partial sums of squares of a row (lane w*4+g owns p[w][g]) in the fixed
// order stated at rmsnorm_kernel, and the row's 1 / sqrt(mean square + eps).
__device__ inline float row_inv_rms(float ss, int d, float eps) {
  ss += __shfl_xor(ss, 1);
  ss += __shfl_xor(ss, 2);
  float total = __shfl(ss, 0);
#pragma unroll
  for (int ww = 1; ww < 16; ++ww) total += __shfl(ss, ww * 4);
  return 1.0f / __builtin_sqrtf(total / (float)d + eps);
}

// y[f .. f+7] = bf16(x * inv * gain), written into the tile layout; yr points at the row's feature 0.
__device__ inline void emit_normed(uint4* yr, int f, const f32x4 a, const f32x4 b, const uint4 gv, float inv) {
  uint4 o;
  o.x = pack2_bf16(a[0] * inv * bf16_bits_to_f32(gv.x & 0xFFFFu), a[1] * inv * bf16_bits_to_f32(gv.x >> 16));
  o.y = pack2_bf16(a[2] * inv * bf16_bits_to_f32(gv.y & 0xFFFFu), a[3] * inv * bf16_bits_to_f32(gv.y >> 16));
  o.z = pack2_bf16(b[0] * inv * bf16_bits_to_f32(gv.z & 0xFFFFu), b[1] * inv * bf16_bits_to_f32(gv.z >> 16));
  o.w = pack2_bf16(b[2] * inv * bf16_bits_to_f32(gv.w & 0xFFFFu), b[3] * inv * bf16_bits_to_f32(gv.w >> 16));
  yr[(f >> 5) * 64 + ((f & 31) >> 3) * 16] = o;
}

// The pending halves of a split GEMM added to U tiles (t0, t0 + 16, ...) of a row's residual stream, which go back to
// memory: old + (p0 + p1), as everywhere.  G tiles at a time: both halves of all 16 tiles of d 8192 do not fit the registers.
template <int U, int G = (U > 8 ? 4 : U)>
__device__ __forceinline__ void add_pending(float* __restrict__ xr, const float* __restrict__ p0, const float* __restrict__ p1,
                                            int fs, int t0, int g, f32x4 (&a)[U], f32x4 (&b)[U]) {
  static_assert(U % G == 0, "whole groups of tiles");
#pragma unroll
  for (int v = 0; v < U; v += G) {
    f32x4 q0[G], q1[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int o = ((t0 + (v + u) * 16) * 8 + g * 2) * fs;
      q0[u] = *(const f32x4*)(p0 + o) + *(const f32x4*)(p1 + o);
      q1[u] = *(const f32x4*)(p0 + o + fs) + *(const f32x4*)(p1 + o + fs);
    }
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int o = ((t0 + (v + u) * 16) * 8 + g * 2) * fs;
      a[v + u] = a[v + u] + q0[u];
      b[v + u] = b[v + u] + q1[u];
      *(f32x4*)(xr + o) = a[v + u];
      *(f32x4*)(xr + o + fs) = b[v + u];
    }
    if (v + G < U) __builtin_amdgcn_sched_barrier(0);
  }
}

// RMSNorm, one wave per row (1 or 4 rows per workgroup); fp32 residual stream in, bf16
// tile layout (the next GEMM's activation operand) out.
// Reduction schedule per row (a function of d only): 64 partial sums p[w][g],
// w = 0..15, g = 0..3; p[w][g] accumulates, in ascending feature order, the squares
// of features t*32 + g*8 .. +7 for t = w, w+16, w+32, ...; then per w the four g
// are added as (p[w][g] + p[w][g^1]) + (p[w][g^2] + p[w][g^3]), and the 16 results
// are added in ascending w.  Lane w*4+g of the row's wave owns p[w][g].
// PEND: the residual GEMM before left its two k-halves in p0 and p1 instead of adding them: the stream is
// x + (p0 + p1), and goes back to x.  (A pass over the stream that reads it anyway; the combining launch that it replaces
// was 4 us at 256 rows and 20 us at 2048, twice a layer.)
template <bool PEND>
__global__ __launch_bounds__(256) void rmsnorm_kernel(float* __restrict__ x, const float* __restrict__ p0,
                                                      const float* __restrict__ p1, ResidLayout rl,
                                                      const uint16_t* __restrict__ gain,
                                                      uint16_t* __restrict__ y, int m_pad, int d, float eps) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= m_pad) return;
  const int w = lane >> 2, g = lane & 3;
  const int col_tiles = d / 32;
  constexpr int U = 8;                                   // tiles in flight per lane
  const int full = col_tiles / (16 * U);                 // rounds in which every lane has U tiles
  const size_t ro = rl.off(row, 0, d);
  const int fs = rl.fs;
  float* xr = x + ro;                                    // features f .. f + 3 of this row: xr + (f / 4) * fs
  uint4* yr = (uint4*)(y + pk_off(row, 0, d));           // 8 features from f (f % 8 == 0): yr + (f/32)*64 + ((f%32)/8)*16
  float ss = 0.f;
  // (no load sits behind a per-load condition: the compiler would serialise such loads)
  if (full == 1 && col_tiles == 16 * U) {
    // d = 4096: the lane's whole share of the row (and of the gains) stays in registers
    f32x4 a[U], b[U];
    uint4 gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = (u * 16 + w) * 32 + g * 8;
      a[u] = *(const f32x4*)(xr + (f >> 2) * fs);
      b[u] = *(const f32x4*)(xr + (f >> 2) * fs + fs);
      gv[u] = *(const uint4*)(gain + f);
    }
    if (PEND) add_pending<U>(xr, p0 + ro, p1 + ro, fs, w, g, a, b);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(a[u][i], a[u][i], ss);
#pragma unroll
      for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(b[u][i], b[u][i], ss);
    }
    const float inv = row_inv_rms(ss, d, eps);
#pragma unroll
    for (int u = 0; u < U; ++u) emit_normed(yr, (u * 16 + w) * 32 + g * 8, a[u], b[u], gv[u], inv);
    return;
  }
  for (int rd = 0; rd < full; ++rd) {
    f32x4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = ((rd * U + u) * 16 + w) * 32 + g * 8;
      a[u] = *(const f32x4*)(xr + (f >> 2) * fs);
      b[u] = *(const f32x4*)(xr + (f >> 2) * fs + fs);
    }
    if (PEND) add_pending<U>(xr, p0 + ro, p1 + ro, fs, rd * U * 16 + w, g, a, b);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(a[u][i], a[u][i], ss);
#pragma unroll
      for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(b[u][i], b[u][i], ss);
    }
  }
  for (int t = full * U * 16 + w; t < col_tiles; t += 16) {
    const int f = t * 32 + g * 8;
    f32x4 a[1] = {*(const f32x4*)(xr + (f >> 2) * fs)}, b[1] = {*(const f32x4*)(xr + (f >> 2) * fs + fs)};
    if (PEND) add_pending<1>(xr, p0 + ro, p1 + ro, fs, t, g, a, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(a[0][i], a[0][i], ss);
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(b[0][i], b[0][i], ss);
  }
  const float inv = row_inv_rms(ss, d, eps);
  for (int rd = 0; rd < full; ++rd) {
    f32x4 a[U], b[U];
    uint4 gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = ((rd * U + u) * 16 + w) * 32 + g * 8;
      a[u] = *(const f32x4*)(xr + (f >> 2) * fs);
      b[u] = *(const f32x4*)(xr + (f >> 2) * fs + fs);
      gv[u] = *(const uint4*)(gain + f);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) emit_normed(yr, ((rd * U + u) * 16 + w) * 32 + g * 8, a[u], b[u], gv[u], inv);
  }
  for (int t = full * U * 16 + w; t < col_tiles; t += 16) {
    const int f = t * 32 + g * 8;
    emit_normed(yr, f, *(const f32x4*)(xr + (f >> 2) * fs), *(const f32x4*)(xr + (f >> 2) * fs + fs),
                *(const uint4*)(gain + f), inv);
  }
}

// RMSNorm at d = 512 U (U = 2, 4, 8, 16): one workgroup of 64 R threads per R neighbouring rows, thread
// (w, g, r) owning the partial sum p[w][g] of row r - the same 64 partials per row, accumulated in
// the same order and combined in the same tree as in rmsnorm_kernel, so the bits are the same; only
// the work distribution differs.  R (see launch_rmsnorm) trades CUs at work against the length of the
// contiguous runs (16 R bytes) that a workgroup writes in the tile layout, and reads where the rows are interleaved.
template <int R, int U, bool PEND>
__global__ __launch_bounds__(64 * R) void rmsnorm_block_kernel(float* __restrict__ x, const float* __restrict__ p0,
                                                               const float* __restrict__ p1, ResidLayout rl,
                                                               const uint16_t* __restrict__ gain,
                                                               uint16_t* __restrict__ y, float eps,
                                                               const int32_t* __restrict__ live) {
  if (live && (int)blockIdx.x * R >= live_rows(live)) return;      // packed rows: only what pads (workgroup-uniform)
  constexpr int D = 512 * U;                             // U tiles of 32 features per thread: t = u * 16 + w
  constexpr bool kLateGain = PEND && U > 8;              // (the gains of d 8192 have no registers before the halves are added)
  __shared__ float part[64][R];
  __shared__ float inv_s[R];
  const int r = threadIdx.x % R, wg = threadIdx.x / R, w = wg >> 2, g = wg & 3;
  const int row = blockIdx.x * R + r;
  const size_t ro = rl.off(row, 0, D);
  const int fs = rl.fs;
  float* xr = x + ro;
  uint4* yr = (uint4*)(y + pk_off(row, 0, D));
  f32x4 a[U], b[U];
  uint4 gv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int f = (u * 16 + w) * 32 + g * 8;
    a[u] = *(const f32x4*)(xr + (f >> 2) * fs);
    b[u] = *(const f32x4*)(xr + (f >> 2) * fs + fs);
    if (!kLateGain) gv[u] = *(const uint4*)(gain + f);
  }
  if (PEND) add_pending<U>(xr, p0 + ro, p1 + ro, fs, w, g, a, b);
  if (kLateGain) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) gv[u] = *(const uint4*)(gain + (u * 16 + w) * 32 + g * 8);
  }
  float ss = 0.f;
#pragma unroll
  for (int u = 0; u < U; ++u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(a[u][i], a[u][i], ss);
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(b[u][i], b[u][i], ss);
  }
  part[wg][r] = ss;
  __syncthreads();
  if (threadIdx.x < R) {
    float total = 0.f;
#pragma unroll
    for (int ww = 0; ww < 16; ++ww) {
      const float s4 = (part[ww * 4][r] + part[ww * 4 + 1][r]) + (part[ww * 4 + 2][r] + part[ww * 4 + 3][r]);
      total = ww == 0 ? s4 : total + s4;
    }
    inv_s[r] = 1.0f / __builtin_sqrtf(total / (float)D + eps);
  }
  __syncthreads();
  const float inv = inv_s[r];
#pragma unroll
  for (int u = 0; u < U; ++u) emit_normed(yr, (u * 16 + w) * 32 + g * 8, a[u], b[u], gv[u], inv);
}

}  // namespace

void launch_prepare(const llm42_model* m, const llm42_kv_cache* kv, const int32_t* seq_lens,
                    const int32_t* candidates, const int32_t* n_valid, int num_seqs, int window,
                    int max_context, const int32_t* dump_seq_ids, int n_dump, int32_t* out_tokens,
                    int32_t* seq_status, const Workspace& ws, hipStream_t st, bool prefill_pass) {
  prepare_kernel<<<num_seqs, 256, 0, st>>>(seq_lens, candidates, n_valid, kv->block_table, kv->max_blocks_per_seq,
                                          kv->num_blocks, window, max_context, m->cfg.vocab, dump_seq_ids, n_dump,
                                          out_tokens, seq_status, ws.row_pos, ws.row_seq, ws.seq_len, ws.seq_n,
                                          ws.dump_slot, (const float2*)m->rope, m->cfg.head_dim / 2, ws.row_blk,
                                          ws.row_rope, prefill_pass ? 0 : 1, prefill_pass ? 1 : 0,
                                          ws.attn, m->d_attn, ws.live != nullptr, ws.m_pad);
}

void launch_prefill_window(const int32_t* prompt_tokens, const int32_t* prompt_offsets, const int32_t* seq_lens,
                           int num_seqs, int window, int chunk_index, int max_prompt_len, int32_t* cand,
                           int32_t* n_valid, int32_t* lens_now, int32_t* seq_status, int32_t* out_next, hipStream_t st) {
  prefill_window_kernel<<<num_seqs, 64, 0, st>>>(prompt_tokens, prompt_offsets, seq_lens, window, chunk_index, max_prompt_len, cand,
                                                 n_valid, lens_now, seq_status, out_next);
}

void launch_prefill_gather(const llm42_model* m, const int32_t* prompt_offsets, int num_seqs, int window, int chunk_index,
                           int max_prompt_len, const int32_t* seq_status, const Workspace& ws, const Workspace& tail,
                           hipStream_t st) {
  prefill_gather_kernel<<<tail.m_pad, 256, 0, st>>>(prompt_offsets, window, chunk_index, num_seqs, max_prompt_len, seq_status,
                                                    ws.seq_n, ws.row_pos, ws.attn, m->d_attn, ws.resid, m->cfg.d_model, ws.rl, tail.rl, tail.row_pos,
                                                    tail.row_seq, tail.attn, tail.resid);
}

void launch_embed(const llm42_model* m, const int32_t* candidates, int window, const Workspace& ws, hipStream_t st) {
  const int tiles = ws.m_pad / 16 * (m->cfg.d_model / 32);   // a multiple of 4 (d_model % 128 == 0 is checked)
  embed_kernel<<<tiles / 4, 256, 0, st>>>(m->embed, candidates, ws.row_pos, ws.row_seq, window, m->cfg.d_model, ws.resid, ws.rl);
}

template <bool PEND>
static void launch_norm(float* x, const float* p0, const float* p1, ResidLayout rl, const uint16_t* gain, uint16_t* y, int m_pad, int d,
                        float eps, const int32_t* live, hipStream_t st) {
  // us per launch behind a launch that wrote the operands (they come from other XCDs' writes then), by the rows per workgroup
  // (1: a wave per row, 4 waves a workgroup from 512 rows on), without | with pending halves:
  //                  row-major                                 token blocks interleaved
  //           1            2            4            8         |  4            8            16
  //    128    3.4 |  4.2   3.4 |  5.0   4.6 |  9.3   6.8 | 16.6 |  4.1 |  7.9   4.4 |  7.8   6.6 | 14.4
  //    256    5.3 |  7.7   4.7 |  7.6   5.7 | 11.8   7.9 | 19.0 |  5.5 |  9.4   5.5 | 10.2   7.7 | 16.3
  //    512    7.7 | 10.9   7.4 | 12.5   7.4 | 12.7   9.6 | 19.5 |  8.2 | 11.6   7.3 | 11.4   9.4 | 20.2
  //   1024   12.0 | 19.9  11.7 | 16.8  10.8 | 19.4  12.3 | 23.9 | 10.4 | 20.9  10.7 | 13.7  12.4 | 20.2
  //   2048   19.8 | 28.5  20.0 | 27.0  17.8 | 29.3  18.0 | 27.0 | 15.5 | 43.5  11.5 | 25.8  19.6 | 24.1
  //   4096   27.1 | 52.0  26.9 | 53.4  25.2 | 52.2  24.6 | 52.2 | 29.2 | 82.3  21.6 | 47.3  23.8 | 46.2
  // Few rows are bound by what a CU pulls from beyond its L2 (20 - 25 GB/s) and want as many CUs as there are, many rows by
  // the length of the runs that they read and write.
  // The widths 1024, 2048 and 8192 follow beyond 512 rows, where a wave per row reads pieces of 16 bytes (norms of one layer and
  // the final one, halves of two projections left to two of the three, wave per row with the halves added before -> this with
  // them: 2048 rows d 2048 44.6 + 2 adding launches -> 38.3, d 8192 197.7 + 2 -> 148.9, d 1024 27.4 + 2 -> 26.8; d 8192 with the
  // halves added in groups that leave no register spilled, two layers of 528 rows 119 -> 107, of 768 128 -> 120).
  const bool rows8 = m_pad > 512;
  auto block8 = [&](auto u) { rmsnorm_block_kernel<8, decltype(u)::value, PEND><<<m_pad / 8, 512, 0, st>>>(x, p0, p1, rl, gain, y, eps, live); };
  if (rows8 && d == 1024) block8(std::integral_constant<int, 2>{});
  else if (rows8 && d == 2048) block8(std::integral_constant<int, 4>{});
  else if (rows8 && d == 4096) block8(std::integral_constant<int, 8>{});
  else if (rows8 && d == 8192) block8(std::integral_constant<int, 16>{});
  else if (d == 4096 && m_pad > 128 && !(PEND && m_pad > 256))
    rmsnorm_block_kernel<2, 8, PEND><<<m_pad / 2, 128, 0, st>>>(x, p0, p1, rl, gain, y, eps, nullptr);
  else if (m_pad <= 256) rmsnorm_kernel<PEND><<<m_pad, 64, 0, st>>>(x, p0, p1, rl, gain, y, m_pad, d, eps);
  else rmsnorm_kernel<PEND><<<(m_pad + 3) / 4, 256, 0, st>>>(x, p0, p1, rl, gain, y, m_pad, d, eps);
}

void launch_rmsnorm(bool pending, const uint16_t* gain, int d, float eps, const Workspace& ws, hipStream_t st) {
  const float* p0 = ws.split_part;
  if (pending) launch_norm<true>(ws.resid, p0, p0 + (size_t)ws.m_pad * d, ws.rl, gain, ws.normed, ws.m_pad, d, eps, ws.live, st);
  else launch_norm<false>(ws.resid, nullptr, nullptr, ws.rl, gain, ws.normed, ws.m_pad, d, eps, ws.live, st);
}
