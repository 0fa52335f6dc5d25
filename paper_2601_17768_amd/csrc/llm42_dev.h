// Device-side helpers and the launcher interface between the translation units
// of the verifier library (gfx950 only).
//
// Packed operand layout ("tile layout") used for every GEMM operand in HBM:
// a matrix [R][C] (R padded to 16, C padded to 32) is cut into tiles of
// 16 rows x 32 columns (1 KiB of bf16).  Tiles are stored row-block major
// (all column tiles of a 16-row block are contiguous) and inside a tile element
// (r, c) sits at ((c / 8) * 16 + r) * 8 + c % 8.  A tile is exactly one operand
// of v_mfma_f32_16x16x32_bf16 in lane order (lane = (c / 8) * 16 + r holds the
// 8 consecutive columns c & ~7 .. ), so a wave fetches an operand with one
// fully coalesced 16-byte-per-lane load and no shuffling.
//
// GEMMs are computed transposed, D[feature][token] = sum_k W[feature][k] X[token][k]:
// weights are the A operand, activations the B operand.  In the result tile a
// lane (token = lane % 16, g = lane / 16) holds features g*4 .. g*4+3 of its
// token, i.e. four consecutive features, which it can store straight back into
// the tile layout of the next GEMM's activation operand.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/llm42.h"
#include "../../include/llm42_measure.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;


__host__ __device__ inline size_t pk_off(int r, int c, int c_padded) {
  return ((size_t)(r >> 4) * (size_t)(c_padded >> 5) + (size_t)(c >> 5)) * 512 +
         (size_t)((((c & 31) >> 3) * 16 + (r & 15)) * 8 + (c & 7));
}

// Residual stream and the halves of a split GEMM: fp32, in pieces of four consecutive features of a row (what a GEMM's lane
// owns).  Few rows: row-major, rs = n and fs = 4, so that a row of the RMSNorm is one contiguous run.  Many rows: the 16
// rows of a token block interleaved, rs = 4 and fs = 64, so that a wave of a GEMM's epilogue accesses 1 KiB in one run.
struct ResidLayout {
  int rs, fs;   // floats from a row to the next of its block of 16, from a group of four features to the next
  __host__ __device__ size_t off(int row, int feat, int n) const {
    return (size_t)(row >> 4) * 16 * (size_t)n + (size_t)((row & 15) * rs) + (size_t)(feat >> 2) * fs + (feat & 3);
  }
};

__device__ inline float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// round-to-nearest-even on the bit pattern (inputs are finite here)
__device__ inline uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}
// the same rounding for two values at once, by the hardware conversion (one instruction on gfx950)
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ inline uint32_t pack2_bf16(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// V tile of the KV cache: [feature block of 16][token group of 4][feature][4 tokens], the order in
// which the lanes of a P V operand read it (8 contiguous bytes per lane, 512 per wave).
__host__ __device__ inline int v_tile_off(int f, int t) {
  return (((f >> 4) * 4 + (t >> 2)) * 16 + (f & 15)) * 4 + (t & 3);
}

__device__ inline f32x4 mfma16(const bf16x8 a, const bf16x8 b, const f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// model and per-call plan (host side)
// ---------------------------------------------------------------------------
struct llm42_model {
  llm42_config cfg;
  int device;       // HIP device the model lives on
  int num_cus;      // compute units of that device
  int group;        // q heads per kv head
  int n_qkv;        // (n_q_heads + 2 n_kv_heads) * head_dim
  int d_attn;       // n_q_heads * head_dim
  int ffn_k;        // d_ffn padded to 32: K of the down projection
  int gu_blocks;    // packed gate/up feature blocks (16 packed rows = 8 hidden features)
  uint16_t* arena;  // one device allocation holding everything below
  size_t arena_bytes;
  uint16_t* embed;  // [vocab][d] row-major (gathered, never multiplied)
  uint16_t* final_norm;
  uint16_t* lm_head;  // packed [vocab][d]
  struct Layer {
    uint16_t *attn_norm, *wqkv, *wo, *ffn_norm, *wgu, *wdown;
  }* layers;          // host array
  float* rope;        // [max_position][head_dim/2][2] (cos, sin), fp32
};

// (at most 65536 rows, windows of at most 512)
// Order of the query rows of a (sequence, kv head): `t` tokens at a time (a power of two that divides the window, and t * group
// divides 16; else 1), heads outside: rows that a partly filled window lacks come last, and neighbouring tokens of a head, which
// the QKV projection computes together, lie side by side (in the plain order of tokens, then heads, Q was written in 16-byte pieces:
// 128 sequences x window 32, us a layer: attention 556, QKV 195.6; so 540 and 192.4).
struct RowOrder {
  int group, t;
  __host__ __device__ int row(int i, int h) const { return (i & -t) * group + h * t + (i & (t - 1)); }
  __host__ __device__ int token(int r) const { return r / (t * group) * t + (r & (t - 1)); }
  __host__ __device__ int head(int r) const { return r % (t * group) / t; }
};
inline RowOrder row_order(int group, int window) {
  int t = 16;
  while (t > 1 && (16 % (t * group) || window % t)) t /= 2;
  return {group, t};
}
__host__ __device__ inline int row_tag(int s, int i) { return s << 10 | i; }
__host__ __device__ inline int tag_seq(int tag) { return tag >> 10; }
__host__ __device__ inline int tag_index(int tag) { return tag & 1023; }
__host__ __device__ inline int seq_tag(int n, int base) { return base << 10 | n; }
__host__ __device__ inline int tag_rows(int tag) { return tag & 1023; }
__host__ __device__ inline int tag_base(int tag) { return tag >> 10; }
// Packed rows end where those of the last sequence do (its tag, Workspace::live, says where).
__device__ inline int live_rows(const int32_t* live) { return tag_base(*live) + tag_rows(*live); }

// How a pass of more than 64 rows runs one of its GEMMs (see plan_gemms): tile, the number of rows that have a launch of their
// own beside it (0: none) and the tile of that one, and whether the halves of a split one follow each other.
struct GemmPlan {
  int tile, fewer, fewer_tile;
  bool in_turn;
};
enum GemmKind { GEMM_QKV, GEMM_O, GEMM_GATE_UP, GEMM_DOWN, GEMM_LM_HEAD, GEMM_KINDS };

// Workspace carving, identical in llm42_workspace_bytes and llm42_verify_window.
struct Workspace {
  int num_cus;    // compute units of the device
  int m_rows;     // num_seqs * window
  int m_pad;      // rows padded for the GEMM grid
  int r_pad;      // query rows per (seq, kv head) padded to 16
  int part_rows;  // rows of an attention partial slot
  int attn_units; // attention partial slots per row (chunks or supers, see attention.hip)
  bool attn_super; // one workgroup per super (many sequences) instead of per chunk
  bool attn_direct; // every sequence fits one super: the attention kernel writes the final output, no merge pass
  bool attn_seq;    // the call may take whole sequences as attention items (the plan kernel decides from the lengths)
  bool attn_split;  // whatever the three above say: a workgroup per (sequence, kv head, block of 16 query rows), chunks
                    // dealt to its waves, output written by the same launch
  bool attn_waves;  // whatever those above say: a wave per chunk, and the merge pass (see wave_use)
  bool attn_choice; // whatever those above say: a wave per chunk or a workgroup per super, as the plan kernel decides from the lengths
  bool attn_list;   // the launches take their items from the plan kernel's list (else: sequence by sequence)
  bool full;        // every window of the call is full: attention by 8 waves need not test for rows that are not there
  bool batch_chosen; // off the fixed schedule (fast-path decode step, cost-of-determinism measurement): the batch may
                     // choose the split of the residual projections and the attention partials
  // Rows of a pass: sequence s has rows base(s) .. base(s) + n(s) - 1.  With n_valid the rows are packed - base(s) is the sum
  // of the counts before - and live_rows(live) of them exist; without, base(s) = s * window and `live` is null.
  int32_t *row_pos, *row_seq;        // position (-1: takes no part), row_tag(s, i)
  int32_t *seq_len, *seq_n;          // cached length (-1: takes no part), seq_tag(n, base)
  int32_t *dump_slot;
  const int32_t* live;               // the last sequence's entry of seq_n
  GemmPlan gemm[GEMM_KINDS];
  bool partly_filled;                // packed rows of a verifier pass (a prefill pass's are packed too, but mostly all there)
  int32_t* row_blk;    // physical KV block that holds the row's position (0 for dead rows)
  float2* row_rope;    // [m_pad][head_dim/2] (cos, sin) at the row's position
  float* resid;
  ResidLayout rl;      // of resid and split_part
  uint16_t *normed, *q, *attn, *hidden;
  float *part_acc, *part_ml;
  int4* attn_items;     // (sequence, unit, length, seq_tag) of every unit that holds keys, built once per call
  int32_t* attn_ctrl;   // [0] number of items, [1 + layer] work queue counter of that layer's attention launch,
                        // [1 + n_layers] 1 if the items are whole sequences
  size_t attn_ctrl_offset;   // byte offset of attn_ctrl in the workspace
  float* split_part;   // fp32 halves of a split GEMM, [2][m_pad][d_model]
  float2* amax;   // [m_pad][vocab/16 or fewer] (value, index bits)
  size_t bytes;
};

// ---------------------------------------------------------------------------
// launchers (each defined in the .hip file that holds its kernel)
// ---------------------------------------------------------------------------
void launch_pack_plain(const uint16_t* src, uint16_t* dst, int rows, int cols, int cols_padded, hipStream_t st);
void launch_pack_qkv(const uint16_t* wq, const uint16_t* wk, const uint16_t* wv, uint16_t* dst,
                     const llm42_config& c, hipStream_t st);
void launch_pack_gate_up(const uint16_t* wg, const uint16_t* wu, uint16_t* dst, int d_ffn, int gu_blocks,
                         int d_model, hipStream_t st);

void launch_prepare(const llm42_model* m, const llm42_kv_cache* kv, const int32_t* seq_lens,
                    const int32_t* candidates, const int32_t* n_valid, int num_seqs, int window,
                    int max_context, const int32_t* dump_seq_ids, int n_dump, int32_t* out_tokens,
                    int32_t* seq_status, const Workspace& ws, hipStream_t st, bool prefill_pass);
void launch_prefill_window(const int32_t* prompt_tokens, const int32_t* prompt_offsets, const int32_t* seq_lens,
                           int num_seqs, int window, int chunk_index, int max_prompt_len, int32_t* cand,
                           int32_t* n_valid, int32_t* lens_now, int32_t* seq_status, int32_t* out_next, hipStream_t st);
void launch_prefill_gather(const llm42_model* m, const int32_t* prompt_offsets, int num_seqs, int window, int chunk_index,
                           int max_prompt_len, const int32_t* seq_status, const Workspace& ws, const Workspace& tail,
                           hipStream_t st);
void launch_embed(const llm42_model* m, const int32_t* candidates, int window, const Workspace& ws, hipStream_t st);
// Whether the RMSNorm behind a split GEMM adds its halves to the residual stream (see launch_gemm).
inline bool norm_adds_halves(int m_pad, int d) { return m_pad <= 512 || d == 1024 || d == 2048 || d == 4096 || d == 8192; }
// pending: the last residual GEMM left its halves in split_part (what launch_gemm_residual returned)
void launch_rmsnorm(bool pending, const uint16_t* gain, int d, float eps, const Workspace& ws, hipStream_t st);

// Fills ws.gemm: the same for every layer, so chosen once per pass (the rule takes 0.3 us a GEMM, and with partly filled windows
// 1 - 13 us at 1024 - 16384 rows; a layer's ten launches take about 40).
void plan_gemms(const llm42_model* m, Workspace& ws);
void launch_gemm_qkv(const llm42_model* m, int layer, const llm42_kv_cache* kv, int window, const Workspace& ws,
                     hipStream_t st);
// true: the residual stream is not complete yet; the halves are in split_part, for the RMSNorm that follows
bool launch_gemm_residual(GemmKind kind, const uint16_t* w, const uint16_t* x, float* resid, int n, int k_padded,
                          const Workspace& ws, hipStream_t st);
void launch_gemm_swiglu(const llm42_model* m, int layer, const Workspace& ws, hipStream_t st);
// Returns the number of arg-max partials per row that it leaves in amax.
int launch_gemm_logits(const llm42_model* m, int window, float* out_logits, const llm42_sampling* sampling,
                       const Workspace& ws, hipStream_t st);

int attention_units(bool super_mode, int max_context);
bool attention_streams(const llm42_model* m, int num_seqs, const Workspace& ws);   // by the 8-wave kernel
void launch_attention_plan(const llm42_model* m, int num_seqs, int max_context, const Workspace& ws, hipStream_t st);
void launch_attention(const llm42_model* m, int layer, const llm42_kv_cache* kv, int num_seqs, int window,
                      int max_context, const Workspace& ws, hipStream_t st);
void launch_argmax_merge(int parts, int num_seqs, int window, int32_t* out_tokens, const Workspace& ws, hipStream_t st);
void launch_commit(const int32_t* candidates, const int32_t* out_tokens, const int32_t* n_valid, int num_seqs,
                   int window, int32_t* seq_lens, int32_t* committed_counts, int32_t* committed_tokens,
                   int32_t* rolled_back_counts, hipStream_t st);
