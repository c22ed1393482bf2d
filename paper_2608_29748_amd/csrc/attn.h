// Paged grouped-query attention for blocks of query rows (verify, draft, prefill).
#pragma once
#include "common.h"

namespace rt {

struct AttnArgs {
  const void* q;                 // [row][n_q_heads * head_dim], row = seq * rows_per_seq + token
  const void* kcache;            // this layer: K pages [page][kv head][token][hd]
  const void* vcache;            // this layer: V pages [page][kv head][hd][token]
  const int32_t* page_table; int max_pages;
  const int32_t* pos0;           // [seq * seq_stride] position of query token 0
  int seq_stride;
  int rows_per_seq;
  int n_seqs;
  int causal;                    // 1: key position <= query position; 0: every key below pos0 + rows_per_seq
  int n_q_heads, n_kv_heads, head_dim;
  int splits;                    // key-range splits per (seq, kv head, row block)
  int slots, fit;                // workgroups per KV head, and those of one pass of the chip: see attn_slots
  int slots_each, fit_each;      // the same per unit, rounded down
  int row_blocks;                // row blocks of rb_rows (token, head) rows per sequence
  int rb_rows;                   // rows per block: 64, or 96 (bf16) when a sequence has 65..96 rows
  // Prompt passes (one key split): grid.z entry z works on the block
  // blocks[z] = {sequence, activation row of its segment's token 0, tokens of the segment,
  // position of token 0, row block within the segment, 0, 0, 0}; n_blocks of them.  pos0,
  // rows_per_seq, n_seqs and row_blocks are then unused.
  const int32_t* blocks; int n_blocks;
  // split partials: per (split, row) the running max and sum (fp32 mlpart) and the
  // split's own normalised output O / sum (opart: fp16 for bf16 models, fp32 otherwise)
  float* opart; float* mlpart;
  int32_t* plan;                 // [2][64] balanced split plan: first partial block, split count per unit
  int span;                      // bf16 kernel without the fused q / k work: balanced launches may
                                 // use the spanning plan (slots cross unit boundaries) when it
                                 // shortens the longest split; 2: whenever it is valid (test hook)
  void* out; int ldo;            // packed GEMM-operand layout of [row][n_q_heads * head_dim]; ldo = group stride
  float scale;                   // 1/sqrt(head_dim)
  // Rounds (at most 16 rows per sequence, one q|k|v slab): the q / k per-head RMSNorm,
  // RoPE and the block's K / V cache write done here instead of by qkv_post.  qkv: the
  // fp32 q|k|v projection [row][ldqkv] (q at column 0, k at q_cols, v at q_cols + kv_cols);
  // null: q comes from `q` and the block's K / V are already cached.  Every workgroup
  // normalises and rotates its own q rows; the workgroups whose chunks hold the block's
  // positions normalise and rotate the block's k rows, write k and v to the caches and
  // into their LDS stages.  Key split 0 of each unit also stores its normalised q rows to
  // q_out ([row][ldq], as qkv_post would).
  const float* qkv; int ldqkv; int q_cols, kv_cols;
  const void* q_norm; const void* k_norm;
  const float* rope; int rope_max_pos; float eps;
  void* q_out; int ldq;
};

// Query (token, head) rows handled by one workgroup: 64, or 96 for bf16 blocks of 65..96
// rows (a GQA group of 5 over a 16-token block), so that every KV head is read once.
constexpr int kAttnRows = 64;
constexpr int kAttnRowsMax = 96;
constexpr int kAttnRowsPrompt = 64;   // bf16 prompt passes
constexpr int kAttnBlockInts = 8;      // int32 per entry of AttnArgs::blocks

// Splits per unit, workgroups (slots) per KV head and, for the balanced plan, the slots per KV
// head that 256 compute units take in one pass, for a launch over n_units (sequence, row block)
// units.  `splits` is the handle's count, about one workgroup per compute unit at max_batch,
// rounded up.  `one_pass` (bf16 handles of at most 64 round rows): workgroups past 256 make the
// launch longer, as a unit that has two runs both slower or one after the other (three
// sequences x 16 rows, 11 splits against 10: 76 and 56 us of attention a round at head_dim 64;
// x 20 rows at head_dim 128 158 and 90), so a launch gets 256 / n_kv_heads slots a head where
// that is two or more a unit.  Below two a unit it keeps the full count and the balanced plan
// decides from the contexts how many to use.  Unbalanced launches take whole splits per unit.
struct AttnSlots { int splits, slots, fit, slots_each, fit_each; };
AttnSlots attn_slots(int n_units, int n_kv_heads, int splits, bool one_pass);

// Attention: attention_partials (per key split), then attention_merge (splits > 1).
template <typename T>
hipError_t attention_partials(const AttnArgs& a, hipStream_t s);
template <typename T>
hipError_t attention_merge(const AttnArgs& a, hipStream_t s);

}  // namespace rt
