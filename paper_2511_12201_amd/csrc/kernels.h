// Internal launch interface between the C-ABI layer (api.hip) and the kernel files.
#pragma once

#include "common.h"

namespace omni {

// score.hip
size_t score_queries_ws(const Layer& L);
int run_score_queries(const Layer& L, int dtype, const void* Q, const void* K, float* probe, float* scores, void* ws,
                      hipStream_t st);
int score_mean_chunks(const Layer& L);
int run_probe_keys(const Layer& L, int dtype, const void* K, float* probe, void* ws, hipStream_t st,
                   const Ragged& rg = Ragged{});

// select.hip
size_t select_ws(const Layer& L);
int run_select_queries(const Layer& L, const float* scores, int mode, float param, int* q_idx, int* q_cnt, void* ws,
                       hipStream_t st);
int run_select_kv(const Layer& L, const float* key_scores, const int* budget, int b_cap, int* kv_idx, void* ws,
                  hipStream_t st);
size_t budget_stats_ws(const Layer& L);
int run_budget_stats(const Layer& L, const float* key_scores, float recall_p, int budget_mode, double* kurt,
                     int* flattest, int* budget, float* recall, void* ws, hipStream_t st);
// Both lists of a prefill step from the two score arrays: statistics of the key scores, the cuts and lists (two
// launches, or three).
size_t select_lists_ws(const Layer& L);
int run_select_lists(const Layer& L, const Ragged& rg, const float* scores, int q_mode, float q_param, int* q_idx,
                     int* q_cnt, const float* key_scores, float recall_p, int budget_mode, double* kurt, int* flattest,
                     int* budget, float* recall, int* kv_idx, int b_cap, void* ws, hipStream_t st);
int run_visual_subset(const Layer& L, const int* kv_idx, const int* budget, int b_cap, int* vis_idx, int* vis_cnt,
                      hipStream_t st);
size_t group_subset_ws(const Layer& L);
int run_group_subset(const Layer& L, const int* kv_idx, const int* budget, int b_cap, int* grp_idx, unsigned* grp_mask,
                     int* grp_cnt, int u_cap, void* ws, hipStream_t st);

// probe.hip
size_t probe_ws(const Layer& L, int dtype, int pb);
// probe_keys / scores not null: and the probe keys and the lazy/active query scores (no extra pass over Q)
int run_probe(const Layer& L, int dtype, const void* Q, const void* K, int pb, float* key_scores, void* ws,
              hipStream_t st, float* probe_keys = nullptr, float* scores = nullptr, const Ragged& rg = Ragged{});

// pack.hip (outputs that are nullptr are skipped; bf16: Vt holds f16 values, and not both Kt and Vt in one call)
// Kn, Vn, Qn, dOn in the order of a 32x32 MFMA's A operand, [32-row block][k step][lane] of 16 bytes (lane = 32 * half + row; a
// k step is 16 bf16 or 8 fp32 values wide); fp32 without k_frag: Kn, Vn row by row
struct PackKv {
  const void *K, *V;
  int per_q_head;                // a copy per query head of the listed rows, or per KV head of all rows
  const int* src_idx;            // [.., idx_stride] token of a slot; null: the slot itself
  int idx_stride;
  const int* budget;             // null: N
  int b_cap, npad, pad_to;       // rows of a head's copy; slots are filled up with zero rows to a multiple of pad_to
  void *Kn, *Vn, *Kt, *Vt;
  int k_frag;
};
struct PackQ {
  const void *Q, *O, *dO;
  const float* lse;
  const int *q_idx, *q_cnt;
  int nqpad;
  void *Qt, *dOt, *Qn, *dOn;
  float *lse2c, *deltac;
};
// What precedes an attention kernel, in one launch: any of the packs and the passes over the lists (sched.h); none may need
// another's results.
struct Bounds;
struct Order;
struct KeyList;
int run_prepare(const Layer& L, int dtype, bool backward, const PackKv* kv, const PackQ* q, const Bounds* bn, const Order* od,
                const KeyList* kl, hipStream_t st);

// attn_fwd.hip
// products of the dense attention of a layer: what the rules between kernels for short and long sequences look at
int attention_route();                       // omni_debug_attention_route of this thread; 0: by the shape
inline bool short_route(bool by_shape) { return attention_route() ? attention_route() == 1 : by_shape; }
inline double attention_work(const Layer& L) { return (double)L.B * L.Hq * L.N * L.N * L.D * (L.causal ? 1.0 : 2.0); }
// fp32, forward and backward: 32-row items whose wavefronts share the other side (as short sequences need them), or 128-row
// items with tiles in LDS.  The long items are the faster ones once they fill the chip, which their number decides (rows of
// all heads, twice as many without the causal mask: each works twice as long); the longer the sequence, the longer the chains
// that the short items save; below 1400 tokens there is little to save and the width counts (at d = 128 one workgroup of the
// short items fills a CU).  Call in us, short / long items; batch x heads, d, N; a third of the queries and half of the keys
// kept, or all (full).  Forward and backward, below the lines: 1 x 28, 128, 1072 289 / 671 and (full) 634 / 919; 6 x 28,
// 128, 256 251 / 357 and (full) 417 / 450; 1 x 28, 128, 3500 1562 / 1983 and (full) 4712 / 4918; 1 x 8, 128, 8192 4300 /
// 4407 and (full) 6339 / 8282; above them: 8 x 28, 128, 256 319 / 385 but (full) 537 / 519; 1 x 28, 128, 4096 2002 / 2356
// but (full) 6183 / 6132; 1 x 8, 128, 10000 6226 / 5405; 1 x 28, 128, 8192 6860 / 5747 and (full) 24707 / 21438; forward
// 16 x 28, 128, 512 (full) 681 / 521.
inline bool f32_short(const Layer& L) {
  const double rows = (double)L.B * L.Hq * L.N * (L.causal ? 1.0 : 2.0);
  return short_route(L.N < 1400 ? rows * L.D <= 6.0e6 : rows <= (L.N <= 3500 ? 9.8e4 : 6.6e4));
}
size_t attn_fwd_ws(const Layer& L, int dtype, int b_cap, bool sparse);
int run_attn_fwd(const Layer& L, int dtype, const void* Q, const void* K, const void* V, const int* q_idx,
                 const int* q_cnt, const int* kv_idx, const int* budget, int b_cap, void* O, float* lse, void* ws,
                 bool sparse, hipStream_t st);

// bf16 only, block % 64 == 0: the forward pass on block lists without a gathered copy of K/V per query head
int attn_fwd_blocks_max_keys();
size_t attn_fwd_blocks_ws(const Layer& L, int cap_keys);   // cap_keys = blk_cap * block
int run_attn_fwd_blocks(const Layer& L, const void* Q, const void* K, const void* V, const int* q_idx, const int* q_cnt,
                        const int* blk_idx, const int* blk_budget, int blk_cap, int block, void* O, float* lse,
                        void* ws, hipStream_t st);

// attn_bwd.hip
size_t attn_bwd_ws(const Layer& L, int dtype, int b_cap);
int run_attn_bwd(const Layer& L, int dtype, const void* Q, const void* K, const void* V, const void* O,
                 const void* dO, const float* lse, const int* q_idx, const int* q_cnt, const int* kv_idx,
                 const int* budget, int b_cap, void* dQ, void* dK, void* dV, void* ws, hipStream_t st);
// the same on block lists walked in place (bf16): K/V of every KV head once, tiles found through a tile map
int attn_bwd_blocks_max_keys();
size_t attn_bwd_blocks_ws(const Layer& L, int cap_keys);   // cap_keys = blk_cap * block
int run_attn_bwd_blocks(const Layer& L, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const float* lse, const int* q_idx, const int* q_cnt, const int* blk_idx, const int* blk_budget,
                        int blk_cap, int block, void* dQ, void* dK, void* dV, void* ws, hipStream_t st);

void set_key_split_len(int tiles);   // attn_bwd.hip; <= 0 restores the default

// decode.hip
size_t decode_ws(const omni_decode_desc* d);
// paged form of the compacted store: Kcomp / Vcomp are a pool [pool_pages, 1 << page_shift, D] shared by all
// (batch, KV head) pairs; position u of a pair's group list lives in page page_table[pair, u >> page_shift]
struct PagePool {
  const int* page_table;   // [B*Hkv, pages_cap]; entries outside [0, pool_pages) mark pages that are not there
  int page_shift, pages_cap, pool_pages;
};
// grp_mask == nullptr: vis_idx / vis_cnt are per query head; otherwise per KV group with membership bits
int run_decode(const omni_decode_desc* d, const void* q, const void* K, const void* V, const int* ctx_len,
               const float* probe, const int* vis_idx, const int* vis_cnt, const unsigned* grp_mask, int b_cap,
               void* O, unsigned char* active, void* ws, hipStream_t st, const void* Kcomp = nullptr,
               const void* Vcomp = nullptr, const PagePool* pool = nullptr);
int run_compact_cache(const omni_decode_desc* d, const void* K, const void* V, const int* grp_idx, const int* grp_cnt,
                      int u_cap, void* Kc, void* Vc, hipStream_t st, const PagePool* pool = nullptr);

// block.hip (block-granular variant of the KV selection)
int block_scores_max_blocks();
size_t block_scores_ws(const Layer& L, int block);
int run_block_scores(const Layer& L, int dtype, const void* Q, const void* K, int block, float* out, void* ws,
                     hipStream_t st);
int run_expand_blocks(const Layer& L, const int* blk_idx, const int* blk_budget, int blk_cap, int block, int* kv_idx,
                      int* budget, int b_cap, hipStream_t st, int* tile_map = nullptr, int last_tile = 0);

// diag.hip
int run_calibration_copy(const void* src, void* dst, size_t bytes, hipStream_t st);
int run_mfma_rate(int random_operands, int iters, double* tflops, double* shader_mhz);

}  // namespace omni
