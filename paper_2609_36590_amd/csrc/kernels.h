// Internal interface between the host runtime and the gfx950 kernels of the SEED decode path.
// Nothing here is part of the public C ABI (include/seed.h).
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dispatch.h"

namespace seedk {

// ---------------------------------------------------------------------------------------------
// Weight layout ("MFMA tile" packing). A linear weight W [N, K] (nn.Linear [out, in]) is stored
// as N/16 x K/32 tiles of 16 rows x 32 columns, tile (nt, kt) at element offset
// (nt * (K/32) + kt) * 512. Inside a tile, lane l (0..63) owns 8 consecutive elements
//   W[nt*16 + (l & 15)][kt*32 + (l >> 4)*8 + j],  j = 0..7,  at offset l*8 + j,
// which is exactly the A-operand fragment of a 16x16x32 MFMA (and 8 16x16x4 fp32 MFMAs), so a
// wave streams one tile as one fully coalesced 1 KB (bf16) / 2 KB (fp32) load.
//
// Fused matrices (row permutations applied when packing):
//  * QKV: rows [Wq; Wk; Wv]. Within each head, tile j (j < head_dim/16) holds dims
//    8j..8j+7 followed by their rotary partners head_dim/2+8j..+7, so RoPE is tile-local.
//  * gate/up: tile t holds gate rows 8t..8t+7 followed by up rows 8t..8t+7.
// ---------------------------------------------------------------------------------------------

// Packed activations. The inputs of the linear kernels (x * gain, attention output, SwiGLU output;
// M rows x K features) are stored by their producers as MFMA B operands: tiles of 16 rows x 32
// features, tile (mt, kt) at byte offset (mt * (K/32) + kt) * ACT_TILE. Row r of a tile has two planes of
// four 16-byte slots, slot kg of plane p for features 8kg .. 8kg+7: bf16 models keep the 8 values' bf16
// hi halves in plane 0 and their lo halves in plane 1, fp32 models values 0..3 and 4..7. Either way the
// slots (r, kg) of both planes are one lane's operand of a 16x16x32 contraction. Passes of at most 16 rows
// keep a row's slots in one 128-byte line (one row reads whole lines: 4 draft steps 998 us, 1033 in
// operand order); passes of more rows keep them in operand order, so that a plane is one wave's 1 KB
// load without gaps (8 x 5 rows through 4 layers: 655 us, 695 as lines).
__host__ __device__ inline bool act_frag(int M) { return M > 16; }
__host__ __device__ inline int act_plane(bool frag) { return frag ? 1024 : 64; }
__host__ __device__ inline int act_slot(bool frag, int row16, int kg) {
  return frag ? kg * 256 + row16 * 16 : row16 * 128 + kg * 16;
}

// Arguments of the linear kernels.
struct LinArgs {
  const void* W;          // packed weights
  int N, K;               // output features, input features
  int M;                  // activation rows in this pass
  int KS;                 // K-ranges, added in order (set by the launchers, from the weight shape)
  // input
  const void* X;          // packed activations [M][K]; of the RMSNormed layers x*g, formed by the producer
  const float* rs;        // passes of more than 64 rows: RMSNorm row scales [M]
  const float* ssq;       // RMSNormed layers: [M][nssq] partial sums of squares of x (per 16 features)
  int nssq;
  float eps;
  // EPI_RESID: h[m][n] += y, xg[m][n] = h[m][n] * gain_next[n] (input of the next RMSNorm
  // consumer), ssq_out[m][n/16] = sum of squares of the 16 updated values
  float* h;
  void* xg;               // packed
  const float* gain_next;
  float* ssq_out;
  float* rs_out;          // passes of more than 64 rows: the updated rows' RMSNorm scales [M] (in place of ssq_out)
  // EPI_SWIGLU: act[m][f] = silu(gate) * up, f = nt*8 + c
  void* act;              // packed
  // EPI_QKV
  float* q;               // [M][n_heads*head_dim] rotated queries (fp32)
  void* kv;               // KV pool
  const int* row_pos;     // [M] absolute position of each row
  const int* row_slot;     // [M] cache position each row's keys/values are written to (= row_pos except for tree rows)
  const int* row_blk;     // [M] KV-pool block holding that position (same block in every layer)
  const float* row_rope;  // [M][head_dim]: cos(pos*theta_i) for i < head_dim/2, then sin(pos*theta_i)
  int layer, n_blocks, n_heads, n_kv, head_dim;
  // EPI_HEAD
  float* logits;          // nullable: logits[m * ld_logits + n]
  long long ld_logits;
  float* amax_val;        // per-workgroup argmax partials [M][amax_stride]
  int* amax_idx;
  int amax_stride;
  // k-range partials [KS][M][N] of the residual projections: of wide passes, and of decode passes of any row
  // count where there are more than 8 k-ranges
  float* part;
};

// Arguments of the split-KV paged attention kernel and its combine kernel.
struct AttnArgs {
  const float* q;         // [M][n_heads*head_dim]
  const void* kv;
  int layer, n_blocks;
  const int* bt;
  int bt_stride;
  const int* row_pos;     // [M]; rows m = b*R + r, consecutive positions within a sequence
  const int* row_slot;    // [M] cache slot of each row's keys/values (tree rows: p + node index;
                          // elsewhere equal to row_pos); the tree variant masks with it
  int B, R;               // sequences, rows per sequence
  int n_heads, n_kv, head_dim, G;  // G = n_heads / n_kv
  int RB, n_rb;           // rows per row-block (G*RB <= 32), row-blocks per sequence
  // block-causal pass of the speculative drafting objective (s_block > 0): row q (position q)
  // attends to the deep cache (kv, bt) at positions < s = floor(q / s_block) * s_block and to
  // the shallow cache skv (this pass's keys/values, block id = position / 16) at s..q
  const void* skv;
  int s_layer, s_n_blocks, s_block;
  int tree;               // 1: packed draft tree rows (mask by row_pos and row_slot)
  // one-launch pass attention (launch_attention_prefill, set by attention_pass_plan): 16 * pf_qt query
  // vectors per wave, and positions split over pf_split workgroups per row-block, whose partials [pf_split][R][n_heads] (o: head_dim floats, then m and l) are
  // merged by a second kernel when pf_split > 1
  int frag;               // layout of out: act_frag(rows of the pass)
  int pf_qt, pf_split;
  float* pf_o;
  float* pf_ml;
  int span;               // positions per workgroup group: 64, 128 or 256 (attention_span)
  int nq_alloc;           // set by the launcher: query vectors per row-block the LDS is sized for
  int n_groups_max;       // grid extent over groups; n_groups_max * span == bt_stride * 16
  float scale_log2;       // log2(e) / sqrt(head_dim)
  float* part;            // group partials [B][n_kv][n_rb][n_groups_max][32][head_dim + 4]
  void* out;              // packed activations [M][n_heads*head_dim]
};

// Sequences that share a wide pass, one after the other: rows row0 .. row0 + rows - 1 of the pass are
// consecutive positions of sequence seq from pos0 on.
constexpr int PASS_SEGS = 64;
struct PassSegs {
  int n;
  int row0[PASS_SEGS], rows[PASS_SEGS], seq[PASS_SEGS], pos0[PASS_SEGS];
};

// Per-pass row setup + embedding gather.
enum SetupMode { SETUP_PREFILL = 0, SETUP_DRAFT = 1, SETUP_VERIFY = 2, SETUP_SPEC = 3, SETUP_TREE = 4 };

struct SetupArgs {
  int mode;
  int M, R;               // rows, rows per sequence
  const int* t;           // [B] committed lengths
  int* drafts;            // [B][dstride]; drafts[b][0] is the pending token
  int dstride;
  int step;               // SETUP_DRAFT: draft step i (>= 1)
  const int* tokens;      // committed tokens [B][tstride]
  int tstride;
  int sim_accept;         // SETUP_VERIFY / SETUP_TREE: -1 or forced acceptance length
  const int* trace;       // [B][tstride] greedy trace by absolute position
  int vocab;
  const void* E;          // packed embedding
  int H;
  int* row_seq;
  int* row_pos;
  int* row_slot;          // [M] cache slot of the row's keys/values
  // nullable host-visible inputs of a call, copied to the device arrays by the rows that read them:
  // SETUP_VERIFY drafts [M / R][R - 1]; SETUP_TREE tokens, parents and depths of the nodes, each [64]
  const int* host_drafts;
  const int* host_tree;
  int* tree_tok;          // SETUP_TREE: node tokens [M] (node 0 = the pending token), then parents at [64..]
  int* tree_depth;        // SETUP_TREE: node depths [M] (rotary position t-1 + depth)
  // per-row KV block and RoPE row for the pass's QKV epilogues
  const int* bt;          // block tables [B][bt_stride]
  int bt_stride;
  const float* rope_cos;  // [max_ctx][head_dim/2]
  const float* rope_sin;
  int head_dim;
  int* row_blk;           // [M]
  float* row_rope;        // [M][head_dim]
  float* h;               // [M][H]
  void* xg;               // packed [M][H]: h * gain (input of the pass's first RMSNorm consumer)
  const float* gain;      // [H]
  float* ssq;             // [M][H/16]
  float* rs;              // nullable [M]: RMSNorm row scales (passes of more than 64 rows)
  float eps;
  // phase clock (nullable): block 0 writes the constant-rate clock to stamp[round * 3 + stamp_col]
  // when the kernel starts (round = *rounds, only while round < stamp_cap)
  long long* stamp;
  int stamp_col, stamp_cap;
  const int* rounds;
};

// Device-resident decoding state.
struct DevState {
  int* t;                 // [B] committed length
  int* len;               // [B] prompt length
  int* limit;             // [B] stop committing once t >= limit
  int* active;            // [B]
  int* nacc;              // [B] last n_accept
  int* bonus;             // [B] last bonus token
  int* rounds;            // [1] rounds run since prefill
  long long* counters;    // [2] drafted, accepted
  int* drafts;            // [B][dstride]
  int dstride;
  int* tokens;            // [B][tstride]
  int tstride;
  int* nacc_log;          // [log_cap][B]
  int log_cap;
  const int* vtok;        // [B*R] verifier argmax per row
  int eos;
  int* hres;              // nullable, host-visible: the acceptance kernel's result per sequence, n_accept [64],
                          // bonus [64], t [64]; of a tree out[0..65] (path length, bonus, path nodes)
  long long* stamp;       // nullable [stamp_cap][3]: the acceptance kernels write column 2 when done
  int stamp_cap;
};

constexpr int PF_SPLIT_MAX = 3;     // position splits of the one-launch pass attention,
constexpr int PF_SPLIT_ROWS = 1024;  // of passes of at most this many rows

// Optional timing events stamped by the launches themselves (hipExtLaunchKernel): `start` at the
// start of the first kernel of the operation, `stop` at the end of its last kernel.
struct LaunchEvents {
  hipEvent_t start, stop;
};

// Linear layer with its epilogue (inputs of QKV, gate/up and the head are RMSNormed): passes of at most
// 64 rows stream the weights (rows.hip, head.hip), wider ones are compute-bound (wide.hip).
template <typename T>
void launch_linear(const LinArgs& a, int epilogue, hipStream_t s, const LaunchEvents* ev = nullptr);
template <typename T>
void launch_linear_rows(const LinArgs& a, int epilogue, hipStream_t s, const LaunchEvents* ev);
template <typename T>
void launch_linear_wide(const LinArgs& a, int epilogue, hipStream_t s, const LaunchEvents* ev);
// Attention partials per group of span positions (the final output when the rows see one group).
template <typename T>
void launch_attention(const AttnArgs& a, hipStream_t s, const LaunchEvents* ev = nullptr);
// Causal (a.s_block > 0: block-causal) attention of a pass of more than 64 rows, every segment's rows over
// its own sequence's cache, written directly.
bool attention_prefill_supported(const AttnArgs& a);
// sets pf_qt and pf_split of a pass
void attention_pass_plan(AttnArgs& a, const PassSegs& sg, bool bf16);
template <typename T>
void launch_attention_prefill(const AttnArgs& a, const PassSegs& sg, hipStream_t s, const LaunchEvents* ev = nullptr);
// Merge of the group partials; needed when the context capacity spans more than one group.
bool attention_needs_combine(const AttnArgs& a);
template <typename T>
void launch_attn_combine(const AttnArgs& a, hipStream_t s, const LaunchEvents* ev = nullptr);
template <typename T>
void launch_setup(const SetupArgs& a, const PassSegs& sg, hipStream_t s);   // sg: SETUP_PREFILL, SETUP_SPEC
void launch_accept(const DevState& st, int B, int k, hipStream_t s);
// Tree acceptance for one sequence (packed tree of n nodes: tokens, parents, depths; the verifier
// argmax per node in st.vtok) and the move of an accepted leaf's keys/values in every layer to the
// cache position of its depth. out[0] = accepted path length, out[1] = bonus, out[2..] = path.
void launch_accept_tree(const DevState& st, int n, const int* tree_tok, const int* tree_par, const int* tree_depth,
                        int* out, void* kv, int n_layers, int n_blocks, int n_kv, int head_dim, int esize,
                        const int* bt, int* hstat, hipStream_t s);
// Confidence-aware dynamic drafting (Method, Adaptive Drafting with Tree-Based Verification;
// appendix "Confidence-Aware Dynamic Drafting"): after each drafting step, the top-1 probability
// p0 of the step's logits and its ranked top candidates; the top-p table gives the fan-out, the
// threshold tau the stop, and the tree is packed when drafting stops.
constexpr int TOPK_MAX = 16;        // largest fan-out a table may ask for
constexpr int TREE_MAX_STEPS = 16;  // drafting steps of one round (max_draft <= 15)
constexpr int TOPK_PARTS = 256;     // first-stage waves (each covers a contiguous logit chunk)

struct TreeDraftArgs {
  const float* logits;   // [V] the step's drafter logits
  int V, chunk;          // chunk: logits per first-stage wave (multiple of 64)
  int step;              // drafting step i >= 1 (X_draft[i] is being chosen)
  float* pval;           // first stage: [TOPK_PARTS][TOPK_MAX] candidate logits
  int* pidx;             //   and token ids (-1 = none)
  float* pmax;           //   [TOPK_PARTS] chunk maximum
  float* psum;           //   [TOPK_PARTS] sum of exp(z - chunk maximum)
  // fan-out rule: k = kk[j] for the first j with p0 > thr[j], else k_rest
  float tau;
  int n_levels;
  float thr[4];
  int kk[4];
  int k_rest, k_max;     // k_max: the table's largest fan-out (candidates kept per wave)
  int max_depth, max_nodes;
  // the round's drafting state
  int* cand;             // [TREE_MAX_STEPS][TOPK_MAX] ranked candidates of step i
  int* kcnt;             // [TREE_MAX_STEPS] fan-out used at step i
  float* p0;             // [TREE_MAX_STEPS] top-1 probability of step i
  int* dstate;           // [0] drafting stopped, [1] nodes so far (root included)
  int* drafts;           // sequence 0's drafts row: [0] the root X[p], [i] the chain token of step i
  int* tree;             // packed tree: token [64], parent [64], depth [64]; tree[192] = node count
  const int* rounds;     // rounds run so far: tags the status written when drafting stops
  int* hstat;            // nullable host-visible status: [0] round tag, [1] nodes, [2] depth
};
void launch_tree_topk(const TreeDraftArgs& a, hipStream_t s);
int tree_topk_chunk(int V);

// nll[r] = logsumexp(logits[r]) - logits[r][target[r]] for r < rows (row stride V)
void launch_row_nll(const float* logits, int rows, int V, const int* target, float* nll, hipStream_t s);
// Reduce the head's per-workgroup argmax partials of M rows; row m's token goes to
// tok_out[m * tok_stride] (lowest token id among equal maxima).
// (and to the host-visible host_out[m * host_stride], if given).
void launch_argmax_finalize(const float* val, const int* idx, int stride, int n_parts, int M, int* tok_out,
                            int tok_stride, int* host_out, int host_stride, hipStream_t s);
template <typename T>
void launch_pack(const void* src, void* dst, const int* dst_row, int rows, int K, hipStream_t s);
void launch_to_f32(const void* src, int src_is_bf16, float* dst, long long n, hipStream_t s);
void launch_fill_u32(void* dst, unsigned value, long long n_words, hipStream_t s);

// whether the current device grants a workgroup the LDS that the launch rules count on
hipError_t check_device();
}  // namespace seedk
