// Internal launch interface between the C ABI layer and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sx {

// Rotary embedding + cache write behind the q/k/v projection: row r of the step is sequence r / W, rotary position pos[r / W] + level, cache entry
// pos[r / W] + node[r % W] (node null: the entry at pos).
struct RopeArgs {
  const int32_t* pos;
  int level;
  const int32_t* node;
  int W;
  float theta;
  double inv_freq[64];       // theta^(-2c/d) for c < d/2, filled on the host
  int Hq, Hkv, d;
  void* q_out;               // [rows][Hq][d], bf16 or (row-streaming kernel, fp32 model) fp32
  int paged;
  void *kc, *vc;
  const int32_t* page_table;
  int page_size, max_pages;
  int64_t l_max;
  int64_t n_pages;           // paged: pages in the pool (page ids are forced into it)
  int* status;               // device error word or nullptr
};

// Activations in the operand order of the weight-stream kernels: [k block of 128][16-row tile][k step of 32][lane]
// 16-byte pieces; lane (c = lane % 16, q = lane / 16) of a piece holds row c of the tile, k = 32 step + 8 q .. + 7.
// With two planes tile 2 o holds the bf16 rounding of rows 16 o .. + 15, tile 2 o + 1 the bf16 rounding of the rest.
__host__ __device__ inline int packed_tiles(int M, int planes) { return (M + 15) / 16 * planes; }
__host__ __device__ inline size_t packed_byte(int NT, int tile, int m, int k) {
  return ((static_cast<size_t>(k >> 7) * NT + tile) * 4 + ((k >> 5) & 3)) * 1024 + ((k >> 3) & 3) * 256 + (m & 15) * 16 + (k & 7) * 2;
}

// Projection of the draft layer over more rows than the row-streaming kernel takes (gemm_proj.hip): partial sums, added by the kernel behind it.
struct ProjArgs {
  const void* w[3];    // up to three row blocks (q/k/v or gate/up share one launch)
  int seg_end[3];      // exclusive end row of each block in the concatenated row space, multiples of 16
  int nseg;
  int N, K, M;
  int planes;          // 1: bf16 activations, 2: bf16 value + rest
  const void* a_packed;  // two planes: activations in operand order
  const void* a_src;     // one plane: bf16 rows [M][K]; with a_embed [embed[tok[m]] ; a_src[m]], each K/2 wide
  const void* a_embed;   // embedding table [V][K/2] or nullptr
  const int32_t* a_tok;  // token ids [M], forced into 0 .. a_vocab-1
  int a_vocab;
  int* status;         // device error word or nullptr (first out-of-range token id seen)
  int W;               // workgroups
  float* partial;      // proj_partial_bytes()
};
// where the partial sums of a projection lie (see gemm_proj.hip)
struct ProjSum {
  const float* partial;   // [slot][M][128]
  int T;                  // blocks of the projection
  uint32_t inv_T;         // 2^32 / T, rounded down
  int KB, W, M;           // k blocks of a group, workgroups, rows
};
__host__ __device__ inline int proj_groups(int N) { return N / 128; }
// Workgroup that has block x of T dealt to W: the last that starts at or before it, (x + 1) W - 1 over T, rounded down.  (The product
// with 2^32 / T is off by one at most; T W < 2^32 as long as the weights are less than 137 GB with 1024 workgroups, 550 GB with 256.)
__host__ __device__ inline uint32_t proj_inverse(int T) { return T > 1 ? static_cast<uint32_t>((1ull << 32) / static_cast<uint64_t>(T)) : 0u; }
__host__ __device__ inline int proj_owner(int T, uint32_t inv_T, int W, int x) {
  const uint32_t a = static_cast<uint32_t>(x + 1) * static_cast<uint32_t>(W) - 1;
  const uint32_t q = static_cast<uint32_t>((static_cast<uint64_t>(a) * inv_T) >> 32);
  return static_cast<int>(a - q * static_cast<uint32_t>(T) >= static_cast<uint32_t>(T) ? q + 1 : q);
}
bool proj_supported(int M, int N, int K);
void proj_plan(ProjArgs& g, int num_cus);
size_t proj_partial_bytes(const ProjArgs& g);
hipError_t launch_proj(const ProjArgs& g, hipStream_t s);
// rows = sums (+ residual) -> out_x fp32 / out_store bf16 (either may be null); RMSNorm of the rows -> packed (two planes)
hipError_t launch_proj_norm(const ProjArgs& g, const float* residual, const void* gain, float eps, float* out_x, void* out_store, void* packed,
                            hipStream_t s);
// silu(gate) * up of the gate|up projection -> packed (two planes)
hipError_t launch_proj_silu(const ProjArgs& g, void* packed, hipStream_t s);
hipError_t launch_proj_rope(const ProjArgs& g, const RopeArgs& ra, hipStream_t s);

// Head GEMMs (gemm_wide.hip) and the plain-ALU GEMM (gemm.hip): out[m][n] = sum_k act[m][k] * w[n][k].
// Head: rows n < V enter a fused argmax, rows V.. are the signal rows of the widened head.
struct GemmArgs {
  const void* w[3];    // up to three row blocks
  int seg_end[3];      // exclusive end row of each block in the concatenated row space
  int nseg;
  int N, K, M;
  int planes;          // head: 1 = activations exact in bf16, 2 = bf16 hi + lo parts
  const float* act;    // ALU path: fp32 [M][K]
  float* partial;      // ALU path: out [M][N]
  // head: where the activations come from
  int a_mode;          // 1: bf16 rows [M][K]; 3: RMSNorm of fp32 rows: a_src[m][k] * rsqrt(sum_j a_ssq[m][j] / K + a_eps) * a_gain[k];
                       // 4: a_packed already holds them in operand order
  const void* a_src;
  const float* a_ssq;  // mode 3: [M][a_nssq] pieces of the rows' sums of squares
  int a_nssq;
  const void* a_gain;  // mode 3: [K] bf16 norm gain
  float a_eps;
  void* a_packed;      // head_wide_pack_bytes() for the activations in operand order
  int wide_w;          // workgroups (each walks an equal share of the weight tiles)
  int wide_slots;      // candidate slots per workgroup and row, each of max(top_b, 1) candidates
  int V;               // head when >= 0
  int n_extra;
  int top_b;           // candidates kept per slot (0 or 1 = the argmax only)
  float* part_val;     // [M][head_wide_groups][top_b] best values, best first
  int* part_idx;       // their row indices (INT_MAX = none)
  float* extra_out;    // [M][n_extra] or nullptr
  float* logits_dbg;   // [M][V] or nullptr
};

// Row-streaming GEMV (gemv.hip) for bf16 steps of up to four rows and for fp32 ones: no split over K, the
// epilogue runs in the wave that owns a pair of weight rows.
struct GemvArgs {
  int f32;               // weights, gains, stored rows and cache entries are fp32, else bf16
  const void* w[3];
  int seg_end[3];
  int nseg;
  int N, K, M;
  int a_mode;            // 0 fp32 rows, 1 bf16 rows (not with f32), 2 [embed[tok] ; hidden], 3 RMSNorm of fp32 rows
  const void* a_src;
  const void* a_embed;
  const int32_t* a_tok;  // mode 2: token ids [M], forced into 0 .. a_vocab-1
  int a_vocab;
  int* status;           // device error word or nullptr
  const float* a_ssq;
  int a_nssq;
  const void* a_gain;
  float a_eps;
  int epi;               // 0: rows (2p, 2p+1) -> residual add, out_x / out_store / out_ssq
                         // 1: rotary pairs of the q|k|v projection -> q_out / cache entries
                         // 2: (gate p, up p) of the gate|up projection -> out_x[m][p] = silu(gate) * up
                         // 3: widened head: rows < V -> per-workgroup argmax candidates part_val / part_idx
                         //    [M][grid], rows V.. -> extra_out [M][n_extra]; N may be odd
                         // 4: out_x[m][n] = sums, N may be odd (f32 only)
  const float* residual;
  float* out_x;
  void* out_store;
  float* out_ssq;        // [M][grid]
  int V, n_extra;        // epi 3
  float* part_val;
  int* part_idx;
  float* extra_out;
  RopeArgs rope;
  int stream;            // 1: weights read with non-temporal loads (read once; always for the head), 0: ordinary loads
  int grid, waves;       // launch shape, from gemv_plan
};
bool gemv_supported(bool f32, int M, int N, int K);
void gemv_plan(GemvArgs& g, int num_cus, int per_cu = 3);   // at most per_cu workgroups per compute unit
hipError_t launch_gemv(const GemvArgs& g, hipStream_t s);

inline int gemm_ntiles(int N) { return (N + 15) / 16; }
hipError_t launch_zero_i32(int* p, int n, hipStream_t s);
hipError_t launch_gemm_valu(const GemmArgs& g, bool bf16, hipStream_t s);
bool head_wide_supported(const GemmArgs& g);
void head_wide_plan(GemmArgs& g, int num_cus);   // sets wide_w, wide_slots
int head_wide_groups(const GemmArgs& g);      // candidates per activation row
size_t head_wide_pack_bytes(const GemmArgs& g);
hipError_t launch_head_wide(const GemmArgs& g, hipStream_t s);
// reduce per-tile partial argmaxes: one result per activation row
// (with `sig` set it also applies the signal activations to extra[M][3]: the draft head's epilogue)
hipError_t launch_argmax_finalize(const float* part_val, const int* part_idx, int ntiles, int M,
                                  int32_t* argmax, float* max_logit, hipStream_t s,
                                  const float* extra = nullptr, int rem_activation = 0,
                                  float* sig_raw = nullptr, float* sig = nullptr);
// the top_b best per row, best first, from per-tile candidates (idxs given; C pairs per row)
// or from full rows of logits (idxs null; C = V values per row); rows lie `stride` apart
hipError_t launch_topb_finalize(const float* vals, const int* idxs, int C, int stride, int top_b, int M,
                                int32_t* cand_tok, float* cand_logit, hipStream_t s,
                                const float* extra = nullptr, int rem_activation = 0,
                                float* sig_raw = nullptr, float* sig = nullptr);
// VALU head path: logits [M][N] -> argmax over n < V, copy of signal rows and of logits
hipError_t launch_argmax_rows(const float* logits, int M, int N, int V, int n_extra,
                              int32_t* argmax, float* max_logit, float* extra_out,
                              float* logits_dbg, hipStream_t s, int rem_activation = 0, float* sig_raw = nullptr,
                              float* sig = nullptr);   // (with `sig` set: the three signal rows' activations too)
// storage-type rows -> fp32 rows (ALU GEMM path only)
hipError_t launch_unpack_rows(const void* src, bool bf16, int M, int K, float* act, hipStream_t s);

// ---- attention -------------------------------------------------------------------------
struct AttnArgs {
  int dtype;                 // 0 fp32, 1 bf16
  int paged;
  const void *k, *v;
  const int32_t* page_table;
  int page_size, max_pages;
  int64_t l_max;
  int B, n_q, Hq, Hkv, d;
  const void* q;             // [B, n_q, Hq, d]
  const int32_t* ctx_len;    // [B] number of context entries before the block
  const uint64_t* mask;      // [B, n_q] or nullptr = chain
  int G, g_inv;              // Hq / Hkv and ceil(65536 / G): r / G = r g_inv >> 16 for r < 128 (attn_plan)
  int pad, wide_from;        // work split: padding per unit, granules from which more workgroups than compute units take part
                             // (attn_sched.hpp)
  int n_blk;                 // block entries stored after the context (normally n_q; tree drafting:
                             // every node written so far, of which n_q are this call's queries)
  int mask_stride;           // mask words between two sequences' rows (n_q; 0 = all sequences share)
  float scale;
  void* out;                 // [B, n_q, Hq, d] in dtype
  int wgrid;                 // workgroups of the split kernel; the keys of all (sequence, KV head) units
                             // are dealt to them in equal shares on the device (attn_sched.hpp)
  float* part_o;             // [wgrid + B*Hkv slots][R][d]
  float* part_ml;            // [wgrid + B*Hkv slots][R][2]  (running max, sum)
  int* sched;                // written by the split kernel for the merging kernel: the first and the last workgroup of every
                             // unit, [B*Hkv][2]
  int64_t n_pages;           // paged: pages in the pool (page ids are forced into it)
  int* status;               // device error word or nullptr: first out-of-range length / page id seen
  // for the host; in bytes, so that the arguments of the kernels are three 64-byte lines
  int8_t rings, stages;      // matrix-core kernel: tile rings of a workgroup, slots of a ring (attn_plan)
  bool draft;                // the call goes on to rank logits that follow from the output (a draft step or tree level)
  int use_mfma;              // 0, or matrix-core kernel (bf16; its maxima are in log2 units): kOnePart or kTwoPart
};
static_assert(sizeof(AttnArgs) <= 192, "a fourth line costs every launch of the merging kernels 40 ns");
constexpr int kOnePart = 1, kTwoPart = 2;       // parts of bf16 that the matrix-core kernel has its probabilities in
bool attn_mfma_supported(const AttnArgs& a);
size_t attn_mfma_lds_bytes(const AttnArgs& a);  // dynamic LDS of the matrix-core kernel as planned
int attn_mfma_rings(const AttnArgs& a);         // its tile rings per workgroup
int attn_mfma_per_cu(const AttnArgs& a);        // workgroups per compute unit
int attn_mfma_stages(const AttnArgs& a);        // and slots per tile ring
bool attn_mfma_two_part(const AttnArgs& a);     // probabilities in two bf16 parts
int attn_mfma_max_chunk(const AttnArgs& a);   // longest chunk the matrix-core kernel takes
int attn_slots(const AttnArgs& a);            // partial-result slots a launch can write
hipError_t launch_attn_mfma(const AttnArgs& a, hipStream_t s);
bool attn_plan(AttnArgs& a, int num_cus);      // false: the problem is outside what one launch can split
size_t attn_workspace_bytes(const AttnArgs& a);
void attn_carve(AttnArgs& a, void* workspace);   // points part_o / part_ml / sched into a workspace of that size
// hook(id, 0 / 1, stream) is called right before / after the split-KV kernel's launch
typedef void (*KernelHook)(int id, int phase, hipStream_t s);
hipError_t launch_attn(const AttnArgs& a, hipStream_t s, KernelHook hook = nullptr, int hook_id = 0);

// ---- draft-step glue kernels -----------------------------------------------------------
struct DraftDims {
  int dtype, D, Hq, Hkv, d, I, V;
  float rms_eps, rope_theta;
  int rem_activation;
};
hipError_t launch_embed_concat(const DraftDims& dm, int B, const void* embed, const int32_t* tok,
                               const void* hidden_in, float* act, hipStream_t s, int* status = nullptr);
// v[b][:] = rows[b][:] (+ residual[b][:]); optional copy to `sum_out` (fp32) and
// `hidden_out` (storage type); then RMSNorm with gain -> act (fp32)
hipError_t launch_row_norm(const DraftDims& dm, int B, int N, const float* rows, const float* residual, const void* gain, float* sum_out,
                           void* hidden_out, float* act, hipStream_t s);
// rows r = b * W + w: rotary position pos[b] + level, cache entry pos[b] + node[w] (node null: pos[b])
hipError_t launch_rope_kvwrite(const DraftDims& dm, int M, int W, const float* rows, const int32_t* pos, int level,
                               const int32_t* node, void* q_out, int kv_paged, void* kc, void* vc, const int32_t* page_table,
                               int page_size, int max_pages, int64_t l_max, hipStream_t s, int64_t n_pages = 0x7fffffff,
                               int* status = nullptr);
hipError_t launch_silu_mul(const DraftDims& dm, int B, const float* rows, float* act, hipStream_t s);

// ---- measurement aid: copy of known size through the streaming load path -------------------
hipError_t launch_copy_probe(const void* src, void* dst, size_t bytes, bool nontemporal, hipStream_t s);

// ---- cache compaction after acceptance ---------------------------------------------------
struct CompactArgs {
  int paged;
  void *k, *v;
  const int32_t* page_table;
  int page_size, max_pages;
  int64_t l_max;
  int64_t n_pages;           // paged: pages in the pool (page ids are forced into it)
  int64_t layer_stride_bytes;
  int n_layers, B, n_q, Hkv;
  int row_bytes;             // head_dim * element size
  const int32_t *ctx_len, *accept_path, *accept_len, *last_node;
  int* status;               // device error word or nullptr
  const void* block_hidden;  // [B][n_q][hidden_row_bytes] or nullptr
  void* hidden_next;         // [B][hidden_row_bytes]
  int hidden_row_bytes;
};
bool kv_compact_supported(const CompactArgs& a);
hipError_t launch_kv_compact(const CompactArgs& a, hipStream_t s);

// ---- tree drafting: hand tokens and hidden states from one level to the next ----------------
struct TreeGatherArgs {
  int B, W_prev, top_b, W_next, n_q;
  int row_bytes;               // D * element size
  const int32_t *src_row, *rank, *node;   // [W_next]
  const int32_t* cand_tok;     // [B][W_prev][top_b]
  const void* hidden_prev;     // [B][W_prev][row_bytes]
  int32_t* tok_next;           // [B][W_next]
  void* hidden_next;           // [B][W_next][row_bytes] or nullptr
  int32_t* block_tok;          // [B][n_q] or nullptr
};
hipError_t launch_tree_gather(const TreeGatherArgs& a, hipStream_t s);

// ---- controller ------------------------------------------------------------------------
constexpr int kSmoothWords = 48;   // 3 signals x 16 words
struct ExitArgs {
  float alpha, thr_conf, thr_prog, thr_rem;
  uint32_t signal_mask;
  int smoother, window, split_pick, check_root, stop_think_token;
  int B, n_q, S;
  const int32_t *block_tok, *parent, *target_argmax;
  const float* sig;
  const int32_t *ctx_len, *split_tok;
  float* ewma;
  int32_t *n_obs, *is_thinking;
  float* smooth_state;       // [B][kSmoothWords] history of the window / momentum / paragraph smoothers
  int32_t *accept_len, *accept_path, *recover_tok, *last_node, *exit_flag, *new_ctx_len;
};
hipError_t launch_accept_exit(const ExitArgs& a, hipStream_t s);

}  // namespace sx
