// Internal launcher declarations shared by the translation units of libmulo.
// Every launcher only enqueues work on `st`; shapes are validated by the caller
// (mulo_api.hip) before any of them runs.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mulo {

// A HIP call made while configuring a kernel (not a launch) failed: the entry point that is running returns
// MULO_ERR_HIP.  The launcher that notes an error does not launch.
void note_hip_error(hipError_t e);
// Raises the dynamic-LDS limit of `kern` to `bytes` once per process (state: 0 = not tried, 1 = done, -1 = failed);
// false, with the error noted, when the runtime refuses.
bool ensure_dynamic_lds(const void* kern, int bytes, int* state);

int cu_count();   // compute units of the device (gemm.hip)

// Launches of at most STREAM_MAX_TOKENS tokens (single-token decoding of a few sequences, island passes) run every
// bf16 projection in the weight-streaming kernel.  That kernel feeds its MFMA straight from registers, so its token
// operand [M, K] is kept in the order the instruction reads it (FRAGMENT ORDER): tokens in groups of 16, k in steps of
// 32; the 1 KB of (group t, step s) is contiguous, and inside it lane 16 c + r of a wavefront owns 16 bytes: k
// 32 s + 8 c .. + 7 of token 16 t + r.  The kernels that produce such an operand (RMSNorm, attention, the SwiGLU
// epilogue) write it in this order when the launch streams; one load instruction then reads a whole contiguous KB
// and no lane exchange is needed.  Buffers are sized for whole groups of 16 tokens.
constexpr int STREAM_MAX_TOKENS = 64;
inline bool streams_weights(int M) { return M <= STREAM_MAX_TOKENS; }
// With the context's weight copy in fragment order, launches of up to STREAM_MAX_TOKENS_COPY tokens stream: above
// STREAM_SHARED_MIN_TOKENS they run in the kernel that shares the token operand through LDS and splits K over workgroups.
constexpr int STREAM_MAX_TOKENS_COPY = 256;
#ifndef STREAM_SHARED_MIN_TOKENS
#define STREAM_SHARED_MIN_TOKENS 64
#endif
inline bool shares_tokens(int M, bool w_frag) { return w_frag && M > STREAM_SHARED_MIN_TOKENS; }
// How a launch of few tokens runs its projections (decided once per forward, the same for every kernel of it):
//   stream  the token operands are in fragment order and the projections run in the weight-streaming kernels
//   w_frag  the weight pointers are the context's copies in fragment order
//   ksums   scratch for the sums of the K slices when the launch streams: the context's own for launches that share tokens
//           (stream_ksum_floats), the attention's partial results for out and down of the others (STREAM_RESID_SLICES [M, d])
//   ksum_floats   what that scratch holds; more is an error
// and, for the tests of the tiled kernels, which tile a launch that does not stream runs on:
//   tile    index into the tile table (gemm.hip), taken where the projection has it; -1: the rule's choice
//   ran     host variable that receives the tile (-1: streamed)
struct StreamMode { bool stream, w_frag; float* ksums; int64_t ksum_floats; int tile; int32_t* ran; };
// K slices per 128-column group in the LDS-sharing kernel: as many as keep the launch within one round of 256
// workgroups, at most 8, at least 8 k-steps each.  A function of the projection's shape only, so the order of every
// sum is fixed by the model.
inline int stream_ksplit(int ncols, int K) {
    const int groups = (ncols + 127) / 128, steps = K / 32;
    int ks = 256 / groups;
    ks = ks < 1 ? 1 : (ks > 8 ? 8 : ks);
    const int most = steps / 8 > 1 ? steps / 8 : 1;
    return ks > most ? most : ks;
}
// Out and down projections of 17 to STREAM_MAX_TOKENS tokens whose sums are STREAM_RESID_K long or longer: the eight shares of K that
// k_gemv_bf16 deals to the wavefronts of a workgroup go to a workgroup each (k_gemv_shared), which shares the token operand of its
// slice among 64 or 128 columns, and the norm behind adds the eight in the order that kernel adds them in: the same bits as up to 16
// tokens.  52 tokens, us: 4096 x 4096 17.7 -> 13.8, from the copy 16.2 -> 12.9, 4096 x 11008 38.6 -> 26.6 and 36.4 -> 23.9, the norms
// 6.4 -> 8.5; 4096 x 1024 15.7 -> 8.9.  Shorter sums gain less: 8 layers of width 1024 with 2816 feed-forward columns, neither / both in slices,
// 17 tokens 282 / 256, 40 278 / 279, 64 315 / 311, from the copy 251 / 236, 260 / 261, 295 / 292.  One group of tokens loses by
// slices (4096 x 11008: 22 -> 26, from the copy 19.6 -> 20.7, with four of them).
constexpr int STREAM_RESID_SLICES = 8, STREAM_RESID_K = 4096;
// K slices that a projection of a streamed launch leaves in its scratch (0: none); resid: out or down
inline int stream_slices(int M, int ncols, int K, bool w_frag, bool resid) {
    if (shares_tokens(M, w_frag)) return stream_ksplit(ncols, K);
    return resid && M > 16 && K >= STREAM_RESID_K ? STREAM_RESID_SLICES : 0;
}
// floats of partial sums a launch of M shared tokens over `ncols` output columns (gate|up: 2 f, q|k|v: 3 d) needs
inline size_t stream_ksum_floats(int M, int ncols, int K) { return (size_t)stream_ksplit(ncols, K) * M * ncols; }
__host__ __device__ inline int64_t frag_index(int m, int k, int K) {   // in elements; runs of 8 k stay contiguous
    return ((int64_t)(m >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (m & 15)) * 8 + (k & 7);
}

// ---- decision stage (decide.hip) -------------------------------------------
struct DecideArgs {
    int B, L, V;
    int H, W, n0;
    int rho;          // Chebyshev radius expand*radius; -1 = raster-scan rule
    int pool_k;
    const int32_t* nbr;
    int resample_mode;   // 0 residual, 1 residual for rejected / p for expanded, 2 p
    int accept_mode;     // 0: u q < pbar (Eq. 1 / 3), 1: pbar >= tau (Eq. 5)
    float tau;
    uint32_t key0, key1, ctr_lo, ctr_hi24;
    const float* logits;        // [B, L, V]
    const float* logits_u;      // [B, L, V] unconditional logits (classifier-free guidance) or nullptr
    float cfg_scale;
    const float* q;             // rows of V floats
    const int32_t* q_row;       // [L] or nullptr
    int64_t q_batch_stride;
    const int32_t* draft_tokens;  // [B, L]
    int32_t* tokens_out;
    uint8_t* accept;
    uint8_t* mask;
    int32_t* t0;      // [B]
    int32_t* stats;   // [B, 4]
    float* p_probs;   // [B, L, V] or nullptr
    float* rowmax;    // [B*L] workspace
    float* rowinv;    // [B*L] workspace: 1 / sum exp, negative: a near tie
    // Replication geometry of the draft rows (a verification step): position (r I + a) W + r J + c of the block reads
    // draft row I up_w + J, W = up_r * up_w.  0: unknown (q_row is the caller's).  Only used to place the r * r
    // children of a draft row on one XCD next to each other, so that the row is fetched into one L2 once.
    int up_r, up_w;
};
// Replication of the draft's tokens (h x w cells a sequence, ratio r) to their children, with the table of the children's draft rows
struct UpTokens { const int32_t* lo; int32_t *hi, *q_row; int h, w, r; };
// up.hi: also what launch_upsample_tokens does, for the cells whose rows these are; nullptr: not
void launch_softmax_rows(const float* in, float* out, int64_t rows, int V, const UpTokens& up, hipStream_t st);
void launch_copy_rows(const float* in, float* out, int64_t n_floats, hipStream_t st);
// dst[b * dst_stride + c] = src[b * V + c] for B rows of V floats (V a multiple of 4)
void launch_copy_rows_strided(const float* src, float* dst, int B, int V, int64_t dst_stride, hipStream_t st);
void launch_upsample_tokens(const int32_t* draft_tokens, int32_t* tokens_hi, int32_t* q_row, int B,
                            int h, int w, int r, hipStream_t st);
void launch_gather_rows(const float* q_lo, const int32_t* q_row, float* q_hi, int B, int n_lo,
                        int n_hi, int V, hipStream_t st);
void launch_islands(const uint8_t* mask, int32_t* island, int32_t* rank, int32_t* counts, int B, int W, int n0, int L,
                    hipStream_t st);
void launch_seq_input(const int32_t* prev, const int32_t* tokens, int32_t* inp, int B, int L, int u, hipStream_t st);
void launch_seq_draw(const float* logits, const uint8_t* mask, int32_t* tokens, int B, int L, int V, int u,
                     uint64_t seed, uint64_t rng_counter, hipStream_t st);
// island-parallel re-sampling, pass `pass`: slots of the rank-`pass` positions (pos_tab, inputs), the hidden set
// of the pass, and afterwards the draws of the slots from their logit rows
void launch_island_select(const int32_t* prev, const int32_t* tokens, const uint8_t* mask, const int32_t* rank,
                          int32_t* pos_tab, int32_t* inp, uint8_t* hide, int32_t* overflow, int B, int L, int P,
                          int cap, int pass, hipStream_t st);
void launch_island_draw(const float* logits, const int32_t* pos_tab, int32_t* tokens, float* logits_out, int B,
                        int L, int V, int P, int cap, uint64_t seed, uint64_t rng_counter, hipStream_t st);
// softmax statistics + accept test.  sums: nullptr, or B * L * ceil(V / 256) integers for the chunk sums of the re-draw's
// weights; returns whether they were written (then launch_sample_sums finishes and draws, else launch_mask_sample)
bool launch_accept(const DecideArgs& a, unsigned long long* sums, hipStream_t st);
void launch_sample_sums(const DecideArgs& a, const unsigned long long* sums, hipStream_t st);
// the accept test from row parts (m, s per 128 columns, float pairs [rows, n_parts]) that the lm-head GEMM left;
// needs pool_k <= 1, no probability output and no guidance
void launch_accept_from_parts(const DecideArgs& a, const float* parts, int n_parts, hipStream_t st);
void launch_mask_sample(const DecideArgs& a, hipStream_t st);    // t0, Eq. 6-7 mask and the step's counters, residual draw of the marked positions

// ---- decoder forward (elementwise.hip, gemm.hip, attention.hip) ------------
struct RopeArgs {
    const float* cos;   // [max_seq, dh/2]
    const float* sin;
    int L, P, n_heads, head_dim, max_seq, max_batch, layer;
    // Scattered single-token queries (island-parallel re-sampling): token m is slot m % L of sequence m / L and
    // sits at cache row pos_tab[m] (< 0: an unused slot, nothing of it is written).  nullptr: token m is position
    // m % L of sequence m / L, at cache row P + m % L.
    const int32_t* pos_tab = nullptr;
};
// The inputs of a step: row j of sequence b (of seqs; those behind them are their unconditional twins) takes prev[b] (j == 0) or the
// up-sampled token of position j - 1
struct StepTokens { UpTokens up; const int32_t* prev; int seqs; };
// x[m, :] = embed[clamp(tok[m])]  (float32 residual stream); T = float or bf16 storage.  in.up.lo: the tokens are those of a step,
// and the up-sampled tokens and the table of draft rows are written on the way.
void launch_embed(const void* embed, int dtype, const int32_t* tok, const void* in_embeds, const StepTokens& in, float* x,
                  int M, int d, int V, hipStream_t st);
// Sums of the K slices of a projection whose residual add is still to come: n slices [M, d] in `sums` (n == 0: none).
struct Slices { const float* sums; int n; };
// frag: write `out` in fragment order (bf16 launches that stream the weights); x first takes the slices, added in index order
void launch_rmsnorm(float* x, const void* gain, int dtype, void* out, int M, int d, float eps, bool frag, Slices add,
                    hipStream_t st);

// bf16 MFMA GEMMs, C = A[M,K] * W[N,K]^T with fused epilogues
void launch_gemm_qkv_bf16(const void* xh, const void* wq, const void* wk, const void* wv, void* q_out,
                          void* k_cache, void* v_cache, int M, int d, const RopeArgs& ra, const StreamMode& sm,
                          hipStream_t st);
// x += A W^T; or, where K is dealt to several workgroups, the slices' sums, which the norm behind it adds to x
Slices launch_gemm_resid_bf16(const void* a, const void* w, float* x, int M, int N, int K, const StreamMode& sm,
                              hipStream_t st);
void launch_gemm_swiglu_bf16(const void* xh, const void* wg, const void* wu, void* h, int M, int f,
                             int d, const StreamMode& sm, hipStream_t st);
// Copies `layers` bf16 matrices [rows, K] (contiguous, rows % 16 == 0 or layers == 1) into fragment order: rows in
// groups of 16, k in steps of 32, the KB of (group, step) contiguous with lane 16 c + r holding k 8 c .. 8 c + 7 of
// row r; rows past the last are zeros.  dst holds layers * ceil16(rows) * K elements.
void launch_pack_weights(const void* src, void* dst, int layers, int rows, int K, hipStream_t st);
inline size_t packed_weight_elems(int layers, int rows, int K) { return (size_t)layers * ((rows + 15) / 16 * 16) * K; }
// parts: nullptr, or float pairs [M, ceil(V / 128)] that receive the softmax statistics of every 128-column part of
// every row (row_parts.h); returns whether they were written (only the kernels whose wavefront tile is 128 columns
// wide produce them)
bool launch_gemm_logits_bf16(const void* xh, const void* w, float* logits, float* parts, int M, int V, int d,
                             const StreamMode& sm, hipStream_t st);
size_t attention_scratch_bytes(int max_batch, int n_heads, int head_dim);   // partial results of the key split
// frag_out: `out` feeds a weight-streaming projection: written in fragment order
void launch_attention_bf16(const void* q, const void* k_cache, const void* v_cache, void* out, float* scratch,
                           int B, int L, int P, int n_heads, int head_dim, int max_seq, int max_batch,
                           int layer, bool frag_out, hipStream_t st);
// cap single-token queries per sequence at scattered cache rows: slot j of sequence b sits at row
// pos_tab[b * cap + j] (< 0: unused slot, its output row is zeroed) and attends to rows <= its own except the rows
// P0 + t of its sequence with hide[b, t] set (t < Lblk; its own row is never hidden).  Rows are in [P0, P0 + Lblk).
void launch_attention_scattered_bf16(const void* q, const void* k_cache, const void* v_cache, void* out,
                                     float* scratch, int B, const int32_t* pos_tab, int cap, const uint8_t* hide,
                                     int P0, int Lblk, int n_heads, int head_dim, int max_seq, int max_batch,
                                     int layer, bool frag_out, hipStream_t st);

// float32 path (forward_f32.hip): x is the residual stream, its RMSNorm with `gain` is part of the projection; rotary and
// cache append, the SwiGLU product and the residual add are the projections' epilogues
void launch_qkv_f32(const float* x, const float* gain, float eps, const float* wq, const float* wk, const float* wv,
                    float* q_out, float* k_cache, float* v_cache, int M, int d, const RopeArgs& ra, hipStream_t st);
void launch_swiglu_f32(const float* x, const float* gain, float eps, const float* wg, const float* wu, float* h, int M,
                       int f, int d, hipStream_t st);
void launch_resid_f32(const float* a, const float* w, float* x, int M, int N, int K, hipStream_t st);
void launch_logits_f32(const float* xh, const float* w, float* logits, int M, int V, int d, hipStream_t st);
void launch_attention_f32(const float* q, const float* k_cache, const float* v_cache, float* out, int B, int L, int P,
                          int n_heads, int head_dim, int max_seq, int max_batch, int layer, hipStream_t st);

}  // namespace mulo
