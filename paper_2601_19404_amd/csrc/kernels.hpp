// Launchers of the HIP kernels behind the RPO rollout C ABI (host-callable).
// Every launcher validates nothing: callers (rpo_api.hip) check shapes first.
#pragma once

#include "common.hpp"

namespace rpo {

// g * sigmoid(g); the hardware reciprocal (1 ulp) replaces the IEEE division sequence
__device__ inline float silu_f(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// 16 bytes per lane from global memory (uniform base + 32-bit lane offset) straight into LDS at
// lds_byte_addr + off + 16 * lane.  The compiler does not see the load: every wait for it is written out.
// ONCE is for data from HBM that is read once (weights that no other workgroup reads): the non-temporal hint keeps it
// from taking the place of other lines on its way.  256 CUs streaming rows of 128 bytes from HBM: 6.15 -> 7.05 TB/s; for
// lines that others read as well it is a loss (activations, each read by every CU: 113 -> 59 GB/s per CU).
template <bool ONCE>
__device__ inline void dma_load16_at(const void* sbase, uint32_t voff, uint32_t lds_byte_addr, int off) {
    if constexpr (ONCE)
        asm volatile(
            "s_add_u32 m0, %2, %3\n\t"
            "s_nop 0\n\t"
            "global_load_lds_dwordx4 %0, %1 nt\n\t"
            :
            : "v"(voff), "s"(sbase), "s"(lds_byte_addr), "i"(off)
            : "memory", "scc");
    else
        asm volatile(
            "s_add_u32 m0, %2, %3\n\t"
            "s_nop 0\n\t"
            "global_load_lds_dwordx4 %0, %1\n\t"
            :
            : "v"(voff), "s"(sbase), "s"(lds_byte_addr), "i"(off)
            : "memory", "scc");
}

enum DType : int { kF32 = 0, kBF16 = 1 };

inline size_t dtype_size(int dt) { return dt == kF32 ? 4 : 2; }

// One packed sequence of token rows inside a chunk pushed through the layers.
struct SeqDesc {
    int row_start;  // first row of the sequence in the packed row buffer
    int n_rows;     // rows of this sequence in the buffer
    int pos0;       // absolute position (0-based over prompt || answer) of its first row
    int table_off;  // offset (in int32) of its page table inside the table array
};

// ---- GEMM: C[M,N] (op)= A[M,K] * W[N,K]^T, fp32 accumulation -----------------
enum Epilogue : int {
    kEpiStore = 0,     // C has the input dtype
    kEpiStoreF32 = 1,  // C is fp32
    kEpiAddF32 = 2,    // C is fp32 and is accumulated into (residual stream)
    kEpiSwiglu = 3,    // W = [gate rows; up rows] (N = 2F): C[M, F] = silu(A Wg^T) * (A Wu^T), input dtype
    kEpiPartial = 4,   // internal: fp32 partial sums of one K split
    kEpiRope = 5,      // internal: rotary embedding + KV page write from the accumulators (QKV projection)
    kEpiLse = 8,       // internal: no C; per row and 64-column block the maximum and the sum of
                       // 2^((z - max) k2), plus the value at the row's target column (LM head of the
                       // log-prob pass: the logits never reach memory)
    kEpiLogitsMax = 9, // internal: kEpiStoreF32 that also leaves each row's maximum per 64-column block
};
// Outputs of the kEpiLse epilogue (GemmArgs::lse): see launch_lse_combine for what follows.
struct LseFuse {
    float* part = nullptr;          // [M, blocks, 2] (max, sum) per row and column block
    float* target_logit = nullptr;  // [M] z[row, target[row]]
    const int32_t* target = nullptr;  // [M] column ids (out of range: target_logit untouched)
    float k2 = 0.f;                 // log2(e) / temperature
    int blocks = 0;                 // filled in by the launch: column blocks per row
};
// RMSNorm taken apart for a few rows: the accumulating projection leaves h = bf16(x * gain) and each row's sums of
// squares per 16 columns, the SwiGLU projection that reads h multiplies its results by 1 / sqrt(mean(x^2) + eps).
// (bf16 rounding is relative: h is as precise as the normalised row.)
struct NormFuse {
    float* part = nullptr;  // [M, blocks]
    int blocks = 0;         // filled in by the launch that takes the norm apart; 0: norm_out holds normalised rows as usual
    const bf16* gain = nullptr;
    bf16* h = nullptr;
    float eps = 0.f;
};
struct RopeKvArgs;
struct GemmArgs {
    const void* A;
    int64_t lda;
    const void* W;
    int64_t ldw;
    void* C;
    int64_t ldc;
    int M, N, K;
    int dtype;     // element type of A and W
    int epilogue;  // Epilogue
    int path;      // 0 = pick, 1 = force the generic (non-MFMA) kernel
    void* ws;      // fp32 scratch for K-split partial sums (may be null: no splitting)
    size_t ws_bytes;
    // Optional, with kEpiAddF32 only: after C += A W^T, also write the RMS-normalised rows
    // norm_out[m, :] = C[m, :] / sqrt(mean(C[m, :]^2) + norm_eps) * norm_gain (input dtype, row
    // stride N).  Fused into the K-split reduction when the problem is split.
    const void* norm_gain = nullptr;
    void* norm_out = nullptr;
    float norm_eps = 0.f;
    // Optional, with kEpiStore only (the QKV projection): after C = A W^T, rotate q and k of every
    // row and write k, v into the KV pages (rope->qkv must be C).  Fused into the K-split
    // reduction when the problem is split (the rotation then reads the fp32 sums: one rounding).
    const RopeKvArgs* rope = nullptr;
    // Optional, with kEpiStoreF32 only (the LM head of the log-prob pass): if the launch can fuse the
    // log-sum-exp (gemm_fuses_lse), C is not written and *lse receives the partial results instead.
    LseFuse* lse = nullptr;
    // Optional, with kEpiStoreF32 only (the LM head of a decode step): if the launch can (gemm_fuses_max),
    // it also writes block_max->part[row, block] = max of the row over that column block.
    LseFuse* block_max = nullptr;
    // Optional, with kEpiAddF32 and norm_out: the launch may take the norm apart (norm_split->part is given, blocks set).
    NormFuse* norm_split = nullptr;
    // Bytes of weights that a program reads from one use of W to the next, where it is known (a model's); 0: a call by itself.
    size_t turn_bytes = 0;
    // Optional, with kEpiSwiglu, where gemm_takes_norm says so: A is the h of a norm taken apart.
    const NormFuse* norm_in = nullptr;
};
// Whether W comes from HBM each time it is read, i.e. has left the memory-side cache since its last use.
bool gemm_weights_pass(const GemmArgs& a);
// Whether these (SwiGLU) arguments can come with norm_in.
bool gemm_takes_norm(const GemmArgs& a);
hipError_t launch_gemm(const GemmArgs& a, hipStream_t s);
// The weight-streaming kernel for few rows (bf16, K a multiple of 64, 16-byte aligned rows: checked by
// launch_gemm).  epi: kEpiStore / kEpiStoreF32 / kEpiAddF32 / kEpiSwiglu, kEpiRope (a.rope, head_dim 128) or
// kEpiLogitsMax (a.block_max: row maxima per 64 columns).
// splits > 1: fp32 partial sums of that many K ranges to a.ws[splits][M][N] instead.
hipError_t launch_gemm_skinny(const GemmArgs& a, int epi, int splits, hipStream_t s);
int gemm_skinny_splits(const GemmArgs& a);
bool gemm_skinny_splits_norm(const GemmArgs& a);  // honours GemmArgs::norm_split
// Up to 64 rows: whether that kernel is the faster one, given whether the tiles would split K.
bool gemm_skinny_takes(const GemmArgs& a, bool tiles_split_k);
// More than 64 rows: whether that kernel takes the problem in groups of 64 rows (> 0) or not at all (0).
int gemm_skinny_groups(const GemmArgs& a);
// Whether launch_gemm would honour GemmArgs::lse for these arguments, and with how many column
// blocks per row (0 = it would write C as usual).
int gemm_fuses_lse(const GemmArgs& a);
int gemm_fuses_max(const GemmArgs& a);
// out[r] = max_b part[r, b]  /  out[r] = max_i logits[r, i]
hipError_t launch_row_max_blocks(const float* part, int blocks, float* out, int rows, hipStream_t s);
hipError_t launch_row_max(const float* logits, int64_t row_stride, int vocab, float* out, int rows, hipStream_t s);

// Practical-ceiling probes (probes.hip): a plain copy (GB/s, read + write) and an MFMA issue loop.
hipError_t probe_copy(const void* src, void* dst, size_t bytes, int reps, double* gbps, hipStream_t s);
hipError_t probe_mfma(float* scratch, int iters, int reps, double* tflops, hipStream_t s);

// Identifiers of the kernels whose launches can be timed (rpo_profile_start).
enum KernelId : int {
    kKidNone = 0,
    // tile shapes of gemm_dma_kernel / gemm_mfma_kernel <BM, BN, waves along M, waves along N>
    kKidGemm256 = 1,        // <256,256,2,4> (many-tile problems), and <128,256,2,4> (LM head of 33 to 128 rows)
    kKidGemm128 = 3,        // <128,128,2,2> (decode-sized problems with a deep K, K split; gate/up of 65 to 128 rows; chunks of up to a few thousand rows)
    kKidGemm64 = 4,         // <64,128,1,2>  (the same for M <= 64, where the few-row kernel does not take them)
    kKidGemm32 = 5,         // <32,128,1,4>  (QKV projection of more rows than the few-row kernel takes and of chunks: one head per tile of 32, 64 or 128 rows, no K split)
    kKidGemm64x64 = 6,      // <64,64,2,2>   (decode-sized problems and small chunks with a shallow K, no K split)
    kKidGemmGeneric = 7,
    kKidGemm256x192 = 11,   // <256,192,4,2> (large M, narrow N: fewer idle CUs in the last round)
    kKidAttnDecode = 8,     // attn_decode_mfma_kernel
    kKidAttnChunk = 9,      // attn_chunk_mfma_kernel
    kKidSample = 10,        // sample_kernel
    kKidGemm256Swiglu = 12, // <256,256,2,4> with the fused SwiGLU epilogue (gate/up of prefill / log-prob chunks)
    kKidGemm256x160 = 13,   // <256,160,4,1> fused SwiGLU only (gate/up of a decode step in one round of workgroups on more CUs, and of up to 2816 rows where it fills its rounds better)
    kKidGemm128x160 = 14,   // <128,160,4,1> the same with four stages, where 256-row tiles would be half padding or too few
    kKidGemmSkinny = 15,    // gemm_skinny_kernel (few rows, every epilogue; a K split includes its reduction)
    kKidCount = 16,
};
// Has the runtime load the code objects of the GEMM kernels onto the current device now (it does so, a few MB each, at
// the first launch out of each of them otherwise).
hipError_t gemm_load_kernels();
hipError_t gemm_skinny_load_kernels();
// Which kernel launch_gemm picks for these arguments.
int gemm_kernel_id(const GemmArgs& a);
// The rest of its choice (host-only; for tests).
struct GemmPlan {
    int kernel_id;
    int splits;      // K ranges whose sums go through the scratch, 1: not split
    int first_rows;  // rows of the first of two launches, 0: one launch
    int waves;       // generic kernels: 1 for gemm_generic_wave_kernel
    int passing;     // weights asked for with the non-temporal hint (where few enough rows leave them to one reader)
    int norm_apart;  // kEpiAddF32: leaves an RMSNorm taken apart if asked for one; kEpiSwiglu: takes one
};
GemmPlan gemm_plan(const GemmArgs& a);
// Bytes of fp32 K-split partial sums launch_gemm would write for these arguments if the
// workspace were unlimited (0 = the problem is not split along K); a.ws / a.ws_bytes are ignored.
size_t gemm_splitk_scratch_bytes(const GemmArgs& a);
// Whether these arguments are a chunk of more than 512 rows that 128x128 tiles hold in one round: launch_gemm then finds a way
// with any amount of scratch, a K split that fits it or none.
bool gemm_narrow_tiles_hold(const GemmArgs& a);

// ---- elementwise ---------------------------------------------------------------
// x[r, :] = embed[tokens[idx(r)], :] as fp32, idx(r) = tok_index ? tok_index[r] : r;
// out-of-range ids and idx(r) < 0 give a zero row.
hipError_t launch_embed(const int32_t* tokens, const int32_t* tok_index, const void* embed, int dtype,
                        int vocab, int d, float* x, int rows, hipStream_t s);
// h[r, :] = x[src(r), :] / sqrt(mean(x^2) + eps) * gain, src(r) = row_idx ? row_idx[r] : r.
// x fp32, gain and h in `dtype`.
hipError_t launch_rmsnorm(const float* x, const int32_t* row_idx, const void* gain, int dtype, int d,
                          float eps, void* h, int rows, hipStream_t s);
// act[r, j] = silu(gu[r, j]) * gu[r, F + j]
hipError_t launch_swiglu(const void* gu, int dtype, int F, void* act, int rows, hipStream_t s);
// dst[r, :] = src[row_idx[r], :] (fp32 rows of width d)
hipError_t launch_gather_rows(const float* src, const int32_t* row_idx, int d, float* dst, int rows,
                              hipStream_t s);

// Rotate q and k of every row by its position, write k and v into the row's KV page.
struct RopeKvArgs {
    void* qkv;  // [rows, (Hq + 2 Hkv) dh], q rotated in place
    int dtype;
    int rows;
    int Hq, Hkv, dh;
    const float* rope;      // [max_pos, dh/2, 2] (cos, sin)
    const int32_t* row_seq;  // row -> sequence index (< 0: a padding row, nothing is written), or NULL: sequence = row
    const SeqDesc* seqs;
    int pos_add;             // added to every position (decode step)
    int single_row = 0;      // 1: every row is THE row of its sequence (position pos0 + pos_add) wherever it
                             // sits in the row buffer (decode step over a compacted batch)
    const int32_t* tables;
    const uint8_t* active;  // per row, or NULL
    void* kv_pool;
    KvGeom geom;
    int layer;
};
hipError_t launch_rope_kv(const RopeKvArgs& a, hipStream_t s);

// Copy the partially filled last prefix page of each group into the first private
// page of each of its rollouts, all layers.  src_page/dst_page per rollout; src < 0 = nothing.
hipError_t launch_fork_copy(void* kv_pool, int dtype, KvGeom geom, int n_layers, const int32_t* src_page,
                            const int32_t* dst_page, int n_rollouts, hipStream_t s);

// ---- attention over the paged cache --------------------------------------------
// Causal attention of packed rows: row i of sequence s (position pos0 + i + pos_add) sees
// positions [0, pos0 + i + pos_add] of that sequence's pages.
struct AttnArgs {
    const void* q;  // [rows, q_stride]; head h at column h * dh
    int64_t q_stride;
    void* out;  // [rows, Hq * dh]
    int dtype;
    int rows;
    int Hq, Hkv, dh;
    const int32_t* row_seq;  // or NULL: sequence = row; < 0: a padding row (skipped)
    int single_row = 0;      // as in RopeKvArgs
    const SeqDesc* seqs;
    int n_seqs;
    int max_seq_rows;  // largest n_rows among seqs (grid sizing)
    int pos_add;
    const int32_t* tables;
    const uint8_t* active;  // per row, or NULL
    const void* kv_pool;
    KvGeom geom;
    int layer;
    float scale;
    int path;  // 0 = pick, 1 = force generic
};
hipError_t launch_attn_chunk(const AttnArgs& a, hipStream_t s);
// Whether the MFMA attention kernels take these arguments.
bool attn_uses_mfma(const AttnArgs& a);

// Decode attention with a shared prefix: rollout rows r = g * G + i, one new query row
// each; rows of a group share the group's first shared_pages[g] pages.
struct DecodeAttnArgs {
    AttnArgs base;               // seqs = per-rollout descriptors (n_rows = 1); base.rows = query rows
    int n_rollouts;              // rollout rows r = g * G + i covered (= base.rows unless compacted)
    const int32_t* row_of = nullptr;  // compacted batch: rollout -> query / output row, < 0 = finished
                                      // (base.row_seq is then the inverse map); NULL: row = rollout
    int G;
    const int32_t* shared_pages;  // per group: full prefix pages shared by its rollouts
    int max_shared_pages;
    int max_own_pages;  // private pages any rollout can hold at this step
    float* partial;     // split-KV scratch
    size_t partial_floats;
};
hipError_t launch_attn_decode(const DecodeAttnArgs& a, hipStream_t s);
size_t attn_decode_partial_floats(int rows, int Hq, int dh, int max_shared_pages);

// ---- sampling, log-probs, advantages -------------------------------------------
struct SampleArgs {
    const float* logits;
    int n_logit_rows, vocab;
    int64_t row_stride;
    const int32_t* row_map;
    int n_out_rows;
    float inv_t;
    uint64_t seed;
    const uint64_t* seq_id;
    uint32_t step;
    int32_t* tokens_out;
    float* logprob_out;
    int eos_id;          // < 0: no end-of-sequence token
    uint8_t* active;     // in/out per output row, or NULL: all rows live
    int32_t* lengths;    // in/out per output row (tokens generated so far), or NULL
    const float* row_max = nullptr;  // per logits row: its maximum, or NULL: the kernel finds it
};
hipError_t launch_sample(const SampleArgs& a, hipStream_t s);

// out[r] = logits[r, target[r]] * inv_t - logsumexp(logits[r, :] * inv_t)
// out[r] = (target_logit[r] - M) / T - ln(sum_b part[r, b].sum * 2^((part[r, b].max - M) k2)),
// M = max_b part[r, b].max: the log-softmax value of the target from the pieces kEpiLse leaves.
// (NaN for a target outside [0, vocab))
hipError_t launch_lse_combine(const float* part, int blocks, const float* target_logit, const int32_t* target,
                              int vocab, float inv_t, float* out, int rows, hipStream_t s);
hipError_t launch_lse_gather(const float* logits, int64_t row_stride, int vocab, const int32_t* target,
                             float inv_t, float* out, int rows, hipStream_t s);

// ---- experience cache (cache.hip) ----------------------------------------------
hipError_t launch_cut_pack(const int32_t* prompts, int64_t prompt_stride, const int32_t* prompt_len,
                           const int32_t* pool, int64_t pool_stride, const int32_t* question,
                           const int32_t* cu_len, int n_groups, int32_t* out, hipStream_t s);
hipError_t launch_cache_update(int32_t* pool, int64_t pool_stride, int32_t* answer_len, const int32_t* question,
                               const int32_t* m,
                               const int32_t* tokens, int64_t tok_stride, const int32_t* lengths,
                               const float* rewards, const float* u, const int32_t* g_prime, int n_groups, int G,
                               float eps, int32_t* chosen_out, hipStream_t s);

hipError_t launch_objective(const float* lp_new, const float* lp_old, const float* lp_ref, const int32_t* cu,
                            const float* adv, int n_groups, int G, float eps_clip, float beta, float* tok_out,
                            double* per_rollout, float* j_out, hipStream_t s);
hipError_t launch_shape_rewards(const float* rewards, const int32_t* lengths, int n_groups, int G, float alpha,
                                float lo, float hi, float* out, hipStream_t s);
// Compaction of a decode batch: live[c] = c-th rollout row r < n_rows with active[r] != 0 (in
// increasing r; -1 for c >= their number), row_of[r] = c or -1, and their number to *count_dev
// and, if given, as (generation << 32 | number) to *mailbox (device address of mapped host memory).
hipError_t launch_compact_rows(const uint8_t* active, int n_rows, int32_t* live, int32_t* row_of,
                               int32_t* count_dev, uint64_t* mailbox, uint32_t generation, hipStream_t s);
hipError_t launch_advantages(const float* rewards, int n_groups, int G, int ddof, float eps, float* adv,
                             hipStream_t s);

}  // namespace rpo
