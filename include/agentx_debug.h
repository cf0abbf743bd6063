/*
 * agentx_debug.h - test-only entry points of libagentx.so: they expose single kernels and the
 * intermediates of the last forward so that GPU tests can localise a mismatch against the CPU
 * oracle.  Not part of the serving API; they synchronise the device.
 */
#ifndef AGENTX_DEBUG_H
#define AGENTX_DEBUG_H

#include "agentx.h"

#ifdef __cplusplus
extern "C" {
#endif

/* C = A[M,K] * W[N,K]^T through the library's GEMM dispatcher (the projection / MLP / LM-head
 * contraction of the decoder).  All pointers are device memory.  dtype AX_F32: A, W, W2 fp32;
 * AX_BF16: W, W2 bf16 and A fp16 (the activation type of bf16-weight models).  epilogue: 0 store
 * float C[M,N]; 1 float C[M,N] += ; 2 SwiGLU, C (activation type) = silu(A W^T) * (A W2^T).
 * AX_BF16 needs K % 64 == 0 and N % 16 == 0.  Synchronises. */
ax_status ax_dbg_gemm(int dtype, int epilogue, const void *A, const void *W, const void *W2, void *C,
                      int M, int N, int K, void *hip_stream);

/* How the attention of a verify step or short extend would be launched: `items` = tiles of 32 stacked rows x KV heads, max_steps =
 * key steps of 32 of the longest sequence.  Writes the wavefronts per block (1 or 4) and the key slices per item.  Host only. */
ax_status ax_dbg_split_plan(const ax_model_config *cfg, int items, int max_steps, int *waves, int *slices);

/* The pass over the keys of a prefix that the sequences of a call share: groups of 128 of the call's stacked rows, and key slices of each.  own_tiles:
 * tiles of 32 stacked rows of the sequences, own_steps: key steps of 32 of them all behind the prefix; one_launch: these go in one launch with the pass
 * (ax_dbg_split_plan: 4 wavefronts).  Host only. */
ax_status ax_dbg_shared_plan(const ax_model_config *cfg, int rows, int keys, int own_tiles, long long own_steps, int one_launch, int *groups,
                             int *slices);

/* Whether that many records (tiles of 32 stacked rows x KV heads) of so many key slices each (a shared prefix's among them) are added up by a block
 * per record (1) or by blocks of 4 output channels (0).  Host only. */
ax_status ax_dbg_merge_plan(int records, int slices, int *by_record);

/* What a bf16-weight GEMM of more than 256 rows runs on: *kernel (static text) "block", "tile" or "stream", rows of A and of W per block
 * (SwiGLU: half of the latter gate, half up) and K slices; "" and zeros for fewer rows or N not a multiple of 64.  epilogue as
 * ax_dbg_gemm, 3 = QKV (rotary, KV append).  split: activations in hi + lo parts.  split_ws_bytes: scratch for K slices.  Host only. */
ax_status ax_dbg_gemm_plan(int epilogue, int M, int N, int K, int split, size_t split_ws_bytes, const char **kernel, int *rows, int *cols,
                           int *slices);

/* The same for activations in panels (M > 256, N % 64 == 0: only the block kernel reads those), and whether a call of that many rows of a
 * model keeps its layers' activations in panels: 1 or 0 (rows, or strips: ax_dbg_gemm_regs).  Host only. */
ax_status ax_dbg_panel_plan(int epilogue, int M, int N, int K, int split, size_t split_ws_bytes, int *rows, int *cols, int *slices);
ax_status ax_dbg_layer_panels(const ax_model_config *cfg, int rows, int *panels);

/* What a layer's GEMM of 17 to 256 rows runs on (epilogues 1 to 3, arguments as ax_dbg_gemm_plan): *kernel "regs" (ax_dbg_gemm_regs) or, with split,
 * "block" (ax_dbg_gemm_block, on strips).  Host only. */
ax_status ax_dbg_strip_plan(int epilogue, int M, int N, int K, int split, size_t split_ws_bytes, const char **kernel, int *rows, int *cols,
                            int *slices);

/* One GEMM of a bf16-weight layer on a block shape of the many-row kernel that the caller names, with everything a layer uses: hi + lo
 * activations, a pending RMSNorm of A's rows, K slices and each epilogue.  All pointers are device memory; weights row-major bf16.
 * rows x cols: 256 x 256, 128 x 256 or 128 x 128 (not for SwiGLU).  N % 64 == 0, K % 64 == 0, head_dim 64 or 128. */
typedef struct {
    int epilogue;                       /* 0 C = product; 1 C += product, C16 = C * gain; 2 C16 = silu(A W^T) (A W2^T); 3 QKV */
    int rows, cols, slices;             /* slices > 1 (epilogues 1 and 3): K % (32 slices) == 0, split_ws of slices x M x N floats */
    int M, N, K;
    const void *A; long long a_lo;      /* fp16 [M, K]; lo parts this many elements behind (0 = none) */
    const void *W, *W2;                 /* [N, K] */
    const float *ssq; int n_parts;      /* partial sums of x^2 of the rows of A, [M][n_parts]; NULL = A as it is */
    float eps;
    float *C;                           /* [M, N] (epilogues 0, 1) */
    void *C16; long long c_lo;          /* fp16 [M, N]; epilogue 3: q after rotary [M, n_q_heads * head_dim]; lo parts as for A */
    const void *gain; float *ssq_out;   /* epilogue 1: bf16 [N]; [M][*n_parts_out], room for M * N / 8 */
    int n_parts_out;                    /* written */
    int n_q_heads, n_kv_heads, head_dim;                        /* epilogue 3: N = (n_q_heads + 2 n_kv_heads) * head_dim ... */
    void *pool; long long pool_blocks;                          /* ... a one-layer KV pool of 16-token blocks ... */
    const int *row_pos, *row_slot; const float *cos, *sin;      /* ... position and slot of the rows, rotary tables [pos][head_dim / 2] */
    void *split_ws; size_t split_ws_bytes;
    int a_panels, c_panels;             /* A (and ssq, as [n_parts][M]), C16 (and ssq_out; epilogues 1 and 2) in panels of 16 rows, as calls of many
                                           rows hold them: 8 columns of a panel's rows at a time, each row's 8 side by side.  2: in strips, 32 columns
                                           of all rows at a time, panel after panel of 16 rows (the last one too: C16 has room for whole panels), inside
                                           them as panels, ssq and ssq_out as beside panels; refused without lo parts.  0: in rows */
} ax_dbg_block_gemm;
ax_status ax_dbg_gemm_block(ax_dbg_block_gemm *args, void *hip_stream);
/* The same on the kernel of 17 to 256 rows (any M <= 256 here): a tile of `rows` x `cols` (SwiGLU: half of them gate, half up), refused where there is
 * no such tile; epilogues 1 to 3, slices for epilogue 1 only.  Strips with or without lo parts; ssq and ssq_out are [n_parts][M] beside strips and
 * beside panels of more than 32 rows. */
ax_status ax_dbg_gemm_regs(ax_dbg_block_gemm *args, void *hip_stream);

/* Work of the attention of one call of long extends (n sequences of P cached and T new tokens): items (128 stacked rows x a range of keys),
 * groups of rows whose keys several items share, and the partial-record slots those use per KV head.  Host only. */
ax_status ax_dbg_attention_items(const ax_model_config *cfg, int n, const int *P, const int *T, int *items, int *merges, int *slots);

/* The residual GEMM as a bf16-weight decoder layer runs it (O and down projections): x[M,N] (float,
 * updated in place) += A[M,K] W[N,K]^T, then a16[M,N] = fp16(x * gain[n]) and per-row partial sums
 * of x^2: ssq[m * (*n_parts) + p], p < *n_parts (written by the call; at most N / 8), whose sum
 * over p is sum_n x[m,n]^2.  A fp16, W and gain bf16, all device memory; ssq must hold M * N / 8
 * floats.  K % 64 == 0, N % 16 == 0, and N % 32 == 0 with more than 16 rows (N is a model width there).
 * split_ws / split_ws_bytes: device scratch for K-slice partial products (the launcher
 * cuts K only when scratch is given and it pays); 0 bytes = never.  Synchronises. */
ax_status ax_dbg_gemm_residual(const void *A, const void *W, const void *gain, float *x, void *a16, float *ssq,
                               int *n_parts, int M, int N, int K, void *split_ws, size_t split_ws_bytes,
                               void *hip_stream);

/* Times `iters` back-to-back launches of the same GEMM with HIP events on hip_stream and writes the
 * average microseconds per launch to *avg_us.  Launch i reads its weights at W + (i % w_count) *
 * w_stride_bytes (same for W2), so that a set of weight copies larger than the caches can be
 * cycled through (w_count = 1: always the same weights).  Arguments otherwise as ax_dbg_gemm. */
ax_status ax_dbg_gemm_time(int dtype, int epilogue, const void *A, const void *W, const void *W2, void *C,
                           int M, int N, int K, int iters, size_t w_stride_bytes, int w_count,
                           float *avg_us, void *hip_stream);

/* Plain device-to-device copy kernel (16-byte words, grid-stride) of `bytes` bytes (a multiple of
 * 16): the kernel of known traffic that hardware-counter readings are scaled against. */
ax_status ax_dbg_copy(void *dst, const void *src, size_t bytes, void *hip_stream);

/* What the machine delivers, measured beside the nominal peaks the roofline fractions are quoted
 * against.  buf: device memory of `bytes` bytes (a multiple of 16; use a few hundred MiB so that no
 * cache holds it).  Runs 2 untimed and `reps` timed launches each of (i) a read-only stream over buf,
 * (ii) the plain copy kernel from the first half of buf to the second, (iii) a register-resident
 * fp16 MFMA loop (32x32x16, fp32 accumulate) on every compute unit; HIP events on hip_stream.
 * Writes GB/s read, GB/s copied (read + written bytes) and TFLOP/s.  Synchronises. */
ax_status ax_dbg_peaks(void *buf, size_t bytes, int reps, float *read_gbs, float *copy_gbs,
                       float *mfma_f16_tflops, void *hip_stream);

/* What one compute unit can pull.  256 workgroups of 512 threads (one per compute unit of an otherwise idle MI355X)
 * each read a region of their own with many more loads in flight than the memory pipeline keeps outstanding: a 64 KB
 * region 256 times (served by the L2 of the workgroup's XCD from the second pass on), then a region of bytes / 256 once
 * (from HBM, all compute units pulling together; whatever of buf the 256 MB memory-side cache still holds from the caller's own
 * last pass over it comes from there - use a buffer of 1 GiB or more).  buf: device memory of `bytes` bytes, at least 256 MiB and a multiple of
 * 4096, read only.  Writes GB/s PER COMPUTE UNIT for both.  Synchronises. */
ax_status ax_dbg_cu_fill(void *buf, size_t bytes, float *l2_gbs_per_cu, float *hbm_gbs_per_cu, void *hip_stream);

/* The two ways to order the dependent phases of a step, timed: `rounds` back-to-back launches of an
 * empty kernel of `blocks` workgroups of 512 threads on hip_stream (microseconds per kernel boundary),
 * and one launch of the same shape that crosses a barrier over all its workgroups `rounds` times
 * (microseconds per barrier; two-level counters, device-scope atomics, fences on both sides).  blocks: a
 * multiple of 8, at most 256 (one workgroup per compute unit, so that all are resident on an otherwise
 * idle device); buf: at least 4096 bytes of device memory, overwritten.  Every wait of the barrier kernel
 * is bounded: AX_ERR_DEVICE if a workgroup gave up.  Synchronises. */
ax_status ax_dbg_phase_order(void *buf, size_t bytes, int blocks, int rounds, float *boundary_us,
                             float *barrier_us, void *hip_stream);

/* Copies a workspace buffer as left by the last ax_extend* call to host memory (synchronises).
 * which: 0 residual stream x float[rows][d_model]; 1 qkv float[rows][(Hq+2Hkv)*hd] (pre-rotary,
 * last layer); 2 q after rotary, act[rows][Hq*hd]; 3 attention output act[rows][Hq*hd];
 * 4 SwiGLU activations act[rows][d_ff]; 5 LM-head input, where act is float for AX_F32 models
 * and fp16 for AX_BF16 models.  AX_F32: buffer 5 is rmsnorm(x) * gain of the n_out output rows.
 * AX_BF16: buffer 1 is unused and buffer 5 is fp16(x * final gain) of all rows (the division by
 * the rms happens inside the LM-head GEMM).
 * 12 - 15: the lo parts of buffers 2 - 5 of a model with split activations (2 - 5 are the hi parts).
 * Copies min(bytes, buffer size) bytes. */
ax_status ax_dbg_read(ax_model *model, int which, void *host_dst, size_t bytes);

/* The workspace of a model is cut into regions (rotary tables, descriptor slots, residual stream, activations,
 * norm partial sums, fp32 q/k/v of fp32 models, q, attention output, SwiGLU activations, attention slice records, GEMM
 * slabs, logits chunk, argmax scratch, argmax output, result words, packed weights - in this order), each followed by
 * 256 guard bytes that ax_model_create fills with a pattern and nothing may write.  Synchronises the device, reads
 * the guards back and writes the index of the first region whose guard was touched (an overrun of that region), or
 * -1 if all are intact. */
ax_status ax_dbg_check_guards(ax_model *model, int *first_bad);

/* ax_verify replays one captured HIP graph per (draft count, key-slice count); enable = 0 makes it
 * enqueue the same launches one by one instead (the reference a test compares the replays with). */
ax_status ax_dbg_use_graphs(ax_model *model, int enable);

/* Per-kernel timing with HIP events on the caller's stream.  While enabled, every launch of the
 * classes below inside ax_extend* / ax_verify is bracketed by a pair of events (this perturbs
 * the step a little, so enable it only for steps whose total time is not reported).
 * Classes: 0 QKV projection, 1 attention (split + combine), 2 O projection, 3 SwiGLU gate/up,
 * 4 down projection, 5 LM head, 6 an empty bracket (once per layer of a bf16-weight model): what a
 * pair of events measures around nothing, to be subtracted.  ax_dbg_profile_read synchronises, adds up the elapsed
 * milliseconds and the launch count of each class since the last read and clears them. */
#define AX_DBG_PROFILE_CLASSES 7
ax_status ax_dbg_profile(ax_model *model, int enable);
ax_status ax_dbg_profile_read(ax_model *model, double *ms_by_class, int64_t *launches_by_class);

#ifdef __cplusplus
}
#endif
#endif /* AGENTX_DEBUG_H */
