// Internal interface between the C-ABI host code and the HIP kernels (gfx950 only).
// Every launcher only enqueues work on `stream`; shapes are validated by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "kv_geom.h"

namespace ax {

// F32: fp32 weights, activations and KV.  BF16: bf16 weights; activations and KV are fp16
// ("the activation type" below), products on the fp16 MFMA with fp32 accumulation.
enum DType { F32 = 0, BF16 = 1 };

constexpr int SHARED_TILES = 4;
// Device views of the per-call descriptor (one packed int32 buffer uploaded per call).
struct StepView {
    const int* row_tok;     // [n_rows] token id
    const int* row_pos;     // [n_rows] absolute position
    const int* row_seq;     // [n_rows] sequence index within the call
    const int* row_slot;    // [n_rows] KV slot the row is written to: block id * 16 + position % 16
    const int* seq_P;       // [n_seq] cached length before the call
    const int* seq_T;       // [n_seq] new rows
    const int* seq_row0;    // [n_seq] first row
    const int* seq_bt;      // [n_seq] offset of the sequence's block table inside bt
    const int* bt;          // concatenated block tables
    const int* out_rows;    // [n_out] rows that go through the LM head
    // attention work, 8 ints (32 bytes, aligned) a record.  Stacked rows of a sequence: row t of query head g of a KV head is t * G + g.
    //   tile_nq == 1 (fp32 models; verify steps and short extends): n_tiles records of one 32-row tile each -
    //     sequence, first stacked row, P, T, first row of the sequence, block-table offset, 0, first key;
    //     then (n_tiles_shared > 0: sequences whose block tables start alike) the items of a pass of groups of SHARED_TILES tiles over
    //     ALL rows of the call against keys [0, shared_len), shared_splits items per group
    //   tile_nq == 4 (long extends): n_items ITEMS of 4 tiles and a range of key steps of 32 each -
    //     slot of the partial records (-1: all the keys, writes the output itself), first stacked row, P, T, first row of the
    //     sequence, block-table offset, end of the range, first step;
    //     then n_merge records of the tiles several items share -
    //     first slot, first stacked row, number of slots, T, first row of the sequence, 0, 0, 0
    const int* tile_info;
    int n_rows, n_seq, n_out, n_tiles, tile_nq, n_items, n_merge;
    int n_tiles_shared, shared_len, shared_splits;                 // 0 groups = no shared-prefix pass
};

enum Epilogue { EPI_STORE_F32 = 0, EPI_RESIDUAL = 1, EPI_SWIGLU = 2, EPI_QKV = 3 };

// Rotary + KV-append part of the QKV epilogue (bf16-weight models).
struct RopeArgs {
    KVGeom kv;
    int layer, n_q_heads;
    void* q_out;                      // fp16 [n_rows, Hq, hd]
    const int *row_pos;               // [n_rows] absolute position
    const int *row_slot;              // [n_rows] KV slot of the row: block id * 16 + position % 16
    const float *cos, *sin;           // [max_pos][hd/2]
};

// Split activations.  An fp16 value keeps 11 significant bits; the rounding of the five activation tensors a
// layer hands from kernel to kernel is what separates the logits of a deep, wide decoder from the exact ones
// (measured: ~1B x 16 layers 5e-3, ~3B x 28 layers 1.3e-2, ~8B x 32 layers 2.7e-2 max-abs).  A model created
// with split activations stores every such tensor as TWO fp16 values per element, hi = fp16(v) and
// lo = fp16(v - hi) (together ~22 bits), the second tensor `*_lo_off` elements behind the first, and every
// consumer multiplies both parts against the SAME weight fragment (two MFMAs per fragment: no extra weight
// traffic, twice the matrix-core work and activation traffic).  An offset of 0 means "not split".
//
// Both parts have to come from the same fp32 v.  Left alone the compiler folds a product in front into the conversion (v_fma_mixlo: one
// rounding from the exact product) for one of them and rounds to fp32 first for the other; where the two disagree - near a tie, one value
// in 30 000 - hi + lo was a whole fp16 step off.  So v is made a value of its own before it is split.
__device__ __forceinline__ float split_value(float v) {
    asm("" : "+v"(v));
    return v;
}

// How the activations of a call lie between the kernels of a layer (gemm_layer_layout): an [M, K] matrix
//   in rows;
//   in panels of 16 rows, like the packed weights, each k-group of 8 of a panel as one run of its rows.  A last panel of fewer rows has shorter
//     runs, so the matrix takes no more room than as rows.  A GEMM's copy of 16 rows x 32 k to LDS is then 1 KB of whole 128-byte lines,
//     where rows make it 16 half lines;
//   in strips: 32 k of all rows at a time, panel after panel, the last one of 16 rows like the others - what a kernel that takes many row tiles
//     at once reads is one run, at one offset for all calls of as many panels.
enum ActLayout : unsigned char { ACT_ROWS = 0, ACT_PANELS = 1, ACT_STRIPS = 2 };
__host__ __device__ __forceinline__ long long act_index(ActLayout layout, int m, int k, int M, int K) {
    // (one formula: rows are panels of one row, and a strip's panels lie 512 apart; three formulas to choose from cost every epilogue 0.1 us)
    const int in_panel = layout == ACT_ROWS ? 0 : m & 15, first = m - in_panel;
    const int run = layout == ACT_ROWS ? 1 : layout == ACT_STRIPS || M - first >= 16 ? 16 : M - first;        // rows side by side
    const int strip = layout == ACT_STRIPS ? (M + 15) / 16 * 512 : run * 32;
    return (long long)first * (layout == ACT_STRIPS ? 32 : K) + in_panel * 8 + (long long)(k >> 5) * strip + ((k >> 3) & 3) * (run * 8) + (k & 7);
}

// The same for rows and panels only: what the few-row kernels write.  (With the formula for all three a residual GEMM of 9 rows took 8.32 us, 8.24 with this.)
__host__ __device__ __forceinline__ long long act_index_few(bool panels, int m, int k, int M, int K) {
    if (!panels) return (long long)m * K + k;
    const int first = m & ~15, rows = M - first < 16 ? M - first : 16;
    return (long long)first * K + (long long)(k >> 3) * (rows * 8) + (m & 15) * 8 + (k & 7);
}
// Partial sums of x^2 behind activations that await their norm: [rows][parts]; behind strips, and panels of more than 32 rows, [parts][rows], so
// that a thread that adds up a row reads beside its neighbours.
__host__ __device__ __forceinline__ bool ssq_by_part(ActLayout layout, int M) { return layout == ACT_STRIPS || (layout == ACT_PANELS && M > 32); }
__host__ __device__ __forceinline__ long long ssq_index(bool by_part, int m, int part, int M, int nparts) {
    return by_part ? (long long)part * M + m : (long long)m * nparts + part;
}

// One GEMM of a bf16-weight model: C = A[M,K] * W[N,K]^T, A fp16, W bf16.
struct GemmArgs {
    const void* A;                    // fp16 [rows, K]
    long long a_lo_off;               // split activations: the lo parts of A lie this many elements behind A (0 = none)
    long long c_lo_off;               // ... and the lo parts of C16 (and of rope.q_out) this many elements behind it
    ActLayout a_layout, c_layout;     // of A and C16
    int a_total_rows;                 // rows A has (a gather picks M of them)
    const int* a_rows;                // optional gather: A row of output row m is a_rows[m]
    const void *W, *W2;               // [N, K] packed by launch_pack_weights (fp16, MFMA operand order); W2 only for EPI_SWIGLU
    int M, N, K;
    // deferred RMSNorm of the A rows: ssq[row][nparts] partial sums of x^2 over d_norm columns;
    // the accumulators are scaled by 1 / sqrt(sum / d_norm + eps).  NULL = no scaling.
    const float* ssq;
    int nparts, d_norm;
    float eps;
    float* Cf;                        // EPI_STORE_F32: out [M,N]; EPI_RESIDUAL: x [M,N], updated in place
    void* C16;                        // EPI_SWIGLU: fp16 out [M,N]; EPI_RESIDUAL: fp16(x * gain_next) [M,N]
    const void* gain_next;            // EPI_RESIDUAL: bf16 [N] gain of the next norm, NULL = plain residual add
    float* ssq_out;                   // EPI_RESIDUAL: [M][parts] partial sums of x^2, parts = what launch_gemm_bf16 returns
    RopeArgs rope;                    // EPI_QKV
    // EPI_RESIDUAL on the tile kernels with few output tiles: K may be cut into ksplit slices (chosen by
    // the launcher) whose fp32 partial products go to split_ws [ksplit][M][N]; a second kernel
    // adds them up and runs the residual epilogue.  split_ws == NULL: never split.
    float* split_ws;
    size_t split_ws_bytes;
    int ksplit;
};
constexpr int SPLITK_MAX = 8;
// EPI_RESIDUAL with gain_next: returns the number of partial sums of x^2 per row the launch leaves in
// ssq_out (rows are that many floats apart): the consumer of the pending norm passes it as nparts.
// It depends on which kernel ran (a few per row after a K-split reduce kernel, N / 64, N / 32 or N / 8-16
// from kernels that finish a column block on their own).  Other epilogues return 0.
// EPI_QKV writes its raw products to split_ws first on the tile kernel (where the plan takes it, up to 512 rows) and in K slices; of plans that do
// not, -1 and nothing launched if one [M, N] fp32 slab does not fit there.
int launch_gemm_bf16(Epilogue epi, const GemmArgs& g, hipStream_t s);
// The plan of a GEMM of more than 256 rows that are not gathered ("" = fewer rows, or N not a multiple of 64): kernel ("block", "tile" or
// "stream"), rows of A and of W per block (EPI_SWIGLU: half of the latter gate, half up) and K slices.
struct GemmPlan { const char* kernel; int rows, cols, slices; };
GemmPlan gemm_plan(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes);
GemmPlan gemm_panel_plan(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes);      // with A in panels
// The plan of a layer's GEMM (not EPI_STORE_F32) of 17 to 256 rows: "regs", or in hi + lo parts "block".
GemmPlan gemm_strip_plan(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes);
// How the layers of a call of M rows keep their activations from kernel to kernel: all four GEMMs then run with this a_layout.  Panels up to 16 rows
// on the few-row kernel, to 32 rows (plain activations) on the register kernel and from 257 on the block kernel, on its plan for panels; strips
// on the register kernel and, in hi + lo parts, on the block kernel.  N of a GEMM: the layer's sizes, all multiples of 64.
ActLayout gemm_layer_layout(int M, int d_model, int qkv, int qdim, int d_ff, bool split, size_t ws_bytes);
// A GEMM on the block kernel with the shape and slices of `rows`, `cols`, `slices` whatever the plan would say (tests); returns as launch_gemm_bf16.
int launch_gemm_block_as(Epilogue epi, const GemmArgs& g, int rows, int cols, int slices, hipStream_t s);
// The same for the register kernel (up to 256 rows), and whether there is such a tile.
int launch_gemm_regs_as(Epilogue epi, const GemmArgs& g, int rows, int cols, int slices, hipStream_t s);
bool gemm_regs_built(Epilogue epi, bool split, int rows, int cols, int slices);
// Repacks a row-major bf16 [N, K] matrix (N % 16 == 0, K % 32 == 0) into what every bf16-model GEMM
// kernel reads: fp16 values in 16-row panels, 32-k chunks in MFMA operand order; src and dst must not overlap.
// `bad` (device int, may be NULL) is set to 1 if some weight does not survive the narrowing (not finite in fp16).
void launch_pack_weights(const void* src, void* dst, int N, int K, hipStream_t s, int* bad = nullptr);
// bf16-weight models: x[r,:] = emb[tok], a[r,:] = fp16(x * gain), ssq[r][0] = sum x^2, ssq[r][1..nparts) = 0
// a_lo_off != 0: also the lo parts fp16(x * gain - a), that many elements behind a.  d % 8 == 0
void launch_embed_norm(const void* emb, const int* row_tok, const void* gain, float* x, void* a, long long a_lo_off, ActLayout layout,
                       float* ssq, int nparts, int n_rows, int d, hipStream_t s);

// fp32 models: h[i, :] = rmsnorm(x[rows[i], :]) * gain
void launch_rmsnorm_f32(const float* x, const float* gain, float* h, const int* rows, int n_rows, int d, float eps, hipStream_t s);
// One GEMM of an fp32 model: C = A[M,K] * W[N,K]^T.  EPI_STORE_F32: C [M,N].  EPI_RESIDUAL: C [M,N] = res + product.
// EPI_SWIGLU: C [M,N] = silu(A W^T) * (A W2^T).  EPI_QKV: rotary on q and k, q -> rope.q_out [M, Hq, hd], k and v -> the
// rows' KV slots, C [M,N] = the products before the rotation; N = (Hq + 2 Hkv) * hd.
struct GemmF32Args {
    const float* A;                   // [rows, K]
    const int* a_rows;                // optional gather: A row of output row m is a_rows[m]
    const float *W, *W2;              // [N, K]; W2 only for EPI_SWIGLU
    const float* gain;                // [K]: the A rows are RMS-normalised with this gain first; NULL = taken as they are
    float eps;
    int M, N, K;
    float* C;
    const float* res;                 // EPI_RESIDUAL: NULL = C itself (updated in place)
    const int* res_rows;              // ... row of res that belongs to output row m (NULL = m)
    RopeArgs rope;                    // EPI_QKV (q_out is fp32)
};
void launch_gemm_f32(Epilogue epi, const GemmF32Args& g, hipStream_t s);
// C = A[M,K] * W[N,K]^T with fp32 accumulation.  A is of the activation type, W of the weight
// type.  EPI_STORE_F32: C float [M,N].  EPI_RESIDUAL: C float [M,N] += .
// EPI_SWIGLU: C (activation type) [M,N] = silu(A*W^T) * (A*W2^T).
void launch_gemm(DType dt, Epilogue epi, const void* A, const void* W, const void* W2, void* C,
                 int M, int N, int K, hipStream_t s);
// Causal attention of the new rows over the paged cache (which already holds the new rows).
// out [n_rows, Hq, hd] in the activation type.  `partials` is fp32 scratch for the split-KV
// path (bf16 only); n_splits >= 1, split_waves 1 or 4 wavefronts per block of it.
// q_lo_off / out_lo_off: split activations (see GemmArgs): lo parts of q read, lo parts of out written (0 = none).  out_layout (bf16
// only): how out lies.
void launch_attention(DType dt, const void* q, void* out, KVGeom kv, int layer,
                      const StepView& sv, int n_q_heads, float* partials, int n_splits, int split_waves,
                      hipStream_t s, long long q_lo_off = 0, long long out_lo_off = 0, ActLayout out_layout = ACT_ROWS);
// Which kernel adds up the key slices of single tiles: a block per record (tile x KV head) that walks the record's slices (true), or blocks of 4
// output channels that spread a record's slices over threads (false).  The first takes about 4 us + 0.4 a slice (head_dim 64: 0.2) while there is a
// CU for every record, the second 2 us + 0.1 a record (0.05), so the line lies at records / 5 slices.  First / second in us, head_dim 128: 64 records
// with 17 / 24 slices 10.9 and 7.9 / 12.7 and 8.0, 96 with 10 / 18 7.5 and 9.6 / 11.0 and 10.4, 128 with 18 11.1 and 13.2, 256 with 10 9.4 and 21.9;
// head_dim 64: 64 with 17 7.4 and 5.0, 128 with 18 8.2 and 7.8, 256 with 10 6.7 and 12.3.  Over 32 slices the second, up to 128 records: 17.9 and 14.9.
inline bool attention_merge_by_record(int records, int slices) { return records >= 64 && slices <= 32 && slices <= records / 5; }
// Floats of `partials` launch_attention needs for n_tiles q tiles (of 32 rows) and n_splits splits.
size_t attention_partial_floats(int n_tiles, int n_kv_heads, int head_dim, int n_splits);
// out[r] = argmax of logits[r, 0..V), lowest index on ties.  scratch: 2*rows*ARGMAX_PARTS ints.
constexpr int ARGMAX_PARTS = 64;
void launch_argmax(const float* logits, int rows, int V, int* out, int* scratch, hipStream_t s);
// Greedy acceptance per sequence of a verify call: the sequence's rows are [pending, drafts],
// g[row] the greedy token after each row.  result[2s] = a (longest prefix of the drafts equal to
// g), result[2s + 1] = g[row0 + a].
void launch_accept(const int* g, const StepView& sv, int* result, hipStream_t s);
// The same two steps fused for verify calls whose rows fit one LM-head pass: launch_argmax_partials
// is stage 1 alone (per row ARGMAX_PARTS (value, id) candidates into scratch), launch_argmax_accept
// finishes every row of a sequence (g[row], as launch_argmax would write it), votes, and writes
// (a, next token) to result and - when result_host is given: pinned host memory the device can
// address - straight to the host, so no copy has to follow.  At most ACCEPT_MAX_ROWS rows per sequence.
constexpr int ACCEPT_MAX_ROWS = 1024;
void launch_argmax_partials(const float* logits, int rows, int V, int* scratch, hipStream_t s);
void launch_argmax_accept(const int* scratch, int rows, int* g, const StepView& sv, int* result, int* result_host,
                          hipStream_t s);
// Plain copy of n16 16-byte words (calibration kernel for hardware counters).
void launch_plain_copy(void* dst, const void* src, size_t n16, hipStream_t s);
void launch_read_stream(const void* src, size_t n16, void* sink, hipStream_t s);   // read-only stream; sink: 4 writable bytes, never written
double launch_mfma_loop(int iters, void* sink, hipStream_t s);                    // register-resident fp16 MFMA loop; returns its flops
void launch_cu_fill(const void* src, size_t words_per_block, int blocks, int passes, void* sink, hipStream_t s);   // block b reads words [b, b + 1) * words_per_block, `passes` times; sink never written
void launch_grid_barrier(void* ctr, int* err, int blocks, int rounds, hipStream_t s);   // ctr: 3072 zeroed bytes; blocks: a multiple of 8, all resident
void launch_boundary(void* sink, int blocks, hipStream_t s);                          // an empty kernel of `blocks` x 512 threads; sink never written
// Copy one KV block (all layers, K and V, all heads) src -> dst: copy on write.
void launch_block_copy(DType dt, KVGeom kv, int n_layers, int src, int dst, hipStream_t s);

// Gather (to_image) or scatter the blocks `ids[0..n_seq_blocks)` of a sequence between the pool and
// an image buffer (device-accessible memory) that holds them back to back in logical order.
// last_fill: tokens in the last block (export zero-fills the slots beyond).
void launch_kv_image(bool to_image, DType dt, KVGeom kv, int n_layers, const int* ids, int n_seq_blocks,
                     void* image, int last_fill, hipStream_t s);

}  // namespace ax
