// Device helpers shared by the GEMM kernels of bf16-weight models: types, activation stores, the packed weight layout and
// the 1 / rms tables of the deferred RMSNorm.
#pragma once

#include "kernels.h"

namespace ax {

typedef __bf16 bf16;
typedef _Float16 f16;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }
// The same for epilogues with 64 results a lane: the division without the scaling a divisor of 1 or more does not need (7 instructions
// instead of 11).  One Newton step makes the reciprocal good to half a unit, one residual the quotient; the quotient misses
// correct rounding only within 2^-45 of a tie.  fixup: infinities and NaNs as a division has them.
__device__ __forceinline__ float silu_lean(float g) {
    const float d = 1.0f + __expf(-g);
    float r = __builtin_amdgcn_rcpf(d);
    r = fmaf(fmaf(-d, r, 1.0f), r, r);
    const float q = g * r;
    return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-d, q, g), r, q), d, g);
}

// 8 bf16 (one 16-byte fragment) -> 8 fp16.  A bf16 is the top half of an fp32, so each half of
// a dword becomes an fp32 by a shift or a mask; bf16 has fewer significant bits than fp16, so
// the round-toward-zero pack is exact in fp16's normal range.
__device__ __forceinline__ f16x8 bf16x8_to_f16x8(u32x4 raw) {
    f16x8 out;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float lo = __uint_as_float(raw[i] << 16), hi = __uint_as_float(raw[i] & 0xffff0000u);
        const f16x2 h = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(lo, hi));
        out[2 * i] = h[0];
        out[2 * i + 1] = h[1];
    }
    return out;
}
__device__ __forceinline__ f16x8 load_w(const bf16* p) { return *(const f16x8*)p; }     // packed weights are already fp16

// Split activations (see GemmArgs): v goes out as hi = fp16(v) and, lo_off elements further on, lo = fp16(v - hi).
__device__ __forceinline__ void store_split(f16* p, long long lo_off, float v) {
    v = split_value(v);
    const f16 hi = (f16)v;
    *p = hi;
    if (lo_off) p[lo_off] = (f16)(v - (float)hi);
}
__device__ __forceinline__ void store_split4(f16* p, long long lo_off, const float (&v)[4]) {
    f16x4 hi, lo;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float x = split_value(v[r]);
        hi[r] = (f16)x;
        lo[r] = (f16)(x - (float)hi[r]);
    }
    *(f16x4*)p = hi;
    if (lo_off) *(f16x4*)(p + lo_off) = lo;
}

// ------------------------------------------------------------------------------ weight layout
// bf16 weight matrices are not read as given.  ax_model_create repacks every [N, K] matrix once,
// widening each bf16 to fp16 on the way (the round-toward-zero pack above: exact in fp16's normal
// range; the kernels multiply on the fp16 MFMA), into panels of 16 rows; a panel is cut into chunks of 32 k, and a chunk (1 KB) is stored in
// the order the 16x16x32 MFMA takes it: 4 k-groups of 8, inside a group the 16 rows, each with
// its 8 consecutive k (16 bytes).  A wavefront's weight load for one MFMA step is then 1 KB of
// contiguous memory instead of 16 pieces of 64 bytes from 16 rows - measured 7-19 % faster
// streaming in the skinny kernels and ~1.4x in the tile kernels that feed MFMA operands straight
// from global memory.  Element (n, k) sits at
//     (n / 16) * 16 K  +  (k / 32) * 512  +  ((k % 32) / 8) * 128  +  (n % 16) * 8  +  k % 8.
// N % 16 == 0 and K % 32 == 0 (guaranteed by the model configuration checks).
__device__ __forceinline__ long long packed_row(int n, int K) { return (long long)(n >> 4) * 16 * K + (n & 15) * 8; }
constexpr int PK_KG = 128;        // elements between k-groups of 8 inside a chunk
constexpr int PK_CHUNK = 512;     // elements per chunk of 32 k  (so k advances by 32 -> +512: "k * 16")

// 1 / rms of A rows from the column-block partial sums of x^2 their producer left behind.
// A kernel of this size is a chain of memory round trips, so every helper here requests all
// the partials it will need before it adds anything up: the index is clamped instead of
// branched on (no load sits behind a branch), values past the end are dropped when summing.
//
// One row's partials spread over a group of G lanes (gl = lane within the group), 4 G per round.
template <int G>
__device__ __forceinline__ float ssq_lane_sum(const float* __restrict__ src, int nparts, int gl) {
    float v = 0.f;
    for (int base = 0; base < nparts; base += 4 * G) {
        float t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = src[min(base + u * G + gl, nparts - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) v += base + u * G + gl < nparts ? t[u] : 0.f;
    }
    return v;
}
// One row by one wavefront; every lane gets the result.
__device__ __forceinline__ float wave_inv_rms(const float* __restrict__ ssq, int row, int nparts,
                                              int d_norm, float eps, int lane) {
    float v = ssq_lane_sum<64>(ssq + (long long)row * nparts, nparts, lane);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return 1.0f / sqrtf(v / (float)d_norm + eps);
}

// Block-wide: 1 / rms of `rows` A-rows into s_inv[0..rows).  Half a wavefront (32 lanes) owns a
// row and a thread works on INV_BATCH rows at a time (a power of two up to 16): their
// 4 x INV_BATCH loads are in flight together, so the table costs one memory round trip per
// INV_BATCH rows of a thread (and per 128 partials of a row), not one per load.
// The INV_BATCH per-lane sums are then added across the 32 lanes with a transposing butterfly:
// at each stage a lane hands half of its values to its partner and keeps the other half, so the
// batch costs INV_BATCH - 1 + (5 - log2 INV_BATCH) cross-lane exchanges instead of 5 per row and
// ends with each row's total in its own lanes - one division and square root per thread, not one
// per row.  (Five exchanges and a square root per row, one row after the other, were ~4 us of a
// 128-row block's prologue.)  The caller synchronises before reading s_inv.
template <int INV_BATCH>
__device__ __forceinline__ void block_inv_rms(const GemmArgs& g, int first_row, int rows, float* s_inv) {
    static_assert(INV_BATCH == 1 || INV_BATCH == 2 || INV_BATCH == 4 || INV_BATCH == 8 || INV_BATCH == 16, "power of two up to 16");
    constexpr int LOG = INV_BATCH == 16 ? 4 : INV_BATCH == 8 ? 3 : INV_BATCH == 4 ? 2 : INV_BATCH == 2 ? 1 : 0;
    const int hw = threadIdx.x >> 5, hl = threadIdx.x & 31, nhw = blockDim.x >> 5;
    for (int base = 0; base < rows; base += INV_BATCH * nhw) {
        long long src[INV_BATCH];
        float v[INV_BATCH];
#pragma unroll
        for (int p = 0; p < INV_BATCH; ++p) {
            const int gm = min(first_row + min(base + p * nhw + hw, rows - 1), g.M - 1);
            src[p] = (long long)(g.a_rows ? g.a_rows[gm] : gm) * g.nparts;
            v[p] = 0.f;
        }
        for (int q0 = 0; q0 < g.nparts; q0 += 128) {
            float t[INV_BATCH][4];
#pragma unroll
            for (int p = 0; p < INV_BATCH; ++p)
#pragma unroll
                for (int u = 0; u < 4; ++u) t[p][u] = g.ssq[src[p] + min(q0 + u * 32 + hl, g.nparts - 1)];
#pragma unroll
            for (int p = 0; p < INV_BATCH; ++p)
#pragma unroll
                for (int u = 0; u < 4; ++u) v[p] += q0 + u * 32 + hl < g.nparts ? t[p][u] : 0.f;
        }
        // stage st: partner = lane ^ (16 >> st); the lane with that bit set keeps the upper half of
        // the remaining values, so after LOG stages it holds the row whose index (within the batch)
        // is the top LOG bits of its lane number
#pragma unroll
        for (int st = 0; st < LOG; ++st) {
            const int n = INV_BATCH >> st, o = 16 >> st;
            const bool upper = (hl & o) != 0;
#pragma unroll
            for (int j = 0; j < n / 2; ++j) {
                const float send = upper ? v[j] : v[j + n / 2];
                const float keep = upper ? v[j + n / 2] : v[j];
                v[j] = keep + __shfl_xor(send, o, 64);
            }
        }
#pragma unroll
        for (int o = 16 >> LOG; o > 0; o >>= 1) v[0] += __shfl_xor(v[0], o, 64);
        const int r = base + (hl >> (5 - LOG)) * nhw + hw;
        if ((hl & ((32 >> LOG) - 1)) == 0 && r < rows) s_inv[r] = 1.0f / sqrtf(v[0] / (float)g.d_norm + g.eps);
    }
}

// The same for rows that left at most 4 partial sums behind (their producer was a K-split GEMM's
// reduce kernel, or the embedding): four lanes per row, one load each, the rows of up to four
// passes in flight together - cheap enough in registers to sit behind the operand loads of a
// kernel's prologue, where its cold misses overlap theirs.
__device__ __forceinline__ void block_inv_rms_few(const GemmArgs& g, int first_row, int rows, float* s_inv) {
    const int p = threadIdx.x & 3, per_pass = blockDim.x >> 2;
    for (int base = 0; base < rows; base += 4 * per_pass) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int gm = min(first_row + min(base + u * per_pass + (int)(threadIdx.x >> 2), rows - 1), g.M - 1);
            v[u] = g.ssq[(long long)(g.a_rows ? g.a_rows[gm] : gm) * g.nparts + min(p, g.nparts - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float t = p < g.nparts ? v[u] : 0.f;
            t += __shfl_xor(t, 1, 64);
            t += __shfl_xor(t, 2, 64);
            const int r = base + u * per_pass + (int)(threadIdx.x >> 2);
            if (p == 0 && r < rows) s_inv[r] = 1.0f / sqrtf(t / (float)g.d_norm + g.eps);
        }
    }
}

// The same with activations in panels, partial sums as [parts][rows]: a thread adds up a row (or, with twice as many threads as rows, half of one),
// 16 loads in flight.  `rows` is the number of threads or half of it.
__device__ __forceinline__ void block_inv_rms_panels(const GemmArgs& g, int first_row, int rows, float* s_inv) {
    const int r = threadIdx.x & (rows - 1), gm = min(first_row + r, g.M - 1), groups = blockDim.x / rows;
    float v = 0.f;
    for (int p0 = threadIdx.x / rows; p0 < g.nparts; p0 += 16 * groups) {
        float t[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) t[u] = g.ssq[(long long)min(p0 + u * groups, g.nparts - 1) * g.M + gm];
#pragma unroll
        for (int u = 0; u < 16; ++u) v += p0 + u * groups < g.nparts ? t[u] : 0.f;
    }
    if (groups > 1) {
        if (threadIdx.x >= rows) s_inv[r] = v;
        __syncthreads();
        if (threadIdx.x < rows) v += s_inv[r];
    }
    if (threadIdx.x < rows) s_inv[r] = 1.0f / sqrtf(v / (float)g.d_norm + g.eps);
}

// ------------------------------------------------------------------------------ host interface between the GEMM files
// Many-row GEMMs (k_gemm_block.hip): which tile shape and how many K slices, and the time the plan expects.
struct BlockPlan { int shape, ks; float us; };
BlockPlan plan_gemm_block(Epilogue epi, int M, int N, int K, bool split, bool panels, size_t ws_bytes);      // panels: A (and C16) in panels
float gemm_reduce_us(Epilogue epi, int M, int N, int ks, bool panels);      // time of the kernel that adds up ks slabs (EPI_QKV, EPI_RESIDUAL)
// What a whole residual GEMM costs the GEMM behind it: N / 64 or N / 32 partial sums of x^2 a row to read in every block's prologue, where
// slabs added up leave a few (~3B at 1200 rows: O whole 40.9 us + gate / up 149.7, O in slices 39.1 + 143.6).
float gemm_partials_us(int M, bool panels);
// a_rows must be NULL and N % 64 == 0; returns the partial sums per row it leaves, as launch_gemm_bf16.
int launch_gemm_block(Epilogue epi, const GemmArgs& g, const BlockPlan& p, hipStream_t s);
// Second halves of K-sliced GEMMs (k_gemm_bf16.hip): add the g.ksplit slabs of g.split_ws and run the epilogue.
int launch_residual_reduce(const GemmArgs& g, hipStream_t s);
void launch_qkv_reduce(const GemmArgs& g, hipStream_t s);

}  // namespace ax
