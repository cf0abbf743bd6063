// GEMMs of bf16-weight models on the gfx950 matrix cores: C = A[M,K] * W[N,K]^T, fp32
// accumulation.  The caller's weights are bf16; the kernels read the library's own 16-bit copy,
// made once at model creation: each bf16 widened to fp16 (exact for every |w| >= 2^-14, absolute
// error below 2^-25 beneath that) and laid out in MFMA operand order (see "weight layout" below).
// Activations are fp16 and the product runs on the fp16 MFMA, which has the same rate as the
// bf16 one.  Reason: bf16 activations (8 significant bits) put the logits of a 16-layer decoder
// ~0.05 away from the exact result; fp16 activations (11 bits) keep them within 0.01.
//
//   * skinny kernel (up to 16 rows, narrow logits to 32: decoding, verify steps, pure weight streaming): one block owns 16 output columns, its
//     wavefronts split K, W goes HBM -> registers -> v_mfma_f32_16x16x32_f16 with no LDS in the streaming loop; the per-wavefront partial
//     sums meet in LDS.
//   * register kernel (17-256 rows; k_gemm_regs.h): the same idea with tiles of up to 128 x 128 outputs.
//   * tile kernel   (some QKV and residual GEMMs of 257-512 rows, narrow logits): 8 wavefronts, LDS-staged 64 x 128 x 64 tiles,
//     v_mfma_f32_32x32x16_f16, global loads several K slices ahead.
//   * stream kernel (logits from 17 rows, some SwiGLU GEMMs of 257-640): activations through LDS, weights straight into MFMA operands.
//   * block kernel  (more than 256 rows; k_gemm_block.hip; which of the three, plan_many below).
//
// RMSNorm is folded into the GEMMs around it.  The GEMM that produces the residual stream x
// also writes a = fp16(x * gain_next) and, per row and per block of columns, a partial sum of
// x^2.  The GEMM that consumes a multiplies its accumulators by 1 / sqrt(mean(x^2) + eps) in
// the epilogue: (x * g / rms) W^T = (1 / rms) * ((x * g) W^T).  No separate norm kernel runs.
//
// Epilogues: fp32 store (optionally rms-scaled), residual add (+ norm preparation), SwiGLU
// (two weight matrices share the A operand), and QKV (rms scale, rotary embedding, q to the
// activation buffer, k and v straight into the KV pages).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "gemm_device.h"
#include "k_gemm_regs.h"

namespace ax {

// out-of-place repack: one thread per 16-byte unit of the destination (coalesced writes)
// A bf16 weight beyond fp16's range (|w| > 65504, infinities, NaNs) does not survive: `bad` reports it.
__global__ void pack_weights_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int N, int K, int* __restrict__ bad) {
    const long long units = (long long)N * K / 8, stride = (long long)gridDim.x * blockDim.x;
    const int upp = 2 * K;                                   // 16-byte units per panel
    bool lost = false;
    for (long long u = (long long)blockIdx.x * blockDim.x + threadIdx.x; u < units; u += stride) {
        const int panel = (int)(u / upp), w = (int)(u % upp);
        const int c = w >> 6, kg = (w >> 4) & 3, r = w & 15;
        const u32x4 raw = src[((long long)(panel * 16 + r) * K + c * 32 + kg * 8) / 8];
#pragma unroll
        for (int i = 0; i < 4; ++i)       // checked on the exact values: the narrowing itself rounds toward zero and would saturate
            lost |= !(__builtin_fabsf(__uint_as_float(raw[i] << 16)) <= 65504.0f) ||
                    !(__builtin_fabsf(__uint_as_float(raw[i] & 0xffff0000u)) <= 65504.0f);
        dst[u] = __builtin_bit_cast(u32x4, bf16x8_to_f16x8(raw));
    }
    if (bad && lost) *bad = 1;                               // every writer stores the same value
}

void launch_pack_weights(const void* src, void* dst, int N, int K, hipStream_t s, int* bad) {
    pack_weights_kernel<<<2048, 256, 0, s>>>((const u32x4*)src, (u32x4*)dst, N, K, bad);
}

// ------------------------------------------------------------------------------ tile kernel
// MFMA 32x32x16 operand layout (wave64): lane l supplies row/col (l % 32) and the 8 k values
// 8*(l/32) .. +7; result register r of lane l is C[(r/4)*8 + (l/32)*4 + r%4][l % 32].
// Block = WM x WN wavefronts, wavefront tile = (TM*32) x (TN*32).  (The QKV projection runs
// as a plain store GEMM followed by qkv_reduce_rope_kernel.)
// SPLIT: the A operand comes as hi and lo parts (split activations): both are staged and multiplied against the
// same B fragments.
template <int EPI, int TM, int TN, int WM = 2, int WN = 2, bool SPLIT = false>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_tile_kernel(GemmArgs g) {
    constexpr int NT = 64 * WM * WN;                                         // threads per block
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 64, LS = BK + 8;  // LS: padded row
    constexpr int A_CH = BM * 8 / NT, B_CH = BN * 8 / NT;                  // 16-byte chunks per thread
    constexpr int D = 4;                                                     // prefetch distance (even)
    constexpr int NA = SPLIT ? 2 : 1;
    __shared__ __attribute__((aligned(16))) f16 sA[2][NA][BM * LS];
    __shared__ __attribute__((aligned(16))) f16 sB[2][BN * LS];
    __shared__ float s_inv[BM];

    const f16* __restrict__ A = (const f16*)g.A;
    const bf16* __restrict__ W = (const bf16*)g.W;
    const int M = g.M, N = g.N, K = g.K;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WN, wn = wave % WN;
    const int lrow = lane & 31, lg = lane >> 5;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int kspan = g.ksplit > 1 ? K / g.ksplit : K, kbase = blockIdx.z * kspan;   // this block's K slice

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Software pipeline: global loads run D k-steps ahead in a register ring (slot = step % D),
    // LDS is double buffered, one barrier per k-step.  At step s: issue the loads of s + D,
    // multiply out of LDS buffer s % 2, move the registers of s + 1 into the other buffer.
    f16x8 ra[D][NA][A_CH];
    u32x4 rb[D][B_CH];          // weights as packed (fp16, MFMA operand order)
    long long a_off[A_CH], b_off[B_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        const int c = tid + NT * i, row = c >> 3, cc = c & 7;
        const int gm = min(m0 + row, M - 1);
        a_off[i] = (long long)(g.a_rows ? g.a_rows[gm] : gm) * K + kbase + cc * 8;
    }
    // weights (packed layout): a 64-wide k-step of one 16-row panel is 2 KB of contiguous memory,
    // 128 units of 16 bytes: unit = chunk (k / 32) * 64 + k-group * 16 + row
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
        const int c = tid + NT * i, panel = min((n0 >> 4) + (c >> 7), (N >> 4) - 1);
        b_off[i] = (long long)panel * 16 * K + (long long)kbase * 16 + (c & 127) * 8;
    }
    auto load_global = [&](int slot, int k0) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            ra[slot][0][i] = *(const f16x8*)(A + a_off[i] + k0);
            if (SPLIT) ra[slot][NA - 1][i] = *(const f16x8*)(A + a_off[i] + k0 + g.a_lo_off);
        }
#pragma unroll
        for (int i = 0; i < B_CH; ++i) rb[slot][i] = __builtin_nontemporal_load((const u32x4*)(W + b_off[i] + (long long)k0 * 16));
    };
    auto store_lds = [&](int slot, int buf) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            const int c = tid + NT * i, row = c >> 3, cc = c & 7;
#pragma unroll
            for (int p = 0; p < NA; ++p) *(f16x8*)(sA[buf][p] + row * LS + cc * 8) = ra[slot][p][i];
        }
#pragma unroll
        for (int i = 0; i < B_CH; ++i) {
            const int c = tid + NT * i, u = c & 127;
            const int row = (c >> 7) * 16 + (u & 15), col = (u >> 6) * 32 + ((u >> 4) & 3) * 8;
            *(f16x8*)(sB[buf] + row * LS + col) = __builtin_bit_cast(f16x8, rb[slot][i]);
        }
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            f16x8 fa[NA][TM], fb[TN];
#pragma unroll
            for (int p = 0; p < NA; ++p)
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    fa[p][i] = *(const f16x8*)(sA[buf][p] + ((wm * TM + i) * 32 + lrow) * LS + kk * 16 + lg * 8);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[j] = *(const f16x8*)(sB[buf] + ((wn * TN + j) * 32 + lrow) * LS + kk * 16 + lg * 8);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int p = 0; p < NA; ++p)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[p][i], fb[j], acc[i][j], 0, 0, 0);
        }
    };

    const int nsteps = kspan / BK;
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (s < nsteps) load_global(s, s * BK);
    // deferred RMSNorm: 1/rms of this block's rows, 64 rows per batch (more loads in flight would cost the 64-row
    // blocks the registers for their second block per CU)
    if (g.ssq) {
        if (g.nparts <= 4) block_inv_rms_few(g, m0, BM, s_inv);
        else block_inv_rms<BM >= 128 ? 4 : 2>(g, m0, BM, s_inv);
    }
    store_lds(0, 0);
    __syncthreads();
    // steady state: groups of D steps with every load and store unconditional (branch-free, so
    // the loads of the next D steps stay in flight across the barriers)
    int step0 = 0;
    for (; step0 + 2 * D <= nsteps; step0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {                    // D is even: buffer = u % 2, slot = u
            load_global(u, (step0 + u + D) * BK);
            multiply(u & 1);
            store_lds((u + 1) % D, (u + 1) & 1);
            __syncthreads();
        }
    }
    // drain: at most 2 D - 1 steps, loads only while there is something left to load
    for (; step0 < nsteps; step0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int step = step0 + u;
            if (step < nsteps) {
                if (step + D < nsteps) load_global(u, (step + D) * BK);
                multiply(u & 1);
                if (step + 1 < nsteps) store_lds((u + 1) % D, (u + 1) & 1);
                __syncthreads();
            }
        }
    }

    // Epilogues.  Each one first requests everything it needs from memory for all of the
    // thread's 16 * TM * TN outputs and only then computes and stores: stores and loads through
    // the same pointers would otherwise be kept in program order, one round trip per element.
    auto row_of = [&](int i, int r) { return (wm * TM + i) * 32 + (r >> 2) * 8 + lg * 4 + (r & 3); };
    auto col_of = [&](int j) { return n0 + (wn * TN + j) * 32 + lrow; };
    float inv[TM][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) inv[i][r] = g.ssq ? s_inv[row_of(i, r)] : 1.0f;

    if constexpr (EPI == EPI_STORE_F32) {
        float* __restrict__ C = g.Cf + (g.ksplit > 1 ? (long long)blockIdx.z * M * N : 0);   // K slice: its own slab
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int m = m0 + row_of(i, r), n = col_of(j);
                    if (m < M && n < N) C[(long long)m * N + n] = acc[i][j][r] * inv[i][r];
                }
    } else if constexpr (EPI == EPI_RESIDUAL) {
        if (g.ksplit > 1) {          // K slice: raw partial products, finished by residual_reduce_kernel
            float* part = g.split_ws + (long long)blockIdx.z * M * N;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int m = m0 + row_of(i, r), n = col_of(j);
                        if (m < M && n < N) part[(long long)m * N + n] = acc[i][j][r];
                    }
            return;
        }
        float gain[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) gain[j] = g.gain_next ? (float)((const bf16*)g.gain_next)[min(col_of(j), N - 1)] : 0.f;
        float xv[TM][TN][16];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = min(m0 + row_of(i, r), M - 1), n = min(col_of(j), N - 1);
                    xv[i][j][r] = g.Cf[(long long)m * N + n];
                }
        f16* __restrict__ a16 = (f16*)g.C16;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + row_of(i, r);
                float ss = 0.f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int n = col_of(j);
                    if (m < M && n < N) {
                        const long long o = (long long)m * N + n;
                        const float xn = xv[i][j][r] + acc[i][j][r];
                        g.Cf[o] = xn;
                        if (g.gain_next) {
                            store_split(a16 + o, g.c_lo_off, xn * gain[j]);
                            ss += xn * xn;
                        }
                    }
                }
                if (g.gain_next) {   // partial sum of squares over this wavefront's TN*32 columns
#pragma unroll
                    for (int o = 16; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
                    const int part = n0 / (TN * 32) + wn;                 // this wavefront's block of columns
                    if (lrow == 0 && m < M && part < N / (TN * 32)) g.ssq_out[(long long)m * (N / (TN * 32)) + part] = ss;
                }
            }
    }
}

// Second half of a K-split residual GEMM: x += sum of the K-slice partials (in slice order),
// a = fp16(x * gain_next), and the sum of x^2 over the block's columns.  Block = 1024 columns of
// one row (four per thread, every operand requested before anything is added), so a row leaves
// only ceil(N / 1024) partial sums behind - the GEMM that consumes the pending norm reads 2-4
// values per row instead of N / 32.  grid (ceil(N / 1024), M); N % 4 == 0.
constexpr int REDUCE_COLS = 1024;
__global__ __launch_bounds__(256) void residual_reduce_kernel(GemmArgs g) {
    __shared__ float s_ss[4];
    const int m = blockIdx.y, n = (blockIdx.x * 256 + threadIdx.x) * 4;
    const bool live = n < g.N;
    const int nc = min(n, g.N - 4);
    const long long o = (long long)m * g.N + nc, slab = (long long)g.M * g.N;
    f32x4 part[SPLITK_MAX];
#pragma unroll
    for (int ks = 0; ks < SPLITK_MAX; ++ks)
        part[ks] = ks < g.ksplit ? *(const f32x4*)(g.split_ws + ks * slab + o) : (f32x4){0.f, 0.f, 0.f, 0.f};
    f32x4 xn = *(const f32x4*)(g.Cf + o);
    float gain[4] = {0.f, 0.f, 0.f, 0.f};
    if (g.gain_next) {
#pragma unroll
        for (int r = 0; r < 4; ++r) gain[r] = (float)((const bf16*)g.gain_next)[nc + r];
    }
#pragma unroll
    for (int ks = 0; ks < SPLITK_MAX; ++ks) xn += part[ks];
    if (live) *(f32x4*)(g.Cf + o) = xn;
    if (g.gain_next) {
        float ss = 0.f;
        if (live) {
            float h[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                h[r] = xn[r] * gain[r];
                ss += xn[r] * xn[r];
            }
            store_split4((f16*)g.C16 + o, g.c_lo_off, h);
        }
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) ss += __shfl_xor(ss, w, 64);
        if ((threadIdx.x & 63) == 0) s_ss[threadIdx.x >> 6] = ss;
        __syncthreads();
        if (threadIdx.x == 0) g.ssq_out[(long long)m * gridDim.x + blockIdx.x] = (s_ss[0] + s_ss[1]) + (s_ss[2] + s_ss[3]);
    }
}
// The same with a in panels.  A block is a panel of 16 rows x COLS columns, 16 lanes to a row: a wavefront reads 256 bytes of four rows at a
// time, all loads of a slab in flight together, and writes 64-byte pieces of the panel's runs.  Leaves ceil(N / COLS) sums a row.
template <int COLS>
__global__ __launch_bounds__(256) void residual_reduce_panels_kernel(GemmArgs g) {
    constexpr int IT = COLS / 64;
    const int m = blockIdx.y * 16 + (threadIdx.x >> 4), mc = min(m, g.M - 1);
    const long long slab = (long long)g.M * g.N;
    f32x4 xn[IT];
    int n[IT];
    long long o[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        n[it] = blockIdx.x * COLS + it * 64 + (threadIdx.x & 15) * 4;
        o[it] = (long long)mc * g.N + min(n[it], g.N - 4);
        xn[it] = *(const f32x4*)(g.Cf + o[it]);
    }
    for (int ks = 0; ks < g.ksplit; ++ks) {
        f32x4 part[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) part[it] = *(const f32x4*)(g.split_ws + ks * slab + o[it]);
#pragma unroll
        for (int it = 0; it < IT; ++it) xn[it] += part[it];
    }
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        if (n[it] >= g.N) continue;
        float h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h[r] = xn[it][r] * (float)((const bf16*)g.gain_next)[n[it] + r];
            ss += xn[it][r] * xn[it][r];
        }
        if (m < g.M) {
            *(f32x4*)(g.Cf + o[it]) = xn[it];
            store_split4((f16*)g.C16 + act_index(g.c_layout, m, n[it], g.M, g.N), g.c_lo_off, h);
        }
    }
#pragma unroll
    for (int w = 8; w > 0; w >>= 1) ss += __shfl_xor(ss, w, 64);
    if ((threadIdx.x & 15) == 0 && m < g.M) g.ssq_out[ssq_index(ssq_by_part(g.c_layout, g.M), m, blockIdx.x, g.M, gridDim.x)] = ss;
}
// launches it; returns the partial sums per row it leaves
int launch_residual_reduce(const GemmArgs& g, hipStream_t s) {
    if (g.c_layout != ACT_ROWS) {
        const unsigned panels = (unsigned)(g.M + 15) / 16;
        const int cols = (long long)panels * g.N >= 512 * 512 ? 512 : 256, parts = (g.N + cols - 1) / cols;
        if (cols == 512) residual_reduce_panels_kernel<512><<<dim3((unsigned)parts, panels), 256, 0, s>>>(g);
        else residual_reduce_panels_kernel<256><<<dim3((unsigned)parts, panels), 256, 0, s>>>(g);
        return parts;
    }
    const int parts = (g.N + REDUCE_COLS - 1) / REDUCE_COLS;
    residual_reduce_kernel<<<dim3((unsigned)parts, (unsigned)g.M), 256, 0, s>>>(g);
    return parts;
}

// Second half of a K-split QKV GEMM: sums the K-slice partials, applies 1 / rms of the row,
// rotates q and k heads by the row's position and writes q to the activation buffer, k and v
// into the row's KV slot.  A thread owns four channel pairs of one head of one row, a block 1024 / (head_dim / 2) rows of
// the head: for q and k neighbours are channels (whole runs of 128 or 256 bytes in, 64 or 128 out), for v rows, whose tokens lie side by
// side in a page.  grid (blocks of rows, heads).
template <int HD>
__global__ __launch_bounds__(256) void qkv_reduce_rope_kernel(GemmArgs g) {
    constexpr int half = HD / 2, QUADS = half / 4, ROWS = 256 / QUADS, TPR = 256 / ROWS;      // TPR threads add up a row's sum of squares
    __shared__ float s_inv[ROWS];
    const RopeArgs& ro = g.rope;
    const int N = g.N, M = g.M, Hq = ro.n_q_heads, Hkv = ro.kv.n_kv_heads, head = blockIdx.y;
    const bool is_v = head >= Hq + Hkv;
    const int row = is_v ? threadIdx.x % ROWS : threadIdx.x / QUADS, j = (is_v ? threadIdx.x / ROWS : threadIdx.x % QUADS) * 4;
    const int m = blockIdx.x * ROWS + row, mc = min(m, M - 1);
    const int pos = ro.row_pos[mc], slot = ro.row_slot[mc];
    const long long slab = (long long)M * N;
    const float* p = g.split_ws + (long long)mc * N + head * HD + j;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll 4
    for (int ks = 0; ks < g.ksplit; ++ks) {
        a += *(const f32x4*)(p + ks * slab);
        b += *(const f32x4*)(p + ks * slab + half);
    }
    f32x4 c = a, sn = a;
    if (!is_v) {
        c = *(const f32x4*)(ro.cos + (long long)pos * half + j);
        sn = *(const f32x4*)(ro.sin + (long long)pos * half + j);
    }
    if (g.ssq) {
        const int r = threadIdx.x / TPR, rm = min((int)blockIdx.x * ROWS + r, M - 1);
        float v = 0.f;
        for (int q = threadIdx.x % TPR; q < g.nparts; q += TPR) v += g.ssq[ssq_index(ssq_by_part(g.a_layout, M), rm, q, M, g.nparts)];
#pragma unroll
        for (int o = TPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (threadIdx.x % TPR == 0) s_inv[r] = 1.0f / sqrtf(v / (float)g.d_norm + g.eps);
    } else if (threadIdx.x < ROWS) {
        s_inv[threadIdx.x] = 1.0f;
    }
    __syncthreads();
    if (m >= M) return;
    const float inv = s_inv[row];
    f16* pool = (f16*)ro.kv.base;
    a *= inv;
    b *= inv;
    if (!is_v) {
        f16* dst = head < Hq ? (f16*)ro.q_out + ((long long)m * Hq + head) * HD
                             : pool + ro.kv.plane(ro.layer, 0, head - Hq) + (long long)slot * HD;
        const long long lo_off = head < Hq ? g.c_lo_off : 0;      // q may be split; the cache holds one fp16 per entry
        float va[4], vb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            va[r] = a[r] * c[r] - b[r] * sn[r];
            vb[r] = b[r] * c[r] + a[r] * sn[r];
        }
        store_split4(dst + j, lo_off, va);
        store_split4(dst + j + half, lo_off, vb);
    } else {
        f16* dst = pool + ro.kv.plane(ro.layer, 1, head - Hq - Hkv) + (long long)(slot >> 4) * 16 * HD + (slot & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dst[(long long)(j + r) * 16] = (f16)a[r];
            dst[(long long)(j + r + half) * 16] = (f16)b[r];
        }
    }
}

void launch_qkv_reduce(const GemmArgs& g, hipStream_t s) {
    const unsigned heads = (unsigned)(g.rope.n_q_heads + 2 * g.rope.kv.n_kv_heads);
    if (g.rope.kv.head_dim == 64) qkv_reduce_rope_kernel<64><<<dim3((unsigned)(g.M + 31) / 32, heads), 256, 0, s>>>(g);
    else qkv_reduce_rope_kernel<128><<<dim3((unsigned)(g.M + 15) / 16, heads), 256, 0, s>>>(g);
}

// ------------------------------------------------------------------------------ stream kernel
// The LDS-staged kernel above moves both operands through LDS and spends more cycles there than on the matrix cores (a 32 x 64
// wavefront tile reads 1.5 KB of LDS per MFMA).  Here only the activation tile goes through LDS; every wavefront
// streams its own weight rows HBM/L2 -> registers -> MFMA, as the skinny kernel does.  Block = 4
// wavefronts side by side along N, all working on the same BM = TM*32 rows; a wavefront owns 32
// output columns, i.e. one 32-row tile each of W (gate) and W2 (up).  The weight loads run D
// k-steps ahead in a register ring, the activation tile is double buffered in LDS, one barrier
// per k-step of 64.  With thousands of rows the block kernel is faster (~1B gate / up at 4096 rows: 382 -> 262 us).
//
// Blocks are renumbered so that the gy row tiles that share a weight tile have consecutive ids
// on one XCD (workgroups are dealt to the 8 XCDs round robin), i.e. share that XCD's L2.
//
// EPI_STORE_F32 (logits): a wavefront's two weight streams are two 32-row tiles of the ONE matrix, 32 columns apart, and a block covers 256
// output columns.
//
// SPLIT: split activations - the hi and lo parts of the A tile are both staged in LDS and multiplied against the
// same weight registers.
template <int EPI, int TM, int D, bool SPLIT = false>
__global__ __launch_bounds__(256) void gemm_bf16_stream_kernel(GemmArgs g, int gx, int gy) {
    static_assert(EPI == EPI_SWIGLU || EPI == EPI_STORE_F32, "two epilogues");
    constexpr int BM = TM * 32, BN = EPI == EPI_SWIGLU ? 128 : 256, BK = 64, LS = BK + 8, NS = 2;
    constexpr int A_CH = BM * 8 / 256;                       // 16-byte chunks of the A tile per thread
    constexpr int NA = SPLIT ? 2 : 1;
    __shared__ __attribute__((aligned(16))) f16 sA[2][NA][BM * LS];
    __shared__ float s_inv[BM];

    const f16* __restrict__ A = (const f16*)g.A;
    const int M = g.M, N = g.N, K = g.K;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int lrow = lane & 31, lg = lane >> 5;
    const int nblk = gx * gy;
    int bid = blockIdx.x;
    if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);
    const int bx = bid / gy, by = bid - bx * gy;
    const int m0 = by * BM, n0 = bx * BN;

    // this lane's output columns = weight rows of its two streams: row n of W and of W2 (SwiGLU),
    // or rows n and n + 32 of W
    int ncol[NS];
    const bf16* wp[NS];
    // packed layout: MFMA step c of a k-step covers k = 16 c + 8 lg .. + 7, i.e. chunk c / 2, k-group 2 (c % 2) + lg
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        ncol[t] = n0 + wave * (BN / 4) + lrow + (EPI == EPI_SWIGLU ? 0 : 32 * t);
        wp[t] = (const bf16*)(EPI == EPI_SWIGLU && t == 1 ? g.W2 : g.W) + packed_row(min(ncol[t], N - 1), K) + lg * PK_KG;
    }
    long long a_off[A_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        const int c = tid + 256 * i, row = c >> 3, cc = c & 7;
        const int gm = min(m0 + row, M - 1);
        a_off[i] = (long long)(g.a_rows ? g.a_rows[gm] : gm) * K + cc * 8;
    }

    f32x16 acc[NS][TM];
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][i][r] = 0.f;

    u32x4 rw[D][NS][4];             // weights: 4 chunks of 8 k per stream and k-step
    f16x8 ra[D][NA][A_CH];
    auto load_global = [&](int slot, int k0) {
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) rw[slot][t][c] = __builtin_nontemporal_load((const u32x4*)(wp[t] + (long long)k0 * 16 + (c >> 1) * PK_CHUNK + (c & 1) * 2 * PK_KG));
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            ra[slot][0][i] = *(const f16x8*)(A + a_off[i] + k0);
            if (SPLIT) ra[slot][NA - 1][i] = *(const f16x8*)(A + a_off[i] + k0 + g.a_lo_off);
        }
    };
    auto store_lds = [&](int slot, int buf) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            const int c = tid + 256 * i, row = c >> 3, cc = c & 7;
#pragma unroll
            for (int p = 0; p < NA; ++p) *(f16x8*)(sA[buf][p] + row * LS + cc * 8) = ra[slot][p][i];
        }
    };
    auto multiply = [&](int slot, int buf) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f16x8 fa[NA][TM], fw[NS];
#pragma unroll
            for (int p = 0; p < NA; ++p)
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[p][i] = *(const f16x8*)(sA[buf][p] + (i * 32 + lrow) * LS + c * 16 + lg * 8);
#pragma unroll
            for (int t = 0; t < NS; ++t) fw[t] = __builtin_bit_cast(f16x8, rw[slot][t][c]);
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int p = 0; p < NA; ++p)
                        acc[t][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[p][i], fw[t], acc[t][i], 0, 0, 0);
        }
    };

    const int nsteps = K / BK;
    // deferred RMSNorm: 1/rms of this block's rows, before the operand rings take the registers (16
    // rows x 4 loads per thread in flight: one or two round trips; behind the ring loads the same
    // table cost four to six, 10-15 % of the launch at 512-1024 rows).
    // Few partials per row (K-split producer): behind the ring loads, their cold misses overlap.
    const bool inv_here = g.ssq != nullptr;
    if (inv_here && g.nparts > 4) block_inv_rms<16>(g, m0, BM, s_inv);
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (s < nsteps) load_global(s, s * BK);
    if (inv_here && g.nparts <= 4) block_inv_rms_few(g, m0, BM, s_inv);
    store_lds(0, 0);
    __syncthreads();
    // steady state, branch free: multiply step s out of ring slot s % D and LDS buffer s % 2,
    // refill the slot with step s + D, move the activations of step s + 1 into the other buffer
    int step0 = 0;
    for (; step0 + 2 * D <= nsteps; step0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int buf = (step0 + u) & 1;
            multiply(u, buf);
            store_lds((u + 1) % D, buf ^ 1);
            load_global(u, (step0 + u + D) * BK);
            __syncthreads();
        }
    }
    for (; step0 < nsteps; step0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int step = step0 + u;
            if (step < nsteps) {
                const int buf = step & 1;
                multiply(u, buf);
                if (step + 1 < nsteps) store_lds((u + 1) % D, buf ^ 1);
                if (step + D < nsteps) load_global(u, (step + D) * BK);
                __syncthreads();
            }
        }
    }

    auto row_of = [&](int i, int r) { return i * 32 + (r >> 2) * 8 + lg * 4 + (r & 3); };
    if constexpr (EPI == EPI_SWIGLU) {
        f16* __restrict__ out = (f16*)g.C16;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = row_of(i, r), m = m0 + row;
                const float inv = g.ssq ? s_inv[row] : 1.0f;
                if (m < M && ncol[0] < N)
                    store_split(out + (long long)m * N + ncol[0], g.c_lo_off, silu_f(acc[0][i][r] * inv) * (acc[1][i][r] * inv));
            }
    } else {
        float* __restrict__ C = g.Cf;
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = row_of(i, r), m = m0 + row;
                    const float inv = g.ssq ? s_inv[row] : 1.0f;
                    if (m < M && ncol[t] < N) C[(long long)m * N + ncol[t]] = acc[t][i][r] * inv;
                }
    }
}

// ------------------------------------------------------------------------------ skinny kernel
// MFMA 16x16x32 operand layout: lane l supplies row/col (l % 16) and the 8 k values
// 8*(l/16) .. +7; result register r of lane l is D[4*(l/16) + r][l % 16].  Here D = W_tile * x^T:
// D rows are output columns n, D columns are activation rows m, so a lane ends up with four
// consecutive n of one row m (one 16-byte store).
//
// COLS < 16 (residual GEMMs): a block owns fewer columns so that every CU gets a block; the
// unused MFMA rows are zero and their lanes issue no loads.
//
// For EPI_QKV the 16 columns of a block are 8 + 8 rotary partners of one head: local columns
// 0..7 are channels j0..j0+7, local columns 8..15 are channels hd/2 + j0 .. +7, so the partner
// of a lane's value lives in lane ^ 32.
//
// SPLIT: split activations - each weight fragment meets the hi and the lo part of the activation rows (two MFMAs);
// weight traffic is unchanged, the activation slice a wavefront reads doubles.
template <int EPI, int MT, int NW, int COLS = 16, bool SPLIT = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(1, NW >= 8 ? 4 : 8)))
void gemm_bf16_skinny_kernel(GemmArgs g) {
    static_assert(MT <= 2, "up to 32 rows");
    constexpr int NB = EPI == EPI_SWIGLU ? 2 : 1;
    constexpr int NA = SPLIT ? 2 : 1;
    __shared__ __attribute__((aligned(16))) f32x4 red[NW][NB][MT][64];
    __shared__ float s_inv[MT * 16];

    // The kernel is a chain of memory round trips, and the scalar loads of its arguments are the first: everything the loads below need is
    // asked for here, in one trip (left alone, the compiler fetches arguments where they are used, five trips one after the other).
    const f16* __restrict__ X = (const f16*)g.A;
    const bf16* __restrict__ W = (const bf16*)g.W;
    const bf16* __restrict__ W2 = (const bf16*)g.W2;
    const int M = g.M, N = g.N, K = g.K;
#define AX_ARGS "s"(X), "s"(W), "s"(M), "s"(N), "s"(K), "s"(g.a_lo_off), "s"((int)g.a_layout), "s"(g.a_total_rows), "s"(g.ssq), "s"(g.nparts)
    if constexpr (EPI == EPI_QKV) asm volatile("" :: AX_ARGS, "s"(g.rope.kv.head_dim), "s"(g.rope.row_pos), "s"(g.rope.row_slot), "s"(g.rope.cos), "s"(g.rope.sin));
    else if constexpr (EPI == EPI_RESIDUAL) asm volatile("" :: AX_ARGS, "s"(g.Cf), "s"(g.gain_next));
    else if constexpr (EPI == EPI_SWIGLU) asm volatile("" :: AX_ARGS, "s"(W2));
    else asm volatile("" :: AX_ARGS, "s"(g.a_rows));
#undef AX_ARGS
    const int* const a_rows = EPI == EPI_STORE_F32 ? g.a_rows : nullptr;      // only logits pick their rows
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const int n0 = blockIdx.x * COLS;
    const int kslice = K / NW, kbeg = wave * kslice, kend = kbeg + kslice;

    int wrow;                            // weight row this lane streams
    int q_head = 0, q_j0 = 0;            // EPI_QKV: head and first channel of the block
    if (EPI == EPI_QKV) {
        const int hd = g.rope.kv.head_dim, blocks = hd == 64 ? 2 : 3;        // log2 of the blocks of a head
        q_head = blockIdx.x >> blocks;
        q_j0 = (blockIdx.x & ((1 << blocks) - 1)) * 8;
        wrow = q_head * hd + (lr < 8 ? q_j0 + lr : hd / 2 + q_j0 + lr - 8);
    } else {
        wrow = min(n0 + min(lr, COLS - 1), N - 1);
    }
    const bool wlane = lr < COLS;      // COLS < 16: the other MFMA rows are zero, their lanes request nothing
    // Loads are a wavefront's own address (scalar registers, advanced by the scalar unit) and a lane's 32-bit offset to it: none of a load's
    // address takes vector instructions, or more than one register.  Weights: from the block's first panel.
    const long long first_panel = packed_row((EPI == EPI_QKV ? q_head * g.rope.kv.head_dim + q_j0 : n0) & ~15, K);
    const char* wb = (const char*)(W + first_panel);
    const char* wb2 = NB == 2 ? (const char*)(W2 + first_panel) : nullptr;
    const unsigned wo = (unsigned)(packed_row(wrow, K) - first_panel + lg * PK_KG) * 2u;      // packed layout: k advances by 32 -> + 1 KB
    // 8-column blocks: a load instruction costs the memory pipeline the same with half of its lanes
    // idle (the 8 MFMA rows that are not there), and these launches are bound by exactly that - a CU
    // pulled 16 GB/s of weights against 26 GB/s from 16-column blocks.  So the upper half of each
    // 16-lane row fetches the block's 8 rows at the NEXT k-step (one chunk further), and for that
    // step the operand is shifted down 8 lanes; MFMA rows 8-15 then hold products nobody reads.
    constexpr bool DUAL = COLS == 8 && NB == 1;
    const unsigned wod = (unsigned)(packed_row(min(n0 + (lr & 7), N - 1), K) - first_panel + lg * PK_KG + (lr >> 3) * PK_CHUNK) * 2u;
    auto weights = [&](const char* base, unsigned off, int k) { return (const u32x4*)(base + (long long)k * 32 + off); };
    // A in panels (act_index), up to 16 rows only: the row tile is the panel.  32 k of 9 rows are 576 bytes in a row, 4 or 5 lines instead of 9 halves.
    unsigned xo[MT];
    int xs[MT];                                                     // bytes per k
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int m = min(t * 16 + lr, M - 1);
        const int row = a_rows ? a_rows[m] : m;
        const int first = t * 16, panel_rows = min(16, g.a_total_rows - first);
        const bool panel = MT == 1 && g.a_layout;
        xs[t] = panel ? panel_rows * 2 : 2;
        xo[t] = panel ? (unsigned)first * (unsigned)K * 2u + (row - first) * 16u + lg * panel_rows * 16u : (unsigned)row * (unsigned)K * 2u + lg * 16u;
    }
    auto acts = [&](int t, int part, int k) { return (const f16x8*)((const char*)(part ? X + g.a_lo_off : X) + (long long)k * xs[t] + xo[t]); };

    f32x4 acc[NB][MT];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[b][t] = (f32x4){0.f, 0.f, 0.f, 0.f};


    // Epilogue operands that do not depend on the product are requested now, by the wavefront
    // that will run the epilogue: at these sizes a kernel is a chain of memory latencies, and
    // anything loaded after the K loop would add a full round trip to it.
    f32x4 pre_x[MT], pre_cs[MT], pre_sn[MT];
    unsigned pre_g[4] = {0u, 0u, 0u, 0u};      // bf16 as it is: converted or packed here, they would be waited for ahead of the first weights
    int pre_pos[MT], pre_slot[MT];
    if (wave == 0) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const int m = min(t * 16 + lr, M - 1);
            if (EPI == EPI_RESIDUAL) {
                pre_x[t] = *(const f32x4*)(g.Cf + (long long)m * N + min(n0 + lg * 4, N - 4));
            } else if (EPI == EPI_QKV) {
                pre_pos[t] = g.rope.row_pos[m];
                pre_slot[t] = g.rope.row_slot[m];
            }
        }
        if (EPI == EPI_RESIDUAL && g.gain_next) {
#pragma unroll
            for (int r = 0; r < 4; ++r) pre_g[r] = ((const unsigned short*)g.gain_next)[min(n0 + lg * 4 + r, N - 1)];
        }
    }

    // The same for the partial sums of x^2 behind the deferred RMSNorm: wavefront w turns those of
    // rows w, w + NW, .. into 1 / rms behind its first operands, from registers filled here (up to 256 partials per
    // row and 4 rows per wavefront; anything larger is fetched after the loop).
    constexpr int RPW = (MT * 16 + NW - 1) / NW;
    constexpr bool NORMED = EPI != EPI_RESIDUAL;           // (what a residual GEMM reads awaits no norm)
    constexpr bool PRE_SSQ = NORMED && RPW <= 4;
    float pre_ss[PRE_SSQ ? RPW : 1][4];
    const bool pre_ssq = PRE_SSQ && g.ssq && g.nparts <= 256;
    if constexpr (PRE_SSQ) {                               // (no branch around the loads, see below: without a norm something else is read, and not used)
        const float* sums = g.ssq ? g.ssq : (const float*)X;
        const int nparts = g.ssq ? g.nparts : 1;
#pragma unroll
        for (int j = 0; j < RPW; ++j) {
            const int m = min(wave + j * NW, M - 1);
            const float* src = sums + (long long)(a_rows ? a_rows[m] : m) * nparts;
#pragma unroll
            for (int u = 0; u < 4; ++u) pre_ss[j][u] = src[min(u * 64 + lane, nparts - 1)];
        }
    }

    // ... and turned into 1 / rms while the first trip's operands are on their way (the partial sums were
    // requested before them, so waiting for these does not wait for those): nothing of it is left after the K loop,
    // and its registers are free during the loop.
    auto finish_pre_ssq = [&]() {
#pragma unroll
        for (int j = 0; j < (PRE_SSQ ? RPW : 1); ++j) {
            float v = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) v += u * 64 + lane < g.nparts ? pre_ss[j][u] : 0.f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            const int r = wave + j * NW;
            if (lane == 0 && r < MT * 16) s_inv[r] = 1.0f / sqrtf(v / (float)g.d_norm + g.eps);
        }
    };

    // the angles follow from the positions, a second round trip: asked for behind the first operands
    auto request_angles = [&]() {
        if (EPI != EPI_QKV || wave != 0) return;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const long long ao = (long long)pre_pos[t] * (g.rope.kv.head_dim / 2) + q_j0 + (lg & 1) * 4;
            pre_cs[t] = *(const f32x4*)(g.rope.cos + ao);
            pre_sn[t] = *(const f32x4*)(g.rope.sin + ao);
        }
    };

    // One trip = U MFMA k-steps (32 each).  All weight and activation loads of trip i + 1 are issued
    // before trip i is multiplied (two register sets), so a wavefront always has a trip's worth
    // of loads (U KB of weights) in flight while its matrix pipe is busy.
    int k = kbeg;
    constexpr int U = 4, S = 32 * U;
    u32x4 rw[2][NB][DUAL ? U / 2 : U];
    f16x8 fx[2][NA][MT][U];
    auto loads = [&](int set, int kk) {
        if constexpr (DUAL) {
#pragma unroll
            for (int v = 0; v < U / 2; ++v) rw[set][0][v] = __builtin_nontemporal_load(weights(wb, wod, kk + 64 * v));
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                rw[set][0][u] = (COLS == 16 || wlane) ? __builtin_nontemporal_load(weights(wb, wo, kk + 32 * u)) : (u32x4){0u, 0u, 0u, 0u};
                if (NB == 2) rw[set][NB - 1][u] = __builtin_nontemporal_load(weights(wb2, wo, kk + 32 * u));
            }
        }
        // activation rows past M: the last row's address again, which costs no line of its own (a block re-reads its wavefronts' whole
        // activation slice, at 9 rows of 16 most of what the CU's load pipeline carries); their products go nowhere.  A branch around
        // the loads instead, and the compiler no longer knows how many are out: it waited for all of them ahead of the second trip.
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int p = 0; p < NA; ++p)
#pragma unroll
                for (int u = 0; u < U; ++u) fx[set][p][t][u] = *acts(t, p, kk + 32 * u);
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                u32x4 raw = rw[set][b][DUAL ? u >> 1 : u];
                if (DUAL && (u & 1)) {                 // odd k-step: lanes 8-15 of each row hold it; row_shl:8 brings it to lanes 0-7
#pragma unroll
                    for (int i = 0; i < 4; ++i) raw[i] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)raw[i], 0x108, 0xf, 0xf, true);
                }
                const f16x8 fw = __builtin_bit_cast(f16x8, raw);
#pragma unroll
                for (int t = 0; t < MT; ++t)
#pragma unroll
                    for (int p = 0; p < NA; ++p)
                        acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fw, fx[set][p][t][u], acc[b][t], 0, 0, 0);
            }
    };
    const int ntr = kslice / S;
    auto issue = [&](int set, int trip) {                        // all of a trip's loads, before anything that follows
        loads(set, kbeg + trip * S);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (ntr > 0) {
        issue(0, 0);
        request_angles();
        if (pre_ssq) finish_pre_ssq();
        int t = 0;
        for (; t + 2 < ntr; t += 2) {                            // both loads unconditional
            issue(1, t + 1);
            compute(0);
            issue(0, t + 2);
            compute(1);
        }
        if (t + 1 < ntr) {
            issue(1, t + 1);
            compute(0);
            compute(1);
        } else {
            compute(0);
        }
    } else {
        request_angles();
        if (pre_ssq) finish_pre_ssq();
    }
    k = kbeg + ntr * S;
    for (; k < kend; k += 32) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const f16x8 fw = __builtin_bit_cast(f16x8, *weights(b == 0 ? wb : wb2, wo, k));
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const f16x8 fx = *acts(t, 0, k);
                acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fw, fx, acc[b][t], 0, 0, 0);
                if (SPLIT) {
                    const f16x8 fl = *acts(t, 1, k);
                    acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fw, fl, acc[b][t], 0, 0, 0);
                }
            }
        }
    }

#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int t = 0; t < MT; ++t) red[wave][b][t][lane] = acc[b][t];
    if (!pre_ssq && NORMED && g.ssq) {   // deferred RMSNorm, not finished behind the first loads: the wavefronts share the rows
        for (int r = wave; r < min(MT * 16, M); r += NW) {
            const float inv = wave_inv_rms(g.ssq, a_rows ? a_rows[r] : r, g.nparts, g.d_norm, g.eps, lane);
            if (lane == 0) s_inv[r] = inv;
        }
    }
    __syncthreads();
    if (wave != 0) return;

#pragma unroll
    for (int t = 0; t < MT; ++t) {
        f32x4 sum[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            sum[b] = red[0][b][t][lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum[b] += red[w][b][t][lane];
        }
        const int m = t * 16 + lr, n = n0 + lg * 4;
        const bool mok = m < M && lg * 4 < COLS;
        const float inv = NORMED && g.ssq ? s_inv[t * 16 + lr] : 1.0f;
        const long long o = (long long)m * N + n;
        if (EPI == EPI_STORE_F32) {
            if (mok && n < N) *(f32x4*)(g.Cf + o) = sum[0] * inv;
        } else if (EPI == EPI_SWIGLU) {
            if (mok && n < N) {
                float h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) h[r] = silu_f(sum[0][r] * inv) * (sum[NB - 1][r] * inv);
                store_split4((f16*)g.C16 + act_index_few(g.c_layout == ACT_PANELS, m, n, M, N), g.c_lo_off, h);
            }
        } else if (EPI == EPI_RESIDUAL) {
            float ss = 0.f;
            if (mok && n < N) {
                const f32x4 xn = pre_x[t] + sum[0];
                *(f32x4*)(g.Cf + o) = xn;
                if (g.gain_next) {
                    float h[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        h[r] = xn[r] * __uint_as_float(pre_g[r] << 16);
                        ss += xn[r] * xn[r];
                    }
                    store_split4((f16*)g.C16 + act_index_few(g.c_layout == ACT_PANELS, m, n, M, N), g.c_lo_off, h);
                }
            }
            if (g.gain_next) {           // sum of squares over the block's COLS columns, per row
                ss += __shfl_xor(ss, 16, 64);
                ss += __shfl_xor(ss, 32, 64);
                if (lg == 0 && mok) g.ssq_out[(long long)m * (N / COLS) + blockIdx.x] = ss;
            }
        } else {                         // EPI_QKV
            const RopeArgs& ro = g.rope;
            const int Hq = ro.n_q_heads, Hkv = ro.kv.n_kv_heads, hd = ro.kv.head_dim;
            const int mm = min(m, M - 1);
            f16* pool = (f16*)ro.kv.base;
            const int chan = (lg < 2 ? q_j0 + lg * 4 : hd / 2 + q_j0 + (lg - 2) * 4);   // first of 4 channels
            f32x4 own = sum[0] * inv, other;
#pragma unroll
            for (int r = 0; r < 4; ++r) other[r] = __shfl_xor(own[r], 32, 64);
            if (q_head < Hq + Hkv) {
                const f32x4 cs = pre_cs[t], sn = pre_sn[t];      // angles q_j0 + (lg & 1) * 4 + r at the row's position
                float h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    h[r] = lg < 2 ? own[r] * cs[r] - other[r] * sn[r]                   // first half: a c - b s
                                  : own[r] * cs[r] + other[r] * sn[r];                  // second half: b c + a s
                f16* dst;
                long long lo_off = 0;                                                    // the cache holds one fp16 per entry
                if (q_head < Hq) {
                    dst = (f16*)ro.q_out + ((long long)mm * Hq + q_head) * hd;
                    lo_off = g.c_lo_off;
                } else {
                    dst = pool + ro.kv.plane(ro.layer, 0, q_head - Hq) + (long long)pre_slot[t] * hd;
                }
                if (mok) store_split4(dst + chan, lo_off, h);
            } else if (mok) {
                f16* dst = pool + ro.kv.plane(ro.layer, 1, q_head - Hq - Hkv) + (long long)(pre_slot[t] >> 4) * 16 * hd + (pre_slot[t] & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r) dst[(long long)(chan + r) * 16] = (f16)own[r];
            }
        }
    }
}

// Launch KERNEL<TARGS..., SPLIT>: the split-activation instantiation when the GEMM's A operand comes in two parts.
#define AX_UNPAREN(...) __VA_ARGS__
#define AX_SPLIT_LAUNCH(split_, KERNEL, TARGS, GRID, BLOCK, ...)                                        \
    do {                                                                                                \
        if (split_) KERNEL<AX_UNPAREN TARGS, true><<<GRID, BLOCK, 0, s>>>(__VA_ARGS__);                  \
        else KERNEL<AX_UNPAREN TARGS, false><<<GRID, BLOCK, 0, s>>>(__VA_ARGS__);                        \
    } while (0)

// Columns per block of the skinny kernel.  A CU pulls only ~26 GB/s of weights however many
// wavefronts it runs (measured), so a launch streams at the chip's rate only if every CU has a
// block: residual GEMMs (N = d_model, too few blocks of 16 columns) use 12 or 8 columns per
// block when that shortens rounds-of-256-blocks x columns.
static int skinny_cols(int epi, int N) {
    if (epi != EPI_RESIDUAL) return 16;
    int best = 16, best_cost = ((N / 16 + 255) / 256) * 16;
    for (int c : {12, 8}) {
        if (N % c) continue;
        const int cost = ((N / c + 255) / 256) * c;
        if (cost < best_cost) { best = c; best_cost = cost; }
    }
    return best;
}

template <int EPI, int MT, int COLS>
static void launch_skinny_cols(const GemmArgs& g, int nw, hipStream_t s) {
    const int grid = (g.N + COLS - 1) / COLS;
    if (nw == 16) AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_skinny_kernel, (EPI, MT, 16, COLS), grid, 1024, g);
    else if (nw == 1) AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_skinny_kernel, (EPI, MT, 1, COLS), grid, 64, g);
    else if (nw == 2) AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_skinny_kernel, (EPI, MT, 2, COLS), grid, 128, g);
    else if (nw == 8) AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_skinny_kernel, (EPI, MT, 8, COLS), grid, 512, g);
    else AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_skinny_kernel, (EPI, MT, 4, COLS), grid, 256, g);
}

template <int EPI, int MT>
static void launch_skinny_nw(const GemmArgs& g, int nw, hipStream_t s) {
    if constexpr (EPI == EPI_RESIDUAL) {
        const int c = skinny_cols(EPI, g.N);
        if (c == 8) { launch_skinny_cols<EPI, MT, 8>(g, nw, s); return; }
        if (c == 12) { launch_skinny_cols<EPI, MT, 12>(g, nw, s); return; }
    }
    launch_skinny_cols<EPI, MT, 16>(g, nw, s);
}

static constexpr int kPanelRows = 32;        // rows up to which plain activations lie in panels of few rows

// Dispatch thresholds.  Each is a measured crossover (figures at its use); the product build compiles them in
// as constants.  Only a build with -DAX_TUNING_KNOBS (kernel tuning sessions) lets the environment override them.
#ifdef AX_TUNING_KNOBS
static int env_int(const char* name, int dflt) {
    const char* v = std::getenv(name);
    return v && *v ? std::atoi(v) : dflt;
}
#else
static constexpr int env_int(const char*, int dflt) { return dflt; }
#endif
static const int kSwigluWaves = env_int("AX_SWIGLU_WAVES", 4096);   // wavefronts in flight the SwiGLU launch aims for (two weight streams per wavefront)
static const int kLmStream = env_int("AX_LM_STREAM", 1);   // experiment knob
static const int kForceNW = env_int("AX_SKINNY_NW", 0);   // experiment knob: wavefronts per block, 0 = automatic

// More rows: LDS-staged tiles.
static const int kQkvTile = env_int("AX_QKV_TILE", -1);   // experiment knobs: force 64-row (0) or 128-row (1) blocks
static const int kResTile = env_int("AX_RES_TILE", -1);
static const int kResBig = env_int("AX_RES_BIG", 256);
static const int kQkvKs = env_int("AX_QKV_KS", 0);   // experiment knob: K slices of the QKV GEMM (1 = never split)
// Which blocks and how many K slices the tile kernel takes for a QKV or residual GEMM (ws_bytes: room for slabs).  Reached by layers that keep rows,
// 257-304 rows of most widths and up to 512 of layers much wider than d_model (plan_many weighs it against the block kernel), and by widths that
// are no multiple of 64.  Two block shapes, both of 8 wavefronts: 64 x 128 (2 x 4 wavefronts of 32 x 32) and 128 x 128 (wavefront tile 64 x 32), which
// pulls a third fewer operand bytes per output.  At 257-304 rows of the ~1B, ~3B and ~8B layers it is 64-row blocks that stay ahead of the block
// kernel, in us: ~1B QKV in 2 slices 12.9 (block kernel 13.1), ~3B down in 2 slices 28.4 (31.2), ~8B QKV in hi + lo parts, whole, 41.5 (43.7).
struct TilePlan { bool big; int ks; };
template <int EPI>
static TilePlan plan_tile(int M, int N, int K, size_t ws_bytes) {
    const long long tiles64 = (long long)((N + 127) / 128) * ((M + 63) / 64);
    const long long tiles128 = (long long)((N + 127) / 128) * ((M + 127) / 128);
    // 128-row blocks only when their row padding costs at most ~15 % more rows than 64-row blocks' (M = 144 does not qualify)
    const bool pad_ok = (long long)((M + 127) / 128) * 128 * 100 <= (long long)((M + 63) / 64) * 64 * 115;
    const size_t slab = (size_t)M * N * sizeof(float);
    if constexpr (EPI == EPI_QKV) {
        // 128-row blocks from 80 tiles up: fewer leave too many CUs idle.  64-row blocks: two slices only while both fit one round of 256 blocks
        // (more blocks than CUs run two to a CU and gain nothing from the cut: ~1B at 384 rows 26.8 -> 24.7 us whole, ~3B / ~8B at 320 rows
        // 35.2 -> 32.3 / 43.0 -> 39.1 us)
        const bool big = kQkvTile >= 0 ? kQkvTile > 0 : (pad_ok && tiles128 >= 80);
        int ks = big ? (tiles128 < 128 ? 2 : 1) : (tiles64 * 2 <= 256 ? 2 : 1);
        // three slices of 128-row blocks where they fill the chip better than two and K divides (80 tiles: 240 blocks instead of 160; four, 320
        // blocks, would be two rounds)
        if (big && ks == 2 && tiles128 * 3 <= 256 && K % (3 * 64) == 0 && K / (3 * 64) >= 8 && 3 * slab <= ws_bytes) ks = 3;
        if (kQkvKs > 0) ks = kQkvKs;
        while (ks > 1 && (K % (ks * 64) != 0 || ks * slab > ws_bytes)) ks >>= 1;
        return {big, ks};
    } else {
        // Few output tiles (320 rows against N = 2048 are 80 tiles of 64 x 128 for 256 CUs): cut K until there are ~256 blocks, each still with 8 or
        // more k-steps; fp32 partial slabs go to the workspace and residual_reduce_kernel finishes.
        auto slices = [&](long long tiles) {
            int ks = 1;
            if (!ws_bytes || N % 64 != 0) return ks;
            // (a cut that would overshoot one round of 256 blocks is not taken once 144 or more CUs have a block: ~1B at 384 rows 37.5 -> 30.2 us,
            // ~8B O projection at 384 rows 39.3 -> 31.0)
            static const int fill = env_int("AX_SLICE_FILL", 144);   // measurement switch: 256 = always cut up to a full round
            while (ks < SPLITK_MAX && tiles * ks < 256 && !(tiles * ks >= fill && tiles * ks * 2 > 256) &&
                   K % (ks * 2 * 64) == 0 && K / (ks * 2 * 64) >= 8 && ks * 2 * slab <= ws_bytes)
                ks *= 2;
            return ks;
        };
        // 128-row blocks: when there are plenty of tiles without any cut (or more 64-row tiles than one round of two per CU), or when K is long (down
        // projection) and at most 4 slices give ~200 blocks or more (~8B down projection at 512 rows 98 -> 81 us).
        const int ks128 = slices(tiles128);
        const bool big = kResTile >= 0 ? kResTile > 0 : (pad_ok && (tiles128 >= kResBig || tiles64 > 256 || (K >= 4096 && ks128 <= 4 && tiles128 * ks128 >= 192)));
        return {big, big ? ks128 : slices(tiles64)};
    }
}

template <int EPI>
static int launch_lds_tile(const GemmArgs& g, hipStream_t s) {
    const int M = g.M, N = g.N, K = g.K;
    if constexpr (EPI == EPI_QKV) {
        // A plain store GEMM writes fp32 products, a second kernel does the rms scaling, rotary
        // embedding and KV append: measured faster than a fused epilogue (one head per wavefront)
        // at 512 rows of all three model shapes.  With few tiles K is cut in slices that the second
        // kernel adds up.
        // (The workspace holds at least one [M, N] fp32 slab - a model's layout reserves max_tokens x N of it
        // whatever the ratio of N to d_model; a caller that brings less gets nothing launched.)
        const TilePlan t = plan_tile<EPI>(M, N, K, g.split_ws ? g.split_ws_bytes : 0);
        if (!g.split_ws || (size_t)M * N * sizeof(float) > g.split_ws_bytes) return -1;
        GemmArgs gs = g;
        gs.ksplit = t.ks;
        GemmArgs gp = gs;                                 // the products: no scaling, no epilogue work
        gp.ssq = nullptr;
        gp.Cf = g.split_ws;
        if (t.big) {
            dim3 grid((N + 127) / 128, (M + 127) / 128, t.ks);
            AX_SPLIT_LAUNCH(gp.a_lo_off != 0, gemm_bf16_tile_kernel, (EPI_STORE_F32, 2, 1, 2, 4), grid, 512, gp);
        } else {
            dim3 grid((N + 127) / 128, (M + 63) / 64, t.ks);
            AX_SPLIT_LAUNCH(gp.a_lo_off != 0, gemm_bf16_tile_kernel, (EPI_STORE_F32, 1, 1, 2, 4), grid, 512, gp);
        }
        launch_qkv_reduce(gs, s);
        return 0;
    } else if constexpr (EPI == EPI_RESIDUAL) {
        const TilePlan t = plan_tile<EPI>(M, N, K, g.split_ws ? g.split_ws_bytes : 0);
        GemmArgs gs = g;
        gs.ksplit = t.ks;
        if (t.big) {
            dim3 grid((N + 127) / 128, (M + 127) / 128, t.ks);
            AX_SPLIT_LAUNCH(gs.a_lo_off != 0, gemm_bf16_tile_kernel, (EPI_RESIDUAL, 2, 1, 2, 4), grid, 512, gs);
        } else {
            dim3 grid((N + 127) / 128, (M + 63) / 64, t.ks);
            AX_SPLIT_LAUNCH(gs.a_lo_off != 0, gemm_bf16_tile_kernel, (EPI_RESIDUAL, 1, 1, 2, 4), grid, 512, gs);
        }
        return t.ks > 1 ? launch_residual_reduce(gs, s) : N / 32;
    } else {
        static_assert(EPI == EPI_STORE_F32, "SwiGLU runs on other kernels");
        const bool split = g.a_lo_off != 0;     // (streaming blocks of at most 128 rows: a second A ring does not fit the registers of larger ones)
        // logits (N >= 64 K columns) of 17 rows or more: streaming blocks of up to 192 rows per 256 columns
        // read the LM head once per block row at 5-6 TB/s; the skinny kernel re-reads its activations
        // per 16 columns (17 rows of the ~3B shape: 182 -> 128 us) and 64-row tiles read the weights
        // once per tile (96-128 rows: 282-294 -> 149-157 us; 144 rows: 436 -> 202 us).  Rows per
        // block by the same rounds x block cost as the SwiGLU kernel.
        if (M > 16 && N >= 256 * 256 && N % 32 == 0 && kLmStream) {
            const int gx = (N + 255) / 256;
            int tm = (M + 31) / 32;
            if (M > 512) {
                tm = 4;                                    // compute-bound there: 128-row blocks (1024 rows: 669 us against 804 with 192-row blocks)
            } else if (tm > (split ? 4 : 6)) {
                long long best = -1;
                for (int t : {4, 3, 5, 6}) {
                    if (split && t > 4) continue;
                    const long long blocks = (long long)gx * ((M + 32 * t - 1) / (32 * t));
                    const long long cost = ((blocks + 255) / 256) * (32 * t + 512) * (t >= 5 ? 115 : 100);
                    if (best < 0 || cost < best) { best = cost; tm = t; }
                }
            }
            const int gy = (M + 32 * tm - 1) / (32 * tm);
            switch (tm) {
                case 1: AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_STORE_F32, 1, 3), gx * gy, 256, g, gx, gy); break;
                case 2: AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_STORE_F32, 2, 3), gx * gy, 256, g, gx, gy); break;
                case 3: AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_STORE_F32, 3, 3), gx * gy, 256, g, gx, gy); break;
                case 4: AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_STORE_F32, 4, 3), gx * gy, 256, g, gx, gy); break;
                case 5: gemm_bf16_stream_kernel<EPI_STORE_F32, 5, 3><<<gx * gy, 256, 0, s>>>(g, gx, gy); break;
                default: gemm_bf16_stream_kernel<EPI_STORE_F32, 6, 3><<<gx * gy, 256, 0, s>>>(g, gx, gy); break;
            }
            return 0;
        }
        // last-row logits of more than 512 sequences (their rows gathered, which the block kernel does not do): 128 x 256 streaming
        // blocks where they fill the 256 CUs evenly - a single round of 128 or more, or rounds at least 3/4 full
        const long long sblocks = (long long)((N + 255) / 256) * ((M + 127) / 128), rounds = (sblocks + 255) / 256;
        if (M >= 512 && N % 32 == 0 && sblocks >= 128 && (rounds == 1 || sblocks * 4 >= rounds * 256 * 3)) {
            const int gx = (N + 255) / 256, gy = (M + 127) / 128;
            AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_STORE_F32, 4, 3), gx * gy, 256, g, gx, gy);
            return 0;
        }
        dim3 grid((N + 127) / 128, (M + 63) / 64);
        AX_SPLIT_LAUNCH(split, gemm_bf16_tile_kernel, (EPI_STORE_F32, 1, 1, 2, 4), grid, 512, g);
    }
    return 0;
}

// ------------------------------------------------------------------------------ more than 256 rows
// Activations in rows: the block kernel has the largest tiles and wins wherever they fill the chip; two kernels made for fewer rows are ahead of
// it where its plan leaves CUs idle or pads rows, and stay candidates (times fitted to the same calls as the block kernel's):
//   * the tile kernel, QKV and residual GEMMs of up to 512 rows whose blocks fit one round (with the reduce kernels behind both: ~1B QKV at
//     288 rows 18.6 -> 16.6 us, ~3B down at 257 rows 36.2 -> 33.5, ~8B QKV in hi + lo parts at 272 rows 53.1 -> 49.2);
//   * streaming blocks of 96 to 192 rows (plain activations; 96 or 128 in hi + lo parts), SwiGLU of up to 640 rows (~8B width at 320 rows:
//     block kernel, 512 padded rows, 100 us, 2 x 160 rows 89; at 576 rows 185 and 180; in hi + lo parts at 576 rows 307 and 285).
enum ManyRows { MANY_BLOCK, MANY_TILE, MANY_STREAM };
struct ManyPlan { ManyRows kernel; BlockPlan block; int stream_tm; float us; };

template <int EPI>
static float tile_us(int M, int N, int K, bool split, size_t ws_bytes) {
    static constexpr struct { float lo, full, fixed, whole, qkv; } kTile[2][2] = {      // [128-row blocks][split]; a step is 64 k
        {{0.328f, 0.372f, 5.6f, 5.1f, 0.4f}, {0.492f, 0.567f, 6.1f, 5.0f, 0.4f}}, {{0.346f, 0.620f, 7.0f, 12.2f, 1.5f}, {0.590f, 1.071f, 7.3f, 6.6f, 1.3f}}};
    const TilePlan p = plan_tile<EPI>(M, N, K, ws_bytes);
    const int rows = p.big ? 128 : 64;
    const long long blocks = (long long)((N + 127) / 128) * ((M + rows - 1) / rows) * p.ks;
    if (blocks > 256) return 1e30f;
    const auto& t = kTile[p.big][split];
    const float us = t.fixed + K / p.ks / 64 * (t.lo + (t.full - t.lo) * blocks / 256);
    if (EPI == EPI_QKV) return us + t.qkv + gemm_reduce_us(EPI_QKV, M, N, p.ks, false);
    return us + (p.ks > 1 ? gemm_reduce_us(EPI_RESIDUAL, M, N, p.ks, false) : t.whole + gemm_partials_us(M, false));
}

// SwiGLU streaming blocks of 32 tm rows x 128 columns of gate and of up, one on a CU at a time
static float stream_us(int M, int N, int K, bool split, int tm) {
    const long long blocks = (long long)((N + 127) / 128) * ((M + 32 * tm - 1) / (32 * tm)), rest = blocks % 256;
    const float step = split ? 0.44f * tm : 0.076f + 0.239f * tm, fixed = split ? 13.6f : 12.6f, lo = split ? 0.65f : 0.71f;
    return blocks / 256 * (step * (K / 64) + fixed) + (rest ? step * (lo + (1.f - lo) * rest / 256) * (K / 64) + fixed : 0.f);
}

template <int EPI>
static ManyPlan plan_many(int M, int N, int K, bool split, size_t ws_bytes) {
    ManyPlan p{MANY_BLOCK, plan_gemm_block((Epilogue)EPI, M, N, K, split, false, ws_bytes), 0, 0.f};
    p.us = p.block.us;
    if constexpr (EPI == EPI_QKV || EPI == EPI_RESIDUAL) {
        if (M <= 512 && (EPI == EPI_RESIDUAL || (size_t)M * N * sizeof(float) <= ws_bytes)) {
            const float us = tile_us<EPI>(M, N, K, split, ws_bytes);
            if (us < p.us) { p.us = us; p.kernel = MANY_TILE; }
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        for (int tm = 3; M <= 640 && tm <= (split ? 4 : 6); ++tm) {      // (a second ring of activations does not fit the registers of larger blocks)
            const float us = stream_us(M, N, K, split, tm);
            if (us < p.us) { p.us = us; p.kernel = MANY_STREAM; p.stream_tm = tm; }
        }
    }
    return p;
}
static bool many_rows(int M, int N, bool gathered) { return M > 256 && !gathered && N % 64 == 0; }

static void launch_swiglu_stream(const GemmArgs& g, int tm, hipStream_t s) {
    const int gx = (g.N + 127) / 128, gy = (g.M + 32 * tm - 1) / (32 * tm);
    switch (tm) {
        case 3: AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_SWIGLU, 3, 3), gx * gy, 256, g, gx, gy); break;
        case 5: gemm_bf16_stream_kernel<EPI_SWIGLU, 5, 3><<<gx * gy, 256, 0, s>>>(g, gx, gy); break;
        case 6: gemm_bf16_stream_kernel<EPI_SWIGLU, 6, 3><<<gx * gy, 256, 0, s>>>(g, gx, gy); break;
        default: AX_SPLIT_LAUNCH(g.a_lo_off != 0, gemm_bf16_stream_kernel, (EPI_SWIGLU, 4, 3), gx * gy, 256, g, gx, gy); break;
    }
}

// ------------------------------------------------------------------------------ 17-256 rows
// The register kernel (k_gemm_regs.h): tile and K slices by a time fitted to all tiles that are built, alone and on cold weights, for the four GEMMs
// of the ~1B, ~3B and ~8B (hi + lo) layers at 2-16 panels of rows, 600 launches, most within 1.5 us.  A round of 256 blocks is 3.4-4.4 us of first round trips,
// sums and epilogue and, per 32 k, 0.025 us for each panel of W that no other row block has brought to the L2 (1 KB: 41 GB/s a CU; less while few CUs
// ask) and 0.0145 for every other panel (70 GB/s).  Slices cost slabs and the kernel that adds them up.  Inside models the forms chosen so are the fastest or
// within 2 us of it at 17-256 rows.  More than one round is taken where it pulls less (~8B gate / up at 176 rows: 448 blocks).
struct RegsPlan { int shape, ks; float us; };
static RegsPlan plan_regs(Epilogue epi, int M, int N, int K, bool split, bool slices, size_t ws_bytes) {
    RegsPlan best{-1, 1, 0.f};
    const int panels = (M + 15) / 16, chunks = K / 32, na = split ? 2 : 1;
    const int force = env_int("AX_REGS", -1), force_epi = env_int("AX_REGS_EPI", -1), force_ks = env_int("AX_REGS_KS", 1);
    for (int c = 0; c < kRegsShapes; ++c) {
        const RegsShape& t = kRegs[split][c];
        if (t.mt > panels + 1) continue;
        const int cols = (epi == EPI_SWIGLU ? 8 : 16) * t.nt;
        for (int ks = 1; ks <= 8; ks *= 2) {
            if (ks > 1 && (epi != EPI_RESIDUAL || !slices || (size_t)ks * M * N * sizeof(float) > ws_bytes || chunks / ks < 16)) break;
            if (!regs_built(epi, split, ks > 1, c)) continue;
            const int gy = (panels + t.mt - 1) / t.mt, gx = (N + cols - 1) / cols;
            const long long blocks = (long long)gx * gy * ks;
            const float rounds = (blocks + 255) / 256, crowd = std::min(1.f, std::max(0.6f, blocks / 256.f));
            const float miss = (float)t.nt / gy, hit = t.nt - miss + t.mt * na;
            const int tiles = t.mt * t.nt;
            float us = rounds * ((tiles <= 4 ? 3.4f : 4.4f) + 0.12f * std::max(0, tiles - 24) + (float)chunks / ks * (0.025f * crowd * miss + 0.0145f * hit));
            if (ks > 1) us += 3.4f + 0.4f * ks + 0.4e-6f * ks * M * N;
            else if (epi == EPI_RESIDUAL) us += 0.01f * std::max(0, gx - 192);      // (partial sums of x^2 a row, for the next GEMM to read)
            if (force >= 0 && force_epi == (epi == EPI_RESIDUAL && K > 2 * N ? 4 : epi) && !(c == force && ks == force_ks)) us += 1e6f;
            if (best.shape < 0 || us <= best.us) best = {c, ks, us};
        }
    }
    return best;
}
static int launch_regs_plan(Epilogue epi, const GemmArgs& g, const RegsPlan& p, hipStream_t s) {
    if (epi == EPI_QKV) { launch_regs_qkv(g, p.shape, s); return 0; }
    if (epi == EPI_SWIGLU) { launch_regs_swiglu(g, p.shape, s); return 0; }
    if (p.ks == 1) {
        launch_regs_residual(g, p.shape, s);
        const int cols = 16 * kRegs[g.a_lo_off != 0][p.shape].nt;
        return (g.N + cols - 1) / cols;
    }
    GemmArgs gs = g;
    gs.ksplit = p.ks;
    launch_regs_slices(gs, p.shape, s);
    return launch_residual_reduce(gs, s);
}
// Hi + lo parts in strips have the block kernel beside it, by the times that both plans expect: bound by their products, many rows multiply faster
// through LDS (~8B gate / up at 200-256 rows 130-140 us here, 100 on 128 x 256 blocks).
struct StripPlan { bool block; RegsPlan regs; BlockPlan tiles; };
static StripPlan plan_strips(Epilogue epi, int M, int N, int K, bool split, bool strips, bool slices, size_t ws_bytes) {
    StripPlan p{false, plan_regs(epi, M, N, K, split, slices, ws_bytes), {}};
    if (split && strips && N % 64 == 0) {
        p.tiles = plan_gemm_block(epi, M, N, K, split, true, ws_bytes);
        const int fb = env_int("AX_BLOCK", -1);
        p.block = fb < 0 ? p.tiles.us < p.regs.us && env_int("AX_REGS", -1) < 0 : fb == (epi == EPI_RESIDUAL && K > 2 * N ? 4 : epi);
    }
    return p;
}
static int launch_regs(Epilogue epi, const GemmArgs& g, hipStream_t s) {
    const StripPlan p = plan_strips(epi, g.M, g.N, g.K, g.a_lo_off != 0, g.a_layout == ACT_STRIPS, g.split_ws != nullptr, g.split_ws ? g.split_ws_bytes : 0);
    return p.block ? launch_gemm_block(epi, g, p.tiles, s) : launch_regs_plan(epi, g, p.regs, s);
}

static int regs_shape(bool split, int rows, int cols) {
    for (int c = 0; c < kRegsShapes; ++c)
        if (kRegs[split][c].mt * 16 == rows && kRegs[split][c].nt * 16 == cols) return c;
    return -1;
}
bool gemm_regs_built(Epilogue epi, bool split, int rows, int cols, int slices) {
    const int c = regs_shape(split, rows, cols);
    return c >= 0 && epi != EPI_STORE_F32 && (slices == 1 || epi == EPI_RESIDUAL) && regs_built(epi, split, slices > 1, c);
}
int launch_gemm_regs_as(Epilogue epi, const GemmArgs& g, int rows, int cols, int slices, hipStream_t s) {
    return launch_regs_plan(epi, g, {regs_shape(g.a_lo_off != 0, rows, cols), slices, 0.f}, s);
}

template <int EPI>
static int launch_bf16(const GemmArgs& g, hipStream_t s) {
    const int M = g.M, N = g.N, K = g.K;
    if (g.a_layout == ACT_PANELS && M > 256) return launch_gemm_block((Epilogue)EPI, g, plan_gemm_block((Epilogue)EPI, M, N, K, g.a_lo_off != 0, true, g.split_ws ? g.split_ws_bytes : 0), s);
    if (many_rows(M, N, g.a_rows != nullptr)) {
        const ManyPlan p = plan_many<EPI>(M, N, K, g.a_lo_off != 0, g.split_ws ? g.split_ws_bytes : 0);
        if (p.kernel == MANY_BLOCK) return launch_gemm_block((Epilogue)EPI, g, p.block, s);
        if constexpr (EPI != EPI_SWIGLU) return launch_lds_tile<EPI>(g, s);
        launch_swiglu_stream(g, p.stream_tm, s);
        return 0;
    }
    if (EPI != EPI_STORE_F32 && M > 16 && M <= 256) return launch_regs((Epilogue)EPI, g, s);
    const bool far_rows = g.a_rows && (unsigned long long)g.a_total_rows * K * 2 > 0xffffffffull;      // gathered rows past what the offsets below hold
    // logits of 17-32 rows: narrow ones only (wide ones on streaming blocks, see launch_lds_tile)
    if ((M <= 16 || (M <= 32 && EPI == EPI_STORE_F32 && !(N >= 256 * 256 && kLmStream))) && !far_rows) {
        // wavefronts per block (= K slices): enough to keep ~2k wavefronts in flight (~4k for the SwiGLU
        // GEMM: 8 instead of 4 wavefronts per block took the ~1B verify kernel from 16.6 to 14.7 us), each with
        // at least 128 of K; K / nw must stay a multiple of the MFMA k (32)
        const int cols = skinny_cols(EPI, N);
        const long long tiles = (N + cols - 1) / cols;
        int nw = 1;
        const int wave_target = EPI == EPI_SWIGLU ? kSwigluWaves : 2048;
        while (nw < 16 && tiles * nw < wave_target && K % (nw * 2 * 32) == 0 && K / (nw * 2) >= 128) nw *= 2;
        if (kForceNW > 0 && K % (std::max(kForceNW, 1) * 32) == 0) nw = kForceNW;
        if (EPI == EPI_SWIGLU && nw == 16) nw = 8;        // LDS reduction buffer stays <= 64 KB
        if (M <= 16) launch_skinny_nw<EPI, 1>(g, nw, s);
        else if constexpr (EPI == EPI_STORE_F32) launch_skinny_nw<EPI, 2>(g, nw, s);
        return EPI == EPI_RESIDUAL ? N / cols : 0;
    }
    if constexpr (EPI != EPI_SWIGLU) return launch_lds_tile<EPI>(g, s);
    return 0;                                                  // (SwiGLU: no rows are gathered, and N of a layer is a multiple of 64)
}

static GemmPlan block_plan(const BlockPlan& p) { return {"block", p.shape == 0 ? 256 : 128, p.shape == 2 ? 128 : 256, p.ks}; }
template <int EPI>
static GemmPlan many_rows_plan(int M, int N, int K, bool split, size_t ws_bytes) {
    const ManyPlan p = plan_many<EPI>(M, N, K, split, ws_bytes);
    if (p.kernel == MANY_STREAM) return {"stream", 32 * p.stream_tm, 256, 1};
    if constexpr (EPI == EPI_QKV || EPI == EPI_RESIDUAL)
        if (p.kernel == MANY_TILE) {
            const TilePlan t = plan_tile<EPI>(M, N, K, ws_bytes);
            return {"tile", t.big ? 128 : 64, 128, t.ks};
        }
    return block_plan(p.block);
}
GemmPlan gemm_plan(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes) {
    if (!many_rows(M, N, false)) return {"", 0, 0, 0};
    if (epi == EPI_STORE_F32) return many_rows_plan<EPI_STORE_F32>(M, N, K, split, ws_bytes);
    if (epi == EPI_RESIDUAL) return many_rows_plan<EPI_RESIDUAL>(M, N, K, split, ws_bytes);
    if (epi == EPI_SWIGLU) return many_rows_plan<EPI_SWIGLU>(M, N, K, split, ws_bytes);
    return many_rows_plan<EPI_QKV>(M, N, K, split, ws_bytes);
}

GemmPlan gemm_strip_plan(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes) {
    const StripPlan p = plan_strips(epi, M, N, K, split, M > kPanelRows || split, ws_bytes > 0, ws_bytes);
    if (p.block) return block_plan(p.tiles);
    const RegsShape& t = kRegs[split][p.regs.shape];
    return {"regs", 16 * t.mt, 16 * t.nt, p.regs.ks};
}

GemmPlan gemm_panel_plan(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes) {
    return block_plan(plan_gemm_block(epi, M, N, K, split, true, ws_bytes));
}

// Up to 16 rows one panel, which the few-row kernel reads in fewer lines than rows; up to 256 rows strips, except plain activations of 17-32 rows, which
// keep panels: both are read by the register kernel, at 17-20 rows panels are ahead (us a call, panels / strips: ~1B 17 rows 937 / 954, ~3B 2066 / 2116), at
// 24-32 strips (~1B 976 / 963 and 1020 / 974, ~3B 2153 / 2133 and 2258 / 2149).
// More than 256 rows, by the times that the plans expect: panels make the block kernel faster at every size, but only that kernel reads them,
// and the ones made for fewer rows are ahead of it where its third row tile is mostly padding (~8B at 257 rows: rows 11.4 ms, panels 11.8) and
// in layers much wider than d_model.  Rows where they are expected 4 % ahead, 8 % with more than 3/8 of that tile filled: over 19 layers at 17
// row counts from 257 to 512 the calls chosen so take 0.4 % (d_model 2048 and more) and 2 % (less) longer than with the faster layout and forms.
ActLayout gemm_layer_layout(int M, int d_model, int qkv, int qdim, int d_ff, bool split, size_t ws_bytes) {
    if (M <= 16 || (M <= kPanelRows && !split)) return ACT_PANELS;
    if (M <= 256) return ACT_STRIPS;
    auto panels = [&](Epilogue epi, int N, int K) { return plan_gemm_block(epi, M, N, K, split, true, ws_bytes).us; };
    const float rows = plan_many<EPI_QKV>(M, qkv, d_model, split, ws_bytes).us + plan_many<EPI_RESIDUAL>(M, d_model, qdim, split, ws_bytes).us +
                       plan_many<EPI_SWIGLU>(M, d_ff, d_model, split, ws_bytes).us + plan_many<EPI_RESIDUAL>(M, d_model, d_ff, split, ws_bytes).us;
    return panels(EPI_QKV, qkv, d_model) + panels(EPI_RESIDUAL, d_model, qdim) + panels(EPI_SWIGLU, d_ff, d_model) + panels(EPI_RESIDUAL, d_model, d_ff) < (M <= 304 ? 1.04f : 1.08f) * rows ? ACT_PANELS : ACT_ROWS;
}

int launch_gemm_bf16(Epilogue epi, const GemmArgs& g, hipStream_t s) {
    if (epi == EPI_STORE_F32) return launch_bf16<EPI_STORE_F32>(g, s);
    if (epi == EPI_RESIDUAL) return launch_bf16<EPI_RESIDUAL>(g, s);
    if (epi == EPI_SWIGLU) return launch_bf16<EPI_SWIGLU>(g, s);
    return launch_bf16<EPI_QKV>(g, s);
}

void launch_gemm(DType dt, Epilogue epi, const void* A, const void* W, const void* W2, void* C,
                 int M, int N, int K, hipStream_t s) {
    if (dt == F32) {
        GemmF32Args g{};
        g.A = (const float*)A; g.W = (const float*)W; g.W2 = (const float*)W2; g.C = (float*)C;
        g.M = M; g.N = N; g.K = K;
        launch_gemm_f32(epi, g, s);
        return;
    }
    GemmArgs g{};
    g.A = A; g.W = W; g.W2 = W2; g.M = M; g.N = N; g.K = K;
    g.Cf = (float*)C;
    g.C16 = C;
    const bool odd = epi == EPI_SWIGLU && M > 256 && N % 64 != 0;              // no layer has these, and no kernel of more than 256 rows takes them
    for (int r0 = 0; r0 < M; r0 += odd ? 256 : M) {
        if (odd) {
            g.M = std::min(256, M - r0);
            g.A = (const f16*)A + (long long)r0 * K;
            g.C16 = (f16*)C + (long long)r0 * N;
        }
        launch_gemm_bf16(epi, g, s);
    }
}

}  // namespace ax
