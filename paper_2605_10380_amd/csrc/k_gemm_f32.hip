// fp32 GEMMs of fp32-weight models: C = A[M,K] * W[N,K]^T, any M, N, K, on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products, fp32 accumulation - the fp32 configuration is the exactness
// configuration, 1e-4 against the float64 oracle, so nothing narrower is used here).
//
// What bounds these calls is latency: the fp32 models are small, a verify step of the "tiny" shape multiplies 5 rows.
// A 64 x 64 LDS tile per block (the earlier kernel) gave such a launch 4 to 64 blocks that walked K in 16-wide,
// barrier-separated steps: 26-50 us each.  Here a block owns 16 output columns and 16 * MT rows, its wavefronts take
// every NW-th step of 16 k, read both operands straight from memory (float4 per lane, a batch of steps in flight
// before the first product) and meet once in LDS.  tiny verify step of 5 rows: QKV 26 -> 4.7 us (with rotary and KV append,
// before a kernel of their own), O 27 -> 4.3, gate / up 50 -> 5.0, down 69 -> 5.0 us.
//
// The RMSNorm in front of QKV and gate / up is folded in: the block reads whole rows of x anyway, so it multiplies them
// by the gain on the way, sums the squares itself and scales the finished products by 1 / rms.
//
// MT = 1 (16 rows per block, 8 wavefronts) while that is at most 2048 blocks, MT = 4 (64 rows, 4 wavefronts: every
// weight fragment meets four row tiles) above, where the chip is full either way and operand re-reads count
// (130-256 rows of the tiny shape: 8-10 us a launch with MT = 4, 5 with MT = 1).
#include "kernels.h"

namespace ax {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Operand layout of the 16x16x4 product: lane l supplies row (or column) l % 16 at ONE k per instruction, k = l / 16;
// result register r of lane l is D[4 * (l / 16) + r][l % 16].  A lane loads four consecutive k (4 * (l / 16) .. + 3 of a
// 16-wide step) in one float4 and instruction j of the step takes element j of both operands: the same four k in a
// different order, which a sum does not mind.  D rows are output columns n, D columns are rows m.
//
// ROPE (EPI_QKV): the block's 16 columns are 8 rotary pairs (j, j + hd / 2), pair p = 8 * blockIdx.x + i of head p / (hd / 2);
// local column i is the pair's first channel, 8 + i its second.
template <int EPI, int MT, int NW, int U, bool VEC>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmF32Args g) {
    constexpr int NB = EPI == EPI_SWIGLU ? 2 : 1;
    __shared__ __attribute__((aligned(16))) f32x4 red[NW][NB][MT][64];
    __shared__ float s_ss[NW][MT][16];

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int M = g.M, N = g.N, K = g.K;
    const int m0 = blockIdx.y * 16 * MT;
    const int half = EPI == EPI_QKV ? g.rope.kv.head_dim >> 1 : 1, n_pairs = N >> 1;
    // column of local index c: 16 consecutive ones, or rotary pairs
    auto column = [&](int c) {
        if (EPI != EPI_QKV) return (int)blockIdx.x * 16 + c;
        const int p = (int)blockIdx.x * 8 + (c & 7);
        return p < n_pairs ? (p / half) * 2 * half + p % half + (c >> 3) * half : N;
    };
    const int wrow = min(column(lr), N - 1);
    const float* wp[NB];
    wp[0] = g.W + (long long)wrow * K;
    if (NB == 2) wp[NB - 1] = g.W2 + (long long)wrow * K;
    const float* ap[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int m = min(m0 + t * 16 + lr, M - 1);
        ap[t] = g.A + (long long)(g.a_rows ? g.a_rows[m] : m) * K;
    }

    // four consecutive k from k on, zeros past the end of the row
    auto load4 = [&](const float* row, int k) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (VEC) {
            if (k < K) v = *(const f32x4*)(row + k);             // K % 4 == 0
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) if (k + i < K) v[i] = row[k + i];
        }
        return v;
    };

    f32x4 acc[NB][MT];
    float ss[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        ss[t] = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }

    const int steps = (K + 15) / 16, mine = wave < steps ? (steps - wave + NW - 1) / NW : 0;
    f32x4 fa[2][U][MT], fw[2][U][NB], fg[2][U];
    auto loads = [&](int set, int i0) {                          // steps past the last one load zeros
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = i0 + u < mine ? (wave + (i0 + u) * NW) * 16 + lg * 4 : K;
#pragma unroll
            for (int b = 0; b < NB; ++b) fw[set][u][b] = load4(wp[b], k);
#pragma unroll
            for (int t = 0; t < MT; ++t) fa[set][u][t] = load4(ap[t], k);
            if (g.gain) fg[set][u] = load4(g.gain, k);
        }
    };
    auto multiply = [&](int set) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                f32x4 a = fa[set][u][t];
                if (g.gain) {
                    ss[t] += a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3];
                    a *= fg[set][u];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[set][u][b][j], a[j], acc[b][t], 0, 0, 0);
            }
    };
    loads(0, 0);
    for (int i = 0; i < mine; i += 2 * U) {
        if (i + U < mine) loads(1, i + U);
        multiply(0);
        if (i + U >= mine) break;
        if (i + 2 * U < mine) loads(0, i + 2 * U);
        multiply(1);
    }

#pragma unroll
    for (int t = 0; t < MT; ++t) {
#pragma unroll
        for (int b = 0; b < NB; ++b) red[wave][b][t][lane] = acc[b][t];
        if (g.gain) {
            ss[t] += __shfl_xor(ss[t], 16, 64);
            ss[t] += __shfl_xor(ss[t], 32, 64);
            if (lg == 0) s_ss[wave][t][lr] = ss[t];
        }
    }
    __syncthreads();

    // one output element per thread and pass: 16 consecutive local columns of a row sit in 16 lanes
    for (int e = threadIdx.x; e < MT * 256; e += 64 * NW) {
        const int c = e & 15, ml = (e >> 4) & 15, t = e >> 8, m = m0 + t * 16 + ml, n = column(c);
        const int src = (c >> 2) * 16 + ml;
        float v[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            v[b] = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) v[b] += red[w][b][t][src][c & 3];
        }
        if (g.gain) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += s_ss[w][t][ml];
            const float inv = 1.0f / sqrtf(s / (float)K + g.eps);
#pragma unroll
            for (int b = 0; b < NB; ++b) v[b] *= inv;
        }
        const bool live = m < M && n < N;
        const long long o = (long long)m * N + n;
        if (EPI == EPI_STORE_F32) {
            if (live) g.C[o] = v[0];
        } else if (EPI == EPI_RESIDUAL) {
            if (live) g.C[o] = (g.res ? g.res[(long long)(g.res_rows ? g.res_rows[m] : m) * N + n] : g.C[o]) + v[0];
        } else if (EPI == EPI_SWIGLU) {
            if (live) g.C[o] = v[0] / (1.0f + expf(-v[0])) * v[NB - 1];
        } else {
            const float other = __shfl_xor(v[0], 8, 64);         // the pair's other channel (whole wavefronts get here: MT * 256 is a multiple of 64)
            if (live) {
                g.C[o] = v[0];                                   // the product as it is, for inspection
                const RopeArgs& ro = g.rope;
                const int hd = 2 * half, head = n / hd, ch = n % hd, j = ch < half ? ch : ch - half;
                const int Hq = ro.n_q_heads, Hkv = ro.kv.n_kv_heads, slot = ro.row_slot[m];
                float* pool = (float*)ro.kv.base;
                if (head < Hq + Hkv) {
                    const long long ao = (long long)ro.row_pos[m] * half + j;
                    const float cs = ro.cos[ao], sn = ro.sin[ao];
                    const float r = ch < half ? v[0] * cs - other * sn : v[0] * cs + other * sn;
                    float* dst = head < Hq ? (float*)ro.q_out + ((long long)m * Hq + head) * hd
                                           : pool + ro.kv.plane(ro.layer, 0, head - Hq) + (long long)slot * hd;
                    dst[ch] = r;
                } else {
                    pool[ro.kv.plane(ro.layer, 1, head - Hq - Hkv) + (long long)(slot >> 4) * 16 * hd + (long long)ch * 16 + (slot & 15)] = v[0];
                }
            }
        }
    }
}

template <int EPI, bool VEC>
static void launch_f32(const GemmF32Args& g, hipStream_t s) {
    const unsigned nx = EPI == EPI_QKV ? (unsigned)((g.N / 2 + 7) / 8) : (unsigned)((g.N + 15) / 16);
    if ((long long)nx * ((g.M + 15) / 16) <= 2048) gemm_f32_kernel<EPI, 1, 8, 4, VEC><<<dim3(nx, (unsigned)((g.M + 15) / 16)), 512, 0, s>>>(g);
    else gemm_f32_kernel<EPI, 4, 4, 2, VEC><<<dim3(nx, (unsigned)((g.M + 63) / 64)), 256, 0, s>>>(g);
}

void launch_gemm_f32(Epilogue epi, const GemmF32Args& g, hipStream_t s) {
    // float4 loads: whole rows in 16-byte pieces
    const bool vec = g.K % 4 == 0 && (((uintptr_t)g.A | (uintptr_t)g.W | (uintptr_t)g.W2 | (uintptr_t)g.gain) & 15) == 0;
    switch (epi) {
        case EPI_STORE_F32: vec ? launch_f32<EPI_STORE_F32, true>(g, s) : launch_f32<EPI_STORE_F32, false>(g, s); break;
        case EPI_RESIDUAL: vec ? launch_f32<EPI_RESIDUAL, true>(g, s) : launch_f32<EPI_RESIDUAL, false>(g, s); break;
        case EPI_SWIGLU: vec ? launch_f32<EPI_SWIGLU, true>(g, s) : launch_f32<EPI_SWIGLU, false>(g, s); break;
        case EPI_QKV: vec ? launch_f32<EPI_QKV, true>(g, s) : launch_f32<EPI_QKV, false>(g, s); break;
    }
}

}  // namespace ax
