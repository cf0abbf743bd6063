// GEMMs of 17 to 256 rows (bf16-weight models): C = A[M,K] * W[N,K]^T, both operands straight from memory to registers.
//
// The wavefronts of a block share nothing but their output: each multiplies the block's whole tile of 16 MT rows x 16 NT columns over its own
// part of K, so no operand is read twice by a block, nothing is staged, and there is no barrier until the partial sums meet in LDS.  With A in
// panels of 16 rows and W packed, every load is the 1 KB that one lane order of the 16x16x32 MFMA takes.
//
// What bounds it: how fast a CU is filled.  A probe takes 120 GB/s a CU out of its XCD's L2 and 27 from HBM with all CUs at work, and loads return in
// order, so the two add up; beside its products and its sums this kernel reaches 70 and 41 (weights that few CUs ask for at once among them),
// and a round of blocks starts and ends for 3.4-4.4 us.  plan_regs takes the tile and the K slices with the least such time, mostly one round of 256 blocks or fewer.
// Against the kernels that served these rows before - 64-row tiles in LDS or streaming blocks, with K slices and a
// kernel that adds them up - in us a layer's GEMM, those kernels included: ~3B at 144 rows
// QKV 21.8 -> 18.7, O 18.6 -> 14.4, gate / up 46.5 -> 31.5, down 28.3 -> 27.7; ~8B (hi + lo) at 17 rows 24.8 -> 18.3, 14.6 -> 13.5, 44.8 -> 35, 27.3 -> 29.8;
// at 256 rows of ~1B gate / up 27.5 -> 28.4, the other three and so the call ahead.
// Whole calls, timed in turn: ~1B 48 rows 1298 -> 1030, 100 rows 1508 -> 1281, 256 rows 1717 -> 1640 over 2048 cached keys, 1724 -> 1706 over 4096; ~3B 64 rows 2808 ->
// 2555, 256 rows 4048 -> 4001; ~8B 24 rows 4401 -> 4075, 160 rows 10134 -> 7552, 256 rows 10213 -> 9054.
#pragma once

#include "gemm_device.h"

namespace ax {

// EPI: the epilogue (GemmArgs).  NW wavefronts; D register sets of operands, of which D - 1 are in flight.
// SPLIT: A in hi and lo parts, both multiplied with the same fragments of W.
// SLICED: K is cut into g.ksplit slices over extra blocks; raw products go to slabs of g.split_ws.
// Columns: tile j of a block is 16 columns.  SwiGLU: the first NT / 2 tiles are gate, the others up; QKV: tile j and j + NT / 2 are the rotary
// partners of 16 channels of a head.  A and C16 in any layout.
template <int EPI, int MT, int NT, int NW, int D, bool SPLIT, bool SLICED>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4)))
void gemm_regs_kernel(GemmArgs g, int gy) {
    constexpr bool PAIRED = !SLICED && (EPI == EPI_SWIGLU || EPI == EPI_QKV);
    constexpr int NA = SPLIT ? 2 : 1, NO = PAIRED ? NT / 2 : NT;           // NO: column tiles (or pairs of them) a block finishes
    static_assert(!PAIRED || NT % 2 == 0, "column tiles in pairs");
    // Row tiles whose partial sums lie in LDS at a time, and what one wavefront finishes at a time, a unit: a row tile, of 1 / CS of the columns
    constexpr int FIT = 144 / (NW * NT), MR = FIT < MT ? FIT : MT, ROUNDS = (MT + MR - 1) / MR;
    static_assert(FIT > 0, "a row tile's partial sums fit LDS");
    constexpr bool CUT = EPI != EPI_RESIDUAL || SLICED;                    // (the sum of x^2 of a row is taken over all of a unit's columns)
    constexpr int CS = CUT && NO % 4 == 0 && MR * 4 <= NW ? 4 : CUT && NO % 2 == 0 && MR * 2 <= NW ? 2 : 1, NU = NO / CS;
    constexpr int UPW = (MR * CS + NW - 1) / NW, U = ROUNDS * UPW;         // units per wavefront and round, and altogether
    __shared__ f32x4 red[NW][MR][NT][64];

    const int M = g.M, N = g.N, K = g.K;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    // block -> tile: XCD c (workgroups are dealt out round robin) takes the c-th eighth, row blocks of the same columns side by side, so that
    // they read W out of one L2
    const int slices = SLICED ? g.ksplit : 1, nblk = gridDim.x / slices, kz = SLICED ? blockIdx.x / nblk : 0;
    int id = (int)blockIdx.x - kz * nblk;
    {
        const int q = nblk >> 3, r = nblk & 7, c = id & 7;
        id = c * q + min(c, r) + (id >> 3);
    }
    const int bx = id / gy, by = id - bx * gy;

    // this wavefront's chunks of 32 k
    const int chunks = K >> 5, k0 = SLICED ? chunks * kz / slices : 0, kn = SLICED ? chunks * (kz + 1) / slices - k0 : chunks;
    const int c0 = k0 + kn * wave / NW, n = k0 + kn * (wave + 1) / NW - c0;

    // operands: buffer descriptors and a lane's 32-bit offset to each panel, advanced by a scalar
    const bool strips = g.a_layout == ACT_STRIPS, a_panels = g.a_layout == ACT_PANELS;
    const int panels = (M + 15) >> 4, p0 = by * MT, last_rows = a_panels ? M - (panels - 1) * 16 : 16;
    const unsigned a_bytes = (unsigned)(strips ? panels * 16 : M) * (unsigned)K * 2u;
    const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)g.A, 0, (int)a_bytes, 0x00027000);
    const auto rl = __builtin_amdgcn_make_buffer_rsrc((void*)((const f16*)g.A + (SPLIT ? g.a_lo_off : 0)), 0, (int)a_bytes, 0x00027000);
    const int step = strips ? panels * 1024 : a_panels ? 1024 : 64, step_tail = a_panels ? last_rows * 64 : step;      // bytes per 32 k
    unsigned ao[MT];
    bool tail[MT];                                                          // the last panel, whose runs may be shorter (ACT_PANELS)
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int p = min(p0 + i, panels - 1), row = min(p * 16 + lr, M - 1);
        tail[i] = p == panels - 1;
        const int rows = tail[i] ? last_rows : 16;
        ao[i] = strips     ? (unsigned)p * 1024u + lane * 16u
                : a_panels ? (unsigned)p * (unsigned)K * 32u + (unsigned)(lg * rows + min(lr, rows - 1)) * 16u
                           : (unsigned)row * (unsigned)K * 2u + lg * 16u;
    }
    const int hd = EPI == EPI_QKV && !SLICED ? g.rope.kv.head_dim : 64, pph = hd >> 5;       // rotary pairs of tiles in a head
    auto panel_of = [&](int j) {                                            // panel of W (or W2) of column tile j; past the end: the last one again
        if (PAIRED && EPI == EPI_QKV) {
            const int pair = min(bx * NO + j % NO, (N >> 5) - 1), head = pair / pph;
            return head * 2 * pph + (pair - head * pph) + (j >= NO ? pph : 0);
        }
        return min(bx * NO + (PAIRED ? j % NO : j), (N >> 4) - 1);
    };
    const long long first = (long long)panel_of(0) * 16 * K;
    const unsigned w_bytes = (unsigned)min(((long long)N * K - first) * 2, 0x7fffffffll);
    const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)((const f16*)g.W + first), 0, (int)w_bytes, 0x00027000);
    const auto rw2 = __builtin_amdgcn_make_buffer_rsrc((void*)((const f16*)(EPI == EPI_SWIGLU ? g.W2 : g.W) + first), 0, w_bytes, 0x00027000);
    unsigned wo[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) wo[j] = (unsigned)(panel_of(j) - panel_of(0)) * (unsigned)K * 32u + lane * 16u;

    // Partial sums of x^2 of the units' rows, and their positions: the first requests, before the operands
    constexpr int BATCH = 16;
    constexpr bool NORMED = PAIRED;
    const int row_tile0 = wave / CS, cg = wave % CS;                        // unit u of round r: row tile r * MR + (wave + u * NW) / CS
    static_assert(NW % CS == 0, "a wavefront's units are of the same columns");
    auto tile_of_unit = [&](int u) { return u / UPW * MR + (u % UPW) * (NW / CS) + row_tile0; };
    auto row_of_unit = [&](int u) { return (p0 + tile_of_unit(u)) * 16 + lr; };
    float ss[NORMED ? U : 1][BATCH];
    int pos[U], slot[U];
    const bool by_part = ssq_by_part(g.a_layout, M);
    const float* sums = g.ssq ? g.ssq : (const float*)g.A;                  // (no branch around the loads: without a norm M floats of A are read, and not used)
    const int nparts = g.ssq ? g.nparts : 1;
    auto request_ssq = [&](int part0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < BATCH; ++b) ss[u][b] = sums[ssq_index(by_part, min(row_of_unit(u), M - 1), min(part0 + b * 4 + lg, nparts - 1), M, nparts)];
    };
    float inv[U];
    auto add_ssq = [&](int part0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < BATCH; ++b) inv[u] += part0 + b * 4 + lg < nparts ? ss[u][b] : 0.f;
    };
#pragma unroll
    for (int u = 0; u < U; ++u) inv[u] = 0.f;
    if constexpr (NORMED) request_ssq(0);
    if constexpr (PAIRED && EPI == EPI_QKV) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pos[u] = g.rope.row_pos[min(row_of_unit(u), M - 1)];
            slot[u] = g.rope.row_slot[min(row_of_unit(u), M - 1)];
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x4 acc[MT][NT];
    u32x4 fa[D][NA * MT], fw[D][NT];
    auto issue = [&](auto may_end, int set, int c) {
        const int so = (c0 + c) * 1024, sa = (c0 + c) * step, st = (c0 + c) * step_tail;
        // a chunk past the last one: an offset past the descriptor's end, which loads zeros from nowhere (no branch, so that the compiler knows how
        // many loads are out)
        const unsigned past = decltype(may_end)::value && c >= n ? 0x80000000u : 0u;
#pragma unroll
        for (int j = 0; j < NT; ++j) fw[set][j] = __builtin_amdgcn_raw_buffer_load_b128(PAIRED && j >= NO ? rw2 : rw, wo[j] | past, so, 2);      // (not temporal: HBM 6.0 -> 7.0 TB/s)
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            fa[set][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, ao[i] | past, tail[i] ? st : sa, 0);
            if (SPLIT) fa[set][(NA - 1) * MT + i] = __builtin_amdgcn_raw_buffer_load_b128(rl, ao[i] | past, tail[i] ? st : sa, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int p = 0; p < NA; ++p)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, fw[set][j]), __builtin_bit_cast(f16x8, fa[set][p * MT + i]), acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // one wavefront per SIMD: its sums stay in accumulation registers (left alone, the compiler moves them back and forth between the loops)
    auto pin = [&]() {
        if constexpr (NW == 4) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
    };
    // what the epilogue needs from memory, asked for behind the last operands
    constexpr bool RES = EPI == EPI_RESIDUAL && !SLICED, ROPE = PAIRED && EPI == EPI_QKV;
    f32x4 pre0[RES || ROPE ? U : 1][NU], pre1[ROPE ? U : 1][NU];            // x, or the cosines and sines
    unsigned gain[RES ? NU : 1][4];                                         // bf16 as it is
    auto request = [&]() {
        if constexpr (RES) {
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                const int col = min((bx * NO + cg * NU + j) * 16, N - 16) + lg * 4;
#pragma unroll
                for (int u = 0; u < U; ++u) pre0[u][j] = *(const f32x4*)(g.Cf + (long long)min(row_of_unit(u), M - 1) * N + col);
                const unsigned short* gp = (const unsigned short*)(g.gain_next ? g.gain_next : (const void*)g.Cf) + col;
#pragma unroll
                for (int x = 0; x < 4; ++x) gain[j][x] = gp[x];
            }
        }
        if constexpr (ROPE) {
#pragma unroll
            for (int j = 0; j < NU; ++j) {
                const int pair = min(bx * NO + cg * NU + j, (N >> 5) - 1), ch = pair % pph * 16 + lg * 4;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const long long at = (long long)pos[u] * (hd >> 1) + ch;
                    pre0[u][j] = *(const f32x4*)(g.rope.cos + at);
                    pre1[u][j] = *(const f32x4*)(g.rope.sin + at);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto norm = [&]() {                                                     // 1 / rms of the units' rows, while the first operands are on their way
        if constexpr (NORMED) {
            add_ssq(0);
            for (int part0 = BATCH * 4; part0 < nparts; part0 += BATCH * 4) {
                request_ssq(part0);
                add_ssq(part0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                inv[u] += __shfl_xor(inv[u], 16, 64);
                inv[u] += __shfl_xor(inv[u], 32, 64);
                inv[u] = g.ssq ? 1.0f / sqrtf(inv[u] / (float)g.d_norm + g.eps) : 1.0f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    constexpr std::true_type may_end{};
    constexpr std::false_type whole{};
#pragma unroll
    for (int s = 0; s < D - 1; ++s) issue(may_end, s, s);
    norm();
    pin();
    int t = 0;
    for (; t + 2 * D - 1 <= n; t += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            issue(whole, (u + D - 1) % D, t + u + D - 1);
            compute(u);
        }
        pin();
    }
#pragma unroll
    for (int u = 0; u < 2 * D - 1; ++u) {
        if (u < D) issue(may_end, (u + D - 1) % D, t + u + D - 1);
        if (u == D - 1) request();
        if (t + u < n) compute(u % D);
    }
    pin();

#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        if (r) __syncthreads();                                             // the round before has been read
#pragma unroll
        for (int i = 0; i < MR; ++i)
            if (r * MR + i < MT)
#pragma unroll
                for (int j = 0; j < NT; ++j) red[wave][i][j][lane] = acc[r * MR + i][j];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < UPW; ++q) {
            const int u = r * UPW + q, i = q * (NW / CS) + row_tile0, m = (p0 + r * MR + i) * 16 + lr;
            if (i >= MR || r * MR + i >= MT) continue;                      // wavefront-uniform
            auto sum = [&](int j) {
                f32x4 s = red[0][i][j][lane];
#pragma unroll
                for (int w = 1; w < NW; ++w) s += red[w][i][j][lane];
                return s;
            };
            const bool live = m < M;
            if constexpr (SLICED) {
#pragma unroll
                for (int j = 0; j < NU; ++j) {
                    const int col = (bx * NO + cg * NU + j) * 16 + lg * 4;
                    const f32x4 v = sum(cg * NU + j);
                    if (live && col < N) *(f32x4*)(g.split_ws + ((long long)kz * M + m) * N + col) = v;
                }
            } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
                for (int j = 0; j < NU; ++j) {
                    const int col = (bx * NO + cg * NU + j) * 16 + lg * 4;
                    const f32x4 a = sum(cg * NU + j), b = sum(NO + cg * NU + j);
                    float h[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) h[x] = silu_lean(a[x] * inv[u]) * (b[x] * inv[u]);
                    if (live && col < N) store_split4((f16*)g.C16 + act_index(g.c_layout, m, col, M, N), g.c_lo_off, h);
                }
            } else if constexpr (EPI == EPI_RESIDUAL) {
                float sq = 0.f;
#pragma unroll
                for (int j = 0; j < NU; ++j) {
                    const int col = (bx * NO + cg * NU + j) * 16 + lg * 4;
                    const f32x4 x = pre0[u][j] + sum(cg * NU + j);
                    if (live && col < N) {
                        *(f32x4*)(g.Cf + (long long)m * N + col) = x;
                        if (g.gain_next) {
                            float h[4];
#pragma unroll
                            for (int y = 0; y < 4; ++y) h[y] = x[y] * __uint_as_float(gain[j][y] << 16);
                            store_split4((f16*)g.C16 + act_index(g.c_layout, m, col, M, N), g.c_lo_off, h);
                            sq += x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
                        }
                    }
                }
                if (g.gain_next) {
                    sq += __shfl_xor(sq, 16, 64);
                    sq += __shfl_xor(sq, 32, 64);
                    const int parts = (N + NO * 16 - 1) / (NO * 16);
                    if (lg == 0 && live) g.ssq_out[ssq_index(ssq_by_part(g.c_layout, M), m, bx, M, parts)] = sq;
                }
            } else {                                                        // EPI_QKV
                const RopeArgs& ro = g.rope;
                const int Hq = ro.n_q_heads, Hkv = ro.kv.n_kv_heads, half = hd >> 1;
                f16* pool = (f16*)ro.kv.base;
#pragma unroll
                for (int j = 0; j < NU; ++j) {
                    const int pair = bx * NO + cg * NU + j, head = pair / pph, ch = (pair - head * pph) * 16 + lg * 4;
                    const f32x4 a = sum(cg * NU + j) * inv[u], b = sum(NO + cg * NU + j) * inv[u];
                    if (pair >= N >> 5 || !live) continue;
                    if (head < Hq + Hkv) {
                        const f32x4 cs = pre0[u][j], sn = pre1[u][j];
                        f16* dst = head < Hq ? (f16*)ro.q_out + ((long long)m * Hq + head) * hd
                                             : pool + ro.kv.plane(ro.layer, 0, head - Hq) + (long long)slot[u] * hd;
                        const long long lo_off = head < Hq ? g.c_lo_off : 0;         // q may be split; the cache holds one fp16 per entry
                        float va[4], vb[4];
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            va[x] = a[x] * cs[x] - b[x] * sn[x];
                            vb[x] = b[x] * cs[x] + a[x] * sn[x];
                        }
                        store_split4(dst + ch, lo_off, va);
                        store_split4(dst + ch + half, lo_off, vb);
                    } else {
                        f16* dst = pool + ro.kv.plane(ro.layer, 1, head - Hq - Hkv) + (long long)(slot[u] >> 4) * 16 * hd + (slot[u] & 15);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            dst[(long long)(ch + x) * 16] = (f16)a[x];
                            dst[(long long)(ch + x + half) * 16] = (f16)b[x];
                        }
                    }
                }
            }
        }
    }
}

// The tiles that are built: row tiles, column tiles, wavefronts, register sets.
struct RegsShape { int mt, nt, nw, d; };
static constexpr int kRegsShapes = 20;
static constexpr RegsShape kRegs[2][kRegsShapes] = {       // [split]
    {{2, 1, 8, 4}, {2, 2, 8, 4}, {2, 4, 8, 4}, {3, 2, 8, 4}, {3, 3, 8, 4}, {3, 4, 8, 4}, {4, 2, 8, 4}, {4, 3, 8, 4}, {4, 4, 4, 6},
     {5, 4, 4, 4}, {6, 4, 4, 4}, {8, 4, 4, 4}, {9, 4, 4, 4}, {2, 8, 4, 4}, {3, 8, 4, 4}, {4, 8, 4, 4}, {5, 8, 4, 3},
     {6, 8, 4, 3}, {7, 8, 4, 3}, {8, 8, 4, 3}},
    {{2, 1, 8, 4}, {2, 2, 8, 4}, {2, 4, 8, 3}, {3, 2, 8, 3}, {3, 4, 8, 2}, {4, 2, 8, 3}, {4, 4, 4, 4}, {5, 4, 4, 3}, {6, 4, 4, 3},
     {8, 4, 4, 2}, {9, 4, 4, 2}, {2, 8, 4, 4}, {3, 8, 4, 3}, {4, 8, 4, 3}, {5, 8, 4, 2}, {6, 8, 4, 2}, {7, 8, 4, 2}, {8, 8, 4, 2}}};
// Which of them an epilogue runs on: column tiles in pairs; residual GEMMs that finish on their own have few columns.
constexpr bool regs_built(int epi, bool split, bool sliced, int shape) {
    const RegsShape s = kRegs[split][shape];
    if (s.mt == 0) return false;
    if (sliced) return s.nt >= 2;
    if (epi == EPI_RESIDUAL) return s.mt <= 5 && s.nt <= 4;
    return s.nt % 2 == 0;
}
template <int EPI, bool SPLIT, bool SLICED, int SHAPE = 0>
void launch_regs_shape(const GemmArgs& g, int shape, hipStream_t s) {
    if constexpr (SHAPE < kRegsShapes) {
        if (shape != SHAPE) return launch_regs_shape<EPI, SPLIT, SLICED, SHAPE + 1>(g, shape, s);
        if constexpr (regs_built(EPI, SPLIT, SLICED, SHAPE)) {
            constexpr RegsShape r = kRegs[SPLIT][SHAPE];
            constexpr int cols = (EPI == EPI_SWIGLU && !SLICED ? 8 : 16) * r.nt;
            const int gx = (g.N + cols - 1) / cols, gy = ((g.M + 15) / 16 + r.mt - 1) / r.mt;
            gemm_regs_kernel<EPI, r.mt, r.nt, r.nw, r.d, SPLIT, SLICED><<<gx * gy * (SLICED ? g.ksplit : 1), 64 * r.nw, 0, s>>>(g, gy);
        }
    }
}
void launch_regs_qkv(const GemmArgs& g, int shape, hipStream_t s);
void launch_regs_swiglu(const GemmArgs& g, int shape, hipStream_t s);
void launch_regs_residual(const GemmArgs& g, int shape, hipStream_t s);
void launch_regs_slices(const GemmArgs& g, int shape, hipStream_t s);

}  // namespace ax
