// GEMMs of many rows (bf16-weight models): C = A[M,K] * W[N,K]^T on the fp16 matrix cores, both operands staged through LDS by
// the memory pipeline itself (global_load_lds: no registers, no ds_write in between), blocks of up to 256 x 256 outputs.
//
// What bounds it: a CU takes ~20 bytes per clock out of L2 (64 lines of 128 B in flight over ~400 clocks), and 256 x 256 outputs
// need 32 KB of operands per 32 k, 1024 clocks of its matrix cores - so ~64 % of the matrix rate is what the largest tile that fits the
// registers can reach.  Counters (gate / up of the ~3B shape at 4096 rows; profiles/config5_block_kernel_counters.txt): matrix cores busy
// 60 % of the cycles, 19.1 B per clock and CU, pending-request queue full half of the time, LDS instructions in a quarter of the cycles and
// under 1 % of them in conflict, clock held at 1.79 GHz by power.
//   * Stages of 32 k, up to four in LDS, so that the copies of three steps are in flight: with two stages of 64 k the queue of outstanding
//     lines ran dry between a stage's arrival and the issue of the next one (~1B gate / up, 4096 rows: 283 -> 264 us).
//   * 8 wavefronts, two per SIMD.  4 wavefronts of 128 x 128 outputs need a third fewer LDS reads but were 5-15 % slower: one
//     wavefront per SIMD leaves the matrix cores idle at every barrier.
//   * Smaller tiles (128 x 256, 128 x 128) move 1.5x / 2x the operands per product; they are for launches that would leave CUs without a
//     block (the planner at the end weighs tile and K-slice choices by measured times).
#include "gemm_device.h"
#include "lds_copy.h"

#include <algorithm>

namespace ax {

// 16 rows' sums over 32 lanes (v[r]: this lane's share of row r) with a transposing butterfly: at each stage a lane hands half of its
// values to its partner and keeps the other half.  Returns the total of row (lane % 32) >> 1.
__device__ __forceinline__ float rows16_sum(float (&v)[16], int lane) {
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int n = 16 >> st, o = 16 >> st;
        const bool upper = (lane & o) != 0;
#pragma unroll
        for (int j = 0; j < n / 2; ++j) {
            const float send = upper ? v[j] : v[j + n / 2], keep = upper ? v[j + n / 2] : v[j];
            v[j] = keep + __shfl_xor(send, o, 64);
        }
    }
    return v[0] + __shfl_xor(v[0], 1, 64);
}

// Two values of one column (rows r and r + 1 of an accumulator) become two columns of one row: a lane trades one of them with its
// neighbour, so that fp16 results leave as 4-byte stores.  Even lanes end up with row r, odd lanes with row r + 1, columns
// n & ~1 and + 1 either way.
__device__ __forceinline__ f32x2 pair_of_columns(float r0, float r1, bool odd) {
    const float send = odd ? r0 : r1;
    const float got = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xb1, 0xf, 0xf, true));   // lane ^ 1
    return odd ? (f32x2){got, r1} : (f32x2){r0, got};
}
__device__ __forceinline__ void store_split2(f16* p, long long lo_off, f32x2 v) {
    v = (f32x2){split_value(v[0]), split_value(v[1])};
    const f16x2 hi = {(f16)v[0], (f16)v[1]};
    *(f16x2*)p = hi;
    if (lo_off) *(f16x2*)(p + lo_off) = (f16x2){(f16)(v[0] - (float)hi[0]), (f16)(v[1] - (float)hi[1])};
}

// EPI: the epilogue (GemmArgs).  TM x TN tiles of 32 x 32 outputs per wavefront, WM x WN wavefronts, S stages in LDS.
// SPLIT: split activations - hi and lo parts of A are staged and multiplied against the same B fragments.
// SLICED: K is cut into g.ksplit slices over extra blocks; raw products go to slabs of g.split_ws.
// Blocks are renumbered: XCD c (workgroups are dealt out round robin) takes the c-th eighth of the tiles, in groups of `group` row tiles
// walked column by column, so that the ~32 tiles an XCD works on at a time share operands in its L2.
template <int EPI, int TM, int TN, int WM, int WN, int S, bool SPLIT, bool SLICED>
__global__ __launch_bounds__(64 * WM * WN) void gemm_block_kernel(GemmArgs g, int gx, int gy, int group) {
    constexpr int NW = WM * WN, BM = WM * TM * 32, BN = WN * TN * 32, BK = 32, NA = SPLIT ? 2 : 1;
    constexpr int A_BYTES = NA * BM * 64, B_BYTES = BN * 64, STAGE = A_BYTES + B_BYTES;
    constexpr int LA = NA * BM / 16 / NW, LB = BN / 16 / NW, L = LA + LB;      // copies per wavefront and stage
    static_assert(NA * BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "whole copies per wavefront");
    static_assert(EPI != EPI_SWIGLU || TN == 2, "SwiGLU: one gate and one up tile per wavefront");
    constexpr int OUT_N = EPI == EPI_SWIGLU ? BN / 2 : BN;
    __shared__ __attribute__((aligned(1024))) char smem[S * STAGE];
    __shared__ float s_inv[BM];

    const int M = g.M, N = g.N, K = g.K;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave / WN, wn = wave % WN, lrow = lane & 31, lg = lane >> 5;

    // block -> tile
    const int nblk = gx * gy, kz = SLICED ? blockIdx.x / nblk : 0;
    int id = SLICED ? (int)blockIdx.x - kz * nblk : (int)blockIdx.x;
    {
        const int q = nblk >> 3, r = nblk & 7, c = id & 7;
        id = c * q + min(c, r) + (id >> 3);
    }
    const int gsz = group * gx, gi = id / gsz, first = gi * group, height = min(group, gy - first), rem = id - gi * gsz;
    const int bx = rem / height, by = first + rem - bx * height;
    const int m0 = by * BM, n0 = bx * OUT_N;
    const int kspan = SLICED ? K / g.ksplit : K, kbase = kz * kspan;

    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
    // copies of this wavefront: A units of 16 rows x 32 k (lane: row lane / 4, 16-byte slot lane % 4), B units of one chunk of a panel
    // (1 KB as packed).  Slot s of row r holds k-group s ^ swz(r): see the operand reads.
    auto swz = [](int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); };
    const char* a_base = (const char*)g.A + ((long long)m0 * K + kbase) * 2;
    unsigned a_off[LA];
    const char* a_ptr[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int unit = wave * LA + i, part = unit / (BM / 16), row = (unit % (BM / 16)) * 16 + (lane >> 2);
        a_off[i] = (unsigned)min(row, M - 1 - m0) * (unsigned)K * 2u + (unsigned)(((lane & 3) ^ swz(row)) * 16);
        a_ptr[i] = a_base + (SPLIT && part ? g.a_lo_off * 2 : 0);
    }
    const char* b_ptr[LB];
    const unsigned b_off = (unsigned)lane * 16;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int pl = wave * LB + i;                                  // panel of the stage
        const bool second = EPI == EPI_SWIGLU && pl >= BN / 32;
        const int panel = min((n0 >> 4) + (second ? pl - BN / 32 : pl), (N >> 4) - 1);
        b_ptr[i] = (const char*)(second ? g.W2 : g.W) + ((long long)panel * 16 * K + (long long)kbase * 16) * 2;
    }
    auto load_stage = [&](int s, int buf) {
        const unsigned at = lds0 + buf * STAGE;
#pragma unroll
        for (int i = 0; i < LA; ++i) copy_to_lds(a_ptr[i] + (long long)s * 64, a_off[i], at + (wave * LA + i) * 1024);
#pragma unroll
        for (int i = 0; i < LB; ++i) copy_to_lds(b_ptr[i] + (long long)s * 1024, b_off, at + A_BYTES + (wave * LB + i) * 1024);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int nsteps = kspan / BK;
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < nsteps) load_stage(s, s);
    const bool inv_here = g.ssq && !SLICED;
    if (inv_here) {
        if (g.nparts <= 4) block_inv_rms_few(g, m0, BM, s_inv);
        else block_inv_rms<4>(g, m0, BM, s_inv);
    }

    // operand reads.  A: row r, k-group kg at r * 64 + (kg ^ swz(r)) * 16 - at one k-group, eight rows in a row fall into all eight 16-byte
    // columns of 128 bytes and sixteen into all sixteen of 256.  B: as packed, contiguous.
    unsigned a_at[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) a_at[c] = (wm * TM * 32 + lrow) * 64 + ((2 * c + lg) ^ swz(lrow)) * 16;
    // first panel of column tile j
    const int half_tiles = EPI == EPI_QKV ? g.rope.kv.head_dim >> 6 : 1;      // QKV: 32-column tiles in half a head (1 or 2)
    auto tile_panel = [&](int j) {
        if (EPI == EPI_SWIGLU) return wn * 2 + j * (BN / 32);
        if (EPI == EPI_QKV) return ((wn / half_tiles) * 2 * half_tiles + wn % half_tiles + j * half_tiles) * 2;   // j = 0, 1: the halves of a head
        return (wn * TN + j) * 2;
    };
    unsigned b_at[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) b_at[j] = A_BYTES + (tile_panel(j) + (lrow >> 4)) * 1024 + lg * 256 + (lrow & 15) * 16;

    // Fragments of the stage's two MFMA steps (16 k each) live in two register sets: the reads of the next step are issued ahead of the
    // products of the current one.  A stage's second step reads ahead into the next stage, so that is where the stages change: by
    // then every read of the current buffer has been issued, and (lgkmcnt) come back.
    f16x8 fa[2][NA][TM], fb[2][TN];
    auto read = [&](int set, const char* st, int c) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[set][j] = *(const f16x8*)(st + b_at[j] + c * 512);
#pragma unroll
        for (int p = 0; p < NA; ++p)
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[set][p][i] = *(const f16x8*)(st + a_at[c] + p * BM * 64 + i * 2048);
    };
    auto multiply = [&](int set) {
#pragma unroll
        for (int p = 0; p < NA; ++p)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[set][p][i], fb[set][j], acc[i][j], 0, 0, 0);
    };
    constexpr int READS = NA * TM + TN, PRODUCTS = NA * TM * TN;
    auto interleave = [&]() {                                // one product between two reads
#pragma unroll
        for (int k = 0; k < READS; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        if (PRODUCTS > READS) __builtin_amdgcn_sched_group_barrier(0x008, PRODUCTS - READS, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto stage = [&](int s) { return smem + (s % S) * STAGE; };

    auto first_step = [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
        read(1, stage(s), 1);
        multiply(0);
        interleave();
    };
    if (nsteps >= S) wait_copies_and_sync<(S - 2) * L>(); else wait_copies_and_sync<0>();
    read(0, stage(0), 0);
    if (S - 1 < nsteps) load_stage(S - 1, S - 1);
    int s = 0;
    for (; s + S < nsteps; ++s) {
        first_step(s);
        wait_copies_and_sync<(S - 2) * L>();                 // stage s + 1 has landed for everybody, nobody reads stage s any more
        load_stage(s + S, s % S);
        read(0, stage(s + 1), 0);
        multiply(1);
        interleave();
    }
    for (; s < nsteps; ++s) {
        first_step(s);
        if (s + 1 < nsteps) {
            wait_copies_and_sync<0>();
            read(0, stage(s + 1), 0);
        }
        multiply(1);
    }

    auto row_of = [&](int i, int r) { return (wm * TM + i) * 32 + (r >> 2) * 8 + lg * 4 + (r & 3); };
    const bool odd = lane & 1;
    auto col_of = [&](int j) { return n0 + (EPI == EPI_SWIGLU ? wn * 32 : tile_panel(j) * 16) + lrow; };

    if constexpr (SLICED) {                                  // raw products of this K slice: its own slab
        const long long ld = EPI == EPI_SWIGLU ? 2 * N : N;
        float* __restrict__ C = g.split_ws + (long long)kz * M * ld;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int m = m0 + row_of(i, r), n = col_of(j);
                    if (m < M && n < N) C[m * ld + (EPI == EPI_SWIGLU ? j * N : 0) + n] = acc[i][j][r];
                }
    } else if constexpr (EPI == EPI_STORE_F32) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = row_of(i, r), m = m0 + row;
                const float inv = g.ssq ? s_inv[row] : 1.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int n = col_of(j);
                    if (m < M && n < N) g.Cf[(long long)m * N + n] = acc[i][j][r] * inv;
                }
            }
    } else if constexpr (EPI == EPI_SWIGLU) {
        f16* __restrict__ out = (f16*)g.C16;
        const int n = col_of(0) & ~1;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                float h[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float inv = g.ssq ? s_inv[row_of(i, r + q)] : 1.0f, ga = acc[i][0][r + q] * inv;
                    h[q] = silu_lean(ga) * (acc[i][1][r + q] * inv);
                }
                const int m = m0 + row_of(i, r + odd);
                const f32x2 v = pair_of_columns(h[0], h[1], odd);
                if (m < M && n < N) store_split2(out + (long long)m * N + n, g.c_lo_off, v);
            }
    } else if constexpr (EPI == EPI_RESIDUAL) {              // N % 64 == 0: a wavefront's columns are all there or none of them
        f16* __restrict__ a16 = (f16*)g.C16;
        float gain[TN];
        const bool live_n = col_of(0) < N;
#pragma unroll
        for (int j = 0; j < TN; ++j) gain[j] = g.gain_next ? (float)((const bf16*)g.gain_next)[min(col_of(j), N - 1)] : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float xv[TN][16], ss[16];
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < TN; ++j) xv[j][r] = g.Cf[(long long)min(m0 + row_of(i, r), M - 1) * N + min(col_of(j), N - 1)];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + row_of(i, r);
                ss[r] = 0.f;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    xv[j][r] += acc[i][j][r];
                    ss[r] += xv[j][r] * xv[j][r];
                    if (m < M && live_n) g.Cf[(long long)m * N + col_of(j)] = xv[j][r];
                }
            }
            if (g.gain_next) {
#pragma unroll
                for (int r = 0; r < 16; r += 2) {
                    const int m = m0 + row_of(i, r + odd);
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const f32x2 v = pair_of_columns(xv[j][r] * gain[j], xv[j][r + 1] * gain[j], odd);
                        if (m < M && live_n) store_split2(a16 + (long long)m * N + (col_of(j) & ~1), g.c_lo_off, v);
                    }
                }
            }
            if (g.gain_next) {                               // partial sums of squares over the wavefront's TN * 32 columns
                const float t = rows16_sum(ss, lane);
                const int m = m0 + row_of(i, lrow >> 1);
                if ((lrow & 1) == 0 && m < M && live_n) g.ssq_out[(long long)m * (N / (TN * 32)) + n0 / (TN * 32) + wn] = t;
            }
        }
    } else {                                                 // EPI_QKV: tiles j = 0, 1 are the two halves of 32 rotary pairs
        const RopeArgs& ro = g.rope;
        const int hd = ro.kv.head_dim, half = hd >> 1, Hq = ro.n_q_heads, Hkv = ro.kv.n_kv_heads;
        const int n = col_of(0), head = n / hd, ch = n - head * hd;          // head: wavefront-uniform
        f16* pool = (f16*)ro.kv.base;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float cs[16], sn[16];
            int slot[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = min(m0 + row_of(i, r), M - 1);
                slot[r] = ro.row_slot[m];
                const long long ao = (long long)ro.row_pos[m] * half + ch;
                cs[r] = ro.cos[ao];
                sn[r] = ro.sin[ao];
            }
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                float a[2], b[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float inv = g.ssq ? s_inv[row_of(i, r + q)] : 1.0f;
                    a[q] = acc[i][0][r + q] * inv;
                    b[q] = acc[i][1][r + q] * inv;
                }
                if (head < Hq + Hkv) {
                    const f32x2 v0 = pair_of_columns(a[0] * cs[r] - b[0] * sn[r], a[1] * cs[r + 1] - b[1] * sn[r + 1], odd);
                    const f32x2 v1 = pair_of_columns(b[0] * cs[r] + a[0] * sn[r], b[1] * cs[r + 1] + a[1] * sn[r + 1], odd);
                    const int m = m0 + row_of(i, r + odd);
                    if (m >= M || n >= N) continue;
                    f16* dst = head < Hq ? (f16*)ro.q_out + ((long long)m * Hq + head) * hd
                                         : pool + ro.kv.plane(ro.layer, 0, head - Hq) + (long long)(odd ? slot[r + 1] : slot[r]) * hd;
                    const long long lo_off = head < Hq ? g.c_lo_off : 0;     // q may be split; the cache holds one fp16 per entry
                    store_split2(dst + (ch & ~1), lo_off, v0);
                    store_split2(dst + (ch & ~1) + half, lo_off, v1);
                } else {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        if (m0 + row_of(i, r + q) >= M || n >= N) continue;
                        const int sl = slot[r + q];
                        f16* dst = pool + ro.kv.plane(ro.layer, 1, head - Hq - Hkv) + (long long)(sl >> 4) * 16 * hd + (sl & 15);
                        dst[(long long)ch * 16] = (f16)a[q];
                        dst[(long long)(ch + half) * 16] = (f16)b[q];
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------ planning
// Tile shapes and their times in microseconds, fitted (to 4 %) to the four GEMMs of seven decoder layers (d_model 2048-5120, plain and split
// activations) at 27 row counts from 257 to 4096, every shape and slice count: over these the plan's choice is 0.2-0.7 % off the
// fastest.  A block's step is 32 k.
struct BlockShape {
    int bm, bn, capacity;             // capacity: blocks that run at once
    float epilogue;                   // a fused epilogue, as a share of the 256 x 256 block's
    struct Times {
        float lo, half, full;         // a step with few blocks at work, with one on every CU (128 x 128: two run on a CU), at capacity
        float fixed;                  // a block's prologue and end
        float padding;                // share of the time that rows past M cost (they re-read the last row: L2 hits)
        float tail;                   // what a partial round behind whole ones takes of its time alone
    } plain, split;
};
static constexpr BlockShape kShapes[] = {
    {256, 256, 256, 1.00f, {0.54f, 0.f, 0.836f, 3.0f, 0.79f, 1.f}, {0.97f, 0.f, 1.62f, 3.7f, 0.87f, 1.f}},
    {128, 256, 256, 0.49f, {0.41f, 0.f, 0.505f, 2.4f, 0.44f, 1.f}, {0.49f, 0.f, 0.836f, 2.9f, 0.74f, 1.f}},
    {128, 128, 512, 0.38f, {0.257f, 0.321f, 0.58f, 2.75f, 0.42f, 0.85f}, {0.416f, 0.576f, 0.984f, 2.3f, 0.53f, 0.95f}},
};

// QKV slabs much beyond the L2s are slow to add up (the K and V of the sum are scattered into pages): 5120 x 7168 at 3072 rows, two slices
// of 88 MB, 311 us, whole 251.  (Residual slabs pay up to 280 MB: 13824 x 5120 at 3520 rows, four slices 542 us, whole 641.)
static constexpr size_t kMaxQkvSlabs = 96u << 20;

float gemm_reduce_us(Epilogue epi, int M, int N, int ks) {
    const float mb = M * (float)N * 4e-6f;
    return epi == EPI_QKV ? 4.7f + (0.287f * ks + 0.306f) * mb : 3.f + (0.371f * ks + 0.226f) * mb;
}

float gemm_partials_us(int M) { return std::min(4e-3f * M, 7.f); }

BlockPlan plan_gemm_block(Epilogue epi, int M, int N, int K, bool split, size_t ws_bytes) {
    BlockPlan best{-1, 1, 0.f};
    for (int c = 0; c < 3; ++c) {
        const BlockShape& s = kShapes[c];
        const BlockShape::Times& t = split ? s.split : s.plain;
        const int on = epi == EPI_SWIGLU ? s.bn / 2 : s.bn, gy = (M + s.bm - 1) / s.bm;
        if (epi == EPI_SWIGLU && c == 2) continue;           // gate and up of 64 columns: not built
        for (int ks = 1; ks <= 4; ++ks) {
            if (ks > 1 && (epi == EPI_STORE_F32 || epi == EPI_SWIGLU || K % (32 * ks) != 0 || K / ks < 512 ||
                           (size_t)ks * M * N * sizeof(float) > (epi == EPI_QKV ? std::min(ws_bytes, kMaxQkvSlabs) : ws_bytes)))
                continue;
            const long long blocks = (long long)((N + on - 1) / on) * gy * ks, rounds = blocks / s.capacity, rest = blocks % s.capacity;
            // (QKV: 2 us less than fitted - in a model the residual GEMM before it is mostly sliced, which leaves fewer partial sums of x^2 to read)
            const float steps = K / ks / 32, end = t.fixed + (ks > 1 ? 0.f : s.epilogue * (epi == EPI_SWIGLU ? 11.f : 27.f) - (epi == EPI_QKV ? 2.f : 0.f));
            float us = rounds * (t.full * steps + end);
            if (rest) {
                const float step = s.capacity == 256 ? t.lo + (t.full - t.lo) * rest / 256
                                   : rest <= 256     ? t.lo + (t.half - t.lo) * rest / 256 : t.full;
                us += (step * steps + end) * (rounds ? t.tail : 1.f);
            }
            us *= t.padding + (1.f - t.padding) * M / (gy * s.bm);
            us += ks > 1 ? gemm_reduce_us(epi, M, N, ks) : epi == EPI_RESIDUAL ? gemm_partials_us(M) : 0.f;
            if (best.shape < 0 || us < best.us) best = {c, ks, us};
        }
    }
    return best;
}

template <int EPI, int TM, int TN, int WM, int WN, int S, bool SPLIT, bool SLICED>
static void launch_tiles(const GemmArgs& g, hipStream_t s) {
    constexpr int BM = WM * TM * 32, ON = EPI == EPI_SWIGLU ? WN * TN * 16 : WN * TN * 32;
    const int gx = (g.N + ON - 1) / ON, gy = (g.M + BM - 1) / BM;
    gemm_block_kernel<EPI, TM, TN, WM, WN, S, SPLIT, SLICED><<<gx * gy * (SLICED ? g.ksplit : 1), 64 * WM * WN, 0, s>>>(g, gx, gy, gy < 8 ? gy : 8);
}
template <int EPI, bool SPLIT, bool SLICED>
static void launch_shape(const GemmArgs& g, int shape, hipStream_t s) {
    if (shape == 0) launch_tiles<EPI, 4, 2, 2, 4, SPLIT ? 3 : 4, SPLIT, SLICED>(g, s);
    else if (shape == 1) launch_tiles<EPI, 2, 2, 2, 4, 4, SPLIT, SLICED>(g, s);
    else if constexpr (EPI != EPI_SWIGLU) launch_tiles<EPI, 2, 2, 2, 2, SPLIT ? 3 : 4, SPLIT, SLICED>(g, s);
}

template <int EPI>
static int launch_block(const GemmArgs& g, const BlockPlan& p, hipStream_t s) {
    const bool split = g.a_lo_off != 0;
    if constexpr (EPI == EPI_RESIDUAL || EPI == EPI_QKV) {
        if (p.ks > 1) {
            GemmArgs gs = g;
            gs.ksplit = p.ks;
            if (split) launch_shape<EPI_RESIDUAL, true, true>(gs, p.shape, s);       // raw products: one kernel for both epilogues
            else launch_shape<EPI_RESIDUAL, false, true>(gs, p.shape, s);
            if (EPI == EPI_RESIDUAL) return launch_residual_reduce(gs, s);
            launch_qkv_reduce(gs, s);
            return 0;
        }
    }
    GemmArgs g1 = g;
    g1.ksplit = 1;
    if (split) launch_shape<EPI, true, false>(g1, p.shape, s);
    else launch_shape<EPI, false, false>(g1, p.shape, s);
    return EPI == EPI_RESIDUAL ? g.N / 64 : 0;
}

int launch_gemm_block(Epilogue epi, const GemmArgs& g, const BlockPlan& p, hipStream_t s) {
    switch (epi) {
        case EPI_STORE_F32: return launch_block<EPI_STORE_F32>(g, p, s);
        case EPI_RESIDUAL: return launch_block<EPI_RESIDUAL>(g, p, s);
        case EPI_SWIGLU: return launch_block<EPI_SWIGLU>(g, p, s);
        default: return launch_block<EPI_QKV>(g, p, s);
    }
}

int launch_gemm_block_as(Epilogue epi, const GemmArgs& g, int rows, int cols, int slices, hipStream_t s) {
    return launch_gemm_block(epi, g, {rows == 256 ? 0 : cols == 256 ? 1 : 2, slices, 0.f}, s);
}

}  // namespace ax
