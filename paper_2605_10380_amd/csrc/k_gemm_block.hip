// GEMMs of many rows (bf16-weight models): C = A[M,K] * W[N,K]^T on the fp16 matrix cores, both operands staged through LDS by
// the memory pipeline itself (global_load_lds: no registers, no ds_write in between), blocks of up to 256 x 256 outputs.
//
// What bounds it: power.  With all compute units at work the clock sinks until the matrix cores' energy fits (8192 x 8192 x 8192: 1324 TFLOP/s
// on random values at 1.65 GHz, 1764 on zeros at 2.35, the same instructions; profiles/block_gemm_8192_power.txt), so what counts is energy
// and idle clocks around the products.
//   * 4 wavefronts of 128 x 128 outputs: a third fewer LDS reads per product than 8 of 128 x 64, whose reads and copies together also
//     took every clock that LDS has.  One wavefront per SIMD has nobody to fill its gaps, so the order of its instructions is written
//     out: one LDS read or copy at most between two products, 32 clocks each.  (4096 x 16384 x 2048, store of fp16: 264 us on 8
//     wavefronts, 228 on 4; the same loop in the compiler's order was no faster than 8 wavefronts.)
//   * A in panels: 16 rows x 32 k are 1 KB in one piece, in rows 16 half lines of 128 bytes.
//   * Stages of 32 k, up to four in LDS, so that the copies of three steps are in flight: with two stages of 64 k the queue of outstanding
//     lines ran dry between a stage's arrival and the issue of the next one.
//   * SwiGLU and QKV multiply transposed (C^T: a lane is a row, its registers neighbouring columns): 1 / rms is one value a lane, and eight
//     columns leave as 16 bytes, which in panels are whole lines.
//   * 1 / rms of the rows: a thread sums a row's partial sums, which panels keep [part][row].  (In rows, half a wavefront a row and a butterfly:
//     SwiGLU of ~1B at 4096 rows 285 us a launch, so 239.)
//   * Smaller tiles (128 x 256, 128 x 128) move 1.5x / 2x the operands per product; they are for launches that would leave CUs without a
//     block, and where two on a CU hide the epilogue (the planner at the end weighs tile and K-slice choices by measured times).
#include "gemm_device.h"
#include "lds_copy.h"

#include <algorithm>
#include <type_traits>

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

// f(0), f(1), .. f(N - 1) with the numbers as types (a loop this long is not unrolled, and accumulators indexed by its counter would go to memory).
template <int N, class F>
__device__ __forceinline__ void for_each(F f) {
    if constexpr (N > 0) {
        for_each<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Two quads of columns (registers 8 p .. 8 p + 3 and + 4 .. + 7 of a transposed accumulator, packed to fp16) of one row, of which lanes l and
// l + 32 hold four columns each: afterwards the lane holds all eight of quad 2 p + lane / 32, 16 bytes that lie together in memory.
__device__ __forceinline__ u32x4 eight_columns(const f16x4 (&q)[2]) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 a = __builtin_bit_cast(u32x2, q[0]), b = __builtin_bit_cast(u32x2, q[1]);
    u32x4 out;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const auto t = __builtin_amdgcn_permlane32_swap(a[d], b[d], false, false);
        out[d] = t[0];
        out[2 + d] = t[1];
    }
    return out;
}
// Eight fp32 values of a lane (columns as above) -> fp16 at p, and their lo parts lo_off elements behind.
__device__ __forceinline__ void store_eight(f16* p, long long lo_off, const float (&v)[8]) {
    f16x4 hi[2], lo[2];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const float x = split_value(v[r]);
        hi[r >> 2][r & 3] = (f16)x;
        lo[r >> 2][r & 3] = (f16)(x - (float)hi[r >> 2][r & 3]);
    }
    const u32x4 h = eight_columns(hi);
    if (p) *(u32x4*)p = h;
    if (lo_off) {
        const u32x4 l = eight_columns(lo);
        if (p) *(u32x4*)(p + lo_off) = l;
    }
}

// EPI: the epilogue (GemmArgs).  TM x TN tiles of 32 x 32 outputs per wavefront, WM x WN wavefronts, S stages in LDS.
// SPLIT: split activations - hi and lo parts of A are staged and multiplied against the same B fragments.
// SLICED: K is cut into g.ksplit slices over extra blocks; raw products go to slabs of g.split_ws.
// Blocks are renumbered: XCD c (workgroups are dealt out round robin) takes the c-th eighth of the tiles, in groups of `group` row tiles
// walked column by column, so that the ~32 tiles an XCD works on at a time share operands in its L2.
template <int EPI, int TM, int TN, int WM, int WN, int S, int OCC, bool SPLIT, bool SLICED>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_block_kernel(GemmArgs g, int gx, int gy, int group) {
    constexpr int NW = WM * WN, BM = WM * TM * 32, BN = WN * TN * 32, BK = 32, NA = SPLIT ? 2 : 1;
    constexpr int A_BYTES = NA * BM * 64, B_BYTES = BN * 64, STAGE = A_BYTES + B_BYTES;
    constexpr int LA = NA * BM / 16 / NW, LB = BN / 16 / NW, L = LA + LB;      // copies per wavefront and stage
    static_assert(NA * BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "whole copies per wavefront");
    static_assert(TN % 2 == 0, "column tiles come in pairs: gate and up, the halves of a head, 64 columns of x");
    constexpr int OUT_N = EPI == EPI_SWIGLU ? BN / 2 : BN;
    constexpr bool TRANSPOSED = !SLICED && (EPI == EPI_SWIGLU || EPI == EPI_QKV);      // accumulators hold C^T: a lane is a row of C
    __shared__ __attribute__((aligned(1024))) char smem[S * STAGE];
    __shared__ float s_inv[BM];

    const int M = g.M, N = g.N, K = g.K;
    // (strips: calls of up to 256 rows, which only come here with hi + lo parts)
    const bool in_panels = g.a_layout != ACT_ROWS, strips = SPLIT && g.a_layout == ACT_STRIPS;
    const ActLayout c_layout = SPLIT || g.c_layout != ACT_STRIPS ? g.c_layout : ACT_ROWS;
    auto out_index = [&](int m, int n) {                         // (plain activations never leave here in strips)
        if constexpr (SPLIT) return act_index(c_layout, m, n, g.M, g.N);
        else return act_index_few(c_layout != ACT_ROWS, m, n, g.M, g.N);
    };
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
    // copies of this wavefront: A units of 16 rows x 32 k, B units of one chunk of a panel (1 KB as packed).
    // A as rows: lane l copies slot l % 4 of row l / 4; slot s of row r holds k-group s ^ swz(r): see the operand reads.
    // A in panels or strips (act_index): the unit is a chunk, copied as it lies; rows a short last panel does not have are its last one again.
    auto swz = [](int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); };
    unsigned a_off[LA];
    const char* a_ptr[LA];
    int a_step[LA];                                          // bytes from one stage to the next
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int unit = wave * LA + i, part = unit / (BM / 16), u = unit % (BM / 16);
        const char* base = (const char*)g.A + (SPLIT && part ? g.a_lo_off * 2 : 0);
        if (in_panels) {
            const int panel = min((m0 >> 4) + u, (M - 1) >> 4), rows = strips ? 16 : min(16, M - panel * 16);
            a_step[i] = strips ? ((M + 15) >> 4) * 1024 : rows * 64;
            a_ptr[i] = base + (strips ? (long long)panel * 1024 : (long long)panel * 32 * K) + (long long)(kbase >> 5) * a_step[i];
            a_off[i] = (unsigned)((lane >> 4) * rows + min(lane & 15, rows - 1)) * 16u;
        } else {
            const int row = u * 16 + (lane >> 2);
            a_step[i] = 64;
            a_ptr[i] = base + ((long long)m0 * K + kbase) * 2;
            a_off[i] = (unsigned)min(row, M - 1 - m0) * (unsigned)K * 2u + (unsigned)(((lane & 3) ^ swz(row)) * 16);
        }
    }
    const char* b_ptr[LB];
    unsigned b_off = (unsigned)lane * 16;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int pl = wave * LB + i;                                  // panel of the stage
        const bool second = EPI == EPI_SWIGLU && pl >= BN / 32;
        const int panel = min((n0 >> 4) + (second ? pl - BN / 32 : pl), (N >> 4) - 1);
        b_ptr[i] = (const char*)(second ? g.W2 : g.W) + ((long long)panel * 16 * K + (long long)kbase * 16) * 2;
    }
    // copy i of this wavefront for the next stage not copied yet, into buffer `buf`.  The offsets move on in vector registers, one addition
    // beside each copy of A and one for B: scalar pointers, advanced together, were 20 instructions in a row behind the last product.
    auto copy = [&](int buf, int i) {
        const unsigned at = lds0 + buf * STAGE;
        if (i < LA) {
            copy_to_lds(a_ptr[i], a_off[i], at + (wave * LA + i) * 1024);
            a_off[i] += a_step[i];
            asm volatile("" : "+v"(a_off[i]));               // (here, not with the others at the loop's end)
        } else {
            copy_to_lds(b_ptr[i - LA], b_off, at + A_BYTES + (wave * LB + i - LA) * 1024);
            if (i == L - 1) b_off += 1024;
        }
    };

    const int nsteps = kspan / BK;
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < nsteps)
#pragma unroll
            for (int i = 0; i < L; ++i) copy(s, i);
    const bool inv_here = g.ssq && !SLICED;
    if (inv_here) {
        if (in_panels) block_inv_rms_panels(g, m0, BM, s_inv);
        else if (g.nparts <= 4) block_inv_rms_few(g, m0, BM, s_inv);
        else block_inv_rms<16>(g, m0, BM, s_inv);
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // the large tiles' accumulators stay in accumulation registers from here to the epilogue (left alone, the compiler moves all of them
    // to ordinary ones and back between the loops)
    auto pin = [&]() {
        if constexpr (OCC == 1) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
    };

    // operand reads.  A as rows: row r, k-group kg at r * 64 + (kg ^ swz(r)) * 16 - at one k-group, eight rows in a row fall into all eight
    // 16-byte columns of 128 bytes and sixteen into all sixteen of 256.  B, and A in panels: as packed, contiguous.
    unsigned a_at[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
        a_at[c] = wm * TM * 2048 + (in_panels ? (lrow >> 4) * 1024 + (2 * c + lg) * 256 + (lrow & 15) * 16 : lrow * 64 + ((2 * c + lg) ^ swz(lrow)) * 16);
    // column tile j of the wavefront, as a tile of the stage: j and j + 1 are gate and up, or the halves of a head
    const int half_tiles = EPI == EPI_QKV ? g.rope.kv.head_dim >> 6 : 1;      // QKV: 32-column tiles in half a head (1 or 2)
    auto tile_of = [&](int j) {
        if (EPI == EPI_SWIGLU) return (j & 1) * (BN / 64) + wn * (TN / 2) + (j >> 1);
        if (EPI == EPI_QKV && half_tiles == 2) return TN == 4 ? wn * 4 + (j >> 1) + (j & 1) * 2 : (wn >> 1) * 4 + (wn & 1) + j * 2;
        return wn * TN + j;
    };
    unsigned b_at[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) b_at[j] = A_BYTES + (tile_of(j) * 2 + (lrow >> 4)) * 1024 + lg * 256 + (lrow & 15) * 16;

    // A stage is two MFMA steps of 16 k; the fragments of the step being multiplied and of the one after it live in two register sets.
    // One wavefront per SIMD: what it issues is in this order and nothing fills a gap, so reads (and, in a stage's first step, the
    // copies of the stage S - 1 ahead) go one by one between products, 32 clocks apart.  A stage's second step reads from the
    // next stage, so that is where the stages change: by then the reads of the current one have come back (lgkmcnt).
    f16x8 fb[2][TN], fa[2][NA * TM];
    constexpr int READS = NA * TM + TN, PRODUCTS = NA * TM * TN;
    auto read = [&](int set, const char* st, int c, int i) {
        if (i < TN) fb[set][i] = *(const f16x8*)(st + b_at[i] + c * 512);
        else fa[set][i - TN] = *(const f16x8*)(st + a_at[c] + (i - TN) / TM * BM * 64 + (i - TN) % TM * 2048);
    };
    auto product = [&](int set, int q) {                     // columns back and forth: every product keeps one operand of the one before
        const int p = q / (TM * TN), i = q / TN % TM, j = i & 1 ? TN - 1 - q % TN : q % TN;
        if constexpr (TRANSPOSED) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[set][j], fa[set][p * TM + i], acc[i][j], 0, 0, 0);
        else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[set][p * TM + i], fb[set][j], acc[i][j], 0, 0, 0);
    };
    auto step = [&](auto with_copies, int set, const char* next, int c, int copy_buf) {     // products of `set`, reads of the other one, copies
        constexpr bool COPIES = decltype(with_copies)::value;
#pragma unroll
        for (int q = 0; q < PRODUCTS; ++q) {
            __builtin_amdgcn_sched_barrier(0);
            if (q < READS) read(set ^ 1, next, c, q);
            if constexpr (COPIES) {
#pragma unroll
                for (int i = 0; i < L; ++i)
                    if ((2 * i + 1) * PRODUCTS / (2 * L) == q) {
                        __builtin_amdgcn_sched_barrier(0);
                        copy(copy_buf, i);
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
            product(set, q);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    static_assert(READS <= PRODUCTS, "a read per product");
    constexpr std::true_type copies{};
    constexpr std::false_type no_copies{};
    auto after = [](int buf) { return buf + 1 == S ? 0 : buf + 1; };

    pin();
    if (nsteps >= S - 1) wait_copies_and_sync<(S - 2) * L>(); else wait_copies_and_sync<0>();
#pragma unroll
    for (int i = 0; i < READS; ++i) read(0, smem, 0, i);
    __builtin_amdgcn_s_waitcnt(0xc07f);                      // (with a scalar load still out, the loop's first product would wait for every read)
    __builtin_amdgcn_sched_barrier(0);
    int s = 0, buf = 0, done = S - 1;                        // done: the buffer of step s - 1, which nobody reads any more
    for (; s + S - 1 < nsteps; ++s) {
        step(copies, 0, smem + buf * STAGE, 1, done);
        done = buf;
        buf = after(buf);
        wait_copies_and_sync<(S - 2) * L>();                 // step s + 1 has landed for everybody, step s has been read
        step(no_copies, 1, smem + buf * STAGE, 0, 0);
    }
    pin();
    for (; s < nsteps; ++s) {
        step(no_copies, 0, smem + buf * STAGE, 1, 0);
        buf = after(buf);
        wait_copies_and_sync<0>();
        step(no_copies, 1, smem + buf * STAGE, 0, 0);        // (the last one reads a buffer nobody needs, and its values go unused)
    }
    pin();

    // products as they are (C): register r of a lane is row row_of(i, r), column col_of(j)
    auto row_of = [&](int i, int r) { return (wm * TM + i) * 32 + (r >> 2) * 8 + lg * 4 + (r & 3); };
    const bool odd = lane & 1;
    auto col_of = [&](int j) { return n0 + tile_of(j) * 32 + lrow; };

    if constexpr (SLICED) {                                  // raw products of this K slice: its own slab
        float* __restrict__ C = g.split_ws + (long long)kz * M * N;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int m = m0 + row_of(i, r), n = col_of(j);
                    if (m < M && n < N) C[(long long)m * N + n] = acc[i][j][r];
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
    } else if constexpr (EPI == EPI_RESIDUAL) {              // N % 64 == 0: a pair of column tiles is there or it is not
        f16* __restrict__ a16 = (f16*)g.C16;
        float gain[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) gain[j] = g.gain_next ? (float)((const bf16*)g.gain_next)[min(col_of(j), N - 1)] : 0.f;
        for_each<TM>([&](auto i_) {
            for_each<TN / 2>([&](auto jp_) {
                constexpr int i = decltype(i_)::value, jp = 2 * decltype(jp_)::value;
                const bool live_n = col_of(jp) < N;
                float xv[2][16], ss[16];
#pragma unroll
                for (int r = 0; r < 16; ++r)
#pragma unroll
                    for (int j = 0; j < 2; ++j) xv[j][r] = g.Cf[(long long)min(m0 + row_of(i, r), M - 1) * N + min(col_of(jp + j), N - 1)];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = m0 + row_of(i, r);
                    ss[r] = 0.f;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        xv[j][r] += acc[i][jp + j][r];
                        ss[r] += xv[j][r] * xv[j][r];
                        if (m < M && live_n) g.Cf[(long long)m * N + col_of(jp + j)] = xv[j][r];
                    }
                }
                if (g.gain_next) {
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        const int m = m0 + row_of(i, r + odd);
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const f32x2 v = pair_of_columns(xv[j][r] * gain[jp + j], xv[j][r + 1] * gain[jp + j], odd);
                            if (m < M && live_n) store_split2(a16 + out_index(m, col_of(jp + j) & ~1), g.c_lo_off, v);
                        }
                    }
                    const float t = rows16_sum(ss, lane);    // partial sums of squares over the 64 columns
                    const int m = m0 + row_of(i, lrow >> 1);
                    const int part = (n0 + tile_of(jp) * 32) / 64;
                    if ((lrow & 1) == 0 && m < M && live_n) g.ssq_out[ssq_index(ssq_by_part(c_layout, M), m, part, M, N / 64)] = t;
                }
            });
        });
    } else if constexpr (EPI == EPI_SWIGLU) {                // C^T: a lane is row lrow of tile i, registers are columns (r / 4) * 8 + lg * 4 + r % 4
        f16* __restrict__ out = (f16*)g.C16;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = (wm * TM + i) * 32 + lrow, m = m0 + row;
            const float inv = g.ssq ? s_inv[row] : 1.0f;
#pragma unroll
            for (int j = 0; j < TN; j += 2) {
                const int nt = n0 + tile_of(j) * 32;
                if (nt >= N) continue;
#pragma unroll
                for (int r = 0; r < 16; r += 8) {
                    float h[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) h[q] = silu_lean(acc[i][j][r + q] * inv) * (acc[i][j + 1][r + q] * inv);
                    store_eight(m < M ? out + out_index(m, nt + r * 2 + lg * 8) : nullptr, g.c_lo_off, h);
                }
            }
        }
    } else {                                                 // EPI_QKV, C^T: tiles j and j + 1 are the two halves of 32 rotary pairs
        const RopeArgs& ro = g.rope;
        const int hd = ro.kv.head_dim, half = hd >> 1, Hq = ro.n_q_heads, Hkv = ro.kv.n_kv_heads;
        f16* pool = (f16*)ro.kv.base;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = (wm * TM + i) * 32 + lrow, m = m0 + row, mc = min(m, M - 1);
            const float inv = g.ssq ? s_inv[row] : 1.0f;
            const int slot = ro.row_slot[mc];
            const long long angle = (long long)ro.row_pos[mc] * half;
#pragma unroll
            for (int j = 0; j < TN; j += 2) {
                const int nt = n0 + tile_of(j) * 32, head = nt / hd, ch0 = nt - head * hd;      // wavefront-uniform
                if (nt >= N) continue;
                if (head < Hq + Hkv) {
                    f16* dst = head < Hq ? (f16*)ro.q_out + ((long long)m * Hq + head) * hd
                                         : pool + ro.kv.plane(ro.layer, 0, head - Hq) + (long long)slot * hd;
                    const long long lo_off = head < Hq ? g.c_lo_off : 0;     // q may be split; the cache holds one fp16 per entry
#pragma unroll
                    for (int r = 0; r < 16; r += 8) {
                        float va[8], vb[8];
#pragma unroll
                        for (int q4 = 0; q4 < 8; q4 += 4) {
                            const int ch = ch0 + (r + q4) * 2 + lg * 4;
                            const f32x4 cs = *(const f32x4*)(ro.cos + angle + ch), sn = *(const f32x4*)(ro.sin + angle + ch);
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const float a = acc[i][j][r + q4 + q] * inv, b = acc[i][j + 1][r + q4 + q] * inv;
                                va[q4 + q] = a * cs[q] - b * sn[q];
                                vb[q4 + q] = b * cs[q] + a * sn[q];
                            }
                        }
                        f16* at = m < M ? dst + ch0 + r * 2 + lg * 8 : nullptr;
                        store_eight(at, lo_off, va);
                        store_eight(at ? at + half : nullptr, lo_off, vb);
                    }
                } else if (m < M) {
                    f16* dst = pool + ro.kv.plane(ro.layer, 1, head - Hq - Hkv) + (long long)(slot >> 4) * 16 * hd + (slot & 15);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int ch = ch0 + (r >> 2) * 8 + lg * 4 + (r & 3);
                        dst[(long long)ch * 16] = (f16)(acc[i][j][r] * inv);
                        dst[(long long)(ch + half) * 16] = (f16)(acc[i][j + 1][r] * inv);
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------ planning
// 128 x 256 blocks of plain activations, more of them than CUs: two on a CU (three stages of LDS each), so that one's epilogue runs under the
// other's products (~1B at 4096 rows, SwiGLU 285 us one on a CU, 247 two; ~3B QKV at 4666 rows 156 and 145, in 256 x 256 blocks 166).
// With no more than a CU each the fourth stage is worth more (2048 x 8192 at 4096 rows: 118 us, with three stages 127).
static bool two_on_a_cu(long long blocks, bool split) { return blocks > 256 && !split; }

// Tile shapes and their times in microseconds, a block's step being 32 k.  Up to 512 rows, where launches are one round or a part of one: kernel
// times inside models of 4-12 layers, fitted to the four GEMMs of 19 decoder layers (d_model 192-5120, plain and split activations), every
// shape and slice count at 27 row counts from 257 to 1024, and the logits of 5 matrices; forms near the fastest and layers of 2048
// and wider weigh most (half of the forms within 25 % of the fastest are within 3 % of it).  More rows, all in panels, whole rounds at the
// clock that power leaves: the three GEMM classes of layers of 2048-4096 at 21 row counts from 257 to 4666.
struct BlockShape {
    int bm, bn, capacity;             // capacity: blocks that run at once
    struct Times {
        struct { float swiglu, store, qkv, residual, slab; } end;      // a block's prologue and end: fused epilogues, raw products to a slab
        float lo, half, full;         // a step with few blocks at work, with one on every CU (two run on a CU), at capacity
        float padding;                // share of the time that rows past M cost (they re-read the last row: L2 hits)
        float tail;                   // what a partial round behind whole ones takes of its time alone
        float crowd;                  // raw products of two blocks on a CU, as a multiple of one's alone
    } times[3][2];                    // [A in rows; in panels, up to 512 rows; more][split]
};
static constexpr int kBlockShapes = 4;                       // 3: 128 x 256, two on a CU with three stages each (plain activations)
static constexpr int kFewRounds = 512;
static constexpr BlockShape kShapes[kBlockShapes] = {
    {256, 256, 256,
     {{{{11.3f, 17.f, 20.f, 45.f, 14.3f}, 0.381f, 0.f, 0.883f, 0.73f, 1.f, 1.f},
       {{13.5f, 20.f, 21.f, 50.f, 14.4f}, 0.667f, 0.f, 1.558f, 0.85f, 1.03f, 1.f}},
      {{{11.3f, 17.f, 20.f, 45.f, 14.3f}, 0.297f, 0.f, 0.79f, 0.9f, 1.05f, 1.f},
       {{13.5f, 20.f, 21.f, 50.f, 14.4f}, 0.525f, 0.f, 1.505f, 0.9f, 1.01f, 1.f}},
      {{{7.8f, 20.2f, 20.2f, 20.2f, 10.5f}, 0.419f, 0.f, 0.755f, 0.97f, 0.98f, 1.f},
       {{6.4f, 18.8f, 18.8f, 18.8f, 9.1f}, 0.809f, 0.f, 1.538f, 0.94f, 0.9f, 1.f}}}},
    {128, 256, 256,
     {{{{7.5f, 8.f, 11.f, 23.f, 8.6f}, 0.341f, 0.f, 0.55f, 0.5f, 0.96f, 1.f},
       {{8.8f, 9.5f, 13.6f, 24.2f, 9.f}, 0.391f, 0.f, 0.852f, 0.68f, 1.05f, 1.f}},
      {{{7.8f, 8.3f, 11.4f, 23.9f, 8.9f}, 0.263f, 0.f, 0.483f, 0.9f, 0.97f, 1.f},
       {{9.2f, 9.9f, 14.1f, 25.2f, 9.4f}, 0.338f, 0.f, 0.817f, 0.9f, 1.02f, 1.f}},
      {{{8.6f, 13.1f, 13.1f, 13.1f, 7.4f}, 0.278f, 0.f, 0.411f, 0.95f, 0.77f, 1.f},
       {{9.5f, 14.f, 14.f, 14.f, 8.3f}, 0.42f, 0.f, 0.738f, 0.91f, 0.95f, 1.f}}}},
    {128, 128, 512,
     {{{{0.f, 5.6f, 7.5f, 11.9f, 5.4f}, 0.222f, 0.353f, 0.582f, 0.56f, 0.95f, 1.59f},
       {{0.f, 6.f, 9.f, 12.1f, 5.5f}, 0.366f, 0.583f, 0.94f, 0.56f, 0.96f, 1.49f}},
      {{{0.f, 5.7f, 7.7f, 12.1f, 5.5f}, 0.169f, 0.319f, 0.473f, 0.9f, 1.01f, 1.55f},
       {{0.f, 6.1f, 9.2f, 12.3f, 5.6f}, 0.271f, 0.527f, 0.794f, 0.9f, 1.05f, 1.43f}},
      {{{3.9f, 5.4f, 5.4f, 5.4f, 5.f}, 0.222f, 0.27f, 0.485f, 0.71f, 0.87f, 1.f},
       {{1.f, 2.5f, 2.5f, 2.5f, 2.1f}, 0.361f, 0.479f, 0.932f, 0.77f, 0.99f, 1.f}}}},
    {128, 256, 512,
     {{{{6.2f, 6.f, 9.6f, 22.f, 7.8f}, 0.418f, 0.586f, 0.974f, 0.68f, 0.91f, 1.37f},
       {}},
      {{{6.4f, 6.2f, 9.9f, 22.7f, 8.f}, 0.332f, 0.553f, 0.844f, 0.9f, 1.05f, 1.28f},
       {}},
      {{{2.8f, 3.f, 3.f, 3.f, 6.3f}, 0.268f, 0.468f, 0.877f, 0.57f, 0.98f, 1.f},
       {}}}}};

// QKV slabs much beyond the L2s are slow to add up (the K and V of the sum are scattered into pages): 5120 x 7168 at 3072 rows, two slices
// of 88 MB, 311 us, whole 251.  (Residual slabs pay up to 280 MB: 13824 x 5120 at 3520 rows, four slices 542 us, whole 641.)
static constexpr size_t kMaxQkvSlabs = 96u << 20;

float gemm_reduce_us(Epilogue epi, int M, int N, int ks, bool panels) {
    const float mb = M * (float)N * 4e-6f;
    if (panels && M > kFewRounds) return epi == EPI_QKV ? 1.9f + (0.141f * ks + 0.15f) * mb : 2.4f + (0.145f * ks + 0.344f) * mb;
    if (epi == EPI_QKV) return 3.2f + (0.13f * ks + 0.15f) * mb;
    return panels ? 4.f + (0.122f * ks + 0.3f) * mb : 4.1f + (0.088f * ks + 0.215f) * mb;
}

float gemm_partials_us(int M, bool panels) { return !panels ? std::min(3e-3f * M, 4.f) : M > kFewRounds ? std::min(1e-3f * M, 2.f) : 0.5f; }

BlockPlan plan_gemm_block(Epilogue epi, int M, int N, int K, bool split, bool panels, size_t ws_bytes) {
    BlockPlan best{-1, 1, 0.f};
    const bool few = panels && M <= kFewRounds;
    for (int c = 0; c < (split ? 3 : 4); ++c) {
        const BlockShape& s = kShapes[c];
        const BlockShape::Times& t = s.times[!panels ? 0 : few ? 1 : 2][split];
        const float fused = epi == EPI_SWIGLU ? t.end.swiglu : epi == EPI_STORE_F32 ? t.end.store : epi == EPI_QKV ? t.end.qkv : t.end.residual;
        const int on = epi == EPI_SWIGLU ? s.bn / 2 : s.bn, gy = (M + s.bm - 1) / s.bm;
        if (epi == EPI_SWIGLU && c == 2) continue;           // gate and up of 64 columns: not built
        for (int ks = 1; ks <= 4; ++ks) {
            if (ks > 1 && (epi == EPI_STORE_F32 || epi == EPI_SWIGLU || K % (32 * ks) != 0 || K / ks < 512 ||
                           (size_t)ks * M * N * sizeof(float) > (epi == EPI_QKV ? std::min(ws_bytes, kMaxQkvSlabs) : ws_bytes)))
                continue;
            const long long blocks = (long long)((N + on - 1) / on) * gy * ks, rounds = blocks / s.capacity, rest = blocks % s.capacity;
            // two on a CU: in rows only whole (raw products gained nothing anywhere: ~3B QKV, O and down at 640-1024 rows 0-20 % behind)
            if (c == 3 && !panels && ks > 1) continue;
            if ((c == 1 || c == 3) && (panels || ks == 1) && two_on_a_cu(blocks, split) != (c == 3)) continue;
            // (slices are for CUs without a block: ~3B QKV in hi + lo parts, 320 rows, four slices on 480 blocks 40.2 us, two on 240 33.6)
            if (few && c == 2 && ks > 1 && blocks > 256) continue;
            const float steps = K / ks / 32, end = ks > 1 ? t.end.slab : fused, crowd = ks > 1 ? t.crowd : 1.f;
            float us = rounds * (t.full * steps + crowd * end);
            if (rest) {
                const float step = s.capacity == 256 ? t.lo + (t.full - t.lo) * rest / 256
                                   : rest <= 256     ? t.lo + (t.half - t.lo) * rest / 256 : t.full;
                us += (step * steps + (rest > 256 ? crowd : 1.f) * end) * (rounds ? t.tail : 1.f);
            }
            us *= t.padding + (1.f - t.padding) * M / (gy * s.bm);
            us += ks > 1 ? gemm_reduce_us(epi, M, N, ks, panels) : epi == EPI_RESIDUAL ? gemm_partials_us(M, panels) : 0.f;
            if (few) us *= 1.f + 0.015f * (ks - 1);          // of forms that come out alike, more slices were mostly the slower ones
            if (best.shape < 0 || us < best.us) best = {c, ks, us};
        }
    }
    return best;
}

template <int EPI, int TM, int TN, int WM, int WN, int S, int OCC, bool SPLIT, bool SLICED>
static void launch_tiles(const GemmArgs& g, hipStream_t s) {
    constexpr int BM = WM * TM * 32, ON = EPI == EPI_SWIGLU ? WN * TN * 16 : WN * TN * 32;
    const int gx = (g.N + ON - 1) / ON, gy = (g.M + BM - 1) / BM;
    gemm_block_kernel<EPI, TM, TN, WM, WN, S, OCC, SPLIT, SLICED><<<gx * gy * (SLICED ? g.ksplit : 1), 64 * WM * WN, 0, s>>>(g, gx, gy, gy < 8 ? gy : 8);
}
template <int EPI, bool SPLIT, bool SLICED>
static void launch_shape(const GemmArgs& g, int shape, hipStream_t s) {
    if (shape == 0) launch_tiles<EPI, 4, 4, 2, 2, SPLIT ? 3 : 4, 1, SPLIT, SLICED>(g, s);
    else if (shape == 1) launch_tiles<EPI, 2, 4, 2, 2, 4, 1, SPLIT, SLICED>(g, s);
    else if (shape == 3) {
        if constexpr (!SPLIT) launch_tiles<EPI, 2, 4, 2, 2, 3, 2, false, SLICED>(g, s);
    }
    else if constexpr (EPI != EPI_SWIGLU) launch_tiles<EPI, 2, 2, 2, 2, SPLIT ? 3 : 4, 2, SPLIT, SLICED>(g, s);
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
    const int out = epi == EPI_SWIGLU ? cols / 2 : cols, blocks = (g.N + out - 1) / out * ((g.M + rows - 1) / rows) * slices;
    return launch_gemm_block(epi, g, {rows == 256 ? 0 : cols == 128 ? 2 : two_on_a_cu(blocks, g.a_lo_off != 0) ? 3 : 1, slices, 0.f}, s);
}

}  // namespace ax
