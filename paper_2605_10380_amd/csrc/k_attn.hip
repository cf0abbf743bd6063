// Causal "extend" attention over the paged KV cache (grouped-query attention): the T new rows
// of a sequence attend to the P cached positions and to each other; row at position p sees
// keys 0..p (prefix caching relies on exactly this causality, paper Sec. 2.3).
//
//   * attn_f32_kernel: the fp32 models' path, fp32 matrix instructions, any even head_dim up to 256.
//   * attn_split_kernel + attn_combine_kernel: 16-bit path on the matrix cores (fp16 q, K, V and
//     probabilities, fp32 accumulation; used by bf16-weight models).  The query rows
//     of the G heads that share one KV head are stacked into one matrix (row = t*G + g), cut
//     into tiles of 32 rows; one block of 1 or 4 wavefronts owns (tile, KV head, slice of the key range), each wavefront
//     streams its share of the slice from the pages straight into MFMA operand registers with an online
//     softmax per row; the block adds them up in LDS and writes an unnormalised partial (O, m, l); the combine
//     kernel merges the slices.  Splitting the key range is what fills 256 CUs when T is small (verify:
//     T = 1 + k) and it is harmless when T is large.
#include "kernels.h"
#include "lds_copy.h"

#include <type_traits>

namespace ax {

typedef _Float16 f16;      // activation and KV-cache type of bf16-weight models
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------ fp32 kernel
// fp32 models: everything on the fp32 matrix instruction (16x16x4), one block per tile of 16 stacked rows (t * G + g) and
// KV head; its NW wavefronts take every NW-th page of 16 keys with their own online softmax and meet in LDS at the end,
// so a call of a few rows still keeps NW chains of page loads in flight and needs no second kernel.  (A wavefront
// per (row, query head) walking its keys 64 at a time took 137 us on a 5-row step over 512 keys; this takes 12 us.)
//
// S^T = K * Q^T per page: lane l supplies slot l % 16 of the page (and stacked row l % 16 of q) at channels 16 c +
// 4 * (l / 16) .. + 3 - one float4, element j for instruction j, the same order of channels on both sides - and receives
// the scores of keys 4 * (l / 16) .. + 3 for stacked row l % 16.  That is the B operand of O^T = V^T * P^T as it
// stands: V pages are token-minor, so the matching A operand (channel l % 16 of a 16-channel tile, keys 4 * (l / 16) .. + 3)
// is one float4 as well.
//
// HDT: 16-channel tiles the registers hold (head_dim <= 16 * HDT; channels past head_dim are zeros).
// FULL: head_dim is 16 * HDT; operands of the next page are then asked for while this one's are used (AHEAD below).  Other head_dims test every load
// against it, and the tests between the products cost more than that hides: they load a page where they use it (2 layers' attention, ahead / not:
// head_dim 32, 16 rows over 80 / 528 keys 7.0 / 6.5 and 13.1 / 12.2 us, 96 over 576 15.1 / 14.0, 192 over 528 56.8 / 53.9).
// OT: 16-channel tiles of the OUTPUT that the block computes (blockIdx.z: which).  A call of a few rows leaves most of the chip idle,
// and on the one CU that its block runs on the products of 33 pages alone take 4.4 us.  With a block per 16 output channels each CU does the
// scores again but only its part of the second product, of the V loads and of the merge.  5 rows over 517 keys: 13.3 -> 11.6 us,
// with the loads ahead of the products (below) and the merge's weights worked out once instead of by every wavefront.
template <int HDT, int OT, int NW, bool FULL>
__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(const float* __restrict__ q, float* __restrict__ out, KVGeom kv, int layer,
                                                           const int* __restrict__ tile_info, const int* __restrict__ bt, int Hq,
                                                           int subs) {
    __shared__ __attribute__((aligned(16))) f32x4 s_o[NW][OT][64];
    __shared__ float s_m[NW][16], s_l[NW][16], s_w[NW][16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int hd = kv.head_dim, Hkv = kv.n_kv_heads, G = Hq / Hkv, hk = blockIdx.y;
    const int* ti = tile_info + (blockIdx.x / subs) * 8;         // a record covers subs tiles of 16 rows
    const int4 ti0 = *(const int4*)ti, ti1 = *(const int4*)(ti + 4);
    const int P = ti0.z, T = ti0.w, row0 = ti1.x, r0 = ti0.y + (int)(blockIdx.x % subs) * 16, n_stacked = T * G, c0 = blockIdx.z * OT;
    if (r0 >= n_stacked) return;                                 // the record's last tiles may lie past the sequence's rows
    const int* tab = bt + ti1.y;
    const int kv_len = P + T;

    const int rq = min(r0 + lr, n_stacked - 1), tq = rq / G, pos_q = P + tq;
    const float* qrow = q + ((long long)(row0 + tq) * Hq + hk * G + rq % G) * hd;
    const float* Kp = (const float*)kv.base + kv.plane(layer, 0, hk);
    const float* Vp = (const float*)kv.base + kv.plane(layer, 1, hk);
    const bool vec = (hd & 3) == 0;
    auto load_row = [&](const float* row, int c) {               // channels 16 c + 4 lg .. + 3 of a row of hd channels
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        const int ch = c * 16 + lg * 4;
        if (FULL) {
            v = *(const f32x4*)(row + ch);
        } else if (vec) {
            if (ch < hd) v = *(const f32x4*)(row + ch);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) if (ch + i < hd) v[i] = row[ch + i];
        }
        return v;
    };
    f32x4 qf[HDT];
#pragma unroll
    for (int c = 0; c < HDT; ++c) qf[c] = load_row(qrow, c);

    const float scale = 1.0f / sqrtf((float)hd);
    float m = -INFINITY, l = 0.f;                                // l: this lane's keys only, summed over the lanes at the end
    f32x4 o[OT];
#pragma unroll
    for (int c = 0; c < OT; ++c) o[c] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int r_last = min(r0 + 15, n_stacked - 1);
    const int pages = (P + r_last / G + 16) >> 4;                // up to the page of the tile's last visible key
    // AHEAD: page ids of up to 64 of this wavefront's pages at a time; K of its next page is asked for behind this one's scores, V behind its output, in the
    // same registers: one chain of loads less a page, and the loop stays one body (with a second one for a second set of operands the
    // instruction fetches cost more than the loads it hid, 12.9 -> 15.6 us)
    constexpr bool AHEAD = FULL;
    const int mine = wave < pages ? (pages - wave + NW - 1) / NW : 0;
    int ids = 0;
    auto page_id = [&](int i) {
        if ((i & 63) == 0) ids = tab[min(wave + NW * (i + lane), pages - 1)];
        return __builtin_amdgcn_readlane(ids, i & 63);
    };
    f32x4 kf[HDT], vf[OT];
    auto load_k = [&](int blk) {
        const float* kp = Kp + ((long long)blk * 16 + lr) * hd;
#pragma unroll
        for (int c = 0; c < HDT; ++c) kf[c] = load_row(kp, c);
    };
    auto load_v = [&](int blk) {
        const float* vp = Vp + (long long)blk * 16 * hd + lg * 4;
#pragma unroll
        for (int c = 0; c < OT; ++c) {
            if (!FULL) vf[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (FULL || c * 16 + lr < hd) vf[c] = *(const f32x4*)(vp + ((c0 + c) * 16 + lr) * 16);
        }
    };
    int blk = 0;
    if (AHEAD && mine > 0) {
        blk = page_id(0);
        load_k(blk);
        load_v(blk);
    }
    for (int i = 0; i < mine; ++i) {
        const int kv0 = (wave + i * NW) * 16;
        if constexpr (!AHEAD) {
            blk = tab[wave + i * NW];
            load_k(blk);
            load_v(blk);
        } else if (i + 1 < mine) {
            blk = page_id(i + 1);                                // (the last page's again at the end: no branch around the loads)
        }
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};     // two chains of dependent products
#pragma unroll
        for (int c = 0; c < HDT; ++c) {
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][0], qf[c][0], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][1], qf[c][1], s1, 0, 0, 0);
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][2], qf[c][2], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][3], qf[c][3], s1, 0, 0, 0);
        }
        if constexpr (AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            load_k(blk);
            __builtin_amdgcn_sched_barrier(0);
        }
        float mx = -INFINITY;
        f32x4 p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = kv0 + lg * 4 + i <= pos_q ? (s0[i] + s1[i]) * scale : -INFINITY;
            mx = fmaxf(mx, p[i]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m, mx), mu = mn == -INFINITY ? 0.f : mn;  // nothing visible yet: exp(-inf) = 0 all the same
        const float alpha = expf(m - mu);
        l *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = expf(p[i] - mu);
            l += p[i];
        }
        m = mn;
        if (kv0 + 16 > kv_len) {                                 // slots past the sequence's end hold anything: exact zeros
#pragma unroll
            for (int c = 0; c < OT; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) if (kv0 + lg * 4 + i >= kv_len) vf[c][i] = 0.f;
        }
#pragma unroll
        for (int c = 0; c < OT; ++c) {
            o[c] *= alpha;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][i], p[i], o[c], 0, 0, 0);
        }
        if constexpr (AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            load_v(blk);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (lg == 0) { s_m[wave][lr] = m; s_l[wave][lr] = l; }
#pragma unroll
    for (int c = 0; c < OT; ++c) s_o[wave][c][lane] = o[c];
    __syncthreads();
    if (threadIdx.x < 16 * NW) {                                 // one (wavefront, row) per thread: its weight and its part of the row's sum
        const int w = threadIdx.x >> 4;
        float M = s_m[0][lr];
#pragma unroll
        for (int j = 1; j < NW; ++j) M = fmaxf(M, s_m[j][lr]);   // finite: every row sees key 0
        const float e = expf(s_m[w][lr] - M);
        s_w[w][lr] = e;
        s_l[w][lr] *= e;
    }
    __syncthreads();
    // wavefront w finishes channel tiles w, w + NW, ..: register i of lane l is channel 4 * (l / 16) + i of stacked row l % 16
    if (wave >= OT || r0 + lr >= n_stacked) return;
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) L += s_l[w][lr];
    float* orow = out + ((long long)(row0 + tq) * Hq + hk * G + rq % G) * hd;
    for (int c = wave; c < OT; c += NW) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) v += s_w[w][lr] * s_o[w][c][lane];
        const int ch = (c0 + c) * 16 + lg * 4;
        if (FULL) {
            *(f32x4*)(orow + ch) = v / L;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) if (ch + i < hd) orow[ch + i] = v[i] / L;
        }
    }
}

// ------------------------------------------------------------------------------ MFMA split kernel
// One block = one (q tile of 32 stacked rows, KV head, key slice).
//
// S^T = K * Q^T is computed so that the score tile comes out with lane <-> query row
// (column l % 32) and registers <-> keys: register r of lane l is key (r/4)*8 + (l/32)*4 + r%4
// of the 32-key step.  Row max / sum therefore need the 16 registers of the lane plus one
// exchange with lane ^ 32, and the softmax rescale is a per-lane scalar.  The probabilities
// are already laid out as the B operand of O^T = V^T * P^T: registers 0..7 cover keys
// {4g..4g+3, 8+4g..8+4g+3} of the first 16-key block, registers 8..15 the same of the second
// block (g = l/32).  V pages are token-minor ([head_dim][16]), so the matching A operand of a
// lane (channel d) is two 8-byte loads from its channel's 16-token row.
// One 32-key step of the online softmax for the lane's query row.  s: raw scores q.k of the
// lane's 16 keys (key of register r: kv0 + (r/4)*8 + g*4 + r%4); c = log2(e)/sqrt(hd).  m is the
// reference exponent of the row (scaled, base-2 domain), l the running sum of 2^(s*c - m) over the
// LANE's keys (the caller adds l of lane and lane ^ 32 when it is done).  The
// reference is NOT kept equal to the running maximum: it is only raised when some row of the
// wavefront has a score more than SOFTMAX_SLACK above it (then every row moves to its current
// maximum, the function returns true and the caller multiplies its output accumulators by
// alpha).  In between, probabilities may exceed 1 by at most 2^SOFTMAX_SLACK, far inside the
// range of fp16 operands and fp32 sums, and the per-step rescale of the accumulators - as much
// vector work as the exponentials themselves - runs a handful of times per row instead of on
// every step.  (m, l, o) stay mutually consistent, which is all the slice merge needs.
// The probabilities are packed to fp16 (round toward zero, one instruction per pair) as the two
// PV operands, and l sums exactly those packed values (dot product with ones), so the
// normalisation matches the weights the PV product really uses.  The causal mask is applied only
// on steps that reach past the tile's earliest row (`diagonal`, wavefront-uniform).  v_exp_f32
// is used directly: a result that underflows to 0 is exact enough for a probability.
constexpr float SOFTMAX_SLACK = 8.0f;
template <bool PAGES = false>          // key of register r: PAGES: kv0 + (r / 8) * 16 + g * 8 + r % 8 (block kernel)
__device__ __forceinline__ bool online_softmax_step(f32x16& s, int kv0, int g, int pos_q, bool diagonal, float c,
                                                    float& m, float& l, float& alpha, f16x8 (&pb)[2]) {
    if (diagonal) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int kj = PAGES ? kv0 + (r >> 3) * 16 + g * 8 + (r & 7) : kv0 + (r >> 2) * 8 + g * 4 + (r & 3);
            s[r] = (kj <= pos_q) ? s[r] : -INFINITY;
        }
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx *= c;                                                    // c > 0: max commutes with the scaling
    // mx covers the lane's 16 keys, i.e. half of its row's 32: the test below is the same over
    // half rows as over whole rows, so the two halves only meet (one cross-lane exchange) when the
    // reference really moves
    const bool raise = __any(mx > m + SOFTMAX_SLACK);           // m = -inf: any visible key raises it
    alpha = 1.0f;
    if (raise) {
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m, mx);
        alpha = (mn == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - mn);   // m = -inf -> 0
        l *= alpha;
        m = mn;
    }
    const float mu = (m == -INFINITY) ? 0.f : m;               // row with nothing visible yet
    const f16x2 ones = {(f16)1.0f, (f16)1.0f};
    float ps = 0.f;
    u32x4 pw[2];
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[r], c, -mu));       // masked: -inf -> 0
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[r + 1], c, -mu));
        const auto h = __builtin_amdgcn_cvt_pkrtz(p0, p1);
        ps = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, h), ones, ps, false);
        pw[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(unsigned, h);
    }
    pb[0] = __builtin_bit_cast(f16x8, pw[0]);
    pb[1] = __builtin_bit_cast(f16x8, pw[1]);
    l += ps;                                                    // the lane's half of the row; halves are added at the end
    return raise;
}

// Which (q-tile group, KV head, key slice) a workgroup works on.  Workgroups are dealt to the 8 XCDs round robin
// in launch order (x fastest), and each XCD has its own L2: with the plain blockIdx mapping the q-tile groups that
// read the SAME keys (same KV head, same slice) have consecutive ids and land on 8 different L2s, so every K/V
// byte crossed HBM once per group (measured 7.9x the cache's bytes on a 256-row extend, 2x on a verify step).
// Renumbered: XCD c takes the c-th eighth of the (head, slice, group) order, group fastest - all groups of one
// (head, slice) share one L2 and run at the same time, and so do the slices of one head, which all read that
// head's q rows (with 8 KV heads: one head per XCD; K, V and q each cross HBM once).
struct AttnWork { int tile, hk, split; };
__device__ __forceinline__ AttnWork attn_work(unsigned id, unsigned nx, unsigned ny, unsigned nz) {
    const unsigned total = nx * ny * nz;                                             // nz: a power of two (choose_splits)
    if ((total & 7u) == 0) id = (id & 7u) * (total >> 3) + (id >> 3);
    const unsigned rest = id / nx;
    return {(int)(id - rest * nx), (int)(rest >> __builtin_ctz(nz)), (int)(rest & (nz - 1))};
}
// r / G for stacked rows of the split kernel (r < 2^20: a step away from the next integer is more than the rounding of two fp32 operations)
__device__ __forceinline__ int row_of_stacked(int r, float inv_g) { return (int)((r + 0.5f) * inv_g); }

// A tile record (StepView::tile_info): wavefront-uniform and not written while a kernel runs, so one scalar load.
typedef int i32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ i32x8 tile_record(const int* info, int tile) {
    return *(const __attribute__((address_space(4))) i32x8*)(info + tile * 8);
}

struct AttnArgs {
    const f16* q;
    f16* out;
    long long q_lo_off, out_lo_off;   // split activations: lo parts of q / out this many elements behind (0 = not split)
    int n_rows;
    ActLayout out_layout;             // of out [n_rows, Hq * hd]
    KVGeom kv;
    int layer, Hq, G, n_splits;       // G: query heads per KV head; n_splits: a power of two
    const int* tile_info;      // 8 ints per q tile, item or merge record (see StepView)
    const int* bt;
    float* partials;
    // shared-prefix pass of a many-sequence call (see launch_attention); unused otherwise
    const float* shared_partials;
    int shared_splits, shared_len;
};
// Element (m, k) of the output: strips on a branch of their own, since the one formula for all layouts costs every store more.
__device__ __forceinline__ long long out_index(const AttnArgs& a, int m, int k) {
    if (a.out_layout == ACT_STRIPS) return act_index(ACT_STRIPS, m, k, a.n_rows, a.Hq * a.kv.head_dim);
    return act_index_few(a.out_layout == ACT_PANELS, m, k, a.n_rows, a.Hq * a.kv.head_dim);
}

// Everything a step needs from memory is requested as early as possible, because at verify
// sizes the kernel is a chain of dependent memory latencies, not a bandwidth problem: the tile
// record is one 32-byte load, the block-table entries of the whole key slice are fetched by
// one wavefront-wide load (and handed out with shuffles), and the K/V operands of step s + 1
// are in flight while step s is multiplied.
// NW = 4: the wavefronts of a block meet in LDS, so a wavefront's serial chain of key steps is a quarter of the slice while only one
// partial record per slice goes to memory and through the combine kernel.  Whole steps: ~8B verify over 8704 keys 4108 -> 4021 us, 16 ~3B
// sessions verified together 5359 -> 5162 us (~1B verify over 4352 keys 843 -> 826 us, no more than its runs differ).
// NW = 1: caches too short to give every CU such a block (~1B decode over 1301 keys: 727 us a step, 755 with NW = 4).
// QS: q comes as hi and lo parts (split activations): the score product takes both against the same K operand.
// wk: the block's work; lds: split_lds(HD, NW) bytes of LDS.
constexpr int split_lds(int hd, int nw) { return nw * ((nw > 1 ? hd / 8 : 1) * 1024 + 256); }
// AHEAD: a key step's operands have registers of their own while the step before is multiplied (one block on a CU); else K of the next step is
// asked for behind this one's scores and V behind its output, in the same registers (two blocks on a CU).
template <int HD, int NW, bool QS, bool AHEAD>
__device__ __forceinline__ void attn_split(const AttnArgs& a, AttnWork wk, char* lds) {
    constexpr int KQ = HD / 16;          // MFMA k-steps of the score product
    constexpr int NP = QS ? 2 : 1;
    constexpr int DT = HD / 32;          // 32-channel tiles of the output
    constexpr int PS = HD * 32 + 64;     // floats of one partial: O^T [HD][32], m[32], l[32]
    auto s_o = (f32x4(*)[NW > 1 ? DT * 4 : 1][64])lds;
    auto s_m = (float(*)[32])(lds + NW * (NW > 1 ? DT * 4 : 1) * 1024), s_l = s_m + NW;
    const int tile = wk.tile, hk = wk.hk, split = wk.split;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, ql = lane & 31, g = lane >> 5;
    const int Hq = a.Hq, Hkv = a.kv.n_kv_heads, G = a.G;
    const float inv_g = 1.0f / (float)G;
    const i32x8 ti = tile_record(a.tile_info, tile);
    const int r0 = ti[1], P = ti[2], T = ti[3], row0 = ti[4];
    const int n_stacked = T * G;
    const int* tab = a.bt + ti[5];
    const int kv_len = P + T, last_blk = (kv_len - 1) >> 4;

    // keys this group can see at all: up to the position of its last valid row.  (Keys past the end of the
    // sequence, reached only by its last step, re-read the last valid K row - see fetch - and their scores are
    // replaced by -inf, so K is never read from unwritten slots; V is, and process() zeroes those operands.)
    const int r_last = min(r0 + 31, n_stacked - 1);
    const int kv_end = P + row_of_stacked(r_last, inv_g) + 1;
    const int first = ti[7] >> 5;                        // first key step (keys before it belong to the shared pass)
    const int steps = (kv_end + 31) / 32;
    const int per = (steps - first + a.n_splits - 1) >> __builtin_ctz(a.n_splits);
    const int b_lo = first + split * per, b_hi = min(steps, b_lo + per);      // the block's key steps
    const int per_w = (max(b_hi - b_lo, 0) + NW - 1) / NW;
    const int s_lo = b_lo + wave * per_w, s_hi = min(b_hi, s_lo + per_w);     // this wavefront's (may be none)

    // this lane's query row (clamped rows compute garbage that is never written)
    const int rq = min(r0 + ql, n_stacked - 1), tq = row_of_stacked(rq, inv_g);
    const int pos_q = P + tq, pos_min = P + row_of_stacked(min(r0, n_stacked - 1), inv_g);       // pos_min: earliest position of the tile (uniform)
    const f16* qrow = a.q + ((long long)(row0 + tq) * Hq + hk * G + rq - tq * G) * HD;
    f16x8 qf[NP][KQ];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) qf[p][kk] = *(const f16x8*)(qrow + (p ? a.q_lo_off : 0) + kk * 16 + g * 8);

    const f16* Kp = (const f16*)a.kv.base + a.kv.plane(a.layer, 0, hk);
    const f16* Vp = (const f16*)a.kv.base + a.kv.plane(a.layer, 1, hk);

    const float c = 1.4426950408889634f / sqrtf((float)HD);   // log2(e) / sqrt(hd)
    float m = -INFINITY, l = 0.f;
    f32x16 o[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] = 0.f;

    f16x8 kf[AHEAD ? 2 : 1][KQ];         // K / V operands of the current and the next step
    f16x4 vq[AHEAD ? 2 : 1][DT][4];
    int tabv = 0;                        // block ids of steps [chunk, chunk + 32): lane i holds block 2*chunk + i
    auto fetch_k = [&](int buf, int st, int chunk) {
        const int kv0 = st * 32;
        const int key = min(kv0 + ql, kv_len - 1);
        const int kblk = __shfl(tabv, min(key >> 4, last_blk) - 2 * chunk, 64);
        const f16* krow = Kp + ((long long)kblk * 16 + (key & 15)) * HD + g * 8;
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) kf[buf][kk] = *(const f16x8*)(krow + kk * 16);
    };
    auto fetch_v = [&](int buf, int st, int chunk) {
        const int kv0 = st * 32;
        const int b0 = __shfl(tabv, min(kv0 >> 4, last_blk) - 2 * chunk, 64);
        const int b1 = __shfl(tabv, min((kv0 >> 4) + 1, last_blk) - 2 * chunk, 64);
#pragma unroll
        for (int d = 0; d < DT; ++d) {
            const f16* v0 = Vp + ((long long)b0 * HD + d * 32 + ql) * 16 + g * 4;
            const f16* v1 = Vp + ((long long)b1 * HD + d * 32 + ql) * 16 + g * 4;
            vq[buf][d][0] = *(const f16x4*)v0;
            vq[buf][d][1] = *(const f16x4*)(v0 + 8);
            vq[buf][d][2] = *(const f16x4*)v1;
            vq[buf][d][3] = *(const f16x4*)(v1 + 8);
        }
    };
    auto process = [&](int buf, int st, auto behind_scores) {
        const int kv0 = st * 32;
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk)
#pragma unroll
            for (int p = 0; p < NP; ++p) s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[buf][kk], qf[p][kk], s, 0, 0, 0);
        behind_scores();
        float alpha;
        f16x8 pb[2];
        if (online_softmax_step(s, kv0, g, pos_q, kv0 + 31 > pos_min, c, m, l, alpha, pb)) {
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
        }
        if (kv0 + 32 > kv_len) {
            // the sequence ends inside this step (its last one): slots of the last block past the end were never
            // written by this sequence and may hold anything - their V operands become exact zeros, so that a
            // probability of 0 times whatever lies in caller memory cannot turn into a NaN
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int qd = 0; qd < 4; ++qd)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (kv0 + qd * 8 + g * 4 + i >= kv_len) vq[buf][d][qd][i] = (f16)0.f;
        }
#pragma unroll
        for (int d = 0; d < DT; ++d) {
            const f16x4 *v = vq[buf][d];
            const f16x8 va = {v[0][0], v[0][1], v[0][2], v[0][3], v[1][0], v[1][1], v[1][2], v[1][3]};
            const f16x8 vb = {v[2][0], v[2][1], v[2][2], v[2][3], v[3][0], v[3][1], v[3][2], v[3][3]};
            o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, pb[0], o[d], 0, 0, 0);
            o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vb, pb[1], o[d], 0, 0, 0);
        }
    };

    for (int chunk = s_lo; chunk < s_hi; chunk += 32) {          // 32 steps = 64 blocks = one table load
        tabv = tab[min(2 * chunk + lane, last_blk)];
        const int c_hi = min(s_hi, chunk + 32);
        // (no fetch sits behind a branch that the products ahead of it do not share: the compiler then knows how many loads are out and
        // waits for one step's operands while the next one's stay in flight)
        auto issue = [&](int buf, int st) {
            fetch_k(buf, st, chunk);
            fetch_v(buf, st, chunk);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto nothing = [] {};
        issue(0, chunk);
        int st = chunk;
        if constexpr (!AHEAD) {
            for (; st + 1 < c_hi; ++st) {
                process(0, st, [&] {
                    __builtin_amdgcn_sched_barrier(0);
                    fetch_k(0, st + 1, chunk);
                    __builtin_amdgcn_sched_barrier(0);
                });
                __builtin_amdgcn_sched_barrier(0);
                fetch_v(0, st + 1, chunk);
                __builtin_amdgcn_sched_barrier(0);
            }
            process(0, st, nothing);
            continue;
        }
        for (; st + 2 < c_hi; st += 2) {
            issue(1, st + 1);
            process(0, st, nothing);
            issue(0, st + 2);
            process(1, st + 1, nothing);
        }
        if (st + 1 < c_hi) {
            issue(1, st + 1);
            process(0, st, nothing);
            process(1, st + 1, nothing);
        } else {
            process(0, st, nothing);
        }
    }

    // one (O^T, m, l) record per (tile, KV head, slice); rows past the end of the sequence are not written (and never read)
    float* part = a.partials + ((long long)(tile * Hkv + hk) * a.n_splits + split) * PS;
    if constexpr (NW == 1) {
        l += __shfl_xor(l, 32, 64);                              // both halves of each row
        if (r0 + ql >= n_stacked) return;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) part[(d * 32 + (r >> 2) * 8 + g * 4 + (r & 3)) * 32 + ql] = o[d][r];
        if (g == 0) {
            part[HD * 32 + ql] = m;
            part[HD * 32 + 32 + ql] = l;
        }
        return;
    }
    // the wavefronts' sums, brought to the block's largest reference exponent, meet in LDS
    l += __shfl_xor(l, 32, 64);                                  // both halves of each row
    if (g == 0) s_m[wave][ql] = m;
    __syncthreads();
    float M = s_m[0][ql];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w][ql]);
    const float scale = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);    // no visible key in this wavefront's steps: 0
    if (g == 0) s_l[wave][ql] = l * scale;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int r = 0; r < 16; r += 4)
            s_o[wave][d * 4 + (r >> 2)][lane] = (f32x4){o[d][r] * scale, o[d][r + 1] * scale, o[d][r + 2] * scale, o[d][r + 3] * scale};
    __syncthreads();
    if (r0 + ql >= n_stacked) return;
#pragma unroll
    for (int i = 0; i < DT * 4 / NW; ++i) {                      // a wavefront writes its share of the channels
        const int e = wave * (DT * 4 / NW) + i;                             // channels (e / 4) * 32 + (e % 4) * 8 + 4 g .. + 3
        f32x4 t = s_o[0][e][lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += s_o[w][e][lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) part[((e >> 2) * 32 + (e & 3) * 8 + g * 4 + q) * 32 + ql] = t[q];
    }
    if (wave == 0 && g == 0) {
        float t = s_l[0][ql];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += s_l[w][ql];
        part[HD * 32 + ql] = M;
        part[HD * 32 + 32 + ql] = t;
    }
}

template <int HD, int NW, bool QS>
__global__ __launch_bounds__(64 * NW) void attn_split_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[split_lds(HD, NW)];
    // all arguments in one round trip (left alone, the compiler fetches them where they are used)
    asm volatile("" :: "s"(a.q), "s"(a.q_lo_off), "s"(a.kv.base), "s"(a.kv.n_blocks), "s"(a.kv.n_kv_heads), "s"(a.layer), "s"(a.Hq), "s"(a.G), "s"(a.n_splits),
                       "s"(a.tile_info), "s"(a.bt), "s"(a.partials));
    attn_split<HD, NW, QS, true>(a, attn_work(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x, gridDim.y, gridDim.z), lds);
}

// ------------------------------------------------------------------------------ MFMA block kernel
// Long extends (many q tiles per KV head) and the shared-prefix pass: a block of NQ = 4 wavefronts owns 4 consecutive q tiles (128
// stacked rows) of one KV head and a range of key steps - one ITEM of the list the host planned (StepView::items).  The K and V pages of
// a 32-key step are copied to LDS by the memory pipeline (no registers in between), S stages deep, one barrier per step, and
// shared by the NQ tiles; everything after that is the per-wavefront online softmax of attn_split_kernel.  An item that
// holds all the keys of its tiles writes the attention output itself; the others leave (O, m, l) records for
// attn_merge_items_kernel.
//
// A key step is 32 keys = 2 pages: 4 * HD bytes of K and V each, copied in 1 KB units (wavefront w takes units w, w + NQ, ..).
//   K: [32 keys][HD]; the 16-byte columns of a row are rotated by swz(key) (which column a lane COPIES is free to choose, where it
//      lands is not), so that 16 keys at one column fall into all 16-byte columns of 256 bytes.
//   V: [2 pages][HD channels][16 tokens]; the two halves of a channel's 32 bytes trade places in every other group of 8 channels.
// The score product takes the keys in the order 0-3, 8-11, 4-7, 12-15 (of each page): then a lane ends up with the scores of
// keys 8 g .. 8 g + 7 of both pages (g = lane / 32), and its V operand is ONE 16-byte read.
constexpr int STAGES = 3;
// id: the block's number of n_items * KV heads, items first; smem: STAGES * 128 * HD bytes of LDS.
template <int HD, bool QS>
__device__ __forceinline__ void attn_block(const AttnArgs& a, unsigned id, unsigned nx, char* smem) {
    constexpr int NQ = 4, S = STAGES;
    constexpr int KQ = HD / 16, DT = HD / 32, PS = HD * 32 + 64;
    constexpr int NP = QS ? 2 : 1;                    // q in hi and lo parts (split activations)
    constexpr int KB = 32 * HD * 2, STAGE = 2 * KB;   // bytes of K (and of V) per step
    constexpr int U = STAGE / 1024, L = (U + NQ - 1) / NQ, PU = U / 4;      // copy units per step, per wavefront, per page of K or V
    static_assert(U % NQ == 0, "whole units per wavefront");
    const unsigned total = nx * (unsigned)a.kv.n_kv_heads;      // (see attn_work: with 8 KV heads, one head per XCD)
    if ((total & 7u) == 0) id = (id & 7u) * (total >> 3) + (id >> 3);
    const int item = (int)(id % nx), hk = (int)(id / nx);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, ql = lane & 31, g = lane >> 5;
    const int Hq = a.Hq, Hkv = a.kv.n_kv_heads, G = Hq / Hkv;
    const int4 ti0 = *(const int4*)(a.tile_info + item * 8), ti1 = *(const int4*)(a.tile_info + item * 8 + 4);
    const int slot = ti0.x, r0 = ti0.y, P = ti0.z, T = ti0.w, row0 = ti1.x, s_hi = ti1.z, s_lo = ti1.w;
    const int n_stacked = T * G;
    const int* tab = a.bt + ti1.y;
    const int kv_len = P + T, last_blk = min((kv_len - 1) >> 4, 2 * s_hi - 1);

    // this wavefront's q tile (a tile past the sequence's rows copies and synchronises with the others, nothing more)
    const bool idle = r0 + wave * 32 >= n_stacked;
    const int rq = min(r0 + wave * 32 + ql, n_stacked - 1);
    const int tq = rq / G, gq = rq % G;
    const int pos_q = P + tq;
    const f16* qrow = a.q + ((long long)(row0 + tq) * Hq + hk * G + gq) * HD;
    f16x8 qf[NP][KQ];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) qf[p][kk] = *(const f16x8*)(qrow + (p ? a.q_lo_off : 0) + kk * 16 + g * 8);

    const char* Kp = (const char*)((const f16*)a.kv.base + a.kv.plane(a.layer, 0, hk));
    const char* Vp = (const char*)((const f16*)a.kv.base + a.kv.plane(a.layer, 1, hk));
    const float c = 1.4426950408889634f / sqrtf((float)HD);
    const int pos_tile_min = P + min(r0 + wave * 32, n_stacked - 1) / G;       // earliest and latest position among this tile's rows
    const int pos_tile_max = P + min(r0 + wave * 32 + 31, n_stacked - 1) / G;
    float m = -INFINITY, l = 0.f;
    f32x16 o[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] = 0.f;

    // copies: unit x < U / 2 is K (page x / PU, part x % PU of it), the others V
    auto swz = [](int key) { return HD == 128 ? key & 15 : (key & 7) ^ ((key >> 3) & 1); };
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
    unsigned off[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int x = wave + NQ * i, part = x % PU;
        const int unit16 = part * 64 + lane;                   // 16-byte piece within the page, as it lies in LDS
        const int key = unit16 / (HD / 8), col = unit16 % (HD / 8), ch = unit16 >> 1, half = unit16 & 1;
        off[i] = x < U / 2 ? (unsigned)(key * HD * 2 + (col ^ swz(key)) * 16) : (unsigned)(ch * 32 + (half ^ ((ch >> 3) & 1)) * 16);
    }
    // page ids: lane i of tabv holds page 2 * tab_at + i, the pages of 32 steps; the next 64 are on their way in tabn
    int tab_at = s_lo, tabv = tab[min(2 * s_lo + lane, last_blk)], tabn = tab[min(2 * s_lo + 64 + lane, last_blk)];
    auto load_stage = [&](int buf, int st) {
        if (st - tab_at >= 32) {
            tab_at += 32;
            tabv = tabn;
            tabn = tab[min(2 * tab_at + 64 + lane, last_blk)];
        }
        const int rel = 2 * (st - tab_at), lim = last_blk - 2 * tab_at;       // table lanes of the step's two pages
        const int b0 = __builtin_amdgcn_readlane(tabv, min(rel, lim)), b1 = __builtin_amdgcn_readlane(tabv, min(rel + 1, lim));
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const int x = wave + NQ * i, page = (x / PU) & 1;
            const char* base = (x < U / 2 ? Kp : Vp) + (long long)(page ? b1 : b0) * 16 * HD * 2;
            copy_to_lds(base, off[i], lds0 + buf * STAGE + x * 1024);
        }
    };
    // operand addresses.  Score product: MFMA row i takes key i with bits 2 and 3 swapped
    const int key_of = (ql & 0x13) | ((ql & 4) << 1) | ((ql & 8) >> 1);
    const unsigned k_at = key_of * HD * 2 + ((g ^ swz(key_of & 15)) * 16);     // column 2 kk + g of the row: k_at ^ (kk * 32)
    const unsigned v_at = KB + ql * 32 + (g ^ ((ql >> 3) & 1)) * 16;

    auto process = [&](const char* stg, int st) {
        const int kv0 = st * 32;
        if (idle || kv0 > pos_tile_max) return;                // none of the tile's rows sees these keys
        // K operands are requested four products ahead and half of the V operands before the softmax, the other half behind it (what the
        // registers of three wavefronts per SIMD hold): left alone, the compiler keeps two reads in flight
        f16x8 kf[4], v0[DT], v1[DT];
        unsigned ka = k_at;
        asm volatile("" : "+v"(ka));                         // (one xor per read instead of eight registers for the addresses)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) kf[kk] = *(const f16x8*)(stg + (ka ^ (kk * 32)));
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < NP; ++p) s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[kk & 3], qf[p][kk], s, 0, 0, 0);
            if (kk + 4 < KQ) kf[kk & 3] = *(const f16x8*)(stg + (ka ^ ((kk + 4) * 32)));
        }
#pragma unroll
        for (int d = 0; d < DT; ++d) v0[d] = *(const f16x8*)(stg + v_at + d * 1024);
        __builtin_amdgcn_sched_barrier(0);
        float alpha;
        f16x8 pb[2];
        if (online_softmax_step<true>(s, kv0, g, pos_q, kv0 + 31 > pos_tile_min, c, m, l, alpha, pb)) {
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < DT; ++d) v1[d] = *(const f16x8*)(stg + v_at + HD * 32 + d * 1024);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < DT; ++d) o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v0[d], pb[0], o[d], 0, 0, 0);
#pragma unroll
        for (int d = 0; d < DT; ++d) o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v1[d], pb[1], o[d], 0, 0, 0);
    };

    const int n = s_hi - s_lo;
#pragma unroll
    for (int u = 0; u < S - 1; ++u)
        if (u < n) load_stage(u, s_lo + u);
    int i = 0;
    for (; i + 2 * S - 2 < n; i += S) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
            wait_copies_and_sync<(S - 2) * L>();                 // step i + u has landed for everybody, nobody reads step i + u - 1 any more
            load_stage((u + S - 1) % S, s_lo + i + u + S - 1);
            process(smem + u * STAGE, s_lo + i + u);
        }
    }
    for (; i < n; i += S) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
            if (i + u >= n) break;
            wait_copies_and_sync<0>();
            if (i + u + S - 1 < n) load_stage((u + S - 1) % S, s_lo + i + u + S - 1);
            const int left = kv_len - (s_lo + i + u) * 32;       // keys from the step's first one to the sequence's end
            if (left < 32) {
                // the sequence ends inside this step (its last one): the slots behind hold whatever the pool memory held - exact
                // zeros instead, so that their probability of 0 cannot meet a NaN or an infinity
                for (int x = tid; x < 2 * HD; x += 64 * NQ) {
                    const int ch = x % HD, page = x / HD;
                    char* at = smem + u * STAGE + KB + page * HD * 32 + ch * 32;
                    for (int t = max(left - page * 16, 0); t < 16; ++t)
                        *(f16*)(at + (((t >> 3) ^ ((ch >> 3) & 1)) * 16) + (t & 7) * 2) = (f16)0.f;
                }
                __syncthreads();
            }
            process(smem + u * STAGE, s_lo + i + u);
        }
    }

    const float l_row = l + __shfl_xor(l, 32, 64);               // both halves of the row
    if (r0 + wave * 32 + ql >= n_stacked) return;
    if (slot < 0) {
        const float inv = 1.0f / l_row;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                f16* dst = a.out + out_index(a, row0 + tq, (hk * G + gq) * HD + d * 32 + r * 2 + g * 4);
                f16x4 hi, lo;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = split_value(o[d][r + q] * inv);
                    hi[q] = (f16)v;
                    lo[q] = (f16)(v - (float)hi[q]);
                }
                *(f16x4*)dst = hi;
                if (a.out_lo_off) *(f16x4*)(dst + a.out_lo_off) = lo;
            }
        return;
    }
    float* part = a.partials + (((long long)slot * Hkv + hk) * NQ + wave) * PS;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ch = d * 32 + (r >> 2) * 8 + g * 4 + (r & 3);
            part[ch * 32 + ql] = o[d][r];
        }
    if (g == 0) {
        part[HD * 32 + ql] = m;
        part[HD * 32 + 32 + ql] = l_row;
    }
}

template <int HD, bool QS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HD == 64 ? (QS ? 3 : 4) : (QS ? 2 : 3))))
void attn_block_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(1024))) char smem[STAGES * 128 * HD];
    attn_block<HD, QS>(a, blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, smem);
}

// The shared-prefix pass of a many-sequence call and the private keys of its sequences in one launch: blocks of the former first, one on every CU, the
// latter beside them.  The pass is bound by its products and the private keys by memory (16 sessions of the ~3B shape over 6144 shared and 1024-2048
// private keys: 21.1 and 26.8 us one after the other, 38.9 together; with half as many records of the shared keys, on blocks of 4 tiles instead of 8, the
// merge takes 8.2 instead of 12.6).
template <int HD, bool QS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void attn_shared_kernel(AttnArgs sh, AttnArgs a, int items, int tiles) {
    constexpr int PASS = STAGES * 128 * HD, OWN = split_lds(HD, 4);
    __shared__ __attribute__((aligned(1024))) char lds[PASS > OWN ? PASS : OWN];
    const unsigned heads = (unsigned)a.kv.n_kv_heads, n = (unsigned)items * heads;
    if (blockIdx.x < n) attn_block<HD, QS>(sh, blockIdx.x, (unsigned)items, lds);
    else attn_split<HD, 4, QS, false>(a, attn_work(blockIdx.x - n, (unsigned)tiles, heads, (unsigned)a.n_splits), lds);
}

// Merges the key slices of one q tile.  grid (n_tiles * Hkv, HD / 4), 256 threads =
// 32 query rows x 8 slice groups; a block produces 4 output channels.  A thread loads the
// (m, l, 4 channels) of its slices s = sg, sg + 8, ... in one go (up to 16 slices in registers),
// the row maximum and then the weighted sums meet in LDS.  With a shared-prefix pass the slices
// of that pass follow the tile's own: they live in the records of the shared pass's tile group
// that holds the row (rows of all sequences stacked: global row * G + g).
template <int HD>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnArgs a) {
    constexpr int PS = HD * 32 + 64;
    constexpr int MAXS = 16;                                   // slices per thread held in registers
    __shared__ float red[8][6][32];
    // (all arguments in one round trip, as in attn_split_kernel)
    asm volatile("" :: "s"(a.out), "s"(a.out_lo_off), "s"(a.n_rows), "s"((int)a.out_layout), "s"(a.kv.n_kv_heads), "s"(a.Hq), "s"(a.G), "s"(a.n_splits),
                       "s"(a.tile_info), "s"(a.partials), "s"(a.shared_splits));
    const int Hkv = a.kv.n_kv_heads, G = a.G;
    const int hk = blockIdx.x % Hkv, tile = blockIdx.x / Hkv;
    const int ch0 = blockIdx.y * 4;
    const int ql = threadIdx.x & 31, sg = threadIdx.x >> 5;
    const i32x8 ti = tile_record(a.tile_info, tile);
    const int row0 = ti[4], r_first = ti[1], n_stacked = ti[3] * G;
    if (r_first >= n_stacked) return;                          // whole q tile past the end (block-uniform)
    const int r = r_first + ql;
    const bool valid = r < n_stacked;
    const int own_splits = a.n_splits, n_splits = own_splits + a.shared_splits;
    const float* base = a.partials + (long long)(tile * Hkv + hk) * own_splits * PS + ql;
    const long long stride = PS;                               // between slices
    const float* sbase = nullptr;                              // the row's record in the shared pass, slice 0
    long long sstride = 0;
    if (a.shared_splits > 0) {
        const int rc = min(r, n_stacked - 1), R = (row0 + rc / G) * G + rc % G, gsz = 32 * SHARED_TILES;
        sbase = a.shared_partials + ((long long)((R / gsz) * a.shared_splits * Hkv + hk) * SHARED_TILES + (R % gsz) / 32) * PS + (R & 31);
        sstride = (long long)Hkv * SHARED_TILES * PS;
    }
    auto slice = [&](int s) { return s < own_splits ? base + s * stride : sbase + (s - own_splits) * sstride; };

    // rows past the sequence's end read records like the others, and write nothing
    float mv[MAXS], lv[MAXS], ov[MAXS][4];
    float mloc = -INFINITY;
#pragma unroll
    for (int i = 0; i < MAXS; ++i) {
        mv[i] = -INFINITY;
        lv[i] = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) ov[i][c] = 0.f;
        if (8 * i >= n_splits) continue;                       // wavefront-uniform, and so are the loads behind it
        const int s = sg + 8 * i;
        const float* p = slice(min(s, n_splits - 1));
        mv[i] = p[HD * 32];
        lv[i] = p[HD * 32 + 32];
#pragma unroll
        for (int c = 0; c < 4; ++c) ov[i][c] = p[(ch0 + c) * 32];
    }
#pragma unroll
    for (int i = 0; i < MAXS; ++i) {
        if (sg + 8 * i >= n_splits) mv[i] = -INFINITY;
        mloc = fmaxf(mloc, mv[i]);
    }
    if (valid)                                                 // more than 128 slices: the rest from memory
        for (int s = sg + 8 * MAXS; s < n_splits; s += 8) mloc = fmaxf(mloc, slice(s)[HD * 32]);
    red[sg][0][ql] = mloc;
    __syncthreads();
    float M = red[0][0][ql];
#pragma unroll
    for (int i = 1; i < 8; ++i) M = fmaxf(M, red[i][0][ql]);   // finite: slice 0 always sees key 0
    __syncthreads();

    float l = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < MAXS; ++i) {
        if (8 * i >= n_splits) continue;
        // absent slices: 2^-inf = 0, times 0 and not the values of the slice read instead, which may be infinite.  (Selects here, behind the
        // barrier: zeroing the values above had the compiler wait for each group's loads in turn, ~1B k = 8 3.7 -> 4.6 us.)
        const bool here = sg + 8 * i < n_splits;
        const float w = exp2f(mv[i] - M);
        l += w * (here ? lv[i] : 0.f);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] += w * (here ? ov[i][c] : 0.f);
    }
    if (valid)
        for (int s = sg + 8 * MAXS; s < n_splits; s += 8) {
            const float* p = slice(s);
            const float w = exp2f(p[HD * 32] - M);
            l += w * p[HD * 32 + 32];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] += w * p[(ch0 + c) * 32];
        }
    red[sg][1][ql] = l;
#pragma unroll
    for (int c = 0; c < 4; ++c) red[sg][2 + c][ql] = acc[c];
    __syncthreads();
    if (sg >= 4 || !valid) return;                   // 128 threads finish: (channel sg, row ql)
    float L = 0.f, o = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) { L += red[i][1][ql]; o += red[i][2 + sg][ql]; }
    f16* dst = a.out + out_index(a, row0 + r / G, (hk * G + r % G) * HD + ch0 + sg);
    const float res = split_value(o / L);
    const f16 hi = (f16)res;
    *dst = hi;
    if (a.out_lo_off) dst[a.out_lo_off] = (f16)(res - (float)hi);
}

// Slice merge for launches with many tile records and few slices each: ITEMS - the tiles the block kernel's items cut into several
// key ranges (records of the host's merge list: first slot, first stacked row, slices, T, first row); otherwise single-tile launches
// over many sequences, with their shared-prefix slices.
// One block per (group, KV head, tile): 256 threads = 32 query rows x 8 channel groups, a thread
// owns HD/8 consecutive channels of its row and walks the slices itself, so nothing meets in
// LDS and every load of a pass is independent.  Pass 1: the row's reference exponents of all
// slices -> maximum.  Pass 2: weights 2^(m_s - M), weighted sums, one 16-byte (HD = 64) or
// 32-byte store of the normalised fp16 outputs.
template <int HD, bool ITEMS>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
    constexpr int NQ = ITEMS ? 4 : 1;                          // tiles per group
    constexpr int PS = HD * 32 + 64, CPT = HD / 8;
    const int Hkv = a.kv.n_kv_heads, G = a.Hq / Hkv;
    // a head's tiles on one XCD (with 8 KV heads), the one whose attn_block_kernel left their records: tiles of a group end inside each other's
    // lines of a panel, and spread over XCDs every such line was written in parts (~3B, T = 1024 over 6144 keys: 11.15 -> 10.6 us)
    const int hk = blockIdx.x % Hkv, t = (blockIdx.x / Hkv) % NQ, tile = blockIdx.x / (NQ * Hkv);
    const int ql = threadIdx.x & 31, cg = threadIdx.x >> 5;
    const int4 ti0 = *(const int4*)(a.tile_info + tile * 8);
    const int row0 = a.tile_info[tile * 8 + 4];
    const int r = ti0.y + t * 32 + ql, n_stacked = ti0.w * G;
    if (r >= n_stacked) return;
    const int own_splits = ITEMS ? ti0.z : a.n_splits, n_splits = own_splits + a.shared_splits;
    const float* base = a.partials + (ITEMS ? ((long long)ti0.x * Hkv + hk) * NQ + t : (long long)(tile * Hkv + hk) * own_splits * NQ + t) * PS + ql;
    const long long stride = (long long)(ITEMS ? Hkv * NQ : NQ) * PS;               // between slices
    const float* sbase = nullptr;                              // the row's record in a shared-prefix pass, slice 0
    long long sstride = 0;
    if (a.shared_splits > 0) {
        const int R = (row0 + r / G) * G + r % G, gsz = 32 * SHARED_TILES;
        sbase = a.shared_partials + ((long long)((R / gsz) * a.shared_splits * Hkv + hk) * SHARED_TILES + (R % gsz) / 32) * PS + (R & 31);
        sstride = (long long)Hkv * SHARED_TILES * PS;
    }
    auto slice = [&](int s) { return s < own_splits ? base + s * stride : sbase + (s - own_splits) * sstride; };

    float M = -INFINITY;
    for (int s0 = 0; s0 < n_splits; s0 += 8) {
        float mv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) mv[i] = s0 + i < n_splits ? slice(s0 + i)[HD * 32] : -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) M = fmaxf(M, mv[i]);
    }                                                          // finite: slice 0 always sees its first key
    float L = 0.f, acc[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) acc[c] = 0.f;
    // N slices from s0 on, all their loads in flight together.  (The last ones as a group of their own size: a fourth slot that repeats a slice
    // with weight 0 would turn an infinite value into NaN.)
    auto add = [&](auto n_, int s0) {
        constexpr int N = decltype(n_)::value;
        float mv[N], lv[N], ov[N][CPT];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float* p = slice(s0 + i);
            mv[i] = p[HD * 32];
            lv[i] = p[HD * 32 + 32];
#pragma unroll
            for (int c = 0; c < CPT; ++c) ov[i][c] = p[(cg * CPT + c) * 32];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float w = exp2f(mv[i] - M);
            L += w * lv[i];
#pragma unroll
            for (int c = 0; c < CPT; ++c) acc[c] += w * ov[i][c];
        }
    };
    int s0 = 0;
    for (; s0 + 4 <= n_splits; s0 += 4) add(std::integral_constant<int, 4>{}, s0);
    if (n_splits - s0 == 3) add(std::integral_constant<int, 3>{}, s0);
    else if (n_splits - s0 == 2) add(std::integral_constant<int, 2>{}, s0);
    else if (n_splits - s0 == 1) add(std::integral_constant<int, 1>{}, s0);
    const float inv = 1.0f / L;
#pragma unroll
    for (int c0 = 0; c0 < CPT; c0 += 8) {
        f16* dst = a.out + out_index(a, row0 + r / G, (hk * G + r % G) * HD + cg * CPT + c0);
        f16x8 v, lo;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float ov = split_value(acc[c0 + c] * inv);
            v[c] = (f16)ov;
            lo[c] = (f16)(ov - (float)v[c]);
        }
        *(f16x8*)dst = v;
        if (a.out_lo_off) *(f16x8*)(dst + a.out_lo_off) = lo;
    }
}

size_t attention_partial_floats(int n_tiles, int n_kv_heads, int head_dim, int n_splits) {
    return (size_t)n_tiles * n_kv_heads * n_splits * ((size_t)head_dim * 32 + 64);
}

template <int HD>
static void launch_tiles(const AttnArgs& a, int n_tiles, int waves, hipStream_t s) {
    dim3 grid(n_tiles, a.kv.n_kv_heads, a.n_splits);
    if (waves == 0) {                                          // done by attn_shared_kernel
    } else if (waves == 4) {
        if (a.q_lo_off) attn_split_kernel<HD, 4, true><<<grid, 256, 0, s>>>(a);
        else attn_split_kernel<HD, 4, false><<<grid, 256, 0, s>>>(a);
    } else {
        if (a.q_lo_off) attn_split_kernel<HD, 1, true><<<grid, 64, 0, s>>>(a);
        else attn_split_kernel<HD, 1, false><<<grid, 64, 0, s>>>(a);
    }
    const int records = n_tiles * a.kv.n_kv_heads;
    if (attention_merge_by_record(records, a.n_splits + a.shared_splits)) attn_merge_kernel<HD, false><<<records, 256, 0, s>>>(a);
    else attn_combine_kernel<HD><<<dim3(records, HD / 4), 256, 0, s>>>(a);
}

template <int HD>
static void launch_block(const AttnArgs& a, int n_items, hipStream_t s) {
    dim3 grid((unsigned)n_items, (unsigned)a.kv.n_kv_heads);
    if (a.q_lo_off) attn_block_kernel<HD, true><<<grid, 256, 0, s>>>(a);
    else attn_block_kernel<HD, false><<<grid, 256, 0, s>>>(a);
}
// The items of a block-kernel pass, then the groups of 4 tiles whose keys they cut (n_merge; the shared-prefix pass has none).
static void launch_items(const AttnArgs& a, int n_items, int n_merge, hipStream_t s) {
    if (a.kv.head_dim == 64) launch_block<64>(a, n_items, s);
    else launch_block<128>(a, n_items, s);
    if (n_merge == 0) return;
    AttnArgs mg = a;
    mg.tile_info = a.tile_info + (size_t)n_items * 8;
    const unsigned mgrid = (unsigned)(n_merge * a.kv.n_kv_heads * 4);
    if (a.kv.head_dim == 64) attn_merge_kernel<64, true><<<mgrid, 256, 0, s>>>(mg);
    else attn_merge_kernel<128, true><<<mgrid, 256, 0, s>>>(mg);
}

void launch_attention(DType dt, const void* q, void* out, KVGeom kv, int layer, const StepView& sv,
                      int n_q_heads, float* partials, int n_splits, int split_waves, hipStream_t s, long long q_lo_off,
                      long long out_lo_off, ActLayout out_layout) {
    if (dt == F32) {
        const int subs = 2 * sv.tile_nq, hd = kv.head_dim;      // 16-row tiles per record of 32 * tile_nq rows
        dim3 grid(sv.n_tiles * subs, kv.n_kv_heads);
        const float* qf = (const float*)q;
        float* of = (float*)out;
        // Blocks of 16 output channels while there is a CU for each: 8 / 256 rows over 512 keys (head_dim 64, 2 KV heads) 13.1 -> 11.7 / 16.2 -> 14.6 us;
        // at 512 rows, two rounds of blocks, the scores they repeat cost more than the idle CUs: 19.8 -> 30.6 us.
        const long long blocks = (long long)grid.x * grid.y;
        if (hd == 64 && blocks * 4 <= 256) {
            grid.z = 4;
            attn_f32_kernel<4, 1, 16, true><<<grid, 1024, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        } else if (hd == 128 && blocks * 8 <= 256) {
            grid.z = 8;
            attn_f32_kernel<8, 1, 16, true><<<grid, 1024, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        }
        // wavefronts per block: as many as the LDS record of their partial outputs (4 KB per 64 channels each) leaves room for
        else if (hd == 64) attn_f32_kernel<4, 4, 16, true><<<grid, 1024, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        else if (hd < 64) attn_f32_kernel<4, 4, 16, false><<<grid, 1024, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        else if (hd == 128) attn_f32_kernel<8, 8, 8, true><<<grid, 512, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        else if (hd < 128) attn_f32_kernel<8, 8, 8, false><<<grid, 512, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        else if (hd == 256) attn_f32_kernel<16, 16, 4, true><<<grid, 256, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        else attn_f32_kernel<16, 16, 4, false><<<grid, 256, 0, s>>>(qf, of, kv, layer, sv.tile_info, sv.bt, n_q_heads, subs);
        return;
    }
    AttnArgs a{};
    a.q = (const f16*)q; a.out = (f16*)out; a.kv = kv; a.layer = layer; a.Hq = n_q_heads; a.G = n_q_heads / kv.n_kv_heads; a.n_splits = n_splits;
    a.tile_info = sv.tile_info; a.bt = sv.bt; a.partials = partials;
    a.q_lo_off = q_lo_off; a.out_lo_off = out_lo_off; a.n_rows = sv.n_rows; a.out_layout = out_layout;
    const int hd = kv.head_dim;
    if (sv.tile_nq == 4) {                                     // long extends: 4 tiles per block, K/V through LDS
        launch_items(a, sv.n_items, sv.n_merge, s);
    } else {
        if (sv.n_tiles_shared > 0) {
            // Many sequences that share a cached prefix (the same leading blocks): the keys of the
            // prefix are applied ONCE to the rows of all sequences - a pass of the block kernel over
            // one virtual sequence made of every row of the call, keys [0, shared_len), no causal
            // mask needed - instead of being pulled from L2 once per sequence; the per-sequence
            // wavefronts below start at shared_len, and the merge adds the shared pass's slices.
            AttnArgs sh = a;
            sh.tile_info = sv.tile_info + (size_t)sv.n_tiles * 8;
            sh.partials = partials + attention_partial_floats(sv.n_tiles, kv.n_kv_heads, hd, n_splits);
            const int items = sv.n_tiles_shared * sv.shared_splits;
            if (split_waves == 4) {
                const unsigned blocks = (unsigned)(items + sv.n_tiles * n_splits) * (unsigned)kv.n_kv_heads;
                if (hd == 64 && q_lo_off) attn_shared_kernel<64, true><<<blocks, 256, 0, s>>>(sh, a, items, sv.n_tiles);
                else if (hd == 64) attn_shared_kernel<64, false><<<blocks, 256, 0, s>>>(sh, a, items, sv.n_tiles);
                else if (q_lo_off) attn_shared_kernel<128, true><<<blocks, 256, 0, s>>>(sh, a, items, sv.n_tiles);
                else attn_shared_kernel<128, false><<<blocks, 256, 0, s>>>(sh, a, items, sv.n_tiles);
                split_waves = 0;
            } else {
                launch_items(sh, items, 0, s);
            }
            a.shared_partials = sh.partials;
            a.shared_splits = sv.shared_splits;
            a.shared_len = sv.shared_len;
        }
        if (hd == 64) launch_tiles<64>(a, sv.n_tiles, split_waves, s); else launch_tiles<128>(a, sv.n_tiles, split_waves, s);
    }
}

}  // namespace ax
