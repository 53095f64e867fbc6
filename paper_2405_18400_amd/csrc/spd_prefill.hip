// Dense prefix pass: the first-timestep forward over the prefix M (Section 3, "First
// Timestep") for a whole chunk of prefix tokens at once, so that the weights are read once per
// chunk instead of once per token.  Here the work IS a dense contraction, [tokens, d] x
// [rows, d]^T, and runs on the matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Precision: the step path multiplies bf16 weights with fp32 activations.  To stay within
// rounding of it, an activation x is fed as two bf16 terms, hi = bf16(x) and lo = bf16(x - hi)
// (16 mantissa bits together), and W x = W hi + W lo is two matrix-core products into the same
// fp32 accumulator.  Feeding bf16(x) alone costs about 2e-2 of the logit scale over 32 layers.
//
// Operands need no transposition: with W row-major [rows, d] and activations [tokens, d], both
// MFMA operands are "row index in the lane, 8 consecutive k in the register", i.e. plain
// 16-byte pieces.
#include "spd_device.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

using namespace spdd;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

__device__ __forceinline__ uint16_t bf16_rn(float v) {
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// x = hi + lo up to 2^-17 |x|
__device__ __forceinline__ void split_store(uint16_t *hi, uint16_t *lo, size_t at, float x) {
    const uint16_t h = bf16_rn(x);
    as_global(hi)[at] = h;
    as_global(lo)[at] = bf16_rn(x - bf16_f(h));
}

// Four consecutive elements, one 8-byte store per half.
__device__ __forceinline__ void split_store4(uint16_t *hi, uint16_t *lo, size_t at, f32x4 y) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) { h[e] = bf16_rn(y[e]); l[e] = bf16_rn(y[e] - bf16_f((uint16_t)h[e])); }
    *(u32x2 __attribute__((address_space(1))) *)(hi + at) = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
    *(u32x2 __attribute__((address_space(1))) *)(lo + at) = u32x2{l[0] | (l[1] << 16), l[2] | (l[3] << 16)};
}
// Eight consecutive elements, one 16-byte store per half.
__device__ __forceinline__ void split_store8(uint16_t *hi, uint16_t *lo, size_t at, const float (&y)[8]) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const uint16_t h0 = bf16_rn(y[e]), h1 = bf16_rn(y[e + 1]);
        h[e / 2] = (uint32_t)h0 | ((uint32_t)h1 << 16);
        l[e / 2] = (uint32_t)bf16_rn(y[e] - bf16_f(h0)) | ((uint32_t)bf16_rn(y[e + 1] - bf16_f(h1)) << 16);
    }
    *(u32x4 __attribute__((address_space(1))) *)(hi + at) = u32x4{h[0], h[1], h[2], h[3]};
    *(u32x4 __attribute__((address_space(1))) *)(lo + at) = u32x4{l[0], l[1], l[2], l[3]};
}

// ------------------------------------------------------------------ residual stream, norms, rotary table
// The residual stream between two products, one block per token: h = embedding of the token (EMBED), or
// h = residual + the partial sums of the product before it, added in split order; then
// xn = h * rsqrt(mean h^2 + eps) * gain as the (hi, lo) pair.  A thread has 8 consecutive features (d_model / 8 threads, whole
// waves, at most 1024: d_model <= 8192) and asks for all it needs at once, up to eight splits and the gain: one trip to memory.
// Bound by that trip with few tokens, by the bytes with many: 64 tokens of 4096 in 8 splits 6.5 -> 5.2 us, 1024 tokens in 2
// splits 15.6 -> 15.2 (256 threads with two to four runs of 8 features, splits four at a time, the gain behind the sum of squares).
struct PrefillNormArgs {
    const uint16_t *embed;       // EMBED: [vocab, d]
    const int32_t *tokens;       // EMBED: token ids of the chunk
    const float *part;           // [splits, T, d]
    float *h;                    // [T, d]: the residual, updated in place
    const uint16_t *gain;
    uint16_t *hi, *lo;           // [T, d]
    int32_t T, d, splits;
    float eps;
    // EMBED: the chunk's rotary table comes along, a launch less: (cos, sin) of (p0 + t) * theta^(-2i/d_head), in double as everywhere else
    const double *inv_freq;
    float2 *rope;                // [T, half]
    int32_t p0, half;
};

template <bool EMBED>
__global__ __launch_bounds__(1024) void prefill_norm_kernel(const PrefillNormArgs a) {
    __shared__ float red[1024 / WAVE];
    const int t = blockIdx.x, d = a.d, c = 8 * threadIdx.x;
    const bool mine = c < d;
    const size_t at = (size_t)t * d + (mine ? c : 0);
    auto take = [&](const float *x, float (&y)[8]) {
        const float4 p = global_load_float4(x), q = global_load_float4(x + 4);
        y[0] = p.x; y[1] = p.y; y[2] = p.z; y[3] = p.w; y[4] = q.x; y[5] = q.y; y[6] = q.z; y[7] = q.w;
    };
    auto widen = [](u32x4 g, float (&y)[8]) {
        const uint32_t w[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
        for (int e = 0; e < 8; e += 2) { y[e] = __uint_as_float(w[e / 2] << 16); y[e + 1] = __uint_as_float(w[e / 2] & 0xFFFF0000u); }
    };
    float v[8];
    const u32x4 gw = global_load16(a.gain + (mine ? c : 0));
    if (EMBED) {
        widen(global_load16(a.embed + (size_t)as_global(a.tokens)[t] * d + (mine ? c : 0)), v);
    } else {
        constexpr int AT_ONCE = 8;
        float more[AT_ONCE][8], sum[8];
        take(a.h + at, v);
        for (int s = 0; s < a.splits; s += AT_ONCE) {
#pragma unroll
            for (int q = 0; q < AT_ONCE; ++q)
                if (s + q < a.splits) take(a.part + (size_t)(s + q) * a.T * d + at, more[q]);
#pragma unroll
            for (int q = 0; q < AT_ONCE; ++q)
                if (s + q < a.splits) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) sum[e] = s + q == 0 ? more[q][e] : sum[e] + more[q][e];
                }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += sum[e];
    }
    if (EMBED && (int)threadIdx.x < a.half) a.rope[(size_t)t * a.half + threadIdx.x] = rope_cos_sin(a.inv_freq, threadIdx.x, a.p0 + t);
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
    ss = wave_sum_last(mine ? ss : 0.f);
    if (threadIdx.x % WAVE == WAVE - 1) red[threadIdx.x / WAVE] = ss;
    if (mine) {
        *(f32x4 __attribute__((address_space(1))) *)(a.h + at) = f32x4{v[0], v[1], v[2], v[3]};
        *(f32x4 __attribute__((address_space(1))) *)(a.h + at + 4) = f32x4{v[4], v[5], v[6], v[7]};
    }
    __syncthreads();
    if (!mine) return;
    float tot = 0.f, g[8];
    for (int w = 0; w < (int)blockDim.x / WAVE; ++w) tot += red[w];
    const float rs = 1.0f / sqrtf(tot / (float)d + a.eps);
    widen(gw, g);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * rs * g[e];
    split_store8(a.hi, a.lo, at, v);
}
static int norm_threads(int d) { return (d / 8 + WAVE - 1) / WAVE * WAVE; }

// ------------------------------------------------------------------ GEMM on the matrix cores
// PE_PART: partial sums over this block's share of k, to `part`; the consumer adds the splits.
enum { PE_PART = 0, PE_QKV = 1, PE_SWIGLU = 2 };

struct PrefillGemmArgs {
    const uint16_t *xhi, *xlo;   // [T, K] bf16 pair
    // [N, K] bf16; W2: the "up" matrix (PE_SWIGLU), or columns N .. 2 N - 1 of the partial sums (PE_PART), or null.  Each matrix
    // has n_tiles column tiles of its own; the last may be ragged: its rows are clamped and its stores masked (nc < N).
    const uint16_t *W, *W2;
    int32_t T, N, K;
    int32_t t_tiles, n_tiles;    // token tiles; column tiles of W (and W2)
    int32_t splits, split_steps; // blocks that share a tile's k range, and steps per block
    int32_t rotate;              // blocks start at different places of their k range
    float *part;                 // PE_PART: [splits, T, N (2 N with W2)]
    // PE_QKV
    float *q;                    // [T, n_q_rows]
    void *kcache, *vcache;       // [n_kv_heads, cap_ctx, d_head] fp32, or fp16 (kv_half)
    int32_t kv_half;
    const float2 *rope;          // [T, d_head / 2]
    int32_t n_q_rows, n_kv_rows, d_head, cap_ctx, p0;
    uint16_t *uhi, *ulo;         // PE_SWIGLU: [T, N]
};

// Rows nc .. nc + 3 of the fused QKV product (nc a multiple of 4, d_head of 8: one head's, two rotary pairs): what their values become,
// and where they go.
struct QkvRows {
    bool rotates, is_q;
    int pair;                    // the first of the head's two rotary pairs
    char *to;                    // token 0's element nc
    size_t stride;               // elements from token to token
    __device__ __forceinline__ QkvRows(const PrefillGemmArgs &a, int nc) {
        rotates = nc < a.n_q_rows + a.n_kv_rows; is_q = nc < a.n_q_rows;
        const int rr = is_q ? nc : rotates ? nc - a.n_q_rows : nc - a.n_q_rows - a.n_kv_rows;
        const int head = rr / a.d_head, f = rr % a.d_head;
        pair = f / 2;
        if (is_q) {
            to = (char *)(a.q + nc);
            stride = (size_t)a.n_q_rows;
        } else {
            to = (char *)(rotates ? a.kcache : a.vcache) + (((size_t)head * a.cap_ctx + a.p0) * a.d_head + f) * (a.kv_half ? 2 : 4);
            stride = (size_t)a.d_head;
        }
    }
    // (cos, sin) of both pairs; only asked for where it rotates
    __device__ __forceinline__ float4 angles(const PrefillGemmArgs &a, int t) const {
        return global_load_float4((const float *)(a.rope + (size_t)t * (a.d_head / 2) + pair));
    }
    __device__ __forceinline__ void put(const PrefillGemmArgs &a, int t, f32x4 v, float4 cs) const {
        if (rotates) {
            const f32x4 x = v;
            v.x = __fsub_rn(__fmul_rn(x.x, cs.x), __fmul_rn(x.y, cs.y));
            v.y = __fadd_rn(__fmul_rn(x.x, cs.y), __fmul_rn(x.y, cs.x));
            v.z = __fsub_rn(__fmul_rn(x.z, cs.z), __fmul_rn(x.w, cs.w));
            v.w = __fadd_rn(__fmul_rn(x.z, cs.w), __fmul_rn(x.w, cs.z));
        }
        if (is_q || !a.kv_half) {
            *(f32x4 __attribute__((address_space(1))) *)((float *)to + (size_t)t * stride) = v;
        } else {
            const uint32_t lo = (uint32_t)Store<half_t>::bits(v.x) | ((uint32_t)Store<half_t>::bits(v.y) << 16);
            const uint32_t hi = (uint32_t)Store<half_t>::bits(v.z) | ((uint32_t)Store<half_t>::bits(v.w) << 16);
            *(u32x2 __attribute__((address_space(1))) *)((uint16_t *)to + (size_t)t * stride) = u32x2{lo, hi};
        }
    }
};

// A block of WM x WN waves makes a tile of BM = 16 TT WM tokens x BN = 16 NT WN columns; a wave's share is
// TT x NT accumulators of 16 x 16 (v_mfma_f32_16x16x32_bf16: with random operands it holds 1.87 .. 2.03 PFLOP/s where the
// 32 x 32 x 16 form holds 1.70 .. 1.76: power is the limit, both reach 2.48 on zeros).  Per step of 64 k the tile's operands
// (x hi, x lo, W: rows of 64 elements) go from memory straight into LDS (no registers in between), ST steps deep, and from there
// half a step ahead into registers: while one half is multiplied the other is read, the first half of the next step behind
// the step's one barrier, so the matrix cores have work while it is passed.  A load instruction fills 1 KB of LDS in lane
// order, so the rows lie unpadded; the 16-byte pieces of a row are permuted by the row number (`swz`: the lane picks which
// piece of the row it fetches) so that the lanes LDS serves together in such a read -- 0 .. 3, 12 .. 15 and 20 .. 27, and so on --
// find rows of both parities, eight different pieces each: no bank conflicts (row & 7 ^ row >> 3 & 1, right for operands of 32
// rows, left half of the reads' cycles to conflicts).
// What bounds it: with 128-token tiles the matrix cores at the clock they hold under such products (on zeros the same launch takes
// 20 % less) and the loads' way into LDS (without them 18 % less); with few tokens the weight stream and each launch's ramp.
// Before (products of 32 x 32 x 16, operands read behind the barrier, a lane's results in a column) -> after, us: 1024 tokens,
// 12288 x 4096 with the rotary epilogue 187 -> 176; gate and up 2 x 11008 x 4096 335 -> 313; 4096 x 11008 175 -> 163; 512 tokens,
// 2 x 28672 x 8192 838 -> 760; the best shape of each product over the widths of 1B .. 70B: 0.99 times the time up to 64 tokens,
// 0.96 at 160 .. 384, 0.92 at 1024.
// Tried: four waves of 64 x 128 (20 % slower: one wave per SIMD), steps of 32 k (64 bytes of a row: half of every cache line
// fetched twice, 2.5 instead of 4.8 TB/s), a second barrier that frees a buffer earlier, wave priorities, touching the lines of
// coming steps so that they are in the L2 (0 .. 5 % slower), waves that load x only or W only (-9 .. +13 %), four waves of 64 x 192 with the
// order below (8 .. 22 % slower), W from memory straight into the registers of the one wave that multiplies it, x alone through LDS (two to six
// steps ahead; 1.00 .. 1.08 times the time from 256 tokens on, 1.1 .. 1.2 at 64).
// Where a block starts within its k range (`turn`): rows whose length is a power of two lie 8 KB or 16 KB apart, and blocks that all
// walk them from the same end keep hitting the same memory channels: 4.9 and 4.5 TB/s for a stream of 128-byte pieces, 7.0
// from rows of 10 or 22 KB.  Blocks of different XCDs, and neighbours on one, therefore start an eighth of the range apart and wrap
// round: 7B gate and up for 8 tokens 39.5 -> 33, for 64 45.3 -> 38 (two splits); the 70B widths' products 0.84 .. 0.98 times.
// Other row lengths gain nothing, and with more than one token tile the L2 loses the x that neighbours read together (2 .. 5 % slower).
// Weights go past the L2's keep list (STREAM_W) in the tiles of 32 and 64 tokens: 2 .. 4 % faster where one token tile reads them, no
// difference (1 %) at two to eight, up to 3 % slower at eleven and twelve; no difference in the tiles of 128 tokens.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

template <int EPI, int WM, int WN, int TT, int NT, int KS, int ST, bool STREAM_W>
__global__ __launch_bounds__(64 * WM * WN, WM * WN >= 4 ? WM * WN / 4 : 1) void prefill_gemm_kernel(const PrefillGemmArgs a) {
    constexpr int NWV = WM * WN, BM = 16 * TT * WM, BN = 16 * NT * WN;
    constexpr int ROWB = KS * 2, RPL = 1024 / ROWB;        // bytes per row; rows one load instruction of a wave brings
    constexpr int ROWS = 2 * BM + BN;                      // rows of a stage: x hi, x lo, W
    constexpr int PER = ROWS / (RPL * NWV);                // load instructions per wave and stage
    constexpr int STAGE = ROWS * ROWB;
    constexpr int NG = EPI == PE_SWIGLU ? NT / 2 : NT;     // column tiles of a wave per matrix (PE_SWIGLU: gate, then the same units of up)
    static_assert(KS == 64 && ST >= 2, "two halves of 32 k; rows of 128 bytes");
    static_assert(ROWS % (RPL * NWV) == 0 && BM % RPL == 0 && BN % (2 * RPL) == 0, "whole load instructions");
    extern __shared__ __align__(16) char stages[];         // [ST][STAGE]
    const int lane = threadIdx.x & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    // Workgroups go to the 8 XCDs round-robin and each XCD has its own L2: all token tiles of a column tile run on
    // one XCD, one after the other, so that a weight tile enters one L2 only.
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int n_mats = EPI == PE_PART && a.W2 != nullptr ? 2 : 1;
    const int col = (slot / a.t_tiles) * 8 + xcd, tile_x = slot % a.t_tiles;
    if (col >= a.n_tiles * n_mats * a.splits) return;
    const int split = col / (a.n_tiles * n_mats), tile_y = col % (a.n_tiles * n_mats);
    const bool second = EPI == PE_PART && tile_y >= a.n_tiles;
    const int t0 = tile_x * BM;
    const int n0 = (second ? tile_y - a.n_tiles : tile_y) * (EPI == PE_SWIGLU ? BN / 2 : BN);   // first row of the weight matrix
    const int s0 = split * a.split_steps, n_steps = min(a.split_steps, a.K / KS - s0);

    // This wave's loads of a stage: load i brings rows RPL (w + NWV i) ..; lane -> row l / (64 / RPL), piece l % (64 / RPL).
    // A row past the end re-reads the last one (its products are dropped).
    __amdgpu_buffer_rsrc_t rsrc[PER];
    uint32_t off[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int q = RPL * (w + NWV * i), r = lane / (WAVE / RPL);           // (q is uniform; a load lies within one operand)
        const char *base;
        int row, rows;
        if (q < 2 * BM) {
            base = (const char *)(q < BM ? a.xhi : a.xlo);
            row = t0 + (q < BM ? q : q - BM) + r;
            rows = a.T;
        } else {
            const int c = q - 2 * BM;
            const bool up = EPI == PE_SWIGLU ? c >= BN / 2 : second;
            base = (const char *)(up ? a.W2 : a.W);
            row = n0 + (EPI == PE_SWIGLU && up ? c - BN / 2 : c) + r;
            rows = a.N;
        }
        rsrc[i] = row_resource(base, (uint32_t)rows * (uint32_t)a.K * 2u);
        off[i] = ((uint32_t)min(row, rows - 1) * (uint32_t)a.K + (uint32_t)s0 * KS) * 2u + 16u * (uint32_t)((lane % (WAVE / RPL)) ^ swz(q + r));
    }
    const int turn = a.rotate ? (xcd + 3 * (slot / a.t_tiles)) % 8 * n_steps / 8 : 0;
    auto load = [&](int step, int i) {
        char *to = stages + (step % ST) * STAGE;
        const int s = step + turn < n_steps ? step + turn : step + turn - n_steps;
        if (STREAM_W && RPL * NWV * i >= 2 * BM) load16_to_lds<2>(rsrc[i], to + (w + NWV * i) * 1024, off[i], s * ROWB);
        else load16_to_lds<0>(rsrc[i], to + (w + NWV * i) * 1024, off[i], s * ROWB);
    };

    // Operands of half a step in registers, 16 rows of 32 k per piece of work: lane -> row l % 16, k 8 (l / 16) ..  The weights
    // are the first operand, so a lane ends up with one token's values of four consecutive columns.
    const int wm = w / WN, wn = w % WN;
    const int x_row = 16 * TT * wm + lane % 16;
    auto w_row = [&](int nt) { return 2 * BM + lane % 16 + (nt / NG) * (BN / 2) + 16 * (NG * wn + nt % NG); };
    struct Half { bf16x8 w[NT], hi[TT], lo[TT]; };
    f32x4 acc[NT][TT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[nt][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The order is written out, an instruction of the memory pipes between every few products (`sched_barrier`): left to itself the
    // compiler sinks a half's reads to the end of the products they should run beside, and every half begins with a wait for all of
    // them.  us, so -> written out: 1024 tokens, 12288 x 4096 169 -> 163, gate and up 306 -> 295, 4096 x 4096 70 -> 66; 256 tokens,
    // 15360 x 5120 131 -> 125 (128 x 256); whole passes 1.01 (64 and 256 tokens) .. 1.03 times as fast (1024).  What is left is power: the same
    // launch on zeros takes 115 us instead of 163, without its loads 139, without its reads 135, its products alone 107.
    auto half_of = [&](int s, int half) { return (uint32_t)((s % ST) * STAGE + 16 * ((4 * half + lane / 16) ^ swz(lane % 16))); };   // (16 rows on: the same permutation)
    constexpr int READS = NT + 2 * TT, PRODUCTS = 2 * NT * TT;
    auto read = [&](Half &f, uint32_t at, int i) {         // in the order of use
        auto piece = [&](int row) { return __builtin_bit_cast(bf16x8, *(const u32x4 *)(stages + at + row * ROWB)); };
        if (i == 0) f.hi[0] = piece(x_row);
        else if (i <= NT) f.w[i - 1] = piece(w_row(i - 1));
        else if (i < NT + TT) f.hi[i - NT] = piece(x_row + 16 * (i - NT));
        else f.lo[i - NT - TT] = piece(BM + x_row + 16 * (i - NT - TT));
    };
    auto product = [&](const Half &f, int i) {
        const int tt = i / NT % TT, nt = i % NT;
        acc[nt][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[nt], i < NT * TT ? f.hi[tt] : f.lo[tt], acc[nt][tt], 0, 0, 0);
    };
    // the products of one half, the reads of the next and (behind the barrier) the loads of a coming step beside them
    auto work = [&](const Half &f, Half &g, uint32_t at, bool reads, bool loads, int step) {
        int r = 0, l = 0;
#pragma unroll
        for (int i = 0; i < PRODUCTS; ++i) {
            constexpr int UNTIL = PRODUCTS * 3 / 4;
            if (reads && i < UNTIL) {
#pragma unroll
                for (; r < ((i + 1) * READS + UNTIL - 1) / UNTIL; ++r) read(g, at, r);
            }
            if (loads && i < UNTIL) {
#pragma unroll
                for (; l < ((i + 1) * PER + UNTIL - 1) / UNTIL; ++l) load(step, l);
            }
            product(f, i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // The compiler does not count loads into LDS: the waits are written out.  One barrier per step, in its middle: before it every
    // wave has its own loads of step s + 1 in LDS (all but the (ST - 2) PER youngest have arrived: loads arrive in order) and
    // its last reads of step s behind it, so behind it step s + 1 may be read and the buffer of step s filled again.
    Half f0, f1;
    for (int s = 0; s < ST && s < n_steps; ++s) {
#pragma unroll
        for (int i = 0; i < PER; ++i) load(s, i);
    }
    if (n_steps >= ST) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((ST - 1) * PER) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < READS; ++i) read(f0, half_of(0, 0), i);
    int s = 0;
    for (; s + ST < n_steps; ++s) {
        work(f0, f1, half_of(s, 1), true, false, 0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((ST - 2) * PER) : "memory");
        work(f1, f0, half_of(s + 1, 0), true, true, s + ST);
    }
    for (; s + 1 < n_steps; ++s) {
        work(f0, f1, half_of(s, 1), true, false, 0);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        work(f1, f0, half_of(s + 1, 0), true, false, 0);
    }
    work(f0, f1, half_of(s, 1), true, false, 0);
    work(f1, f0, 0, false, false, 0);

    // lane -> token l % 16 of a piece, register r -> column 4 (l / 16) + r
#pragma unroll
    for (int nt = 0; nt < NG; ++nt) {
        const int nc = n0 + 16 * (NG * wn + nt) + 4 * (lane / 16);
        const QkvRows rows(a, EPI == PE_QKV ? nc : 0);
        float4 cs[TT];
        if (EPI == PE_QKV && rows.rotates) {    // (one trip for all)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) cs[tt] = rows.angles(a, min(t0 + 16 * (TT * wm + tt) + lane % 16, a.T - 1));
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const int t = t0 + 16 * (TT * wm + tt) + lane % 16;
            if (t >= a.T || nc >= a.N) continue;
            const f32x4 v = acc[nt][tt];
            if (EPI == PE_QKV) {
                rows.put(a, t, v, cs[tt]);
            } else if (EPI == PE_PART) {
                const size_t ld = (size_t)a.N * n_mats;
                *(f32x4 __attribute__((address_space(1))) *)(a.part + ((size_t)split * a.T + t) * ld + (second ? a.N : 0) + nc) = v;
            } else {
                const f32x4 up = acc[(nt + NG) % NT][tt];
                f32x4 y;
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = v[r] / (1.0f + expf(-v[r])) * up[r];
                split_store4(a.uhi, a.ulo, (size_t)t * a.N + nc, y);
            }
        }
    }
}

// The partial sums of a split QKV product, added in split order, through its epilogue.  A thread has four rows.
__global__ __launch_bounds__(256) void prefill_qkv_sum_kernel(const PrefillGemmArgs a) {
    const int t = blockIdx.y, nc = 4 * (blockIdx.x * 256 + threadIdx.x);
    if (nc >= a.N) return;
    const QkvRows rows(a, nc);
    const float4 cs = rows.rotates ? rows.angles(a, t) : make_float4(1.f, 0.f, 1.f, 0.f);
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < a.splits; s += 4) {
        float4 p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = global_load_float4(a.part + ((size_t)min(s + q, a.splits - 1) * a.T + t) * a.N + nc);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (s + q < a.splits) { v.x += p[q].x; v.y += p[q].y; v.z += p[q].z; v.w += p[q].w; }
    }
    rows.put(a, t, v, cs);
}

// The same for gate and up: SiLU(gate) * up as the (hi, lo) pair.  A thread has 8 units.
__global__ __launch_bounds__(256) void prefill_swiglu_sum_kernel(const PrefillGemmArgs a) {
    const int t = blockIdx.y, nc = 8 * (blockIdx.x * 256 + threadIdx.x);
    if (nc >= a.N) return;
    float g[8], u[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = u[e] = 0.f;
    for (int s = 0; s < a.splits; ++s) {
        const float *p = a.part + ((size_t)s * a.T + t) * 2 * a.N + nc;
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const float4 x = global_load_float4(p + e), y = global_load_float4(p + a.N + e);
            g[e] += x.x; g[e + 1] += x.y; g[e + 2] += x.z; g[e + 3] += x.w;
            u[e] += y.x; u[e + 1] += y.y; u[e + 2] += y.z; u[e + 3] += y.w;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
    split_store8(a.uhi, a.ulo, (size_t)t * a.N + nc, g);
}

// ------------------------------------------------------------------ causal attention over the chunk
// Four consecutive elements of the key/value cache, element type KT, from element `at`.
template <typename KT> __device__ __forceinline__ float4 kv_load4(const void *base, size_t at);
template <> __device__ __forceinline__ float4 kv_load4<float>(const void *base, size_t at) { return global_load_float4((const float *)base + at); }
template <> __device__ __forceinline__ float4 kv_load4<half_t>(const void *base, size_t at) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const u32x2 w = *(const u32x2 __attribute__((address_space(1))) *)((const uint16_t *)base + at);
    const uint32_t x = w.x, y = w.y;   // (bit casts of copies, not of the vector's elements)
    const h2 lo = __builtin_bit_cast(h2, x), hi = __builtin_bit_cast(h2, y);
    return make_float4((float)lo.x, (float)lo.y, (float)hi.x, (float)hi.y);
}
// One block: one query head, AQ queries of the chunk; keys / values streamed through LDS in
// chunks of AK cached positions (cache elements of type KT, widened on load), online softmax.  Output as the (hi, lo) pair.
constexpr int ANT = 256, AQ = 32, AK = 64;

struct PrefillAttnArgs {
    const float *q;               // [T, n_heads * d_head]
    const void *kcache, *vcache;  // [n_kv_heads, cap_ctx, d_head] in the kernel's KT
    uint16_t *ohi, *olo;          // [T_pad, n_heads * d_head]
    float *o32;                   // heads of 64 and 128 over an fp32 cache: the output in fp32 instead, or null
    int32_t T, p0, n_heads, n_kv_heads, d_head, cap_ctx;
};

template <typename KT>
__global__ __launch_bounds__(ANT) void prefill_attn_kernel(const PrefillAttnArgs a) {
    extern __shared__ __align__(16) float lds[];
    // row strides: 16-byte aligned, and consecutive rows 4 banks apart (no conflicts for the
    // 8 rows the 8 threads of a query read side by side)
    const int dh = a.d_head, ldk = dh + 4, lds_s = AK + 1;
    float *Qs = lds;                       // [AQ][dh + 4]
    float *Ks = Qs + AQ * ldk;             // [AK][dh + 4]
    float *Vs = Ks + AK * ldk;             // [AK][dh]
    float *Ss = Vs + AK * dh;              // [AQ][AK + 1]
    const int tid = threadIdx.x;
    const int h = blockIdx.y, g = h / (a.n_heads / a.n_kv_heads);
    const int q0 = blockIdx.x * AQ;
    const int nqd = a.n_heads * dh, dh4 = dh / 4;
    const float scale = 1.0f / sqrtf((float)dh);
    for (int e = tid; e < AQ * dh4; e += ANT) {
        const int i = e / dh4, c = 4 * (e % dh4), t = q0 + i;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (t < a.T) v = global_load_float4(a.q + (size_t)t * nqd + (size_t)h * dh + c);
        *(float4 *)(Qs + i * ldk + c) = v;
    }
    const int qi = tid / 8, sub = tid % 8;          // this thread's query, and its share of keys / dims
    const int qpos = a.p0 + q0 + qi;                // cached positions 0 .. qpos are visible
    float m = -INFINITY, l = 0.f;
    float4 acc[4];                                  // dims 4 (sub + 8 g4) .. + 3, g4 = 0 .. 3 (d_head <= 128)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) acc[g4] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int last = min(a.p0 + q0 + AQ - 1, a.p0 + a.T - 1);   // last position any query of the tile sees
    const size_t head_at = (size_t)g * a.cap_ctx * dh;
    for (int c0 = 0; c0 <= last; c0 += AK) {
        __syncthreads();
        for (int e = tid; e < AK * dh4; e += ANT) {
            const int j = e / dh4, c = 4 * (e % dh4), pos = c0 + j;
            float4 kv = make_float4(0.f, 0.f, 0.f, 0.f), vv = kv;
            if (pos <= last) {
                kv = kv_load4<KT>(a.kcache, head_at + (size_t)pos * dh + c);
                vv = kv_load4<KT>(a.vcache, head_at + (size_t)pos * dh + c);
            }
            *(float4 *)(Ks + j * ldk + c) = kv;
            *(float4 *)(Vs + j * dh + c) = vv;
        }
        __syncthreads();
        // scores of query qi with keys sub + 8 jj
        float s[8], cmax = -INFINITY;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) s[jj] = 0.f;
        for (int d = 0; d < dh; d += 4) {
            const float4 qv = *(const float4 *)(Qs + qi * ldk + d);
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                const float4 kv = *(const float4 *)(Ks + (sub + 8 * jj) * ldk + d);
                s[jj] = fmaf(qv.x, kv.x, s[jj]); s[jj] = fmaf(qv.y, kv.y, s[jj]);
                s[jj] = fmaf(qv.z, kv.z, s[jj]); s[jj] = fmaf(qv.w, kv.w, s[jj]);
            }
        }
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int pos = c0 + sub + 8 * jj;
            s[jj] = pos <= qpos ? s[jj] * scale : -INFINITY;
            cmax = fmaxf(cmax, s[jj]);
        }
        // the 8 threads of a query sit in consecutive lanes
        cmax = fmaxf(cmax, __shfl_xor(cmax, 1, WAVE));
        cmax = fmaxf(cmax, __shfl_xor(cmax, 2, WAVE));
        cmax = fmaxf(cmax, __shfl_xor(cmax, 4, WAVE));
        const float m_new = fmaxf(m, cmax);
        float psum = 0.f;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const float p = m_new == -INFINITY ? 0.f : expf(s[jj] - m_new);
            Ss[qi * lds_s + sub + 8 * jj] = p;
            psum += p;
        }
        psum += __shfl_xor(psum, 1, WAVE);
        psum += __shfl_xor(psum, 2, WAVE);
        psum += __shfl_xor(psum, 4, WAVE);
        const float corr = m == -INFINITY ? 0.f : expf(m - m_new);
        l = l * corr + psum;
        m = m_new;
        __syncthreads();
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) { acc[g4].x *= corr; acc[g4].y *= corr; acc[g4].z *= corr; acc[g4].w *= corr; }
        for (int j = 0; j < AK; ++j) {
            const float p = Ss[qi * lds_s + j];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                if (4 * (sub + 8 * g4) < dh) {
                    const float4 v = *(const float4 *)(Vs + j * dh + 4 * (sub + 8 * g4));
                    acc[g4].x = fmaf(p, v.x, acc[g4].x); acc[g4].y = fmaf(p, v.y, acc[g4].y);
                    acc[g4].z = fmaf(p, v.z, acc[g4].z); acc[g4].w = fmaf(p, v.w, acc[g4].w);
                }
        }
    }
    const int t = q0 + qi;
    if (t < a.T) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
            if (4 * (sub + 8 * g4) < dh) {
                const size_t at = (size_t)t * nqd + h * dh + 4 * (sub + 8 * g4);
                split_store(a.ohi, a.olo, at, acc[g4].x / l); split_store(a.ohi, a.olo, at + 1, acc[g4].y / l);
                split_store(a.ohi, a.olo, at + 2, acc[g4].z / l); split_store(a.ohi, a.olo, at + 3, acc[g4].w / l);
            }
    }
}

// The same attention over an fp32 cache on the matrix cores, in fp32 (v_mfma_f32_32x32x2_f32: exact fp32
// products, as on the step path), for d_head 64 and 128.  One block: 32 queries of one head; its four
// waves share the cached positions between them (wave w takes the 32-key tiles w, w + 4, ...),
// each flash-style (running maximum and sum per query), and their partial results are merged
// through LDS at the end.  Both products are formed transposed, so that a query lives in a
// lane from start to end:
//   S^T [key, query] = K [key, d] Q^T [d, query]      -- d_head / 2 products
//   O^T [d, query]  += V^T [d, key] P^T [key, query]  -- 16 products per 32 features d; tile dt holds
//                                                        features {(d_head / 32) rho + dt}, so that a lane
//                                                        reads a key's values as one 16-byte piece
// The accumulator layout (lane = column, register r = row 8 (r / 4) + 4 (lane / 32) + r % 4)
// of S^T is, register by register, the operand layout the second product wants for P^T when
// its k index (step i, lane half h) stands for key 8 (i / 4) + 4 h + i % 4: the probabilities
// never leave their registers.  For the first product k index (i, h) stands for feature
// (d_head / 2) h + i, so a lane reads half a row of K as contiguous 16-byte pieces.
// Q and a wave's 32-key tile of K go through LDS, pieces permuted by the row: fetched by the lane that multiplies them, every load
// touches 64 cache lines for 16 bytes each, and what the 8 waves of a compute unit fetch that way does not stay in its 32 KB cache.
// V's rows are contiguous over the lanes and come straight into registers, asked for in front of the first product; K's next tile
// is asked for behind it.  Two waves share a SIMD (80 KB of LDS per block) and one computes while the other waits.
// What bounds it: the fp32 products with long contexts (1024 tokens of 32 heads of 128 cannot take less than 56 us), start, merge
// and end with short ones.  Before (K from each lane's own rows, results stored two bytes at a time) -> this, heads of 128, with the
// placement below: 256 tokens of 40 heads 33.5 -> 21.5 us, 512 of 64 (8 cached) 87 -> 63, 1024 of 32 130 -> 105; the same results.
// F32: for an fp32 model, output in fp32 and no sum longer than on the step path: scores in eight chains, a tile's
// part of the output in four, and what an addition to the running output and sum rounds away is kept beside them.
template <int DH> constexpr int attn_mfma_lds() { return (4 * 32 + 32) * DH * 4; }
template <int DH, bool F32>
__global__ __launch_bounds__(256, F32 ? 1 : 2) void prefill_attn_mfma_kernel(const PrefillAttnArgs a) {
    constexpr int HALF = DH / 2, NT = DH / 32, NWV = 4;
    constexpr int ROWB = DH * 4, PIECES = ROWB / 16, TILE = 32 * ROWB, LOADS = TILE / 1024;
    constexpr int SLOT = (2 + 16 * NT) * WAVE;               // one wave's partial result: m, sum, O^T (floats)
    static_assert(2 * SLOT * 4 <= attn_mfma_lds<DH>(), "the partial results take the place of the tiles");
    extern __shared__ __align__(16) char tiles[];            // [NWV] tiles of K, then Q: 32 rows each
    const int lane = threadIdx.x & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), h = lane / 32, c = lane % 32;
    // Workgroups go to the 8 XCDs round-robin: all query tiles of a head are placed on one XCD (its
    // L2 then holds that head's keys and values once), over all its heads the tiles that see the most keys first: head after
    // head the last heads' longest tiles start last (heads of 128, us: fp32 cache, 256 tokens of 40 heads 26 -> 21.5, 1024 of 32
    // 124 -> 105; fp16 cache, 512 of 64 35 -> 30, 1024 of 32 47 -> 44).
    const int q_tiles = (a.T + 31) / 32;
    const int xcd = blockIdx.x % 8, slot_in_xcd = blockIdx.x / 8, head_groups = (a.n_heads + 7) / 8;
    const int head = (slot_in_xcd % head_groups) * 8 + xcd;
    if (head >= a.n_heads) return;
    const int kvh = head / (a.n_heads / a.n_kv_heads);
    const int q0 = (q_tiles - 1 - slot_in_xcd / head_groups) * 32;
    const int nqd = a.n_heads * DH;
    const float scale = 1.0f / sqrtf((float)DH);
    const size_t head_at = (size_t)kvh * a.cap_ctx * DH;
    const int qpos = a.p0 + q0 + c;                          // cached positions 0 .. qpos are visible to this lane's query
    const int last_key = a.p0 + min(q0 + 31, a.T - 1);       // last position any query of the tile sees
    char *k_tile = tiles + w * TILE, *q_tile = tiles + NWV * TILE;
    auto fetch = [&](int k0) {                               // (a row past the last re-reads it: its scores are masked)
        const int rows = min(32, last_key - k0 + 1);
        const __amdgpu_buffer_rsrc_t rsrc = row_resource((const float *)a.kcache + head_at + (size_t)k0 * DH, (uint32_t)rows * ROWB);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int row = (lane + WAVE * i) / PIECES;
            load16_to_lds(rsrc, k_tile + 1024 * i, (uint32_t)min(row, rows - 1) * ROWB + 16u * (uint32_t)((lane % PIECES) ^ (row & 15)), 0);
        }
    };
    int k0 = 32 * w;
    if (k0 <= last_key) fetch(k0);
#pragma unroll
    for (int i = 0; i < 32 * PIECES / 256; ++i) {
        const int row = (threadIdx.x + 256 * i) / PIECES, piece = threadIdx.x % PIECES;
        const float4 v = global_load_float4(a.q + (size_t)min(q0 + row, a.T - 1) * nqd + (size_t)head * DH + 4 * piece);
        *(float4 *)(q_tile + row * ROWB + 16 * (piece ^ (row & 15))) = v;
    }
    float m = -INFINITY, lsum = 0.f;
    constexpr int CHAINS = F32 ? 8 : 1, PV_CHAINS = F32 ? 4 : 1;
    f32x16 o[NT], rest[NT];
    float lrest = 0.f;
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = rest[dt][r] = 0.f;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");           // Q is in place (K stays under way)

    for (; k0 <= last_key; k0 += 32 * NWV) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                      // K of this tile is in LDS
        float vreg[NT][16];
        auto request_v = [&]() {         // one 16-byte piece per key: features NT c .. NT c + NT - 1, one for each product tile
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const size_t vrow = head_at + (size_t)min(k0 + 8 * (i / 4) + 4 * h + i % 4, last_key) * DH + NT * c;
                if (NT == 4) {
                    const float4 v = global_load_float4((const float *)a.vcache + vrow);
                    vreg[0][i] = v.x; vreg[1][i] = v.y; vreg[2][i] = v.z; vreg[3 % NT][i] = v.w;
                } else {
                    vreg[0][i] = as_global((const float *)a.vcache)[vrow]; vreg[1 % NT][i] = as_global((const float *)a.vcache)[vrow + 1];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if (!F32) request_v();
        f32x16 st;
        {
            f32x16 part[CHAINS];
#pragma unroll
            for (int q = 0; q < CHAINS; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r) part[q][r] = 0.f;
#pragma unroll
            for (int j = 0; j < HALF / 4; ++j) {
                const int at = c * ROWB + 16 * (((PIECES / 2) * h + j) ^ (c & 15));
                const float4 kv = *(const float4 *)(k_tile + at), qv = *(const float4 *)(q_tile + at);
                const float ke[4] = {kv.x, kv.y, kv.z, kv.w}, qe[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) part[(4 * j + e) % CHAINS] = __builtin_amdgcn_mfma_f32_32x32x2f32(ke[e], qe[e], part[(4 * j + e) % CHAINS], 0, 0, 0);
                if (F32 && j % 2 == 1) __builtin_amdgcn_sched_barrier(0);     // (all pieces at once: spills)
            }
#pragma unroll
            for (int n = CHAINS / 2; n > 0; n /= 2)
#pragma unroll
                for (int q = 0; q < n; ++q) part[q] += part[q + n];
            st = part[0];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                    // K has been read
        if (F32) request_v();                                                 // (the chains leave no registers for it before)
        if (k0 + 32 * NWV <= last_key) fetch(k0 + 32 * NWV);
        __builtin_amdgcn_sched_barrier(0);
        float mx = m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = k0 + 8 * (r / 4) + 4 * h + r % 4;
            st[r] = key <= qpos ? st[r] * scale : -INFINITY;
            mx = fmaxf(mx, st[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));                  // the other half of the keys
        // a query that sees none of this tile's keys and none before it: keep exp() away from inf - inf
        const float ref = mx == -INFINITY ? 0.f : mx;
        const float alpha = expf(m - ref);
        float psum = 0.f;
        if (F32) {
#pragma unroll
            for (int r = 0; r < 16; ++r) st[r] = expf(st[r] - ref);
            float two[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) two[r] = st[r] + st[r + 8];
            psum = ((two[0] + two[4]) + (two[1] + two[5])) + ((two[2] + two[6]) + (two[3] + two[7]));
            const float before = lsum * alpha, after = before + psum, moved = after - before;
            lrest = lrest * alpha + ((before - (after - moved)) + (psum - moved));
            lsum = after;
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) { st[r] = expf(st[r] - ref); psum += st[r]; }
            lsum = lsum * alpha + psum;
        }
        m = mx;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt) {
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
            if (F32) {
                f32x16 part[PV_CHAINS];
#pragma unroll
                for (int q = 0; q < PV_CHAINS; ++q)
#pragma unroll
                    for (int r = 0; r < 16; ++r) part[q][r] = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) part[i % PV_CHAINS] = __builtin_amdgcn_mfma_f32_32x32x2f32(vreg[dt][i], st[i], part[i % PV_CHAINS], 0, 0, 0);
                const f32x16 v = (part[0] + part[1 % PV_CHAINS]) + (part[2 % PV_CHAINS] + part[3 % PV_CHAINS]);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float after = o[dt][r] + v[r], moved = after - o[dt][r];
                    rest[dt][r] = rest[dt][r] * alpha + ((o[dt][r] - (after - moved)) + (v[r] - moved));
                    o[dt][r] = after;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vreg[dt][i], st[i], o[dt], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    if (F32) {
        lsum += lrest;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt) o[dt] += rest[dt];
    }
    // merge: waves 2, 3 -> waves 0, 1; then all threads put those two together (over the tiles, which nobody needs any
    // more).  Wave 0 holds key 0, visible to every query, so the merged maximum is finite.
    auto put = [&](int slot) {
        float *b = (float *)tiles + slot * SLOT;
        b[lane] = m; b[WAVE + lane] = lsum;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) b[(2 + 16 * dt + r) * WAVE + lane] = o[dt][r];
    };
    auto take = [&](int slot) {
        const float *b = (const float *)tiles + slot * SLOT;
        const float m2 = b[lane], mt = fmaxf(m, m2);
        const float ref = mt == -INFINITY ? 0.f : mt;
        const float f1 = expf(m - ref), f2 = expf(m2 - ref);
        lsum = lsum * f1 + b[WAVE + lane] * f2;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = o[dt][r] * f1 + b[(2 + 16 * dt + r) * WAVE + lane] * f2;
        m = mt;
    };
    __syncthreads();
    if (last_key >= 2 * 32) {            // (else those waves had no keys)
        if (w >= 2) put(w - 2);
        __syncthreads();
        if (w < 2) take(w);
        __syncthreads();
    }
    if (w < 2) put(w);
    __syncthreads();
    // thread -> query c, features F (tid / 32) .. + F - 1; row rho of product tile dt is feature NT rho + dt
    constexpr int F = DH / 8;
    const float *b0 = (const float *)tiles, *b1 = b0 + SLOT;
    const int qc = threadIdx.x % 32, f0 = F * (threadIdx.x / 32), t = q0 + qc;
    const float mt = fmaxf(b0[qc], b1[qc]);
    const float f1 = expf(b0[qc] - mt), f2 = expf(b1[qc] - mt);
    const float sum = (b0[WAVE + qc] * f1 + b1[WAVE + qc] * f2) + (b0[WAVE + 32 + qc] * f1 + b1[WAVE + 32 + qc] * f2), inv = 1.0f / sum;
    if (t >= a.T) return;
#pragma unroll
    for (int e0 = 0; e0 < F; e0 += 8) {
        float y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int f = f0 + e0 + e, dt = f % NT, rho = f / NT, r = 4 * (rho / 8) + rho % 4, at = (2 + 16 * dt + r) * WAVE + 32 * ((rho / 4) % 2) + qc;
            const float v = b0[at] * f1 + b1[at] * f2;
            y[e] = F32 ? v / sum : v * inv;
        }
        const size_t at = (size_t)t * nqd + head * DH + f0 + e0;
        if (F32) {
            *(f32x4 __attribute__((address_space(1))) *)(a.o32 + at) = f32x4{y[0], y[1], y[2], y[3]};
            *(f32x4 __attribute__((address_space(1))) *)(a.o32 + at + 4) = f32x4{y[4], y[5], y[6], y[7]};
        } else {
            split_store8(a.ohi, a.olo, at, y);
        }
    }
}

// The same over an fp16 cache, for d_head 64 and 128, through v_mfma_f32_32x32x16_f16: sixteen times the rate of the fp32
// products.  The cached keys and values are fp16 and enter as they are; what multiplies them is split in two: a query's
// row, scaled by a power of two that puts its largest element into [2^14, 2^15), and the probabilities times 2^14 go in as
// hi = fp16(x) and lo = fp16(x - hi): 22 bits and an absolute floor 2^-38 below the largest, two products into one fp32
// accumulator.  Error of the output against 64 bits, the fp32 products -> this (2-norm, 64 .. 1024 tokens): 2.06 .. 1.63e-6 ->
// 2.05 .. 1.62e-6, most of it the rounding to the (hi, lo) pair.  Before that rounding, 205 inputs (1 .. 1024 tokens at positions 0
// and 700, heads of 64 and 128, queries of 0.01 .. 25, outlying features, values over 17 octaves, a position that draws most
// of the weight): 0.67 times the fp32 products' error in the geometric mean (their chains of fp32 roundings are longer), at most 0.94
// times from 300 tokens on, larger for 24 of the 145 shorter ones, where few rows decide (at most 2.8 times: 1.2e-7 against 0.4e-7).
// Layouts as above (a query stays in its lane); contraction index (step j, lane half h, element i) stands for feature
// (d_head / 2) h + 8 j + i in the first product and for key 8 ((8 j + i) / 4) + 4 h + i % 4 in the second, which are the eight
// registers 8 j .. 8 j + 7 of S^T.  A wave brings its 32-key tiles of K and of V into LDS of its own (16-byte pieces of a
// key's row permuted by the row, as in the GEMM), each tile as soon as the one before has been read: no barrier, and the
// waits are counted by hand.  What bounds it now is the vector unit (16 exponentials and 32 splits per lane and tile).
// us per chunk and layer, heads of 128, the fp32 products -> this, in one placement: 1024 tokens of 32 heads 143 -> 51, 512 of 64 (8 cached) 98 -> 45,
// 64 of 32 16 -> 8.6; with the present one 44, 30 and 8.0 (the fp32 products 105, 63).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
constexpr float P_SCALE = 16384.f;

__device__ __forceinline__ void split_f16(float x, _Float16 &hi, _Float16 &lo) {
    hi = (_Float16)x;
    lo = (_Float16)(x - (float)hi);
}

template <int DH>
__global__ __launch_bounds__(256, 2) void prefill_attn_f16_kernel(const PrefillAttnArgs a) {
    constexpr int NT = DH / 32, NJ = DH / 16, NWV = 4;
    constexpr int ROWB = DH * 2, PIECES = ROWB / 16, TILE = 32 * ROWB, LOADS = TILE / 1024;
    constexpr int SLOT = (2 + 16 * NT) * WAVE * 4;           // one wave's partial result: m, sum, O^T
    static_assert(2 * SLOT <= NWV * 2 * TILE + 32 * DH * 4, "the partial results take the place of the tiles and of Q");
    extern __shared__ __align__(16) char tiles[];            // [NWV][K, V][TILE], then Q: 32 rows of fp32, pieces permuted by the row
    const int lane = threadIdx.x & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), h = lane / 32, c = lane % 32;
    const int q_tiles = (a.T + 31) / 32;
    const int xcd = blockIdx.x % 8, slot_in_xcd = blockIdx.x / 8, head_groups = (a.n_heads + 7) / 8;   // (placement as above)
    const int head = (slot_in_xcd % head_groups) * 8 + xcd;
    if (head >= a.n_heads) return;
    const int kvh = head / (a.n_heads / a.n_kv_heads);
    const int q0 = (q_tiles - 1 - slot_in_xcd / head_groups) * 32;
    const int nqd = a.n_heads * DH;
    const int qpos = a.p0 + q0 + c;                          // cached positions 0 .. qpos are visible to this lane's query
    const int last_key = a.p0 + min(q0 + 31, a.T - 1);       // last position any query of the tile sees

    // one head's rows 0 .. last_key; a row past the last re-reads it (its scores are masked)
    const size_t head_at = (size_t)kvh * a.cap_ctx * DH;
    const __amdgpu_buffer_rsrc_t k_rsrc = row_resource((const uint16_t *)a.kcache + head_at, (uint32_t)(last_key + 1) * ROWB);
    const __amdgpu_buffer_rsrc_t v_rsrc = row_resource((const uint16_t *)a.vcache + head_at, (uint32_t)(last_key + 1) * ROWB);
    char *k_tile = tiles + (2 * w) * TILE, *v_tile = k_tile + TILE;
    auto swizzle = [](int row) { return DH == 128 ? row & 15 : (row & 7) ^ ((row >> 3) & 1); };
    auto fetch = [&](__amdgpu_buffer_rsrc_t rsrc, char *to, int k0) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int row = (lane + WAVE * i) / PIECES;
            load16_to_lds(rsrc, to + 1024 * i, (uint32_t)min(k0 + row, last_key) * ROWB + 16u * (uint32_t)((lane % PIECES) ^ swizzle(row)), 0);
        }
    };
    int k0 = 32 * w;
    if (k0 <= last_key) { fetch(k_rsrc, k_tile, k0); fetch(v_rsrc, v_tile, k0); }

    // Q through LDS: fetched by the row (a lane's own row fetched directly makes every load touch 64 cache lines)
    char *q_tile = tiles + NWV * 2 * TILE;
    constexpr int Q_PIECES = DH / 4;
#pragma unroll
    for (int i = 0; i < 32 * Q_PIECES / 256; ++i) {
        const int row = (threadIdx.x + 256 * i) / Q_PIECES, piece = threadIdx.x % Q_PIECES;
        const float4 v = global_load_float4(a.q + (size_t)min(q0 + row, a.T - 1) * nqd + (size_t)head * DH + 4 * piece);
        *(float4 *)(q_tile + row * (DH * 4) + 16 * (piece ^ (row & 15))) = v;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");           // (the tiles stay under way)
    // this lane's operand values of Q: query q0 + c, features (DH / 2) h + 8 j + i
    f16x8 qh[NJ], ql[NJ];
    float unscale;
    {
        float q[NJ][8], top = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 8; e += 4) {
                const float4 v = *(const float4 *)(q_tile + c * (DH * 4) + 16 * (((DH / 8) * h + 2 * j + e / 4) ^ (c & 15)));
                q[j][e] = v.x; q[j][e + 1] = v.y; q[j][e + 2] = v.z; q[j][e + 3] = v.w;
            }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) top = fmaxf(top, fabsf(q[j][e]));
        top = fmaxf(top, __shfl_xor(top, 32));
        int ex = 15;
        if (top > 0.f && top < INFINITY) (void)frexpf(top, &ex);
        ex = max(ex, -100);
        const float up = ldexpf(1.f, 15 - ex);
        unscale = ldexpf(1.f, ex - 15) * (1.0f / sqrtf((float)DH));
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                _Float16 hi, lo;
                split_f16(q[j][e] * up, hi, lo);
                qh[j][e] = hi; ql[j][e] = lo;
            }
    }
    float m = -INFINITY, lsum = 0.f;
    f32x16 o[NT];
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;

    for (; k0 <= last_key; k0 += 32 * NWV) {
        const int next = k0 + 32 * NWV;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");          // K of this tile is in LDS (V's loads are younger)
        f32x16 st;
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const f16x8 k = __builtin_bit_cast(f16x8, *(const u32x4 *)(k_tile + c * ROWB + 16 * (((PIECES / 2) * h + j) ^ swizzle(c))));
            st = __builtin_amdgcn_mfma_f32_32x32x16_f16(k, qh[j], st, 0, 0, 0);
            st = __builtin_amdgcn_mfma_f32_32x32x16_f16(k, ql[j], st, 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                    // and has been read
        if (next <= last_key) fetch(k_rsrc, k_tile, next);
        float mx = m;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = k0 + 8 * (r / 4) + 4 * h + r % 4;
            st[r] = key <= qpos ? st[r] * unscale : -INFINITY;
            mx = fmaxf(mx, st[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));                  // the other half of the keys
        // a query that sees none of this tile's keys and none before it: keep exp() away from inf - inf
        const float ref = mx == -INFINITY ? 0.f : mx;
        const float alpha = expf(m - ref);
        float psum = 0.f;
        f16x8 ph[2], pl[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = expf(st[r] - ref);
            psum += p;
            _Float16 hi, lo;
            split_f16(p * P_SCALE, hi, lo);
            ph[r / 8][r % 8] = hi; pl[r / 8][r % 8] = lo;
        }
        lsum = lsum * alpha + psum;
        m = mx;
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int dt = 0; dt < NT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
        }
        if (next <= last_key) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");   // V of this tile is in LDS (the next K's loads are younger)
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // features NT c .. NT c + NT - 1 of eight keys, then turned round: eight keys of each feature
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            _Float16 v[8][NT];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = 8 * ((8 * j + i) / 4) + 4 * h + i % 4, byte = 2 * NT * c;
                const char *from = v_tile + row * ROWB + 16 * ((byte / 16) ^ swizzle(row)) + byte % 16;
                typedef _Float16 f16xn __attribute__((ext_vector_type(NT)));
                const f16xn x = *(const f16xn *)from;
#pragma unroll
                for (int dt = 0; dt < NT; ++dt) v[i][dt] = x[dt];
            }
#pragma unroll
            for (int dt = 0; dt < NT; ++dt) {
                f16x8 vt;
#pragma unroll
                for (int i = 0; i < 8; ++i) vt[i] = v[i][dt];
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vt, ph[j], o[dt], 0, 0, 0);
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vt, pl[j], o[dt], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (next <= last_key) fetch(v_rsrc, v_tile, next);
    }

    // merge: waves 2, 3 -> waves 0, 1; then all threads put those two together (over the tiles, which nobody needs any
    // more).  Wave 0 holds key 0, visible to every query, so the merged maximum is finite.
    auto put = [&](int slot) {
        float *b = (float *)(tiles + slot * SLOT);
        b[lane] = m; b[WAVE + lane] = lsum;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) b[(2 + 16 * dt + r) * WAVE + lane] = o[dt][r];
    };
    auto take = [&](int slot) {
        const float *b = (const float *)(tiles + slot * SLOT);
        const float m2 = b[lane], mt = fmaxf(m, m2);
        const float ref = mt == -INFINITY ? 0.f : mt;
        const float f1 = expf(m - ref), f2 = expf(m2 - ref);
        lsum = lsum * f1 + b[WAVE + lane] * f2;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = o[dt][r] * f1 + b[(2 + 16 * dt + r) * WAVE + lane] * f2;
        m = mt;
    };
    __syncthreads();
    if (last_key >= 2 * 32) {            // (else those waves had no keys)
        if (w >= 2) put(w - 2);
        __syncthreads();
        if (w < 2) take(w);
        __syncthreads();
    }
    if (w < 2) put(w);
    __syncthreads();
    // thread -> query c, features F (tid / 32) .. + F - 1; row rho of product tile dt is feature NT rho + dt
    constexpr int F = DH / 8;
    const float *b0 = (const float *)tiles, *b1 = (const float *)(tiles + SLOT);
    const int qc = threadIdx.x % 32, f0 = F * (threadIdx.x / 32), t = q0 + qc;
    const float mt = fmaxf(b0[qc], b1[qc]);
    const float f1 = expf(b0[qc] - mt), f2 = expf(b1[qc] - mt);
    const float inv = 1.0f / (((b0[WAVE + qc] + b0[WAVE + 32 + qc]) * f1 + (b1[WAVE + qc] + b1[WAVE + 32 + qc]) * f2) * P_SCALE);
#pragma unroll
    for (int e0 = 0; e0 < F; e0 += 8) {
        float y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int f = f0 + e0 + e, dt = f % NT, rho = f / NT, r = 4 * (rho / 8) + rho % 4, at = (2 + 16 * dt + r) * WAVE + 32 * ((rho / 4) % 2) + qc;
            y[e] = (b0[at] * f1 + b1[at] * f2) * inv;
        }
        if (t < a.T) split_store8(a.ohi, a.olo, (size_t)t * nqd + head * DH + f0 + e0, y);
    }
}

// ------------------------------------------------------------------ fp32 models
// The same pass in fp32 (v_mfma_f32_16x16x4_f32): these models' token-by-token pass takes a chain of dependent phases per token
// whatever they weigh.  A block of four waves makes a tile of 16 TT tokens x 16 NT columns (PE_SWIGLU: 16 units, gate and up); the
// waves take every fourth piece of 16 k, straight from memory into registers, U pieces ahead.  A lane holds four consecutive k
// of its row, so product c of a piece contracts k = 4 (lane / 16) + c, in accumulators of its own; after U pieces they are added up, and
// what that addition to the running sum rounds away is kept beside it.  So no sum is longer than in the matrix-vector kernel:
// logits behind 3 .. 1030 tokens of four models (256 .. 2048 wide, six seeds each) differ from 64 bits by 0.98 times what the
// token-by-token pass leaves (0.90 .. 1.08; with one chain per product and plain sums 1.3, up to 1.5).
// RMSNorm has no pass of its own: x * gain is what is multiplied, the sum of squares comes along (a block reads its tokens' rows
// from end to end), and the results are scaled.
// Bound by latency: 16 tokens of two layers of 256 wide, 13 launches, 812 us token by token -> 74 with the logits; 1030 tokens 55 700 -> 271,
// of two layers of 2048 wide 97 000 -> 2700.  Few tokens, 768 .. 2048 wide: the 48 .. 128 blocks of a product fetch its rows in
// pieces of 64 bytes, 2 TB/s where the matrix-vector kernels reach 4.5, so two tokens may go one by one.
enum { PE_RESID = 3 };
struct Prefill32Args : PrefillGemmArgs {
    const float *x;              // [T, K]
    const float *gain;           // [K] or null: no normalisation
    const float *W32, *W232;     // [N, K]; "up" (PE_SWIGLU)
    float *y;                    // PE_RESID: [T, N], added to in place; PE_SWIGLU: [T, N]
    float eps;
};

template <int EPI, int TT, int NT>
__global__ __launch_bounds__(256) void prefill32_gemm_kernel(const Prefill32Args a) {
    constexpr int U = TT * NT == 1 ? 4 : 2;
    static_assert(EPI != PE_SWIGLU || NT == 2, "gate, up");
    __shared__ float4 sums[4][NT * TT][WAVE];
    __shared__ float squares[4][TT][WAVE];
    const int lane = threadIdx.x & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;       // all token tiles of a column tile on one XCD
    const int tile_y = (slot / a.t_tiles) * 8 + xcd, t0 = (slot % a.t_tiles) * 16 * TT;
    if (tile_y >= a.n_tiles) return;
    const int n0 = tile_y * 16 * (EPI == PE_SWIGLU ? 1 : NT);
    const uint32_t row_bytes = (uint32_t)a.K * 4u, none = 0xFFFFFFF0u;      // (past every extent: zeros, no traffic)
    const __amdgpu_buffer_rsrc_t xr = row_resource(a.x, (uint32_t)a.T * row_bytes), gr = row_resource(a.gain, a.gain != nullptr ? row_bytes : 0u);
    const __amdgpu_buffer_rsrc_t wr = row_resource(a.W32, (uint32_t)a.N * row_bytes);
    const __amdgpu_buffer_rsrc_t ur = row_resource(EPI == PE_SWIGLU ? a.W232 : a.W32, (uint32_t)a.N * row_bytes);
    uint32_t x_at[TT], w_at[NT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) { const int t = t0 + 16 * tt + lane % 16; x_at[tt] = t < a.T ? (uint32_t)t * row_bytes : none; }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) { const int n = n0 + lane % 16 + (EPI == PE_SWIGLU ? 0 : 16 * nt); w_at[nt] = n < a.N ? (uint32_t)n * row_bytes : none; }
    const int pieces = a.K / 16, mine = (pieces - w + 3) / 4;    // piece i of this wave: 4 i + w
    const bool normed = a.gain != nullptr;
    struct Batch { float4 x[U][TT], w[U][NT], g[U]; };
    auto as_float4 = [](u32x4 v) { return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)); };
    auto request = [&](Batch &b, int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool there = i0 + u < mine;
            const uint32_t k = 64u * (uint32_t)(4 * (i0 + u) + w) + 16u * (uint32_t)(lane / 16);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) b.x[u][tt] = as_float4(buffer_load16(xr, there && x_at[tt] != none ? x_at[tt] + k : none));
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) b.w[u][nt] = as_float4(buffer_load16(EPI == PE_SWIGLU && nt == 1 ? ur : wr, there && w_at[nt] != none ? w_at[nt] + k : none));
            if (normed) b.g[u] = as_float4(buffer_load16(gr, there ? k : none));
        }
    };
    f32x4 total[NT][TT], rest[NT][TT];
    float ss[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        ss[tt] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            total[nt][tt] = rest[nt][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    auto multiply = [&](const Batch &b) {
        f32x4 acc[2][4][NT][TT];                                 // (two pieces of U take turns: chains of U / 2 products)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float xv[TT][4];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const float4 v = b.x[u][tt];
                xv[tt][0] = v.x; xv[tt][1] = v.y; xv[tt][2] = v.z; xv[tt][3] = v.w;
                if (normed) {
                    ss[tt] += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
                    xv[tt][0] *= b.g[u].x; xv[tt][1] *= b.g[u].y; xv[tt][2] *= b.g[u].z; xv[tt][3] *= b.g[u].w;
                }
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float wv[4] = {b.w[u][nt].x, b.w[u][nt].y, b.w[u][nt].z, b.w[u][nt].w};
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[u % 2][c][nt][tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[c], xv[tt][c], u < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[u % 2][c][nt][tt], 0, 0, 0);
            }
        }
        // what an addition to the running sum rounds away is kept beside it
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                auto four = [&](int q) { return (acc[q][0][nt][tt] + acc[q][1][nt][tt]) + (acc[q][2][nt][tt] + acc[q][3][nt][tt]); };
                const f32x4 v = four(0) + four(1);
                const f32x4 t = total[nt][tt] + v, moved = t - total[nt][tt];
                rest[nt][tt] += (total[nt][tt] - (t - moved)) + (v - moved);
                total[nt][tt] = t;
            }
    };
    Batch b0, b1;
    request(b0, 0);
    for (int i = 0; i < mine; i += 2 * U) {
        request(b1, i + U);
        multiply(b0);
        request(b0, i + 2 * U);
        multiply(b1);
    }

    // lane -> token l % 16 of a piece, register r -> column 4 (l / 16) + r; the waves' shares in wave order
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const f32x4 v = total[nt][tt] + rest[nt][tt];
            sums[w][nt * TT + tt][lane] = make_float4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) squares[w][tt][lane] = ss[tt];
    __syncthreads();
    constexpr int FIRST = EPI == PE_SWIGLU ? TT : NT * TT;       // (gate and up go together)
    for (int e = w; e < FIRST; e += 4) {
        const int nt = e / TT, tt = e % TT, t = t0 + 16 * tt + lane % 16, nc = n0 + 16 * nt + 4 * (lane / 16);
        float rs = 1.f;
        if (normed) {
            float sq = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float part = 0.f;
#pragma unroll
                for (int g = 0; g < 4; ++g) part += squares[q][tt][16 * g + lane % 16];
                sq += part;
            }
            rs = 1.0f / sqrtf(sq / (float)a.K + a.eps);
        }
        auto sum = [&](int at) {
            const float4 p = sums[0][at][lane], q = sums[1][at][lane], r = sums[2][at][lane], s = sums[3][at][lane];
            return f32x4{(p.x + q.x) + (r.x + s.x), (p.y + q.y) + (r.y + s.y), (p.z + q.z) + (r.z + s.z), (p.w + q.w) + (r.w + s.w)} * rs;
        };
        const f32x4 v = sum(e);
        if (t >= a.T || nc >= a.N) continue;
        if (EPI == PE_QKV) {
            const QkvRows rows(a, nc);
            rows.put(a, t, v, rows.rotates ? rows.angles(a, t) : make_float4(1.f, 0.f, 1.f, 0.f));
        } else {
            f32x4 __attribute__((address_space(1))) *to = (f32x4 __attribute__((address_space(1))) *)(a.y + (size_t)t * a.N + nc);
            if (EPI == PE_RESID) {
                *to = *to + v;
            } else {
                const f32x4 up = sum(TT + tt);
                f32x4 y;
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = v[r] / (1.0f + expf(-v[r])) * up[r];
                *to = y;
            }
        }
    }
}

// The chunk's embeddings and its rotary table.
__global__ __launch_bounds__(256) void prefill32_start_kernel(const float *embed, const int32_t *tokens, float *h, int d, const double *inv_freq, int p0, int T, int half, float2 *table) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < T * (d / 4)) {
        const float4 v = global_load_float4(embed + (size_t)as_global(tokens)[i / (d / 4)] * d + 4 * (i % (d / 4)));
        *(f32x4 __attribute__((address_space(1))) *)(h + 4 * (size_t)i) = f32x4{v.x, v.y, v.z, v.w};
    }
    if (i < T * half) table[i] = rope_cos_sin(inv_freq, i % half, p0 + i / half);
}

template <int DH> constexpr int attn_f16_lds() { return 4 * 2 * 32 * DH * 2 + 32 * DH * 4; }

}  // namespace

namespace spdk {

size_t prefill_attn_lds(int d_head) { return (size_t)(AQ * (d_head + 4) + AK * (d_head + 4) + AK * d_head + AQ * (AK + 1)) * sizeof(float); }

// The tile shapes: one block per compute unit, k steps of 64.  Gate and up, the widest product, leaves the chip idlest where its tiles do
// not come out even (7B widths: 86 tiles of 256 columns; three rounds at 1024 tokens where 2.7 would do), and has shapes of its own:
// its time over 41 lengths from 8 to 1024 and four widths 0.91 in the geometric mean, 0.61 at best (7B, 384 tokens: 175 -> 107 us), the four
// products' of a layer 0.96.  The other products were not measured with them; entry 11 is entry 4 with its waves the other way round, which
// gate and up needs for its halves, and of the two the faster per step.  What a step takes a block: `step_us` when all compute units
// have one, `alone_us` when few do (fitted to the sweep below; at 128 tokens the products bound it, at 32 the loads).
constexpr int KS = 64;
struct Tile { int bm, bn, stages, waves; double step_us, alone_us; };
constexpr Tile TILES[] = {{32, 256, 4, 8, 0.75, 0.75}, {64, 256, 3, 8, 1.00, 0.89}, {64, 384, 2, 8, 1.62, 1.52}, {128, 256, 2, 8, 1.60, 1.46},
                          {128, 384, 2, 8, 2.30, 2.10}, {64, 128, 4, 4, 0.62, 0.45}, {32, 128, 5, 2, 0.51, 0.51},
                          // gate and up only
                          {64, 96, 5, 4, 0.58, 0.45}, {64, 192, 4, 8, 0.86, 0.73}, {128, 192, 2, 8, 1.49, 1.10}, {128, 320, 2, 8, 1.92, 1.72},
                          {128, 384, 2, 8, 2.16, 1.95}, {192, 192, 2, 8, 1.78, 1.53}, {192, 256, 2, 8, 2.16, 1.87}};
constexpr int N_ANY = 7, N_TILES = 14;
constexpr int tile_lds(int i) { return TILES[i].stages * (2 * TILES[i].bm + TILES[i].bn) * KS * 2; }

typedef void (*GemmFn)(PrefillGemmArgs);
template <int EPI> static GemmFn gemm_kernel(int tile) {
    constexpr bool GU = EPI == PE_SWIGLU, QKV = EPI == PE_QKV;    // gate and up side by side take an even number of column pieces per wave
    constexpr int ANY = QKV ? (int)PE_PART : EPI;
    switch (tile) {
        case 0: return GU ? nullptr : prefill_gemm_kernel<GU ? (int)PE_PART : EPI, 1, 8, 2, 2, KS, 4, true>;
        case 1: return prefill_gemm_kernel<EPI, 2, 4, 2, 4, KS, 3, true>;
        case 2: return GU ? nullptr : prefill_gemm_kernel<GU ? (int)PE_PART : EPI, 2, 4, 2, 6, KS, 2, true>;
        case 3: return prefill_gemm_kernel<EPI, 2, 4, 4, 4, KS, 2, false>;
        case 4: return GU ? nullptr : prefill_gemm_kernel<GU ? (int)PE_PART : EPI, 2, 4, 4, 6, KS, 2, false>;
        case 5: return prefill_gemm_kernel<EPI, 2, 2, 2, 4, KS, 4, true>;
        case 6: return prefill_gemm_kernel<EPI, 1, 2, 2, 4, KS, 5, true>;
        case 7: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 1, 1, 6, KS, 5, true>;
        case 8: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 2, 1, 6, KS, 4, true>;
        case 9: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 2, 2, 6, KS, 2, false>;
        case 10: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 2, 2, 10, KS, 2, false>;
        case 11: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 2, 2, 12, KS, 2, false>;
        case 12: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 2, 3, 6, KS, 2, false>;
        default: return QKV ? nullptr : prefill_gemm_kernel<ANY, 4, 2, 3, 8, KS, 2, false>;
    }
}

// The tile shape and the number of blocks that share a tile's k range: the cheapest by estimate.  A block's steps take
// step_us each.  All token tiles of a column run on one of the 8 XCDs, so the busiest XCD's blocks count, in rounds over its
// compute units: counted over the whole chip 22 columns x 11 token tiles seem to fit 256 compute units once, and take two
// rounds (7B output projection, 700 tokens, 64 x 384 in two splits: 114 us; 128 x 256: 63).  A last, partly empty round takes
// between alone_us and step_us a step (128 x 256 at 1.25 and 1.75 rounds: 3.2 and 3.5 us).  The weights come at
// 7.8 TB/s at best (part of them from the memory-side cache); partial sums are written and read at 4.6 TB/s
// and, where the product has an epilogue, cost one more launch.
// Held against every shape and split, products of the 1B, 7B, 13B and 70B widths: the four products of a layer take 1.0 % longer than with
// the best choice for each at the 28 lengths the constants were fitted to and 0.9 % at 14 others (at most 8 %).
static PrefillCut cut_product(const PrefillChunk &c, const PrefillForce &force, int T, int N, int mats, int K, int epi, size_t part_floats) {
    PrefillCut best{};
    double best_us = 1e30;
    for (int tile = 0; tile < (epi == PE_SWIGLU ? N_TILES : N_ANY); ++tile) {
        if (force.tile_1 != 0 && tile != force.tile_1 - 1) continue;
        const Tile &t = TILES[tile];
        const int t_tiles = (T + t.bm - 1) / t.bm, steps = K / KS;
        const bool can_fuse = epi == PE_QKV || (epi == PE_SWIGLU && gemm_kernel<PE_SWIGLU>(tile) != nullptr);
        for (int want = 1; want <= 16; ++want) {
            const int split_steps = (steps + want - 1) / want, splits = (steps + split_steps - 1) / split_steps;
            const bool fused = can_fuse && splits == 1;
            if (want > 1 && split_steps < 4) break;
            if (force.tile_1 != 0 && splits != force.splits) continue;
            if (!fused && (size_t)splits * T * N * mats > part_floats) continue;
            const int n_tiles = fused && epi == PE_SWIGLU ? (2 * N + t.bn - 1) / t.bn : (N + t.bn - 1) / t.bn;
            const int cols = n_tiles * splits * (fused ? 1 : mats);
            const double rounds = (double)((cols + 7) / 8) * t_tiles / (c.num_cu / 8.0), whole = std::floor(rounds), rest = rounds - whole;
            const double step = whole * t.step_us + (rest > 0.0 ? t.alone_us + (t.step_us - t.alone_us) * rest : 0.0);
            double us = std::max(step * split_steps, (double)N * K * mats * 2 / 7.8e6);
            if (!fused) us += (double)splits * T * N * mats * 8 / 4.6e6 + (epi == PE_PART ? 0.0 : 2.2);
            if (us < best_us) { best_us = us; best = PrefillCut{tile, t_tiles, n_tiles, splits, split_steps, fused}; }
        }
    }
    if (best.t_tiles == 0 && force.tile_1 != 0) return cut_product(c, PrefillForce{0, 0}, T, N, mats, K, epi, part_floats);   // (what was asked for does not fit)
    return best;
}

void prefill_cuts(const PrefillChunk &c, int T, PrefillCut (&cut)[4]) {
    const int d = c.d_model, dh = d / c.n_heads, nq = c.n_heads * dh, nkv = c.n_kv_heads * dh;
    const size_t room = (size_t)PREFILL_CHUNK * (d + nq);
    cut[0] = cut_product(c, c.force[0], T, nq + 2 * nkv, 1, d, PE_QKV, (size_t)PREFILL_CHUNK * c.d_ffn);
    cut[1] = cut_product(c, c.force[1], T, d, 1, nq, PE_PART, room);
    cut[2] = cut_product(c, c.force[2], T, c.d_ffn, 2, d, PE_SWIGLU, room);
    cut[3] = cut_product(c, c.force[3], T, d, 1, c.d_ffn, PE_PART, room);
}

int prefill_tile(int tile, int &tokens, int &columns) { tokens = TILES[tile].bm; columns = TILES[tile].bn; return N_TILES; }

static void launch_gemm(hipStream_t s, GemmFn kernel, PrefillGemmArgs &a, const PrefillCut &cut, int mats) {
    a.t_tiles = cut.t_tiles; a.n_tiles = cut.n_tiles; a.splits = cut.splits; a.split_steps = cut.split_steps;
    a.rotate = cut.t_tiles == 1 && a.K >= 4096 && (a.K & (a.K - 1)) == 0;
    const int cols = cut.n_tiles * mats * cut.splits;
    hipLaunchKernelGGL(kernel, dim3((cols + 7) / 8 * 8 * cut.t_tiles), dim3(TILES[cut.tile].waves * WAVE), tile_lds(cut.tile), s, a);
}

hipError_t prefill_init() {
    hipError_t e = hipFuncSetAttribute((const void *)prefill_attn_kernel<float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)prefill_attn_lds(128));
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_attn_kernel<half_t>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)prefill_attn_lds(128));
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_attn_f16_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, attn_f16_lds<128>());
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_attn_mfma_kernel<128, false>, hipFuncAttributeMaxDynamicSharedMemorySize, attn_mfma_lds<128>());
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)prefill_attn_mfma_kernel<128, true>, hipFuncAttributeMaxDynamicSharedMemorySize, attn_mfma_lds<128>());
    for (int tile = 0; tile < N_TILES; ++tile)
        for (GemmFn k : {gemm_kernel<PE_PART>(tile), gemm_kernel<PE_QKV>(tile), gemm_kernel<PE_SWIGLU>(tile)})
            if (e == hipSuccess && k != nullptr) e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds(tile));
    return e;
}

hipError_t prefill_attention(hipStream_t s, int kv_half, const float *q, const void *kcache, const void *vcache, uint16_t *ohi, uint16_t *olo,
                             int T, int p0, int n_heads, int n_kv_heads, int dh, int cap_ctx, float *out32) {
    const PrefillAttnArgs at{q, kcache, vcache, ohi, olo, out32, T, p0, n_heads, n_kv_heads, dh, cap_ctx};
    const dim3 mfma_grid(((T + 31) / 32) * ((n_heads + 7) / 8) * 8), plain_grid((T + AQ - 1) / AQ, n_heads);
    if (kv_half) {
        if (dh == 128) hipLaunchKernelGGL(prefill_attn_f16_kernel<128>, mfma_grid, dim3(256), attn_f16_lds<128>(), s, at);
        else if (dh == 64) hipLaunchKernelGGL(prefill_attn_f16_kernel<64>, mfma_grid, dim3(256), attn_f16_lds<64>(), s, at);
        else hipLaunchKernelGGL(prefill_attn_kernel<half_t>, plain_grid, dim3(ANT), prefill_attn_lds(dh), s, at);
    } else {
        if (dh == 128 && out32) hipLaunchKernelGGL((prefill_attn_mfma_kernel<128, true>), mfma_grid, dim3(256), attn_mfma_lds<128>(), s, at);
        else if (dh == 64 && out32) hipLaunchKernelGGL((prefill_attn_mfma_kernel<64, true>), mfma_grid, dim3(256), attn_mfma_lds<64>(), s, at);
        else if (out32) return hipErrorInvalidValue;
        else if (dh == 128) hipLaunchKernelGGL((prefill_attn_mfma_kernel<128, false>), mfma_grid, dim3(256), attn_mfma_lds<128>(), s, at);
        else if (dh == 64) hipLaunchKernelGGL((prefill_attn_mfma_kernel<64, false>), mfma_grid, dim3(256), attn_mfma_lds<64>(), s, at);
        else hipLaunchKernelGGL(prefill_attn_kernel<float>, plain_grid, dim3(ANT), prefill_attn_lds(dh), s, at);
    }
    return hipGetLastError();
}

// What is left of the last layer for the prefix's last token, whose query is in `q`: attention, output projection and feed-forward through the
// timestep's own operators, on row T - 1 of c.h in place.
static hipError_t last_token(hipStream_t s, const PrefillChunk &c, int dtype, const float *q, float *att, float *u) {
    const spd_layer_weights &w = c.layers[c.n_layers - 1];
    const int T = c.T, d = c.d_model, dh = d / c.n_heads, nq = c.n_heads * dh;
    float *h = c.h + (size_t)(T - 1) * d;
    const char *kv = c.kv + (size_t)(2 * (c.n_layers - 1)) * c.kv_layer_bytes;
    const AttnArgs at{q, kv, kv + c.kv_layer_bytes, att, c.attn_part, nullptr, nullptr, c.p0 + T, c.n_heads, c.n_kv_heads, dh, c.cap_ctx, 0, c.max_splits};
    hipError_t e = attention(s, c.kv_half ? SPD_DTYPE_FP16 : SPD_DTYPE_FP32, at);
    GemvArgs o{};
    o.W = w.wo; o.x = att; o.resid = o.y = h; o.rows = d; o.cols = nq;
    if (e == hipSuccess) e = gemv(s, dtype, EPI_RESID, o, c.num_cu);
    GemvArgs f{};
    f.W = w.w_gate; f.W2 = w.w_up; f.gain = w.ffn_norm; f.eps = c.eps; f.x = h; f.y = u; f.rows = c.d_ffn; f.cols = d;
    if (e == hipSuccess) e = gemv(s, dtype, EPI_SWIGLU, f, c.num_cu);
    GemvArgs dn{};
    dn.W = w.w_down; dn.x = u; dn.resid = dn.y = h; dn.rows = d; dn.cols = c.d_ffn;
    if (e == hipSuccess) e = gemv(s, dtype, EPI_RESID, dn, c.num_cu);
    return e;
}

// The last layer's query rows stay in the product of all tokens while that costs less than a launch of their own (a matrix-vector product over
// them, in fp32): up to this many tokens x rows x k.  A whole pass over two layers, rows in the product against by themselves: 1B widths
// 0.92 (8 tokens) .. 0.99 (512); 7B 0.94 (8) .. 0.98 (160), 1.01 (192), 1.04 (512); 13B 0.96 .. 0.98 (128), 1.01 (192); 70B 0.98 (8) .. 0.99 (64), 1.01 (96).
constexpr long long LAST_QUERY_WITH = 3000000000ll;
bool prefill_own_query(const PrefillChunk &c, int T) {
    return c.force_query != 0 ? c.force_query == 2 : (long long)T * c.d_model * c.d_model > LAST_QUERY_WITH;
}

// One chunk of T prefix tokens at positions p0 .. p0 + T - 1 through the whole stack.  Only the prefix's last token goes
// on into the final norm and the LM head, and nothing reads what the last layer makes of the others but their keys and values.
// So that layer's big product has the key and value rows only (with few tokens the query rows too: LAST_QUERY_WITH), and the rest
// of it runs for that one token, through the timestep's own operators (fp32 activations); a chunk that is not the prefix's last ends
// with the keys and values.  Bound of that tail: the layer's weights at HBM's rate, whatever T is.  us for a whole pass, all tokens
// -> this: four layers of the 7B widths, 1024 tokens 3292 -> 2705, 64 tokens 658 -> 626; three of the 13B, 256 tokens 1277 -> 1063.
// On return (stream order) the caches are extended and, after the final chunk, c.h holds the last token's residual stream after
// the last layer in row T - 1; the caller finishes that token (final norm + LM head).
hipError_t prefill_chunk(hipStream_t s, const PrefillChunk &c) {
    const int T = c.T, d = c.d_model, dh = d / c.n_heads, nq = c.n_heads * dh, nkv = c.n_kv_heads * dh;
    PrefillCut cut[4];
    prefill_cuts(c, T, cut);
    const PrefillCut &cut_o = cut[1], &cut_gu = cut[2], &cut_down = cut[3];
    const bool own_query = prefill_own_query(c, T);
    const PrefillCut cut_last = own_query ? cut_product(c, c.force[0], T, 2 * nkv, 1, d, PE_QKV, (size_t)PREFILL_CHUNK * c.d_ffn) : cut[0];
    for (int l = 0; l < c.n_layers; ++l) {
        const spd_layer_weights &w = c.layers[l];
        const bool last = l == c.n_layers - 1;
        PrefillNormArgs n{};
        n.h = c.h; n.gain = (const uint16_t *)w.attn_norm; n.hi = c.xhi; n.lo = c.xlo; n.T = T; n.d = d; n.eps = c.eps; n.part = c.part;
        if (l == 0) {
            n.embed = (const uint16_t *)c.embed; n.tokens = c.prefix + c.p0;
            n.inv_freq = c.inv_freq; n.rope = c.rope; n.p0 = c.p0; n.half = dh / 2;
            hipLaunchKernelGGL((prefill_norm_kernel<true>), dim3(T), dim3(norm_threads(d)), 0, s, n);
        } else {
            n.splits = cut_down.splits;
            hipLaunchKernelGGL((prefill_norm_kernel<false>), dim3(T), dim3(norm_threads(d)), 0, s, n);
        }
        PrefillGemmArgs g{};
        g.n_q_rows = last && own_query ? 0 : nq; g.n_kv_rows = nkv; g.N = g.n_q_rows + 2 * nkv;
        g.xhi = c.xhi; g.xlo = c.xlo; g.W = (const uint16_t *)w.wqkv + (size_t)(nq - g.n_q_rows) * d; g.T = T; g.K = d; g.part = (float *)c.uhi;
        g.q = c.q; g.kcache = c.kv + (size_t)(2 * l) * c.kv_layer_bytes;
        g.vcache = c.kv + (size_t)(2 * l + 1) * c.kv_layer_bytes; g.kv_half = c.kv_half;
        g.rope = c.rope; g.d_head = dh; g.cap_ctx = c.cap_ctx; g.p0 = c.p0;
        const PrefillCut &cut_qkv = last ? cut_last : cut[0];
        launch_gemm(s, cut_qkv.fused ? gemm_kernel<PE_QKV>(cut_qkv.tile) : gemm_kernel<PE_PART>(cut_qkv.tile), g, cut_qkv, 1);
        if (!cut_qkv.fused) hipLaunchKernelGGL(prefill_qkv_sum_kernel, dim3((g.N / 4 + 255) / 256, T), dim3(256), 0, s, g);
        if (last) break;

        const hipError_t e = prefill_attention(s, c.kv_half, c.q, g.kcache, g.vcache, c.xhi, c.xlo, T, c.p0, c.n_heads, c.n_kv_heads, dh, c.cap_ctx);
        if (e != hipSuccess) return e;

        PrefillGemmArgs o{};
        o.xhi = c.xhi; o.xlo = c.xlo; o.W = (const uint16_t *)w.wo; o.T = T; o.N = d; o.K = nq; o.part = c.part;
        launch_gemm(s, gemm_kernel<PE_PART>(cut_o.tile), o, cut_o, 1);
        n.splits = cut_o.splits; n.gain = (const uint16_t *)w.ffn_norm;
        hipLaunchKernelGGL((prefill_norm_kernel<false>), dim3(T), dim3(norm_threads(d)), 0, s, n);

        PrefillGemmArgs f{};
        f.xhi = c.xhi; f.xlo = c.xlo; f.W = (const uint16_t *)w.w_gate; f.W2 = (const uint16_t *)w.w_up; f.T = T; f.N = c.d_ffn; f.K = d; f.part = c.part;
        f.uhi = c.uhi; f.ulo = c.ulo;
        launch_gemm(s, cut_gu.fused ? gemm_kernel<PE_SWIGLU>(cut_gu.tile) : gemm_kernel<PE_PART>(cut_gu.tile), f, cut_gu, cut_gu.fused ? 1 : 2);
        if (!cut_gu.fused) hipLaunchKernelGGL(prefill_swiglu_sum_kernel, dim3((f.N / 8 + 255) / 256, T), dim3(256), 0, s, f);

        PrefillGemmArgs dn{};
        dn.xhi = c.uhi; dn.xlo = c.ulo; dn.W = (const uint16_t *)w.w_down; dn.T = T; dn.N = d; dn.K = c.d_ffn; dn.part = c.part;
        launch_gemm(s, gemm_kernel<PE_PART>(cut_down.tile), dn, cut_down, 1);
    }
    if (!c.final) return hipGetLastError();
    if (!own_query) return last_token(s, c, SPD_DTYPE_BF16, c.q + (size_t)(T - 1) * nq, (float *)c.xhi, (float *)c.uhi);    // (buffers the products are done with)

    GemvArgs q{};
    q.W = c.layers[c.n_layers - 1].wqkv; q.gain = c.layers[c.n_layers - 1].attn_norm; q.eps = c.eps; q.x = c.h + (size_t)(T - 1) * d; q.y = c.q;
    q.rows = q.n_q_rows = nq; q.cols = d; q.n_kv_rows = nkv; q.d_head = dh; q.cap_ctx = c.cap_ctx; q.inv_freq = c.inv_freq; q.pos = c.p0 + T - 1;
    const hipError_t e = gemv(s, SPD_DTYPE_BF16, EPI_QKV, q, c.num_cu);
    if (e != hipSuccess) return e;
    return last_token(s, c, SPD_DTYPE_BF16, c.q, (float *)c.xhi, (float *)c.uhi);
}

// The same pass for an fp32 model, without partial sums.
hipError_t prefill32_chunk(hipStream_t s, const PrefillChunk &c) {
    const int T = c.T, d = c.d_model, dh = d / c.n_heads, nq = c.n_heads * dh, nkv = c.n_kv_heads * dh;
    float *att = (float *)c.xhi, *u = (float *)c.uhi;
    // (one head: its angles outnumber a token's pieces of four)
    hipLaunchKernelGGL(prefill32_start_kernel, dim3((T * std::max(d / 4, dh / 2) + 255) / 256), dim3(256), 0, s, (const float *)c.embed, c.prefix + c.p0, c.h, d, c.inv_freq,
                       c.p0, T, dh / 2, c.rope);
    auto product = [&](auto epi, Prefill32Args &a, const float *x, const void *gain, const void *W, const void *W2, int N, int K, float *y) {
        constexpr int EPI = decltype(epi)::value;
        a.x = x; a.gain = (const float *)gain; a.W32 = (const float *)W; a.W232 = (const float *)W2; a.N = N; a.K = K; a.y = y; a.T = T; a.eps = c.eps;
        // one piece of 16 tokens where there are no more; two of 16 columns where that still gives every compute unit a block
        const int tt = T <= 16 ? 1 : 2, nt = EPI == PE_SWIGLU || (long long)N * T >= 1024ll * c.num_cu ? 2 : 1;
        a.t_tiles = (T + 16 * tt - 1) / (16 * tt); a.n_tiles = EPI == PE_SWIGLU ? (N + 15) / 16 : (N + 16 * nt - 1) / (16 * nt);
        constexpr int N1 = EPI == PE_SWIGLU ? 2 : 1;
        void (*kernel)(Prefill32Args) = tt == 1 ? (nt == 1 ? prefill32_gemm_kernel<EPI, 1, N1> : prefill32_gemm_kernel<EPI, 1, 2>)
                                                : (nt == 1 ? prefill32_gemm_kernel<EPI, 2, N1> : prefill32_gemm_kernel<EPI, 2, 2>);
        hipLaunchKernelGGL(kernel, dim3((a.n_tiles + 7) / 8 * 8 * a.t_tiles), dim3(256), 0, s, a);
    };
    for (int l = 0; l < c.n_layers; ++l) {
        const spd_layer_weights &w = c.layers[l];
        Prefill32Args g{};
        g.q = c.q; g.kcache = c.kv + (size_t)(2 * l) * c.kv_layer_bytes; g.vcache = c.kv + (size_t)(2 * l + 1) * c.kv_layer_bytes;
        g.rope = c.rope; g.n_q_rows = nq; g.n_kv_rows = nkv; g.d_head = dh; g.cap_ctx = c.cap_ctx; g.p0 = c.p0;
        product(std::integral_constant<int, PE_QKV>{}, g, c.h, w.attn_norm, w.wqkv, nullptr, nq + 2 * nkv, d, nullptr);
        if (l == c.n_layers - 1) break;
        const hipError_t e = prefill_attention(s, 0, c.q, g.kcache, g.vcache, nullptr, nullptr, T, c.p0, c.n_heads, c.n_kv_heads, dh, c.cap_ctx, att);
        if (e != hipSuccess) return e;
        Prefill32Args o{}, f{}, dn{};
        product(std::integral_constant<int, PE_RESID>{}, o, att, nullptr, w.wo, nullptr, d, nq, c.h);
        product(std::integral_constant<int, PE_SWIGLU>{}, f, c.h, w.ffn_norm, w.w_gate, w.w_up, c.d_ffn, d, u);
        product(std::integral_constant<int, PE_RESID>{}, dn, u, nullptr, w.w_down, nullptr, d, c.d_ffn, c.h);
    }
    if (!c.final) return hipGetLastError();
    return last_token(s, c, SPD_DTYPE_FP32, c.q + (size_t)(T - 1) * nq, att, u);
}

}  // namespace spdk
