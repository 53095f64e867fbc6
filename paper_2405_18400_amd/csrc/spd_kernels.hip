// HIP kernels for one Superposed Decoding timestep on gfx950 (wave64).
//
// Batch-1 decode is a chain of matrix-vector products, so every kernel here is built
// around streaming weights from HBM exactly once with 128-bit loads; the only arithmetic
// that matters for time is keeping enough bytes in flight.  Reductions use a fixed order
// (no float atomics), so results are bit-reproducible run to run.
#include "spd_device.h"

#include <algorithm>
#include <type_traits>

using namespace spdd;

namespace {

constexpr int BLOCK = 256;
constexpr int NWAVE = BLOCK / WAVE;

// ------------------------------------------------------------------ matrix-vector product
// For rows and operands gemv_stream_kernel below does not take.  One wave owns two output rows at a time (EPI_SWIGLU: row r of the gate and of the up
// matrix) and walks the columns 64 lanes x 16 bytes at a time; x lives in LDS as fp32.
// Loads of the next 4-iteration chunk are issued before the current chunk is consumed, and
// the very first chunk is issued before x is staged, so HBM latency overlaps the prologue.
constexpr int GEMV_U = 4;

template <typename WT>
__device__ __forceinline__ void gemv_issue(const char *w0, const char *w1, int chunk, int lane, int cols,
                                           u32x4 *a, u32x4 *b) {
    constexpr int VEC = Store<WT>::VEC;
#pragma unroll
    for (int u = 0; u < GEMV_U; ++u) {
        const int c = ((chunk * GEMV_U + u) * WAVE + lane) * VEC;
        if (c < cols) {
            a[u] = stream_load16(w0 + (size_t)c * sizeof(WT));
            b[u] = stream_load16(w1 + (size_t)c * sizeof(WT));
        } else {
            a[u] = (u32x4)(0u);
            b[u] = (u32x4)(0u);
        }
    }
}

template <typename WT>
__device__ __forceinline__ void gemv_consume(const u32x4 *a, const u32x4 *b, int chunk, int lane,
                                             const float *xs, float &acc0, float &acc1) {
    constexpr int VEC = Store<WT>::VEC;
#pragma unroll
    for (int u = 0; u < GEMV_U; ++u) {
        const int c = ((chunk * GEMV_U + u) * WAVE + lane) * VEC;
        float xv[VEC], fa[VEC], fb[VEC];
#pragma unroll
        for (int v = 0; v < VEC; v += 4) {
            const float4 t = *(const float4 *)(xs + c + v);   // LDS
            xv[v] = t.x; xv[v + 1] = t.y; xv[v + 2] = t.z; xv[v + 3] = t.w;
        }
        Store<WT>::unpack(a[u], fa);
        Store<WT>::unpack(b[u], fb);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            acc0 = fmaf(fa[v], xv[v], acc0);
            acc1 = fmaf(fb[v], xv[v], acc1);
        }
    }
}

template <typename WT, int EPI>
__global__ __launch_bounds__(BLOCK) void gemv_kernel(const GemvArgs a) {
    constexpr int VEC = Store<WT>::VEC;
    extern __shared__ __align__(16) float xs[];   // x, zero-padded to whole chunks
    __shared__ float red[NWAVE];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid / WAVE;
    const int cols = a.cols;
    const int chunk_cols = GEMV_U * WAVE * VEC;
    const int n_chunks = (cols + chunk_cols - 1) / chunk_cols;
    const int n_units = (EPI == EPI_SWIGLU) ? a.rows : a.rows / 2;
    const int wave_stride = gridDim.x * NWAVE;
    int unit = blockIdx.x * NWAVE + wid;
    const size_t row_bytes = (size_t)cols * sizeof(WT);

    auto rows_of = [&](int un, const char *&w0, const char *&w1) {
        if (EPI == EPI_SWIGLU) {
            w0 = (const char *)a.W + (size_t)un * row_bytes;
            w1 = (const char *)a.W2 + (size_t)un * row_bytes;
        } else {
            w0 = (const char *)a.W + (size_t)(2 * un) * row_bytes;
            w1 = w0 + row_bytes;
        }
    };

    u32x4 A[GEMV_U], B[GEMV_U], A2[GEMV_U], B2[GEMV_U];
    const char *w0 = nullptr, *w1 = nullptr;
    if (unit < n_units) {
        rows_of(unit, w0, w1);
        gemv_issue<WT>(w0, w1, 0, lane, cols, A, B);
    }

    // stage x (RMS-normalised when a gain is given)
    const int padded = n_chunks * chunk_cols;
    float ss = 0.f;
    for (int c = tid; c < padded; c += BLOCK) {
        const float v = (c < cols) ? a.x[c] : 0.f;
        xs[c] = v;
        ss += v * v;
    }
    if (a.gain != nullptr) {
        const float tot = block_sum<BLOCK>(ss, red);
        const float rs = 1.0f / sqrtf(tot / (float)cols + a.eps);
        for (int c = tid; c < cols; c += BLOCK) xs[c] = xs[c] * rs * Store<WT>::load1(a.gain, c);
    }
    __syncthreads();

    while (unit < n_units) {
        float acc0 = 0.f, acc1 = 0.f;
        const int next_unit = unit + wave_stride;
        for (int ch = 0; ch < n_chunks; ++ch) {
            const bool last = (ch + 1 == n_chunks);
            bool have_next = true;
            if (!last) {
                gemv_issue<WT>(w0, w1, ch + 1, lane, cols, A2, B2);
            } else if (next_unit < n_units) {
                rows_of(next_unit, w0, w1);
                gemv_issue<WT>(w0, w1, 0, lane, cols, A2, B2);
            } else {
                have_next = false;
            }
            gemv_consume<WT>(A, B, ch, lane, xs, acc0, acc1);
            if (have_next) {
#pragma unroll
                for (int u = 0; u < GEMV_U; ++u) { A[u] = A2[u]; B[u] = B2[u]; }
            }
        }
        acc0 = wave_sum(acc0);
        acc1 = wave_sum(acc1);
        if (lane == 0) gemv_epilogue<WT, EPI>(a, unit, acc0, acc1, EPI == EPI_QKV ? gemv_pos(a) : 0);
        unit = next_unit;
    }
}

// The same product for rows of up to 64 pieces of 64 x 16 bytes (32768 bf16 columns): nothing but the weight stream between
// memory and registers.  A wave owns a segment of NI pieces of a row's columns, the same one for every row, so its
// part of x stays in registers (normalised once); `wpr` waves side by side make up a row, and finish through LDS.
// A group of wpr waves takes two rows (EPI_SWIGLU: gate and up) at a time: each of the 2 NI registers in flight is
// re-requested for the group's next two rows as soon as it has been consumed, so that 2 NI KB per wave are always on
// their way.  Past the last row the descriptor is empty: the request costs no traffic and needs no branch.
// Bound: HBM.  us per call with the weights out of cache, the kernel above -> this one: gate and up 2 x 13824 x 5120
// 62.9 -> 41.4 (6.8 TB/s), 32000 x 4096 63 -> 42, 4096 x 4096 8.8 -> 5.9.
// waves per SIMD by the registers an instantiation needs
constexpr int gemv_waves(int ni) { return ni <= 2 ? 8 : ni == 3 ? 6 : ni == 4 ? 5 : ni <= 6 ? 4 : 3; }

template <typename WT, int EPI, int NI, int NW>
__global__ __launch_bounds__(NW * WAVE, gemv_waves(NI)) void gemv_stream_kernel(const GemvArgs a, const int wpr) {
    constexpr int VEC = Store<WT>::VEC, PIECE = WAVE * 16;
    __shared__ float red[NW];
    __shared__ float2 part[2][NW];
    const int lane = threadIdx.x & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int seg = w % wpr, n_groups = (int)gridDim.x * (NW / wpr);
    const int n_units = EPI == EPI_SWIGLU ? a.rows : a.rows / 2;
    const uint32_t row_bytes = (uint32_t)a.cols * sizeof(WT);
    int unit = (int)blockIdx.x * (NW / wpr) + w / wpr;
    const uint32_t at = (uint32_t)(seg * NI * PIECE + lane * 16);
    auto row0 = [&](int un) {
        return row_resource((const char *)a.W + (size_t)min(un, n_units - 1) * row_bytes * (EPI == EPI_SWIGLU ? 1 : 2), un < n_units ? row_bytes : 0u);
    };
    auto row1 = [&](int un) {
        const char *p = EPI == EPI_SWIGLU ? (const char *)a.W2 + (size_t)min(un, n_units - 1) * row_bytes
                                          : (const char *)a.W + (size_t)min(un, n_units - 1) * row_bytes * 2 + row_bytes;
        return row_resource(p, un < n_units ? row_bytes : 0u);
    };
    u32x4 A[NI], B[NI];
    {
        const __amdgpu_buffer_rsrc_t r0 = row0(unit), r1 = row1(unit);
#pragma unroll
        for (int i = 0; i < NI; ++i) { A[i] = stream_load16(r0, at + i * PIECE); B[i] = stream_load16(r1, at + i * PIECE); }
    }
    // this lane's part of x (zero past the row's end), normalised where a gain is given
    float x[NI][VEC];
    const __amdgpu_buffer_rsrc_t xr = row_resource(a.x, (uint32_t)a.cols * 4u);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int v = 0; v < VEC; v += 4) {
            const u32x4 t = buffer_load16(xr, (at + i * PIECE) * (4 / sizeof(WT)) + v * 4);
            x[i][v] = __uint_as_float(t.x); x[i][v + 1] = __uint_as_float(t.y); x[i][v + 2] = __uint_as_float(t.z); x[i][v + 3] = __uint_as_float(t.w);
        }
    if (a.gain != nullptr) {
        const __amdgpu_buffer_rsrc_t gr = row_resource(a.gain, row_bytes);
        u32x4 g[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) g[i] = buffer_load16(gr, at + i * PIECE);
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int v = 0; v < VEC; ++v) ss += x[i][v] * x[i][v];
        ss = wave_sum_last(ss);
        if (lane == WAVE - 1) red[w] = ss;
        __syncthreads();
        float tot = 0.f;
        for (int q = 0; q < wpr; ++q) tot += red[q];
        const float rs = 1.0f / sqrtf(tot / (float)a.cols + a.eps);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            float gf[VEC];
            Store<WT>::unpack(g[i], gf);
#pragma unroll
            for (int v = 0; v < VEC; ++v) x[i][v] = x[i][v] * rs * gf[v];
        }
    }
    const int rounds = (n_units + n_groups - 1) / n_groups;
    for (int r = 0; r < rounds; ++r, unit += n_groups) {
        const __amdgpu_buffer_rsrc_t r0 = row0(unit + n_groups), r1 = row1(unit + n_groups);
        float acc0 = 0.f, acc1 = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            float f0[VEC], f1[VEC];
            Store<WT>::unpack(A[i], f0);
            Store<WT>::unpack(B[i], f1);
            A[i] = stream_load16(r0, at + i * PIECE);
            B[i] = stream_load16(r1, at + i * PIECE);
            __builtin_amdgcn_sched_barrier(0);   // (the compiler would first wait for half of the pieces)
#pragma unroll
            for (int v = 0; v < VEC; ++v) { acc0 = fmaf(f0[v], x[i][v], acc0); acc1 = fmaf(f1[v], x[i][v], acc1); }
        }
        acc0 = wave_sum_last(acc0);
        acc1 = wave_sum_last(acc1);
        if (wpr > 1) {     // (two buffers: the waves of a group are at most one barrier apart)
            if (lane == WAVE - 1) part[r & 1][w] = make_float2(acc0, acc1);
            __syncthreads();
            if (seg == 0) {
                acc0 = acc1 = 0.f;
                for (int q = 0; q < wpr; ++q) { acc0 += part[r & 1][w + q].x; acc1 += part[r & 1][w + q].y; }
            }
        }
        if (seg == 0 && lane == WAVE - 1 && unit < n_units) gemv_epilogue<WT, EPI>(a, unit, acc0, acc1, EPI == EPI_QKV ? gemv_pos(a) : 0);
    }
}

// ------------------------------------------------------------------ superposed embedding
// Section 3.1: gamma_i = p_i / sum_j p_j (from log p_i), x~ = sum_i gamma_i z_i.
// mode 0 feeds a prefix token's own embedding (gamma = 1) during the prefix pass.
template <typename WT>
__global__ __launch_bounds__(BLOCK) void superpose_kernel(const SuperposeArgs a) {
    superpose_element<WT>(a, blockIdx.x * BLOCK + threadIdx.x, a.mode == 0 ? a.st->pos : 0);
}

// ------------------------------------------------------------------ vocabulary top-k
// Total order used everywhere: larger value first, then smaller index.  As unsigned integers: a value's key rises with it and is 0 for an absent entry and for a NaN, which is never
// better than anything; -0 and 0 are equal.  With the inverted id below it an entry is one 64-bit word.
__device__ __forceinline__ uint32_t value_key(float v) {
    const uint32_t u = __float_as_uint(v + 0.f);
    return v != v ? 0u : (u & 0x80000000u) ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float key_value(uint32_t key) { return key == 0u ? -INFINITY : __uint_as_float((key & 0x80000000u) ? key & 0x7FFFFFFFu : ~key); }
__device__ __forceinline__ unsigned long long entry_key(float v, int id) { return ((unsigned long long)value_key(v) << 32) | (uint32_t)~id; }
__device__ __forceinline__ float read_lane(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_max_key(uint32_t v) {
    v = dpp_max<0xB1, 0xF>(v); v = dpp_max<0x4E, 0xF>(v); v = dpp_max<0x141, 0xF>(v);
    v = dpp_max<0x140, 0xF>(v); v = dpp_max<0x142, 0xA>(v); v = dpp_max<0x143, 0xC>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, WAVE - 1);
}
// The k best of the NR entries per lane (keys; id(q) rises with q) end up one per lane, best first, in lanes 0 .. k - 1.
// No LDS, no barrier, no branch on a lane's data: a round takes 0.1 us where one over a block with its two barriers took
// 0.75, and so did one whose lanes compared (value, id) pairs under branches.
template <int NR, typename ID> __device__ __forceinline__ void wave_top_k(int k, uint32_t (&key)[NR], ID id, float &kv, int &ki) {
    const int lane = threadIdx.x & (WAVE - 1);
    kv = -INFINITY; ki = INT_MAX;
    for (int r = 0; r < k; ++r) {
        uint32_t best = key[0];
        int at = id(0);
#pragma unroll
        for (int q = 1; q < NR; ++q) {
            at = key[q] > best ? id(q) : at;
            best = max(best, key[q]);
        }
        const uint32_t m = wave_max_key(best);
        if (m == 0u) return;                    // (the wave as a whole: nothing is left)
        unsigned long long who = __ballot(best == m);
        if (__popcll(who) != 1) {               // a tie: the lowest id
            int lowest = best == m ? at : INT_MAX;
#pragma unroll
            for (int o = WAVE / 2; o > 0; o >>= 1) lowest = min(lowest, __shfl_xor(lowest, o, WAVE));
            who = __ballot(best == m && at == lowest);
        }
        const int won = __builtin_amdgcn_readlane(at, __builtin_amdgcn_readfirstlane(__ffsll((long long)who) - 1));
        if (lane == r) { kv = key_value(m); ki = won; }
#pragma unroll
        for (int q = 0; q < NR; ++q) key[q] = id(q) == won ? 0u : key[q];
    }
}
// Where entry tid / PARTS of n stands in the order; equal words (absent entries) in the order they lie in.  PARTS lanes
// (a power of two up to 16) compare with every PARTS-th entry each: one thread walking all of 64 took 2.4 us.
template <int PARTS> __device__ __forceinline__ int rank_among(const unsigned long long *e, int n) {
    const int t = threadIdx.x / PARTS, part = threadIdx.x % PARTS;
    int rank = 0;
    if (t < n) {
        const unsigned long long mine = e[t];
        for (int c = part; c < n; c += PARTS) {
            const unsigned long long other = e[c];
            rank += (int)(other > mine) + (int)((other == mine) & (c < t));
        }
    }
#pragma unroll
    for (int o = PARTS / 2; o > 0; o >>= 1) rank += __shfl_xor(rank, o, WAVE);
    return rank;
}

// Each block scans a contiguous slice of the logits: its k best entries, its max and min and its sum of
// exp(z - max) with z = logit / tau.  Every wave does so for its share, then the waves' results are merged: one
// barrier.  A chain of latencies (launch, one trip to memory, k rounds): 9.2 -> 5.3 us at k = 8 against the kernel whose
// rounds went over the block.
// NR: entries of the slice per thread, the least of 4, 8, 16 and 32 that hold it (4 up to vocabularies of 131072): each is looked at
// in every round (131074 entries, the kernel: 4.1 us at k = 1 with the rounds over the block, 5.6 with 32 entries, 4.1 with 8; 262144: 5.4, 6.0, 4.4).
struct TopkScratch {
    unsigned long long entry[NWAVE * SPD_K_MAX];
    float sv[NWAVE * SPD_K_MAX], wave_max[NWAVE], wave_exp[NWAVE], wave_min[NWAVE];
    int si[NWAVE * SPD_K_MAX];
};
// Before the barrier: every wave's share; behind it: the block's result (COH: written through, for a block of the same launch).
template <int NR> __device__ __forceinline__ void topk_share(const TopkArgs &a, TopkScratch &s) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE, b = blockIdx.x, k = a.k;
    const int lo = b * a.per_part, hi = min(a.vocab, lo + a.per_part);
    float rv[NR];
    uint32_t key[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const int i = lo + tid + q * BLOCK;
        rv[q] = i < hi ? as_global(a.logits)[i] : -INFINITY;
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) key[q] = lo + tid + q * BLOCK < hi ? value_key(rv[q]) : 0u;
    float kv;
    int ki;
    wave_top_k(k, key, [&](int q) { return lo + tid + q * BLOCK; }, kv, ki);
    if (lane < k) { s.sv[w * k + lane] = kv; s.si[w * k + lane] = ki; s.entry[w * k + lane] = ki == INT_MAX ? 0ull : entry_key(kv, ki); }
    // x -> x / tau is monotonic for tau > 0: the largest logit gives the largest z
    const float mx = __fdiv_rn(read_lane(kv, 0), a.tau), ref = mx == -INFINITY ? 0.f : mx;   // (a share without entries, or of -inf alone: every term is 0)
    float sm = 0.f, lowest = INFINITY;
#pragma unroll
    for (int q = 0; q < NR; ++q)
        if (lo + tid + q * BLOCK < hi) { sm += expf(__fdiv_rn(rv[q], a.tau) - ref); lowest = fminf(lowest, rv[q]); }
    sm = wave_sum_last(sm);
    lowest = -wave_max_last(-lowest);
    if (lane == WAVE - 1) { s.wave_max[w] = mx; s.wave_exp[w] = sm; s.wave_min[w] = lowest; }
}
template <bool COH> __device__ __forceinline__ void topk_result(const TopkArgs &a, const TopkScratch &s) {
    const int tid = threadIdx.x, b = blockIdx.x, k = a.k;
    const int lo = b * a.per_part, hi = min(a.vocab, lo + a.per_part);
    constexpr int PARTS = BLOCK / (NWAVE * SPD_K_MAX);
    const int rank = rank_among<PARTS>(s.entry, NWAVE * k), t = tid / PARTS;
    if (t < NWAVE * k && rank < k && tid % PARTS == 0) {
        act_store<COH>(a.pv + b * SPD_K_MAX + rank, s.sv[t]);
        act_store<COH>((float *)a.pi + b * SPD_K_MAX + rank, __int_as_float(s.si[t]));
    }
    if (tid == BLOCK - 1) {
        float m = -INFINITY, sum = 0.f, l = INFINITY;
#pragma unroll
        for (int q = 0; q < NWAVE; ++q) { m = fmaxf(m, s.wave_max[q]); l = fminf(l, s.wave_min[q]); }
#pragma unroll
        for (int q = 0; q < NWAVE; ++q) sum += s.wave_max[q] == -INFINITY ? s.wave_exp[q] : s.wave_exp[q] * expf(s.wave_max[q] - m);
        act_store<COH>(a.pm + b, m);
        act_store<COH>(a.ps + b, sum);
        if (!COH) a.pn[b] = lo < hi ? __fdiv_rn(l, a.tau) : INFINITY;      // (for the nucleus sampler alone)
    }
}
template <int NR>
__global__ __launch_bounds__(BLOCK) void topk_partial_kernel(const TopkArgs a) {
    __shared__ TopkScratch s;
    topk_share<NR>(a, s);
    __syncthreads();
    topk_result<false>(a, s);
}

// ------------------------------------------------------------------ expand, interpolate, prune
// Linear probing.  The eight lanes of a group look at eight consecutive slots (256 bytes) of one probe's walk at a time, N
// probes of a group side by side: every trip is a random access into a table far larger than any cache, so what
// counts is the number of trips (at a load factor of 0.7 some of a step's 60 .. 360 probes walk past four slots, few past
// eight) and of cache lines a load instruction touches (with a probe per lane every one of its 16 loads touched 64
// lines); 360 probes 6 .. 15 -> 5.5 us, with the table in order of home slots.
// The slots are examined in probing order, so the result is that of a slot-by-slot walk.  found(u, count) is called by the lane whose slot
// holds probe u's key, if any does.  All waves of a block probe on one compute unit, so instructions count as much as trips do: the hitting
// lane goes on by itself (no shuffles), an 8-lane mask is cut from half a ballot, the keys come from where they were hashed, and a group
// takes only as many probes as its wave has.  Cycles for the counts of k = 5, 8, 10 and five orders: 13600, 14500, 16400 -> 3900, 7100, 11300.
constexpr int PROBE_LANES = 8;
// Between a result's zero, stored by one lane, and its count, stored by the lane of the same wave that hits: a wave's LDS stores stay in program
// order, and this keeps the compiler from changing that order.
__device__ __forceinline__ void cleared_before_probes() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// `home`: the key's home slot, NO_HOME: not wanted (its 64-bit multiplications are dear: one lane's work, not eight's).
constexpr uint64_t NO_HOME = ~0ull;
template <int N, typename F>
__device__ __forceinline__ void ngram_probes(const NgramDev &ng, const int32_t (&key)[N][6], const uint64_t (&home)[N], F &&found) {
    const int lane = threadIdx.x & (WAVE - 1), j = lane % PROBE_LANES, first = (lane - j) % 32;
    auto group_of = [&](unsigned long long mask) { return ((lane < 32 ? (uint32_t)mask : (uint32_t)(mask >> 32)) >> first) & 0xFFu; };
    const uint32_t before = (1u << j) - 1u;
    uint64_t at[N];
    bool open[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        open[u] = home[u] != NO_HOME;
        at[u] = home[u] + (uint64_t)j;
        while (open[u] && at[u] >= ng.capacity) at[u] -= ng.capacity;
    }
    for (int p = 0; p <= ng.max_probe; p += PROBE_LANES) {
        u32x4 lo[N], hi[N];
        bool more = false;
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (open[u]) {
                const NgramSlot *sl = ng.slots + at[u];
                lo[u] = global_load16(sl);
                hi[u] = global_load16((const char *)sl + 16);
            }
        const bool past = p + j > ng.max_probe;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            bool hit = false, end = false;
            if (open[u]) {
                const uint32_t differs = (lo[u].x ^ (uint32_t)key[u][0]) | (lo[u].y ^ (uint32_t)key[u][1]) | (lo[u].z ^ (uint32_t)key[u][2]) |
                                         (lo[u].w ^ (uint32_t)key[u][3]) | (hi[u].x ^ (uint32_t)key[u][4]) | (hi[u].y ^ (uint32_t)key[u][5]);
                end = past || (int32_t)lo[u].x == NG_EMPTY;
                hit = !past && differs == 0u;
            }
            const uint32_t hits = group_of(__ballot(hit)), ends = group_of(__ballot(end));
            if (hit && (ends & before) == 0u) found(u, ((unsigned long long)hi[u].w << 32) | hi[u].z);
            open[u] = open[u] && (hits | ends) == 0u;
            at[u] += PROBE_LANES;
            while (open[u] && at[u] >= ng.capacity) at[u] -= ng.capacity;
            more = more || open[u];
        }
        if (!__any(more)) break;
    }
}

// Merges the per-slice top-k into the global KeepTopK and log-softmax, builds the
// k x k options, probes the n-gram store for every (draft, kept token, order), applies the
// mixture (Eq. 3), the interpolation (Eq. 4) or the penalty form (Eq. 5), keeps the k best
// options and rewrites the draft state.  One block's work; SLICES: the block that is last to finish its slice goes on with it.
// A chain of latencies.  Whatever does not depend on the kept tokens is asked for at the start: the first MERGE threads
// select in the block's slice while the others look up the drafts' context totals, in every block, since any may be the last.  With
// few drafts the totals are looked up together with the counts, a group of lanes for each probe (ONE_GO: the kernel at
// k = 1 .. 4, five orders, 9.2 .. 10.2 -> 5.7 .. 7.1 us).
// One launch or two (not SLICES: they are a launch of their own), a timestep's decisions from 32000 logits, launched one by one, two
// -> one: no n-grams 8.9 -> 7.6 us at k = 1, 11.2 -> 10.9 at 8; five orders 15.6 -> 15.5 at k = 5, 22.8 -> 21.8 at 10.  With few drafts and
// n-grams there is nothing to hide in the slices' time (10.35 -> 10.53 at k = 3) and two stay.  Two also where a slice has more than 1024
// entries (vocabularies from 131074 on): of a block of 1024 threads 256 select, 5 .. 32 entries each, in every one of 128 blocks.  One -> two there,
// 131074 .. 700000 entries, k = 1 .. 8: 0.83 .. 1.00 times for the first timestep and without n-grams (262146, k = 4: 12.8 -> 11.7 us), 0.93 .. 0.98 with
// them from k = 5 on.
// k = 8, five orders, 120 000 n-grams of each, cycles from the block's start: its slice 7400, published and counted 4000, merge 6200, hashes 2300, probes
// 7100, mixture and scores 2100, prune and state 3300: 40900 -> 32500 in all with the leaner probes and a lane per draft at the end (k = 5: 36500 -> 25500,
// 10: 52000 -> 43300); four timesteps and their results 92.7 -> 79.6 us.
constexpr int ENT = 1024, MERGE = 256, MERGE_WAVES = MERGE / WAVE, GROUPS = ENT / PROBE_LANES;

constexpr bool probes_in_one_go(int k) { return (k * k + k) * SPD_N_ORDERS <= GROUPS; }

template <bool SLICES, bool ONE_GO>
__global__ __launch_bounds__(ENT) void expand_prune_kernel(const TopkArgs slice, const ExpandArgs a) {
    static_assert(MERGE == BLOCK, "the waves that merge are those that select");
    __shared__ TopkScratch scratch;
    __shared__ int is_last;
    __shared__ unsigned long long entry[MERGE_WAVES * SPD_K_MAX], option[SPD_KK];
    __shared__ float sv[MERGE_WAVES * SPD_K_MAX];
    __shared__ int si[MERGE_WAVES * SPD_K_MAX];
    __shared__ int s_top[SPD_K_MAX];
    __shared__ float s_logp[SPD_K_MAX];
    __shared__ float s_lse;
    __shared__ float s_new[SPD_K_MAX];
    __shared__ int s_tails[SPD_K_MAX][SPD_TAIL];
    __shared__ float s_old[SPD_K_MAX];
    __shared__ unsigned long long s_cnt[SPD_KK * SPD_N_ORDERS];
    __shared__ uint64_t s_home[SPD_KK * SPD_N_ORDERS];
    __shared__ int2 s_key[ONE_GO ? 1 : SPD_KK * SPD_N_ORDERS][3];
    __shared__ unsigned long long s_tot[SPD_K_MAX * SPD_N_ORDERS];
    __shared__ float s_png[SPD_KK];
    __shared__ int s_any[SPD_K_MAX];
    __shared__ float s_score[SPD_KK];
    __shared__ int s_valid[SPD_KK];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), k = a.k;
    DevState *st = a.st;
    const int gen = st->n_gen, pos = st->pos;

    // The n-gram (the last n - 1 tokens of a draft, token) as a key (token NG_TOTAL: its context's total); false: it cannot
    // be in the store (no table of that order; the last n - 1 tokens of the history must all exist).
    auto make_key = [&](const int (&tail)[SPD_TAIL], int n, int token, int32_t (&key)[6]) {
#pragma unroll
        for (int q = 0; q < 6; ++q) key[q] = NG_PAD;
#pragma unroll
        for (int q = 0; q < SPD_TAIL; ++q) {     // (constant indices: the key stays in registers)
#pragma unroll
            for (int m = SPD_MIN_ORDER; m < SPD_MIN_ORDER + SPD_N_ORDERS; ++m)
                if (m == n) {
                    if (q < m - 1) key[q] = tail[SPD_TAIL - (m - 1) + q];
                    if (q == m - 2) key[q + 1] = token;
                }
        }
        return a.ng.slots != nullptr && a.ng.present[n - SPD_MIN_ORDER] && key[0] >= 0;
    };
    const bool use_ng = !a.first && a.alpha != 0.0f;
    const int n_count = k * k * SPD_N_ORDERS, n_total = k * SPD_N_ORDERS;
    if (tid < MERGE) {
        if constexpr (SLICES) topk_share<4>(slice, scratch);
    } else {
        const int u = tid - MERGE;
        if (u < SPD_K_MAX) {
            s_old[u] = st->logscore[u];
            s_any[u] = 0;
            for (int q = 0; q < SPD_TAIL; ++q) s_tails[u][q] = a.first ? st->prefix_tail[q] : st->tails[u][q];
        }
        const int e = u / PROBE_LANES;
        static_assert((ENT - MERGE) / PROBE_LANES >= SPD_K_MAX * SPD_N_ORDERS, "a group of lanes per context");
        if (!ONE_GO && use_ng && e < (n_total + PROBE_LANES - 1) / PROBE_LANES * PROBE_LANES) {   // (whole waves)
            int tail[SPD_TAIL];
            int32_t key[1][6];
#pragma unroll
            for (int q = 0; q < SPD_TAIL; ++q) tail[q] = st->tails[min(e / SPD_N_ORDERS, SPD_K_MAX - 1)][q];
            const bool known = make_key(tail, SPD_MIN_ORDER + e % SPD_N_ORDERS, NG_TOTAL, key[0]);
            const uint64_t home[1] = {known && e < n_total ? ngram_home(ngram_hash(key[0]), a.ng.capacity) : NO_HOME};
            if (e < n_total && u % PROBE_LANES == 0) s_tot[e] = 0ull;
            cleared_before_probes();
            ngram_probes<1>(a.ng, key, home, [&](int, unsigned long long total) { s_tot[e] = total; });
        }
    }
    if constexpr (SLICES) {
        __syncthreads();
        if (tid < MERGE) {
            topk_result<true>(slice, scratch);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's write-through stores have been acknowledged
        }
        __syncthreads();
        if (tid == 0) is_last = __hip_atomic_fetch_add(as_global(a.arrived), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        __syncthreads();
        if (!is_last) return;
        if (tid == 0) __hip_atomic_store(as_global(a.arrived), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    }
    if (tid < MERGE) {
        const int n_cand = a.n_part * k;
        constexpr int NC = TOPK_PART_MAX * SPD_K_MAX / MERGE;
        auto candidate = [&](int q, float &v, int &i) {
            const int c = tid + q * MERGE, at = (c / k) * SPD_K_MAX + (c % k);
            v = c < n_cand ? act_load<SLICES>(a.pv + at) : -INFINITY;
            i = c < n_cand ? __float_as_int(act_load<SLICES>((const float *)a.pi + at)) : INT_MAX;
        };
        float cv[NC];
        int ci[NC];
        candidate(0, cv[0], ci[0]);
        if (n_cand > MERGE) {
#pragma unroll
            for (int q = 1; q < NC; ++q)
                if (q < 2 || n_cand > 2 * MERGE) candidate(q, cv[q], ci[q]);
        }
        if (tid < WAVE) {   // log-sum-exp over the slices: M = max of the maxima, S = sum of sum-exp * exp(max - M)
            static_assert(TOPK_PART_MAX == 2 * WAVE, "two slices per lane");
            float pm[2], ps[2], sum = 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int b = lane + q * WAVE;
                pm[q] = b < a.n_part ? act_load<SLICES>(a.pm + b) : -INFINITY;
                ps[q] = b < a.n_part ? act_load<SLICES>(a.ps + b) : 0.f;
            }
            const float M = read_lane(wave_max_last(fmaxf(pm[0], pm[1])), WAVE - 1);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (lane + q * WAVE < a.n_part) sum += ps[q] * expf(pm[q] - M);
            const float S = read_lane(wave_sum_last(sum), WAVE - 1);
            if (lane == 0) s_lse = M + logf(S);
        }
        float kv;
        int ki;
        auto select = [&](auto count) {
            constexpr int N = decltype(count)::value;
            uint32_t key[N];
#pragma unroll
            for (int q = 0; q < N; ++q) key[q] = ci[q] == INT_MAX ? 0u : value_key(cv[q]);
            wave_top_k(k, key, [&](int q) { return ci[q]; }, kv, ki);
        };
        if (n_cand > 2 * MERGE) select(std::integral_constant<int, NC>());
        else if (n_cand > MERGE) select(std::integral_constant<int, 2>());
        else select(std::integral_constant<int, 1>());
        if (lane < k) {
            const int at = (tid / WAVE) * k + lane;
            sv[at] = kv; entry[at] = ki == INT_MAX ? 0ull : entry_key(kv, ki);
            si[at] = ki == INT_MAX ? 0 : ki;     // (fewer than k logits are numbers: the next forward still looks up a token there is)
        }
    }
    __syncthreads();
    {
        constexpr int PARTS = 16;
        const int rank = rank_among<PARTS>(entry, MERGE_WAVES * k), t = tid / PARTS;
        if (t < MERGE_WAVES * k && rank < k && tid % PARTS == 0) {
            const float logp = __fdiv_rn(sv[t], a.tau) - s_lse;
            s_top[rank] = si[t];
            s_logp[rank] = logp;
            st->top_ids[rank] = si[t];
            st->top_logp[rank] = logp;
        }
    }
    __syncthreads();

    if (a.first) {  // Section 3, "First Timestep"
        if (tid < k) {
            for (int q = 0; q < SPD_TAIL - 1; ++q) st->tails[tid][q] = s_tails[tid][q + 1];
            st->tails[tid][SPD_TAIL - 1] = s_top[tid];
            st->logscore[tid] = s_logp[tid];
            s_new[tid] = s_logp[tid];
            st->new_tok[tid] = s_top[tid];
            st->new_parent[tid] = -1;
            a.hist_tok[tid] = s_top[tid];
            a.hist_par[tid] = -1;
        }
        for (int c = tid; c < k * k; c += ENT) {
            st->cand_score[c] = (c < k) ? s_logp[c] : -INFINITY;
            st->cand_valid[c] = (c < k);
            st->cand_png[c] = 0.f;
        }
    } else {
        if (use_ng) {
            auto key_of = [&](int e, int32_t (&key)[6]) {          // probe e: draft, kept token, order; behind the counts: draft, order of a total
                const bool total = ONE_GO && e >= n_count;
                const int i = total ? (e - n_count) / SPD_N_ORDERS : e / n_total;
                int tail[SPD_TAIL];
#pragma unroll
                for (int q = 0; q < SPD_TAIL; ++q) tail[q] = s_tails[i][q];
                return make_key(tail, SPD_MIN_ORDER + e % SPD_N_ORDERS, total ? NG_TOTAL : s_top[(e / SPD_N_ORDERS) % k], key);
            };
            if constexpr (ONE_GO) {
                const int n_probe = n_count + n_total, e = tid / PROBE_LANES;
                if (tid / WAVE * (WAVE / PROBE_LANES) < n_probe) {     // (whole waves)
                    int32_t key[1][6];
                    const bool known = key_of(min(e, n_probe - 1), key[0]);
                    const uint64_t home[1] = {known && e < n_probe ? ngram_home(ngram_hash(key[0]), a.ng.capacity) : NO_HOME};
                    auto put = [&](unsigned long long count) {
                        if (e < n_count) s_cnt[e] = count;
                        else s_tot[e - n_count] = count;
                    };
                    if (e < n_probe && tid % PROBE_LANES == 0) put(0ull);
                    cleared_before_probes();
                    ngram_probes<1>(a.ng, key, home, [&](int, unsigned long long count) { put(count); });
                }
            } else {
                for (int e = tid; e < n_count; e += ENT) {
                    int32_t key[6];
                    s_home[e] = key_of(e, key) ? ngram_home(ngram_hash(key), a.ng.capacity) : NO_HOME;
#pragma unroll
                    for (int q = 0; q < 6; q += 2) s_key[e][q / 2] = make_int2(key[q], key[q + 1]);
                    s_cnt[e] = 0ull;
                }
                __syncthreads();
                auto probe = [&](auto n, int e0) {                 // n probes per group of lanes
                    constexpr int N = decltype(n)::value;
                    int32_t key[N][6];
                    uint64_t home[N];
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const int e = e0 + u * GROUPS, f = min(e, n_count - 1);
#pragma unroll
                        for (int q = 0; q < 6; q += 2) { const int2 w = s_key[f][q / 2]; key[u][q] = w.x; key[u][q + 1] = w.y; }
                        home[u] = e < n_count ? s_home[f] : NO_HOME;
                    }
                    ngram_probes<N>(a.ng, key, home, [&](int u, unsigned long long count) { s_cnt[e0 + u * GROUPS] = count; });
                };
                // (all of up to k = 10 in one go)
                for (int e0 = 0; e0 < n_count; e0 += 4 * GROUPS) {
                    const int e = e0 + tid / PROBE_LANES, left = n_count - e0 - __builtin_amdgcn_readfirstlane(tid / WAVE) * (WAVE / PROBE_LANES);     // (by the wave's first probe)
                    if (left > 3 * GROUPS) probe(std::integral_constant<int, 4>(), e);
                    else if (left > 2 * GROUPS) probe(std::integral_constant<int, 3>(), e);
                    else if (left > GROUPS) probe(std::integral_constant<int, 2>(), e);
                    else if (left > 0) probe(std::integral_constant<int, 1>(), e);
                }
            }
            __syncthreads();
            if (tid < k * k) {  // Eq. 3
                const int i = tid / k;
                float acc = 0.f;
                for (int o = 0; o < SPD_N_ORDERS; ++o) {
                    const unsigned long long C = s_tot[i * SPD_N_ORDERS + o];
                    const float p = C ? __fdiv_rn(__ull2float_rn(s_cnt[tid * SPD_N_ORDERS + o]), __ull2float_rn(C)) : 0.f;
                    acc = __fadd_rn(acc, __fmul_rn(a.ng.lambda[o], p));
                }
                s_png[tid] = acc;
                if (acc > 0.f) atomicOr(&s_any[i], 1);
            }
            __syncthreads();
        }
        if (tid < k * k) {
            const int i = tid / k, j = tid % k;
            float score;
            int valid = 1;
            if (!use_ng) {
                score = __fadd_rn(s_old[i], s_logp[j]);
            } else {
                const float lm = __fmul_rn(__fsub_rn(1.0f, a.alpha), s_logp[j]);
                float lpf;
                if (s_png[tid] > 0.f) lpf = __fadd_rn(lm, __fmul_rn(a.alpha, logf(s_png[tid])));   // Eq. 4
                else if (s_any[i]) { lpf = 0.f; valid = 0; }   // token outside the overlap set
                else lpf = __fadd_rn(logf(a.delta), lm);       // Eq. 5
                score = __fadd_rn(s_old[i], lpf);
            }
            s_score[tid] = valid ? score : -INFINITY;
            s_valid[tid] = valid;
            option[tid] = valid ? entry_key(score, tid) : 0ull;   // score desc, then parent asc, then token rank asc
            st->cand_score[tid] = s_score[tid];
            st->cand_valid[tid] = valid;
            st->cand_png[tid] = use_ng ? s_png[tid] : 0.f;
        }
        __syncthreads();
        // the options' ranks: 16 lanes for each of up to 64, 4 for each of up to 256
        const bool few = k * k <= ENT / 16;
        const int rank = few ? rank_among<16>(option, k * k) : rank_among<4>(option, k * k), c = few ? tid / 16 : tid / 4;
        if (c < k * k && s_valid[c] && (few ? tid % 16 : tid % 4) == 0) {
            if (rank < k) {
                const int i = c / k, j = c % k;
                for (int q = 0; q < SPD_TAIL - 1; ++q) st->tails[rank][q] = s_tails[i][q + 1];
                st->tails[rank][SPD_TAIL - 1] = s_top[j];
                st->logscore[rank] = s_score[c];
                s_new[rank] = s_score[c];
                st->new_tok[rank] = s_top[j];
                st->new_parent[rank] = i;
                if (gen < a.max_gen) {
                    a.hist_tok[(size_t)gen * SPD_K_MAX + rank] = s_top[j];
                    a.hist_par[(size_t)gen * SPD_K_MAX + rank] = i;
                }
            }
        }
    }
    __syncthreads();
    if (tid < WAVE) {  // Eq. 2 on the new scores: a lane per draft, added in draft order (every lane walking all of them: 1800 cycles at k = 8, so 600)
        const float mine = lane < k ? s_new[lane] : -INFINITY;
        const float mx = read_lane(wave_max_last(mine), WAVE - 1);
        const float e = expf(mine - mx);
        float sum = 0.f;
        for (int i = 0; i < k; ++i) sum += read_lane(e, i);
        if (lane < k) st->gamma[lane] = e / sum;
        if (tid == 0) {
            st->k = k;
            st->n_gen = a.first ? 1 : gen + 1;
            if (a.advance) st->pos = pos + 1;
        }
    }
}

__global__ void advance_kernel(DevState *st) { st->pos += 1; }

// The drafts and their scores come as arguments, 388 bytes: with two copies to the device, a wait for them and one for a kernel of one
// thread the whole call took 17.4 us, with this 12.5 (through the Python entry 20.4 and 13.4).  (Results the other way: a kernel that
// stores them into pinned memory takes as long as the copy.)
__global__ __launch_bounds__(WAVE) void set_drafts_kernel(DevState *st, const DraftArgs a) {
    const int i = threadIdx.x;
    for (int e = i; e < SPD_K_MAX * SPD_TAIL; e += WAVE) (&st->tails[0][0])[e] = (&a.tails[0][0])[e];
    if (i < SPD_K_MAX) st->logscore[i] = a.logscore[i];
    if (i == 0) st->k = a.k;
    if (i >= a.k) return;
    float mx = -INFINITY, sum = 0.f;   // Eq. 2
    for (int j = 0; j < a.k; ++j) mx = fmaxf(mx, a.logscore[j]);
    for (int j = 0; j < a.k; ++j) sum += expf(a.logscore[j] - mx);
    st->gamma[i] = expf(a.logscore[i] - mx) / sum;
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void fill3_i32_kernel(FillRange a, FillRange b, FillRange c) {
    const int at = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    for (int i = at; i < a.n; i += step) a.p[i] = a.v;
    for (int i = at; i < b.n; i += step) b.p[i] = b.v;
    for (int i = at; i < c.n; i += step) c.p[i] = c.v;
}

template <typename WT, int EPI>
hipError_t gemv_launch(hipStream_t s, const GemvArgs &a, int num_cu, size_t lds) {
    const int units = EPI == EPI_SWIGLU ? a.rows : a.rows / 2;
    const int pieces = (int)(((size_t)a.cols * sizeof(WT) + WAVE * 16 - 1) / (WAVE * 16));
    const uintptr_t all = (uintptr_t)a.W | (uintptr_t)a.W2 | (uintptr_t)a.gain | (uintptr_t)a.x;
    if (pieces > 64 || (all & 15)) {   // wider rows, operands off the 16-byte grid: x through LDS
        const int blocks = std::max(1, std::min((units + NWAVE - 1) / NWAVE, num_cu * 8));
        hipLaunchKernelGGL((gemv_kernel<WT, EPI>), dim3(blocks), dim3(BLOCK), lds, s, a);
        return hipGetLastError();
    }
    // Waves per row: as few as hold the row in 8 pieces each, more while the units do not give every SIMD two waves
    // (256 rows of 4096: 128 units, each split four ways).
    int wpr = 1;
    while ((pieces + wpr - 1) / wpr > 8) wpr *= 2;
    while (wpr < 4 && (pieces + wpr - 1) / wpr > 1 && units * wpr < num_cu * 8) wpr *= 2;
    const int nw = wpr == 8 ? 8 : 4, ni = (pieces + wpr - 1) / wpr;
    // as many blocks as fit the chip, each with the same number of rounds
    const int need = (units * wpr + nw - 1) / nw, cap = num_cu * (nw == 8 ? 1 : gemv_waves(ni));
    const int rounds = (need + cap - 1) / cap, blocks = (need + rounds - 1) / rounds;
#define SPD_GEMV(NI, NW) hipLaunchKernelGGL((gemv_stream_kernel<WT, EPI, NI, NW>), dim3(blocks), dim3(NW * WAVE), 0, s, a, wpr)
    if (nw == 8) {
        if (ni <= 6) SPD_GEMV(6, 8);
        else SPD_GEMV(8, 8);
    } else {
        switch (ni) {
            case 1: SPD_GEMV(1, 4); break;
            case 2: SPD_GEMV(2, 4); break;
            case 3: SPD_GEMV(3, 4); break;
            case 4: SPD_GEMV(4, 4); break;
            case 5: SPD_GEMV(5, 4); break;
            case 6: SPD_GEMV(6, 4); break;
            case 7: SPD_GEMV(7, 4); break;
            default: SPD_GEMV(8, 4); break;
        }
    }
#undef SPD_GEMV
    return hipGetLastError();
}

template <typename WT>
hipError_t gemv_dispatch(hipStream_t s, int epi, const GemvArgs &a, int num_cu, size_t lds) {
    switch (epi) {
        case EPI_PLAIN: return gemv_launch<WT, EPI_PLAIN>(s, a, num_cu, lds);
        case EPI_RESID: return gemv_launch<WT, EPI_RESID>(s, a, num_cu, lds);
        case EPI_QKV: return gemv_launch<WT, EPI_QKV>(s, a, num_cu, lds);
        case EPI_SWIGLU: return gemv_launch<WT, EPI_SWIGLU>(s, a, num_cu, lds);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

namespace spdk {

size_t gemv_lds_bytes(int dtype, int cols) {
    const int vec = dtype == SPD_DTYPE_BF16 ? 8 : 4;
    const int chunk_cols = GEMV_U * WAVE * vec;
    return (size_t)((cols + chunk_cols - 1) / chunk_cols) * chunk_cols * sizeof(float);
}

hipError_t gemv(hipStream_t s, int dtype, int epi, const GemvArgs &a, int num_cu) {
    const size_t lds = gemv_lds_bytes(dtype, a.cols);
    if (dtype == SPD_DTYPE_BF16) return gemv_dispatch<bf16_t>(s, epi, a, num_cu, lds);
    return gemv_dispatch<float>(s, epi, a, num_cu, lds);
}

hipError_t superpose(hipStream_t s, int dtype, const SuperposeArgs &a) {
    const int blocks = (a.d_model + BLOCK - 1) / BLOCK;
    if (dtype == SPD_DTYPE_BF16) hipLaunchKernelGGL(superpose_kernel<bf16_t>, dim3(blocks), dim3(BLOCK), 0, s, a);
    else hipLaunchKernelGGL(superpose_kernel<float>, dim3(blocks), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t topk_partial(hipStream_t s, const TopkArgs &a) {
    if (a.per_part <= 4 * BLOCK) hipLaunchKernelGGL(topk_partial_kernel<4>, dim3(a.n_part), dim3(BLOCK), 0, s, a);
    else if (a.per_part <= 8 * BLOCK) hipLaunchKernelGGL(topk_partial_kernel<8>, dim3(a.n_part), dim3(BLOCK), 0, s, a);
    else if (a.per_part <= 16 * BLOCK) hipLaunchKernelGGL(topk_partial_kernel<16>, dim3(a.n_part), dim3(BLOCK), 0, s, a);
    else if (a.per_part <= 32 * BLOCK) hipLaunchKernelGGL(topk_partial_kernel<32>, dim3(a.n_part), dim3(BLOCK), 0, s, a);
    else return hipErrorInvalidValue;   // (vocabularies stay below 2^20)
    return hipGetLastError();
}

static bool in_one_go(const ExpandArgs &a) { return !a.first && a.alpha != 0.0f && probes_in_one_go(a.k); }
bool expand_needs_topk(const TopkArgs &t, const ExpandArgs &a) { return in_one_go(a) || t.per_part > 4 * BLOCK; }

hipError_t expand_prune(hipStream_t s, const TopkArgs &t, const ExpandArgs &a) {
    auto go = [&](auto kernel, int blocks) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(ENT), 0, s, t, a);
        return hipGetLastError();
    };
    if (in_one_go(a)) return go(expand_prune_kernel<false, true>, 1);
    if (expand_needs_topk(t, a)) return go(expand_prune_kernel<false, false>, 1);
    return go(expand_prune_kernel<true, false>, t.n_part);
}

hipError_t advance(hipStream_t s, DevState *st) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(1), 0, s, st);
    return hipGetLastError();
}

hipError_t set_drafts(hipStream_t s, DevState *st, const DraftArgs &a) {
    hipLaunchKernelGGL(set_drafts_kernel, dim3(1), dim3(WAVE), 0, s, st, a);
    return hipGetLastError();
}

hipError_t fill_i32(hipStream_t s, int32_t *p, int32_t v, int n) {
    hipLaunchKernelGGL(fill_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t fill3_i32(hipStream_t s, const FillRange &a, const FillRange &b, const FillRange &c) {
    const int most = std::max(a.n, std::max(b.n, c.n));
    hipLaunchKernelGGL(fill3_i32_kernel, dim3(std::max(1, std::min((most + 255) / 256, 2048))), dim3(256), 0, s, a, b, c);
    return hipGetLastError();
}

hipError_t init() {
    // Needed only for rows wider than 64 KB of fp32 x (e.g. d_ffn = 28672); a refusal here
    // surfaces later as a launch error for exactly those shapes.
    const int big = 160 * 1024 - 256;
    hipError_t e = hipSuccess;
#define SPD_SET(K) (void)hipFuncSetAttribute((const void *)(K), hipFuncAttributeMaxDynamicSharedMemorySize, big)
    SPD_SET((gemv_kernel<bf16_t, EPI_PLAIN>)); SPD_SET((gemv_kernel<bf16_t, EPI_RESID>));
    SPD_SET((gemv_kernel<bf16_t, EPI_QKV>)); SPD_SET((gemv_kernel<bf16_t, EPI_SWIGLU>));
    SPD_SET((gemv_kernel<float, EPI_PLAIN>)); SPD_SET((gemv_kernel<float, EPI_RESID>));
    SPD_SET((gemv_kernel<float, EPI_QKV>)); SPD_SET((gemv_kernel<float, EPI_SWIGLU>));
#undef SPD_SET
    (void)hipGetLastError();
    return e;
}

}  // namespace spdk
