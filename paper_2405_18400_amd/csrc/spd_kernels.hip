// HIP kernels for one Superposed Decoding timestep on gfx950 (wave64).
//
// Batch-1 decode is a chain of matrix-vector products, so every kernel here is built
// around streaming weights from HBM exactly once with 128-bit loads; the only arithmetic
// that matters for time is keeping enough bytes in flight.  Reductions use a fixed order
// (no float atomics), so results are bit-reproducible run to run.
#include "spd_device.h"

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
        if (lane == 0) gemv_epilogue<WT, EPI>(a, unit, acc0, acc1, EPI == EPI_QKV ? a.st->pos : 0);
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
        if (seg == 0 && lane == WAVE - 1 && unit < n_units) gemv_epilogue<WT, EPI>(a, unit, acc0, acc1, EPI == EPI_QKV ? a.st->pos : 0);
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
// Total order used everywhere: larger value first, then smaller index.
__device__ __forceinline__ bool better(float va, int ia, float vb, int ib) {
    return va > vb || (va == vb && ia < ib);
}
// Block-wide arg-best; every thread gets the winner.  sv / si have NWAVE entries.
__device__ __forceinline__ void block_best(float &v, int &i, float *sv, int *si) {
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        const float ov = __shfl_xor(v, o, WAVE);
        const int oi = __shfl_xor(i, o, WAVE);
        if (better(ov, oi, v, i)) { v = ov; i = oi; }
    }
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) { sv[threadIdx.x / WAVE] = v; si[threadIdx.x / WAVE] = i; }
    __syncthreads();
    v = sv[0]; i = si[0];
#pragma unroll
    for (int w = 1; w < NWAVE; ++w)
        if (better(sv[w], si[w], v, i)) { v = sv[w]; i = si[w]; }
}

// Each block scans a contiguous slice of the logits: its k best entries, its max and its
// sum of exp((z - max)) with z = logit / tau.
__global__ __launch_bounds__(BLOCK) void topk_partial_kernel(const TopkArgs a) {
    __shared__ float sv[NWAVE];
    __shared__ int si[NWAVE];
    __shared__ float red[NWAVE];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int lo = b * a.per_part, hi = min(a.vocab, lo + a.per_part);
    // A thread's first NR entries of the slice stay in registers (all of them for slices of up
    // to NR * BLOCK entries); the kernel is a chain of block-wide reductions, so it reads its
    // logits once and takes the maximum from the first arg-best round (x -> x / tau is
    // monotonic for tau > 0: the largest logit gives the largest z).
    constexpr int NR = 4;
    float rv[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const int i = lo + tid + q * BLOCK;
        rv[q] = i < hi ? a.logits[i] : -INFINITY;
    }
    float pv = INFINITY;   // previous winner: everything "after" it in the total order is eligible
    int pi = -1;
    for (int r = 0; r < a.k; ++r) {
        float bv = -INFINITY;
        int bi = INT_MAX;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int i = lo + tid + q * BLOCK;
            if (i < hi && better(pv, pi, rv[q], i) && better(rv[q], i, bv, bi)) { bv = rv[q]; bi = i; }
        }
        for (int i = lo + tid + NR * BLOCK; i < hi; i += BLOCK) {
            const float v = a.logits[i];
            if (better(pv, pi, v, i) && better(v, i, bv, bi)) { bv = v; bi = i; }
        }
        block_best(bv, bi, sv, si);
        if (tid == 0) { a.pv[b * SPD_K_MAX + r] = bv; a.pi[b * SPD_K_MAX + r] = bi; }
        pv = bv; pi = bi;
        if (r == 0) {
            const float mx = lo < hi ? __fdiv_rn(bv, a.tau) : -INFINITY;
            float sm = 0.f;
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (lo + tid + q * BLOCK < hi) sm += expf(__fdiv_rn(rv[q], a.tau) - mx);
            for (int i = lo + tid + NR * BLOCK; i < hi; i += BLOCK) sm += expf(__fdiv_rn(a.logits[i], a.tau) - mx);
            sm = block_sum<BLOCK>(sm, red);
            float lowest = INFINITY;   // of the logits: x -> x / tau is monotonic
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (lo + tid + q * BLOCK < hi) lowest = fminf(lowest, rv[q]);
            for (int i = lo + tid + NR * BLOCK; i < hi; i += BLOCK) lowest = fminf(lowest, a.logits[i]);
            lowest = -block_max<BLOCK>(-lowest, red);
            if (tid == 0) { a.pm[b] = mx; a.ps[b] = sm; a.pn[b] = lo < hi ? __fdiv_rn(lowest, a.tau) : INFINITY; }
        }
    }
}

// ------------------------------------------------------------------ expand, interpolate, prune
// Linear probing, NG_PROBE_BATCH consecutive slots per trip to memory (32-byte slots: a batch
// is two or three cache lines; every trip is a random access into a table far larger than any
// cache, and the kernel waits for the longest chain of all its probes: at a load factor of 0.7
// some of a step's 60..360 probes walk past four slots, few past eight).  The slots are then
// examined in probing order, so the result is that of a slot-by-slot walk.
constexpr int NG_PROBE_BATCH = 8;
__device__ __forceinline__ unsigned long long ngram_probe(const NgramDev &ng, const int32_t *key) {
    uint64_t at = ngram_home(ngram_hash(key), ng.capacity);
    for (int p = 0; p <= ng.max_probe; p += NG_PROBE_BATCH) {
        u32x4 lo[NG_PROBE_BATCH], hi[NG_PROBE_BATCH];
#pragma unroll
        for (int j = 0; j < NG_PROBE_BATCH; ++j) {
            uint64_t idx = at + (uint64_t)j;
            while (idx >= ng.capacity) idx -= ng.capacity;
            const NgramSlot *sl = ng.slots + idx;
            lo[j] = *(const u32x4 *)sl;
            hi[j] = *((const u32x4 *)sl + 1);
        }
#pragma unroll
        for (int j = 0; j < NG_PROBE_BATCH; ++j) {
            if (p + j > ng.max_probe || (int32_t)lo[j].x == NG_EMPTY) return 0ull;
            if ((int32_t)lo[j].x == key[0] && (int32_t)lo[j].y == key[1] && (int32_t)lo[j].z == key[2] &&
                (int32_t)lo[j].w == key[3] && (int32_t)hi[j].x == key[4] && (int32_t)hi[j].y == key[5])
                return ((unsigned long long)hi[j].w << 32) | hi[j].z;
        }
        at += NG_PROBE_BATCH;
        while (at >= ng.capacity) at -= ng.capacity;
    }
    return 0ull;
}

// One block.  Merges the per-slice top-k into the global KeepTopK and log-softmax, builds the
// k x k options, probes the n-gram store for every (draft, kept token, order), applies the
// mixture (Eq. 3), the interpolation (Eq. 4) or the penalty form (Eq. 5), keeps the k best
// options and rewrites the draft state.
__global__ __launch_bounds__(BLOCK) void expand_prune_kernel(const ExpandArgs a) {
    __shared__ float sv[NWAVE];
    __shared__ int si[NWAVE];
    __shared__ int s_top[SPD_K_MAX];
    __shared__ float s_logp[SPD_K_MAX];
    __shared__ float s_lse;
    __shared__ float s_red[NWAVE];
    __shared__ float s_new[SPD_K_MAX];
    __shared__ int s_tails[SPD_K_MAX][SPD_TAIL];
    __shared__ float s_old[SPD_K_MAX];
    __shared__ unsigned long long s_cnt[SPD_KK * SPD_N_ORDERS];
    __shared__ unsigned long long s_tot[SPD_K_MAX * SPD_N_ORDERS];
    __shared__ float s_png[SPD_KK];
    __shared__ int s_any[SPD_K_MAX];
    __shared__ float s_score[SPD_KK];
    __shared__ int s_valid[SPD_KK];
    const int tid = threadIdx.x, k = a.k;
    DevState *st = a.st;

    // Everything this kernel reads from memory before the probes is requested at once: the
    // slices' candidates (a thread's first one stays in registers for all k rounds), the
    // slices' (max, sum-exp) pairs, the drafts' state.
    const int n_cand = a.n_part * k;
    float c0v = -INFINITY;
    int c0i = INT_MAX;
    if (tid < n_cand) {
        const int at = (tid / k) * SPD_K_MAX + (tid % k);
        c0v = a.pv[at];
        c0i = a.pi[at];
    }
    float my_m = -INFINITY;
    for (int b = tid; b < a.n_part; b += BLOCK) my_m = fmaxf(my_m, a.pm[b]);
    if (tid < SPD_K_MAX) {
        s_old[tid] = st->logscore[tid];
        s_any[tid] = 0;
        for (int q = 0; q < SPD_TAIL; ++q)
            s_tails[tid][q] = a.first ? st->prefix_tail[q] : st->tails[tid][q];
    }
    // log-sum-exp over the slices: M = max of the maxima, S = sum of sum-exp * exp(max - M)
    const float M = block_max<BLOCK>(my_m, s_red);
    float my_s = 0.f;
    for (int b = tid; b < a.n_part; b += BLOCK) my_s += a.ps[b] * expf(a.pm[b] - M);
    const float S = block_sum<BLOCK>(my_s, s_red);
    if (tid == 0) s_lse = M + logf(S);
    // global top-k of the slices' candidates
    float pv = INFINITY;
    int pi = -1;
    for (int r = 0; r < k; ++r) {
        float bv = -INFINITY;
        int bi = INT_MAX;
        if (better(pv, pi, c0v, c0i) && better(c0v, c0i, bv, bi)) { bv = c0v; bi = c0i; }
        for (int c = tid + BLOCK; c < n_cand; c += BLOCK) {
            const int at = (c / k) * SPD_K_MAX + (c % k);
            const float v = a.pv[at];
            const int i = a.pi[at];
            if (better(pv, pi, v, i) && better(v, i, bv, bi)) { bv = v; bi = i; }
        }
        block_best(bv, bi, sv, si);
        if (tid == 0) { s_top[r] = bi; s_logp[r] = bv; }
        pv = bv; pi = bi;
    }
    __syncthreads();
    if (tid < k) {
        s_logp[tid] = __fdiv_rn(s_logp[tid], a.tau) - s_lse;
        st->top_ids[tid] = s_top[tid];
        st->top_logp[tid] = s_logp[tid];
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
        for (int c = tid; c < k * k; c += BLOCK) {
            st->cand_score[c] = (c < k) ? s_logp[c] : -INFINITY;
            st->cand_valid[c] = (c < k);
            st->cand_png[c] = 0.f;
        }
    } else {
        const bool use_ng = a.alpha != 0.0f;
        if (use_ng) {
            const int n_probe = k * SPD_N_ORDERS + k * k * SPD_N_ORDERS;
            for (int e = tid; e < n_probe; e += BLOCK) {
                int i, j, n;
                const bool total = e < k * SPD_N_ORDERS;
                if (total) { i = e / SPD_N_ORDERS; j = 0; n = SPD_MIN_ORDER + e % SPD_N_ORDERS; }
                else {
                    const int f = e - k * SPD_N_ORDERS;
                    i = f / (k * SPD_N_ORDERS); j = (f / SPD_N_ORDERS) % k; n = SPD_MIN_ORDER + f % SPD_N_ORDERS;
                }
                unsigned long long res = 0ull;
                // the last n-1 tokens of the history must all exist
                if (a.ng.slots != nullptr && a.ng.present[n - SPD_MIN_ORDER] && s_tails[i][SPD_TAIL - (n - 1)] >= 0) {
                    int32_t key[6];
#pragma unroll
                    for (int q = 0; q < 6; ++q) key[q] = NG_PAD;
                    for (int q = 0; q < n - 1; ++q) key[q] = s_tails[i][SPD_TAIL - (n - 1) + q];
                    key[n - 1] = total ? NG_TOTAL : s_top[j];
                    res = ngram_probe(a.ng, key);
                }
                if (total) s_tot[i * SPD_N_ORDERS + (n - SPD_MIN_ORDER)] = res;
                else s_cnt[(i * k + j) * SPD_N_ORDERS + (n - SPD_MIN_ORDER)] = res;
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
            st->cand_score[tid] = s_score[tid];
            st->cand_valid[tid] = valid;
            st->cand_png[tid] = use_ng ? s_png[tid] : 0.f;
        }
        __syncthreads();
        if (tid < k * k && s_valid[tid]) {
            // rank among valid options: score desc, then parent asc, then token rank asc
            int rank = 0;
            for (int c = 0; c < k * k; ++c)
                if (s_valid[c] && better(s_score[c], c, s_score[tid], tid)) ++rank;
            if (rank < k) {
                const int i = tid / k, j = tid % k, gen = st->n_gen;
                for (int q = 0; q < SPD_TAIL - 1; ++q) st->tails[rank][q] = s_tails[i][q + 1];
                st->tails[rank][SPD_TAIL - 1] = s_top[j];
                st->logscore[rank] = s_score[tid];
                s_new[rank] = s_score[tid];
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
    __threadfence_block();
    if (tid == 0) {  // Eq. 2 on the new scores
        float mx = -INFINITY, sum = 0.f, g[SPD_K_MAX];
        for (int i = 0; i < k; ++i) mx = fmaxf(mx, s_new[i]);
        for (int i = 0; i < k; ++i) { g[i] = expf(s_new[i] - mx); sum += g[i]; }
        for (int i = 0; i < k; ++i) st->gamma[i] = g[i] / sum;
        st->k = k;
        st->n_gen = a.first ? 1 : st->n_gen + 1;
        if (a.advance) st->pos += 1;
    }
}

__global__ void advance_kernel(DevState *st) { st->pos += 1; }

__global__ void renorm_kernel(DevState *st, int k) {
    float mx = -INFINITY, sum = 0.f, g[SPD_K_MAX];
    for (int i = 0; i < k; ++i) mx = fmaxf(mx, st->logscore[i]);
    for (int i = 0; i < k; ++i) { g[i] = expf(st->logscore[i] - mx); sum += g[i]; }
    for (int i = 0; i < k; ++i) st->gamma[i] = g[i] / sum;
    st->k = k;
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
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
    hipLaunchKernelGGL(topk_partial_kernel, dim3(a.n_part), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t expand_prune(hipStream_t s, const ExpandArgs &a) {
    hipLaunchKernelGGL(expand_prune_kernel, dim3(1), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t advance(hipStream_t s, DevState *st) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(1), 0, s, st);
    return hipGetLastError();
}

hipError_t renorm(hipStream_t s, DevState *st, int k) {
    hipLaunchKernelGGL(renorm_kernel, dim3(1), dim3(1), 0, s, st, k);
    return hipGetLastError();
}

hipError_t fill_i32(hipStream_t s, int32_t *p, int32_t v, int n) {
    hipLaunchKernelGGL(fill_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, v, n);
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
