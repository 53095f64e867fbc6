// Single-query attention over a key/value cache, one kernel per call (or two): the stand-alone
// operator and the forward that runs one kernel per operator.
//
// Bound: the cached keys and values stream through once (HBM, or the Infinity Cache where the
// cache fits it); the arithmetic is a few per cent of that.  So
//   * a block owns (key/value head, chunk of positions) and serves ALL query heads that share the
//     head from one read of its rows, GH of them side by side (a tile of query heads each);
//   * a position's row lies across LPP = d_head / VEC lanes (16-byte pieces), R rows of keys and of
//     values are requested per lane before the first is used;
//   * every group of LPP lanes runs its own flash-style softmax (running maximum and sum), so the
//     loop holds no barrier and no trip through LDS: a score is summed over its lanes with the
//     vector unit's lane-crossing moves and then known to all of them.  Groups meet at the end:
//     across the wave, then the waves through LDS, in a fixed order (bit-reproducible).
// A context cut into chunks leaves (max, sum, O) per chunk and a second kernel merges them in
// chunk order.  It replaces a kernel that kept the group's query heads in sequence (each
// re-reading the chunk) and whose last block per head merged, found by counters that a fill
// kernel cleared first.  Measured, us per call in a row, before -> after: 32 heads x 128, fp16, 80
// positions 9.8 -> 7.0 (host-bound; the kernel alone 2.0 + 5.8 -> 5.4), 1024 positions 27.7 -> 9.7;
// fp32, 4096 positions 150 -> 29 (4.6 TB/s); 64 query heads on 8 key/value heads, fp32, 4097
// positions 204 -> 16.0 through the C entry (kernels 201 -> 11.8 + 3.8; the Python entry also waits for its result: 33).
#include "spd_device.h"

using namespace spdd;

namespace {

constexpr int NTA = 256;             // threads per block
constexpr int NWA = NTA / WAVE;
constexpr int ONE_BYTES = 128 * 1024;// keys (or values) per head up to which a context is one chunk and one launch
constexpr int BLOCKS = 256;          // blocks a longer context is cut for
constexpr int SPLITS_MAX = 1024;     // chunks per head at most (the merge keeps their weights in LDS)

// Sum over groups of lpp consecutive lanes (a power of two), complete in every lane; N values
// step by step, so that the N independent moves of a step overlap.
template <int N>
__device__ __forceinline__ void group_sums_all(float (&v)[N], int lpp) {
    if (lpp >= 2) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_move<0xB1, 0xF>(v[i], 0.f);    // quad_perm [1,0,3,2]
    }
    if (lpp >= 4) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_move<0x4E, 0xF>(v[i], 0.f);    // quad_perm [2,3,0,1]
    }
    if (lpp >= 8) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_move<0x141, 0xF>(v[i], 0.f);   // row_half_mirror
    }
    if (lpp >= 16) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += dpp_move<0x140, 0xF>(v[i], 0.f);   // row_mirror
    }
    if (lpp >= 32) {
#pragma unroll
        for (int i = 0; i < N; ++i) {   // rows of 16 lanes in pairs
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i]), false, false);
            v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
    }
    if (lpp >= 64) {
#pragma unroll
        for (int i = 0; i < N; ++i) {   // the wave's two halves
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i]), false, false);
            v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
    }
}

// exp(a - b) with exp(-inf - anything) = 0, also where b is -inf (nothing seen yet).
__device__ __forceinline__ float exp_below(float a, float b) { return expf(a - (b == -INFINITY ? 0.f : b)); }

// Chunks per key/value head at most: one block per compute unit, two where a block's turn is long
// and it seldom has a second one.
__host__ __device__ inline int attn_splits(int group, int n_kv_heads, int max_splits) {
    const int splits = (group > 2 ? 2 * BLOCKS : BLOCKS) / n_kv_heads;
    return splits < 1 ? 1 : splits < max_splits ? splits : max_splits;
}

// Chunk length for n_ctx positions.  One chunk, and so one launch, while a block reads its head's
// rows faster than a second launch starts (32 heads of 128, us one chunk / cut: 256 positions fp16
// 6.8 / 9.2, 512 fp16 8.6 / 9.7, 256 fp32 7.6 / 9.9, 1024 fp16 14.2 / 9.7; 8 groups of 8, 512 fp32:
// 18.5 / 11.7); beyond, whole turns of a block's waves.
__host__ __device__ inline int attn_chunk(int n_ctx, int group, int n_kv_heads, int row_bytes, int max_splits) {
    if ((long long)n_ctx * row_bytes <= (group > 2 ? ONE_BYTES / 2 : ONE_BYTES)) return n_ctx;
    const int turn = group > 2 ? 128 : 64;   // positions a block takes at once (the least, over the element types)
    int splits = attn_splits(group, n_kv_heads, max_splits);
    return ((n_ctx + splits - 1) / splits + turn - 1) / turn * turn;
}

// Feature c of query head hq over one chunk: the result itself where there is only one.
__device__ __forceinline__ void store_chunk(const AttnArgs &a, int hq, int s, int n_splits, int c, float M, float L, float O) {
    if (n_splits == 1) {
        as_global(a.out)[(size_t)hq * a.d_head + c] = O / L;
        return;
    }
    float *pp = a.part + ((size_t)hq * a.max_splits + s) * (a.d_head + 2);
    as_global(pp)[2 + c] = O;
    if (c == 0) { as_global(pp)[0] = M; as_global(pp)[1] = L; }
}

// GH: query heads side by side; R: rows of keys and of values in flight per lane.
template <typename KT, int GH, int R>
__global__ __launch_bounds__(NTA, 2) void attn_split_kernel(const AttnArgs a) {
    constexpr int VEC = Store<KT>::VEC;
    typedef typename Store<KT>::piece_t piece_t;
    extern __shared__ __align__(16) float lds[];   // [NWA][GH][d_head] partial outputs
    __shared__ float lds_m[NWA][GH], lds_l[NWA][GH];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid / WAVE;
    const int dh = a.d_head, lpp = dh / VEC, ppw = WAVE / lpp, ppb = ppw * NWA;
    const int sub = lane / lpp, li = lane % lpp;
    const int n_ctx = a.st ? as_global(a.st)->pos + 1 : a.n_ctx;
    const int chunk = a.st ? attn_chunk(n_ctx, a.n_heads / a.n_kv_heads, a.n_kv_heads, dh * (int)sizeof(KT), a.max_splits) : a.chunk;
    const int n_splits = (n_ctx + chunk - 1) / chunk;
    const int g = blockIdx.x, s = blockIdx.y;
    if (s >= n_splits) return;
    const int t0 = s * chunk, t1 = min(n_ctx, t0 + chunk);
    const int group = a.n_heads / a.n_kv_heads;
    const float scale = 1.0f / sqrtf((float)dh);
    const char *Kg = (const char *)a.K + ((size_t)g * a.cap_ctx * dh + li * VEC) * sizeof(KT);
    const char *Vg = (const char *)a.V + ((size_t)g * a.cap_ctx * dh + li * VEC) * sizeof(KT);
    const size_t row = (size_t)dh * sizeof(KT);

    for (int h0 = 0; h0 < group; h0 += GH) {
        float qv[GH][VEC], acc[GH][VEC], m[GH], l[GH];
#pragma unroll
        for (int h = 0; h < GH; ++h) {
            const int hq = g * group + min(h0 + h, group - 1);   // (a ragged tile repeats its last head)
#pragma unroll
            for (int v = 0; v < VEC; ++v) { qv[h][v] = as_global(a.q)[(size_t)hq * dh + li * VEC + v]; acc[h][v] = 0.f; }
            m[h] = -INFINITY; l[h] = 0.f;
        }
        // (the bound is wave-uniform: every lane takes part in the lane-crossing sums)
        for (int b0 = t0 + wid * ppw; b0 < t1; b0 += R * ppb) {
            piece_t kb[R], vb[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {   // a row past the chunk re-reads the last one and gets weight zero
                const int t = min(b0 + sub + r * ppb, t1 - 1);
                kb[r] = kv_piece<KT>(Kg + (size_t)t * row);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int t = min(b0 + sub + r * ppb, t1 - 1);
                vb[r] = kv_piece<KT>(Vg + (size_t)t * row);
            }
            float d[R * GH];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float kf[VEC];
                Store<KT>::unpack(kb[r], kf);
#pragma unroll
                for (int h = 0; h < GH; ++h) {
                    float x = 0.f;
#pragma unroll
                    for (int v = 0; v < VEC; ++v) x = fmaf(kf[v], qv[h][v], x);
                    d[r * GH + h] = x;
                }
            }
            group_sums_all<R * GH>(d, lpp);
            float corr[GH];
#pragma unroll
            for (int h = 0; h < GH; ++h) {
                float mx = m[h];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool there = b0 + sub + r * ppb < t1;
                    d[r * GH + h] = there ? d[r * GH + h] * scale : -INFINITY;
                    mx = fmaxf(mx, d[r * GH + h]);
                }
                corr[h] = exp_below(m[h], mx);
                m[h] = mx;
                float ps = 0.f;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float p = exp_below(d[r * GH + h], mx);
                    d[r * GH + h] = p;
                    ps += p;
                }
                l[h] = l[h] * corr[h] + ps;
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[h][v] *= corr[h];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool there = b0 + sub + r * ppb < t1;
                float vf[VEC];
                Store<KT>::unpack(vb[r], vf);
#pragma unroll
                for (int h = 0; h < GH; ++h)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[h][v] = there ? fmaf(d[r * GH + h], vf[v], acc[h][v]) : acc[h][v];
            }
        }
        // the lane groups of the wave, ascending distance; then the waves, in wave order
#pragma unroll
        for (int dist = 1; dist < WAVE; dist <<= 1) {
            if (dist >= lpp) {
#pragma unroll
                for (int h = 0; h < GH; ++h) {
                    const float m2 = __shfl_xor(m[h], dist, WAVE), mx = fmaxf(m[h], m2);
                    const float f1 = exp_below(m[h], mx), f2 = exp_below(m2, mx);
                    l[h] = l[h] * f1 + __shfl_xor(l[h], dist, WAVE) * f2;
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[h][v] = acc[h][v] * f1 + __shfl_xor(acc[h][v], dist, WAVE) * f2;
                    m[h] = mx;
                }
            }
        }
        __syncthreads();   // the buffers of the previous tile of query heads have been read
        if (sub == 0) {
#pragma unroll
            for (int h = 0; h < GH; ++h) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) lds[(size_t)(wid * GH + h) * dh + li * VEC + v] = acc[h][v];
                if (li == 0) { lds_m[wid][h] = m[h]; lds_l[wid][h] = l[h]; }
            }
        }
        __syncthreads();
        for (int e = tid; e < GH * dh; e += NTA) {
            const int h = e / dh, c = e % dh, hq = g * group + h0 + h;
            if (h0 + h >= group) break;
            float M = lds_m[0][h], L = 0.f, O = 0.f;
#pragma unroll
            for (int w = 1; w < NWA; ++w) M = fmaxf(M, lds_m[w][h]);
#pragma unroll
            for (int w = 0; w < NWA; ++w) {
                const float f = exp_below(lds_m[w][h], M);
                L += f * lds_l[w][h];
                O += f * lds[(size_t)(w * GH + h) * dh + c];
            }
            store_chunk(a, hq, s, n_splits, c, M, L, O);
        }
    }
}

// Three or more query heads per key/value head: both products on the matrix cores, in fp32
// (v_mfma_f32_16x16x4_f32, exact products of fp32 values, as the vector path forms them), up to 16
// query heads side by side.  The vector path spends eight exponentials and eight lane-crossing
// sums per row and lane on the scores of a group of eight (26 us for 8 heads x 4097 positions, of
// which the bytes account for 7); here a lane holds four keys' scores of ONE head.
//   S^T [key, head] = K [key, d] Q^T [d, head]: k index kk of product (j, c) stands for feature
//     16 j + 4 kk + c, so a lane's share of a key is 16-byte pieces (four features each);
//   O^T [d, head] += V^T [d, key] P^T [key, head]: S^T's accumulator register r holds key 4 kk + r,
//     which is the operand layout of P^T when k index kk stands for that key -- the probabilities
//     stay in their registers; row i of product tile (jj, c) stands for feature 64 jj + 4 i + c.
// A wave takes two 16-key tiles per turn.
constexpr int HT = 16;               // query heads per tile
typedef float f32x4v __attribute__((ext_vector_type(4)));

template <typename KT> __device__ __forceinline__ void kv_four(const char *p, float *f);
template <> __device__ __forceinline__ void kv_four<float>(const char *p, float *f) {
    const float4 v = global_load_float4((const float *)p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
template <> __device__ __forceinline__ void kv_four<half_t>(const char *p, float *f) { Store<half4_t>::unpack(kv_piece<half4_t>(p), f); }
template <> __device__ __forceinline__ void kv_four<bf16_t>(const char *p, float *f) {
    const u32x2 v = kv_piece<half4_t>(p);
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
}

template <typename KT, int DH>
__global__ __launch_bounds__(NTA, DH <= 128 ? 2 : 1) void attn_group_kernel(const AttnArgs a) {
    constexpr int NJ = DH / 16, NV = DH / 64, TK = 2;   // 16-byte pieces of a key per lane; of a value row; tiles per turn
    __shared__ __align__(16) float lds[NWA][HT][DH];
    __shared__ float lds_m[NWA][HT], lds_l[NWA][HT];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid / WAVE, col = lane % 16, kk = lane / 16;
    const int n_ctx = a.st ? as_global(a.st)->pos + 1 : a.n_ctx;
    const int chunk = a.st ? attn_chunk(n_ctx, a.n_heads / a.n_kv_heads, a.n_kv_heads, DH * (int)sizeof(KT), a.max_splits) : a.chunk;
    const int n_splits = (n_ctx + chunk - 1) / chunk;
    const int g = blockIdx.x, s = blockIdx.y;
    if (s >= n_splits) return;
    const int t0 = s * chunk, t1 = min(n_ctx, t0 + chunk);
    const int group = a.n_heads / a.n_kv_heads;
    const float scale = 1.0f / sqrtf((float)DH);
    constexpr size_t ROW = (size_t)DH * sizeof(KT);
    const char *Kg = (const char *)a.K + (size_t)g * a.cap_ctx * ROW + 4 * kk * sizeof(KT);
    const char *Vg = (const char *)a.V + (size_t)g * a.cap_ctx * ROW + 4 * col * sizeof(KT);

    for (int h0 = 0; h0 < group; h0 += HT) {
        const int hq = g * group + min(h0 + col, group - 1);   // (columns past the group repeat its last head)
        float qv[NJ][4];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) qv[j][c] = as_global(a.q)[(size_t)hq * DH + 16 * j + 4 * kk + c];
        f32x4v o[NV][4];
#pragma unroll
        for (int jj = 0; jj < NV; ++jj)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[jj][c] = f32x4v{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, l = 0.f;
        for (int k0 = t0 + wid * 16 * TK; k0 < t1; k0 += NWA * 16 * TK) {
            float kf[TK][NJ][4], vf[TK][4][NV][4];
#pragma unroll
            for (int u = 0; u < TK; ++u) {
                const char *row = Kg + (size_t)min(k0 + 16 * u + col, t1 - 1) * ROW;
#pragma unroll
                for (int j = 0; j < NJ; ++j) kv_four<KT>(row + 16 * j * sizeof(KT), kf[u][j]);
            }
#pragma unroll
            for (int u = 0; u < TK; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const char *row = Vg + (size_t)min(k0 + 16 * u + 4 * kk + r, t1 - 1) * ROW;
#pragma unroll
                    for (int jj = 0; jj < NV; ++jj) kv_four<KT>(row + 64 * jj * sizeof(KT), vf[u][r][jj]);
                }
            // eight accumulators per tile: one chain of d_head / 4 products doubles the result's error
            f32x4v st[TK], part[TK][8];
#pragma unroll
            for (int u = 0; u < TK; ++u)
#pragma unroll
                for (int c = 0; c < 8; ++c) part[u][c] = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int u = 0; u < TK; ++u) part[u][4 * (j % 2) + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[u][j][c], qv[j][c], part[u][4 * (j % 2) + c], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < TK; ++u) st[u] = ((part[u][0] + part[u][1]) + (part[u][2] + part[u][3])) + ((part[u][4] + part[u][5]) + (part[u][6] + part[u][7]));
            float mx = m;
#pragma unroll
            for (int u = 0; u < TK; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    st[u][r] = k0 + 16 * u + 4 * kk + r < t1 ? st[u][r] * scale : -INFINITY;
                    mx = fmaxf(mx, st[u][r]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));   // the four lane groups hold different keys of the same heads
            mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
            const float corr = exp_below(m, mx);
            m = mx;
            l *= corr;
#pragma unroll
            for (int u = 0; u < TK; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    st[u][r] = exp_below(st[u][r], mx);
                    l += st[u][r];
                }
            if (k0 + 16 * TK > t1) {   // ragged end: rows past it must not meet an infinity in the row they repeat
#pragma unroll
                for (int u = 0; u < TK; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int jj = 0; jj < NV; ++jj)
#pragma unroll
                            for (int c = 0; c < 4; ++c) vf[u][r][jj][c] = k0 + 16 * u + 4 * kk + r < t1 ? vf[u][r][jj][c] : 0.f;
            }
#pragma unroll
            for (int jj = 0; jj < NV; ++jj)
#pragma unroll
                for (int c = 0; c < 4; ++c) o[jj][c] *= corr;
#pragma unroll
            for (int u = 0; u < TK; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int jj = 0; jj < NV; ++jj)
#pragma unroll
                        for (int c = 0; c < 4; ++c) o[jj][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[u][r][jj][c], st[u][r], o[jj][c], 0, 0, 0);
        }
        l += __shfl_xor(l, 16, WAVE);
        l += __shfl_xor(l, 32, WAVE);
        __syncthreads();   // the buffers of the previous tile of query heads have been read
#pragma unroll
        for (int jj = 0; jj < NV; ++jj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *(f32x4v *)&lds[wid][col][64 * jj + 4 * (4 * kk + r)] = f32x4v{o[jj][0][r], o[jj][1][r], o[jj][2][r], o[jj][3][r]};
        if (kk == 0) { lds_m[wid][col] = m; lds_l[wid][col] = l; }
        __syncthreads();
        for (int e = tid; e < min(HT, group - h0) * DH; e += NTA) {
            const int h = e / DH, c = e % DH;
            float M = lds_m[0][h], L = 0.f, O = 0.f;
#pragma unroll
            for (int w = 1; w < NWA; ++w) M = fmaxf(M, lds_m[w][h]);
#pragma unroll
            for (int w = 0; w < NWA; ++w) {
                const float f = exp_below(lds_m[w][h], M);
                L += f * lds_l[w][h];
                O += f * lds[w][h][c];
            }
            store_chunk(a, g * group + h0 + h, s, n_splits, c, M, L, O);
        }
    }
}

// One block per query head: the chunks' partial results in chunk order, thread group gi taking every
// (NTA / d_head)-th chunk.  A thread's first MB outputs are requested together with the chunks'
// (max, sum) pairs, so that up to MB * NTA / d_head chunks cost one trip to memory, not two.
constexpr int MB = 32;
__global__ __launch_bounds__(NTA) void attn_merge_kernel(const AttnArgs a, int row_bytes) {
    __shared__ float w[SPLITS_MAX], wl[SPLITS_MAX], sum[NTA];
    __shared__ float red[NWA];
    const int tid = threadIdx.x, dh = a.d_head, h = blockIdx.x;
    const int n_ctx = a.st ? as_global(a.st)->pos + 1 : a.n_ctx;
    const int chunk = a.st ? attn_chunk(n_ctx, a.n_heads / a.n_kv_heads, a.n_kv_heads, row_bytes, a.max_splits) : a.chunk;
    const int n_splits = (n_ctx + chunk - 1) / chunk;
    if (n_splits == 1) return;
    const float *ph = a.part + (size_t)h * a.max_splits * (dh + 2);
    const int groups = NTA / dh, gi = tid / dh, c = tid % dh;   // (d_head is at most NTA)
    float pv[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) pv[j] = as_global(ph)[(size_t)min(gi + j * groups, n_splits - 1) * (dh + 2) + 2 + c];
    float mq = -INFINITY;
    for (int q = tid; q < n_splits; q += NTA) {
        w[q] = as_global(ph)[(size_t)q * (dh + 2)];
        wl[q] = as_global(ph)[(size_t)q * (dh + 2) + 1];
        mq = fmaxf(mq, w[q]);
    }
    const float M = block_max<NTA>(mq, red);
    for (int q = tid; q < n_splits; q += NTA) {
        const float f = exp_below(w[q], M);
        w[q] = f;
        wl[q] *= f;
    }
    __syncthreads();
    float O = 0.f;
    if (gi < groups) {
#pragma unroll
        for (int j = 0; j < MB; ++j)
            if (gi + j * groups < n_splits) O += w[gi + j * groups] * pv[j];
        for (int q = gi + MB * groups; q < n_splits; q += groups) O += w[q] * as_global(ph)[(size_t)q * (dh + 2) + 2 + c];
    }
    sum[tid] = O;
    __syncthreads();
    if (tid >= dh) return;
    float L = 0.f;
    for (int q = 0; q < n_splits; ++q) L += wl[q];
    O = 0.f;
    for (int q = 0; q < groups; ++q) O += sum[q * dh + tid];
    as_global(a.out)[(size_t)h * dh + tid] = O / L;
}

template <typename KT>
hipError_t launch_attention(hipStream_t s, const AttnArgs &a_in) {
    AttnArgs a = a_in;
    a.max_splits = a.max_splits < SPLITS_MAX ? a.max_splits : SPLITS_MAX;
    const int group = a.n_heads / a.n_kv_heads, row_bytes = a.d_head * (int)sizeof(KT);
    // a position known to the device only: enough blocks for the longest context, and the merge unless that is one chunk
    int splits = attn_splits(group, a.n_kv_heads, a.max_splits);
    if (a.st && attn_chunk(a.cap_ctx, group, a.n_kv_heads, row_bytes, a.max_splits) == a.cap_ctx) splits = 1;
    if (!a.st) {
        a.chunk = attn_chunk(a.n_ctx, group, a.n_kv_heads, row_bytes, a.max_splits);
        splits = (a.n_ctx + a.chunk - 1) / a.chunk;
    }
    const dim3 grid(a.n_kv_heads, splits);
    auto lds = [&](int gh) { return (size_t)NWA * gh * a.d_head * sizeof(float); };
    if (group == 1) hipLaunchKernelGGL((attn_split_kernel<KT, 1, 8>), grid, dim3(NTA), lds(1), s, a);
    else if (group > 2 && a.d_head == 64) hipLaunchKernelGGL((attn_group_kernel<KT, 64>), grid, dim3(NTA), 0, s, a);
    else if (group > 2 && a.d_head == 128) hipLaunchKernelGGL((attn_group_kernel<KT, 128>), grid, dim3(NTA), 0, s, a);
    else if (group > 2 && a.d_head == 256) hipLaunchKernelGGL((attn_group_kernel<KT, 256>), grid, dim3(NTA), 0, s, a);
    else hipLaunchKernelGGL((attn_split_kernel<KT, 2, 8>), grid, dim3(NTA), lds(2), s, a);
    if (splits > 1) hipLaunchKernelGGL(attn_merge_kernel, dim3(a.n_heads), dim3(NTA), 0, s, a, row_bytes);
    return hipGetLastError();
}

}  // namespace

namespace spdk {

hipError_t attention(hipStream_t s, int dtype, const AttnArgs &a) {
    if (dtype == SPD_DTYPE_BF16) return launch_attention<bf16_t>(s, a);
    if (dtype == SPD_DTYPE_FP16) return launch_attention<half_t>(s, a);
    return launch_attention<float>(s, a);
}

}  // namespace spdk
