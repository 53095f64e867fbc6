// Nucleus (top-p) sampling of one token from the logits of a batch-1 forward pass: the
// comparison decoder of the paper's latency study (Section 4.3), k independent passes of which
// Superposed Decoding is timed against.  Section 2: keep the smallest set of most probable
// tokens whose cumulative probability reaches p, renormalise, sample.
//
// No sort.  With the vocabulary ordered by (probability descending, id ascending) both
// questions -- where does the nucleus end, which token does the draw u select by inverse CDF --
// are "the first entry, in that order, whose cumulative probability reaches (exceeds) x".
// Every entry's probability is a 40-bit fixed-point integer, so that probability masses are
// sums of integers: exact, and the same in whatever order they are added (the histograms below
// are built with atomic adds); its 64-bit sort key, ascending in that order, is that integer,
// inverted, above the token id.
//
//   stage A (one block per slice of the vocabulary, all compute units in parallel): scaled
//     logit z, probability, and a bucket number that is linear in z between the largest and the
//     smallest z with a probability above zero (2048 buckets), which is stored; mass and count per bucket of the slice (LDS
//     atomics), added to the histogram in memory (one atomic per bucket the slice touches; sums
//     of integers: the same in any order); the last block to finish goes on alone;
//   stage B: that histogram, prefix sums over the buckets, the bucket in which the cumulative
//     mass crosses x; should it hold more than a list's worth of entries it is cut again by key
//     range (2048 sub-buckets per round: at most a few rounds even where thousands of entries
//     tie); the bucket's entries are then ranked against one another (all pairs) and the first
//     one whose cumulative mass crosses x is the answer.
//   The first-level histogram serves both questions.
#include "spd_device.h"

#include <type_traits>

using namespace spdd;

namespace {

constexpr int SNT = 1024;          // threads per block
constexpr int SNW = SNT / WAVE;
constexpr int NB = 2 * SNT;        // buckets per level: two per thread in the prefix sums
constexpr int LC = 256;            // entries that are ranked pairwise
constexpr int ID_BITS = 23;        // token ids in a key (vocab <= 2^23)
constexpr int PIECE = 8 * SNT;     // entries of one 16-byte piece of bucket numbers per thread
constexpr float FX_ONE = 1099511627776.0f;   // 2^40: probability 1 in fixed point

// exp(x) in fixed point, <= 2^40 (1 + a few ulp); the same bits wherever it is formed from an entry's logit.
__device__ __forceinline__ unsigned long long fixed_point(float x) { return (unsigned long long)(expf(x) * FX_ONE); }
// Ascending in (probability descending, id ascending); pf < 2^41.
__device__ __forceinline__ unsigned long long sort_key(unsigned long long pf, int id) {
    return (((1ull << 41) - 1ull - pf) << ID_BITS) | (unsigned long long)(unsigned)id;
}

// A sum over the wave that every lane gets (no LDS, no barrier).
__device__ __forceinline__ float wave_all_sum(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_sum_last(v)), WAVE - 1)); }
__device__ __forceinline__ float wave_all_max(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_max_last(v)), WAVE - 1)); }

// 64-bit sums by lane-crossing moves (a shuffle is a trip through LDS per half and step).
template <int CTRL, int ROW_MASK = 0xF> __device__ __forceinline__ unsigned long long dpp_add64(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROW_MASK, 0xF, false);
    return v + (((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ unsigned long long wave_scan64(unsigned long long v) {   // inclusive
    v = dpp_add64<0x111>(v); v = dpp_add64<0x112>(v); v = dpp_add64<0x114>(v); v = dpp_add64<0x118>(v);   // row_shr 1, 2, 4, 8
    v = dpp_add64<0x142, 0xA>(v);                                                                       // row 0 -> 1, row 2 -> 3
    return dpp_add64<0x143, 0xC>(v);                                                                    // rows 0, 1 -> 2, 3
}
template <int LANES> __device__ __forceinline__ unsigned long long group_sum64(unsigned long long v) {   // over 4 or 16 lanes, in all of them
    static_assert(LANES == 4 || LANES == 16, "a quad or a row");
    v = dpp_add64<0xB1>(v); v = dpp_add64<0x4E>(v);
    if (LANES == 16) { v = dpp_add64<0x141>(v); v = dpp_add64<0x140>(v); }
    return v;
}

struct Stage {                                  // LDS of stage B
    unsigned long long hm[2][NB + 1];          // [level 1 / deeper levels]: per bucket, entry count above mass (one atomic add per
                                                // entry); then the exclusive prefix sums of both (totals at NB)
    unsigned long long wm[SNW];                 // per-wave totals of the prefix sums
    unsigned long long lk[LC], lp[LC], lcum[LC];   // the list: key, probability, mass of the entries up to and including it
    unsigned lrank[LC];                         // entries of the list before it
    int lid[LC];
    unsigned long long kmin, kmax;
    int found, lastb, n_list, best;
    int r_id;                                   // result of a search: the entry, its cumulative mass, its position in the order
    unsigned long long r_mass, r_key;
    unsigned r_index;
    float r_logit;
    int is_last;
    int q_bucket[2];                            // the two questions' crossings in the first-level histogram: the bucket (or -1),
    unsigned long long q_from[2], q_to[2];      // and the prefix sums before and behind it
    float ll[LC];                               // the list's logits
};

// A histogram word: entry count (20 bits: vocab <= 2^20... the sums of all masses stay below
// 2^41) above the mass.
constexpr int CNT_SHIFT = 44;
constexpr unsigned long long ONE_ENTRY = 1ull << CNT_SHIFT;
__device__ __forceinline__ unsigned long long mass_of(unsigned long long w) { return w & (ONE_ENTRY - 1ull); }
__device__ __forceinline__ unsigned count_of(unsigned long long w) { return (unsigned)(w >> CNT_SHIFT); }

// hm (NB values, this thread's two given) -> exclusive prefix sums, totals at index NB; this thread's three come back in
// registers, everybody's are in LDS after the next barrier.
__device__ __forceinline__ void prefix_sums(Stage &s, int lv, unsigned long long a0, unsigned long long a1, unsigned long long (&out)[3]) {
    const int t = threadIdx.x, lane = t & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(t / WAVE);
    const unsigned long long m = wave_scan64(a0 + a1);
    if (lane == WAVE - 1) s.wm[w] = m;
    __syncthreads();
    unsigned long long pm = 0;
#pragma unroll
    for (int q = 0; q < SNW - 1; ++q) pm += q < w ? s.wm[q] : 0ull;
    const unsigned long long em = pm + m - (a0 + a1);
    s.hm[lv][2 * t] = em; s.hm[lv][2 * t + 1] = em + a0;
    if (t == SNT - 1) s.hm[lv][NB] = em + a0 + a1;
    out[0] = em; out[1] = em + a0; out[2] = em + a0 + a1;
}

// The bucket in which the cumulative mass first reaches x (STRICT: exceeds x), or, if the
// total does not get there, the last bucket that holds an entry.  Every thread gets it.
template <bool STRICT>
__device__ __forceinline__ int crossing(Stage &s, int lv, unsigned long long x) {
    const int t = threadIdx.x;
    if (t == 0) { s.found = -1; s.lastb = 0; }
    __syncthreads();
    int last = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int b = 2 * t + q;
        const unsigned long long e = mass_of(s.hm[lv][b]), i = mass_of(s.hm[lv][b + 1]);
        if (STRICT ? (e <= x && i > x) : (e < x && i >= x)) s.found = b;     // one bucket at most
        if (count_of(s.hm[lv][b + 1]) > count_of(s.hm[lv][b])) last = b;
    }
    __syncthreads();
    if (s.found < 0) {   // (the same for every thread) nothing reaches x: one atomic per wave, not one per bucket on one address
        last = (int)wave_all_max((float)last);   // bucket numbers are exact in a float
        if ((t & (WAVE - 1)) == 0) atomicMax(&s.lastb, last);
        __syncthreads();
    }
    const int b = s.found >= 0 ? s.found : s.lastb;
    __syncthreads();
    return b;
}

// The bucket numbers (one more, so that zero is no entry: past the vocabulary, where a load past the array's end returns zeros), 16 bits
// per entry, written through to memory by stage A and read back coherently (the writers sit behind other L2 caches; a device-wide fence
// would write back and invalidate whole caches -- tens of microseconds).  Stage B looks for the entries of ONE bucket at a time and reads
// the logits of those.  A thread keeps PIECES pieces of eight numbers in registers; 0: the vocabulary has more, every walk reads them
// again.  Beyond 32768 entries the last block used to build the histogram itself from eight bytes per entry, which every walk read again.
// The kernel by events, top_p 0.9, 32000 / 40000 / 50258 / 65536 / 100000 / 131072 / 262144 entries: 14.4 / 28.7 / 33.5 / 38.2 / 54.9 / 64.6 / 175 ->
// 13.7 / 15.2 / 16.3 / 17.6 / 22.9 / 26.0 / 47.6 us.
constexpr int REREAD = 8;          // pieces per trip of a walk that reads the numbers again
template <int PIECES>
struct Entries {
    static constexpr int HELD = PIECES ? PIECES : REREAD;
    __amdgpu_buffer_rsrc_t ids;
    int vocab;
    const float *logits;
    float tau, lse;
    unsigned bk[4 * HELD];
    __device__ __forceinline__ void load(int first) {
#pragma unroll
        for (int r = 0; r < HELD; ++r) {
            const u32x4 v = coherent_load16(ids, 16u * (threadIdx.x + (unsigned)((first + r) * SNT)));
            bk[4 * r] = v.x; bk[4 * r + 1] = v.y; bk[4 * r + 2] = v.z; bk[4 * r + 3] = v.w;
        }
    }
    // entry c of this thread
    static __device__ __forceinline__ int entry(int c) { return 8 * ((int)threadIdx.x + (c / 8) * SNT) + (c % 8); }
    // f(i, its probability, its logit) for every entry of bucket b1 that this thread holds, its first one number 8 first
    template <typename F>
    __device__ __forceinline__ void walk_held(int first, int b1, F &&f) {
        constexpr int G = HELD / 4;
        static_assert(HELD % 4 == 0, "a word of hits has one bit per entry of four pieces");
        const unsigned both = (unsigned)(b1 + 1) | ((unsigned)(b1 + 1) << 16);
        unsigned hits[G], any = 0u;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            unsigned others = 0u;                   // bit 15 - r: the lower number of register r is another; bit 31 - r: the upper one
#pragma unroll
            for (int r = 0; r < 16; ++r) {          // (three instructions for two bucket numbers: the block's waves share four SIMDs)
                unsigned other;
                asm("v_pk_min_u16 %0, %1, %2" : "=v"(other) : "v"(bk[16 * g + r] ^ both), "v"(0x00010001u));
                others = (others << 1) | other;
            }
            hits[g] = ~others;
            any |= hits[g];
        }
        auto next = [&]() {                         // (of the first word that has one, so that a lane's turns are as many as its entries)
            unsigned word = hits[G - 1];
            int at = G - 1;
#pragma unroll
            for (int g = G - 2; g >= 0; --g)
                if (hits[g]) { word = hits[g]; at = g; }
            const int bit = __ffs(word) - 1;
            word &= word - 1u;
            any = 0u;
#pragma unroll
            for (int g = 0; g < G; ++g) { hits[g] = g == at ? word : hits[g]; any |= hits[g]; }
            return entry(8 * first + 32 * at + 2 * (15 - bit % 16) + bit / 16);
        };
        while (any) {   // (few: a bucket holds some dozens of the block's entries; two at a time)
            const int i0 = next();
            const bool two = any != 0u;
            int i1 = i0;
            if (two) i1 = next();
            const float l0 = as_global(logits)[i0], l1 = as_global(logits)[i1];
            f(i0, fixed_point(__fdiv_rn(l0, tau) - lse), l0);
            if (two) f(i1, fixed_point(__fdiv_rn(l1, tau) - lse), l1);
        }
    }
    // the same for every entry of the bucket among this thread's
    template <typename F>
    __device__ __forceinline__ void walk_bucket(int b1, F &&f) {
        if (PIECES) { walk_held(0, b1, f); return; }
        for (int first = 0; first * PIECE < vocab; first += REREAD) {
            load(first);
            walk_held(first, b1, f);
        }
    }
    // the highest token of the bucket among this thread's, -1: none
    __device__ __forceinline__ int last_of_bucket(int b1) {
        int last = -1;
        for (int first = 0; PIECES ? first == 0 : first * PIECE < vocab; first += REREAD) {
            if (!PIECES) load(first);
#pragma unroll
            for (int r = 0; r < 4 * HELD; ++r) {    // (a thread's tokens ascend)
                if ((bk[r] & 0xFFFFu) == (unsigned)(b1 + 1)) last = entry(8 * first + 2 * r);
                if (bk[r] >> 16 == (unsigned)(b1 + 1)) last = entry(8 * first + 2 * r + 1);
            }
        }
        return last;
    }
};

// The first entry in the order whose cumulative mass reaches (STRICT: exceeds) x; the last
// entry if none does.  Level-1 prefix sums are in s.hm[0].  Result in s.r_*.
template <bool STRICT, int PIECES>
__device__ __forceinline__ void search(Stage &s, Entries<PIECES> &en, unsigned long long x) {
    const int t = threadIdx.x;
    const int b1 = crossing<STRICT>(s, 0, x);
    unsigned long long base_m = mass_of(s.hm[0][b1]);
    unsigned base_c = count_of(s.hm[0][b1]);
    unsigned n = count_of(s.hm[0][b1 + 1]) - base_c;
    if (mass_of(s.hm[0][b1 + 1]) == base_m) {   // (the same for every thread) nothing reaches x and the last bucket has no mass: its entries stand by id.
                                                // (50258 entries, 97 % of them -inf, top_p 1: 548 -> 15 us)
        if (t == 0) s.best = -1;
        __syncthreads();
        const int last = (int)wave_all_max((float)en.last_of_bucket(b1));   // (ids are exact in a float)
        if ((t & (WAVE - 1)) == 0) atomicMax(&s.best, last);
        __syncthreads();
        if (t == 0) { s.r_id = s.best; s.r_key = sort_key(0ull, s.best); s.r_mass = base_m; s.r_index = base_c + n - 1u; }
        __syncthreads();
        return;
    }
    // the candidates: level-1 bucket b1, and within it the key range [klo, khi] once it has been cut
    unsigned long long klo = 0ull, khi = ~0ull;
    bool cut = false;
    while (n > (unsigned)LC) {
        if (!cut) {   // the key range of the bucket's entries
            if (t == 0) { s.kmin = ~0ull; s.kmax = 0ull; }
            __syncthreads();
            unsigned long long lowest = ~0ull, highest = 0ull;   // (joined by wave: an atomic per entry, all on two addresses, was most of the search; equal logits, 32000 / 131072 entries: 670 / 2687 -> 107 / 413 us)
            en.walk_bucket(b1, [&](int i, unsigned long long pf, float) {
                const unsigned long long k = sort_key(pf, i);
                lowest = min(lowest, k);
                highest = max(highest, k);
            });
#pragma unroll
            for (int o = WAVE / 2; o > 0; o >>= 1) {
                lowest = min(lowest, (unsigned long long)__shfl_xor(lowest, o, WAVE));
                highest = max(highest, (unsigned long long)__shfl_xor(highest, o, WAVE));
            }
            if ((t & (WAVE - 1)) == 0) { atomicMin(&s.kmin, lowest); atomicMax(&s.kmax, highest); }
            __syncthreads();
            klo = s.kmin; khi = s.kmax;
            cut = true;
        }
        const unsigned long long width = khi - klo;                 // > 0: more than one entry, keys are distinct
        const int bits = 64 - __clzll((long long)width);
        const int sh = bits > 11 ? bits - 11 : 0;                  // (k - klo) >> sh < 2048
        s.hm[1][2 * t] = 0ull; s.hm[1][2 * t + 1] = 0ull;
        __syncthreads();
        en.walk_bucket(b1, [&](int i, unsigned long long pf, float) {
            const unsigned long long k = sort_key(pf, i);
            if (k >= klo && k <= khi) {
                const int b2 = (int)((k - klo) >> sh);
                atomicAdd(&s.hm[1][b2], pf + ONE_ENTRY);
            }
        });
        __syncthreads();
        unsigned long long sums[3];
        prefix_sums(s, 1, s.hm[1][2 * t], s.hm[1][2 * t + 1], sums);
        __syncthreads();
        const int b2 = crossing<STRICT>(s, 1, x - base_m);          // (x >= base_m: the crossing lies in this range or beyond everything)
        base_m += mass_of(s.hm[1][b2]);
        base_c += count_of(s.hm[1][b2]);
        n = count_of(s.hm[1][b2 + 1]) - count_of(s.hm[1][b2]);
        klo += (unsigned long long)b2 << sh;
        const unsigned long long span = (1ull << sh) - 1ull;       // (klo + span itself may pass 2^64: keys of probabilities near zero end there)
        khi = khi - klo > span ? klo + span : khi;
        __syncthreads();
    }
    // the candidates into the list (in any order: they are ranked below)
    if (t == 0) { s.n_list = 0; s.best = INT_MAX; }
    if (t < LC) { s.lrank[t] = 0u; s.lcum[t] = 0ull; }
    __syncthreads();
    en.walk_bucket(b1, [&](int i, unsigned long long pf, float) {
        const unsigned long long k = sort_key(pf, i);
        if (k >= klo && k <= khi) {
            const int at = atomicAdd(&s.n_list, 1);
            s.lk[at] = k; s.lp[at] = pf; s.lid[at] = i;
        }
    });
    __syncthreads();
    const int nl = s.n_list;   // == n
    {   // all pairs: entry i against one part of the list each; the shorter the list, the more parts
        const int slots = nl <= 32 ? 32 : nl <= 64 ? 64 : nl <= 128 ? 128 : LC;
        const int i = t % slots, part = t / slots;
        const int PARTS = SNT / slots;
        if (i < nl) {
            const unsigned long long ki = s.lk[i];
            unsigned cnt = 0u;
            unsigned long long mass = 0ull;
            for (int j = part; j < nl; j += PARTS) {
                const unsigned long long kj = s.lk[j];
                if (kj < ki) ++cnt;
                if (kj <= ki) mass += s.lp[j];
            }
            atomicAdd(&s.lrank[i], cnt);
            atomicAdd(&s.lcum[i], mass);
        }
    }
    __syncthreads();
    if (t < nl) {
        const unsigned long long tot = base_m + s.lcum[t];
        if (STRICT ? tot > x : tot >= x) atomicMin(&s.best, (int)s.lrank[t]);
    }
    __syncthreads();
    const int pick = s.best == INT_MAX ? nl - 1 : s.best;   // nothing reaches x: the last entry
    if (t < nl && (int)s.lrank[t] == pick) {
        s.r_id = s.lid[t]; s.r_key = s.lk[t];
        s.r_mass = base_m + s.lcum[t];
        s.r_index = base_c + (unsigned)pick;
    }
    __syncthreads();
}

// The same question where the crossing bucket of the first-level histogram fits the list (nearly always): three barriers
// instead of nine.  w[0 .. 2]: the prefix sums around this thread's two buckets, still in its registers; the bucket's
// entry whose cumulative mass crosses x is the one that reaches it while the entry before does not, which each entry
// knows by itself once it has its rank and mass.  Slots of Stage are per question, cleared beforehand.  32000 entries, the kernel:
// 15.2 -> 13.2 us.
template <bool STRICT, int PIECES>
__device__ __forceinline__ void ask(Stage &s, Entries<PIECES> &en, const float *logits, int which, unsigned long long x, const unsigned long long (&w)[3]) {
    const int t = threadIdx.x;
    auto reaches = [&](unsigned long long m) { return STRICT ? m > x : m >= x; };
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (!reaches(mass_of(w[q])) && reaches(mass_of(w[q + 1]))) { s.q_bucket[which] = 2 * t + q; s.q_from[which] = w[q]; s.q_to[which] = w[q + 1]; }
    __syncthreads();
    const int b1 = s.q_bucket[which];
    const unsigned long long from = s.q_from[which];
    const unsigned base_c = count_of(from);
    if (b1 < 0 || count_of(s.q_to[which]) - base_c > (unsigned)LC) {   // (the same for every thread)
        if constexpr (PIECES == 8) {   // (its own registers beside these would be more than there are: the numbers are read again)
            Entries<0> again;
            again.ids = en.ids; again.vocab = en.vocab; again.logits = en.logits; again.tau = en.tau; again.lse = en.lse;
            search<STRICT, 0>(s, again, x);
            if (!STRICT) en.load(0);
        } else {
            search<STRICT, PIECES>(s, en, x);
        }
        if (t == 0) s.r_logit = as_global(logits)[s.r_id];
        __syncthreads();
        return;
    }
    en.walk_bucket(b1, [&](int i, unsigned long long pf, float l) {
        const int at = atomicAdd(&s.n_list, 1);
        s.lk[at] = sort_key(pf, i); s.lp[at] = pf; s.lid[at] = i; s.ll[at] = l;
    });
    __syncthreads();
    const int nl = s.n_list;
    auto rank = [&](auto parts) {      // PARTS lanes side by side compare an entry with every PARTS-th one each
        constexpr int PARTS = decltype(parts)::value;
        const int i = t / PARTS, part = t % PARTS;
        unsigned cnt = 0u;
        unsigned long long mass = 0ull;
        if (i < nl) {
            const unsigned long long ki = s.lk[i];
            constexpr int SIDE = 4;    // pairs side by side: their reads of the list are one trip to LDS (one by one: 65536 entries, top_p 0.98 19.5 -> 18.0 us)
            for (int j0 = part; j0 < nl; j0 += SIDE * PARTS) {
                unsigned long long kj[SIDE], pj[SIDE];
#pragma unroll
                for (int q = 0; q < SIDE; ++q) { const int j = min(j0 + q * PARTS, LC - 1); kj[q] = s.lk[j]; pj[q] = s.lp[j]; }
#pragma unroll
                for (int q = 0; q < SIDE; ++q)
                    if (j0 + q * PARTS < nl && kj[q] < ki) { ++cnt; mass += pj[q]; }
            }
        }
        mass = group_sum64<PARTS>(mass + ((unsigned long long)cnt << CNT_SHIFT));   // (as in a histogram word: at most 256 entries, masses below 2^42)
        cnt = count_of(mass);
        mass = mass_of(mass);
        if (i < nl && part == 0) {
            const unsigned long long before = mass_of(from) + mass, tot = before + s.lp[i];
            const bool crosses = reaches(tot) && (cnt == 0u || !reaches(before));
            if (crosses || (cnt == (unsigned)nl - 1u && !reaches(tot))) {   // (nothing reaches x: the last entry)
                s.r_id = s.lid[i]; s.r_key = s.lk[i]; s.r_logit = s.ll[i];
                s.r_mass = tot; s.r_index = base_c + cnt;
            }
        }
    };
    if (nl <= 64) rank(std::integral_constant<int, 16>());
    else rank(std::integral_constant<int, 4>());
    __syncthreads();
}

template <int PIECES>
__global__ __launch_bounds__(SNT) void nucleus_kernel(const NucleusArgs a) {
    __shared__ Stage s;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    global_ptr<DevState> st = as_global(a.st);
    // log-sum-exp, largest and smallest scaled logit from the per-slice statistics (every wave for itself); this thread's first logit comes
    // along: one trip to memory instead of three.  32000 entries, cycles from the block's start, before -> now (with the sums by lane-crossing
    // moves, probabilities of a bucket's entries formed again from their logits instead of stored and fetched, and three instructions
    // instead of eight for two bucket numbers): slice 5400 -> 5200, counted 9100 -> 9500, histogram and sums 12800 -> 13900, the nucleus 20300 ->
    // 20100, the draw 25200 -> 23800, end 26500 -> 24500; four tokens 77.3 -> 73.8 us.
    const int lo = blockIdx.x * a.per_part, hi = min(a.vocab, lo + a.per_part);
    const float first_logit = as_global(a.logits)[min(lo + tid, a.vocab - 1)];
    static_assert(TOPK_PART_MAX == 2 * WAVE, "two slices per lane");
    float pm[2], pn[2], ps[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int b = min(lane + q * WAVE, a.n_part - 1);
        pm[q] = as_global(a.pm)[b]; pn[q] = as_global(a.pn)[b]; ps[q] = as_global(a.ps)[b];
    }
    const float M = wave_all_max(fmaxf(pm[0], pm[1])), mn = -wave_all_max(-fminf(pn[0], pn[1]));   // (a slice looked at twice changes neither)
    float S = 0.f;
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (lane + q * WAVE < a.n_part) S += ps[q] * expf(pm[q] - M);
    const float lse = M + logf(wave_all_sum(S));
    // The buckets end where the fixed-point probabilities do (exp(-29) 2^40 < 1), the rest shares the last one: masked logits (-inf, -FLT_MAX, -1e9)
    // would stretch them until all live entries fell into one.  Half of the entries -inf, top_p 0.9,
    // 32000 / 50258 / 131072 entries, the kernel by events: 382 / 603 / 1482 -> 12.9 / 14.7 / 20.9 us.
    const float range = M - fmaxf(mn, lse - 29.f);
    const float scale = range > 0.f ? (float)NB / range : 0.f;

    // ---- stage A: this block's slice
    s.hm[1][2 * tid] = 0ull; s.hm[1][2 * tid + 1] = 0ull;          // the slice's histogram
    __syncthreads();
    const int end = hi == a.vocab ? (hi + 7) & ~7 : hi;           // (a piece that the vocabulary ends in: no entries behind it)
    for (int i = lo + tid; i < end; i += SNT) {
        if (i >= hi) { __hip_atomic_store(as_global(a.sc_bk) + i, (uint16_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); continue; }
        const float z = __fdiv_rn(i < lo + SNT ? first_logit : as_global(a.logits)[i], a.tau);
        const float fb = (M - z) * scale;                          // monotonic in z; anything beyond lands in the last bucket
        const int b = fb < (float)(NB - 1) ? (int)fb : NB - 1;
        const int bb = b < 0 ? 0 : b;
        __hip_atomic_store(as_global(a.sc_bk) + i, (uint16_t)(bb + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicAdd(&s.hm[1][bb], fixed_point(z - lse) + ONE_ENTRY);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const unsigned long long w = s.hm[1][2 * tid + q];
        if (w) (void)__hip_atomic_fetch_add(as_global(a.sc_hist) + 2 * tid + q, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's write-through stores have been acknowledged
    __syncthreads();
    if (tid == 0) s.is_last = (__hip_atomic_fetch_add(as_global(a.sc_count), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(gridDim.x - 1));
    __syncthreads();
    if (!s.is_last) return;

    // ---- stage B: first-level histogram
    // (the state it ends with is asked for now: at the end it would be one more trip to memory)
    const float u = a.u >= 0.f ? a.u : st->sample_u, old_score = a.first ? 0.f : st->logscore[0];
    const int gen = a.first ? 0 : st->n_gen, pos = st->pos;
    int tail[SPD_TAIL];
#pragma unroll
    for (int q = 0; q < SPD_TAIL; ++q) tail[q] = a.first ? st->prefix_tail[q] : st->tails[0][q];
    Entries<PIECES> en;
    en.ids = __builtin_amdgcn_make_buffer_rsrc(a.sc_bk, 0, ((a.vocab + 7) & ~7) * 2, 0x00020000);
    en.vocab = a.vocab; en.logits = a.logits; en.tau = a.tau; en.lse = lse;
    if (tid == 0) { s.q_bucket[0] = s.q_bucket[1] = -1; s.n_list = 0; }
    // the histogram all blocks have added to (left at zero for the next call), and this thread's bucket numbers
    const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(a.sc_hist, 0, NB * 8, 0x00020000);
    const u32x4 v = coherent_load16(hrs, 16u * (unsigned)tid);   // one 16-byte piece: this thread's two words
    if (PIECES) en.load(0);
    const unsigned long long h0 = ((unsigned long long)v.y << 32) | v.x, h1 = ((unsigned long long)v.w << 32) | v.z;
    unsigned long long sums[3];
    prefix_sums(s, 0, h0, h1, sums);

    // 1. the nucleus: the first entry whose cumulative probability reaches top_p, and all before it
    // (at least one unit: a top_p below 2^-40 is the likeliest entry alone, not a mass that nothing has to reach)
    const unsigned long long x_p = max(1ull, (unsigned long long)((double)a.top_p * (double)FX_ONE));
    ask<false, PIECES>(s, en, a.logits, 0, x_p, sums);
    const unsigned long long mass_fx = s.r_mass, key_T = s.r_key;
    const unsigned size = s.r_index + 1u;
    const int id_T = s.r_id;
    const float logit_T = s.r_logit;
    if (tid == 0) s.n_list = 0;     // (everybody has read it; the next barrier stands before its next use)
    // 2. the draw: the first entry whose cumulative probability exceeds u * mass (within the nucleus)
    const unsigned long long x_u = (unsigned long long)((double)u * (double)mass_fx);
    ask<true, PIECES>(s, en, a.logits, 1, x_u, sums);
    int tok = s.r_id;
    float logit = s.r_logit;
    if (s.r_key > key_T) { tok = id_T; logit = logit_T; }   // (only rounding could take it past the nucleus)

    __hip_atomic_store(as_global(a.sc_hist) + 2 * tid, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(as_global(a.sc_hist) + 2 * tid + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) {   // the pass's state: one draft (k = 1, gamma = 1)
        const float logp = __fdiv_rn(logit, a.tau) - lse;
#pragma unroll
        for (int q = 0; q < SPD_TAIL - 1; ++q) st->tails[0][q] = tail[q + 1];
        st->tails[0][SPD_TAIL - 1] = tok;
        st->logscore[0] = a.first ? logp : old_score + logp;
        st->gamma[0] = 1.f;
        st->new_tok[0] = tok;
        st->new_parent[0] = a.first ? -1 : 0;
        st->top_ids[0] = tok;
        st->top_logp[0] = logp;
        if (gen < a.max_gen) { as_global(a.hist_tok)[(size_t)gen * SPD_K_MAX] = tok; as_global(a.hist_par)[(size_t)gen * SPD_K_MAX] = a.first ? -1 : 0; }
        st->nucleus_size = (int)size;
        st->nucleus_mass = (float)((double)mass_fx / (double)FX_ONE);
        st->k = 1;
        st->n_gen = gen + 1;
        if (a.advance) st->pos = pos + 1;
        __hip_atomic_store(as_global(a.sc_count), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next call
    }
}

}  // namespace

namespace spdk {

// As many pieces of bucket numbers per thread as hold the vocabulary, up to eight.  The kernel by events, 40000 and 65536 entries, eight held
// 14.2 and 15.8 us at top_p 0.5, 15.2 and 17.6 at 0.9; read again 14.4 and 15.9, 15.4 and 17.7.  65538 and 131072 entries, top_p 0.5, sixteen held 18.7
// and 22.2 (and four registers spilled), read again 17.7 and 21.6.
hipError_t nucleus(hipStream_t s, const NucleusArgs &a) {
    const dim3 grid(a.n_part), block(SNT);
    if (a.vocab <= 4 * PIECE) hipLaunchKernelGGL(nucleus_kernel<4>, grid, block, 0, s, a);
    else if (a.vocab <= 8 * PIECE) hipLaunchKernelGGL(nucleus_kernel<8>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(nucleus_kernel<0>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace spdk
