// Host-side construction of the device n-gram store: one exact-key open-addressing table
// holding every n-gram's count (the frequency tables of Section 4: one entry per distinct n-gram)
// plus, per distinct context, the sum of the counts of its continuations -- the denominator of
// p_{n-gram}(x | context) = count(context, x) / sum_x' count(context, x').
#include "spd_internal.h"

#include <algorithm>
#include <cstring>

uint64_t ngram_capacity_for(const spd_ngram_host_tables *t) {
    uint64_t n = 0;
    for (int o = 0; o < SPD_N_ORDERS; ++o) n += (uint64_t)(t->n_entries[o] > 0 ? t->n_entries[o] : 0);
    // every entry may add one context-total entry; keep the load factor <= 0.7
    uint64_t cap = (uint64_t)((double)(2 * n) / 0.7) + 64;
    return cap;
}

namespace {
// Linear probing with the entries of every run of taken slots in the order of their home slots: the longest displacement is then
// the least there is.  It bounds the device's walk for a key that is not stored, and a walk is a chain of trips to memory (120000
// n-grams: 15 slots, 50 .. 70 in the order they came in).  The order is kept while inserting: displacements lie beside the slots,
// a walk compares keys only where the home slots agree, and what has to make room moves up by one.
struct Builder {
    NgramHostTable &tab;
    uint64_t cap;
    std::vector<int32_t> dist;      // displacement of the entry in each slot, -1: empty

    Builder(NgramHostTable &t, uint64_t capacity) : tab(t), cap(capacity), dist(capacity, -1) {}
    uint64_t next(uint64_t at) const { return at + 1 == cap ? 0 : at + 1; }
    void prefetch(uint64_t home) const {
        __builtin_prefetch(&dist[home], 1);
        __builtin_prefetch(&tab.slots[home], 1);
    }

    // The slot of `key`, which it gets where it has none yet (count 0).
    NgramSlot &slot_of(const int32_t *key, uint64_t home, bool &found) {
        uint64_t at = home;
        int32_t p = 0;
        for (; dist[at] >= p; at = next(at), ++p)       // (the load factor is below 1: there is an empty slot)
            if (dist[at] == p && std::memcmp(tab.slots[at].tok, key, sizeof(tab.slots[at].tok)) == 0) {
                found = true;
                return tab.slots[at];
            }
        found = false;
        uint64_t end = at;
        while (dist[end] >= 0) end = next(end);
        for (uint64_t to = end; to != at;) {
            const uint64_t from = to == 0 ? cap - 1 : to - 1;
            tab.slots[to] = tab.slots[from];
            dist[to] = dist[from] + 1;
            tab.max_probe = std::max(tab.max_probe, dist[to]);
            to = from;
        }
        NgramSlot &s = tab.slots[at];
        std::memcpy(s.tok, key, sizeof(s.tok));
        s.cnt_lo = s.cnt_hi = 0;
        dist[at] = p;
        tab.max_probe = std::max(tab.max_probe, p);
        return s;
    }
};
}  // namespace

int ngram_build(const spd_ngram_host_tables *t, int32_t vocab, uint64_t capacity, NgramHostTable &out,
                std::string &err) {
    NgramSlot empty;
    for (int q = 0; q < 6; ++q) empty.tok[q] = NG_PAD;
    empty.tok[0] = NG_EMPTY;
    empty.cnt_lo = empty.cnt_hi = 0;
    out.slots.assign(capacity, empty);
    out.max_probe = 0;
    Builder b(out, capacity);
    // Every entry touches two places far apart: the home slots of a batch are asked for before the first is used (2 M
    // n-grams, the build: 340 ms one by one and unordered, 440 with a pass that ordered the runs afterwards, 270 so; 120000:
    // 9, 16, 6.6).
    constexpr int BATCH = 16;
    struct { int32_t key[6]; uint64_t home, total_home; const char *bad; } batch[BATCH];
    for (int o = 0; o < SPD_N_ORDERS; ++o) {
        const int n = o + SPD_MIN_ORDER;
        const int64_t N = t->n_entries[o];
        out.present[o] = N > 0;
        if (N < 0) { err = "negative entry count"; return SPD_EINVAL; }
        if (N > 0 && (!t->keys[o] || !t->counts[o])) { err = "null keys/counts for a non-empty order"; return SPD_EINVAL; }
        for (int64_t e0 = 0; e0 < N; e0 += BATCH) {
            const int m = (int)std::min<int64_t>(BATCH, N - e0);
            for (int i = 0; i < m; ++i) {
                auto &x = batch[i];
                const int32_t *src = t->keys[o] + (e0 + i) * n;
                x.bad = t->counts[o][e0 + i] == 0 ? "zero count" : nullptr;
                for (int q = 0; q < 6; ++q) {
                    x.key[q] = q < n ? src[q] : NG_PAD;
                    if (q < n && (src[q] < 0 || src[q] >= vocab)) x.bad = "token id outside [0, vocab)";
                }
                if (x.bad) continue;
                x.home = ngram_home(ngram_hash(x.key), capacity);
                b.prefetch(x.home);
                const int32_t token = x.key[n - 1];
                x.key[n - 1] = NG_TOTAL;   // the context's running total
                x.total_home = ngram_home(ngram_hash(x.key), capacity);
                b.prefetch(x.total_home);
                x.key[n - 1] = token;
            }
            for (int i = 0; i < m; ++i) {
                auto &x = batch[i];
                bool found = false;
                const char *why = x.bad;
                if (!why) {
                    NgramSlot &s = b.slot_of(x.key, x.home, found);
                    if (found) why = "duplicate key";
                    else s.cnt_lo = t->counts[o][e0 + i];
                }
                if (why) {
                    err = "order " + std::to_string(n) + " entry " + std::to_string(e0 + i) + ": " + why;
                    return SPD_ETABLE;
                }
                x.key[n - 1] = NG_TOTAL;
                NgramSlot &s = b.slot_of(x.key, x.total_home, found);
                const uint64_t tot = (((uint64_t)s.cnt_hi << 32) | s.cnt_lo) + t->counts[o][e0 + i];
                s.cnt_lo = (uint32_t)tot;
                s.cnt_hi = (uint32_t)(tot >> 32);
            }
        }
    }
    return SPD_OK;
}
