// Host-side check of the hash that spreads history ids over the tables of the grouping and the cache (id_hash in
// device_utils.h), compiled for the host only and run by tests/test_host_hash.py: ids with their information in few of their
// bits (counters at every position, pairs of counters, numbers as floating point, pointers) take no longer probe chains than 64 random bits
// do, with slots one apart and with a step of the id's own, in tables half full.  Prints "ok" or the first chain that is too long.
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "device_utils.h"

using namespace rnnlm;

static uint64_t next_random(uint64_t &s) {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

static int longest_chain(const std::vector<uint64_t> &ids, bool own_step) {
    size_t cap = 64;
    while (cap < 2 * ids.size()) cap <<= 1;
    std::vector<char> taken(cap, 0);
    int longest = 0;
    for (uint64_t id : ids) {
        const uint32_t h = id_hash(id), step = own_step ? h >> 16 | 1 : 1;
        size_t s = h & (cap - 1);
        int probes = 1;
        for (; taken[s]; ++probes) s = (s + step) & (cap - 1);
        taken[s] = 1;
        longest = std::max(longest, probes);
    }
    return longest;
}

static int check(const char *what, int a, int b, std::vector<uint64_t> ids) {
    std::sort(ids.begin(), ids.end());
    ids.erase(std::unique(ids.begin(), ids.end()), ids.end());
    uint64_t seed = ids.size();
    for (size_t i = ids.size(); i > 1; --i) std::swap(ids[i - 1], ids[next_random(seed) % i]);
    // 4000 random ids: chains of up to 35 and 13 over twenty draws; the mixed 64 bits of counters on the sets below 40 and 19
    const int one = longest_chain(ids, false), own = longest_chain(ids, true);
    if (one <= 60 && own <= 25) return 0;
    printf("FAILED %s %d %d, %zu ids: %d probes one apart, %d with a step of the id's own\n", what, a, b, ids.size(), one, own);
    return 1;
}

int main() {
    int bad = 0;
    for (size_t n : {60u, 500u, 1000u, 2000u, 4000u}) {
        auto set = [&](auto id_of) {
            std::vector<uint64_t> ids;
            for (uint64_t i = 3; i < n + 3; ++i) ids.push_back(id_of(i));
            return ids;
        };
        uint64_t seed = n;
        bad += check("random", 0, 0, set([&](uint64_t) { return next_random(seed); }));
        bad += check("counter over random bits", 0, 0, set([&](uint64_t i) { return i << 32 | (next_random(seed) & 0x7FFFFFFF); }));
        for (int s = 0; s <= 50; ++s) bad += check("counter <<", s, 0, set([=](uint64_t i) { return i << s; }));
        for (int s = 0; s <= 44; s += 4) bad += check("pointer <<", s, 0, set([=](uint64_t i) { return 0x7F1234560000ull + (i << s); }));
        for (int bits : {4, 6, 8, 10, 12})
            for (int lo = 0; lo <= 28; lo += 4)
                for (int hi = 32; hi <= 52; hi += 4)
                    bad += check("pair", lo, hi, set([=](uint64_t i) { return ((i & ((1u << bits) - 1)) << lo) + ((i >> bits) << hi); }));
        bad += check("double", 0, 0, set([](uint64_t i) {
            const double d = (double)i;
            uint64_t u;
            memcpy(&u, &d, 8);
            return u;
        }));
        bad += check("inverse double", 0, 0, set([](uint64_t i) {
            const double d = 1.0 / (double)i;
            uint64_t u;
            memcpy(&u, &d, 8);
            return u;
        }));
    }
    if (bad == 0) printf("ok\n");
    return bad != 0;
}
