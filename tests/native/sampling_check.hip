// Host-side check of the sampling kernels' helpers.
#include <stdio.h>

#include "../../paper_1901_05423_amd/csrc/rtf_internal.h"

// A walk that never leaves the forest ends after nt + 1 nodes, also in the
// largest forest (the last steps of it, so that the check ends either way).
static int check_walk(int32_t nt) {
    uint32_t steps = (uint32_t)nt - 3;
    int read = 0;
    while (read < 16 && rtf::descent_goes_on(0, steps, nt)) {
        ++steps;
        ++read;
    }
    if (read != 4) printf("walk of %d nodes: %d steps past %u\n", nt, read, (uint32_t)nt - 3);
    return read != 4;
}

typedef unsigned __int128 u128;

static uint64_t state = 0x9E3779B97F4A7C15ull;
static uint64_t next64() {  // splitmix64
    uint64_t z = (state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// The interval [C, C + w) of a distribution with total W: its lower key, and
// its weight back from the two keys.
static int check_interval(uint64_t C, uint64_t w, uint64_t W) {
    const uint32_t s = (uint32_t)rtf::clz64(W);
    const uint64_t v = rtf::reciprocal_2by1(W << s);
    auto key = [&](uint64_t c) { return c < W ? rtf::fixed_point_key(c, W << s, v, s) : rtf::KEY_END; };
    const uint64_t lo = key(C), hi = key(C + w);
    if ((u128)lo != (((u128)C << 64) + (W - 1)) / W) {
        printf("key C=%llu W=%llu\n", (unsigned long long)C, (unsigned long long)W);
        return 1;
    }
    const double back = rtf::interval_weight(lo, hi, rtf::mulhi64(lo, W), W, s);
    if (back != (double)w) {
        printf("weight C=%llu w=%llu W=%llu: %.17g\n", (unsigned long long)C, (unsigned long long)w,
               (unsigned long long)W, back);
        return 1;
    }
    return 0;
}

static int check_intervals() {
    int bad = 0;
    // totals of every magnitude: powers of two, next to them, and any
    for (int bits = 1; bits <= 63 && !bad; ++bits)
        for (int it = 0; it < 4000 && !bad; ++it) {
            const uint64_t p = 1ull << (bits - 1);
            uint64_t W = it % 4 == 0 ? p : it % 4 == 1 ? 2 * p - 1 - next64() % 50 % p : p + next64() % p;
            const uint64_t top = W < 0xFFFFFFFFull ? W : 0xFFFFFFFFull;
            uint64_t w = it % 3 == 0 ? 1 + next64() % (top < 4 ? top : 4) : it % 3 == 1 ? top - next64() % (top < 50 ? top : 50)
                                                                                  : 1 + next64() % top;
            const uint64_t room = W - w;  // C in [0, room]; at room the interval is the last
            const uint64_t C = it % 5 == 0 ? 0 : it % 5 == 1 ? room : next64() % (room + 1);
            bad += check_interval(C, w, W);
        }
    return bad;
}

int main() {
    int bad = check_intervals();
    for (int32_t nt : {3, 4, 1000, 1 << 30, 2147483646, 2147483647}) bad += check_walk(nt);
    bad += rtf::descent_goes_on(-1, 0, 5) || rtf::descent_goes_on(5, 0, 5) || !rtf::descent_goes_on(4, 0, 5);
    printf(bad ? "FAIL\n" : "OK\n");
    return bad ? 1 : 0;
}
