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

int main() {
    int bad = 0;
    for (int32_t nt : {3, 4, 1000, 1 << 30, 2147483646, 2147483647}) bad += check_walk(nt);
    bad += rtf::descent_goes_on(-1, 0, 5) || rtf::descent_goes_on(5, 0, 5) || !rtf::descent_goes_on(4, 0, 5);
    printf(bad ? "FAIL\n" : "OK\n");
    return bad ? 1 : 0;
}
