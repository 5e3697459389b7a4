// Host check of how the restriction divides the test vectors over workgroups
// (run by tests/test_restrict_split.py): for every count of test vectors and
// launches of every size the parts are consecutive ranges that cover [0, N),
// and each holds at least one vector, since a workgroup loads the first column
// of its part before its loop.
#include <cstdio>

#include "../paper_1202_2462_amd/csrc/transfer.h"

int main() {
    for (int N = 1; N <= 32; N++)
        for (size_t wgs : {1, 2, 16, 255, 256, 257, 511, 512, 513, 1023, 1024, 100000}) {
            const mgdd::RestrictSplit s = mgdd::restrict_split(N, wgs);
            int covered = 0;
            for (int part = 0; part < s.parts; part++) {
                const int b = part * s.per, e = b + s.per < N ? b + s.per : N;
                if (b != covered || e <= b) {
                    printf("FAIL N %d, %zu workgroups, part %d of %d: [%d, %d)\n", N, wgs, part, s.parts, b, e);
                    return 1;
                }
                covered = e;
            }
            if (covered != N || s.parts > 4) { printf("FAIL N %d covered %d\n", N, covered); return 1; }
        }
    printf("SPLIT OK\n");
    return 0;
}
