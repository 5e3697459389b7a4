// Host check of how the restriction divides the test vectors, and the D_c build
// the sites of an aggregate, over workgroups (run by tests/test_restrict_split.py):
// for every count of test vectors or sites and launches of every size the parts
// are consecutive ranges that cover it, and each holds at least one element,
// since a workgroup loads the first of its part before its loop.
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
    for (int Va = 1; Va <= 4096; Va++)
        for (int Vc : {1, 16, 512, 513, 100000}) {
            const mgdd::DcSplit s = mgdd::dc_split(Va, Vc, 16);
            int covered = 0;
            for (int part = 0; part < s.parts; part++) {
                const int b = part * s.per, e = b + s.per < Va ? b + s.per : Va;
                if (b != covered || e <= b) {
                    printf("FAIL %d sites, %d aggregates, part %d of %d: [%d, %d)\n", Va, Vc, part, s.parts, b, e);
                    return 1;
                }
                covered = e;
            }
            if (covered != Va || s.parts > 4 || s.per % 16) { printf("FAIL %d sites covered %d\n", Va, covered); return 1; }
        }
    printf("SPLIT OK\n");
    return 0;
}
