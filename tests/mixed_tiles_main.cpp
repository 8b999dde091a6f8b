// Outputs shared by two kinds of tiles (mixed_first(), mixed_second() of csrc/kernels.h), walked on the host.  A line of the input is a division: M N rows split first second
// bm.  Every piece of 64 rows and 256 columns (64 divides the first outputs of all tiles) belongs to one workgroup, and no tile lies outside
// the output.  Prints "mixed-tiles ok".
#include <stdio.h>

#include <vector>

#include "../paper_2505_19115_amd/csrc/kernels.h"

using namespace nvfp4;

int main()
{
    long M, N;
    int bm, walked = 0;
    WideMix X;
    while (scanf("%ld %ld %d %d %u %u %d", &M, &N, &X.rows, &X.split, &X.first, &X.second, &bm) == 7) {
        const long ny = (M + 63) / 64, nx = (N + 255) / 256;
        std::vector<int> seen(ny * nx, 0);
        for (unsigned wg = 0; wg < X.first + X.second; ++wg) {
            int64_t m0 = -1, n0 = -1;
            if (wg < X.first) mixed_first(X, wg, M, N, m0, n0);
            else mixed_second(X, wg, M, N, bm, m0, n0);
            const int rows = wg < X.first ? 256 : bm;
            if (m0 < 0 || n0 < 0 || m0 >= M || n0 >= N || m0 % 64 || n0 % 256) {
                fprintf(stderr, "%ld x %ld: workgroup %u at %ld, %ld\n", M, N, wg, (long)m0, (long)n0);
                return 1;
            }
            for (long y = m0 / 64; y < (m0 + rows) / 64 && y < ny; ++y) ++seen[y * nx + n0 / 256];
        }
        for (long i = 0; i < ny * nx; ++i)
            if (seen[i] != 1) {
                fprintf(stderr, "%ld x %ld: outputs at %ld, %ld belong to %d workgroups\n", M, N, i / nx * 64, i % nx * 256, seen[i]);
                return 1;
            }
        ++walked;
    }
    printf("mixed-tiles ok %d\n", walked);
    return 0;
}
