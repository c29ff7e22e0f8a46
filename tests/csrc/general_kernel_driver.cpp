// For every N: the length of the transforms and whether they run in rows at 256
// and at 257 (PRN, Doppler bin) items, one line each.
#include <algorithm>
#include <cstdio>

#include "../../paper_1309_0052_amd/csrc/general_rate.hpp"

int main()
{
    for (int N = 1; N <= gnss::kGenMaxN; ++N) {
        const int M = gnss::gen_transform_len(N);
        const int P = gnss::gen_two_segments(N, M) ? M / 2 : std::min(M, gnss::kGenLds);
        std::printf("%d %d %d\n", P, gnss::gen_in_rows(P, 1, 256) ? 1 : 0, gnss::gen_in_rows(P, 1, 257) ? 1 : 0);
    }
    return 0;
}
