// Walks every position of every code replica of the general-rate path and
// prints "N h j n" for the first one that leaves the code's N samples.
#include <algorithm>
#include <cstdio>

#include "../../paper_1309_0052_amd/csrc/general_rate.hpp"

int main()
{
    long long read = 0;
    for (int N = 1; N <= gnss::kGenMaxN; ++N) {
        const int M = gnss::gen_transform_len(N);
        const bool two = gnss::gen_two_segments(N, M);
        const int seg = two ? gnss::gen_segment(N) : N, P = two ? M / 2 : M;
        for (int h = 0; h < (two ? 2 : 1); ++h) {
            const int n0 = h * seg, n1 = std::min(N, n0 + seg);
            int len = 0;
            for (int j = 0; j < P; ++j) {
                const int n = gnss::gen_code_sample(j, n0, n1, N);
                if (n < 0) continue;
                if (n >= N || n != (n0 + j) % N || j != len) {
                    std::printf("%d %d %d %d\n", N, h, j, n);
                    return 1;
                }
                ++len;
            }
            // the whole replica (one period where N is a power of two: P = N)
            if (len != std::min(P, n1 - n0 + N) || (two && P < n1 - n0 + N)) {
                std::printf("%d %d length %d\n", N, h, len);
                return 1;
            }
            read += len;
        }
    }
    std::printf("%lld positions inside their code\n", read);
    return 0;
}
