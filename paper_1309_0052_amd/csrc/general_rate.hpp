// general_rate.hpp -- sizes and index rules of the general-rate path, in plain
// C++: constexpr, so that the launches and the kernels share them and a host
// program can check them.
#pragma once

namespace gnss {

// General rates: N <= kGenMaxN samples per ms, transforms of length
// M = 2^ceil(log2(2N)) <= 2 kGenLds (M = N when N is a power of two) done as
// one (M <= kGenLds) or two (M = 2 kGenLds, even and odd bins) transforms of
// at most kGenLds points in a workgroup's LDS.
constexpr int kGenMaxN = 16384;
constexpr int kGenLds = 16384;
constexpr int kGenTwLen = 2 * kGenLds;  // twiddle table W_32768^j, j < 32768
constexpr int kGenThreads = 1024;
constexpr int gen_transform_len(int N)
{
    // N a power of two (>= 64): the length-N circular correlation is the
    // N-point one, no padding needed
    if (N >= 64 && (N & (N - 1)) == 0) return N;
    int M = 64;
    while (M < 2 * N) M *= 2;
    return M;
}

// Two segments of the block on transforms of half the length (see the
// general-rate kernels): each segment has at most gen_segment(N) samples, and
// its correlation at N lags fits M / 2 points.  The shortest transform has 64.
constexpr int gen_segment(int N) { return (N + 1) / 2; }
constexpr bool gen_two_segments(int N, int M) { return M > N && M >= 128 && N + gen_segment(N) <= M / 2; }

// The replica of samples n0 .. n1 - 1 of a block has n1 - n0 + N values (the
// second segment of an odd N is one sample shorter than the first): the sample
// number, below N, at position j of it, or -1 past its end.
constexpr int gen_code_sample(int j, int n0, int n1, int N)
{
    if (j >= n1 - n0 + N) return -1;
    const int n = n0 + j;  // below n1 + N <= 2N
    return n >= N ? n - N : n;
}

// PRNs per correlation workgroup at transform length P, in rows
constexpr int gen_group(int P) { return P == 4096 ? 2 : 1; }
// Whether a request's transforms of P points run as rows (see the
// general-rate kernels).  At 4096 points a row workgroup does two of a CU's
// six transforms with four waves, a one-piece one its CU's only transform
// with sixteen: up to one item per CU the latter ends sooner (N = 2000, 10
// blocks, 168 items: 88 us against 121), above that the former (1952 items:
// 233 us against 406; 3872 items of 25 blocks: 0.79 ms against 1.81).  The
// rule takes only the request's own sizes, so its results do not depend on
// its batch.
constexpr bool gen_in_rows(int P, int n_prn, int n_dopp)
{
    return P > 4096 || (P == 4096 && (long long)n_prn * n_dopp > 256);
}

}  // namespace gnss
