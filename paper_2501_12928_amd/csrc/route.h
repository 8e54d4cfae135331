// Which theta of a call are spread over all workgroups (spread.hip) and which
// have a workgroup of their own (likelihood.hip). The results are the same bits
// either way, so the choice is by time alone; host code without HIP.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <functional>
#include <queue>
#include <vector>

namespace eor {

// Estimated times (us) on 256 CUs, N the 64-wide tile rows. Measured at n = 50 to
// 1010 (N = 1 .. 16) with 1 to 256 theta, where all are within 13% (spread, N = 1 and
// 2; else 9%), and at N = 24, 32, 47 and 64 with up to 64 theta (10%).
//
// One workgroup takes a theta in lone_us, more the more of the CUs have one
// (load, 0 to 1): N = 1 30 us, of 256 at a time 48; N = 4 168 and 230; N = 8 753 and
// 878; N = 16 4609 and 4950; N = 64 253 and 297 ms.
inline double lone_us(int64_t N, double load) {
    const double n = (double)N, n3 = n * n * n;
    return 10.0 + 17.0 * n + 2.2 * n * n + 0.92 * n3 + load * (16.0 * n + 0.149 * std::min(1.0, n / 32.0) * n3);
}

// Spread, a theta's diagonal tiles follow one another every 27 us, and its N (N +
// 1) / 2 tiles take the whole GPU 0.08 us each plus their products at 78 TFLOP/s.
inline double spread_chain_us(int64_t N) { return 27.0 * N; }
inline double spread_work_us(int64_t N) { return 0.04 * N * (N + 1) + 4.0 / 3.0 * 262144.0 * N * N * N / 78e6; }

// The chain and the work of all theta overlap the better the more tile rows there
// are: (chain^p + work^p)^(1/p), with p from 1.2 (nearly their sum: there is too
// little of either to fill the other's gaps) to large (the longer of the two).
// One tile row is one unit, which waits for nothing. Fitted, p is 1.1 to 1.3 at N
// = 2 to 4, 1.4 at 5, 1.85 at 8, 2.2 at 11 and 2.95 at 16.
inline double spread_us(double chain, double work, int64_t N) {
    const double p = N == 1 ? 4.0 : std::max(1.2, 0.8 + 0.125 * (double)N);
    const double a = std::max(chain, work), b = std::min(chain, work);
    return a * std::pow(1.0 + std::pow(b / a, p), 1.0 / p);
}

// Where the chain bounds, one workgroup per CU: a second one's matrix
// instructions hold up the single wave that factors a diagonal tile (19 us
// beside them, 14 alone). With much more work than chain, two, so that one
// computes while the other waits. The line, as work over chain, rises with the
// tile rows N, since longer sums leave less waiting to cover. Measured, one
// against two per CU: N = 4, 64 theta (work 0.6 times the chain) 164 / 162 us; N = 9,
// 32 (0.9) 364 / 378, 40 (1.1) 415 / 388; N = 16, 14 (1.0) 550 / 638, 24 (1.6) 859 /
// 744; N = 24, 10 (1.3) 932 / 1022, 12 (1.6) 1129 / 1092; N = 32, 8 (1.8) 1531 /
// 1563, 10 (2.2) 1955 / 1830; N = 47, 4 (1.8) 2.21 / 2.37 ms, 6 (2.6) 3.19 / 3.18; N =
// 64, two (1.6) 2.64 / 3.06, four (3.1) 4.94 / 5.12.
inline int spread_per_cu(double chain, double work, int64_t N) { return work < (0.5 + N / 22.0) * chain ? 1 : 2; }

// Of a call of B theta in rounds of `round` (the resident workgroups, or the
// slots if they are fewer), how many of the last ones to spread: none, what is left
// after whole rounds, or all. Spread, every round is a launch that ends before the
// next begins; with a workgroup each, one launch takes all rounds and a workgroup
// goes on to its next theta at once, so that a further round costs little more
// than one theta's time and a last partial round some us less than by itself. All
// rounds are spread where the rounds are small (slots for a few theta: 100 theta at
// n = 1000 in rounds of 10, 4.9 ms against 60), or at one tile row up to about 2000
// theta: 1000 theta at n = 64 121 us against 150, 2000 237 and 252, 5000 590 and
// 556.
inline int64_t spread_count(int64_t N, int64_t B, int64_t round, int num_cu) {
    auto spread = [&](int64_t n) { return n ? spread_us(spread_chain_us(N), n * spread_work_us(N), N) : 0.0; };
    auto lone = [&](int64_t n) { return n ? lone_us(N, std::min<double>(1.0, (double)n / num_cu)) : 0.0; };
    if (std::min(B, round) * (N * (N + 1) / 2) >= ((int64_t)1 << 31) - 4096) return 0;  // the units of a launch
    if (B <= round) return spread(B) < 0.97 * lone(B) ? B : 0;
    const int64_t rounds = B / round, rest = B % round;
    const double tail = rest ? lone(rest) - 4.0 * N : 0.0, part = rest ? spread(rest) + 3.0 : 0.0;
    const double whole = lone(round) + (rounds - 1) * (lone_us(N, 0.0) - 2.0) + std::min(tail, part);
    if (rounds * spread(round) + spread(rest) < whole) return B;
    return part < tail ? rest : 0;
}

// Theta of one size in a group: tile rows and how many.
struct Sizes {
    int64_t N, count;
};

// Estimated time (us) of a group with a workgroup per theta, the sizes largest
// first: the longest of num_cu workgroups that each take the next theta when they
// are done. Beyond 8192 theta the mean load, or the longest theta, which many small
// ones fill up evenly (the schedule itself took the host 1 ms for 100000 theta).
inline double lone_group_us(const std::vector<Sizes> &sizes, int num_cu) {
    int64_t n = 0;
    for (const Sizes &s : sizes) n += s.count;
    const double load = std::min(1.0, (double)n / num_cu);
    double sum = 0.0, longest = 0.0;
    for (const Sizes &s : sizes) {
        if (s.count < 1) continue;
        const double us = lone_us(s.N, load);
        sum += s.count * us;
        longest = std::max(longest, us);
    }
    if (n > 8192) return std::max(longest, sum / num_cu);
    std::priority_queue<double, std::vector<double>, std::greater<double>> busy;
    for (int i = 0; i < num_cu; ++i) busy.push(0.0);
    double end = 0.0;
    for (const Sizes &s : sizes) {
        const double us = lone_us(s.N, load);
        for (int64_t b = 0; b < s.count; ++b) {
            const double t = busy.top() + us;
            busy.pop();
            busy.push(t);
            end = std::max(end, t);
        }
    }
    return end;
}

}  // namespace eor
