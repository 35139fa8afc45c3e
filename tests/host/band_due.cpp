// The next band predicted by the update kernel (record_listed, then next_step) is the one that finish_listed predicts at once, and until
// then mode and band stay as they are.
#include <cstdio>
#include <cstring>
#include <random>
#include "kernels/rows.hpp"

using namespace liec;

int main() {
    std::mt19937 rng(11);
    auto upto = [&](uint32_t n) { return (uint32_t)(rng() % (n + 1ull)); };
    int failed = 0;
    for (int chain = 0; chain < 2000; ++chain) {
        RowDesc a;
        std::memset(&a, 0, sizeof a);
        a.mode = kCold;
        RowDesc b = a;
        uint32_t tau = upto(0x7f000000u);
        for (int step = 0; step < 40; ++step) {
            tau = upto(3) ? tau + upto(1u << 18) : upto(0x7f000000u);
            if (tau > 0x7f7fffffu) tau = 0x7f000000u;
            const bool cold = a.mode != kWarm || upto(5) == 0;
            const ListFound f{tau, 1 + upto(99), 1 + upto(99), upto(1000000)};
            const uint32_t mode = b.mode, lo = b.lo, hi = b.hi;
            if (upto(7) == 0) {                                 // a general search in between predicts at once
                const SlowFound g{tau, f.rank, f.ties, f.cut, 0u, upto(1) ? 1u : 100000u};
                const bool degenerate = upto(1) != 0;
                finish_general(a, g, degenerate, 0u, 0u, 0u);
                finish_general(b, g, degenerate, 0u, 0u, 0u);
            } else {
                finish_listed(a, f, 77, 1, cold, cold ? 1u : 0u, 0u, 0u);
                record_listed(b, f, 77, 1, cold, cold ? 1u : 0u);
                failed += b.due == 0 || a.due != 0;
            }
            failed += b.mode != mode || b.lo != lo || b.hi != hi;
            next_step(a);
            next_step(b);
            failed += std::memcmp(&a, &b, sizeof a) != 0;
        }
    }
    std::printf(failed ? "FAILED %d\n" : "band due ok\n", failed);
    return failed != 0;
}
