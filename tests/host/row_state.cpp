// Every block of a row must derive the same work from the row's descriptor whenever it starts: before block 0 finishes the
// row's search or after.  Runs the descriptor's state changes (kernels/rows.hpp) over many states and compares.
#include <cstdio>
#include <cstring>
#include <random>
#include "kernels/rows.hpp"

using namespace liec;

static bool same_work(const RowDesc& a, const RowDesc& b, uint32_t cap, uint32_t k) {
    const RowWork p = row_work(a, cap, k), q = row_work(b, cap, k);
    return p.cold == q.cold && p.lo == q.lo && p.width == q.width && p.n == q.n && p.rank == q.rank && a.mode == b.mode &&
           wants_cold(a, cap, k) == wants_cold(b, cap, k);
}

int main() {
    std::mt19937 rng(7);
    auto upto = [&](uint32_t n) { return (uint32_t)(rng() % (n + 1ull)); };
    int failed = 0, warm = 0, cold = 0, moved = 0;
    for (int chain = 0; chain < 2000; ++chain) {
        RowDesc r;
        std::memset(&r, 0, sizeof r);
        const uint32_t cap = 4096 + 2 * upto(100000), k = 1 + upto(50000);
        const bool rk = chain % 8 == 0;
        const uint32_t fix_lo = 0x70000000u, fix_hi = rk ? 0x72000000u : 0u;
        r.mode = rk ? kWarm : kCold;
        r.lo = rk ? fix_lo : 0u;
        r.hi = fix_hi;
        uint32_t tau = upto(0x7f000000u);
        for (int step = 0; step < 30; ++step) {
            if (upto(9) == 0) r.mode = upto(1) ? kCold : kSlow;             // forced by a caller
            if (r.mode == kWarm) {                                          // the first pass
                r.n_sure = upto(3) ? upto(k - 1) : upto(2 * k);
                r.n_cand = upto(3) ? k - (r.n_sure < k ? r.n_sure : k) + upto(cap / 2) : upto(2 * cap);
            }
            tau = upto(3) ? tau + upto(1u << 18) : upto(0x7f000000u);
            if (tau > 0x7f7fffffu) tau = 0x7f000000u;
            const RowWork work = row_work(r, cap, k);
            RowDesc now = r;
            (work.cold ? cold : warm) += 1;
            const int how = (int)upto(2);                                   // any block may find a wait has run out
            if (!work.cold || how == 0)
                finish_listed(now, ListFound{tau, 1, 1, 5}, work.n, 1u, work.cold, 0u, fix_lo, fix_hi);
            else
                finish_general(now, SlowFound{tau, 1, 1, 5, 0, upto(2 * cap)}, how == 1, 0u, fix_lo, fix_hi);
            if (!same_work(r, now, cap, k)) {
                if (failed++ < 5) std::printf("chain %d step %d: a block that starts after the row is finished sees other work\n", chain, step);
            }
            const RowDesc done = now;
            const bool listed = !work.cold || how == 0;                     // what is reported of the search
            if (done.general != (listed ? 0u : 1u) || done.n_list != (listed ? work.n : 0u)) {
                if (failed++ < 5) std::printf("chain %d step %d: general %u, %u listed\n", chain, step, done.general, done.n_list);
            }
            next_step(now);
            if (now.lo != done.next_lo || now.hi != done.next_hi || now.mode != done.next_mode || now.tau != tau || now.n_cand || now.n_sure ||
                now.nonfinite_acc || now.hi - now.lo > (1u << (2 * kListBits))) {
                if (failed++ < 5) std::printf("chain %d step %d: the next step does not start on what this one left\n", chain, step);
            }
            moved += now.mode == kWarm && now.lo != r.lo;
            r = now;
        }
    }
    // a wait that runs out has cost no more than block 0 takes to do the work alone (us, as measured; see the bounds)
    for (uint32_t nwt = 17; nwt < (1u << 21); nwt += 1 + nwt / 7) {
        const uint32_t polls = search_wait(nwt);
        const double waited = 64 * 0.25 + (polls - 64) * 0.65, alone = 15 + 0.58 * nwt;
        if (waited > 1.2 * alone || (nwt < 65536 && waited < 0.25 * alone)) {
            if (failed++ < 5) std::printf("%u tiles: a wait of %.0f us against a search of %.0f\n", nwt, waited, alone);
        }
        const uint32_t n = nwt * 64, short_wait = list_wait(polls, n);     // the longest list of the row
        if (short_wait > polls || short_wait > 64 + n / 1024) ++failed;
    }
    if (!warm || !cold || !moved) ++failed;
    std::printf("%s: %d rows on a list, %d without, %d bands moved\n", failed ? "FAILED" : "row state ok", warm, cold, moved);
    return failed != 0;
}
