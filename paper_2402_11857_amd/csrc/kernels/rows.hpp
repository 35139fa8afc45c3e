// What a row's threshold search keeps in its descriptor and how it changes from step to step: plain integer state, without
// device code, so that a host program can run it too.
#pragma once
#include <stddef.h>
#include <stdint.h>
#if defined(__HIPCC__)
#define LIEC_HD __host__ __device__ __forceinline__
#else
#define LIEC_HD inline
#endif

namespace liec {

constexpr int kListBits = 13;           // widest radix digit of the list select (two digits cover a band of 2^26 keys)
constexpr uint32_t kBandStart = 1u << 17;    // swing after a step without a prediction (an eighth of the band's half width then)
constexpr uint32_t kBandFloor = 1u << 15;    // least half width, in key units, of the predicted band (about 0.27 % in value)

// How a row's top-k threshold search starts its step.  Every kernel re-derives what the row needs from the mode, the band
// and the row's counters, so nothing that any of them looks at changes before the update kernel: whoever finishes the
// row's search (one block speaks for the row) leaves the next step's mode and band beside the present ones, or only what the update
// kernel predicts them from (due).  The one
// exception is the list select on long rows, one block a row, which sends a row to the general search by its mode.
enum SelMode : uint32_t {
    kWarm = 0,      // a band [lo, hi) predicted from the previous step is filtered
    kCold = 1,      // no prediction: the band is the first-radix-digit bin holding rank k
    kSlow = 4       // needs the general (multi pass) search over the row
};

// One per worker row, plus one (index N) for the server's vector v.
struct alignas(128) RowDesc {
    // first 128-byte line: what the kernels read, written once a step by whoever finishes the row's search
    double l1;             // scaled sign: sum |v_j| (fp64)
    float scale;           // scaled sign: fp32(l1 / d)
    uint32_t tau;          // top-k: key of the k-th kept entry
    uint32_t rank;         // top-k: how many entries with key == tau are kept
    uint32_t ties;         // top-k: how many entries have key == tau
    uint32_t cutoff;       // top-k: largest kept index among entries with key == tau
    uint32_t nonfinite;    // a NaN/Inf reached the L1 sum or a key (last step)
    uint32_t lo, hi;       // candidate band: keys in [lo, hi) are listed, keys >= hi are surely kept
    uint32_t mode;         // SelMode
    uint32_t n_list;       // candidates listed in the last step (0 after a general search), for whoever asks
    uint32_t dense;        // the row's candidate bitmap is not valid: test every column
    uint32_t form;         // top-k worker: form of that bitmap, 1 a bit per 4 columns, 2 per 64-byte line, 0 not valid or none yet
    uint32_t prev_tau;     // tau of the step before (valid when have_prev)
    uint32_t have_prev;
    uint32_t misses;       // steps in which the predicted band was not usable (since the context was created)
    uint32_t centre;       // where the last change of tau, continued, leads
    uint32_t swing;        // decaying maximum of the distances between tau and that
    uint32_t swing_still;  // and of those between tau and prev_tau
    uint32_t far;          // a slowly decaying maximum of the smaller of the two distances
    uint32_t was_cold;     // the last band came from the first-digit histogram, not from a prediction
    uint32_t next_lo, next_hi, next_mode;      // band and mode of the next step, which the update kernel puts into force
    uint32_t due;          // the band of the next step is still to be predicted (by the update kernel)
    uint32_t general;      // the last step took the general search: no list could hold the row's candidates, a caller asked for it, or a wait ran out
    // second line: what the blocks of the passes add to with atomics (kept off the line every block reads when
    // it starts).  Counters of the pass over the predicted band, one 64-bit word that a block of the filter adds
    // to with a single atomic.  Low half: candidates appended (may exceed the capacity: overflow); high half:
    // keys at or above the band.
    alignas(128) uint32_t n_cand;
    uint32_t n_sure;
    // the same for the pass over the first-digit band, which runs when there is no prediction or the predicted
    // band failed (its own set, so that every kernel can still tell from the first set that the row needed it)
    alignas(8) uint32_t n_cand2;
    uint32_t n_sure2;
    uint32_t n_short;      // entries of the first list digit's bin collected into the row's short list
    uint32_t nonfinite_acc;   // this step's Inf / NaN sightings (moved to `nonfinite` when the search finishes)
};
static_assert(sizeof(RowDesc) == 256, "two lines per row");

LIEC_HD uint32_t sure_count(const RowDesc& r) { return r.n_sure; }
LIEC_HD uint32_t sure_count2(const RowDesc& r) { return r.n_sure2; }
// The second line back to zero.
LIEC_HD void clear_counts(RowDesc& r) {
    r.n_cand = 0;
    r.n_cand2 = 0;
    r.n_short = 0;
    r.n_sure = r.n_sure2 = 0;
    r.nonfinite_acc = 0;
}

// After a filter pass: the band is usable when its list did not overflow and rank k falls inside it.
LIEC_HD bool band_ok(const RowDesc& r, uint32_t cap, uint32_t k) {
    const uint32_t n_sure = sure_count(r);
    return r.n_cand <= cap && n_sure < k && (uint64_t)k <= (uint64_t)n_sure + r.n_cand &&
           r.hi - r.lo <= (1u << (2 * kListBits));       // the list select's two digits must span the band
}
// Rows that need the first-digit histogram: no prediction, or the predicted band failed.  Stable from the
// end of the pass over the predicted band until the row's search is finished.
LIEC_HD bool wants_cold(const RowDesc& r, uint32_t cap, uint32_t k) {
    return r.mode == kCold || (r.mode == kWarm && !band_ok(r, cap, k));
}

// Bounds, in polls, of the waits of blocks that share a row for one another.  Blocks of two launches on two streams can each
// be resident in part and wait for the rest, so a wait lasts no longer than block 0 needs to do the work alone: 0.58 us
// per wave tile of 1024 columns for a search of the row, about 15 us for a list and a third of a microsecond per 1024 entries
// of a long one; a poll takes 0.25 us, from the 65th on 0.65.  (A meeting takes 3 us.)
LIEC_HD uint32_t search_wait(uint32_t nwt) { return nwt < 64u ? 64u : nwt < 65536u ? nwt : 65536u; }
LIEC_HD uint32_t list_wait(uint32_t bound, uint32_t n) {
    const uint32_t polls = 64u + n / 1024u;
    return polls < bound ? polls : bound;
}

// What a row needs of the kernel that finishes searches (k_select).  Every block of the row derives it for itself, whenever it
// starts: block 0 may have finished the row by then.
struct RowWork {
    bool cold;                 // no usable list: search the row
    uint32_t lo, width;        // otherwise the list of the predicted band,
    uint32_t n, rank;          // its entries and the rank searched among them
};
LIEC_HD RowWork row_work(const RowDesc& r, uint32_t cap, uint32_t k) {
    return RowWork{r.mode != kWarm || !band_ok(r, cap, k), r.lo, r.hi - r.lo, r.n_cand, k - sure_count(r)};
}

// Band for the next step.  Two predictions of tau compete: the last one, and the last one extrapolated by its last change.
// Each has a `swing` of its own, a maximum of its misses that decays by an eighth per step -- by a half while the last
// miss was under 1/64 of it, so that very quiet rows narrow quickly -- and the one with the smaller swing is the band's
// centre: the trend while thresholds drift, the last value where they go up and down from step to step, which a trend would
// follow the wrong way (and with three times the variance of the noise).  The band's half width is six times that swing, for a trend never
// less than twice the last change of tau, between kBandFloor and 2^25 key units.  After a step without a usable prediction
// the band starts 2^20 keys wide on either side.  `far` remembers, four times as long, the largest miss of the better of
// the two, and the half width is never less than twice that: thresholds that stand still for ten steps and then jump
// (gradients of bf16 mantissas, by 2^16 keys) stay inside.  It is cut off at kBandStart, so that the large misses of a row's
// first steps do not stay with it.
// A band that misses costs two more passes over the row; one that is wider than needed only lengthens the
// candidate list.  Against the trend alone, eight times its swing, us per step of two batches in turn: 8 x 1M columns, 1 %, 53.8 -> 52.6,
// 5 x 3M of bf16 mantissas 105 -> 98.5.  Means over 56 steps whose gradient scale changes, steps without a usable prediction among
// them (row-steps that missed in brackets): a random walk of 5 % a step 83 -> 79 (63, 1) and 130 -> 120 (42, 2), 30 % of noise
// 81 -> 79 (148, 73) and 134 -> 125 (101, 46), 30 % up and down in turn 94 -> 89 (289, 257) and 183 -> 151 (200, 161), growth by 10 % a
// step 83 -> 80 and 121 -> 119.
constexpr int kBandSwings = 6;
LIEC_HD int64_t distance(int64_t a, int64_t b) { return a < b ? b - a : a - b; }
LIEC_HD int64_t next_swing(int64_t last, int64_t miss) {
    int64_t swing = 64 * miss < last ? last / 2 : last - last / 8;
    if (swing < miss) swing = miss;
    return swing > (int64_t)1 << 22 ? (int64_t)1 << 22 : swing;
}
LIEC_HD void predict_band(RowDesc& r, uint32_t fix_lo, uint32_t fix_hi) {
    if (fix_hi) {                                   // random-k: the band does not depend on the data
        r.next_lo = fix_lo;
        r.next_hi = fix_hi;
        r.prev_tau = r.tau;
        r.have_prev = 1;
        r.was_cold = 0;
        return;
    }
    const int64_t tau = (int64_t)r.tau;
    int64_t delta = r.have_prev ? tau - (int64_t)r.prev_tau : 0;
    // a change of more than 2^22 keys (a factor of 1.4 in value) that the last prediction missed is a jump, not a
    // trend: extrapolating it would put the next band as far off again
    if (r.was_cold && (delta > ((int64_t)1 << 22) || delta < -((int64_t)1 << 22))) delta = 0;
    int64_t swing = kBandStart, swing_still = kBandStart, far = 0;
    int64_t margin = (int64_t)8 * kBandStart;
    bool still = false;
    if (r.have_prev) {
        const int64_t miss = distance(tau, (int64_t)r.centre), miss_still = distance(tau, (int64_t)r.prev_tau);
        const int64_t least = miss < miss_still ? miss : miss_still;
        far = (int64_t)r.far - (int64_t)r.far / 32;
        if (far < least) far = least < (int64_t)kBandStart ? least : (int64_t)kBandStart;
        if (!r.was_cold) {
            swing = next_swing((int64_t)r.swing, miss);
            swing_still = next_swing((int64_t)r.swing_still, miss_still);
            still = swing_still < swing;
            margin = kBandSwings * (still ? swing_still : swing);
        }
    }
    int64_t trend = tau + delta;
    if (trend < 0) trend = 0;
    if (trend > 0x7fffffffll) trend = 0x7fffffffll;
    if (!still && margin < 2 * distance(delta, 0)) margin = 2 * distance(delta, 0);
    if (margin < 2 * far) margin = 2 * far;
    if (margin < (int64_t)kBandFloor) margin = kBandFloor;
    if (margin > (int64_t)1 << 25) margin = (int64_t)1 << 25;   // two list digits cover a band of 2^26 keys
    const int64_t centre = still ? tau : trend;
    const int64_t lo = centre - margin, hi = centre + margin;
    r.next_lo = lo < 0 ? 0u : (uint32_t)lo;
    r.next_hi = hi > 0x80000000ll ? 0x80000000u : (uint32_t)hi;
    r.centre = (uint32_t)trend;
    r.swing = (uint32_t)swing;
    r.swing_still = (uint32_t)swing_still;
    r.far = (uint32_t)far;
    r.prev_tau = r.tau;
    r.have_prev = 1;
    r.was_cold = 0;
}

// The update kernel, for every row, once nobody looks at the mode, the band or the counters of this step any more.
LIEC_HD void next_step(RowDesc& r) {
    if (r.due) {
        predict_band(r, 0u, 0u);
        r.next_mode = kWarm;
        r.due = 0;
    }
    r.lo = r.next_lo;
    r.hi = r.next_hi;
    r.mode = r.next_mode;
    clear_counts(r);
}

// What a search over a list found.
struct ListFound {
    uint32_t tau, rank, ties, cut;
};
// And what it leaves in the row's descriptor (thread 0): n_all candidates were listed.  The band of the next step comes with it,
// or (due) from the update kernel, where nothing waits for it: 0.6 us of one thread's integer arithmetic at the end of k_select (us per
// step, top-k both sides: 4 x 65536 columns 25.3 -> 24.3, 8 x 262144 30.5 -> 29.4, 8 x 1M 50.6 -> 49.8).
LIEC_HD void record_listed(RowDesc& r, const ListFound& f, uint32_t n_all, uint32_t form, bool cold, uint32_t missed) {
    r.n_list = n_all;
    r.tau = f.tau;
    r.rank = f.rank;
    r.ties = f.ties;
    r.cutoff = f.cut;
    r.dense = r.general = 0;
    r.form = form;
    r.nonfinite = r.nonfinite_acc;
    r.was_cold = cold ? 1u : 0u;
    r.misses += missed;
    r.due = 1;
}
LIEC_HD void finish_listed(RowDesc& r, const ListFound& f, uint32_t n_all, uint32_t form, bool cold, uint32_t missed,
                           uint32_t fix_lo, uint32_t fix_hi) {
    record_listed(r, f, n_all, form, cold, missed);
    r.due = 0;
    predict_band(r, fix_lo, fix_hi);
    r.next_mode = kWarm;
}

// What a general search found.
struct SlowFound {
    uint32_t tau, rank, ties, cut, bad;
    uint32_t first;                            // entries that share tau's first digit
};
// A candidate bitmap is worth having while most of the row is not in it (a constant row is read faster without one: 40M
// columns packed in 63 us against 90).
LIEC_HD bool bitmap_pays(const SlowFound& f, uint32_t k, uint32_t d) { return (uint64_t)(k - f.rank + f.ties) * 8 <= d; }
// And what it leaves in the row's descriptor (thread 0).  degenerate: no candidate list could hold the row, so there is
// no use in a prediction; form: of the row's candidate bitmap, 0 none.
LIEC_HD void finish_general(RowDesc& r, const SlowFound& f, bool degenerate, uint32_t form, uint32_t fix_lo,
                                               uint32_t fix_hi) {
    r.tau = f.tau;
    r.rank = f.rank;
    r.ties = f.ties;
    r.cutoff = f.cut;
    r.dense = form ? 0u : 1u;
    r.form = form;
    r.general = 1;
    r.nonfinite = r.nonfinite_acc;
    r.n_list = 0;
    if (degenerate && !fix_hi) {
        r.have_prev = 0;
        r.was_cold = 0;
        r.next_mode = kCold;
        return;
    }
    if (degenerate) r.have_prev = 0;           // the band of a random-k draw is known without a prediction
    r.was_cold = 1;
    predict_band(r, fix_lo, fix_hi);
    r.next_mode = kWarm;
}

}  // namespace liec
