// Threshold search behind top-k (Definition 2) and random-k (Definition 3).
#pragma once
#include "common.hpp"
#include <type_traits>

namespace liec {

// ---------------------------------------------------------------------------------------------
// Top-k (Definition 2).  The k-th largest magnitude key tau of a row and the index cut-off
// among its ties are found without sorting, on long rows by five kernels the host enqueues every step (on short rows, and
// for random-k, one kernel, k_select, does what 2 to 5 do):
//   1. k_filter (pass over the predicted band) streams the row once against a band [lo, hi) of keys
//      expected to hold tau, predicted from the previous steps' tau (rows in kWarm mode): keys >= hi are
//      only counted, keys inside the band are appended to a candidate list (key, index), and a group
//      bitmap is written for the aggregation kernel, in one of two forms the host picks from the row
//      length.  Fine: 4 words of 64 bits per wave tile, bit l of word u set when any of the 4 columns
//      1024t + 256u + 4l .. + 3 has key >= lo.  Coarse: one word per wave tile, bit 4m + u set when any
//      of the 16 columns 1024t + 256u + 16m .. + 15 (one 64-byte line, the unit a gather fetches anyway)
//      has one -- 8 bytes written per 4 KiB read (writes are what a read stream pays most for); measured
//      faster for rows of 48M columns and more, slower for 25M.  The band is usable when the list did
//      not overflow and rank k falls inside it (band_ok).
//   2. k_hist0, for rows without a prediction (kCold) or whose predicted band was not usable: the
//      histogram of the first radix digit (12 bits) of the whole row.  For rows on their predicted band
//      with a long list it counts the first digit of the listed keys instead (list_first_digit).
//   3. k_filter (pass over the first-digit band), for the rows of the first kind: every block picks the
//      bin holding rank k from that histogram, and the row is filtered again with that bin as its band,
//      counting into a second set of counters.  For the rows of the second kind every block picks the
//      first list digit's bin and the bin's entries are collected into a short list (list_collect).
//   4. k_list_select, one block per row: radix digits over the listed keys, taken relative to the band's
//      lower end (over the short list when there is one) until few entries are left to compare, or, among
//      more entries of one key, a radix select over their indices; writes (tau, cut-off), predicts
//      the next band.  Rows whose band the list cannot hold (constant or near-constant rows) are put
//      into kSlow mode.
//   5. k_slow_select takes the kSlow rows.
// All decisions are taken on the device per row, each kernel re-deriving from the row's mode and
// counters whether it has work; in the steady state kernels 2 and 3 only touch the lists and 5 returns at once.  A row's mode
// and its result are written only by k_list_select, k_slow_select and k_select, its counters cleared by the update.
// `row0` is added to blockIdx.y to address per-row state (the server's vector uses row N).
// ---------------------------------------------------------------------------------------------
// Coarse group bitmap: bit 4m of the result is set when some lane of 4m .. 4m + 3 has its bit set in the
// ballot (those four lanes own one 64-byte line of the row).  Chunk u of a wave tile shifts its result
// left by u, so bit 4m + u of the tile's word stands for line m of chunk u.
__device__ __forceinline__ uint64_t any_of_four_lanes(uint64_t b) {
    b |= b >> 1;
    b |= b >> 2;
    return b & 0x1111111111111111ull;
}

// One chunk (256 columns, 4 per lane) of the filter: updates the per-lane count of keys >= hi and the
// running maximum key, returns the ballot of "any of my 4 columns has key >= lo" and, per component q,
// the ballot bc[q] of the candidates lo <= key < hi.  The comparisons stay wave ballots (scalar
// registers) and are combined there, which leaves the vector unit two compares, one add and half a
// maximum per key.  FULL: every column of the chunk is below d.  BITS: also hi4, bit q set when my
// column q has key >= hi.
template <bool FULL, bool BITS>
__device__ __forceinline__ uint64_t filter_chunk(const uint32_t (&keys)[4], uint32_t j, uint32_t d, uint32_t lo, uint32_t hi,
                                                 uint64_t (&bc)[4], uint32_t& n_hi, uint32_t& kmax, uint32_t& hi4) {
    uint64_t any_lo = 0;
    hi4 = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t key = keys[q];
        const bool valid = FULL || j + q < d;
        const bool ge_lo = valid && key >= lo, ge_hi = valid && key >= hi;
        kmax = max(kmax, valid ? key : 0u);
        n_hi += ge_hi ? 1u : 0u;
        if (BITS) hi4 |= (ge_hi ? 1u : 0u) << q;
        const uint64_t b_lo = __ballot(ge_lo);
        bc[q] = b_lo & ~__ballot(ge_hi);
        any_lo |= b_lo;
    }
    return any_lo;
}

// List select: the keys of a band are taken relative to its lower end and need b <= 26 bits.  The first
// digit is their top kFirstBits bits when many blocks build its histogram in global memory (256 bins: the
// blocks' LDS histograms then merge with few global atomics, which are slow across the chip's dies); one block
// that builds it in LDS, and the digits after it, take kHeldBits (a list held in LDS: another pass is
// cheap) or kListBits bits each.
constexpr int kFirstBits = 8;
__device__ __forceinline__ int band_bits(uint32_t width) {            // width: 1 .. 2^26
    return width > 1 ? 32 - __clz((int)(width - 1)) : 1;
}
__device__ __forceinline__ int first_shift(uint32_t width, int first_bits) {   // bits below the first digit
    const int b = band_bits(width);
    return b > first_bits ? b - first_bits : 0;
}

// Blocks that share a pass over a list of n entries: one per 2048 entries.
__device__ __forceinline__ uint32_t list_blocks_for(uint32_t n, uint32_t grid) {
    const uint32_t want = (n + 2047u) / 2048u;
    return want < 1u ? 1u : (want > grid ? grid : want);
}

// The two passes over a row's candidate list that are shared by many blocks.  They ride in the two kernels
// that otherwise only work for rows without a usable prediction (k_hist0 and the second k_filter pass), for the
// rows whose predicted band holds rank k:
//   list_first_digit  adds the first digit of every listed key to the row's global histogram;
//   list_collect      picks the bin holding rank k from that histogram (every block redoes the pick) and, when
//                     that bin has at most kShortCap entries, appends them to the row's short list.
// k_list_select then finishes on the short list alone.  Lists of at most kDirectList entries skip both: one block
// walks those as fast as the shared passes' fixed costs.  Every thread of the block calls them.
__device__ __forceinline__ void list_first_digit(const RowDesc* __restrict__ desc, uint32_t row,
                                                 const uint2* __restrict__ in, uint32_t* __restrict__ hrow,
                                                 uint32_t* lds_h /* 256 words */) {
    const uint32_t n = desc[row].n_cand, nb = list_blocks_for(n, gridDim.x);
    if (n <= (uint32_t)kDirectList || blockIdx.x >= nb) return;
    const uint32_t lo = desc[row].lo, lane = threadIdx.x & 63;
    const int shift = first_shift(desc[row].hi - lo, kFirstBits);
    for (uint32_t b = threadIdx.x; b < 256; b += blockDim.x) lds_h[b] = 0;
    __syncthreads();
    for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += nb * blockDim.x) {    // uniform for the block
        const uint32_t e = base + threadIdx.x;
        const bool valid = e < n;
        const uint32_t key = valid ? in[e].x : lo;
        wave_count(lds_h, valid, (key - lo) >> shift, lane);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < 256; b += blockDim.x) {
        const uint32_t c = lds_h[b];
        if (c) atomicAdd(&hrow[b], c);
    }
}

__device__ __forceinline__ void list_collect(RowDesc* __restrict__ desc, uint32_t row, const uint2* __restrict__ in,
                                             const uint32_t* __restrict__ hrow, uint2* __restrict__ out, uint32_t k,
                                             uint32_t* part, uint32_t* res) {
    const uint32_t n = desc[row].n_cand, nb = list_blocks_for(n, gridDim.x);
    if (n <= (uint32_t)kDirectList || blockIdx.x >= nb) return;
    const uint32_t lo = desc[row].lo, lane = threadIdx.x & 63;
    const int shift = first_shift(desc[row].hi - lo, kFirstBits);
    const Pick p = block_pick(hrow, 1 << kFirstBits, k - sure_count(desc[row]), part, res);
    if (p.count > (uint32_t)kShortCap) return;                  // too many for the short list: k_list_select walks the list
    for (uint32_t base = blockIdx.x * blockDim.x; base < n; base += nb * blockDim.x) {    // uniform for the block
        const uint32_t e = base + threadIdx.x;
        const uint2 kv = e < n ? in[e] : make_uint2(0u, 0u);
        const bool hit = e < n && ((kv.x - lo) >> shift) == p.bin;
        const uint64_t m = __ballot(hit);
        if (m) {                                                // wave-uniform
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&desc[row].n_short, (uint32_t)__popcll(m));
            at = __builtin_amdgcn_readfirstlane(at);
            if (hit) out[at + lanes_below(m)] = kv;             // the bin's count bounds the total: at most kShortCap
        }
    }
}

// The band a row is filtered against and the counters the pass adds to.  cold_pass false: rows in kWarm
// mode, their predicted band, the first counter set.  cold_pass true: rows for which wants_cold holds,
// the first-digit bin that holds rank k (every block redoes that pick from the row's finished histogram;
// needs 256 threads and 259 words of LDS), the second counter set.  False when the block has no work.
struct FilterBand {
    uint32_t lo, hi;
    uint2* out;                                  // the row's list and its capacity
    uint32_t cap;
    unsigned long long* counts;                  // the pass's counter word: candidates (low half), keys above the band (high half)
};
__device__ __forceinline__ bool filter_band(RowDesc* __restrict__ desc, uint32_t row, bool cold_pass,
                                            const uint32_t* __restrict__ ghist, uint2* __restrict__ list, uint32_t cap,
                                            uint32_t k, uint32_t* part, uint32_t* res, FilterBand& fb) {
    fb.out = list + (size_t)row * cap;
    fb.cap = cap;
    if (!cold_pass) {
        if (desc[row].mode != kWarm) return false;
        fb.lo = desc[row].lo;
        fb.hi = desc[row].hi;
        fb.counts = reinterpret_cast<unsigned long long*>(&desc[row].n_cand);
        return true;
    }
    if (!wants_cold(desc[row], cap, k)) return false;
    const Pick p = block_pick(ghist + (size_t)row * kHistBins, kHistBins, k, part, res);
    if (p.count > cap) return false;             // the list cannot hold the bin: the row takes the general search
    fb.lo = p.bin << 19;
    fb.hi = (p.bin + 1) << 19;                   // 0x80000000 for the top bin: no key reaches it
    fb.counts = reinterpret_cast<unsigned long long*>(&desc[row].n_cand2);
    return true;
}

// Where the results of a filter block go.  Atomics on a row's counters are what the pass pays most for besides
// its stores.  Measured alone on 16 rows of 138M columns: a pass that writes nothing runs at the read ceiling
// (1.29 ms); one atomic per block, and nothing else written, takes it to 1.44 ms whether 2 000 or 15 000 blocks
// do it; an atomic per wave for the list and one per block for the count gave 1.5-1.6 ms, and 3.7 ms with 2 800
// blocks a row while the counters shared a line with the fields every block reads when it starts.  So the
// block's waves append their candidates to one stage in LDS (an LDS counter hands out the positions), and when
// the block is done a single 64-bit atomic adds its keys above the band to the high half of the row's counter
// word and reserves, in the low half, the list slots of what was staged.  Once that stage (kStage entries) is
// full -- wide bands, candidates crowded into one stretch of the row -- every wave goes on into a small stage
// of its own (kWaveStage entries) that it empties into list slots reserved with an atomic of its own.
struct StagePos {
    uint32_t pos;                                // block position of the wave's first entry
    uint32_t first_spill;                        // first of its positions beyond the block's stage
    uint32_t wbase;                              // slot of that entry in the wave's own stage
    bool drop;                                   // the list is full: nothing is kept any more
};
// Words that blocks of one launch hand to one another (they may run on dies with an L2 of their own): stored past the L2,
// loaded past it.  Complete once the wave that stored them has waited for its stores.
template <typename T>
__device__ __forceinline__ void st_shared(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T ld_shared(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// An entry of a list; SHARED: for another block of this launch.
template <bool SHARED>
__device__ __forceinline__ void put_entry(uint2* at, uint2 e) {
    if (SHARED) st_shared(reinterpret_cast<unsigned long long*>(at), (unsigned long long)e.y << 32 | e.x);
    else *at = e;
}
// Empties the wave's own stage into the list.  staged[1] is set once a reservation of this block has gone past
// the list's capacity: the row's count then stays above the capacity, which is all that anyone reads from an
// overflowed list, and the block stops listing and counting candidates.
template <bool SHARED>
__device__ __forceinline__ void flush_wave_stage(const FilterBand& fb, const uint2* wst, uint32_t cnt, uint32_t* staged,
                                                 uint32_t lane) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    uint32_t base = 0;
    if (lane == 0) {
        base = (uint32_t)atomicAdd(fb.counts, (unsigned long long)cnt);
        if ((uint64_t)base + cnt > fb.cap) staged[1] = 1;
    }
    base = __builtin_amdgcn_readfirstlane(base);
    for (uint32_t s = lane; s < cnt; s += 64)
        if (base + s < fb.cap) put_entry<SHARED>(&fb.out[base + s], wst[s]);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// The wave has m <= kWaveStage entries to append (wave-uniform, every lane calls).  staged[0]: the block's LDS
// counter of stage positions handed out; wst / wcnt: the wave's own stage and how many entries it holds.
template <bool SHARED = false>
__device__ __forceinline__ StagePos reserve_stage(const FilterBand& fb, uint32_t m, uint32_t* staged, const uint2* wst,
                                                  uint32_t& wcnt, uint32_t lane) {
    StagePos sp;
    sp.pos = sp.first_spill = sp.wbase = 0;
    sp.drop = *reinterpret_cast<volatile uint32_t*>(&staged[1]) != 0;   // uniform
    if (sp.drop) return sp;
    uint32_t pos = 0;
    if (lane == 0) pos = atomicAdd(&staged[0], m);              // LDS
    sp.pos = __builtin_amdgcn_readfirstlane(pos);
    sp.first_spill = max(sp.pos, (uint32_t)kStage);
    if (sp.pos + m > (uint32_t)kStage) {                        // uniform
        const uint32_t nsp = sp.pos + m - sp.first_spill;
        if (wcnt + nsp > (uint32_t)kWaveStage) {
            flush_wave_stage<SHARED>(fb, wst, wcnt, staged, lane);
            wcnt = 0;
        }
        sp.wbase = wcnt;
        wcnt += nsp;
    }
    return sp;
}
// Entry number `ord` of those m (any subset of lanes).
__device__ __forceinline__ void put_candidate(uint2* stage, uint2* wst, const StagePos& sp, uint32_t ord, uint2 entry) {
    if (sp.drop) return;
    const uint32_t p = sp.pos + ord;
    if (p < (uint32_t)kStage) stage[p] = entry;
    else wst[sp.wbase + (p - sp.first_spill)] = entry;
}

// Appends a chunk's candidates: those of component q are the lanes of bc[q], at column j + q.
template <bool SHARED = false>
__device__ __forceinline__ void stage_candidates(const FilterBand& fb, const uint32_t (&keys)[4], uint32_t j,
                                                 const uint64_t (&bc)[4], uint2* stage, uint2* wst, uint32_t& wcnt,
                                                 uint32_t* staged, uint32_t lane) {
    if ((bc[0] | bc[1] | bc[2] | bc[3]) == 0) return;           // wave-uniform
    const uint32_t m = __popcll(bc[0]) + __popcll(bc[1]) + __popcll(bc[2]) + __popcll(bc[3]);
    const StagePos sp = reserve_stage<SHARED>(fb, m, staged, wst, wcnt, lane);
    uint32_t off = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if ((bc[q] >> lane) & 1) put_candidate(stage, wst, sp, off + lanes_below(bc[q]), make_uint2(keys[q], j + q));
        off += __popcll(bc[q]);
    }
}

// End of a filter block of WAVES waves.  n_hi: keys above the band, per lane; wst / wcnt: the wave's own stage.  Every
// thread of the block calls it.
template <int WAVES = kBlock / 64, bool SHARED = false>
__device__ __forceinline__ void finish_filter_block(const FilterBand& fb, const uint2* stage, const uint2* wst, uint32_t wcnt,
                                                    uint32_t n_hi, uint32_t* staged, uint32_t* wsure /* WAVES + 1 words */) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    n_hi = wave_sum(n_hi);
    if (lane == 0) wsure[wave] = n_hi;
    if (wcnt) flush_wave_stage<SHARED>(fb, wst, wcnt, staged, lane);    // wave-uniform
    __syncthreads();
    const uint32_t n_staged = min(staged[0], (uint32_t)kStage);
    if (threadIdx.x == 0) {
        uint32_t sure = 0, base = 0;
        for (int w = 0; w < WAVES; ++w) sure += wsure[w];
        if (sure | n_staged) base = (uint32_t)atomicAdd(fb.counts, ((unsigned long long)sure << 32) | n_staged);
        wsure[WAVES] = base;
    }
    __syncthreads();
    const uint32_t base = wsure[WAVES];
    for (uint32_t s = threadIdx.x; s < n_staged; s += WAVES * 64)
        if (base + s < fb.cap) put_entry<SHARED>(&fb.out[base + s], stage[s]);
}

// RK: the keys are the priorities of a random-k draw (nothing is read from src), and instead of the
// group bitmap the kernel writes, per column, whether its key is at or above the band (lane-major
// half-words like the sign bits, at row `row` of kbits); k_rk_mark later adds the kept candidates.
template <bool VEC, bool RK>
__global__ __launch_bounds__(kBlock) void k_filter(const float* __restrict__ src, size_t row_stride, uint32_t d,
                                                    uint32_t nwt, uint32_t row0, RowDesc* __restrict__ desc,
                                                    bool cold_pass, const uint32_t* __restrict__ ghist, uint32_t k,
                                                    uint64_t* __restrict__ gbits,
                                                    uint16_t* __restrict__ kbits, uint2* __restrict__ list, uint32_t cap,
                                                    uint2* __restrict__ shortl, RkDraw rk, bool coarse, uint32_t run) {
    __shared__ uint2 stage[kStage], wstage[4][kWaveStage];
    __shared__ uint32_t wsure[5], staged[2];
    __shared__ uint32_t part[256], res[3];
    const uint32_t row = row0 + blockIdx.y;
    if (!RK && cold_pass && desc[row].mode == kWarm && !wants_cold(desc[row], cap, k)) {   // uniform for the block
        list_collect(desc, row, list + (size_t)row * cap, ghist + (size_t)row * kHistBins,
                     shortl + (size_t)row * kShortCap, k, part, res);
        return;
    }
    FilterBand fb;
    if (!filter_band(desc, row, !RK && cold_pass, ghist, list, cap, k, part, res, fb)) return;   // uniform for the block
    if (threadIdx.x < 2) staged[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lo = fb.lo, hi = fb.hi;
    const float* __restrict__ g = src + (size_t)blockIdx.y * row_stride;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint32_t k0 = 0, k1 = 0;
    if (RK) {
        const uint64_t stream = rk_stream(rk.state->seed, rk.state->draw, row);
        k0 = (uint32_t)stream;
        k1 = (uint32_t)(stream >> 32);
    }
    uint32_t n_hi = 0, kmax = 0;                                // per lane: keys >= hi seen, largest key seen
    uint2* wst = wstage[wave];                                  // the wave's own stage and its fill (wave-uniform)
    uint32_t wcnt = 0;
    // the body for one wave tile; FULL (every column of the tile is below d) drops the bounds checks
    uint64_t pend = 0;                                          // group words of the run so far: coarse, lane i holds tile i's;
                                                                // fine, lane 4i + u holds word u of tile i
    auto tile = [&](auto full_c, uint32_t t, uint32_t ti) {
        constexpr bool FULL = decltype(full_c)::value;
        float4 a[4];
        if (!RK) {
            if (FULL) {
                ld_tile<VEC>(g, t, lane, a);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) a[u] = ld4<VEC, true>(g, t * kWaveTile + u * kChunk + lane * 4, d);
            }
        }
        uint64_t line_word = 0;                                 // the tile's one coarse group word (wave-uniform)
        uint32_t sure16 = 0;                                    // RK: bit 4u + q: my column q of chunk u has key >= hi
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            uint32_t keys[4];
            if (RK) {
#pragma unroll
                for (int q = 0; q < 4; ++q) keys[q] = rk_priority(k0, k1, j + q);
            } else {
                keys[0] = key_of(a[u].x);
                keys[1] = key_of(a[u].y);
                keys[2] = key_of(a[u].z);
                keys[3] = key_of(a[u].w);
            }
            uint64_t bc[4];
            uint32_t hi4;
            const uint64_t any_lo = filter_chunk<FULL, RK>(keys, j, d, lo, hi, bc, n_hi, kmax, hi4);
            if (!RK) {                                          // both forms, without a branch: a few scalar operations
                line_word |= any_of_four_lanes(any_lo) << u;
                if (!coarse) pend = lane == 4 * ti + (uint32_t)u ? any_lo : pend;
            }
            sure16 |= hi4 << (4 * u);
            stage_candidates(fb, keys, j, bc, stage, wst, wcnt, staged, lane);
        }
        if (RK) kbits[((size_t)row * nwt + t) * 64 + lane] = (uint16_t)sure16;
        else if (coarse) pend = lane == ti ? line_word : pend;
    };
    // A wave takes `run` (at most 16) consecutive wave tiles at a time and stores their group words together
    // (a block's four waves then fill whole 128-byte lines of the coarse bitmap with run = 4; measured equal to a
    // store per tile, and to longer runs: what the bitmap costs the pass, a tenth of its time, goes with the
    // bytes written, not with the number of stores).  Short rows keep run = 1, so that enough blocks are in flight.
    for (uint32_t tb = (blockIdx.x * 4 + wave) * run; tb < nwt; tb += gridDim.x * 4 * run) {
        const uint32_t te = min(tb + run, nwt);
        for (uint32_t t = tb; t < te; ++t) {
            if ((t + 1) * (uint32_t)kWaveTile <= d) tile(std::true_type{}, t, t - tb);    // wave-uniform
            else tile(std::false_type{}, t, t - tb);
        }
        if (!RK && gbits) {
            if (coarse) {
                if (lane < te - tb) gbits[(size_t)blockIdx.y * nwt + tb + lane] = pend;
            } else if (lane < 4 * (te - tb)) {
                gbits[((size_t)blockIdx.y * nwt + tb) * 4 + lane] = pend;
            }
        }
    }
    // keys at or above 0x7f800000 are Inf / NaN (magnitude keys only: priorities use the whole range)
    if (!RK && __ballot(kmax >= 0x7f800000u) && lane == 0) atomicOr(&desc[row].nonfinite_acc, 1u);
    finish_filter_block(fb, stage, wst, wcnt, n_hi, staged, wsure);
}

// Random-k when the band is thin against the row (k * 2^32 / d well below d): instead of computing the
// priority of every column, walk the 32-bit words y whose priority y >> 1 is at or above the band's
// lower end and invert the permutation; words that land on a column below d are the row's keys >= lo.
// The work is O(k * 2^32 / d) per row instead of O(d).  Same outputs as k_filter<., true>: the count of
// keys above the band, the candidate list, and the bits of the columns above the band -- set with
// atomic ORs into a bitmap that k_rk_zero cleared.  grid = (blocks, rows).
// Bound by its integer arithmetic and the atomics of the columns above the band (8e5 to as many lines for 32 rows of
// 25.6M columns, k/d = 0.1 %).  Two multiplications and every step for each of the 1.5e8 words took 128 us there, one
// multiplication and a look at the index's upper half 99.
constexpr int kInverseWords = 4;                                // words per lane and iteration (8: 5 us slower)
__global__ __launch_bounds__(kBlock) void k_rk_zero(uint32_t nwt, uint32_t row0, const RowDesc* __restrict__ desc,
                                                     uint16_t* __restrict__ kbits) {
    const uint32_t row = row0 + blockIdx.y;
    if (desc[row].mode != kWarm) return;
    uint4* __restrict__ words = reinterpret_cast<uint4*>(kbits + (size_t)row * nwt * 64);
    const uint32_t n = nwt * 8;
    for (uint32_t q = blockIdx.x * kBlock + threadIdx.x; q < n; q += gridDim.x * kBlock) words[q] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(kBlock) void k_rk_filter_inverse(uint32_t d, uint32_t nwt, uint32_t row0,
                                                               RowDesc* __restrict__ desc, uint16_t* __restrict__ kbits,
                                                               uint2* __restrict__ list, uint32_t cap, RkDraw rk) {
    __shared__ uint2 stage[kStage], wstage[4][kWaveStage];
    __shared__ uint32_t wsure[5], staged[2];
    const uint32_t row = row0 + blockIdx.y;
    FilterBand fb;
    if (!filter_band(desc, row, false, nullptr, list, cap, 0u, nullptr, nullptr, fb)) return;   // uniform for the block
    if (threadIdx.x < 2) staged[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lo = fb.lo, hi = fb.hi;
    uint32_t* __restrict__ words = reinterpret_cast<uint32_t*>(kbits + (size_t)row * nwt * 64);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint64_t stream = rk_stream(rk.state->seed, rk.state->draw, row);
    const uint32_t k0 = (uint32_t)stream, k1 = (uint32_t)(stream >> 32);
    // The index whose 32-bit word (priority with its dropped bit put back) is y: every step of rk_priority undone in reverse
    // order (the multipliers' inverses modulo 2^32; x ^= x >> 13 is undone by two shifts, x ^= x >> 16 by itself).
    // The words y whose priority is at least lo, y in [2 lo, 2^32), are walked as w = y ^ (y >> 16), the inverse's first
    // step (its own inverse, and a permutation of each block of 2^16 words): w runs over whole such blocks, from the one
    // that holds 2 lo.  The multiplication that follows is linear in w, so a step to the next words is one addition.
    // Almost every word lands beyond d, which the upper half of the index shows before the last step.
    const uint32_t y_first = 2u * lo, top = (d - 1) | 0xffffu;
    const uint64_t w_end = 1ull << 32;
    uint32_t n_hi = 0;
    uint2* wst = wstage[wave];
    uint32_t wcnt = 0;
    const uint32_t stride = gridDim.x * 4 * 64 * kInverseWords;
    uint64_t base = (y_first & 0xffff0000u) + ((uint64_t)blockIdx.x * 4 + wave) * 64 * kInverseWords;
    uint32_t p = ((uint32_t)base + lane) * 0x7ED1B41Du - k1;    // 0xC2B2AE35^-1
    for (; base < w_end; base += stride, p += stride * 0x7ED1B41Du) {
        uint32_t h[kInverseWords];
        uint32_t hit = 0;
#pragma unroll
        for (int i = 0; i < kInverseWords; ++i) {
            const uint32_t f = p + (uint32_t)i * (64u * 0x7ED1B41Du);
            h[i] = (f ^ (f >> 13) ^ (f >> 26)) * 0xA5CB9243u;   // 0x85EBCA6B^-1
            hit |= ((h[i] ^ k0) <= top ? 1u : 0u) << i;         // the last step only changes the lower half
        }
        if (__ballot(hit != 0) == 0) continue;                  // wave-uniform
#pragma unroll
        for (int i = 0; i < kInverseWords; ++i) {
            const uint32_t w = (uint32_t)base + (uint32_t)i * 64u + lane, y = w ^ (w >> 16), key = y >> 1;
            const uint32_t j = h[i] ^ (h[i] >> 16) ^ k0;
            const bool ok = j < d && y >= y_first;
            if (__ballot(ok) == 0) continue;                    // wave-uniform
            const bool ge_hi = ok && key >= hi;
            if (ge_hi) {
                const uint32_t t = j / kWaveTile, o = j % kWaveTile;
                const uint32_t half = t * 64 + (o % kChunk) / 4;              // half-word of the row holding the column
                atomicOr(&words[half >> 1], 1u << ((half & 1) * 16 + 4 * (o / kChunk) + o % 4));
                ++n_hi;
            }
            const uint64_t bc = __ballot(ok && !ge_hi);         // candidates: lo <= key < hi
            if (bc) {                                           // wave-uniform
                const uint32_t m = __popcll(bc);
                const StagePos sp = reserve_stage(fb, m, staged, wst, wcnt, lane);
                if ((bc >> lane) & 1) put_candidate(stage, wst, sp, lanes_below(bc), make_uint2(key, j));
            }
        }
    }
    finish_filter_block(fb, stage, wst, wcnt, n_hi, staged, wsure);
}

// First radix digit (12 bits) of every key of the rows that have no usable band; for the rows whose
// predicted band holds rank k, the first digit of the listed keys instead (list_first_digit).  Either
// histogram goes to the row's kHistBins words of `hist`.  grid = (blocks, rows).
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_hist0(const float* __restrict__ src, size_t row_stride, uint32_t d,
                                                   uint32_t nwt, uint32_t row0, const RowDesc* __restrict__ desc,
                                                   uint32_t* __restrict__ hist, const uint2* __restrict__ list, uint32_t cap,
                                                   uint32_t k) {
    __shared__ uint32_t h[kHistBins];
    const uint32_t row = row0 + blockIdx.y;
    if (!wants_cold(desc[row], cap, k)) {                       // uniform for the block
        if (desc[row].mode == kWarm) list_first_digit(desc, row, list + (size_t)row * cap, hist + (size_t)row * kHistBins, h);
        return;
    }
    const float* __restrict__ g = src + (size_t)blockIdx.y * row_stride;
    for (int b = threadIdx.x; b < kHistBins; b += kBlock) h[b] = 0;
    __syncthreads();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (uint32_t t = blockIdx.x * 4 + wave; t < nwt; t += gridDim.x * 4) {
        float4 a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = ld4<VEC, true>(g, t * kWaveTile + u * kChunk + lane * 4, d);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            const uint32_t keys[4] = {key_of(a[u].x), key_of(a[u].y), key_of(a[u].z), key_of(a[u].w)};
#pragma unroll
            for (int q = 0; q < 4; ++q) wave_count(h, j + q < d, keys[q] >> 19, lane);
        }
    }
    __syncthreads();
    uint32_t* __restrict__ out = hist + (size_t)row * kHistBins;
    for (int b = threadIdx.x; b < kHistBins; b += kBlock) {
        const uint32_t c = h[b];
        if (c) atomicAdd(&out[b], c);
    }
}

// One pass of the block over the n listed entries, two entries per 128-bit load and eight loads in flight
// per thread (a row's list starts 16-byte aligned): fn(entry, valid) is called in wave-uniform control
// flow (valid false beyond n), so it may use wave_count.  SHARED: blocks of this launch may have written the entries
// (put_entry<true>); they are then loaded past the caches, one at a time (an acquire fence instead drops an L2's lines, once for
// every wave of the block: a step without predictions of 64 x 65536 columns 104 us against 78).
constexpr int kSelectBlock = 1024;
template <bool SHARED>
__device__ __forceinline__ uint4 two_entries(const uint4* __restrict__ at) {
    if (!SHARED) return *at;
    const unsigned long long* const e = reinterpret_cast<const unsigned long long*>(at);
    const unsigned long long a = ld_shared(e), b = ld_shared(e + 1);
    return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
}
template <bool SHARED, typename F>
__device__ __forceinline__ void for_each_listed(const uint2* __restrict__ in, uint32_t n, F fn) {
    const uint32_t tid = threadIdx.x;
    const uint4* __restrict__ in2 = reinterpret_cast<const uint4*>(in);
    const uint32_t npairs = (n + 1) / 2;                    // the slot after an odd n is inside the row's capacity
    for (uint32_t base = 0; base < npairs; base += 8 * kSelectBlock) {     // uniform trip count
        uint4 a[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t e = base + q * kSelectBlock + tid;
            a[q] = e < npairs ? two_entries<SHARED>(&in2[e]) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t e = 2 * (base + q * kSelectBlock + tid);
            fn(make_uint2(a[q].x, a[q].y), e < n);
            fn(make_uint2(a[q].z, a[q].w), e + 1 < n);
        }
    }
}

// What is left of a row's search once its candidates are listed: radix digits over the listed keys narrow them down to
// the at most kFewHeld (kFewEntries) that share the digits found so far, and those are compared with one another, which gives tau
// and the cut-off at once.  When more entries than that share the whole key (quantised gradients: thousands of equal
// magnitudes), the cut-off is the `rank`-th smallest index among them, found by radix digits of those indices
// until at most so many are left, which are compared as before.
// One block of kSelectBlock threads, bound by latency: barriers, round trips to LDS, the code itself, which every launch
// fetches anew, and on thousands of entries the instructions of one compute unit.  A list of up to kHeldMax entries is copied into LDS
// once, so that every pass over it is a short loop (held in registers, each pass was that loop unrolled sixteen times); its
// digits take kHeldBits bits, with 16 copies of every bin for lanes that name the same one (gradients of few mantissa bits
// put thousands of entries on one key: with one copy of 1024 bins the first digit of 9000 entries took 5 us, now 1.5), picked by
// one wave.  Among n <= kFewHeld there are no digits at all (128: comparing costs the square).  us per step, before and after: 5 x 3M
// columns of bf16 mantissas 99.1 -> 90.5, 8 x 4.2M of them 150 -> 144, 8 x 262144 31.3 -> 30.5, 8 x 1M and 64 x 524288 even.  A digit of the
// indices counted in the hope that the first digit's bin holds one key alone saves the workers' rows 2 us and costs the
// server's, whose bins hold several, as much.
// A list of more than kHeldShort entries (12 a thread) takes the place of half the copies: 20 KB of LDS are left on the compute unit, enough for a
// block of k_filter (17 KB), so that contexts on streams of their own overlap (two of 8 x 1M columns, us a round of steps: 95, with the list in
// registers 104; with 16 copies beside 16 entries a thread, 13.6 KB left, half as long again).  Lists of 12600 to 16000 entries that one block
// does not hold cost more, us per step of one row of 1M columns: 30.5 against 28.8 now, without a prediction and with thousands of equal
// keys 56.5 against 48.8.
// A list that is not held is read again for every digit: it stops at kFewEntries, and waves none of whose entries
// carry the digits found so far are done with them at once.  us per step with 128 and without that, with 256, with both: blockwise / top-k
// 2 x 20M, 1 %, whose server lists 250 000 to 430 000 entries, 560, 558, 461; top-k on both sides, 5 %, of bf16 mantissas 617, 617, 549;
// sign / top-k 2 x 20M 389, 380, 355, 3 x 5M 184, 180, 174.
constexpr uint32_t kHeldMax = 16u * kSelectBlock, kHeldShort = 12u * kSelectBlock;
static_assert(kHeldMax == (uint32_t)kDirectList && kHeldMax == kShortCapOne, "what one block selects from it holds");
constexpr uint32_t kHeldShifts = 4;            // log2 of the copies of a bin, one less over a list longer than kHeldShort
constexpr int kHeldBins = 1 << kHeldBits;
struct ListLds {
    union {
        struct {
            __align__(16) uint2 held[kHeldMax];                            // the list
            __align__(16) uint32_t h_long[kHeldBins << (kHeldShifts - 1)];  // digit histogram of the held list,
        };
        struct {
            uint2 held_short[kHeldShort];
            __align__(16) uint32_t h_short[kHeldBins << kHeldShifts];       // where it begins while the list is short
        };
        uint32_t wide[kListBins];              // digit histogram over a list that is not held
    };
    __align__(16) uint32_t sums[kHeldBins];
    __align__(16) uint2 few[kFewEntries];      // the last few entries
    uint32_t part[256], res[3];
    uint32_t tau, cut, rank, nties;            // the result
};
static_assert(sizeof(ListLds) + 2 * sizeof(RowDesc) + 17 * 1024 <= 160 * 1024, "LDS of a compute unit, a block of the filter beside it");
static_assert(kHeldBits == 8 && kHeldShifts == 4 && kSelectBlock == 1024, "a thread clears and adds up four copies of a bin, a wave picks among the bins");
static_assert(4 * kFewEntries <= kSelectBlock, "four threads compare one of the last entries");

// The list of n <= kHeldMax entries into LDS.  shared (uniform): blocks of this launch wrote it.
template <bool SHARED>
__device__ __forceinline__ void hold_listed(ListLds& s, const uint2* __restrict__ in, uint32_t n, bool shared) {
    const uint4* __restrict__ in2 = reinterpret_cast<const uint4*>(in);
    uint4* const out = reinterpret_cast<uint4*>(s.held);
    const uint32_t npairs = (n + 1) / 2, tid = threadIdx.x;    // the slot after an odd n is inside the row's capacity
    // requested together, without a branch among them, in one round
    auto hold = [&](auto loads, auto fresh) {
        constexpr int L = decltype(loads)::value;
        uint4 a[L];
#pragma unroll
        for (int q = 0; q < L; ++q) a[q] = two_entries<decltype(fresh)::value>(&in2[min(q * kSelectBlock + tid, npairs - 1)]);
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (q * kSelectBlock + tid < npairs) out[q * kSelectBlock + tid] = a[q];
    };
    using One = std::integral_constant<int, 1>;
    using Short = std::integral_constant<int, kHeldShort / (2 * kSelectBlock)>;
    using All = std::integral_constant<int, kHeldMax / (2 * kSelectBlock)>;
    if (SHARED && shared) hold(All{}, std::true_type{});
    else if (npairs <= kSelectBlock) hold(One{}, std::false_type{});
    else if (n <= kHeldShort) hold(Short{}, std::false_type{});
    else hold(All{}, std::false_type{});
    __syncthreads();
}
// fn(entry, valid) for every listed entry, in wave-uniform control flow.
template <bool HELD, bool SHARED, typename F>
__device__ __forceinline__ void walk_list(const ListLds& s, const uint2* __restrict__ in, uint32_t n, F fn) {
    if (HELD) {
#pragma unroll 1
        for (uint32_t base = 0; base < n; base += kSelectBlock) fn(s.held[base + threadIdx.x], base + threadIdx.x < n);
    } else {
        for_each_listed<SHARED>(in, n, fn);
    }
}
// The bin of a digit of at most `bits` bits that holds the entry of rank `rank` (1-based, largest first), of the entries for which
// digit(entry, valid, bin) is true and leaves their bin.
template <bool HELD, bool SHARED, typename D>
__device__ __forceinline__ Pick pick_digit(ListLds& s, const uint2* __restrict__ in, uint32_t n, int bits, uint32_t rank, D digit) {
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    if (!HELD) {
        const uint32_t nbins = max(256u, 1u << bits);
        for (uint32_t b = tid; b < nbins; b += kSelectBlock) s.wide[b] = 0;
        __syncthreads();
        walk_list<false, SHARED>(s, in, n, [&](uint2 kv, bool valid) {
            uint32_t bin = 0;
            valid = digit(kv, valid, bin);
            if (__ballot(valid)) wave_count(s.wide, valid, bin, lane);     // uniform: after the first digit most waves have none
        });
        __syncthreads();
        return block_pick(s.wide, (int)nbins, rank, s.part, s.res);
    }
    const bool is_short = n <= kHeldShort;                      // uniform
    const uint32_t shift = is_short ? kHeldShifts : kHeldShifts - 1, own_copy = lane & ((1u << shift) - 1u);
    uint32_t* const h = is_short ? s.h_short : s.h_long;
    const bool mine4 = tid < (uint32_t)kHeldBins << (shift - 2);       // whole waves
    if (mine4) reinterpret_cast<uint4*>(h)[tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    walk_list<true, SHARED>(s, in, n, [&](uint2 kv, bool valid) {
        uint32_t bin = 0;
        valid = digit(kv, valid, bin);
        if (valid) atomicAdd(&h[(bin << shift) + own_copy], 1u);
    });
    __syncthreads();
    if (mine4) {
        const uint4 c = reinterpret_cast<const uint4*>(h)[tid];
        uint32_t sum = c.x + c.y + c.z + c.w;                   // four threads a bin, or two
        sum += dpp_or_zero<0xb1, 0xf>(sum);                     // lanes 1 0 3 2 of every four
        const uint32_t other = dpp_or_zero<0x4e, 0xf>(sum);     // lanes 2 3 0 1
        if (is_short) sum += other;
        if ((tid & ((1u << (shift - 2)) - 1u)) == 0) s.sums[tid >> (shift - 2)] = sum;
    }
    __syncthreads();
    if (tid < 64) {                                             // lane l: bins 4l .. 4l + 3
        const uint4 b = reinterpret_cast<const uint4*>(s.sums)[lane];
        const uint32_t own = b.x + b.y + b.z + b.w, upto = wave_scan(own), above = last_lane(upto) - upto;
        const bool mine = above < rank && rank <= above + own;
        uint32_t bin = 4 * lane + 3, ahead = above, count = b.w;
        if (rank > ahead + count) {
            ahead += count;
            count = b.z;
            --bin;
            if (rank > ahead + count) {
                ahead += count;
                count = b.y;
                --bin;
                if (rank > ahead + count) {
                    ahead += count;
                    count = b.x;
                    --bin;
                }
            }
        }
        const bool none = __ballot(mine) == 0;                  // (a vote of all lanes: one lane writes)
        if (mine || (lane == 0 && none)) {
            s.res[0] = mine ? bin : 0u;
            s.res[1] = mine ? rank - ahead : 1u;
            s.res[2] = mine ? count : 0u;
        }
    }
    __syncthreads();
    return Pick{s.res[0], s.res[1], s.res[2]};                  // (two more barriers before anyone writes them again)
}

// The search itself, see select_listed.
template <bool HELD, bool SHARED>
__device__ __forceinline__ void narrow_list(ListLds& s, const uint2* __restrict__ in, uint32_t n, uint32_t lo, uint32_t width,
                                            uint32_t rank, bool first, Pick ph, int shift, uint32_t d, bool shared) {
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const int key_bits = HELD ? kHeldBits : kListBits, index_bits = HELD ? kHeldBits : kIndexBits;
    constexpr uint32_t kFew = HELD ? kFewHeld : kFewEntries;
    if (HELD) hold_listed<SHARED>(s, in, n, shared);
    if (first && n <= kFew) {                                   // all of them are compared
        shift = band_bits(width);
        ph = Pick{0u, rank, n};
    } else if (first) {
        shift = first_shift(width, key_bits);
        ph = pick_digit<HELD, SHARED>(s, in, n, band_bits(width) - shift, rank, [&](uint2 kv, bool valid, uint32_t& bin) {
            bin = (kv.x - lo) >> shift;
            return valid;
        });
    }
    // The following digits, over the entries that carry the digits found so far, until few are left or the key is known.
    uint32_t prefix = ph.bin, want = ph.rank_in, left = ph.count;
#pragma unroll 1
    while (shift > 0 && left > kFew) {
        const int bits = shift < key_bits ? shift : key_bits, below = shift - bits;
        const uint32_t mask = (1u << bits) - 1u;
        const Pick p = pick_digit<HELD, SHARED>(s, in, n, bits, want, [&](uint2 kv, bool valid, uint32_t& bin) {
            const uint32_t rel = kv.x - lo;
            bin = (rel >> below) & mask;
            return valid && (rel >> shift) == prefix;
        });
        prefix = (prefix << bits) | p.bin;
        want = p.rank_in;
        left = p.count;
        shift = below;
    }
    // Many entries of one key (quantised gradients): the want-th of them in index order.  Digits of the
    // indices, counted down from the largest, which turns "want-th smallest" into the "want-th largest" that the pick
    // finds; again until few are left.
    const uint32_t ties = left, want_key = want;                // entries of the key, when it is known here
    const uint32_t top = d - 1;
    int ishift = band_bits(d);                                  // index bits below the digits found so far
    uint32_t ifound = 0;
#pragma unroll 1
    while (left > kFew) {                                       // indices are distinct: ends before ishift would go below 0
        const int bits = ishift < index_bits ? ishift : index_bits, below = ishift - bits;
        const uint32_t mask = (1u << bits) - 1u;
        const Pick p = pick_digit<HELD, SHARED>(s, in, n, bits, want, [&](uint2 kv, bool valid, uint32_t& bin) {
            const uint32_t inv = top - kv.y;
            bin = (inv >> below) & mask;
            return valid && kv.x == lo + prefix && (inv >> ishift) == ifound;
        });
        ifound = (ifound << bits) | p.bin;
        want = p.rank_in;
        left = p.count;
        ishift = below;
    }
    // The entries that are left, compared with one another: the one with want - 1 others ahead of it (larger key, or
    // the same key and a lower index) is the row's k-th.
    if (tid == 0) s.nties = 0;
    __syncthreads();
    walk_list<HELD, SHARED>(s, in, n, [&](uint2 kv, bool valid) {
        const bool hit = valid && ((kv.x - lo) >> shift) == prefix && ((top - kv.y) >> ishift) == ifound;
        const uint64_t m = __ballot(hit);
        if (m == 0) return;                                     // uniform
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s.nties, (uint32_t)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + lanes_below(m);
        if (hit && at < kFew) s.few[at] = kv;
    });
    __syncthreads();
    if ((tid >> 2) < left) {                                    // four threads an entry, each a quarter of the others
        const uint2 mine = s.few[tid >> 2];
        uint32_t larger = 0, equal = 0, earlier = 0;
#pragma unroll 4
        for (uint32_t r = tid & 3; r < left; r += 4) {
            const uint2 o = s.few[r];
            larger += o.x > mine.x ? 1u : 0u;
            equal += o.x == mine.x ? 1u : 0u;
            earlier += o.x == mine.x && o.y < mine.y ? 1u : 0u;
        }
        larger += dpp_or_zero<0xb1, 0xf>(larger);
        equal += dpp_or_zero<0xb1, 0xf>(equal);
        earlier += dpp_or_zero<0xb1, 0xf>(earlier);
        larger += dpp_or_zero<0x4e, 0xf>(larger);
        equal += dpp_or_zero<0x4e, 0xf>(equal);
        earlier += dpp_or_zero<0x4e, 0xf>(earlier);
        if ((tid & 3) == 0 && larger + earlier + 1 == want) {   // indices are distinct: one thread
            const bool by_index = ties != left;                 // the entries went through the index digits
            s.tau = mine.x;
            s.cut = mine.y;
            s.rank = by_index ? want_key : want - larger;
            s.nties = by_index ? ties : equal;
        }
    }
    __syncthreads();
}
// in: n entries with keys in [lo, lo + width), `rank`: how many from the top the searched one is.  first: the first digit
// is not known yet; otherwise ph and shift say what is.  Every thread of the block calls it; the result is in s (all threads
// see it).
// shared (uniform): blocks of this launch wrote the list; SHARED: they may have.
template <bool SHARED>
__device__ __forceinline__ void select_listed(ListLds& s, const uint2* __restrict__ in, uint32_t n, uint32_t lo, uint32_t width,
                                              uint32_t rank, bool first, Pick ph, int shift, uint32_t d, bool shared) {
    if (n <= kHeldMax) narrow_list<true, SHARED>(s, in, n, lo, width, rank, first, ph, shift, d, shared);       // uniform for the block
    else narrow_list<false, SHARED>(s, in, n, lo, width, rank, first, ph, shift, d, shared);
}

// The row's descriptor in LDS, in one round trip instead of one per dependent field.  64 threads or more; the caller
// synchronises.
static_assert(sizeof(RowDesc) == 64 * sizeof(uint32_t), "64 lanes copy the descriptor");
__device__ __forceinline__ void fetch_desc(RowDesc& now, const RowDesc* __restrict__ desc) {
    if (threadIdx.x < 64) reinterpret_cast<uint32_t*>(&now)[threadIdx.x] = reinterpret_cast<const uint32_t*>(desc)[threadIdx.x];
}
// And back, its first line: the counters of the second stay as the passes left them (every block of a kernel that finishes
// searches can still tell from them what the row needed) until the update kernel clears them.  Every thread calls it, after
// thread 0 has changed `now`.
constexpr uint32_t kFirstLineWords = 32;
__device__ __forceinline__ void put_result(RowDesc* __restrict__ desc, const RowDesc& now) {
    __syncthreads();
    if (threadIdx.x < kFirstLineWords)
        reinterpret_cast<uint32_t*>(desc)[threadIdx.x] = reinterpret_cast<const uint32_t*>(&now)[threadIdx.x];
}
__device__ __forceinline__ ListFound found_in(const ListLds& s) { return ListFound{s.tau, s.rank, s.nties, s.cut}; }

// grid = rows, kSelectBlock threads: finishes the list select of a row.  Which band the row's list was filtered
// against -- the predicted one, or the first-digit bin picked (again, here) from the row's histogram --
// follows from the row's mode and first counter set, as in the filter passes.  For a row on its predicted band the first
// digit's histogram is ready (k_hist0) and,
// when the bin holding rank k was small enough, so is the short list of that bin's entries (second k_filter
// pass): the rest of the select then reads those few entries only.  Otherwise the block walks the list
// itself.  Then the row's histogram is
// cleared, the next step's band is predicted and the row is back in kWarm mode.
// Rows whose list does not hold rank k
// (overflow, a bin larger than the list, rank outside the band) are put into kSlow mode.
__global__ __launch_bounds__(kSelectBlock) void k_list_select(uint32_t row0, RowDesc* __restrict__ desc,
                                                               uint32_t* __restrict__ ghist,
                                                               const uint2* __restrict__ list, uint32_t cap,
                                                               const uint2* __restrict__ shortl, uint32_t k, uint32_t d,
                                                               uint32_t form) {
    __shared__ ListLds s;
    __shared__ RowDesc now;                                    // the row's descriptor as the kernel found it
    const uint32_t row = row0 + blockIdx.x, tid = threadIdx.x;
    fetch_desc(now, desc + row);
    __syncthreads();
    if (now.mode == kSlow) return;
    const bool cold = wants_cold(now, cap, k);                  // uniform for the block
    const uint32_t missed = (cold && now.mode == kWarm) ? 1u : 0u;    // there was a prediction and it failed
    uint32_t* __restrict__ hrow = ghist + (size_t)row * kHistBins;
    const uint2* __restrict__ in = list + (size_t)row * cap;
    uint32_t lo, hi, n, n_sure;
    bool ok = true;
    Pick ph{0, 0, 0};                                           // first digit: bin holding rank k, rank inside it
    bool direct = cold;                                         // this block builds the first digit's histogram itself
    if (cold) {
        const Pick p = block_pick(hrow, kHistBins, k, s.part, s.res);
        lo = p.bin << 19;
        hi = (p.bin + 1) << 19;
        n = now.n_cand2;
        n_sure = sure_count2(now);
        ok = p.count <= cap && n <= cap && n_sure < k && (uint64_t)k <= (uint64_t)n_sure + n;
    } else {                                                    // kWarm and band_ok
        lo = now.lo;
        hi = now.hi;
        n = now.n_cand;
        n_sure = sure_count(now);
        direct = n <= (uint32_t)kDirectList;
        if (!direct) ph = block_pick(hrow, 1 << kFirstBits, k - n_sure, s.part, s.res);
    }
    if (cold || !direct)
        for (int b = tid; b < kHistBins; b += kSelectBlock) hrow[b] = 0;    // the row's histogram is ready for the next step
    if (!ok) {
        if (tid == 0) {
            now.n_list = 0;
            now.misses += missed;
            now.mode = kSlow;
        }
        put_result(desc + row, now);
        return;
    }
    const uint32_t n_all = n;
    if (!direct && ph.count <= (uint32_t)kShortCap && now.n_short == ph.count) {
        in = shortl + (size_t)row * kShortCap;                  // the bin's entries, collected by the second filter pass
        n = ph.count;
    }
    select_listed<false>(s, in, n, lo, hi - lo, k - n_sure, direct, ph, first_shift(hi - lo, kFirstBits), d, false);
    if (tid == 0) finish_listed(now, found_in(s), n_all, form, cold, missed, 0u, 0u);
    put_result(desc + row, now);
}

// ---------------------------------------------------------------------------------------------
// General search: three radix digits over the whole row, then the ties in
// index order.  On long rows only degenerate ones come here (constant or mostly-zero rows, values on a handful of
// levels: a threshold shared by more entries than the candidate list holds).
//   grid = (B, rows), 1024 threads.  With B > 1 the B blocks of a row split it into contiguous ranges
// and meet between the phases at a counter (every block adds one and polls
// until all B have arrived); the histograms of the three digits and the blocks' tie counts live in
// global memory.  The poll is bounded: when a wait runs out (blocks that could not all be resident
// at once, a GPU shared with other work) the row is flagged, every block leaves, and block 0
// repeats the search on its own with LDS histograms -- the B = 1 path.  Results are identical.
// Block 0 is the only writer of the row's result on either path, so a row cannot leave the kernel
// still in kSlow mode whatever the order in which waits run out.
// The host chooses B so that B * rows blocks fit the chip at one block per compute unit.
// ---------------------------------------------------------------------------------------------
constexpr int kSlowMaxBlocks = 64;
constexpr uint32_t kSlowHistWords = 4096 + 1024 + 512;        // the three digit histograms of a row
constexpr uint32_t kSyncWords = 4;                            // of a row: arrivals; some block has given up; the histograms are not zero

struct SlowLds {
    uint32_t h[kHistBins];
    uint32_t part[256], res[3];
    uint32_t wtot[16];
    uint32_t cut, bad, ok, dirty;
    RowDesc now;
};

// the 4 keys of columns j .. j + 3 (columns at or beyond d give unspecified keys; callers test j + q < d)
template <bool VEC, bool RK>
__device__ __forceinline__ void slow_keys_at(const float* __restrict__ g, uint32_t d, uint32_t k0, uint32_t k1, uint32_t j,
                                             uint32_t (&key)[4]) {
    if (RK) {
#pragma unroll
        for (int q = 0; q < 4; ++q) key[q] = rk_priority(k0, k1, j + q);
    } else {
        const float4 a = ld4<VEC>(g, j, d);
        key[0] = key_of(a.x);
        key[1] = key_of(a.y);
        key[2] = key_of(a.z);
        key[3] = key_of(a.w);
    }
}

// the keys of this lane's 16 columns of wave tile t.  A whole tile's loads have no branch among them: 62 rows of 2.1M + 1 columns
// without predictions, searched in one launch, 642 -> 563 us a step, 8 of 1M + 1 102 -> 92, 5 of 3M + 17 145 -> 135.
template <bool VEC, bool RK>
__device__ __forceinline__ void tile_keys(const float* __restrict__ g, uint32_t d, uint32_t k0, uint32_t k1, uint32_t t, uint32_t lane,
                                          uint32_t (&key)[4][4]) {
    if (!RK && (t + 1) * (uint32_t)kWaveTile <= d) {            // wave-uniform
        float4 a[4];
        ld_tile<VEC, false>(g, t, lane, a);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            key[u][0] = key_of(a[u].x);
            key[u][1] = key_of(a[u].y);
            key[u][2] = key_of(a[u].z);
            key[u][3] = key_of(a[u].w);
        }
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) slow_keys_at<VEC, RK>(g, d, k0, k1, t * kWaveTile + u * kChunk + lane * 4, key[u]);
    }
}

// One block on its own, histograms in LDS.
template <bool VEC, bool RK>
__device__ __forceinline__ SlowFound slow_single(SlowLds& s, const float* __restrict__ g, uint32_t d, uint32_t k, uint32_t k0, uint32_t k1) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t prefix = 0, rank = k, ties = 0, first = 0;
    if (tid == 0) s.bad = 0;
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = digit_shift(pass), nbins = 1 << digit_bits(pass);
        const int hi_shift = pass == 0 ? 31 : digit_shift(pass - 1);
        for (int b = tid; b < nbins; b += 1024) s.h[b] = 0;
        __syncthreads();
        for (uint32_t j = tid * 4; j < d; j += 4096) {
            uint32_t key[4];
            slow_keys_at<VEC, RK>(g, d, k0, k1, j, key);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + q < d && ((key[q] ^ prefix) >> hi_shift) == 0) atomicAdd(&s.h[(key[q] >> shift) & (nbins - 1)], 1u);
        }
        __syncthreads();
        if (pass == 0 && !RK) {                       // keys >= 0x7f800000 (Inf/NaN) sit in the bins from 0xff0 up
            bool bad = false;
            for (int b = 0xff0 + (int)tid; b < kHistBins; b += 1024) bad |= s.h[b] != 0;
            if (bad) s.bad = 1;
        }
        const Pick p = block_pick(s.h, nbins, rank, s.part, s.res);
        prefix |= p.bin << shift;
        rank = p.rank_in;
        ties = p.count;
        if (pass == 0) first = p.count;
    }
    // the rank-th entry with key == prefix, in index order
    if (tid == 0) s.cut = 0xffffffffu;
    __syncthreads();
    uint32_t seen = 0;
    for (uint32_t base = 0; base < d; base += 4096) {          // uniform trip count and exit
        const uint32_t j = base + tid * 4;
        uint32_t key[4];
        slow_keys_at<VEC, RK>(g, d, k0, k1, j, key);
        const bool m0 = j < d && key[0] == prefix, m1 = j + 1 < d && key[1] == prefix;
        const bool m2 = j + 2 < d && key[2] == prefix, m3 = j + 3 < d && key[3] == prefix;
        const uint32_t mine = m0 + m1 + m2 + m3;
        const uint32_t incl = wave_scan(mine);
        if (lane == 63) s.wtot[wave] = incl;
        __syncthreads();
        uint32_t before = seen, total = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < (int)wave) before += s.wtot[w];
            total += s.wtot[w];
        }
        before += incl - mine;
        if (before < rank && rank <= before + mine) {
            uint32_t need = rank - before, idx = j + 3;
            if (m0 && --need == 0) idx = j;
            else if (m1 && --need == 0) idx = j + 1;
            else if (m2 && --need == 0) idx = j + 2;
            s.cut = idx;
        }
        seen += total;
        __syncthreads();
        if (seen >= rank) break;
    }
    __syncthreads();
    return SlowFound{prefix, rank, ties, s.cut, s.bad, first};
}

// Meeting point of blocks that share a row: true when `target` arrivals have been counted, false when the
// wait ran out or another block has given up (the row is then flagged).  Every thread calls it.
// No fence: what the blocks hand to one another goes past their L2s (st_shared, ld_shared, atomics), and every wave waits
// for its own stores.  With a device-wide fence (an L2 written back and its stale lines dropped) in every one
// of the blocks' 16 waves a meeting took 0.1 ms: a general search of 8 x 262144 columns, 5 meetings, 580 us; with one fence a
// block 55.
__device__ __forceinline__ void slow_written() {                // what the block has stored past the L2 is there for all to load
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    __syncthreads();
}
__device__ __forceinline__ void slow_arrive(uint32_t* __restrict__ sync) {
    slow_written();
    if (threadIdx.x == 0) atomicAdd(&sync[0], 1u);
}
__device__ __forceinline__ bool slow_meet(uint32_t& ok_lds, uint32_t* __restrict__ sync, uint32_t target, uint32_t spin_limit) {
    slow_arrive(sync);
    if (threadIdx.x == 0) {
        uint32_t ok = 0;
        for (uint32_t spin = 0; spin < spin_limit; ++spin) {
            if (ld_shared(&sync[1])) break;
            if (ld_shared(&sync[0]) >= target) {
                ok = 1;
                break;
            }
            if (spin < 64) __builtin_amdgcn_s_sleep(1);
            else __builtin_amdgcn_s_sleep(16);
        }
        if (!ok) atomicExch(&sync[1], 1u);
        ok_lds = ok;
    }
    __syncthreads();
    return ok_lds != 0;
}

// The B blocks of a row together (one block on its own has nothing to hand over, to meet for or to give up).  Only block 0's return value matters: kGaveUp when one of its waits ran out (the
// caller then repeats the search on block 0 alone), kFound when `found` is the result.  A block other than 0 whose
// wait runs out just leaves (block 0 then fails its next wait, because the give-up flag is set or the
// arrivals never add up).  groups: the row's candidate bitmap (top-k, in the form that k_filter writes), for which the
// blocks flag the groups that hold a key of at least tau while they count the ties; valid when block 0 returns kFound.
// kListed (to every block): at most list_cap entries share the first digit found.tau that holds rank k, as number
// found.rank of its found.first, and the caller goes on with a list of those.
// The histograms are zero before and after; when waits have run out, sync[2] says that they may not be, and the next
// search starts by clearing them.
__device__ __forceinline__ void clear_slow_hist(uint32_t* __restrict__ ghist, uint32_t* __restrict__ sync) {    // block 0, the others are done
    for (uint32_t q = threadIdx.x; q < kSlowHistWords; q += 1024) ghist[q] = 0;
    if (threadIdx.x == 0) sync[2] = 0;
}
enum SlowEnd : int { kGaveUp = 0, kFound = 1, kListed = 2 };
template <bool VEC, bool RK>
__device__ __forceinline__ SlowEnd slow_multi(SlowLds& s, const float* __restrict__ g, uint32_t d, uint32_t nwt, uint32_t k, uint32_t k0, uint32_t k1,
                              uint32_t* __restrict__ ghist, uint32_t* __restrict__ gcnt, uint32_t* __restrict__ sync,
                              uint32_t spin_limit, uint64_t* __restrict__ groups, bool coarse, uint32_t list_cap, uint32_t& meetings,
                              SlowFound& found) {
    const uint32_t B = gridDim.x, b = blockIdx.x;
    const bool shared = B > 1;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t tpb = (nwt + B - 1) / B;                     // wave tiles per block: a contiguous range of the row
    const uint32_t t0 = min(b * tpb, nwt), t1 = min(t0 + tpb, nwt);
    meetings = 0;
    if (tid == 0) {
        s.bad = 0;
        s.dirty = shared ? ld_shared(&sync[2]) : 0u;
        s.ok = shared ? ld_shared(&sync[1]) == 0 : 1u;
    }
    __syncthreads();
    if (!s.ok) return kGaveUp;                                  // somebody's wait has run out before this block started
    // whatever an earlier, abandoned search left in the global histograms goes first
    if (s.dirty) {                                              // uniform for the block
        for (uint32_t q = b * 1024 + tid; q < kSlowHistWords; q += B * 1024) st_shared(&ghist[q], 0u);
        if (!slow_meet(s.ok, sync, B * ++meetings, spin_limit)) return kGaveUp;
    }
    uint32_t prefix = 0, rank = k, ties = 0, off = 0, first = 0;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = digit_shift(pass), nbins = 1 << digit_bits(pass);
        const int hi_shift = pass == 0 ? 31 : digit_shift(pass - 1);
        for (int q = tid; q < nbins; q += 1024) s.h[q] = 0;
        __syncthreads();
        for (uint32_t t = t0 + wave; t < t1; t += 16) {
            uint32_t key[4][4];
            tile_keys<VEC, RK>(g, d, k0, k1, t, lane, key);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool valid = j + q < d && ((key[u][q] ^ prefix) >> hi_shift) == 0;
                    const uint32_t bin = (key[u][q] >> shift) & (uint32_t)(nbins - 1);
                    wave_count(s.h, valid, bin, lane);
                }
            }
        }
        __syncthreads();
        if (shared) {
            for (int q = tid; q < nbins; q += 1024) {
                const uint32_t c = s.h[q];
                if (c) atomicAdd(&ghist[off + q], c);
            }
            if (!slow_meet(s.ok, sync, B * ++meetings, spin_limit)) return kGaveUp;
            for (int q = tid; q < nbins; q += 1024) s.h[q] = ld_shared(&ghist[off + q]);
            __syncthreads();
        }
        if (pass == 0 && !RK) {                       // keys >= 0x7f800000 (Inf/NaN) sit in the bins from 0xff0 up
            if (tid < 16 && s.h[0xff0 + tid] != 0) s.bad = 1;
        }
        const Pick p = block_pick(s.h, nbins, rank, s.part, s.res);
        prefix |= p.bin << shift;
        rank = p.rank_in;
        ties = p.count;
        if (pass == 0) {
            first = p.count;
            if (first <= list_cap) {                            // uniform for the row
                found = SlowFound{p.bin, rank, 0u, 0u, s.bad, first};
                return kListed;
            }
        }
        off += nbins;
    }
    // ties inside my range; block 0 then walks the range that holds the rank-th tie in index order
    uint32_t mine = 0;
    for (uint32_t t = t0 + wave; t < t1; t += 16) {
        uint64_t line_word = 0, fine = 0;                       // lane u holds fine word u
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            uint32_t key[4];
            slow_keys_at<VEC, RK>(g, d, k0, k1, j, key);
            bool any = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                mine += (j + q < d && key[q] == prefix) ? 1u : 0u;
                any |= j + q < d && key[q] >= prefix;
            }
            const uint64_t flags = __ballot(any);
            line_word |= any_of_four_lanes(flags) << u;
            fine = lane == (uint32_t)u ? flags : fine;
        }
        if (!RK && groups) {
            if (coarse) {
                if (lane == 0) groups[t] = line_word;
            } else if (lane < 4) {
                groups[(size_t)t * 4 + lane] = fine;
            }
        }
    }
    uint32_t before = 0, owner = 0;
    if (shared) {
        const uint32_t total = block_sum_u32(mine, s.wtot);     // valid on thread 0
        if (tid == 0) st_shared(&gcnt[b], total);
        // Last meeting.  From here on block 0 alone speaks for the row: the other blocks publish their count,
        // arrive and leave without waiting, so no block can pass this meeting while the one that would have
        // written the result gives up.  Block 0 either sees every count and walks the range that holds the
        // rank-th tie itself (1/B of the row), or its wait runs out and the caller repeats the search alone.
        ++meetings;
        if (b != 0) {
            slow_arrive(sync);
            return kFound;
        }
        if (!slow_meet(s.ok, sync, B * meetings, spin_limit)) return kGaveUp;
        clear_slow_hist(ghist, sync);
        if (tid < (uint32_t)kSlowMaxBlocks) s.part[tid] = tid < B ? ld_shared(&gcnt[tid]) : 0u;
        __syncthreads();
        owner = B;
        for (uint32_t q = 0; q < B; ++q) {                      // uniform for the block
            const uint32_t here = s.part[q];
            if (before < rank && rank <= before + here) {
                owner = q;
                break;
            }
            before += here;
        }
        if (owner == B) return kGaveUp;                         // counts that do not add up to the histogram: search alone
    }
    const uint32_t need = rank - before;
    const uint32_t w0 = min(owner * tpb, nwt), w1 = min(w0 + tpb, nwt);   // the owner's range of wave tiles
    if (tid == 0) s.cut = 0xffffffffu;
    __syncthreads();
    uint32_t seen = 0;
    for (uint32_t tb = w0; tb < w1; tb += 16) {                 // uniform trip count and exit
        const uint32_t t = tb + wave;
        uint64_t kb[4][4];
        uint32_t cnt = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            uint32_t key[4] = {0, 0, 0, 0};
            if (t < w1) slow_keys_at<VEC, RK>(g, d, k0, k1, j, key);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                kb[u][q] = __ballot(t < w1 && j + q < d && key[q] == prefix);
                cnt += (uint32_t)__popcll(kb[u][q]);
            }
        }
        if (lane == 0) s.wtot[wave] = cnt;
        __syncthreads();
        uint32_t below = seen, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < (int)wave) below += s.wtot[w];
            all += s.wtot[w];
        }
        if (below < need && need <= below + cnt) {              // uniform for the wave: the tie is in my tile
            uint32_t n = need - below;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t cu =
                    (uint32_t)(__popcll(kb[u][0]) + __popcll(kb[u][1]) + __popcll(kb[u][2]) + __popcll(kb[u][3]));
                if (n != 0 && n <= cu) {
                    const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
                    const uint32_t lb = lanes_below(kb[u][0]) + lanes_below(kb[u][1]) + lanes_below(kb[u][2]) +
                                        lanes_below(kb[u][3]);
                    uint32_t r = n > lb ? n - lb : 0u;           // 1-based rank among my own ties, 0: before me
                    uint32_t own = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if ((kb[u][q] >> lane) & 1) {
                            ++own;
                            if (own == r) s.cut = j + q;
                        }
                    }
                    n = 0;                                      // found in this chunk
                } else if (n != 0) {
                    n -= cu;
                }
            }
        }
        seen += all;
        __syncthreads();
        if (seen >= need) break;
    }
    __syncthreads();
    found = SlowFound{prefix, rank, ties, s.cut, s.bad, first};
    return kFound;
}

// Scratch of the kernels whose blocks share rows: slot y for the y-th row of a launch with B > 1 blocks a row.
struct SharedRows {
    uint32_t* hist;                            // [rows * kSlowHistWords] digit histograms of a general search
    uint32_t* cnt;                             // [rows * kSlowMaxBlocks] ties per block
    uint32_t* list_hist;                       // [rows * B * 256] first list digit per block
    uint32_t* sync;                            // [rows * kSyncWords]; arrivals and give-up flag zero when a step starts (see the update)
    uint32_t spin_limit;                       // bound, in polls, of the waits (those for a share of a list are shorter)
};

// The top-k rows in kSlow mode (long rows; k_select does it for short ones).
template <bool VEC>
__global__ __launch_bounds__(1024) void k_slow_select(const float* __restrict__ src, size_t row_stride, uint32_t d,
                                                       uint32_t nwt, uint32_t row0, RowDesc* __restrict__ desc, uint32_t k,
                                                       uint64_t* __restrict__ gbits, bool coarse, SharedRows sh) {
    __shared__ SlowLds s;
    const uint32_t row = row0 + blockIdx.y;
    if (desc[row].mode != kSlow) return;
    const float* __restrict__ g = src + (size_t)blockIdx.y * row_stride;
    SlowFound f;
    SlowEnd end = kGaveUp;
    if (gridDim.x > 1) {
        uint32_t* const sync = sh.sync + (size_t)blockIdx.y * kSyncWords;
        uint32_t meetings;
        end = slow_multi<VEC, false>(s, g, d, nwt, k, 0u, 0u, sh.hist + (size_t)blockIdx.y * kSlowHistWords,
                                     sh.cnt + (size_t)blockIdx.y * kSlowMaxBlocks, sync, sh.spin_limit,
                                     gbits + (size_t)blockIdx.y * nwt * (coarse ? 1 : 4), coarse, 0u, meetings, f);
        if (blockIdx.x != 0) return;
        if (end == kGaveUp && threadIdx.x == 0) sync[2] = 1;
    }
    if (end != kFound) f = slow_single<VEC, false>(s, g, d, k, 0u, 0u);
    if (threadIdx.x == 0) {
        s.now = desc[row];
        s.now.nonfinite_acc |= f.bad;
        const bool bitmap = end == kFound && bitmap_pays(f, k, d);
        finish_general(s.now, f, true, bitmap ? (coarse ? 2u : 1u) : 0u, 0u, 0u);
    }
    put_result(desc + row, s.now);
}

// Random-k: completes the kept bitmap of a row once (tau, cut-off) are known.  The first pass has set the
// bits of the columns whose key is above the band; here the listed candidates that are kept get
// theirs (atomic OR on the 32-bit word holding the lane's half-word).
__device__ __forceinline__ void mark_listed(const uint2* __restrict__ in, uint32_t n, uint32_t tau, uint32_t cut,
                                            uint32_t* __restrict__ words) {
    for (uint32_t base = threadIdx.x; base < n; base += 4 * kSelectBlock) {
        uint2 kv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) kv[i] = base + i * kSelectBlock < n ? in[base + i * kSelectBlock] : make_uint2(0u, 0u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (base + i * kSelectBlock < n && (kv[i].x > tau || (kv[i].x == tau && kv[i].y <= cut))) {
                const uint32_t t = kv[i].y / kWaveTile, o = kv[i].y % kWaveTile;
                const uint32_t u = o / kChunk, l = (o % kChunk) / 4, q = o % 4;
                const uint32_t half = t * 64 + l;                     // half-word of the row holding the column
                atomicOr(&words[half >> 1], 1u << ((half & 1) * 16 + 4 * u + q));
            }
        }
    }
}
// A row whose predicted band did not hold rank k: the first pass's bits are those of the wrong band.  Its priorities are
// computed again and whole half-words written, by block 0 (3 ms for 25.6M columns, two draws of 10^6 for k = 1 and far
// less often for larger k).
__device__ __forceinline__ void mark_row(uint64_t stream, uint32_t d, uint32_t nwt, uint32_t tau, uint32_t cut,
                                         uint16_t* __restrict__ row_bits) {
    const uint32_t k0 = (uint32_t)stream, k1 = (uint32_t)(stream >> 32), lane = threadIdx.x & 63;
    for (uint32_t t = threadIdx.x >> 6; t < nwt; t += kSelectBlock / 64) {
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t j = t * kWaveTile + u * kChunk + lane * 4 + q;
                const uint32_t key = rk_priority(k0, k1, j);
                m |= ((j < d && (key > tau || (key == tau && j <= cut))) ? 1u : 0u) << (4 * u + q);
            }
        row_bits[(size_t)t * 64 + lane] = (uint16_t)m;
    }
}

// ---------------------------------------------------------------------------------------------
// Everything that follows the pass over the predicted band, in one launch, for rows on which what a launch costs (2 us)
// counts: four launches of a steady-state top-k step become one.  grid = (B, rows), kSelectBlock threads.
// Block 0 finishes a row whose list holds rank k and is short; up to B blocks share a longer list's first digit (each
// leaves a histogram of its share, all add them up, and the entries of the digit's bin go to the row's short list); all B
// share the search of a row without a usable list: the first digit of the whole row, then a list of the entries of
// the bin that holds rank k, or, when those are too many, the rest of the general search.  Which of the three it is every
// block decides by itself from the mode, the band and the counters of the
// first pass, which this kernel leaves as they are: block 0 may have finished the row before another block starts.
// ---------------------------------------------------------------------------------------------
struct CollectLds {                            // the second pass of a row without a usable prediction
    uint2 stage[kStage], wstage[kSelectBlock / 64][kWaveStage];
    uint32_t wsure[kSelectBlock / 64 + 1], staged[2];
};
// Lists the entries of keys [lo, lo + 2^19) of this block's share of the row, for block 0, and leaves their group bitmap.
// (The kept bitmap of a random-k row is block 0's alone: a block that is still here when block 0's wait runs out, and
// block 0 searches and marks the row by itself, would put the bits of the keys above the band in place of finished ones.
// The group bitmap of a row that ends so is not used.)
template <bool VEC, bool RK>
__device__ __forceinline__ void collect_bin(CollectLds& s, const float* __restrict__ g, uint32_t d, uint32_t nwt, uint32_t lo,
                                            uint2* out, uint32_t cap, unsigned long long* counts, uint64_t* __restrict__ groups,
                                            bool coarse, uint64_t stream) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, B = gridDim.x;
    const uint32_t tpb = (nwt + B - 1) / B, t0 = min(blockIdx.x * tpb, nwt), t1 = min(t0 + tpb, nwt);
    FilterBand fb;
    fb.lo = lo;
    fb.hi = lo + (1u << 19);                                    // 0x80000000 for the top bin: no key reaches it
    fb.out = out;
    fb.cap = cap;
    fb.counts = counts;
    __syncthreads();                                            // what shared this memory is done
    if (tid < 2) s.staged[tid] = 0;
    __syncthreads();
    uint32_t n_hi = 0, kmax = 0, wcnt = 0;
    for (uint32_t t = t0 + wave; t < t1; t += kSelectBlock / 64) {
        uint32_t key[4][4];
        tile_keys<VEC, RK>(g, d, (uint32_t)stream, (uint32_t)(stream >> 32), t, lane, key);
        uint64_t line_word = 0, fine = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            uint64_t bc[4];
            uint32_t hi4;
            const uint64_t flags = filter_chunk<false, false>(key[u], j, d, fb.lo, fb.hi, bc, n_hi, kmax, hi4);
            line_word |= any_of_four_lanes(flags) << u;
            fine = lane == (uint32_t)u ? flags : fine;
            stage_candidates<true>(fb, key[u], j, bc, s.stage, s.wstage[wave], wcnt, s.staged, lane);
        }
        if (RK) continue;
        if (coarse) {
            if (lane == 0) groups[t] = line_word;
        } else if (lane < 4) {
            groups[(size_t)t * 4 + lane] = fine;
        }
    }
    finish_filter_block<kSelectBlock / 64, true>(fb, s.stage, s.wstage[wave], wcnt, 0u, s.staged, s.wsure);
}

template <bool VEC, bool RK>
__global__ __launch_bounds__(kSelectBlock) void k_select(RowDesc* __restrict__ desc, uint2* __restrict__ list, uint32_t d, uint32_t row0,
                                                          uint32_t cap, uint32_t k, uint32_t nwt, uint32_t short_cap,
                                                          uint2* __restrict__ shortl, bool coarse, const float* __restrict__ src,
                                                          size_t row_stride, RkDraw rk, uint64_t* __restrict__ gbits,
                                                          uint16_t* __restrict__ kbits, SharedRows sh) {
    __shared__ union {
        ListLds list;
        SlowLds slow;
        CollectLds collect;
    } s;
    __shared__ RowDesc now;
    __shared__ uint32_t met;
    const uint32_t row = row0 + blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const bool srv = RK && row == rk.srv_row;
    if (srv) k = rk.srv_k;
    const uint32_t fix_lo = srv ? rk.srv_lo : rk.fix_lo, fix_hi = srv ? rk.srv_hi : rk.fix_hi;
    // What the row needs follows from words of its descriptor that stay as they are, in scalar registers; the whole of it, a word a
    // thread until it has arrived, is for thread 0 at the end.
    RowDesc seen;
    seen.mode = ld_const(&desc[row].mode);
    seen.lo = ld_const(&desc[row].lo);
    seen.hi = ld_const(&desc[row].hi);
    seen.n_cand = ld_const(&desc[row].n_cand);
    seen.n_sure = ld_const(&desc[row].n_sure);
    const uint32_t desc_word = tid < 64 ? reinterpret_cast<const uint32_t*>(desc + row)[tid] : 0u;
    const uint32_t form = RK ? 0u : coarse ? 2u : 1u;
    uint16_t* const row_bits = RK ? kbits + (size_t)row * nwt * 64 : nullptr;
    const uint64_t stream = RK ? rk_stream(rk.state->seed, rk.state->draw, row) : 0ull;
    uint2* const row_list = list + (size_t)row * cap;
    uint32_t* const sync = sh.sync + (size_t)blockIdx.y * kSyncWords;
    const RowWork work = row_work(seen, cap, k);                // the same in every block of the row, however late it starts
    const bool cold = work.cold;
    uint32_t lo = work.lo, width = work.width, n = work.n, rank = work.rank;
    auto keep_desc = [&] {
        if (tid < 64) reinterpret_cast<uint32_t*>(&now)[tid] = desc_word;
    };
    if (cold) {
        keep_desc();
        const float* __restrict__ g = src + (size_t)blockIdx.y * row_stride;
        uint64_t* const groups = gbits ? gbits + (size_t)blockIdx.y * nwt * (coarse ? 1 : 4) : nullptr;
        SlowFound f{0, 0, 0, 0, 0, 0};
        uint32_t* const hist = sh.hist + (size_t)blockIdx.y * kSlowHistWords;
        uint32_t meetings;
        // (a caller can send a row through the whole of the general search)
        SlowEnd end = slow_multi<VEC, RK>(s.slow, g, d, nwt, k, (uint32_t)stream, (uint32_t)(stream >> 32), hist,
                                          sh.cnt + (size_t)blockIdx.y * kSlowMaxBlocks, sync, sh.spin_limit, groups, coarse,
                                          seen.mode == kSlow ? 0u : cap, meetings, f);
        if (end == kListed) {                                   // every block of the row
            collect_bin<VEC, RK>(s.collect, g, d, nwt, f.tau << 19, row_list, cap,
                                 reinterpret_cast<unsigned long long*>(&desc[row].n_cand2), groups, coarse, stream);
            if (blockIdx.x != 0) {
                slow_arrive(sync);
                return;
            }
            if (gridDim.x == 1) slow_written();
            else if (slow_meet(met, sync, gridDim.x * (meetings + 1), sh.spin_limit)) clear_slow_hist(hist, sync);
            else end = kGaveUp;
        }
        if (blockIdx.x != 0) return;
        if (end == kGaveUp && tid == 0) sync[2] = 1;            // (a block on its own never gives up)
        if (end == kGaveUp) f = slow_single<VEC, RK>(s.slow, g, d, k, (uint32_t)stream, (uint32_t)(stream >> 32));
        if (tid == 0) {
            now.misses += now.mode == kWarm ? 1u : 0u;          // there was a prediction and it failed
            now.nonfinite_acc |= f.bad;
        }
        if (end != kListed) {
            const bool bitmap = end == kFound && groups && bitmap_pays(f, k, d);
            if (tid == 0) finish_general(now, f, now.mode == kSlow || f.first > cap, bitmap ? form : 0u, fix_lo, fix_hi);
            put_result(desc + row, now);
            if (RK) mark_row(stream, d, nwt, f.tau, f.cut, row_bits);
            return;
        }
        lo = f.tau << 19;
        width = 1u << 19;
        n = f.first;
        rank = f.rank;
    }
    const uint2* in = row_list;
    uint32_t n_in = n;
    const uint32_t nb = !cold && n > (uint32_t)kDirectList ? list_blocks_for(n, gridDim.x) : 1u;
    if (blockIdx.x >= nb) return;
    bool first = true;
    Pick ph{0, 0, 0};
    const int shift = first_shift(width, kFirstBits);
    if (nb > 1) {
        uint32_t* const h = s.list.h_long;
        uint32_t* const hists = sh.list_hist + (size_t)blockIdx.y * gridDim.x * 256;
        if (tid < 256) h[tid] = 0;
        __syncthreads();
        for (uint32_t base = blockIdx.x * kSelectBlock; base < n; base += nb * kSelectBlock) {    // uniform for the block
            const uint32_t e = base + tid;
            wave_count(h, e < n, ((e < n ? row_list[e].x : lo) - lo) >> shift, lane);
        }
        __syncthreads();
        if (tid < 256) st_shared(&hists[blockIdx.x * 256 + tid], h[tid]);
        const bool ok = slow_meet(met, sync, nb, list_wait(sh.spin_limit, n));
        if (!ok && blockIdx.x != 0) return;
        if (ok) {
            uint32_t sum = 0;
            for (uint32_t b = tid >> 8; b < nb; b += kSelectBlock / 256) sum += ld_shared(&hists[b * 256 + (tid & 255)]);
            if (tid < 256) h[tid] = 0;
            __syncthreads();
            if (sum) atomicAdd(&h[tid & 255], sum);
            __syncthreads();
            ph = block_pick(h, 256, rank, s.list.part, s.list.res);
            if (ph.count > short_cap) {                         // too many for the short list: block 0 walks the list
                if (blockIdx.x != 0) return;
                first = false;
            } else {
                // where my entries go follows from the histograms (with an atomic on the row's counter for every wave that has
                // some, one after another, and bins of at most 4096: 2 x 4.2M columns, 5 %, a step 90 -> 82 us)
                static_assert(kSlowMaxBlocks <= 64, "a lane for every block");
                if (tid < 64) {
                    const uint32_t ahead = wave_sum(lane < blockIdx.x ? ld_shared(&hists[lane * 256 + ph.bin]) : 0u);
                    if (tid == 0) s.list.nties = ahead;
                }
                __syncthreads();
                uint2* const out = shortl + (size_t)row * short_cap;
                for (uint32_t base = blockIdx.x * kSelectBlock; base < n; base += nb * kSelectBlock) {
                    const uint32_t e = base + tid;
                    const uint2 kv = e < n ? row_list[e] : make_uint2(0u, 0u);
                    const bool hit = e < n && ((kv.x - lo) >> shift) == ph.bin;
                    const uint64_t m = __ballot(hit);
                    if (m) {                                    // wave-uniform
                        uint32_t at = 0;
                        if (lane == 0) at = atomicAdd(&s.list.nties, (uint32_t)__popcll(m));       // LDS
                        at = __builtin_amdgcn_readfirstlane(at);
                        if (hit) put_entry<true>(&out[at + lanes_below(m)], kv);      // the bin's count bounds the total: at most short_cap
                    }
                }
                if (blockIdx.x != 0) {
                    slow_arrive(sync);
                    return;
                }
                if (slow_meet(met, sync, 2 * nb, list_wait(sh.spin_limit, n))) {
                    first = false;
                    in = out;
                    n_in = ph.count;
                }
            }
        }
    }
    __syncthreads();
    if (!cold) keep_desc();
    select_listed<true>(s.list, in, n_in, lo, width, rank, first, ph, shift, d, cold || in != row_list);
    if (tid == 0) {
        if (RK) finish_listed(now, found_in(s.list), n, form, cold, 0u, fix_lo, fix_hi);
        else record_listed(now, found_in(s.list), n, form, cold, 0u);
    }
    put_result(desc + row, now);
    if (RK) {
        if (cold) mark_row(stream, d, nwt, s.list.tau, s.list.cut, row_bits);
        else mark_listed(row_list, n, s.list.tau, s.list.cut, reinterpret_cast<uint32_t*>(row_bits));
    }
}

}  // namespace liec
