// Shared pieces of the LIEC-SGD device kernels for gfx950 (CDNA4, wave64): constants, the per-row
// descriptor, the random-k generator, 128-bit accessors, block reductions and the histogram walk.
//
// Element ownership in the streaming kernels: a wave walks "wave tiles" of 1024 consecutive
// columns (4 chunks of 256); in chunk u, lane l owns columns 256u + 4l .. 256u + 4l + 3 (one
// 128-bit access per lane, 1 KiB contiguous per wave and instruction).  A block of 256 threads
// (4 waves) covers 4096 consecutive columns per iteration.  All fp32 arithmetic that reaches the
// outputs is written as single IEEE operations (__fadd_rn / __fsub_rn / __fmaf_rn) so that the
// result does not depend on compiler contraction.  Streams that are read or written once are
// accessed with non-temporal hints.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include "rows.hpp"

namespace liec {

constexpr int kBlock = 256;             // threads per block (4 waves)
constexpr int kChunk = 256;             // columns per wave and load instruction
constexpr int kWaveTile = 1024;         // columns per wave iteration
constexpr int kColTile = 1024;          // columns per block of the update kernel
constexpr int kHistBins = 4096;         // first radix digit of a whole row (12 bits)
constexpr int kListBins = 1 << kListBits;
constexpr int kStage = 1024;            // LDS staging slots of a block of the candidate filter
constexpr int kWaveStage = 256;         // and of each of its waves once the block's are used up (a chunk lists at most 256)
constexpr int kDirectList = 16384;      // candidate lists up to this length are selected by one block on its own
constexpr int kShortCap = 4096;         // entries of the first list digit's bin that are handed to the list select on their own
constexpr uint32_t kShortCapOne = 16384;     // the same where one launch does the search: as many as one block holds in LDS
constexpr int kHeldBits = 8;            // radix digit of the list select over a list it holds in LDS
constexpr int kIndexBits = 11;          // its radix digit over the indices of entries that share one key, of a longer list
constexpr uint32_t kFewHeld = 128;      // entries left that the list select compares with one another instead of taking further digits,
constexpr uint32_t kFewEntries = 256;   // and of a list it does not hold
constexpr uint32_t kUpdatePanel = 4096; // column tiles per panel of the update kernel

enum Comp : int { kIdentity = 0, kSign = 1, kTopk = 2, kBlockSign = 3, kRandk = 4 };

// Radix digits of the 31-bit magnitude key, most significant first.
__host__ __device__ constexpr int digit_shift(int pass) { return pass == 0 ? 19 : (pass == 1 ? 9 : 0); }
__host__ __device__ constexpr int digit_bits(int pass) { return pass == 0 ? 12 : (pass == 1 ? 10 : 9); }

__device__ __forceinline__ uint32_t key_of(float v) { return __float_as_uint(v) & 0x7fffffffu; }
constexpr uint32_t kInfKey = 0x7f800000u;                       // keys of Inf and NaN start here
__device__ __forceinline__ bool any_nonfinite(float a, float b, float c, float d) {
    return max(max(key_of(a), key_of(b)), max(key_of(c), key_of(d))) >= kInfKey;
}

// ---------------------------------------------------------------------------------------------
// Random-k (Definition 3): the k-subset is drawn by giving index j the priority
// rk_priority(stream, j) and keeping the k highest (ties, at most pairs, to the lower index), so the
// draw is a top-k search over keys that do not depend on the data.  `stream` is one 64-bit word per
// (seed, draw, row): three rounds of a multiply-xorshift finalizer over seed, draw counter and row
// (worker index, or N for the server).  The per-index part is a keyed permutation of 32-bit words
// (every step is a bijection) with its lowest bit dropped: a 31-bit key like a magnitude key.
// ---------------------------------------------------------------------------------------------
struct RkState {               // in device memory, so that a captured step draws anew on every replay
    uint64_t seed, draw;       // draw: number of the draw the next step makes
};
struct RkDraw {
    const RkState* state = nullptr;
    uint32_t fix_lo = 0, fix_hi = 0;   // band that holds rank k of uniform priorities (set by the host); fix_hi == 0: not random-k
    // random-k on both sides: the server's draw, which no gradient enters, is one more row of the workers' launches, with
    // a k and a band of its own
    uint32_t srv_row = 0xffffffffu, srv_k = 0, srv_lo = 0, srv_hi = 0;
};

__host__ __device__ __forceinline__ uint64_t rk_mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__host__ __device__ __forceinline__ uint64_t rk_stream(uint64_t seed, uint64_t draw, uint32_t row) {
    const uint64_t gamma = 0x9E3779B97F4A7C15ull;
    uint64_t z = rk_mix64(seed + gamma);
    z = rk_mix64(z + draw + gamma);
    return rk_mix64(z + (uint64_t)row + gamma);
}
__host__ __device__ __forceinline__ uint32_t rk_priority(uint32_t k0, uint32_t k1, uint32_t j) {
    uint32_t h = j ^ k0;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h += k1;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h >> 1;
}

// 128 bits at any multiple of 16 bytes (VEC: the row starts there and its length is a multiple of 4) or of 4 bytes.
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
template <bool VEC>
struct Vec4 {
    typedef v4f type;
};
template <>
struct Vec4<false> {
    typedef v4f_any type;
};

// 4 consecutive floats starting at column j of a row of length d; zero beyond d.
// Rows that start at any multiple of 4 bytes (VEC false) take the same 128-bit instructions: global memory serves
// them at any 4-byte address, and a wave still touches 1 KiB in one piece, one cache line more than when aligned.
// Only the group of columns that holds the end of such a row goes element by element.  Against four 32-bit accesses
// per group, which issue four times the memory instructions for the same lines: the update of 8 rows of 11.7M + 2
// columns 373 -> 195 us (3.0 -> 5.8 TB/s; an aligned row runs at 6.0), the top-k filter of 5 rows of 3M + 1 27 -> 16 us.
template <bool VEC, bool NT = false>
__device__ __forceinline__ float4 ld4(const float* __restrict__ row, uint32_t j, uint32_t d) {
    typedef typename Vec4<VEC>::type vec;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (VEC ? j < d : j + 3 < d) {
        const vec t = NT ? __builtin_nontemporal_load(reinterpret_cast<const vec*>(row + j)) : *reinterpret_cast<const vec*>(row + j);
        r = make_float4(t.x, t.y, t.z, t.w);
    } else if (!VEC) {
        if (j < d) r.x = row[j];
        if (j + 1 < d) r.y = row[j + 1];
        if (j + 2 < d) r.z = row[j + 2];
    }
    return r;
}

// The 16 columns of this lane of a whole wave tile (all of them below d), as streaming loads unless NT is false.  No branch stands around the
// accesses: with the one that ld4 needs at the end of a row off a 16-byte boundary, the compiler does not keep a wave's four
// loads together.  7 x 7.3M + 1 columns: first pass of scaled sign 40.5 -> 35.9 us (as aligned rows), blockwise 42.9 -> 36.9;
// the update and the averaging kernels, one load of a kind at a time, gain nothing by it.
template <bool VEC, bool NT = true>
__device__ __forceinline__ void ld_tile(const float* __restrict__ row, uint32_t t, uint32_t lane, float4 (&a)[4]) {
    typedef typename Vec4<VEC>::type vec;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const vec* const p = reinterpret_cast<const vec*>(row + (size_t)t * kWaveTile + u * kChunk + lane * 4);
        const vec w = NT ? __builtin_nontemporal_load(p) : *p;
        a[u] = make_float4(w.x, w.y, w.z, w.w);
    }
}

template <bool VEC, bool NT = false>
__device__ __forceinline__ void st4(float* __restrict__ row, uint32_t j, uint32_t d, float4 v) {
    typedef typename Vec4<VEC>::type vec;
    if (VEC ? j < d : j + 3 < d) {
        const vec t = {v.x, v.y, v.z, v.w};
        if (NT) __builtin_nontemporal_store(t, reinterpret_cast<vec*>(row + j));
        else *reinterpret_cast<vec*>(row + j) = t;
    } else if (!VEC) {
        if (j < d) row[j] = v.x;
        if (j + 1 < d) row[j + 1] = v.y;
        if (j + 2 < d) row[j + 2] = v.z;
    }
}

// A value that no block of the running kernel writes: with an address that is the same for the whole wave it comes through the scalar
// cache into scalar registers, also in loops that store elsewhere.
template <typename T>
__device__ __forceinline__ T ld_const(const T* p) {
    return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}
__device__ __forceinline__ float lane_value(float v, uint32_t lane) {     // lane: the same for the whole wave
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), (int)lane));
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {   // set bits of mask below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Histogram step of a whole wave (call it in wave-uniform control flow): adds one to LDS bin `bin` for every
// lane with `valid`.  When all of them name the same bin -- a degenerate row puts whole waves on one
// magnitude -- the wave issues one atomic instead of serialising 64 on one address.
__device__ __forceinline__ void wave_count(uint32_t* h, bool valid, uint32_t bin, uint32_t lane) {
    const uint32_t bin0 = __builtin_amdgcn_readfirstlane(bin);
    const uint64_t act = __ballot(valid);
    if (__ballot(valid && bin != bin0) == 0) {
        if (lane == 0 && act) atomicAdd(&h[bin0], (uint32_t)__popcll(act));
    } else if (valid) {
        atomicAdd(&h[bin], 1u);
    }
}

// Sums over the wave in a fixed order; all 64 lanes call them.  The lanes' values move through the vector
// unit's own data path (inside rows of 16 lanes, then from row to row), a few cycles a step where a shuffle through LDS
// takes a hundred (scaled sign, four such sums in a row: 8 x 262144 columns 16.1 -> 15.3 us a step).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint64_t lo = dpp_or_zero<CTRL, ROWS>((uint32_t)b), hi = dpp_or_zero<CTRL, ROWS>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(hi << 32 | lo));
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ double last_lane(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)((uint64_t)last_lane((uint32_t)(b >> 32)) << 32 | last_lane((uint32_t)b)));
}
// Sum of the lanes up to and including this one.
template <typename T>
__device__ __forceinline__ T wave_scan(T v) {
    v += dpp_or_zero<0x111, 0xf>(v);           // row_shr:1, 2, 4, 8: lane 15 of a row has the row's sum
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);           // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xc>(v);           // row_bcast:31 into rows 2 and 3
    return v;
}
template <typename T>
__device__ __forceinline__ T wave_sum(T v) { return last_lane(wave_scan(v)); }

// Sum over the block in a fixed order (wave_sum, then waves in order).  Valid on thread 0.
__device__ __forceinline__ double block_sum_f64(double v, double* lds_waves) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (lane == 0) lds_waves[wave] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < nw; ++w) r += lds_waves[w];
    return r;
}

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* lds_waves) {
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (lane == 0) lds_waves[wave] = v;
    __syncthreads();
    uint32_t r = 0;
    if (threadIdx.x == 0)
        for (int w = 0; w < nw; ++w) r += lds_waves[w];
    return r;
}

// Walks a histogram of nbins (a power of two from 256 to 8192) counts from the top bin down to the bin that
// holds the entry of rank `rank` (1-based, largest first).  Needs blockDim.x >= 256; every thread
// of the block must call it.  part: 256 words of LDS, res: 3 words of LDS.
// Thread t < 256 adds up the nbins / 256 consecutive bins t * per .. t * per + per - 1, starting at a bin of its
// own ((q + t) mod per: neighbouring threads then read different LDS banks -- read in the same order, the 32
// bins per thread of an 8192-bin histogram all fell on one bank and the pick took 4 us); a suffix sum over the
// threads finds the one whose bins hold the rank, and one wave walks that thread's bins.
struct Pick {
    uint32_t bin, rank_in, count;
};
__device__ __forceinline__ Pick block_pick(const uint32_t* __restrict__ h, int nbins, uint32_t rank,
                                           uint32_t* part, uint32_t* res) {
    const int per = nbins >> 8;   // 1 .. 32 bins per thread, a power of two
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t sum = 0;
    if (tid < 256) {
#pragma unroll 8
        for (int q = 0; q < per; ++q) sum += h[tid * per + ((q + tid) & (per - 1))];
    }
    // count in the bins above this thread's range: suffix sum over the 256 threads (lanes, then waves)
    const uint32_t upto = wave_scan(sum), incl = last_lane(upto) - upto + sum;
    if (tid < 256 && lane == 0) part[wave] = incl;             // total of wave `wave`
    if (tid == 0) {
        part[8] = 0xffffffffu;                                  // the thread whose bins hold the rank: none yet
        res[0] = 0;
        res[1] = 1;
        res[2] = 0;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t above = incl - sum;
        for (uint32_t w = wave + 1; w < 4; ++w) above += part[w];
        if (above < rank && rank <= above + sum) {   // true for at most one thread
            part[8] = tid;
            part[9] = above;
        }
    }
    __syncthreads();
    const uint32_t owner = part[8];
    if (owner != 0xffffffffu && tid < 64) {                     // wave 0 walks the owner's bins from the top
        const uint32_t above = part[9];
        const uint32_t c = (int)lane < per ? h[owner * per + lane] : 0u;
        const uint32_t upto_me = wave_scan(c), suf = last_lane(upto_me) - upto_me + c;      // sum over the lanes at and above mine
        const uint64_t reach = __ballot((int)lane < per && above + suf >= rank);    // lane 0 always does
        const uint32_t top = 63u - (uint32_t)__clzll((long long)reach);
        if (lane == top) {
            res[0] = owner * per + lane;
            res[1] = rank - (above + suf - c);
            res[2] = c;
        }
    }
    __syncthreads();
    Pick p;
    p.bin = res[0];
    p.rank_in = res[1];
    p.count = res[2];
    __syncthreads();
    return p;
}

}  // namespace liec
