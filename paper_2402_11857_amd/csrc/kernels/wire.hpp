// Wire forms of the compressed messages.
#pragma once
#include "common.hpp"
#include "sign.hpp"

namespace liec {

// ---------------------------------------------------------------------------------------------
// Wire form of a (blockwise) scaled-sign message: one bit per element, bit j % 8 of byte j / 8 set
// when the element is negative.  k_pack_sign turns one row of the lane-major bitmap into that
// form (a thread turns the 16 bytes of 8 lanes into four 32-bit words, one per chunk; one thread per output byte
// took 4.7 us for 1.5 MB, this 2.9); k_unpack_sign expands wire bits and scale(s) into the dense
// message p_j = -s or +s (one 128-bit streaming store per 4 columns: 8 messages of 11.7M columns packed and unpacked
// took 125 us with plain stores, 98 with streaming ones, 94 with larger blocks).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_pack_sign(const uint16_t* __restrict__ row_bits, uint32_t nwt, uint32_t nbytes,
                                                       uint8_t* __restrict__ out) {
    typedef uint32_t u32_any __attribute__((aligned(1)));
    const uint32_t q = blockIdx.x * kBlock + threadIdx.x;      // 8 lanes' half-words of one wave tile
    if (q >= nwt * 8) return;
    const uint4 w = reinterpret_cast<const uint4*>(row_bits)[q];
    const uint32_t h[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {                               // their 32 columns of chunk u
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) m |= (((h[i] >> (4 * u)) & 0xfu) | ((h[i] >> (16 + 4 * u)) & 0xfu) << 4) << (8 * i);
        const uint32_t b = (q >> 3) * (kWaveTile / 8) + u * (kChunk / 8) + (q & 7) * 4;
        if (b + 4 <= nbytes) {
            *reinterpret_cast<u32_any*>(out + b) = m;           // the caller's buffer may start at any byte
        } else {
            for (uint32_t i = 0; b + i < nbytes; ++i) out[b + i] = (uint8_t)(m >> (8 * i));
        }
    }
}

template <bool VEC>
__global__ __launch_bounds__(1024) void k_unpack_sign(const uint8_t* __restrict__ bytes, uint32_t d,
                                                         const float* __restrict__ scales, float scale0,
                                                         BlockTable bt, float* __restrict__ p) {
    const uint32_t nq = (d + 3) / 4;                            // groups of 4 columns = half a wire byte
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nq; q += gridDim.x * blockDim.x) {
        const uint32_t j0 = q * 4;
        const uint32_t m = (uint32_t)bytes[q >> 1] >> (4 * (q & 1u));
        float v[4];
        if (bt.B) {
            const uint32_t tb = bt.tile_blk[j0 / kColTile], first = tb & 0x7fffffffu;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t j = j0 + c < d ? j0 + c : d - 1;
                const float s = scales[(tb >> 31) ? block_of(bt, first, j) : first];
                v[c] = ((m >> c) & 1u) ? -s : s;
            }
        } else {
            const float s = scale0;                             // Definition 4: one scale, passed by value
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = ((m >> c) & 1u) ? -s : s;
        }
        st4<VEC, true>(p, j0, d, make_float4(v[0], v[1], v[2], v[3]));
    }
}

// ---------------------------------------------------------------------------------------------
// Wire form of a top-k or random-k message: the kept entries of one row as (index, value) pairs in increasing index
// order.  Two kernels over the same blocks, each owning `per` consecutive wave tiles: k_kept_count leaves the kept
// entries of every tile and block, k_kept_emit adds up the counts before its own tiles and writes the pairs.  Inside
// a wave tile the order is chunk, then lane, then component.  What is kept follows from what the step left behind:
// the candidate bitmap (top-k: only the flagged groups of columns are fetched and compared with the threshold) or
// the kept bitmap (random-k: the count reads no gradients at all).  Count and emit, against a count and an emit that read
// the whole row and a one-block scan of the tiles between them (us): 11.7M columns, k = 1 %, 5 + 9, 10 + 11 + 8; 60M
// columns, 1 %, 13 + 24, 35 + 37 + 35, and all columns kept, 69 + 215, 64 + 186 + 36; 8.4M columns of one magnitude, which
// have no bitmap, 1.25 %, 7 + 7, 6 + 7 + 6.
// ---------------------------------------------------------------------------------------------
// At most so many blocks; every block of k_kept_emit adds up the counts of those ahead of it.  No row (d < 2^31) has more
// than kBlock tiles to a block, one per thread of k_kept_emit.  With 4096: 60M columns 16 + 29 and 72 + 230 us; with 2048
// 11.7M columns 7 + 13.
constexpr uint32_t kWireBlocks = 8192;
static_assert((uint64_t)kWireBlocks * kBlock * kWaveTile >= (1ull << 31), "a block's tiles have a thread each");
struct KeptRow {
    const float* g;                                             // the row's gradients
    const RowDesc* rd;
    const uint64_t* groups;                                     // top-k: the workers' candidate bitmaps
    uint32_t worker;                                            // and the row's number
    const uint16_t* kept;                                       // random-k: the row's kept bitmap
};
// Ballots of the kept columns of tile t: kb[u][q] for component q of chunk u.  VALUES: also the gradients of the
// groups of 4 columns that hold one (a[u], valid where a bit of kb[u] is set).  False when the tile keeps nothing.
template <bool VEC, bool VALUES>
__device__ __forceinline__ bool kept_ballots(const KeptRow& r, uint32_t t, uint32_t lane, uint32_t d, uint32_t nwt, uint32_t tau,
                                             uint32_t cut, uint32_t form, float4 (&a)[4], uint64_t (&kb)[4][4]) {
    const uint32_t j0 = t * kWaveTile + lane * 4;
    if (r.kept) {                                               // uniform
        const uint32_t m = r.kept[(size_t)t * 64 + lane];
        if (__ballot(m != 0) == 0) return false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (VALUES && ((m >> (4 * u)) & 0xfu)) a[u] = ld4<VEC>(r.g, j0 + u * kChunk, d);
#pragma unroll
            for (int q = 0; q < 4; ++q) kb[u][q] = __ballot((m >> (4 * u + q)) & 1u);
        }
        return true;
    }
    uint32_t mask = 0xfu;                                       // bit u: my group of chunk u may hold a kept column
    if (form) {                                                 // uniform
        const size_t at = (size_t)r.worker * nwt + t;
        if (form == 2) {
            mask = (uint32_t)(r.groups[at] >> (4 * (lane >> 2))) & 0xfu;
        } else {
            const uint64_t* __restrict__ w = r.groups + at * 4;
            mask = (uint32_t)((w[0] >> lane) & 1) | (uint32_t)((w[1] >> lane) & 1) << 1 | (uint32_t)((w[2] >> lane) & 1) << 2 |
                   (uint32_t)((w[3] >> lane) & 1) << 3;
        }
        if (__ballot(mask != 0) == 0) return false;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if ((mask >> u) & 1u) a[u] = ld4<VEC>(r.g, j0 + u * kChunk, d);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t j = j0 + u * kChunk;
        const float av[4] = {a[u].x, a[u].y, a[u].z, a[u].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t key = key_of(av[q]);
            kb[u][q] = __ballot(((mask >> u) & 1u) && j + q < d && (key > tau || (key == tau && j + q <= cut)));
        }
    }
    return true;
}

template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_kept_count(KeptRow r, uint32_t d, uint32_t nwt, uint32_t per,
                                                        uint32_t* __restrict__ tile_cnt, uint32_t* __restrict__ block_cnt) {
    __shared__ uint32_t lds_w[4];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t tau = r.rd->tau, cut = r.rd->cutoff;
    const uint32_t form = r.rd->form;                           // of the bitmap, 0: look at every column
    const uint32_t t0 = blockIdx.x * per, t1 = min(t0 + per, nwt);
    uint32_t total = 0;
    for (uint32_t t = t0 + wave; t < t1; t += 4) {
        float4 a[4];
        uint64_t kb[4][4];
        uint32_t n = 0;
        if (kept_ballots<VEC, false>(r, t, lane, d, nwt, tau, cut, form, a, kb)) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) n += __popcll(kb[u][q]);
        }
        if (lane == 0) tile_cnt[t] = n;
        total += n;
    }
    if (lane == 0) lds_w[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) block_cnt[blockIdx.x] = lds_w[0] + lds_w[1] + lds_w[2] + lds_w[3];
}

template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_kept_emit(KeptRow r, uint32_t d, uint32_t nwt, uint32_t per,
                                                       const uint32_t* __restrict__ tile_cnt,
                                                       const uint32_t* __restrict__ block_cnt, uint32_t k,
                                                       uint32_t* __restrict__ idx_out, float* __restrict__ val_out) {
    __shared__ uint32_t wave_before[4], wave_n[4], first[kBlock];
    const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const uint32_t tau = r.rd->tau, cut = r.rd->cutoff;
    const uint32_t form = r.rd->form;
    const bool all = !r.kept && form == 0;                      // uniform: neither bitmap
    // kept entries in the blocks ahead of this one: the first 4096 counts requested at once (one after another they cost
    // this kernel half its time)
    constexpr int kLoads = 4;
    uint4 c[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const uint32_t b = (q * kBlock + tid) * 4;
        c[q] = b < blockIdx.x ? *reinterpret_cast<const uint4*>(block_cnt + b) : make_uint4(0u, 0u, 0u, 0u);
    }
    const uint32_t t0 = blockIdx.x * per, t1 = min(t0 + per, nwt);     // at most kBlock tiles
    const uint32_t n = t0 + tid < t1 ? tile_cnt[t0 + tid] : 0u;
    float4 a[4];
    uint64_t kb[4][4];
    // a row without a valid bitmap is not read where it keeps nothing
    auto look = [&](uint32_t t) {
        return (!all || tile_cnt[t] != 0) && kept_ballots<VEC, true>(r, t, lane, d, nwt, tau, cut, form, a, kb);
    };
    uint32_t t = t0 + wave;
    bool any = t < t1 && look(t);                               // (its loads run beside the sums)
    auto count4 = [&](uint4 v, uint32_t b) {
        return (b < blockIdx.x ? v.x : 0u) + (b + 1 < blockIdx.x ? v.y : 0u) + (b + 2 < blockIdx.x ? v.z : 0u) +
               (b + 3 < blockIdx.x ? v.w : 0u);
    };
    uint32_t before = 0;
#pragma unroll
    for (int q = 0; q < kLoads; ++q) before += count4(c[q], (q * kBlock + tid) * 4);
    for (uint32_t b = (kLoads * kBlock + tid) * 4; b < blockIdx.x; b += kBlock * 4)     // rows of more than 16.8M columns
        before += count4(*reinterpret_cast<const uint4*>(block_cnt + b), b);
    const uint32_t incl = wave_scan(n);
    before = wave_sum(before);
    if (lane == 63) {
        wave_before[wave] = before;
        wave_n[wave] = incl;
    }
    __syncthreads();
    uint32_t ahead = wave_before[0] + wave_before[1] + wave_before[2] + wave_before[3];
    for (uint32_t w = 0; w < wave; ++w) ahead += wave_n[w];
    first[tid] = ahead + incl - n;
    __syncthreads();
    for (; t < t1; t += 4) {
        if (t >= t0 + 4) any = look(t);
        if (!any) continue;
        uint32_t at = first[t - t0];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            const float av[4] = {a[u].x, a[u].y, a[u].z, a[u].w};
            // entries of lower lanes come first, then this lane's lower components
            uint32_t pos = at + lanes_below(kb[u][0]) + lanes_below(kb[u][1]) + lanes_below(kb[u][2]) + lanes_below(kb[u][3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if ((kb[u][q] >> lane) & 1) {
                    if (pos < k) {
                        idx_out[pos] = j + q;
                        val_out[pos] = av[q];
                    }
                    ++pos;
                }
            }
            at += __popcll(kb[u][0]) + __popcll(kb[u][1]) + __popcll(kb[u][2]) + __popcll(kb[u][3]);
        }
    }
}

// Dense vector from (index, value) pairs: the caller zero-fills p first.
__global__ __launch_bounds__(kBlock) void k_scatter_pairs(const uint32_t* __restrict__ idx, const float* __restrict__ val,
                                                           uint32_t k, uint32_t d, float* __restrict__ p) {
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r < k && idx[r] < d) p[idx[r]] = val[r];
}

// One 128-bit streaming store per thread (8 top-k messages of 11.7M columns, packed and unpacked: 268 us, with plain
// stores 293).
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_clear_f32(float* __restrict__ p, uint32_t n) {
    const uint32_t j = (blockIdx.x * kBlock + threadIdx.x) * 4;
    if (j < n) st4<VEC, true>(p, j, n, make_float4(0.f, 0.f, 0.f, 0.f));
}

}  // namespace liec
