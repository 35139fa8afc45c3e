// Scaled sign (Definition 4) and its blockwise form (Definition 5): L1 norms in fp64 and sign bits.
#pragma once
#include "common.hpp"

namespace liec {

// ---------------------------------------------------------------------------------------------
// Scaled sign, worker side (Definition 4): per-row partial sums of |g| in fp64 and the sign bits
// of the row.  Bit layout ("lane-major"): wave tile t of row i owns 64 half-words
// bits[(i*nwt + t)*64 + l]; bit 4u + q of half-word l is (g[1024t + 256u + 4l + q] < 0), i.e. every
// lane keeps the 16 bits of the 16 columns it owns, and a wave reads or writes 128 contiguous bytes.
// grid = (blocks per row, rows), blocks of 4 or 16 waves; waves stride over the row's wave tiles.
// ---------------------------------------------------------------------------------------------
template <bool VEC>
__global__ __launch_bounds__(1024) void k_l1_bits(const float* __restrict__ src, size_t row_stride, uint32_t d,
                                                     uint32_t nwt, double* __restrict__ partial,
                                                     uint16_t* __restrict__ bits) {
    __shared__ double lds_w[16];
    const uint32_t row = blockIdx.y;
    const float* __restrict__ g = src + (size_t)row * row_stride;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    double acc = 0.0;
    for (uint32_t t = blockIdx.x * waves + wave; t < nwt; t += gridDim.x * waves) {
        float4 a[4];
        if ((t + 1) * (uint32_t)kWaveTile <= d) {               // wave-uniform
            ld_tile<VEC>(g, t, lane, a);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = ld4<VEC, true>(g, t * kWaveTile + u * kChunk + lane * 4, d);
        }
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            acc += (double)fabsf(a[u].x);
            acc += (double)fabsf(a[u].y);
            acc += (double)fabsf(a[u].z);
            acc += (double)fabsf(a[u].w);
            m |= (a[u].x < 0.f ? 1u : 0u) << (4 * u);
            m |= (a[u].y < 0.f ? 1u : 0u) << (4 * u + 1);
            m |= (a[u].z < 0.f ? 1u : 0u) << (4 * u + 2);
            m |= (a[u].w < 0.f ? 1u : 0u) << (4 * u + 3);
        }
        // streaming hint on the bits store: 3.5 % faster than a plain store (the store still costs this
        // pass a fifth of its time: without it the kernel reads at 6.8 TB/s)
        __builtin_nontemporal_store((uint16_t)m, &bits[((size_t)row * nwt + t) * 64 + lane]);
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // let the small store land before the next loads (~2 % faster)
#endif
    }
    const double s = block_sum_f64(acc, lds_w);
    if (threadIdx.x == 0) partial[(size_t)row * gridDim.x + blockIdx.x] = s;
}

// A finished L1 norm and what follows from it, in the row's descriptor.
__device__ __forceinline__ void set_scale(RowDesc& r, double s, uint32_t d) {
    r.l1 = s;
    r.scale = (float)(s / (double)d);
    r.nonfinite = (s - s == 0.0) ? 0u : 1u;                     // s - s is NaN for NaN and Inf
}

// Finishes the L1 norm of each row from its block partials (fixed order) and sets the scale.
// grid = rows, desc points at the first row's descriptor.  256 threads, or 1024 for long rows: the kernel is a round
// trip or two to memory, and fewer rounds of loads shorten it (16 rows of 33779 partials 15 -> 8 us, event-timed).
__global__ __launch_bounds__(1024) void k_l1_final(const double* __restrict__ partial, uint32_t nparts,
                                                   uint32_t d, RowDesc* __restrict__ desc) {
    __shared__ double lds_w[16];
    const uint32_t row = blockIdx.x, step = blockDim.x;
    const double* __restrict__ p = partial + (size_t)row * nparts;
    // four independent running sums per thread (fixed assignment, fixed combination order) keep
    // four loads in flight
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    for (uint32_t q = threadIdx.x; q < nparts; q += 4 * step) {
        const double b0 = p[q];
        const double b1 = q + step < nparts ? p[q + step] : 0.0;
        const double b2 = q + 2 * step < nparts ? p[q + 2 * step] : 0.0;
        const double b3 = q + 3 * step < nparts ? p[q + 3 * step] : 0.0;
        a0 += b0;
        a1 += b1;
        a2 += b2;
        a3 += b3;
    }
    const double acc = (a0 + a1) + (a2 + a3);
    const double s = block_sum_f64(acc, lds_w);
    if (threadIdx.x == 0) set_scale(desc[row], s, d);
}

// The same by one wave for ROWS rows at once (row r's partials at p + r * stride, those from row n on left out), for the
// kernels that finish a few short sums themselves instead of waiting for a kernel that does.  Every lane has the sums, and
// they are the same in every wave that forms them.
template <int ROWS>
__device__ __forceinline__ void wave_l1(const double* __restrict__ p, size_t stride, int n, uint32_t nparts, uint32_t lane,
                                        double (&s)[ROWS]) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) s[r] = 0.0;
    for (uint32_t q = lane; q < nparts; q += 128) {
        double b[ROWS][2];
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int i = 0; i < 2; ++i) b[r][i] = r < n && q + 64 * i < nparts ? p[r * stride + q + 64 * i] : 0.0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) s[r] += b[r][0] + b[r][1];
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (r < n) s[r] = wave_sum(s[r]);                       // uniform
}

// ---------------------------------------------------------------------------------------------
// Blockwise scaled sign (Definition 5): Definition 4 on each of B consecutive column blocks
// [off[b], off[b+1]) with its own length.  Sign bits are the same as for Definition 4; only the
// scale depends on the column's block.
// ---------------------------------------------------------------------------------------------
struct BlockTable {
    const uint32_t* tile_blk;   // [ceil(d/1024)] block of the tile's first column; bit 31: the tile spans a boundary
    const uint32_t* off;        // [B + 1] block offsets, off[0] = 0, off[B] = d
    const float* scales;        // [(N + 1) * B] scale of block b of row r at r*B + b (row N: the server's v)
    uint32_t B;
};

__device__ __forceinline__ uint32_t block_of(const BlockTable& bt, uint32_t first, uint32_t j) {
    uint32_t b = first;
    while (b + 1 < bt.B && j >= bt.off[b + 1]) ++b;
    return b;
}

// One unit of the blockwise L1 pass: the part [lo, hi) of one compression block that falls into the
// 4096-column tile `tile`.  Items are ordered by block, then by tile.
struct L1Item {
    uint32_t tile, lo, hi, write_bits;
};

// grid = (items, rows).  Partial sum of |src| over the item's columns (fp64) and, for the item that
// owns the tile's bits, the sign bits of the whole tile.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_l1_items(const float* __restrict__ src, size_t row_stride, uint32_t d,
                                                      uint32_t nwt, uint32_t row0, const L1Item* __restrict__ items,
                                                      double* __restrict__ partial, uint16_t* __restrict__ bits) {
    __shared__ double lds_w[4];
    const L1Item it = items[blockIdx.x];
    const float* __restrict__ g = src + (size_t)blockIdx.y * row_stride;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t t = it.tile * 4 + wave;
    double acc = 0.0;
    if (t < nwt) {
        float4 a[4];
        if ((t + 1) * (uint32_t)kWaveTile <= d) {               // wave-uniform
            ld_tile<VEC>(g, t, lane, a);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = ld4<VEC, true>(g, t * kWaveTile + u * kChunk + lane * 4, d);
        }
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
            if (j >= it.lo && j < it.hi) acc += (double)fabsf(a[u].x);
            if (j + 1 >= it.lo && j + 1 < it.hi) acc += (double)fabsf(a[u].y);
            if (j + 2 >= it.lo && j + 2 < it.hi) acc += (double)fabsf(a[u].z);
            if (j + 3 >= it.lo && j + 3 < it.hi) acc += (double)fabsf(a[u].w);
            m |= (a[u].x < 0.f ? 1u : 0u) << (4 * u);
            m |= (a[u].y < 0.f ? 1u : 0u) << (4 * u + 1);
            m |= (a[u].z < 0.f ? 1u : 0u) << (4 * u + 2);
            m |= (a[u].w < 0.f ? 1u : 0u) << (4 * u + 3);
        }
        if (bits && it.write_bits) bits[((size_t)blockIdx.y * nwt + t) * 64 + lane] = (uint16_t)m;
    }
    const double s = block_sum_f64(acc, lds_w);
    if (threadIdx.x == 0) partial[(size_t)(row0 + blockIdx.y) * gridDim.x + blockIdx.x] = s;
}

// The same sums by tile, for the aggregation, which has all of a 4096-column tile of v at hand.
struct TileItems {
    const uint2* tile;          // [tiles] x: the tile's item when it has one (y == 1), else where its y items start in `of`
    const uint32_t* of;         // [items]
    const L1Item* items;        // [items]
};
// The partial sums of |a| of one 4096-column tile, which a block of 4 waves holds as wave tiles of 16 columns a lane
// (a[u]: columns j0 + 256u .. + 3 of this lane, 0 beyond the row's end).  Every thread of the block calls it, with the
// tile's entry of it.tile (read ahead of the columns, or its latency comes on top of theirs); lds_w: 4 words.  out: the
// row's partials.
__device__ __forceinline__ void l1_of_tile(const TileItems& it, uint2 entry, uint32_t j0, const float4 (&a)[4], double* lds_w,
                                           double* __restrict__ out) {
    for (uint32_t q = 0; q < entry.y; ++q) {                    // uniform
        const uint32_t item = entry.y == 1 ? entry.x : it.of[entry.x + q];
        double acc = 0.0;
        if (entry.y == 1) {                                     // the whole tile lies in one block
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc += (double)fabsf(a[u].x);
                acc += (double)fabsf(a[u].y);
                acc += (double)fabsf(a[u].z);
                acc += (double)fabsf(a[u].w);
            }
        } else {
            const uint2 r = make_uint2(it.items[item].lo, it.items[item].hi);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = j0 + u * kChunk;
                if (j >= r.x && j < r.y) acc += (double)fabsf(a[u].x);
                if (j + 1 >= r.x && j + 1 < r.y) acc += (double)fabsf(a[u].y);
                if (j + 2 >= r.x && j + 2 < r.y) acc += (double)fabsf(a[u].z);
                if (j + 3 >= r.x && j + 3 < r.y) acc += (double)fabsf(a[u].w);
            }
        }
        const double s = block_sum_f64(acc, lds_w);
        if (threadIdx.x == 0) out[item] = s;
        __syncthreads();                                        // lds_w is free for the next item
    }
}

// grid = (B, rows).  Adds up the item partials of block b in a fixed order and sets its scale.
__global__ __launch_bounds__(kBlock) void k_l1_items_final(const double* __restrict__ partial, uint32_t nitems,
                                                            const uint32_t* __restrict__ item_start,
                                                            const uint32_t* __restrict__ off, uint32_t B, uint32_t row0,
                                                            float* __restrict__ scales, double* __restrict__ l1s) {
    __shared__ double lds_w[4];
    const uint32_t b = blockIdx.x, row = row0 + blockIdx.y;
    const double* __restrict__ p = partial + (size_t)row * nitems;
    const uint32_t q0 = item_start[b], q1 = item_start[b + 1];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    uint32_t q = q0 + threadIdx.x;
    for (; q + 3 * kBlock < q1; q += 4 * kBlock) {
        a0 += p[q];
        a1 += p[q + kBlock];
        a2 += p[q + 2 * kBlock];
        a3 += p[q + 3 * kBlock];
    }
    for (; q < q1; q += kBlock) a0 += p[q];
    const double s = block_sum_f64((a0 + a1) + (a2 + a3), lds_w);
    if (threadIdx.x == 0) {
        l1s[(size_t)row * B + b] = s;
        scales[(size_t)row * B + b] = (float)(s / (double)(off[b + 1] - off[b]));
    }
}

}  // namespace liec
