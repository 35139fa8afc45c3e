// Server compensation, server compression, error update and the workers' update (Algorithm 1).
#pragma once
#include "common.hpp"
#include "select.hpp"
#include "sign.hpp"

namespace liec {

// acc[u].{x,y,z,w} += (bit 4u + q of m) ? -s : s  -- one scaled-sign message, 16 columns of a lane.
__device__ __forceinline__ float signed_scale(uint32_t m, int b, float s) {
    // bit b of m moved to the sign position and merged over +s (s >= 0)
    return __uint_as_float(((m << (31 - b)) & 0x80000000u) | __float_as_uint(s));
}
__device__ __forceinline__ void add_signed(float4 (&acc)[4], uint32_t m, float s) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        acc[u].x = __fadd_rn(acc[u].x, signed_scale(m, 4 * u + 0, s));
        acc[u].y = __fadd_rn(acc[u].y, signed_scale(m, 4 * u + 1, s));
        acc[u].z = __fadd_rn(acc[u].z, signed_scale(m, 4 * u + 2, s));
        acc[u].w = __fadd_rn(acc[u].w, signed_scale(m, 4 * u + 3, s));
    }
}

// ---------------------------------------------------------------------------------------------
// Worker message element p^i_j rebuilt from g_ij and the row's descriptor.
// ---------------------------------------------------------------------------------------------
template <int WC>
__device__ __forceinline__ float message_of(float g, uint32_t j, float scale, uint32_t tau, uint32_t cutoff,
                                            uint32_t keep) {
    if (WC == kSign || WC == kBlockSign) return g < 0.f ? -scale : scale;
    if (WC == kRandk) return keep ? g : 0.f;
    if (WC == kTopk) {
        const uint32_t key = key_of(g);
        return (key > tau || (key == tau && j <= cutoff)) ? g : 0.f;
    }
    return g;
}

// ---------------------------------------------------------------------------------------------
// Server compensation (Algorithm 1): v_j = e_j + (1/N) sum_i p^i_j, messages added in worker
// order; v goes to its own buffer.  With SRV_L1 the kernel also emits per-block partial sums of
// |v| (fp64) for the server's scaled-sign operator.  grid = blocks; waves stride over wave tiles.
//   WC == kSign / kBlockSign  read the packed sign bits instead of the gradients (blockwise: the scale
//                   comes from the column's block);
// (k_aggregate_sparse and k_aggregate_chunk below serve the other operators.)
// With `vbits` the kernel also leaves the sign bits of v (lane-major half-words like the workers' sign
// bits) for the update kernel of a scaled-sign server.
// FOLD (scaled sign, few workers on short rows): the block forms the workers' scales from the partial sums itself.
// ITEMS (blockwise server): the block's round is one 4096-column tile, and it leaves the partial L1 sums of that
// tile's items as k_l1_items would after reading v back (7 x 7.3M columns: 19 -> 23 us, and 11 us less for the
// pass over v).
// AHEAD (blockwise workers, rows whose e and v are more than the last-level cache keeps): e is requested ahead of the bits, and the rows'
// scales come with one load, a lane each.  What short rows wait for is not e, and there the registers and the extra load only cost: the
// tile's block and the rows' scales then come by vector loads that all lanes make (one scalar load after the other: 16 x 7M 26 -> 35 us).  us
// per step with and without, blockwise on both sides: 1 x 5M columns 42.8, 41.1, 2 x 9M + 1 85.8, 81.8, 1 x 25M 131.4, 128.2, 6 x 9M 174.6, 171.1,
// 32 x 9M 789, 783, 8 x 25M + 1 even, 5 x 30M + 1 470, 483, 3 x 40M + 1 450, 462, 3 x 75M + 1 826, 860, 3 x 99.4M 1068, 1088; blockwise / sign
// 1 x 5M 42.2, 39.8, 8 x 25M + 1 589, 583, 5 x 30M + 1 465, 474, 1 x 70M + 1 388, 399.
// ---------------------------------------------------------------------------------------------
constexpr int kFoldRows = 16;                                   // workers whose scales a block forms at most, 4 to a wave
template <int WC, bool SRV_L1, bool VEC, bool FOLD, bool ITEMS, bool AHEAD = false>
__global__ __launch_bounds__(kBlock) void k_aggregate(const uint16_t* __restrict__ bits, int N, uint32_t d, uint32_t nwt, float inv_n,
                                                       RowDesc* __restrict__ desc, const float* __restrict__ e_in,
                                                       float* __restrict__ v_out, double* __restrict__ srv_partial,
                                                       BlockTable bt, uint16_t* __restrict__ vbits,
                                                       const double* __restrict__ w_partial, uint32_t w_parts, TileItems items,
                                                       double* __restrict__ item_partial) {
    __shared__ double lds_w[4];
    __shared__ float folded[FOLD ? kFoldRows : 1];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // FOLD: what the first tile needs is requested ahead of the sums, or its latency comes on top of theirs (here and in the
    // update, with sums in the vector unit: 8 x 262144 columns 17.4 -> 14.8 us a step, 16 x 65536 16.7 -> 14.0).  Not
    // the tile that holds the row's end: among its guards the compiler waits for one of the loads before it asks for
    // the sums (so for all tiles, 1 x 65536 11.2 us instead of 10.7, slower than without the requests).
    uint32_t m0[8];
    float4 e0[4];
    if (FOLD) {
        const uint32_t t = min(blockIdx.x * 4 + wave, nwt - 1);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (r < N) m0[r] = bits[((size_t)r * nwt + t) * 64 + lane];         // uniform
        if ((t + 1) * (uint32_t)kWaveTile <= d) ld_tile<VEC, false>(e_in, t, lane, e0);
        // a wave's share of the workers: wave, wave + 4, ..
        double s[kFoldRows / 4];
        wave_l1(w_partial + (size_t)wave * w_parts, (size_t)4 * w_parts, (N - (int)wave + 3) / 4, w_parts, lane, s);
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < kFoldRows / 4; ++q) {
                const uint32_t i = wave + 4 * q;
                if (i < (uint32_t)N) {
                    folded[i] = (float)(s[q] / (double)d);
                    if (blockIdx.x == 0) set_scale(desc[i], s[q], d);   // for the update and the caller's queries
                }
            }
        }
        __syncthreads();
    }
    double l1 = 0.0;
    for (uint32_t tb = blockIdx.x * 4; tb < nwt; tb += gridDim.x * 4) {        // uniform for the block
        const uint32_t t = tb + wave;
        if (!ITEMS && t >= nwt) break;
        const uint32_t j0 = t * kWaveTile + lane * 4;
        const bool ahead = FOLD && tb == blockIdx.x * 4;        // requested ahead of the sums
        const uint64_t* const entry_at = reinterpret_cast<const uint64_t*>(items.tile) + tb / 4;
        const uint64_t ent = !ITEMS ? 0ull : WC == kSign || AHEAD ? ld_const(entry_at) : *entry_at;
        const bool whole = (t + 1) * (uint32_t)kWaveTile <= d;  // wave-uniform
        if (AHEAD && whole) ld_tile<VEC, false>(e_in, t, lane, e0);
        float4 acc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ITEMS && t >= nwt) {                                // a wave without a tile still takes part in the block's sums
        } else {
            const uint16_t* __restrict__ bw = bits + (size_t)t * 64 + lane;
            const size_t brow = (size_t)nwt * 64;
            const uint32_t tblk = WC != kBlockSign ? 0u : AHEAD ? ld_const(bt.tile_blk + t) : bt.tile_blk[t], first = tblk & 0x7fffffffu;
            if (WC == kSign || (!AHEAD && !(tblk >> 31))) {     // (blockwise: the whole wave tile lies in one block)
                auto scale_of = [&](int i) {
                    return WC == kBlockSign ? bt.scales[(size_t)i * bt.B + first] : FOLD ? folded[i] : desc[i].scale;
                };
                int i = 0;
                if (ahead) {
#pragma unroll
                    for (int r = 0; r < 8; ++r)
                        if (r < N) add_signed(acc, m0[r], scale_of(r));     // uniform
                    i = 8;
                }
                for (; i + 8 <= N; i += 8) {                    // 8 rows of bits in flight
                    uint32_t m[8];
#pragma unroll
                    for (int r = 0; r < 8; ++r) m[r] = bw[(size_t)(i + r) * brow];
#pragma unroll
                    for (int r = 0; r < 8; ++r) add_signed(acc, m[r], scale_of(i + r));
                }
                if (i < N) {                                    // and the rest of them
                    uint32_t m[7];
#pragma unroll
                    for (int r = 0; r < 7; ++r) m[r] = bw[(size_t)min(i + r, N - 1) * brow];
#pragma unroll
                    for (int r = 0; r < 7; ++r)
                        if (i + r < N) add_signed(acc, m[r], scale_of(i + r));      // uniform
                }
            } else if (AHEAD && !(tblk >> 31)) {
                float sc = 0.f;                                 // lane i: scale of the i-th of 64 rows
                for (int i = 0; i < N; i += 8) {
                    if ((i & 63) == 0 && i + (int)lane < N) sc = bt.scales[(size_t)(i + lane) * bt.B + first];
                    uint32_t m[8];
#pragma unroll
                    for (int r = 0; r < 8; ++r) m[r] = bw[(size_t)min(i + r, N - 1) * brow];
#pragma unroll
                    for (int r = 0; r < 8; ++r)
                        if (i + r < N) add_signed(acc, m[r], lane_value(sc, (uint32_t)(i + r) & 63));     // uniform
                }
            } else {
                uint32_t bidx[16];
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    const uint32_t j = j0 + (b >> 2) * kChunk + (b & 3);
                    bidx[b] = block_of(bt, b ? bidx[b - 1] : first, j < d ? j : d - 1);     // columns ascend with b
                }
                for (int i = 0; i < N; ++i) {
                    const uint32_t m = bw[(size_t)i * brow];
                    const float* __restrict__ sc = bt.scales + (size_t)i * bt.B;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        acc[u].x = __fadd_rn(acc[u].x, signed_scale(m, 4 * u + 0, sc[bidx[4 * u + 0]]));
                        acc[u].y = __fadd_rn(acc[u].y, signed_scale(m, 4 * u + 1, sc[bidx[4 * u + 1]]));
                        acc[u].z = __fadd_rn(acc[u].z, signed_scale(m, 4 * u + 2, sc[bidx[4 * u + 2]]));
                        acc[u].w = __fadd_rn(acc[u].w, signed_scale(m, 4 * u + 3, sc[bidx[4 * u + 3]]));
                    }
                }
            }
        }
        uint32_t vm = 0;                                        // sign bits of my 16 values of v
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = j0 + u * kChunk;
            const float4 e = (AHEAD || ahead) && whole ? e0[u] : ld4<VEC>(e_in, j, d);
            float4 v;
            v.x = __fmaf_rn(acc[u].x, inv_n, e.x);
            v.y = __fmaf_rn(acc[u].y, inv_n, e.y);
            v.z = __fmaf_rn(acc[u].z, inv_n, e.z);
            v.w = __fmaf_rn(acc[u].w, inv_n, e.w);
            if (ITEMS) acc[u] = make_float4(j < d ? v.x : 0.f, j + 1 < d ? v.y : 0.f, j + 2 < d ? v.z : 0.f, j + 3 < d ? v.w : 0.f);
            vm |= ((v.x < 0.f ? 1u : 0u) | (v.y < 0.f ? 2u : 0u) | (v.z < 0.f ? 4u : 0u) | (v.w < 0.f ? 8u : 0u)) << (4 * u);
            st4<VEC>(v_out, j, d, v);
            if (SRV_L1) {
                if (j < d) l1 += (double)fabsf(v.x);
                if (j + 1 < d) l1 += (double)fabsf(v.y);
                if (j + 2 < d) l1 += (double)fabsf(v.z);
                if (j + 3 < d) l1 += (double)fabsf(v.w);
            }
        }
        // a scaled-sign server's message is these bits and one scale: the update kernel reads them instead of v
        if (vbits && (!ITEMS || t < nwt)) vbits[(size_t)t * 64 + lane] = (uint16_t)vm;
        if (ITEMS) l1_of_tile(items, make_uint2((uint32_t)ent, (uint32_t)(ent >> 32)), j0, acc, lds_w, item_partial);
    }
    if (SRV_L1) {
        const double s = block_sum_f64(l1, lds_w);
        if (threadIdx.x == 0) srv_partial[blockIdx.x] = s;
    }
}

// ---------------------------------------------------------------------------------------------
// Top-k and random-k on long rows: the same sums, a wave per wave tile, from each row's bitmap -- top-k, the candidate
// bitmap (one bit per 4 columns, or `coarse`: per 64-byte line), whose groups are fetched and tested against (tau,
// cut-off); random-k, the kept bitmap.  A tile holds a few flagged groups per row, so going row after row spends a
// dependent gather, and instructions for 64 lanes, on a handful of lanes each time.  Instead the lanes share 16 rows'
// flags (4 lanes a row), write the flagged groups to a list in LDS in row order, and take it 64 entries at a time:
// one gather for 64 groups of all rows.  Sums live in LDS, one float4 per group.  Entries of one batch that fall on
// the same group are added in row order: every lane offers its row to the group's slot (atomic minimum), the lowest
// one adds, the others offer again.  Tiles with more flagged groups than pay (layers of large gradients, few rows, rows
// without a valid bitmap) go row by row, two rows' groups requested together: a row then costs its share of four gathers,
// an entry of the list 1/64 of a gather and its turns at the slots.  Row after row with one dependent
// gather each, against this: random-k 32 x 25.6M columns 159 -> 72 us, top-k of the same size 108 -> 64 (90 with a list
// of 128), both 0.1 %; top-k 16 x 16M, 1 %, 85 -> 59, 5 % 101 -> 71, 40 % 191 -> 170; 8 x 50M, 3 %, 147 -> 143; 16 x 138M,
// 0.5 % (1.1 GB of e and v and 0.8 GB of gradients in layers where every line holds a candidate), 383 -> 365.  The line
// between the two ways: with every tile of up to 512 entries listed, 1 x 16M, 40 %, took 51 us, row by row 34 (2 rows 64
// and 41; 8 x 50M in the coarse form, whose entries are four groups, 409 and 283); with 16 or 24 groups per row as the
// limit 32 x 25.6M, 0.1 %, took 80 us, with 48 64; 32, 48 and 64 differ by no more than runs do but at 16 x 138M (375,
// 365, 366).
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kSparseList = 512;                           // flagged groups (coarse: lines) of 16 rows the list holds,
constexpr uint32_t kSparseGroups = 48;                          // and groups per row up to which it is used
__device__ __forceinline__ void wave_sync() {                   // LDS traffic between the lanes of one wave
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ uint32_t nonzero_nibbles(uint32_t x) {
    x |= x >> 1;
    x |= x >> 2;
    return x & 0x11111111u;
}
// Which of the 4 columns j .. j + 3 are kept, by the threshold.
__device__ __forceinline__ uint32_t kept_of_4(float4 g, uint32_t j, uint32_t d, uint32_t tau, uint32_t cut) {
    const float gv[4] = {g.x, g.y, g.z, g.w};
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t key = key_of(gv[q]);
        m |= (j + q < d && (key > tau || (key == tau && j + q <= cut)) ? 1u : 0u) << q;
    }
    return m;
}
__device__ __forceinline__ void add_kept(float4& acc, float4 g, uint32_t keep) {
    if (keep & 1u) acc.x = __fadd_rn(acc.x, g.x);
    if (keep & 2u) acc.y = __fadd_rn(acc.y, g.y);
    if (keep & 4u) acc.z = __fadd_rn(acc.z, g.z);
    if (keep & 8u) acc.w = __fadd_rn(acc.w, g.w);
}
template <int WC, bool SRV_L1, bool VEC>
__global__ __launch_bounds__(kBlock) void k_aggregate_sparse(const float* __restrict__ grads, const uint16_t* __restrict__ bits,
                                                              const uint64_t* __restrict__ gbits, int N, uint32_t d,
                                                              uint32_t nwt, float inv_n, const RowDesc* __restrict__ desc,
                                                              const float* __restrict__ e_in, float* __restrict__ v_out,
                                                              double* __restrict__ srv_partial, bool coarse,
                                                              uint16_t* __restrict__ vbits) {
    __shared__ double lds_w[4];
    __shared__ float4 accs[4][256];
    __shared__ uint32_t slots[4][256], lists[4][kSparseList];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float4* const acc = accs[wave];                             // group 64u + l: the 4 columns of lane l in chunk u
    uint32_t* const slot = slots[wave];
    uint32_t* const list = lists[wave];
#pragma unroll
    for (int u = 0; u < 4; ++u) slot[u * 64 + lane] = 0xffffffffu;
    double l1 = 0.0;
    for (uint32_t t = blockIdx.x * 4 + wave; t < nwt; t += gridDim.x * 4) {
        const uint32_t j0 = t * kWaveTile + lane * 4;
        float4 e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            e[u] = ld4<VEC>(e_in, j0 + u * kChunk, d);
            acc[u * 64 + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        wave_sync();
        for (int i0 = 0; i0 < N; i0 += 16) {
            const uint32_t row = (uint32_t)i0 + (lane >> 2), part = lane & 3;
            uint64_t w = 0;                                     // top-k: my share of my row's flags
            uint32_t x[8] = {0, 0, 0, 0, 0, 0, 0, 0};           // random-k: my 16 half-words of them
            uint32_t cnt = 0;
            if (row < (uint32_t)N) {
                if (WC == kTopk) {
                    if (coarse) w = (gbits[(size_t)row * nwt + t] >> (16 * part)) & 0xffffu;
                    else w = gbits[((size_t)row * nwt + t) * 4 + part];
                    if (desc[row].dense) w = coarse ? 0xffffull : ~0ull;
                    cnt = (uint32_t)__popcll(w);
                } else {
                    const uint4* __restrict__ b = reinterpret_cast<const uint4*>(bits + ((size_t)row * nwt + t) * 64) + part * 2;
                    const uint4 b0 = b[0], b1 = b[1];
                    x[0] = b0.x; x[1] = b0.y; x[2] = b0.z; x[3] = b0.w;
                    x[4] = b1.x; x[5] = b1.y; x[6] = b1.z; x[7] = b1.w;
#pragma unroll
                    for (int q = 0; q < 8; ++q) cnt += (uint32_t)__popc(nonzero_nibbles(x[q]));
                }
            }
            const uint32_t incl = wave_scan(cnt), total = last_lane(incl);
            if (total == 0) continue;
            const uint32_t per_row = WC == kTopk && coarse ? kSparseGroups / 4 : kSparseGroups;
            if (total <= min(kSparseList, (uint32_t)min(16, N - i0) * per_row)) {     // wave-uniform
                uint32_t pos = incl - cnt;
                if (WC == kTopk) {
                    while (w) {
                        const uint32_t b = (uint32_t)__builtin_ctzll(w), line = 16 * part + b;
                        w &= w - 1;
                        list[pos++] = row << 16 | (coarse ? (line & 3) * 64 + (line >> 2) * 4 : part * 64 + b) << 4;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        uint32_t m = nonzero_nibbles(x[q]);
                        while (m) {
                            const uint32_t b = (uint32_t)__builtin_ctz(m);
                            m &= m - 1;
                            list[pos++] = row << 16 | ((b >> 2 & 3) * 64 + part * 16 + q * 2 + (b >> 4)) << 4 | (x[q] >> b & 0xfu);
                        }
                    }
                }
                wave_sync();
                const uint32_t sub = WC == kTopk && coarse ? 2 : 0, n = total << sub;      // a line is 4 groups
                for (uint32_t base = 0; base < n; base += 64) {
                    const uint32_t at = base + lane;
                    const bool live = at < n;
                    const uint32_t ent = live ? list[at >> sub] : 0u;
                    const uint32_t r = ent >> 16, gi = (ent >> 4 & 0xffu) + (sub ? at & 3u : 0u);
                    const uint32_t j = t * kWaveTile + (gi >> 6) * kChunk + (gi & 63) * 4;
                    float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
                    uint32_t keep = 0;
                    if (live) {
                        g = ld4<VEC>(grads + (size_t)r * d, j, d);
                        keep = WC == kRandk ? ent & 0xfu : kept_of_4(g, j, d, desc[r].tau, desc[r].cutoff);
                    }
                    while (__ballot(keep != 0)) {
                        if (keep) atomicMin(&slot[gi], r);
                        wave_sync();
                        const bool mine = keep && slot[gi] == r;
                        wave_sync();
                        if (mine) {
                            float4 a = acc[gi];
                            add_kept(a, g, keep);
                            acc[gi] = a;
                            slot[gi] = 0xffffffffu;
                            keep = 0;
                        }
                        wave_sync();
                    }
                }
            } else {
                const int end = min(i0 + 16, N);
                for (int i = i0; i < end; i += 2) {
                    float4 g[2][4];
                    uint32_t flag[2];                           // top-k: bit u, my group of chunk u; random-k: my kept bits
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const size_t ir = (size_t)min(i + r, N - 1);
                        if (WC == kRandk) {
                            flag[r] = bits[(ir * nwt + t) * 64 + lane];
                        } else if (coarse) {
                            flag[r] = (uint32_t)(gbits[ir * nwt + t] >> (4 * (lane >> 2))) & 0xfu;
                        } else {
                            const uint64_t* __restrict__ f = gbits + (ir * nwt + t) * 4;
                            flag[r] = (uint32_t)((f[0] >> lane) & 1) | (uint32_t)((f[1] >> lane) & 1) << 1 |
                                      (uint32_t)((f[2] >> lane) & 1) << 2 | (uint32_t)((f[3] >> lane) & 1) << 3;
                        }
                        if (WC == kTopk && desc[ir].dense) flag[r] = 0xfu;
                        if (i + r >= N) flag[r] = 0;
                    }
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const float* __restrict__ gr = grads + (size_t)min(i + r, N - 1) * d;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const bool want = WC == kRandk ? ((flag[r] >> (4 * u)) & 0xfu) != 0 : ((flag[r] >> u) & 1u) != 0;
                            g[r][u] = make_float4(0.f, 0.f, 0.f, 0.f);
                            if (want) g[r][u] = ld4<VEC>(gr, j0 + u * kChunk, d);
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const int ir = min(i + r, N - 1);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            uint32_t keep = (flag[r] >> (4 * u)) & 0xfu;
                            if (WC == kTopk)
                                keep = ((flag[r] >> u) & 1u) ? kept_of_4(g[r][u], j0 + u * kChunk, d, desc[ir].tau, desc[ir].cutoff) : 0u;
                            if (keep) {                         // my own groups: no other lane adds to them here
                                float4 a = acc[u * 64 + lane];
                                add_kept(a, g[r][u], keep);
                                acc[u * 64 + lane] = a;
                            }
                        }
                    }
                }
            }
            wave_sync();
        }
        uint32_t vm = 0;                                        // sign bits of my 16 values of v
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t j = j0 + u * kChunk;
            const float4 a = acc[u * 64 + lane];
            float4 v;
            v.x = __fmaf_rn(a.x, inv_n, e[u].x);
            v.y = __fmaf_rn(a.y, inv_n, e[u].y);
            v.z = __fmaf_rn(a.z, inv_n, e[u].z);
            v.w = __fmaf_rn(a.w, inv_n, e[u].w);
            vm |= ((v.x < 0.f ? 1u : 0u) | (v.y < 0.f ? 2u : 0u) | (v.z < 0.f ? 4u : 0u) | (v.w < 0.f ? 8u : 0u)) << (4 * u);
            st4<VEC, true>(v_out, j, d, v);
            if (SRV_L1) {
                if (j < d) l1 += (double)fabsf(v.x);
                if (j + 1 < d) l1 += (double)fabsf(v.y);
                if (j + 2 < d) l1 += (double)fabsf(v.z);
                if (j + 3 < d) l1 += (double)fabsf(v.w);
            }
        }
        if (vbits) vbits[(size_t)t * 64 + lane] = (uint16_t)vm;
        wave_sync();                                            // the sums are read before the next tile clears them
    }
    if (SRV_L1) {
        const double s = block_sum_f64(l1, lds_w);
        if (threadIdx.x == 0) srv_partial[blockIdx.x] = s;
    }
}

struct ServerFilter {          // the first filter pass of the server's row, ridden by the aggregation
    uint2* list;
    uint32_t cap, k;
    uint64_t* sgbits;
};

// ---------------------------------------------------------------------------------------------
// The same sums with a wave owning one chunk (256 columns, 4 per lane) and a block one wave tile at a time: four times
// as many waves.  For rows too short to fill the chip with a wave per tile, where the kernel is bound by the latency
// of its dependent loads (group word, then gather, row after row) and not by bytes -- the loads of 8 rows are
// requested together and added in worker order afterwards -- and for the identity operator on rows of any length:
// four rows of one 128-bit load per lane in flight stream 8 x 11.7M gradients at 6.2 TB/s, a wave walking the four
// chunks of row after row at 3.9.  On long rows the work per row and chunk (a group word for 256 columns) costs more
// instructions than the gathers do; the host's rule has both sides' times.
// ---------------------------------------------------------------------------------------------
// SRV_FILTER (top-k server): the values of v are filtered against the server's predicted band while they are in
// registers, as k_filter's first pass would after reading them back.
// ROWS: rows requested together.  Words are requested for that many rows whether they are there or not, so up to kFewRows top-k rows take a
// kernel of that many (us per step with 4 and with 8, top-k / sign: 1 x 2.5M columns 34.3, 36.5, 1 x 8M 82.9, 88.8, 2 x 4M + 1 64.9, 67.6,
// 4 x 3M 71.3, 74.5, 4 x 65536 even).
// Identity workers under a random-k server: vodd receives, per chunk, a bit for every 4 columns in which v is not finite,
// for the update.
constexpr int kFewRows = 4;
template <int WC, bool SRV_L1, bool VEC, bool SRV_FILTER, int ROWS = 8>
__global__ __launch_bounds__(kBlock) void k_aggregate_chunk(const float* __restrict__ grads, const uint16_t* __restrict__ bits,
                                                             const uint64_t* __restrict__ gbits, int N, uint32_t d,
                                                             uint32_t nwt, float inv_n, RowDesc* __restrict__ desc,
                                                             const float* __restrict__ e_in, float* __restrict__ v_out,
                                                             double* __restrict__ srv_partial, BlockTable bt, bool coarse,
                                                             uint16_t* __restrict__ vbits, uint64_t* __restrict__ vodd,
                                                             ServerFilter sf) {
    __shared__ double lds_w[4];
    __shared__ uint32_t nibs[4][64];
    // a block has one tile, so its stage never overflows into stages of the waves' own
    static_assert(!SRV_FILTER || kStage >= kWaveTile, "a tile's candidates fit the block's stage");
    __shared__ uint2 stage[SRV_FILTER ? kStage : 1];
    __shared__ uint32_t wsure[5], staged[2];
    constexpr int kRows = ROWS;
    FilterBand fb{};
    bool filter = false;                                        // uniform: the server's row has a predicted band
    uint32_t n_hi = 0, kmax = 0, wcnt = 0;
    if (SRV_FILTER) {                                           // (what filter_band does for a first pass, without a branch or a wait here)
        filter = ld_const(&desc[N].mode) == kWarm;
        fb.lo = ld_const(&desc[N].lo);
        fb.hi = ld_const(&desc[N].hi);
        fb.out = sf.list + (size_t)N * sf.cap;
        fb.cap = sf.cap;
        fb.counts = reinterpret_cast<unsigned long long*>(&desc[N].n_cand);
        if (threadIdx.x < 2) staged[threadIdx.x] = 0;
    }
    const uint32_t u = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;   // my chunk of the tile
    double l1 = 0.0;
    for (uint32_t t = blockIdx.x; t < nwt; t += gridDim.x) {   // uniform for the block
        const uint32_t j = t * kWaveTile + u * kChunk + lane * 4;
        const float4 e = ld4<VEC>(e_in, j, d);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (WC == kBlockSign) {
            const uint16_t* __restrict__ bw = bits + (size_t)t * 64 + lane;
            const size_t brow = (size_t)nwt * 64;
            const uint32_t tb = ld_const(bt.tile_blk + t), first = tb & 0x7fffffffu;
            uint32_t blk[4] = {first, first, first, first};
            if (tb >> 31) {               // the tile spans a block boundary
#pragma unroll
                for (int q = 0; q < 4; ++q) blk[q] = block_of(bt, first, j + q < d ? j + q : d - 1);
            }
            // lane i: scale of the i-th of 64 rows (a tile in one block), one load instead of a scalar one after the other (us per step:
            // 8 x 1M 41.9 -> 40.1, 20 x 104143 33.9 -> 29.0, blockwise / sign 64 x 500000 125 -> 109)
            float sc = 0.f;
            for (int i0 = 0; i0 < N; i0 += kRows) {
                if (!(tb >> 31) && (i0 & 63) == 0 && i0 + (int)lane < N) sc = bt.scales[(size_t)(i0 + lane) * bt.B + first];
                uint32_t m[kRows];
#pragma unroll
                for (int r = 0; r < kRows; ++r) m[r] = bw[(size_t)min(i0 + r, N - 1) * brow];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    if (i0 + r < N) {                           // uniform
                        float s[4];
                        if (!(tb >> 31)) {
                            s[0] = s[1] = s[2] = s[3] = lane_value(sc, (uint32_t)(i0 + r) & 63);
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q) s[q] = bt.scales[(size_t)(i0 + r) * bt.B + blk[q]];
                        }
                        const uint32_t b = m[r] >> (4 * u);
                        acc.x = __fadd_rn(acc.x, signed_scale(b, 0, s[0]));
                        acc.y = __fadd_rn(acc.y, signed_scale(b, 1, s[1]));
                        acc.z = __fadd_rn(acc.z, signed_scale(b, 2, s[2]));
                        acc.w = __fadd_rn(acc.w, signed_scale(b, 3, s[3]));
                    }
                }
            }
        } else if (WC == kTopk || WC == kRandk) {
            // which of my 4 columns to fetch: top-k, the candidate bit of my group (coarse: of its 64-byte line); random-k, the kept bits
            const uint64_t* __restrict__ gw = gbits + (coarse ? (size_t)t : (size_t)t * 4 + u);
            const size_t grow = coarse ? (size_t)nwt : (size_t)nwt * 4;
            const uint16_t* __restrict__ bw = bits + (size_t)t * 64 + lane;
            for (int i0 = 0; i0 < N; i0 += kRows) {
                // requested together and without a branch among them: under one for each row the compiler waits for a row's words
                // before it asks for the next row's
                uint32_t pick[kRows], tau[kRows], cut[kRows], dense[kRows];
                uint64_t w[kRows];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    const int i = min(i0 + r, N - 1);
                    if (WC == kRandk) {
                        pick[r] = bw[(size_t)i * nwt * 64];
                    } else {
                        tau[r] = ld_const(&desc[i].tau);
                        cut[r] = ld_const(&desc[i].cutoff);
                        dense[r] = ld_const(&desc[i].dense);
                        w[r] = ld_const(gw + (size_t)i * grow);
                    }
                }
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    if (WC == kRandk) {
                        pick[r] = i0 + r < N ? (pick[r] >> (4 * u)) & 0xfu : 0u;
                    } else {
                        if (dense[r]) w[r] = ~0ull;             // uniform
                        pick[r] = i0 + r < N ? (uint32_t)(w[r] >> (coarse ? 4 * (lane >> 2) + u : lane)) & 1u : 0u;
                    }
                }
                float4 gq[kRows];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    gq[r] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (pick[r]) gq[r] = ld4<VEC>(grads + (size_t)(i0 + r) * d, j, d);
                }
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    if (pick[r]) {
                        const float gv[4] = {gq[r].x, gq[r].y, gq[r].z, gq[r].w};
                        float* av[4] = {&acc.x, &acc.y, &acc.z, &acc.w};
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t key = key_of(gv[q]);
                            const bool keep = WC == kRandk ? ((pick[r] >> q) & 1u) != 0
                                                           : j + q < d && (key > tau[r] || (key == tau[r] && j + q <= cut[r]));
                            if (keep) *av[q] = __fadd_rn(*av[q], gv[q]);
                        }
                    }
                }
            }
        } else {
            int i = 0;
            for (; i + 4 <= N; i += 4) {
                float4 g[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) g[r] = ld4<VEC, true>(grads + (size_t)(i + r) * d, j, d);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc.x = __fadd_rn(acc.x, g[r].x);
                    acc.y = __fadd_rn(acc.y, g[r].y);
                    acc.z = __fadd_rn(acc.z, g[r].z);
                    acc.w = __fadd_rn(acc.w, g[r].w);
                }
            }
            for (; i < N; ++i) {
                const float4 g = ld4<VEC, true>(grads + (size_t)i * d, j, d);
                acc.x = __fadd_rn(acc.x, g.x);
                acc.y = __fadd_rn(acc.y, g.y);
                acc.z = __fadd_rn(acc.z, g.z);
                acc.w = __fadd_rn(acc.w, g.w);
            }
        }
        float4 v;
        v.x = __fmaf_rn(acc.x, inv_n, e.x);
        v.y = __fmaf_rn(acc.y, inv_n, e.y);
        v.z = __fmaf_rn(acc.z, inv_n, e.z);
        v.w = __fmaf_rn(acc.w, inv_n, e.w);
        st4<VEC>(v_out, j, d, v);
        if (WC == kIdentity && vodd) {
            const uint64_t odd = __ballot(any_nonfinite(v.x, v.y, v.z, v.w));
            if (lane == 0) vodd[(size_t)t * 4 + u] = odd;
        }
        if (SRV_FILTER) __syncthreads();                        // the stage's counters are set (a block that filters has one tile)
        if (SRV_FILTER && filter) {
            const uint32_t keys[4] = {key_of(v.x), key_of(v.y), key_of(v.z), key_of(v.w)};
            uint64_t bc[4];
            uint32_t hi4;
            const uint64_t any_lo = filter_chunk<false, false>(keys, j, d, fb.lo, fb.hi, bc, n_hi, kmax, hi4);
            if (lane == 0) sf.sgbits[(size_t)t * 4 + u] = any_lo;
            stage_candidates(fb, keys, j, bc, stage, nullptr, wcnt, staged, lane);
        }
        if (SRV_L1) {
            if (j < d) l1 += (double)fabsf(v.x);
            if (j + 1 < d) l1 += (double)fabsf(v.y);
            if (j + 2 < d) l1 += (double)fabsf(v.z);
            if (j + 3 < d) l1 += (double)fabsf(v.w);
        }
        if (vbits) {                                            // uniform; the four chunks' bits of a lane form one half-word
            nibs[u][lane] = (v.x < 0.f ? 1u : 0u) | (v.y < 0.f ? 2u : 0u) | (v.z < 0.f ? 4u : 0u) | (v.w < 0.f ? 8u : 0u);
            __syncthreads();
            if (u == 0)
                vbits[(size_t)t * 64 + lane] =
                    (uint16_t)(nibs[0][lane] | nibs[1][lane] << 4 | nibs[2][lane] << 8 | nibs[3][lane] << 12);
            __syncthreads();
        }
    }
    if (SRV_L1) {
        const double s = block_sum_f64(l1, lds_w);
        if (threadIdx.x == 0) srv_partial[blockIdx.x] = s;
    }
    if (SRV_FILTER && filter) {
        if (__ballot(kmax >= 0x7f800000u) && lane == 0) atomicOr(&desc[N].nonfinite_acc, 1u);     // Inf / NaN
        finish_filter_block(fb, stage, nullptr, wcnt, n_hi, staged, wsure);
    }
}

// What the last kernel of a step with a threshold search leaves behind it: the rows are in the next step's mode, on its band
// and with counters of zero, the meeting points of the blocks that share rows are zero, and the next compressed iteration
// makes the next draw.  None of its other blocks looks at any of these.  (The grid has at least one thread a row.)
struct StepTail {
    RowDesc* desc;              // [rows]; a pointer of its own, so that the kernel's loads of what it does not change stay scalar
    uint32_t* sync;             // [nsync]
    uint64_t* draw;             // random-k on a side, else null
    uint32_t rows, nsync;
};
__device__ __forceinline__ void end_searches(const StepTail& t) {
    const uint32_t q = blockIdx.x * kBlock + threadIdx.x;
    if (blockIdx.x * kBlock >= max(t.rows, t.nsync)) return;    // uniform for the block
    if (q < t.rows) {
        RowDesc r = t.desc[q];                                  // in registers while the next band is predicted
        const bool due = r.due != 0;
        next_step(r);
        RowDesc& to = t.desc[q];                                // (what the other blocks read stays unwritten)
        to.lo = r.lo;
        to.hi = r.hi;
        to.mode = r.mode;
        if (due) {
            to.prev_tau = r.prev_tau;
            to.have_prev = r.have_prev;
            to.centre = r.centre;
            to.swing = r.swing;
            to.swing_still = r.swing_still;
            to.far = r.far;
            to.was_cold = r.was_cold;
            to.next_lo = r.next_lo;
            to.next_hi = r.next_hi;
            to.next_mode = r.next_mode;
            to.due = 0;
        }
        clear_counts(to);
    }
    if (q < t.nsync && (q & (kSyncWords - 1)) < 2) t.sync[q] = 0;      // (the third word is the searches' own)
    if (q == 0 && t.draw) *t.draw += 1;
}

// ---------------------------------------------------------------------------------------------
// Server compression + error update + broadcast + local immediate compensation (Algorithm 1):
//   p_j = C_s(v)_j ; e_j <- v_j - p_j ; x_ij <- x_ij - lr * (p_j + (g_ij - p^i_j)).
// One block = 1024 columns of one row.  Blocks are ordered panel by panel (a panel is `panel`
// consecutive column tiles), inside a panel row by row, so every row is walked in long contiguous
// runs while the panel's slice of v stays in cache for the N rows that reuse it; the row-0 block of
// a tile also writes e.  grid = number of panels * panel * N.
// FOLD (scaled-sign server, few blocks): every wave forms the server's scale from the partial sums itself.
// ---------------------------------------------------------------------------------------------
template <int WC, int SC, bool VEC, bool FOLD = false>
__global__ __launch_bounds__(kBlock) void k_update(const float* __restrict__ grads, float* __restrict__ x,
                                                    const float* __restrict__ v_in, float* __restrict__ e_out, int N,
                                                    uint32_t panel, uint32_t ncol_tiles, uint32_t d, float neg_lr,
                                                    RowDesc* __restrict__ desc, BlockTable bt,
                                                    const uint16_t* __restrict__ kbits, const uint16_t* __restrict__ vbits,
                                                    const uint64_t* __restrict__ sgbits, const uint64_t* __restrict__ vodd,
                                                    const double* __restrict__ s_partial, uint32_t s_parts, StepTail tail) {
    if (WC == kTopk || WC == kRandk || SC == kTopk || SC == kRandk) end_searches(tail);
    const uint32_t per_panel = panel * (uint32_t)N;
    const uint32_t pn = blockIdx.x / per_panel, r = blockIdx.x % per_panel;
    const uint32_t i = r / panel, tile = pn * panel + r % panel;
    if (tile >= ncol_tiles) return;
    const uint32_t j = tile * kColTile + threadIdx.x * 4;
    const float* __restrict__ gi = grads + (size_t)i * d;
    float* __restrict__ xi = x + (size_t)i * d;
    float4 g0 = make_float4(0.f, 0.f, 0.f, 0.f), x0 = g0;
    float folded = 0.f;
    if (FOLD) {                                                 // the streams are requested ahead of the sum, which every wave forms
        if (WC != kIdentity) g0 = ld4<VEC, true>(gi, j, d);
        x0 = ld4<VEC, true>(xi, j, d);
        double s[1];
        wave_l1(s_partial, 0, 1, s_parts, threadIdx.x & 63, s);
        folded = (float)(s[0] / (double)d);
        if (blockIdx.x == 0 && threadIdx.x == 0) set_scale(desc[N], s[0], d);
    }
    if (j >= d) return;
    const uint32_t lane = threadIdx.x & 63, chunk = threadIdx.x >> 6;   // this thread is lane `lane` of chunk `chunk` of wave tile `tile`
    uint32_t tb = 0;
    if (WC == kBlockSign || SC == kBlockSign) tb = bt.tile_blk[tile];   // issued ahead of the streams
    // random-k: the 4 kept bits of this thread's columns; row N of the bitmap is the server's draw
    uint32_t wkeep = 0, skeep = 0;
    if (WC == kRandk) wkeep = (kbits[((size_t)i * ncol_tiles + tile) * 64 + lane] >> (4 * chunk)) & 0xfu;
    if (SC == kRandk) skeep = (kbits[((size_t)N * ncol_tiles + tile) * 64 + lane] >> (4 * chunk)) & 0xfu;
    uint64_t vo = 0;                                       // identity workers, random-k server: where v is not finite
    if (WC == kIdentity && SC == kRandk) vo = vodd[(size_t)tile * 4 + chunk];
    const RowDesc* __restrict__ sd = desc + N;
    // What the server's message needs of v.  The row-0 block of a tile reads v in full (it writes e).  The other
    // rows' blocks take what the server side left behind instead of re-reading 4 d bytes of v per row: the sign
    // bits of v (scaled sign, either form), the candidate bit of these 4 columns (top-k: v is read only where
    // a candidate sits, unless the row's bitmap is not valid), the kept bits (random-k).
    uint32_t sbits = 0;
    bool need_v = true;
    // The sign bits of v, for most pairs with a blockwise side: every row's block asks for them, no branch stands around the load, and their
    // half-words stay in a register until the gradients are there.  With the shift next to the load, under the branch for i != 0, the compiler
    // waits for them before it asks for the gradients.  Update kernel, us, so against under the branch, aligned rows and others: blockwise on both
    // sides 24 x 9M 409, 424 (432, 445), 64 x 1M 122, 127 (127, 130); sign / blockwise 24 x 9M 415, 424 (433, 446); top-k / blockwise 421, 463 (449,
    // 485); random-k / blockwise 412, 457 (439, 478); blockwise / sign 415, 419 (433, 442); top-k / sign 414, 414 (428, 434).  Under the branch is
    // better where the scaled sign or no operator is the workers': sign on both sides 24 x 9M 417, 407 (433, 433), 64 x 1M 122, 120; identity / sign
    // 2 x 25M 90.5, 87.5; identity / blockwise 2 x 25M 96.6, 93.0, 24 x 9M 330, 330 (344, 332); and random-k / sign 24 x 9M 414, 407.
    constexpr bool kSignsFirst = WC == kBlockSign ? SC == kSign || SC == kBlockSign
                                                  : (SC == kBlockSign && WC != kIdentity) || (SC == kSign && WC == kTopk);
    if (kSignsFirst) sbits = vbits[(size_t)tile * 64 + lane];
    if (i != 0) {
        if (SC == kSign || SC == kBlockSign) {
            if (!kSignsFirst) sbits = ((uint32_t)vbits[(size_t)tile * 64 + lane] >> (4 * chunk)) & 0xfu;
            need_v = false;
        } else if (SC == kTopk) {
            need_v = sd->dense || ((sgbits[(size_t)tile * 4 + chunk] >> lane) & 1u);
        } else if (SC == kRandk) {
            need_v = skeep != 0;
        }
    }
    // an uncompressed message leaves no local error: g - p^i is g - g = +0 for every finite gradient (the others: see the
    // end), and the gradients are not read a second time (8 rows of 11.7M + 2 columns: 195 -> 139 us)
    const float4 g = FOLD ? g0 : WC == kIdentity ? make_float4(0.f, 0.f, 0.f, 0.f) : ld4<VEC, true>(gi, j, d);
#if defined(__HIP_DEVICE_COMPILE__)
    // One stream at a time per wave: waiting for the gradients before asking for the model measured
    // 2-4 % faster than having both 128-bit loads in flight.
    if (!FOLD && kSignsFirst) asm volatile("s_waitcnt vmcnt(0)" : "+v"(sbits)::"memory");
    else if (!FOLD) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    const float4 xv = FOLD ? x0 : ld4<VEC, true>(xi, j, d);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (need_v) v = ld4<VEC>(v_in, j, d);
    if (kSignsFirst) sbits = (sbits >> (4 * chunk)) & 0xfu;
    const uint32_t stau = sd->tau, scut = sd->cutoff;
    float sw[4], ss[4];                                    // worker / server scale of each of the 4 columns
    if (WC == kBlockSign || SC == kBlockSign) {
        const uint32_t first = tb & 0x7fffffffu;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t b = (tb >> 31) ? block_of(bt, first, j + c < d ? j + c : d - 1) : first;
            sw[c] = WC == kBlockSign ? bt.scales[(size_t)i * bt.B + b] : desc[i].scale;
            ss[c] = SC == kBlockSign ? bt.scales[(size_t)N * bt.B + b] : FOLD ? folded : sd->scale;
        }
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            sw[c] = desc[i].scale;
            ss[c] = FOLD ? folded : sd->scale;
        }
    }
    float4 p;
    if ((SC == kSign || SC == kBlockSign) && i != 0) {
        p.x = (sbits & 1u) ? -ss[0] : ss[0];
        p.y = (sbits & 2u) ? -ss[1] : ss[1];
        p.z = (sbits & 4u) ? -ss[2] : ss[2];
        p.w = (sbits & 8u) ? -ss[3] : ss[3];
    } else {                                               // for columns whose v was not read p is +0, as v is
        p.x = message_of<SC>(v.x, j, ss[0], stau, scut, skeep & 1u);
        p.y = message_of<SC>(v.y, j + 1, ss[1], stau, scut, skeep & 2u);
        p.z = message_of<SC>(v.z, j + 2, ss[2], stau, scut, skeep & 4u);
        p.w = message_of<SC>(v.w, j + 3, ss[3], stau, scut, skeep & 8u);
    }
    if (i == 0) {
        float4 en;
        en.x = __fsub_rn(v.x, p.x);
        en.y = __fsub_rn(v.y, p.y);
        en.z = __fsub_rn(v.z, p.z);
        en.w = __fsub_rn(v.w, p.w);
        st4<VEC>(e_out, j, d, en);
    }
    const uint32_t tau = desc[i].tau, cut = desc[i].cutoff;
    float4 o;
    o.x = __fmaf_rn(neg_lr, __fadd_rn(p.x, __fsub_rn(g.x, message_of<WC>(g.x, j, sw[0], tau, cut, wkeep & 1u))), xv.x);
    o.y = __fmaf_rn(neg_lr, __fadd_rn(p.y, __fsub_rn(g.y, message_of<WC>(g.y, j + 1, sw[1], tau, cut, wkeep & 2u))), xv.y);
    o.z = __fmaf_rn(neg_lr, __fadd_rn(p.z, __fsub_rn(g.z, message_of<WC>(g.z, j + 2, sw[2], tau, cut, wkeep & 4u))), xv.z);
    o.w = __fmaf_rn(neg_lr, __fadd_rn(p.w, __fsub_rn(g.w, message_of<WC>(g.w, j + 3, sw[3], tau, cut, wkeep & 8u))), xv.w);
    if (WC == kIdentity) {
        // g - g is NaN for an Inf or NaN.  A gradient that is one leaves v not finite in its column (nothing that is added
        // brings a sum back), and that shows in v, in the scale, in a threshold above every finite key when v was not
        // read for want of a candidate, or, with a random-k server, in the aggregation's bits: the gradients are read
        // where it does.  (The look costs 0.2-0.6 us on steps of up to 25 us, within 1 % at 8 x 11.7M + 2 columns, 2.5 %
        // with a blockwise server.)
        bool odd = any_nonfinite(v.x, v.y, v.z, v.w);
        if (SC == kSign || SC == kBlockSign) odd = any_nonfinite(ss[0], ss[1], ss[2], ss[3]);
        if (SC == kTopk) odd = odd || stau >= kInfKey;
        if (SC == kRandk) odd = (vo >> lane) & 1u;
        if (odd) {
            const float4 a = ld4<VEC>(gi, j, d);
            if (key_of(a.x) >= kInfKey) o.x = __fsub_rn(a.x, a.x);
            if (key_of(a.y) >= kInfKey) o.y = __fsub_rn(a.y, a.y);
            if (key_of(a.z) >= kInfKey) o.z = __fsub_rn(a.z, a.z);
            if (key_of(a.w) >= kInfKey) o.w = __fsub_rn(a.w, a.w);
        }
    }
    st4<VEC, true>(xi, j, d, o);
}

}  // namespace liec
