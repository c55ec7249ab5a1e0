// The sample of the single-pass selections (one count: spec_select.hip, a portfolio's: spec_multi.hip).
#pragma once

#include <algorithm>

#include "dev_common.h"

namespace shifter {

// The sample: from every quarter (1024 weights) of every sample_tile_stride-th tile one
// 64-byte sector of 16 weights, at a position that rotates with the tile and the quarter.
// Every filter of 1024 or more weights is thus sampled in proportion to its size - the
// sample is stratified by filter, which matters because filters differ in scale by
// orders of magnitude and a sample clustered on few filters misjudges the quantiles.
// A wavefront takes four tiles per step (16 lanes per tile, 4 lanes per sector, one
// float4 each).  The samples go to a per-block LDS histogram first: a global atomic
// costs about 11 ns per lane on one address, and the bins around the mode are hot.
__host__ __device__ __forceinline__ uint32_t sample_sector(uint32_t tile, uint32_t quarter) {
    return (tile * 37u + quarter * 11u) & 63u;
}

constexpr uint32_t SAMPLE_THREADS = 1024;   // sixteen wavefronts on the block's CU keep its loads in flight
constexpr uint32_t SAMPLE_ONE_BLOCK = 512;   // sampled tiles that one block takes alone

struct SampleIn {
    const DevTensor* tens;
    const uint32_t* tile_prefix;
    const uint16_t* tile_tensor;
    uint32_t n_tiles, tile_stride;
    const float* w;
    uint32_t* shist;      // SAMPLE_BINS counts, then the ticket; all zero before and after
};

// Blocks of the kernel that samples and predicts.  Up to SAMPLE_ONE_BLOCK tiles one block needs at most
// four steps of loads, as long as several blocks take to meet at the histogram in global memory (264
// tiles, fifteen ranks: 22.2 us on one block, 21.7 on five), and leaves their atomics out.
// Beyond that one block per CU at most: more shorten the loop, but each flushes its
// histogram with global atomics.
inline uint32_t sample_grid(const shifter_model* m) {
    const uint32_t sampled = (m->n_tiles + m->sample_tile_stride - 1) / m->sample_tile_stride;
    return sampled <= SAMPLE_ONE_BLOCK ? 1u : std::min(256u, (sampled + 63) / 64);   // 64 tiles per block and step
}

inline SampleIn sample_in(const shifter_model* m, const float* d_w) {
    return SampleIn{m->b.tens, m->b.tile_prefix, m->b.tile_tensor, m->n_tiles, m->sample_tile_stride, d_w, m->b.shist};
}

// Every block counts its part of the sample in h (SAMPLE_BINS words of LDS).  True in the block that
// ends last, which goes on with the prediction: in h it finds the inclusive prefix of the whole
// sample's counts.  The histogram in global memory is cleared for the next ranking.
// What bounds it is a chain of latencies: table, tensor and weights behind one another, then the
// prediction on one block.  In the last block of this launch the prediction costs no launch of its own
// (kernel times: one count of 24 k weights 3 + 11 us apart, 6.7 here; of 295 M 13.6 + 11.7 and 19.1;
// a portfolio's on 10 M 7.2 + 11.4 and 16.2, on 0.86 M 7.4 + 12.4 and 16.7, less a launch's gap).
__device__ __forceinline__ bool sample_prefix(const SampleIn& in, uint32_t* h) {
    const DevTensor* __restrict__ tens = in.tens;
    const uint32_t* __restrict__ tile_prefix = in.tile_prefix;
    const uint16_t* __restrict__ tile_tensor = in.tile_tensor;
    const uint32_t n_tiles = in.n_tiles, tile_stride = in.tile_stride;
    const float* __restrict__ w = in.w;
    __shared__ uint32_t s_last, s_seg[64];
    for (uint32_t i = threadIdx.x; i < SAMPLE_BINS; i += SAMPLE_THREADS) h[i] = 0;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = blockIdx.x * (SAMPLE_THREADS / 64) + (threadIdx.x >> 6);
    const uint32_t n_waves = gridDim.x * (SAMPLE_THREADS / 64);
    const uint32_t quarter = (lane >> 2) & 3u, part = lane & 3u;
    // address of this lane's four samples of sampled tile s, or nullptr; the tensor of a
    // tile comes from a table (one load instead of a search per lane)
    auto locate = [&](uint64_t s) -> const float* {
        if (s * tile_stride >= n_tiles) return nullptr;
        const uint32_t tile = (uint32_t)(s * tile_stride);
        const uint32_t t = tile_tensor[tile];
        if (!tens[t].prunable) return nullptr;
        const uint32_t e0 = (tile - tile_prefix[t]) * TILE;
        const uint32_t n = min(TILE, tens[t].numel - e0);
        const uint32_t j = quarter * 1024u + sample_sector(tile, quarter) * 16u + part * 4u;
        return j + 3 < n ? w + tens[t].offset + e0 + j : nullptr;
    };
    auto fetch = [&](const float* p) -> float4 {
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p) {
            if ((reinterpret_cast<uintptr_t>(p) & 15u) == 0) {
                x = *reinterpret_cast<const float4*>(p);
            } else {
                x.x = p[0]; x.y = p[1]; x.z = p[2]; x.w = p[3];
            }
        }
        return x;
    };
    auto count = [&](const float* p, const float4& x) {
        if (!p) return;
        atomicAdd(&h[sample_bin(key_of(x.x))], 1u);
        atomicAdd(&h[sample_bin(key_of(x.y))], 1u);
        atomicAdd(&h[sample_bin(key_of(x.z))], 1u);
        atomicAdd(&h[sample_bin(key_of(x.w))], 1u);
    };
    // two sampled tiles per lane group and step, their loads in flight together
    const uint64_t step = (uint64_t)n_waves * 4;
    for (uint64_t s = (uint64_t)wave * 4 + (lane >> 4); s * tile_stride < n_tiles; s += 2 * step) {
        const float* pa = locate(s);
        const float* pb = locate(s + step);
        const float4 xa = fetch(pa);
        const float4 xb = fetch(pb);
        count(pa, xa);
        count(pb, xb);
    }
    const uint32_t wid = threadIdx.x >> 6;
    constexpr uint32_t SEG = 256, WAVES = SAMPLE_THREADS / 64, PER_WAVE = SAMPLE_BINS / SEG / WAVES;
    static_assert(SAMPLE_BINS == 64u * SEG, "one segment sum per lane");
    __syncthreads();
    uint4 x[PER_WAVE];
    if (gridDim.x == 1) {
#pragma unroll
        for (uint32_t i = 0; i < PER_WAVE; ++i) x[i] = reinterpret_cast<const uint4*>(h + (wid + i * WAVES) * SEG)[lane];
    } else {
        // the blocks start at different segments of the histogram: the populated bins are few
        // and neighbours, and atomics that meet at one address take their turns
        constexpr uint32_t SEGS = SAMPLE_BINS / SAMPLE_THREADS;
        for (uint32_t it = 0; it < SEGS; ++it) {
            const uint32_t i = ((it + blockIdx.x) % SEGS) * SAMPLE_THREADS + threadIdx.x;
            const uint32_t c = h[i];
            if (c) atomicAdd(&in.shist[i], c);
        }
        if (!last_block(&in.shist[SAMPLE_BINS], gridDim.x, &s_last)) return false;
        // each wavefront's segments are loaded once, all loads in flight together, and cleared
#pragma unroll
        for (uint32_t i = 0; i < PER_WAVE; ++i) {
            const uint2* src = reinterpret_cast<const uint2*>(in.shist + (wid + i * WAVES) * SEG) + 2u * lane;
            const uint2 a = load_device(src), b = load_device(src + 1);
            x[i] = make_uint4(a.x, a.y, b.x, b.y);
        }
#pragma unroll
        for (uint32_t i = 0; i < PER_WAVE; ++i)
            reinterpret_cast<uint4*>(in.shist + (wid + i * WAVES) * SEG)[lane] = make_uint4(0, 0, 0, 0);
        if (threadIdx.x == 0) in.shist[SAMPLE_BINS] = 0;
    }
    // inclusive prefix inside each segment, the segments' sums, then their exclusive scan in every
    // wavefront
    uint32_t incl[PER_WAVE];
#pragma unroll
    for (uint32_t i = 0; i < PER_WAVE; ++i) incl[i] = x[i].x + x[i].y + x[i].z + x[i].w;
    for (uint32_t d = 1; d < 64; d <<= 1) {
#pragma unroll
        for (uint32_t i = 0; i < PER_WAVE; ++i) {
            const uint32_t y = __shfl_up(incl[i], d, 64);
            if (lane >= d) incl[i] += y;
        }
    }
    if (lane == 63) {
#pragma unroll
        for (uint32_t i = 0; i < PER_WAVE; ++i) s_seg[wid + i * WAVES] = incl[i];
    }
    __syncthreads();
    const uint32_t mine = s_seg[lane];
    uint32_t upto = mine;
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(upto, d, 64);
        if (lane >= d) upto += y;
    }
#pragma unroll
    for (uint32_t i = 0; i < PER_WAVE; ++i) {
        const uint32_t sg = wid + i * WAVES;
        uint32_t run = __shfl(upto - mine, (int)sg, 64) + incl[i] - (x[i].x + x[i].y + x[i].z + x[i].w);
        uint4 p;
        run += x[i].x; p.x = run;
        run += x[i].y; p.y = run;
        run += x[i].z; p.z = run;
        run += x[i].w; p.w = run;
        reinterpret_cast<uint4*>(h + sg * SEG)[lane] = p;
    }
    __syncthreads();
    return true;
}

// First bin whose prefix exceeds target (the last bin if none does): the bin that holds the sample
// with that 0-based rank.
__device__ __forceinline__ uint32_t sample_bin_of_rank(const uint32_t* prefix, uint32_t target) {
    uint32_t a = 0;       // bins known to have a prefix of at most target
#pragma unroll
    for (uint32_t step = SAMPLE_BINS / 2; step >= 1; step >>= 1)
        if (prefix[a + step - 1] <= target) a += step;
    return a;
}

// The last step of a finish, n distinct composites (at most THREADS of them) of one key: counting for each those below it is
// quadratic, so more than TIED_DIRECT go by the upper bits of their indices first.  Leaves those that share them with
// the one of 0-based rank `want` in `few` and returns their number and the rank among them; the caller meets
// a barrier before.  Ten ranks of 14.7 M weights in half precision, some with hundreds of ties: the finish 30.9 us by counting
// alone, 17.1 so; one count of 14.7 M 114 -> 103 us a step.
constexpr uint32_t TIED_DIRECT = 256;
struct TiedLds {
    uint64_t base;
    uint32_t any, bin, n;
};
template <uint32_t THREADS, uint32_t BINS>
__device__ __forceinline__ uint2 tied_stretch(const uint64_t* comp, uint32_t n, uint32_t want, uint32_t* h, uint64_t* smem,
                                                 uint64_t* few, TiedLds* s) {
    const uint32_t idx = threadIdx.x < n ? (uint32_t)comp[threadIdx.x] : 0u;
    uint32_t any = idx;
    for (uint32_t d = 32; d > 0; d >>= 1) any |= (uint32_t)__shfl_xor((int)any, (int)d, 64);
    constexpr uint32_t PER = BINS / THREADS;
    const uint32_t b0 = threadIdx.x * PER;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) h[b0 + i] = 0;
    if (threadIdx.x == 0) { s->any = 0; s->n = 0; }
    __syncthreads();
    if ((threadIdx.x & 63u) == 0 && any) atomicOr(&s->any, any);
    __syncthreads();
    static_assert(BINS == 1u << 12, "twelve bits a bin");
    const uint32_t bits = 32u - (uint32_t)__clz((int)s->any), sh = bits > 12u ? bits - 12u : 0u;
    if (threadIdx.x < n) atomicAdd(&h[idx >> sh], 1u);
    __syncthreads();
    uint32_t c[PER];
    uint64_t sum = 0, tot;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) { c[i] = h[b0 + i]; sum += c[i]; }
    uint64_t base = block_excl_scan_u64<THREADS>(sum, smem, &tot);
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        if (base <= want && want < base + c[i]) { s->bin = b0 + i; s->base = base; }
        base += c[i];
    }
    __syncthreads();
    if (threadIdx.x < n && (idx >> sh) == s->bin) few[atomicAdd(&s->n, 1u)] = comp[threadIdx.x];
    __syncthreads();
    return make_uint2(s->n, want - (uint32_t)s->base);
}

}  // namespace shifter
