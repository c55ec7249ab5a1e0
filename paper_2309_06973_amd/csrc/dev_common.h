// Device helpers shared by the kernels (wave64, gfx950).
#pragma once

#include "internal.h"

namespace shifter {

// Largest t with prefix[t] <= tile; requires prefix[0] <= tile < prefix[n].
// `tile` is uniform over the block, so the search runs on scalar registers.
__device__ __forceinline__ uint32_t find_tensor(const uint32_t* __restrict__ prefix,
                                                uint32_t n, uint32_t tile) {
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (prefix[mid] <= tile) lo = mid; else hi = mid;
    }
    return lo;
}

// Bins of the sample histogram of the single-pass selections: SAMPLE_BINS bins of 2^15 keys
// (1/256 of a binade, 0.27 % of a magnitude) over the 64 binades from 2^-50 to 2^14, where
// the weights of networks live; the keys below that window (zeros among them) share bin 0,
// the keys above it the last bin.  The intervals predicted from the sample are rounded
// outward to whole bins, so narrow bins mean few candidates; no result depends on the
// binning (weights all outside the window only send the selection to its multi-pass form).
constexpr uint32_t SAMPLE_BIN_SHIFT = 15;
constexpr uint32_t SAMPLE_KEY0 = (127u - 50u) << 23;      // first key of the window
static_assert(((uint64_t)SAMPLE_BINS << SAMPLE_BIN_SHIFT) == (64ull << 23), "64 binades");
__device__ __forceinline__ uint32_t sample_bin(uint32_t key) {
    return key < SAMPLE_KEY0 ? 0u : min((key - SAMPLE_KEY0) >> SAMPLE_BIN_SHIFT, SAMPLE_BINS - 1u);
}
__device__ __forceinline__ uint32_t sample_bin_first_key(uint32_t bin) {
    return bin == 0u ? 0u : SAMPLE_KEY0 + (bin << SAMPLE_BIN_SHIFT);
}
__device__ __forceinline__ uint32_t sample_bin_last_key(uint32_t bin) {
    return bin >= SAMPLE_BINS - 1u ? 0x7fffffffu : SAMPLE_KEY0 + ((bin + 1u) << SAMPLE_BIN_SHIFT) - 1u;
}

// A value that is the same in every lane, moved to scalar registers.  The builtin returns
// a signed int: without the casts the low word of a 64-bit value would be sign-extended.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
    return ((uint64_t)uniform_u32((uint32_t)(x >> 32)) << 32) | (uint64_t)uniform_u32((uint32_t)x);
}

// Small-quotient division used to index tile-relative flag slots.  The host sets
// magic = floor(2^32 / d) + 1 when 1 < d <= 2 * TILE (exact while x * d < 2^32, and here
// x < d + TILE + 2); for larger d the callers guarantee x < 2 * d.
__device__ __forceinline__ uint32_t div_small(uint32_t x, uint32_t d, uint32_t magic) {
    return d == 1 ? x : (magic ? __umulhi(x, magic) : (x >= d ? 1u : 0u));
}
__device__ __forceinline__ uint32_t mod_small(uint32_t x, uint32_t d, uint32_t magic) {
    return d == 1 ? 0u : (magic ? x - __umulhi(x, magic) * d : (x >= d ? x - d : x));
}

// 16-byte and 4-byte global accesses with an optional non-temporal (streaming) hint:
// arenas larger than the last-level cache are read once and written once per pass, and
// the hint gains about 8 % of copy bandwidth on this chip.
// Weights need no more than the 4-byte alignment every fp32 element has, mask bytes none at
// all: the memory system takes these accesses at any such address, so a full tile of a
// tensor at an odd offset (a network that was pruned before has little else) goes the same
// way as an aligned one.  Counting and masking eight variants of 10 M weights at odd offsets:
// 71 + 83 us with one 4-byte access per weight, 29 + 79 us with these.
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32_a1 __attribute__((aligned(1)));
template <bool NT>
__device__ __forceinline__ uint4 load_u4(const float* p) {
    const u32x4_a4* q = reinterpret_cast<const u32x4_a4*>(p);
    const u32x4_a4 v = NT ? __builtin_nontemporal_load(q) : *q;
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool NT>
__device__ __forceinline__ void store_u4(float* p, uint4 v) {
    u32x4_a4 x;
    x.x = v.x; x.y = v.y; x.z = v.z; x.w = v.w;
    u32x4_a4* q = reinterpret_cast<u32x4_a4*>(p);
    if (NT) __builtin_nontemporal_store(x, q); else *q = x;
}
template <bool NT>
__device__ __forceinline__ void store_mask4(uint8_t* p, uint32_t v) {
    u32_a1* q = reinterpret_cast<u32_a1*>(p);
    if (NT) __builtin_nontemporal_store(v, q); else *q = v;
}
__device__ __forceinline__ void store_mask16(uint8_t* p, uint4 v) {
    u32x4_a1 x;
    x.x = v.x; x.y = v.y; x.z = v.z; x.w = v.w;
    *reinterpret_cast<u32x4_a1*>(p) = x;
}

// What the blocks of a launch leave for the one that ends last: accesses at device scope, past the
// L2 of their chiplet, and a wait for a wavefront's own before its block draws its ticket.  A
// fence at device scope writes the whole L2 back instead: with one per block the finish of fifteen
// ranks took 142 us, 18 without.
__device__ __forceinline__ void store_device(uint2* p, uint2 v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), ((unsigned long long)v.y << 32) | v.x, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint2 load_device(const uint2* p) {
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// True in the block that is the last of `blocks` to call this.  Contains barriers; s_last: a word of LDS.
__device__ __forceinline__ bool last_block(uint32_t* ticket, uint32_t blocks, uint32_t* s_last) {
    wait_memory();
    __syncthreads();
    if (threadIdx.x == 0) *s_last = atomicAdd(ticket, 1u) == blocks - 1u;
    __syncthreads();
    return *s_last != 0;
}

__device__ __forceinline__ uint32_t key_of(float w) {
    return __float_as_uint(w) & 0x7fffffffu;
}

// Exclusive scan of one u64 per thread over a block of THREADS threads.
// smem: at least THREADS / 64 + 1 entries.  Contains two barriers.
template <uint32_t THREADS = BLOCK>
__device__ __forceinline__ uint64_t block_excl_scan_u64(uint64_t v, uint64_t* smem,
                                                        uint64_t* total) {
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    unsigned long long x = v;
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    __syncthreads();   // protects smem against a previous use
    if (lane == 63) smem[wid] = x;
    __syncthreads();
    uint64_t woff = 0, tot = 0;
    for (uint32_t i = 0; i < THREADS / 64; ++i) {
        const uint64_t s = smem[i];
        if (i < wid) woff += s;
        tot += s;
    }
    *total = tot;
    return woff + x - v;
}

// Adds one to h[bin] for every lane with `want`.  Ties make lanes meet at one bin, where an LDS
// atomic takes a turn per lane: the lanes that share the first one's bin go as one addition.
__device__ __forceinline__ void lds_count(uint32_t* h, uint32_t bin, bool want) {
    const uint64_t todo = __ballot(want);
    if (todo == 0ull) return;
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)bin, (int)__ffsll((unsigned long long)todo) - 1);
    const bool same = want && bin == first;
    const uint64_t peers = __ballot(same);
    if (want && !same) atomicAdd(&h[bin], 1u);
    if (same && (peers & ((1ull << (threadIdx.x & 63u)) - 1ull)) == 0ull) atomicAdd(&h[first], (uint32_t)__popcll(peers));
}

// The thread's number, worked out where it is asked for: addresses that follow from it are not kept in registers
// around a loop (26 of them spilled in the kernel that ranks lists in a loop over the ranks).
__device__ __forceinline__ uint32_t this_thread() {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// f(valid, pair) for the n pairs at src, which starts on 16 bytes and has room for an even number
// of them; DEPTH loads of two pairs per thread in flight; every thread of the block makes the same
// calls.  A list that these loads cover is kept in registers from one walk to the next.
template <uint32_t THREADS, uint32_t DEPTH>
struct PairWalk {
    const uint4* __restrict__ src;
    uint32_t n, tid;
    uint4 c[DEPTH];
    __device__ __forceinline__ PairWalk(const uint2* __restrict__ pairs, uint32_t count, uint32_t thread)
        : src(reinterpret_cast<const uint4*>(pairs)), n(count), tid(thread) { fetch(0); }
    __device__ __forceinline__ void fetch(uint32_t i0) {
#pragma unroll
        for (uint32_t u = 0; u < DEPTH; ++u) {
            const uint32_t i = i0 + 2u * (u * THREADS + tid);
            c[u] = src[(n ? min(i, n - 1u) : 0u) / 2u];       // behind the end: the last ones again
        }
    }
    template <typename F>
    __device__ __forceinline__ void operator()(F&& f) {
        for (uint32_t i0 = 0; i0 < n; i0 += 2u * THREADS * DEPTH) {
            if (n > 2u * THREADS * DEPTH) fetch(i0);
#pragma unroll
            for (uint32_t u = 0; u < DEPTH; ++u) {
                const uint32_t i = i0 + 2u * (u * THREADS + tid);
                if (i0 + 2u * u * THREADS < n) {
                    f(i < n, make_uint2(c[u].x, c[u].y));
                    f(i + 1u < n, make_uint2(c[u].z, c[u].w));
                }
            }
        }
    }
};

// The r-th smallest (1-based) of n distinct pairs (bits, global index) in the order (|bits|,
// index), by one block.  All n lie in the window of 2^width composites (|bits| << 32 | index)
// from c_lo on, width <= 63.  4096-bin histograms of the composite narrow the window, first over
// the key, then, where that many weights share it, over the index; a window of at most
// RANK_DIRECT pairs is ranked by counting.  Afterwards sh.sel is the pair and, if count, sh.lt
// and sh.eq are the numbers of pairs in the list with a smaller and with the same key.  Returns
// false if the list does not hold r pairs of the window.
constexpr uint32_t RANK_BINS = 4096, RANK_DIRECT = 96;
template <uint32_t THREADS>
struct RankShared {
    uint32_t h[RANK_BINS];
    uint64_t comp[RANK_DIRECT];
    uint64_t smem[THREADS / 64 + 1];
    uint64_t sel, base;
    uint32_t bin, cnt, nb, lt, eq;
};
template <uint32_t THREADS, uint32_t DEPTH>
__device__ bool rank_in_list(const uint2* __restrict__ src, uint32_t n, uint64_t c_lo, uint32_t width,
                             uint64_t r, bool count, RankShared<THREADS>& sh) {
    auto composite = [](uint2 c) { return ((uint64_t)(c.x & 0x7fffffffu) << 32) | c.y; };
    uint32_t in_window = n, below = 0;          // pairs in the window, pairs of the list below it
    const uint32_t tid = this_thread();
    PairWalk<THREADS, DEPTH> walk(src, n, tid);
    if (tid == 0) { sh.sel = 0; sh.nb = 0; sh.lt = 0; sh.eq = 0; }
    while (in_window > RANK_DIRECT) {
        if (width == 0) return false;           // composites are distinct: cannot happen
        const uint32_t shift = width >= 44u ? width - 12u : (width > 32u ? 32u : (width > 12u ? width - 12u : 0u));
        for (uint32_t i = tid; i < RANK_BINS; i += THREADS) sh.h[i] = 0;
        __syncthreads();
        walk([&](bool valid, uint2 c) {
            const uint64_t d = composite(c) - c_lo;               // wraps for pairs below the window
            lds_count(sh.h, (uint32_t)(d >> shift) & (RANK_BINS - 1u), valid && (d >> width) == 0);
        });
        __syncthreads();
        constexpr uint32_t PER = RANK_BINS / THREADS;
        uint32_t c[PER];
        uint64_t sum = 0, tot;
#pragma unroll
        for (uint32_t i = 0; i < PER; ++i) { c[i] = sh.h[tid * PER + i]; sum += c[i]; }
        uint64_t base = block_excl_scan_u64<THREADS>(sum, sh.smem, &tot);
        if (tot < r) return false;
#pragma unroll
        for (uint32_t i = 0; i < PER; ++i) {
            if (base < r && r <= base + c[i]) { sh.bin = tid * PER + i; sh.cnt = c[i]; sh.base = base; }
            base += c[i];
        }
        __syncthreads();
        r -= sh.base;
        below += (uint32_t)sh.base;
        c_lo += (uint64_t)sh.bin << shift;
        width = shift;
        in_window = sh.cnt;
        __syncthreads();
    }
    __syncthreads();
    walk([&](bool valid, uint2 c) {
        const uint64_t comp = composite(c);
        if (valid && ((comp - c_lo) >> width) == 0) {
            const uint32_t pos = atomicAdd(&sh.nb, 1u);
            if (pos < RANK_DIRECT) sh.comp[pos] = comp;
        }
    });
    __syncthreads();
    if (sh.nb != in_window || r == 0 || r > in_window) return false;
    for (uint32_t i = tid; i < in_window; i += THREADS) {
        const uint64_t c = sh.comp[i];
        uint32_t rank = 0;
        for (uint32_t f = 0; f < in_window; ++f) rank += sh.comp[f] < c;
        if (rank == r - 1) sh.sel = c;          // composites are distinct: exactly one hit
    }
    __syncthreads();
    if (!count) return true;
    const uint32_t key = (uint32_t)(sh.sel >> 32);
    uint32_t lt = 0, eq = 0;
    if (width >= 32u) {                         // the window holds whole keys
        for (uint32_t i = tid; i < in_window; i += THREADS) {
            const uint32_t k = (uint32_t)(sh.comp[i] >> 32);
            lt += k < key;
            eq += k == key;
        }
        if (tid == 0) lt += below;
    } else {                                    // it is a part of one key's indices
        walk([&](bool valid, uint2 c) {
            const uint32_t k = c.x & 0x7fffffffu;
            lt += valid && k < key;
            eq += valid && k == key;
        });
        for (uint32_t d = 32; d > 0; d >>= 1) { lt += __shfl_down(lt, d, 64); eq += __shfl_down(eq, d, 64); }
        if ((tid & 63u) != 0) lt = eq = 0;
    }
    if (lt) atomicAdd(&sh.lt, lt);
    if (eq) atomicAdd(&sh.eq, eq);
    __syncthreads();
    return true;
}

}  // namespace shifter
