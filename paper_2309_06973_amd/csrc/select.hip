// Exact multi-rank selection of the P-th smallest (|w|, g) pair: the unstructured
// magnitude ranking of Sec. II-A / Sec. III-C of the paper in the form that needs no decision
// on the host, for any number of prune counts, any distribution and any number of ties.
//
//   top     one read of the arena: a histogram of all keys on the 16384 bins of sample_bin
//           (1/256 of a binade where the weights of networks live), zeros counted apart;
//   stage   every rank has a window of composites (key << 32 | g) that holds its pair and the
//           number of weights in it.  A stage reads the arena once: windows of no more pairs
//           than are good in a list (sel_plan.h) are written out as lists, the others are split by
//           a further histogram, first by key down to a single key, then by index;
//   final   one block per rank ranks its list and writes the record.
//
// The first stage lists the ranks whose top bin holds no more than a list: 65536 pairs, in a
// flat run's scratch 2^19 / K if that is less.  A bin of normally distributed weights holds up to 0.2 % of
// them, so 10 counts of 25 M weights, or 20 of 13 M, are read three times with no ties at all, fewer twice.
//
// The launches are the same for every input (their number follows from N and K alone), so the
// calls can be recorded into a graph.  What bounds it: the reads of the arena, and one launch
// after the other around them (about 5 us each, 2 to 5 for a stage with nothing to do).
// Equal weights are what the rest is built around: zeros take a window of their own from the start,
// a window that turns out to hold a single key goes on with its index, a lane keeps counts that would meet at
// one counter, windows that follow each other in one bin are found by halving.  us a call, flat
// run, the radix select of 11 + 10 + 10 bits with one read per distinct key for the ties that this
// replaces / lists of up to 2^20 pairs and none of these / now:
//   counts of weights     normal              half of them zero     all equal             30 levels a sigma
//    1 of   1 M           85 /   35 /   33    88 / 1336 /   59      92 /  121 /   75      89 /  90 /  48
//   10 of   1 M          197 /   38 /   35   140 /  132 /   64     140 /  143 /   82     196 /  93 /  54
//    1 of  14.7 M        174 /   53 /   52   200 /  273 /  122     246 /  331 /  188     181 / 685 /  96
//   10 of  14.7 M        418 /   71 /   63   258 /  359 /  146     296 /  421 /  213     390 / 165 / 138
//    1 of 100 M          481 /  175 /  180   723 / 1279 /  508    1210 / 1662 /  857     469 / 617 / 346
//   10 of 100 M         1276 /  312 /  268   850 / 2287 /  801    1261 / 2781 / 1236    1271 / 693 / 596
#include <algorithm>

#include "dev_common.h"

namespace shifter {

constexpr uint32_t SEL_THREADS = 1024;
constexpr uint32_t SEL_GROUPS = SEL_THREADS / BLOCK;   // tiles a block walks side by side
constexpr uint32_t SEL_STAGE_CAP = 4096;               // listed pairs a block collects in LDS
constexpr uint32_t SEL_QUADS = TILE / BLOCK / 4;        // of a full tile per thread
constexpr uint32_t NONE8 = 0xffu;
// What the walk of a stage has to know of a window, in one word: width | shift << 6 | these |
// leader << 16 | windows in its top bin << 24.
constexpr uint32_t SEL_ABOUT_SPLIT = 1u << 12;
constexpr uint32_t SEL_ABOUT_TIES = 1u << 13;     // likely to hold equal weights
constexpr uint32_t SEL_ABOUT_RUNS = 1u << 14;     // many of a wavefront's lanes meet at one counter

// Where the map of windows is looked up: the key's bin, one more for zero.
__device__ __forceinline__ uint32_t top_bin(uint32_t key) { return key ? sample_bin(key) : SEL_BINS; }

__global__ __launch_bounds__(BLOCK) void sel_clear_kernel(SelState* st, uint32_t* ghist, uint32_t hists,
                                                          PruneCounts pc, MultiPerm perm, uint32_t k,
                                                          DevTensor* flat_tens, uint32_t* flat_prefix, uint64_t flat_n,
                                                          uint32_t* zero_ptr, uint32_t zero_n) {
    const uint32_t tid = blockIdx.x * BLOCK + threadIdx.x;
    uint4* g4 = reinterpret_cast<uint4*>(ghist);
    for (uint32_t i = tid; i < hists * (SEL_BINS / 4); i += gridDim.x * BLOCK) g4[i] = make_uint4(0, 0, 0, 0);
    for (uint32_t i = tid; i < zero_n; i += gridDim.x * BLOCK) zero_ptr[i] = 0;
    if (tid < (SEL_STAGES + 1u) * MAXK) {
        (&st->key_lo[0][0])[tid] = 0xffffffffu;
        (&st->key_hi[0][0])[tid] = 0;
    }
    if (tid < MAXK) {
        st->p[tid] = tid < k ? pc.p[tid] : 0;
        st->perm[tid] = tid < k ? perm.v[tid] : 0;
        st->list_cnt[tid] = 0;
        st->fin[tid].mode = SEL_IDLE;
        if (tid <= SEL_STAGES) st->done[tid] = 0;
    }
    if (tid == 0) {
        st->nan_seen = 0;
        st->n_zero = 0;
        if (flat_tens) {
            // a flat run of weights as a one-tensor model: filter 0 of a 1 x n linear layer at
            // element 0, prunable, global index = element index
            DevTensor d;
            d.offset = 0;
            d.gbase = 0;
            d.numel = (uint32_t)flat_n;
            d.out_ch = 1;
            d.in_ch = (uint32_t)flat_n;
            d.khw = 1;
            d.row_len = (uint32_t)flat_n;
            d.kk = 1;
            d.cin = (uint32_t)flat_n;
            d.magic_khw = d.magic_row = d.magic_in = d.magic_kk = d.shift_kk = 0;
            d.out_group = 1;
            d.in_group = 0;
            d.out_flag_off = d.in_flag_off = 0;
            d.prunable = 1;
            d.band_rows = d.chunk_ch = d.src_chunks = 1;
            flat_tens[0] = d;
            flat_prefix[0] = 0;
            flat_prefix[1] = (uint32_t)((flat_n + TILE - 1) / TILE);
        }
    }
}

// whole(bits of a thread's sixteen weights of a full tile, g of the first) and one(bits, g) for the
// prunable weights; the four quads of the sixteen lie 4 * BLOCK weights apart.  Four tiles at a time per block, one per 256 threads,
// a thread's 64 bytes in flight together; no barriers, so the wavefronts drift apart and one's
// loads overlap with another's work.
template <typename Q, typename F>
__device__ __forceinline__ void sel_walk(const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix,
                                         uint32_t n_t, uint32_t n_tiles, const float* __restrict__ w, Q&& whole, F&& one) {
    const uint32_t tid = threadIdx.x & (BLOCK - 1u);
    const uint32_t group = uniform_u32(threadIdx.x / BLOCK);
    for (uint32_t tile = blockIdx.x * SEL_GROUPS + group; tile < n_tiles; tile += gridDim.x * SEL_GROUPS) {
        const uint32_t t = n_t == 1u ? 0u : find_tensor(tile_prefix, n_t, tile);
        if (!tens[t].prunable) continue;
        const uint32_t e0 = (tile - tile_prefix[t]) * TILE;
        const uint32_t n = min(TILE, tens[t].numel - e0);
        const uint32_t g0 = (uint32_t)(tens[t].gbase + e0);
        const float* src = w + tens[t].offset + e0;
        if (n == TILE) {
            uint4 v[SEL_QUADS];
            constexpr uint32_t U = SEL_QUADS;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = load_u4<false>(src + 4u * tid + 4u * BLOCK * u);
            whole(v, g0 + 4u * tid);
        } else {
            for (uint32_t j = tid; j < n; j += BLOCK) one(__float_as_uint(src[j]), g0 + j);
        }
    }
}

// Counts of one histogram entry that a lane has not added to it yet.  Equal weights would have
// all lanes meet at one counter, where an LDS atomic takes a turn per lane.
struct RunCount {
    uint32_t at = 0, n = 0;
    __device__ __forceinline__ void add(uint32_t* h, uint32_t entry, uint32_t c) {
        if (entry != at) { flush(h); at = entry; }
        n += c;
    }
    __device__ __forceinline__ void flush(uint32_t* h) {
        if (n) atomicAdd(&h[at], n);
        n = 0;
    }
};

// Smallest and largest key that a lane has met in a window.
struct KeyRange {
    uint32_t of = 0, lo = 0xffffffffu, hi = 0;
    __device__ __forceinline__ void add(uint32_t* s_lo, uint32_t* s_hi, uint32_t window, uint32_t key) {
        if (window != of) { flush(s_lo, s_hi); of = window; lo = 0xffffffffu; hi = 0; }
        lo = min(lo, key);
        hi = max(hi, key);
    }
    __device__ __forceinline__ void flush(uint32_t* s_lo, uint32_t* s_hi) {
        if (lo <= hi) {
            if (lo < s_lo[of]) atomicMin(&s_lo[of], lo);
            if (hi > s_hi[of]) atomicMax(&s_hi[of], hi);
        }
    }
};

// Zeros, half of the weights or more in a model that was pruned before, are counted apart, a
// counter for each lane.  Four neighbours of one bin (weights that are equal or sorted) are counted as a run.
__global__ __launch_bounds__(SEL_THREADS) void sel_top_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix, uint32_t n_t, uint32_t n_tiles,
    const float* __restrict__ w, SelState* st, uint32_t* ghist) {
    __shared__ uint32_t h[SEL_BINS + 64u];
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t i = threadIdx.x; i < SEL_BINS + 64u; i += SEL_THREADS) h[i] = 0;
    __syncthreads();
    uint32_t key_max = 0, turn = 0;
    bool runs = false;
    RunCount run;
    auto bin_of = [&](uint32_t key) { return key ? sample_bin(key) : SEL_BINS + lane; };
    sel_walk(tens, tile_prefix, n_t, n_tiles, w, [&](const uint4 (&quads)[SEL_QUADS], uint32_t) {
#pragma unroll
        for (uint32_t u = 0; u < SEL_QUADS; ++u) {
            const uint4 v = quads[u];
            const uint32_t k0 = v.x & 0x7fffffffu, k1 = v.y & 0x7fffffffu, k2 = v.z & 0x7fffffffu, k3 = v.w & 0x7fffffffu;
            const uint32_t b0 = bin_of(k0), b1 = bin_of(k1), b2 = bin_of(k2), b3 = bin_of(k3);
            key_max = max(max(key_max, max(k0, k1)), max(k2, k3));
            // every fourth time, until some lane has met a run
            bool same = false;
            if (runs || (turn++ & 3u) == 0u) {
                same = (b0 == b1) & (b1 == b2) & (b2 == b3);
                runs = __ballot(same) != 0ull;
            }
            if (same) {
                run.add(h, b0, 4u);
            } else {
                atomicAdd(&h[b0], 1u);
                atomicAdd(&h[b1], 1u);
                atomicAdd(&h[b2], 1u);
                atomicAdd(&h[b3], 1u);
            }
        }
    }, [&](uint32_t bits, uint32_t) {
        const uint32_t key = bits & 0x7fffffffu;
        key_max = max(key_max, key);
        atomicAdd(&h[bin_of(key)], 1u);
    });
    run.flush(h);
    if (key_max > 0x7f800000u) st->nan_seen = 1;
    __syncthreads();
    if (threadIdx.x < 64u) {
        uint32_t zeros = h[SEL_BINS + lane];
        for (uint32_t d = 32; d > 0; d >>= 1) zeros += __shfl_down(zeros, d, 64);
        if (lane == 0 && zeros) atomicAdd(&st->n_zero, zeros);
    }
    // the blocks start at different segments: the populated bins are few and neighbours
    constexpr uint32_t SEGS = SEL_BINS / SEL_THREADS;
    for (uint32_t it = 0; it < SEGS; ++it) {
        const uint32_t i = ((it + blockIdx.x) % SEGS) * SEL_THREADS + threadIdx.x;
        const uint32_t c = h[i];
        if (c) atomicAdd(&ghist[i], c);
    }
}

// Stage `stage` (1 ..): every block first works out the windows from the histograms of the
// stage before (the same in every block; the first one publishes them), then walks the arena.
__global__ __launch_bounds__(SEL_THREADS) void sel_stage_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix, uint32_t n_t, uint32_t n_tiles,
    const float* __restrict__ w, SelState* st, uint32_t* ghist, uint2* __restrict__ lists, uint32_t list_cap,
    uint32_t k, uint32_t n_weights, uint32_t g_bits, uint32_t stage, uint32_t stages) {
    // bytes of the map: first of the stage's windows, in order, that lies in that top bin
    __shared__ __align__(16) uint8_t s_map[SEL_BINS + 16u];
    __shared__ uint32_t s_hist[SEL_BINS];
    __shared__ __align__(16) uint2 s_pair[SEL_STAGE_CAP];
    __shared__ uint8_t s_of[SEL_STAGE_CAP];
    __shared__ SelWindow s_win[MAXK];
    __shared__ uint64_t s_lo[MAXK];       // of the windows in order: the first composite,
    __shared__ uint32_t s_about[MAXK];    // what else the walk needs
    __shared__ uint64_t smem[SEL_THREADS / 64 + 1];
    __shared__ uint32_t s_cnt[MAXK], s_base[MAXK], s_key_lo[MAXK], s_key_hi[MAXK], s_n, s_left, s_ties;
    if (stage > 1u && st->done[stage - 1u]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->done[stage] = 1;
        return;
    }
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t bits = sel_bits(k);
    if (threadIdx.x < MAXK) {
        SelWindow W;
        W.c_lo = W.r = W.less = W.key_less = W.key_eq = W.cnt = 0;
        W.width = 0; W.leader = threadIdx.x; W.mode = SEL_IDLE; W.stage = 0;
        s_win[threadIdx.x] = W;
        s_cnt[threadIdx.x] = 0;
        s_key_lo[threadIdx.x] = 0xffffffffu;
        s_key_hi[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) { s_n = 0; s_left = 0; s_ties = 0; }
    if (stage == 1u) {
        // sixteen bins per thread, their exclusive prefix over the block (in the room of the
        // pairs), then a search per rank
        uint64_t* base_of = reinterpret_cast<uint64_t*>(s_pair);
        static_assert(sizeof(s_pair) >= sizeof(uint64_t) * SEL_THREADS && SEL_BINS == 16u * SEL_THREADS, "prefix");
        const uint4* h4 = reinterpret_cast<const uint4*>(ghist) + threadIdx.x * 4u;
        uint64_t sum = 0, tot;
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) { const uint4 x = h4[i]; sum += (uint64_t)x.x + x.y + x.z + x.w; }
        const uint64_t n_zero = st->n_zero;
        base_of[threadIdx.x] = n_zero + block_excl_scan_u64<SEL_THREADS>(sum, smem, &tot);
        __syncthreads();
        if (threadIdx.x < k) {
            const uint64_t r = st->p[threadIdx.x];
            SelWindow W;
            W.c_lo = W.less = W.key_less = W.key_eq = 0;
            W.leader = threadIdx.x;
            W.mode = SEL_SPLIT;
            W.stage = 0;
            if (r != 0 && r <= n_zero) {                      // among the zeros, a window of one key
                W.r = r;
                W.key_eq = W.cnt = n_zero;
                W.width = 32u;
                s_win[threadIdx.x] = W;
            } else if (r != 0 && r <= n_zero + tot) {
                uint32_t a = 0, b = SEL_THREADS;              // last thread whose base is below r
                while (b - a > 1u) {
                    const uint32_t m = (a + b) >> 1;
                    if (base_of[m] < r) a = m; else b = m;
                }
                uint64_t base = base_of[a];
                const uint32_t* hb = ghist + a * 16u;
                uint32_t c[16];
#pragma unroll
                for (uint32_t i = 0; i < 16u; ++i) c[i] = hb[i];
                uint32_t bin = 0, cnt = 0;
                uint64_t below = 0;
#pragma unroll
                for (uint32_t i = 0; i < 16u; ++i) {
                    if (base < r && r <= base + c[i]) { bin = a * 16u + i; cnt = c[i]; below = base; }
                    base += c[i];
                }
                // the bins at both ends of the binning span up to 2^30 keys; zeros are not in theirs
                W.c_lo = (uint64_t)max(sample_bin_first_key(bin), 1u) << 32;
                W.width = (bin == 0u || bin == SAMPLE_BINS - 1u) ? SEL_MAX_WIDTH : 32u + SAMPLE_BIN_SHIFT;
                W.r = r - below;
                W.less = below;
                W.cnt = cnt;
                s_win[threadIdx.x] = W;
            }
        }
    } else {
        // one wavefront per rank: the bin of its leader's histogram that holds its pair
        __syncthreads();
        const uint32_t nb = 1u << bits, per = nb / 64u;       // 4 .. 64 bins per lane
        for (uint32_t q = wid; q < k; q += SEL_THREADS / 64u) {
            const SelWindow W = st->win[stage - 1u][q];
            if (W.mode != SEL_SPLIT) continue;
            const uint32_t key = st->key_lo[stage - 1u][W.leader];
            if (W.stage != 0u && W.width > 32u && key == st->key_hi[stage - 1u][W.leader]) {
                // all its weights are equal: on with the index
                if (lane == 0) {
                    SelWindow V = W;
                    V.c_lo = (uint64_t)key << 32;
                    V.width = 32u;
                    V.key_less = W.less;
                    V.key_eq = W.cnt;
                    s_win[q] = V;
                }
                continue;
            }
            const uint32_t* hist = ghist + (size_t)(stage - 1u) * SEL_BINS + W.leader * nb + lane * per;
            uint64_t sum = 0;
            for (uint32_t i = 0; i < per; ++i) sum += hist[i];
            unsigned long long incl = sum;
            for (uint32_t d = 1; d < 64; d <<= 1) {
                const unsigned long long y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            uint64_t base = incl - sum;
            if (base < W.r && W.r <= incl) {
                uint32_t i = 0, c = hist[0];
                while (W.r > base + c) { base += c; c = hist[++i]; }
                const uint32_t shift = sel_shift(W.width, bits, g_bits);
                SelWindow V = W;
                V.c_lo = W.c_lo + ((uint64_t)(lane * per + i) << shift);
                V.r = W.r - base;
                V.less = W.less + base;
                V.cnt = c;
                V.width = shift;
                if (shift == 32u) { V.key_less = V.less; V.key_eq = c; }
                s_win[q] = V;
            }
        }
    }
    // no window in a top bin yet
    static_assert(SEL_BINS == 16u * SEL_THREADS, "one 16-byte piece of the map per thread");
    reinterpret_cast<uint4*>(s_map)[threadIdx.x] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (threadIdx.x == 0) s_map[SEL_BINS] = (uint8_t)NONE8;
    for (uint32_t i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) s_hist[i] = 0;
    __syncthreads();
    // the windows in order: the ranks are sorted, so equal windows are neighbours (the first rank
    // leads) and those in one top bin follow each other
    if (wid == 0) {
        const SelWindow W = s_win[lane];
        const bool live = W.mode == SEL_SPLIT;
        const uint64_t prev_lo = __shfl_up((unsigned long long)W.c_lo, 1, 64);
        const uint32_t prev_live = __shfl_up(live ? 1u : 0u, 1, 64), prev_w = __shfl_up(W.width, 1, 64);
        const bool opens = live && !(lane > 0u && prev_live && prev_lo == W.c_lo && prev_w == W.width);
        const unsigned long long open_mask = __ballot(opens);
        const unsigned long long upto = open_mask & (~0ull >> (63u - lane));
        const uint32_t leader = upto ? 63u - (uint32_t)__clzll(upto) : lane;
        const uint32_t top = top_bin((uint32_t)(W.c_lo >> 32));
        const unsigned long long before = open_mask & ((1ull << lane) - 1ull);
        const uint32_t prev_top = __shfl(top, before ? 63 - __clzll((long long)before) : 0, 64);
        const bool first = opens && !(before && prev_top == top);
        const unsigned long long first_mask = __ballot(first);
        const unsigned long long behind = lane == 63u ? 0ull : first_mask & (~0ull << (lane + 1u));
        const unsigned long long here = behind ? (1ull << (__ffsll(behind) - 1)) - 1ull : ~0ull;   // lanes before the next top bin
        const uint32_t in_top = (uint32_t)__popcll(open_mask & here & (~0ull << lane));
        if (live) {
            const uint32_t mode = W.cnt <= (stage < stages ? min(list_cap, SEL_LIST_GOOD) : list_cap) ? SEL_LISTED : SEL_SPLIT;
            s_win[lane].leader = leader;
            s_win[lane].mode = mode;
            // more weights than any spread-out distribution has in 1/256 of a binade, or one key
            const bool ties = W.width <= 32u || W.cnt > (n_weights >> 7);
            s_win[lane].stage = ties ? stage : 0u;
            if (ties) s_ties = 1;
            if (opens) {
                const uint32_t at = (uint32_t)__popcll(before);
                s_lo[at] = W.c_lo;
                s_about[at] = W.width | (sel_shift(W.width, bits, g_bits) << 6) | (mode == SEL_SPLIT ? SEL_ABOUT_SPLIT : 0u) |
                              (ties ? SEL_ABOUT_TIES : 0u) | (W.cnt > (n_weights >> 4) ? SEL_ABOUT_RUNS : 0u) | (lane << 16) | (in_top << 24);
                if (first) s_map[top] = (uint8_t)at;
            }
            if (mode == SEL_SPLIT) s_left = 1;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0) {
        if (threadIdx.x < k) {
            const SelWindow W = s_win[threadIdx.x];
            st->win[stage][threadIdx.x] = W;
            if (W.mode == SEL_LISTED) st->fin[threadIdx.x] = W;
        }
        if (threadIdx.x == 0) st->done[stage] = s_left ? 0u : 1u;
    }
    RunCount run;
    KeyRange keys;
    auto one = [&](uint32_t wbits, uint32_t g) {
        const uint32_t key = wbits & 0x7fffffffu;
        uint32_t i = s_map[top_bin(key)];
        if (i == NONE8) return;
        const uint64_t comp = ((uint64_t)key << 32) | g;
        uint32_t about = s_about[i];
        if (about >= 2u << 24) {                    // several windows in this top bin: the last that begins by here
            for (uint32_t n = about >> 24; n > 1u;) {
                const uint32_t half = n >> 1;
                if (s_lo[i + half] <= comp) { i += half; n -= half; } else { n = half; }
            }
            about = s_about[i];
        }
        const uint64_t d = comp - s_lo[i];
        if ((d >> (about & 63u)) != 0) return;
        const uint32_t s = (about >> 16) & 0xffu;
        if (about & SEL_ABOUT_SPLIT) {
            const uint32_t entry = (s << bits) + (uint32_t)(d >> ((about >> 6) & 63u));
            if (about & SEL_ABOUT_RUNS) run.add(s_hist, entry, 1u); else atomicAdd(&s_hist[entry], 1u);
            if (about & SEL_ABOUT_TIES) keys.add(s_key_lo, s_key_hi, s, key);
            return;
        }
        // one reservation for the lanes that list a pair now, if they are many
        uint32_t pos = 0;
        const uint64_t all = __ballot(true);
        if (__popcll(all) > 16) {
            const uint32_t before = (uint32_t)__popcll(all & ((1ull << lane) - 1ull));
            if (before == 0) pos = atomicAdd(&s_n, (uint32_t)__popcll(all));
            pos = __shfl(pos, (int)__ffsll((unsigned long long)all) - 1, 64) + before;
        } else {
            pos = atomicAdd(&s_n, 1u);
        }
        if (pos < SEL_STAGE_CAP) {
            s_pair[pos] = make_uint2(wbits, g);
            s_of[pos] = (uint8_t)s;
            return;
        }
        if (about & SEL_ABOUT_TIES) keys.add(s_key_lo, s_key_hi, s, key);
        // more than the block's share (weights that are sorted or clustered by size): straight
        // to the list, one reservation for the lanes that meet at it
        // (the base comes to a lane by its own group's leader: the compiler may take the end of
        // the loop's body for all groups at once)
        uint64_t peers = 0;
        for (bool found = false; !found;) {
            const uint32_t first = uniform_u32(s);
            const uint64_t same = __ballot(s == first);
            if (s == first) { peers = same; found = true; }
        }
        const uint32_t rank = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
        uint32_t base = 0;
        if (rank == 0) base = atomicAdd(&st->list_cnt[s], (uint32_t)__popcll(peers));
        const uint32_t at = __shfl(base, (int)__ffsll((unsigned long long)peers) - 1, 64) + rank;
        if (at < list_cap) lists[(size_t)s * list_cap + at] = make_uint2(wbits, g);
    };
    sel_walk(tens, tile_prefix, n_t, n_tiles, w, [&](const uint4 (&v)[SEL_QUADS], uint32_t g) {
        // first which of the sixteen are met by a window, without a branch, then those one by one: few are,
        // and the long body stands here once (in line sixteen times: 20 ranks of 14.7 M weights 34 us, 24 so; 30
        // levels a sigma, one rank of 100 M 134 and 92; all 100 M equal 170 and 265)
        static_assert(SEL_QUADS == 4u, "sixteen weights");
        uint32_t met = 0;
#pragma unroll
        for (uint32_t u = 0; u < 4u; ++u) {
            const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) met |= (s_map[top_bin(x[q] & 0x7fffffffu)] != NONE8 ? 1u : 0u) << (4u * u + q);
        }
        while (met) {
            const uint32_t j = (uint32_t)__builtin_ctz(met);
            met &= met - 1u;
            const uint32_t u = j >> 2, q = j & 3u;
            const uint4 lo = (u & 1u) ? v[1] : v[0], hi = (u & 1u) ? v[3] : v[2], x = (u & 2u) ? hi : lo;
            const uint32_t a = (q & 1u) ? x.y : x.x, b = (q & 1u) ? x.w : x.z;
            one((q & 2u) ? b : a, g + 4u * BLOCK * u + q);
        }
    }, one);
    run.flush(s_hist);
    keys.flush(s_key_lo, s_key_hi);
    __syncthreads();
    constexpr uint32_t PER = SEL_STAGE_CAP / SEL_THREADS;
    const uint32_t n = min(s_n, SEL_STAGE_CAP);
    if (s_ties) {
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u) {
            const uint32_t i = u * SEL_THREADS + threadIdx.x;
            if (i < n) {
                const uint32_t key = s_pair[i].x & 0x7fffffffu, s = s_of[i];
                if (key < s_key_lo[s]) atomicMin(&s_key_lo[s], key);
                if (key > s_key_hi[s]) atomicMax(&s_key_hi[s], key);
            }
        }
        __syncthreads();
        if (threadIdx.x < k && s_key_lo[threadIdx.x] <= s_key_hi[threadIdx.x]) {
            atomicMin(&st->key_lo[stage][threadIdx.x], s_key_lo[threadIdx.x]);
            atomicMax(&st->key_hi[stage][threadIdx.x], s_key_hi[threadIdx.x]);
        }
    }
    if (s_left) {
        uint32_t* out = ghist + (size_t)stage * SEL_BINS;
        for (uint32_t i = threadIdx.x; i < (k << bits); i += SEL_THREADS) {
            const uint32_t c = s_hist[i];
            if (c) atomicAdd(&out[i], c);
        }
    }
    // the collected pairs: count per list, one reservation each, then the writes
    if (n == 0) return;
    uint32_t pos[PER];
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
        const uint32_t i = u * SEL_THREADS + threadIdx.x;
        pos[u] = i < n ? atomicAdd(&s_cnt[s_of[i]], 1u) : 0u;
    }
    __syncthreads();
    if (threadIdx.x < k && s_cnt[threadIdx.x]) s_base[threadIdx.x] = atomicAdd(&st->list_cnt[threadIdx.x], s_cnt[threadIdx.x]);
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
        const uint32_t i = u * SEL_THREADS + threadIdx.x;
        if (i < n) {
            const uint32_t s = s_of[i], at = s_base[s] + pos[u];
            if (at < list_cap) lists[(size_t)s * list_cap + at] = s_pair[i];
        }
    }
}

// One block per rank: the record from its list.
__global__ __launch_bounds__(SEL_THREADS) void sel_final_kernel(
    const SelState* __restrict__ st, const uint2* __restrict__ lists, uint32_t list_cap, uint32_t g_bits,
    shifter_threshold* __restrict__ thr, shifter_threshold* host_rec, uint32_t* host_nan) {
    __shared__ RankShared<SEL_THREADS> sh;
    const uint32_t q = blockIdx.x;
    shifter_threshold out;
    out.cut = 0; out.t_key = 0; out.reserved = 0; out.g_cut = ~0ull; out.n_less = 0; out.n_equal = 0;
    out.n_prune = st->p[q];
    if (out.n_prune != 0) {
        const SelWindow W = st->fin[q];
        if (W.mode == SEL_LISTED) {
            // the list's own keys are a narrower window; with a single one the index decides
            uint64_t c_lo = W.c_lo, key_less = W.key_less, key_eq = W.key_eq;
            uint32_t width = W.width;
            if (width > 32u && W.stage != 0u) {
                const uint32_t lo = st->key_lo[W.stage][W.leader], hi = st->key_hi[W.stage][W.leader];
                c_lo = (uint64_t)lo << 32;
                width = 32u;
                while (((hi - lo) >> (width - 32u)) != 0u) ++width;
                if (lo == hi) { key_less = W.less; key_eq = W.cnt; }
            }
            const bool one_key = width <= 32u;
            if (width == 32u) width = g_bits;
            // the window's pairs are all in the list: the r-th of them is the pair
            if (rank_in_list<SEL_THREADS, 4>(lists + (size_t)W.leader * list_cap, min((uint32_t)W.cnt, list_cap), c_lo,
                                             width, W.r, !one_key, sh)) {
                out.cut = sh.sel + 1;
                out.t_key = (uint32_t)(sh.sel >> 32);
                out.g_cut = sh.sel & 0xffffffffull;
                // what shares a single key was counted when the window came down to it
                out.n_less = one_key ? key_less : W.less + sh.lt;
                out.n_equal = one_key ? key_eq : sh.eq;
            }
        }
    }
    if (threadIdx.x == 0) {
        thr[st->perm[q]] = out;
        if (host_rec) host_rec[st->perm[q]] = out;
        if (host_nan && q == 0) *host_nan = st->nan_seen;
    }
}

void launch_select(shifter_ctx* ctx, const shifter_model* m, const float* d_w,
                   const PruneCounts& pc, uint32_t k, shifter_threshold* d_thr, bool mirror, uint32_t* zero_ptr,
                   uint32_t zero_n) {
    const auto& b = m->b;
    // the candidate buffer of the single-pass selections is idle here: it holds the lists
    const SelectTables tb{b.tens, b.tile_prefix, (uint32_t)m->t.size(), m->n_tiles, m->info.n_prunable, b.sel, b.ghist,
                          b.cand, (uint64_t)b.cand_cap_sb * SPEC_SUB, nullptr, nullptr, zero_ptr, zero_n,
                          mirror ? b.dev_multi_rec : nullptr, mirror ? b.dev_multi_status : nullptr};
    launch_select_tables(ctx, tb, d_w, pc, k, d_thr);
}

void launch_select_tables(shifter_ctx* ctx, const SelectTables& tb, const float* d_w,
                          const PruneCounts& pc, uint32_t k, shifter_threshold* d_thr) {
    const uint32_t n_t = tb.n_t, n_tiles = tb.n_tiles;
    hipStream_t s = ctx->stream;
    uint32_t idx[MAXK];
    for (uint32_t i = 0; i < k; ++i) idx[i] = i;
    std::stable_sort(idx, idx + k, [&](uint32_t x, uint32_t y) { return pc.p[x] < pc.p[y]; });
    PruneCounts sorted{};
    MultiPerm perm{};
    for (uint32_t i = 0; i < k; ++i) { sorted.p[i] = pc.p[idx[i]]; perm.v[i] = idx[i]; }
    const uint32_t g_bits = sel_g_bits(tb.n_weights), list_cap = sel_list_cap(tb.list_pairs, k);
    const uint32_t stages = sel_stages(tb.n_weights, k, tb.list_pairs);
    const uint32_t grid = std::max(1u, std::min((n_tiles + SEL_GROUPS - 1) / SEL_GROUPS, ctx->hist_grid));
    {
        ProfileScope p(ctx, K_SEL_INIT);
        sel_clear_kernel<<<64, BLOCK, 0, s>>>(tb.sel, tb.ghist, stages, sorted, perm, k, tb.flat_tens, tb.flat_prefix,
                                              tb.n_weights, tb.zero_ptr, tb.zero_n);
    }
    {
        ProfileScope p(ctx, K_HIST0);
        sel_top_kernel<<<grid, SEL_THREADS, 0, s>>>(tb.tens, tb.tile_prefix, n_t, n_tiles, d_w, tb.sel, tb.ghist);
    }
    for (uint32_t stage = 1; stage <= stages; ++stage) {
        ProfileScope p(ctx, K_SEL_STAGE);
        sel_stage_kernel<<<grid, SEL_THREADS, 0, s>>>(tb.tens, tb.tile_prefix, n_t, n_tiles, d_w, tb.sel, tb.ghist,
                                                      tb.lists, list_cap, k, (uint32_t)tb.n_weights, g_bits, stage, stages);
    }
    {
        ProfileScope p(ctx, K_SEL_FINAL);
        sel_final_kernel<<<k, SEL_THREADS, 0, s>>>(tb.sel, tb.lists, list_cap, g_bits, d_thr, tb.host_rec, tb.host_nan);
    }
}

}  // namespace shifter
