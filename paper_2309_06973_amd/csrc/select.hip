// Exact multi-rank selection of the P-th smallest (|w|, g) pair: the unstructured
// magnitude ranking of Sec. II-A / Sec. III-C of the paper in the form that needs no decision
// on the host, for any number of prune counts, any distribution and any number of ties.
//
//   top     one read of the arena: a histogram of all keys on 16384 bins (sel_plan.h: 1/512 of a binade where the
//           thresholds of networks lie, 1/64 around), zeros counted apart;
//   stage   every rank has a window of composites (key << 32 | g) that holds its pair and the
//           number of weights in it.  A stage reads the arena once: windows of no more pairs
//           than are good in a list (sel_plan.h) are written out as lists, the others are split by
//           a further histogram, first by key down to a single key, then by index;
//   rest    the stages that are left where the first one has not listed every rank, then one block
//           per rank ranks its list and writes the record.
//
// The first stage lists the ranks whose top bin holds no more than a list: 65536 pairs, in a
// flat run's scratch 2^19 / K if that is less.  A fine bin of normally distributed weights holds up to 0.095 % of
// them, of uniform ones 0.1 %, so 10 counts of up to 50 M weights are read twice where there are no ties.
//
// The launches are the same for every input (their number follows from N and K alone), so the
// calls can be recorded into a graph.  What bounds it: the reads of the arena (100 M weights at 5.6 TB/s), and one launch
// after the other around them: clear, top, stage and rest 4.5 + 14.5 + 19 + 9.5 us on ten counts of 14.7 M.
// Equal weights are what the rest is built around: zeros take a window of their own from the start,
// a window that turns out to hold a single key goes on with its index, a lane keeps counts that would meet at
// one counter, windows that follow each other in one bin are found by halving.  us a call, flat
// run, bins of 1/256 of a binade from 2^-50 to 2^14 and a launch for each stage, used or not / now:
//   counts of weights     normal        half of them zero   all equal       30 levels a sigma   half precision   times 2^-30   60 % 10^-12
//    1 of   1 M           32 / 24       33 / 24             78 / 71         49 / 38             41 / 31          33 / 27       34 / 25
//   10 of   1 M           34 / 25       60 / 57             81 / 79         55 / 45             43 / 33          35 / 31       35 / 28
//    1 of  14.7 M         56 / 42       55 / 43             178 / 182       113 / 108           76 / 54          56 / 61       59 / 45
//   10 of  14.7 M         64 / 46       137 / 131           208 / 208       145 / 150           96 / 62          64 / 98       61 / 63
//    1 of 100 M           249 / 161     246 / 160           850 / 853       399 / 402           273 / 207        245 / 255     198 / 167
//   10 of 100 M           252 / 248     745 / 722           1214 / 1210     605 / 606           298 / 308        252 / 298     276 / 277
// (With all bins 1/512 of a binade, which left out what lies below 2^-25 and above 2^7: the first columns 1 % less, the last two
// 55, 101, 165, 217, 760, 1050 and 29, 72, 59, 203, 255, 960.  With the fine ones from 2^-19 to 2^3 and 1/128 around, the last but
// one 26, 29, 53, 66, 249, 278, but 2 % more on weights of many magnitudes, of which more lie in no fine bin.)
// (The radix select of 11 + 10 + 10 bits before all this: 85 us for 1 of 1 M, 418 for 10 of 14.7 M.)
#include <algorithm>

#include "dev_common.h"

namespace shifter {

constexpr uint32_t SEL_THREADS = 1024;
constexpr uint32_t SEL_GROUPS = SEL_THREADS / BLOCK;   // tiles a block walks side by side
constexpr uint32_t SEL_STAGE_CAP = 4096;               // listed pairs a block collects in LDS
constexpr uint32_t SEL_QUADS = TILE / BLOCK / 4;        // of a full tile per thread
constexpr uint32_t SEL_DEPTH = 8;                       // loads of two listed pairs per thread in flight
constexpr uint32_t NONE8 = 0xffu;
// What the walk of a stage has to know of a window, in one word: width | shift << 6 | these |
// leader << 16 | windows in its top bin << 24.
constexpr uint32_t SEL_ABOUT_SPLIT = 1u << 12;
constexpr uint32_t SEL_ABOUT_TIES = 1u << 13;     // likely to hold equal weights
constexpr uint32_t SEL_ABOUT_RUNS = 1u << 14;     // many of a wavefront's lanes meet at one counter

// The record that removes nothing: of a rank of 0, and of one whose wait ran out (see sel_rest_kernel).
__host__ __device__ __forceinline__ shifter_threshold sel_no_record(uint64_t p) {
    shifter_threshold r;
    r.cut = 0; r.t_key = 0; r.reserved = 0; r.g_cut = ~0ull; r.n_less = 0; r.n_equal = 0;
    r.n_prune = p;
    return r;
}

// A window's place in the map: its bin, one more for those among the zeros.
__device__ __forceinline__ uint32_t top_bin(uint32_t key) { return key ? sel_top_bin(key) : SEL_BINS; }

__global__ __launch_bounds__(BLOCK) void sel_clear_kernel(SelState* st, uint32_t* ghist, uint32_t hists,
                                                          PruneCounts pc, MultiPerm perm, uint32_t k, shifter_threshold* thr,
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
    if (tid < k) thr[perm.v[tid]] = sel_no_record(pc.p[tid]);
    if (tid < MAXK) {
        st->p[tid] = tid < k ? pc.p[tid] : 0;
        st->perm[tid] = tid < k ? perm.v[tid] : 0;
        st->list_cnt[tid] = 0;
        st->fin[tid].mode = SEL_IDLE;
        if (tid <= SEL_STAGES) st->done[tid] = st->ticket[tid] = st->arrived[tid] = 0;
        if (tid < SEL_GO)
            for (uint32_t i = 0; i <= SEL_STAGES; ++i) st->go[i][tid * SEL_GO_WORDS] = 0;
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

struct SelArena {
    const DevTensor* __restrict__ tens;
    const uint32_t* __restrict__ tile_prefix;
    const uint16_t* __restrict__ tile_tensor;     // nullptr: one tensor
    uint32_t n_tiles;
    const float* __restrict__ w;
};

// The weights of one part of several: four tiles at a time per block, one per 256 threads, a thread's 64 bytes in
// flight together; no barriers, so the wavefronts drift apart and one's loads overlap with another's work.
// A tensor's last, ragged tile goes the same way as a full one.
struct SelWalk {
    const SelArena& a;
    uint32_t n, g0;                  // the tile at hand: its weights (0: not prunable) and the first one's global index
    uint4 v[SEL_QUADS];              // sixteen of them: four quads 4 * BLOCK weights apart

    __device__ __forceinline__ explicit SelWalk(const SelArena& arena) : a(arena) {}
    __device__ __forceinline__ uint32_t thread() const { return threadIdx.x & (BLOCK - 1u); }
    __device__ __forceinline__ void fetch(uint32_t tile) {
        n = 0;
        const uint32_t t = a.tile_tensor ? a.tile_tensor[tile] : 0u;
        const DevTensor& T = a.tens[t];
        if (!T.prunable) return;
        const uint32_t e0 = (tile - a.tile_prefix[t]) * TILE;
        n = min(TILE, T.numel - e0);
        g0 = (uint32_t)(T.gbase + e0);
        const float* src = a.w + T.offset + e0;
        if (n == TILE) {
#pragma unroll
            for (uint32_t u = 0; u < SEL_QUADS; ++u) v[u] = load_u4<false>(src + 4u * thread() + 4u * BLOCK * u);
        } else {
            // missing ones read as the last one there is
#pragma unroll
            for (uint32_t u = 0; u < SEL_QUADS; ++u) {
                const uint32_t j = (thread() + BLOCK * u) * 4u;
                auto at = [&](uint32_t q) { return __float_as_uint(src[min(j + q, n - 1u)]); };
                v[u] = make_uint4(at(0), at(1), at(2), at(3));
            }
        }
    }
    // down: from the last tile to the first
    template <typename F>
    __device__ __forceinline__ void run(uint32_t part, uint32_t parts, bool down, F&& f) {
        for (uint32_t i = part * SEL_GROUPS + uniform_u32(threadIdx.x / BLOCK); i < a.n_tiles; i += parts * SEL_GROUPS) {
            fetch(down ? a.n_tiles - 1u - i : i);
            if (n) f();
        }
    }
    // bit 4 u + q: weight q of quad u is there (of a ragged tile's)
    __device__ __forceinline__ uint32_t there() const {
        uint32_t m = 0;
#pragma unroll
        for (uint32_t u = 0; u < SEL_QUADS; ++u) m |= ((1u << min(4u, n - min((thread() + BLOCK * u) * 4u, n))) - 1u) << (4u * u);
        return m;
    }
    // weight j of the sixteen, and its global index
    __device__ __forceinline__ uint32_t bits(uint32_t j) const {
        const uint32_t u = j >> 2, q = j & 3u;
        const uint4 lo = (u & 1u) ? v[1] : v[0], hi = (u & 1u) ? v[3] : v[2], x = (u & 2u) ? hi : lo;
        const uint32_t a = (q & 1u) ? x.y : x.x, b = (q & 1u) ? x.w : x.z;
        return (q & 2u) ? b : a;
    }
    __device__ __forceinline__ uint32_t index(uint32_t j) const {
        return g0 + 4u * thread() + 4u * BLOCK * (j >> 2) + (j & 3u);
    }
};
static_assert(SEL_QUADS == 4u, "sixteen weights");

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
__global__ __launch_bounds__(SEL_THREADS) void sel_top_kernel(const SelArena arena, SelState* st, uint32_t* ghist) {
    __shared__ uint32_t h[SEL_BINS + 64u];
    const uint32_t lane = threadIdx.x & 63u;
    SelWalk walk(arena);
    for (uint32_t i = threadIdx.x; i < SEL_BINS + 64u; i += SEL_THREADS) h[i] = 0;
    __syncthreads();
    uint32_t key_max = 0, turn = 0;              // key_max: of those that are in no fine bin
    bool runs = false;
    RunCount run;
    // Counters by their distance from the first fine one.  A zero's has two upper bits set, which are shifted out of its address and
    // tell it from the keys that are in no fine bin: as signed numbers those alone are SEL_FINE_BINS or more.  One look at the
    // largest of a lane's sixteen finds them, and the wavefront then takes the bins of the quads they are in from sel_top_bin.
    // (That for every weight: 14.7 M 14.7 -> 15.9 us.)
    const uint32_t zero_at = (3u << 30) + SEL_BINS + lane - SEL_BIN_FINE;
    auto counter = [&](uint32_t at) { return reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(h) + ((at << 2) + 4u * SEL_BIN_FINE)); };
    auto any_bin = [&](uint32_t key) {
        key_max = max(key_max, key);
        uint32_t at = sel_top_bin(key) - SEL_BIN_FINE;
        asm("" : "+v"(at));                              // for zeros too: a branch around it takes longer
        return key ? at : zero_at;
    };
    walk.run(blockIdx.x, gridDim.x, false, [&] {
        if (walk.n != TILE) {
            for (uint32_t left = walk.there(); left; left &= left - 1u) {
                const uint32_t key = walk.bits((uint32_t)__builtin_ctz(left)) & 0x7fffffffu;
                atomicAdd(counter(any_bin(key)), 1u);
            }
            return;
        }
        uint32_t at[SEL_QUADS][4];
        int32_t most = 0;
#pragma unroll
        for (uint32_t u = 0; u < SEL_QUADS; ++u) {
            const uint32_t x[4] = {walk.v[u].x, walk.v[u].y, walk.v[u].z, walk.v[u].w};
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t key = x[q] & 0x7fffffffu;
                at[u][q] = key ? sel_fine_bin(key) : zero_at;
                most = max(most, (int32_t)at[u][q]);
            }
        }
        if (__builtin_expect(__ballot(most >= (int32_t)SEL_FINE_BINS) != 0ull, 0)) {
#pragma unroll
            for (uint32_t u = 0; u < SEL_QUADS; ++u) {
                const int32_t of_quad = max(max((int32_t)at[u][0], (int32_t)at[u][1]), max((int32_t)at[u][2], (int32_t)at[u][3]));
                if (__ballot(of_quad >= (int32_t)SEL_FINE_BINS) == 0ull) continue;
                const uint32_t x[4] = {walk.v[u].x, walk.v[u].y, walk.v[u].z, walk.v[u].w};
#pragma unroll
                for (uint32_t q = 0; q < 4u; ++q) at[u][q] = any_bin(x[q] & 0x7fffffffu);
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < SEL_QUADS; ++u) {
            const uint32_t b0 = at[u][0], b1 = at[u][1], b2 = at[u][2], b3 = at[u][3];
            // every fourth time, until some lane has met a run
            bool same = false;
            if (runs || (turn++ & 3u) == 0u) {
                same = (b0 == b1) & (b1 == b2) & (b2 == b3);
                runs = __ballot(same) != 0ull;
            }
            if (same) {
                run.add(h, (b0 + SEL_BIN_FINE) & ~(3u << 30), 4u);
            } else {
                atomicAdd(counter(b0), 1u);
                atomicAdd(counter(b1), 1u);
                atomicAdd(counter(b2), 1u);
                atomicAdd(counter(b3), 1u);
            }
        }
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

// Stores of what the blocks of one launch leave each other (DEV: past the L2 of their chiplet; the readers drop what theirs
// holds when they have waited, see sel_rest_kernel), or of what one launch leaves the next.
template <bool DEV>
__device__ __forceinline__ void sel_put(uint32_t* p, uint32_t v) {
    if (DEV) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); else *p = v;
}
template <bool DEV>
__device__ __forceinline__ void sel_put(uint2* p, uint2 v) {
    if (DEV) store_device(p, v); else *p = v;
}
static_assert(sizeof(SelWindow) % 8 == 0, "moved by eight bytes");
template <bool DEV>
__device__ __forceinline__ void sel_put(SelWindow* p, const SelWindow& W) {
    if (!DEV) { *p = W; return; }
#pragma unroll
    for (uint32_t i = 0; i < sizeof(SelWindow) / 8u; ++i)
        store_device(reinterpret_cast<uint2*>(p) + i, reinterpret_cast<const uint2*>(&W)[i]);
}

struct SelShared {
    // bytes of the map: first of the stage's windows, in order, that lies in that top bin
    alignas(16) uint8_t map[SEL_BINS + 16u];
    uint32_t hist[SEL_BINS];
    alignas(16) uint2 pair[SEL_STAGE_CAP];
    uint8_t of[SEL_STAGE_CAP];
    SelWindow win[MAXK];
    uint64_t lo[MAXK];       // of the windows in order: the first composite,
    uint32_t about[MAXK];    // what else the walk needs
    uint64_t smem[SEL_THREADS / 64 + 1];
    uint32_t cnt[MAXK], base[MAXK], key_lo[MAXK], key_hi[MAXK], n, left, ties, wide;
};

// What the stages and the ranking of the lists work on.
struct SelJob {
    SelState* st;
    uint32_t* ghist;
    uint2* lists;
    uint32_t list_cap, k, n_weights, g_bits, stages, polls;
};

// The windows of a stage from the histograms of the stage before: the same in every block, and one of them publishes
// them.
template <bool FIRST, bool DEV>
__device__ __forceinline__ void sel_windows(const SelJob& J, SelShared& S, uint32_t stage, bool publish) {
    SelState* const st = J.st;
    const uint32_t* const ghist = J.ghist;
    const uint32_t k = J.k, g_bits = J.g_bits, list_cap = J.list_cap, stages = J.stages, n_weights = J.n_weights;
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t bits = sel_bits(k);
    if (threadIdx.x < MAXK) {
        SelWindow W;
        W.c_lo = W.r = W.less = W.key_less = W.key_eq = W.cnt = 0;
        W.width = 0; W.leader = threadIdx.x; W.mode = SEL_IDLE; W.stage = 0;
        S.win[threadIdx.x] = W;
        S.cnt[threadIdx.x] = 0;
        S.key_lo[threadIdx.x] = 0xffffffffu;
        S.key_hi[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) { S.n = 0; S.left = 0; S.ties = 0; S.wide = 0; }
    if (FIRST) {
        // sixteen bins per thread, their exclusive prefix over the block (in the room of the
        // pairs), then a search per rank
        uint64_t* base_of = reinterpret_cast<uint64_t*>(S.pair);
        static_assert(sizeof(SelShared::pair) >= sizeof(uint64_t) * SEL_THREADS && SEL_BINS == 16u * SEL_THREADS, "prefix");
        const uint4* h4 = reinterpret_cast<const uint4*>(ghist) + threadIdx.x * 4u;
        uint64_t sum = 0, tot;
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) { const uint4 x = h4[i]; sum += (uint64_t)x.x + x.y + x.z + x.w; }
        const uint64_t n_zero = st->n_zero;
        base_of[threadIdx.x] = n_zero + block_excl_scan_u64<SEL_THREADS>(sum, S.smem, &tot);
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
                S.win[threadIdx.x] = W;
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
                uint32_t first = SEL_KEY_FINE + ((bin - SEL_BIN_FINE) << SEL_FINE_SHIFT), width = 32u + SEL_FINE_SHIFT;
                if (!sel_bin_is_fine(bin)) { first = sel_bin_first_key(bin); width = sel_bin_width(bin); }
                W.c_lo = (uint64_t)first << 32;
                W.width = width;
                W.r = r - below;
                W.less = below;
                W.cnt = cnt;
                S.win[threadIdx.x] = W;
            }
        }
    } else {
        // one wavefront per rank: the bin of its leader's histogram that holds its pair
        __syncthreads();
        const uint32_t nb = 1u << bits, per = nb / 64u;       // 4 .. 64 bins per lane
        for (uint32_t q = wid; q < k; q += SEL_THREADS / 64u) {
            const SelWindow& was = st->win[stage - 1u][q];
            if (was.mode != SEL_SPLIT) continue;
            SelWindow& W = S.win[q];
            const uint32_t leader = was.leader, width = was.width;
            const uint64_t r = was.r;
            const uint32_t key = st->key_lo[stage - 1u][leader];
            if (was.stage != 0u && width > 32u && key == st->key_hi[stage - 1u][leader]) {
                // all its weights are equal: on with the index
                if (lane == 0) {
                    W.c_lo = (uint64_t)key << 32;
                    W.r = r;
                    W.less = W.key_less = was.less;
                    W.cnt = W.key_eq = was.cnt;
                    W.width = 32u;
                    W.mode = SEL_SPLIT;
                }
                continue;
            }
            const uint32_t* hist = ghist + (size_t)(stage - 1u) * SEL_BINS + leader * nb;
            uint64_t sum = 0;
#pragma unroll 4
            for (uint32_t i = 0; i < per; i += 2u) {
                const uint2 c = *reinterpret_cast<const uint2*>(hist + lane * per + i);
                sum += (uint64_t)c.x + c.y;
            }
            unsigned long long incl = sum;
            for (uint32_t d = 1; d < 64; d <<= 1) {
                const unsigned long long y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            const uint64_t at = __ballot(incl - sum < r && r <= incl);
            if (at == 0ull) continue;
            // that lane's bins, one to a lane
            const uint32_t owner = (uint32_t)__ffsll((unsigned long long)at) - 1u;
            const uint64_t below = __shfl((unsigned long long)(incl - sum), (int)owner, 64);
            const uint32_t c = lane < per ? hist[owner * per + lane] : 0u;
            incl = c;
            for (uint32_t d = 1; d < 64; d <<= 1) {
                const unsigned long long y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            const uint64_t base = below + incl - c;
            if (base < r && r <= base + c) {
                const uint32_t shift = sel_shift(width, bits, g_bits);
                W.c_lo = was.c_lo + ((uint64_t)(owner * per + lane) << shift);
                W.r = r - base;
                W.less = was.less + base;
                W.cnt = c;
                W.width = shift;
                W.key_less = shift == 32u ? W.less : was.key_less;
                W.key_eq = shift == 32u ? c : was.key_eq;
                W.mode = SEL_SPLIT;
            }
        }
    }
    // no window in a top bin yet
    static_assert(SEL_BINS == 16u * SEL_THREADS, "one 16-byte piece of the map per thread");
    reinterpret_cast<uint4*>(S.map)[threadIdx.x] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (threadIdx.x == 0) S.map[SEL_BINS] = (uint8_t)NONE8;
    __syncthreads();
    // the windows in order: the ranks are sorted, so equal windows are neighbours (the first rank
    // leads) and those in one top bin follow each other
    if (wid == 0) {
        const SelWindow W = S.win[lane];
        const bool live = W.mode == SEL_SPLIT;
        const uint64_t prev_lo = __shfl_up((unsigned long long)W.c_lo, 1, 64);
        const uint32_t prev_live = __shfl_up(live ? 1u : 0u, 1, 64), prev_w = __shfl_up(W.width, 1, 64);
        const bool opens = live && !(lane > 0u && prev_live && prev_lo == W.c_lo && prev_w == W.width);
        const unsigned long long open_mask = __ballot(opens);
        const unsigned long long upto = open_mask & (~0ull >> (63u - lane));
        const uint32_t leader = upto ? 63u - (uint32_t)__clzll(upto) : lane;
        const uint32_t key = (uint32_t)(W.c_lo >> 32), fine = sel_fine_bin(key);
        uint32_t top = SEL_BIN_FINE + fine;
        if (live && fine >= SEL_FINE_BINS) top = top_bin(key);
        const unsigned long long before = open_mask & ((1ull << lane) - 1ull);
        const uint32_t prev_top = __shfl(top, before ? 63 - __clzll((long long)before) : 0, 64);
        const bool first = opens && !(before && prev_top == top);
        const unsigned long long first_mask = __ballot(first);
        const unsigned long long behind = lane == 63u ? 0ull : first_mask & (~0ull << (lane + 1u));
        const unsigned long long here = behind ? (1ull << (__ffsll(behind) - 1)) - 1ull : ~0ull;   // lanes before the next top bin
        const uint32_t in_top = (uint32_t)__popcll(open_mask & here & (~0ull << lane));
        if (live) {
            const uint32_t mode = W.cnt <= (stage < stages ? min(list_cap, SEL_LIST_GOOD) : list_cap) ? SEL_LISTED : SEL_SPLIT;
            S.win[lane].leader = leader;
            S.win[lane].mode = mode;
            // more weights than any spread-out distribution has in a bin (normal ones 0.76 % in a wide one), or one key
            const bool ties = W.width <= 32u || W.cnt > (n_weights >> 7);
            S.win[lane].stage = ties ? stage : 0u;
            if (ties) S.ties = 1;
            if (key != 0u && fine >= SEL_FINE_BINS) S.wide = 1;
            if (opens) {
                const uint32_t at = (uint32_t)__popcll(before);
                S.lo[at] = W.c_lo;
                S.about[at] = W.width | (sel_shift(W.width, bits, g_bits) << 6) | (mode == SEL_SPLIT ? SEL_ABOUT_SPLIT : 0u) |
                              (ties ? SEL_ABOUT_TIES : 0u) | (W.cnt > (n_weights >> 4) ? SEL_ABOUT_RUNS : 0u) |
                              (lane << 16) | (in_top << 24);
                if (first) S.map[top] = (uint8_t)at;
            }
            if (mode == SEL_SPLIT) S.left = 1;
        }
    }
    __syncthreads();
    if (publish) {
        if (threadIdx.x < k) {
            const SelWindow W = S.win[threadIdx.x];
            sel_put<DEV>(&st->win[stage][threadIdx.x], W);
            if (W.mode == SEL_LISTED) sel_put<DEV>(&st->fin[threadIdx.x], W);
        }
        if (threadIdx.x == 0) sel_put<DEV>(&st->done[stage], S.left ? 0u : 1u);
    }
    if (S.left) {                                 // the same in every thread
        for (uint32_t i = threadIdx.x; i < (k << bits); i += SEL_THREADS) S.hist[i] = 0;
        __syncthreads();
    }
}

// The reads of the arena go up and down in turn: what the last-level cache still holds of one larger than itself is the end that was
// read last.  One count of 100 M weights 176 us a call all the same way, 159 so; ten 265 and 245.
__device__ __forceinline__ constexpr bool sel_down(uint32_t stage) { return (stage & 1u) != 0u; }

// The weights of a part into the stage's histograms and lists.
template <bool DEV>
struct SelCollect {
    const SelJob& J;
    SelShared& S;
    RunCount run;
    KeyRange keys;
    __device__ __forceinline__ SelCollect(const SelJob& job, SelShared& shared) : J(job), S(shared) {}
    __device__ __forceinline__ void part(const SelArena& arena, uint32_t part, uint32_t parts, bool down) {
        if (__builtin_expect(uniform_u32(S.wide) != 0u, 0)) part_of<true>(arena, part, parts, down); else part_of<false>(arena, part, parts, down);
    }
    template <bool WIDE>
    __device__ __forceinline__ void part_of(const SelArena& arena, uint32_t part, uint32_t parts, bool down);
    __device__ __forceinline__ void leave(uint32_t stage);
};
// Most times all windows, but for zeros', lie in fine bins: the keys of others read the place behind those, where no window is
// then.  WIDE: some window lies in another bin.
template <bool DEV>
template <bool WIDE>
__device__ __forceinline__ void SelCollect<DEV>::part_of(const SelArena& arena, uint32_t part, uint32_t parts, bool down) {
    SelWalk walk(arena);
    SelState* const st = J.st;
    uint2* const lists = J.lists;
    const uint32_t lane = threadIdx.x & 63u, bits = sel_bits(J.k), list_cap = J.list_cap;
    // where the map is looked up
    auto place = [](uint32_t key) {
        if (!WIDE) return SEL_BIN_FINE + (key ? min(sel_fine_bin(key), SEL_FINE_BINS) : SEL_BINS - SEL_BIN_FINE);
        uint32_t bin = sel_top_bin(key);
        asm("" : "+v"(bin));                             // for zeros too, without a branch
        return key ? bin : SEL_BINS;
    };
    auto one = [&](uint32_t wbits, uint32_t g) {
        const uint32_t key = wbits & 0x7fffffffu;
        uint32_t i = S.map[place(key)];
        if (i == NONE8) return;
        const uint64_t comp = ((uint64_t)key << 32) | g;
        uint32_t about = S.about[i];
        if (about >= 2u << 24) {                    // several windows in this top bin: the last that begins by here
            for (uint32_t n = about >> 24; n > 1u;) {
                const uint32_t half = n >> 1;
                if (S.lo[i + half] <= comp) { i += half; n -= half; } else { n = half; }
            }
            about = S.about[i];
        }
        const uint64_t d = comp - S.lo[i];
        if ((d >> (about & 63u)) != 0) return;
        const uint32_t s = (about >> 16) & 0xffu;
        if (about & SEL_ABOUT_SPLIT) {
            const uint32_t entry = (s << bits) + (uint32_t)(d >> ((about >> 6) & 63u));
            if (about & SEL_ABOUT_RUNS) run.add(S.hist, entry, 1u); else atomicAdd(&S.hist[entry], 1u);
            if (about & SEL_ABOUT_TIES) keys.add(S.key_lo, S.key_hi, s, key);
            return;
        }
        // one reservation for the lanes that list a pair now, if they are many
        uint32_t pos = 0;
        const uint64_t all = __ballot(true);
        if (__popcll(all) > 16) {
            const uint32_t before = (uint32_t)__popcll(all & ((1ull << lane) - 1ull));
            if (before == 0) pos = atomicAdd(&S.n, (uint32_t)__popcll(all));
            pos = __shfl(pos, (int)__ffsll((unsigned long long)all) - 1, 64) + before;
        } else {
            pos = atomicAdd(&S.n, 1u);
        }
        if (pos < SEL_STAGE_CAP) {
            S.pair[pos] = make_uint2(wbits, g);
            S.of[pos] = (uint8_t)s;
            return;
        }
        if (about & SEL_ABOUT_TIES) keys.add(S.key_lo, S.key_hi, s, key);
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
        if (at < list_cap) sel_put<DEV>(&lists[(size_t)s * list_cap + at], make_uint2(wbits, g));
    };
    walk.run(part, parts, down, [&] {
        const uint4 (&v)[SEL_QUADS] = walk.v;
        // first which of the sixteen are met by a window, without a branch, then those one by one: few are,
        // and the long body stands here once (in line sixteen times: 20 ranks of 14.7 M weights 34 us, 24 so; 30
        // levels a sigma, one rank of 100 M 134 and 92; all 100 M equal 170 and 265)
        uint32_t met = 0;
#pragma unroll
        for (uint32_t u = 0; u < 4u; ++u) {
            const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) met |= (S.map[place(x[q] & 0x7fffffffu)] != NONE8 ? 1u : 0u) << (4u * u + q);
        }
        if (walk.n != TILE) met &= walk.there();
        while (met) {
            const uint32_t j = (uint32_t)__builtin_ctz(met);
            met &= met - 1u;
            one(walk.bits(j), walk.index(j));
        }
    });
}

// What the block has gathered goes to memory.
template <bool DEV>
__device__ __forceinline__ void SelCollect<DEV>::leave(uint32_t stage) {
    SelState* const st = J.st;
    uint2* const lists = J.lists;
    const uint32_t k = J.k, bits = sel_bits(J.k), list_cap = J.list_cap;
    run.flush(S.hist);
    keys.flush(S.key_lo, S.key_hi);
    __syncthreads();
    constexpr uint32_t PER = SEL_STAGE_CAP / SEL_THREADS;
    const uint32_t n = min(S.n, SEL_STAGE_CAP);
    if (S.ties) {
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u) {
            const uint32_t i = u * SEL_THREADS + threadIdx.x;
            if (i < n) {
                const uint32_t key = S.pair[i].x & 0x7fffffffu, s = S.of[i];
                if (key < S.key_lo[s]) atomicMin(&S.key_lo[s], key);
                if (key > S.key_hi[s]) atomicMax(&S.key_hi[s], key);
            }
        }
        __syncthreads();
        if (threadIdx.x < k && S.key_lo[threadIdx.x] <= S.key_hi[threadIdx.x]) {
            atomicMin(&st->key_lo[stage][threadIdx.x], S.key_lo[threadIdx.x]);
            atomicMax(&st->key_hi[stage][threadIdx.x], S.key_hi[threadIdx.x]);
        }
    }
    if (S.left) {
        uint32_t* out = J.ghist + (size_t)stage * SEL_BINS;
        for (uint32_t i = threadIdx.x; i < (k << bits); i += SEL_THREADS) {
            const uint32_t c = S.hist[i];
            if (c) atomicAdd(&out[i], c);
        }
    }
    // the collected pairs: count per list, one reservation each, then the writes
    if (n == 0) return;
    uint32_t pos[PER];
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
        const uint32_t i = u * SEL_THREADS + threadIdx.x;
        pos[u] = i < n ? atomicAdd(&S.cnt[S.of[i]], 1u) : 0u;
    }
    __syncthreads();
    if (threadIdx.x < k && S.cnt[threadIdx.x]) S.base[threadIdx.x] = atomicAdd(&st->list_cnt[threadIdx.x], S.cnt[threadIdx.x]);
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
        const uint32_t i = u * SEL_THREADS + threadIdx.x;
        if (i < n) {
            const uint32_t s = S.of[i], at = S.base[s] + pos[u];
            if (at < list_cap) sel_put<DEV>(&lists[(size_t)s * list_cap + at], S.pair[i]);
        }
    }
}

// The record of rank q, by one block, from its list.
__device__ __forceinline__ void sel_record(const SelJob& J, uint32_t q, RankShared<SEL_THREADS>& sh,
                                           shifter_threshold* __restrict__ thr, shifter_threshold* host_rec, uint32_t* host_nan) {
    const SelState* const st = J.st;
    const uint32_t list_cap = J.list_cap;
    shifter_threshold out = sel_no_record(st->p[q]);
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
            if (width == 32u) width = J.g_bits;
            // the window's pairs are all in the list: the r-th of them is the pair
            if (rank_in_list<SEL_THREADS, SEL_DEPTH>(J.lists + (size_t)W.leader * list_cap, min((uint32_t)W.cnt, list_cap),
                                                          c_lo, width, W.r, !one_key, sh)) {
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
        // inside the caller's records also where an overlapping call has left another permutation
        const uint32_t to = min(st->perm[q], J.k - 1u);
        thr[to] = out;
        if (host_rec) host_rec[to] = out;
        if (host_nan && q == 0) *host_nan = st->nan_seen;
    }
}

// The first stage, or the second in a launch of its own (see launch_select_tables).
template <uint32_t STAGE>
__global__ __launch_bounds__(SEL_THREADS) void sel_stage_kernel(const SelArena arena, const SelJob J) {
    __shared__ SelShared S;
    if (STAGE > 1u && J.st->done[STAGE - 1u]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) J.st->done[STAGE] = 1;
        return;
    }
    sel_windows<STAGE == 1u, false>(J, S, STAGE, blockIdx.x == 0);
    SelCollect<false> collect(J, S);
    collect.part(arena, blockIdx.x, gridDim.x, sel_down(STAGE));
    collect.leave(STAGE);
}

// The ranking of the lists, a block each, where there is one stage, which certainly lists every rank.
__global__ __launch_bounds__(SEL_THREADS) void sel_final_kernel(const SelJob J, shifter_threshold* __restrict__ thr,
                                                                shifter_threshold* host_rec, uint32_t* host_nan) {
    __shared__ RankShared<SEL_THREADS> sh;
    sel_record(J, blockIdx.x, sh, thr, host_rec, host_nan);
}

// The ranking of the lists, a block each.  Where the stages before have not listed every rank (many weights in one bin, equal
// ones mostly), the further stages come first, in the same launch: with a launch for each, the four that found nothing left
// took 4 us each of a call that has no ties (ten counts of 14.7 M weights, flat run, 64 us with them, 56 without).  There
// the parts of a stage are handed out by a ticket, and a block that finds none left waits until all that were taken have
// arrived.  Every wait of calls in order ends, however many of the blocks run at a time: a part is only ever held by a
// block that runs, and that leaves what it has gathered before it waits for its stage; what it may hold then is a part of
// the next stage, for which nobody waits before this one is over.  Two flat runs at once, which share their words and
// may clear each other's, could wait for ever: a wait is given up after J.polls looks.  The block then leaves without another
// word, the part or rank that it may hold is nobody's, and who waits for it gives up too: records not written stay
// those that remove nothing, which the first launch wrote.
__global__ __launch_bounds__(SEL_THREADS) void sel_rest_kernel(const SelArena arena, const SelJob J, uint32_t before, uint32_t parts,
                                                               shifter_threshold* __restrict__ thr, shifter_threshold* host_rec,
                                                               uint32_t* host_nan) {
    __shared__ SelShared S;
    __shared__ RankShared<SEL_THREADS> sh;
    __shared__ uint32_t s_take, s_over;
    SelState* const st = J.st;
    if (st->done[before]) {
        if (blockIdx.x < J.k) sel_record(J, blockIdx.x, sh, thr, host_rec, host_nan);
        return;
    }
    // a ticket is drawn while the block still works on what it has, and looked at by all when it is wanted
    uint32_t drawn = 0;
    auto draw = [&](uint32_t* ticket) {
        if (threadIdx.x == 0) drawn = atomicAdd(ticket, 1u);
    };
    auto taken = [&]() {
        __syncthreads();
        if (threadIdx.x == 0) s_take = drawn;
        __syncthreads();
        return uniform_u32(s_take);
    };
    draw(&st->ticket[before + 1u]);
    for (uint32_t stage = before + 1u;; ++stage) {
        uint32_t part = taken(), mine = 0;
        if (part < parts) {
            sel_windows<false, true>(J, S, stage, part == 0);
            SelCollect<true> collect(J, S);
            for (; part < parts; part = taken(), ++mine) {
                draw(&st->ticket[stage]);
                collect.part(arena, part, parts, sel_down(stage));
            }
            collect.leave(stage);
            wait_memory();
            __syncthreads();
            // the last to arrive says so on several lines: polls at the counter's own would hold up its additions
            if (threadIdx.x == 0) s_take = atomicAdd(&st->arrived[stage], mine) + mine;
            __syncthreads();
            if (s_take >= parts && threadIdx.x < SEL_GO) sel_put<true>(&st->go[stage][threadIdx.x * SEL_GO_WORDS], 1u);
        }
        const bool last = stage == J.stages;
        draw(&st->ticket[last ? 0u : stage + 1u]);
        if (threadIdx.x == 0) {
            uint32_t over = 0;
            for (uint32_t look = 0; look < J.polls && !over; ++look) {
                if (look) __builtin_amdgcn_s_sleep(8);
                over = __hip_atomic_load(&st->go[stage][blockIdx.x % SEL_GO * SEL_GO_WORDS], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            s_over = over;
        }
        __syncthreads();
        if (!uniform_u32(s_over)) return;
        if (last) break;
        if (st->done[stage]) {               // the same in every thread
            draw(&st->ticket[0]);
            break;
        }
    }
    for (uint32_t q = taken(); q < J.k; q = taken()) {
        sel_record(J, q, sh, thr, host_rec, host_nan);
        draw(&st->ticket[0]);
    }
}

void launch_select(shifter_ctx* ctx, const shifter_model* m, const float* d_w,
                   const PruneCounts& pc, uint32_t k, shifter_threshold* d_thr, bool mirror, uint32_t* zero_ptr,
                   uint32_t zero_n) {
    const auto& b = m->b;
    // the candidate buffer of the single-pass selections is idle here: it holds the lists
    if (mirror) {
        // no call is under way that writes them: what the kernels leave out stays that way
        shifter_threshold* rec = reinterpret_cast<shifter_threshold*>(b.host_multi + MULTI_MIRROR_REC_OFF);
        for (uint32_t i = 0; i < k; ++i) rec[i] = sel_no_record(pc.p[i]);
        *reinterpret_cast<uint32_t*>(b.host_multi) = 0;
    }
    const SelectTables tb{b.tens, b.tile_prefix, b.tile_tensor, m->n_tiles, m->info.n_prunable, b.sel, b.ghist,
                          b.cand, (uint64_t)b.cand_cap_sb * SPEC_SUB, nullptr, nullptr, zero_ptr, zero_n,
                          mirror ? b.dev_multi_rec : nullptr, mirror ? b.dev_multi_status : nullptr};
    launch_select_tables(ctx, tb, d_w, pc, k, d_thr);
}

void launch_select_tables(shifter_ctx* ctx, const SelectTables& tb, const float* d_w,
                          const PruneCounts& pc, uint32_t k, shifter_threshold* d_thr) {
    const uint32_t n_tiles = tb.n_tiles;
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
    const SelArena arena{tb.tens, tb.tile_prefix, tb.tile_tensor, n_tiles, d_w};
    const SelJob job{tb.sel, tb.ghist, tb.lists, list_cap, k, (uint32_t)tb.n_weights, g_bits, stages, ctx->select_polls};
    // Where a bin of spread-out weights is likely to outgrow a good list, the first stage will hardly list them all, and a launch
    // costs the second one less than the tickets do (ten of 100 M weights 252 us, 268 with them, all reads in one direction).
    // 1/1536 of the weights is a measured line, not a bound (a bin holds up to 1/1024): with 1/1024 one count of 70 to 90 M normal
    // weights 2 us more, of 56 to 90 M uniform ones 6 us less.
    const uint32_t before = stages > 1u && tb.n_weights / 1536u > std::min(list_cap, SEL_LIST_GOOD) ? 2u : 1u;
    {
        ProfileScope p(ctx, K_SEL_INIT);
        sel_clear_kernel<<<64, BLOCK, 0, s>>>(tb.sel, tb.ghist, stages, sorted, perm, k, d_thr, tb.flat_tens, tb.flat_prefix,
                                              tb.n_weights, tb.zero_ptr, tb.zero_n);
    }
    {
        ProfileScope p(ctx, K_HIST0);
        sel_top_kernel<<<grid, SEL_THREADS, 0, s>>>(arena, tb.sel, tb.ghist);
    }
    {
        ProfileScope p(ctx, K_SEL_STAGE);
        sel_stage_kernel<1><<<grid, SEL_THREADS, 0, s>>>(arena, job);
        if (before == 2u) sel_stage_kernel<2><<<grid, SEL_THREADS, 0, s>>>(arena, job);
    }
    {
        ProfileScope p(ctx, K_SEL_FINAL);
        if (stages == 1u) sel_final_kernel<<<k, SEL_THREADS, 0, s>>>(job, d_thr, tb.host_rec, tb.host_nan);
        else sel_rest_kernel<<<std::max(grid, k), SEL_THREADS, 0, s>>>(arena, job, before, grid, d_thr, tb.host_rec, tb.host_nan);
    }
}

}  // namespace shifter
