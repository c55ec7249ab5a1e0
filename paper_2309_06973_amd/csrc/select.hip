// Exact multi-rank selection of the P-th smallest (|w|, g) pair: the unstructured
// magnitude ranking of Sec. II-A / Sec. III-C of the paper in the form that needs no decision
// on the host, for any number of prune counts, any distribution and any number of ties.
//
//   top     one read of the arena: a histogram of all keys on the 16384 bins of sample_bin
//           (1/256 of a binade where the weights of networks live);
//   stage   every rank has a window of composites (key << 32 | g) that holds its pair and the
//           number of weights in it.  A stage reads the arena once: windows of no more pairs
//           than their list holds are written out as lists, the others are split by a further
//           histogram, first by key down to a single key, then by index.  On weights without
//           mass ties the first stage lists every rank and the stages behind it return at once;
//   final   one block per rank ranks its list and writes the record.
//
// The launches are the same for every input (their number follows from N and K alone), so the
// calls can be recorded into a graph.  What bounds it: two reads of the arena, and one launch
// after the other around them (about 5 us each, 3 for a stage with nothing to do).  The form it replaces - a
// radix select of 11 + 10 + 10 bits with eight prefixes per read and one read per distinct
// key for the ties - read the arena seven times for ten counts and walked the ranks one by one
// on one block between the reads: 394 us a call against 61 for ten counts of 14.7 M weights.
#include <algorithm>

#include "dev_common.h"

namespace shifter {

constexpr uint32_t SEL_THREADS = 1024;
constexpr uint32_t SEL_GROUPS = SEL_THREADS / BLOCK;   // tiles a block walks side by side
constexpr uint32_t SEL_STAGE_CAP = 4096;               // listed pairs a block collects in LDS
constexpr uint32_t NONE8 = 0xffu;

// log2 of the bins of one window's histogram: what K of them may share SEL_BINS counters.
__host__ __device__ __forceinline__ uint32_t sel_bits(uint32_t k) {
    uint32_t b = 12;
    while (b > 8 && (k << b) > SEL_BINS) --b;
    return b;
}

// A window of 2^width composites is split into bins of 2^shift: by key until it holds a single
// one (width 32), then by index, of which the lowest g_bits can be set.
__host__ __device__ __forceinline__ uint32_t sel_shift(uint32_t width, uint32_t bits, uint32_t g_bits) {
    if (width > 32u) return width - 32u > bits ? width - bits : 32u;
    const uint32_t w = width == 32u ? g_bits : width;
    return w > bits ? w - bits : 0u;
}

__global__ __launch_bounds__(BLOCK) void sel_clear_kernel(SelState* st, uint32_t* ghist, uint32_t hists,
                                                          PruneCounts pc, MultiPerm perm, uint32_t k,
                                                          DevTensor* flat_tens, uint32_t* flat_prefix, uint64_t flat_n) {
    const uint32_t tid = blockIdx.x * BLOCK + threadIdx.x;
    uint4* g4 = reinterpret_cast<uint4*>(ghist);
    for (uint32_t i = tid; i < hists * (SEL_BINS / 4); i += gridDim.x * BLOCK) g4[i] = make_uint4(0, 0, 0, 0);
    if (tid < MAXK) {
        st->p[tid] = tid < k ? pc.p[tid] : 0;
        st->perm[tid] = tid < k ? perm.v[tid] : 0;
        st->list_cnt[tid] = 0;
        st->fin[tid].mode = SEL_IDLE;
        if (tid <= SEL_STAGES) st->done[tid] = 0;
    }
    if (tid == 0) {
        st->nan_seen = 0;
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

// f(bits, g) for every prunable weight.  Four tiles at a time per block, one per 256 threads,
// a thread's 64 bytes in flight together; no barriers, so the wavefronts drift apart and one's
// loads overlap with another's work.
template <typename F>
__device__ __forceinline__ void sel_walk(const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix,
                                         uint32_t n_t, uint32_t n_tiles, const float* __restrict__ w, F&& f) {
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
            constexpr uint32_t U = TILE / BLOCK / 4;
            uint4 v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = load_u4<false>(src + 4u * tid + 4u * BLOCK * u);
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t g = g0 + 4u * tid + 4u * BLOCK * u;
                f(v[u].x, g); f(v[u].y, g + 1u); f(v[u].z, g + 2u); f(v[u].w, g + 3u);
            }
        } else {
            for (uint32_t j = tid; j < n; j += BLOCK) f(__float_as_uint(src[j]), g0 + j);
        }
    }
}

__global__ __launch_bounds__(SEL_THREADS) void sel_top_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix, uint32_t n_t, uint32_t n_tiles,
    const float* __restrict__ w, SelState* st, uint32_t* ghist) {
    __shared__ uint32_t h[SEL_BINS];
    for (uint32_t i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) h[i] = 0;
    __syncthreads();
    uint32_t key_max = 0;
    sel_walk(tens, tile_prefix, n_t, n_tiles, w, [&](uint32_t bits, uint32_t) {
        const uint32_t key = bits & 0x7fffffffu;
        key_max = max(key_max, key);
        atomicAdd(&h[sample_bin(key)], 1u);
    });
    if (key_max > 0x7f800000u) st->nan_seen = 1;
    __syncthreads();
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
    uint32_t k, uint32_t g_bits, uint32_t stage) {
    // bytes of the map: first leader whose window lies in that top bin
    __shared__ __align__(16) uint8_t s_map[SEL_BINS];
    __shared__ uint32_t s_hist[SEL_BINS];
    __shared__ __align__(16) uint2 s_pair[SEL_STAGE_CAP];
    __shared__ uint8_t s_of[SEL_STAGE_CAP];
    __shared__ SelWindow s_win[MAXK];
    __shared__ uint64_t smem[SEL_THREADS / 64 + 1];
    __shared__ uint32_t s_next[MAXK], s_cnt[MAXK], s_base[MAXK], s_n, s_left;
    if (stage > 1u && st->done[stage - 1u]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->done[stage] = 1;
        return;
    }
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t bits = sel_bits(k);
    if (threadIdx.x < MAXK) {
        SelWindow W;
        W.c_lo = W.r = W.less = W.key_less = W.key_eq = W.cnt = 0;
        W.width = 0; W.leader = threadIdx.x; W.mode = SEL_IDLE; W.pad = 0;
        s_win[threadIdx.x] = W;
        s_cnt[threadIdx.x] = 0;
        s_next[threadIdx.x] = NONE8;
    }
    if (threadIdx.x == 0) { s_n = 0; s_left = 0; }
    if (stage == 1u) {
        // sixteen bins per thread, their exclusive prefix over the block (in the room of the
        // pairs), then a search per rank
        uint64_t* base_of = reinterpret_cast<uint64_t*>(s_pair);
        static_assert(sizeof(s_pair) >= sizeof(uint64_t) * SEL_THREADS && SEL_BINS == 16u * SEL_THREADS, "prefix");
        const uint4* h4 = reinterpret_cast<const uint4*>(ghist) + threadIdx.x * 4u;
        uint64_t sum = 0, tot;
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) { const uint4 x = h4[i]; sum += (uint64_t)x.x + x.y + x.z + x.w; }
        base_of[threadIdx.x] = block_excl_scan_u64<SEL_THREADS>(sum, smem, &tot);
        __syncthreads();
        if (threadIdx.x < k) {
            const uint64_t r = st->p[threadIdx.x];
            if (r != 0 && r <= tot) {
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
                SelWindow W;
                W.c_lo = (uint64_t)sample_bin_first_key(bin) << 32;
                // the bins at both ends of the binning span up to 2^30 keys
                W.width = 32u + ((bin == 0u || bin == SAMPLE_BINS - 1u) ? 30u : SAMPLE_BIN_SHIFT);
                W.r = r - below;
                W.less = below;
                W.key_less = W.key_eq = 0;
                W.cnt = cnt;
                W.leader = threadIdx.x;
                W.mode = SEL_SPLIT;
                W.pad = 0;
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
    for (uint32_t i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) s_hist[i] = 0;
    __syncthreads();
    // leaders: the ranks are sorted, so equal windows are neighbours; windows that share a top
    // bin are chained
    if (wid == 0) {
        const SelWindow W = s_win[lane];
        const bool live = W.mode == SEL_SPLIT;
        const uint64_t prev_lo = __shfl_up((unsigned long long)W.c_lo, 1, 64);
        const uint32_t prev_live = __shfl_up(live ? 1u : 0u, 1, 64), prev_w = __shfl_up(W.width, 1, 64);
        const bool opens = live && !(lane > 0u && prev_live && prev_lo == W.c_lo && prev_w == W.width);
        const unsigned long long open_mask = __ballot(opens);
        const unsigned long long upto = open_mask & (~0ull >> (63u - lane));
        const uint32_t leader = upto ? 63u - (uint32_t)__clzll(upto) : lane;
        const uint32_t top = sample_bin((uint32_t)(W.c_lo >> 32));
        const unsigned long long before = open_mask & ((1ull << lane) - 1ull);
        const uint32_t prev = before ? 63u - (uint32_t)__clzll(before) : 0u;
        const uint32_t prev_top = __shfl(top, prev, 64);
        if (live) {
            const uint32_t mode = W.cnt <= list_cap ? SEL_LISTED : SEL_SPLIT;
            s_win[lane].leader = leader;
            s_win[lane].mode = mode;
            if (opens) {
                if (before && prev_top == top) s_next[prev] = lane; else s_map[top] = (uint8_t)lane;
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
    sel_walk(tens, tile_prefix, n_t, n_tiles, w, [&](uint32_t wbits, uint32_t g) {
        const uint32_t key = wbits & 0x7fffffffu;
        uint32_t s = s_map[sample_bin(key)];
        if (s == NONE8) return;
        const uint64_t comp = ((uint64_t)key << 32) | g;
        uint64_t d = comp - s_win[s].c_lo;
        while ((d >> s_win[s].width) != 0) {
            s = s_next[s];
            if (s == NONE8) return;
            d = comp - s_win[s].c_lo;
        }
        if (s_win[s].mode == SEL_SPLIT) {
            atomicAdd(&s_hist[(s << bits) + (uint32_t)(d >> sel_shift(s_win[s].width, bits, g_bits))], 1u);
            return;
        }
        const uint32_t pos = atomicAdd(&s_n, 1u);
        if (pos < SEL_STAGE_CAP) {
            s_pair[pos] = make_uint2(wbits, g);
            s_of[pos] = (uint8_t)s;
            return;
        }
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
    });
    __syncthreads();
    if (s_left) {
        uint32_t* out = ghist + (size_t)stage * SEL_BINS;
        for (uint32_t i = threadIdx.x; i < (k << bits); i += SEL_THREADS) {
            const uint32_t c = s_hist[i];
            if (c) atomicAdd(&out[i], c);
        }
    }
    // the collected pairs: count per list, one reservation each, then the writes
    const uint32_t n = min(s_n, SEL_STAGE_CAP);
    if (n == 0) return;
    constexpr uint32_t PER = SEL_STAGE_CAP / SEL_THREADS;
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
    const SelState* __restrict__ st, const uint2* __restrict__ lists, uint32_t list_cap,
    shifter_threshold* __restrict__ thr) {
    __shared__ RankShared<SEL_THREADS> sh;
    const uint32_t q = blockIdx.x;
    shifter_threshold out;
    out.cut = 0; out.t_key = 0; out.reserved = 0; out.g_cut = ~0ull; out.n_less = 0; out.n_equal = 0;
    out.n_prune = st->p[q];
    if (out.n_prune != 0) {
        const SelWindow W = st->fin[q];
        // the window's pairs are all in the list: the r-th of them is the pair
        if (W.mode == SEL_LISTED &&
            rank_in_list<SEL_THREADS, 8>(lists + (size_t)W.leader * list_cap, min((uint32_t)W.cnt, list_cap), W.c_lo,
                                         W.width, W.r, sh)) {
            out.cut = sh.sel + 1;
            out.t_key = (uint32_t)(sh.sel >> 32);
            out.g_cut = sh.sel & 0xffffffffull;
            // a window inside one key: what shares that key was counted when it was split
            out.n_less = W.width < 32u ? W.key_less : W.less + sh.lt;
            out.n_equal = W.width < 32u ? W.key_eq : sh.eq;
        }
    }
    if (threadIdx.x == 0) thr[st->perm[q]] = out;
}

// Stages that certainly suffice: a window of the widest kind is split until no more weights
// than a list holds can lie in it, and listed.
static uint32_t sel_stages(uint64_t n, uint32_t bits, uint32_t g_bits, uint32_t list_cap) {
    uint32_t width = 62, stages = 1;
    while (std::min<uint64_t>(n, 1ull << width) > list_cap) {
        width = sel_shift(width, bits, g_bits);
        ++stages;
    }
    return stages;
}

void launch_select(shifter_ctx* ctx, const shifter_model* m, const float* d_w,
                   const PruneCounts& pc, uint32_t k, shifter_threshold* d_thr) {
    const auto& b = m->b;
    // the candidate buffer of the single-pass selections is idle here: it holds the lists
    const SelectTables tb{b.tens, b.tile_prefix, (uint32_t)m->t.size(), m->n_tiles, m->info.n_prunable, b.sel, b.ghist,
                          b.cand, (uint64_t)b.cand_cap_sb * SPEC_SUB, nullptr, nullptr};
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
    const uint32_t bits = sel_bits(k);
    uint32_t g_bits = 0;
    while (g_bits < 32u && (tb.n_weights >> g_bits) != 0) ++g_bits;
    const uint32_t list_cap = (uint32_t)std::min<uint64_t>(tb.list_pairs / k, 1u << 20);
    const uint32_t stages = sel_stages(tb.n_weights, bits, g_bits, list_cap);
    const uint32_t grid = std::max(1u, std::min((n_tiles + SEL_GROUPS - 1) / SEL_GROUPS, ctx->hist_grid));
    {
        ProfileScope p(ctx, K_SEL_INIT);
        sel_clear_kernel<<<64, BLOCK, 0, s>>>(tb.sel, tb.ghist, stages, sorted, perm, k, tb.flat_tens, tb.flat_prefix,
                                              tb.n_weights);
    }
    {
        ProfileScope p(ctx, K_HIST0);
        sel_top_kernel<<<grid, SEL_THREADS, 0, s>>>(tb.tens, tb.tile_prefix, n_t, n_tiles, d_w, tb.sel, tb.ghist);
    }
    for (uint32_t stage = 1; stage <= stages; ++stage) {
        ProfileScope p(ctx, K_SEL_STAGE);
        sel_stage_kernel<<<grid, SEL_THREADS, 0, s>>>(tb.tens, tb.tile_prefix, n_t, n_tiles, d_w, tb.sel, tb.ghist,
                                                      tb.lists, list_cap, k, g_bits, stage);
    }
    {
        ProfileScope p(ctx, K_SEL_FINAL);
        sel_final_kernel<<<k, SEL_THREADS, 0, s>>>(tb.sel, tb.lists, list_cap, d_thr);
    }
}

}  // namespace shifter
