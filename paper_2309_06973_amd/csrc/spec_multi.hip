// Single-pass exact selection for ALL prune counts of a portfolio at once: the ranking of
// Sec. II-A / Sec. III-C of the paper for K sparsity levels in one read of the arena.
//
// Same scheme as the one-count selection (sample, predict, one pass, finish), with the
// prune counts sorted ascending so that the predicted key intervals [lo_k, hi_k] have
// non-decreasing ends.  Intervals that overlap are merged into one (a cluster of ranks
// sharing lo and hi), so two intervals are either the same or disjoint.  For a weight with
// key x let j = #{k : lo_k <= x}; then
//   x < lo_k  <=>  j <= k            (so below_k is a prefix sum of the counts per j)
//   x is a candidate  <=>  j >= 1 and x <= hi_{j-1}; it belongs to the cluster whose last
//                          rank is j - 1
// so one search per weight replaces K interval tests.  The pass appends a candidate to the
// region of its cluster (split CAND_SUB ways by block, one reservation per block and cluster).
#include "spec_sample.h"

namespace shifter {

// The counters all blocks add to are split CAND_SUB ways by block (one 128-byte line per
// part), and so is a cluster's candidate region: few enough parts that each averages over
// hundreds of tiles - filters differ in scale by orders of magnitude, so the candidates of
// one threshold crowd into few tiles - and enough that the additions of all blocks do not
// queue on one address.
constexpr uint32_t CAND_SUB = 32;
static_assert(CAND_SUB <= SPEC_SUB, "the counters use the first CAND_SUB lines of a row");
constexpr uint32_t FIN_THREADS = 1024;   // the last step of the finish: one block per rank
constexpr uint32_t FIN_BINS = 4096;      // bins of one refinement level there
constexpr uint32_t FIN_LIST = 1024;      // pairs the last bin may hold (too many equal keys beyond that)
constexpr uint32_t FIN_DIRECT = 96;      // pairs ranked by counting without refining further

// Split counters, one 128-byte line each: row j (0 <= j <= MAXK) counts the weights with
// exactly j lower ends at or below their key; row MAXK + 1 + r the candidates appended to
// the region of the cluster whose last rank is r.
__device__ __forceinline__ uint32_t* mcnt_below(uint32_t* cnt, uint32_t j, uint32_t sb) {
    return cnt + ((size_t)j * SPEC_SUB + sb) * 32u;
}
__device__ __forceinline__ uint32_t* mcnt_cand(uint32_t* cnt, uint32_t r, uint32_t sb) {
    return cnt + ((size_t)(MAXK + 1u + r) * SPEC_SUB + sb) * 32u;
}

// #{k : lo_k <= key} by a branch-free binary search; s_lo holds MAXK + 1 entries, padded
// with 0xffffffff.
__device__ __forceinline__ uint32_t count_lower_ends(const uint32_t* s_lo, uint32_t key) {
    uint32_t j = 0;
#pragma unroll
    for (uint32_t step = MAXK / 2; step >= 1; step >>= 1)
        if (s_lo[j + step - 1] <= key) j += step;
    return j + (s_lo[j] <= key ? 1u : 0u);
}

// Sample and prediction in one launch.  On the way the scratch of the kernels behind it is cleared: the
// split counters' rows in use, the clusters' histograms, the finish's per-rank words and one
// more array of the caller's.
// The block that ends last sets up the ranking (the state, the zero-count records) and works out,
// for every rank, the interval from the sample's order statistics at P/N -/+ margin, monotone
// ends, clusters, and each cluster's share of the candidate buffer.
// sorted_p / perm: the k prune counts > 0 in ascending order and their original positions;
// zero_mask: bit i set = original position i asked for P = 0 and gets its record here.
__global__ __launch_bounds__(SAMPLE_THREADS) void ms_front_kernel(
    SampleIn sample, MultiState* ms, uint32_t* __restrict__ cnt, uint32_t* __restrict__ ghist,
    uint32_t* __restrict__ rank_words, uint32_t* __restrict__ extra, uint32_t extra_n, PruneCounts sorted_p,
    MultiPerm perm, uint32_t k_var, uint32_t m, uint64_t zero_mask, shifter_threshold* thr,
    shifter_threshold* host_rec, uint64_t n_prunable, double margin_sigmas,
    uint8_t* __restrict__ tab, uint32_t cap_sb_total) {
    __shared__ __align__(16) uint32_t prefix[SAMPLE_BINS];          // 64 KB
    __shared__ uint32_t s_lo_bin[MAXK], s_hi_bin[MAXK], s_bins[3][64];
    {
        // rows 0 .. k and MAXK + 1 .. MAXK + k of the split counters (the first word of each
        // 128-byte line)
        const uint32_t tid = blockIdx.x * SAMPLE_THREADS + threadIdx.x, nthr = gridDim.x * SAMPLE_THREADS;
        for (uint32_t i = tid; i < (2u * k_var + 1u) * SPEC_SUB; i += nthr) {
            const uint32_t row = i / SPEC_SUB, sb = i % SPEC_SUB;
            const uint32_t r = row <= k_var ? row : MAXK + 1u + (row - (k_var + 1u));
            cnt[((size_t)r * SPEC_SUB + sb) * 32u] = 0;
        }
        for (uint32_t i = tid; i < k_var * 256u; i += nthr) ghist[i] = 0;
        for (uint32_t i = tid; i < extra_n; i += nthr) extra[i] = 0;
        if (tid < 3u * MAXK) rank_words[tid] = 0;
    }
    if (k_var != 0 && !sample_prefix(sample, prefix)) return;     // no rank: one block, no sample
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    if (threadIdx.x < MAXK) {
        const uint32_t t = threadIdx.x;
        ms->p[t] = t < k_var ? sorted_p.p[t] : 0;
        ms->perm[t] = t < k_var ? perm.v[t] : 0;
        if (t >= k_var) {                  // padding sorts last in the searches
            ms->lo[t] = 0xffffffffu;
            ms->hi[t] = 0xffffffffu;
            ms->mid[t] = 0xffffffffu;
            ms->clast[t] = t;
            ms->cand_off[t] = 0;
            ms->cand_cap[t] = 0;
        }
        if ((zero_mask >> t) & 1ull) {
            shifter_threshold out;
            out.cut = 0; out.t_key = 0; out.reserved = 0; out.g_cut = ~0ull; out.n_prune = 0;
            out.n_less = 0; out.n_equal = 0;
            thr[t] = out;
            host_rec[t] = out;
        }
    }
    if (threadIdx.x == 0) {
        ms->k = k_var;
        ms->m_valid = m;
        ms->status = 0;
    }
    if (k_var == 0) return;
    // rank k in lane k (k_var <= 64); the low end, the high end and the centre by a wavefront each
    const uint32_t total = prefix[SAMPLE_BINS - 1u];
    const uint64_t p = lane < k_var ? sorted_p.p[lane] : 0;
    const bool use = lane < k_var && p > 0 && m >= 256 && n_prunable > 0 && total == m;
    double r_lo = 0, r_hi = 0;
    if (wid < 3 && use) {
        const double frac = (double)p / (double)n_prunable;
        const double centre = frac * (double)m;
        const double delta = margin_sigmas * sqrt((double)m * frac * (1.0 - frac)) + 16.0;
        r_lo = centre - delta;
        r_hi = centre + delta;
        const double r = wid == 0 ? r_lo : wid == 1 ? r_hi : min(max(centre, 0.0), (double)(m - 1));
        s_bins[wid][lane] = sample_bin_of_rank(prefix, r > 0.0 ? (uint32_t)min(r, (double)(m - 1)) : 0u);
    }
    __syncthreads();
    if (wid == 0) {
        uint32_t lo = 0, hi = 0x7fffffffu, mid = 0;
        if (use) {
            if (r_lo > 0.0) lo = sample_bin_first_key(s_bins[0][lane]);
            if (r_hi < (double)(m - 1)) hi = sample_bin_last_key(s_bins[1][lane]);
            mid = sample_bin_first_key(s_bins[2][lane]);
        }
        // widen so that both ends are non-decreasing in k (ranks are sorted by P): a running
        // maximum of hi from the left, a running minimum of lo from the right; lanes past
        // the last rank hold the neutral values
        if (lane >= k_var) { lo = 0xffffffffu; hi = 0; }
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t yh = __shfl_up(hi, d, 64);
            const uint32_t yl = __shfl_down(lo, d, 64);
            if (lane >= d) hi = max(hi, yh);
            if (lane + d < 64) lo = min(lo, yl);
        }
        // clusters: rank k opens one unless its interval meets that of rank k - 1; every
        // rank of a cluster takes the first one's lo and the last one's hi
        const uint32_t hi_prev = __shfl_up(hi, 1, 64);
        const bool opens = lane < k_var && (lane == 0 || lo > hi_prev);
        const unsigned long long open_mask = __ballot(opens);
        const unsigned long long upto = open_mask & (~0ull >> (63u - lane));     // openers at or below this lane
        const uint32_t first = upto ? 63u - (uint32_t)__clzll(upto) : 0u;
        const unsigned long long after = lane < 63u ? open_mask >> (lane + 1u) : 0ull;   // openers above it
        uint32_t last = after ? lane + (uint32_t)__ffsll(after) - 1u : k_var - 1u;
        if (lane >= k_var) last = lane;
        lo = __shfl(lo, first, 64);
        hi = __shfl(hi, min(last, 63u), 64);
        // provisional threshold of the fused pass: inside the interval, non-decreasing (a
        // running maximum: it stays below hi because hi is non-decreasing)
        uint32_t pm = lane < k_var ? min(max(mid, lo), hi) : 0u;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(pm, d, 64);
            if (lane >= d) pm = max(pm, y);
        }
        // each cluster's share of the candidate buffer, in proportion to the samples inside
        // its interval (plus a little for the empty ones); the region belongs to the
        // cluster's last rank
        uint32_t wt = 0;
        if (lane < k_var && last == lane) {
            const uint32_t b_lo = sample_bin(lo), b_hi = sample_bin(hi);
            wt = prefix[b_hi] - (b_lo ? prefix[b_lo - 1u] : 0u) + 64u;
        }
        uint64_t wsum = wt;
        for (uint32_t d = 32; d > 0; d >>= 1) wsum += __shfl_down(wsum, d, 64);
        wsum = __shfl(wsum, 0, 64);
        // cap_sb_total pairs per 1/SPEC_SUB of the buffer; a part of a region is 1/CAND_SUB of it
        const uint32_t cap = wt ? (uint32_t)((uint64_t)cap_sb_total * (SPEC_SUB / CAND_SUB) * wt / wsum) : 0u;
        uint32_t cinc = cap;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(cinc, d, 64);
            if (lane >= d) cinc += y;
        }
        if (lane < k_var) {
            ms->lo[lane] = lo;
            ms->hi[lane] = hi;
            ms->mid[lane] = pm;
            ms->clast[lane] = last;
            ms->cand_cap[lane] = cap;
            ms->cand_off[lane] = (cinc - cap) * CAND_SUB;     // at most cap_sb_total * SPEC_SUB pairs
            s_lo_bin[lane] = sample_bin(lo);
            s_hi_bin[lane] = sample_bin(hi);
        }
        // the finish's view of a rank: its cluster's region and first histogram
        const uint32_t cap_cl = __shfl(cap, min(last, 63u), 64);
        const uint32_t off_cl = __shfl((cinc - cap) * CAND_SUB, min(last, 63u), 64);
        if (lane < k_var) {
            const uint32_t span = hi - lo;
            RankIn in;
            in.p = p;
            in.lo = lo;
            in.sh = span < 256u ? 0u : (32u - (uint32_t)__clz(span)) - 8u;
            in.clast = last;
            in.cand_off = off_cl;
            in.cand_cap = cap_cl;
            in.perm = perm.v[lane];
            ms->rin[lane] = in;
        }
    }
    // The pass's table: what it has to know of a weight follows from its bin of the sample histogram,
    // because all interval ends are edges of those bins.  Bits 0-5 = #{k : lo_k <= key}, bit 7: the
    // key lies in the interval of the last of those ranks.  Entry 0 is for the bins below the first
    // rank's lower end, entry i for the i-th bin from there on, the last entry for all above it too; where
    // the intervals span more bins than that, a table of all bins follows it and is used instead.  The last
    // bin has no upper edge: entries that lie behind it are of its class.
    __syncthreads();
    auto classes = [&](uint32_t bin0) {      // of four bins from bin0 on; -1 is bin 0, any behind the last is the last
        int32_t bin[4];
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) bin[i] = min(max((int32_t)(bin0 + i), 0), (int32_t)SAMPLE_BINS - 1);
        uint32_t j[4] = {0, 0, 0, 0}, four = 0;
        for (uint32_t k = 0; k < k_var; ++k) {
            const int32_t lo = (int32_t)s_lo_bin[k];
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) j[i] += lo <= bin[i] ? 1u : 0u;
        }
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i)
            four |= (j[i] | (j[i] != 0u && bin[i] <= (int32_t)s_hi_bin[j[i] - 1u] ? 0x80u : 0u)) << (8u * i);
        return four;
    };
    static_assert(PASS_TAB == 4u * SAMPLE_THREADS, "four entries a thread");
    const uint32_t first = s_lo_bin[0];
    uint32_t* tab4 = reinterpret_cast<uint32_t*>(tab);
    tab4[threadIdx.x] = classes(first - 1u + 4u * threadIdx.x);
    // the last bin whose class differs from the one below it
    const uint32_t change = max(s_lo_bin[k_var - 1u], min(s_hi_bin[k_var - 1u] + 1u, SAMPLE_BINS - 1u));
    const bool wide = change - first > PASS_TAB - 2u;
    if (wide)
        for (uint32_t i = threadIdx.x; i < SAMPLE_BINS / 4u; i += SAMPLE_THREADS) tab4[PASS_TAB / 4u + i] = classes(4u * i);
    if (threadIdx.x == 0) {
        ms->tab_first = (SAMPLE_KEY0 >> SAMPLE_BIN_SHIFT) + first - 1u;
        ms->tab_wide = wide ? 1u : 0u;
    }
}

// Appends the candidates a block found to the regions of their clusters: count per cluster
// in LDS, one global reservation per cluster the block met, then the writes.  `for_each`
// calls its argument once per candidate of the calling thread with (bits, global index,
// cluster = last rank whose lower end lies at or below the key).  All threads of the block
// call this; it contains barriers.
template <typename ForEach>
__device__ __forceinline__ void ms_append_candidates(
    bool have, const uint32_t* s_coff, const uint32_t* s_ccap, uint32_t* s_rc, uint32_t* s_rc2,
    uint32_t* s_rbase, uint32_t k_var, uint32_t* cnt, uint32_t csb, uint2* __restrict__ cand,
    ForEach&& for_each) {
    if (!__syncthreads_or(have ? 1 : 0)) return;      // uniform: no candidate in this block
    if (have) for_each([&](uint32_t, uint32_t, uint32_t cl) { atomicAdd(&s_rc[cl], 1u); });
    __syncthreads();
    if (threadIdx.x < k_var) {
        const uint32_t c = s_rc[threadIdx.x];
        if (c) s_rbase[threadIdx.x] = atomicAdd(mcnt_cand(cnt, threadIdx.x, csb), c);
    }
    __syncthreads();
    if (have)
        for_each([&](uint32_t bits, uint32_t g, uint32_t cl) {
            const uint32_t pos = s_rbase[cl] + atomicAdd(&s_rc2[cl], 1u);
            const uint32_t cap = s_ccap[cl];
            if (pos < cap) cand[(size_t)s_coff[cl] + (size_t)csb * cap + pos] = make_uint2(bits, g);
        });
}

// The one pass over the arena: counts per j and candidate pairs.
// What bounds it are a wavefront's vector instructions where many tiles wait (eight wavefronts a SIMD, a
// block's life 18 us with 1650 of them) and the latencies one behind the other where few do; the arena's
// bytes, which come from the cache, lie far behind.  So a weight's class is one look at a table on bins
// of the sample histogram, a cluster's candidates are counted by eight counters, and a
// tensor's last, ragged tile goes the same way as a full one, the weights it lacks counted in a row of their own.  Against
// a 4096-entry table of 1/16 binades with compares behind it, one counter a cluster and one global
// addition per candidate in the ragged tiles (kernel, us): fifteen ranks of 0.86 M weights, where
// over half are candidates, 19.2 -> 8.3; eight of 10 M 27.8 -> 16.0; ten of 14.7 M 39.4 -> 28.3; twenty of
// 25.5 M 67.4 -> 51.9.  A table of all 16384 bins in LDS (six blocks to a compute unit, not eight): 8.3, 20.3,
// 32.0, 55.4.  Tried and dropped: four tiles a block (19.3, 35.5, 60.4 beyond the first), blocks that fetch their next
// tile while they work on one (registers spill: twice the time).
constexpr uint32_t PASS_COPIES = 8;      // counters of a cluster's candidates: one for eight lanes
template <bool NT>
__global__ __launch_bounds__(BLOCK, 8) void ms_pass_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix, const uint16_t* __restrict__ tile_tensor,
    const float* __restrict__ w, MultiState* ms, uint32_t k_var, uint32_t* cnt, uint2* __restrict__ cand,
    const uint8_t* __restrict__ tab, uint32_t* zero_ptr, uint32_t zero_n) {
    // an array the step behind this pass wants cleared (or nullptr)
    for (uint32_t i = blockIdx.x * BLOCK + threadIdx.x; i < zero_n; i += gridDim.x * BLOCK) zero_ptr[i] = 0;
    // counts per j: one private byte column per thread (a thread sees 16 weights; no
    // conflicts, no atomics), summed at the end; rows 0 .. k_var of BLOCK bytes and one for the
    // weights that a ragged tile lacks (the launch sizes it)
    extern __shared__ __align__(16) uint32_t s_col[];
    __shared__ __align__(16) uint8_t s_tab[PASS_TAB];
    // candidates by cluster and eight lanes, then their places in the block's part of the cluster's region;
    // where that part starts and how many pairs it holds
    __shared__ uint32_t s_cnt[SPEC_MULTI_MAXK * PASS_COPIES];
    __shared__ uint2 s_part[SPEC_MULTI_MAXK];
    __shared__ uint32_t s_nan;
    constexpr uint32_t U = TILE / BLOCK / 4;
    const uint32_t tile = blockIdx.x, tid = threadIdx.x;
    const uint32_t sb = tile & (SPEC_SUB - 1), csb = tile & (CAND_SUB - 1);
    const uint32_t t = tile_tensor[tile];
    const uint4 piece = reinterpret_cast<const uint4*>(tab)[tid];
    static_assert(PASS_TAB == 16u * BLOCK, "one 16-byte piece of the table per thread");
    const uint32_t tab_first = ms->tab_first;
    const bool wide = ms->tab_wide != 0;
    uint32_t coff = 0, ccap = 0;
    if (tid < k_var) {
        coff = ms->cand_off[tid];
        ccap = ms->cand_cap[tid];
    }
    if (!tens[t].prunable) return;
    // the tile's loads: the set-up below runs while they are in flight
    const uint32_t e0 = (tile - tile_prefix[t]) * TILE;
    const uint32_t n = min(TILE, tens[t].numel - e0);
    const uint32_t g0 = (uint32_t)(tens[t].gbase + e0);
    const float* src = w + tens[t].offset + e0;
    uint4 v[U];
    uint32_t missing = 0;                   // bit 4 u + q: no such weight in a ragged tile
    if (n == TILE) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) v[u] = load_u4<NT>(src + 4u * tid + 4u * BLOCK * u);
    } else {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t j = (tid + BLOCK * u) * 4u;
            v[u] = make_uint4(0, 0, 0, 0);
            if (j + 3u < n) {
                v[u] = load_u4<NT>(src + j);
            } else {
                if (j < n) v[u].x = __float_as_uint(src[j]);
                if (j + 1u < n) v[u].y = __float_as_uint(src[j + 1u]);
                if (j + 2u < n) v[u].z = __float_as_uint(src[j + 2u]);
                missing |= (0xfu << (j < n ? n - j : 0u) & 0xfu) << (4u * u);
            }
        }
    }
    for (uint32_t i = tid; i < (k_var + 2u) * (BLOCK / 16u); i += BLOCK)
        reinterpret_cast<uint4*>(s_col)[i] = make_uint4(0, 0, 0, 0);
    s_cnt[tid] = 0;
    static_assert(SPEC_MULTI_MAXK * PASS_COPIES == BLOCK, "one counter per thread");
    if (tid < k_var) s_part[tid] = make_uint2(coff + csb * ccap, ccap);
    if (tid == 0) s_nan = 0;
    reinterpret_cast<uint4*>(s_tab)[tid] = piece;
    __syncthreads();

    uint32_t key_max = 0;   // a NaN's key is above that of +inf
    // of every weight: j, and for a candidate the counter it goes by (slot << 16) and its place there
    uint32_t cl[4 * U], cmask = 0;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
        const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) {
            const uint32_t key = x[q] & 0x7fffffffu;
            key_max = max(key_max, key);
            const uint32_t at = key >> SAMPLE_BIN_SHIFT;
            cl[4u * u + q] = s_tab[min(at > tab_first ? at - tab_first : 0u, PASS_TAB - 1u)];
            if (wide) cl[4u * u + q] = tab[PASS_TAB + sample_bin(key)];
        }
    }
    if (n != TILE) {
#pragma unroll
        for (uint32_t i = 0; i < 4u * U; ++i)
            if ((missing >> i) & 1u) cl[i] = k_var + 1u;
    }
    uint8_t* my_col = reinterpret_cast<uint8_t*>(s_col) + tid;
#pragma unroll
    for (uint32_t i = 0; i < 4u * U; ++i) {
        cmask |= (cl[i] >> 7) << i;
        cl[i] &= 63u;
        my_col[cl[i] * BLOCK] += 1;          // private byte, at most 16
    }
    // the candidates to the regions of their clusters: counted by cluster and eight lanes in LDS (all
    // of a wavefront's may belong to one cluster, and additions that meet take their turns), one
    // global reservation per cluster the block met, then the writes
    if (__syncthreads_or(cmask ? 1 : 0)) {   // uniform
        const uint32_t copy = (tid >> 3) & (PASS_COPIES - 1u);
#pragma unroll
        for (uint32_t i = 0; i < 4u * U; ++i) {
            if ((cmask >> i) & 1u) {
                const uint32_t slot = (cl[i] - 1u) * PASS_COPIES + copy;
                cl[i] = atomicAdd(&s_cnt[slot], 1u) | (slot << 16);
            }
        }
        __syncthreads();
        {
            const uint32_t mine = s_cnt[tid], last = PASS_COPIES - 1u;
            uint32_t incl = mine;
            for (uint32_t d = 1; d < PASS_COPIES; d <<= 1) {
                const uint32_t y = __shfl_up(incl, d, PASS_COPIES);
                if ((tid & last) >= d) incl += y;
            }
            uint32_t base = 0;
            if ((tid & last) == last && incl) base = atomicAdd(mcnt_cand(cnt, tid / PASS_COPIES, csb), incl);
            base = __shfl(base, (int)last, PASS_COPIES);
            s_cnt[tid] = base + incl - mine;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t i = 4u * u + q;
                if ((cmask >> i) & 1u) {
                    const uint32_t at = s_cnt[cl[i] >> 16] + (cl[i] & 0xffffu);
                    const uint2 part = s_part[(cl[i] >> 16) / PASS_COPIES];
                    if (at < part.y) cand[part.x + at] = make_uint2(x[q], g0 + (tid + BLOCK * u) * 4u + q);
                }
            }
        }
    }
    if (key_max > 0x7f800000u) s_nan = 1;
    __syncthreads();
    // column sums: four threads per j, a quarter of the row's words each (rotated by j: the
    // rows start in the same bank); bytes are added in two 16-bit lanes per word
    if (tid < 4 * (k_var + 1)) {
        const uint32_t j = tid >> 2, q = tid & 3u;
        constexpr uint32_t ROW_W = BLOCK / 4;
        uint32_t even = 0, odd = 0;
        for (uint32_t i = 0; i < ROW_W / 4; ++i) {
            const uint32_t x = s_col[j * ROW_W + ((q * (ROW_W / 4) + i + j) & (ROW_W - 1))];
            even += x & 0x00ff00ffu;
            odd += (x >> 8) & 0x00ff00ffu;
        }
        const uint32_t c = (even & 0xffffu) + (even >> 16) + (odd & 0xffffu) + (odd >> 16);
        if (c) atomicAdd(mcnt_below(cnt, j, sb), c);
    }
    if (tid == 0 && s_nan) atomicOr(&ms->status, 2u);
}

// The finish, two launches over the candidates.
//   hist    grid (part, rank): a 256-bin histogram of (key - lo) >> sh over one part of a
//           cluster's region, added to the cluster's histogram in global memory;
//   finish  grid (part, rank): every block first locates its rank - totals of the split
//           counters, the check that makes the result exact (below < P <= below + candidates
//           of the cluster), the bin holding the P-th pair - and then moves its part's pairs
//           of that bin to the rank's list (one reservation per block).  The rank's block that
//           ends last refines the list with 4096-bin histograms until a bin holds
//           at most FIN_LIST pairs, ranks those exactly by counting and writes the record,
//           to d_thr and to its mirror in pinned host memory, with the rank's status word
//           (bit 0: could not decide; bit 1: NaN; bit 2: a buffer was full or too many
//           weights share the threshold's key - wider intervals would not help).
// What bounds it is the chain of latencies: the counters, the histogram and the part's first
// candidates are loaded before the first of them is used, the sums are taken side by side by
// different wavefronts, and the ranking costs no launch of its own (filter + rank of fifteen ranks
// on 0.86 M weights 11.9 + 6.6 us, 18.1 as one; of eight on 10 M 9.3 + 6.7 and 11.9).
constexpr uint32_t MF_THREADS = 1024, MF_DEPTH = 8;
constexpr uint32_t MF_BINS1 = 256;
constexpr uint32_t MF_STAGE = 2048;      // pairs of the selected bin that one part may hold
// Parts that one block of the finish takes at most.  Its 96 registers let a compute unit run one block of 1024
// threads, so with a block for each of 32 parts nine ranks and more took two rounds or three: a block
// takes as many parts as make one round, with room in LDS for all of them (90 KB, which alone keeps a second block
// out now).  Kernel, us: fifteen ranks of 0.86 M weights 17.2 -> 12.3, twenty of 25.5 M
// 20.4 -> 15.4, ten of 14.7 M with ties 33.0 -> 30.0.  (Registers cut to what two blocks need, with one part's room
// in LDS, spill: 19.9, 24.2, 37.3.)
constexpr uint32_t MF_PARTS = 4;

// f(pair) for the n pairs at src, MF_DEPTH loads per thread in flight.
template <typename F>
__device__ __forceinline__ void ms_walk(const uint2* __restrict__ src, uint32_t n, F&& f) {
    for (uint32_t i0 = 0; i0 < n; i0 += MF_THREADS * MF_DEPTH) {
        uint2 c[MF_DEPTH];
#pragma unroll
        for (uint32_t u = 0; u < MF_DEPTH; ++u) {
            const uint32_t i = i0 + u * MF_THREADS + threadIdx.x;
            c[u] = i < n ? src[i] : make_uint2(0xffffffffu, 0xffffffffu);
        }
#pragma unroll
        for (uint32_t u = 0; u < MF_DEPTH; ++u)
            if (i0 + u * MF_THREADS + threadIdx.x < n) f(c[u]);
    }
}

__global__ __launch_bounds__(MF_THREADS) void ms_hist_kernel(
    const MultiState* __restrict__ ms, const uint32_t* __restrict__ cnt,
    const uint2* __restrict__ cand, uint32_t* ghist, uint64_t* rowsum, uint32_t k_var) {
    __shared__ uint32_t h[MF_BINS1];
    if (blockIdx.y == k_var) {
        // the layer of blocks past the ranks adds up the rows of split counters (row j:
        // weights with exactly j lower ends at or below their key), one row per wavefront
        static_assert(SPEC_SUB == 256, "four counters per lane");
        const uint32_t lane = threadIdx.x & 63u;
        const uint32_t j = blockIdx.x * (MF_THREADS / 64) + (threadIdx.x >> 6);
        if (j <= k_var) {
            uint64_t v = 0;
#pragma unroll
            for (uint32_t q = 0; q < SPEC_SUB / 64; ++q) v += cnt[((size_t)j * SPEC_SUB + q * 64u + lane) * 32u];
            for (uint32_t d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
            if (lane == 0) rowsum[j] = v;
        }
        return;
    }
    const uint32_t part = blockIdx.x, cl = blockIdx.y;
    const RankIn R = ms->rin[cl];
    if (R.clast != cl) return;                       // only a cluster's last rank owns a region
    const uint32_t cap = R.cand_cap;
    const uint32_t n = min(cnt[((size_t)(MAXK + 1u + cl) * SPEC_SUB + part) * 32u], cap);
    if (n == 0) return;
    if (threadIdx.x < MF_BINS1) h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lo = R.lo, sh = R.sh;
    ms_walk(cand + (size_t)R.cand_off + (size_t)part * cap, n,
            [&](uint2 c) { lds_count(h, ((c.x & 0x7fffffffu) - lo) >> sh, true); });
    __syncthreads();
    if (threadIdx.x < MF_BINS1) {
        const uint32_t c = h[threadIdx.x];
        if (c) atomicAdd(&ghist[cl * MF_BINS1 + threadIdx.x], c);
    }
}

__global__ __launch_bounds__(MF_THREADS) void ms_finish_kernel(
    MultiState* ms, const uint32_t* __restrict__ cnt, const uint2* __restrict__ cand,
    const uint32_t* __restrict__ ghist, const uint64_t* __restrict__ rowsum, uint2* list, uint32_t* rank_words,
    uint32_t n_parts, shifter_threshold* thr, shifter_threshold* host_rec, uint32_t* host_status) {
    static_assert(MF_THREADS == FIN_THREADS && MF_BINS1 == 4u * 64u && CAND_SUB <= 64u, "a wavefront for each sum");
    __shared__ uint2 stage[MF_STAGE * MF_PARTS];
    __shared__ uint32_t h[FIN_BINS];
    __shared__ uint64_t comp[FIN_LIST];
    __shared__ uint64_t smem[FIN_THREADS / 64 + 1];
    __shared__ uint64_t s_below, s_inside, s_r2, s_less, s_sel, s_base2;
    __shared__ uint32_t s_over, s_n, s_base, s_bin, s_cnt, s_last, s_why, s_lt, s_eq, s_nb;
    __shared__ TiedLds s_tied;
    static_assert(FIN_LIST <= FIN_THREADS && FIN_DIRECT <= TIED_DIRECT, "more than TIED_DIRECT have one key, and a thread each");
    const uint32_t part = blockIdx.x, k = blockIdx.y;     // the block's parts: part, part + gridDim.x, ...
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const RankIn R = ms->rin[k];
    const uint32_t nan_bit = ms->status & 2u;      // the pass has ended
    const uint32_t cl = R.clast, cap = R.cand_cap, lo = R.lo;
    const uint64_t p = R.p;
    uint32_t *list_cnt = rank_words + k, *ticket = rank_words + MAXK + k, *fail = rank_words + 2u * MAXK + k;
    const uint32_t* parts = cnt + (size_t)(MAXK + 1u + cl) * SPEC_SUB * 32u;
    // this part's first candidates, on their way while the rank is located
    uint32_t n_of[MF_PARTS];
#pragma unroll
    for (uint32_t i = 0; i < MF_PARTS; ++i)
        n_of[i] = part + i * gridDim.x < n_parts ? min(parts[(part + i * gridDim.x) * 32u], cap) : 0u;
    const uint32_t n_part = n_of[0];
    const uint2* src1 = cand + (size_t)R.cand_off + (size_t)part * cap;
    uint2 ahead[MF_DEPTH];
#pragma unroll
    for (uint32_t u = 0; u < MF_DEPTH; ++u) {
        const uint32_t i = u * MF_THREADS + threadIdx.x;
        ahead[u] = i < n_part ? src1[i] : make_uint2(0u, 0u);
    }
    uint4 hc = make_uint4(0, 0, 0, 0);
    uint32_t incl = 0;
    if (wid == 0) {
        // weights below the cluster's interval: rows 0 .. k of the split counters
        uint64_t v = lane <= k ? rowsum[lane] : 0;     // k < MAXK = 64
        for (uint32_t d = 32; d > 0; d >>= 1) v += __shfl_down((unsigned long long)v, d, 64);
        if (lane == 0) { s_below = v; s_n = 0; s_bin = 0xffffffffu; }
    } else if (wid == 1) {
        const uint32_t c = lane < CAND_SUB ? parts[lane * 32u] : 0u;
        const bool over = __ballot(c > cap) != 0ull;
        uint64_t v = c;
        for (uint32_t d = 32; d > 0; d >>= 1) v += __shfl_down((unsigned long long)v, d, 64);
        if (lane == 0) { s_inside = v; s_over = over; }
    } else if (wid == 2) {
        hc = reinterpret_cast<const uint4*>(ghist + cl * MF_BINS1)[lane];
        incl = hc.x + hc.y + hc.z + hc.w;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
    }
    __syncthreads();
    const uint64_t below = s_below, inside = s_inside;
    const bool reached = !s_over && below < p && p <= below + inside;
    if (wid == 2 && reached) {
        const uint64_t r = p - below;
        const uint32_t c4[4] = {hc.x, hc.y, hc.z, hc.w};
        uint64_t base = incl - (hc.x + hc.y + hc.z + hc.w);
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            if (base < r && r <= base + c4[i]) {
                s_bin = lane * 4u + i;
                s_cnt = c4[i];
                s_r2 = r - base;
                s_less = below + base;
            }
            base += c4[i];
        }
    }
    __syncthreads();
    auto give_up = [&](uint32_t why) {             // by one block of the rank
        if (threadIdx.x == 0) {
            atomicOr(&ms->status, 1u);
            host_status[k] = why | 1u | nan_bit;
        }
    };
    const uint32_t bin = s_bin;
    {
        // the same in every block of the rank (no bin: cannot happen unless the buffers were disturbed)
        uint32_t why = 0;
        if (s_over) why = 5u;
        else if (!reached || bin == 0xffffffffu) why = 1u;
        else if (s_cnt > SPEC_LIST_CAP) why = 5u;
        if (why) {
            if (part == 0) give_up(why);
            return;
        }
    }
    // the parts' pairs of the selected bin -> the rank's list
    {
        const uint32_t sh = R.sh;
        auto take = [&](uint2 x) {
            if ((((x.x & 0x7fffffffu) - lo) >> sh) == bin) {
                const uint32_t pos = atomicAdd(&s_n, 1u);
                if (pos < MF_STAGE * MF_PARTS) stage[pos] = x;
            }
        };
#pragma unroll
        for (uint32_t u = 0; u < MF_DEPTH; ++u)
            if (u * MF_THREADS + threadIdx.x < n_part) take(ahead[u]);
        if (n_part > MF_DEPTH * MF_THREADS) ms_walk(src1 + MF_DEPTH * MF_THREADS, n_part - MF_DEPTH * MF_THREADS, take);
        __syncthreads();
        uint32_t m = s_n;
        bool over = m > MF_STAGE;
#pragma unroll
        for (uint32_t i = 1; i < MF_PARTS; ++i) {
            if (part + i * gridDim.x >= n_parts) break;          // the same in every thread
            __syncthreads();                                     // all have read s_n
            ms_walk(src1 + (size_t)i * gridDim.x * cap, n_of[i], take);
            __syncthreads();
            over = over || s_n - m > MF_STAGE;
            m = s_n;
        }
        if (over) {
            if (threadIdx.x == 0) atomicOr(fail, 5u);
        } else if (m != 0) {
            if (threadIdx.x == 0) s_base = atomicAdd(list_cnt, m);
            __syncthreads();
            uint2* dst = list + (size_t)k * SPEC_LIST_CAP;
            for (uint32_t i = threadIdx.x; i < m; i += MF_THREADS)
                if (s_base + i < SPEC_LIST_CAP) store_device(&dst[s_base + i], stage[i]);
        }
    }
    // the list is complete when the rank's last ticket is drawn
    if (!last_block(ticket, gridDim.x, &s_last)) return;
    if (threadIdx.x == 0) {
        s_n = atomicAdd(list_cnt, 0u);
        s_why = atomicOr(fail, 0u);
    }
    __syncthreads();
    const uint32_t n = s_n;
    if (s_why) { give_up(s_why); return; }
    if (n != s_cnt || n > SPEC_LIST_CAP) { give_up(5u); return; }
    // a list that fits stays in LDS
    const uint2* src = list + (size_t)k * SPEC_LIST_CAP;
    const bool staged = n <= MF_STAGE * MF_PARTS;
    if (staged) {
        for (uint32_t i = threadIdx.x; i < n; i += FIN_THREADS) stage[i] = load_device(&src[i]);
        __syncthreads();
    }
    auto walk = [&](auto&& f) {
        for (uint32_t i = threadIdx.x; i < n; i += FIN_THREADS) f(staged ? stage[i] : load_device(&src[i]));
    };
    if (threadIdx.x == 0) { s_sel = 0; s_nb = 0; s_lt = 0; s_eq = 0; }
    uint64_t r = s_r2;               // 1-based rank among the pairs still in play
    uint64_t less = s_less;          // weights below them
    uint32_t width_sh = R.sh;        // the pairs in play have (key - lo_cur) >> width_sh == 0
    uint32_t lo_cur = R.lo + (bin << width_sh);
    uint32_t cnt_sel = n;
    // refine while it pays: ranking by counting is quadratic; a bin of equal keys cannot be
    // refined and must fit the list
    while (cnt_sel > FIN_DIRECT) {
        if (width_sh == 0) {
            if (cnt_sel > FIN_LIST) { give_up(5u); return; }   // the multi-pass select ranks so many ties
            break;
        }
        const uint32_t sh = width_sh > 12u ? width_sh - 12u : 0u;
        for (uint32_t i = threadIdx.x; i < FIN_BINS; i += FIN_THREADS) h[i] = 0;
        __syncthreads();
        walk([&](uint2 c) {
            const uint32_t d = (c.x & 0x7fffffffu) - lo_cur;      // wraps for keys below lo_cur
            if ((d >> width_sh) == 0) lds_count(h, d >> sh, true);
        });
        __syncthreads();
        constexpr uint32_t PER = FIN_BINS / FIN_THREADS;
        const uint32_t b0 = threadIdx.x * PER;
        uint64_t sum = 0, tot;
        uint32_t c4[PER];
#pragma unroll
        for (uint32_t i = 0; i < PER; ++i) { c4[i] = h[b0 + i]; sum += c4[i]; }
        uint64_t base = block_excl_scan_u64<FIN_THREADS>(sum, smem, &tot);
        if (base < r && r <= base + sum) {
#pragma unroll
            for (uint32_t i = 0; i < PER; ++i) {
                if (base < r && r <= base + c4[i]) { s_bin = b0 + i; s_cnt = c4[i]; s_base2 = base; }
                base += c4[i];
            }
        }
        __syncthreads();
        if (tot < r) { give_up(1u); return; }    // cannot happen unless the buffers were disturbed
        less += s_base2;
        r -= s_base2;
        lo_cur += s_bin << sh;
        width_sh = sh;
        cnt_sel = s_cnt;
        __syncthreads();
    }
    __syncthreads();
    // the pairs of the last bin, then the r-th of them by counting
    walk([&](uint2 c) {
        const uint32_t key = c.x & 0x7fffffffu, d = key - lo_cur;
        if ((d >> width_sh) == 0) {
            const uint32_t pos = atomicAdd(&s_nb, 1u);
            if (pos < FIN_LIST) comp[pos] = ((uint64_t)key << 32) | c.y;
        }
    });
    __syncthreads();
    if (s_nb != cnt_sel || r == 0 || r > cnt_sel) { give_up(1u); return; }
    uint32_t want = (uint32_t)r - 1u;
    auto count = [&](const uint64_t* among, uint32_t n_among) {
        for (uint32_t i = threadIdx.x; i < n_among; i += FIN_THREADS) {
            const uint64_t c = among[i];
            uint32_t rank = 0;
            for (uint32_t f = 0; f < n_among; ++f) rank += among[f] < c;
            if (rank == want) s_sel = c;        // composites are distinct: exactly one hit
        }
    };
    if (cnt_sel > TIED_DIRECT) {
        uint64_t* few = reinterpret_cast<uint64_t*>(stage);      // the list has been read
        const uint2 left = tied_stretch<FIN_THREADS, FIN_BINS>(comp, cnt_sel, want, h, smem, few, &s_tied);
        want = left.y;
        count(few, left.x);
    } else {
        count(comp, cnt_sel);
    }
    __syncthreads();
    const uint64_t sel = s_sel;
    const uint32_t key = (uint32_t)(sel >> 32);
    uint32_t lt = 0, eq = 0;
    for (uint32_t i = threadIdx.x; i < cnt_sel; i += FIN_THREADS) {
        const uint32_t kk = (uint32_t)(comp[i] >> 32);
        lt += kk < key;
        eq += kk == key;
    }
    if (lt) atomicAdd(&s_lt, lt);
    if (eq) atomicAdd(&s_eq, eq);
    __syncthreads();
    if (threadIdx.x == 0) {
        shifter_threshold out;
        out.reserved = 0;
        out.n_prune = p;
        out.t_key = key;
        out.g_cut = sel & 0xffffffffull;
        out.cut = sel + 1;
        out.n_less = less + s_lt;
        out.n_equal = s_eq;
        thr[R.perm] = out;
        host_rec[R.perm] = out;
        host_status[k] = nan_bit;
    }
}

// ---------------------------------------------------------------------------------------
// Steps 1-3 for the K variants of a portfolio in ONE read of the arena: ms_pass_kernel's
// counting and candidate capture merged with the batched mask pass.  For a weight with
// j = #{r : lo_r <= key} over the sorted ranks, rank r removes it for sure when r >= j and
// keeps it for sure when hi_r < key; in between it is a candidate of r.  The pass writes
// every variant's sparse weight and mask byte - candidates provisionally - and the
// levels of the weights that are no rank's candidate; ms_fixup_kernel, once the exact cuts
// are known, rewrites the candidates written on the wrong side of their rank's cut (the
// pass decides by the predicted threshold mid of the last rank) and adds their levels.
// rv[v] = sorted rank of variant v, or -1 for a variant that removes nothing (P = 0).
// Bound by its stores: ten variants of 322 M weights take 3.42 ms, the same loads and stores without any of the work
// 3.33.  So the classification by search, an atomic per weight for the levels and ragged tiles weight by weight, which
// ms_pass_kernel and mask_scan_batch_kernel have left for faster forms, stay here.
struct VariantRanks {
    int32_t r[MAXK];
};

template <bool NT>
__global__ __launch_bounds__(BLOCK) void ms_fused_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix, uint32_t n_t,
    const float* __restrict__ w, MultiState* ms, uint32_t* cnt, uint2* __restrict__ cand,
    VariantRanks rv, uint32_t k_all, float* __restrict__ w_out,
    uint64_t w_stride, uint8_t* __restrict__ mask, uint64_t mask_stride, uint32_t* out_level,
    uint32_t* in_level) {
    __shared__ uint32_t rowmax[TILE + 16];
    __shared__ uint32_t colmax[TILE + 16];
    __shared__ uint32_t s_lo[MAXK + 1], s_hi[MAXK + 1], s_mid[MAXK + 1];
    __shared__ uint32_t s_coff[MAXK], s_ccap[MAXK], s_rc[MAXK], s_rc2[MAXK], s_rbase[MAXK];
    __shared__ int32_t s_rv[MAXK];
    __shared__ uint8_t s_col[(SPEC_MULTI_MAXK + 1) * BLOCK];   // private counters, <= 16 each
    __shared__ __align__(16) uint32_t s_xm[TILE / 4];
    __shared__ uint32_t s_nan;

    const uint32_t tile = blockIdx.x;
    const uint32_t t = find_tensor(tile_prefix, n_t, tile);
    const DevTensor T = tens[t];
    const uint32_t e0 = (tile - tile_prefix[t]) * TILE;
    const uint32_t n = min(TILE, T.numel - e0);
    const bool ranked = T.prunable != 0;
    const uint32_t g0 = (uint32_t)(T.gbase + e0);
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t sb = blockIdx.x & (SPEC_SUB - 1);
    const uint32_t k_var = ms->k;
    const uint32_t c0 = e0 % T.khw, r0 = e0 % T.row_len;
    const uint32_t nrows = (r0 + n - 1) / T.row_len + 1;
    const uint32_t ncols = (c0 + n - 1) / T.khw + 1;
    for (uint32_t s = threadIdx.x; s < nrows; s += BLOCK) rowmax[s] = 0;
    for (uint32_t s = threadIdx.x; s < ncols; s += BLOCK) colmax[s] = 0;
    if (threadIdx.x <= MAXK) {
        s_lo[threadIdx.x] = threadIdx.x < MAXK ? ms->lo[threadIdx.x] : 0xffffffffu;
        s_hi[threadIdx.x] = threadIdx.x < MAXK ? ms->hi[threadIdx.x] : 0xffffffffu;
        s_mid[threadIdx.x] = threadIdx.x < MAXK ? ms->mid[threadIdx.x] : 0xffffffffu;
    }
    if (threadIdx.x < MAXK) {
        s_rv[threadIdx.x] = rv.r[threadIdx.x];
        s_coff[threadIdx.x] = ms->cand_off[threadIdx.x];
        s_ccap[threadIdx.x] = ms->cand_cap[threadIdx.x];
        s_rc[threadIdx.x] = 0;
        s_rc2[threadIdx.x] = 0;
    }
    for (uint32_t j = 0; j <= k_var; ++j) s_col[j * BLOCK + threadIdx.x] = 0;
    if (threadIdx.x == 0) s_nan = 0;
    __syncthreads();

    uint32_t nan = 0;
    // number of ranks that keep one weight in what the pass writes (127 in tensors that are
    // not ranked: no rank removes it) and whether it is a candidate; counts it under
    // j = #{r : lo_r <= key}.  Ranks below j keep a weight that is no candidate.
    auto classify = [&](uint32_t bits, bool& is_cand, bool& below_mid) -> uint32_t {
        is_cand = false;
        below_mid = false;
        if (!ranked) return 127u;
        const uint32_t key = bits & 0x7fffffffu;
        nan |= key > 0x7f800000u ? 1u : 0u;
        uint32_t j = count_lower_ends(s_lo, key);
        is_cand = j >= 1 && key <= s_hi[j - 1];
        s_col[j * BLOCK + threadIdx.x] += 1;
        // a candidate is written as kept by the ranks below j - 1 and by rank j - 1 iff it
        // does not lie below that rank's predicted threshold (the fix-up settles it, in every
        // rank of its cluster)
        below_mid = is_cand && key < s_mid[j - 1];
        if (below_mid) j -= 1;
        return j;
    };
    auto mark = [&](uint32_t j, uint32_t bits, uint32_t level) {
        if (level && (bits & 0x7fffffffu)) {
            atomicMax(&rowmax[div_small(r0 + j, T.row_len, T.magic_row)], level);
            atomicMax(&colmax[div_small(c0 + j, T.khw, T.magic_khw)], level);
        }
    };

    const float* src = w + T.offset + e0;
    const bool want_mask = ranked && mask != nullptr;
    if (n == TILE) {
        constexpr uint32_t U = TILE / BLOCK / 4;
        const uint32_t q0 = wid * (64u * U) + lane;      // quad of step 0 (see the batched mask pass)
        uint4 v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) v[u] = load_u4<NT>(src + 4u * q0 + 256u * u);
        uint32_t jj[U], cmask = 0, bmask = 0, lvl[U][4];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            bool c_0, c_1, c_2, c_3, b_0, b_1, b_2, b_3;
            const uint32_t j_0 = classify(v[u].x, c_0, b_0), j_1 = classify(v[u].y, c_1, b_1);
            const uint32_t j_2 = classify(v[u].z, c_2, b_2), j_3 = classify(v[u].w, c_3, b_3);
            jj[u] = j_0 | (j_1 << 8) | (j_2 << 16) | (j_3 << 24);
            cmask |= ((c_0 ? 1u : 0u) | (c_1 ? 2u : 0u) | (c_2 ? 4u : 0u) | (c_3 ? 8u : 0u)) << (4 * u);
            bmask |= ((b_0 ? 1u : 0u) | (b_1 ? 2u : 0u) | (b_2 ? 4u : 0u) | (b_3 ? 8u : 0u)) << (4 * u);
            lvl[u][0] = lvl[u][1] = lvl[u][2] = lvl[u][3] = 0;
        }
        uint32_t* xm = s_xm + wid * (64u * U);
        for (uint32_t k = 0; k < k_all; ++k) {
            const int32_t r = s_rv[k];
            float* dst = w_out + (uint64_t)k * w_stride + T.offset + e0;
            uint8_t* mdst = want_mask ? mask + (uint64_t)k * mask_stride + T.gbase + e0 : nullptr;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t b[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                uint32_t o[4], keep[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    keep[q] = r < (int32_t)((jj[u] >> (8 * q)) & 0xffu) ? 1u : 0u;
                    o[q] = keep[q] ? b[q] : 0u;
                    lvl[u][q] += keep[q];
                }
                if (w_out)
                    store_u4<NT>(dst + 4u * q0 + 256u * u,
                                 make_uint4(o[0], o[1], o[2], o[3]));
                if (mdst) xm[64u * u + lane] = keep[0] | (keep[1] << 8) | (keep[2] << 16) | (keep[3] << 24);
            }
            if (mdst) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                store_mask16(mdst + wid * (256u * U) + 16u * lane, *reinterpret_cast<const uint4*>(xm + 4u * lane));
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t j = (q0 + 64u * u) * 4;
            const uint32_t b[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if (!(cmask & (1u << (4 * u + q)))) mark(j + q, b[q], lvl[u][q]);
        }
        // candidate pairs: to the regions of their clusters
        ms_append_candidates(cmask != 0, s_coff, s_ccap, s_rc, s_rc2, s_rbase, k_var, cnt,
                             blockIdx.x & (CAND_SUB - 1), cand,
                             [&](auto&& f) {
#pragma unroll
                                 for (uint32_t u = 0; u < U; ++u) {
                                     const uint32_t j = (q0 + 64u * u) * 4;
                                     const uint32_t vv[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                                     for (uint32_t q = 0; q < 4; ++q)
                                         if (cmask & (1u << (4 * u + q)))
                                             f(vv[q], g0 + j + q,
                                               ((jj[u] >> (8 * q)) & 0xffu) - 1u + ((bmask >> (4 * u + q)) & 1u));
                                 }
                             });
    } else {
        for (uint32_t j0 = 0; j0 < n; j0 += BLOCK) {
            const uint32_t j = j0 + threadIdx.x;
            if (j < n) {
                const uint32_t bits = __float_as_uint(src[j]);
                bool is_cand, below_mid;
                const uint32_t jr = classify(bits, is_cand, below_mid);
                uint32_t level = 0;
                for (uint32_t k = 0; k < k_all; ++k) {
                    const bool keep = s_rv[k] < (int32_t)jr;
                    level += keep ? 1u : 0u;
                    if (w_out)
                        w_out[(uint64_t)k * w_stride + T.offset + e0 + j] = keep ? __uint_as_float(bits) : 0.0f;
                    if (want_mask) mask[(uint64_t)k * mask_stride + T.gbase + e0 + j] = keep ? 1 : 0;
                }
                if (is_cand) {
                    const uint32_t cl = jr - 1u + (below_mid ? 1u : 0u);
                    const uint32_t csb = blockIdx.x & (CAND_SUB - 1);
                    const uint32_t pos = atomicAdd(mcnt_cand(cnt, cl, csb), 1u);
                    const uint32_t cap = s_ccap[cl];
                    if (pos < cap) cand[(size_t)s_coff[cl] + (size_t)csb * cap + pos] = make_uint2(bits, g0 + j);
                } else {
                    mark(j, bits, level);
                }
            }
        }
    }
    for (uint32_t d = 32; d > 0; d >>= 1) nan |= __shfl_down(nan, d, 64);
    if (lane == 0 && nan) s_nan = 1;
    __syncthreads();
    // column sums: four threads per j, a quarter of the columns each
    if (ranked && threadIdx.x < 4 * (k_var + 1)) {
        const uint32_t j = threadIdx.x >> 2, q = threadIdx.x & 3u;
        uint32_t c = 0;
        for (uint32_t i = 0; i < BLOCK / 4; ++i) c += s_col[j * BLOCK + ((i * 4 + q + j) & (BLOCK - 1))];
        if (c) atomicAdd(mcnt_below(cnt, j, sb), c);
    }
    if (threadIdx.x == 0 && s_nan) atomicOr(&ms->status, 2u);
    // levels of the tile's filters and input features
    const uint32_t row_first = e0 / T.row_len;
    for (uint32_t s = threadIdx.x; s < nrows; s += BLOCK) {
        const uint32_t l = rowmax[s];
        if (l) {
            uint32_t* f = out_level + T.out_flag_off + row_first + s;
            if (*f < l) atomicMax(f, l);
        }
    }
    const uint32_t bfeat = (e0 / T.khw) % T.in_ch;
    for (uint32_t s = threadIdx.x; s < ncols; s += BLOCK) {
        const uint32_t l = colmax[s];
        if (l) {
            uint32_t* f = in_level + T.in_flag_off + mod_small(bfeat + s, T.in_ch, T.magic_in);
            if (*f < l) atomicMax(f, l);
        }
    }
}

// ranks whose interval holds key: [ka, kb)
__device__ __forceinline__ void rank_range(const uint32_t* s_lo, const uint32_t* s_hi, uint32_t key,
                                           uint32_t* ka, uint32_t* kb) {
    uint32_t j = 0, a = 0;
#pragma unroll
    for (uint32_t step = MAXK / 2; step >= 1; step >>= 1) {
        if (s_lo[j + step - 1] <= key) j += step;
        if (s_hi[a + step - 1] < key) a += step;
    }
    j += s_lo[j] <= key ? 1u : 0u;
    a += s_hi[a] < key ? 1u : 0u;
    *ka = a;   // first k with hi_k >= key
    *kb = j;   // #{k : lo_k <= key}
}

// Settles the candidates of ms_fused_kernel with the exact cuts: the pass wrote a
// candidate of ranks [a, j) as kept in all of them but the last, and in rank j - 1 iff
// key >= mid_{j-1}; here it is rewritten in every rank where that was the wrong side of
// the exact cut, and its level (variants that keep it: those that remove nothing, the
// ranks below a, and the ranks of [a, j) that keep it) goes into the level arrays.
// blockIdx.x: part of the region, blockIdx.y: rank (only a cluster's last rank owns a
// region), blockIdx.z: which of gridDim.z interleaved slices of the part.
__global__ __launch_bounds__(BLOCK) void ms_fixup_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ ranked_ids, uint32_t n_ranked,
    const MultiState* __restrict__ ms, const uint32_t* __restrict__ cnt,
    const uint2* __restrict__ cand, const shifter_threshold* __restrict__ thr,
    uint32_t n_zero, float* __restrict__ w_out, uint64_t w_stride, uint8_t* __restrict__ mask,
    uint64_t mask_stride, uint32_t* out_level, uint32_t* in_level) {
    constexpr uint32_t LDS_T = 1024;
    __shared__ uint32_t s_gbase[LDS_T];
    __shared__ uint32_t s_lo[MAXK + 1], s_hi[MAXK + 1], s_mid[MAXK], s_perm[MAXK];
    __shared__ uint64_t s_cut[MAXK];
    if (ms->status & 1u) return;
    const uint32_t cl = blockIdx.y, sb = blockIdx.x;
    if (ms->clast[cl] != cl) return;
    const uint32_t cap = ms->cand_cap[cl];
    const uint32_t n = min(cnt[((size_t)(MAXK + 1u + cl) * SPEC_SUB + sb) * 32u], cap);
    if (n == 0) return;
    const uint2* src = cand + (size_t)ms->cand_off[cl] + (size_t)sb * cap;
    const uint32_t k_var = ms->k;
    const bool in_lds = n_ranked <= LDS_T;
    if (in_lds)
        for (uint32_t i = threadIdx.x; i < n_ranked; i += BLOCK)
            s_gbase[i] = (uint32_t)tens[ranked_ids[i]].gbase;
    if (threadIdx.x <= MAXK) {
        s_lo[threadIdx.x] = threadIdx.x < MAXK ? ms->lo[threadIdx.x] : 0xffffffffu;
        s_hi[threadIdx.x] = threadIdx.x < MAXK ? ms->hi[threadIdx.x] : 0xffffffffu;
    }
    if (threadIdx.x < k_var) {
        s_perm[threadIdx.x] = ms->perm[threadIdx.x];
        s_cut[threadIdx.x] = thr[ms->perm[threadIdx.x]].cut;
        s_mid[threadIdx.x] = ms->mid[threadIdx.x];
    }
    __syncthreads();
    auto settle = [&](uint2 c) {
        const uint32_t key = c.x & 0x7fffffffu;
        uint32_t ka, kb;
        rank_range(s_lo, s_hi, key, &ka, &kb);
        kb = min(kb, k_var);
        const uint64_t comp = ((uint64_t)key << 32) | c.y;
        uint32_t a = 0, b = n_ranked;   // tensor holding global index c.y
        while (b - a > 1) {
            const uint32_t m2 = (a + b) >> 1;
            const uint32_t gb = in_lds ? s_gbase[m2] : (uint32_t)tens[ranked_ids[m2]].gbase;
            if (gb <= c.y) a = m2; else b = m2;
        }
        const DevTensor& T = tens[ranked_ids[a]];
        const uint32_t e = c.y - (uint32_t)T.gbase;
        uint32_t level = n_zero + ka;
        for (uint32_t r = ka; r < kb; ++r) {
            const bool removed = comp < s_cut[r];
            const bool written_removed = r + 1 == kb && key < s_mid[r];
            if (removed != written_removed) {    // written on the wrong side of the exact cut
                const uint32_t v = s_perm[r];
                if (w_out) w_out[(uint64_t)v * w_stride + T.offset + e] = removed ? 0.0f : __uint_as_float(c.x);
                if (mask) mask[(uint64_t)v * mask_stride + c.y] = removed ? 0 : 1;
            }
            level += removed ? 0u : 1u;
        }
        if (key != 0 && level != 0) {
            uint32_t* f = out_level + T.out_flag_off + e / T.row_len;
            if (*f < level) atomicMax(f, level);
            f = in_level + T.in_flag_off + (e / T.khw) % T.in_ch;
            if (*f < level) atomicMax(f, level);
        }
    };
    // four pairs per thread and step, their loads in flight together
    constexpr uint32_t U = 4;
    for (uint32_t i0 = blockIdx.z * U * BLOCK; i0 < n; i0 += gridDim.z * U * BLOCK) {
        uint2 c[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * BLOCK + threadIdx.x;
            c[u] = i < n ? src[i] : make_uint2(0, 0);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (i0 + u * BLOCK + threadIdx.x < n) settle(c[u]);
    }
}

void launch_spec_multi(shifter_ctx* ctx, const shifter_model* m, const float* d_w,
                       const PruneCounts& sorted_p, const MultiPerm& perm, uint32_t k,
                       uint64_t zero_mask, shifter_threshold* d_thr, const FusedBatch* fb,
                       uint32_t* zero_ptr, uint32_t zero_n) {
    const auto& b = m->b;
    const uint32_t n_t = (uint32_t)m->t.size();
    hipStream_t s = ctx->stream;
    if (k == 0 && fb) launch_zero_levels(ctx, m);
    {
        // the fused pass adds to the level arrays: cleared on the way.  At least a block per rank: the
        // ranks' counters lie on 512 lines each, too many for one block to clear (fifteen ranks, 264
        // tiles: 22.2 us with one block, 16.7 with fifteen)
        ProfileScope ps(ctx, K_SPEC_SAMPLE);
        ms_front_kernel<<<k ? std::max(sample_grid(m), k) : 1u, SAMPLE_THREADS, 0, s>>>(
            sample_in(m, d_w), b.multi, b.multi_cnt, b.multi_hist, b.multi_list_cnt, fb && k ? b.levels : nullptr,
            fb && k ? (uint32_t)(m->info.sum_out_ch + m->info.sum_in_ch) : 0u, sorted_p, perm, k, m->sample_size,
            zero_mask, d_thr, b.dev_multi_rec, m->info.n_prunable, ctx->margin_sigmas, b.multi_tab, b.cand_cap_sb);
    }
    if (k == 0 && !fb) {         // every count was zero: no pass, which would have cleared zero_ptr
        if (zero_ptr) launch_zero_levels(ctx, m);
        return;
    }
    const bool nt = m->info.w_extent * 4 > (192ull << 20);
    if (fb) {
        VariantRanks rv;
        for (uint32_t v = 0; v < MAXK; ++v) rv.r[v] = -1;
        for (uint32_t r = 0; r < k; ++r) rv.r[perm.v[r]] = (int32_t)r;
        ProfileScope ps(ctx, K_MASK_SCAN_BATCH);
        // non-temporal hint as in the batched mask pass: only for cache-sized arenas
        auto kern = !nt ? ms_fused_kernel<true> : ms_fused_kernel<false>;
        kern<<<m->n_tiles, BLOCK, 0, s>>>(b.tens, b.tile_prefix, n_t, d_w, b.multi, b.multi_cnt, b.cand,
                                          rv, fb->k_all, fb->d_w_out, fb->w_stride,
                                          fb->d_mask, fb->mask_stride, b.levels,
                                          b.levels + m->info.sum_out_ch);
    } else {
        ProfileScope ps(ctx, K_SPEC_PASS);
        auto kern = nt ? ms_pass_kernel<true> : ms_pass_kernel<false>;
        kern<<<m->n_tiles, BLOCK, (k + 2) * BLOCK, s>>>(
            b.tens, b.tile_prefix, b.tile_tensor, d_w, b.multi, k, b.multi_cnt, b.cand, b.multi_tab, zero_ptr, zero_n);
    }
    if (k != 0) {
        {
            ProfileScope ps(ctx, K_SPEC_FINISH);
            // CAND_SUB * 16 wavefronts in the extra layer cover the MAXK + 1 rows
            static_assert(CAND_SUB * (MF_THREADS / 64) >= MAXK + 1, "a wavefront per row of counters");
            ms_hist_kernel<<<dim3(CAND_SUB, k + 1), MF_THREADS, 0, s>>>(b.multi, b.multi_cnt, b.cand, b.multi_hist,
                                                                      b.multi_rowsum, k);
        }
        {
            ProfileScope ps(ctx, K_SPEC_FINISH2);
            // the parts that a pass over this many tiles can have filled (twenty ranks of a 24 k weight network, 9
            // tiles: 34 us with 32 parts a rank, 14 with 9), shared out to no more blocks than run at a time
            const uint32_t parts = std::min(CAND_SUB, m->n_tiles);
            const uint32_t per = std::min(MF_PARTS, (parts * k + 255u) / 256u);
            ms_finish_kernel<<<dim3((parts + per - 1u) / per, k), MF_THREADS, 0, s>>>(
                b.multi, b.multi_cnt, b.cand, b.multi_hist, b.multi_rowsum, b.multi_list, b.multi_list_cnt, parts,
                d_thr, b.dev_multi_rec, b.dev_multi_status);
        }
    }
    if (fb) {
        if (k != 0) {
            ProfileScope ps(ctx, K_SPEC_FIXUP);
            ms_fixup_kernel<<<dim3(CAND_SUB, k, 16), BLOCK, 0, s>>>(
                b.tens, b.ranked_ids, m->n_ranked, b.multi, b.multi_cnt, b.cand, d_thr,
                fb->k_all - k, fb->d_w_out, fb->w_stride, fb->d_mask, fb->mask_stride, b.levels,
                b.levels + m->info.sum_out_ch);
        }
        if (!fb->levels_only) launch_expand_levels(ctx, m, d_thr, fb->k_all, fb->d_out_alive, fb->d_in_alive);
    }
}

}  // namespace shifter
