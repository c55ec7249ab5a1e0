// Single-pass exact selection of the P-th smallest (|w|, g) pair for one prune count:
// the unstructured magnitude ranking of Sec. II-A / Sec. III-C of the paper, reached in
// one read of the arena.
//
//   1. sample      a stratified sample of the prunable weights (four 64-byte sectors out of
//                  every sampled tile, spec_sample.h) is histogrammed on 16384 bins of 1/256 of a
//                  binade;
//   2. predict     from the sample's order statistics around P/N, widened by a margin,
//                  a key interval [lo, hi] that should contain the threshold key;
//   3. one pass    over the arena counts the weights below lo and appends the
//                  (key, g) pairs inside [lo, hi] to a candidate buffer.  In the fused
//                  form the same pass already writes the sparse weights, the mask and
//                  the alive flags for every weight outside the interval;
//   4. finish      if  n_below < P <= n_below + n_candidates  the P-th pair is the
//                  (P - n_below)-th candidate: a 256-bin histogram over the candidates,
//                  a 4096-bin one over the selected bin, and an exact rank inside the
//                  last bin give the record; the fused form then settles the candidates.
//
// The result is exact whenever step 4's check holds; otherwise (a sample that misled,
// an interval with too many ties, a full buffer) a status bit is raised and the host
// runs the multi-pass select instead.  Steps 1 and 2 are one launch, and so are the two later
// parts of step 4 (the block that ends last goes on).
#include <algorithm>

#include "spec_sample.h"

namespace shifter {

constexpr uint32_t FBINS1 = 256;        // round-1 finishing histogram: one bin per thread
constexpr uint32_t FHIST_COPIES = 4;    // of it in global memory: blocks that meet at one bin take their turns
constexpr uint32_t FBINS = 4096;        // round-2 finishing histogram (one block, LDS)
// Up to this many tiles the pass counts the candidates' first histogram itself (its blocks add at most 256 bins each to
// four copies), beyond it a launch of its own does.  us a step: 24 k weights (9 tiles) 67.0 -> 65.5, 0.13 M 72.4 -> 71.2, 0.9 M
// (232) 79.8 -> 78.1; with thousands of tiles the pass is bound by memory and the blocks' additions would queue.
constexpr uint32_t PASS_HIST_TILES = SPEC_SUB;
// A tensor's last tile of up to this many weights goes one weight a thread, with an addition per candidate, a longer one
// by fours like a full one: there the quads' branches, the block's prefix sum and the barriers around its one
// addition cost more than they save.  Kernel, us, by fours / singly: 300 tiles of 64 weights 7.2 / 5.4, of 256 6.9 / 5.6, of
// 400 7.0 / 6.2, of 576 7.4 / 8.1; 4000 of 64 20.3 / 14.5.
constexpr uint32_t PASS_SINGLES = 2 * BLOCK;
constexpr uint32_t FIN_BLOCKS = SPEC_FIN_BLOCKS;  // blocks of the passes over candidates
// The last one: few blocks, because all draw a ticket of one address at its end (14 ns each), wide ones, because
// the block that ends last ranks alone; each takes up to FIN_SUBS sub-buffers.
constexpr uint32_t FIN_THREADS = 1024, FIN_SUBS = 4, FIN_AHEAD = 2;
static_assert(FIN_AHEAD * FIN_THREADS <= 2 * TILE, "a sub-buffer's least capacity");

// Global atomics to one address serialise (about 11 ns each on this chip), so every
// counter that all blocks touch is split into SPEC_SUB copies, one 128-byte line each,
// chosen by blockIdx; the candidate buffer is split the same way.
enum { CNT_CAND = 0, CNT_BELOW = 1 };
__device__ __forceinline__ uint32_t* sub_counter(uint32_t* cnt, uint32_t which, uint32_t sb) {
    return cnt + (which * SPEC_SUB + sb) * 32u;
}

// Sample and prediction in one launch.  On the way the scratch of the kernels behind it is cleared: the
// split counters, the candidates' histogram, the caller's flag arrays.
// The block that ends last takes the sample's order statistics around P/N for the candidate
// interval [lo, hi] and a provisional threshold mid (the fused pass writes candidates below mid as
// removed, the others as kept; few of them then need correcting).
__global__ __launch_bounds__(SAMPLE_THREADS) void spec_front_kernel(
    SampleIn in, SpecState* __restrict__ ss, uint32_t* __restrict__ cnt, uint32_t* __restrict__ hist,
    uint8_t* __restrict__ fa, uint64_t na, uint8_t* __restrict__ fb, uint64_t nb, uint64_t p, uint32_t m,
    uint64_t n_prunable, double margin_sigmas) {
    __shared__ __align__(16) uint32_t h[SAMPLE_BINS];
    {
        const uint64_t tid = (uint64_t)blockIdx.x * SAMPLE_THREADS + threadIdx.x;
        const uint64_t stride = (uint64_t)gridDim.x * SAMPLE_THREADS;
        for (uint64_t i = tid; i < 2u * SPEC_SUB; i += stride) cnt[i * 32u] = 0;
        for (uint64_t i = tid; i < FHIST_COPIES * FBINS1; i += stride) hist[i] = 0;
        for (uint64_t i = tid; i < na; i += stride) fa[i] = 0;
        for (uint64_t i = tid; i < nb; i += stride) fb[i] = 0;
    }
    if (!sample_prefix(in, h)) return;
    if (threadIdx.x >= 64u) return;
    // lanes 0, 1, 2: low end, high end, centre
    const uint32_t lane = threadIdx.x;
    const bool use = p > 0 && m >= 256 && n_prunable > 0 && h[SAMPLE_BINS - 1u] == m;
    uint32_t bin = 0xffffffffu;
    double r_hi = 0;
    if (use) {
        const double frac = (double)p / (double)n_prunable;
        const double centre = frac * (double)m;
        // a multiple of the binomial deviation of a simple random sample of this size
        const double delta = margin_sigmas * sqrt((double)m * frac * (1.0 - frac)) + 16.0;
        r_hi = centre + delta;
        const double r = lane == 0 ? centre - delta : lane == 1 ? r_hi : centre;     // 0-based sample rank
        if (r >= 0.0 && r < (double)m) bin = sample_bin_of_rank(h, (uint32_t)r);
    }
    const uint32_t bin_lo = __shfl(bin, 0, 64), bin_hi = __shfl(bin, 1, 64), bin_mid = __shfl(bin, 2, 64);
    if (lane != 0) return;
    uint32_t lo = 0, hi = 0x7fffffffu;
    if (bin_lo != 0xffffffffu) lo = sample_bin_first_key(bin_lo);
    if (bin_hi != 0xffffffffu && r_hi < (double)(m - 1)) hi = sample_bin_last_key(bin_hi);
    uint32_t mid = lo;
    if (bin_mid != 0xffffffffu)      // the middle of the bin
        mid = sample_bin_first_key(bin_mid) + (sample_bin_last_key(bin_mid) - sample_bin_first_key(bin_mid)) / 2u;
    mid = max(lo, min(mid, hi));
    uint32_t sh = 0;
    while (((hi - lo) >> sh) >= FBINS1) ++sh;
    ss->p = p;
    ss->n_below = 0;
    ss->n_inside = 0;
    ss->m_valid = m;
    ss->status = 0;
    ss->list_cnt = 0;
    ss->ticket = 0;
    ss->lo = lo;
    ss->hi = hi;
    ss->mid = mid;
    ss->sh = sh;
}

// The one pass over the arena.  FUSED also writes the sparse weights and the mask of
// every weight (those of the candidates provisionally: removed below mid, kept from mid
// on) and the alive flags of the kept weights outside the candidate interval;
// spec_fixup_kernel settles the candidates.  A candidate pair holds the weight's full bit
// pattern (sign included, so a wrongly removed weight can be restored) and its index.
// HIST: the candidates' first histogram is counted on the way, in LDS, and added to the global one bin by bin.
template <bool FUSED, bool NT, bool HIST>
__global__ __launch_bounds__(BLOCK) void spec_pass_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ tile_prefix,
    uint32_t n_t, const float* __restrict__ w, SpecState* ss, uint32_t* cnt,
    uint2* __restrict__ cand, uint32_t cap_sb, uint32_t* __restrict__ hist, float* __restrict__ w_out,
    uint8_t* __restrict__ mask, uint8_t* out_alive, uint8_t* in_alive) {
    __shared__ uint32_t s_h[HIST ? FBINS1 : 1];
    __shared__ uint8_t rowf[FUSED ? TILE + 16 : 16];
    __shared__ uint8_t colf[FUSED ? TILE + 16 : 16];
    __shared__ uint32_t s_below, s_nan, s_base, s_wtot[BLOCK / 64];

    const uint32_t tile = blockIdx.x;
    const uint32_t t = find_tensor(tile_prefix, n_t, tile);
    const DevTensor T = tens[t];
    if (!FUSED && !T.prunable) return;
    const bool ranked = T.prunable != 0 && ss->p != 0;   // P = 0: nothing is removed
    const uint32_t lo = ss->lo, hi = ss->hi, mid = ss->mid;
    const uint32_t e0 = (tile - tile_prefix[t]) * TILE;
    const uint32_t n = min(TILE, T.numel - e0);
    const uint32_t g0 = (uint32_t)(T.gbase + e0);
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t sb = blockIdx.x & (SPEC_SUB - 1);
    uint2* my_cand = cand + (size_t)sb * cap_sb;
    uint32_t c0 = 0, r0 = 0, nrows = 0, ncols = 0;
    if (threadIdx.x == 0) { s_below = 0; s_nan = 0; s_base = 0; }
    const uint32_t sh = HIST ? ss->sh : 0u;
    if (HIST) s_h[threadIdx.x] = 0;
    if (FUSED) {
        c0 = e0 % T.khw;
        r0 = e0 % T.row_len;
        nrows = (r0 + n - 1) / T.row_len + 1;
        ncols = (c0 + n - 1) / T.khw + 1;
        for (uint32_t s = threadIdx.x; s < nrows; s += BLOCK) rowf[s] = 0;
        for (uint32_t s = threadIdx.x; s < ncols; s += BLOCK) colf[s] = 0;
    }
    __syncthreads();

    const float* src = w + T.offset + e0;
    float* dst = FUSED ? w_out + T.offset + e0 : nullptr;
    uint8_t* mdst = (FUSED && T.prunable && mask) ? mask + T.gbase + e0 : nullptr;
    uint32_t below = 0, nan = 0;

    // classifies one weight: returns the bits to store, sets keep / is_cand
    auto one = [&](uint32_t j, uint32_t bits, uint32_t& keep, bool& is_cand) -> uint32_t {
        const uint32_t key = bits & 0x7fffffffu;
        const bool removed = ranked && key < mid;       // lo <= mid <= hi
        is_cand = ranked && key >= lo && key <= hi;
        below += (ranked && key < lo) ? 1u : 0u;
        nan |= (ranked && key > 0x7f800000u) ? 1u : 0u;
        keep = removed ? 0u : 1u;
        if (FUSED && !removed && !is_cand && key != 0) {
            rowf[div_small(r0 + j, T.row_len, T.magic_row)] = 1;
            colf[div_small(c0 + j, T.khw, T.magic_khw)] = 1;
        }
        return removed ? 0u : bits;
    };

    constexpr uint32_t U = TILE / BLOCK / 4;
    uint4 v[U];
    uint32_t cmask = 0;
    if (n == TILE) {
        const float* src4 = src + 4u * threadIdx.x;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) v[u] = load_u4<NT>(src4 + 4u * BLOCK * u);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t j = (threadIdx.x + BLOCK * u) * 4;
            uint32_t k0, k1, k2, k3;
            bool q0, q1, q2, q3;
            uint4 o;
            o.x = one(j, v[u].x, k0, q0);
            o.y = one(j + 1, v[u].y, k1, q1);
            o.z = one(j + 2, v[u].z, k2, q2);
            o.w = one(j + 3, v[u].w, k3, q3);
            cmask |= ((q0 ? 1u : 0u) | (q1 ? 2u : 0u) | (q2 ? 4u : 0u) | (q3 ? 8u : 0u)) << (4 * u);
            if (FUSED) {
                store_u4<NT>(dst + 4u * threadIdx.x + 4u * BLOCK * u, o);
                if (mdst) store_mask4<NT>(mdst + 4u * threadIdx.x + 4u * BLOCK * u, k0 | (k1 << 8) | (k2 << 16) | (k3 << 24));
            }
        }
    } else if (n <= PASS_SINGLES) {
        // a tensor's last tile with few weights: one a thread and step, one addition per candidate
        for (uint32_t j = threadIdx.x; j < n; j += BLOCK) {
            uint32_t k;
            bool q;
            const uint32_t bits = __float_as_uint(src[j]);
            const uint32_t o = one(j, bits, k, q);
            if (FUSED) {
                dst[j] = __uint_as_float(o);
                if (mdst) mdst[j] = (uint8_t)k;
            }
            if (q) {
                const uint32_t pos = atomicAdd(sub_counter(cnt, CNT_CAND, sb), 1u);
                if (pos < cap_sb) {
                    my_cand[pos] = make_uint2(bits, g0 + j);
                    if (HIST) lds_count(s_h, ((bits & 0x7fffffffu) - lo) >> sh, true);
                }
            }
        }
    } else {
        // the tensor's last, ragged tile: the same as a full one, as far as there are weights
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t j = (threadIdx.x + BLOCK * u) * 4u, here = j < n ? min(n - j, 4u) : 0u;
            v[u] = make_uint4(0, 0, 0, 0);
            if (BLOCK * 4u * u >= n) continue;           // the same in every thread
            if (here == 4u) {
                v[u] = load_u4<NT>(src + j);
            } else {
                if (here > 0u) v[u].x = __float_as_uint(src[j]);
                if (here > 1u) v[u].y = __float_as_uint(src[j + 1u]);
                if (here > 2u) v[u].z = __float_as_uint(src[j + 2u]);
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t j = (threadIdx.x + BLOCK * u) * 4u, here = j < n ? min(n - j, 4u) : 0u;
            const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            uint32_t o[4] = {0, 0, 0, 0}, k[4] = {0, 0, 0, 0};
            if (BLOCK * 4u * u >= n) continue;
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                if (q < here) {
                    bool is_cand;
                    o[q] = one(j + q, x[q], k[q], is_cand);
                    cmask |= (is_cand ? 1u : 0u) << (4u * u + q);
                }
            }
            if (FUSED) {
                if (here == 4u) {
                    store_u4<NT>(dst + j, make_uint4(o[0], o[1], o[2], o[3]));
                    if (mdst) store_mask4<NT>(mdst + j, k[0] | (k[1] << 8) | (k[2] << 16) | (k[3] << 24));
                } else {
#pragma unroll
                    for (uint32_t q = 0; q < 3u; ++q) {
                        if (q < here) {
                            dst[j + q] = __uint_as_float(o[q]);
                            if (mdst) mdst[j + q] = (uint8_t)k[q];
                        }
                    }
                }
            }
        }
    }
    if (n > PASS_SINGLES) {
        // append the block's candidates with one global atomic: scan the per-thread
        // counts over the block, reserve a range in this block's sub-buffer, scatter
        const uint32_t c = __popc(cmask);
        uint32_t incl = c;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        if (lane == 63) s_wtot[wid] = incl;
        __syncthreads();
        uint32_t woff = 0, btot = 0;
#pragma unroll
        for (uint32_t i = 0; i < BLOCK / 64; ++i) {
            const uint32_t x = s_wtot[i];
            if (i < wid) woff += x;
            btot += x;
        }
        if (btot) {   // uniform over the block
            if (threadIdx.x == 0) s_base = atomicAdd(sub_counter(cnt, CNT_CAND, sb), btot);
            __syncthreads();
            uint32_t pos = s_base + woff + incl - c;
            if (cmask) {
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) {
                    const uint32_t j = (threadIdx.x + BLOCK * u) * 4;
                    const uint32_t vv[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        if (cmask & (1u << (4 * u + q))) {
                            if (pos < cap_sb) {
                                my_cand[pos] = make_uint2(vv[q], g0 + j + q);
                                if (HIST) lds_count(s_h, ((vv[q] & 0x7fffffffu) - lo) >> sh, true);
                            }
                            ++pos;
                        }
                    }
                }
            }
        }
    }
    for (uint32_t d = 32; d > 0; d >>= 1) {
        below += __shfl_down(below, d, 64);
        nan |= __shfl_down(nan, d, 64);
    }
    if (lane == 0) {
        if (below) atomicAdd(&s_below, below);
        if (nan) s_nan = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_below) atomicAdd(sub_counter(cnt, CNT_BELOW, sb), s_below);
        if (s_nan) atomicOr(&ss->status, 2u);
    }
    if (HIST) {
        const uint32_t c = s_h[threadIdx.x];
        if (c) atomicAdd(&hist[(blockIdx.x % FHIST_COPIES) * FBINS1 + threadIdx.x], c);
    }
    if (FUSED) {
        const uint32_t row_first = e0 / T.row_len;
        for (uint32_t s = threadIdx.x; s < nrows; s += BLOCK) {
            if (rowf[s]) {
                uint8_t* f = out_alive + T.out_flag_off + row_first + s;
                if (*f == 0) *f = 1;
            }
        }
        const uint32_t b = (e0 / T.khw) % T.in_ch;
        for (uint32_t s = threadIdx.x; s < ncols; s += BLOCK) {
            if (colf[s]) {
                uint8_t* f = in_alive + T.in_flag_off + mod_small(b + s, T.in_ch, T.magic_in);
                if (*f == 0) *f = 1;
            }
        }
    }
}

// Visits every candidate pair.  The grid is a multiple of SPEC_SUB blocks: block b walks
// sub-buffer b % SPEC_SUB, taking every (gridDim / SPEC_SUB)-th chunk of BLOCK pairs.
// Every thread of the block calls f the same number of times; `valid` is false for the
// threads past the end of the last, ragged chunk.
template <typename F>
__device__ __forceinline__ void for_each_candidate(const uint32_t* cnt, const uint2* cand,
                                                   uint32_t cap_sb, F&& f) {
    const uint32_t sb = blockIdx.x % SPEC_SUB, part = blockIdx.x / SPEC_SUB;
    const uint32_t parts = gridDim.x / SPEC_SUB;
    const uint32_t n = min(cnt[(CNT_CAND * SPEC_SUB + sb) * 32u], cap_sb);
    const uint2* src = cand + (size_t)sb * cap_sb;
    // four chunks per step: the loads of a step are all in flight before the first is used
    // (a block holds few wavefronts, so one load per thread at a time leaves the walk
    // waiting on memory latency)
    constexpr uint32_t U = 4;
    for (uint32_t i0 = part * BLOCK; i0 < n; i0 += U * parts * BLOCK) {
        uint2 c[U];
        bool valid[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * parts * BLOCK + threadIdx.x;
            valid[u] = i < n;
            c[u] = valid[u] ? src[i] : make_uint2(0, 0);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) f(c[u], valid[u]);
    }
}

// Round 1: a 256-bin histogram of (key - lo) >> sh over the candidates.
__global__ __launch_bounds__(BLOCK) void spec_hist_kernel(const SpecState* __restrict__ ss,
                                                          const uint32_t* __restrict__ cnt,
                                                          const uint2* __restrict__ cand,
                                                          uint32_t cap_sb, uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[FBINS1];
    static_assert(FBINS1 == BLOCK, "one round-1 bin per thread");
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lo = ss->lo, sh = ss->sh;
    for_each_candidate(cnt, cand, cap_sb, [&](uint2 c, bool valid) {
        lds_count(h, ((c.x & 0x7fffffffu) - lo) >> sh, valid);
    });
    __syncthreads();
    const uint32_t c = h[threadIdx.x];
    if (c) atomicAdd(&hist[(blockIdx.x % FHIST_COPIES) * FBINS1 + threadIdx.x], c);
}

// The rest of the finish in one launch.  Every block first locates the P-th pair from the same
// counters and histogram and gets the same answer: totals of the split counters, the check that
// makes the result exact, the round-1 bin.  Then it moves its share of the bin's candidates to the
// list (staged in LDS, one reservation), and the block that ends last ranks the list: a
// round-2 histogram, an exact rank by counting among the pairs of the selected bin, the record.
// Whatever the outcome, the state (status, counts, the record) is left in its mirror in pinned
// host memory as the last thing: the host reads it after waiting for the stream, with no copy
// on the stream.
// What bounds it is the chain of latencies, so the counters, the histogram and the first
// candidates are all loaded before the first of them is used, and the ranking costs no launch of
// its own (filter + rank of one count of 77 M weights 10.0 + 6.0 us, 13.7 as one).  With 64 blocks of 1024 threads, not 256
// of 256: 322 M weights 20.0 -> 13.1, 37 M 14.3 -> 11.8, 24 k 13.3 -> 12.4.
__global__ __launch_bounds__(FIN_THREADS) void spec_finish_kernel(
    SpecState* ss, const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ hist,
    const uint2* __restrict__ cand, uint32_t cap_sb, uint32_t n_sub, uint2* list, shifter_threshold* thr,
    SpecState* host_mirror) {
    constexpr uint32_t STAGE = 2048, WAVES = BLOCK / 64;       // of the wavefronts that add up the counters
    __shared__ uint2 stage[STAGE * FIN_SUBS];
    __shared__ uint32_t h[FBINS];
    __shared__ uint64_t comp[SPEC_SMALL_CAP];
    __shared__ uint64_t smem[FIN_THREADS / 64 + 1];
    __shared__ uint64_t s_sel, s_less2, s_r3;
    __shared__ uint32_t s_below[WAVES], s_inside[WAVES], s_hist[WAVES], s_over[WAVES];
    __shared__ uint32_t s_n, s_base, s_bin, s_cnt1, s_last, s_status, s_sub[FIN_SUBS];
    __shared__ uint64_t s_r2, s_less;
    __shared__ uint32_t s_lt, s_eq, s_bin2, s_cnt2, s_nb;
    __shared__ TiedLds s_tied;
    static_assert(SPEC_SMALL_CAP <= FIN_THREADS, "a thread for each");
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    static_assert(SPEC_SUB == BLOCK && FBINS1 == BLOCK, "one split counter and one round-1 bin per thread");
    // the first candidates of the block's sub-buffers, on their way while the P-th pair is located (a sub-buffer has
    // room for more than these, whatever it holds)
    uint2 ahead0[FIN_SUBS], ahead1[FIN_SUBS];
    uint32_t n_of[FIN_SUBS];
#pragma unroll
    for (uint32_t i = 0; i < FIN_SUBS; ++i) {
        const uint32_t sub = min(blockIdx.x + i * gridDim.x, n_sub - 1u);
        n_of[i] = min(cnt[(CNT_CAND * SPEC_SUB + sub) * 32u], cap_sb);
        ahead0[i] = cand[(size_t)sub * cap_sb + threadIdx.x];
        ahead1[i] = cand[(size_t)sub * cap_sb + FIN_THREADS + threadIdx.x];
    }
    const bool counts = threadIdx.x < BLOCK;
    uint32_t n_cand = 0, n_less = 0, in_bin = 0;
    if (counts) {
        n_cand = cnt[(CNT_CAND * SPEC_SUB + threadIdx.x) * 32u];
        n_less = cnt[(CNT_BELOW * SPEC_SUB + threadIdx.x) * 32u];
#pragma unroll
        for (uint32_t i = 0; i < FHIST_COPIES; ++i) in_bin += hist[i * FBINS1 + threadIdx.x];
    }
    const uint64_t p = ss->p;
    const uint32_t lo = ss->lo, sh = ss->sh;
    shifter_threshold out;                 // nothing removed
    out.reserved = 0; out.n_prune = p;
    out.cut = 0; out.t_key = 0; out.g_cut = ~0ull; out.n_less = 0; out.n_equal = 0;
    if (p == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            *thr = out;
            ss->rec = out;
            *host_mirror = *ss;
        }
        return;
    }
    if (threadIdx.x < FIN_SUBS) s_sub[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        s_n = 0; s_bin = 0xffffffffu;
        s_lt = 0; s_eq = 0; s_sel = 0; s_nb = 0; s_cnt2 = 0; s_bin2 = 0;
    }
    uint32_t sum_c = n_cand, sum_b = n_less, incl = in_bin;    // N < 2^32: the sums fit 32 bits
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, 64), yc = __shfl_up(sum_c, d, 64), yb = __shfl_up(sum_b, d, 64);
        if (lane >= d) { incl += y; sum_c += yc; sum_b += yb; }
    }
    const bool over = __ballot(n_cand > cap_sb) != 0ull;
    if (lane == 63 && counts) { s_below[wid] = sum_b; s_inside[wid] = sum_c; s_hist[wid] = incl; s_over[wid] = over; }
    __syncthreads();
    uint64_t below = 0, inside = 0, base = incl - in_bin;
    bool any_over = false;
#pragma unroll
    for (uint32_t i = 0; i < WAVES; ++i) {
        below += s_below[i];
        inside += s_inside[i];
        if (i < wid) base += s_hist[i];
        any_over = any_over || s_over[i] != 0;
    }
    const bool reached = !any_over && below < p && p <= below + inside;
    if (reached && counts) {
        const uint64_t r = p - below;
        if (base < r && r <= base + in_bin) {
            s_bin = threadIdx.x;
            s_cnt1 = in_bin;
            s_r2 = r - base;
            s_less = below + base;
        }
    }
    __syncthreads();
    const uint32_t bin = s_bin;
    // Undecided: the host redoes the ranking and every step behind it.  What is enqueued
    // behind this kernel still runs once on the record it finds, so leave a harmless one
    // (nothing removed) rather than the record of some earlier call.  By one block's first thread.
    auto publish = [&](bool decided) {
        ss->n_below = below;
        ss->n_inside = inside;
        if (bin != 0xffffffffu) { ss->bin = bin; ss->bin_cnt = s_cnt1; ss->r2 = s_r2; ss->less = s_less; }
        if (decided) ss->rec = out;
        *thr = out;
        const uint32_t undecided = decided ? 0u : 1u;
        const uint32_t status = atomicOr(&ss->status, undecided) | undecided;
        *host_mirror = *ss;               // no copy of it in between, which would be scratch memory
        host_mirror->status = status;
    };
    if (!reached || bin == 0xffffffffu || s_cnt1 > SPEC_LIST_CAP) {      // the same in every block
        if (blockIdx.x == 0 && threadIdx.x == 0) publish(false);
        return;
    }
    {
        auto take = [&](uint2 c, uint32_t i) {
            if ((((c.x & 0x7fffffffu) - lo) >> sh) == bin) {
                const uint32_t pos = atomicAdd(&s_n, 1u);
                atomicAdd(&s_sub[i], 1u);
                if (pos < STAGE * FIN_SUBS) stage[pos] = c;
            }
        };
#pragma unroll
        for (uint32_t i = 0; i < FIN_SUBS; ++i) {
            const uint32_t sub = blockIdx.x + i * gridDim.x;
            if (sub < n_sub) {
                if (threadIdx.x < n_of[i]) take(ahead0[i], i);
                if (FIN_THREADS + threadIdx.x < n_of[i]) take(ahead1[i], i);
                for (uint32_t j = FIN_AHEAD * FIN_THREADS + threadIdx.x; j < n_of[i]; j += FIN_THREADS)
                    take(cand[(size_t)sub * cap_sb + j], i);
            }
        }
        __syncthreads();
        const uint32_t n = s_n;
        bool over = false;
#pragma unroll
        for (uint32_t i = 0; i < FIN_SUBS; ++i) over = over || s_sub[i] > STAGE;
        if (over) {              // far more ties than the stage holds: leave it to the multi-pass select
            if (threadIdx.x == 0) atomicOr(&ss->status, 1u);
        } else if (n != 0) {
            if (threadIdx.x == 0) s_base = atomicAdd(&ss->list_cnt, n);
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < n; i += FIN_THREADS)
                if (s_base + i < SPEC_LIST_CAP) store_device(&list[s_base + i], stage[i]);
        }
    }
    // the list is complete when the last ticket is drawn
    if (!last_block(&ss->ticket, gridDim.x, &s_last)) return;
    if (threadIdx.x == 0) {
        s_n = atomicAdd(&ss->list_cnt, 0u);
        s_status = atomicOr(&ss->status, 0u);
    }
    for (uint32_t i = threadIdx.x; i < FBINS; i += FIN_THREADS) h[i] = 0;
    __syncthreads();
    const uint32_t n = s_n;
    // the second cannot happen unless the buffers were disturbed
    if ((s_status & 1u) || n != s_cnt1) {
        if (threadIdx.x == 0) publish(false);
        return;
    }
    // a list that fits stays in LDS
    const bool staged = n <= STAGE * FIN_SUBS;
    if (staged) {
        for (uint32_t i = threadIdx.x; i < n; i += FIN_THREADS) stage[i] = load_device(&list[i]);
        __syncthreads();
    }
    auto walk = [&](auto&& f) {
        for (uint32_t i = threadIdx.x; i < n; i += FIN_THREADS) f(staged ? stage[i] : load_device(&list[i]));
    };
    // round 2: the list's keys span 2^sh values starting at lo + (bin << sh)
    const uint32_t sh2 = sh > 12 ? sh - 12 : 0;   // 2^sh keys over FBINS = 2^12 bins
    const uint32_t lo1 = lo + (bin << sh);
    walk([&](uint2 c) { lds_count(h, ((c.x & 0x7fffffffu) - lo1) >> sh2, true); });
    __syncthreads();
    constexpr uint32_t PER = FBINS / FIN_THREADS;
    const uint32_t b0 = threadIdx.x * PER;
    uint64_t sum = 0, tot;
    for (uint32_t i = 0; i < PER; ++i) sum += h[b0 + i];
    base = block_excl_scan_u64<FIN_THREADS>(sum, smem, &tot);
    const uint64_t r = s_r2;
    if (base < r && r <= base + sum) {
        for (uint32_t i = 0; i < PER; ++i) {
            const uint32_t c = h[b0 + i];
            if (r <= base + c) {
                s_bin2 = b0 + i;
                s_cnt2 = c;
                s_r3 = r - base;
                s_less2 = base;
                break;
            }
            base += c;
        }
    }
    __syncthreads();
    const uint32_t bin2 = s_bin2, cnt2 = s_cnt2;
    if (cnt2 == 0 || cnt2 > SPEC_SMALL_CAP) {
        if (threadIdx.x == 0) publish(false);
        return;
    }
    walk([&](uint2 c) {
        const uint32_t key = c.x & 0x7fffffffu;
        if (((key - lo1) >> sh2) == bin2) {
            const uint32_t pos = atomicAdd(&s_nb, 1u);
            comp[pos] = ((uint64_t)key << 32) | c.y;   // pos < cnt2 <= SPEC_SMALL_CAP
        }
    });
    __syncthreads();
    uint32_t want = (uint32_t)s_r3 - 1u;         // 0-based rank inside the bin
    auto count = [&](const uint64_t* among, uint32_t n_among) {
        for (uint32_t i = threadIdx.x; i < n_among; i += FIN_THREADS) {
            const uint64_t c = among[i];
            uint32_t rank = 0;
            for (uint32_t f = 0; f < n_among; ++f) rank += among[f] < c;
            if (rank == want) s_sel = c;        // composites are distinct: exactly one hit
        }
    };
    if (cnt2 > TIED_DIRECT && sh2 == 0) {
        uint64_t* few = reinterpret_cast<uint64_t*>(stage);      // the list has been read
        const uint2 left = tied_stretch<FIN_THREADS, FBINS>(comp, cnt2, want, h, smem, few, &s_tied);
        want = left.y;
        count(few, left.x);
    } else {
        count(comp, cnt2);
    }
    __syncthreads();
    const uint64_t sel = s_sel;
    const uint32_t key = (uint32_t)(sel >> 32);
    uint32_t lt = 0, eq = 0;
    for (uint32_t i = threadIdx.x; i < cnt2; i += FIN_THREADS) {
        const uint32_t k = (uint32_t)(comp[i] >> 32);
        lt += k < key;
        eq += k == key;
    }
    if (lt) atomicAdd(&s_lt, lt);
    if (eq) atomicAdd(&s_eq, eq);
    __syncthreads();
    if (threadIdx.x == 0) {
        out.t_key = key;
        out.g_cut = sel & 0xffffffffull;
        out.cut = sel + 1;
        out.n_less = s_less + s_less2 + s_lt;
        out.n_equal = s_eq;
        publish(true);
    }
}

// Fused form only: settle the candidates.  The pass wrote those below mid as removed and
// the others as kept without flags; with the exact cut known, the few on the wrong side
// are rewritten and every kept non-zero candidate marks its filter and input feature.
__global__ __launch_bounds__(BLOCK) void spec_fixup_kernel(
    const DevTensor* __restrict__ tens, const uint32_t* __restrict__ ranked_ids,
    uint32_t n_ranked, const SpecState* __restrict__ ss, const uint32_t* __restrict__ cnt,
    const uint2* __restrict__ cand, uint32_t cap_sb, const shifter_threshold* __restrict__ thr,
    float* __restrict__ w_out, uint8_t* __restrict__ mask, uint8_t* out_alive,
    uint8_t* in_alive) {
    constexpr uint32_t LDS_T = 1024;
    __shared__ uint32_t s_gbase[LDS_T];
    if (ss->p == 0 || (ss->status & 1u)) return;
    const uint64_t cut = thr->cut;
    const uint32_t mid = ss->mid;
    const bool in_lds = n_ranked <= LDS_T;
    if (in_lds)
        for (uint32_t i = threadIdx.x; i < n_ranked; i += BLOCK)
            s_gbase[i] = (uint32_t)tens[ranked_ids[i]].gbase;
    __syncthreads();
    for_each_candidate(cnt, cand, cap_sb, [&](uint2 c, bool valid) {
        if (!valid) return;
        const uint32_t key = c.x & 0x7fffffffu;
        const bool removed = (((uint64_t)key << 32) | c.y) < cut;
        const bool written_removed = key < mid;
        if (removed == written_removed && (removed || key == 0)) return;   // nothing to do
        // tensor holding global index c.y: last ranked tensor with gbase <= g
        uint32_t a = 0, b = n_ranked;
        while (b - a > 1) {
            const uint32_t m2 = (a + b) >> 1;
            const uint32_t gb = in_lds ? s_gbase[m2] : (uint32_t)tens[ranked_ids[m2]].gbase;
            if (gb <= c.y) a = m2; else b = m2;
        }
        const DevTensor& T = tens[ranked_ids[a]];
        const uint32_t e = c.y - (uint32_t)T.gbase;
        if (removed != written_removed) {
            w_out[T.offset + e] = removed ? 0.0f : __uint_as_float(c.x);
            if (mask) mask[c.y] = removed ? 0 : 1;
        }
        if (!removed && key != 0) {
            uint8_t* f = out_alive + T.out_flag_off + e / T.row_len;
            if (*f == 0) *f = 1;
            f = in_alive + T.in_flag_off + (e / T.khw) % T.in_ch;
            if (*f == 0) *f = 1;
        }
    });
}

void launch_spec_select(shifter_ctx* ctx, const shifter_model* m, const float* d_w, uint64_t p,
                        shifter_threshold* d_thr, float* d_w_out, uint8_t* d_mask,
                        uint8_t* d_out_alive, uint8_t* d_in_alive, SpecState* host_mirror) {
    const auto& b = m->b;
    const uint32_t n_t = (uint32_t)m->t.size();
    const bool fused = d_w_out != nullptr;
    // few tiles: their candidates' histogram costs the pass less than the launch behind it
    const bool small = m->n_tiles <= PASS_HIST_TILES;
    hipStream_t s = ctx->stream;
    {
        ProfileScope ps(ctx, K_SPEC_SAMPLE);
        spec_front_kernel<<<sample_grid(m), SAMPLE_THREADS, 0, s>>>(
            sample_in(m, d_w), b.spec, b.spec_cnt, b.partial, d_out_alive, fused ? m->info.sum_out_ch : 0, d_in_alive,
            fused ? m->info.sum_in_ch : 0, p, m->sample_size, m->info.n_prunable, ctx->margin_sigmas);
    }
    {
        ProfileScope ps(ctx, K_SPEC_PASS);
        const bool nt = m->info.w_extent * 4 > (192ull << 20);   // beyond the last-level cache
        auto k = small ? (fused ? spec_pass_kernel<true, false, true> : spec_pass_kernel<false, false, true>)
                 : fused ? (nt ? spec_pass_kernel<true, true, false> : spec_pass_kernel<true, false, false>)
                         : (nt ? spec_pass_kernel<false, true, false> : spec_pass_kernel<false, false, false>);
        k<<<m->n_tiles, BLOCK, 0, s>>>(b.tens, b.tile_prefix, n_t, d_w, b.spec, b.spec_cnt, b.cand,
                                       b.cand_cap_sb, b.partial, d_w_out, d_mask, d_out_alive, d_in_alive);
    }
    if (!small) {
        ProfileScope ps(ctx, K_SPEC_FINISH);
        spec_hist_kernel<<<FIN_BLOCKS, BLOCK, 0, s>>>(b.spec, b.spec_cnt, b.cand, b.cand_cap_sb,
                                                      b.partial);
    }
    {
        ProfileScope ps(ctx, K_SPEC_FINISH2);
        const uint32_t n_sub = std::min(SPEC_SUB, std::max(1u, m->n_tiles));      // sub-buffers that can hold anything
        spec_finish_kernel<<<std::min(n_sub, SPEC_SUB / FIN_SUBS), FIN_THREADS, 0, s>>>(b.spec, b.spec_cnt, b.partial, b.cand, b.cand_cap_sb, n_sub, b.list,
                                                        d_thr, host_mirror);
    }
    if (fused) {
        ProfileScope ps(ctx, K_SPEC_FIXUP);
        spec_fixup_kernel<<<SPEC_SUB * 4, BLOCK, 0, s>>>(
            b.tens, b.ranked_ids, m->n_ranked, b.spec, b.spec_cnt, b.cand, b.cand_cap_sb, d_thr,
            d_w_out, d_mask, d_out_alive, d_in_alive);
    }
}

}  // namespace shifter
