// Portfolio codec (Sec. III-E, Modules 7 and 8): inactive models are kept as DEFLATE
// streams (RFC 1951) and inflated when they are to run.  The encoder is built for
// chunk-parallel work on both sides:
//   - chunks of 32768 bytes, each its own byte-aligned segment of the stream; inside a
//     chunk 64 sub-chunks of 512 bytes, one lane each;
//   - tokens: literals, and for a run of r >= 4 equal bytes inside a sub-chunk one literal
//     followed by distance-1 matches over the other r - 1 bytes (258 while more than 260
//     remain, then one piece, or (rest - 3, 3) when 259 or 260 remain);
//   - a sub-chunk whose tokens would take more than 8 * bytes + 48 bits is stored: a stored
//     block of its own; the others are coded with the fixed Huffman codes;
//   - a segment walks its sub-chunks: a coded one opens a fixed-Huffman block unless one is
//     open and appends its tokens, a stored one closes the open block and is a stored
//     block; at the end the open block is closed and an empty stored block pads to a byte
//     (and carries BFINAL in the last segment).  If that is not shorter than one stored
//     block with the whole chunk, the segment is that block;
//   - side information for the decoder: the byte offset of every segment, and per
//     sub-chunk its token bits, or 0xFFFF if stored (all 0: whole chunk in one block).
//   - a mark per coded sub-chunk, so that four lanes share it: for each of its later three
//     quarters of 128 bytes, the token bits of the quarter before (11 bits) and how far past
//     the quarter's start its first literal lies (9 bits); a run's matches go with the
//     literal that starts the run, so a lane never needs another lane's bytes.
// Any inflater reads the stream; the encoder works with 512 threads per chunk and 32 lanes per
// sub-chunk, the decoder with 256 and four.
#include <string>
#include <type_traits>

#include "chain.h"
#include "dev_common.h"

namespace shifter {

constexpr uint32_t CODEC_CHUNK = SHIFTER_CODEC_CHUNK;
constexpr uint32_t CODEC_SUB = SHIFTER_CODEC_SUB;
constexpr uint32_t CODEC_NSUB = CODEC_CHUNK / CODEC_SUB;      // 64: one wave
constexpr uint32_t CODEC_SUBW = CODEC_SUB / 4;                // dwords per sub-chunk
constexpr uint32_t CODEC_SLOT = CODEC_CHUNK + 8;              // bytes of a chunk's slot in the workspace
constexpr uint32_t CODEC_MARGIN = 48;                         // bits a stored sub-chunk must save
constexpr uint32_t CODEC_STORED = 0xFFFFu;                    // side information of a stored sub-chunk
static_assert(CODEC_NSUB == 64, "one lane per sub-chunk");

// Sub-chunk l, dword j of the chunk staged in LDS: every row is rotated by l 16-byte
// vectors, so that the lanes of a wave, each walking its own sub-chunk at the same pace,
// spread over the banks while a vector stays whole.
__device__ __forceinline__ uint32_t sub_word(uint32_t l, uint32_t j) {
    return l * CODEC_SUBW + ((j + 4u * l) & (CODEC_SUBW - 1));
}

// Appends bits to the chunk's bit buffer in LDS, which starts zeroed: every dword is OR-ed
// in, so neighbouring lanes may share the dwords at the ends of their ranges.  At most 32
// bits per call.
struct BitWriter {
    uint32_t* buf;
    uint64_t acc;
    uint32_t cnt, widx;
    __device__ __forceinline__ BitWriter(uint32_t* b, uint32_t start_bit)
        : buf(b), acc(0), cnt(start_bit & 31u), widx(start_bit >> 5) {}
    __device__ __forceinline__ void put(uint32_t code, uint32_t n) {
        acc |= (uint64_t)code << cnt;
        cnt += n;
        if (cnt >= 32u) {
            atomicOr(&buf[widx], (uint32_t)acc);
            ++widx;
            acc >>= 32;
            cnt -= 32u;
        }
    }
    __device__ __forceinline__ void finish() {
        if (cnt) atomicOr(&buf[widx], (uint32_t)acc);
    }
};

__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t lane, uint32_t* total) {
    uint32_t x = v;
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    *total = __shfl(x, 63, 64);
    return x - v;
}

// Where every sub-chunk's part of a segment starts, one lane per sub-chunk: v its side
// information (token bits, or CODEC_STORED; 0 where nothing is left of the chunk), n its
// bytes.  start: bit position of the first bit this lane's sub-chunk is responsible for (a
// coded one: the block header if it opens a block, then its tokens; a stored one: the
// end-of-block of the block it closes, then its own header); in_block: whether a Huffman
// block is open at that point.  tail_*: the same for what follows the last sub-chunk.
// Returns the segment's size in bytes.
// A stored sub-chunk ends on a byte, so a run of coded ones always starts on one: two prefix
// sums, of the token bits and of the bytes up to the end of each stored sub-chunk, place
// all of them at once (a walk over the 64 sub-chunks, which any stored one needed before,
// took about 4 us of a chunk's life).  Without a stored one the first sum does (with
// both, 12288 chunks of half-full weights inflated in 805 us, with the first alone in 792, as with the walk; 39347
// sparse ones deflated in 1198 and 1172).
__device__ __forceinline__ uint32_t place_subs(uint32_t v, uint32_t n, uint32_t lane, uint32_t* start,
                                               bool* in_block, uint32_t* tail_start, bool* tail_in_block) {
    const bool stored = n != 0u && v == CODEC_STORED;
    uint32_t bits_total;
    const uint32_t bits = wave_excl_scan(n != 0u && !stored ? v : 0u, lane, &bits_total);   // coded bits before this lane
    const uint64_t st = __ballot(stored);
    const uint64_t before = st & ((1ull << lane) - 1ull);
    uint32_t run = bits, tail_run = bits_total;         // coded bits since the last stored sub-chunk (or the start)
    uint32_t byte0 = 0, bytes_total = 0;
    if (st == 0ull) {                                   // most chunks: one Huffman block
        *start = run ? 3u + run : 0u;
    } else {
        const uint32_t at_stored = __shfl(bits, before ? 63 - __clzll((long long)before) : 0, 64);
        run = bits - (before ? at_stored : 0u);
        const uint32_t head = run ? 3u + run : 0u;                    // with the block's header
        const uint32_t bytes = stored ? ((head + (run ? 7u : 0u) + 3u + 7u) >> 3) + 4u + n : 0u;
        byte0 = wave_excl_scan(bytes, lane, &bytes_total);
        *start = 8u * byte0 + head;
        tail_run = bits_total - __shfl(bits, 63 - __clzll((long long)st), 64);
    }
    *in_block = run != 0u;
    const uint32_t pos = 8u * bytes_total + (tail_run ? 3u + tail_run : 0u);
    *tail_start = pos;
    *tail_in_block = tail_run != 0u;
    return ((pos + (tail_run ? 7u : 0u) + 3u + 7u) >> 3) + 4u;
}

constexpr uint32_t CODEC_Q = 4;                               // lanes per sub-chunk
constexpr uint32_t CODEC_QB = CODEC_SUB / CODEC_Q;            // 128 bytes of a sub-chunk per lane
constexpr uint32_t CODEC_THREADS = CODEC_NSUB * CODEC_Q;      // 256: one block per chunk
constexpr uint32_t CODEC_LOOP_GRID = 1536;                    // blocks of an instance that walks a list

// --- the encoder -------------------------------------------------------------------------
// 512 threads per chunk, one or two chunks a block.  A lane holds 16 consecutive bytes of a sub-chunk (32
// lanes a sub-chunk, so a wavefront takes 1 KiB at a time and four of those in turn); the
// chunk stays in registers and only the segment being built is in LDS: 37 KB with the codes, whatever its
// size, room for four chunks a compute unit.  (The bound on registers asks for fewer; the 58 that the
// compiler takes let four run.)  First every piece finds its literals,
// the runs they start and its token bits, and prefix sums over the lanes place the pieces in
// their sub-chunk; then, with the sub-chunks placed in the segment, every lane appends its
// own piece's tokens.
// Bound by vector instructions for two thirds of its time (counters: 27 M of 41 M issue slots with 474 of them per
// KiB and wavefront; fewer now), the rest is the latency of the ticket, of the chunk's bytes and
// of the chain, and in small inputs the life of one block.  So the codes come from tables in LDS (literals, short
// matches, long ones: the arithmetic took a third of the instructions), lanes exchange by DPP, a match is appended once
// for four bytes and not for two, the marks are put together by one wavefront for all sub-chunks, and a full
// chunk takes no care of its end.
// Ten rebuilt variants of a 14.7 M weight network (3/10 to all of the
// weights not zero), one after the other: 2780 us with four lanes walking a sub-chunk's tokens
// one by one, a second instance for the chunks with long segments and a pack pass; 845 with 256
// threads of this form, 690 with 512, 650 without loops for the matches and with two chunks a
// block, 570 with the tables and what goes with them (the kernels alone 492 -> 409).  1.3 GB of a model with
// 5 % of its weights: 4820 us, 1097, 838 now; with 30 % 1196 -> 906; all of its weights 713 -> 708; all zeros 409 -> 414 (64 to
// 256 MB of zeros 43 -> 46, 61 -> 64, 100 -> 105: the one input that the tables' form is slower for).

// Bits 0-15 of a piece: which bytes differ from the byte before them, and which are >= 144
// (9-bit literals).  prev: the byte before the piece.
__device__ __forceinline__ uint32_t nibbles(const uint32_t (&t)[4]) {   // bit 7 of the bytes of t -> 16 bits
    const uint32_t a = __builtin_amdgcn_udot4(t[1], 0x80402010u, __builtin_amdgcn_udot4(t[0], 0x08040201u, 0u, false), false);
    const uint32_t b = __builtin_amdgcn_udot4(t[3], 0x80402010u, __builtin_amdgcn_udot4(t[2], 0x08040201u, 0u, false), false);
    return (a >> 7) | (b >> 7 << 8);
}
__device__ __forceinline__ uint32_t not_low144(uint32_t w) {            // bit 7 of every byte >= 0x90
    return w & ((w & 0x70707070u) + 0x70707070u) & 0x80808080u;
}
__device__ __forceinline__ uint32_t changes16(const uint4& v, uint32_t prev) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t ne[4];
#pragma unroll
    for (uint32_t d = 0; d < 4u; ++d) {
        const uint32_t x = w[d] ^ ((w[d] << 8) | (d ? w[d - 1u] >> 24 : prev));
        ne[d] = (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
    }
    return nibbles(ne);
}
__device__ __forceinline__ uint32_t nines16(const uint4& v) {
    const uint32_t ge[4] = {not_low144(v.x), not_low144(v.y), not_low144(v.z), not_low144(v.w)};
    return nibbles(ge);
}

// What a lane keeps of a piece between the two passes.
struct Piece {
    uint4 v;          // the bytes
    uint32_t lit;     // the bytes sent as literals
    uint32_t place;   // bits 0-15 token bits of the sub-chunk before this piece; 16-25 the first
                      //   literal behind the piece (offset in the sub-chunk; its length if none)
    uint32_t runs;    // bits 0-15 Runs::near, 16-24 Runs::far
};

// The runs of 4 or more that start in a piece.  lit: its literals; end: the sub-chunk's end, where
// that lies inside the piece; next: the first literal behind it, relative to its start.
struct Runs {
    uint32_t ends;    // where a run in the piece can end: literals, the end, and `next` if below 32
    uint32_t near;    // literals that start a run whose other 3 to 14 bytes one match covers
    uint32_t far;     // the other bytes of a longer run, which only the last literal can start; or 0
};
__device__ __forceinline__ Runs find_runs(uint32_t lit, uint32_t end, uint32_t next) {
    Runs r;
    r.ends = lit | end | (next < 32u ? 1u << next : 0u);
    r.near = lit & ~(r.ends >> 1);                  // the next byte is neither a literal nor the end
    const uint32_t p = 31u - (uint32_t)__clz((int)(lit | 1u));
    const uint32_t rest = next - p - 1u;            // (the end inside the piece is `next` too)
    r.far = ((r.near >> p) & 1u) != 0u && rest >= 15u ? rest : 0u;
    if (r.far) r.near &= ~(1u << p);
    return r;
}

// Codes by table, in LDS: of the 256 literals, of the matches that cover 3 to 14 bytes, by that
// number, and of those that cover up to a sub-chunk.
struct alignas(16) CodeTable {
    uint32_t match[32];           // code | length << 16; others: 0
    uint32_t far[CODEC_SUB];      // by rest, from 15 on (Runs::far): the code
    uint16_t literal[256];        // code | length << 12
    uint8_t far_bits[CODEC_SUB];  // length of far's
};
constexpr uint32_t reversed(uint32_t x, uint32_t n) {
    uint32_t y = 0;
    for (uint32_t i = 0; i < n; ++i) y |= ((x >> i) & 1u) << (n - 1u - i);
    return y;
}
// A match of `len` (3..258) at distance 1: length code, extra bits, 5-bit distance code 0.
constexpr uint32_t match_code(uint32_t len, uint32_t* code) {
    uint32_t idx = 28u, e = 0, extra = 0;
    if (len < 11u) {
        idx = len - 3u;
    } else if (len != 258u) {
        const uint32_t x = len - 3u;              // 8..254
        while ((x >> (e + 3u)) != 0u) ++e;        // floor(log2 x) - 2
        idx = 4u * e + 4u + ((x >> e) & 3u);
        extra = x & ((1u << e) - 1u);
    }
    // symbols 257..279 in 7 bits, 280..285 in 8
    const uint32_t n = idx < 23u ? 7u : 8u;
    *code = reversed(idx < 23u ? 1u + idx : 0xC0u + (idx - 23u), n) | (extra << n);
    return n + e + 5u;
}
// The matches that cover the rest (15..511) bytes behind a run's first one: one of 258 where
// more than 260 remain, then one, or the pieces (rest - 3, 3) of 259 and 260.  At most 31 bits.
constexpr uint32_t far_matches(uint32_t rest, uint32_t* code) {
    uint32_t a = 0, b = 0;
    if (rest > 258u) {
        const uint32_t first = rest > 260u ? 258u : rest - 3u;
        const uint32_t na = match_code(first, &a), nb = match_code(rest - first, &b);
        *code = a | (b << na);
        return na + nb;
    }
    return match_code(rest, code);
}
constexpr CodeTable make_code_table() {
    CodeTable t{};
    for (uint32_t i = 0; i < 256u; ++i)           // 0x30 + i in 8 bits below 144, 0x190 + i - 144 in 9 from there on
        t.literal[i] = (uint16_t)(i < 144u ? reversed(0x30u + i, 8) | (8u << 12) : reversed(0x190u + i - 144u, 9) | (9u << 12));
    for (uint32_t i = 0; i < CODEC_SUB; ++i) {
        uint32_t c = 0;
        if (i >= 3u && i <= 14u) t.match[i] = match_code(i, &c) << 16 | c;
        if (i >= 15u) {
            t.far_bits[i] = (uint8_t)far_matches(i, &c);
            t.far[i] = c;
        }
    }
    return t;
}
static __device__ const CodeTable kCodeTable = make_code_table();
static_assert(sizeof(CodeTable) % 16 == 0 && sizeof(CodeTable) / 16 <= 512 - 64, "one piece a thread behind the first wavefront");

// Appends the tokens of a piece at bit position `bit` of the (zeroed) buffer.  ends, near, far: see Runs.
__device__ __forceinline__ void emit_tokens(const CodeTable& t, uint32_t* out, uint32_t bit, const uint4& v, uint32_t lit,
                                            uint32_t ends, uint32_t near, uint32_t far) {
    const uint32_t dw[4] = {v.x, v.y, v.z, v.w};
    auto append = [&](uint32_t bits, uint32_t n) {       // at most 32 bits
        const uint64_t code = (uint64_t)bits << (bit & 31u);
        atomicOr(&out[bit >> 5], (uint32_t)code);
        atomicOr(&out[(bit >> 5) + 1u], (uint32_t)(code >> 32));
        bit += n;
    };
#pragma unroll
    for (uint32_t d = 0; d < 4u; ++d) {
        if (__ballot((lit >> (4u * d)) & 15u) == 0ull) continue;
        uint32_t e[4];
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) e[q] = t.literal[(dw[d] >> (8u * q)) & 0xffu] & (0u - ((lit >> (4u * d + q)) & 1u));
        // two bytes: up to 18 bits
        const uint32_t n0 = e[0] >> 12, n2 = e[2] >> 12;
        append((e[0] & 0xfffu) | ((e[1] & 0xfffu) << n0), n0 + (e[1] >> 12));
        uint32_t c = (e[2] & 0xfffu) | ((e[3] & 0xfffu) << n2), n = n2 + (e[3] >> 12);
        // runs that start in a piece are at least four bytes apart: at most one starts among these four, the
        // rest of them belong to it, and its match comes behind their literals
        const uint32_t run = (near >> (4u * d)) & 15u;
        if (__ballot(run != 0u) != 0ull) {
            const uint32_t first = (uint32_t)__builtin_ctz(run | 16u);
            const uint32_t rest = (uint32_t)__builtin_ctz((ends >> (4u * d + 1u) >> first) | 0x80000000u);
            const uint32_t m = t.match[run ? rest : 0u];
            c |= (m & 0xffffu) << n;
            n += m >> 16;
        }
        append(c, n);
    }
    if (far) append(t.far[far], 0u);
}

// Lane exchanges without a trip through LDS: the value of the lane below and above in the wavefront (0
// at its ends), and the inclusive sum over 32 lanes.
__device__ __forceinline__ uint32_t lane_below(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xf, 0xf, true);       // wave_shr:1
}
__device__ __forceinline__ uint32_t lane_above(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xf, 0xf, true);       // wave_shl:1
}
__device__ __forceinline__ uint32_t incl_sum32(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);         // row_shr:1, 2, 4, 8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
    // lane 15 of a 32's first row to its second (row_bcast:15 into rows 1 and 3)
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);
}

// Chained offsets of the segments (the decoupled look-back of Merrill and Garland's single-pass
// scan; chain.h has its rules).  Their words belong to the context, two arrays that calls use in turn, all zero to begin with:
// the block with a call's last link clears the other one, so that no launch has to do it before
// (us a call: up to 64 chunks 25 -> 23.5, 640 46 -> 43, ten variants of a 14.7 M weight network 568 -> 539).  In the header: the ticket, whose
// bit 31 says which array is in use, and how many words of either are.  A recorded call has one array, in the caller's
// workspace, that a launch clears.
constexpr uint32_t CHAIN_HEADER = 32, CHAIN_TICKET = 0, CHAIN_USED = 16;
constexpr uint32_t CHAIN_SIDE = 1u << 31;
constexpr uint32_t CHAIN_POLLS = 1u << 22;     // seconds: far beyond any wait that ends
__device__ __forceinline__ void chain_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Sum of the sizes before link c, by one wavefront.  Links (a block's one chunk, or its two) are numbered by
// a ticket that the block draws when it starts, and a block stores its sizes before it waits for anything: every predecessor
// is running or done and its size arrives without it waiting for this block.
__device__ __forceinline__ ChainWalk chain_before(const uint64_t* status, uint32_t c, uint32_t lane) {
    ChainWalk walk(c);
    while (walk.waits()) {
        const int64_t i = walk.last - (int64_t)lane;
        const uint64_t x = i >= 0 ? __hip_atomic_load(status + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 2ull << 62;
        const uint32_t kind = (uint32_t)(x >> 62);
        const uint64_t need = walk.look(__ballot(kind == 2u), __ballot(kind != 0u), __ballot(kind == 3u), CHAIN_POLLS);
        if (need == 0ull) { __builtin_amdgcn_s_sleep(4); continue; }
        uint64_t part = (need >> lane) & 1ull ? x & CHAIN_VALUE : 0ull;
        for (uint32_t d = 32; d > 0; d >>= 1) part += __shfl_xor((unsigned long long)part, d, 64);
        walk.sum += part;
    }
    return walk;
}

// A whole sub-chunk of zeros: the literal 0 (00110000) and the matches 258 (symbol 285: 11000101)
// and 253 (symbol 284: 11000100, extra bits 253 - 227 = 26), each with the distance code 00000.
// All codes start from their first bit in bit 0.  Its quarters: all token bits before the
// second one, and no further literal before the end.
constexpr uint32_t ZERO_SUB_BITS = 8u + 13u + 18u;
constexpr uint32_t ZERO_SUB_LOW = 0x0Cu | (0xA3u << 8);                    // the literal and the first match, 21 bits
constexpr uint32_t ZERO_SUB_HIGH = 0x23u | (26u << 8);
static_assert(CODEC_SUB == 512u, "258 + 253 + 1");

// DIRECT: the segments go straight to their place in the stream, which cannot overflow (the
// host checked that it holds the largest possible one).  The tickets take 13.8 ns each on their one
// address, a bound where chunks hold next to nothing: 1.3 GB of zeros take 538 us a call with a ticket for
// each chunk, 414 with one for two (GROUPS: 512 threads each, side by side in a block; they are one link of the
// chain too: dense weights 889 and 708 us; 724 and zeros 421 where a barrier stood between the sizes and
// their sum).  Otherwise every segment goes to its
// slot of the workspace, and the two kernels behind this one add up the sizes and, if the
// stream is large enough, move the segments.
constexpr uint32_t CODEC_OUT_DW = CODEC_CHUNK / 4 + 8;
constexpr uint32_t DEF_THREADS = 512;
template <bool DIRECT, uint32_t GROUPS>
__global__ __launch_bounds__(DEF_THREADS * GROUPS, GROUPS == 1 ? 6 : 4) void deflate_kernel(
    const uint8_t* __restrict__ in, uint64_t n_bytes, uint32_t n_chunks, uint16_t* __restrict__ side,
    uint64_t* __restrict__ marks, uint8_t* __restrict__ slots, uint32_t* __restrict__ seg_size,
    uint64_t* chain, uint32_t chain_cap, uint64_t* __restrict__ seg_off,
    uint8_t* __restrict__ stream, uint64_t* __restrict__ mirror) {
    __shared__ __align__(16) uint32_t g_out[GROUPS][CODEC_OUT_DW];
    // of every sub-chunk's quarters the token bits before it (bits 0-15) and how far past its start its first
    // literal lies
    __shared__ __align__(16) uint32_t g_quarter[GROUPS][CODEC_NSUB * CODEC_Q];
    __shared__ uint32_t g_side[GROUPS][CODEC_NSUB];
    __shared__ CodeTable s_codes;
    __shared__ uint64_t g_off[GROUPS];
    __shared__ uint32_t s_c, s_sized, g_size[GROUPS];
    constexpr uint32_t STEPS = CODEC_CHUNK / 1024u / (DEF_THREADS / 64u);     // KiB per wavefront
    const uint32_t group = GROUPS == 1 ? 0u : uniform_u32(threadIdx.x / DEF_THREADS), tid = threadIdx.x % DEF_THREADS;
    uint32_t* s_out = g_out[group];
    uint32_t* s_quarter = g_quarter[group];
    uint32_t* s_side = g_side[group];
    const uint32_t lane = threadIdx.x & 63u, wid = uniform_u32(tid >> 6), half = lane >> 5, hl = lane & 31u;
    uint32_t link = blockIdx.x, c = link * GROUPS + group;
    if (DIRECT && threadIdx.x == 0) {
        s_c = atomicAdd(reinterpret_cast<uint32_t*>(chain + CHAIN_TICKET), 1u);
        s_sized = 0;
    }
    // while the first wavefront waits for the ticket
    if (threadIdx.x - 64u < sizeof(CodeTable) / 16u)
        reinterpret_cast<uint4*>(&s_codes)[threadIdx.x - 64u] = reinterpret_cast<const uint4*>(&kCodeTable)[threadIdx.x - 64u];
    __syncthreads();
    uint32_t side_now = 0;                              // which of the chain's two arrays is this call's
    if (DIRECT) {
        link = uniform_u32(s_c);
        side_now = link >> 31;
        link &= CHAIN_SIDE - 1u;
        c = link * GROUPS + group;
        if (link == 0u && threadIdx.x == 0) chain_store(mirror + CHAIN_BROKE, 0ull);
    }
    uint64_t* status = chain + CHAIN_HEADER + (uint64_t)side_now * chain_cap;
    const bool alive = c < n_chunks;                    // of the last block's groups maybe the first alone
    const uint64_t base = (uint64_t)c * CODEC_CHUNK;
    const uint32_t m = (uint32_t)min((uint64_t)CODEC_CHUNK, n_bytes - min(n_bytes, base));
    const uint32_t last = c + 1u == n_chunks ? 1u : 0u;
    const uint32_t p0 = hl * 16u;                       // this lane's pieces start here in their sub-chunks
    Piece P[STEPS];
    uint32_t zero_kib = 0;                              // bit i: piece i is part of 1 KiB of zeros
#pragma unroll
    for (uint32_t i = 0; i < STEPS; ++i) {
        const uint32_t at = (i * (DEF_THREADS / 64u) + wid) * 1024u + lane * 16u;
        P[i].v = make_uint4(0, 0, 0, 0);
        if (at + 16u <= m) {
            P[i].v = *reinterpret_cast<const uint4*>(in + base + at);
        } else if (at < m) {
            uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
            for (uint32_t k = 0; k < 16u; ++k)
                if (at + k < m) w[k >> 2] |= (uint32_t)in[base + at + k] << (8u * (k & 3u));
            P[i].v = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    for (uint32_t k = tid; k < CODEC_OUT_DW / 4u; k += DEF_THREADS)
        reinterpret_cast<uint4*>(s_out)[k] = make_uint4(0, 0, 0, 0);
    // --- first pass: literals, token bits, side information and the quarters.  FULL: a chunk of whole sub-chunks
    auto first_pass = [&](auto FULL) {
        constexpr bool full = decltype(FULL)::value;
#pragma unroll
        for (uint32_t i = 0; i < STEPS; ++i) {
            const uint32_t sub = (i * (DEF_THREADS / 64u) + wid) * 2u + half;
            const uint32_t n_l = full ? CODEC_SUB : min(CODEC_SUB, m - min(m, sub * CODEC_SUB));
            const uint4 v = P[i].v;
            if (full && __ballot((v.x | v.y | v.z | v.w) != 0u) == 0ull) {
                // 1 KiB of zeros (common in sparse models): both sub-chunks are one run
                if (hl == 0u) s_side[sub] = ZERO_SUB_BITS;
                if ((hl & 7u) == 0u) s_quarter[sub * CODEC_Q + (hl >> 3)] = ZERO_SUB_BITS | ((CODEC_SUB - p0) << 16);
                zero_kib |= 1u << i;
                continue;
            }
            uint32_t s = changes16(v, lane_below(v.w >> 24)), end = 0;   // end: the sub-chunk's end, where it lies inside the piece
            if (hl == 0u) s |= 1u;
            const uint32_t nine = nines16(v);
            uint32_t valid = 0xffffu;
            if (!full) {
                // the end counts as a change
                const uint32_t left = n_l > p0 ? n_l - p0 : 0u;
                if (n_l >= p0 && left < 16u) end = 1u << left;
                valid = left >= 16u ? 0xffffu : (1u << left) - 1u;
                s = (s & valid) | end;
            }
            const uint32_t below = lane_below(s), above = lane_above(s);
            // bits 2-17 the piece, two bits of the neighbours on either side
            const uint32_t S = (hl ? below >> 14 : 0u) | (s << 2) | ((hl == 31u ? 1u : above & 3u) << 18);
            const uint32_t Z = ~S & (hl ? ~0u : ~3u);
            const uint32_t lit = ((S >> 2) | ((Z >> 2) & (((S >> 1) & (S >> 3)) | ((S >> 1) & (Z >> 3) & (S >> 4)) |
                                                          ((Z >> 1) & S & (S >> 3))))) & valid;
            const uint64_t any = __ballot(lit != 0u);
            const uint32_t later = (uint32_t)(any >> (32u * half)) & (hl == 31u ? 0u : ~0u << (hl + 1u));
            const uint32_t first = lit ? p0 + (uint32_t)__ffs((int)lit) - 1u : 0u;
            const uint32_t behind = __shfl(first, later ? (int)(32u * half + (uint32_t)__ffs((int)later) - 1u) : 0, 64);
            const uint32_t next = later ? behind : n_l;     // first literal behind the piece
            uint32_t bits = 8u * (uint32_t)__popc(lit) + (uint32_t)__popc(lit & nine);
            const Runs run = find_runs(lit, end, next - p0);
            {
                // 12 bits a match, one more where none of the eleven bytes behind its literal ends the run
                uint32_t e = run.ends | (run.ends >> 1);
                e |= e >> 2;
                e |= e >> 4;
                e |= e >> 3;
                bits += 12u * (uint32_t)__popc(run.near) + (uint32_t)__popc(run.near & ~(e >> 1));
                bits += s_codes.far_bits[run.far];       // [0] is 0
            }
            const uint32_t incl = incl_sum32(bits), before = incl - bits;
            if (hl == 31u) s_side[sub] = n_l > 0u && incl > 8u * n_l + CODEC_MARGIN ? CODEC_STORED : incl;
            // a quarter starts at every eighth lane
            if ((hl & 7u) == 0u)
                s_quarter[sub * CODEC_Q + (hl >> 3)] = before | (((lit ? first : next) - min(p0, n_l)) << 16);
            P[i].lit = lit;
            P[i].place = before | (next << 16);
            P[i].runs = run.near | (run.far << 16);
        }
    };
    if (m == CODEC_CHUNK) first_pass(std::true_type{}); else first_pass(std::false_type{});
    __syncthreads();
    // --- every wavefront places the sub-chunks for itself, lane = sub-chunk
    uint32_t start, tail_start;
    bool in_block, tail_in_block;
    const uint32_t side_l = s_side[lane];
    const uint32_t coded_bytes = place_subs(side_l, min(CODEC_SUB, m - min(m, lane * CODEC_SUB)), lane, &start, &in_block,
                                            &tail_start, &tail_in_block);
    const bool whole = m + 5u <= coded_bytes;           // not shorter than one stored block
    const uint32_t seg_bytes = whole ? m + 5u : coded_bytes;
    bool walks = false;
    if (DIRECT) {
        // a block's chunks are one link of the chain: the wavefront that brings the last size leaves their sum
        // and, behind its part of the second pass, walks back
        if (wid == 0u) {
            uint32_t done = GROUPS - 1u;
            if (GROUPS > 1) {
                if (lane == 0u) {
                    g_size[group] = alive ? seg_bytes : 0u;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    done = atomicAdd(&s_sized, 1u);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                }
                done = uniform_u32(done);
            }
            if (done == GROUPS - 1u) {
                walks = true;
                uint32_t size = seg_bytes;
                if (GROUPS > 1) {
                    size = 0;
                    for (uint32_t g = 0; g < GROUPS; ++g) size += g_size[g];
                }
                if (lane == 0u) chain_store(status + link, chain_size(link, size));
            }
        }
    } else if (tid == 0 && alive) {
        seg_size[c] = seg_bytes;
    }
    if (wid == 0u && alive) {
        side[(uint64_t)c * CODEC_NSUB + lane] = whole ? 0 : (uint16_t)side_l;
        uint64_t mark = 0;
        uint32_t b_prev = 0;
#pragma unroll
        for (uint32_t q = 1; q < CODEC_Q; ++q) {
            const uint32_t x = s_quarter[lane * CODEC_Q + q], b_q = x & 0xffffu;
            mark |= (uint64_t)((b_q - b_prev) | ((x >> 16) << 11)) << (20u * (q - 1u));
            b_prev = b_q;
        }
        const bool coded = !whole && side_l != CODEC_STORED && lane * CODEC_SUB < m;
        marks[(uint64_t)c * CODEC_NSUB + lane] = coded ? mark : 0ull;
    }
    // --- second pass: the segment
    auto second_pass = [&](auto FULL) {
        constexpr bool full = decltype(FULL)::value;
#pragma unroll
        for (uint32_t i = 0; i < STEPS; ++i) {
            const uint32_t kib = i * (DEF_THREADS / 64u) + wid, sub = kib * 2u + half;
            const uint32_t n_l = full ? CODEC_SUB : min(CODEC_SUB, m - min(m, sub * CODEC_SUB));
            const uint32_t left = full ? 16u : min(16u, n_l > p0 ? n_l - p0 : 0u);
            // two sub-chunks a wavefront: what concerns them comes by scalar reads
            auto of_sub = [&](uint32_t x) {
                const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, (int)(2u * kib));
                const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)x, (int)(2u * kib + 1u));
                return half ? b : a;
            };
            const uint32_t st = of_sub(start), sd = of_sub(side_l);
            const bool open = of_sub(in_block ? 1u : 0u) != 0u;
            const uint4 v = P[i].v;
            if (whole || sd == CODEC_STORED) {
                // bytes as they are: behind the header of the one block, or of the sub-chunk's own
                uint32_t data_bit = 40u + 8u * (sub * CODEC_SUB);
                if (!whole) {
                    const uint32_t at = st + (open ? 10u : 3u);
                    data_bit = ((at + 7u) & ~7u) + 32u;
                    if (hl == 0u && n_l > 0u) {
                        BitWriter w(s_out, st);
                        if (open) w.put(0u, 7u);              // end of the open block
                        w.put(0u, 3u);                        // BFINAL = 0, BTYPE = 00
                        w.put(0u, (8u - (at & 7u)) & 7u);
                        w.put(n_l, 16u);
                        w.put(n_l ^ 0xffffu, 16u);
                        w.finish();
                    }
                }
                if (left) {                                   // bytes past the end are zero and change nothing
                    const uint32_t at = data_bit + 8u * p0, sh = at & 31u;
                    uint32_t* o = &s_out[at >> 5];
                    auto high = [&](uint32_t hi, uint32_t lo) { return (uint32_t)((((uint64_t)hi << 32 | lo) << sh) >> 32); };
                    atomicOr(&o[0], v.x << sh);
                    atomicOr(&o[1], high(v.y, v.x));
                    atomicOr(&o[2], high(v.z, v.y));
                    atomicOr(&o[3], high(v.w, v.z));
                    if (sh) atomicOr(&o[4], high(0u, v.w));
                }
            } else if ((zero_kib >> i) & 1u) {
                if (hl == 0u) {
                    BitWriter w(s_out, st);
                    if (!open) w.put(2u, 3u);                     // BFINAL = 0, BTYPE = 01
                    w.put(ZERO_SUB_LOW, 21u);
                    w.put(ZERO_SUB_HIGH, ZERO_SUB_BITS - 21u);
                    w.finish();
                }
            } else {
                const uint32_t lit = P[i].lit, next = (P[i].place >> 16) - p0;
                if (lit) {
                    const uint32_t end = !full && n_l >= p0 && n_l - p0 < 16u ? 1u << (n_l - p0) : 0u;
                    if (hl == 0u && !open) atomicOr(&s_out[st >> 5], 2u << (st & 31u));       // BFINAL = 0, BTYPE = 01 ...
                    if (hl == 0u && !open && (st & 31u) == 31u) atomicOr(&s_out[(st >> 5) + 1u], 1u);
                    emit_tokens(s_codes, s_out, st + (open ? 0u : 3u) + (P[i].place & 0xffffu), v, lit,
                                lit | end | (next < 32u ? 1u << next : 0u), P[i].runs & 0xffffu, P[i].runs >> 16);
                }
            }
        }
    };
    if (m == CODEC_CHUNK) second_pass(std::true_type{}); else second_pass(std::false_type{});
    if (tid == DEF_THREADS - 1u) {
        if (whole) {
            BitWriter w(s_out, 0);
            w.put(last, 8u);                              // BFINAL, BTYPE = 00
            w.put(m, 16u);
            w.put(m ^ 0xffffu, 16u);
            w.finish();
        } else {
            BitWriter w(s_out, tail_start);
            if (tail_in_block) w.put(0u, 7u);             // end of block
            w.put(last, 3u);                              // empty stored block: BFINAL, BTYPE = 00
            const uint32_t at = tail_start + (tail_in_block ? 10u : 3u);
            w.put(0u, (8u - (at & 7u)) & 7u);
            w.put(0x0000u, 16u);
            w.put(0xffffu, 16u);
            w.finish();
        }
    }
    uint8_t* dst = slots + (uint64_t)c * CODEC_SLOT;
    if (DIRECT) {
        if (walks) {
            const uint32_t c0 = link * GROUPS;
            const ChainWalk walk = chain_before(status, link, lane);
            if (lane == 0u) {
                uint64_t end = walk.sum;
                for (uint32_t g = 0; g < GROUPS; ++g) {
                    const uint32_t size = GROUPS > 1 ? g_size[g] : seg_bytes;
                    if (c0 + g < n_chunks) seg_off[c0 + g] = end;
                    g_off[g] = walk.broken ? ~0ull : end;
                    end += size;
                }
                const bool ends = c0 + GROUPS >= n_chunks;
                if (ends) seg_off[n_chunks] = end;
                chain_leave(walk, link, ends, end - walk.sum, status + link, mirror, chain_store);
            }
        }
        __syncthreads();
        if (link == gridDim.x - 1u) {
            // All tickets are drawn: the next call starts from 0 on the other array, of which this block clears what
            // the call before left there.  (Nobody reads it now; this call's is left to the next one.)
            const uint32_t other = side_now ^ 1u;
            uint64_t* old = chain + CHAIN_HEADER + (uint64_t)other * chain_cap;
            const uint32_t used = (uint32_t)chain[CHAIN_USED + other];
            for (uint32_t i = threadIdx.x; i < used; i += DEF_THREADS * GROUPS) old[i] = 0;
            __syncthreads();
            if (threadIdx.x == 0) {
                chain[CHAIN_USED + other] = 0;
                chain[CHAIN_USED + side_now] = gridDim.x;
                chain_store(chain + CHAIN_TICKET, (uint64_t)other << 31);
            }
        }
        const uint64_t off = g_off[group];
        if (!alive || off == ~0ull) return;
        dst = stream + off;
    } else {
        __syncthreads();
        if (!alive) return;
    }
    // --- to memory: the first bytes up to a dword, whole dwords put together from two, the rest
    const uint32_t head = min(seg_bytes, (uint32_t)((4u - (reinterpret_cast<uintptr_t>(dst) & 3u)) & 3u));
    const uint32_t n_w = (seg_bytes - head) / 4u, sh = head * 8u;
    const uint8_t* out8 = reinterpret_cast<const uint8_t*>(s_out);
    if (tid < head) dst[tid] = out8[tid];
    uint32_t* dst32 = reinterpret_cast<uint32_t*>(dst + head);
#pragma unroll 4
    for (uint32_t k = tid; k < n_w; k += DEF_THREADS)
        dst32[k] = __builtin_amdgcn_alignbit(s_out[k + 1u], s_out[k], sh);
    const uint32_t done = head + n_w * 4u;
    if (tid < seg_bytes - done) dst[done + tid] = out8[done + tid];
}

__global__ __launch_bounds__(BLOCK) void chain_zero_kernel(uint64_t* chain, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (uint64_t)gridDim.x * BLOCK) chain[i] = 0;
}

// Byte offsets of the segments: exclusive prefix sums of their sizes (one block).  A row is
// 64 consecutive chunks, one per lane.  Every wavefront first sums its rows (every 16th),
// eight rows' loads in flight together and nothing shared but the row sums in LDS; then one
// block-wide scan over the thread totals of the row sums (a thread owns a run of rows); then
// the wavefronts visit their rows again and write the offsets: the row's base from the
// owner's total and the rows before it in the run, plus a scan across the lanes.  Three
// barriers per SCAN_ROWS_MAX rows (2 GiB of input), whatever the number of chunks below.
constexpr uint32_t SCAN_ROWS_MAX = 1024;
__global__ __launch_bounds__(1024) void codec_scan_kernel(const uint32_t* __restrict__ seg_size,
                                                          uint32_t n_chunks,
                                                          uint64_t* __restrict__ seg_off,
                                                          uint64_t stream_cap,
                                                          uint64_t* __restrict__ result) {
    __shared__ uint32_t s_row[SCAN_ROWS_MAX];           // a row's sizes sum to less than 2^32
    __shared__ uint64_t s_tbase[1024];                  // exclusive prefix of the threads' runs
    __shared__ uint64_t s_wave[16];
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    constexpr uint32_t R = 8;
    uint64_t carry = 0;                                 // the same in every thread
    for (uint32_t c0 = 0; c0 < n_chunks; c0 += SCAN_ROWS_MAX * 64u) {
        const uint32_t n_here = min(n_chunks - c0, SCAN_ROWS_MAX * 64u);
        const uint32_t* size = seg_size + c0;
        const uint32_t rows = (n_here + 63u) / 64u;
        const uint32_t rpt = (rows + 1023u) / 1024u;    // rows per thread in the scan
        for (uint32_t j0 = wid; j0 < rows; j0 += 16u * R) {
            uint32_t v[R];
#pragma unroll
            for (uint32_t u = 0; u < R; ++u) {
                const uint32_t i = (j0 + 16u * u) * 64u + lane;       // rows j0, j0 + 16, ...
                v[u] = i < n_here ? size[i] : 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < R; ++u) {
                uint32_t x = v[u];
                for (uint32_t d = 32; d > 0; d >>= 1) x += __shfl_down(x, d, 64);
                if (lane == 0 && j0 + 16u * u < rows) s_row[j0 + 16u * u] = x;
            }
        }
        __syncthreads();
        {
            uint64_t mine = 0;
            for (uint32_t i = 0; i < rpt; ++i) {
                const uint32_t j = threadIdx.x * rpt + i;
                if (j < rows) mine += s_row[j];
            }
            unsigned long long x = mine;
            for (uint32_t d = 1; d < 64; d <<= 1) {
                const unsigned long long y = __shfl_up(x, d, 64);
                if (lane >= d) x += y;
            }
            if (lane == 63u) s_wave[wid] = x;
            __syncthreads();
            uint64_t off = carry, total = 0;
            for (uint32_t k = 0; k < 16u; ++k) {
                const uint64_t w = s_wave[k];
                if (k < wid) off += w;
                total += w;
            }
            s_tbase[threadIdx.x] = off + x - mine;
            carry += total;
        }
        __syncthreads();
        for (uint32_t j0 = wid; j0 < rows; j0 += 16u * R) {
            uint32_t v[R];
#pragma unroll
            for (uint32_t u = 0; u < R; ++u) {
                const uint32_t i = (j0 + 16u * u) * 64u + lane;
                v[u] = i < n_here ? size[i] : 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < R; ++u) {
                const uint32_t j = j0 + 16u * u, i = j * 64u + lane;
                if (j < rows) {                             // the same in every lane
                    const uint32_t owner = j / rpt;
                    uint64_t base = s_tbase[owner];
                    for (uint32_t r = owner * rpt; r < j; ++r) base += s_row[r];
                    uint32_t x = v[u];
                    for (uint32_t d = 1; d < 64; d <<= 1) {
                        const uint32_t y = __shfl_up(x, d, 64);
                        if (lane >= d) x += y;
                    }
                    if (i < n_here) seg_off[(uint64_t)c0 + i] = base + x - v[u];
                }
            }
        }
        __syncthreads();                                // s_row and s_tbase are free again
    }
    if (threadIdx.x == 0) {
        seg_off[n_chunks] = carry;
        result[0] = carry;
        result[1] = carry > stream_cap ? CODEC_CAPACITY : 0u;
    }
}

// Moves every segment from its slot to its place in the stream (one wave per chunk).  The
// slot is dword aligned, the destination is not: whole destination dwords are assembled
// from two source dwords, the ragged ends go byte by byte.
__global__ __launch_bounds__(64) void codec_pack_kernel(const uint8_t* __restrict__ slots,
                                                        const uint32_t* __restrict__ seg_size,
                                                        const uint64_t* __restrict__ seg_off,
                                                        const uint64_t* __restrict__ result,
                                                        uint8_t* __restrict__ stream) {
    if (result[1] != 0) return;                       // the stream does not fit: write nothing
    const uint32_t c = blockIdx.x, lane = threadIdx.x;
    const uint8_t* src = slots + (uint64_t)c * CODEC_SLOT;
    const uint32_t* src32 = reinterpret_cast<const uint32_t*>(src);
    uint8_t* dst = stream + seg_off[c];
    const uint32_t len = seg_size[c];
    const uint32_t head = min(len, (uint32_t)((4u - (reinterpret_cast<uintptr_t>(dst) & 3u)) & 3u));
    if (lane < head) dst[lane] = src[lane];
    const uint32_t n_w = (len - head) / 4u;
    uint32_t* dst32 = reinterpret_cast<uint32_t*>(dst + head);
    const uint32_t sh = head * 8u;
    for (uint32_t k = lane; k < n_w; k += 64u) {
        // bytes head + 4k .. head + 4k + 3 of the slot (its last dword + 1 is still inside it)
        const uint32_t lo = src32[k];
        dst32[k] = sh ? (lo >> sh) | (src32[k + 1] << (32u - sh)) : lo;
    }
    const uint32_t done = head + n_w * 4u;
    if (lane < len - done) dst[done + lane] = src[done + lane];
}

// Dwords of the longest segment that the decoder's instance for chunks of few tokens takes (4.5 KiB): it keeps the segment in
// LDS, and no image of the chunk.
constexpr uint32_t CODEC_SEG_SMALL = 1152;
// n <= 32 bits at bit position pos of the staged segment
__device__ __forceinline__ uint32_t seg_peek(const uint32_t* s_seg, uint32_t pos, uint32_t n) {
    const uint32_t w = pos >> 5, sh = pos & 31u;
    const uint64_t two = (uint64_t)s_seg[w] | ((uint64_t)s_seg[w + 1u] << 32);
    return (uint32_t)(two >> sh) & (n >= 32u ? ~0u : (1u << n) - 1u);
}
__device__ __forceinline__ uint32_t seg_byte(const uint32_t* s_seg, uint32_t b) {
    return (s_seg[b >> 2] >> ((b & 3u) * 8u)) & 0xffu;
}

// What the next 9 bits of a fixed-Huffman block mean (RFC 1951 section 3.2.6), indexed by
// those bits as they come out of the stream (first bit = bit 0):
//   bits 0-4 bits used (a match: code + extra + 5 distance bits); bit 5 match; bit 6 not a
//   token (end of block, 286, 287); bits 7-15 the base length (1 for a literal); bits 16-23
//   the literal; bits 24-27 length of a match's code; bits 28-30 its number of extra bits.
// With these a literal reads as a match of length 1 of itself, and one sequence of
// operations without a branch serves both.
struct TokenTable {
    uint32_t v[512];
};
constexpr TokenTable make_token_table() {
    TokenTable t{};
    for (uint32_t r = 0; r < 512u; ++r) {
        uint32_t c9 = 0;                               // the 9 bits in code order
        for (uint32_t k = 0; k < 9u; ++k) c9 |= ((r >> k) & 1u) << (8u - k);
        uint32_t e = 0;
        if (c9 >= 0x190u) {                            // 9 bits: literals 144..255
            e = 9u | (1u << 7) | ((c9 - 0x100u) << 16);
        } else if ((c9 >> 1) >= 0x30u && (c9 >> 1) <= 0xBFu) {   // 8 bits: literals 0..143
            e = 8u | (1u << 7) | (((c9 >> 1) - 0x30u) << 16);
        } else {
            const bool seven = (c9 >> 2) <= 23u;       // 7 bits: 256..279; 8 bits: 280..287
            const uint32_t sym = seven ? 256u + (c9 >> 2) : 280u + (c9 >> 1) - 0xC0u;
            const uint32_t ncode = seven ? 7u : 8u;
            if (sym == 256u || sym > 285u) {
                e = ncode | 32u | 64u | (ncode << 24);
            } else {
                const uint32_t idx = sym - 257u;
                const uint32_t ex = (idx < 8u || idx == 28u) ? 0u : (idx - 4u) >> 2;
                const uint32_t lbase = idx < 8u ? 3u + idx : (idx == 28u ? 258u : 3u + ((4u + (idx & 3u)) << ex));
                e = (ncode + ex + 5u) | 32u | (lbase << 7) | (ncode << 24) | (ex << 28);
            }
        }
        t.v[r] = e;
    }
    return t;
}
static __device__ const TokenTable kTokenTable = make_token_table();

// Byte k of sub-chunk l in the LDS image of a chunk (rows rotated like the encoder's).
__device__ __forceinline__ uint32_t img_byte(uint32_t l, uint32_t k) {
    return sub_word(l, k >> 2) * 4u + (k & 3u);
}

// A chunk's segment as the decoder sees it: dwords aligned to the stream's start.  The stream's last dword
// may be partly beyond stream_bytes: an aligned dword never crosses a page, and what lies beyond the segment is
// never interpreted.
struct Segment {
    const uint32_t* dw;
    uint64_t s0;
    uint32_t len;       // bytes; 0: not a segment
    uint32_t byte0;     // of dw where it begins
    uint32_t max_w;     // last readable dword
};
__device__ __forceinline__ Segment segment_of(const uint8_t* __restrict__ stream, uint64_t stream_bytes, uint64_t s0, uint64_t s1) {
    Segment g;
    g.s0 = s0;
    g.len = s1 < s0 || s1 > stream_bytes || s1 - s0 < 5u || s1 - s0 > CODEC_SLOT ? 0u : (uint32_t)(s1 - s0);
    g.byte0 = (uint32_t)(s0 & 3u);
    g.dw = reinterpret_cast<const uint32_t*>(stream + (s0 & ~(uint64_t)3u));
    g.max_w = (uint32_t)(((stream_bytes + 3u) / 4u) - (s0 >> 2)) - 1u;
    return g;
}
// Dwords of a segment to be staged: two more for the look-ahead.
__device__ __forceinline__ uint32_t segment_words(uint32_t byte0, uint32_t len) { return (byte0 + len + 3u) / 4u + 2u; }

__device__ __forceinline__ void bad_stream(uint64_t* result) {
    atomicOr(reinterpret_cast<unsigned long long*>(&result[1]), (unsigned long long)CODEC_BAD_STREAM);
}

// A chunk in one stored block, copied by the block's threads.
__device__ __forceinline__ void inflate_whole(const Segment& g, const uint8_t* __restrict__ stream, uint32_t my_side, uint32_t m,
                                              uint8_t* __restrict__ dst, uint64_t* __restrict__ result) {
    const uint32_t tid = this_thread();
    const uint8_t* seg = stream + g.s0;
    const uint32_t len = seg[1] | ((uint32_t)seg[2] << 8), nlen = seg[3] | ((uint32_t)seg[4] << 8);
    if (my_side != 0u) bad_stream(result);
    if (((seg[0] >> 1) & 3u) != 0u || len != m || (len ^ nlen) != 0xffffu || g.len != m + 5u) {
        if (tid == 0) bad_stream(result);
        return;
    }
    // sixteen bytes a step, from the five dwords they lie in (loads at any byte are slower: 1.3 GB 509 us, 479 so, 466 with two
    // dwords read for each one written, which takes 124 us for 268 MB, not 115, and 30 for 33 MB, not 26)
    const uint32_t w0 = (g.byte0 + 5u) >> 2, sh = ((g.byte0 + 5u) & 3u) * 8u;
    uint4* dst16 = reinterpret_cast<uint4*>(dst);
    constexpr uint32_t U = 4;
    for (uint32_t k0 = tid; k0 * 16u + 16u <= m; k0 += U * CODEC_THREADS) {
        uint4 v[U];
        uint32_t next[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t k = k0 + u * CODEC_THREADS;
            if (k * 16u + 16u <= m) {
                v[u] = load_u4<false>(reinterpret_cast<const float*>(g.dw + w0 + 4u * k));
                next[u] = g.dw[min(w0 + 4u * k + 4u, g.max_w)];
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t k = k0 + u * CODEC_THREADS;
            auto join = [&](uint32_t hi, uint32_t lo) { return __builtin_amdgcn_alignbit(hi, lo, sh); };
            if (k * 16u + 16u <= m)
                dst16[k] = make_uint4(join(v[u].y, v[u].x), join(v[u].z, v[u].y), join(v[u].w, v[u].z), join(next[u], v[u].w));
        }
    }
    if (tid < (m & 15u)) dst[(m & ~15u) + tid] = seg[5u + (m & ~15u) + tid];
}

// A lane's part of a sub-chunk from its mark: bits [b_lo, b_hi) of the sub-chunk's tokens make
// bytes [o_lo, o_hi).
struct LanePart {
    uint32_t b_lo, b_hi, o_lo, o_hi;
    bool ok;
};
__device__ __forceinline__ LanePart lane_part(uint64_t mark, uint32_t q, uint32_t side, uint32_t n_l) {
    LanePart r{0u, side, 0u, n_l, true};
    uint32_t b_acc = 0;
#pragma unroll
    for (uint32_t j = 1; j < CODEC_Q; ++j) {
        const uint32_t field = (uint32_t)(mark >> (20u * (j - 1u))) & 0xfffffu;
        b_acc += field & 0x7ffu;
        const uint32_t o_j = min(j * CODEC_QB, n_l) + (field >> 11);
        if (j == q) { r.b_lo = b_acc; r.o_lo = o_j; }
        if (j == q + 1u) { r.b_hi = b_acc; r.o_hi = o_j; }
    }
    if ((mark >> 60) != 0ull || r.b_lo > r.b_hi || r.b_hi > side || r.o_lo > r.o_hi || r.o_hi > n_l || r.o_lo < min(q * CODEC_QB, n_l))
        r.ok = false;
    return r;
}

// The state of a lane that decodes: a 64-bit window of the token bits in two registers, from dword pos / 32 on, and
// where it writes.  Bytes travel where the table has them, in bits 16-23.
struct TokenReader {
    uint32_t pos, end, w_lo, w_hi, i, prev, seen, dist;
    // prev stays 0 until there is a literal: a lane starts with one
    __device__ __forceinline__ void begin(const uint32_t* tab, uint32_t first, uint32_t last, uint32_t lo, uint32_t hi, uint32_t at) {
        pos = first;
        end = last;
        w_lo = lo;
        w_hi = hi;
        i = at;
        prev = dist = 0;
        seen = pos < end ? (tab[__builtin_amdgcn_alignbit(w_hi, w_lo, pos) & 511u] & 32u) << 1 : 0u;
    }
    // Up to two tokens, without branches but for the stores: the table gives
    // a token's bits, kind and value, and a literal reads as a match of length 1 of
    // itself; when the token behind it is a literal (three quarters of all tokens are,
    // in half-empty data) that one is taken in the same turn (a third one gained 1 %).  Offsets are not checked
    // on the way: a store wraps inside its sub-chunk's row, offsets only
    // grow, and the end must come out exactly right.  w_new: the dword behind the window.
    // put(offset, byte << 16): only bytes that are not zero.
    template <typename Put>
    __device__ __forceinline__ void turn(const uint32_t* tab, uint32_t w_new, Put&& put) {
        const uint32_t x = __builtin_amdgcn_alignbit(w_hi, w_lo, pos);
        const uint32_t t = tab[x & 511u];
        const uint32_t nb = t & 31u;
        const uint32_t t2 = tab[__builtin_amdgcn_ubfe(x, nb, 9u)];  // at most 18 of the 32 bits are used
        const uint32_t mm = 0u - ((t >> 5) & 1u);                  // all ones for a match
        const uint32_t len = ((t >> 7) & 0x1ffu) + __builtin_amdgcn_ubfe(x, (t >> 24) & 15u, t >> 28);
        const uint32_t byte = (prev & mm) | t;                      // a match repeats the byte before it
        // not a token of this library's set (bit 6), or a match at a distance other than 1
        seen |= t;
        dist |= __builtin_amdgcn_ubfe(x, nb - 5u, 5u) & mm;
        if ((byte & 0xff0000u) != 0u) {                             // zeros are already there
            put(i, byte);
            for (uint32_t u = 1; u < len; ++u) put(i + u, byte);
        }
        i += len;
        // the second token: a literal that starts before the lane's last bit
        const bool two = (t2 & 0x60u) == 0u && pos + nb < end;
        if (two && (t2 & 0xff0000u) != 0u) put(i, t2);
        const uint32_t next = pos + nb + (two ? t2 & 31u : 0u);    // at most 18 + 9 bits on
        prev = two ? t2 : byte;
        i += two ? 1u : 0u;
        const bool take = ((pos ^ next) & 32u) != 0u;
        w_lo = take ? w_hi : w_lo;
        w_hi = take ? w_new : w_hi;
        pos = next;
    }
    __device__ __forceinline__ bool fine(uint32_t at) const { return ((seen & 64u) | dist) == 0u && pos == end && i == at; }
};

// The decoder: one block of 256 threads per chunk, four lanes per sub-chunk.  A chunk stored as one block
// is copied.  Otherwise every sub-chunk's place follows from
// the side information and every lane's from the sub-chunk's mark: lane q decodes the tokens
// from bit b_q on (or copies its 128 stored bytes).  Two instances share the chunks by segment
// size where there are many; few are all taken by the second.  The segment's size must be
// what the side information implies, every lane must end exactly where the next one
// starts, and anything but this library's own token set marks the stream as bad; no access
// leaves the stream, the staged segment, the image or the output.
//
// The instance of the short segments (chunks that are mostly zeros) visits every chunk and also takes those stored as one
// block.  It stages the segment in LDS and keeps no image of
// the chunk: it writes the chunk's zeros to memory at once, 16 bytes per thread and
// store, and after the block's barrier every lane stores its few non-zero bytes one by
// one on top.  Without the 32 KiB image many more blocks fit a compute unit, and the
// zeros are on their way while the segment is still being fetched.
__global__ __launch_bounds__(CODEC_THREADS, 5) void inflate_sparse_kernel(
    const uint8_t* __restrict__ stream, uint64_t stream_bytes, const uint64_t* __restrict__ seg_off,
    const uint16_t* __restrict__ side, const uint64_t* __restrict__ marks, uint64_t n_bytes, uint32_t n_chunks,
    uint8_t* __restrict__ out, uint64_t* __restrict__ result) {
    __shared__ uint32_t s_seg[CODEC_SEG_SMALL];
    __shared__ uint32_t s_tab[512];
    __shared__ uint32_t s_start[CODEC_NSUB];       // bit 31: a block is open there
    __shared__ uint32_t s_misc[3];                 // segment bytes, tail start, tail in block
    const uint32_t c = blockIdx.x, tid = threadIdx.x, l = tid >> 2, q = tid & 3u;
    const uint64_t base = (uint64_t)c * CODEC_CHUNK;
    const uint32_t m = (uint32_t)min((uint64_t)CODEC_CHUNK, n_bytes - min(n_bytes, base));
    const Segment g = segment_of(stream, stream_bytes, seg_off[c], seg_off[c + 1]);
    if (g.len == 0u) {
        if (tid == 0) bad_stream(result);
        return;
    }
    const uint32_t my_side = side[(uint64_t)c * CODEC_NSUB + l];
    // One stored block iff the first sub-chunk's side information is 0 (the list of the
    // other instance is made from it too); every thread then checks that its own
    // sub-chunk agrees: a coded or stored sub-chunk never has 0, a chunk stored whole has
    // nothing else.
    const bool whole = side[(uint64_t)c * CODEC_NSUB] == 0u;
    const uint32_t seg_w = segment_words(g.byte0, g.len);
    if (!whole && seg_w > CODEC_SEG_SMALL) return;                 // the other instance's chunk
    uint8_t* dst = out + base;
    if (whole) {
        inflate_whole(g, stream, my_side, m, dst, result);
        return;
    }
    const uint32_t n_l = min(CODEC_SUB, m - min(m, l * CODEC_SUB));
    const uint64_t mark = marks[(uint64_t)c * CODEC_NSUB + l];
    const bool stored_sub = my_side == CODEC_STORED;
    bool ok = stored_sub ? n_l > 0u : (n_l > 0u ? my_side <= 8u * n_l + CODEC_MARGIN : my_side == 0u);
    // The first wavefront, one lane per sub-chunk, works out where every sub-chunk's part of
    // the segment starts while the others stage the segment: one barrier
    // before the decoding, one after it.
    if (tid < CODEC_NSUB) {
        const uint32_t n_s = min(CODEC_SUB, m - min(m, tid * CODEC_SUB));
        const uint32_t v = side[(uint64_t)c * CODEC_NSUB + tid];
        const bool st = v == CODEC_STORED;
        const bool ok_s = st ? n_s > 0u : (n_s > 0u ? v != 0u && v <= 8u * n_s + CODEC_MARGIN : v == 0u);
        const bool all_ok = __ballot(!ok_s) == 0ull;
        uint32_t start, tail_start;
        bool in_block, tail_in_block;
        const uint32_t sb = place_subs(ok_s ? v : 0u, n_s, tid, &start, &in_block, &tail_start, &tail_in_block);
        s_start[tid] = start | (in_block ? 0x80000000u : 0u);
        if (tid == 0) {
            s_misc[0] = all_ok ? sb : 0xffffffffu;      // never a segment's size
            s_misc[1] = tail_start;
            s_misc[2] = tail_in_block ? 1u : 0u;
        }
    }
    for (uint32_t k = tid; k < seg_w; k += CODEC_THREADS) s_seg[k] = k <= g.max_w ? g.dw[k] : 0u;
    s_tab[tid] = kTokenTable.v[tid];
    s_tab[tid + CODEC_THREADS] = kTokenTable.v[tid + CODEC_THREADS];
    if (m == CODEC_CHUNK) {
#pragma unroll
        for (uint32_t j = 0; j < CODEC_CHUNK / 16 / CODEC_THREADS; ++j)
            *reinterpret_cast<uint4*>(dst + (j * CODEC_THREADS + tid) * 16u) = make_uint4(0, 0, 0, 0);
    } else {
        for (uint32_t v = tid; v * 16u < m; v += CODEC_THREADS) {
            if (v * 16u + 16u <= m) *reinterpret_cast<uint4*>(dst + v * 16u) = make_uint4(0, 0, 0, 0);
            else for (uint32_t k = v * 16u; k < m; ++k) dst[k] = 0;
        }
    }
    // orders the block's zeros in memory before the bytes its lanes store on top of them
    __syncthreads();
    if (s_misc[0] != g.len) {
        if (tid == 0) bad_stream(result);
        return;
    }
    const uint32_t bit0 = g.byte0 * 8u;
    const uint32_t start = s_start[l] & 0x7fffffffu;
    const bool in_block = (s_start[l] >> 31) != 0u;
    // the structure around the sub-chunks: block headers, ends of blocks, the closing
    // empty stored block
    if (n_l > 0u && q == 0u) {
        if (!stored_sub && !in_block && seg_peek(s_seg, bit0 + start, 3u) != 2u) ok = false;
        if (stored_sub && seg_peek(s_seg, bit0 + start, in_block ? 10u : 3u) != 0u) ok = false;
    }
    if (tid == CODEC_THREADS - 1u) {
        const uint32_t last = c + 1u == n_chunks ? 1u : 0u;
        uint32_t at = bit0 + s_misc[1];
        if (s_misc[2]) {
            if (seg_peek(s_seg, at, 7u) != 0u) ok = false;
            at += 7u;
        }
        if (seg_peek(s_seg, at, 3u) != last) ok = false;
        at = (at + 3u + 7u) & ~7u;
        if (seg_peek(s_seg, at, 32u) != 0xffff0000u) ok = false;
    }
    const uint32_t p_lo = min(q * CODEC_QB, n_l), p_hi = min(p_lo + CODEC_QB, n_l);
    if (stored_sub) {
        // end-of-block of the open block (7 zero bits), header 000, padding, LEN, NLEN, bytes
        const uint32_t at = bit0 + start + (in_block ? 10u : 3u);
        const uint32_t b0 = ((at + 7u) >> 3);      // byte position of LEN
        const uint32_t len = seg_byte(s_seg, b0) | (seg_byte(s_seg, b0 + 1u) << 8);
        const uint32_t nlen = seg_byte(s_seg, b0 + 2u) | (seg_byte(s_seg, b0 + 3u) << 8);
        if (len != n_l || (len ^ nlen) != 0xffffu || mark != 0ull) ok = false;
        if (ok && p_hi > p_lo) {
            const uint32_t d0 = b0 + 4u + p_lo;    // this lane's first byte
            const uint32_t shb = (d0 & 3u) * 8u, w0 = d0 >> 2, nw = (p_hi - p_lo) / 4u;
            uint32_t* out32 = reinterpret_cast<uint32_t*>(dst + l * CODEC_SUB + p_lo);   // 128-byte aligned
#pragma unroll 8
            for (uint32_t k = 0; k < nw; ++k) {
                const uint32_t lo = s_seg[w0 + k];
                out32[k] = shb ? (lo >> shb) | (s_seg[w0 + k + 1u] << (32u - shb)) : lo;
            }
            for (uint32_t k = p_lo + nw * 4u; k < p_hi; ++k) dst[l * CODEC_SUB + k] = (uint8_t)seg_byte(s_seg, d0 + k - p_lo);
        }
    } else if (n_l > 0u) {
        const LanePart part = lane_part(mark, q, my_side, n_l);
        if (!part.ok) ok = false;
        if (ok) {
            const uint32_t row = l * CODEC_SUB;
            TokenReader r;
            const uint32_t first = bit0 + start + (in_block ? 0u : 3u) + part.b_lo;
            r.begin(s_tab, first, first + (part.b_hi - part.b_lo), s_seg[first >> 5], s_seg[(first >> 5) + 1u], part.o_lo);
            while (r.pos < r.end) {
                // the window's next dword, on its way while the tokens are looked up
                const uint32_t w_new = s_seg[min((r.pos >> 5) + 2u, CODEC_SEG_SMALL - 1u)];
                // straight to memory, inside the sub-chunk and the output
                r.turn(s_tab, w_new, [&](uint32_t i, uint32_t byte) {
                    const uint32_t at = row + (i & (CODEC_SUB - 1u));
                    if (at < m) dst[at] = (uint8_t)(byte >> 16);
                });
            }
            if (!r.fine(part.o_hi)) ok = false;
        }
    } else if (mark != 0ull) {
        ok = false;
    }
    if (__syncthreads_and(ok) == 0 && tid == 0) bad_stream(result);
}

// The instance of all other segments decodes into a zeroed LDS image of the chunk, which is then written out as whole lines.
// A lane reads its own part of the segment, 56 bytes on half-full data, from memory: four dwords of it are in LDS, the two
// behind them in registers or on their way, and every second turn moves on.  What bounds it is vector issue (some 42 instructions a
// turn) and, in one round of chunks, a chunk's chain of latencies.  The whole segment staged in LDS took 68 KB with the
// image: two blocks to a compute unit, and a second round of chunks beyond 512; with 39 KB four run.  us a call
// (densities 0.05 / 0.3 / 0.5, before and now): 256 chunks 33 / 36 / 37 and 32 / 35 / 35, 1000 chunks 60 / 70 / 74 and 45 / 49 /
// 52, 8192 chunks, where a third instance took the segments of up to 16 KiB, 412 / 469 / 514 and 258 / 295 / 319, 39347
// chunks 1849 / 2192 / 2409 and 1080 / 1243 / 1333; 28 MB of a rebuilt variant, a third of it not zero, 71 and 52.  The turn
// with ten instructions less (the bit position alone says where the window and the ring are, bytes stay where the table has
// them, offsets in the image are turned once): 8192 chunks of 30 % 296 -> 276, 39347 1241 -> 1170, the rebuilt variant 51.2 -> 48.4.
constexpr uint32_t INFLATE_RING = 4;
typedef uint32_t u32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ void inflate_dense(
    uint32_t* s_img, uint32_t* s_ring, uint32_t* s_tab, uint32_t c, bool all, const uint8_t* __restrict__ stream,
    uint64_t stream_bytes, const uint64_t* __restrict__ seg_off, const uint16_t* __restrict__ side,
    const uint64_t* __restrict__ marks, uint64_t n_bytes, uint32_t n_chunks, uint8_t* __restrict__ out, uint64_t* __restrict__ result) {
    const uint32_t tid = this_thread(), l = tid >> 2, q = tid & 3u, lane = tid & 63u, wid = uniform_u32(tid >> 6);
    const uint64_t base = (uint64_t)c * CODEC_CHUNK;
    const uint32_t m = (uint32_t)min((uint64_t)CODEC_CHUNK, n_bytes - min(n_bytes, base));
    const uint32_t side_s = side[(uint64_t)c * CODEC_NSUB + lane];        // lane = sub-chunk
    const uint64_t mark = marks[(uint64_t)c * CODEC_NSUB + l];
    const Segment g = segment_of(stream, stream_bytes, seg_off[c], seg_off[c + 1]);
    const uint32_t tab0 = kTokenTable.v[tid], tab1 = kTokenTable.v[tid + CODEC_THREADS];
    if (g.len == 0u) {
        if (all && tid == 0) bad_stream(result);
        return;
    }
    uint8_t* dst = out + base;
    const uint32_t my_side = __shfl(side_s, (int)l, 64);
    if (uniform_u32(side_s) == 0u) {                                     // in one stored block
        if (all) inflate_whole(g, stream, my_side, m, dst, result);
        return;
    }
    s_tab[tid] = tab0;
    s_tab[tid + CODEC_THREADS] = tab1;
    // this wavefront's sixteen rows of the image
    static_assert(CODEC_CHUNK / 16 == 8u * CODEC_THREADS, "eight pieces a thread");
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) reinterpret_cast<uint4*>(s_img)[(wid * 8u + j) * 64u + lane] = make_uint4(0, 0, 0, 0);
    // every wavefront places the sub-chunks for itself, lane = sub-chunk
    uint32_t start, tail_start, seg_bytes;
    bool in_block, tail_in_block, ok;
    {
        const uint32_t n_s = min(CODEC_SUB, m - min(m, lane * CODEC_SUB));
        const bool ok_s = side_s == CODEC_STORED ? n_s > 0u : (n_s > 0u ? side_s != 0u && side_s <= 8u * n_s + CODEC_MARGIN : side_s == 0u);
        uint32_t start_s;
        bool in_block_s;
        seg_bytes = place_subs(ok_s ? side_s : 0u, n_s, lane, &start_s, &in_block_s, &tail_start, &tail_in_block);
        if (__ballot(!ok_s) != 0ull || seg_bytes != g.len) {
            if (tid == 0) bad_stream(result);
            return;
        }
        const uint32_t both = __shfl(start_s | (in_block_s ? 0x80000000u : 0u), (int)l, 64);
        start = both & 0x7fffffffu;
        in_block = (both >> 31) != 0u;
        ok = true;
    }
    __syncthreads();                                                     // the table
    const uint32_t n_l = min(CODEC_SUB, m - min(m, l * CODEC_SUB));
    const bool stored_sub = my_side == CODEC_STORED;
    const uint32_t bit0 = g.byte0 * 8u;
    // n <= 32 bits at bit position pos of the segment
    auto peek = [&](uint32_t pos, uint32_t n) {
        const uint32_t w = pos >> 5;
        const uint32_t lo = g.dw[min(w, g.max_w)], hi = g.dw[min(w + 1u, g.max_w)];
        return __builtin_amdgcn_alignbit(hi, lo, pos & 31u) & (n >= 32u ? ~0u : (1u << n) - 1u);
    };
    // the structure around the sub-chunks: block headers, ends of blocks, the closing
    // empty stored block
    if (n_l > 0u && q == 0u && (stored_sub || !in_block)) {
        const uint32_t head = peek(bit0 + start, stored_sub && in_block ? 10u : 3u);
        if (head != (stored_sub ? 0u : 2u)) ok = false;
    }
    if (tid == CODEC_THREADS - 1u) {
        const uint32_t last = c + 1u == n_chunks ? 1u : 0u, at = bit0 + tail_start, eob = tail_in_block ? 7u : 0u;
        const uint32_t head = peek(at, eob + 3u), lens = peek((at + eob + 3u + 7u) & ~7u, 32u);
        if (head != last << eob || lens != 0xffff0000u) ok = false;
    }
    uint8_t* img8 = reinterpret_cast<uint8_t*>(s_img);
    const uint32_t p_lo = min(q * CODEC_QB, n_l), p_hi = min(p_lo + CODEC_QB, n_l);
    if (stored_sub) {
        // end-of-block of the open block (7 zero bits), header 000, padding, LEN, NLEN, bytes
        const uint32_t at = bit0 + start + (in_block ? 10u : 3u);
        const uint32_t b0 = (at + 7u) >> 3;        // byte position of LEN
        if (peek(8u * b0, 32u) != (n_l | (~n_l << 16)) || mark != 0ull) ok = false;
        if (ok && p_hi > p_lo) {
            // this lane's bytes, at any alignment
            const uint8_t* src = reinterpret_cast<const uint8_t*>(g.dw) + b0 + 4u + p_lo;
            const uint32_t nw = (p_hi - p_lo) / 4u;
#pragma unroll 8
            for (uint32_t k = 0; k < nw; ++k) s_img[sub_word(l, p_lo / 4u + k)] = reinterpret_cast<const u32_a1*>(src)[k];
            for (uint32_t k = p_lo + nw * 4u; k < p_hi; ++k) img8[img_byte(l, k)] = src[k - p_lo];
        }
    } else if (n_l > 0u) {
        const LanePart part = lane_part(mark, q, my_side, n_l);
        if (!part.ok) ok = false;
        if (ok) {
            const uint32_t row = l * CODEC_SUB, rot = 16u * l;   // image byte of offset k: row + ((k + rot) & 511)
            const uint32_t first = bit0 + start + (in_block ? 0u : 3u) + part.b_lo;
            // Dwords at, at + 1.  The tokens end at least four bytes before the segment does, so none lies in the stream's
            // last dword: what is read again there is not used.
            auto two = [&](uint32_t at) { return *reinterpret_cast<const u32x2_a4*>(g.dw + min(at, g.max_w - 1u)); };
            const uint32_t behind = (first >> 5) + 2u;
            uint32_t filled = behind + 2u;                       // the ring holds the two dwords behind the window, up to this one
            const u32x2_a4 window = two(behind - 2u), next = two(behind);
            u32x2_a4 ahead = two(filled);
            uint32_t* ring = s_ring + tid;
            auto slot = [&](uint32_t at) { return (at & (INFLATE_RING - 1u)) * CODEC_THREADS; };
            ring[slot(behind)] = next.x;
            ring[slot(behind + 1u)] = next.y;
            TokenReader r;
            r.begin(s_tab, first, first + (part.b_hi - part.b_lo), window.x, window.y, part.o_lo + rot);
            auto put = [&](uint32_t i, uint32_t byte) { img8[row | (i & (CODEC_SUB - 1u))] = (uint8_t)(byte >> 16); };
            while (r.pos < r.end) {
                // two turns take in two dwords at most
                if (filled - (r.pos >> 5) <= 4u) {
                    ring[slot(filled)] = ahead.x;
                    ring[slot(filled + 1u)] = ahead.y;
                    filled += 2u;
                    ahead = two(filled);
                }
                r.turn(s_tab, ring[slot((r.pos >> 5) + 2u)], put);
                if (r.pos < r.end) r.turn(s_tab, ring[slot((r.pos >> 5) + 2u)], put);
            }
            if (!r.fine(part.o_hi + rot)) ok = false;
        }
    } else if (mark != 0ull) {
        ok = false;
    }
    const bool fine = __syncthreads_and(ok) != 0;
    if (!fine) {
        if (tid == 0) bad_stream(result);
        return;
    }
    // write-out: 16 bytes per thread and step, whole lines per wave
    if (m == CODEC_CHUNK) {
#pragma unroll
        for (uint32_t r = 0; r < CODEC_CHUNK / 16 / CODEC_THREADS; ++r) {
            const uint32_t v = r * CODEC_THREADS + tid;                 // 16-byte vector of the chunk
            *reinterpret_cast<uint4*>(dst + v * 16u) = *reinterpret_cast<const uint4*>(&s_img[sub_word(v >> 5, (v & 31u) * 4u)]);
        }
    } else {
        for (uint32_t r = 0; r < CODEC_CHUNK / 16 / CODEC_THREADS; ++r) {
            const uint32_t v = r * CODEC_THREADS + tid;
            if (v * 16u >= m) continue;
            const uint4 v4 = *reinterpret_cast<const uint4*>(&s_img[sub_word(v >> 5, (v & 31u) * 4u)]);
            if (v * 16u + 16u <= m) {
                *reinterpret_cast<uint4*>(dst + v * 16u) = v4;
            } else {
                const uint32_t x[4] = {v4.x, v4.y, v4.z, v4.w};
                for (uint32_t k = 0; v * 16u + k < m; ++k) dst[v * 16u + k] = (uint8_t)(x[k >> 2] >> (8u * (k & 3u)));
            }
        }
    }
}

// list: the chunks to take; nullptr: all, a block each.
__global__ __launch_bounds__(CODEC_THREADS, 4) void inflate_dense_kernel(
    const uint8_t* __restrict__ stream, uint64_t stream_bytes, const uint64_t* __restrict__ seg_off,
    const uint16_t* __restrict__ side, const uint64_t* __restrict__ marks, uint64_t n_bytes, uint32_t n_chunks,
    uint8_t* __restrict__ out, uint64_t* __restrict__ result, const uint32_t* __restrict__ list,
    const uint32_t* __restrict__ list_count) {
    __shared__ __align__(16) uint32_t s_img[CODEC_CHUNK / 4];
    __shared__ uint32_t s_ring[INFLATE_RING * CODEC_THREADS];
    __shared__ uint32_t s_tab[512];
    const uint32_t n = list ? *list_count : blockIdx.x + 1u;       // written by the classifying kernel
    for (uint32_t it = blockIdx.x; it < n; it += gridDim.x) {
        inflate_dense(s_img, s_ring, s_tab, list ? list[it] : it, !list, stream, stream_bytes, seg_off, side, marks, n_bytes,
                      n_chunks, out, result);
        __syncthreads();
    }
}

__global__ void codec_clear_kernel(uint64_t* result) {
    result[0] = 0;
    result[1] = 0;
    result[2] = 0;      // length of the decoder's chunk list
}

// The call's outcome (stream bytes, status bits) into the pinned mirror the host reads after
// its wait; the result words are then cleared for the next call (zero after use: the next
// call needs no clearing launch of its own).
__global__ void codec_publish_kernel(uint64_t* __restrict__ result, uint64_t* __restrict__ mirror) {
    mirror[CHAIN_BYTES] = result[0];
    mirror[CHAIN_STATUS] = result[1];
    mirror[CHAIN_BROKE] = 0;
    result[0] = 0;
    result[1] = 0;
    result[2] = 0;
}

// The result words are zero when a call starts: the context allocates them cleared and every
// call's last kernel leaves them so.  Only a call that could not enqueue all of its kernels
// leaves them in doubt; the call after it clears them itself.  (What a recorded call enqueues has not run: it says
// nothing about the words.)
static void codec_begin(shifter_ctx* ctx, bool recording) {
    if (ctx->codec_dirty) codec_clear_kernel<<<1, 1, 0, ctx->stream>>>(ctx->d_codec);
    if (!recording) ctx->codec_dirty = true;
}
static void codec_end(shifter_ctx* ctx, bool recording) {
    codec_publish_kernel<<<1, 1, 0, ctx->stream>>>(ctx->d_codec, ctx->dev_codec_mirror);
    if (!recording && hipPeekAtLastError() == hipSuccess) ctx->codec_dirty = false;
}

// Up to this many chunks, three to each of 256 compute units, a block takes one chunk, beyond it two: they
// wait for each other at the barriers, which a chip that is not full notices, and share a ticket and a link.  us a
// call, one / two, by the share of weights that are not zero (both with a launch that cleared the chain, 1.5 us, since gone):
//   chunks    none        0.5 %       5 %         30 %        all
//   769       34 / 30     42 / 41     48 / 46     51 / 49     44 / 40
//   1024      41 / 33     49 / 44     53 / 49     56 / 52     52 / 45
//   4096      82 / 64     97 / 94     110 / 112   118 / 121   112 / 106
//   39347     538 / 414   617 / 636   745 / 838   815 / 906   889 / 708
// From 4096 chunks on a partly sparse input would gain up to a tenth from one, an empty or a dense one lose a fifth; which
// it is nobody knows before the pass.  (4 chunks 27 / 33, 256 32 / 35, 640 47 / 51 before the barrier went, 30 %.)
constexpr uint32_t DEFLATE_ONE_EACH = 768;

// Room for a chunk list, kept by the context and doubled when a longer input comes.  A list that is outgrown goes with the
// context: a recorded call of the decoder still writes and reads it.
static hipError_t codec_ensure_list(shifter_ctx* ctx, uint64_t entries) {
    if (ctx->codec_list_cap >= entries) return hipSuccess;
    uint64_t cap = 1024;
    while (cap < entries) cap *= 2u;
    uint32_t* list = nullptr;
    const hipError_t e = hipMalloc(reinterpret_cast<void**>(&list), sizeof(uint32_t) * cap);
    if (e != hipSuccess) return e;
    if (ctx->d_codec_list) ctx->codec_retired.push_back(ctx->d_codec_list);
    ctx->d_codec_list = list;
    ctx->codec_list_cap = cap;
    return hipSuccess;
}

// Whether the context's stream is recording (the null stream never is).
static hipError_t codec_recording(const shifter_ctx* ctx, bool* recording) {
    *recording = false;
    if (!ctx->stream) return hipSuccess;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(ctx->stream, &status);
    *recording = status != hipStreamCaptureStatusNone;
    return e;
}

// A block takes one chunk or two (DEFLATE_ONE_EACH).
static uint32_t deflate_links(uint32_t n_chunks) { return n_chunks > DEFLATE_ONE_EACH ? (n_chunks + 1u) / 2u : n_chunks; }

// Words for the chain of an input of so many chunks.  Every call that is not recorded makes room for it, the decoder's too:
// nothing is allocated behind a call of that size.  Recorded calls have their chain elsewhere.
static hipError_t codec_ensure_chain(shifter_ctx* ctx, uint32_t n_chunks) {
    const uint32_t links = deflate_links(n_chunks);
    if (ctx->codec_chain_cap >= links) return hipSuccess;
    uint32_t cap = 1024;
    while (cap < links) cap *= 2u;                       // links < 2^31
    const uint64_t words = CHAIN_HEADER + 2ull * cap;
    uint64_t* chain = nullptr;
    const hipError_t e = hipMalloc(reinterpret_cast<void**>(&chain), words * sizeof(uint64_t));
    if (e != hipSuccess) return e;
    chain_zero_kernel<<<64, BLOCK, 0, ctx->stream>>>(chain, words);
    const hipError_t zeroed = hipPeekAtLastError();
    if (zeroed != hipSuccess) {
        (void)hipFree(chain);
        return zeroed;
    }
    if (ctx->d_codec_chain) ctx->codec_retired.push_back(ctx->d_codec_chain);
    ctx->d_codec_chain = chain;
    ctx->codec_chain_cap = cap;
    return hipSuccess;
}

// Kernels only, nothing waited for.  Returns a HIP error code (0: fine).
int launch_deflate(shifter_ctx* ctx, const uint8_t* d_in, uint64_t n_bytes, uint32_t n_chunks,
                   uint8_t* d_work, uint8_t* d_stream, uint64_t stream_cap, uint64_t* d_seg_off,
                   uint16_t* d_sub_bits, uint64_t* d_sub_marks) {
    // the decoder's list and the encoder's chain: a call of either kind makes room for both, so that
    // either may be recorded into a graph behind it
    bool recording;
    hipError_t e = codec_recording(ctx, &recording);
    if (e == hipSuccess) e = codec_ensure_list(ctx, n_chunks);
    if (e == hipSuccess && !recording) e = codec_ensure_chain(ctx, n_chunks);
    if (e != hipSuccess) return (int)e;
    if (stream_cap >= n_bytes + 5ull * n_chunks) {
        // the stream holds every segment stored: it cannot overflow, so the segments go straight
        // to their places
        const bool two = n_chunks > DEFLATE_ONE_EACH;
        const uint32_t links = deflate_links(n_chunks);
        uint64_t* chain = ctx->d_codec_chain;
        uint32_t chain_cap = ctx->codec_chain_cap;
        if (recording) {
            // The context's words are its own calls' in turn, and grow: a replay, which may come at any time, has none of
            // them.  The workspace holds a slot of 32776 bytes a chunk, which this form leaves empty.
            static_assert((CHAIN_HEADER + 1u) * sizeof(uint64_t) <= CODEC_SLOT, "a header and a word for each chunk");
            chain = reinterpret_cast<uint64_t*>(d_work);
            chain_cap = links;
            const uint32_t words = CHAIN_HEADER + links;
            ProfileScope ps(ctx, K_CODEC_SCAN);
            chain_zero_kernel<<<std::min((words + BLOCK - 1u) / BLOCK, 64u), BLOCK, 0, ctx->stream>>>(chain, words);
        }
        ProfileScope ps(ctx, K_DEFLATE_CHUNK);
        const auto kernel = two ? deflate_kernel<true, 2> : deflate_kernel<true, 1>;
        kernel<<<links, two ? 2u * DEF_THREADS : DEF_THREADS, 0, ctx->stream>>>(
            d_in, n_bytes, n_chunks, d_sub_bits, d_sub_marks, nullptr, nullptr, chain, chain_cap, d_seg_off,
            d_stream, ctx->dev_codec_mirror);
        return 0;
    }
    uint32_t* seg_size = reinterpret_cast<uint32_t*>(d_work);
    uint8_t* slots = d_work + codec_slots_offset(n_chunks);
    codec_begin(ctx, recording);
    {
        ProfileScope ps(ctx, K_DEFLATE_CHUNK);
        deflate_kernel<false, 1><<<n_chunks, DEF_THREADS, 0, ctx->stream>>>(
            d_in, n_bytes, n_chunks, d_sub_bits, d_sub_marks, slots, seg_size, nullptr, 0u, nullptr, nullptr, nullptr);
    }
    {
        ProfileScope ps(ctx, K_CODEC_SCAN);
        codec_scan_kernel<<<1, 1024, 0, ctx->stream>>>(seg_size, n_chunks, d_seg_off, stream_cap,
                                                       ctx->d_codec);
    }
    {
        ProfileScope ps(ctx, K_CODEC_PACK);
        codec_pack_kernel<<<n_chunks, 64, 0, ctx->stream>>>(slots, seg_size, d_seg_off, ctx->d_codec,
                                                            d_stream);
    }
    codec_end(ctx, recording);
    return 0;
}

// The list of the chunks whose segments the second instance of the decoder takes (the same rule as inside the
// first); its length in result[2].  One atomic per block (atomics to one address take their turns, about 10 ns
// each): the wavefronts' counts meet in LDS and share the range the block reserves.
constexpr uint32_t CLASSIFY_THREADS = 1024;
__global__ __launch_bounds__(CLASSIFY_THREADS) void codec_classify_kernel(
    uint64_t stream_bytes, const uint64_t* __restrict__ seg_off, const uint16_t* __restrict__ side,
    uint32_t n_chunks, uint32_t* __restrict__ list, uint64_t* __restrict__ result) {
    constexpr uint32_t WAVES = CLASSIFY_THREADS / 64u;
    __shared__ uint32_t s_cnt[WAVES], s_base;
    const uint32_t c = blockIdx.x * CLASSIFY_THREADS + threadIdx.x, lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    bool dense = false;
    if (c < n_chunks) {
        const uint64_t s0 = seg_off[c], s1 = seg_off[c + 1];
        // a broken offset is reported by the first instance; one stored block is its chunk too
        if (!(s1 < s0 || s1 > stream_bytes || s1 - s0 < 5u || s1 - s0 > CODEC_SLOT) &&
            side[(uint64_t)c * CODEC_NSUB] != 0u)
            dense = segment_words((uint32_t)(s0 & 3u), (uint32_t)(s1 - s0)) > CODEC_SEG_SMALL;
    }
    const uint64_t votes = __ballot(dense);
    if (lane == 0) s_cnt[wid] = (uint32_t)__popcll(votes);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (uint32_t w = 0; w < WAVES; ++w) total += s_cnt[w];
        s_base = total ? atomicAdd(reinterpret_cast<uint32_t*>(&result[2]), total) : 0u;
    }
    __syncthreads();
    if (dense) {
        uint32_t at = s_base;
        for (uint32_t w = 0; w < wid; ++w) at += s_cnt[w];
        list[at + (uint32_t)__popcll(votes & ((1ull << lane) - 1ull))] = c;
    }
}

// Up to this many chunks - one round of four blocks on each of 256 compute units - the second instance takes them all. An
// instance's time is then the latency of a chunk, and two instances one behind the other cost two; beyond it the
// chunks of few tokens fare better with their own.  us a call, chunks of one density from 0.05 to 0.5 / of densities from 0
// to 1: 1000 chunks 45-52 / 52, 1030 58-67 / 65.
constexpr uint32_t INFLATE_ONE_LAUNCH = 1024;

// Kernels only, nothing waited for: the list of the second instance is made on the
// device and walked by a fixed grid.  Returns a HIP error code (0: fine).
int launch_inflate(shifter_ctx* ctx, const uint8_t* d_stream, uint64_t stream_bytes,
                   const uint64_t* d_seg_off, const uint16_t* d_sub_bits, const uint64_t* d_sub_marks,
                   uint64_t n_bytes, uint32_t n_chunks, uint8_t* d_out) {
    bool recording;
    hipError_t e0 = codec_recording(ctx, &recording);
    if (e0 == hipSuccess) e0 = codec_ensure_list(ctx, n_chunks);
    if (e0 == hipSuccess && !recording) e0 = codec_ensure_chain(ctx, n_chunks);
    if (e0 != hipSuccess) return (int)e0;
    codec_begin(ctx, recording);
    if (n_chunks <= INFLATE_ONE_LAUNCH) {
        ProfileScope ps(ctx, K_INFLATE_CHUNK);
        inflate_dense_kernel<<<n_chunks, CODEC_THREADS, 0, ctx->stream>>>(d_stream, stream_bytes, d_seg_off, d_sub_bits, d_sub_marks,
                                                                          n_bytes, n_chunks, d_out, ctx->d_codec, nullptr, nullptr);
    } else {
        ProfileScope ps(ctx, K_INFLATE_CHUNK);
        codec_classify_kernel<<<(n_chunks + CLASSIFY_THREADS - 1) / CLASSIFY_THREADS, CLASSIFY_THREADS, 0, ctx->stream>>>(
            stream_bytes, d_seg_off, d_sub_bits, n_chunks, ctx->d_codec_list, ctx->d_codec);
        // the long segments first: their blocks run longest
        inflate_dense_kernel<<<std::min(n_chunks, CODEC_LOOP_GRID), CODEC_THREADS, 0, ctx->stream>>>(
            d_stream, stream_bytes, d_seg_off, d_sub_bits, d_sub_marks, n_bytes, n_chunks, d_out, ctx->d_codec, ctx->d_codec_list,
            reinterpret_cast<const uint32_t*>(ctx->d_codec + 2));
        inflate_sparse_kernel<<<n_chunks, CODEC_THREADS, 0, ctx->stream>>>(d_stream, stream_bytes, d_seg_off, d_sub_bits, d_sub_marks,
                                                                          n_bytes, n_chunks, d_out, ctx->d_codec);
    }
    codec_end(ctx, recording);
    return 0;
}

}  // namespace shifter
