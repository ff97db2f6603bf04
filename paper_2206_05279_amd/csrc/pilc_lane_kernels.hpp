// One thread per lane: the kernels for batches with many lanes (gfx950).
//
// Every thread walks its own lane (App. A eqs. (11)-(12) of arXiv 2206.05279 are serial per
// lane), so neighbouring threads read memory a whole lane apart.  A lane is consumed in chunks of
// 8 pixels held in registers: when the geometry keeps every chunk 8-pixel aligned (kVec) the
// 24 + 48 + 48 bytes of a chunk arrive as 64- and 128-bit loads, and decoded pixels leave as
// 64-bit stores; otherwise, and for ragged chunk tails, the same registers are filled element by
// element.  The coded words, which a thread produces or consumes one at a time, never go to
// memory one at a time: the encoder writes them to a scratch laid out [word number][thread], so
// that the 64 lanes of a wavefront fill whole lines, and the decoder reads them through a ring
// of 32 words per thread in LDS that is refilled with 16-byte loads between chunks.
#pragma once

#include <type_traits>

#include "pilc_device.hpp"

namespace pilc {

constexpr int kChunk = 8;  // pixels per chunk
constexpr int kLaneMaxThreads = 256;  // the lane kernels run in workgroups of 64 or 256

struct Chunk {
    int x[kChunk][3];   // pixel values (encode)
    int m[kChunk][3];   // mu, Q8.8
    int l[kChunk][3];   // log-scale, Q4.12
};

__device__ __forceinline__ int byte_of(const uint32_t *w, int i) { return (w[i >> 2] >> (8 * (i & 3))) & 0xFF; }
__device__ __forceinline__ int half_of(const uint32_t *w, int i) { return (w[i >> 1] >> (16 * (i & 1))) & 0xFFFF; }

// The 8 pixels held in the words wx (6 dwords of pixels), wm and wl (12 dwords each) into `c`.
template <bool kPixels>
__device__ __forceinline__ void unpack_chunk(Chunk &c, const uint32_t *wx, const uint32_t *wm,
                                             const uint32_t *wl)
{
#pragma unroll
    for (int i = 0; i < kChunk; ++i)
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            if (kPixels) c.x[i][ch] = byte_of(wx, 3 * i + ch);
            c.m[i][ch] = half_of(wm, 3 * i + ch);
            c.l[i][ch] = (int)(short)half_of(wl, 3 * i + ch);
        }
}

// Fills `c` with the pixels p .. p+len-1 (len <= 8).  kVec: p is a multiple of 8 and the arrays
// are 16-byte aligned, so a full chunk is 3 x 8 bytes of pixels and 3 x 16 bytes of each parameter.
// Otherwise the same loads at whatever address they fall on, also for a row's last pixels, which are followed by other
// pixels' values that nobody looks at; one by one only where eight pixels would reach past the
// array's end (`total_px`).  (One by one everywhere, 72 loads of one or two bytes a chunk were what such batches
// waited for: 8 images of 1365 x 2047 in tiles 733 -> 383 us to decode, 681 -> 376 to encode.)
template <bool kVec, bool kPixels>
__device__ __forceinline__ void load_chunk(Chunk &c, uint32_t p, uint32_t len, uint32_t total_px,
                                           const uint8_t *__restrict__ img,
                                           const uint16_t *__restrict__ mu,
                                           const int16_t *__restrict__ ls)
{
    const size_t s = (size_t)p * 3;
    uint32_t wx[6] = {0, 0, 0, 0, 0, 0}, wm[12] = {}, wl[12] = {};
    if (kVec ? len == (uint32_t)kChunk : total_px - p >= (uint32_t)kChunk) {
        if (kVec) {
            const uint4 *pm = reinterpret_cast<const uint4 *>(mu + s);
            const uint4 *pl = reinterpret_cast<const uint4 *>(ls + s);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const uint4 a = pm[q], b = pl[q];
                wm[4 * q] = a.x; wm[4 * q + 1] = a.y; wm[4 * q + 2] = a.z; wm[4 * q + 3] = a.w;
                wl[4 * q] = b.x; wl[4 * q + 1] = b.y; wl[4 * q + 2] = b.z; wl[4 * q + 3] = b.w;
            }
        } else {
            __builtin_memcpy(wm, mu + s, 48);
            __builtin_memcpy(wl, ls + s, 48);
        }
        if (kPixels) {
            if (kVec) {
                const uint2 *px = reinterpret_cast<const uint2 *>(img + s);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const uint2 a = px[q];
                    wx[2 * q] = a.x; wx[2 * q + 1] = a.y;
                }
            } else {
                __builtin_memcpy(wx, img + s, 24);
            }
        }
    } else if (!kVec && kPixels) {
        // into the same words, so that the two ways meet in 30 registers and not in 72
#pragma unroll
        for (int e = 0; e < 3 * kChunk; ++e) {
            const size_t at = s + ((uint32_t)e < 3u * len ? e : 0);
            wx[e >> 2] |= (uint32_t)img[at] << (8 * (e & 3));
            wm[e >> 1] |= (uint32_t)mu[at] << (16 * (e & 1));
            wl[e >> 1] |= (uint32_t)(uint16_t)ls[at] << (16 * (e & 1));
        }
    } else {
#pragma unroll
        for (int i = 0; i < kChunk; ++i)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const bool in = (uint32_t)i < len;
                const size_t e = in ? s + 3 * i + ch : s;
                if (kPixels) c.x[i][ch] = img[e];
                c.m[i][ch] = mu[e];
                c.l[i][ch] = ls[e];
            }
        return;
    }
    unpack_chunk<kPixels>(c, wx, wm, wl);
}

// Two neighbouring chunks (16 pixels from p, a multiple of 16) as raw words: 96 bytes of each
// parameter array and 48 of pixels in 16-byte loads.  Taking two chunks at a time halves the
// number of times a thread comes back to a 128-byte line.
struct ChunkPair {
    uint32_t wx[12], wm[24], wl[24];
};
template <bool kPixels>
__device__ __forceinline__ void load_pair(ChunkPair &r, uint32_t p, const uint8_t *__restrict__ img,
                                          const uint16_t *__restrict__ mu,
                                          const int16_t *__restrict__ ls)
{
    const size_t s = (size_t)p * 3;
    const uint4 *pm = reinterpret_cast<const uint4 *>(mu + s);
    const uint4 *pl = reinterpret_cast<const uint4 *>(ls + s);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const uint4 a = pm[q], b = pl[q];
        r.wm[4 * q] = a.x; r.wm[4 * q + 1] = a.y; r.wm[4 * q + 2] = a.z; r.wm[4 * q + 3] = a.w;
        r.wl[4 * q] = b.x; r.wl[4 * q + 1] = b.y; r.wl[4 * q + 2] = b.z; r.wl[4 * q + 3] = b.w;
    }
    if (kPixels) {
        const uint4 *px = reinterpret_cast<const uint4 *>(img + s);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint4 a = px[q];
            r.wx[4 * q] = a.x; r.wx[4 * q + 1] = a.y; r.wx[4 * q + 2] = a.z; r.wx[4 * q + 3] = a.w;
        }
    }
}

// Whole-line feeding of ChunkPair for flat lanes made of 64-pixel groups that start on a 128-byte
// line of the parameter arrays (a group is three lines of each, a line 21 1/3 pixels).  A pair of
// chunks takes 96 bytes of each array, so three of every four pairs straddle a line; asked for by
// the pair, every line would be fetched twice, because it has left the caches when the thread
// comes back to it.  Here a thread asks for whole lines, eight 16-byte pieces at once, when a pair
// first needs one, and carries the pieces the pair does not use in registers to the pairs that
// do: every line is fetched once.  The pixels go the same way in halves of a group (96 bytes).
// `v` is the pair's number within its group (0..3); the encoder walks its lane backwards, so the
// pairs come in the order 3, 2, 1, 0.
struct LineCarry {
    uint4 m[6], l[6], x[3];
};
__device__ __forceinline__ void put_piece(uint32_t *w, int i, const uint4 &q)
{
    w[4 * i] = q.x; w[4 * i + 1] = q.y; w[4 * i + 2] = q.z; w[4 * i + 3] = q.w;
}
// One array's share of a pair: `grp` points at the group's 24 pieces.  Every piece is loaded
// straight into the place it is used from (the pair's words or the carry), so no more registers
// are alive than the pair and the carry take.
__device__ __forceinline__ void load_piece(uint32_t *w, int i, const uint4 *__restrict__ src)
{
    put_piece(w, i, *src);
}
__device__ __forceinline__ void feed_array(uint32_t *w, uint4 *carry, uint32_t v, const uint4 *__restrict__ grp)
{
    // v=3 line C: use C2-7, keep C0,1 | v=2 line B: B4-7 + kept, keep B0-3 |
    // v=1 line A: A6,7 + kept, keep A0-5 | v=0: kept
    switch (v) {
    case 3:
#pragma unroll
        for (int i = 0; i < 6; ++i) load_piece(w, i, grp + 18 + i);
        carry[0] = grp[16]; carry[1] = grp[17];
        break;
    case 2:
#pragma unroll
        for (int i = 0; i < 4; ++i) load_piece(w, i, grp + 12 + i);
        put_piece(w, 4, carry[0]); put_piece(w, 5, carry[1]);
#pragma unroll
        for (int i = 0; i < 4; ++i) carry[i] = grp[8 + i];
        break;
    case 1:
        load_piece(w, 0, grp + 6); load_piece(w, 1, grp + 7);
#pragma unroll
        for (int i = 0; i < 4; ++i) put_piece(w, 2 + i, carry[i]);
#pragma unroll
        for (int i = 0; i < 6; ++i) carry[i] = grp[i];
        break;
    default:
#pragma unroll
        for (int i = 0; i < 6; ++i) put_piece(w, i, carry[i]);
        break;
    }
}
// The pair `v` of the group whose first pixel is `pg` (a multiple of 64 pixels from the lane's start).
__device__ __forceinline__ void feed_pair(ChunkPair &r, LineCarry &c, uint32_t v, uint32_t pg,
                                          const uint8_t *__restrict__ img, const uint16_t *__restrict__ mu,
                                          const int16_t *__restrict__ ls)
{
    const size_t s = (size_t)pg * 3;
    feed_array(r.wm, c.m, v, reinterpret_cast<const uint4 *>(mu + s));
    feed_array(r.wl, c.l, v, reinterpret_cast<const uint4 *>(ls + s));
    const uint4 *px = reinterpret_cast<const uint4 *>(img + s);  // 12 pieces a group, 3 a pair
    if ((v & 1u) != 0u) {  // first pair of its half
        const uint32_t h = 6u * (v >> 1);
        uint4 n[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) n[i] = px[h + i];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            put_piece(r.wx, i, n[3 + i]);
            c.x[i] = n[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) put_piece(r.wx, i, c.x[i]);
    }
}

// A little more than 1 / f, for floor(S / f) of a state S < 2^32 as the low word of a double: S r + 2^52 - 1/2 rounded to
// the nearest whole number is 2^52 + floor(S r) (S r is never whole, and S >= f), and that is the quotient while r lies in
// 1/f .. (1 + 2^-33) / f.  One step of Newton's towards (1 + 2^-35) / f takes the single-precision reciprocal's error of 2^-22
// to 2^-44.
__device__ __forceinline__ double over_reciprocal(uint32_t f)
{
    const double r0 = (double)__builtin_amdgcn_rcpf((float)f);
    return __builtin_fma(r0, __builtin_fma(-(double)f, r0, 1.0 + 0x1p-35), r0);
}
__device__ __forceinline__ uint32_t quotient(uint32_t n, double r)
{
    return (uint32_t)__builtin_bit_cast(unsigned long long, __builtin_fma((double)n, r, 0x1p52 - 0.5));
}

// Chunk c of a lane: rows of sh.tw pixels, g.w apart, each cut into pieces of 8 pixels.
struct ChunkPos {
    uint32_t p, len;
};
__device__ __forceinline__ ChunkPos chunk_pos(const Geo &g, const LaneShape &sh, uint32_t per_row,
                                              uint32_t c)
{
    const uint32_t row = c / per_row, k = c - row * per_row;
    ChunkPos r;
    r.p = sh.first + row * g.w + k * kChunk;
    r.len = min((uint32_t)kChunk, sh.tw - k * kChunk);
    return r;
}

// --------------------------------------------------------------------------------------------
// Encode.  Symbols are pushed last-first (App. A eq. (11)), so the 16-bit words come out in the
// reverse of the order the decoder reads them.  Scratch is laid out per wavefront as
// [word number][thread]: the k-th word of the 64 lanes of a wavefront share a 128-byte line, and
// since neighbouring lanes emit at nearly the same pace a line is complete soon after it is first
// touched.  `lane_cap` is the room every lane has (words); the packer reads a lane's words back
// from the highest number down.
// --------------------------------------------------------------------------------------------
constexpr uint32_t kLaneMostSymbols = (1u << 25) - 1u;  // of a lane: 64 lanes' words are placed by 32 bits of bytes
__device__ __forceinline__ size_t lane_scratch_base(uint32_t lane, uint32_t lane_cap)
{
    return (size_t)(lane & ~63u) * lane_cap + (lane & 63u);
}

// kPair (with kVec): every row of every lane is a whole number of 16-pixel pairs of chunks that
// start at multiples of 16 pixels, and the arrays allow 16-byte loads.
// kLine (with kPair, flat lanes): lanes are whole 64-pixel groups that start on 128-byte lines.
// Encodes lane `lane` into its column of the scratch; returns the number of words, the final
// state in `state_out`.
template <bool kVec, bool kPair, bool kLine>
__device__ __forceinline__ uint32_t encode_lane(const Geo &g, uint32_t lane, const uint8_t *__restrict__ img,
                                                const uint16_t *__restrict__ mu,
                                                const int16_t *__restrict__ ls,
                                                const int16_t *__restrict__ coef,
                                                uint16_t *__restrict__ scratch, uint32_t lane_cap,
                                                const LdsTables &tab, uint32_t &state_out)
{
    const LaneShape sh = lane_shape(g, lane);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), top = 1u << m_bits;
    const uint32_t per_row = (sh.tw + kChunk - 1) / kChunk;
    const uint32_t chunks = per_row * (sh.npx / sh.tw);

    // the wavefront's columns, and the place of the lane's next word in them in bytes (below 2^32: kLaneMostSymbols)
    char *columns = reinterpret_cast<char *>(scratch + (size_t)__builtin_amdgcn_readfirstlane(lane & ~63u) * lane_cap);
    const uint32_t first_word = 2u * (lane & 63u);
    uint32_t next_word = first_word;
    uint32_t S = 1u << 16;

    // whole: a compile-time constant, no thread's chunk is a shorter one
    auto encode_chunk = [&](const Chunk &ck, const ChunkPos cp, auto whole) {
        // a chunk never straddles two images when kVec; otherwise take the image per pixel
        uint32_t im = g.by_hw.div(cp.p);
        int a_gr = coef[3 * im], a_br = coef[3 * im + 1], a_bg = coef[3 * im + 2];
        // The chunk in parts of four pixels (two in the whole-line variant, which has no registers for more), the last
        // part first.  Phase 1 of a part: cum and freq of its symbols; nothing there depends on the state, so the
        // evaluations overlap freely.  Phase 2: the serial chain (App. A eq. (11)), last symbol first.  What bounds the
        // kernel is vector instructions (56 a symbol, 65 before), the waits for the tables and the stores of words.
        // The quotient is exact at the first go (quotient above), where a single-precision estimate took a
        // remainder and a correction; an edge takes one conversion less (EdgeStep).  Whole calls, us, before and
        // now: 16,384 images of 64 x 64 with a lane a row 641 and 578, 1024 of 256 x 256 721 and 616, 30 frames of 1080 x 1920 in
        // tiles of 16 x 16 523 and 491, 8 images of 1365 x 2047 in the same 359 and 308.  A store in every step, of a word that
        // is written over if it does not count, leaves no branch in a part but costs more than the branches: 689,
        // 749, 580 and 328.
        constexpr int kHalf = kLine ? kChunk / 4 : kChunk / 2;
#pragma unroll
        for (int hb = kChunk / kHalf - 1; hb >= 0; --hb) {
            uint32_t cum[3 * kHalf], freq[3 * kHalf];
#pragma unroll
            for (int ii = 0; ii < kHalf; ++ii) {
                const int i = kHalf * hb + ii;
                if (!kVec && (uint32_t)i < cp.len) {
                    const uint32_t im_i = g.by_hw.div(cp.p + i);
                    if (im_i != im) {
                        im = im_i;
                        a_gr = coef[3 * im]; a_br = coef[3 * im + 1]; a_bg = coef[3 * im + 2];
                    }
                }
                // 256 x - mean of the three channels, from the last two what the channels before them say
                const int e_r = ck.x[i][0] * 256 - ck.m[i][0], e_g = ck.x[i][1] * 256 - ck.m[i][1];
                const int e[3] = {e_r, e_g - rsh14_mul(a_gr, e_r),
                                  ck.x[i][2] * 256 - ck.m[i][2] - rsh14_mul(a_br, e_r) - rsh14_mul(a_bg, e_g)};
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) {
                    const int x = ck.x[i][ch];
                    const EdgeStep edge(e[ch] - 128, inv_scale(ck.l[i][ch], tab));
                    // both edges always, so that no branch keeps the evaluations of the half apart (the
                    // compiler would skip the one that is not needed): 0.48 -> 0.45 ms on 30 frames of
                    // 1080 x 1920 in tiles
                    uint32_t lo = cum_inner(x, edge.y, scale, tab);
                    uint32_t hi = cum_inner(x + 1, edge.above(), scale, tab);
                    asm("" : "+v"(lo), "+v"(hi));
                    lo = x == 0 ? 0u : lo;
                    hi = x == 255 ? top : hi;
                    cum[3 * ii + ch] = lo;
                    freq[3 * ii + ch] = hi - lo;
                }
            }
#pragma unroll
            for (int kk = 3 * kHalf - 1; kk >= 0; --kk) {
                const uint32_t f = freq[kk];
                const bool coded = decltype(whole)::value || (uint32_t)(3 * kHalf * hb + kk) < 3u * cp.len;
                // S >= f << (32-M) gives its low word off
                const uint32_t high = S >> 16;
                const bool gives = high >= f << (16u - m_bits);
                if (coded && gives) *reinterpret_cast<uint16_t *>(columns + next_word) = (uint16_t)S;
                next_word += (coded && gives) ? 128u : 0u;
                const uint32_t s = gives ? high : S;
                uint32_t with_cum = s + cum[kk];
                asm("" : "+v"(with_cum));  // (the multiply-add below takes it whole)
                // (q << M) + (s - q f) + cum
                const uint32_t next = (uint32_t)__umul24(quotient(s, over_reciprocal(f)), top - f) + with_cum;
                S = coded ? next : S;
            }
        }
    };

    if (kVec && kPair) {
        // chunks 2i and 2i + 1 of a lane are neighbours in a row; the right one is coded first
        LineCarry carry;
        for (uint32_t c = chunks; c >= 2u; c -= 2u) {
            const ChunkPos left = chunk_pos(g, sh, per_row, c - 2u);
            ChunkPair raw;
            if (kLine) {
                const uint32_t pair = (c - 2u) >> 1;  // pairs of a flat lane are 16 pixels apart
                feed_pair(raw, carry, pair & 3u, sh.first + 16u * (pair & ~3u), img, mu, ls);
            } else {
                load_pair<true>(raw, left.p, img, mu, ls);
            }
            auto half = [&](auto h) {  // h: which chunk of the pair, as a compile-time constant
                constexpr int kH = decltype(h)::value;
                Chunk ck;
                unpack_chunk<true>(ck, raw.wx + 6 * kH, raw.wm + 12 * kH, raw.wl + 12 * kH);
                ChunkPos cp;
                cp.p = left.p + (uint32_t)(kChunk * kH);
                cp.len = (uint32_t)kChunk;
                encode_chunk(ck, cp, std::true_type{});
            };
            half(std::integral_constant<int, 1>{});
            half(std::integral_constant<int, 0>{});
        }
    } else {
        for (uint32_t c = chunks; c-- > 0u;) {
            const ChunkPos cp = chunk_pos(g, sh, per_row, c);
            Chunk ck;
            load_chunk<kVec, true>(ck, cp.p, cp.len, g.total_px, img, mu, ls);
            // Rows that do not align have one copy of the code, for chunks of any length: with one for whole chunks beside it they
            // take 150 registers for 124, three wavefronts a SIMD for four.  Policy 1, us, two copies and one: tiles of 10 x 10
            // 66,000 lanes 190 and 182, 262,080 375 and 331; of 7 x 13 262,080 296 and 262, 499,950 506 and 460; flat lanes of 100
            // 500,000 660 and 616, of 5 86 and 83.  (Aligned rows are not ahead with fewer: tiles of 8 x 24 at 114,984
            // lanes 274 with 138 registers, 287 with 93.)
            if (kVec && __all(cp.len == (uint32_t)kChunk))
                encode_chunk(ck, cp, std::true_type{});
            else
                encode_chunk(ck, cp, std::false_type{});
        }
    }
    state_out = S;
    // (first_word, below 128, goes with the shift, and the whole-line variant has no register to keep it in; the others are
    // no faster without it: tiles of 16 x 16 of 1024 images of 256 x 256 509 and 511 us)
    return (next_word - (kLine ? 0u : first_word)) >> 7;
}

// --------------------------------------------------------------------------------------------
// One-pass encode: the workgroup that has coded a group of lanes also places them in the
// container.  It needs the bytes of all lanes before the group, which it gets by looking back over
// the descriptors of the groups before it (a group's bytes are published as soon as they are
// known, and the bytes of everything up to and including the group once its workgroup has looked
// back).  Groups are handed out by a ticket counter, so every group with a smaller number has been
// taken by a workgroup that is running, and no workgroup ever waits for a larger number: the
// smallest unfinished group never waits at all.  A workgroup codes its next group before it looks
// back for the one it has just coded, so the groups before that one have usually been coded by
// then and the wait is short; the placing (memory) of one group overlaps the coding (arithmetic)
// of others on the same compute unit.  The wait is bounded all the same: a workgroup that sees an
// empty descriptor for longer than `wait_ticks` of the constant-rate clock raises ST_TIMEOUT, marks
// its own descriptor as abandoned and leaves, and every workgroup that meets an abandoned
// descriptor does the same, so the grid drains.
// --------------------------------------------------------------------------------------------
struct OnePass {
    unsigned long long *desc;  // [groups], zero before the launch; null: two-pass encode
    uint32_t *ticket;          // zero before the launch
    Status *status;
    uint8_t *coded;            // the container: header, offset table, payload
    unsigned long long payload_capacity;  // bytes the payload may take
    unsigned long long wait_ticks;
    uint32_t groups;           // groups of blockDim.x lanes
    uint32_t withhold_first;   // tests of the give-up path: group 0 publishes nothing
    HeaderWords head;
};
constexpr unsigned long long kDescOwn = 1ull, kDescUpTo = 2ull, kDescAbandoned = 3ull;
constexpr int kTailRows = 32;  // word numbers a wavefront moves through its LDS tile at a time

__device__ __forceinline__ void desc_publish(const OnePass &op, uint32_t group, unsigned long long v,
                                             unsigned long long flag)
{
    __hip_atomic_store(&op.desc[group], (v << 2) | flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bytes of the workgroup's lanes before this thread's lane; *total = bytes of all its lanes.
// Ends with a barrier (after which every word the workgroup's lanes stored is visible to it).
__device__ __forceinline__ unsigned long long group_bytes_before(uint32_t t, unsigned long long bytes,
                                                                 unsigned long long *total)
{
    __shared__ unsigned long long s_wave_sum[kLaneMaxThreads / 64];
    const uint32_t wl = t & 63u, wv = t >> 6, nwaves = blockDim.x >> 6;
    unsigned long long inc = bytes;
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long o = __shfl_up(inc, d, 64);
        if (wl >= (uint32_t)d) inc += o;
    }
    __syncthreads();  // the previous use of s_wave_sum is over
    if (wl == 63u) s_wave_sum[wv] = inc;
    __syncthreads();
    unsigned long long before = 0, all = 0;
    for (uint32_t i = 0; i < nwaves; ++i) {
        if (i < wv) before += s_wave_sum[i];
        all += s_wave_sum[i];
    }
    *total = all;
    return before + inc - bytes;
}

// Looks back for group `group` (its own bytes: `total`), then every wavefront places its 64
// lanes.  Returns false if the workgroup has to leave (abandoned wait).
__device__ __forceinline__ bool place_group(const OnePass &op, const Geo &g, uint32_t t, uint32_t group,
                                            unsigned long long total, unsigned long long before,
                                            uint32_t nwords, uint32_t S, uint32_t lane_cap,
                                            const uint16_t *__restrict__ scratch)
{
    __shared__ unsigned long long s_base;
    __shared__ int s_abandon;
    __shared__ __align__(4) uint16_t s_tile[kLaneMaxThreads / 64][kTailRows * kPackTileStride];
    const uint32_t wl = t & 63u, wv = t >> 6;
    const uint32_t lane = group * blockDim.x + t;
    const bool active = lane < g.lanes;

    if (wv == 0u) {
        unsigned long long running = 0;
        int abandon = 0;
        if (group != 0u) {
            long long pos = (long long)group;  // descriptors below pos are still to be added
            const unsigned long long t0 = wall_clock64();
            for (;;) {
                const long long idx = pos - 1 - (long long)wl;
                const unsigned long long d =
                    idx >= 0 ? __hip_atomic_load(&op.desc[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                             : kDescUpTo;  // before the first group: nothing, and final
                const unsigned long long f = d & 3ull;
                const unsigned long long m_upto = __ballot(f == kDescUpTo);
                // the descriptors that matter: from the nearest one back to the first final sum
                const unsigned long long need =
                    m_upto ? ((2ull << (__ffsll((long long)m_upto) - 1)) - 1ull) : ~0ull;
                if (__ballot(f == kDescAbandoned) & need) {
                    abandon = 1;
                    break;
                }
                if (__ballot(f == 0ull) & need) {
                    if (wall_clock64() - t0 > op.wait_ticks) {
                        abandon = 2;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(4);
                    continue;
                }
                unsigned long long v = ((need >> wl) & 1ull) ? d >> 2 : 0ull;
                for (int dd = 32; dd >= 1; dd >>= 1) v += __shfl_xor(v, dd, 64);
                running += v;
                if (m_upto) break;
                pos -= 64;
            }
            if (wl == 0u) {
                if (abandon) {
                    desc_publish(op, group, 0ull, kDescAbandoned);
                    if (abandon == 2) atomicMax(&op.status->code, (int)ST_TIMEOUT);
                } else {
                    desc_publish(op, group, running + total, kDescUpTo);
                }
            }
        }
        if (wl == 0u) {
            s_base = running;
            s_abandon = abandon;
        }
    }
    __syncthreads();
    const unsigned long long base = s_base, upto = base + total;
    const bool leave = s_abandon != 0;
    __syncthreads();  // s_base and s_abandon may be written again
    if (leave) return false;
    uint32_t *offsets = reinterpret_cast<uint32_t *>(op.coded + kHeaderBytes);
    uint16_t *payload = reinterpret_cast<uint16_t *>(op.coded + kHeaderBytes + 4ull * ((size_t)g.lanes + 1ull));
    if (group + 1u == op.groups && t == 0u) {
        // the last group knows the size of the payload: header and closing offset
        uint32_t *h = reinterpret_cast<uint32_t *>(op.coded);
        for (int i = 0; i < 12; ++i) h[i] = op.head.w[i];
        h[12] = (uint32_t)upto;
        h[13] = (uint32_t)(upto >> 32);
        h[14] = 0u;
        h[15] = 0u;
        offsets[g.lanes] = (uint32_t)upto;
        op.status->payload_bytes = upto;
    }
    if (upto >= (1ull << 32) || upto > op.payload_capacity) {
        // this group's lanes do not fit: nothing of them is written (the groups before it that did
        // fit have been written inside the capacity); later groups will find the same
        if (t == 0u) atomicMax(&op.status->code, upto >= (1ull << 32) ? (int)ST_TOO_LARGE : (int)ST_CAPACITY);
        return true;
    }

    // From here on a wavefront meets no other: the words of its 64 lanes are rows of 64 in the
    // scratch ([word number][thread]); 32 rows at a time go through an LDS tile and leave as runs
    // of 32 consecutive words of a lane, two lanes per instruction.
    const uint32_t first = (uint32_t)((base + before) >> 1);  // payload word index of the lane's state
    if (active) {
        offsets[lane] = (uint32_t)(base + before);
        payload[first] = (uint16_t)S;
        payload[first + 1u] = (uint16_t)(S >> 16);
    }
    const uint32_t my_nw = active ? nwords : 0u;
    uint32_t max_nw = my_nw;
    for (int dd = 32; dd >= 1; dd >>= 1) max_nw = max(max_nw, (uint32_t)__shfl_xor((int)max_nw, dd, 64));
    const uint16_t *rows = scratch + (size_t)(lane - wl) * lane_cap;
    uint16_t *tile = s_tile[wv];
    const uint32_t half = wl >> 5, u = wl & 31u;
    for (uint32_t k0 = 0; k0 < max_nw; k0 += kTailRows) {
        wave_lds_sync();
        // two rows an instruction, a dword (two lanes) a thread; all rows of the turn are asked for
        // before the first is stored (guarded one by one, every load would wait for the one before);
        // rows past the last one repeat it and are never read
        uint32_t v[kTailRows / 2];
#pragma unroll
        for (int j = 0; j < kTailRows / 2; ++j)
            v[j] = *reinterpret_cast<const uint32_t *>(rows + (size_t)min(k0 + 2u * j + half, max_nw - 1u) * 64u + 2u * u);
#pragma unroll
        for (int j = 0; j < kTailRows / 2; ++j)
            *reinterpret_cast<uint32_t *>(&tile[(2u * j + half) * kPackTileStride + 2u * u]) = v[j];
        wave_lds_sync();
#pragma unroll 4
        for (int j = 0; j < 32; ++j) {  // lanes 2 j and 2 j + 1; thread u of a half has word numbers k0 + u, + 32, ...
            const uint32_t i = 2u * j + half;
            const uint32_t nw_i = (uint32_t)__shfl((int)my_nw, (int)i, 64);
            const uint32_t first_i = (uint32_t)__shfl((int)first, (int)i, 64);
#pragma unroll
            for (uint32_t part = 0; part < (uint32_t)kTailRows; part += 32u) {
                const uint32_t k = k0 + part + u;
                if (k < nw_i) payload[first_i + 2u + (nw_i - 1u - k)] = tile[(part + u) * kPackTileStride + i];
            }
        }
    }
    return true;
}

// kOnePass: the kernel also places the lanes in the container (`op`); otherwise it leaves word
// counts and states for the scan and pack kernels.  (Three wavefronts per SIMD are asked for: the
// one-pass whole-line variant would otherwise settle at 175 registers, two wavefronts.)
template <bool kOnePass, bool kVec, bool kPair, bool kLine = false>
__global__ __launch_bounds__(kLaneMaxThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_encode_lanes(Geo g, const uint8_t *__restrict__ img,
                               const uint16_t *__restrict__ mu, const int16_t *__restrict__ ls,
                               const int16_t *__restrict__ coef, uint16_t *__restrict__ scratch,
                               uint32_t lane_cap, uint32_t *__restrict__ lane_words,
                               uint32_t *__restrict__ lane_state, OnePass op)
{
    __shared__ LdsTables tab;
    load_tables(tab);  // ends with a barrier
    if (!kOnePass) {
        if (blockIdx.x == 0u && threadIdx.x == 0u) init_status(op.status);  // (for the kernels that follow)
        const uint32_t lane = blockIdx.x * blockDim.x + threadIdx.x;
        if (lane >= g.lanes) return;
        uint32_t S;
        const uint32_t nwords = encode_lane<kVec, kPair, kLine>(g, lane, img, mu, ls, coef, scratch, lane_cap, tab, S);
        lane_words[lane] = nwords;
        lane_state[lane] = S;
        return;
    }
    // what the group coded last still needs: kept in LDS while the next group is coded
    __shared__ uint32_t s_ticket;
    __shared__ uint32_t s_words[kLaneMaxThreads], s_state[kLaneMaxThreads];
    __shared__ unsigned long long s_before[kLaneMaxThreads];
    bool have = false;
    uint32_t last_group = 0u;
    unsigned long long last_total = 0ull;
    for (;;) {
        // the thread index afresh in every round: nothing derived from it (LDS addresses of the
        // arrays below, wavefront numbers) is to be carried in registers through the coding
        uint32_t t = threadIdx.x;
        asm volatile("" : "+v"(t));
        if (t == 0u) s_ticket = atomicAdd(op.ticket, 1u);
        __syncthreads();
        const uint32_t group = s_ticket;
        if (group < op.groups) {
            const uint32_t lane = group * blockDim.x + t;
            uint32_t nwords = 0u, S = 0u;
            if (lane < g.lanes)
                nwords = encode_lane<kVec, kPair, kLine>(g, lane, img, mu, ls, coef, scratch, lane_cap, tab, S);
            t = threadIdx.x;
            asm volatile("" : "+v"(t));  // (as above: what follows starts from the thread index again)
            unsigned long long total;
            const bool coded = group * blockDim.x + t < g.lanes;
            const unsigned long long before = group_bytes_before(t, coded ? 4ull + 2ull * nwords : 0ull, &total);
            if (t == 0u && !(group == 0u && op.withhold_first))
                desc_publish(op, group, total, group == 0u ? kDescUpTo : kDescOwn);
            if (have && !place_group(op, g, t, last_group, last_total, s_before[t], s_words[t], s_state[t],
                                     lane_cap, scratch))
                return;
            s_words[t] = nwords;  // a thread reads back only what it wrote itself
            s_state[t] = S;
            s_before[t] = before;
            last_group = group;
            last_total = total;
            have = true;
        } else {
            if (have) place_group(op, g, t, last_group, last_total, s_before[t], s_words[t], s_state[t], lane_cap, scratch);
            return;
        }
    }
}

// --------------------------------------------------------------------------------------------
// Decode.  The symbol (App. A names a binary search for it) is guessed from the inverse of the law (guide_edge) and checked
// at two or three edges of the exact C (kOneSide); from a guess that is not good enough the lanes concerned walk on edge by edge
// (walk_to_symbol), which wide laws at a low precision take.  Bound by vector instructions where the lanes fill
// the chip, by the length of a symbol's chain where they do not; the guess and three edges, whose
// table reads are under way together, have two waits for LDS, with two edges three, in place of the eight
// of eight steps of bisection (104 instructions without the rest of a symbol; with it 94 and 85 now): 30 frames of 1080 x 1920 in tiles
// of 16 x 16 809 -> 515 us, 16,384 images of 64 x 64 with a lane a row 805 -> 603, 256 lanes of 16,384 pixels 25.1 -> 14.1 ms.
// --------------------------------------------------------------------------------------------

// A lane's 16-bit words, fetched as aligned 32-byte pairs of 16-byte pieces, a piece ahead of
// their use: a refill of the state (App. A eq. (12)) never waits for memory, and a 128-byte line
// of the stream is asked for four times instead of once per word.  A piece is loaded only if it
// starts below `lim`, the end of the container: it then holds at least one byte of it and cannot
// leave the container's last page.  Words beyond the lane's own end are whatever follows; a lane
// that takes them fails its final check of the number of words taken.
struct WordStream {
    uint32_t w0, w1, w2, w3;  // the words not yet taken from the current piece, lowest first
    uint4 x, y;               // the piece after the current one; the piece after that when the
                              // current one is the second of its pair
    uint32_t next;            // word offset from `base` of the next pair to load
    uint32_t count;           // words of the current pair skipped or taken, plus 16 per pair done:
                              // bits 0..2 count within a piece, bit 3 tells the piece of the pair

    // the 8 words at word offset `off` of the 32-byte aligned `base`, if they start below `lim`
    __device__ __forceinline__ static uint4 fetch(const uint16_t *base, uint32_t off, uint32_t lim)
    {
        return off < lim ? *reinterpret_cast<const uint4 *>(base + off) : make_uint4(0u, 0u, 0u, 0u);
    }
    // the lane's first word is at word offset `first` < lim
    __device__ __forceinline__ void open(const uint16_t *base, uint32_t first, uint32_t lim)
    {
        const uint32_t q = first & ~7u;
        const uint4 c = fetch(base, q, lim);
        x = fetch(base, q + 8u, lim);
        y = make_uint4(0u, 0u, 0u, 0u);
        if ((first & 8u) != 0u) y = fetch(base, q + 16u, lim);  // second piece: x, y are the next pair
        next = (first & ~15u) + 16u + (first & 8u) * 2u;
        const uint32_t skip = first & 7u;  // words of the first piece before `first`
        unsigned long long lo = (unsigned long long)c.x | ((unsigned long long)c.y << 32);
        unsigned long long hi = (unsigned long long)c.z | ((unsigned long long)c.w << 32);
        if (skip >= 4u) {
            lo = hi >> (16u * (skip - 4u));
            hi = 0ull;
        } else if (skip != 0u) {
            lo = (lo >> (16u * skip)) | (hi << (64u - 16u * skip));
            hi >>= 16u * skip;
        }
        w0 = (uint32_t)lo; w1 = (uint32_t)(lo >> 32); w2 = (uint32_t)hi; w3 = (uint32_t)(hi >> 32);
        count = first & 15u;
    }
    __device__ __forceinline__ uint32_t take(const uint16_t *base, uint32_t lim)
    {
        const uint32_t wd = w0 & 0xFFFFu;
        w0 = __builtin_amdgcn_alignbit(w1, w0, 16);
        w1 = __builtin_amdgcn_alignbit(w2, w1, 16);
        w2 = __builtin_amdgcn_alignbit(w3, w2, 16);
        w3 >>= 16;
        if ((++count & 7u) == 0u) {
            w0 = x.x; w1 = x.y; w2 = x.z; w3 = x.w;
            if ((count & 8u) != 0u) {  // now in the second piece of a pair: fetch the next pair
                x = fetch(base, next, lim);
                y = fetch(base, next + 8u, lim);
                next += 16u;
            } else {
                x = y;
            }
        }
        return wd;
    }
    // words taken by a stream opened at word offset `first`
    __device__ __forceinline__ uint32_t taken(uint32_t first) const { return count - (first & 15u); }
};

// The same stream for a decoder that works in chunks of at most kRingChunk symbols: the words wait
// in a ring of 32 per thread in LDS.  Before a chunk the ring is looked at: while it still holds 24
// words or more (what a chunk can take) nothing happens, otherwise it is filled to the brim with
// aligned 16-byte loads, one to four at once, together with the chunk's parameter loads.  No refill
// inside the chunk ever touches memory or branches on the fill level.  A thread's 32 words lie side
// by side (rows of 17 dwords, so that the threads of a wavefront start in different banks): the word at
// stream position pos is one 16-bit read at (pos mod 32), fetched ahead of its use.
// The size is what lets four workgroups of 256 threads share a compute unit (160 KB: 22 KB of tables
// and 17 KB of rings each).  With 64 words a line of the stream is asked for half as often, but only
// three workgroups fit, which do not fill the issue slots (30 frames of 1080 x 1920 in tiles, with a
// search by bisection: 0.96 against 0.87 ms).
constexpr int kRingChunk = 24;
constexpr int kRingPieces = 4;                      // 16-byte pieces per thread: 32 words
constexpr int kRingWordsHeld = 8 * kRingPieces;
constexpr int kRingRow = kRingWordsHeld + 2;        // 16-bit elements per thread, padding included
static_assert(3 * kChunk <= kRingChunk, "a chunk must not take more words than the ring guarantees");

struct WordRing {
    typedef uint32_t __attribute__((may_alias)) word_pair;  // two ring words stored at once
    uint16_t *row;      // this thread's words
    uint32_t pos;       // word offset (from the 16-byte aligned `base`) of the next word
    uint32_t filled;    // word offset up to which the ring holds the stream: a multiple of 8
    uint32_t nextw;     // the word at `pos`

    __device__ __forceinline__ static uint4 fetch(const uint16_t *base, uint32_t off, uint32_t lim)
    {
        return off < lim ? *reinterpret_cast<const uint4 *>(base + off) : make_uint4(0u, 0u, 0u, 0u);
    }
    __device__ __forceinline__ uint32_t peek() const { return row[pos & (kRingWordsHeld - 1)]; }
    // Brings `filled` to (pos rounded down to 8) + 32 if a chunk could take more words than are held.
    __device__ __forceinline__ void fill(const uint16_t *base, uint32_t lim)
    {
        if ((int)(filled - pos) < kRingChunk) {  // signed: at the opening `filled` may lie below `pos`
            const uint32_t want = (pos & ~7u) + kRingWordsHeld;
            const uint32_t n = (want - filled) >> 3;  // 1..4
            uint4 piece[kRingPieces];
#pragma unroll
            for (int i = 0; i < kRingPieces; ++i)
                if ((uint32_t)i < n) piece[i] = fetch(base, filled + 8u * i, lim);
#pragma unroll
            for (int i = 0; i < kRingPieces; ++i)
                if ((uint32_t)i < n) {
                    word_pair *d = reinterpret_cast<word_pair *>(row + ((filled + 8u * i) & (kRingWordsHeld - 1)));
                    d[0] = piece[i].x; d[1] = piece[i].y; d[2] = piece[i].z; d[3] = piece[i].w;
                }
            filled = want;
        }
        nextw = peek();
    }
    // the lane's first word is at word offset `first` < lim
    __device__ __forceinline__ void open(uint16_t *ring, const uint16_t *base, uint32_t first, uint32_t lim)
    {
        row = ring + threadIdx.x * kRingRow;
        pos = first;
        filled = first & ~7u;
        fill(base, lim);
    }
    __device__ __forceinline__ uint32_t take()
    {
        const uint32_t wd = nextw;
        ++pos;
        nextw = peek();  // (after the last word held, which only a whole chunk takes: not yet the next one, but `fill` reads it again)
        return wd;
    }
};

// On from one of the two symbols that meet at edge `mid` to the one that holds `slot`, which is neither: an edge a step.
// `below`, `mass`: of the symbol begun with and then of the one returned, the slots of its own below this one (negative
// where the symbol is further down) and its mass; position(k): of edge k.  Nearly always one step; two or three are
// rare while the mean is within the values of a pixel.  8 frames of 1080 x 1920 in tiles, by log-scale, us, against a search by
// bisection for every symbol and one behind each guess that missed: 2^M = 1024: 3.4 326, 462, 579; 4.0 384, 461, 712; 4.6
// 376, 460, 692; 5.5 370, 455, 586; 2^M = 4096: 4.0 312, 460, 480; guesses that are all good 281.  (Slower than
// the search alone only where nothing is known of a pixel: scales of 150 and more with means hundreds away from
// every value, 545 against 463.)
template <class Position>
__device__ __forceinline__ uint32_t walk_to_symbol(uint32_t mid, uint32_t &below, uint32_t &mass, uint32_t slot, uint32_t scale,
                                                   uint32_t m_bits, const LdsTables &tab, Position position)
{
    const bool down = (int)below < 0;
    uint32_t k = down ? mid - 1u : mid + 1u;  // the edge that was looked at last
    uint32_t c_near = slot - below + (down ? 0u : mass);
    do {
        k = down ? k - 1u : k + 1u;  // within 0 .. 256: C(0) = 0 <= slot < 2^M = C(256)
        uint32_t c = cum_inner((int)k, position(k), scale, tab);
        c = k == 0u ? 0u : c;
        c = k == 256u ? 1u << m_bits : c;
        below = slot - (down ? c : c_near);
        mass = down ? c_near - c : c - c_near;
        c_near = c;
    } while (below >= mass);
    return down ? k : k - 1u;
}

// (Four wavefronts per SIMD are asked for, which keep the vector ALUs busy where the lanes fill the chip.  A variant
// that carries the rest of every parameter line in registers, as the encoder does, reads half the
// bytes from memory but needs 172 registers, i.e. two wavefronts per SIMD, and was slower: 0.91 against
// 0.86 ms on 16,384 images of 64 x 64.)
// kOneSide: after C at the guessed edge only the neighbour on the symbol's side is evaluated, behind a wait of its own: ten
// instructions and a table read a symbol less, with the rest of it 85 instructions for 94.  For more than a wavefront a SIMD, where
// instructions are what is waited for: 30 frames of 1080 x 1920 in tiles of 16 x 16 549 and 511 us, 8 images of 1365 x 2047 in
// the same (88,064 lanes) 370 and 363, 16,384 images of 64 x 64 in tiles of 8 x 8 518 and 485, with a lane a row 616
// and 597, 76,800 lanes of 64 109 and 106; up to there the wait is what counts: 65,472 lanes of 64 103 and 105, 38,400 95 and
// 97, 65,536 tiles of 16 x 16 at 2^M = 1024 272 and 279.  Long rows that do not align wait for memory as much, also with
// two wavefronts a SIMD: flat lanes of 100 67,000 165 and 163, 131,000 193 and 197, 139,000 214 and 207, 262,000 348 and 349;
// of 250 80,000 442 and 447, 131,000 503 and 508, 139,000 585 and 585; of 500 67,000 822 and 830; tiles of 8 x 61 115,000 960
// and 970; short ones do not: tiles of 24 x 24 67,000 851 and 847, of 7 x 13 154 and 152, of 10 x 10 197 and 192.
template <bool kVec, bool kPair, bool kOneSide>
__global__ __launch_bounds__(kLaneMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_decode_lanes(Geo g, const uint8_t *__restrict__ coded,
                               unsigned long long coded_bytes, const uint16_t *__restrict__ mu,
                               const int16_t *__restrict__ ls, const int16_t *__restrict__ coef,
                               uint8_t *__restrict__ out, Report *__restrict__ report)
{
    __shared__ int s_state;
    __shared__ unsigned long long s_payload;
    if (threadIdx.x == 0u) s_state = check_header(g, kMagicPilc, 0u, coded, coded_bytes, &s_payload);
    __shared__ LdsTables tab;
    __shared__ float2 guide[kGuideEntries];
    extern __shared__ __align__(16) uint16_t ring[];  // [thread][word]: kRingRow elements a thread
    for (int i = threadIdx.x; i < kGuideEntries; i += blockDim.x) guide[i] = g_guide[i];
    load_tables(tab);  // ends with a barrier
    const GuideScale gs(g.prec_bits);
    if (s_state != ST_OK) {
        if (blockIdx.x == 0u && threadIdx.x == 0u) raise_code(report, s_state);
        return;
    }
    const uint32_t lane = blockIdx.x * blockDim.x + threadIdx.x;
    if (lane >= g.lanes) return;
    const LaneShape sh = lane_shape(g, lane);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), mask = (1u << m_bits) - 1u;
    uint32_t top = 1u << m_bits;
    asm("" : "+v"(top));  // (in a vector register, where the choice below takes it from)
    const uint32_t payload_bytes = (uint32_t)s_payload;
    const uint32_t per_row = (sh.tw + kChunk - 1) / kChunk;
    const uint32_t chunks = per_row * (sh.npx / sh.tw);

    const uint32_t *offsets = reinterpret_cast<const uint32_t *>(coded + 64);
    const uint16_t *payload =
        reinterpret_cast<const uint16_t *>(coded + 64 + 4ull * ((size_t)g.lanes + 1));
    const uint32_t begin = offsets[lane], end = offsets[lane + 1];
    if (end < begin || end > payload_bytes || end - begin < 4u || ((begin | end) & 1u)) {
        raise_code(report, ST_CORRUPT);
        return;
    }
    // word offsets from the last 16-byte boundary at or below the payload (the payload is < 4 GiB)
    const uint32_t adj = (uint32_t)(reinterpret_cast<uintptr_t>(payload) & 15u);
    const uint16_t *base = reinterpret_cast<const uint16_t *>(reinterpret_cast<const uint8_t *>(payload) - adj);
    const uint32_t first = (adj + begin) >> 1;
    const uint32_t lim = (uint32_t)(((unsigned long long)adj + payload_bytes + 1ull) >> 1);
    WordRing words;
    words.open(ring, base, first, lim);
    uint32_t S = words.take();
    S |= words.take() << 16;

    // decodes the chunk into its 24 bytes (6 dwords)
    // tiles and flat lanes no longer than an image lie in one image: its coefficients are loaded once
    auto decode_chunk = [&](const Chunk &ck, const ChunkPos cp, uint32_t *wout) {
        uint32_t im = g.by_hw.div(cp.p);
        int a_gr = coef[3 * im], a_br = coef[3 * im + 1], a_bg = coef[3 * im + 2];
#pragma unroll
        for (int b = 0; b < 6; ++b) wout[b] = 0u;
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
            if ((uint32_t)i < cp.len) {
                if (!kVec) {
                    const uint32_t im_i = g.by_hw.div(cp.p + i);
                    if (im_i != im) {
                        im = im_i;
                        a_gr = coef[3 * im]; a_br = coef[3 * im + 1]; a_bg = coef[3 * im + 2];
                    }
                }
                int x[3] = {0, 0, 0};
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) {
                    int me = ck.m[i][0];
                    if (ch == 1) me = ck.m[i][1] + rsh14_mul(a_gr, (x[0] * 256 - ck.m[i][0]));
                    if (ch == 2)
                        me = ck.m[i][2] + rsh14_mul(a_br, (x[0] * 256 - ck.m[i][0])) +
                             rsh14_mul(a_bg, (x[1] * 256 - ck.m[i][1]));
                    const uint32_t inv_s = inv_scale(ck.l[i][ch], tab);
                    const uint32_t slot = S & mask;
                    // C at the edge where the symbol should begin or end, and at the one that it should have on the other
                    // side, or at both neighbours
                    uint32_t lo, below, mass;
                    if (kOneSide) {
                        const uint32_t mid = guide_edge<false>(slot, me, inv_s, 0, gs, guide);
                        int from_mean = -128 - me;
                        asm("" : "+v"(from_mean));  // (formed before the guess is there)
                        const EdgeStep edge((int)(mid << 8) + from_mean, inv_s);
                        const uint32_t c_mid = cum_inner((int)mid, edge.y, scale, tab);
                        const bool down = slot < c_mid;
                        const uint32_t other = mid + (down ? 0u - 1u : 1u);
                        uint32_t c = cum_inner((int)other, __builtin_fma(down ? -256.0 : 256.0, edge.unit, edge.y), scale, tab);
                        asm("" : "+v"(c));  // (no branch around its evaluation)
                        c = other == 0u ? 0u : c;
                        c = other == 256u ? top : c;
                        lo = min(mid, other);
                        const uint32_t c_lo = min(c_mid, c);
                        below = slot - c_lo;
                        mass = max(c_mid, c) - c_lo;
                        if (__builtin_expect(__any(below >= mass), 0)) {
                            if (below >= mass)
                                lo = walk_to_symbol(mid, below, mass, slot, scale, m_bits, tab, [&](uint32_t k) {
                                    return __builtin_fma((double)(int)(k - mid), 256.0 * edge.unit, edge.y);
                                });
                        }
                    } else {
                        const EdgeLaw law = edge_law(me, inv_s);
                        uint32_t mid = guide_edge<true>(slot, me, inv_s, scale_index(ck.l[i][ch]), gs, guide);
                        const double y = edge_y((int)mid, law);
                        const uint32_t c_mid = cum_inner((int)mid, y, scale, tab);
                        uint32_t c_below = cum_inner((int)mid - 1, y - law.a, scale, tab);
                        uint32_t c_above = cum_inner((int)mid + 1, y + law.a, scale, tab);
                        c_below = mid == 1u ? 0u : c_below;
                        c_above = mid == 255u ? top : c_above;
                        bool up = c_mid <= slot;
                        const uint32_t c_lo = up ? c_mid : c_below;
                        below = slot - c_lo;
                        mass = (up ? c_above : c_mid) - c_lo;
                        if (__builtin_expect(__any(below >= mass), 0)) {
                            if (below >= mass) {
                                mid = walk_to_symbol(mid, below, mass, slot, scale, m_bits, tab, [&](uint32_t k) { return edge_y((int)k, law); });
                                up = true;
                            }
                        }
                        lo = up ? mid : mid - 1u;
                    }
                    x[ch] = (int)lo;
                    // App. A eq. (12)
                    // the mass is at most 2^16 and S >> M below 2^22: a 24-bit multiply is exact
                    S = (uint32_t)__umul24(mass, S >> m_bits) + below;
                    if (S < (1u << 16)) S = (S << 16) | words.take();
                    const int b = 3 * i + ch;
                    wout[b >> 2] |= lo << (8 * (b & 3));
                }
            }
        }
    };

    if (kVec && kPair) {
        // two neighbouring chunks per round: 96 bytes of each parameter array in, 48 bytes out
        for (uint32_t c = 0; c + 2u <= chunks; c += 2u) {
            const ChunkPos left = chunk_pos(g, sh, per_row, c);
            ChunkPair raw;
            load_pair<false>(raw, left.p, nullptr, mu, ls);
            uint32_t wout[12];
            auto half = [&](auto h) {  // h: which chunk of the pair, as a compile-time constant
                constexpr int kH = decltype(h)::value;
                words.fill(base, lim);
                Chunk ck;
                unpack_chunk<false>(ck, nullptr, raw.wm + 12 * kH, raw.wl + 12 * kH);
                ChunkPos cp;
                cp.p = left.p + (uint32_t)(kChunk * kH);
                cp.len = (uint32_t)kChunk;
                decode_chunk(ck, cp, wout + 6 * kH);
            };
            half(std::integral_constant<int, 0>{});
            half(std::integral_constant<int, 1>{});
            uint4 *po = reinterpret_cast<uint4 *>(out + (size_t)left.p * 3);
            po[0] = make_uint4(wout[0], wout[1], wout[2], wout[3]);
            po[1] = make_uint4(wout[4], wout[5], wout[6], wout[7]);
            po[2] = make_uint4(wout[8], wout[9], wout[10], wout[11]);
        }
    } else {
        for (uint32_t c = 0; c < chunks; ++c) {
            const ChunkPos cp = chunk_pos(g, sh, per_row, c);
            Chunk ck;
            load_chunk<kVec, false>(ck, cp.p, cp.len, g.total_px, nullptr, mu, ls);
            words.fill(base, lim);  // its loads travel with the chunk's
            uint32_t wout[6];
            decode_chunk(ck, cp, wout);
            const size_t s = (size_t)cp.p * 3;
            if (kVec && cp.len == (uint32_t)kChunk) {
                uint2 *po = reinterpret_cast<uint2 *>(out + s);
                po[0] = make_uint2(wout[0], wout[1]);
                po[1] = make_uint2(wout[2], wout[3]);
                po[2] = make_uint2(wout[4], wout[5]);
            } else if (!kVec && cp.len == (uint32_t)kChunk) {
                __builtin_memcpy(out + s, wout, 24);
            } else {
#pragma unroll
                for (int b = 0; b < 3 * kChunk; ++b)
                    if ((uint32_t)b < 3u * cp.len) out[s + b] = (uint8_t)(wout[b >> 2] >> (8 * (b & 3)));
            }
        }
    }
    if (S != (1u << 16) || words.pos - first != (end - begin) >> 1) raise_code(report, ST_CORRUPT);
}

}  // namespace pilc
