// rANS lanes under a mixture of K logistic laws per subpixel (gfx950): an encoder whose evaluations are shared out by
// pixels (k_mix_encode_chunks), a decoder of many lanes with a thread per lane (k_mix_decode) and one of few with a row of
// 16 threads per lane (k_mix_decode_rows).  The first two want arrays on 4-byte boundaries and are built for every
// component count K; arrays that are not there go a thread per lane through general kernels (k_mix_encode, k_mix_decode<0>).
//
// Sec. 2 of arXiv 2206.05279 names this workload (a dynamic rANS coder fed a mixture of ten
// logistic laws per symbol) as what holds earlier learned codecs near 1 MB/s; the coder itself is
// App. A eqs. (11)-(12).  A pixel has K weights (Q0.15, summing to 2^15), a subpixel K means and
// K log-scales.  The mixed 24-bit edge CDF is F(k) = floor(sum_j w_j F_j(k) / 2^15) with F_j the
// single-law edge CDF, and C(k) = k + floor(F(k) (2^M - 256) / 2^24); the channel conditioning
// of Sec. 3.1 eqs. (3)-(4) shifts every component's mean with that component's own innovations.
//
// In the general kernels K is a run-time value, so nothing per component lives in registers.  A thread first copies
// the 7 K 16-bit parameters of a pixel into its own LDS slots in one burst of loads (every
// 128-byte line of the arrays is then asked for by one or two bursts rather than by dozens of
// separate loads spread over the pixel's work), then, before a subpixel is coded, turns the
// channel's components into {shifted mean, 1/scale} pairs in further slots; every evaluation of
// C(k) walks those.  The thread-per-lane decoder built for one K has the raw parameters in such slots, the channel's
// components and the pixel's weights in registers.  All slots are [index][thread] arrays of dwords, so a wavefront's
// accesses are conflict free.  The 16-bit words go through the thread-per-lane scratch layout and packer.
#pragma once

#include "pilc_lane_kernels.hpp"

namespace pilc {

constexpr int kMixMaxComp = 16;
constexpr int kMixThreads = 256;

struct MixArgs {
    const uint16_t *mu;      // [px][3][K]
    const int16_t *ls;       // [px][3][K]
    const uint16_t *weight;  // [px][K]
    const int16_t *coef;     // [n][3]
    uint32_t k;
};

// Dynamic LDS of the mixture kernels: K {mean, 1/scale} pairs per thread as [component][thread]
// 8-byte elements, then per thread the pixel's raw means (3 K halfwords), log-scales (3 K) and
// weights (K), each rounded up to dwords, as [dword][thread].  The kernels built for one K have
// neither the pairs nor the weights there.
constexpr uint32_t kMixImageBlock = 32;  // bytes of the image a thread of the general encoder keeps in LDS

struct MixSlots {
    uint2 *pairs;    // this thread's column of the pairs
    uint32_t *base;  // this thread's column of the raw parameters
    uint32_t k, stride, raw_ls, raw_w, image_block;
    static constexpr uint32_t raw_mu = 0u;
    __device__ __forceinline__ MixSlots(uint32_t *lds, uint32_t k_, bool with_pairs = true)
        : pairs(reinterpret_cast<uint2 *>(lds) + threadIdx.x),
          base(lds + (with_pairs ? 2u * k_ * blockDim.x : 0u) + threadIdx.x), k(k_), stride(blockDim.x),
          raw_ls((3u * k_ + 1u) / 2u), raw_w(2u * ((3u * k_ + 1u) / 2u)),
          image_block(2u * ((3u * k_ + 1u) / 2u) + (k_ + 1u) / 2u)
    {
    }
    __device__ __forceinline__ uint32_t &dword(uint32_t i) const { return base[i * stride]; }
    // halfword e of the array that starts at dword `first`
    __device__ __forceinline__ uint32_t half(uint32_t first, uint32_t e) const
    {
        return reinterpret_cast<const uint16_t *>(&base[(first + (e >> 1)) * stride])[e & 1u];
    }
    __device__ __forceinline__ void set_half(uint32_t first, uint32_t e, uint32_t v) const
    {
        reinterpret_cast<uint16_t *>(&base[(first + (e >> 1)) * stride])[e & 1u] = (uint16_t)v;
    }
    __device__ __forceinline__ void set_pair(uint32_t j, int me, uint32_t inv_s) const
    {
        pairs[j * stride] = make_uint2((uint32_t)me, inv_s);
    }
};

// with_pairs false: the decoders built for one K, which keep the pairs and the weights in registers.  (The block of
// image bytes is the general encoder's; the general decoder has it too, unused: one layout for both.)
static inline size_t mix_lds_bytes(uint32_t k, bool with_pairs)
{
    return (size_t)kMixThreads * 4u *
           ((with_pairs ? 2u * k + (k + 1u) / 2u + kMixImageBlock / 4u : 0u) + 2u * ((3u * k + 1u) / 2u));
}

// An aligned block of kBytes of global memory in a thread's LDS column ([dword][thread]), loaded
// when an address outside it is asked for.  With the lines long gone from the L2 when a lane
// reaches its next pixel, every separate load costs a fetch of its whole 128-byte line; through a
// block a line is asked for 128 / kBytes times instead of once per pixel.  A block that holds a
// byte of an array lies inside the array's pages even where it reaches past its ends.
template <uint32_t kBytes> struct LdsBlock {
    uint32_t *col;
    uint32_t stride;
    uintptr_t tag;  // address of the block held; 1: none
    __device__ __forceinline__ LdsBlock(uint32_t *column, uint32_t stride_) : col(column), stride(stride_), tag(1u) {}
    __device__ __forceinline__ uint32_t dword(uintptr_t at)  // the aligned dword that holds byte `at`
    {
        const uintptr_t blk = at & ~(uintptr_t)(kBytes - 1u);
        if (blk != tag) {
            const uint4 *src = reinterpret_cast<const uint4 *>(blk);
            uint4 v[kBytes / 16u];
#pragma unroll
            for (uint32_t i = 0; i < kBytes / 16u; ++i) v[i] = src[i];
#pragma unroll
            for (uint32_t i = 0; i < kBytes / 16u; ++i) {
                col[(4u * i) * stride] = v[i].x;
                col[(4u * i + 1u) * stride] = v[i].y;
                col[(4u * i + 2u) * stride] = v[i].z;
                col[(4u * i + 3u) * stride] = v[i].w;
            }
            tag = blk;
        }
        return col[(((uint32_t)at & (kBytes - 1u)) >> 2) * stride];
    }
};

// The encoder's image bytes.
struct PixelBytes {
    LdsBlock<kMixImageBlock> block;
    __device__ __forceinline__ PixelBytes(const MixSlots &s) : block(s.base + s.image_block * s.stride, s.stride) {}
    __device__ __forceinline__ uint32_t byte(const uint8_t *a)
    {
        const uintptr_t at = reinterpret_cast<uintptr_t>(a);
        return (block.dword(at) >> (8u * ((uint32_t)at & 3u))) & 0xFFu;
    }
    // R | G << 8 | B << 16 of pixel q, highest address first: the encoder walks its lane backwards
    __device__ __forceinline__ uint32_t pixel(const uint8_t *img, uint32_t q)
    {
        const uint8_t *a = img + 3 * (size_t)q;
        const uint32_t b = byte(a + 2), g = byte(a + 1), r = byte(a);
        return r | (g << 8) | (b << 16);
    }
};

// The pixel's parameters into the slots of a general kernel; false if its weights do not sum to 2^15.
__device__ __forceinline__ bool mix_load_pixel(const MixArgs &a, uint32_t p, const MixSlots &s)
{
    const size_t px = (size_t)p * 3u * a.k;
    for (uint32_t e = 0; e < 3u * a.k; ++e) s.set_half(s.raw_mu, e, a.mu[px + e]);
    for (uint32_t e = 0; e < 3u * a.k; ++e) s.set_half(s.raw_ls, e, (uint16_t)a.ls[px + e]);
    for (uint32_t e = 0; e < a.k; ++e) s.set_half(s.raw_w, e, a.weight[(size_t)p * a.k + e]);
    uint32_t sum = 0;
    for (uint32_t j = 0; j < a.k; ++j) sum += s.half(s.raw_w, j);
    return sum == (1u << 15);
}

// Dword-aligned arrays: a pixel's raw parameters lie in ceil(3 K / 2) + ceil(3 K / 2) + ceil(K / 2)
// aligned dwords (for odd K the blocks of every other pixel start on the upper half of a dword and
// end on a lower half: the same number of dwords, one halfword of a neighbour at either end), and
// the decoder keeps the NEXT pixel's dwords in registers while it works on the current one, so that
// the loads have a pixel's worth of arithmetic to arrive in.
template <int kK> struct MixAhead {
    static constexpr int kMu = (3 * kK + 1) / 2, kW = (kK + 1) / 2;
    uint32_t m[kMu], l[kMu], w[kW];
};

// The components of the channel being coded, in registers: every index into these arrays is a compile-time constant.
template <int kK> struct MixRegs {
    EdgeLaw law[kK];     // position of an edge under the component
    uint32_t w[kK];      // the pixel's weights
};

template <int kK>
__device__ __forceinline__ void mix_fetch_ahead(const MixArgs &a, uint32_t p, MixAhead<kK> &r)
{
    const size_t px = (size_t)p * (3u * kK);  // in halfwords: the aligned dwords from px / 2 on
    const uint32_t *gm = reinterpret_cast<const uint32_t *>(a.mu) + (px >> 1);
    const uint32_t *gl = reinterpret_cast<const uint32_t *>(a.ls) + (px >> 1);
    const uint32_t *gw = reinterpret_cast<const uint32_t *>(a.weight) + (((size_t)p * kK) >> 1);
#pragma unroll
    for (int i = 0; i < MixAhead<kK>::kMu; ++i) r.m[i] = gm[i];
#pragma unroll
    for (int i = 0; i < MixAhead<kK>::kMu; ++i) r.l[i] = gl[i];
#pragma unroll
    for (int i = 0; i < MixAhead<kK>::kW; ++i) r.w[i] = gw[i];
}

// The fetched pixel into the slots, its weights into `regs`; false if the weights do not sum to 2^15.  `upper`: the
// pixel's blocks start on the upper half of the first dword fetched (odd K, every other pixel) and are moved down
// by a halfword on the way.
template <int kK>
__device__ __forceinline__ bool mix_store_ahead(const MixAhead<kK> &r, const MixSlots &s, MixRegs<kK> &regs,
                                                bool upper)
{
    constexpr bool kOdd = kK % 2 != 0;
    auto lowered = [&](const uint32_t *d, int i, int n) {  // dword i of the block, from the n fetched
        if constexpr (!kOdd) return d[i];
        const uint32_t next = i + 1 < n ? d[i + 1] : 0u;
        return upper ? __builtin_amdgcn_alignbit(next, d[i], 16) : d[i];
    };
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < MixAhead<kK>::kMu; ++i) s.dword(s.raw_mu + i) = lowered(r.m, i, MixAhead<kK>::kMu);
#pragma unroll
    for (int i = 0; i < MixAhead<kK>::kMu; ++i) s.dword(s.raw_ls + i) = lowered(r.l, i, MixAhead<kK>::kMu);
#pragma unroll
    for (int i = 0; i < MixAhead<kK>::kW; ++i) {
        const uint32_t w2 = lowered(r.w, i, MixAhead<kK>::kW);
        regs.w[2 * i] = w2 & 0xFFFFu;
        sum += w2 & 0xFFFFu;
        if (2 * i + 1 < kK) {
            regs.w[2 * i + 1] = w2 >> 16;
            sum += w2 >> 16;
        }
    }
    return sum == (1u << 15);
}

// {shifted mean, 1/scale} of every component of channel `ch` of the loaded pixel into the pair
// slots; x_r and x_g are the pixel's red and green values (used for ch >= 1 and ch == 2).
__device__ __forceinline__ void mix_load_channel(const MixSlots &s, int ch, int x_r, int x_g, int a_gr,
                                                 int a_br, int a_bg, const LdsTables &tab)
{
    for (uint32_t j = 0; j < s.k; ++j) {
        int me = (int)s.half(s.raw_mu, (uint32_t)ch * s.k + j);
        if (ch >= 1) {
            const int e_r = x_r * 256 - (int)s.half(s.raw_mu, j);
            if (ch == 1) {
                me += rsh14_mul(a_gr, e_r);
            } else {
                const int e_g = x_g * 256 - (int)s.half(s.raw_mu, s.k + j);
                me += rsh14_mul(a_br, e_r) + rsh14_mul(a_bg, e_g);
            }
        }
        const int l = (int)(short)s.half(s.raw_ls, (uint32_t)ch * s.k + j);
        s.set_pair(j, me, inv_scale(l, tab));
    }
}

// The same into registers, two components (one dword of each raw array) at a time.
template <int kK>
__device__ __forceinline__ void mix_load_channel(const MixSlots &s, MixRegs<kK> &regs, int ch, int x_r,
                                                 int x_g, int a_gr, int a_br, int a_bg, const LdsTables &tab)
{
    if constexpr (kK % 2 != 0) {  // a channel's block starts on either half of a dword: halfword reads
        // (the scales before the means: the branches on the channel below would part their table reads, and every
        // component would wait for its own; encode of 3000 images of 64 x 64 at K = 13 1912 -> 1748 us)
        uint32_t inv_s[kK];
#pragma unroll
        for (int j = 0; j < kK; ++j) inv_s[j] = inv_scale((int)(short)s.half(s.raw_ls, (uint32_t)ch * kK + j), tab);
#pragma unroll
        for (int j = 0; j < kK; ++j) {
            int me = (int)s.half(s.raw_mu, (uint32_t)ch * kK + j);
            if (ch >= 1) {
                const int e_r = x_r * 256 - (int)s.half(s.raw_mu, j);
                if (ch == 1)
                    me += rsh14_mul(a_gr, e_r);
                else
                    me += rsh14_mul(a_br, e_r) + rsh14_mul(a_bg, x_g * 256 - (int)s.half(s.raw_mu, kK + j));
            }
            regs.law[j] = edge_law(me, inv_s[j]);
        }
        return;
    }
    const uint32_t *mu_r = s.base + s.raw_mu * s.stride;
    const uint32_t *mu_g = mu_r + (kK / 2) * s.stride;
    const uint32_t *mu_c = mu_r + (uint32_t)ch * (kK / 2) * s.stride;
    const uint32_t *ls_c = s.base + (s.raw_ls + (uint32_t)ch * (kK / 2)) * s.stride;
#pragma unroll
    for (int jj = 0; jj < kK / 2; ++jj) {
        const uint32_t m2 = mu_c[jj * s.stride], l2 = ls_c[jj * s.stride];
        int me[2] = {(int)(m2 & 0xFFFFu), (int)(m2 >> 16)};
        if (ch >= 1) {
            const uint32_t r2 = mu_r[jj * s.stride];
            const int e_r[2] = {x_r * 256 - (int)(r2 & 0xFFFFu), x_r * 256 - (int)(r2 >> 16)};
            if (ch == 1) {
                me[0] += rsh14_mul(a_gr, e_r[0]);
                me[1] += rsh14_mul(a_gr, e_r[1]);
            } else {
                const uint32_t g2 = mu_g[jj * s.stride];
                me[0] += rsh14_mul(a_br, e_r[0]) + rsh14_mul(a_bg, x_g * 256 - (int)(g2 & 0xFFFFu));
                me[1] += rsh14_mul(a_br, e_r[1]) + rsh14_mul(a_bg, x_g * 256 - (int)(g2 >> 16));
            }
        }
        regs.law[2 * jj] = edge_law(me[0], inv_scale((int)(short)(l2 & 0xFFFFu), tab));
        regs.law[2 * jj + 1] = edge_law(me[1], inv_scale((int)(short)(l2 >> 16), tab));
    }
}

// C(k), 1 <= k <= 255, from the slots.
__device__ __forceinline__ uint32_t mix_cum_inner(int k, const MixSlots &s, uint32_t scale,
                                                  const LdsTables &tab)
{
    auto term = [&](uint32_t j) -> unsigned long long {
        const uint2 c = s.pairs[j * s.stride];
        return (unsigned long long)s.half(s.raw_w, j) * edge_cdf(256 * k + (-128 - (int)c.x), c.y, tab);
    };
    // four (then two) components per round, so that their table reads are in flight together
    unsigned long long acc = 0ull;
    uint32_t j = 0;
    for (; j + 3u < s.k; j += 4u) {
        const unsigned long long t0 = term(j), t1 = term(j + 1u), t2 = term(j + 2u), t3 = term(j + 3u);
        acc += (t0 + t1) + (t2 + t3);
    }
    if (j + 1u < s.k) {
        const unsigned long long t0 = term(j), t1 = term(j + 1u);
        acc += t0 + t1;
        j += 2u;
    }
    if (j < s.k) acc += term(j);
    return (uint32_t)k + mass_of((uint32_t)(acc >> 15), scale);
}

// C(k), 1 <= k <= 255, from the registers: the table reads of several components are under way together (see mix_waves).
template <int kK>
__device__ __forceinline__ uint32_t mix_cum_inner(int k, const MixRegs<kK> &regs, uint32_t scale,
                                                  const LdsTables &tab)
{
    unsigned long long acc = 0ull;
#pragma unroll
    for (int j = 0; j < kK; ++j)
        acc += (unsigned long long)regs.w[j] * edge_at(edge_y(k, regs.law[j]), tab);
    return (uint32_t)k + mass_of((uint32_t)(acc >> 15), scale);
}

// Most wavefronts on a SIMD of the decoder with a thread a lane.  LDS (the tables and 12 K bytes a thread) has room for five
// workgroups of 256 on a compute unit at K = 4, four at 5 and 6, three from 7 to 11, two from 12 on.  From five to eight components the
// decoder has them all that its registers allow: with two against these, lanes of 64 pixels, us: 160,000 lanes K = 5 1069
// and 807, 6 1068 and 830, 8 1214 and 956; 262,144 lanes 1259 and 1150, 1300 and 1273, 1517 and 1408; 131,072 the same.
// From nine on two: left to itself the compiler saves registers for a third by taking the table reads of an evaluation
// one at a time (131,072 lanes of 42 pixels, K = 9, 650 and 738), and from ten on it takes too many for it anyway.  With four
// components more are in each other's way: 160,000 lanes 860 and, with four, 713, but 262,144 1048 and 1081 (their lines are
// gone from the L2 before the lanes come back).
constexpr int mix_waves(int k) { return k <= 3 ? 8 : k == 5 ? 4 : k >= 6 && k <= 8 ? 3 : 2; }

// The encoder for arrays off the 4-byte grid: any K, components in LDS, a thread per lane.
__global__ __launch_bounds__(kMixThreads) void k_mix_encode(
    Geo g, const uint8_t *__restrict__ img, MixArgs a, uint16_t *__restrict__ scratch,
    uint32_t lane_cap, uint32_t *__restrict__ lane_words, uint32_t *__restrict__ lane_state,
    int *__restrict__ status_code)
{
    __shared__ LdsTables tab;
    extern __shared__ uint32_t mix_lds[];
    load_tables(tab);
    const uint32_t lane = blockIdx.x * blockDim.x + threadIdx.x;
    if (lane >= g.lanes) return;
    const MixSlots slots(mix_lds, a.k, true);
    const LaneShape sh = lane_shape(g, lane);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), top = 1u << m_bits;

    uint16_t *wout = scratch + lane_scratch_base(lane, lane_cap);
    uint32_t nwords = 0, S = 1u << 16;
    bool ok = true;
    // pixels last-first, and B, G, R inside a pixel (App. A eq. (11) runs against the decoder)
    PixelBytes bytes(slots);
    uint32_t im_now = 0xFFFFFFFFu;
    int a_gr = 0, a_br = 0, a_bg = 0;
    for (uint32_t t = sh.npx; t-- > 0u;) {
        const uint32_t p = lane_pixel(g, sh, t);
        const uint32_t im = g.by_hw.div(p);
        if (im != im_now) {
            im_now = im;
            a_gr = a.coef[3 * im]; a_br = a.coef[3 * im + 1]; a_bg = a.coef[3 * im + 2];
        }
        ok = mix_load_pixel(a, p, slots) && ok;
        const uint32_t xb = bytes.pixel(img, p);
        const int x[3] = {(int)(xb & 0xFFu), (int)((xb >> 8) & 0xFFu), (int)(xb >> 16)};
#pragma unroll 1
        for (int ch = 2; ch >= 0; --ch) {
            const int v = ch == 0 ? x[0] : (ch == 1 ? x[1] : x[2]);
            mix_load_channel(slots, ch, x[0], x[1], a_gr, a_br, a_bg, tab);
            const uint32_t lo = v == 0 ? 0u : mix_cum_inner(v, slots, scale, tab);
            const uint32_t hi = v == 255 ? top : mix_cum_inner(v + 1, slots, scale, tab);
            const uint32_t f = hi - lo;
            if (S >= (f << (32u - m_bits))) {
                *wout = (uint16_t)(S & 0xFFFFu);
                wout += 64;
                ++nwords;
                S >>= 16;
            }
            S = (uint32_t)__umul24(quotient(S, over_reciprocal(f)), top - f) + (S + lo);
        }
    }
    if (!ok) atomicMax(status_code, 7);
    lane_words[lane] = nwords;
    lane_state[lane] = S;
}

// --------------------------------------------------------------------------------------------
// The encoder for arrays on 4-byte boundaries, built for each component count.
//
// All an encoder has to evaluate is known beforehand, so the evaluations are shared out by where the parameters lie: a
// wavefront takes 2^log_lanes lanes, and of every lane a chunk of 2^log_chunk pixels at a time, last chunk first.  Its threads
// evaluate the chunk, neighbouring threads neighbouring pixels, and leave {C, mass} of every symbol in LDS; then a thread
// per lane runs the serial chain over them.  A pixel's parameters go straight from memory to the registers of the thread
// that uses them, and those of a chunk are one run of memory, so a line is fetched once or twice instead of once a
// pixel.  (A thread per lane, which comes back for the rest of a line when it has long left the L2, read 2.7 times the
// parameters, at 6.1 TB/s: 2048 images of 64 x 64, ten components, a lane a row, whole call 558 us, now 368, 1.1 times the
// parameters read and 79 % of the issue slots used; and a small batch went a pixel after another: 64 such images 366 us,
// now 91; two photographs of 1365 x 2047 with a lane a row 13.3 ms, now 1.2.)
// The wavefronts share nothing but the tables, so there is no barrier.
// --------------------------------------------------------------------------------------------
// Four wavefronts on a SIMD, in workgroups of eight that share the tables; from twelve components on the registers are those of
// three, in workgroups of four (at four, K = 16 spills 164 bytes a thread: 1024 images of 64 x 64 595 us, now 300; with those of
// two, two photographs of 1365 x 2047 in tiles of 16 x 16 580, now 470).
constexpr int mix_encode_waves(int k) { return k >= 12 ? 3 : 4; }
constexpr int mix_encode_threads(int k) { return k >= 12 ? 256 : 512; }
constexpr uint32_t kMixEncRecords = 512;  // pixels of a wavefront's chunks: most lanes times pixels

struct MixChunk {  // how a launch shares out its lanes: lanes of a wavefront and pixels of a lane at a time
    uint32_t log_lanes, log_chunk;
};

// Pixels a chunk: sixteen where lanes have four chunks and more (a run of 960 bytes with ten components, 1.13 lines fetched for
// one; with eight 425 us for 417), fewer where they would leave threads without a pixel.  Lanes a wavefront: the chain is run by
// a thread a lane and costs 4 / lanes of the evaluations, so 32, unless that leaves less than one and a half wavefronts a
// SIMD; at least so many that every thread has a pixel.  Lines at 1024, 1536, 3072, 4096 wavefronts, us: 32,768 lanes of 64
// pixels 216, 150, 156, 156; 16,384 137, 113, 121, 123; 15,876 tiles 301, 299, 327, 325.
static MixChunk mix_chunk(uint32_t lanes, uint32_t lane_pixels)
{
    MixChunk c;
    c.log_chunk = lane_pixels >= 64u ? 4u : lane_pixels >= 16u ? 3u : lane_pixels >= 4u ? 2u : lane_pixels >= 2u ? 1u : 0u;
    c.log_lanes = 6u - c.log_chunk;
    while (c.log_lanes < 5u && (lanes >> (c.log_lanes + 1u)) >= 1536u) ++c.log_lanes;
    return c;
}

static inline size_t mix_encode_lds_bytes(int k) { return (size_t)(mix_encode_threads(k) / 64) * (kMixEncRecords * 12u + 64u * 16u); }

template <int kK>
__global__ __launch_bounds__(mix_encode_threads(kK)) __attribute__((amdgpu_waves_per_eu(mix_encode_waves(kK)))) void k_mix_encode_chunks(
    Geo g, MixChunk c, const uint8_t *__restrict__ img, MixArgs a, uint16_t *__restrict__ scratch, uint32_t lane_cap,
    uint32_t *__restrict__ lane_words, uint32_t *__restrict__ lane_state, int *__restrict__ status_code)
{
    __shared__ LdsTables tab;
    extern __shared__ uint32_t mix_lds[];
    load_tables(tab);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), t = threadIdx.x & 63u;
    const uint32_t lanes_here = 1u << c.log_lanes, chunk = 1u << c.log_chunk;
    const uint32_t lane0 = (blockIdx.x * (mix_encode_threads(kK) / 64) + wave) << c.log_lanes;
    if (lane0 >= g.lanes) return;
    uint32_t *rec = mix_lds + wave * (kMixEncRecords * 3u + 64u * 4u);  // [symbol of the chunk][lane]: C | mass << 16
    uint4 *shapes = reinterpret_cast<uint4 *>(rec + kMixEncRecords * 3u);
    const uint32_t m_bits = g.prec_bits, scale = mass_scale(m_bits), top = 1u << m_bits;

    // this thread's lane in the chain; the shapes of all lanes for whoever has one of their pixels
    const uint32_t lane = lane0 + t;
    const bool mine = t < lanes_here && lane < g.lanes;
    uint32_t npx = 0u;
    if (mine) {
        const LaneShape sh = lane_shape(g, lane);
        npx = sh.npx;
        shapes[t] = make_uint4(sh.first, sh.npx, sh.tw, 0u);
    } else if (t < lanes_here) {
        shapes[t] = make_uint4(0u, 0u, 1u, 0u);
    }
    wave_lds_sync();
    uint32_t longest = npx;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) longest = max(longest, (uint32_t)__shfl_xor((int)longest, d));
    const uint32_t turns = 1u << (c.log_lanes + c.log_chunk - 6u);

    uint16_t *wout = scratch + lane_scratch_base(lane, lane_cap);
    uint32_t nwords = 0, S = 1u << 16;
    // With sixteen components there are no registers left for what only the chain needs: it lies beside the lane's shape.
    constexpr bool kChainInLds = kK >= 16;
    bool ok = true;
    for (uint32_t q = (longest + chunk - 1u) >> c.log_chunk; q-- > 0u;) {
        const uint32_t px0 = q << c.log_chunk;
#pragma unroll 1
        for (uint32_t turn = 0; turn < turns; ++turn) {
            const uint32_t task = (turn << 6) + t, l = task >> c.log_chunk, i = task & (chunk - 1u);
            const uint4 sh = shapes[l];
            if (px0 + i >= sh.y) continue;
            uint32_t p = sh.x + px0 + i;
            if (g.lane_mode != 0u) {
                const uint32_t row = (px0 + i) / sh.z;
                p += row * (g.w - sh.z);
            }
            constexpr int kHalves = 3 * kK;
            uint32_t m[(kHalves + 1) / 2] = {}, s[(kHalves + 1) / 2] = {}, wt[(kK + 1) / 2] = {};
            __builtin_memcpy(m, a.mu + (size_t)p * kHalves, 2 * kHalves);
            __builtin_memcpy(s, a.ls + (size_t)p * kHalves, 2 * kHalves);
            __builtin_memcpy(wt, a.weight + (size_t)p * kK, 2 * kK);
            uint32_t xb = 0;
            __builtin_memcpy(&xb, img + 3 * (size_t)p, 3);
            const int16_t *coef = a.coef + 3 * g.by_hw.div(p);
            const int a_gr = coef[0], a_br = coef[1], a_bg = coef[2];
            auto half = [](const uint32_t *d, int e) { return (e & 1) != 0 ? d[e >> 1] >> 16 : d[e >> 1] & 0xFFFFu; };
            uint32_t sum = 0;
#pragma unroll
            for (int j = 0; j < kK; ++j) sum += half(wt, j);
            ok = ok && sum == 1u << 15;
            const int x[3] = {(int)(xb & 0xFFu), (int)((xb >> 8) & 0xFFu), (int)((xb >> 16) & 0xFFu)};
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const int v = (int)((xb >> (8 * ch)) & 0xFFu);
                unsigned long long acc_lo = 0ull, acc_hi = 0ull;
#pragma unroll
                for (int j = 0; j < kK; ++j) {
                    int me = (int)half(m, ch * kK + j);
                    if (ch >= 1) {
                        const int e_r = x[0] * 256 - (int)half(m, j);
                        if (ch == 1)
                            me += rsh14_mul(a_gr, e_r);
                        else
                            me += rsh14_mul(a_br, e_r) + rsh14_mul(a_bg, x[1] * 256 - (int)half(m, kK + j));
                    }
                    const EdgeStep e(256 * v - 128 - me, inv_scale((int)(short)half(s, ch * kK + j), tab));
                    const uint32_t w = half(wt, j);
                    acc_lo += (unsigned long long)w * edge_at(e.y, tab);
                    acc_hi += (unsigned long long)w * edge_at(e.above(), tab);
                }
                const uint32_t lo = v == 0 ? 0u : (uint32_t)v + mass_of((uint32_t)(acc_lo >> 15), scale);
                const uint32_t hi = v == 255 ? top : (uint32_t)v + 1u + mass_of((uint32_t)(acc_hi >> 15), scale);
                rec[((3u * i + ch) << c.log_lanes) + l] = lo | ((hi - lo) << 16);
            }
        }
        wave_lds_sync();
        // pixels last-first, and B, G, R inside a pixel (App. A eq. (11) runs against the decoder)
        uint32_t own = npx;
        if (kChainInLds) {
            own = t < lanes_here ? shapes[t].y : 0u;
            nwords = shapes[t].w;
        }
        for (uint32_t i = own > px0 ? min(own - px0, chunk) : 0u; i-- > 0u;) {
            uint32_t r[3];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) r[ch] = rec[((3u * i + ch) << c.log_lanes) + t];
#pragma unroll
            for (int ch = 2; ch >= 0; --ch) {
                const uint32_t lo = r[ch] & 0xFFFFu, f = r[ch] >> 16;
                if (S >= (f << (32u - m_bits))) {
                    *wout = (uint16_t)(S & 0xFFFFu);
                    wout += 64;
                    ++nwords;
                    S >>= 16;
                }
                S = (uint32_t)__umul24(quotient(S, over_reciprocal(f)), top - f) + (S + lo);
            }
        }
        if (kChainInLds && mine) shapes[t].w = nwords;
        wave_lds_sync();
    }
    if (!ok) atomicMax(status_code, 7);
    if (mine) {
        lane_words[lane] = nwords;
        lane_state[lane] = S;
    }
}

// Decoded bytes of consecutive addresses, gathered into aligned 8-byte stores; single bytes only
// up to the first 8-byte boundary of a run and for what is left at its end.
struct ByteRun {
    unsigned __int128 acc;
    uint32_t n;   // bytes in acc (< 11)
    size_t addr;  // where the first of them goes
    __device__ __forceinline__ void begin(size_t a) { acc = 0; n = 0u; addr = a; }
    __device__ __forceinline__ void put3(uint8_t *out, uint32_t v)
    {
        acc |= (unsigned __int128)v << (8u * n);
        n += 3u;
        while (n != 0u && (addr & 7u) != 0u) {
            out[addr++] = (uint8_t)acc;
            acc >>= 8;
            --n;
        }
        if (n >= 8u) {
            *reinterpret_cast<unsigned long long *>(out + addr) = (unsigned long long)acc;
            acc >>= 64;
            n -= 8u;
            addr += 8u;
        }
    }
    __device__ __forceinline__ void end(uint8_t *out)
    {
        while (n != 0u) {
            out[addr++] = (uint8_t)acc;
            acc >>= 8;
            --n;
        }
    }
};

// A thread per lane.  kK > 0: built for that many components (arrays on 4-byte boundaries: the host checks), which live
// in registers; 0: any number, in LDS, and arrays at any address.
template <int kK>
__global__ __launch_bounds__(kMixThreads) __attribute__((amdgpu_waves_per_eu(1, mix_waves(kK)))) void k_mix_decode(
    Geo g, const uint8_t *__restrict__ coded, unsigned long long coded_bytes, MixArgs a, uint8_t *__restrict__ out,
    Report *__restrict__ report)
{
    constexpr int kBuilt = kK > 0 ? kK : 1;
    __shared__ LdsTables tab;
    __shared__ int s_state;
    __shared__ unsigned long long s_payload;
    extern __shared__ uint32_t mix_lds[];
    if (threadIdx.x == 0u) s_state = check_header(g, kMagicMix, a.k, coded, coded_bytes, &s_payload);
    load_tables(tab);  // ends with a barrier
    if (s_state != ST_OK) {
        if (blockIdx.x == 0u && threadIdx.x == 0u) raise_code(report, s_state);
        return;
    }
    const uint32_t lane = blockIdx.x * blockDim.x + threadIdx.x;
    if (lane >= g.lanes) return;
    const MixSlots slots(mix_lds, kK > 0 ? (uint32_t)kK : a.k, kK == 0);
    const LaneShape sh = lane_shape(g, lane);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), mask = (1u << m_bits) - 1u;
    const uint32_t payload_bytes = (uint32_t)s_payload;

    // (k_mix_decode_rows opens its lanes likewise.  With one function for both, the registers of this loop come out otherwise: 2048
    // images of 64 x 64, K = 16, 1312 us, 1533 with the function.)
    const uint32_t *offsets = reinterpret_cast<const uint32_t *>(coded + 64);
    const uint16_t *payload =
        reinterpret_cast<const uint16_t *>(coded + 64 + 4ull * ((size_t)g.lanes + 1));
    const uint32_t begin = offsets[lane], end = offsets[lane + 1];
    if (end < begin || end > payload_bytes || end - begin < 4u || ((begin | end) & 1u)) {
        raise_code(report, ST_CORRUPT);
        return;
    }
    const uint32_t adj = (uint32_t)(reinterpret_cast<uintptr_t>(payload) & 31u);
    const uint16_t *base = reinterpret_cast<const uint16_t *>(reinterpret_cast<const uint8_t *>(payload) - adj);
    const uint32_t first = (adj + begin) >> 1;
    const uint32_t lim = (uint32_t)(((unsigned long long)adj + payload_bytes + 1ull) >> 1);
    WordStream words;
    words.open(base, first, lim);
    uint32_t S = words.take(base, lim);
    S |= words.take(base, lim) << 16;

    bool ok = true;
    ByteRun run;
    run.begin(0);
    uint32_t p_next = 0xFFFFFFFFu;  // the pixel that would continue the current run of bytes
    MixAhead<kBuilt> pre;  // (of the kernels built for one K, as are the registers)
    MixRegs<kBuilt> regs;
    uint32_t im_now = 0xFFFFFFFFu;
    int a_gr = 0, a_br = 0, a_bg = 0;
    if constexpr (kK > 0)
        if (sh.npx != 0u) mix_fetch_ahead(a, lane_pixel(g, sh, 0u), pre);
    for (uint32_t t = 0; t < sh.npx; ++t) {
        const uint32_t p = lane_pixel(g, sh, t);
        if (p != p_next) {  // a new row of the lane
            run.end(out);
            run.begin(3 * (size_t)p);
        }
        p_next = p + 1u;
        const uint32_t im = g.by_hw.div(p);
        if (im != im_now) {
            im_now = im;
            a_gr = a.coef[3 * im]; a_br = a.coef[3 * im + 1]; a_bg = a.coef[3 * im + 2];
        }
        if constexpr (kK > 0) {
            ok = mix_store_ahead(pre, slots, regs, (kK & 1) != 0 && (p & 1u) != 0u) && ok;
            if (t + 1u < sh.npx) mix_fetch_ahead(a, lane_pixel(g, sh, t + 1u), pre);
        } else {
            ok = mix_load_pixel(a, p, slots) && ok;
        }
        int x_r = 0, x_g = 0, x_b = 0;
#pragma unroll 1
        for (int ch = 0; ch < 3; ++ch) {
            if constexpr (kK > 0)
                mix_load_channel(slots, regs, ch, x_r, x_g, a_gr, a_br, a_bg, tab);
            else
                mix_load_channel(slots, ch, x_r, x_g, a_gr, a_br, a_bg, tab);
            const uint32_t slot = S & mask;
            // the symbol is in lo .. lo + 2 * step - 1, and c_hi = C(lo + 2 * step)
            int lo = 0;
            uint32_t c_lo = 0u, c_hi = 1u << m_bits;
#pragma unroll 1
            for (int step = 128; step >= 1; step >>= 1) {
                uint32_t cv;
                if constexpr (kK > 0)
                    cv = mix_cum_inner(lo + step, regs, scale, tab);
                else
                    cv = mix_cum_inner(lo + step, slots, scale, tab);
                const bool ge = cv <= slot;
                lo = ge ? lo + step : lo;
                c_lo = ge ? cv : c_lo;
                c_hi = ge ? c_hi : cv;
            }
            // App. A eq. (12)
            // the mass is at most 2^16 and S >> M below 2^22: a 24-bit multiply is exact
            S = (uint32_t)__umul24(c_hi - c_lo, S >> m_bits) + slot - c_lo;
            if (S < (1u << 16)) S = (S << 16) | words.take(base, lim);
            x_b = ch == 2 ? lo : x_b;
            x_g = ch == 1 ? lo : x_g;
            x_r = ch == 0 ? lo : x_r;
        }
        run.put3(out, (uint32_t)x_r | ((uint32_t)x_g << 8) | ((uint32_t)x_b << 16));
    }
    run.end(out);
    if (!ok) raise_code(report, ST_PARAMS);
    if (S != (1u << 16) || words.taken(first) != (end - begin) >> 1) raise_code(report, ST_CORRUPT);
}

// --------------------------------------------------------------------------------------------
// The decoder for few lanes: a row of 16 threads a lane, four lanes a wavefront, for arrays at any address.
//
// A lane is a serial chain, and a thread by itself evaluates C(k) eight times a symbol, ten laws each.  Here the row evaluates it
// at sixteen places at once, so twice a symbol: every sixteenth value, then the sixteen between two of them.  Thread j has the
// parameters of component j, asked for a pixel ahead, forms its law (the scales, which need no decoded value, a
// pixel ahead as well) and leaves it in LDS for the row.
// Bound by the length of that chain while a SIMD has one wavefront, then by the instructions of the sixteen evaluations.
// --------------------------------------------------------------------------------------------
constexpr int kMixRowThreads = 256;
// Up to so many lanes.  Rows against thread per lane, lanes of 64 pixels, us: ten components 2048 178 and 635, 8192 237 and 650, 16,384 393
// and 670, 24,576 532 and 670, 32,768 700 and 690; two 16,384 201 and 284, 24,576 269 and 292, 32,768 339 and 301; sixteen 16,384
// 653 and 972, 24,576 961 and 979, 32,768 1264 and 987; a photograph of 1365 x 2047 in tiles of 16 x 16 1118 and 2636.
constexpr uint32_t kMixRowLanes = 24576;

template <int kK>
__global__ __launch_bounds__(kMixRowThreads) void k_mix_decode_rows(
    Geo g, const uint8_t *__restrict__ coded, unsigned long long coded_bytes, MixArgs a, uint8_t *__restrict__ out,
    Report *__restrict__ report)
{
    __shared__ LdsTables tab;
    __shared__ int s_state;
    __shared__ unsigned long long s_payload;
    __shared__ EdgeLaw s_law[kMixRowThreads / 16][kK];
    __shared__ uint32_t s_weight[kMixRowThreads / 16][kK];
    if (threadIdx.x == 0u) s_state = check_header(g, kMagicMix, a.k, coded, coded_bytes, &s_payload);
    load_tables(tab);  // ends with a barrier
    if (s_state != ST_OK) {
        if (blockIdx.x == 0u && threadIdx.x == 0u) raise_code(report, s_state);
        return;
    }
    const uint32_t j = threadIdx.x & 15u, row = threadIdx.x >> 4, first_of_row = threadIdx.x & 48u;
    const uint32_t lane = blockIdx.x * (kMixRowThreads / 16) + row;
    if (lane >= g.lanes) return;
    const LaneShape sh = lane_shape(g, lane);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), mask = (1u << m_bits) - 1u, top = 1u << m_bits;
    const uint32_t payload_bytes = (uint32_t)s_payload;
    const uint32_t *offsets = reinterpret_cast<const uint32_t *>(coded + 64);
    const uint16_t *payload = reinterpret_cast<const uint16_t *>(coded + 64 + 4ull * ((size_t)g.lanes + 1));
    const uint32_t begin = offsets[lane], end = offsets[lane + 1];
    if (end < begin || end > payload_bytes || end - begin < 4u || ((begin | end) & 1u)) {
        if (j == 0u) raise_code(report, ST_CORRUPT);
        return;
    }
    const uint32_t adj = (uint32_t)(reinterpret_cast<uintptr_t>(payload) & 31u);
    const uint16_t *base = reinterpret_cast<const uint16_t *>(reinterpret_cast<const uint8_t *>(payload) - adj);
    const uint32_t first = (adj + begin) >> 1;
    const uint32_t lim = (uint32_t)(((unsigned long long)adj + payload_bytes + 1ull) >> 1);
    WordStream words;  // (every thread of the row the same)
    words.open(base, first, lim);
    uint32_t S = words.take(base, lim);
    S |= words.take(base, lim) << 16;

    struct Own {  // of component j (threads past the last one have its)
        uint32_t m[3], w;
        int l[3], c[3];
    };
    const uint32_t own = min(j, (uint32_t)kK - 1u);
    auto fetch = [&](uint32_t t) {
        const uint32_t p = lane_pixel(g, sh, min(t, sh.npx - 1u));
        const size_t at = (size_t)p * (3u * kK) + own;
        const int16_t *coef = a.coef + 3 * g.by_hw.div(p);
        Own o;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            o.m[ch] = a.mu[at + ch * kK];
            o.l[ch] = a.ls[at + ch * kK];
            o.c[ch] = coef[ch];
        }
        o.w = a.weight[(size_t)p * kK + own];
        return o;
    };
    bool ok = true;
    uint32_t w[kK];
    EdgeLaw law[kK];
    auto cum = [&](uint32_t k) {  // C(k), 0 <= k <= 255
        unsigned long long acc = 0ull;
#pragma unroll
        for (int c = 0; c < kK; ++c) acc += (unsigned long long)w[c] * edge_at(edge_y((int)k, law[c]), tab);
        return k == 0u ? 0u : k + mass_of((uint32_t)(acc >> 15), scale);
    };
    auto row_count = [&](bool pred) { return (uint32_t)__popc((uint32_t)(__ballot(pred) >> first_of_row) & 0xFFFFu); };
    auto from_thread = [&](uint32_t n, uint32_t v) {  // v of thread n of the row
        return (uint32_t)__builtin_amdgcn_ds_bpermute((int)((first_of_row + n) << 2), (int)v);
    };
    Own now = fetch(0u);
    uint32_t inv_s[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) inv_s[ch] = inv_scale(now.l[ch], tab);
    for (uint32_t t = 0; t < sh.npx; ++t) {
        const Own next = fetch(t + 1u);
        if (j < (uint32_t)kK) s_weight[row][j] = now.w;
        int x[3] = {0, 0, 0};
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            int me = (int)now.m[ch];
            if (ch >= 1) {
                const int e_r = x[0] * 256 - (int)now.m[0];
                me += ch == 1 ? rsh14_mul(now.c[0], e_r) : rsh14_mul(now.c[1], e_r) + rsh14_mul(now.c[2], x[1] * 256 - (int)now.m[1]);
            }
            wave_lds_sync();  // (the channel before has been read)
            if (j < (uint32_t)kK) s_law[row][j] = edge_law(me, inv_s[ch]);
            wave_lds_sync();
            if (ch == 0) {
                uint32_t sum = 0;
#pragma unroll
                for (int c = 0; c < kK; ++c) {
                    w[c] = s_weight[row][c];
                    sum += w[c];
                }
                ok = ok && sum == 1u << 15;
            }
#pragma unroll
            for (int c = 0; c < kK; ++c) law[c] = s_law[row][c];
            const uint32_t slot = S & mask;
            // the band of sixteen values: n - 1, of which C(16 (n - 1)) <= slot < C(16 n)
            const uint32_t c16 = cum(16u * j);
            const uint32_t n = row_count(c16 <= slot);
            const uint32_t beyond = n < 16u ? from_thread(n, c16) : top;
            // (with weights that do not sum to 2^15 there may be none: a value all the same)
            const uint32_t band = 16u * (max(n, 1u) - 1u);
            const uint32_t c1 = cum(band + j);
            const uint32_t k = max(row_count(c1 <= slot), 1u) - 1u;
            const uint32_t c_lo = from_thread(k, c1), c_next = from_thread(min(k + 1u, 15u), c1);
            const uint32_t c_hi = k < 15u ? c_next : beyond;
            x[ch] = (int)(band + k);
            // App. A eq. (12); the mass is at most 2^16 and S >> M below 2^22: a 24-bit multiply is exact
            S = (uint32_t)__umul24(c_hi - c_lo, S >> m_bits) + slot - c_lo;
            if (S < (1u << 16)) S = (S << 16) | words.take(base, lim);
        }
        if (j < 3u) out[3 * (size_t)lane_pixel(g, sh, t) + j] = (uint8_t)(j == 0u ? x[0] : j == 1u ? x[1] : x[2]);
        now = next;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) inv_s[ch] = inv_scale(now.l[ch], tab);
    }
    if (!ok) raise_code(report, ST_PARAMS);
    if (j == 0u && (S != (1u << 16) || words.taken(first) != (end - begin) >> 1)) raise_code(report, ST_CORRUPT);
}

}  // namespace pilc
