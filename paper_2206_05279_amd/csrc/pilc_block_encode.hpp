// Workgroup-cooperative encoder for batches with few, long lanes (gfx950).
//
// The rANS push (App. A eq. (11) of arXiv 2206.05279) is a serial chain per lane, but only
// the state update itself is serial: the symbol's (cum, freq) and an exact reciprocal of freq
// do not depend on the state.  A workgroup owns 16 lanes.  Wave 0 keeps the 16 states, one per
// thread, and does nothing but the chain; the other waves run ahead by one batch of pixels (one
// per thread, 24 or 12 per lane) and leave, per symbol, one ready-made 16-byte record in LDS (see
// encode_record).  One barrier per batch hands a buffer over; the two roles never wait for each
// other inside a batch.  The chain is branch-free: a word is stored on every step, below the
// lane's words so far, and counted only when the state renormalises.
#pragma once

#include "pilc_device.hpp"

namespace pilc {

constexpr int kEncLanes = 16;  // lanes per workgroup (threads 0..15 of wave 0 chain)
// Wavefronts that prepare records (`kProducers`): six, or three where there are more workgroups than compute units, so that
// workgroups that share one do not crowd its four SIMDs.  Six against three, us: 4000 lanes of 4096 pixels 466 and 523, 6000 of
// 1024 256 and 206, 25,600 of 64 117 and 84, 28,000 of 256 265 and 193.  (Seven: 1 to 2 % slower than six.)
constexpr int kEncMostProducers = 6, kEncFewProducers = 3;
constexpr int enc_threads(int producers) { return 64 * (1 + producers); }
constexpr int enc_pixels(int producers) { return 64 * producers / kEncLanes; }  // per lane and batch

// floor(2^32 * a / f) for a < f < 2^17, by two 16-bit digits of long division
__device__ __forceinline__ uint32_t frac32(uint32_t a, uint32_t f)
{
    uint32_t n1 = a << 16;
    uint32_t q1 = n1 / f;
    uint32_t r1 = n1 - q1 * f;
    uint32_t q0 = (r1 << 16) / f;
    return (q1 << 16) | q0;
}

// Record of one symbol for the chain: { T, m, add, k | sh << 24 } such that one step is
//     if (S > T) { emit low 16 bits; S >>= 16; }
//     t = mulhi(m, S);  q = (t + ((S - t) >> 1)) >> sh;  S = S + add + q * k.
// For f >= 2 this is App. A eq. (11) with the division by f done by multiplication (Granlund &
// Montgomery, round-up method, l = ceil(log2 f), m = floor(2^32 (2^l - f) / f) + 1, sh = l - 1):
// T = (f << (32-M)) - 1, add = cum, k = 2^M - f, since (q << M) + (S - q f) + cum = S + cum + q k.
// For f = 1 the same formula with m = 2^32 - 1, sh = 0 yields q = S - 1, so add = cum + 2^M - 1
// makes up for the missing k.  An all-identity record (T = 2^32 - 1, add = k = 0) skips a slot.
// k and sh share a word without any unpacking: the 24-bit multiply looks at the low 24 bits only,
// and the shift takes its count from the top byte.
__device__ __forceinline__ uint4 encode_record(uint32_t cum, uint32_t f, uint32_t m_bits)
{
    const uint32_t k = (1u << m_bits) - f;
    if (f == 1u) return make_uint4((1u << (32u - m_bits)) - 1u, 0xFFFFFFFFu, cum + k, k);
    const uint32_t l = 32u - (uint32_t)__clz(f - 1u);
    const uint32_t magic = frac32((1u << l) - f, f) + 1u;
    return make_uint4((f << (32u - m_bits)) - 1u, magic, cum, k | ((l - 1u) << 24));
}

// The chain of one lane.
struct EncChain {
    uint32_t S;     // the state
    uint32_t at;    // where the word below the words so far goes, in bytes ...
    uint32_t back;  // ... once this has been taken off: 2 if the last step's word counts, else 0
};

// One step by a record.  The state's low word belongs at c.at after it.  The step is written out for its order: an
// instruction that reads a condition has to stand three after the one that makes it, and left to itself the
// compiler waits that out, and once more after each single instruction that is written out by itself: 12 of the 86
// cycles of a step, and the kernel is as fast as its chain (3125 lanes of 16,384 pixels 1854 -> 1750 us, with six producers instead of seven 1726).
__device__ __forceinline__ void encode_step(EncChain &c, const uint4 &r)
{
    uint32_t next, high, t;
    asm("v_cmp_gt_u32_e32 vcc, %[s], %[T]\n"
        "v_lshrrev_b32_e32 %[h], 16, %[s]\n"
        "v_sub_u32_e32 %[at], %[at], %[back]\n"
        "v_cndmask_b32_e32 %[n], %[s], %[h], vcc\n"
        "v_mul_hi_u32 %[t], %[n], %[m]\n"
        "v_cndmask_b32_e32 %[back], 0, %[two], vcc\n"
        "v_sub_u32_e32 %[h], %[n], %[t]\n"
        "v_lshrrev_b32_e32 %[h], 1, %[h]\n"
        "v_add_u32_e32 %[t], %[h], %[t]\n"
        "v_lshrrev_b32_sdwa %[t], %[w], %[t] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n"
        "v_mul_u32_u24_e32 %[t], %[t], %[w]\n"
        "v_add3_u32 %[n], %[t], %[add], %[n]"
        : [n] "=&v"(next), [h] "=&v"(high), [t] "=&v"(t), [at] "+&v"(c.at), [back] "+&v"(c.back)
        : [s] "v"(c.S), [T] "v"(r.x), [m] "v"(r.y), [add] "v"(r.z), [w] "v"(r.w), [two] "v"(2u)
        : "vcc");
    c.S = next;
}

// C(k), 1 <= k <= 255, with the position of the edge formed in integers.  (What bounds this kernel is the wavefront of
// chains, which shares its SIMD with one producer, so a producer has to leave issue cycles free, and
// instructions in double and 32-bit high products take more of them than their number says.  With the
// position in double as everywhere else and mass_of, against the lines below, whole calls: 200 lanes of
// 4096 pixels 515 against 511 us, 256 of 16,384 1938 against 1924, 512 of 65,536 7668 against 7593.)
// w = clamp(floor(d * inv_s / 2^17) + 2^20, 1, 2^21 - 1) is bits 17..48 of d * inv_s + 2^37 (the first cell is
// flat: 1 for 0 changes nothing); it saturates exactly when the high word of that sum leaves 0..63, and
// with that word in -1..64 the shift keeps the side.  2^11 w - 1 is the position that interpolate takes.
__device__ __forceinline__ uint32_t cum_of_integers(int k, int mu_eff, uint32_t inv_s, uint32_t scale,
                                                    const LdsTables &t)
{
    long long p = (long long)(256 * k - 128 - mu_eff) * (long long)(int)inv_s + (1ll << 37);  // Q.33
    asm("" : "+v"(p));  // keep the clamps below on 32-bit words
    const int high = min(max((int)(p >> 32), -1), 64);
    const int w = min(max((int)__builtin_amdgcn_alignbit((uint32_t)high, (uint32_t)p, 17), 1), (1 << 21) - 1);
    const uint32_t u = ((uint32_t)w << 11) - 1u;
    const uint32_t f = interpolate(u, t.sig[u >> 21]);
    return (uint32_t)k + ((uint32_t)__umul24(f, scale >> 16) >> 16);
}

// kWide: lanes of 2^27 symbols and more, whose words lie further from the workgroup's first than 32 bits of bytes reach.
template <int kProducers, bool kWide>
__global__ __launch_bounds__(enc_threads(kProducers)) void k_encode_block(
    Geo g, const uint8_t *__restrict__ img, const uint16_t *__restrict__ mu,
    const int16_t *__restrict__ ls, const int16_t *__restrict__ coef, uint16_t *__restrict__ scratch,
    uint32_t *__restrict__ lane_words, uint32_t *__restrict__ lane_state, Status *__restrict__ status)
{
    constexpr uint32_t kEncPix = enc_pixels(kProducers), kEncSyms = 3u * kEncPix;
    __shared__ LdsTables tab;
    if (blockIdx.x == 0u && threadIdx.x == 0u) init_status(status);  // (for the kernels that follow)
    __shared__ uint4 rec[2][kEncSyms][kEncLanes];
    __shared__ uint32_t s_max_px;
    if (threadIdx.x == 0) s_max_px = 0;
    load_tables(tab);  // ends with a barrier

    const uint32_t tid = threadIdx.x;
    const uint32_t lane0 = blockIdx.x * kEncLanes;
    const uint32_t nl = min((uint32_t)kEncLanes, g.lanes - lane0);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), top = 1u << m_bits;

    const bool producer = tid >= 64u;
    const uint32_t q = tid - 64u;
    const uint32_t my = producer ? q / kEncPix : tid;  // lane of the workgroup this thread serves
    const uint32_t pj = producer ? q - my * kEncPix : 0u;
    const bool has_lane = my < nl;
    LaneShape sh = lane_shape(g, lane0 + (has_lane ? my : 0u));
    if (!producer && has_lane) atomicMax(&s_max_px, sh.npx);
    __syncthreads();
    const uint32_t batches = (s_max_px + kEncPix - 1u) / kEncPix;

    // chain state (threads 0..nl-1 of wave 0)
    // index into scratch, one past the lane's slot (block_slot_end: one spare word below every slot)
    const uint32_t slot_end = block_slot_end(sh, lane0 + (has_lane ? my : 0u));
    // the words' places are counted from the first lane's slot (kWide: each lane's from its own, downwards)
    const uint32_t first = kWide ? slot_end - 1u : block_slot_end(lane_shape(g, lane0), lane0) - 3u * lane_shape(g, lane0).npx - 1u;
    uint16_t *const words = scratch + first;
    EncChain chain = {1u << 16, kWide ? 0u : 2u * (slot_end - 1u - first), 0u};
    uint32_t count = 0u;  // (kWide) words so far

    // producers: the nine input values of the pixel of batch b, loaded one batch ahead
    struct PixelIn {
        int x[3], m[3], ls[3], a[3];
        bool valid;
    };
    auto fetch = [&](uint32_t b) {
        PixelIn in;
        const uint32_t idx = b * kEncPix + pj;  // pixel counted from the lane's end
        in.valid = has_lane && idx < sh.npx;
        const uint32_t t = in.valid ? sh.npx - 1u - idx : 0u;
        const uint32_t row = t / sh.tw;
        const uint32_t p = sh.first + row * g.w + (t - row * sh.tw);
        const size_t s = (size_t)p * 3;
        const uint32_t im = g.by_hw.div(p);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            in.x[c] = img[s + c];
            in.m[c] = mu[s + c];
            in.ls[c] = ls[s + c];
            in.a[c] = coef[3 * im + c];
        }
        return in;
    };
    auto produce = [&](const PixelIn &in, uint32_t buf) {
        if (!(my < (uint32_t)kEncLanes)) return;
        const int e_r = in.x[0] * 256 - in.m[0], e_g = in.x[1] * 256 - in.m[1];
        const int me[3] = {in.m[0], in.m[1] + rsh14_mul(in.a[0], e_r),
                           in.m[2] + rsh14_mul(in.a[1], e_r) + rsh14_mul(in.a[2], e_g)};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint32_t inv_s = inv_scale(in.ls[c], tab);
            const uint32_t lo = in.x[c] == 0 ? 0u : cum_of_integers(in.x[c], me[c], inv_s, scale, tab);
            const uint32_t hi = in.x[c] == 255 ? top : cum_of_integers(in.x[c] + 1, me[c], inv_s, scale, tab);
            // the chain walks a batch last symbol first: pixel pj from the end, B before G before R
            rec[buf][3u * pj + (2 - c)][my] =
                in.valid ? encode_record(lo, hi - lo, m_bits) : make_uint4(0xFFFFFFFFu, 0u, 0u, 0u);
        }
    };

    auto consume = [&](uint32_t buf) {
        // all records of the batch first: the loads do not depend on the state
        uint4 r[kEncSyms];
#pragma unroll
        for (uint32_t k = 0; k < kEncSyms; ++k) r[k] = rec[buf][k][my];
#pragma unroll
        for (uint32_t k = 0; k < kEncSyms; ++k) {
            // The word is stored on every step, just below the words already there, and counted
            // only when the state renormalises: an uncounted word is overwritten by the next one
            // or stays below the lane's first word.  After i symbols at most i words are counted
            // and the slot has room for one per symbol, so the store stays in the slot, or, for the
            // empty steps after a lane's last symbol, in the spare word below it.
            const uint16_t low = (uint16_t)chain.S;
            encode_step(chain, r[k]);
            if (kWide) {
                words[-(ptrdiff_t)count] = low;
                count += chain.back >> 1;
            } else {
                *reinterpret_cast<uint16_t *>(reinterpret_cast<uint8_t *>(words) + chain.at) = low;
            }
        }
    };

    PixelIn cur = {};
    if (producer) {
        cur = fetch(0);
        produce(cur, 0);
        cur = fetch(1);
    }
    __syncthreads();
    for (uint32_t b = 0; b < batches; ++b) {
        if (producer) {
            const PixelIn nxt = fetch(b + 2u);
            if (b + 1u < batches) produce(cur, (b + 1u) & 1u);
            cur = nxt;
        } else if (tid < (uint32_t)kEncLanes && has_lane) {
            consume(b & 1u);
        }
        __syncthreads();
    }
    if (!producer && has_lane) {
        lane_words[lane0 + my] = kWide ? count : slot_end - 1u - first - ((chain.at - chain.back) >> 1);
        lane_state[lane0 + my] = chain.S;
    }
}

}  // namespace pilc
