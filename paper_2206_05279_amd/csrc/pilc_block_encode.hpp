// Workgroup-cooperative encoder for batches with few, long lanes (gfx950).
//
// The rANS push (App. A eq. (11) of arXiv 2206.05279) is a serial chain per lane, but only
// the state update itself is serial: the symbol's (cum, freq) and an exact reciprocal of freq
// do not depend on the state, and which states give a word off, and where it goes, is known from the
// states afterwards.  A workgroup owns 16 lanes.  Wave 0 keeps the 16 states, one per
// thread, and does nothing but the chain; producer waves run ahead by one batch of pixels (one
// per thread, 20, 12 or 8 per lane) and leave, per symbol, one ready-made 16-byte record in LDS (see
// encode_record); the last wave comes a batch behind, with the states that the chain has left in LDS,
// and stores the words.  One barrier per batch hands all buffers over; nobody waits inside a batch.
//
// What bounds the kernel is the issue of the chain's wavefront, alone on its SIMD: an instruction of four bytes
// every four cycles, one of eight every five, whether it depends on the one before or not; a memory
// instruction after an arithmetic one ten, after another memory instruction five.  So a step is six arithmetic
// instructions and one read, and every fourth a write.  Whole calls before (a division by multiplication, twelve instructions
// a step, and the chain stored its words itself: 67 cycles a step with nothing beside it, of which the store took twelve) and
// now: 3125 lanes of 16,384 pixels 1740 and 1060 us, 3000 of 4096 456 and 288, 1000 of 1024 137 and 93, 28,672 of 256 198
// and 147, 4000 of 64 42 and 40.  A producer evaluates both edges of its three symbols at once: with a branch around each
// edge that is not needed, one wait after the other, the producers alone took 1290 us of the first, now 750.
#pragma once

#include "pilc_device.hpp"

namespace pilc {

constexpr int kEncLanes = 16;  // lanes per workgroup (threads 0..15 of wave 0 chain)
// Wavefronts that prepare records (`kProducers`), by how many workgroups share a compute unit: five while none does, three
// for two of them, else two, which with 37 KB of LDS lets four share it.  Three against two, us: 8192 lanes of 1024 pixels 161
// and 181, 20,000 of 1024 373 and 345, 28,672 of 256 188 and 147; five against three, 3125 of 16,384 1060
// and 1360.
// With five there is also a wavefront that does nothing, the fifth, so that the chain has its SIMD for itself.
constexpr int kEncAloneProducers = 5, kEncPairProducers = 3, kEncManyProducers = 2;
constexpr bool enc_idles(int producers) { return producers > 3; }
constexpr int enc_waves(int producers) { return 2 + producers + (enc_idles(producers) ? 1 : 0); }
constexpr int enc_threads(int producers) { return 64 * enc_waves(producers); }
constexpr int enc_pixels(int producers) { return 64 * producers / kEncLanes; }  // per lane and batch
constexpr uint32_t kEncGroup = 4u;  // symbols that the chain reads, steps through and writes at a time

// Record of one symbol for the chain: R (a double, its lowest 16 bits replaced by cum), -bound, k, such that one step is
//     if (S >> 16 >= bound) { emit low 16 bits; S >>= 16; }
//     q = floor(S / f);  S = S + cum + q * k.
// This is App. A eq. (11): bound = f << (16-M) (a state renormalises from f << (32-M) on, whose low 16 bits are
// zero) and k = 2^M - f, since (q << M) + (S - q f) + cum = S + cum + q k.
// The division is one multiply-add in double, rounded towards zero: a state as the low word of a double whose high word
// is zero is the number S 2^-1074, and R = r 2^1022 with r a little above 1/f, so S 2^-1074 R + 1 = 1 + S r 2^-52, whose
// low word after the rounding is floor(S r).  That is the quotient while r lies in 1/f .. (1 + 2^-33) / f, because
// S < 2^32: one step of Newton's takes the single-precision reciprocal's error of 2^-22 to 2^-44, the factor
// 1 + 2^-35 puts the result above 1/f, and the lowest 16 bits change it by less than 2^-36.
// The renormalisation is the middle one of three numbers: with h = S >> 16 and d = h - bound mod 2^32, d < h < S where the
// state gives a word off, and h < S < d where it does not (S < bound << 16 <= 2^32 - (255 << 16) < d).
// An all-identity record (R = 0, cum = k = 0, bound = 2^16) skips a slot.
__device__ __forceinline__ u32x4 encode_record(uint32_t cum, uint32_t f, uint32_t m_bits)
{
    const double d = (double)f, r0 = (double)__builtin_amdgcn_rcpf((float)f);
    const double r1 = __builtin_fma(r0, __builtin_fma(-d, r0, 1.0), r0);
    const unsigned long long r = __builtin_bit_cast(unsigned long long, r1 * ((1.0 + 0x1p-35) * 0x1p1022));
    return u32x4{((uint32_t)r & 0xFFFF0000u) | cum, (uint32_t)(r >> 32), 0u - (f << (16u - m_bits)), (1u << m_bits) - f};
}
__device__ __forceinline__ u32x4 empty_record() { return u32x4{0u, 0u, 0xFFFF0000u, 0u}; }

// Rounds double-precision results towards zero in this wavefront from here on (bits 2 and 3 of the mode register),
// which encode_step needs.  (Written out: of the builtin the compiler makes a switch back wherever it uses double itself.)
__device__ __forceinline__ void round_double_to_zero() { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3"); }

// Four steps by four records: `before` receives the state before each, `state` the one after the last; `zero` is 0 and stays
// it.  The steps are written out together: the division needs the state in the low word of a register pair with a zero
// beside it, and the compiler would wait once after every piece that is written out by itself.
__device__ __forceinline__ void encode_steps(uint32_t &state, u32x4 &before, const u32x4 (&rec)[4], uint32_t &zero)
{
    double r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __builtin_bit_cast(double, ((unsigned long long)rec[i].y << 32) | rec[i].x);
    uint32_t s1, s2, s3, s4, t;
#define PILC_ENC_STEP(from, to, i)                    \
    "v_lshrrev_b32_e32 %[t], 16, %[" from "]\n"       \
    "v_add_u32_e32 v4, %[t], %[b" i "]\n"             \
    "v_med3_u32 v2, %[" from "], %[t], v4\n"          \
    "v_fma_f64 v[4:5], v[2:3], %[r" i "], 1.0\n"      \
    "v_add_u32_sdwa %[t], v2, %[c" i "] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n" \
    "v_mad_u32_u24 %[" to "], v4, %[k" i "], %[t]\n"
    asm(PILC_ENC_STEP("s0", "s1", "0") PILC_ENC_STEP("s1", "s2", "1") PILC_ENC_STEP("s2", "s3", "2")
        PILC_ENC_STEP("s3", "s4", "3")
        : [s1] "=&v"(s1), [s2] "=&v"(s2), [s3] "=&v"(s3), [s4] "=&v"(s4), [t] "=&v"(t), [z] "={v3}"(zero)
        : [s0] "v"(state), [b0] "v"(rec[0].z), [r0] "v"(r[0]), [c0] "v"(rec[0].x), [k0] "v"(rec[0].w),
          [b1] "v"(rec[1].z), [r1] "v"(r[1]), [c1] "v"(rec[1].x), [k1] "v"(rec[1].w),
          [b2] "v"(rec[2].z), [r2] "v"(r[2]), [c2] "v"(rec[2].x), [k2] "v"(rec[2].w),
          [b3] "v"(rec[3].z), [r3] "v"(r[3]), [c3] "v"(rec[3].x), [k3] "v"(rec[3].w), "[z]"(zero)
        : "v2", "v4", "v5");
#undef PILC_ENC_STEP
    before = u32x4{state, s1, s2, s3};
    state = s4;
}

template <int kProducers>
__global__ __launch_bounds__(enc_threads(kProducers)) void k_encode_block(
    Geo g, const uint8_t *__restrict__ img, const uint16_t *__restrict__ mu,
    const int16_t *__restrict__ ls, const int16_t *__restrict__ coef, uint16_t *__restrict__ scratch,
    uint32_t *__restrict__ lane_words, uint32_t *__restrict__ lane_state, Status *__restrict__ status)
{
    constexpr uint32_t kEncPix = enc_pixels(kProducers), kEncSyms = 3u * kEncPix, kGroups = kEncSyms / kEncGroup;
    static_assert(kEncSyms % kEncGroup == 0u && 64 * kProducers % kEncLanes == 0, "a batch is whole groups");
    constexpr uint32_t kLastWave = (uint32_t)enc_waves(kProducers) - 1u;
    __shared__ LdsTables tab;
    // records (the odd row spreads a producer's column over the banks), the states before every step, and the records'
    // bounds once more (less one), which outlive them by a batch
    __shared__ u32x4 rec[2][kEncSyms][kEncLanes + 1];
    __shared__ u32x4 states[2][kGroups][kEncLanes];
    __shared__ __align__(8) uint16_t limits[3][kGroups][kEncLanes][kEncGroup];
    __shared__ uint32_t s_max_px;
    if (blockIdx.x == 0u && threadIdx.x == 0u) init_status(status);  // (for the kernels that follow)
    if (threadIdx.x == 0) s_max_px = 0;
    load_tables(tab);  // ends with a barrier

    const uint32_t tid = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane0 = blockIdx.x * kEncLanes;
    const uint32_t nl = min((uint32_t)kEncLanes, g.lanes - lane0);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t scale = mass_scale(m_bits), top = 1u << m_bits;

    const bool chains = wave == 0u, writer = wave == kLastWave, idle = enc_idles(kProducers) && wave == 4u;
    const bool producer = !chains && !writer && !idle;
    const uint32_t q = 64u * (wave - (enc_idles(kProducers) && wave > 4u ? 2u : 1u)) + tid;  // number among the producers
    const uint32_t my = producer ? q / kEncPix : (writer ? tid >> 2 : tid);  // lane of the workgroup this thread serves
    const uint32_t pj = producer ? q - my * kEncPix : 0u;
    const bool has_lane = my < nl;
    const LaneShape sh = lane_shape(g, lane0 + (has_lane ? my : 0u));
    if (chains && has_lane) atomicMax(&s_max_px, sh.npx);
    __syncthreads();
    const uint32_t batches = (s_max_px + kEncPix - 1u) / kEncPix;

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
    auto produce = [&](const PixelIn &in, uint32_t b) {
        const int e_r = in.x[0] * 256 - in.m[0], e_g = in.x[1] * 256 - in.m[1];
        const int me[3] = {in.m[0], in.m[1] + rsh14_mul(in.a[0], e_r),
                           in.m[2] + rsh14_mul(in.a[1], e_r) + rsh14_mul(in.a[2], e_g)};
        uint32_t lo[3], hi[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const EdgeLaw law = edge_law(me[c], inv_scale(in.ls[c], tab));
            const double y = edge_y(in.x[c], law);
            lo[c] = cum_inner(in.x[c], y, scale, tab);
            hi[c] = cum_inner(in.x[c] + 1, y + law.a, scale, tab);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            asm("" : "+v"(lo[c]), "+v"(hi[c]));  // both edges always: the reads of all six are under way together
            lo[c] = in.x[c] == 0 ? 0u : lo[c];
            hi[c] = in.x[c] == 255 ? top : hi[c];
            const u32x4 full = encode_record(lo[c], hi[c] - lo[c], m_bits), none = empty_record();
            // the chain walks a batch last symbol first: pixel pj from the end, B before G before R
            const uint32_t k = 3u * pj + (2 - c);
            const u32x4 r = in.valid ? full : none;
            rec[b & 1u][k][my] = r;
            limits[b % 3u][k / kEncGroup][my][k % kEncGroup] = (uint16_t)~r.z;
        }
    };

    uint32_t S = 1u << 16, zero = 0u;  // (chains)
    auto consume = [&](uint32_t b) {
        // a group's records are read while the group before it is stepped through
        const uint32_t buf = b & 1u;
        u32x4 r[kEncGroup], next[kEncGroup];
#pragma unroll
        for (uint32_t k = 0; k < kEncGroup; ++k) next[k] = rec[buf][k][my];
#pragma unroll
        for (uint32_t grp = 0; grp < kGroups; ++grp) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t k = 0; k < kEncGroup; ++k) {
                r[k] = next[k];
                if (grp + 1u < kGroups) next[k] = rec[buf][kEncGroup * (grp + 1u) + k][my];
            }
            __builtin_amdgcn_sched_barrier(0);
            u32x4 before;
            encode_steps(S, before, r, zero);
            __builtin_amdgcn_sched_barrier(0);
            states[buf][grp][my] = before;
        }
    };

    // (writer) four threads a lane, each a run of the batch's groups
    constexpr uint32_t kRun = (kGroups + 3u) / 4u;
    const uint32_t part = tid & 3u;
    const uint32_t slot_end = block_slot_end(sh, lane0 + (has_lane ? my : 0u));
    uint32_t words = 0u;  // of the lane so far
    auto store_words = [&](uint32_t b) {
        u32x4 s[kRun];
        uint2 l[kRun];
#pragma unroll
        for (uint32_t i = 0; i < kRun; ++i) {
            const uint32_t grp = min(part * kRun + i, kGroups - 1u);
            s[i] = states[b & 1u][grp][my];
            l[i] = *reinterpret_cast<const uint2 *>(&limits[b % 3u][grp][my][0]);
        }
        uint32_t flags = 0u;
#pragma unroll
        for (uint32_t i = 0; i < kRun; ++i) {
            const uint32_t limit[4] = {l[i].x & 0xFFFFu, l[i].x >> 16, l[i].y & 0xFFFFu, l[i].y >> 16};
            uint32_t four = 0u;
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) four |= (s[i][k] >> 16 > limit[k] ? 1u : 0u) << k;
            flags |= (part * kRun + i < kGroups ? four : 0u) << (4u * i);
        }
        const uint32_t mine = (uint32_t)__popc(flags);
        uint32_t before = 0u, all = 0u;
#define PILC_ENC_PART(n)                                                                                          \
    {                                                                                                             \
        const uint32_t c = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, 0x55 * n /* quad_perm: n n n n */, 0xF, 0xF, true); \
        before += n##u < part ? c : 0u;                                                                           \
        all += c;                                                                                                 \
    }
        PILC_ENC_PART(0) PILC_ENC_PART(1) PILC_ENC_PART(2) PILC_ENC_PART(3)
#undef PILC_ENC_PART
        // the lane's words so far end where its slot does; the next goes below them
        uint16_t *to = scratch + ((size_t)slot_end - words - before);
#pragma unroll
        for (uint32_t i = 0; i < kRun; ++i)
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k)
                if ((flags >> (4u * i + k)) & 1u) *--to = (uint16_t)s[i][k];
        words += all;
    };

    PixelIn cur = {};
    if (chains) round_double_to_zero();
    if (producer) {
        cur = fetch(0);
        produce(cur, 0);
        cur = fetch(1);
    }
    __syncthreads();
    for (uint32_t b = 0; b <= batches; ++b) {
        if (producer) {
            const PixelIn nxt = fetch(b + 2u);
            if (b + 1u < batches) produce(cur, b + 1u);
            cur = nxt;
        } else if (chains) {
            if (b < batches && tid < (uint32_t)kEncLanes && has_lane) consume(b);
        } else if (writer) {
            if (b != 0u && has_lane) store_words(b - 1u);
        }
        __syncthreads();
    }
    if (chains && has_lane) lane_state[lane0 + my] = S;
    if (writer && has_lane && part == 0u) lane_words[lane0 + my] = words;
}

}  // namespace pilc
