// Device-side arithmetic shared by the libpilc kernels (gfx950 only).
//
// Everything here is integer and must produce, bit for bit, the tables that Sec. 3.2 of
// arXiv 2206.05279 asks for (integer masses summing to 2^M with C_x their running sum) from a
// logistic law with location mu and scale s on 0..255 (Sec. 3.1 eq. (7), Sec. 3.3), after the
// channel conditioning of Sec. 3.1 eqs. (3)-(4).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pilc {

constexpr int kSigEntries = 2048;  // interpolation cells of the sigmoid table
constexpr int kExpHiEntries = 640;
constexpr int kExpLoEntries = 64;
constexpr int kGuideOctaves = 21, kGuideBits = 4;  // sixteen lines an octave of 1 .. 2^21
constexpr int kGuideEntries = kGuideOctaves << kGuideBits;
constexpr float kGuideShift = 9.0f, kGuideLine = 4.25f;

// Constant tables in device globals, filled by the host once per device.
//   g_sig_cell[i] = { D[i] * 2^11, (T[i] - D[i] * i) mod 2^32 },  D[i] = T[i+1] - T[i],
//     T[i] = round(2^24 * sigmoid((i-1024)/64)): the line through a cell's two ends as the 64-bit
//     addend of one multiply-add (interpolate below)
//   g_exp_hi[i]   = round(2^26 * exp(4 - i/64)),  g_exp_lo[j] = round(2^31 * exp(-j/4096))
extern __device__ uint2 g_sig_cell[kSigEntries];
extern __device__ float2 g_guide[kGuideEntries];  // see guide_edge
extern __device__ uint32_t g_exp_hi[kExpHiEntries];
extern __device__ uint32_t g_exp_lo[kExpLoEntries];

// LDS copy of the tables; every coding kernel stages them once per workgroup.
struct LdsTables {
    uint2 sig[kSigEntries];
    uint32_t exp_hi[kExpHiEntries];
    uint32_t exp_lo[kExpLoEntries];
};

__device__ __forceinline__ void load_tables(LdsTables &t)
{
    for (int i = threadIdx.x; i < kSigEntries; i += blockDim.x) t.sig[i] = g_sig_cell[i];
    for (int i = threadIdx.x; i < kExpHiEntries; i += blockDim.x) t.exp_hi[i] = g_exp_hi[i];
    for (int i = threadIdx.x; i < kExpLoEntries; i += blockDim.x) t.exp_lo[i] = g_exp_lo[i];
    __syncthreads();
}

// Sixteen bytes as the compiler's own vector type (arrays of it stay in registers where arrays of
// the HIP struct type of the same size go to private memory).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Orders this wavefront's LDS accesses: LDS instructions of one wavefront execute in order, so
// all that is needed is that the compiler keeps them in order too.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 24-bit signed multiply and multiply-add as the single instructions they are.  (Written through
// the 32-bit product, the compiler first sign-extends operands it cannot prove to be 24 bits wide,
// which costs more instructions than the multiply.)  Operands must lie within +-2^23; only plain
// vector ALU instructions consume the results.
__device__ __forceinline__ int mad_i24(int a, int b, int c)
{
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// Division of a 32-bit number by a divisor fixed at launch (1 <= d < 2^31), as one multiply-high,
// an add, a subtract and two shifts: with l = ceil(log2 d) and m = floor(2^32 (2^l - d) / d) + 1,
// n / d = (t + ((n - t) >> 1)) >> (l - 1) for t = floor(m n / 2^32) and l >= 1; d = 1 is passed on.
// (The division the compiler makes from `/` goes through a float reciprocal and two corrections:
// some fifteen instructions.)
struct FastDiv {
    uint32_t m, s, d;
    static FastDiv make(uint32_t d)
    {
        FastDiv f;
        uint32_t l = 0;
        while ((1ull << l) < d) ++l;
        f.m = l == 0 ? 0u : (uint32_t)((((1ull << l) - d) << 32) / d + 1ull);
        f.s = l == 0 ? 0u : l - 1u;
        f.d = d;
        return f;
    }
    __device__ __forceinline__ uint32_t div(uint32_t n) const
    {
        if (d == 1u) return n;  // the same for every thread
        const uint32_t t = __umulhi(m, n);
        return (t + ((n - t) >> 1)) >> s;
    }
};

// Batch geometry as the kernels see it (derived on the host from pilc_geom).
struct Geo {
    uint32_t n, h, w, hw;
    uint32_t prec_bits;
    uint32_t lane_mode, lane_a, lane_b;
    uint32_t tiles_x, tiles_per_img;  // mode 1
    uint32_t total_px;                // n*h*w   (< 2^32 / 3)
    uint32_t lanes;
    FastDiv by_hw;                    // which image a pixel belongs to: once a chunk or pixel in every kernel
};

// One lane's pixel set: `npx` pixels starting at flat pixel `first`, laid out as rows of `tw`
// pixels with a stride of `w` pixels between row starts (flat lanes are a single row).
struct LaneShape {
    uint32_t first, npx, tw;
    uint32_t sym_base;  // symbols of all lanes before this one (lane-major order)
};

__device__ __forceinline__ LaneShape lane_shape(const Geo &g, uint32_t lane)
{
    LaneShape s;
    if (g.lane_mode == 0) {
        uint64_t first = (uint64_t)lane * g.lane_a;
        uint64_t last = first + g.lane_a;
        if (last > g.total_px) last = g.total_px;
        s.first = (uint32_t)first;
        s.npx = (uint32_t)(last - first);
        s.tw = s.npx;
        s.sym_base = 3u * s.first;
    } else {
        uint32_t img = lane / g.tiles_per_img;
        uint32_t r = lane - img * g.tiles_per_img;
        uint32_t ty = r / g.tiles_x, tx = r - ty * g.tiles_x;
        uint32_t y0 = ty * g.lane_a, x0 = tx * g.lane_b;
        uint32_t th = min(g.lane_a, g.h - y0);
        uint32_t tw = min(g.lane_b, g.w - x0);
        s.first = (img * g.h + y0) * g.w + x0;
        s.npx = th * tw;
        s.tw = tw;
        // tiles above cover y0 full rows; tiles to the left in this tile row are th high
        s.sym_base = 3u * (img * g.hw + y0 * g.w + x0 * th);
    }
    return s;
}

// Where lane `lane`'s words end in the scratch of the few-lane encoder: slots in lane order, one
// word per symbol, and one spare word below every slot.
__device__ __forceinline__ uint32_t block_slot_end(const LaneShape &sh, uint32_t lane)
{
    return sh.sym_base + 3u * sh.npx + lane + 1u;
}

// Flat pixel index of the t-th pixel of a lane (rows of sh.tw pixels, g.w apart).
__device__ __forceinline__ uint32_t lane_pixel(const Geo &g, const LaneShape &sh, uint32_t t)
{
    if (g.lane_mode == 0) return sh.first + t;  // a flat lane is one run of pixels (the same for every thread)
    uint32_t row = t / sh.tw;
    return sh.first + row * g.w + (t - row * sh.tw);
}

// Rounded Q2.14 * Q8.8 product: floor((v + 2^13) / 2^14).
__device__ __forceinline__ int rsh14(int v) { return (v + 8192) >> 14; }

// rsh14(a * e) for a Q2.14 coefficient a (16 bits) and an innovation e = 256 x - mu (18 bits): the
// product is below 2^31 in magnitude, so the 24-bit multiply-add gives it exactly at full rate.
__device__ __forceinline__ int rsh14_mul(int a, int e) { return mad_i24(a, e, 8192) >> 14; }

// log_scale Q4.12 clamped to [-4, 6), counted from -4.
__device__ __forceinline__ int scale_index(int ls) { return min(max(ls, -16384), 24575) + 16384; }

// Q6.25 value of exp(-log_scale).
__device__ __forceinline__ uint32_t inv_scale(int ls, const LdsTables &t)
{
    const int u = scale_index(ls);
    uint32_t inv_s = __umulhi(t.exp_hi[u >> 6], t.exp_lo[u & 63]);
    asm("" : "+v"(inv_s));  // (else its conversion to double is made from the 64-bit product)
    return inv_s;
}

// F(k) in 24 bits at the edge k - 1/2:  d = 256*k - 128 - mu'  (Q8.8), inv_s Q6.25 < 2^31,
// w = clamp(floor(d * inv_s / 2^17) + 2^20, 0, 2^21 - 1), and F = T[i] + floor(D[i] * r / 2^10) for
// i = w >> 10, r = w & 1023.
// What bounds the kernels that evaluate this is vector instruction issue, and on this chip a
// double-precision multiply-add and the conversions to and from double issue like any other
// instruction (4.3 cycles a wavefront with four on a SIMD, measured; min, max, alignbit, mul24 the
// same; plain add, and, or, shift right 2.6), so the position is formed in double: the product and
// the sum have at most 51 significant bits, hence every step is exact, and the conversion to
// uint32 brings the floor and both clamps.  For that the position is scaled by 2^11 (the top of
// its range is the top of the uint32 range) and lowered by one:
//     u = sat(floor((d * inv_s / 2^17 + 2^20 - 1) * 2^11)),   u >> 11 = w - 1 within the clamps.
// The cell is then taken from w - 1 = 1024 i + r', with 1 + r' instead of r along its line: where r
// is 0 that is the far end of the cell before, which has the same value.  At the ends of the range w
// counts as 1 for 0 and 2^21 for 2^21 - 1; the first and the last cell are flat, so F is the same.
constexpr double kEdgeBias = 1048575.0 * 2048.0;  // (2^20 - 1) * 2^11

__device__ __forceinline__ uint32_t edge_pos(double y)
{
    uint32_t u;  // (the language leaves conversions of values out of range open; the instruction saturates)
    asm("v_cvt_u32_f64 %0, %1" : "=v"(u) : "v"(y));
    return u;
}

// F at position u: with the cell's slope s = D * 2^11 and R = u | 2^11 - 1 = i * 2^21 + (r' + 1) * 2^11 - 1,
// s * (R + 1) = D * (i * 2^32 + (r' + 1) * 2^22), so the upper word of s * R + {s, T - D i} is
// T + floor(D * (r' + 1) / 2^10): one OR and one 64-bit multiply-add, no field of u is cut out.
__device__ __forceinline__ uint32_t interpolate(uint32_t u, const uint2 cell)
{
    const unsigned long long line = ((unsigned long long)cell.y << 32) | cell.x;
    return (uint32_t)((line + (unsigned long long)cell.x * (u | 2047u)) >> 32);
}

__device__ __forceinline__ uint32_t edge_at(double y, const LdsTables &t)
{
    const uint32_t u = edge_pos(y);
    return interpolate(u, t.sig[u >> 21]);
}

// The position as a function of k, for laws that are evaluated more than once: y(k) = k a + b.
struct EdgeLaw {
    double a, b;
};
__device__ __forceinline__ EdgeLaw edge_law(int mu_eff, uint32_t inv_s)
{
    const double inv = (double)inv_s;
    EdgeLaw l;
    l.a = inv * 4.0;
    l.b = __builtin_fma((double)(-128 - mu_eff), inv * 0x1p-6, kEdgeBias);
    return l;
}
__device__ __forceinline__ double edge_y(int k, const EdgeLaw &l) { return __builtin_fma((double)k, l.a, l.b); }

// The position of one edge of a value, y(k) from d = 256 k - 128 - mu', and what the next is away: one conversion and one
// multiply-add, and another for each neighbour.  (Times 2^-6 is an addition to the exponent, inv_s is never 0; it issues in
// half a multiplication's time.)
struct EdgeStep {
    double y, unit;  // unit: inv_s * 2^-6
    __device__ __forceinline__ EdgeStep(int d, uint32_t inv_s)
    {
        unit = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, (double)inv_s) - (6ull << 52));
        y = __builtin_fma((double)d, unit, kEdgeBias);
    }
    __device__ __forceinline__ double above() const { return __builtin_fma(256.0, unit, y); }
};

__device__ __forceinline__ uint32_t edge_cdf(int d, uint32_t inv_s, const LdsTables &t)
{
    return edge_at(__builtin_fma((double)d, (double)inv_s * 0x1p-6, kEdgeBias), t);
}

// 2^M - 256 as the multiplier of mass_of: 2^M - 256 = 256 * (2^(M-8) - 1).
__device__ __forceinline__ uint32_t mass_scale(uint32_t prec_bits) { return ((1u << (prec_bits - 8u)) - 1u) << 16; }

// floor(f * (2^M - 256) / 2^24) for a 24-bit f
__device__ __forceinline__ uint32_t mass_of(uint32_t f, uint32_t scale) { return __umulhi(f, scale); }

// C(k), 1 <= k <= 255:  k + floor(F(k) * (2^M - 256) / 2^24).
__device__ __forceinline__ uint32_t cum_inner(int k, double y, uint32_t scale, const LdsTables &t)
{
    return (uint32_t)k + mass_of(edge_at(y, t), scale);
}

// C(k) for any k in 0..256.
__device__ __forceinline__ uint32_t cum_at(int k, int mu_eff, uint32_t inv_s, uint32_t prec_bits,
                                           const LdsTables &t)
{
    if (k <= 0) return 0u;
    if (k >= 256) return 1u << prec_bits;
    return cum_inner(k, edge_y(k, edge_law(mu_eff, inv_s)), mass_scale(prec_bits), t);
}

// --------------------------------------------------------------------------------------------
// Where a symbol lies, from the lower part of the state (`slot`), by solving C(k) = k + N F(k) for k (N = 2^M - 256)
// in single precision instead of searching.  With m = mean + 1/2, v = k - m and T = slot + 1 - m - N / 2 the equation is
//     v + N (sigmoid(v / s) - 1/2) = T,
// which is odd in v and T, so take T <= 0, v = -u and y = sigmoid(-u / s) = (A + u) / N with A = N / 2 - |T|.  From
// ln y - ln(1 - y) = -u / s, the number w = N y / s satisfies
//     w + ln w = q,   q = A / s + ln(N / s) + ln(1 - y),
// so ln w is a function psi of q alone (the logarithm of the Wright omega function), and
//     u = s (ln(N / s) + ln(1 - y) - psi(q)).
// psi comes from a table of lines (g_guide: over x = q + kGuideShift, cut by the leading bits of x as a float; below
// it psi is q), and ln(1 - y) changes so slowly that y may be taken from a straight line through the sigmoid's middle,
// 1 - y = min(1/2 + |T| / (N + c s), 1); the tangent has c = 4, and a line a little less steep is nearer over the range of y
// that is met.  The two values around the nearest edge to the result hold the symbol while 2^M is large against s.  Over
// all slots, with means within the values of a pixel, they miss for 2^M = 1024 none up to s = 20, 1.5 % of the symbols at 33, 8 %
// at 55 and 90, 3 % at 150 and 5 % at 400, by one and now and then by two; for 4096 at most 1 %, by one; from 2^14 on
// none.  (With the tangent 2.6, 11, 14, 10 and 5 %, by up to three.)  The caller evaluates the exact C at two or three
// edges and goes on from there where they do not hold the symbol.
// --------------------------------------------------------------------------------------------
struct GuideScale {  // per launch
    float half, mid, full, log_n, log_s;
    __device__ __forceinline__ explicit GuideScale(uint32_t prec_bits)
    {
        const float n = (float)((1u << prec_bits) - 256u);
        full = n;
        half = 0.5f * n;
        mid = 0.5f * n - 0.5f + 1.0f / 64;  // (a little below slot + 1, so that rounding does not reach the next edge)
        log_n = __logf(n) + kGuideShift;
        log_s = log_n + 4.0f;
    }
};

// The edge nearest to where the symbol begins, 1 .. 255, under the law with mean `mu_eff` and inverse scale `inv_s` (Q6.25).
// kShortChain: ln(1 / s) from the scale index `su`, before `slot` is needed, instead of with ln(1 - y) in one logarithm: two
// instructions more, but one less between the slot and the edge.
template <bool kShortChain>
__device__ __forceinline__ uint32_t guide_edge(uint32_t slot, int mu_eff, uint32_t inv_s, int su, const GuideScale &gs,
                                               const float2 *guide)
{
    const float mean = (float)mu_eff, inv = (float)inv_s * 0x1p-25f;
    const float s = __builtin_amdgcn_rcpf(inv);
    const float t = (float)slot - __builtin_fmaf(mean, 1.0f / 256, gs.mid);
    // (the middle one of three is a modifier of the multiply-add)
    const float not_y = __builtin_amdgcn_fmed3f(__builtin_fmaf(__builtin_fabsf(t), __builtin_amdgcn_rcpf(__builtin_fmaf(kGuideLine, s, gs.full)), 0.5f), 0.0f, 1.0f);
    const float b = kShortChain ? __builtin_fmaf(__builtin_amdgcn_logf(not_y), 0.693147181f, __builtin_fmaf((float)su, -1.0f / 4096, gs.log_s))
                                : __builtin_fmaf(__builtin_amdgcn_logf(not_y * inv), 0.693147181f, gs.log_n);
    const float q = __builtin_fmaf(gs.half - __builtin_fabsf(t), inv, b);
    const float x = __builtin_fmaxf(q, 1.0f);  // below 2^21: half <= 32640, inv <= 54.6, b < 25
    const float2 line = guide[(__float_as_uint(x) >> (23 - kGuideBits)) - (127u << kGuideBits)];
    const float psi = __builtin_fminf(__builtin_fmaf(x, line.x, line.y), q);
    const float k = __builtin_fmaf(__builtin_copysignf(s, t), b - psi, __builtin_fmaf(mean, 1.0f / 256, 1.0f));
    uint32_t edge;  // (saturates)
    asm("v_cvt_u32_f32 %0, %1" : "=v"(edge) : "v"(k));
    return min(max(edge, 1u), 255u);
}

}  // namespace pilc
