// The Three-Way Auto-regressive residual transform of Sec. 3.1 (eqs. (2)-(4)) for gfx950.
//
//   R(u,v) is predicted from R(u-1,v-1), R(u-1,v), R(u,v-1)   (up-left, up, left)
//   G(u,v)                from G(u,v-1),   R(u,v-1), R(u,v)     (left G, left R, this pixel's R)
//   B(u,v)                from B(u,v-1),   G(u,v-1), G(u,v)     (left B, left G, this pixel's G)
// with three weights and a bias each, zero padding above and to the left, and the residual
// r = (x - x^) mod 256.  Forward, every pixel is independent (k_twar_forward4, k_twar_forward_any).  Inverse, a pixel
// needs its left, upper and upper-left neighbours: the paper's schedule runs the red channel along
// anti-diagonals and then green and blue column by column; here a wavefront takes 64 rows, one
// per thread, and walks the anti-diagonals once, recovering R, G and B of a pixel in the same
// step (G and B only need values of the same row, which the thread already holds), with the two
// values a row needs from the row above passed down by a cross-lane shift (k_twar_inverse).
//
// Included at the end of pilc.hip.
#pragma once

#include "pilc_twar_rules.hpp"

namespace pilc {

struct TwarK {
    int w[3][3];  // Q2.14
    int bias[3];  // Q8.14
};

__device__ __forceinline__ int twar_predict(const TwarK &p, int ch, int a, int b, int c)
{
    // 16-bit weights times 8-bit values: 24-bit multiplies are exact and run at full rate
    const int acc = __mul24(p.w[ch][0], a) + __mul24(p.w[ch][1], b) + __mul24(p.w[ch][2], c) + p.bias[ch] + 8192;
    return min(max(acc >> 14, 0), 255);  // arithmetic shift: floor
}

// (a + b) mod 256 for a pixel value: one instruction that adds and keeps the low byte.
__device__ __forceinline__ int add_low_byte(int a, int b)
{
    int r;
    asm("v_add_u32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD"
        : "=v"(r)
        : "v"(a), "v"(b));
    return r;
}

// Byte b (-4 <= b < 12) of the 16 bytes {prev, c0, c1, c2}, b = 0 being the first byte of c0.
template <int B>
__device__ __forceinline__ int byte_at(uint32_t prev, uint32_t c0, uint32_t c1, uint32_t c2)
{
    constexpr int i = B + 4;
    const uint32_t word = i < 4 ? prev : (i < 8 ? c0 : (i < 12 ? c1 : c2));
    return (int)((word >> (8 * (i & 3))) & 255u);
}

// Four pixels (12 bytes, three dwords) per thread, for rows that are a whole number of such
// groups in 4-byte aligned arrays: dword loads and stores only.
__global__ __launch_bounds__(256) void k_twar_forward4(TwarK p, uint32_t groups, FastDiv by_h,
                                                       FastDiv by_groups_per_row,
                                                       const uint32_t *__restrict__ img,
                                                       uint32_t *__restrict__ res)
{
    const uint32_t gi = blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= groups) return;
    const uint32_t groups_per_row = by_groups_per_row.d;
    const uint32_t row = by_groups_per_row.div(gi), k = gi - row * groups_per_row;
    const uint32_t u = row - by_h.div(row) * by_h.d;
    const uint32_t *x = img + (size_t)gi * 3u;
    const uint32_t c0 = x[0], c1 = x[1], c2 = x[2];
    const uint32_t prev = k > 0 ? x[-1] : 0u;  // the pixel to the left of the group (its last 3 bytes)
    uint32_t u0 = 0u, u1 = 0u, u2 = 0u, uprev = 0u;
    if (u > 0) {
        const uint32_t *y = x - (size_t)groups_per_row * 3u;
        u0 = y[0];
        u1 = y[1];
        u2 = y[2];
        uprev = k > 0 ? y[-1] : 0u;
    }
    uint32_t out[3] = {0u, 0u, 0u};
#define PILC_TWAR_PIXEL(J)                                                                         \
    {                                                                                              \
        const int r0 = byte_at<3 * J>(prev, c0, c1, c2), g0 = byte_at<3 * J + 1>(prev, c0, c1, c2); \
        const int b0 = byte_at<3 * J + 2>(prev, c0, c1, c2);                                       \
        const int rl = byte_at<3 * J - 3>(prev, c0, c1, c2), gl = byte_at<3 * J - 2>(prev, c0, c1, c2); \
        const int bl = byte_at<3 * J - 1>(prev, c0, c1, c2);                                       \
        const int ru = byte_at<3 * J>(uprev, u0, u1, u2), rul = byte_at<3 * J - 3>(uprev, u0, u1, u2); \
        const uint32_t e0 = (uint32_t)(r0 - twar_predict(p, 0, rul, ru, rl)) & 255u;               \
        const uint32_t e1 = (uint32_t)(g0 - twar_predict(p, 1, gl, rl, r0)) & 255u;                \
        const uint32_t e2 = (uint32_t)(b0 - twar_predict(p, 2, bl, gl, g0)) & 255u;                \
        out[(3 * J) >> 2] |= e0 << (8 * ((3 * J) & 3));                                            \
        out[(3 * J + 1) >> 2] |= e1 << (8 * ((3 * J + 1) & 3));                                    \
        out[(3 * J + 2) >> 2] |= e2 << (8 * ((3 * J + 2) & 3));                                    \
    }
    PILC_TWAR_PIXEL(0)
    PILC_TWAR_PIXEL(1)
    PILC_TWAR_PIXEL(2)
    PILC_TWAR_PIXEL(3)
#undef PILC_TWAR_PIXEL
    uint32_t *o = res + (size_t)gi * 3u;
    o[0] = out[0];
    o[1] = out[1];
    o[2] = out[2];
}

// The same four pixels a thread for rows of any width at any address: the groups are counted through the
// rows without regard to where one ends, and every pixel knows its own place.  Bound by memory
// (a byte at a time, a pixel a thread, 16 images of 1365 x 2047 took 168 us and 40,000 of 31 x 33 166; now
// 66 and 60 us, 4.0 and 4.1 TB/s read and written).  `first_row`: the flat row the launch starts with,
// `pixels`: how many it has.
__global__ __launch_bounds__(256) void k_twar_forward_any(TwarK p, uint32_t first_row, uint32_t pixels, FastDiv by_h,
                                                          FastDiv by_w, const uint8_t *__restrict__ img,
                                                          uint8_t *__restrict__ res)
{
    const uint32_t q = 4u * (blockIdx.x * blockDim.x + threadIdx.x);
    if (q >= pixels) return;
    const uint32_t w = by_w.d, h = by_h.d;
    const uint32_t in = by_w.div(q), row = first_row + in;
    uint32_t v = q - in * w, u = row - by_h.div(row) * h;
    const size_t off = ((size_t)first_row * w + q) * 3u;
    const uint8_t *x = img + off;
    uint32_t c[4], a[4];  // the four pixels with the four bytes before them, and the same of the row above
    const uint32_t here = min(4u, pixels - q);
    if (here == 4u && off >= (size_t)3u * w + 4u) {
        __builtin_memcpy(c, x - 4, 16);
        __builtin_memcpy(a, x - 3 * (size_t)w - 4, 16);
    } else {  // the first row of all and the last pixels of all: bytes that are not there are never used
        uint8_t cb[16] = {}, ab[16] = {};
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (off + k >= 4u && (uint32_t)k < 4u + 3u * here) cb[k] = x[k - 4];
            if (off + k >= (size_t)3u * w + 4u && (uint32_t)k < 4u + 3u * here) ab[k] = x[k - 4 - 3ll * w];
        }
        __builtin_memcpy(c, cb, 16);
        __builtin_memcpy(a, ab, 16);
    }
    uint32_t out[3] = {0u, 0u, 0u};
#define PILC_TWAR_PIXEL(J)                                                                         \
    {                                                                                              \
        const bool left = v != 0u, up = u != 0u;                                                   \
        const int r0 = byte_at<3 * J>(c[0], c[1], c[2], c[3]), g0 = byte_at<3 * J + 1>(c[0], c[1], c[2], c[3]); \
        const int b0 = byte_at<3 * J + 2>(c[0], c[1], c[2], c[3]);                                 \
        const int rl = left ? byte_at<3 * J - 3>(c[0], c[1], c[2], c[3]) : 0;                      \
        const int gl = left ? byte_at<3 * J - 2>(c[0], c[1], c[2], c[3]) : 0;                      \
        const int bl = left ? byte_at<3 * J - 1>(c[0], c[1], c[2], c[3]) : 0;                      \
        const int ru = up ? byte_at<3 * J>(a[0], a[1], a[2], a[3]) : 0;                            \
        const int rul = up && left ? byte_at<3 * J - 3>(a[0], a[1], a[2], a[3]) : 0;               \
        const uint32_t e0 = (uint32_t)(r0 - twar_predict(p, 0, rul, ru, rl)) & 255u;               \
        const uint32_t e1 = (uint32_t)(g0 - twar_predict(p, 1, gl, rl, r0)) & 255u;                \
        const uint32_t e2 = (uint32_t)(b0 - twar_predict(p, 2, bl, gl, g0)) & 255u;                \
        out[(3 * J) >> 2] |= e0 << (8 * ((3 * J) & 3));                                            \
        out[(3 * J + 1) >> 2] |= e1 << (8 * ((3 * J + 1) & 3));                                    \
        out[(3 * J + 2) >> 2] |= e2 << (8 * ((3 * J + 2) & 3));                                    \
        const bool wraps = v + 1u == w;                                                            \
        v = wraps ? 0u : v + 1u;                                                                   \
        u = wraps ? (u + 1u == h ? 0u : u + 1u) : u;                                               \
    }
    PILC_TWAR_PIXEL(0)
    PILC_TWAR_PIXEL(1)
    PILC_TWAR_PIXEL(2)
    PILC_TWAR_PIXEL(3)
#undef PILC_TWAR_PIXEL
    uint8_t *o = res + off;
    if (here == 4u) {
        __builtin_memcpy(o, out, 12);
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k)
            if ((uint32_t)k < 3u * here) o[k] = (uint8_t)(out[k >> 2] >> (8 * (k & 3)));
    }
}

// A flat copy by one wavefront: `total` >= 1 elements, element lane + 64 i, four of them a turn, so
// that four loads are under way together (taken one at a time, every load waits for the one
// before).  Loads past the end read the last element again instead of being skipped (a register
// that is only sometimes written costs more in moves than the load it saves); stores past the end
// are skipped.
template <typename T>
__device__ __forceinline__ void flat_copy(const T *__restrict__ src, T *__restrict__ dst, uint32_t total, uint32_t lane)
{
    for (uint32_t base = 0; base < total; base += 256u) {  // the same for the whole wavefront
        T v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) v[k] = src[min(base + lane + 64u * k, total - 1u)];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k)
            if (base + lane + 64u * k < total) dst[base + lane + 64u * k] = v[k];
    }
}

// A wavefront per group of up to 64 rows: whole images when h <= 64 (64 / h of them side by side),
// else the bands of 64 rows of one image one after the other, the last row's red values of a band
// kept in LDS for the first row of the next.  The group's residuals are copied to LDS
// first and the pixels copied back at the end, so that global memory only sees whole, coalesced
// rows.  The tile is the group exactly as it lies in memory (its rows are contiguous there), copied as a flat run of
// elements of type T (16 bytes, 4 bytes or single bytes: what the sizes and addresses allow); the
// skew between rows keeps the threads' accesses on different banks without any padding.
constexpr int kTwarWaves = 4;

template <typename T>
__global__ __launch_bounds__(64 * kTwarWaves) void k_twar_inverse(TwarK p, uint32_t n, uint32_t h,
                                                                  uint32_t w, uint32_t last_bytes,
                                                                  const uint8_t *__restrict__ res,
                                                                  uint8_t *__restrict__ img)
{
    extern __shared__ uint8_t twar_lds[];
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t per = h <= 64u ? 64u / h : 1u;          // images side by side in a wavefront
    const uint32_t groups = (n + per - 1u) / per;
    const uint32_t g = blockIdx.x * kTwarWaves + wave;
    if (g >= groups) return;
    const uint32_t bands = h <= 64u ? 1u : (h + 63u) / 64u;
    // LDS of this wavefront: [last_bytes >= w, a multiple of 16: red values of the row above a band][tile]
    const uint32_t row_stride = 3u * w;
    uint8_t *lastrow = twar_lds + (size_t)wave * (last_bytes + 64u * row_stride);
    uint8_t *tile = lastrow + last_bytes;
    const size_t row_bytes = (size_t)w * 3u;

    for (uint32_t band = 0; band < bands; ++band) {
        // this thread's row
        uint32_t image, u;
        bool have;
        if (h <= 64u) {
            image = g * per + lane / h;
            u = lane % h;
            have = lane < per * h && image < n;
        } else {
            image = g;
            u = band * 64u + lane;
            have = u < h;
        }
        const uint32_t rows_here = h <= 64u ? min(per, n - g * per) * h : min(64u, h - band * 64u);
        {  // the group's rows are contiguous in memory: copy them row by row
            const size_t first = h <= 64u ? (size_t)g * per * h * row_bytes : ((size_t)g * h + band * 64u) * row_bytes;
            wave_lds_sync();
            flat_copy(reinterpret_cast<const T *>(res + first), reinterpret_cast<T *>(tile),
                      rows_here * row_stride / (uint32_t)sizeof(T), lane);
            wave_lds_sync();
        }
        const bool top = u == 0u;                // the row above is padding: its two weights are zero here
        const int w_upleft = top ? 0 : p.w[0][0], w_up = top ? 0 : p.w[0][1];
        // the rounding biases in vector registers of their own: as scalar operands they would be
        // copied into one at every use (a multiply-add takes one scalar operand, and has a weight)
        int bias_r = p.bias[0] + 8192, bias_g = p.bias[1] + 8192, bias_b = p.bias[2] + 8192;
        asm volatile("" : "+v"(bias_r), "+v"(bias_g), "+v"(bias_b));
        // likewise the weights of the multiply-adds that are written out below
        int w_g0 = p.w[1][0], w_g1 = p.w[1][1], w_b0 = p.w[2][0], w_b1 = p.w[2][1];
        asm volatile("" : "+v"(w_g0), "+v"(w_g1), "+v"(w_b0), "+v"(w_b1));
        const bool from_lds = lane == 0u && !top;  // the row above belongs to the previous band
        int rl = 0, gl = 0, bl = 0;
        int above = 0;  // the red value above the pixel decoded last: above-left of the next one
        // row k of an image (or band) runs k positions behind row 0: w + rows - 1 steps in all
        const uint32_t skew = h <= 64u ? lane % h : lane;
        const uint32_t steps = w + min(h, 64u) - 1u;
        for (uint32_t d = 0; d < steps; ++d) {
            int up = __builtin_amdgcn_update_dpp(0, rl, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
            const int v = (int)d - (int)skew;
            const bool on = have && v >= 0 && v < (int)w;
            if (from_lds && on) up = lastrow[v];
            if (on) {
                const uint8_t *s = tile + lane * row_stride + 3u * v;
                const int r0 = s[0], r1 = s[1], r2 = s[2];
                // Three multiply-adds each.  What only needs the pixel to the left comes first, so
                // that each new value can take the place of the one it replaces; the operand that
                // arrives last (the value just decoded) goes into the last multiply-add.
                auto clamp8 = [](int acc) { return min(max(acc >> 14, 0), 255); };
                const int tg = mad_i24(w_g1, rl, mad_i24(w_g0, gl, bias_g));
                const int tb = mad_i24(w_b1, gl, mad_i24(w_b0, bl, bias_b));
                const int tr = mad_i24(w_up, up, mad_i24(w_upleft, above, bias_r));
                const int xr = add_low_byte(r0, clamp8(__mul24(p.w[0][2], rl) + tr));
                const int xg = add_low_byte(r1, clamp8(__mul24(p.w[1][2], xr) + tg));
                const int xb = add_low_byte(r2, clamp8(__mul24(p.w[2][2], xg) + tb));
                uint8_t *o = tile + lane * row_stride + 3u * v;
                o[0] = (uint8_t)xr;
                o[1] = (uint8_t)xg;
                o[2] = (uint8_t)xb;
                // the last row of a band leaves its red values for the next band; it runs 63
                // positions behind the first row's reads of the same buffer
                if (bands > 1u && lane == 63u) lastrow[v] = (uint8_t)xr;
                above = up;
                rl = xr;
                gl = xg;
                bl = xb;
            }
        }
        {
            const size_t first = h <= 64u ? (size_t)g * per * h * row_bytes : ((size_t)g * h + band * 64u) * row_bytes;
            wave_lds_sync();
            flat_copy(reinterpret_cast<const T *>(tile), reinterpret_cast<T *>(img + first),
                      rows_here * row_stride / (uint32_t)sizeof(T), lane);
        }
        wave_lds_sync();
    }
}

// Everything that does not fit the tile kernel (images taller than 64 rows, or rows wider than a
// tile's): the walk along the anti-diagonals with a wavefront per colour channel.
//
// What bounds this is the chain of the red channel: an image takes at least w + h dependent steps,
// however many threads work on it.  Only red needs the row above; green and blue of a row need that
// row alone.  So the channels of 64 rows (a thread per row) are decoded by three wavefronts, green
// a block of 16 columns or two behind red and blue as far behind green, and moving the data is the
// business of two more, one that fetches residuals four blocks ahead and one that stores pixels.
// (One wavefront that did all three channels took 280 cycles a step: 30 frames of 1080 x 1920 487 us;
// and rows that were not whole 16-byte pieces went 64 at a time through one wavefront, 16
// images of 1365 x 2047 in 37.8 ms, now 206 us.)
//
// Two kernels.  k_twar_inverse_strips goes a band of 64 rows at a time and is made small, four workgroups to a compute
// unit, for batches of many strips.  k_twar_inverse_bands runs an image's bands at the same time and is made for
// a short interval between barriers, as every interval and the trip from band to band are waited for by all
// below.  (With the former's steps, bands anywhere on the chip, and words cleared by a launch before, 30 frames of
// 1080 x 1920 took 286 us, now 211; 16 images of 1365 x 2047 257 and 206; 112 of 1024 x 400 400 and 179.)
//
// Thread r of a wavefront runs r columns behind thread 0, so its block of 16 columns number b is
// the window [16 b - r, 16 b - r + 16) of its row.  Data is moved in these windows, as 48 bytes at
// whatever address they start, so rows need no alignment, every block is the same for all threads,
// and a step needs no address arithmetic: the 16 steps are unrolled over registers.  A window
// reaches past the ends of its row at the row's first and last blocks; what is read there is not
// used, what is decoded there is not stored.
//
// A workgroup takes 64 rows, a band, and steps in time with one barrier per block.  Bands that run together
// follow each other some thirteen blocks apart: the last row of a band is passed on through global memory, a 32-bit word a
// value with the launch's mark above it, stored and loaded at device scope, so that a word that has the mark has its
// value and neither side waits for anything but the word itself.  A sixth wavefront asks for the next eight
// blocks of such words over and over and puts what has arrived into LDS.  Bands number themselves
// with a ticket (the first bands of all strips, then the second ones: those that share a compute unit, or come one after the
// other on it, are then many bands apart), so the band above is always a workgroup that is
// already running and never waits for the band below.  The wait is bounded by the constant-rate clock;
// a band that gives up sets an abort word and goes on with what it has, bands below it that find the
// word set do the same, every loop has a fixed count, and the host returns PILC_E_TIMEOUT.
// (Two or three times 64 rows in a workgroup, which pass their last rows on through LDS, save
// that trip through memory, but the wavefronts that then share a SIMD cost more: with the steps of the other kernel one
// frame of 2160 x 3840 took 0.30 ms with 64 rows, 0.35 with 128, 0.45 with 192.)
constexpr int kDiagAhead = 4;   // blocks between asking for a window and putting it into LDS
constexpr int kStripSlots = 6;  // intervals a window stays in LDS: put, taken apart, red, green, blue, stored
constexpr int kDiagSlots = 8;   // with bands together: put, taken up, red, taken up, green, taken up, blue, stored
constexpr int kDiagCarry = 32;  // blocks of the row above a band kept in LDS
constexpr int kDiagPolls = 4;   // requests for words of the row above under way at once
constexpr int kDeviceScope = 16;  // of a buffer store: seen by every compute unit (sc1)

struct Diag {
    uint32_t h, w;
    uint32_t strip_rows;        // consecutive rows decoded together: an image, or as many whole ones as fit a band
    unsigned long long rows;    // n h
    uint32_t blocks;            // of 16 columns, ceil((w + 63) / 16): the last thread has to get through its row
    unsigned long long strip0;  // this launch: strips from strip0 on, bands band0 .. band0 + bands - 1
    uint32_t strips, band0, bands;
    // of bands that run together (k_twar_inverse_bands):
    uint32_t *words;            // [strip, band][block][16]: red values of a band's last row, the mark above each
    uint32_t mark;              // of this launch, 1 .. 255
    uint32_t *ticket;
    uint32_t first_ticket;      // what it stands at before this launch
    uint32_t *abort_word;
    Report *report;
    unsigned long long wait_ticks;
    uint32_t withhold;          // tests of the give-up path: nothing is passed on
};

// The 24-bit signed multiply by the name the compiler's own operation has.  (__mul24 first extends both operands from 24
// bits where the compiler cannot see that they are no wider: one frame of 2160 x 3840 318 against 314 us.)
extern "C" __device__ int mul_i24(int a, int b) __asm("llvm.amdgcn.mul.i24.i32");

// A weight, and the start of a sum.  The sums are kept times four, so that the prediction is the upper
// half of the clamped sum; beyond 2^26 a bias saturates the prediction whatever the three products are.
__device__ __forceinline__ int diag_weight(int w) { return 4 * w; }
__device__ __forceinline__ int diag_bias(int bias) { return 4 * (min(max(bias, -(1 << 26)), 1 << 26) + 8192); }

// (the prediction with sum `acc` plus the residual) mod 256
__device__ __forceinline__ int diag_value(int acc, int residual)
{
    return (int)(((uint32_t)min(max(acc, 0), 0xFFFFFF) >> 16) + (uint32_t)residual) & 255;
}

__device__ __forceinline__ int byte_value(uint32_t w, int i) { return (int)((w >> (8 * i)) & 255u); }

// Sixteen steps of a channel once every thread has entered its row, the values packed four to a register
// as they are made: the instructions that form a value put it into its byte, and those that use it
// pick the byte (sub-dword operands), so nothing is shifted, masked or gathered.  The steps are
// written out because an instruction that reads a register whose byte the instruction before it
// wrote, or reads a neighbour's register less than three instructions after it was written, would get
// old values: the order below keeps both apart.
//
// Red, eight instructions a step.  `up` holds, by bytes, what the thread above packed, a step behind; thread
// 0 has no thread above and its lane of `up` is not written by the shift: it keeps the four
// values of `above` that are moved there before every fourth step.
#define PILC_RED_STEP(X, L, E, K, KP, KPP, DST, SWITCH)                                              \
    "v_mul_i32_i24_sdwa %[t], %[up], %[w_upleft] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #KPP " src1_sel:DWORD\n" \
    "v_add_u32_e32 %[t], %[bias], %[t]\n" SWITCH                                                     \
    "v_mov_b32_dpp %[up], %[" L "] wave_shr:1 row_mask:0xf bank_mask:0xf\n"                          \
    "v_mul_i32_i24_sdwa %[m], %[" L "], %[w_left] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #KP " src1_sel:DWORD\n" \
    "v_mul_i32_i24_sdwa %[n], %[up], %[w_up] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #KP " src1_sel:DWORD\n" \
    "v_add3_u32 %[t], %[t], %[m], %[n]\n"                                                            \
    "v_med3_i32 %[t], %[t], 0, %[most]\n"                                                            \
    "v_add_u32_sdwa %[" X "], %[t], %[" E "] dst_sel:BYTE_" #K " dst_unused:" DST " src0_sel:WORD_1 src1_sel:BYTE_" #K "\n"
#define PILC_RED_FOUR(X, L, E, A)                                                                    \
    PILC_RED_STEP(X, L, E, 0, 3, 2, "UNUSED_PAD", "")                                                \
    PILC_RED_STEP(X, X, E, 1, 0, 3, "UNUSED_PRESERVE", "v_mov_b32_e32 %[up], %[" A "]\n")           \
    PILC_RED_STEP(X, X, E, 2, 1, 0, "UNUSED_PRESERVE", "")                                           \
    PILC_RED_STEP(X, X, E, 3, 2, 1, "UNUSED_PRESERVE", "")
// `left`: the four values before these; `above`: those above thread 0 from the second step on (the one above the
// first step is the last of the block before and still stands in `up`)
__device__ __forceinline__ void red_steps(int w_upleft, int w_up, int w_left, int bias, const uint32_t (&e)[4],
                                          const uint32_t (&above)[4], uint32_t left, uint32_t &up, uint32_t (&x)[4])
{
    int t, m, n;
    uint32_t u = up;
    asm(PILC_RED_FOUR("x0", "left", "e0", "a0") PILC_RED_FOUR("x1", "x0", "e1", "a1")
        PILC_RED_FOUR("x2", "x1", "e2", "a2") PILC_RED_FOUR("x3", "x2", "e3", "a3")
        : [x0] "=&v"(x[0]), [x1] "=&v"(x[1]), [x2] "=&v"(x[2]), [x3] "=&v"(x[3]), [up] "+&v"(u), [t] "=&v"(t),
          [m] "=&v"(m), [n] "=&v"(n)
        : [e0] "v"(e[0]), [e1] "v"(e[1]), [e2] "v"(e[2]), [e3] "v"(e[3]), [a0] "v"(above[0]), [a1] "v"(above[1]),
          [a2] "v"(above[2]), [a3] "v"(above[3]), [left] "v"(left), [w_upleft] "v"(w_upleft), [w_up] "v"(w_up),
          [w_left] "v"(w_left), [bias] "v"(bias), [most] "v"(0xFFFFFF));
    up = u;
}
#undef PILC_RED_FOUR
#undef PILC_RED_STEP

// Green and blue, seven instructions a step, from the channel decoded before (`before`, with its four values
// before these in `before_left`).
#define PILC_ROW_STEP(X, L, E, B, BL, K, KP, DST)                                                    \
    "v_mul_i32_i24_sdwa %[t], %[" B "], %[w_before] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #K " src1_sel:DWORD\n" \
    "v_mul_i32_i24_sdwa %[m], %[" BL "], %[w_left_before] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #KP " src1_sel:DWORD\n" \
    "v_add3_u32 %[t], %[t], %[m], %[bias]\n"                                                         \
    "v_mul_i32_i24_sdwa %[m], %[" L "], %[w_left] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #KP " src1_sel:DWORD\n" \
    "v_add_u32_e32 %[t], %[t], %[m]\n"                                                               \
    "v_med3_i32 %[t], %[t], 0, %[most]\n"                                                            \
    "v_add_u32_sdwa %[" X "], %[t], %[" E "] dst_sel:BYTE_" #K " dst_unused:" DST " src0_sel:WORD_1 src1_sel:BYTE_" #K "\n"
#define PILC_ROW_FOUR(X, L, E, B, BL)                                                                \
    PILC_ROW_STEP(X, L, E, B, BL, 0, 3, "UNUSED_PAD")                                                \
    PILC_ROW_STEP(X, X, E, B, B, 1, 0, "UNUSED_PRESERVE")                                            \
    PILC_ROW_STEP(X, X, E, B, B, 2, 1, "UNUSED_PRESERVE")                                            \
    PILC_ROW_STEP(X, X, E, B, B, 3, 2, "UNUSED_PRESERVE")
__device__ __forceinline__ void row_steps(int w_left, int w_left_before, int w_before, int bias, const uint32_t (&e)[4],
                                          const uint32_t (&before)[4], uint32_t before_left, uint32_t left,
                                          uint32_t (&x)[4])
{
    int t, m;
    asm(PILC_ROW_FOUR("x0", "left", "e0", "b0", "bl") PILC_ROW_FOUR("x1", "x0", "e1", "b1", "b0")
        PILC_ROW_FOUR("x2", "x1", "e2", "b2", "b1") PILC_ROW_FOUR("x3", "x2", "e3", "b3", "b2")
        : [x0] "=&v"(x[0]), [x1] "=&v"(x[1]), [x2] "=&v"(x[2]), [x3] "=&v"(x[3]), [t] "=&v"(t), [m] "=&v"(m)
        : [e0] "v"(e[0]), [e1] "v"(e[1]), [e2] "v"(e[2]), [e3] "v"(e[3]), [b0] "v"(before[0]), [b1] "v"(before[1]),
          [b2] "v"(before[2]), [b3] "v"(before[3]), [bl] "v"(before_left), [left] "v"(left), [w_left] "v"(w_left),
          [w_left_before] "v"(w_left_before), [w_before] "v"(w_before), [bias] "v"(bias), [most] "v"(0xFFFFFF));
}
#undef PILC_ROW_FOUR
#undef PILC_ROW_STEP

// The 16 values of channel kCh from a window's 48 interleaved bytes.
template <int kCh>
__device__ __forceinline__ void window_channel(const u32x4 (&d)[3], uint32_t (&out)[4])
{
    const uint32_t w[12] = {d[0].x, d[0].y, d[0].z, d[0].w, d[1].x, d[1].y, d[1].z, d[1].w, d[2].x, d[2].y, d[2].z, d[2].w};
    // of four pixels' twelve bytes: numbers kCh, kCh + 3, kCh + 6, kCh + 9
    constexpr uint32_t kFirst = kCh == 0 ? 0x00060300u : kCh == 1 ? 0x00070401u : 0x00000502u;
    constexpr uint32_t kThen = kCh == 0 ? 0x05020100u : kCh == 1 ? 0x06020100u : 0x07040100u;
#pragma unroll
    for (int g = 0; g < 4; ++g)
        out[g] = __builtin_amdgcn_perm(w[3 * g + 2], __builtin_amdgcn_perm(w[3 * g + 1], w[3 * g], kFirst), kThen);
}

// The 48 bytes of a window from its three channels.
__device__ __forceinline__ void window_pixels(const uint32_t (&r)[4], const uint32_t (&g)[4], const uint32_t (&b)[4],
                                              u32x4 (&d)[3])
{
    uint32_t w[12];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        w[3 * k] = __builtin_amdgcn_perm(b[k], __builtin_amdgcn_perm(g[k], r[k], 0x01000400u), 0x03040100u);
        w[3 * k + 1] = __builtin_amdgcn_perm(b[k], __builtin_amdgcn_perm(g[k], r[k], 0x06020005u), 0x03020500u);
        w[3 * k + 2] = __builtin_amdgcn_perm(b[k], __builtin_amdgcn_perm(g[k], r[k], 0x00070300u), 0x07020106u);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        d[i].x = w[4 * i];
        d[i].y = w[4 * i + 1];
        d[i].z = w[4 * i + 2];
        d[i].w = w[4 * i + 3];
    }
}

typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));  // sixteen bytes at any address

// A barrier at the head of a loop whose turns write to LDS.  (The wait for those writes is written out: at
// the head of a loop, the compiler leaves it away.)
__device__ __forceinline__ void interval_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
}

// The wavefront that brings the windows of residuals from memory to LDS, and the one that takes the pixels back from there.
// `raw`: [slot][third of the window][row], kSlots of them; `lag`: intervals from a block's turn in red to its store.
template <int kSlots>
__device__ __forceinline__ void fetch_windows(const Diag &a, const uint8_t *__restrict__ res, u32x4 (*raw)[3][64],
                                              unsigned long long strip, uint32_t band_row0, uint32_t lane, int times)
{
    // the windows of 64 rows move as 192 pieces of 16 bytes, three neighbouring threads taking the
    // 48 bytes of a row.  An address outside the array is moved inside; that brings the wrong
    // bytes only where none is used, or at the end of the array's last row, where they are put right.
    const long long last = (long long)(a.rows * a.w * 3ull) - 16;
    long long at[3];
    uint32_t put[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t k = 64u * i + lane, r = (k * 171u) >> 9, part = k - 3u * r;  // r = k / 3 for k < 192
        const unsigned long long row = strip * a.strip_rows + band_row0 + r;
        at[i] = (long long)(row * a.w * 3ull) + 16ll * part - 3ll * r;  // block 0
        put[i] = part * 64u + r;
    }
    u32x4 ahead[kDiagAhead][3];
#pragma unroll
    for (int j = 0; j < kDiagAhead; ++j)
#pragma unroll
        for (int i = 0; i < 3; ++i) ahead[j][i] = u32x4{};
    // Without a condition on anything, so that the number of loads under way is known when one is
    // waited for: what is put before the first block or after the last is not looked at (a
    // slot is written again no sooner than the interval after its pixels have been stored).
    uint32_t slot = kSlots - kDiagAhead;  // of block -kDiagAhead
    static_assert(kSlots >= kDiagAhead, "");
    for (int time0 = 0; time0 < times; time0 += kDiagAhead) {
#pragma unroll
        for (int j = 0; j < kDiagAhead; ++j) {
            interval_barrier();
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                (&raw[slot][0][0])[put[i]] = ahead[j][i];
                const long long over = at[i] - 48 * kDiagAhead - last;
                if (over > 0 && over < 16) {  // the array's end is inside the piece: a few pieces near it
                    uint8_t *q = reinterpret_cast<uint8_t *>(&raw[slot][0][0] + put[i]);
#pragma unroll 1
                    for (int k = 0; k < 16 - (int)over; ++k) q[k] = q[k + (int)over];
                }
            }
            slot = slot + 1u == (uint32_t)kSlots ? 0u : slot + 1u;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const long long from = min(max(at[i], 0ll), last);
                ahead[j][i] = *reinterpret_cast<const u32x4_any *>(res + from);
                at[i] += 48;
            }
        }
    }
}

template <int kSlots>
__device__ __forceinline__ void store_windows(const Diag &a, uint8_t *__restrict__ img, const u32x4 (*raw)[3][64],
                                              unsigned long long strip, uint32_t band_row0, uint32_t lane, int times,
                                              int lead, int lag)
{
    const int blocks = (int)a.blocks;
    const int row_bytes = (int)(3u * a.w);
    uint8_t *to[3];
    int in_row[3];  // where the piece lies in its row
    uint32_t get[3];
    bool have[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t k = 64u * i + lane, r = (k * 171u) >> 9, part = k - 3u * r;
        const uint32_t u = band_row0 + r;
        const unsigned long long row = strip * a.strip_rows + u;
        have[i] = u < a.strip_rows && row < a.rows;
        in_row[i] = 16 * (int)part - 3 * (int)r;
        to[i] = img + (long long)((have[i] ? row : 0ull) * a.w * 3ull) + in_row[i];
        get[i] = part * 64u + r;
    }
    uint32_t slot = 0;
    for (int time = 0; time < times; ++time) {
        interval_barrier();
        const int b = time - lead - lag;
        if (b < 0 || b >= blocks) continue;
        u32x4 v[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = (&raw[slot][0][0])[get[i]];
        slot = slot + 1u == (uint32_t)kSlots ? 0u : slot + 1u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int first = in_row[i] + 48 * b;
            uint8_t *q = to[i] + 48ll * b;
            if (!have[i]) continue;
            if (first >= 0 && first + 16 <= row_bytes) {
                *reinterpret_cast<u32x4_any *>(q) = v[i];
            } else if (first > -16 && first < row_bytes) {  // an end of the row
                const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (first + k >= 0 && first + k < row_bytes) q[k] = (uint8_t)(w[k >> 2] >> (8 * (k & 3)));
            }
        }
    }
}

// A band of each strip, a workgroup each; the row above, if any, is in the image.  25,088 bytes of LDS and 80 registers: four workgroups
// share a compute unit, which is what batches of many strips live on.
__global__ __launch_bounds__(64 * 6) void k_twar_inverse_strips(TwarK p, Diag a, const uint8_t *__restrict__ res,
                                                              uint8_t *__restrict__ img)
{
    __shared__ u32x4 raw[kStripSlots][3][64];  // [slot][third of the window][row]: residuals, then pixels
    __shared__ u32x4 red[4][64];              // [block mod 4][row]
    __shared__ u32x4 green[2][64];            // [block mod 2][row]
    __shared__ uint32_t carry[kDiagCarry][4]; // [block mod kDiagCarry][word]: red of the row above
    const uint32_t band = a.band0;
    const unsigned long long strip = a.strip0 + blockIdx.x;
    const uint32_t role = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t band_row0 = band * 64u;       // row of the strip
    const int blocks = (int)a.blocks;
    // intervals between barriers, a multiple of 4: a window is fetched kDiagAhead intervals before it is put
    // into LDS, red takes it apart in the next and decodes it in the one after, then green, blue, and the store
    const int lead = kDiagAhead + 2;
    const int times = (lead + blocks + 3 + 3) & ~3;

    if (role == 0u) {  // ---- red
        const uint32_t u = band_row0 + lane;
        const bool top = u % a.h == 0u;  // the row above is padding: its two weights are zero here
        const int w_upleft = top ? 0 : diag_weight(p.w[0][0]), w_up = top ? 0 : diag_weight(p.w[0][1]);
        const int w_left = diag_weight(p.w[0][2]);
        const int bias = diag_bias(p.bias[0]);
        uint32_t left = 0, up = 0;  // the last four values, and the four above them as red_steps keeps them
        uint32_t slot = 0, e[4] = {};
        for (int time = 0; time < times; ++time) {
            interval_barrier();
            const int b = time - lead;
            if (b < -1 || b >= blocks) continue;
            if (b >= 0) {
                uint32_t above[4], x[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                // thread 0 is at columns 16 b .. + 15; column v of the row above is value v + 63 of its blocks
                for (int k = 0; k < 4; ++k) above[k] = carry[(b + 4) % kDiagCarry][k];
                if (b >= 4) {
                    red_steps(w_upleft, w_up, w_left, bias, e, above, left, up, x);
                } else {
                    // some thread has not reached its row's first column yet and keeps zeros
                    if (b == 0 && lane == 0u) up = carry[3][3] & 0xFF000000u;  // column 0; left of it is padding
                    const int left_to_go = (int)lane - 16 * b;
                    int last_up = byte_value(up, 2), rl = byte_value(left, 3);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const uint32_t word = i == 0 ? up : above[(i - 1) >> 2];
                        // thread 0 has no neighbour to take from and keeps what stands there: the value above it
                        const int now_up = __builtin_amdgcn_update_dpp(byte_value(word, (i + 3) & 3), rl,
                                                                       0x138 /* wave_shr:1 */, 0xF, 0xF, false);
                        const int acc = mul_i24(w_up, now_up) + (mul_i24(w_left, rl) + (mul_i24(w_upleft, last_up) + bias));
                        int v = diag_value(acc, byte_value(e[i >> 2], i & 3));
                        v = i >= left_to_go ? v : 0;
                        x[i >> 2] |= (uint32_t)v << (8 * (i & 3));
                        rl = v;
                        last_up = now_up;
                    }
                    up = (uint32_t)__builtin_amdgcn_update_dpp((int)above[3], (int)x[3], 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
                }
                left = x[3];
                u32x4 o;
                o.x = x[0];
                o.y = x[1];
                o.z = x[2];
                o.w = x[3];
                red[b & 3][lane] = o;
            }
            // the next block's residuals, which no barrier has to be waited for
            u32x4 d[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) d[i] = raw[slot][i][lane];
            slot = slot + 1u == (uint32_t)kStripSlots ? 0u : slot + 1u;
            window_channel<0>(d, e);
        }
    } else if (role == 1u || role == 2u) {  // ---- green and blue
        auto channel = [&](auto blue) {
            constexpr int kCh = decltype(blue)::value ? 2 : 1;
            // green from the left green, the left red and the red here; blue likewise from blue and green
            const int w_left = diag_weight(p.w[kCh][0]), w_left_before = diag_weight(p.w[kCh][1]);
            const int w_before = diag_weight(p.w[kCh][2]);
            const int bias = diag_bias(p.bias[kCh]);
            uint32_t left = 0, before_left = 0;  // the last four values of this channel and of the one decoded before it
            uint32_t slot = 0;
            for (int time = 0; time < times; ++time) {
                interval_barrier();
                const int b = time - lead - kCh;
                if (b < 0 || b >= blocks) continue;
                u32x4 d[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) d[i] = raw[slot][i][lane];
                const u32x4 r = red[b & 3][lane];
                const uint32_t rd[4] = {r.x, r.y, r.z, r.w};
                uint32_t gr[4] = {0u, 0u, 0u, 0u};
                if (kCh == 2) {
                    const u32x4 g = green[b & 1][lane];
                    gr[0] = g.x;
                    gr[1] = g.y;
                    gr[2] = g.z;
                    gr[3] = g.w;
                }
                const uint32_t(&before)[4] = kCh == 2 ? gr : rd;
                uint32_t e[4], x[4] = {0u, 0u, 0u, 0u};
                window_channel<kCh>(d, e);
                if (b >= 4) {
                    row_steps(w_left, w_left_before, w_before, bias, e, before, before_left, left, x);
                } else {
                    const int left_to_go = (int)lane - 16 * b;
                    int v = byte_value(left, 3), last = byte_value(before_left, 3);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int here = byte_value(before[i >> 2], i & 3);
                        const int acc = mul_i24(w_left, v) + (mul_i24(w_before, here) + (mul_i24(w_left_before, last) + bias));
                        v = diag_value(acc, byte_value(e[i >> 2], i & 3));
                        v = i >= left_to_go ? v : 0;
                        x[i >> 2] |= (uint32_t)v << (8 * (i & 3));
                        last = here;
                    }
                }
                left = x[3];
                before_left = before[3];
                if (kCh == 1) {
                    u32x4 o;
                    o.x = x[0];
                    o.y = x[1];
                    o.z = x[2];
                    o.w = x[3];
                    green[b & 1][lane] = o;
                } else {  // all three channels are here: the window's pixels take the place of its residuals
                    window_pixels(rd, gr, x, d);
#pragma unroll
                    for (int i = 0; i < 3; ++i) raw[slot][i][lane] = d[i];
                }
                slot = slot + 1u == (uint32_t)kStripSlots ? 0u : slot + 1u;
            }
        };
        if (role == 1u)
            channel(std::false_type{});
        else
            channel(std::true_type{});
    } else if (role == 3u) {
        fetch_windows<kStripSlots>(a, res, raw, strip, band_row0, lane, times);
    } else if (role == 4u) {
        store_windows<kStripSlots>(a, img, raw, strip, band_row0, lane, times, lead, 3);
    } else {  // ---- red of the row above the band, which is in the image
        // Block q, word k of the band above holds columns 16 q + 4 k - 63 .. + 3 of its last row.  Red's block
        // b needs blocks b + 3 and b + 4.  Threads 0 .. 31 fetch eight blocks every four intervals, an interval or more ahead.
        if (band == 0u) {
            for (int time = 0; time < times; ++time) interval_barrier();
            return;
        }
        const uint8_t *above_row = img + (size_t)((strip * a.strip_rows + band_row0 - 1u) * a.w) * 3u;
        const int k = (int)(lane & 3u);
        // (The four bytes stay apart until they are wanted: gathered where they are asked for, every fourth interval waits for
        // the loads, at the cost of all six wavefronts.  256 images of 236 x 2047 one band at a time 347 us, now 329.)
        uint32_t v[4] = {};
        int base = 0, got = 0;  // blocks asked for from `base` on; blocks in LDS so far
        for (int time0 = 0; time0 < times; time0 += 4) {
            interval_barrier();
            const int now = time0 - lead;
            if (time0 != 0) {
                const int upto = min(min(base + 8, blocks), now + kDiagCarry), q = base + (int)(lane >> 2);
                if (lane < 32u && q < upto) carry[q % kDiagCarry][k] = v[0] | v[1] << 8 | v[2] << 16 | v[3] << 24;
                got = max(got, upto);
            }
            base = got;
            const int q = min(base + (int)((lane & 31u) >> 2), blocks - 1);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int col = 16 * q + 4 * k + i - 63;
                v[i] = above_row[3 * min(max(col, 0), (int)a.w - 1)];  // (outside the row: not used)
            }
#pragma unroll
            for (int j = 1; j < 4; ++j) interval_barrier();
        }
    }
}

// ---- bands together
// Sixteen steps of a channel, four a piece of assembly, a register a value.  The steps are written out for
// three reasons.  The prediction, the residual's byte and the mod 256 are one instruction (sub-dword operands pick the
// upper half of the sum and a byte of the window as it was loaded, and only the low byte of the value's register
// is written).  An instruction that reads a register whose byte the instruction before it wrote, or a
// neighbour's register less than three instructions after it was written, would get old values: the order keeps
// both apart.  And nothing of the neighbour's value has to be moved before it is used:
//
// Red, six instructions a step: the value above is moved over from the thread above as it is wanted, and is
// the one above to the left of the next step.  Thread 0 has no thread above, the move leaves its lane alone, and
// this holds the value of the row above the band beforehand.
// (With four values packed to a register, which took a byte picked for every product, a step took eight.)
//
// `MASK`: in the first four blocks a thread gets through the column before its row's first, where its
// value has to read as zero; a bit that moves up by one thread a step says whose turn it is.
#define PILC_BAND_RED_STEP(X, L, U, UL, E, B, MASK)                                                       \
    "v_mad_i32_i24 %[t], " UL ", %[w_upleft], %[bias]\n"                                            \
    "v_mad_i32_i24 %[t], " L ", %[w_left], %[t]\n"                                                  \
    "v_mov_b32_dpp " U ", " L " wave_shr:1 row_mask:0xf bank_mask:0xf\n"                            \
    "v_mad_i32_i24 %[t], " U ", %[w_up], %[t]\n"                                                    \
    "v_med3_i32 %[t], %[t], 0, %[most]\n"                                                           \
    "v_add_u32_sdwa " X ", %[t], %[" E "] dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:WORD_1 src1_sel:BYTE_" #B "\n" MASK(X)
// Green and blue, five instructions a step, from the channel decoded before.
#define PILC_BAND_ROW_STEP(X, L, V, VL, E, B, MASK)                                                       \
    "v_mad_i32_i24 %[t], %[" V "], %[w_before], %[bias]\n"                                          \
    "v_mad_i32_i24 %[t], %[" VL "], %[w_left_before], %[t]\n"                                       \
    "v_mad_i32_i24 %[t], " L ", %[w_left], %[t]\n"                                               \
    "v_med3_i32 %[t], %[t], 0, %[most]\n"                                                           \
    "v_add_u32_sdwa " X ", %[t], %[" E "] dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:WORD_1 src1_sel:BYTE_" #B "\n" MASK(X)
#define PILC_NO_MASK(X) ""
#define PILC_MASK(X)                                                                                 \
    "s_lshl_b64 %[mask], %[mask], 1\n"                                                              \
    "v_cndmask_b32_e64 " X ", " X ", %[zero], %[mask]\n"

// The sixteen values, and those above them, have fixed registers: four of them are one operand of a load or store
// of sixteen bytes, whose parts the assembly could not name otherwise, and as operands of their own they
// cost a move each.
struct RedWeights {
    int upleft, up, left, bias;
};
#define PILC_BAND_RED_FOUR(MASK, X0, X1, X2, X3, L, U0, U1, U2, U3)                                       \
    PILC_BAND_RED_STEP(X0, L, U0, "%[ul]", "e0", 0, MASK)                                                \
    PILC_BAND_RED_STEP(X1, X0, U1, U0, "e0", 3, MASK)                                                    \
    PILC_BAND_RED_STEP(X2, X1, U2, U1, "e1", 2, MASK)                                                    \
    PILC_BAND_RED_STEP(X3, X2, U3, U2, "e2", 1, MASK)
#define PILC_RED_INPUTS                                                                              \
    [ul] "v"(last_up), [e0] "v"(e0), [e1] "v"(e1), [e2] "v"(e2), [w_upleft] "v"(w.upleft), [w_up] "v"(w.up),      \
        [w_left] "v"(w.left), [bias] "v"(w.bias), [most] "v"(0xFFFFFF)
#define PILC_RED_GROUP(G, XQ, PQ, UQ, ...)                                                           \
    if (kG == G) {                                                                                  \
        if (kFirst)                                                                                 \
            asm(PILC_BAND_RED_FOUR(PILC_MASK, __VA_ARGS__)                                               \
                : "+{" XQ "}"(x[G]), "+{" UQ "}"(above), [t] "=&v"(t), [mask] "+s"(mask)            \
                : "{" PQ "}"(x[(G + 3) & 3]), PILC_RED_INPUTS, [zero] "v"(zero) : "scc");           \
        else                                                                                        \
            asm(PILC_BAND_RED_FOUR(PILC_NO_MASK, __VA_ARGS__)                                            \
                : "+{" XQ "}"(x[G]), "+{" UQ "}"(above), [t] "=&v"(t)                               \
                : "{" PQ "}"(x[(G + 3) & 3]), PILC_RED_INPUTS);                                     \
    }
// `x`: all sixteen values; group kG of four is decoded here, from the group before it, or, for the first, from the
// last of the block before.  `above`: the values above thread 0; `last_up`: the value above the one before these.
// `e`: the window's three dwords of these pixels.
template <int kG, bool kFirst>
__device__ __forceinline__ void red_four(const RedWeights &w, u32x4 (&x)[4], u32x4 above, uint32_t &last_up,
                                         const uint32_t e0, const uint32_t e1, const uint32_t e2, uint32_t zero,
                                         unsigned long long &mask)
{
    int t;
    PILC_RED_GROUP(0, "v[64:67]", "v[76:79]", "v[48:51]", "v64", "v65", "v66", "v67", "v79", "v48", "v49", "v50", "v51")
    PILC_RED_GROUP(1, "v[68:71]", "v[64:67]", "v[52:55]", "v68", "v69", "v70", "v71", "v67", "v52", "v53", "v54", "v55")
    PILC_RED_GROUP(2, "v[72:75]", "v[68:71]", "v[56:59]", "v72", "v73", "v74", "v75", "v71", "v56", "v57", "v58", "v59")
    PILC_RED_GROUP(3, "v[76:79]", "v[72:75]", "v[60:63]", "v76", "v77", "v78", "v79", "v75", "v60", "v61", "v62", "v63")
    last_up = above.w;
}
#undef PILC_RED_GROUP
#undef PILC_RED_INPUTS
#undef PILC_BAND_RED_FOUR

struct RowWeights {
    int left, left_before, before, bias;
};
#define PILC_GREEN_FOUR(MASK, X0, X1, X2, X3, L)                                                     \
    PILC_BAND_ROW_STEP(X0, L, "v0", "vl", "e0", 1, MASK)                                                 \
    PILC_BAND_ROW_STEP(X1, X0, "v1", "v0", "e1", 0, MASK)                                                \
    PILC_BAND_ROW_STEP(X2, X1, "v2", "v1", "e1", 3, MASK)                                                \
    PILC_BAND_ROW_STEP(X3, X2, "v3", "v2", "e2", 2, MASK)
#define PILC_BLUE_FOUR(MASK, X0, X1, X2, X3, L)                                                      \
    PILC_BAND_ROW_STEP(X0, L, "v0", "vl", "e0", 2, MASK)                                                 \
    PILC_BAND_ROW_STEP(X1, X0, "v1", "v0", "e1", 1, MASK)                                                \
    PILC_BAND_ROW_STEP(X2, X1, "v2", "v1", "e2", 0, MASK)                                                \
    PILC_BAND_ROW_STEP(X3, X2, "v3", "v2", "e2", 3, MASK)
#define PILC_ROW_INPUTS                                                                              \
    [v0] "v"(v.x), [v1] "v"(v.y), [v2] "v"(v.z), [v3] "v"(v.w), [vl] "v"(vl), [e0] "v"(e0), [e1] "v"(e1), [e2] "v"(e2), \
        [w_left] "v"(w.left), [w_left_before] "v"(w.left_before), [w_before] "v"(w.before), [bias] "v"(w.bias),         \
        [most] "v"(0xFFFFFF)
#define PILC_ROW_GROUP(G, FOUR, XQ, PQ, ...)                                                         \
    if (kG == G) {                                                                                  \
        if (kFirst)                                                                                 \
            asm(FOUR(PILC_MASK, __VA_ARGS__)                                                        \
                : "+{" XQ "}"(x[G]), [t] "=&v"(t), [mask] "+s"(mask)                                \
                : "{" PQ "}"(x[(G + 3) & 3]), PILC_ROW_INPUTS, [zero] "v"(0) : "scc");              \
        else                                                                                        \
            asm(FOUR(PILC_NO_MASK, __VA_ARGS__)                                                     \
                : "+{" XQ "}"(x[G]), [t] "=&v"(t)                                                   \
                : "{" PQ "}"(x[(G + 3) & 3]), PILC_ROW_INPUTS);                                     \
    }
// Likewise for channel kCh; `v`: the values of the channel decoded before, `vl`: the one before these.
template <int kCh, int kG, bool kFirst>
__device__ __forceinline__ void row_four(const RowWeights &w, u32x4 (&x)[4], const u32x4 v, const uint32_t vl,
                                         const uint32_t e0, const uint32_t e1, const uint32_t e2, unsigned long long &mask)
{
    int t;
    if (kCh == 1) {
        PILC_ROW_GROUP(0, PILC_GREEN_FOUR, "v[64:67]", "v[76:79]", "v64", "v65", "v66", "v67", "v79")
        PILC_ROW_GROUP(1, PILC_GREEN_FOUR, "v[68:71]", "v[64:67]", "v68", "v69", "v70", "v71", "v67")
        PILC_ROW_GROUP(2, PILC_GREEN_FOUR, "v[72:75]", "v[68:71]", "v72", "v73", "v74", "v75", "v71")
        PILC_ROW_GROUP(3, PILC_GREEN_FOUR, "v[76:79]", "v[72:75]", "v76", "v77", "v78", "v79", "v75")
    } else {
        PILC_ROW_GROUP(0, PILC_BLUE_FOUR, "v[64:67]", "v[76:79]", "v64", "v65", "v66", "v67", "v79")
        PILC_ROW_GROUP(1, PILC_BLUE_FOUR, "v[68:71]", "v[64:67]", "v68", "v69", "v70", "v71", "v67")
        PILC_ROW_GROUP(2, PILC_BLUE_FOUR, "v[72:75]", "v[68:71]", "v72", "v73", "v74", "v75", "v71")
        PILC_ROW_GROUP(3, PILC_BLUE_FOUR, "v[76:79]", "v[72:75]", "v76", "v77", "v78", "v79", "v75")
    }
}
#undef PILC_ROW_GROUP
#undef PILC_GREEN_FOUR
#undef PILC_BLUE_FOUR
#undef PILC_ROW_INPUTS
#undef PILC_BAND_RED_STEP
#undef PILC_BAND_ROW_STEP
#undef PILC_MASK
#undef PILC_NO_MASK

// The twelve bytes of four pixels from their channels (the low bytes of the registers).
__device__ __forceinline__ void four_pixels(const u32x4 r, const u32x4 g, const u32x4 b, uint32_t (&w)[3])
{
    auto perm = [](uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); };
    w[0] = perm(perm(r.y, b.x, 0x04000000u), perm(g.x, r.x, 0x0C0C0400u), 0x07060100u);
    w[1] = perm(perm(g.z, r.z, 0x04000000u), perm(b.y, g.y, 0x0C0C0400u), 0x07060100u);
    w[2] = perm(perm(b.w, g.w, 0x04000000u), perm(r.w, b.z, 0x0C0C0400u), 0x07060100u);
}

__device__ __forceinline__ uint32_t dword_of(const u32x4 (&d)[3], int i)
{
    const u32x4 v = d[i >> 2];
    return (i & 3) == 0 ? v.x : (i & 3) == 1 ? v.y : (i & 3) == 2 ? v.z : v.w;
}

constexpr uint32_t kDiagRawBytes = kDiagSlots * 3 * 64 * 16;  // the dynamic part of its LDS; the rest is 30 KB
constexpr uint32_t kDiagAloneBytes = 56 * 1024;                // as much as leaves no room for a second workgroup

__global__ __launch_bounds__(64 * 6) void k_twar_inverse_bands(TwarK p, Diag a, const uint8_t *__restrict__ res,
                                                              uint8_t *__restrict__ img)
{
    // (The windows in dynamic memory: told of all 55 KB, of which a compute unit holds two, the compiler gives the kernel as
    // many registers as leave a SIMD three wavefronts, and two workgroups of six then do not always fit.)
    extern __shared__ u32x4 diag_lds[];
    u32x4(*const raw)[3][64] = reinterpret_cast<u32x4(*)[3][64]>(diag_lds);  // [slot][third of the window][row]: residuals, then pixels
    __shared__ u32x4 red[5][4][64];         // [block mod 5][four of its values][row]: blue is four blocks behind
    __shared__ u32x4 green[2][4][64];       // [block mod 2][four of its values][row]
    __shared__ u32x4 carry[kDiagCarry][4];  // [block + 4, mod kDiagCarry][four of them]: red of the row above the band
    __shared__ uint32_t s_id;
    if (threadIdx.x == 0u) s_id = atomicAdd(a.ticket, 1u) - a.first_ticket;
    __syncthreads();
    const uint32_t id = s_id;
    const uint32_t in_launch = id / a.strips, in_strip = id - in_launch * a.strips, band = a.band0 + in_launch;
    const unsigned long long strip = a.strip0 + in_strip;
    const uint32_t place = in_strip * a.bands + in_launch;  // of this band's words
    const uint32_t role = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t band_row0 = band * 64u;       // row of the strip
    const int blocks = (int)a.blocks;
    // intervals between barriers, a multiple of 4: a window is fetched kDiagAhead intervals before it is put
    // into LDS, red takes it up in the next and decodes it in the one after; green takes it up in the next and
    // decodes it in the one after, blue likewise, and then it is stored
    const int lead = kDiagAhead + 2;
    const int times = (lead + blocks + 5 + 3) & ~3;

    if (role == 0u) {  // ---- red
        const uint32_t u = band_row0 + lane;
        const bool top = u % a.h == 0u;  // the row above is padding: its two weights are zero here
        RedWeights w = {top ? 0 : diag_weight(p.w[0][0]), top ? 0 : diag_weight(p.w[0][1]), diag_weight(p.w[0][2]),
                        diag_bias(p.bias[0])};
        // (in vector registers: from scalar ones they would be copied at every use)
        asm volatile("" : "+v"(w.left), "+v"(w.bias));
        const bool passes_on = a.withhold == 0u && band + 1u < a.band0 + a.bands;
        uint32_t *out = a.words + (size_t)place * (16u * a.blocks);
        const __amdgpu_buffer_rsrc_t out_buffer =
            __builtin_amdgcn_make_buffer_rsrc(out, 0, 64 * blocks, 0x00020000);
        // the values, with the mark of this launch above them
        const uint32_t mark = a.mark << 24;
        u32x4 x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = u32x4{mark, mark, mark, mark};
        uint32_t last_up = 0;
        unsigned long long mask = 1ull;
        uint32_t slot = 0;
        u32x4 d[2][3] = {};
        for (int time0 = 0; time0 < times; time0 += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                interval_barrier();
                const int b = time0 + j - lead;
                if (b < -1 || b >= blocks) continue;
                // the next block's residuals, which are wanted after the next barrier
#pragma unroll
                for (int i = 0; i < 3; ++i) d[1 - j][i] = raw[slot][i][lane];
                slot = slot + 1u == (uint32_t)kDiagSlots ? 0u : slot + 1u;
                if (b < 0) continue;
                // thread 0 is at columns 16 b .. + 15; column v of the row above is value v + 63 of its blocks
                const uint32_t c = (uint32_t)(b + 4) % kDiagCarry;
                auto steps = [&](auto first) {
                    constexpr bool kFirst = decltype(first)::value;
#define PILC_RED_GROUP(G)                                                                            \
    red_four<G, kFirst>(w, x, carry[c][G], last_up, dword_of(d[j], 3 * G), dword_of(d[j], 3 * G + 1),   \
                        dword_of(d[j], 3 * G + 2), mark, mask);                                     \
    red[(uint32_t)b % 5u][G][lane] = x[G];
                    PILC_RED_GROUP(0)
                    PILC_RED_GROUP(1)
                    PILC_RED_GROUP(2)
                    PILC_RED_GROUP(3)
#undef PILC_RED_GROUP
                };
                if (b >= 4)
                    steps(std::false_type{});
                else
                    steps(std::true_type{});
                if (passes_on && lane == 63u) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)  // at device scope
                        __builtin_amdgcn_raw_buffer_store_b128(x[k], out_buffer, 64 * b + 16 * k, 0, kDeviceScope);
                }
            }
        }
    } else if (role == 1u || role == 2u) {  // ---- green and blue
        auto channel = [&](auto blue) {
            constexpr int kCh = decltype(blue)::value ? 2 : 1;
            // green from the left green, the left red and the red here; blue likewise from blue and green
            RowWeights w = {diag_weight(p.w[kCh][0]), diag_weight(p.w[kCh][1]), diag_weight(p.w[kCh][2]),
                            diag_bias(p.bias[kCh])};
            // (in vector registers: from scalar ones they would be copied at every use)
            asm volatile("" : "+v"(w.left), "+v"(w.left_before), "+v"(w.before), "+v"(w.bias));
            u32x4 x[4] = {};
            uint32_t before_left = 0;  // the last value of the channel decoded before this one
            unsigned long long mask = 1ull;
            uint32_t slot = 0, next_slot = 0;
            u32x4 d[2][3] = {}, v[2][4] = {};  // a block's residuals and the channel before, asked for an interval ahead
            auto interval = [&](int time, auto odd, auto first) {
                constexpr bool kFirst = decltype(first)::value;
                constexpr int j = decltype(odd)::value ? 1 : 0;
                interval_barrier();
                const int b = time - lead - 2 * kCh;
                if (b < -1 || b >= blocks) return;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[1 - j][k] = kCh == 1 ? red[(uint32_t)(b + 1) % 5u][k][lane] : green[(b + 1) & 1][k][lane];
#pragma unroll
                for (int i = 0; i < 3; ++i) d[1 - j][i] = raw[next_slot][i][lane];
                next_slot = next_slot + 1u == (uint32_t)kDiagSlots ? 0u : next_slot + 1u;
                if (b < 0) return;
                u32x4 r[4];
                if (kCh == 2)
#pragma unroll
                    for (int k = 0; k < 4; ++k) r[k] = red[(uint32_t)b % 5u][k][lane];
                uint32_t pixels[12];
#define PILC_ROW_FOUR(G, VL)                                                                         \
    row_four<kCh, G, kFirst>(w, x, v[j][G], VL, dword_of(d[j], 3 * G), dword_of(d[j], 3 * G + 1),       \
                             dword_of(d[j], 3 * G + 2), mask);                                      \
    if (kCh == 1) {                                                                                 \
        green[b & 1][G][lane] = x[G];                                                               \
    } else {                                                                                        \
        uint32_t q[3];                                                                              \
        four_pixels(r[G], v[j][G], x[G], q);                                                        \
        pixels[3 * G] = q[0];                                                                       \
        pixels[3 * G + 1] = q[1];                                                                   \
        pixels[3 * G + 2] = q[2];                                                                   \
    }
                PILC_ROW_FOUR(0, before_left)
                PILC_ROW_FOUR(1, v[j][0].w)
                PILC_ROW_FOUR(2, v[j][1].w)
                PILC_ROW_FOUR(3, v[j][2].w)
#undef PILC_ROW_FOUR
                if (kCh == 2) {  // all three channels are here: the window's pixels take the place of its residuals
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        raw[slot][i][lane] = u32x4{pixels[4 * i], pixels[4 * i + 1], pixels[4 * i + 2], pixels[4 * i + 3]};
                    slot = slot + 1u == (uint32_t)kDiagSlots ? 0u : slot + 1u;
                }
                before_left = v[j][3].w;
            };
            int time = 0;
            for (; time < min(times, lead + 2 * kCh + 4); time += 2) {
                interval(time, std::false_type{}, std::true_type{});
                interval(time + 1, std::true_type{}, std::true_type{});
            }
            for (; time < times; time += 2) {
                interval(time, std::false_type{}, std::false_type{});
                interval(time + 1, std::true_type{}, std::false_type{});
            }
        };
        if (role == 1u)
            channel(std::false_type{});
        else
            channel(std::true_type{});
    } else if (role == 3u) {
        fetch_windows<kDiagSlots>(a, res, raw, strip, band_row0, lane, times);
    } else if (role == 4u) {
        store_windows<kDiagSlots>(a, img, raw, strip, band_row0, lane, times, lead, 5);
    } else {  // ---- the row above the band
        // Block q, value k of the band above is column 16 q + k - 63 of its last row.  Red's block
        // b needs the last two values of block b + 3 and b + 4 but for its last.  A thread asks for two values, the
        // wavefront for eight blocks at a time, and leaves what has arrived in `carry`.
        const bool some = band != 0u, first_of_launch = band == a.band0;
        // (the first band of a launch: the band above is done, its last row is in the image)
        const uint8_t *above_row =
            img + (size_t)((strip * a.strip_rows + (some ? band_row0 - 1u : 0u)) * a.w) * 3u;
        const unsigned long long *words = reinterpret_cast<const unsigned long long *>(
            a.words + (size_t)(place - (some && !first_of_launch ? 1u : 0u)) * (16u * a.blocks));
        int got = 0;  // blocks in LDS so far
        bool gave_up = false;
        auto follow = [&](auto in_image) {
            auto ask = [&](int base) -> unsigned long long {
                const int q = min(base + (int)(lane >> 3), blocks - 1), k = (int)(lane & 7u);
                if (!decltype(in_image)::value)
                    return __hip_atomic_load(words + 8 * q + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                unsigned long long v = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int col = 16 * q + 2 * k + i - 63;
                    const uint32_t x = above_row[3 * min(max(col, 0), (int)a.w - 1)];
                    // (left of the row is padding; what is right of it is not used)
                    v |= (unsigned long long)((a.mark << 24) | (col < 0 ? 0u : x)) << (32 * i);
                }
                return v;
            };
            // `now`: the block red is at; a block goes into LDS once the one it replaces has been used
            auto take = [&](unsigned long long v, int base, int now) {
                const uint32_t v0 = (uint32_t)v, v1 = (uint32_t)(v >> 32);
                const unsigned long long missing = ~__ballot((v0 >> 24) == a.mark && (v1 >> 24) == a.mark);
                const int whole = missing == 0u ? 8 : (__ffsll(missing) - 1) >> 3;
                const int upto = min(min(base + whole, blocks), now + kDiagCarry);
                const int q = base + (int)(lane >> 3);
                if (q >= got && q < upto) {
                    // value number v is above thread 0 at step v - 63
                    uint32_t *up = reinterpret_cast<uint32_t *>(&carry[0][0]);
                    const uint32_t at = 16u * (uint32_t)q + 2u * (lane & 7u), size = 16u * kDiagCarry;
                    up[(at + 1u) % size] = v0;
                    up[(at + 2u) % size] = v1;
                }
                got = max(got, upto);
            };
            unsigned long long asked[kDiagPolls] = {};
            int asked_at[kDiagPolls] = {};
            for (int time0 = 0; time0 < times; time0 += kDiagPolls) {
#pragma unroll
                for (int j = 0; j < kDiagPolls; ++j) {
                    interval_barrier();
                    if (decltype(in_image)::value && j != 0) continue;  // eight blocks every four intervals will do
                    const int now = time0 + j - lead;
                    take(asked[j], asked_at[j], now);
                    // what red reads after the next barrier (or by the time this is looked at again)
                    const int need = min(now + (decltype(in_image)::value ? 6 + kDiagPolls - 1 : 6), blocks);
                    if (got < need && !gave_up) {
                        const unsigned long long since = wall_clock64();
                        for (;;) {
                            const int base = got;
                            take(ask(base), base, now);
                            if (got >= need) break;
                            if (__hip_atomic_load(a.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
                                gave_up = true;
                                break;
                            }
                            if (wall_clock64() - since > a.wait_ticks) {
                                gave_up = true;
                                __hip_atomic_store(a.abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                raise_code(a.report, ST_TIMEOUT);
                                break;
                            }
                            __builtin_amdgcn_s_sleep(8);
                        }
                    }
                    asked_at[j] = got;
                    asked[j] = ask(got);
                }
            }
        };
        if (!some) {
            for (int time = 0; time < times; ++time) interval_barrier();
        } else if (first_of_launch) {
            follow(std::true_type{});
        } else {
            follow(std::false_type{});
        }
    }
}

// The words that bands pass on, with the ticket and the abort word: a few sets in device globals (the
// entry points take no workspace), handed out under a lock so that concurrent calls do not share
// one; a call that finds none free goes a band at a time, a launch each, every band reading the row
// above it from the image.
//
// A set is not cleared between calls: the words of a launch carry its mark, of which there are 255, and its
// workgroups count on from where the ticket stands.  It is cleared before a mark comes back, and after a call that
// gave up or failed.  (Cleared by a kernel before each launch, and with the abort word copied back instead of raised in
// pinned memory, 30 frames of 1080 x 1920 took 12 us more.)
constexpr uint32_t kTileManyImages = 1024;  // a wavefront for every SIMD
constexpr int kBandSlots = 4;
constexpr uint32_t kBandMarks = 255;
struct BandSet {
    uint32_t words[kBandWords];
    uint32_t ticket, abort_word;
    Report report;  // of a call that finds no place in pinned memory
};
struct BandState {  // what the host knows of a set; its holder's alone while it is taken
    bool taken = false, stale = false;
    uint32_t mark = 0, tickets = 0;  // of the last launch; workgroups that have taken a ticket so far
};
static __device__ BandSet g_band_sets[kBandSlots];
struct BandDevice {
    BandSet *sets = nullptr;
    BandState state[kBandSlots];
};
static std::mutex g_band_mutex;
static std::map<int, BandDevice> g_band_devices;

__global__ __launch_bounds__(256) void k_band_clear(BandSet *set)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < kBandWords; i += gridDim.x * blockDim.x) set->words[i] = 0u;
    if (blockIdx.x == 0u && threadIdx.x == 0u) set->ticket = set->abort_word = 0u;
}

// A free set on the current device (null if none), given back at the end.
class BandLease {
public:
    BandLease() = default;
    ~BandLease()
    {
        if (!state_) return;
        std::lock_guard<std::mutex> lock(g_band_mutex);
        state_->taken = false;
    }
    BandLease(const BandLease &) = delete;
    BandLease &operator=(const BandLease &) = delete;
    void acquire()
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return;
        std::lock_guard<std::mutex> lock(g_band_mutex);
        BandDevice &d = g_band_devices[dev];
        if (!d.sets) {
            void *ptr = nullptr;
            if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_band_sets)) != hipSuccess) return;
            d.sets = static_cast<BandSet *>(ptr);
        }
        for (int i = 0; i < kBandSlots; ++i)
            if (!d.state[i].taken) {
                set_ = d.sets + i;
                state_ = &d.state[i];  // (a map's elements stay where they are)
                state_->taken = true;
                clear_ = state_->stale;
                state_->stale = true;  // until the call says that all went well
                return;
            }
    }
    BandSet *set() const { return set_; }
    // The mark of the next launch, of `workgroups`, and where the ticket stands before it.
    void next_launch(uint32_t workgroups, hipStream_t stream, uint32_t *mark, uint32_t *first_ticket)
    {
        if (clear_ || state_->mark == kBandMarks) {
            k_band_clear<<<1024, 256, 0, stream>>>(set_);
            state_->mark = state_->tickets = 0u;
            clear_ = false;
        }
        *mark = ++state_->mark;
        *first_ticket = state_->tickets;
        state_->tickets += workgroups;
    }
    void all_went_well() { state_->stale = false; }

private:
    BandSet *set_ = nullptr;
    BandState *state_ = nullptr;
    bool clear_ = false;
};

static int make_twar(const pilc_twar_params *in, uint32_t n, uint32_t h, uint32_t w, TwarK *k)
{
    if (!in || n == 0 || h == 0 || w == 0) return PILC_E_ARG;
    if ((uint64_t)n * h * w * 3 + 4096 >= (1ull << 40)) return PILC_E_TOO_LARGE;
    if (w > 65535u) return PILC_E_TOO_LARGE;
    for (int c = 0; c < 3; ++c) {
        for (int j = 0; j < 3; ++j) k->w[c][j] = in->w[c][j];
        // the sum of three products and the bias must stay inside 32 bits: |w| <= 2^15, values <= 255
        if (in->bias[c] > (1 << 30) || in->bias[c] < -(1 << 30)) return PILC_E_ARG;
        k->bias[c] = in->bias[c];
    }
    return PILC_OK;
}

}  // namespace pilc

extern "C" {

int pilc_twar_forward(uint32_t n, uint32_t h, uint32_t w, const uint8_t *img_dev,
                      const pilc_twar_params *params_host, uint8_t *res_dev, void *hip_stream)
{
    TwarK k;
    int rc = make_twar(params_host, n, h, w, &k);
    if (rc != PILC_OK) return rc;
    if (!img_dev || !res_dev || img_dev == res_dev) return PILC_E_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    const uint64_t rows = (uint64_t)n * h;
    if (rows >= (1ull << 31)) return PILC_E_TOO_LARGE;
    Timer timer(stream);
    const uint64_t groups = rows * (w / 4);
    if (w % 4 == 0 && ((((uintptr_t)img_dev) | ((uintptr_t)res_dev)) & 3) == 0 && groups < (1ull << 32))
        k_twar_forward4<<<(uint32_t)((groups + 255) / 256), 256, 0, stream>>>(
            k, (uint32_t)groups, FastDiv::make(h), FastDiv::make(w / 4), reinterpret_cast<const uint32_t *>(img_dev),
            reinterpret_cast<uint32_t *>(res_dev));
    else {
        // whole rows of less than 2^31 pixels a launch
        const uint32_t most = std::max(1u, (1u << 31) / w - 1u);
        for (uint64_t row = 0; row < rows; row += most) {
            const uint32_t pixels = (uint32_t)std::min<uint64_t>(most, rows - row) * w;
            k_twar_forward_any<<<(uint32_t)ceil_div64(pixels, 1024), 256, 0, stream>>>(
                k, (uint32_t)row, pixels, FastDiv::make(h), FastDiv::make(w), img_dev, res_dev);
        }
    }
    timer.mark("k_twar_forward");
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(stream));
    timer.finish();
    return PILC_OK;
}

// pilc_twar_inverse along the diagonals.
static int twar_inverse_diag(uint32_t n, uint32_t h, uint32_t w, const uint8_t *res_dev, const TwarK &k,
                             uint8_t *img_dev, hipStream_t stream, Timer &timer)
{
    Diag a = {};
    a.h = h;
    a.w = w;
    a.rows = (unsigned long long)n * h;
    a.strip_rows = h <= 64u ? 64u / h * h : h;
    a.blocks = (w + 63u + 15u) / 16u;
    const uint64_t strips = (a.rows + a.strip_rows - 1u) / a.strip_rows;
    const uint32_t bands = (a.strip_rows + 63u) / 64u;
    BandLease lease;
    if (bands > 1u && !bands_one_at_a_time(strips, bands, a.blocks)) lease.acquire();
    BandSet *const set = lease.set();
    std::optional<CallReport> report;
    const BandLaunch launch = band_launches(strips, bands, a.blocks);
    const uint32_t together = set ? launch.bands : 1u;
    const uint64_t most_strips = set ? launch.strips : 1u << 20;
    int dev = 0, khz = 0;
    const unsigned long long wait = g_one_pass_wait.load(std::memory_order_relaxed);
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
        khz = 100000;
    a.wait_ticks = wait ? wait : 2000ull * (unsigned long long)khz;
    a.withhold = (uint32_t)g_one_pass_withhold.load(std::memory_order_relaxed);
    if (set) {
        report.emplace(&set->report, stream, true);
        a.words = set->words;
        a.ticket = &set->ticket;
        a.abort_word = &set->abort_word;
        a.report = report->dev();
    }
    for (uint64_t s = 0; s < strips; s += most_strips) {
        const uint32_t here = (uint32_t)std::min<uint64_t>(most_strips, strips - s);
        for (uint32_t b = 0; b < bands; b += together) {
            a.strip0 = s;
            a.strips = here;
            a.band0 = b;
            a.bands = std::min(together, bands - b);
            if (a.bands > 1u) {
                lease.next_launch(here * a.bands, stream, &a.mark, &a.first_ticket);
                const uint32_t lds = bands_alone_on_a_unit(here, a.bands, a.blocks) ? kDiagAloneBytes : kDiagRawBytes;
                k_twar_inverse_bands<<<here * a.bands, 64 * 6, lds, stream>>>(k, a, res_dev, img_dev);
            } else {
                k_twar_inverse_strips<<<here, bands > 1u ? 64 * 6 : 64 * 5, 0, stream>>>(k, a, res_dev, img_dev);
            }
        }
    }
    timer.mark("k_twar_inverse");
    HIP_TRY(hipGetLastError());
    Report seen = {};
    if (set)
        HIP_TRY(report->wait(&seen));
    else
        HIP_TRY(hipStreamSynchronize(stream));
    timer.finish();
    if (raised_code(seen) != ST_OK) return status_to_error(raised_code(seen));
    if (set) lease.all_went_well();
    return PILC_OK;
}

// Whether images of more than 64 rows whose rows fit a tile go 64 rows after 64 through the tile kernel.  That takes
// a wavefront an image, whose time does not change until every SIMD has one; the diagonal kernel takes a
// workgroup an image and slows down with every further one on a compute unit.  Rows of less than 16 pixels are
// too short for the diagonal kernel; tiles copied by single bytes are slower.  Tile against diagonal, us,
// images of 500 rows:
//   images    20 columns   28 columns   40 columns   60 columns   17 columns (single bytes)
//     500     127  131     146  138     169  142     211  155     174  128
//     700     128  152     146  160     170  166     211  181     174  147
//     850     128  204     147  218     170  224     212  246     175  197
//    1000     128  207     147  221     171  227     213  250     176  199
// and the last band of an image costs the tile kernel less if it has few rows: 700 images of 65 rows 44 against 47 us
// at 40 columns.
static bool tall_in_tiles(uint32_t n, uint32_t h, uint32_t w, int elem)
{
    if (w < 16u || n >= kTileManyImages) return true;
    const uint32_t each = (n + 255u) / 256u;  // workgroups of the diagonal kernel on a compute unit
    const uint32_t most = elem == 1 ? (each >= 4u ? 28u : 0u) : each >= 4u ? 84u : each == 3u ? 36u : each == 2u ? 24u : 0u;
    return most != 0u && w <= most + (h <= 96u ? 12u : 0u);
}

int pilc_twar_inverse(uint32_t n, uint32_t h, uint32_t w, const uint8_t *res_dev,
                      const pilc_twar_params *params_host, uint8_t *img_dev, void *hip_stream)
{
    TwarK k;
    int rc = make_twar(params_host, n, h, w, &k);
    if (rc != PILC_OK) return rc;
    if (!img_dev || !res_dev || img_dev == res_dev) return PILC_E_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    Timer timer(stream);
    const uint32_t last_bytes = (w + 15u) & ~15u;
    const size_t tile_lds = (size_t)kTwarWaves * (last_bytes + 64u * (size_t)w * 3u);
    // the element of the tile copies: every group (whole images, or a band of 64 rows) must start
    // and end on a multiple of it
    const uint32_t row_bytes = w * 3u;
    const uintptr_t both = (uintptr_t)img_dev | (uintptr_t)res_dev;
    const bool whole_images = h <= 64;
    const uint32_t unit_bytes = whole_images ? h * row_bytes : row_bytes;
    const int elem = unit_bytes % 16u == 0u && (both & 15) == 0 ? 16 : unit_bytes % 4u == 0u && (both & 3) == 0 ? 4 : 1;
    if (tile_lds > 64 * 1024 || (!whole_images && !tall_in_tiles(n, h, w, elem)))
        return twar_inverse_diag(n, h, w, res_dev, k, img_dev, stream, timer);
    const uint32_t per = h <= 64 ? 64 / h : 1;
    const uint32_t groups = (n + per - 1) / per;
    const uint32_t blocks = (groups + kTwarWaves - 1) / kTwarWaves;
    if (elem == 16)
        k_twar_inverse<u32x4><<<blocks, 64 * kTwarWaves, tile_lds, stream>>>(k, n, h, w, last_bytes, res_dev, img_dev);
    else if (elem == 4)
        k_twar_inverse<uint32_t><<<blocks, 64 * kTwarWaves, tile_lds, stream>>>(k, n, h, w, last_bytes, res_dev, img_dev);
    else
        k_twar_inverse<uint8_t><<<blocks, 64 * kTwarWaves, tile_lds, stream>>>(k, n, h, w, last_bytes, res_dev, img_dev);
    timer.mark("k_twar_inverse");
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(stream));
    timer.finish();
    return PILC_OK;
}

}  // extern "C"
