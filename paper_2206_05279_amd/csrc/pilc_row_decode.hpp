// Decoder for batches with few, long lanes: a row of 16 threads owns one lane (gfx950).
//
// A lane is a serial chain (App. A eq. (12) of arXiv 2206.05279: every state depends on the one
// before), so with a few thousand lanes a wavefront must be alone on its SIMD and the time is
// (symbols per lane) x (instructions the wavefront issues per symbol) x some 5 cycles: a wavefront alone
// issues a plain instruction every five cycles and a 64-bit one every nine, whether it depends on the one before or not, and
// a wait state costs nearly as much.  This kernel is built to keep that count low (3125 lanes of 16,384 pixels 8110 us with 177
// vector instructions and 13 waits a pixel, 6830 with 166 and 3, 1000 cycles a pixel):
//   - a wavefront carries four lanes, one per 16-thread row, so 4096 lanes still leave every SIMD
//     of the chip with at most one wavefront;
//   - per symbol every thread evaluates C(k) at two neighbouring candidates of a 32-value window
//     around the predicted mean, together with the mass up to its successor;
//     once the state is known, one subtraction and one compare per candidate tell the thread
//     whether it holds the symbol (App. A: the x with C_x <= S mod 2^M < C_x + P_x), every thread
//     forms the next state for its own candidates, and an OR over the row (four rotate-and-OR
//     steps on the data-parallel-primitive path, no LDS round trip, no ballot) hands the one
//     non-zero value to all 16 threads;
//   - the mean of the next channel comes from the value first, up to asking for its table cells, and the state, the
//     stream's position and what else there is to do for the symbol is done while the cells are on their way;
//   - a pixel is decoded without a branch: whether every symbol was inside its window is
//     looked at once per pixel, and a pixel with a symbol outside is decoded again from the state
//     saved at its start by a bounded two-level search (32 values eight apart, then the nine of
//     the band);
//   - the candidates of a pixel's first channel do not depend on decoded values and are evaluated
//     a batch ahead;
//   - per-pixel parameters are prepared 16 pixels at a time, one pixel per thread, two batches
//     ahead of their use, and handed over through LDS; the 96 stream words a batch can reach are
//     fetched a batch ahead and wait in LDS, and the word a refill would take is read ahead of
//     time;
//   - none of that, nor the stores of the decoded pixels, is done by the wavefront that decodes:
//     every decoding wavefront has a second wavefront on its SIMD, its stager, which does it a
//     batch ahead in the issue slots the decoder leaves empty (a decoder that staged its own
//     batches spent 6 % of its time on it).  The two hand over through counts in LDS.
// Every loop has a trip count fixed by the geometry; the waits of the hand-over are bounded by the
// constant-rate clock and end in a time-out error.
#pragma once

#include <type_traits>

#include "pilc_device.hpp"

namespace pilc {

constexpr int kRowWaves = 4;                  // wavefronts per workgroup
constexpr int kRowLanes = 4 * kRowWaves;      // lanes per workgroup
constexpr int kRowBatch = 16;                 // pixels prepared at a time, one per thread of the row
constexpr int kRowWords = 112;                // stream words kept per lane and batch: a batch takes at
                                              // most 48 and is fetched before the previous one's 48
constexpr int kRowWindow = 32;                // candidates per symbol
constexpr int kRowBaseMax = 256 - kRowWindow; // window bases 0..224: candidates stay within 0..255
constexpr int kRowRedoLimit = 4;              // a batch with this many pixels outside their windows sends
constexpr int kRowSearchBatches = 7;          // the wavefront's next 7 batches straight to the search

// What the threads of a row make of their candidates {t < f}: the winner's x and next state f q + t (App. A eq. (12)), ORed over
// the row, where all others have 0, into every thread.  Rotations by 1, 2, 4 and 8 by the DPP path, which may read a register
// only two instructions after it was written: the two reductions and a third instruction, F1 .. F4 (something else
// that has to be done there or a wait), take turns.  The choices read their masks two instructions after these were made.
#define PILC_ROW_TURN(rotate, filler)                                                       \
    "v_or_b32_dpp %[x], %[x], %[x] " rotate " row_mask:0xf bank_mask:0xf bound_ctrl:0\n"   \
    "v_or_b32_dpp %[s], %[s], %[s] " rotate " row_mask:0xf bank_mask:0xf bound_ctrl:0\n" filler
#define PILC_ROW_PICK(F1, F2, F3, F4)                                                       \
    "v_cmp_lt_u32_e32 vcc, %[t0], %[f0]\n"                                                 \
    "v_cmp_lt_u32_e64 %[m], %[t1], %[f1]\n"                                                \
    "v_mad_u32_u24 %[s], %[f0], %[q], %[t0]\n"                                             \
    "v_mad_u32_u24 %[u], %[f1], %[q], %[t1]\n"                                             \
    "v_cndmask_b32_e32 %[x], 0, %[xw0], vcc\n"                                             \
    "v_cndmask_b32_e32 %[s], 0, %[s], vcc\n"                                               \
    "v_cndmask_b32_e64 %[x], %[x], %[xw1], %[m]\n"                                         \
    "v_cndmask_b32_e64 %[s], %[s], %[u], %[m]\n" F1                                        \
    PILC_ROW_TURN("row_ror:1", F2) PILC_ROW_TURN("row_ror:2", F3) PILC_ROW_TURN("row_ror:4", F4) PILC_ROW_TURN("row_ror:8", "")
#define PILC_ROW_PICK_OUT [x] "=&v"(x), [s] "=&v"(s_new), [u] "=&v"(u), [m] "=&s"(m)
#define PILC_ROW_PICK_IN                                                                    \
    [t0] "v"(slot - cd.cv0), [f0] "v"(cd.f0), [t1] "v"(slot - cd.cv1), [f1] "v"(cd.f1), [q] "v"(q), [xw0] "v"(xw0), [xw1] "v"(xw1)

// What follows from a value up to the addresses of the next channel's two table cells, in one piece with the pick (the compiler
// waits after every piece that is written out by itself): e = 256 x - m of the value, the next effective mean as
// -1 - n = mean - rsh14_mul(a, e), the window (w and b2, its base), and from the positions u0 and u of the thread's
// edges there (edge_pos) the cells' places in the table, w and d.
#define PILC_ROW_AIM                                                                        \
    "v_add3_u32 %[e], %[x], %[base], %[n]\n"                                               \
    "v_mad_i32_i24 %[w], %[a], %[e], %[half]\n"                                            \
    "v_ashrrev_i32_e32 %[w], 14, %[w]\n"                                                   \
    "v_sub_u32_e32 %[d], %[mean], %[w]\n"                                                  \
    "v_sub_u32_e32 %[w], %[centre], %[d]\n"                                                \
    "v_and_b32_e32 %[w], 0xffffff00, %[w]\n"                                               \
    "v_med3_i32 %[b2], %[w], 0, %[most]\n"                                                 \
    "v_add3_u32 %[d], %[d], %[edge], %[b2]\n"                                              \
    "v_cvt_f64_i32_e32 %[y], %[d]\n"                                                       \
    "v_fma_f64 %[y], %[y], %[unit], %[bias]\n"                                             \
    "v_cvt_u32_f64_e32 %[u0], %[y]\n"                                                      \
    "v_add_f64 %[y], %[y], %[per_k]\n"                                                     \
    "v_cvt_u32_f64_e32 %[u], %[y]\n"                                                       \
    "v_lshrrev_b32_e32 %[w], 18, %[u0]\n"                                                  \
    "v_lshrrev_b32_e32 %[d], 18, %[u]\n"                                                   \
    "v_and_b32_e32 %[w], 0x3ff8, %[w]\n"                                                   \
    "v_and_b32_e32 %[d], 0x3ff8, %[d]"
#define PILC_ROW_AIM_OUT [e] "=&v"(e), [w] "=&v"(w), [d] "=&v"(d), [b2] "=&v"(am.base), [y] "=&v"(y), [u0] "=&v"(am.u[0])
#define PILC_ROW_AIM_IN                                                                     \
    [base] "v"(cd.base), [n] "v"(n), [a] "v"(a), [half] "v"(8192), [mean] "v"(mean), [centre] "s"(kRowCentre),        \
    [most] "v"(256 * kRowBaseMax), [edge] "v"(j_edge), [unit] "v"(per_unit), [bias] "s"(kEdgeBias), [per_k] "v"(per_k)
// The window's base less the effective mean: the mean lies between its middle two candidates.
constexpr int kRowCentre = -1 - (256 * (kRowWindow / 2 - 1) - 128);
static_assert(sizeof(uint2[kSigEntries]) - sizeof(uint2) == 0x3ff8, "a position's upper 11 bits are its cell");

// thread j of a row receives the value of thread j + 1 of the same row, the last one `last`
__device__ __forceinline__ uint32_t row_next(uint32_t v, uint32_t last)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x101 /* row_shl:1 */, 0xF, 0xF, false);
}

// What one pixel's preparing thread leaves in LDS for the row (64 bytes).  Values and window bases are kept times 256, like
// the means, and a decoded one has its lowest bit set (`hit` below), so 256 x - m is the decoded number less 1 + m.  The
// inverse scale of a channel comes as what one step of k and one unit of the mean move the position of an edge by
// (see EdgeLaw: 1/s times 4 and times 2^-6, both exact).
struct RowPixel {
    uint4 r;            // -1 - m_r, -1 - m_g, -1 - m_b (Q8.8), window of R times 256
    uint4 s;            // a_gr, a_br, a_bg (Q2.14, sign-extended), 1/s of R
    double g[2], b[2];  // G and B: 1/s times 4, times 2^-6
};

// The candidates of one symbol as a thread holds them: C(k) - base at k = base + 2 j and base + 2 j + 1
// and the masses up to their successors (0 for a candidate that cannot be the symbol); base times 256.
struct RowCand {
    uint32_t cv0, cv1, f0, f1;
    int base;
};

// Everything that the workgroup keeps in LDS, the tables first: an address below 2^16 fits into the instruction that reads them.
template <bool kStaged>
struct RowShared {
    LdsTables tab;
    RowPixel stage[2][kRowLanes][kRowBatch];
    uint16_t words[2][kRowLanes][kRowWords];
    // The candidates of every thread for the first channel of every pixel of a batch, {cv0 | f0 << 16, cv1 | f1 << 16}
    // (a candidate is at most 255, so C and the masses are below 2^M <= 2^16)
    uint2 first_cand[kStaged ? 2 : 1][kStaged ? kRowLanes : 1][kRowBatch][16];
    // The workgroup has two wavefronts per four lanes: one decodes, the other (its stager) prepares
    // the next batch's parameters and stream words in LDS meanwhile.  What passes between them:
    uint32_t word_base[2][kRowLanes];  // stream position of words[buf][lane][0]
    // Of batch b, in slot b & 1: the lane's stream position at its start and its 16 decoded pixels.
    // (The decoder writes a slot again two batches later, and cannot start that batch before the
    // stager, which reads the slot first, has staged it.)
    uint32_t pos[2][kRowLanes];
    uint32_t out[2][kStaged ? kRowLanes : 1][kRowBatch];
    uint32_t posted[kRowWaves];        // batches the decoding wavefront has finished
    uint32_t staged[kRowWaves];        // batches the stager has made ready
    uint32_t abort;                    // a wait was given up: everybody leaves
    int state;
    unsigned long long payload;
};

// kStaged: with a stager per decoding wavefront (see above).  That form keeps twice the LDS per
// lane (the first channel's candidates of two batches), so only one workgroup of 16 lanes fits a
// compute unit; it is for batches of up to 16 lanes per compute unit.  Without it a decoding
// wavefront stages its own batches, and two workgroups share a compute unit.
template <bool kRagged, bool kStaged>
__global__ __launch_bounds__((kStaged ? 2 : 1) * 64 * kRowWaves) void k_decode_rows(
    Geo g, const uint8_t *__restrict__ coded, unsigned long long coded_bytes, const uint16_t *__restrict__ mu,
    const int16_t *__restrict__ ls, const int16_t *__restrict__ coef, uint8_t *__restrict__ out,
    Report *__restrict__ report, unsigned long long wait_ticks, uint32_t withhold)
{
    // wait_ticks: the bound of a wait between a decoding wavefront and its stager, in ticks of the
    // constant-rate clock; withhold: the stagers never say that a batch is ready (tests of the
    // give-up path)
    __shared__ RowShared<kStaged> sm;
    const LdsTables &tab = sm.tab;
    auto &stage = sm.stage;
    auto &words = sm.words;
    auto &first_cand = sm.first_cand;
    auto &s_word_base = sm.word_base;
    auto &s_pos = sm.pos;
    auto &s_out = sm.out;
    auto &s_posted = sm.posted;
    auto &s_staged = sm.staged;
    auto &s_abort = sm.abort;
    auto &s_state = sm.state;
    auto &s_payload = sm.payload;
    if (threadIdx.x < (uint32_t)kRowWaves) {
        s_posted[threadIdx.x] = 0u;
        s_staged[threadIdx.x] = 0u;
    }
    if (threadIdx.x == 0u) {
        s_abort = 0u;
        s_state = check_header(g, kMagicPilc, 0u, coded, coded_bytes, &s_payload);
    }
    const bool stager = kStaged && threadIdx.x >= 64u * kRowWaves;
    const uint32_t tix = threadIdx.x - (stager ? 64u * kRowWaves : 0u);  // index among the threads of its kind
    const uint32_t tid = tix & 63u, wv = tix >> 6;
    const uint32_t j = tid & 15u, gbase = tid & 48u;
    const uint32_t lrow = tix >> 4;  // lane slot of the workgroup
    // a row beyond the last lane decodes the last lane once more and keeps the result to itself,
    // so that every row of a wavefront always does valid work
    const bool has_lane = blockIdx.x * kRowLanes + lrow < g.lanes;
    const uint32_t lane = has_lane ? blockIdx.x * kRowLanes + lrow : g.lanes - 1u;
    const LaneShape sh = lane_shape(g, lane);
    const uint32_t m_bits = g.prec_bits;
    const uint32_t mask = (1u << m_bits) - 1u, top = 1u << m_bits;
    const uint32_t scale = mass_scale(m_bits);
    // (The offsets are asked for before the header and the tables are waited for: the host has seen that they fit in coded_bytes.)
    const uint32_t *offsets = reinterpret_cast<const uint32_t *>(coded + 64);
    const uint32_t begin = offsets[lane], end = offsets[lane + 1];
    const uint16_t *payload =
        reinterpret_cast<const uint16_t *>(coded + 64 + 4ull * ((size_t)g.lanes + 1));
    const uint2 *sig = tab.sig;
    load_tables(sm.tab);  // ends with a barrier
    if (s_state != ST_OK) {
        if (blockIdx.x == 0u && threadIdx.x == 0u) raise_code(report, s_state);
        return;
    }
    const uint32_t payload_bytes = (uint32_t)s_payload;

    // row-uniform state: S, the stream position `pos` (word index into the payload) and the end
    // of the lane's words `stop`
    uint32_t npx = 0, stop = 0, S = 1u << 16, pos = 0;
    if (end < begin || end > payload_bytes || end - begin < 4u || ((begin | end) & 1u)) {
        if (j == 0 && has_lane) raise_code(report, ST_CORRUPT);
    } else {
        npx = sh.npx;
        stop = end >> 1;
        pos = begin >> 1;
        S = (uint32_t)payload[pos] | ((uint32_t)payload[pos + 1] << 16);
        pos += 2;
    }
    // The stream words from `from` on, thread j those at j, j + 16, ...: words past `stop` read
    // as 0, and an overrun shows at the end of the lane as pos != stop.
    struct Ahead {
        uint32_t w[kRowWords / 16];
    };
    auto fetch_words = [&](uint32_t from) {
        Ahead a;
#pragma unroll
        for (int r = 0; r < kRowWords / 16; ++r) {
            const uint32_t at = from + 16u * r + j;
            a.w[r] = at < stop ? (uint32_t)payload[at] : 0u;
        }
        return a;
    };

    // ---- per-pixel parameters: thread j prepares pixel t0 + j of its lane ----
    struct Raw {
        uint32_t m[3];
        int l[3], a[3];
    };
    auto fetch_raw = [&](uint32_t t0) {
        Raw r;
        const uint32_t t = t0 + j;
        const uint32_t p = lane_pixel(g, sh, t < npx ? t : 0u);
        const size_t s = (size_t)p * 3;
        const uint32_t im = g.by_hw.div(p);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r.m[c] = mu[s + c];
            r.l[c] = ls[s + c];
            r.a[c] = coef[3 * im + c];
        }
        return r;
    };
    // The window of a symbol whose effective mean is -1 - n: its base times 256, whole and within 0 .. kRowBaseMax.
    auto window_base = [](int n) {
        return min(max((kRowCentre - n) & ~255, 0), 256 * kRowBaseMax);
    };
    auto put_stage = [&](const Raw &r, uint32_t buf) {
        RowPixel px;
        const int n_r = -1 - (int)r.m[0];
        px.r = make_uint4((uint32_t)n_r, (uint32_t)(-1 - (int)r.m[1]), (uint32_t)(-1 - (int)r.m[2]),
                          (uint32_t)window_base(n_r));
        px.s = make_uint4((uint32_t)r.a[0], (uint32_t)r.a[1], (uint32_t)r.a[2], inv_scale(r.l[0], tab));
        const double i1 = (double)inv_scale(r.l[1], tab), i2 = (double)inv_scale(r.l[2], tab);
        px.g[0] = i1 * 4.0;
        px.g[1] = i1 * 0x1p-6;
        px.b[0] = i2 * 4.0;
        px.b[1] = i2 * 0x1p-6;
        stage[buf][lrow][j] = px;
    };

    // Window of a symbol with effective mean -1 - n, and this thread's candidates k = base + 2 j and
    // base + 2 j + 1 in it; `per_k` and `per_unit` as in RowPixel.  The evaluation comes in two
    // halves so that the wait for one symbol's table cells can be filled with another symbol's
    // arithmetic: `aim` goes as far as asking for the cells, `finish` takes it from there.
    struct RowAim {
        uint2 cell[2];
        uint32_t u[2];
        int base;
        uint32_t c0_most;  // of C at the first candidate: 0 where that is C(0)
        bool last;         // the last window
    };
    const uint32_t j2 = 2u * j;
    const int j_edge = 512 * (int)j - 127;  // from the window's base and n to 256 k - 128 - mean
    const uint32_t j_not_first = j == 0u ? 0u : 0x7FFFFFFFu;
    uint32_t top_left = top - (uint32_t)kRowBaseMax;  // C(256) less the last window's base
    asm("" : "+v"(top_left));  // (in a vector register)
    auto aim = [&](int n, double per_k, double per_unit) {
        RowAim am;
        am.base = window_base(n);
        const double y = __builtin_fma((double)(am.base + j_edge + n), per_unit, kEdgeBias);
        am.u[0] = edge_pos(y);
        am.u[1] = edge_pos(y + per_k);
#pragma unroll
        for (int c = 0; c < 2; ++c) am.cell[c] = sig[am.u[c] >> 21];
        return am;
    };
    // what else `finish` needs of the window: for the wait for the cells
    auto aimed = [&](RowAim &am) {
        am.c0_most = ((uint32_t)am.base << 8) | j_not_first;
        am.last = am.base == 256 * kRowBaseMax;
#pragma unroll
        for (int c = 0; c < 2; ++c) am.u[c] |= 2047u;  // (see interpolate)
    };
    auto aim_first = [&](const RowPixel &px) {  // the first channel, whose 1/s comes as it is
        const double inv = (double)px.s.w;
        RowAim am = aim((int)px.r.x, inv * 4.0, inv * 0x1p-6);
        aimed(am);
        return am;
    };
    // The candidates of a symbol, from the cells `aim` asked for.  The second candidate is followed by the
    // next thread's first; candidate 31 by C(base + 32), which is known only when it is C(256) = 2^M.
    auto finish = [&](const RowAim &am) {
        RowCand cd;
        cd.base = am.base;
        cd.cv0 = min(j2 + mass_of(interpolate(am.u[0], am.cell[0]), scale), am.c0_most);
        cd.cv1 = j2 + 1u + mass_of(interpolate(am.u[1], am.cell[1]), scale);
        cd.f0 = cd.cv1 - cd.cv0;
        cd.f1 = row_next(cd.cv0, am.last ? top_left : cd.cv1) - cd.cv1;
        return cd;
    };
    // the same for a pixel's first channel, which the stager has left in LDS
    auto first_channel = [&](uint2 pair, uint32_t window) {
        return RowCand{pair.x & 0xFFFFu, pair.y & 0xFFFFu, pair.x >> 16, pair.y >> 16, (int)window};
    };
    // (stager) the first channel of the 16 pixels from t0 on, staged in `buf`, every thread its two candidates; four at a time and
    // as far as a lane of the wavefront goes: all 16 delay the first pixel by 3 us (4096 lanes of one pixel 27.8 us a call, 24.6 now;
    // of 17 35.7 and 33.4)
    auto put_first_cand = [&](uint32_t buf, uint32_t t0) {
        wave_lds_sync();  // the parameters were written by this wavefront
#pragma unroll 1
        for (uint32_t i0 = 0; i0 < (uint32_t)kRowBatch && (!kRagged || __any(t0 + i0 < npx)); i0 += 4u) {
#pragma unroll
            for (uint32_t i = i0; i < i0 + 4u; ++i) {
                const RowCand cd = finish(aim_first(stage[buf][lrow][i]));
                first_cand[buf][lrow][i][j] = make_uint2(cd.cv0 | (cd.f0 << 16), cd.cv1 | (cd.f1 << 16));
            }
        }
    };

    const uint32_t xw0 = 512u * j | 1u, xw1 = xw0 | 256u;  // what a winning candidate contributes
    const uint16_t *flat_words = &words[0][0][0];
    uint32_t at = 0;     // place of the next word in `flat_words`, which holds the current batch's words
    uint32_t wnext = 0;  // the word there
    // One symbol of the four lanes of the wavefront, no branch, in two steps.  `pick`: 256 times the value less the window's base,
    // and 1 (0 where the window does not hold the symbol), and in `s_new` the next state before it takes a word; `after_pick`:
    // S, at and wnext of rows with `act`.  What needs the value comes between the two, so that its table reads are under way.
    auto slot_in = [&](int base) { return (S & mask) - (((uint32_t)base >> 8) & 255u); };
    auto ask_cells = [&](RowAim &am, uint32_t w, uint32_t d) {
        am.cell[0] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(sig) + w);
        am.cell[1] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(sig) + d);
    };
    // the first channel, and from e of its value the second channel's aim; beside it thread `before` takes the three second bytes
    // of the pixel before, pair and last, into v_out
    auto pick_first = [&](const RowCand &cd, uint32_t slot, uint32_t q, uint32_t &s_new, int n, int a, int mean, double per_k,
                          double per_unit, int &e, RowAim &am, uint32_t before, uint32_t pair, uint32_t last, uint32_t &v_out) {
        uint32_t x, u, w, d, rgb;
        unsigned long long m, taker;
        double y;
        asm(PILC_ROW_PICK("v_cmp_eq_u32_e64 %[taker], %[j], %[before]\n", "v_perm_b32 %[rgb], %[last], %[pair], %[sel]\n",
                          "v_cndmask_b32_e64 %[v_out], %[v_out], %[rgb], %[taker]\n", "s_nop 0\n") PILC_ROW_AIM
            : PILC_ROW_PICK_OUT, PILC_ROW_AIM_OUT, [taker] "=&s"(taker), [rgb] "=&v"(rgb), [v_out] "+v"(v_out)
            : PILC_ROW_PICK_IN, PILC_ROW_AIM_IN, [j] "v"(j), [before] "s"(before), [last] "v"(last), [pair] "v"(pair),
              [sel] "s"(0x0C050100u)
            : "vcc");
        am.u[1] = u;
        ask_cells(am, w, d);
        return x;
    };
    // the second channel, and what the first says of the third's mean (a2, e2) on the way to the third's aim
    auto pick_second = [&](const RowCand &cd, uint32_t slot, uint32_t q, uint32_t &s_new, int n, int a, int mean, int a2, int e2,
                           double per_k, double per_unit, RowAim &am) {
        uint32_t x, u, w, d;
        unsigned long long m;
        double y;
        int e;
        asm(PILC_ROW_PICK("v_mad_i32_i24 %[e2], %[a2], %[e2], %[half]\n", "v_ashrrev_i32_e32 %[e2], 14, %[e2]\n",
                          "v_sub_u32_e32 %[mean], %[mean], %[e2]\n", "s_nop 0\n") PILC_ROW_AIM
            : PILC_ROW_PICK_OUT, PILC_ROW_AIM_OUT, [mean] "+v"(mean), [e2] "+v"(e2)
            : PILC_ROW_PICK_IN, [base] "v"(cd.base), [n] "v"(n), [a] "v"(a), [a2] "v"(a2), [half] "v"(8192), [centre] "s"(kRowCentre),
              [most] "v"(256 * kRowBaseMax), [edge] "v"(j_edge), [unit] "v"(per_unit), [bias] "s"(kEdgeBias), [per_k] "v"(per_k)
            : "vcc");
        am.u[1] = u;
        ask_cells(am, w, d);
        return x;
    };
    // the third channel; beside it the second bytes of lo and hi as the two lowest of `pair`, p & q of the first two channels and,
    // of what the stager left for the next pixel's first, the masses
    auto pick_third = [&](const RowCand &cd, uint32_t slot, uint32_t q, uint32_t &s_new, uint32_t lo, uint32_t hi, uint32_t &pair,
                          uint2 next, uint2 &next_f, uint32_t p0, uint32_t p1, uint32_t &both) {
        uint32_t x, u, r, b;
        unsigned long long m;
        if (kStaged) {
            uint32_t g0, g1;
            asm(PILC_ROW_PICK("v_perm_b32 %[r], %[hi], %[lo], %[sel]\n", "v_lshrrev_b32_e32 %[g0], 16, %[h0]\n",
                              "v_lshrrev_b32_e32 %[g1], 16, %[h1]\n", "v_and_b32_e32 %[b], %[p0], %[p1]\n")
                : PILC_ROW_PICK_OUT, [r] "=&v"(r), [g0] "=&v"(g0), [g1] "=&v"(g1), [b] "=&v"(b)
                : PILC_ROW_PICK_IN, [lo] "v"(lo), [hi] "v"(hi), [sel] "s"(0x0C0C0501u), [h0] "v"(next.x), [h1] "v"(next.y),
                  [p0] "v"(p0), [p1] "v"(p1)
                : "vcc");
            next_f = make_uint2(g0, g1);
        } else {
            asm(PILC_ROW_PICK("v_perm_b32 %[r], %[hi], %[lo], %[sel]\n", "v_and_b32_e32 %[b], %[p0], %[p1]\n", "s_nop 0\n", "s_nop 0\n")
                : PILC_ROW_PICK_OUT, [r] "=&v"(r), [b] "=&v"(b)
                : PILC_ROW_PICK_IN, [lo] "v"(lo), [hi] "v"(hi), [sel] "s"(0x0C0C0501u), [p0] "v"(p0), [p1] "v"(p1)
                : "vcc");
            next_f = make_uint2(0u, 0u);
        }
        pair = r;
        both = b;
        return x;
    };
    auto after_pick = [&](bool act, uint32_t s_new) {
        const bool refill = s_new < (1u << 16);
        const uint32_t s_ref = (s_new << 16) | wnext;
        if (kRagged) {
            S = act ? (refill ? s_ref : s_new) : S;
            at += (act && refill) ? 1u : 0u;
        } else {
            S = refill ? s_ref : s_new;
            at += refill ? 1u : 0u;
        }
        asm("" : "+v"(at));  // (one count, from which the address is made)
        wnext = flat_words[at];
    };
    // The same by a bounded search with the general evaluation, on the state (Sr, pr): every 8th
    // value first (C(0) = 0 always counts), then the nine values of the band.
    auto search_symbol = [&](int me, uint32_t inv_s, uint32_t &Sr, uint32_t &pr) -> uint32_t {
        auto row_count = [&](bool pred) -> uint32_t {
            return (uint32_t)__popc((uint32_t)(__ballot(pred) >> gbase) & 0xFFFFu);
        };
        const uint32_t slot = Sr & mask, q = Sr >> m_bits;
        const uint32_t below = row_count(cum_at(8 * (int)j, me, inv_s, m_bits, tab) <= slot) +
                               row_count(cum_at(8 * (int)j + 128, me, inv_s, m_bits, tab) <= slot);
        const int kb = 8 * ((int)below - 1);
        const uint32_t cf = cum_at(min(kb + (int)j, 256), me, inv_s, m_bits, tab);
        const uint32_t n = row_count(j <= 8u && cf <= slot);  // 1..8: C(kb) <= slot < C(kb + 8)
        const uint32_t c_lo = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((gbase + n - 1u) << 2), (int)cf);
        const uint32_t c_hi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((gbase + n) << 2), (int)cf);
        uint32_t s_new = (uint32_t)__umul24(c_hi - c_lo, q) + (slot - c_lo);
        if (s_new < (1u << 16)) {
            s_new = (s_new << 16) | flat_words[pr];
            ++pr;
        }
        Sr = s_new;
        return (uint32_t)kb + n - 1u;
    };

    // Hand-over between a decoding wavefront and its stager: a count in LDS, raised by one thread
    // after the wavefront's LDS writes are done, and waited for by the whole partner wavefront.  A
    // wait is bounded by the constant-rate clock; who gives up says so to everybody (no wavefront
    // is left waiting) and the call ends in a time-out error.
    auto raise = [&](uint32_t *count, uint32_t value) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (tid == 0u) __hip_atomic_store(count, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto wait_for = [&](uint32_t *count, uint32_t value) -> bool {
        if (__hip_atomic_load(count, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= value) return true;
        const unsigned long long since = wall_clock64();
        for (;;) {
            if (__hip_atomic_load(count, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= value) return true;
            if (__hip_atomic_load(&s_abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u) return false;
            if (wall_clock64() - since > wait_ticks) {
                __hip_atomic_store(&s_abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (tid == 0u) raise_code(report, ST_TIMEOUT);
                return false;
            }
            __builtin_amdgcn_s_sleep(8);
        }
    };
    auto put_words = [&](const Ahead &a, uint32_t buf, uint32_t from) {
#pragma unroll
        for (int r = 0; r < kRowWords / 16; ++r) words[buf][lrow][16 * r + j] = (uint16_t)a.w[r];
        if (j == 0u) s_word_base[buf][lrow] = from;
    };

    // the pixels of the batch that began at pixel t0 of the lane, from slot `slot`, to the image
    auto store_batch = [&](uint32_t t0, uint32_t slot) {
        const uint32_t nb = t0 < npx ? min((uint32_t)kRowBatch, npx - t0) : 0u;
        if (j < nb && has_lane) {
            const uint32_t v = s_out[slot][lrow][j];
            const size_t s = (size_t)lane_pixel(g, sh, t0 + j) * 3;
            out[s] = (uint8_t)v;
            out[s + 1] = (uint8_t)(v >> 8);
            out[s + 2] = (uint8_t)(v >> 16);
        }
    };

    if (kStaged && stager) {
        // Batch 0 first; then, while the partner decodes batch b, the parameters of batch b + 1 (loaded
        // a batch ago) and its stream words: the 112 words from where the stream stood when batch b
        // began, of which batch b takes at most 48 and batch b + 1 at most 48 more; and the pixels of
        // batch b - 1 go to the image.
        const Ahead first_words = fetch_words(pos);
        put_stage(fetch_raw(0), 0);
        Raw raw_next = fetch_raw(kRowBatch);
        put_first_cand(0u, 0u);
        put_words(first_words, 0u, pos);
        if (!withhold) raise(&s_staged[wv], 1u);
        uint32_t from = pos, t0 = 0, b = 0;
        for (; __any(t0 < npx); t0 += kRowBatch, ++b) {
            const uint32_t buf = b & 1u;
            if (b != 0u) {
                // the partner has finished batch b - 1: buffer buf ^ 1 is free, and the position is known
                if (!wait_for(&s_posted[wv], b)) return;
                from = s_pos[buf][lrow];
                store_batch(t0 - kRowBatch, buf ^ 1u);
            }
            const Ahead ahead = fetch_words(from);
            put_stage(raw_next, buf ^ 1u);
            raw_next = fetch_raw(t0 + 2 * kRowBatch);
            put_first_cand(buf ^ 1u, t0 + kRowBatch);
            put_words(ahead, buf ^ 1u, from);
            if (!withhold) raise(&s_staged[wv], b + 2u);
        }
        if (b != 0u && wait_for(&s_posted[wv], b)) store_batch(t0 - kRowBatch, (b & 1u) ^ 1u);  // the last batch's pixels
        return;
    }

    uint32_t search_batches = 0;  // wavefront-uniform: batches still to decode by search alone
    // (without a stager) batch 0 staged, batch 1 in flight
    Raw raw_next = {};
    Ahead ahead = {};
    uint32_t ahead_base = pos;
    if (!kStaged) {
        put_stage(fetch_raw(0), 0);
        raw_next = fetch_raw(kRowBatch);
        ahead = fetch_words(pos);
    }
    for (uint32_t t0 = 0, b = 0; __any(t0 < npx); t0 += kRowBatch, ++b) {
        const uint32_t buf = b & 1u;
        const uint32_t nb = t0 < npx ? min((uint32_t)kRowBatch, npx - t0) : 0u;
        if (kStaged) {
            if (!wait_for(&s_staged[wv], b + 1u)) break;
            at = s_word_base[buf][lrow];
        } else {
            // this batch's words (fetched a batch ago, from where the stream stood then) into LDS, the
            // next batch's requested from where the stream stands now; the next batch's parameters
            // staged from the registers loaded a batch ago, and the batch after that requested
            at = ahead_base;
#pragma unroll
            for (int r = 0; r < kRowWords / 16; ++r) words[buf][lrow][16 * r + j] = (uint16_t)ahead.w[r];
            ahead = fetch_words(pos);
            ahead_base = pos;
            put_stage(raw_next, buf ^ 1u);
            raw_next = fetch_raw(t0 + 2 * kRowBatch);
            wave_lds_sync();
        }
        at = (buf * kRowLanes + lrow) * kRowWords + pos - at;
        const uint32_t at_start = at;
        wnext = flat_words[at];

        const RowPixel *px = stage[buf][lrow];
        uint32_t v_out = 0;
        // The three symbols of a pixel by search, on the state (Sr, pr).
        auto search_pixel = [&](const RowPixel &cur, uint32_t &Sr, uint32_t &pr, uint32_t &y_r, uint32_t &y_g,
                                uint32_t &y_b) {
            const int m_r = -1 - (int)cur.r.x, m_g = -1 - (int)cur.r.y, m_b = -1 - (int)cur.r.z;
            const int a_gr = (int)cur.s.x, a_br = (int)cur.s.y, a_bg = (int)cur.s.z;
            y_r = search_symbol(m_r, cur.s.w, Sr, pr);
            const int f_r = (int)(y_r << 8) - m_r;
            y_g = search_symbol(m_g + rsh14_mul(a_gr, f_r), (uint32_t)(cur.g[0] * 0.25), Sr, pr);
            y_b = search_symbol(m_b + rsh14_mul(a_br, f_r) + rsh14_mul(a_bg, (int)(y_g << 8) - m_g),
                                (uint32_t)(cur.b[0] * 0.25), Sr, pr);
        };
        if (search_batches != 0) {
            // data the model does not fit (such as uniformly random pixels): the windows are not tried
            --search_batches;
            for (uint32_t i = 0; kRagged ? __any(i < nb) : i < (uint32_t)kRowBatch; ++i) {
                uint32_t Sr = S, pr = at, y_r, y_g, y_b;
                search_pixel(px[i], Sr, pr, y_r, y_g, y_b);
                if (!kRagged || i < nb) {
                    S = Sr;
                    at = pr;
                }
                v_out = j == i ? (y_r | (y_g << 8) | (y_b << 16)) : v_out;
            }
        } else {
            uint32_t redone = 0;  // pixels of this batch that had a symbol outside its window
            // One pixel: `cur` holds its parameters (read from LDS a pixel ago), `nxt` receives the
            // next pixel's, and `cr` enters with this pixel's first-channel candidates and leaves
            // with the next pixel's.
            // of the pixel before, until thread i - 1 takes them: the first two values, and the third times 256
            uint32_t pair = 0, x_b = 0;
            auto pixel = [&](uint32_t i, const RowPixel &cur, RowPixel &nxt, RowCand &cr) {
                const bool act = i < nb;
                nxt = px[(i + 1u) & (kRowBatch - 1)];
                const uint2 next_pair = kStaged ? first_cand[buf][lrow][(i + 1u) & (kRowBatch - 1)][j] : uint2{0u, 0u};
                __builtin_amdgcn_sched_barrier(0);  // asked for here, used a pixel later
                const int n_r = (int)cur.r.x, n_g = (int)cur.r.y, n_b = (int)cur.r.z;
                const int a_gr = (int)cur.s.x, a_br = (int)cur.s.y, a_bg = (int)cur.s.z;
                const uint32_t S0 = S, at0 = at;
                uint32_t s_new, both;

                RowAim ag, ab;
                int e_r;
                const uint32_t p_r = pick_first(cr, slot_in(cr.base), S >> m_bits, s_new, n_r, a_gr, n_g, cur.g[0], cur.g[1],
                                                e_r, ag, i - 1u, pair, x_b, v_out);
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t x_r = (uint32_t)cr.base + p_r;
                after_pick(act, s_new);
                aimed(ag);
                const uint32_t slot_g = slot_in(ag.base), q_g = S >> m_bits;
                // The next pixel's first channel depends on no decoded value.  The stager has evaluated
                // it; without a stager its evaluation fills the waits of the two channels that do depend.
                RowAim an = {};
                if (!kStaged) an = aim_first(nxt);
                __builtin_amdgcn_sched_barrier(0);
                const RowCand cg = finish(ag);
                const uint32_t p_g = pick_second(cg, slot_g, q_g, s_new, n_g, a_bg, n_b, a_br, e_r, cur.b[0], cur.b[1], ab);
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t x_g = (uint32_t)cg.base + p_g;
                after_pick(act, s_new);
                aimed(ab);
                const uint32_t slot_b = slot_in(ab.base), q_b = S >> m_bits;
                __builtin_amdgcn_sched_barrier(0);
                if (!kStaged) {
                    cr = finish(an);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const RowCand cb = finish(ab);
                uint2 next_f;
                const uint32_t p_b = pick_third(cb, slot_b, q_b, s_new, x_r, x_g, pair, next_pair, next_f, p_r, p_g, both);
                if (kStaged)
                    cr = RowCand{next_pair.x & 0xFFFFu, next_pair.y & 0xFFFFu, next_f.x, next_f.y, (int)nxt.r.w};
                x_b = (uint32_t)cb.base + p_b;
                after_pick(act, s_new);

                bool bad = (both & p_b & 1u) == 0u;
                if (kRagged) bad = bad && act;
                if (__builtin_expect(__any(bad), 0)) {
                    // the pixel once more, from the state at its start, for the rows that need it
                    uint32_t Sr = S0, pr = at0, y_r, y_g, y_b;
                    search_pixel(cur, Sr, pr, y_r, y_g, y_b);
                    if (bad) {
                        S = Sr;
                        at = pr;
                        pair = y_r | (y_g << 8);
                        x_b = y_b << 8;
                    }
                    wnext = flat_words[at];
                    ++redone;
                }
            };
            RowPixel pe = px[0], po;
            RowCand cr = kStaged ? first_channel(first_cand[buf][lrow][0][j], pe.r.w)
                                 : finish(aim_first(pe));
            uint32_t i = 0;
            for (; kRagged ? __any(i < nb) : i < (uint32_t)kRowBatch; i += 2) {
                pixel(i, pe, po, cr);
                pixel(i + 1u, po, pe, cr);
            }
            v_out = j == i - 1u ? __builtin_amdgcn_perm(x_b, pair, 0x0C050100u) : v_out;
            if (redone >= (uint32_t)kRowRedoLimit) search_batches = kRowSearchBatches;
        }
        pos += at - at_start;
        if (kStaged) {
            // the pixels and the position go to the stager, which may then go on to the batch after next
            s_out[buf][lrow][j] = v_out;
            if (j == 0u) s_pos[buf ^ 1u][lrow] = pos;
            raise(&s_posted[wv], b + 1u);
        } else if (j < nb && has_lane) {
            const size_t s = (size_t)lane_pixel(g, sh, t0 + j) * 3;
            out[s] = (uint8_t)v_out;
            out[s + 1] = (uint8_t)(v_out >> 8);
            out[s + 2] = (uint8_t)(v_out >> 16);
        }
    }
    if (has_lane && npx != 0u && (S != (1u << 16) || pos != stop) && j == 0) raise_code(report, ST_CORRUPT);
}

#undef PILC_ROW_TURN
#undef PILC_ROW_PICK
#undef PILC_ROW_PICK_OUT
#undef PILC_ROW_PICK_IN
#undef PILC_ROW_AIM
#undef PILC_ROW_AIM_OUT
#undef PILC_ROW_AIM_IN

}  // namespace pilc
