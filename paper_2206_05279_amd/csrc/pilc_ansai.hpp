// The table-driven coder of Sec. 3.2 (Alg. 3 "ANS-AI: Encode x", Alg. 4 "ANS-AI: Decode one
// symbol") for gfx950: one thread per piece (Sec. 4.3), the tables of a workgroup in LDS.
//
// A symbol costs some twenty instructions and two to three bytes of HBM traffic, and the layout work is
// about moving whole cache lines:
//   - the symbol and index rows of a wavefront's 64 pieces are staged through LDS in chunks (in the
//     encoder chunks that are aligned in the arrays), with 16-byte loads in which consecutive threads cover one
//     row's chunk, so every line is fetched once and fully used;
//   - the encoder's words go to a row per piece of a scratch area, 32 bytes at a time;
//   - k_ansai_pack copies the rows into the container's records.
//
// Included at the end of pilc.hip (needs its Status, scan kernels, Timer and host helpers).
#pragma once

namespace pilc {

// ---------------------------------------------------------------------------------------------
// Shapes and the table blob
// ---------------------------------------------------------------------------------------------
struct AShape {
    uint32_t pieces, count;  // pieces * count < 2^32
    uint32_t M, D, X;
};

constexpr uint32_t kAnsaiMagic = 0x534E4150u;     // "PANS"
constexpr uint32_t kAnsaiTabMagic = 0x42544150u;  // tag of a built table blob
constexpr int ST_ARG = 1;                         // a symbol / index out of range, or foreign tables

// Device blob written by k_ansai_build: 256-byte header, then
//   enc   uint2 [D][256] + 1  { delta, phi }, index d << 8 | x; the last entry, index D << 8,
//                             is the identity step {-2^M, 0}: no bits pushed, state kept (Alg. 3)
//   theta uint8 [D << M]      symbol                               (Alg. 4)
//   nb    u16 or u32 [D << M] (N - 2^M) << 4 | (15 - B); 32-bit entries when M > 12
struct ATabHeader {
    uint32_t magic, M, D, X, ok;
    uint32_t pad[59];
};

struct ATabLayout {
    size_t enc_off, theta_off, nb_off, total;
    bool wide;
};

static inline ATabLayout ansai_tab_layout(uint32_t M, uint32_t D, uint32_t X)
{
    ATabLayout t;
    t.wide = M > 12;
    t.enc_off = sizeof(ATabHeader);
    t.theta_off = (t.enc_off + 8 * ((size_t)D * 256 + 1) + 255) & ~(size_t)255;
    t.nb_off = (t.theta_off + ((size_t)D << M) + 255) & ~(size_t)255;
    t.total = (t.nb_off + ((size_t)D << M) * (t.wide ? 4 : 2) + 255) & ~(size_t)255;
    return t;
}

__global__ void k_ansai_build_begin(ATabHeader *head, uint32_t M, uint32_t D, uint32_t X)
{
    head->magic = kAnsaiTabMagic;
    head->M = M;
    head->D = D;
    head->X = X;
    head->ok = 1u;
}

// One workgroup per distribution.  Validates the masses (every P_x >= 1, sum 2^M) and writes
// delta = k 2^M - P_x 2^k for the k with P_x 2^k in [2^M, 2^(M+1)) (App. B, lemma on the range
// of delta), phi = 2^M - P_x + C_x, and for every state value the outcome of Alg. 2: the symbol,
// the number of bits it pops and the state it reaches before they are added.
template <bool kWide>
__global__ __launch_bounds__(256) void k_ansai_build(uint32_t M, uint32_t X,
                                                     const uint32_t *__restrict__ mass,
                                                     ATabHeader *head, uint2 *__restrict__ enc,
                                                     uint8_t *__restrict__ theta,
                                                     void *__restrict__ nb_raw)
{
    __shared__ uint32_t cum[257];
    __shared__ int bad;
    const uint32_t d = blockIdx.x, top = 1u << M;
    if (threadIdx.x == 0) {
        unsigned long long run = 0;
        int b = 0;
        for (uint32_t x = 0; x < X; ++x) {
            const uint32_t p = mass[d * X + x];
            cum[x] = (uint32_t)run;
            if (p == 0 || p > top) b = 1;
            run += p;
        }
        cum[X] = (uint32_t)run;
        if (run != top) b = 1;
        bad = b;
        if (b) atomicExch(&head->ok, 0u);
    }
    __syncthreads();
    if (bad) return;
    if (d == 0 && threadIdx.x == 0) enc[gridDim.x * 256u] = make_uint2(0u - top, 0u);
    for (uint32_t x = threadIdx.x; x < X; x += blockDim.x) {
        const uint32_t p = cum[x + 1] - cum[x];
        const uint32_t k = M - (31u - __clz(p));
        enc[d * 256u + x] = make_uint2(k * top - (p << k), top - p + cum[x]);
    }
    for (uint32_t s = threadIdx.x; s < top; s += blockDim.x) {
        uint32_t lo = 0, hi = X - 1;  // largest x with cum[x] <= s
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (cum[mid] <= s)
                lo = mid;
            else
                hi = mid - 1;
        }
        const uint32_t t = s - cum[lo] + (cum[lo + 1] - cum[lo]);  // in [P_x, 2 P_x)
        const uint32_t len = 32u - __clz(t);
        const uint32_t b = len > M ? 0u : M + 1u - len;
        const uint32_t nrel = (t << b) - top;
        theta[((size_t)d << M) + s] = (uint8_t)lo;
        if (kWide)
            static_cast<uint32_t *>(nb_raw)[((size_t)d << M) + s] = nrel << 4 | (b ^ 15u);
        else
            static_cast<uint16_t *>(nb_raw)[((size_t)d << M) + s] = (uint16_t)(nrel << 4 | (b ^ 15u));
    }
}

// ---------------------------------------------------------------------------------------------
// Moving a wavefront's 64 rows between the arrays and LDS
// ---------------------------------------------------------------------------------------------
// A row is the `count` bytes of one piece in a [pieces, count] array.  The encoder cuts rows at multiples
// of 128 bytes of the array ("lines"); line-stage number `ls` of a row is its ls-th line from the
// back.  A wavefront fetches a line-stage of all its rows with
// 16-byte loads in which eight consecutive threads cover one row's line: thread `lane` holds, for
// i = 0..7, bytes [16c, 16c+16) of the line of row 8i + lane/8, with c = lane%8.  Every line is
// thus requested once, whole.  The threads then pass the line through LDS in two halves of 64
// bytes, where thread r finds the bytes of row r; the registers of the second half simply wait.

typedef uint32_t u32x4_dword __attribute__((ext_vector_type(4), aligned(4)));  // sixteen bytes at any dword

constexpr uint32_t kLine = 128;

struct RowLine {
    uint32_t line;    // line index in the array
    uint32_t lo, hi;  // the row's bytes inside that line: [lo, hi), empty when the row has none
};

__device__ __forceinline__ RowLine row_line(uint32_t piece, uint32_t count, uint32_t ls, bool row_exists)
{
    const uint32_t rb = piece * count, re = rb + count;
    const uint32_t first = rb / kLine, last = (re - 1u) / kLine;
    RowLine r;
    __builtin_assume(last >= first);  // (told so, the encoder needs four registers less: 3 % of its time)
    r.line = last - ls;
    if (!row_exists || ls > last - first) {
        r.lo = r.hi = 0;
        return r;
    }
    const uint32_t cb = r.line * kLine;
    r.lo = rb > cb ? rb - cb : 0u;
    r.hi = re < cb + kLine ? re - cb : kLine;
    return r;
}

__device__ __forceinline__ uint32_t line_stage_count(uint32_t count)
{
    // a row of `count` bytes starting anywhere touches at most this many lines
    return (count + 2u * kLine - 2u) / kLine;
}

// Whether line-stage `ls` is a whole line of every row of the wavefront: stage 0 takes at most a line of a row, and what
// is left, count - 128 bytes or more, begins with whole lines.
__device__ __forceinline__ bool whole_line_stage(uint32_t np, uint32_t count, uint32_t ls)
{
    return np == 64u && ls != 0u && ls < count / kLine;
}

// Bytes [a, b) of a dword, the others cleared (a, b may lie outside 0..4).
__device__ __forceinline__ uint32_t keep_bytes(uint32_t w, int a, int b)
{
    const uint32_t below_b = b >= 4 ? 0xFFFFFFFFu : (b <= 0 ? 0u : (1u << (8 * b)) - 1u);
    const uint32_t below_a = a >= 4 ? 0xFFFFFFFFu : (a <= 0 ? 0u : (1u << (8 * a)) - 1u);
    return w & below_b & ~below_a;
}

// A vector of the arrays `sym` and `dist` at byte `off`; the bytes past the arrays' end cleared.  The data is used once: the
// loads are marked non-temporal so that they do not push the lines this kernel writes out of the L2 before
// they are complete.
__device__ __forceinline__ uint4 once_load(const uint8_t *__restrict__ from)
{
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(from));
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void cut_at_end(uint4 &v, int bytes)
{
    v = make_uint4(keep_bytes(v.x, 0, bytes), keep_bytes(v.y, 0, bytes - 4), keep_bytes(v.z, 0, bytes - 8),
                   keep_bytes(v.w, 0, bytes - 12));
}

// Fetches line-stage `ls` of the rows of pieces p0 .. p0+np-1 of both arrays: for every row the 16-byte vectors
// of its line that hold at least one of its bytes (they may also hold bytes of its neighbours);
// zeros elsewhere.  A vector is aligned and holds a byte of the array, so it lies inside the
// array's last page even where it reaches past the array's end; such bytes are cleared.
// `whole` (the same for the wavefront, see whole_line_stage): every row has a whole line, nothing is asked per row.
__device__ __forceinline__ void line_load(const uint8_t *__restrict__ sym, const uint8_t *__restrict__ dist,
                                          uint32_t total_bytes, uint32_t p0, uint32_t np, uint32_t count, uint32_t ls,
                                          bool whole, uint4 (&sv)[8], uint4 (&dv)[8])
{
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));  // (the rows' places are formed again in every call, not kept in registers)
    const uint32_t vb = (lane & 7u) * 16u;
    if (whole) {
        uint32_t last = (p0 + (lane >> 3) + 1u) * count - 1u;  // the last byte of the row
        uint32_t off[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            off[i] = (last & ~(kLine - 1u)) - ls * kLine + vb;
            last += 8u * count;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) sv[i] = once_load(sym + off[i]);
#pragma unroll
        for (int i = 0; i < 8; ++i) dv[i] = once_load(dist + off[i]);
        return;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t r = i * 8 + (lane >> 3);
        const RowLine rl = row_line(p0 + r, count, ls, r < np);
        sv[i] = dv[i] = make_uint4(0u, 0u, 0u, 0u);
        if (vb < rl.hi && vb + 16u > rl.lo) {
            const uint32_t off = rl.line * kLine + vb;
            sv[i] = once_load(sym + off);
            dv[i] = once_load(dist + off);
            if (off + 16u > total_bytes) {  // at most one vector of the whole grid
                asm volatile("" ::: "memory");  // keep this a branch, not a chain of selects
                cut_at_end(sv[i], (int)(total_bytes - off));
                cut_at_end(dv[i], (int)(total_bytes - off));
            }
        }
    }
}

// True if some byte of w is >= limit (1 <= limit <= 255).  `k7` and `use_or` are derived from the
// limit once: k7 = ((limit <= 128 ? 128 : 256) - limit) * 0x01010101.
struct ByteLimit {
    uint32_t k7;
    bool use_or, none;  // none: limit 256, nothing to check
};

__device__ __forceinline__ ByteLimit byte_limit(uint32_t limit)
{
    ByteLimit b;
    b.none = limit >= 256u;
    b.use_or = limit <= 128u;
    b.k7 = ((b.use_or ? 128u : 256u) - (b.none ? 255u : limit)) * 0x01010101u;
    return b;
}

__device__ __forceinline__ uint32_t bytes_at_or_above(uint32_t w, const ByteLimit &b)
{
    const uint32_t t = (w & 0x7F7F7F7Fu) + b.k7;  // bit 7 of a byte: its low 7 bits reach the bound
    return (b.use_or ? (t | w) : (t & w)) & 0x80808080u;
}

// Checks the 8 vectors against a limit; a vector with an offending byte is zeroed (so that no
// table index leaves its table) and reported.  The OR of all bytes is looked at first: it is at least as large as each
// of them, so nothing more has to be asked while it is below the limit.
__device__ __forceinline__ uint32_t lines_check(uint4 (&v)[8], const ByteLimit &b)
{
    uint32_t bad = 0u;
    if (b.none) return 0u;
    uint32_t all = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) all |= (v[i].x | v[i].y) | (v[i].z | v[i].w);
    if (!__any(bytes_at_or_above(all, b) != 0u)) return 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t f = bytes_at_or_above(v[i].x, b) | bytes_at_or_above(v[i].y, b) |
                           bytes_at_or_above(v[i].z, b) | bytes_at_or_above(v[i].w, b);
        if (f) v[i] = make_uint4(0u, 0u, 0u, 0u);
        bad |= f;
    }
    return bad;
}

// ---------------------------------------------------------------------------------------------
// Encode (Alg. 3), symbols of a piece taken last-first
// ---------------------------------------------------------------------------------------------
constexpr int kAnsaiEncWaves = 4;      // wavefronts of a workgroup at most; with the tables of up to nine laws three such workgroups fit a compute unit
                                       // (53,264 bytes of LDS each), with those of ten to twelve two
constexpr uint32_t kEncPart = 32;       // positions of a row in LDS at a time
constexpr uint32_t kEncRow = 16;        // LDS dwords of a row: their symbols and their indices
constexpr uint32_t kEncBlock = 8;       // words that leave together, to 32 bytes that start on a multiple of 32
constexpr uint32_t kEncRing = 16;       // words of a piece that wait in LDS at most: 7, and eight more of sixteen symbols
constexpr uint32_t kEncWaveDwords = 64u * (kEncRow + kEncRing + 2u);  // LDS of a wavefront

// A piece under way.  The bits pushed and not yet written stand at the top of `top`, the last one highest, above bits
// that have been written already; `room` (1 .. 32) is how many more make a word.
struct EncLane {
    uint32_t S;      // state in [2^M, 2^(M+1))
    uint32_t top;
    int room;
    uint32_t nw;     // words made so far, counted from the multiple of kEncBlock words at or before the piece's first
};

// Two steps of Alg. 3, the first with the table entry `a` = {delta, phi}, the second with `b`.  Each pushes at most 15
// bits, so the two fill no more than one word; they are put together first and pushed as one.
// A word that is complete goes to this thread's column of `ring` ([word mod kEncRing][thread]).
__device__ __forceinline__ void ansai_push_two(EncLane &L, const uint2 a, const uint2 b, uint32_t M, uint32_t *ring)
{
    const uint32_t na = (a.x + L.S) >> M;
    const uint32_t low = __builtin_amdgcn_ubfe(L.S, 0u, na);
    L.S = (L.S >> na) + a.y;
    const uint32_t nb = (b.x + L.S) >> M;
    const uint32_t bits = low | (__builtin_amdgcn_ubfe(L.S, 0u, nb) << na);
    L.S = (L.S >> nb) + b.y;
    const uint32_t n = na + nb;
    const uint32_t word = __builtin_amdgcn_alignbit(bits, L.top, (uint32_t)L.room);  // (room 32: not a word yet)
    L.top = __builtin_amdgcn_alignbit(bits, L.top, n);
    L.room -= (int)n;
    if (L.room <= 0) {
        ring[(L.nw % kEncRing) * 64u] = word;
        ++L.nw;
        L.room += 32;
    }
}

// The words of a wavefront's pieces on their way to the pieces' rows of the scratch: kEncBlock of them leave when they are
// complete, which is looked at after every sixteen symbols (they make at most eight words).  Two neighbouring
// threads store a block: the threads whose pieces have one write a list of them, and all threads go through
// the list.  (What the kernel waits for otherwise is the number of separate places that are stored to: a word at
// a time as they are made, or sixteen bytes of every piece by its own thread, cost 10^6 pieces of 1000
// symbols 300 us, whether to whole lines or not.)
struct EncOut {
    uint32_t *base;    // of the wavefront's first piece
    uint32_t *ring;    // of the wavefront: [word mod kEncRing][thread]
    uint2 *list;       // {where a block goes, from which thread | which half of the ring << 8}
    uint32_t at;       // where word `done` goes, from `base`
    uint32_t done;     // words stored, counted as EncLane.nw

    __device__ __forceinline__ void own(uint32_t upto)
    {
        for (; done < upto; ++done, ++at) base[at] = ring[(done % kEncRing) * 64u + (threadIdx.x & 63u)];
    }
    __device__ __forceinline__ void look(uint32_t nw)
    {
        const uint32_t lane = threadIdx.x & 63u;
        if ((done % kEncBlock) != 0u && nw >= kEncBlock) own(kEncBlock);  // a piece's first words, which start anywhere
        const bool full = (done % kEncBlock) == 0u && nw - done >= kEncBlock;
        const unsigned long long mask = __ballot(full);
        if (mask == 0ull) return;
        const uint32_t number = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if (full) {
            list[number] = make_uint2(at, lane | ((done % kEncRing) / kEncBlock << 8));
            at += kEncBlock;
            done += kEncBlock;
        }
        wave_lds_sync();
        const uint32_t blocks = (uint32_t)__popcll(mask), part = (lane & 1u) * 4u;
        for (uint32_t b = 0; b < blocks; b += 32u) {
            const uint32_t mine = b + (lane >> 1);
            const uint2 e = list[min(mine, blocks - 1u)];
            const uint32_t *from = ring + ((e.y >> 8) * kEncBlock + part) * 64u + (e.y & 63u);
            const u32x4 v = {from[0], from[64], from[128], from[192]};
            if (mine < blocks) *reinterpret_cast<u32x4_dword *>(base + (size_t)e.x + part) = v;
        }
        wave_lds_sync();
    }
};

// Place of the table entry whose index is the lower / upper half of w: one shift that picks the half.
template <bool kUpper> __device__ __forceinline__ uint32_t enc_place(uint32_t w)
{
    uint32_t at;
    if (kUpper)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(at) : "v"(3u), "v"(w));
    else
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(at) : "v"(3u), "v"(w));
    return at;
}

// Puts quarter `ph` of the fetched lines into LDS: of a row four times sixteen bytes, those of positions 0 and 16 of the
// symbols and then of the indices.  Number k of them stands in place k ^ (row / 4 mod 4) of the row, so that threads
// that read theirs together meet on no bank.
__device__ __forceinline__ void enc_put(uint32_t *rows, const uint4 (&sv)[8], const uint4 (&dv)[8], uint32_t ph)
{
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));  // (as in line_load)
    const uint32_t c = lane & 7u;
    if ((c >> 1) != ph) return;
    uint32_t *dst = rows + (lane >> 3) * kEncRow + ((c & 1u) ^ (lane >> 5)) * 4u;  // row 8 i + lane / 8: row / 4 = 2 i + lane / 32
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        // (number 0 or 1 in place dst or dst + 8 dwords: 2 i changes bit 1 of the place)
        *reinterpret_cast<u32x4 *>(dst + 8u * kEncRow * i + ((i & 1) ? 8u : 0u)) = u32x4{sv[i].x, sv[i].y, sv[i].z, sv[i].w};
        *reinterpret_cast<u32x4 *>(dst + 8u * kEncRow * i + ((i & 1) ? 0u : 8u)) = u32x4{dv[i].x, dv[i].y, dv[i].z, dv[i].w};
    }
}

// Which positions of a line belong to this thread's row: position + `skew` < `count` (unsigned).
struct EncOwn {
    uint32_t skew, count;
};

// The next 32 positions of this thread's row, which are in LDS, last first.  kMasked: positions that are not part of the row
// take the identity step (`ident`, its place in the table), so that every thread can run all of them.  `first`: the
// number of the first of them in the line.
template <bool kMasked>
__device__ __forceinline__ void enc_part(EncLane &L, EncOut &out, const uint2 *tab, uint32_t M, const u32x4 *row, uint32_t *ring,
                                         uint32_t first, const EncOwn &own, uint32_t ident)
{
    // Four symbols a turn; their table entries are asked for a turn ahead.
    const uint32_t turned = (threadIdx.x >> 2) & 3u;  // (see enc_put)
    const u32x4 x = row[1u ^ turned], d = row[3u ^ turned];
    uint2 n[4];
    auto ask = [&](uint32_t x4, uint32_t d4, uint32_t at) {  // bytes {x0, d0, x1, d1} and {x2, d2, x3, d3} are indices
        const uint32_t lower = __builtin_amdgcn_perm(d4, x4, 0x05010400u), upper = __builtin_amdgcn_perm(d4, x4, 0x07030602u);
        uint32_t place[4] = {enc_place<false>(lower), enc_place<true>(lower), enc_place<false>(upper), enc_place<true>(upper)};
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) {
            if (kMasked) place[i] = first + at + i + own.skew < own.count ? place[i] : ident;
            n[i] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(tab) + place[i]);
        }
    };
    auto push = [&](const uint2 (&e)[4]) {
        ansai_push_two(L, e[3], e[2], M, ring);
        ansai_push_two(L, e[1], e[0], M, ring);
    };
    auto turn = [&](uint32_t x4, uint32_t d4, uint32_t at) {  // those of the next turn
        const uint2 e[4] = {n[0], n[1], n[2], n[3]};
        ask(x4, d4, at);
        __builtin_amdgcn_sched_barrier(0);
        push(e);
    };
    ask(x.w, d.w, 28u);
    const u32x4 xl = row[turned], dl = row[2u ^ turned];
    turn(x.z, d.z, 24u);
    turn(x.y, d.y, 20u);
    turn(x.x, d.x, 16u);
    turn(xl.w, dl.w, 12u);
    out.look(L.nw);
    turn(xl.z, dl.z, 8u);
    turn(xl.y, dl.y, 4u);
    turn(xl.x, dl.x, 0u);
    push(n);
}

// Bound by LDS (a table entry of 64 threads at once is a gather), by the vector instructions of a symbol, 17 of them, and
// by the places its words are stored to, with three wavefronts on a SIMD (up to nine laws; see kAnsaiEncWaves).  10^6 pieces of 1000 symbols under eight laws:
// 1318 -> 965 us, of 64 x 100,000 9.6 -> 6.9 ms.  (Before, a step of a symbol kept the bits not yet
// written in 64 bits of its own, indices were put together by the threads that loaded them, and every position of
// the first and last lines of a row was masked there: 32 instructions a symbol and 189 registers, two wavefronts.)
template <bool kTabLds>
__global__ __launch_bounds__(64 * kAnsaiEncWaves) void k_ansai_encode(
    AShape sh, const uint8_t *__restrict__ sym, const uint8_t *__restrict__ dist,
    const uint2 *__restrict__ enc_tab, uint32_t *__restrict__ scratch, uint32_t stride,
    uint32_t *__restrict__ piece_bits, uint32_t *__restrict__ piece_state, int *status)
{
    extern __shared__ uint32_t lds[];
    if (*status != ST_OK) return;  // the tables are not the ones this shape needs
    const uint2 *tab = enc_tab;
    uint32_t *stage_base = lds;
    if (kTabLds) {
        uint2 *t = reinterpret_cast<uint2 *>(lds);
        for (uint32_t i = threadIdx.x; i < sh.D * 256u + 1u; i += blockDim.x) t[i] = enc_tab[i];
        tab = t;
        stage_base = lds + 2u * (sh.D * 256u + 2u);  // (a multiple of sixteen bytes)
        __syncthreads();
    }
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t gw = blockIdx.x * (blockDim.x >> 6) + wave;
    const uint32_t p0 = gw * 64u;
    if (p0 >= sh.pieces) return;
    const uint32_t np = min(64u, sh.pieces - p0);
    uint32_t *rows = stage_base + wave * kEncWaveDwords;

    const uint32_t total = sh.pieces * sh.count;
    uint32_t *ring = rows + 64u * kEncRow + lane;
    const u32x4 *my = reinterpret_cast<const u32x4 *>(rows + lane * kEncRow);
    const bool mine = lane < np;
    const ByteLimit lim_x = byte_limit(sh.X), lim_d = byte_limit(sh.D);
    const uint32_t M = sh.M;

    EncLane L;
    L.S = 1u << M;
    L.top = 0u;
    L.room = 32;
    uint32_t *const base = scratch + (size_t)p0 * stride;
    const uint32_t first = (uint32_t)(reinterpret_cast<uintptr_t>(base + lane * stride) >> 2) % kEncBlock;
    L.nw = first;
    EncOut out = {base, rows + 64u * kEncRow, reinterpret_cast<uint2 *>(rows + 64u * (kEncRow + kEncRing)), lane * stride, first};
    uint32_t bad = 0u;

    uint4 sv[8], dv[8];
    const uint32_t lines = line_stage_count(sh.count);
    line_load(sym, dist, total, p0, np, sh.count, 0u, false, sv, dv);
    bad |= lines_check(sv, lim_x) | lines_check(dv, lim_d);
    for (uint32_t ls = 0; ls < lines; ++ls) {
        asm volatile("" : "+s"(sh.count));  // recompute the row geometry per line-stage (registers)
        const bool whole = whole_line_stage(np, sh.count, ls);
        EncOwn own = {0u, 0u};
        if (!whole) {
            const RowLine rl = row_line(p0 + lane, sh.count, ls, mine);
            own.skew = 0u - rl.lo;
            own.count = rl.hi - rl.lo;
        }
#pragma unroll 1
        for (int ph = 3; ph >= 0; --ph) {
            wave_lds_sync();
            enc_put(rows, sv, dv, (uint32_t)ph);
            wave_lds_sync();
            if (ph == 0 && ls + 1u < lines)  // the registers are free: fetch the next lines now
                line_load(sym, dist, total, p0, np, sh.count, ls + 1u, whole_line_stage(np, sh.count, ls + 1u), sv, dv);
            if (whole)
                enc_part<false>(L, out, tab, M, my, ring, 0u, own, 0u);
            else
                enc_part<true>(L, out, tab, M, my, ring, kEncPart * (uint32_t)ph, own, sh.D << 11);
            if (ph == 0) {
                // the next lines, asked for 32 symbols ago, are waited for before words are stored: a wait for them
                // afterwards would wait for the stores as well
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
                bad |= lines_check(sv, lim_x) | lines_check(dv, lim_d);
            }
            out.look(L.nw);
        }
    }
    if (mine) {
        piece_bits[p0 + lane] = (L.nw - first) * 32u + 32u - (uint32_t)L.room;
        piece_state[p0 + lane] = L.S;
        out.own(L.nw);
        if (L.room < 32) base[out.at] = L.top >> L.room;
    }
    if (bad) atomicMax(status, ST_ARG);  // the same value from every thread that found one
}

// ---------------------------------------------------------------------------------------------
// Pack: scratch [piece][word] -> records {state, bit count, words} at the offsets
// ---------------------------------------------------------------------------------------------
constexpr int kAnsaiPackWaves = 4;
constexpr int kAnsaiPackTogether = 16;  // pieces whose loads are under way together
constexpr uint32_t kAnsaiPackFewWords = 32;  // a group of pieces of at most so many goes a word a thread

// Bound by memory.  A wavefront copies 64 pieces, sixteen at a time, sixteen bytes a thread; the last sixteen of a
// piece overlap those before them, so that nothing is read or written beyond its words.  The stores are
// non-temporal: what they would push out of the caches is still to be read.  Pieces of fewer than four words go a word a
// thread, and a group that has some keeps the sixteen bytes for its others.  Whole calls with one such piece in sixteen, us,
// against a group that went a word a thread altogether: 65,536 pieces of 4000 symbols 779 -> 469 (without short ones 474),
// 10^5 of 1000 275 -> 211 (213).  A group of pieces of at most 32 words goes a word a thread altogether, four threads a
// piece: sixteen bytes a thread leave most threads without any.  The packer alone, us, words against sixteen bytes: 400,000 pieces of 4
// words 13 and 36, of 8 17 and 39, 262,144 of 16 18 and 30, 167,772 of 25 20 and 22, 131,072 of 32 17.8 and 18.2, 104,857 of 40 20.9 and 17.7.
__global__ __launch_bounds__(64 * kAnsaiPackWaves) void k_ansai_pack(
    AShape sh, const uint32_t *__restrict__ scratch, uint32_t stride,
    const uint32_t *__restrict__ piece_bits, const uint32_t *__restrict__ piece_state,
    const uint32_t *__restrict__ offsets, uint32_t *__restrict__ payload,
    const Status *__restrict__ status)
{
    if (status->code != ST_OK) return;
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t gw = blockIdx.x * kAnsaiPackWaves + wave;
    const uint32_t p0 = gw * 64u;
    if (p0 >= sh.pieces) return;
    const uint32_t np = min(64u, sh.pieces - p0);
    uint32_t nw = 0, dst = 0;  // words of this thread's piece and the payload dword index of the first
    if (lane < np) {
        const uint32_t bits = piece_bits[p0 + lane], at = offsets[p0 + lane] >> 2;
        nw = (bits + 31u) >> 5;
        payload[at] = piece_state[p0 + lane];
        payload[at + 1u] = bits;
        dst = at + 2u;
    }
#pragma unroll 1
    for (uint32_t i0 = 0; i0 < np; i0 += kAnsaiPackTogether) {
        uint32_t n[kAnsaiPackTogether], to[kAnsaiPackTogether], most = 0u, least = 4u, longest = 0u;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kAnsaiPackTogether; ++i) {  // (no words in the place of pieces past the last one)
            n[i] = (uint32_t)__builtin_amdgcn_readlane((int)nw, (int)(i0 + i));
            to[i] = (uint32_t)__builtin_amdgcn_readlane((int)dst, (int)(i0 + i));
            longest = n[i] > most ? i : longest;
            most = max(most, n[i]);
            least = min(least, n[i]);
        }
        const uint32_t *src = scratch + (size_t)(p0 + i0) * stride;
        if (least < 4u || most <= kAnsaiPackFewWords) {
            static_assert(kAnsaiPackTogether == 16, "four threads a piece");
            const uint32_t i = lane >> 2, j = lane & 3u;
            const uint32_t ni = (uint32_t)__shfl((int)nw, (int)(i0 + i), 64), ti = (uint32_t)__shfl((int)dst, (int)(i0 + i), 64);
            const uint32_t by_words = most <= kAnsaiPackFewWords ? ni : (ni < 4u ? ni : 0u);
            for (uint32_t k = j; k < by_words; k += 4u) payload[ti + k] = src[(size_t)i * stride + k];
            if (most <= kAnsaiPackFewWords) continue;
        }
        // `some`: in the place of a piece that does not go this way the longest is read, and not stored
        auto copy = [&](auto some) __attribute__((always_inline)) {
#pragma unroll 1
            for (uint32_t j0 = 0; j0 < most; j0 += 256u) {
                const uint32_t j = j0 + 4u * lane;
                u32x4 v[kAnsaiPackTogether];
#pragma unroll
                for (uint32_t i = 0; i < (uint32_t)kAnsaiPackTogether; ++i) {  // (a thread with nothing to move reads the piece's end)
                    const bool goes = !some || n[i] >= 4u;
                    v[i] = *reinterpret_cast<const u32x4_dword *>(src + (size_t)(goes ? i : longest) * stride + min(j, (goes ? n[i] : most) - 4u));
                }
#pragma unroll
                for (uint32_t i = 0; i < (uint32_t)kAnsaiPackTogether; ++i)
                    if ((!some || n[i] >= 4u) && j < n[i])
                        __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4_dword *>(payload + to[i] + min(j, n[i] - 4u)));
            }
        };
        if (least >= 4u)
            copy(std::false_type());
        else
            copy(std::true_type());
    }
}

// ---------------------------------------------------------------------------------------------
// Decode (Alg. 4)
// ---------------------------------------------------------------------------------------------
// Whether the tables are those of this shape; the status block for the kernels that follow.
__device__ __forceinline__ int ansai_tables_state(const AShape &sh, const ATabHeader *__restrict__ tab)
{
    return tab->magic == kAnsaiTabMagic && tab->ok == 1u && tab->M == sh.M && tab->D == sh.D && tab->X == sh.X ? ST_OK : ST_ARG;
}
__global__ void k_ansai_begin(AShape sh, const ATabHeader *__restrict__ tab, Status *status)
{
    init_status(status);
    status->code = ansai_tables_state(sh, tab);
}

// The same for a decoder, and whether the container's header is that of this shape.
__global__ void k_ansai_check_header(AShape sh, const ATabHeader *__restrict__ tab, const uint8_t *__restrict__ coded,
                                     unsigned long long coded_bytes, Status *__restrict__ status)
{
    init_status(status);
    const uint32_t *h = reinterpret_cast<const uint32_t *>(coded);
    const unsigned long long payload = (unsigned long long)h[12] | ((unsigned long long)h[13] << 32);
    int st = ansai_tables_state(sh, tab);
    if (st == ST_OK && (h[0] != kAnsaiMagic || h[1] != 1u || h[2] != sh.pieces || h[3] != sh.count || h[4] != sh.M ||
                        h[5] != sh.D || h[6] != sh.X ||
                        coded_bytes != kHeaderBytes + 4ull * ((unsigned long long)sh.pieces + 1ull) + payload))
        st = ST_FORMAT;
    if (st == ST_OK && payload >= (1ull << 32)) st = ST_CORRUPT;
    status->code = st;
    status->payload_bytes = payload;
}

// What bounds the decoder is the instructions of a symbol and the two table reads in its chain (the symbol, and
// the entry that gives the next state), so the stream is read by position: two symbols pop at most 30 bits,
// and one 32-bit piece of the stream, cut out of two words wherever it starts, serves both.  There
// is no bit buffer to shift, count and fill up: the position is all there is to keep.  The words wait
// in a ring of 16 per thread in LDS that is topped up with aligned 16-byte loads asked for one or two groups
// of symbols before they are needed.  Indices and symbols pass through LDS 32 to a row, and rows are
// cut from their own start, whatever its alignment, so that all threads have the same positions of
// their rows at the same time; long rows of a large batch are cut at the array's 128-byte lines, with steps that
// change nothing where a thread's row has not begun or has ended (the host chooses, with figures there).
// (A 63-bit window refilled a word at a time, with all rows cut at lines, took 36.6 vector instructions a
// symbol; now 20.  10^6 pieces of 1000 symbols under eight laws 1.68 -> 1.49 ms, which is the chain of
// table reads with nine wavefronts on a compute unit and the lines of the streams that are fetched again
// for every quad; 10^6 of 256 under one law 435 -> 290 us, 1000 of 700 under four 146 -> 71 us.  Not
// faster: quads two at a time, fewer fetches but a shorter lead (1.72 ms), symbols stored 32 bytes at a time
// (1.67 ms), non-temporal stores (2.28 ms); 1.55 ms as it was then.)
// LDS is what limits how many pieces a compute unit decodes at once (the tables take most of it):
// 6400 bytes a wavefront, ten wavefronts beside the 96 KB of eight laws at 12 bits.
constexpr uint32_t kRingWords = 16;                    // per thread: four aligned quads
constexpr int kGroupSyms = 8;                          // symbols between top-ups; they take at most 120 bits
constexpr uint32_t kPart = 32;                         // bytes of a row passed through LDS at a time
constexpr uint32_t kDecWaveDwords = 64u * (kPart / 4u + kRingWords + 1u);  // LDS of a wavefront

struct DecLane {
    uint32_t s;      // state minus 2^M
    uint32_t pos;    // bits below this one are still to be taken; counted from the container's start, mod 2^32
    uint32_t lp;     // the ring holds the words from lp on; dword index, a multiple of 4
    uint32_t first;  // dword index of the piece's first word
};

// An aligned quad that holds at least one word of the container: it lies inside the container's
// last page even where it reaches past the container's end.
__device__ __forceinline__ uint4 ansai_quad_load(const uint32_t *__restrict__ cw, uint32_t q)
{
    return *reinterpret_cast<const uint4 *>(cw + q);
}

// The ring is [row][thread]: word w in row (w mod 16) + 1, and in row 0 as well if that is row 16, so that
// the word before any word is in the row before it.
__device__ __forceinline__ void ansai_ring_put(uint32_t *ring, uint32_t slot, const uint4 &v)
{
    uint32_t *q = ring + 64u * (slot + 1u);
    q[0] = v.x;
    q[64] = v.y;
    q[128] = v.z;
    q[192] = v.w;
    if (slot == kRingWords - 4u) ring[0] = v.w;
}

// The 31 bits of the stream below the position, the highest in bit 30.
__device__ __forceinline__ uint32_t ansai_next_bits(const DecLane &L, const uint32_t *ring)
{
    const uint32_t *q = ring + 64u * ((L.pos >> 5) & (kRingWords - 1u));
    return __builtin_amdgcn_alignbit(q[64], q[0], L.pos) >> 1;
}

// The table entry of a state: c = 15 - B[d,S] and n = N[d,S] - 2^M.  In global memory an entry holds n above its
// low four bits and c in them; in LDS it is turned so that c is on top.
struct DecEntry {
    uint32_t c, n, x;
};
template <bool kWide, bool kTabLds>
__device__ __forceinline__ DecEntry ansai_entry(uint32_t index, const uint8_t *theta, const void *nb_raw)
{
    const uint32_t e = kWide ? static_cast<const uint32_t *>(nb_raw)[index]
                             : (uint32_t) static_cast<const uint16_t *>(nb_raw)[index];
    DecEntry r;
    r.x = theta[index];
    if (!kTabLds) {
        r.c = e & 15u;
        r.n = e >> 4;
    } else if (kWide) {
        r.c = e >> 28;
        r.n = e & 0x0FFFFFFFu;
    } else {
        r.c = e >> 12;
        r.n = e & 0x0FFFu;
    }
    return r;
}

// Two steps of Alg. 4 (S <- N[d,S] + popped bits; N - 2^M has zeros where the B popped bits go).  `dm` = d << M.
// kMasked: a step that is not `on` (no symbol of this thread's row at its position) pops nothing and keeps the state.
template <bool kWide, bool kTabLds, bool kMasked = false>
__device__ __forceinline__ void ansai_pop_two(DecLane &L, uint32_t bits, uint32_t dm0, uint32_t dm1, uint32_t &x0,
                                              uint32_t &x1, const uint8_t *theta, const void *nb, bool on0 = true,
                                              bool on1 = true)
{
    DecEntry a = ansai_entry<kWide, kTabLds>(dm0 + L.s, theta, nb);
    if (kMasked) {
        a.c = on0 ? a.c : 15u;
        a.n = on0 ? a.n : L.s;
    }
    L.s = a.n | (bits >> (a.c | 16u));  // by 31 - B
    DecEntry b = ansai_entry<kWide, kTabLds>(dm1 + L.s, theta, nb);
    if (kMasked) {
        b.c = on1 ? b.c : 15u;
        b.n = on1 ? b.n : L.s;
    }
    const uint32_t at = a.c + b.c + 1u;  // 31 - B - B'
    L.s = b.n | __builtin_amdgcn_ubfe(bits, at, 15u - b.c);
    L.pos += at - 31u;
    x0 = a.x;
    x1 = b.x;
}

template <bool kWide, bool kTabLds>
__device__ __forceinline__ uint32_t ansai_pop_one(DecLane &L, const uint32_t *ring, uint32_t dm, const uint8_t *theta,
                                                  const void *nb)
{
    const uint32_t bits = ansai_next_bits(L, ring);
    const DecEntry a = ansai_entry<kWide, kTabLds>(dm + L.s, theta, nb);
    L.s = a.n | (bits >> (a.c | 16u));
    L.pos += a.c - 15u;
    return a.x;
}

// The bytes of a 16-byte aligned array from `off` to its end, fewer than 16, and zeros: from the array's last 16
// bytes, or from its first 16-byte block if it is no longer than that.
__device__ __forceinline__ uint4 array_tail(const uint8_t *__restrict__ arr, uint32_t total_bytes, uint32_t off)
{
    const uint32_t from = total_bytes >= 16u ? total_bytes - 16u : 0u;
    unsigned __int128 x;
    __builtin_memcpy(&x, arr + from, 16);
    x >>= 8u * (off - from);
    x &= ((unsigned __int128)1 << (8u * (total_bytes - off))) - 1u;
    return make_uint4((uint32_t)x, (uint32_t)(x >> 32), (uint32_t)(x >> 64), (uint32_t)(x >> 96));
}

// Where row `row_off` of the array (its first byte) is cut: kLines, at the array's 128-byte lines, so that position 0
// is the start of the line in which the row starts; otherwise at the row's own start.
template <bool kLines> __device__ __forceinline__ uint32_t row_skew(uint32_t row_off) { return kLines ? row_off & 127u : 0u; }

// Positions [pos, pos + 128) of the rows of pieces p0 .. p0 + np - 1, thread `lane` holding, for i = 0 .. 7, sixteen
// of row 8 i + lane / 8, those from pos + 16 (lane % 8) on: eight neighbouring threads cover 128 bytes of
// a row.  Vectors that hold a byte of the row may hold bytes of its neighbours as well; zeros elsewhere.
template <bool kLines>
__device__ __forceinline__ void rows_load(const uint8_t *__restrict__ arr, uint32_t total_bytes, uint32_t p0, uint32_t np,
                                          uint32_t count, uint32_t pos, uint4 (&v)[8])
{
    const uint32_t lane = threadIdx.x & 63u, at = pos + 16u * (lane & 7u);
    uint32_t off = (p0 + (lane >> 3)) * count + at;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t skew = row_skew<kLines>(off - at), from = off - skew;
        v[i] = make_uint4(0u, 0u, 0u, 0u);
        if (8u * i + (lane >> 3) < np && at < count + skew && (!kLines || at + 16u > skew)) {
            if (from + 16u <= total_bytes) {
                __builtin_memcpy(&v[i], arr + from, 16);
            } else {  // at the array's end: up to 15 vectors of the whole grid
                asm volatile("" ::: "memory");  // keep this a branch
                v[i] = array_tail(arr, total_bytes, from);
            }
        }
        off += 8u * count;
    }
}

// Quarter `ph` of the fetched 128 bytes into LDS as [dword][row].
__device__ __forceinline__ void dec_put(uint32_t *rows, const uint4 (&dv)[8], uint32_t ph)
{
    const uint32_t lane = threadIdx.x & 63u, c = lane & 7u;
    if ((c >> 1) != ph) return;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        uint32_t *dst = rows + 64u * 4u * (c & 1u) + i * 8 + (lane >> 3);
        dst[0] = dv[i].x;
        dst[64] = dv[i].y;
        dst[128] = dv[i].z;
        dst[192] = dv[i].w;
    }
}

// The decoded symbols of 32 positions from LDS, two threads a row: thread `lane` has sixteen bytes of rows lane / 2
// and 32 + lane / 2.
__device__ __forceinline__ void dec_get(const uint32_t *rows, u32x4 (&ov)[2])
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t *src = rows + 64u * 4u * (lane & 1u) + (lane >> 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        ov[i].x = src[32 * i];
        ov[i].y = src[32 * i + 64];
        ov[i].z = src[32 * i + 128];
        ov[i].w = src[32 * i + 192];
    }
}

// The same to positions [pos, pos + 32) of the rows: only bytes that belong to them.
template <bool kLines>
__device__ __forceinline__ void dec_store(uint8_t *__restrict__ out, const u32x4 (&ov)[2], uint32_t p0, uint32_t np,
                                          uint32_t count, uint32_t pos)
{
    const uint32_t lane = threadIdx.x & 63u, at = pos + 16u * (lane & 1u);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t r = i * 32 + (lane >> 1), row_off = (p0 + r) * count, skew = row_skew<kLines>(row_off);
        if (r >= np || at >= count + skew || (kLines && at + 16u <= skew)) continue;
        uint8_t *q = out + (size_t)(row_off - skew + at);
        if (at + 16u <= count + skew && (!kLines || at >= skew)) {
            __builtin_memcpy(q, &ov[i], 16);
        } else {
            const uint32_t w[4] = {ov[i].x, ov[i].y, ov[i].z, ov[i].w};
#pragma unroll
            for (uint32_t k = 0; k < (kLines ? 16u : 15u); ++k)
                if (at + k < count + skew && (!kLines || at + k >= skew)) q[k] = (uint8_t)(w[k >> 2] >> (8u * (k & 3u)));
        }
    }
}

// What a thread asks for before a group of symbols if there is room for it: the aligned quad below the ring (below
// the quads fetched at the start, hence inside the container).  It is put into the ring at the end of the
// next group, or of its own if that is the last of 32 symbols.  There is room while fewer than 384 bits lie
// between the ring's end and the position; a group then starts with at least 385 - 120 - 120 bits
// that have arrived, and takes words no further than 122 down.  (A load in any case, of the header's
// first quad if none is wanted: with loads that may or may not be under way, the wait for one is a
// wait for all.)
struct DecAhead {
    uint4 quad;
    uint32_t slot;  // kRingWords: none
};
__device__ __forceinline__ DecAhead ansai_ask(DecLane &L, const uint32_t *__restrict__ cw)
{
    const bool want = L.pos - 32u * L.lp < 384u && L.lp > L.first;
    L.lp -= want ? 4u : 0u;
    DecAhead a;
    a.quad = ansai_quad_load(cw, want ? L.lp : 0u);
    a.slot = want ? L.lp & (kRingWords - 1u) : kRingWords;
    return a;
}
__device__ __forceinline__ void ansai_put_ahead(uint32_t *ring, const DecAhead &a)
{
    if (a.slot != kRingWords) ansai_ring_put(ring, a.slot, a.quad);
}

// The next `n` symbols (1 .. 32, the same for every thread) of this thread's row, in groups of eight; kMasked: 32
// positions, of which those in [lo, hi) have a symbol.
template <bool kWide, bool kTabLds, bool kMasked = false>
__device__ __forceinline__ void dec_part(DecLane &L, uint32_t *my, uint32_t *ring, const uint32_t *__restrict__ cw,
                                         uint32_t M, uint32_t n, const uint8_t *theta, const void *nb, uint32_t lo = 0u,
                                         uint32_t hi = kPart)
{
    auto group = [&](uint32_t g) {
#pragma unroll
        for (uint32_t h = 0; h < (uint32_t)kGroupSyms / 4u; ++h) {
            uint32_t *cell = my + 64u * (g / 4u + h);
            const uint32_t d4 = *cell;
            uint32_t x[4];
            const uint32_t j = g + 4u * h - lo, m = hi - lo;  // position k of the four: j + k < m
            ansai_pop_two<kWide, kTabLds, kMasked>(L, ansai_next_bits(L, ring), (d4 & 255u) << M, ((d4 >> 8) & 255u) << M,
                                                   x[0], x[1], theta, nb, j < m, j + 1u < m);
            ansai_pop_two<kWide, kTabLds, kMasked>(L, ansai_next_bits(L, ring), ((d4 >> 16) & 255u) << M, (d4 >> 24) << M,
                                                   x[2], x[3], theta, nb, j + 2u < m, j + 3u < m);
            *cell = x[0] | (x[1] << 8) | (x[2] << 16) | (x[3] << 24);
        }
    };
    if (n == kPart) {
        DecAhead a = ansai_ask(L, cw);
        group(0u);
        DecAhead b = ansai_ask(L, cw);
        group(8u);
        ansai_put_ahead(ring, a);
        a = ansai_ask(L, cw);
        group(16u);
        ansai_put_ahead(ring, b);
        b = ansai_ask(L, cw);
        group(24u);
        ansai_put_ahead(ring, a);
        ansai_put_ahead(ring, b);
        return;
    }
    uint32_t g = 0;
#pragma unroll 1
    for (; g + kGroupSyms <= n; g += kGroupSyms) {
        const DecAhead a = ansai_ask(L, cw);
        group(g);
        ansai_put_ahead(ring, a);
    }
    // the row's last symbols, fewer than a group
#pragma unroll 1
    for (; g < n; ++g) {
        uint8_t *cell = reinterpret_cast<uint8_t *>(my + 64u * (g / 4u)) + (g & 3u);
        *cell = (uint8_t)ansai_pop_one<kWide, kTabLds>(L, ring, (uint32_t)*cell << M, theta, nb);
    }
}

constexpr int kAnsaiDecMaxWaves = 12;
// Three wavefronts a compute unit with the tables in LDS are still faster than many with the tables in global memory
// (200,000 pieces of 500 symbols under 91 laws at 9 bits 486 against 813 us, under 23 at 11 bits 482
// against 815; 2000 pieces under 91 laws 96 against 134); tables for which only two would fit were not
// timed in LDS and stay in global memory.
constexpr int kAnsaiDecLeastWaves = 3;

template <bool kWide, bool kTabLds, bool kLines>
__global__ __launch_bounds__(64 * kAnsaiDecMaxWaves) void k_ansai_decode(
    AShape sh, const uint8_t *__restrict__ coded, const uint8_t *__restrict__ dist, const uint8_t *__restrict__ theta_g,
    const void *__restrict__ nb_g, uint8_t *__restrict__ out, uint32_t maxw, const Status *__restrict__ status,
    Report *__restrict__ report)
{
    extern __shared__ uint32_t lds[];
    if (status->code != ST_OK) {
        if (blockIdx.x == 0u && threadIdx.x == 0u) raise_code(report, status->code);
        return;
    }
    const uint8_t *theta = theta_g;
    const void *nb = nb_g;
    uint32_t *stage_base = lds;
    if (kTabLds) {  // the chain's table first, so that its LDS address is the index times its size
        const uint32_t entries = sh.D << sh.M;
        const uint32_t th_dw = (entries + 3u) >> 2, nb_dw = kWide ? entries : (entries + 1u) >> 1;
        const uint32_t *tg = reinterpret_cast<const uint32_t *>(theta_g);
        const uint32_t *ng = reinterpret_cast<const uint32_t *>(nb_g);
        for (uint32_t i = threadIdx.x; i < nb_dw; i += blockDim.x) {  // (entries turned: see DecEntry)
            const uint32_t e = ng[i];
            lds[i] = kWide ? __builtin_amdgcn_alignbit(e, e, 4)
                           : ((e >> 4) & 0x0FFF0FFFu) | ((e << 12) & 0xF000F000u);
        }
        for (uint32_t i = threadIdx.x; i < th_dw; i += blockDim.x) lds[nb_dw + i] = tg[i];
        nb = lds;
        theta = reinterpret_cast<const uint8_t *>(lds + nb_dw);
        stage_base = lds + nb_dw + th_dw;
        __syncthreads();
    }
    const uint32_t waves = blockDim.x >> 6;
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t gw = blockIdx.x * waves + wave;
    const uint32_t p0 = gw * 64u;
    if (p0 >= sh.pieces) return;
    const uint32_t np = min(64u, sh.pieces - p0);
    uint32_t *rows = stage_base + wave * kDecWaveDwords;
    uint32_t *my = rows + lane;
    uint32_t *ring = rows + 64u * (kPart / 4u) + lane;
    const uint32_t total = sh.pieces * sh.count;
    const uint32_t top = 1u << sh.M, M = sh.M;
    const uint32_t *cw = reinterpret_cast<const uint32_t *>(coded);
    const uint32_t off_dw = kHeaderBytes / 4u, pay_dw = off_dw + sh.pieces + 1u;
    const uint32_t payload_bytes = (uint32_t)status->payload_bytes;
    const ByteLimit lim_d = byte_limit(sh.D);

    bool mine = lane < np;
    uint32_t corrupt = 0u, bad = 0u;
    DecLane L;
    L.s = 0u;
    L.first = pay_dw;
    L.pos = 32u * L.first;
    L.lp = L.first;
    if (mine) {
        const uint32_t begin = cw[off_dw + p0 + lane], end = cw[off_dw + p0 + lane + 1u];
        bool ok = end >= begin && end - begin >= 8u && end <= payload_bytes && ((begin | end) & 3u) == 0u;
        if (ok) {
            const uint32_t rec = pay_dw + (begin >> 2);
            const uint32_t state = cw[rec], bits = cw[rec + 1u];
            const uint32_t nw = (end - begin - 8u) >> 2;
            // no piece of `count` symbols holds more than maxw words
            ok = nw <= maxw && state >= top && state < 2u * top && bits <= 32u * nw && bits + 31u >= 32u * nw;
            if (ok) {
                L.s = state - top;
                L.first = rec + 2u;
                L.pos = 32u * L.first + bits;
                L.lp = L.first;
                if (nw > 0u) {  // the 16 words that end with the aligned quad holding the last one
                    L.lp = ((L.first + nw - 1u) & ~3u) - 12u;  // (below the first piece's words lie header and offsets)
#pragma unroll
                    for (uint32_t i = 0; i < 4u; ++i)
                        ansai_ring_put(ring, (L.lp + 4u * i) & (kRingWords - 1u), ansai_quad_load(cw, L.lp + 4u * i));
                }
            }
        }
        if (!ok) {
            corrupt = 1u;
            mine = false;
        }
    }

    uint4 dv[8];
    rows_load<kLines>(dist, total, p0, np, sh.count, 0u, dv);
    const uint32_t skew = row_skew<kLines>((p0 + lane) * sh.count), row_end = skew + sh.count;  // this thread's symbols
    const uint32_t end = sh.count + (kLines ? 127u : 0u);  // positions that any row may have
    for (uint32_t pos0 = 0; pos0 < end; pos0 += 4u * kPart) {
        if (kLines) asm volatile("" : "+s"(sh.count));  // the rows' places are formed again, not kept in registers
        bad |= lines_check(dv, lim_d);
#pragma unroll 1
        for (uint32_t half = 0; half < 2u; ++half) {
            // two times 32 symbols, which leave together: memory takes writes 64 bytes at a time
            u32x4 ov[2][2] = {};
#pragma unroll
            for (uint32_t h = 0; h < 2u; ++h) {
                const uint32_t pos = pos0 + (2u * half + h) * kPart;
                if (pos >= end) break;
                wave_lds_sync();
                dec_put(rows, dv, 2u * half + h);
                wave_lds_sync();
                if (h == 1u && half == 1u && pos0 + 4u * kPart < end)
                    rows_load<kLines>(dist, total, p0, np, sh.count, pos0 + 4u * kPart, dv);
                if (!kLines) {
                    dec_part<kWide, kTabLds>(L, my, ring, cw, M, min(kPart, sh.count - pos), theta, nb);
                } else {
                    const uint32_t lo = max(skew, pos) - pos, hi = min(max(row_end, pos) - pos, kPart);
                    if (__all(lo == 0u && hi == kPart))
                        dec_part<kWide, kTabLds>(L, my, ring, cw, M, kPart, theta, nb);
                    else
                        dec_part<kWide, kTabLds, true>(L, my, ring, cw, M, kPart, theta, nb, min(lo, hi), hi);
                }
                wave_lds_sync();
                dec_get(rows, ov[h]);
            }
            const uint32_t pos = pos0 + 2u * half * kPart;
            if (pos < end) dec_store<kLines>(out, ov[0], p0, np, sh.count, pos);
            if (pos + kPart < end) dec_store<kLines>(out, ov[1], p0, np, sh.count, pos + kPart);
        }
    }
    if (mine && (L.s != 0u || L.pos != 32u * L.first)) corrupt = 1u;
    // many threads may report: the highest code (a damaged container) is the call's
    if (corrupt)
        raise_code(report, ST_CORRUPT);
    else if (bad)
        raise_code(report, ST_ARG);
}

// ---------------------------------------------------------------------------------------------
// Re-centring (Sec. 3.3): code (r - mu + 128) mod 256 so that the distribution index only has to
// tell the scale.  Four bytes per 32-bit lane operation: byte-wise subtraction / addition without
// carries between bytes, and + 128 mod 256 is a flip of every byte's top bit.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t bytes_sub(uint32_t a, uint32_t b)
{
    return ((a | 0x80808080u) - (b & 0x7F7F7F7Fu)) ^ ((a ^ ~b) & 0x80808080u);
}

__device__ __forceinline__ uint32_t bytes_add(uint32_t a, uint32_t b)
{
    return ((a & 0x7F7F7F7Fu) + (b & 0x7F7F7F7Fu)) ^ ((a ^ b) & 0x80808080u);
}

template <bool kInverse>
__global__ __launch_bounds__(256) void k_ansai_center(const uint8_t *in, const uint8_t *__restrict__ mu,
                                                      unsigned long long n, uint8_t *out)  // out may be in
{
    const unsigned long long vecs = n / 16ull, stride = (unsigned long long)gridDim.x * blockDim.x;
    for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < vecs; i += stride) {
        const uint4 a = reinterpret_cast<const uint4 *>(in)[i], m = reinterpret_cast<const uint4 *>(mu)[i];
        uint4 r;
        if (kInverse) {
            r = make_uint4(bytes_add(a.x ^ 0x80808080u, m.x), bytes_add(a.y ^ 0x80808080u, m.y),
                           bytes_add(a.z ^ 0x80808080u, m.z), bytes_add(a.w ^ 0x80808080u, m.w));
        } else {
            r = make_uint4(bytes_sub(a.x, m.x) ^ 0x80808080u, bytes_sub(a.y, m.y) ^ 0x80808080u,
                           bytes_sub(a.z, m.z) ^ 0x80808080u, bytes_sub(a.w, m.w) ^ 0x80808080u);
        }
        reinterpret_cast<uint4 *>(out)[i] = r;
    }
    if (blockIdx.x == 0 && threadIdx.x < (n & 15ull)) {  // the last, partial vector
        const unsigned long long i = vecs * 16ull + threadIdx.x;
        out[i] = kInverse ? (uint8_t)(in[i] + mu[i] - 128u) : (uint8_t)(in[i] - mu[i] + 128u);
    }
}

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
static int make_ashape(const pilc_ansai_shape *in, AShape *sh)
{
    if (!in || in->pieces == 0 || in->count == 0) return PILC_E_ARG;
    if (in->prec_bits < 1 || in->prec_bits > 15 || in->num_dist < 1 || in->num_dist > 255 ||
        in->num_sym < 2 || in->num_sym > 256 || (1u << in->prec_bits) < in->num_sym)
        return PILC_E_ARG;
    // 32-bit byte offsets into the [pieces, count] arrays and 32-bit scratch word indices
    const uint64_t padded = ((uint64_t)in->pieces + 63) / 64 * 64;
    const uint64_t maxw = ((uint64_t)in->count * in->prec_bits + 31) / 32;
    if (padded * in->count + 4096 >= (1ull << 32) || padded * maxw + 4096 >= (1ull << 32))
        return PILC_E_TOO_LARGE;
    sh->pieces = in->pieces;
    sh->count = in->count;
    sh->M = in->prec_bits;
    sh->D = in->num_dist;
    sh->X = in->num_sym;
    return PILC_OK;
}

struct AWorkspace {
    size_t status_off, report_off, bits_off, state_off, sums_off, scratch_off, total;
    uint32_t scan_blocks, maxw, waves;
};

static AWorkspace ansai_layout(const AShape &sh)
{
    AWorkspace w;
    w.scan_blocks = (uint32_t)ceil_div64(sh.pieces, kScanTile);
    w.maxw = (uint32_t)(((uint64_t)sh.count * sh.M + 31) / 32);
    w.waves = (uint32_t)ceil_div64(sh.pieces, 64);
    size_t off = 0;
    static_assert(sizeof(Status) <= 64 && sizeof(Report) <= 128, "both in the first 256 bytes");
    w.status_off = off;
    w.report_off = off + 128;
    off = align256(off + 256);
    w.bits_off = off;
    off = align256(off + 4 * (size_t)sh.pieces);
    w.state_off = off;
    off = align256(off + 4 * (size_t)sh.pieces);
    w.sums_off = off;
    off = align256(off + 8 * (size_t)w.scan_blocks);
    w.scratch_off = off;
    off = align256(off + 4 * (size_t)w.waves * 64 * w.maxw);
    w.total = off;
    return w;
}

static int ansai_status_to_error(int st) { return st == ST_ARG ? PILC_E_ARG : status_to_error(st); }


// LDS one workgroup may use on gfx950: the whole 160 KB of a compute unit.
constexpr size_t kLdsBytes = 160 * 1024;

}  // namespace pilc

using namespace pilc;

extern "C" {

size_t pilc_ansai_table_bytes(uint32_t prec_bits, uint32_t num_dist, uint32_t num_sym)
{
    pilc_ansai_shape s = {1u, 1u, prec_bits, num_dist, num_sym};
    AShape sh;
    if (make_ashape(&s, &sh) != PILC_OK) return 0;
    return ansai_tab_layout(sh.M, sh.D, sh.X).total;
}

int pilc_ansai_build_tables(uint32_t prec_bits, uint32_t num_dist, uint32_t num_sym,
                            const uint32_t *mass_dev, void *tables_dev, size_t tables_bytes,
                            void *hip_stream)
{
    pilc_ansai_shape s = {1u, 1u, prec_bits, num_dist, num_sym};
    AShape sh;
    int rc = make_ashape(&s, &sh);
    if (rc != PILC_OK) return rc;
    if (!mass_dev || !tables_dev || ((uintptr_t)mass_dev & 3) || ((uintptr_t)tables_dev & 255))
        return PILC_E_ARG;
    const ATabLayout t = ansai_tab_layout(sh.M, sh.D, sh.X);
    if (tables_bytes < t.total) return PILC_E_WORKSPACE;
    hipStream_t stream = (hipStream_t)hip_stream;
    uint8_t *base = static_cast<uint8_t *>(tables_dev);
    ATabHeader *head = reinterpret_cast<ATabHeader *>(base);
    k_ansai_build_begin<<<1, 1, 0, stream>>>(head, sh.M, sh.D, sh.X);
    if (t.wide)
        k_ansai_build<true><<<sh.D, 256, 0, stream>>>(sh.M, sh.X, mass_dev, head,
                                                      reinterpret_cast<uint2 *>(base + t.enc_off),
                                                      base + t.theta_off, base + t.nb_off);
    else
        k_ansai_build<false><<<sh.D, 256, 0, stream>>>(sh.M, sh.X, mass_dev, head,
                                                       reinterpret_cast<uint2 *>(base + t.enc_off),
                                                       base + t.theta_off, base + t.nb_off);
    HIP_TRY(hipGetLastError());
    ATabHeader host;
    HIP_TRY(hipMemcpyAsync(&host, head, sizeof(host), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return host.ok == 1u ? PILC_OK : PILC_E_ARG;
}

int pilc_ansai_center(const uint8_t *in_dev, const uint8_t *mu_dev, uint64_t count, int inverse,
                      uint8_t *out_dev, void *hip_stream)
{
    if (!in_dev || !mu_dev || !out_dev || count == 0) return PILC_E_ARG;
    if (((uintptr_t)in_dev & 15) || ((uintptr_t)mu_dev & 15) || ((uintptr_t)out_dev & 15)) return PILC_E_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    const uint64_t vecs = count / 16;
    uint32_t blocks = (uint32_t)(vecs / 256 > 16384 ? 16384 : (vecs + 255) / 256);
    if (blocks == 0) blocks = 1;
    if (inverse)
        k_ansai_center<true><<<blocks, 256, 0, stream>>>(in_dev, mu_dev, count, out_dev);
    else
        k_ansai_center<false><<<blocks, 256, 0, stream>>>(in_dev, mu_dev, count, out_dev);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(stream));
    return PILC_OK;
}

int pilc_ansai_workspace_size(const pilc_ansai_shape *shape, size_t *workspace_bytes_host,
                              size_t *max_coded_bytes_host)
{
    AShape sh;
    int rc = make_ashape(shape, &sh);
    if (rc != PILC_OK) return rc;
    const AWorkspace ws = ansai_layout(sh);
    if (workspace_bytes_host) *workspace_bytes_host = ws.total;
    if (max_coded_bytes_host)
        *max_coded_bytes_host =
            kHeaderBytes + 4 * ((size_t)sh.pieces + 1) + (size_t)sh.pieces * (8 + 4 * (size_t)ws.maxw);
    return PILC_OK;
}

int pilc_ansai_encode(const pilc_ansai_shape *shape, const uint8_t *sym_dev, const uint8_t *dist_dev,
                      const void *tables_dev, void *workspace_dev, size_t workspace_bytes,
                      uint8_t *coded_dev, size_t coded_capacity, uint64_t *coded_bytes_host,
                      void *hip_stream)
{
    AShape sh;
    int rc = make_ashape(shape, &sh);
    if (rc != PILC_OK) return rc;
    if (!sym_dev || !dist_dev || !tables_dev || !workspace_dev || !coded_dev || !coded_bytes_host)
        return PILC_E_ARG;
    if (((uintptr_t)sym_dev & 15) || ((uintptr_t)dist_dev & 15) || ((uintptr_t)tables_dev & 255) ||
        ((uintptr_t)workspace_dev & 255) || ((uintptr_t)coded_dev & 15))
        return PILC_E_ARG;
    const AWorkspace ws = ansai_layout(sh);
    if (workspace_bytes < ws.total) return PILC_E_WORKSPACE;
    const size_t table_end = kHeaderBytes + 4 * ((size_t)sh.pieces + 1);
    if (coded_capacity < table_end) return PILC_E_CAPACITY;

    hipStream_t stream = (hipStream_t)hip_stream;
    uint8_t *base = static_cast<uint8_t *>(workspace_dev);
    Status *status = reinterpret_cast<Status *>(base + ws.status_off);
    uint32_t *piece_bits = reinterpret_cast<uint32_t *>(base + ws.bits_off);
    uint32_t *piece_state = reinterpret_cast<uint32_t *>(base + ws.state_off);
    unsigned long long *sums = reinterpret_cast<unsigned long long *>(base + ws.sums_off);
    uint32_t *scratch = reinterpret_cast<uint32_t *>(base + ws.scratch_off);
    uint32_t *offsets = reinterpret_cast<uint32_t *>(coded_dev + kHeaderBytes);
    uint32_t *payload = reinterpret_cast<uint32_t *>(coded_dev + table_end);
    const ATabLayout t = ansai_tab_layout(sh.M, sh.D, sh.X);
    const uint8_t *tb = static_cast<const uint8_t *>(tables_dev);
    const uint2 *enc_tab = reinterpret_cast<const uint2 *>(tb + t.enc_off);

    CallReport report(reinterpret_cast<Report *>(base + ws.report_off), stream, true);
    Timer timer(stream);
    k_ansai_begin<<<1, 1, 0, stream>>>(sh, reinterpret_cast<const ATabHeader *>(tb), status);
    const size_t tab_lds = 8 * ((size_t)sh.D * 256 + 2);
    const bool tab_in_lds = tab_lds <= 24576 + 16;
    int dev = 0, cus = 0;  // (a batch of few wavefronts is spread over all compute units)
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    const uint32_t waves = (uint32_t)std::min<uint64_t>(kAnsaiEncWaves, ceil_div64(ws.waves, (uint64_t)cus));
    const uint32_t blocks = (uint32_t)ceil_div64(ws.waves, waves);
    auto kern = tab_in_lds ? k_ansai_encode<true> : k_ansai_encode<false>;
    if ((rc = allow_large_lds(reinterpret_cast<const void *>(kern))) != PILC_OK) return rc;
    kern<<<blocks, 64 * waves, (size_t)waves * kEncWaveDwords * 4 + (tab_in_lds ? tab_lds : 0), stream>>>(
        sh, sym_dev, dist_dev, enc_tab, scratch, ws.maxw, piece_bits, piece_state, &status->code);
    timer.mark("k_ansai_encode");
    const ItemBytes piece_bytes = {8u, 4u, 31u, 5u};  // state, bit count, 32-bit words
    const HeaderWords head = {{kAnsaiMagic, 1u, sh.pieces, sh.count, sh.M, sh.D, sh.X, 0u, 0u, 0u, 0u, 0u}};
    (void)launch_scan(head, sh.pieces, ws.scan_blocks, piece_bytes, piece_bits, sums, coded_dev, coded_capacity, status, report.dev(),
                      offsets, true, stream);
    timer.mark("scan");
    k_ansai_pack<<<(uint32_t)ceil_div64(ws.waves, kAnsaiPackWaves), 64 * kAnsaiPackWaves, 0, stream>>>(
        sh, scratch, ws.maxw, piece_bits, piece_state, offsets, payload, status);
    timer.mark("k_ansai_pack");
    HIP_TRY(hipGetLastError());
    Report seen;
    HIP_TRY(report.wait(&seen));
    timer.finish();
    if (raised_code(seen) != ST_OK) return ansai_status_to_error(raised_code(seen));
    *coded_bytes_host = table_end + seen.payload_bytes;
    return PILC_OK;
}

int pilc_set_ansai_decode_waves(int waves)
{
    if (waves < 0 || waves > kAnsaiDecMaxWaves) return PILC_E_ARG;
    g_ansai_decode_waves.store(waves, std::memory_order_relaxed);
    return PILC_OK;
}

int pilc_ansai_decode(const pilc_ansai_shape *shape, const uint8_t *coded_dev, size_t coded_bytes,
                      const uint8_t *dist_dev, const void *tables_dev, void *workspace_dev,
                      size_t workspace_bytes, uint8_t *sym_out_dev, void *hip_stream)
{
    AShape sh;
    int rc = make_ashape(shape, &sh);
    if (rc != PILC_OK) return rc;
    if (!coded_dev || !dist_dev || !tables_dev || !workspace_dev || !sym_out_dev) return PILC_E_ARG;
    if (((uintptr_t)sym_out_dev & 15) || ((uintptr_t)dist_dev & 15) || ((uintptr_t)tables_dev & 255) ||
        ((uintptr_t)workspace_dev & 255) || ((uintptr_t)coded_dev & 15))
        return PILC_E_ARG;
    const AWorkspace ws = ansai_layout(sh);
    if (workspace_bytes < ws.total) return PILC_E_WORKSPACE;
    const size_t table_end = kHeaderBytes + 4 * ((size_t)sh.pieces + 1);
    if (coded_bytes < table_end) return PILC_E_FORMAT;
    const size_t lds_max = kLdsBytes;

    hipStream_t stream = (hipStream_t)hip_stream;
    Status *status = reinterpret_cast<Status *>(static_cast<uint8_t *>(workspace_dev) + ws.status_off);
    const ATabLayout t = ansai_tab_layout(sh.M, sh.D, sh.X);
    const uint8_t *tb = static_cast<const uint8_t *>(tables_dev);

    // Workgroup shape: the decode tables in LDS when they leave room for at least kAnsaiDecLeastWaves
    // wavefronts' staging rows; as many wavefronts (<= kAnsaiDecMaxWaves) as then fit.
    const size_t entries = (size_t)sh.D << sh.M;
    const size_t tab_lds = ((entries + 3) / 4 + (t.wide ? entries : (entries + 1) / 2)) * 4;
    const size_t row_lds = (size_t)kDecWaveDwords * 4;
    bool tab_in_lds = tab_lds + kAnsaiDecLeastWaves * row_lds <= lds_max;
    uint32_t waves = 4;
    if (tab_in_lds) {
        // small tables: several workgroups per compute unit; large ones: one big workgroup
        size_t fit = (lds_max - tab_lds) / row_lds;
        waves = tab_lds <= 16384 ? 4u : (uint32_t)(fit > kAnsaiDecMaxWaves ? kAnsaiDecMaxWaves : fit);
        // a batch too small to fill every compute unit that densely is spread over all of them
        // (a piece is a serial chain: its pace falls with the wavefronts that share its SIMD)
        int dev = 0, cus = 0;
        if (waves > 4u && hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0) {
            const uint32_t each = (uint32_t)ceil_div64(ws.waves, (uint64_t)cus);
            if (each <= waves)
                waves = std::max(4u, each);
            else if (waves >= 8u && sh.count >= 256u) {
                // Several rounds: workgroups of a size that fills them all, not full ones and a remainder, because a
                // compute unit takes its next workgroup when the last wavefront of this one is done.  (Eight
                // laws at 12 bits, ten wavefronts at most: 175,000 pieces of 4000 symbols, 2735
                // wavefronts, 1368 us with ten, 1133 with six; 10^6 of 1000 1572 with ten, 1512 with nine.  With small
                // workgroups to begin with, and with short rows, the tables that every workgroup loads cost
                // more: 100,000 of 500 under ten laws 180 us with six, 194 with four; 10^6 of 128 259 with ten, 268
                // with nine.)
                const uint32_t rounds = (each + waves - 1u) / waves;
                waves = (each + rounds - 1u) / rounds;
            }
        }
    }
    const uint32_t asked = (uint32_t)g_ansai_decode_waves.load(std::memory_order_relaxed);
    if (asked != 0u) {  // pilc_set_ansai_decode_waves: that many, if they fit
        const size_t fit = tab_in_lds ? (lds_max - tab_lds) / row_lds : (size_t)kAnsaiDecMaxWaves;
        waves = asked < fit ? asked : (uint32_t)fit;
    }
    Timer timer(stream);
    CallReport report(reinterpret_cast<Report *>(static_cast<uint8_t *>(workspace_dev) + ws.report_off), stream, true);
    k_ansai_check_header<<<1, 1, 0, stream>>>(sh, reinterpret_cast<const ATabHeader *>(tb), coded_dev,
                                              (unsigned long long)coded_bytes, status);
    timer.mark("k_ansai_check_header");
    // A build of this kernel that needed private memory (register spills) once decoded wrongly in
    // the wavefronts beyond the fourth of a workgroup, and the cause was never found.  The kernel as
    // written compiles without private memory; a build that does not is refused rather than run.
#define PILC_ANSAI_DECODE(WIDE, LDS, LINES)                                                           \
    do {                                                                                              \
        auto kern = k_ansai_decode<WIDE, LDS, LINES>;                                                 \
        hipFuncAttributes fa;                                                                         \
        HIP_TRY(hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(kern)));                     \
        if (fa.localSizeBytes != 0) {                                                                 \
            snprintf(t_hip_error, sizeof(t_hip_error),                                                \
                     "k_ansai_decode was built with %zu bytes of private memory per thread; this "   \
                     "library only runs a build of it that has none", (size_t)fa.localSizeBytes);     \
            return PILC_E_HIP;                                                                        \
        }                                                                                             \
        const size_t lds_bytes = (LDS ? tab_lds : 0) + waves * row_lds;                               \
        const uint32_t blocks = (uint32_t)ceil_div64(ws.waves, waves);                                \
        if ((rc = allow_large_lds(reinterpret_cast<const void *>(kern))) != PILC_OK) return rc;       \
        kern<<<blocks, 64 * waves, lds_bytes, stream>>>(sh, coded_dev, dist_dev, tb + t.theta_off,    \
                                                        tb + t.nb_off, sym_out_dev, ws.maxw, status,  \
                                                        report.dev());                                \
    } while (0)
    // Rows cut at the array's lines or at their own start.  A row cut at its own start has no step without a symbol, but
    // its lines are asked for twice, 128 symbols apart, and written in pieces; that costs nothing while the
    // batch fits the 256 MB of cache in front of memory, and little in rows of whole half lines.  Own start
    // against lines, us: 100,000 pieces of 1001 symbols 197 and 201, 80,000 of 2001 357 and 340, 160,000 of 4001
    // 1132 and 848, 556,881 of 1257 1127 and 907, 10^6 of 700 1124 and 985, of 501 787 and 767, of 333 553
    // and 574, 700,000 of 960 790 and 811 (four laws at 10 bits).
    const bool lines = sh.count % 64u != 0u && sh.count >= 640u && (uint64_t)sh.pieces * sh.count >= (1ull << 27);
#define PILC_ANSAI_DECODE_CUT(WIDE, LDS)          \
    do {                                          \
        if (lines)                                \
            PILC_ANSAI_DECODE(WIDE, LDS, true);   \
        else                                      \
            PILC_ANSAI_DECODE(WIDE, LDS, false);  \
    } while (0)
    if (t.wide) {
        if (tab_in_lds)
            PILC_ANSAI_DECODE_CUT(true, true);
        else
            PILC_ANSAI_DECODE_CUT(true, false);
    } else {
        if (tab_in_lds)
            PILC_ANSAI_DECODE_CUT(false, true);
        else
            PILC_ANSAI_DECODE_CUT(false, false);
    }
#undef PILC_ANSAI_DECODE_CUT
#undef PILC_ANSAI_DECODE
    timer.mark("k_ansai_decode");
    HIP_TRY(hipGetLastError());
    Report seen;
    HIP_TRY(report.wait(&seen));
    timer.finish();
    return ansai_status_to_error(raised_code(seen));
}

}  // extern "C"
