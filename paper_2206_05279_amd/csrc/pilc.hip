// libpilc: kernels and C ABI of the PILC entropy-coding stage for gfx950 (arXiv 2206.05279).
//
// Path per call
//   encode: lane kernel (mean shift -> (cum,freq) -> rANS, words to per-lane scratch slots)
//           -> prefix sums of lane byte counts by tiles (header)
//           -> pack (offset table, lane streams copied to their offsets)
//   decode: lane kernel (header check, search of the symbol, state update, refill)
// Lane kernels: pilc_lane_kernels.hpp (thread per lane), pilc_block_encode.hpp and
// pilc_row_decode.hpp (few long lanes).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <optional>
#include <utility>

#include "../../include/pilc.h"
#include "pilc_device.hpp"

namespace pilc {

__device__ uint2 g_sig_cell[kSigEntries];
__device__ float2 g_guide[kGuideEntries];
__device__ uint32_t g_exp_hi[kExpHiEntries];
__device__ uint32_t g_exp_lo[kExpLoEntries];

constexpr uint32_t kHeaderBytes = 64;

// status word kinds (device side), mapped to PILC_E_* on the host
constexpr uint32_t kMagicPilc = 0x434C4950u;  // "PILC"
constexpr uint32_t kMagicMix = 0x58494D50u;   // "PMIX"
enum : int { ST_OK = 0, ST_TOO_LARGE = 4, ST_FORMAT = 5, ST_CORRUPT = 6, ST_CAPACITY = 3, ST_PARAMS = 7, ST_TIMEOUT = 8 };

struct Status {
    int code;
    uint32_t ticket;  // workgroups number themselves from it, in the order in which they begin or end
    unsigned long long payload_bytes;
};
__device__ __forceinline__ void init_status(Status *status)
{
    status->code = ST_OK;
    status->ticket = 0;
    status->payload_bytes = 0;
}

// What a call hands back to the host besides its output: which of the codes above were raised (the highest is the
// call's), and the payload size of an encoder.  It lies in pinned host memory, so that neither a copy nor a
// kernel that clears it is in the call's way; where there is none, in the workspace.
struct Report {
    uint32_t raised[16];
    unsigned long long payload_bytes;
};
__device__ __forceinline__ void raise_code(Report *report, int code)
{
    __hip_atomic_store(&report->raised[code], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// --------------------------------------------------------------------------------------------
// Per-pixel helper: effective means of the three channels (Sec. 3.1 eqs. (3)-(4), innovation
// form).  e_G uses the unshifted mu_G so the three means are independent of each other.
// --------------------------------------------------------------------------------------------
__device__ __forceinline__ void mean_shift(const int x[3], const int m[3], int a_gr, int a_br,
                                           int a_bg, int out[3])
{
    int e_r = x[0] * 256 - m[0];
    int e_g = x[1] * 256 - m[1];
    out[0] = m[0];
    out[1] = m[1] + rsh14_mul(a_gr, e_r);
    out[2] = m[2] + rsh14_mul(a_br, e_r) + rsh14_mul(a_bg, e_g);
}

// --------------------------------------------------------------------------------------------
// pilc_symbol_tables: one thread per pixel.
// --------------------------------------------------------------------------------------------
__global__ void k_symbol_tables(Geo g, const uint8_t *__restrict__ img,
                                const uint16_t *__restrict__ mu, const int16_t *__restrict__ ls,
                                const int16_t *__restrict__ coef, uint32_t *__restrict__ cum_out,
                                uint32_t *__restrict__ freq_out)
{
    __shared__ LdsTables tab;
    load_tables(tab);
    uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= g.total_px) return;
    size_t s = (size_t)p * 3;
    uint32_t im = g.by_hw.div(p);
    int x[3] = {img[s], img[s + 1], img[s + 2]};
    int m[3] = {mu[s], mu[s + 1], mu[s + 2]};
    int me[3];
    mean_shift(x, m, coef[3 * im], coef[3 * im + 1], coef[3 * im + 2], me);
    for (int c = 0; c < 3; ++c) {
        uint32_t inv_s = inv_scale(ls[s + c], tab);
        uint32_t lo = cum_at(x[c], me[c], inv_s, g.prec_bits, tab);
        uint32_t hi = cum_at(x[c] + 1, me[c], inv_s, g.prec_bits, tab);
        cum_out[s + c] = lo;
        freq_out[s + c] = hi - lo;
    }
}

// --------------------------------------------------------------------------------------------
// Prefix scan of per-item byte counts into a container's offset table.
// --------------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ __forceinline__ unsigned long long block_exclusive_scan(unsigned long long v,
                                                                   unsigned long long *total)
{
    __shared__ unsigned long long wave_sum[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long inc = v;
    for (int d = 1; d < 64; d <<= 1) {
        unsigned long long o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    unsigned long long base = 0, all = 0;
    for (int i = 0; i < kScanThreads / 64; ++i) {
        if (i < wave) base += wave_sum[i];
        all += wave_sum[i];
    }
    __syncthreads();
    *total = all;
    return base + inc - v;
}

// Bytes an item (a lane, a piece) takes in the payload, from the count its coder left behind:
// base + unit * ((count + add) >> shift).
struct ItemBytes {
    uint32_t base, unit, add, shift;
    __device__ __forceinline__ unsigned long long operator()(uint32_t count) const
    {
        return (unsigned long long)base + (unsigned long long)unit * ((count + add) >> shift);
    }
};

constexpr ItemBytes kLaneBytes = {4u, 2u, 0u, 0u};  // of a lane: a 32-bit state and 16-bit words

// The first twelve 32-bit words of a container header (the payload size follows them).
struct HeaderWords {
    uint32_t w[12];
};

// One workgroup: the sums of the tiles into what lies before each tile; the header; the outcome (`report` may be null).
__device__ __forceinline__ void spine_scan(const HeaderWords &head, uint32_t items, uint32_t nblocks,
                                           unsigned long long *block_sums, uint8_t *__restrict__ coded,
                                           unsigned long long coded_capacity, Status *status, Report *report)
{
    unsigned long long carry = 0;
    for (uint32_t b0 = 0; b0 < nblocks; b0 += kScanThreads) {
        const uint32_t i = b0 + threadIdx.x;
        const unsigned long long sum =
            i < nblocks ? __hip_atomic_load(&block_sums[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
        unsigned long long total;
        const unsigned long long ex = block_exclusive_scan(sum, &total);
        if (i < nblocks) block_sums[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) {
        status->payload_bytes = carry;
        const unsigned long long need = kHeaderBytes + 4ull * ((unsigned long long)items + 1ull) + carry;
        if (status->code == ST_OK) {  // an earlier error stays
            if (carry >= (1ull << 32))
                status->code = ST_TOO_LARGE;
            else if (need > coded_capacity)
                status->code = ST_CAPACITY;
        }
        if (report != nullptr) {
            if (status->code != ST_OK) raise_code(report, status->code);
            __hip_atomic_store(&report->payload_bytes, carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        uint32_t *h = reinterpret_cast<uint32_t *>(coded);
        for (int i = 0; i < 12; ++i) h[i] = head.w[i];
        h[12] = (uint32_t)carry;
        h[13] = (uint32_t)(carry >> 32);
        h[14] = 0u;
        h[15] = 0u;
    }
}

__global__ void k_scan_partials(uint32_t items, ItemBytes bytes, const uint32_t *__restrict__ counts,
                                unsigned long long *__restrict__ block_sums)
{
    uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    unsigned long long v = 0;
    for (int i = 0; i < kScanItems; ++i)
        if (base + i < items) v += bytes(counts[base + i]);
    unsigned long long total;
    block_exclusive_scan(v, &total);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// Single workgroup: exclusive scan of the block sums in place; writes the header.
__global__ void k_scan_spine(HeaderWords head, uint32_t items, uint32_t nblocks,
                             unsigned long long *__restrict__ block_sums,
                             uint8_t *__restrict__ coded, unsigned long long coded_capacity,
                             Status *__restrict__ status, Report *__restrict__ report)
{
    spine_scan(head, items, nblocks, block_sums, coded, coded_capacity, status, report);
}

// For a batch of few tiles (but too large for scans_alone) the two in one: the workgroup that is done last goes on with the
// sums of all.  `status->ticket` is zero before the launch.  The packers of such a batch form the offset table themselves
// (lane_offsets), so that one launch stands where there were three.  Up to kScanFewTiles: 100,000 lanes of 63 pixels
// 153 -> 139 us; with 1600 tiles, where every workgroup's fence and every packer's sums of its tile
// cost more than two launches, 50,000 images of 32 x 32 in lanes of 32 pixels 508 -> 573.
constexpr uint32_t kScanFewTiles = 128;
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(HeaderWords head, uint32_t items, ItemBytes bytes,
                                                            const uint32_t *__restrict__ counts,
                                                            unsigned long long *block_sums, uint8_t *__restrict__ coded,
                                                            unsigned long long coded_capacity, Status *status, Report *report)
{
    __shared__ uint32_t s_last;
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems, nblocks = gridDim.x;
    unsigned long long v = 0;
    for (int i = 0; i < kScanItems; ++i)
        if (base + i < items) v += bytes(counts[base + i]);
    unsigned long long total;
    block_exclusive_scan(v, &total);
    if (threadIdx.x == 0) {
        __hip_atomic_store(&block_sums[blockIdx.x], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
        s_last = atomicAdd(&status->ticket, 1u) + 1u == nblocks ? 1u : 0u;
        __threadfence();
    }
    __syncthreads();
    if (s_last == 0u) return;
    spine_scan(head, items, nblocks, block_sums, coded, coded_capacity, status, report);
}

// A batch of few lanes has no scan at all: every workgroup of the packer sums the counts of all lanes, and of those before its own,
// and the first one writes the header and the outcome.  What that costs is a read of all counts from the L2 by every
// workgroup; what it saves is a launch.  With the launch and without, whole encode calls, us: 2048 lanes of 32 pixels 35.8 and 31.1,
// 4000 of 512 69.5 and 67.2, 8000 of 32 38.4 and 37.8, 16,000 of 32 42.0 and 45.6.  Long lanes have a workgroup for every few
// of them, so the line is also at so many workgroups times lanes.  What the calls take longer without the launch, us, mean of
// some hundred batches: at 10 million -0.7, 12 -1 (of 200 to 300), 20 -1.2, 25 0.3 to 2.4 (of 320 to 490), 60 7.5 (of 520).
constexpr uint32_t kScanAloneLanes = 8192;
constexpr uint64_t kScanAloneReads = 1u << 24;
static bool scans_alone(uint32_t lanes, uint32_t pack_blocks)
{
    return lanes <= kScanAloneLanes && (uint64_t)lanes * pack_blocks <= kScanAloneReads;
}
struct PackAlone {
    uint32_t alone;  // else the rest is not looked at
    HeaderWords head;
    uint8_t *coded;
    unsigned long long capacity;
    Report *report;
};

// Whether the kernels before have raised an error, which without a scan nobody else reports.
__device__ __forceinline__ bool nothing_to_pack(const Status *status, const PackAlone &pk)
{
    if (status->code == ST_OK) return false;
    if (pk.alone != 0u && blockIdx.x == 0u && threadIdx.x == 0u) raise_code(pk.report, status->code);
    return true;
}

// The sums of `v` and `w` over the workgroup.
__device__ __forceinline__ void block_sum_two(unsigned long long &v, unsigned long long &w)
{
    __shared__ unsigned long long wave_sum[2][kScanThreads / 64];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        v += __shfl_xor(v, d, 64);
        w += __shfl_xor(w, d, 64);
    }
    if ((threadIdx.x & 63u) == 0u) {
        wave_sum[0][threadIdx.x >> 6] = v;
        wave_sum[1][threadIdx.x >> 6] = w;
    }
    __syncthreads();
    v = w = 0ull;
#pragma unroll
    for (int i = 0; i < kScanThreads / 64; ++i) {
        v += wave_sum[0][i];
        w += wave_sum[1][i];
    }
}

// What lies before lane l0 in the payload of a batch without a scan; false if the payload does not fit (then nothing is packed).
__device__ __forceinline__ bool sum_alone(const PackAlone &pk, uint32_t l0, uint32_t lanes, const ItemBytes &bytes,
                                          const uint32_t *__restrict__ counts, unsigned long long *before_out)
{
    unsigned long long before = 0ull, all = 0ull;
    for (uint32_t i0 = threadIdx.x; i0 < lanes; i0 += 8u * kScanThreads) {
        uint32_t c[8];
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) c[k] = counts[min(i0 + k * kScanThreads, lanes - 1u)];
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) {
            const uint32_t i = i0 + k * kScanThreads;
            const unsigned long long b = i < lanes ? bytes(c[k]) : 0ull;
            all += b;
            before += i < l0 ? b : 0ull;
        }
    }
    block_sum_two(before, all);
    *before_out = before;
    const int code = all >= (1ull << 32) ? ST_TOO_LARGE
                     : kHeaderBytes + 4ull * ((unsigned long long)lanes + 1ull) + all > pk.capacity ? ST_CAPACITY : ST_OK;
    if (blockIdx.x == 0u && threadIdx.x < 16u) {
        uint32_t *h = reinterpret_cast<uint32_t *>(pk.coded);
        const uint32_t w = threadIdx.x;
        h[w] = w < 12u ? pk.head.w[w] : w == 12u ? (uint32_t)all : w == 13u ? (uint32_t)(all >> 32) : 0u;
        if (w == 0u) {
            if (code != ST_OK) raise_code(pk.report, code);
            __hip_atomic_store(&pk.report->payload_bytes, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    return code == ST_OK;
}

// Where the bytes of lanes l0 .. l0 + n - 1 (n <= kScanThreads) begin in the payload, thread i that of lane l0 + i, from
// the sums before the tiles and the counts of l0's tile; the same into the offset table.
// `formed`: the table is there already.  `fits`: false if the batch turns out here not to fit (PackAlone).
__device__ __forceinline__ unsigned long long lane_offsets(const PackAlone &pk, bool formed, uint32_t l0, uint32_t n, uint32_t lanes,
                                                           const ItemBytes &bytes, const uint32_t *__restrict__ counts,
                                                           const unsigned long long *__restrict__ block_sums,
                                                           uint32_t *__restrict__ offsets, unsigned long long *end, bool *fits)
{
    *fits = true;
    if (formed) {  // (the same for every thread)
        __syncthreads();
        *end = threadIdx.x < n ? offsets[l0 + threadIdx.x + 1u] : 0u;
        return threadIdx.x < n ? offsets[l0 + threadIdx.x] : 0u;
    }
    unsigned long long before = 0, total;
    const unsigned long long mine = threadIdx.x < n ? bytes(counts[l0 + threadIdx.x]) : 0ull;
    if (pk.alone != 0u) {
        *fits = sum_alone(pk, l0, lanes, bytes, counts, &before);
        if (!*fits) return 0ull;
    } else {
        const uint32_t tile = l0 / kScanTile;
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kScanItems; ++k) {
            const uint32_t i = tile * kScanTile + k * kScanThreads + threadIdx.x;
            if (i < l0) before += bytes(counts[i]);
        }
        (void)block_exclusive_scan(before, &total);
        before = total + block_sums[tile];
    }
    const unsigned long long at = block_exclusive_scan(mine, &total) + before;
    if (threadIdx.x < n) {
        offsets[l0 + threadIdx.x] = (uint32_t)at;
        if (l0 + threadIdx.x + 1u == lanes) offsets[lanes] = (uint32_t)(at + mine);
    }
    *end = at + mine;
    return at;
}

__global__ void k_scan_apply(uint32_t items, ItemBytes bytes, const uint32_t *__restrict__ counts,
                             const unsigned long long *__restrict__ block_sums,
                             uint32_t *__restrict__ offsets)
{
    uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    unsigned long long item[kScanItems], v = 0;
    for (int i = 0; i < kScanItems; ++i) {
        item[i] = base + i < items ? bytes(counts[base + i]) : 0ull;
        v += item[i];
    }
    unsigned long long total;
    unsigned long long ex = block_exclusive_scan(v, &total) + block_sums[blockIdx.x];
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i < items) offsets[base + i] = (uint32_t)ex;
        ex += item[i];
        // the closing entry offsets[items] = payload size
        if (base + i + 1 == items) offsets[items] = (uint32_t)ex;
    }
}

// --------------------------------------------------------------------------------------------
// Pack: a workgroup copies the streams of a run of consecutive lanes (their bytes are contiguous
// in the payload).  Offsets, scratch positions and states of the run sit in LDS; each payload
// word finds its lane by bisection there.
// --------------------------------------------------------------------------------------------
constexpr int kPackMaxLanes = 256;
constexpr uint32_t kPackBlocks = 1024, kPackLeast = 512;
// Up to so many lanes a workgroup they are moved a wavefront a lane, eight words a thread (a word a thread otherwise; bound by the
// number of loads and stores: 214 MB in 75 us on 3125 lanes of 16,384 pixels, in 38 this way).  Those are lanes of a thousand symbols
// and more, and in batches below some 17,400 lanes, which are cut into 1024 runs, nearly all others, where few of a wavefront's threads
// have words to move, but it is no slower.  A word a thread and eight, this kernel, us: 500 lanes of 40 pixels 7.2 and 6.4; 2048 of 16
// 8.5 and 8.3, of 32 8.3 and 7.8, of 64 8.3 and 8.2; 8192 of 16 9.2 and 8.9, of 64 9.7 and 8.8; 16,384 of 16 9.8 and 9.9, of 32 9.7
// and 9.9, of 64 11.9 and 10.1, of 128 15.5 and 10.8; 4096 of 512 13.2 and 8.9.
constexpr uint32_t kPackByWave = 16;

__global__ __launch_bounds__(kScanThreads) void k_pack(Geo g, uint32_t lanes_per_block,
                                                       const uint16_t *__restrict__ scratch,
                                                       const uint32_t *__restrict__ lane_words,
                                                       const uint32_t *__restrict__ lane_state,
                                                       const unsigned long long *__restrict__ block_sums,
                                                       bool formed, uint32_t *__restrict__ offsets,
                                                       uint16_t *__restrict__ payload,
                                                       const Status *__restrict__ status, PackAlone pk)
{
    if (nothing_to_pack(status, pk)) return;
    __shared__ uint32_t s_off[kPackMaxLanes + 1];
    __shared__ uint32_t s_src[kPackMaxLanes];    // scratch index of the lane's first word
    __shared__ uint32_t s_state[kPackMaxLanes];
    const uint32_t l0 = blockIdx.x * lanes_per_block;
    const uint32_t n = min(lanes_per_block, g.lanes - l0);
    static_assert(kPackMaxLanes <= kScanThreads, "a thread per lane");
    unsigned long long lane_end;
    bool fits;
    const uint32_t begin = (uint32_t)lane_offsets(pk, formed, l0, n, g.lanes, kLaneBytes, lane_words, block_sums, offsets, &lane_end, &fits);
    if (!fits) return;  // (the same for every thread)
    const uint32_t i = threadIdx.x;
    if (i < n) {
        const LaneShape sh = lane_shape(g, l0 + i);
        s_off[i] = begin;
        if (i + 1 == n) s_off[n] = (uint32_t)lane_end;
        s_src[i] = block_slot_end(sh, l0 + i) - (((uint32_t)lane_end - begin - 4u) >> 1);
        s_state[i] = lane_state[l0 + i];
    }
    __syncthreads();
    const uint32_t w_begin = s_off[0] >> 1, w_end = s_off[n] >> 1;
    if (w_begin == w_end) return;
    if (lanes_per_block <= kPackByWave) {
        // eight words a thread at whatever address they fall on, a wavefront a lane, or the whole workgroup where it
        // has fewer than four; a lane's last eight are moved as such, whether or not some of them have been already
        const uint32_t team = n < 4u ? blockDim.x : 64u, member = threadIdx.x & (team - 1u);
        for (uint32_t l = n < 4u ? 0u : threadIdx.x >> 6; l < n; l += n < 4u ? 1u : blockDim.x >> 6) {
            const uint32_t words = ((s_off[l + 1] - s_off[l]) >> 1) - 2u;  // (after the state)
            const uint16_t *from = scratch + s_src[l];
            uint16_t *to = payload + (s_off[l] >> 1);
            if (member < 2u) to[member] = (uint16_t)(s_state[l] >> (16u * member));
            to += 2;
            if (words < 8u) {
                if (member < words) to[member] = from[member];
                continue;
            }
            for (uint32_t j = 8u * member; j < words; j += 16u * team) {
                const uint32_t at[2] = {min(j, words - 8u), min(j + 8u * team, words - 8u)};
                u32x4 v[2];
                __builtin_memcpy(&v[0], from + at[0], 16);
                __builtin_memcpy(&v[1], from + at[1], 16);
                __builtin_memcpy(to + at[0], &v[0], 16);
                __builtin_memcpy(to + at[1], &v[1], 16);
            }
        }
        return;
    }
    // four words per thread and turn, so that four loads are under way together (words past the
    // end read the last one again and are not written)
    for (uint32_t w0 = w_begin + threadIdx.x; w0 - threadIdx.x < w_end; w0 += 4u * blockDim.x) {
        uint16_t v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t byte = 2u * min(w0 + k * blockDim.x, w_end - 1u);
            uint32_t lo = 0, hi = n - 1;  // largest i with s_off[i] <= byte
            while (lo < hi) {
                const uint32_t mid = (lo + hi + 1) >> 1;
                if (s_off[mid] <= byte)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            const uint32_t local = byte - s_off[lo];
            // a lane's state is its first four bytes; for those the load goes to the word below the
            // lane's words (inside its slot: a lane has a pixel or more) and is not used
            const uint16_t word = scratch[local < 4u ? s_src[lo] - 1u : s_src[lo] + ((local - 4u) >> 1)];
            v[k] = local < 4u ? (uint16_t)(s_state[lo] >> (8u * local)) : word;
        }
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k)
            if (w0 + k * blockDim.x < w_end) payload[w0 + k * blockDim.x] = v[k];
    }
}

// The packer for the thread-per-lane encoder, whose scratch is [word number][thread] per 64
// lanes with room for lane_cap words each, the words of a lane in the reverse of the stream
// order.  A workgroup owns 64 lanes: it reads kPackTile word numbers at a time as whole 128-byte
// rows into an LDS tile and writes every lane's piece of the stream from there, 64 consecutive words
// per wavefront instruction.  kPackTile word numbers a turn: the more, the longer the runs a lane's
// words are written in (128 for lanes of up to 256 symbols, where more would mostly be read in
// vain, 256 for longer ones; on the stress workload 64 / 128 / 256 take 0.61 / 0.52 / 0.47 ms).
constexpr int kPackTileStride = 66;  // 16-bit elements: 33 dwords, odd, so a column read spreads over the banks

template <int kPackTile>
__global__ __launch_bounds__(kScanThreads) void k_pack_by_thread(uint32_t lanes, uint32_t lane_cap,
                                                                 const uint16_t *__restrict__ scratch,
                                                                 const uint32_t *__restrict__ lane_words,
                                                                 const uint32_t *__restrict__ lane_state,
                                                                 const unsigned long long *__restrict__ block_sums,
                                                                 bool formed, uint32_t *__restrict__ offsets,
                                                                 uint16_t *__restrict__ payload,
                                                                 const Status *__restrict__ status, PackAlone pk)
{
    if (nothing_to_pack(status, pk)) return;
    __shared__ uint32_t s_first[64];  // payload word index of the lane's state
    __shared__ uint32_t s_nw[64];     // words after the state
    __shared__ uint32_t s_max;
    __shared__ __align__(4) uint16_t tile[kPackTile * kPackTileStride];
    const uint32_t t = threadIdx.x;
    const uint32_t l0 = blockIdx.x * 64u;
    if (t == 0) s_max = 0u;
    unsigned long long lane_end;  // (ends with a barrier)
    bool fits;
    const uint32_t begin = (uint32_t)lane_offsets(pk, formed, l0, min(64u, lanes - l0), lanes, kLaneBytes, lane_words, block_sums,
                                                  offsets, &lane_end, &fits);
    if (!fits) return;  // (the same for every thread)
    if (t < 64u) {
        uint32_t nw = 0u, first = 0u;
        if (l0 + t < lanes) {
            const uint32_t st = lane_state[l0 + t];
            first = begin >> 1;
            nw = ((uint32_t)lane_end - begin - 4u) >> 1;
            payload[first] = (uint16_t)st;
            payload[first + 1u] = (uint16_t)(st >> 16);
            atomicMax(&s_max, nw);
        }
        s_first[t] = first;
        s_nw[t] = nw;
    }
    __syncthreads();
    const uint32_t max_nw = s_max;
    const uint16_t *rows = scratch + (size_t)l0 * lane_cap;
    for (uint32_t k0 = 0; k0 < max_nw; k0 += kPackTile) {
        // rows k0 .. k0 + 63 of the block, two lanes (one dword) per thread and 8 rows apart; all
        // eight are asked for before the first is stored (guarded one by one, every load would wait
        // for the one before); rows past the last one repeat it and are never read
        uint32_t v[kPackTile / 8];
#pragma unroll
        for (int j = 0; j < kPackTile / 8; ++j) {
            const uint32_t r = min(k0 + (t >> 5) + 8u * j, max_nw - 1u);
            v[j] = *reinterpret_cast<const uint32_t *>(rows + (size_t)r * 64u + 2u * (t & 31u));
        }
#pragma unroll
        for (int j = 0; j < kPackTile / 8; ++j)
            *reinterpret_cast<uint32_t *>(&tile[((t >> 5) + 8u * j) * kPackTileStride + 2u * (t & 31u)]) = v[j];
        __syncthreads();
        // wavefront w writes lanes 16 w .. 16 w + 15; its thread u has word numbers k0 + u, k0 + 64 + u, ...
#pragma unroll 4
        for (int j = 0; j < 16; ++j) {
            const uint32_t i = (t >> 6) * 16u + j;
            const uint32_t nw = s_nw[i];
#pragma unroll
            for (uint32_t part = 0; part < (uint32_t)kPackTile; part += 64u) {
                const uint32_t row = part + (t & 63u), k = k0 + row;
                if (k < nw) payload[s_first[i] + 2u + (nw - 1u - k)] = tile[row * kPackTileStride + i];
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------------------------------------------------
// Decode.
// --------------------------------------------------------------------------------------------
__global__ void k_init_status(Status *status) { init_status(status); }

__global__ void k_clear_report(Report *report)
{
    if (threadIdx.x < 16u) report->raised[threadIdx.x] = 0u;
    if (threadIdx.x == 16u) report->payload_bytes = 0ull;
}

// The same, and the look-back descriptors of the one-pass encoder cleared.
__global__ void k_init_one_pass(Status *status, unsigned long long *desc, uint32_t n)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0u) init_status(status);
    if (i < n) desc[i] = 0ull;
}

// Whether a container's header is that of this batch.  `word11` is header word 11 for containers that use it (the
// number of mixture components); containers that leave it reserved pass 0 and it is not looked at.
__device__ __forceinline__ int check_header(const Geo &g, uint32_t magic, uint32_t word11, const uint8_t *__restrict__ coded,
                                            unsigned long long coded_bytes, unsigned long long *payload_bytes)
{
    const uint32_t *h = reinterpret_cast<const uint32_t *>(coded);
    int st = ST_OK;
    const unsigned long long payload = (unsigned long long)h[12] | ((unsigned long long)h[13] << 32);
    // (the callers have seen that a header and the offsets fit in coded_bytes: asked for beside the header)
    const uint32_t *offsets = h + kHeaderBytes / 4;
    const uint32_t first = offsets[0], last = offsets[g.lanes];
    if (h[0] != magic || h[1] != PILC_VERSION) st = ST_FORMAT;
    if (word11 != 0u && h[11] != word11) st = ST_FORMAT;
    if (h[2] != g.n || h[3] != g.h || h[4] != g.w || h[5] != 3u || h[6] != g.prec_bits ||
        h[7] != g.lane_mode || h[8] != g.lane_a || h[9] != g.lane_b || h[10] != g.lanes)
        st = ST_FORMAT;
    if (coded_bytes != kHeaderBytes + 4ull * ((unsigned long long)g.lanes + 1ull) + payload)
        st = ST_FORMAT;
    if (st == ST_OK && (payload >= (1ull << 32) || first != 0u || last != (uint32_t)payload)) st = ST_CORRUPT;
    *payload_bytes = payload;
    return st;
}

}  // namespace pilc

#include "pilc_lane_kernels.hpp"
#include "pilc_block_encode.hpp"
#include "pilc_row_decode.hpp"
#include "pilc_mix.hpp"

namespace pilc {

// --------------------------------------------------------------------------------------------
// Host side
// --------------------------------------------------------------------------------------------
// 0 chosen from the lane count, 1 thread per lane, 2 the kernels for few long lanes, 3 thread per
// lane with the one-pass encoder (the lane kernel also scans and packs)
static std::atomic<int> g_kernel_policy{0};
static std::atomic<int> g_ansai_decode_waves{0};  // 0: chosen per call
// Bound of a look-back wait of the one-pass encoder in ticks of the constant-rate clock (0: two
// seconds), and the switch that makes its first workgroup publish nothing (tests only).
static std::atomic<unsigned long long> g_one_pass_wait{0};
static std::atomic<int> g_one_pass_withhold{0};

static uint32_t compute_units()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    return (uint32_t)cus;
}

thread_local char t_hip_error[256] = "";
thread_local float t_timing_ms[16];
thread_local const char *t_timing_name[16];
thread_local int t_timing_count = 0;
static std::atomic<int> g_timing_enabled{0};

static int hip_fail(hipError_t e, const char *what)
{
    snprintf(t_hip_error, sizeof(t_hip_error), "%s: %s", what, hipGetErrorString(e));
    return PILC_E_HIP;
}

#define HIP_TRY(expr)                                   \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) return hip_fail(e_, #expr); \
    } while (0)

static std::mutex g_table_mutex;
static bool g_table_ready[64] = {false};

// psi(q) = ln w where w + ln w = q, by Newton's method for e^p + p = q (convex and increasing: from above it converges
// without overshooting).
static double guide_psi(double q)
{
    double p = q > 1.0 ? std::log(q) : q;
    for (int i = 0; i < 50; ++i) {
        const double e = std::exp(p);
        p -= (e + p - q) / (e + 1.0);
    }
    return p;
}

// The lines of g_guide: chords of psi(x - kGuideShift) + kGuideShift, moved by half of what they miss the middle by.
static void make_guide(float2 *guide)
{
    for (int i = 0; i < kGuideEntries; ++i) {
        const int octave = i >> kGuideBits, part = i & ((1 << kGuideBits) - 1);
        const double x0 = std::ldexp(1.0 + std::ldexp(part, -kGuideBits), octave);
        const double x1 = x0 + std::ldexp(1.0, octave - kGuideBits);
        const double p0 = guide_psi(x0 - kGuideShift), p1 = guide_psi(x1 - kGuideShift);
        const double pm = guide_psi(0.5 * (x0 + x1) - kGuideShift);
        const float slope = (float)((p1 - p0) / (x1 - x0));
        guide[i] = make_float2(slope, (float)(p0 - slope * x0 + 0.5 * (pm - 0.5 * (p0 + p1)) + kGuideShift));
    }
}

static int ensure_tables()
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return PILC_E_ARG;
    std::lock_guard<std::mutex> lock(g_table_mutex);
    if (g_table_ready[dev]) return PILC_OK;
    static uint32_t sig[kSigEntries + 1];
    static uint2 cell[kSigEntries];
    static uint32_t eh[kExpHiEntries], el[kExpLoEntries];
    for (int i = 0; i <= kSigEntries; ++i)
        sig[i] = (uint32_t)std::llround(std::ldexp(1.0 / (1.0 + std::exp(-(i - 1024) / 64.0)), 24));
    for (int i = 0; i < kSigEntries; ++i) {
        const uint32_t rise = sig[i + 1] - sig[i];  // at most 2^16
        cell[i] = make_uint2(rise << 11, sig[i] - rise * (uint32_t)i);
    }
    for (int i = 0; i < kExpHiEntries; ++i)
        eh[i] = (uint32_t)std::llround(std::ldexp(std::exp(4.0 - i / 64.0), 26));
    for (int i = 0; i < kExpLoEntries; ++i)
        el[i] = (uint32_t)std::llround(std::ldexp(std::exp(-i / 4096.0), 31));
    HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(g_sig_cell), cell, sizeof(cell)));
    static float2 guide[kGuideEntries];
    make_guide(guide);
    HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(g_guide), guide, sizeof(guide)));
    HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(g_exp_hi), eh, sizeof(eh)));
    HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(g_exp_lo), el, sizeof(el)));
    HIP_TRY(hipDeviceSynchronize());
    g_table_ready[dev] = true;
    return PILC_OK;
}

static uint64_t ceil_div64(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// Validates a geometry and derives the kernel-side view.  Returns PILC_OK / PILC_E_*.
static int make_geo(const pilc_geom *in, Geo *g)
{
    if (!in || in->n == 0 || in->h == 0 || in->w == 0) return PILC_E_ARG;
    if (in->prec_bits < 10 || in->prec_bits > 16) return PILC_E_ARG;
    uint64_t hw = (uint64_t)in->h * in->w;
    uint64_t total = hw * in->n;
    uint64_t lanes;
    if (in->lane_mode == 0) {
        if (in->lane_a == 0) return PILC_E_ARG;
        if (hw % in->lane_a != 0 && in->lane_a % hw != 0) return PILC_E_ARG;
        lanes = ceil_div64(total, in->lane_a);
    } else if (in->lane_mode == 1) {
        if (in->lane_a == 0 || in->lane_b == 0) return PILC_E_ARG;
        lanes = (uint64_t)in->n * ceil_div64(in->h, in->lane_a) * ceil_div64(in->w, in->lane_b);
    } else {
        return PILC_E_ARG;
    }
    // 32-bit symbol indices and lane numbers inside the kernels
    if (total * 3 + lanes + 4096 >= (1ull << 32)) return PILC_E_TOO_LARGE;
    g->n = in->n;
    g->h = in->h;
    g->w = in->w;
    g->hw = (uint32_t)hw;
    g->prec_bits = in->prec_bits;
    g->lane_mode = in->lane_mode;
    g->lane_a = in->lane_a;
    g->lane_b = in->lane_b;
    g->tiles_x = in->lane_mode == 1 ? (uint32_t)ceil_div64(in->w, in->lane_b) : 1u;
    g->tiles_per_img =
        in->lane_mode == 1 ? (uint32_t)(ceil_div64(in->h, in->lane_a) * g->tiles_x) : 1u;
    g->total_px = (uint32_t)total;
    g->lanes = (uint32_t)lanes;
    g->by_hw = FastDiv::make(g->hw);
    return PILC_OK;
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Symbols of the longest lane.
static uint32_t max_lane_symbols(const Geo &g)
{
    const uint64_t px = g.lane_mode == 0 ? (uint64_t)(g.lane_a < g.total_px ? g.lane_a : g.total_px)
                                         : (uint64_t)(g.lane_a < g.h ? g.lane_a : g.h) *
                                               (g.lane_b < g.w ? g.lane_b : g.w);
    return (uint32_t)(3u * px);
}

struct Workspace {
    size_t status_off, report_off, words_off, state_off, sums_off, desc_off, scratch_off, total;
    uint32_t scan_blocks;
};

static Workspace layout(const Geo &g)
{
    Workspace w;
    w.scan_blocks = (uint32_t)ceil_div64(g.lanes, kScanTile);
    static_assert(sizeof(Status) <= 64 && sizeof(Report) <= 128, "both in the first 256 bytes");
    size_t off = 0;
    w.status_off = off;
    w.report_off = 128;
    off = align256(off + sizeof(Status));
    w.words_off = off;
    off = align256(off + 4 * (size_t)g.lanes);
    w.state_off = off;
    off = align256(off + 4 * (size_t)g.lanes);
    w.sums_off = off;
    off = align256(off + 8 * (size_t)w.scan_blocks);
    w.desc_off = off;  // one look-back descriptor per workgroup of the one-pass encoder (>= 64 lanes each)
    off = align256(off + 8 * (size_t)ceil_div64(g.lanes, 64));
    w.scratch_off = off;
    // one 16-bit word per symbol, plus one spare word per lane for the branch-free encoder; the
    // thread-per-lane encoder gives every lane of a block of 64 the room of the longest lane
    const size_t linear = (size_t)g.total_px * 3 + g.lanes + 64;
    const size_t by_thread = (((size_t)g.lanes + 63) & ~(size_t)63) * max_lane_symbols(g);
    off = align256(off + 2 * (linear > by_thread ? linear : by_thread));
    w.total = off;
    return w;
}

static int status_to_error(int st)
{
    switch (st) {
    case ST_OK: return PILC_OK;
    case ST_CAPACITY: return PILC_E_CAPACITY;
    case ST_TOO_LARGE: return PILC_E_TOO_LARGE;
    case ST_FORMAT: return PILC_E_FORMAT;
    case ST_PARAMS: return PILC_E_ARG;
    case ST_TIMEOUT: return PILC_E_TIMEOUT;
    default: return PILC_E_CORRUPT;
    }
}

// Reports in pinned host memory: one allocation of kReports of them, made by the first call that wants one and kept until
// the process ends.  A call has one to itself and gives it back once its stream has been synchronised; a call that
// finds none free (or no memory) keeps its report in the workspace, clears it with a kernel and copies it back.
// (A copy of sixteen bytes costs a call some ten microseconds.  With the scan in one launch and the header checked by the
// decoder itself, 64 images of 32 x 32 encoded and decoded take 85 us, before 110.)
constexpr int kReports = 64;
static std::mutex g_report_mutex;
static Report *g_reports = nullptr;
static bool g_reports_tried = false, g_report_taken[kReports];

class CallReport {
public:
    // `pinned` false: the caller must not make the library allocate anything
    CallReport(Report *in_workspace, hipStream_t stream, bool pinned) : dev_(in_workspace), stream_(stream)
    {
        if (pinned) {
            std::lock_guard<std::mutex> lock(g_report_mutex);
            if (!g_reports_tried) {
                g_reports_tried = true;
                void *ptr = nullptr;
                if (hipHostMalloc(&ptr, sizeof(Report) * kReports, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess)
                    g_reports = static_cast<Report *>(ptr);
                else
                    (void)hipGetLastError();
            }
            for (int i = 0; g_reports && i < kReports; ++i)
                if (!g_report_taken[i]) {
                    g_report_taken[i] = true;
                    slot_ = i;
                    host_ = g_reports + i;
                    break;
                }
        }
        void *seen = nullptr;
        if (host_ && hipHostGetDevicePointer(&seen, host_, 0) == hipSuccess) {
            memset(host_, 0, sizeof(Report));
            dev_ = static_cast<Report *>(seen);
        } else {
            if (host_) (void)hipGetLastError();  // (else the look at the launches would find it and fail the call)
            give_back();
            k_clear_report<<<1, 64, 0, stream_>>>(dev_);
        }
    }
    ~CallReport()
    {
        if (host_ && !done_) (void)hipStreamSynchronize(stream_);  // (kernels may still write to it)
        give_back();
    }
    CallReport(const CallReport &) = delete;
    CallReport &operator=(const CallReport &) = delete;
    Report *dev() const { return dev_; }
    // Waits for the stream; the report is then in *out.
    hipError_t wait(Report *out)
    {
        hipError_t e = host_ ? hipSuccess : hipMemcpyAsync(out, dev_, sizeof(Report), hipMemcpyDeviceToHost, stream_);
        if (e == hipSuccess) e = hipStreamSynchronize(stream_);
        if (e != hipSuccess) return e;
        done_ = true;
        if (host_)
            for (size_t i = 0; i < sizeof(Report) / 4; ++i)
                reinterpret_cast<uint32_t *>(out)[i] = reinterpret_cast<volatile uint32_t *>(host_)[i];
        return e;
    }

private:
    void give_back()
    {
        if (slot_ < 0) return;
        std::lock_guard<std::mutex> lock(g_report_mutex);
        g_report_taken[slot_] = false;
        slot_ = -1;
        host_ = nullptr;
    }
    Report *dev_, *host_ = nullptr;
    hipStream_t stream_;
    int slot_ = -1;
    bool done_ = false;
};

static int raised_code(const Report &r)
{
    for (int i = 15; i > 0; --i)
        if (r.raised[i] != 0u) return i;
    return ST_OK;
}

// Optional per-kernel event timing on the caller's stream.  The events are created once per host
// thread and device and reused by every later call.
struct EventPool {
    int dev = -1;
    hipEvent_t ev[17];
};
thread_local EventPool t_events;

struct Timer {
    hipStream_t stream;
    hipEvent_t *ev = nullptr;
    const char *name[16];
    int n = 0;
    bool on;
    explicit Timer(hipStream_t s, bool allowed = true)
        : stream(s), on(allowed && g_timing_enabled.load(std::memory_order_relaxed) != 0)
    {
        t_timing_count = 0;
        if (!on) return;
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess) {
            on = false;
            return;
        }
        if (t_events.dev != dev) {
            if (t_events.dev >= 0)
                for (auto &e : t_events.ev) (void)hipEventDestroy(e);
            t_events.dev = -1;
            for (auto &e : t_events.ev)
                if (hipEventCreate(&e) != hipSuccess) {
                    on = false;
                    return;
                }
            t_events.dev = dev;
        }
        ev = t_events.ev;
        (void)hipEventRecord(ev[0], stream);
    }
    void mark(const char *what)
    {
        if (on && n < 16) {
            name[n] = what;
            (void)hipEventRecord(ev[++n], stream);
        }
    }
    void finish()  // call after the stream has been synchronised
    {
        if (!on) return;
        t_timing_name[0] = "total";
        (void)hipEventElapsedTime(&t_timing_ms[0], ev[0], ev[n]);
        for (int i = 0; i < n && i < 15; ++i) {
            t_timing_name[i + 1] = name[i];
            (void)hipEventElapsedTime(&t_timing_ms[i + 1], ev[i], ev[i + 1]);
        }
        t_timing_count = n + 1 > 16 ? 16 : n + 1;
    }
};

// Kernels that take more than 64 KB of dynamic LDS need the limit raised once per device; it is
// raised to all of a compute unit's 160 KB less the kernel's static part, so that no later call
// ever has to change it again.
static std::mutex g_lds_mutex;
static std::map<std::pair<const void *, int>, bool> g_lds_raised;
static int allow_large_lds(const void *kernel)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_lds_mutex);
    bool &done = g_lds_raised[std::make_pair(kernel, dev)];
    if (!done) {
        hipFuncAttributes fa;
        HIP_TRY(hipFuncGetAttributes(&fa, kernel));
        HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024 - (int)fa.sharedSizeBytes));
        done = true;
    }
    return PILC_OK;
}

// True when every 8-pixel chunk of every lane starts at a multiple of 8 pixels, never straddles
// two images, and the arrays allow 16-byte (parameters) / 8-byte (pixels) vector accesses.
static bool chunks_aligned(const Geo &g, const void *img, const pilc_params *p)
{
    const bool geo = g.lane_mode == 0 ? (g.lane_a % 8 == 0 && g.hw % 8 == 0)
                                      : (g.w % 8 == 0 && g.lane_b % 8 == 0);
    return geo && ((uintptr_t)img & 7) == 0 && ((uintptr_t)p->mu & 15) == 0 &&
           ((uintptr_t)p->log_scale & 15) == 0;
}

// On top of chunks_aligned: every row of every lane is a whole number of 16-pixel chunk pairs
// that start at multiples of 16 pixels, and the pixels allow 16-byte loads.
static bool chunks_pair_up(const Geo &g, const void *img)
{
    const bool geo = g.lane_mode == 0 ? (g.lane_a % 16 == 0 && g.hw % 16 == 0)
                                      : (g.w % 16 == 0 && g.lane_b % 16 == 0);
    return geo && ((uintptr_t)img & 15) == 0;
}

// On top of chunks_pair_up: flat lanes of whole 64-pixel groups (three 128-byte lines of each
// parameter array) that start on a line.
static bool lanes_line_up(const Geo &g, const pilc_params *p)
{
    return g.lane_mode == 0 && g.lane_a % 64 == 0 && g.total_px % g.lane_a == 0 &&
           ((uintptr_t)p->mu & 127) == 0 && ((uintptr_t)p->log_scale & 127) == 0;
}

// The few-lane kernels pay off while there are too few lanes to fill the chip with one thread
// each (256 CUs x 4 SIMDs x 64 threads = 65,536 threads for a single wave per SIMD).
// Encoder: by then the block encoder's time goes with the number of pixels and the other's with a lane's chunks, so where they meet
// depends on what a chunk costs there.  Block against thread per lane, us (2^M = 8192):
//   rows that align: flat lanes of 32 28,672 52 and 54, 32,768 57 and 56, 40,960 63 and 58; of 64 40,960 84 and 84, 49,152
//   95 and 85; of 96 36,864 98 and 103, 40,960 101 and 101; tiles of 8 x 16 36,864 112 and 115, 40,960 119 and
//   114; of 16 x 16 32,768 154 and 184, 40,960 178 and 187, 49,152 214 and 184; of 32 x 32 40,960 527 and 647, 57,344 702 and 703;
//   rows that do not, where the other's chunks straddle lines and the last one of a row is a short one: tiles of 8 x 8 40,800 83 and
//   91, 48,960 92 and 90; flat lanes of 99 57,344 136 and 136, 65,536 148 and 132, of 333 98,304 453 and 545; tiles of 10 x 10 65,520
//   141 and 163, 98,160 185 and 187; of 16 x 16 57,120 244 and 253, 65,520 274 and 262; and in lanes of 512 pixels and more latest:
//   30 x 20 98,300 710 and 851, 114,600 815 and 893; 32 x 32 114,600 1333 and 1631; flat lanes of 515 114,000 767 and 936, of 777 1067
//   and 1456; 35 x 15 114,000 742 and 742; 74 x 7 98,000 644 and 729, 114,000 732 and 756; but in tiles of one or two whole chunks a row,
//   which waste nothing thread per lane, sooner: 64 x 8 80,000 531 and 574, 89,000 578 and 585, 97,000 618 and 597, 113,000 706 and 620;
//   96 x 8 90,000 829 and 903, 114,000 1019 and 969; 32 x 16 89,000 579 and 622, 105,000 666 and 651, 113,000 711 and 664.
// The lines of lanes below 512 pixels lie where the two met before the block encoder became faster: between a line and where they meet
// now a call takes up to 1.45 times the better time (aligned tiles of 32 x 32 at 36,864 lanes 644 and not 479, of 16 x 16 186 and
// not 164; unaligned ones of 10 x 10 at 44,880 156 and not 112; flat lanes of 333 at 45,056 315 and not 237).  All for 256 compute units.
static bool use_few_lane_encoder(const Geo &g, bool aligned, bool lines)
{
    const int policy = g_kernel_policy.load(std::memory_order_relaxed);
    if (max_lane_symbols(g) > kLaneMostSymbols) return true;  // (the other's words would be out of its reach)
    if (policy == 1 || policy == 3) return false;
    if (policy == 2) return true;
    const uint32_t pixels = max_lane_symbols(g) / 3u;
    if (pixels <= 40u) return g.lanes <= 28672u;
    if (aligned && !lines) return g.lanes <= 32768u;
    if (!aligned && pixels >= 512u)
        return g.lanes <= (g.lane_mode == 1u && (g.lane_b == 8u || g.lane_b == 16u) ? 92160u : 114688u);
    return g.lanes <= (aligned || pixels > 64u ? 40960u : 36864u);
}

// Decoder: the rows are ahead while one round of their workgroups (two on a compute unit, kRowLanes lanes each) takes
// all lanes, and behind from the second round on, whatever the lanes' shape.  Rows against thread per lane, us: flat lanes of
// 64, 256 and 1024 pixels: 6804 lanes 76 and 79, 238 and 249, 854 and 917; 8192 lanes 76 and 79, 241 and 252, 874 and 925;
// 8334 lanes 102 and 79, 335 and 254, 1243 and 915; tiles of 16 x 16 and 32 x 32 at their clipped edges: 8192 lanes
// 248 and 277, 915 and 1031; 8384 lanes 358 and 277, 1345 and 1029.  Where the model does not fit, the thread-per-lane
// decoder is ahead earlier (uniformly random pixels, 6250 lanes: 11.2 against 7.4 ms; an error of the means of 4 under
// scales around 1, 7360 lanes of 128: 192 against 132 us), but that is not known here.
static bool use_few_lane_decoder(const Geo &g)
{
    const int policy = g_kernel_policy.load(std::memory_order_relaxed);
    if (policy == 1 || policy == 3) return false;
    if (policy == 2) return true;
    return g.lanes <= 2u * compute_units() * (uint32_t)kRowLanes;
}

// Launches the scan of the items' bytes; true if it has also formed the offset table.
static bool launch_scan(const HeaderWords &head, uint32_t items, uint32_t blocks, const ItemBytes &bytes, const uint32_t *counts,
                        unsigned long long *sums, uint8_t *coded, size_t capacity, Status *status, Report *report,
                        uint32_t *offsets, bool always_form, hipStream_t stream)
{
    const unsigned long long room = capacity;
    if (blocks <= kScanFewTiles) {
        k_scan_sums<<<blocks, kScanThreads, 0, stream>>>(head, items, bytes, counts, sums, coded, room, status, report);
        if (!always_form) return false;
    } else {
        k_scan_partials<<<blocks, kScanThreads, 0, stream>>>(items, bytes, counts, sums);
        k_scan_spine<<<1, kScanThreads, 0, stream>>>(head, items, blocks, sums, coded, room, status, report);
    }
    k_scan_apply<<<blocks, kScanThreads, 0, stream>>>(items, bytes, counts, sums, offsets);
    return true;
}

// Workgroup size of the thread-per-lane kernels.
static int lane_block_threads(const Geo &g) { return g.lanes >= (1u << 16) ? kLaneMaxThreads : 64; }

}  // namespace pilc

using namespace pilc;

extern "C" {

uint32_t pilc_version(void) { return PILC_VERSION; }

const char *pilc_strerror(int code)
{
    switch (code) {
    case PILC_OK: return "success";
    case PILC_E_ARG: return "invalid argument (null or misaligned pointer, or bad geometry)";
    case PILC_E_WORKSPACE: return "workspace too small";
    case PILC_E_CAPACITY: return "coded output does not fit the given capacity";
    case PILC_E_TOO_LARGE: return "batch too large for 32-bit offsets";
    case PILC_E_FORMAT: return "container header does not match (magic, version, geometry or size)";
    case PILC_E_CORRUPT: return "container is corrupt (offsets, lane overrun or final state)";
    case PILC_E_HIP: return "HIP runtime failure";
    case PILC_E_TIMEOUT: return "a bounded wait between workgroups ran out";
    default: return "unknown error code";
    }
}

const char *pilc_last_hip_error(void) { return t_hip_error; }

void pilc_set_timing(int enabled) { g_timing_enabled.store(enabled, std::memory_order_relaxed); }

int pilc_set_kernel_policy(int policy)
{
    if (policy < 0 || policy > 3) return PILC_E_ARG;
    g_kernel_policy.store(policy, std::memory_order_relaxed);
    return PILC_OK;
}

void pilc_set_one_pass_wait(uint64_t ticks, int withhold_first)
{
    g_one_pass_wait.store(ticks, std::memory_order_relaxed);
    g_one_pass_withhold.store(withhold_first != 0, std::memory_order_relaxed);
}

int pilc_last_timing(float *ms_out_host, int capacity)
{
    int k = t_timing_count < capacity ? t_timing_count : capacity;
    for (int i = 0; i < k; ++i) ms_out_host[i] = t_timing_ms[i];
    return k;
}

const char *pilc_timing_name(int i)
{
    return (i >= 0 && i < t_timing_count) ? t_timing_name[i] : "";
}

uint64_t pilc_lane_count(const pilc_geom *geom)
{
    Geo g;
    return make_geo(geom, &g) == PILC_OK ? g.lanes : 0;
}

int pilc_workspace_size(const pilc_geom *geom, size_t *workspace_bytes_host,
                        size_t *max_coded_bytes_host)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (workspace_bytes_host) *workspace_bytes_host = layout(g).total;
    if (max_coded_bytes_host)
        *max_coded_bytes_host = kHeaderBytes + 4 * ((size_t)g.lanes + 1) + 4 * (size_t)g.lanes +
                                2 * (size_t)g.total_px * 3;
    return PILC_OK;
}

static bool params_ok(const pilc_params *p)
{
    return p && p->mu && p->log_scale && p->chan_coef && ((uintptr_t)p->mu & 1) == 0 &&
           ((uintptr_t)p->log_scale & 1) == 0 && ((uintptr_t)p->chan_coef & 1) == 0;
}

int pilc_symbol_tables(const pilc_geom *geom, const uint8_t *img_dev, const pilc_params *params,
                       uint32_t *cum_out_dev, uint32_t *freq_out_dev, void *hip_stream)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (!img_dev || !params_ok(params) || !cum_out_dev || !freq_out_dev ||
        ((uintptr_t)cum_out_dev & 3) || ((uintptr_t)freq_out_dev & 3))
        return PILC_E_ARG;
    if ((rc = ensure_tables()) != PILC_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;
    uint32_t blocks = (uint32_t)ceil_div64(g.total_px, 256);
    k_symbol_tables<<<blocks, 256, 0, stream>>>(g, img_dev, params->mu, params->log_scale,
                                                params->chan_coef, cum_out_dev, freq_out_dev);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(stream));
    return PILC_OK;
}

// The body of pilc_encode once the arguments have been checked: `workspace_dev` holds at least
// layout(g).total bytes.  `timed` is false for callers that must not create HIP events.
static int encode_checked(const Geo &g, const uint8_t *img_dev, const pilc_params *params,
                          void *workspace_dev, uint8_t *coded_dev, size_t coded_capacity,
                          uint64_t *coded_bytes_host, hipStream_t stream, bool timed)
{
    const Workspace ws = layout(g);
    const size_t table_end = kHeaderBytes + 4 * ((size_t)g.lanes + 1);
    uint8_t *base = static_cast<uint8_t *>(workspace_dev);
    Status *status = reinterpret_cast<Status *>(base + ws.status_off);
    uint32_t *lane_words = reinterpret_cast<uint32_t *>(base + ws.words_off);
    uint32_t *lane_state = reinterpret_cast<uint32_t *>(base + ws.state_off);
    unsigned long long *sums = reinterpret_cast<unsigned long long *>(base + ws.sums_off);
    uint16_t *scratch = reinterpret_cast<uint16_t *>(base + ws.scratch_off);
    uint32_t *offsets = reinterpret_cast<uint32_t *>(coded_dev + kHeaderBytes);
    uint16_t *payload = reinterpret_cast<uint16_t *>(coded_dev + table_end);

    Timer timer(stream, timed);
    const bool vec = chunks_aligned(g, img_dev, params);
    const bool pair = vec && chunks_pair_up(g, img_dev);
    const bool line = pair && lanes_line_up(g, params);
    const bool few_lanes = use_few_lane_encoder(g, vec, line);
    const uint32_t lane_cap = few_lanes ? 0u : max_lane_symbols(g);  // selects the scratch layout
    const HeaderWords head = {{kMagicPilc, PILC_VERSION, g.n, g.h, g.w, 3u, g.prec_bits,
                               g.lane_mode, g.lane_a, g.lane_b, g.lanes, 0u}};
    // Policy 3: the lane kernel also scans and packs (one pass).  Not the default: measured 5 %
    // (64 x 64 images, one lane per row) to 10 % (16 x 16 tiles of video frames) slower than the
    // lane kernel followed by the scan and pack kernels.
    const bool one_pass = !few_lanes && g_kernel_policy.load(std::memory_order_relaxed) == 3;
    OnePass op = {};
    if (one_pass) {
        const int bt = lane_block_threads(g);
        const uint32_t nb = (uint32_t)ceil_div64(g.lanes, bt);
        int dev = 0, khz = 0;
        HIP_TRY(hipGetDevice(&dev));
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
            khz = 100000;
        const unsigned long long wait = g_one_pass_wait.load(std::memory_order_relaxed);
        op.desc = reinterpret_cast<unsigned long long *>(base + ws.desc_off);
        op.ticket = &status->ticket;
        op.status = status;
        op.coded = coded_dev;
        op.payload_capacity = coded_capacity - table_end;
        op.wait_ticks = wait ? wait : 2000ull * (unsigned long long)khz;
        op.groups = nb;
        op.withhold_first = (uint32_t)g_one_pass_withhold.load(std::memory_order_relaxed);
        op.head = head;
        k_init_one_pass<<<(nb + 255u) / 256u, 256, 0, stream>>>(status, op.desc, nb);
    }
    op.status = status;  // (set to zero by the lane kernel unless it works in one pass)
    std::optional<CallReport> report;  // (in one pass the outcome is in `status`)
    if (!one_pass) report.emplace(reinterpret_cast<Report *>(base + ws.report_off), stream, timed);
    if (few_lanes) {
        const uint32_t cus = compute_units();
        const uint32_t blocks = (uint32_t)ceil_div64(g.lanes, kEncLanes);
        auto launch = [&](auto producers) {
            constexpr int kProducers = decltype(producers)::value;
            k_encode_block<kProducers><<<blocks, enc_threads(kProducers), 0, stream>>>(
                g, img_dev, params->mu, params->log_scale, params->chan_coef, scratch, lane_words, lane_state, status);
        };
        if (blocks <= cus) launch(std::integral_constant<int, kEncAloneProducers>{});
        else if (blocks <= 2u * cus) launch(std::integral_constant<int, kEncPairProducers>{});
        else launch(std::integral_constant<int, kEncManyProducers>{});
    } else {
        const int bt = lane_block_threads(g);
        uint32_t nb = (uint32_t)ceil_div64(g.lanes, bt);
        if (one_pass) {
            // workgroups take groups of lanes from a counter until none is left: no more of them
            // than the chip holds at once (a workgroup that starts late finds nothing to do)
            int dev = 0, cus = 0;
            HIP_TRY(hipGetDevice(&dev));
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
                cus = 256;
            const uint32_t resident = (uint32_t)cus * (uint32_t)(1024 / bt);
            if (nb > resident) nb = resident;
        }
#define PILC_LAUNCH_ENCODE(ONE, VEC, PAIR, LINE)                                                      \
    k_encode_lanes<ONE, VEC, PAIR, LINE><<<nb, bt, 0, stream>>>(g, img_dev, params->mu, params->log_scale, \
                                                               params->chan_coef, scratch, lane_cap,  \
                                                               lane_words, lane_state, op)
        if (one_pass) {
            if (line) PILC_LAUNCH_ENCODE(true, true, true, true);
            else if (pair) PILC_LAUNCH_ENCODE(true, true, true, false);
            else if (vec) PILC_LAUNCH_ENCODE(true, true, false, false);
            else PILC_LAUNCH_ENCODE(true, false, false, false);
        } else {
            if (line) PILC_LAUNCH_ENCODE(false, true, true, true);
            else if (pair) PILC_LAUNCH_ENCODE(false, true, true, false);
            else if (vec) PILC_LAUNCH_ENCODE(false, true, false, false);
            else PILC_LAUNCH_ENCODE(false, false, false, false);
        }
#undef PILC_LAUNCH_ENCODE
    }
    timer.mark(few_lanes ? "k_encode_block" : "k_encode_lanes");
    if (!one_pass) {
        // a run of lanes per workgroup: about 16K symbols' worth, at most 256 lanes; of a small batch less, so that
        // there are kPackBlocks workgroups, but not less than kPackLeast symbols (64 images of 32 x 32 in
        // 2048 lanes 28.5 -> 8.0 us, 400 of 64 x 64 in 25,600 lanes 28.7 -> 13.4; with 512 workgroups of
        // 1024 symbols 8.4 and 20.0)
        const uint32_t lane_sym = std::max(1u, max_lane_symbols(g));
        uint32_t pack_lanes = 16384u / lane_sym;
        pack_lanes = std::min(pack_lanes, std::max(g.lanes / kPackBlocks, kPackLeast / lane_sym));
        pack_lanes = lane_cap != 0u ? 64u : std::min(std::max(pack_lanes, 1u), (uint32_t)kPackMaxLanes);
        const uint32_t pack_blocks = (uint32_t)ceil_div64(g.lanes, pack_lanes);
        const PackAlone pk = {scans_alone(g.lanes, pack_blocks) ? 1u : 0u, head, coded_dev, coded_capacity, report->dev()};
        const bool formed = pk.alone == 0u && launch_scan(head, g.lanes, ws.scan_blocks, kLaneBytes, lane_words, sums, coded_dev,
                                                          coded_capacity, status, report->dev(), offsets, false, stream);
        if (pk.alone == 0u) timer.mark("scan");
        if (lane_cap != 0u)
            (lane_cap <= 256u ? k_pack_by_thread<128> : k_pack_by_thread<256>)<<<pack_blocks, kScanThreads, 0, stream>>>(
                g.lanes, lane_cap, scratch, lane_words, lane_state, sums, formed, offsets, payload, status, pk);
        else
            k_pack<<<pack_blocks, kScanThreads, 0, stream>>>(
                g, pack_lanes, scratch, lane_words, lane_state, sums, formed, offsets, payload, status, pk);
        timer.mark(lane_cap != 0u ? "k_pack_by_thread" : "k_pack");
    }
    HIP_TRY(hipGetLastError());
    if (one_pass) {
        Status host_status;
        HIP_TRY(hipMemcpyAsync(&host_status, status, sizeof(Status), hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        timer.finish();
        if (host_status.code != ST_OK) return status_to_error(host_status.code);
        *coded_bytes_host = table_end + host_status.payload_bytes;
        return PILC_OK;
    }
    Report seen;
    HIP_TRY(report->wait(&seen));
    timer.finish();
    if (raised_code(seen) != ST_OK) return status_to_error(raised_code(seen));
    *coded_bytes_host = table_end + seen.payload_bytes;
    return PILC_OK;
}

int pilc_encode(const pilc_geom *geom, const uint8_t *img_dev, const pilc_params *params,
                void *workspace_dev, size_t workspace_bytes, uint8_t *coded_dev,
                size_t coded_capacity, uint64_t *coded_bytes_host, void *hip_stream)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (!img_dev || !params_ok(params) || !workspace_dev || !coded_dev || !coded_bytes_host)
        return PILC_E_ARG;
    if (((uintptr_t)workspace_dev & 255) || ((uintptr_t)coded_dev & 15)) return PILC_E_ARG;
    if (workspace_bytes < layout(g).total) return PILC_E_WORKSPACE;
    if (coded_capacity < kHeaderBytes + 4 * ((size_t)g.lanes + 1)) return PILC_E_CAPACITY;
    if ((rc = ensure_tables()) != PILC_OK) return rc;
    return encode_checked(g, img_dev, params, workspace_dev, coded_dev, coded_capacity,
                          coded_bytes_host, (hipStream_t)hip_stream, true);
}

// --------------------------------------------------------------------------------------------
// pilc_encode for callers that cannot allocate device memory: the workspace is a file-scope
// device array.  Every GPU holds its own copy at its own address; the address is asked for once
// per device, with that device current, and host code uses only that pointer (the array's name
// is not a device address in host code).
// --------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PILC_STATIC_SCRATCH_BYTES];

static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[64] = {nullptr};

static int static_scratch(void **out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return PILC_E_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || ((uintptr_t)ptr & 255)) {
            snprintf(t_hip_error, sizeof(t_hip_error), "hipGetSymbolAddress(scratch) gave %p", ptr);
            return PILC_E_HIP;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return PILC_OK;
}

int pilc_encode_static(const pilc_geom *geom, const uint8_t *img_dev, const pilc_params *params,
                       uint8_t *coded_dev, size_t coded_capacity, uint64_t *coded_bytes_host,
                       void *hip_stream)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (!img_dev || !params_ok(params) || !coded_dev || !coded_bytes_host) return PILC_E_ARG;
    if ((uintptr_t)coded_dev & 15) return PILC_E_ARG;
    if (layout(g).total > (size_t)PILC_STATIC_SCRATCH_BYTES) return PILC_E_WORKSPACE;
    if (coded_capacity < kHeaderBytes + 4 * ((size_t)g.lanes + 1)) return PILC_E_CAPACITY;
    if ((rc = ensure_tables()) != PILC_OK) return rc;
    void *ws = nullptr;
    if ((rc = static_scratch(&ws)) != PILC_OK) return rc;
    // Nothing in the workspace has to start at zero: the status block is set by the first kernel
    // and every count, state and scratch word that is read has been written by this call.
    return encode_checked(g, img_dev, params, ws, coded_dev, coded_capacity, coded_bytes_host,
                          (hipStream_t)hip_stream, false);
}

int pilc_decode(const pilc_geom *geom, const uint8_t *coded_dev, size_t coded_bytes,
                const pilc_params *params, void *workspace_dev, size_t workspace_bytes,
                uint8_t *img_out_dev, void *hip_stream)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (!coded_dev || !params_ok(params) || !workspace_dev || !img_out_dev) return PILC_E_ARG;
    if (((uintptr_t)workspace_dev & 255) || ((uintptr_t)coded_dev & 15)) return PILC_E_ARG;
    const Workspace ws = layout(g);
    if (workspace_bytes < ws.total) return PILC_E_WORKSPACE;
    const size_t table_end = kHeaderBytes + 4 * ((size_t)g.lanes + 1);
    if (coded_bytes < table_end) return PILC_E_FORMAT;  // cannot even hold header + offsets
    if ((rc = ensure_tables()) != PILC_OK) return rc;

    hipStream_t stream = (hipStream_t)hip_stream;
    CallReport report(reinterpret_cast<Report *>(static_cast<uint8_t *>(workspace_dev) + ws.report_off), stream, true);

    Timer timer(stream);
    const bool few_lanes = use_few_lane_decoder(g);
    if (few_lanes) {
        // all lanes alike and made of whole batches of 16 pixels: no per-row activity masks
        const bool even = g.lane_mode == 0 ? (g.lane_a % kRowBatch == 0 && g.total_px % g.lane_a == 0)
                                           : (g.h % g.lane_a == 0 && g.w % g.lane_b == 0 &&
                                              (g.lane_a * g.lane_b) % kRowBatch == 0);
        const uint32_t nblk = (uint32_t)ceil_div64(g.lanes, kRowLanes);
        // a stager beside every decoding wavefront while one workgroup per compute unit holds all lanes
        int dev = 0, khz = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
            khz = 100000;
        const bool staged = nblk <= compute_units();
        // the bound of the waits between a decoding wavefront and its stager, and the test switch
        const unsigned long long asked = g_one_pass_wait.load(std::memory_order_relaxed);
        const unsigned long long wait_ticks = asked ? asked : 2000ull * (unsigned long long)khz;
        const uint32_t withhold = (uint32_t)g_one_pass_withhold.load(std::memory_order_relaxed);
#define PILC_DECODE_ROWS(RAGGED, STAGED)                                                              \
    k_decode_rows<RAGGED, STAGED><<<nblk, (STAGED ? 2 : 1) * 64 * kRowWaves, 0, stream>>>(           \
        g, coded_dev, (unsigned long long)coded_bytes, params->mu, params->log_scale, params->chan_coef, \
        img_out_dev, report.dev(), wait_ticks, withhold)
        if (even && staged) PILC_DECODE_ROWS(false, true);
        else if (even) PILC_DECODE_ROWS(false, false);
        else if (staged) PILC_DECODE_ROWS(true, true);
        else PILC_DECODE_ROWS(true, false);
#undef PILC_DECODE_ROWS
    } else {
        const bool vec = chunks_aligned(g, img_out_dev, params);
        const bool pair = vec && chunks_pair_up(g, img_out_dev);
        // more than a wavefront a SIMD, or than two in long rows that do not align (figures at the kernel)
        const bool one_side = g.lanes > compute_units() * (vec || (g.lane_mode == 1u ? g.lane_b : g.lane_a) <= 32u ? 256u : 512u);
        auto kern = one_side ? (pair ? k_decode_lanes<true, true, true> : vec ? k_decode_lanes<true, false, true> : k_decode_lanes<false, false, true>)
                             : (pair ? k_decode_lanes<true, true, false> : vec ? k_decode_lanes<true, false, false> : k_decode_lanes<false, false, false>);
        const int bt = lane_block_threads(g);
        const uint32_t nb = (uint32_t)ceil_div64(g.lanes, bt);
        kern<<<nb, bt, (size_t)bt * kRingRow * sizeof(uint16_t), stream>>>(g, coded_dev, (unsigned long long)coded_bytes,
                                                                           params->mu, params->log_scale,
                                                                           params->chan_coef, img_out_dev, report.dev());
    }
    timer.mark(few_lanes ? "k_decode_rows" : "k_decode_lanes");
    HIP_TRY(hipGetLastError());
    Report seen;
    HIP_TRY(report.wait(&seen));
    timer.finish();
    return status_to_error(raised_code(seen));
}

// --------------------------------------------------------------------------------------------
// Mixture of K logistic laws per subpixel
// --------------------------------------------------------------------------------------------
static bool mix_params_ok(const pilc_mix_params *p)
{
    return p && p->mu && p->log_scale && p->weight && p->chan_coef && p->num_comp >= 1u &&
           p->num_comp <= (uint32_t)kMixMaxComp && ((uintptr_t)p->mu & 1) == 0 &&
           ((uintptr_t)p->log_scale & 1) == 0 && ((uintptr_t)p->weight & 1) == 0 &&
           ((uintptr_t)p->chan_coef & 1) == 0;
}

// The component count a mixture kernel was built for (components in registers: arrays on 4-byte
// boundaries), or 0 for the kernels that take any K at run time.
static int mix_built_for(const pilc_mix_params *p)
{
    const bool aligned =
        (((uintptr_t)p->mu | (uintptr_t)p->log_scale | (uintptr_t)p->weight) & 3) == 0;
    return aligned ? (int)p->num_comp : 0;
}

#define PILC_MIX_KERNEL_FOR(NAME, NONE)                                                          \
    static decltype(&NAME<1>) NAME##_for(int built)                                              \
    {                                                                                            \
        switch (built) {                                                                         \
        case 1: return NAME<1>;                                                                  \
        case 2: return NAME<2>;                                                                  \
        case 3: return NAME<3>;                                                                  \
        case 4: return NAME<4>;                                                                  \
        case 5: return NAME<5>;                                                                  \
        case 6: return NAME<6>;                                                                  \
        case 7: return NAME<7>;                                                                  \
        case 8: return NAME<8>;                                                                  \
        case 9: return NAME<9>;                                                                  \
        case 10: return NAME<10>;                                                                \
        case 11: return NAME<11>;                                                                \
        case 12: return NAME<12>;                                                                \
        case 13: return NAME<13>;                                                                \
        case 14: return NAME<14>;                                                                \
        case 15: return NAME<15>;                                                                \
        case 16: return NAME<16>;                                                                \
        default: return NONE;                                                                    \
        }                                                                                        \
    }
PILC_MIX_KERNEL_FOR(k_mix_encode_chunks, nullptr)
PILC_MIX_KERNEL_FOR(k_mix_decode, k_mix_decode<0>)
PILC_MIX_KERNEL_FOR(k_mix_decode_rows, nullptr)
#undef PILC_MIX_KERNEL_FOR

int pilc_mix_encode(const pilc_geom *geom, const uint8_t *img_dev, const pilc_mix_params *params,
                    void *workspace_dev, size_t workspace_bytes, uint8_t *coded_dev,
                    size_t coded_capacity, uint64_t *coded_bytes_host, void *hip_stream)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (!img_dev || !mix_params_ok(params) || !workspace_dev || !coded_dev || !coded_bytes_host)
        return PILC_E_ARG;
    if (((uintptr_t)workspace_dev & 255) || ((uintptr_t)coded_dev & 15)) return PILC_E_ARG;
    const Workspace ws = layout(g);
    if (workspace_bytes < ws.total) return PILC_E_WORKSPACE;
    const size_t table_end = kHeaderBytes + 4 * ((size_t)g.lanes + 1);
    if (coded_capacity < table_end) return PILC_E_CAPACITY;
    if ((rc = ensure_tables()) != PILC_OK) return rc;

    hipStream_t stream = (hipStream_t)hip_stream;
    uint8_t *base = static_cast<uint8_t *>(workspace_dev);
    Status *status = reinterpret_cast<Status *>(base + ws.status_off);
    uint32_t *lane_words = reinterpret_cast<uint32_t *>(base + ws.words_off);
    uint32_t *lane_state = reinterpret_cast<uint32_t *>(base + ws.state_off);
    unsigned long long *sums = reinterpret_cast<unsigned long long *>(base + ws.sums_off);
    uint16_t *scratch = reinterpret_cast<uint16_t *>(base + ws.scratch_off);
    uint32_t *offsets = reinterpret_cast<uint32_t *>(coded_dev + kHeaderBytes);
    uint16_t *payload = reinterpret_cast<uint16_t *>(coded_dev + table_end);
    const MixArgs args = {params->mu, params->log_scale, params->weight, params->chan_coef,
                          params->num_comp};
    const int built = mix_built_for(params);
    const uint32_t lane_cap = max_lane_symbols(g);
    auto chunks = k_mix_encode_chunks_for(built);
    const size_t lds = chunks ? mix_encode_lds_bytes(built) : mix_lds_bytes(params->num_comp, true);
    if ((rc = allow_large_lds(chunks ? reinterpret_cast<const void *>(chunks) : reinterpret_cast<const void *>(&k_mix_encode))) != PILC_OK)
        return rc;

    CallReport report(reinterpret_cast<Report *>(base + ws.report_off), stream, true);
    Timer timer(stream);
    k_init_status<<<1, 1, 0, stream>>>(status);
    if (chunks) {
        const MixChunk c = mix_chunk(g.lanes, lane_cap / 3u);
        const uint64_t waves = ceil_div64(g.lanes, 1u << c.log_lanes);
        const uint32_t threads = (uint32_t)mix_encode_threads(built);
        chunks<<<(uint32_t)ceil_div64(waves, threads / 64u), threads, lds, stream>>>(
            g, c, img_dev, args, scratch, lane_cap, lane_words, lane_state, &status->code);
    } else {
        k_mix_encode<<<(uint32_t)ceil_div64(g.lanes, kMixThreads), kMixThreads, lds, stream>>>(
            g, img_dev, args, scratch, lane_cap, lane_words, lane_state, &status->code);
    }
    timer.mark(chunks ? "k_mix_encode_chunks" : "k_mix_encode");
    const HeaderWords head = {{kMagicMix, PILC_VERSION, g.n, g.h, g.w, 3u, g.prec_bits, g.lane_mode,
                               g.lane_a, g.lane_b, g.lanes, params->num_comp}};
    const uint32_t pack_blocks = (uint32_t)ceil_div64(g.lanes, 64);
    const PackAlone pk = {scans_alone(g.lanes, pack_blocks) ? 1u : 0u, head, coded_dev, coded_capacity, report.dev()};
    const bool formed = pk.alone == 0u && launch_scan(head, g.lanes, ws.scan_blocks, kLaneBytes, lane_words, sums, coded_dev,
                                                      coded_capacity, status, report.dev(), offsets, false, stream);
    if (pk.alone == 0u) timer.mark("scan");
    (lane_cap <= 256u ? k_pack_by_thread<128> : k_pack_by_thread<256>)<<<pack_blocks, kScanThreads, 0, stream>>>(
        g.lanes, lane_cap, scratch, lane_words, lane_state, sums, formed, offsets, payload, status, pk);
    timer.mark("k_pack_by_thread");
    HIP_TRY(hipGetLastError());
    Report seen;
    HIP_TRY(report.wait(&seen));
    timer.finish();
    if (raised_code(seen) != ST_OK) return status_to_error(raised_code(seen));
    *coded_bytes_host = table_end + seen.payload_bytes;
    return PILC_OK;
}

int pilc_mix_decode(const pilc_geom *geom, const uint8_t *coded_dev, size_t coded_bytes,
                    const pilc_mix_params *params, void *workspace_dev, size_t workspace_bytes,
                    uint8_t *img_out_dev, void *hip_stream)
{
    Geo g;
    int rc = make_geo(geom, &g);
    if (rc != PILC_OK) return rc;
    if (!coded_dev || !mix_params_ok(params) || !workspace_dev || !img_out_dev) return PILC_E_ARG;
    if (((uintptr_t)workspace_dev & 255) || ((uintptr_t)coded_dev & 15)) return PILC_E_ARG;
    const Workspace ws = layout(g);
    if (workspace_bytes < ws.total) return PILC_E_WORKSPACE;
    const size_t table_end = kHeaderBytes + 4 * ((size_t)g.lanes + 1);
    if (coded_bytes < table_end) return PILC_E_FORMAT;
    if ((rc = ensure_tables()) != PILC_OK) return rc;

    hipStream_t stream = (hipStream_t)hip_stream;
    const MixArgs args = {params->mu, params->log_scale, params->weight, params->chan_coef,
                          params->num_comp};
    const int policy = g_kernel_policy.load(std::memory_order_relaxed);
    const bool rows = policy == 0 ? g.lanes <= kMixRowLanes : policy == 2;
    const int built = mix_built_for(params);
    const size_t lds = rows ? 0 : mix_lds_bytes(params->num_comp, built == 0);
    auto kern = rows ? k_mix_decode_rows_for((int)params->num_comp) : k_mix_decode_for(built);
    const uint32_t group = rows ? kMixRowThreads / 16u : (uint32_t)kMixThreads;  // lanes of a workgroup
    static_assert(kMixRowThreads == kMixThreads, "one launch for both");
    if ((rc = allow_large_lds(reinterpret_cast<const void *>(kern))) != PILC_OK) return rc;

    CallReport report(reinterpret_cast<Report *>(static_cast<uint8_t *>(workspace_dev) + ws.report_off), stream, true);
    Timer timer(stream);
    kern<<<(uint32_t)ceil_div64(g.lanes, group), kMixThreads, lds, stream>>>(
        g, coded_dev, (unsigned long long)coded_bytes, args, img_out_dev, report.dev());
    timer.mark(rows ? "k_mix_decode_rows" : "k_mix_decode");
    HIP_TRY(hipGetLastError());
    Report seen;
    HIP_TRY(report.wait(&seen));
    timer.finish();
    return status_to_error(raised_code(seen));
}

}  // extern "C"

#include "pilc_ansai.hpp"
#include "pilc_twar.hpp"
