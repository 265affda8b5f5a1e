// Vision operators of detection post-processing (paper Sec. 3.1.1): the
// three-stage prefix sum (Fig. 3), segmented argsort (Fig. 2) and box_nms,
// with their C ABI (include/mivision.h).
//
// The paper's designs target integrated GPUs; what carries over to gfx950 is
// the structure: the scan's register blocking with a Hillis-Steele scan of
// block totals, the sort's equal-block local sorts followed by cooperative
// merges that only move segments spanning blocks, and NMS's
// mapping of the innermost loop onto threads with the output set invalid as a
// whole first.  On a 64-wide wavefront the Hillis-Steele passes are lane
// shuffles, the merge path of a work-group is found by a 64-way search (one
// dependent memory round trip per factor of 64), and NMS's suppression test
// becomes 64-bit masks, so that the one sequential walk per image is a
// broadcast and an OR per candidate.
#include "internal.h"
#include "../../include/miconv.h"
#include "../../include/mivision.h"

#include <algorithm>
#include <cmath>

namespace miconv {
namespace {

// ----------------------------------------------------------------- scan

constexpr int kScanThreads = 256;                     // work-groups across a row
constexpr int kScanItems = 16;                        // values per thread (register block)
constexpr int kScanTile = kScanThreads * kScanItems;  // 4096 values per tile
constexpr int kScanWide = 1024;                       // a work-group owning one of few rows

// Hillis-Steele inclusive scan of one value per thread over a work-group of
// NT threads: in pass d every thread adds the value held by the thread 2^d
// before it.  Within a wavefront the passes are lane shuffles; the NT/64
// wavefront totals are scanned the same way by the first wavefront, through
// LDS.  Returns the thread's inclusive prefix; *total gets the work-group sum.
template <int NT>
__device__ int wg_scan_incl(int v, int *wsum, int *total)
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(v, d);
        if (lane >= d) v += u;
    }
    if (lane == 63) wsum[wid] = v;
    __syncthreads();
    if (wid == 0) {
        int w = lane < NW ? wsum[lane] : 0;
#pragma unroll
        for (int d = 1; d < NW; d <<= 1) {
            const int u = __shfl_up(w, d);
            if (lane >= d) w += u;
        }
        if (lane < NW) wsum[lane] = w;
    }
    __syncthreads();
    const int r = v + (wid ? wsum[wid - 1] : 0);
    *total = wsum[NW - 1];
    __syncthreads();   // wsum is free for the next call
    return r;
}

// Lane l gets the sum of lanes 0..l of its wavefront (every lane active):
// Hillis-Steele passes within rows of 16 lanes, then the row totals
// broadcast, all as DPP operands of the adds (no LDS).
__device__ __forceinline__ int wave_scan_incl(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return v;
}

// A tile of NT * kScanItems values in registers.  A wavefront owns 1024
// consecutive values in four groups of 256; a lane holds four consecutive
// values of each group, so that loads and stores are 16 bytes per lane and
// contiguous over the wavefront as they stand: no pass through LDS.  Global
// 16-byte accesses need 4-byte alignment only, which an int32 array has.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef i32x4 i32x4_dw __attribute__((aligned(4)));
constexpr int kScanGroups = kScanItems / 4;

__device__ __forceinline__ int scan_pos(int j)
{
    return (int)((threadIdx.x >> 6) * (64 * kScanItems) + j * 256 + 4 * (threadIdx.x & 63));
}

// The first len values at x; the rest of the tile is zero.
template <int NT>
__device__ __forceinline__ void scan_load(const int32_t *x, long len, i32x4 (&q)[kScanGroups])
{
    if (len >= NT * kScanItems) {
#pragma unroll
        for (int j = 0; j < kScanGroups; ++j) q[j] = *reinterpret_cast<const i32x4_dw *>(x + scan_pos(j));
        return;
    }
    // the buffer's range check makes what lies past len zero, without branches
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(x), (short)0, (int)len * 4, 0x00020000);
#pragma unroll
    for (int j = 0; j < kScanGroups; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            q[j][e] = (int)__builtin_amdgcn_raw_buffer_load_b32(r, (scan_pos(j) + e) * 4, 0, 0);
}

// What the values of this lane's groups are preceded by within the tile, and
// the tile's sum.  wsum: NT/64 words no wavefront still reads (one barrier).
template <int NT>
__device__ __forceinline__ int scan_before(const i32x4 (&q)[kScanGroups], int (&before)[kScanGroups], int *wsum)
{
    constexpr int NW = NT / 64;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int run = 0;
#pragma unroll
    for (int j = 0; j < kScanGroups; ++j) {
        const int s = q[j][0] + q[j][1] + q[j][2] + q[j][3];
        const int incl = wave_scan_incl(s);
        before[j] = run + incl - s;
        run += __builtin_amdgcn_readlane(incl, 63);
    }
    if (lane == 0) wsum[wid] = run;
    __syncthreads();
    const int incl = wave_scan_incl(lane < NW ? wsum[lane] : 0);
    const int pre = __builtin_amdgcn_readlane(incl, wid) - run;
#pragma unroll
    for (int j = 0; j < kScanGroups; ++j) before[j] += pre;
    return __builtin_amdgcn_readlane(incl, NW - 1);
}

// Stores the first len scanned values of a tile; NTS: whole tiles are stored
// non-temporally.
template <int NT, bool NTS>
__device__ __forceinline__ void scan_store(int32_t *y, long len, i32x4 (&q)[kScanGroups],
                                           const int (&before)[kScanGroups], int carry, bool exclusive)
{
#pragma unroll
    for (int j = 0; j < kScanGroups; ++j) {
        const int b = carry + before[j];
        const int s0 = b + q[j][0], s1 = s0 + q[j][1], s2 = s1 + q[j][2], s3 = s2 + q[j][3];
        q[j] = exclusive ? i32x4{b, s0, s1, s2} : i32x4{s0, s1, s2, s3};
    }
    if (len >= NT * kScanItems) {
#pragma unroll
        for (int j = 0; j < kScanGroups; ++j) {
            if constexpr (NTS)
                __builtin_nontemporal_store(q[j], reinterpret_cast<i32x4_dw *>(y + scan_pos(j)));
            else
                *reinterpret_cast<i32x4_dw *>(y + scan_pos(j)) = q[j];
        }
        return;
    }
    const int m = (int)len;
#pragma unroll
    for (int j = 0; j < kScanGroups; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (scan_pos(j) + e < m) y[scan_pos(j) + e] = q[j][e];
}

// One work-group per row, its tiles in order with a running carry, the next
// tile's loads in flight meanwhile: the three stages inside the work-group,
// nothing shared across work-groups.  Row r is elements [r*n, r*n + n).
// row_totals[r] (if given) gets the row's sum.  NT = 1024 when the rows are
// few (a tile of 16384 values per round trip).
template <int NT>
__global__ __launch_bounds__(NT) void scan_rows_kernel(const int32_t *x, long n, int32_t *y, int exclusive,
                                                       int32_t *row_totals)
{
    constexpr int TILE = NT * kScanItems;
    __shared__ int wsum[2][NT / 64];
    x += (long)blockIdx.x * n;
    y += (long)blockIdx.x * n;
    int carry = 0;
    long b = 0;
    i32x4 q0[kScanGroups], q1[kScanGroups];
    auto step = [&](i32x4 (&q)[kScanGroups], int *ws) {
        int before[kScanGroups];
        const int total = scan_before<NT>(q, before, ws);
        scan_store<NT, false>(y + b, n - b, q, before, carry, exclusive != 0);
        carry += total;
        b += TILE;
    };
    scan_load<NT>(x, n, q0);
    while (true) {
        if (b + TILE >= n) {
            step(q0, wsum[0]);
            break;
        }
        scan_load<NT>(x + b + TILE, n - b - TILE, q1);
        step(q0, wsum[0]);
        if (b + TILE >= n) {
            step(q1, wsum[1]);
            break;
        }
        scan_load<NT>(x + b + TILE, n - b - TILE, q0);
        step(q1, wsum[1]);
    }
    if (row_totals && threadIdx.x == 0) row_totals[blockIdx.x] = carry;
}

// The stages across work-groups (a few long rows), two launches bound by HBM:
// 2^26 values 123.5 us, 4.35 TB/s of the 8 bytes per value it cannot do
// without (three launches over tiles transposed through LDS: 128.0); 4 rows of
// 16000001, unaligned, 181.7 -> 119.1 us; up to 4 million values, where the
// launches count, 14.5 -> 11.9.  Up-sweep: the sum of every chunk of `chunk`
// values, whole tiles (grid: chunks x rows).
__global__ __launch_bounds__(kScanThreads) void scan_upsweep_kernel(const int32_t *x, long n, long chunk, int32_t *sums)
{
    __shared__ int wsum[kScanThreads / 64];
    const long c0 = (long)blockIdx.x * chunk;
    const long len = n - c0 < chunk ? n - c0 : chunk;
    x += (long)blockIdx.y * n + c0;
    int s = 0;
#pragma unroll 2
    for (long b = 0; b < len; b += kScanTile) {
        i32x4 q[kScanGroups];
        scan_load<kScanThreads>(x + b, len - b, q);
#pragma unroll
        for (int j = 0; j < kScanGroups; ++j) s += q[j][0] + q[j][1] + q[j][2] + q[j][3];
    }
    int total;
    wg_scan_incl<kScanThreads>(s, wsum, &total);
    if (threadIdx.x == 0) sums[(long)blockIdx.y * gridDim.x + blockIdx.x] = total;
}

// Scan and down-sweep: each work-group adds up the sums of the chunks before
// its own (at most kScanChunks, from L2), then scans its chunk's tiles, the
// last first, each preceded by what the chunk's end is less the tile's own
// sum.  The up-sweep has just read the chunks in order, so their last tiles
// are still in the caches; y is stored non-temporally so that it does not
// evict them.
__global__ __launch_bounds__(kScanThreads) void scan_downsweep_kernel(const int32_t *x, long n, long chunk,
                                                                      const int32_t *sums, int32_t *y, int exclusive)
{
    __shared__ int wsum[2][kScanThreads / 64];
    const long c0 = (long)blockIdx.x * chunk;
    const long len = n - c0 < chunk ? n - c0 : chunk;
    x += (long)blockIdx.y * n + c0;
    y += (long)blockIdx.y * n + c0;
    i32x4 q0[kScanGroups], q1[kScanGroups];
    long b = (len - 1) / kScanTile * kScanTile;
    scan_load<kScanThreads>(x + b, len - b, q0);
    sums += (long)blockIdx.y * gridDim.x;
    int s = 0, end;
    for (unsigned i = threadIdx.x; i <= blockIdx.x; i += kScanThreads) s += sums[i];
    wg_scan_incl<kScanThreads>(s, wsum[0], &end);
    auto step = [&](i32x4 (&q)[kScanGroups], int *ws) {
        int before[kScanGroups];
        end -= scan_before<kScanThreads>(q, before, ws);
        scan_store<kScanThreads, true>(y + b, len - b, q, before, end, exclusive != 0);
        b -= kScanTile;
    };
    while (true) {
        if (b == 0) {
            step(q0, wsum[0]);
            break;
        }
        scan_load<kScanThreads>(x + b - kScanTile, kScanTile, q1);
        step(q0, wsum[0]);
        if (b == 0) {
            step(q1, wsum[1]);
            break;
        }
        scan_load<kScanThreads>(x + b - kScanTile, kScanTile, q0);
        step(q1, wsum[1]);
    }
}

// Rows this long or more, fewer than this many of them, go across work-groups.
constexpr long kScanLongRow = 4L * kScanTile;
constexpr int kScanFewRows = 64;
// Work-groups of a launch over long rows: four per CU, 16 wavefronts, so that
// all run at once (2^26 values 123.5 us, 11234567 20.9; with 4096 125.2, 22.6).
constexpr int kScanChunks = 1024;

bool scan_across(int rows, long n) { return rows < kScanFewRows && n > kScanLongRow; }

// Values per chunk: whole tiles, at most about kScanChunks chunks over all rows.
long scan_chunk(int rows, long n)
{
    const long tiles = (n + kScanTile - 1) / kScanTile;
    return (tiles * rows + kScanChunks - 1) / kScanChunks * kScanTile;
}

long scan_ws_bytes(int rows, long n)
{
    if (!scan_across(rows, n)) return 0;
    const long chunk = scan_chunk(rows, n);
    return ((long)rows * ((n + chunk - 1) / chunk) * 4 + 255) / 256 * 256;
}

hipError_t launch_scan(const int32_t *x, int rows, long n, int32_t *y, bool exclusive, void *ws, hipStream_t st)
{
    if (!scan_across(rows, n)) {
        if (rows < 256 && n > kScanTile)
            launch_kernel(scan_rows_kernel<kScanWide>, dim3((unsigned)rows), dim3(kScanWide), 0, st, x, n, y,
                          exclusive ? 1 : 0, (int32_t *)nullptr);
        else
            launch_kernel(scan_rows_kernel<kScanThreads>, dim3((unsigned)rows), dim3(kScanThreads), 0, st, x, n, y,
                          exclusive ? 1 : 0, (int32_t *)nullptr);
        return hipGetLastError();
    }
    const long chunk = scan_chunk(rows, n);
    const dim3 grid((unsigned)((n + chunk - 1) / chunk), (unsigned)rows);
    int32_t *sums = static_cast<int32_t *>(ws);
    launch_kernel(scan_upsweep_kernel, grid, dim3(kScanThreads), 0, st, x, n, chunk, sums);
    launch_kernel(scan_downsweep_kernel, grid, dim3(kScanThreads), 0, st, x, n, chunk,
                  static_cast<const int32_t *>(sums), y, exclusive ? 1 : 0);
    return hipGetLastError();
}

// ----------------------------------------------------------------- argsort

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;   // 2048: merge output per work-group

// Order-preserving image of an fp32 key: ascending (or, descending != 0,
// descending) float order becomes ascending unsigned order; -0 maps with +0,
// and every NaN to the largest value, so NaNs come last in either order.
__device__ __forceinline__ uint32_t key_bits(float f, int descending)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) == 0) u = 0;
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return 0xffffffffu;
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return descending ? ~u : u;   // never 0xffffffff for a number
}

// Offset s of the segment table, clamped to [0, limit].
__device__ __forceinline__ long seg_at(const int32_t *off, int s, long limit)
{
    const long o = off[s];
    return o < 0 ? 0 : (o > limit ? limit : o);
}

// Segment of position i: the last s < S with offsets[s] <= i (binary search;
// any offsets give some s in [0, S-1]).
__device__ int find_segment(const int32_t *off, int S, long n, long i)
{
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg_at(off, mid, n) <= i) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The same search by a whole wavefront for a uniform i: 64 probes per round,
// so a table of S offsets costs about log64(S) dependent round trips.
__device__ int find_segment_wave(const int32_t *off, int S, long n, long i)
{
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = S - 1;   // the answer is in [lo, hi]
    while (lo < hi) {
        const int span = hi - lo;                   // probes lo + 1 .. hi
        const int step = (span + 63) / 64;
        const int m = lo + 1 + lane * step;
        const bool f = m <= hi && seg_at(off, m, n) <= i;   // true ... true false ... false
        const uint64_t bal = __ballot(f);
        if (!bal) {
            hi = lo;                                // no probe at or below i: the answer is lo
        } else {
            const int l = 63 - __clzll((long long)bal);   // last true probe
            const int ml = lo + 1 + l * step;
            lo = ml;
            const int next = ml + step;             // the first false probe (if any) bounds hi
            hi = next - 1 < hi ? next - 1 : hi;
        }
    }
    return lo;
}

// The lanes of the wavefront whose 8-bit digit equals this lane's, as two
// 32-bit halves: one ballot per bit.
__device__ __forceinline__ uint64_t match_digit(uint32_t d)
{
    uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);   // all ones where the bit is set
        asm("" : "+v"(m));                                            // (the comparison reads m, not d again)
        const uint64_t bal = __ballot(m != 0);
        lo &= ~((uint32_t)bal ^ m);
        hi &= ~((uint32_t)(bal >> 32) ^ m);
    }
    return ((uint64_t)hi << 32) | lo;
}

// The wavefront's lanes meet: what each has read from or written to LDS before
// comes before what any of them does after.  The hardware runs them in step;
// this holds the compiler to it (no instruction).
__device__ __forceinline__ void wave_step()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int lanes_before(uint64_t set)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(set >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)set, 0));
}

// One stable radix pass in LDS over the digit (x >> shift) & 255 of THREADS *
// ITEMS words, each with a 16-bit index v: wavefront w holds 64 * ITEMS
// consecutive ones, lane l of round r word 64 r + l.  On return x and v hold
// the words in their new order.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void lds_radix_pass(uint32_t (&x)[ITEMS], int (&v)[ITEMS], int shift, uint32_t *sk,
                                               uint16_t *sv, uint16_t (*cnt)[256], int *wsum)
{
    constexpr int WAVES = THREADS / 64;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int w0 = wid * 64 * ITEMS + lane;
    for (int i = t; i < WAVES * 128; i += THREADS) reinterpret_cast<uint32_t *>(&cnt[0][0])[i] = 0;
    __syncthreads();
    int rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = (x[r] >> shift) & 255;
        const uint64_t same = match_digit(d);
        const int before = lanes_before(same);
        const int c = cnt[wid][d];
        rank[r] = c + before;
        wave_step();                           // every lane has read the counters
        if (before == 0) cnt[wid][d] = (uint16_t)(c + __popcll(same));
        wave_step();                           // and the next round reads them written
    }
    __syncthreads();
    int mine = 0, total;
    if (t < 256)
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mine += cnt[w][t];
    int at = wg_scan_incl<THREADS>(mine, wsum, &total) - mine;
    if (t < 256) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int c = cnt[w][t];
            cnt[w][t] = (uint16_t)at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int slot = cnt[wid][(x[r] >> shift) & 255] + rank[r];
        sk[slot] = x[r];
        sv[slot] = (uint16_t)v[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        x[r] = sk[w0 + 64 * r];
        v[r] = sv[w0 + 64 * r];
    }
}

// Equal blocks sorted locally: one work-group sorts a block of consecutive
// positions in LDS by (segment, key, position), as stable radix passes over
// 8-bit digits, least significant first: four over the key bits and then, if
// the block holds more than one segment, one or two over the segments.  A
// pass ranks every element within its wavefront (each holds 64 * ITEMS
// consecutive elements, lane l of round r element 64 r + l): lanes with the
// same digit are matched by ballots, earlier rounds counted per wavefront and
// digit.  Bound by the ballots' VALU work, 5 instructions per bit and round,
// and in a single block by the passes' chains of barriers (7 us a pass):
// 2^22 elements take 68 us, one block of 2048 elements 9 us (a bitonic network
// in 64-bit words: 90 and 21 us).  Lanes finding each other through a table in LDS (an atomic or, a
// read and a write per round instead of 50 VALU instructions): 84 and 40 us.
//   Segments that lie within the block are finished: their answers go to out.
// The elements of the one that began before the block (`head`) and of the
// one that goes on after it (`tail`) leave as (key bits, position) for the
// merge passes, with both segments' extents in ext[block].
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;

struct TileArgs {
    const float *keys;
    const int32_t *off;
    int S;
    long n;
    int descending;
    uint32_t *K;      // key bits and positions of elements of unfinished segments
    int32_t *V;
    int4 *ext;        // per block: [start, end) of its head and tail segments (empty: none)
    int32_t *out;
};

// ITEMS per thread: blocks of 8192 positions (16; 70 KB of LDS, two
// work-groups per CU), 4096 or 2048.  Two work-groups leave a thread 128 VGPRs:
// with 16 items the compiler spills 20 of them (84 bytes of scratch per lane).
template <int ITEMS>
__global__ __launch_bounds__(kTileThreads, 4) void segsort_tile_kernel(TileArgs a)
{
    constexpr int BLOCK = kTileThreads * ITEMS;
    __shared__ uint32_t sk[BLOCK];
    __shared__ uint16_t sv[BLOCK];
    __shared__ uint16_t first[BLOCK];    // first position in the block of its q-th segment
    __shared__ uint16_t cnt[kTileWaves][256];
    __shared__ int wsum[kTileWaves];
    __shared__ int s_lo, s_num, s_head, s_tail;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const long base = (long)blockIdx.x * BLOCK;
    const long end = seg_at(a.off, a.S, a.n);          // positions from here on belong to no segment
    const long lim = base + BLOCK < end ? base + BLOCK : end;
    const int w0 = wid * 64 * ITEMS + lane;
    uint32_t k[ITEMS];
    int v[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        v[r] = w0 + 64 * r;
        const long g = base + v[r];
        k[r] = g < end ? key_bits(a.keys[g], a.descending) : 0xffffffffu;
    }
    if (wid == 0) {
        int lo = 0, num = 0;
        long h0 = base, h1 = base, t0 = lim, t1 = lim;
        if (base < lim) {
            lo = find_segment_wave(a.off, a.S, a.n, base);
            const int hi = find_segment_wave(a.off, a.S, a.n, lim - 1);
            num = hi - lo + 1;
            const long s0 = seg_at(a.off, lo, a.n), s1 = seg_at(a.off, hi, a.n);
            const long e0 = seg_at(a.off, lo + 1, a.n), e1 = seg_at(a.off, hi + 1, a.n);
            if (s0 < base || (num == 1 && e0 > lim)) {
                h0 = s0;
                h1 = e0;
            }
            if (num > 1 && e1 > lim) {
                t0 = s1;
                t1 = e1;
            }
        }
        if (lane == 0) {
            s_lo = lo;
            s_num = num;
            // slots [0, s_head) and [s_tail, ..) are the head's and the tail's
            const long hh = h1 > h0 ? h1 : base;
            s_head = (int)((hh < lim ? hh : lim) - base);
            const long tt = t1 > t0 ? t0 : lim;
            s_tail = (int)((tt > base ? tt : base) - base);
            if (a.ext) a.ext[blockIdx.x] = make_int4((int)h0, (int)h1, (int)t0, (int)t1);
        }
        if (num > 1 && num <= BLOCK)
            for (int q = lane; q < num; q += 64) {
                const long f = seg_at(a.off, lo + q, a.n) - base;
                first[q] = (uint16_t)(f < 0 ? 0 : (f < BLOCK ? f : BLOCK - 1));
            }
    }

    __syncthreads();
    const int num = s_num, lo = s_lo;
    int bits = 0;                            // of a segment's order among the block's
    if (num > BLOCK) bits = 13;
    else while ((1 << bits) < num) ++bits;
    const int passes = 4 + (bits + 7) / 8;
    // One copy of the pass's code: a block runs it from a cold instruction cache.
#pragma clang loop unroll(disable)
    for (int p = 0; p < passes; ++p) {
        const int shift = p < 4 ? 8 * p : 8 * (p - 4);
        if (p == 4) {
            // the words become (segment's first position in the block << 16 | its order)
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) k[r] = 0;
            if (num <= BLOCK) {
                for (int len = num; len > 1;) {         // the last q with first[q] <= v, side by side
                    const int half = len >> 1;
#pragma unroll
                    for (int r = 0; r < ITEMS; ++r)
                        if (first[k[r] + half] <= v[r]) k[r] += half;
                    len -= half;
                }
#pragma unroll
                for (int r = 0; r < ITEMS; ++r) k[r] |= (uint32_t)first[k[r]] << 16;
            } else {
                // more segments than positions (most of them empty): a
                // segment's first position stands for its order
                for (int r = 0; r < ITEMS; ++r) {
                    const long g = base + v[r] < lim ? base + v[r] : lim - 1;
                    const long f = seg_at(a.off, find_segment(a.off, a.S, a.n, g), a.n) - base;
                    k[r] = (uint32_t)(f < 0 ? 0 : f) * 0x10001u;
                }
            }
        }
        lds_radix_pass<kTileThreads, ITEMS>(k, v, shift, sk, sv, cnt, wsum);
    }
    // the words are key bits if the block holds one segment
    const long s0 = num == 1 ? seg_at(a.off, lo, a.n) : 0;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int slot = w0 + 64 * r;
        const long g = base + slot;
        if (g >= a.n) break;
        const long pos = base + v[r];
        if (g >= end) {
            a.out[g] = -1;
        } else if (slot < s_head || slot >= s_tail) {
            a.K[g] = num == 1 ? k[r] : key_bits(a.keys[pos], a.descending);
            a.V[g] = (int32_t)pos;
        } else {
            a.out[g] = num == 1 ? (int32_t)(pos - s0) : v[r] - (int32_t)(k[r] >> 16);
        }
    }
}

// One merge pass over the segments that span blocks.  A segment's part in
// each of its blocks is a sorted run; pass j merges its runs of 2^j blocks,
// counted from the segment's first block, pairwise, so a segment over m blocks
// is finished after ceil(log2 m) passes wherever it lies, and segments that
// are finished are not touched: a pass moves only what is still unsorted.
// 2^22 keys in 4096 segments take 27 us in all nine passes (the first, which
// finishes all of them, 14; each of the others, whose work-groups read ext and
// leave, 1.6), where moving every element in every pass took 40 us a pass.
// Work-group (w, y) writes outputs [w*C, w*C + C) (C = kSortTile) as far as
// they belong to the head (y = 0) or tail (1) segment of its block: the first
// two wavefronts find where the chunk's ends cross the merge path (64 probes
// per round), the elements between are staged in LDS, every thread finds its
// own crossing by bisection and merges kSortItems outputs.  Equal keys: the
// first run's come first (its positions are lower).  The pass that completes
// a segment writes its answers.
struct MergeArgs {
    const uint32_t *Ki;
    const int32_t *Vi;
    uint32_t *Ko;
    int32_t *Vo;
    const int4 *ext;
    int32_t *out;
    long n;
    int log_block;    // positions per block: 2^log_block
    int log_run;      // the pass's runs: 2^log_run blocks
};

__global__ __launch_bounds__(kSortThreads) void segsort_merge_kernel(MergeArgs a)
{
    __shared__ uint32_t sk[kSortTile];
    __shared__ int32_t sv[kSortTile];
    __shared__ long split[2];
    const long w0 = (long)blockIdx.x * kSortTile;
    const int4 e = a.ext[w0 >> a.log_block];
    const long sa = blockIdx.y ? e.z : e.x, sb = blockIdx.y ? e.w : e.y;   // the segment
    if (sb <= sa) return;
    const long ta = sa >> a.log_block;                                        // its first block
    const long runs = (((sb - 1) >> a.log_block) - ta) >> a.log_run;            // runs of this pass, less one
    if (runs == 0) return;                                                 // finished before
    const long c0 = sa > w0 ? sa : w0;
    const long w1 = w0 + kSortTile < a.n ? w0 + kSortTile : a.n;
    const long c1 = sb < w1 ? sb : w1;
    if (c1 <= c0) return;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const long pair = ((w0 >> a.log_block) - ta) >> (a.log_run + 1);
    const long p0 = (ta + (pair << (a.log_run + 1))) << a.log_block;
    const long L = 1L << (a.log_block + a.log_run);
    const long pm = p0 + L, p1 = pm + L;
    const long A0 = sa > p0 ? sa : p0, A1 = sb < pm ? sb : pm;             // the first run
    const long B0 = pm, B1 = sb < p1 ? sb : p1;                            // the second
    const long na = A1 - A0, nb = B1 > B0 ? B1 - B0 : 0;
    const long base = A0;
    const bool last = runs == 1;
    const uint32_t *KA = a.Ki + A0, *KB = a.Ki + B0;
    const int32_t *VA = a.Vi + A0, *VB = a.Vi + B0;
    const long d0 = c0 - base, d1 = c1 - base;
    const int cnt = (int)(c1 - c0);
    if (wid < 2) {
        const long d = wid ? d1 : d0;
        long lo = d - nb > 0 ? d - nb : 0, hi = d < na ? d : na;
        // f(m) = "A[m] is not among the first d outputs" = B[d-1-m] < A[m]:
        // false below the crossing, true from it on
        while (hi > lo) {
            const long span = hi - lo;
            const long step = (span + 63) / 64;
            const long m = lo + (long)lane * step;
            bool f = false;
            if (m < hi) f = KB[d - 1 - m] < KA[m];
            const uint64_t bal = __ballot(f);
            if (bal) {
                const int l = __ffsll((unsigned long long)bal) - 1;
                const long ml = lo + (long)l * step;
                lo = l ? lo + (long)(l - 1) * step + 1 : lo;
                hi = ml;
            } else {
                const long past = (span - 1) / step < 63 ? (span - 1) / step : 63;
                lo = lo + past * step + 1;
            }
        }
        if (lane == 0) split[wid] = lo;
    }
    __syncthreads();
    const long a0 = split[0], a1 = split[1] > split[0] ? split[1] : split[0];
    const int ca = (int)(a1 - a0 < cnt ? a1 - a0 : cnt);   // crossings are monotone: 0 <= ca <= cnt
    const long b0 = d0 - a0;
    for (int i = t; i < cnt; i += kSortThreads) {
        sk[i] = i < ca ? KA[a0 + i] : KB[b0 + (i - ca)];
        sv[i] = i < ca ? VA[a0 + i] : VB[b0 + (i - ca)];
    }
    __syncthreads();
    const int cb = cnt - ca;
    const int dt = t * kSortItems < cnt ? t * kSortItems : cnt;
    int lo = dt - cb > 0 ? dt - cb : 0, hi = dt < ca ? dt : ca;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sk[ca + dt - 1 - mid] < sk[mid]) hi = mid;
        else lo = mid + 1;
    }
    int ia = lo, ib = dt - lo;
    uint32_t rk[kSortItems];
    int32_t rv[kSortItems];
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        rk[k] = 0;
        rv[k] = 0;
        if (dt + k >= cnt) continue;
        const bool take_a = ib >= cb || (ia < ca && sk[ia] <= sk[ca + ib]);
        const int src = take_a ? ia++ : ca + ib++;
        rk[k] = sk[src];
        rv[k] = sv[src];
    }
    __syncthreads();   // every thread has read its inputs
#pragma unroll
    for (int k = 0; k < kSortItems; ++k)
        if (dt + k < cnt) {
            sk[dt + k] = rk[k];
            sv[dt + k] = rv[k];
        }
    __syncthreads();
    for (int i = t; i < cnt; i += kSortThreads) {
        if (last) a.out[c0 + i] = (int32_t)(sv[i] - sa);
        else {
            a.Ko[c0 + i] = sk[i];
            a.Vo[c0 + i] = sv[i];
        }
    }
}

// Long segments: least-significant-digit radix passes over the whole array,
// four over the key bits and, with more than one segment (at most 256), one
// over the segment.  Each reads and writes 8 bytes per element once, whatever
// the segments' lengths, where the merge passes move every element of a
// segment log2(its blocks) times.  A pass is three launches: digit counts of
// every tile (radix_count_kernel), their exclusive scan digit by digit
// (scan_rows_kernel, one row of tile counts per digit), and the scatter
// (radix_scatter_kernel, 20 us for 2^22 elements, VALU-bound by the ballots as
// the block sort is).  Every step is stable.
constexpr int kRadixThreads = 512;
constexpr int kRadixItems = 16;
constexpr int kRadixTile = kRadixThreads * kRadixItems;   // 8192: two work-groups per CU in the scatter
constexpr int kRadixBins = 256;
constexpr int kRadixWaves = kRadixThreads / 64;

struct RadixArgs {
    const float *keys;        // first pass: the keys as given, positions implied
    const uint32_t *Ki;       // other passes: key bits, or segments in the segment passes
    const int32_t *Vi;        // positions
    uint32_t *Ko;
    int32_t *Vo;
    int32_t *out;             // last pass: the answers
    const int32_t *off;
    int32_t *counts;          // [256][tiles]
    const int32_t *totals;    // [256]
    long n;
    int S, tiles, descending;
    int shift;                // the digit: 8 bits from here
    int to_segment;           // write the element's segment in place of its key
};

// Key bits of element i of the first pass: positions past the segments sort
// after everything (NaNs, which share their bits, come earlier in the array).
__device__ __forceinline__ uint32_t radix_key(const RadixArgs &a, long i, long end)
{
    return a.keys ? (i < end ? key_bits(a.keys[i], a.descending) : 0xffffffffu) : a.Ki[i];
}

__global__ __launch_bounds__(kRadixThreads) void radix_count_kernel(RadixArgs a)
{
    __shared__ int cnt[kRadixWaves][kRadixBins];
    const int t = threadIdx.x, wid = t >> 6;
    for (int i = t; i < kRadixWaves * kRadixBins; i += kRadixThreads) (&cnt[0][0])[i] = 0;
    const long base = (long)blockIdx.x * kRadixTile;
    const long end = a.keys ? seg_at(a.off, a.S, a.n) : 0;
    constexpr uint32_t mask = kRadixBins - 1;
    uint32_t k[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
        const long i = base + r * kRadixThreads + t;
        k[r] = i < a.n ? radix_key(a, i, end) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r)
        if (base + r * kRadixThreads + t < a.n) atomicAdd(&cnt[wid][(k[r] >> a.shift) & mask], 1);
    __syncthreads();
    if (t < kRadixBins) {
        int s = 0;
#pragma unroll
        for (int w = 0; w < kRadixWaves; ++w) s += cnt[w][t];
        a.counts[(long)t * a.tiles + blockIdx.x] = s;
    }
}

// One tile's elements to their places.  Wavefront w holds 1024 consecutive
// elements, lane l of round r element 64 r + l: the elements of one digit
// before it in its round are counted by matching the digit's bits across the
// lanes, those in earlier rounds in a counter per wavefront and digit.  The
// tile is then gathered digit by digit in LDS, so that the elements of a digit
// leave as one run.
__global__ __launch_bounds__(kRadixThreads, 4) void radix_scatter_kernel(RadixArgs a)
{
    __shared__ uint32_t skv[2 * kRadixTile];
    uint32_t *sk = skv;
    int32_t *sv = reinterpret_cast<int32_t *>(skv) + kRadixTile;
    __shared__ int cnt[kRadixWaves][kRadixBins];
    __shared__ int gbase[kRadixBins];
    __shared__ int wsum[kRadixWaves];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const long base = (long)blockIdx.x * kRadixTile;
    const long end = seg_at(a.off, a.S, a.n);
    const long w0 = base + wid * 64 * kRadixItems;
    constexpr uint32_t mask = kRadixBins - 1;
    uint32_t k[kRadixItems];
    int v[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
        const long i = w0 + r * 64 + lane;
        k[r] = i < a.n ? radix_key(a, i, end) : 0;
        v[r] = i < a.n ? (a.keys ? (int)i : a.Vi[i]) : 0;
    }
    // where the tile's elements of digit t go
    int place = 0;
    if (t < kRadixBins) place = a.counts[(long)t * a.tiles + blockIdx.x];
    int total;
    {
        const int tot = t < kRadixBins ? a.totals[t] : 0;
        place += wg_scan_incl<kRadixThreads>(tot, wsum, &total) - tot;
    }
    for (int i = t; i < kRadixWaves * kRadixBins; i += kRadixThreads) (&cnt[0][0])[i] = 0;
    // segments of the elements' positions: the last with offset <= v, the
    // searches side by side
    uint32_t seg[kRadixItems];
    if (a.to_segment) {
        if (t < a.S) sv[t] = (int32_t)seg_at(a.off, t, a.n);     // S <= 256
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRadixItems; ++r) seg[r] = 0;
        for (int len = a.S; len > 1;) {
            const int half = len >> 1;
#pragma unroll
            for (int r = 0; r < kRadixItems; ++r)
                if (sv[seg[r] + half] <= v[r]) seg[r] += half;
            len -= half;
        }
    }
    __syncthreads();
    int rank[kRadixItems];
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
        const bool ok = w0 + r * 64 + lane < a.n;
        const uint32_t d = (k[r] >> a.shift) & mask;
        const uint64_t same = __ballot(ok) & match_digit(d);
        const int before = lanes_before(same);
        const int c = cnt[wid][d];
        rank[r] = c + before;
        wave_step();                           // as in lds_radix_pass
        if (ok && before == 0) cnt[wid][d] = c + __popcll(same);
        wave_step();
    }
    __syncthreads();
    // first local slot of every digit, and of every wavefront's share of it
    int mine = 0;
    if (t < kRadixBins) {
#pragma unroll
        for (int w = 0; w < kRadixWaves; ++w) {
            const int c = cnt[w][t];
            cnt[w][t] = mine;
            mine += c;
        }
    }
    const int start = wg_scan_incl<kRadixThreads>(mine, wsum, &total) - mine;
    if (t < kRadixBins) {
        gbase[t] = place - start;
#pragma unroll
        for (int w = 0; w < kRadixWaves; ++w) cnt[w][t] += start;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRadixItems; ++r) {
        if (w0 + r * 64 + lane >= a.n) continue;
        const uint32_t d = (k[r] >> a.shift) & mask;
        const int slot = cnt[wid][d] + rank[r];
        // the segment travels with the digit that places it
        sk[slot] = a.to_segment ? seg[r] | (d << 24) : k[r];
        sv[slot] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const int slot = i * kRadixThreads + t;
        if (base + slot >= a.n) break;
        const uint32_t key = sk[slot];
        const uint32_t d = a.to_segment ? key >> 24 : (key >> a.shift) & mask;
        const long dst = gbase[d] + slot;
        const int pos = sv[slot];
        if (a.out) {
            const uint32_t s = a.S == 1 ? 0 : key;
            a.out[dst] = pos < end ? (int32_t)(pos - seg_at(a.off, (int)s, a.n)) : -1;
        } else {
            a.Ko[dst] = a.to_segment ? key & 0xffffffu : key;
            a.Vo[dst] = pos;
        }
    }
}

long align256(long b) { return (b + 255) / 256 * 256; }

long argsort_ws_bytes(long n) { return n <= kSortTile ? 0 : 2 * align256(n * 8) + 2 * align256(n * 4); }

// Where the radix passes win over block sorts and merges (measured, us: one
// segment of 500 thousand keys 102 and 101, of 1 million 137 and 110, of 2^22
// 295 and 147; 2^22 keys in 30 segments 212 and 191, in 100 175 and 193; 2
// million in 6 157 and 143, in 20 even; 1 million in 10 123 and 140).
bool radix_pays(long n, int S)
{
    return S == 1 ? n >= 500000 : n >= 1500000 && S <= kRadixBins && n / S >= 100000;
}

hipError_t launch_radix(const float *keys, const int32_t *off, int S, long n, int descending, int32_t *out, void *ws,
                        hipStream_t st)
{
    // 16 n bytes of keys and positions, n/8 of counts: within argsort_ws_bytes
    char *p = static_cast<char *>(ws);
    uint32_t *K[2];
    int32_t *V[2];
    for (int i = 0; i < 2; ++i) {
        K[i] = reinterpret_cast<uint32_t *>(p);
        V[i] = reinterpret_cast<int32_t *>(p + align256(n * 4));
        p += 2 * align256(n * 4);
    }
    RadixArgs a{};
    a.off = off;
    a.n = n;
    a.S = S;
    a.tiles = (int)((n + kRadixTile - 1) / kRadixTile);
    a.descending = descending;
    int32_t *totals = reinterpret_cast<int32_t *>(p);
    a.totals = totals;
    a.counts = totals + kRadixBins;
    const int passes = S > 1 ? 5 : 4;
    for (int i = 0; i < passes; ++i) {
        a.keys = i == 0 ? keys : nullptr;
        a.Ki = K[(i & 1) ^ 1];
        a.Vi = V[(i & 1) ^ 1];
        a.Ko = K[i & 1];
        a.Vo = V[i & 1];
        a.out = i == passes - 1 ? out : nullptr;
        a.to_segment = i == 3 && S > 1;
        a.shift = i < 4 ? 8 * i : 0;
        launch_kernel(radix_count_kernel, dim3((unsigned)a.tiles), dim3(kRadixThreads), 0, st, a);
        launch_kernel(scan_rows_kernel<kScanThreads>, dim3(kRadixBins), dim3(kScanThreads), 0, st,
                      a.counts, (long)a.tiles, a.counts, 1, totals);
        launch_kernel(radix_scatter_kernel, dim3((unsigned)a.tiles), dim3(kRadixThreads), 0, st, a);
    }
    return hipGetLastError();
}

// Elements per thread of the block sorts.  Small blocks have the shorter chain
// of rounds and put more CUs to work, large ones leave fewer merge passes
// (measured with 4 / 8 / 16, us: 1500 keys in 6 segments 13 / 19 / 34; 4096 in
// one 19 / 16 / 28; 200 thousand in 300 33 / 39 / 55, in 3 72 / 70 / 78; 1
// million in 1000 52 / 53 / 62; 2^22 in 4096 124 / 117 / 96).
int sort_items(long n, int S)
{
    if (n > 1500000) return 16;
    return n > 2048 && (n <= 4096 || n / S >= 8192) ? 8 : 4;
}

// The whole sort: local block sorts, then, for segments that span blocks,
// merge passes over runs of 1, 2, 4, ... blocks, ping-ponging between two
// key/position buffers.
hipError_t launch_segsort(const float *keys, const int32_t *off, int S, long n, int descending, int32_t *out,
                          void *ws, hipStream_t st)
{
    if (radix_pays(n, S)) return launch_radix(keys, off, S, n, descending, out, ws, st);
    const int items = sort_items(n, S);
    const int block = kTileThreads * items;
    const unsigned blocks = (unsigned)((n + block - 1) / block);
    TileArgs ta{keys, off, S, n, descending, nullptr, nullptr, nullptr, out};
    auto launch_blocks = [&] {
        if (items == 4) launch_kernel(segsort_tile_kernel<4>, dim3(blocks), dim3(kTileThreads), 0, st, ta);
        else if (items == 8) launch_kernel(segsort_tile_kernel<8>, dim3(blocks), dim3(kTileThreads), 0, st, ta);
        else launch_kernel(segsort_tile_kernel<16>, dim3(blocks), dim3(kTileThreads), 0, st, ta);
    };
    if (blocks == 1) {
        launch_blocks();
        return hipGetLastError();
    }
    char *p = static_cast<char *>(ws);
    uint32_t *K[2];
    int32_t *V[2];
    for (int i = 0; i < 2; ++i) {
        K[i] = reinterpret_cast<uint32_t *>(p);
        V[i] = reinterpret_cast<int32_t *>(p + align256(n * 4));
        p += 2 * align256(n * 4);
    }
    ta.K = K[0];
    ta.V = V[0];
    ta.ext = reinterpret_cast<int4 *>(p);     // 16 bytes per block: within argsort_ws_bytes
    launch_blocks();
    MergeArgs m{};
    while ((1 << m.log_block) < block) ++m.log_block;
    m.ext = ta.ext;
    m.out = out;
    m.n = n;
    int cur = 0;
    for (int j = 0; (1L << j) < (long)blocks; ++j, cur ^= 1) {
        m.Ki = K[cur];
        m.Vi = V[cur];
        m.Ko = K[cur ^ 1];
        m.Vo = V[cur ^ 1];
        m.log_run = j;
        launch_kernel(segsort_merge_kernel, dim3((unsigned)((n + kSortTile - 1) / kSortTile), 2), dim3(kSortThreads),
                      0, st, m);
    }
    return hipGetLastError();
}

// ----------------------------------------------------------------- box_nms

constexpr int kNmsMax = MIVISION_NMS_MAX_CANDIDATES;

constexpr int kNmsChunk = 1024;       // input rows per work-group of the collecting kernel

struct NmsArgs {
    const float *data;
    float *out;
    int B, N, width;
    int cand_max;      // candidates compared per image at most: min(topk, N), or N
    int capw;          // 64-bit mask words per candidate row: ceil(cand_max / 64)
    int mrows;         // mask rows per image: 64 * capw
    float overlap, valid;
    int id_index, score_index, coord_start, force;
    int chunks;        // per image
    int slice, slices; // chunks per slice and slices per image of the first of two picks
                       // (one pick: 1, chunks)
    uint32_t *ckey;           // [B][N]: each chunk's candidates from its first row's slot on: key bits
    int32_t *corig;           // and input rows, in row order
    int32_t *ccount;          // [B][chunks] candidates of each chunk
    int32_t *count;           // [B] compared candidates
    float4 *cbox;             // [B][mrows] box of the candidate of rank r
    float *ccls;              // [B][mrows] its class
    int32_t *crow;            // [B][mrows] its input row
    uint64_t *mask;           // [B][mrows][capw]
};

// First pass over the rows, one work-group per chunk of 1024: every value of
// out is set invalid (Sec. 4.3: no per-row decision), and the chunk's
// candidates leave as (descending key bits, row), in row order.  No slot
// depends on another chunk, so no scan over the image is needed first (a
// three-stage scan of the candidate flags, one work-group per image, took 12
// us for 24564 rows, and a compaction launch 3).
__global__ __launch_bounds__(256) void nms_collect_kernel(NmsArgs a)
{
    __shared__ int found[16];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int b = blockIdx.x / a.chunks;
    const int chunk = blockIdx.x - b * a.chunks;
    const int r0 = chunk * kNmsChunk;
    const int rows = a.N - r0 < kNmsChunk ? a.N - r0 : kNmsChunk;
    const long first = (long)b * a.N + r0;
    float s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = t + 256 * j;
        s[j] = r < rows ? a.data[(first + r) * a.width + a.score_index] : 0.f;
    }
    float *o = a.out + first * a.width;
    const int vals = rows * a.width;
    const int lead = min(vals, (int)((16 - ((uintptr_t)o & 15)) & 15) / 4);   // up to 16-byte alignment
    const int quads = (vals - lead) / 4;
    for (int i = t; i < quads; i += 256) reinterpret_cast<float4 *>(o + lead)[i] = make_float4(-1.f, -1.f, -1.f, -1.f);
    if (t < lead) o[t] = -1.f;
    if (t < vals - lead - 4 * quads) o[lead + 4 * quads + t] = -1.f;

    uint64_t bal[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bal[j] = __ballot(t + 256 * j < rows && s[j] > a.valid);
        if (lane == 0) found[4 * j + wid] = __popcll(bal[j]);
    }
    __syncthreads();
    int before[4], total = 0;               // candidates in earlier rounds and wavefronts
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if ((i & 3) == wid) before[i >> 2] = total;
        total += found[i];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (bal[j] >> lane & 1) {
            const long slot = first + before[j] + lanes_before(bal[j]);
            a.ckey[slot] = key_bits(s[j], 1);
            a.corig[slot] = r0 + t + 256 * j;
        }
    if (t == 0) a.ccount[blockIdx.x] = total;
}

__device__ __forceinline__ float4 load_box(const NmsArgs &a, int b, int i, float *cls)
{
    const float *row = a.data + ((long)b * a.N + i) * a.width;
    *cls = a.id_index >= 0 ? row[a.id_index] : 0.f;
    const float *c = row + a.coord_start;
    return make_float4(c[0], c[1], c[2], c[3]);
}

// The best cand_max candidates of an image in rank order, one work-group per
// image.  If there are more, the key of the last one is found first by
// counting digits of 11, 11 and 10 bits from the top (radix select), then
// those above it and the first rows of those equal to it are gathered in row
// order, and ranked: by comparing each with each (up to 512), or by radix
// passes in LDS.  Boxes, classes and rows leave in rank order, so that the
// mask and walk kernels read them with one request each.
//   One work-group's chain of reads, counts and barriers: 20 us for the best 400
// of 24564 rows (2400 candidates), where a segmented argsort of all of them
// and a gathering launch took 31 (box_nms of one image 54 -> 35 us, of 26
// images of 20565 rows 82 -> 32).
//   With many rows (kNmsOnePick) a first launch (SLICE), one work-group per
// slice of an image's chunks, leaves the best cand_max of every slice in the
// slice's first slots, in row order; the pick then reads one list per slice.
constexpr int kPickThreads = 1024;
constexpr int kPickWaves = kPickThreads / 64;
constexpr int kPickItems = kNmsMax / kPickThreads;     // per thread in the radix passes
constexpr int kPickCount = 512;                        // most that are ranked by comparing

// Images of more rows are picked in two launches, through slices of sqrt(rows *
// cand_max) rows, where both launches' work-groups read about as many
// candidates (all rows valid, best 400 of one image, before -> with it: 100
// thousand rows 197 -> 103 us, 200 thousand 343 -> 120, a million 1367 -> 173;
// best 4096 of 200 thousand 867 -> 694; best 400 of 32 images of 100 thousand
// 247 -> 152; a tenth of 200 thousand valid 109 -> 95).  At 30000 rows the one
// launch takes 111.
constexpr int kNmsOnePick = 1 << 16;

int nms_slice_chunks(int N, int cand_max)
{
    if (N <= kNmsOnePick || cand_max < 1) return 1;
    return std::max(1, (int)(std::sqrt((double)N * cand_max) / kNmsChunk + 0.5));
}

template <bool SLICE>
__global__ __launch_bounds__(kPickThreads) void nms_pick_kernel(NmsArgs a)
{
    __shared__ uint32_t key[kNmsMax];                  // picked: key bits, input rows
    __shared__ int32_t row[kNmsMax];
    __shared__ uint16_t sv[SLICE ? 1 : kNmsMax];       // ranking
    __shared__ uint16_t cnt[SLICE ? 1 : kPickWaves][256];
    __shared__ uint32_t hist[2048];
    __shared__ int wsum[kPickWaves];
    __shared__ int wlt[kPickWaves], weq[kPickWaves];
    __shared__ uint32_t s_digit;
    __shared__ int s_left, s_in;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    // the lists this work-group picks from: the chunks of a slice, or the slices of an image
    const int b = SLICE ? blockIdx.x / a.slices : blockIdx.x;
    const int sl = SLICE ? blockIdx.x - b * a.slices : 0;
    const int step = SLICE ? 1 : a.slice;              // chunks per list
    const int lists = SLICE ? min(a.slice, a.chunks - sl * a.slice) : a.slices;
    const int pitch = step * kNmsChunk;                // rows per list
    const int row0 = sl * a.slice * kNmsChunk;
    uint32_t *ck = a.ckey + (long)b * a.N + row0;
    int32_t *cr = a.corig + (long)b * a.N + row0;
    int32_t *cc = a.ccount + (long)b * a.chunks + sl * a.slice;
    // Wavefront w looks after a contiguous range of pieces, lists or (of fewer
    // than 16) equal parts of them: n candidates from slot `at` on.
    const int parts = lists < kPickWaves ? kPickWaves / lists : 1;
    const int per = (lists * parts + kPickWaves - 1) / kPickWaves;
    const int c0 = min(lists * parts, wid * per), c1 = min(lists * parts, c0 + per);
    struct Piece {
        int at, n;
    };
    auto piece = [&](int c) {
        const int l = parts == 1 ? c : c / parts, part = c - l * parts;
        // never past the list's rows
        const int n = min(max(cc[l * step], 0), min(pitch, a.N - row0 - l * pitch));
        if (parts == 1) return Piece{l * pitch, n};
        const int lo = n * part / parts;
        return Piece{l * pitch + lo, n * (part + 1) / parts - lo};
    };
    int mine = 0, total;
    for (int c = c0 + lane; c < c1; c += 64) mine += piece(c).n;
    wg_scan_incl<kPickThreads>(mine, wsum, &total);
    const int want = min(total, a.cand_max);
    // last: the largest key that is taken, and how many of its equals are
    uint32_t last = 0xffffffffu;
    int equals = total;
    if (want < total) {
        uint32_t prefix = 0, known = 0;                // digits found so far, and their mask
        int left = want;                               // rank of the last among those with the prefix
#pragma unroll 1
        for (int p = 0; p < 3; ++p) {
            const int shift = p == 0 ? 21 : p == 1 ? 10 : 0;
            const uint32_t dm = p == 2 ? 1023u : 2047u;
            hist[t] = 0;
            hist[t + 1024] = 0;
            __syncthreads();
            for (int c = c0; c < c1; ++c) {
                const Piece pc = piece(c);
                for (int i = lane; i < pc.n; i += 64) {
                    const uint32_t k = ck[pc.at + i];
                    if ((k & known) == prefix) atomicAdd(&hist[(k >> shift) & dm], 1u);
                }
            }
            __syncthreads();
            const int h0 = (int)hist[2 * t], h1 = (int)hist[2 * t + 1];
            int all;
            const int incl = wg_scan_incl<kPickThreads>(h0 + h1, wsum, &all);
            const int before = incl - h0 - h1;
            // the digit whose elements include rank `left` (1-based)
            if (before < left && left <= before + h0) {
                s_digit = 2 * t;
                s_left = left - before;
                s_in = h0;
            } else if (before + h0 < left && left <= incl) {
                s_digit = 2 * t + 1;
                s_left = left - before - h0;
                s_in = h1;
            }
            __syncthreads();
            prefix |= s_digit << shift;
            known |= dm << shift;
            left = s_left;
            if (s_in == left) {                        // all of them: no need to tell them apart
                prefix |= ~known;
                left = a.N;
                break;
            }
            __syncthreads();
        }
        last = prefix;
        equals = left;
    }
    // gather in row order: count per wavefront, then place
    int lt = 0, eq = 0;
    for (int c = c0; c < c1; ++c) {
        const Piece pc = piece(c);
        for (int i = lane; i < pc.n; i += 64) {
            const uint32_t k = ck[pc.at + i];
            lt += k < last;
            eq += k == last;
        }
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        lt += __shfl_xor(lt, d);
        eq += __shfl_xor(eq, d);
    }
    if (lane == 0) {
        wlt[wid] = lt;
        weq[wid] = eq;
    }
    __syncthreads();
    lt = eq = 0;
    for (int w = 0; w < wid; ++w) {
        lt += wlt[w];
        eq += weq[w];
    }
    for (int c = c0; c < c1; ++c) {
        const Piece pc = piece(c);
        const int n = pc.n;
        for (int i0 = 0; i0 < n; i0 += 64) {
            const int i = i0 + lane;
            const uint32_t k = i < n ? ck[pc.at + i] : 0xffffffffu;
            const int32_t r = i < n ? cr[pc.at + i] : 0;
            const uint64_t bl = __ballot(i < n && k < last), be = __ballot(i < n && k == last);
            const int nl = lt + lanes_before(bl), ne = eq + lanes_before(be);
            const bool take = i < n && (k < last || (k == last && ne < equals));
            const int slot = nl + min(ne, equals);
            if (take && slot < want) {
                key[slot] = k;
                row[slot] = min(max(r, 0), a.N - 1);
            }
            lt += __popcll(bl);
            eq += __popcll(be);
        }
    }
    __syncthreads();                                   // and every read of the lists is done
    if constexpr (SLICE) {
        for (int i = t; i < want; i += kPickThreads) {
            ck[i] = key[i];
            cr[i] = row[i];
        }
        if (t == 0) cc[0] = want;
        return;
    }
    auto emit = [&](int rank, int i) {
        float c;
        const long o = (long)b * a.mrows + rank;
        a.cbox[o] = load_box(a, b, row[i], &c);
        a.ccls[o] = c;
        a.crow[o] = row[i];
    };
    if (want <= kPickCount) {
        // rank = how many come before: two threads per candidate, half each
        int *rank = reinterpret_cast<int *>(hist);
        if (t < kPickCount) rank[t] = 0;
        __syncthreads();
        const int i = t & (kPickCount - 1), half = (want + 1) / 2;
        const int j0 = t < kPickCount ? 0 : half, j1 = t < kPickCount ? half : want;
        if (i < want) {
            const uint32_t k = key[i];
            int n = 0;
#pragma unroll 8
            for (int j = j0; j < j1; ++j) n += key[j] < k || (key[j] == k && j < i);
            atomicAdd(&rank[i], n);
        }
        __syncthreads();
        if (t < want) emit(rank[t], t);
    } else {
        uint32_t x[kPickItems];
        int v[kPickItems];
#pragma unroll
        for (int r = 0; r < kPickItems; ++r) {
            v[r] = wid * 64 * kPickItems + lane + 64 * r;
            x[r] = v[r] < want ? key[v[r]] : 0xffffffffu;     // the rest last
        }
        __syncthreads();
#pragma unroll 1
        for (int p = 0; p < 4; ++p)
            lds_radix_pass<kPickThreads, kPickItems>(x, v, 8 * p, key, sv, cnt, wsum);
#pragma unroll
        for (int r = 0; r < kPickItems; ++r) {
            const int rank = wid * 64 * kPickItems + lane + 64 * r;
            if (rank < want) emit(rank, v[r]);
        }
    }
    if (t == 0) a.count[b] = want;
}

// Compared candidates of image b.
__device__ __forceinline__ int nms_count(const NmsArgs &a, int b) { return min(max(a.count[b], 0), a.cand_max); }

// IoU of two corner-encoded boxes, each operation rounded to fp32 in the
// order of the definition.  Contraction into fused multiply-adds is switched
// off here: the compiler would otherwise fold the area products into the
// union's sums, whose single rounding moves the IoU by an ulp and flips
// comparisons at the threshold.
__device__ __forceinline__ float box_iou(float4 p, float4 q)
{
#pragma clang fp contract(off)
    const float iw = fmaxf(0.f, fminf(p.z, q.z) - fmaxf(p.x, q.x));
    const float ih = fmaxf(0.f, fminf(p.w, q.w) - fmaxf(p.y, q.y));
    const float inter = iw * ih;
    const float ap = fmaxf(0.f, p.z - p.x) * fmaxf(0.f, p.w - p.y);
    const float aq = fmaxf(0.f, q.z - q.x) * fmaxf(0.f, q.w - q.y);
    const float uni = (ap + aq) - inter;
    return uni <= 0.f ? 0.f : inter / uni;
}

// Suppression masks: work-group (column block cb, row block rb, image b),
// four wavefronts.  Lane t of wavefront q takes candidate i = 64*rb + t (the
// loop above the innermost one, on work-groups and lanes) and tests it
// against the 16 candidates j = 64*cb + 16*q .. + 15 staged in LDS (the
// innermost loop): bit j - 64*cb of mask[b][i][cb] is set when j comes later
// and i, once kept, suppresses it.  Each wavefront writes its 16 bits of the
// word.  Blocks below the diagonal are never read and not computed.
__global__ __launch_bounds__(256) void nms_mask_kernel(NmsArgs a)
{
    __shared__ float4 cbox[64];
    __shared__ float ccls[64];
    const int cb = blockIdx.x, rb = blockIdx.y, b = blockIdx.z;
    if (cb < rb) return;
    const int count = nms_count(a, b);
    if (rb * 64 >= count) return;
    const int t = threadIdx.x & 63, q = threadIdx.x >> 6;
    const long base = (long)b * a.mrows;
    if (threadIdx.x < 64) {
        const int j = cb * 64 + t;
        if (j < count) {
            cbox[t] = a.cbox[base + j];
            ccls[t] = a.ccls[base + j];
        }
    }
    __syncthreads();
    const int i = rb * 64 + t;
    if (i >= count) return;
    const float4 bi = a.cbox[base + i];
    const float ci = a.ccls[base + i];
    const bool any_class = a.force || a.id_index < 0;
    uint32_t bits = 0;
    const int j0 = cb * 64 + 16 * q;
    const int jn = count - j0 < 16 ? count - j0 : 16;
    for (int jj = 0; jj < jn; ++jj) {
        const int jg = j0 + jj;
        if (jg <= i) continue;
        if (!any_class && !(ccls[16 * q + jj] == ci)) continue;
        if (box_iou(bi, cbox[16 * q + jj]) > a.overlap) bits |= 1u << jj;
    }
    // bits 16q .. 16q+15 of the 64-bit word (little-endian halves of halves)
    reinterpret_cast<uint16_t *>(a.mask)[((base + i) * a.capw + cb) * 4 + q] = (uint16_t)bits;
}

// The greedy walk, one work-group per image.  The mask rows of the image's
// candidates are staged in LDS by all 256 threads at once (as many rows as
// fit; all requests in flight together), then the first wavefront walks:
// lane w holds word w of the removed set, candidate i (rank order) is kept
// unless its bit is set (the word is read from its lane with readlane, i
// being uniform), and a kept candidate ORs its mask row (words from its own
// on) into the set.  The kept ranks are listed in LDS, and afterwards all
// threads copy the kept rows, one value each, to the first output rows.
// The 64-bit value v of lane w (uniform w), as a scalar.
__device__ __forceinline__ uint64_t lane_word(uint64_t v, int w)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, w);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), w);
    return ((uint64_t)hi << 32) | lo;
}

constexpr int kSweepThreads = 256;
constexpr int kSweepWords = 6144;   // 48 KB of mask rows per staging round

__global__ __launch_bounds__(kSweepThreads) void nms_sweep_kernel(NmsArgs a)
{
    __shared__ uint64_t rows[kSweepWords];
    __shared__ int kept_rank[kNmsMax];
    __shared__ int kept_n;
    const int b = blockIdx.x, t = threadIdx.x, lane = t & 63;
    const int count = nms_count(a, b);
    const long base = (long)b * a.mrows;
    const int per = kSweepWords / a.capw / 64 * 64;   // rows per staging round: whole words, >= 64
    uint64_t removed = 0;
    int kept = 0;
    for (int r0 = 0; r0 < count; r0 += per) {
        const int nr = count - r0 < per ? count - r0 : per;
        const int words = nr * a.capw;
        __syncthreads();
        for (int e0 = 0; e0 < words; e0 += kSweepThreads * 8) {
            uint64_t v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int e = e0 + k * kSweepThreads + t;
                const int rr = e / a.capw, w = e - rr * a.capw;
                // words left of the row's own block are never written; read as 0
                v[k] = e < words && w >= (r0 + rr) / 64 ? a.mask[(base + r0 + rr) * a.capw + w] : 0;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int e = e0 + k * kSweepThreads + t;
                if (e < words) rows[e] = v[k];
            }
        }
        __syncthreads();
        if (t < 64) {
            // word by word: the next candidate not yet removed is the lowest
            // clear bit above the last one taken, so removed candidates cost
            // nothing and the walk takes one step per kept candidate
            for (int w = r0 >> 6; w * 64 < r0 + nr; ++w) {
                const int valid = r0 + nr - w * 64 < 64 ? r0 + nr - w * 64 : 64;
                const uint64_t live = valid == 64 ? ~0ull : (1ull << valid) - 1;
                uint64_t cur = lane_word(removed, w);
                uint64_t avail = ~cur & live;
                while (avail) {
                    const int bit = __builtin_ctzll(avail);
                    const int i = w * 64 + bit;
                    if (lane == 0) kept_rank[kept] = i;
                    ++kept;
                    if (lane < a.capw) removed |= rows[(i - r0) * a.capw + lane];
                    cur = lane_word(removed, w);
                    avail = ~cur & live & ~((2ull << bit) - 1);   // bits above `bit` (none when bit = 63)
                }
            }
        }
    }
    if (t == 0) kept_n = kept;
    __syncthreads();
    const int nk = kept_n;
    for (int e = t; e < nk * a.width; e += kSweepThreads) {
        const int k = e / a.width, c = e - k * a.width;
        const float *src = a.data + ((long)b * a.N + a.crow[base + kept_rank[k]]) * a.width;
        a.out[((long)b * a.N + k) * a.width + c] = src[c];
    }
}

struct NmsLayout {
    long ckey, corig, ccount, count, cbox, ccls, crow, mask, total;
};

NmsLayout nms_layout(int B, int N, int cap)
{
    const long n = (long)B * N;
    const int capw = (cap + 63) / 64;
    NmsLayout l{};
    long o = 0;
    l.ckey = o;
    o += align256(n * 4);
    l.corig = o;
    o += align256(n * 4);
    l.ccount = o;
    o += align256((long)B * ((N + kNmsChunk - 1) / kNmsChunk) * 4);
    l.count = o;
    o += align256((long)B * 4);
    const long mrows = (long)B * capw * 64;
    l.cbox = o;
    o += align256(mrows * 16);
    l.ccls = o;
    o += align256(mrows * 4);
    l.crow = o;
    o += align256(mrows * 4);
    l.mask = o;
    o += align256(mrows * capw * 8);
    l.total = o;
    return l;
}

int nms_cap(int N, int topk) { return topk < 0 ? N : (topk < N ? topk : N); }

bool ws_ok(void *ws, size_t bytes, long need)
{
    if (need == 0) return true;
    return ws && ((uintptr_t)ws & 255) == 0 && (long)bytes >= need;
}

}  // namespace
}  // namespace miconv

using namespace miconv;

extern "C" {

long vision_scan_workspace_bytes(int rows, long n)
{
    if (rows < 1 || n < 1) return MICONV_ERR_SHAPE;
    if ((long)rows * n >= (1L << 31)) return MICONV_ERR_TOO_LARGE;
    return scan_ws_bytes(rows, n);
}

int vision_scan_i32(int rows, long n, const int32_t *x, int32_t *y, int exclusive, void *ws, size_t ws_bytes,
                    void *stream)
{
    if (!x || !y) return MICONV_ERR_NULL;
    const long need = vision_scan_workspace_bytes(rows, n);
    if (need < 0) return (int)need;
    if (!ws_ok(ws, ws_bytes, need)) return MICONV_ERR_WORKSPACE;
    const hipError_t e = launch_scan(x, rows, n, y, exclusive != 0, ws,
                                     static_cast<hipStream_t>(stream));
    return e == hipSuccess ? MICONV_OK : set_hip_error(e);
}

long vision_argsort_workspace_bytes(long n, int segments)
{
    if (n < 1 || segments < 1) return MICONV_ERR_SHAPE;
    if (n >= (1L << 31) || segments >= (1 << 21) - 1) return MICONV_ERR_TOO_LARGE;
    return argsort_ws_bytes(n);
}

int vision_segmented_argsort(long n, int segments, const float *keys, const int32_t *offsets, int descending,
                             int32_t *out, void *ws, size_t ws_bytes, void *stream)
{
    if (!keys || !offsets || !out) return MICONV_ERR_NULL;
    const long need = vision_argsort_workspace_bytes(n, segments);
    if (need < 0) return (int)need;
    if (!ws_ok(ws, ws_bytes, need)) return MICONV_ERR_WORKSPACE;
    const hipError_t e = launch_segsort(keys, offsets, segments, n, descending != 0 ? 1 : 0, out, ws,
                                        static_cast<hipStream_t>(stream));
    return e == hipSuccess ? MICONV_OK : set_hip_error(e);
}

long vision_box_nms_workspace_bytes(int batch, int num, int width, int topk)
{
    if (batch < 1 || num < 1 || width < 1) return MICONV_ERR_SHAPE;
    if ((long)batch * num * width >= (1L << 31) || batch >= (1 << 21) - 1) return MICONV_ERR_TOO_LARGE;
    const int cap = nms_cap(num, topk);
    if (cap > kNmsMax) return MICONV_ERR_UNSUPPORTED;
    return nms_layout(batch, num, cap).total;
}

int vision_box_nms(int batch, int num, int width, const float *data, float *out, float overlap_thresh,
                   float valid_thresh, int topk, int id_index, int score_index, int coord_start,
                   int force_suppress, void *ws, size_t ws_bytes, void *stream)
{
    if (!data || !out) return MICONV_ERR_NULL;
    const long need = vision_box_nms_workspace_bytes(batch, num, width, topk);
    if (need < 0) return (int)need;
    if (score_index < 0 || score_index >= width || coord_start < 0 || coord_start + 4 > width ||
        id_index >= width)
        return MICONV_ERR_SHAPE;
    if (((uintptr_t)data & 3) || ((uintptr_t)out & 3)) return MICONV_ERR_ALIGN;
    if (!ws_ok(ws, ws_bytes, need)) return MICONV_ERR_WORKSPACE;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const int cap = nms_cap(num, topk);
    const NmsLayout l = nms_layout(batch, num, cap);
    char *w = static_cast<char *>(ws);
    NmsArgs a{};
    a.data = data;
    a.out = out;
    a.B = batch;
    a.N = num;
    a.width = width;
    a.cand_max = cap;
    a.capw = (cap + 63) / 64;
    a.mrows = a.capw * 64;
    a.overlap = overlap_thresh;
    a.valid = valid_thresh;
    a.id_index = id_index < 0 ? -1 : id_index;
    a.score_index = score_index;
    a.coord_start = coord_start;
    a.force = force_suppress != 0;
    a.chunks = (num + kNmsChunk - 1) / kNmsChunk;
    a.slice = nms_slice_chunks(num, cap);
    a.slices = (a.chunks + a.slice - 1) / a.slice;
    a.ckey = reinterpret_cast<uint32_t *>(w + l.ckey);
    a.corig = reinterpret_cast<int32_t *>(w + l.corig);
    a.ccount = reinterpret_cast<int32_t *>(w + l.ccount);
    a.count = reinterpret_cast<int32_t *>(w + l.count);
    a.cbox = reinterpret_cast<float4 *>(w + l.cbox);
    a.ccls = reinterpret_cast<float *>(w + l.ccls);
    a.crow = reinterpret_cast<int32_t *>(w + l.crow);
    a.mask = reinterpret_cast<uint64_t *>(w + l.mask);
    launch_kernel(nms_collect_kernel, dim3((unsigned)((long)batch * a.chunks)), dim3(256), 0, st, a);
    if (a.capw > 0) {   // topk == 0: no candidate, the output stays invalid
        if (a.slices < a.chunks)
            launch_kernel(nms_pick_kernel<true>, dim3((unsigned)(batch * a.slices)), dim3(kPickThreads), 0, st, a);
        launch_kernel(nms_pick_kernel<false>, dim3((unsigned)batch), dim3(kPickThreads), 0, st, a);
        launch_kernel(nms_mask_kernel, dim3((unsigned)a.capw, (unsigned)a.capw, (unsigned)batch), dim3(256), 0, st,
                      a);
        launch_kernel(nms_sweep_kernel, dim3((unsigned)batch), dim3(kSweepThreads), 0, st, a);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MICONV_OK : set_hip_error(e);
}

}  // extern "C"
