// Dense conv2d in fp32 on the bf16 matrix cores, for layers large enough to
// be bound by the fp32 MFMA rate.
//
// Every fp32 value is the exact sum of three bf16 values (the bf16x3 scheme of
// Henry, Tang and Heinecke, 2019): hi = bf16(v), mid = bf16(v - hi), lo = v -
// hi - mid, each rounded to nearest even, so |mid| <= 2^-8 |v| and |lo| <= 2^-17
// |v| and nothing is left over (24 significand bits in three times 8).  A
// product is then
//   x w = xh wh + (xh wm + xm wh + xm wm + xh wl + xl wh) + (xm wl + xl wm + xl wl)
// and the last bracket, at most 2^-24 of |x w| (about 2^-28 on random data), is
// dropped: no more than fp32's own rounding of the product.  Six bf16 MFMAs of
// 16 taps replace eight fp32 MFMAs of 2 taps: 192 cycles per 32 x 32 x 16 block
// instead of 512.
// xh wh goes to one fp32 accumulator and the five small products to another,
// so the roundings of the small ones do not add to the large sum's: in the
// 2-norm against 64 bits the result is no further off than the fp32 MFMA
// kernel's (0.31 to 0.92 of its error on 100 drawn layers).  As one accumulator
// takes the whole reduction, of which that kernel's wavefronts hold an eighth
// each, the error grows more with an output's size: outputs beyond twice the
// rms are 1.1 to 1.6 times as far off as there, at most 1.6e-7 of the sum of
// magnitudes (0.8e-7 there).
//
// A call
//  1. splits x into a channel-last copy xs [N*H*W][groups][CB][3][16] (CB
//     blocks of 16 channels, zero-padded; the three parts of a block are 96
//     contiguous bytes), one HBM pass;
//  2. reads filters split the same way, [groups][K/64][chunk][64 filters][3][16]
//     (packed per call, or once by the stack executor);
//  3. runs the implicit GEMM: the reduction is walked in chunks of one
//     16-channel block at one filter position (r, s), block outermost, both
//     operands moved straight into LDS (NST stages), 12 LDS reads and 24
//     MFMAs per wavefront and chunk: three times the MFMA work per byte of
//     LDS and L2 traffic of the plain bf16 kernel.
//
// Bound by the bf16 MFMA rate and by how evenly the tiles fill the CUs: VGG-16
// 256 -> 256 3x3 at 56x56, batch 8 (29.6 GFLOP): 302 us on the fp32 MFMA
// kernel, 178 us here, 13 us of it the split copy of x (4.9 TB/s).  Counted:
// MFMAs busy 49% of the cycles of all SIMDs (392 tiles in 512 places; 56% at
// 28x28, 980 work-groups), no LDS bank conflicts (64 x 128 tiles: 6 cycles per
// 100 LDS instructions).  Three stages of 16-channel chunks leave two
// work-groups per CU; five stages (one fewer) were slower on every shape.
//
// Both operands are split at 2^24 times their value and the sums scaled back,
// so that no part of any fp32 value, subnormal ones included, falls below
// bf16's normal numbers (2^-149 becomes 2^-125), nor any product of parts that
// counts below fp32's.  The other end pays: values from 2^104 and sums from
// 2^80 overflow, and are served as infinities are.
//
// Infinities, NaNs and values that overflow have a part that is not finite,
// which makes every sum they enter NaN or infinite.  A wavefront that holds such a sum
// therefore runs its tile's reduction again on the fp32 matrix cores before
// bias, residual and activation, and takes those sums that are not finite from
// there (plain_sums; ordinary data never takes that path).
#include "internal.h"

#include <algorithm>
#include <cstdio>

namespace miconv {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr float kScaleUp = 0x1p24f, kScaleDown = 0x1p-24f;

// The three parts of 8 values times kScaleUp, packed in pairs.
struct Parts {
    uint4 hi, mid, lo;
};

__device__ __forceinline__ Parts split8(const float (&v)[8])
{
    uint32_t d[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float a = v[2 * e] * kScaleUp, b = v[2 * e + 1] * kScaleUp;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t q = pack_bf16x2(a, b);
            d[p][e] = q;
            a -= __uint_as_float(q << 16);
            b -= __uint_as_float(q & 0xFFFF0000u);
        }
    }
    return Parts{make_uint4(d[0][0], d[0][1], d[0][2], d[0][3]), make_uint4(d[1][0], d[1][1], d[1][2], d[1][3]),
                 make_uint4(d[2][0], d[2][1], d[2][2], d[2][3])};
}

struct SplitCopyArgs {
    const float *x;
    uint16_t *xs;
    int C, Cg, HW, CB, npx;   // CB: 16-channel blocks per group; npx = N*H*W
    int blocks;               // groups * CB
    int tiles_c;              // pairs of blocks
    FastDiv dv_hw, dv_cb;
};

// x fp32 NCHW -> xs.  A work-group moves 32 (padded) channels x 64 pixels
// (flattened over images) through LDS; V = pixels per global load (4 when
// H*W % 4 == 0 and x is 16-byte aligned, else 1).  Each thread then gathers 8
// channels of one pixel and writes its three parts, 16 bytes each.
template <int V>
__global__ __launch_bounds__(256) void split3_copy_kernel(SplitCopyArgs a)
{
    constexpr int PITCH = 66;                 // 4 lanes 8 channels apart, 16 pixels each: 64 banks
    __shared__ __attribute__((aligned(16))) float tile[32][PITCH];
    const int t = threadIdx.x;
    const int b0 = (blockIdx.x % a.tiles_c) * 2;
    const int p0 = (blockIdx.x / a.tiles_c) * 64;
    constexpr int GR = 64 / V;
#pragma unroll
    for (int i = 0; i < 32 * GR / 256; ++i) {
        const int id = t + 256 * i;
        const int cl = id / GR, px = p0 + V * (id % GR);
        const int blk = b0 + (cl >> 4);
        const int g = fdiv(blk, a.dv_cb);
        const int cc = (blk - g * a.CB) * 16 + (cl & 15);
        const bool ok = blk < a.blocks && cc < a.Cg && px < a.npx;
        const unsigned n = fdiv(ok ? px : 0, a.dv_hw);
        const float *src = a.x + ((long)n * a.C + (ok ? g * a.Cg + cc : 0)) * a.HW + ((ok ? px : 0) - (int)n * a.HW);
        float *dst = &tile[cl][V * (id % GR)];
        if constexpr (V == 4) {
            const float4 v = ok ? *reinterpret_cast<const float4 *>(src) : make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<float2 *>(dst) = make_float2(v.x, v.y);
            *reinterpret_cast<float2 *>(dst + 2) = make_float2(v.z, v.w);
        } else {
            *dst = ok ? *src : 0.f;
        }
    }
    __syncthreads();
    const int o = t & 3, px = t >> 2;          // octet of the 32 channels, pixel
    const int blk = b0 + (o >> 1);
    if (blk >= a.blocks || p0 + px >= a.npx) return;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile[8 * o + e][px];
    const Parts p = split8(v);
    uint4 *dst = reinterpret_cast<uint4 *>(a.xs) + ((long)(p0 + px) * a.blocks + blk) * 6 + (o & 1);
    dst[0] = p.hi;
    dst[2] = p.mid;
    dst[4] = p.lo;
}

// 16-byte unit j (0..5: part j/2, channel half j%2) of a 96-byte operand row
// sits at slot j ^ ((row >> 3) & 1): 16 consecutive rows read at one unit then
// fall in 16 distinct 16-byte bank groups (6 * row covers the even ones twice).
__device__ __forceinline__ int row_flip(int row) { return (row >> 3) & 1; }

// Filters: one thread per (group, 64-filter tile, chunk, filter, half); the
// slots of a filter's row carry the LDS permutation, so a tile's chunk is
// copied to LDS as it lies.  Zero past K/groups and C/groups.
__global__ __launch_bounds__(256) void split3_pack_kernel(const float *__restrict__ w, uint4 *__restrict__ dst,
                                                          int Kg, int Cg, int RS, int KT, int NC, long total)
{
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
        const int half = (int)(i & 1), row = (int)((i >> 1) & 63);
        const long tc = i >> 7;                 // (g * KT + kt) * NC + chunk
        const int t = (int)(tc % NC);
        const long gk = tc / NC;
        const int kt = (int)(gk % KT), g = (int)(gk / KT);
        const int cb = t / RS, rs = t - cb * RS;
        const int k = kt * 64 + row;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = cb * 16 + half * 8 + e;
            v[e] = k < Kg && c < Cg ? w[(((long)g * Kg + k) * Cg + c) * RS + rs] : 0.f;
        }
        const Parts p = split8(v);
        uint4 *d = dst + (tc * 64 + row) * 6;
        const int f = row_flip(row);
        d[(0 + half) ^ f] = p.hi;
        d[(2 + half) ^ f] = p.mid;
        d[(4 + half) ^ f] = p.lo;
    }
}

struct SplitArgs {
    ConvArgs a;             // x, w: the fp32 tensors as given (for sums that are not finite)
    const uint16_t *xs;     // split channel-last copy of x
    const uint16_t *wp;     // split packed filters
    int CB, NC;             // 16-channel blocks per group, chunks (CB * R * S)
    unsigned px_bytes;      // bytes per pixel of xs
};

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The sums of a wavefront's tile over chunks t0 .. t1-1 on the fp32 matrix
// cores: pixels moff + 32 bj + lane % 32 (past M: zero), filters koff + 32 bi +
// lane % 32 of group g (past K/groups: zero), in the accumulator layout of the
// split products.  Taps in the padding are zeros, as in every other kernel.
// Every four chunks are summed apart, so that the roundings are no more than
// where the fp32 wave kernel's wavefronts divide the reduction among themselves.
// x is read as given (a wavefront's loads are runs of pixels); filters are put
// together again from their parts, whose rows lie together, except where they
// are not finite.  256 -> 256 3x3 at 56x56, batch 8 (180 us of finite data): x
// NaN throughout 658 us, one NaN in x 477 (the fp32 wave kernel 334 and 368);
// with filters read as given, a line per lane and load, 854 and 584; a sum per
// lane, element by element, 20.7 and 16.5 ms.
template <int BJ, int BI>
__device__ inline void plain_sums(const SplitArgs &sa, int g, int moff, int koff, int t0, int t1,
                                  floatx16 (&sum)[BJ][BI])
{
    const ConvArgs &a = sa.a;
    const int h = (threadIdx.x & 63) >> 5, ll = threadIdx.x & 31;
    const int RS = a.R * a.S;
    const int KT = (a.Kg + 63) / 64;
    constexpr unsigned kOutside = 0xffffffffu;
    const float *w = static_cast<const float *>(a.w);
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void *>(a.x), (short)0, (int)((long)a.N * a.C * a.HW * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(sa.wp), (short)0, (int)((long)a.groups * KT * sa.NC * 6144), 0x00020000);
    int ih0[BJ], iw0[BJ];
    unsigned xoff[BJ], woff[BI];
    floatx16 acc[BJ][BI];
#pragma unroll
    for (int bj = 0; bj < BJ; ++bj) {
        const int m = moff + 32 * bj + ll;
        const int n = fdiv(m < a.M ? m : 0, a.dv_pq);
        const int pq = (m < a.M ? m : 0) - n * a.PQ;
        const int p = fdiv(pq, a.dv_q);
        ih0[bj] = m < a.M ? p * a.stride - a.pad : -(1 << 28);   // never inside the image
        iw0[bj] = (pq - p * a.Q) * a.stride - a.pad;
        // wraps below zero for a padding origin, and back for every tap inside the image
        xoff[bj] = 4u * ((unsigned)((n * a.C + g * a.Cg + 8 * h) * a.HW) + (unsigned)ih0[bj] * (unsigned)a.W +
                         (unsigned)iw0[bj]);
    }
#pragma unroll
    for (int bi = 0; bi < BI; ++bi) {
        const int k = koff + 32 * bi + ll;
        woff[bi] = k < a.Kg ? (unsigned)((((long)g * KT + k / 64) * sa.NC * 64 + k % 64) * 96) + 16u * (h ^ row_flip(k))
                            : kOutside;
#pragma unroll
        for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bj][bi][v] = sum[bj][bi][v] = 0.f;
    }
#pragma unroll 1
    for (int u = 2 * t0; u < 2 * t1; ++u) {               // channels 8 h + 4 (u % 2) + e of chunk u / 2's block
        const int t = u >> 1, cb = t / RS, rs = t - cb * RS;
        const int r = rs / a.S, s = rs - r * a.S;
        const int c = cb * 16 + 8 * h + 4 * (u & 1);
        const unsigned xd = 4u * (unsigned)((cb * 16 + 4 * (u & 1)) * a.HW + r * a.W + s);
        float xv[BJ][4], wv[BI][4];
        uint2 part[BI][3];
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                part[bi][p] = __builtin_bit_cast(
                    uint2, __builtin_amdgcn_raw_buffer_load_b64(
                               wres, woff[bi] == kOutside ? kOutside : woff[bi] + 6144u * t + 8u * (u & 1) + 32u * p, 0, 0));
#pragma unroll
        for (int bj = 0; bj < BJ; ++bj) {
            const bool in = (unsigned)(ih0[bj] + r) < (unsigned)a.H && (unsigned)(iw0[bj] + s) < (unsigned)a.W;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                xv[bj][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    xres, in && c + e < a.Cg ? xoff[bj] + xd + 4u * e * a.HW : kOutside, 0, 0));
        }
#pragma unroll
        for (int bi = 0; bi < BI; ++bi) {
            const int k = koff + 32 * bi + ll;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const uint32_t q = e < 2 ? part[bi][p].x : part[bi][p].y;
                    v[p] = __uint_as_float(e & 1 ? q & 0xFFFF0000u : q << 16);
                }
                wv[bi][e] = (v[0] + v[1] + v[2]) * kScaleDown;
                if (!(fabsf(v[0]) < __builtin_inff()))    // never a zero of the padding past K or C
                    wv[bi][e] = w[(((long)g * a.Kg + k) * a.Cg + c + e) * RS + rs];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
                for (int bi = 0; bi < BI; ++bi)
                    acc[bj][bi] = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[bj][e], wv[bi][e], acc[bj][bi], 0, 0, 0);
        if (((u - 2 * t0) & 7) == 7 || u + 1 == 2 * t1)
#pragma unroll
            for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
                for (int bi = 0; bi < BI; ++bi)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        sum[bj][bi][v] += acc[bj][bi][v];
                        acc[bj][bi][v] = 0.f;
                    }
    }
}

template <int BPX, int BKC, int WPX, int WCH, int NST>
__global__ __launch_bounds__(256, 2) void igemm_split3_kernel(SplitArgs sa)
{
    const ConvArgs &a = sa.a;
    constexpr int NT = 256;
    static_assert(WPX * WCH == 4, "four wavefronts");
    constexpr int TPX = BPX / WPX, TCH = BKC / WCH;     // one wavefront's tile
    constexpr int BJ = TPX / 32, BI = TCH / 32;
    constexpr int LA = (BKC * 6 + NT - 1) / NT, LB = (BPX * 6 + NT - 1) / NT;
    constexpr int UA = LA * NT, UB = LB * NT;           // units per stage, whole loads
    constexpr int LOADS = LA + LB;
    constexpr int OP = BPX + 4;
    constexpr int EPI = BKC * OP / 4;
    constexpr int SMEM = NST * (UA + UB) > EPI ? NST * (UA + UB) : EPI;
    __shared__ __attribute__((aligned(16))) uint4 smem[SMEM];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = tid >> 6;
    const int wpx = wid % WPX, wch = wid / WPX;
    const int h = lane >> 5, ll = lane & 31;
    // XCD-aware tile order: each XCD gets one contiguous range of tiles, the
    // filter tiles of one pixel tile adjacent (they share its L2).
    const int T = gridDim.x;
    const int xcd = blockIdx.x % 8, jx = blockIdx.x / 8;
    const int L = xcd * (T / 8) + min(xcd, T % 8) + jx;
    const int ktiles = (a.Kg + BKC - 1) / BKC;
    const int mtiles = (a.M + BPX - 1) / BPX;
    const int ky = L % ktiles;
    const int mx = (L / ktiles) % mtiles;
    const int z = L / (ktiles * mtiles);
    const int g = z % a.groups;
    const int split = z / a.groups;
    const int m0 = mx * BPX;
    const int k0 = ky * BKC;
    const int t_begin = split * a.kr_per_split;         // in chunks
    const int t_end = min(sa.NC, t_begin + a.kr_per_split);
    const int RS = a.R * a.S;

    constexpr unsigned kOutside = 0xffffffffu;          // past either buffer: zeros
    const int KT = (a.Kg + 63) / 64;                    // 64-filter tiles per group
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(sa.wp), (short)0, (int)((long)a.groups * KT * sa.NC * 6144), 0x00020000);
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(sa.xs), (short)0, (int)((long)a.N * a.HW * sa.px_bytes), 0x00020000);

    // Filter loader: load i fills unit u = i*NT + tid of the tile's chunk (64
    // filters x 6 units contiguous per 64-filter tile).
    unsigned aoffs[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int u = i * NT + tid;
        const int row = u / 6;
        const int kt = k0 / 64 + row / 64;
        aoffs[i] = row < BKC && kt < KT
                       ? (unsigned)((((long)g * KT + kt) * sa.NC * 384 + (u - row / 64 * 384)) * 16)
                       : kOutside;
    }
    // Pixel loader: unit u is slot u % 6 of pixel row u / 6.
    int bih[LB], biw[LB];
    unsigned boffs[LB];
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int u = i * NT + tid;
        const int row = u / 6;
        const int j = (u - row * 6) ^ row_flip(row);
        const int m = m0 + row;
        const bool ok = row < BPX && m < a.M;
        const int mm = ok ? m : 0;
        const int n = fdiv(mm, a.dv_pq);
        const int pq = mm - n * a.PQ;
        const int p = fdiv(pq, a.dv_q);
        const int q = pq - p * a.Q;
        const int ih0 = p * a.stride - a.pad;
        bih[i] = ok ? ih0 : -(1 << 28);                 // never inside the image
        biw[i] = q * a.stride - a.pad;
        // of tap (0, 0), block 0 of the group; wraps below zero for a padding
        // origin, and back for every tap that passes the bounds test
        boffs[i] = (unsigned)((n * a.H + ih0) * a.W + biw[i]) * sa.px_bytes + (unsigned)(g * sa.CB * 96 + j * 16);
    }

    // position of the next chunk to request
    int icb = __builtin_amdgcn_readfirstlane(t_begin / RS);
    int irs = __builtin_amdgcn_readfirstlane(t_begin - icb * RS);
    int ir = __builtin_amdgcn_readfirstlane(irs / a.S), is = __builtin_amdgcn_readfirstlane(irs - ir * a.S);
    auto issue = [&](int t, int stage) {
        uint4 *st = smem + stage * (UA + UB);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const unsigned off = aoffs[i] == kOutside ? kOutside : aoffs[i] + 6144u * t;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wres, (lds_void_t *)(st + i * NT + wid * 64), 16, off, 0, 0, 0);
        }
        const unsigned delta = (unsigned)(ir * a.W + is) * sa.px_bytes + (unsigned)icb * 96u;
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const bool ok = (unsigned)(bih[i] + ir) < (unsigned)a.H && (unsigned)(biw[i] + is) < (unsigned)a.W;
            const unsigned off = ok ? boffs[i] + delta : kOutside;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_void_t *)(st + UA + i * NT + wid * 64), 16, off, 0, 0,
                                                     0);
        }
        if (++is == a.S) {
            is = 0;
            if (++ir == a.R) {
                ir = 0;
                ++icb;
            }
        }
    };

    // Operand reads: 16-byte unit 2*part + h of the lane's rows.
    int aoff[BI], boff[BJ];
    const int sl = h ^ row_flip(ll);
#pragma unroll
    for (int bi = 0; bi < BI; ++bi) aoff[bi] = (wch * TCH + bi * 32 + ll) * 6 + sl;
#pragma unroll
    for (int bj = 0; bj < BJ; ++bj) boff[bj] = UA + (wpx * TPX + bj * 32 + ll) * 6 + sl;

    // A wavefront with one block of its own keeps two accumulators of small
    // products, so that its MFMAs do not all wait for one another.
    constexpr int NS = BI * BJ == 1 ? 2 : 1;
    floatx16 big[BJ][BI], small[NS][BJ][BI];
#pragma unroll
    for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
        for (int bi = 0; bi < BI; ++bi)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                big[bj][bi][v] = 0.f;
                for (int i = 0; i < NS; ++i) small[i][bj][bi][v] = 0.f;
            }

    // The next chunk is requested between the operand reads and the MFMAs,
    // which run at raised priority: the two work-groups of a CU then
    // alternate, one in its MFMAs while the other waits and requests (128 x
    // 128 tiles 183 -> 179 us, 221 -> 204 us on VGG-16's 56x56 and 112x112
    // layers at batch 8).
    auto compute = [&](int stage, bool more, int tn, int fill) {
        const uint4 *st = smem + stage * (UA + UB);
        bf16x8 wv[3][BI], xv[3][BJ];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int bi = 0; bi < BI; ++bi) wv[p][bi] = *reinterpret_cast<const bf16x8 *>(st + aoff[bi] + 2 * p);
#pragma unroll
            for (int bj = 0; bj < BJ; ++bj) xv[p][bj] = *reinterpret_cast<const bf16x8 *>(st + boff[bj] + 2 * p);
        }
        if (more) issue(tn, fill);
        // All reads at once, not as the MFMAs need them: a wavefront that starts
        // its MFMAs sooner only stalls among them (204 -> 199 us on VGG-16's 128 ->
        // 128 layer at 112x112, batch 8).
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_setprio(1);
        constexpr int px[6] = {0, 0, 1, 1, 0, 2}, pw[6] = {0, 1, 0, 1, 2, 0};   // hh, hm, mh, mm, hl, lh
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
                for (int bi = 0; bi < BI; ++bi) {
                    floatx16 &d = q == 0 ? big[bj][bi] : small[q % NS][bj][bi];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[px[q]][bj], wv[pw[q]][bi], d, 0, 0, 0);
                }
        __builtin_amdgcn_s_setprio(0);
    };

    const int n = t_end > t_begin ? t_end - t_begin : 0;
#pragma unroll
    for (int t = 0; t < NST - 1; ++t)
        if (t < n) issue(t_begin + t, t);
    int stage = 0, fill = NST - 1;                      // stage of chunk t, and of chunk t + NST - 1
    for (int t = 0; t < n; ++t) {
        // chunk t has landed once only the later chunks' loads are outstanding
        if (n - 1 - t >= NST - 2)
            wait_vmcnt<(NST - 2) * LOADS>();
        else
            wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // for every lane; and chunk t-1 is done with
        compute(stage, t + NST - 1 < n, t_begin + t + NST - 1, fill);
        stage = stage + 1 == NST ? 0 : stage + 1;
        fill = fill + 1 == NST ? 0 : fill + 1;
    }

    // Epilogue through LDS, channel-major, so that rows leave as contiguous
    // 16-byte stores: both accumulators in one, at the values' own scale.
    __syncthreads();
    float *ot = reinterpret_cast<float *>(smem);
    bool bad = false;
    const auto at = [&](int bj, int bi, int q4) {           // four pixels of a filter
        return ot + (wch * TCH + bi * 32 + ll) * OP + wpx * TPX + bj * 32 + 8 * q4 + 4 * h;
    };
#pragma unroll
    for (int bi = 0; bi < BI; ++bi)
#pragma unroll
        for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                float v4[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float sm = small[0][bj][bi][4 * q4 + e];
                    if constexpr (NS == 2) sm += small[1][bj][bi][4 * q4 + e];
                    v4[e] = (big[bj][bi][4 * q4 + e] + sm) * (kScaleDown * kScaleDown);
                    bad |= !(fabsf(v4[e]) < __builtin_inff());
                }
                *reinterpret_cast<float4 *>(at(bj, bi, q4)) = make_float4(v4[0], v4[1], v4[2], v4[3]);
            }
    if (__builtin_expect(__ballot(bad) != 0, 0)) {          // each lane's own sums, where they are not finite
        floatx16 sum[BJ][BI];
        plain_sums<BJ, BI>(sa, g, m0 + wpx * TPX, k0 + wch * TCH, t_begin, t_end, sum);
#pragma unroll
        for (int bj = 0; bj < BJ; ++bj)
#pragma unroll
            for (int bi = 0; bi < BI; ++bi)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float *o = at(bj, bi, v / 4) + v % 4;
                    if (!(fabsf(*o) < __builtin_inff())) *o = sum[bj][bi][v];
                }
    }
    __syncthreads();
    const bool split_out = a.splits > 1;
    float *out = split_out ? a.ws + (long)split * a.K * a.M : a.y;
    const bool vec = split_out ? (a.M & 3) == 0 : ((a.PQ & 3) == 0 && ((uintptr_t)a.y & 15) == 0 && (a.ysn & 3) == 0);
    constexpr int C4 = BPX / 4;
    constexpr int KS = NT / C4;                         // filter rows per pass of the work-group
    const int c4 = tid % C4;
    const int m = m0 + 4 * c4;
    if (m >= a.M) return;
    const int im = split_out ? 0 : (int)fdiv(m, a.dv_pq);
    const long kstride = split_out ? (long)a.M : (long)a.PQ;
    const long base = split_out ? (long)m : (long)im * a.ysn + (m - im * a.PQ);
    const bool quad = vec && m + 3 < a.M;               // in one image plane (P*Q % 4 == 0)
#pragma unroll 4
    for (int kl = tid / C4; kl < BKC; kl += KS) {
        const int k = k0 + kl;
        if (k >= a.Kg) break;
        const int kg = g * a.Kg + k;
        const float4 v = *reinterpret_cast<const float4 *>(ot + kl * OP + 4 * c4);
        float ve[4] = {v.x, v.y, v.z, v.w};
        const float bv = !split_out && a.bias ? a.bias[kg] : 0.f;
        if (quad) {
            const long off = base + kg * kstride;
            if (!split_out) {
                float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
                if (a.res) r = *reinterpret_cast<const float4 *>(a.res + off);
                const float re[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    ve[e] += bv;
                    if (a.res) ve[e] += re[e];
                    if (a.relu) ve[e] = fmaxf(ve[e], 0.f);
                }
            }
            *reinterpret_cast<float4 *>(out + off) = make_float4(ve[0], ve[1], ve[2], ve[3]);
            continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int mm = m + e;
            if (mm >= a.M) break;
            const int ne = split_out ? 0 : (int)fdiv(mm, a.dv_pq);
            const long off = split_out ? (long)kg * a.M + mm : (long)ne * a.ysn + (long)kg * a.PQ + (mm - ne * a.PQ);
            float val = ve[e];
            if (!split_out) {
                val += bv;
                if (a.res) val += a.res[off];
                if (a.relu) val = fmaxf(val, 0.f);
            }
            out[off] = val;
        }
    }
}

// Tiles, and what one costs on this part (us, fitted to 600 timings of 46
// layer shapes from 0.4 to 40 GFLOP; the tile and split the model picks are
// within 1.3% of the fastest of those tried on average): `alone` per chunk for
// a work-group that has its CU to itself (latency: barrier, LDS reads,
// requests and MFMAs one after the other), `share` per chunk and work-group
// on a full CU, and a tile's `fixed` prologue and epilogue.
struct TileS {
    int bpx, bkc, wpx, wch, nst;
    double alone, share, fixed;
};
const TileS kTilesS[] = {
    {128, 128, 2, 2, 3, 0.83, 0.50, 3.9},   // 72 KB of LDS: two work-groups per CU, as every tile but the last
    {256, 64, 4, 1, 2, 0.96, 0.59, 3.3},
    {128, 64, 2, 2, 3, 0.57, 0.34, 3.4},
    {64, 128, 2, 2, 3, 0.55, 0.32, 3.6},
    {64, 64, 2, 2, 3, 0.43, 0.22, 1.7},     // 48 KB: three
};

int chunk_blocks(const ConvProblem &p) { return ceil_div(p.Cg, 16); }

long xs_bytes_of(const ConvProblem &p) { return (long)p.N * p.H * p.W * p.groups * chunk_blocks(p) * 96; }

}  // namespace

size_t split3_packed_bytes(const ConvProblem &p)
{
    return (size_t)p.groups * ceil_div(p.Kg, 64) * chunk_blocks(p) * p.R * p.S * 6144;
}

// The cheapest tile and split by the model above: the copy of x (and, when
// filters are packed per call, theirs) at the 4.6 TB/s it moves; the larger
// of a work-group's own chain of chunks and its CU's share of them; a split's
// reduce launch and its partials' round trip.
SplitPlan plan_split3(const ConvProblem &p, int num_cus, int max_splits, bool pack_per_call)
{
    SplitPlan plan{};
    plan.us = 1e30;
    const int nc = chunk_blocks(p) * p.R * p.S;
    const double bw = 4.6e6;                                  // bytes per us
    const double out = 4.0 * p.K * p.M;
    const double px = (double)p.N * p.H * p.W;
    double prep = 4.5 + (px * p.C * 4 + (double)xs_bytes_of(p)) / bw;
    if (pack_per_call) prep += 3.0 + 1.7 * split3_packed_bytes(p) / bw;
    for (int t = 0; t < (int)(sizeof kTilesS / sizeof *kTilesS); ++t) {
        const TileS &d = kTilesS[t];
        if (p.Kg <= d.bkc / 2 && t != 4) continue;            // over half of the tile would be padding
        const long tiles = (long)ceil_div(p.M, d.bpx) * ceil_div(p.Kg, d.bkc) * p.groups;
        const int most = (int)std::max(1L, std::min({(long)max_splits, (long)nc / 4, 4L * num_cus / tiles}));
        for (int sp = 1; sp <= most; ++sp) {
            const int per = ceil_div(nc, sp);
            if (ceil_div(nc, per) != sp) continue;
            // 32-bit offsets into the partials (splitk_reduce_kernel reads up to 7 planes past them)
            if (sp > 1 && (double)(sp + 7) * out >= 2147483648.0) break;
            const double rounds = (double)((tiles * sp + num_cus - 1) / num_cus);
            const double us = prep + 4.0 + std::max(per * d.alone + d.fixed, rounds * (per * d.share + d.fixed)) +
                              (sp > 1 ? 3.0 + (2 * sp + 1) * out / bw : 0.6 * out / bw);
            if (us < plan.us) {
                plan.us = us;
                plan.tile = t;
                plan.splits = sp;
                plan.per_split = per;
            }
        }
    }
    plan.xs_bytes = (size_t)xs_bytes_of(p);
    plan.partial_bytes = plan.splits > 1 ? (size_t)(plan.splits * out) : 0;
    return plan;
}

// Whether the split kernels serve a layer, against the wave kernel's time:
// 93 TFLOP/s and about 10 us on the layers it runs well; 1.8 times that where
// its reduction is gathered tap by tap (C/groups not a multiple of 8), else
// 1.2 with a stride and 1.4 for filters of several taps read as given instead
// of packed.  Measured on 70 drawn layers of 0.3 to 6 GFLOP: every one the
// rule sends here is faster (64 -> 256 3x3 at 32x32, batch 9, single call:
// 51 -> 32 us; 201 -> 250 3x3 stride 2 at 55x57, batch 6: 129 -> 53 us; 256 ->
// 512 3x3 at 11x12, batch 16, in a stack: 71 -> 50 us); 1x1 layers of few
// filters and layers of 32 filters mostly stay with the wave kernel (512 ->
// 32 3x3 at 51x51, batch 17: 170 us, 237 us here).
bool split3_pays(const ConvProblem &p, const SplitPlan &plan, bool packed)
{
    const bool gather = p.Cg % 8 != 0 && p.Cg > 4;
    const double f = gather ? 1.8 : (p.stride > 1 ? 1.2 : 1.0) * (!packed && p.R * p.S > 1 ? 1.4 : 1.0);
    const double wave = 10.0 + f * 2.0 * p.M * p.K * p.Kred / 93e6 + 4.0 * p.K * p.M / 10e6;
    return plan.us * 1.05 < wave;
}

bool split3_fits(const ConvProblem &p)
{
    // 32-bit offsets into the split copy and the packed filters; below 1.2
    // GFLOP the three launches cost what the matrix cores save (100 -> 120
    // 3x3 stride 2 at 55x57, batch 5, 0.88 GFLOP: 23.4 -> 27.4 us)
    return xs_bytes_of(p) < (1L << 31) && (long)split3_packed_bytes(p) < (1L << 31) &&
           2.0 * p.M * p.K * p.Kred >= 1.2e9;
}

hipError_t launch_pack_split3(const ConvProblem &p, const float *w, void *packed, hipStream_t st)
{
    const long total = (long)(split3_packed_bytes(p) / 48);   // filter halves
    long blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    launch_kernel(split3_pack_kernel, dim3((unsigned)blocks), dim3(256), 0, st, w, static_cast<uint4 *>(packed), p.Kg,
                  p.Cg, p.R * p.S, ceil_div(p.Kg, 64), chunk_blocks(p) * p.R * p.S, total);
    return hipGetLastError();
}

void describe_split3(const ConvProblem &p, const SplitPlan &plan, char *buf, int len, int *launches)
{
    (void)p;
    const TileS &t = kTilesS[plan.tile];
    snprintf(buf, len, "split3_copy_kernel<%d> + igemm_split3_kernel<%d, %d, %d, %d, %d>%s",
             (p.H * p.W) % 4 == 0 ? 4 : 1, t.bpx, t.bkc, t.wpx, t.wch, t.nst, plan.splits > 1 ? " + splitk_reduce_kernel" : "");
    *launches = plan.splits > 1 ? 3 : 2;
}

hipError_t launch_split3(const ConvProblem &p, const SplitPlan &plan, const float *x, const float *w,
                         const void *packed, const float *bias, float *y, void *xs, float *partials, hipStream_t st,
                         const LaunchHook *hook)
{
    hipError_t e = hook ? hook->before_launch(hook->ctx, st) : hipSuccess;
    if (e != hipSuccess) return e;
    SplitCopyArgs ca{};
    ca.x = x;
    ca.xs = static_cast<uint16_t *>(xs);
    ca.C = p.C;
    ca.Cg = p.Cg;
    ca.HW = p.H * p.W;
    ca.CB = chunk_blocks(p);
    ca.npx = p.N * ca.HW;
    ca.blocks = p.groups * ca.CB;
    ca.tiles_c = ceil_div(ca.blocks, 2);
    ca.dv_hw = make_fastdiv(ca.HW);
    ca.dv_cb = make_fastdiv(ca.CB);
    const dim3 cg((unsigned)((long)ceil_div(ca.npx, 64) * ca.tiles_c));
    if (ca.HW % 4 == 0 && (uintptr_t)x % 16 == 0)
        launch_kernel(split3_copy_kernel<4>, cg, dim3(256), 0, st, ca);
    else
        launch_kernel(split3_copy_kernel<1>, cg, dim3(256), 0, st, ca);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (hook && (e = hook->before_launch(hook->ctx, st)) != hipSuccess) return e;

    SplitArgs s{};
    s.a = make_args(p);
    s.a.x = x;
    s.a.w = w;
    s.a.bias = bias;
    s.a.y = y;
    s.a.ws = plan.splits > 1 ? partials : nullptr;
    s.a.splits = plan.splits;
    s.a.kr_per_split = plan.per_split;
    s.xs = static_cast<const uint16_t *>(xs);
    s.wp = static_cast<const uint16_t *>(packed);
    s.CB = ca.CB;
    s.NC = ca.CB * p.R * p.S;
    s.px_bytes = (unsigned)(ca.blocks * 96);
    const TileS &t = kTilesS[plan.tile];
    const dim3 grid((unsigned)((long)ceil_div(p.M, t.bpx) * ceil_div(p.Kg, t.bkc) * p.groups * plan.splits));
    switch (plan.tile) {
    case 0: launch_kernel((igemm_split3_kernel<128, 128, 2, 2, 3>), grid, dim3(256), 0, st, s); break;
    case 1: launch_kernel((igemm_split3_kernel<256, 64, 4, 1, 2>), grid, dim3(256), 0, st, s); break;
    case 2: launch_kernel((igemm_split3_kernel<128, 64, 2, 2, 3>), grid, dim3(256), 0, st, s); break;
    case 3: launch_kernel((igemm_split3_kernel<64, 128, 2, 2, 3>), grid, dim3(256), 0, st, s); break;
    default: launch_kernel((igemm_split3_kernel<64, 64, 2, 2, 3>), grid, dim3(256), 0, st, s); break;
    }
    if ((e = hipGetLastError()) != hipSuccess || plan.splits == 1) return e;
    if (hook && (e = hook->before_launch(hook->ctx, st)) != hipSuccess) return e;
    return launch_splitk_reduce(s.a, st);
}

}  // namespace miconv
