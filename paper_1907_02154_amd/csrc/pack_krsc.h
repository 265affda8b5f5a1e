// bf16 KCRS filters -> the KRSC orders of pack.hip, as a work-group's body: run
// by pack_krsc_run_kernel, and by the first work-groups of the channel-last
// copy where one call needs both.
#pragma once

#include "internal.h"

namespace miconv {

constexpr int kPackRS = 25;                          // taps, at most (pack_krsc_runs)
constexpr int kPackTile = 64 * kPackRS;              // LDS values per wavefront: 3.2 KB

struct PackRuns {
    const uint16_t *src;
    uint16_t *dst;
    int units, blocks;   // runs of up to 64 channels of one filter; work-groups, four runs each
    int Cg, RS, cblk;
    int vec;             // src is 16-byte aligned
};

inline PackRuns make_pack_runs(const ConvProblem &p, const uint16_t *src, uint16_t *dst, int cblk)
{
    PackRuns r{};
    r.src = src;
    r.dst = dst;
    r.units = p.K * ceil_div(p.Cg, 64);
    r.blocks = (r.units + 3) / 4;
    r.Cg = p.Cg;
    r.RS = p.R * p.S;
    r.cblk = cblk > 0 ? cblk : p.Cg;
    r.vec = (uintptr_t)src % 16 == 0 ? 1 : 0;
    return r;
}

// One wavefront per run: up to 64 channels of one filter are a contiguous run
// of the source, turned through LDS into RS contiguous runs of the destination,
// both with 16-byte accesses (2-byte loads where the source is not aligned).
// Gathering 2 bytes per lane behind three divisions, as pack_krsc_kernel does,
// took 5.0 us for 256 -> 256 3x3 filters (1.2 MB) and 11.8 us for 512 -> 512
// (4.7 MB); here 3.8 and 4.4 us, mostly the launch and one round trip.
// cblk is Cg or a multiple of 64.  tile: 4 * kPackTile values of LDS.
__device__ __forceinline__ void pack_krsc_run(const PackRuns &a, int block, uint16_t *tile)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int u = block * 4 + wv;
    uint16_t *t = tile + wv * kPackTile;
    const int nb = (a.Cg + 63) / 64;
    const int k = u / nb, c0 = (u - k * nb) * 64;
    const int n = min(64, a.Cg - c0);                // channels of this run, a multiple of 8
    if (u < a.units) {
        const uint16_t *s = a.src + ((long)k * a.Cg + c0) * a.RS;
        if (a.vec) {
            for (int i = lane; i < n * a.RS / 8; i += 64)
                reinterpret_cast<uint4 *>(t)[i] = reinterpret_cast<const uint4 *>(s)[i];
        } else {
            for (int i = lane; i < n * a.RS; i += 64) t[i] = s[i];
        }
    }
    __syncthreads();
    if (u >= a.units) return;
    const int no = n / 8;                            // octets per tap
    // a tap's channels lie cblk apart from the next tap's
    uint16_t *d = a.dst + (long)k * a.Cg * a.RS + (long)(c0 / a.cblk) * a.cblk * a.RS + c0 % a.cblk;
    for (int i = lane; i < no * a.RS; i += 64) {
        const int rs = i / no, o = i - rs * no;
        const uint16_t *q = t + 8 * o * a.RS + rs;
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = q[2 * e * a.RS] | (uint32_t)q[(2 * e + 1) * a.RS] << 16;
        *reinterpret_cast<uint4 *>(d + (long)rs * a.cblk + 8 * o) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

}  // namespace miconv
