// batch_multi.h -- several steps per launch for the batched 16-bit members.
//
// A tick of a class on these kernels is one single step (it also reads members
// that start from the natural layout), launches of four (2D) or two (3D) steps
// on the tilings of march2d.h and pair3d.h, and single steps for what is left
// of each member.  Work items of all members are numbered by multi_base; the
// rows and planes per chunk are those of the group, so that its members
// together fill the GPU.  A member with too few steps left skips a launch.
#pragma once
#include "pair3d.h"

namespace lbem {

// launch j: steps 1 + 4j .. 4 + 4j of the tick
template <typename H, bool GH, bool MU>
__global__ __launch_bounds__(NT) void k_batch_march2d(const BatchHdr* __restrict__ hdr,
                                                     const BatchGrid* __restrict__ tab, const int j)
{
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (NT / 64)) + (int)(threadIdx.x >> 6));
    if (w >= hdr->total_multi) return;
    const BatchGrid& G = tab[batch_find<&BatchGrid::multi_base>(tab, hdr->count, w)];
    if (G.nsteps - 1 < 4 * (j + 1)) return;
    const int s = (G.cur0 + 1 + j) & 1;
    typedef MarchDev<H, GH, 1> IO;
    const IO io{gmem<const float>(G.buf[s]), gmem<const H>(G.dev[s]), gmem<float>(G.buf[s ^ 1]),
                gmem<H>(G.dev[s ^ 1]), G.mgeo.n};
    const MarchGeo g = G.mgeo;
    MarchSrc<float> ms;
    ms.idx = gmem<const int>(G.msrc_idx);
    ms.val = gmem<const float>(G.msrc_val);
#pragma unroll
    for (int k = 0; k < 8; ++k) ms.mask[k] = G.msrc_mask[k];
    AmpPack<float, 4> a;
#pragma unroll
    for (int k = 0; k < 4; ++k) a.a[k] = G.amp ? gmem<const float>(G.amp)[1 + 4 * j + k] : 0.f;
    march2d_work<IO, 4, 1, MU, false>(io, gmem<const float>(G.cl2), MU ? gmem<const float>(G.dlnmu) : nullptr, g, ms, a,
                                      (float)G.omega, G.tau_half != 0, w - G.multi_base);
}

// launch j: steps 1 + 2j and 2 + 2j of the tick
template <typename H, bool GH, bool MU>
__global__ __launch_bounds__(1024, 4) void k_batch_pair3d(const BatchHdr* __restrict__ hdr,
                                                         const BatchGrid* __restrict__ tab, const int j)
{
    __shared__ float ly[2][2][6][1024];
    const int b = blockIdx.x;
    if (b >= hdr->total_multi) return;
    const BatchGrid& G = tab[batch_find<&BatchGrid::multi_base>(tab, hdr->count, b)];
    if (G.nsteps - 1 < 2 * (j + 1)) return;
    const int s = (G.cur0 + 1 + j) & 1;
    const PairGeo g = G.pgeo;
    // a member's tiles are dealt to the XCDs as the solo launch deals them (its first
    // block may run on any of the 8)
    const int t = remap_block(b - G.multi_base, g.nblocks, g.xcd), tx = t % g.tiles_x, r = t / g.tiles_x;
    const int y0 = (r % g.tiles_y) * g.sy, z0 = (r / g.tiles_y) * g.lz;
    const PairSrc ps{nullptr, gmem<const int>(G.psrc_idx), gmem<const float>(G.psrc_val), G.psrc_pair};
    AmpPack<float, 2> a;
#pragma unroll
    for (int k = 0; k < 2; ++k) a.a[k] = G.amp ? gmem<const float>(G.amp)[1 + 2 * j + k] : 0.f;
    const float* dl = MU ? gmem<const float>(G.dlnmu) : nullptr;
    if (G.psrc_idx != nullptr)
        pair_march<H, GH, MU, true>(gmem<const float>(G.buf[s]), gmem<const H>(G.dev[s]), gmem<float>(G.buf[s ^ 1]),
                                    gmem<H>(G.dev[s ^ 1]), gmem<const float>(G.cl2), dl, g, ps, a, (float)G.omega,
                                    G.tau_half != 0, tx, y0, z0, ly);
    else
        pair_march<H, GH, MU, false>(gmem<const float>(G.buf[s]), gmem<const H>(G.dev[s]), gmem<float>(G.buf[s ^ 1]),
                                     gmem<H>(G.dev[s ^ 1]), gmem<const float>(G.cl2), dl, g, ps, a, (float)G.omega,
                                     G.tau_half != 0, tx, y0, z0, ly);
}

}  // namespace lbem
