// pair3f.h -- 3D FP32, two time steps per launch, with the cell-local extras.
//
// The march of pair3d.h for populations held as they are: a block of 16 waves
// owns 64 columns (the lanes) and marches along z.  15 waves hold a row each,
// 13 of them stored; the last wave holds the two columns beside the tile.  Each
// iteration pulls one plane of the stored state and takes the first step on it
// (level 1), then the second on the plane before (level 2).  Between the levels
// the rest and +-x populations stay in registers (+-x cross lanes by DPP wave
// shifts, the outermost from the side columns through LDS), +z for two planes,
// -z is handed over in the same iteration, and +-y go through LDS, two buffers,
// one barrier per plane.  The arithmetic is the single-step kernels', so two
// single steps and one launch give the same bits.
//
// Why this shape: rows of 64 start and end on whole lines where the lattice's
// do, for one wave of scattered loads; with the side columns in the lanes (62 x
// 14 stored) every row straddled three lines and half of the stores two tiles
// (256^3 502 us per step, here 303).  One block per CU, 96-126 of 128 VGPRs, so
// the next plane is loaded before level 2 runs.  Bound by memory: 198 B counted
// per cell and two steps at 512^3 (172 without halos), 5.5 TB/s; us per step,
// column tiles of k_step_fused3d (two blocks per CU, all exchange through LDS) ->
// these: 512^3 2529 -> 2422, 160^3 97 -> 88, 250x190x171 212 -> 172, but 256^3 302 /
// 299 and 257^3, whose last tile is one column, 483 / 518.
//
// EXT: an absorbing layer and the dispersion pole.  P and J of a cell advance
// with it: level 1 reads them from one buffer, keeps the new pair in registers
// for level 2, and level 2 writes the other buffer (neighbouring tiles still
// read the old values of their halo).  Per step a pole reads and writes 60 B per
// cell, an absorber 4; single steps add 168.  us per step, single -> this
// kernel: pole 160^3 153 -> 124, 256^3 683 -> 432; absorber 256^3 478 -> 318.
// A block with source cells runs 5 % longer.
#pragma once
#include "pair3d.h"

namespace lbem {

constexpr int PFX = 64, PFY = 13;        // most columns and rows that a tile stores
constexpr int PFW = PFY + 3;             // waves: the stored rows, one on each side, and the side columns
constexpr int PFSEG = PFX + 2;           // columns of a source segment: x0-1 .. x0+64

// the value of one lane in all of them
__device__ __forceinline__ float lane_of(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

struct PairExt {
    const float* keep;                   // per-cell 1 - sigma, or nullptr
    const float* ade;                    // [3][n] c1, c2, c3, or nullptr
    const float* pin;                    // [2P][n] P_p then J_p
    float* pout;
};

template <bool MU, bool EXT, bool TH, bool NTS, bool SRC>
__device__ __forceinline__ void pair_march_f(const float* src, float* dst, const float* cl2a, const float* dlnmu,
                                             const PairGeo& g, const PairSrc& ps, const AmpPack<float, 2>& amps,
                                             const float omega, const bool tau_half, const PairExt& ex, const int tx,
                                             const int y0, const int z0, float (&ly)[2][6][1024],
                                             float (&lx)[2][2][3][16])
{
    constexpr int D = 3, Q = 7, P = 3;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int tid = threadIdx.x;
    const int x0 = tx * g.sx;
    const int planes = min(g.lz, g.nz - z0);
    const int width = min(g.sx, g.nx - x0);
    auto wrap = [](int v, int m) { v %= m; return v < 0 ? v + m : v; };
    // this thread's cell: row waves hold row y0-1+w, the last wave the columns
    // x0-1 (lanes 0..31) and x0+width (lanes 32..63) of the stored rows
    const bool sides = w == PFW - 1;
    const bool right = sides && lane >= 32;
    const int row = sides ? lane & 31 : w;
    const int gx = wrap(sides ? (right ? x0 + width : x0 - 1) : x0 + lane, g.nx);
    const int gy = wrap(y0 - 1 + row, g.ny);
    const bool live = sides ? g.tiles_x > 1 && row >= 1 && row <= g.sy && y0 - 1 + row < g.ny
                            : row <= g.sy + 1 && lane < width;
    const bool inner = !sides && w >= 1 && w <= g.sy && y0 - 1 + w < g.ny;   // rows that take both steps
    const bool keep = inner && lane < width;
    const int64_t nxy = (int64_t)g.nx * g.ny;
    const unsigned ro = (unsigned)gy * g.nx, c0 = ro + gx;
    const unsigned cxm = ro + (gx == 0 ? g.nx - 1 : gx - 1), cxp = ro + (gx == g.nx - 1 ? 0 : gx + 1);
    const unsigned cym = (unsigned)(gy == 0 ? g.ny - 1 : gy - 1) * g.nx + gx;
    const unsigned cyp = (unsigned)(gy == g.ny - 1 ? 0 : gy + 1) * g.nx + gx;
    const bool pole = EXT && ex.ade != nullptr, damp = EXT && ex.keep != nullptr;

    float f[Q][P] = {}, cl = 1.f, sv = 0.f;
    float ca[3] = {}, po[P] = {}, jo[P] = {}, kp = 1.f;
    int seg = -1;                        // source segment of the plane loaded next
    auto fetch = [&](const int z) {
        const int64_t zo = (int64_t)z * nxy, zm = (int64_t)(z == 0 ? g.nz - 1 : z - 1) * nxy,
                      zp = (int64_t)(z == g.nz - 1 ? 0 : z + 1) * nxy;
        unsigned c = c0, xm = cxm, xp = cxp, ym = cym, yp = cyp;
        asm volatile("" : "+v"(c), "+v"(xm), "+v"(xp), "+v"(ym), "+v"(yp));
#pragma unroll
        for (int p = 0; p < P; ++p) {
            f[0][p] = at32(src + (int64_t)(0 * P + p) * g.n + zo, c);
            f[1][p] = at32(src + (int64_t)(1 * P + p) * g.n + zo, xm);
            f[2][p] = at32(src + (int64_t)(2 * P + p) * g.n + zo, ym);
            f[3][p] = at32(src + (int64_t)(3 * P + p) * g.n + zm, c);
            f[4][p] = at32(src + (int64_t)(4 * P + p) * g.n + zo, xp);
            f[5][p] = at32(src + (int64_t)(5 * P + p) * g.n + zo, yp);
            f[6][p] = at32(src + (int64_t)(6 * P + p) * g.n + zp, c);
        }
        cl = at32(cl2a + zo, c);
        if constexpr (EXT) {
            if (pole) {
#pragma unroll
                for (int k = 0; k < 3; ++k) ca[k] = at32(ex.ade + (int64_t)k * g.n + zo, c);
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    po[p] = at32(ex.pin + (int64_t)p * g.n + zo, c);
                    jo[p] = at32(ex.pin + (int64_t)(P + p) * g.n + zo, c);
                }
            }
            if (damp) kp = at32(ex.keep + zo, c);
        }
        if constexpr (SRC) {
            // the segment of a plane is looked up one plane ahead
            sv = seg >= 0 ? ps.val[(int64_t)seg * PFSEG + (sides ? (right ? width + 1 : 0) : lane + 1)] : 0.f;
            seg = ps.idx[((int64_t)tx * g.nz + (z == g.nz - 1 ? 0 : z + 1)) * g.ny + gy];
        }
    };
    // one step of a cell: `f` arrived, P and J advance in place
    auto update = [&](const float (&fi)[Q][P], float cl2, float s_, int z, const float (&cc)[3], float (&Pp)[P],
                      float (&Jp)[P], float k, float (&out)[Q][P]) {
        float rho[P], K[D], Sp[P];
        moments<D, float>(fi, rho, K);
#pragma unroll
        for (int p = 0; p < P; ++p) Sp[p] = SRC && p == ps.pair ? s_ : 0.f;
        if constexpr (MU) {
            const int64_t o = (int64_t)wrap(z, g.nz) * nxy;
            float dl[D];
#pragma unroll
            for (int a = 0; a < D; ++a) dl[a] = at32(dlnmu + (int64_t)a * g.n + o, c0);
            add_mu_source<D, float>(K, cl2, dl, Sp);
        }
        if constexpr (EXT) {
            if (pole) {
#pragma unroll
                for (int p = 0; p < P; ++p) ade_advance<float>(cc[0], cc[1], cc[2], cl2, rho[p], Pp[p], Jp[p]);
            }
        }
        collide<D, float>(fi, cl2, Sp, SRC || MU, omega, TH || tau_half, rho, K, out);
        if constexpr (EXT) {
            if (pole) {
#pragma unroll
                for (int p = 0; p < P; ++p) out[0][p] += Jp[p] / cl2;
            }
            if (damp) {
#pragma unroll
                for (int i = 0; i < Q; ++i)
#pragma unroll
                    for (int p = 0; p < P; ++p) out[i][p] *= k;
            }
        }
    };
    // of the plane of level 2: what it left behind, +z of the last two planes
    float rest[P] = {}, px[P] = {}, mx[P] = {}, pz[P] = {}, pzo[P] = {};
    float cl1 = 1.f, sv1 = 0.f, ca1[3] = {}, p1[P] = {}, j1[P] = {}, kp1 = 1.f;
    int gz = wrap(z0 - 1, g.nz);         // the plane loaded last
    if constexpr (SRC) seg = ps.idx[((int64_t)tx * g.nz + gz) * g.ny + gy];
    if (live) fetch(gz);
    for (int it = 0; it < planes + 2; ++it) {
        // level 1 on plane z0-1+it, level 2 on the one before
        const int bw = it & 1, br = bw ^ 1;
        float out[Q][P] = {};
        const float cl0 = cl, sv0 = sv, kp0 = kp;
        float ca0[3], p0[P], j0[P];
#pragma unroll
        for (int k = 0; k < 3; ++k) ca0[k] = ca[k];
#pragma unroll
        for (int p = 0; p < P; ++p) { p0[p] = po[p]; j0[p] = jo[p]; }
        gz = gz + 1 == g.nz ? 0 : gz + 1;
        if (live) {
            update(f, cl0, SRC ? source_term(sv0, amps.a[0]) : 0.f, z0 - 1 + it, ca0, p0, j0, kp0, out);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (sides) {
                    lx[bw][right][p][row] = right ? out[4][p] : out[1][p];
                } else {
                    ly[bw][p][tid] = out[2][p];
                    ly[bw][P + p][tid] = out[5][p];
                }
            }
            if (it + 1 < planes + 2) fetch(gz);
        }
        if (it >= 2 && inner) {
            float f2[Q][P], o2[Q][P];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                f2[0][p] = rest[p];
                const float xl = lane_shift<1>(px[p]), xr = lane_shift<-1>(mx[p]);
                f2[1][p] = lane == 0 ? (g.tiles_x > 1 ? lx[br][0][p][w] : lane_of(px[p], width - 1)) : xl;
                f2[2][p] = ly[br][p][tid - 64];
                f2[3][p] = pzo[p];
                f2[4][p] = lane == width - 1 ? (g.tiles_x > 1 ? lx[br][1][p][w] : lane_of(mx[p], 0)) : xr;
                f2[5][p] = ly[br][P + p][tid + 64];
                f2[6][p] = out[6][p];
            }
            update(f2, cl1, SRC ? source_term(sv1, amps.a[1]) : 0.f, z0 - 2 + it, ca1, p1, j1, kp1, o2);
            const int64_t o = (int64_t)(z0 - 2 + it) * nxy;
            if (keep) {
                unsigned c = c0;
                asm volatile("" : "+v"(c));
#pragma unroll
                for (int i = 0; i < Q; ++i)
#pragma unroll
                    for (int p = 0; p < P; ++p) st_stream<NTS>(&at32(dst + (int64_t)(i * P + p) * g.n + o, c), o2[i][p]);
                if constexpr (EXT) {
                    if (pole) {
#pragma unroll
                        for (int p = 0; p < P; ++p) {
                            at32(ex.pout + (int64_t)p * g.n + o, c) = p1[p];
                            at32(ex.pout + (int64_t)(P + p) * g.n + o, c) = j1[p];
                        }
                    }
                }
            }
        }
        // the march moves on one plane
#pragma unroll
        for (int p = 0; p < P; ++p) {
            rest[p] = out[0][p];
            px[p] = out[1][p];
            mx[p] = out[4][p];
            pzo[p] = pz[p];
            pz[p] = out[3][p];
            p1[p] = p0[p];
            j1[p] = j0[p];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) ca1[k] = ca0[k];
        cl1 = cl0; sv1 = sv0; kp1 = kp0;
        __syncthreads();
    }
}

template <bool MU, bool EXT, bool TH, bool NTS>
__global__ __launch_bounds__(1024, 4) void k_pair_f32(const float* src, float* dst, const float* cl2a,
                                                     const float* dlnmu, const PairGeo g, const PairSrc ps,
                                                     const AmpPack<float, 2> amps, const float omega,
                                                     const int tau_half, const PairExt ex)
{
    __shared__ float ly[2][6][1024];     // [buffer][+y 0..2, -y 3..5][row * 64 + lane]
    __shared__ float lx[2][2][3][16];    // [buffer][left, right][pair][row]
    const int b = remap_block(blockIdx.x, g.nblocks, g.xcd);
    const int tx = b % g.tiles_x, r = b / g.tiles_x;
    const int ty = r % g.tiles_y, zc = r / g.tiles_y;
    if (ps.flag != nullptr && ps.flag[b] != 0)
        pair_march_f<MU, EXT, TH, NTS, true>(src, dst, cl2a, dlnmu, g, ps, amps, omega, tau_half != 0, ex, tx, ty * g.sy,
                                             zc * g.lz, ly, lx);
    else
        pair_march_f<MU, EXT, TH, NTS, false>(src, dst, cl2a, dlnmu, g, ps, amps, omega, tau_half != 0, ex, tx, ty * g.sy,
                                              zc * g.lz, ly, lx);
}

}  // namespace lbem
