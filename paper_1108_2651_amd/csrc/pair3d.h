// pair3d.h -- 3D 16-bit formats, two time steps per launch.
//
// A block of 16 waves owns a tile of 64 columns (the lanes) by 16 rows (the
// waves) and marches along z.  Iteration it decodes plane z0-2+it of the
// stored state once (level 0), takes the first step on the plane before
// (level 1: collide, encode as it would be stored, decode that as every reader
// would) and the second on the one before that (level 2: collide, encode,
// store).  Between the levels the rest and +-x populations stay in registers
// (+-x cross lanes by DPP wave shifts), +z for two planes, -z is handed over in
// the same iteration, and +-y go through LDS, two buffers, one barrier per
// plane.  The two outer columns and rows on each side are recomputed by the
// neighbouring tiles: up to 60 x 12 cells are stored, the lattice cut into even
// tiles (with full tiles and a rest the lanes of the last one load again what
// others hold: ten steps of FP16 ghost 512^3 26.9 ms, even tiles of 57 x 12
// 25.2); the outermost rows load and decode only what their +-y populations
// need.  The arithmetic is the
// single-step kernels', so two single steps and one launch give the same bits.
//
// Why this shape: the persistent state of a cell between planes is 40 floats,
// so one cell per thread and 1024 threads fill the registers of a CU (118-128
// of 128 VGPRs); a narrower or lower tile recomputes and re-reads more.  What
// bounds it: L1 -> L2 requests (0.12 per cycle and CU, the rate of every 3D
// kernel here) and bytes: counted traffic of 147 B per cell and two steps at
// 512^3, 4.62 TB/s, the rate of a large copy, against 254 B of two single
// steps.  With every plane the same (no traffic beyond L2) a launch there takes
// 2.67 of its 4.27 ms.  Stores are plain: the partial lines at tile edges
// merge in L2 (streaming stores ran 5.7 against 4.4 ms, on full tiles).  Tiles are dealt to
// the XCDs in runs of one row of tiles, which share their x-halo lines (512^3,
// us per launch, runs of 0 / 1 / 3 / 9 tiles: 5350 / 5340 / 4810 / 4360).
// Measured, us per step, row tiles (one step per launch) -> this kernel: FP16
// ghost 512^3 2890 -> 2135, 256^3 370 -> 316, 160^3 105 -> 72, 250x190x171 274
// -> 133; FP16-dev 256^3 438 -> 374, 250x190x171 358 -> 163.
#pragma once
#include "march2d.h"

namespace lbem {

// Element idx of a row: a 32-bit offset off a scalar base.
template <typename T>
__device__ __forceinline__ T& at32(T* base, unsigned idx)
{
    return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + idx * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ const T& at32(const T* base, unsigned idx)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + idx * (unsigned)sizeof(T));
}

constexpr int PRX = 60, PRY = 12;        // most columns and rows that a tile stores (64 lanes x 16 waves)

struct PairSrc {
    const unsigned char* flag;           // per block: some row it updates holds source cells (nullptr: no source)
    const int* idx;                      // [tile_x][z][y]: segment of the 64 columns of that strip's row, or -1
    const float* val;                    // segments: S per unit amplitude
    int pair;                            // the pair that carries it
};

// whether stored code s takes part in decoding a +y or -y population
template <bool GH>
__host__ __device__ constexpr bool pair_edge_code(int s)
{
    for (int i = 1; i < 7; ++i)
        for (int p = 0; p < 3; ++p) {
            if (dev_slot<3, GH>(i, p) != s) continue;
            if (i == 2 || i == 5) return true;
            for (int j = 2; j <= 5; j += 3)
                for (int q = 0; q < 3; ++q) {
                    const int e = GH ? ghost_dropped_by(3, j, q) : -1;
                    if (e >= 0 && kcoef(3, i, p, e) != 0) return true;
                }
        }
    return false;
}

// One tile and chunk.  SRC: the block holds source cells.
template <typename H, bool GH, bool MU, bool SRC>
__device__ __forceinline__ void pair_march(const float* Min, const H* Din, float* Mout, H* Dout, const float* cl2a,
                                           const float* dlnmu, const PairGeo& g, const PairSrc& ps,
                                           const AmpPack<float, 2>& amps, const float omega, const bool tau_half,
                                           const int tx, const int y0, const int z0, float (&ly)[2][2][6][1024])
{
    constexpr int D = 3, Q = 7, P = 3, NM = 6, NC = DevSlots<D, GH>::N;
    constexpr bool RW = !GH;             // the reciprocal of w0/c^2 is kept for the rest codes
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int tid = threadIdx.x;
    const int x0 = tx * g.sx;
    const int planes = min(g.lz, g.nz - z0);
    auto wrap = [](int v, int m) { v %= m; return v < 0 ? v + m : v; };
    const unsigned col0 = (unsigned)wrap(x0 - 2 + lane, g.nx);
    const int gy = wrap(y0 - 2 + w, g.ny);
    const int64_t nxy = (int64_t)g.nx * g.ny, rowo = (int64_t)gy * g.nx;
    const bool live = w < g.sy + 4, col = lane < g.sx + 4;   // the tile and its halo
    const bool edge = w == 0 || w >= g.sy + 3;         // rows decoded for their +y / -y populations only
    const bool inner = w >= 2 && w < 2 + g.sy;         // rows that take both steps and are stored
    const bool keep = inner && lane >= 2 && lane < 2 + g.sx && x0 - 2 + lane < g.nx && y0 - 2 + w < g.ny;

    float m[NM] = {}, cl = 1.f, sv = 0.f;
    H cd[NC] = {};
    int gz = wrap(z0 - 2, g.nz);
    auto fetch = [&]() {
        const int64_t o = (int64_t)gz * nxy + rowo;
        if (col) {
            unsigned c = col0;
            asm volatile("" : "+v"(c));
#pragma unroll
            for (int t = 0; t < NM; ++t) m[t] = at32(Min + (int64_t)t * g.n + o, c);
#pragma unroll
            for (int s = 0; s < NC; ++s)
                if (pair_edge_code<GH>(s)) cd[s] = at32(Din + (int64_t)s * g.n + o, c);
            if (!edge) {
#pragma unroll
                for (int s = 0; s < NC; ++s)
                    if (!pair_edge_code<GH>(s)) cd[s] = at32(Din + (int64_t)s * g.n + o, c);
                cl = at32(cl2a + o, c);
            }
        }
        if constexpr (SRC) {
            const int seg = ps.idx[((int64_t)tx * g.nz + gz) * g.ny + gy];
            sv = seg >= 0 ? ps.val[(int64_t)seg * 64 + lane] : 0.f;
        }
        gz = gz + 1 == g.nz ? 0 : gz + 1;
    };
    // what a level leaves for the next: rest and +-x of its newest plane, +z of
    // the last two
    struct Left { float rest[P], px[P], mx[P], pz[P], pzo[P]; };
    Left L0, L1;
    float cl1 = 1.f, wc1 = 0.f, rw1 = 0.f, sv1 = 0.f;  // coefficients of the plane of level 1
    float cl2 = 1.f, wc2 = 0.f, rw2 = 0.f, sv2 = 0.f;  // and of level 2
#pragma unroll
    for (int p = 0; p < P; ++p) {
        L0.rest[p] = L0.px[p] = L0.mx[p] = L0.pz[p] = L0.pzo[p] = 0.f;
        L1.rest[p] = L1.px[p] = L1.mx[p] = L1.pz[p] = L1.pzo[p] = 0.f;
    }
    // the populations of a cell from its moments and codes: +-y to LDS, the
    // others (full) to L and -z to mz
    auto spread = [&](const float (&M)[NM], const H (&code)[NC], float wc0, float (*l)[1024], bool full, Left& L,
                      float (&mz)[P]) {
        const float sc = row_scale(M);
        float cf[NC];
#pragma unroll
        for (int s = 0; s < NC; ++s) cf[s] = h2f<H>(code[s]);
        auto get = [&](int s) { return cf[s]; };
#pragma unroll
        for (int p = 0; p < P; ++p) {
            l[p][tid] = row_pop<GH>(M, get, sc, wc0, 2, p);
            l[P + p][tid] = row_pop<GH>(M, get, sc, wc0, 5, p);
        }
        if (!full) return;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            L.rest[p] = row_pop<GH>(M, get, sc, wc0, 0, p);
            L.px[p] = row_pop<GH>(M, get, sc, wc0, 1, p);
            L.mx[p] = row_pop<GH>(M, get, sc, wc0, 4, p);
            L.pz[p] = row_pop<GH>(M, get, sc, wc0, 3, p);
            mz[p] = row_pop<GH>(M, get, sc, wc0, 6, p);
        }
    };
    // collide and encode what arrives at a plane: in-plane and +z from L, +-y
    // from l, -z from mz
    auto update = [&](const Left& L, const float (*l)[1024], const float (&mz)[P], float cl_, float wc_, float rw_, float s_, int z, float (&M)[NM], H (&code)[NC]) {
        float f[Q][P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            f[0][p] = L.rest[p];
            f[1][p] = lane_shift<1>(L.px[p]);
            f[2][p] = l[p][tid - 64];
            f[3][p] = L.pzo[p];
            f[4][p] = lane_shift<-1>(L.mx[p]);
            f[5][p] = l[P + p][tid + 64];
            f[6][p] = mz[p];
        }
        float rho[P], K[D], Sp[P];
        moments<D, float>(f, rho, K);
#pragma unroll
        for (int p = 0; p < P; ++p) Sp[p] = SRC && p == ps.pair ? s_ : 0.f;
        if constexpr (MU) {
            const int64_t o = (int64_t)wrap(z, g.nz) * nxy + rowo;
            float dl[D];
#pragma unroll
            for (int a = 0; a < D; ++a) dl[a] = at32(dlnmu + (int64_t)a * g.n + o, col0);
            add_mu_source<D, float>(K, cl_, dl, Sp);
        }
        dev_encode<D, H, GH, RW>(f, cl_, RW ? rw_ : wc_, Sp, SRC || MU, omega, tau_half, rho, K, M, code);
    };
    fetch();
    for (int it = 0; it < planes + 4; ++it) {
        // level 0 on plane z0-2+it, level 1 on the one before, level 2 on the
        // one before that
        const int bw = it & 1, br = bw ^ 1;
        Left N0 = L0, N1 = L1;
        float mz0[P], mz1[P];
        const float cl0 = cl, sv0 = sv, wc0 = 1.f / cl0 - float(D);
        if (live) {
            spread(m, cd, wc0, ly[bw][0], !edge, N0, mz0);
            if (it + 1 < planes + 4) fetch();
        }
        if (it >= 2 && !edge) {
            float M[NM];
            H code[NC];
            update(L0, ly[br][0], mz0, cl1, wc1, rw1, SRC ? source_term(sv1, amps.a[0]) : 0.f, z0 - 3 + it, M, code);
            spread(M, code, wc1, ly[bw][1], inner, N1, mz1);
        }
        if (it >= 4 && inner) {
            float M[NM];
            H code[NC];
            update(L1, ly[br][1], mz1, cl2, wc2, rw2, SRC ? source_term(sv2, amps.a[1]) : 0.f, z0 - 4 + it, M, code);
            const int64_t o = (int64_t)(z0 - 4 + it) * nxy + rowo;
            if (keep) {
                unsigned col = col0;
                asm volatile("" : "+v"(col));
#pragma unroll
                for (int t = 0; t < NM; ++t) at32(Mout + (int64_t)t * g.n + o, col) = M[t];
#pragma unroll
                for (int s = 0; s < NC; ++s) at32(Dout + (int64_t)s * g.n + o, col) = code[s];
            }
        }
        // the march moves on one plane
#pragma unroll
        for (int p = 0; p < P; ++p) {
            N0.pzo[p] = L0.pz[p];
            N1.pzo[p] = L1.pz[p];
        }
        L0 = N0;
        L1 = N1;
        cl2 = cl1; wc2 = wc1; sv2 = sv1;
        cl1 = cl0; wc1 = wc0; sv1 = sv0;
        if constexpr (RW) {
            rw2 = rw1;
            rw1 = 1.f / wc0;
        }
        __syncthreads();
    }
}

template <typename H, bool GH, bool MU>
__global__ __launch_bounds__(1024, 4) void k_pair_dev3(const float* Min, const H* Din, float* Mout, H* Dout,
                                                      const float* cl2a, const float* dlnmu, const PairGeo g,
                                                      const PairSrc ps, const AmpPack<float, 2> amps,
                                                      const float omega, const int tau_half)
{
    __shared__ float ly[2][2][6][1024];  // [buffer][level][+y 0..2, -y 3..5][row * 64 + lane]
    const int b = remap_block(blockIdx.x, g.nblocks, g.xcd);
    const int tx = b % g.tiles_x, r = b / g.tiles_x;
    const int ty = r % g.tiles_y, zc = r / g.tiles_y;
    if (ps.flag != nullptr && ps.flag[b] != 0)
        pair_march<H, GH, MU, true>(Min, Din, Mout, Dout, cl2a, dlnmu, g, ps, amps, omega, tau_half != 0, tx, ty * g.sy,
                                    zc * g.lz, ly);
    else
        pair_march<H, GH, MU, false>(Min, Din, Mout, Dout, cl2a, dlnmu, g, ps, amps, omega, tau_half != 0, tx, ty * g.sy,
                                     zc * g.lz, ly);
}

// E and B of a 3D 16-bit state not yet streamed, on the tiles of the march
// above with one level: every stored cell is decoded once (the per-cell reader
// decodes each arrival from its neighbour's moments and codes), up to 62 x 14 cells
// of a tile are written, even tiles.  Same arithmetic as k_fields, so the same bits.
// Bound by memory, 58 B read and 48 B written per cell (FP16 ghost): 256^3 792
// -> 491 us per call (3.6 TB/s), 512^3 6.4 -> 3.4 ms.
constexpr int FLX = 62, FLY = 14;

template <typename H, bool GH>
__global__ __launch_bounds__(1024, 4) void k_fields_dev3(const float* Min, const H* Din, const float* cl2a,
                                                        const PairGeo g, double* E, double* B)
{
    constexpr int D = 3, Q = 7, P = 3, NM = 6, NC = DevSlots<D, GH>::N;
    __shared__ float ly[2][2 * P][1024];  // [buffer][+y 0..2, -y 3..5][row * 64 + lane]
    const int b = remap_block(blockIdx.x, g.nblocks, g.xcd);
    const int tx = b % g.tiles_x, r = b / g.tiles_x;
    const int ty = r % g.tiles_y, zc = r / g.tiles_y;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int tid = threadIdx.x;
    const int x0 = tx * g.sx, y0 = ty * g.sy, z0 = zc * g.lz;
    const int planes = min(g.lz, g.nz - z0);
    auto wrap = [](int v, int m) { v %= m; return v < 0 ? v + m : v; };
    const unsigned col0 = (unsigned)wrap(x0 - 1 + lane, g.nx);
    const int64_t nxy = (int64_t)g.nx * g.ny, rowo = (int64_t)wrap(y0 - 1 + w, g.ny) * g.nx;
    const bool live = w < g.sy + 2, col = lane < g.sx + 2;   // the tile and its halo
    const bool edge = w == 0 || w >= g.sy + 1;         // rows decoded for their +y / -y populations only
    const bool keep = !edge && lane >= 1 && lane < 1 + g.sx && x0 - 1 + lane < g.nx && y0 - 1 + w < g.ny;

    float m[NM] = {}, cl = 1.f;
    H cd[NC] = {};
    int gz = wrap(z0 - 1, g.nz);
    auto fetch = [&]() {
        const int64_t o = (int64_t)gz * nxy + rowo;
        if (col) {
            unsigned c = col0;
            asm volatile("" : "+v"(c));
#pragma unroll
            for (int t = 0; t < NM; ++t) m[t] = at32(Min + (int64_t)t * g.n + o, c);
#pragma unroll
            for (int s = 0; s < NC; ++s)
                if (pair_edge_code<GH>(s)) cd[s] = at32(Din + (int64_t)s * g.n + o, c);
            if (!edge) {
#pragma unroll
                for (int s = 0; s < NC; ++s)
                    if (!pair_edge_code<GH>(s)) cd[s] = at32(Din + (int64_t)s * g.n + o, c);
                cl = at32(cl2a + o, c);
            }
        }
        gz = gz + 1 == g.nz ? 0 : gz + 1;
    };
    float rest[P] = {}, px[P] = {}, mx[P] = {}, pz[P] = {}, pzo[P] = {}, clp = 1.f;   // of the plane before
    if (live) fetch();
    for (int it = 0; it < planes + 2; ++it) {
        const int bw = it & 1, br = bw ^ 1;
        const float wc0 = 1.f / cl - float(D), sc = row_scale(m), cl0 = cl;
        float cf[NC], nrest[P], npx[P], nmx[P], npz[P], mz[P];
#pragma unroll
        for (int s = 0; s < NC; ++s) cf[s] = h2f<H>(cd[s]);
        auto get = [&](int s) { return cf[s]; };
#pragma unroll
        for (int p = 0; p < P; ++p) {
            ly[bw][p][tid] = row_pop<GH>(m, get, sc, wc0, 2, p);
            ly[bw][P + p][tid] = row_pop<GH>(m, get, sc, wc0, 5, p);
            nrest[p] = row_pop<GH>(m, get, sc, wc0, 0, p);
            npx[p] = row_pop<GH>(m, get, sc, wc0, 1, p);
            nmx[p] = row_pop<GH>(m, get, sc, wc0, 4, p);
            npz[p] = row_pop<GH>(m, get, sc, wc0, 3, p);
            mz[p] = row_pop<GH>(m, get, sc, wc0, 6, p);
        }
        if (live && it + 1 < planes + 2) fetch();
        if (it >= 2 && !edge) {
            double f[Q][P];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                f[0][p] = (double)rest[p];
                f[1][p] = (double)lane_shift<1>(px[p]);
                f[2][p] = (double)ly[br][p][tid - 64];
                f[3][p] = (double)pzo[p];
                f[4][p] = (double)lane_shift<-1>(mx[p]);
                f[5][p] = (double)ly[br][P + p][tid + 64];
                f[6][p] = (double)mz[p];
            }
            double rho[P], K[D];
            moments<D, double>(f, rho, K);
            const int64_t o = (int64_t)(z0 + it - 2) * nxy + rowo;
            if (keep) {
                const double cld = (double)clp;
                if (E) {
#pragma unroll
                    for (int p = 0; p < P; ++p)
                        at32(E + (int64_t)pair_g(D, p) * g.n + o, col0) = -(double)pair_s(D, p) * (cld * rho[p]);
                }
                if (B) {
#pragma unroll
                    for (int k = 0; k < D; ++k) at32(B + (int64_t)k * g.n + o, col0) = K[k];
                }
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            rest[p] = nrest[p];
            px[p] = npx[p];
            mx[p] = nmx[p];
            pzo[p] = pz[p];
            pz[p] = npz[p];
        }
        clp = cl0;
        __syncthreads();
    }
}

}  // namespace lbem
