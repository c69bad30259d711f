// march2d.h -- 2D temporal blocking in registers: NS time steps per launch.
//
// One wave owns a strip of 64*CPL columns (CPL neighbouring cells per lane)
// and a chunk of rows, and marches along the rows.  Iteration i reads row i of
// the stored state once (level 0), and level s = 1..NS advances row i-s by its
// s-th step from what level s-1 left in registers: the rest and +-x
// populations of its previous row, the ones that move along the march of the
// row before that (a ring of two) and the ones that move against it of the
// row it has just made.  The +-x populations cross lanes by DPP wave shifts.
// There is no LDS, no barrier and no frame addressing: every lane runs every
// update, and the MARCH_HX columns at each end of the strip, whose neighbours
// belong to other waves, are computed but not stored.  Ring indices are fixed
// at compile time by unrolling four rows.  Neighbouring chunks march towards
// and away from each other in turn, so that the rows both read are read at
// about the same time and meet in one L2.  Each update is the single-step
// kernel's arithmetic (moments, collide), so NS fused steps equal NS single
// steps bit for bit.  In the 16-bit formats level 0 decodes each stored cell
// once, where the per-cell kernel decodes every neighbour, and a level between
// the first and the last step encodes its result as it would be stored and
// decodes that in registers, as every reader would.
//
// Walls, an absorbing layer and a dispersion pole (plain formats) are applied at
// every level: what a wall reflects is in the cell's own registers, sigma, the
// pole's coefficients, P and J ride in the ring of rows, and P and J go to a
// second buffer with the last level.
//
// What bounds it: 21.5 VALU instructions per update (one cell, one step)
// against 74 of the LDS-frame kernel it replaces, so the state's bytes do.
// Measured per launch of four steps, LDS frame (64x16 tiles, 512 threads) ->
// this kernel: FP32 2048^2 43.1 -> 31.8 us (44 B per cell and launch at 5.8
// TB/s, Infinity Cache), 8192^2 740 -> 645 us (4.6 TB/s, the rate of a large
// copy here), 96x64 5.5 -> 3.6 us (launch latency).  16-bit formats, per step,
// one step per launch of the per-cell kernel -> four of this one: 3000x2500
// FP16-dev 113 -> 32 us (12 B per update at 2.8 TB/s: VALU bound, about 90
// instructions per update for encoding and decoding), FP16 ghost 20 us.  They
// take one cell per lane (two need more than 256 registers: 32 against 37 us).
// With extras, single steps -> this kernel: 40 steps of FP32 1023x767 with walls
// and an absorber 368 -> 196 us (116 VGPRs, 4 waves per SIMD; a pole 153).
#pragma once
#include "kernels.h"

namespace lbem {

// the value of the lane before (dir > 0) or after (dir < 0); the end lane gets 0
template <int DIR>
__device__ __forceinline__ int lane_shift_b32(int v)
{
    // DPP wave_shr:1 / wave_shl:1
    return __builtin_amdgcn_update_dpp(0, v, DIR > 0 ? 0x138 : 0x130, 0xf, 0xf, true);
}
template <int DIR, typename T>
__device__ __forceinline__ T lane_shift(T v)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, lane_shift_b32<DIR>(__builtin_bit_cast(int, v)));
    } else {
        struct Two { int a, b; };
        Two t = __builtin_bit_cast(Two, v);
        t.a = lane_shift_b32<DIR>(t.a);
        t.b = lane_shift_b32<DIR>(t.b);
        return __builtin_bit_cast(T, t);
    }
}

// Sparse current source: idx[strip*ny + row] is the segment of that strip's
// row (64*CPL values, S per unit amplitude, periodic images included) or -1.
// Bit strip % 256 of mask is set for every strip that holds a source: the
// others start without waiting for an index.
template <typename T>
struct MarchSrc {
    const int* idx;
    const T* val;
    unsigned mask[8];    // all zero: no source
};

// CPL neighbouring elements at a byte offset off a scalar base.  A pair (FP32)
// moves as one 8-byte access, aligned to 4 bytes.  The offset within a row has 32
// bits where every row fits them (offsets32), as all FP32 rows do.
typedef float MarchPair __attribute__((ext_vector_type(2)));
typedef MarchPair MarchPairU __attribute__((aligned(4)));
template <typename S, int CPL, typename Off>
__device__ __forceinline__ void march_load(const S* base, Off off, S (&v)[CPL])
{
    const char* p = reinterpret_cast<const char*>(base) + off;
    if constexpr (CPL == 1) {
        v[0] = *reinterpret_cast<const S*>(p);
    } else {
        static_assert(CPL == 1 || std::is_same<S, float>::value, "pairs are FP32");
        const MarchPair w = *reinterpret_cast<const MarchPairU*>(p);
        v[0] = w[0];
        v[1] = w[1];
    }
}
template <typename S, int CPL, typename Off>
__device__ __forceinline__ void march_store(S* base, Off off, const S (&v)[CPL])
{
    char* p = reinterpret_cast<char*>(base) + off;
    if constexpr (CPL == 1) {
        *reinterpret_cast<S*>(p) = v[0];
    } else {
        static_assert(CPL == 1 || std::is_same<S, float>::value, "pairs are FP32");
        const MarchPair w = {v[0], v[1]};
        *reinterpret_cast<MarchPairU*>(p) = w;
    }
}

// storage of the plain formats: five populations of type T per cell.  WIDE:
// 64-bit offsets within a row.
template <typename T_, int CPL, bool WIDE = false>
struct MarchPlain {
    typedef T_ T;
    typedef typename std::conditional<WIDE, size_t, unsigned>::type Off;
    const T* src;
    T* dst;
    int64_t n;
    struct Raw { T v[5][CPL]; };
    static constexpr bool DEV = false, REST = false;
    __device__ __forceinline__ void load(Raw& r, int64_t row, unsigned col) const
    {
#pragma unroll
        for (int k = 0; k < 5; ++k) march_load<T, CPL>(src + (int64_t)k * n + row, (Off)col * (Off)sizeof(T), r.v[k]);
    }
    __device__ __forceinline__ void decode(const Raw& r, const T (&)[CPL], T (&o)[5][CPL]) const
    {
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
            for (int c = 0; c < CPL; ++c) o[k][c] = r.v[k][c];
    }
    __device__ __forceinline__ void store(const Raw& r, int64_t row, unsigned col) const
    {
#pragma unroll
        for (int k = 0; k < 5; ++k)
            march_store<T, CPL>(dst + (int64_t)k * n + row, (Off)col * (Off)sizeof(T), r.v[k]);
    }
};

// storage of the 16-bit formats: three FP32 moments and the codes
template <typename H, bool GH, int CPL>
struct MarchDev {
    typedef float T;
    typedef unsigned Off;
    typedef H Code;
    static constexpr bool GHOST = GH;
    static constexpr int NC = DevSlots<2, GH>::N;
    const float* Min;
    const H* Din;
    float* Mout;
    H* Dout;
    int64_t n;
    struct Raw { float m[3][CPL]; H c[NC][CPL]; };
    static constexpr bool DEV = true, REST = !GH;
    __device__ __forceinline__ void load(Raw& r, int64_t row, unsigned col) const
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) march_load<float, CPL>(Min + (int64_t)k * n + row, col * 4u, r.m[k]);
#pragma unroll
        for (int k = 0; k < NC; ++k) march_load<H, CPL>(Din + (int64_t)k * n + row, col * 2u, r.c[k]);
    }
    // the five populations of a cell from its stored moments and codes, as dev_load forms them
    static __device__ __forceinline__ void pops(const float (&m)[3], const H (&code)[NC], float wc0, float (&o)[5])
    {
        float mag = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) mag = fmaxf(mag, fabsf(m[k]));
        float s, inv;
        pow2_scale(mag, s, inv);
        const float Lam[1] = {m[0]}, Bb[2] = {m[1], m[2]};
        auto get = [&](int sl) { return h2f<H>(code[sl]); };
#pragma unroll
        for (int i = 0; i < 5; ++i) o[i] = dev_pop<2, GH>(get, i, 0, Lam, Bb, s, wc0);
    }
    __device__ __forceinline__ void decode(const Raw& r, const float (&wc0)[CPL], float (&o)[5][CPL]) const
    {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            float m[3], v[5];
            H cd[NC];
#pragma unroll
            for (int k = 0; k < 3; ++k) m[k] = r.m[k][c];
#pragma unroll
            for (int k = 0; k < NC; ++k) cd[k] = r.c[k][c];
            pops(m, cd, wc0[c], v);
#pragma unroll
            for (int k = 0; k < 5; ++k) o[k][c] = v[k];
        }
    }
    __device__ __forceinline__ void store(const Raw& r, int64_t row, unsigned col) const
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) march_store<float, CPL>(Mout + (int64_t)k * n + row, col * 4u, r.m[k]);
#pragma unroll
        for (int k = 0; k < NC; ++k) march_store<H, CPL>(Dout + (int64_t)k * n + row, col * 2u, r.c[k]);
    }
};

// Cell-local extras (plain formats).  Walls: a population that would enter from
// beyond one is the cell's own outgoing one of the level before, negated or not;
// rows and columns past a wall run on wrapped data that nothing stored depends on.
template <typename T>
struct MarchExt {
    bool wx, wy, nx_, ny_;   // walls on the axis, and whether they negate
    const T* keep;       // per-cell 1 - sigma, or nullptr
    const T* ade;        // [3][n] c1, c2, c3, or nullptr
    const T* pin;        // [2][n] P then J
    T* pout;
};

// One work item: strip x chunk.  SRC: the chunk holds source cells.  EXT: 0 no
// extras, 1 walls and an absorber, 2 a dispersion pole as well.
template <class IO, int NS, int CPL, bool MU, bool TH, bool SRC, bool UP, int EXT>
__device__ __forceinline__ void march2d_item(const IO& io, const typename IO::T* __restrict__ cl2a,
                                             const typename IO::T* __restrict__ dlnmu, const MarchGeo& g,
                                             const MarchSrc<typename IO::T>& ms,
                                             const AmpPack<typename IO::T, NS>& amps,
                                             const typename IO::T omega, const bool tau_half,
                                             const MarchExt<typename IO::T>& ex, const int strip, const int y0,
                                             const int segs)
{
    typedef typename IO::T T;
    typedef typename IO::Off Off;
    constexpr int RING = 4, PF = 2;
    static_assert(NS <= RING && NS <= MARCH_HX && RING % PF == 0, "ring indices repeat every RING rows");
    constexpr int HX = MARCH_HX, OW = 64 * CPL - 2 * HX;
    const int nx = g.nx, ny = g.ny;
    const int lane = threadIdx.x & 63;
    const int x0 = strip * OW;
    // column of the lane's first cell, wrapped (any box width)
    int gx = (x0 - HX + lane * CPL) % nx;
    if (gx < 0) gx += nx;
    const unsigned col0 = (unsigned)gx;
    const int xo = x0 - HX + lane * CPL;         // unwrapped: stored if inside the strip's own columns
    const bool keep = lane * CPL >= HX && lane * CPL < HX + OW && xo < nx;
    const int rows = min(g.rows, ny - y0);
    const int total = rows + 2 * NS;
    int pr = (UP ? y0 + rows - 1 + NS : y0 - NS) % ny;   // next row to load, wrapped
    if (pr < 0) pr += ny;

    struct Row {
        typename IO::Raw raw;
        T cl[CPL];
        T dl[MU ? 2 : 1][CPL];
        T sv[CPL];
        T kp[EXT ? CPL : 1];
        T co[EXT == 2 ? 5 : 1][CPL];             // c1, c2, c3, P, J
    };
    Row pf[PF];
    const bool damp = EXT && ex.keep != nullptr, pole = EXT == 2 && ex.ade != nullptr;
    T kp[EXT ? RING : 1][CPL], co[EXT == 2 ? RING : 1][5][CPL], a4[EXT ? NS : 1][CPL];
    constexpr bool WC = IO::DEV;                 // w0/c^2 is kept per row
    constexpr bool RW = IO::REST;                // and its reciprocal (stored rest codes)
    T cl[RING][CPL], wc[WC ? RING : 1][CPL], rw[RW ? RING : 1][CPL], dl[MU ? RING : 1][2][CPL], sv[SRC ? RING : 1][CPL];
    T a0[NS][CPL], a1[NS][CPL], a3[NS][CPL], a2[NS][2][CPL];

    int nf = 0;                                  // rows fetched
    auto fetch = [&](Row& r) {
        const int64_t ro = (int64_t)pr * nx;
        unsigned col = col0;
        asm volatile("" : "+v"(col));            // keeps the 32-bit offset next to its loads (scalar-base form)
        io.load(r.raw, ro, col);
        march_load<T, CPL>(cl2a + ro, (Off)col * (Off)sizeof(T), r.cl);
        if constexpr (MU) {
            march_load<T, CPL>(dlnmu + ro, (Off)col * (Off)sizeof(T), r.dl[0]);
            march_load<T, CPL>(dlnmu + g.n + ro, (Off)col * (Off)sizeof(T), r.dl[MU ? 1 : 0]);
        }
        if constexpr (SRC) {
            const int seg = __builtin_amdgcn_readlane(segs, nf);   // lane k holds the segment of input row k
            nf = nf + 1;
#pragma unroll
            for (int c = 0; c < CPL; ++c) r.sv[c] = T(0);
            if (seg >= 0) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) r.sv[c] = ms.val[(int64_t)seg * (64 * CPL) + lane * CPL + c];
            }
        }
        if constexpr (EXT) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) r.kp[c] = T(1);
            if (damp) march_load<T, CPL>(ex.keep + ro, (Off)col * (Off)sizeof(T), r.kp);
        }
        if constexpr (EXT == 2) {
            if (pole) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    march_load<T, CPL>(ex.ade + (int64_t)k * g.n + ro, (Off)col * (Off)sizeof(T), r.co[EXT == 2 ? k : 0]);
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    march_load<T, CPL>(ex.pin + (int64_t)k * g.n + ro, (Off)col * (Off)sizeof(T), r.co[EXT == 2 ? 3 + k : 0]);
            }
        }
        if constexpr (UP) pr = pr == 0 ? ny - 1 : pr - 1;
        else pr = pr + 1 == ny ? 0 : pr + 1;
    };

    // iteration i (i % RING == U): level 0 and levels 1..LV
    auto iter = [&](auto Uc, auto LVc, const int i) {
        constexpr int U = decltype(Uc)::value, LV = decltype(LVc)::value;
        Row& row = pf[U % PF];
        T wnew[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) wnew[c] = WC ? T(1) / row.cl[c] - T(2) : T(0);
        T o[5][CPL];
        io.decode(row.raw, wnew, o);
        T clnew[CPL], dlnew[2][CPL], svnew[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            clnew[c] = row.cl[c];
            if constexpr (MU) {
                dlnew[0][c] = row.dl[0][c];
                dlnew[1][c] = row.dl[MU ? 1 : 0][c];
            }
            if constexpr (SRC) svnew[c] = row.sv[c];
        }
        T kpnew[CPL], conew[5][CPL];
        if constexpr (EXT) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                kpnew[c] = row.kp[c];
                if constexpr (EXT == 2) {
#pragma unroll
                    for (int k = 0; k < 5; ++k) conew[k][c] = row.co[EXT == 2 ? k : 0][c];
                }
            }
        }
        if (i + PF < total) fetch(row);
#pragma unroll
        for (int s = 1; s <= NS; ++s) {
            if (s > LV + 1) continue;
            T f[CPL][5][1];
            if (s <= LV) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    f[c][0][0] = a0[s - 1][c];
                    f[c][1][0] = c > 0 ? a1[s - 1][c > 0 ? c - 1 : 0] : lane_shift<1>(a1[s - 1][CPL - 1]);
                    f[c][3][0] = c < CPL - 1 ? a3[s - 1][c < CPL - 1 ? c + 1 : 0] : lane_shift<-1>(a3[s - 1][0]);
                    f[c][UP ? 4 : 2][0] = a2[s - 1][U & 1][c];
                    f[c][UP ? 2 : 4][0] = o[UP ? 2 : 4][c];
                }
                if constexpr (EXT != 0) {
                    if (ex.wx) {
#pragma unroll
                        for (int c = 0; c < CPL; ++c) {
                            if (xo + c == 0) f[c][1][0] = ex.nx_ ? -a3[s - 1][c] : a3[s - 1][c];
                            if (xo + c == nx - 1) f[c][3][0] = ex.nx_ ? -a1[s - 1][c] : a1[s - 1][c];
                        }
                    }
                    if (ex.wy) {
                        const int y = UP ? y0 + rows - 1 + NS - (i - s) : y0 - NS + (i - s);
                        if (y == (UP ? ny - 1 : 0)) {
#pragma unroll
                            for (int c = 0; c < CPL; ++c)
                                f[c][UP ? 4 : 2][0] = ex.ny_ ? -a4[s - 1][c] : a4[s - 1][c];
                        }
                        if (y == (UP ? 0 : ny - 1)) {
#pragma unroll
                            for (int c = 0; c < CPL; ++c)
                                f[c][UP ? 2 : 4][0] = ex.ny_ ? -a2[s - 1][(U & 1) ^ 1][c] : a2[s - 1][(U & 1) ^ 1][c];
                        }
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                a0[s - 1][c] = o[0][c];
                a1[s - 1][c] = o[1][c];
                a3[s - 1][c] = o[3][c];
                a2[s - 1][U & 1][c] = o[UP ? 4 : 2][c];
                if constexpr (EXT != 0) a4[EXT ? s - 1 : 0][c] = o[UP ? 2 : 4][c];
            }
            if (s <= LV) {
                constexpr int R4 = RING;
                const int q = (U + R4 - s % R4) % R4;     // ring slot of row i - s
                const int64_t orow = (int64_t)(UP ? y0 + rows - 1 - (i - 2 * NS) : y0 + i - 2 * NS) * nx;
                typename IO::Raw st;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    T rho[1], K[2], Sp[1];
                    moments<2, T>(f[c], rho, K);
                    Sp[0] = SRC ? source_term(sv[SRC ? q : 0][c], amps.a[s - 1]) : T(0);
                    if constexpr (MU) {
                        const T d2[2] = {dl[MU ? q : 0][0][c], dl[MU ? q : 0][1][c]};
                        add_mu_source<2, T>(K, cl[q][c], d2, Sp);
                    }
                    if constexpr (IO::DEV) {
                        float M[3];
                        typename IO::Code cd[IO::NC];
                        dev_encode<2, typename IO::Code, IO::GHOST, RW>(f[c], cl[q][c], RW ? rw[RW ? q : 0][c] : wc[q][c],
                                                                        Sp, SRC || MU, omega, TH || tau_half, rho, K,
                                                                        M, cd);
                        if (s == NS) {
#pragma unroll
                            for (int k = 0; k < 3; ++k) st.m[k][c] = M[k];
#pragma unroll
                            for (int k = 0; k < IO::NC; ++k) st.c[k][c] = cd[k];
                        } else {
                            float v[5];
                            IO::pops(M, cd, wc[q][c], v);
#pragma unroll
                            for (int k = 0; k < 5; ++k) o[k][c] = v[k];
                        }
                    } else {
                        T out[5][1];
                        if constexpr (EXT == 2) {
                            T (&e)[5][CPL] = co[EXT == 2 ? q : 0];
                            if (pole) ade_advance<T>(e[0][c], e[1][c], e[2][c], cl[q][c], rho[0], e[3][c], e[4][c]);
                        }
                        collide<2, T>(f[c], cl[q][c], Sp, SRC || MU, omega, TH || tau_half, rho, K, out);
                        if constexpr (EXT == 2) {
                            if (pole) out[0][0] += co[EXT == 2 ? q : 0][4][c] / cl[q][c];
                        }
                        if constexpr (EXT != 0) {
                            if (damp) {
#pragma unroll
                                for (int k = 0; k < 5; ++k) out[k][0] *= kp[EXT ? q : 0][c];
                            }
                        }
#pragma unroll
                        for (int k = 0; k < 5; ++k) {
                            if (s == NS) st.v[k][c] = out[k][0];
                            else o[k][c] = out[k][0];
                        }
                    }
                }
                if (s == NS && keep) {
                    unsigned xc = (unsigned)xo;
                    asm volatile("" : "+v"(xc));
                    io.store(st, orow, xc);
                    if constexpr (EXT == 2) {
                        if (pole) {
#pragma unroll
                            for (int k = 0; k < 2; ++k)
                                march_store<T, CPL>(ex.pout + (int64_t)k * g.n + orow, (Off)xc * (Off)sizeof(T),
                                                    co[EXT == 2 ? q : 0][3 + k]);
                        }
                    }
                }
            }
        }
        // row i's coefficients replace row i - RING's
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            cl[U][c] = clnew[c];
            if constexpr (WC) wc[WC ? U : 0][c] = wnew[c];
            if constexpr (RW) rw[RW ? U : 0][c] = T(1) / wnew[c];
            if constexpr (MU) {
                dl[MU ? U : 0][0][c] = dlnew[0][c];
                dl[MU ? U : 0][1][c] = dlnew[1][c];
            }
            if constexpr (SRC) sv[SRC ? U : 0][c] = svnew[c];
            if constexpr (EXT != 0) kp[EXT ? U : 0][c] = kpnew[c];
            if constexpr (EXT == 2) {
#pragma unroll
                for (int k = 0; k < 5; ++k) co[EXT == 2 ? U : 0][k][c] = conew[k][c];
            }
        }
    };
#define LBEM_IC(v) std::integral_constant<int, (v)>{}
#pragma unroll
    for (int k = 0; k < PF; ++k) fetch(pf[k]);
    // the first 2 NS rows fill the levels one after another
    iter(LBEM_IC(0), LBEM_IC(0), 0);
    iter(LBEM_IC(1), LBEM_IC(0), 1);
    iter(LBEM_IC(2), LBEM_IC(1), 2);
    iter(LBEM_IC(3), LBEM_IC(1), 3);
    if constexpr (NS >= 3) {
        iter(LBEM_IC(0), LBEM_IC(2), 4);
        iter(LBEM_IC(1), LBEM_IC(2), 5);
    }
    if constexpr (NS >= 4) {
        iter(LBEM_IC(2), LBEM_IC(3), 6);
        iter(LBEM_IC(3), LBEM_IC(3), 7);
    }
    int i = 2 * NS;
    while (true) {
        iter(LBEM_IC((2 * NS) % RING), LBEM_IC(NS), i);
        if (++i >= total) break;
        iter(LBEM_IC((2 * NS + 1) % RING), LBEM_IC(NS), i);
        if (++i >= total) break;
        iter(LBEM_IC((2 * NS + 2) % RING), LBEM_IC(NS), i);
        if (++i >= total) break;
        iter(LBEM_IC((2 * NS + 3) % RING), LBEM_IC(NS), i);
        if (++i >= total) break;
    }
#undef LBEM_IC
}

// Work item w (uniform over the wave).
template <class IO, int NS, int CPL, bool MU, bool TH, int EXT = 0>
__device__ __forceinline__ void march2d_work(const IO& io, const typename IO::T* __restrict__ cl2a,
                                             const typename IO::T* __restrict__ dlnmu, const MarchGeo& g,
                                             const MarchSrc<typename IO::T>& ms,
                                             const AmpPack<typename IO::T, NS>& amps,
                                             const typename IO::T omega, const bool tau_half, const int w,
                                             const MarchExt<typename IO::T>& ex = MarchExt<typename IO::T>{})
{
    const int strip = w % g.strips, y0 = (w / g.strips) * g.rows;
    unsigned m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) m = ((strip >> 5) & 7) == k ? ms.mask[k] : m;
    bool src = false;
    int segs = -1;
    if ((m >> (strip & 31)) & 1u) {
        // the segments of the rows this item reads (at most 64), one per lane
        const int k = threadIdx.x & 63;
        if (k < min(g.rows, g.ny - y0) + 2 * NS) {
            int r = (y0 - NS + k) % g.ny;
            if (r < 0) r += g.ny;
            segs = ms.idx[strip * g.ny + r];
        }
        src = __any(segs >= 0);
    }
    const bool up = (w / g.strips) & 1;
    if (src)
        march2d_item<IO, NS, CPL, MU, TH, true, false, EXT>(io, cl2a, dlnmu, g, ms, amps, omega, tau_half, ex, strip, y0, segs);
    else if (up)
        march2d_item<IO, NS, CPL, MU, TH, false, true, EXT>(io, cl2a, dlnmu, g, ms, amps, omega, tau_half, ex, strip, y0, segs);
    else
        march2d_item<IO, NS, CPL, MU, TH, false, false, EXT>(io, cl2a, dlnmu, g, ms, amps, omega, tau_half, ex, strip, y0, segs);
}

template <class IO, int NS, int CPL, bool MU, bool TH, int EXT = 0>
__global__ __launch_bounds__(NT) void k_march2d(const IO io, const typename IO::T* __restrict__ cl2a,
                                               const typename IO::T* __restrict__ dlnmu, const MarchGeo g,
                                               const MarchSrc<typename IO::T> ms,
                                               const AmpPack<typename IO::T, NS> amps,
                                               const typename IO::T omega, const int tau_half,
                                               const MarchExt<typename IO::T> ex)
{
    const int b = remap_block(blockIdx.x, g.nblocks, 1);
    const int w = __builtin_amdgcn_readfirstlane(b * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6));
    if (w >= g.nwork) return;
    march2d_work<IO, NS, CPL, MU, TH, EXT>(io, cl2a, dlnmu, g, ms, amps, omega, tau_half != 0, w, ex);
}

}  // namespace lbem
