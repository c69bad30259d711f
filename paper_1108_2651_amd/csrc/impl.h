// impl.h -- the handle and the kernel dispatch of one (dimension, format) pair,
// shared by lbem.hip (the C ABI) and impl.hip (the dispatch instantiations).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <shared_mutex>
#include <vector>

#include "../../include/lbem.h"
#include "kernels.h"
#include "limits.h"
#include "march2d.h"
#include "pair3d.h"
#include "pair3f.h"

using namespace lbem;

namespace {

enum Layout { LAYOUT_NATURAL = 0, LAYOUT_PULL_PENDING = 1, LAYOUT_AA_SWAPPED = 2 };

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

int env_int(const char* name, int dflt)
{
    const char* v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : dflt;
}

struct Sizes {
    size_t pop_one;   // bytes of one copy of the population state
    size_t copies;
    size_t medium;    // c_L^2
    size_t mu;        // mu_r (double) + grad ln mu (medium type) if mu_varies
    size_t scratch;   // 3*n doubles
    size_t total;
};

// the formats with FP32 moments + 16-bit deviations or ghost coordinates
bool is_dev(int prec) { return prec >= LBEM_F16DEV && prec <= LBEM_BF16GHOST; }

bool valid_cfg(const lbem_config* c)
{
    if (!c) return false;
    if (c->dim != 2 && c->dim != 3) return false;
    if (c->prec < LBEM_F64 || c->prec > LBEM_F16) return false;
    if (c->nx < 1 || c->ny < 1 || c->nz < 1) return false;
    if (c->dim == 2 && c->nz != 1) return false;
    if (c->nx > (1 << 30) || c->ny > (1 << 30) || c->nz > (1 << 30)) return false;
    const double n = (double)c->nx * (double)c->ny * (double)c->nz;
    if (n >= 2147483648.0) return false;
    if (!(c->tau > 0.0) || !std::isfinite(c->tau)) return false;
    if (!(c->w0_vac >= 0.0 && c->w0_vac < 1.0)) return false;
    if (c->streaming < LBEM_STREAM_AUTO || c->streaming > LBEM_STREAM_AA) return false;
    if (c->streaming == LBEM_STREAM_AA && is_dev(c->prec)) return false;
    return true;
}

// 3D FP32 runs two fused steps per launch from this many cells on (about
// 100^3), single AA steps below, where the state is Infinity-Cache resident
// and the pair's tiles cannot fill the chip.  Measured, us per step, fused
// pair (64 x 8 tiles) against single AA steps: 64^3 20.6 / 7.2, 80^3 23.6 /
// 15.1, 96^3 23.8 / 24.3, 112^3 29.7 / 37.5, 128^3 47.4 / 58.5, 144^3 76.1 /
// 82.5, 160^3 96.0 / 133.1.
constexpr double FUSE3D_MIN = 1.0e6;
// The column-tile z-march of the 16-bit formats (rows longer than the row
// tiles take) from this many cells on: the cache-residency threshold every 3D
// z-marching kernel shared before the row tiles and the 64 x 8 FP32 pair got
// their own, kept for these rare shapes (not re-measured).
constexpr double SMALL3D = 3.5e6;
// The 3D 16-bit formats take the whole-row tiles once the state one step
// touches (stored values read and written, c_L^2 read: 112 B per cell with
// ghost coordinates, 136 B with all deviations) exceeds the 256 MB Infinity
// Cache; per-cell tiles below.  Measured, us per step, per-cell against row
// tiles: FP16 ghost 128^3 (224 MiB) 48.4 / 67.1, 144^3 122.1 / 88.2; FP16-dev
// 128^3 (272 MiB) 76.3 / 74.5, 144^3 130.7 / 109.3.
constexpr double ROWTILE_BYTES = 256.0 * (1 << 20);
// plain FP16 storage on whole-row blocks: measured from 6e6 cells on
constexpr double XROW3D = 6.0e6;

int resolve_streaming(const lbem_config* c)
{
    // Pull by default: the fused multi-step kernels need the second copy.
    // 3D FP64 never fuses and small 3D FP32 boxes run single steps: there the
    // in-place AA pattern (half the memory) is as fast or faster.
    if (c->streaming != LBEM_STREAM_AUTO) return c->streaming;
    const double n = (double)c->nx * (double)c->ny * (double)c->nz;
    if (c->dim == 3 && (c->prec == LBEM_F64 || (c->prec == LBEM_F32 && n < FUSE3D_MIN))) return LBEM_STREAM_AA;
    return LBEM_STREAM_PULL;
}

Sizes sizes_of(const lbem_config* c)
{
    Sizes s{};
    const int D = c->dim, Q = 2 * D + 1, P = D * (D - 1) / 2;
    const size_t n = (size_t)(c->nx * c->ny * c->nz);
    const size_t tm = c->prec == LBEM_F64 ? 8 : 4;
    if (!is_dev(c->prec))
        s.pop_one = align256((size_t)Q * P * n * (c->prec == LBEM_F16 ? 2 : tm));
    else
        s.pop_one = align256((size_t)(P + D) * n * 4) +
                    align256((size_t)(c->prec >= LBEM_F16GHOST ? 2 * D * P - D : Q * P) * n * 2);
    s.copies = resolve_streaming(c) == LBEM_STREAM_AA ? 1 : 2;
    s.medium = align256(n * tm);
    s.mu = c->mu_varies ? align256(n * 8) + align256((size_t)D * n * tm) : 0;
    s.scratch = align256(3 * n * 8);
    s.total = s.pop_one * s.copies + s.medium + s.mu + s.scratch;
    return s;
}

}  // namespace

struct Impl;

struct lbem_s {
    lbem_config cfg;
    int D, Q, P, prec, streaming;
    int64_t n;
    hipStream_t stream;
    int device;
    bool own_mem;
    char* arena;
    size_t arena_bytes;
    // population state
    char* pop[2];
    int cur;
    int layout;
    // medium
    void* cl2;
    double* mu_r;
    void* dlnmu;
    bool mu_set;
    // scratch / reductions
    double* scratch;
    double* partials;   // nb_diag*4 + 4
    int nb_diag;
    // source (device tables, handle-owned)
    int* src_off;
    int2* src_ent;
    void* src_val;
    int64_t nsrc;
    // tiling of the step kernels
    Geo geo;
    int vec;
    // temporal blocking (fuse_ns steps per launch; 1 = off): 2D wave strips of
    // mcpl cells per lane, mwpb waves per block; 3D column tiles f3_tx x f3_ty
    // marching over chunks of f3_lz planes
    int fuse_ns;
    MarchGeo mgeo;
    int mcpl, mwpb;
    MarchGeo mgeo_x[2];      // the same with walls or an absorber, and with a pole (more registers)
    int mwpb_x[2];
    int* msrc_idx;
    void* msrc_val;
    unsigned msrc_mask[8];
    int64_t nmsrc;       // source segments of the strips
    int f3_tx, f3_ty, f3_lz;
    bool pair_f32;           // 3D FP32 without extras: pairs on pgeo
    int ext_ns;              // steps per launch with extras (plain formats; 1 = off)
    Geo fgeo;
    // 3D 16-bit formats: two steps per launch (k_pair_dev3) and its source
    // segments
    PairGeo pgeo;
    PairGeo ftgeo;       // tiles of the field reader (k_fields_dev3), no blocks: the per-cell reader
    unsigned char* psrc_flag;
    int* psrc_idx;
    float* psrc_val;
    int psrc_pair;
    int* fsrc_off;
    int2* fsrc_ent;
    void* fsrc_val;
    int64_t nfsrc;
    // single steps with the streaming cache policy on the stored state
    // (lattices whose state a launch touches exceeds the last-level cache)
    int nts;
    // 3D deviation kernel marching along z (column tiles x z-chunks)
    int zmarch, zlz;
    Geo zgeo;
    int* zsrc_off;
    int2* zsrc_ent;
    void* zsrc_val;
    int64_t nzsrc;
    // 3D plain single steps on whole-row blocks (k_step_xrow)
    int xrow;
    XRowGeo xgeo;
    int* xsrc_off;
    int2* xsrc_ent;
    void* xsrc_val;
    int64_t nxsrc;
    // 3D deviation kernel on whole-row tiles (k_step_dev3r), marching along z
    int rowk;
    RowGeo rgeo;
    int rntb;            // threads per block of the row tiles
    int* rsrc_off;
    int2* rsrc_ent;
    float* rsrc_val;
    int64_t nrsrc;
    // the whole-row tiling of this handle inside a batch (3D deviation formats,
    // rows of up to 2 BROW_NT cells, BROW_NT-thread blocks) and its source table
    int brow;
    RowGeo bgeo;
    int* bsrc_off;
    int2* bsrc_ent;
    float* bsrc_val;
    int64_t nbsrc;
    // state
    // non-periodic faces and absorbing layer
    int bc_kind[3];
    void* keep;              // handle-owned, medium precision, or nullptr
    // frequency-dispersive permittivity (one Lorentz pole per cell)
    void* ade;               // [3][n] coefficients, handle-owned, or nullptr
    void* pol;               // [2P][n] auxiliary P and J per pair
    void* pol2;              // the buffer a two-step launch writes them to (they swap), or nullptr
    // anisotropy (plain formats): [D][n] ratios r_a, handle-owned; valid while ra_set
    void* ra;
    bool ra_set;
    int64_t t;
    bool have_medium, have_fields;
    bool graphed;            // lbem_step has been captured: a graph may hold the copies the state moves between
    Impl* impl;
    hipEvent_t sync_ev;      // set-up work on this handle's stream before a batch tick
    hipEvent_t tick_ev;      // end of the last batch tick that advanced this handle
    bool tick_pending;       // this handle's stream has not yet waited on tick_ev
};

// Work on the handle's own stream that touches its state follows the batch
// ticks that advanced it.  The wait is added here, at the handle's next use,
// not when the tick is enqueued: the stream may be shared with other
// handles' set-up, which need not wait for the tick.
static hipError_t follow_ticks(lbem_s* h)
{
    if (!h->tick_pending) return hipSuccess;
    h->tick_pending = false;
    return hipStreamWaitEvent(h->stream, h->tick_ev, 0);
}

// Set-up staging buffers: stream-ordered allocations, whose release does not
// wait for other streams' work (batch ticks in flight).  Buffers above 1 GiB
// (lattices of 4e7 cells and more, never served in batches) and any request
// the pool refuses use hipMalloc, whose hipFree synchronises the device: the
// pool keeps freed memory until the next synchronisation, which must not hold
// tens of GB beside a 2^30-cell lattice.
struct Staging {
    void* p = nullptr;
    bool pooled = false;
};
static bool stage_alloc(Staging& st, size_t bytes, hipStream_t s)
{
    if (bytes <= (size_t(1) << 30) && hipMallocAsync(&st.p, bytes, s) == hipSuccess) {
        st.pooled = true;
        return true;
    }
    (void)hipGetLastError();
    st.p = nullptr;
    st.pooled = false;
    return hipMalloc(&st.p, bytes) == hipSuccess;
}
static void stage_free(Staging& st, hipStream_t s)
{
    if (!st.p) return;
    if (st.pooled) (void)hipFreeAsync(st.p, s);
    else (void)hipFree(st.p);
    st.p = nullptr;
}

#define HIP_OK(x)                                  \
    do {                                           \
        hipError_t e_ = (x);                       \
        if (e_ != hipSuccess) return LBEM_EDEVICE; \
    } while (0)

// ---------------------------------------------------------------------------
// per (dimension, format) kernel dispatch
// ---------------------------------------------------------------------------
struct Impl {
    virtual ~Impl() {}
    virtual hipError_t step(lbem_s* h, double amp) = 0;
    // advance ns steps in one launch (2D: 2..fuse_ns, 3D: fuse_ns; only when
    // fused_ok and pull-pending)
    virtual hipError_t step_fused(lbem_s* h, const double* amp, int ns) { return hipErrorInvalidValue; }
    virtual hipError_t fields(lbem_s* h, double* E, double* B, double* partials) = 0;
    virtual hipError_t init(lbem_s* h, const double* dE, const double* dB) = 0;
    virtual hipError_t medium(lbem_s* h, const double* deps, const double* dmu, int* dflag) = 0;
};

static Geo1 geo1(const lbem_s* h)
{
    Geo1 g;
    g.nx = (int)h->cfg.nx; g.ny = (int)h->cfg.ny; g.nz = (int)h->cfg.nz; g.n = h->n;
    return g;
}

static int blocks1(int64_t n) { return (int)((n + NT - 1) / NT); }

static CellExt ext_of(const lbem_s* h)
{
    CellExt b;
    for (int a = 0; a < 3; ++a) b.kind[a] = h->bc_kind[a];
    b.keep = h->keep;
    b.ade = h->ade;
    b.pol = h->pol;
    b.ra = h->ra_set ? h->ra : nullptr;
    return b;
}
// walls, an absorber or dispersion: the single-step kernels with cell extras
static bool has_bx(const lbem_s* h)
{
    return h->keep != nullptr || h->ade != nullptr || h->ra_set || ext_of(h).walls();
}
static size_t medium_size(const lbem_s* h) { return h->prec == LBEM_F64 ? 8 : 4; }
static size_t pol_bytes(const lbem_s* h) { return h->ade ? (size_t)2 * h->P * h->n * medium_size(h) : 0; }

template <int D, typename TM>
static hipError_t launch_medium(lbem_s* h, const double* deps, const double* dmu, int* dflag)
{
    hipLaunchKernelGGL((k_medium<TM>), dim3(blocks1(h->n)), dim3(NT), 0, h->stream, deps, dmu, D,
                       h->cfg.w0_vac, geo1(h), (TM*)h->cl2, h->cfg.mu_varies ? h->mu_r : nullptr,
                       (TM*)h->dlnmu, dflag, ext_of(h));
    return hipGetLastError();
}

template <typename TM>
static hipError_t launch_aniso(lbem_s* h, const double* dfac, int* dflag, int write)
{
    hipLaunchKernelGGL((k_aniso<TM>), dim3(blocks1(h->n)), dim3(NT), 0, h->stream, dfac, h->D, h->n,
                       (TM*)h->cl2, (TM*)h->ra, dflag, write);
    return hipGetLastError();
}

template <int D, typename TM, class R>
static hipError_t launch_fields(lbem_s* h, const R& rd, double* E, double* B, double* partials)
{
    hipLaunchKernelGGL((k_fields<D, TM, R>), dim3(blocks1(h->n)), dim3(NT), 0, h->stream, rd,
                       (const TM*)h->cl2, h->mu_set ? h->mu_r : nullptr, geo1(h), E, B, partials,
                       (const TM*)(h->ra_set ? h->ra : nullptr));
    return hipGetLastError();
}

template <typename T>
static MarchExt<T> march_ext(const lbem_s* h)
{
    MarchExt<T> e{};
    const CellExt b = ext_of(h);
    e.wx = b.kind[0] != 0;
    e.wy = b.kind[1] != 0;
    e.nx_ = e.wx && (b.kind[0] == 1) == (pair_a(2, 0) == 0 || pair_b(2, 0) == 0);
    e.ny_ = e.wy && (b.kind[1] == 1) == (pair_a(2, 0) == 1 || pair_b(2, 0) == 1);
    e.keep = (const T*)h->keep;
    e.ade = (const T*)h->ade;
    e.pin = (const T*)h->pol;
    e.pout = (T*)h->pol2;
    return e;
}

// 2D multi-step launches (k_march2d).  The paper's tau = 1/2 gets its own
// instantiation: the reflection collision folds at compile time.
template <class IO, int NS, int CPL, bool MU, bool TH, int EXT = 0>
static void launch_march(lbem_s* h, const IO& io, const double* amp)
{
    typedef typename IO::T T;
    MarchSrc<T> ms;
    ms.idx = h->msrc_idx;
    ms.val = (const T*)h->msrc_val;
    for (int k = 0; k < 8; ++k) ms.mask[k] = h->nmsrc ? h->msrc_mask[k] : 0u;
    AmpPack<T, NS> a;
    for (int j = 0; j < NS; ++j) a.a[j] = (T)(amp ? amp[j] : 0.0);
    const MarchGeo& g = EXT ? h->mgeo_x[EXT ? EXT - 1 : 0] : h->mgeo;
    const int wpb = EXT ? h->mwpb_x[EXT ? EXT - 1 : 0] : h->mwpb;
    hipLaunchKernelGGL((k_march2d<IO, NS, CPL, MU, TH, EXT>), dim3(g.nblocks), dim3(64 * wpb), 0, h->stream, io,
                       (const T*)h->cl2, (const T*)h->dlnmu, g, ms, a, (T)(1.0 / h->cfg.tau),
                       (int)(h->cfg.tau == 0.5), march_ext<T>(h));
}

template <class IO, int NS, int CPL, bool MU>
static void launch_march_th(lbem_s* h, const IO& io, const double* amp)
{
    // (the 16-bit formats scale by one factor either way)
    if constexpr (IO::DEV) launch_march<IO, NS, CPL, MU, false>(h, io, amp);
    else if (h->cfg.tau == 0.5) launch_march<IO, NS, CPL, MU, true>(h, io, amp);
    else launch_march<IO, NS, CPL, MU, false>(h, io, amp);
}

template <class IO, int CPL>
static hipError_t go_march(lbem_s* h, const IO& io, const double* amp, int ns)
{
    if (h->mu_set) {
        if (ns == 4) launch_march_th<IO, 4, CPL, true>(h, io, amp);
        else if (ns == 3) launch_march_th<IO, 3, CPL, true>(h, io, amp);
        else if (ns == 2) launch_march_th<IO, 2, CPL, true>(h, io, amp);
        else return hipErrorInvalidValue;
    } else {
        if (ns == 4) launch_march_th<IO, 4, CPL, false>(h, io, amp);
        else if (ns == 3) launch_march_th<IO, 3, CPL, false>(h, io, amp);
        else if (ns == 2) launch_march_th<IO, 2, CPL, false>(h, io, amp);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// with walls, an absorber or a pole: launches of four and two
template <class IO, int CPL, bool MU>
static hipError_t go_march_ext(lbem_s* h, const IO& io, const double* amp, int ns)
{
    if (ns == 4 && h->ade) launch_march<IO, 4, CPL, MU, false, 2>(h, io, amp);
    else if (ns == 4) launch_march<IO, 4, CPL, MU, false, 1>(h, io, amp);
    else if (ns == 2 && h->ade) launch_march<IO, 2, CPL, MU, false, 2>(h, io, amp);
    else if (ns == 2) launch_march<IO, 2, CPL, MU, false, 1>(h, io, amp);
    else return hipErrorInvalidValue;
    if (h->ade) std::swap(h->pol, h->pol2);
    return hipGetLastError();
}

template <typename T, int CPL>
static hipError_t go_fused_c(lbem_s* h, const T* src, T* dst, const double* amp, int ns)
{
    typedef MarchPlain<T, CPL> IO;
    const IO io{src, dst, h->n};
    if (!has_bx(h)) return go_march<IO, CPL>(h, io, amp, ns);
    return h->mu_set ? go_march_ext<IO, CPL, true>(h, io, amp, ns) : go_march_ext<IO, CPL, false>(h, io, amp, ns);
}

template <typename T>
static hipError_t go_fused(lbem_s* h, const T* src, T* dst, const double* amp, int ns)
{
    if constexpr (sizeof(T) == 4) {
        if (h->mcpl == 2) return go_fused_c<T, 2>(h, src, dst, amp, ns);
    } else if (!offsets32(h->cfg.nx, sizeof(T))) {
        // launches of two without extras (make_fused_geo)
        typedef MarchPlain<T, 1, true> IO;
        const IO io{src, dst, h->n};
        if (ns != 2 || has_bx(h)) return hipErrorInvalidValue;
        if (h->mu_set) launch_march<IO, 2, 1, true, false>(h, io, amp);
        else launch_march<IO, 2, 1, false, false>(h, io, amp);
        return hipGetLastError();
    }
    return go_fused_c<T, 1>(h, src, dst, amp, ns);
}

template <typename T, int TX, int TY, bool MU, bool NTS>
static hipError_t go_fused3_t(lbem_s* h, const T* src, T* dst, const double* amp)
{
    FusedSrc<T> fs;
    fs.off = h->nfsrc ? h->fsrc_off : nullptr;
    fs.ent = h->fsrc_ent;
    fs.val = (const T*)h->fsrc_val;
    AmpPack<T, 2> a;
    for (int j = 0; j < 2; ++j) a.a[j] = (T)(amp ? amp[j] : 0.0);
    // tau = 1/2 folded at compile time (4.5 % at 256^3), other tau general
    if (h->cfg.tau == 0.5)
        hipLaunchKernelGGL((k_step_fused3d<T, TX, TY, MU, NTS, true>), dim3(h->fgeo.nblocks), dim3(TX * TY), 0,
                           h->stream, src, dst, (const T*)h->cl2, (const T*)h->dlnmu, h->fgeo, h->f3_lz, fs, a,
                           (T)(1.0 / h->cfg.tau), 1);
    else
        hipLaunchKernelGGL((k_step_fused3d<T, TX, TY, MU, NTS, false>), dim3(h->fgeo.nblocks), dim3(TX * TY), 0,
                           h->stream, src, dst, (const T*)h->cl2, (const T*)h->dlnmu, h->fgeo, h->f3_lz, fs, a,
                           (T)(1.0 / h->cfg.tau), 0);
    return hipGetLastError();
}

template <typename T, bool NTS>
static hipError_t go_fused3_n(lbem_s* h, const T* src, T* dst, const double* amp)
{
    if constexpr (std::is_same<T, float>::value) {
        if (h->f3_tx == 64 && h->f3_ty == 8) {
            if (h->mu_set) return go_fused3_t<T, 64, 8, true, NTS>(h, src, dst, amp);
            return go_fused3_t<T, 64, 8, false, NTS>(h, src, dst, amp);
        }
    }
    if (h->mu_set) {
        if (h->f3_tx == 64) return go_fused3_t<T, 64, 4, true, NTS>(h, src, dst, amp);
        return go_fused3_t<T, 32, 8, true, NTS>(h, src, dst, amp);
    }
    if (h->f3_tx == 64) return go_fused3_t<T, 64, 4, false, NTS>(h, src, dst, amp);
    return go_fused3_t<T, 32, 8, false, NTS>(h, src, dst, amp);
}

template <typename T>
static hipError_t go_fused3(lbem_s* h, const T* src, T* dst, const double* amp)
{
    return h->nts ? go_fused3_n<T, true>(h, src, dst, amp) : go_fused3_n<T, false>(h, src, dst, amp);
}

// formats with a multi-step kernel: all but plain FP16
static bool fused_format(const lbem_s* h) { return h->prec <= LBEM_F32 || is_dev(h->prec); }

// steps per launch of lbem_step
static int fused_steps(const lbem_s* h)
{
    if (!fused_format(h) || h->streaming != LBEM_STREAM_PULL) return 1;
    if (!has_bx(h)) return h->fuse_ns;
    // walls (2D), an absorber or a pole, no anisotropy
    return !h->ra_set && (h->D == 2 || !ext_of(h).walls()) && (!h->ade || h->pol2) ? std::max(1, h->ext_ns) : 1;
}

// 3D FP32 pairs on tiles of up to 64 x 13 stored cells
template <bool MU, bool EXT, bool TH>
static hipError_t launch_pair_f32(lbem_s* h, const float* src, float* dst, const AmpPack<float, 2>& a, const PairExt& ex)
{
    PairSrc ps;
    ps.flag = h->psrc_flag;
    ps.idx = h->psrc_idx;
    ps.val = h->psrc_val;
    ps.pair = h->psrc_pair;
    if (h->nts)
        hipLaunchKernelGGL((k_pair_f32<MU, EXT, TH, true>), dim3(h->pgeo.nblocks), dim3(1024), 0, h->stream, src, dst,
                           (const float*)h->cl2, (const float*)h->dlnmu, h->pgeo, ps, a, (float)(1.0 / h->cfg.tau),
                           (int)TH, ex);
    else
        hipLaunchKernelGGL((k_pair_f32<MU, EXT, TH, false>), dim3(h->pgeo.nblocks), dim3(1024), 0, h->stream, src, dst,
                           (const float*)h->cl2, (const float*)h->dlnmu, h->pgeo, ps, a, (float)(1.0 / h->cfg.tau),
                           (int)TH, ex);
    return hipGetLastError();
}

static hipError_t go_pair_f32(lbem_s* h, const float* src, float* dst, const double* amp)
{
    AmpPack<float, 2> a;
    for (int j = 0; j < 2; ++j) a.a[j] = (float)(amp ? amp[j] : 0.0);
    PairExt ex;
    ex.keep = (const float*)h->keep;
    ex.ade = (const float*)h->ade;
    ex.pin = (const float*)h->pol;
    ex.pout = (float*)h->pol2;
    const bool th = h->cfg.tau == 0.5;
    if (!has_bx(h)) {
        if (h->mu_set)
            return th ? launch_pair_f32<true, false, true>(h, src, dst, a, ex)
                      : launch_pair_f32<true, false, false>(h, src, dst, a, ex);
        return th ? launch_pair_f32<false, false, true>(h, src, dst, a, ex)
                  : launch_pair_f32<false, false, false>(h, src, dst, a, ex);
    }
    hipError_t e;
    if (h->mu_set)
        e = th ? launch_pair_f32<true, true, true>(h, src, dst, a, ex)
               : launch_pair_f32<true, true, false>(h, src, dst, a, ex);
    else
        e = th ? launch_pair_f32<false, true, true>(h, src, dst, a, ex)
               : launch_pair_f32<false, true, false>(h, src, dst, a, ex);
    if (h->ade) std::swap(h->pol, h->pol2);
    return e;
}

// plain formats: populations stored as S, arithmetic in T
template <int D, typename T, typename S = T>
struct PlainImpl : Impl {
    template <int RM, int WM, bool MU, bool NTS>
    static hipError_t go_xrow(lbem_s* h, const S* src, S* dst, T amp)
    {
        hipLaunchKernelGGL((k_step_xrow<T, RM, WM, MU, S, NTS, 2>), dim3(h->xgeo.nblocks), dim3(NT), 0, h->stream,
                           src, dst, (const T*)h->cl2, (const T*)h->dlnmu, h->xgeo,
                           h->nxsrc ? h->xsrc_off : nullptr, h->xsrc_ent, (const T*)h->xsrc_val, amp,
                           (T)(1.0 / h->cfg.tau), (int)(h->cfg.tau == 0.5));
        return hipGetLastError();
    }
    template <int RM, int WM, int V, bool MU, bool BX = false>
    static hipError_t go(lbem_s* h, const S* src, S* dst, T amp)
    {
        if constexpr (D == 3 && !BX && V == 1) {
            if (h->xrow) return h->nts ? go_xrow<RM, WM, MU, true>(h, src, dst, amp)
                                       : go_xrow<RM, WM, MU, false>(h, src, dst, amp);
        }
        SrcArgs<T> s;
        s.off = h->nsrc ? h->src_off : nullptr;
        s.ent = h->src_ent;
        s.val = (const T*)h->src_val;
        s.amp = amp;
        const double om = 1.0 / h->cfg.tau;
        if (h->nts) {
            hipLaunchKernelGGL((k_step_plain<D, T, RM, WM, V, MU, BX, S, true>), dim3(h->geo.nblocks), dim3(NT), 0,
                               h->stream, src, dst, (const T*)h->cl2, (const T*)h->dlnmu, h->geo, s, (T)om,
                               (int)(h->cfg.tau == 0.5), ext_of(h));
            return hipGetLastError();
        }
        hipLaunchKernelGGL((k_step_plain<D, T, RM, WM, V, MU, BX, S>), dim3(h->geo.nblocks), dim3(NT), 0,
                           h->stream, src, dst, (const T*)h->cl2, (const T*)h->dlnmu, h->geo, s, (T)om,
                           (int)(h->cfg.tau == 0.5), ext_of(h));
        return hipGetLastError();
    }
    template <int RM, int WM>
    static hipError_t go_v(lbem_s* h, const S* src, S* dst, T amp)
    {
        if constexpr (WM == W_LOCAL && RM != R_PULL_SWAP) {
            if (has_bx(h)) {   // pull streaming only (AA is refused with walls or an absorber)
                if (h->mu_set) return go<RM, WM, 1, true, true>(h, src, dst, amp);
                return go<RM, WM, 1, false, true>(h, src, dst, amp);
            }
        }
        if (h->mu_set) return go<RM, WM, 1, true>(h, src, dst, amp);
        switch (h->vec) {
            case 2: return go<RM, WM, 2, false>(h, src, dst, amp);
            case 4:
                if constexpr (D == 2) return go<RM, WM, 4, false>(h, src, dst, amp);
                return hipErrorInvalidValue;
            default: return go<RM, WM, 1, false>(h, src, dst, amp);
        }
    }
    hipError_t step(lbem_s* h, double amp) override
    {
        S* a = (S*)h->pop[h->cur];
        if (h->streaming == LBEM_STREAM_AA) {
            hipError_t e;
            if (h->layout == LAYOUT_NATURAL) {
                e = go_v<R_LOCAL, W_SWAP>(h, a, a, (T)amp);
                h->layout = LAYOUT_AA_SWAPPED;
            } else {
                e = go_v<R_PULL_SWAP, W_PUSH>(h, a, a, (T)amp);
                h->layout = LAYOUT_NATURAL;
            }
            return e;
        }
        S* b = (S*)h->pop[1 - h->cur];
        hipError_t e = h->layout == LAYOUT_NATURAL ? go_v<R_LOCAL, W_LOCAL>(h, a, b, (T)amp)
                                                   : go_v<R_PULL, W_LOCAL>(h, a, b, (T)amp);
        h->cur = 1 - h->cur;
        h->layout = LAYOUT_PULL_PENDING;
        return e;
    }
    hipError_t step_fused(lbem_s* h, const double* amp, int ns) override
    {
        if constexpr (!std::is_same<S, T>::value) {
            return hipErrorInvalidValue;   // the multi-step kernels keep FP64/FP32 storage
        } else {
            const T* a = (const T*)h->pop[h->cur];
            T* b = (T*)h->pop[1 - h->cur];
            hipError_t e;
            if constexpr (D == 2) e = go_fused<T>(h, a, b, amp, ns);
            else if constexpr (std::is_same<T, float>::value)
                e = h->pair_f32 || has_bx(h) ? go_pair_f32(h, a, b, amp) : go_fused3<T>(h, a, b, amp);
            else e = go_fused3<T>(h, a, b, amp);
            h->cur = 1 - h->cur;
            return e;
        }
    }
    hipError_t fields(lbem_s* h, double* E, double* B, double* partials) override
    {
        const S* a = (const S*)h->pop[h->cur];
        const CellExt bc = ext_of(h);
        if (h->layout == LAYOUT_NATURAL)
            return launch_fields<D, T>(h, PlainReader<D, S, R_LOCAL>{a, h->n, bc}, E, B, partials);
        if (h->layout == LAYOUT_PULL_PENDING)
            return launch_fields<D, T>(h, PlainReader<D, S, R_PULL>{a, h->n, bc}, E, B, partials);
        return launch_fields<D, T>(h, PlainReader<D, S, R_PULL_SWAP>{a, h->n, bc}, E, B, partials);
    }
    hipError_t init(lbem_s* h, const double* dE, const double* dB) override
    {
        h->cur = 0;
        h->layout = LAYOUT_NATURAL;
        hipLaunchKernelGGL((k_init_plain<D, T, S>), dim3(blocks1(h->n)), dim3(NT), 0, h->stream, dE, dB,
                           (const T*)h->cl2, h->n, (S*)h->pop[0], (const T*)(h->ra_set ? h->ra : nullptr));
        return hipGetLastError();
    }
    hipError_t medium(lbem_s* h, const double* deps, const double* dmu, int* dflag) override
    {
        return launch_medium<D, T>(h, deps, dmu, dflag);
    }
};

template <int D, typename H, bool GH>
struct DevImpl : Impl {
    static float* M(lbem_s* h, int k) { return (float*)h->pop[k]; }
    static H* Dv(lbem_s* h, int k)
    {
        const int P = Lat<D>::P;
        return (H*)(h->pop[k] + align256((size_t)(P + D) * h->n * 4));
    }
    template <bool MU, bool NTS, int NTB, int EXT = 0>
    static void go_row_n(lbem_s* h, int from, int to, const int* so, float amp, float om, int th)
    {
        hipLaunchKernelGGL((k_step_dev3r<H, GH, MU, NTS, 2, NTB, EXT>), dim3(h->rgeo.nblocks), dim3(NTB), 0,
                           h->stream, M(h, from), Dv(h, from), M(h, to), Dv(h, to), (const float*)h->cl2,
                           (const float*)h->dlnmu, h->rgeo, so, h->rsrc_ent, h->rsrc_val, amp, om, th, ext_of(h));
    }
    // the row-tile step with cell extras (walls, dispersion, absorbing
    // layer): 512-thread tiles, no anisotropy
    static bool row_ext_ok(const lbem_s* h)
    {
        return h->rowk && !h->ra_set && h->rntb == 512;
    }
    template <bool MU>
    static hipError_t go_row(lbem_s* h, int from, int to, const int* so, float amp, float om, int th)
    {
        if constexpr (D == 3) {
            const int nb = h->rntb;
            if (h->nts) {
                if (nb == 1024) go_row_n<MU, true, 1024>(h, from, to, so, amp, om, th);
                else if (nb == 512) go_row_n<MU, true, 512>(h, from, to, so, amp, om, th);
                else go_row_n<MU, true, 256>(h, from, to, so, amp, om, th);
            } else {
                if (nb == 1024) go_row_n<MU, false, 1024>(h, from, to, so, amp, om, th);
                else if (nb == 512) go_row_n<MU, false, 512>(h, from, to, so, amp, om, th);
                else go_row_n<MU, false, 256>(h, from, to, so, amp, om, th);
            }
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    }
    // BX: 0 no cell extras, 1 walls only, 2 walls, dispersion and absorber
    template <int RM, int V, bool MU, int BX = 0>
    static hipError_t go(lbem_s* h, int from, int to, float amp)
    {
        SrcArgs<float> s;
        if constexpr (D == 3 && BX != 0 && RM == R_PULL) {
            if (row_ext_ok(h)) {
                const int* so = h->nrsrc ? h->rsrc_off : nullptr;
                const float om = (float)(1.0 / h->cfg.tau);
                const int th = h->cfg.tau == 0.5;
                // row extras mask: 1 walls, 2 dispersion / absorber
                if constexpr (BX == 1) {
                    if (h->nts) go_row_n<MU, true, 512, 1>(h, from, to, so, amp, om, th);
                    else go_row_n<MU, false, 512, 1>(h, from, to, so, amp, om, th);
                } else if (ext_of(h).walls()) {
                    if (h->nts) go_row_n<MU, true, 512, 3>(h, from, to, so, amp, om, th);
                    else go_row_n<MU, false, 512, 3>(h, from, to, so, amp, om, th);
                } else {
                    if (h->nts) go_row_n<MU, true, 512, 2>(h, from, to, so, amp, om, th);
                    else go_row_n<MU, false, 512, 2>(h, from, to, so, amp, om, th);
                }
                return hipGetLastError();
            }
        }
        if constexpr (D == 3 && !BX && RM == R_PULL) {
            if (h->rowk) {
                const int* so = h->nrsrc ? h->rsrc_off : nullptr;
                const float om = (float)(1.0 / h->cfg.tau);
                const int th = h->cfg.tau == 0.5;
                return go_row<MU>(h, from, to, so, amp, om, th);
            }
        }
        if constexpr (D == 3 && !BX) {
            if (h->zmarch) {
                s.off = h->nzsrc ? h->zsrc_off : nullptr;
                s.ent = h->zsrc_ent;
                s.val = (const float*)h->zsrc_val;
                s.amp = amp;
                if (h->nts)
                    hipLaunchKernelGGL((k_step_dev3z<H, GH, RM, MU, true>), dim3(h->zgeo.nblocks), dim3(NT), 0,
                                       h->stream, M(h, from), Dv(h, from), M(h, to), Dv(h, to),
                                       (const float*)h->cl2, (const float*)h->dlnmu, h->zgeo, h->zlz, s,
                                       (float)(1.0 / h->cfg.tau), (int)(h->cfg.tau == 0.5));
                else
                    hipLaunchKernelGGL((k_step_dev3z<H, GH, RM, MU>), dim3(h->zgeo.nblocks), dim3(NT), 0,
                                       h->stream, M(h, from), Dv(h, from), M(h, to), Dv(h, to),
                                       (const float*)h->cl2, (const float*)h->dlnmu, h->zgeo, h->zlz, s,
                                       (float)(1.0 / h->cfg.tau), (int)(h->cfg.tau == 0.5));
                return hipGetLastError();
            }
        }
        s.off = h->nsrc ? h->src_off : nullptr;
        s.ent = h->src_ent;
        s.val = (const float*)h->src_val;
        s.amp = amp;
        if (h->nts) {
            hipLaunchKernelGGL((k_step_dev<D, H, GH, RM, V, MU, BX, true>), dim3(h->geo.nblocks), dim3(NT), 0,
                               h->stream, M(h, from), Dv(h, from), M(h, to), Dv(h, to), (const float*)h->cl2,
                               (const float*)h->dlnmu, h->geo, s, (float)(1.0 / h->cfg.tau),
                               (int)(h->cfg.tau == 0.5), ext_of(h));
            return hipGetLastError();
        }
        hipLaunchKernelGGL((k_step_dev<D, H, GH, RM, V, MU, BX>), dim3(h->geo.nblocks), dim3(NT), 0,
                           h->stream, M(h, from), Dv(h, from), M(h, to), Dv(h, to), (const float*)h->cl2,
                           (const float*)h->dlnmu, h->geo, s, (float)(1.0 / h->cfg.tau),
                           (int)(h->cfg.tau == 0.5), ext_of(h));
        return hipGetLastError();
    }
    template <int RM>
    static hipError_t go_v(lbem_s* h, int from, int to, float amp)
    {
        if (has_bx(h)) {
            // walls only: the closed-form collision (no anisotropy in 16 bits)
            const bool walls_only = h->ade == nullptr && h->keep == nullptr;
            if (h->mu_set)
                return walls_only ? go<RM, 1, true, 1>(h, from, to, amp) : go<RM, 1, true, 2>(h, from, to, amp);
            return walls_only ? go<RM, 1, false, 1>(h, from, to, amp) : go<RM, 1, false, 2>(h, from, to, amp);
        }
        if (h->mu_set) return go<RM, 1, true>(h, from, to, amp);
        switch (h->vec) {
            case 2: return go<RM, 2, false>(h, from, to, amp);
            case 4:
                if constexpr (D == 2) return go<RM, 4, false>(h, from, to, amp);
                return hipErrorInvalidValue;
            default: return go<RM, 1, false>(h, from, to, amp);
        }
    }
    hipError_t step(lbem_s* h, double amp) override
    {
        hipError_t e = h->layout == LAYOUT_NATURAL ? go_v<R_LOCAL>(h, h->cur, 1 - h->cur, (float)amp)
                                                   : go_v<R_PULL>(h, h->cur, 1 - h->cur, (float)amp);
        h->cur = 1 - h->cur;
        h->layout = LAYOUT_PULL_PENDING;
        return e;
    }
    hipError_t step_fused(lbem_s* h, const double* amp, int ns) override
    {
        if constexpr (D == 3) {
            const PairSrc ps{h->psrc_flag, h->psrc_idx, h->psrc_val, h->psrc_pair};
            AmpPack<float, 2> a;
            for (int j = 0; j < 2; ++j) a.a[j] = (float)(amp ? amp[j] : 0.0);
            const int from = h->cur, to = 1 - h->cur;
            const float om = (float)(1.0 / h->cfg.tau);
            const int th = h->cfg.tau == 0.5;
            if (h->mu_set)
                hipLaunchKernelGGL((k_pair_dev3<H, GH, true>), dim3(h->pgeo.nblocks), dim3(1024), 0, h->stream,
                                   M(h, from), Dv(h, from), M(h, to), Dv(h, to), (const float*)h->cl2,
                                   (const float*)h->dlnmu, h->pgeo, ps, a, om, th);
            else
                hipLaunchKernelGGL((k_pair_dev3<H, GH, false>), dim3(h->pgeo.nblocks), dim3(1024), 0, h->stream,
                                   M(h, from), Dv(h, from), M(h, to), Dv(h, to), (const float*)h->cl2,
                                   (const float*)h->dlnmu, h->pgeo, ps, a, om, th);
            h->cur = to;
            return hipGetLastError();
        } else {
            typedef MarchDev<H, GH, 1> IO;
            const int from = h->cur, to = 1 - h->cur;
            h->cur = to;
            return go_march<IO, 1>(h, IO{M(h, from), Dv(h, from), M(h, to), Dv(h, to), h->n}, amp, ns);
        }
    }
    hipError_t fields(lbem_s* h, double* E, double* B, double* partials) override
    {
        if (h->layout == LAYOUT_NATURAL)
            return launch_fields<D, float>(h, DevReader<D, H, GH, R_LOCAL>{M(h, h->cur), Dv(h, h->cur), h->n,
                                                                            ext_of(h)},
                                           E, B, partials);
        if constexpr (D == 3) {
            // fields alone: tiles that decode each cell once (the diagnostics'
            // partial sums keep the per-cell kernel's order)
            if (!partials && h->ftgeo.nblocks && !ext_of(h).walls()) {
                hipLaunchKernelGGL((k_fields_dev3<H, GH>), dim3(h->ftgeo.nblocks), dim3(1024), 0, h->stream,
                                   M(h, h->cur), Dv(h, h->cur), (const float*)h->cl2, h->ftgeo, E, B);
                return hipGetLastError();
            }
        }
        return launch_fields<D, float>(h, DevReader<D, H, GH, R_PULL>{M(h, h->cur), Dv(h, h->cur), h->n,
                                                                       ext_of(h)}, E,
                                       B, partials);
    }
    hipError_t init(lbem_s* h, const double* dE, const double* dB) override
    {
        h->cur = 0;
        h->layout = LAYOUT_NATURAL;
        hipLaunchKernelGGL((k_init_dev<D, H, GH>), dim3(blocks1(h->n)), dim3(NT), 0, h->stream, dE, dB,
                           (const float*)h->cl2, h->n, M(h, 0), Dv(h, 0));
        return hipGetLastError();
    }
    hipError_t medium(lbem_s* h, const double* deps, const double* dmu, int* dflag) override
    {
        return launch_medium<D, float>(h, deps, dmu, dflag);
    }
};

// the dispatch objects, one instantiation unit of impl.hip each
Impl* make_plain2d(int prec);
Impl* make_dev2d(int prec);
Impl* make_plain3d(int prec);
Impl* make_dev3d_f16(int prec);
Impl* make_dev3d_bf16(int prec);
