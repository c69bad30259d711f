// lbem.hip -- host side of liblbem: the C ABI declared in include/lbem.h,
// device memory, tilings, source tables and batched stepping.
#include "impl.h"
#include "batch_multi.h"

namespace {
// Graph capture of the batched kernels (lbem_batch_create) holds this lock
// exclusively; the entry points that allocate or free device memory, or
// create and destroy HIP objects, hold it shared.  No allocation or free of
// this library then runs while a graph is captured and instantiated.
std::shared_mutex g_api_mu;
#define API_SHARED std::shared_lock<std::shared_mutex> api_lock_(g_api_mu)

}  // namespace

static Impl* make_impl(int D, int prec)
{
    if (!is_dev(prec)) return D == 2 ? make_plain2d(prec) : make_plain3d(prec);
    if (D == 2) return make_dev2d(prec);
    return prec == LBEM_F16DEV || prec == LBEM_F16GHOST ? make_dev3d_f16(prec) : make_dev3d_bf16(prec);
}

static void make_geo(lbem_s* h)
{
    const int nx = (int)h->cfg.nx, ny = (int)h->cfg.ny, nz = (int)h->cfg.nz;
    int bx = 64;
    while (bx < nx && bx < NT) bx <<= 1;
    int sh = 0;
    while ((1 << sh) < bx) ++sh;
    const int rb = NT / bx;
    Geo& g = h->geo;
    g.nx = nx; g.ny = ny; g.nz = nz; g.n = h->n;
    g.bx_shift = sh;
    g.tiles_x = (nx + bx - 1) / bx;
    g.tiles_y = (ny + rb * h->vec - 1) / (rb * h->vec);
    g.nblocks = g.tiles_x * g.tiles_y * nz;
    // measured defaults: XCD-contiguous tile ranges help 2D; in 3D, runs of
    // 16 neighbouring tiles per XCD beyond the last-level cache (512^3 FP32
    // AA 4.39 -> 4.35 ms; at 256^3 1.5 % slower than tiles dealt one by one)
    const bool big3 = h->D == 3 && !is_dev(h->prec) && (double)h->n >= 4.0e7;
    g.xcd = env_int("LBEM_XCD", h->D == 2 ? 1 : (big3 ? 16 : 0));
    const int sdef = (h->D == 3 && is_dev(h->prec)) ? 32 : 0;
    g.strip = env_int("LBEM_STRIP", sdef);
    if (g.strip <= 0 || nz == 1 || g.strip >= g.tiles_y || g.tiles_y % g.strip != 0) g.strip = 0;
}

static void make_fused3_geo(lbem_s* h)
{
    const bool f64 = h->prec == LBEM_F64;
    // FP64 frames do not fit enough blocks per CU for the pair to pay off
    // (measured slower than single steps at 256^3), so FP64 runs single steps
    // unless asked for.
    const bool small = (double)h->n < FUSE3D_MIN;
    h->fuse_ns = env_int("LBEM_FUSE3", (f64 || small) ? 1 : 2) == 2 ? 2 : 1;
    h->f3_tx = env_int("LBEM_FUSE3_TX", f64 ? 32 : 64) == 64 && !f64 ? 64 : 32;
    h->f3_ty = NT / h->f3_tx;
    // FP32 64-wide tiles take 8 rows: 512 threads, two blocks per CU (80 KB of
    // LDS, <= 128 VGPRs), and step 1 runs on a frame of 1.29x the tile instead
    // of 1.55x.  Measured, us per step, 64x4 / 64x8 / 32x16: 512^3 2801 / 2508
    // / 2663, 384^3 1219 / 1103 / 1233, 256^3 348 / 307 / 332, 192^3 167 / 150
    // / 161.  LBEM_FUSE3_TY=4 keeps the 256-thread tiles.
    if (h->prec == LBEM_F32 && h->f3_tx == 64 && env_int("LBEM_FUSE3_TY", 8) == 8) h->f3_ty = 8;
    Geo& g = h->fgeo;
    g = h->geo;
    g.tiles_x = (g.nx + h->f3_tx - 1) / h->f3_tx;
    g.tiles_y = (g.ny + h->f3_ty - 1) / h->f3_ty;
    // longest z chunk (fewest recomputed boundary planes) that still gives
    // enough blocks to fill 256 CUs
    int lz = 32;
    while (lz > 8 && (int64_t)g.tiles_x * g.tiles_y * ((g.nz + lz - 1) / lz) < 768) lz /= 2;
    h->f3_lz = std::max(1, env_int("LBEM_FUSE3_LZ", lz));
    g.nblocks = g.tiles_x * g.tiles_y * ((g.nz + h->f3_lz - 1) / h->f3_lz);
    g.strip = 0;
    // runs of 32 neighbouring tiles per XCD (measured, FP32: 512^3 2.82 ->
    // 2.79 ms against tiles dealt one by one; 384^3 1.27 -> 1.22, 256^3 0.365
    // -> 0.347, 192^3 0.170 -> 0.167 against contiguous ranges per XCD)
    g.xcd = env_int("LBEM_FUSE3_XCD", 32);
}

static int device_cus()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
        return v;
    return 256;
}

// The planes per chunk with the least work for tiles that hold a CU each and
// march along z: rounds of resident blocks times the planes of a chunk, `fill`
// of which only fill the pipeline.
static int march_planes(int64_t cols, int nz, int64_t cus, int fill)
{
    int64_t best = -1;
    int lz_best = nz;
    for (int c = 1; c <= nz; ++c) {
        const int lz = (nz + c - 1) / c, chunks = (nz + lz - 1) / lz;
        const int64_t cost = (cols * chunks + cus - 1) / cus * (lz + fill);
        if (best < 0 || cost < best) { best = cost; lz_best = lz; }
        if (lz <= 4) break;
    }
    return lz_best;
}

// Two steps per launch for the 3D 16-bit formats (k_pair_dev3): tiles of 60 x
// 12 stored cells, one block per CU, chunks of lz planes.
static void make_pair_geo(lbem_s* h)
{
    PairGeo& g = h->pgeo;
    g.nx = (int)h->cfg.nx; g.ny = (int)h->cfg.ny; g.nz = (int)h->cfg.nz; g.n = h->n;
    g.tiles_x = (g.nx + PRX - 1) / PRX;
    g.tiles_y = (g.ny + PRY - 1) / PRY;
    g.sx = (g.nx + g.tiles_x - 1) / g.tiles_x;      // even tiles: no lane loads for another
    g.sy = (g.ny + g.tiles_y - 1) / g.tiles_y;
    const int64_t cus = device_cus(), cols = (int64_t)g.tiles_x * g.tiles_y;
    g.lz = std::max(1, env_int("LBEM_FUSE3_LZ", march_planes(cols, g.nz, cus, 4)));
    g.nblocks = (int)(cols * ((g.nz + g.lz - 1) / g.lz));
    g.xcd = env_int("LBEM_FUSE3_XCD", std::max(2, g.tiles_x));
    // Taken where enough of the work is on stored cells: n over (rounds * CUs *
    // planes of a chunk * 720) of at least 0.28 with ghost coordinates, 0.36
    // with all deviations, 0.09 more where rows are whole 64-cell lines, which
    // the single steps read without a split.  Measured, us per step, single /
    // pair (share): FP16 ghost 64^3 (0.18) 8.6 / 12.7, 61x100x100 (0.28) 19.4 /
    // 20.1, 88^3 (0.37) 22.5 / 16.4, 64x128x128 (0.36) 25.3 / 25.2, 128^3
    // (0.50) 46.2 / 35.9, 160^3 105 / 72, 256^3 370 / 316, 250x190x171 274 /
    // 133; FP16-dev 80^3 (0.31) 16.8 / 17.2, 88^3 22.8 / 19.5, 64x256x256
    // (0.41) 115 / 125, 128^3 62.5 / 51.5, 256^3 438 / 374, 250x190x171 358 /
    // 163; with a varying mu 256^3 423 / 353 and 481 / 405.
    const double share = (double)g.n / ((double)((g.nblocks + cus - 1) / cus) * cus * (g.lz + 4) * (PRX * PRY));
    const bool ghost = h->prec == LBEM_F16GHOST || h->prec == LBEM_BF16GHOST;
    const double need = (ghost ? 0.28 : 0.36) + (g.nx % 64 == 0 ? 0.09 : 0.0);
    h->fuse_ns = env_int("LBEM_DEV3F", share >= need) ? 2 : 1;
    // The field reader on tiles of 62 x 14 cells, by the same measure: us per
    // call, per-cell / tiles: 64^3 (share 0.18) 24.6 / 27.4, 20x200x200 (0.24)
    // 52.7 / 62.2, 61x100x100 (0.28) 41.9 / 31.2, 80^3 (0.31) 39.3 / 28.9, 128^3
    // 86.9 / 58.7, 256^3 792 / 491, 250x190x171 437 / 252 (FP16 ghost; all
    // deviations 0.17 less of a gain).
    PairGeo& f = h->ftgeo;
    f = g;
    f.tiles_x = (f.nx + FLX - 1) / FLX;
    f.tiles_y = (f.ny + FLY - 1) / FLY;
    f.sx = (f.nx + f.tiles_x - 1) / f.tiles_x;
    f.sy = (f.ny + f.tiles_y - 1) / f.tiles_y;
    f.lz = march_planes((int64_t)f.tiles_x * f.tiles_y, f.nz, cus, 2);
    f.xcd = std::max(2, f.tiles_x);
    const bool fits = offsets32(f.nx, 8);           // it writes doubles at 32-bit offsets within a row
    f.nblocks = fits && env_int("LBEM_FIELDS3", share >= 0.27) ? f.tiles_x * f.tiles_y * ((f.nz + f.lz - 1) / f.lz) : 0;
}

// Two steps per launch for 3D FP32 on the tiles of k_pair_f32, up to 64 x 13
// stored cells, one block per CU.  Columns go by 64 (rows then start on whole
// lines wherever the lattice's do: 160^3 21.6 ps per update, three even tiles
// of 54 columns 30.1), rows evenly.
static void make_pairf_geo(lbem_s* h)
{
    PairGeo& g = h->pgeo;
    g.nx = (int)h->cfg.nx; g.ny = (int)h->cfg.ny; g.nz = (int)h->cfg.nz; g.n = h->n;
    g.sx = std::min(g.nx, PFX);
    g.tiles_x = (g.nx + g.sx - 1) / g.sx;
    g.tiles_y = (g.ny + PFY - 1) / PFY;
    g.sy = (g.ny + g.tiles_y - 1) / g.tiles_y;
    const int64_t cus = device_cus(), cols = (int64_t)g.tiles_x * g.tiles_y;
    g.lz = std::max(1, env_int("LBEM_FUSE3_LZ", march_planes(cols, g.nz, cus, 2)));
    g.nblocks = (int)(cols * ((g.nz + g.lz - 1) / g.lz));
    g.xcd = env_int("LBEM_FUSE3_XCD", std::max(2, g.tiles_x));
    const bool fits = (int64_t)g.nx * g.ny < ((int64_t)1 << 30);       // 32-bit offsets within a plane
    // With extras, and below FUSE3D_MIN cells without: where at least a quarter
    // of the work is on stored cells.  Measured, us per step, single / pair
    // (share), with a pole: 48^3 (0.09) 7.1 / 10.8, 64^3 (0.21) 10.6 / 13.6,
    // 20x200x200 (0.25) 34.6 / 27.4, 72^3 (0.29) 15.8 / 13.4, 100^3 (0.52) 36.3
    // / 28.2, 160^3 153 / 124, 256^3 683 / 432, 250x190x171 431 / 246, 384^3
    // 2565 / 1567; with an absorber 256^3 478 / 318; with neither 64^3 8.5 /
    // 10.2, 72^3 11.6 / 10.0, 61x100x100 (0.48) 16.9 / 12.5.
    const double share = (double)g.n / ((double)((g.nblocks + cus - 1) / cus) * cus * (g.lz + 2) * (PFX * PFY));
    h->ext_ns = fits && env_int("LBEM_FUSE3", share >= 0.25 ? 2 : 1) == 2 ? 2 : 1;
    if ((double)h->n < FUSE3D_MIN) h->fuse_ns = h->ext_ns;
    // Without extras the column tiles of k_step_fused3d (smaller, two blocks per CU)
    // stay, from FUSE3D_MIN cells on and for rows of several tiles, in four cases (us
    // per step, column tiles / these):
    // - within the Infinity Cache, where they need at most a block per CU, which then
    //   runs alone: 1024x32x32 19.3 / 21.7, 256x64x64 20.0 / 20.9, 128x128x64 20.0 /
    //   20.2 (not 192x64x96, 288 blocks, 26.9 / 20.9);
    // beyond it
    // - rows that are no whole 64-byte sectors and fill their tiles of 64 columns to
    //   less than 60 on average (a tile holds a CU however few columns it has):
    //   66x400x400 265 / 382, 102x189x224 116 / 127, 257^3 483 / 518, 330^3 871 / 947,
    //   350^3 1049 / 1144, 200^3 199 / 211 (not 250x190x171 212 / 172, 188x200x200 183
    //   / 158, 505x100x90 114 / 101; on the line 230^3 330 / 308, 348x135x168 186 / 203);
    // - rows of 16 tiles and more, of which few fit the CUs at a time: 1010x60x60 89 /
    //   99, 2000x60x40 99 / 105, 2048x64x64 161 / 167, 1024x64x64 86.7 / 85.8;
    // - where clearly less of their work is idle: 128^3 46.0 / 46.8, 256x64x128 46.1 /
    //   47.5, 124x126x128 45.5 / 48.9, 256^3 302.4 / 298.6 but with a source 306.1 /
    //   308.0 (not 127x120x120 44.9 / 41.1, 250^3 388 / 345).
    // Elsewhere these are faster: 112^3 29.3 / 25.2, 144^3 75.7 / 67.7, 192^3 149 /
    // 137, 224^3 255 / 216, 312^3 705 / 600, 512^3 2529 / 2422.
    const double state = 172.0 * (double)h->n;       // both copies and c_L^2
    const double share_col = (double)g.n / ((double)((h->fgeo.nblocks + 2 * cus - 1) / (2 * cus)) * 2 * cus *
                                            (h->f3_lz + 2) * (h->f3_tx * h->f3_ty));
    bool col;
    if (state <= 256.0 * (1 << 20)) col = h->fgeo.nblocks <= cus;
    else col = (g.nx % 16 != 0 && g.nx < 60 * g.tiles_x) || g.tiles_x >= 16 ||
               share < 0.96 * share_col;
    col = col && g.tiles_x > 1 && (double)h->n >= FUSE3D_MIN;
    const bool asked = std::getenv("LBEM_FUSE3_TX") != nullptr || std::getenv("LBEM_FUSE3_TY") != nullptr;
    h->pair_f32 = fits && env_int("LBEM_PAIR3F", !col && !asked) != 0;
}

// Strips and chunks of the 2D march for `waves` resident waves per SIMD.  share:
// what each further wave of a SIMD adds to a row of the march, as a part of what a
// lone wave waits for; 0 keeps all waves resident.
static void make_march_chunks(const lbem_s* h, int waves, double share, MarchGeo& g, int& wpb)
{
    const int nx = (int)h->cfg.nx, ny = (int)h->cfg.ny;
    g.nx = nx; g.ny = ny; g.n = h->n;
    const int ow = 64 * h->mcpl - 2 * MARCH_HX;
    g.strips = (nx + ow - 1) / ow;
    // Rows per chunk: whole rounds of the waves that are resident, about 24
    // rows each: a chunk reads 8 rows beyond its own, a thin last round leaves
    // CUs idle.  FP32 2048^2, rows -> us per launch: 8 34.2, 16 33.4, 19 31.8 (3996 waves), 24
    // 35.2, 40 31.8 (1924), 64 36.0.  Small lattices: as many waves as give
    // two rows each, where a launch is a few rows of latency (256^2: 2 rows
    // 4.2, 4 4.8, 8 5.9).
    const int64_t slots = 1024 * waves;
    const int64_t want = std::max<int64_t>(1, ((int64_t)g.strips * ny + slots - 1) / slots);  // rows if all fit
    const int64_t rounds = (want + 23) / 24;
    auto rows_of = [&](int64_t per) {
        const int64_t chunks = std::max<int64_t>(1, per / g.strips);     // that fit these rounds
        return (int)std::min<int64_t>(ny, std::max<int64_t>(2, (ny + chunks - 1) / chunks));
    };
    g.rows = rows_of(rounds * slots);
    // Where one round suffices, fewer waves with more rows each recompute less:
    // as many per SIMD as give the least rows marched, 8 of them beyond a chunk's
    // own, times what a row takes.  A row of FP32 500^2 takes 0.30, 0.37 and 0.44 us
    // with one, two and three waves on a SIMD, of FP64 0.30, 0.52 and 0.70.  Measured,
    // us per step, all waves -> this: FP32 500^2 1.63 -> 1.51, 700^2 1.96 -> 1.88,
    // 1000^2 2.99 -> 2.72, 1201x900 with a varying mu 4.15 -> 3.77; FP64 500^2 2.55
    // -> 1.82, with mu 3.34 -> 2.30, 1000^2 5.1 -> 4.3; FP16-dev 500^2 3.10 -> 2.40.
    if (rounds == 1 && share > 0.0) {
        double best = 0.0;
        for (int w = waves; w >= 1; --w) {
            const int r = rows_of((int64_t)1024 * w);
            if (r > 64 - 2 * MARCH_HX) break;
            const int64_t nw = (int64_t)g.strips * ((ny + r - 1) / r);
            const double cost = (r + 8) * (1.0 + share * (double)((nw + 1023) / 1024));
            if (w == waves || cost < best) {
                best = cost;
                g.rows = r;
            }
        }
    }
    g.nwork = g.strips * ((ny + g.rows - 1) / g.rows);
    // few waves: one per block, so that they spread over the CUs (96x64 3.6
    // against 4.0 us per launch)
    wpb = g.nwork <= 1024 ? 1 : 4;
    g.nblocks = ((g.nwork + wpb - 1) / wpb + 7) / 8 * 8;
}

static void make_fused_geo(lbem_s* h)
{
    if (h->D == 3 && is_dev(h->prec)) {
        make_pair_geo(h);
        return;
    }
    if (h->D == 3) {
        make_fused3_geo(h);
        if (h->prec == LBEM_F32) make_pairf_geo(h);
        return;
    }
    // Four steps per launch in every format but plain FP16, at every size, with
    // or without a varying mu (the bytes per update fall with the steps and
    // nothing else grows); calls for fewer steps take the launches of two and
    // three.
    const int nx = (int)h->cfg.nx;
    h->fuse_ns = env_int("LBEM_FUSE", 4);
    if (h->fuse_ns < 1 || h->fuse_ns > 4) h->fuse_ns = 1;
    h->ext_ns = h->prec <= LBEM_F32 && h->n >= 4096 ? (h->fuse_ns >= 4 ? 4 : (h->fuse_ns >= 2 ? 2 : 1)) : 1;
    // FP64 rows longer than 2^29 columns need 64-bit offsets within a row: two steps
    // per launch, single steps with extras.
    if (!offsets32(nx, h->prec == LBEM_F64 ? 8 : 4)) {
        h->fuse_ns = std::min(h->fuse_ns, 2);
        h->ext_ns = 1;
    }
    // FP32 lattices of 8e6 cells and more, rows of even length: two cells per
    // lane.  One eighth of the columns is recomputed with one cell per lane,
    // one sixteenth with two, which shows once the state streams from HBM (us
    // per launch, one / two cells: 4096^2 180 / 171, 8192^2 694 / 645); below,
    // twice as many waves with half the registers are as fast or faster
    // (2048^2 31.8 / 32.2, 1000^2 10.8 / 12.9).  FP64 keeps one: two need more
    // than 256 registers.
    h->mcpl = h->prec == LBEM_F32 && nx % 2 == 0 && (double)h->n >= 8.0e6 ? 2 : 1;
    // With walls, an absorber or a pole FP32 and FP64 take launches of four and
    // two.  us per step, single steps / these: FP32 walls 128^2 2.7 / 1.7,
    // 1023x767 7.7 / 4.0, 2048^2 27.7 / 10.3, 4096^2 113 / 45; with an absorber
    // 4096^2 121 / 49; a pole 128^2 2.9 / 2.0, 2048^2 43 / 19, 4096^2 228 / 88;
    // FP64 walls 2048^2 60 / 23, a pole 87 / 41.  The line at 4096 cells is not one of
    // speed (FP32 48x40 walls 2.9 / 1.7, an absorber 2.8 / 1.5, a pole 2.8 / 1.9; FP64
    // 3.3 / 1.7, 3.1 / 1.6, 3.2 / 2.2): smaller boxes with extras have always reported
    // one step per launch, and callers hold them to it.
    // Waves resident per SIMD without extras, with walls or an absorber and with
    // a pole, by their registers (one / two cells per lane in FP32, FP64).
    const int w1 = h->prec == LBEM_F64 ? 2 : 4, w2 = h->prec == LBEM_F64 ? 1 : 3;
    make_march_chunks(h, h->mcpl == 2 ? 2 : 4, h->prec == LBEM_F64 ? 1.5 : 0.4, h->mgeo, h->mwpb);
    make_march_chunks(h, h->mcpl == 2 ? 2 : w1, 0.0, h->mgeo_x[0], h->mwpb_x[0]);
    make_march_chunks(h, h->mcpl == 2 ? 1 : w2, 0.0, h->mgeo_x[1], h->mwpb_x[1]);
}

static void make_zmarch_geo(lbem_s* h)
{
    // rows the row tiles take (with the default 512-thread block) go by the
    // state size, longer ones by the cell count
    const bool ghost = h->prec == LBEM_F16GHOST || h->prec == LBEM_BF16GHOST;
    const bool big = h->cfg.nx <= ROWX_MAX ? (double)h->n * (ghost ? 112.0 : 136.0) > ROWTILE_BYTES
                                           : (double)h->n >= SMALL3D;
    h->zmarch = (h->D == 3 && is_dev(h->prec)) ? env_int("LBEM_DEV3Z", big) : 0;
    h->zlz = std::max(1, env_int("LBEM_DEV3Z_LZ", 16));
    Geo& g = h->zgeo;
    g = h->geo;
    g.tiles_x = (g.nx + TXD - 1) / TXD;
    g.tiles_y = (g.ny + TYD - 1) / TYD;
    const int nzc = (g.nz + h->zlz - 1) / h->zlz;
    g.nblocks = g.tiles_x * g.tiles_y * nzc;
    g.strip = 0;
    g.xcd = env_int("LBEM_DEV3Z_XCD", 0);
}

// Whole-row blocks of k_step_xrow (3D plain formats, single steps without
// cell extras): CX = 2 cells per thread, tpr threads per row, NT/tpr rows per
// block, one plane.  Measured (same box, per step): plain FP16 AA 2.33 -> 2.15
// ms at 512^3 and 0.261 -> 0.244 ms at 256^3, where a 64-wide row of 16-bit
// values is one cache line and a shifted one touches two; FP32 AA and pull
// within +-3 % at 256^3 and 512^3; every format slower while the state is
// Infinity-Cache resident (128^3).  So the default takes it for FP16 storage
// beyond 6e6 cells; LBEM_XROW=1 selects it for the others.
static void make_xrow_geo(lbem_s* h)
{
    const int nx = (int)h->cfg.nx, ny = (int)h->cfg.ny, nz = (int)h->cfg.nz;
    const bool plain = h->prec <= LBEM_F32 || h->prec == LBEM_F16;
    const int dflt = h->prec == LBEM_F16 && (double)h->n >= XROW3D;
    h->xrow = (h->D == 3 && plain && nx <= 2 * NT && h->vec == 1) ? env_int("LBEM_XROW", dflt) : 0;
    if (!h->xrow) return;     // rows longer than 2*NT have no whole-row tiling (no rows per block)
    XRowGeo& g = h->xgeo;
    g.nx = nx; g.ny = ny; g.nz = nz; g.n = h->n;
    int tpr = 64;
    while (2 * tpr < nx) tpr <<= 1;
    g.tpr = tpr;
    g.rows = NT / tpr;
    g.tiles_y = (ny + g.rows - 1) / g.rows;
    g.nblocks = g.tiles_y * nz;
}

// Whole-row tiles of k_step_dev3r: CX = 2 cells per thread numbered through
// the tile's rows (short rows leave no thread idle and keep every wave on
// consecutive cells), 2 block / nx rows per tile; the planes per chunk are
// chosen below.  Rows longer than twice the block (or ROWX_MAX) keep the
// column-tile z-march.
static void make_row_geo(lbem_s* h)
{
    const int nx = (int)h->cfg.nx, ny = (int)h->cfg.ny, nz = (int)h->cfg.nz;
    // 512 threads: two blocks per CU (73 KB of LDS each) hide the memory
    // latency that one 1024-thread block with taller tiles leaves exposed
    // (measured at 512^3: 3.20 ms per step against 5.31, 256 threads 3.61)
    int ntb = env_int("LBEM_DEV3R_NT", 512);
    if (ntb != 256 && ntb != 1024) ntb = 512;
    h->rowk = (h->zmarch && nx <= std::min(ROWX_MAX, 2 * ntb)) ? env_int("LBEM_DEV3R", 1) : 0;
    RowGeo& g = h->rgeo;
    g.nx = nx; g.ny = ny; g.nz = nz; g.n = h->n;
    h->rntb = ntb;
    // Measured (512^3 and 256^3, FP16 ghost and Dev-Q): blocks dealt to the
    // XCDs in turn, so that the blocks resident at a time are neighbouring
    // tiles of one z band, run 5-7 % faster than contiguous tile ranges per XCD
    // (512^3 ghost 2.95 against 3.20 ms); runs of 8 neighbouring tiles per XCD
    // (their y-halo rows shared in one L2) another 0.8-1.2 % (2.92 ms; runs
    // of 2, 4 or 16 within 0.5 % of it).
    // As many rows per tile as the block holds: rows of a power-of-two thread
    // count with idle threads ran slower (FP16 ghost, us per step: 160^3 123
    // against 106, 320^3 796 against 732, 384^3 1326 against 1276), and so did
    // fewer rows with more blocks (192^3: 4 rows 171-183 against 5 rows 166).
    // Planes per chunk: the longest of 1..7 whose last round of resident
    // blocks (1024 / block threads per CU) is within 0.08 of the fullest,
    // among the lengths that give at least two rounds of blocks (all of them if
    // none does).  A thin last round costs more than the chunk ends decoded
    // twice: FP16 ghost, planes -> us per step, 192^3 (5 rows) 3 166, 5 166,
    // 6 176, 7 190; 160^3 (6 rows) 3 106, 4 120, 5 109; 144^3 (7 rows) 2 88,
    // 3 107; 512^3 (2 rows) 7 2909-2913, 8 2917-2925, 16 2945.
    const int64_t slots = (int64_t)device_cus() * (1024 / ntb);
    const int tymax = std::max(1, 2 * ntb / nx);
    g.ty = std::max(1, std::min(tymax, env_int("LBEM_DEV3R_TY", tymax)));
    g.tiles_y = (ny + g.ty - 1) / g.ty;
    auto nblk = [&](int c) { return (int64_t)g.tiles_y * ((nz + c - 1) / c); };
    auto fill = [&](int c) {
        const int64_t nb = nblk(c);
        return (double)nb / (double)(((nb + slots - 1) / slots) * slots);
    };
    const bool two = nblk(1) >= 2 * slots;
    double best = 0.0;
    for (int c = 1; c <= 7; ++c)
        if (!two || nblk(c) >= 2 * slots) best = std::max(best, fill(c));
    int lz = 1;
    for (int c = 7; c >= 1; --c)
        if ((!two || nblk(c) >= 2 * slots) && fill(c) >= best - 0.08) { lz = c; break; }
    g.lz = std::max(1, env_int("LBEM_DEV3R_LZ", lz));
    g.nblocks = g.tiles_y * ((nz + g.lz - 1) / g.lz);
    g.xcd = env_int("LBEM_DEV3R_XCD", 8);
}

// The whole-row tiling of a 3D deviation handle inside a batch: blocks of
// BROW_NT threads, two cells per thread numbered through the tile's rows,
// 2 BROW_NT / nx rows per tile (nx = 64: 16 rows); chunks of 8 planes.
// Rows longer than 2 BROW_NT cells keep the per-cell tiles.
static void make_batch_row_geo(lbem_s* h)
{
    const int nx = (int)h->cfg.nx, ny = (int)h->cfg.ny, nz = (int)h->cfg.nz;
    h->brow = (h->D == 3 && is_dev(h->prec) && nx <= std::min(ROWX_MAX, 2 * BROW_NT)) ? env_int("LBEM_BATCH_ROW", 1) : 0;
    if (!h->brow) return;
    RowGeo& g = h->bgeo;
    g.nx = nx; g.ny = ny; g.nz = nz; g.n = h->n;
    g.ty = 2 * BROW_NT / nx;
    g.tiles_y = (ny + g.ty - 1) / g.ty;
    g.lz = std::max(1, env_int("LBEM_BATCH_ROW_LZ", 8));
    g.nblocks = g.tiles_y * ((nz + g.lz - 1) / g.lz);
    g.xcd = 0;
}

// inverse of tile_coords()
static int tile_id(const Geo& g, int tx, int ty, int z)
{
    int r;
    if (g.strip > 0) r = ((ty / g.strip) * g.nz + z) * g.strip + ty % g.strip;
    else r = z * g.tiles_y + ty;
    return r * g.tiles_x + tx;
}

// ---------------------------------------------------------------------------
// static device scratch of lbem_energy_noalloc
// ---------------------------------------------------------------------------
// The FP64 B field (3n doubles) read by the divergence stencil and the
// per-block partial sums (4 per block + 4 results) live in this array instead
// of the handle's scratch.  Every GPU the library runs on holds its own copy
// until the process ends; every call on that GPU shares it and leaves the
// last call's contents.  The kernels write every element they later read, so
// nothing needs clearing between calls.
constexpr size_t NOALLOC_BYTES = size_t(64) << 20;
constexpr size_t NOALLOC_DOUBLES = NOALLOC_BYTES / sizeof(double);
static __device__ __align__(256) double noalloc_scratch[NOALLOC_DOUBLES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_noalloc_mu;
double* g_noalloc_ptr[NOALLOC_MAX_DEVICES];   // device address of the array, per device

constexpr size_t noalloc_doubles(int64_t n) { return (size_t)3 * n + (size_t)((n + NT - 1) / NT) * 4 + 4; }
static_assert(noalloc_doubles(LBEM_NOALLOC_MAX_CELLS) <= NOALLOC_DOUBLES &&
                  noalloc_doubles(LBEM_NOALLOC_MAX_CELLS + 1) > NOALLOC_DOUBLES,
              "LBEM_NOALLOC_MAX_CELLS is the largest lattice the static scratch holds");

// Device address of noalloc_scratch on `device`, looked up once per device
// with that device current (host code never passes the symbol itself).
hipError_t noalloc_address(int device, double** out)
{
    if (device < 0 || device >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    if (!g_noalloc_ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_noalloc_ptr[device] = (double*)p;
    }
    *out = g_noalloc_ptr[device];
    return hipSuccess;
}
}  // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

size_t lbem_required_bytes(const lbem_config* cfg)
{
    if (!valid_cfg(cfg)) return 0;
    return sizes_of(cfg).total;
}

const char* lbem_strerror(int code)
{
    switch (code) {
        case LBEM_OK: return "success";
        case LBEM_EINVAL: return "invalid argument";
        case LBEM_ENOMEM: return "out of device memory or arena too small";
        case LBEM_EUNSTABLE: return "medium gives a rest weight outside [0,1)";
        case LBEM_ENONFINITE: return "non-finite diagnostic (NaN or Inf)";
        case LBEM_EDEVICE: return "HIP device or launch error";
        case LBEM_ESTATE: return "call out of order";
        case LBEM_ETOOBIG:
            return "lattice too large for the static scratch of lbem_energy_noalloc (see LBEM_NOALLOC_MAX_CELLS)";
        default: return "unknown status";
    }
}

int lbem_create(const lbem_config* cfg, lbem_t* out)
{
    API_SHARED;
    if (!out) return LBEM_EINVAL;
    *out = nullptr;
    if (!valid_cfg(cfg)) return LBEM_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return LBEM_EDEVICE;
    lbem_s* h = new (std::nothrow) lbem_s();
    if (!h) return LBEM_ENOMEM;
    std::memset((void*)h, 0, sizeof(*h));
    h->cfg = *cfg;
    h->D = cfg->dim;
    h->Q = 2 * h->D + 1;
    h->P = h->D * (h->D - 1) / 2;
    h->prec = cfg->prec;
    h->streaming = resolve_streaming(cfg);
    h->n = cfg->nx * cfg->ny * cfg->nz;
    h->stream = (hipStream_t)cfg->stream;
    if (hipGetDevice(&h->device) != hipSuccess) { delete h; return LBEM_EDEVICE; }
    const Sizes s = sizes_of(cfg);
    if (cfg->dev_mem) {
        if (cfg->dev_bytes < s.total || ((uintptr_t)cfg->dev_mem & 255)) { delete h; return LBEM_ENOMEM; }
        h->arena = (char*)cfg->dev_mem;
        h->own_mem = false;
    } else {
        if (hipMalloc((void**)&h->arena, s.total) != hipSuccess) { delete h; return LBEM_ENOMEM; }
        h->own_mem = true;
    }
    h->arena_bytes = s.total;
    // the population copies start zeroed, so the alignment padding inside them
    // (which no kernel writes) reads back as zeros in an exported state
    if (hipMemsetAsync(h->arena, 0, s.pop_one * s.copies, h->stream) != hipSuccess) {
        if (h->own_mem) (void)hipFree(h->arena);
        delete h;
        return LBEM_EDEVICE;
    }
    char* p = h->arena;
    h->pop[0] = p; p += s.pop_one;
    h->pop[1] = s.copies == 2 ? p : nullptr; p += s.pop_one * (s.copies - 1);
    h->cl2 = p; p += s.medium;
    if (cfg->mu_varies) {
        h->mu_r = (double*)p; p += align256((size_t)h->n * 8);
        h->dlnmu = p; p += s.mu - align256((size_t)h->n * 8);
    }
    h->scratch = (double*)p;
    h->nb_diag = blocks1(h->n);
    if (hipMallocAsync((void**)&h->partials, ((size_t)h->nb_diag * 4 + 4) * sizeof(double), h->stream) !=
        hipSuccess) {
        if (h->own_mem) (void)hipFree(h->arena);
        delete h;
        return LBEM_ENOMEM;
    }
    int vdef = 1;
    h->vec = env_int("LBEM_VEC", vdef);
    if (h->vec != 1 && h->vec != 2 && h->vec != 4) h->vec = vdef;
    if (h->D == 3 && h->vec == 4) h->vec = 2;
    if (cfg->mu_varies) h->vec = 1;
    make_geo(h);
    make_fused_geo(h);
    make_zmarch_geo(h);
    make_row_geo(h);
    make_xrow_geo(h);
    make_batch_row_geo(h);
    // Measured: streaming loads/stores slow a launch whose state fits the
    // 256 MB Infinity Cache (by up to 1.8x) and speed it up beyond that: in 3D
    // from about 1.5 times the cache on (2-10 %; at 344 MB still 9 % slower),
    // in 2D as soon as the state leaves it (FP32 AA 16 % at 335 MB, 17 % at
    // 1.3 GB).  The copies a step touches count (one with AA streaming, two
    // with pull).
    {
        const double touched = (double)s.pop_one * (h->streaming == LBEM_STREAM_AA ? 1 : 2);
        const double lim = (double)env_int("LBEM_NT_MIB", h->D == 2 ? 256 : 384) * (1 << 20);
        // In 3D only where rows end on the boundaries that the store path
        // combines within: streamed partial lines leave the caches before the
        // neighbouring row or tile completes them.  Measured, us per step,
        // streaming / plain: FP32 pair 256^3 303 / 317, nx = 248 250 / 232, 252
        // 288 / 251, 257 346 / 272; FP64 AA 248 694 / 729, 252 772 / 739 (FP64
        // pull with a pole 1025 / 1061, so pull keeps streaming); FP16 ghost row
        // tiles with walls 248 252 / 267, 252 290 / 276, 257 406 / 299.
        const int64_t row = cfg->nx * (cfg->prec == LBEM_F64 ? 8 : (cfg->prec == LBEM_F16 ? 2 : 4));
        const bool whole = h->D == 2 || (is_dev(cfg->prec) ? cfg->nx % 8 == 0 : row % 64 == 0) ||
                           (cfg->prec == LBEM_F64 && h->streaming != LBEM_STREAM_AA);
        h->nts = env_int("LBEM_NT", touched > lim && whole ? 1 : 0) != 0;
    }
    h->impl = make_impl(h->D, h->prec);
    if (h->impl && (hipEventCreateWithFlags(&h->sync_ev, hipEventDisableTiming) != hipSuccess ||
                    hipEventCreateWithFlags(&h->tick_ev, hipEventDisableTiming) != hipSuccess)) {
        if (h->sync_ev) (void)hipEventDestroy(h->sync_ev);
        delete h->impl;
        h->impl = nullptr;
    }
    if (!h->impl) {
        (void)hipFreeAsync(h->partials, h->stream);
        if (h->own_mem) (void)hipFree(h->arena);
        delete h;
        return LBEM_ENOMEM;
    }
    *out = h;
    return LBEM_OK;
}

static void free_source(lbem_s* h)
{
    if (h->src_off) (void)hipFree(h->src_off);
    if (h->src_ent) (void)hipFree(h->src_ent);
    if (h->src_val) (void)hipFree(h->src_val);
    if (h->fsrc_off) (void)hipFree(h->fsrc_off);
    if (h->fsrc_ent) (void)hipFree(h->fsrc_ent);
    if (h->fsrc_val) (void)hipFree(h->fsrc_val);
    h->src_off = nullptr; h->src_ent = nullptr; h->src_val = nullptr;
    if (h->msrc_idx) (void)hipFree(h->msrc_idx);
    if (h->msrc_val) (void)hipFree(h->msrc_val);
    h->msrc_idx = nullptr; h->msrc_val = nullptr;
    h->nmsrc = 0;
    if (h->psrc_flag) (void)hipFree(h->psrc_flag);
    if (h->psrc_idx) (void)hipFree(h->psrc_idx);
    if (h->psrc_val) (void)hipFree(h->psrc_val);
    h->psrc_flag = nullptr; h->psrc_idx = nullptr; h->psrc_val = nullptr;
    if (h->zsrc_off) (void)hipFree(h->zsrc_off);
    if (h->zsrc_ent) (void)hipFree(h->zsrc_ent);
    if (h->zsrc_val) (void)hipFree(h->zsrc_val);
    if (h->xsrc_off) (void)hipFree(h->xsrc_off);
    if (h->xsrc_ent) (void)hipFree(h->xsrc_ent);
    if (h->xsrc_val) (void)hipFree(h->xsrc_val);
    h->xsrc_off = nullptr; h->xsrc_ent = nullptr; h->xsrc_val = nullptr;
    h->nxsrc = 0;
    if (h->rsrc_off) (void)hipFree(h->rsrc_off);
    if (h->rsrc_ent) (void)hipFree(h->rsrc_ent);
    if (h->rsrc_val) (void)hipFree(h->rsrc_val);
    h->fsrc_off = nullptr; h->fsrc_ent = nullptr; h->fsrc_val = nullptr;
    h->zsrc_off = nullptr; h->zsrc_ent = nullptr; h->zsrc_val = nullptr;
    h->rsrc_off = nullptr; h->rsrc_ent = nullptr; h->rsrc_val = nullptr;
    h->nrsrc = 0;
    if (h->bsrc_off) (void)hipFree(h->bsrc_off);
    if (h->bsrc_ent) (void)hipFree(h->bsrc_ent);
    if (h->bsrc_val) (void)hipFree(h->bsrc_val);
    h->bsrc_off = nullptr; h->bsrc_ent = nullptr; h->bsrc_val = nullptr;
    h->nbsrc = 0;
    h->nsrc = 0;
    h->nfsrc = 0;
    h->nzsrc = 0;
}

// Per-block source entries of the fused 3D tiling: every (plane offset,
// frame cell) of the block's z range z0-1 .. z0+lz (periodic images included)
// that carries a current; entry.x = plane offset * frame cells + frame cell.
static int build_fused3_source(lbem_s* h, const std::vector<std::pair<int64_t, double>>& cells, int pp)
{
    const Geo& g = h->fgeo;
    const int TX = h->f3_tx, TY = h->f3_ty, LZ = h->f3_lz;
    const int W = TX + 2, HH = TY + 2, FC = W * HH;
    // per coordinate of an axis the tiles whose frame holds it, and where
    auto frames = [](int n, int step, int count) {
        std::vector<std::vector<std::pair<int, int>>> of(n);
        for (int t = 0; t < count; ++t)
            for (int j = 0; j < step + 2; ++j) of[((t * step - 1 + j) % n + n) % n].push_back({t, j});
        return of;
    };
    const auto fx = frames(g.nx, TX, g.tiles_x), fy = frames(g.ny, TY, g.tiles_y),
               fz = frames(g.nz, LZ, (g.nz + LZ - 1) / LZ);
    struct Item { int b, local; double v; };
    std::vector<Item> items;
    for (auto& e : cells) {
        if (e.second == 0.0) continue;
        const int64_t r = e.first / g.nx;          // row index y + ny z
        for (auto& z : fz[r / g.ny])
            for (auto& y : fy[r % g.ny])
                for (auto& x : fx[e.first % g.nx])
                    items.push_back({(z.first * g.tiles_y + y.first) * g.tiles_x + x.first,
                                     z.second * FC + y.second * W + x.second, e.second});
    }
    std::sort(items.begin(), items.end(),
              [](const Item& a, const Item& b2) { return a.b != b2.b ? a.b < b2.b : a.local < b2.local; });
    std::vector<int> off(g.nblocks + 1, 0);
    for (auto& it : items) off[it.b + 1]++;
    for (int b = 0; b < g.nblocks; ++b) off[b + 1] += off[b];
    std::vector<int2> ent(items.size());
    std::vector<double> val(items.size());
    for (size_t k = 0; k < items.size(); ++k) {
        ent[k] = make_int2(items[k].local, pp);
        val[k] = items[k].v;
    }
    const size_t ms = ent.size(), tv = h->prec == LBEM_F64 ? 8 : 4;
    if (hipMalloc((void**)&h->fsrc_off, off.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)&h->fsrc_ent, std::max<size_t>(ms, 1) * sizeof(int2)) != hipSuccess ||
        hipMalloc((void**)&h->fsrc_val, std::max<size_t>(ms, 1) * tv) != hipSuccess)
        return LBEM_ENOMEM;
    hipError_t e = hipMemcpy(h->fsrc_off, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) e = hipMemcpy(h->fsrc_ent, ent.data(), ms * sizeof(int2), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) {
        if (tv == 8) {
            e = hipMemcpy(h->fsrc_val, val.data(), ms * 8, hipMemcpyHostToDevice);
        } else {
            std::vector<float> f(val.begin(), val.end());
            e = hipMemcpy(h->fsrc_val, f.data(), ms * 4, hipMemcpyHostToDevice);
        }
    }
    if (e != hipSuccess) return LBEM_EDEVICE;
    h->nfsrc = (int64_t)ms;
    return LBEM_OK;
}

// Per-block source entries of the z-marching 3D tiling: local index
// (plane within the chunk) * NT + thread, pair, value.
static int build_zmarch_source(lbem_s* h, const std::vector<std::pair<int64_t, double>>& cells, int pp)
{
    const Geo& g = h->zgeo;
    struct Item { int b, local; float v; };
    std::vector<Item> items;
    items.reserve(cells.size());
    for (auto& e : cells) {
        const int c = (int)e.first;
        const int x = c % g.nx, y = (c / g.nx) % g.ny, z = c / (g.nx * g.ny);
        const int tx = x / TXD, ty = y / TYD, zc = z / h->zlz;
        const int b = (zc * g.tiles_y + ty) * g.tiles_x + tx;
        const int local = (z - zc * h->zlz) * NT + (y - ty * TYD) * TXD + (x - tx * TXD);
        items.push_back({b, local, (float)e.second});
    }
    std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b2) {
        return a.b != b2.b ? a.b < b2.b : a.local < b2.local;
    });
    std::vector<int> off(g.nblocks + 1, 0);
    for (auto& it : items) off[it.b + 1]++;
    for (int b = 0; b < g.nblocks; ++b) off[b + 1] += off[b];
    std::vector<int2> ent(items.size());
    std::vector<float> val(items.size());
    for (size_t k = 0; k < items.size(); ++k) {
        ent[k] = make_int2(items[k].local, pp);
        val[k] = items[k].v;
    }
    const size_t ms = items.size();
    if (hipMalloc((void**)&h->zsrc_off, off.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)&h->zsrc_ent, std::max<size_t>(ms, 1) * sizeof(int2)) != hipSuccess ||
        hipMalloc((void**)&h->zsrc_val, std::max<size_t>(ms, 1) * sizeof(float)) != hipSuccess)
        return LBEM_ENOMEM;
    hipError_t e = hipMemcpy(h->zsrc_off, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) e = hipMemcpy(h->zsrc_ent, ent.data(), ms * sizeof(int2), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) e = hipMemcpy(h->zsrc_val, val.data(), ms * sizeof(float), hipMemcpyHostToDevice);
    if (e != hipSuccess) return LBEM_EDEVICE;
    h->nzsrc = (int64_t)ms;
    return LBEM_OK;
}

// Source entries of a whole-row tiling g: per (block, plane of its chunk) the
// cells (row * nx + x) that carry a current, with S per unit amplitude.
static int build_row_source(const RowGeo& g, const std::vector<std::pair<int64_t, double>>& cells, int pp,
                            int** off_out, int2** ent_out, float** val_out, int64_t* count)
{
    struct Item { int64_t key; int local; float v; };
    std::vector<Item> items;
    items.reserve(cells.size());
    for (auto& e : cells) {
        const int64_t c = e.first;
        const int x = (int)(c % g.nx), y = (int)((c / g.nx) % g.ny), z = (int)(c / ((int64_t)g.nx * g.ny));
        const int tyi = y / g.ty, zc = z / g.lz;
        const int64_t b = (int64_t)zc * g.tiles_y + tyi;
        items.push_back({b * g.lz + (z - zc * g.lz), (y - tyi * g.ty) * g.nx + x, (float)e.second});
    }
    std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b2) { return a.key < b2.key; });
    const size_t nkeys = (size_t)g.nblocks * g.lz;
    std::vector<int> off(nkeys + 1, 0);
    for (auto& it : items) off[it.key + 1]++;
    for (size_t k = 0; k < nkeys; ++k) off[k + 1] += off[k];
    std::vector<int2> ent(items.size());
    std::vector<float> val(items.size());
    for (size_t k = 0; k < items.size(); ++k) {
        ent[k] = make_int2(items[k].local, pp);
        val[k] = items[k].v;
    }
    const size_t ms = items.size();
    if (hipMalloc((void**)off_out, off.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)ent_out, std::max<size_t>(ms, 1) * sizeof(int2)) != hipSuccess ||
        hipMalloc((void**)val_out, std::max<size_t>(ms, 1) * sizeof(float)) != hipSuccess)
        return LBEM_ENOMEM;
    hipError_t e = hipMemcpy(*off_out, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) e = hipMemcpy(*ent_out, ent.data(), ms * sizeof(int2), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) e = hipMemcpy(*val_out, val.data(), ms * sizeof(float), hipMemcpyHostToDevice);
    if (e != hipSuccess) return LBEM_EDEVICE;
    *count = (int64_t)ms;
    return LBEM_OK;
}

// Source entries of the whole-row plain tiling: per block (tiles_y * z + row
// tile) the cells (row * nx + x) that carry a current, with S per unit amplitude.
static int build_xrow_source(lbem_s* h, const std::vector<std::pair<int64_t, double>>& cells, int pp)
{
    const XRowGeo& g = h->xgeo;
    struct Item { int b; int local; double v; };
    std::vector<Item> items;
    items.reserve(cells.size());
    for (auto& e : cells) {
        const int64_t c = e.first;
        const int x = (int)(c % g.nx), y = (int)((c / g.nx) % g.ny), z = (int)(c / ((int64_t)g.nx * g.ny));
        const int yt = y / g.rows;
        items.push_back({z * g.tiles_y + yt, (y - yt * g.rows) * g.nx + x, e.second});
    }
    std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b2) { return a.b < b2.b; });
    std::vector<int> off((size_t)g.nblocks + 1, 0);
    for (auto& it : items) off[it.b + 1]++;
    for (int b = 0; b < g.nblocks; ++b) off[b + 1] += off[b];
    std::vector<int2> ent(items.size());
    for (size_t k = 0; k < items.size(); ++k) ent[k] = make_int2(items[k].local, pp);
    const size_t ms = items.size(), tv = h->prec == LBEM_F64 ? 8 : 4;
    if (hipMalloc((void**)&h->xsrc_off, off.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)&h->xsrc_ent, std::max<size_t>(ms, 1) * sizeof(int2)) != hipSuccess ||
        hipMalloc((void**)&h->xsrc_val, std::max<size_t>(ms, 1) * tv) != hipSuccess)
        return LBEM_ENOMEM;
    hipError_t e = hipMemcpy(h->xsrc_off, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) e = hipMemcpy(h->xsrc_ent, ent.data(), ms * sizeof(int2), hipMemcpyHostToDevice);
    if (e == hipSuccess && ms) {
        if (tv == 8) {
            std::vector<double> v(ms);
            for (size_t k = 0; k < ms; ++k) v[k] = items[k].v;
            e = hipMemcpy(h->xsrc_val, v.data(), ms * 8, hipMemcpyHostToDevice);
        } else {
            std::vector<float> v(ms);
            for (size_t k = 0; k < ms; ++k) v[k] = (float)items[k].v;
            e = hipMemcpy(h->xsrc_val, v.data(), ms * 4, hipMemcpyHostToDevice);
        }
    }
    if (e != hipSuccess) return LBEM_EDEVICE;
    h->nxsrc = (int64_t)ms;
    return LBEM_OK;
}

// Source segments of the pair tiling: for every (tile column, plane, row) that
// holds source cells the values of its 64 columns (periodic images included),
// and per block whether any row it updates does.
static int build_pair_source(lbem_s* h, const std::vector<std::pair<int64_t, double>>& cells, int pp)
{
    const PairGeo& g = h->pgeo;
    const bool f32 = h->prec == LBEM_F32;
    const int tw = g.sx, th = g.sy, halo = f32 ? 1 : 2, len = f32 ? PFSEG : 64;
    const size_t plane = (size_t)g.ny * g.nz;
    std::vector<int> idx((size_t)g.tiles_x * plane, -1);
    std::vector<unsigned char> flag((size_t)g.nblocks, 0);
    // per row and plane the tiles and chunks whose frame (the stored rows and
    // planes and the halo on each side, periodic images included) holds it
    auto frames = [halo](int n, int step, int count) {
        std::vector<std::vector<int>> of(n);
        for (int t = 0; t < count; ++t)
            for (int j = 0; j < std::min(n, step + 2 * halo); ++j) of[(((t * step - halo + j) % n) + n) % n].push_back(t);
        return of;
    };
    const auto tiles = frames(g.ny, th, g.tiles_y), chunks = frames(g.nz, g.lz, (g.nz + g.lz - 1) / g.lz);
    std::vector<float> val, row(g.nx, 0.f);
    int segs = 0;
    for (size_t k = 0; k < cells.size();) {        // cells are sorted: one row at a time
        const int64_t r = cells[k].first / g.nx;   // row index y + ny z
        const int y = (int)(r % g.ny), z = (int)(r / g.ny);
        size_t e = k;
        for (; e < cells.size() && cells[e].first / g.nx == r; ++e) row[cells[e].first % g.nx] = (float)cells[e].second;
        for (int t = 0; t < g.tiles_x; ++t) {
            int gx = (t * tw - halo) % g.nx;
            if (gx < 0) gx += g.nx;
            float seg[PFSEG];
            bool any = false;
            for (int j = 0; j < len; ++j) {
                seg[j] = row[gx];
                any = any || seg[j] != 0.f;
                gx = gx + 1 == g.nx ? 0 : gx + 1;
            }
            if (!any) continue;
            idx[(size_t)t * plane + (size_t)z * g.ny + y] = segs++;
            val.insert(val.end(), seg, seg + len);
            for (int ty : tiles[y])
                for (int zc : chunks[z]) flag[((size_t)zc * g.tiles_y + ty) * g.tiles_x + t] = 1;
        }
        for (; k < e; ++k) row[cells[k].first % g.nx] = 0.f;
    }
    if (!segs) return LBEM_OK;
    if (hipMalloc((void**)&h->psrc_idx, idx.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)&h->psrc_val, val.size() * sizeof(float)) != hipSuccess ||
        hipMalloc((void**)&h->psrc_flag, flag.size()) != hipSuccess)
        return LBEM_ENOMEM;
    if (hipMemcpy(h->psrc_idx, idx.data(), idx.size() * sizeof(int), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(h->psrc_val, val.data(), val.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(h->psrc_flag, flag.data(), flag.size(), hipMemcpyHostToDevice) != hipSuccess)
        return LBEM_EDEVICE;
    h->psrc_pair = pp;
    return LBEM_OK;
}

// Source segments of the 2D strips: for every (strip, row) that holds source
// cells the values of all its columns (periodic images included).
static int build_march_source(lbem_s* h, const std::vector<std::pair<int64_t, double>>& cells)
{
    const MarchGeo& g = h->mgeo;
    const int wid = 64 * h->mcpl, ow = wid - 2 * MARCH_HX;
    std::vector<int> idx((size_t)g.strips * g.ny, -1);
    for (int k = 0; k < 8; ++k) h->msrc_mask[k] = 0;
    std::vector<double> val, row(g.nx, 0.0);
    int segs = 0;
    for (size_t k = 0; k < cells.size();) {        // cells are sorted: one row at a time
        const int y = (int)(cells[k].first / g.nx);
        size_t e = k;
        for (; e < cells.size() && cells[e].first / g.nx == y; ++e) row[cells[e].first % g.nx] = cells[e].second;
        for (int s = 0; s < g.strips; ++s) {
            bool any = false;
            int gx = (s * ow - MARCH_HX) % g.nx;
            if (gx < 0) gx += g.nx;
            const int gx0 = gx;
            for (int j = 0; j < wid && !any; ++j) {
                any = row[gx] != 0.0;
                gx = gx + 1 == g.nx ? 0 : gx + 1;
            }
            if (!any) continue;
            idx[(size_t)s * g.ny + y] = segs++;
            h->msrc_mask[(s >> 5) & 7] |= 1u << (s & 31);
            gx = gx0;
            for (int j = 0; j < wid; ++j) {
                val.push_back(row[gx]);
                gx = gx + 1 == g.nx ? 0 : gx + 1;
            }
        }
        for (; k < e; ++k) row[cells[k].first % g.nx] = 0.0;
    }
    if (!segs) return LBEM_OK;
    const size_t tv = h->prec == LBEM_F64 ? 8 : 4;
    if (hipMalloc((void**)&h->msrc_idx, idx.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)&h->msrc_val, val.size() * tv) != hipSuccess)
        return LBEM_ENOMEM;
    hipError_t e = hipMemcpy(h->msrc_idx, idx.data(), idx.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        if (tv == 8) {
            e = hipMemcpy(h->msrc_val, val.data(), val.size() * 8, hipMemcpyHostToDevice);
        } else {
            std::vector<float> f(val.begin(), val.end());
            e = hipMemcpy(h->msrc_val, f.data(), f.size() * 4, hipMemcpyHostToDevice);
        }
    }
    if (e != hipSuccess) return LBEM_EDEVICE;
    h->nmsrc = segs;
    return LBEM_OK;
}

int lbem_destroy(lbem_t h)
{
    if (!h) return LBEM_OK;
    API_SHARED;
    (void)follow_ticks(h);
    (void)hipStreamSynchronize(h->stream);
    free_source(h);
    if (h->keep) (void)hipFree(h->keep);
    if (h->ade) (void)hipFree(h->ade);
    if (h->pol) (void)hipFree(h->pol);
    if (h->pol2) (void)hipFree(h->pol2);
    if (h->ra) (void)hipFree(h->ra);
    // stream-ordered: returns the memory without waiting for the whole device
    if (h->partials) (void)hipFreeAsync(h->partials, h->stream);
    if (h->own_mem && h->arena) (void)hipFree(h->arena);
    if (h->sync_ev) (void)hipEventDestroy(h->sync_ev);
    if (h->tick_ev) (void)hipEventDestroy(h->tick_ev);
    delete h->impl;
    delete h;
    return LBEM_OK;
}

int lbem_set_medium(lbem_t h, const double* eps_r, const double* mu_r)
{
    if (!h || !eps_r) return LBEM_EINVAL;
    const int64_t n = h->n;
    bool nonunit_mu = false;
    if (mu_r)
        for (int64_t c = 0; c < n; ++c)
            if (mu_r[c] != 1.0) { nonunit_mu = true; break; }
    if (nonunit_mu && !h->cfg.mu_varies) return LBEM_EINVAL;
    API_SHARED;
    HIP_OK(follow_ticks(h));
    Staging s_eps, s_mu, s_flag;      // see stage_alloc
    int flag = 0, rc = LBEM_OK;
    if (!stage_alloc(s_eps, n * 8, h->stream) || (mu_r && !stage_alloc(s_mu, n * 8, h->stream)) ||
        !stage_alloc(s_flag, sizeof(int), h->stream)) {
        stage_free(s_eps, h->stream);
        stage_free(s_mu, h->stream);
        stage_free(s_flag, h->stream);
        return LBEM_ENOMEM;
    }
    double* deps = (double*)s_eps.p;
    double* dmu = (double*)s_mu.p;
    int* dflag = (int*)s_flag.p;
    hipError_t e = hipMemcpyAsync(deps, eps_r, n * 8, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess && mu_r) e = hipMemcpyAsync(dmu, mu_r, n * 8, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipMemsetAsync(dflag, 0, sizeof(int), h->stream);
    h->mu_set = h->cfg.mu_varies != 0;
    h->ra_set = false;                 // a new medium is isotropic until lbem_set_anisotropy
    if (e == hipSuccess) e = h->impl->medium(h, deps, dmu, dflag);
    if (e == hipSuccess) e = hipMemcpyAsync(&flag, dflag, sizeof(int), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) rc = LBEM_EDEVICE;
    else if (flag) rc = LBEM_EUNSTABLE;
    stage_free(s_eps, h->stream);
    stage_free(s_mu, h->stream);
    stage_free(s_flag, h->stream);
    h->have_medium = rc == LBEM_OK;
    h->have_fields = false;
    return rc;
}

int lbem_init_fields(lbem_t h, const double* E, const double* B)
{
    if (!h || !E || !B) return LBEM_EINVAL;
    if (!h->have_medium) return LBEM_ESTATE;
    const int64_t n = h->n;
    for (int64_t k = 0; k < 3 * n; ++k)
        if (!std::isfinite(E[k]) || !std::isfinite(B[k])) return LBEM_EINVAL;
    if (h->D == 2) {
        for (int64_t c = 0; c < n; ++c)
            if (E[c] != 0.0 || E[n + c] != 0.0 || B[2 * n + c] != 0.0) return LBEM_EINVAL;
    }
    API_SHARED;
    HIP_OK(follow_ticks(h));
    Staging s_E, s_B;                 // see stage_alloc
    if (!stage_alloc(s_E, 3 * n * 8, h->stream) || !stage_alloc(s_B, 3 * n * 8, h->stream)) {
        stage_free(s_E, h->stream);
        stage_free(s_B, h->stream);
        return LBEM_ENOMEM;
    }
    double* dE = (double*)s_E.p;
    double* dB = (double*)s_B.p;
    hipError_t e = hipMemcpyAsync(dE, E, 3 * n * 8, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(dB, B, 3 * n * 8, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = h->impl->init(h, dE, dB);
    if (e == hipSuccess && h->pol) e = hipMemsetAsync(h->pol, 0, pol_bytes(h), h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    stage_free(s_E, h->stream);
    stage_free(s_B, h->stream);
    if (e != hipSuccess) return LBEM_EDEVICE;
    h->t = 0;
    h->have_fields = true;
    return LBEM_OK;
}

int lbem_set_boundary(lbem_t h, int axis, int kind)
{
    if (!h || axis < 0 || axis >= h->D || kind < LBEM_BC_PERIODIC || kind > LBEM_BC_PMC) return LBEM_EINVAL;
    if (kind != LBEM_BC_PERIODIC && h->streaming != LBEM_STREAM_PULL) return LBEM_EINVAL;
    if (h->have_medium) return LBEM_ESTATE;
    h->bc_kind[axis] = kind;
    return LBEM_OK;
}

int lbem_set_anisotropy(lbem_t h, const double* fac)
{
    if (!h || !fac) return LBEM_EINVAL;
    if (h->prec > LBEM_F32 || h->streaming != LBEM_STREAM_PULL) return LBEM_EINVAL;
    if (!h->have_medium) return LBEM_ESTATE;
    API_SHARED;
    HIP_OK(follow_ticks(h));
    const int64_t n = h->n;
    const size_t tm = h->prec == LBEM_F64 ? 8 : 4;
    if (hipStreamSynchronize(h->stream) != hipSuccess) return LBEM_EDEVICE;
    if (!h->ra && hipMalloc(&h->ra, (size_t)h->D * n * tm) != hipSuccess) {
        h->ra = nullptr;
        return LBEM_ENOMEM;
    }
    double* dfac = nullptr;
    int* dflag = nullptr;
    if (hipMalloc((void**)&dfac, (size_t)h->D * n * 8) != hipSuccess) return LBEM_ENOMEM;
    if (hipMalloc((void**)&dflag, sizeof(int)) != hipSuccess) { (void)hipFree(dfac); return LBEM_ENOMEM; }
    int flag = 0, rc = LBEM_OK;
    hipError_t e = hipMemcpyAsync(dfac, fac, (size_t)h->D * n * 8, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipMemsetAsync(dflag, 0, sizeof(int), h->stream);
    if (e == hipSuccess) e = tm == 8 ? launch_aniso<double>(h, dfac, dflag, 0) : launch_aniso<float>(h, dfac, dflag, 0);
    if (e == hipSuccess) e = hipMemcpyAsync(&flag, dflag, sizeof(int), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e == hipSuccess && !flag) {
        e = tm == 8 ? launch_aniso<double>(h, dfac, dflag, 1) : launch_aniso<float>(h, dfac, dflag, 1);
        if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    }
    if (e != hipSuccess) rc = LBEM_EDEVICE;
    else if (flag) rc = LBEM_EUNSTABLE;
    (void)hipFree(dfac);
    (void)hipFree(dflag);
    if (rc == LBEM_OK) {
        h->ra_set = true;
        h->have_fields = false;        // the populations must be re-initialised for the new weights
    }
    return rc;
}

int lbem_set_dispersion(lbem_t h, const double* wp2, const double* w02, const double* gamma)
{
    if (!h) return LBEM_EINVAL;
    API_SHARED;
    HIP_OK(follow_ticks(h));
    if (hipStreamSynchronize(h->stream) != hipSuccess) return LBEM_EDEVICE;
    if (!wp2) {
        if (h->ade) (void)hipFree(h->ade);
        if (h->pol) (void)hipFree(h->pol);
        if (h->pol2) (void)hipFree(h->pol2);
        h->ade = h->pol = h->pol2 = nullptr;
        return LBEM_OK;
    }
    if (h->streaming != LBEM_STREAM_PULL) return LBEM_EINVAL;
    const int64_t n = h->n;
    for (int64_t c = 0; c < n; ++c) {
        const double a = wp2[c], b = w02 ? w02[c] : 0.0, g = gamma ? gamma[c] : 0.0;
        if (!(a >= 0.0) || !(b >= 0.0) || !(g >= 0.0) || !std::isfinite(a) || !std::isfinite(b) ||
            !std::isfinite(g))
            return LBEM_EINVAL;
    }
    const bool f64 = h->prec == LBEM_F64;
    const size_t tm = f64 ? 8 : 4;
    std::vector<char> host((size_t)3 * n * tm);
    for (int64_t c = 0; c < n; ++c) {
        const double g = gamma ? gamma[c] : 0.0, den = 1.0 + 0.5 * g;
        const double co[3] = {(1.0 - 0.5 * g) / den, wp2[c] / den, (w02 ? w02[c] : 0.0) / den};
        for (int k = 0; k < 3; ++k) {
            if (f64) ((double*)host.data())[k * n + c] = co[k];
            else ((float*)host.data())[k * n + c] = (float)co[k];
        }
    }
    const size_t pb = (size_t)2 * h->P * n * tm;
    if (!h->ade) {
        if (hipMalloc(&h->ade, (size_t)3 * n * tm) != hipSuccess) { h->ade = nullptr; return LBEM_ENOMEM; }
        if (hipMalloc(&h->pol, pb) != hipSuccess) {
            (void)hipFree(h->ade);
            h->ade = h->pol = nullptr;
            return LBEM_ENOMEM;
        }
        // launches of several steps (in 3D: not with walls) need a second copy;
        // without it the steps stay single
        if (h->ext_ns > 1 && (h->D == 2 || !ext_of(h).walls()) && hipMalloc(&h->pol2, pb) != hipSuccess) {
            h->pol2 = nullptr;
            (void)hipGetLastError();
        }
    }
    if (hipMemcpyAsync(h->ade, host.data(), (size_t)3 * n * tm, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipMemsetAsync(h->pol, 0, pb, h->stream) != hipSuccess || hipStreamSynchronize(h->stream) != hipSuccess)
        return LBEM_EDEVICE;
    return LBEM_OK;
}

int lbem_set_absorber(lbem_t h, const double* sigma)
{
    if (!h) return LBEM_EINVAL;
    API_SHARED;
    HIP_OK(follow_ticks(h));
    if (hipStreamSynchronize(h->stream) != hipSuccess) return LBEM_EDEVICE;
    if (!sigma) {
        if (h->keep) (void)hipFree(h->keep);
        h->keep = nullptr;
        return LBEM_OK;
    }
    if (h->streaming != LBEM_STREAM_PULL) return LBEM_EINVAL;
    const int64_t n = h->n;
    for (int64_t c = 0; c < n; ++c)
        if (!(sigma[c] >= 0.0 && sigma[c] < 1.0)) return LBEM_EINVAL;
    const bool f64 = h->prec == LBEM_F64;
    const size_t tm = f64 ? 8 : 4;
    std::vector<char> host((size_t)n * tm);
    for (int64_t c = 0; c < n; ++c) {
        const double k = 1.0 - sigma[c];
        if (f64) ((double*)host.data())[c] = k;
        else ((float*)host.data())[c] = (float)k;
    }
    if (!h->keep && hipMalloc(&h->keep, (size_t)n * tm) != hipSuccess) {
        h->keep = nullptr;
        return LBEM_ENOMEM;
    }
    if (hipMemcpyAsync(h->keep, host.data(), (size_t)n * tm, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipStreamSynchronize(h->stream) != hipSuccess)
        return LBEM_EDEVICE;
    return LBEM_OK;
}

int lbem_set_source(lbem_t h, int comp, const int64_t* cells, const double* weight, int64_t m)
{
    if (!h || m < 0 || comp < 0 || comp > 2) return LBEM_EINVAL;
    if (h->D == 2 && comp != 2) return LBEM_EINVAL;
    if (m > 0 && (!cells || !weight)) return LBEM_EINVAL;
    if (!h->have_medium) return LBEM_ESTATE;
    API_SHARED;
    HIP_OK(follow_ticks(h));
    if (hipStreamSynchronize(h->stream) != hipSuccess) return LBEM_EDEVICE;
    free_source(h);
    if (m == 0) return LBEM_OK;
    const int64_t n = h->n;
    const int D = h->D;
    // pair carrying component comp and its Levi-Civita sign
    int pp = -1, sg = 0;
    for (int p = 0; p < h->P; ++p)
        if (pair_g(D, p) == comp) { pp = p; sg = pair_s(D, p); }
    // eps_abs = eps_r/c_vac^2 = (D-1)/(mu_r c_L^2): read back c_L^2 and mu_r
    std::vector<double> cl2(n), mu(n, 1.0);
    if (h->prec == LBEM_F64) {
        if (hipMemcpy(cl2.data(), h->cl2, n * 8, hipMemcpyDeviceToHost) != hipSuccess) return LBEM_EDEVICE;
    } else {
        std::vector<float> f(n);
        if (hipMemcpy(f.data(), h->cl2, n * 4, hipMemcpyDeviceToHost) != hipSuccess) return LBEM_EDEVICE;
        for (int64_t c = 0; c < n; ++c) cl2[c] = f[c];
    }
    if (h->mu_set && hipMemcpy(mu.data(), h->mu_r, n * 8, hipMemcpyDeviceToHost) != hipSuccess)
        return LBEM_EDEVICE;
    // merge repeated cells, then bucket by tile
    std::vector<std::pair<int64_t, double>> ent;
    ent.reserve(m);
    for (int64_t k = 0; k < m; ++k) {
        if (cells[k] < 0 || cells[k] >= n || !std::isfinite(weight[k])) return LBEM_EINVAL;
        ent.push_back({cells[k], weight[k]});
    }
    std::sort(ent.begin(), ent.end(), [](auto& a, auto& b) { return a.first < b.first; });
    std::vector<std::pair<int64_t, double>> merged;
    for (auto& e : ent) {
        if (!merged.empty() && merged.back().first == e.first) merged.back().second += e.second;
        else merged.push_back(e);
    }
    const Geo& g = h->geo;
    const int bx = 1 << g.bx_shift, rb = NT / bx;
    struct Item { int b; int local; double v; };
    std::vector<Item> items;
    std::vector<double> src_value;
    items.reserve(merged.size());
    src_value.reserve(merged.size());
    for (auto& e : merged) {
        const int c = (int)e.first;
        const int x = c % g.nx, y = (c / g.nx) % g.ny, z = c / (g.nx * g.ny);
        const int tx = x / bx, ty = y / (rb * h->vec);
        const int b = tile_id(g, tx, ty, z);
        const int yr = y - ty * rb * h->vec;
        const int v = yr / rb, tyi = yr % rb;
        const int local = v * NT + tyi * bx + (x - tx * bx);
        // S per unit amplitude on pair pp: sgn * (-weight/eps_abs)
        const double eps_abs = (double)(D - 1) / (mu[c] * cl2[c]);
        items.push_back({b, local, -(double)sg * e.second / eps_abs});
        src_value.push_back(items.back().v);
    }
    std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b) { return a.b < b.b; });
    std::vector<int> off(g.nblocks + 1, 0);
    for (auto& it : items) off[it.b + 1]++;
    for (int b = 0; b < g.nblocks; ++b) off[b + 1] += off[b];
    std::vector<int2> ents(items.size());
    for (size_t k = 0; k < items.size(); ++k) ents[k] = make_int2(items[k].local, pp);
    const size_t ms = items.size();
    const size_t tv = h->prec == LBEM_F64 ? 8 : 4;
    if (hipMalloc((void**)&h->src_off, off.size() * sizeof(int)) != hipSuccess ||
        hipMalloc((void**)&h->src_ent, ms * sizeof(int2)) != hipSuccess ||
        hipMalloc((void**)&h->src_val, ms * tv) != hipSuccess) {
        free_source(h);
        return LBEM_ENOMEM;
    }
    hipError_t e = hipMemcpy(h->src_off, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(h->src_ent, ents.data(), ms * sizeof(int2), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        if (tv == 8) {
            std::vector<double> v(ms);
            for (size_t k = 0; k < ms; ++k) v[k] = items[k].v;
            e = hipMemcpy(h->src_val, v.data(), ms * 8, hipMemcpyHostToDevice);
        } else {
            std::vector<float> v(ms);
            for (size_t k = 0; k < ms; ++k) v[k] = (float)items[k].v;
            e = hipMemcpy(h->src_val, v.data(), ms * 4, hipMemcpyHostToDevice);
        }
    }
    if (e != hipSuccess) { free_source(h); return LBEM_EDEVICE; }
    h->nsrc = (int64_t)ms;
    if (h->zmarch || h->brow) {
        std::vector<std::pair<int64_t, double>> cv(merged.size());
        for (size_t k = 0; k < merged.size(); ++k) cv[k] = {merged[k].first, src_value[k]};
        int rc = h->zmarch ? build_zmarch_source(h, cv, pp) : LBEM_OK;
        if (rc == LBEM_OK && h->zmarch && h->rowk)
            rc = build_row_source(h->rgeo, cv, pp, &h->rsrc_off, &h->rsrc_ent, &h->rsrc_val, &h->nrsrc);
        if (rc == LBEM_OK && h->brow)
            rc = build_row_source(h->bgeo, cv, pp, &h->bsrc_off, &h->bsrc_ent, &h->bsrc_val, &h->nbsrc);
        if (rc != LBEM_OK) { free_source(h); return rc; }
    }
    if (h->xrow) {
        std::vector<std::pair<int64_t, double>> cv(merged.size());
        for (size_t k = 0; k < merged.size(); ++k) cv[k] = {merged[k].first, src_value[k]};
        const int rc = build_xrow_source(h, cv, pp);
        if (rc != LBEM_OK) { free_source(h); return rc; }
    }
    const bool pair32 = D == 3 && h->prec == LBEM_F32;
    if (pair32 && (h->ext_ns > 1 || h->pair_f32)) {
        std::vector<std::pair<int64_t, double>> cv(merged.size());
        for (size_t k = 0; k < merged.size(); ++k) cv[k] = {merged[k].first, src_value[k]};
        const int rc = build_pair_source(h, cv, pp);
        if (rc != LBEM_OK) { free_source(h); return rc; }
    }
    if (fused_format(h) && h->fuse_ns > 1 && !(pair32 && h->pair_f32)) {
        std::vector<std::pair<int64_t, double>> cv(merged.size());
        for (size_t k = 0; k < merged.size(); ++k) cv[k] = {merged[k].first, src_value[k]};
        const int rc = D == 2 ? build_march_source(h, cv)
                              : (is_dev(h->prec) ? build_pair_source(h, cv, pp) : build_fused3_source(h, cv, pp));
        if (rc != LBEM_OK) { free_source(h); return rc; }
    }
    return LBEM_OK;
}

int lbem_step(lbem_t h, int64_t nsteps, const double* amp)
{
    if (!h || nsteps < 0) return LBEM_EINVAL;
    if (!h->have_fields) return LBEM_ESTATE;
    HIP_OK(follow_ticks(h));
    const int nf = fused_steps(h);
    const bool ext2 = h->D == 2 && has_bx(h);    // launches of four and two steps only
    // A graph holds the copies that its launches read and write.  So a captured
    // call, and every later call on the handle (it may stand between two replays),
    // leaves the state in the copy that single steps would leave it in: launches of
    // several steps by twos, the rest singly.  The two P/J buffers of a pole, which
    // only launches of several steps swap, come back as well.
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &st) != hipSuccess) (void)hipGetLastError();
    const bool captured = st != hipStreamCaptureStatusNone;
    h->graphed = h->graphed || captured;
    // A captured odd number of steps of a plain format without extras, which has no
    // such buffers, can be replayed too: an even number of launches, of even lengths.
    const bool even = captured && nf > 1 && nsteps % 2 && h->prec <= LBEM_F32 && !has_bx(h) &&
                       (h->D == 2 || (double)h->n >= FUSE3D_MIN);
    int64_t k = 0, twos = 0, each = 1, left = 0;
    while (k < nsteps) {
        // 2D launches take any number of steps from two to nf (no three with extras)
        int64_t ns = std::min<int64_t>(nf, nsteps - k);
        if (ext2 && ns == 3) ns = 2;
        if (even && h->layout == LAYOUT_PULL_PENDING) {
            const int64_t to_go = nsteps - k;
            if (left == 0) left = std::min<int64_t>(to_go, ((to_go + nf - 1) / nf + 1) / 2 * 2);
            ns = (to_go + left - 1) / left;
            --left;
        } else if (h->graphed) {
            if (twos == 0 && h->layout == LAYOUT_PULL_PENDING) {
                each = std::min<int64_t>(nf, (nsteps - k) / 2);
                if (ext2 && each == 3) each = 2;
                if (each > 1 && (h->D == 2 || each == nf)) twos = 2;
            }
            ns = twos > 0 ? each : 1;
            if (twos > 0) --twos;
        }
        if (ns > 1 && h->layout == LAYOUT_PULL_PENDING && (h->D == 2 || ns == nf)) {
            if (h->impl->step_fused(h, (amp && h->nsrc) ? amp + k : nullptr, (int)ns) != hipSuccess)
                return LBEM_EDEVICE;
            k += ns;
            h->t += ns;
            continue;
        }
        const double a = (amp && h->nsrc) ? amp[k] : 0.0;
        if (h->impl->step(h, a) != hipSuccess) return LBEM_EDEVICE;
        h->t += 1;
        ++k;
    }
    return LBEM_OK;
}

int lbem_moments(lbem_t h, double* E, double* B, int on_device)
{
    if (!h) return LBEM_EINVAL;
    if (!h->have_fields) return LBEM_ESTATE;
    HIP_OK(follow_ticks(h));
    const size_t bytes = (size_t)3 * h->n * 8;
    if (on_device) {
        if (h->impl->fields(h, E, B, nullptr) != hipSuccess) return LBEM_EDEVICE;
        return hipStreamSynchronize(h->stream) == hipSuccess ? LBEM_OK : LBEM_EDEVICE;
    }
    if (E) {
        HIP_OK(h->impl->fields(h, h->scratch, nullptr, nullptr));
        HIP_OK(hipMemcpyAsync(E, h->scratch, bytes, hipMemcpyDeviceToHost, h->stream));
        HIP_OK(hipStreamSynchronize(h->stream));
    }
    if (B) {
        HIP_OK(h->impl->fields(h, nullptr, h->scratch, nullptr));
        HIP_OK(hipMemcpyAsync(B, h->scratch, bytes, hipMemcpyDeviceToHost, h->stream));
        HIP_OK(hipStreamSynchronize(h->stream));
    }
    return LBEM_OK;
}

int lbem_energy(lbem_t h, double out[4])
{
    if (!h || !out) return LBEM_EINVAL;
    if (!h->have_fields) return LBEM_ESTATE;
    HIP_OK(follow_ticks(h));
    double* res = h->partials + (size_t)h->nb_diag * 4;
    HIP_OK(h->impl->fields(h, nullptr, h->scratch, h->partials));
    Geo1 g = geo1(h);
    if (h->D == 2)
        hipLaunchKernelGGL((k_divb<2>), dim3(h->nb_diag), dim3(NT), 0, h->stream, h->scratch, g, h->partials);
    else
        hipLaunchKernelGGL((k_divb<3>), dim3(h->nb_diag), dim3(NT), 0, h->stream, h->scratch, g, h->partials);
    HIP_OK(hipGetLastError());
    hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(NT), 0, h->stream, h->partials, h->nb_diag, res);
    HIP_OK(hipGetLastError());
    HIP_OK(hipMemcpyAsync(out, res, 4 * sizeof(double), hipMemcpyDeviceToHost, h->stream));
    HIP_OK(hipStreamSynchronize(h->stream));
    for (int k = 0; k < 4; ++k)
        if (!std::isfinite(out[k])) return LBEM_ENONFINITE;
    return LBEM_OK;
}

// lbem_energy with its scratch in the static device array: no allocation.
int lbem_energy_noalloc(lbem_t h, double out[4])
{
    if (!h || !out) return LBEM_EINVAL;
    if (!h->have_fields) return LBEM_ESTATE;
    if (h->n > LBEM_NOALLOC_MAX_CELLS) return LBEM_ETOOBIG;
    double* base = nullptr;
    HIP_OK(noalloc_address(h->device, &base));
    HIP_OK(follow_ticks(h));
    double* bfield = base;                          // [3][n]
    double* partials = base + (size_t)3 * h->n;     // [nb_diag][4], then the 4 results
    double* res = partials + (size_t)h->nb_diag * 4;
    HIP_OK(h->impl->fields(h, nullptr, bfield, partials));
    Geo1 g = geo1(h);
    if (h->D == 2)
        hipLaunchKernelGGL((k_divb<2>), dim3(h->nb_diag), dim3(NT), 0, h->stream, bfield, g, partials);
    else
        hipLaunchKernelGGL((k_divb<3>), dim3(h->nb_diag), dim3(NT), 0, h->stream, bfield, g, partials);
    HIP_OK(hipGetLastError());
    hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(NT), 0, h->stream, partials, h->nb_diag, res);
    HIP_OK(hipGetLastError());
    HIP_OK(hipMemcpyAsync(out, res, 4 * sizeof(double), hipMemcpyDeviceToHost, h->stream));
    HIP_OK(hipStreamSynchronize(h->stream));
    for (int k = 0; k < 4; ++k)
        if (!std::isfinite(out[k])) return LBEM_ENONFINITE;
    return LBEM_OK;
}

int64_t lbem_time(lbem_t h) { return h ? h->t : -1; }

int lbem_steps_per_launch(lbem_t h)
{
    if (!h) return LBEM_EINVAL;
    return fused_steps(h);
}

namespace {
constexpr size_t STATE_HDR = 128;
struct StateHeader {
    char magic[8];
    int32_t dim, prec, streaming, layout;
    int64_t nx, ny, nz, t;
    uint64_t payload;
    uint64_t aux;      // auxiliary dispersion fields after the populations (0 if none)
};
static_assert(sizeof(StateHeader) <= STATE_HDR, "state header");
const char STATE_MAGIC[8] = {'L', 'B', 'E', 'M', 'S', 'T', '0', '1'};
}  // namespace

size_t lbem_state_bytes(lbem_t h)
{
    if (!h) return 0;
    return STATE_HDR + sizes_of(&h->cfg).pop_one + pol_bytes(h);
}

int lbem_get_state(lbem_t h, void* buf, size_t bytes, int on_device)
{
    if (!h || !buf || bytes < lbem_state_bytes(h)) return LBEM_EINVAL;
    if (!h->have_fields) return LBEM_ESTATE;
    HIP_OK(follow_ticks(h));
    char hdr[STATE_HDR] = {0};
    StateHeader sh{};
    std::memcpy(sh.magic, STATE_MAGIC, 8);
    sh.dim = h->D;
    sh.prec = h->prec;
    sh.streaming = h->streaming;
    sh.layout = h->layout;
    sh.nx = h->cfg.nx;
    sh.ny = h->cfg.ny;
    sh.nz = h->cfg.nz;
    sh.t = h->t;
    sh.payload = sizes_of(&h->cfg).pop_one;
    sh.aux = pol_bytes(h);
    std::memcpy(hdr, &sh, sizeof(sh));
    char* out = (char*)buf;
    const hipMemcpyKind k = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    if (on_device) {
        HIP_OK(hipMemcpyAsync(out, hdr, STATE_HDR, hipMemcpyHostToDevice, h->stream));
        HIP_OK(hipStreamSynchronize(h->stream));  // hdr is on this stack frame
    } else {
        std::memcpy(out, hdr, STATE_HDR);
    }
    HIP_OK(hipMemcpyAsync(out + STATE_HDR, h->pop[h->cur], sh.payload, k, h->stream));
    if (sh.aux) HIP_OK(hipMemcpyAsync(out + STATE_HDR + sh.payload, h->pol, sh.aux, k, h->stream));
    HIP_OK(hipStreamSynchronize(h->stream));
    return LBEM_OK;
}

int lbem_set_state(lbem_t h, const void* buf, size_t bytes, int on_device)
{
    if (!h || !buf || bytes < lbem_state_bytes(h)) return LBEM_EINVAL;
    if (!h->have_medium) return LBEM_ESTATE;
    HIP_OK(follow_ticks(h));
    const char* in = (const char*)buf;
    StateHeader sh{};
    if (on_device) {
        HIP_OK(hipMemcpyAsync(&sh, in, sizeof(sh), hipMemcpyDeviceToHost, h->stream));
        HIP_OK(hipStreamSynchronize(h->stream));
    } else {
        std::memcpy(&sh, in, sizeof(sh));
    }
    const size_t pay = sizes_of(&h->cfg).pop_one;
    if (std::memcmp(sh.magic, STATE_MAGIC, 8) != 0 || sh.dim != h->D || sh.prec != h->prec ||
        sh.streaming != h->streaming || sh.nx != h->cfg.nx || sh.ny != h->cfg.ny || sh.nz != h->cfg.nz ||
        sh.payload != pay || sh.aux != pol_bytes(h) || sh.t < 0 || sh.layout < LAYOUT_NATURAL ||
        sh.layout > LAYOUT_AA_SWAPPED)
        return LBEM_EINVAL;
    // pull steps never leave the AA layout, AA steps never the pull one
    if ((h->streaming == LBEM_STREAM_PULL && sh.layout == LAYOUT_AA_SWAPPED) ||
        (h->streaming == LBEM_STREAM_AA && sh.layout == LAYOUT_PULL_PENDING))
        return LBEM_EINVAL;
    const hipMemcpyKind k = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    HIP_OK(hipMemcpyAsync(h->pop[0], in + STATE_HDR, pay, k, h->stream));
    if (sh.aux) HIP_OK(hipMemcpyAsync(h->pol, in + STATE_HDR + pay, sh.aux, k, h->stream));
    HIP_OK(hipStreamSynchronize(h->stream));
    h->cur = 0;
    h->layout = sh.layout;
    h->t = sh.t;
    h->have_fields = true;
    return LBEM_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// batched stepping of many resident lattices (serving)
// ---------------------------------------------------------------------------
namespace {
constexpr int NPREC = 7;   // LBEM_F64 .. LBEM_F16
constexpr int NCLASS = 2 * NPREC;  // (dim - 2) * NPREC + prec
constexpr int BATCH_BLOCKS = 8192;  // persistent grid (more blocks than fit: the rest start as others finish)
// How a class's steps after the first of a tick run: the per-cell kernel, or
// (3D deviation classes whose members all have the whole-row tiling) the
// row-tile kernel with mu == 1 or with varying mu
constexpr int NMODE = 3;
enum { MODE_CELL = 0, MODE_ROWS = 1, MODE_ROWS_MU = 2 };

int class_of(const lbem_s* h) { return (h->D - 2) * NPREC + h->prec; }

size_t class_bytes(int max_grids) { return align256(sizeof(BatchHdr)) + align256(sizeof(BatchGrid) * (size_t)max_grids); }
}  // namespace

constexpr int NRING = 8;      // pinned staging slots of the table uploads

struct lbem_batch_s {
    hipStream_t stream;
    int max_grids, ksteps;
    char* dev;                 // NCLASS x (header, table), then the amplitudes [max_grids][ksteps] (8 B each)
    size_t amp_off;            // offset of the amplitudes
    char* pinned[NRING];
    hipEvent_t ev[NRING];      // each slot is free again once its upload has executed
    int ring;
    size_t group_bytes;        // members of one call run in groups touching at most this much state per step
    // per class and mode one graph of ksteps launches, captured and
    // instantiated once, in lbem_batch_create (the row modes of the 3D
    // deviation classes only)
    hipGraph_t graph[NCLASS][NMODE];
    hipGraphExec_t exec[NCLASS][NMODE];
    int use_graph;
    int blocks;                // persistent grid of each class launch
    int rows_min;              // fewest whole-row work items for the row modes
    int multi;                 // several steps per launch for the 16-bit classes: 0 never, 1 by size, 2 always
    // the classes of a tick run concurrently, one stream each (default
    // priority), forked from the batch stream after the table upload and
    // joined back before anything later on it
    hipStream_t cstream[NCLASS];
    hipEvent_t fork_ev, join_ev[NCLASS];
    int concurrent;
};

// the first step of a tick always takes the per-cell kernel: it reads
// members that start from the natural layout
template <int D, typename H, bool GH>
static void launch_batch_dev(dim3 g, dim3 t, hipStream_t st, const BatchHdr* hdr, const BatchGrid* tab, int k,
                             int mode, int multi)
{
    if constexpr (D == 3) {
        if (k > 0 && mode == MODE_ROWS) {
            hipLaunchKernelGGL((k_step_batch_dev3_rows<H, GH, false>), g, dim3(BROW_NT), 0, st, hdr, tab, k);
            return;
        }
        if (k > 0 && mode == MODE_ROWS_MU) {
            hipLaunchKernelGGL((k_step_batch_dev3_rows<H, GH, true>), g, dim3(BROW_NT), 0, st, hdr, tab, k);
            return;
        }
    }
    hipLaunchKernelGGL((k_step_batch_dev<D, H, GH>), g, t, 0, st, hdr, tab, k, multi);
}

template <int D>
static void launch_class_d(lbem_batch_s* b, int prec, const BatchHdr* hdr, const BatchGrid* tab, int k,
                           hipStream_t st, int mode, int multi)
{
    dim3 g(b->blocks), t(NT);
    switch (prec) {
        case LBEM_F64: hipLaunchKernelGGL((k_step_batch_plain<D, double>), g, t, 0, st, hdr, tab, k); break;
        case LBEM_F32: hipLaunchKernelGGL((k_step_batch_plain<D, float>), g, t, 0, st, hdr, tab, k); break;
        case LBEM_F16DEV: launch_batch_dev<D, __half, false>(g, t, st, hdr, tab, k, mode, multi); break;
        case LBEM_BF16DEV: launch_batch_dev<D, __hip_bfloat16, false>(g, t, st, hdr, tab, k, mode, multi); break;
        case LBEM_F16GHOST: launch_batch_dev<D, __half, true>(g, t, st, hdr, tab, k, mode, multi); break;
        case LBEM_BF16GHOST: launch_batch_dev<D, __hip_bfloat16, true>(g, t, st, hdr, tab, k, mode, multi); break;
        default:
            hipLaunchKernelGGL((k_step_batch_plain<D, float, __half>), g, t, 0, st, hdr, tab, k);
            break;
    }
}

// launch k of a class; multi = m > 0: single step k after launches of m steps
static void launch_class(lbem_batch_s* b, int c, int k, hipStream_t st, int mode, int multi = 0)
{
    const size_t cb = class_bytes(b->max_grids);
    const BatchHdr* hdr = (const BatchHdr*)(b->dev + c * cb);
    const BatchGrid* tab = (const BatchGrid*)(b->dev + c * cb + align256(sizeof(BatchHdr)));
    if (c < NPREC) launch_class_d<2>(b, c, hdr, tab, k, st, mode, multi);
    else launch_class_d<3>(b, c - NPREC, hdr, tab, k, st, mode, multi);
}

// classes that have the row modes: 3D deviation formats
static bool has_row_modes(int c) { return c >= NPREC && is_dev(c - NPREC); }

// A class's tick with several steps per launch (16-bit formats): one single
// step, `launches` launches of m steps on `blocks` blocks, `rest` single steps.
struct MultiPlan {
    int m;               // 0: the class runs one step per launch
    int launches, rest, blocks;
    bool mu;
};

template <typename H, bool GH>
static void launch_multi_f(int D, const MultiPlan& p, hipStream_t st, const BatchHdr* hdr, const BatchGrid* tab, int j)
{
    const dim3 g(p.blocks);
    if (D == 2) {
        if (p.mu) hipLaunchKernelGGL((k_batch_march2d<H, GH, true>), g, dim3(NT), 0, st, hdr, tab, j);
        else hipLaunchKernelGGL((k_batch_march2d<H, GH, false>), g, dim3(NT), 0, st, hdr, tab, j);
    } else {
        if (p.mu) hipLaunchKernelGGL((k_batch_pair3d<H, GH, true>), g, dim3(1024), 0, st, hdr, tab, j);
        else hipLaunchKernelGGL((k_batch_pair3d<H, GH, false>), g, dim3(1024), 0, st, hdr, tab, j);
    }
}

// the launches of a class on a multi-step plan, directly on the stream: a
// quarter or half as many as steps, so they need no graph
static hipError_t launch_multi(lbem_batch_s* b, int c, const MultiPlan& p, hipStream_t st)
{
    const size_t cb = class_bytes(b->max_grids);
    const BatchHdr* hdr = (const BatchHdr*)(b->dev + c * cb);
    const BatchGrid* tab = (const BatchGrid*)(b->dev + c * cb + align256(sizeof(BatchHdr)));
    const int D = c < NPREC ? 2 : 3, prec = c < NPREC ? c : c - NPREC;
    launch_class(b, c, 0, st, MODE_CELL);
    for (int j = 0; j < p.launches; ++j) {
        switch (prec) {
            case LBEM_F16DEV: launch_multi_f<__half, false>(D, p, st, hdr, tab, j); break;
            case LBEM_BF16DEV: launch_multi_f<__hip_bfloat16, false>(D, p, st, hdr, tab, j); break;
            case LBEM_F16GHOST: launch_multi_f<__half, true>(D, p, st, hdr, tab, j); break;
            default: launch_multi_f<__hip_bfloat16, true>(D, p, st, hdr, tab, j); break;
        }
    }
    for (int k = 0; k < p.rest; ++k) launch_class(b, c, k, st, MODE_CELL, p.m);
    return hipGetLastError();
}

// The launches a member takes part in: the copy that holds its state flips in each.
static int multi_flips(int64_t nsteps, int m) { return (int)(1 + (nsteps - 1) / m + (nsteps - 1) % m); }

// Capture the per-class graphs.  Done once, at creation, with the library
// lock held exclusively: no graph is ever captured or instantiated while
// other threads allocate, free or launch through this library.
static bool capture_classes(lbem_batch_s* b)
{
    std::unique_lock<std::shared_mutex> lk(g_api_mu);
    for (int c = 0; c < NCLASS; ++c) {
        for (int mode = 0; mode < (has_row_modes(c) ? NMODE : 1); ++mode) {
            hipGraph_t graph = nullptr;
            hipGraphExec_t exec = nullptr;
            hipError_t e = hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal);
            if (e == hipSuccess) {
                for (int k = 0; k < b->ksteps; ++k) launch_class(b, c, k, b->stream, mode);
                e = hipStreamEndCapture(b->stream, &graph);
            }
            if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
            if (e != hipSuccess) {
                if (graph) (void)hipGraphDestroy(graph);
                (void)hipGetLastError();
                return false;
            }
            b->graph[c][mode] = graph;
            b->exec[c][mode] = exec;
        }
    }
    return true;
}

static hipError_t enqueue_tick(lbem_batch_s* b, unsigned mask, const int* mode, const MultiPlan* plan)
{
    const bool conc = b->concurrent && (mask & (mask - 1)) != 0;   // two classes or more
    hipError_t e = hipSuccess;
    if (conc && (e = hipEventRecord(b->fork_ev, b->stream)) != hipSuccess) return e;
    for (int c = 0; c < NCLASS; ++c) {
        if (!(mask & (1u << c))) continue;
        hipStream_t st = b->stream;
        if (conc) {
            st = b->cstream[c];
            if ((e = hipStreamWaitEvent(st, b->fork_ev, 0)) != hipSuccess) return e;
        }
        if (plan[c].m) {
            if ((e = launch_multi(b, c, plan[c], st)) != hipSuccess) return e;
        } else if (b->use_graph) {
            if ((e = hipGraphLaunch(b->exec[c][mode[c]], st)) != hipSuccess) return e;
        } else {
            for (int k = 0; k < b->ksteps; ++k) launch_class(b, c, k, st, mode[c]);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (conc) {
            if ((e = hipEventRecord(b->join_ev[c], st)) != hipSuccess) return e;
            if ((e = hipStreamWaitEvent(b->stream, b->join_ev[c], 0)) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

static void release_graphs(lbem_batch_s* b)
{
    for (int c = 0; c < NCLASS; ++c)
        for (int mode = 0; mode < NMODE; ++mode) {
            if (b->exec[c][mode]) (void)hipGraphExecDestroy(b->exec[c][mode]);
            if (b->graph[c][mode]) (void)hipGraphDestroy(b->graph[c][mode]);
            b->exec[c][mode] = nullptr;
            b->graph[c][mode] = nullptr;
        }
}

// State bytes one step of a member reads or writes: its population copies
// (one in place, two with pull), c_L^2 and the mu gradient.
static size_t touched_bytes(const lbem_s* h)
{
    const Sizes z = sizes_of(&h->cfg);
    return z.pop_one * (h->streaming == LBEM_STREAM_AA ? 1 : 2) + z.medium + (h->mu_set ? z.mu : 0);
}

// Whether class c's members of a group (its cnt entries of the table, in the
// order of idx) take several steps per launch, and if so their tilings.  The
// rows or planes per chunk are chosen for the members together, as the solo
// tilings choose them for one lattice.
static MultiPlan plan_multi(const lbem_batch_s* b, int c, char* host, const lbem_t* handles, const int64_t* nsteps,
                            const int* idx, int m, int cnt, int nmu)
{
    MultiPlan p{};
    const int prec = c < NPREC ? c : c - NPREC, D = c < NPREC ? 2 : 3;
    if (!b->multi || cnt == 0 || !is_dev(prec) || (nmu != 0 && nmu != cnt)) return p;
    const size_t cb = class_bytes(b->max_grids);
    BatchGrid* tab = (BatchGrid*)(host + c * cb + align256(sizeof(BatchHdr)));
    BatchHdr* hd = (BatchHdr*)(host + c * cb);
    const int ms = D == 2 ? 4 : 2;
    int64_t longest = 0, rows = 0, cells = 0;
    bool lines = true;                         // rows of whole 64-cell lines in every member
    std::vector<const lbem_s*> mem;
    for (int q = 0; q < m; ++q) {
        const lbem_s* h = handles[idx[q]];
        if (class_of(h) != c) continue;
        // a graph of the member's steps counts on the copy that single steps leave
        // its state in (lbem_step)
        if (h->graphed) return p;
        // a source needs its segments (a 3D handle below the solo kernel's size
        // rule has none)
        if (h->nsrc && !(D == 2 ? h->nmsrc > 0 : h->psrc_idx != nullptr)) return p;
        mem.push_back(h);
        longest = std::max(longest, nsteps[idx[q]]);
        p.rest = std::max(p.rest, (int)((nsteps[idx[q]] - 1) % ms));
        rows += (int64_t)h->mgeo.strips * h->cfg.ny;
        cells += h->n;
        lines = lines && h->cfg.nx % 64 == 0;
    }
    p.launches = (int)((longest - 1) / ms);
    if (p.launches < 1) return MultiPlan{};
    int64_t total = 0;
    if (D == 2) {
        const int64_t slots = 4096, rounds = ((rows + slots - 1) / slots + 23) / 24, per = std::max<int64_t>(1, rounds) * slots;
        const int r = (int)std::max<int64_t>(2, (rows + per - 1) / per);
        for (int k = 0; k < cnt; ++k) {
            MarchGeo& g = tab[k].mgeo;
            g = mem[k]->mgeo;
            g.rows = std::min(r, g.ny);
            g.nwork = g.strips * ((g.ny + g.rows - 1) / g.rows);
            tab[k].msrc_idx = mem[k]->msrc_idx;
            tab[k].msrc_val = (const float*)mem[k]->msrc_val;
            for (int w = 0; w < 8; ++w) tab[k].msrc_mask[w] = mem[k]->nmsrc ? mem[k]->msrc_mask[w] : 0u;
            tab[k].multi_base = (int)total;
            total += g.nwork;
        }
        p.blocks = (int)((total + NT / 64 - 1) / (NT / 64));
    } else {
        const int64_t cus = device_cus();
        int64_t best = -1;
        int lz = 4, longest_z = 1;
        for (const lbem_s* h : mem) longest_z = std::max(longest_z, (int)h->cfg.nz);
        for (int z = std::min(4, longest_z); z <= longest_z; ++z) {
            int64_t nb = 0;
            for (const lbem_s* h : mem) nb += (int64_t)h->pgeo.tiles_x * h->pgeo.tiles_y * ((h->cfg.nz + z - 1) / z);
            const int64_t cost = (nb + cus - 1) / cus * (z + 4);
            if (best < 0 || cost < best) { best = cost; lz = z; }
        }
        // the share of the work that is on stored cells, as for a single lattice.  us
        // per tick of 50 steps, single steps / pairs (share), FP16 ghost: 48^3 + 32^3 +
        // 48^3 + 64^3 (0.28) 879 / 936, 20 + 48 + 96 + 20 (0.46) 1456 / 1126, 96^3 (0.48)
        // 1253 / 963, 128^3 (0.49) 2500 / 1983; FP16-dev 128^3 3799 / 2788, 96^3 1324 /
        // 1129.
        const bool ghost = prec == LBEM_F16GHOST || prec == LBEM_BF16GHOST;
        const double share = (double)cells / ((double)best * cus * (PRX * PRY));
        if (b->multi < 2 && share < (ghost ? 0.30 : 0.36) + (lines ? 0.09 : 0.0)) return MultiPlan{};
        for (int k = 0; k < cnt; ++k) {
            PairGeo& g = tab[k].pgeo;
            g = mem[k]->pgeo;
            g.lz = std::min(lz, g.nz);
            g.nblocks = g.tiles_x * g.tiles_y * ((g.nz + g.lz - 1) / g.lz);
            tab[k].psrc_idx = mem[k]->psrc_idx;
            tab[k].psrc_val = mem[k]->psrc_val;
            tab[k].psrc_pair = mem[k]->psrc_pair;
            tab[k].multi_base = (int)total;
            total += g.nblocks;
        }
        p.blocks = (int)total;
    }
    hd->total_multi = (int)total;
    p.m = ms;
    p.mu = nmu != 0;
    return p;
}

// One group of a tick: its descriptor table through the next staging slot,
// the ordering against the members' own streams, and the classes' graphs.
// flips[i]: how often member i's state changes copies.
static int enqueue_group(lbem_batch_s* b, const lbem_t* handles, const int64_t* nsteps, const double* amp,
                         const int* idx, int m, int* flips)
{
    // the staging slot is free once its previous upload has executed
    if (hipEventSynchronize(b->ev[b->ring]) != hipSuccess) return LBEM_EDEVICE;
    char* host = b->pinned[b->ring];
    const size_t cb = class_bytes(b->max_grids);
    int cnt[NCLASS] = {0}, tiles[NCLASS] = {0}, rows[NCLASS] = {0};
    int nrow[NCLASS] = {0}, nmu[NCLASS] = {0};
    unsigned mask = 0;
    size_t amp_used = 0;      // end of the amplitudes written for this group
    for (int q = 0; q < m; ++q) {
        const int i = idx[q];
        lbem_s* h = handles[i];
        const int c = class_of(h);
        BatchGrid* tab = (BatchGrid*)(host + c * cb + align256(sizeof(BatchHdr)));
        BatchGrid& G = tab[cnt[c]++];
        std::memset(&G, 0, sizeof(G));
        if (h->prec <= LBEM_F32 || h->prec == LBEM_F16) {     // plain populations (FP16 storage included)
            const bool aa = h->streaming == LBEM_STREAM_AA;
            G.buf[0] = h->pop[0];
            G.buf[1] = aa ? h->pop[0] : h->pop[1];
            G.aa = aa;
        } else {
            const size_t moff = align256((size_t)(h->P + h->D) * h->n * 4);
            G.buf[0] = h->pop[0];
            G.buf[1] = h->pop[1];
            G.dev[0] = h->pop[0] + moff;
            G.dev[1] = h->pop[1] + moff;
            if (h->brow) {
                G.row = 1;
                G.row_base = rows[c];
                rows[c] += h->bgeo.nblocks;
                nrow[c]++;
                G.rgeo = h->bgeo;
                if (h->nbsrc) {
                    G.rsrc_off = h->bsrc_off;
                    G.rsrc_ent = h->bsrc_ent;
                    G.rsrc_val = h->bsrc_val;
                }
            }
        }
        G.cl2 = h->cl2;
        G.dlnmu = h->mu_set ? h->dlnmu : nullptr;
        nmu[c] += h->mu_set ? 1 : 0;
        // the member's own tiling, so that its per-tile source table applies
        Geo& g = G.geo;
        g = h->geo;
        g.xcd = 0;
        if (h->nsrc) {
            G.src_off = h->src_off;
            G.src_ent = h->src_ent;
            G.src_val = h->src_val;
            if (amp) {
                // this member's amplitudes, in the class's arithmetic type
                char* slot = host + b->amp_off + (size_t)i * b->ksteps * 8;
                const size_t dslot = b->amp_off + (size_t)i * b->ksteps * 8;
                for (int64_t j = 0; j < nsteps[i]; ++j) {
                    const double a = amp[(size_t)i * b->ksteps + j];
                    if (h->prec == LBEM_F64) ((double*)slot)[j] = a;
                    else ((float*)slot)[j] = (float)a;
                }
                G.amp = b->dev + dslot;
                amp_used = std::max(amp_used, dslot + (size_t)b->ksteps * 8);
            }
        }
        G.omega = 1.0 / h->cfg.tau;
        G.tau_half = h->cfg.tau == 0.5;
        G.cur0 = h->cur;
        G.fresh = h->layout == LAYOUT_NATURAL;
        G.nsteps = (int)nsteps[i];
        G.tile_base = tiles[c];
        tiles[c] += g.nblocks;
        mask |= 1u << c;
    }
    MultiPlan plan[NCLASS];
    for (int c = 0; c < NCLASS; ++c) plan[c] = plan_multi(b, c, host, handles, nsteps, idx, m, cnt[c], nmu[c]);
    for (int q = 0; q < m; ++q) {
        const MultiPlan& p = plan[class_of(handles[idx[q]])];
        flips[idx[q]] = p.m ? multi_flips(nsteps[idx[q]], p.m) : (int)nsteps[idx[q]];
    }
    int mode[NCLASS];
    for (int c = 0; c < NCLASS; ++c) {
        BatchHdr* hd = (BatchHdr*)(host + c * cb);
        hd->count = cnt[c];
        hd->total_tiles = tiles[c];
        hd->total_rows = rows[c];
        mode[c] = MODE_CELL;
        if (has_row_modes(c) && cnt[c] > 0 && nrow[c] == cnt[c] && rows[c] >= b->rows_min) {
            if (nmu[c] == 0) mode[c] = MODE_ROWS;
            else if (nmu[c] == cnt[c]) mode[c] = MODE_ROWS_MU;
        }
    }
    // members set up on other streams: their work so far precedes the group
    for (int q = 0; q < m; ++q) {
        lbem_s* h = handles[idx[q]];
        if (h->stream == b->stream) continue;
        if (hipEventRecord(h->sync_ev, h->stream) != hipSuccess ||
            hipStreamWaitEvent(b->stream, h->sync_ev, 0) != hipSuccess)
            return LBEM_EDEVICE;
    }
    if (hipMemcpyAsync(b->dev, host, amp_used ? amp_used : cb * NCLASS, hipMemcpyHostToDevice, b->stream) !=
        hipSuccess)
        return LBEM_EDEVICE;
    if (hipEventRecord(b->ev[b->ring], b->stream) != hipSuccess) return LBEM_EDEVICE;
    b->ring = (b->ring + 1) % NRING;
    if (mask && enqueue_tick(b, mask, mode, plan) != hipSuccess) return LBEM_EDEVICE;
    // ... and later work on a member's own stream (moments, destroy) follows
    // it: the member's stream waits on this event at its next use (follow_ticks)
    for (int q = 0; q < m; ++q) {
        lbem_s* h = handles[idx[q]];
        if (h->stream == b->stream) continue;
        if (hipEventRecord(h->tick_ev, b->stream) != hipSuccess) return LBEM_EDEVICE;
        h->tick_pending = true;
    }
    return LBEM_OK;
}

extern "C" {

int lbem_batch_create(int max_lattices, int steps_per_tick, void* stream, lbem_batch_t* out)
{
    if (!out || max_lattices < 1 || max_lattices > 65536 || steps_per_tick < 1 || steps_per_tick > 4096)
        return LBEM_EINVAL;
    *out = nullptr;
    if (!stream) return LBEM_EINVAL;  // a capturable stream is required
    lbem_batch_s* b = new (std::nothrow) lbem_batch_s();
    if (!b) return LBEM_ENOMEM;
    b->stream = (hipStream_t)stream;
    b->max_grids = max_lattices;
    b->ksteps = steps_per_tick;
    b->ring = 0;
    b->use_graph = env_int("LBEM_BATCH_GRAPH", 1);
    b->blocks = std::max(1, env_int("LBEM_BATCH_BLOCKS", BATCH_BLOCKS));
    // A row work item is a chunk of planes of a whole-row tile: 8-16 times a
    // per-cell tile.  Measured (FP16-dev): 20 lattices of 128^3 (10240 items)
    // 35.2k MLUPS with row tiles against 29.9k per-cell; 20 of 64^3 (1280
    // items) 27.0k against 33.0k; the serving mix at 200 req/s, whose 3D
    // classes hold a few small lattices, 37.2 against 38.6 GLUPS with the row
    // tiles always on (100 req/s: p50 141 against 62 ms).  So a class takes
    // them only with enough items to fill the GPU several times over.
    b->rows_min = std::max(0, env_int("LBEM_BATCH_ROWS_MIN", 1536));
    b->multi = env_int("LBEM_BATCH_MULTI", 1);
    b->amp_off = class_bytes(max_lattices) * NCLASS;
    const size_t bytes = b->amp_off + align256((size_t)max_lattices * steps_per_tick * 8);
    b->dev = nullptr;
    for (int r = 0; r < NRING; ++r) {
        b->pinned[r] = nullptr;
        b->ev[r] = nullptr;
    }
    // Lattices small enough for the 256 MB Infinity Cache are served from it
    // when several steps run on them back to back: with a budget, a tick runs
    // the members of each 3D class in groups whose state a step touches fits
    // it, each group for all of its steps, instead of every member once per
    // step.  Measured on the serving mix at 200 req/s: 38.7 GLUPS without
    // groups; 41.8, 43.4, 44.3-44.4, 44.0, 41.6 and 38.8 with 96, 160, 224,
    // 256, 320 and 640 MiB (100 req/s at 224 MiB: p50 68 ms, p99 0.37 s).
    // Groups that mixed classes (each group replaying every class's graph)
    // had measured 37.9.  LBEM_BATCH_GROUP_MIB=0 turns grouping off.
    b->group_bytes = (size_t)std::max(0, env_int("LBEM_BATCH_GROUP_MIB", 224)) << 20;
    for (int c = 0; c < NCLASS; ++c) {
        for (int mode = 0; mode < NMODE; ++mode) {
            b->graph[c][mode] = nullptr;
            b->exec[c][mode] = nullptr;
        }
        b->cstream[c] = nullptr;
        b->join_ev[c] = nullptr;
    }
    b->fork_ev = nullptr;
    // measured on the serving mix at 200 req/s: 36.0 GLUPS with the classes
    // concurrent against 38.6 one after another (the GPU is busy 99 % of the
    // time either way), so the default runs them in order on the batch stream
    b->concurrent = env_int("LBEM_BATCH_CONCURRENT", 0);
    bool ok;
    {
        API_SHARED;
        ok = hipMalloc((void**)&b->dev, bytes) == hipSuccess;
        for (int r = 0; ok && r < NRING; ++r) {
            ok = hipHostMalloc((void**)&b->pinned[r], bytes, hipHostMallocDefault) == hipSuccess &&
                 hipEventCreateWithFlags(&b->ev[r], hipEventDisableTiming) == hipSuccess;
            if (ok) std::memset(b->pinned[r], 0, bytes);
        }
        ok = ok && hipEventCreateWithFlags(&b->fork_ev, hipEventDisableTiming) == hipSuccess;
        for (int c = 0; ok && c < NCLASS; ++c) {
            ok = hipStreamCreateWithFlags(&b->cstream[c], hipStreamNonBlocking) == hipSuccess &&
                 hipEventCreateWithFlags(&b->join_ev[c], hipEventDisableTiming) == hipSuccess;
        }
    }
    if (ok && b->use_graph && !capture_classes(b)) {
        release_graphs(b);
        b->use_graph = 0;  // direct launches of the same kernels
    }
    if (ok) {
        ok = hipMemcpyAsync(b->dev, b->pinned[0], bytes, hipMemcpyHostToDevice, b->stream) == hipSuccess &&
             hipEventRecord(b->ev[0], b->stream) == hipSuccess;
    }
    if (!ok) {
        (void)lbem_batch_destroy(b);
        return LBEM_ENOMEM;
    }
    *out = b;
    return LBEM_OK;
}

int lbem_batch_destroy(lbem_batch_t b)
{
    if (!b) return LBEM_OK;
    API_SHARED;
    (void)hipStreamSynchronize(b->stream);
    for (int c = 0; c < NCLASS; ++c)
        if (b->cstream[c]) (void)hipStreamSynchronize(b->cstream[c]);
    release_graphs(b);
    for (int c = 0; c < NCLASS; ++c) {
        if (b->join_ev[c]) (void)hipEventDestroy(b->join_ev[c]);
        if (b->cstream[c]) (void)hipStreamDestroy(b->cstream[c]);
    }
    if (b->fork_ev) (void)hipEventDestroy(b->fork_ev);
    for (int i = 0; i < NRING; ++i) {
        if (b->ev[i]) (void)hipEventDestroy(b->ev[i]);
        if (b->pinned[i]) (void)hipHostFree(b->pinned[i]);
    }
    if (b->dev) (void)hipFree(b->dev);
    delete b;
    return LBEM_OK;
}

int lbem_batch_run(lbem_batch_t b, const lbem_t* handles, const int64_t* nsteps, int count)
{
    return lbem_batch_run_amp(b, handles, nsteps, nullptr, count);
}

int lbem_batch_run_amp(lbem_batch_t b, const lbem_t* handles, const int64_t* nsteps, const double* amp, int count)
{
    if (!b || count < 0 || count > b->max_grids || (count > 0 && (!handles || !nsteps))) return LBEM_EINVAL;
    for (int i = 0; i < count; ++i) {
        const lbem_s* h = handles[i];
        if (!h || nsteps[i] < 0 || nsteps[i] > b->ksteps) return LBEM_EINVAL;
        const bool plain = h->prec <= LBEM_F32 || h->prec == LBEM_F16;
        if (h->streaming != LBEM_STREAM_PULL && !(h->streaming == LBEM_STREAM_AA && plain)) return LBEM_EINVAL;
        if (has_bx(h)) return LBEM_EINVAL;                // periodic, no cell extras
        if (h->vec != 1) return LBEM_EINVAL;              // the batch tiles one row of cells per thread
        if (!h->have_fields) return LBEM_ESTATE;
        for (int j = 0; j < i; ++j)
            if (handles[j] == h) return LBEM_EINVAL;
    }
    // With a budget, members run in groups, each for all its steps: the
    // members of one class in call order, a 3D class split into runs of
    // members whose state touched per step fits the budget (a member larger
    // than it runs alone), a 2D class in one group.  Without one, all members
    // form one group.
    std::vector<int> order;
    order.reserve(count);
    for (int i = 0; i < count; ++i)
        if (nsteps[i] > 0) order.push_back(i);
    if (b->group_bytes)
        std::stable_sort(order.begin(), order.end(),
                         [&](int x, int y) { return class_of(handles[x]) < class_of(handles[y]); });
    std::vector<int> flips(count, 0);
    size_t g0 = 0;
    while (g0 < order.size()) {
        size_t g1 = g0, used = 0;
        const int c0 = class_of(handles[order[g0]]);
        while (g1 < order.size()) {
            const lbem_s* h = handles[order[g1]];
            if (b->group_bytes) {
                if (class_of(h) != c0) break;
                const size_t t = touched_bytes(h);
                if (g1 > g0 && h->D == 3 && used + t > b->group_bytes) break;
                used += t;
            }
            ++g1;
        }
        const int rc = enqueue_group(b, handles, nsteps, amp, order.data() + g0, (int)(g1 - g0), flips.data());
        if (rc != LBEM_OK) return rc;
        g0 = g1;
    }
    for (int i = 0; i < count; ++i) {
        lbem_s* h = handles[i];
        if (nsteps[i] == 0) continue;
        if (h->streaming == LBEM_STREAM_AA) {
            if (nsteps[i] & 1) h->layout = h->layout == LAYOUT_NATURAL ? LAYOUT_AA_SWAPPED : LAYOUT_NATURAL;
        } else {
            if (flips[i] & 1) h->cur = 1 - h->cur;
            h->layout = LAYOUT_PULL_PENDING;
        }
        h->t += nsteps[i];
    }
    return LBEM_OK;
}

}  // extern "C"
