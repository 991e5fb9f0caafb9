// Host runtime of libnd: argument validation, device buffers, batched launch
// sequences and the C ABI declared in include/nd.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "nd_dev.h"
#include "csr_layout.h"
#include "runtime.h"

namespace nd {

// ------------------------------------------------------------------ errors
static thread_local std::string g_err;

nd_status fail(nd_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

nd_status hip_fail(hipError_t e, const char* what) {
    if (e == hipErrorOutOfMemory) return fail(ND_ERR_OUT_OF_MEMORY, "%s: %s", what, hipGetErrorString(e));
    return fail(ND_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define HIPC(expr)                                        \
    do {                                                  \
        hipError_t e_ = (expr);                           \
        if (e_ != hipSuccess) return hip_fail(e_, #expr); \
    } while (0)

// ------------------------------------------------------------ validation
int nvars_of(int model) { return model == ND_KURAMOTO ? 1 : (model == ND_HH ? 4 : 2); }

static bool finite_all(const double* p, int n) {
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(p[i])) return false;
    return true;
}

nd_status validate_problem(const nd_problem* p) {
    if (!p) return fail(ND_ERR_INVALID_ARG, "problem is NULL");
    if (p->reserved != 0) return fail(ND_ERR_INVALID_ARG, "reserved field must be 0");
    if (p->precision != ND_FP64 && p->precision != ND_FP32_BULK)
        return fail(ND_ERR_INVALID_ARG, "unknown precision %d", p->precision);
    if (p->n < 1) return fail(ND_ERR_INVALID_ARG, "n must be >= 1 (got %lld)", (long long)p->n);
    if (p->n > (int64_t(1) << 31) - 1) return fail(ND_ERR_INVALID_ARG, "n must be < 2^31");
    if (p->model < 0 || p->model > 3) return fail(ND_ERR_INVALID_ARG, "unknown model %d", p->model);
    const int np = p->model == ND_KURAMOTO ? 3 : (p->model == ND_FHN ? 4 : (p->model == ND_HH ? 10 : 5));
    if (!finite_all(p->params, np)) return fail(ND_ERR_INVALID_ARG, "model parameters must be finite");
    if (p->model == ND_FHN && p->params[0] == 0.0) return fail(ND_ERR_INVALID_ARG, "FHN eps must be non-zero");
    if (p->model == ND_KURAMOTO_INERTIA && p->params[3] == 0.0)
        return fail(ND_ERR_INVALID_ARG, "the mass m must be non-zero (m = 0 is ND_KURAMOTO)");
    if (p->model == ND_HH && (p->params[0] == 0.0 || p->params[9] == 0.0))
        return fail(ND_ERR_INVALID_ARG, "HH C and k_s must be non-zero");
    switch (p->topo) {
        case ND_RING:
            if (p->model == ND_HH) return fail(ND_ERR_INVALID_ARG, "HH needs the CSR topology");
            if (p->radius < 1 || 2 * p->radius + 1 > p->n)
                return fail(ND_ERR_INVALID_ARG, "ring radius P must satisfy 1 <= P and 2P+1 <= n (n=%lld, P=%lld)",
                            (long long)p->n, (long long)p->radius);
            if (p->n >= (int64_t(1) << 29))
                return fail(ND_ERR_INVALID_ARG, "ring networks hold at most 2^29 - 1 elements (n=%lld)", (long long)p->n);
            break;
        case ND_CUBE3D: {
            if (p->model != ND_KURAMOTO && p->model != ND_KURAMOTO_INERTIA)
                return fail(ND_ERR_INVALID_ARG, "the cube topology is for the Kuramoto models");
            const int64_t side = 2 * p->radius + 1;
            if (p->radius < 1 || p->n1 < side || p->n2 < side || p->n3 < side)
                return fail(ND_ERR_INVALID_ARG, "cube extents must be >= 2h+1");
            if (p->n1 * p->n2 * p->n3 != p->n) return fail(ND_ERR_INVALID_ARG, "n must equal n1*n2*n3");
            if (p->n >= (int64_t(1) << 29))
                return fail(ND_ERR_INVALID_ARG, "lattices hold at most 2^29 - 1 elements (n=%lld)", (long long)p->n);
            break;
        }
        case ND_BALL3D: {
            if (p->model != ND_KURAMOTO && p->model != ND_KURAMOTO_INERTIA)
                return fail(ND_ERR_INVALID_ARG, "the ball topology is for the Kuramoto models");
            const int64_t side = 2 * p->radius + 1;
            if (p->radius < 1 || p->radius > kBallMaxP)
                return fail(ND_ERR_INVALID_ARG, "ball radius must be in [1, %d]", kBallMaxP);
            if (p->n1 < side || p->n2 < side || p->n3 < side)
                return fail(ND_ERR_INVALID_ARG, "lattice extents must be >= 2P+1");
            if (p->n1 * p->n2 * p->n3 != p->n) return fail(ND_ERR_INVALID_ARG, "n must equal n1*n2*n3");
            if (p->n >= (int64_t(1) << 29))
                return fail(ND_ERR_INVALID_ARG, "lattices hold at most 2^29 - 1 elements (n=%lld)", (long long)p->n);
            break;
        }
        case ND_DISK2D: {
            if (p->model != ND_KURAMOTO && p->model != ND_KURAMOTO_INERTIA)
                return fail(ND_ERR_INVALID_ARG, "the disk topology is for the Kuramoto models");
            const int64_t side = 2 * p->radius + 1;
            if (p->radius < 1 || p->radius > kBallMaxP)
                return fail(ND_ERR_INVALID_ARG, "disk radius must be in [1, %d]", kBallMaxP);
            if (p->n1 < side || p->n2 < side || p->n3 != 1)
                return fail(ND_ERR_INVALID_ARG, "the disk needs n1, n2 >= 2P+1 and n3 = 1");
            if (p->n1 * p->n2 != p->n) return fail(ND_ERR_INVALID_ARG, "n must equal n1*n2");
            if (p->n >= (int64_t(1) << 29))
                return fail(ND_ERR_INVALID_ARG, "lattices hold at most 2^29 - 1 elements (n=%lld)", (long long)p->n);
            break;
        }
        case ND_LINKS: {
            if (p->model == ND_HH) return fail(ND_ERR_INVALID_ARG, "HH needs the CSR topology (weighted links)");
            if (!p->row_ptr || (p->nnz > 0 && !p->col))
                return fail(ND_ERR_INVALID_ARG, "the links topology needs row_ptr and col");
            if (p->row_ptr[0] != 0 || p->row_ptr[p->n] != p->nnz)
                return fail(ND_ERR_INVALID_ARG, "row_ptr must start at 0 and end at nnz");
            if (p->n >= (int64_t(1) << 29))
                return fail(ND_ERR_INVALID_ARG, "link matrices hold at most 2^29 - 1 elements (n=%lld)", (long long)p->n);
            // row order and ranges are checked while compressing
            break;
        }
        case ND_CSR: {
            if (p->model != ND_HH) return fail(ND_ERR_INVALID_ARG, "the CSR topology is for HH");
            if (!p->row_ptr || (p->nnz > 0 && (!p->col || !p->weight)) || !p->per_elem)
                return fail(ND_ERR_INVALID_ARG, "CSR needs row_ptr, col, weight and per_elem");
            if (p->row_ptr[0] != 0 || p->row_ptr[p->n] != p->nnz)
                return fail(ND_ERR_INVALID_ARG, "row_ptr must start at 0 and end at nnz");
            for (int64_t i = 0; i < p->n; ++i)
                if (p->row_ptr[i + 1] < p->row_ptr[i]) return fail(ND_ERR_INVALID_ARG, "row_ptr must be non-decreasing");
            for (int64_t e = 0; e < p->nnz; ++e)
                if (p->col[e] < 0 || p->col[e] >= p->n) return fail(ND_ERR_INVALID_ARG, "col[%lld] out of range", (long long)e);
            if (!finite_all(p->weight, (int)std::min<int64_t>(p->nnz, INT32_MAX)))
                return fail(ND_ERR_INVALID_ARG, "weights must be finite");
            if (!finite_all(p->per_elem, (int)p->n)) return fail(ND_ERR_INVALID_ARG, "per_elem must be finite");
            break;
        }
        default:
            return fail(ND_ERR_INVALID_ARG, "unknown topology %d", p->topo);
    }
    return ND_OK;
}

// Lattice points within distance P of the origin, the origin included.
int64_t disk_points(int64_t P) {
    int64_t c = 0;
    for (int64_t dy = -P; dy <= P; ++dy)
        for (int64_t dx = -P; dx <= P; ++dx) c += dx * dx + dy * dy <= P * P;
    return c;
}

int64_t ball_points(int64_t P) {
    int64_t c = 0;
    for (int64_t dz = -P; dz <= P; ++dz)
        for (int64_t dy = -P; dy <= P; ++dy)
            for (int64_t dx = -P; dx <= P; ++dx) c += dx * dx + dy * dy + dz * dz <= P * P;
    return c;
}

// (dy, dz) runs of the ball of radius P, padded to the kernel's unroll of 8.
static int ball_runs(int P, int pz) {
    int c = 0;
    for (int dz = -pz; dz <= pz; ++dz)
        for (int dy = -P; dy <= P; ++dy) c += dz * dz + dy * dy <= P * P;
    return (c + 7) / 8 * 8;
}

// The distinct splits of n3 planes into at most 256 runs: (planes per run, runs).
static std::vector<std::pair<int, int>> z_splits(int n3) {
    std::vector<std::pair<int, int>> s;
    for (int zt = 1; zt <= std::min(n3, 256); ++zt) {
        const int cz = (n3 + zt - 1) / zt;
        if ((n3 + cz - 1) / cz == zt) s.emplace_back(cz, zt);
    }
    if (s.empty() || s[0].second != 1) s.insert(s.begin(), {n3, 1});
    return s;
}

// Plane-scatter form: 512-thread workgroups, two per CU where the radius is built
// for it and the two prefix planes fit twice in LDS.  The stage time of a tiling is
// predicted by a sum whose terms are what a work item does and whose weights (us)
// were fitted to 700 measured stages (radii 1 to 8, lattices of 33 to 100 an edge,
// both models and precisions; 7 % rms): per plane a constant and the halo rows, as
// rounds over the waves and as rows; per run pair executed (a pair is skipped where
// neither of its output planes is the item's) a constant and the output waves; per
// output plane the output waves.  `resident` work items share a CU and `rounds` of
// them follow one another.  It replaced a model fitted at P = 6 to the kernel before
// (us per stage, that one / now, inertia FP64: 100^3 P = 6 82 / 77; 33 x 37 x 41 P = 6
// 34 / 28, P = 4 24 / 19).  Below radius kBallScatterMinP the gather form is the
// default; block 512 selects this one there too.
constexpr int kBallScatterMinP = 3;
static bool ball_tiles_scatter(const nd_problem* p, int cus, int* cx_, int* cy_, int* cz_) {
    const int P = (int)p->radius;
    if (p->topo != ND_BALL3D || !ball_scatter_available(P) || P < kBallScatterMinP) return false;
    const int n1 = (int)p->n1, n2 = (int)p->n2, n3 = (int)p->n3;
    const int waves = kBallScatterBlock / 64;
    int pairs[kBallMaxP + 1];  // run pairs of |dz| = A
    for (int A = 0; A <= P; ++A) {
        pairs[A] = 0;
        for (int dy = -P; dy <= P; ++dy) pairs[A] += A * A + dy * dy <= P * P;
    }
    std::vector<std::pair<int, double>> runs;  // planes per work item, run pairs it executes
    for (const auto& [cz, zt] : z_splits(n3)) {
        (void)zt;
        double e = 0.0;
        for (int A = 0; A <= P; ++A) {
            // planes q with an output plane q - P - A or q - P + A in [0, cz)
            const int hit = A == 0 ? cz : 2 * cz - std::max(0, cz - 2 * A);
            e += (double)pairs[A] * hit;
        }
        runs.emplace_back(cz, e);
    }
    double best = 1e300;
    bool found = false;
    for (int cx = 1; cx <= std::min(n1, 64 - 2 * P); ++cx) {
        for (int cy = 1; cy <= std::min(n2, 4 * waves - 2 * P); ++cy) {
            if (cx * cy > kBallScatterBlock) break;
            const size_t sm = ball_scatter_smem_bytes(P, cx, cy);
            if (sm > kBallSmemMax) break;
            const int per_cu = P <= kBallScatterPairedMaxP && 2 * sm <= kBallSmemMax ? 2 : 1;
            const int64_t tiles = (int64_t)((n1 + cx - 1) / cx) * ((n2 + cy - 1) / cy);
            const double rows = (double)(cy + 2 * P) / waves, row_rounds = std::ceil(rows);
            const int out_waves = (cx * cy + 63) / 64;
            for (const auto& [cz, e] : runs) {
                const int64_t G = tiles * ((n3 + cz - 1) / cz);
                const int64_t rounds = (G + (int64_t)cus * per_cu - 1) / ((int64_t)cus * per_cu);
                const int resident = (int)std::min<int64_t>(per_cu, (G + cus - 1) / cus);
                const int planes = cz + 2 * P;
                const double item = planes * (0.349 + resident * (0.149 * row_rounds + 0.166 * rows)) +
                                    e * (0.0325 + 0.0021 * resident * out_waves) + 0.056 * cz * resident * out_waves;
                const double cost = 5.2 + rounds * item - 1e-6 * cx * cy;
                if (cost < best) {
                    best = cost;
                    found = true;
                    *cx_ = cx, *cy_ = cy, *cz_ = cz;
                }
            }
        }
    }
    return found;
}

// Gather form (disks, and balls below radius kBallScatterMinP).  Halo rows of HX =
// cx + 2P <= 64 lanes, at most 4 rows per wave and one output per thread, the prefix
// ring within the LDS budget.  A 256-thread workgroup leaves room for up to 4 per CU
// (LDS permitting), a 1024-thread one holds the CU alone.  The estimated time is
// (rounds of workgroups over the CU slots) x (planes per work item incl. the 2P
// lead-in) x (halo rows per wave + the outputs' prefix reads / 10).
// With `fitted` the tile for the workgroup size *bs_ is chosen by a predicted stage
// time (us) fitted to 860 measured stages of radius 1 and 2 (lattices of 30 to 120 an
// edge, 9 % rms): per plane a constant and the halo rows, per output plane a
// constant and the output waves' runs.  The estimate's tile / this one's, us per
// stage, inertia FP64: 100^3 P = 1 27 / 24, 60 x 50 x 40 P = 1 10.9 / 9.2, 33 x 37 x 41
// P = 2 12.1 / 10.4.
static void ball_tiles_gather(const nd_problem* p, int cus, bool fitted, int* cx_, int* cy_, int* cz_, int* bs_) {
    const int P = (int)p->radius, pz = ball_pz(p->topo, p->radius);
    const int n1 = (int)p->n1, n2 = (int)p->n2, n3 = (int)p->n3;
    const double runs = ball_runs(P, pz), reads = 0.1 * runs;
    const auto splits = z_splits(n3);
    double best = 1e300;
    *cx_ = 1, *cy_ = 1, *cz_ = n3;
    if (!fitted) *bs_ = 1024;
    const int only = fitted ? *bs_ : 0;
    for (int bs : {256, 1024}) {
        if (only && bs != only) continue;
        const int waves = bs / 64;
        for (int cx = 1; cx <= std::min(n1, 64 - 2 * P); ++cx) {
            for (int cy = 1; cy <= std::min(n2, 4 * waves - 2 * P); ++cy) {
                if (cx * cy > bs) break;
                const size_t sm = ball_smem_bytes(P, pz, cx, cy);
                if (sm > kBallSmemMax) break;
                const int per_cu = bs == 1024 ? 1 : std::max(1, std::min<int>(4, (int)(kBallSmemMax / sm)));
                const int64_t tiles = (int64_t)((n1 + cx - 1) / cx) * ((n2 + cy - 1) / cy);
                const double plane_cost = (double)((cy + 2 * P + waves - 1) / waves) + reads;
                for (const auto& [cz, zt] : splits) {
                    const int64_t rounds = (tiles * zt + (int64_t)cus * per_cu - 1) / ((int64_t)cus * per_cu);
                    double cost = (double)rounds * (cz + 2 * pz) * plane_cost - 1e-6 * cx * cy;
                    if (fitted) {
                        const int resident = (int)std::min<int64_t>(per_cu, (tiles * zt + cus - 1) / cus);
                        const double share = resident * waves / 16.0, rows = (double)(cy + 2 * P) / waves;
                        const double outs = (cx * cy + 63) / 64 * resident / 16.0;
                        cost = 5.7 +
                               rounds * ((cz + 2 * pz) * (0.208 + share * (0.263 * std::ceil(rows) + 0.436 * rows)) +
                                         cz * (0.8 + outs * (0.668 + 0.0629 * runs))) -
                               1e-6 * cx * cy;
                    }
                    if (cost < best) {
                        best = cost;
                        *cx_ = cx, *cy_ = cy, *cz_ = cz, *bs_ = bs;
                    }
                }
            }
        }
    }
}

static void ball_tiles(const nd_problem* p, int cus, int* cx_, int* cy_, int* cz_, int* bs_) {
    if (ball_tiles_scatter(p, cus, cx_, cy_, cz_)) {
        *bs_ = kBallScatterBlock;
        return;
    }
    ball_tiles_gather(p, cus, false, cx_, cy_, cz_, bs_);
    if (p->topo == ND_BALL3D) ball_tiles_gather(p, cus, true, cx_, cy_, cz_, bs_);
}

nd_kernel_config ball_gather_config(const nd_problem* p) {
    nd_kernel_config c = default_config(p);
    int cx, cy, cz, bs;
    ball_tiles_gather(p, device_cu_count(), false, &cx, &cy, &cz, &bs);
    c.tile = cx;
    c.tile_y = cy;
    c.tile_z = cz;
    c.block = bs;
    return c;
}

// ------------------------------------------------------------ configuration
// Compute units of the current device (256 on MI355X; also the answer when no
// device can be queried, e.g. for footprint estimates on a host without GPU).
int device_cu_count() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            return 256;
        }
        return n;
    }();
    return cus;
}

// Cube tiling.  A work item of cz planes takes a launch and lead-in share, 2h
// planes of mapping, and cz + 3 phases of the pipelined plane loop; a phase takes
// about 0.4 us plus 0.05 us per wave resident on the CU (its barrier and LDS round
// trips, then the waves' issue): measured 0.55 us at 3 waves, 0.72 at 6, 1.1 at 13,
// 1.15 at 15, a tenth less where two or more work items share a CU (they fill each
// other's waits).  Up to 16 waves (128 VGPRs) and the LDS of a CU are shared by its work
// items, which run in rounds.  Tiles whose extents the run length does not divide
// pay for the idle part of the last run.  Rounds x threads alone (the rule before)
// took few long work items on small lattices: us per stage (that rule and the loop
// it was made for / now) 40^3 h = 4 12.4 / 8.0, 31 x 37 x 29 h = 2 9.5 / 6.1, 101 x 90
// x 77 h = 2 FP32-bulk 16.5 / 12.9.
static void cube_tiles(const nd_problem* p, int cus, int* cx_, int* cy_, int* cz_) {
    const int h = (int)p->radius;
    const int n1 = (int)p->n1, n2 = (int)p->n2, n3 = (int)p->n3;
    const int run = cube_run(h);
    const auto splits = z_splits(n3);
    double best = 1e300;
    *cx_ = 1, *cy_ = 1, *cz_ = n3;
    for (int cx = 1; cx <= std::min(n1, 64); ++cx) {
        for (int cy = 1; cy <= std::min(n2, 64); ++cy) {
            const int halo = (cx + 2 * h) * (cy + 2 * h);
            if (halo > 1024) break;
            const int waves = (halo + 63) / 64;
            const size_t smem = cube_smem_bytes(h, cx, cy);
            const int per_cu = std::max(1, std::min(16 / waves, (int)(kBallSmemMax / smem)));
            const int64_t tiles = (int64_t)((n1 + cx - 1) / cx) * ((n2 + cy - 1) / cy);
            // share of the run threads' work that is kept
            const double fill = (double)cx * cy / (((cx + run - 1) / run * run) * (double)((cy + run - 1) / run * run));
            for (const auto& [cz, zt] : splits) {
                const int64_t G = tiles * zt, slots = (int64_t)cus * per_cu;
                const int64_t rounds = (G + slots - 1) / slots;
                const int res = waves * (int)std::min<int64_t>(per_cu, (G + cus - 1) / cus);
                // wide tiles run into LDS bank conflicts in the x runs (200^3, h = 4: 40 x 12
                // 86 us per stage, 12 x 40 81 us)
                const double phase = (0.4 + 0.05 * res * (0.7 + 0.3 / fill)) * (cx > cy + 4 ? 1.06 : 1.0) *
                                     (res > waves ? 0.9 : 1.0);
                const double cost = rounds * (3.0 + 2 * h * 0.02 * res + (cz + 3) * phase) + 1e-5 * halo - 1e-6 * cx;
                if (cost < best) {
                    best = cost;
                    *cx_ = cx, *cy_ = cy, *cz_ = cz;
                }
            }
        }
    }
}

nd_kernel_config default_config(const nd_problem* p) {
    nd_kernel_config c{};
    c.grid = 0;
    c.chunk = 64;
    if (p->topo == ND_RING) {
        // rings up to 4096 elements stay resident in one workgroup (negative tile =
        // resident capacity); larger rings use the per-stage tiled kernel
        if (p->n <= 1024) c.tile = -1024;
        else if (p->n <= 2048) c.tile = -2048;
        else if (p->n <= 4096) c.tile = -4096;
        else c.tile = p->n <= (int64_t(1) << 20) ? 512 : 1024;
        c.block = ring_block(c.tile);
    } else if (p->topo == ND_CUBE3D) {
        const int h = (int)p->radius;
        int cx, cy, cz;
        cube_tiles(p, device_cu_count(), &cx, &cy, &cz);
        c.tile = cx;
        c.tile_y = cy;
        c.tile_z = cz;
        c.block = cube_block(h, cx, cy);
    } else if (p->topo == ND_BALL3D || p->topo == ND_DISK2D) {
        int cx, cy, cz, bs;
        ball_tiles(p, device_cu_count(), &cx, &cy, &cz, &bs);
        c.tile = cx;
        c.tile_y = cy;
        c.tile_z = cz;
        c.block = bs;
    } else if (p->topo == ND_LINKS) {
        c.tile = kLinksRows;  // rows per work item
        c.block = 256;
    } else {
        c.tile = c.block = csr_rows(p->n);
        // edges per thread in flight: as many as the mean (512-row tile, source block)
        // half fills.  2e5 neurons, us per stage with 4 / 8 / 16 (FP64): degree 100
        // 88 / 81 / 73, degree 10 27 / 29 / 34 (more registers, fewer waves)
        const int64_t edges = p->nnz / kCsrSourceBlocks * 512 / p->n;
        c.tile_y = edges > 8 * 512 ? 16 : edges > 4 * 512 ? 8 : 4;
    }
    return c;
}

nd_kernel_config config_for(const nd_problem* p) {
    nd_kernel_config c = default_config(p);
    nd_kernel_config tuned;
    if (tuned_config(p, &tuned)) c = tuned;
    return c;
}

int ring_block(int tile) {
    if (tile < 0) return tile == -1024 ? 256 : 512;
    return tile == 128 ? 64 : (tile == 256 ? 128 : 256);  // two elements per thread up to 512
}

static int64_t bulk_bytes(int prec) { return prec == ND_FP64 ? 8 : 4; }

static int64_t ring_tiles(int64_t n, int tile) { return tile < 0 ? 1 : (n + tile - 1) / tile; }

int64_t footprint_bytes(const nd_problem* p, const nd_kernel_config& c) {
    const int64_t V = nvars_of(p->model), n = p->n, kb = bulk_bytes(p->precision);
    int64_t b = 3 * V * n * 8 + 3 * V * n * kb;  // y[2], acc, k[3]
    if (p->topo == ND_RING) b += 3 * 2 * ring_tiles(n, c.tile) * 8;
    if (p->topo == ND_CUBE3D || p->topo == ND_BALL3D || p->topo == ND_DISK2D)
        b += 3 * 2 * 8 * ((p->n1 + c.tile - 1) / c.tile) * ((p->n2 + c.tile_y - 1) / c.tile_y) *
             ((p->n3 + c.tile_z - 1) / c.tile_z);
    if (p->topo == ND_CSR)
        b += kCsrSourceBlocks * (n + 1) * 8 + p->nnz * (4 + kb) + n * 8 + 2 * n * kb + kCsrSourceBlocks * n * 8;
    if (p->topo == ND_LINKS) {
        // the compressed matrix (sized by compressing it), the two exchanged-map buffers and
        // the per-work-item sums
        LinksCompressed lc;
        if (compress_links(n, p->row_ptr, p->col, &lc) == ND_OK) b += links_device_bytes(lc);
        b += 2 * n * (int64_t)links_map_bytes(p->model, p->precision) + 3 * 2 * 8 * ((n + kLinksRows - 1) / kLinksRows);
    }
    b += sizeof(NetDesc) + 64;
    return b;
}

// -------------------------------------------------------------- allocation
// Buffers of networks the caller owns come from the device's stream-ordered
// pool, allocated and freed on a stream of the library's own (one per device,
// non-blocking, default priority).  A network's buffers are freed only after its
// own work has completed (its event), so destroying or reconfiguring a network
// waits for that network alone; hipFree would wait for the whole device.
constexpr int kMaxDevices = 64;
static std::mutex g_ls_mu;
static hipStream_t g_ls[kMaxDevices] = {};

static nd_status lib_stream(int dev, hipStream_t* out) {
    if (dev < 0 || dev >= kMaxDevices) return fail(ND_ERR_UNSUPPORTED, "device %d beyond %d devices", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_ls_mu);
    if (!g_ls[dev]) {
        int cur = 0;
        HIPC(hipGetDevice(&cur));
        if (cur != dev) HIPC(hipSetDevice(dev));
        const hipError_t e = hipStreamCreateWithFlags(&g_ls[dev], hipStreamNonBlocking);
        if (cur != dev) (void)hipSetDevice(cur);
        if (e != hipSuccess) return hip_fail(e, "hipStreamCreate (allocation stream)");
    }
    *out = g_ls[dev];
    return ND_OK;
}

nd_status Net::alloc(void** ptr, size_t bytes) {
    *ptr = nullptr;
    if (bytes == 0) bytes = 8;
    hipError_t e;
    if (astream) {
        e = hipMallocAsync(ptr, bytes, astream);
    } else {
        hipStream_t ls;
        const nd_status s = lib_stream(dev, &ls);
        if (s) return s;
        // ready for use on any stream once the allocation stream has passed it
        e = hipMallocAsync(ptr, bytes, ls);
        if (e == hipSuccess) e = hipStreamSynchronize(ls);
    }
    if (e != hipSuccess) return hip_fail(e, "hipMallocAsync");
    allocs.push_back(*ptr);
    return ND_OK;
}

// Pinned host words for the networks' status read-backs, carved from blocks
// that live until the process ends (hipHostFree would wait for the device).
static std::mutex g_pin_mu;
static std::vector<int32_t*> g_pin_free;

static nd_status pinned_word(int32_t** out) {
    std::lock_guard<std::mutex> lk(g_pin_mu);
    if (g_pin_free.empty()) {
        constexpr int kWords = 4096;
        int32_t* blk = nullptr;
        HIPC(hipHostMalloc((void**)&blk, kWords * sizeof(int32_t)));
        for (int i = kWords - 1; i >= 0; --i) g_pin_free.push_back(blk + i);
    }
    *out = g_pin_free.back();
    g_pin_free.pop_back();
    return ND_OK;
}

static void pinned_word_put(int32_t* w) {
    std::lock_guard<std::mutex> lk(g_pin_mu);
    g_pin_free.push_back(w);
}

// Return one of this network's buffers to the pool; the device no longer uses
// it (the caller has waited for the network's work, or owns astream's order).
void Net::free_buf(void* q) {
    if (astream) {
        (void)hipFreeAsync(q, astream);
        return;
    }
    hipStream_t ls;
    if (lib_stream(dev, &ls) == ND_OK) (void)hipFreeAsync(q, ls);
}

RunEvent::~RunEvent() {
    if (ev) (void)hipEventDestroy(ev);
}

void Net::quiesce() {
    if (ev_recorded) {
        (void)hipEventSynchronize(batch_ev ? batch_ev->ev : last_ev);
        ev_recorded = false;
    }
    batch_ev.reset();
}

nd_status Net::touch(hipStream_t st) {
    batch_ev.reset();
    hipError_t e = hipEventRecord(last_ev, st);
    if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
    ev_recorded = true;
    return ND_OK;
}

void Net::touch_shared(const std::shared_ptr<RunEvent>& ev) {
    batch_ev = ev;
    ev_recorded = true;
}

void Net::drop_graphs() {
    for (auto& g : solo_graph)
        if (g) {
            (void)hipGraphExecDestroy(g);
            g = nullptr;
        }
}

Net::~Net() {
    // server networks: the owner has seen the last work complete and the frees
    // are ordered on astream; others: wait for this network's own work
    if (!astream) quiesce();
    drop_graphs();
    for (void* q : allocs) free_buf(q);
    if (status_host && own_status_host) pinned_word_put(status_host);
    if (last_ev) (void)hipEventDestroy(last_ev);
}

// Host-to-device copy of set-up data (sources are host temporaries): synchronous,
// or on astream, waiting for that stream only, not for the device.
static hipError_t setup_copy(hipStream_t astream, void* dst, const void* src, size_t bytes) {
    if (!astream) return hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice);
    const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, astream);
    return e != hipSuccess ? e : hipStreamSynchronize(astream);
}

static void derive_params(const nd_problem* p, NetDesc& d) {
    std::memset(d.p, 0, sizeof d.p);
    if (p->model == ND_KURAMOTO || p->model == ND_KURAMOTO_INERTIA) {
        // links: the kernels divide each row's sum by its own link count
        const double L = p->topo == ND_RING     ? 2.0 * (double)p->radius
                         : p->topo == ND_BALL3D ? (double)ball_points(p->radius)
                         : p->topo == ND_DISK2D ? (double)disk_points(p->radius)
                         : p->topo == ND_LINKS  ? 1.0
                                                : std::pow(2.0 * (double)p->radius + 1.0, 3.0) - 1.0;
        d.p[0] = p->params[0];
        d.p[1] = p->params[1] / L;
        d.p[2] = std::cos(p->params[2]);
        d.p[3] = std::sin(p->params[2]);
        if (p->model == ND_KURAMOTO_INERTIA) {
            d.p[4] = p->params[4];        // eps
            d.p[5] = 1.0 / p->params[3];  // 1/m
        }
    } else if (p->model == ND_FHN) {
        d.p[0] = p->params[0];
        d.p[1] = p->params[1];
        // links: the kernels pass the row's mean, so kappa = sigma and the count is 1
        const double L = p->topo == ND_LINKS ? 1.0 : 2.0 * (double)p->radius;
        d.p[2] = p->params[2] / L;
        d.p[3] = std::cos(p->params[3]);
        d.p[4] = std::sin(p->params[3]);
        d.p[5] = L;
        d.p[6] = 1.0 / p->params[0];
    } else {
        for (int i = 0; i < 10; ++i) d.p[i] = p->params[i];
    }
}

// Upload a CSR network's edges in the gather kernel's layout.
template <class KT>
nd_status Net::upload_edges(const nd_problem* pr) {
    const int64_t nnz = pr->nnz;
    const CsrLayout<KT> L = csr_layout<KT>(pr->n, pr->row_ptr, pr->col, pr->weight);
    csr_edges = L.edges;
    NetDesc& d = tmpl;
    nd_status s;
    if ((s = alloc((void**)&d.row_ptr, L.bptr.size() * 8))) return s;
    if ((s = alloc((void**)&d.col, std::max<int64_t>(nnz, 1) * 4))) return s;
    if ((s = alloc((void**)&d.w, std::max<int64_t>(nnz, 1) * sizeof(KT)))) return s;
    HIPC(setup_copy(astream, (void*)d.row_ptr, L.bptr.data(), L.bptr.size() * 8));
    if (nnz > 0) {
        HIPC(setup_copy(astream, (void*)d.col, L.col.get(), nnz * 4));
        HIPC(setup_copy(astream, (void*)d.w, L.w.get(), nnz * sizeof(KT)));
    }
    return ND_OK;
}

nd_status Net::create(const nd_problem* pr) {
    HIPC(hipGetDevice(&dev));
    prob = *pr;
    prob.row_ptr = nullptr;
    prob.col = nullptr;
    prob.weight = nullptr;
    prob.per_elem = nullptr;
    cfg = config_for(pr);
    const int64_t V = nvars_of(pr->model), n = pr->n, kb = bulk_bytes(pr->precision);
    std::memset(&tmpl, 0, sizeof tmpl);
    NetDesc& d = tmpl;
    d.n = n;
    d.P = pr->radius;
    d.n1 = (int32_t)pr->n1;
    d.n2 = (int32_t)pr->n2;
    d.n3 = (int32_t)pr->n3;
    d.model = pr->model;
    d.prec = pr->precision;
    derive_params(pr, d);
    nd_status s;
    for (int b = 0; b < 2; ++b)
        if ((s = alloc((void**)&d.y[b], V * n * 8))) return s;
    if ((s = alloc((void**)&d.acc, V * n * 8))) return s;
    for (int b = 0; b < 3; ++b)
        if ((s = alloc(&d.k[b], V * n * kb))) return s;
    if (pr->topo == ND_CSR) {
        if ((s = kb == 8 ? upload_edges<double>(pr) : upload_edges<float>(pr))) return s;
        if ((s = alloc((void**)&d.acc_part, (size_t)kCsrSourceBlocks * n * 8))) return s;
        if ((s = alloc((void**)&d.iapp, n * 8))) return s;
        for (int b = 0; b < 2; ++b)
            if ((s = alloc(&d.sx[b], n * kb))) return s;
        HIPC(setup_copy(astream, (void*)d.iapp, pr->per_elem, n * 8));
    }
    if (pr->topo == ND_LINKS) {
        LinksCompressed lc;
        if ((s = compress_links(n, pr->row_ptr, pr->col, &lc))) return s;
        if ((int64_t)lc.dpos.size() >= (int64_t(1) << 31))
            return fail(ND_ERR_UNSUPPORTED, "links: the difference table holds 2^31 or more positions");
        LinksDeviceForm f;
        links_device_form(lc, &f);
        const size_t K = f.inv.size();
        if ((s = alloc((void**)&d.lrow, n * 4))) return s;
        if ((s = alloc((void**)&d.lvpos, lc.V.size() * 4))) return s;
        if ((s = alloc((void**)&d.ldptr, (K + 1) * 4))) return s;
        if ((s = alloc((void**)&d.ldpos, f.dsig.size() * 4))) return s;
        if ((s = alloc((void**)&d.linv, K * 8))) return s;
        for (int b = 0; b < 2; ++b)
            if ((s = alloc(&d.sx[b], n * (int64_t)links_map_bytes(pr->model, pr->precision)))) return s;
        d.lnv = (int32_t)lc.V.size();
        HIPC(setup_copy(astream, (void*)d.lrow, lc.C.data(), n * 4));
        if (!lc.V.empty()) HIPC(setup_copy(astream, (void*)d.lvpos, lc.V.data(), lc.V.size() * 4));
        HIPC(setup_copy(astream, (void*)d.ldptr, f.dptr.data(), (K + 1) * 4));
        if (!f.dsig.empty()) HIPC(setup_copy(astream, (void*)d.ldpos, f.dsig.data(), f.dsig.size() * 4));
        HIPC(setup_copy(astream, (void*)d.linv, f.inv.data(), K * 8));
    }
    if ((s = alloc((void**)&solo_desc, sizeof(NetDesc)))) return s;
    if ((s = alloc((void**)&status_dev, sizeof(int32_t)))) return s;
    HIPC(astream ? hipMemsetAsync(status_dev, 0, sizeof(int32_t), astream) : hipMemset(status_dev, 0, sizeof(int32_t)));
    if (own_status_host && (s = pinned_word(&status_host))) return s;
    *status_host = 0;
    HIPC(hipEventCreateWithFlags(&last_ev, hipEventDisableTiming));
    d.status = status_dev;
    return apply_config(cfg);
}

// (Re)build everything that depends on the kernel configuration: the work
// decomposition and the per-work-item sum buffers.
nd_status Net::apply_config(const nd_kernel_config& c) {
    quiesce();  // the buffers below may be in use by enqueued work
    drop_graphs();
    auto release = [&](void*& q) {
        if (!q) return;
        free_buf(q);
        allocs.erase(std::find(allocs.begin(), allocs.end(), q));
        q = nullptr;
    };
    release((void*&)tmpl.tsum[0]);
    release((void*&)tmpl.tsum[1]);
    release((void*&)tmpl.rsum);
    cfg = c;
    const int64_t n = prob.n;
    if (prob.topo == ND_RING) {
        cfg.block = ring_block(cfg.tile);
        tmpl.tile = cfg.tile;
        tmpl.G = (int32_t)ring_tiles(n, cfg.tile);
    } else if (prob.topo == ND_CUBE3D || prob.topo == ND_BALL3D || prob.topo == ND_DISK2D) {
        const int h = (int)prob.radius;
        if (prob.topo == ND_CUBE3D) cfg.block = cube_block(h, cfg.tile, cfg.tile_y);
        tmpl.cx = cfg.tile;
        tmpl.cy = cfg.tile_y;
        tmpl.cz = cfg.tile_z;
        tmpl.gx = (int32_t)((prob.n1 + cfg.tile - 1) / cfg.tile);
        tmpl.gy = (int32_t)((prob.n2 + cfg.tile_y - 1) / cfg.tile_y);
        tmpl.pz = ball_pz(prob.topo, prob.radius);
        const int32_t gz = (int32_t)((prob.n3 + cfg.tile_z - 1) / cfg.tile_z);
        tmpl.G = tmpl.gx * tmpl.gy * gz;
    } else if (prob.topo == ND_LINKS) {
        cfg.block = 256;
        cfg.tile = kLinksRows;  // rows per work item (fixed by the kernel)
        tmpl.tile = kLinksRows;
        tmpl.G = (int32_t)((n + kLinksRows - 1) / kLinksRows);
    } else {
        cfg.tile = cfg.block = csr_rows(n);  // rows per work item (fixed by the layout of the edges)
        tmpl.tile = csr_rows(n);
        tmpl.G = (int32_t)(kCsrSourceBlocks * ((n + csr_rows(n) - 1) / csr_rows(n)));  // (row tile, source block)
    }
    nd_status s;
    if (prob.topo != ND_CSR) {
        for (int b = 0; b < 2; ++b)
            if ((s = alloc((void**)&tmpl.tsum[b], 2 * (int64_t)tmpl.G * 8))) return s;
        if ((s = alloc((void**)&tmpl.rsum, 2 * (int64_t)tmpl.G * 8))) return s;
    }
    return ND_OK;
}

int64_t Net::work_items() const { return tmpl.G; }

Net::Class Net::kernel_class() const {
    if (prob.topo == ND_CSR) return {prob.model, prob.topo, prob.precision, 0, 0, 0, 0};
    const bool ball = prob.topo == ND_BALL3D || prob.topo == ND_DISK2D;
    return {prob.model, prob.topo, prob.precision, cfg.tile, cfg.tile_y,
            ball || prob.topo == ND_CUBE3D ? (int)prob.radius : 0, ball ? cfg.block : 0};
}

Group::Group(const Net::Class& c)
    : model(c[0]), topo(c[1]), prec(c[2]), tile(c[3]), tile_y(c[4]), h(c[5]), block(c[6]) {}

int Net::part() const { return prob.topo == ND_CSR && csr_rows(prob.n) > 256; }

// CSR: one update launch for all, one gather launch for each row count, with the edges
// in flight of its network that has the most links (see csr_unroll).  us per step of
// batches in a set of launches for each row count and each value of edges in flight, one
// after the other / so: 12 networks of 2000 neurons and degrees 5 to 100 127 / 59, 12 of
// 10^4 168 / 113, four of 5 10^4 and degrees 10 to 100 220 / 161, six of 2000 to 10^5
// neurons and degrees 10 to 100 316 / 222, of 2000 to 2 10^5 and degree 20 229 / 210.  (One
// gather launch for both row counts: four of degree 100 beside 10^5 neurons of degree 10 take
// 201 against 174 us, the LDS of the fullest items holds back the others' workgroups.)
void Group::take(const Net& n) {
    mv = mv || n.mv_start >= 0;
    if (topo != ND_CSR) return;
    CsrPart& c = csr[n.part()];
    c.items += n.work_items();
    c.edges = std::max(c.edges, n.csr_edges);
    c.mixed = c.mixed || (c.unroll && c.unroll != n.cfg.tile_y);
    if (!c.unroll || n.prob.nnz > c.nnz) {
        c.nnz = n.prob.nnz;
        c.unroll = n.cfg.tile_y;
    }
}

// Edges in flight of a gather launch: 16 take twice the registers of 8, which halves
// the waves of the lighter networks where the products' LDS would allow them, i.e. of
// 256-row work items (us per step with 16 / 8: 12 of 10^4 120 / 114, four of 5 10^4
// 170 / 162; all of degree 100 148 / 148).  The LDS of 512-row items binds first.
static int csr_unroll(const CsrPart& c, int part) { return c.mixed && part == 0 ? std::min(c.unroll, 8) : c.unroll; }

nd_status Net::prepare_observe(int64_t steps, const nd_observe* obs, bool may_alloc) {
    last_steps = steps;
    r_every = 0;
    mv_start = -1;
    if (!obs) return ND_OK;
    if (obs->record_every < 0) return fail(ND_ERR_INVALID_ARG, "record_every must be >= 0");
    if (obs->mv_start_step < -1) return fail(ND_ERR_INVALID_ARG, "mv_start_step must be >= -1");
    const bool want_r = obs->record_every > 0, want_mv = obs->mv_start_step >= 0;
    if ((want_r || want_mv) && prob.model == ND_HH)
        return fail(ND_ERR_INVALID_ARG, "R and mean phase velocity are not defined for HH");
    if ((want_r || want_mv) && steps < 1) return fail(ND_ERR_INVALID_ARG, "recording observables needs steps >= 1");
    if (want_mv && obs->mv_start_step >= steps) return fail(ND_ERR_INVALID_ARG, "mv_start_step must be < steps");
    nd_status s;
    if (want_r) {
        const int64_t len = steps / obs->record_every + 1;
        if (len > R_cap && !may_alloc)
            return fail(ND_ERR_INVALID_ARG,
                        "recording %lld values of R needs a buffer an earlier run sized (it holds %lld)",
                        (long long)len, (long long)R_cap);
        if (len > R_cap) {
            if (R_dev) {
                quiesce();  // earlier runs may still record into it
                free_buf(R_dev);
                allocs.erase(std::find(allocs.begin(), allocs.end(), (void*)R_dev));
            }
            if ((s = alloc((void**)&R_dev, len * 8))) return s;
            R_cap = len;
        }
        r_every = obs->record_every;
    }
    if (want_mv) {
        if (!mv_dev && !may_alloc)
            return fail(ND_ERR_INVALID_ARG, "recording the mean phase velocity needs a buffer an earlier run sized");
        if (!mv_dev && (s = alloc((void**)&mv_dev, prob.n * 8))) return s;
        mv_start = obs->mv_start_step;
    }
    return ND_OK;
}

NetDesc Net::run_desc(double dt, int64_t steps) const {
    NetDesc d = tmpl;
    d.dt = dt;
    d.dt3 = dt / 3.0;
    d.dt6 = dt / 6.0;
    d.obs = (r_every > 0 ? OBS_R : 0) | (mv_start >= 0 ? OBS_MV : 0);
    d.R = R_dev;
    d.r_every = r_every > 0 ? r_every : 1;
    d.mv = mv_dev;
    d.mv_start = mv_start;
    d.mv_scale = mv_start >= 0 ? 1.0 / ((double)(steps - mv_start) * dt) : 0.0;
    d.g0 = 0;
    d.nsteps = steps;
    d.ypar = ypar;
    d.tag = status_tag;
    return d;
}

nd_status Net::begin_run(double dt, int64_t steps, const nd_observe* obs) {
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(ND_ERR_INVALID_ARG, "dt must be finite and > 0");
    if (steps < 1) return fail(ND_ERR_INVALID_ARG, "steps must be >= 1");
    nd_status s = prepare_observe(steps, obs);
    if (s) return s;
    run_dt = dt;
    run_total = steps;
    run_done = 0;
    return ND_OK;
}

NetDesc Net::chunk_desc() const {
    NetDesc d = run_desc(run_dt, run_total);
    d.g0 = run_done;
    d.nsteps = run_total - run_done;
    return d;
}

// ----------------------------------------------------------- launch groups
__global__ void k_advance(NetDesc* D, int ndesc, int chunk) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ndesc) {
        NetDesc& d = D[i];
        if (d.nsteps > 0) {
            const int64_t done = d.nsteps < chunk ? d.nsteps : (int64_t)chunk;
            d.g0 += done;
            d.nsteps -= done;
            d.ypar ^= (int)(done & 1);
        }
    }
}

// Enqueue one chunk of `chunk` steps for a group of networks of one kernel
// class.  Each network runs min(chunk, remaining) steps.
nd_status enqueue_chunk(const Group& g, int chunk, hipStream_t st) {
    const int grid = g.grid;
    hipError_t e;
    if (g.topo == ND_RING) {
        RingLaunch L;
        if (!ring_select(g.model, g.prec, g.tile, &L)) return fail(ND_ERR_UNSUPPORTED, "no ring kernel for tile %d", g.tile);
        if (g.tile < 0) {
            if (!L.resident || L.bs > -g.tile) return fail(ND_ERR_UNSUPPORTED, "bad resident ring entry");
            if ((e = ring_launch_resident(L, grid, st, g.desc, g.work, g.nwork, chunk, g.mv)) != hipSuccess)
                return hip_fail(e, "ring resident");
        } else {
            if ((e = ring_launch_prologue(L, grid, st, g.desc, g.work, g.nwork)) != hipSuccess)
                return hip_fail(e, "ring prologue");
            for (int j = 0; j < chunk; ++j)
                for (int s = 1; s <= 4; ++s)
                    if ((e = ring_launch_stage(L, grid, st, g.desc, g.work, g.nwork, s, j, g.mv)) != hipSuccess)
                        return hip_fail(e, "ring stage");
        }
        if ((e = ring_launch_epilogue(L, grid, st, g.desc, g.work, g.nwork, chunk)) != hipSuccess)
            return hip_fail(e, "ring epilogue");
    } else if (g.topo == ND_CUBE3D) {
        CubeLaunch L;
        if (!cube_select(g.model, g.prec, g.h, &L))
            return fail(ND_ERR_UNSUPPORTED, "no cube kernel for model %d, h = %d", g.model, g.h);
        const int block = cube_block(g.h, g.tile, g.tile_y);
        const size_t smem = cube_smem_bytes(g.h, g.tile, g.tile_y);
        for (int j = 0; j < chunk; ++j)
            for (int s = 1; s <= 4; ++s)
                if ((e = cube_launch_stage(L, grid, block, smem, st, g.desc, g.work, g.nwork, s, j, g.mv)) != hipSuccess)
                    return hip_fail(e, "cube stage");
        if ((e = cube_launch_final(L, grid, st, g.desc, g.work, g.nwork, chunk)) != hipSuccess)
            return hip_fail(e, "cube final");
    } else if (g.topo == ND_BALL3D || g.topo == ND_DISK2D) {
        CubeLaunch L;
        const bool scatter = g.block == kBallScatterBlock;
        if (scatter ? !ball_scatter_select(g.model, g.prec, g.h, &L) : !ball_select(g.model, g.prec, g.block, &L))
            return fail(ND_ERR_UNSUPPORTED, "no ball kernel for model %d, block %d, radius %d", g.model, g.block, g.h);
        const size_t smem = scatter ? ball_scatter_smem_bytes(g.h, g.tile, g.tile_y)
                                    : ball_smem_bytes(g.h, ball_pz(g.topo, g.h), g.tile, g.tile_y);
        for (int j = 0; j < chunk; ++j)
            for (int s = 1; s <= 4; ++s)
                if ((e = cube_launch_stage(L, grid, g.block, smem, st, g.desc, g.work, g.nwork, s, j, g.mv)) != hipSuccess)
                    return hip_fail(e, "ball stage");
        if ((e = cube_launch_final(L, grid, st, g.desc, g.work, g.nwork, chunk)) != hipSuccess)
            return hip_fail(e, "ball final");
    } else if (g.topo == ND_LINKS) {
        LinksLaunch L;
        if (!links_select(g.model, g.prec, &L)) return fail(ND_ERR_UNSUPPORTED, "no links kernel for model %d", g.model);
        if ((e = links_launch_chunk(L, grid, st, g.desc, g.work, g.nwork, chunk, g.mv)) != hipSuccess)
            return hip_fail(e, "links chunk");
    } else {
        CsrLaunch L[2];
        for (int p = 0; p < 2; ++p)
            if (g.csr[p].items && !csr_select(g.prec, csr_unroll(g.csr[p], p), p ? 512 : 256, &L[p]))
                return fail(ND_ERR_UNSUPPORTED, "no CSR kernel for %d edges per thread", csr_unroll(g.csr[p], p));
        const CsrLaunch& all = L[g.csr[1].items ? 1 : 0];  // the larger workgroups
        const bool both = g.csr[0].items && g.csr[1].items;
        if ((e = csr_launch_prologue(all, grid, st, g.desc, g.work, g.nwork)) != hipSuccess) return hip_fail(e, "csr prologue");
        for (int j = 0; j < chunk; ++j)
            for (int s = 1; s <= 4; ++s) {
                int w0 = 0;
                for (int p = 0; p < 2; ++p) {
                    if (!g.csr[p].items) continue;
                    // (a part that is alone takes all items: in a captured chunk their number varies)
                    const int m = both ? (int)g.csr[p].items : INT32_MAX;
                    if ((e = csr_launch_gather(L[p], std::min(grid, m), g.csr[p].edges, st, g.desc, g.work, g.nwork, w0,
                                               both ? w0 + m : m, s, j)) != hipSuccess)
                        return hip_fail(e, "csr gather");
                    w0 += m;
                }
                if ((e = csr_launch_update(all, grid, st, g.desc, g.work, g.nwork, s, j)) != hipSuccess)
                    return hip_fail(e, "csr update");
            }
    }
    hipLaunchKernelGGL(k_advance, dim3((g.ndesc + 255) / 256), dim3(256), 0, st, g.desc, g.ndesc, chunk);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "advance");
    return ND_OK;
}

bool graphs_enabled() {
    static const bool on = [] {
        const char* v = getenv("ND_GRAPHS");
        return !(v && v[0] == '0');
    }();
    return on;
}

// Capture one chunk of K steps of group g into an executable graph.
nd_status capture_chunk(const Group& g, int K, hipGraphExec_t* out) {
    hipStream_t cap;
    HIPC(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        (void)hipStreamDestroy(cap);
        return hip_fail(e, "hipStreamBeginCapture");
    }
    nd_status s = enqueue_chunk(g, K, cap);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(cap, &graph);
    (void)hipStreamDestroy(cap);
    if (s) {
        if (graph) (void)hipGraphDestroy(graph);
        return s;
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    e = hipGraphInstantiate(out, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return hip_fail(e, "hipGraphInstantiate");
    return ND_OK;
}

// State values per launch from which a group runs without graph capture.
constexpr int64_t kEagerValues = int64_t(1) << 20;

// Steps per launch of rings resident in one workgroup.  A chunk is one kernel
// there, so replaying captured 64-step chunks only added launches (and a capture
// per batch): 0.97 us per stage of one 1024-ring in replays, 0.93 us in one launch;
// 512 rings 1.77 and 1.67 us.  Beyond 4 10^6 elements, where a step of the batch takes
// 36 us (4096 Kuramoto rings of 1024, FP64) and more rings take as much longer, the
// steps are cut so that a launch stays at some tens of milliseconds; 64 steps at the
// least, whose launch costs nothing beside them.
static int64_t resident_steps(int64_t elements) {
    return std::clamp((int64_t(1) << 32) / elements, int64_t(64), int64_t(1024));
}

// A group of resident rings of so many elements: chunks launched directly.
static nd_status run_resident(const Group& g, int64_t elements, int64_t maxsteps, hipStream_t st) {
    const int64_t K = resident_steps(elements);
    for (int64_t done = 0; done < maxsteps; done += K) {
        const nd_status s = enqueue_chunk(g, (int)std::min(K, maxsteps - done), st);
        if (s) return s;
    }
    return ND_OK;
}

__global__ void k_put_desc(NetDesc* dst, NetDesc d) { *dst = d; }
__global__ void k_clear_status(int32_t* status) { *status = 0; }

// Work enqueued on st is being recorded into a graph (the default stream never is).
static bool capturing(hipStream_t st) {
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    return st && hipStreamIsCapturing(st, &c) == hipSuccess && c == hipStreamCaptureStatusActive;
}

hipError_t put_desc(NetDesc* dst, const NetDesc& d, hipStream_t st) {
    hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(1), 0, st, dst, d);
    return hipGetLastError();
}

// Pinned host staging for the descriptor tables and work maps of batched runs.
// A block is handed out again only after the event recorded behind its upload
// has completed, so a run returns without waiting for the device and the host
// never rewrites a block a pending copy still reads.
namespace {
struct Staging {
    void* p = nullptr;
    size_t cap = 0;
    hipEvent_t ev = nullptr;
    bool busy = false;      // handed out, upload not yet recorded
    bool pending = false;   // an upload from it may still be in flight
};
std::mutex g_stage_mu;
std::vector<std::unique_ptr<Staging>> g_stage;

// Graph executables of batched runs, destroyed once their last replay is done.
struct DeadGraph {
    hipGraphExec_t exec;
    hipEvent_t ev;
};
std::mutex g_dead_mu;
std::vector<DeadGraph> g_dead;

void reap_graphs() {
    std::lock_guard<std::mutex> lk(g_dead_mu);
    std::vector<DeadGraph> keep;
    for (const DeadGraph& d : g_dead) {
        if (hipEventQuery(d.ev) == hipSuccess) {
            (void)hipGraphExecDestroy(d.exec);
            (void)hipEventDestroy(d.ev);
        } else {
            keep.push_back(d);
        }
    }
    g_dead.swap(keep);
}

nd_status retire_graph(hipGraphExec_t exec, hipStream_t st) {
    hipEvent_t ev;
    hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(ev, st);
    if (e != hipSuccess) {  // fall back to waiting here
        (void)hipStreamSynchronize(st);
        (void)hipGraphExecDestroy(exec);
        return hip_fail(e, "graph retirement event");
    }
    std::lock_guard<std::mutex> lk(g_dead_mu);
    g_dead.push_back({exec, ev});
    return ND_OK;
}

nd_status staging_get(size_t bytes, Staging** out) {
    std::lock_guard<std::mutex> lk(g_stage_mu);
    for (auto& b : g_stage) {
        if (b->busy || b->cap < bytes) continue;
        if (b->pending) {
            if (hipEventQuery(b->ev) != hipSuccess) continue;
            b->pending = false;
        }
        b->busy = true;
        *out = b.get();
        return ND_OK;
    }
    auto b = std::make_unique<Staging>();
    b->cap = std::max<size_t>(bytes, 64 * 1024);
    hipError_t e = hipHostMalloc(&b->p, b->cap);
    if (e != hipSuccess) return hip_fail(e, "hipHostMalloc (staging)");
    e = hipEventCreateWithFlags(&b->ev, hipEventDisableTiming);
    if (e != hipSuccess) {
        (void)hipHostFree(b->p);
        return hip_fail(e, "hipEventCreate (staging)");
    }
    b->busy = true;
    *out = b.get();
    g_stage.push_back(std::move(b));
    return ND_OK;
}

// The uploads from `b` are enqueued on st: record that and release the block.
nd_status staging_put(Staging* b, hipStream_t st) {
    hipError_t e = hipEventRecord(b->ev, st);
    std::lock_guard<std::mutex> lk(g_stage_mu);
    b->busy = false;
    b->pending = true;
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(st);
        b->pending = false;
        return hip_fail(e, "hipEventRecord (staging)");
    }
    return ND_OK;
}

// Kernel classes of one call's networks.  CSR networks of both row counts share their
// launches only while the edges of all stay in the Infinity Cache (256 MB) from stage to
// stage; beyond, the smaller networks run their steps before the larger ones, each set
// with more of its edges in the cache.  Six networks of 2000 to 2 10^5 neurons, us per
// step together / one after the other: degree 20 (86 MB) 210 / 222, degree 50 (214 MB)
// 356 / 302, degree 100 (428 MB) 543 / 524; 139 MB (eight of 2000 and one of 10^5, degree
// 100) 175 / 181.
class BatchClasses {
public:
    BatchClasses(Net* const* nets, int count, const int64_t* steps) {
        for (int i = 0; i < count; ++i)
            if (nets[i]->prob.topo == ND_CSR && steps[i] > 0)
                edge_bytes_[fp64(nets[i])] += nets[i]->prob.nnz * (fp64(nets[i]) ? 12 : 8);
    }
    Net::Class of(const Net* n) const {
        Net::Class c = n->kernel_class();
        if (n->prob.topo == ND_CSR && edge_bytes_[fp64(n)] > kSharedBytes) c[6] = n->part();
        return c;
    }

private:
    static constexpr int64_t kSharedBytes = int64_t(192) << 20;
    static bool fp64(const Net* n) { return n->prob.precision == ND_FP64; }
    int64_t edge_bytes_[2] = {0, 0};
};
}  // namespace

// Run a set of networks (possibly of different classes) for their own step
// counts.  Everything is enqueued on st and the call returns without waiting
// for the device: descriptors of a single network travel as a kernel argument,
// those of batches through pinned staging blocks; each network records an event
// behind its work so that reconfiguring or destroying it waits for exactly that.
nd_status run_nets(Net* const* nets, int count, const double* dt, const int64_t* steps, const nd_observe* obs,
                   hipStream_t st) {
    // validate and prepare observables
    for (int i = 0; i < count; ++i) {
        if (!nets[i]) return fail(ND_ERR_INVALID_ARG, "handle %d is NULL", i);
        if (!(dt[i] > 0.0) || !std::isfinite(dt[i])) return fail(ND_ERR_INVALID_ARG, "dt must be finite and > 0");
        if (steps[i] < 0) return fail(ND_ERR_INVALID_ARG, "steps must be >= 0");
    }
    {
        std::vector<Net*> sorted(nets, nets + count);
        std::sort(sorted.begin(), sorted.end());
        if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end())
            return fail(ND_ERR_INVALID_ARG, "a handle appears twice in one batch");
    }
    reap_graphs();
    nd_status s;
    for (int i = 0; i < count; ++i)
        if ((s = nets[i]->prepare_observe(steps[i], obs ? &obs[i] : nullptr))) return s;
    if (capturing(st))
        for (int i = 0; i < count; ++i) nets[i]->captured = true;
    // group by kernel class
    const BatchClasses classes(nets, count, steps);
    std::map<Net::Class, std::vector<int>> groups;
    for (int i = 0; i < count; ++i)
        if (steps[i] > 0) groups[classes.of(nets[i])].push_back(i);
    for (auto& kv : groups) {
        std::vector<int>& idx = kv.second;
        const Net* n0 = nets[idx[0]];
        std::stable_partition(idx.begin(), idx.end(), [&](int q) { return nets[q]->part() == 0; });
        Group g(kv.first);
        g.ndesc = (int)idx.size();
        int64_t maxsteps = 0, nwork = 0;
        for (int q : idx) {
            g.take(*nets[q]);
            nwork += nets[q]->work_items();
            maxsteps = std::max(maxsteps, steps[q]);
        }
        const bool solo = idx.size() == 1;
        void* scratch = nullptr;
        hipError_t e;
        if (solo) {
            Net* n = nets[idx[0]];
            // the kernels need no map for one network (work_count, work_at)
            g.desc = n->solo_desc;
            g.work = nullptr;
            g.nwork = nullptr;
            if ((e = put_desc(g.desc, n->run_desc(dt[idx[0]], steps[idx[0]]), st)) != hipSuccess)
                return hip_fail(e, "descriptor upload");
        } else {
            const size_t bd = idx.size() * sizeof(NetDesc), bw = (size_t)nwork * sizeof(int2);
            Staging* sb = nullptr;
            if ((s = staging_get(bd + bw + 16, &sb))) return s;
            NetDesc* hd = (NetDesc*)sb->p;
            int2* hw = (int2*)((char*)sb->p + bd);
            int w = 0;
            for (int q = 0; q < (int)idx.size(); ++q) {
                Net* n = nets[idx[q]];
                hd[q] = n->run_desc(dt[idx[q]], steps[idx[q]]);
                const int64_t m = n->work_items();
                for (int64_t t = 0; t < m; ++t) hw[w++] = make_int2(q, (int)t);
            }
            *(int*)((char*)sb->p + bd + bw) = w;
            e = hipMallocAsync(&scratch, bd + bw + 16, st);
            if (e == hipSuccess) e = hipMemcpyAsync(scratch, sb->p, bd + bw + 16, hipMemcpyHostToDevice, st);
            const nd_status sp = staging_put(sb, st);
            if (e != hipSuccess) return hip_fail(e, "batch descriptor upload");
            if (sp) return sp;
            g.desc = (NetDesc*)scratch;
            g.work = (int2*)((char*)scratch + bd);
            g.nwork = (int*)((char*)scratch + bd + bw);
        }
        const int cfg_grid = n0->cfg.grid;
        g.grid = cfg_grid > 0 ? (int)std::min<int64_t>(cfg_grid, nwork) : (int)nwork;
        const int K = std::max(1, n0->cfg.chunk);
        // Replaying a captured chunk saves the host's per-launch cost, which matters
        // for short kernels; groups whose stage kernels are long (many state values
        // per launch) run eagerly, which measured a few percent faster per launch.
        int64_t values = 0;
        for (int q : idx) values += nets[q]->prob.n * nvars_of(nets[q]->prob.model);
        const bool eager = values >= kEagerValues;
        if (g.topo == ND_RING && g.tile < 0) {
            if ((s = run_resident(g, values / nvars_of(g.model), maxsteps, st))) return s;
        } else if (maxsteps <= K || !graphs_enabled() || eager) {
            // one eager chunk covering every network's steps
            if ((s = enqueue_chunk(g, (int)std::min<int64_t>(maxsteps, 1 << 30), st))) return s;
        } else {
            // replay a captured K-step chunk; the descriptors advance on the
            // device, so every replay continues where the last one stopped
            const int64_t reps = (maxsteps + K - 1) / K;
            hipGraphExec_t exec = nullptr;
            Net* so = solo ? nets[idx[0]] : nullptr;
            const int slot = g.mv ? 1 : 0;
            if (so && so->solo_graph[slot] && so->solo_graph_key[slot][0] == K &&
                so->solo_graph_key[slot][1] == g.grid) {
                exec = so->solo_graph[slot];
            } else {
                if ((s = capture_chunk(g, K, &exec))) return s;
                if (so) {
                    if (so->solo_graph[slot]) (void)retire_graph(so->solo_graph[slot], st);
                    so->solo_graph[slot] = exec;
                    so->solo_graph_key[slot][0] = K;
                    so->solo_graph_key[slot][1] = g.grid;
                }
            }
            e = hipSuccess;
            for (int64_t r = 0; r < reps && e == hipSuccess; ++r) e = hipGraphLaunch(exec, st);
            if (!so) {
                const nd_status rs = retire_graph(exec, st);
                if (e == hipSuccess && rs) return rs;
            }
            if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
        }
        if (scratch) HIPC(hipFreeAsync(scratch, st));
    }
    for (int i = 0; i < count; ++i) nets[i]->ypar ^= (int)(steps[i] & 1);
    if (count == 1) return nets[0]->touch(st);
    // one event behind the whole batch, shared by its networks
    auto ev = std::make_shared<RunEvent>();
    HIPC(hipEventCreateWithFlags(&ev->ev, hipEventDisableTiming));
    HIPC(hipEventRecord(ev->ev, st));
    for (int i = 0; i < count; ++i) nets[i]->touch_shared(ev);
    return ND_OK;
}

// ------------------------------------------------- runs that allocate nothing
// nd_run_batch_noalloc keeps the descriptor tables, the per-group work counts and
// the work maps in `scratch`, one fixed array per GPU, instead of memory taken per
// call.  Layout: ND_NOALLOC_MAX_NETS descriptors, then ND_NOALLOC_MAX_NETS work
// counts, then ND_NOALLOC_MAX_WORK work items; a call lays its groups out one
// after the other.  Host code reaches the array only through the address
// hipGetSymbolAddress returns for the current device (the symbol itself is a
// host-side stand-in, not a device address).
constexpr size_t kNaDescBytes = ((size_t)ND_NOALLOC_MAX_NETS * sizeof(NetDesc) + 255) / 256 * 256;
constexpr size_t kNaCountBytes = ((size_t)ND_NOALLOC_MAX_NETS * sizeof(int) + 255) / 256 * 256;
constexpr size_t kNaBytes = kNaDescBytes + kNaCountBytes + (size_t)ND_NOALLOC_MAX_WORK * sizeof(int2);
static_assert(kNaBytes <= (size_t)ND_NOALLOC_SCRATCH_BYTES, "scratch layout exceeds its stated size");
static __device__ __align__(256) unsigned char scratch[ND_NOALLOC_SCRATCH_BYTES];

constexpr int kNaMaxDevices = 64;
static std::mutex g_na_mu;
static unsigned char* g_na_ptr[kNaMaxDevices] = {};

// The scratch array's device address on the current device, looked up once per
// device (with that device current) and kept.
static nd_status noalloc_scratch(unsigned char** out) {
    int dev = 0;
    HIPC(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNaMaxDevices) return fail(ND_ERR_UNSUPPORTED, "device %d beyond %d devices", dev, kNaMaxDevices);
    std::lock_guard<std::mutex> lk(g_na_mu);
    if (!g_na_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress (no-allocation scratch)");
        g_na_ptr[dev] = (unsigned char*)p;
    }
    *out = g_na_ptr[dev];
    return ND_OK;
}

// Work map of one group, built on the device from its descriptors (the same
// order as the host-built map of nd_run_batch: networks in turn, tiles ascending).
__global__ void k_noalloc_work(const NetDesc* D, int ndesc, int2* work, int* nwork) {
    __shared__ int off[ND_NOALLOC_MAX_NETS + 1];
    if (threadIdx.x == 0) {
        int o = 0;
        for (int q = 0; q < ndesc; ++q) {
            off[q] = o;
            o += D[q].G;
        }
        off[ndesc] = o;
        *nwork = o;
    }
    __syncthreads();
    for (int q = 0; q < ndesc; ++q) {
        const int G = off[q + 1] - off[q];
        for (int t = threadIdx.x; t < G; t += blockDim.x) work[off[q] + t] = make_int2(q, t);
    }
}

// nd_run_batch without allocation: the same groups, descriptors, work maps and
// kernels as run_nets, with the tables in `scratch`, descriptors passed to the
// device as kernel arguments and chunks launched eagerly (no graph capture).
// Fixed-size host arrays only; nothing is allocated on the success path.
static nd_status run_nets_noalloc(Net* const* nets, int count, const double* dt, const int64_t* steps,
                                  const nd_observe* obs, hipStream_t st) {
    if (count > ND_NOALLOC_MAX_NETS)
        return fail(ND_ERR_INVALID_ARG, "%d networks, the no-allocation run takes at most %d", count,
                    ND_NOALLOC_MAX_NETS);
    int64_t total_work = 0;
    for (int i = 0; i < count; ++i) {
        if (!nets[i]) return fail(ND_ERR_INVALID_ARG, "handle %d is NULL", i);
        if (!(dt[i] > 0.0) || !std::isfinite(dt[i])) return fail(ND_ERR_INVALID_ARG, "dt must be finite and > 0");
        if (steps[i] < 0) return fail(ND_ERR_INVALID_ARG, "steps must be >= 0");
        for (int k = 0; k < i; ++k)
            if (nets[k] == nets[i]) return fail(ND_ERR_INVALID_ARG, "a handle appears twice in one batch");
        if (steps[i] > 0) total_work += nets[i]->work_items();
    }
    if (total_work > ND_NOALLOC_MAX_WORK)
        return fail(ND_ERR_INVALID_ARG, "%lld work items, the no-allocation run takes at most %d",
                    (long long)total_work, ND_NOALLOC_MAX_WORK);
    unsigned char* base = nullptr;
    nd_status s = noalloc_scratch(&base);
    if (s) return s;
    for (int i = 0; i < count; ++i)
        if ((s = nets[i]->prepare_observe(steps[i], obs ? &obs[i] : nullptr, false))) return s;
    if (capturing(st))
        for (int i = 0; i < count; ++i) nets[i]->captured = true;
    NetDesc* descs = (NetDesc*)base;
    int* counts = (int*)(base + kNaDescBytes);
    int2* works = (int2*)(base + kNaDescBytes + kNaCountBytes);
    // groups of one kernel class, in order of first appearance
    const BatchClasses classes(nets, count, steps);
    Net::Class key[ND_NOALLOC_MAX_NETS];
    int grp[ND_NOALLOC_MAX_NETS];
    int ngroups = 0;
    for (int i = 0; i < count; ++i) {
        grp[i] = -1;
        if (steps[i] == 0) continue;
        const Net::Class k = classes.of(nets[i]);
        int gi = 0;
        while (gi < ngroups && key[gi] != k) ++gi;
        if (gi == ngroups) key[ngroups++] = k;
        grp[i] = gi;
    }
    int dnext = 0;
    int64_t wnext = 0;
    hipError_t e;
    for (int gi = 0; gi < ngroups; ++gi) {
        Group g(key[gi]);
        g.desc = descs + dnext;
        g.work = works + wnext;
        g.nwork = counts + gi;
        int64_t maxsteps = 0, nwork = 0, values = 0;
        const Net* n0 = nullptr;
        for (int i = 0; i < count && !n0; ++i)
            if (grp[i] == gi) n0 = nets[i];
        for (int q = 0; q < 2 * count; ++q) {  // the networks of part 0, then those of part 1
            const int i = q % count;
            const Net* n = nets[i];
            if (grp[i] != gi || n->part() != q / count) continue;
            if ((e = put_desc(g.desc + g.ndesc, n->run_desc(dt[i], steps[i]), st)) != hipSuccess)
                return hip_fail(e, "descriptor upload");
            ++g.ndesc;
            g.take(*n);
            nwork += n->work_items();
            values += n->prob.n * nvars_of(n->prob.model);
            maxsteps = std::max(maxsteps, steps[i]);
        }
        hipLaunchKernelGGL(k_noalloc_work, dim3(1), dim3(256), 0, st, g.desc, g.ndesc, g.work, g.nwork);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "work map");
        dnext += g.ndesc;
        wnext += nwork;
        const int cfg_grid = n0->cfg.grid;
        g.grid = cfg_grid > 0 ? (int)std::min<int64_t>(cfg_grid, nwork) : (int)nwork;
        // the chunking of nd_run_batch: one chunk, or chunks of K steps where that
        // call replays a captured K-step graph (here launched directly)
        const int K = std::max(1, n0->cfg.chunk);
        const bool eager = values >= kEagerValues;
        if (g.topo == ND_RING && g.tile < 0) {
            if ((s = run_resident(g, values / nvars_of(g.model), maxsteps, st))) return s;
        } else if (maxsteps <= K || !graphs_enabled() || eager) {
            if ((s = enqueue_chunk(g, (int)std::min<int64_t>(maxsteps, 1 << 30), st))) return s;
        } else {
            const int64_t reps = (maxsteps + K - 1) / K;
            for (int64_t r = 0; r < reps; ++r)
                if ((s = enqueue_chunk(g, K, st))) return s;
        }
    }
    for (int i = 0; i < count; ++i) {
        nets[i]->ypar ^= (int)(steps[i] & 1);
        if ((s = nets[i]->touch(st))) return s;
    }
    return ND_OK;
}

}  // namespace nd

// =================================================================== C ABI
using namespace nd;

extern "C" {

nd_status nd_create(const nd_problem* p, nd_handle* out) {
    if (!out) return fail(ND_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    nd_status s = validate_problem(p);
    if (s) return s;
    Net* n = new (std::nothrow) Net();
    if (!n) return fail(ND_ERR_OUT_OF_MEMORY, "host allocation failed");
    if ((s = n->create(p))) {
        delete n;
        return s;
    }
    *out = reinterpret_cast<nd_handle>(n);
    return ND_OK;
}

nd_status nd_footprint(const nd_problem* p, int64_t* bytes) {
    if (!bytes) return fail(ND_ERR_INVALID_ARG, "bytes is NULL");
    nd_status s = validate_problem(p);
    if (s) return s;
    if (p->topo == ND_LINKS) {  // malformed rows show up while compressing
        LinksCompressed lc;
        if ((s = compress_links(p->n, p->row_ptr, p->col, &lc))) return s;
    }
    *bytes = footprint_bytes(p, config_for(p));
    return ND_OK;
}

static Net* as_net(nd_handle h) { return reinterpret_cast<Net*>(h); }

nd_status nd_set_state(nd_handle h, const double* y, int64_t len, int32_t on_device, void* stream) {
    Net* n = as_net(h);
    if (!n || !y) return fail(ND_ERR_INVALID_ARG, "NULL handle or state");
    const int64_t want = nvars_of(n->prob.model) * n->prob.n;
    if (len != want) return fail(ND_ERR_INVALID_ARG, "state length %lld, expected %lld", (long long)len, (long long)want);
    hipStream_t st = (hipStream_t)stream;
    HIPC(hipMemcpyAsync(n->tmpl.y[n->ypar], y, len * 8, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, st));
    // A new state starts with a clean status word: it takes the next number, which no
    // earlier run stores, instead of a launch that clears the word (2 us a call: 512
    // rings of 1,024 set and run 20.2 -> 19.2 ms, adaptively 10.6 -> 9.1 ms).  Graphs
    // replay without the host side of the run or of this call, so networks that take
    // part in one keep their number and get the launch (so do those out of numbers).
    if (capturing(st)) n->captured = true;
    if (n->captured || n->status_tag == INT32_MAX) {
        hipLaunchKernelGGL(k_clear_status, dim3(1), dim3(1), 0, st, n->status_dev);
        HIPC(hipGetLastError());
    } else {
        ++n->status_tag;
    }
    if (!on_device) HIPC(hipStreamSynchronize(st));
    return n->touch(st);
}

// After the work enqueued on st so far: ND_ERR_NUMERIC when a stage kernel
// flagged a non-finite state value in this network (synchronises st).
static nd_status sync_status(Net* n, hipStream_t st, const char* what) {
    HIPC(hipMemcpyAsync(n->status_host, n->status_dev, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIPC(hipStreamSynchronize(st));
    if (*n->status_host == n->status_tag)
        return fail(ND_ERR_NUMERIC, "%s: the state holds a non-finite value (a run produced NaN or Inf)", what);
    return ND_OK;
}

nd_status nd_get_state(nd_handle h, double* y, int64_t len, int32_t on_device, void* stream) {
    Net* n = as_net(h);
    if (!n || !y) return fail(ND_ERR_INVALID_ARG, "NULL handle or state");
    const int64_t want = nvars_of(n->prob.model) * n->prob.n;
    if (len != want) return fail(ND_ERR_INVALID_ARG, "state length %lld, expected %lld", (long long)len, (long long)want);
    hipStream_t st = (hipStream_t)stream;
    HIPC(hipMemcpyAsync(y, n->tmpl.y[n->ypar], len * 8, on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st));
    if (!on_device) return sync_status(n, st, "nd_get_state");
    return n->touch(st);
}

nd_status nd_run(nd_handle h, double dt, int64_t steps, const nd_observe* obs, void* stream) {
    Net* n = as_net(h);
    if (!n) return fail(ND_ERR_INVALID_ARG, "NULL handle");
    return run_nets(&n, 1, &dt, &steps, obs, (hipStream_t)stream);
}

nd_status nd_run_batch(const nd_handle* hs, int32_t count, const double* dt, const int64_t* steps,
                       const nd_observe* obs, void* stream) {
    if (!hs || !dt || !steps || count < 0) return fail(ND_ERR_INVALID_ARG, "bad batch arguments");
    std::vector<Net*> nets(count);
    for (int i = 0; i < count; ++i) nets[i] = as_net(hs[i]);
    return run_nets(nets.data(), count, dt, steps, obs, (hipStream_t)stream);
}

nd_status nd_run_batch_noalloc(const nd_handle* hs, int32_t count, const double* dt, const int64_t* steps,
                               const nd_observe* obs, void* stream) {
    if (!hs || !dt || !steps || count < 0) return fail(ND_ERR_INVALID_ARG, "bad batch arguments");
    if (count > ND_NOALLOC_MAX_NETS)
        return fail(ND_ERR_INVALID_ARG, "%d networks, the no-allocation run takes at most %d", count,
                    ND_NOALLOC_MAX_NETS);
    Net* nets[ND_NOALLOC_MAX_NETS];
    for (int i = 0; i < count; ++i) nets[i] = as_net(hs[i]);
    return run_nets_noalloc(nets, count, dt, steps, obs, (hipStream_t)stream);
}

nd_status nd_get_observables(nd_handle h, double* R, int64_t r_len, double* mean_vel, int64_t mv_len,
                             int32_t on_device, void* stream) {
    Net* n = as_net(h);
    if (!n) return fail(ND_ERR_INVALID_ARG, "NULL handle");
    hipStream_t st = (hipStream_t)stream;
    const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    if (R) {
        if (n->r_every <= 0) return fail(ND_ERR_INVALID_ARG, "the last run recorded no R");
        const int64_t want = n->last_steps / n->r_every + 1;
        if (r_len != want) return fail(ND_ERR_INVALID_ARG, "r_len %lld, expected %lld", (long long)r_len, (long long)want);
        HIPC(hipMemcpyAsync(R, n->R_dev, want * 8, kind, st));
    }
    if (mean_vel) {
        if (n->mv_start < 0) return fail(ND_ERR_INVALID_ARG, "the last run recorded no mean velocity");
        if (mv_len != n->prob.n) return fail(ND_ERR_INVALID_ARG, "mv_len must equal n");
        HIPC(hipMemcpyAsync(mean_vel, n->mv_dev, mv_len * 8, kind, st));
    }
    if (!on_device) return sync_status(n, st, "nd_get_observables");
    return n->touch(st);
}

nd_status nd_sync(nd_handle h, void* stream) {
    Net* n = as_net(h);
    if (!n) return fail(ND_ERR_INVALID_ARG, "NULL handle");
    return sync_status(n, (hipStream_t)stream, "nd_sync");
}

nd_status nd_destroy(nd_handle h) {
    Net* n = as_net(h);
    if (!n) return fail(ND_ERR_INVALID_ARG, "NULL handle");
    delete n;  // waits for the work enqueued for this network only
    return ND_OK;
}

nd_status nd_get_config(nd_handle h, nd_kernel_config* cfg) {
    Net* n = as_net(h);
    if (!n || !cfg) return fail(ND_ERR_INVALID_ARG, "NULL argument");
    *cfg = n->cfg;
    return ND_OK;
}

nd_status nd_set_config(nd_handle h, const nd_kernel_config* cfg) {
    Net* n = as_net(h);
    if (!n || !cfg) return fail(ND_ERR_INVALID_ARG, "NULL argument");
    if (cfg->grid < 0 || cfg->chunk < 1) return fail(ND_ERR_INVALID_ARG, "grid must be >= 0 and chunk >= 1");
    nd_kernel_config c = *cfg;
    const nd_problem& p = n->prob;
    if (p.topo == ND_RING) {
        RingLaunch L;
        if (!ring_select(p.model, p.precision, c.tile, &L))
            return fail(ND_ERR_INVALID_ARG, "no ring kernel for tile %d", c.tile);
        if (c.tile < 0 && -c.tile < p.n)
            return fail(ND_ERR_INVALID_ARG, "a resident ring needs n <= %d", -c.tile);
    } else if (p.topo == ND_CUBE3D) {
        const int h = (int)p.radius;
        if (c.tile < 1 || c.tile_y < 1 || c.tile_z < 1)
            return fail(ND_ERR_INVALID_ARG, "cube tile extents must be >= 1");
        c.tile = (int32_t)std::min<int64_t>(c.tile, p.n1);
        c.tile_y = (int32_t)std::min<int64_t>(c.tile_y, p.n2);
        c.tile_z = (int32_t)std::min<int64_t>(c.tile_z, p.n3);
        if ((c.tile + 2 * h) * (c.tile_y + 2 * h) > 1024)
            return fail(ND_ERR_INVALID_ARG, "cube tile: (tile+2h)*(tile_y+2h) must be <= 1024");
    } else if (p.topo == ND_BALL3D || p.topo == ND_DISK2D) {
        const int P = (int)p.radius, pz = ball_pz(p.topo, p.radius);
        if (c.tile < 1 || c.tile_y < 1 || c.tile_z < 1)
            return fail(ND_ERR_INVALID_ARG, "ball tile extents must be >= 1");
        c.tile = (int32_t)std::min<int64_t>(c.tile, p.n1);
        c.tile_y = (int32_t)std::min<int64_t>(c.tile_y, p.n2);
        c.tile_z = (int32_t)std::min<int64_t>(c.tile_z, p.n3);
        if (c.block == kBallScatterBlock) {
            if (p.topo != ND_BALL3D || !ball_scatter_available(P))
                return fail(ND_ERR_INVALID_ARG, "block %d (plane-scatter ball) is not built for this radius or topology",
                            kBallScatterBlock);
        } else if (c.block != 256 && c.block != 1024) {
            c.block = 1024;
        }
        const int rows = 4 * (c.block / 64);
        const size_t sm = c.block == kBallScatterBlock ? ball_scatter_smem_bytes(P, c.tile, c.tile_y)
                                                       : ball_smem_bytes(P, pz, c.tile, c.tile_y);
        if (c.tile + 2 * P > 64 || c.tile_y + 2 * P > rows || c.tile * c.tile_y > c.block || sm > kBallSmemMax)
            return fail(ND_ERR_INVALID_ARG, "ball tile: need tile+2P <= 64, tile_y+2P <= 4*block/64, "
                                            "tile*tile_y <= block and the prefix planes within LDS");
    } else if (p.topo == ND_LINKS) {
        if (c.tile != kLinksRows) return fail(ND_ERR_INVALID_ARG, "links work items hold %d rows (tile must be %d)",
                                              kLinksRows, kLinksRows);
    } else {
        // 256 for every size too: configurations written when all networks had 256 rows
        if (c.tile != 256 && c.tile != csr_rows(p.n))
            return fail(ND_ERR_INVALID_ARG, "CSR work items of this network hold %d rows (tile must be %d or 256)",
                        csr_rows(p.n), csr_rows(p.n));
        if (c.tile_y < 2 || c.tile_y > 16 || (c.tile_y & (c.tile_y - 1)))
            return fail(ND_ERR_INVALID_ARG, "CSR edges per thread must be 2, 4, 8 or 16");
    }
    return n->apply_config(c);
}

const char* nd_status_str(nd_status s) {
    switch (s) {
        case ND_OK: return "ok";
        case ND_ERR_INVALID_ARG: return "invalid argument";
        case ND_ERR_OUT_OF_MEMORY: return "out of device memory";
        case ND_ERR_DEVICE: return "device error";
        case ND_ERR_NOT_READY: return "not ready";
        case ND_ERR_NUMERIC: return "non-finite value";
        case ND_ERR_UNSUPPORTED: return "unsupported";
        default: return "unknown status";
    }
}

const char* nd_last_error(void) { return g_err.c_str(); }

}  // extern "C"
