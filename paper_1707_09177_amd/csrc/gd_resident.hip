// gd_resident.hip -- plan and launch of the register-resident stencil solve.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "gd_resident.h"
#include "gd_resident_kernel.h"

namespace gdres {

using gd::fail;

constexpr size_t kLdsMax = 158 * 1024;  // of 160 KB per CU, the reductions' share kept free

const void *kernels_f32_2d(int solver, const Plan &p);
const void *kernels_f32_3d(int solver, const Plan &p);
const void *kernels_f64_2d(int solver, const Plan &p);
const void *kernels_f64_3d(int solver, const Plan &p);

__global__ void k_res_prep(uint64_t *slot, int64_t nslot, uint32_t *flag, int64_t nflag, uint32_t *abort) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, n = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = t; i < nslot; i += n) slot[i] = 0;
    for (int64_t i = t; i < nflag; i += n) flag[i] = 0;
    if (t == 0) abort[0] = abort[kEnded] = 0;
}

const void *kernel_of(int dtype, int ndim, int solver, const Plan &p) {
    if (dtype == GD_F32) return ndim == 2 ? kernels_f32_2d(solver, p) : kernels_f32_3d(solver, p);
    return ndim == 2 ? kernels_f64_2d(solver, p) : kernels_f64_3d(solver, p);
}

// ---- the rule: resident or streamed, and in which boxes
//
// A batch is solved in rounds of as many fields as fit the CUs at once, and a
// round's time depends on the points per thread and the exchanges, not on how
// full the boxes are.  So fields that fill their boxes badly, or leave CUs
// without a field, lose against the streaming solver in large batches (10
// passes, resident and streamed: 8 x 160^3 FP32 Van Cittert, 189 boxes, one field
// at a time, 2525 and 1545 us; 51 x 623 x 1240 FP64 steepest descent, 156 boxes,
// 6130 and 5017), and small fields in short columns against the same fields in
// full ones (1312 x 15 x 24 x 45 FP64 Van Cittert, 8 boxes and 4, 3212 and 1948).
// Both times are estimated from the tables below (us, 256 CUs) for solves of
// kPasses passes.  Of 670 timed solves of random shapes and batches (300 to 6 M
// points per field, up to 48 M in all) five took more than 1.1 times the better
// choice's time.

constexpr double kPasses = 8;
// A pass of a round of fields of 17 to 64 (2D) or 65 to 128 boxes (3D), by points
// per thread (4, 8, 16, and 12 or 24), and a round's start and end
constexpr double kPass[4][2][4] = {{{4.9, 6.1, 7.2, 0}, {7, 10, 12, 21}},               // Van Cittert, 2D and 3D
                                   {{7.1, 9.7, 10.5, 17.5}, {10.1, 15, 17.9, 27}},      // CG
                                   {{13.5, 18.5, 24, 0}, {18.9, 27.5, 34.5, 0}},        // BiCGSTAB
                                   {{7, 8.4, 9.7, 0}, {10.1, 14.5, 17.3, 27}}};         // steepest descent
constexpr double kEnds[2][4] = {{17, 23, 28, 70}, {20, 32, 44, 105}};

int64_t fields_at_once(const Plan &p, int ncu) {
    const int64_t cap = std::min<int64_t>(ncu, gdcl::kMaxW);
    return p.W == 1 ? ncu : cap / p.W;
}

double resident_us(int solver, int ndim, const Plan &p, int64_t batch, int ncu) {
    const int points = p.kc * p.kz, by = points == 4 ? 0 : points == 8 ? 1 : points == 16 ? 2 : 3;
    const int64_t at_once = fields_at_once(p, ncu), rounds = (batch + at_once - 1) / at_once;
    // one box exchanges nothing; more boxes are more words to collect and, in 3D, more neighbours elsewhere
    // (2D boxes of four long rows: more of a box is boundary)
    const double rows = p.kc * p.kz == 8 && p.kc == 2 ? 1.2 : 1.0;
    const double share = ndim == 2 ? rows * (p.W == 1 ? 0.42 : p.W <= 16 ? 0.95 : p.W <= 64 ? 1.0 : 1.05)
                                   : (p.W == 1 ? 0.38 : p.W <= 16 ? 0.73 : p.W <= 64 ? 0.9 : p.W <= 128 ? 1.0 : 1.08);
    return (double)rounds * ((p.W == 1 ? 0.55 : share) * kEnds[ndim - 2][by] + kPasses * share * kPass[solver][ndim - 2][by]);
}

// The streaming solver: the field accesses at 4.1 TB/s or the waves' steps (a
// row of a tile in 2D, four rows in 3D; ns, FP32 and FP64), and the grid barriers
double streamed_us(int solver, int ndim, int64_t nx, int64_t ny, int64_t nz, int tsize, int64_t batch) {
    // accesses as measured at that rate: 3D tiles read their halo rows again
    constexpr double accesses[2][4][2] = {{{4, 4}, {8, 7.4}, {14, 14}, {6, 5.2}},
                                          {{5.2, 4.5}, {9.5, 8.6}, {17, 15.5}, {7.5, 6.2}}};
    constexpr double barriers[4] = {17, 34, 51, 34};
    constexpr double step[4][2][2] = {
        {{0.45, 0.52}, {0.86, 1.0}}, {{0.85, 1.05}, {1.72, 2.25}}, {{1.35, 1.9}, {4.0, 5.3}}, {{0.73, 0.83}, {1.5, 1.65}}};
    const int64_t lanes = 64 * (nx % (16 / tsize) == 0 ? 16 / tsize : 1), segs = (nx + lanes - 1) / lanes;
    const double b = (double)batch, rows = (double)(ndim == 2 ? ny : nz), halo = 1.0 + 2.0 / rows;
    const double steps = b * (double)segs * rows * halo * (double)(ndim == 2 ? 1 : ny >= 4 ? (ny + 3) / 4 : ny);
    const double bytes = b * (double)(nx * ny * nz) * tsize * accesses[ndim - 2][solver][tsize == 8];
    return (kPasses + 1.5) * (std::max(bytes / 4.1e6, steps * step[solver][ndim - 2][tsize == 8] * 1e-3) + barriers[solver]);
}

bool faster(int solver, int ndim, int64_t nx, int64_t ny, int64_t nz, int tsize, int64_t batch, int ncu, const Plan &p) {
    // streamed where it leads clearly: the streaming estimate leaves out how its
    // tiles divide, which matters less for the many small fields of one box
    const double lead = p.W == 1 ? 0.88 : 0.78;
    return resident_us(solver, ndim, p, batch, ncu) * lead <= streamed_us(solver, ndim, nx, ny, nz, tsize, batch);
}

bool plan(int solver, int ndim, int64_t nx, int64_t ny, int64_t nz, int tsize, int64_t batch, int ncu, Plan *p) {
    const int64_t cap = std::min<int64_t>(ncu, gdcl::kMaxW);
    if (nx > 2 * kThreads || nx * ny > int64_t(0x7fffffff) || nx * ny * nz > int64_t(0x7fffffff)) return false;
    const int kc = nx > kThreads ? 2 : 1;
    if (ndim == 3 && kc > 1) return false;
    auto shape = [&](int kz, bool f0_lds) {
        auto box = [&](int64_t rows) {  // elements in LDS, even
            const int64_t lines = ndim == 3 ? (kz + 2) * (rows + 2) : (rows + kz - 1) / kz * kz + 2;
            return (lines * (nx + 2) + 1) & ~int64_t(1);
        };
        auto lds = [&](int64_t rows) {
            const int64_t f0 = f0_lds ? kThreads * kc * kz : 0;
            return (size_t)((box(rows) + f0) * tsize);
        };
        int64_t rows = std::min<int64_t>(ny, kThreads * kc / nx * (ndim == 3 ? 1 : kz));
        while (rows > 1 && lds(rows) > kLdsMax) --rows;
        if (lds(rows) > kLdsMax) return false;
        p->kc = kc;
        p->kz = kz;
        p->nby = (ny + rows - 1) / rows;
        p->rows = (ny + p->nby - 1) / p->nby;  // even boxes
        p->nby = (ny + p->rows - 1) / p->rows;
        p->nbz = ndim == 3 ? (nz + kz - 1) / kz : 1;
        p->W = p->nby * p->nbz;
        p->f0_lds = f0_lds;
        p->f0_ofs = box(p->rows);
        p->lds = lds(p->rows);
        return p->W <= cap;
    };
    const int some = points(tsize) / kc, most = most_points(solver, ndim, tsize) / kc;
    const bool full = (solver == GD_BICGSTAB && shape(some, true)) || shape(some, false) ||
                      (most > some && shape(most, false));
    // Short columns while that leaves room for 16 fields at a time: a pass's
    // work within a workgroup then takes a quarter of the time, and the
    // exchanges and reductions take the same.  Not where a batch that does not
    // fit at once takes so many more rounds then that full columns are faster.
    const Plan whole = *p;
    if (kc == 1 && shape(kSmallZ, false) && p->W <= kSmallW &&
        (!full || batch <= fields_at_once(*p, ncu) ||
         resident_us(solver, ndim, *p, batch, ncu) <= resident_us(solver, ndim, whole, batch, ncu)))
        return true;
    *p = whole;
    return full;
}

struct Control {
    int64_t nclusters;
    size_t slot, flag, abort, total;
};
Control control_of(const Plan &p, int64_t batch, int ncu) {
    Control c;
    c.nclusters = p.W == 1 ? batch : std::min<int64_t>(batch, fields_at_once(p, ncu));
    c.slot = 0;
    c.flag = gd::align_up((size_t)c.nclusters * 2 * p.W * gdcl::kWords * sizeof(uint64_t), 256);
    c.abort = c.flag + (size_t)c.nclusters * p.W * 128;
    c.total = c.abort + 256;
    return c;
}

bool scratch_ok(const Plan &p, int64_t batch, int ncu, size_t field_bytes, size_t vec_bytes) {
    if (batch > (int64_t(1) << 30)) return false;
    return p.W == 1 || gd::align_up(field_bytes, 256) + control_of(p, batch, ncu).total <= vec_bytes;
}

int solve(int solver, const gd_grid *g, const Plan &p, double hw, const void *ubar, void *u, const gd_opts *o,
          int32_t max_replace, int64_t wait_ticks, int ncu, void *scratch, size_t field_bytes, size_t vec_bytes,
          gd_info *info, hipStream_t st) {
    (void)vec_bytes;
    Params P;
    const Control c = control_of(p, g->batch, ncu);
    char *ctl = (char *)scratch + gd::align_up(field_bytes, 256);
    P.ubar = ubar;
    P.u = u;
    P.xch = scratch;
    P.slot = (uint64_t *)(ctl + c.slot);
    P.flag = (uint32_t *)(ctl + c.flag);
    P.abort = (uint32_t *)(ctl + c.abort);
    P.info = info;
    P.hist = o->history;
    P.nx = (int32_t)g->n[0];
    P.ny = (int32_t)g->n[1];
    P.nz = g->ndim == 3 ? (int32_t)g->n[2] : 1;
    P.npts = (int64_t)P.nx * P.ny * P.nz;
    P.batch = g->batch;
    P.nclusters = c.nclusters;
    P.rows = (int32_t)p.rows;
    P.nby = (int32_t)p.nby;
    P.f0_ofs = (int32_t)p.f0_ofs;
    P.hist_stride = (int64_t)o->max_iter + 1;
    P.wait_ticks = wait_ticks;
    P.hw = hw;
    P.tol = o->tol;
    P.W = (int32_t)p.W;
    P.init = o->init;
    P.norm_ref = o->norm_ref;
    P.max_iter = o->max_iter;
    P.max_replace = max_replace;
    const void *kern = kernel_of(g->dtype, g->ndim, solver, p);
    if (p.W > 1) {
        hipLaunchKernelGGL(k_res_prep, dim3(32), dim3(256), 0, st, P.slot, (int64_t)((c.flag - c.slot) / 8), P.flag,
                           (int64_t)((c.abort - c.flag) / 4), P.abort);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(GD_EHIP, "prep launch: %s", hipGetErrorString(e));
    }
    void *args[] = {&P};
    const hipError_t e = hipLaunchKernel(kern, dim3((unsigned)(c.nclusters * p.W)), dim3(kThreads), args, p.lds, st);
    if (e != hipSuccess) return fail(GD_EHIP, "solve launch: %s", hipGetErrorString(e));
    gd_launch_info li{};
    li.variant = 10000 + g->ndim * 100 + p.kc;
    li.vw = 1;
    li.R = (int32_t)p.rows;
    li.L = p.kz;
    li.tiles = p.W * g->batch;
    li.blocks = c.nclusters * p.W;
    li.waves = li.blocks * kWaves;
    gd::note_launch(li);
    return GD_OK;
}

}  // namespace gdres
