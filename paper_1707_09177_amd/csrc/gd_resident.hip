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

bool plan(int solver, int ndim, int64_t nx, int64_t ny, int64_t nz, int tsize, int ncu, Plan *p) {
    const int64_t cap = std::min<int64_t>(ncu, gdcl::kMaxW);
    if (nx > 2 * kThreads || nx * ny > int64_t(0x7fffffff) || nx * ny * nz > int64_t(0x7fffffff)) return false;
    // The plan depends on the field alone, so a field's result does not
    // depend on the batch it is solved in.
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
    // Short columns while that leaves room for 16 fields at a time: a pass's
    // work within a workgroup then takes a quarter of the time, and the
    // exchanges and reductions take the same.
    const int some = points(tsize) / kc, most = most_points(solver, ndim, tsize) / kc;
    return (kc == 1 && shape(kSmallZ, false) && p->W <= kSmallW) || (solver == GD_BICGSTAB && shape(some, true)) ||
           shape(some, false) || (most > some && shape(most, false));
}

struct Control {
    int64_t nclusters;
    size_t slot, flag, abort, total;
};
Control control_of(const Plan &p, int64_t batch, int ncu) {
    Control c;
    c.nclusters = p.W == 1 ? batch : std::min<int64_t>(batch, std::min<int64_t>(ncu, gdcl::kMaxW) / p.W);
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
