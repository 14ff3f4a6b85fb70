// gd_resident.h -- the stencil solve of fields that fit the chip's registers (gd_resident.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "gd_internal.h"
#include "gdecon.h"

namespace gdres {

// How a field is cut into boxes, one per workgroup.
struct Plan {
    int kc, kz;          // columns per thread, points per column
    int64_t rows;        // rows (y) per box; 3D: planes per box kz
    int64_t nby, nbz;    // boxes along y and z (2D: nbz = 1)
    int64_t W;           // boxes per field
    bool f0_lds;         // BiCGSTAB: f0 is in LDS,
    int64_t f0_ofs;      // from this element
    size_t lds;          // bytes of the box with its halo
};

// The plan for a batch of one grid, or false where only the streaming solver
// can take it: a row is longer than the threads can hold, a box of one row does
// not fit LDS, or the field needs more boxes than the GPU has CUs.
bool plan(int solver, int ndim, int64_t nx, int64_t ny, int64_t nz, int tsize, int64_t batch, int ncu, Plan *p);
// whether the plan is expected to be no slower than the streaming solver
bool faster(int solver, int ndim, int64_t nx, int64_t ny, int64_t nz, int tsize, int64_t batch, int ncu, const Plan &p);

// scratch: vec_bytes of the caller's workspace, first `field_bytes` of them the exchange buffer
int solve(int solver, const gd_grid *g, const Plan &p, double hw, const void *ubar, void *u, const gd_opts *o,
          int32_t max_replace, int64_t wait_ticks, int ncu, void *scratch, size_t field_bytes, size_t vec_bytes,
          gd_info *info, hipStream_t st);
// whether `vec_bytes` of scratch are enough for this batch
bool scratch_ok(const Plan &p, int64_t batch, int ncu, size_t field_bytes, size_t vec_bytes);

}  // namespace gdres
