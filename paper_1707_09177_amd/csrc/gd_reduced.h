// gd_reduced.h -- the differential-filter solve on wavenumber classes (gd_reduced.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "gd_internal.h"
#include "gdecon.h"

namespace gdred {

// Which wavenumbers share a class: those that differ in the signs of k_y and
// k_z, and on a square (2D) or a cube (3D) in the order of the components.
enum FoldKind : int { FOLD_SIGNS = 0, FOLD_SQUARE = 1, FOLD_CUBE = 2 };

struct Fold {
    int64_t nx, ny, nz, nxs;  // logical grid, stored reals per row
    int64_t field;            // stored reals per field
    int64_t hx, hy, hz;       // n / 2 + 1 (hz = 1 in 2D)
    int64_t K;                // classes
    double inv_kc2;
    int32_t kind, pad;
};

Fold fold_of(int ndim, int64_t nx, int64_t ny, int64_t nz, int64_t nxs, double inv_kc2);
// whether solve() takes a solve from this start with `scratch` bytes
bool fits(const Fold &f, int solver, int init, int64_t batch, size_t scratch, int ncu);
// UB: stored spectra of ubar; U: stored spectra of u (output).  resume: fields
// that miss the tolerance in the storage type are flagged in state / sync for
// the general solver.
int solve(int solver, int dtype, const Fold &f, int64_t batch, double hw, const gd_opts *o, int32_t max_replace,
          int64_t wait_ticks, int ncu, const void *UB, void *U, void *scratch, gd_info *info, gd::State *state,
          gd::Sync *sync, bool resume, hipStream_t st);

}  // namespace gdred
