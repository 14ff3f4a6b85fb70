// gd_reduced.hip -- the differential-filter solve on wavenumber classes.
//
// G_hat depends on |k|^2 only, and from u0 = ubar or u0 = 0 every vector of
// Algorithms 1-4 is a polynomial in G times ubar: at a wavenumber k it is
// ubar_hat(k) times a factor that only depends on G_hat(k).  Wavenumbers that
// share |k|^2 therefore share their factor, and an inner product only needs
// the sum of |ubar_hat|^2 over each group of them.  So the solve runs on one
// real number per class,
//     x_j = sqrt(sum over the class of |ubar_hat|^2),   G x_j = G_hat_j x_j,
// whose inner products equal the field's, and u_hat(k) = (u_j / x_j)
// ubar_hat(k) for every k of class j.  A class holds (k_x, +-k_y, +-k_z), both
// real and imaginary parts, and on square 2D and cubic 3D grids also the
// permutations of the components: 4 (2D), 8 (2D square or 3D) or 48 (3D cube)
// stored reals per class.
//
// What bounds it: the general path streams 8 to 15 field accesses per pass
// through HBM and pays a grid barrier per sweep.  Here a field's classes stay
// in registers (up to 16 per thread, 512 threads per workgroup) for the whole
// solve and a sweep is a few FP64 operations per class and one all-reduce of
// at most three FP64 sums, so a pass costs its reductions.
// Everything on the classes is FP64, whatever the storage type.
// Measured, whole call with its FFTs: 8 x 1024^2 FP32 BiCGSTAB to 1e-2 at
// gamma = 0.1 1920 -> 250 us, 64^3 FP64 CG 672 -> 89 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "gd_cluster.h"
#include "gd_kernels.h"
#include "gd_reduced.h"

namespace gdred {

using gd::fail;

using gdcl::kMaxW;
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
// classes per thread, so that a solver's vectors (three, four or BiCGSTAB's
// five, in FP64) fit the 256 registers of two waves per SIMD without spilling
constexpr int max_e(int solver) { return solver == GD_BICGSTAB ? 12 : 16; }
constexpr int kExpand = 256;   // threads of the expand kernel

// What a field's solve leaves for the expand pass.
struct Rec {
    double r_ref, r0, rr;
    int32_t iters, status, verify, start;
};

struct Ctl {
    uint32_t abort;
    uint32_t pad[63];
};

struct Params {
    Fold f;
    double *x;        // [batch][K]: x_j, then the factors u_j / x_j
    double *lam;      // [K]: G_hat_j
    uint64_t *slot;   // [cluster][2][W][6] tagged words of the all-reduce
    Ctl *ctl;
    Rec *rec;         // [batch]
    uint32_t *done;   // [batch]: expand workgroups finished
    double *part;     // [batch][chunks]: partial sums of the true residual
    int64_t batch, nclusters, nslots;
    int32_t W, chunks;
    int32_t init, norm_ref, max_iter, max_replace, resume;
    int64_t hist_stride;
    double tol, hw;
    double *hist;
    gd_info *info;
    int64_t wait_ticks;
    gd::State *st;    // the general solver's state (resume != 0)
    gd::Sync *sync;
};

// ---------------------------------------------------------------- classes
__device__ __forceinline__ int64_t class_of(const Fold &f, int a, int b, int c) {
    if (f.kind == FOLD_SIGNS) return ((int64_t)c * f.hy + b) * f.hx + a;
    if (f.kind == FOLD_SQUARE) {
        const int64_t hi = max(a, b), lo = min(a, b);
        return hi * (hi + 1) / 2 + lo;
    }
    const int64_t hi = max(a, max(b, c)), lo = min(a, min(b, c)), mid = (int64_t)a + b + c - hi - lo;
    return hi * (hi + 1) * (hi + 2) / 6 + mid * (mid + 1) / 2 + lo;
}

__device__ __forceinline__ double ghat(const Fold &f, int a, int b, int c) {
    const double k2 = (double)((int64_t)a * a + (int64_t)b * b + (int64_t)c * c);
    return 1.0 / (1.0 + k2 * f.inv_kc2);
}

// |scale coefficient|^2 summed over the signs of k_y and k_z at (kx, |ky|, |kz|)
template <typename T>
__device__ __forceinline__ double power(const Fold &f, const T *F, double scale, int kx, int ky, int kz) {
    double s = 0.0;
    const int ys = (ky == 0 || 2 * ky == f.ny) ? 1 : 2, zs = (kz == 0 || 2 * kz == f.nz) ? 1 : 2;
    for (int zi = 0; zi < zs; ++zi)
        for (int yi = 0; yi < ys; ++yi) {
            const int64_t row = (int64_t)(zi ? f.nz - kz : kz) * f.ny + (yi ? f.ny - ky : ky);
            const T *p = F + row * f.nxs + 2 * kx;
            const double re = scale * (double)p[0], im = scale * (double)p[1];
            s += re * re + im * im;
        }
    return s;
}

// x_j and G_hat_j from the stored spectrum; also clears what the launches
// that follow count in.  Bound by reading the spectrum once.  A wave takes
// 64 x-adjacent classes where only signs fold, 8 x 8 classes of a square and
// 4 x 4 x 4 of a cube: every permuted read is then a run of 8 or 4 adjacent
// coefficients instead of a column.
template <typename T>
__global__ __launch_bounds__(256) void k_fold(const T *X, Params P) {
    const Fold f = P.f;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
    if (blockIdx.y == 0) {
        for (int64_t i = t; i < P.nslots; i += nt) P.slot[i] = 0;
        for (int64_t i = t; i < P.batch; i += nt) {
            P.done[i] = 0;
            P.rec[i] = Rec{};  // what a solve that is ended by the wait bound leaves of its fields
        }
        if (t == 0) P.ctl->abort = 0;
    }
    const int lane = threadIdx.x & 63;
    const int64_t wv = t >> 6;
    int a, b, c = 0;
    if (f.kind == FOLD_SIGNS) {
        const int64_t segs = (f.hx + 63) / 64;
        a = (int)(wv % segs) * 64 + lane;
        const int64_t q = wv / segs;
        b = (int)(q % f.hy);
        const int64_t cc = q / f.hy;
        if (a >= f.hx || cc >= f.hz) return;
        c = (int)cc;
    } else if (f.kind == FOLD_SQUARE) {
        const int64_t n = (f.hx + 7) / 8;
        const int64_t ta = wv / n, tb = wv % n;
        if (ta >= n || tb > ta) return;
        a = (int)ta * 8 + (lane >> 3);
        b = (int)tb * 8 + (lane & 7);
        if (a >= f.hx || b > a) return;
    } else {
        const int64_t n = (f.hx + 3) / 4;
        const int64_t ta = wv / (n * n), tb = wv / n % n, tc = wv % n;
        if (ta >= n || tb > ta || tc > tb) return;
        a = (int)ta * 4 + (lane >> 4);
        b = (int)tb * 4 + ((lane >> 2) & 3);
        c = (int)tc * 4 + (lane & 3);
        if (a >= f.hx || b > a || c > b) return;
    }
    const int64_t fld = blockIdx.y;
    const T *F = X + fld * f.field;
    auto at = [&](int kx, int ky, int kz) { return power(f, F, 1.0, kx, ky, kz); };
    double s = at(a, b, c), unscale = 1.0;
    if (f.kind == FOLD_SQUARE) {
        if (a != b) s += at(b, a, 0);
    } else if (f.kind == FOLD_CUBE) {
        // the distinct permutations of (a, b, c), a >= b >= c
        if (b != c) s += at(a, c, b);
        if (a != b) s += at(b, a, c);
        if (a != b && b != c) s += at(b, c, a) + at(c, a, b) + at(c, b, a);
        if (a != b && b == c) s += at(b, b, a);
        if (a == b && b != c) s += at(c, a, b);
    }
    // FP64 coefficients whose squares leave the range (a class's part in the
    // solve's sums may still be in it: the mean has no residual): summed again,
    // scaled, all permutations in a loop (in the path above, the scale and a
    // second round doubled the registers: 105 x 256 x 64 x 2 344 -> 486 us)
    if (sizeof(T) == 8 && !(s >= 0x1p-900 && s <= 0x1p900)) {
        const double scale = s < 1.0 ? 0x1p600 : 0x1p-600;
        unscale = s < 1.0 ? 0x1p-600 : 0x1p600;
        const int perms = f.kind == FOLD_SIGNS ? 1 : f.kind == FOLD_SQUARE ? 2 : 6;
        s = 0.0;
        int kx = a, ky = b, kz = c;
#pragma unroll 1
        for (int q = 0; q < perms; ++q) {
            s += power(f, F, scale, kx, ky, kz);
            int t = kx;  // swap the first two, or (every second time) the last two
            if (q & 1) t = kz, kz = ky, ky = t;
            else kx = ky, ky = t;
        }
        if (perms == 2 && a == b) s /= 2.0;  // each distinct one, as often as it came
        if (perms == 6) s /= a == b && b == c ? 6.0 : (a == b || b == c) ? 2.0 : 1.0;
    }
    const int64_t j = class_of(f, a, b, c);
    P.x[fld * f.K + j] = unscale * sqrt(s);
    if (fld == 0) P.lam[j] = ghat(f, a, b, c);
}

// ------------------------------------------------------------------ solve
// One solve per cluster of W workgroups; clusters take fields in turn.  The
// scalars, the guards and the stopping rule are those of the persistent
// solve kernel (update_scalars); every thread holds them.
template <int SOLVER, int E>
__global__ __launch_bounds__(kThreads) void k_red_solve(Params P) {
    __shared__ gdcl::Shared<kWaves> sh;
    const int cl = blockIdx.x / P.W, wg = blockIdx.x % P.W;
    const int64_t K = P.f.K;
    gdcl::Cluster cluster;
    cluster.slot = P.slot + (int64_t)cl * 2 * P.W * gdcl::kWords;
    cluster.abort = &P.ctl->abort;
    cluster.wait_ticks = P.wait_ticks;
    cluster.W = P.W;
    cluster.wg = wg;
    cluster.seq = 0;
    if (threadIdx.x == 0) sh.abort = 0;
    double lam[E], r[E], u[E];
    double p[SOLVER == GD_CG || SOLVER == GD_BICGSTAB ? E : 1], f0[SOLVER == GD_BICGSTAB ? E : 1];
    const int64_t j0 = (int64_t)wg * E * kThreads + threadIdx.x;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int64_t j = j0 + (int64_t)e * kThreads;
        lam[e] = j < K ? P.lam[j] : 0.0;
    }
    for (int64_t fld = cl; fld < P.batch; fld += P.nclusters) {
        double *x = P.x + fld * K;
        double *hist = P.hist && wg == 0 && threadIdx.x == 0 ? P.hist + fld * P.hist_stride : nullptr;
        double s0[2] = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int64_t j = j0 + (int64_t)e * kThreads;
            const double xv = j < K ? x[j] : 0.0, rv = xv - lam[e] * xv;
            u[e] = P.init == GD_INIT_UBAR ? xv : 0.0;
            r[e] = P.init == GD_INIT_UBAR ? rv : xv;
            const double q = P.norm_ref == GD_REF_UBAR ? xv : rv;
            s0[0] += r[e] * r[e];
            s0[1] += q * q;
            if constexpr (SOLVER == GD_CG || SOLVER == GD_BICGSTAB) p[e] = r[e];
            if constexpr (SOLVER == GD_BICGSTAB) f0[e] = r[e];
        }
        if (!gdcl::all_sum<2>(cluster, sh, s0)) return;
        double rr = P.hw * s0[0], rho = rr;
        const double r0 = sqrt(rr);
        const double r_ref = (P.init == GD_INIT_UBAR && P.norm_ref == GD_REF_R0UBAR) ? r0 : sqrt(P.hw * s0[1]);
        const double thr = P.tol > 0.0 ? P.tol * r_ref : 0.0;
        int iters = 0, status = -1, verify = 0;  // status < 0: still iterating
        if (hist) hist[0] = r0;
        // the stopping test after n passes with residual norm rn
        auto stop = [&](double rn, int n) {
            if (!isfinite(rn)) status = GD_NONFINITE;
            else if (rn == 0.0 || (P.tol > 0.0 && rn <= thr)) {
                status = GD_CONVERGED;
                verify = n > 0 && P.tol > 0.0;
            } else if (n >= P.max_iter) status = GD_MAXITER;
            return status >= 0;
        };
        if (!isfinite(r_ref)) status = GD_NONFINITE;
        else if (r_ref == 0.0) status = GD_ZERO_REF;
        else stop(r0, 0);
        while (status < 0) {
            if constexpr (SOLVER == GD_VANCITTERT) {
                double s[1] = {0.0};
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    u[e] += r[e];
                    r[e] -= lam[e] * r[e];
                    s[0] += r[e] * r[e];
                }
                if (!gdcl::all_sum<1>(cluster, sh, s)) return;
                rr = P.hw * s[0];
                ++iters;
                if (hist) hist[iters] = sqrt(rr);
                stop(sqrt(rr), iters);
            } else if constexpr (SOLVER == GD_STEEPEST_DESCENT || SOLVER == GD_CG) {
                double s[1] = {0.0};
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const double d = SOLVER == GD_CG ? p[e] : r[e];
                    s[0] += d * (lam[e] * d);
                }
                if (!gdcl::all_sum<1>(cluster, sh, s)) return;
                const double pd = P.hw * s[0];
                if (!isfinite(pd)) {
                    status = GD_NONFINITE;
                    break;
                }
                if (pd == 0.0) {
                    status = GD_BREAKDOWN_RHO;
                    break;
                }
                const double alpha = rr / pd;
                s[0] = 0.0;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const double d = SOLVER == GD_CG ? p[e] : r[e];
                    u[e] += alpha * d;
                    r[e] -= alpha * (lam[e] * d);
                    s[0] += r[e] * r[e];
                }
                if (!gdcl::all_sum<1>(cluster, sh, s)) return;
                const double rn = P.hw * s[0];
                ++iters;
                if (hist) hist[iters] = sqrt(rn);
                if (!stop(sqrt(rn), iters)) {
                    if constexpr (SOLVER == GD_CG) {
                        const double beta = rn / rr;
#pragma unroll
                        for (int e = 0; e < E; ++e) p[e] = r[e] + beta * p[e];
                    }
                }
                rr = rn;
            } else {
                double s[1] = {0.0};
#pragma unroll
                for (int e = 0; e < E; ++e) s[0] += f0[e] * (lam[e] * p[e]);
                if (!gdcl::all_sum<1>(cluster, sh, s)) return;
                const double fq = P.hw * s[0];
                if (!isfinite(fq)) {
                    status = GD_NONFINITE;
                    break;
                }
                if (fq == 0.0) {
                    status = GD_BREAKDOWN_RHO;
                    break;
                }
                const double alpha = rho / fq;
                double b[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    r[e] -= alpha * (lam[e] * p[e]);  // s
                    const double t = lam[e] * r[e];
                    b[0] += r[e] * t;
                    b[1] += t * t;
                    b[2] += r[e] * r[e];
                }
                if (!gdcl::all_sum<3>(cluster, sh, b)) return;
                const double st = P.hw * b[0], tt = P.hw * b[1], ss = P.hw * b[2];
                // a sweep that ends here leaves u untouched
                if (!isfinite(st) || !isfinite(tt) || !isfinite(ss)) {
                    status = GD_NONFINITE;
                    break;
                }
                const bool half = ss == 0.0 || sqrt(ss) <= thr;
                if (!half && tt == 0.0) {
                    status = GD_BREAKDOWN_OMEGA;
                    break;
                }
                const double omega = half ? 0.0 : st / tt;
                double c[2] = {0.0, 0.0};
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    u[e] += alpha * p[e] + omega * r[e];
                    r[e] -= omega * (lam[e] * r[e]);
                    c[0] += f0[e] * r[e];
                    c[1] += r[e] * r[e];
                }
                if (!gdcl::all_sum<2>(cluster, sh, c)) return;
                const double fr = P.hw * c[0];
                rr = P.hw * c[1];
                ++iters;
                if (hist) hist[iters] = sqrt(rr);
                if (half) {
                    if (!isfinite(rr)) status = GD_NONFINITE;
                    else {
                        status = GD_CONVERGED;
                        verify = P.tol > 0.0;
                    }
                    break;
                }
                if (stop(sqrt(rr), iters)) break;
                if (!isfinite(fr)) status = GD_NONFINITE;
                else if (fr == 0.0) status = GD_BREAKDOWN_RHO;
                else {
                    const double beta = (alpha / omega) * (fr / rho);
                    rho = fr;
#pragma unroll
                    for (int e = 0; e < E; ++e) p[e] = r[e] + beta * (p[e] - omega * (lam[e] * p[e]));
                }
            }
        }
        // the factors u_j / x_j; a class without content, and every class of a
        // field that did not finish a pass (it may not be finite), keeps the start's
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int64_t j = j0 + (int64_t)e * kThreads;
            if (j < K) {
                const double xv = x[j];
                x[j] = iters == 0 || xv == 0.0 ? (P.init == GD_INIT_UBAR ? 1.0 : 0.0) : u[e] / xv;
            }
        }
        if (wg == 0 && threadIdx.x == 0) {
            Rec o;
            o.r_ref = r_ref;
            o.r0 = r0;
            o.rr = rr;
            o.iters = iters;
            o.status = status;
            o.verify = verify;
            o.start = P.init;
            P.rec[fld] = o;
        }
    }
}

// ----------------------------------------------------------------- expand
// u_hat = factor(class) ubar_hat in the storage type, and the true residual
// ||ubar - G u|| of the stored coefficients in FP64; the workgroup that
// completes a field writes its info record.  A field whose recursive residual
// met the tolerance and whose true residual does not (the rounding of the
// storage type) is handed to the general solver, which replaces its residual
// and goes on.  Bound by what it computes per coefficient (G_hat's FP64 division,
// the index's divisions, 64-bit class numbers) with one load in flight: 349 us
// for 16 x 2048^2 FP32, 1.5 TB/s of the one read and the one write.
template <typename T>
__global__ __launch_bounds__(kExpand) void k_expand(const T *UB, T *U, Params P) {
    typedef T V2 __attribute__((ext_vector_type(2)));
    const Fold f = P.f;
    const int64_t fld = blockIdx.y;
    const double *fac = P.x + fld * f.K;
    const uint32_t nxh = (uint32_t)(f.nxs / 2), ncol = (uint32_t)(f.field / 2);
    const V2 *B = reinterpret_cast<const V2 *>(UB + fld * f.field);
    V2 *O = reinterpret_cast<V2 *>(U + fld * f.field);
    const uint32_t per = (ncol + P.chunks - 1) / P.chunks;
    const uint32_t i0 = blockIdx.x * per, i1 = min(ncol, i0 + per);
    double acc = 0.0;
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += kExpand) {
        const uint32_t row = i / nxh;
        const int kx = (int)(i - row * nxh);
        V2 o = {T(0), T(0)};
        if (kx < f.hx) {
            const int ky = (int)(row % (uint32_t)f.ny), kz = (int)(row / (uint32_t)f.ny);
            const int a = kx, b = min(ky, (int)f.ny - ky), c = min(kz, (int)f.nz - kz);
            const V2 v = B[i];
            const double m = fac[class_of(f, a, b, c)], g = ghat(f, a, b, c);
            if (m != 0.0) {  // 0 is 0 for coefficients that are not finite too
                o[0] = T(m * (double)v[0]);
                o[1] = T(m * (double)v[1]);
            }
            const double d0 = (double)v[0] - g * (double)o[0], d1 = (double)v[1] - g * (double)o[1];
            acc += d0 * d0 + d1 * d1;
        }
        O[i] = o;
    }
    __shared__ double red[kExpand / 64];
    __shared__ int s_last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    acc = gd::wave_sum(acc);
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kExpand / 64; ++w) s += red[w];
        __hip_atomic_store(&P.part[fld * P.chunks + blockIdx.x], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gd::wait_vm_stores();
        const uint32_t n = __hip_atomic_fetch_add(&P.done[fld], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = n == (uint32_t)P.chunks - 1;
    }
    __syncthreads();
    if (!s_last || threadIdx.x >= 64) return;
    double s = 0.0;
    for (int k = lane; k < P.chunks; k += 64) s += gd::ld_f64(&P.part[fld * P.chunks + k]);
    s = gd::wave_sum(s);
    if (lane != 0) return;
    const Rec q = P.rec[fld];
    const double rt = sqrt(P.hw * s);
    int status = q.status;
    if (q.verify) {
        if (!isfinite(rt)) status = GD_NONFINITE;
        else if (rt <= P.tol * q.r_ref) status = GD_CONVERGED;
        else if (q.iters >= P.max_iter) status = GD_MAXITER;
        else status = GD_STAGNATED;
    }
    gd_info out;
    out.iters = q.iters;
    out.status = status;
    out.r_ref = q.r_ref;
    out.r0 = q.r0;
    out.r_final = sqrt(q.rr);
    out.r_true = rt;
    out.start = q.start;
    out.replaced = 0;
    if (P.ctl->abort) out.status = GD_TIMEOUT;
    else if (status == GD_STAGNATED && P.resume && P.max_replace > 0) {
        gd::State *S = &P.st[fld];
        S->iters = q.iters;
        S->r_ref = q.r_ref;
        S->r0 = q.r0;
        S->rr = q.rr;
        S->start = q.start;
        S->done = 0;
        S->tknown = 0;
        S->replace = 1;
        gd::count(&P.sync->live.active, 1);
        gd::count(&P.sync->live.replace, 1);
    }
    P.info[fld] = out;
}

template <int SOLVER>
const void *solve_ptr(int e) {
    switch (e) {
    case 1: return (const void *)k_red_solve<SOLVER, 1>;
    case 4: return (const void *)k_red_solve<SOLVER, 4>;
    default: return (const void *)k_red_solve<SOLVER, max_e(SOLVER)>;
    }
}

const void *kernel_of(int solver, int e) {
    switch (solver) {
    case GD_VANCITTERT: return solve_ptr<GD_VANCITTERT>(e);
    case GD_CG: return solve_ptr<GD_CG>(e);
    case GD_BICGSTAB: return solve_ptr<GD_BICGSTAB>(e);
    default: return solve_ptr<GD_STEEPEST_DESCENT>(e);
    }
}

Fold fold_of(int ndim, int64_t nx, int64_t ny, int64_t nz, int64_t nxs, double inv_kc2) {
    Fold f;
    f.nx = nx;
    f.ny = ny;
    f.nz = nz;
    f.nxs = nxs;
    f.field = nz * ny * nxs;
    f.hx = nx / 2 + 1;
    f.hy = ny / 2 + 1;
    f.hz = ndim == 3 ? nz / 2 + 1 : 1;
    f.inv_kc2 = inv_kc2;
    if (ndim == 2 && nx == ny) {
        f.kind = FOLD_SQUARE;
        f.K = f.hx * (f.hx + 1) / 2;
    } else if (ndim == 3 && nx == ny && ny == nz) {
        f.kind = FOLD_CUBE;
        f.K = f.hx * (f.hx + 1) * (f.hx + 2) / 6;
    } else {
        f.kind = FOLD_SIGNS;
        f.K = f.hx * f.hy * f.hz;
    }
    return f;
}

struct Layout {
    int e;                    // classes per thread
    int64_t W, nclusters, chunks;
    size_t lam, slot, ctl, rec, done, part, total;
};

// Workgroups per field and the scratch layout; false where the classes of one
// field do not fit the registers of the GPU's CUs at once.
bool layout_of(const Fold &f, int solver, int64_t batch, int ncu, Layout *L) {
    L->e = 1;
    while (L->e < max_e(solver) && f.K > (int64_t)L->e * kThreads) L->e = L->e == 1 ? 4 : max_e(solver);
    L->W = (f.K + (int64_t)L->e * kThreads - 1) / ((int64_t)L->e * kThreads);
    const int64_t cap = std::min<int64_t>(ncu, kMaxW);
    if (L->W > cap || batch > 65535 || f.field / 2 > int64_t(0x7fffffff)) return false;
    L->nclusters = L->W == 1 ? batch : std::min<int64_t>(batch, cap / L->W);
    L->chunks = std::max<int64_t>(1, std::min<int64_t>(512, f.field / 2 / 2048));
    size_t off = (size_t)batch * f.K * sizeof(double);
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = gd::align_up(off + bytes, 256);
        return o;
    };
    off = gd::align_up(off, 256);
    L->lam = take((size_t)f.K * sizeof(double));
    L->slot = take((size_t)L->nclusters * 2 * L->W * gdcl::kWords * sizeof(uint64_t));
    L->ctl = take(sizeof(Ctl));
    L->rec = take((size_t)batch * sizeof(Rec));
    L->done = take((size_t)batch * sizeof(uint32_t));
    L->part = take((size_t)batch * L->chunks * sizeof(double));
    L->total = off;
    return true;
}

template <typename T>
int run(Params &P, const Layout &L, const void *kern, const T *UB, T *U, hipStream_t st) {
    const Fold &f = P.f;
    int64_t waves;
    if (f.kind == FOLD_SIGNS) waves = (f.hx + 63) / 64 * f.hy * f.hz;
    else if (f.kind == FOLD_SQUARE) waves = (f.hx + 7) / 8 * ((f.hx + 7) / 8);
    else waves = (f.hx + 3) / 4 * ((f.hx + 3) / 4) * ((f.hx + 3) / 4);
    hipLaunchKernelGGL(k_fold<T>, dim3((unsigned)((waves + 3) / 4), (unsigned)P.batch), dim3(256), 0, st, UB, P);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(GD_EHIP, "class fold launch: %s", hipGetErrorString(e));
    void *args[] = {&P};
    e = hipLaunchKernel(kern, dim3((unsigned)(L.nclusters * L.W)), dim3(kThreads), args, 0, st);
    if (e != hipSuccess) return fail(GD_EHIP, "class solve launch: %s", hipGetErrorString(e));
    hipLaunchKernelGGL(k_expand<T>, dim3((unsigned)L.chunks, (unsigned)P.batch), dim3(kExpand), 0, st, UB, U, P);
    e = hipGetLastError();
    return e == hipSuccess ? GD_OK : fail(GD_EHIP, "expand launch: %s", hipGetErrorString(e));
}

// The rule: starts from ubar or zero (other starts are not multiples of
// ubar_hat), a field's classes fit the chip, and the scratch fits the general
// solver's vectors (it does not for a few points per field).
bool fits(const Fold &f, int solver, int init, int64_t batch, size_t scratch, int ncu) {
    Layout L;
    return (init == GD_INIT_UBAR || init == GD_INIT_ZERO) && layout_of(f, solver, batch, ncu, &L) && L.total <= scratch;
}

int solve(int solver, int dtype, const Fold &f, int64_t batch, double hw, const gd_opts *o, int32_t max_replace,
          int64_t wait_ticks, int ncu, const void *UB, void *U, void *scratch, gd_info *info, gd::State *state,
          gd::Sync *sync, bool resume, hipStream_t st) {
    Layout L;
    if (!layout_of(f, solver, batch, ncu, &L)) return fail(GD_EINVAL, "too many wavenumber classes");
    char *w = (char *)scratch;
    Params P;
    P.f = f;
    P.x = (double *)w;
    P.lam = (double *)(w + L.lam);
    P.slot = (uint64_t *)(w + L.slot);
    P.ctl = (Ctl *)(w + L.ctl);
    P.rec = (Rec *)(w + L.rec);
    P.done = (uint32_t *)(w + L.done);
    P.part = (double *)(w + L.part);
    P.batch = batch;
    P.nclusters = L.nclusters;
    P.nslots = L.nclusters * 2 * L.W * gdcl::kWords;
    P.W = (int32_t)L.W;
    P.chunks = (int32_t)L.chunks;
    P.init = o->init;
    P.norm_ref = o->norm_ref;
    P.max_iter = o->max_iter;
    P.max_replace = max_replace;
    P.resume = resume ? 1 : 0;
    P.hist_stride = (int64_t)o->max_iter + 1;
    P.tol = o->tol;
    P.hw = hw;
    P.hist = o->history;
    P.info = info;
    P.wait_ticks = wait_ticks;
    P.st = state;
    P.sync = sync;
    const void *kern = kernel_of(solver, L.e);
    gd_launch_info li{};
    li.vw = li.R = 1;
    li.L = L.e;
    li.tiles = batch * L.W;
    li.blocks = L.nclusters * L.W;
    li.waves = li.blocks * kWaves;
    gd::note_launch(li);
    return dtype == GD_F32 ? run<float>(P, L, kern, (const float *)UB, (float *)U, st)
                           : run<double>(P, L, kern, (const double *)UB, (double *)U, st);
}

}  // namespace gdred
