// gd_resident_kernel.h -- the stencil solve of fields that fit the chip's registers.
//
// The persistent solve kernel (gd_kernels.h) streams every vector through HBM
// once per sweep and separates sweeps by a grid barrier over all workgroups:
// 4 to 15 field accesses and 1 to 3 barriers (about 17 us each) per pass.  A
// field of up to 4 M points (FP32 BiCGSTAB; 2 M in FP64) fits the registers of
// 256 CUs together with the solver's vectors.  Here a field is cut into
// boxes, one per workgroup of 1024 threads, and a thread keeps its points of
// u, r, p, q and f0 in registers from the first sweep to the last.  Per
// application of G a box's vector goes to LDS, and only the box's boundary
// rows go through memory to the neighbours, ordered by one flag per
// workgroup; inner products are all-reduced among the field's workgroups
// (gd_cluster.h).  A field of one box exchanges nothing: its solve is one
// launch with LDS barriers only.
//
// What bounds it: the stencil's LDS reads and the latency of exchanges and
// reductions (2 to 3 us each; 5 per BiCGSTAB pass, 3 per CG pass, 2 per Van
// Cittert pass); a batch runs as many fields at a time as fit.  Measured, 5
// passes, streamed -> resident: 64^2 FP64 BiCGSTAB 285 -> 47 us, 16 x 256^2
// FP32 CG 342 -> 55, 8 x 1024^2 FP32 BiCGSTAB 1146 -> 322, 16 x 2048^2 FP32
// BiCGSTAB 5016 -> 2915 (16 rounds) and Van Cittert 1752 -> 1171, 3 x 128^3
// FP32 BiCGSTAB 1742 -> 400, FP64 CG on three fields of 97 x 100 x 90 points (z, y,
// x; 130 boxes, three rounds) 769 -> 327 and of 90 x 100 x 97 (120, two) 702 -> 223.
//
// Layout: a column of a box is one x and KZ consecutive points of the march
// axis (y in 2D, z in 3D): a thread marches its columns with a three-value
// window, reading the in-plane neighbours from LDS.  2D boxes are whole rows,
// stacked bands of KZ rows; 3D boxes are `rows` whole rows of KZ planes.
// Arithmetic and order of operations per point are those of gd_ops.h; only
// the order in which inner products are summed differs.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "gd_cluster.h"
#include "gd_kernels.h"

namespace gdres {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

// Points per thread (KC columns of KZ points): a solver's vectors take 32 to 64
// of the 128 registers of four waves per SIMD.  With addresses and temporaries
// Van Cittert and steepest descent then spill up to 6 registers, CG 3 to 42 and
// BiCGSTAB 21 to 125 (60 in two columns of 8 points, FP32), the kernels of 12 and
// 24 points 125 to 181; columns of 4 points none.  With 32 points a Van Cittert pass on 1024^2 took 2.4 times as long as with
// 16, CG with 24 1.7 times as long.  BiCGSTAB's fifth vector, f0, is in LDS where a thread
// has more than kSmallZ points and the box leaves room (8 x 1024^2 FP32: 320 us
// for 5 passes, in registers 378).  CG and, in 3D, Van Cittert and steepest
// descent take 24 points where a field fits in no other way (160^3 FP32 CG: 249 us
// for 5 passes, streamed 923).  Two columns only where a 2D row is longer
// than the threads.
constexpr int kSmallZ = 4;   // a short column for fields that need few workgroups:
constexpr int kSmallW = 16;  // at most this many
constexpr int points(int tsize) { return tsize == 4 ? 16 : 8; }
constexpr int most_points(int solver, int ndim, int tsize) {
    return solver != GD_BICGSTAB && (solver == GD_CG || ndim == 3) ? points(tsize) * 3 / 2 : points(tsize);
}

constexpr int kEnded = 32;   // word of the abort line that counts ended workgroups

struct Params {
    const void *ubar;
    void *u;
    void *xch;          // exchange buffer: boundary points at their place in the field
    uint64_t *slot;     // [cluster][2][W][kWords]
    uint32_t *flag;     // [cluster][W][32]: exchanges published
    uint32_t *abort;    // [0] set when a wait exceeded its bound, [kEnded] workgroups that have ended
    gd_info *info;
    double *hist;
    int64_t npts, batch, nclusters, hist_stride, wait_ticks;
    double hw, tol;
    int32_t nx, ny, nz, rows, nby;
    int32_t f0_ofs;     // of f0 in LDS, in elements
    int32_t W, init, norm_ref, max_iter, max_replace;
};

template <typename T>
__device__ __forceinline__ void st_agent(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T ld_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// v as a value the compiler takes as new: without it, the addresses and
// predicates of every point of a column are computed once before the
// iteration and kept, several times the registers that the vectors need
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// F0_LDS: BiCGSTAB's f0 in LDS
template <typename T, int NDIM, int SOLVER, int KC, int KZ, bool F0_LDS>
__global__ __launch_bounds__(kThreads) void k_resident(Params P) {
    extern __shared__ __attribute__((aligned(16))) unsigned char box_lds[];
    T *box = reinterpret_cast<T *>(box_lds);
    __shared__ gdcl::Shared<kWaves> sh;
    constexpr bool HAS_P = SOLVER == GD_CG || SOLVER == GD_BICGSTAB, HAS_Q = SOLVER == GD_BICGSTAB;
    constexpr int KP = HAS_P ? KC : 1, KQ = HAS_Q ? KC : 1, KF = HAS_Q && !F0_LDS ? KC : 1;
    const int tid = threadIdx.x;
    const int cl = blockIdx.x / P.W, wg = blockIdx.x % P.W;
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    // the box: rows [y0, y1); 3D: planes [z0, z1)
    const int iby = wg % P.nby, ibz = wg / P.nby, nbz = P.W / P.nby;
    const int y0 = iby * P.rows, y1 = min(ny, y0 + P.rows);
    const int z0 = NDIM == 3 ? ibz * KZ : 0, z1 = NDIM == 3 ? min(nz, z0 + KZ) : 1;
    const int by = y1 - y0, bz = z1 - z0;
    // LDS: 2D rows, row 0 the halo row before the box; 3D [plane][by + 2] rows.
    // A row is nx + 2 points: x at x + 1, the periodic neighbours at the ends,
    // so that a point's three x neighbours are one address.  Room for whole
    // columns: one past the box's end reads unused points.
    // SJ: one step along the march axis in LDS, SG: in the field
    const int RS = nx + 2;
    const int SJ = NDIM == 3 ? (by + 2) * RS : RS;
    const int SG = NDIM == 3 ? nx * ny : nx;
    const int bands = NDIM == 3 ? by : (by + KZ - 1) / KZ;
    // this thread's columns: left neighbour of the point before the first in
    // LDS, place in the field, valid points (0: no column)
    int off[KC], gofs[KC], nv[KC];
    auto column = [&](int k, int &x, int &b) {  // also where the loops need x or the band again
        const int c = fresh(tid) + kThreads * k;
        b = c / nx;
        x = c - b * nx;
        return b < bands;
    };
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        int x, b;
        const bool ok = column(k, x, b);
        if (!ok) x = b = 0;
        if constexpr (NDIM == 3) {
            off[k] = (b + 1) * RS + x;
            gofs[k] = (z0 * ny + y0 + b) * nx + x;
            nv[k] = ok ? bz : 0;
        } else {
            off[k] = b * KZ * RS + x;
            gofs[k] = (y0 + b * KZ) * nx + x;
            nv[k] = ok ? min(KZ, by - b * KZ) : 0;
        }
    }
    gdcl::Cluster C;
    C.slot = P.slot + (int64_t)cl * 2 * P.W * gdcl::kWords;
    C.abort = P.abort;
    C.wait_ticks = P.wait_ticks;
    C.W = P.W;
    C.wg = wg;
    C.seq = 0;
    uint32_t xseq = 0;  // exchanges published
    uint32_t *flags = P.flag + (int64_t)cl * P.W * 32;
    if (tid == 0) sh.abort = 0;
    __syncthreads();

    // f(std::true_type or false_type, n) for the n points of column k: true
    // where every column that this wave holds is whole (no test per point:
    // half the instructions of a sweep), else f tests j < n itself
    auto column_do = [&](int k, auto &&f) {
        const int n = fresh(nv[k]);
        if (__ballot(n != 0 && n != KZ) == 0) {
            if (n != 0) f(std::true_type{}, KZ);
        } else {
            f(std::false_type{}, n);
        }
    };
    // f(k, j, place in the field) at this thread's points
    auto points_do = [&](auto &&f) {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int n = fresh(nv[k]);
            int g = fresh(gofs[k]);
#pragma unroll
            for (int j = 0; j < KZ; ++j) {
                if (j < n) f(k, j, g);
                g += SG;
            }
        }
    };
    // point x of a row in LDS, with the periodic copies
    auto put = [&](T *row, int x, T v) {
        row[x + 1] = v;
        if (x == 0) row[nx + 1] = v;
        if (x == nx - 1) row[0] = v;
    };
    // the box's halo into LDS, four points of a thread at a time:
    // v = get(y, z, x) in the field
    // i / nx = i by_nx >> 32 (i nx < 2^32, nx > 1)
    const uint32_t by_nx = nx > 1 ? (uint32_t)(((1ull << 32) + nx - 1) / nx) : 0;
    auto fill_halo = [&](auto &&get) {
        const int full = 2 * (by + 2);  // 3D: rows of the planes before and after
        const int n = (NDIM == 3 ? full + 2 * bz : 2) * nx;
        for (int i0 = tid; i0 < n; i0 += 4 * kThreads) {
            T v[4];
            T *dst[4];
            int xs[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int i = min(i0 + m * kThreads, n - 1);
                const int h = nx > 1 ? (int)__umulhi((uint32_t)i, by_nx) : i, x = i - h * nx;
                int ly, lz = 0;
                if constexpr (NDIM == 3) {
                    const int e = h - full;
                    lz = h < by + 2 ? 0 : (e < 0 ? bz + 1 : 1 + (e >> 1));
                    ly = h < by + 2 ? h : (e < 0 ? h - (by + 2) : ((e & 1) ? by + 1 : 0));
                } else {
                    ly = h == 0 ? 0 : by + 1;
                }
                const int y = y0 + ly - 1, z = NDIM == 3 ? z0 + lz - 1 : 0;
                xs[m] = x;
                dst[m] = box + lz * SJ + ly * RS;
                v[m] = get(y < 0 ? y + ny : (y >= ny ? y - ny : y), z < 0 ? z + nz : (z >= nz ? z - nz : z), x);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) put(dst[m], xs[m], v[m]);
        }
    };
    // this thread's points of v into LDS
    auto put_box = [&](const T (&v)[KC][KZ]) {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            column_do(k, [&](auto whole, int n) {
                T *o = box + fresh(off[k]) + 1;
#pragma unroll
                for (int j = 0; j < KZ; ++j) {
                    o += SJ;
                    if (whole.value || j < n) *o = v[k][j];
                }
            });
            int x, b;
            if (column(k, x, b) && (x == 0 || x == nx - 1)) {
                const int m = fresh(nv[k]);
                T *o = box + fresh(off[k]) + 1;
#pragma unroll
                for (int j = 0; j < KZ; ++j) {
                    o += SJ;
                    if (j < m) {
                        if (x == 0) o[nx] = v[k][j];
                        if (x == nx - 1) o[-nx] = v[k][j];
                    }
                }
            }
        }
    };
    // own points of a field vector into v and LDS, and its halo into LDS: for
    // vectors that no workgroup writes meanwhile
    auto load_box = [&](const T *src, T (&v)[KC][KZ]) {
        points_do([&](int k, int j, int g) { v[k][j] = src[g]; });
        put_box(v);
        fill_halo([&](int y, int z, int x) { return src[(z * ny + y) * nx + x]; });
        __syncthreads();
    };
    // v into LDS and its boundary to the neighbours; their boundaries into the halo
    auto exchange = [&](T *xch, const T (&v)[KC][KZ]) -> bool {
        if (C.W > 1) {
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                int x, b;
                column(k, x, b);
                const int n = fresh(nv[k]);
                T *g = xch + fresh(gofs[k]);
                // 2D: the first row of the first band, the last of the last;
                // 3D: the rows at the box's y ends, elsewhere the first and last plane
                const bool all = NDIM == 3 && (b == 0 || b == by - 1);
                const bool lo = NDIM == 3 || b == 0, hi = NDIM == 3 || b == bands - 1;
                if (all || lo || hi) {
#pragma unroll
                    for (int j = 0; j < KZ; ++j) {
                        if (j < n && (all || (lo && j == 0) || (hi && j == n - 1))) st_agent(g, v[k][j]);
                        g += SG;
                    }
                }
            }
        }
        put_box(v);
        if (C.W == 1) {
            __syncthreads();
            fill_halo([&](int y, int z, int x) { return box[(NDIM == 3 ? (z + 1) * SJ : 0) + (y + 1) * RS + x + 1]; });
            __syncthreads();
            return true;
        }
        ++xseq;
        gd::wait_vm_stores();
        __syncthreads();
        if (tid == 0) st_agent(&flags[wg * 32], xseq);
        if (tid < (NDIM == 3 ? 8 : 2)) {  // wait for the neighbours (diagonal ones too in 3D)
            int ay, az = 0;
            if constexpr (NDIM == 3) {
                const int d = tid + (tid >= 4);  // 0 .. 8 without the centre
                ay = d % 3 - 1;
                az = d / 3 - 1;
            } else {
                ay = 2 * tid - 1;
            }
            const int n = (ibz + az + nbz) % nbz * P.nby + (iby + ay + P.nby) % P.nby;
            const int64_t t0 = wall_clock64();
            while ((int32_t)(ld_agent(&flags[n * 32]) - xseq) < 0) {
                if (ld_agent(P.abort) || wall_clock64() - t0 > P.wait_ticks) {
                    st_agent(P.abort, 1u);
                    sh.abort = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        __syncthreads();
        if (sh.abort) return false;
        fill_halo([&](int y, int z, int x) { return ld_agent(xch + (z * ny + y) * nx + x); });
        __syncthreads();
        return true;
    };
    // f(k, j, S, G S) at this thread's points in arithmetic A, S the vector in LDS
    auto filter = [&]<typename A>(A, auto &&f) {
#pragma unroll
        for (int k = 0; k < KC; ++k)
            column_do(k, [&](auto whole, int n) {
                const T *a = box + fresh(off[k]);
                A w0 = A(0), w1 = A(0), w2 = A(0), c0 = A(0), c1 = A(0);
                auto row = [&](const T *q) { return A(0.5) * A(q[1]) + A(0.25) * (A(q[0]) + A(q[2])); };
#pragma unroll
                for (int j = 0; j < KZ + 2; ++j) {
                    c0 = c1;
                    c1 = A(a[1]);
                    w0 = w1;
                    w1 = w2;
                    if constexpr (NDIM == 3) w2 = A(0.5) * row(a) + A(0.25) * (row(a - RS) + row(a + RS));
                    else w2 = row(a);
                    if (j >= 2)
                        if (whole.value || j - 2 < n) f(k, j - 2, c0, A(0.5) * w1 + A(0.25) * (w0 + w2));
                    a += SJ;
                }
            });
    };

    T r[KC][KZ], u[KC][KZ], p[KP][KZ], q[KQ][KZ], f0_reg[KF][KZ];
    T *f0_lds = box + P.f0_ofs + tid;
    auto f0 = [&](int k, int j) -> T & {
        if constexpr (F0_LDS) return f0_lds[(k * KZ + j) * kThreads];
        else return f0_reg[k][j];
    };
    bool ok = true;
    int64_t fld = cl;
    for (; fld < P.batch; fld += P.nclusters) {
        const T *ub = static_cast<const T *>(P.ubar) + fld * P.npts;
        T *uo = static_cast<T *>(P.u) + fld * P.npts;
        T *xch = static_cast<T *>(P.xch) + fld * P.npts;
        double *hist = P.hist && wg == 0 && tid == 0 ? P.hist + fld * P.hist_stride : nullptr;
        double r_ub = 0.0, r_ref = 0.0, r0 = 0.0, rr = 0.0, thr = 0.0, rho = 0.0, r_true = 0.0;
        double alpha = 1.0, beta = 0.0, omega = 1.0;
        int iters = 0, nrep = 0, status = -1;  // status < 0: still iterating
        int start = P.init == GD_INIT_WARM ? GD_INIT_GIVEN : P.init;
        bool first = true;
        // the stopping test after n passes with residual norm rn: whether the
        // true residual is to be checked
        bool verify = false;
        auto stop = [&](double rn, int n) {
            if (!isfinite(rn)) status = GD_NONFINITE;
            else if (rn == 0.0 || (P.tol > 0.0 && rn <= thr)) {
                if (n > 0 && P.tol > 0.0) verify = true;
                else status = GD_CONVERGED;
            } else if (n >= P.max_iter) status = GD_MAXITER;
        };
        // What the residual ubar - G u (FP64 arithmetic, into r) is taken for:
        // the ubar start's norm, the start's, the check of a met tolerance or
        // the exit's record
        enum { R_UBAR, R_START, R_VERIFY, R_EXIT };
        int what = R_UBAR;
        load_box(ub, u);
        for (;;) {
            double s2[2] = {0.0, 0.0};
            points_do([&](int k, int j, int g) { r[k][j] = ub[g]; });  // ubar, for the filter below
            filter(double(0), [&](int k, int j, double, double g) {
                const double v = double(r[k][j]), d = v - g;
                r[k][j] = T(d);
                s2[0] += d * d;
                s2[1] += v * v;
            });
            if (!(ok = gdcl::all_sum<2>(C, sh, s2))) break;
            const double rn = sqrt(P.hw * s2[0]);
            if (what == R_UBAR) {
                r_ub = rn;
                r_ref = P.norm_ref == GD_REF_UBAR ? sqrt(P.hw * s2[1]) : rn;
                rr = P.hw * s2[0];
                if (P.init == GD_INIT_ZERO) {
                    rr = P.hw * s2[1];
#pragma unroll
                    for (int k = 0; k < KC; ++k)
#pragma unroll
                        for (int j = 0; j < KZ; ++j) {
                            r[k][j] = u[k][j];
                            u[k][j] = T(0);
                        }
                } else if (P.init != GD_INIT_UBAR && start != GD_INIT_UBAR) {
                    what = R_START;
                    load_box(uo, u);
                    continue;
                }
            } else if (what == R_START) {
                if (P.init == GD_INIT_WARM && (!isfinite(rn) || !(rn < r_ub))) {
                    start = GD_INIT_UBAR;  // no better than the paper's start
                    what = R_UBAR;
                    load_box(ub, u);
                    continue;
                }
                rr = P.hw * s2[0];
            }
            if (what == R_UBAR || what == R_START) {
                r0 = sqrt(rr);
                thr = P.tol > 0.0 ? P.tol * r_ref : 0.0;
                if (hist) hist[0] = r0;
                if (!isfinite(r_ref)) status = GD_NONFINITE;
                else if (r_ref == 0.0) status = GD_ZERO_REF;
                else stop(r0, 0);
            } else {
                r_true = rn;
                if (what == R_EXIT) break;
                if (!isfinite(rn)) status = GD_NONFINITE;
                else if (rn <= P.tol * r_ref) status = GD_CONVERGED;
                else if (iters >= P.max_iter) status = GD_MAXITER;
                else if (nrep >= P.max_replace) status = GD_STAGNATED;
                if (status >= 0) break;
                // the residual is replaced by the true one (in r)
                ++nrep;
                rr = P.hw * s2[0];
            }
            // a (fresh) Krylov sequence from u and r
            rho = rr;
            alpha = omega = 1.0;
            beta = 0.0;
            first = true;
            verify = false;
            if constexpr (HAS_Q) {
#pragma unroll
                for (int k = 0; k < KC; ++k)
#pragma unroll
                    for (int j = 0; j < KZ; ++j) {
                        f0(k, j) = r[k][j];
                        q[k][j] = T(0);
                    }
            }
            if constexpr (HAS_P) {
#pragma unroll
                for (int k = 0; k < KC; ++k)
#pragma unroll
                    for (int j = 0; j < KZ; ++j) p[k][j] = T(0);
            }
            while (status < 0 && !verify) {
                if constexpr (SOLVER == GD_VANCITTERT) {
                    if (!(ok = exchange(xch, r))) break;
                    double s[1] = {0.0};
                    filter(T(0), [&](int k, int j, T c, T g) {
                        u[k][j] = u[k][j] + c;
                        r[k][j] = c - g;
                        s[0] += double(r[k][j]) * double(r[k][j]);
                    });
                    if (!(ok = gdcl::all_sum<1>(C, sh, s))) break;
                    rr = P.hw * s[0];
                    ++iters;
                    if (hist && iters <= P.max_iter) hist[iters] = sqrt(rr);
                    stop(sqrt(rr), iters);
                } else if constexpr (SOLVER == GD_CG || SOLVER == GD_STEEPEST_DESCENT) {
                    if constexpr (SOLVER == GD_CG) {
                        const T be = T(beta);
#pragma unroll
                        for (int k = 0; k < KC; ++k)
#pragma unroll
                            for (int j = 0; j < KZ; ++j) p[k][j] = first ? r[k][j] : r[k][j] + be * p[k][j];
                        if (!(ok = exchange(xch, p))) break;
                    } else {
                        if (!(ok = exchange(xch, r))) break;
                    }
                    first = false;
                    double s[1] = {0.0};
                    filter(T(0), [&](int, int, T c, T g) { s[0] += double(c) * double(g); });
                    if (!(ok = gdcl::all_sum<1>(C, sh, s))) break;
                    const double pd = P.hw * s[0];
                    if (!isfinite(pd)) {
                        status = GD_NONFINITE;
                        break;
                    }
                    if (pd == 0.0) {
                        status = GD_BREAKDOWN_RHO;
                        break;
                    }
                    alpha = (SOLVER == GD_CG ? rho : rr) / pd;
                    const T al = T(alpha);
                    s[0] = 0.0;
                    filter(T(0), [&](int k, int j, T c, T g) {
                        u[k][j] = u[k][j] + al * c;
                        r[k][j] = (SOLVER == GD_CG ? r[k][j] : c) - al * g;
                        s[0] += double(r[k][j]) * double(r[k][j]);
                    });
                    if (!(ok = gdcl::all_sum<1>(C, sh, s))) break;
                    rr = P.hw * s[0];
                    ++iters;
                    if (hist && iters <= P.max_iter) hist[iters] = sqrt(rr);
                    stop(sqrt(rr), iters);
                    beta = rr / rho;
                    rho = rr;
                } else {
                    const T be = T(beta), om0 = T(omega);
#pragma unroll
                    for (int k = 0; k < KC; ++k)
#pragma unroll
                        for (int j = 0; j < KZ; ++j)
                            p[k][j] = first ? r[k][j] : r[k][j] + be * (p[k][j] - om0 * q[k][j]);
                    first = false;
                    if (!(ok = exchange(xch, p))) break;
                    double s[1] = {0.0};
                    filter(T(0), [&](int k, int j, T, T g) {
                        q[k][j] = g;
                        s[0] += double(f0(k, j)) * double(g);
                    });
                    if (!(ok = gdcl::all_sum<1>(C, sh, s))) break;
                    const double fq = P.hw * s[0];
                    if (!isfinite(fq)) {
                        status = GD_NONFINITE;
                        break;
                    }
                    if (fq == 0.0) {
                        status = GD_BREAKDOWN_RHO;
                        break;
                    }
                    alpha = rho / fq;
                    const T al = T(alpha);
#pragma unroll
                    for (int k = 0; k < KC; ++k)
#pragma unroll
                        for (int j = 0; j < KZ; ++j) r[k][j] = r[k][j] - al * q[k][j];  // s
                    if (!(ok = exchange(xch, r))) break;
                    double b[3] = {0.0, 0.0, 0.0};
                    filter(T(0), [&](int, int, T c, T g) {
                        b[0] += double(c) * double(g);
                        b[1] += double(g) * double(g);
                        b[2] += double(c) * double(c);
                    });
                    if (!(ok = gdcl::all_sum<3>(C, sh, b))) break;
                    const double st = P.hw * b[0], tt = P.hw * b[1], ss = P.hw * b[2];
                    if (!isfinite(st) || !isfinite(tt) || !isfinite(ss)) {
                        status = GD_NONFINITE;
                        break;
                    }
                    const bool half = ss == 0.0 || sqrt(ss) <= thr;
                    if (!half && tt == 0.0) {
                        status = GD_BREAKDOWN_OMEGA;
                        break;
                    }
                    omega = half ? 0.0 : st / tt;
                    const T om = T(omega);
                    double c2[2] = {0.0, 0.0};
                    filter(T(0), [&](int k, int j, T c, T g) {
                        u[k][j] = u[k][j] + (al * p[k][j] + om * c);
                        r[k][j] = c - om * g;
                        c2[0] += double(f0(k, j)) * double(r[k][j]);
                        c2[1] += double(r[k][j]) * double(r[k][j]);
                    });
                    if (!(ok = gdcl::all_sum<2>(C, sh, c2))) break;
                    const double fr = P.hw * c2[0];
                    rr = P.hw * c2[1];
                    ++iters;
                    if (hist && iters <= P.max_iter) hist[iters] = sqrt(rr);
                    if (half) {
                        if (!isfinite(rr)) status = GD_NONFINITE;
                        else if (P.tol > 0.0) verify = true;
                        else status = GD_CONVERGED;
                    } else {
                        stop(sqrt(rr), iters);
                        if (status < 0 && !verify) {
                            if (!isfinite(fr)) status = GD_NONFINITE;
                            else if (fr == 0.0) status = GD_BREAKDOWN_RHO;
                            else {
                                beta = (alpha / omega) * (fr / rho);
                                rho = fr;
                            }
                        }
                    }
                }
            }
            if (!ok) break;
            what = status < 0 ? R_VERIFY : R_EXIT;
            if (!(ok = exchange(xch, u))) break;
        }
        if (!ok) break;
        points_do([&](int k, int j, int g) { __builtin_nontemporal_store(u[k][j], uo + g); });
        if (wg == 0 && tid == 0) {
            gd_info *out = P.info + fld;
            out->iters = iters;
            // not left in this L2: the mark below may come from another one
            st_agent(&out->status, (int32_t)status);
            out->r_ref = r_ref;
            out->r0 = r0;
            out->r_final = sqrt(rr);
            out->r_true = r_true;
            out->start = start;
            out->replaced = nrep;
        }
    }
    if (!ok && wg == 0 && tid == 0)
        for (; fld < P.batch; fld += P.nclusters) {
            st_agent(&P.info[fld].status, (int32_t)GD_TIMEOUT);
            P.info[fld].iters = 0;
        }
    // A workgroup gives up by itself, so after a reduction some may have gone
    // on and others not: workgroup 0 may have written the record of a field
    // whose other boxes were not stored.  The workgroup that ends last sees
    // whether any gave up, and marks every field then.
    if (P.W > 1 && tid == 0) {
        gd::wait_vm_stores();
        const uint32_t n =
            __hip_atomic_fetch_add(P.abort + kEnded, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n == gridDim.x - 1 && ld_agent(P.abort))
            for (int64_t b = 0; b < P.batch; ++b) st_agent(&P.info[b].status, (int32_t)GD_TIMEOUT);
    }
}

}  // namespace gdres
