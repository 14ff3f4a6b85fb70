// gd_cnn.hip -- learned warm start for the deconvolution solve: a small
// periodic convolutional network u0 = ubar + s * f(ubar / s), trained on
// (ubar = G u, u) pairs, whose output starts a solver with GD_INIT_GIVEN.
//
// The paper starts every iteration from u0 = ubar (Algorithms 1-4); the
// network only replaces that starting point, the solve itself is unchanged.
//
// Network: 6 layers of periodic 3x3 (2D) or 3x3x3 (3D) cross-correlation with
// bias, 1 -> 32 -> 32 -> 32 -> 32 -> 32 -> 1 channels, ReLU after every layer
// but the last, then the deconvolution filter G itself, u0 = ubar + s * G z: the
// correction stays in the range of G like the paper's start u0 = ubar, so it
// adds nothing where G's transfer function vanishes (where the Krylov solvers
// are slowest); s is the per-sample RMS of ubar.  Weights of layer l are
// W[cout][tap][cin] (tap = 3 (dy + 1) + (dx + 1), in 3D 9 (dz + 1) + ...)
// followed by bias[cout], all layers packed into one FP32 parameter vector.
//
// A 3D field is a stack of nz planes and a 3D convolution is the sum of three
// 2D convolutions of the planes shifted by dz = -1, 0, +1, each with its own
// 3x3 slice of the weights.
//
// Data layout: activations are bfloat16, channels fastest (NHWC, 64 bytes per
// point).  The four 32 -> 32 layers run as implicit GEMMs on the matrix cores
// (v_mfma_f32_32x32x16_bf16: 32 points x 32 output channels per wave, K = 9
// taps x 32 input channels = 18 MFMA steps per slice, FP32 accumulation); the
// input tile with its periodic halo sits in LDS and the layer's weights in
// registers.  Their input gradients reuse the same kernels with transposed,
// tap-flipped weights.  Layer 1 and the input gradient of layer 6 use plain
// FP32 arithmetic (288 or 864 multiply-adds per point), as do the weight
// gradients of the end layers; layer 6 and the 32 -> 32 weight gradients run
// on the matrix cores too.  Weight gradients are reduced deterministically
// (per-block partial sums added in a fixed order).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>

#include "gdecon.h"

namespace gd {
void set_error_text(const char *msg);
int64_t checked_points(const int64_t *n, int ndim, int64_t cap);
}

namespace gdcnn {

typedef __bf16 bf16;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int C = 32;           // channels
constexpr int K9 = 9 * C;       // reduction length of one 3x3 slice
constexpr int NL = 6;           // layers
constexpr int K = K9;           // reduction length of a 2D 32 -> 32 layer (one MFMA pass)
constexpr int NMID = NL - 2;    // 32 -> 32 layers
constexpr int TX = 32;          // columns of a conv tile or a weight-gradient strip (one MFMA tile)
constexpr int NW_MID = C * K + C;  // weights + biases of a 32 -> 32 layer
constexpr int NW_END = K + C;      // either end layer's weights (288) + up to 32 biases
constexpr int RMS_CHUNKS = 64;

struct Offsets {
    int64_t W[NL], b[NL], total;
};

// parameter offsets for NT taps per layer (9 in 2D, 27 in 3D)
Offsets offsets(int NT) {
    Offsets o;
    int64_t off = 0;
    for (int l = 0; l < NL; ++l) {
        const int ci = l == 0 ? 1 : C, co = l == NL - 1 ? 1 : C;
        o.W[l] = off;
        off += (int64_t)co * NT * ci;
        o.b[l] = off;
        off += co;
    }
    o.total = off;
    return o;
}

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// plane pz = sample * nz + z shifted by dz planes within its sample (periodic)
__device__ __forceinline__ int64_t plane_shift(int64_t pz, int nz, int dz) {
    const int z = (int)(pz % nz);
    return pz - z + wrap(z + dz, nz);
}

// ---------------------------------------------------------------- small kernels

// the bf16 weights, and FP32 copies of them for the two end layers (k_conv_end's order)
__global__ void k_cvt(const float *p, bf16 *q, int64_t n, float *wend, int64_t off_w1, int64_t off_w6, int NT) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) q[i] = (bf16)p[i];
    if (i < C * NT) {
        const int c = (int)i / NT, t = (int)i % NT;
        const int to = ((c >> 3) * (NT / 9) + t / 9) * 72 + (c & 7) * 9 + t % 9;
        wend[to] = (float)(bf16)p[off_w1 + c * NT + t];
        wend[C * NT + to] = (float)(bf16)p[off_w6 + t * C + c];
    }
}

// Per-dz 3x3 weight slices of the 32 -> 32 layers for the matrix-core kernel,
// out[m][dzi][row][t * 32 + col] (ndz = NT / 9 slices):
//   forward (BWD = false): row = cout, col = cin: W[m][cout][dzi * 9 + t][cin];
//   input gradient (BWD):  row = cin, col = cout: W[m][cout][NT - 1 - (dzi * 9 + t)][cin]
// (the mirrored tap: the input gradient correlates with the flipped kernel).
template <bool BWD>
__global__ void k_repack(const bf16 *wbf, int64_t off_w1, int64_t layer_stride, int NT, bf16 *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int ndz = NT / 9;
    if (i >= (int64_t)NMID * ndz * C * K9) return;
    const int m = (int)(i / ((int64_t)ndz * C * K9));
    const int r = (int)(i % ((int64_t)ndz * C * K9));
    const int dzi = r / (C * K9), r2 = r % (C * K9);
    const int row = r2 / K9, t = (r2 % K9) / C, col = r2 % C;
    const int cout = BWD ? col : row, cin = BWD ? row : col;
    const int tap = BWD ? NT - 1 - (dzi * 9 + t) : dzi * 9 + t;
    out[i] = wbf[off_w1 + m * layer_stride + ((int64_t)cout * NT + tap) * C + cin];
}

template <typename T>
__global__ void k_rms_part(const T *ub, int64_t P, double *part) {
    __shared__ double red[256];
    const int b = blockIdx.y, chunk = blockIdx.x;
    const int64_t lo = P * chunk / RMS_CHUNKS, hi = P * (chunk + 1) / RMS_CHUNKS;
    double acc = 0.0;
#pragma unroll 8
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
        const double v = (double)ub[(int64_t)b * P + i];
        acc += v * v;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(int64_t)b * RMS_CHUNKS + chunk] = red[0];
}

__global__ void k_rms_fin(const double *part, int B, int64_t P, double *s) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    double acc = 0.0;
    for (int k = 0; k < RMS_CHUNKS; ++k) acc += part[(int64_t)b * RMS_CHUNKS + k];
    const double r = sqrt(acc / (double)P);
    s[b] = r > 0.0 ? r : 1.0;
}

// One channel -> 32 channels: layer 1 (in = ubar / s, + bias, ReLU) and, with
// GRAD, the input gradient of layer 6 through the ReLU of layer 5 (in = dL/dz,
// taps mirrored, masked by a5 > 0).  wt: FP32 copies of the bf16 weights,
// [channel / 8][dz][channel % 8][tap of the slice].  Bound by the 288 or 864
// FP32 multiply-adds per point and the 64-byte stores.  A thread takes EPT
// rows of one column and all channels: the weights are wave-uniform (scalar
// registers, 72 at a time, each used EPT times) and the window slides along z
// (3D), a value being loaded once per plane.  The channels of a row of points
// pass through LDS (wave-private, chunks permuted like the conv tiles) and
// leave as whole lines.  One point per thread, with the weights converted
// from bf16 at every use and 16-byte stores 64 bytes apart, took 578 us for
// 4 x 128^3 (64 us for 8 x 512^2; the input gradient 77 us); this takes
// 267 us (38 and 62 us).
constexpr int EPT = 4, EZ = 16;  // rows per thread; most planes per run
// LDS position (in 16-byte chunks) of chunk c of point pix: the four chunks of
// a point are permuted by its index, so that the 16-byte accesses of 8
// adjacent points hit 8 different bank groups
__device__ __forceinline__ int swz(int pix, int c) { return pix * 4 + (c ^ ((pix >> 1) & 3)); }
template <typename T, int NT, bool GRAD>
__global__ __launch_bounds__(256) void k_conv_end(const T *in, const double *s, const float *__restrict__ wt,
                                                  const float *__restrict__ bias, const bf16 *mask, bf16 *out, int H,
                                                  int W, int nz, int tiles_x, int tiles_y, int zruns, int zrun) {
    constexpr int ND = NT / 9;
    __shared__ uint4 stage[4][EPT][64 * 4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int blk = blockIdx.x;
    const int x0 = (blk % tiles_x) * 64, x = min(x0 + lane, W - 1);
    const int y0 = (blk / tiles_x % tiles_y * 4 + wave) * EPT;
    const int rest = blk / (tiles_x * tiles_y), zr = rest % zruns;
    const int64_t smp = rest / zruns;
    if (y0 >= H) return;  // the whole wave
    const int64_t HW = (int64_t)H * W;
    const int zlo = zr * zrun, zhi = min(nz, zlo + zrun);
    const float inv = GRAD ? 1.0f : (float)(1.0 / s[smp]);
    const int xm = wrap(x - 1, W), xp = wrap(x + 1, W);
    float v[ND][EPT + 2][3];
    auto load = [&](int z, float (&p)[EPT + 2][3]) {
        const T *pl = in + (smp * nz + wrap(z, nz)) * HW;
#pragma unroll
        for (int r = 0; r < EPT + 2; ++r) {
            int y = y0 + r - 1;
            y = y < 0 ? y + H : (y >= H ? (y == H ? 0 : H - 1) : y);  // rows past H feed points that are not stored
            const T *row = pl + (int64_t)y * W;
            p[r][0] = (float)row[xm] * inv;
            p[r][1] = (float)row[x] * inv;
            p[r][2] = (float)row[xp] * inv;
        }
    };
    if constexpr (ND == 3) {
        load(zlo - 1, v[1]);
        load(zlo, v[2]);
    }
    for (int z = zlo; z < zhi; ++z) {
        if constexpr (ND == 3) {
#pragma unroll
            for (int r = 0; r < EPT + 2; ++r)
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    v[0][r][k] = v[1][r][k];
                    v[1][r][k] = v[2][r][k];
                }
            load(z + 1, v[2]);
        } else {
            load(z, v[0]);
        }
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {  // 8 channels at a time
            float acc[EPT][8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float b = GRAD ? 0.0f : bias[8 * q + k];
#pragma unroll
                for (int i = 0; i < EPT; ++i) acc[i][k] = b;
            }
#pragma unroll
            for (int d = 0; d < ND; ++d) {
                const float *w = wt + (q * ND + d) * 72;
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int t = 0; t < 9; ++t)
#pragma unroll
                        for (int i = 0; i < EPT; ++i)
                            acc[i][k] += w[k * 9 + t] *
                                         (GRAD ? v[ND - 1 - d][i + 2 - t / 3][2 - t % 3] : v[d][i + t / 3][t % 3]);
            }
#pragma unroll
            for (int i = 0; i < EPT; ++i) {
                alignas(16) bf16 o[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) o[k] = (bf16)(GRAD ? acc[i][k] : fmaxf(acc[i][k], 0.0f));
                stage[wave][i][swz(lane, q)] = *reinterpret_cast<const uint4 *>(o);
            }
        }
        // a wave reads back what it wrote itself: 16 points of 64 bytes per store
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            if (y0 + i >= H) continue;
            const int64_t at = ((smp * nz + z) * HW + (int64_t)(y0 + i) * W + x0) * C;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int pt = g * 16 + (lane >> 2);
                if (x0 + pt >= W) continue;
                uint4 r = stage[wave][i][swz(pt, lane & 3)];
                const int64_t to = at + (int64_t)pt * C + (lane & 3) * 8;
                if constexpr (GRAD) {
                    alignas(16) bf16 m[8], o[8];
                    *reinterpret_cast<uint4 *>(m) = *reinterpret_cast<const uint4 *>(mask + to);
                    *reinterpret_cast<uint4 *>(o) = r;
#pragma unroll
                    for (int k = 0; k < 8; ++k) o[k] = (float)m[k] > 0.0f ? o[k] : (bf16)0.0f;
                    r = *reinterpret_cast<const uint4 *>(o);
                }
                *reinterpret_cast<uint4 *>(out + to) = r;
            }
        }
    }
}

// 32 -> 32 layers on the matrix cores.  wmat: [dz][cout][K], K = tap * 32 + cin.
// MODE kFwd: out = relu(conv(in) + bias); kBwd (input gradient): out =
// conv'(in) * (mask > 0), with `in` the output gradient, the transposed,
// mirrored weights and `mask` the layer's input activation.
//
// A workgroup of four waves owns 4 RB rows x 32 columns of a plane, wave w
// rows w RB ...  A plane's tile with its halo sits in LDS, written by
// direct-to-LDS loads (no registers), 64 bytes per point with its chunks
// permuted (tile_at).  An input row is read from LDS once (six
// operands: three taps, two channel halves) and used for the three output
// rows it belongs to, with the weights in registers.  Products per output run
// dz, dy, dx, channel half in order.
constexpr int kFwd = 0, kBwd = 1, kFused = 2;  // kFused: the bias is in the sums already
constexpr int TXH = TX + 2;  // tile columns with the halo
constexpr int RB = 4;        // output rows per wave (8 in 2D measured the same)
constexpr size_t kConvLds = (size_t)(4 * RB + 2) * TXH * C * sizeof(bf16);  // one plane's tile

// Workgroup barrier ordering LDS only: the threads of the kernels that use
// it share data through LDS alone, and a full barrier would also wait for the
// global loads and stores they keep in flight across steps.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// contiguous ranges of the grid per XCD (workgroups are dealt round-robin over
// the 8 XCDs), so that tiles sharing halos and planes share an L2
__device__ __forceinline__ int64_t xcd_order() {
    const int64_t nb = gridDim.x, per = nb / 8, rem = nb % 8, xcd = blockIdx.x % 8, k = blockIdx.x / 8;
    return xcd * per + (xcd < rem ? xcd : rem) + k;
}

// chunk c (of four, 16 bytes each) of point (row, col) of a tile, in chunks.
// The permutation depends on the column only, so that a lane's rows are one
// address plus constants.
__device__ __forceinline__ int tile_at(int row, int col, int c) { return (row * TXH + col) * 4 + (c ^ ((col >> 1) & 3)); }

// A plane's tile (rows y0 - 1 .., columns x0 - 1 .., periodic) is loaded in
// 16-byte pieces, piece k 256 + thread by a thread: one of the four chunks of a
// point.  A plane has up to 2^31 - 1 points, so a piece's place takes 33 bits:
// the point and the chunk are apart until the load.
constexpr int CH = (4 * RB + 2) * TXH * 4, CPL = (CH + 255) / 256;  // pieces, per thread
struct Piece {
    uint32_t point, chunk;
};
__device__ __forceinline__ Piece tile_piece(int k, int x0, int y0, int H, int W) {
    const int q = min(k * 256 + (int)threadIdx.x, CH - 1);
    const int pix = q >> 2, r = pix / TXH, cc = pix - r * TXH, c = (q & 3) ^ ((cc >> 1) & 3);
    int gy = y0 + r - 1, gx = x0 + cc - 1;
    gy = gy < 0 ? gy + H : (gy >= H ? (gy == H ? 0 : H - 1) : gy);  // points past the halo are not used
    gx = gx < 0 ? gx + W : (gx >= W ? (gx == W ? 0 : W - 1) : gx);
    return {(uint32_t)gy * (uint32_t)W + (uint32_t)gx, (uint32_t)c};
}
// start the load of piece k, `at` elements into the plane, into LDS
__device__ __forceinline__ void stage_piece(const bf16 *plane, unsigned char *tile, int k, uint64_t at, int wave) {
    if ((k + 1) * 256 <= CH || k * 256 + (int)threadIdx.x < CH)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(plane + at),
                                         (__attribute__((address_space(3))) void *)(tile + (k * 256 + wave * 64) * 16), 16,
                                         0, 0);
}
// wait for this wave's outstanding loads (vmcnt 0), tile loads included
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// the products of one 3x3 slice: input rows of `tile` into the wave's RB output rows
__device__ __forceinline__ void conv_slice(const bf16 *tile, const bf16x8 (&Wf)[K / 16], f32x16 (&acc)[RB], int wave,
                                           int j, int kh) {
#pragma unroll
    for (int ir = 0; ir < RB + 2; ++ir) {
        bf16x8 A[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            A[k] = *reinterpret_cast<const bf16x8 *>(tile + tile_at(wave * RB + ir, j + (k >> 1), (k & 1) * 2 + kh) * 8);
        }
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int i = ir - dy;
                if (i >= 0 && i < RB)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Wf[dy * 6 + k], A[k], acc[i], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);  // all rows' reads at the front would not fit the registers
    }
}

// max(x, 0) as one integer max on the bits (a negative float is a negative
// integer): fmaxf also quiets signalling NaNs, one more instruction per value
__device__ __forceinline__ float relu_bits(float x) {
    return __builtin_bit_cast(float, max(__builtin_bit_cast(int, x), 0));
}

// A lane's outputs of a row: point x, output channels 8 g + 4 kh .. + 3.  The
// half-waves exchange half of their channels (v_permlane32_swap), so that a
// lane stores 16 channels as two 16-byte pieces (lower half channels 0 - 15,
// upper half 16 - 31) and not four of 8 bytes.
struct alignas(16) Packed {
    uint32_t q[8];
};
template <int MODE>
__device__ __forceinline__ Packed conv_pack(const f32x16 &acc, const f32x16 &bv) {
    uint32_t p[4][2];  // [g][channel pair]
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float a = acc[4 * g + 2 * k], b = acc[4 * g + 2 * k + 1];
            if constexpr (MODE == kFwd) {
                a = fmaxf(a + bv[4 * g + 2 * k], 0.0f);
                b = fmaxf(b + bv[4 * g + 2 * k + 1], 0.0f);
            } else if constexpr (MODE == kFused) {
                a = relu_bits(a);
                b = relu_bits(b);
            }
            const bf16x2 o = {(bf16)a, (bf16)b};
            p[g][k] = __builtin_bit_cast(uint32_t, o);
        }
    Packed r;
#pragma unroll
    for (int g = 0; g < 2; ++g)  // lower half: channels 8 g .. 8 g + 7; upper half: 16 + 8 g ..
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(p[g][k], p[g + 2][k], false, false));
            r.q[4 * g + k] = x[0];
            r.q[4 * g + 2 + k] = x[1];
        }
    return r;
}
// rows y0 .. y0 + RB - 1 of plane pz
template <int MODE>
__device__ __forceinline__ void conv_store(Packed (&v)[RB], const bf16 *mask, bf16 *out, int64_t pz, int y0, int x,
                                           int H, int W, int kh) {
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int y = y0 + i;
        if (y >= H || x >= W) continue;
        const int64_t idx = ((pz * H + y) * (int64_t)W + x) * C + 16 * kh;
        if constexpr (MODE == kBwd) {
            alignas(16) bf16 m[16];
            bf16 *o = reinterpret_cast<bf16 *>(v[i].q);
            *reinterpret_cast<uint4 *>(m) = *reinterpret_cast<const uint4 *>(mask + idx);
            *reinterpret_cast<uint4 *>(m + 8) = *reinterpret_cast<const uint4 *>(mask + idx + 8);
#pragma unroll
            for (int k = 0; k < 16; ++k) o[k] = (float)m[k] > 0.0f ? o[k] : (bf16)0.0f;
        }
        *reinterpret_cast<uint4 *>(out + idx) = *reinterpret_cast<const uint4 *>(v[i].q);
        *reinterpret_cast<uint4 *>(out + idx + 8) = *reinterpret_cast<const uint4 *>(v[i].q + 4);
    }
}

template <int MODE>
__device__ __forceinline__ f32x16 conv_bias(const float *bias, int kh) {
    f32x16 bv = {};
    if constexpr (MODE == kFwd)
#pragma unroll
        for (int v = 0; v < 16; ++v) bv[v] = bias[8 * (v >> 2) + 4 * kh + (v & 3)];
    return bv;
}

// 2D.  Bound by HBM: one read and one write of 64 bytes per point, the input
// gradient two reads.  Two or more workgroups per CU: one loads its tile
// while another computes.  A tile of eight rows with every operand read from
// LDS for each output row and 2-byte stores took 131 (input gradient 311) us
// for 8 x 512^2; this takes 72 (91) us.
template <int MODE>
__global__ __launch_bounds__(256, 3) void k_conv_mid(const bf16 *in, const bf16 *wmat, const float *bias,
                                                     const bf16 *mask, bf16 *out, int H, int W, int tiles_x,
                                                     int tiles_y) {
    extern __shared__ __attribute__((aligned(16))) unsigned char conv_tile[];
    const int64_t blk = xcd_order();
    const int x0 = (int)(blk % tiles_x) * TX, y0 = (int)(blk / tiles_x % tiles_y) * 4 * RB;
    const int64_t pz = blk / ((int64_t)tiles_x * tiles_y);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, kh = lane >> 5;
#pragma unroll 1
    for (int k = 0; k < CPL; ++k) {
        const Piece p = tile_piece(k, x0, y0, H, W);
        stage_piece(in + pz * H * W * C, conv_tile, k, (uint64_t)p.point * C + p.chunk * 8, wave);
    }
    bf16x8 Wf[K / 16];
#pragma unroll
    for (int ks = 0; ks < K / 16; ++ks) Wf[ks] = *reinterpret_cast<const bf16x8 *>(wmat + j * K + ks * 16 + kh * 8);
    f32x16 acc[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[i] = f32x16{};
    wait_loads();
    __syncthreads();
    conv_slice(reinterpret_cast<const bf16 *>(conv_tile), Wf, acc, wave, j, kh);
    const f32x16 bv = conv_bias<MODE>(bias, kh);
    Packed v[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) v[i] = conv_pack<MODE>(acc[i], bv);
    conv_store<MODE>(v, mask, out, pz, y0 + wave * RB, x0 + j, H, W, kh);
}

// 3D: a workgroup marches along z through a run of planes.  Four plane tiles
// sit in LDS (157 KB: one workgroup per CU, one wave per SIMD): the three an
// output plane needs and the next one, in flight while the products run, so an
// activation is loaded once per run and not once per plane that needs it.
// With a whole SIMD's registers a wave keeps the weights of all 27 taps (216
// registers) for the whole run.  One wave per SIMD has no other to hide its
// waits: each input row's operands are read during the products of the row
// before, an output row is packed during the products after its last, and
// the scheduler is kept from moving reads back to their use (it did, to save
// registers: 500 us).  Bound by the matrix cores (216 products of 32 clocks
// per wave and plane; 4 x 128^3 in 402 us are 1150 TFLOP/s, about what a large
// bf16 matrix product reaches on this card).  All three planes' tiles in LDS
// per output plane, the weights loaded per plane and every operand read from
// LDS for each output row took 1387 us.
// WIDE: for planes of more than 2^30 points, whose pieces' places do not fit 32
// bits (32-bit places for the others: forward 4 x 128^3 2181 -> 2160 us)
template <int MODE, bool WIDE>
__global__ __launch_bounds__(256, 1) void k_conv_mid3(const bf16 *in, const bf16 *slices, const float *bias,
                                                      const bf16 *mask, bf16 *out, int H, int W, int nz, int tiles_x,
                                                      int tiles_y, int zruns, int zrun) {
    extern __shared__ __attribute__((aligned(16))) unsigned char conv_tile[];
    const int64_t blk = xcd_order();
    const int x0 = (int)(blk % tiles_x) * TX, y0 = (int)(blk / tiles_x % tiles_y) * 4 * RB;
    const int64_t rest = blk / ((int64_t)tiles_x * tiles_y);
    const int zlo = (int)(rest % zruns) * zrun, zhi = min(nz, zlo + zrun);
    const int64_t p0 = rest / zruns * nz;  // the sample's first plane
    const int64_t HW = (int64_t)H * W;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 31, kh = lane >> 5;
    constexpr size_t TB = kConvLds;
    // plane z (periodic) into ring slot (z - zlo + 1) mod 4
    // the pieces' places; WIDE: their points, and two bits of chunk each
    uint32_t piece[CPL], chunks = 0;
    static_assert(CPL <= 16);
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        const Piece p = tile_piece(k, x0, y0, H, W);
        piece[k] = WIDE ? p.point : p.point * 4 + p.chunk;
        chunks |= p.chunk << 2 * k;
    }
    auto stage = [&](int z) {
        const bf16 *plane = in + (p0 + wrap(z, nz)) * HW * C;
#pragma unroll
        for (int k = 0; k < CPL; ++k)
            stage_piece(plane, conv_tile + (size_t)((z - zlo + 1) & 3) * TB, k,
                        WIDE ? (uint64_t)piece[k] * C + (chunks >> 2 * k & 3) * 8 : (uint64_t)piece[k] * 8, wave);
    };
    stage(zlo - 1);
    stage(zlo);
    stage(zlo + 1);
    bf16x8 Wf[3][K / 16];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int ks = 0; ks < K / 16; ++ks)
            Wf[d][ks] = *reinterpret_cast<const bf16x8 *>(slices + (size_t)d * C * K9 + j * K + ks * 16 + kh * 8);
    const f32x16 bv = conv_bias<MODE>(bias, kh);
    int a6[6];  // this lane's six operands of a row, in the wave's first
#pragma unroll
    for (int k = 0; k < 6; ++k) a6[k] = tile_at(wave * RB, j + (k >> 1), (k & 1) * 2 + kh) * 8;
    wait_loads();
    for (int z = zlo; z < zhi; ++z) {
        lds_barrier();  // every wave's share of plane z + 1 is in LDS, and plane z - 2 has been read by all
        if (z + 2 <= zhi) stage(z + 2);
        f32x16 acc[RB];
        Packed v[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) acc[i] = f32x16{};
        constexpr int NR = RB + 2, NG = 3 * NR;
        const bf16 *slot[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) slot[d] = reinterpret_cast<const bf16 *>(conv_tile + (size_t)((z - zlo + d) & 3) * TB);
        auto row = [&](int g, bf16x8 (&A)[6]) {  // input row g % NR of slice g / NR
            const bf16 *tile = slot[g / NR];
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                A[k] = *reinterpret_cast<const bf16x8 *>(tile + a6[k] + (g % NR) * TXH * C);
            }
        };
        bf16x8 A[2][6];
        row(0, A[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) row(g + 1, A[(g + 1) & 1]);
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int i = g % NR - dy;
                    if (i >= 0 && i < RB)
                        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Wf[g / NR][dy * 6 + k], A[g & 1][k], acc[i], 0,
                                                                        0, 0);
                }
            // a row's sums are complete after its last input row: packed during the next products
            if (g > NG - RB) v[g - 1 - (NG - RB)] = conv_pack<MODE>(acc[g - 1 - (NG - RB)], bv);
            __builtin_amdgcn_sched_barrier(0);
        }
        v[RB - 1] = conv_pack<MODE>(acc[RB - 1], bv);
        wait_loads();  // plane z + 2, before the stores: they need not be waited for
        conv_store<MODE>(v, mask, out, p0 + z, y0 + wave * RB, x0 + j, H, W, kh);
    }
}

// ---------------------------------------------------------------- fused 2D forward
//
// Inference in 2D runs all six layers in one kernel, so no activation goes
// through HBM.  A workgroup owns a strip of FV output columns and up to FY
// rows of one sample and marches down it, two rows of every layer per step.
// Layer l keeps the rows of its input that its 3x3 taps need in an LDS ring
// (layers 2 .. 6; layer 1 reads ubar / s from a ring of its own); at step s
// layer l computes rows ys + 2 s - 3 (l - 1) and the next, three rows behind
// layer l - 1: the four input rows it reads were written in the two steps
// before, and the two it writes go to slots that no layer reads in that step,
// so a ring has six slots and a step one barrier.  The slots depend on s mod 3
// alone: the step loop is unrolled by three, and every LDS address is a
// register set up once plus a constant.  A layer outside its rows computes on
// stale ring rows; what it writes reaches no row that is needed.
// Columns: a frame of FW = 64 columns starting 5 left of the strip.  Layer l's
// row is needed on frame columns l - 1 .. FV + 10 - l, so with FV = 54 every
// layer computes the frame's 64 columns (two MFMA tiles for the 32 -> 32
// layers, one column per lane for layer 1) and layer 6 the strip's 54.
// Layer 6 runs on the matrix cores too, as the products of an input column
// with all nine taps, which the next step sums.  Layer 1 stays on the vector
// units: as matrix products of exact bf16 terms of ubar / s it took 100 us
// less, but another order of its sums flips bf16 roundings of its output.
// Bound by the matrix cores (37 products of 32 clocks per wave and step, two
// waves per SIMD: 60 % of the time) and a step's latency.  16 x 1024^2: one row
// per step, with layer 6 on the vector units, 1824 us; two rows per step 1571;
// this 1396 (890 TFLOP/s of the 32 -> 32 layers alone).
constexpr int FW = 64, FV = FW - 10, FY = 256, FRC = FW + 2;  // frame, strip, rows per workgroup, ring columns
constexpr int FTHREADS = 512;
constexpr int RSL = 6;        // ring slots: four rows read, two written in the same step
constexpr int RROW = FRC * C; // elements of a ring row
constexpr int URC = FRC;      // ubar ring columns: frame -1 .. FW
constexpr int URS = 32;       // ubar ring rows
constexpr int UBATCH = 6;     // ubar rows loaded together, every three steps
static_assert(UBATCH * FRC <= FTHREADS, "one ubar value per thread");
constexpr size_t kRingBytes = (size_t)(NL - 1) * RSL * RROW * sizeof(bf16);
constexpr size_t kURingBytes = (size_t)URS * URC * sizeof(float);
constexpr size_t kFusedLds = kRingBytes + kURingBytes + (size_t)RSL * 3 * FW * sizeof(f32x4);
static_assert(kFusedLds <= 160 * 1024, "LDS of one CU");

// a value that is the same in every lane, in a scalar register
__device__ __forceinline__ float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

template <typename T>
__global__ __launch_bounds__(FTHREADS) void k_fwd2d_fused(const T *ub, const double *s, const bf16 *wbf,
                                                          const float *params, Offsets off, float *z, int H, int W) {
    extern __shared__ __attribute__((aligned(16))) unsigned char fused_lds[];
    bf16 *ring = reinterpret_cast<bf16 *>(fused_lds);                  // [layer 2..6][slot RSL][FRC][C]
    float *uring = reinterpret_cast<float *>(fused_lds + kRingBytes);  // ubar / s: [row slot URS][URC]
    // layer 6's products: [slot RSL][taps 4 t .. 4 t + 3][frame column]
    f32x4 *zring = reinterpret_cast<f32x4 *>(fused_lds + kRingBytes + kURingBytes);
    // channels 8 c .. 8 c + 7 of a ring column, in slot 0 of layer l's input;
    // a column's four chunks are permuted by its index
    auto at = [&](int l, int col, int c) { return ring + (l - 2) * RSL * RROW + col * C + (c ^ ((col >> 2) & 3)) * 8; };
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.z;
    const int x0 = blockIdx.x * FV, y0 = blockIdx.y * FY;
    const int rows = min(FY, H - y0);
    const int ys = y0 - 5;  // first row of layer 1's output
    const int64_t HW = (int64_t)H * W;
    const T *ubs = ub + (int64_t)b * HW;
    const float inv = (float)(1.0 / s[b]);
    // clear the rings once: ring columns 0 and FRC - 1 are never written and
    // feed only frame columns whose results are not needed
    for (int i = tid; i < (int)(kRingBytes / 16); i += FTHREADS) reinterpret_cast<uint4 *>(fused_lds)[i] = uint4{0, 0, 0, 0};

    // matrix-core role: wave w computes layer ML = 2 + w / 2, frame columns 32 (w % 2) ..
    const int ML = 2 + (wave >> 1), mh = wave & 1;
    const int j = lane & 31, kh = lane >> 5;
    bf16x8 Wf[K / 16];
    {
        const bf16 *wm = wbf + off.W[ML - 1];
#pragma unroll
        for (int ks = 0; ks < K / 16; ++ks) Wf[ks] = *reinterpret_cast<const bf16x8 *>(wm + j * K + ks * 16 + kh * 8);
    }
    f32x16 mb;  // biases of the output channels this lane holds: the accumulator's start
#pragma unroll
    for (int v = 0; v < 16; ++v) mb[v] = params[off.b[ML - 1] + 8 * (v >> 2) + 4 * kh + (v & 3)];
    // layer 1: wave w takes channels 4 w .. 4 w + 3, so its weights are uniform
    // across the wave
    float w1r[4][9], b1r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        b1r[k] = uniform(params[off.b[0] + 4 * wave + k]);
#pragma unroll
        for (int t = 0; t < 9; ++t) w1r[k][t] = uniform((float)wbf[off.W[0] + (4 * wave + k) * 9 + t]);
    }
    // layer 6: wave w takes frame columns 16 (w % 4) .. of the step's first (w < 4)
    // or second row, lane group g4 = lane / 16 a quarter of the channels
    const int orow = wave >> 2, pcol = 16 * (wave & 3) + (lane & 15), g4 = lane >> 4;
    bf16x8 W6f;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        W6f[e] = (lane & 15) < 9 ? wbf[off.W[NL - 1] + (lane & 15) * C + 8 * g4 + e] : (bf16)0.0f;
    const float b6 = params[off.b[NL - 1]];

    // ubar / s enters a ring of URS rows (row ys - 1 + rho in slot rho % URS),
    // six rows per three steps and one value per thread: loaded three steps
    // before they are stored, and stored before the steps that read them
    const int ur = tid / URC, uc = tid - ur * URC;
    const int64_t ux = ((x0 - 6 + uc) % W + W) % W;
    const int nu = rows + 12;  // rows rho = 0 .. rows + 11 feed layer 1
    auto u_load = [&](int rho0) {
        const int rho = rho0 + ur;
        return ur < UBATCH && rho < nu ? (float)ubs[(int64_t)((((ys - 1 + rho) % H) + H) % H) * W + ux] * inv : 0.0f;
    };
    auto u_store = [&](int rho0, float v) {
        if (ur < UBATCH) uring[((rho0 + ur) & (URS - 1)) * URC + uc] = v;
    };
    u_store(0, u_load(0));
    u_store(UBATCH, u_load(UBATCH));
    float unext = u_load(2 * UBATCH);
    __syncthreads();

    const int nstep = 11 + (rows + 1) / 2;  // z of rows y0 .. from step 11 on
    // this lane's places in the rings, in slot 0
    const bf16 *am[6];  // layer ML's operands of an input row: taps k / 2, channel halves k % 2
#pragma unroll
    for (int k = 0; k < 6; ++k) am[k] = at(ML, 32 * mh + j + (k >> 1), (k & 1) * 2 + kh);
    const bf16 *a6 = at(NL, pcol + 1, g4);  // layer 6's input
    f32x4 *z6 = zring + g4 * FW + pcol;     // and products
    bf16 *wm[2];  // layer ML's outputs, 16 channels per lane
#pragma unroll
    for (int g = 0; g < 2; ++g) wm[g] = at(ML + 1, 32 * mh + j + 1, 2 * kh + g);
    bf16 *w1 = at(2, lane + 1, wave >> 1) + (wave & 1) * 4;  // layer 1's
    auto row = [&](int slot, bf16x8 (&A)[6]) {
#pragma unroll
        for (int k = 0; k < 6; ++k) A[k] = *reinterpret_cast<const bf16x8 *>(am[k] + slot * RROW);
    };
    // a step's first two input rows are older than the step before and are
    // read ahead of its barrier
    bf16x8 A[2][6];
    row(2, A[0]);
    row(3, A[1]);
    auto step = [&](auto phase, int st) {
        constexpr int c = phase.value;
        constexpr int in_slot[4] = {2 * ((c + 1) % 3), 2 * ((c + 1) % 3) + 1, 2 * ((c + 2) % 3), 2 * ((c + 2) % 3) + 1};
        float xv[4][3];
#pragma unroll
        for (int r = 0; r < 4; ++r) {  // frame column lane + dx - 1
            const float *u = uring + ((2 * st + r) & (URS - 1)) * URC + lane;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) xv[r][dx] = u[dx];
        }
        const bf16x8 A6 = *reinterpret_cast<const bf16x8 *>(a6 + (orow ? in_slot[3] : in_slot[2]) * RROW);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc[2] = {mb, mb};
        // the products of input row g, per output row and tap in order
        auto products = [&](int g) {
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int dy = g - o;
                    if (dy >= 0 && dy < 3)
                        acc[o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Wf[dy * 6 + k], A[g & 1][k], acc[o], 0, 0, 0);
                }
        };
        auto layer1 = [&](int o) {
            alignas(8) bf16 v1[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float v = b1r[k];
#pragma unroll
                for (int t = 0; t < 9; ++t) v += w1r[k][t] * xv[o + t / 3][t % 3];
                v1[k] = (bf16)relu_bits(v);
            }
            *reinterpret_cast<uint2 *>(w1 + (2 * c + o) * RROW) = *reinterpret_cast<const uint2 *>(v1);
        };
        auto write = [&](int o) {
            const Packed v = conv_pack<kFused>(acc[o], mb);
#pragma unroll
            for (int g = 0; g < 2; ++g)
                *reinterpret_cast<uint4 *>(wm[g] + (2 * c + o) * RROW) = *reinterpret_cast<const uint4 *>(v.q + 4 * g);
        };
        products(0);
        layer1(0);
        __builtin_amdgcn_sched_barrier(0);
        row(in_slot[2], A[0]);
        products(1);
        layer1(1);
        const f32x4 d6 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W6f, A6, f32x4{}, 0, 0, 0);
        if (g4 < 3) z6[(orow ? 2 * c + 1 : 2 * c) * 3 * FW] = d6;
        __builtin_amdgcn_sched_barrier(0);
        row(in_slot[3], A[1]);
        products(2);
        __builtin_amdgcn_sched_barrier(0);
        row(in_slot[2], A[0]);  // the next step's first
        products(3);
        write(0);
        __builtin_amdgcn_sched_barrier(0);
        row(in_slot[3], A[1]);
        write(1);
        // z of rows y0 + 2 st - 22 and the next: their input rows' products are
        // those of the two steps before
        if (wave < 2) {
            const int y = 2 * (st - 11) + wave, x = x0 + lane;
            float zs = b6;
#pragma unroll
            for (int t = 0; t < 9; ++t)
                zs += zring[((wave ? in_slot[t / 3 + 1] : in_slot[t / 3]) * 3 + (t >> 2)) * FW + min(lane, FV - 1) + 4 + t % 3][t & 3];
            if (st >= 11 && lane < FV && y < rows && x < W) z[(int64_t)b * HW + (int64_t)(y0 + y) * W + x] = zs;
        }
        lds_barrier();
    };
    for (int st = 0; st < nstep; st += 3) {
        // layer 1 reads rows 2 st .. 2 st + 9 in these three steps
        u_store(2 * st + 2 * UBATCH, unext);
        unext = u_load(2 * st + 3 * UBATCH);
        step(std::integral_constant<int, 0>{}, st);
        if (st + 1 < nstep) step(std::integral_constant<int, 1>{}, st + 1);
        if (st + 2 < nstep) step(std::integral_constant<int, 2>{}, st + 2);
    }
}

// layer 6: 32 channels -> 1, no activation: z.  On the matrix cores: one
// product pair gives, for 32 points, the contributions D[tap][point] =
// sum_c a[point][c] w6[tap][c] of all 9 or 27 taps; they go to LDS, and z at a
// point is the sum over the taps of D[tap][point + off(tap)].  A workgroup
// owns 16 x 32 points of a run of OZ planes (3D; one plane in 2D) and marches
// along z, keeping the sums of the planes that still miss a neighbour in
// registers, so an activation is read once and not once per tap.
// Bound by that read: reading 64 bytes per tap and point took 1191 us for
// 4 x 128^3 (113 us for 8 x 512^2); this takes 137 (29) us.
constexpr int OY = 16, OX = 32, OZ = 16;  // OZ: most planes per run
constexpr int OPTS = (OY + 2) * (OX + 2), OGRP = (OPTS + 31) / 32;  // tile points with the halo, groups of 32
constexpr int OST = OGRP * 32;                                      // LDS row of one tap
template <int NT>
__global__ __launch_bounds__(256) void k_conv_out(const bf16 *a, const bf16 *w6, const float *b6, float *z, int H,
                                                  int W, int nz, int tiles_x, int tiles_y, int zruns, int zrun) {
    constexpr int ND = NT / 9;
    constexpr int GPW = (OGRP + 3) / 4;  // groups per wave
    __shared__ float D[NT * OST];
    const int64_t blk = xcd_order();
    const int x0 = (int)(blk % tiles_x) * OX, y0 = (int)(blk / tiles_x % tiles_y) * OY;
    const int64_t rest = blk / ((int64_t)tiles_x * tiles_y);
    const int zr = (int)(rest % zruns);
    const int64_t smp = rest / zruns, HW = (int64_t)H * W;
    // 2D: every plane is a sample of its own (nz = 1)
    const int zlo = zr * zrun, zhi = min(nz, zlo + zrun);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 31, kh = lane >> 5;
    // weights: row = tap (rows past NT are zero), k = channel
    bf16x8 Wf[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) Wf[h][e] = j < NT ? w6[min(j, NT - 1) * C + h * 16 + kh * 8 + e] : (bf16)0.0f;
    // this lane's point of each of its wave's groups, as an offset in a plane
    int64_t poff[GPW];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        const int pix = min((wave + 4 * g) * 32 + j, OPTS - 1);
        const int r = pix / (OX + 2), c = pix - r * (OX + 2);
        int gy = y0 + r - 1, gx = x0 + c - 1;
        gy = gy < 0 ? gy + H : (gy >= H ? (gy == H ? 0 : H - 1) : gy);
        gx = gx < 0 ? gx + W : (gx >= W ? (gx == W ? 0 : W - 1) : gx);
        poff[g] = ((int64_t)gy * W + gx) * C + kh * 8;
    }
    bf16x8 A[GPW][2];
    auto load = [&](int q) {  // plane q of the sample, periodic
        const bf16 *pl = a + (smp * nz + wrap(q, nz)) * HW * C;
#pragma unroll
        for (int g = 0; g < GPW; ++g)
            if (wave + 4 * g < OGRP) {
                A[g][0] = *reinterpret_cast<const bf16x8 *>(pl + poff[g]);
                A[g][1] = *reinterpret_cast<const bf16x8 *>(pl + poff[g] + 16);
            }
    };
    constexpr int PP = OY * OX / 256;  // output points per thread
    float prev[PP], cur[PP];           // sums of output planes q - 1 and q
#pragma unroll
    for (int i = 0; i < PP; ++i) prev[i] = cur[i] = 0.0f;
    const float b = b6[0];
    const int q0 = ND == 1 ? zlo : zlo - 1, q1 = ND == 1 ? zhi : zhi + 1;
    load(q0);
    for (int q = q0; q < q1; ++q) {
#pragma unroll
        for (int g = 0; g < GPW; ++g) {
            if (wave + 4 * g >= OGRP) continue;
            f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Wf[0], A[g][0], f32x16{}, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Wf[1], A[g][1], d, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = 8 * (v >> 2) + 4 * kh + (v & 3);
                if (8 * (v >> 2) < NT && t < NT) D[t * OST + (wave + 4 * g) * 32 + j] = d[v];
            }
        }
        if (q + 1 < q1) load(q + 1);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PP; ++i) {
            const int pt = tid + 256 * i, py = pt / OX, px = pt % OX;
            float sd[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) {
                sd[d] = 0.0f;
#pragma unroll
                for (int t = 0; t < 9; ++t)
                    sd[d] += D[(d * 9 + t) * OST + (py + t / 3) * (OX + 2) + px + t % 3];
            }
            const int y = y0 + py, x = x0 + px;
            const bool ok = y < H && x < W;
            if constexpr (ND == 1) {
                if (ok) z[(smp * nz + q) * HW + (int64_t)y * W + x] = sd[0] + b;
            } else {
                // dz = +1 taps of plane q complete output plane q - 1; dz = -1 taps open plane q + 1
                if (ok && q - 1 >= zlo && q - 1 < zhi)
                    z[(smp * nz + q - 1) * HW + (int64_t)y * W + x] = prev[i] + sd[2] + b;
                prev[i] = cur[i] + sd[1];
                cur[i] = sd[0];
            }
        }
        __syncthreads();
    }
}

// out = G in: the periodic trapezoidal filter (1/4, 1/2, 1/4) per axis (the
// z pass only when the field has several planes)
__device__ __forceinline__ float g_apply(const float *in, int64_t pz, int y, int x, int H, int W, int nz) {
    const int ym = wrap(y - 1, H), yp = wrap(y + 1, H), xm = wrap(x - 1, W), xp = wrap(x + 1, W);
    const int64_t HW = (int64_t)H * W;
    auto plane = [&](int64_t q) {
        auto row = [&](int yy) {
            const float *r = in + q * HW + (int64_t)yy * W;
            return 0.5f * r[x] + 0.25f * (r[xm] + r[xp]);
        };
        return 0.5f * row(y) + 0.25f * (row(ym) + row(yp));
    };
    if (nz == 1) return plane(pz);
    return 0.5f * plane(pz) + 0.25f * (plane(plane_shift(pz, nz, -1)) + plane(plane_shift(pz, nz, 1)));
}

// y = G z; writes y (training) and/or u0 = ubar + s * y
template <typename T>
__global__ void k_gfin(const float *z, const T *ub, const double *s, float *y_out, T *u0, int H, int W, int nz,
                       int64_t N) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int64_t HW = (int64_t)H * W;
    const int64_t pz = p / HW;
    const int rem = (int)(p % HW), y = rem / W, x = rem % W;
    const float v = g_apply(z, pz, y, x, H, W, nz);
    if (y_out) y_out[p] = v;
    if (u0) u0[p] = ub[p] + (T)(s[pz / nz] * (double)v);
}

// out = G in (the adjoint of the final filter: G is symmetric)
__global__ void k_gfilt(const float *in, float *out, int H, int W, int nz, int64_t N) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int64_t HW = (int64_t)H * W;
    const int64_t pz = p / HW;
    const int rem = (int)(p % HW), y = rem / W, x = rem % W;
    out[p] = g_apply(in, pz, y, x, H, W, nz);
}

// dL/dy = 2 (y - t) / N with t = (u - ubar) / s; per-block partial sums of (y - t)^2
template <typename T>
__global__ void k_loss(const float *yv, const T *ub, const T *u, const double *s, float *dy, double *part, int64_t HW,
                       int64_t N) {
    __shared__ double red[256];
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double r2 = 0.0;
    if (p < N) {
        const int64_t b = p / HW;
        const double t = ((double)u[p] - (double)ub[p]) / s[b];
        const double r = (double)yv[p] - t;
        dy[p] = (float)(2.0 * r / (double)N);
        r2 = r * r;
    }
    red[threadIdx.x] = r2;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void k_loss_fin(const double *part, int64_t nblk, int64_t N, double *loss) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t k = threadIdx.x; k < nblk; k += blockDim.x) acc += part[k];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0] / (double)N;
}

// ------------------------------------------------------- weight gradients
// A unit of work is one strip of columns of one plane, `ru` rows; a wave
// marches down its units and keeps the sums in registers; a workgroup adds
// its four waves' sums in wave order.

// plane, first column and rows of unit n
struct Unit {
    int64_t b;
    int x0, ya, yb;
};
__device__ __forceinline__ Unit unit_of(int64_t n, int strip, int tiles_x, int chunks, int ru, int H) {
    Unit u;
    u.x0 = (int)(n % tiles_x) * strip;
    u.ya = (int)(n / tiles_x % chunks) * ru;
    u.yb = min(H, u.ya + ru);
    u.b = n / ((int64_t)tiles_x * chunks);
    return u;
}

// End layers, one 3x3 slice: 32 channels v (bf16) against one FP32 channel f,
//   OUT = false (layer 1):  dW[o][t] = sum_p v[p][o] f[p + off(t)],  v = dz, f = ubar / s
//   OUT = true  (layer 6):  dW[t][c] = sum_q v[q][c] f[q - off(t)],  v = a5, f = dL/dz
// and the bias gradient.  Four lanes hold a point's 32 channels (one 16-byte
// load each), 16 points per wave; f's 3x3 window slides down the march, three
// new values per row.  FP32 throughout.  Bound by reading v once (64 bytes
// per point): one thread per weight over an LDS tile took 422 and 502 us for
// 8 x 512^2; this takes 63 and 50 us.
constexpr int ENS = 16;  // columns per unit
template <typename T, bool OUT>
__global__ __launch_bounds__(256) void k_wgrad_end(const bf16 *va, const T *f, const double *s, float *part, int H,
                                                   int W, int nz, int dzo, int tiles_x, int chunks, int ru,
                                                   int64_t nunits) {
    constexpr int NWL = OUT ? K9 + 1 : K9 + C;
    __shared__ float red[NWL];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ch = lane & 3;
    const int64_t HW = (int64_t)H * W;
    float acc[8][9], db[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        db[k] = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[k][t] = 0.0f;
    }
    for (int64_t n = (int64_t)blockIdx.x * 4 + wave; n < nunits; n += (int64_t)gridDim.x * 4) {
        const Unit u = unit_of(n, ENS, tiles_x, chunks, ru, H);
        const int x = u.x0 + (lane >> 2);
        const bool ok = x < W;
        const int xc = ok ? x : W - 1, xm = wrap(xc - 1, W), xp = wrap(xc + 1, W);
        const T *fp = f + plane_shift(u.b, nz, OUT ? -dzo : dzo) * HW;
        const float inv = OUT ? 1.0f : (float)(1.0 / s[u.b / nz]);
        const bf16 *vp = va + (u.b * HW + xc) * C + ch * 8;
        float w[3][3];
        auto row = [&](int y, float (&r)[3]) {
            const T *q = fp + (int64_t)wrap(y, H) * W;
            r[0] = (float)q[xm] * inv;
            r[1] = (float)q[xc] * inv;
            r[2] = (float)q[xp] * inv;
        };
        uint4 nv = *reinterpret_cast<const uint4 *>(vp + (int64_t)u.ya * W * C);
        float nr[3];
        row(u.ya - 1, w[1]);
        row(u.ya, w[2]);
        row(u.ya + 1, nr);
        for (int y = u.ya; y < u.yb; ++y) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                w[0][k] = w[1][k];
                w[1][k] = w[2][k];
                w[2][k] = nr[k];
            }
            alignas(16) bf16 v[8];
            *reinterpret_cast<uint4 *>(v) = nv;
            if (y + 1 < u.yb) {
                nv = *reinterpret_cast<const uint4 *>(vp + (int64_t)(y + 1) * W * C);
                row(y + 2 > H ? y + 2 - H : y + 2, nr);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float val = ok ? (float)v[k] : 0.0f;  // points outside the field contribute nothing
#pragma unroll
                for (int t = 0; t < 9; ++t) acc[k][t] += val * (OUT ? w[2 - t / 3][2 - t % 3] : w[t / 3][t % 3]);
                if constexpr (!OUT) db[k] += val;
            }
            if constexpr (OUT) db[0] += ok ? w[1][1] : 0.0f;
        }
    }
    // the 16 points of a wave, then the waves in order
    auto points = [&](float v) {
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
        return v;
    };
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        db[k] = points(db[k]);
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[k][t] = points(acc[k][t]);
    }
    for (int i = tid; i < NWL; i += 256) red[i] = 0.0f;
    __syncthreads();
    for (int wv = 0; wv < 4; ++wv) {
        if (wave == wv && lane < 4) {
            auto put = [&](int i, float v) { red[i] += v; };
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int c = ch * 8 + k;
#pragma unroll
                for (int t = 0; t < 9; ++t) put(OUT ? t * C + c : c * 9 + t, acc[k][t]);
                if constexpr (!OUT) put(K9 + c, db[k]);
            }
            if constexpr (OUT)
                if (ch == 0) put(K9, db[0]);
        }
        __syncthreads();
    }
    for (int i = tid; i < NWL; i += 256) part[(int64_t)blockIdx.x * NWL + i] = red[i];
}

// Weight gradient of a 32 -> 32 layer (one 3x3 slice, the input read from the
// plane shifted by dzo) on the matrix cores: for every tap t the 32 x 32
// block dW[o][t][c] = sum_p g[p][o] x[p + off(t)][c] is a product over points.
// Its operands hold one channel per lane and 8 points per register group,
// the transpose of what a load gives (one point per lane, 8 channels).  The
// matrix cores transpose: points x channels times the identity (exact, one
// nonzero term per element) comes back with one channel per lane and 16 of
// the 32 points in its registers, in an order that is the same for g and x, so
// the product over points may use it as it is.  A wave marches down a strip
// of 32 columns with one x-shift of the input: an input row meets the
// transposed gradient rows above, at and below it, six products and four for
// the transposes per row, no LDS (all three shifts in one wave need 144
// accumulators: two waves per SIMD with one row in flight took 208 us).  Also db[o] = sum_p g[p][o].  part[block][32*288+32].
// Bound by reading g and x once (128 bytes per point): transposing through
// LDS with 2-byte accesses took 725 us for 8 x 512^2; this takes 100 us.
constexpr size_t kWgradLds = (size_t)(C * K + C) * sizeof(float);
constexpr int WGT = 384;  // six waves: two units, three x-shifts each
__global__ __launch_bounds__(WGT, 3) void k_wgrad_mid(const bf16 *xa, const bf16 *ga, float *part, int H, int W,
                                                      int nz, int dzo, int tiles_x, int chunks, int ru,
                                                      int64_t nunits) {
    constexpr int NWL = C * K + C;
    extern __shared__ __attribute__((aligned(16))) unsigned char wgrad_lds[];
    float *red = reinterpret_cast<float *>(wgrad_lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, kh = lane >> 5;
    const int sub = wave / 3, dx = wave - 3 * sub;  // this wave's unit of the two, and its taps (dy, dx)
    const int64_t HW = (int64_t)H * W;
    bf16x8 Id[2];  // identity: row k = 16 half + 8 kh + e, column j
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) Id[h][e] = (bf16)(16 * h + 8 * kh + e == j ? 1.0f : 0.0f);
    f32x16 acc[3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) acc[dy] = f32x16{};
    float db = 0.0f;
    struct Row {
        bf16x8 h[2];
    };
    // one channel per lane; the values are bf16 numbers, so the upper halves hold them
    auto transpose = [&](const Row &r, bf16x8 (&o)[2]) {
        f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r.h[0], Id[0], f32x16{}, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r.h[1], Id[1], d, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint4 p;
            auto pk = [&](int e) {
                const float lo = d[8 * q + e], hi = d[8 * q + e + 1];
                return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo),
                                             0x07060302u);
            };
            p.x = pk(0);
            p.y = pk(2);
            p.z = pk(4);
            p.w = pk(6);
            o[q] = __builtin_bit_cast(bf16x8, p);
        }
        return d;
    };
    const bf16x8 zero = {};
    // this lane's column of a unit's gradient and, with the wave's shift, of its input
    auto g_column = [&](const Unit &u) {
        return ga + u.b * HW * C + (int64_t)min(u.x0 + j, W - 1) * C + kh * 8;
    };
    auto x_column = [&](const Unit &u) {
        const int c = u.x0 + j + dx - 1;
        return xa + plane_shift(u.b, nz, dzo) * HW * C + kh * 8 +
               (int64_t)(c < 0 ? c + W : (c >= W ? (c == W ? 0 : W - 1) : c)) * C;
    };
    auto load_row = [&](const bf16 *column, int y, Row &r) {
        const bf16 *q = column + (int64_t)y * W * C;
        r.h[0] = *reinterpret_cast<const bf16x8 *>(q);
        r.h[1] = *reinterpret_cast<const bf16x8 *>(q + 16);
    };
    for (int64_t n = (int64_t)blockIdx.x * 2 + sub; n < nunits; n += (int64_t)gridDim.x * 2) {
        const Unit u = unit_of(n, TX, tiles_x, chunks, ru, H);
        const bool ok = u.x0 + j < W;
        const bf16 *gp = g_column(u), *xp = x_column(u);
        auto load_g = [&](int y, Row &r) { load_row(gp, min(y, u.yb - 1), r); };  // rows past the unit are loaded again and not used
        auto load_x = [&](int y, Row &r) { load_row(xp, wrap(min(y, u.yb), H), r); };
        // step r: input row r against the gradient rows r + 1 (dy = 0), r (1)
        // and r - 1 (2); two rows of loads in flight
        bf16x8 G0[2], G1[2], G2[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) G0[q] = G1[q] = G2[q] = zero;
        Row ga_[2], xa_[2];
        load_g(u.ya, ga_[0]);
        load_x(u.ya - 1, xa_[0]);
        load_g(u.ya + 1, ga_[1]);
        load_x(u.ya, xa_[1]);
        auto step = [&](int r, Row &gn, Row &xn) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                G2[q] = G1[q];
                G1[q] = G0[q];
            }
            if (r + 1 < u.yb) {
                if (!ok) gn.h[0] = gn.h[1] = zero;  // points outside the field contribute nothing
                const f32x16 d = transpose(gn, G0);
                float sum = 0.0f;
#pragma unroll
                for (int v = 0; v < 16; ++v) sum += d[v];
                db += sum;
            } else {
                G0[0] = G0[1] = zero;
            }
            bf16x8 X[2];
            transpose(xn, X);
            load_g(r + 3, gn);
            load_x(r + 2, xn);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(G0[q], X[q], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(G1[q], X[q], acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(G2[q], X[q], acc[2], 0, 0, 0);
            }
        };
        for (int r = u.ya - 1; r <= u.yb; r += 2) {
            step(r, ga_[0], xa_[0]);
            if (r + 1 <= u.yb) step(r + 1, ga_[1], xa_[1]);
        }
    }
    // An infinity or NaN in one channel of a point comes back from the
    // transpose as NaN in all 32 (0 times it), and any of the sums is NaN then:
    // the sums are taken again, the transposes through LDS.
    float zeros[4] = {db * 0.0f, 0.0f, 0.0f, 0.0f};  // 0, or NaN from an infinity or NaN
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) zeros[dy + 1] = __builtin_fmaf(acc[dy][v], 0.0f, zeros[dy + 1]);
    if (__any(!(zeros[0] + zeros[1] + zeros[2] + zeros[3] == 0.0f))) {
        bf16 *stage = reinterpret_cast<bf16 *>(wgrad_lds) + wave * TX * C;  // this wave's: [point][channel]
        auto transpose_lds = [&](const Row &r, bf16x8 (&o)[2]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<bf16x8 *>(stage + j * C + 16 * h + 8 * kh) = r.h[h];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int v = 0; v < 16; ++v) o[v >> 3][v & 7] = stage[(8 * (v >> 2) + 4 * kh + (v & 3)) * C + j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        };
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) acc[dy] = f32x16{};
        db = 0.0f;
        for (int64_t n = (int64_t)blockIdx.x * 2 + sub; n < nunits; n += (int64_t)gridDim.x * 2) {
            const Unit u = unit_of(n, TX, tiles_x, chunks, ru, H);
            const bool ok = u.x0 + j < W;
            const bf16 *gp = g_column(u), *xp = x_column(u);
#pragma unroll 1
            for (int r = u.ya - 1; r <= u.yb; ++r) {
                Row row;
                bf16x8 X[2], G[2];
                load_row(xp, wrap(r, H), row);
                if (!ok) row.h[0] = row.h[1] = zero;
                transpose_lds(row, X);
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int y = r + 1 - dy;
                    if (y < u.ya || y >= u.yb) continue;
                    load_row(gp, y, row);
                    if (!ok) row.h[0] = row.h[1] = zero;
                    transpose_lds(row, G);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        acc[dy] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(G[q], X[q], acc[dy], 0, 0, 0);
                        if (dy == 1)
#pragma unroll
                            for (int e = 0; e < 8; ++e) db += (float)G[q][e];
                    }
                }
            }
        }
    }
    db += __shfl_xor(db, 32, 64);
    __syncthreads();  // no wave stages in `red` any more
    for (int i = tid; i < NWL; i += WGT) red[i] = 0.0f;
    __syncthreads();
    for (int sv = 0; sv < 2; ++sv) {  // the three shifts of a unit write different taps
        if (sub == sv) {
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    red[((8 * (v >> 2) + 4 * kh + (v & 3)) * 9 + 3 * dy + dx) * C + j] += acc[dy][v];
            if (dx == 0 && lane < C) red[C * K + j] += db;
        }
        __syncthreads();
    }
    for (int i = tid; i < NWL; i += WGT) part[(int64_t)blockIdx.x * NWL + i] = red[i];
}

// grad = sum over blocks (in a fixed order) of part[block][w], where part
// holds one 3x3 slice [o][9][c] + biases; slice dzi of NT taps is scattered to
// W[o][dzi * 9 + t][c] (the identity in 2D) and the biases are written by the
// slice `bias_dzi` only.  grad points at the layer's first weight.
__global__ void k_reduce(const float *part, int nblk, int nw, float *grad, int NT, int dzi, int bias_dzi, int CI,
                         int CO) {
    // 32 weights per workgroup, 32 lanes per weight summing every 32nd block,
    // then the 32 lane sums in lane order: a fixed order for every run
    __shared__ double red[32][32];
    const int wl = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + wl;
    double acc = 0.0;
    if (i < nw)
#pragma unroll 4
        for (int k = g; k < nblk; k += 32) acc += (double)part[(int64_t)k * nw + i];
    red[g][wl] = acc;
    __syncthreads();
    if (g == 0 && i < nw) {
        double t = 0.0;
        for (int q = 0; q < 32; ++q) t += red[q][wl];
        const int nwt = CO * 9 * CI;
        if (i < nwt) {
            const int o = i / (9 * CI), tp = (i / CI) % 9, c = i % CI;
            grad[((int64_t)o * NT + dzi * 9 + tp) * CI + c] = (float)t;
        } else if (dzi == bias_dzi) {
            grad[(int64_t)CO * NT * CI + (i - nwt)] = (float)t;
        }
    }
}

__global__ void k_adam(float *p, float *m, float *v, const float *g, int64_t n, const int32_t *step, float lr, float b1,
                       float b2, float eps) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int t = step[0] + 1;
    const float bc1 = (float)(1.0 - pow((double)b1, (double)t));
    const float bc2 = (float)(1.0 - pow((double)b2, (double)t));
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

__global__ void k_step_inc(int32_t *step) {
    if (blockIdx.x == 0 && threadIdx.x == 0) step[0] = step[0] + 1;
}

// ---------------------------------------------------------------- host side

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    gd::set_error_text(buf);
    return code;
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct Layout {
    size_t wbf, wend, wT, wf, s, rms, act, z, zt, y, dy, dyz, dz, lpart, wpart, grad, total;
    int64_t N, nblk_pix;
    int nblk_w;
};

int taps_of(int ndim) { return ndim == 3 ? 27 : 9; }
int64_t planes_of(const gd_grid *g) { return g->batch * (g->ndim == 3 ? g->n[2] : 1); }

// Weight-gradient work: rows per unit (the two halo rows of a unit are work on
// top), halved down to 8 until the units of `strip` columns occupy 512
// workgroups of `per` units.
constexpr int kWgradBlocks = 512;
struct Units {
    int tiles_x, chunks, ru, per;
    int64_t n;
};
// units a workgroup works on at a time: k_wgrad_mid two, k_wgrad_end one per wave
int units_per_block(int strip) { return strip == TX ? 2 : 4; }
Units units_of(const gd_grid *g, int strip) {
    const int per = units_per_block(strip);
    Units u;
    u.tiles_x = (int)((g->n[0] + strip - 1) / strip);
    for (u.ru = 64;; u.ru /= 2) {
        u.chunks = (int)((g->n[1] + u.ru - 1) / u.ru);
        u.n = planes_of(g) * u.tiles_x * u.chunks;
        if (u.ru == 8 || u.n >= (int64_t)per * kWgradBlocks) break;
    }
    u.per = per;
    return u;
}
int blocks_of(const Units &u) { return (int)std::min<int64_t>((u.n + u.per - 1) / u.per, kWgradBlocks); }

// applications of G to the network's output (the struct's 0 means 1)
int smooth_of(const gd_cnn *net) { return net->smooth > 0 ? net->smooth : 1; }
constexpr int kMaxSmooth = 8;

Layout layout(const gd_grid *g, bool training, bool own_grad, int smooth) {
    const int NT = taps_of(g->ndim), ndz = NT / 9;
    const Offsets off = offsets(NT);
    Layout L;
    std::memset(&L, 0, sizeof L);
    L.N = planes_of(g) * g->n[0] * g->n[1];
    L.nblk_pix = (L.N + 255) / 256;
    L.nblk_w = blocks_of(units_of(g, TX));
    const size_t slices = (size_t)NMID * ndz * C * K9 * 2;  // bf16 weight slices of the 32 -> 32 layers
    size_t o = 0;
    L.wbf = o;
    o = align_up(o + (size_t)off.total * 2, 256);
    L.wend = o;
    o = align_up(o + (size_t)2 * C * NT * 4, 256);
    L.wT = o;
    if (training) o = align_up(o + slices, 256);
    L.wf = o;
    if (ndz > 1) o = align_up(o + slices, 256);
    L.s = o;
    o = align_up(o + (size_t)g->batch * 8, 256);
    L.rms = o;
    o = align_up(o + (size_t)g->batch * RMS_CHUNKS * 8, 256);
    L.act = o;
    const size_t actb = align_up((size_t)L.N * C * 2, 256);
    o += (training ? NL - 1 : 2) * actb;
    L.z = o;
    o = align_up(o + (size_t)L.N * 4, 256);
    L.zt = o;  // the second buffer of G^m z (m > 1)
    if (smooth > 1) o = align_up(o + (size_t)L.N * 4, 256);
    if (training) {
        L.y = o;
        o = align_up(o + (size_t)L.N * 4, 256);
        L.dy = o;
        o = align_up(o + (size_t)L.N * 4, 256);
        L.dyz = o;
        o = align_up(o + (size_t)L.N * 4, 256);
        L.dz = o;
        o += 2 * actb;
        L.lpart = o;
        o = align_up(o + (size_t)L.nblk_pix * 8, 256);
        L.wpart = o;
        o = align_up(o + std::max((size_t)L.nblk_w * NW_MID, (size_t)blocks_of(units_of(g, ENS)) * NW_END) * 4, 256);
        if (own_grad) {
            L.grad = o;
            o = align_up(o + (size_t)off.total * 4, 256);
        }
    }
    L.total = o;
    return L;
}

int check_net(const gd_cnn *net, bool training) {
    if (!net) return fail(GD_EINVAL, "network is NULL");
    if (net->ndim != 2 && net->ndim != 3) return fail(GD_EINVAL, "the network is 2D or 3D (ndim %d)", net->ndim);
    if (net->channels != C || net->layers != NL)
        return fail(GD_EINVAL, "the network has %d layers of %d channels", NL, C);
    if (!net->params) return fail(GD_EINVAL, "params is NULL");
    if (net->smooth < 0 || net->smooth > kMaxSmooth)
        return fail(GD_EINVAL, "smooth must be 0 .. %d (got %d)", kMaxSmooth, net->smooth);
    if (training && (!net->adam_m || !net->adam_v || !net->step))
        return fail(GD_EINVAL, "training needs adam_m, adam_v and step");
    return GD_OK;
}

int check_grid(const gd_cnn *net, const gd_grid *g) {
    if (!g) return fail(GD_EINVAL, "grid is NULL");
    if (g->ndim != net->ndim) return fail(GD_EINVAL, "a %dD network needs %dD fields", net->ndim, net->ndim);
    if (g->dtype != GD_F32 && g->dtype != GD_F64) return fail(GD_EINVAL, "dtype must be GD_F32 or GD_F64");
    if (g->n[0] < 1 || g->n[1] < 1 || g->batch < 1 || (g->ndim == 3 && g->n[2] < 1))
        return fail(GD_EINVAL, "sizes must be >= 1");
    // bound the factors before multiplying them
    if (g->batch > 65535 || (g->ndim == 3 && g->n[2] > (int64_t(1) << 24))) return fail(GD_EINVAL, "field too large");
    const int64_t planes = planes_of(g), n01 = gd::checked_points(g->n, 2, (int64_t(1) << 31) - 1);
    if (n01 < 0 || planes > (int64_t(1) << 24) || planes > (int64_t(1) << 34) / n01)
        return fail(GD_EINVAL, "field too large");
    return GD_OK;
}

#define GD_LAUNCH(...)                                                                   \
    do {                                                                                 \
        hipLaunchKernelGGL(__VA_ARGS__);                                                 \
        hipError_t e_ = hipGetLastError();                                               \
        if (e_ != hipSuccess) return fail(GD_EHIP, "launch: %s", hipGetErrorString(e_)); \
    } while (0)

template <int MODE>
int launch_mid2(const gd_grid *g, const bf16 *in, const bf16 *wmat, const float *bias, const bf16 *mask, bf16 *out,
                hipStream_t st) {
    const int H = (int)g->n[1], W = (int)g->n[0];
    const int tiles_x = (W + TX - 1) / TX, tiles_y = (H + 4 * RB - 1) / (4 * RB);
    const int64_t blk = planes_of(g) * tiles_x * tiles_y;
    if (blk > 0x7fffffff) return fail(GD_EINVAL, "field too large");
    auto kern = k_conv_mid<MODE>;
    GD_LAUNCH(kern, dim3((unsigned)blk), dim3(256), kConvLds, st, in, wmat, bias, mask, out, H, W, tiles_x,
              tiles_y);
    return GD_OK;
}

template <int MODE>
int launch_mid3(const gd_grid *g, const bf16 *in, const bf16 *slices, const float *bias, const bf16 *mask, bf16 *out,
                hipStream_t st) {
    const int H = (int)g->n[1], W = (int)g->n[0], nz = (int)g->n[2];
    const int tiles_x = (W + TX - 1) / TX, tiles_y = (H + 4 * RB - 1) / (4 * RB);
    const int64_t cols = g->batch * tiles_x * tiles_y;
    // planes per run: the runs of one round fill the 256 CUs (one workgroup
    // each); a run costs two planes more to load, and about one plane's time
    // to start, so the rounds x (planes + 1) are minimised
    int zrun = nz;
    int64_t best = INT64_MAX;
    for (int r = 1; r <= nz; ++r) {
        const int len = (nz + r - 1) / r;
        const int64_t rounds = (cols * ((nz + len - 1) / len) + 255) / 256, cost = rounds * (len + 1);
        if (cost < best) {
            best = cost;
            zrun = len;
        }
        if (rounds > 64 && r > 1) break;
    }
    const int zruns = (nz + zrun - 1) / zrun;
    const int64_t blk = cols * zruns;
    if (blk > 0x7fffffff) return fail(GD_EINVAL, "field too large");
    const bool wide = (int64_t)H * W > int64_t(1) << 30;
    const auto kern = wide ? k_conv_mid3<MODE, true> : k_conv_mid3<MODE, false>;
    GD_LAUNCH(kern, dim3((unsigned)blk), dim3(256), 4 * kConvLds, st, in, slices, bias, mask, out, H, W, nz,
              tiles_x, tiles_y, zruns, zrun);
    return GD_OK;
}

// One 32 -> 32 layer (forward, or its input gradient with bwd).
int mid_layer(bool bwd, const gd_grid *g, const bf16 *in, const bf16 *slices, const float *bias, const bf16 *mask,
              bf16 *out, hipStream_t st) {
    if (g->ndim == 3)
        return bwd ? launch_mid3<kBwd>(g, in, slices, bias, mask, out, st)
                   : launch_mid3<kFwd>(g, in, slices, bias, mask, out, st);
    return bwd ? launch_mid2<kBwd>(g, in, slices, bias, mask, out, st)
               : launch_mid2<kFwd>(g, in, slices, bias, mask, out, st);
}

// Planes per run of a 3D end layer: at most `most`, fewer (at least `least`)
// where that leaves fewer than `want` workgroups.  A run loads two planes more
// than it has.  1 x 32^3 with runs of 16: layer 1 131 us, layer 6 33 us, for 4
// workgroups; with short runs the whole forward takes 89 us (125 before the
// layers marched along z), 2 x 64^3 187 (470).
int run_planes(int64_t cols, int nz, int most, int least, int64_t want) {
    return (int)std::max<int64_t>(least, std::min<int64_t>(most, cols * nz / want));
}

// layer 1, or with mask the input gradient of layer 6 (in = dL/dz)
template <typename T, bool GRAD>
int end_layer(const gd_grid *g, const T *in, const double *s, const float *wt, const float *bias, const bf16 *mask,
              bf16 *out, hipStream_t st) {
    const int H = (int)g->n[1], W = (int)g->n[0], nz = g->ndim == 3 ? (int)g->n[2] : 1;
    const int tiles_x = (W + 63) / 64, tiles_y = (H + 4 * EPT - 1) / (4 * EPT);
    const int zrun = run_planes(g->batch * tiles_x * tiles_y, nz, EZ, 1, 1024), zruns = (nz + zrun - 1) / zrun;
    const int64_t blk = (int64_t)g->batch * tiles_x * tiles_y * zruns;
    if (blk > 0x7fffffff) return fail(GD_EINVAL, "field too large");
    auto k2 = k_conv_end<T, 9, GRAD>;
    auto k3 = k_conv_end<T, 27, GRAD>;
    GD_LAUNCH(g->ndim == 2 ? k2 : k3, dim3((unsigned)blk), dim3(256), 0, st, in, s, wt, bias, mask, out, H, W, nz,
              tiles_x, tiles_y, zruns, zrun);
    return GD_OK;
}

// layer 6
int out_layer(const gd_grid *g, const bf16 *a, const bf16 *w6, const float *b6, float *z, hipStream_t st) {
    const int H = (int)g->n[1], W = (int)g->n[0], nz = g->ndim == 3 ? (int)g->n[2] : 1;
    const int tiles_x = (W + OX - 1) / OX, tiles_y = (H + OY - 1) / OY;
    const int zrun = run_planes(g->batch * tiles_x * tiles_y, nz, OZ, 2, 512), zruns = (nz + zrun - 1) / zrun;
    const int64_t blk = (int64_t)g->batch * tiles_x * tiles_y * zruns;
    if (blk > 0x7fffffff) return fail(GD_EINVAL, "field too large");
    GD_LAUNCH(g->ndim == 2 ? k_conv_out<9> : k_conv_out<27>, dim3((unsigned)blk), dim3(256), 0, st, a, w6, b6, z, H, W,
              nz, tiles_x, tiles_y, zruns, zrun);
    return GD_OK;
}

// y = G^m z: m - 1 filter passes ping-ponging between z and zt, then the last
// one fused with u0 = ubar + s y (inference) or writing y (training)
template <typename T>
int finish_forward(const gd_cnn *net, const Layout &L, char *w, const T *ub, T *u0, bool train, int H, int W, int nz,
                   hipStream_t st) {
    const int64_t N = L.N;
    const unsigned pblk = (unsigned)L.nblk_pix;
    const double *s = (const double *)(w + L.s);
    const float *zin = (const float *)(w + L.z);
    for (int k = 1; k < smooth_of(net); ++k) {
        float *zo = (k & 1) ? (float *)(w + L.zt) : (float *)(w + L.z);
        GD_LAUNCH(k_gfilt, dim3(pblk), dim3(256), 0, st, zin, zo, H, W, nz, N);
        zin = zo;
    }
    GD_LAUNCH(k_gfin<T>, dim3(pblk), dim3(256), 0, st, zin, ub, s, train ? (float *)(w + L.y) : (float *)nullptr,
              train ? (T *)nullptr : u0, H, W, nz, N);
    return GD_OK;
}

// forward (train = false: u0 out; train = true: keep every activation and y)
template <typename T>
int run_forward(const gd_cnn *net, const gd_grid *g, const Layout &L, char *w, const T *ub, T *u0, bool train,
                hipStream_t st) {
    const int NT = taps_of(g->ndim), ndz = NT / 9;
    const Offsets off = offsets(NT);
    const int H = (int)g->n[1], W = (int)g->n[0], nz = g->ndim == 3 ? (int)g->n[2] : 1;
    const int64_t P = (int64_t)H * W * nz, N = L.N;
    bf16 *wbf = (bf16 *)(w + L.wbf);
    double *s = (double *)(w + L.s);
    const size_t actb = align_up((size_t)N * C * 2, 256);
    auto act = [&](int i) { return (bf16 *)(w + L.act + (size_t)i * actb); };
    const unsigned pblk = (unsigned)L.nblk_pix;
    float *wend = (float *)(w + L.wend);
    GD_LAUNCH(k_cvt, dim3((unsigned)((off.total + 255) / 256)), dim3(256), 0, st, net->params, wbf, off.total, wend,
              off.W[0], off.W[NL - 1], NT);
    bf16 *wf = (bf16 *)(w + L.wf);  // 3D: forward weight slices
    if (ndz > 1)
        GD_LAUNCH(k_repack<false>, dim3((unsigned)((NMID * ndz * C * K9 + 255) / 256)), dim3(256), 0, st,
                  (const bf16 *)wbf, off.W[1], off.W[2] - off.W[1], NT, wf);
    GD_LAUNCH(k_rms_part<T>, dim3(RMS_CHUNKS, (unsigned)g->batch), dim3(256), 0, st, ub, P, (double *)(w + L.rms));
    GD_LAUNCH(k_rms_fin, dim3((unsigned)((g->batch + 63) / 64)), dim3(64), 0, st, (const double *)(w + L.rms),
              (int)g->batch, P, s);
    if (NT == 9 && !train) {  // 2D inference: the six layers in one kernel
        const dim3 grid((unsigned)((W + FV - 1) / FV), (unsigned)((H + FY - 1) / FY), (unsigned)g->batch);
        GD_LAUNCH(k_fwd2d_fused<T>, grid, dim3(FTHREADS), kFusedLds, st, ub, (const double *)s, (const bf16 *)wbf,
                  (const float *)net->params, off, (float *)(w + L.z), H, W);
        return finish_forward<T>(net, L, w, ub, u0, false, H, W, nz, st);
    }
    int rc;
    if ((rc = end_layer<T, false>(g, ub, s, wend, net->params + off.b[0], nullptr, act(0), st))) return rc;
    for (int m = 0; m < NMID; ++m) {
        const int l = m + 1;
        bf16 *src = train ? act(m) : act(m & 1);
        bf16 *dst = train ? act(m + 1) : act((m + 1) & 1);
        const bf16 *slices = ndz > 1 ? wf + (size_t)m * ndz * C * K9 : wbf + off.W[l];
        if ((rc = mid_layer(false, g, src, slices, net->params + off.b[l], nullptr, dst, st))) return rc;
    }
    bf16 *last = train ? act(NL - 2) : act(NMID & 1);
    if ((rc = out_layer(g, last, wbf + off.W[NL - 1], net->params + off.b[NL - 1], (float *)(w + L.z), st))) return rc;
    return finish_forward<T>(net, L, w, ub, u0, train, H, W, nz, st);
}

// Weight gradient of a layer into grad_layer (its first weight): one pass per
// 3x3 slice (dz), each reduced and scattered into place.  CI, CO: 32 -> 32
// (v = dz at the output, x its input), 1 -> 32 (v = dz, f = ubar) or 32 -> 1
// (v = a5, f = dL/dz).
template <int CI, int CO, typename T>
int wgrad_layer(const gd_grid *g, const Layout &L, char *w, const bf16 *x, const bf16 *v, const T *f, const double *s,
                float *grad_layer, hipStream_t st) {
    constexpr int NWL = CO * 9 * CI + CO;
    const int NT = taps_of(g->ndim), ndz = NT / 9;
    const int H = (int)g->n[1], W = (int)g->n[0], nz = g->ndim == 3 ? (int)g->n[2] : 1;
    const Units u = units_of(g, CI == C && CO == C ? TX : ENS);
    const int blocks = blocks_of(u);
    float *part = (float *)(w + L.wpart);
    for (int dzi = 0; dzi < ndz; ++dzi) {
        const int dzo = ndz > 1 ? dzi - 1 : 0;
        if constexpr (CI == C && CO == C) {
            GD_LAUNCH(k_wgrad_mid, dim3((unsigned)blocks), dim3(WGT), kWgradLds, st, x, v, part, H, W, nz, dzo,
                      u.tiles_x, u.chunks, u.ru, u.n);
        } else {
            auto kern = k_wgrad_end<T, CO == 1>;
            GD_LAUNCH(kern, dim3((unsigned)blocks), dim3(256), 0, st, v, f, s, part, H, W, nz, dzo, u.tiles_x,
                      u.chunks, u.ru, u.n);
        }
        GD_LAUNCH(k_reduce, dim3((NWL + 31) / 32), dim3(1024), 0, st, (const float *)part, blocks, NWL, grad_layer, NT,
                  dzi, (ndz - 1) / 2, CI, CO);
    }
    return GD_OK;
}

template <typename T>
int run_train(const gd_cnn *net, const gd_grid *g, const Layout &L, char *w, const T *ub, const T *u, double *loss,
              hipStream_t st) {
    const int NT = taps_of(g->ndim), ndz = NT / 9;
    const Offsets off = offsets(NT);
    int rc = run_forward<T>(net, g, L, w, ub, nullptr, true, st);
    if (rc) return rc;
    const int H = (int)g->n[1], W = (int)g->n[0], nz = g->ndim == 3 ? (int)g->n[2] : 1;
    const int64_t P = (int64_t)H * W * nz, N = L.N;
    bf16 *wbf = (bf16 *)(w + L.wbf);
    bf16 *wT = (bf16 *)(w + L.wT);
    const double *s = (const double *)(w + L.s);
    const size_t actb = align_up((size_t)N * C * 2, 256);
    auto act = [&](int i) { return (bf16 *)(w + L.act + (size_t)i * actb); };
    auto dz = [&](int i) { return (bf16 *)(w + L.dz + (size_t)(i & 1) * actb); };
    float *grad = net->grad ? net->grad : (float *)(w + L.grad);
    float *dy = (float *)(w + L.dy);
    const unsigned pblk = (unsigned)L.nblk_pix;
    GD_LAUNCH(k_repack<true>, dim3((unsigned)((NMID * ndz * C * K9 + 255) / 256)), dim3(256), 0, st, (const bf16 *)wbf,
              off.W[1], off.W[2] - off.W[1], NT, wT);
    GD_LAUNCH(k_loss<T>, dim3(pblk), dim3(256), 0, st, (const float *)(w + L.y), ub, u, s, dy,
              (double *)(w + L.lpart), P, N);
    GD_LAUNCH(k_loss_fin, dim3(1), dim3(256), 0, st, (const double *)(w + L.lpart), L.nblk_pix, N, loss);
    // through the final filters: dL/dz = G^m dL/dy (G is symmetric), m passes
    // ping-ponging between dyz and dy
    float *dyz = (float *)(w + L.dyz);
    {
        const float *gin = dy;
        for (int k = 0; k < smooth_of(net); ++k) {
            float *go = (k & 1) ? dy : (float *)(w + L.dyz);
            GD_LAUNCH(k_gfilt, dim3(pblk), dim3(256), 0, st, gin, go, H, W, nz, N);
            gin = go;
        }
        dyz = const_cast<float *>(gin);
    }
    // layer 6
    if ((rc = wgrad_layer<C, 1, float>(g, L, w, nullptr, act(NL - 2), dyz, s, grad + off.W[NL - 1], st))) return rc;
    const float *w6 = (const float *)(w + L.wend) + C * NT;
    if ((rc = end_layer<float, true>(g, dyz, s, w6, nullptr, act(NL - 2), dz(0), st))) return rc;
    // layers 5 .. 2: dz(k) holds the gradient at the output of layer l
    int k = 0;
    for (int l = NL - 2; l >= 1; --l, ++k) {
        const bf16 *xin = act(l - 1);  // input activation of layer l
        if ((rc = wgrad_layer<C, C, T>(g, L, w, xin, dz(k), nullptr, s, grad + off.W[l], st))) return rc;
        if ((rc = mid_layer(true, g, dz(k), wT + (size_t)(l - 1) * ndz * C * K9, nullptr, xin, dz(k + 1), st)))
            return rc;
    }
    // layer 1 (input x0 = ubar / s)
    if ((rc = wgrad_layer<1, C, T>(g, L, w, nullptr, dz(k), ub, s, grad + off.W[0], st))) return rc;
    GD_LAUNCH(k_adam, dim3((unsigned)((off.total + 255) / 256)), dim3(256), 0, st, net->params, net->adam_m,
              net->adam_v, (const float *)grad, off.total, (const int32_t *)net->step, net->lr, net->beta1, net->beta2,
              net->eps);
    GD_LAUNCH(k_step_inc, dim3(1), dim3(64), 0, st, net->step);
    return GD_OK;
}

}  // namespace gdcnn

using namespace gdcnn;

extern "C" {

int64_t warmstart_param_count(const gd_cnn *net) {
    if (!net || (net->ndim != 2 && net->ndim != 3) || net->channels != C || net->layers != NL) return 0;
    return offsets(taps_of(net->ndim)).total;
}

size_t warmstart_workspace_bytes(const gd_cnn *net, const gd_grid *g, int32_t training) {
    if (check_net(net, false) || check_grid(net, g)) return 0;
    return layout(g, training != 0, !net->grad, smooth_of(net)).total;
}

int warmstart_forward(const gd_cnn *net, const gd_grid *g, const void *ubar, void *u0, void *work, size_t work_bytes,
                      void *stream) {
    int rc = check_net(net, false);
    if (rc) return rc;
    if ((rc = check_grid(net, g))) return rc;
    if (!ubar || !u0) return fail(GD_EINVAL, "ubar and u0 must be non-NULL");
    if (ubar == u0) return fail(GD_EINVAL, "ubar and u0 must differ");
    if (!work) return fail(GD_EWORKSPACE, "workspace is NULL");
    if ((uintptr_t)work % 256) return fail(GD_EALIGN, "workspace must be 256-byte aligned");
    const Layout L = layout(g, false, false, smooth_of(net));
    if (work_bytes < L.total) return fail(GD_EWORKSPACE, "workspace too small: need %zu bytes", L.total);
    hipStream_t st = (hipStream_t)stream;
    if (g->dtype == GD_F32)
        return run_forward<float>(net, g, L, (char *)work, (const float *)ubar, (float *)u0, false, st);
    return run_forward<double>(net, g, L, (char *)work, (const double *)ubar, (double *)u0, false, st);
}

int warmstart_train_step(const gd_cnn *net, const gd_grid *g, const void *ubar, const void *u, void *work,
                         size_t work_bytes, double *loss, void *stream) {
    int rc = check_net(net, true);
    if (rc) return rc;
    if ((rc = check_grid(net, g))) return rc;
    if (!ubar || !u || !loss) return fail(GD_EINVAL, "ubar, u and loss must be non-NULL");
    if (!work) return fail(GD_EWORKSPACE, "workspace is NULL");
    if ((uintptr_t)work % 256) return fail(GD_EALIGN, "workspace must be 256-byte aligned");
    const Layout L = layout(g, true, !net->grad, smooth_of(net));
    if (work_bytes < L.total) return fail(GD_EWORKSPACE, "workspace too small: need %zu bytes", L.total);
    hipStream_t st = (hipStream_t)stream;
    if (g->dtype == GD_F32)
        return run_train<float>(net, g, L, (char *)work, (const float *)ubar, (const float *)u, loss, st);
    return run_train<double>(net, g, L, (char *)work, (const double *)ubar, (const double *)u, loss, st);
}

}  // extern "C"
