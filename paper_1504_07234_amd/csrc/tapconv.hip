// Tap-by-tap convolution on the vector units: every output is one chain of
// fused multiply-adds over the taps, row by row.  It serves the calls whose
// result hangs on the order of that sum:
//   - the single operators A u and g - A u: P multiplies the rounding of
//     g - A u by up to 1 / alpha (measured at 226 x 226, p = 31, alpha = 0.02:
//     another order of the sum moves P(g - A u) by 4e-5 of its size);
//   - iterations with the explicit state, which the unrolled form
//     differentiates: the gradient depends on the active sets {|z| > mu}, and a
//     coefficient within rounding of its threshold changes them (another order
//     moves the gradient of the observations by 6e-5 of its size at 16 x 256 x
//     256, p = 15, 30 iterations).
// The implicit state, A^T for p > 7 and the norm estimates use the matrix cores
// (conv.hip), whose sums are more accurate and whose A takes 18 / 25 / 73 us at
// 2048 x 2048 (p = 5 / 15 / 31) where these take 17 / 33 / 98.
// Bound by the vector units at large p (8.1 GFLOP in those 98 us) and on small
// images by the latency of staging the window.
//
// One workgroup computes a tile of 64 output columns; the input window is
// staged once in LDS under the requested boundary extension.  Every thread owns
// an RY x RX block of outputs and walks the p + RY - 1 input rows that feed it:
// each row segment (RX + p - 1 values) is loaded into registers once and
// applied to every output row it contributes to.  PSF taps are
// wavefront-uniform and are read through the scalar cache.  The PSF side is a
// template parameter for the odd sizes 1..33 (fully unrolled tap loops);
// larger PSFs use a generic body.  The arithmetic of an output does not depend
// on the shape of its tile.
#include "common.hpp"
#include "kernels.hpp"

namespace mlba {

constexpr int TAP_TX = 64;  // output columns per workgroup, RX of them per thread

// rows of a tile: 256 threads with RY x RX outputs each
__host__ __device__ constexpr int tap_ty(int ry, int rx) { return 4 * rx * ry; }

__host__ __device__ constexpr int tap_stride(int w) { return ((w + 7) / 8) * 8 + 1; }

__host__ __device__ constexpr int tap_lds_floats(int p, int ty) { return (ty + p - 1) * tap_stride(TAP_TX + p - 1); }

static int tap_tiles(int D, int ty) { return ((D + TAP_TX - 1) / TAP_TX) * ((D + ty - 1) / ty); }

template <int P, bool FLIP>
__device__ __forceinline__ float tap_of(const float* __restrict__ psf, int a, int b) {
    return FLIP ? psf[(P - 1 - a) * P + (P - 1 - b)] : psf[a * P + b];
}

__device__ __forceinline__ void tap_stage_window(const ConvJob& j, int P, int TY, int oy0, int ox0, float* tile) {
    const int TH = TY + P - 1;
    const int TW = TAP_TX + P - 1;
    const int LS = tap_stride(TW);
    for (int i = threadIdx.x; i < TH * TW; i += kBlock) {
        const int ly = i / TW;
        const int lx = i - ly * TW;
        tile[ly * LS + lx] = fetch_ext(j.src, j.S, oy0 + j.org + ly, ox0 + j.org + lx, j.ext);
    }
}

// The same with P known: a wave takes every fourth row's first 64 columns (the
// row's source is uniform), the columns after them lie row by row over the
// threads, and all loads are in flight before the first is stored.  Element by
// element the window was a chain of up to 14 round trips at p = 15: the batched
// blur of 16 x 256 x 256 took 21 us, now 15.6 (A^T 22 -> 17.5); 64 x 64, p = 9:
// 5.6 -> 4.6 us.
template <int P, int TY>
__device__ __forceinline__ void tap_stage(const ConvJob& j, int oy0, int ox0, float* tile) {
    constexpr int TH = TY + P - 1, LS = tap_stride(TAP_TX + P - 1);
    constexpr int WV = kBlock / 64, KM = (TH + WV - 1) / WV;  // rows of a wave
    constexpr int PT = P > 1 ? P - 1 : 1, NT = TH * (P - 1), KT = (NT + kBlock - 1) / kBlock;
    const int S = j.S, y0 = oy0 + j.org, x0 = ox0 + j.org;
    const bool inside = y0 >= 0 && x0 >= 0 && y0 + TH <= S && x0 + TAP_TX + P - 1 <= S;
    if (j.ext == EXT_ANTIREFLECT && !inside) return tap_stage_window(j, P, TY, oy0, ox0, tile);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float m[KM], t[KT > 0 ? KT : 1];
    bool hx;
    const int xs = ext_axis(x0 + lane, S, j.ext, &hx);
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        bool hy;
        const int ys = ext_axis(y0 + min(wave + k * WV, TH - 1), S, j.ext, &hy);
        const float v = j.src[(size_t)ys * S + xs];
        m[k] = hx && hy ? v : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int i = min((int)threadIdx.x + k * kBlock, NT - 1);
        bool hy, ht;
        const int ys = ext_axis(y0 + i / PT, S, j.ext, &hy), xt = ext_axis(x0 + TAP_TX + i % PT, S, j.ext, &ht);
        const float v = j.src[(size_t)ys * S + xt];
        t[k] = hy && ht ? v : 0.0f;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < KM; ++k)
        if (wave + k * WV < TH) tile[(wave + k * WV) * LS + lane] = m[k];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int i = (int)threadIdx.x + k * kBlock;
        if (i < NT) tile[(i / PT) * LS + TAP_TX + i % PT] = t[k];
    }
}

// Writes (g - s) or s for the thread's outputs; returns its sum of squares of
// the written residuals (0 without g).
template <int RY, int RX>
__device__ __forceinline__ double tap_store(const ConvJob& j, int oy0, int ox0, int ty, int tx0,
                                            const float (*acc)[RX]) {
    double ss = 0.0;
#pragma unroll
    for (int h = 0; h < RY; ++h) {
        const int y = oy0 + RY * ty + h;
        if (y < j.D) {
#pragma unroll
            for (int r = 0; r < RX; ++r) {
                const int x = ox0 + tx0 + r;
                if (x < j.D) {
                    const size_t i = (size_t)y * j.D + x;
                    float v = acc[h][r];
                    if (j.g) {
                        v = j.g[i] - v;
                        ss += (double)v * (double)v;
                    }
                    j.dst[i] = v;
                }
            }
        }
    }
    return ss;
}

// One output tile at tile coordinates (bx, by); `tile` is the LDS window.
template <int P, bool FLIP, int RY, int RX>
__device__ __forceinline__ double tap_tile(const ConvJob& j, int bx, int by, float* tile) {
    constexpr int TW = TAP_TX + P - 1;
    constexpr int LS = tap_stride(TW);  // 8k+1 row stride: rows start on distinct banks
    constexpr int TY = tap_ty(RY, RX), TPR = TAP_TX / RX;
    const int oy0 = by * TY;
    const int ox0 = bx * TAP_TX;
    tap_stage<P, TY>(j, oy0, ox0, tile);
    __syncthreads();

    // thread: output rows RY*ty .. RY*ty+RY-1, columns tx0 .. tx0+RX-1; input
    // row RY*ty + q feeds output row RY*ty + h with kernel row q - h
    const int ty = threadIdx.x / TPR;
    const int tx0 = (threadIdx.x % TPR) * RX;
    float acc[RY][RX];
#pragma unroll
    for (int h = 0; h < RY; ++h)
#pragma unroll
        for (int r = 0; r < RX; ++r) acc[h][r] = 0.0f;
#pragma unroll 1
    for (int q = 0; q < P + RY - 1; ++q) {
        const float* row = tile + (RY * ty + q) * LS + tx0;
        float seg[RX + P - 1];
#pragma unroll
        for (int k = 0; k < RX + P - 1; ++k) seg[k] = row[k];
#pragma unroll
        for (int h = 0; h < RY; ++h) {
            const int a = q - h;
            if (a >= 0 && a < P) {
#pragma unroll
                for (int b = 0; b < P; ++b) {
                    const float t = tap_of<P, FLIP>(j.psf, a, b);
#pragma unroll
                    for (int r = 0; r < RX; ++r) acc[h][r] = fmaf(t, seg[r + b], acc[h][r]);
                }
            }
        }
    }
    return tap_store<RY, RX>(j, oy0, ox0, ty, tx0, acc);
}

// Runtime PSF side, 64-row tile, taps read from LDS after the window.
constexpr int TAP_GENERIC_TY = 64;
__device__ __forceinline__ double tap_tile_generic(const ConvJob& j, int P, int flip, int bx, int by,
                                                   float* smem) {
    constexpr int RY = 2, RX = 8, TY = TAP_GENERIC_TY;
    const int LS = tap_stride(TAP_TX + P - 1);
    float* tile = smem;
    float* kern = smem + (TY + P - 1) * LS;
    const int oy0 = by * TY;
    const int ox0 = bx * TAP_TX;
    tap_stage_window(j, P, TY, oy0, ox0, tile);
    for (int i = threadIdx.x; i < P * P; i += kBlock) kern[i] = flip ? j.psf[P * P - 1 - i] : j.psf[i];
    __syncthreads();
    const int ty = threadIdx.x >> 3;
    const int tx0 = (threadIdx.x & 7) * RX;
    float acc[RY][RX];
    for (int h = 0; h < RY; ++h) {
#pragma unroll
        for (int r = 0; r < RX; ++r) acc[h][r] = 0.0f;
        for (int a = 0; a < P; ++a) {
            const float* row = tile + (RY * ty + h + a) * LS + tx0;
            for (int b = 0; b < P; ++b) {
                const float k = kern[a * P + b];
#pragma unroll
                for (int r = 0; r < RX; ++r) acc[h][r] = fmaf(k, row[r + b], acc[h][r]);
            }
        }
    }
    return tap_store<RY, RX>(j, oy0, ox0, ty, tx0, acc);
}

__device__ __forceinline__ void tap_partial(double ss, double* red, double* out) {
    const double t = block_sum(ss, red);
    if (threadIdx.x == 0) *out = t;
}

#define MLBA_TAP_SIDES(X) \
    X(1) X(3) X(5) X(7) X(9) X(11) X(13) X(15) X(17) X(19) X(21) X(23) X(25) X(27) X(29) X(31) X(33)

// ---- single image ----------------------------------------------------------

template <int P, bool FLIP, int RY, int RX>
__global__ __launch_bounds__(kBlock) void tapconv_kernel(ConvJob j, double* __restrict__ partials) {
    __shared__ float tile[tap_lds_floats(P, tap_ty(RY, RX))];
    __shared__ double red[kBlock / 64];
    int bx, by;
    xcd_tile(&bx, &by);
    const double ss = tap_tile<P, FLIP, RY, RX>(j, bx, by, tile);
    if (partials) tap_partial(ss, red, partials + blockIdx.y * gridDim.x + blockIdx.x);
}

__global__ __launch_bounds__(kBlock) void tapconv_kernel_generic(ConvJob j, int P, int flip,
                                                                 double* __restrict__ partials) {
    extern __shared__ float smem[];
    __shared__ double red[kBlock / 64];
    int bx, by;
    xcd_tile(&bx, &by);
    const double ss = tap_tile_generic(j, P, flip, bx, by, smem);
    if (partials) tap_partial(ss, red, partials + blockIdx.y * gridDim.x + blockIdx.x);
}

template <int P, int RY, int RX>
static hipError_t launch_tap(const ConvJob& j, int flip, double* partials, int* n_partials, hipStream_t s) {
    constexpr int TY = tap_ty(RY, RX);
    dim3 grid((j.D + TAP_TX - 1) / TAP_TX, (j.D + TY - 1) / TY);
    if (n_partials) *n_partials = (int)(grid.x * grid.y);
    if (flip) hipLaunchKernelGGL((tapconv_kernel<P, true, RY, RX>), grid, dim3(kBlock), 0, s, j, partials);
    else hipLaunchKernelGGL((tapconv_kernel<P, false, RY, RX>), grid, dim3(kBlock), 0, s, j, partials);
    return hipGetLastError();
}

bool tapconv_small(int D, int p) { return p <= 33 && tap_tiles(D, tap_ty(1, 8)) < 128; }

// Output tile: two columns a thread (8-row tiles) while 32-row tiles would
// leave most of the chip idle (at 226 x 226 and p = 31, 116 workgroups instead
// of 32); two rows a thread (64-row tiles, fewer LDS reads per multiply-add)
// unless that tiling leaves a nearly empty second round of workgroups; else
// one.
template <int P>
static hipError_t launch_tap_side(const ConvJob& j, int flip, double* partials, int* n_partials, hipStream_t s,
                                  bool tall) {
    if (!tall && tapconv_small(j.D, P)) return launch_tap<P, 1, 2>(j, flip, partials, n_partials, s);
    const long t2 = tap_tiles(j.D, tap_ty(2, 8));
    const int lds2 = tap_lds_floats(P, tap_ty(2, 8)) * 4;
    const long slots = 256L * (160 * 1024 / lds2);
    const long rounds = (t2 + slots - 1) / slots;
    return (double)t2 / (double)(rounds * slots) >= 0.75 ? launch_tap<P, 2, 8>(j, flip, partials, n_partials, s)
                                                         : launch_tap<P, 1, 8>(j, flip, partials, n_partials, s);
}

int tapconv_partials_count(int D) { return tap_tiles(D, tap_ty(1, 2)); }  // upper bound over the tilings

static size_t tap_generic_lds(int p) { return (size_t)(tap_lds_floats(p, TAP_GENERIC_TY) + p * p) * sizeof(float); }

hipError_t launch_tapconv(const ConvJob& j, int p, int flip, double* partials, int* n_partials, hipStream_t s,
                          bool tall) {
    switch (p) {
#define MLBA_TAP_CASE(PP) \
    case PP:              \
        return launch_tap_side<PP>(j, flip, partials, n_partials, s, tall);
        MLBA_TAP_SIDES(MLBA_TAP_CASE)
#undef MLBA_TAP_CASE
        default: {
            dim3 grid((j.D + TAP_TX - 1) / TAP_TX, (j.D + TAP_GENERIC_TY - 1) / TAP_GENERIC_TY);
            if (n_partials) *n_partials = (int)(grid.x * grid.y);
            const size_t lds = tap_generic_lds(p);
            if (lds > 64 * 1024) return hipErrorInvalidValue;
            hipLaunchKernelGGL(tapconv_kernel_generic, grid, dim3(kBlock), lds, s, j, p, flip, partials);
            return hipGetLastError();
        }
    }
}

// ---- batched kernel: tiles of many images in one launch ------------------
// Workgroup b serves image bmap[b], local tile b - bfirst[image].  FLIP:
// r = g - A u with the residual-norm partial of the tile written to
// partials[pbase + local tile]; otherwise the A^T correlation.  P > 0: every
// image has that PSF side (one tap loop in the kernel); P == 0: any sides.
// One tile height, one row a thread: with two an iteration of the explicit state
// took as long or longer at every batch measured (32 uneven images 707 us and 731
// with two rows in both products, 16 x 256 x 256, p = 15: 137 and 148, 8 x 1024 x
// 1024, p = 15: 518 and 530, p = 25 and 31: even).

template <bool FLIP>
__device__ __forceinline__ double tap_tile_any(const ConvJob& j, int p, int bx, int by, float* lds) {
    switch (p) {
#define MLBA_TAP_CASE(PP) \
    case PP:              \
        return tap_tile<PP, FLIP, 1, 8>(j, bx, by, lds);
        MLBA_TAP_SIDES(MLBA_TAP_CASE)
#undef MLBA_TAP_CASE
        default:
            return tap_tile_generic(j, p, FLIP ? 1 : 0, bx, by, lds);
    }
}

template <int P, bool FLIP>
__global__ __launch_bounds__(kBlock) void tapconv_batched_kernel(const BatchImage* __restrict__ imgs,
                                                                 const int* __restrict__ bmap,
                                                                 const int* __restrict__ bfirst,
                                                                 double* __restrict__ partials) {
    extern __shared__ float smem[];
    __shared__ double red[kBlock / 64];
    const int im = bmap[blockIdx.x];
    const BatchImage& I = imgs[im];
    const ConvJob j = FLIP ? blur_job(I) : blurT_job(I);
    const int local = blockIdx.x - bfirst[im];
    const int gx = (j.D + TAP_TX - 1) / TAP_TX;
    const int by = local / gx;
    const int bx = local - by * gx;
    double ss;
    if constexpr (P > 0) ss = tap_tile<P, FLIP, 1, 8>(j, bx, by, smem);
    else ss = tap_tile_any<FLIP>(j, I.p, bx, by, smem);
    if (FLIP && partials) tap_partial(ss, red, partials + I.pbase + local);
}

int tapconv_batched_tiles(const BatchImage& I, int flip) {
    const ConvJob j = flip ? blur_job(I) : blurT_job(I);
    return tap_tiles(j.D, I.p > 33 ? TAP_GENERIC_TY : tap_ty(1, 8));
}

template <int P>
static hipError_t launch_tb(const BatchImage* imgs, const int* bmap, const int* bfirst, int nblocks, int flip,
                            int pmax, double* partials, hipStream_t s) {
    size_t lds = (size_t)tap_lds_floats(pmax < 33 ? pmax : 33, tap_ty(1, 8)) * sizeof(float);
    if (pmax > 33 && tap_generic_lds(pmax) > lds) lds = tap_generic_lds(pmax);
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    if (flip)
        hipLaunchKernelGGL((tapconv_batched_kernel<P, true>), dim3(nblocks), dim3(kBlock), lds, s, imgs, bmap, bfirst,
                           partials);
    else
        hipLaunchKernelGGL((tapconv_batched_kernel<P, false>), dim3(nblocks), dim3(kBlock), lds, s, imgs, bmap,
                           bfirst, nullptr);
    return hipGetLastError();
}

hipError_t launch_tapconv_batched(const BatchImage* imgs, const int* bmap, const int* bfirst, int nblocks, int flip,
                                  int pmax, int same_p, double* partials, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    switch (same_p ? pmax : 0) {
#define MLBA_TAP_CASE(PP) \
    case PP:              \
        return launch_tb<PP>(imgs, bmap, bfirst, nblocks, flip, pmax, partials, s);
        MLBA_TAP_SIDES(MLBA_TAP_CASE)
#undef MLBA_TAP_CASE
        default: return launch_tb<0>(imgs, bmap, bfirst, nblocks, flip, pmax, partials, s);
    }
}

}  // namespace mlba
