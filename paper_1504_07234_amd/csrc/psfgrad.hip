// Kernels of the reverse sweep through K unrolled iterations of eq. (MLBA2)
// (rectangular blur of section 2.1, BCCB preconditioner of Algorithm 1) that
// have no forward counterpart:
//
//  * the PSF correlations: A u = sum_{a,q} H[a][q] u[. + p-1-a][. + p-1-q]
//    is linear in H, so d<y, A u>/dH[a][q] is the correlation of y with u at
//    lag (a, q).  Each step contributes corr(W^T zbar, t_k) - corr(u_k, rbar);
//  * the observation gradient (sum of the rbar) and the alpha gradient
//    (-<rbar, t_k>, from dP/dalpha = -P^2);
//  * the spectral term through P: with E = sum_k Re(conj(F rbar) F t_k) / n^2
//    (accumulated inside the preconditioner's column pass) and Lambda the
//    DFT of the zero-padded PSF, the derivative of |Lambda|^2 gives
//    -2 Re sum E conj(Lambda) e^{-2 pi i (ua + vq)/n}, which equals
//    -2 sum_{a',q'} H[a'][q'] e[(a'-a) mod n][(q'-q) mod n] with e the
//    (real, even) inverse transform of E;
//  * the final fixed-order reduction of every running partial.
//
// Running partials: every launch of a phase uses the same workgroup -> tile
// map, so workgroup b adds its tile's contribution to slot b at each step; the
// sums are therefore deterministic.
#include "common.hpp"
#include "kernels.hpp"

namespace mlba {

constexpr int PC_TY = 32;       // rows of a tile of the observed grid
constexpr int PC_TX = 64;       // columns
constexpr int PC_TS = PC_TX + 4;  // LDS row stride of the t and rbar tiles: 16 rows on distinct banks
constexpr int PC_WCOLS = 128;     // most columns of a window, two rows at a time

typedef float corr_f32x4 __attribute__((ext_vector_type(4)));

// Lags come in blocks of 16 x 16.
struct CorrShape {
    int nb, padl, wr, wc;
};

__host__ __device__ inline CorrShape corr_shape(int p) {
    CorrShape c;
    c.nb = (p + 15) / 16;
    c.padl = 16 * c.nb - p;          // window columns left of the image for the lags past p
    c.wr = PC_TY + p - 1;
    c.wc = PC_TX + 16 * c.nb - 1;
    return c;
}

static size_t corr_lds_floats(int p) {
    const CorrShape c = corr_shape(p);
    return 2 * (size_t)c.wr * c.wc + 2 * PC_TY * PC_TS;
}

int psf_corr_tiles(const BatchImage& I) {
    return ((I.n + PC_TX - 1) / PC_TX) * ((I.n + PC_TY - 1) / PC_TY);
}

// The correlation sums over pixels, so it is a matrix product over them: row r
// of the window and the tile's rows r - (p-1) + a give
//   C[q][a] += sum_x W[r][x + p-1-q] t[r - (p-1) + a][x],
// 16 lags q by 16 lags a and four pixels per v_mfma_f32_16x16x4_f32 (float32
// products and sums).  With one block of lags (p <= 16) the four waves share the
// window's rows and add up in LDS; otherwise each wave takes whole blocks.  A step
// of 16 images of 256 x 256, p = 15, takes 28 us: the staging of the four tiles and
// the waves' LDS reads.  On the vector units, with 46 LDS values read for 128
// multiply-adds, it took 47.
__global__ __launch_bounds__(kBlock) void psf_corr_batched_kernel(const BatchImage* __restrict__ imgs,
                                                                  const int* __restrict__ bmap,
                                                                  const int* __restrict__ bfirst, int first,
                                                                  double* __restrict__ part,
                                                                  double* __restrict__ apart) {
    extern __shared__ float smem[];
    __shared__ double red[kBlock / 64];
    const int xb = xcd_block(blockIdx.x, gridDim.x);  // adjacent tiles of an image in one L2
    const int im = bmap[xb];
    const BatchImage& I = imgs[im];
    const int n = I.n, N = I.N, p = I.p;
    const CorrShape cs = corr_shape(p);
    const int gx = (n + PC_TX - 1) / PC_TX;
    const int local = xb - bfirst[im];
    const int by = local / gx;
    const int oy0 = by * PC_TY, ox0 = (local - by * gx) * PC_TX;

    float* Wl = smem;                  // W^T zbar window
    float* Ul = Wl + cs.wr * cs.wc;    // u_k window
    float* Tl = Ul + cs.wr * cs.wc;    // t_k tile
    float* Rl = Tl + PC_TY * PC_TS;    // -rbar tile
    const float* wbar = I.u;
    const float* uk = I.uk;
    // the tile's loads, then the window's in rounds of WU rows: all of a round
    // in flight together
    constexpr int PER = PC_TY * PC_TX / kBlock, WU = 12;
    float tv[PER], rv[PER], dv[PER];
    const int ty = (int)threadIdx.x / PC_TX, tx = threadIdx.x % PC_TX;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int y = oy0 + ty + k * (kBlock / PC_TX), x = ox0 + tx;
        const bool in = y < n && x < n;
        const size_t o = in ? (size_t)y * n + x : 0;
        const float a = I.tk[o], b = I.t[o], c = I.dg && !first ? I.dg[o] : 0.0f;
        tv[k] = in ? a : 0.0f;
        rv[k] = in ? b : 0.0f;
        dv[k] = c;
    }
    {
        const int lx = threadIdx.x % PC_WCOLS, x = ox0 + lx - cs.padl, ly0 = (int)threadIdx.x / PC_WCOLS;
        const bool col = lx < cs.wc && x >= 0 && x < N;
        for (int l0 = ly0; l0 < cs.wr; l0 += WU * (kBlock / PC_WCOLS)) {
            float w[WU], u[WU];
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                const int y = oy0 + l0 + k * (kBlock / PC_WCOLS);
                const bool in = col && y < N;
                const size_t o = in ? (size_t)y * N + x : 0;
                w[k] = wbar[o];
                u[k] = uk[o];
                if (!in) w[k] = u[k] = 0.0f;
            }
#pragma unroll
            for (int k = 0; k < WU; ++k) {
                const int ly = l0 + k * (kBlock / PC_WCOLS);
                if (lx < cs.wc && ly < cs.wr) {
                    Wl[ly * cs.wc + lx] = w[k];
                    Ul[ly * cs.wc + lx] = u[k];
                }
            }
        }
    }
    double dot = 0.0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int ly = ty + k * (kBlock / PC_TX), y = oy0 + ly, x = ox0 + tx;
        if (I.dg && y < n && x < n) I.dg[(size_t)y * n + x] = first ? rv[k] : dv[k] + rv[k];
        dot += (double)rv[k] * (double)tv[k];
        Tl[ly * PC_TS + tx] = tv[k];
        Rl[ly * PC_TS + tx] = -rv[k];
    }
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, kk = lane >> 4;
    const int split = cs.nb == 1 ? kBlock / 64 : 1;  // waves that share a block's window rows
    for (int blk = split > 1 ? 0 : wave; blk < cs.nb * cs.nb; blk += kBlock / 64) {
        const int bq = blk / cs.nb, ba = blk - bq * cs.nb;
        corr_f32x4 c0 = {0.0f, 0.0f, 0.0f, 0.0f}, c1 = c0;
        // lane's A column: lag q = 16 bq + m at pixel kk; its B row: lag a = 16 ba + m
        const int acol = kk + p - 1 - (16 * bq + m) + cs.padl;
        for (int r = split > 1 ? wave : 0; r < cs.wr; r += split) {
            const int y = r - (p - 1) + 16 * ba + m;
            const bool ok = y >= 0 && y < PC_TY;
            const float* wrow = Wl + r * cs.wc + acol;
            const float* urow = Ul + r * cs.wc + acol;
            const float* trow = Tl + (ok ? y : 0) * PC_TS + kk;
            const float* rrow = Rl + (ok ? y : 0) * PC_TS + kk;
#pragma unroll 8
            for (int x0 = 0; x0 < PC_TX; x0 += 4) {
                const float tb = ok ? trow[x0] : 0.0f, rb = ok ? rrow[x0] : 0.0f;
                c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wrow[x0], tb, c0, 0, 0, 0);
                c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(urow[x0], rb, c1, 0, 0, 0);
            }
        }
        c0 += c1;
        double* out = part + (size_t)blockIdx.x * p * p;
        if (split > 1) {
            __syncthreads();  // the windows are no longer read: reuse LDS for the waves' sums
#pragma unroll
            for (int i = 0; i < 4; ++i) smem[wave * 256 + (4 * kk + i) * 16 + m] = c0[i];
            __syncthreads();
            const int q = threadIdx.x >> 4, a = threadIdx.x & 15;
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < kBlock / 64; ++w) sum += smem[w * 256 + threadIdx.x];
            if (q < p && a < p) out[a * p + q] += (double)sum;
        } else {
            const int a = 16 * ba + m;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = 16 * bq + 4 * kk + i;
                if (q < p && a < p) out[a * p + q] += (double)c0[i];
            }
        }
        if (split > 1) break;
    }
    const double d = block_sum(dot, red);
    if (threadIdx.x == 0) apart[blockIdx.x] -= d;
}

hipError_t launch_psf_corr_batched(const BatchImage* imgs, const int* bmap, const int* bfirst, int nblocks, int p,
                                   int first, double* part, double* apart, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    const size_t lds = corr_lds_floats(p) * sizeof(float);
    // 128 columns of the window are staged (p <= 49)
    if (lds > 160 * 1024 || corr_shape(p).wc > PC_WCOLS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(psf_corr_batched_kernel, dim3(nblocks), dim3(kBlock), lds, s, imgs, bmap, bfirst, first,
                       part, apart);
    return hipGetLastError();
}

// One workgroup per image; e = I.t holds the inverse transform of E / n^2.
__global__ __launch_bounds__(kBlock) void psf_spectral_kernel(const BatchImage* __restrict__ imgs, int p,
                                                              double* __restrict__ spec) {
    const BatchImage& I = imgs[blockIdx.x];
    const int n = I.n;
    const float* e = I.t;
    const float* H = I.psf;
    const double scale = -2.0 * (double)n * (double)n;
    for (int l = threadIdx.x; l < p * p; l += kBlock) {
        const int a = l / p, q = l - (l / p) * p;
        double s = 0.0;
        for (int a2 = 0; a2 < p; ++a2) {
            const float* erow = e + (size_t)mod_pos(a2 - a, n) * n;
            for (int q2 = 0; q2 < p; ++q2) s += (double)H[a2 * p + q2] * (double)erow[mod_pos(q2 - q, n)];
        }
        spec[(size_t)blockIdx.x * p * p + l] = scale * s;
    }
}

hipError_t launch_psf_spectral_batched(const BatchImage* imgs, int count, int p, double* spec, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(psf_spectral_kernel, dim3(count), dim3(kBlock), 0, s, imgs, p, spec);
    return hipGetLastError();
}

// Workgroup o reduces output o: o < bands -> dmu[o]; o == bands -> dalpha;
// o > bands -> dpsf[o - bands - 1].  Sums in a fixed order.
__global__ __launch_bounds__(kBlock) void unrolled_reduce_kernel(UnrolledSums S, double* __restrict__ dmu,
                                                                 double* __restrict__ dalpha,
                                                                 double* __restrict__ dpsf) {
    __shared__ double red[kBlock / 64];
    const int o = blockIdx.x;
    double s = 0.0;
    if (o < S.bands) {
        const int lev = o == 0 ? S.levels : (o - 1) / 8 + 1;
        const int slot = o == 0 ? 8 : (o - 1) % 8;
        const double* pl = S.mu_part[lev - 1];
        for (int b = threadIdx.x; b < S.mu_blocks[lev - 1]; b += kBlock) s += pl[(size_t)b * 9 + slot];
    } else if (o == S.bands) {
        for (int b = threadIdx.x; b < S.corr_blocks; b += kBlock) s += S.alpha_part[b];
    } else {
        const int l = o - S.bands - 1;
        const int pp = S.p * S.p;
        for (int b = threadIdx.x; b < S.corr_blocks; b += kBlock) s += S.corr_part[(size_t)b * pp + l];
        for (int i = threadIdx.x; i < S.count; i += kBlock) s += S.spec[(size_t)i * pp + l];
    }
    const double t = block_sum(s, red);
    if (threadIdx.x == 0) {
        if (o < S.bands) dmu[o] = t;
        else if (o == S.bands) *dalpha = t;
        else dpsf[o - S.bands - 1] = t;
    }
}

hipError_t launch_unrolled_reduce(const UnrolledSums& S, double* dmu, double* dalpha, double* dpsf, hipStream_t s) {
    const int outs = S.bands + 1 + S.p * S.p;
    hipLaunchKernelGGL(unrolled_reduce_kernel, dim3(outs), dim3(kBlock), 0, s, S, dmu, dalpha, dpsf);
    return hipGetLastError();
}

}  // namespace mlba
