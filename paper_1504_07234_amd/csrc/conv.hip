// Direct convolution for the blur A and its transpose A^T (paper section 2:
// A f is the valid part of the 2-D convolution of the extended image with the
// PSF; A^T y is the full correlation of y with the PSF, followed for imposed
// boundaries by the transpose of the padding), on the matrix cores.
//
// Every float32 value x is split into three bfloat16 parts x = x1 + x2 + x3
// (8 + 8 + 8 significand bits: the sum is x itself), the window's while it is
// staged, the taps' when the PSF is set.  A product of the blur is then the
// six products x1 h1, x1 h2, x2 h1, x2 h2, x1 h3, x3 h1 (each exact in float32;
// the three left out are below 2^-24 of |x h|, as a rule below 2^-27), summed in
// float32 by v_mfma_f32_16x16x32_bf16: 6 x 16 cycles for the work of 16 x 16 x 32
// multiply-adds, against 512 cycles of vector FMAs.  x1 h1, the bulk of the sum,
// is added up apart from the rest and loses few bits, so the result is nearer to
// the exact one than a chain of FMAs.  Error of A^T in the 2-norm, FMAs -> here,
// 1024 x 1024, units of 1e-8:
//                        p = 3           p = 9         p = 17         p = 31
//   Gaussian           5.7 -> 3.0     16.2 -> 8.1   30.4 -> 13.0   55.3 -> 22.7
//   disk               4.4 -> 2.6     12.6 -> 3.8   25.2 ->  5.5   47.5 -> 13.0
//   random             5.0 -> 2.7     16.2 -> 5.4   29.4 ->  8.8   54.9 -> 17.3
//   streak             4.4 -> 2.7      7.2 -> 3.0    9.7 ->  3.9   13.3 ->  4.5
//   a row or a column  3.6 -> 2.7      5.7 -> 2.7    7.6 ->  3.0   10.1 ->  2.7
//   one tap            2.51 -> 2.54   2.52 -> 2.55  2.52 -> 2.54   2.52 -> 2.54
//
// One matrix product: D[m][s] += T_t[m][k] X_t[k][s].  A column s of D is a
// block of 2 rows x 8 columns of outputs (m = 8 yr + xo), X_t[k][s] the input
// row t under it from its first column on, and T_t[m][k] = tap(t - yr, k - xo)
// (zero outside the PSF), so p + 1 products of depth K = 8 + p - 1 (padded to
// 32 up to p = 25, to 64 up to CONV_PMAX = 49) give the 256 outputs of D.  A wave
// holds R such D's, one below the other: an input row is read from LDS once
// and used by the R of them through a rolling window of 2 R rows in
// registers, and the fragments of T_t, laid out in the order of the lanes when
// the PSF is set, are read from global memory (they stay in the caches) one
// row ahead.  A workgroup's four waves cover 64 columns x 16 R rows.
//
// The products alone run at the rate of the matrix cores (4096 x 4096, p = 15: 42
// us), the staging and its split add to that, in series (30 us): the matrix cores
// are busy for 0.15 / 0.34 / 0.62 of the CUs' time (A^T at 512, p = 17; 1024 and
// 2048, p = 15) and for 0.74 / 0.75 at 2048, p = 25 / 31.  At p > 25 and in the tiles
// of one or two row pairs 0.43 to 0.47 of the LDS cycles are bank conflicts.  A and A^T with vector FMAs in the order of the taps -> here, on random
// values (on zeros the matrix cores are up to a fifth faster), us: 512 x 512, p =
// 15: 11.0 / 11.5 -> 6.4 / 7.9; 1024 x 1024, p = 15 / 31: 15.2 / 18.1 -> 10.5 / 12.1
// and 40.7 / 52.7 -> 22.4 / 28.1; 2048 x 2048: 38.5 / 44.1 -> 25.0 / 25.8 and 126 /
// 139 -> 73 / 73.
//
// bfloat16 has float32's exponent range, so nothing is scaled.  What the split
// cannot hold takes the plain tap loop:
//   - infinities, NaN and values above bfloat16's largest, and sums of the rounded
//     first parts that overflow: some sum of the tile is then not finite.  In the
//     loop infinities and NaN reach exactly the outputs whose taps touch them;
//   - a window or a PSF whose largest value is below 2^-95, where the third parts
//     leave bfloat16's range (2^-133): at 2^-115 the error was 5.6e-7, in the tap
//     loop 1.5e-7.  A smaller value beside larger ones loses less than 2^-133.
//
// The tile body is a device function shared by the single-image kernels and
// the batched kernel (one launch covering the tiles of many images); an
// output's arithmetic does not depend on R or on the tile it lies in.
#include "common.hpp"
#include "kernels.hpp"

namespace mlba {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int CONV_TX = 64;     // output columns per workgroup
constexpr int CONV_SPLITS = 3;  // bfloat16 parts of a float32 value
constexpr int CONV_K1 = 25;     // largest PSF side whose rows fit one product of depth 32
constexpr int CONV_PMAX = 49;

__host__ __device__ constexpr int conv_ty(int r) { return 16 * r; }
// products of depth 32 per input row
__host__ __device__ constexpr int conv_depth(int p) { return p <= CONV_K1 ? 1 : 2; }
// window columns (bfloat16 values) of one part of one row: the last block's K
__host__ __device__ constexpr int conv_cols(int kc) { return CONV_TX - 8 + 32 * kc; }
__host__ __device__ constexpr int conv_row_elems(int kc) { return CONV_SPLITS * conv_cols(kc); }

// rows fetched ahead of the last product, of the window and of the taps
constexpr int CONV_AHEAD = 3;
static size_t conv_lds_bytes(int p, int r) {
    return (size_t)(conv_ty(r) + p - 1 + CONV_AHEAD) * conv_row_elems(conv_depth(p)) * sizeof(__bf16);
}

// The deepest tile (R row pairs per lane) of a PSF side: R = 4 with the
// two-product rows would take 66 to 80 KB of LDS.
static int conv_max_r(int p) { return p <= CONV_K1 ? 4 : 2; }

static int conv_tiles_r(int D, int r) {
    return ((D + CONV_TX - 1) / CONV_TX) * ((D + conv_ty(r) - 1) / conv_ty(r));
}

// PSF rows a = -1 .. p + CONV_AHEAD (zero outside [0, p)), then one element with
// whether the taps are too small for the split
__host__ __device__ constexpr int conv_taps_flag(int p) {
    return (p + 2 + CONV_AHEAD) * CONV_SPLITS * conv_depth(p) * 32;
}
size_t conv_taps_elems(int p) { return (size_t)conv_taps_flag(p) + 1; }

// Of the or of some values' bits: whether one of them is 2^-95 or more (the
// exponents below are the 32 smallest), and whether one is not zero.
__device__ __forceinline__ bool conv_any_large(unsigned bits) { return (bits & 0x70000000u) != 0; }
__device__ __forceinline__ bool conv_any(unsigned bits) { return (bits & 0x7fffffffu) != 0; }

__device__ __forceinline__ void split3(float x, __bf16* h) {
    h[0] = (__bf16)x;
    const float r1 = x - (float)h[0];
    h[1] = (__bf16)r1;
    h[2] = (__bf16)(r1 - (float)h[1]);
}

// Fragments for both directions: taps[flip][(((a + 1) S + s) KC + q) 32 + 8 kg
// + xo] holds tap(a, k - xo), k = 32 q + 8 kg .. + 7; T_t is row a = t in its
// upper half (yr = 0) and row a = t - 1 in its lower one.
__global__ __launch_bounds__(64) void conv_taps_kernel(const float* __restrict__ psf, int p, int kc,
                                                       uint4* __restrict__ taps0, uint4* __restrict__ taps1,
                                                       double* __restrict__ l1) {
    if (l1 && blockIdx.x == 0 && blockIdx.y == 0) {  // sum |psf| in index order, for Algorithm 4-NS
        __shared__ float h[CONV_PMAX * CONV_PMAX];
        for (int i = threadIdx.x; i < p * p; i += 64) h[i] = fabsf(psf[i]);
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int i = 0; i < p * p; ++i) sum += (double)h[i];
            *l1 = sum;
        }
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        unsigned bits = 0;
        for (int i = threadIdx.x; i < p * p; i += 64) bits |= __builtin_bit_cast(unsigned, psf[i]);
        const bool tiny = __any(conv_any(bits)) && !__any(conv_any_large(bits));
        if (threadIdx.x < 2)
            (threadIdx.x ? taps1 : taps0)[conv_taps_flag(p)] = make_uint4(tiny ? 1u : 0u, 0u, 0u, 0u);
    }
    const int a = (int)blockIdx.x - 1, q = blockIdx.y, flip = threadIdx.x >> 5, l = threadIdx.x & 31;
    bf16x8 f[CONV_SPLITS];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int b = 32 * q + 8 * (l >> 3) + e - (l & 7);
        float v = 0.0f;
        if (a >= 0 && a < p && b >= 0 && b < p) v = psf[flip ? p * p - 1 - (a * p + b) : a * p + b];
        __bf16 h[CONV_SPLITS];
        split3(v, h);
#pragma unroll
        for (int s = 0; s < CONV_SPLITS; ++s) f[s][e] = h[s];
    }
    uint4* out = flip ? taps1 : taps0;
#pragma unroll
    for (int s = 0; s < CONV_SPLITS; ++s)
        out[((size_t)((a + 1) * CONV_SPLITS + s) * kc + q) * 32 + l] = __builtin_bit_cast(uint4, f[s]);
}

hipError_t launch_conv_taps(const float* psf, int p, uint4* taps0, uint4* taps1, double* l1, hipStream_t s) {
    const int kc = conv_depth(p);
    hipLaunchKernelGGL(conv_taps_kernel, dim3(p + 2 + CONV_AHEAD, kc), dim3(64), 0, s, psf, p, kc, taps0, taps1, l1);
    return hipGetLastError();
}

struct __attribute__((packed, aligned(4))) FloatQuad {
    float v[4];
};

// Splits four values into the rows of the window; bits collects the or of theirs.
template <int C>
__device__ __forceinline__ void conv_put_split(__bf16* win, const float* v, unsigned* bits) {
    unsigned w[CONV_SPLITS][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        float r0 = v[2 * e], r1 = v[2 * e + 1];
        *bits |= __builtin_bit_cast(unsigned, r0) | __builtin_bit_cast(unsigned, r1);
#pragma unroll
        for (int s = 0; s < CONV_SPLITS; ++s) {
            w[s][e] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)r0, (__bf16)r1});
            if (s + 1 < CONV_SPLITS) {  // the part back as a float: its bits are the upper half
                r0 -= __builtin_bit_cast(float, w[s][e] << 16);
                r1 -= __builtin_bit_cast(float, w[s][e] & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int s = 0; s < CONV_SPLITS; ++s) *(uint2*)(win + s * C) = make_uint2(w[s][0], w[s][1]);
}

// The window of the tile at (oy0, ox0) is rows x conv_cols(KC) values (the
// columns past the last tap of the last output only have to be finite: their
// taps are zero).  A thread keeps one group of four columns and takes every
// eighth row, U in all: conv_fetch issues their loads, conv_commit splits them
// into LDS.
template <int KC, int U>
__device__ __forceinline__ void conv_fetch(const ConvJob& j, int P, int TY, int oy0, int ox0, float (&v)[U][4]) {
    constexpr int C = conv_cols(KC), RS = kBlock / 32;
    static_assert(C % 4 == 0 && C / 4 <= 32, "one group of four columns per lane of a half wave");
    const int rows = TY + P - 1;
    const int lx = min(4 * ((int)threadIdx.x & 31), C - 4), ly0 = (int)threadIdx.x >> 5;
    const int S = j.S, ext = j.ext, y0 = oy0 + j.org, x0 = ox0 + j.org;
    if (y0 >= 0 && x0 >= 0 && y0 + rows <= S && x0 + C <= S) {  // the whole window lies in the image
        const float* src = j.src + (size_t)(y0 + ly0) * S + x0 + lx;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const FloatQuad q = *(const FloatQuad*)(ly0 + u * RS < rows ? src + (size_t)u * RS * S : src);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = q.v[e];
        }
    } else if (ext != EXT_ANTIREFLECT) {
        int xi[4];
        bool hx[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) xi[e] = ext_axis(x0 + lx + e, S, ext, &hx[e]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bool hy;
            const float* row = j.src + (size_t)ext_axis(y0 + min(ly0 + u * RS, rows - 1), S, ext, &hy) * S;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float q = row[xi[e]];
                v[u][e] = hy && hx[e] ? q : 0.0f;
            }
        }
    }
}

// Returns the or of the bits of the thread's values.  A window that leaves the
// image under the antireflective extension (up to four sources a value) is read
// here, row by row.
template <int KC, int U>
__device__ __forceinline__ unsigned conv_commit(const ConvJob& j, int P, int TY, int oy0, int ox0, float (&v)[U][4],
                                            __bf16* win) {
    constexpr int C = conv_cols(KC), LS = conv_row_elems(KC), RS = kBlock / 32;
    const int rows = TY + P - 1;
    const int lx = 4 * ((int)threadIdx.x & 31), ly0 = (int)threadIdx.x >> 5;
    const int S = j.S, y0 = oy0 + j.org, x0 = ox0 + j.org;
    unsigned bits = 0;
    if (lx >= C) return bits;
    if (j.ext == EXT_ANTIREFLECT && !(y0 >= 0 && x0 >= 0 && y0 + rows <= S && x0 + C <= S)) {
#pragma unroll 1
        for (int ly = ly0; ly < rows; ly += RS) {
            float q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = fetch_antireflect(j.src, S, y0 + ly, x0 + lx + e);
            conv_put_split<C>(win + ly * LS + lx, q, &bits);
        }
        return bits;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (ly0 + u * RS < rows) conv_put_split<C>(win + (ly0 + u * RS) * LS + lx, v[u], &bits);
    return bits;
}

// dst = g - v (returning v's square sum), dst + v or v
__device__ __forceinline__ double conv_put(const ConvJob& j, int y, int x, float v) {
    const size_t i = (size_t)y * j.D + x;
    double ss = 0.0;
    if (j.g) {
        v = j.g[i] - v;
        ss = (double)v * (double)v;
    } else if (j.acc) {
        v = j.dst[i] + v;
    }
    j.dst[i] = v;
    return ss;
}

// the same for four columns.  A side that is no multiple of four puts the rows off
// the 16-byte boundaries; one access of four bytes' alignment still takes half of
// what four accesses take (A^T at 1024 x 1024, p = 7: 11.4 -> 9.9 us; 2048 x 2048,
// p = 3: 21.1 -> 16.5).
__device__ __forceinline__ double conv_put4(const ConvJob& j, int y, int x, f32x4 v) {
    typedef f32x4 __attribute__((aligned(4))) Quad;
    const size_t i = (size_t)y * j.D + x;
    double ss = 0.0;
    if (j.g) {
        v = *(const Quad*)(j.g + i) - v;
#pragma unroll
        for (int e = 0; e < 4; ++e) ss += (double)v[e] * (double)v[e];
    } else if (j.acc) {
        v = *(const Quad*)(j.dst + i) + v;
    }
    *(Quad*)(j.dst + i) = v;
    return ss;
}

// Plain tap loop over the tile, for a window that the split cannot hold: the
// values themselves take the split ones' place in LDS.  A thread owns four or
// eight columns of a row; eight taps at a time meet a segment of them.  With
// every value read from global memory instead, a restoration whose state had
// become NaN took 35 times as long (512 x 512, p = 15: 287 us a blur).
template <int KC, int R>
__device__ __forceinline__ double conv_tile_taps(const ConvJob& j, int P, int flip, int oy0, int ox0, float* win) {
    constexpr int TY = conv_ty(R), C = conv_cols(KC), LS = C + 1;  // an odd stride: rows start on distinct banks
    static_assert(LS * sizeof(float) <= conv_row_elems(KC) * sizeof(__bf16), "fits the split window");
    const int rows = TY + P - 1, cols = CONV_TX + P - 1;
    for (int ly = (int)threadIdx.x >> 6; ly < rows; ly += kBlock / 64)
        for (int lx = threadIdx.x & 63; lx < cols; lx += 64)
            win[ly * LS + lx] = fetch_ext(j.src, j.S, oy0 + j.org + ly, ox0 + j.org + lx, j.ext);
    __syncthreads();
    constexpr int E = R == 1 ? 4 : 8;  // columns of a thread
    double ss = 0.0;
#pragma unroll 1
    for (int i = threadIdx.x; i < TY * (CONV_TX / E); i += kBlock) {
        const int ly = i / (CONV_TX / E), lx = E * (i % (CONV_TX / E));
        float acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.0f;
#pragma unroll 1
        for (int a = 0; a < P; ++a) {
            const float* row = win + (ly + a) * LS + lx;
            const float* tap = j.psf + (flip ? P * P - 1 - a * P : a * P);
            int b = 0;
#pragma unroll 1
            for (; b + 8 <= P; b += 8) {
                float v[E + 7], t[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) t[k] = tap[flip ? -(b + k) : b + k];
#pragma unroll
                for (int k = 0; k < E + 7; ++k) v[k] = row[b + k];
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[e] = fmaf(t[k], v[k + e], acc[e]);
            }
#pragma unroll 1
            for (; b < P; ++b) {
                const float t = tap[flip ? -b : b];
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = fmaf(t, row[b + e], acc[e]);
            }
        }
        const int y = oy0 + ly;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (y < j.D && ox0 + lx + e < j.D) ss += conv_put(j, y, ox0 + lx + e, acc[e]);
    }
    return ss;
}

// The sums of the tile whose split window is in LDS: v[i] holds those of the lane's
// block in row pair i (conv_store).  Returns whether all are finite: an infinity, a
// NaN or a value above bfloat16's largest in the window or the taps gives NaN (its
// first part meets a zero of T_t or its own second part), and where the rounded
// first parts overflow, infinity.
template <int KC, int R>
__device__ __forceinline__ bool conv_products(const ConvJob& j, int P, const __bf16* win, f32x4 (&v)[R]) {
    constexpr int C = conv_cols(KC), LS = conv_row_elems(KC), S = CONV_SPLITS;
    constexpr int NF = R == 1 ? 4 : 2 * R;  // rolling window rows
    constexpr int NT = R == 4 ? 2 : 4;      // rolling tap rows
    constexpr int UN = NF > NT ? NF : NT;
    static_assert(NF - 2 * R + 1 <= CONV_AHEAD && NT - 1 <= CONV_AHEAD, "rows fetched ahead");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int seg = lane & 7, rb = (lane >> 3) & 1, kg = lane >> 4;
    const int row0 = wave * 4 * R + rb * 2 * R;  // the lane's first window (and output) row
    const __bf16* src = win + row0 * LS + 8 * seg + 8 * kg;
    const uint4* taps = j.taps;  // uniform; row t of the half waves' lanes below
    const int depth = KC == 1 ? 1 : conv_depth(P), tstep = S * depth * 32;
    const int tl = 8 * kg + (lane & 7) + (((lane >> 3) & 1) ? 0 : tstep);
    f32x4 acc[R], low[R];  // the products x1 h1, and the others
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = low[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    bf16x8 f[NF][S];  // window rows t .. t + NF - 1, row r in slot r % NF
    bf16x8 tp[NT][S]; // T_t .. T_{t + NT - 1}
    auto load_row = [&](bf16x8 (&d)[S], int r) {
#pragma unroll
        for (int s = 0; s < S; ++s) d[s] = *(const bf16x8*)(src + r * LS + s * C);
    };
    auto load_taps = [&](bf16x8 (&d)[S]) {
#pragma unroll
        for (int s = 0; s < S; ++s) d[s] = __builtin_bit_cast(bf16x8, taps[s * depth * 32 + tl]);
        taps += tstep;
    };
#pragma unroll 1
    for (int q = 0; q < depth; ++q) {  // depth 32 at a time: the other half's rows and taps would not fit the registers
#pragma unroll
        for (int r = 0; r < NT - 1; ++r) load_taps(tp[r]);
#pragma unroll
        for (int r = 0; r < NF - 1; ++r) load_row(f[r], r);
#pragma unroll 1
        for (int t0 = 0; t0 <= P; t0 += UN) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int t = t0 + u;
                if (t > P) break;
                load_taps(tp[(u + NT - 1) % NT]);
                load_row(f[(u + NF - 1) % NF], t + NF - 1);
                __builtin_amdgcn_sched_barrier(0);  // the loads ahead stay ahead of this step's products
                constexpr int PS[5] = {2, 0, 1, 1, 0}, PT[5] = {0, 2, 1, 0, 1};
#pragma unroll
                for (int i = 0; i < R; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tp[u % NT][0], f[(u + 2 * i) % NF][0], acc[i],
                                                                     0, 0, 0);
#pragma unroll
                for (int w = 0; w < 5; ++w)
#pragma unroll
                    for (int i = 0; i < R; ++i)
                        low[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tp[u % NT][PT[w]], f[(u + 2 * i) % NF][PS[w]],
                                                                         low[i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        src += 32;
        taps = j.taps + 32;
    }

    float zero = 0.0f;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        v[i] = acc[i] + low[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) zero = fmaf(v[i][e], 0.0f, zero);
    }
    return zero == 0.0f;
}

// Writes the tile's outputs.  Returns the thread's sum of squares of the residuals
// (0 without g).
template <int R>
__device__ __forceinline__ double conv_store(const ConvJob& j, int oy0, int ox0, const f32x4 (&v)[R]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int seg = lane & 7, rb = (lane >> 3) & 1, kg = lane >> 4;
    // lane: output block (seg, rb), rows 2 i + (kg >> 1), columns 4 (kg & 1) .. + 3
    const int x = ox0 + 8 * seg + 4 * (kg & 1), row0 = wave * 4 * R + rb * 2 * R;
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int y = oy0 + row0 + 2 * i + (kg >> 1);
        if (y < j.D) {
            if (x + 4 <= j.D) {
                ss += conv_put4(j, y, x, v[i]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (x + e < j.D) ss += conv_put(j, y, x + e, v[i][e]);
            }
        }
    }
    return ss;
}

// One output tile of the job at (oy0, ox0): the thread's sum of squares.
template <int KC, int R>
__device__ __forceinline__ double conv_tile(const ConvJob& j, int P, int flip, int oy0, int ox0, __bf16* win) {
    constexpr int PMAX = KC == 1 ? CONV_K1 : CONV_PMAX;
    constexpr int U = (conv_ty(R) + PMAX - 1 + 7) / 8;
    __shared__ int bad, large, some;
    const unsigned tiny = j.taps[conv_taps_flag(P)].x;
    if (threadIdx.x == 0) {
        bad = tiny;
        large = some = 0;
    }
    float w[U][4];
    conv_fetch<KC, U>(j, P, conv_ty(R), oy0, ox0, w);
    __syncthreads();
    const unsigned bits = conv_commit<KC, U>(j, P, conv_ty(R), oy0, ox0, w, win);
    if (conv_any_large(bits)) large = 1;
    else if (conv_any(bits)) some = 1;
    __syncthreads();
    if (large || !some) {
        f32x4 v[R];
        if (!conv_products<KC, R>(j, P, win, v)) bad = 1;
        __syncthreads();
        if (!bad) return conv_store<R>(j, oy0, ox0, v);
    }
    return conv_tile_taps<KC, R>(j, P, flip, oy0, ox0, (float*)win);
}

// ---- single-image kernels -----------------------------------------------

template <int KC, int R>
__global__ __launch_bounds__(kBlock, 3) void conv_kernel(ConvJob j, int P, int flip, double* __restrict__ partials) {
    extern __shared__ __align__(16) __bf16 conv_win[];
    __shared__ double red[kBlock / 64];
    int bx, by;
    xcd_tile(&bx, &by);
    const double ss = conv_tile<KC, R>(j, P, flip, by * conv_ty(R), bx * CONV_TX, conv_win);
    if (partials) {
        const double t = block_sum(ss, red);
        if (threadIdx.x == 0) partials[blockIdx.y * gridDim.x + blockIdx.x] = t;
    }
}

// Row pairs per lane of a D x D output: the deepest tile that still leaves most CUs
// two workgroups.  Two pairs from 400 tiles: A / A^T at 900 x 900, 435 tiles or 855
// of one pair: p = 7: 7.9 / 8.3 and 8.9 / 9.1 us, p = 31: 20.9 / 21.7 and 28.5 /
// 30.4; 768 x 768, 288 or 576: p = 3: 6.8 / 7.1 and 6.5 / 6.7, p = 7: even.  Four
// from 512: with them an iteration of 1280 x 1280, 400 tiles, takes 90.1 / 99.0 us
// (p = 3 / 15), with two 86.1 / 95.2.
static int conv_default_r(int D, int p) {
    int r = conv_max_r(p);
    while (r > 1 && conv_tiles_r(D, r) < (r == 4 ? 512 : 400)) r /= 2;
    return r;
}

int conv_partials_count(int D) { return conv_tiles_r(D, 1); }  // upper bound over the tilings

template <int KC, int R>
static hipError_t launch_cr(const ConvJob& j, int p, int flip, double* partials, int* n_partials, hipStream_t s) {
    dim3 grid((j.D + CONV_TX - 1) / CONV_TX, (j.D + conv_ty(R) - 1) / conv_ty(R));
    if (n_partials) *n_partials = (int)(grid.x * grid.y);
    hipLaunchKernelGGL((conv_kernel<KC, R>), grid, dim3(kBlock), conv_lds_bytes(p, R), s, j, p, flip, partials);
    return hipGetLastError();
}

hipError_t launch_conv_job(const ConvJob& j, int p, int flip, double* partials, int* n_partials, hipStream_t s) {
    if (p < 1 || p > CONV_PMAX || !j.taps) return hipErrorInvalidValue;
    const int r = conv_default_r(j.D, p);
    if (conv_depth(p) == 1) {
        if (r == 4) return launch_cr<1, 4>(j, p, flip, partials, n_partials, s);
        if (r == 2) return launch_cr<1, 2>(j, p, flip, partials, n_partials, s);
        return launch_cr<1, 1>(j, p, flip, partials, n_partials, s);
    }
    if (r == 2) return launch_cr<2, 2>(j, p, flip, partials, n_partials, s);
    return launch_cr<2, 1>(j, p, flip, partials, n_partials, s);
}

// ---- batched kernel: tiles of many images in one launch ------------------
// Workgroup b serves image bmap[b], local tile b - bfirst[image].
// FLIP: r = g - A u with the residual-norm partial of the tile written to
// partials[pbase + local tile]; otherwise the A^T correlation.  An image of
// smaller PSF side than the launch's widest runs in the same window.

template <bool FLIP, int KC, int R>
__global__ __launch_bounds__(kBlock, 3) void conv_batched_kernel(const BatchImage* __restrict__ imgs,
                                                                 const int* __restrict__ bmap,
                                                                 const int* __restrict__ bfirst,
                                                                 double* __restrict__ partials) {
    extern __shared__ __align__(16) __bf16 conv_win[];
    __shared__ double red[kBlock / 64];
    const int im = bmap[blockIdx.x];
    const BatchImage& I = imgs[im];
    const ConvJob j = FLIP ? blur_job(I) : blurT_job(I);
    const int local = blockIdx.x - bfirst[im];
    const int gx = (j.D + CONV_TX - 1) / CONV_TX;
    const int by = local / gx;
    const double ss = conv_tile<KC, R>(j, I.p, FLIP, by * conv_ty(R), (local - by * gx) * CONV_TX, conv_win);
    if (FLIP && partials) {
        const double t = block_sum(ss, red);
        if (threadIdx.x == 0) partials[I.pbase + local] = t;
    }
}

// row pairs per lane of a launch's tiles (32 or 64 rows, half of it with the
// two-product rows)
static int batched_r(int pmax, int ry) { return pmax <= CONV_K1 ? 2 * ry : ry; }

int conv_batched_tiles(const BatchImage& I, int flip, int pmax, int ry) {
    const ConvJob j = flip ? blur_job(I) : blurT_job(I);
    return conv_tiles_r(j.D, batched_r(pmax, ry));
}

template <bool FLIP, int KC, int R>
static hipError_t launch_cb(const BatchImage* imgs, const int* bmap, const int* bfirst, int tiles, int pmax,
                            double* partials, hipStream_t s) {
    hipLaunchKernelGGL((conv_batched_kernel<FLIP, KC, R>), dim3(tiles), dim3(kBlock), conv_lds_bytes(pmax, R), s,
                       imgs, bmap, bfirst, partials);
    return hipGetLastError();
}

template <bool FLIP>
static hipError_t launch_cbf(const BatchImage* imgs, const int* bmap, const int* bfirst, int tiles, int pmax,
                             double* partials, hipStream_t s, int ry) {
    const int r = batched_r(pmax, ry);
    if (pmax > CONV_K1) return r == 2 ? launch_cb<FLIP, 2, 2>(imgs, bmap, bfirst, tiles, pmax, partials, s)
                                      : launch_cb<FLIP, 2, 1>(imgs, bmap, bfirst, tiles, pmax, partials, s);
    return r == 4 ? launch_cb<FLIP, 1, 4>(imgs, bmap, bfirst, tiles, pmax, partials, s)
                  : launch_cb<FLIP, 1, 2>(imgs, bmap, bfirst, tiles, pmax, partials, s);
}

hipError_t launch_conv_batched(const BatchImage* imgs, const int* bmap, const int* bfirst, int nblocks, int flip,
                               int pmax, double* partials, hipStream_t s, int ry) {
    if (nblocks <= 0) return hipSuccess;
    if (pmax > CONV_PMAX) return hipErrorInvalidValue;
    return flip ? launch_cbf<true>(imgs, bmap, bfirst, nblocks, pmax, partials, s, ry)
                : launch_cbf<false>(imgs, bmap, bfirst, nblocks, pmax, nullptr, s, ry);
}

// ---- transpose of the reflective padding ---------------------------------
// A pixel k of the n-point axis is copied to padded positions k + c, c - 1 - k
// (when k < c) and 2n - 1 - k + c (when k >= n - c); p <= n keeps these
// distinct.
__device__ __forceinline__ int pad_preimages(int k, int n, int c, int* pre) {
    int cnt = 0;
    pre[cnt++] = k + c;
    if (k < c) pre[cnt++] = c - 1 - k;
    if (k >= n - c) pre[cnt++] = 2 * n - 1 - k + c;
    return cnt;
}

__device__ __forceinline__ void fold_pixel(const float* __restrict__ wext, int m, float* __restrict__ w, int n,
                                           int c, int y, int x, int accum = 0) {
    int py[3], px[3];
    const int cy = pad_preimages(y, n, c, py);
    const int cx = pad_preimages(x, n, c, px);
    float acc = 0.0f;
    for (int i = 0; i < cy; ++i)
        for (int k = 0; k < cx; ++k) acc += wext[(size_t)py[i] * m + px[k]];
    w[(size_t)y * n + x] = accum ? w[(size_t)y * n + x] + acc : acc;
}

__global__ __launch_bounds__(kBlock) void fold_reflect_kernel(const float* __restrict__ wext, int m,
                                                              float* __restrict__ w, int n, int c, int accum) {
    const int x = blockIdx.x * kBlock + threadIdx.x;
    if (x < n) fold_pixel(wext, m, w, n, c, blockIdx.y, x, accum);
}

hipError_t launch_fold_reflect(const float* wext, int m, float* w, int n, int c, hipStream_t s, int accum) {
    dim3 grid((n + kBlock - 1) / kBlock, n);
    hipLaunchKernelGGL(fold_reflect_kernel, grid, dim3(kBlock), 0, s, wext, m, w, n, c, accum);
    return hipGetLastError();
}

// batched fold: workgroup b covers row (b - bfirst[img]) of image bmap[b]
__global__ __launch_bounds__(kBlock) void fold_batched_kernel(const BatchImage* __restrict__ imgs,
                                                              const int* __restrict__ bmap,
                                                              const int* __restrict__ bfirst) {
    const int im = bmap[blockIdx.x];
    const BatchImage& I = imgs[im];
    const int y = blockIdx.x - bfirst[im];
    const int m = I.n + I.p - 1;
    for (int x = threadIdx.x; x < I.n; x += kBlock) fold_pixel(I.wext, m, I.w, I.n, I.c, y, x, I.blur_acc);
}

hipError_t launch_fold_batched(const BatchImage* imgs, const int* bmap, const int* bfirst, int nblocks,
                               hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(fold_batched_kernel, dim3(nblocks), dim3(kBlock), 0, s, imgs, bmap, bfirst);
    return hipGetLastError();
}

}  // namespace mlba
