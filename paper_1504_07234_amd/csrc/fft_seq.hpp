// Compiled transforms of short sequences, several to a workgroup: the image
// sides n = 2^a and 3 2^a from 64 to 1536 of the preconditioner's passes.
//
// The run-time plan (lds_stockham) spends such a pass on latency: table reads
// in front of every stage, two barriers per stage, index arithmetic with
// run-time strides, and few workgroups.  Here a sequence belongs to n / 8
// threads (rounded up to a power of two), one radix-8 butterfly each: up to
// n = 512 they lie in one wave, whose LDS accesses need no barrier at all.  The
// table entries of every stage are loaded with the data, the first stage takes
// its inputs from registers and the last leaves its outputs there.  The radices
// and their order are the run-time plan's, so the values are too, bit for bit.
//
// Forward rows / columns / inverse rows, on the run-time plan -> here, us:
//   64 x 64 BCCB       5.0 / 10.2 / 4.2  -> 2.8 / 3.7 / 2.7
//   512 x 512 BCCB     5.7 / 13.3 / 5.7  -> 3.2 / 4.7 / 3.8
//   512 x 512 DCT      6.4 / 18.3 / 7.3  -> 4.6 / 5.5 / 4.7
//   1536 x 1536 DCT    15.4 / 25.5 / 20.1 -> 11.8 / 15.3 / 14.7
// Below 64 a sequence leaves threads without a butterfly; above 1536 one fills a
// workgroup, which the compiled 2048 and 2304 transforms serve.
#pragma once

#include "fft_core.hpp"

namespace mlba {

__host__ __device__ constexpr bool seq_length(int n) {
    int m = n % 3 == 0 ? n / 3 : n;
    if (n < 64 || n > 1536) return false;
    while (m % 2 == 0) m /= 2;
    return m == 1;
}

// threads of a sequence
__host__ __device__ constexpr int seq_threads(int n) {
    int t = 8;
    while (8 * t < n) t *= 2;
    return t;
}

// the run-time plan's radices: 8 .. 8, then 4 or 2, then 3
__host__ __device__ constexpr FixedPlan seq_plan(int n) {
    FixedPlan p{};
    int a = 0, m = n;
    while (m % 2 == 0) {
        m /= 2;
        ++a;
    }
    for (; a >= 3; a -= 3) p.radix[p.nst++] = 8;
    if (a == 2) p.radix[p.nst++] = 4;
    if (a == 1) p.radix[p.nst++] = 2;
    if (m == 3) p.radix[p.nst++] = 3;
    int ns = 1;
    for (int s = 0; s < p.nst; ++s) {
        p.ns[s] = ns;
        ns *= p.radix[s];
    }
    return p;
}

// LDS slots of a sequence; an odd multiple of 2 slots apart, so that the
// sequences of a wave start on distinct banks
__host__ __device__ constexpr int seq_slots(int n) { return ((n + lds_pad_of(n - 1) + 1) / 4) * 4 + 2 + 4; }
__host__ __device__ constexpr size_t seq_lds_bytes(int n, int seqs) { return (size_t)seq_slots(n) * seqs * 8; }

// Orders a sequence's LDS accesses: a wave's are in order by themselves.
template <int N>
__device__ __forceinline__ void seq_sync() {
    if constexpr (seq_threads(N) <= 64) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

__host__ __device__ constexpr int seq_butterflies(int n, int s) {  // per thread, stage s
    return (n / seq_plan(n).radix[s] + seq_threads(n) - 1) / seq_threads(n);
}

__host__ __device__ constexpr int seq_tw_offset(int n, int stage) {
    const FixedPlan p = seq_plan(n);
    int off = 0;
    for (int s = 1; s < stage && s < p.nst; ++s) off += seq_butterflies(n, s) * tw_table_loads(p.radix[s]);
    return off;
}

template <int N>
struct Seq {
    static constexpr FixedPlan P = seq_plan(N);
    static constexpr int T = seq_threads(N);
    static constexpr int NB0 = N / 8;                    // the first stage: one radix-8 butterfly per thread
    static constexpr int L = P.nst - 1, RL = P.radix[L];  // the last stage
    static constexpr int NBL = N / RL, BL = seq_butterflies(N, L);
    static constexpr int TW = seq_tw_offset(N, P.nst) > 0 ? seq_tw_offset(N, P.nst) : 1;
    static_assert(P.radix[0] == 8 && NB0 <= T && P.nst >= 2, "one radix-8 butterfly per thread first");

    float2 tw[TW];  // the table entries of every stage but the first

    template <int S = 1>
    __device__ __forceinline__ void load_tw(const float2* __restrict__ table, int t) {
        if constexpr (S < P.nst) {
            constexpr int R = P.radix[S], NS = P.ns[S], nb = N / R, off = seq_tw_offset(N, S), E = tw_table_loads(R);
#pragma unroll
            for (int i = 0; i < seq_butterflies(N, S); ++i) {
                const int e = ((t + i * T) % NS) * (N / (NS * R));
                if (nb % T == 0 || t + i * T < nb)
#pragma unroll
                    for (int q = 0; q < E; ++q) tw[off + i * E + q] = table[e << q];
            }
            load_tw<S + 1>(table, t);
        }
    }

    // stage 0 from registers (v[r] = element t + r NB0)
    template <int DIR>
    __device__ __forceinline__ void first(float2 (&v)[8], float2* buf, int t) {
        if (NB0 == T || t < NB0) {
            dft<8, DIR>(v);
#pragma unroll
            for (int r = 0; r < 8; ++r) buf[lds_slot(t * 8 + r)] = v[r];
        }
        seq_sync<N>();
    }

    template <int S, int DIR>
    __device__ __forceinline__ void read(const float2* buf, int t, float2 (*v)[P.radix[S]]) {
        constexpr int R = P.radix[S], nb = N / R, E = tw_table_loads(R);
#pragma unroll
        for (int i = 0; i < seq_butterflies(N, S); ++i) {
            const int j = t + i * T;
            if (nb % T == 0 || j < nb) {
                float2 w[R];
                twiddle_powers_raw<R, DIR>(tw + seq_tw_offset(N, S) + i * E, w);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float2 x = buf[lds_slot(j + r * nb)];
                    if (r > 0) x = cmul(x, w[r]);
                    v[i][r] = x;
                }
                dft<R, DIR>(v[i]);
            }
        }
    }

    template <int DIR, int S = 1>
    __device__ __forceinline__ void middle(float2* buf, int t) {
        if constexpr (S < L) {
            constexpr int R = P.radix[S], NS = P.ns[S], nb = N / R;
            float2 v[seq_butterflies(N, S)][R];
            read<S, DIR>(buf, t, v);
            seq_sync<N>();
#pragma unroll
            for (int i = 0; i < seq_butterflies(N, S); ++i) {
                const int j = t + i * T;
                if (nb % T == 0 || j < nb) {
                    const int jm = j % NS, dst = (j - jm) * R + jm;
#pragma unroll
                    for (int r = 0; r < R; ++r) buf[lds_slot(dst + r * NS)] = v[i][r];
                }
            }
            seq_sync<N>();
            middle<DIR, S + 1>(buf, t);
        }
    }

    // From v (first-stage inputs) to u: u[i][r] = element (t + i T) + r NBL.
    template <int DIR>
    __device__ __forceinline__ void run(float2 (&v)[8], float2 (&u)[BL][RL], float2* buf, int t) {
        first<DIR>(v, buf, t);
        middle<DIR>(buf, t);
        read<L, DIR>(buf, t, u);
    }

    // f(i, r, element) over the last stage's outputs of thread t
    template <class F>
    static __device__ __forceinline__ void outputs(int t, F f) {
#pragma unroll
        for (int i = 0; i < BL; ++i) {
            const int j = t + i * T;
            if (NBL % T == 0 || j < NBL)
#pragma unroll
                for (int r = 0; r < RL; ++r) f(i, r, j + r * NBL);
        }
    }

    // f(r, element) over the first stage's inputs of thread t
    template <class F>
    static __device__ __forceinline__ void inputs(int t, F f) {
        if (NB0 == T || t < NB0)
#pragma unroll
            for (int r = 0; r < 8; ++r) f(r, t + r * NB0);
    }

    static __device__ __forceinline__ void put(const float2 (&u)[BL][RL], float2* buf, int t) {
        outputs(t, [&](int i, int r, int e) { buf[lds_slot(e)] = u[i][r]; });
    }
};

// A sequence inside one wave orders its accesses by itself and may leave the
// kernel when it has nothing to do; one of several waves stays for the
// workgroup's barriers.
template <int N>
constexpr bool seq_alone() {
    return seq_threads(N) <= 64;
}

// Whether sequence k of `count`, G to a workgroup, is one of them.
template <int COUNT, int G>
__device__ __forceinline__ bool seq_live(int k) {
    if constexpr (COUNT % G == 0) return true;
    else return k < COUNT;
}

// Workgroup-wide order where a pass touches other sequences' slots.
template <int N, int THREADS>
__device__ __forceinline__ void seq_sync_all() {
    if constexpr (THREADS > 64) __syncthreads();
    else seq_sync<N>();
}

// ---- Bluestein form ----------------------------------------------------------

// Length-n DFT of the one sequence in buf[0, n) by Bluestein's identity
// jk = (j^2 + k^2 - (k - j)^2) / 2:
//   X_k = c_k sum_j (x_j c_j) conj(c_{k-j}),  c_k = exp(-i pi k^2 / n),
// the sum a circular convolution of length M >= 2n - 1 done with two M-point
// transforms and the stored spectrum of conj(c) (scaled by 1/M).  The inverse
// direction is conj(DFT(conj x)).  The sequence's M / 8 threads do the work:
// within one wave the other waves wait at the end, above that they repeat it
// (the same values to the same slots) to keep the barriers.  A pass is bound by
// the latency of its chain of stages: on the run-time plan of the smallest
// 2^a 3^b 5^c >= 2n - 1 each of them had a table read, run-time strides and two
// barriers.  P at n = 66 / 226 / 514 / 1022, DCT: 42 / 45 / 69 / 74 -> 21 / 23 /
// 37 / 47 us; antireflective n = 196 / 500: 50 / 86 -> 30 / 35 us.  M is a power of
// two also where 3 2^a or 5-smooth is shorter (n = 66: m = 135 -> 256, 514:
// 1080 -> 2048): the longer compiled chain is still half the run-time plan's.
template <int DIR, int M>
__device__ __forceinline__ void seq_bluestein(float2* buf, int n, const float2* __restrict__ tw) {
    using Q = Seq<M>;
    const float2* __restrict__ chirp = tw + M;
    const float2* __restrict__ bspec = tw + M + n;
    const int t = threadIdx.x & (Q::T - 1);
    if (Q::T > 64 || threadIdx.x < 64) {
        Q q;
        q.load_tw(tw, t);
        float2 v[8], c[8], u[Q::BL][Q::RL], b[Q::BL][Q::RL], co[Q::BL][Q::RL];
        Q::inputs(t, [&](int r, int k) {
            c[r] = k < n ? chirp[k] : make_float2(0.0f, 0.0f);
            v[r] = k < n ? buf[lds_slot(k)] : make_float2(0.0f, 0.0f);
        });
        Q::outputs(t, [&](int i, int r, int k) {
            b[i][r] = bspec[k];
            co[i][r] = k < n ? chirp[k] : make_float2(0.0f, 0.0f);
        });
        Q::inputs(t, [&](int r, int) {
            if (DIR > 0) v[r].y = -v[r].y;
            v[r] = cmul(v[r], c[r]);
        });
        seq_sync<M>();  // every x read before the transform's stages overwrite it
        q.template run<-1>(v, u, buf, t);
        Q::outputs(t, [&](int i, int r, int) { u[i][r] = cmul(u[i][r], b[i][r]); });
        seq_sync<M>();
        Q::put(u, buf, t);
        seq_sync<M>();
        Q::inputs(t, [&](int r, int k) { v[r] = buf[lds_slot(k)]; });
        seq_sync<M>();
        q.template run<1>(v, u, buf, t);
        seq_sync<M>();
        Q::outputs(t, [&](int i, int r, int k) {
            if (k < n) {
                float2 x = cmul(u[i][r], co[i][r]);
                if (DIR > 0) x.y = -x.y;
                buf[lds_slot(k)] = x;
            }
        });
    }
    __syncthreads();
}

template <int DIR>
__device__ void lds_bluestein_seq(float2* buf, const FftDesc& fd, const float2* __restrict__ tw) {
    switch (fd.m) {
        case 64: return seq_bluestein<DIR, 64>(buf, fd.n, tw);
        case 128: return seq_bluestein<DIR, 128>(buf, fd.n, tw);
        case 256: return seq_bluestein<DIR, 256>(buf, fd.n, tw);
        case 512: return seq_bluestein<DIR, 512>(buf, fd.n, tw);
        case 1024: return seq_bluestein<DIR, 1024>(buf, fd.n, tw);
        default: return seq_bluestein<DIR, 2048>(buf, fd.n, tw);
    }
}

// ---- BCCB passes: THREADS / seq_threads(N) sequences per workgroup -----------

// row pairs -> T[k][row], k = 0 .. N/2; pair0: the workgroup's first pair.
// src.load(i), src.value(i, loaded): the value at flat index i of the N x N input
// (each called once per element, every load of a thread before its first value).
template <int N, int THREADS, class Src>
__device__ __forceinline__ void seq_rows_r2c(Src src, float2* __restrict__ T, int ts, const float2* __restrict__ tw,
                                             int blk, float2* lds) {
    constexpr int TH = seq_threads(N), G = THREADS / TH, half = N / 2 + 1;
    static_assert(TH <= 64 || (N / 2) % G == 0, "a sequence of several waves is live: barriers inside the branch");
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, pair0 = blk * G;
    float2* buf = lds + g * seq_slots(N);
    Seq<N> q;
    q.load_tw(tw, t);
    if (2 * (pair0 + g) < N) {
        float2 v[8], u[Seq<N>::BL][Seq<N>::RL];
        const size_t ra = (size_t)2 * (pair0 + g) * N;
        typename Src::Raw a[8], b[8];
        Seq<N>::inputs(t, [&](int r, int x) {
            a[r] = src.load(ra + x);
            b[r] = src.load(ra + N + x);
        });
        Seq<N>::inputs(t, [&](int r, int x) {
            v[r] = make_float2(src.value(ra + x, a[r]), src.value(ra + N + x, b[r]));
        });
        q.template run<-1>(v, u, buf, t);
        seq_sync<N>();
        Seq<N>::put(u, buf, t);
    }
    seq_sync_all<N, THREADS>();
    for (int idx = threadIdx.x; idx < G * half; idx += THREADS) {
        const int k = idx / G, h = idx % G;
        if (2 * (pair0 + h) >= N) continue;
        const float2* b = lds + h * seq_slots(N);
        const float2 Z = b[lds_slot(k)];
        const float2 Zc = cconj(b[lds_slot(k == 0 ? 0 : N - k)]);
        const float2 Xa = cscale(cadd(Z, Zc), 0.5f);
        const float2 D = csub(Z, Zc);
        const float2 Xb = make_float2(0.5f * D.y, -0.5f * D.x);  // D / (2i)
        *reinterpret_cast<float4*>(T + (size_t)k * ts + 2 * (pair0 + h)) = make_float4(Xa.x, Xa.y, Xb.x, Xb.y);
    }
}

// columns: forward, inv / (spec + alpha) (times conj(lamc)), inverse; sstore,
// sfwd and eacc as in fft_cols_body
template <int N, int THREADS>
__device__ __forceinline__ void seq_cols(float2* __restrict__ T, int ts, const float* __restrict__ spec, float alpha,
                                         float inv, const float2* __restrict__ tw, int blk, float2* lds,
                                         const float2* __restrict__ lamc = nullptr,
                                         float2* __restrict__ sstore = nullptr,
                                         const float2* __restrict__ sfwd = nullptr,
                                         float* __restrict__ eacc = nullptr) {
    constexpr int TH = seq_threads(N), G = THREADS / TH, half = N / 2 + 1;
    using Q = Seq<N>;
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, k = blk * G + g;
    float2* buf = lds + g * seq_slots(N);
    const bool live = seq_live<half, G>(k);
    if (seq_alone<N>() && !live) return;
    Q q;
    q.load_tw(tw, t);
    float2 v[8], u[Q::BL][Q::RL];
    float sp[Q::BL][Q::RL];
    float2* col = T + (size_t)k * ts;
    const size_t base = (size_t)k * N;  // dense [N/2+1][N] spectrum
    Q::inputs(t, [&](int r, int y) { v[r] = live ? col[y] : make_float2(0.0f, 0.0f); });
    Q::outputs(t, [&](int i, int r, int y) { sp[i][r] = live ? spec[base + y] : 1.0f; });
    q.template run<-1>(v, u, buf, t);
    Q::outputs(t, [&](int i, int r, int y) {
        if (!live) return;
        float2 x = cscale(u[i][r], inv / (sp[i][r] + alpha));
        if (lamc) x = cmul(x, cconj(lamc[base + y]));
        if (sstore) sstore[base + y] = x;  // reverse sweep of unrolled iterations
        if (eacc) {
            const float2 f = sfwd[base + y];
            eacc[base + y] += fmaf(x.x, f.x, x.y * f.y);
        }
        u[i][r] = x;
    });
    seq_sync<N>();
    if constexpr (Q::RL == 8 && Q::BL == 1) {  // the last stage's outputs are the first one's inputs
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = u[0][r];
    } else {
        Q::put(u, buf, t);
        seq_sync<N>();
        Q::inputs(t, [&](int r, int y) { v[r] = buf[lds_slot(y)]; });
        seq_sync<N>();
    }
    q.template run<1>(v, u, buf, t);
    Q::outputs(t, [&](int i, int r, int y) {
        if (live) col[y] = u[i][r];
    });
}

// columns: inverse transform of the real dense spectrum e into T
template <int N, int THREADS>
__device__ __forceinline__ void seq_cols_inverse_real(const float* __restrict__ e, float2* __restrict__ T, int ts,
                                                      const float2* __restrict__ tw, int blk, float2* lds) {
    constexpr int TH = seq_threads(N), G = THREADS / TH, half = N / 2 + 1;
    using Q = Seq<N>;
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, k = blk * G + g;
    const bool live = seq_live<half, G>(k);
    if (seq_alone<N>() && !live) return;
    Q q;
    q.load_tw(tw, t);
    float2 v[8], u[Q::BL][Q::RL];
    Q::inputs(t, [&](int r, int y) { v[r] = make_float2(live ? e[(size_t)k * N + y] : 0.0f, 0.0f); });
    q.template run<1>(v, u, lds + g * seq_slots(N), t);
    Q::outputs(t, [&](int i, int r, int y) {
        if (live) T[(size_t)k * ts + y] = u[i][r];
    });
}

// put(i, v): the value v of flat index i of the N x N output
template <int N, int THREADS, class Put>
__device__ __forceinline__ void seq_rows_c2r(const float2* __restrict__ T, int ts, Put put,
                                             const float2* __restrict__ tw, int blk, float2* lds) {
    constexpr int TH = seq_threads(N), G = THREADS / TH, half = N / 2 + 1;
    using Q = Seq<N>;
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, pair0 = blk * G;
    float2* buf = lds + g * seq_slots(N);
    Q q;
    q.load_tw(tw, t);
    constexpr int PER = (G * half + THREADS - 1) / THREADS;
    float4 in[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int idx = threadIdx.x + i * THREADS, k = idx / G, h = idx % G;
        if (idx < G * half && 2 * (pair0 + h) < N)
            in[i] = *reinterpret_cast<const float4*>(T + (size_t)k * ts + 2 * (pair0 + h));
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int idx = threadIdx.x + i * THREADS, k = idx / G, h = idx % G;
        if (idx < G * half && 2 * (pair0 + h) < N) {
            float2* b = lds + h * seq_slots(N);
            float2 Xa = make_float2(in[i].x, in[i].y), Xb = make_float2(in[i].z, in[i].w);
            const bool edge = k == 0 || 2 * k == N;
            if (edge) Xa.y = Xb.y = 0.0f;  // spectra of real rows are real at DC and Nyquist
            b[lds_slot(k)] = make_float2(Xa.x - Xb.y, Xa.y + Xb.x);                 // Xa + i Xb
            if (!edge) b[lds_slot(N - k)] = make_float2(Xa.x + Xb.y, -Xa.y + Xb.x);  // conj(Xa) + i conj(Xb)
        }
    }
    seq_sync_all<N, THREADS>();
    static_assert(seq_alone<N>() || (N / 2) % G == 0, "a sequence of several waves is live: barriers ahead");
    if (2 * (pair0 + g) >= N) return;
    float2 v[8], u[Q::BL][Q::RL];
    Q::inputs(t, [&](int r, int k) { v[r] = buf[lds_slot(k)]; });
    seq_sync<N>();
    q.template run<1>(v, u, buf, t);
    const size_t ra = (size_t)2 * (pair0 + g) * N;
    Q::outputs(t, [&](int i, int r, int x) {
        put(ra + x, u[i][r].x);
        put(ra + N + x, u[i][r].y);
    });
}

// ---- DCT passes ------------------------------------------------------------

// sample at position q of the reordered sequence (evens ascending, odds descending)
__device__ __forceinline__ int dct_sample(int q, int n) { return 2 * q < n ? 2 * q : 2 * (n - 1 - q) + 1; }

// V = conj(w_k) (Y_k - i Y_{n-k}) of both rows, packed: the input of the DCT-III's transform
__device__ __forceinline__ float2 dct_unfold(float2 w, float2 Y, float2 Yr) {
    const float2 wc = cconj(w);
    const float2 V1 = cmul(wc, make_float2(Y.x, -Yr.x));
    const float2 V2 = cmul(wc, make_float2(Y.y, -Yr.y));
    return make_float2(V1.x - V2.y, V1.y + V2.x);  // V1 + i V2
}

// both rows' coefficients from Z_k and Z_{n-k}
__device__ __forceinline__ float2 dct_fold(float2 w, float2 Z, float2 Zr) {
    const float2 Zc = cconj(Zr);
    const float2 Va = cscale(cadd(Z, Zc), 0.5f);
    const float2 D = csub(Z, Zc);
    const float2 Vb = make_float2(0.5f * D.y, -0.5f * D.x);
    return make_float2(w.x * Va.x - w.y * Va.y, w.x * Vb.x - w.y * Vb.y);
}

template <int N, int THREADS>
__device__ __forceinline__ void seq_dct_rows_fwd(const float* __restrict__ src, float* __restrict__ Tr, int ts,
                                                 const float2* __restrict__ tw, const float2* __restrict__ dtw,
                                                 int blk, float2* lds) {
    constexpr int TH = seq_threads(N), G = THREADS / TH;
    static_assert(TH <= 64 || (N / 2) % G == 0, "a sequence of several waves is live: barriers inside the branch");
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, pair0 = blk * G;
    float2* buf = lds + g * seq_slots(N);
    Seq<N> q;
    q.load_tw(tw, t);
    if (2 * (pair0 + g) < N) {
        float2 v[8], u[Seq<N>::BL][Seq<N>::RL];
        const float* row = src + (size_t)2 * (pair0 + g) * N;
        Seq<N>::inputs(t, [&](int r, int e) {
            const int x = dct_sample(e, N);
            v[r] = make_float2(row[x], row[N + x]);
        });
        q.template run<-1>(v, u, buf, t);
        seq_sync<N>();
        Seq<N>::put(u, buf, t);
    }
    seq_sync_all<N, THREADS>();
    for (int idx = threadIdx.x; idx < G * N; idx += THREADS) {
        const int k = idx / G, h = idx % G;
        if (2 * (pair0 + h) >= N) continue;
        const float2* b = lds + h * seq_slots(N);
        *reinterpret_cast<float2*>(Tr + (size_t)k * ts + 2 * (pair0 + h)) =
            dct_fold(dtw[k], b[lds_slot(k)], b[lds_slot(k == 0 ? 0 : N - k)]);
    }
}

// pairs of Tr rows: DCT-II, inv / (spec + alpha) (times lamr), DCT-III
template <int N, int THREADS>
__device__ __forceinline__ void seq_dct_cols(float* __restrict__ Tr, int ts, const float* __restrict__ spec,
                                             float alpha, float inv, const float2* __restrict__ tw,
                                             const float2* __restrict__ dtw, int blk, float2* lds,
                                             const float* __restrict__ lamr = nullptr) {
    constexpr int TH = seq_threads(N), G = THREADS / TH;
    using Q = Seq<N>;
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, p = blk * G + g;
    float2* buf = lds + g * seq_slots(N);
    static_assert(seq_alone<N>() || (N / 2) % G == 0, "a sequence of several waves is live: barriers ahead");
    if (2 * p >= N) return;
    Q q;
    q.load_tw(tw, t);
    float* r1 = Tr + (size_t)2 * p * ts;
    float* r2 = r1 + ts;
    const size_t s1 = (size_t)2 * p * N;  // dense [N][N] spectrum
    float2 v[8], u[Q::BL][Q::RL], w[8], f[8];
    Q::inputs(t, [&](int r, int e) {
        const int l = dct_sample(e, N);
        v[r] = make_float2(r1[l], r2[l]);
    });
    Q::inputs(t, [&](int r, int l) {
        w[r] = dtw[l];
        f[r] = make_float2(spec[s1 + l], spec[s1 + N + l]);
    });
    q.template run<-1>(v, u, buf, t);
    seq_sync<N>();
    Q::put(u, buf, t);
    seq_sync<N>();
    float2 Y[8];
    Q::inputs(t, [&](int r, int l) {
        float f1 = inv / (f[r].x + alpha), f2 = inv / (f[r].y + alpha);
        if (lamr) {
            f1 *= lamr[s1 + l];
            f2 *= lamr[s1 + N + l];
        }
        const float2 c = dct_fold(w[r], buf[lds_slot(l)], buf[lds_slot(l == 0 ? 0 : N - l)]);
        Y[r] = make_float2(c.x * f1, c.y * f2);
    });
    seq_sync<N>();
    Q::inputs(t, [&](int r, int l) { buf[lds_slot(l)] = Y[r]; });
    seq_sync<N>();
    Q::inputs(t, [&](int r, int l) {
        v[r] = dct_unfold(w[r], Y[r], l == 0 ? make_float2(0.0f, 0.0f) : buf[lds_slot(N - l)]);
    });
    seq_sync<N>();
    q.template run<1>(v, u, buf, t);
    Q::outputs(t, [&](int i, int r, int e) {
        const int l = dct_sample(e, N);
        r1[l] = u[i][r].x;
        r2[l] = u[i][r].y;
    });
}

template <int N, int THREADS>
__device__ __forceinline__ void seq_dct_rows_inv(const float* __restrict__ Tr, int ts, float* __restrict__ dst,
                                                 const float2* __restrict__ tw, const float2* __restrict__ dtw,
                                                 int blk, float2* lds, int accum = 0) {
    constexpr int TH = seq_threads(N), G = THREADS / TH;
    using Q = Seq<N>;
    const int g = threadIdx.x / TH, t = threadIdx.x % TH, pair0 = blk * G;
    float2* buf = lds + g * seq_slots(N);
    Q q;
    q.load_tw(tw, t);
    constexpr int PER = (G * N + THREADS - 1) / THREADS;
    float2 in[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int idx = threadIdx.x + i * THREADS, k = idx / G, h = idx % G;
        if (idx < G * N && 2 * (pair0 + h) < N)
            in[i] = *reinterpret_cast<const float2*>(Tr + (size_t)k * ts + 2 * (pair0 + h));
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int idx = threadIdx.x + i * THREADS, k = idx / G, h = idx % G;
        if (idx < G * N && 2 * (pair0 + h) < N) lds[h * seq_slots(N) + lds_slot(k)] = in[i];
    }
    seq_sync_all<N, THREADS>();
    static_assert(seq_alone<N>() || (N / 2) % G == 0, "a sequence of several waves is live: barriers ahead");
    if (2 * (pair0 + g) >= N) return;
    float2 v[8], u[Q::BL][Q::RL];
    Q::inputs(t, [&](int r, int k) {
        v[r] = dct_unfold(dtw[k], buf[lds_slot(k)], k == 0 ? make_float2(0.0f, 0.0f) : buf[lds_slot(N - k)]);
    });
    seq_sync<N>();
    q.template run<1>(v, u, buf, t);
    float* row = dst + (size_t)2 * (pair0 + g) * N;
    Q::outputs(t, [&](int i, int r, int e) {
        const int x = dct_sample(e, N);
        row[x] = accum ? row[x] + u[i][r].x : u[i][r].x;
        row[N + x] = accum ? row[N + x] + u[i][r].y : u[i][r].y;
    });
}

// the lengths of seq_length
#define MLBA_SEQ_LENGTHS(X) X(64) X(96) X(128) X(192) X(256) X(384) X(512) X(768) X(1024) X(1536)

// Threads of a single image's workgroup: one wave, or one sequence above that.
__host__ __device__ constexpr int seq_block(int n) { return seq_threads(n) > 64 ? seq_threads(n) : 64; }
// sequences of a workgroup of `threads`
__host__ __device__ constexpr int seq_group(int n, int threads) { return threads / seq_threads(n); }

}  // namespace mlba
