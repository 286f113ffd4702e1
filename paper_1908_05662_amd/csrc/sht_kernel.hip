// Spherical-harmonic analysis of HEALPix I, Q, U maps and their angular power
// spectra, in FP64: the spectrum estimator the paper applies to maps made from
// the TOD (Sec. 6.2).  Definitions (orthonormal Y_lm with the Condon-Shortley
// phase; spin-2 harmonics of Goldberg et al. 1967; E and B as in Zaldarriaga &
// Seljak 1997 with the HEALPix sign convention) are stated in include/pisco.h.
//
// Kernels:
//   ring_fourier_kernel  one workgroup per ring: F_r(m) = w sum_j x_j e^{-i m phi_j}
//                        for every field, by an FFT in LDS (direct DFT over the
//                        odd factor of the ring length, then radix-2 Stockham
//                        passes over its power-of-two factor), read at m mod n;
//   steps_kernel         the recurrence steps of every (l, m), once per call;
//   alm_kernel           one workgroup per m: lanes own north/south ring pairs,
//                        run the recurrences of lambda_lm and of the spin-2
//                        functions in l (mantissa plus a carried power-of-two
//                        exponent, so sin^m theta cannot underflow) and
//                        accumulate against the pair's ring sums; every four l a
//                        wave adds its lanes, every 64 l the workgroup its waves;
//   alm2cl_kernel        C_l of a pair of a_lm, or of the six pairs of T, E, B;
//   alm2ring_kernel      the synthesis: the same recurrences, lanes own ring pairs
//                        and sum over l in registers (no cross-lane sums);
//   ring_synth_kernel    one workgroup per ring: the m sums folded onto the ring
//                        length, then the same LDS FFT as the analysis.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "sht_internal.h"

namespace pisco {
namespace {

constexpr int SCALE = 256;               // exponent step of the carried recurrence
constexpr int NCOMP = 6;                 // a^T, a^E, a^B (re, im)
constexpr int LCHUNK = 64;               // l values per coefficient table

struct RingGeom {
    int64_t first;
    int n;
    double z, s, phi0_over_pi;
    double omz;                          // 1 - z without the cancellation next to the north pole
};

// Ring i = r + 1 of the RING scheme (Gorski et al. 2005, Sec. 4): colatitude
// from exact integer ratios, first pixel and its longitude / pi.
__device__ inline RingGeom sht_ring(int N, int r) {
    const int i = r + 1;
    RingGeom g;
    const double n3 = 3.0 * (double)N * (double)N;
    if (i < N || i > 3 * N) {
        const int k = i < N ? i : 4 * N - i;
        const double t = (double)k * (double)k / n3;      // 1 - |z|
        g.n = 4 * k;
        g.first = i < N ? 2LL * k * (k - 1) : 12LL * N * N - 2LL * k * (k + 1);
        g.z = i < N ? 1.0 - t : t - 1.0;
        g.s = sqrt(t * (2.0 - t));
        g.omz = i < N ? t : 2.0 - t;
        g.phi0_over_pi = 0.25 / (double)k;
    } else {
        g.n = 4 * N;
        g.first = 2LL * N * (N - 1) + (int64_t)(i - N) * 4 * N;
        g.z = (double)(4 * N - 2 * i) / (3.0 * N);
        g.s = sqrt((double)(2 * i - N) * (double)(7 * N - 2 * i)) / (3.0 * N);
        g.omz = (double)(2 * i - N) / (3.0 * N);
        g.phi0_over_pi = ((i - N) & 1) == 0 ? 0.25 / (double)N : 0.0;
    }
    return g;
}

// ----------------------------------------------------------------------
// Ring transforms.  A workgroup takes a north ring and its mirror (same length n =
// 4 k and first longitude) and transforms up to three complex signals:
// T_N + i T_S, Q_N + i U_N and Q_S + i U_S.  The sums the other kernels want of a
// signal z are P_m = sum_j z_j e^{-i m phi_j} and M_m = sum_j conj(z_j) e^{-i m phi_j},
// with Z the signal's DFT P_m = e^{-i m phi_0} Z[m], M_m = e^{-i m phi_0} conj Z[-m]
// (indices mod n): for spin signals these are the sums of Q + iU and Q - iU, for
// T of T_N + i T_S and T_N - i T_S.  Stored [signal][m][pair][P, M].
//
// A power-of-two n (the belt, a few polar rings) is one FFT in LDS: radix-4
// Stockham passes in place (a pass reads everything into registers, then writes),
// twiddles from a quarter-wave table.  Any other k splits n = 4 k by one radix-4
// step into four transforms of length k, each a chirp convolution (Bluestein 1970)
// of power-of-two length >= 2 k - 1 by the same FFT; the chirp's spectrum stays in
// registers, and the chirps and the radix-4 step's twiddles are one exponential
// e^{-i pi (4 j^2 + 2 a j) / n} of an exact integer.  (A DFT of the odd factor of n
// summed directly took O(n) operations a point, an LDS read per multiply-add, and
// the passes called sincospi for every butterfly: 3.4 ms at nside 1024, lmax 3071,
// now 0.86 ms, in passes of LDS reads, barriers and writes; 54 us at nside 128 in three
// launches, now 20.)
// ----------------------------------------------------------------------
// Pair of workgroup b: the chirp rings first (the longest), then the belt; four
// consecutive pairs on one die (workgroups are dealt to the eight in turn), so
// that the 32-byte results of neighbouring pairs meet in one L2.
__device__ inline int pair_of_block(int N) {
    int b = blockIdx.x;
    if (N >= 16) b = ((b >> 5) << 5) + ((b & 7) << 2) + ((b >> 3) & 3);
    return b < N ? N - 1 - b : b;
}

// e^{-i pi t / n}
__device__ inline double2 cis(int t, int n) {
    double sn, cs;
    sincospi((double)t / (double)n, &sn, &cs);
    return make_double2(cs, -sn);
}

__device__ inline double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

// (-i)^p z
__device__ inline double2 turn(double2 z, int p) {
    p &= 3;
    const double x = p & 1 ? z.y : z.x, y = p & 1 ? -z.x : z.y;
    return p & 2 ? make_double2(-x, -y) : make_double2(x, y);
}

// Orders this wave's LDS writes before its later LDS reads (lanes exchange
// values inside one wave; no other wave touches the region).
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// FFT of 2^L values in LDS by a group of NT threads (at most 4 B NT values), thread
// tid of the group; groups of a workgroup run side by side on their own data, in
// step.  A group of one wave needs no barrier.
template <int NT, int B>
struct LdsFft {
    double2 *x;                          // data
    const double2 *tab;                  // e^{-2 pi i t / M}, t < M / 4
    int L, M, tid;
    static __device__ inline void sync() {
        if constexpr (NT == 64) wave_sync();
        else __syncthreads();
    }
    __device__ inline void init(double2 *data, double2 *table, int log2m, int t) {
        x = data;
        tab = table;
        L = log2m;
        M = 1 << log2m;
        tid = t;
        for (int i = threadIdx.x; 4 * i < M; i += blockDim.x) table[i] = cis(2 * i, M);
        __syncthreads();
    }
    // x <- DFT(x), natural order; the group's writes to x need no barrier of their own, the result none
    __device__ inline void run() const {
        sync();
        int ls = 0;                                                   // log2 of the finished length
        if (L & 1) {
            double2 u[2 * B], v[2 * B];
#pragma unroll
            for (int i = 0; i < 2 * B; ++i) {
                const int j = tid + i * NT;
                if (2 * j < M) {
                    u[i] = x[j];
                    v[i] = x[j + M / 2];
                }
            }
            sync();
#pragma unroll
            for (int i = 0; i < 2 * B; ++i) {
                const int j = tid + i * NT;
                if (2 * j < M) {
                    x[2 * j] = make_double2(u[i].x + v[i].x, u[i].y + v[i].y);
                    x[2 * j + 1] = make_double2(u[i].x - v[i].x, u[i].y - v[i].y);
                }
            }
            sync();
            ls = 1;
        }
        const int q = M / 4;
        for (; ls < L; ls += 2) {
            double2 o[B][4];
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int j = tid + i * NT;
                if (j < q) {
                    const int t = (j & ((1 << ls) - 1)) << (L - 2 - ls);
                    const int t2 = 2 * t, t3 = 3 * t;
                    const double2 w1 = tab[t], w2 = turn(tab[t2 & (q - 1)], t2 >> (L - 2));
                    const double2 w3 = turn(tab[t3 & (q - 1)], t3 >> (L - 2));
                    const double2 x0 = x[j], x1 = cmul(x[j + q], w1), x2 = cmul(x[j + 2 * q], w2), x3 = cmul(x[j + 3 * q], w3);
                    const double2 a = make_double2(x0.x + x2.x, x0.y + x2.y), b = make_double2(x0.x - x2.x, x0.y - x2.y);
                    const double2 c = make_double2(x1.x + x3.x, x1.y + x3.y);
                    const double2 d = make_double2(x1.y - x3.y, x3.x - x1.x);       // -i (x1 - x3)
                    o[i][0] = make_double2(a.x + c.x, a.y + c.y);
                    o[i][1] = make_double2(b.x + d.x, b.y + d.y);
                    o[i][2] = make_double2(a.x - c.x, a.y - c.y);
                    o[i][3] = make_double2(b.x - d.x, b.y - d.y);
                }
            }
            sync();
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int j = tid + i * NT;
                if (j < q) {
                    const int k = j & ((1 << ls) - 1), at = ((j - k) << 2) + k;
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[at + (r << ls)] = o[i][r];
                }
            }
            sync();
        }
    }
};

// The chirp transform of length k (not a power of two, k <= B NT), element
// j = tid + i NT in u[i].
template <int NT, int B>
struct Chirp {
    LdsFft<NT, B> f;
    int k, n;
    double2 spec[2 * B];                 // DFT of e^{i pi j^2 / k}, over M
    __device__ inline double2 phase(int j, int a) const {             // e^{-i pi (4 j^2 + 2 a j) / n}
        return cis((4 * j * j + 2 * a * j) % (2 * n), n);              // j <= 1024
    }
    __device__ inline void init(double2 *data, double2 *table, int ring_k, int tid) {
        k = ring_k;
        n = 4 * k;
        f.init(data, table, 32 - __clz(2 * k - 2), tid);              // 2^L >= 2 k - 1
        const double inv = 1.0 / (double)f.M;
#pragma unroll
        for (int i = 0; i < 2 * B; ++i) {
            const int j = tid + i * NT;
            if (j < f.M) {
                const int d = j < k ? j : f.M - j;
                const double2 c = d < k ? phase(d, 0) : make_double2(0.0, 0.0);
                f.x[j] = make_double2(inv * c.x, -inv * c.y);
            }
        }
        f.run();
#pragma unroll
        for (int i = 0; i < 2 * B; ++i) {
            const int j = tid + i * NT;
            if (j < f.M) spec[i] = f.x[j];
        }
    }
    // u: inputs times their phases (0 past k); returns the sums before the output phases
    __device__ inline void run(double2 *u, int tid) const {
        f.sync();
#pragma unroll
        for (int i = 0; i < 2 * B; ++i) {
            const int j = tid + i * NT;
            if (j < f.M) f.x[j] = i < B && j < k ? u[i < B ? i : 0] : make_double2(0.0, 0.0);
        }
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            f.run();
            if (half) break;
#pragma unroll
            for (int i = 0; i < 2 * B; ++i) {
                const int j = tid + i * NT;
                if (j < f.M) {
                    const double2 p = cmul(f.x[j], spec[i]);
                    f.x[j] = make_double2(p.x, -p.y);                 // the inverse DFT as conj DFT conj
                }
            }
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int j = tid + i * NT;
            u[i] = j < k ? make_double2(f.x[j].x, -f.x[j].y) : make_double2(0.0, 0.0);
        }
    }
};

// One ring pair: where a signal's samples are (null: zero).
struct RingPair {
    int n, k;
    bool pow2, equator;
    bool shifted;                        // first longitude: pi / n or 0
    int64_t north, south;                // first pixels
    __device__ inline RingPair(int N, int pair) {
        const RingGeom g = sht_ring(N, pair), m = sht_ring(N, 4 * N - 2 - pair);
        n = g.n;
        k = n / 4;
        pow2 = (k & (k - 1)) == 0;
        equator = pair == 2 * N - 1;
        shifted = g.phi0_over_pi > 0.0;
        north = g.first;
        south = m.first;
    }
    // real and imaginary parts of signal s in maps x[3]
    template <class T>
    __device__ inline void parts(T *const x[3], int s, T *&re, T *&im) const {
        re = s == 0 ? x[0] + north : x[1] + (s == 1 ? north : south);
        im = s == 0 ? (equator ? nullptr : x[0] + south) : x[2] + (s == 1 ? north : south);
    }
    __device__ inline int signals(int nfields) const { return nfields == 1 ? 1 : equator ? 2 : 3; }
    // e^{-i m phi_0} z, times w
    __device__ inline double2 phased(double2 z, int m, double w) const {
        const double2 p = cmul(z, shifted ? cis(m, n) : make_double2(1.0, 0.0));
        return make_double2(w * p.x, w * p.y);
    }
};

// G groups of NT threads.  Large maps: one group, a transform at a time, two
// workgroups a compute unit (nside 1024).  Small maps: a workgroup's transforms (three
// signals, or the twelve quarter-length ones of a chirp ring) side by side, since
// the number of rings leaves the chip idle and the chain of passes is the time.
// LDS in units of nside values: see ring_lds.
template <int G>
constexpr int ring_lds(bool syn) {
    const int chirp = 2 * G + (syn ? (G >= 12 ? 12 : 4) : 0), belt = 4 * (G >= 12 ? 3 : G);
    return 1 + (chirp > belt ? chirp : belt);
}

template <int NT, int B, int G>
__global__ void __launch_bounds__(NT * G) ring_fourier_kernel(ShtArgs a) {
    extern __shared__ double2 sh_ring[];
    const int N = a.nside, npairs = 2 * N, grp = threadIdx.x / NT, tid = threadIdx.x % NT;
    const int pair = pair_of_block(N);
    const RingPair R(N, pair);
    const int n = R.n, k = R.k;
    const double w = 4.0 * M_PI / (12.0 * (double)N * (double)N);
    const int ns = R.signals(a.nfields);
    double2 *table = sh_ring, *data = sh_ring + N;
    auto out = [&](int s, int m) { return a.F + (((size_t)s * (a.mmax + 1) + m) * npairs + pair) * 2; };
    if (R.pow2) {
        LdsFft<NT, B> f;
        f.init(data + grp * 4 * N, table, 31 - __clz(n), tid);        // (groups past the signals: no data)
#pragma unroll 1
        for (int s0 = 0; s0 < ns; s0 += G) {
            const int s = s0 + grp;
            const bool ok = s < ns;
            const double *re, *im;
            if (ok) {
                R.parts(a.map, s, re, im);
                for (int j = tid; j < n; j += NT) f.x[j] = make_double2(re[j], im ? im[j] : 0.0);
            }
            if (ok || NT > 64) f.run();                               // idle groups keep the barriers
            if (ok) {
                for (int m = tid; m <= a.mmax; m += NT) {
                    const int i = m & (n - 1);
                    const double2 p = f.x[i], q = f.x[(n - i) & (n - 1)];
                    double2 *o = out(s, m);
                    o[0] = R.phased(p, m, w);
                    o[1] = R.phased(make_double2(q.x, -q.y), m, w);
                }
            }
            __syncthreads();
        }
        return;
    }
    Chirp<NT, B> c;
    c.init(data + grp * 2 * N, table, k, tid);
    double2 post[B];
#pragma unroll
    for (int i = 0; i < B; ++i) post[i] = c.phase(min(tid + i * NT, k), 0);
#pragma unroll 1
    for (int q0 = 0; q0 < 4 * ns; q0 += G) {
        const int t = (q0 + grp) & 3, s = (q0 + grp) >> 2;            // Z[4 j + t] of signal s
        const bool ok = s < ns;
        const double *re = nullptr, *im = nullptr;
        if (ok) R.parts(a.map, s, re, im);
        double2 u[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int j = tid + i * NT;
            double2 z = make_double2(0.0, 0.0);
            if (ok && j < k) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const double2 v = turn(make_double2(re[j + b * k], im ? im[j + b * k] : 0.0), b * t);
                    z.x += v.x;
                    z.y += v.y;
                }
                z = cmul(z, c.phase(j, t));
            }
            u[i] = z;
        }
        c.run(u, tid);
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int j = tid + i * NT;
            if (!ok || j >= k) continue;
            // phi_0 = pi / n: e^{-i m phi_0} changes sign from m to m + n
            const int at = 4 * j + t;
            double2 z = R.phased(cmul(u[i], post[i]), at, w);
            double2 y = at ? make_double2(-z.x, z.y) : make_double2(z.x, -z.y);
            for (int m = at; m <= a.mmax; m += n) {
                out(s, m)[0] = z;
                z = make_double2(-z.x, -z.y);
            }
            for (int m = at ? n - at : 0; m <= a.mmax; m += n) {
                out(s, m)[1] = y;
                y = make_double2(-y.x, -y.y);
            }
        }
    }
}

// The inverse: z_j = sum_m P_m e^{i m phi_j} + sum_{m > 0} conj(M_m) e^{-i m phi_j}
// (at m = 0 half of each), as conj DFT conj of the sums folded onto the ring, into
// the maps, or the reference maps less them.
template <int NT, int B, int G>
__global__ void __launch_bounds__(NT * G) ring_synth_kernel(ShtArgs a) {
    extern __shared__ double2 sh_ring[];
    const int N = a.nside, npairs = 2 * N, grp = threadIdx.x / NT, tid = threadIdx.x % NT;
    const int pair = pair_of_block(N);
    const RingPair R(N, pair);
    const int n = R.n, k = R.k;
    const int ns = R.signals(a.nfields);
    double2 *table = sh_ring, *data = sh_ring + N;
    // conj of the folded sum at index i of the ring
    auto folded = [&](int s, int i) {
        const double2 *F = a.F + ((size_t)s * (a.mmax + 1) * npairs + pair) * 2;
        // e^{i m phi_0} changes sign from m to m + n on the shifted rings: its value at i
        // (P_m e^{i m phi_0}) serves both sums
        const double turn_sign = R.shifted ? -1.0 : 1.0;
        double2 h = make_double2(0.0, 0.0);
        double w = i ? 1.0 : 0.5;
#pragma unroll 4
        for (int m = i; m <= a.mmax; m += n) {                        // conj(P_m)
            const double2 p = F[(size_t)m * npairs * 2];
            h.x = fma(w, p.x, h.x);
            h.y = fma(-w, p.y, h.y);
            w = m ? w * turn_sign : turn_sign;
        }
        w = i ? turn_sign : 0.5;
#pragma unroll 4
        for (int m = i ? n - i : 0; m <= a.mmax; m += n) {            // M_m
            const double2 p = F[(size_t)m * npairs * 2 + 1];
            h.x = fma(w, p.x, h.x);
            h.y = fma(w, p.y, h.y);
            w = m ? w * turn_sign : turn_sign;
        }
        h = R.phased(h, i, 1.0);
        return h;
    };
    auto put = [&](int s, int j, double2 z) {                         // z: conj of the signal
        double *re, *im;
        R.parts(a.map_out, s, re, im);
        if (a.residual) {
            const double *r0, *i0;
            R.parts(a.map, s, r0, i0);
            re[j] = r0[j] - z.x;
            if (im) im[j] = i0[j] + z.y;
        } else {
            re[j] = z.x;
            if (im) im[j] = -z.y;
        }
    };
    if (R.pow2) {
        LdsFft<NT, B> f;
        f.init(data + grp * 4 * N, table, 31 - __clz(n), tid);        // (groups past the signals: no data)
#pragma unroll 1
        for (int s0 = 0; s0 < ns; s0 += G) {
            const int s = s0 + grp;
            const bool ok = s < ns;
            if (ok)
                for (int i = tid; i < n; i += NT) f.x[i] = folded(s, i);
            if (ok || NT > 64) f.run();
            if (ok)
                for (int j = tid; j < n; j += NT) put(s, j, f.x[j]);
            __syncthreads();
        }
        return;
    }
    constexpr int SPB = G >= 12 ? 3 : 1;                              // signals side by side
    double2 *sums = data + 2 * N * G;                                 // [SPB][n]
    Chirp<NT, B> c;
    c.init(data + grp * 2 * N, table, k, tid);
    double2 post[B];
#pragma unroll
    for (int i = 0; i < B; ++i) post[i] = c.phase(min(tid + i * NT, k), 0);
#pragma unroll 1
    for (int s0 = 0; s0 < ns; s0 += SPB) {
        for (int i = threadIdx.x; i < min(SPB, ns - s0) * n; i += NT * G) sums[i] = folded(s0 + i / n, i % n);
        __syncthreads();
#pragma unroll 1
        for (int q0 = 0; q0 < 4 * SPB; q0 += G) {
            const int t = (q0 + grp) & 3, s = (q0 + grp) >> 2;        // samples 4 j + t of signal s0 + s
            const bool ok = s < SPB && s0 + s < ns;
            double2 u[B];
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int j = tid + i * NT;
                double2 z = make_double2(0.0, 0.0);
                if (ok && j < k) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const double2 v = turn(sums[s * n + j + b * k], b * t);
                        z.x += v.x;
                        z.y += v.y;
                    }
                    z = cmul(z, c.phase(j, t));
                }
                u[i] = z;
            }
            c.run(u, tid);
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int j = tid + i * NT;
                if (ok && j < k) put(s0 + s, 4 * j + t, cmul(u[i], post[i]));
            }
        }
        __syncthreads();
    }
}

// ----------------------------------------------------------------------
// The colatitude functions of one m, for the analysis and the synthesis.
//
// lambda_lm and the spin-2 functions f^+- = W_lm +- X_lm obey
//   A_l g_l = (z + s_l) g_{l-1} - A_{l-1} g_{l-2},
//   lambda: s_l = 0,                  A_l^2 = (l^2 - m^2) / (4 l^2 - 1),
//   f^+-:   s_l = +- 2m / (l (l-1)),  A_l^2 = (l^2 - m^2)(l^2 - 4) / (l^2 (4 l^2 - 1))
// (the standard recurrences of spin-weighted harmonics).  The mirror ring has
// lambda -> (-1)^(l+m) lambda and f^+- -> (-1)^(l+m) f^-+, so a north / south
// pair's three functions take nine instructions, and with
//   P = Q + iU, M = Q - iU (complex sums at each m, not conjugates):
//   S+ = sum f^+ P_N + (-1)^(l+m) f^- P_S,  S- = sum f^- M_N + (-1)^(l+m) f^+ M_S,
//   a^E = -(S+ + S-) / 2,  a^B = i (S+ - S-) / 2;
//   P = -sum (a^E + i a^B) f^+,  M = -sum (a^E - i a^B) f^-
// eight multiply-adds for E and B.  Forming W and X from lambda_l and
// lambda_{l-1} takes eight instructions where f^+- takes six, and loses digits
// to the 1 / s^2 terms next to the poles.  (Scaling the functions so that the
// last coefficient is 1 saves three more instructions, but the rounding of the
// first one then shifts z at every step, which next to the poles is ten times
// the plain recurrence's error.)
// ----------------------------------------------------------------------
struct Step {
    double aT, bT;       // 1 / A_l and A_{l-1} of lambda
    double aS, sS;       // 1 / A_l of f^+- and s_l of f^+
    double bS, abS;      // A_{l-1} and A_{l-1} / A_l of f^+-
};
static_assert(sizeof(Step) == SHT_STEP_BYTES, "size of the steps in the workspace");

// The steps of every (l, m), packed like the a_lm: written once per call, then
// read with scalar loads (a step is uniform over a workgroup), so that no vector
// register or LDS read is spent on them.  The first (l = m) gives g_l = -g_{l-2},
// see start_pair.
__global__ void __launch_bounds__(256) steps_kernel(ShtArgs a) {
    const int m = blockIdx.y, l = m + (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (l > a.lmax) return;
    const double dl = l, dm = m, d1 = dl - 1.0;
    const double p = (dl - dm) * (dl + dm), p1 = (d1 - dm) * (d1 + dm);       // l^2 - m^2, (l-1)^2 - m^2
    const double q = 4.0 * dl * dl - 1.0, q1 = 4.0 * d1 * d1 - 1.0;
    Step s{1.0, 1.0, 1.0, 0.0, 1.0, 1.0};
    if (l > m) {
        s.aT = sqrt(q / p);
        s.bT = sqrt(p1 / q1);
    }
    if (l > max(m, 2)) {
        const double u = (dl - 2.0) * (dl + 2.0), u1 = (d1 - 2.0) * (d1 + 2.0);
        s.aS = dl * sqrt(q / (p * u));
        s.bS = sqrt(p1 * u1 / q1) / d1;
        s.sS = 2.0 * dm / (dl * d1);
        s.abS = s.aS * s.bS;
    }
    static_cast<Step *>(a.steps)[(int64_t)m * (2 * a.lmax + 1 - m) / 2 + l] = s;
}

typedef const double __attribute__((address_space(4))) *uniform_ptr;
__device__ inline uniform_ptr steps_of(const ShtArgs &a, int64_t index) {
    return (uniform_ptr)(unsigned long long)(static_cast<const Step *>(a.steps) + index);
}
__device__ inline Step load_step(uniform_ptr p) { return Step{p[0], p[1], p[2], p[3], p[4], p[5]}; }

// Small maps have few waves to hide the scalar loads' misses behind (a step is a
// new cache line every 1.3 l, 480 clocks per l at nside 128): there a workgroup
// copies the steps (or the a_lm) of 64 l at a time into LDS, fetched while the
// 64 before are used.
template <int NT, int W>                 // W doubles per l
struct Staged {
    static constexpr int PER = (LCHUNK * W + NT - 1) / NT;
    double r[PER];
    // values first .. first + LCHUNK W of an array, as far as it has `count`
    __device__ inline void fetch(const double *src, int64_t first, int64_t count, int tid) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t at = first + i * NT + tid;
            r[i] = i * NT + tid < LCHUNK * W && at < count ? src[at] : 0.0;
        }
    }
    __device__ inline void put(double *dst, int tid) const {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i * NT + tid < LCHUNK * W) dst[i * NT + tid] = r[i];
    }
};

// A ring pair's functions before the step to l = m, in units of 2^(SCALE e).
struct PairState {
    double z;
    double v, vp, fp, fpp, fm, fmp;    // lambda, f^+ and f^-, each with its predecessor
    int e;
};

// Powers of two: the values' window is [2^-HALF, 2^HALF) at the start and after
// each rescaling, so a lane with e < 0 holds lambda below 2^-HALF and f^+- below 2^24
// times that (5e-32 of the O(1) values its ring reaches later): they add nothing in FP64.
constexpr int HALF = SCALE / 2;

// c s^m, split into a mantissa and a multiple of SCALE in the exponent
__device__ inline void power_start(double s, int m, double c, double *v, int *e) {
    int es;
    const double fs = frexp(s, &es);
    double base = fs, res = 1.0;
    long long be = 0, re = 0;
    for (int k = m; k; k >>= 1) {
        int t;
        if (k & 1) {
            res = frexp(res * base, &t);
            re += be + t;
        }
        base = frexp(base * base, &t);
        be = 2 * be + t;
    }
    const long long E = re + (long long)es * m;
    long long q = (E + HALF) / SCALE;
    if (q * SCALE > E + HALF) --q;                // floor
    *e = (int)q;
    *v = c * ldexp(res, (int)(E - q * SCALE));
}

// Start values, placed so that the first step (g_l = -g_{l-2}) brings them up at l = m:
//   lambda_mm = (-1)^m c_m s^m,
//   f^+-_mm = sqrt(m (m-1) / ((m+1)(m+2))) lambda_mm ((1 -+ z) / (1 +- z))  (m >= 2).
// North ring or equator: z >= 0 and 1 - z = omz, exact next to the pole.
__device__ inline PairState start_pair(const RingGeom &g, int m, double cm, bool ok) {
    PairState p;
    p.z = g.z;
    double v;
    power_start(g.s, m, (m & 1) ? -cm : cm, &v, &p.e);
    if (!ok) {                                     // a lane without a ring: zero, and never rescaled
        p.e = -1;
        v = 0.0;
    }
    p.v = p.fp = p.fm = 0.0;
    p.vp = -v;
    const double c = m >= 2 ? sqrt((double)m * (m - 1.0) / ((m + 1.0) * (m + 2.0))) : 0.0, opz = 1.0 + g.z;
    p.fpp = -c * v * (g.omz / opz);
    p.fmp = -c * v * (opz / g.omz);
    return p;
}

// One step.  POLAR: f^+- by a ((z +- s) f - b f_prev), one instruction more each:
// next to a pole the roundings of (z +- s) a count (it differs from 2 by the order
// of theta^2).
template <bool POL, bool POLAR>
__device__ inline void advance(PairState &p, const Step &c) {
    const double vn = c.aT * fma(p.z, p.v, -c.bT * p.vp);
    p.vp = p.v;
    p.v = vn;
    if (POL) {
        double pn, mn;
        if (POLAR) {
            pn = c.aS * fma(p.z + c.sS, p.fp, -c.bS * p.fpp);
            mn = c.aS * fma(p.z - c.sS, p.fm, -c.bS * p.fmp);
        } else {
            const double as = c.aS * c.sS;
            pn = fma(fma(c.aS, p.z, as), p.fp, -c.abS * p.fpp);
            mn = fma(fma(c.aS, p.z, -as), p.fm, -c.abS * p.fmp);
        }
        p.fpp = p.fp;
        p.fmp = p.fm;
        p.fp = pn;
        p.fm = mn;
    }
}

// After up to eight steps of a lane with e < 0 (a step grows by less than 2^16, and
// f differs from lambda by less than 2^24, so nothing overflows in between).
template <bool POL>
__device__ inline void rescale(PairState &p) {
    if (fabs(p.v) > 0x1p128) {
        p.v *= 0x1p-256;
        p.vp *= 0x1p-256;
        if (POL) {
            p.fp *= 0x1p-256;
            p.fpp *= 0x1p-256;
            p.fm *= 0x1p-256;
            p.fmp *= 0x1p-256;
        }
        p.e += 1;
    }
}

// c_m = sqrt((4 pi)^-1 prod_{k=1..m} (2k + 1) / (2k)): partial products per lane, then across the wave
__device__ inline double start_norm(int m, int lane) {
    double pr = 1.0;
    for (int k = lane + 1; k <= m; k += 64) pr *= (2.0 * k + 1.0) / (2.0 * k);
    for (int o = 32; o; o >>= 1) pr *= __shfl_xor(pr, o, 64);
    return sqrt(pr / (4.0 * M_PI));
}

// An a_lm value into place, or added to it (the refinement steps' corrections).
__device__ inline void put_alm(const ShtArgs &a, double *dst, double re, double im) {
    if (a.add) {
        re += dst[0];
        im += dst[1];
    }
    dst[0] = re;
    dst[1] = im;
}

// Ring sums of one pair: T north +- south, and P, M of each hemisphere.
struct PairSums {
    double2 Tp, Tm, Pn, Ps, Mn, Ms;
};

template <bool POL>
__device__ inline PairSums load_pair(const ShtArgs &a, int m, int pair, bool ok) {
    const int npairs = 2 * a.nside;
    const bool south = ok && pair != npairs - 1;                      // the equator is its own mirror
    const double2 zero = make_double2(0.0, 0.0);
    auto at = [&](int s) { return a.F + (((size_t)s * (a.mmax + 1) + m) * npairs + pair) * 2; };
    PairSums f;
    const double2 P = ok ? at(0)[0] : zero, M = ok ? at(0)[1] : zero;
    // T_N = (P + M) / 2, T_S = (P - M) / 2i
    const double2 n = make_double2(0.5 * (P.x + M.x), 0.5 * (P.y + M.y));
    const double2 t = south ? make_double2(0.5 * (P.y - M.y), -0.5 * (P.x - M.x)) : zero;
    f.Tp = make_double2(n.x + t.x, n.y + t.y);
    f.Tm = make_double2(n.x - t.x, n.y - t.y);
    f.Pn = f.Mn = f.Ps = f.Ms = zero;
    if (POL) {
        if (ok) {
            f.Pn = at(1)[0];
            f.Mn = at(1)[1];
        }
        if (south) {
            f.Ps = at(2)[0];
            f.Ms = at(2)[1];
        }
    }
    return f;
}

// lambda and f of one l (parity ODD of l - m) against the pair's sums: acc = (T, S+, S-)
template <bool ODD, bool POL>
__device__ inline void pair_terms(const PairState &p, const PairSums &f, double *acc) {
    const double2 FT = ODD ? f.Tm : f.Tp;
    acc[0] = fma(p.v, FT.x, acc[0]);
    acc[1] = fma(p.v, FT.y, acc[1]);
    if (POL) {
        const double sp = ODD ? -p.fp : p.fp, sm = ODD ? -p.fm : p.fm;
        acc[2] = fma(sm, f.Ps.x, fma(p.fp, f.Pn.x, acc[2]));
        acc[3] = fma(sm, f.Ps.y, fma(p.fp, f.Pn.y, acc[3]));
        acc[4] = fma(sp, f.Ms.x, fma(p.fm, f.Mn.x, acc[4]));
        acc[5] = fma(sp, f.Ms.y, fma(p.fm, f.Mn.y, acc[5]));
    }
}

// LB steps of one pair, its terms added to acc[l][comp].
template <bool POL, bool POLAR, int LB>
__device__ inline void block_terms(PairState &p, const PairSums &f, const Step *st, double *acc) {
    constexpr int NC = POL ? NCOMP : 2;
    if (p.e >= 0) {
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            advance<POL, POLAR>(p, st[j]);
            if (j & 1) pair_terms<true, POL>(p, f, acc + j * NC);
            else pair_terms<false, POL>(p, f, acc + j * NC);
        }
    } else {
#pragma unroll
        for (int j = 0; j < LB; ++j) advance<POL, POLAR>(p, st[j]);
        rescale<POL>(p);
    }
}

// x and y of the lanes' halves exchanged and added: x over the first half's
// place, y over the second's (32: halves of the wave; 16: rows of each half)
template <int ROW>
__device__ inline double swap_add(double x, double y) {
    const unsigned long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
    uint32_t xl = (uint32_t)bx, xh = (uint32_t)(bx >> 32), yl = (uint32_t)by, yh = (uint32_t)(by >> 32);
    if constexpr (ROW == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
        xl = l[0], yl = l[1], xh = h[0], yh = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
        xl = l[0], yl = l[1], xh = h[0], yh = h[1];
    }
    return __longlong_as_double(((unsigned long long)xh << 32) | xl) +
           __longlong_as_double(((unsigned long long)yh << 32) | yl);
}

// LDS of the analysis: the waves' sums of two chunks, then per wave the 16
// partial sums of each of a block's sums (rows of 17)
template <bool POL>
constexpr int alm_comps() { return POL ? NCOMP : 2; }
template <bool POL, int NW, int LB>
constexpr size_t alm_lds() {
    return (2 * LCHUNK * alm_comps<POL>() + LB * alm_comps<POL>() * 17) * NW * sizeof(double);
}

// The wave's sums of NS values over its lanes: 64 lanes to 16 by exchanges (row i
// of a set of four then holds value 0, 2, 1, 3) into LDS, the rest from there, in a
// fixed order.  The second half is left to the next block: its LDS reads are
// issued before that block's arithmetic and added after it.
template <int NS>
struct WaveSums {
    static constexpr int PARTS = NS > 32 ? 1 : 64 / NS >= 8 ? 8 : 64 / NS >= 4 ? 4 : 2;   // lanes that share one sum
    static_assert(NS % 4 == 0 && NS * PARTS <= 64, "one sum a lane group");
    double q[16 / PARTS];
    double *dst;            // where the values in LDS belong; null: none
    __device__ inline void push(const double *acc, double *red, int lane, double *to) {
        double h[NS / 2];
#pragma unroll
        for (int t = 0; t < NS / 2; ++t) h[t] = swap_add<32>(acc[2 * t], acc[2 * t + 1]);
#pragma unroll
        for (int t = 0; t < NS / 4; ++t)
            red[(4 * t + (lane >> 4)) * 17 + (lane & 15)] = swap_add<16>(h[2 * t], h[2 * t + 1]);
        wave_sync();
        dst = to;
    }
    __device__ inline void load(const double *red, int lane) {
        const int o = min(lane / PARTS, NS - 1), part = lane % PARTS;
        const double *p = red + ((o & ~3) + ((o & 1) << 1 | (o >> 1 & 1))) * 17 + part;
#pragma unroll
        for (int u = 0; u < 16 / PARTS; ++u) q[u] = p[u * PARTS];
    }
    __device__ inline void store(int lane) {
#pragma unroll
        for (int w = 8 / PARTS; w; w >>= 1)
#pragma unroll
            for (int u = 0; u < w; ++u) q[u] += q[u + w];
        double sum = q[0];
#pragma unroll
        for (int x = 1; x < PARTS; x <<= 1) sum += __shfl_xor(sum, x, 64);
        if (lane % PARTS == 0 && lane / PARTS < NS) dst[lane / PARTS] = sum;
        wave_sync();
    }
};

// ----------------------------------------------------------------------
// The polarised analysis of the first m forms W and X from lambda_l and
// lambda_{l-1}: m < 2, whose f^+- start at l = 2, and on large maps m < WX_M.  A
// pixel's z, rounded to a double, and its sin(theta) do not belong to one angle,
// and next to the poles that moves this evaluation and the one by f^+- apart: by
// 5e-12 of the largest a_lm at m = 0, 1e-12 at m = 3 and 3e-13 at m = 17 at nside
// 1024 (f^+- is the nearer to the exact harmonics: 2e-12 against 1e-11 at m = 0),
// 5e-13 at nside 256.  These few a_lm keep the definition's own evaluation, so that they
// do not move by that.  They are the longest chains of l, so a workgroup takes one m and 64 NW
// ring pairs, one a lane; with more parts than one, wx_reduce_kernel adds them.
// ----------------------------------------------------------------------
constexpr int WX_M = 16, WX_NSIDE = 256;

struct WxStep {
    double ra, rb;           // lambda_l = ra (z lambda_{l-1} - rb lambda_{l-2})
    double A, B, C, D;       // W = -(A / s^2 + B) lambda_l + C (z / s^2) lambda_{l-1}; X = (m / s^2)(C lambda_{l-1} - D z lambda_l)
};

__device__ inline WxStep wx_step(int l, int m) {
    WxStep c{1.0, 1.0, 0.0, 0.0, 0.0, 0.0};
    const double dl = l, dm = m;
    if (l > m) {
        c.ra = sqrt((4.0 * dl * dl - 1.0) / (dl * dl - dm * dm));
        c.rb = sqrt(((dl - 1.0) * (dl - 1.0) - dm * dm) / (4.0 * (dl - 1.0) * (dl - 1.0) - 1.0));
    }
    if (l >= 2) {
        const double nl = 2.0 / sqrt((dl - 1.0) * dl * (dl + 1.0) * (dl + 2.0));
        const double clm = l > m ? sqrt((2.0 * dl + 1.0) * (dl - dm) / ((2.0 * dl - 1.0) * (dl + dm))) : 0.0;
        c.A = nl * (dl - dm * dm);
        c.B = nl * dl * (dl - 1.0) * 0.5;
        c.C = nl * (dl + dm) * clm;
        c.D = nl * (dl - 1.0);
    }
    return c;
}

// LDS: as alm_kernel's, then two chunks of steps
template <int NW, int LB>
__device__ void alm_wx(const ShtArgs &a, int m, int part, int tid, double *lds) {
    constexpr int NS = LB * NCOMP, NT = 64 * NW;
    const int lane = tid & 63, wave = tid >> 6;
    double *red = lds + 2 * NW * LCHUNK * NCOMP + wave * NS * 17;
    WxStep *steps = reinterpret_cast<WxStep *>(lds + (2 * LCHUNK * NCOMP + NS * 17) * NW);
    const int npairs = 2 * a.nside, pi = part * NT + tid;
    const bool ok = pi < npairs;
    const int rn = ok ? pi : 0;
    const PairSums F = load_pair<true>(a, m, rn, ok);
    double2 P[3], M[3];                                               // T, Q, U: north +- south
    {
        const double2 qn = make_double2(0.5 * (F.Pn.x + F.Mn.x), 0.5 * (F.Pn.y + F.Mn.y));
        const double2 qs = make_double2(0.5 * (F.Ps.x + F.Ms.x), 0.5 * (F.Ps.y + F.Ms.y));
        const double2 un = make_double2(0.5 * (F.Pn.y - F.Mn.y), -0.5 * (F.Pn.x - F.Mn.x));
        const double2 us = make_double2(0.5 * (F.Ps.y - F.Ms.y), -0.5 * (F.Ps.x - F.Ms.x));
        P[0] = F.Tp;
        M[0] = F.Tm;
        P[1] = make_double2(qn.x + qs.x, qn.y + qs.y);
        M[1] = make_double2(qn.x - qs.x, qn.y - qs.y);
        P[2] = make_double2(un.x + us.x, un.y + us.y);
        M[2] = make_double2(un.x - us.x, un.y - us.y);
    }
    const RingGeom g = sht_ring(a.nside, rn);
    PairState p = start_pair(g, m, start_norm(m, lane), ok);
    const double inv_s2 = 1.0 / (g.s * g.s), z_s2 = g.z * inv_s2, m_s2 = (double)m * inv_s2;

    const int nl = a.lmax - m + 1;
    const int64_t base = (int64_t)m * (2 * a.lmax + 1 - m) / 2 + m, nalm = (int64_t)(a.lmax + 1) * (a.lmax + 2) / 2;
    if (wave == 0) steps[lane] = wx_step(m + lane, m);
    __syncthreads();
    WaveSums<NS> ws;
    for (int c0 = 0, ch = 0; c0 < nl; c0 += LCHUNK, ++ch) {
        if (wave == (ch + 1) % NW) steps[((ch + 1) & 1) * LCHUNK + lane] = wx_step(m + c0 + LCHUNK + lane, m);
        const int cend = min(nl - c0, LCHUNK);
        for (int b0 = 0; b0 < cend; b0 += LB) {
            double acc[NS];
            if (b0) ws.load(red, lane);
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                const WxStep c = steps[(ch & 1) * LCHUNK + b0 + j];
                const double vn = c.ra * fma(p.z, p.v, -c.rb * p.vp);
                p.vp = p.v;
                p.v = vn;
                const double on = p.e >= 0 ? 1.0 : 0.0;
                const double L = on * p.v, Lp = on * p.vp;
                const double W = fma(-fma(c.A, inv_s2, c.B), L, c.C * z_s2 * Lp);
                const double X = m_s2 * fma(c.C, Lp, -c.D * g.z * L);
                const double2 T = (j & 1) ? M[0] : P[0], Qa = (j & 1) ? M[1] : P[1], Ua = (j & 1) ? M[2] : P[2];
                const double2 Qb = (j & 1) ? P[1] : M[1], Ub = (j & 1) ? P[2] : M[2];
                double *x = acc + j * NCOMP;
                x[0] = L * T.x;
                x[1] = L * T.y;
                x[2] = fma(-X, Ub.y, W * Qa.x);
                x[3] = fma(X, Ub.x, W * Qa.y);
                x[4] = fma(X, Qb.y, W * Ua.x);
                x[5] = fma(-X, Qb.x, W * Ua.y);
            }
            if (p.e < 0) rescale<false>(p);
            if (b0) ws.store(lane);
            ws.push(acc, red, lane, lds + (((ch & 1) * NW + wave) * LCHUNK + b0) * NCOMP);
        }
        ws.load(red, lane);
        ws.store(lane);
        __syncthreads();
        const double *all = lds + (ch & 1) * NW * LCHUNK * NCOMP;
        if (a.wx_parts > 1) {
            for (int i = tid; i < cend * NCOMP; i += NT) {
                double x = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) x += all[w * LCHUNK * NCOMP + i];
                a.partial[((int64_t)part * nalm + base + c0) * NCOMP + i] = x;
            }
        } else {
            for (int i = tid; i < cend * 3; i += NT) {
                const int c = i % 3, li = i / 3;
                double re = 0.0, im = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    re += all[(w * LCHUNK + li) * NCOMP + 2 * c];
                    im += all[(w * LCHUNK + li) * NCOMP + 2 * c + 1];
                }
                put_alm(a, a.alm[c] + 2 * (base + c0 + li), c ? -re : re, c ? -im : im);
            }
        }
    }
}

// One workgroup of NW waves per m, K ring pairs a lane (64 K NW >= 2 nside).
// Bound by FP64 issue: 19 instructions per (l, pair) and, per LB l and wave,
// the 6 LB cross-lane sums (at LB = 4: 36 lane exchanges and 18 adds, then 6 writes
// and 8 reads of LDS).  A pair whose values are still negligible (e < 0) only steps.
// The waves' sums meet in LDS once per 64 l, in a fixed order.  The first band of
// pairs takes the polar form (all of them with one pair a lane).  At nside 1024,
// lmax 3071: 8.6 ms, 25 vector instructions per (l, band of 64 pairs), the vector
// ALU issuing 80% of the time; 16.5 ms and 43 when W and X were formed from
// lambda, most values carried an exponent, and each (l, pair) had branches of its
// own.  Small maps: see launch_alm_t.
template <bool POL, int K, int NW, int LB>
__global__ void __launch_bounds__(64 * NW, K >= 4 ? 2 : 1) alm_kernel(ShtArgs a) {
    constexpr int NC = alm_comps<POL>(), NS = LB * NC, NT = 64 * NW;
    constexpr bool STAGE = K == 1;
    extern __shared__ double sh_alm[];                               // [2][NW][LCHUNK][NC], [NW][NS * 17], 2 chunks of steps
    const int N = a.nside, lmax = a.lmax;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wx = a.wx_m * a.wx_parts;
    if (POL && (int)blockIdx.x < wx) {
        alm_wx<NW, LB>(a, blockIdx.x / a.wx_parts, blockIdx.x % a.wx_parts, tid, sh_alm);
        return;
    }
    const int m = a.wx_m + (int)blockIdx.x - wx;
    double *red = sh_alm + 2 * NW * LCHUNK * NC + wave * NS * 17;
    const int npairs = 2 * N;
    const double cm = start_norm(m, lane);

    PairState ps[K];
    PairSums f[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int pi = tid + k * NT;
        const bool ok = pi < npairs;
        const int rn = ok ? pi : 0;
        f[k] = load_pair<POL>(a, m, rn, ok);
        ps[k] = start_pair(sht_ring(N, rn), m, cm, ok);
    }

    const int nl = lmax - m + 1;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2 + m;     // index of l = m
    constexpr int SD = sizeof(Step) / sizeof(double);
    const int64_t nsteps = (int64_t)(lmax + 1) * (lmax + 2) / 2 * SD;
    const double *steps = static_cast<const double *>(a.steps);
    double *staged = sh_alm + (2 * LCHUNK * NC + NS * 17) * NW;
    Staged<NT, SD> sg;
    Step s[LB];                                                   // steps past lmax: not used (see the workspace)
    if constexpr (STAGE) {
        sg.fetch(steps, base * SD, nsteps, tid);
        sg.put(staged, tid);
        __syncthreads();
    } else {
#pragma unroll
        for (int j = 0; j < LB; ++j) s[j] = load_step(steps_of(a, base + j));
    }
    WaveSums<NS> ws;
    for (int c0 = 0, ch = 0; c0 < nl; c0 += LCHUNK, ++ch) {
        const Step *st = reinterpret_cast<const Step *>(staged) + (ch & 1) * LCHUNK;
        if constexpr (STAGE) sg.fetch(steps, (base + c0 + LCHUNK) * SD, nsteps, tid);
        double *mine = sh_alm + ((ch & 1) * NW + wave) * LCHUNK * NC;
        const int cend = min(nl - c0, LCHUNK);
        for (int b0 = 0; b0 < cend; b0 += LB) {
            double acc[NS];
#pragma unroll
            for (int t = 0; t < NS; ++t) acc[t] = 0.0;
            if (b0) ws.load(red, lane);
            if constexpr (STAGE) {
#pragma unroll
                for (int j = 0; j < LB; ++j) s[j] = st[b0 + j];
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k == 0) block_terms<POL, true, LB>(ps[k], f[k], s, acc);
                else block_terms<POL, false, LB>(ps[k], f[k], s, acc);
            }
            if constexpr (!STAGE) {
                // the next block's steps, in flight during the sums
#pragma unroll
                for (int j = 0; j < LB; ++j) s[j] = load_step(steps_of(a, base + c0 + b0 + LB + j));
            }
            if (b0) ws.store(lane);
            ws.push(acc, red, lane, mine + b0 * NC);
        }
        ws.load(red, lane);
        ws.store(lane);
        if constexpr (STAGE) sg.put(staged + ((ch + 1) & 1) * LCHUNK * SD, tid);
        __syncthreads();
        // a_lm of the chunk: the waves' sums in order, and a^E, a^B from S+, S-
        const double *all = sh_alm + (ch & 1) * NW * LCHUNK * NC;
        for (int i = tid; i < cend * (POL ? 2 : 1); i += NT) {
            const int li = POL ? i >> 1 : i;
            const bool spin = POL && (i & 1);
            double x[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const double *q = all + (w * LCHUNK + li) * NC + (spin ? 2 : 0);
                x[0] += q[0];
                x[1] += q[1];
                if (spin) {
                    x[2] += q[2];
                    x[3] += q[3];
                }
            }
            const int64_t idx = 2 * (base + c0 + li);
            if (!spin) {
                put_alm(a, a.alm[0] + idx, x[0], x[1]);
            } else {
                put_alm(a, a.alm[1] + idx, -0.5 * (x[0] + x[2]), -0.5 * (x[1] + x[3]));
                put_alm(a, a.alm[2] + idx, -0.5 * (x[1] - x[3]), 0.5 * (x[0] - x[2]));
            }
        }
    }
}

// a_lm of the first m: the parts' sums (T, -E, -B) in order.
__global__ void __launch_bounds__(256) wx_reduce_kernel(ShtArgs a, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count * 3) return;
    const int64_t nalm = (int64_t)(a.lmax + 1) * (a.lmax + 2) / 2;
    const int c = (int)(i % 3);
    double re = 0.0, im = 0.0;
    for (int q = 0; q < a.wx_parts; ++q) {
        const double *x = a.partial + ((int64_t)q * nalm + i / 3) * NCOMP + 2 * c;
        re += x[0];
        im += x[1];
    }
    put_alm(a, a.alm[c] + 2 * (i / 3), c ? -re : re, c ? -im : im);
}

// ----------------------------------------------------------------------
// Synthesis: the sums over l of each ring pair, G_m = sum_l a_lm lambda_lm and
// P_m, M_m (see above), in the lane's registers: no cross-lane sums.
// ----------------------------------------------------------------------
// The a_lm of one l (uniform over the workgroup: scalar loads), T then E, B.
typedef const double __attribute__((address_space(4))) *uniform_alm;
template <bool POL>
struct SynAlm {
    double t[2], e[2], b[2];
    __device__ inline void load(const ShtArgs &a, int64_t i) {
        const uniform_alm T = (uniform_alm)(unsigned long long)(a.alm_in[0] + 2 * i);
        t[0] = T[0];
        t[1] = T[1];
        if (POL) {
            const uniform_alm E = (uniform_alm)(unsigned long long)(a.alm_in[1] + 2 * i);
            const uniform_alm B = (uniform_alm)(unsigned long long)(a.alm_in[2] + 2 * i);
            e[0] = E[0];
            e[1] = E[1];
            b[0] = B[0];
            b[1] = B[1];
        }
    }
};

// Sums of one pair: T split by the parity of l - m (the south takes the odd ones
// with a minus sign), and -P, -M of each hemisphere.
struct SynSums {
    double2 Te, To, Pn, Ps, Mn, Ms;
};

template <bool POL, bool POLAR, int LB>
__device__ inline void syn_block(PairState &p, SynSums &f, const Step *st, const SynAlm<POL> *al) {
    if (p.e >= 0) {
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            advance<POL, POLAR>(p, st[j]);
            double2 &T = (j & 1) ? f.To : f.Te;
            T.x = fma(p.v, al[j].t[0], T.x);
            T.y = fma(p.v, al[j].t[1], T.y);
            if (POL) {
                // a^E + i a^B with f^+, a^E - i a^B with f^-; the south's exchanged, times (-1)^(l+m)
                const double px = al[j].e[0] - al[j].b[1], py = al[j].e[1] + al[j].b[0];
                const double mx = al[j].e[0] + al[j].b[1], my = al[j].e[1] - al[j].b[0];
                const double sp = (j & 1) ? -p.fp : p.fp, sm = (j & 1) ? -p.fm : p.fm;
                f.Pn.x = fma(p.fp, px, f.Pn.x);
                f.Pn.y = fma(p.fp, py, f.Pn.y);
                f.Ps.x = fma(sm, px, f.Ps.x);
                f.Ps.y = fma(sm, py, f.Ps.y);
                f.Mn.x = fma(p.fm, mx, f.Mn.x);
                f.Mn.y = fma(p.fm, my, f.Mn.y);
                f.Ms.x = fma(sp, mx, f.Ms.x);
                f.Ms.y = fma(sp, my, f.Ms.y);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < LB; ++j) advance<POL, POLAR>(p, st[j]);
        rescale<POL>(p);
    }
}

// One l of either parity, for the ends of the loop.
template <bool POL>
__device__ inline void syn_one(PairState &p, SynSums &f, const Step &st, const SynAlm<POL> &al, bool odd) {
    advance<POL, true>(p, st);
    if (p.e < 0) {
        rescale<POL>(p);
        return;
    }
    const double s = odd ? -1.0 : 1.0;
    // (values are selected, not a reference to one of the sums: that would keep the
    // lane's sums in scratch memory, read and written at every l of the main loop too)
    const double x = fma(p.v, al.t[0], odd ? f.To.x : f.Te.x), y = fma(p.v, al.t[1], odd ? f.To.y : f.Te.y);
    f.Te = make_double2(odd ? f.Te.x : x, odd ? f.Te.y : y);
    f.To = make_double2(odd ? x : f.To.x, odd ? y : f.To.y);
    if (POL) {
        const double px = al.e[0] - al.b[1], py = al.e[1] + al.b[0], mx = al.e[0] + al.b[1], my = al.e[1] - al.b[0];
        f.Pn.x = fma(p.fp, px, f.Pn.x);
        f.Pn.y = fma(p.fp, py, f.Pn.y);
        f.Ps.x = fma(s * p.fm, px, f.Ps.x);
        f.Ps.y = fma(s * p.fm, py, f.Ps.y);
        f.Mn.x = fma(p.fm, mx, f.Mn.x);
        f.Mn.y = fma(p.fm, my, f.Mn.y);
        f.Ms.x = fma(s * p.fp, mx, f.Ms.x);
        f.Ms.y = fma(s * p.fp, my, f.Ms.y);
    }
}

// m < 2: f^+- start at l = 2, so that the step there (which gives -f_prev) yields
//   f^+-_21 = -+ sqrt(5 / 16 pi) s (1 -+ z),  f^+-_20 = sqrt(15 / 32 pi) s^2;
// none below.
__device__ inline void late_start(PairState &p, const RingGeom &g, int m) {
    const double c = m ? sqrt(5.0 / (16.0 * M_PI)) : sqrt(15.0 / (32.0 * M_PI));
    p.fp = p.fm = 0.0;
    p.fpp = m ? c * g.s * g.omz : -c * g.s * g.s;
    p.fmp = m ? -c * g.s * (1.0 + g.z) : -c * g.s * g.s;
}

// One workgroup of NW waves per m, K ring pairs a lane, LB l a step of the loop.
// Bound by FP64 issue: 19 instructions per (l, pair); at nside 128, lmax 383 by the
// chain of l (1.5 waves a SIMD): 42 us, 114 with W and X in 768-lane workgroups.  A
// whole polarised synthesis at nside 1024, lmax 3071: 11.2 ms, 18.3 with W and X and
// the directly summed ring DFTs (193 registers; no scratch memory, see syn_one).
template <bool POL, int K, int NW, int LB>
__global__ void __launch_bounds__(64 * NW, K >= 4 ? 2 : 1) alm2ring_kernel(ShtArgs a) {
    constexpr int NT = 64 * NW;
    const int m = blockIdx.x;
    const int N = a.nside, lmax = a.lmax;
    const int tid = threadIdx.x, lane = tid & 63;
    const int npairs = 2 * N;
    const double cm = start_norm(m, lane);
    PairState ps[K];
    SynSums f[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int pi = tid + k * NT;
        const bool ok = pi < npairs;
        ps[k] = start_pair(sht_ring(N, ok ? pi : 0), m, cm, ok);
        f[k].Te = f[k].To = f[k].Pn = f[k].Ps = f[k].Mn = f[k].Ms = make_double2(0.0, 0.0);
    }
    const int nl = lmax - m + 1;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2 + m;     // index of l = m
    int li = 0;                                                       // l - m
    if (POL && m < 2) {
        // up to l = 3, one by one
        for (; li <= 3 - m && li < nl; ++li) {
            const Step s = load_step(steps_of(a, base + li));
            SynAlm<POL> al;
            al.load(a, base + li);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int pi = tid + k * NT;
                if (m + li < 2) ps[k].fp = ps[k].fm = ps[k].fpp = ps[k].fmp = 0.0;
                if (m + li == 2 && pi < npairs) late_start(ps[k], sht_ring(N, pi), m);
                syn_one<POL>(ps[k], f[k], s, al, li & 1);
            }
        }
        if ((li & 1) && li < nl) {                                    // to an even l - m
            const Step s = load_step(steps_of(a, base + li));
            SynAlm<POL> al;
            al.load(a, base + li);
#pragma unroll
            for (int k = 0; k < K; ++k) syn_one<POL>(ps[k], f[k], s, al, true);
            ++li;
        }
    }
    if constexpr (K == 1) {
        // 64 l at a time from LDS
        constexpr int SD = sizeof(Step) / sizeof(double);
        __shared__ double st[2][LCHUNK * SD], al[POL ? 3 : 1][2][LCHUNK * 2];
        const int64_t nalm = (int64_t)(lmax + 1) * (lmax + 2) / 2;
        Staged<NT, SD> gs;
        Staged<NT, 2> ga[POL ? 3 : 1];
        auto fetch = [&](int from) {
            gs.fetch(static_cast<const double *>(a.steps), (base + from) * SD, nalm * SD, tid);
#pragma unroll
            for (int c = 0; c < (POL ? 3 : 1); ++c) ga[c].fetch(a.alm_in[c], (base + from) * 2, nalm * 2, tid);
        };
        auto put = [&](int to) {
            gs.put(st[to], tid);
#pragma unroll
            for (int c = 0; c < (POL ? 3 : 1); ++c) ga[c].put(al[c][to], tid);
        };
        fetch(li);
        put(0);
        __syncthreads();
        for (int ch = 0; li < nl; ++ch) {
            const int end = min(li + LCHUNK, nl), c0 = li;
            fetch(c0 + LCHUNK);
            auto at = [&](int i, Step &s, SynAlm<POL> &x) {
                s = reinterpret_cast<const Step *>(st[ch & 1])[i];
                x.t[0] = al[0][ch & 1][2 * i];
                x.t[1] = al[0][ch & 1][2 * i + 1];
                if constexpr (POL) {
                    x.e[0] = al[1][ch & 1][2 * i];
                    x.e[1] = al[1][ch & 1][2 * i + 1];
                    x.b[0] = al[2][ch & 1][2 * i];
                    x.b[1] = al[2][ch & 1][2 * i + 1];
                }
            };
            for (; li + LB <= end; li += LB) {
                Step s[LB];
                SynAlm<POL> x[LB];
#pragma unroll
                for (int j = 0; j < LB; ++j) at(li - c0 + j, s[j], x[j]);
                syn_block<POL, true, LB>(ps[0], f[0], s, x);
            }
            for (; li < end; ++li) {                                  // only at lmax: a chunk holds whole blocks
                Step s;
                SynAlm<POL> x;
                at(li - c0, s, x);
                syn_one<POL>(ps[0], f[0], s, x, li & 1);
            }
            put((ch + 1) & 1);
            __syncthreads();
        }
    } else if (li + LB <= nl) {
        Step s[LB];
        SynAlm<POL> al[LB];
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            s[j] = load_step(steps_of(a, base + li + j));
            al[j].load(a, base + li + j);
        }
        for (; li + LB <= nl; li += LB) {
            // the next block's steps and a_lm, in flight during this one (the last block's: again its own)
            const int64_t next = base + (li + 2 * LB <= nl ? li + LB : li);
            Step sn[LB];
            SynAlm<POL> an[LB];
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                sn[j] = load_step(steps_of(a, next + j));
                an[j].load(a, next + j);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k == 0) syn_block<POL, true, LB>(ps[k], f[k], s, al);
                else syn_block<POL, false, LB>(ps[k], f[k], s, al);
            }
#pragma unroll
            for (int j = 0; j < LB; ++j) {
                s[j] = sn[j];
                al[j] = an[j];
            }
        }
    }
    for (; li < nl; ++li) {
        const Step s = load_step(steps_of(a, base + li));
        SynAlm<POL> al;
        al.load(a, base + li);
#pragma unroll
        for (int k = 0; k < K; ++k) syn_one<POL>(ps[k], f[k], s, al, li & 1);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int pi = tid + k * NT;
        if (pi >= npairs) continue;
        const SynSums &x = f[k];
        auto at = [&](int s) { return a.F + (((size_t)s * (a.mmax + 1) + m) * npairs + pi) * 2; };
        // T_N +- i T_S
        const double2 n = make_double2(x.Te.x + x.To.x, x.Te.y + x.To.y), t = make_double2(x.Te.x - x.To.x, x.Te.y - x.To.y);
        at(0)[0] = make_double2(n.x - t.y, n.y + t.x);
        at(0)[1] = make_double2(n.x + t.y, n.y - t.x);
        if (POL) {
            at(1)[0] = make_double2(-x.Pn.x, -x.Pn.y);
            at(1)[1] = make_double2(-x.Mn.x, -x.Mn.y);
            at(2)[0] = make_double2(-x.Ps.x, -x.Ps.y);
            at(2)[1] = make_double2(-x.Ms.x, -x.Ms.y);
        }
    }
}

// C_l: a workgroup takes CL_L consecutive l, half a wave of lanes over them (an
// a_lm column is contiguous in l) and the 2 CL_WAVES half waves over m, then adds the
// halves in a fixed order.  Reads each a_lm once for all the spectra (TEB: T, E, B
// and their six pairs; else one pair).  Bound by the reads: lmax 3071, 0.10 ms for 226
// MB; 0.73 with a wave per l, whose lanes over m read a line each, six times over.
constexpr int CL_L = 32, CL_WAVES = 16;
template <bool TEB>
__global__ void __launch_bounds__(64 * CL_WAVES) alm2cl_kernel(ClArgs a) {
    constexpr int NX = TEB ? 6 : 1, HALVES = 2 * CL_WAVES;
    __shared__ double part[NX][HALVES][CL_L];
    const int li = threadIdx.x % CL_L, half = threadIdx.x / CL_L;
    const int l = blockIdx.x * CL_L + li;
    double acc[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) acc[t] = 0.0;
    if (l <= a.lmax) {
        for (int m = half; m <= l; m += HALVES) {
            const int64_t i = (int64_t)m * (2 * a.lmax + 1 - m) / 2 + l;
            const double w = m == 0 ? 1.0 : 2.0;
            if constexpr (TEB) {
                const double2 T = reinterpret_cast<const double2 *>(a.x[0])[i];
                const double2 E = reinterpret_cast<const double2 *>(a.x[1])[i];
                const double2 B = reinterpret_cast<const double2 *>(a.x[2])[i];
                acc[0] = fma(w, fma(T.x, T.x, T.y * T.y), acc[0]);
                acc[1] = fma(w, fma(E.x, E.x, E.y * E.y), acc[1]);
                acc[2] = fma(w, fma(B.x, B.x, B.y * B.y), acc[2]);
                acc[3] = fma(w, fma(T.x, E.x, T.y * E.y), acc[3]);
                acc[4] = fma(w, fma(E.x, B.x, E.y * B.y), acc[4]);
                acc[5] = fma(w, fma(T.x, B.x, T.y * B.y), acc[5]);
            } else {
                const double2 x = reinterpret_cast<const double2 *>(a.x[0])[i];
                const double2 y = reinterpret_cast<const double2 *>(a.y[0])[i];
                acc[0] = fma(w, fma(x.x, y.x, x.y * y.y), acc[0]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NX; ++t) part[t][half][li] = acc[t];
    __syncthreads();
    for (int i = threadIdx.x; i < NX * CL_L; i += blockDim.x) {
        const int t = i / CL_L, j = i % CL_L, lo = blockIdx.x * CL_L + j;
        if (lo > a.lmax) continue;
        double s = 0.0;
        for (int h = 0; h < HALVES; ++h) s += part[t][h][j];
        a.cl[(size_t)t * (a.lmax + 1) + lo] = s / (2.0 * lo + 1.0);
    }
}

}  // namespace

// One launch for all ring pairs (see ring_fourier_kernel on the groups).
template <bool SYN, int NT, int B, int G>
static hipError_t launch_rings_t(const ShtArgs &a, hipStream_t s) {
    const size_t lds = (size_t)ring_lds<G>(SYN) * a.nside * sizeof(double2);
    if (lds > 64 * 1024) {
        const void *k = SYN ? (const void *)ring_synth_kernel<NT, B, G> : (const void *)ring_fourier_kernel<NT, B, G>;
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (SYN) hipLaunchKernelGGL((ring_synth_kernel<NT, B, G>), dim3(2 * a.nside), dim3(NT * G), lds, s, a);
    else hipLaunchKernelGGL((ring_fourier_kernel<NT, B, G>), dim3(2 * a.nside), dim3(NT * G), lds, s, a);
    return hipGetLastError();
}

template <bool SYN>
static hipError_t launch_rings(const ShtArgs &a, hipStream_t s) {
    static_assert(SHT_MAX_NSIDE <= 2 * 512, "butterflies of the longest ring");
    if (a.nside > 512) return launch_rings_t<SYN, 512, 2, 1>(a, s);
    if (a.nside > 256) return launch_rings_t<SYN, 256, 2, 4>(a, s);
    if (a.nside > 128) return launch_rings_t<SYN, 128, 2, 4>(a, s);
    return launch_rings_t<SYN, 64, 2, 12>(a, s);
}

hipError_t launch_ring_fourier(const ShtArgs &a, hipStream_t s) { return launch_rings<false>(a, s); }

template <bool POL>
static void launch_alm2ring(const ShtArgs &a, hipStream_t s) {
    const dim3 g(a.mmax + 1);
    if (a.nside > 512) hipLaunchKernelGGL((alm2ring_kernel<POL, 4, 8, 2>), g, dim3(512), 0, s, a);
    else if (a.nside > 256) hipLaunchKernelGGL((alm2ring_kernel<POL, 4, 4, 2>), g, dim3(256), 0, s, a);
    else if (a.nside > 128) hipLaunchKernelGGL((alm2ring_kernel<POL, 2, 4, 2>), g, dim3(256), 0, s, a);
    else if (a.nside > 64) hipLaunchKernelGGL((alm2ring_kernel<POL, 1, 4, 4>), g, dim3(256), 0, s, a);
    else if (a.nside > 32) hipLaunchKernelGGL((alm2ring_kernel<POL, 1, 2, 4>), g, dim3(128), 0, s, a);
    else hipLaunchKernelGGL((alm2ring_kernel<POL, 1, 1, 4>), g, dim3(64), 0, s, a);
}

hipError_t launch_alm2map(const ShtArgs &a, hipStream_t s) {
    if (a.nfields == 3) launch_alm2ring<true>(a, s);
    else launch_alm2ring<false>(a, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_rings<true>(a, s);
}

hipError_t launch_steps(const ShtArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(steps_kernel, dim3((unsigned)(a.lmax / 256 + 1), (unsigned)(a.mmax + 1)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// K and NW cover 2 nside pairs with one workgroup: four pairs a lane on large maps
// (the cross-lane sums are shared by four pairs), one on small ones, where the
// workgroups are few and the chain of l is the time (nside 128, lmax 383: 70 us,
// 178 with eight waves and four pairs a lane for any map; eight l a block there,
// 70 against 76 with four).
template <bool POL, int K, int NW, int LB>
static hipError_t launch_alm_t(ShtArgs a, hipStream_t s) {
    static_assert(sizeof(WxStep) == sizeof(Step), "either kind of staged steps");
    const size_t lds = alm_lds<POL, NW, LB>() + 2 * LCHUNK * sizeof(Step);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)alm_kernel<POL, K, NW, LB>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (POL) {
        a.wx_m = min(a.nside > WX_NSIDE ? WX_M : 2, a.mmax + 1);
        a.wx_parts = (2 * a.nside + 64 * NW - 1) / (64 * NW);
    }
    const int blocks = a.wx_m * a.wx_parts + a.mmax + 1 - a.wx_m;
    hipLaunchKernelGGL((alm_kernel<POL, K, NW, LB>), dim3(blocks), dim3(64 * NW), lds, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.wx_parts < 2) return e;
    const int64_t count = (int64_t)a.wx_m * (2 * a.lmax + 3 - a.wx_m) / 2;      // a_lm of m < wx_m
    hipLaunchKernelGGL(wx_reduce_kernel, dim3((unsigned)((3 * count + 255) / 256)), dim3(256), 0, s, a, count);
    return hipGetLastError();
}

template <bool POL>
static hipError_t launch_alm_p(const ShtArgs &a, hipStream_t s) {
    if (a.nside > 512) return launch_alm_t<POL, 4, 8, 4>(a, s);
    if (a.nside > 256) return launch_alm_t<POL, 4, 4, 4>(a, s);
    if (a.nside > 128) return launch_alm_t<POL, 2, 4, 4>(a, s);
    if (a.nside > 64) return launch_alm_t<POL, 1, 4, 8>(a, s);
    if (a.nside > 32) return launch_alm_t<POL, 1, 2, 8>(a, s);
    return launch_alm_t<POL, 1, 1, 8>(a, s);
}

hipError_t launch_alm(const ShtArgs &a, hipStream_t s) {
    return a.nfields == 3 ? launch_alm_p<true>(a, s) : launch_alm_p<false>(a, s);
}

hipError_t launch_alm2cl(const ClArgs &a, hipStream_t s) {
    const dim3 g(a.lmax / CL_L + 1), t(64 * CL_WAVES);
    if (a.teb) hipLaunchKernelGGL(alm2cl_kernel<true>, g, t, 0, s, a);
    else hipLaunchKernelGGL(alm2cl_kernel<false>, g, t, 0, s, a);
    return hipGetLastError();
}

}  // namespace pisco
