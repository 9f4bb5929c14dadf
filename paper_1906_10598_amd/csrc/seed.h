// seed.h -- initial-range estimation of Sec. 3.1.1 on the device.
//
// The initial search box comes from short pieces of the block: the
// frequency at the block centre from the spectrum of a centred snippet, the
// frequency rate from a central difference of three equally spaced
// snippets, and the amplitude from the same spectrum.  One workgroup per
// snippet:
//   1. the M samples (M a power of two), two by two as M/2 complex numbers,
//      go from memory into the first pass of a radix-4 self-sorting FFT over
//      LDS (a radix-2 pass first where log2 M/2 is odd), and the even and odd
//      samples' spectra are separated where a bin is looked at;
//   2. the peak bin k* maximises |X_k|^2 over 1 <= k < M/2 (lowest k on
//      ties) by an argmax over lanes, then waves;
//   3. the frequency is refined between bins with Candan's bias-corrected
//      interpolator for a rectangular window (IEEE Signal Proc. Lett. 2011):
//      d = tan(pi/M)/(pi/M) * Re[(X_{k-1} - X_{k+1}) / (2 X_k - X_{k-1} - X_{k+1})];
//   4. the amplitude is 2 |sum_n x_n exp(-2 pi i f n / fs)| / M at the refined
//      frequency (phase in turns, exactly reduced), and the noise variance is
//      mean(x^2) - A^2 / 2.
// The estimates are per snippet; the host forms f0, f1, f2 and the box.
#pragma once

#include "kernels.h"

namespace pt {

constexpr int kSeedThreads = 1024;
constexpr int kSeedMaxLog = 13;  // M <= 8192 (64 KiB of LDS: M / 2 complex numbers)

struct SeedSnippet {
    double f;      // Hz
    double amp;    // amplitude
    double noise;  // noise standard deviation
    int bin;       // peak bin k*
    int pad;
};

struct SeedStarts {
    int64_t v[3];  // first sample of each snippet
};

// (power, bin) order of the peak search: larger power, then lower bin.
__device__ __forceinline__ bool seed_better(double p, int k, double q, int m) {
    return p > q || (p == q && k < m);
}

struct Cplx {
    double re, im;
};
__device__ __forceinline__ Cplx cadd(Cplx a, Cplx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ Cplx csub(Cplx a, Cplx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ Cplx cmul(Cplx a, Cplx b) {
    return {__fma_rn(a.re, b.re, -(a.im * b.im)), __fma_rn(a.re, b.im, a.im * b.re)};
}
// exp(-2 pi i turns), turns exact and small
__device__ __forceinline__ Cplx cturn(double turns) {
    double sn, cs;
    sincospi(2.0 * turns, &sn, &cs);
    return {cs, -sn};
}
// exp(-2 pi i nu n): the exact product's turns, reduced first
__device__ __forceinline__ Cplx cphase(double nu, double n) {
    const double q = nu * n, low = __fma_rn(nu, n, -q);
    return cturn((q - rint(q)) + low);
}

// A chain of short steps with little in each: the passes over LDS, the search,
// the amplitude.  Three workgroups and one wave per SIMD or two, so latency
// bounds it: as few passes and barriers as the registers allow (radix 4 on half
// the points: 6 passes for M = 4096 instead of 12), one twiddle pair per pass
// rather than a table (its power-of-two strides fall on one LDS bank), nothing
// serial over waves, samples held from the load on, results straight into host
// memory.  M = 4096: kernel 30 -> 13 us, the call 47 -> 30 us
// (1024: 28.5 -> 23 us).
template <typename T>
__global__ __launch_bounds__(kSeedThreads) void k_seed_spectrum(const T* __restrict__ s, SeedStarts starts,
                                                                int logM, double fs, double tanc,
                                                                SeedSnippet* __restrict__ out) {
    extern __shared__ double lds[];
    const int M = 1 << logM, N = M >> 1;
    Cplx* z = reinterpret_cast<Cplx*>(lds);  // N
    __shared__ double wp[kSeedThreads / 64];
    __shared__ int wk[kSeedThreads / 64];
    __shared__ double wsum[3][kSeedThreads / 64];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, nwave = blockDim.x >> 6;
    const T* x = s + starts.v[blockIdx.x];

    // First pass from memory.  R = 4: z[j + r N / 4] of the first N / 4 threads;
    // R = 2 (log2 N odd): z[j + r N / 2] of the first N / 2.
    const int lgN = logM - 1, R = lgN & 1 ? 2 : 4, stride = N / R;
    const bool mine = tid < stride;
    Cplx v[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    if (mine) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (r < R) v[r] = {(double)x[2 * (tid + r * stride)], (double)x[2 * (tid + r * stride) + 1]};
        if (R == 4) {
            const Cplx a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = csub(v[1], v[3]);
            z[4 * tid] = cadd(a, c);
            z[4 * tid + 1] = {b.re + d.im, b.im - d.re};
            z[4 * tid + 2] = csub(a, c);
            z[4 * tid + 3] = {b.re - d.im, b.im + d.re};
        } else {
            z[2 * tid] = cadd(v[0], v[1]);
            z[2 * tid + 1] = csub(v[0], v[1]);
        }
    }
    for (int l = lgN & 1 ? 1 : 2; l < lgN; l += 2) {
        const int Ns = 1 << l, k = tid & (Ns - 1), q = N >> 2;
        const double turn = ldexp((double)k, -(l + 2));
        const Cplx w1 = cturn(turn), w2 = cturn(2.0 * turn), w3 = cmul(w1, w2);
        Cplx t0, t1, t2, t3;
        __syncthreads();
        if (tid < q) {
            t0 = z[tid];
            t1 = cmul(w1, z[tid + q]);
            t2 = cmul(w2, z[tid + 2 * q]);
            t3 = cmul(w3, z[tid + 3 * q]);
        }
        __syncthreads();
        if (tid < q) {
            const Cplx a = cadd(t0, t2), b = csub(t0, t2), c = cadd(t1, t3), d = csub(t1, t3);
            Cplx* o = z + ((tid - k) << 2) + k;
            o[0] = cadd(a, c);
            o[Ns] = {b.re + d.im, b.im - d.re};
            o[2 * Ns] = csub(a, c);
            o[3 * Ns] = {b.re - d.im, b.im + d.re};
        }
    }
    __syncthreads();

    // peak bin: bins k and N - k share the two points they are made of
    // (Z_k + conj Z_{N-k}) / 2 = E, (Z_k - conj Z_{N-k}) / 2i = O:
    // X_k = E + exp(-2 pi i k / M) O, X_{N-k} = conj(E - exp(-2 pi i k / M) O)
    auto parts = [&](int k, Cplx& e, Cplx& wo) {
        const Cplx a = z[k & (N - 1)], b = z[(N - k) & (N - 1)];
        e = {0.5 * (a.re + b.re), 0.5 * (a.im - b.im)};
        wo = cmul(cturn(ldexp((double)k, -logM)), {0.5 * (a.im + b.im), 0.5 * (b.re - a.re)});
    };
    double bp = -1.0;
    int bk = 0x7fffffff;
    for (int k = 1 + tid; k <= (N >> 1); k += blockDim.x) {
        Cplx e, wo;
        parts(k, e, wo);
        const Cplx lo = cadd(e, wo), hi = csub(e, wo);
        const double p = __fma_rn(lo.re, lo.re, lo.im * lo.im), q = __fma_rn(hi.re, hi.re, hi.im * hi.im);
        if (seed_better(p, k, bp, bk)) {
            bp = p;
            bk = k;
        }
        if (seed_better(q, N - k, bp, bk)) {
            bp = q;
            bk = N - k;
        }
    }
    // the wave's largest power, then the lowest bin that has it
    auto best_of = [&] {
        const double top = wave_extreme<true>(bp);
        bk = (int)wave_extreme<false>(bp == top ? (double)bk : 2147483647.0);
        bp = top;
    };
    best_of();
    if (lane == 0) {
        wp[wave] = bp;
        wk[wave] = bk;
    }
    __syncthreads();
    // (every wave by itself: no barrier and no broadcast through LDS)
    bp = lane < nwave ? wp[lane] : -1.0;
    bk = lane < nwave ? wk[lane] : 0x7fffffff;
    best_of();
    // (non-finite samples leave no candidate: fall back to bin 1, in range)
    const int k = (bk >= 1 && bk < N) ? bk : 1;
    // Candan's interpolator; X_{k-1} and X_{k+1} exist for 1 <= k < M/2
    Cplx e, wo;
    parts(k - 1 + min(lane, 2), e, wo);
    const Cplx X = cadd(e, wo);
    const Cplx xl = {__shfl(X.re, 0), __shfl(X.im, 0)}, xc = {__shfl(X.re, 1), __shfl(X.im, 1)},
               xr = {__shfl(X.re, 2), __shfl(X.im, 2)};
    const double nr = xl.re - xr.re, ni = xl.im - xr.im;
    const double dr = 2.0 * xc.re - xl.re - xr.re, di = 2.0 * xc.im - xl.im - xr.im;
    const double den = __fma_rn(dr, dr, di * di);
    double d = 0.0;
    if (den > 0.0) d = tanc * (__fma_rn(nr, dr, ni * di) / den);
    const double f = ((double)k + d) * fs / (double)M;

    // amplitude at the refined frequency, and the snippet's power: sample
    // 2 (j + r stride) + h turns by exp(-2 pi i nu 2 j) times the r-th power of
    // one common factor and, for h = 1, another
    const double nu = f / fs;  // turns per sample
    double y[3] = {0.0, 0.0, 0.0};  // real and imaginary part, sum of squares
    if (mine) {
        Cplx p = cphase(nu, (double)(2 * tid));
        const Cplx odd = cphase(nu, 1.0), step = cphase(nu, (double)(2 * stride));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (r >= R) break;
            const Cplx po = cmul(p, odd);
            y[0] = __fma_rn(v[r].re, p.re, __fma_rn(v[r].im, po.re, y[0]));
            y[1] = __fma_rn(v[r].re, p.im, __fma_rn(v[r].im, po.im, y[1]));
            y[2] = __fma_rn(v[r].re, v[r].re, __fma_rn(v[r].im, v[r].im, y[2]));
            p = cmul(p, step);
        }
    }
    wave_sums(y);
    if (lane < 3) wsum[lane][wave] = lane == 0 ? y[0] : lane == 1 ? y[1] : y[2];
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) y[q] = lane < nwave ? wsum[q][lane] : 0.0;
        wave_sums(y);
        const double A = 2.0 * sqrt(__fma_rn(y[0], y[0], y[1] * y[1])) / (double)M;
        const double var = y[2] / (double)M - 0.5 * A * A;
        if (lane == 0) {
            SeedSnippet o;
            o.f = f;
            o.amp = A;
            o.noise = var > 0.0 ? sqrt(var) : 0.0;
            o.bin = k;
            o.pad = 0;
            out[blockIdx.x] = o;
        }
    }
}

}  // namespace pt
