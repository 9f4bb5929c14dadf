// nodes.hip -- kernels and plan of the node-weight fits (see nodes.h).
#define PT_INSTANCE_TU  // kernels.h: device functions only
#include "nodes.h"

#include <algorithm>
#include <cmath>

#include "kernels.h"

namespace pt {
namespace {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
// One step of a sum over a row of 16 lanes (0-3), pairs of rows (4) and the
// halves of the wave (5): the steps of wave_sums.
template <int STEP, int N>
__device__ __forceinline__ void sum_step(double (&v)[N]) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
        if constexpr (STEP < 4)
            v[r] += dpp_move(v[r], STEP);
        else
            v[r] = swap_add<STEP == 5>(v[r]);
    }
}

// Sum over the row of 16 lanes, in every lane of the row.
template <int N>
__device__ __forceinline__ void row_sums(double (&v)[N]) {
    sum_step<0>(v);
    sum_step<1>(v);
    sum_step<2>(v);
    sum_step<3>(v);
}

// Lane L of each row of 16, in every lane of the row.
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + L, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + L, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

template <bool MAX>
__device__ __forceinline__ double wave_extreme(double v) {
    auto pick = [](double a, double b) { return MAX ? fmax(a, b) : fmin(a, b); };
#pragma unroll
    for (int s = 0; s < 4; ++s) v = pick(v, dpp_move(v, s));
    v = pick(v, __shfl_xor(v, 16, 64));
    return pick(v, __shfl_xor(v, 32, 64));
}

// cos(2 pi a / n) for integers a >= 0, n > 0, reduced exactly.
__device__ __forceinline__ double cos_ratio(int a, int n, double inv) {
    const int q = (int)((double)a * inv);
    const int rem = a - q * n;  // within one n of [0, n)
    const double t = (double)rem * inv;
    const double r = t - rint(t);
    return cos_turns64(r * r);
}

__device__ __forceinline__ int node_block_of(const NodeDesc* nd, int nblk, int wg, bool mom) {
    int lo = 0, hi = nblk - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((mom ? nd[mid].mom_begin : nd[mid].proj_begin) <= wg) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Packed draws of one member: r1, r2, r3 in bytes 0-2, the slots the binomial
// crossover takes from the mutant in byte 3.
__device__ __forceinline__ uint32_t node_pack(const BlockDesc* d, const Draws& w) {
    uint32_t m = 0;
    for (int a = 0; a < d->D; ++a)
        if ((w.cross >> a) & 1u) m |= 1u << d->act[a];
    return (uint32_t)w.r1 | ((uint32_t)w.r2 << 8) | ((uint32_t)w.r3 << 16) | (m << 24);
}

// The draws of generations g .. g + ngen - 1 of every member, by workgroups
// of 256 threads beside the kernel's own work: they depend on nothing but the
// stream, so they are kept off the fit's chain of generations (three Philox
// calls cost as much as a whole evaluation there).
__device__ __forceinline__ void node_draws(const NodeDesc* nd, const BlockDesc* bd, int slice, int slices, int P, int g_off,
                                           int ngen, int chunk, int flip) {
    const int b = slice / slices, id = (slice - b * slices) * (int)blockDim.x + (int)threadIdx.x;
    if (id >= P * ngen) return;
    const NodeDesc* n = nd + b;
    const BlockDesc* d = bd + b;
    const int gl = id / P, i = id - gl * P;
    const Draws w = trial_draws(d, i, (uint32_t)(n->g0 + g_off + gl));
    n->draws[(size_t)((n->parity + flip) & 1) * chunk * P + id] = node_pack(d, w);
}

// ---------------------------------------------------------------------------
// Projection: a lane takes 16 consecutive samples at a time, forms s e and
// e^2 (e = exp(i phi_ref), the phase reduced exactly in turns) and adds them
// to 16 Chebyshev moments of its tile's coordinate; the lanes of a tile add
// up by DPP moves and the moments become values at the tile's 16 nodes.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void project_unit(const NodeDesc* nd, const BlockDesc* d, int wg, double* tab, double* red) {
    constexpr int S = 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t N = d->n;
    const int LL = nd->lanes_log, runs = nd->runs;
    const int64_t B = (int64_t)S * runs << LL, Be = B < N ? B : N;
    const int64_t tt = LL == 8 ? wg : (((int64_t)wg << 8) + tid) >> LL;
    const int64_t ts = tt * B < N - Be ? tt * B : N - Be;
    const double cen = (double)ts + 0.5 * (double)(Be - 1), ih = 2.0 / (double)(Be - 1);
    const double r1h = nd->r1h, r1l = nd->r1l, r2 = nd->r2, r3 = nd->r3, r4 = nd->r4, ref = d->ref;

    if (tid < 64) {
        const double r = tid * (1.0 / 64.0), q = r - rint(r);
        tab[tid] = cos_turns64(q * q);  // cos(2 pi k / 64)
    }
    double M[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) M[k] = 0.0;
    double s2[1] = {0.0};
    for (int q = 0; q < runs; ++q) {
        const int tile = wg * runs + q;
        T raw[S];
        double sv[S];
        bool full;
        int valid;
        load_lane_raw<T, S>(d, tile, raw);
        finish_lane<double, T, S>(d, tile, raw, sv, full, valid);
        const double n0 = (double)((int64_t)tile * kNodeRun + tid * S);
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const double n = n0 + (double)j, m = n - ref, x = (n - cen) * ih;
            double p = r1h * m;
            const double e = __fma_rn(r1h, m, -p);
            p -= rint(p);
            double q2 = m * m * __fma_rn(__fma_rn(r4, m, r3), m, r2);
            q2 -= rint(q2);
            double r = p + (q2 + __fma_rn(r1l, m, e));
            r -= rint(r);
            double c, sn;
            sincos_turns64(r, c, sn);
            const double keep = j < valid ? 1.0 : 0.0;  // (samples past the end are zero already)
            const double v = sv[j];
            s2[0] = __fma_rn(v, v, s2[0]);
            const double zr = v * c, zi = v * sn;
            const double wr = keep * __fma_rn(c, c, -(sn * sn)), wi = keep * (2.0 * c * sn);
            double t0 = 1.0, t1 = x;
            M[0] += zr;
            M[1] += zi;
            M[2] += wr;
            M[3] += wi;
#pragma unroll
            for (int k = 1; k < 16; ++k) {
                M[4 * k] = __fma_rn(t1, zr, M[4 * k]);
                M[4 * k + 1] = __fma_rn(t1, zi, M[4 * k + 1]);
                M[4 * k + 2] = __fma_rn(t1, wr, M[4 * k + 2]);
                M[4 * k + 3] = __fma_rn(t1, wi, M[4 * k + 3]);
                const double t2 = __fma_rn(2.0 * x, t1, -t0);
                t0 = t1;
                t1 = t2;
            }
        }
    }
    __syncthreads();  // tab complete
    // lanes of one tile (2^LL)
    if (LL > 0) sum_step<0>(M);
    if (LL > 1) sum_step<1>(M);
    if (LL > 2) sum_step<2>(M);
    if (LL > 3) sum_step<3>(M);
    if (LL > 4) sum_step<4>(M);
    if (LL > 5) sum_step<5>(M);
    wave_sums(s2);
    if (lane == 0) red[256 + wave] = s2[0];
    if (LL > 6 && lane == 0) {
#pragma unroll
        for (int k = 0; k < 64; ++k) red[wave * 64 + k] = M[k];
    }
    __syncthreads();
    if (tid == 0) nd->s2[wg] = (red[256] + red[257]) + (red[258] + red[259]);
    const int L = 1 << LL, first = LL > 6 ? tid & (L - 1) : lane & (L - 1);
    if (LL > 6) {
        // two or four waves share a tile
        const int w0 = LL == 8 ? 0 : wave & ~1;
#pragma unroll
        for (int k = 0; k < 64; ++k) {
            double a = red[w0 * 64 + k] + red[(w0 + 1) * 64 + k];
            if (LL == 8) a += red[128 + k] + red[192 + k];
            M[k] = a;
        }
    }
    if (tt >= nd->ntile) return;
    for (int i = first; i < kNodePts; i += L) {
        double v[4] = {0.5 * M[0], 0.5 * M[1], 0.5 * M[2], 0.5 * M[3]};
#pragma unroll
        for (int k = 1; k < 16; ++k) {
            const double t = tab[(k * (2 * i + 1)) & 63];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = __fma_rn(t, M[4 * k + q], v[q]);
        }
        double* o = nd->pts + ((size_t)tt * kNodePts + i) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) gst(o + q, 0.125 * v[q]);
    }
}

__global__ __launch_bounds__(256) void k_node_project(const NodeDesc* __restrict__ nds, const BlockDesc* __restrict__ bds,
                                                      int nblk, int total, int P, int ngen, int chunk, int slices) {
    __shared__ double tab[64], red[260];
    const int wg = blockIdx.x;
    if (wg >= total) {
        node_draws(nds, bds, wg - total, slices, P, 0, ngen, chunk, 0);
        return;
    }
    const int b = node_block_of(nds, nblk, wg, false);
    const NodeDesc* nd = nds + b;
    const BlockDesc* d = bds + b;
    if (d->dtype == PT_F64)
        project_unit<double>(nd, d, wg - nd->proj_begin, tab, red);
    else
        project_unit<float>(nd, d, wg - nd->proj_begin, tab, red);
}

// ---------------------------------------------------------------------------
// Moments: sum over 128 points of value x T_j(x_point) for j < K; a lane holds
// one j, the waves share the points.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_node_moments(const NodeDesc* __restrict__ nds, const BlockDesc* __restrict__ bds,
                                                      int nblk) {
    __shared__ double th[kNodeGroup], v[kNodeGroup][4], red[4][64][4];
    const int b = node_block_of(nds, nblk, blockIdx.x, true);
    const NodeDesc* nd = nds + b;
    const BlockDesc* d = bds + b;
    const int wg = blockIdx.x - nd->mom_begin, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t N = d->n;
    const int64_t B = (int64_t)16 * nd->runs << nd->lanes_log, Be = B < N ? B : N;
    const int npt = nd->ntile * kNodePts, p0 = wg * kNodeGroup, np = min(kNodeGroup, npt - p0);
    if (tid < np) {
        const int pt = p0 + tid, i = pt & (kNodePts - 1);
        const int64_t t = pt / kNodePts;
        const int64_t ts = t * B < N - Be ? t * B : N - Be;
        const double xi = cos_ratio(2 * i + 1, 4 * kNodePts, 1.0 / (4 * kNodePts));
        const double n = (double)ts + 0.5 * (double)(Be - 1) * (1.0 + xi);
        double x = (n - 0.5 * (double)(N - 1)) / nd->h;
        x = x > 1.0 ? 1.0 : (x < -1.0 ? -1.0 : x);
        th[tid] = acos(x) * 0.15915494309189533577;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[tid][q] = gld(nd->pts + (size_t)pt * 4 + q);
    }
    __syncthreads();
    const int K = nd->K;
    for (int j0 = 0; j0 < K; j0 += 64) {
        const double j = (double)(j0 + lane);
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int p = wave; p < np; p += 4) {
            const double t = th[p], y = j * t, e = __fma_rn(j, t, -y);
            const double r = (y - rint(y)) + e;
            const double c = cos_turns64(r * r);
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = __fma_rn(c, v[p][q], a[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) red[wave][lane][q] = a[q];
        __syncthreads();
        const int jl = tid >> 2, q = tid & 3;
        if (j0 + jl < K)
            gst(nd->mom + ((size_t)wg * K + j0 + jl) * 4 + q,
                (red[0][jl][q] + red[1][jl][q]) + (red[2][jl][q] + red[3][jl][q]));
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// The fit: one workgroup per block runs `ngen` generations.
//
// Member m belongs to a row of 16 lanes (waves 0 .. W - 1, four rows each, NM
// members per row): lanes 0-6 of the row hold the member's slots, build its
// trial from the rows of the previous generation in LDS and turn it into the
// coefficients of delta; all 16 lanes then evaluate delta, exp(i delta) and
// the weighted sums at the nodes k = lane, lane + 16, ... and the row adds up
// by DPP moves, so selection needs no exchange between waves.  One barrier
// per generation separates writing the selected rows from reading them (two
// copies alternate).  Wave W keeps the books one generation behind: best
// member, history, stop rule.
//
// Once the population has drawn together so far that every trial stays
// within an eighth of a turn of the best member's phase, the weights are
// re-expanded about that member's phase on 16 nodes (relevel): one node per
// lane, held in registers, no phase reduction, a shorter sine and cosine.  A
// trial outside the re-expansion's limits is evaluated on the full set.
//
// The step of Table 4 (selection, random draws, bound rule, stop rule) is that
// of de_step_body.
// ---------------------------------------------------------------------------
struct FitLds {
    double *xs, *fs, *zw, *un, *nar, *scr, *ring;
    uint32_t* dr;
};

__host__ __device__ inline size_t fit_lds_doubles(int P, int maxK) {
    return (size_t)((2 * P * kSlots + 1) & ~1) + ((2 * P + 1) & ~1) + 9 * (size_t)maxK + 5 * kNodePts + kNodeRing;
}

__device__ __forceinline__ FitLds fit_lds(double* base, int P, int maxK) {
    FitLds l;
    l.xs = base;
    l.fs = l.xs + ((2 * P * kSlots + 1) & ~1);
    l.zw = l.fs + ((2 * P + 1) & ~1);
    l.scr = l.zw + 4 * maxK;
    l.un = l.scr + 4 * maxK;
    l.nar = l.un + maxK;
    l.ring = l.nar + 5 * kNodePts;
    l.dr = reinterpret_cast<uint32_t*>(l.ring + kNodeRing);
    return l;
}

struct FitShared {
    double mid[8], lim[8];  // centre and limits of the narrow set, per slot
    double S2, best_f;
    int stop[2];            // DeState flags of a stop, by generation parity
    int pend;               // generation before which the weights are re-expanded, -1: none
    int best, stop_gen;
};

// Coefficients of one candidate's phase difference (turns, in u) and its
// amplitude A + B u.
struct NodeCand {
    double p0, p1, p2, p3, p4, A, B;
};

template <bool SLOPE, bool QUART>
__device__ __forceinline__ NodeCand node_cand(double dj) {
    NodeCand q;
    q.A = row_bcast<0>(dj);
    q.p0 = row_bcast<1>(dj);
    q.p1 = row_bcast<2>(dj);
    q.p2 = row_bcast<3>(dj);
    q.p3 = row_bcast<4>(dj);
    q.B = SLOPE ? row_bcast<5>(dj) : 0.0;
    q.p4 = QUART ? row_bcast<6>(dj) : 0.0;
    return q;
}

template <bool QUART>
__device__ __forceinline__ double node_delta(const NodeCand& q, double u) {
    double t = QUART ? __fma_rn(q.p4, u, q.p3) : q.p3;
    t = __fma_rn(t, u, q.p2);
    t = __fma_rn(t, u, q.p1);
    return __fma_rn(t, u, q.p0);
}

// One node's terms: a1 += amp Re(-2 Z e), a2 += s t with t = Wr s + Wi c
// (Re(W e^2) = Wr - 2 s t), or with a slope amp^2 Re(W e^2).
template <bool SLOPE>
__device__ __forceinline__ void node_terms(const NodeCand& q, double u, double c, double s, double zr, double zi,
                                           double wr, double wi, double& a1, double& a2) {
    const double t = __fma_rn(wr, s, wi * c);
    if constexpr (SLOPE) {
        const double amp = __fma_rn(q.B, u, q.A);
        a1 = __fma_rn(amp, __fma_rn(zr, c, -(zi * s)), a1);
        a2 = __fma_rn(amp * amp, __fma_rn(-2.0 * s, t, wr), a2);
    } else {
        a1 = __fma_rn(zr, c, __fma_rn(-zi, s, a1));
        a2 = __fma_rn(s, t, a2);
    }
}

// Objective from a row's sums.
template <bool SLOPE>
__device__ __forceinline__ double node_objective(const NodeDesc* nd, const NodeCand& q, double a1, double a2, bool cor,
                                                 double S2, double energy0, double N) {
    double v[1];
    if (cor)
        v[0] = SLOPE ? a1 : q.A * a1;
    else
        v[0] = SLOPE ? __fma_rn(0.5, a2, a1) : q.A * __fma_rn(-q.A, a2, a1);
    row_sums(v);
    // correlation objective, Eq. (2-2-5): F = 1 / (arctan(C) + pi/2)
    if (cor) return 1.0 / (atan(-0.5 * v[0]) + 1.5707963267948966192);
    double e;  // half the energy of the amplitude (with the mean of cos 2 phi's constant part)
    if constexpr (SLOPE)
        e = 0.5 * __fma_rn(q.B * q.B, nd->su2, __fma_rn(2.0 * q.A * q.B, nd->su1, q.A * q.A * N));
    else
        e = q.A * q.A * energy0;
    return (S2 + e) + v[0];
}

// Sums over the full node set for one candidate (the row's 16 lanes share the
// nodes).
template <bool SLOPE, bool QUART>
__device__ __forceinline__ void wide_sums(const NodeCand& q, const double* zw, const double* un, int l16, int K, double& a1,
                                          double& a2) {
#pragma unroll 2
    for (int k = l16; k < K; k += 16) {
        const double u = un[k];
        double r = node_delta<QUART>(q, u);
        r -= rint(r);
        double c, s;
        sincos_turns64(r, c, s);
        node_terms<SLOPE>(q, u, c, s, zw[4 * k], zw[4 * k + 1], zw[4 * k + 2], zw[4 * k + 3], a1, a2);
    }
}

// Half of (N + sum of Wr), the constant part of the energy: Wr at w[0],
// w[stride], ..., summed over the wave.
__device__ __forceinline__ double node_energy(const double* w, int n, int stride, double N) {
    double v[1] = {0.0};
    for (int k = threadIdx.x & 63; k < n; k += 64) v[0] += w[k * stride];
    wave_sums(v);
    return 0.5 * (N + v[0]);
}

// Weights re-expanded about the phase of the member in sh.mid, by the whole
// workgroup: Z exp(i d), W exp(2 i d) (d: that member's delta) as Chebyshev
// moments over the full nodes, then values at 16 nodes.
__device__ __noinline__ void relevel(const NodeDesc* nd, const FitLds& l, FitShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, NT = blockDim.x, K = nd->K;
    const NodeCand q{sh.mid[1] * nd->sc[1],
                     (sh.mid[2] - nd->mid[2]) * nd->sc[2],
                     (sh.mid[3] - nd->mid[3]) * nd->sc[3],
                     (sh.mid[4] - nd->mid[4]) * nd->sc[4],
                     (sh.mid[6] - nd->mid[6]) * nd->sc[6],
                     0.0,
                     0.0};
    for (int k = tid; k < K; k += NT) {
        double r = node_delta<true>(q, l.un[k]);
        r -= rint(r);
        double c, s;
        sincos_turns64(r, c, s);
        const double zr = l.zw[4 * k], zi = l.zw[4 * k + 1], wr = l.zw[4 * k + 2], wi = l.zw[4 * k + 3];
        const double c2 = __fma_rn(c, c, -(s * s)), s2 = 2.0 * c * s;
        l.scr[4 * k] = __fma_rn(zr, c, -(zi * s));
        l.scr[4 * k + 1] = __fma_rn(zr, s, zi * c);
        l.scr[4 * k + 2] = __fma_rn(wr, c2, -(wi * s2));
        l.scr[4 * k + 3] = __fma_rn(wr, s2, wi * c2);
    }
    __syncthreads();
    for (int j = wave; j < kNodePts; j += NT >> 6) {
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        for (int k = lane; k < K; k += 64) {
            const double t = cos_ratio(j * (2 * k + 1), 4 * K, 0.25 / (double)K);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = __fma_rn(t, l.scr[4 * k + e], a[e]);
        }
        wave_sums(a);
        if (lane == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) l.nar[e * kNodePts + j] = a[e];
        }
    }
    __syncthreads();
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (tid < kNodePts) {
        for (int j = 0; j < kNodePts; ++j) {
            const double t = j ? cos_ratio(j * (2 * tid + 1), 4 * kNodePts, 1.0 / (4 * kNodePts)) : 0.5;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __fma_rn(t, l.nar[e * kNodePts + j], v[e]);
        }
    }
    __syncthreads();
    if (tid < kNodePts) {
#pragma unroll
        for (int e = 0; e < 4; ++e) l.nar[e * kNodePts + tid] = 0.125 * v[e];
        l.nar[4 * kNodePts + tid] = cos_ratio(2 * tid + 1, 4 * kNodePts, 1.0 / (4 * kNodePts)) + nd->c;
    }
    if (tid == 0) sh.lim[7] = 1.0;
    __syncthreads();
}

// The bookkeeping of generation g, by one wave: best member, history, stop
// rule, and every 16th generation whether the narrow set can take over.
__device__ __forceinline__ void book(const NodeDesc* nd, const BlockDesc* d, const FitLds& l, FitShared& sh, int g) {
    const int lane = threadIdx.x & 63, P = d->P;
    const double* f = l.fs + (g & 1) * P;
    double fv[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) fv[t] = lane + 64 * t < P ? f[lane + 64 * t] : __builtin_inf();
    const double bf = wave_extreme<false>(fmin(fmin(fv[0], fv[1]), fmin(fv[2], fv[3])));
    int best = 0;  // lowest index on ties
#pragma unroll
    for (int t = 3; t >= 0; --t) {
        const unsigned long long hit = __ballot(lane + 64 * t < P && fv[t] == bf);
        if (hit) best = 64 * t + __ffsll(hit) - 1;
    }
    const int win = d->window;
    const bool wrule = d->rel_tol > 0.0 && win > 0 && g >= win;
    double old = 0.0;
    if (wrule) old = win < kNodeRing ? l.ring[(g - win) & (kNodeRing - 1)] : gld(d->hist + (g - win));
    int flags = 0;
    if (bf <= d->vtr) flags |= 4;                          // PT_FLAG_VTR
    if (wrule && old - bf <= d->rel_tol * bf) flags |= 1;  // PT_FLAG_CONVERGED
    if (!flags && g >= d->max_gens) flags |= 2;            // PT_FLAG_MAXGEN
    if (d->objective == 0 && !(bf >= kNodeCancel * sh.S2)) flags = kFlagNodeAbort;
    if (lane == 0) {
        l.ring[g & (kNodeRing - 1)] = bf;
        gst(d->hist + g, bf);
        sh.stop[(g + 1) & 1] = flags;
        sh.best = best;
        sh.best_f = bf;
        sh.stop_gen = g;
    }
    if ((g & 15) != 15 || flags || sh.pend >= 0) return;
    // largest distance of a member from the best one, per slot, and in turns
    const double* x = l.xs + (g & 1) * P * kSlots;
    const double* xb = x + best * kSlots;
    double rng[kSlots], q[5];
#pragma unroll
    for (int j = 1; j < kSlots; ++j) {
        double a = 0.0;
        for (int m = lane; m < P; m += 64) a = fmax(a, fabs(x[m * kSlots + j] - xb[j]));
        rng[j] = wave_extreme<true>(a);
        if (j != 5) q[j == 6 ? 4 : j - 1] = rng[j] * nd->sc[j];
    }
    // growth of |exp(2 i delta)| on the ellipse of sum of half axes e^3 for a
    // polynomial with these coefficients about x = 0: the interpolation error
    // on 16 nodes is below 1e-15 while it stays below 15 (9 with the two
    // further degrees of a sloping amplitude)
    const double c = fabs(nd->c);
    const double b1 = q[1] + c * (2.0 * q[2] + c * (3.0 * q[3] + 4.0 * c * q[4]));
    const double b2 = q[2] + c * (3.0 * q[3] + 6.0 * c * q[4]), b3 = q[3] + 4.0 * c * q[4];
    const double G = 12.566370614359172 * (10.018 * b1 + 100.86 * b2 + 1020.4 * b3 + 10273.0 * q[4]);
    const double w = 1.0 + c;
    const double sum = q[0] + w * (q[1] + w * (q[2] + w * (q[3] + w * q[4])));
    // the limits: the distances scaled up as far as both bounds allow; worth it
    // once a mutant x1 + F (x2 - x3) of such members lies well inside
    const double scale = fmin((nd->slope ? 9.0 : 15.0) / G, 0.125 / sum);
    if (scale >= 1.5 * (1.0 + 2.0 * d->F) && lane == 0) {
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            const bool amp = j == 0 || j == 5;
            sh.mid[j] = amp ? 0.0 : xb[j];
            sh.lim[j] = amp ? __builtin_inf() : rng[j] * scale;
        }
        sh.pend = g + 2;
    }
}

// The generations of the members' waves; returns the generation at which the
// loop ended (g1, or the one dropped after a stop).
template <int NM, bool SLOPE, bool QUART>
__device__ __forceinline__ int member_loop(const NodeDesc* nd, const BlockDesc* d, int g0, int g1, bool fresh,
                                           const FitLds& l, FitShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15;
    const int W = (blockDim.x >> 6) - 1, P = d->P, K = nd->K;
    const bool cor = d->objective != 0;
    const double N = (double)d->n, S2 = sh.S2, Fm = d->F;

    // constants of the slot this lane holds (lanes 7-15: none)
    const int jl = l16 < kSlots ? l16 : kSlots - 1;
    const bool slot = l16 < kSlots;
    const double lo_j = gld(&d->lo[jl]), hi_j = gld(&d->hi[jl]);
    const double mid_w = slot ? gld(&nd->mid[jl]) : 0.0, sc_j = slot ? gld(&nd->sc[jl]) : 0.0;
    const double en_w = node_energy(l.zw + 2, K, 4, N);

    // the members of this row
    const int row = (wave << 2) + (lane >> 4), nrow = 4 * W;
    double xi[NM], fo[NM];
#pragma unroll
    for (int t = 0; t < NM; ++t) {
        const int m = min(row + t * nrow, P - 1);
        xi[t] = l.xs[((g0 + 1) & 1) * P * kSlots + m * kSlots + jl];
        fo[t] = fresh ? __builtin_inf() : l.fs[((g0 + 1) & 1) * P + m];
    }

    // trial coordinate of member m (generation g, draws w): apply_trial's arithmetic
    auto trial = [&](const double* xin, uint32_t w, double x) {
        const double x1 = xin[(w & 255u) * kSlots + jl];
        const double x2 = xin[((w >> 8) & 255u) * kSlots + jl];
        const double x3 = xin[((w >> 16) & 255u) * kSlots + jl];
        double v = __fma_rn(Fm, x2 - x3, x1);
        if (v < lo_j) v = (lo_j + x1) * 0.5;
        if (v > hi_j) v = (hi_j + x1) * 0.5;
        return (w >> (24 + jl)) & 1u ? v : x;
    };
    auto wide = [&](double y) {
        const NodeCand q = node_cand<SLOPE, QUART>((y - mid_w) * sc_j);
        double a1 = 0.0, a2 = 0.0;
        wide_sums<SLOPE, QUART>(q, l.zw, l.un, l16, K, a1, a2);
        return node_objective<SLOPE>(nd, q, a1, a2, cor, S2, en_w, N);
    };
    auto keep = [&](int t, int g, double y, double ft) {
        const bool take = g == 0 || ft <= fo[t];
        xi[t] = take ? y : xi[t];
        fo[t] = take ? ft : fo[t];
        const int m = row + t * nrow;
        if (m < P) {
            if (slot) l.xs[(g & 1) * P * kSlots + m * kSlots + l16] = xi[t];
            if (l16 == 0) l.fs[(g & 1) * P + m] = fo[t];
        }
    };

    int g = g0;
    bool narrow = sh.lim[7] > 0.0;  // (slot 7 of lim holds the flag)
    if (!narrow) {
        for (; g < g1; ++g) {
            if (sh.pend == g) {
                relevel(nd, l, sh);
                narrow = true;
                break;
            }
            const double* xin = l.xs + ((g + 1) & 1) * P * kSlots;
#pragma unroll
            for (int t = 0; t < NM; ++t) {
                double y = xi[t];
                if (g > 0) y = trial(xin, l.dr[(g - g0) * P + min(row + t * nrow, P - 1)], y);
                keep(t, g, y, wide(y));
            }
            __syncthreads();
            if (g > g0 && sh.stop[g & 1]) return g;
        }
        if (!narrow) return g;
    }

    const double nzr = l.nar[l16], nzi = l.nar[kNodePts + l16], nwr = l.nar[2 * kNodePts + l16],
                 nwi = l.nar[3 * kNodePts + l16], nu = l.nar[4 * kNodePts + l16];
    const double en_n = node_energy(l.nar + 2 * kNodePts, kNodePts, 1, N);
    const double mid_n = slot ? sh.mid[jl] : 0.0, lim = slot ? sh.lim[jl] : __builtin_inf();
    double kc[kNarDeg64 + 1], ks[kNarDeg64 + 1];  // held in vector registers
#pragma unroll
    for (int k = 0; k <= kNarDeg64; ++k) {
        kc[k] = kCosNar64[k];
        ks[k] = kSinNar64[k];
        asm volatile("" : "+v"(kc[k]), "+v"(ks[k]));
    }
    for (; g < g1; ++g) {
        const double* xin = l.xs + ((g + 1) & 1) * P * kSlots;
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            const double y = trial(xin, l.dr[(g - g0) * P + min(row + t * nrow, P - 1)], xi[t]);
            const double dn = y - mid_n;
            double ft;
            if (__builtin_expect(__ballot(fabs(dn) <= lim) == ~0ull, 1)) {
                const NodeCand q = node_cand<SLOPE, QUART>(dn * sc_j);
                const double r = node_delta<QUART>(q, nu), u = r * r;
                double c = kc[0], s = ks[0];
#pragma unroll
                for (int k = 1; k <= kNarDeg64; ++k) {
                    c = __fma_rn(c, u, kc[k]);
                    s = __fma_rn(s, u, ks[k]);
                }
                s *= r;
                double a1 = 0.0, a2 = 0.0;
                node_terms<SLOPE>(q, nu, c, s, nzr, nzi, nwr, nwi, a1, a2);
                ft = node_objective<SLOPE>(nd, q, a1, a2, cor, S2, en_n, N);
            } else {
                ft = wide(y);
            }
            keep(t, g, y, ft);
        }
        __syncthreads();
        if (g > g0 && sh.stop[g & 1]) return g;
    }
    return g;
}

// The same barriers for the bookkeeping wave, one generation behind.
__device__ __forceinline__ int book_loop(const NodeDesc* nd, const BlockDesc* d, int g0, int g1, const FitLds& l,
                                         FitShared& sh) {
    bool narrow = sh.lim[7] > 0.0;
    for (int g = g0; g < g1; ++g) {
        if (!narrow && sh.pend == g) {
            relevel(nd, l, sh);
            narrow = true;
        }
        if (g > g0) book(nd, d, l, sh, g - 1);
        __syncthreads();
        if (g > g0 && sh.stop[g & 1]) return g;
    }
    return g1;
}

template <int NM>
__device__ __forceinline__ void fit_run(const NodeDesc* nd, const BlockDesc* d, int g0, int ngen, bool fresh, const FitLds& l,
                                        FitShared& sh) {
    const int tid = threadIdx.x, NT = blockDim.x, W = (NT >> 6) - 1, P = d->P, g1 = g0 + ngen;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int g;
    if (wave == W) {
        g = book_loop(nd, d, g0, g1, l, sh);
    } else if (nd->slope) {
        g = d->quartic ? member_loop<NM, true, true>(nd, d, g0, g1, fresh, l, sh)
                       : member_loop<NM, true, false>(nd, d, g0, g1, fresh, l, sh);
    } else {
        g = d->quartic ? member_loop<NM, false, true>(nd, d, g0, g1, fresh, l, sh)
                       : member_loop<NM, false, false>(nd, d, g0, g1, fresh, l, sh);
    }
    int flags;
    if (g < g1) {
        flags = sh.stop[g & 1];  // generation g - 1 stopped the fit; g is dropped
    } else {
        if (wave == W) book(nd, d, l, sh, g1 - 1);
        __syncthreads();
        flags = sh.stop[g1 & 1];
    }

    // state for the next launch: the population after the last kept generation
    const int gl = flags ? sh.stop_gen : g1 - 1;
    const double* xl = l.xs + (gl & 1) * P * kSlots;
    const double* fl = l.fs + (gl & 1) * P;
    for (int e = tid; e < P * kSlots; e += NT) {
        const int m = e / kSlots;
        gst(d->pop + (size_t)m * kStride + (e - m * kSlots), xl[e]);
    }
    for (int m = tid; m < P; m += NT) gst(d->fpop + m, fl[m]);
    if (!flags) {
        for (int e = tid; e < 5 * kNodePts; e += NT) gst(nd->nar + e, l.nar[e]);
        if (tid < 8) {
            gst(nd->nar + 5 * kNodePts + tid, sh.mid[tid]);
            gst(nd->nar + 5 * kNodePts + 8 + tid, sh.lim[tid]);
        }
        if (tid == 0) gst(reinterpret_cast<int*>(nd->nar + kNodeNarrow), sh.pend);
    }
    if (tid == 0) {
        DeState* st = d->st;
        st->gen = flags ? gl : g1;
        st->done = flags != 0;
        st->flags = flags;
        st->best = sh.best;
        st->best_f = sh.best_f;
    }
}

template <int NM>
__global__ __launch_bounds__(1024) void k_node_fit(const NodeDesc* __restrict__ nds, const BlockDesc* __restrict__ bds,
                                                   int nblk, int P, int maxK, int off, int ngen, int next_ngen, int chunk,
                                                   int flip, int slices) {
    extern __shared__ __align__(16) double lds[];
    __shared__ FitShared sh;
    if ((int)blockIdx.x >= nblk) {
        node_draws(nds, bds, blockIdx.x - nblk, slices, P, off + ngen, next_ngen, chunk, flip + 1);
        return;
    }
    const NodeDesc* nd = nds + blockIdx.x;
    const BlockDesc* d = bds + blockIdx.x;
    const int g0 = nd->g0 + off, tid = threadIdx.x, NT = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const bool fresh = g0 == 0;
    if (!fresh && d->st->done) return;
    const FitLds l = fit_lds(lds, P, maxK);
    const int K = nd->K;

    const uint32_t* dr = nd->draws + (size_t)((nd->parity + flip) & 1) * chunk * P;
    for (int e = tid; e < ngen * P; e += NT) l.dr[e] = gld(dr + e);
    for (int k = tid; k < K; k += NT) l.un[k] = cos_ratio(2 * k + 1, 4 * K, 0.25 / (double)K) + nd->c;
    if (fresh) {
        init_block(d);
        if (tid < 8) sh.mid[tid] = sh.lim[tid] = 0.0;
        if (tid == 0) sh.pend = -1;
        const int n4 = 4 * K;
        for (int e = tid; e < n4; e += NT) {
            double s = 0.0;
            for (int w = 0; w < nd->nmom; ++w) s += gld(nd->mom + (size_t)w * n4 + e);
            l.scr[e] = s;
        }
        if (wave == 0) {
            double s[1] = {0.0};
            for (int w = lane; w < nd->nproj; w += 64) s[0] += gld(nd->s2 + w);
            wave_sums(s);
            if (lane == 0) sh.S2 = s[0];
        }
        __syncthreads();
        // values at the nodes from the moments: a row of 16 lanes per node
        const int l16 = lane & 15;
        const double inv = 0.25 / (double)K;
        for (int k = tid >> 4; k < K; k += NT >> 4) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            for (int j = l16; j < K; j += 16) {
                const double t = j ? cos_ratio(j * (2 * k + 1), 4 * K, inv) : 0.5;
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = __fma_rn(t, l.scr[4 * j + q], a[q]);
            }
            row_sums(a);
            if (l16 < 4) {
                const double v = l16 == 0 ? a[0] : (l16 == 1 ? a[1] : (l16 == 2 ? a[2] : a[3]));
                const double w = v * (2.0 / (double)K) * (l16 < 2 ? -2.0 : 1.0);  // -2 Z, W
                l.zw[4 * k + l16] = w;
                gst(nd->wts + 4 * k + l16, w);
            }
        }
        if (tid == 0) gst(nd->wts + 4 * kNodeMaxK, sh.S2);
        for (int e = tid; e < P * kSlots; e += NT) {
            const int m = e / kSlots;
            l.xs[P * kSlots + e] = d->pop[(size_t)m * kStride + (e - m * kSlots)];  // written by init_block
        }
    } else {
        for (int e = tid; e < 4 * K; e += NT) l.zw[e] = gld(nd->wts + e);
        for (int e = tid; e < 5 * kNodePts; e += NT) l.nar[e] = gld(nd->nar + e);
        if (tid < 8) {
            sh.mid[tid] = gld(nd->nar + 5 * kNodePts + tid);
            sh.lim[tid] = gld(nd->nar + 5 * kNodePts + 8 + tid);
        }
        if (tid == 0) {
            sh.pend = gld(reinterpret_cast<const int*>(nd->nar + kNodeNarrow));
            sh.S2 = gld(nd->wts + 4 * kNodeMaxK);
        }
        const int slot = (g0 + 1) & 1;
        for (int e = tid; e < P * kSlots; e += NT) {
            const int m = e / kSlots;
            l.xs[slot * P * kSlots + e] = gld(d->pop + (size_t)m * kStride + (e - m * kSlots));
        }
        for (int m = tid; m < P; m += NT) l.fs[slot * P + m] = gld(d->fpop + m);
        for (int g = g0 - 1 - tid; g >= 0 && g >= g0 - kNodeRing; g -= NT)
            l.ring[g & (kNodeRing - 1)] = gld(d->hist + g);
    }
    if (tid < 2) sh.stop[tid] = 0;
    __syncthreads();
    if (fresh && !(sh.S2 < 1e290)) {
        // samples that are not finite (or overflow): the per-sample objective decides
        if (tid == 0) {
            d->st->done = 1;
            d->st->flags = kFlagNodeAbort;
        }
        return;
    }
    fit_run<NM>(nd, d, g0, ngen, fresh, l, sh);
}

using FitKernel = void (*)(const NodeDesc*, const BlockDesc*, int, int, int, int, int, int, int, int, int);

// members per row: the fewest that leave a wave for the bookkeeping
int members_per_row(int P) { return P <= 60 ? 1 : (P <= 120 ? 2 : 4); }
int fit_waves(int P) {
    const int nm = members_per_row(P);
    return (P + 4 * nm - 1) / (4 * nm) + 1;
}
FitKernel fit_kernel(int P) {
    switch (members_per_row(P)) {
        case 1: return k_node_fit<1>;
        case 2: return k_node_fit<2>;
        default: return k_node_fit<4>;
    }
}

// log of the largest |exp(i p(x))| on the Bernstein ellipse of parameter eta
// (half axes cosh eta and sinh eta) for a polynomial with |coefficient of x^j| <= b[j] rad
double ellipse_growth(const double* b, double eta) {
    const double s1 = std::sinh(eta), s2 = std::sinh(2 * eta), s3 = std::sinh(3 * eta), s4 = std::sinh(4 * eta);
    return b[1] * s1 + b[2] / 2 * s2 + b[3] / 4 * (s3 + 3 * s1) + b[4] / 8 * (s4 + 4 * s2);
}

// Chebyshev nodes that interpolate exp(i p(x)) (times a polynomial of degree
// `extra`) on [-1, 1] to 1e-15: error <= 4 M rho^-K / (rho - 1), M the largest
// modulus on the ellipse, rho = e^eta, for any eta; the best of a grid.
double nodes_needed(const double* b, int extra) {
    double best = 1e18;
    for (int i = 1; i <= 160; ++i) {
        const double eta = 0.025 * i;
        best = std::min(best, (std::log(4e15 / (std::exp(eta) - 1.0)) + ellipse_growth(b, eta)) / eta + extra);
    }
    return best;
}

}  // namespace

bool node_plan(const pt_block& B, double ref, int P, NodePlan* out) {
    if (P > kNodeMaxP || B.n < 64 || B.n > (int64_t)1 << 26) return false;
    const double N = (double)B.n, h = 0.5 * (N - 1.0), c = (h - ref) / h, fs = B.fs;
    NodeDesc nd{};
    const double sc[kSlots] = {1.0,
                               0.15915494309189533577,
                               h / fs,
                               h * h / (2.0 * fs * fs),
                               h * h * h / (6.0 * fs * fs * fs),
                               h / fs,
                               h * h * h * h / (24.0 * fs * fs * fs * fs)};
    double d[5] = {0, 0, 0, 0, 0};  // largest |coefficient of u^j| of delta, turns
    const int slot_of[5] = {1, 2, 3, 4, 6};
    for (int j = 0; j < kSlots; ++j) {
        nd.sc[j] = sc[j];
        const double lo = B.box.lo[j], hi = B.box.hi[j];
        nd.mid[j] = j >= 2 && j != 5 ? 0.5 * lo + 0.5 * hi : 0.0;
        if (!(std::fabs(lo) <= 1e100 && std::fabs(hi) <= 1e100)) return false;  // (squares stay finite)
    }
    for (int j = 1; j < 5; ++j) {
        const int q = slot_of[j];
        d[j] = std::max(B.box.hi[q] - nd.mid[q], nd.mid[q] - B.box.lo[q]) * sc[q];
    }
    // coefficients in x (u = x + c), of 2 delta, rad
    const double a = std::fabs(c);
    const double t[5] = {0.0, d[1] + a * (2 * d[2] + a * (3 * d[3] + 4 * a * d[4])), d[2] + a * (3 * d[3] + 6 * a * d[4]),
                         d[3] + 4 * a * d[4], d[4]};
    nd.slope = B.box.lo[5] != 0.0 || B.box.hi[5] != 0.0;
    const int extra = nd.slope ? 2 : 0;
    double b[5];
    for (int j = 0; j < 5; ++j) b[j] = 4.0 * M_PI * t[j];
    const double k = nodes_needed(b, extra);
    if (!(k <= (double)kNodeMaxK)) return false;
    nd.K = ((int)std::ceil(k) + 15) & ~15;
    if (nd.K < 16) nd.K = 16;

    // tiles: the longest (up to a workgroup's 4096 samples, or more of them for
    // long blocks, so that a block takes at most 1024 projection workgroups) in
    // which 16 nodes interpolate; bounds on the Taylor coefficients anywhere in x
    const double loc[5] = {0.0, t[1] + 2 * t[2] + 3 * t[3] + 4 * t[4], t[2] + 3 * t[3] + 6 * t[4], t[3] + 4 * t[4], t[4]};
    auto fits = [&](double samples) {
        const double tau = 0.5 * samples / h;
        double q[5] = {0, 0, 0, 0, 0};
        for (int j = 1; j < 5; ++j) q[j] = 4.0 * M_PI * loc[j] * std::pow(tau, j);
        return nodes_needed(q, extra) <= 16.0;
    };
    nd.lanes_log = 8;
    nd.runs = 1;
    while (nd.lanes_log > 0 && !fits(16.0 * (1 << nd.lanes_log))) --nd.lanes_log;
    if (nd.lanes_log < 1) return false;
    if (nd.lanes_log == 8)
        while (B.n > (int64_t)1024 * kNodeRun * nd.runs && fits(2.0 * kNodeRun * nd.runs)) nd.runs *= 2;
    const int64_t tile = (int64_t)16 * nd.runs << nd.lanes_log, wgs = (int64_t)kNodeRun * nd.runs;
    if ((B.n + tile - 1) / tile > (int64_t)1 << 20) return false;
    nd.ntile = (int)((B.n + tile - 1) / tile);
    nd.nproj = (int)((B.n + wgs - 1) / wgs);
    nd.nmom = (nd.ntile * kNodePts + kNodeGroup - 1) / kNodeGroup;

    // reference phase: f0 / fs as a double-double
    nd.r1h = nd.mid[2] / fs;
    nd.r1l = std::fma(-nd.r1h, fs, nd.mid[2]) / fs;
    nd.r2 = nd.mid[3] / (2.0 * fs * fs);
    nd.r3 = nd.mid[4] / (6.0 * fs * fs * fs);
    nd.r4 = nd.mid[6] / (24.0 * fs * fs * fs * fs);
    nd.h = h;
    nd.c = c;
    nd.su1 = N * c;                                           // sum of x + c
    nd.su2 = N * (N + 1.0) / (3.0 * (N - 1.0)) + N * c * c;  // sum of (x + c)^2
    out->nd = nd;
    out->pts_doubles = (size_t)nd.ntile * kNodePts * 4;
    out->s2_doubles = (size_t)nd.nproj;
    out->mom_doubles = (size_t)nd.nmom * nd.K * 4;
    return true;
}

size_t node_fit_lds(int P, int maxK, int chunk) {
    return fit_lds_doubles(P, maxK) * sizeof(double) + (((size_t)chunk * P * 4 + 15) & ~(size_t)15);
}

int node_chunk(int P, int maxK, int lds_max) {
    const int64_t room = (int64_t)lds_max - 1024 - (int64_t)node_fit_lds(P, maxK, 0) - 16;
    return (int)std::max<int64_t>(0, std::min<int64_t>(500, room / (4 * P)));
}

hipError_t node_setup(int lds_max) {
    const void* k[] = {reinterpret_cast<const void*>(k_node_fit<1>), reinterpret_cast<const void*>(k_node_fit<2>),
                       reinterpret_cast<const void*>(k_node_fit<4>)};
    for (const void* f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max - 1024);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t node_project(const NodeDesc* nd, const BlockDesc* bd, int nblk, int total_proj, int P, int ngen, int chunk,
                        hipStream_t s) {
    const int slices = (P * ngen + 255) / 256;
    hipLaunchKernelGGL(k_node_project, dim3((unsigned)(total_proj + nblk * slices)), dim3(256), 0, s, nd, bd, nblk,
                       total_proj, P, ngen, chunk, slices);
    return hipGetLastError();
}

hipError_t node_moments(const NodeDesc* nd, const BlockDesc* bd, int nblk, int total_mom, hipStream_t s) {
    hipLaunchKernelGGL(k_node_moments, dim3((unsigned)total_mom), dim3(256), 0, s, nd, bd, nblk);
    return hipGetLastError();
}

hipError_t node_fit(const NodeDesc* nd, const BlockDesc* bd, int nblk, int P, int maxK, int off, int ngen, int next_ngen,
                    int chunk, int flip, hipStream_t s) {
    const int nt = 64 * fit_waves(P);
    const int slices = (P * next_ngen + nt - 1) / nt;
    const FitKernel k = fit_kernel(P);
    hipLaunchKernelGGL(k, dim3((unsigned)(nblk + nblk * slices)), dim3((unsigned)nt),
                       (unsigned)node_fit_lds(P, maxK, ngen), s, nd, bd, nblk, P, maxK, off, ngen, next_ngen, chunk, flip,
                       slices > 0 ? slices : 1);
    return hipGetLastError();
}

}  // namespace pt
