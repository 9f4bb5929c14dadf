// nodes.hip -- kernels and plan of the node-weight fits (see nodes.h).
#define PT_INSTANCE_TU  // kernels.h: device functions only
#include "nodes.h"

#include <algorithm>
#include <array>
#include <cmath>

#include "kernels.h"

// Every operation here rounds as written: a fit runs the same objective through
// several inlined copies (full and re-expanded sets, first and later
// generations), which must agree bit for bit, and a sum over lanes must come
// out the same in all of them (a product fused into its first step would not).
#pragma clang fp contract(off)

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

// DPP move of a double.
template <int CTRL>
__device__ __forceinline__ double lane_move(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false));
}

// Lane J of each octet (lanes 8 q .. 8 q + 7), in every lane of the octet: a
// broadcast over the row of 16, then over its upper half.
template <int J>
__device__ __forceinline__ double oct_bcast(double v) {
    const long long x = __double_as_longlong(v);
    long long a = __builtin_amdgcn_mov_dpp(x, 0x150 + J, 0xF, 0xF, false);
    a = __builtin_amdgcn_update_dpp(a, x, 0x158 + J, 0xF, 0xC, false);
    return __longlong_as_double(a);
}

// Sum over the octet, in every lane of it (pairs, quads, the two quads).
__device__ __forceinline__ double oct_sum(double v) {
    v += lane_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += lane_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += lane_move<0x141>(v);  // row_half_mirror
    return v;
}

// Barrier that orders LDS only: a wave does not wait for its global stores (the
// history's) to be acknowledged, which takes longer than a generation.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
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

// Packed draws of one member: the byte offsets of rows r1, r2 and r3 in 16 bits
// each, then the slots the binomial crossover takes from the mutant.
__device__ __forceinline__ uint64_t node_pack(const BlockDesc* d, const Draws& w) {
    uint32_t m = 0;
    for (int a = 0; a < d->D; ++a)
        if ((w.cross >> a) & 1u) m |= 1u << d->act[a];
    constexpr int kRow = kStride * sizeof(double);
    static_assert(kNodeMaxP * kRow <= 65536, "row offsets fit 16 bits");
    return (uint64_t)((uint32_t)(w.r1 * kRow) | ((uint32_t)(w.r2 * kRow) << 16)) |
           ((uint64_t)((uint32_t)(w.r3 * kRow) | (m << 16)) << 32);
}

// The draws of generations g_off .. g_off + ngen - 1 of every member, by
// workgroups beside the kernel's own work: they depend on nothing but the
// stream, so they are kept off the fit's chain of generations (three Philox
// calls cost as much as a whole evaluation there).  Order: per 16 generations
// (from a multiple of 16 on), per wave and member of its octets, generation,
// octet -- 1 KB that a wave of the fit reads with one load.
__device__ __forceinline__ void node_draws(const NodeDesc* nd, const BlockDesc* bd, int slice, int slices, int P, int g_off,
                                           int ngen, int chunk, int flip) {
    const int b = slice / slices, id = (slice - b * slices) * (int)blockDim.x + (int)threadIdx.x;
    const int nm = node_nm(P), W = node_waves(P), part = id >> 7;
    const NodeDesc* n = nd + b;
    const BlockDesc* d = bd + b;
    const int g0 = n->g0 + g_off, g = (g0 & ~15) + 16 * (part / (nm * W)) + ((id >> 3) & 15), wt = part % (nm * W);
    if (g < g0 || g >= g0 + ngen) return;
    const int i = min(8 * (wt / nm) + (id & 7) + 8 * W * (wt % nm), P - 1);
    const Draws w = trial_draws(d, i, (uint32_t)g);
    n->draws[((n->parity + flip) & 1) * node_draw_words(P, chunk) + id] = node_pack(d, w);
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
                                                      int nblk) {
    __shared__ double tab[64], red[260];
    const int wg = blockIdx.x;
    const int b = node_block_of(nds, nblk, wg, false);
    const NodeDesc* nd = nds + b;
    const BlockDesc* d = bds + b;
    if (d->dtype == PT_F64)
        project_unit<double>(nd, d, wg - nd->proj_begin, tab, red);
    else
        project_unit<float>(nd, d, wg - nd->proj_begin, tab, red);
}

// ---------------------------------------------------------------------------
// Moments: sum over 128 points of value x T_j(x_point) for 64 of the K values of
// j; a lane holds one j, the waves share the points (all K values in one workgroup
// took 8 to 13 us for 144 to 256 nodes, 5 apart).  Workgroups past `total` make the draws of
// the fit's first launch (here rather than beside the projection, whose registers
// allow two waves on a SIMD: 64 blocks' draws of 1500 generations, 3.8e6 of them,
// 58 us there, 41 here).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_node_moments(const NodeDesc* __restrict__ nds, const BlockDesc* __restrict__ bds,
                                                      int nblk, int total, int P, int ngen, int chunk, int slices) {
    __shared__ double th[kNodeGroup], v[kNodeGroup][4], red[4][64][4];
    if ((int)blockIdx.x >= total) {
        node_draws(nds, bds, blockIdx.x - total, slices, P, 0, ngen, chunk, 0);
        return;
    }
    const int b = node_block_of(nds, nblk, blockIdx.x, true);
    const NodeDesc* nd = nds + b;
    const BlockDesc* d = bds + b;
    const int K = nd->K, parts = (K + 63) >> 6, at = blockIdx.x - nd->mom_begin, wg = at / parts, j0 = (at - wg * parts) * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
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
        gst(nd->mom + ((size_t)wg * K + j0 + jl) * 4 + q, (red[0][jl][q] + red[1][jl][q]) + (red[2][jl][q] + red[3][jl][q]));
}

// ---------------------------------------------------------------------------
// The fit: one workgroup per block runs `ngen` generations.
//
// Member m belongs to an octet of lanes (waves 0 .. W - 1, eight octets each, NM
// members per octet): lane j < 7 holds the member's slot j, builds its trial
// coordinate from the rows of the previous generation in LDS and turns it into
// a coefficient of delta; all eight lanes then evaluate delta, exp(i delta) and
// the weighted sums at the nodes k = lane, lane + 8, ... and add up by DPP
// moves, so selection needs no exchange between octets.  One barrier per
// generation separates writing the selected rows from reading them (two copies
// alternate).  Wave W keeps the books one generation behind: best member,
// history, stop rule.
//
// What bounds it: a generation is a chain of dependent operations (an LDS round
// trip, about forty FP64 operations, the barrier), which a wave alone on its
// SIMD issues at five to six cycles an instruction and two on one SIMD at four
// each.  So the fewest instructions a wave needs and the fewest waves a SIMD
// holds pull against each other; measured for P = 40: 16 lanes a member (ten
// waves) 0.99 us a generation, 8 lanes (five) 0.45, 4 lanes (three) 0.54; 8 lanes
// with the bound rule and the stop flag off the chain where they can be 0.41, with
// what waits for a multiple of 8 out of the loop 0.35, two a turn of it 0.34 (P = 64 0.38,
// 120 0.58, 240 1.17).  The draws pass through LDS 16 generations at a time, so a launch runs
// as many generations as there are; while all of a launch's lay there, a fit of
// 2000 generations took five launches, each ~14 us for its start.
//
// As the population draws together fewer nodes do: every 16th generation the
// bookkeeping wave measures its spread, and when markedly fewer nodes would
// carry any trial it asks for the weights to be re-expanded about the best
// member's phase (relevel), first on any smaller number of nodes, at last on 16
// and then 8 (kinds 1 and 2), which each lane holds in registers, two or one a
// lane; there the phase difference needs no reduction and a shorter sine and
// cosine do.  A trial outside the limits of the re-expansion is evaluated on
// the full set.
//
// The step of Table 4 (selection, random draws, bound rule, stop rule) is that
// of de_step_body.
// ---------------------------------------------------------------------------
constexpr int kRowD = kStride;  // doubles of a member's row in LDS: seven slots, then its objective

// draws of a wave and member of its octets in LDS: 32 generations of eight, then
// the first again (a stretch of eight reads one past its end without a wrap)
constexpr int kDrawRing = 33 * 8;

struct FitLds {
    double *xs;        // two generations of P rows
    double *zw, *un;   // full node set: -2 Z and W (4 doubles a node), u
    double *lz, *lu;   // re-expanded set
    double *tab, *tl;  // cos_table of both
    double *scr;       // 4 doubles a node
    double *ring;      // best-so-far values
    uint64_t* dr;      // draws: 32 generations per wave and member of its octets
};

// largest re-expanded set, for a full set of K nodes
__host__ __device__ inline int level_cap(int K) { return K <= 2 * kNodePts ? kNodePts : K / 8 * 5; }

__host__ __device__ inline size_t fit_lds_doubles(int P, int maxK) {
    return (size_t)2 * P * kRowD + 11 * (size_t)maxK + 7 * (size_t)level_cap(maxK) + 2 + kNodeRing +
           (size_t)kDrawRing * node_nm(P) * node_waves(P);
}

__device__ __forceinline__ FitLds fit_lds(double* base, int P, int maxK) {
    FitLds l;
    l.xs = base;
    l.zw = l.xs + 2 * P * kRowD;
    l.scr = l.zw + 4 * maxK;
    l.lz = l.scr + 4 * maxK;
    l.un = l.lz + 4 * level_cap(maxK);
    l.lu = l.un + maxK;
    l.tab = l.lu + level_cap(maxK);
    l.tl = l.tab + 2 * maxK + 1;
    l.ring = l.tl + 2 * level_cap(maxK) + 1;
    l.dr = reinterpret_cast<uint64_t*>(l.ring + kNodeRing);
    return l;
}

// A re-expanded node set.
struct Level {
    double mid[8], lim[8];  // per slot: centre, and the distance a trial may lie from it
    int K, kind;            // nodes (0: none yet, the full set); kind 1, 2: 16 or 8 in registers
    int pend;               // generation before which it takes effect, -1: in effect
    int pad;
};

struct FitShared {
    Level lev, next;  // in effect, and asked for (next.pend >= 0)
    double S2, best_f;
    int stop[2];      // DeState flags of a stop, by generation parity
    int best, stop_gen;
    int abandoned;    // generation after which the fit was abandoned, kNeverGen: not
};
constexpr int kNeverGen = 0x7fffffff;

// Whether waves on the smallest set (kind 2) look for a stop in every generation.
// A fit of a fixed number of generations is stopped there by nothing but its
// abandonment, unless the launch (its last generation g1 - 1) reaches past its end;
// its waves look for that every kAbandonLook generations, and leave together there
// (every 8th cost 0.7 % of a fit of 2000: an LDS read on the chain).
constexpr int kAbandonLook = 64;
__device__ __forceinline__ bool stops_anywhere(const BlockDesc* d, int g1) {
    return (d->rel_tol > 0.0 && d->window > 0) || d->vtr > -__builtin_inf() || g1 - 1 > d->max_gens;
}

// Coefficients of one candidate's phase difference (turns, in u) and its
// amplitude A + B u.
struct NodeCand {
    double p0, p1, p2, p3, p4, A, B;
};

template <bool SLOPE, bool QUART>
__device__ __forceinline__ NodeCand node_cand(double dj) {
    NodeCand q;
    q.p3 = oct_bcast<4>(dj);
    q.p4 = QUART ? oct_bcast<6>(dj) : 0.0;
    q.p2 = oct_bcast<3>(dj);
    q.p1 = oct_bcast<2>(dj);
    q.p0 = oct_bcast<1>(dj);
    q.A = oct_bcast<0>(dj);
    q.B = SLOPE ? oct_bcast<5>(dj) : 0.0;
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
template <bool SLOPE, bool COR>
__device__ __forceinline__ void node_terms(const NodeCand& q, double u, double c, double s, double zr, double zi,
                                           double wr, double wi, double& a1, double& a2) {
    if constexpr (SLOPE) {
        const double amp = __fma_rn(q.B, u, q.A);
        a1 = __fma_rn(amp, __fma_rn(zr, c, -(zi * s)), a1);
        if constexpr (!COR) a2 = __fma_rn(amp * amp, __fma_rn(-2.0 * s, __fma_rn(wr, s, wi * c), wr), a2);
    } else {
        a1 = __fma_rn(zr, c, __fma_rn(-zi, s, a1));
        if constexpr (!COR) a2 = __fma_rn(s, __fma_rn(wr, s, wi * c), a2);
    }
}

// Correlation objective, Eq. (2-2-5): F = 1 / (arctan(C) + pi/2), of f = -C.
__device__ __noinline__ double cor_value(double f) { return 1.0 / (atan(-f) + 1.5707963267948966192); }

// Objective from an octet's sums; en: half of (N + sum Wr).  COR: -C, which
// rises and falls with F: members are compared by it, and F is formed where a
// value leaves the generations (an arctangent and a division in each cost 0.25 of
// 0.60 us; F itself cannot tell apart correlations closer than ~1e-10 relative).
template <bool SLOPE, bool COR>
__device__ __forceinline__ double node_objective(const NodeDesc* nd, const NodeCand& q, double a1, double a2, double S2,
                                                 double en, double N) {
    if constexpr (COR) return 0.5 * oct_sum(SLOPE ? a1 : q.A * a1);
    const double v = oct_sum(SLOPE ? __fma_rn(0.5, a2, a1) : q.A * __fma_rn(-q.A, a2, a1));
    // half the energy of the amplitude (with the constant part of cos 2 phi's sum)
    if constexpr (SLOPE)
        return __fma_rn(0.5, __fma_rn(q.B * q.B, nd->su2, __fma_rn(2.0 * q.A * q.B, nd->su1, q.A * q.A * N)), S2) + v;
    return __fma_rn(q.A * q.A, en, S2) + v;
}

// Sums over a node set in LDS for one candidate (the octet's lanes share
// the nodes; n a multiple of 8): two nodes at a time, the next two on their way.
template <bool SLOPE, bool QUART, bool COR>
__device__ __forceinline__ void lds_sums(const NodeCand& q, const double* zw, const double* un, int l8, int n, double& a1,
                                         double& a2) {
    struct Node {
        double u, zr, zi, wr, wi;
    };
    auto load = [&](int k) { return Node{un[k], zw[4 * k], zw[4 * k + 1], zw[4 * k + 2], zw[4 * k + 3]}; };
    auto term = [&](const Node& t) {
        double r = node_delta<QUART>(q, t.u);
        r -= rint(r);
        double c, s;
        sincos_turns64(r, c, s);
        node_terms<SLOPE, COR>(q, t.u, c, s, t.zr, t.zi, t.wr, t.wi, a1, a2);
    };
    Node a = load(l8), b = load(l8 + 8 < n ? l8 + 8 : l8);
    int k = l8;
#pragma unroll 2
    for (; k + 8 < n; k += 16) {
        const int k2 = k + 16 < n ? k + 16 : k, k3 = k + 24 < n ? k + 24 : k;
        const Node c = load(k2), d = load(k3);
        term(a);
        term(b);
        a = c;
        b = d;
    }
    if (k < n) term(a);
}

// Half of (N + sum of Wr), the constant part of the energy, over the wave.
__device__ __forceinline__ double node_energy(const double* zw, int n, double N) {
    double v[1] = {0.0};
    for (int k = threadIdx.x & 63; k < n; k += 64) v[0] += zw[4 * k + 2];
    wave_sums(v);
    return 0.5 * (N + v[0]);
}

// cos(2 pi i / 4n), i = 0 .. 2n, by the whole workgroup.  The sums between moments
// and nodes take T_j(x_k) = cos(2 pi j (2k + 1) / 4n) from it: an index kept
// modulo 4n and one LDS read instead of a reduction and a polynomial for each (with
// these, and the outputs spread over all octets, a fit's re-expansions and the
// weights from their moments take 20 to 30 us less of 280 for 4096 samples, 100 of
// 1410 for the quartic block).
__device__ __forceinline__ void cos_table(double* tab, int n) {
    const double inv = 0.25 / (double)n;
    for (int i = threadIdx.x; i <= 2 * n; i += blockDim.x) {
        const double r = (double)i * inv;
        tab[i] = cos_turns64(r * r);
    }
}
// a mod n, 0 <= a < 2^23
__device__ __forceinline__ int mod_of(int a, int n, float inv) {
    int r = a - (int)((float)a * inv) * n;
    r += r < 0 ? n : 0;
    return r - (r >= n ? n : 0);
}

// Values at n nodes from n moments (4 doubles each), times `scale`: an octet of
// lanes per pair of nodes k and n - 1 - k, whose sums share their even and odd
// terms (a lane's terms are all even or all odd).  out(node, component, value).
template <typename Out>
__device__ __forceinline__ void node_values(const double* tab, const double* mom, int n, double scale, Out out) {
    const int tid = threadIdx.x, l8 = tid & 7, n4 = 4 * n;
    const float inv = 1.0f / (float)n4;
    for (int k = tid >> 3; k < n >> 1; k += blockDim.x >> 3) {
        int m = mod_of(l8 * (2 * k + 1), n4, inv);
        const int st = mod_of(8 * (2 * k + 1), n4, inv);
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int j = l8; j < n; j += 8) {
            const double t = j ? tab[min(m, n4 - m)] : 0.5;
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = __fma_rn(t, mom[4 * j + e], a[e]);
            m += st;
            m -= m >= n4 ? n4 : 0;
        }
        double p[4], q[4];  // even + odd terms: node k; even - odd: node n - 1 - k
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double v = a[e] + lane_move<0x4E>(a[e]);  // quad_perm [2, 3, 0, 1]
            const double o = lane_move<0xB1>(v);            // quad_perm [1, 0, 3, 2]
            p[e] = v + o;
            q[e] = l8 & 1 ? o - v : v - o;
            p[e] += lane_move<0x141>(p[e]);  // row_half_mirror
            q[e] += lane_move<0x141>(q[e]);
        }
        const int e = l8 & 3;
        const double pe = e == 0 ? p[0] : e == 1 ? p[1] : e == 2 ? p[2] : p[3];
        const double qe = e == 0 ? q[0] : e == 1 ? q[1] : e == 2 ? q[2] : q[3];
        out(l8 < 4 ? k : n - 1 - k, e, (l8 < 4 ? pe : qe) * scale);
    }
}

// The set asked for in sh.next, by the whole workgroup: Z exp(i d), W exp(2 i d)
// (d: the delta of the member at its centre) as Chebyshev moments over the full
// nodes, then values at the new nodes.
__device__ __noinline__ void relevel(const NodeDesc* nd, const FitLds& l, FitShared& sh) {
    const int tid = threadIdx.x, NT = blockDim.x, K = nd->K, n = sh.next.K, l8 = tid & 7;
    const NodeCand q{sh.next.mid[1] * nd->sc[1],
                     (sh.next.mid[2] - nd->mid[2]) * nd->sc[2],
                     (sh.next.mid[3] - nd->mid[3]) * nd->sc[3],
                     (sh.next.mid[4] - nd->mid[4]) * nd->sc[4],
                     (sh.next.mid[6] - nd->mid[6]) * nd->sc[6],
                     0.0,
                     0.0};
    auto turned = [&](int k, double* o) {
        double r = node_delta<true>(q, l.un[k]);
        r -= rint(r);
        double c, s;
        sincos_turns64(r, c, s);
        const double zr = l.zw[4 * k], zi = l.zw[4 * k + 1], wr = l.zw[4 * k + 2], wi = l.zw[4 * k + 3];
        const double c2 = __fma_rn(c, c, -(s * s)), s2 = 2.0 * c * s;
        o[0] = __fma_rn(zr, c, -(zi * s));
        o[1] = __fma_rn(zr, s, zi * c);
        o[2] = __fma_rn(wr, c2, -(wi * s2));
        o[3] = __fma_rn(wr, s2, wi * c2);
    };
    // sums and differences of nodes k and K - 1 - k: all that the even and the odd
    // moments need
    for (int k = tid; k < K >> 1; k += NT) {
        double a[4], b[4];
        turned(k, a);
        turned(K - 1 - k, b);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            l.scr[4 * k + e] = a[e] + b[e];
            l.scr[4 * (K - 1 - k) + e] = a[e] - b[e];
        }
    }
    cos_table(l.tl, n);
    __syncthreads();
    const int K4 = 4 * K;
    const float inv = 1.0f / (float)K4;
    for (int j = tid >> 3; j < n; j += NT >> 3) {
        int m = mod_of(j * (2 * l8 + 1), K4, inv), at = j & 1 ? K - 1 - l8 : l8;
        const int st = mod_of(16 * j, K4, inv), dir = j & 1 ? -8 : 8;
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int k = l8; k < K >> 1; k += 8) {
            const double t = l.tab[min(m, K4 - m)];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = __fma_rn(t, l.scr[4 * at + e], a[e]);
            at += dir;
            m += st;
            m -= m >= K4 ? K4 : 0;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = oct_sum(a[e]);
        if (l8 < 4) l.lz[4 * j + l8] = l8 == 0 ? a[0] : l8 == 1 ? a[1] : l8 == 2 ? a[2] : a[3];
    }
    __syncthreads();
    node_values(l.tl, l.lz, n, 2.0 / (double)n, [&](int k, int e, double v) { l.scr[4 * k + e] = v; });
    for (int k = tid; k < n; k += NT) l.lu[k] = l.tl[2 * k + 1] + nd->c;
    __syncthreads();
    for (int e = tid; e < 4 * n; e += NT) l.lz[e] = l.scr[e];
    if (tid == 0) {
        sh.lev = sh.next;
        sh.lev.pend = -1;
        sh.next.pend = -1;
    }
    __syncthreads();
}

// Growth of exp(i p) off [-1, 1]: log of its largest modulus on the ellipse of
// sum of half axes e^eta, for |coefficients| <= b1 .. b4 of x .. x^4 (rad).
__host__ __device__ inline double ellipse_growth(double b1, double b2, double b3, double b4, double eta) {
    const double e = exp(eta), f = 1.0 / e, s1 = 0.5 * (e - f), c1 = 0.5 * (e + f);
    const double s2 = 2.0 * s1 * c1, s3 = s1 * (3.0 + 4.0 * s1 * s1), s4 = 2.0 * s2 * (1.0 + 2.0 * s1 * s1);
    return b1 * s1 + 0.5 * b2 * s2 + 0.25 * b3 * (s3 + 3.0 * s1) + 0.125 * b4 * (s4 + 4.0 * s2);
}

// 1 / v to a part in 1e15 (v normal): for limits and node counts only.
__device__ __forceinline__ double near_rcp(double v) {
    const double r = __builtin_amdgcn_rcp(v), e = __fma_rn(-v, r, 1.0);
    const double s = __fma_rn(r, e, r);
    return __fma_rn(s, __fma_rn(-v, s, 1.0), s);
}

// Whether a smaller node set would carry the population: by one wave, a lane per
// ellipse.  What depends on neither population nor generation is worked out once
// per launch and the eight slots are reduced side by side: all waves wait for a
// look, every 16th generation until the smallest set is in use, and it took 1.4 us
// longer with the exponentials, logarithms and one reduction after the other.
struct LevelRule {
    double eta, reta, at0, g[4];  // the lane's ellipse (nodes_needed)
    double sc, c;                 // scale of the lane's slot (lane & 7); centre
    int K, extra;

    __device__ __forceinline__ void init(const NodeDesc* nd) {
        const int lane = threadIdx.x & 63, j = lane & 7;
        eta = 0.1 * (double)(lane + 1);
        reta = 1.0 / eta;
        at0 = log(4e15 / (exp(eta) - 1.0));
        g[0] = ellipse_growth(1.0, 0.0, 0.0, 0.0, eta);
        g[1] = ellipse_growth(0.0, 1.0, 0.0, 0.0, eta);
        g[2] = ellipse_growth(0.0, 0.0, 1.0, 0.0, eta);
        g[3] = ellipse_growth(0.0, 0.0, 0.0, 1.0, eta);
        sc = j < kSlots ? gld(&nd->sc[j]) : 0.0;
        c = fabs(nd->c);
        K = nd->K;
        extra = nd->slope ? 2 : 0;
    }
    // after generation gen, whose best member is `best`
    __device__ __forceinline__ void look(const FitLds& l, FitShared& sh, int P, double F, int gen, int best) const {
        const int lane = threadIdx.x & 63, j = lane & 7;
        const double* x = l.xs + (gen & 1) * P * kRowD;
        // largest distance of a member from the best one in the lane's slot (eight
        // lanes share a slot's members), with room for a mutant x1 + F (x2 - x3) of
        // such members (half as much again makes the sets shrink later: 1 to 2.5 % of
        // a fit)
        const double xb = x[best * kRowD + j];
        double a = 0.0;
        for (int m = lane >> 3; m < P; m += 8) a = fmax(a, fabs(x[m * kRowD + j] - xb));
        a = fmax(a, lane_move<0x128>(a));  // row_ror:8
        a = rows_extreme<true>(a);
        const double rng = (1.0 + 2.0 * F) * a, turns = rng * sc;
        auto of = [&](int slot) {
            return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(turns), slot),
                                    __builtin_amdgcn_readlane(__double2loint(turns), slot));
        };
        const double q0 = of(1), q1 = of(2), q2 = of(3), q3 = of(4), q4 = of(6);
        // coefficients in x (u = x + c), of 2 delta, rad
        const double w = 1.0 + c, pi4 = 12.566370614359172;
        const double b1 = pi4 * (q1 + c * (2.0 * q2 + c * (3.0 * q3 + 4.0 * c * q4)));
        const double b2 = pi4 * (q2 + c * (3.0 * q3 + 6.0 * c * q4)), b3 = pi4 * (q3 + 4.0 * c * q4), b4 = pi4 * q4;
        const double rsum = near_rcp(q0 + w * (q1 + w * (q2 + w * (q3 + w * q4))) + 1e-300);  // 1 / largest |delta|
        // the distances scaled up as far as 8 or 16 nodes allow (their bound is
        // linear in the coefficients at a fixed ellipse: the best of the wave's
        // ellipses) and delta stays within the polynomials' range
        const double slope = (b1 * g[0] + b2 * g[1]) + (b3 * g[2] + b4 * g[3]), rs = near_rcp(slope + 1e-300);
        const double s8 = fmin(wave_extreme<true>(((8 - extra) * eta - at0) * rs), kNodeTurns8 * rsum);
        const double s16 = fmin(wave_extreme<true>(((16 - extra) * eta - at0) * rs), kNodeTurns16 * rsum);
        const double need = wave_extreme<false>((at0 + slope) * reta + extra);
        int n = 0, kind = 0;
        double scale = 1.0;
        if (s8 >= 1.0) {
            n = 8;
            kind = 2;
            scale = s8;
        } else if (s16 >= 1.0) {
            n = 16;
            kind = 1;
            scale = s16;
        } else if (need <= (double)kNodeMaxK) {
            n = ((int)ceil(need) + 7) & ~7;
        }
        // worth it for fewer than five eighths of the nodes
        const int cur = sh.lev.K ? sh.lev.K : K;
        if (n == 0 || (kind ? kind <= sh.lev.kind : 8 * n > 5 * cur) || n > level_cap(K)) return;
        if (lane < kSlots) {
            const bool amp = j == 0 || j == 5;
            sh.next.mid[j] = amp ? 0.0 : xb;
            sh.next.lim[j] = amp ? __builtin_inf() : rng * fmin(scale, 1e9);  // (finite: rng may be 0)
        }
        if (lane == 0) {
            sh.next.K = n;
            sh.next.kind = kind;
            sh.next.pend = gen + 2;
        }
    }
};

// The bookkeeping of each generation, by one wave: best objective, history, stop
// rule, and every 16th generation a look at the node set.  It runs one
// generation behind the members and must stay shorter than one of theirs:
// what it needs every time is in registers (the flags it sets itself among
// them), the best member's index is looked up only when something needs it, and
// fits without a window rule run without its branches (with all of these in LDS
// and in branches it took 1050 of a generation's 1190 cycles).
// NV: values per lane (P <= 64 NV).
template <int NV, bool WINDOW>
struct Book {
    const NodeDesc* nd;
    const BlockDesc* blk;
    const FitLds& l;
    FitShared& sh;
    int P, lane, win, max_gens, kind, pend;
    double vtr, rel_tol, floor, F, bf, low;  // low: the best member's comparison value, bf: its objective
    bool cor;
    double* hist;
    LevelRule rule;

    __device__ __forceinline__ Book(const NodeDesc* nd_, const BlockDesc* d, const FitLds& l_, FitShared& sh_)
        : nd(nd_), blk(d), l(l_), sh(sh_) {
        P = d->P;
        lane = threadIdx.x & 63;
        win = d->window;
        max_gens = d->max_gens;
        vtr = d->vtr;
        rel_tol = d->rel_tol;
        floor = d->objective == 0 ? nd_->cancel * sh.S2 : -__builtin_inf();
        F = d->F;
        hist = d->hist;
        kind = __builtin_amdgcn_readfirstlane(sh.lev.kind);
        pend = __builtin_amdgcn_readfirstlane(sh.next.pend);
        bf = low = __builtin_inf();
        cor = d->objective != 0;
        if (kind < 2) rule.init(nd);
    }
    // (lanes past the population repeat its last member)
    __device__ __forceinline__ double value(int g, int t) const {
        return l.xs[(g & 1) * P * kRowD + min(lane + 64 * t, P - 1) * kRowD + kSlots];
    }
    // lowest index of the members of generation g that have the best value
    __device__ __forceinline__ int best_of(int g) const {
        int best = 0;
#pragma unroll
        for (int t = NV - 1; t >= 0; --t) {
            const unsigned long long hit = __ballot(lane + 64 * t < P && value(g, t) == low);
            if (hit) best = 64 * t + __ffsll(hit) - 1;
        }
        return best;
    }
    // flags of the stop after generation g, 0: none
    __device__ __forceinline__ int step(int g, bool last) {
        double f = value(g, 0);
#pragma unroll
        for (int t = 1; t < NV; ++t) {
            const double v = value(g, t);
            f = v < f ? v : f;
        }
        // objectives only fall, so the best changes only when one lies below it
        // (seldom, once the population has drawn together)
        if (__ballot(f < low)) {
            low = wave_extreme<false>(f);
            bf = cor ? cor_value(low) : low;
        }
        int flags = bf <= vtr ? 4 : 0;  // PT_FLAG_VTR
        if constexpr (WINDOW) {
            if (g >= win) {
                const double old = win < kNodeRing ? l.ring[(g - win) & (kNodeRing - 1)] : gld(hist + (g - win));
                if (old - bf <= rel_tol * bf) flags |= 1;  // PT_FLAG_CONVERGED
            }
            if (lane == 0) l.ring[g & (kNodeRing - 1)] = bf;
        }
        if (!flags && g >= max_gens) flags = 2;  // PT_FLAG_MAXGEN
        if (!(bf >= floor)) flags = kFlagNodeAbort;
        if (lane == 0) {
            gst(hist + g, bf);
            sh.stop[g & 1] = flags;
            if (flags == kFlagNodeAbort) sh.abandoned = g;
        }
        flags = __builtin_amdgcn_readfirstlane(flags);
        const bool look = (g & 15) == 14 && kind < 2 && pend < 0;  // takes effect at a multiple of 16
        if (__builtin_expect(flags || last || look, 0)) {
            const int best = best_of(g);
            if (lane == 0) {
                sh.best = best;
                sh.best_f = bf;
                sh.stop_gen = g;
            }
            if (look && !flags) {
                rule.look(l, sh, P, F, g, best);
                pend = __builtin_amdgcn_readfirstlane(sh.next.pend);
            }
        }
        return flags;
    }
    // the members' barriers, one generation behind them, and the last
    // generation's books.  This wave leaves where the members do: two generations
    // after a stop, or at the next multiple of kAbandonLook where they look no more often.
    __device__ __forceinline__ int run(int g0, int g1) {
        const bool stops = stops_anywhere(blk, g1);
        int f2 = 0, f1 = 0;  // flags of generations g - 2 and g - 1; kept after a stop
        asm volatile(".p2align 6, , 60");  // (as the members' loop)
        for (int g = g0; g < g1; ++g) {
            if (pend == g) {
                relevel(nd, l, sh);
                pend = -1;
                kind = __builtin_amdgcn_readfirstlane(sh.lev.kind);
            }
            if (f2) {
                if (stops || kind < 2 || !(g & (kAbandonLook - 1))) return g;
            } else if (g > g0) {
                f1 = step(g - 1, false);
            }
            lds_barrier();
            f2 = f1;
        }
        if (!f2) step(g1 - 1, true);
        return g1;
    }
};

// The generations of the members' waves.  A stop after generation g is found
// while g + 1 runs and seen by every wave while it works on g + 2, before it
// writes anything (where the flag's LDS read costs nothing): g + 2 is returned.
// g1: the launch's generations are done.  On the smallest set of a fit that only
// its abandonment can stop, that is looked for seldom (stops_anywhere).
template <int NM, bool SLOPE, bool QUART, bool COR>
struct Members {
    const NodeDesc* nd;
    const FitLds& l;
    FitShared& sh;
    int g0, g1, P, K, l8;
    bool slot, stops;  // the lane holds a slot; a stop rule is on
    double N, S2, F, lo, hi, mid_w, sc, en_w;
    int m[NM];         // members (an octet past the population repeats its last member)
    double xi[NM], fo[NM];
    const uint64_t* src;  // the wave's draws: next block of 16 generations, this lane's 16 bytes
    uint64_t pre[NM][2];  // on their way
    uint64_t* ring;       // and their places in LDS

    __device__ __forceinline__ Members(const NodeDesc* nd_, const BlockDesc* d, int g0_, int g1_, bool fresh,
                                       const uint64_t* draws, const FitLds& l_, FitShared& sh_)
        : nd(nd_), l(l_), sh(sh_), g0(g0_), g1(g1_) {
        const int tid = threadIdx.x;
        P = d->P;
        K = nd->K;
        N = (double)d->n;
        S2 = sh.S2;
        F = d->F;
        l8 = tid & 7;
        // constants of the slot this lane holds (lane 7: the objective's place)
        slot = l8 < kSlots;
        const int j = slot ? l8 : kSlots - 1;
        lo = gld(&d->lo[j]);
        hi = gld(&d->hi[j]);
        mid_w = slot ? gld(&nd->mid[j]) : 0.0;
        sc = slot ? gld(&nd->sc[j]) : 0.0;
        en_w = node_energy(l.zw, K, N);
        stops = stops_anywhere(d, g1);
        const double* x = l.xs + ((g0 + 1) & 1) * P * kRowD;
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            m[t] = min((tid >> 3) + t * 8 * waves(), P - 1);
            xi[t] = slot ? x[m[t] * kRowD + l8] : 0.0;
            fo[t] = fresh ? __builtin_inf() : x[m[t] * kRowD + kSlots];
        }
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        src = draws + wave * NM * 128 + 2 * lane;
        ring = l.dr + wave * NM * kDrawRing;
        fetch();
        put(g0 >> 4);
        if (g0 & 15) {
            if ((g0 | 15) + 1 < g1) fetch();
            if (g0 & 8) put((g0 >> 4) + 1);
        }
    }
    __device__ __forceinline__ static int waves() { return (int)(blockDim.x >> 6) - 1; }
    // The draws come 16 generations at a time, a block ahead: loaded when one
    // begins, put into LDS when half of it is over (by the wave that reads them).
    __device__ __forceinline__ void fetch() {
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            typedef uint64_t pair_t __attribute__((ext_vector_type(2)));
            const pair_t v = *(const PT_GLOBAL pair_t*)(src + t * 128);
            pre[t][0] = v.x;
            pre[t][1] = v.y;
        }
        src += waves() * NM * 128;
    }
    __device__ __forceinline__ void put(int block) {
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            const int lane = threadIdx.x & 63;
            uint64_t* o = ring + t * kDrawRing + (block & 1) * 128 + 2 * lane;
            o[0] = pre[t][0];
            o[1] = pre[t][1];
            if (!(block & 1) && lane < 4) {
                o[256] = pre[t][0];
                o[257] = pre[t][1];
            }
        }
    }
    // at multiples of 8
    __device__ __forceinline__ void feed(int g) {
        if (g & 8)
            put((g >> 4) + 1);
        else if (g + 16 < g1)
            fetch();
    }
    __device__ __forceinline__ uint64_t draw(int t, int g) const {
        return draws(g)[t * kDrawRing];
    }
    __device__ __forceinline__ const uint64_t* draws(int g) const {
        return ring + (g & 31) * 8 + ((threadIdx.x >> 3) & 7);
    }

    // this lane's column of the rows that generation g reads
    __device__ __forceinline__ const char* column(int g) const {
        return reinterpret_cast<const char*>(l.xs + ((g + 1) & 1) * P * kRowD + l8);
    }
    // mutant coordinate v of draws w and its base x1: apply_trial's arithmetic
    __device__ __forceinline__ void mutant(const char* x, uint64_t w, double& v, double& x1) const {
        const uint32_t a = (uint32_t)w, b = (uint32_t)(w >> 32);
        x1 = *reinterpret_cast<const double*>(x + (a & 0xFFFFu));
        const double x2 = *reinterpret_cast<const double*>(x + (a >> 16));
        const double x3 = *reinterpret_cast<const double*>(x + (b & 0xFFFFu));
        v = __fma_rn(F, x2 - x3, x1);
    }
    __device__ __forceinline__ bool crossed(uint64_t w) const { return (uint32_t)(w >> 48) >> l8 & 1u; }
    // the bound rule (a mutant put half-way to one bound lies inside the other)
    __device__ __forceinline__ double bounded(double v, double x1) const {
        double vl = (lo + x1) * 0.5, vh = (hi + x1) * 0.5;
        asm volatile("" : "+v"(vl), "+v"(vh));  // (selects, not branches around a sum and a product)
        return v < lo ? vl : (v > hi ? vh : v);
    }
    __device__ __forceinline__ double full(double y) const {
        const NodeCand q = node_cand<SLOPE, QUART>((y - mid_w) * sc);
        double a1 = 0.0, a2 = 0.0;
        lds_sums<SLOPE, QUART, COR>(q, l.zw, l.un, l8, K, a1, a2);
        return node_objective<SLOPE, COR>(nd, q, a1, a2, S2, en_w, N);
    }
    __device__ __forceinline__ void keep(int t, char* x, double y, double ft) {
        const bool take = ft <= fo[t];
        xi[t] = take ? y : xi[t];
        fo[t] = take ? ft : fo[t];
        // (octets that repeat the last member write the same values)
        *reinterpret_cast<double*>(x) = slot ? xi[t] : fo[t];
    }
    // member t's place in the rows that generation g writes
    __device__ __forceinline__ char* place(int t, int g) const {
        return reinterpret_cast<char*>(l.xs + (g & 1) * P * kRowD + m[t] * kRowD + l8);
    }
    // in generation g: whether generation g - 2 stopped the fit
    __device__ __forceinline__ int stop_flag(int g) const { return g > g0 + 1 ? sh.stop[g & 1] : 0; }
    // centre of the set in effect and the range it carries within the box, of the
    // lane's slot
    __device__ __forceinline__ void limits(double& mid, double& nlo, double& nhi) const {
        mid = slot ? sh.lev.mid[l8] : 0.0;
        const double lim = slot ? sh.lev.lim[l8] : __builtin_inf();
        nlo = slot ? fmax(lo, mid - lim) : -__builtin_inf();
        nhi = slot ? fmin(hi, mid + lim) : __builtin_inf();
    }

    // generations on the full set, or a re-expanded one in LDS, until one of kind
    // 1 or 2 is in effect (in stretches, like register_loop's)
    __device__ __forceinline__ bool lds_loop(int& g) {
        // the set in use: the full one carries every trial
        const double *zs, *us;
        int n;
        double mid, nlo, nhi, en;
        auto level = [&]() {
            const bool whole = sh.lev.K == 0;
            zs = whole ? l.zw : l.lz;
            us = whole ? l.un : l.lu;
            n = whole ? K : sh.lev.K;
            limits(mid, nlo, nhi);
            mid = whole ? mid_w : mid;
            nlo = whole ? -__builtin_inf() : nlo;
            nhi = whole ? __builtin_inf() : nhi;
            en = whole ? en_w : node_energy(l.lz, n, N);
        };
        level();
        if (g == 0) {  // the initial population, accepted as it is
            feed(0);
#pragma unroll
            for (int t = 0; t < NM; ++t) {
                fo[t] = full(xi[t]);
                *reinterpret_cast<double*>(place(t, 0)) = slot ? xi[t] : fo[t];
            }
            lds_barrier();
            ++g;
        }
        uint64_t w[NM];
#pragma unroll
        for (int t = 0; t < NM; ++t) w[t] = draw(t, g);
        while (g < g1) {
            if (!(g & 7)) {
                if (!(g & 15) && sh.next.pend == g) {
                    relevel(nd, l, sh);
                    if (sh.lev.kind) return false;
                    level();
                }
                feed(g);
            }
            const char* xr = column(g);
            char* xw[NM];
#pragma unroll
            for (int t = 0; t < NM; ++t) xw[t] = place(t, g);
            int swap = (g & 1 ? 1 : -1) * P * kRowD * (int)sizeof(double);
            const int end = min((g | 7) + 1, g1);
            do {
                const int stop = stop_flag(g);
#pragma unroll
                for (int t = 0; t < NM; ++t) {
                    double v, x1;
                    mutant(xr, w[t], v, x1);
                    const double y = crossed(w[t]) ? bounded(v, x1) : xi[t];
                    const unsigned long long inside = __ballot(y >= nlo) & __ballot(y <= nhi);
                    const NodeCand q = node_cand<SLOPE, QUART>((y - mid) * sc);
                    double a1 = 0.0, a2 = 0.0;
                    lds_sums<SLOPE, QUART, COR>(q, zs, us, l8, n, a1, a2);
                    double ft = node_objective<SLOPE, COR>(nd, q, a1, a2, S2, en, N);
                    asm volatile("" : "+v"(ft));
                    if (__builtin_expect(inside != ~0ull, 0)) ft = full(y);
                    w[t] = draw(t, g + 1);
                    if (t == 0 && __builtin_expect(__builtin_amdgcn_readfirstlane(stop), 0)) return true;
                    keep(t, xw[t], y, ft);
                    xw[t] -= swap;
                }
                xr += swap;
                swap = -swap;
                lds_barrier();
            } while (++g < end);
        }
        return false;
    }

    // generations on 16 (KIND 1) or 8 (KIND 2) nodes in registers.  BOUNDS: the
    // bound rule is applied on the way; otherwise a mutant outside the box takes
    // the side path of those outside the set's limits, and a wave that takes it
    // often (a population pressed against a bound) goes over to BOUNDS: `often` is
    // set.  Both give the same bits.
    template <int KIND, bool STOPS, bool BOUNDS>
    __device__ __forceinline__ bool register_loop(int& g, bool& often) {
        constexpr int R = KIND == 1 ? 2 : 1;  // nodes per lane
        constexpr int D = KIND == 1 ? kNarDeg64 : kNar8Deg64;
        double zr[R], zi[R], wr[R], wi[R], u[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int k = l8 + 8 * r;
            zr[r] = l.lz[4 * k];
            zi[r] = l.lz[4 * k + 1];
            wr[r] = l.lz[4 * k + 2];
            wi[r] = l.lz[4 * k + 3];
            u[r] = l.lu[k];
        }
        const double en = node_energy(l.lz, 8 * R, N);
        double mid, nlo, nhi;
        limits(mid, nlo, nhi);
        double kc[D + 1], ks[D + 1];  // held in vector registers
#pragma unroll
        for (int k = 0; k <= D; ++k) {
            kc[k] = KIND == 1 ? kCosNar64[k] : kCosNar8[k];
            ks[k] = KIND == 1 ? kSinNar64[k] : kSinNar8[k];
            asm volatile("" : "+v"(kc[k]), "+v"(ks[k]));
        }
        auto value = [&](double y) {
            const NodeCand q = node_cand<SLOPE, QUART>((y - mid) * sc);
            double a1 = 0.0, a2 = 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double x = node_delta<QUART>(q, u[r]), x2 = x * x;
                double c = kc[0], s = ks[0];
#pragma unroll
                for (int k = 1; k <= D; ++k) {
                    c = __fma_rn(c, x2, kc[k]);
                    s = __fma_rn(s, x2, ks[k]);
                }
                node_terms<SLOPE, COR>(q, u[r], c, s * x, zr[r], zi[r], wr[r], wi[r], a1, a2);
            }
            return node_objective<SLOPE, COR>(nd, q, a1, a2, S2, en, N);
        };
        uint64_t w[NM];
#pragma unroll
        for (int t = 0; t < NM; ++t) w[t] = draw(t, g);
        // In stretches to the next multiple of 8: what can wait is done between
        // them (draws, a pending set, the count of side paths), and the two copies'
        // places are held and swapped instead of worked out (P = 40: 115
        // instructions and 0.44 us a generation with these inside, 90 and 0.35
        // without; 85 and 0.34 two generations at a time).
        while (g < g1) {
            if (!(g & 7)) {
                if (KIND == 1 && !(g & 15) && sh.next.pend == g) {
                    relevel(nd, l, sh);
                    return false;
                }
                // (an abandonment after generation g - 1 may be on its way: not before the
                // next look, for any wave)
                if (!STOPS && !(g & (kAbandonLook - 1)) &&
                    __builtin_expect(__builtin_amdgcn_readfirstlane(sh.abandoned) <= g - 2, 0))
                    return true;
                feed(g);
            }
            int side = 0;
            // one generation: rows read from xr, written to xw; next: the draws of the one
            // after it (not made after the last generation, and not used)
            auto one = [&](const char* xr, char* const (&xw)[NM], const uint64_t* next, int stop) {
#pragma unroll
                for (int t = 0; t < NM; ++t) {
                    double v, x1;
                    mutant(xr, w[t], v, x1);
                    double y = crossed(w[t]) ? (BOUNDS ? bounded(v, x1) : v) : xi[t];
                    const unsigned long long inside = __ballot(y >= nlo) & __ballot(y <= nhi);
                    double ft = value(y);
                    // (the limits are tested last, off the chain of dependent operations:
                    // outside them the value above is dropped)
                    asm volatile("" : "+v"(ft));
                    if (__builtin_expect(inside != ~0ull, 0)) {
                        if constexpr (BOUNDS) {
                            ft = full(y);
                        } else {
                            y = crossed(w[t]) ? bounded(v, x1) : xi[t];
                            ft = __ballot(y >= nlo && y <= nhi) == ~0ull ? value(y) : full(y);
                            ++side;
                        }
                    }
                    w[t] = next[t * kDrawRing];
                    if (STOPS && t == 0 && __builtin_expect(__builtin_amdgcn_readfirstlane(stop), 0)) return true;
                    keep(t, xw[t], y, ft);
                }
                lds_barrier();
                return false;
            };
            if (!STOPS && !(g & 7) && g + 8 <= g1) {
                // a whole stretch, two generations at a time: places and draws at fixed offsets
                const char *even = column(g), *odd = column(g + 1);
                char *to_even[NM], *to_odd[NM];
#pragma unroll
                for (int t = 0; t < NM; ++t) {
                    to_even[t] = place(t, g);
                    to_odd[t] = place(t, g + 1);
                }
                const uint64_t *next = draws(g) + 8, *last = next + 64;
                // (the loop at a multiple of 64 bytes: 1.3 % of a fit between the best and the
                // worst place for it)
                asm volatile(".p2align 6, , 60");
                do {
                    one(even, to_even, next, 0);
                    one(odd, to_odd, next + 8, 0);
                } while ((next += 16) != last);
                g += 8;
            } else {
                const char* xr = column(g);
                char* xw[NM];
#pragma unroll
                for (int t = 0; t < NM; ++t) xw[t] = place(t, g);
                int swap = (g & 1 ? 1 : -1) * P * kRowD * (int)sizeof(double);  // from the copy read to the one written
                const int end = min((g | 7) + 1, g1);
                asm volatile(".p2align 6, , 60");
                do {
                    if (one(xr, xw, draws(g + 1), STOPS ? stop_flag(g) : 0)) return true;
#pragma unroll
                    for (int t = 0; t < NM; ++t) xw[t] -= swap;
                    xr += swap;
                    swap = -swap;
                } while (++g < end);
            }
            if (!BOUNDS && side > 2 * NM) {
                often = true;
                return false;
            }
        }
        return false;
    }
    template <bool STOPS>
    __device__ __forceinline__ void narrow(int& g) {
        bool often = false;
        if (register_loop<2, STOPS, false>(g, often)) return;
        if (often && g < g1) register_loop<2, STOPS, true>(g, often);
    }

    __device__ __forceinline__ int run() {
        int g = g0;
        bool often = false;
        if (sh.lev.kind == 0 && lds_loop(g)) return g;
        if (g < g1 && sh.lev.kind == 1) {
            often = false;
            if (register_loop<1, true, false>(g, often)) return g;
            if (often && g < g1 && register_loop<1, true, true>(g, often)) return g;
        }
        if (g < g1) {
            if (stops)
                narrow<true>(g);
            else
                narrow<false>(g);
        }
        return g;
    }
};

// State of a fit after a launch, and the rest of its record if that ended it.
__device__ __forceinline__ void node_leave(const NodeDesc* nd, const BlockDesc* d, int gen, int flags, int bound, int best,
                                           double best_f) {
    DeState s = *d->st;
    s.gen = gen;
    s.done = flags != 0;
    s.flags = flags;
    s.best = best;
    s.best_f = best_f;
    *d->st = s;
    *nd->state = s;
    if (flags) {
        nd->rec->f = best_f;
        nd->rec->gens = gen;
        nd->rec->flags = flags | bound;
    }
}

template <int NM, bool COR>
__device__ __forceinline__ void fit_run(const NodeDesc* nd, const BlockDesc* d, int g0, int ngen, bool fresh,
                                        const uint64_t* draws, const FitLds& l, FitShared& sh) {
    const int tid = threadIdx.x, NT = blockDim.x, W = (NT >> 6) - 1, P = d->P, g1 = g0 + ngen;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int g;
    if (wave == W) {
        const bool window = d->rel_tol > 0.0 && d->window > 0;
        if (P <= 64)
            g = window ? Book<1, true>(nd, d, l, sh).run(g0, g1) : Book<1, false>(nd, d, l, sh).run(g0, g1);
        else
            g = window ? Book<4, true>(nd, d, l, sh).run(g0, g1) : Book<4, false>(nd, d, l, sh).run(g0, g1);
    } else if (nd->slope) {
        g = d->quartic ? Members<NM, true, true, COR>(nd, d, g0, g1, fresh, draws, l, sh).run()
                       : Members<NM, true, false, COR>(nd, d, g0, g1, fresh, draws, l, sh).run();
    } else {
        g = d->quartic ? Members<NM, false, true, COR>(nd, d, g0, g1, fresh, draws, l, sh).run()
                       : Members<NM, false, false, COR>(nd, d, g0, g1, fresh, draws, l, sh).run();
    }
    __syncthreads();
    // a stop of the last generation but one, or of the last; otherwise the last is kept
    int flags = sh.stop[g & 1];
    if (g == g1 && !(ngen > 1 && flags)) flags = sh.stop[(g1 - 1) & 1];
    if (sh.abandoned != kNeverGen) flags = kFlagNodeAbort;

    // state for the next launch: the population after the last kept generation
    const int gl = flags ? sh.stop_gen : g1 - 1;
    const double* xl = l.xs + (gl & 1) * P * kRowD;
    for (int e = tid; e < P * kRowD; e += NT) {
        const int j = e & (kRowD - 1);
        if (j < kSlots)
            gst(d->pop + e, xl[e]);
        else
            gst(d->fpop + e / kRowD, COR && flags ? cor_value(xl[e]) : xl[e]);
    }
    if (!flags) {
        double* o = nd->nar;
        constexpr int nl = 2 * sizeof(Level) / sizeof(double);
        static_assert(nl <= kNodeLevelHead, "both level records fit their place");
        for (int e = tid; e < nl; e += NT) gst(o + e, reinterpret_cast<const double*>(&sh.lev)[e]);
        o += kNodeLevelHead;
        const int n = sh.lev.K;
        for (int e = tid; e < 4 * n; e += NT) gst(o + e, l.lz[e]);
        for (int e = tid; e < n; e += NT) gst(o + 4 * n + e, l.lu[e]);
    }
    // the state, and of a fit that has ended its record (k_finalize's), for the
    // device's next launch and for the host
    if (wave == 0) {
        const int lane = tid & 63;
        int bound = 0;
        if (flags) {
            const int j = lane < kSlots ? lane : 0;
            const double x = xl[sh.best * kRowD + j], lo = gld(&d->lo[j]), hi = gld(&d->hi[j]), w = hi - lo;
            const bool at = lane < kSlots && (d->amask >> j & 1) && j != 1 && (x - lo <= 1e-6 * w || hi - x <= 1e-6 * w);
            bound = __ballot(at) ? 8 : 0;
            if (lane < kSlots) nd->rec->x[j] = x;
        }
        if (lane == 0) node_leave(nd, d, flags ? gl : g1, flags, bound, sh.best, sh.best_f);
    }
}

// MAXT: largest workgroup (512 threads leave each lane twice the registers).
template <int NM, bool COR, int MAXT>
__global__ __launch_bounds__(MAXT) void k_node_fit(const NodeDesc* __restrict__ nds, const BlockDesc* __restrict__ bds,
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

    const uint64_t* draws = nd->draws + ((nd->parity + flip) & 1) * node_draw_words(P, chunk);
    cos_table(l.tab, K);
    if (fresh) {
        init_block(d);
        if (tid == 0) {
            sh.lev.K = sh.lev.kind = 0;
            sh.lev.pend = sh.next.pend = -1;
        }
        const int n4 = 4 * K;
        const int nmom = nd->nmom;
        for (int e = tid; e < n4; e += NT) {
            double s = 0.0;
            for (int w = 0; w < nmom; w += 8) {  // eight loads in flight
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = w + q < nmom ? gld(nd->mom + (size_t)(w + q) * n4 + e) : 0.0;
#pragma unroll
                for (int q = 0; q < 8; ++q) s += v[q];
            }
            l.scr[e] = s;
        }
        if (wave == 0) {
            double s[1] = {0.0};
            for (int w = lane; w < nd->nproj; w += 256) {
                double v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = w + 64 * q < nd->nproj ? gld(nd->s2 + w + 64 * q) : 0.0;
                s[0] += (v[0] + v[1]) + (v[2] + v[3]);
            }
            wave_sums(s);
            if (lane == 0) sh.S2 = s[0];
        }
        __syncthreads();
        node_values(l.tab, l.scr, K, 2.0 / (double)K, [&](int k, int e, double v) {
            const double w = v * (e < 2 ? -2.0 : 1.0);  // -2 Z, W
            l.zw[4 * k + e] = w;
            gst(nd->wts + 4 * k + e, w);
        });
        if (tid == 0) gst(nd->wts + 4 * kNodeMaxK, sh.S2);
        for (int e = tid; e < P * kRowD; e += NT) l.xs[P * kRowD + e] = d->pop[e];  // written by init_block
    } else {
        for (int e = tid; e < 4 * K; e += NT) l.zw[e] = gld(nd->wts + e);
        const double* o = nd->nar;
        for (int e = tid; e < (int)(2 * sizeof(Level) / sizeof(double)); e += NT)
            reinterpret_cast<double*>(&sh.lev)[e] = gld(o + e);
        const int n = reinterpret_cast<const Level*>(o)->K;
        o += kNodeLevelHead;
        for (int e = tid; e < 4 * n; e += NT) l.lz[e] = gld(o + e);
        for (int e = tid; e < n; e += NT) l.lu[e] = gld(o + 4 * n + e);
        if (tid == 0) sh.S2 = gld(nd->wts + 4 * kNodeMaxK);
        double* x = l.xs + ((g0 + 1) & 1) * P * kRowD;
        for (int e = tid; e < P * kRowD; e += NT)
            x[e] = (e & (kRowD - 1)) < kSlots ? gld(d->pop + e) : gld(d->fpop + e / kRowD);
        for (int g = g0 - 1 - tid; g >= 0 && g >= g0 - kNodeRing; g -= NT)
            l.ring[g & (kNodeRing - 1)] = gld(d->hist + g);
    }
    if (tid < 2) sh.stop[tid] = 0;
    if (tid == 0) sh.abandoned = kNeverGen;
    if (!fresh) __syncthreads();  // tab complete
    for (int k = tid; k < K; k += NT) l.un[k] = l.tab[2 * k + 1] + nd->c;
    __syncthreads();
    if (fresh && !(sh.S2 < 1e290)) {
        // samples that are not finite (or overflow): the per-sample objective decides
        if (tid == 0) node_leave(nd, d, 0, kFlagNodeAbort, 0, 0, 0.0);
        return;
    }
    fit_run<NM, COR>(nd, d, g0, ngen, fresh, draws, l, sh);
}

using FitKernel = void (*)(const NodeDesc*, const BlockDesc*, int, int, int, int, int, int, int, int, int);

int fit_waves(int P) { return node_waves(P) + 1; }
template <bool COR>
FitKernel pick_fit(int P) {
    if (node_nm(P) == 2) return k_node_fit<2, COR, 1024>;
    return fit_waves(P) <= 8 ? k_node_fit<1, COR, 512> : k_node_fit<1, COR, 1024>;
}
FitKernel fit_kernel(int P, bool cor) { return cor ? pick_fit<true>(P) : pick_fit<false>(P); }

// Chebyshev nodes that interpolate exp(i p(x)) (times a polynomial of degree
// `extra`) on [-1, 1] to 1e-15, |coefficients| of p <= b1 .. b4: on an ellipse
// rho = e^eta the error is <= 4 M rho^-K / (rho - 1), M the largest modulus there.
// Every eta gives a valid bound: the best of a grid, whose part that does not
// depend on the coefficients is kept (6 -> 1 us of host time for a block's plan).
double nodes_needed(const double* b, int extra) {
    struct Ellipse {
        double eta, at0, g[4];
    };
    static const std::array<Ellipse, 160> grid = [] {
        std::array<Ellipse, 160> g;
        for (int i = 0; i < 160; ++i) {
            const double eta = 0.025 * (i + 1);
            g[i] = {eta, std::log(4e15 / (std::exp(eta) - 1.0)),
                    {ellipse_growth(1, 0, 0, 0, eta), ellipse_growth(0, 1, 0, 0, eta), ellipse_growth(0, 0, 1, 0, eta),
                     ellipse_growth(0, 0, 0, 1, eta)}};
        }
        return g;
    }();
    double best = 1e18;
    for (const Ellipse& e : grid)
        best = std::min(best, (e.at0 + (b[1] * e.g[0] + b[2] * e.g[1] + b[3] * e.g[2] + b[4] * e.g[3])) / e.eta + extra);
    return best;
}

}  // namespace

bool node_plan(const pt_block& B, double ref, int P, int max_gens, NodePlan* out) {
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
    if (!node_pays(nd.K, B.n, P, max_gens)) return false;

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

size_t node_fit_lds(int P, int maxK) { return fit_lds_doubles(P, maxK) * sizeof(double); }

bool node_fits(int P, int maxK, int lds_max) { return (int64_t)node_fit_lds(P, maxK) <= (int64_t)lds_max - 1024; }

hipError_t node_setup(int lds_max) {
    for (int P : {4, 100, kNodeMaxP})
        for (bool cor : {false, true}) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fit_kernel(P, cor)),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds_max - 1024);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t node_project(const NodeDesc* nd, const BlockDesc* bd, int nblk, int total_proj, hipStream_t s) {
    hipLaunchKernelGGL(k_node_project, dim3((unsigned)total_proj), dim3(256), 0, s, nd, bd, nblk);
    return hipGetLastError();
}

hipError_t node_moments(const NodeDesc* nd, const BlockDesc* bd, int nblk, int total_mom, int P, int ngen, int chunk,
                        hipStream_t s) {
    const int slices = (int)((node_draw_words(P, ngen) + 255) / 256);
    hipLaunchKernelGGL(k_node_moments, dim3((unsigned)(total_mom + nblk * slices)), dim3(256), 0, s, nd, bd, nblk, total_mom,
                       P, ngen, chunk, slices);
    return hipGetLastError();
}

hipError_t node_fit(const NodeDesc* nd, const BlockDesc* bd, int nblk, int P, int maxK, int off, int ngen, int next_ngen,
                    int chunk, int flip, bool cor, hipStream_t s) {
    const int nt = 64 * fit_waves(P);
    // workgroups that make the next launch's draws: none without one (each would
    // take the fit's LDS, the place of a fit in a batch larger than the chip)
    const int slices = (int)((node_draw_words(P, next_ngen) + nt - 1) / nt);
    const FitKernel k = fit_kernel(P, cor);
    hipLaunchKernelGGL(k, dim3((unsigned)(nblk + nblk * slices)), dim3((unsigned)nt),
                       (unsigned)node_fit_lds(P, maxK), s, nd, bd, nblk, P, maxK, off, ngen, next_ngen, chunk, flip,
                       slices > 0 ? slices : 1);
    return hipGetLastError();
}

}  // namespace pt
