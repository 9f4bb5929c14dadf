// nodes.h -- the fit of a block through node weights (host side interface).
//
// Over one block the model phase of a candidate differs from a reference
// phase phi_ref (the box's centre) by a smooth polynomial delta(x), x in
// [-1, 1] along the block, whose range the search box bounds.  exp(i delta)
// and exp(2 i delta) are therefore their own interpolants at K Chebyshev
// nodes x_k to FP64 rounding, and the sums over samples that the objective of
// Eq. (2-2-4) needs become sums over nodes:
//   sum_n s_n cos phi_n  = Re sum_k Z_k exp(i delta(x_k)),
//   sum_n cos 2 phi_n    = Re sum_k W_k exp(2 i delta(x_k)),
//   Z_k = sum_n s_n exp(i phi_ref(n)) L_k(x_n),
//   W_k = sum_n exp(2 i phi_ref(n)) L_k(x_n),
// L_k the Lagrange polynomials of the nodes.  With S2 = sum_n s_n^2,
//   chi^2 = S2 - 2 A sum s cos phi + A^2 (N + sum cos 2 phi) / 2
// (amplitude slope: the same with A + Adot t inside the sums).  A fit
// computes Z, W and S2 once from its samples and evaluates every candidate
// of every generation at K points (about a hundred) instead of N samples.
//
// Measured against one launch per generation over all samples (each generation
// a chain of ~9 us in its leading-step form; same machine): the 400 000-sample
// block, P = 40, 2000 generations 18.2 -> 0.90 ms; the quartic 1e6-sample block
// 39.5 -> 1.19 ms; 64 uneven blocks, 1500 generations 183 -> 0.97 ms (the
// blocks' generations then run on 64 compute units at once instead of sharing
// the chip's issue slots sample by sample).
//
// Three kernels:
//   k_node_project  samples -> 16 points per tile of samples (the same
//                   interpolation inside a tile, whose phase span needs only
//                   16 nodes)
//   k_node_moments  points -> Chebyshev moments of the block, partial sums; also
//                   the random draws of the first launch of generations
//   k_node_fit      moments -> Z, W (first launch), then whole generations of
//                   Differential Evolution, one workgroup per block; also the
//                   random draws of the next launch, if there is one
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/phasetrack.h"
#include "device.h"

namespace pt {

constexpr int kNodeMaxK = 512;    // largest node count of a block
constexpr int kNodeMaxP = 240;    // largest population (two members per octet of lanes, 15 waves)
constexpr int kNodePts = 16;      // nodes per tile
constexpr int kNodeRun = 4096;    // samples a projection workgroup takes at a time (16 per lane)
constexpr int kNodeGroup = 128;   // points per moments workgroup
constexpr int kNodeRing = 512;    // best-so-far values k_node_fit keeps in LDS for the window rule
constexpr int kNodeLevelHead = 48;  // doubles before a saved re-expanded set's weights
// largest |delta| (turns) of the sets of 16 and 8 nodes: the range of their
// sine and cosine polynomials
constexpr double kNodeTurns16 = 1.0 / 8, kNodeTurns8 = 1.0 / 48;
// Chi-square is taken as a difference from S2, so its error is a few ulp of S2 and
// its relative error grows with the signal to noise: a fit whose best falls below
// this share of S2 is abandoned and run over its samples.  FP64: 12 dB.  Rms error
// relative to chi-square, nodes / samples: up to 10 dB 6e-15 or less / 7e-15 to
// 1e-13 (carriers of tens of Hz and more, n = 256 to 1e5); at 13 dB 1.9e-14 / 4e-15
// for 256 samples whose phase covers 30 turns, 1.4e-14 / 2.2e-14 for 20 000; at 28 dB
// 3.7e-13 / 1.2e-13 for those.  (Where the phase stays within a few turns, a carrier
// near zero, the samples' sums are exact to 2e-16 at any signal to noise.)  Mixed: 30
// dB, its sums over the samples are off by 1e-9 and more.
__host__ __device__ constexpr double node_cancel(bool mixed) { return mixed ? 1e-3 : 1.0 / 16; }
enum { kFlagNodeAbort = 1 << 16 };  // DeState::flags of an abandoned fit

struct DeState;
struct FitRecord;

// One block of a node-weight launch, beside its BlockDesc.
struct NodeDesc {
    // reference phase in turns, a polynomial in m = n - ref: r1 (hi + lo), r2, r3, r4
    double r1h, r1l, r2, r3, r4;
    // x = (n - (N - 1) / 2) / h, h = (N - 1) / 2; m = h (x + c)
    double h, c;
    // slot -> coefficient of u = m / h: (value - mid) * sc (turns; amplitude units for slots 0 and 5)
    double mid[kSlots], sc[kSlots];
    double su1, su2;   // sum over samples of u and u^2 (energy of a sloping amplitude)
    double cancel;     // node_cancel of the fit's precision
    int K;             // nodes, a multiple of 16
    int slope;         // the amplitude slope is active
    int lanes_log;     // log2 of the lanes (16 samples each) sharing a tile
    int runs;          // kNodeRun-sample runs per projection workgroup
    int ntile;         // tiles
    int proj_begin, nproj;  // projection workgroups
    int mom_begin, nmom;    // moments workgroups before it; groups of points
    int g0;            // next generation of the block when the descriptors were uploaded
    int parity;        // which half of `draws` the next launch reads
    double* pts;       // ntile x 16 x (Re s e, Im s e, Re e^2, Im e^2)
    double* s2;        // nproj partial sums of s^2
    double* mom;       // nmom x K x 4 partial moments
    double* wts;       // K x 4 weights, then S2
    double* nar;       // the re-expanded set between launches
    uint64_t* draws;   // two halves of packed draws, node_draw_words each
    // in host memory: the state after each launch, and the record of a fit that has
    // ended (written by the fit: a kernel and two copies of ~4 us each otherwise)
    DeState* state;
    FitRecord* rec;
};

struct NodePlan {
    NodeDesc nd;       // everything but the pointers, prefixes, limit, g0 and parity
    size_t pts_doubles, s2_doubles, mom_doubles;  // working space of the projection
};
constexpr size_t kNodeWtsDoubles = 4 * kNodeMaxK + 2;
constexpr size_t kNodeNarDoubles = kNodeLevelHead + 5 * (kNodeMaxK / 8 * 5);

// Whether a block's fits go through node weights, and its plan: depends on
// the block (length, rate, reference, box), the population size and the
// generations only.
bool node_plan(const pt_block& b, double ref, int P, int max_gens, NodePlan* out);

// Dynamic LDS bytes of k_node_fit for population P and nodes up to maxK, and
// whether the device has them.
size_t node_fit_lds(int P, int maxK);
bool node_fits(int P, int maxK, int lds_max);

// Members per octet of lanes (the fewest that leave a wave for the bookkeeping)
// and waves of members of a population's workgroup; 8-byte words that the packed
// draws of some generations take (from any generation on, in blocks of 16).
__host__ __device__ inline int node_nm(int P) { return P <= 120 ? 1 : 2; }
__host__ __device__ inline int node_waves(int P) { return (P + 8 * node_nm(P) - 1) / (8 * node_nm(P)); }
__host__ __device__ inline size_t node_draw_words(int P, int gens) {
    return gens ? (size_t)((gens + 30) / 16) * 128 * node_nm(P) * node_waves(P) : 0;
}

// Whether a fit is shorter through K nodes than over n samples, both without what
// they share.  Only a few generations on many nodes are not: sets shrink after some
// 40, while a generation over the samples of a small block has the whole chip.  In
// microseconds, fitted to single fits of 2 to 501 generations, 8 to 240 members, 512
// to 4e5 samples and 48 to 464 nodes (nodes / samples: 464 nodes, P = 40, 5e4 samples
// 101 / 56 for 2 generations, 266 / 191 for 21, 536 / 784 for 101; 256 nodes, P = 240,
// 4096 samples 482 / 203 for 21, 1415 / 3692 for 501; 112 nodes, P = 40 52 / 49 for 2,
// 97 / 147 for 21): of 480 fits the rule leaves five slower, by 7 to 22.
inline bool node_pays(int K, int64_t n, int P, int max_gens) {
    const double G = max_gens + 1.0, W = node_waves(P);
    const double per_simd = W * node_nm(P) / 4;  // members of an octet, on the fullest SIMD
    const double gen = 0.0093 * K * (per_simd > 1 ? (double)(int64_t)(per_simd + 0.75) : 1.3);
    const double nodes = 0.06 * P + 1e-3 * K * K / (W + 1) + (G < 40 ? G : 40) * gen;
    return nodes <= 2.4 + G * (5.1 + 7e-7 * P * (double)n);
}

// Launches (nd / bd: device tables of nblk blocks; chunk: generations per
// half of `draws`).  `off`: generations run since the tables were uploaded.
inline int node_mom_wgs(const NodeDesc& n) { return n.nmom * ((n.K + 63) / 64); }
hipError_t node_project(const NodeDesc* nd, const BlockDesc* bd, int nblk, int total_proj, hipStream_t s);
hipError_t node_moments(const NodeDesc* nd, const BlockDesc* bd, int nblk, int total_mom, int P, int ngen, int chunk,
                        hipStream_t s);
hipError_t node_fit(const NodeDesc* nd, const BlockDesc* bd, int nblk, int P, int maxK, int off, int ngen, int next_ngen,
                    int chunk, int flip, bool cor, hipStream_t s);
hipError_t node_setup(int lds_max);  // once per device

}  // namespace pt
