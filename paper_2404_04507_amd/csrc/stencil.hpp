// stencil.hpp - the Hamiltonian apply of a potential with few Fourier modes,
// as the wrapped convolution it is.
//
// By the discrete convolution theorem on the lifted grid (App. C), the
// potential block F* diag(V) F*^{-1} of Sec. 4.1 equals
//     (C psi)[k*] = sum_m Vhat_m psi[(k* - m) mod ext],
// so a potential of a few modes needs a few neighbours per point instead of
// two transforms.  The modes come in pairs (m, -m) with conjugate
// coefficients (V is real), plus the constant one.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace iwfpm {

// Exact division of dividends below 2^31 by a fixed divisor (Granlund and
// Montgomery, "Division by invariant integers using multiplication", 1994):
// q = (mulhi(a, m) + a) >> s.
struct FastDiv {
    unsigned d = 1, m = 1, s = 0;
};
inline FastDiv fast_div(unsigned d) {
    FastDiv f;
    f.d = d;
    while ((1ull << f.s) < d) ++f.s;
    f.m = (unsigned)(((1ull << 32) * ((1ull << f.s) - d)) / d + 1);
    return f;
}
__host__ __device__ inline unsigned fdiv(unsigned a, const FastDiv& f) {
    return (unsigned)((((unsigned long long)a * f.m) >> 32) + a) >> f.s;
}

// k_I axes and mode pairs that the kernels are compiled for
constexpr int kStencilMaxD = 3;
constexpr int kStencilMaxPairs = 16;
// pairs of the compiled kernels; a plan takes the next larger one
#define IWFPM_STENCIL_PAIRS(X) X(1) X(2) X(3) X(4) X(6) X(8) X(12) X(16)
constexpr int kStencilThreads = 256;

struct StencilDesc {
    int np;                                      // mode pairs of the kernel (padded with zero coefficients)
    int real;                                    // every coefficient real
    int tile_row;                                // tiles of one XCD's share of a row of tiles (see stencil_tile)
    int ns_max;                                  // slices that a tile can touch
    double c0;                                   // constant mode
    double cr[kStencilMaxPairs];                 // Re, Im of the pair's Vhat_m
    double ci[kStencilMaxPairs];
    short off[kStencilMaxPairs][kMaxAxes];       // m mod ext, by storage axis
    FastDiv dslice;                              // points per k_I slice
    FastDiv dext[kMaxAxes];                      // extents
};

// One pair per axis (pair j along storage axis j, |m_0| = 1): the walk along
// axis 0.
struct StarDesc {
    int ok;
    int plane, planes;   // points of a plane (the last L axes), planes per workgroup
    int ptiles, tiles;   // workgroups that cover one (i0, i1), one step of axis 0
    int whole;           // an XCD takes whole steps
    int steps, chunks;   // steps that a workgroup walks, workgroups that cover axis 0
};

// slices that `points` consecutive points can touch
inline int stencil_slices(const DevGeom& g, int points) { return (points + g.nkI - 2) / g.nkI + 1; }
inline size_t stencil_lds(const DevGeom& g, const StencilDesc& sd) {
    return (size_t)sd.ns_max * 2 * sd.np * 16;
}

// threads of a star workgroup
inline int star_block(const StarDesc& w) { return (w.planes * w.plane + 63) / 64 * 64; }
bool star_supported(int n, int d);

hipError_t launch_stencil(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, const StarDesc& w,
                          const void* psi, void* hpsi, int nvec, hipStream_t st);
hipError_t prepare_stencil();

// Ragged batches: one launch per kind of kernel over the batch's items of that
// kind.  What a plan has is uploaded once, what a call brings with each apply.
struct FewItem {
    DevGeom g;
    DevTabs t;
    StencilDesc sd;
    StarDesc w;
    int kind;        // few_kind or few_joint_kind, -1: not a few-mode plan
};
struct FewCall {
    StarDesc w;      // star: the item's, with this call's walk
    const double2* psi;
    double2* hpsi;
    int nvec;
    int rot;         // star: XCDs that its groups of workgroups are turned by
    int gx, vb;      // point kernel: workgroups per group of vectors, vectors of a group
};
struct FewLaunch {
    int kind, threads, grid;
    size_t lds;
};
int few_kind(const DevGeom& g, const StencilDesc& sd, const StarDesc& w);
// the kind of the point kernel that takes any number of pairs
inline int few_joint_kind(int d) { return 1000 + d; }
// sets the call's walk for a launch of `total` points; its workgroups (a multiple of 8)
int few_blocks(const FewItem& it, FewCall& call, double total);
// threads, LDS and grid of the launch of l.kind, for any counts of vectors
hipError_t few_launch_config(FewLaunch& l, const FewItem* items, int B);
// start: first workgroup of each item (items of another kind have none), start[B] the total
hipError_t launch_few_batch(const FewLaunch& l, const FewItem* items, const FewCall* calls, const int* start, int B,
                            hipStream_t st);

}  // namespace iwfpm
