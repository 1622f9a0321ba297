// stencil.hip - kernels of the few-mode Hamiltonian apply (see stencil.hpp).
//
// What bounds it: 32 B per point and vector (psi read once, H psi written
// once) against the transforms' 80 B (float32) or 112 B (float64) in three
// passes; a point's 4 n + 2 products are far below the ridge.  What it costs
// beyond that is the neighbours: read one by one they are 2 n more 16-byte
// loads per point through the L1 (64 B per clock and CU), and those along the
// slow axes come from beyond the 4 MB L2 of an XCD.  The star kernel takes
// most of them from registers and LDS.  Measured per apply, inputs rotating
// through three sets (a 2 GiB device copy reaches 4.9 TB/s on the same card):
//   24^2 x 32^2 points, 16 vectors: transforms 181 us (float32) and 332 us
//     (float64), point kernel 96 us, star kernel 78 us, floor 60 us
//   16^6, 8 vectors: transforms 3.13 ms (float32), point kernel 1.90 ms, star
//     kernel 1.20 ms, floor 0.87 ms
#include <hip/hip_runtime.h>

#include <algorithm>

#include "stencil.hpp"

namespace iwfpm {
namespace {

typedef double st_d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned umod1(unsigned a, unsigned E) { return min(a, a - E); }  // a < 2 E

// The arithmetic of one point, the same in every kernel, so that a vector's
// result does not depend on the block or the launch it is applied in: the
// pairs are added in storage-axis order, each product fused.
struct StencilSum {
    double re, im;
    __device__ __forceinline__ void diag(double l, double2 c) {
        re = l * c.x;
        im = l * c.y;
    }
    __device__ __forceinline__ void pair_real(double cr, double2 A, double2 B) {
        re = fma(cr, A.x + B.x, re);
        im = fma(cr, A.y + B.y, im);
    }
    // Vhat psi[k* - m] + conj(Vhat) psi[k* + m]
    __device__ __forceinline__ void pair_cplx(double cr, double ci, double2 A, double2 B) {
        re = fma(-ci, A.y - B.y, fma(cr, A.x + B.x, re));
        im = fma(ci, A.x - B.x, fma(cr, A.y + B.y, im));
    }
    __device__ __forceinline__ void store(double2* y) const {
        __builtin_nontemporal_store(st_d2{re, im}, reinterpret_cast<st_d2*>(y));
    }
};

// 1/2 sum_j (g_j + sum_i (2 pi P_I)_{j i} k_i)^2, g the slice's 2 pi P_II k_II
template <int D>
__device__ __forceinline__ double stencil_kinetic(const double* P1, const double* gs, const double (&k)[D]) {
    double lam = 0.0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        double b = gs[j];
#pragma unroll
        for (int i = 0; i < D; ++i) b = fma(P1[j * D + i], k[i], b);
        lam = fma(b, b, lam);
    }
    return 0.5 * lam;
}

// Neighbour tables of the slices [s0, s0 + ns): entry 2 m + (0: -m, 1: +m) of
// a slice holds the first vector position of the neighbour's slice and, per
// k_I axis, the rotation taking the point's coordinate in its vector order to
// the neighbour's.  In grid order that is -+ m_j; in window order the
// coordinate counts from the slice's own lower window end a_j, so
// p' = p + a_j -+ m_j - a'_j (mod the extent); of the ends modulo the extent, as
// ends of nearly 2^31 have no 32-bit difference.
template <int D>
__device__ __forceinline__ void stencil_tables(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, int s0,
                                               int ns, int4* tab) {
    const int np2 = 2 * sd.np, nII = g.n - D;
    const int nslice = (int)fdiv(g.N, sd.dslice);
    for (int e = threadIdx.x; e < ns * np2; e += blockDim.x) {
        const int sl = e / np2, k = e - sl * np2, m = k >> 1;
        const int s = s0 + sl;
        if (s >= nslice) continue;
        unsigned r = (unsigned)s;
        int sn = s, stride = 1;
        for (int ax = nII - 1; ax >= 0; --ax) {
            const unsigned q = fdiv(r, sd.dext[ax]);
            const int E = g.ext[ax], c = (int)(r - q * E), o = sd.off[m][ax];
            r = q;
            int cn = (k & 1) ? c + o : c - o;
            cn += cn < 0 ? E : 0;
            cn -= cn >= E ? E : 0;
            sn += (cn - c) * stride;
            stride *= E;
        }
        int dl[3] = {0, 0, 0};
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const int E = g.ext[nII + j], o = sd.off[m][nII + j];
            int v = (k & 1) ? o : -o;
            if (g.order) v += t.slice_m[s * D + j] - t.slice_m[sn * D + j];
            v %= E;
            dl[j] = v < 0 ? v + E : v;
        }
        tab[e] = make_int4(sn * g.nkI, dl[0], dl[1], dl[2]);
    }
}

// y = (Lambda + Vhat_0) x + sum over the pairs, for the vectors [v0, v1) of the
// block, one point per thread: its neighbours' positions and its kinetic term
// are formed once for all of the vectors.
template <int D, int NP>
__device__ __forceinline__ void stencil_body(const DevGeom& g, const DevTabs& t, const StencilDesc& sd,
                                             const double2* __restrict__ psi, double2* __restrict__ hpsi, int tile,
                                             int v0, int v1, int4* tab) {
    const int nII = g.n - D;
    const int e0 = tile * (int)blockDim.x;
    const int s0 = (int)fdiv(e0, sd.dslice);
    const int elast = g.N - e0 > (int)blockDim.x ? e0 + (int)blockDim.x - 1 : g.N - 1;
    stencil_tables<D>(g, t, sd, s0, (int)fdiv(elast, sd.dslice) - s0 + 1, tab);
    __syncthreads();
    const int e = e0 + threadIdx.x;
    if (e >= g.N) return;
    const int s = (int)fdiv(e, sd.dslice);
    unsigned q = (unsigned)(e - s * g.nkI), p[D], E[D];
#pragma unroll
    for (int j = D - 1; j >= 0; --j) {
        E[j] = g.ext[nII + j];
        const unsigned h = fdiv(q, sd.dext[nII + j]);
        p[j] = q - h * E[j];
        q = h;
    }
    int idx[2 * NP];
    const int4* row = tab + (s - s0) * 2 * NP;
#pragma unroll
    for (int k = 0; k < 2 * NP; ++k) {
        const int4 en = row[k];
        unsigned i = en.x;
        i += umod1(p[0] + en.y, E[0]) * g.stride[nII];
        if constexpr (D > 1) i += umod1(p[1] + en.z, E[1]) * g.stride[nII + 1];
        if constexpr (D > 2) i += umod1(p[2] + en.w, E[2]) * g.stride[nII + 2];
        idx[k] = (int)i;
    }
    double lam = 0.0;
    if (g.kin) {
        double kl[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const int a = t.slice_a[s * D + j];
            int pj = (int)p[j];
            if (!g.order) {  // window coordinate of the grid coordinate
                pj -= t.slice_m[s * D + j];
                pj += pj < 0 ? (int)E[j] : 0;
            }
            kl[j] = (double)(a + pj);
        }
        lam = stencil_kinetic<D>(g.P1, t.slice_g + (long long)s * D, kl);
    }
    lam += sd.c0;
    const bool real = sd.real != 0;
    const long long N = g.N;
    double cr[NP], ci[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        cr[m] = sd.cr[m];
        ci[m] = sd.ci[m];
    }
    for (int v = v0; v < v1; ++v) {
        const double2* __restrict__ x = psi + v * N;
        const double2 c = x[e];
        double2 A[NP], B[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            A[m] = x[idx[2 * m]];
            B[m] = x[idx[2 * m + 1]];
        }
        StencilSum y;
        y.diag(lam, c);
        if (real) {
#pragma unroll
            for (int m = 0; m < NP; ++m) y.pair_real(cr[m], A[m], B[m]);
        } else {
#pragma unroll
            for (int m = 0; m < NP; ++m) y.pair_cplx(cr[m], ci[m], A[m], B[m]);
        }
        y.store(hpsi + v * N + e);
    }
}

// Workgroups are dealt round-robin over the 8 XCDs.  Tiles run in rows of
// 8 c; XCD x takes the x-th c tiles of every row.  With a row about as long as
// one step of the slowest axis, an XCD keeps the same part of the plane from
// step to step, and the neighbours along that axis are in its own L2.
__device__ __forceinline__ int stencil_tile(int b, int c) {
    const int xcd = b & 7, l = b >> 3;
    const int r = l / c;
    return (r * 8 + xcd) * c + l - r * c;
}

// ---------------------------------------------------------------------------
// star: one pair per axis (a cosine lattice), the slowest axis walked
// ---------------------------------------------------------------------------

// Shape of the kernel for n axes, D of them k_I axes: the last L axes are the
// plane, NG axes lie between it and the axes held in registers (axis 0, and
// axis 1 where there are two k_II axes or more).
template <int N, int D>
struct StarShape {
    static constexpr int L = D < 2 ? D : 2;
    static constexpr int nII = N - D;
    static constexpr int F = nII > 1 ? 2 : 1;  // first axis after those in registers
    static constexpr int NG = N - L - F;
    static constexpr int NN = nII - F;         // of the NG axes, those that change the slice
};

// per-slice data of the walk, in LDS
template <int N, int D>
struct StarRow {
    static constexpr int NN = StarShape<N, D>::NN;
    double g[D];                      // 2 pi P_II k_II
    int a[D];                         // lower window end
    int am[D];                        // a mod extent
    int nm[NN ? 2 * NN : 1][D];       // window order: am of the two neighbours along each of the NN axes
};

// what the walk reads again and again, by value: in a batch the descriptors
// are in global memory, and every store could change them
template <int N, int D>
struct StarConst {
    int ext[N], str[N];
    double cr[N], ci[N], P1[D * D], c0;
    bool window, kin, real;
    __device__ __forceinline__ StarConst(const DevGeom& g, const StencilDesc& sd)
        : c0(sd.c0), window(g.order != 0), kin(g.kin != 0), real(sd.real != 0) {
#pragma unroll
        for (int a = 0; a < N; ++a) {
            ext[a] = g.ext[a];
            str[a] = g.stride[a];
            cr[a] = sd.cr[a];
            ci[a] = sd.ci[a];
        }
#pragma unroll
        for (int j = 0; j < D * D; ++j) P1[j] = g.P1[j];
    }
    // vector position within its slice of the point with grid coordinates c
    __device__ __forceinline__ unsigned pos(const unsigned (&c)[D], const int* am) const {
        unsigned i = 0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const unsigned E = ext[N - D + j];
            i += umod1(c[j] + E - am[j], E) * str[N - D + j];
        }
        return i;
    }
};

// A workgroup holds, per thread, B points along axis 1 (B = 1 and no such axis
// when there is one k_II axis) and walks `steps` steps of axis 0: the
// neighbours along axis 0 are the thread's own previous and next values, those
// along axis 1 its other points (and one more on either side), those along the
// last L axes come from an LDS copy of the step's planes, and only the axes in
// between are read again from the caches.
template <int N, int D, int B>
__device__ __forceinline__ void star_body(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, const StarDesc& w,
                                          const double2* __restrict__ x, double2* __restrict__ y, int tile, int i_lo,
                                          unsigned char* smem) {
    using Sh = StarShape<N, D>;
    using Row = StarRow<N, D>;
    constexpr int nII = Sh::nII, F = Sh::F, NG = Sh::NG, L = Sh::L, NN = Sh::NN;
    constexpr bool two = F == 2;
    constexpr int H = two ? 1 : 0;    // halo points of axis 1 on either side
    const StarConst<N, D> cst(g, sd);
    const int nkI = g.nkI;
    const int E0 = cst.ext[0], E1 = two ? cst.ext[1] : 1;
    const int R0 = cst.str[0], R1 = cst.str[F - 1];  // points of one step, of one (i0, i1)
    const int T = blockDim.x, tid = threadIdx.x;
    const int steps = min(w.steps, E0 - i_lo);
    double2* lds = reinterpret_cast<double2*>(smem);  // two buffers of B x T points
    Row* rows = reinterpret_cast<Row*>(lds + 2 * B * T);
    const int j1 = tile / w.ptiles;
    const int pts = w.planes * w.plane;
    const int r0 = (tile - j1 * w.ptiles) * pts;
    const bool live = tid < pts && r0 + tid < R1;
    const unsigned r = live ? (unsigned)(r0 + tid) : (unsigned)r0;
    const int own = live ? tid : 0;
    // axis-1 coordinate of point b (wrapped: the points past the axis' end are
    // loaded as the neighbours they are, and not stored)
    auto i1_of = [&](int b) -> int {
        int i = j1 * B + b;
        i += i < 0 ? E1 : 0;
        while (i >= E1) i -= E1;
        return i;
    };
    unsigned c[D], e2[N];  // grid coordinates within (i0, i1)
    const unsigned sr = fdiv(r, sd.dslice);
    {
        unsigned q = r - sr * nkI;
#pragma unroll
        for (int j = D - 1; j >= 0; --j) {
            const unsigned h = fdiv(q, sd.dext[nII + j]);
            c[j] = q - h * cst.ext[nII + j];
            q = h;
        }
        q = sr;
#pragma unroll
        for (int j = nII - 1; j >= F; --j) {
            const unsigned h = fdiv(q, sd.dext[j]);
            e2[j] = q - h * cst.ext[j];
            q = h;
        }
    }
    const int sp0 = R0 / nkI, sp1 = R1 / nkI;  // slices of a step, of one (i0, i1)
    const int s_lo = (int)fdiv((unsigned)r0, sd.dslice);
    const int ns = (int)fdiv((unsigned)(min(r0 + pts, R1) - 1), sd.dslice) - s_lo + 1;
    // slice data: entry ((k (B + 2 H) + b) ns + s) for step i_lo - 1 + k, axis-1 point b - H
    constexpr int BW = B + 2 * H;
    for (int e = tid; e < (steps + 2) * BW * ns; e += T) {
        const int s = e % ns, kb = e / ns;
        const int k = kb / BW, b = kb - k * BW;
        int i = i_lo - 1 + k;
        i += i < 0 ? E0 : 0;
        while (i >= E0) i -= E0;
        const int sl = i * sp0 + (two ? i1_of(b - H) * sp1 : 0) + s_lo + s;
        Row& row = rows[e];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            row.a[j] = t.slice_a[sl * D + j];
            row.am[j] = t.slice_m[sl * D + j];
            row.g[j] = t.slice_g[(long long)sl * D + j];
        }
        if (NN > 0 && cst.window) {
            unsigned q = (unsigned)(s_lo + s);
            int st = 1;
#pragma unroll
            for (int ax = nII - 1; ax >= F; --ax) {
                const int E = cst.ext[ax], o = sd.off[ax][ax];
                const unsigned h = fdiv(q, sd.dext[ax]);
                const int cx = (int)(q - h * E);
                q = h;
                int lo = cx - o, hi = cx + o;
                lo += lo < 0 ? E : 0;
                hi -= hi >= E ? E : 0;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    row.nm[2 * (ax - F)][j] = t.slice_m[(sl + (lo - cx) * st) * D + j];
                    row.nm[2 * (ax - F) + 1][j] = t.slice_m[(sl + (hi - cx) * st) * D + j];
                }
                st *= E;
            }
        }
    }
    // neighbours of the other axes, relative to the point in grid order
    int del[2 * (NG + L)];
#pragma unroll
    for (int j = 0; j < NG + L; ++j) {
        const int ax = F + j;
        const int E = cst.ext[ax], o = sd.off[ax][ax];
        const int cj = ax < nII ? (int)e2[ax < nII ? ax : 0] : (int)c[ax >= nII ? ax - nII : 0];
        int lo = cj - o, hi = cj + o;
        lo += lo < 0 ? E : 0;
        hi -= hi >= E ? E : 0;
        del[2 * j] = (lo - cj) * cst.str[ax];
        del[2 * j + 1] = (hi - cj) * cst.str[ax];
    }
    __syncthreads();
    const bool window = cst.window;
    const unsigned rb = sr * nkI;
    const Row* row = rows + ((int)sr - s_lo);  // (step, point b): row[((k + 1) BW + b + H) ns]
    auto row_of = [&](int k, int b) -> const Row* { return row + ((k + 1) * BW + b + H) * ns; };
    // position within (i0, i1) of this thread's point b at step i_lo + k
    auto at = [&](int k, int b) -> unsigned { return window ? rb + cst.pos(c, row_of(k, b)->am) : r; };
    long long boff[BW];
#pragma unroll
    for (int b = 0; b < BW; ++b) boff[b] = two ? (long long)i1_of(b - H) * R1 : 0;
    auto base = [&](int i, int b) -> long long { return (long long)i * R0 + boff[b + H]; };
    auto load = [&](long long first, unsigned off) -> double2 {
        return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(x + first) + (off << 4));
    };
    auto wrap0 = [&](int i) -> int { return i < 0 ? i + E0 : (i < E0 ? i : i - E0); };
    double2 prev[B], cur[B];
    unsigned pos[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        prev[b] = load(base(wrap0(i_lo - 1), b), at(-1, b));
        pos[b] = at(0, b);
        cur[b] = load(base(i_lo, b), pos[b]);
    }
    int buf = 0;
    for (int k = 0; k < steps; ++k) {
        const int i = i_lo + k;
        double2 nxt[B];
        unsigned npos[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            npos[b] = at(k + 1, b);
            nxt[b] = load(base(wrap0(i + 1), b), npos[b]);
        }
        double2 lo1 = make_double2(0.0, 0.0), hi1 = lo1;
        if constexpr (two) {
            lo1 = load(base(i, -1), at(k, -1));
            hi1 = load(base(i, B), at(k, B));
        }
        double2 gv[B][NG ? 2 * NG : 1];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const long long first = base(i, b);
            const Row* rw = row_of(k, b);
#pragma unroll
            for (int q = 0; q < 2 * NG; ++q) {
                unsigned o = r + del[q];
                if (window) {
                    const int ax = F + (q >> 1);
                    if (ax < nII) {
                        // another slice of the same step: its own rotation
                        o = rb + del[q] + cst.pos(c, rw->nm[NN && ax < nII ? q : 0]);
                    } else {
                        unsigned cn[D];
#pragma unroll
                        for (int j = 0; j < D; ++j) cn[j] = c[j];
                        cn[ax >= nII ? ax - nII : 0] += del[q] / cst.str[ax];
                        o = rb + cst.pos(cn, rw->am);
                    }
                }
                gv[b][q] = load(first, o);
            }
        }
        double2* const tileb = lds + buf * B * T;
#pragma unroll
        for (int b = 0; b < B; ++b) tileb[b * T + tid] = cur[b];
        // LDS alone is ordered here: the global loads stay in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
        for (int b = 0; b < B; ++b) {
            double lam = 0.0;
            if (cst.kin) {
                const Row* rw = row_of(k, b);
                double kl[D];
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const unsigned E = cst.ext[nII + j];
                    kl[j] = (double)(rw->a[j] + (int)umod1(c[j] + E - rw->am[j], E));
                }
                lam = stencil_kinetic<D>(cst.P1, rw->g, kl);
            }
            lam += cst.c0;
            const double2* nb = tileb + b * T + own;
            const double2 lo = b > 0 ? cur[b > 0 ? b - 1 : 0] : lo1;
            const double2 hi = b + 1 < B ? cur[b + 1 < B ? b + 1 : 0] : hi1;
            StencilSum s;
            s.diag(lam, cur[b]);
            if (cst.real) {
                s.pair_real(cst.cr[0], prev[b], nxt[b]);
                if constexpr (two) s.pair_real(cst.cr[1], lo, hi);
#pragma unroll
                for (int j = 0; j < NG; ++j) s.pair_real(cst.cr[F + j], gv[b][2 * j], gv[b][2 * j + 1]);
#pragma unroll
                for (int j = NG; j < NG + L; ++j) s.pair_real(cst.cr[F + j], nb[del[2 * j]], nb[del[2 * j + 1]]);
            } else {
                s.pair_cplx(cst.cr[0], cst.ci[0], prev[b], nxt[b]);
                if constexpr (two) s.pair_cplx(cst.cr[1], cst.ci[1], lo, hi);
#pragma unroll
                for (int j = 0; j < NG; ++j)
                    s.pair_cplx(cst.cr[F + j], cst.ci[F + j], gv[b][2 * j], gv[b][2 * j + 1]);
#pragma unroll
                for (int j = NG; j < NG + L; ++j)
                    s.pair_cplx(cst.cr[F + j], cst.ci[F + j], nb[del[2 * j]], nb[del[2 * j + 1]]);
            }
            if (live && j1 * B + b < E1) s.store(y + base(i, b) + pos[b]);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            prev[b] = cur[b];
            cur[b] = nxt[b];
            pos[b] = npos[b];
        }
        buf ^= 1;
    }
}

// The workgroup's place: groups (one vector's chunk of steps) of w.tiles tiles,
// dealt round-robin over the 8 XCDs.  A step of few tiles belongs to one XCD
// as a whole (its neighbours then meet in that XCD's L2); a longer one is cut
// into 8 contiguous shares.  false: nothing to do.
__device__ __forceinline__ bool star_place(const StarDesc& w, int nvec, int b, int& tile, int& v, int& chunk) {
    int grp;
    if (w.whole) {
        const int l = b >> 3, q = l / w.tiles;
        grp = q * 8 + (b & 7);
        tile = l - q * w.tiles;
    } else {
        const int per = (w.tiles + 7) / 8;
        grp = b / (8 * per);
        const int l = b - grp * 8 * per;
        tile = (l & 7) * per + (l >> 3);
        if (tile >= w.tiles) return false;
    }
    v = grp / w.chunks;
    chunk = grp - v * w.chunks;
    return v < nvec;
}
int star_blocks(const StarDesc& w, int nvec) {
    const int groups = w.chunks * nvec;
    return w.whole ? (groups + 7) / 8 * 8 * w.tiles : groups * 8 * ((w.tiles + 7) / 8);
}

// workgroups of up to 512 threads where a thread's 4 points need the registers
constexpr int star_threads(int N) { return N == 6 ? 512 : 1024; }

template <int N, int D, int B>
__global__ void __launch_bounds__(star_threads(N)) k_star(DevGeom g, DevTabs t, StencilDesc sd, StarDesc w,
                                                          const double2* __restrict__ psi,
                                                          double2* __restrict__ hpsi, int nvec) {
    extern __shared__ __align__(16) unsigned char smem[];
    int tile, v, chunk;
    if (!star_place(w, nvec, blockIdx.x, tile, v, chunk)) return;
    const long long off = (long long)v * g.N;
    star_body<N, D, B>(g, t, sd, w, psi + off, hpsi + off, tile, chunk * w.steps, smem);
}

template <int D, int NP>
__global__ void __launch_bounds__(kStencilThreads) k_stencil(DevGeom g, DevTabs t, StencilDesc sd,
                                                             const double2* __restrict__ psi,
                                                             double2* __restrict__ hpsi, int nvec, int vb) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tile = stencil_tile(blockIdx.x, sd.tile_row);
    if ((long long)tile * blockDim.x >= g.N) return;
    const int v0 = blockIdx.y * vb;
    stencil_body<D, NP>(g, t, sd, psi, hpsi, tile, v0, min(nvec, v0 + vb), reinterpret_cast<int4*>(smem));
}

// ---------------------------------------------------------------------------
// ragged batches: the items of one kernel's kind in one launch whose grid does
// not depend on the counts (a captured graph of it stays valid); workgroups
// stride over the items' workgroups, start[i] being item i's first.  The
// grid and every start are multiples of 8, so the dealing over XCDs holds.
// ---------------------------------------------------------------------------

__device__ __forceinline__ int few_item(const int* __restrict__ start, int B, int w) {
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Items and calls are not written while a launch reads them, and as constant
// memory their fields can stay in registers across a workgroup's stores.  As
// plain memory they were read again after every store (a sweep of eight windows
// with 1 to 8 vectors 191 -> 181 us).
template <typename T>
__device__ __forceinline__ const T& constant_item(const T* items, int i) {
    typedef const __attribute__((address_space(4))) T* ConstantItems;
    return *(const T*)((ConstantItems)(unsigned long long)items + i);
}

template <int N, int D>
__global__ void __launch_bounds__(star_threads(N)) k_batch_star(const FewItem* __restrict__ items,
                                                                const FewCall* __restrict__ calls,
                                                                const int* __restrict__ start, int B) {
    extern __shared__ __align__(16) unsigned char smem[];
    for (int w = blockIdx.x; w < start[B]; w += gridDim.x) {
        const int i = few_item(start, B, w);
        const FewItem& it = constant_item(items, i);
        const FewCall& c = constant_item(calls, i);
        int tile, v, chunk;
        const int local = w - start[i];
        if (!star_place(c.w, c.nvec, (local & ~7) | ((local + c.rot) & 7), tile, v, chunk)) continue;
        const long long off = (long long)v * it.g.N;
        __syncthreads();  // the previous item's LDS is no longer read
        star_body<N, D, 1>(it.g, it.t, it.sd, c.w, c.psi + off, c.hpsi + off, tile, chunk * c.w.steps, smem);
    }
}

// NP = 0: items of any number of pairs
template <int D, int NP>
__global__ void __launch_bounds__(kStencilThreads) k_batch_stencil(const FewItem* __restrict__ items,
                                                                   const FewCall* __restrict__ calls,
                                                                   const int* __restrict__ start, int B) {
    extern __shared__ __align__(16) unsigned char smem[];
    for (int w = blockIdx.x; w < start[B]; w += gridDim.x) {
        const int i = few_item(start, B, w);
        const FewItem& it = constant_item(items, i);
        const FewCall& c = constant_item(calls, i);
        const int local = w - start[i], vg = local / c.gx;
        const int tile = stencil_tile(local - vg * c.gx, it.sd.tile_row);
        if ((long long)tile * kStencilThreads >= it.g.N) continue;
        const int v0 = vg * c.vb, v1 = min(c.nvec, v0 + c.vb);
        int4* tab = reinterpret_cast<int4*>(smem);
        __syncthreads();
        if constexpr (NP > 0) {
            stencil_body<D, NP>(it.g, it.t, it.sd, c.psi, c.hpsi, tile, v0, v1, tab);
        } else {
            switch (it.sd.np) {
#define IWFPM_CASE(np_) \
    case np_: stencil_body<D, np_>(it.g, it.t, it.sd, c.psi, c.hpsi, tile, v0, v1, tab); break;
                IWFPM_STENCIL_PAIRS(IWFPM_CASE)
#undef IWFPM_CASE
            }
        }
    }
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------

constexpr int kMaxLds = 160 * 1024;
constexpr long long kMaxGridThreads = 1LL << 31;

template <int N, int D, int B>
size_t star_rows(const DevGeom& g, const StarDesc& w, int steps) {
    constexpr int BW = B + (StarShape<N, D>::F == 2 ? 2 : 0);
    return sizeof(StarRow<N, D>) * (steps + 2) * BW * stencil_slices(g, w.planes * w.plane);
}
template <int N, int D, int B>
size_t star_lds(const DevGeom& g, const StarDesc& w, int steps) {
    return (size_t)2 * B * star_block(w) * 16 + star_rows<N, D, B>(g, w, steps);
}

// The walk of one launch with `total` points (all its vectors, or all plans
// of a batch): planes to about 512 threads, and the longest walk (the two
// extra steps that it reads at its ends cost least) that still gives the
// chip kStarBlocks workgroups.  Measured on 24^2 x 32^2 points, walks of
// 2 / 4 / 8 / 16: 1 vector 6.7 / 6.6 / 9.1 / 14.9 us, 3 vectors 19.1 / 15.3 /
// 14.2 / 15.4 us, 16 vectors 76.8 / 59.1 / 52.9 / 52.2 us.  On 16^6 a
// walk of 16 loses to 8 (530 against 497 us, 3 vectors): its window on the
// slowest axis no longer shares the last-level cache with its neighbours'.
constexpr int kStarBlocks = 320;
template <int N, int D, int B>
StarDesc star_config(const DevGeom& g, StarDesc w, double total) {
    using Sh = StarShape<N, D>;
    const int nplanes = g.stride[Sh::F - 1] / w.plane;
    w.planes = std::max(1, std::min(nplanes, 512 / w.plane));
    while (B == 1 && w.planes > 1 && star_lds<N, D, B>(g, w, 16) > 64 * 1024) w.planes /= 2;
    w.ptiles = (nplanes + w.planes - 1) / w.planes;
    w.tiles = w.ptiles * (Sh::F == 2 ? (g.ext[1] + B - 1) / B : 1);
    w.whole = w.tiles <= 128;  // about the workgroups that an XCD holds at once
    w.steps = B > 1 ? 16 : (N == 6 ? 8 : 16);
    const double per_step = w.tiles * (double)g.ext[0] * (total / g.N);  // one-step workgroups
    while (w.steps > 2 && (w.steps > g.ext[0] || per_step / w.steps < kStarBlocks)) w.steps /= 2;
    w.steps = std::min(w.steps, g.ext[0]);
    w.chunks = (g.ext[0] + w.steps - 1) / w.steps;
    return w;
}

template <int N, int D, int B>
hipError_t launch_star_t(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, const StarDesc& w,
                         const double2* psi, double2* hpsi, int nvec, hipStream_t st) {
    const int T = star_block(w);
    const int nv = (int)std::max<long long>(1, std::min<long long>(nvec, kMaxGridThreads / T / star_blocks(w, 8) * 8));
    for (int v = 0; v < nvec; v += nv) {
        const int n = std::min(nv, nvec - v);
        k_star<N, D, B><<<dim3(star_blocks(w, n)), T, star_lds<N, D, B>(g, w, w.steps), st>>>(
            g, t, sd, w, psi + (size_t)v * g.N, hpsi + (size_t)v * g.N, n);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Four points of axis 1 per thread: half of that axis' neighbours, which come
// from beyond the L2 on grids of this kind, are then a thread's own (16^6, 8
// vectors: 1.21 against 1.31 ms; 40^3 x 8^3, 2 vectors: 0.57 against 0.64
// ms).  It takes the longest walk and enough of the 209-register workgroups;
// extents that 4 does not divide waste lanes (20^2 x 10^2 ...: 142 against
// 127 us), and in window order the rotations cost more than it saves (549
// against 511 us on 16^6, 3 vectors).
template <int N, int D>
hipError_t launch_star(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, const StarDesc& w0,
                       const double2* psi, double2* hpsi, int nvec, hipStream_t st) {
    const double total = (double)g.N * nvec;
    if constexpr (N == 6) {
        if (!g.order && g.ext[1] % 4 == 0 && g.ext[0] >= 16) {
            const StarDesc w = star_config<N, D, 4>(g, w0, total);
            if (w.steps == 16 && star_blocks(w, nvec) >= 512 && star_lds<N, D, 4>(g, w, w.steps) <= kMaxLds)
                return launch_star_t<N, D, 4>(g, t, sd, w, psi, hpsi, nvec, st);
        }
    }
    return launch_star_t<N, D, 1>(g, t, sd, star_config<N, D, 1>(g, w0, total), psi, hpsi, nvec, st);
}

// vectors per workgroup of the point kernel: up to 4 share the neighbour
// positions (24^2 x 32^2 points, 4 pairs off the axes, 16 vectors: 129 / 93 /
// 86 us with 1 / 2 / 4) as long as the chip stays full, and one where the planes
// of several vectors would crowd each other out of the last-level cache (16^6,
// 3 vectors: 934 / 1008 / 1104 us)
int stencil_vb(const DevGeom& g, double total) {
    if ((double)g.stride[0] * 16 * 3 * 2 > 64e6) return 1;
    for (int vb = 4; vb > 1; vb /= 2)
        if (total / kStencilThreads / vb >= 1024) return vb;
    return 1;
}
int stencil_gx(const DevGeom& g, const StencilDesc& sd) {
    const int tiles = (g.N + kStencilThreads - 1) / kStencilThreads, row = 8 * sd.tile_row;
    return (tiles + row - 1) / row * row;
}

template <int D, int NP>
hipError_t launch_points(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, const double2* psi, double2* hpsi,
                         int nvec, hipStream_t st) {
    const int vb = std::min(stencil_vb(g, (double)g.N * nvec), nvec), nv = 65535 * vb;
    for (int v = 0; v < nvec; v += nv) {
        const int n = std::min(nv, nvec - v);
        k_stencil<D, NP><<<dim3(stencil_gx(g, sd), (n + vb - 1) / vb), kStencilThreads, stencil_lds(g, sd), st>>>(
            g, t, sd, psi + (size_t)v * g.N, hpsi + (size_t)v * g.N, n, vb);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// workgroups of a kernel that the device holds at once, a multiple of 8
template <typename F>
hipError_t resident(F* kernel, int threads, size_t lds, int* out) {
    int per_cu = 0, dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds);
    *out = std::max(1, per_cu) * std::max(8, cus / 8 * 8);
    return e;
}

}  // namespace

bool star_supported(int n, int d) {
    return (n == 2 && d == 1) || (n == 3 && d == 2) || (n == 4 && d == 2) || (n == 6 && d == 3);
}

// Small launches take the point kernel: below some 32k points both are a few
// microseconds of latency, and the walk has to fill its tables first (512
// points: 3.6 against 3.7 us, 14,400 points: 4.4 against 5.2 us).
static bool star_pays(const StarDesc& w, double total) { return w.ok && total >= 32768; }

hipError_t launch_stencil(const DevGeom& g, const DevTabs& t, const StencilDesc& sd, const StarDesc& w,
                          const void* psi, void* hpsi, int nvec, hipStream_t st) {
    const double2* x = reinterpret_cast<const double2*>(psi);
    double2* y = reinterpret_cast<double2*>(hpsi);
    if (star_pays(w, (double)g.N * nvec)) {
        if (g.n == 2) return launch_star<2, 1>(g, t, sd, w, x, y, nvec, st);
        if (g.n == 3) return launch_star<3, 2>(g, t, sd, w, x, y, nvec, st);
        if (g.n == 4) return launch_star<4, 2>(g, t, sd, w, x, y, nvec, st);
        return launch_star<6, 3>(g, t, sd, w, x, y, nvec, st);
    }
#define IWFPM_CASE(np_)                                                       \
    if (sd.np == np_) {                                                       \
        if (g.d == 1) return launch_points<1, np_>(g, t, sd, x, y, nvec, st); \
        if (g.d == 2) return launch_points<2, np_>(g, t, sd, x, y, nvec, st); \
        return launch_points<3, np_>(g, t, sd, x, y, nvec, st);               \
    }
    IWFPM_STENCIL_PAIRS(IWFPM_CASE)
#undef IWFPM_CASE
    return hipErrorInvalidValue;
}

hipError_t prepare_stencil() {
    return hipFuncSetAttribute((const void*)k_star<6, 3, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
}

int few_kind(const DevGeom& g, const StencilDesc& sd, const StarDesc& w) {
    return w.ok ? g.n : 100 * g.d + sd.np;
}

int few_blocks(const FewItem& it, FewCall& c, double total) {
    if (c.nvec == 0) return 0;
    const DevGeom& g = it.g;
    if (it.w.ok) {
        if (g.n == 2) c.w = star_config<2, 1, 1>(g, it.w, total);
        else if (g.n == 3) c.w = star_config<3, 2, 1>(g, it.w, total);
        else if (g.n == 4) c.w = star_config<4, 2, 1>(g, it.w, total);
        else c.w = star_config<6, 3, 1>(g, it.w, total);
        return star_blocks(c.w, c.nvec);
    }
    c.vb = std::min(stencil_vb(g, total), c.nvec);
    c.gx = stencil_gx(g, it.sd);
    return c.gx * ((c.nvec + c.vb - 1) / c.vb);
}

// threads that the plan's star workgroups have, and the LDS of their rows on
// the longest walk
template <int N, int D>
static void star_need(const FewItem& it, int* threads, size_t* rows) {
    const StarDesc w = star_config<N, D, 1>(it.g, it.w, 1e18);
    *threads = std::max(*threads, star_block(w));
    *rows = std::max(*rows, star_rows<N, D, 1>(it.g, w, 16));
}

// the kernel of a kind, for a launch or an occupancy query
template <typename F>
static hipError_t with_batch_kernel(int kind, F&& f) {
    switch (kind) {
        case 2: return f(k_batch_star<2, 1>);
        case 3: return f(k_batch_star<3, 2>);
        case 4: return f(k_batch_star<4, 2>);
        case 6: return f(k_batch_star<6, 3>);
#define IWFPM_CASE(np_)                                    \
        case 100 + np_: return f(k_batch_stencil<1, np_>); \
        case 200 + np_: return f(k_batch_stencil<2, np_>); \
        case 300 + np_: return f(k_batch_stencil<3, np_>);
        IWFPM_STENCIL_PAIRS(IWFPM_CASE)
#undef IWFPM_CASE
        case 1001: return f(k_batch_stencil<1, 0>);
        case 1002: return f(k_batch_stencil<2, 0>);
        case 1003: return f(k_batch_stencil<3, 0>);
        default: return hipErrorInvalidValue;
    }
}

hipError_t few_launch_config(FewLaunch& l, const FewItem* items, int B) {
    l.threads = 64;
    l.lds = 0;
    for (int i = 0; i < B; ++i) {
        const FewItem& it = items[i];
        if (it.kind != l.kind) continue;
        if (!it.w.ok) {
            l.threads = kStencilThreads;
            l.lds = std::max(l.lds, stencil_lds(it.g, it.sd));
        } else if (it.g.n == 2) star_need<2, 1>(it, &l.threads, &l.lds);
        else if (it.g.n == 3) star_need<3, 2>(it, &l.threads, &l.lds);
        else if (it.g.n == 4) star_need<4, 2>(it, &l.threads, &l.lds);
        else star_need<6, 3>(it, &l.threads, &l.lds);
    }
    if (l.kind < 100) l.lds += (size_t)2 * l.threads * 16;  // the planes' copies
    return with_batch_kernel(l.kind, [&](auto* k) {
        hipError_t e = hipSuccess;
        if (l.lds > 64 * 1024) e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
        return e == hipSuccess ? resident(k, l.threads, l.lds, &l.grid) : e;
    });
}

hipError_t launch_few_batch(const FewLaunch& l, const FewItem* items, const FewCall* calls, const int* start, int B,
                            hipStream_t st) {
    return with_batch_kernel(l.kind, [&](auto* k) {
        k<<<dim3(l.grid), l.threads, l.lds, st>>>(items, calls, start, B);
        return hipGetLastError();
    });
}

}  // namespace iwfpm
