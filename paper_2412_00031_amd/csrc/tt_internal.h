// tt_internal.h -- library-private types and device helpers of libtt.
//
// Numerics (Chen et al., TomoATT, arXiv 2412.00031; Sec. 2.1 Eq. (4), Sec. 3.1):
//   T = T0 * tau with T0 = s0 sqrt(d^T M0^{-1} d), d = x - x_s in the source's
//   local (r^, theta^, phi^) frame; scaled gradient p = (dT/dr, dT/dtheta / r,
//   dT/dphi / (r cos theta)); Lax-Friedrichs update of the factored equation
//   with viscosity sigma_a = kappa T0 g_a.  Everything in FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>
#include <vector>

#include "tt.h"

namespace tt {

// Record a printf-style message for tt_last_error() and return `code`.
int fail(int code, const char* fmt, ...);

constexpr int kBI = 8;        // column block of one wave: 8 x 8 (i, j) columns
constexpr int kBJ = 8;
constexpr int kWave = 64;
constexpr int kBndThreads = 256;
constexpr int kMaxTileK = 62;  // k-extent of a forward sweep tile; the staged column (tk + 2) fits one wave
constexpr int kLineDepth = 16;  // nodes of a line: the depth of the forward sweeps' slabs of whole lines

// Kernel-argument copy of the grid.
struct Geo {
    int n[3];          // nodes per axis
    int m[3];          // interior nodes per axis (n - 2)
    int coord;         // 0 Cartesian, 1 spherical
    int nt[2];         // tile columns along i' and j'
    int tk;            // hyperplane steps of a tile (its extent along u = i' + j' + k')
    int ncols;         // tile columns: nt0 * nt1
    long long N;       // n0 * n1 * n2
    long long si, sj;  // strides of axes 0 and 1 of the solution fields (axis 2 has stride 1)
    long long Nf;      // elements of a solution field: N, or more if its rows are padded to whole lines
    long long NB;      // boundary nodes
    int W;             // n1 + n2 - 1: width of the row-coalesced layouts
    int n1p;           // aligned layouts: row pitch (a multiple of 8 records, >= n1 + 7)
    int joff[2];       // aligned layouts: record offset of j in a row for sweeps with s1 > 0, s1 < 0
    long long Sa;      // records per aligned layout: n0 * W * n1p
    double o[3], h[3], inv2h[3], invh[3];
};

// Sheared sweep tiles.  In sweep-relative interior coordinates (i', j', k')
// a tile is the 8 x 8 (i', j') tile column (TI, TJ) intersected with the slab
// TK tk <= u < (TK + 1) tk of the hyperplane index u = i' + j' + k'.  Tile column
// TI + TJ = s spans u in [8 s, 8 s + 14 + m2) (full columns; ragged ones end
// earlier), i.e. slabs lo(s)..hi(s).  A tile reads its upstream neighbours'
// nodes at u - 1 (slabs TK - 1 and TK of the neighbouring columns) and its
// downstream ones' old values at u + 1 (slabs TK and TK + 1): it may start once
// slab TK of the two upstream columns and its own slab TK - 1 are done, and a
// downstream column cannot overwrite what it reads before it is done itself.
__host__ __device__ inline int col_tile_lo(const Geo& G, int s) { return (kBI * s) / G.tk; }
__host__ __device__ inline int col_tile_hi(const Geo& G, int s) {
    return (kBI * s + (kBI - 1) + (kBJ - 1) + G.m[2] - 1) / G.tk;
}
// tile columns with TI + TJ = s
__host__ __device__ inline int diag_first(const Geo& G, int s) { return s - (G.nt[1] - 1) > 0 ? s - (G.nt[1] - 1) : 0; }
__host__ __device__ inline int diag_count(const Geo& G, int s) {
    const int hi = s < G.nt[0] - 1 ? s : G.nt[0] - 1;
    return hi - diag_first(G, s) + 1;
}
// tile column number b in [0, ncols): columns ordered by TI + TJ, then TI, so
// that both upstream neighbours of a column have lower numbers
__host__ __device__ inline void col_decode(const Geo& G, int b, int& TI, int& TJ) {
    int s = 0;
    for (; s < G.nt[0] + G.nt[1] - 2; ++s) {
        const int c = diag_count(G, s);
        if (b < c) break;
        b -= c;
    }
    TI = diag_first(G, s) + b;
    TJ = s - TI;
}
// LDS doubles per staged column: the tk + 2 entries, rounded up to an even
// count (the window is staged two doubles per lane and load)
__host__ __device__ inline int tile_pitch(int tk) { return (tk + 3) & ~1; }

// Per-source constants, produced on the device by k_src_setup.
struct Src {
    double Xs[3];      // source position in the embedding (spherical) or (z,y,x)
    double E[9];       // rows: source-frame unit vectors r^_s, theta^_s, phi^_s
    double mi11, mi12, mi22;  // lower-right block of M0^{-1}
    double s0;
    double rh;         // distance from the axis, r cos theta (spherical)
    double rhl, zl;    // what rounding left out of rh and of Xs[2]
    int fb[3];         // base corner of the fixed cell
    int pad;
};

// Per-axis tables, built on the device by k_tables into the caller's workspace.
//   tab0[i]  = r (spherical) or z (Cartesian)
//   tab1[j]  = (cos theta, sin theta) (spherical) or (y, 0) (Cartesian)
//   tab2[k]  = (cos phi, sin phi) (spherical) or (x, 0) (Cartesian)
struct Tabs {
    const double* t0;
    const double2* t1;
    const double2* t2;
};

// Lane-constant geometry of an (i, j) column.
struct Col {
    double x0;         // r or z
    double ct, st;     // cos/sin latitude (spherical), y in ct (Cartesian)
    double rct;        // r cos theta
    double g1, g2;     // scaled-gradient factors of axes 1, 2 (g0 = 1)
};

__device__ __forceinline__ Col make_col(const Geo& G, const Tabs& T, int i, int j) {
    Col c;
    c.x0 = T.t0[i];
    double2 a1 = T.t1[j];
    c.ct = a1.x;
    c.st = a1.y;
    if (G.coord == 1) {
        c.rct = c.x0 * c.ct;
        c.g1 = 1.0 / c.x0;
        c.g2 = 1.0 / c.rct;
    } else {
        c.rct = 0.0;
        c.g1 = c.g2 = 1.0;
    }
    return c;
}

__device__ __forceinline__ bool in_fixed(const Src& S, int i, int j, int k) {
    return (unsigned)(i - S.fb[0]) <= 1u && (unsigned)(j - S.fb[1]) <= 1u && (unsigned)(k - S.fb[2]) <= 1u;
}

// 1/sqrt(x) for x > 0 to about an ulp: the hardware estimate (good to about
// 23 bits) refined by two Newton steps y <- y (3 - x y^2) / 2.
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    y *= fma(-h * y, y, 1.5);
    y *= fma(-h * y, y, 1.5);
    return y;
}

// T0 and its scaled gradient t at a node of column c with axis-2 table value
// (c2, s2) = (cos phi, sin phi) or (x, 0); zeros at the source itself, where the
// factor vanishes.
template <int COORD>
__device__ __forceinline__ void factor(const Src& S, const Col& c, double c2, double s2, double& T0, double t[3]) {
    double d0, d1, d2;
    if (COORD == 1) {
        // (one rounding each, whichever of the products the caller keeps over a loop)
        double D0 = fma(c.rct, c2, -S.Xs[0]);
        double D1 = fma(c.rct, s2, -S.Xs[1]);
        double D2 = fma(c.x0, c.st, -S.Xs[2]);
        d0 = D0 * S.E[0] + D1 * S.E[1] + D2 * S.E[2];
        d1 = D0 * S.E[3] + D1 * S.E[4] + D2 * S.E[5];
        d2 = D0 * S.E[6] + D1 * S.E[7] + D2 * S.E[8];
    } else {
        d0 = c.x0 - S.Xs[0];
        d1 = c.ct - S.Xs[1];
        d2 = c2 - S.Xs[2];
    }
    double m0 = d0;
    double m1 = S.mi11 * d1 + S.mi12 * d2;
    double m2 = S.mi12 * d1 + S.mi22 * d2;
    double Q = d0 * m0 + d1 * m1 + d2 * m2;
    if (!(Q > 0.0)) {
        T0 = 0.0;
        t[0] = t[1] = t[2] = 0.0;
        return;
    }
    const double rq = rsqrt_nr(Q);
    T0 = S.s0 * (Q * rq);
    double f = S.s0 * rq;
    if (COORD == 1) {
        // gradient in the embedding, then on the node's local unit vectors
        // r^ = (ct c2, ct s2, st), theta^ = (-st c2, -st s2, ct), phi^ = (-s2, c2, 0)
        double G0 = f * (m0 * S.E[0] + m1 * S.E[3] + m2 * S.E[6]);
        double G1 = f * (m0 * S.E[1] + m1 * S.E[4] + m2 * S.E[7]);
        double G2 = f * (m0 * S.E[2] + m1 * S.E[5] + m2 * S.E[8]);
        double hz = G0 * c2 + G1 * s2;
        t[0] = c.ct * hz + c.st * G2;
        t[1] = c.ct * G2 - c.st * hz;
        t[2] = G1 * c2 - G0 * s2;
    } else {
        t[0] = f * m0;
        t[1] = f * m1;
        t[2] = f * m2;
    }
}

// Local state of the factored Hamiltonian at an interior node: P, M P, H.
struct Loc {
    double T0, t[3], P[3], MP[3], H;
};

template <int COORD>
__device__ __forceinline__ void local_state(const Geo& G, const Src& S, const Col& c, double c2, double s2,
                                            double xi, double eta, double tx, double up0, double dn0,
                                            double up1, double dn1, double up2, double dn2, Loc& L) {
    // up_a = tau(x - e_a), dn_a = tau(x + e_a) in absolute axis directions
    factor<COORD>(S, c, c2, s2, L.T0, L.t);
    double q0 = (dn0 - up0) * G.inv2h[0];
    double q1 = c.g1 * (dn1 - up1) * G.inv2h[1];
    double q2 = c.g2 * (dn2 - up2) * G.inv2h[2];
    L.P[0] = L.T0 * q0 + tx * L.t[0];
    L.P[1] = L.T0 * q1 + tx * L.t[1];
    L.P[2] = L.T0 * q2 + tx * L.t[2];
    L.MP[0] = L.P[0];
    L.MP[1] = (1.0 - 2.0 * xi) * L.P[1] + 2.0 * eta * L.P[2];
    L.MP[2] = 2.0 * eta * L.P[1] + (1.0 + 2.0 * xi) * L.P[2];
    L.H = sqrt(L.P[0] * L.MP[0] + L.P[1] * L.MP[1] + L.P[2] * L.MP[2]);
}

// Lax-Friedrichs update: the tau(x) that zeroes
//   G_x = H(q, tau_old(x)) - sum_a sigma_a (dn_a - 2 tau(x) + up_a) / (2 h_a) - s(x),
// sigma_a = kappa T0 g_a.  With C = sum_a g_a / h_a (g_0 = 1) it reads
//   tau(x) = (s - H) / (kappa T0 C) + sum_a w_a (up_a + dn_a),  w_a = g_a / (2 h_a C),
// and 1 / (kappa T0 C) = rho / sqrt(Q) with rho = 1 / (kappa s0 C): LfCol holds
// the column's constants, so an update has no division.
//
// The factor enters through T0 = s0 Q rq and its scaled gradient t = s0 rq u
// (rq = 1 / sqrt(Q), u = m on the node's unit vectors, m = M0^{-1} d), so
// P_a = T0 q_a + tau t_a = s0 rq R_a with R_a = Q q_a + tau u_a and
// H = s0 rq sqrt(R . M R): the update forms R, not T0 and t.
//
// Neither d = E (X - Xs) nor u needs the embedding.  With ths the source's latitude
// and F, S the cosine and sine of the longitude difference, the horizontal direction
// of the node is (cos ths F, -sin ths F, S) in the source frame and the axis is
// (sin ths, cos ths, 0).  So with the column's distances D_r, D_z from the source,
// away from the axis and along it,
//   d_0 = cos ths (D_r + rct (F - 1)) + sin ths D_z,
//   d_1 = cos ths D_z - sin ths (D_r + rct (F - 1)),  d_2 = rct S,
// one operation each with column constants, and m is turned by the source's
// latitude, by the longitude difference and by the node's latitude th:
//   w = cos ths d_0 - sin ths m_1,  z = sin ths d_0 + cos ths m_1,
//   g = F w + S m_2,                u_2 = F m_2 - S w,
//   u_0 = cos th g + sin th z,      u_1 = cos th z - sin th g.
// F - 1 and S come from a table per source (k_lon), rounded once: F - 1 is small where
// d is, and what the source's own coordinates lose to rounding is kept beside them, so
// that nothing in d rounds at the Earth's radius (rms error of 12 iterations on 25^3 nodes
// at latitude 80 1.4e-16, 4.8e-16 with d from the rounded embedding, 6.4e-16 with one that
// is projected back).  3 and 12 operations; 6 and 16 with F and S formed in every update
// (101^3 x 7 forward 89.7 / 93.0 ms, 61^3 x 17 29.7 / 31.1); u_1 from u_0 by a division by
// cos th is one operation cheaper still but has 4 times the error at 86 degrees.
//
// The average of the neighbours sum_a w_a p_a, p_a = up_a + dn_a, has weights of sum
// 1/2 that add up to it in doubles only nearly; what they miss shifts every node the
// same way.  Formed as p_0 / 2 + w_1 (p_1 - p_0) + w_2 (p_2 - p_0) nothing is missed:
// error of a 12-iteration solve on 25^3 Cartesian nodes 1.2e-16, was 1.06e-15.
struct LfCol {
    double v1, v2;      // g_a / (2 h_a) of axes 1, 2 (central differences)
    double w1, w2;      // averaging weights w_a
    double rho;
    double ct, st;      // the column's latitude (spherical)
    double rct, A[2], C[2];  // d along the column: d_i = A_i (F - 1) + C_i (spherical); Cartesian: C = (x0, y) - Xs
};

template <int COORD>
__device__ __forceinline__ LfCol lf_col(const Geo& G, const Src& S, const Col& c, double kappa) {
    LfCol W;
    const double iC = 1.0 / (G.invh[0] + c.g1 * G.invh[1] + c.g2 * G.invh[2]);
    W.v1 = c.g1 * G.inv2h[1];
    W.v2 = c.g2 * G.inv2h[2];
    W.w1 = W.v1 * iC;
    W.w2 = W.v2 * iC;
    W.rho = iC / (kappa * S.s0);
    W.ct = c.ct;
    W.st = c.st;
    if (COORD == 1) {
        const double sts = S.E[2], cts = S.E[5];
        const double Dr = fma(c.x0, c.ct, -S.rh) - S.rhl, Dz = fma(c.x0, c.st, -S.Xs[2]) - S.zl;
        W.rct = c.rct;
        W.A[0] = c.rct * cts;
        W.A[1] = -(c.rct * sts);
        W.C[0] = fma(Dr, cts, Dz * sts);
        W.C[1] = fma(Dz, cts, -(Dr * sts));
    } else {
        W.rct = W.A[0] = W.A[1] = 0.0;
        W.C[0] = c.x0 - S.Xs[0];
        W.C[1] = c.ct - S.Xs[1];
    }
    return W;
}

// 1 / sqrt(x) and sqrt(x) for normal x > 0 from the hardware estimate y (good
// to about 2^-23) by one third-order step: with e = 1 - x y^2 the root is
// y (1 - e)^(-1/2) = y (1 + e (1/2 + 3/8 e)) + O(e^3), e^3 ~ 2^-67.
__device__ __forceinline__ double rsqrt_3(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y, e * fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ double sqrt_3(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double t = x * y;
    const double e = fma(-t, y, 1.0);
    return fma(t, e * fma(0.375, e, 0.5), t);
}

// (f1, sn) = (F - 1, S), or (distance along axis 2, 0).
// (every contraction is spelled out: all instances round alike)
template <int COORD>
__device__ __forceinline__ double lf_update(const Geo& G, const Src& S, const LfCol& W, double f1, double sn, double sx,
                                            double ma, double mb, double mc, double tx, double up0, double dn0,
                                            double up1, double dn1, double up2, double dn2) {
    double d0, d1, d2;
    if (COORD == 1) {
        d0 = fma(f1, W.A[0], W.C[0]);
        d1 = fma(f1, W.A[1], W.C[1]);
        d2 = W.rct * sn;
    } else {
        d0 = W.C[0];
        d1 = W.C[1];
        d2 = f1;
    }
    const double m1 = fma(S.mi11, d1, S.mi12 * d2);
    const double m2 = fma(S.mi12, d1, S.mi22 * d2);
    const double Q = fma(d2, m2, fma(d1, m1, d0 * d0));  // > 0: the sweeps skip the fixed cell
    const double rq = rsqrt_3(Q);
    double u0, u1, u2;
    if (COORD == 1) {
        const double sts = S.E[2], cts = S.E[5];
        const double w = fma(cts, d0, -sts * m1), z = fma(sts, d0, cts * m1);
        const double g = fma(f1, w, fma(sn, m2, w));
        u0 = fma(W.ct, g, W.st * z);
        u1 = fma(W.ct, z, -W.st * g);
        u2 = fma(f1, m2, fma(-sn, w, m2));
    } else {
        u0 = d0;
        u1 = m1;
        u2 = m2;
    }
    const double R0 = fma(Q, (dn0 - up0) * G.inv2h[0], tx * u0);
    const double R1 = fma(Q, (dn1 - up1) * W.v1, tx * u1);
    const double R2 = fma(Q, (dn2 - up2) * W.v2, tx * u2);
    // (ma, mb, mc) = (1 - 2 xi, 2 eta, 1 + 2 xi): the lower-right block of M
    const double MR1 = fma(ma, R1, mb * R2);
    const double MR2 = fma(mb, R1, mc * R2);
    // (+ DBL_MIN: the root of 0 stays finite; Hamiltonians that small do not occur)
    const double V = fma(R2, MR2, fma(R1, MR1, fma(R0, R0, 2.2250738585072014e-308)));
    const double f = fma(-(S.s0 * rq), sqrt_3(V), sx);  // s - H
    const double p0 = up0 + dn0;
    return fma(f, W.rho * rq, fma((up2 + dn2) - p0, W.w2, fma((up1 + dn1) - p0, W.w1, 0.5 * p0)));
}

// ----- state of one batched solve (host side) -----
struct Plan {
    Geo G;
    Tabs T;
    int nsrc = 0;
    int nbblocks = 0;         // boundary-pass blocks per source
    int nslots = 0;           // 8-byte slots per source in part (see SweepArgs)
    double kappa = 1.0, tol = 1e-6;
    int max_iter = 1;         // iteration budget of this group
    int hist_stride = 1;      // row length of eps_hist (the call's max_iter)
    double* eps_hist = nullptr;
    // workspace views
    Src* src = nullptr;
    double* tab0 = nullptr;
    double2* tab1 = nullptr;
    double2* tab2 = nullptr;
    double2* lon = nullptr;   // forward: longitude differences [nsrc][n2] (k_lon)
    int* active = nullptr;
    int* iter = nullptr;
    int* counter = nullptr;
    double* part = nullptr;
    double* part2 = nullptr;
    double* coef = nullptr;   // adjoint: [nsrc][4][Sa][6] (line-aligned row-coalesced layouts) or [nsrc][N][6]
    double* diag = nullptr;   // adjoint: diagonal of each node's row [nsrc][N]
    double* rhs = nullptr;    // adjoint: right-hand side divided by the diagonal [nsrc][N]
    int* box = nullptr;       // adjoint: index box of each source's nonzero rhs [nsrc][6]
    double* model = nullptr;  // forward: [4][Sa][4] = (s, 1 - 2 xi, 2 eta, 1 + 2 xi) (aligned row-coalesced layouts)
    double* pad = nullptr;    // forward: the solution fields with padded rows, [nsrc][Nf], if Nf != N
    double* bnd_in = nullptr; // adjoint: [nsrc][NB] (continuous adjoint: boundary pass scratch)
    double* bnd_rhs = nullptr; // adjoint: right-hand side of the boundary nodes, [nsrc][NB]
    double2* bnd_rec = nullptr;  // continuous adjoint: the boundary nodes' records, [nsrc][3][NB], in place of diag
    bool continuous = false;  // adjoint: upwind discretisation of Eq. (5) instead of the exact transpose
    bool compact = false;     // adjoint: one node-order copy of the coefficient records
    // optional timing of the sweep kernels: an event pair around the
    // launches of each directional sweep, with the launch count
    std::vector<std::pair<std::pair<hipEvent_t, hipEvent_t>, int>>* timing = nullptr;
};

// Kernel-argument bundle of the sweep kernels.
struct SweepArgs {
    Geo G;
    Tabs T;
    const double *s, *xi, *eta;
    const Src* src;
    const double2* lon;     // forward: (cos - 1, sin) of the longitude difference or (x - x_s, 0), [nsrc][n2]
    double* field;          // tau or lambda [nsrc][Nf]
    const double* coef;     // adjoint coefficients [nsrc][4][Sa][6], or [nsrc][N][6] when compact
    const double* rhs;      // adjoint right-hand side / diagonal [nsrc][N]
    const int* box;         // [nsrc][6]: i, j, k ranges of the nonzero rhs (empty: lo > hi)
    const double* model;    // forward model records [4][Sa][4]
    const double* bnd_in;   // adjoint face couplings [nsrc][NB]
    const double* bnd_rhs;  // adjoint right-hand side of the boundary nodes [nsrc][NB]
    int* active;
    int* iter;
    int32_t* status;
    // per source nslots 8-byte slots: the convergence sums of the ncols tile
    // columns and nbblocks boundary blocks over the iteration's directions so
    // far, the columns' sweep progress (ncols 64-bit words), the ticket and
    // owner words of the source's work queue (sweep_claim), and its lost word
    double* part;
    double* part2;          // adjoint: sums of |lambda| in the last direction, same first two ranges
    int* counter;
    double* eps_hist;       // optional [nsrc][hist_stride]
    int nslots, nbblocks, nsrc, max_iter, hist_stride;
    int compact;            // adjoint records in node order (TT_FLAG_COMPACT_ADJOINT)
    int kfaces;             // adjoint: the sweeps set the nodes on a k face only (not the continuous system's)
    double kappa, tol;
};

SweepArgs make_args(const Plan& P, const double* s, const double* xi, const double* eta, double* field,
                    int32_t* status);
void launch_tables(const Plan& P, hipStream_t st);
void launch_src_setup(const Plan& P, const double* src_pos, const double* src_par, hipStream_t st);
void launch_source_params(const Geo& G, const double* s, const double* xi, const double* eta,
                          const double* src_pos, double* src_par, int nsrc, hipStream_t st);
void launch_fwd_init(const Plan& P, const SweepArgs& a, const double* tau_init, const double* s, const double* xi,
                     const double* eta, hipStream_t st);
void launch_fwd_iteration(const Plan& P, const SweepArgs& a, hipStream_t st);
void launch_adj_init(const Plan& P, const SweepArgs& a, const double* tau, int nrec, const double* rec_pos,
                     const double* R, const double* init, hipStream_t st);
void launch_adj_iteration(const Plan& P, const SweepArgs& a, hipStream_t st);
void launch_unpad(const Plan& P, double* tau, hipStream_t st);
void launch_cadj_scale(const Plan& P, const double* s, double* lam, hipStream_t st);
void launch_sample(const Plan& P, const double* tau, int nrec, const double* rec_pos, double* out,
                   hipStream_t st);
void launch_fill(double* p, long long n, double v, hipStream_t st);
void launch_reloc_times(const Plan& P, const double* tau, int nev, const double* ev, const double* t0, double* out,
                        hipStream_t st);
void launch_reloc_kernel(const Plan& P, const double* tau, int nev, const double* ev, const double* R, double* K,
                         hipStream_t st);
void launch_misfit(int nsrc, int nrec, const double* T, const double* Tobs, const double* w, int npair,
                   const int32_t* pairs, const double* wpair, double alpha, double beta, double* R,
                   double* chi, hipStream_t st);
void launch_misfit_cr(int nsrc, int nrec, const double* T, const double* Tobs, const int32_t* off, const int32_t* pair,
                      const double* wcr, double gamma, double* R, double* chi, hipStream_t st);
// Inversion grids of the multiple-grid parameterisation, flattened for kernel
// arguments: sizes, offsets of each grid's axis coordinates in the
// concatenated coords array, and running sums of m2, m1*m2 and 3*m0*m1*m2.
struct MgGrids {
    int H;
    int ncoord;  // total coordinates of all grids
    int m[TT_MG_MAX_GRIDS][3];
    int coff[TT_MG_MAX_GRIDS][3];
    int s2off[TT_MG_MAX_GRIDS + 1];
    int s12off[TT_MG_MAX_GRIDS + 1];
    long long outoff[TT_MG_MAX_GRIDS + 1];
};

// Projection plan: the separable staged form when its LDS fits, with nch
// row chunks per plane and ws_bytes of partial sums; else one wave per node.
constexpr long long kMgMaxLds = 60 * 1024;  // dynamic LDS of the staged forms (static LDS comes on top)
constexpr long long kMgCoordLds = 32 * 1024;  // coordinates staged in LDS up to this size
struct MgPlan {
    bool separable;
    int nch;
    size_t lds;
    size_t ws_bytes;
};

MgGrids make_mg(int H, const int* m);
MgPlan plan_mg_project(const Geo& G, const MgGrids& Q);
void launch_mg_project(const Geo& G, int H, const int* m, const double* coords, const double* K, double* out,
                       double* ws, hipStream_t st);
void launch_mg_expand(const Geo& G, int H, const int* m, const double* coords, const double* C, double* field,
                      hipStream_t st);
void launch_kernel_density(const Geo& G, const double* s, const double* dens, const double* grad, double eps,
                           double zeta, double* K, double* Kd, hipStream_t st);
void launch_kernel_accum(const Plan& P, const double* xi, const double* eta, const double* tau,
                         const double* lam, double* grad, int accumulate, hipStream_t st);

}  // namespace tt
