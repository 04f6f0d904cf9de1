// tt_kernels.hip -- CDNA4 (gfx950) kernels of libtt.
//
// Sweep schedule.  One directional sweep must visit the interior nodes in an
// order where x - sigma_a e_a precedes x on every axis a (the Gauss-Seidel
// order of fast sweeping, Sec. 3.1).  The stencil touches only axis neighbours
// and boundary nodes are not written during a sweep, so every such order yields
// the same numbers as the lexicographic one; the hyperplane-stepping idea of
// Sec. 3.4 (nodes with i'+j'+k' = L are independent) is used in this form:
//   - the interior is cut into 8 x 8 (i', j') tile columns (sweep-relative
//     coordinates, ragged last ones), and each tile column into slabs of tk
//     consecutive hyperplanes u = i' + j' + k' (sheared tiles: the 14-step ramp
//     of a skewed 8 x 8 walk is paid once per column, not once per tile);
//   - one launch runs a whole directional sweep of all sources: each wave
//     takes a tile column of a source and marches it slab by slab, waiting for
//     the two upstream columns to pass each slab (see "sweep scheduling"
//     below); the columns of a source are marched by waves of one XCD, so its
//     field moves through that XCD's L2, and consecutive tickets are one
//     column of consecutive sources, which read the same model lines;
//   - inside a tile one 64-lane wave owns the 8 x 8 columns; the tile and its
//     one-node halo are staged in LDS with contiguous column loads, then at
//     step t lane (li, lj) updates the node of its column on hyperplane
//     u = TK' tk + t, reading and writing LDS only, and the tile is written
//     back with contiguous column stores;
//   - per-node records (model, adjoint coefficients) are read from
//     row-coalesced layouts in which the 8 lanes of a tile row find their
//     records side by side on every step.
// Each sweep is followed by a boundary pass (one thread per boundary node), and
// each iteration by a finalize kernel that forms the convergence measure from
// the columns' partial sums in a fixed order (bitwise reproducible run to run).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "tt_device.h"
#include "tt_internal.h"
#include "tt_wait.h"

namespace tt {

// ---------------------------------------------------------------- helpers
// boundary node number b in [0, NB) -> (i, j, k); slabs i = 0 and n0-1 are full,
// slabs in between contribute the ring j in {0, n1-1} or k in {0, n2-1}.
__device__ __forceinline__ void bnd_decode(const Geo& G, long long b, int& i, int& j, int& k) {
    const long long plane = (long long)G.n[1] * G.n[2];
    const long long ring = 2LL * G.n[2] + 2LL * (G.n[1] - 2);
    if (b < plane) {
        i = 0; j = (int)(b / G.n[2]); k = (int)(b % G.n[2]);
        return;
    }
    b -= plane;
    if (b >= (long long)(G.n[0] - 2) * ring) {
        b -= (long long)(G.n[0] - 2) * ring;
        i = G.n[0] - 1; j = (int)(b / G.n[2]); k = (int)(b % G.n[2]);
        return;
    }
    i = 1 + (int)(b / ring);
    long long r = b % ring;
    if (r < G.n[2]) { j = 0; k = (int)r; return; }
    if (r < 2LL * G.n[2]) { j = G.n[1] - 1; k = (int)(r - G.n[2]); return; }
    r -= 2LL * G.n[2];
    j = 1 + (int)(r >> 1);
    k = (r & 1) ? G.n[2] - 1 : 0;
}

// inverse of bnd_decode
__device__ __forceinline__ long long bnd_encode(const Geo& G, int i, int j, int k) {
    const long long plane = (long long)G.n[1] * G.n[2];
    const long long ring = 2LL * G.n[2] + 2LL * (G.n[1] - 2);
    if (i == 0) return (long long)j * G.n[2] + k;
    if (i == G.n[0] - 1) return plane + (long long)(G.n[0] - 2) * ring + (long long)j * G.n[2] + k;
    long long base = plane + (long long)(i - 1) * ring;
    if (j == 0) return base + k;
    if (j == G.n[1] - 1) return base + G.n[2] + k;
    return base + 2LL * G.n[2] + 2LL * (j - 1) + (k == 0 ? 0 : 1);
}

__device__ __forceinline__ bool on_bnd(const Geo& G, int a, int idx) { return idx == 0 || idx == G.n[a] - 1; }
// boundary node (i, j, k) on a k face only: its column is interior
__device__ __forceinline__ bool kface_only(const Geo& G, int i, int j) { return !on_bnd(G, 0, i) && !on_bnd(G, 1, j); }

// Row-coalesced record layouts.  On a sweep hyperplane the 8 lanes of one
// tile row (fixed i, consecutive j) satisfy j + rho k = const with
// rho = sigma_1 sigma_2, so records stored by rows [i][w = j + rho k][j] put
// those 8 lanes' records next to each other (family fam 0: rho = +1, fam 1:
// rho = -1).  Four layouts, lay = 2 fam + (s1 < 0), give each row a pitch of
// n1p records and place j at j + joff[s1 < 0], so that the 8 records a tile
// row reads on one step start on a multiple of 8 records (an aligned run of
// whole 128-byte lines for 32- and 48-byte records) for either sign of the j
// sweep.  Used for the model records and the adjoint coefficients.
__device__ __forceinline__ long long arec_idx(const Geo& G, int lay, int i, int j, int k) {
    const int w = (lay >> 1) == 0 ? j + k : j - k + (G.n[2] - 1);
    return ((long long)i * G.W + w) * G.n1p + j + G.joff[lay & 1];
}

__device__ __forceinline__ int astar_of(const Geo& G, const int p[3]) {
    int as = -1;
    for (int a = 0; a < 3; ++a)
        if (on_bnd(G, a, p[a])) as = a;
    return as;
}

// ---------------------------------------------------------------- set-up
__global__ void k_tables(Geo G, double* __restrict__ t0, double2* __restrict__ t1, double2* __restrict__ t2) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < G.n[0]) t0[q] = G.o[0] + (double)q * G.h[0];
    if (q < G.n[1]) {
        double v = G.o[1] + (double)q * G.h[1];
        t1[q] = G.coord == 1 ? make_double2(cos(v), sin(v)) : make_double2(v, 0.0);
    }
    if (q < G.n[2]) {
        double v = G.o[2] + (double)q * G.h[2];
        t2[q] = G.coord == 1 ? make_double2(cos(v), sin(v)) : make_double2(v, 0.0);
    }
}

// p + q = *hi + *lo exactly
__device__ __forceinline__ void two_sum(double p, double q, double* hi, double* lo) {
#pragma clang fp contract(off)
    const double s = p + q, t = s - p;
    *lo = (p - (s - t)) + (q - t);
    *hi = s;
}

// a b + c d + e, rounded about once (the products' and sums' errors are carried along)
__device__ __forceinline__ double dot_2(double a, double b, double c, double d, double e) {
#pragma clang fp contract(off)
    const double p = a * b, q = c * d;
    const double pl = fma(a, b, -p), ql = fma(c, d, -q);
    double s, sl, r, rl;
    two_sum(p, e, &s, &sl);
    two_sum(s, q, &r, &rl);
    return r + ((sl + rl) + (pl + ql));
}

__global__ void k_src_setup(Geo G, const double* __restrict__ pos, const double* __restrict__ par,
                            Src* __restrict__ out, int nsrc) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nsrc) return;
    Src S;
    const double p0 = pos[3 * q], p1 = pos[3 * q + 1], p2 = pos[3 * q + 2];
    if (G.coord == 1) {
        const double ct = cos(p1), st = sin(p1), cp = cos(p2), sp = sin(p2);
        S.E[0] = ct * cp; S.E[1] = ct * sp; S.E[2] = st;
        S.E[3] = -st * cp; S.E[4] = -st * sp; S.E[5] = ct;
        S.E[6] = -sp; S.E[7] = cp; S.E[8] = 0.0;
        S.rh = p0 * ct;
        // (cp and sp are rounded, and their squares add up to 1 only nearly)
        S.rhl = fma(S.rh, dot_2(cp, cp, sp, sp, -1.0), fma(p0, ct, -S.rh));
        S.zl = fma(p0, st, -(p0 * st));
        S.Xs[0] = p0 * S.E[0]; S.Xs[1] = p0 * S.E[1]; S.Xs[2] = p0 * S.E[2];
    } else {
        for (int a = 0; a < 9; ++a) S.E[a] = (a % 4 == 0) ? 1.0 : 0.0;
        S.Xs[0] = p0; S.Xs[1] = p1; S.Xs[2] = p2;
        S.rh = S.rhl = S.zl = 0.0;
    }
    const double xi0 = par[3 * q + 1], eta0 = par[3 * q + 2];
    const double b = 1.0 - 2.0 * xi0, c = 1.0 + 2.0 * xi0, f = 2.0 * eta0;
    const double det = b * c - f * f;
    S.mi11 = c / det; S.mi12 = -f / det; S.mi22 = b / det;
    S.s0 = par[3 * q];
    S.fb[0] = cell_base(G, 0, p0);
    S.fb[1] = cell_base(G, 1, p1);
    S.fb[2] = cell_base(G, 2, p2);
    S.pad = 0;
    out[q] = S;
}

// Longitude difference of every axis-2 node from every source: (cos - 1, sin) of it
// (Cartesian: (x - x_s, 0)), from the same rounded sines and cosines as elsewhere.
__global__ void k_lon(Geo G, const double2* __restrict__ t2, const Src* __restrict__ src, double2* __restrict__ out,
                      long long n) {
    const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n) return;
    const double2 t = t2[x % G.n[2]];
    const Src& S = src[x / G.n[2]];
    const double sp = -S.E[6], cp = S.E[7];
    out[x] = G.coord == 1 ? make_double2(dot_2(t.x, cp, t.y, sp, -1.0), dot_2(t.y, cp, -t.x, sp, 0.0))
                          : make_double2(t.x - S.Xs[2], 0.0);
}

// trilinear cell and weights at a continuous position (clamped to the grid)
__global__ void k_source_params(Geo G, const double* __restrict__ s, const double* __restrict__ xi,
                                const double* __restrict__ eta, const double* __restrict__ pos,
                                double* __restrict__ par, int nsrc) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nsrc) return;
    const Tri t = tri_of(G, pos[3 * q], pos[3 * q + 1], pos[3 * q + 2]);
    double a = 0.0, b = 0.0, c = 0.0;
    for (int c0 = 0; c0 < 2; ++c0)
        for (int c1 = 0; c1 < 2; ++c1)
            for (int c2 = 0; c2 < 2; ++c2) {
                const double w = tri_w(t, c0, c1, c2);
                const long long x = nidx(G, t.b[0] + c0, t.b[1] + c1, t.b[2] + c2);
                a += w * s[x]; b += w * xi[x]; c += w * eta[x];
            }
    par[3 * q] = a; par[3 * q + 1] = b; par[3 * q + 2] = c;
}

__global__ void k_fill(double* __restrict__ p, long long n, double v) {
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < n;
         x += (long long)gridDim.x * blockDim.x)
        p[x] = v;
}

// initialise a solve: field = init (or v0), fixed nodes = vfix; flags and counters
// init may alias the field: each element is read and then written by one thread
__global__ void k_solve_init(SweepArgs a, const double* init, double v0, double vfix) {
    const int src = blockIdx.y;
    const Src S = a.src[src];
    double* f = a.field + (long long)src * a.G.Nf;
    const double* ti = init ? init + (long long)src * a.G.N : nullptr;
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < a.G.N;
         x += (long long)gridDim.x * blockDim.x) {
        const int k = (int)(x % a.G.n[2]);
        const long long q = x / a.G.n[2];
        const int j = (int)(q % a.G.n[1]), i = (int)(q / a.G.n[1]);
        f[nidx(a.G, i, j, k)] = in_fixed(S, i, j, k) ? vfix : (ti ? ti[x] : v0);
    }
    // sums, sweep progress and queue words start at zero
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < a.nslots;
         x += (long long)gridDim.x * blockDim.x) {
        a.part[(long long)src * a.nslots + x] = 0.0;
        if (a.part2) a.part2[(long long)src * a.nslots + x] = 0.0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.active[src] = 1;
        a.iter[src] = 0;
        a.status[src] = 0;
        if (src == 0) *a.counter = a.nsrc;
    }
}

// --------------------------------------------------------- sweep tiles
// Lane-constant context of one tile of one source in directional sweep DIR
// (signs s_a = -1 where bit 2 - a of DIR is set; compile-time, so every
// sign-dependent index folds to adds).
template <int DIR>
struct Dir {
    static constexpr int s0 = (DIR & 4) ? -1 : 1;
    static constexpr int s1 = (DIR & 2) ? -1 : 1;
    static constexpr int s2 = (DIR & 1) ? -1 : 1;
    static constexpr int fam = ((DIR >> 1) ^ DIR) & 1;  // row-coalesced layout family of this sweep
    static constexpr int lay = 2 * fam + (s1 > 0 ? 0 : 1);  // its aligned layout
};

struct TileCtx {
    int TI, TJ, U0, lane, li, lj, ext_i, ext_j;
    int ip, jp;    // this lane's column (sweep-relative; the tile corner's if the lane owns none)
    int t0, t1;    // wave-uniform walk: steps t0 <= t < t1 (u = U0 + t)
    int kp0;       // this lane's k' at step 0 (k' = kp0 + t)
    int kplo, kphi;  // record fetch clamp: this lane's k' range in the tile (a valid k' if empty)
    int kq0;       // staged entry (ci, cj, kk) holds k' = kq0 - ci - cj + kk
    int kbase;     // absolute k = kbase + s2 k'
    bool colv, fcol;
    int i, j;
    int rbase, rstep;  // record index of this lane's column at k' = 0, and its change per k'
    // forward fetches: record and axis-2 table index at step 0, and the step
    // range [tlo, thi] that the clamp of k' to [kplo, kphi] allows
    int rr0, tt0, tlo, thi;
    // this lane updates its node at the steps ta <= t < ta + tn except tf, tf + 1 (the fixed cell)
    int ta, tf;
    unsigned tn;
};

// the column's part of the context
template <int DIR>
__device__ __forceinline__ TileCtx col_ctx(const Geo& G, const Src& S, int TI, int TJ) {
    using D = Dir<DIR>;
    TileCtx c;
    c.TI = TI;
    c.TJ = TJ;
    c.lane = threadIdx.x;
    c.li = c.lane >> 3;
    c.lj = c.lane & 7;
    c.ext_i = min(kBI, G.m[0] - c.TI * kBI);
    c.ext_j = min(kBJ, G.m[1] - c.TJ * kBJ);
    c.colv = c.li < c.ext_i && c.lj < c.ext_j;
    c.ip = c.TI * kBI + (c.colv ? c.li : 0);
    c.jp = c.TJ * kBJ + (c.colv ? c.lj : 0);
    c.i = D::s0 > 0 ? 1 + c.ip : G.n[0] - 2 - c.ip;
    c.j = D::s1 > 0 ? 1 + c.jp : G.n[1] - 2 - c.jp;
    c.fcol = (unsigned)(c.i - S.fb[0]) <= 1u && (unsigned)(c.j - S.fb[1]) <= 1u;
    c.kbase = D::s2 > 0 ? 1 : G.n[2] - 2;
    // record index ((i W + w) n1p + j + joff) in the aligned layout of this sweep,
    // w = j + k (family 0) or j - k + n2 - 1 (family 1), k = kbase + s2 k': linear
    // in k' with slope s1 n1p in both families
    const int w0 = D::fam == 0 ? c.j + c.kbase : c.j - c.kbase + G.n[2] - 1;
    c.rbase = (c.i * G.W + w0) * G.n1p + c.j + G.joff[D::s1 > 0 ? 0 : 1];
    c.rstep = D::s1 * G.n1p;
    return c;
}

// the slab's part; HELD: records are fetched past the slab's end, for the next one
template <int DIR, bool HELD = false>
__device__ __forceinline__ void slab_ctx(const Geo& G, const Src& S, TileCtx& c, int U0, int depth) {
    using D = Dir<DIR>;
    c.U0 = U0;
    const int ucol = kBI * (c.TI + c.TJ);  // u of the column's first node (i', j' at the tile corner, k' = 0)
    c.t0 = max(0, ucol - U0);
    c.t1 = min(depth, ucol + (c.ext_i - 1) + (c.ext_j - 1) + G.m[2] - U0);
    c.kp0 = U0 - c.ip - c.jp;
    // prefetches past the walk re-read the lane's last record of this tile
    // (a cache hit) instead of the next slab's
    c.kplo = max(0, c.kp0 + c.t0);
    c.kphi = min(G.m[2] - 1, c.kp0 + c.t1 - 1);
    if (c.kplo > c.kphi) c.kplo = c.kphi = min(max(c.kp0 + c.t0, 0), G.m[2] - 1);
    if (HELD) {
        c.kplo = 0;
        c.kphi = G.m[2] - 1;
    }
    c.kq0 = U0 - ucol + 1;
    c.rr0 = c.rbase + c.rstep * c.kp0;
    c.tt0 = c.kbase + D::s2 * c.kp0;
    c.tlo = c.kplo - c.kp0;
    c.thi = c.kphi - c.kp0;
    c.ta = max(c.t0, -c.kp0);
    c.tn = c.colv ? (unsigned)max(min(c.t1, G.m[2] - c.kp0) - c.ta, 0) : 0u;
    // k = kbase + s2 (kp0 + t) in {fb, fb + 1}
    const int tb = D::s2 * (S.fb[2] - c.kbase) - c.kp0;
    c.tf = c.fcol ? (D::s2 > 0 ? tb : tb - 1) : -4;
}

// is step t one of this lane's updates?  (a padded walk's t < t1 + 6, so that -4 never matches)
__device__ __forceinline__ bool step_on(const TileCtx& c, int t) {
    return (unsigned)(t - c.ta) < c.tn && (unsigned)(t - c.tf) > 1u;
}

// ------------------------------------------------------- sweep scheduling
// One launch runs a directional sweep of up to kMarchSources sources.  Its
// workgroups are one wave each; a wave takes a tile column of a source, marches
// it slab by slab from its first to its last, and takes the next.  Between
// slabs it waits for the two upstream columns, which other waves march, to
// have passed the slab it is about to walk.
//
// What this replaces is a launch per tile-plane: at one 41^3 source a sweep
// was 17 dependent launches of 7.5 us, at 128 101^3 sources 52000 launches per
// solve, which the host could not enqueue faster than 7.5 us apiece.
//
// Who may wait for whom.  The sources are dealt to nb <= 8 batches (source
// c0 + b + nb q belongs to batch b).  A batch is claimed by one XCD (the first
// wave to ask sets its owner word) and worked on by waves of that XCD only; its
// columns are handed out by a ticket counter, ordered by TI + TJ, then TI,
// then source.  A column's upstream neighbours have lower tickets, so whoever
// holds them is already running, never waits for a later ticket, and finishes:
// every wait ends, however many waves are resident.  (Should a wave be lost all the
// same, waits for it end after kWaitPolls polls and the source ends unconverged.)
//
// How a slab's values reach the next wave.  All waves of a batch share the
// XCD's L2: a wave's stores are in that L2 once s_waitcnt vmcnt(0) has passed,
// then it stores its progress word; a waiting wave polls that word past its L1
// (agent-scope load) and invalidates its L1 (agent-scope acquire) before it
// stages the tile.  8 KB handed over this way take 1.0 us from wave to wave; a
// release that works across XCDs (it writes the whole L2 back) takes 1.5 us on
// an idle chip and 8.7 us with 256 such chains.
constexpr int kMarchBatches = 8;                    // one per XCD
constexpr int kMarchSources = 64 * kMarchBatches;   // sources of one launch: a batch's active mask is one wave ballot

__device__ __forceinline__ unsigned* queue_words(const SweepArgs& a, int src) {
    return reinterpret_cast<unsigned*>(a.part + (long long)src * a.nslots + 2 * a.G.ncols + a.nbblocks);
}

// word 2 of the queue's: has a wave of this solve given up a wait for this source?
__device__ __forceinline__ unsigned* lost_word(const SweepArgs& a, int src) { return queue_words(a, src) + 2; }

// between two sweeps: every queue back to "no ticket taken, no owner"
__device__ __forceinline__ void queue_reset(const SweepArgs& a, int src) {
    if (threadIdx.x < 2) queue_words(a, src)[threadIdx.x] = 0u;
}

// convergence sums run over the iteration's directions
__device__ __forceinline__ void part_add(double* slot, int dir, double v) { *slot = dir == 0 ? v : *slot + v; }

__device__ __forceinline__ unsigned long long* progress_words(const SweepArgs& a, int src) {
    return reinterpret_cast<unsigned long long*>(a.part + (long long)src * a.nslots + a.G.ncols + a.nbblocks);
}

// The __syncthreads() in these helpers cost nothing in a workgroup of one wave
// (no instruction); they keep the wave together.  Without them the compiler
// joins the "lane 0 only" branch at the end of one column with that at the
// start of the next, lanes 1..63 run ahead with a ticket of their own, and the
// ballots below see half a wave.

// does this wave's XCD own the batch whose queue is q (claiming it if nobody does)?
__device__ __forceinline__ bool sweep_claim(unsigned* q, unsigned me) {
    __syncthreads();
    unsigned own = 0u;
    if (threadIdx.x == 0 && __hip_atomic_compare_exchange_strong(q + 1, &own, me, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT))
        own = me;
    __syncthreads();
    return (unsigned)__builtin_amdgcn_readfirstlane((int)own) == me;
}

__device__ __forceinline__ unsigned sweep_ticket(unsigned* q) {
    __syncthreads();
    unsigned t = 0u;
    if (threadIdx.x == 0) t = __hip_atomic_fetch_add(q, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return (unsigned)__builtin_amdgcn_readfirstlane((int)t);
}

// Wait until both upstream columns have passed slab TK of this sweep (word >=
// target), then drop stale L1 lines.  up: this lane's neighbour's word (lanes
// 0 and 1) or NULL.  A wait that is given up (poll_until) marks the source as
// lost; the caller carries on, so that the launch ends, and the source's
// iteration ends as not converged (finish_iteration).
__device__ __forceinline__ void wait_upstream(const unsigned long long* up, unsigned long long target, unsigned* lost) {
    const bool ok = poll_until(
        [&] {
            const unsigned long long v =
                up ? __hip_atomic_load(up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0ull;
            return (bool)__all(v >= target);
        },
        [&] { return (bool)__any(__hip_atomic_load(lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u); },
        [] { __builtin_amdgcn_s_sleep(1); }, kWaitPolls);
    if (!ok) {
        __syncthreads();
        if (threadIdx.x == 0) __hip_atomic_store(lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// this wave's stores are in the XCD's L2, then its column's progress says so
__device__ __forceinline__ void publish(unsigned long long* word, unsigned long long value) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0) __hip_atomic_store(word, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
}

// Hand out this launch's columns: column(src, TI, TJ) for every one of this
// wave's tickets.  XCDs start at different batches, so that each gets one.
template <class F>
__device__ __forceinline__ void march(const SweepArgs& a, const Geo& G, int c0, int cn, F column) {
    const int xcd = __builtin_amdgcn_s_getreg(20 | (31 << 11)) & 15;  // XCC_ID
    const int nb = min(kMarchBatches, cn);
    for (int e = 0; e < nb; ++e) {
        const int b = (xcd + e) % nb;
        unsigned* q = queue_words(a, c0 + b);
        if (!sweep_claim(q, (unsigned)xcd + 1u)) continue;
        const int mine = b + nb * (int)threadIdx.x;
        const unsigned long long mask = __ballot(mine < cn && a.active[c0 + min(mine, cn - 1)]);
        const unsigned nact = (unsigned)__popcll(mask), ntask = nact * (unsigned)G.ncols;
        // this lane's source is the rank-th active one of the batch
        const unsigned rank = (unsigned)__popcll(mask & ((1ull << threadIdx.x) - 1ull));
        const bool act = (mask >> threadIdx.x) & 1ull;
        if (nact == 0) continue;
        for (;;) {
            const unsigned t = sweep_ticket(q);
            if (t >= ntask) break;
            const unsigned col = t / nact, k = t - col * nact;
            const int l = __ffsll((unsigned long long)__ballot(act && rank == k)) - 1;
            int TI, TJ;
            col_decode(G, (int)col, TI, TJ);
            column(c0 + b + nb * l, TI, TJ);
        }
    }
}

struct Handover {
    const unsigned long long* up;  // this lane's upstream column's progress word or NULL
    unsigned long long target;     // what it must have reached
    unsigned long long* own;       // this column's word, and its value when the slab is done
    unsigned long long done;
    bool more;                     // another slab follows
    unsigned* lost;                // the source's lost word
};

// March one tile column: tile(TK) for every slab in order, each after its wait.
// HELD: the tile publishes its slab itself.
template <int DIR, bool HELD, class F>
__device__ __forceinline__ void march_column(const SweepArgs& a, const Geo& G, int src, int TI, int TJ, F tile) {
    unsigned long long* prog = progress_words(a, src);
    unsigned long long* own = prog + TI * G.nt[1] + TJ;
    const unsigned long long* up = nullptr;
    if (threadIdx.x == 0 && TI > 0) up = own - G.nt[1];
    if (threadIdx.x == 1 && TJ > 0) up = own - 1;
    // progress of sweep number e of the solve: (e << 16) + slabs passed, so
    // that a finished earlier sweep's word is below every target of this one
    const unsigned long long base = ((unsigned long long)a.iter[src] * 8 + DIR + 1) << 16;
    const int hi = col_tile_hi(G, TI + TJ);
    for (int TK = col_tile_lo(G, TI + TJ); TK <= hi; ++TK) {
        const unsigned long long done = TK < hi ? base + TK + 1 : base + 0xffffu;
        tile(TK, Handover{up, base + TK + 1, own, done, TK < hi, lost_word(a, src)});
        if (!HELD) publish(own, done);
    }
}

// Staged tile: the (8+2) x (8+2) columns of the tile and its i'/j' halo, each
// with the entries kk = 0..tk+1, in LDS as [ci][cj][kk] (ci = li + 1,
// cj = lj + 1; column pitch tk + 2: an odd pitch measured no better and costs
// a tile per CU at some depths).  Entry kk of column (ci, cj) is the node
// k' = kq0 - ci - cj + kk: the column windows are sheared along the tile's
// slab, so at step t lane (li, lj) owns entry t + 1 of its column and finds
// its upstream i'/j'/k' neighbours at entry t and its downstream ones at
// entry t + 2.  Everything a step reads from the field is staged (upstream
// tiles are finished, downstream ones untouched), so the walk touches LDS
// only; staged k' are clamped to the column's nodes [-1, m2] (entries outside
// are never read).  Loads and stores move contiguous column segments.
constexpr int kTC = kBI + 2;

// Staging.  The staged window is always the full (8+2) x (8+2) columns
// (columns past a ragged tile's end are staged from clamped, valid rows and
// never read) of Lp = tile_pitch(tk) slots; slot q of a column holds entry
// kk = q in sweeps with s2 > 0 and kk = Lp - 1 - q in sweeps with s2 < 0, so
// that consecutive slots always hold consecutive nodes in memory (ascending
// k).  The window is loaded with direct global-to-LDS loads of 16 bytes per
// lane (lane l of a load writes the l-th slot pair from the load's LDS
// address): each load covers 64 / (Lp / 2) whole columns, so a lane keeps its
// column offset and slot pair in every load, no data passes through
// registers, every load of the window is in flight at once and the wave waits
// once.  Pairs with no node entry (k' outside [-1, m2]) and pairs of columns
// past a ragged tile's halo are not loaded (their slots are never read); a
// pair with one node entry reads one neighbouring element of the field array
// that is never used (its address is clamped into the array).
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) void lds_void;

// LDS bytes of a staged tile: the window's slot pairs
__host__ __device__ inline int stage_bytes(int tk) { return kTC * kTC * tile_pitch(tk) * 8; }

// LDS slot of entry kk of a column (the mirror for sweeps with s2 < 0)
template <int S2>
__device__ __forceinline__ int slot_of(int kk, int Lp) {
    return S2 > 0 ? kk : Lp - 1 - kk;
}

// Absolute index along axis a of staged column/row ci (0 = upstream halo):
// origin + sgn * ci.
template <int SGN>
__device__ __forceinline__ int stage_origin(const Geo& G, int a, int T) {
    return SGN > 0 ? T * kBI : G.n[a] - 1 - T * kBI;
}

// xlo, xhi: the element range of the field array around fld that may be read.
// Load r covers columns cb = r cpi .. cb + cpi - 1 (cpi = 64 / (Lp / 2));
// lane l takes slots q, q + 1 (q = 2 (l % (Lp / 2))) of column cb + l / (Lp / 2)
// (lanes past cpi whole columns stay idle).  Per lane the loop keeps that
// column's (ci, cj), y = the element of its lower slot, and d = the k' test
// value of the pair, each advanced by a constant per load plus a carry when cj
// wraps.  Offsets are 32-bit: the host keeps N below 2^31, and a loaded pair
// lies in [-1, N] around fld.
template <int DIR>
__device__ __forceinline__ void stage_tile(const Geo& G, const TileCtx& c, const double* __restrict__ fld,
                                           long long xlo, long long xhi, double* lds) {
    using D = Dir<DIR>;
    constexpr int sg = D::s2;
    const int Lp = tile_pitch(G.tk);
    const int hp = Lp >> 1, cpi = 64 / hp;
    const int si = (int)G.si, sj = (int)G.sj;
    const int oi = stage_origin<D::s0>(G, 0, c.TI), oj = stage_origin<D::s1>(G, 1, c.TJ);
    const int lo = (int)(xlo > -1 ? xlo : -1), hi = (int)(xhi < G.N ? xhi : G.N);
    // (opaque: or the addresses of every load are kept over the whole column, in 100 registers)
    int lane = c.lane;
    asm volatile("" : "+v"(lane));
    const int dc = lane / hp, q = 2 * (lane - dc * hp);
    const bool lane_on = dc < cpi;
    int ci = dc / kTC, cj = dc - ci * kTC;
    // lower slot q holds entry kk = q (s2 > 0) or Lp - 1 - q (s2 < 0) of the
    // column, node k' = kq0 - ci - cj + kk at element kbase + s2 k'; the pair
    // holds a node entry iff its lower entry's k' + (2 or 1) lies in [0, m2 + 2]
    const int x0 = c.kbase + sg * c.kq0 + (sg > 0 ? 0 : 1 - Lp);
    const int ka0 = sg > 0 ? c.kq0 + 2 : c.kq0 + Lp;
    // (unsigned: columns outside the grid, never loaded, may leave the int range)
    unsigned y = (unsigned)(oi + D::s0 * ci) * si + (unsigned)(oj + D::s1 * cj) * sj - sg * (ci + cj) + x0 + q;
    int d = ka0 - (ci + cj) + sg * q;
    const unsigned kspan = (unsigned)G.m[2] + 2;
    const int ei = c.ext_i + 2, ej = c.ext_j + 2;
    const unsigned dy = (unsigned)cpi * (unsigned)(D::s1 * sj - sg);
    const unsigned dy_w = (unsigned)(D::s0 * si) - (unsigned)(kTC * D::s1 * sj) + sg * (kTC - 1);
    lds_char* lb = (lds_char*)lds;  // the dynamic shared array, in the LDS address space
    for (int cb = 0; cb < kTC * kTC; cb += cpi) {
        if (lane_on && ci < ei && cj < ej && (unsigned)d <= kspan) {
            const int x = min(max((int)y, lo), hi);
            __builtin_amdgcn_global_load_lds(fld + x, (lds_void*)(lb + 16 * cb * hp), 16, 0, 0);
        }
        cj += cpi;
        y += dy;
        d -= cpi;
        // one wrap (taken as selects) unless cpi >= kTC (pitches below 14)
        const bool wrap = cj >= kTC;
        cj -= wrap ? kTC : 0;
        ci += wrap ? 1 : 0;
        y += wrap ? dy_w : 0u;
        d += wrap ? kTC - 1 : 0;
        if (cpi >= kTC) {
            while (cj >= kTC) {
                cj -= kTC;
                ++ci;
                y += dy_w;
                d += kTC - 1;
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // every load of the window (and any earlier one) has landed
}

// Write back the tile's own nodes: entries 1..tk of its columns whose k' is
// an interior node (the others are halo or outside the column).  The columns
// are taken as the full 8 x 8 (those past a ragged tile's end are skipped)
// in chunks of 16 entries: in chunk ch, lane (g, r) = (lane / 16, lane % 16)
// takes entry q + 1, q = ch + r, of own column (li, lj) = (u / 2, 4 (u % 2) + g)
// at step u = 0..15.  A step's element offset and LDS slot then differ from
// the lane's first ones by a wave-uniform amount, and every LDS read of a
// chunk is issued before its stores.  (Reads of skipped entries stay inside
// the window: their slots lie less than 16 past either end of an own
// column, and the columns beside it in LDS are staged ones.)
template <int DIR>
__device__ __forceinline__ void unstage_tile(const Geo& G, const TileCtx& c, double* __restrict__ fld,
                                             const double* lds, int Lp) {
    using D = Dir<DIR>;
    constexpr int sg = D::s2;
    const int ek = G.tk;
    const int si = D::s0 * (int)G.si, sj = D::s1 * (int)G.sj;
    const int base = (int)nidx(G, stage_origin<D::s0>(G, 0, c.TI) + D::s0, stage_origin<D::s1>(G, 1, c.TJ) + D::s1,
                               c.kbase);
    const unsigned kmax = (unsigned)G.m[2];
    int lane = c.lane;
    asm volatile("" : "+v"(lane));  // as in stage_tile
    const int g = lane >> 4, r = lane & 15;
    const bool colj0 = g < c.ext_j, colj1 = g + 4 < c.ext_j;
    // node (li, lj, entry q + 1): element base + li si + lj sj + s2 k', with
    // k' = kq0 - 1 - li - lj + q, and slot ((li + 1) kTC + lj + 1) Lp + q + 1
    // (mirrored: Lp - 2 - q)
    const unsigned xa = (unsigned)(si - sg), xb = 4u * (unsigned)(sj - sg);
    const int la = kTC * Lp, lb = 4 * Lp;
    for (int ch = 0; ch < ek; ch += 16) {
        const int q = ch + r;
        // (unsigned: lanes past the tile's entries, never stored, may leave the int range)
        const unsigned x0 = (unsigned)base + (unsigned)(sg * (c.kq0 - 1 + q)) + (unsigned)g * (unsigned)(sj - sg);
        const int l0 = (kTC + g + 1) * Lp + (sg > 0 ? 1 : Lp - 2) + sg * q;
        const int kp0 = c.kq0 - 1 - g + q;
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            v[u] = lds[l0 + __builtin_amdgcn_readfirstlane((u >> 1) * la + (u & 1) * lb)];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int li = u >> 1, b = u & 1;
            if (li < c.ext_i && (b ? colj1 : colj0) && q < ek && (unsigned)(kp0 - li - 4 * b) < kmax)
                fld[(int)(x0 + (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)li * xa + (unsigned)b * xb)))] =
                    v[u];
        }
    }
}

// Forward sweeps: a boundary node on a k face only (its column is interior)
// copies the column's interior end node k' = 0 or m2 - 1 (the boundary rule
// copies the inward neighbour along the last boundary axis, here k).  Nothing
// else in a sweep reads or writes it, so the tile that finalises the end node
// sets it right after its walk, next to the column it has just written back;
// the boundary pass skips those nodes (strided ones: each sits in a cache line
// of its own) and the change joins the tile's convergence sum.
template <int DIR>
__device__ __forceinline__ void fwd_kface_nodes(const Geo& G, const Src& S, const TileCtx& c, double* __restrict__ fld,
                                                const double* lds, int own, int Lp, double& eps) {
    using D = Dir<DIR>;
    constexpr int sg = D::s2;
    if (!c.colv) return;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int kin = e == 0 ? 0 : G.m[2] - 1;                // the interior end node's k'
        const int t = kin - c.kp0;                              // the step that updated it
        if (t < c.t0 || t >= c.t1) continue;
        const int kb = c.kbase + sg * (e == 0 ? -1 : G.m[2]);  // absolute k of the boundary node
        if (in_fixed(S, c.i, c.j, kb)) continue;
        const int o = sg > 0 ? own + t : own + Lp - 1 - t;
        const double nv = lds[o + sg];                       // entry t + 1: the end node
        const double old = lds[e == 0 ? o : o + 2 * sg];     // entry t or t + 2: the boundary node
        fld[nidx(G, c.i, c.j, kb)] = nv;
        eps += fabs(nv - old);
    }
}

// ------------------------------------------------ windows held across slabs
// The forward sweeps at a depth of 16 steps keep their window between the slabs
// of a column instead of staging it anew.  While slab TK is walked, the entries
// that slab TK + 1 adds -- kk = 2 .. tk + 1 of the tile's own columns and of the
// downstream halo, which no other wave touches before this one has passed TK --
// are loaded into registers; the two entries that the slabs share are carried in
// a register pair; and what is left to load after the wait is the upstream halo,
// two loads.  A walked slab's downstream edges (li = 7, lj = 7) are stored first
// and published when they have arrived; the rest of the tile follows without a
// wait.  The record ring runs on from slab to slab.
//
// Why: a batch that does not fill the chip waits for the hand-over from column to
// column, and staging and the wait for all stores were part of it.  Staged and
// held: 41^3 x 1 source 10.5 / 8.9 ms, 61^3 x 1 23.1 / 19.7, x 4 28.6 / 24.3, x 16
// 32.6 / 28.2, x 32 38.0 / 34.3.  (The adjoint, whose steps are a quarter as long,
// lost by it: 41^3 x 1 11.0 / 11.7, 61^3 x 32 56.6 / 59.6.)
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));   // two doubles at any element of a field
typedef double d2a __attribute__((ext_vector_type(2), aligned(16)));  // a slot pair in LDS

template <int DIR, int TKC>
struct Window {
    static constexpr int sg = Dir<DIR>::s2;
    static constexpr int Lp = TKC + 2;         // = tile_pitch(TKC)
    static constexpr int pairs = TKC / 2;      // lanes of a column: one slot pair each
    static constexpr int cpl = 64 / pairs;     // columns per load
    static constexpr int nload = 80 / cpl;     // loads of the own columns (64) and the downstream halo (16)
    static constexpr int nhalo = 16 / cpl;     // loads of the upstream halo
    static_assert(cpl == 8, "a row of columns per load");
    // column (ci, cj) of load r on this lane
    static __device__ __forceinline__ void col(int r, int sub, int& ci, int& cj) {
        ci = r < 9 ? r + 1 : sub + 1;
        cj = r < 9 ? sub + 1 : kTC - 1;
    }
    static __device__ __forceinline__ void halo_col(int r, int sub, int& ci, int& cj) {
        const int n = r * cpl + sub;
        ci = n < 8 ? 0 : n - 7;
        cj = n < 8 ? n + 1 : 0;
    }
};

// (or what follows from the lane number alone is kept for the whole kernel, in scratch)
__device__ __forceinline__ int opaque_lane(const TileCtx& c) {
    int lane = c.lane;
    asm volatile("" : "+v"(lane));
    return lane;
}

// The element of fld that entry kk = 0 of column (ci, cj) = (0, 0) would have:
// entry kk of (ci, cj) is at org + ci A + cj B + s2 kk, A = s0 si - s2, B = s1 sj - s2.
template <int DIR>
__device__ __forceinline__ unsigned win_org(const Geo& G, const TileCtx& c, int kq0) {
    using D = Dir<DIR>;
    return (unsigned)stage_origin<D::s0>(G, 0, c.TI) * (unsigned)(int)G.si +
           (unsigned)stage_origin<D::s1>(G, 1, c.TJ) * (unsigned)(int)G.sj + (unsigned)(c.kbase + D::s2 * kq0);
}

// Addresses are clamped into the array and columns to the ragged tile's halo
// instead of being skipped (what they then load is never read), so that no
// branch encloses a load.
template <int DIR, int TKC>
__device__ __forceinline__ d2u win_pair(const Geo& G, const TileCtx& c, const double* __restrict__ fld, int lo, int hi,
                                        unsigned org, int ci, int cj, int kk) {
    using D = Dir<DIR>;
    const unsigned A = (unsigned)(D::s0 * (int)G.si - D::s2), B = (unsigned)(D::s1 * (int)G.sj - D::s2);
    const unsigned x = org + (unsigned)min(ci, c.ext_i + 1) * A + (unsigned)min(cj, c.ext_j + 1) * B +
                       (unsigned)(D::s2 * kk);
    return *reinterpret_cast<const d2u*>(fld + min(max((int)x, lo), hi));
}

// the entries that the slab at kq0 adds
template <int DIR, int TKC>
__device__ __forceinline__ void win_load(const Geo& G, const TileCtx& c, const double* __restrict__ fld, int lo, int hi,
                                         int kq0, d2u (&pf)[Window<DIR, TKC>::nload]) {
    using W = Window<DIR, TKC>;
    const int lane = opaque_lane(c);
    const int sub = lane / W::pairs, q = 2 * (lane % W::pairs);
    const unsigned org = win_org<DIR>(G, c, kq0);
#pragma unroll
    for (int r = 0; r < W::nload; ++r) {
        int ci, cj;
        W::col(r, sub, ci, cj);
        // slots q + 2, q + 3 hold entries q + 2, q + 3; mirrored, slots q, q + 1 hold Lp - 1 - q and the one below
        pf[r] = win_pair<DIR, TKC>(G, c, fld, lo, hi, org, ci, cj, W::sg > 0 ? q + 2 : W::Lp - 1 - q);
    }
}

template <int DIR, int TKC>
__device__ __forceinline__ void win_put(const TileCtx& c, double* lds, const d2u (&pf)[Window<DIR, TKC>::nload]) {
    using W = Window<DIR, TKC>;
    const int lane = opaque_lane(c);
    const int sub = lane / W::pairs, q = 2 * (lane % W::pairs);
#pragma unroll
    for (int r = 0; r < W::nload; ++r) {
        int ci, cj;
        W::col(r, sub, ci, cj);
        *reinterpret_cast<d2a*>(lds + (ci * kTC + cj) * W::Lp + (W::sg > 0 ? q + 2 : q)) = pf[r];
    }
}

// the upstream halo's entries 0 .. tk - 1
template <int DIR, int TKC>
__device__ __forceinline__ void win_halo(const Geo& G, const TileCtx& c, const double* __restrict__ fld, int lo, int hi,
                                         double* lds) {
    using W = Window<DIR, TKC>;
    const int lane = opaque_lane(c);
    const int sub = lane / W::pairs, q = 2 * (lane % W::pairs);
    const unsigned org = win_org<DIR>(G, c, c.kq0);
    d2u v[W::nhalo];
#pragma unroll
    for (int r = 0; r < W::nhalo; ++r) {
        int ci, cj;
        W::halo_col(r, sub, ci, cj);
        v[r] = win_pair<DIR, TKC>(G, c, fld, lo, hi, org, ci, cj, W::sg > 0 ? q : W::Lp - 3 - q);
    }
#pragma unroll
    for (int r = 0; r < W::nhalo; ++r) {
        int ci, cj;
        W::halo_col(r, sub, ci, cj);
        *reinterpret_cast<d2a*>(lds + (ci * kTC + cj) * W::Lp + (W::sg > 0 ? q : q + 2)) = v[r];
    }
}

// entries 0 and 1 of this lane's own column, as its slot pair: slots 0, 1 or, mirrored, Lp - 2, Lp - 1
template <int DIR, int TKC>
__device__ __forceinline__ d2u win_first(const Geo& G, const TileCtx& c, const double* __restrict__ fld, int lo, int hi) {
    return win_pair<DIR, TKC>(G, c, fld, lo, hi, win_org<DIR>(G, c, c.kq0), c.li + 1, c.lj + 1, Dir<DIR>::s2 > 0 ? 0 : 1);
}

// the slab's last two entries, which are the next one's entries 0 and 1
template <int DIR, int TKC>
__device__ __forceinline__ d2u win_carry(const double* lds, int own) {
    return *reinterpret_cast<const d2a*>(lds + own + (Dir<DIR>::s2 > 0 ? TKC : 0));
}
template <int DIR, int TKC>
__device__ __forceinline__ void win_put_first(double* lds, int own, d2u v) {
    *reinterpret_cast<d2a*>(lds + own + (Dir<DIR>::s2 > 0 ? 0 : TKC)) = v;
}

// Stores nodes of the walked slab (entries 1 .. tk): EDGES, the columns li = 7
// and lj = 7, or all others.  E entries of 64 / E columns go out per store.
template <int DIR, int TKC, bool EDGES>
__device__ __forceinline__ void win_store(const Geo& G, const TileCtx& c, double* __restrict__ fld, const double* lds) {
    using D = Dir<DIR>;
    using W = Window<DIR, TKC>;
    constexpr int E = TKC < 16 ? TKC : 16, cps = 64 / E, per = 8 / cps;
    const int lane = opaque_lane(c);
    const int sub = lane / E, r = lane % E;
    const unsigned A = (unsigned)(D::s0 * (int)G.si - D::s2), B = (unsigned)(D::s1 * (int)G.sj - D::s2);
    const unsigned kmax = (unsigned)G.m[2];
#pragma unroll
    for (int ch = 0; ch < TKC; ch += E) {
        const int kk = ch + r + 1;
        const unsigned org = win_org<DIR>(G, c, c.kq0) + (unsigned)(W::sg * kk);
        const int kp = c.kq0 + kk, slot = W::sg > 0 ? kk : W::Lp - 1 - kk;
        constexpr int n = EDGES ? 2 * per : 7 * per;
        double v[n];
        int ci[n], cj[n];
#pragma unroll
        for (int u = 0; u < n; ++u) {
            const int h = (u % per) * cps + sub + 1;
            ci[u] = EDGES ? (u < per ? kBI : h) : u / per + 1;
            cj[u] = EDGES ? (u < per ? h : kBJ) : h;
            v[u] = lds[(ci[u] * kTC + cj[u]) * W::Lp + slot];
        }
#pragma unroll
        for (int u = 0; u < n; ++u)
            if (ci[u] <= c.ext_i && cj[u] <= c.ext_j && (EDGES || cj[u] < kBJ) && (!EDGES || u < per || ci[u] < kBI) &&
                (unsigned)(kp - ci[u] - cj[u]) < kmax)
                fld[(int)(org + (unsigned)ci[u] * A + (unsigned)cj[u] * B)] = v[u];
    }
}

// The per-node records a step needs (model, table) are loaded kPre steps
// ahead into a ring slot indexed by the wave-uniform step number.
constexpr int kPre = 4;       // forward: steps are long (the full update)
constexpr int kPreAdj = 6;    // adjoint: short steps, so look further ahead

struct FwdSlot {
    double sx, ma, mb, mc, f1, sn;  // s, the anisotropy block (1 - 2 xi, 2 eta, 1 + 2 xi), longitude difference
};

// unconditional: k' is clamped into the lane's range in the tile, so the address is always valid
template <int DIR>
__device__ __forceinline__ void fwd_fetch(const TileCtx& c, const double* __restrict__ mdl,
                                          const double2* __restrict__ lon, int t, FwdSlot& r) {
    // the step clamped to the lane's k' range; |rstep| = n1p < 2^23 and the
    // step is below 64, so the product is a 24-bit one
    const int tc = min(max(t, c.tlo), c.thi);
    const unsigned ri = (unsigned)(c.rr0 + __mul24(c.rstep, tc));
    const double2* m = reinterpret_cast<const double2*>(mdl + (size_t)ri * 4);
    const double2 m0 = m[0], m1 = m[1];
    r.sx = m0.x;
    r.ma = m0.y;
    r.mb = m1.x;
    r.mc = m1.y;
    const double2 tv = lon[(unsigned)(c.tt0 + Dir<DIR>::s2 * tc)];
    r.f1 = tv.x;
    r.sn = tv.y;
}

// One step of the forward walk at step t of the slab.  No step has a branch:
// every lane forms an update, one that has none to make stores it into the
// window's corner column, which nothing reads.  So the factor of one step fills
// the waits of the step before: 553 cycles a step of a lone wave with a branch
// around each update.
// HELD: t is below the window's depth, so that the corner column has the slot.
template <int COORD, int DIR, bool HELD>
__device__ __forceinline__ void fwd_step(const Geo& G, const Src& S, const LfCol& W, const TileCtx& c, double* lds, int own, int Lp,
                                         int t, const FwdSlot& r, double& eps) {
    using D = Dir<DIR>;
    // sweep-relative neighbours: "up" = already updated this sweep
    // slot of entry t (mirrored columns when s2 < 0): entry t + 1 is at o + s2
    constexpr int sg = D::s2;
    const int o = sg > 0 ? own + t : own + Lp - 1 - t;
    const double cur = lds[o + sg];
    const double up_i = lds[o - kTC * Lp], dn_i = lds[o + kTC * Lp + 2 * sg];
    const double up_j = lds[o - Lp], dn_j = lds[o + Lp + 2 * sg];
    const double up_k = lds[o], dn_k = lds[o + 2 * sg];
    const double m0 = D::s0 > 0 ? up_i : dn_i, p0 = D::s0 > 0 ? dn_i : up_i;
    const double m1 = D::s1 > 0 ? up_j : dn_j, p1 = D::s1 > 0 ? dn_j : up_j;
    const double m2 = D::s2 > 0 ? up_k : dn_k, p2 = D::s2 > 0 ? dn_k : up_k;
    const double nv = lf_update<COORD>(G, S, W, r.f1, r.sn, r.sx, r.ma, r.mb, r.mc, cur, m0, p0, m1, p1, m2, p2);
    const bool on = step_on(c, t);
    lds[HELD ? (on ? own : 0) + (sg > 0 ? t + 1 : Lp - 2 - t) : (on ? o + sg : 0)] = nv;
    eps += on ? fabs(nv - cur) : 0.0;
}

// One column with its window held across slabs, records in a register ring that
// runs on from slab to slab.
template <int COORD, int DIR, int TKC>
__device__ __forceinline__ void fwd_column(const SweepArgs& a, const Geo& G, int src, int TI, int TJ, double* lds) {
    using D = Dir<DIR>;
    using Win = Window<DIR, TKC>;
    constexpr int ng = TKC / kPre, nl = Win::nload;
    const double* __restrict__ mdl = a.model + (long long)D::lay * G.Sa * 4;
    const double2* __restrict__ lon = a.lon + (long long)src * G.n[2];
    const Src S = a.src[src];
    TileCtx c = col_ctx<DIR>(G, S, TI, TJ);
    const Col cl = make_col(G, a.T, c.i, c.j);
    const LfCol W = lf_col<COORD>(G, S, cl, a.kappa);
    double* __restrict__ fld = a.field + (long long)src * G.N;
    const long long xlo = -(long long)src * G.N, xhi = (long long)(a.nsrc - src) * G.N - 2;
    const int lo = (int)(xlo > -1 ? xlo : -1), hi = (int)(xhi < G.N ? xhi : G.N);
    int own = ((c.li + 1) * kTC + c.lj + 1) * Win::Lp;
    double eps = 0.0;
    FwdSlot ring[kPre];
    d2u pf[nl], first;
    slab_ctx<DIR, true>(G, S, c, col_tile_lo(G, TI + TJ) * TKC, TKC);
    win_load<DIR, TKC>(G, c, fld, lo, hi, c.kq0, pf);
    first = win_first<DIR, TKC>(G, c, fld, lo, hi);
#pragma unroll
    for (int u = 0; u < kPre; ++u) fwd_fetch<DIR>(c, mdl, lon, c.t0 + u, ring[u]);
    march_column<DIR, true>(a, G, src, TI, TJ, [&](int TK, const Handover& h) {
        slab_ctx<DIR, true>(G, S, c, TK * TKC, TKC);
        if (c.t1 <= c.t0) {  // a ragged column's slab with no nodes
            publish(h.own, h.done);
            return;
        }
        win_put<DIR, TKC>(c, lds, pf);
        win_put_first<DIR, TKC>(lds, own, first);
        wait_upstream(h.up, h.target, h.lost);
        win_halo<DIR, TKC>(G, c, fld, lo, hi, lds);
        __syncthreads();
        // t0 is a multiple of 8, and so of a group's steps; steps past t1 are off
        auto group = [&](auto gc) {
            constexpr int g = decltype(gc)::value;
            asm volatile("" : "+v"(c.rr0), "+v"(c.tt0), "+v"(own));  // (or the addresses of all groups are formed at once)
            // loads return in order: the next window's, from memory, go out together in front of
            // one group's record loads, so that the records wait for them once a slab
            if (g == 0 && h.more) win_load<DIR, TKC>(G, c, fld, lo, hi, c.kq0 + TKC, pf);
            if (g * kPre < c.t0 || g * kPre >= c.t1) return;
#pragma unroll
            for (int u = 0; u < kPre; ++u) {
                fwd_step<COORD, DIR, true>(G, S, W, c, lds, own, Win::Lp, g * kPre + u, ring[u], eps);
                fwd_fetch<DIR>(c, mdl, lon, g * kPre + u + kPre, ring[u]);
            }
        };
        static_assert(ng == 4, "groups of a slab");
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        group(std::integral_constant<int, 2>{});
        group(std::integral_constant<int, 3>{});
        __syncthreads();
        first = win_carry<DIR, TKC>(lds, own);
        win_store<DIR, TKC, true>(G, c, fld, lds);
        publish(h.own, h.done);
        win_store<DIR, TKC, false>(G, c, fld, lds);
        fwd_kface_nodes<DIR>(G, S, c, fld, lds, own, Win::Lp, eps);
        __syncthreads();
    });
    eps = wave_sum(eps);
    if (c.lane == 0) part_add(a.part + (long long)src * a.nslots + TI * G.nt[1] + TJ, DIR, eps);
}

// ------------------------------------------------------- windows of whole lines
// What a batch that fills the chip waits for is lines: a column's segment of a
// slab lies across two 128-byte lines or more, and the L2 has turned over before
// the next slab wants the last one again (24 sweeps of 128 sources of 101^3 in
// slabs of 28 steps read 5.6e8 lines from beyond the L2s, the fields have 2.0e8;
// whole lines 3.6e8).  Here the field lives in the workspace with its rows padded
// to whole lines (G.sj nodes a row), and a column's window is two of them.  Which
// batches gain by it: lines_of.
//
// Let kappa be a node's place in its row, counted in the sweep's direction: the
// element itself (s2 > 0) or G.sj - 1 minus it, kappa = k' + delta.  Line m of a
// column holds kappa in [16 m, 16 m + 16).  Walk m takes lane (li, lj) over
// kappa = 16 m - 1 - li - lj + t, t = 0 .. 15: with the neighbours at kappa - 1
// and kappa + 1 all lanes stay in [16 m - 16, 16 m + 16), lines m - 1 and m.  After
// it line m - 1 is final in all columns and goes out whole; line m + 1, loaded
// during the walk, takes its place.  kappa is the same for a tile and its
// neighbours: walk m needs line m of the upstream halo, final after walk m + 1
// over there.
//
// In LDS column (ci, cj) has 32 slots at 324 ci + 32 cj, kappa in slot kappa % 32
// (s2 < 0: 31 minus that, so that pairs keep the order of memory); 324 spreads
// the lanes' slots over the banks.  A lane's own value at kappa and the one
// below stay in registers from step to step.
constexpr int kLine = kLineDepth;
constexpr int kLineRow = 324;
constexpr int kLinesLds = kTC * kLineRow * 8;

template <int DIR>
__device__ __forceinline__ int line_slot(int kap) {
    return Dir<DIR>::s2 > 0 ? kap & 31 : (31 - kap) & 31;
}
// first slot of line m, and its first element in a row
template <int DIR>
__device__ __forceinline__ int line_base(int m) {
    return Dir<DIR>::s2 > 0 ? (m & 1) * kLine : (1 - (m & 1)) * kLine;
}
template <int DIR>
__device__ __forceinline__ int line_elem(const Geo& G, int m) {
    return Dir<DIR>::s2 > 0 ? m * kLine : (int)G.sj - kLine - m * kLine;
}
template <int DIR>
__device__ __forceinline__ int line_addr(const Geo& G, const TileCtx& c, int ci, int cj) {
    using D = Dir<DIR>;
    return (stage_origin<D::s0>(G, 0, c.TI) + D::s0 * ci) * (int)G.si +
           (stage_origin<D::s1>(G, 1, c.TJ) + D::s1 * cj) * (int)G.sj;
}

// line m of the tile's own columns and its downstream halo, eight columns a load
// (columns past a ragged tile's halo re-read its last one)
template <int DIR>
__device__ __forceinline__ void line_load(const Geo& G, const TileCtx& c, const double* __restrict__ fld, int m,
                                          d2a (&pf)[10]) {
    const int lane = opaque_lane(c);
    const int sub = lane >> 3, e = line_elem<DIR>(G, m) + 2 * (lane & 7);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        int ci, cj;
        Window<DIR, kLine>::col(r, sub, ci, cj);
        pf[r] = *reinterpret_cast<const d2a*>(fld + line_addr<DIR>(G, c, min(ci, c.ext_i + 1), min(cj, c.ext_j + 1)) + e);
    }
}

template <int DIR>
__device__ __forceinline__ void line_put(const TileCtx& c, double* lds, int m, const d2a (&pf)[10]) {
    const int lane = opaque_lane(c);
    const int sub = lane >> 3, q = line_base<DIR>(m) + 2 * (lane & 7);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        int ci, cj;
        Window<DIR, kLine>::col(r, sub, ci, cj);
        *reinterpret_cast<d2a*>(lds + ci * kLineRow + cj * 32 + q) = pf[r];
    }
}

template <int DIR>
__device__ __forceinline__ void line_halo(const Geo& G, const TileCtx& c, const double* __restrict__ fld, int m,
                                          double* lds) {
    const int lane = opaque_lane(c);
    const int sub = lane >> 3, e = 2 * (lane & 7), h = sub + 1;
    const d2a v0 = *reinterpret_cast<const d2a*>(fld + line_addr<DIR>(G, c, 0, min(h, c.ext_j + 1)) + line_elem<DIR>(G, m) + e);
    const d2a v1 = *reinterpret_cast<const d2a*>(fld + line_addr<DIR>(G, c, min(h, c.ext_i + 1), 0) + line_elem<DIR>(G, m) + e);
    const int q = line_base<DIR>(m) + e;
    *reinterpret_cast<d2a*>(lds + h * 32 + q) = v0;
    *reinterpret_cast<d2a*>(lds + h * kLineRow + q) = v1;
}

// line m of the own columns: EDGES, those with li = 7 or lj = 7, or all others
template <int DIR, bool EDGES>
__device__ __forceinline__ void line_store(const Geo& G, const TileCtx& c, double* __restrict__ fld, int m,
                                           const double* lds) {
    const int lane = opaque_lane(c);
    const int h = (lane >> 3) + 1, e = 2 * (lane & 7), q = line_base<DIR>(m) + e;
    constexpr int n = EDGES ? 2 : 7;
    d2a v[n];
#pragma unroll
    for (int u = 0; u < n; ++u) {
        const int ci = EDGES ? (u == 0 ? kBI : h) : u + 1, cj = EDGES ? (u == 0 ? h : kBJ) : h;
        v[u] = *reinterpret_cast<const d2a*>(lds + ci * kLineRow + cj * 32 + q);
    }
#pragma unroll
    for (int u = 0; u < n; ++u) {
        const int ci = EDGES ? (u == 0 ? kBI : h) : u + 1, cj = EDGES ? (u == 0 ? h : kBJ) : h;
        if (ci <= c.ext_i && cj <= c.ext_j && (EDGES ? u == 0 || ci < kBI : cj < kBJ))
            *reinterpret_cast<d2a*>(fld + line_addr<DIR>(G, c, ci, cj) + line_elem<DIR>(G, m) + e) = v[u];
    }
}

// the own columns' k-face nodes in line m copy their end nodes (fwd_kface_nodes)
template <int DIR>
__device__ __forceinline__ void line_kfaces(const Geo& G, const Src& S, const TileCtx& c, double* lds, int own, int m,
                                            int delta, double& eps) {
    using D = Dir<DIR>;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int kap = e == 0 ? delta - 1 : delta + G.m[2];
        if (kap / kLine != m) continue;
        const int kb = c.kbase + D::s2 * (e == 0 ? -1 : G.m[2]);  // absolute k of the boundary node
        if (!c.colv || in_fixed(S, c.i, c.j, kb)) continue;
        const double nv = lds[own + line_slot<DIR>(e == 0 ? kap + 1 : kap - 1)];
        const double old = lds[own + line_slot<DIR>(kap)];
        lds[own + line_slot<DIR>(kap)] = nv;
        eps += fabs(nv - old);
    }
}

template <int COORD, int DIR>
__device__ __forceinline__ void fwd_line_column(const SweepArgs& a, const Geo& G, int src, int TI, int TJ, double* lds) {
    using D = Dir<DIR>;
    constexpr int ng = kLine / kPre;
    const double* __restrict__ mdl = a.model + (long long)D::lay * G.Sa * 4;
    const double2* __restrict__ lon = a.lon + (long long)src * G.n[2];
    const Src S = a.src[src];
    TileCtx c = col_ctx<DIR>(G, S, TI, TJ);
    const Col cl = make_col(G, a.T, c.i, c.j);
    const LfCol W = lf_col<COORD>(G, S, cl, a.kappa);
    double* __restrict__ fld = a.field + (long long)src * G.Nf;
    const int delta = D::s2 > 0 ? 1 : (int)G.sj + 1 - G.n[2];
    const int nlines = (int)G.sj / kLine, mhi = (G.m[2] + delta + c.ext_i + c.ext_j - 2) / kLine;
    const int u0 = kBI * (TI + TJ) - 1 - delta;  // u of step t = 0 of walk 0
    int own = (c.li + 1) * kLineRow + (c.lj + 1) * 32;
    double eps = 0.0;
    FwdSlot ring[kPre];
    d2a pf[10];
    slab_ctx<DIR, true>(G, S, c, u0, kLine);
    line_load<DIR>(G, c, fld, 0, pf);
    const int tf = (delta + 1) & ~(kPre - 1);  // the first group with a node, counted from walk 0
#pragma unroll
    for (int u = 0; u < kPre; ++u) fwd_fetch<DIR>(c, mdl, lon, tf + u, ring[u]);
    unsigned long long* word = progress_words(a, src) + TI * G.nt[1] + TJ;
    const unsigned long long* up = nullptr;
    if (threadIdx.x == 0 && TI > 0) up = word - G.nt[1];
    if (threadIdx.x == 1 && TJ > 0) up = word - 1;
    // progress: (number of the sweep << 16) + lines that are final
    const unsigned long long base = ((unsigned long long)a.iter[src] * 8 + DIR + 1) << 16;
    for (int m = 0; m <= mhi; ++m) {
        slab_ctx<DIR, true>(G, S, c, u0 + m * kLine, kLine);
        if (m < nlines) {
            line_put<DIR>(c, lds, m, pf);
            wait_upstream(up, base + m + 1, lost_word(a, src));
            line_halo<DIR>(G, c, fld, m, lds);
        }
        __syncthreads();
        auto group = [&](auto gc) {
            constexpr int g = decltype(gc)::value;
            int kap = kLine * m - 1 - c.li - c.lj + g * kPre;
            asm volatile("" : "+v"(c.rr0), "+v"(c.tt0), "+v"(own), "+v"(kap));  // (or the addresses of all groups are formed at once)
            // together and ahead of a group's record loads, as in fwd_column
            if (g == 0 && m + 1 < nlines) line_load<DIR>(G, c, fld, m + 1, pf);
            if (g * kPre + kPre <= c.t0 || g * kPre >= c.t1) return;
            double upk = lds[own + line_slot<DIR>(kap - 1)], cur = lds[own + line_slot<DIR>(kap)];
            int at = own + line_slot<DIR>(kap);
#pragma unroll
            for (int u = 0; u < kPre; ++u) {
                const int t = g * kPre + u;
                FwdSlot& r = ring[u];
                const int an = own + line_slot<DIR>(kap + u + 1);
                const double dnk = lds[an];
                const double up_i = lds[at - kLineRow], dn_i = lds[at + kLineRow];
                const double up_j = lds[at - 32], dn_j = lds[at + 32];
                const double m0 = D::s0 > 0 ? up_i : dn_i, p0 = D::s0 > 0 ? dn_i : up_i;
                const double m1 = D::s1 > 0 ? up_j : dn_j, p1 = D::s1 > 0 ? dn_j : up_j;
                const double m2 = D::s2 > 0 ? upk : dnk, p2 = D::s2 > 0 ? dnk : upk;
                const double nv = lf_update<COORD>(G, S, W, r.f1, r.sn, r.sx, r.ma, r.mb, r.mc, cur, m0, p0, m1, p1, m2, p2);
                const bool on = step_on(c, t);
                lds[on ? at : 0] = nv;  // no branch in a step, as in fwd_step
                eps += on ? fabs(nv - cur) : 0.0;
                upk = on ? nv : cur;
                cur = dnk;
                at = an;
                fwd_fetch<DIR>(c, mdl, lon, t + kPre, r);
            }
        };
        static_assert(ng == 4, "groups of a walk");
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        group(std::integral_constant<int, 2>{});
        group(std::integral_constant<int, 3>{});
        const bool last = m == mhi, prev = m > 0, cur_too = last && m < nlines;
        if (prev) line_kfaces<DIR>(G, S, c, lds, own, m - 1, delta, eps);
        if (cur_too) line_kfaces<DIR>(G, S, c, lds, own, m, delta, eps);
        __syncthreads();
        if (prev) line_store<DIR, true>(G, c, fld, m - 1, lds);
        if (cur_too) line_store<DIR, true>(G, c, fld, m, lds);
        publish(word, last ? base + 0xffffu : base + m);
        if (prev) line_store<DIR, false>(G, c, fld, m - 1, lds);
        if (cur_too) line_store<DIR, false>(G, c, fld, m, lds);
        __syncthreads();
    }
    eps = wave_sum(eps);
    if (c.lane == 0) part_add(a.part + (long long)src * a.nslots + TI * G.nt[1] + TJ, DIR, eps);
}

template <int COORD, int DIR>
__global__ void __launch_bounds__(64, 2) k_fwd_lines(SweepArgs a, int c0, int cn) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    march(a, a.G, c0, cn, [&](int src, int TI, int TJ) { fwd_line_column<COORD, DIR>(a, a.G, src, TI, TJ, lds); });
}

// the solution out of its padded rows
__global__ void __launch_bounds__(256) k_unpad(Geo G, const double* __restrict__ f, double* __restrict__ out) {
    const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= G.N) return;
    const int k = (int)(x % G.n[2]);
    const long long q = x / G.n[2];
    out[(long long)blockIdx.y * G.N + x] = f[(long long)blockIdx.y * G.Nf + q * G.sj + k];
}

// TKC: the tile depth as a compile-time constant (0: read from the geometry); at
// 16 the window is held across slabs.
template <int COORD, int DIR, int TKC>
__global__ void __launch_bounds__(64, TKC == 16 ? 2 : 3) k_fwd_sweep(SweepArgs a, int c0, int cn) {
    using D = Dir<DIR>;
    extern __shared__ __attribute__((aligned(16))) double lds[];
    Geo G = a.G;
    if (TKC > 0) G.tk = TKC;
    if constexpr (TKC == 16) {
        march(a, G, c0, cn, [&](int src, int TI, int TJ) { fwd_column<COORD, DIR, TKC>(a, G, src, TI, TJ, lds); });
    } else {
        const double* __restrict__ mdl = a.model + (long long)D::lay * G.Sa * 4;
        const int Lp = tile_pitch(G.tk);
        march(a, G, c0, cn, [&](int src, int TI, int TJ) {
            const double2* __restrict__ lon = a.lon + (long long)src * G.n[2];
            const Src S = a.src[src];
            TileCtx c = col_ctx<DIR>(G, S, TI, TJ);
            const Col cl = make_col(G, a.T, c.i, c.j);
            const LfCol W = lf_col<COORD>(G, S, cl, a.kappa);
            double* __restrict__ fld = a.field + (long long)src * G.N;
            const int own = ((c.li + 1) * kTC + c.lj + 1) * Lp;
            double eps = 0.0;
            march_column<DIR, false>(a, G, src, TI, TJ, [&](int TK, const Handover& h) {
                slab_ctx<DIR>(G, S, c, TK * G.tk, G.tk);
                if (c.t1 <= c.t0) return;  // a ragged column's slab with no nodes
                FwdSlot ring[kPre];
#pragma unroll
                for (int u = 0; u < kPre; ++u) fwd_fetch<DIR>(c, mdl, lon, c.t0 + u, ring[u]);
                wait_upstream(h.up, h.target, h.lost);
                stage_tile<DIR>(G, c, fld, -(long long)src * G.N, (long long)(a.nsrc - src) * G.N - 2, lds);
                __syncthreads();
                // the step count is padded to a multiple of kPre (the LDS reads of a padded step
                // stay inside the window: at most 3 entries past a column that others follow)
                for (int tb = c.t0; tb < c.t1; tb += kPre) {
#pragma unroll
                    for (int u = 0; u < kPre; ++u) {
                        fwd_step<COORD, DIR, false>(G, S, W, c, lds, own, Lp, tb + u, ring[u], eps);
                        fwd_fetch<DIR>(c, mdl, lon, tb + u + kPre, ring[u]);
                    }
                }
                __syncthreads();
                unstage_tile<DIR>(G, c, fld, lds, Lp);
                fwd_kface_nodes<DIR>(G, S, c, fld, lds, own, Lp, eps);
            });
            eps = wave_sum(eps);
            if (c.lane == 0) part_add(a.part + (long long)src * a.nslots + TI * G.nt[1] + TJ, DIR, eps);
        });
    }
}

// model records (s, 1 - 2 xi, 2 eta, 1 + 2 xi) in the four aligned layouts
__global__ void k_model_records(Geo G, const double* __restrict__ s, const double* __restrict__ xi,
                                const double* __restrict__ eta, double* __restrict__ out) {
    const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= G.N) return;
    const int k = (int)(x % G.n[2]);
    const long long q = x / G.n[2];
    const int j = (int)(q % G.n[1]), i = (int)(q / G.n[1]);
    // the lower-right block of M = [[1 - 2 xi, 2 eta], [2 eta, 1 + 2 xi]]
    const double2 v0 = make_double2(s[x], 1.0 - 2.0 * xi[x]), v1 = make_double2(2.0 * eta[x], 1.0 + 2.0 * xi[x]);
    for (int lay = 0; lay < 4; ++lay) {
        double2* o = reinterpret_cast<double2*>(out + ((long long)lay * G.Sa + arec_idx(G, lay, i, j, k)) * 4);
        o[0] = v0;
        o[1] = v1;
    }
}

// Value of node p once the boundary pass is done: interior and fixed nodes as
// stored; a boundary node copies its inward neighbour along its largest
// boundary axis, which has one boundary axis fewer (depth <= 3).
template <int BUDGET>
__device__ __forceinline__ double fwd_bval(const Geo& G, const Src& S, const double* f, int i, int j, int k) {
    const int p[3] = {i, j, k};
    const int as = astar_of(G, p);
    if constexpr (BUDGET == 0) {
        return f[nidx(G, i, j, k)];
    } else {
        if (as < 0 || in_fixed(S, i, j, k)) return f[nidx(G, i, j, k)];
        int q1[3] = {i, j, k};
        q1[as] += (p[as] == 0) ? 1 : -1;
        return fwd_bval<BUDGET - 1>(G, S, f, q1[0], q1[1], q1[2]);
    }
}

__global__ void __launch_bounds__(kBndThreads) k_fwd_bnd(SweepArgs a, int dir) {
    __shared__ double sh[4];
    const int src = blockIdx.y;
    if (blockIdx.x == 0) queue_reset(a, src);
    if (!a.active[src]) return;
    const Geo& G = a.G;
    const Src S = a.src[src];
    double* fld = a.field + (long long)src * G.Nf;
    const long long b = (long long)blockIdx.x * kBndThreads + threadIdx.x;
    double d = 0.0;
    if (b < G.NB) {
        int i, j, k;
        bnd_decode(G, b, i, j, k);
        // (the sweeps set the nodes on a k face only)
        if (!in_fixed(S, i, j, k) && !kface_only(G, i, j)) {
            const double nv = fwd_bval<3>(G, S, fld, i, j, k);
            const long long x = nidx(G, i, j, k);
            d = fabs(nv - fld[x]);
            fld[x] = nv;
        }
    }
    d = block_sum256(d, sh);
    if (threadIdx.x == 0) part_add(a.part + (long long)src * a.nslots + G.ncols + blockIdx.x, dir, d);
}

__device__ __forceinline__ double fixed_sum(const double* p, int cnt, double* sh) {
    double v = 0.0;
    for (int q = threadIdx.x; q < cnt; q += blockDim.x) v += p[q];
    return block_sum256(v, sh);
}

__device__ __forceinline__ void finish_iteration(const SweepArgs& a, int src, double eps) {
    const int it = a.iter[src] + 1;
    a.iter[src] = it;
    if (a.eps_hist) a.eps_hist[(long long)src * a.hist_stride + (it - 1)] = eps;
    const Outcome o = iteration_outcome(eps, a.tol, it, a.max_iter, *lost_word(a, src) != 0u);
    a.status[src] = o.status;
    if (o.done) {
        a.active[src] = 0;
        atomicSub(a.counter, 1);
    }
}

__global__ void __launch_bounds__(256) k_fwd_finalize(SweepArgs a) {
    __shared__ double sh[4];
    const int src = blockIdx.x;
    if (!a.active[src]) return;
    const double tot = fixed_sum(a.part + (long long)src * a.nslots, a.G.ncols + a.nbblocks, sh);
    if (threadIdx.x == 0) finish_iteration(a, src, tot / (double)a.G.N);
}

// --------------------------------------------------------- adjoint solve
// Local state at an arbitrary interior node, loading what it needs.
template <int COORD>
__device__ __forceinline__ void state_at(const Geo& G, const Tabs& T, const Src& S, const double* __restrict__ tau,
                                         const double* __restrict__ xi, const double* __restrict__ eta, int i,
                                         int j, int k, Col& c, Loc& L) {
    c = make_col(G, T, i, j);
    const long long x = nidx(G, i, j, k);
    const double2 t2 = T.t2[k];
    local_state<COORD>(G, S, c, t2.x, t2.y, xi[x], eta[x], tau[x], tau[x - G.si], tau[x + G.si], tau[x - G.sj],
                       tau[x + G.sj], tau[x - 1], tau[x + 1], L);
}

__device__ __forceinline__ double g_of(const Col& c, int a) { return a == 0 ? 1.0 : (a == 1 ? c.g1 : c.g2); }

// J_{x, x + dirn e_a} of an interior non-fixed row x (dirn = +1 or -1):
//   alpha_a - beta_a or -alpha_a - beta_a with alpha_a = T0 g_a (MP)_a / (2 h_a H),
//   beta_a = kappa T0 g_a / (2 h_a).
__device__ __forceinline__ double row_off(const Geo& G, const Col& c, const Loc& L, double kappa, int a, int dirn) {
    const double ga = g_of(c, a);
    const double alpha = L.T0 * ga * L.MP[a] / (2.0 * G.h[a] * L.H);
    const double beta = kappa * L.T0 * ga / (2.0 * G.h[a]);
    return dirn > 0 ? alpha - beta : -alpha - beta;
}

// Adjoint coefficient records: the six couplings of a node's column equation
// divided by its diagonal (48 bytes).  Default: four line-aligned
// row-coalesced layouts per source (arec_idx), so the 8 records a tile row
// reads on one step are whole 128-byte lines in every sweep direction.
// Compact (TT_FLAG_COMPACT_ADJOINT): one copy per source in node order
// [nsrc][N][6], a ninth of the memory at 101^3; a lane's records for
// consecutive steps are then contiguous along its column, but a tile row's
// records lie on different lines.
constexpr int kRec = 6;

// store a node's row {c+_0, c-_0, c+_1, c-_1, c+_2, c-_2, diag, -} divided by
// its diagonal, the diagonal into diag_all, and a zero right-hand side
// (k_adj_rhs adds to it); a zero diagonal (no row) stores a zero record
__device__ __forceinline__ void store_record(const Geo& G, double* __restrict__ coef_all, double* __restrict__ diag_all,
                                             double* __restrict__ rhs_all, int src, long long x, int i, int j, int k,
                                             const double (&out)[8], int compact) {
    const double d = out[6];
    double2 rec[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
        rec[q] = d != 0.0 ? make_double2(out[2 * q] / d, out[2 * q + 1] / d) : make_double2(0.0, 0.0);
    diag_all[(long long)src * G.N + x] = d;
    rhs_all[(long long)src * G.N + x] = 0.0;
    if (compact) {
        double2* cf = reinterpret_cast<double2*>(coef_all + ((long long)src * G.N + x) * kRec);
#pragma unroll
        for (int q = 0; q < 3; ++q) cf[q] = rec[q];
        return;
    }
    for (int lay = 0; lay < 4; ++lay) {
        double2* cf =
            reinterpret_cast<double2*>(coef_all + (((long long)src * 4 + lay) * G.Sa + arec_idx(G, lay, i, j, k)) * kRec);
#pragma unroll
        for (int q = 0; q < 3; ++q) cf[q] = rec[q];
    }
}

// Coefficients of the transposed system at every node of every source, stored
// as the column equation of x divided by its diagonal
// J_xx: record {in+_0, in-_0, in+_1, in-_1, in+_2, in-_2} / J_xx, with
// in+-_a = J_{x +- e_a, x}, the coefficient of lambda(x +- e_a) (zero unless x
// is interior and not fixed).  J_xx goes to diag [nsrc][N] (0 where there is
// no row); the right-hand side, divided likewise, is added to rhs [nsrc][N] by
// k_adj_rhs.  bnd_in[b] = J_{x, b} for each face node b and its interior
// neighbour x (zero when x is fixed).
template <int COORD>
__global__ void __launch_bounds__(256) k_adj_coef(SweepArgs a, const double* __restrict__ tau_all,
                                                  double* __restrict__ coef_all, double* __restrict__ bnd_all,
                                                  double* __restrict__ diag_all, double* __restrict__ rhs_all) {
    const Geo& G = a.G;
    const int src = blockIdx.y;
    const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= G.N) return;
    const Src S = a.src[src];
    const double* tau = tau_all + (long long)src * G.N;
    const int k = (int)(x % G.n[2]);
    const long long q = x / G.n[2];
    const int j = (int)(q % G.n[1]), i = (int)(q / G.n[1]);
    double out[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const bool interior = i > 0 && i < G.n[0] - 1 && j > 0 && j < G.n[1] - 1 && k > 0 && k < G.n[2] - 1;
    if (interior && !in_fixed(S, i, j, k)) {
        Col c;
        Loc L;
        state_at<COORD>(G, a.T, S, tau, a.xi, a.eta, i, j, k, c, L);
        double diag = (L.t[0] * L.MP[0] + L.t[1] * L.MP[1] + L.t[2] * L.MP[2]) / L.H;
        for (int ax = 0; ax < 3; ++ax) diag += 2.0 * (a.kappa * L.T0 * g_of(c, ax) / (2.0 * G.h[ax]));
        out[6] = diag;
        for (int ax = 0; ax < 3; ++ax) {
            for (int sgn = 0; sgn < 2; ++sgn) {
                const int dirn = sgn == 0 ? 1 : -1;
                int y[3] = {i, j, k};
                y[ax] += dirn;
                double v = 0.0;
                if (!in_fixed(S, y[0], y[1], y[2])) {
                    if (on_bnd(G, ax, y[ax])) {
                        v = -1.0;  // the face row of y copies x
                    } else {
                        Col cy;
                        Loc Ly;
                        state_at<COORD>(G, a.T, S, tau, a.xi, a.eta, y[0], y[1], y[2], cy, Ly);
                        v = row_off(G, cy, Ly, a.kappa, ax, -dirn);
                    }
                }
                out[2 * ax + sgn] = v;
                if (on_bnd(G, ax, y[ax]))
                    bnd_all[(long long)src * G.NB + bnd_encode(G, y[0], y[1], y[2])] =
                        row_off(G, c, L, a.kappa, ax, dirn);
            }
        }
    }
    store_record(G, coef_all, diag_all, rhs_all, src, x, i, j, k, out, a.compact);
}

// d chi / d tau = sum_m R_m w_c T0(c) (discrete adjoint), or the point sources
// sum_m R_m w_c of Eq. (5) (continuous adjoint, with_t0 = 0), added in receiver
// order, one wave per source.  64 receivers are taken at a time, one a lane: a
// lane adds the contributions to those corners of its cell that no earlier lane's
// cell has, its own and, in receiver order, those of the later lanes whose cells
// share the corner, so every node sees the additions of the plain loop in its
// order.  (That loop on one thread per source waited for four dependent reads per
// corner: 64 sources of 101^3 4.3 ms for 500 receivers; a wave per source 0.27.)
template <int COORD>
__global__ void __launch_bounds__(64) k_adj_rhs(SweepArgs a, const double* __restrict__ diag_all,
                                                double* __restrict__ rhs_all, int* __restrict__ box_all, int nrec,
                                                const double* __restrict__ rec, const double* __restrict__ R,
                                                int with_t0) {
    __shared__ int cell[3][64];
    __shared__ double fr[3][64], rm[64];
    const int src = blockIdx.x, lane = threadIdx.x;
    const Geo& G = a.G;
    const Src S = a.src[src];
    const double* dg = diag_all + (long long)src * G.N;
    double* rh = rhs_all + (long long)src * G.N;
    double* brhs = const_cast<double*>(a.bnd_rhs) + (long long)src * G.NB;
    int lo[3] = {G.n[0], G.n[1], G.n[2]}, hi[3] = {-1, -1, -1};
    for (int m0 = 0; m0 < nrec; m0 += 64) {
        const int cnt = min(64, nrec - m0);
        const int m = m0 + min(lane, cnt - 1);
        const bool on = lane < cnt;
        const Tri t = tri_of(G, rec[3 * m], rec[3 * m + 1], rec[3 * m + 2]);
        for (int ax = 0; ax < 3; ++ax) {
            cell[ax][lane] = t.b[ax];
            fr[ax][lane] = t.f[ax];
            lo[ax] = min(lo[ax], t.b[ax]);
            hi[ax] = max(hi[ax], t.b[ax] + 1);
        }
        rm[lane] = R[(long long)src * nrec + m];
        __syncthreads();
        unsigned long long near = 0ull;  // receivers whose cells touch this lane's
        for (int q = 0; q < cnt; ++q)
            if ((unsigned)(cell[0][q] - t.b[0] + 1) <= 2u && (unsigned)(cell[1][q] - t.b[1] + 1) <= 2u &&
                (unsigned)(cell[2][q] - t.b[2] + 1) <= 2u)
                near |= 1ull << q;
        if (on) {
            for (int cc = 0; cc < 8; ++cc) {
                const int i = t.b[0] + (cc >> 2), j = t.b[1] + ((cc >> 1) & 1), k = t.b[2] + (cc & 1);
                const Col c = make_col(G, a.T, i, j);
                const double2 t2 = a.T.t2[k];
                double T0, tt[3];
                factor<COORD>(S, c, t2.x, t2.y, T0, tt);
                const long long xn = nidx(G, i, j, k);
                // divided by the row's diagonal like the records (a row-less node's
                // value is never read by the sweeps)
                const double d = dg[xn];
                const bool face = on_bnd(G, 0, i) || on_bnd(G, 1, j) || on_bnd(G, 2, k);
                const long long bn = face ? bnd_encode(G, i, j, k) : 0;
                double acc = rh[xn], bacc = face ? brhs[bn] : 0.0;
                bool mine = true;
                for (unsigned long long w = near; w; w &= w - 1) {
                    const int q = __ffsll(w) - 1;
                    Tri u;
                    unsigned in = 1u;
                    const int id[3] = {i, j, k};
                    for (int ax = 0; ax < 3; ++ax) {
                        u.b[ax] = id[ax] - cell[ax][q];  // the node's corner of cell q, if it is one
                        u.f[ax] = fr[ax][q];
                        in &= (unsigned)u.b[ax] <= 1u;
                    }
                    if (!in) continue;
                    if (q < lane) {
                        mine = false;
                        break;
                    }
                    const double v = with_t0 ? rm[q] * tri_w(u, u.b[0], u.b[1], u.b[2]) * T0
                                             : rm[q] * tri_w(u, u.b[0], u.b[1], u.b[2]);
                    acc += d != 0.0 ? v / d : v;
                    bacc += v;
                }
                if (mine) {
                    rh[xn] = acc;
                    if (face) brhs[bn] = bacc;
                }
            }
        }
        __syncthreads();
    }
    for (int ax = 0; ax < 3; ++ax) {
        for (int w = 32; w > 0; w >>= 1) {
            lo[ax] = min(lo[ax], __shfl_xor(lo[ax], w, 64));
            hi[ax] = max(hi[ax], __shfl_xor(hi[ax], w, 64));
        }
        if (lane == 0) {
            box_all[src * 6 + 2 * ax] = lo[ax];
            box_all[src * 6 + 2 * ax + 1] = hi[ax];
        }
    }
}

// a step's record (and, in tiles that meet the source's right-hand side, its
// right-hand side value), fetched kPreAdj steps ahead
struct AdjSlot {
    double r[kRec];
    double b;
};

template <int DIR, bool RHS, bool COMPACT>
__device__ __forceinline__ void adj_fetch(const TileCtx& c, const double* __restrict__ cf,
                                          const double* __restrict__ rh, long long xb, int t, AdjSlot& r) {
    using D = Dir<DIR>;
    const int kp = min(max(c.kp0 + t, c.kplo), c.kphi);
    const long long x = xb + D::s2 * kp;
    // |rstep| = n1p < 2^23 and 0 <= kp < n2 <= 8192: a 24-bit product
    const double2* rc =
        reinterpret_cast<const double2*>(cf + (COMPACT ? x : (long long)(c.rbase + __mul24(c.rstep, kp))) * kRec);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double2 v = rc[q];
        r.r[2 * q] = v.x;
        r.r[2 * q + 1] = v.y;
    }
    r.b = RHS ? rh[x] : 0.0;
}

// does the tile (its columns, and the k' range of its slab) meet the index box
// of the source's nonzero right-hand side?
template <int DIR>
__device__ __forceinline__ bool tile_meets_box(const Geo& G, const TileCtx& c, const int* bx) {
    using D = Dir<DIR>;
    const int i0 = 8 * c.TI, i1 = 8 * c.TI + c.ext_i - 1, j0 = 8 * c.TJ, j1 = 8 * c.TJ + c.ext_j - 1;
    const int kq0 = max(0, c.U0 - i1 - j1), kq1 = min(G.m[2] - 1, c.U0 + G.tk - 1 - i0 - j0);
    const int ia = D::s0 > 0 ? 1 + i0 : G.n[0] - 2 - i1, ib = D::s0 > 0 ? 1 + i1 : G.n[0] - 2 - i0;
    const int ja = D::s1 > 0 ? 1 + j0 : G.n[1] - 2 - j1, jb = D::s1 > 0 ? 1 + j1 : G.n[1] - 2 - j0;
    const int ka = D::s2 > 0 ? 1 + kq0 : G.n[2] - 2 - kq1, kb = D::s2 > 0 ? 1 + kq1 : G.n[2] - 2 - kq0;
    return ia <= bx[1] && ib >= bx[0] && ja <= bx[3] && jb >= bx[2] && ka <= bx[5] && kb >= bx[4] && kq0 <= kq1;
}

// A k-face node of an interior column (its row: lambda_b = rhs_b - J_{x, b}
// lambda_x, x the column's end node, no other row refers to it): the tile that
// updates x sets it after its walk, as fwd_kface_nodes does; coupling and
// right-hand side are loaded before the wait for upstream.  (In the boundary
// pass, a line of its own each: 64 sources of 101^3 193 us a pass beside another
// group's sweep, now 161.)
struct AdjFace {
    double in[2], rhs[2];
    bool on[2];
};

template <int DIR>
__device__ __forceinline__ void adj_kface_load(const SweepArgs& a, const Geo& G, const Src& S, const TileCtx& c, int src,
                                               AdjFace& f) {
    using D = Dir<DIR>;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int t = (e == 0 ? 0 : G.m[2] - 1) - c.kp0;          // the step that updates the end node
        const int kb = c.kbase + D::s2 * (e == 0 ? -1 : G.m[2]);  // absolute k of the boundary node
        f.on[e] = c.colv && t >= c.t0 && t < c.t1 && !in_fixed(S, c.i, c.j, kb);
        f.in[e] = f.rhs[e] = 0.0;
        if (f.on[e]) {
            const long long b = (long long)src * G.NB + bnd_encode(G, c.i, c.j, kb);
            f.in[e] = a.bnd_in[b];
            f.rhs[e] = a.bnd_rhs[b];
        }
    }
}

template <int DIR>
__device__ __forceinline__ void adj_kface_nodes(const Geo& G, const TileCtx& c, double* __restrict__ fld,
                                                const double* lds, int own, int Lp, const AdjFace& f, double& dsum,
                                                double& asum) {
    using D = Dir<DIR>;
    constexpr int sg = D::s2;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        if (!f.on[e]) continue;
        const int t = (e == 0 ? 0 : G.m[2] - 1) - c.kp0;
        const int o = sg > 0 ? own + t : own + Lp - 1 - t;
        const double old = lds[e == 0 ? o : o + 2 * sg];  // entry t or t + 2: the boundary node
        const double nv = f.rhs[e] - f.in[e] * lds[o + sg];
        fld[nidx(G, c.i, c.j, c.kbase + sg * (e == 0 ? -1 : G.m[2]))] = nv;
        dsum += fabs(nv - old);
        if (DIR == 7) asum += fabs(nv);
    }
}

template <int DIR, bool RHS, bool COMPACT>
__device__ __forceinline__ void adj_tile(const SweepArgs& a, const Geo& G, const Src& S, const TileCtx& c, int src,
                                         double* lds, const Handover& h, double& dsum, double& asum) {
    using D = Dir<DIR>;
    constexpr bool last = (DIR == 7);
    double* __restrict__ fld = a.field + (long long)src * G.N;
    const double* __restrict__ cf =
        a.coef + (COMPACT ? (long long)src * G.N : ((long long)src * 4 + D::lay) * G.Sa) * kRec;
    const double* __restrict__ rh = a.rhs + (long long)src * G.N;
    const long long xb = nidx(G, c.i, c.j, c.kbase);
    const int Lp = tile_pitch(G.tk);

    AdjSlot ring[kPreAdj];
#pragma unroll
    for (int u = 0; u < kPreAdj; ++u) adj_fetch<DIR, RHS, COMPACT>(c, cf, rh, xb, c.t0 + u, ring[u]);
    AdjFace face;
    if (a.kfaces) adj_kface_load<DIR>(a, G, S, c, src, face);
    wait_upstream(h.up, h.target, h.lost);
    stage_tile<DIR>(G, c, fld, -(long long)src * G.N, (long long)(a.nsrc - src) * G.N - 2, lds);
    __syncthreads();

    const int own = ((c.li + 1) * kTC + c.lj + 1) * Lp;
    // the step count is padded to a multiple of kPreAdj: no branch encloses a load
    for (int tb = c.t0; tb < c.t1; tb += kPreAdj) {
#pragma unroll
        for (int u = 0; u < kPreAdj; ++u) {
            const int t = tb + u;
            AdjSlot& r = ring[u];
            // slot of entry t (mirrored columns when s2 < 0): entry t + 1 is at o + s2
            constexpr int sg = D::s2;
            const int o = sg > 0 ? own + t : own + Lp - 1 - t;
            const double cur = lds[o + sg];
            const double up_i = lds[o - kTC * Lp], dn_i = lds[o + kTC * Lp + 2 * sg];
            const double up_j = lds[o - Lp], dn_j = lds[o + Lp + 2 * sg];
            const double up_k = lds[o], dn_k = lds[o + 2 * sg];
            // record: coefficients of lambda(x + e_a), lambda(x - e_a) at 2a, 2a + 1,
            // divided by the diagonal like the right-hand side.  The
            // sweep-downstream terms (values of the previous sweep) go first, the
            // upstream ones (updated on the previous step) last.
            constexpr int di = D::s0 > 0 ? 0 : 1, dj = D::s1 > 0 ? 2 : 3, dk = D::s2 > 0 ? 4 : 5;
            double acc = r.b;
            acc -= r.r[di] * dn_i;
            acc -= r.r[dj] * dn_j;
            acc -= r.r[dk] * dn_k;
            acc -= r.r[di ^ 1] * up_i;
            acc -= r.r[dj ^ 1] * up_j;
            acc -= r.r[dk ^ 1] * up_k;
            const double nv = acc;
            const bool on = step_on(c, t);
            lds[on ? o + sg : 0] = nv;  // no branch in a step, as in k_fwd_sweep
            dsum += on ? fabs(nv - cur) : 0.0;
            if (last) asum += on ? fabs(nv) : 0.0;
            adj_fetch<DIR, RHS, COMPACT>(c, cf, rh, xb, t + kPreAdj, r);
        }
    }
    __syncthreads();
    unstage_tile<DIR>(G, c, fld, lds, Lp);
    if (a.kfaces) adj_kface_nodes<DIR>(G, c, fld, lds, own, Lp, face, dsum, asum);
}

// TKC: compile-time tile depth as for k_fwd_sweep (0: from the geometry)
template <int COORD, int DIR, bool COMPACT, int TKC>
__global__ void __launch_bounds__(64, 3) k_adj_sweep(SweepArgs a, int c0, int cn) {
    extern __shared__ double lds[];
    Geo G = a.G;
    if (TKC > 0) G.tk = TKC;
    march(a, G, c0, cn, [&](int src, int TI, int TJ) {
        const Src S = a.src[src];
        TileCtx c = col_ctx<DIR>(G, S, TI, TJ);
        double dsum = 0.0, asum = 0.0;
        march_column<DIR, false>(a, G, src, TI, TJ, [&](int TK, const Handover& h) {
            slab_ctx<DIR>(G, S, c, TK * G.tk, G.tk);
            if (c.t1 <= c.t0) return;  // a ragged column's slab with no nodes
            // wave-uniform: only tiles that meet the right-hand side read it
            if (tile_meets_box<DIR>(G, c, a.box + src * 6))
                adj_tile<DIR, true, COMPACT>(a, G, S, c, src, lds, h, dsum, asum);
            else
                adj_tile<DIR, false, COMPACT>(a, G, S, c, src, lds, h, dsum, asum);
        });
        dsum = wave_sum(dsum);
        asum = wave_sum(asum);
        if (c.lane == 0) {
            part_add(a.part + (long long)src * a.nslots + TI * G.nt[1] + TJ, DIR, dsum);
            if (DIR == 7) a.part2[(long long)src * a.nslots + TI * G.nt[1] + TJ] = asum;
        }
    });
}

// Transposed boundary pass: lambda_b = rhs_b - sum_{rows r != b} J_{r, b} lambda_r,
// rhs_b read from the compact per-boundary-node copy (bnd_rhs).
// The rows that reference a boundary node b are its interior neighbour (face
// nodes only, coefficient bnd_in[b]) and boundary rows b' that copy b along an
// axis a' above a*(b) (b' one step outward along a', coefficient -1);
// lambda(b') is evaluated in place (a* grows strictly: depth <= 3).
template <int BUDGET>
__device__ double adj_bval(const Geo& G, const Src& S, const double* lam, const double* brhs, const double* bin,
                           int i, int j, int k) {
    const int p[3] = {i, j, k};
    const int as = astar_of(G, p);
    double acc = brhs[bnd_encode(G, i, j, k)];
    const int nb = (int)on_bnd(G, 0, i) + (int)on_bnd(G, 1, j) + (int)on_bnd(G, 2, k);
    if (nb == 1) {
        int x[3] = {i, j, k};
        x[as] += (p[as] == 0) ? 1 : -1;
        acc -= bin[bnd_encode(G, i, j, k)] * lam[nidx(G, x[0], x[1], x[2])];
    }
    if constexpr (BUDGET > 0) {
        for (int ap = as + 1; ap < 3; ++ap) {
            const int id = p[ap];
            if (on_bnd(G, ap, id)) continue;
            for (int side = 0; side < 2; ++side) {
                const int dist = side == 0 ? id : (G.n[ap] - 1 - id);
                if (dist != 1) continue;
                int q[3] = {i, j, k};
                q[ap] = side == 0 ? 0 : G.n[ap] - 1;
                if (in_fixed(S, q[0], q[1], q[2])) continue;
                acc += adj_bval<BUDGET - 1>(G, S, lam, brhs, bin, q[0], q[1], q[2]);
            }
        }
    }
    return acc;
}

__global__ void __launch_bounds__(kBndThreads) k_adj_bnd(SweepArgs a, int dir) {
    __shared__ double sh[4];
    const int src = blockIdx.y;
    if (blockIdx.x == 0) queue_reset(a, src);
    if (!a.active[src]) return;
    const Geo& G = a.G;
    const Src S = a.src[src];
    double* lam = a.field + (long long)src * G.N;
    const double* brhs = a.bnd_rhs + (long long)src * G.NB;
    const double* bin = a.bnd_in + (long long)src * G.NB;
    const long long b = (long long)blockIdx.x * kBndThreads + threadIdx.x;
    double d = 0.0, av = 0.0;
    if (b < G.NB) {
        int i, j, k;
        bnd_decode(G, b, i, j, k);
        if (!in_fixed(S, i, j, k) && !kface_only(G, i, j)) {  // (the sweeps set the nodes on a k face only)
            const double nv = adj_bval<2>(G, S, lam, brhs, bin, i, j, k);
            const long long x = nidx(G, i, j, k);
            d = fabs(nv - lam[x]);
            av = fabs(nv);
            lam[x] = nv;
        }
    }
    d = block_sum256(d, sh);
    const double as = (dir == 7) ? block_sum256(av, sh) : 0.0;
    if (threadIdx.x == 0) {
        part_add(a.part + (long long)src * a.nslots + G.ncols + blockIdx.x, dir, d);
        if (dir == 7) a.part2[(long long)src * a.nslots + G.ncols + blockIdx.x] = as;
    }
}

__global__ void __launch_bounds__(256) k_adj_finalize(SweepArgs a) {
    __shared__ double sh[4];
    const int src = blockIdx.x;
    if (!a.active[src]) return;
    const double dtot = fixed_sum(a.part + (long long)src * a.nslots, a.G.ncols + a.nbblocks, sh);
    const double atot = fixed_sum(a.part2 + (long long)src * a.nslots, a.G.ncols + a.nbblocks, sh);
    if (threadIdx.x == 0) finish_iteration(a, src, dtot / (atot > 1e-300 ? atot : 1e-300));
}

// ------------------------------------------ continuous adjoint (Eq. (5))
// Upwind finite volumes for div(P w) = sum_m R_m delta(x - x_m), w = -M grad T.
// Each node owns the trapezoidal control volume around it; the flux leaves
// through six faces with the face velocity the mean of the two nodal normal
// components (the node's own on a grid face) and carries the upwind node's P.
// P = 0 on the fixed cell (the source absorbs) and outside the grid.

// w = -M p at any node, p the scaled gradient of T = T0 tau: central
// differences of tau along axes where the node is interior, one-sided where
// it lies on the grid face.
template <int COORD>
__device__ __forceinline__ void cadj_vel(const Geo& G, const Tabs& T, const Src& S, const double* __restrict__ tau,
                                         const double* __restrict__ xi, const double* __restrict__ eta, int i, int j,
                                         int k, double w[3]) {
    const Col c = make_col(G, T, i, j);
    const double2 t2 = T.t2[k];
    double T0, t[3];
    factor<COORD>(S, c, t2.x, t2.y, T0, t);
    const long long x = nidx(G, i, j, k);
    const int id[3] = {i, j, k};
    const long long st[3] = {G.si, G.sj, 1};
    const double tx = tau[x];
    double p[3];
#pragma unroll
    for (int a2 = 0; a2 < 3; ++a2) {
        double q;
        if (id[a2] == 0) q = (tau[x + st[a2]] - tx) * G.invh[a2];
        else if (id[a2] == G.n[a2] - 1) q = (tx - tau[x - st[a2]]) * G.invh[a2];
        else q = (tau[x + st[a2]] - tau[x - st[a2]]) * G.inv2h[a2];
        p[a2] = T0 * g_of(c, a2) * q + tx * t[a2];
    }
    const double xv = xi[x], ev = eta[x];
    w[0] = -p[0];
    w[1] = -((1.0 - 2.0 * xv) * p[1] + 2.0 * ev * p[2]);
    w[2] = -(2.0 * ev * p[1] + (1.0 + 2.0 * xv) * p[2]);
}

// control-volume extent of node index idx along axis a
__device__ __forceinline__ double cv_ext(const Geo& G, int a, int idx) {
    return (idx == 0 || idx == G.n[a] - 1) ? 0.5 * G.h[a] : G.h[a];
}

// Area of the face of node (i, j, k) normal to axis a at coordinate xf of that
// axis: r^2 cos(theta) dtheta dphi (r faces), r cos(theta) dr dphi (theta
// faces), r dr dtheta (phi faces); products of the other extents in Cartesian
// coordinates.
__device__ __forceinline__ double cadj_area(const Geo& G, int a, int i, int j, int k, double xf) {
    const int id[3] = {i, j, k};
    double A = 1.0;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b != a) A *= cv_ext(G, b, id[b]);
    if (G.coord == 1) {
        const double r = G.o[0] + i * G.h[0];
        if (a == 0) A *= xf * xf * cos(G.o[1] + j * G.h[1]);
        else if (a == 1) A *= r * cos(xf);
        else A *= r;
    }
    return A;
}

// Records of the continuous system in the adjoint layout (the row divided by
// its diagonal, store_record): c+-_a = A min(u_out, 0) couples P(x +- e_a)
// (0 when that node is fixed or outside), and the diagonal is the outflow
// sum A max(u_out, 0).  A node without outflow gets outflow = inf, so that its
// update is P = 0.
template <int COORD>
__global__ void __launch_bounds__(256) k_cadj_coef(SweepArgs a, const double* __restrict__ tau_all,
                                                   double* __restrict__ coef_all, double* __restrict__ diag_all,
                                                   double* __restrict__ rhs_all) {
    const Geo& G = a.G;
    const int src = blockIdx.y;
    const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= G.N) return;
    const Src S = a.src[src];
    const double* tau = tau_all + (long long)src * G.N;
    const int k = (int)(x % G.n[2]);
    const long long q = x / G.n[2];
    const int j = (int)(q % G.n[1]), i = (int)(q / G.n[1]);
    double out[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (!in_fixed(S, i, j, k)) {
        double w[3];
        cadj_vel<COORD>(G, a.T, S, tau, a.xi, a.eta, i, j, k, w);
        const int id[3] = {i, j, k};
        double diag = 0.0;
        for (int ax = 0; ax < 3; ++ax) {
            const double xa = G.o[ax] + id[ax] * G.h[ax];
            for (int side = 0; side < 2; ++side) {
                const int sg = side == 0 ? 1 : -1;
                const int nb = id[ax] + sg;
                int y[3] = {i, j, k};
                y[ax] = nb;
                double u, A;
                const bool inside = nb >= 0 && nb < G.n[ax];
                if (inside) {
                    double wy[3];
                    cadj_vel<COORD>(G, a.T, S, tau, a.xi, a.eta, y[0], y[1], y[2], wy);
                    u = sg * 0.5 * (w[ax] + wy[ax]);
                    A = cadj_area(G, ax, i, j, k, 0.5 * (xa + (G.o[ax] + nb * G.h[ax])));
                } else {
                    u = sg * w[ax];
                    A = cadj_area(G, ax, i, j, k, xa);
                }
                diag += A * (u > 0.0 ? u : 0.0);
                out[2 * ax + side] = (inside && !in_fixed(S, y[0], y[1], y[2])) ? A * (u < 0.0 ? u : 0.0) : 0.0;
            }
        }
        out[6] = diag > 0.0 ? diag : HUGE_VAL;
    }
    store_record(G, coef_all, diag_all, rhs_all, src, x, i, j, k, out, a.compact);
}

// The boundary nodes' records, in planes by boundary node, for the boundary pass:
// read in the sweeps' layout a node of a k face takes lines of its own for its
// record every time (128 sources of 61^3 162 us a pass beside another group's
// sweep, now 82).  Gathered once a solve, over the diagonals, which nothing reads
// after the right-hand side.
__global__ void __launch_bounds__(kBndThreads) k_cadj_bnd_records(SweepArgs a, double2* __restrict__ rec_all) {
    const Geo& G = a.G;
    const int src = blockIdx.y;
    const long long b = (long long)blockIdx.x * kBndThreads + threadIdx.x;
    if (b >= G.NB) return;
    int i, j, k;
    bnd_decode(G, b, i, j, k);
    const double2* rc = reinterpret_cast<const double2*>(
        a.coef + (a.compact ? (long long)src * G.N + nidx(G, i, j, k) : (long long)src * 4 * G.Sa + arec_idx(G, 0, i, j, k)) * kRec);
#pragma unroll
    for (int q = 0; q < 3; ++q) rec_all[(long long)src * 3 * G.NB + q * G.NB + b] = rc[q];
}

// Boundary pass of the continuous system, Jacobi: every boundary node's new P
// from the values present before the pass, into tmp [nsrc][NB].  The right-hand
// side is read inside the box where it is not zero.
__global__ void __launch_bounds__(kBndThreads) k_cadj_bnd_calc(SweepArgs a, const double2* __restrict__ rec_all,
                                                               double* __restrict__ tmp_all) {
    const int src = blockIdx.y;
    if (blockIdx.x == 0) queue_reset(a, src);
    if (!a.active[src]) return;
    const Geo& G = a.G;
    const long long b = (long long)blockIdx.x * kBndThreads + threadIdx.x;
    if (b >= G.NB) return;
    const Src S = a.src[src];
    const double* P = a.field + (long long)src * G.N;
    const double2* rc = rec_all + (long long)src * 3 * G.NB + b;
    const int* bx = a.box + src * 6;
    int i, j, k;
    bnd_decode(G, b, i, j, k);
    double nv = 0.0;
    if (!in_fixed(S, i, j, k)) {
        const long long x = nidx(G, i, j, k);
        const int id[3] = {i, j, k};
        const long long st[3] = {G.si, G.sj, 1};
        const bool in = i >= bx[0] && i <= bx[1] && j >= bx[2] && j <= bx[3] && k >= bx[4] && k <= bx[5];
        double acc = in ? a.rhs[(long long)src * G.N + x] : 0.0;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const double2 r = rc[ax * G.NB];  // the row divided by its diagonal
            if (r.x != 0.0 && id[ax] + 1 < G.n[ax]) acc -= r.x * P[x + st[ax]];
            if (r.y != 0.0 && id[ax] > 0) acc -= r.y * P[x - st[ax]];
        }
        nv = acc;
    }
    tmp_all[(long long)src * G.NB + b] = nv;
}

// ... then written back, with the convergence sums in the boundary slots.
__global__ void __launch_bounds__(kBndThreads) k_cadj_bnd_store(SweepArgs a, const double* __restrict__ tmp_all,
                                                                int dir) {
    __shared__ double sh[4];
    const int src = blockIdx.y;
    if (!a.active[src]) return;
    const Geo& G = a.G;
    double* P = a.field + (long long)src * G.N;
    const long long b = (long long)blockIdx.x * kBndThreads + threadIdx.x;
    double d = 0.0, av = 0.0;
    if (b < G.NB) {
        int i, j, k;
        bnd_decode(G, b, i, j, k);
        const long long x = nidx(G, i, j, k);
        const double nv = tmp_all[(long long)src * G.NB + b];
        d = fabs(nv - P[x]);
        av = fabs(nv);
        P[x] = nv;
    }
    d = block_sum256(d, sh);
    const double as = (dir == 7) ? block_sum256(av, sh) : 0.0;
    if (threadIdx.x == 0) {
        part_add(a.part + (long long)src * a.nslots + G.ncols + blockIdx.x, dir, d);
        if (dir == 7) a.part2[(long long)src * a.nslots + G.ncols + blockIdx.x] = as;
    }
}

// The continuous adjoint's P as the derivative it estimates: d chi / d s(x) =
// P s V (Eqs. (6), (9)), V the trapezoidal node volume.
__global__ void __launch_bounds__(256) k_cadj_scale(Geo G, const double* __restrict__ s, double* __restrict__ lam_all,
                                                    int nsrc) {
    const int src = blockIdx.y;
    double* lam = lam_all + (long long)src * G.N;
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < G.N;
         x += (long long)gridDim.x * blockDim.x) {
        const int k = (int)(x % G.n[2]);
        const long long q = x / G.n[2];
        const int j = (int)(q % G.n[1]), i = (int)(q / G.n[1]);
        lam[x] *= s[x] * node_volume(G, i, j, k);
    }
    (void)nsrc;
}

// --------------------------------------------------------- sampling etc.
template <int COORD>
__global__ void k_sample(Geo G, Tabs T, const Src* __restrict__ srcs, int nsrc, const double* __restrict__ tau_all,
                         int nrec, const double* __restrict__ rec, double* __restrict__ out) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long long)nsrc * nrec) return;
    const int src = (int)(q / nrec), m = (int)(q % nrec);
    const Src S = srcs[src];
    const double* tau = tau_all + (long long)src * G.N;
    const Tri t = tri_of(G, rec[3 * m], rec[3 * m + 1], rec[3 * m + 2]);
    double acc = 0.0;
    for (int c0 = 0; c0 < 2; ++c0)
        for (int c1 = 0; c1 < 2; ++c1)
            for (int c2 = 0; c2 < 2; ++c2) {
                const int i = t.b[0] + c0, j = t.b[1] + c1, k = t.b[2] + c2;
                const Col c = make_col(G, T, i, j);
                const double2 t2 = T.t2[k];
                double T0, tt[3];
                factor<COORD>(S, c, t2.x, t2.y, T0, tt);
                acc += tri_w(t, c0, c1, c2) * T0 * tau[nidx(G, i, j, k)];
            }
    out[q] = acc;
}

// Kernels of Eqs. (6)-(8), summed over the sources in order.  A thread takes
// NI nodes in a row along axis 0, lanes run along (j, k): of a node's seven tau
// values axis 0's are shared with the next node and axis 2's come from the lanes
// beside it.  Consecutive workgroups go to different XCDs, so each XCD takes a
// contiguous run of blocks, planes fastest, whose neighbours are then its own.
// Bound by its L1 accesses where it fills the chip: two nodes a thread, six reads a node,
// take 718 us for 128 sources of 101^3, one node (eight reads) 792, four (five reads, but
// half the waves) 807; in the order of the nodes, one a thread, 1055.  A small grid is
// bound by each thread's walk over the sources, and one node a thread is the shortest
// (us, one / two / four): 16^3 x 128 99 / 150 / 234, 41^3 x 128 107 / 130 / 198, 55^3 x 128 169 / 199 /
// 233, 61^3 x 128 212 / 210 / 240, 61^3 x 200 311 / 300 / 351.
constexpr long long kAccFew = 200000;

__device__ __forceinline__ double lane_below(double v) {  // lane 0: its own value
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ double lane_above(double v) {  // lane 63: its own value
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x130, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(lo, lo, 0x130, 0xf, 0xf, false));
}

template <int COORD, int NI>
__global__ void __launch_bounds__(256) k_kernel_accum(Geo G, Tabs T, const Src* __restrict__ srcs, int nsrc,
                                                      const double* __restrict__ xi, const double* __restrict__ eta,
                                                      const double* __restrict__ tau_all,
                                                      const double* __restrict__ lam_all, double* __restrict__ grad,
                                                      int accumulate) {
    const int nib = (G.n[0] + NI - 1) / NI;
    const long long blk = (long long)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int i0 = NI * (int)(blk % nib);
    const long long e = blk / nib * 256 + threadIdx.x, plane = G.si;
    if (blk / nib * 256 >= plane) return;
    const long long jk = e < plane ? e : plane - 1;  // (lanes past the plane keep the last one company)
    const int j = (int)(jk / G.n[2]), k = (int)(jk % G.n[2]);
    const bool in = e < plane && j > 0 && j < G.n[1] - 1 && k > 0 && k < G.n[2] - 1;
    const int lane = threadIdx.x & 63;
    const bool end = lane == 0 || lane == 63;
    // (lanes at the fields' faces read inside them; their sums are dropped)
    const long long jm = j > 0 ? -G.sj : 0, jp = j < G.n[1] - 1 ? G.sj : 0;
    const long long ke = lane == 0 ? (jk > 0 ? -1 : 0) : (jk < plane - 1 ? 1 : 0);
    double gs[NI] = {}, gx[NI] = {}, ge[NI] = {};
    if (nsrc > 0) {  // (no tables without a source)
        Col c[NI];
        double ma[NI], mb[NI], mc[NI];
        long long xo[NI + 2];
#pragma unroll
        for (int u = 0; u < NI + 2; ++u) xo[u] = min(max(i0 + u - 1, 0), G.n[0] - 1) * G.si + jk;
#pragma unroll
        for (int u = 0; u < NI; ++u) {
            c[u] = make_col(G, T, min(i0 + u, G.n[0] - 1), j);
            ma[u] = 1.0 - 2.0 * xi[xo[u + 1]];
            mb[u] = 2.0 * eta[xo[u + 1]];
            mc[u] = 1.0 + 2.0 * xi[xo[u + 1]];
        }
        const double2 t2 = T.t2[k];
        for (int n = 0; n < nsrc; ++n) {
            const Src S = srcs[n];
            const double* tau = tau_all + (long long)n * G.N;
            const double* lam = lam_all + (long long)n * G.N;
            double v[NI + 2], l[NI], vm[NI], vp[NI], vk[NI];
#pragma unroll
            for (int u = 0; u < NI + 2; ++u) v[u] = tau[xo[u]];
#pragma unroll
            for (int u = 0; u < NI; ++u) {
                vm[u] = tau[xo[u + 1] + jm];
                vp[u] = tau[xo[u + 1] + jp];
                l[u] = lam[xo[u + 1]];
            }
#pragma unroll
            for (int u = 0; u < NI; ++u) vk[u] = 0.0;
            if (end)
#pragma unroll
                for (int u = 0; u < NI; ++u) vk[u] = tau[xo[u + 1] + ke];
#pragma unroll
            for (int u = 0; u < NI; ++u) {
                const double tx = v[u + 1];
                const double km = lane_below(tx), kp = lane_above(tx);
                double T0, t[3];
                factor<COORD>(S, c[u], t2.x, t2.y, T0, t);
                const double d2 = (lane == 63 ? vk[u] : kp) - (lane == 0 ? vk[u] : km);
                const double p0 = T0 * ((v[u + 2] - v[u]) * G.inv2h[0]) + tx * t[0];
                const double p1 = T0 * (c[u].g1 * (vp[u] - vm[u]) * G.inv2h[1]) + tx * t[1];
                const double p2 = T0 * (c[u].g2 * d2 * G.inv2h[2]) + tx * t[2];
                const double h2 = p0 * p0 + p1 * (ma[u] * p1 + mb[u] * p2) + p2 * (mb[u] * p1 + mc[u] * p2);
                const double lh = l[u] * rsqrt_3(h2);  // lambda / H
                if (!in_fixed(S, i0 + u, j, k)) {
                    gs[u] += l[u];
                    gx[u] += lh * (p1 * p1 - p2 * p2);
                    ge[u] += -2.0 * lh * p1 * p2;
                }
            }
        }
    }
    if (e >= plane) return;
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        const int i = i0 + u;
        if (i >= G.n[0]) return;
        const bool on = in && i > 0 && i < G.n[0] - 1;
        const long long x = i * G.si + e;
        const double a = on ? gs[u] : 0.0, b = on ? gx[u] : 0.0, d = on ? ge[u] : 0.0;
        if (accumulate) {
            grad[x] += a; grad[G.N + x] += b; grad[2 * G.N + x] += d;
        } else {
            grad[x] = a; grad[G.N + x] = b; grad[2 * G.N + x] = d;
        }
    }
}

// ---------------------------------------------------------------- launchers

SweepArgs make_args(const Plan& P, const double* s, const double* xi, const double* eta, double* field,
                    int32_t* status) {
    SweepArgs a;
    a.G = P.G;
    a.T = P.T;
    a.s = s; a.xi = xi; a.eta = eta;
    a.src = P.src;
    a.lon = P.lon;
    a.field = field;
    a.coef = P.coef;
    a.rhs = P.rhs;
    a.box = P.box;
    a.model = P.model;
    a.bnd_in = P.bnd_in;
    a.bnd_rhs = P.bnd_rhs;
    a.active = P.active;
    a.iter = P.iter;
    a.status = status;
    a.part = P.part;
    a.part2 = P.part2;
    a.counter = P.counter;
    a.eps_hist = P.eps_hist;
    a.nslots = P.nslots;
    a.nbblocks = P.nbblocks;
    a.nsrc = P.nsrc;
    a.compact = P.compact ? 1 : 0;
    a.kfaces = P.continuous ? 0 : 1;
    a.max_iter = P.max_iter;
    a.hist_stride = P.hist_stride;
    a.kappa = P.kappa;
    a.tol = P.tol;
    return a;
}

void launch_tables(const Plan& P, hipStream_t st) {
    int n = P.G.n[0];
    if (P.G.n[1] > n) n = P.G.n[1];
    if (P.G.n[2] > n) n = P.G.n[2];
    hipLaunchKernelGGL(k_tables, dim3(blocks_for(n, 64)), dim3(64), 0, st, P.G, P.tab0, P.tab1, P.tab2);
}

void launch_src_setup(const Plan& P, const double* pos, const double* par, hipStream_t st) {
    hipLaunchKernelGGL(k_src_setup, dim3(blocks_for(P.nsrc, 64)), dim3(64), 0, st, P.G, pos, par, P.src, P.nsrc);
}

void launch_source_params(const Geo& G, const double* s, const double* xi, const double* eta, const double* pos,
                          double* par, int nsrc, hipStream_t st) {
    hipLaunchKernelGGL(k_source_params, dim3(blocks_for(nsrc, 64)), dim3(64), 0, st, G, s, xi, eta, pos, par, nsrc);
}


void launch_fwd_init(const Plan& P, const SweepArgs& a, const double* tau_init, const double* s, const double* xi,
                     const double* eta, hipStream_t st) {
    const long long nl = (long long)P.nsrc * P.G.n[2];
    hipLaunchKernelGGL(k_lon, dim3(blocks_for(nl, 256)), dim3(256), 0, st, P.G, P.tab2, P.src, P.lon, nl);
    hipLaunchKernelGGL(k_model_records, dim3(blocks_for(P.G.N, 256)), dim3(256), 0, st, P.G, s, xi, eta, P.model);
    hipLaunchKernelGGL(k_solve_init, dim3(fill_blocks(P.G.N), P.nsrc), dim3(256), 0, st, a, tau_init, 1.0, 1.0);
}

static size_t tile_lds_bytes(const Geo& G) { return (size_t)(G.Nf != G.N ? kLinesLds : stage_bytes(G.tk)); }

// Workgroups (one wave each) of a sweep launch over cn sources: as many as the
// chip's LDS holds, but no more than there are tile columns on each XCD.
static unsigned march_blocks(const Plan& P, int cn) {
    const long long fit = 256LL * std::min<long long>(16, 163840 / (long long)tile_lds_bytes(P.G));
    const int nb = std::min(kMarchBatches, cn);
    const long long want = (long long)kMarchBatches * ((cn + nb - 1) / nb) * P.G.ncols;
    return (unsigned)std::min(fit, want);
}

static int march_launches(const Plan& P) { return (P.nsrc + kMarchSources - 1) / kMarchSources; }

// Event pair around the launches of one directional sweep when
// timing is on; the launch count of the group is recorded with it.
struct TimedLaunch {
    const Plan& P;
    hipStream_t st;
    hipEvent_t e1 = nullptr;
    TimedLaunch(const Plan& p, hipStream_t s, int launches) : P(p), st(s) {
        if (P.timing) {
            hipEvent_t e0;
            if (hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess) {
                (void)hipEventRecord(e0, st);
                P.timing->push_back({{e0, e1}, launches});
            } else {
                e1 = nullptr;
            }
        }
    }
    ~TimedLaunch() {
        if (P.timing && e1) (void)hipEventRecord(e1, st);
    }
};

// Sweep kernels are instantiated per coordinate system and direction.
typedef void (*SweepFn)(SweepArgs, int, int);

template <int COORD, int TKC, int... DS>
constexpr SweepFn pick_fwd(int d, std::integer_sequence<int, DS...>) {
    SweepFn t[] = {k_fwd_sweep<COORD, DS, TKC>...};
    return t[d];
}

template <int COORD, bool COMPACT, int TKC, int... DS>
constexpr SweepFn pick_adj(int d, std::integer_sequence<int, DS...>) {
    SweepFn t[] = {k_adj_sweep<COORD, DS, COMPACT, TKC>...};
    return t[d];
}

template <int COORD, int... DS>
constexpr SweepFn pick_lines(int d, std::integer_sequence<int, DS...>) {
    SweepFn t[] = {k_fwd_lines<COORD, DS>...};
    return t[d];
}

// forward sweep instances with a compile-time tile depth (16: windows held across
// slabs); other depths run the generic one
template <int COORD>
SweepFn fwd_sweep_fn_c(int tk, int d) {
    const auto seq = std::make_integer_sequence<int, 8>{};
    switch (tk) {
        case 16: return pick_fwd<COORD, 16>(d, seq);
        case 20: return pick_fwd<COORD, 20>(d, seq);
        case 24: return pick_fwd<COORD, 24>(d, seq);
        case 28: return pick_fwd<COORD, 28>(d, seq);
        default: return pick_fwd<COORD, 0>(d, seq);
    }
}

SweepFn fwd_sweep_fn(const Plan& P, int d) {
    const auto seq = std::make_integer_sequence<int, 8>{};
    const Geo& G = P.G;
    if (G.Nf != G.N) return G.coord == 1 ? pick_lines<1>(d, seq) : pick_lines<0>(d, seq);
    return G.coord == 1 ? fwd_sweep_fn_c<1>(G.tk, d) : fwd_sweep_fn_c<0>(G.tk, d);
}

// adjoint instances with a compile-time tile depth for the full record
// layouts (the autotuner's usual choices); compact records and other depths
// run the generic instance
template <int COORD>
SweepFn adj_sweep_fn_c(int tk, int d, bool compact) {
    const auto seq = std::make_integer_sequence<int, 8>{};
    if (compact) return pick_adj<COORD, true, 0>(d, seq);
    switch (tk) {
        case 16: return pick_adj<COORD, false, 16>(d, seq);
        case 28: return pick_adj<COORD, false, 28>(d, seq);
        case 32: return pick_adj<COORD, false, 32>(d, seq);
        case 40: return pick_adj<COORD, false, 40>(d, seq);
        case 48: return pick_adj<COORD, false, 48>(d, seq);
        default: return pick_adj<COORD, false, 0>(d, seq);
    }
}

SweepFn adj_sweep_fn(int coord, int tk, int d, bool compact) {
    return coord == 1 ? adj_sweep_fn_c<1>(tk, d, compact) : adj_sweep_fn_c<0>(tk, d, compact);
}

void launch_fwd_iteration(const Plan& P, const SweepArgs& a, hipStream_t st) {
    for (int d = 0; d < 8; ++d) {
        {
        TimedLaunch tl(P, st, march_launches(P));
        const SweepFn fn = fwd_sweep_fn(P, d);
        for (int c0 = 0; c0 < P.nsrc; c0 += kMarchSources) {
            const int cn = std::min(kMarchSources, P.nsrc - c0);
            hipLaunchKernelGGL(fn, dim3(march_blocks(P, cn)), dim3(64), tile_lds_bytes(P.G), st, a, c0, cn);
        }
        }
        hipLaunchKernelGGL(k_fwd_bnd, dim3(P.nbblocks, P.nsrc), dim3(kBndThreads), 0, st, a, d);
    }
    hipLaunchKernelGGL(k_fwd_finalize, dim3(P.nsrc), dim3(256), 0, st, a);
}

void launch_unpad(const Plan& P, double* tau, hipStream_t st) {
    hipLaunchKernelGGL(k_unpad, dim3(blocks_for(P.G.N, 256), P.nsrc), dim3(256), 0, st, P.G, P.pad, tau);
}

void launch_adj_init(const Plan& P, const SweepArgs& a, const double* tau, int nrec, const double* rec,
                     const double* R, const double* init, hipStream_t st) {
    hipLaunchKernelGGL(k_fill, dim3(fill_blocks(2 * P.G.NB * P.nsrc)), dim3(256), 0, st, P.bnd_in,
                       2 * P.G.NB * P.nsrc, 0.0);  // bnd_in and bnd_rhs
    const dim3 grid(blocks_for(P.G.N, 256), P.nsrc);
    const dim3 rgrid(P.nsrc);
    const int t0 = P.continuous ? 0 : 1;
    if (P.G.coord == 1) {
        if (P.continuous) hipLaunchKernelGGL(k_cadj_coef<1>, grid, dim3(256), 0, st, a, tau, P.coef, P.diag, P.rhs);
        else hipLaunchKernelGGL(k_adj_coef<1>, grid, dim3(256), 0, st, a, tau, P.coef, P.bnd_in, P.diag, P.rhs);
        hipLaunchKernelGGL(k_adj_rhs<1>, rgrid, dim3(64), 0, st, a, P.diag, P.rhs, P.box, nrec, rec, R, t0);
    } else {
        if (P.continuous) hipLaunchKernelGGL(k_cadj_coef<0>, grid, dim3(256), 0, st, a, tau, P.coef, P.diag, P.rhs);
        else hipLaunchKernelGGL(k_adj_coef<0>, grid, dim3(256), 0, st, a, tau, P.coef, P.bnd_in, P.diag, P.rhs);
        hipLaunchKernelGGL(k_adj_rhs<0>, rgrid, dim3(64), 0, st, a, P.diag, P.rhs, P.box, nrec, rec, R, t0);
    }
    if (P.continuous)
        hipLaunchKernelGGL(k_cadj_bnd_records, dim3(P.nbblocks, P.nsrc), dim3(kBndThreads), 0, st, a, P.bnd_rec);
    hipLaunchKernelGGL(k_solve_init, dim3(fill_blocks(P.G.N), P.nsrc), dim3(256), 0, st, a, init, 0.0, 0.0);
}

void launch_adj_iteration(const Plan& P, const SweepArgs& a, hipStream_t st) {
    for (int d = 0; d < 8; ++d) {
        {
        TimedLaunch tl(P, st, march_launches(P));
        const SweepFn fn = adj_sweep_fn(P.G.coord, P.G.tk, d, P.compact);
        for (int c0 = 0; c0 < P.nsrc; c0 += kMarchSources) {
            const int cn = std::min(kMarchSources, P.nsrc - c0);
            hipLaunchKernelGGL(fn, dim3(march_blocks(P, cn)), dim3(64), tile_lds_bytes(P.G), st, a, c0, cn);
        }
        }
        if (P.continuous) {
            hipLaunchKernelGGL(k_cadj_bnd_calc, dim3(P.nbblocks, P.nsrc), dim3(kBndThreads), 0, st, a, P.bnd_rec, P.bnd_in);
            hipLaunchKernelGGL(k_cadj_bnd_store, dim3(P.nbblocks, P.nsrc), dim3(kBndThreads), 0, st, a, P.bnd_in, d);
        } else {
            hipLaunchKernelGGL(k_adj_bnd, dim3(P.nbblocks, P.nsrc), dim3(kBndThreads), 0, st, a, d);
        }
    }
    hipLaunchKernelGGL(k_adj_finalize, dim3(P.nsrc), dim3(256), 0, st, a);
}

void launch_cadj_scale(const Plan& P, const double* s, double* lam, hipStream_t st) {
    hipLaunchKernelGGL(k_cadj_scale, dim3(fill_blocks(P.G.N), P.nsrc), dim3(256), 0, st, P.G, s, lam, P.nsrc);
}

void launch_fill(double* p, long long n, double v, hipStream_t st) {
    if (n > 0) hipLaunchKernelGGL(k_fill, dim3(fill_blocks(n)), dim3(256), 0, st, p, n, v);
}

void launch_sample(const Plan& P, const double* tau, int nrec, const double* rec, double* out, hipStream_t st) {
    const long long tot = (long long)P.nsrc * nrec;
    if (tot == 0) return;
    if (P.G.coord == 1)
        hipLaunchKernelGGL(k_sample<1>, dim3(blocks_for(tot, 256)), dim3(256), 0, st, P.G, P.T, P.src, P.nsrc, tau,
                           nrec, rec, out);
    else
        hipLaunchKernelGGL(k_sample<0>, dim3(blocks_for(tot, 256)), dim3(256), 0, st, P.G, P.T, P.src, P.nsrc, tau,
                           nrec, rec, out);
}

template <int NI>
static void accum(const Plan& P, const double* xi, const double* eta, const double* tau, const double* lam, double* grad,
                  int accumulate, hipStream_t st) {
    const long long blocks = (long long)blocks_for(P.G.si, 256) * ((P.G.n[0] + NI - 1) / NI);
    const dim3 grid((unsigned)((blocks + 7) / 8 * 8));
    if (P.G.coord == 1)
        hipLaunchKernelGGL((k_kernel_accum<1, NI>), grid, dim3(256), 0, st, P.G, P.T, P.src, P.nsrc, xi, eta, tau, lam,
                           grad, accumulate);
    else
        hipLaunchKernelGGL((k_kernel_accum<0, NI>), grid, dim3(256), 0, st, P.G, P.T, P.src, P.nsrc, xi, eta, tau, lam,
                           grad, accumulate);
}

void launch_kernel_accum(const Plan& P, const double* xi, const double* eta, const double* tau, const double* lam,
                         double* grad, int accumulate, hipStream_t st) {
    if (P.G.N < kAccFew)
        accum<1>(P, xi, eta, tau, lam, grad, accumulate, st);
    else
        accum<2>(P, xi, eta, tau, lam, grad, accumulate, st);
}

}  // namespace tt
