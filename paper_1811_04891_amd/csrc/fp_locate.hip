// findpts: candidate lookup, (point, element) pair grouping, trust-region
// Newton per pair with one element per wavefront, owner selection.
//
// Section 2.1 of the paper: hash table -> elementwise bounding boxes ->
// trust-region Newton on ||x^e(r) - x*||^2 started from the closest mapped
// GLL node -> inside / border / not found; session-id exclusion; among
// several sessions the largest distance-to-boundary wins.
//
// Pipeline per pass of at most max_points points, all on the caller's stream:
//   k_cand     per point: hash cell, box + session test, candidate list
//              (ascending element ids) and each pair's rank in its element
//   scan       pair counts per element -> element offsets and work units
//   k_scatter  pair slots grouped by element
//   k_locate_mfma  (orders 1..7) one wavefront per work unit (a run of one
//              element's pairs), element block in LDS, map and Jacobian of 16
//              pairs at a time on the matrix cores (fp_mfma.inc)
//   k_newton_pl  (orders 8..15) blocks of wavefronts per work unit, the element
//              in LDS, matrix cores (fp_newton_pl.inc)
//   k_select   per point: classification and owner rule, caller's order
// Small calls take k_point instead, one wavefront per point (fp_point.inc).
#include <algorithm>
#include <cmath>

#include "fp_basis.h"
#include "fp_internal.h"
#include "fp_mfma.h"
#include "fp_wave.h"

namespace fp {

struct LocArgs {
    const double *geom;
    const double *esize;
    bool first;          // first pass: also test the oriented box
    const double *erec;  // per element, 16 doubles: axis-aligned box, oriented box
    int *redo;           // first pass writes 1 for tasks left without an inside
                         // candidate and with a partial candidate set, else 0
    const int *only;     // non-null (second pass): tasks with only[t] != 0
    int *gate;           // first pass: cleared by k_cand, set by k_select when any
                         // task is flagged; second pass: every kernel returns at
                         // once while it is zero
    const double *delta;
    const int *esess;
    const int *cell_off;
    const float4 *cell_box;  // per cell entry: binary32 outward box, element id
    Grid g;
    const double *pts;
    const int *psess;
    int npts;
    int M;  // candidate slots are candidate-major: slot(t, k) = k * M + t
    double tol;
    int *ncand;
    int *cand_el;
    int *cand_pos;
    int *elem_cnt;
    const int *elem_off;
    const UnitRec *units;  // work units of the pairs
    bool few;              // rank_few ranks the pairs
    int E;
    int *order;
    double *res;
    double *res_dl;
    int *res_in;
    unsigned *cand_part;  // per k_cand block: the method's candidates (first pass)
    unsigned *iter_part;  // per block: Newton iterations of its pairs
    int pair_max;         // second pass: up to this many pairs run on k_newton_pair
                          // (one wavefront per pair)
    unsigned *pt_part;    // small calls: counters of each block
};

__device__ __forceinline__ int cell_of(const Grid &g, int a, double x)
{
    double u = (x - g.lo[a]) * g.inv[a];
    int i = (int)floor(u);
    return i < 0 ? 0 : (i >= g.nc[a] ? g.nc[a] - 1 : i);
}

__device__ __forceinline__ bool task_on(const LocArgs &a, int t)
{
    return t < a.npts && (!a.only || a.only[t] != 0);
}

// res_in of a pair: 0 = solved, not inside; 1 = inside; kUnsolved = left by the
// mixed-precision first pass to the binary64 second pass
constexpr int kUnsolved = 2;
// res_in kOutside: the mixed-precision first pass found the point clearly
// outside the element (binary32 residual far above its rounding level on a
// face of [-1,1]^3): never inside; solved in binary64 only if the point has no
// inside candidate (its distance is then needed)
constexpr int kOutside = 3;

// ncand[t] = candidate count | (1 << kFullBit) when the list is the method's
// whole candidate set (no second pass needed for that point)
constexpr int kFullBit = 30;
constexpr int kCountMask = (1 << kFullBit) - 1;

// Entries q0 .. q0 + cnt - 1 (cnt <= 64) of a cell's list whose binary32 box
// holds the point, as a bit mask: four entries' boxes are loaded at a time and
// nothing branches on their tests, so that the loads of a point do not wait on
// each other and a wavefront runs the exact tests once per hit of its busiest
// lane, not once per entry (1.01e6 points on the annulus: k_cand 255 us one entry
// at a time, 199 us now; 2e7 points on the large box 3.14 -> 2.72 ms).
__device__ __forceinline__ unsigned long long cell_hits(const LocArgs &a, int q0, int cnt,
                                                        double x0, double x1, double x2)
{
    // rounding is monotonic: x in [lo, hi] implies (float)x in the
    // outward-rounded binary32 box
    const float f0 = (float)x0, f1 = (float)x1, f2 = (float)x2;
    const float4 *box = a.cell_box + 2 * (long long)q0;
    unsigned long long m = 0ull;
    for (int i = 0; i < cnt; i += 4) {
        float4 lo[4], hi[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int q = min(i + w, cnt - 1);
            lo[w] = box[2 * q];
            hi[w] = box[2 * q + 1];
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const bool in = (f0 >= lo[w].x) & (f0 <= hi[w].x) & (f1 >= lo[w].y) &
                            (f1 <= hi[w].y) & (f2 >= lo[w].z) & (f2 <= hi[w].z);
            if (in & (i + w < cnt)) m |= 1ull << (i + w);
        }
    }
    return m;
}

// Candidates of one point: hash cell, then the closed axis-aligned box and
// the session exclusion (the method's candidate set), then, in the first
// pass, the oriented box.  The oriented box holds the whole element, so it
// never drops an element that contains the point; points left without an
// inside candidate get, in the second pass, the candidates the first pass
// dropped, appended after its own (whose results stay; a pair the binary32
// phase left unsolved is solved again in its slot).  cand_pos = -1 marks a
// slot that keeps its first-pass result.
__global__ __launch_bounds__(256) void k_cand(LocArgs a)
{
    if (a.only && !*a.gate) return;  // second pass with nothing flagged
    if (a.first && blockIdx.x == 0 && threadIdx.x == 0) *a.gate = 0;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    int naabb = 0, n = 0, n1st = 0;
    int e0 = -1, e1 = -1;  // the first two slots' elements (not read back below)
    if (t < a.npts && a.only && !a.only[t]) {
        a.ncand[t] = 0;
    } else if (t < a.npts) {
        const int p = t;
        const double x0 = a.pts[3 * (long long)p], x1 = a.pts[3 * (long long)p + 1],
                     x2 = a.pts[3 * (long long)p + 2];
        const int ps = a.psess ? a.psess[p] : -1;
        int full = a.first ? 0 : 1;
        bool take = true;
        if (a.only) {  // second pass: the first pass's candidates stay in their slots
            n1st = a.ncand[t] & kCountMask;
            n = n1st;
            // a first-pass list that is already the whole set (taken without
            // the oriented-box filter, or left intact by it) gets nothing
            // appended: only its unsolved slots are solved again
            take = (a.ncand[t] >> kFullBit) == 0;
        }
        const Grid &g = a.g;
        // NaN fails every comparison, so non-finite points find nothing
        if (take && x0 >= g.lo[0] && x0 <= g.hi[0] && x1 >= g.lo[1] && x1 <= g.hi[1] &&
            x2 >= g.lo[2] && x2 <= g.hi[2]) {
            const long long c = cell_of(g, 0, x0) +
                                (long long)g.nc[0] * (cell_of(g, 1, x1) +
                                                      (long long)g.nc[1] * cell_of(g, 2, x2));
            const int qb = a.cell_off[c], qe = a.cell_off[c + 1];
            int *ce = a.cand_el + t;
            // pass 0: oriented-box filter (first pass only); pass 1: every
            // candidate, taken when the filter left none (the point then
            // has its full candidate set and needs no second pass)
            for (int pass = a.first ? 0 : 1; pass < 2 && (n == 0 || a.only); ++pass) {
                for (int q0 = qb; q0 < qe; q0 += 64) {
                    // the binary32 boxes first (outward-rounded: a superset),
                    // then the exact tests of the few that hold the point
                    unsigned long long todo = cell_hits(a, q0, min(qe - q0, 64), x0, x1, x2);
                    while (todo != 0ull) {
                        const int q = q0 + __ffsll((long long)todo) - 1;
                        todo &= todo - 1ull;
                        const int e = __float_as_int(a.cell_box[2 * (long long)q].w);
                        const double *b = a.erec + 16 * (long long)e;  // one line: both boxes
                        if (x0 < b[0] || x0 > b[1] || x1 < b[2] || x1 > b[3] || x2 < b[4] ||
                            x2 > b[5])
                            continue;
                        if (ps >= 0 && a.esess && a.esess[e] == ps) continue;
                        if (pass == 0 || a.only) {
                            ++naabb;
                            const float *o = (const float *)(b + 6);
                            const double d0 = x0 - (double)o[9], d1 = x1 - (double)o[10],
                                         d2 = x2 - (double)o[11];
                            bool in = true;
#pragma unroll
                            for (int ax = 0; ax < 3; ++ax) {
                                const double u = fma((double)o[3 * ax + 2], d2,
                                                     fma((double)o[3 * ax + 1], d1,
                                                         (double)o[3 * ax] * d0));
                                in = in && u >= (double)o[12 + ax] && u <= (double)o[15 + ax];
                            }
                            if (in == (a.only != nullptr)) continue;  // second pass: the dropped
                        }
                        ce[(long long)n * a.M] = e;
                        e0 = n == 0 ? e : e0;
                        e1 = n == 1 ? e : e1;
                        // a slot appended by the second pass is new: no state of
                        // an earlier call may read as a pair to resume
                        if (a.only) a.res_in[(long long)n * a.M + t] = 0;
                        ++n;
                    }
                }
                // the method's whole set: taken in pass 1, or left intact by
                // the oriented-box filter
                if (pass == 1 || naabb == 0 || n == naabb) full = 1;
                if (pass == 0 && naabb == 0) break;     // nothing to take
            }
        }
        a.ncand[t] = n | (full << kFullBit);
    }
    // each pair's rank in its element, from converged code so that lanes
    // sharing an element (a crowded element) share one atomic add
    int nmax = n;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nmax = max(nmax, __shfl_xor(nmax, o, kWave));
    for (int k = 0; k < nmax; ++k) {
        const long long s = (long long)k * a.M + t;
        // a first-pass slot is solved again only if it was left unsolved
        const bool act =
            k < n && (k >= n1st || a.res_in[s] == kUnsolved || a.res_in[s] == kOutside);
        int e = -1;
        if (act) e = (k == 0 && e0 >= 0) ? e0 : ((k == 1 && e1 >= 0) ? e1 : a.cand_el[s]);
        const int r = a.few ? 0 : wave_rank(a.elem_cnt, e, act);
        if (k < n) a.cand_pos[s] = act ? r : -1;
    }
    if (a.first) {  // the method's candidates of this block (first pass covers every point)
        __shared__ unsigned wsum[256 / kWave];
        unsigned v = (unsigned)naabb;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
        if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x / kWave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned b = 0;
            for (int i = 0; i < 256 / kWave; ++i) b += wsum[i];
            a.cand_part[blockIdx.x] = b;
        }
    }
}

__global__ __launch_bounds__(256) void k_scatter(LocArgs a)
{
    if (a.only && !*a.gate) return;
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    // the counts are in the offsets by now: cleared here for the second pass
    if (a.first)
        for (int e = p; e < a.E; e += gridDim.x * blockDim.x) a.elem_cnt[e] = 0;
    if (p >= a.npts) return;
    const int n = a.ncand[p] & kCountMask;  // 0 for tasks the pass skips
    for (int k = 0; k < n; ++k) {
        const long long s = (long long)k * a.M + p;
        const int r = a.cand_pos[s];
        if (r >= 0) a.order[a.elem_off[a.cand_el[s]] + r] = (int)s;
    }
}

// 1 / x from the hardware reciprocal and two Newton-Raphson refinements
// (within an ulp or two of the quotient, no scaling for denormals: the
// trust-region step it scales does not need a correctly rounded quotient).
__device__ __forceinline__ double rcp64(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

// Solve the 3x3 system A d = b by Cramer's rule; false if det is 0 or the
// result is not finite.
__device__ __forceinline__ bool solve3(const double (&A)[9], const double (&b)[3],
                                       double (&d)[3])
{
    const double c00 = A[4] * A[8] - A[5] * A[7];
    const double c01 = A[5] * A[6] - A[3] * A[8];
    const double c02 = A[3] * A[7] - A[4] * A[6];
    const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
    const double c10 = A[2] * A[7] - A[1] * A[8];
    const double c11 = A[0] * A[8] - A[2] * A[6];
    const double c12 = A[1] * A[6] - A[0] * A[7];
    const double c20 = A[1] * A[5] - A[2] * A[4];
    const double c21 = A[2] * A[3] - A[0] * A[5];
    const double c22 = A[0] * A[4] - A[1] * A[3];
    const double inv = rcp64(det);
    d[0] = (c00 * b[0] + c10 * b[1] + c20 * b[2]) * inv;
    d[1] = (c01 * b[0] + c11 * b[1] + c21 * b[2]) * inv;
    d[2] = (c02 * b[0] + c12 * b[1] + c22 * b[2]) * inv;
    return det != 0.0 && isfinite(d[0]) && isfinite(d[1]) && isfinite(d[2]);
}

// Trust-region Newton constants (stop tests, radius rules).
constexpr double kResidStop = 1e-13;  // residual stop: at most kResidStop h_e
constexpr double kStepStop = 1e-13;   // accepted step with |s|_inf below this
constexpr double kStepTiny = 1e-15;   // no progress possible
constexpr int kMaxIter = 50;

// Squared residual at which Newton stops: a tenth of the inside tolerance,
// at most kResidStop, relative to h_e (a point the tolerance accepts is never
// left short of it).
__device__ __forceinline__ double resid_stop(double tol, double he)
{
    const double c = fmin(0.1 * tol, kResidStop) * he;
    return c * c;
}

// Projected trust-region Gauss-Newton on phi(r) = ||x(r) - x*||^2 over
// [-1,1]^3.  A coordinate on a bound whose descent direction points outward
// is held; the step solves J d = -F when every coordinate is free, else the
// reduced normal equations on the free ones (steepest descent if singular);
// it is scaled to the trust radius (max norm) and projected on the cube.
// rho = actual / predicted decrease; accept if rho >= 0.01; radius doubled
// (up to 2) when rho > 0.75 and the radius limited the step, set to |s|/4
// when rho < 0.25.  Stop: phi <= (min(1e-13, tol/10) h_e)^2, an accepted
// step with |s| <= 1e-13 (quadratic convergence: the point it reaches is at
// the map's rounding level), no possible progress, or 50 iterations.
struct TRNewton {
    double r[3], F[3], J[9], phi, D, pred, ns;
    double rt[3];  // next trial point
    double step_stop = kStepStop;
    int max_it = kMaxIter;
    bool limited, have;
    int it;

    __device__ __forceinline__ void start(const double (&r0)[3])
    {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            rt[d] = r0[d];
            r[d] = 0.0;
            F[d] = 0.0;
        }
#pragma unroll
        for (int d = 0; d < 9; ++d) J[d] = 0.0;
        phi = INFINITY;
        D = 1.0;
        pred = 0.0;
        ns = 0.0;
        limited = false;
        have = false;
        it = 0;
    }

    // Consume the map and Jacobian evaluated at rt; returns true when done,
    // otherwise leaves the next trial point in rt.
    __device__ __forceinline__ bool update(const double (&xt)[3], const double (&Jt)[9],
                                           const double (&xs)[3], double rstop)
    {
        return accept(xt, Jt, xs, rstop) || step();
    }

    // The two halves of update.  accept: take or reject the trial point rt
    // (model ratio, radius) and test the stop rules; true when done.
    __device__ __forceinline__ bool accept(const double (&xt)[3], const double (&Jt)[9],
                                           const double (&xs)[3], double rstop)
    {
        const double Ft[3] = {xt[0] - xs[0], xt[1] - xs[1], xt[2] - xs[2]};
        const double phit = fma(Ft[2], Ft[2], fma(Ft[1], Ft[1], Ft[0] * Ft[0]));
        bool acc = true, stop = false;
        if (have) {
            // rho = (phi - phit) / pred against 0.01, 0.75 and 0.25, with
            // pred > 0 (a step is only tried when its predicted decrease is)
            const double ared = phi - phit;
            acc = ared >= 0.01 * pred;
            if (ared > 0.75 * pred && limited)
                D = fmin(2.0 * D, 2.0);
            else if (ared < 0.25 * pred)
                D = 0.25 * ns;
            if (acc && ns <= step_stop) stop = true;
        }
        // branch-free update: the trial Jacobian is consumed on every path,
        // so its half of the contraction is not sunk into a branch away from
        // the pipelined node loads
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            r[d] = acc ? rt[d] : r[d];
            F[d] = acc ? Ft[d] : F[d];
        }
#pragma unroll
        for (int d = 0; d < 9; ++d) J[d] = acc ? Jt[d] : J[d];
        phi = acc ? phit : phi;
        have = true;
        return stop || phi <= rstop || it >= max_it;
    }

    // step: the next trial point rt from the accepted state; true when no
    // step can be taken (the pair is then done).
    __device__ __forceinline__ bool step()
    {
        ++it;
        double g[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) g[d] = fma(J[6 + d], F[2], fma(J[3 + d], F[1], J[d] * F[0]));
        double m[3];
        int nf = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const bool held = (r[d] >= 1.0 && g[d] < 0.0) || (r[d] <= -1.0 && g[d] > 0.0);
            m[d] = held ? 0.0 : 1.0;
            nf += held ? 0 : 1;
        }
        if (nf == 0) return true;
        // one solve for both cases (lanes of a wavefront differ in nf): J d = -F
        // when all coordinates are free, else the reduced normal equations
        // (M J^T J M + I - M) d = -M g; a wavefront whose lanes are all free
        // (the usual case) skips forming the second
        double A[9], b[3], dl[3];
        if (__all(nf == 3)) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
#pragma unroll
                for (int v = 0; v < 3; ++v) A[3 * u + v] = J[3 * u + v];
                b[u] = -F[u];
            }
        } else {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
#pragma unroll
                for (int v = 0; v < 3; ++v) {
                    const double jtj =
                        fma(J[6 + u], J[6 + v], fma(J[3 + u], J[3 + v], J[u] * J[v]));
                    const double red = m[u] * m[v] * jtj + ((u == v) ? 1.0 - m[u] : 0.0);
                    A[3 * u + v] = (nf == 3) ? J[3 * u + v] : red;
                }
                b[u] = (nf == 3) ? -F[u] : -m[u] * g[u];
            }
        }
        const bool ok = solve3(A, b, dl);
        if (!ok) {
#pragma unroll
            for (int d = 0; d < 3; ++d) dl[d] = -m[d] * g[d];
        }
        const double nd = fmax(fabs(dl[0]), fmax(fabs(dl[1]), fabs(dl[2])));
        if (!(nd > 0.0) || !isfinite(nd)) return true;
        limited = nd > D;
        const double sc = limited ? D * rcp64(nd) : 1.0;
        double s[3];
        ns = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double v = fmin(1.0, fmax(-1.0, r[d] + dl[d] * sc));
            rt[d] = v;
            s[d] = v - r[d];
            ns = fmax(ns, fabs(s[d]));
        }
        double q2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double t =
                fma(J[3 * c + 2], s[2], fma(J[3 * c + 1], s[1], fma(J[3 * c], s[0], F[c])));
            q2 = fma(t, t, q2);
        }
        pred = phi - q2;
        return ns <= kStepTiny || !(pred > 0.0);
    }
};

// Squared distance of a node from the point as the closest-node rule defines
// it: the squares of the x, y and z differences summed in that order, each
// operation rounded on its own (no fused multiply-add), so that near-ties are
// decided the same way whatever the scan's arithmetic.
__device__ __forceinline__ double node_dist2(double t0, double t1, double t2)
{
#pragma clang fp contract(off)
    return (t0 * t0 + t1 * t1) + t2 * t2;
}

// Slot and point of one pair of a unit's list, loaded ahead of the element's
// staging so that the two chains of loads (list, then point) overlap it.
struct PairAhead {
    int slot = 0;
    double x[3] = {0.0, 0.0, 0.0};
    __device__ __forceinline__ void load(const LocArgs &a, int q, int end)
    {
        if (q >= end) return;
        slot = a.order[q];
        const double *p = a.pts + 3 * (long long)(slot % a.M);
        x[0] = p[0];
        x[1] = p[1];
        x[2] = p[2];
    }
};

// Reference coordinates of GLL node n (i + n1 (j + n1 k)).
template <int N1>
__device__ __forceinline__ void node_rst(BasisPtr<double> B, int n, double (&r)[3])
{
    const int i0 = n % N1, i1 = (n / N1) % N1, i2 = n / (N1 * N1);
    r[0] = r[1] = r[2] = 0.0;
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        const double zi = B.z(i);
        r[0] = (i == i0) ? zi : r[0];
        r[1] = (i == i1) ? zi : r[1];
        r[2] = (i == i2) ? zi : r[2];
    }
}

// Store one candidate's result.
__device__ __forceinline__ void store_pair(const LocArgs &a, int slot, const TRNewton &t, double he)
{
    double *o = a.res + 4 * (long long)slot;
    o[0] = t.r[0];
    o[1] = t.r[1];
    o[2] = t.r[2];
    o[3] = t.phi;
    a.res_in[slot] = sqrt(t.phi) <= a.tol * he ? 1 : 0;
}

#include "fp_mfma.inc"
#include "fp_start.inc"
#include "fp_newton8.inc"
#include "fp_mixed8.inc"
#include "fp_newton_pl.inc"
#include "fp_pair.inc"
#include "fp_point.inc"

constexpr int kStatsBlocks = 32;

// One pass's partial counts, folded into the handle's counters by the first
// kStatsBlocks blocks of its k_select, each adding its share with one atomic per
// counter (a launch of its own cost 4.5 us in each pass).
struct StatArgs {
    const unsigned *cand_part, *iter_part;
    int nb, ni;         // partial counts of each
    long long located;  // points of the pass
    unsigned long long *stats;
};

__device__ __forceinline__ void fold_stats(const LocArgs &a, const StatArgs &q)
{
    constexpr int T = 256;
    __shared__ unsigned long long sc[T / kWave], si[T / kWave];
    unsigned long long c = 0, it = 0;
    const int i0 = blockIdx.x * T + threadIdx.x;
    for (int i = i0; i < q.nb; i += kStatsBlocks * T) c += q.cand_part[i];
    for (int i = i0; i < q.ni; i += kStatsBlocks * T) it += q.iter_part[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o, kWave);
        it += __shfl_xor(it, o, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        sc[threadIdx.x / kWave] = c;
        si[threadIdx.x / kWave] = it;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long C = 0, I = 0;
        for (int w = 0; w < T / kWave; ++w) {
            C += sc[w];
            I += si[w];
        }
        const unsigned long long pairs =
            blockIdx.x == 0 ? (unsigned long long)a.elem_off[a.E] : 0ull;
        if (pairs) atomicAdd(&q.stats[0], pairs);
        if (I) atomicAdd(&q.stats[1], I);
        if (a.first) {
            if (pairs) atomicAdd(&q.stats[4], pairs);
            if (I) atomicAdd(&q.stats[5], I);
        }
        if (q.located && blockIdx.x == 0) atomicAdd(&q.stats[2], (unsigned long long)q.located);
        if (C) atomicAdd(&q.stats[3], C);
    }
}

// Distance field at a point's inside candidates, for the points whose inside
// candidates belong to two or more sessions (the only ones whose owner it
// decides).  Up to order kDeltaThread each point's thread interpolates its own; above, the
// wavefront takes such points (want) one after another, its lanes sharing each
// interpolation, and the point's own thread stores the values.  A wavefront whose points
// all want it goes through 64 chains that way, each as long as one interpolation by a
// thread at low orders, whose few node rows leave the lanes idle: findpts of 60,000
// points that all lie in two meshes of 4,896 elements each, wavefront / thread, order 1
// 233 / 140 us, 3 312 / 213, 5 422 / 330, 7 454 / 417, and of 500,000 points 798 / 542,
// 1112 / 929, 1591 / 1570, 1765 / 2105 (order 6 2166 / 2429).
//  Every solved pair used to interpolate it in its Newton kernel, by
// the four lanes of its slot through dependent loads from global memory: 57 %
// of that kernel on two overlapping annuli with 1.2e6 points, 10 % of them in
// both meshes.
constexpr int kDeltaThread = 5;

template <int N1>
__device__ __forceinline__ void thread_delta(const LocArgs &a, BasisPtr<double> B, int t, int n)
{
    for (int q = 0; q < n; ++q) {
        const long long s = (long long)q * a.M + t;
        if (a.res_in[s] != 1) continue;
        double hr[N1], hs[N1], ht[N1];
        lagrange<N1>(B, a.res[4 * s], hr);
        lagrange<N1>(B, a.res[4 * s + 1], hs);
        lagrange<N1>(B, a.res[4 * s + 2], ht);
        const double *F = a.delta + (long long)a.cand_el[s] * (N1 * N1 * N1);
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < N1; ++k) {
            double cs = 0.0;
#pragma unroll
            for (int j = 0; j < N1; ++j) {
                double r = 0.0;
#pragma unroll
                for (int i = 0; i < N1; ++i) r = fma(F[N1 * (j + N1 * k) + i], hr[i], r);
                cs = fma(r, hs[j], cs);
            }
            v = fma(cs, ht[k], v);
        }
        a.res_dl[s] = v;
    }
}

template <int N1>
__device__ __forceinline__ void wave_delta(const LocArgs &a, BasisPtr<double> B, int t, int n,
                                           bool want)
{
    unsigned long long todo = __ballot(want);
    if (todo == 0ull) return;
    __shared__ double2 sh[256 / kWave][48];
    WaveBasis<N1> W;
    W.init(B, sh[threadIdx.x / kWave]);
    while (todo != 0ull) {
        const int l = __ffsll((long long)todo) - 1;
        todo &= todo - 1ull;
        const int tl = __builtin_amdgcn_readlane(t, l), nl = __builtin_amdgcn_readlane(n, l);
        for (int k = 0; k < nl; ++k) {
            const long long s = (long long)k * a.M + tl;
            if (a.res_in[s] != 1) continue;
            const double r[3] = {a.res[4 * s], a.res[4 * s + 1], a.res[4 * s + 2]};
            W.basis(r);
            double v = W.field_part(a.delta + (long long)a.cand_el[s] * WaveShape<N1>::V);
            double z1 = 0.0, z2 = 0.0, z3 = 0.0;
            wave_sum4(v, z1, z2, z3);
            if (W.lane == l) a.res_dl[s] = v;
        }
    }
}

// Owner selection per point; ownership and ties go by explicit element ids
// (the second pass appends the candidates the first dropped, unsorted).  N1 =
// 0: a mesh without a distance field.
template <int N1>
__global__ __launch_bounds__(256) void k_select(LocArgs a, StatArgs q,
                                                const double *__restrict__ basis,
                                                int *__restrict__ code,
                                                int *__restrict__ el, double *__restrict__ rst,
                                                double *__restrict__ dist2)
{
    if (a.only && !*a.gate) return;
    if (blockIdx.x < kStatsBlocks) {
        fold_stats(a, q);
        return;
    }
    const int t = (blockIdx.x - kStatsBlocks) * blockDim.x + threadIdx.x;
    const bool on = task_on(a, t);
    if constexpr (N1 > 0) {
        const int n = on ? a.ncand[t] & kCountMask : 0;
        int s0 = -1;
        bool two = false;
        for (int k = 0; k < n; ++k) {
            const long long s = (long long)k * a.M + t;
            if (a.res_in[s] != 1) continue;
            const int sk = a.esess ? a.esess[a.cand_el[s]] : 0;
            two = two || (s0 >= 0 && sk != s0);
            s0 = sk;
        }
        const BasisPtr<double> B{as_const(basis)};
        if constexpr (N1 - 1 <= kDeltaThread) {
            if (two) thread_delta<N1>(a, B, t, n);
        } else {
            wave_delta<N1>(a, B, t, n, two);
        }
    }
    if (!on) return;
    const int p = t;
    const int nv = a.ncand[t];
    const int n = nv & kCountMask;
    const bool full = (nv >> kFullBit) != 0;
    auto S =[&](int k) { return (long long)k * a.M + t; };
    int w = -1, c = 2;
    bool anyin = false, unsolved = false, outside = false;
    for (int k = 0; k < n; ++k) {
        const int in = a.res_in[S(k)];
        anyin |= in == 1;
        unsolved |= in == kUnsolved;
        outside |= in == kOutside;
    }
    if (anyin) {
        c = 0;
        if constexpr (N1 > 0) {
            // best delta of each session among its inside candidates; the
            // largest wins (ties: smaller session), then the smallest element
            int bs = -1, s0 = -1;
            double bd = -INFINITY;
            bool two = false;
            for (int k = 0; k < n; ++k) {
                if (a.res_in[S(k)] != 1) continue;
                const int sk = a.esess ? a.esess[a.cand_el[S(k)]] : 0;
                two = two || (s0 >= 0 && sk != s0);
                s0 = sk;
            }
            if (!two) {
                bs = s0;  // one session: nothing to compare
            } else {
                bool hv = false;
                for (int k = 0; k < n; ++k) {
                    if (a.res_in[S(k)] != 1) continue;
                    const int sk = a.esess[a.cand_el[S(k)]];
                    const double dk = fmax(a.res_dl[S(k)], -INFINITY);  // not a number: last
                    if (!hv || dk > bd || (dk == bd && sk < bs)) {
                        hv = true;
                        bd = dk;
                        bs = sk;
                    }
                }
            }
            for (int k = 0; k < n; ++k) {
                if (a.res_in[S(k)] != 1) continue;
                const int sk = a.esess ? a.esess[a.cand_el[S(k)]] : 0;
                if (sk == bs && (w < 0 || a.cand_el[S(k)] < a.cand_el[S(w)])) w = k;
            }
        } else {
            for (int k = 0; k < n; ++k)
                if (a.res_in[S(k)] == 1 && (w < 0 || a.cand_el[S(k)] < a.cand_el[S(w)])) w = k;
        }
    } else if (unsolved || outside) {
        c = 1;  // provisional: the second pass decides
    } else if (n > 0) {
        c = 1;
        w = 0;
        for (int k = 1; k < n; ++k) {
            const double dk = a.res[4 * (S(k)) + 3], dw = a.res[4 * (S(w)) + 3];
            const bool tie = fabs(dk - dw) <= 1e-14 * fmax(dk, dw);
            // ties go to the smaller element id (the second pass appends the
            // candidates the first dropped, so the list is not sorted)
            if ((!tie && dk < dw) || (tie && a.cand_el[S(k)] < a.cand_el[S(w)])) w = k;
        }
    }
    code[p] = c;
    if (w < 0) {
        el[p] = -1;
        rst[3 * (long long)p] = rst[3 * (long long)p + 1] = rst[3 * (long long)p + 2] = 0.0;
        dist2[p] = INFINITY;
    } else {
        const double *o = a.res + 4 * (S(w));
        el[p] = a.cand_el[S(w)];
        rst[3 * (long long)p] = o[0];
        rst[3 * (long long)p + 1] = o[1];
        rst[3 * (long long)p + 2] = o[2];
        dist2[p] = o[3];
    }
    if (a.first) {
        bool redo = c != 0 && (!full || unsolved || outside);
        if (c == 0 && unsolved) {
            // a pair the binary32 phase left unsolved may be inside too: with
            // the distance field it may belong to a session with a larger
            // delta, without it a smaller element id wins; the second pass
            // solves it in binary64 and selects again
            for (int k = 0; k < n; ++k)
                if (a.res_in[S(k)] == kUnsolved &&
                    (N1 > 0 || a.cand_el[S(k)] < a.cand_el[S(w)]))
                    redo = true;
        }
        a.redo[t] = redo ? 1 : 0;
        // open the second pass (one store per wavefront with a flagged task)
        const unsigned long long b = __ballot(redo);
        if (b != 0ull && (int)(threadIdx.x & (kWave - 1)) == __ffsll((long long)b) - 1) *a.gate = 1;
    }
}

#define FP_DISPATCH_N1(n1, MACRO) \
    switch (n1) {                 \
        case 2: MACRO(2); break;  \
        case 3: MACRO(3); break;  \
        case 4: MACRO(4); break;  \
        case 5: MACRO(5); break;  \
        case 6: MACRO(6); break;  \
        case 7: MACRO(7); break;  \
        case 8: MACRO(8); break;  \
        case 9: MACRO(9); break;  \
        case 10: MACRO(10); break; \
        case 11: MACRO(11); break; \
        case 12: MACRO(12); break; \
        case 13: MACRO(13); break; \
        case 14: MACRO(14); break; \
        case 15: MACRO(15); break; \
        case 16: MACRO(16); break; \
        default: return hipErrorInvalidValue; \
    }

// Orders 8 and 9 have a binary32 phase.
constexpr int kMixedPlMaxN1 = 10;

// Pairs per work unit of a pass of n points: at orders 8 to 15 at least one batch
// per wavefront of the block.
static int unit_pairs(const fp_handle *h, int n)
{
    const int E = h->E;
    switch (h->n1) {
        case 9: return unit_limit(E, n, kUnitPl, 16 * PLShape<9>::W);
        case 10: return unit_limit(E, n, kUnitPl, 16 * PLShape<10>::W);
        case 11: return unit_limit(E, n, kUnitPl, 16 * PLShape<11>::W);
        case 12: return unit_limit(E, n, kUnitPl, 16 * PLShape<12>::W);
        case 13: return unit_limit(E, n, kUnitPl, 16 * PLShape<13>::W);
        case 14: return unit_limit(E, n, kUnitPl, 16 * PLShape<14>::W);
        case 15: return unit_limit(E, n, kUnitPl, 16 * PLShape<15>::W);
        case 16: return unit_limit(E, n, kUnitPl, 16 * PLShape<16>::W);
        default: return unit_limit(E, n, kUnitMfma, 16);
    }
}

// Launches the order's Newton kernel over the work units of the pass's pairs
// (n points); *nblk receives the grid size (one iteration partial per block).
static hipError_t launch_locate_kernel(const fp_handle *h, LocArgs a, int n, int K,
                                       hipStream_t s, int *nblk)
{
    *nblk = unit_grid(h->E, n, K);
    if (a.only) *nblk = std::min(*nblk, kSecondPassGrid);
// a second pass of few pairs: one wavefront per pair
#define FP_LAUNCH_PAIR(N1)                                                  \
    do {                                                                    \
        if constexpr (N1 <= kN8) {                                          \
            if (a.only) k_newton_pair<N1><<<*nblk, kWave, 0, s>>>(a, h->d_basis);      \
        } else {                                                            \
            if (a.only) k_newton_pair_rows<N1><<<*nblk, kWave, 0, s>>>(a, h->d_basis); \
        }                                                                   \
    } while (0)
// mixed precision: first pass only (the second pass is binary64).  At order 5
// the binary64 kernel (two wavefronts per SIMD) is faster than the binary32
// design of orders <= 6, so a mixed-precision handle locates in binary64 there.
constexpr int kBinary64Only = 6;
// mixed precision: first pass only (the second pass is binary64)
#define FP_LAUNCH_MFMA(N1)                                                           \
    do {                                                                             \
        if (h->precision == FP_PREC_MIXED && a.first && N1 == kN8) {                   \
            k_mixed8<<<*nblk, kWave, 0, s>>>(a, h->d_basis, h->d_basis32, h->d_dnode); \
        } else if (h->precision == FP_PREC_MIXED && a.first && N1 != kBinary64Only) {  \
            k_locate_mixed<N1><<<*nblk, kWave, 0, s>>>(a, h->d_basis, h->d_basis32,  \
                                                        h->d_dnode);                 \
        } else if (N1 == kN8) {                                                      \
            k_newton8<<<*nblk, kWave, 0, s>>>(a, h->d_basis, h->d_dnode);            \
        } else {                                                                     \
            k_locate_mfma<N1><<<*nblk, kWave, 0, s>>>(a, h->d_basis, h->d_dnode);     \
        }                                                                            \
        FP_LAUNCH_PAIR(N1);                                                          \
    } while (0)
// orders 8 to 15: matrix cores, one plane per lane; mixed precision at orders
// 8 and 9 (first pass): a binary32 phase, then binary64 Newton from its end points
#define FP_LAUNCH_PL(N1)                                                              \
    do {                                                                              \
        constexpr int T = PLShape<N1>::T;                                             \
        bool done = false;                                                            \
        if constexpr (N1 <= kMixedPlMaxN1) {                                          \
            if (h->precision == FP_PREC_MIXED && a.first) {                           \
                k_mixed_pl<N1><<<*nblk, T, 0, s>>>(a, h->d_basis32, h->d_dnode);      \
                k_newton_pl<N1, true><<<*nblk, T, 0, s>>>(a, h->d_basis, h->d_basis32, \
                                                          h->d_dnode);                \
                done = true;                                                          \
            }                                                                         \
        }                                                                             \
        if (!done)                                                                    \
            k_newton_pl<N1, false><<<*nblk, T, 0, s>>>(a, h->d_basis, h->d_basis32,   \
                                                       h->d_dnode);                   \
        FP_LAUNCH_PAIR(N1);                                                           \
    } while (0)
    switch (h->n1) {
        case 2: FP_LAUNCH_MFMA(2); break;
        case 3: FP_LAUNCH_MFMA(3); break;
        case 4: FP_LAUNCH_MFMA(4); break;
        case 5: FP_LAUNCH_MFMA(5); break;
        case 6: FP_LAUNCH_MFMA(6); break;
        case 7: FP_LAUNCH_MFMA(7); break;
        case 8: FP_LAUNCH_MFMA(8); break;
        case 9: FP_LAUNCH_PL(9); break;
        case 10: FP_LAUNCH_PL(10); break;
        case 11: FP_LAUNCH_PL(11); break;
        case 12: FP_LAUNCH_PL(12); break;
        case 13: FP_LAUNCH_PL(13); break;
        case 14: FP_LAUNCH_PL(14); break;
        case 15: FP_LAUNCH_PL(15); break;
        case 16: FP_LAUNCH_PL(16); break;
        default: return hipErrorInvalidValue;
    }
#undef FP_LAUNCH_PAIR
#undef FP_LAUNCH_MFMA
#undef FP_LAUNCH_PL
    return hipGetLastError();
}

static hipError_t launch_select(const fp_handle *h, const LocArgs &a, const StatArgs &q, int pb,
                                int *code, int *el, double *rst, double *dist2, hipStream_t s)
{
#define FP_SELECT(N1) \
    k_select<N1><<<kStatsBlocks + pb, 256, 0, s>>>(a, q, h->d_basis, code, el, rst, dist2)
    if (!a.res_dl) {
        FP_SELECT(0);
        return hipGetLastError();
    }
    FP_DISPATCH_N1(h->n1, FP_SELECT)
#undef FP_SELECT
    return hipGetLastError();
}

// A small call's pass in one kernel (and the fold of its counters).
static hipError_t launch_point(const fp_handle *h, const LocArgs &a, int *code, int *el,
                               double *rst, double *dist2, hipStream_t s)
{
    const int nblk = a.npts < kPointMax ? a.npts : kPointMax;
#define FP_POINT(N1) k_point<N1><<<nblk, kWave, 0, s>>>(a, h->d_basis, code, el, rst, dist2)
    FP_DISPATCH_N1(h->n1, FP_POINT)
#undef FP_POINT
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_point_stats<<<1, 1024, 0, s>>>(a.pt_part, nblk, a.npts, h->stats);
    return hipGetLastError();
}

}  // namespace fp

using namespace fp;

static void record(fp_handle *h, int phase, hipEvent_t a, hipEvent_t b)
{
    h->timed.push_back(TimedPair{phase, a, b});
}

namespace fp {

int run_findpts(fp_handle *h, const Work &w, int npts, const double *pts, const int *pt_session,
                int *code, int *el, double *rst, double *dist2, hipStream_t s, bool timed)
{
    for (int start = 0; start < npts; start += w.M) {
        const int n = (npts - start < w.M) ? npts - start : w.M;
        LocArgs a{};
        a.geom = h->geom;
        a.esize = h->esize;
        a.erec = h->erec;
        a.delta = h->delta;
        a.esess = h->esess;
        a.cell_off = h->cell_off;
        a.cell_box = h->cell_box;
        a.g = h->grid;
        a.pts = pts + 3 * (long long)start;
        a.psess = pt_session ? pt_session + start : nullptr;
        a.npts = n;
        a.M = w.M;
        a.tol = h->tol;
        a.ncand = w.ncand;
        a.cand_el = w.cand_el;
        a.cand_pos = w.cand_pos;
        a.elem_cnt = w.elem_cnt;
        a.elem_off = w.elem_off;
        a.units = w.units;
        a.E = h->E;
        a.order = w.order;
        a.res = w.res;
        a.res_dl = h->delta ? w.res_dl : nullptr;
        a.res_in = w.res_in;
        a.cand_part = w.cand_part;
        a.iter_part = w.iter_part;
        a.gate = w.gate;
        a.pt_part = w.pt_part;

        hipEvent_t t0 = nullptr, t1 = nullptr, l0 = nullptr, l1 = nullptr;
        if (timed) {
            t0 = pool_event(h);
            t1 = pool_event(h);
            l0 = pool_event(h);
            l1 = pool_event(h);
            FP_HIP(hipEventRecord(t0, s));
        }
        const int pb = (n + 255) / 256;
        int *co = code + start, *eo = el + start;
        double *ro = rst + 3 * (long long)start, *dO = dist2 + start;
        // first pass: oriented-box candidates; tasks without an inside
        // candidate (and with a partial candidate set) are flagged for the
        // second pass
        a.first = true;
        a.redo = w.redo;
        if (small_call(h, npts)) {
            if (timed) FP_HIP(hipEventRecord(l0, s));
            FP_HIP(launch_point(h, a, co, eo, ro, dO, s));
            if (timed) {
                FP_HIP(hipEventRecord(l1, s));
                FP_HIP(hipEventRecord(t1, s));
                record(h, 0, l0, l1);
                record(h, 2, t0, t1);
            }
            continue;
        }
        const int K = std::max(unit_pairs(h, n), pair_unit_min(w.MC));
        a.few = h->E <= kFewMax && n / kFewPoints >= h->E;
        FP_HIP(fill_int(w.elem_cnt, 0, (long long)h->E + 1, s));
        k_cand<<<pb, 256, 0, s>>>(a);
        FP_HIP(hipGetLastError());
        if (a.few)
            FP_HIP(rank_few(w.ncand, kCountMask, w.cand_el, w.cand_pos, w.elem_cnt, n, w.M, h->E,
                            s));
        FP_HIP(scan_units(w.elem_cnt, w.elem_off, w.units, h->E, K, w.scan_tmp, s));
        k_scatter<<<pb, 256, 0, s>>>(a);
        FP_HIP(hipGetLastError());
        if (timed) FP_HIP(hipEventRecord(l0, s));
        int nblk = 0;
        FP_HIP(launch_locate_kernel(h, a, n, K, s, &nblk));
        if (timed) FP_HIP(hipEventRecord(l1, s));
        FP_HIP(launch_select(h, a, StatArgs{w.cand_part, w.iter_part, pb, nblk, n, h->stats}, pb,
                             co, eo, ro, dO, s));
        // second pass over the flagged tasks with the axis-aligned candidates
        // only (other tasks get no candidates and keep their result)
        a.first = a.few = false;
        a.redo = nullptr;
        a.only = w.redo;
        a.pair_max = kPairMax;
        k_cand<<<pb, 256, 0, s>>>(a);
        FP_HIP(hipGetLastError());
        FP_HIP(scan_units(w.elem_cnt, w.elem_off, w.units, h->E, K, w.scan_tmp, s, w.gate));
        k_scatter<<<pb, 256, 0, s>>>(a);
        FP_HIP(hipGetLastError());
        hipEvent_t m0 = nullptr, m1 = nullptr;
        if (timed) {
            m0 = pool_event(h);
            m1 = pool_event(h);
            FP_HIP(hipEventRecord(m0, s));
        }
        FP_HIP(launch_locate_kernel(h, a, n, K, s, &nblk));
        if (timed) {
            FP_HIP(hipEventRecord(m1, s));
            record(h, 4, m0, m1);
        }
        FP_HIP(launch_select(h, a, StatArgs{w.cand_part, w.iter_part, 0, nblk, 0, h->stats}, pb,
                             co, eo, ro, dO, s));
        if (timed) {
            FP_HIP(hipEventRecord(t1, s));
            record(h, 0, l0, l1);
            record(h, 2, t0, t1);
        }
    }
    return FP_OK;
}

}  // namespace fp

extern "C" int findpts(fp_handle *h, int npts, const double *pts, const int *pt_session,
                       int *code, int *el, double *rst, double *dist2, void *stream)
{
    if (!h) {
        set_error("findpts: NULL handle");
        return FP_EINVAL;
    }
    if (npts < 0) {
        set_error("findpts: npts < 0");
        return FP_EINVAL;
    }
    if (npts == 0) return FP_OK;
    if (!pts || !code || !el || !rst || !dist2) {
        set_error("findpts: NULL argument");
        return FP_EINVAL;
    }
    int dev = 0;
    FP_HIP(hipGetDevice(&dev));
    if (dev != h->device) FP_HIP(hipSetDevice(h->device));
    return run_findpts(h, h->work, npts, pts, pt_session, code, el, rst, dist2,
                       (hipStream_t)stream, h->timing);
}
