// findpts_setup and handle management: mesh copy, element boxes (Bernstein
// hull), hash grid, workspace.  Section 2.1 of the paper: a hash table finds
// the potential owners of x*, then elementwise bounding boxes filter them.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "fp_basis.h"
#include "fp_internal.h"
#include "fp_wave.h"

namespace fp {

// ---------------------------------------------------------------------------
// Host-side basis tables (GLL nodes, barycentric weights, Bernstein inverse).
// ---------------------------------------------------------------------------

// Legendre P_n(x) and P_n'(x) by the three-term recurrence.
static void legendre_pd(int n, double x, double &p, double &dp)
{
    double pm = 1.0, pc = x;  // P_0, P_1
    if (n == 0) { p = 1.0; dp = 0.0; return; }
    for (int k = 1; k < n; ++k) {
        double pn = ((2 * k + 1) * x * pc - k * pm) / (k + 1);
        pm = pc;
        pc = pn;
    }
    p = pc;
    // (1 - x^2) P_n' = n (P_{n-1} - x P_n); endpoints are not needed here
    dp = n * (pm - x * pc) / (1.0 - x * x);
}

// GLL nodes: +-1 and the roots of P_N'.  Roots of P_N' are the interior
// extrema of P_N; Newton's method is applied to q(x) = (1 - x^2) P_N'(x),
// whose derivative is -N (N + 1) P_N(x), starting from the Chebyshev-Gauss-
// Lobatto points; nodes are then symmetrised.
static void gll_nodes(int N, double *z)
{
    z[0] = -1.0;
    z[N] = 1.0;
    for (int i = 1; i < N; ++i) {
        double x = -std::cos(M_PI * i / N);
        for (int it = 0; it < 60; ++it) {
            double p, dp;
            legendre_pd(N, x, p, dp);
            double q = (1.0 - x * x) * dp;
            double dq = -N * (N + 1.0) * p;
            double step = q / dq;
            x -= step;
            if (std::fabs(step) <= 1e-17) break;
        }
        z[i] = x;
    }
    for (int i = 0; i < (N + 1) / 2; ++i) {
        double a = 0.5 * (z[N - i] - z[i]);
        z[i] = -a;
        z[N - i] = a;
    }
    if (N % 2 == 0) z[N / 2] = 0.0;
}

Basis make_basis(int N)
{
    Basis b{};
    gll_nodes(N, b.z);
    for (int i = 0; i <= N; ++i) {
        long double d = 1.0L;
        for (int m = 0; m <= N; ++m)
            if (m != i) d *= (long double)b.z[i] - (long double)b.z[m];
        b.wb[i] = (double)(1.0L / d);
    }
    return b;
}

std::vector<double> node_derivatives(const Basis &b, int N)
{
    const int n = N + 1;
    std::vector<double> D((size_t)n * n, 0.0);
    for (int a = 0; a < n; ++a) {
        long double diag = 0.0L;
        for (int c = 0; c < n; ++c) {
            if (c == a) continue;
            const long double v = ((long double)b.wb[c] / (long double)b.wb[a]) /
                                  ((long double)b.z[a] - (long double)b.z[c]);
            D[(size_t)a * n + c] = (double)v;
            diag -= v;
        }
        D[(size_t)a * n + a] = (double)diag;
    }
    return D;
}

// Inverse of M[i][k] = C(N,k) u_i^k (1-u_i)^(N-k), u_i = (1 + z_i)/2: maps
// nodal values to tensor-Bernstein coefficients.  Gauss-Jordan in long
// double on the host.
std::vector<double> bernstein_to_nodal_inverse(int N, const double *z)
{
    const int n = N + 1;
    std::vector<long double> A(n * 2 * n, 0.0L);
    for (int i = 0; i < n; ++i) {
        long double u = 0.5L * (1.0L + z[i]), v = 1.0L - u;
        long double c = 1.0L;  // C(N, k)
        for (int k = 0; k < n; ++k) {
            if (k > 0) c = c * (N - k + 1) / k;
            A[i * 2 * n + k] = c * std::pow(u, (long double)k) * std::pow(v, (long double)(N - k));
        }
        A[i * 2 * n + n + i] = 1.0L;
    }
    for (int c = 0; c < n; ++c) {
        int piv = c;
        for (int i = c + 1; i < n; ++i)
            if (std::fabs(A[i * 2 * n + c]) > std::fabs(A[piv * 2 * n + c])) piv = i;
        if (piv != c)
            for (int k = 0; k < 2 * n; ++k) std::swap(A[c * 2 * n + k], A[piv * 2 * n + k]);
        long double d = A[c * 2 * n + c];
        for (int k = 0; k < 2 * n; ++k) A[c * 2 * n + k] /= d;
        for (int i = 0; i < n; ++i) {
            if (i == c) continue;
            long double f = A[i * 2 * n + c];
            if (f == 0.0L) continue;
            for (int k = 0; k < 2 * n; ++k) A[i * 2 * n + k] -= f * A[c * 2 * n + k];
        }
    }
    std::vector<double> out(n * n);
    for (int i = 0; i < n; ++i)
        for (int k = 0; k < n; ++k) out[i * n + k] = (double)A[i * 2 * n + n + k];
    return out;
}

// ---------------------------------------------------------------------------
// Kernels.
// ---------------------------------------------------------------------------

// Sums (the first nsum values) and minima over a block of W wavefronts, in
// every thread.
template <int W, int NV>
__device__ __forceinline__ void block_reduce(double (&v)[NV], int nsum, double *lds)
{
    static_assert(NV % 4 == 0, "four values at a time");
#pragma unroll
    for (int q = 0; q < NV; q += 4) {
        if (q < nsum)
            wave_sum4(v[q], v[q + 1], v[q + 2], v[q + 3]);
        else
            wave_min4(v[q], v[q + 1], v[q + 2], v[q + 3]);
    }
    if constexpr (W > 1) {
        const int w = threadIdx.x / kWave;
        __syncthreads();
        if ((threadIdx.x & (kWave - 1)) == 0)
#pragma unroll
            for (int q = 0; q < NV; ++q) lds[w * NV + q] = v[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            double r = lds[q];
#pragma unroll
            for (int o = 1; o < W; ++o)
                r = (q < nsum) ? r + lds[o * NV + q] : fmin(r, lds[o * NV + q]);
            v[q] = r;
        }
    }
}

// Everything setup keeps per element, in one pass over its nodes (one block
// per element, one thread per node line): the packed copy, the axis-aligned
// box, h_e, and the oriented box, with non-finite coordinates flagged.
//
// The coefficients are those of the coordinates relative to the element's middle
// node: the transform's rounding then scales with h_e.  The boxes of absolute
// coordinates fell short by 1.5e-6 h_e at order 12 and max|x| = 1e7 h_e, of
// relative ones by 3e-13 (replayed against long double).
//
// Axis-aligned box: min and max of the Bernstein coefficients of each
// coordinate (the inverse nodal-Bernstein matrix applied along r, s, t), with
// the margin 1e-8 h_e + 1e-14 max|x|.
// Oriented box: the frame Q is the Gram-Schmidt basis of the mean edge vectors
// along r, s, t (identity if they are degenerate).  The rotated coordinates
// u = Q (x - centre) are linear in x and the transform keeps constants, so
// their Bernstein coefficients are Q (b - centre) of the coordinates' own, for
// any Q (orthonormal or not).  Margin: the axis-aligned box's, or tol h_e if
// larger, so that the bound holds after rounding too.  The record is binary32 (Q and the centre are
// rounded first, the bounds are computed for the rounded frame, then rounded
// outward) and shares a 128-byte line with the axis-aligned box.
//
// A line's n1 values stay in registers through its transform (n1^2
// multiply-adds with the matrix in scalar registers); LDS only turns the lines
// from one direction to the next (odd pitch: no bank conflicts).  The packing,
// the two box kernels (each transforming three coordinates through LDS, two
// LDS reads per multiply-add) and the record kernel that it replaces took 590
// us on 16,384 elements of order 7, and setup kept a binary32 copy of the
// coordinates that nothing read.
template <int N1>
struct ElemShape {
    static constexpr int L = N1 * N1, V = L * N1;
    static constexpr int W = (L + kWave - 1) / kWave;  // wavefronts per block
    static constexpr int P = N1 | 1;                   // row pitch in LDS
};

template <int N1>
__device__ __forceinline__ void bernstein_line(cptr<double> Bi, const double (&v)[N1],
                                               double (&o)[N1])
{
    if constexpr (N1 <= 13) FP_PIN_SGPR(Bi);  // read per line: kept from one to the next it spills
#pragma unroll
    for (int i = 0; i < N1; ++i) {
        double s = 0.0;
#pragma unroll
        for (int l = 0; l < N1; ++l) s = fma(Bi[i * N1 + l], v[l], s);
        o[i] = s;
    }
}

template <int N1>
__global__ __launch_bounds__(ElemShape<N1>::W *kWave) void k_elem(
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    const double *__restrict__ binv, double tol, double *__restrict__ geom,
    double *__restrict__ bbox, double *__restrict__ esize, double *__restrict__ erec,
    int *__restrict__ bad)
{
    using S = ElemShape<N1>;
    constexpr int L = S::L, V = S::V, P = S::P, W = S::W;
    __shared__ double sA[3 * L * P];
    __shared__ double red[W * 28];
    const long long e = blockIdx.x;
    const int t = threadIdx.x;
    const bool act = t < L;
    const int row = act ? t : 0;
    const int c0 = row % N1, c1 = row / N1;  // the line's two fixed indices, faster first
    cptr<double> Bi = as_const(binv);
    // 9 edge sums; node minima and maxima, coefficient minima and maxima, max|x|
    double v[28];
#pragma unroll
    for (int q = 0; q < 28; ++q) v[q] = q < 12 ? 0.0 : INFINITY;
    int flag = 0;
    constexpr int mid = (N1 / 2) * (1 + N1 + N1 * N1);
    double org[3];  // the middle node
#pragma unroll
    for (int c = 0; c < 3; ++c) {  // lines along r: (j, k) = (c0, c1)
        const double *X = (c == 0 ? x : (c == 1 ? y : z)) + e * V, *src = X + row * N1;
        org[c] = X[mid];
        double *dst = geom + (e * 3 + c) * V + row * N1;
        double a[N1], o[N1];
#pragma unroll
        for (int i = 0; i < N1; ++i) a[i] = src[i];
        double rs = 0.0;
        if (act) {
#pragma unroll
            for (int i = 0; i < N1; ++i) {
                dst[i] = a[i];
                flag |= !isfinite(a[i]);
                rs += a[i] - org[c];
                v[12 + c] = fmin(v[12 + c], a[i]);
                v[15 + c] = fmin(v[15 + c], -a[i]);
                v[24] = fmin(v[24], -fabs(a[i]));
            }
            v[c] = a[N1 - 1] - a[0];
            v[3 + c] = (c0 == N1 - 1 ? rs : 0.0) - (c0 == 0 ? rs : 0.0);
            v[6 + c] = (c1 == N1 - 1 ? rs : 0.0) - (c1 == 0 ? rs : 0.0);
        }
#pragma unroll
        for (int i = 0; i < N1; ++i) a[i] -= org[c];
        bernstein_line<N1>(Bi, a, o);
        if (act) {
#pragma unroll
            for (int i = 0; i < N1; ++i) sA[c * L * P + row * P + i] = o[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {  // lines along s: (i, k) = (c0, c1), in place
        double a[N1], o[N1];
        double *A = sA + c * L * P + N1 * c1 * P + c0;
#pragma unroll
        for (int j = 0; j < N1; ++j) a[j] = A[j * P];
        bernstein_line<N1>(Bi, a, o);
        if (act) {
#pragma unroll
            for (int j = 0; j < N1; ++j) A[j * P] = o[j];
        }
    }
    __syncthreads();
    double b[3][N1];  // Bernstein coefficients of the thread's line along t: (i, j) = (c0, c1)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double a[N1];
        const double *A = sA + c * L * P + c1 * P + c0;
#pragma unroll
        for (int k = 0; k < N1; ++k) a[k] = A[k * N1 * P];
        bernstein_line<N1>(Bi, a, b[c]);
#pragma unroll
        for (int k = 0; k < N1; ++k) {  // (idle threads repeat line 0)
            v[18 + c] = fmin(v[18 + c], b[c][k]);
            v[21 + c] = fmin(v[21 + c], -b[c][k]);
        }
    }
    block_reduce<W>(v, 12, red);
    if (flag) atomicOr(bad, 1);
    double he = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) he = fmax(he, -v[15 + c] - v[12 + c]);
    const double m = 1e-8 * he + 1e-14 * -v[24];
    double bb[6], ctr[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        bb[2 * c] = org[c] + v[18 + c] - m;
        bb[2 * c + 1] = org[c] - v[21 + c] + m;
        ctr[c] = (double)(float)(0.5 * (bb[2 * c] + bb[2 * c + 1]));
    }
    double Q[3][3];
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double w[3] = {v[3 * a], v[3 * a + 1], v[3 * a + 2]};
        const double ne = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
#pragma unroll
        for (int q = 0; q < a; ++q) {
            const double d = w[0] * Q[q][0] + w[1] * Q[q][1] + w[2] * Q[q][2];
#pragma unroll
            for (int c = 0; c < 3; ++c) w[c] -= d * Q[q][c];
        }
        const double nv = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
        ok = ok && isfinite(nv) && nv > 1e-6 * ne && ne > 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) Q[a][c] = ok ? w[c] / nv : 0.0;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            Q[a][c] = ok ? (double)(float)Q[a][c] : (a == c ? 1.0 : 0.0);
    double u[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = INFINITY;
#pragma unroll
    for (int k = 0; k < N1; ++k) {
        const double d0 = b[0][k] - (ctr[0] - org[0]), d1 = b[1][k] - (ctr[1] - org[1]),
                     d2 = b[2][k] - (ctr[2] - org[2]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double w = Q[a][0] * d0 + Q[a][1] * d1 + Q[a][2] * d2;
            u[a] = fmin(u[a], w);
            u[3 + a] = fmin(u[3 + a], -w);
            u[6] = fmin(u[6], -fabs(w));
        }
    }
    block_reduce<W>(u, 0, red);
    if (t == 0) {
        const double cabs = fmax(fabs(ctr[0]), fmax(fabs(ctr[1]), fabs(ctr[2])));
        // the axis-aligned box's margin, or the inside tolerance when that is
        // larger (a point within tol h_e of the element may be inside; the
        // rounded frame's rows have norm 1 to within 1e-7)
        const double mo = fmax(1e-8, (1.0 + 1e-6) * tol) * he + 1e-14 * (-u[6] + cabs);
        double *r = erec + 16 * e;
        float *o = (float *)(r + 6);
        esize[e] = he;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            bbox[6 * e + q] = bb[q];
            r[q] = bb[q];
        }
        r[15] = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int c = 0; c < 3; ++c) o[3 * a + c] = (float)Q[a][c];  // exact
            o[9 + a] = (float)ctr[a];                                   // exact
            const double l = u[a] - mo, h = -u[3 + a] + mo;
            float lf = (float)l, hf = (float)h;
            if ((double)lf > l) lf = nextafterf(lf, -INFINITY);
            if ((double)hf < h) hf = nextafterf(hf, INFINITY);
            o[12 + a] = lf;
            o[15 + a] = hf;
        }
    }
}

// Union of the element boxes (one block) and the non-finite flag, written to
// the handle's pinned host record; the flag is cleared for the next build.
__global__ __launch_bounds__(1024) void k_gbox(const double *__restrict__ bbox, int E,
                                               int *__restrict__ bad, SetupRead *__restrict__ rd)
{
    __shared__ double red[(1024 / kWave) * 8];
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = INFINITY;
#pragma unroll 4
    for (int e = threadIdx.x; e < E; e += 1024) {
        const double *b = bbox + 6 * (long long)e;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[2 * a] = fmin(v[2 * a], b[2 * a]);
            v[2 * a + 1] = fmin(v[2 * a + 1], -b[2 * a + 1]);
        }
    }
    block_reduce<1024 / kWave>(v, 0, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            rd->box[2 * a] = v[2 * a];
            rd->box[2 * a + 1] = -v[2 * a + 1];
        }
        rd->bad = *bad;
        *bad = 0;
    }
}

__device__ __forceinline__ int cell_axis(const Grid &g, int a, double x)
{
    double u = (x - g.lo[a]) * g.inv[a];
    int i = (int)floor(u);
    return i < 0 ? 0 : (i >= g.nc[a] ? g.nc[a] - 1 : i);
}

// One wavefront per element, its lanes over the cells its box meets.  Pass 0
// counts the entries per cell; pass 1 takes each entry's place from the counts
// (counting down) and writes (element, cell) there, unless the lists outgrew
// the room for them (the host then makes room and repeats the pass).
__global__ __launch_bounds__(256) void k_hash_pass(const double *__restrict__ bbox, int E,
                                                   Grid g, int pass, int *__restrict__ cnt,
                                                   const int *__restrict__ off,
                                                   int2 *__restrict__ raw, long long cap)
{
    const int e = blockIdx.x * (256 / kWave) + threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    if (e >= E) return;
    const double *b = bbox + 6 * (long long)e;
    const int i0 = cell_axis(g, 0, b[0]), i1 = cell_axis(g, 0, b[1]);
    const int j0 = cell_axis(g, 1, b[2]), j1 = cell_axis(g, 1, b[3]);
    const int k0 = cell_axis(g, 2, b[4]), k1 = cell_axis(g, 2, b[5]);
    const int ni = i1 - i0 + 1, nj = j1 - j0 + 1;
    const int n = ni * nj * (k1 - k0 + 1);  // at most 1024^3 cells in all
    if (pass == 1 && off[(long long)g.nc[0] * g.nc[1] * g.nc[2]] > cap) return;
    for (int q = lane; q < n; q += kWave) {
        const int i = i0 + q % ni, j = j0 + q / ni % nj, k = k0 + q / (ni * nj);
        const long long c = i + (long long)g.nc[0] * (j + (long long)g.nc[1] * k);
        if (pass == 0)
            atomicAdd(&cnt[c], 1);
        else
            raw[off[c] + atomicSub(&cnt[c], 1) - 1] = make_int2(e, (int)c);
    }
}

// Each entry to its place in its cell's ascending list (its rank among the
// list's elements: lists are short), with the element's box in binary32
// rounded outward (never smaller than the binary64 box) and the element id in
// the spare slot: the candidate lookup streams a cell's entries contiguously
// and tests the exact binary64 box only for the survivors.  Also the longest
// list of each block, into the counters (pass 1 has counted them down; an
// atomic maximum over the wavefronts took 45 us on one address).
__global__ __launch_bounds__(256) void k_hash_place(const double *__restrict__ bbox,
                                                    const int *__restrict__ off, long long ncell,
                                                    const int2 *__restrict__ raw, long long cap,
                                                    int *__restrict__ cell_el,
                                                    float4 *__restrict__ cell_box,
                                                    int *__restrict__ longest_of)
{
    const long long nnz = off[ncell];
    if (nnz > cap) return;
    int longest = 0;
    for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < nnz;
         q += (long long)gridDim.x * blockDim.x) {
        const int2 me = raw[q];
        const int b = off[me.y], n = off[me.y + 1] - b;
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += raw[b + j].x < me.x ? 1 : 0;
        longest = max(longest, n);
        const double *x = bbox + 6 * (long long)me.x;
        float lo[3], hi[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float l = (float)x[2 * a], u = (float)x[2 * a + 1];
            if ((double)l > x[2 * a]) l = nextafterf(l, -INFINITY);
            if ((double)u < x[2 * a + 1]) u = nextafterf(u, INFINITY);
            lo[a] = l;
            hi[a] = u;
        }
        const long long to = b + rank;
        cell_el[to] = me.x;
        cell_box[2 * to] = make_float4(lo[0], lo[1], lo[2], __int_as_float(me.x));
        cell_box[2 * to + 1] = make_float4(hi[0], hi[1], hi[2], 0.0f);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o, kWave));
    __shared__ int red[256 / kWave];
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = longest;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / kWave; ++w) longest = max(longest, red[w]);
        longest_of[blockIdx.x] = longest;
    }
}

// Entry count and longest list to the pinned host record (one wavefront).
__global__ __launch_bounds__(kWave) void k_hash_read(const int *__restrict__ off, long long ncell,
                                                     const int *__restrict__ longest_of, int nblk,
                                                     SetupRead *__restrict__ rd)
{
    int m = 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < nblk; i += kWave) m = max(m, longest_of[i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
    if (threadIdx.x == 0) {
        rd->nnz = off[ncell];
        rd->maxlen = m;
    }
}

}  // namespace fp

// ---------------------------------------------------------------------------
// Workspace layout.
// ---------------------------------------------------------------------------
namespace fp {

namespace {
struct Layout {
    size_t off = 0;
    char *base = nullptr;
    template <class T>
    T *take(size_t count)
    {
        T *p = base ? (T *)(base + off) : nullptr;
        off += ((sizeof(T) * (count ? count : 1) + 255) / 256) * 256;
        return p;
    }
};

// A serving budget admits a request by these bytes, so what one of the two calls
// needs only for itself lies in arrays that only the other one uses, or that are
// dead at that time, and adds none:
//   units     in ev_cnt .. ev_slot, 8 (E + 1) + 12 M bytes in a row.  At most
//             min(E, M MC) + M MC / K + 2 records of 8 bytes with K >= pair_unit_min(MC),
//             so M MC / K <= M.
//   ev_units  in cand_pos .. order, 8 M MC + 8 (E + 1) bytes.  At most
//             min(E, M) + M / kUnitMin + 2 records.
//   pt_part   in res_in .. ev_slot, more than 20 M bytes; a small call uses none of
//             these.  5 counters of 4 bytes for at most M wavefronts.
//   scan_tmp  runs on into iter_part, E ints and more, which the Newton kernels write
//             after the scans and k_select reads before the next ones; the tile sums
//             take (E + 1023) / 1024 x 8 bytes or less.
void lay_out(Layout &L, Work &w, int E, int MC, int M, bool delta)
{
    const size_t m = (size_t)M, mc = (size_t)MC, e1 = (size_t)E + 1;
    w.M = M;
    w.MC = MC;
    w.E = E;
    w.ncand = L.take<int>(m);
    w.cand_el = L.take<int>(m * mc);
    w.cand_pos = L.take<int>(m * mc);
    w.elem_cnt = L.take<int>(e1);
    w.elem_off = L.take<int>(e1);
    w.order = L.take<int>(m * mc);
    w.res = L.take<double>(m * mc * 4);
    w.res_dl = delta ? L.take<double>(m * mc) : nullptr;
    w.res_in = L.take<int>(m * mc);
    w.redo = L.take<int>(m);
    w.gate = L.take<int>(1);
    w.cand_part = L.take<unsigned>((m + 255) / 256);
    w.scan_tmp = L.take<int>((e1 + 4095) / 4096 + 1);
    w.iter_part = L.take<unsigned>((size_t)E + (size_t)unit_spare(M, kUnitMin));
    w.ev_cnt = L.take<int>(e1);
    w.ev_off = L.take<int>(e1);
    w.ev_pos = L.take<int>(m);
    w.ev_order = L.take<int>(m);
    w.ev_slot = L.take<int>(m);
    w.ev_sink = L.take<double>(kEvSink);
    w.units = (UnitRec *)w.ev_cnt;
    w.ev_units = (UnitRec *)w.cand_pos;
    w.pt_part = (unsigned *)w.res_in;
}
}  // namespace

size_t work_bytes(int E, int MC, int M, bool delta)
{
    Layout L;
    Work w;
    lay_out(L, w, E, MC, M, delta);
    return L.off;
}

void work_carve(Work &w, char *base, int E, int MC, int M, bool delta)
{
    Layout L;
    L.base = base;
    lay_out(L, w, E, MC, M, delta);
}

}  // namespace fp

// ---------------------------------------------------------------------------
// Handle lifetime.
// ---------------------------------------------------------------------------
using namespace fp;

static void release(fp_handle *h)
{
    void *ptrs[] = {h->d_basis, h->d_basis32, h->geom, h->esize, h->bbox, h->esess, h->delta,
                    h->cell_off, h->cell_cnt, h->cell_el, h->cell_box, h->cell_raw,
                    h->work_mem, h->scan_tmp, h->stats, h->d_flag, h->d_binv, h->d_dnode,
                    h->erec};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    if (h->h_read) (void)hipHostFree(h->h_read);
    for (auto &t : h->timed) {
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
    }
    for (auto ev : h->event_pool) (void)hipEventDestroy(ev);
    delete h;
}

template <class T>
static hipError_t dalloc(fp_handle *h, T **p, size_t count)
{
    size_t b = sizeof(T) * (count ? count : 1);
    hipError_t e = hipMalloc((void **)p, b);
    if (e == hipSuccess) h->bytes += b;
    return e;
}

#define FP_HIP_H(call)                              \
    do {                                            \
        hipError_t e_ = (call);                     \
        if (e_ != hipSuccess) {                     \
            int rc_ = fp::hip_fail(e_, #call);      \
            release(h);                             \
            return rc_;                             \
        }                                           \
    } while (0)

// Geometry products of the current node coordinates: packed copy, element
// boxes and sizes, oriented boxes, hash grid (with the per-entry binary32
// boxes) and the longest cell list.  Device arrays keep their allocation when
// large enough (an update of a moving mesh allocates only when its hash needs
// more room than before).  Synchronises `s` for the global box (the grid is
// laid out on the host) and for the entry count and longest list, once more
// when the entries need more room than there is.  What the host reads is
// written by the kernels to pinned host memory (three copies to pageable
// memory cost 250 us of an update's 0.9 ms in gaps).
static int build_geometry(fp_handle *h, const double *x, const double *y, const double *z,
                          hipStream_t s, const char *who)
{
    const int E = h->E;
    int *bad = h->d_flag;
#define FP_ELEM(N1)                                                                         \
    case N1:                                                                                \
        k_elem<N1><<<E, ElemShape<N1>::W * kWave, 0, s>>>(x, y, z, h->d_binv, h->tol, h->geom, \
                                                          h->bbox, h->esize, h->erec, bad); \
        break
    switch (h->n1) {
        FP_ELEM(2);
        FP_ELEM(3);
        FP_ELEM(4);
        FP_ELEM(5);
        FP_ELEM(6);
        FP_ELEM(7);
        FP_ELEM(8);
        FP_ELEM(9);
        FP_ELEM(10);
        FP_ELEM(11);
        FP_ELEM(12);
        FP_ELEM(13);
        FP_ELEM(14);
        FP_ELEM(15);
        FP_ELEM(16);
        default: break;
    }
#undef FP_ELEM
    FP_HIP(hipGetLastError());
    SetupRead *rd = h->h_read;
    k_gbox<<<1, 1024, 0, s>>>(h->bbox, E, bad, rd);
    FP_HIP(hipGetLastError());
    FP_HIP(hipStreamSynchronize(s));
    if (rd->bad) {
        set_error(std::string(who) + ": non-finite node coordinates");
        return FP_EINVAL;
    }

    // hash grid: about 8 E cells (two per element and axis, so each cell
    // lists few elements), cell aspect following the extents
    Grid g{};
    double ext[3], vol = 1.0;
    for (int a = 0; a < 3; ++a) {
        g.lo[a] = rd->box[2 * a];
        g.hi[a] = rd->box[2 * a + 1];
        ext[a] = g.hi[a] - g.lo[a];
        if (!(ext[a] > 0.0)) ext[a] = 1e-300;
        vol *= ext[a];
    }
    const double dens = std::cbrt(8.0 * (double)E / vol);
    for (int a = 0; a < 3; ++a) {
        double n = std::floor(ext[a] * dens + 0.5);
        n = std::min(std::max(n, 1.0), 1024.0);
        g.nc[a] = (int)n;
        g.inv[a] = g.nc[a] / ext[a];
    }
    h->grid = g;
    h->ncell = (long long)g.nc[0] * g.nc[1] * g.nc[2];
    if (h->ncell + 1 > h->cell_cap) {
        (void)hipFree(h->cell_off);
        (void)hipFree(h->cell_cnt);
        (void)hipFree(h->scan_tmp);
        h->bytes -= sizeof(int) * (2 * (size_t)h->cell_cap + (size_t)h->scan_tmp_n);
        h->cell_off = h->cell_cnt = h->scan_tmp = nullptr;
        h->cell_cap = h->ncell + 1;
        FP_HIP(dalloc(h, &h->cell_off, h->cell_cap));
        FP_HIP(dalloc(h, &h->cell_cnt, h->cell_cap));
        h->scan_tmp_n = std::max(scan_tmp_size(h->ncell), scan_tmp_size((long long)E + 1));
        FP_HIP(dalloc(h, &h->scan_tmp, h->scan_tmp_n));
    }
    int *cnt = h->cell_cnt;
    const int eb = (E + 256 / kWave - 1) / (256 / kWave);
    FP_HIP(fill_int(cnt, 0, h->ncell + 1, s));
    k_hash_pass<<<eb, 256, 0, s>>>(h->bbox, E, g, 0, cnt, nullptr, nullptr, 0);
    FP_HIP(hipGetLastError());
    FP_HIP(scan_exclusive(cnt, h->cell_off, (int)h->ncell, h->scan_tmp, s));
    // lists in the room there is (kernels that find it too small do nothing)
    for (int turn = 0; turn < 2; ++turn) {
        int nblk = 0;
        if (h->cell_el) {
            k_hash_pass<<<eb, 256, 0, s>>>(h->bbox, E, g, 1, cnt, h->cell_off, h->cell_raw,
                                           h->nnz_cap);
            FP_HIP(hipGetLastError());
            // (one counter per block: no more blocks than cells)
            nblk = (int)std::max(1LL, std::min({(h->nnz_cap + 255) / 256, 4096LL, h->ncell}));
            k_hash_place<<<nblk, 256, 0, s>>>(h->bbox, h->cell_off, h->ncell, h->cell_raw,
                                              h->nnz_cap, h->cell_el, h->cell_box, cnt);
            FP_HIP(hipGetLastError());
        }
        k_hash_read<<<1, kWave, 0, s>>>(h->cell_off, h->ncell, cnt, nblk, rd);
        FP_HIP(hipGetLastError());
        FP_HIP(hipStreamSynchronize(s));
        h->nnz = rd->nnz;
        if (h->cell_el && h->nnz <= h->nnz_cap) break;
        (void)hipFree(h->cell_el);
        (void)hipFree(h->cell_box);
        (void)hipFree(h->cell_raw);
        h->bytes -= (sizeof(int) + 2 * sizeof(float4) + sizeof(int2)) * (size_t)h->nnz_cap;
        h->cell_el = nullptr;
        h->cell_box = nullptr;
        h->cell_raw = nullptr;
        h->nnz_cap = 0;
        FP_HIP(dalloc(h, &h->cell_el, (size_t)h->nnz));
        FP_HIP(dalloc(h, &h->cell_box, 2 * (size_t)h->nnz));
        FP_HIP(dalloc(h, &h->cell_raw, (size_t)h->nnz));
        h->nnz_cap = h->nnz;
    }
    h->max_cell = rd->maxlen;
    h->MC = std::max(1, h->max_cell);
    return FP_OK;
}

// The handle's own workspace, (re)carved when the longest cell list outgrew
// it.  A quarter of headroom on the candidate slots lets a moving mesh whose
// longest list changes by a little keep its workspace (a new allocation is
// also touched for the first time by the next call, which costs tens of ms
// for a workspace of a gigabyte).
static int ensure_workspace(fp_handle *h, const char *who)
{
    if (h->work_mem && h->MC <= h->work.MC) return FP_OK;
    int mc_cap = h->MC + (h->MC + 3) / 4;
    if ((double)h->max_points * (double)mc_cap >= 2147483647.0) mc_cap = h->MC;
    if ((double)h->max_points * (double)mc_cap >= 2147483647.0) {
        set_error(std::string(who) +
                  ": max_points x longest cell list exceeds 2^31; lower max_points");
        return FP_ERANGE;
    }
    if (h->work_mem) {
        FP_HIP(hipDeviceSynchronize());  // calls in flight may still use it
        (void)hipFree(h->work_mem);
        h->bytes -= h->work_bytes;
        h->work_mem = nullptr;
    }
    h->work_bytes = work_bytes(h->E, mc_cap, h->max_points, h->delta != nullptr);
    FP_HIP(hipMalloc(&h->work_mem, h->work_bytes));
    h->bytes += h->work_bytes;
    work_carve(h->work, (char *)h->work_mem, h->E, mc_cap, h->max_points, h->delta != nullptr);
    return FP_OK;
}

extern "C" int findpts_setup(fp_handle **out, const double *x, const double *y,
                             const double *z, int E, int N, double tol,
                             const int *elem_session, const double *delta,
                             int max_points, int precision, void *stream)
{
    if (!out || !x || !y || !z) {
        set_error("findpts_setup: NULL argument");
        return FP_EINVAL;
    }
    *out = nullptr;
    if (N < 1 || N > kMaxN1 - 1) {
        set_error("findpts_setup: N must be in [1, 15]");
        return FP_ERANGE;
    }
    if (E < 1 || max_points < 1 || !(tol > 0.0 && tol < 1.0) ||
        (precision != FP_PREC_FP64 && precision != FP_PREC_MIXED)) {
        set_error("findpts_setup: need E >= 1, max_points >= 1, 0 < tol < 1, known precision");
        return FP_EINVAL;
    }
    const long long n1 = N + 1, V = n1 * n1 * n1;
    if ((long long)E * V * 3 > (1LL << 40)) {
        set_error("findpts_setup: mesh too large");
        return FP_ERANGE;
    }
    hipStream_t s = (hipStream_t)stream;
    fp_handle *h = new fp_handle();
    if (hipGetDevice(&h->device) != hipSuccess) {
        delete h;
        set_error("findpts_setup: no HIP device");
        return FP_EHIP;
    }
    {
        // resolve this device's interpolation scratch array at set-up, so
        // that findpts_eval_noalloc never resolves it inside a capture
        char *sp = nullptr;
        const int rc = scratch_ptr(h->device, &sp);
        if (rc != FP_OK) {
            delete h;
            return rc;
        }
    }
    h->E = E;
    h->N = N;
    h->n1 = (int)n1;
    h->V = (int)V;
    h->tol = tol;
    h->precision = precision;
    h->max_points = max_points;
    h->basis = make_basis(N);
    for (int i = 0; i < kMaxN1; ++i) {
        h->basis32.z[i] = (float)h->basis.z[i];
        h->basis32.wb[i] = (float)h->basis.wb[i];
    }
    const long long EV = (long long)E * V;

    // mesh-size arrays (kept for the handle's lifetime)
    FP_HIP_H(dalloc(h, &h->geom, 3 * EV));
    FP_HIP_H(dalloc(h, &h->esize, E));
    FP_HIP_H(dalloc(h, &h->bbox, 6 * (size_t)E));
    FP_HIP_H(dalloc(h, &h->erec, 16 * (size_t)E));
    FP_HIP_H(dalloc(h, &h->stats, kStats));
    FP_HIP_H(dalloc(h, &h->d_basis, 2 * kMaxN1));
    FP_HIP_H(dalloc(h, &h->d_basis32, 2 * kMaxN1));
    FP_HIP_H(dalloc(h, &h->d_flag, 1));
    FP_HIP_H(hipHostMalloc((void **)&h->h_read, sizeof(SetupRead), hipHostMallocDefault));
    FP_HIP_H(fill_int(h->d_flag, 0, 1, s));
    FP_HIP_H(dalloc(h, &h->d_binv, (size_t)(n1 * n1)));
    FP_HIP_H(dalloc(h, &h->d_dnode, (size_t)(n1 * n1)));
    FP_HIP_H(hipMemcpyAsync(h->d_basis, &h->basis, sizeof(Basis), hipMemcpyHostToDevice, s));
    FP_HIP_H(hipMemcpyAsync(h->d_basis32, &h->basis32, sizeof(Basis32), hipMemcpyHostToDevice, s));
    FP_HIP_H(hipMemsetAsync(h->stats, 0, kStats * sizeof(unsigned long long), s));
    {
        const std::vector<double> binv = bernstein_to_nodal_inverse(N, h->basis.z);
        const std::vector<double> dnode = node_derivatives(h->basis, N);
        FP_HIP_H(hipMemcpyAsync(h->d_binv, binv.data(), sizeof(double) * n1 * n1,
                                hipMemcpyHostToDevice, s));
        FP_HIP_H(hipMemcpyAsync(h->d_dnode, dnode.data(), sizeof(double) * n1 * n1,
                                hipMemcpyHostToDevice, s));
        FP_HIP_H(hipStreamSynchronize(s));  // the host vectors go out of scope
    }
    if (elem_session) {
        FP_HIP_H(dalloc(h, &h->esess, E));
        FP_HIP_H(hipMemcpyAsync(h->esess, elem_session, sizeof(int) * E,
                                hipMemcpyDeviceToDevice, s));
    }
    if (delta) {
        FP_HIP_H(dalloc(h, &h->delta, EV));
        FP_HIP_H(hipMemcpyAsync(h->delta, delta, sizeof(double) * EV,
                                hipMemcpyDeviceToDevice, s));
    }
    int rc = build_geometry(h, x, y, z, s, "findpts_setup");
    if (rc == FP_OK) rc = ensure_workspace(h, "findpts_setup");
    if (rc != FP_OK) {
        release(h);
        return rc;
    }
    FP_HIP_H(hipStreamSynchronize(s));
    *out = h;
    return FP_OK;
}

extern "C" int findpts_update(fp_handle *h, const double *x, const double *y, const double *z,
                              const double *delta, void *stream)
{
    if (!h || !x || !y || !z) {
        set_error("findpts_update: NULL argument");
        return FP_EINVAL;
    }
    if (delta && !h->delta) {
        set_error("findpts_update: the handle was set up without a distance field");
        return FP_ESTATE;
    }
    hipStream_t s = (hipStream_t)stream;
    int dev = 0;
    FP_HIP(hipGetDevice(&dev));
    if (dev != h->device) FP_HIP(hipSetDevice(h->device));
    if (delta)
        FP_HIP(hipMemcpyAsync(h->delta, delta, sizeof(double) * (size_t)h->E * h->V,
                              hipMemcpyDeviceToDevice, s));
    int rc = build_geometry(h, x, y, z, s, "findpts_update");
    if (rc == FP_OK) rc = ensure_workspace(h, "findpts_update");
    return rc;
}

extern "C" int findpts_free(fp_handle *h)
{
    if (!h) return FP_OK;
    (void)hipDeviceSynchronize();
    release(h);
    return FP_OK;
}

extern "C" int findpts_set_precision(fp_handle *h, int precision)
{
    if (!h || (precision != FP_PREC_FP64 && precision != FP_PREC_MIXED)) {
        set_error("findpts_set_precision: bad handle or precision");
        return FP_EINVAL;
    }
    h->precision = precision;
    return FP_OK;
}

extern "C" int findpts_stats(fp_handle *h, long long *h_counts, int reset)
{
    if (!h || !h_counts) {
        set_error("findpts_stats: NULL argument");
        return FP_EINVAL;
    }
    unsigned long long v[kStats];
    FP_HIP(hipDeviceSynchronize());
    FP_HIP(hipMemcpy(v, h->stats, sizeof v, hipMemcpyDeviceToHost));
    for (int i = 0; i < kStats; ++i) h_counts[i] = (long long)v[i];
    if (reset) FP_HIP(hipMemset(h->stats, 0, sizeof v));
    return FP_OK;
}

extern "C" int findpts_get_bbox(fp_handle *h, double *h_bbox, double *h_size)
{
    if (!h || !h_bbox || !h_size) {
        set_error("findpts_get_bbox: NULL argument");
        return FP_EINVAL;
    }
    FP_HIP(hipDeviceSynchronize());
    FP_HIP(hipMemcpy(h_bbox, h->bbox, sizeof(double) * 6 * h->E, hipMemcpyDeviceToHost));
    FP_HIP(hipMemcpy(h_size, h->esize, sizeof(double) * h->E, hipMemcpyDeviceToHost));
    return FP_OK;
}

extern "C" int findpts_get_hash(fp_handle *h, int *h_nc, double *h_lo, double *h_dx,
                                long long *h_meta)
{
    if (!h || !h_nc || !h_lo || !h_dx || !h_meta) {
        set_error("findpts_get_hash: NULL argument");
        return FP_EINVAL;
    }
    for (int a = 0; a < 3; ++a) {
        h_nc[a] = h->grid.nc[a];
        h_lo[a] = h->grid.lo[a];
        h_dx[a] = 1.0 / h->grid.inv[a];
    }
    h_meta[0] = h->ncell;
    h_meta[1] = h->nnz;
    h_meta[2] = h->max_cell;
    return FP_OK;
}

extern "C" int findpts_get_cells(fp_handle *h, int *h_cell_off, int *h_cell_el)
{
    if (!h || !h_cell_off || !h_cell_el) {
        set_error("findpts_get_cells: NULL argument");
        return FP_EINVAL;
    }
    FP_HIP(hipDeviceSynchronize());
    FP_HIP(hipMemcpy(h_cell_off, h->cell_off, sizeof(int) * (h->ncell + 1),
                     hipMemcpyDeviceToHost));
    FP_HIP(hipMemcpy(h_cell_el, h->cell_el, sizeof(int) * (h->nnz ? h->nnz : 0),
                     hipMemcpyDeviceToHost));
    return FP_OK;
}

extern "C" int findpts_footprint(const fp_handle *h, size_t *h_bytes)
{
    if (!h || !h_bytes) {
        set_error("findpts_footprint: NULL argument");
        return FP_EINVAL;
    }
    *h_bytes = h->bytes;
    return FP_OK;
}

// ---------------------------------------------------------------------------
// Timing with events on the call's stream.
// ---------------------------------------------------------------------------
namespace fp {
hipEvent_t pool_event(fp_handle *h)
{
    if (!h->event_pool.empty()) {
        hipEvent_t e = h->event_pool.back();
        h->event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}
}  // namespace fp

extern "C" int findpts_timing(fp_handle *h, int enable)
{
    if (!h) {
        set_error("findpts_timing: NULL handle");
        return FP_EINVAL;
    }
    h->timing = enable != 0;
    return FP_OK;
}

extern "C" int findpts_timing_read(fp_handle *h, double *h_ms, long long *h_n)
{
    if (!h || !h_ms || !h_n) {
        set_error("findpts_timing_read: NULL argument");
        return FP_EINVAL;
    }
    for (int i = 0; i < kTimedPhases; ++i) {
        h_ms[i] = 0.0;
        h_n[i] = 0;
    }
    for (auto &t : h->timed) {
        FP_HIP(hipEventSynchronize(t.b));
        float ms = 0.0f;
        FP_HIP(hipEventElapsedTime(&ms, t.a, t.b));
        if (t.phase >= 0 && t.phase < kTimedPhases) {
            h_ms[t.phase] += ms;
            h_n[t.phase] += 1;
        }
        h->event_pool.push_back(t.a);
        h->event_pool.push_back(t.b);
    }
    h->timed.clear();
    return FP_OK;
}
