// findpts_eval: tensor-product Lagrange interpolation of nodal fields at
// located points (Section 2.1 of the paper).  Points are grouped by element
// (the two-level counting sort of fp_group.h for large passes, atomic
// per-element counters otherwise) so that a wavefront reads an element's
// field values once for a run of its points (a work unit; an element with
// many points is spread over several units).  In large passes at orders
// <= 7 the values go to a staging array in the grouping's order first and
// k_ev_unstage moves them to the caller's output with consecutive stores.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "fp_basis.h"
#include "fp_group.h"
#include "fp_internal.h"
#include "fp_mfma.h"
#include "fp_wave.h"

namespace fp {

struct FieldPtrs {
    const double *f[kMaxEvalFields];
};

struct EvArgs {
    const int *code;
    const int *el;
    const double *rst;
    int npts;
    int E;
    int *cnt;
    const int *off;
    const UnitRec *units;  // work units of the points
    int *pos;
    int *order;
    double *out;   // field-major, stride npts_total
    long long ostride;
    int nf;
    double *out_all;  // first field of the call, for NaN fill
    int nf_all;
    double *sink;     // kEvSink doubles that nothing reads
    double *stage;     // non-null: k_eval_mfma writes the value of field f of the
                       // point at list position u to stage[slot[u] * nf + f], and
                       // k_ev_unstage moves it to out (else it writes out directly)
    const int *slot;   // stage row of each list position (order when not staged)
};

// Grouping key of a point: its element, or -1 when it was not found.
struct EvKey {
    const int *code, *el;
    int E;
    __device__ __forceinline__ int operator()(int p) const
    {
        const int e = el[p];
        return (code[p] != FP_NOT_FOUND && e >= 0 && e < E) ? e : -1;
    }
};

// Count points per element; not-found points get NaN right away.
__global__ __launch_bounds__(256) void k_ev_count(EvArgs a)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int e = p < a.npts ? a.el[p] : -1;
    const bool ok = p < a.npts && a.code[p] != FP_NOT_FOUND && e >= 0 && e < a.E;
    const int r = wave_rank(a.cnt, e, ok);  // converged: every lane of the wave
    if (p >= a.npts) return;
    if (ok) {
        a.pos[p] = r;
    } else {
        a.pos[p] = -1;
        for (int f = 0; f < a.nf_all; ++f) a.out_all[f * a.ostride + p] = NAN;
    }
}

__global__ __launch_bounds__(256) void k_ev_scatter(EvArgs a)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.npts) return;
    const int k = a.pos[p];
    if (k >= 0) a.order[a.off[a.el[p]] + k] = p;
}

// Staged values to the caller's field-major output: each point reads its nf
// values (its stage row is its index in the grouping's bucket order, so the
// rows of a grouping tile's points lie in a few runs) and the stores of
// consecutive points are consecutive.  Points that were not found get NaN.
// One instance per field count: the row's NF loads are issued together
// before any store (the stores could alias the stage for all the compiler
// knows, so loads and stores taken in turn would wait on each load).
template <int NF>
__global__ __launch_bounds__(256) void k_ev_unstage(EvArgs a)
{
    // the blocks of one grouping tile run on one die, whose L2 then holds
    // the tile's runs of stage rows
    const int p = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (p >= a.npts) return;
    const int j = a.pos[p];
    double v[NF];
    if (j < 0) {
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f] = NAN;
    } else {
        const double *src = a.stage + (long long)j * NF;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f] = src[f];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) a.out[f * a.ostride + p] = v[f];
}

static void launch_unstage(const EvArgs &a, int nblk, hipStream_t s)
{
    switch (a.nf) {
        case 1: k_ev_unstage<1><<<nblk, 256, 0, s>>>(a); break;
        case 2: k_ev_unstage<2><<<nblk, 256, 0, s>>>(a); break;
        case 3: k_ev_unstage<3><<<nblk, 256, 0, s>>>(a); break;
        case 4: k_ev_unstage<4><<<nblk, 256, 0, s>>>(a); break;
        case 5: k_ev_unstage<5><<<nblk, 256, 0, s>>>(a); break;
        case 6: k_ev_unstage<6><<<nblk, 256, 0, s>>>(a); break;
        case 7: k_ev_unstage<7><<<nblk, 256, 0, s>>>(a); break;
        default: k_ev_unstage<8><<<nblk, 256, 0, s>>>(a); break;
    }
}

// Interpolation on the matrix cores (orders 1..7): one wavefront per work
// unit (up to kUnitEvalMfma points of one element), points in batches of 16.
// For field f the first contraction a_f(k, j; point) = sum_i F_f[k][j][i]
// h_i(r_point) is a dense product of the field's rows (n1^2 x n1) with the
// basis values of 16 points, one 16x16x4 matrix product per 16 rows and 4
// i-values; the fields' A fragments stay in registers for all points of the
// element.  Lane n + 16 g supplies h_i(r) for i = 4 kb + g of point n
// (evaluating only its own i and j, in its rotated node order), contracts its
// rows j = g + 4 w with h_j(s) and every plane k with h_k(t), and the 4 lanes
// of point n add their partial sums (same order in all 4: the total is
// bit-identical).  T is the arithmetic: binary64, or binary32 with binary32
// accumulation for mixed precision (binary32 basis and matrix products; the
// nodal values are rounded to binary32, the result widened to binary64).  NF
// is the launch's field count (at most 8), so one pass reads each point's r
// and evaluates its basis once for all fields, and no register holds the
// fragments of a field the launch does not have.
constexpr int kUnitEvalMfma = 256;  // points of one element per work unit
constexpr int kEvMfmaMaxN1 = 8;      // orders with the matrix-core kernel
static_assert(kMixed32MaxN1 == kEvMfmaMaxN1, "binary32 interpolation is the matrix-core kernel's");
// Smallest pass that takes the staged path: below it the grouping's launches
// cost more than the scattered stores they avoid, and few elements (counted in
// LDS) need no sort for their counts either.  Staged against direct in us, order 7:
// 16384 elements, 300,000 points 114 / 62 (1 field), 270 / 217 (8 fields), 1e6
// points 158 / 128, 393 / 378; 32768 elements, 2e6 points 228 / 222, 667 / 704, 4e6
// 368 / 394, 1062 / 1241; 4096 elements, 1.5e6 points 178 / 110, 448 / 442; 512
// elements, 3e6 points 293 / 204, 819 / 860.
constexpr int kEvStageMin = 1 << 20;
constexpr int kEvStageMinFew = 1 << 21;  // up to kFewMax elements
// Wavefronts per SIMD the binary64 interpolation kernel with up to 5 fields
// is held to: three (at most 168 registers; a few bytes of spills at order 7
// with 5 fields, 12 % faster than two wavefronts on the large box); the
// other instances take what their registers allow.
template <class T, int NF>
constexpr int kEvMfmaWaves = (sizeof(T) == sizeof(double) && NF <= 5) ? 3 : 1;

template <int N1, class T, int NF>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(kEvMfmaWaves<T, NF>)))
void k_eval_mfma(EvArgs a, FieldPtrs F,
                                                     const double *__restrict__ basis,
                                                     const float *__restrict__ basis32)
{
    using S = MShape<N1>;
    constexpr int V = N1 * N1 * N1;
    constexpr int MBF = (N1 + S::PPB - 1) / S::PPB;  // M blocks per field (planes k)
    const BasisPtr<double> B{as_const(basis)};
    const BasisPtr<float> B32{as_const(basis32)};
    LaneNodes<N1, T> Z;  // h_i(r), h_j(s) only for the lane's own i, j = g + 4 w
    lane_nodes<N1, T>(B, threadIdx.x >> 4, Z);
    const UnitList units(a.units);
    for (int unit = units.first(); unit < units.total; unit += gridDim.x) {
        const Unit U = units.at(unit);
        const int e = U.seg, beg = U.beg, end = U.end;
        const int lane = threadIdx.x, n = lane & 15;
        // A fragment coordinates of this lane: row -> plane p, row jj; column i
        const int row = lane & 15, q = lane >> 4;
        const int gr = MF<T>::grp(row), vr = MF<T>::comp(row);
        const int pr = vr / S::EPP, jj = gr + 4 * (vr % S::EPP);
        T A[NF][MBF][S::KB];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const double *src = F.f[f] + (long long)e * V;
            double raw[MBF][S::KB];
#pragma unroll
            for (int mb = 0; mb < MBF; ++mb) {
                const int k = mb * S::PPB + pr;
#pragma unroll
                for (int kb = 0; kb < S::KB; ++kb) {
                    const int i = 4 * kb + q;
                    const bool ok = k < N1 && jj < N1 && i < N1;
                    if constexpr (sizeof(T) == sizeof(double)) {
                        raw[mb][kb] = ok ? src[N1 * (jj + N1 * k) + i] : 0.0;
                    } else {
                        // binary32: every load is issued unconditionally
                        // (entries past the element's nodes read its first
                        // value and are zeroed below), so that the loads are
                        // in flight together before their conversions wait
                        raw[mb][kb] = src[ok ? N1 * (jj + N1 * k) + i : 0];
                    }
                }
            }
#pragma unroll
            for (int mb = 0; mb < MBF; ++mb) {
                const int k = mb * S::PPB + pr;
#pragma unroll
                for (int kb = 0; kb < S::KB; ++kb) {
                    const bool ok = k < N1 && jj < N1 && 4 * kb + q < N1;
                    A[f][mb][kb] = ok ? (T)raw[mb][kb] : T(0);
                }
            }
        }
        // Software pipeline over the batches of 16 points: the point ids of
        // batch b + 2 and the r of batch b + 1 are in flight while batch b
        // computes.  The loop body has no branch: loads past the unit read
        // its first point again, and the slots past the unit store into the
        // sink, so the wait for the next batch's r counts only the memory
        // operations issued after it and never waits for this batch's stores.
        const auto at = [&](int u) { return u < end ? u : beg; };
        int p_next = a.order[at(beg + n)], j_next = a.slot[at(beg + n)];
        double r_next[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) r_next[d] = a.rst[3 * (long long)p_next + d];
        int p_after = a.order[at(beg + 16 + n)], j_after = a.slot[at(beg + 16 + n)];
        for (int b0 = beg; b0 < end; b0 += 16) {
            const bool act = b0 + n < end;
            const int p = p_next, j = j_next;
            const double r0 = r_next[0], r1 = r_next[1], r2 = r_next[2];
            p_next = p_after;
            j_next = j_after;
#pragma unroll
            for (int d = 0; d < 3; ++d) r_next[d] = a.rst[3 * (long long)p_next + d];
            p_after = a.order[at(b0 + 32 + n)];
            j_after = a.slot[at(b0 + 32 + n)];
            static_assert(S::KB == S::EPP, "r and s rows use the same lane indices");
            T hrl[S::KB], hsl[S::EPP], ht[N1];
            lagrange_lane<N1, T>(Z, (T)r0, hrl);
            lagrange_lane<N1, T>(Z, (T)r1, hsl);
            if constexpr (sizeof(T) == sizeof(double))
                lagrange<N1>(B, r2, ht);
            else
                lagrange<N1>(B32, (float)r2, ht);
            // the 4 lanes of a slot hold bit-identical totals and all store
            // them (to the staging list, or to the caller's output); the
            // slots past the unit store into the sink
            const long long fs = a.stage ? 1 : a.ostride;
            double *dst = !act     ? a.sink + ((unit * 16 + n) & (kEvSink - 1))
                          : a.stage ? a.stage + (long long)j * NF
                                    : a.out + p;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                T v = 0;
#pragma unroll
                for (int mb = 0; mb < MBF; ++mb) {
                    typename MF<T>::acc c = {0, 0, 0, 0};
#pragma unroll
                    for (int kb = 0; kb < S::KB; ++kb) c = MF<T>::mma(A[f][mb][kb], hrl[kb], c);
#pragma unroll
                    for (int pp = 0; pp < S::PPB; ++pp) {
                        const int k = mb * S::PPB + pp;
                        if (k < N1) {
                            T sa = 0;
#pragma unroll
                            for (int w = 0; w < S::EPP; ++w) sa = fma(c[pp * S::EPP + w], hsl[w], sa);
                            v = fma(sa, ht[k], v);
                        }
                    }
                }
                v = slot_sum(v);
                dst[act ? f * fs : 0] = (double)v;
            }
        }
    }
}

// Interpolation on the matrix cores at orders 8 to 15: one wavefront per work
// unit (up to kUnitEvalPl points of one element), binary64.  As k_eval_mfma,
// with the rows laid out one plane per lane: the rows of tile (m, hj) are the
// node rows j = 4 hj + v of the planes k = 4 m + g, so lane g of a point
// contracts whole planes with h_j(s) and weights them with its own h_k(t), and
// needs r and t basis values only at the indices 4 m + g.  An element's fragments
// do not fit in registers (27 to 64 per lane and field): they are read from
// memory, one plane group at a time with the next one's loads in flight, for
// one or two batches of 16 points whose basis values stay in registers through all the
// fields.  Fragments past the last node are zeroed (a field may hold any
// value, so a zero weight would not do).
//
// What bounds it: the fragments' reads (16 pieces of 32 bytes each, through the
// first-level cache) and the matrix products, 64 cycles per 16 rows x 4 x 16
// points, a third to four ninths of them padding at 9, 10 and 13 nodes per
// direction.  Measured against the kernels it replaces: 2e6 points on 20,000
// elements of order 9, 4 fields, 0.95 -> 0.84 ms (every node value of a point
// came from LDS); 1.5e5 points on 46,656 elements, 3 fields, 0.58 -> 0.35 ms
// (the elements' values alone are 1.1 GB); 2e5 points on 2,048 elements of order
// 12, 2 fields, 0.32 -> 0.13 ms (node values through scalar loads).  Units of 128
// or 256 points, three batches per read and staged output: within 3 %.
constexpr int kUnitEvalPl = 64;  // points of one element per work unit
// Batches of 16 points that share a read of the fragments (two spill 110 to 190
// bytes above 12 nodes per direction).
template <int N1>
constexpr int kEvalBatches = N1 <= 12 ? 2 : 1;

template <int N1>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_eval_pl(
    EvArgs a, FieldPtrs F, const double *__restrict__ basis)
{
    constexpr int V = N1 * N1 * N1, Q = (N1 + 3) / 4, BT = kEvalBatches<N1>;
    const BasisPtr<double> B{as_const(basis)};
    // lane-rotated node tables of the 4 lane groups, read at every batch
    // instead of being held in registers
    __shared__ LaneNodes<N1> sZ[4];
    const int lane = threadIdx.x, n = lane & 15, g = lane >> 4;
    if (lane < 4) lane_nodes<N1>(B, lane, sZ[lane]);
    __syncthreads();
    // this lane's fragment: row 4 v + g (plane g, node row v of a tile), column q
    const int rg = n & 3, rv = n >> 2;
    const int off = N1 * (rv + N1 * rg) + g;
    const UnitList units(a.units);
    for (int unit = units.first(); unit < units.total; unit += gridDim.x) {
        const Unit U = units.at(unit);
        for (int c0 = U.beg; c0 < U.end; c0 += 16 * BT) {
            double hr[BT][Q], hs[BT][N1], ht[BT][Q];
            int p[BT], sl[BT];
            bool act[BT];
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const int u = c0 + 16 * b + n;
                act[b] = u < U.end;
                p[b] = a.order[act[b] ? u : U.beg];
                sl[b] = a.slot[act[b] ? u : U.beg];
            }
            double r[BT][3];
#pragma unroll
            for (int b = 0; b < BT; ++b)
#pragma unroll
                for (int d = 0; d < 3; ++d) r[b][d] = a.rst[3 * (long long)p[b] + d];
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const LaneNodes<N1> *zp = sZ + g;
                asm volatile("" : "+v"(zp));  // read per batch, not hoisted
                const LaneNodes<N1> Z = *zp;
                lagrange_lane<N1>(Z, r[b][0], hr[b]);
                lagrange<N1>(B, r[b][1], hs[b]);
                lagrange_lane<N1>(Z, r[b][2], ht[b]);
            }
            const bool two = c0 + 16 < U.end;  // the second batch holds points
            const long long fs = a.stage ? 1 : a.ostride;
            for (int f = 0; f < a.nf; ++f) {
                const double *src = F.f[f] + (long long)U.seg * V;
                const auto frags = [&](int m, double (&A)[Q][Q]) {
#pragma unroll
                    for (int hj = 0; hj < Q; ++hj)
#pragma unroll
                        for (int kb = 0; kb < Q; ++kb) {
                            const int k = 4 * m + rg, j = 4 * hj + rv, i = 4 * kb + g;
                            const bool ok = (4 * m + 3 < N1 || k < N1) &&
                                            (4 * hj + 3 < N1 || j < N1) &&
                                            (4 * kb + 3 < N1 || i < N1);
                            const double v = src[ok ? off + 4 * N1 * N1 * m + 4 * N1 * hj + 4 * kb : 0];
                            A[hj][kb] = ok ? v : 0.0;
                        }
                };
                double v[BT];
#pragma unroll
                for (int b = 0; b < BT; ++b) v[b] = 0.0;
                double A[2][Q][Q];
                frags(0, A[0]);
#pragma unroll
                for (int m = 0; m < Q; ++m) {
                    if (m + 1 < Q) frags(m + 1, A[(m + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int b = 0; b < BT; ++b) {
                        if (b == 0 || two) {
                            // neighbouring products are independent
                            dx4 c[Q];
#pragma unroll
                            for (int kb = 0; kb < Q; ++kb)
#pragma unroll
                                for (int hj = 0; hj < Q; ++hj) {
                                    const dx4 z = {0, 0, 0, 0};
                                    c[hj] = MF<double>::mma(A[m & 1][hj][kb], hr[b][kb],
                                                            kb == 0 ? z : c[hj]);
                                }
                            double sa = 0.0;
#pragma unroll
                            for (int j = 0; j < N1; ++j) sa = fma(c[j / 4][j % 4], hs[b][j], sa);
                            v[b] = fma(sa, ht[b][m], v[b]);
                        }
                    }
                }
#pragma unroll
                for (int b = 0; b < BT; ++b) {
                    const double s = slot_sum(v[b]);
                    if (act[b] && g == 0)
                        (a.stage ? a.stage + (long long)sl[b] * a.nf : a.out + p[b])[f * fs] = s;
                }
            }
        }
    }
}

// Small calls: one wavefront per point, no grouping by element.  A small call
// is bound by the grouping's launches (counters, scan, scatter) and by the few
// wavefronts its work units fill, not by the element values that grouped
// points would share; the lanes take the element's node rows, so a point costs
// one read of them.
template <int N1>
__global__ __launch_bounds__(kWave) void k_eval_point(EvArgs a, FieldPtrs F,
                                                      const double *__restrict__ basis)
{
    __shared__ double2 sh[48];
    const BasisPtr<double> B{as_const(basis)};
    WaveBasis<N1> W;
    W.init(B, sh);
    for (int p = blockIdx.x; p < a.npts; p += gridDim.x) {
        const int e = a.el[p];
        const bool ok = a.code[p] != FP_NOT_FOUND && e >= 0 && e < a.E;
        double v[kMaxEvalFields];
#pragma unroll
        for (int f = 0; f < kMaxEvalFields; ++f) v[f] = 0.0;
        if (ok) {
            const double r[3] = {a.rst[3 * (long long)p], a.rst[3 * (long long)p + 1],
                                 a.rst[3 * (long long)p + 2]};
            W.basis(r);
#pragma unroll
            for (int f = 0; f < kMaxEvalFields; ++f)
                if (f < a.nf) v[f] = W.field_part(F.f[f] + (long long)e * WaveShape<N1>::V);
            wave_sum4(v[0], v[1], v[2], v[3]);
            if (a.nf > 4) wave_sum4(v[4], v[5], v[6], v[7]);
        }
        if (W.lane == 0) {
#pragma unroll
            for (int f = 0; f < kMaxEvalFields; ++f)
                if (f < a.nf) a.out[f * a.ostride + p] = ok ? v[f] : NAN;
        }
    }
}

static hipError_t launch_eval_point(int n1, const EvArgs &a, const FieldPtrs &F, const double *B,
                                    hipStream_t s)
{
    const int nblk = a.npts < kPointMax ? a.npts : kPointMax;
#define FP_EVAL_POINT(N1) \
    case N1: k_eval_point<N1><<<nblk, kWave, 0, s>>>(a, F, B); break
    switch (n1) {
        FP_EVAL_POINT(2);
        FP_EVAL_POINT(3);
        FP_EVAL_POINT(4);
        FP_EVAL_POINT(5);
        FP_EVAL_POINT(6);
        FP_EVAL_POINT(7);
        FP_EVAL_POINT(8);
        FP_EVAL_POINT(9);
        FP_EVAL_POINT(10);
        FP_EVAL_POINT(11);
        FP_EVAL_POINT(12);
        FP_EVAL_POINT(13);
        FP_EVAL_POINT(14);
        FP_EVAL_POINT(15);
        FP_EVAL_POINT(16);
        default: return hipErrorInvalidValue;
    }
#undef FP_EVAL_POINT
    return hipGetLastError();
}

// Blocks of an interpolation launch: one per element that can have points, and
// twice what the chip holds where there are few points per element, many of whose
// blocks would find no unit (an empty block costs its launch).  Capped against not,
// in us: 120,320 points on 27,360 elements, four calls 290 / 279 in all; on 16384
// elements 78 / 88; 150,001 of order 9 on 46,656 elements 317 / 332; but 62 points
// per element 211 / 208, the large box (100 per element) 3.95 / 3.59 ms.
constexpr int kEvSparseGrid = 6144;
constexpr int kEvSparse = 16;  // points per element
static int eval_grid(int E, int n, int K)
{
    const int g = unit_grid(E, n, K);
    return n / kEvSparse < E ? std::min(g, kEvSparseGrid) : g;
}

// Launches the order's interpolation kernel over the work units of n points.
static hipError_t launch_eval_kernel(int n1, int nblk, const EvArgs &a, const FieldPtrs &F,
                                     const double *B, const float *B32, bool mixed, hipStream_t s)
{
#define FP_EVAL_MFMA(N1, T, NF) \
    k_eval_mfma<N1, T, NF><<<nblk, kWave, 0, s>>>(a, F, B, B32)
#define FP_EVAL_NF(N1, T)                   \
    do {                                    \
        switch (a.nf) {                     \
            case 1: FP_EVAL_MFMA(N1, T, 1); break; \
            case 2: FP_EVAL_MFMA(N1, T, 2); break; \
            case 3: FP_EVAL_MFMA(N1, T, 3); break; \
            case 4: FP_EVAL_MFMA(N1, T, 4); break; \
            case 5: FP_EVAL_MFMA(N1, T, 5); break; \
            case 6: FP_EVAL_MFMA(N1, T, 6); break; \
            case 7: FP_EVAL_MFMA(N1, T, 7); break; \
            default: FP_EVAL_MFMA(N1, T, 8); break; \
        }                                   \
    } while (0)
#define FP_LAUNCH_MFMA(N1)             \
    do {                               \
        if (mixed)                     \
            FP_EVAL_NF(N1, float);     \
        else                           \
            FP_EVAL_NF(N1, double);    \
    } while (0)
    switch (n1) {
        case 2: FP_LAUNCH_MFMA(2); return hipGetLastError();
        case 3: FP_LAUNCH_MFMA(3); return hipGetLastError();
        case 4: FP_LAUNCH_MFMA(4); return hipGetLastError();
        case 5: FP_LAUNCH_MFMA(5); return hipGetLastError();
        case 6: FP_LAUNCH_MFMA(6); return hipGetLastError();
        case 7: FP_LAUNCH_MFMA(7); return hipGetLastError();
        case 8: FP_LAUNCH_MFMA(8); return hipGetLastError();
        default: break;
    }
#undef FP_LAUNCH_MFMA
#undef FP_EVAL_NF
#undef FP_EVAL_MFMA
#define FP_LAUNCH_PL(N1)                                                             \
    case N1:                                                                         \
        k_eval_pl<N1><<<nblk, kWave, 0, s>>>(a, F, B);                               \
        break
    switch (n1) {
        FP_LAUNCH_PL(9);
        FP_LAUNCH_PL(10);
        FP_LAUNCH_PL(11);
        FP_LAUNCH_PL(12);
        FP_LAUNCH_PL(13);
        FP_LAUNCH_PL(14);
        FP_LAUNCH_PL(15);
        FP_LAUNCH_PL(16);
        default: return hipErrorInvalidValue;
    }
#undef FP_LAUNCH_PL
    return hipGetLastError();
}

int run_eval(fp_handle *h, const Work &w, int npts, const int *code, const int *el,
             const double *rst, int nfields, const double *const *h_fields, double *out,
             hipStream_t s, bool timed)
{
    const bool small = small_eval(h, npts, nfields);
    const size_t res_bytes = w.res ? (size_t)w.M * w.MC * 4 * sizeof(double) : 0;
    for (int start = 0; start < npts; start += w.M) {
        const int n = (npts - start < w.M) ? npts - start : w.M;
        const int K = h->n1 <= kEvMfmaMaxN1 ? unit_limit(h->E, n, kUnitEvalMfma, 16)
                                            : kUnitEvalPl;  // points per unit
        hipEvent_t t0 = nullptr, t1 = nullptr, l0 = nullptr, l1 = nullptr;
        if (timed) {
            t0 = pool_event(h);
            t1 = pool_event(h);
            l0 = pool_event(h);
            l1 = pool_event(h);
            FP_HIP(hipEventRecord(t0, s));
        }
        // Staged path (matrix-core orders, passes of at least kEvStageMin or
        // kEvStageMinFew points): points grouped by element with the two-level counting
        // sort, values staged in the grouping's bucket order and moved to the
        // output by k_ev_unstage.  The grouping's
        // transient arrays and the staged values live in the pair-results
        // array of the workspace, dead once findpts has returned.  Without
        // that array (the allocation-free entry) or room in it: per-element
        // counters with atomic ranks, values written to the output directly.
        bool plan_ok = false;
        const GroupPlan gp = group_plan(n, h->E, &plan_ok);
        const int nf_max = nfields < kMaxEvalFields ? nfields : kMaxEvalFields;
        const bool staged = !small && h->n1 <= kEvMfmaMaxN1 && plan_ok &&
                            n >= (h->E <= kFewMax ? kEvStageMinFew : kEvStageMin) && w.ev_slot &&
                            res_bytes >= group_transient_bytes(gp) &&
                            res_bytes >= (size_t)n * nf_max * sizeof(double);
        for (int f0 = 0; f0 < nfields; f0 += kMaxEvalFields) {
            const int nf = (nfields - f0 < kMaxEvalFields) ? nfields - f0 : kMaxEvalFields;
            EvArgs a{};
            a.code = code + start;
            a.el = el + start;
            a.rst = rst + 3 * (long long)start;
            a.npts = n;
            a.E = h->E;
            a.cnt = w.ev_cnt;
            a.off = w.ev_off;
            a.units = w.ev_units;
            a.pos = w.ev_pos;
            a.order = w.ev_order;
            a.out = out + (long long)f0 * npts + start;
            a.ostride = npts;
            a.nf = nf;
            a.out_all = out + start;
            a.nf_all = nfields;
            a.sink = w.ev_sink;
            a.stage = staged ? w.res : nullptr;
            a.slot = staged ? w.ev_slot : w.ev_order;
            FieldPtrs F{};
            for (int f = 0; f < nf; ++f) F.f[f] = h_fields[f0 + f];
            const int pb = (n + 255) / 256;
            if (small) {
                if (timed && f0 == 0) FP_HIP(hipEventRecord(l0, s));
                FP_HIP(launch_eval_point(h->n1, a, F, h->d_basis, s));
                continue;
            }
            if (f0 == 0) {
                if (staged) {
                    GroupBufs gb;
                    gb.off = w.ev_off;
                    gb.order = w.ev_order;
                    gb.slot = w.ev_slot;
                    gb.posb = w.ev_pos;
                    group_carve(gp, (char *)w.res, gb);
                    FP_HIP(group_by_key(EvKey{a.code, a.el, h->E}, gp, gb, s));
                    FP_HIP(list_units(w.ev_off, w.ev_units, h->E, K, gb.scan_tmp, s));
                } else {
                    FP_HIP(fill_int(w.ev_cnt, 0, (long long)h->E + 1, s));
                    if (h->E <= kFewMax && h->E < n) {
                        FP_HIP(count_few(a.code, a.el, w.ev_pos, w.ev_cnt, n, h->E, a.out_all,
                                         npts, nfields, s));
                    } else {
                        k_ev_count<<<pb, 256, 0, s>>>(a);
                        FP_HIP(hipGetLastError());
                    }
                    FP_HIP(scan_units(w.ev_cnt, w.ev_off, w.ev_units, h->E, K, w.scan_tmp, s));
                    k_ev_scatter<<<pb, 256, 0, s>>>(a);
                    FP_HIP(hipGetLastError());
                }
                if (timed) FP_HIP(hipEventRecord(l0, s));
            }
            FP_HIP(launch_eval_kernel(h->n1, eval_grid(h->E, n, K), a, F, h->d_basis, h->d_basis32,
                                      h->precision == FP_PREC_MIXED, s));
            if (staged) {
                launch_unstage(a, pb, s);
                FP_HIP(hipGetLastError());
            }
        }
        if (timed) {
            FP_HIP(hipEventRecord(l1, s));
            FP_HIP(hipEventRecord(t1, s));
            h->timed.push_back(TimedPair{1, l0, l1});
            h->timed.push_back(TimedPair{3, t0, t1});
        }
    }
    return FP_OK;
}

// ---------------------------------------------------------------------------
// Interpolation without any allocation: the grouping arrays (element
// counters and offsets, the scan's block sums, each point's rank and the
// element-ordered point list) live in one file-scope device array.  Each
// device holds its own copy at its own address, found once per device with
// hipGetSymbolAddress; the host never passes the array's name to a kernel.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = size_t(32) << 20;  // 32 MiB per device
static __device__ __align__(256) char scratch[kScratchBytes];

constexpr int kScratchDevices = 64;
static std::mutex g_scratch_mu;
static char *g_scratch_ptr[kScratchDevices] = {};

// Address of the current device's scratch array (resolved on first use,
// with that device current).
int scratch_ptr(int dev, char **p)
{
    if (dev < 0 || dev >= kScratchDevices) {
        set_error("scratch: device ordinal out of range");
        return FP_EINVAL;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *q = nullptr;
        const hipError_t e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !q) return hip_fail(e == hipSuccess ? hipErrorUnknown : e,
                                                   "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = (char *)q;
    }
    *p = g_scratch_ptr[dev];
    return FP_OK;
}

// Eval-only workspace carved from the scratch array: counters and offsets
// of E + 1 elements and the scan's block sums, then the unit list and two
// arrays of M points per pass, M as large as the array allows (256 at the largest E).
// Returns false for more elements than that.
constexpr int kScratchMaxE = 4192191;

static size_t round256(size_t b) { return (b + 255) / 256 * 256; }

static bool scratch_carve(char *base, int E, int npts, Work &w)
{
    const size_t e1 = (size_t)E + 1;
    const size_t fixed = 2 * round256(e1 * sizeof(int)) +
                         round256((size_t)scan_tmp_size((long long)E + 1) * sizeof(int)) +
                         round256(kEvSink * sizeof(double));
    if (E > kScratchMaxE) return false;
    // points per pass: the largest number, in steps of 64, whose arrays fit
    const size_t room = kScratchBytes - fixed;
    const auto arrays = [E](size_t m) {
        return 2 * m * sizeof(int) +
               round256(unit_records(E, (long long)m, kUnitMin) * sizeof(UnitRec));
    };
    size_t per = 0;
    for (size_t step = (size_t)1 << 22; step >= 64; step /= 2)
        if (arrays(per + step) <= room) per += step;
    const int M = (int)std::min<size_t>(per, (size_t)std::max(npts, 1));
    char *q = base;
    w = Work{};
    w.M = M;
    w.E = E;
    w.ev_cnt = (int *)q;
    q += round256(e1 * sizeof(int));
    w.ev_off = (int *)q;
    q += round256(e1 * sizeof(int));
    w.scan_tmp = (int *)q;
    q += round256((size_t)scan_tmp_size((long long)E + 1) * sizeof(int));
    w.ev_sink = (double *)q;
    q += round256(kEvSink * sizeof(double));
    w.ev_units = (UnitRec *)q;
    q += round256(unit_records(E, (long long)per, kUnitMin) * sizeof(UnitRec));
    w.ev_pos = (int *)q;
    q += per * sizeof(int);
    w.ev_order = (int *)q;
    return true;
}

}  // namespace fp

using namespace fp;

extern "C" int findpts_eval_noalloc(fp_handle *h, int npts, const int *code, const int *el,
                                    const double *rst, int nfields,
                                    const double *const *h_fields, double *out, void *stream)
{
    if (!h) {
        set_error("findpts_eval_noalloc: NULL handle");
        return FP_EINVAL;
    }
    if (npts < 0 || nfields < 1) {
        set_error("findpts_eval_noalloc: npts < 0 or nfields < 1");
        return FP_EINVAL;
    }
    if (npts == 0) return FP_OK;
    if (!code || !el || !rst || !h_fields || !out) {
        set_error("findpts_eval_noalloc: NULL argument");
        return FP_EINVAL;
    }
    for (int f = 0; f < nfields; ++f)
        if (!h_fields[f]) {
            set_error("findpts_eval_noalloc: NULL field pointer");
            return FP_EINVAL;
        }
    int dev = 0;
    FP_HIP(hipGetDevice(&dev));
    if (dev != h->device) FP_HIP(hipSetDevice(h->device));
    char *base = nullptr;
    const int rc = scratch_ptr(h->device, &base);
    if (rc != FP_OK) return rc;
    Work w;
    if (!scratch_carve(base, h->E, npts, w)) {
        set_error("findpts_eval_noalloc: the mesh has too many elements for the 32 MiB scratch "
                  "array (at most about 4 million)");
        return FP_ERANGE;
    }
    return run_eval(h, w, npts, code, el, rst, nfields, h_fields, out, (hipStream_t)stream,
                    false);
}

extern "C" int findpts_eval(fp_handle *h, int npts, const int *code, const int *el,
                            const double *rst, int nfields, const double *const *h_fields,
                            double *out, void *stream)
{
    if (!h) {
        set_error("findpts_eval: NULL handle");
        return FP_EINVAL;
    }
    if (npts < 0 || nfields < 1) {
        set_error("findpts_eval: npts < 0 or nfields < 1");
        return FP_EINVAL;
    }
    if (npts == 0) return FP_OK;
    if (!code || !el || !rst || !h_fields || !out) {
        set_error("findpts_eval: NULL argument");
        return FP_EINVAL;
    }
    for (int f = 0; f < nfields; ++f)
        if (!h_fields[f]) {
            set_error("findpts_eval: NULL field pointer");
            return FP_EINVAL;
        }
    int dev = 0;
    FP_HIP(hipGetDevice(&dev));
    if (dev != h->device) FP_HIP(hipSetDevice(h->device));
    return run_eval(h, h->work, npts, code, el, rst, nfields, h_fields, out, (hipStream_t)stream,
                    h->timing);
}
