// Internal declarations of the gfx950 findpts library (not installed).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/findpts.h"

namespace fp {

constexpr int kMaxN1 = 16;       // N <= 15
constexpr int kMaxEvalFields = 8; // fields per interpolation launch
constexpr int kEvSink = 512;       // doubles in Work::ev_sink (a power of two)
constexpr int kStats = 6;          // device counters of a handle (findpts_stats)
constexpr int kPointMax = 16384;   // points of the largest call taken one wavefront per point
constexpr int kMixed32MaxN1 = 8;   // orders whose mixed precision interpolates in binary32
constexpr int kPointCounters = 5;  // counters of one wavefront of such a call
constexpr int kTimedPhases = 5;    // timed phases (findpts_timing_read)
constexpr int kWave = 64;
constexpr int kXcds = 8;  // accelerator dies; workgroups are dealt to them in turn

// Block index remapped so that each accelerator die (XCD, own L2) runs one
// contiguous range of the G block indices: workgroup b is dispatched to die
// b mod kXcds, and becomes number b / kXcds of that die's range.  A bijection
// of [0, G); neighbouring work then shares one L2.
__device__ __forceinline__ int xcd_block(int b, int G)
{
    const int x = b % kXcds, i = b / kXcds, q = G / kXcds, r = G % kXcds;
    return x * q + (x < r ? x : r) + i;
}

// Unit walked first by block b of a grid of G blocks (blocks go to the dies
// in turn, b mod kXcds): each die takes runs of kXcdRun consecutive units,
// the runs of the dies interleaved, so that the units of a crowded element
// (consecutive indices) mostly share one die's L2 while the work stays spread
// over all dies.  A bijection of [0, G) (the last partial round of runs
// keeps b).
constexpr int kXcdRun = 8;
__device__ __forceinline__ long long xcd_unit(long long b, long long G)
{
    constexpr long long P = (long long)kXcds * kXcdRun;
    if (b >= (G / P) * P) return b;
    const long long i = b / kXcds, x = b % kXcds;
    return (i / kXcdRun) * P + x * kXcdRun + i % kXcdRun;
}

// GLL nodes z_i and barycentric weights wb_i = 1 / prod_{m != i} (z_i - z_m),
// passed to kernels by value (kernel arguments are read through the scalar
// cache).
struct Basis {
    double z[kMaxN1];
    double wb[kMaxN1];
};

struct Basis32 {
    float z[kMaxN1];
    float wb[kMaxN1];
};

// Hash grid parameters passed by value.
struct Grid {
    double lo[3];
    double hi[3];
    double inv[3];  // cells per unit length
    int nc[3];
};

// What a build's kernels tell the host.
struct SetupRead {
    double box[6];  // union of the element boxes
    int bad;        // a node coordinate is not finite
    int nnz;        // entries of the hash cells
    int maxlen;     // longest cell list
};

struct TimedPair {
    int phase;
    hipEvent_t a, b;
};

struct UnitRec;

// Workspace of one findpts / findpts_eval call on one stream: M points per
// pass, MC candidate slots per point (the longest hash-cell list), E + 1
// element counters.  Carved from one device block; a handle owns one, the
// serving layer carves one per admitted request from its arena.
struct Work {
    int M = 0, MC = 1, E = 0;
    int *ncand = nullptr;     // M
    int *cand_el = nullptr;   // M x MC
    int *cand_pos = nullptr;  // M x MC, rank of the pair within its element
    int *elem_cnt = nullptr;  // E + 1
    int *elem_off = nullptr;  // E + 1
    int *order = nullptr;     // M x MC pair slots grouped by element
    double *res = nullptr;    // M x MC x 4: r, s, t, d2
    double *res_dl = nullptr; // M x MC: delta at the candidate (if delta)
    int *res_in = nullptr;    // M x MC: inside flag
    int *redo = nullptr;      // M: second-pass flag per point
    int *gate = nullptr;      // 1: nonzero when the first pass flagged any point
    unsigned *cand_part = nullptr;  // ceil(M / 256): per-block candidate counts
    int *scan_tmp = nullptr;  // tile sums of the scans (iter_part included)
    unsigned *iter_part = nullptr;  // E + unit_spare(M, kUnitMin): Newton iterations per block
    // in other arrays' room (lay_out)
    UnitRec *units = nullptr;     // unit list of the pairs
    UnitRec *ev_units = nullptr;  // unit list of the points
    unsigned *pt_part = nullptr;  // min(M, kPointMax) x kPointCounters (small calls)
    int *ev_cnt = nullptr;    // E + 1
    int *ev_off = nullptr;    // E + 1
    int *ev_pos = nullptr;    // M
    int *ev_order = nullptr;  // M
    int *ev_slot = nullptr;   // M: stage row of each list position (grouped path)
    double *ev_sink = nullptr;  // kEvSink: stores of interpolation slots past a unit
};

// Bytes of a workspace (256-byte aligned sub-arrays); carve() lays it out
// from `base` (which must be 256-byte aligned).
size_t work_bytes(int E, int MC, int M, bool delta);
void work_carve(Work &w, char *base, int E, int MC, int M, bool delta);

}  // namespace fp

struct fp_handle {
    int device = 0;
    int E = 0, N = 0, n1 = 0, V = 0;
    double tol = 0.0;
    int precision = 0;
    int max_points = 0;

    // mesh (handle-owned)
    double *geom = nullptr;    // E x 3 x V, element-blocked, r index fastest
    double *esize = nullptr;   // E: h_e
    double *bbox = nullptr;    // E x 6
    double *erec = nullptr;    // E x 16 doubles (one 128-byte line per element): the
                               // axis-aligned box (6 doubles) then the oriented box
                               // (18 binary32 values: frame Q, row-major, rows = axes,
                               // centre, rotated lo, rotated hi), for the candidate tests
    int *esess = nullptr;      // E or null
    double *delta = nullptr;   // E x V or null

    // hash grid
    fp::Grid grid{};
    long long ncell = 0, nnz = 0;
    int max_cell = 0;
    int *cell_off = nullptr;   // ncell + 1
    int *cell_cnt = nullptr;   // ncell + 1 (hash build)
    long long cell_cap = 0;    // allocated length of cell_off / cell_cnt
    long long nnz_cap = 0;     // allocated entries of cell_el / cell_box
    int *cell_el = nullptr;    // nnz
    float4 *cell_box = nullptr; // 2 nnz: binary32 outward box + element id per entry

    // workspace of the handle's own calls (max_points per pass)
    int MC = 1;                 // longest hash-cell list (>= 1)
    fp::Work work{};
    void *work_mem = nullptr;
    size_t work_bytes = 0;
    int2 *cell_raw = nullptr;   // nnz: (element, cell) per entry, unsorted (hash build)
    int *d_flag = nullptr;      // hash build: non-finite flag (zero between builds)
    fp::SetupRead *h_read = nullptr;  // pinned host memory the build's kernels write
    double *d_binv = nullptr;   // Bernstein-to-nodal inverse (n1 x n1)
    int *scan_tmp = nullptr;    // setup's scans (cells)
    int scan_tmp_n = 0;

    // [pairs solved, Newton iterations, points located, axis-aligned box
    //  candidates (the hash + box candidate count of the method), pairs
    //  solved by first passes, their Newton iterations]
    unsigned long long *stats = nullptr;

    fp::Basis basis{};
    fp::Basis32 basis32{};
    double *d_basis = nullptr;   // device copy of basis (z, wb)
    double *d_dnode = nullptr;   // n1 x n1: h_b'(z_a) at row a, column b
    float *d_basis32 = nullptr;  // device copy of basis32
    size_t bytes = 0;

    bool timing = false;
    std::vector<fp::TimedPair> timed;
    std::vector<hipEvent_t> event_pool;
};

namespace fp {

void set_error(const std::string &msg);
int hip_fail(hipError_t e, const char *what);
// Device address of the interpolation scratch array of device dev (resolved
// once per device, with dev current); FP_OK or an error code.
int scratch_ptr(int dev, char **p);
hipEvent_t pool_event(fp_handle *h);

#define FP_HIP(call)                                         \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return fp::hip_fail(e_, #call); \
    } while (0)

// Work units of an element-grouped list: the entries [off[e], off[e + 1]) of an
// element with more than K of them are cut into ceil(cnt / K) or fewer equal
// pieces (unit_size entries each, the last one shorter), any other element with
// entries is one unit, and the units are listed without gaps (scan_units writes
// the list together with the offsets).  Record 0 is {units, entries}; record
// 1 + u is {first entry, element} of unit u, and the next record's first entry
// is its end (a last record {entries, E} closes the list).
//
// Cutting the whole list at multiples of K instead, which needs no table, gave an
// element of 60 to 100 entries two units about as often as one, each staging the
// element and draining its slots, and left a unit index per empty element that a
// wavefront had to search for.  Measured, with the scan's launches: annulus of 1.01e6
// points 1242 -> 1212 us (findpts), 275 -> 254 (4 fields); large box of 2e7 21.7 ->
// 21.2 ms, 3.76 -> 3.52; 120,320 known points on 27,360 elements, four interpolations
// 220 -> 145 us; 2D ring of 1.01e6 432 -> 368.
constexpr int kUnitMin = 64;  // smallest K
struct Unit {
    int seg, beg, end;
};
struct UnitRec {
    int beg, seg;
};

// Entries of each unit of an element with cnt > 0 entries: the units of a crowded
// element are equal up to a batch of 16.
__host__ __device__ __forceinline__ int unit_size(int cnt, int K)
{
    if (cnt <= K) return cnt;
    const int nu = (cnt - 1) / K + 1;
    return ((cnt - 1) / nu + 16) & ~15;
}

// Unit size of a list of n entries of E elements whose kernel runs best at `most`:
// less where the elements alone do not make 2048 units (two wavefronts per SIMD),
// in steps of `step` and at least kUnitMin.
inline int unit_limit(int E, int n, int most, int step)
{
    if (E >= 2048) return most;
    const int k = (n / 2048 + step - 1) / step * step;
    const int least = step > kUnitMin ? step : kUnitMin;
    return k < least ? least : (k < most ? k : most);
}

// Smallest unit of the pairs of a workspace with MC candidate slots per point: kUnitMin,
// more where the cell lists are longer, so that the pieces of crowded elements are at
// most one per point (the room for the list, work_carve).
inline int pair_unit_min(int MC)
{
    const int k = (MC + 15) / 16 * 16;
    return k > kUnitMin ? k : kUnitMin;
}

// Records of a list of at most n entries of E elements at unit size K or more.
inline size_t unit_records(long long E, long long n, int K)
{
    return (size_t)((E < n ? E : n) + n / K + 2);
}

struct UnitList {
    const UnitRec *rec;
    int total;

    __device__ __forceinline__ explicit UnitList(const UnitRec *u) : rec(u + 1), total(__builtin_amdgcn_readfirstlane(u->beg)) {}
    // the block's first unit (then every gridDim.x-th one below total)
    __device__ __forceinline__ int first() const
    {
        const int G = min((int)gridDim.x, total), b = (int)blockIdx.x;
        return b < G ? (int)xcd_unit(b, G) : total;
    }
    __device__ __forceinline__ Unit at(int u) const
    {
        // u is the same in all lanes
        return Unit{__builtin_amdgcn_readfirstlane(rec[u].seg),
                    __builtin_amdgcn_readfirstlane(rec[u].beg),
                    __builtin_amdgcn_readfirstlane(rec[u + 1].beg)};
    }
};

// Blocks of a unit launch over E elements for a list of about n entries (n
// points: two candidate pairs each at most, in all but rare cases): the elements
// that can have entries, and up to 2 n / K (at most kUnitSpare) for the pieces of
// crowded ones.  Units beyond the grid are taken by the grid-stride walk.
constexpr long long kUnitSpare = 4096;
inline long long unit_spare(long long n, int K)
{
    const long long extra = 2 * ((n + K - 1) / K);
    return extra < kUnitSpare ? extra : kUnitSpare;
}
inline int unit_grid(int E, long long n, int K)
{
    const long long g = (E < 2 * n ? (long long)E : 2 * n) + unit_spare(n, K);
    return (int)(g < 1 ? 1 : (g > 0x7fffffffLL ? 0x7fffffffLL : g));
}

// Grid of a second-pass launch: usually nearly empty, so a bounded grid walks
// the units with its grid-stride loop instead of one block per element.
constexpr int kSecondPassGrid = 8192;

// Rank of each active lane's entry in its group's counter, cnt[e] += 1 per
// entry.  Lanes of a wavefront that share the group of the first pending
// lane take their ranks from one atomic add (up to four such groups); any
// other lane adds alone.  Call from converged code (every lane of the
// wavefront), act false for lanes without an entry.  The ranks of a group are
// distinct and fill [old count, new count).
__device__ __forceinline__ int wave_rank(int *cnt, int e, bool act)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned long long pending = __ballot(act);
    int rank = 0;
    for (int it = 0; it < 4 && pending; ++it) {
        const int leader = __ffsll((long long)pending) - 1;
        const int e0 = __shfl(e, leader, kWave);
        const unsigned long long grp = __ballot(act && e == e0) & pending;
        const int m = __popcll(grp);
        if (m < 2) break;  // no sharing: the rest add alone
        int base = 0;
        if (lane == leader) base = atomicAdd(&cnt[e0], m);
        base = __shfl(base, leader, kWave);
        if ((grp >> lane) & 1ull) rank = base + __popcll(grp & below);
        pending &= ~grp;
    }
    if ((pending >> lane) & 1ull) rank = atomicAdd(&cnt[e], 1);
    return rank;
}

// Many entries of few elements: the counters of a grouping are then added to by
// thousands of wavefronts each, one after the other (about 0.1 us per add to one
// counter: counting 100,000 points in random order on 64 elements took 150 us).
// Up to kFewMax elements (16 KB of LDS) blocks of a few thousand entries take their
// ranks in LDS, with one add per block and element that occurs.  findpts ranks its
// pairs so from kFewPoints points per element on (it costs a launch there, below
// which the adds cost less: 4096 elements, order 7, 100,000 points 258 -> 263 us,
// 1e6 points 1201 -> 1187), findpts_eval counts so whenever there are more points
// than elements.  Locate / interpolation of 3 fields, order 7, before -> after:
// 64 elements, 100,000 points 475 -> 287 us / 188 -> 41; 512 elements, 600,000
// points 1094 -> 906 / 203 -> 112 (staged before).
constexpr int kFewMax = 4096;
constexpr int kFewPoints = 64;
// Ranks of the candidate pairs of n points in their elements, cnt counted up:
// candidate k < (ncand[t] & mask) of point t is cand_el[k M + t].
hipError_t rank_few(const int *ncand, int mask, const int *cand_el, int *cand_pos, int *cnt, int n,
                    int M, int E, hipStream_t s);
// Ranks of n located points in their elements (-1 and not a number in each of the
// nf fields of out, stride apart, where a point was not found).
hipError_t count_few(const int *code, const int *el, int *pos, int *cnt, int n, int E, double *out,
                     long long stride, int nf, hipStream_t s);

// Exclusive scan of n ints: out[0..n], out[n] = total.  tmp needs
// scan_tmp_size(n) ints.  With gate non-null the kernels do nothing while
// *gate is zero (a pass with no work).
int scan_tmp_size(long long n);
hipError_t scan_exclusive(const int *in, int *out, int n, int *tmp,
                          hipStream_t s, const int *gate = nullptr);
// As scan_exclusive over the E counts of a grouping, and the list of its work
// units of at most K entries.
hipError_t scan_units(const int *cnt, int *off, UnitRec *units, int E, int K, int *tmp, hipStream_t s,
                      const int *gate = nullptr);
// The unit list of offsets that are already there.
hipError_t list_units(const int *off, UnitRec *units, int E, int K, int *tmp, hipStream_t s);

// GLL nodes and barycentric weights of order N; the inverse of the
// Bernstein-to-nodal matrix (n1 x n1, row-major), both computed on the host.
Basis make_basis(int N);
// Differentiation matrix at the nodes, D[a n1 + b] = h_b'(z_a), from the
// barycentric weights (off-diagonal (wb_b / wb_a) / (z_a - z_b), diagonal
// minus the row sum).
std::vector<double> node_derivatives(const Basis &b, int N);
std::vector<double> bernstein_to_nodal_inverse(int N, const double *z);

// Fill n ints with a value (a kernel, so that it may be graph-captured).
hipError_t fill_int(int *p, int value, long long n, hipStream_t s);

// Calls taken one wavefront per point, in one kernel, instead of being grouped
// by element (k_point, k_eval_point): decided by the call's points and fields, so
// that a call's results do not depend on how it is cut into passes.  The grouped
// path costs a call of 1,000 points 92 to 238 us of findpts at orders 3 to 9
// (about 15 launches and a chain of 16-slot rounds) against 30 to 52 us, and 250
// to 500 us at orders 12 and 15 against 83 to 232.  At 16,000 points on 125 or
// 2,048 elements it takes 110 to 235 us against 91 to 134 at orders 3 to 7, 270
// to 350 against 227 to 267 at orders 9 and 10, 443 to 566 against 496 to 547
// at order 12, but 533 to 851 against 866 to 875 at order 13 and 0.67 to 1.11
// ms against 1.21 to 1.31 at order 15, which is level near 6,000.
// Interpolation (of 2 fields): 27 to 28 us against 12 to 13 at 1,000 points; at
// 16,000 points 36 to 41 against 20 to 34 at order 9; level near 8,000 points
// at orders 10 to 12 and 4,000 above.  Mixed precision at the orders that
// interpolate in binary32 stays on its own kernels at every size.
inline bool point_path(const fp_handle *h)
{
    return !(h->precision == FP_PREC_MIXED && h->n1 <= kMixed32MaxN1);
}
inline bool small_call(const fp_handle *h, int npts)
{
    return point_path(h) && npts <= (h->n1 <= 13 ? kPointMax : 6144);
}
// A point's wavefront reads its element's nodes of every field, which grouped points
// share.  At orders up to 9, where the limit in points is the largest, the grouping is
// therefore taken once a call reads more than kEvalNodes node values, its elements
// have points to share (more than 3 each) and its units fill the chip.  Per point /
// grouped in us: order 7, 480 elements, 16,384 points of 4, 8 and 16 fields 25 / 29, 58 / 32
// and 115 / 49, 12,000 of 8 fields 45 / 33, 6,000 of 8 26 / 32; order 9, 16,384 of 16 fields
// 248 / 103; but 3,000 of 16 fields on 11,776 elements of order 8 49 / 119, 1,000 of 16
// fields on one element of order 9 28 / 93.
constexpr double kEvalNodes = 3e7;
inline bool small_eval(const fp_handle *h, int npts, int nfields)
{
    if (!point_path(h)) return false;
    if (h->n1 > 10) return npts <= (h->n1 <= 13 ? 8192 : 4096);
    const bool share = npts / 3 > h->E && h->E + npts / kUnitMin > 560;
    return npts <= kPointMax && !(share && (double)npts * nfields * h->V > kEvalNodes);
}

// findpts / findpts_eval on a given workspace and stream (the public calls
// pass the handle's own workspace; `timed` records the handle's events).
int run_findpts(fp_handle *h, const Work &w, int npts, const double *pts, const int *pt_session,
                int *code, int *el, double *rst, double *dist2, hipStream_t s, bool timed);
int run_eval(fp_handle *h, const Work &w, int npts, const int *code, const int *el,
             const double *rst, int nfields, const double *const *h_fields, double *out,
             hipStream_t s, bool timed);

}  // namespace fp
