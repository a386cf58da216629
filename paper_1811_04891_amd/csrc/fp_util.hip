// Device utilities: exclusive prefix sum, fill, copy, error state.
#include <cstdio>
#include <string>

#include "fp_internal.h"

namespace fp {

static thread_local std::string g_err;

void set_error(const std::string &msg) { g_err = msg; }

int hip_fail(hipError_t e, const char *what)
{
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    if (e == hipErrorOutOfMemory) return FP_ENOMEM;
    return FP_EHIP;
}

// ---------------------------------------------------------------------------
// Exclusive scans, tiles of 256 threads x 4 items (16 in lists of more than 2^20,
// whose tile sums would be many): one launch for one tile, else the tile sums, then
// each block adds up the sums before its own and scans its tile.  A pass groups its
// pairs and its points with these, in a chain where a launch costs 4 to 5 us
// whatever it does: the 16384 elements of the annulus took 15 us in three launches
// (the sums scanned by one of their own), and take 9.  Measured against: one launch
// where each block adds up all items before its tile (25 us), and one block for all
// of them (50 us: its stores go through one CU).
//
// Groupings also get their work units: the sums then carry the entries in the
// low and the units in the high 32 bits.
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int scan_items(long long n) { return n > (1 << 20) ? 16 : 4; }
typedef unsigned long long u64;

// Block-wide exclusive scan of one value per thread; returns the thread's
// exclusive prefix and writes the block total.
template <class T>
__device__ __forceinline__ T block_excl_scan(T v, T *total)
{
    __shared__ T wsum[kScanThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    T inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const T t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    T off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kScanThreads / kWave; ++i) {
        if (i < w) off += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// What is scanned: counts (kCounts: offsets only; kGroup: offsets and units),
// or the differences of offsets that are there (kOffsets: units).
enum ScanMode { kCounts, kGroup, kOffsets };

struct ScanArgs {
    const int *in;  // counts or offsets
    int n, K;
    u64 *tsum;
    int *out;
    UnitRec *units;
    const int *gate;
};

template <ScanMode MODE>
__device__ __forceinline__ u64 scan_value(int cnt, int K)
{
    if constexpr (MODE == kCounts) return (u64)(unsigned)cnt;
    u64 nu = cnt > 0 ? 1u : 0u;
    if (cnt > K) nu = (u64)((cnt - 1) / unit_size(cnt, K) + 1);
    return (u64)(unsigned)cnt | (nu << 32);
}

// The thread's consecutive counts from item i0 (zero past the last).
template <ScanMode MODE, int ITEMS>
__device__ __forceinline__ void scan_load(const ScanArgs &a, long long i0, int (&v)[ITEMS])
{
    constexpr int L = MODE == kOffsets ? ITEMS + 1 : ITEMS;
    const long long m = MODE == kOffsets ? (long long)a.n : (long long)a.n - 1;
    int w[L];
#pragma unroll
    for (int k = 0; k < L; ++k) w[k] = a.in[i0 + k < m ? i0 + k : m];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        v[k] = i0 + k >= a.n ? 0 : (MODE == kOffsets ? w[(k + 1) % L] - w[k] : w[k]);
}

template <ScanMode MODE, int ITEMS>
__device__ __forceinline__ u64 scan_sum(const ScanArgs &a, long long i0)
{
    int v[ITEMS];
    scan_load<MODE, ITEMS>(a, i0, v);
    u64 s = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) s += scan_value<MODE>(v[k], a.K);
    return s;
}

template <ScanMode MODE, int ITEMS>
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(ScanArgs a)
{
    if (a.gate && !*a.gate) return;
    u64 tot;
    block_excl_scan(scan_sum<MODE, ITEMS>(a, (long long)blockIdx.x * (kScanThreads * ITEMS) + threadIdx.x * ITEMS),
                    &tot);
    if (threadIdx.x == 0) a.tsum[blockIdx.x] = tot;
}

template <ScanMode MODE, int ITEMS>
__global__ __launch_bounds__(kScanThreads) void k_scan(ScanArgs a)
{
    if (a.gate && !*a.gate) return;
    const long long i0 = (long long)blockIdx.x * (kScanThreads * ITEMS) + threadIdx.x * ITEMS;
    int v[ITEMS];
    scan_load<MODE, ITEMS>(a, i0, v);
    u64 s = 0, tot, run = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kScanThreads) s += a.tsum[t];
    if (blockIdx.x > 0) block_excl_scan(s, &run);
    s = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) s += scan_value<MODE>(v[k], a.K);
    const u64 before = block_excl_scan(s, &tot);
    const u64 all = run + tot;
    run += before;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const long long i = i0 + k;
        const int beg = (int)(unsigned)run;
        if (MODE != kOffsets && i < a.n) a.out[i] = beg;
        const u64 add = scan_value<MODE>(v[k], a.K);
        if constexpr (MODE != kCounts) {
            // a crowded element's records are written by the whole wavefront
            constexpr int kOwn = 4;
            const int r = 1 + (int)(run >> 32), nu = (int)(add >> 32);
            const int size = nu > 1 ? unit_size(v[k], a.K) : v[k];
            if (nu <= kOwn)
                for (int j = 0; j < nu; ++j) a.units[r + j] = UnitRec{beg + j * size, (int)i};
            u64 big = __ballot(nu > kOwn);
            while (big) {
                const int src = __ffsll((long long)big) - 1;
                big &= big - 1;
                const int bn = __shfl(nu, src, kWave), bs = __shfl(size, src, kWave);
                const int bb = __shfl(beg, src, kWave), bi = __shfl((int)i, src, kWave);
                const int br = __shfl(r, src, kWave);
                for (int j = threadIdx.x & (kWave - 1); j < bn; j += kWave)
                    a.units[br + j] = UnitRec{bb + j * bs, bi};
            }
        }
        run += add;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const int nu = (int)(all >> 32), ne = (int)(unsigned)all;
        if (MODE != kOffsets) a.out[a.n] = ne;
        if constexpr (MODE != kCounts) {
            a.units[0] = UnitRec{nu, ne};
            a.units[1 + nu] = UnitRec{ne, a.n};
        }
    }
}

static int scan_tiles(long long n)
{
    const int tile = kScanThreads * scan_items(n);
    return (int)((n + tile - 1) / tile);
}

// Ints of the tile sums of a scan of at most n items (a list of 2^20 has as many
// tiles as one four times as long).
int scan_tmp_size(long long n)
{
    const int small = scan_tiles(n < (1 << 20) ? n : (1 << 20)), own = scan_tiles(n);
    return 2 * (small > own ? small : own) + 2;
}

__global__ void k_zero_total(int *out, int n) { out[n] = 0; }

template <ScanMode MODE>
static hipError_t launch_scan(ScanArgs a, int *tmp, hipStream_t s)
{
    const int nt = scan_tiles(a.n);
    a.tsum = (u64 *)tmp;
    if (scan_items(a.n) == 4) {
        if (nt > 1) k_scan_tiles<MODE, 4><<<nt, kScanThreads, 0, s>>>(a);
        k_scan<MODE, 4><<<nt, kScanThreads, 0, s>>>(a);
    } else {
        k_scan_tiles<MODE, 16><<<nt, kScanThreads, 0, s>>>(a);
        k_scan<MODE, 16><<<nt, kScanThreads, 0, s>>>(a);
    }
    return hipGetLastError();
}

hipError_t scan_exclusive(const int *in, int *out, int n, int *tmp, hipStream_t s,
                          const int *gate)
{
    if (n <= 0) {
        k_zero_total<<<1, 1, 0, s>>>(out, 0);
        return hipGetLastError();
    }
    return launch_scan<kCounts>(ScanArgs{in, n, 1, nullptr, out, nullptr, gate},
                                tmp, s);
}

hipError_t scan_units(const int *cnt, int *off, UnitRec *units, int E, int K, int *tmp, hipStream_t s,
                      const int *gate)
{
    return launch_scan<kGroup>(ScanArgs{cnt, E, K, nullptr, off, units, gate}, tmp, s);
}

hipError_t list_units(const int *off, UnitRec *units, int E, int K, int *tmp, hipStream_t s)
{
    return launch_scan<kOffsets>(
        ScanArgs{off, E, K, nullptr, nullptr, units, nullptr}, tmp, s);
}

constexpr int kFewThreads = 1024;

// Entries per block of few-element ranks.
static int few_chunk(int n)
{
    const int c = n / 256 / kFewThreads * kFewThreads;
    return c < kFewThreads ? kFewThreads : (c > 8 * kFewThreads ? 8 * kFewThreads : c);
}

// The block's entries counted in c: from here on c[e] is their base in element e.
__device__ __forceinline__ void few_bases(int *c, int *__restrict__ cnt, int E)
{
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kFewThreads)
        if (c[e]) c[e] = atomicAdd(&cnt[e], c[e]);
    __syncthreads();
}

__global__ __launch_bounds__(kFewThreads) void k_rank_few(const int *__restrict__ ncand, int mask,
                                                          const int *__restrict__ cand_el,
                                                          int *cand_pos, int *__restrict__ cnt,
                                                          int npts, int M, int E, int chunk)
{
    __shared__ int c[kFewMax];
    for (int e = threadIdx.x; e < E; e += kFewThreads) c[e] = 0;
    __syncthreads();
    const int beg = blockIdx.x * chunk, end = min(beg + chunk, npts);
    for (int t = beg + (int)threadIdx.x; t < end; t += kFewThreads) {
        const int n = ncand[t] & mask;
        for (int k = 0; k < n; ++k) {
            const long long s = (long long)k * M + t;
            cand_pos[s] = atomicAdd(&c[cand_el[s]], 1);
        }
    }
    few_bases(c, cnt, E);
    for (int t = beg + (int)threadIdx.x; t < end; t += kFewThreads) {
        const int n = ncand[t] & mask;
        for (int k = 0; k < n; ++k) {
            const long long s = (long long)k * M + t;
            cand_pos[s] += c[cand_el[s]];
        }
    }
}

__global__ __launch_bounds__(kFewThreads) void k_count_few(const int *__restrict__ code,
                                                           const int *__restrict__ el, int *pos,
                                                           int *__restrict__ cnt, int n, int E,
                                                           double *__restrict__ out,
                                                           long long stride, int nf, int chunk)
{
    __shared__ int c[kFewMax];
    for (int e = threadIdx.x; e < E; e += kFewThreads) c[e] = 0;
    __syncthreads();
    const int beg = blockIdx.x * chunk, end = min(beg + chunk, n);
    const auto key = [&](int p) {
        const int e = el[p];
        return code[p] != FP_NOT_FOUND && e >= 0 && e < E ? e : -1;
    };
    for (int p = beg + (int)threadIdx.x; p < end; p += kFewThreads) {
        const int e = key(p);
        pos[p] = e < 0 ? -1 : atomicAdd(&c[e], 1);
        if (e < 0)
            for (int f = 0; f < nf; ++f) out[f * stride + p] = NAN;
    }
    few_bases(c, cnt, E);
    for (int p = beg + (int)threadIdx.x; p < end; p += kFewThreads) {
        const int e = key(p);
        if (e >= 0) pos[p] += c[e];
    }
}

hipError_t rank_few(const int *ncand, int mask, const int *cand_el, int *cand_pos, int *cnt, int n,
                    int M, int E, hipStream_t s)
{
    const int chunk = few_chunk(n);
    k_rank_few<<<(n + chunk - 1) / chunk, kFewThreads, 0, s>>>(ncand, mask, cand_el, cand_pos, cnt,
                                                               n, M, E, chunk);
    return hipGetLastError();
}

hipError_t count_few(const int *code, const int *el, int *pos, int *cnt, int n, int E, double *out,
                     long long stride, int nf, hipStream_t s)
{
    const int chunk = few_chunk(n);
    k_count_few<<<(n + chunk - 1) / chunk, kFewThreads, 0, s>>>(code, el, pos, cnt, n, E, out,
                                                                stride, nf, chunk);
    return hipGetLastError();
}

__global__ void k_fill_int(int *__restrict__ p, int v, long long n)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

hipError_t fill_int(int *p, int value, long long n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    k_fill_int<<<(int)blocks, 256, 0, s>>>(p, value, n);
    return hipGetLastError();
}

// Plain streaming copy, 16 bytes per lane per iteration (grid-stride).
__global__ __launch_bounds__(256) void k_copy16(const uint4 *__restrict__ a,
                                               uint4 *__restrict__ b, long long n)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride) b[i] = a[i];
}

}  // namespace fp

extern "C" const char *fp_last_error(void) { return fp::g_err.c_str(); }

extern "C" int fp_copy(const void *src, void *dst, size_t bytes, void *stream)
{
    if (!src || !dst || (bytes & 15) || (((uintptr_t)src | (uintptr_t)dst) & 15)) {
        fp::set_error("fp_copy: pointers must be 16-byte aligned and bytes a multiple of 16");
        return FP_EINVAL;
    }
    long long n = (long long)(bytes / 16);
    if (n == 0) return FP_OK;
    long long blocks = (n + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    fp::k_copy16<<<(int)blocks, 256, 0, (hipStream_t)stream>>>(
        (const uint4 *)src, (uint4 *)dst, n);
    FP_HIP(hipGetLastError());
    return FP_OK;
}
