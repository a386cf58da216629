// One wavefront working on one point: lane exchange through LDS, wave-wide sums
// and the tensor basis spread over the lanes (small calls and short second
// passes, where a pair's or point's latency counts).
#pragma once

#include "fp_mfma.h"

namespace fp {

// Order this wavefront's LDS accesses (its lanes exchange data through LDS).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    return mk64((unsigned)__builtin_amdgcn_readlane((int)lo32(v), lane),
                (unsigned)__builtin_amdgcn_readlane((int)hi32(v), lane));
}

template <int N>
__device__ __forceinline__ double row_ror(double v)  // the value N lanes on in the row of 16
{
    const int l = __builtin_amdgcn_update_dpp(0, (int)lo32(v), 0x120 + N, 0xf, 0xf, false);
    const int h = __builtin_amdgcn_update_dpp(0, (int)hi32(v), 0x120 + N, 0xf, 0xf, false);
    return mk64((unsigned)l, (unsigned)h);
}

// Sums over the 64 lanes of four values, in every lane (and wave-uniform).
__device__ __forceinline__ void wave_sum4(double &a, double &b, double &c, double &d)
{
#pragma clang fp contract(off)
    double x, y;
    swap2<32>(a, c, x, y);
    const double s = x + y;  // lanes 0..31: a, 32..63: c
    swap2<32>(b, d, x, y);
    const double t = x + y;
    swap2<16>(s, t, x, y);
    double u = x + y;  // rows of 16: a, b, c, d
    u = u + row_ror<8>(u);
    u = u + row_ror<4>(u);
    u = u + row_ror<2>(u);
    u = u + row_ror<1>(u);
    a = read_lane(u, 0);
    b = read_lane(u, 16);
    c = read_lane(u, 32);
    d = read_lane(u, 48);
}

// Minima over the 64 lanes of four values, in every lane (and wave-uniform).
__device__ __forceinline__ void wave_min4(double &a, double &b, double &c, double &d)
{
    double x, y;
    swap2<32>(a, c, x, y);
    const double s = fmin(x, y);
    swap2<32>(b, d, x, y);
    const double t = fmin(x, y);
    swap2<16>(s, t, x, y);
    double u = fmin(x, y);
    u = fmin(u, row_ror<8>(u));
    u = fmin(u, row_ror<4>(u));
    u = fmin(u, row_ror<2>(u));
    u = fmin(u, row_ror<1>(u));
    a = read_lane(u, 0);
    b = read_lane(u, 16);
    c = read_lane(u, 32);
    d = read_lane(u, 48);
}

// Lane l owns the node rows (j, k) = l, l + 64, ... of an element.
template <int N1>
struct WaveShape {
    static constexpr int V = N1 * N1 * N1;
    static constexpr int R = (N1 * N1 + kWave - 1) / kWave;  // node rows per lane
};

// The basis values of a point, evaluated once per wavefront (lane 16 a + i:
// index i of direction a, h_i and h_i' as running products over the other
// nodes) and shared through LDS.
template <int N1>
struct WaveBasis {
    using S = WaveShape<N1>;
    double zr[N1 > 1 ? N1 - 1 : 1], wb;  // the lane's index i: the other nodes, its weight
    double2 *sh;                         // LDS, 48 entries: (h_i, h_i') of direction a at 16 a + i
    int lane;

    __device__ __forceinline__ void init(BasisPtr<double> B, double2 *lds)
    {
        lane = (int)threadIdx.x & (kWave - 1);
        sh = lds;
        const int i = (lane & 15) < N1 ? (lane & 15) : 0;
#pragma unroll
        for (int p = 1; p < N1; ++p) zr[p - 1] = B.z((p + i) % N1);
        wb = B.wb(i);
    }

    __device__ __forceinline__ bool has_row(int q) const { return lane + kWave * q < N1 * N1; }
    __device__ __forceinline__ int first_node(int q) const
    {
        return has_row(q) ? (lane + kWave * q) * N1 : 0;
    }

    __device__ __forceinline__ void basis(const double (&r)[3])
    {
        const int a = lane >> 4;
        const double x = a == 0 ? r[0] : (a == 1 ? r[1] : r[2]);
        double p = 1.0, dp = 0.0;
#pragma unroll
        for (int m = 0; m < N1 - 1; ++m) {
            const double t = x - zr[m];
            dp = fma(dp, t, p);
            p = p * t;
        }
        wave_sync();  // the last readers are done
        if (a < 3) sh[lane] = make_double2(wb * p, wb * dp);
        wave_sync();
    }

    // The lane's part of Sum_ijk F_ijk h_i h_j h_k at the basis' point (F: the
    // element's nodes); the sum over the lanes is the value.  A lane past the
    // last row loads row 0, and its sum is dropped by a select: a field may hold
    // any value, and a weight of 0 would make NaN of an infinite one.
    __device__ __forceinline__ double field_part(const double *__restrict__ F) const
    {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < S::R; ++q) {
            const int row = lane + kWave * q;
            const bool in = row < N1 * N1;
            const double w = in ? sh[16 + row % N1].x * sh[32 + row / N1].x : 0.0;
            const double *Fr = F + first_node(q);
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < N1; ++i) s = fma(Fr[i], sh[i].x, s);
            v = fma(w, in ? s : 0.0, v);
        }
        return v;
    }
};

}  // namespace fp
