// Sums across a wavefront without LDS traffic (DPP and the gfx950 lane swaps).
//
// A ds_bpermute shuffle costs an LDS round trip per step; the steps here are
// plain VALU moves: exchanges inside a row of 16 lanes by DPP (quad
// permutations 1 and 2 lanes apart, then the mirrored half row and row, whose
// halves hold equal sums by then), and between rows by v_permlane16_swap /
// v_permlane32_swap.
#pragma once

#include <hip/hip_runtime.h>

#include "mp.h"

namespace zk {

template <int CTRL>
__device__ __forceinline__ double dpp_get(double x)
{
    const int lo = __double2loint(x), hi = __double2hiint(x);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xF, 0xF, true));
}

// (a, b) -> a = [a lanes 0..31 | b lanes 0..31], b = [a lanes 32..63 | b lanes 32..63]
__device__ __forceinline__ void lane_swap32(double &a, double &b)
{
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}
// the same between the rows 2 r and 2 r + 1 of 16 lanes: odd rows of a <-> even rows of b
__device__ __forceinline__ void lane_swap16(double &a, double &b)
{
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}

template <int CTRL>
__device__ __forceinline__ int dpp_get_i(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}

// largest (smallest) value of the wave, in every lane; no NaN
__device__ __forceinline__ double wave_max_all(double x)
{
    x = fmax(x, dpp_get<0xB1>(x));
    x = fmax(x, dpp_get<0x4E>(x));
    x = fmax(x, dpp_get<0x141>(x));
    x = fmax(x, dpp_get<0x140>(x));
    double y = x;
    lane_swap16(x, y);
    x = fmax(x, y);
    y = x;
    lane_swap32(x, y);
    return fmax(x, y);
}
__device__ __forceinline__ int wave_min_all(int x)
{
    x = min(x, dpp_get_i<0xB1>(x));
    x = min(x, dpp_get_i<0x4E>(x));
    x = min(x, dpp_get_i<0x141>(x));
    x = min(x, dpp_get_i<0x140>(x));
    auto p = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    x = min((int)p[0], (int)p[1]);
    p = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    return min((int)p[0], (int)p[1]);
}

// sum over each row of 16 lanes, in every lane of the row
__device__ __forceinline__ double row_sum(double x)
{
    x += dpp_get<0xB1>(x);    // quad_perm [1,0,3,2]
    x += dpp_get<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp_get<0x141>(x);   // row_half_mirror
    x += dpp_get<0x140>(x);   // row_mirror
    return x;
}

// sum over the wave, in every lane
__device__ __forceinline__ double wave_sum_all(double x)
{
    x = row_sum(x);
    double y = x;
    lane_swap16(x, y);
    x += y;
    y = x;
    lane_swap32(x, y);
    return x + y;
}

// Sums of N values (a power of two) over the wave at once: every exchange
// between rows halves the number of values per lane, so N sums cost about
// 3 N instructions instead of 18 N.  Afterwards x[q], q < wave_reduce_regs(N),
// holds in every lane of row r (16 lanes) the sum of the value
// wave_reduce_index<N>(q, r).
__host__ __device__ constexpr int wave_reduce_regs(int N) { return N >= 4 ? N / 4 : 1; }
template <int N>
__device__ __forceinline__ int wave_reduce_index(int q, int row)
{
    return N >= 4 ? q + (row & 1) * (N / 4) + (row >> 1) * (N / 2) : (N == 2 ? row >> 1 : 0);
}
template <int N>
__device__ __forceinline__ void wave_reduce_rows(double (&x)[N])
{
    static_assert(N >= 2 && (N & (N - 1)) == 0, "a power of two");
#pragma unroll
    for (int i = 0; i < N / 2; i++) {
        lane_swap32(x[i], x[i + N / 2]);
        x[i] += x[i + N / 2];
    }
    if (N >= 4) {
#pragma unroll
        for (int i = 0; i < N / 4; i++) {
            lane_swap16(x[i], x[i + N / 4]);
            x[i] += x[i + N / 4];
        }
    } else {
        double y = x[0];
        lane_swap16(x[0], y);
        x[0] += y;
    }
#pragma unroll
    for (int i = 0; i < wave_reduce_regs(N); i++) x[i] = row_sum(x[i]);
}

// value i of N after wave_reduce_rows, uniform
template <int N>
__device__ __forceinline__ double wave_reduce_get(const double (&x)[N], int i)
{
    constexpr int H = N / 2, Q = N >= 4 ? N / 4 : 1;
    const int row = N >= 4 ? 2 * (i / H) + (i % H) / Q : 2 * i;
    const double v = x[N >= 4 ? i % Q : 0];
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 16 * row),
                            __builtin_amdgcn_readlane(__double2loint(v), 16 * row));
}

// (s, e), a sum and its rounding errors, over the wave: leading parts added
// without error (two_sum), the rest rounded; in every lane
template <int CTRL>
__device__ __forceinline__ void acc2_dpp(double &s, double &e)
{
    const double h = dpp_get<CTRL>(s), l = dpp_get<CTRL>(e);
    double t, err;
    two_sum(s, h, t, err);
    s = t;
    e = (e + l) + err;
}
__device__ __forceinline__ void wave_sum_acc2(double &s, double &e)
{
    acc2_dpp<0xB1>(s, e);
    acc2_dpp<0x4E>(s, e);
    acc2_dpp<0x141>(s, e);
    acc2_dpp<0x140>(s, e);
    double h = s, l = e, t, err;
    lane_swap16(s, h);
    lane_swap16(e, l);
    two_sum(s, h, t, err);
    s = t;
    e = (e + l) + err;
    h = s;
    l = e;
    lane_swap32(s, h);
    lane_swap32(e, l);
    two_sum(s, h, t, err);
    s = t;
    e = (e + l) + err;
}

// (s, e, f), a sum in three parts, over the wave: the first two added without
// error, so that a double-double sum is rounded once at its end and not at
// every step
__device__ __forceinline__ void acc3(double &s, double &e, double &f, double h, double l, double m)
{
    double t, err, u, v;
    two_sum(s, h, t, err);
    s = t;
    two_sum(e, l, t, u);
    two_sum(t, err, e, v);
    f += m + (u + v);
}
template <int CTRL>
__device__ __forceinline__ void acc3_dpp(double &s, double &e, double &f)
{
    acc3(s, e, f, dpp_get<CTRL>(s), dpp_get<CTRL>(e), dpp_get<CTRL>(f));
}
__device__ __forceinline__ void wave_sum_acc3(double &s, double &e, double &f)
{
    acc3_dpp<0xB1>(s, e, f);
    acc3_dpp<0x4E>(s, e, f);
    acc3_dpp<0x141>(s, e, f);
    acc3_dpp<0x140>(s, e, f);
    double h = s, l = e, m = f;
    lane_swap16(s, h);
    lane_swap16(e, l);
    lane_swap16(f, m);
    acc3(s, e, f, h, l, m);
    h = s;
    l = e;
    m = f;
    lane_swap32(s, h);
    lane_swap32(e, l);
    lane_swap32(f, m);
    acc3(s, e, f, h, l, m);
}

}  // namespace zk
