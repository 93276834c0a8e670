// Device helpers of the symmetric (rotating-column) kernels: the kick and
// its adjoint.
#pragma once

#include "genga_internal.h"

namespace genga {

// Lane l receives lane (l + 1) mod 64's value.
__device__ __forceinline__ double rotate_down(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x134, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x134, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ float rotate_down(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x134, 0xF, 0xF, false));
}

// Tile of launch index t: group g and slice s (s = -1: an empty narrow slot of
// one of the last groups).
__host__ __device__ __forceinline__ void sym_tile(const SymShape &h, int64_t t, int64_t &g, int64_t &s)
{
    if (t < h.tfull) {
        // largest g with bf(g) <= t: root of e/2 g^2 - (nb0 + e/2) g + t = 0
        const double e = (double)(h.d / h.M), b = (double)h.nb0 + 0.5 * e;
        double r = b * b - 2.0 * e * (double)t;
        r = r > 0.0 ? r : 0.0;
        int64_t gg = (int64_t)((b - __builtin_sqrt(r)) / e);
        gg = gg < 0 ? 0 : (gg > h.gl - 1 ? h.gl - 1 : gg);
        while (gg > 0 && h.bf(gg) > t) --gg;
        while (gg < h.gl - 1 && h.bf(gg + 1) <= t) ++gg;
        g = gg;
        s = h.A + (t - h.bf(gg));
        return;
    }
    const int64_t u = t - h.tfull;
    g = u % h.G;
    s = h.A - 1 - u / h.G;
    if (s >= h.ns(g)) s = -1;
}

// Group of storage tile sid: largest g with tb(g) <= sid.
__host__ __device__ __forceinline__ int64_t sym_group_of(const SymShape &h, int64_t sid)
{
    int64_t g;
    if (sid < h.tb(h.gl)) {
        const double e = (double)(h.d / h.M), b = (double)(h.A + h.nb0) + 0.5 * e;
        double r = b * b - 2.0 * e * (double)sid;
        r = r > 0.0 ? r : 0.0;
        g = (int64_t)((b - __builtin_sqrt(r)) / e);
    } else {
        g = h.gl;   // (at most A / d more groups)
    }
    g = g < 0 ? 0 : (g > h.G - 1 ? h.G - 1 : g);
    while (g > 0 && h.tb(g) > sid) --g;
    while (g < h.G - 1 && h.tb(g + 1) <= sid) ++g;
    return g;
}

// 1/sqrt(v) from v_rsq_f64 with one Newton correction (relative error below
// 5e-15).
__device__ __forceinline__ double rsq_nr(double v)
{
    const double y = __builtin_amdgcn_rsq(v);
    const double e = __builtin_fma(-v, y * y, 1.0);
    return __builtin_fma(y * e, 0.5, y);
}

// 1/v from v_rcp_f64 and two Newton steps.
__device__ __forceinline__ double rcp_nr2(double v)
{
    double t = __builtin_amdgcn_rcp(v);
    t = __builtin_fma(t, __builtin_fma(-v, t, 1.0), t);
    return __builtin_fma(t, __builtin_fma(-v, t, 1.0), t);
}

}  // namespace genga
