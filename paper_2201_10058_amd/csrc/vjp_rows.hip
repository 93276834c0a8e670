// Kick VJP of a small system by row groups (below SYM_MIN_N bodies): the
// gather form of csrc/vjp.hip in the shape of csrc/rows.h.  A block of 256
// threads owns VR_G rows and takes every column, so that it ends with the
// rows' adjoints and no sums pass through memory; the tiled form is a kernel of
// column slices, whose diagonal waves enter the rare path once per column for
// the self pair, and a reduction.  Pairs inside the critical radius are marked
// in an LDS bitmap and evaluated afterwards, as in the kick.
//
// Bound by the binary64 vector units and their latency: 36 instructions and one
// v_rsq_f64 per ordered pair are 15 us at 4,096 bodies, whose kernel takes 37 us,
// in 59 % of which the units work (54 instructions per pair with everything, 3
// waves to a SIMD).  Sums kept as
// factors (sum w abar_j, sum w m_j, sum c d) save three instructions per pair
// and need 32 more registers: 43 us.  Error against extended precision equal
// to the tiled form's.
#include "device_common.h"
#include "genga_internal.h"
#include "rows.h"
#include "sym_common.h"

namespace genga {

constexpr int VR_G = ROWS_G;   // rows of a block

struct VjpRowsDev {
    const double *x, *y, *z, *m, *rc;
    const double *abx, *aby, *abz;
    double scale, G;
    int n;
    genga_adjoint adj;
    int32_t *status;
    double c53, c75;
};

struct VjpRowsSmem {
    uint64_t bits[VR_G][ROWS_MAX / 64];
    double part[4][4 * VR_G];
    double slow[VR_G][5];
    double rc2[VR_G];
    double row[VR_G][8];   // x, y, z, m, rc, scaled abar of the rows
};

struct VjpColumn {
    double x, y, z, m, rc, ax, ay, az;
};

__device__ __forceinline__ VjpColumn vjp_load(const VjpRowsDev &a, int j)
{
    const uint32_t o = (uint32_t)(j < a.n ? j : a.n - 1) * 8u;
    auto at = [o](const double *p) { return *(const double *)((const char *)p + o); };
    return {at(a.x), at(a.y), at(a.z), at(a.m), at(a.rc), at(a.abx), at(a.aby), at(a.abz)};
}

__global__ __launch_bounds__(256) void k_vjp_rows(VjpRowsDev a)
{
    __shared__ VjpRowsSmem sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n, nw = (n + 63) >> 6, r0 = (int)blockIdx.x * VR_G;
    VjpColumn A = vjp_load(a, tid), B;
    // the adjoints that the block adds to, loaded ahead of the columns
    const bool last = tid < VR_G && r0 + tid < n;
    double old[5] = {};
    if (last) {
        const int i = r0 + tid;
        old[0] = a.adj.x[i];
        old[1] = a.adj.y[i];
        old[2] = a.adj.z[i];
        old[3] = a.adj.m[i];
        old[4] = a.adj.rc[i];
    }
    for (int q = 0; q < VR_G; ++q)
        for (int k = tid; k < nw; k += 256) sm.bits[q][k] = 0;
    const int vzero = (int)__builtin_amdgcn_mbcnt_lo(0u, 0u);
    const double c53 = a.c53 + (double)vzero, c75 = a.c75 + (double)vzero;
    const double sc15 = 1.5 * a.scale;
    double xi[VR_G], yi[VR_G], zi[VR_G], mi[VR_G], bx[VR_G], by[VR_G], bz[VR_G], rg = 0.0;
#pragma unroll
    for (int q = 0; q < VR_G; ++q) {
        const int i = r0 + q < n ? r0 + q : n - 1;
        const bool real = r0 + q < n;
        const double r = wave_uniform(a.rc[i]);
        xi[q] = wave_uniform(real ? a.x[i] : 1e18);
        yi[q] = wave_uniform(real ? a.y[i] : 1e18);
        zi[q] = wave_uniform(real ? a.z[i] : 1e18);
        mi[q] = wave_uniform(real ? a.m[i] : 0.0);
        bx[q] = wave_uniform(a.scale * a.abx[i]);
        by[q] = wave_uniform(a.scale * a.aby[i]);
        bz[q] = wave_uniform(a.scale * a.abz[i]);
        const double r2 = real ? r * r : 0.0;
        if (tid == 0) {
            sm.rc2[q] = r2;
            sm.row[q][0] = xi[q];
            sm.row[q][1] = yi[q];
            sm.row[q][2] = zi[q];
            sm.row[q][3] = mi[q];
            sm.row[q][4] = r;
            sm.row[q][5] = bx[q];
            sm.row[q][6] = by[q];
            sm.row[q][7] = bz[q];
        }
        rg = r2 > rg ? r2 : rg;
    }
    rg = wave_uniform(rg);
    // xbar = sum w u - 5 c d and sum w d.abar_j
    double X[VR_G][4] = {};
    int32_t bad = 0;
    __syncthreads();

    auto column = [&](int j0, VjpColumn v) {
        const int j = j0 + tid;
        if (r0 == 0 && !(v.rc >= 0.0 && v.rc < INFINITY)) bad |= ST_RCRIT;
        const bool real = j < n;
        const double Mj = real ? 1.5 * v.m : 0.0;
        const double ax = real ? sc15 * v.ax : 0.0, ay = real ? sc15 * v.ay : 0.0,
                     az = real ? sc15 * v.az : 0.0;
        const double rc2j = v.rc * v.rc;
        double dx[VR_G], dy[VR_G], dz[VR_G], r2[VR_G], near = INFINITY;
#pragma unroll
        for (int q = 0; q < VR_G; ++q) {
            dx[q] = v.x - xi[q];
            dy[q] = v.y - yi[q];
            dz[q] = v.z - zi[q];
            r2[q] = __builtin_fma(dz[q], dz[q], __builtin_fma(dy[q], dy[q], dx[q] * dx[q]));
            near = vmin_f64(near, r2[q]);
        }
        if (__any(near <= vmax_f64(rg, rc2j))) {
            const int word = (j0 >> 6) + w;
#pragma unroll
            for (int q = 0; q < VR_G; ++q) {
                const double rho2 = vmax_f64(sm.rc2[q], rc2j);
                if (!__any(r2[q] <= rho2)) continue;
                const bool same = r2[q] == 0.0;
                const bool inside = r2[q] < rho2 && !same && real;
                if (same && real && j != r0 + q) bad |= ST_NONFINITE;
                const uint64_t mask = __ballot(inside);
                if (mask && lane == 0) sm.bits[q][word] = mask;
                // (at this distance both weights below are exact zeros)
                if (inside || same || !real) r2[q] = 1e300;
            }
        }
#pragma unroll
        for (int q = 0; q < VR_G; ++q) {
            const double y = __builtin_amdgcn_rsq(r2[q]);
            const double y2 = y * y;
            const double p3 = __builtin_fma(-r2[q], y2, c53);
            const double p5 = __builtin_fma(-r2[q], y2, c75);
            const double y3 = y2 * y;
            const double wt = y3 * p3;
            const double da = __builtin_fma(dz[q], az, __builtin_fma(dy[q], ay, dx[q] * ax));
            // u = m_k abar_j - m_j abar_k
            const double ux = __builtin_fma(mi[q], ax, -(Mj * bx[q]));
            const double uy = __builtin_fma(mi[q], ay, -(Mj * by[q]));
            const double uz = __builtin_fma(mi[q], az, -(Mj * bz[q]));
            const double du = __builtin_fma(dz[q], uz, __builtin_fma(dy[q], uy, dx[q] * ux));
            const double cq = ((y3 * y2) * p5) * (-5.0 * du);
            X[q][0] = __builtin_fma(cq, dx[q], __builtin_fma(wt, ux, X[q][0]));
            X[q][1] = __builtin_fma(cq, dy[q], __builtin_fma(wt, uy, X[q][1]));
            X[q][2] = __builtin_fma(cq, dz[q], __builtin_fma(wt, uz, X[q][2]));
            X[q][3] = __builtin_fma(wt, da, X[q][3]);
        }
    };
    for (int j0 = 0; j0 < n; j0 += 512) {
        B = vjp_load(a, j0 + 256 + tid);
        column(j0, A);
        if (j0 + 256 >= n) break;
        A = vjp_load(a, j0 + 512 + tid);
        column(j0 + 256, B);
    }
    if (bad) atomicOr(a.status, bad);
    // 16 sums over the wave; row h of 16 lanes ends with row group member h's
    // four
    double u[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) u[k] = halve32(X[k >> 2][k & 3], X[2 + (k >> 2)][k & 3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double s = row16_sum(halve16(u[k], u[k + 4]));
        if ((lane & 15) == 0) sm.part[w][(lane >> 4) * 4 + k] = s;
    }
    __syncthreads();
    {
        // marked pairs of row w (in true units)
        const int i = r0 + w < n ? r0 + w : n - 1;
        const double *row = sm.row[w];
        const double X = row[0], Y = row[1], Z = row[2], mk = row[3], rck = row[4];
        const double kx = row[5], ky = row[6], kz = row[7];
        double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        bool seen = false;
        auto pair = [&](int j, const VjpColumn &v) {
            const double dx = v.x - X, dy = v.y - Y, dz = v.z - Z;
            const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
            const double jx = a.scale * v.ax, jy = a.scale * v.ay, jz = a.scale * v.az;
            const double yc = rsq_full(r2), irho = rsq_full(rho2_of(rck, v.rc));
            const double yc2 = yc * yc, yc3 = yc2 * yc;
            // K and K' (both by one reciprocal; the clamp gives their values outside
            // the band)
            double y = __builtin_fma((r2 * yc) * irho, 1.0 / 0.9, -1.0 / 9.0);
            y = vmin_f64(vmax_f64(y, 0.0), 1.0);
            const double yy = y * y, h = rcp_nr2(__builtin_fma(2.0, yy - y, 1.0));
            const double K = yy * h, Kp = (2.0 * (y - yy)) * (h * h);
            const double wk = K * yc3;
            // w_r / r = K' / (0.9 rho r^4) - 3 K / r^5
            const double wr_r = (Kp * (irho * (1.0 / 0.9))) * (yc2 * yc2) - (3.0 * K) * (yc3 * yc2);
            const double da = __builtin_fma(dz, jz, __builtin_fma(dy, jy, dx * jx));
            const double db = __builtin_fma(dz, kz, __builtin_fma(dy, ky, dx * kx));
            const double du = __builtin_fma(mk, da, -(v.m * db));
            const double c = wr_r * du;
            s[0] += __builtin_fma(c, dx, wk * __builtin_fma(mk, jx, -(v.m * kx)));
            s[1] += __builtin_fma(c, dy, wk * __builtin_fma(mk, jy, -(v.m * ky)));
            s[2] += __builtin_fma(c, dz, wk * __builtin_fma(mk, jz, -(v.m * kz)));
            s[3] = __builtin_fma(wk, da, s[3]);
            const bool owner = rck > v.rc || (rck == v.rc && i < j);
            if (owner && Kp != 0.0) s[4] += ((Kp * (irho * irho)) * (1.0 / 0.9)) * yc2 * du;
            seen = true;
        };
        crowded_words(sm.bits[w], nw, [&](int j) { return vjp_load(a, j); }, pair);
        for (int k = lane; k < nw; k += 64) {
            uint64_t b = sm.bits[w][k];
            if (__popcll(b) >= ROWS_CROWD) continue;
            while (b) {
                const int j = k * 64 + __ffsll((unsigned long long)b) - 1;
                b &= b - 1;
                pair(j, vjp_load(a, j));
            }
        }
        if (__any(seen)) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
                for (int k = 0; k < 5; ++k) s[k] += __shfl_xor(s[k], off);
        }
        if (lane == 0)
            for (int k = 0; k < 5; ++k) sm.slow[w][k] = s[k];
    }
    __syncthreads();
    if (last) {
        const int i = r0 + tid;
        double t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            t[k] = (((sm.part[0][4 * tid + k] + sm.part[1][4 * tid + k]) + sm.part[2][4 * tid + k]) +
                    sm.part[3][4 * tid + k]) +
                   sm.slow[tid][k];
        a.adj.x[i] = old[0] + a.G * t[0];
        a.adj.y[i] = old[1] + a.G * t[1];
        a.adj.z[i] = old[2] + a.G * t[2];
        a.adj.m[i] = old[3] - a.G * t[3];
        a.adj.rc[i] = old[4] + a.G * sm.slow[tid][4];
    }
}

hipError_t launch_kick_vjp_rows(const genga_bodies *b, double G, double scale, const double *abx,
                                const double *aby, const double *abz, const genga_adjoint *adj,
                                int32_t *status, hipStream_t s)
{
    VjpRowsDev a;
    a.x = b->x; a.y = b->y; a.z = b->z; a.m = b->m; a.rc = b->rc;
    a.abx = abx; a.aby = aby; a.abz = abz;
    a.scale = scale;
    a.G = G;
    a.n = (int)b->n;
    a.adj = *adj;
    a.status = status;
    a.c53 = 5.0 / 3.0;
    a.c75 = 7.0 / 5.0;
    hipLaunchKernelGGL(k_vjp_rows, dim3((unsigned)((b->n + VR_G - 1) / VR_G)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace genga
