// Binary64 kick with few massive bodies among test particles (GENGA II Sect. 8,
// test-particle modes 1 and 2) and the base step on it.
//
// Work and traffic of such a kick are small (16 massive bodies and 65,520 test
// particles: a million pairs, 5 MB), so launches and latency bound it.  The tiled
// kick takes the massive rows and the test particles' rows as two classes of
// tiles; its massive rows fill 16 of 256 lanes of 1,024 blocks, whose sums two
// more kernels add.  Here every pair of a massive body and a test particle is
// evaluated once, by the test particle's thread, for both of them: the thread
// ends with its particle's acceleration and applies everything that is due to
// it (critical radius before, Sun kick after), and a block sums what its 256
// particles give to the massive bodies, four of these at a time by wave
// halvings.  One block per massive body adds the blocks' sums in order, and
// the massive bodies' own pairs.  Pairs inside the critical radius set a bit
// in the massive body's bitmap, whose rows are the encounter list in
// canonical order, written while the bodies drift.  Step of 65,536 bodies, 16
// (64) massive: 37 (53) instead of 80 (95) us, 5 launches instead of 11;
// 4,096 bodies, 8 massive: 28 instead of 57.
#include "device_common.h"
#include "genga_internal.h"
#include "kepler.h"
#include "rows.h"

namespace genga {

struct TpDev {
    double *x, *y, *z, *vx, *vy, *vz;   // positions written with hc_part only
    const double *m;
    double *rc;                         // written with rcrit
    int n, nm, nw;                      // bodies, massive ones, bitmap words per row
    int back;                           // test particles act on the massive bodies (mode 2)
    int rcrit;                          // critical radii first
    double m_star, dt, n1, n2;
    double G, h;                        // v += h a (h = 0: not)
    double *ax, *ay, *az;               // optional
    double *mom;                        // optional: [blocks][3] sums of m v (block 0 incomplete)
    double *q0;                         // with mom: [3][256] m v of the first 256 bodies
    const double *hc_part;              // optional: x += hc_h P / m_star after the velocities
    int hc_nb;
    double hc_h;
    double *xm;                         // [3][TP_MAX] the massive bodies' drifted positions: the
                                        // second kick writes the state's as it shifts them
    double *part;                       // [blocks][nm][3] what the blocks give to the massive bodies
    int emit;
    uint64_t *bits;                     // [nm][nw]
    int32_t *cnt;                       // [nm] pairs of the massive body with a higher index
    int32_t *status;
    double c53;
};

// K(r; rho) of a pair inside rho.
__device__ __forceinline__ double tp_changeover(double r2, double rho2)
{
    const double y = rsq_full(r2), irho = rsq_full(rho2);
    return changeover_of_y(__builtin_fma((r2 * y) * irho, 1.0 / 0.9, -1.0 / 9.0));
}

__device__ __forceinline__ void tp_sum3(double (*sm)[RB], double P[3])
{
    const int t = threadIdx.x;
    __syncthreads();
    for (int h = RB / 2; h > 0; h >>= 1) {
        if (t < h) {
            sm[0][t] += sm[0][t + h];
            sm[1][t] += sm[1][t + h];
            sm[2][t] += sm[2][t + h];
        }
        __syncthreads();
    }
    P[0] = sm[0][0];
    P[1] = sm[1][0];
    P[2] = sm[2][0];
    __syncthreads();
}

// P from nb block sums, in the fixed order of k_hc_apply.
__device__ __forceinline__ void tp_momentum(const double *part, int nb, double (*sm)[RB], double P[3])
{
    double p[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nb; b += RB)
        for (int c = 0; c < 3; ++c) p[c] += part[(size_t)b * 3 + c];
    for (int c = 0; c < 3; ++c) sm[c][threadIdx.x] = p[c];
    tp_sum3(sm, P);
}

struct TpSmem {
    double4 xyzm[TP_MAX];            // massive bodies: position, 3/2 m
    double rc2[TP_MAX];
    double part[4][TP_MAX][3];
    double red[3][RB];
};

// One thread per body; those of the massive bodies only take part in the sums.
__global__ __launch_bounds__(RB) void k_tp_kick(TpDev a)
{
    __shared__ TpSmem sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = (int)blockIdx.x * RB + tid;
    const bool test = i >= a.nm && i < a.n;
    double P[3] = {0.0, 0.0, 0.0};
    double X = -1e18, Y = -1e18, Z = -1e18, V[3] = {0.0, 0.0, 0.0}, mi = 0.0, rci = 0.0;
    const bool vel = a.rcrit || a.mom || a.h != 0.0;
    if (test) {
        X = a.x[i]; Y = a.y[i]; Z = a.z[i];
        mi = a.m[i];
        if (vel) {
            V[0] = a.vx[i]; V[1] = a.vy[i]; V[2] = a.vz[i];
        }
        if (!a.rcrit) rci = a.rc[i];
    }
    const int pad = (a.nm + 3) & ~3;
    if (tid < pad) {
        double4 q = make_double4(1e18, 1e18, 1e18, 0.0);
        double r = 0.0;
        if (tid < a.nm) {
            const double mm = a.m[tid];
            q = make_double4(a.x[tid], a.y[tid], a.z[tid], 1.5 * mm);
            if (a.rcrit) {
                r = rcrit_of(q.x, q.y, q.z, a.vx[tid], a.vy[tid], a.vz[tid], mm, a.m_star, a.dt,
                             a.n1, a.n2);
                if (blockIdx.x == 0) a.rc[tid] = r;
            } else {
                r = a.rc[tid];
            }
            if (!(r >= 0.0 && r < INFINITY)) atomicOr(a.status, ST_RCRIT);
        }
        sm.xyzm[tid] = q;
        sm.rc2[tid] = r * r;
    }
    if (test) {
        if (a.rcrit) {
            rci = rcrit_of(X, Y, Z, V[0], V[1], V[2], mi, a.m_star, a.dt, a.n1, a.n2);
            a.rc[i] = rci;
        }
        if (!(rci >= 0.0 && rci < INFINITY)) atomicOr(a.status, ST_RCRIT);
    }
    if (a.hc_part) tp_momentum(a.hc_part, a.hc_nb, sm.red, P);   // (ends with a barrier)
    else __syncthreads();

    const double c53 = a.c53 + (double)(int)__builtin_amdgcn_mbcnt_lo(0u, 0u);
    const double rc2i = rci * rci, m15 = 1.5 * mi;
    double ax = 0.0, ay = 0.0, az = 0.0;
    uint64_t mine = 0;   // lane l: the wave's bits of massive body l
    for (int q0 = 0; q0 < pad; q0 += 4) {
        double f[12];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double4 b = sm.xyzm[q0 + u];
            const double rc2b = sm.rc2[q0 + u];
            const double dx = b.x - X, dy = b.y - Y, dz = b.z - Z;
            const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
            // r^-3 = (3/2) y^3 (5/3 - r^2 y^2) to first order, as in the other kicks
            const double y = __builtin_amdgcn_rsq(r2);
            const double y2 = y * y;
            double s = (y2 * y) * __builtin_fma(-r2, y2, c53);
            if (__any(r2 <= vmax_f64(rc2i, rc2b))) {
                const double rho2 = rc2i > rc2b ? rc2i : rc2b;
                const bool same = test && r2 == 0.0;
                const bool inside = test && r2 < rho2 && !same && q0 + u < a.nm;
                if (same) {
                    atomicOr(a.status, ST_NONFINITE);
                    s = 0.0;
                }
                if (inside) s *= tp_changeover(r2, rho2);
                const uint64_t mask = __ballot(inside);
                if (lane == q0 + u) mine = mask;
            }
            const double si = s * b.w, sj = s * m15;
            ax = __builtin_fma(dx, si, ax);
            ay = __builtin_fma(dy, si, ay);
            az = __builtin_fma(dz, si, az);
            f[3 * u + 0] = -dx * sj;
            f[3 * u + 1] = -dy * sj;
            f[3 * u + 2] = -dz * sj;
        }
        if (a.back) {
            // 12 sums over the wave; row h of 16 lanes ends with body q0 + h's
            double v[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] = halve32(f[k], f[k + 6]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double t = row16_sum(halve16(v[k], v[k + 3]));
                if ((lane & 15) == 0) sm.part[w][q0 + (lane >> 4)][k] = t;
            }
        }
    }
    const int word = (int)blockIdx.x * (RB / 64) + w;
    if (a.emit && lane < a.nm && word < a.nw) a.bits[(size_t)lane * a.nw + word] = mine;
    double p[3] = {0.0, 0.0, 0.0};
    if (test) {
        const double A[3] = {ax * a.G, ay * a.G, az * a.G};
        if (!(isfinite(A[0]) && isfinite(A[1]) && isfinite(A[2]))) atomicOr(a.status, ST_NONFINITE);
        if (a.h != 0.0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) V[k] = __builtin_fma(a.h, A[k], V[k]);
            a.vx[i] = V[0];
            a.vy[i] = V[1];
            a.vz[i] = V[2];
        }
        if (a.ax) {
            a.ax[i] = A[0];
            a.ay[i] = A[1];
            a.az[i] = A[2];
        }
        if (a.hc_part) {
            a.x[i] = X + (a.hc_h * P[0]) / a.m_star;
            a.y[i] = Y + (a.hc_h * P[1]) / a.m_star;
            a.z[i] = Z + (a.hc_h * P[2]) / a.m_star;
        }
        if (a.back)
            for (int k = 0; k < 3; ++k) p[k] = mi * V[k];
    }
    __syncthreads();
    if (a.back) {
        for (int e = tid; e < 3 * a.nm; e += RB) {
            const int q = e / 3, k = e % 3;
            a.part[((size_t)blockIdx.x * a.nm + q) * 3 + k] =
                ((sm.part[0][q][k] + sm.part[1][q][k]) + sm.part[2][q][k]) + sm.part[3][q][k];
        }
    }
    if (a.mom) {
        // (the massive bodies' velocities are not final yet: k_tp_massive
        // completes the first 256 bodies' values, k_tp_drift sums them)
        if (i >= a.nm && i < RB)
            for (int k = 0; k < 3; ++k) a.q0[k * RB + i] = p[k];
        for (int k = 0; k < 3; ++k) sm.red[k][tid] = p[k];
        tp_sum3(sm.red, p);
        if (tid < 3) a.mom[(size_t)blockIdx.x * 3 + tid] = p[tid];
    }
}

// One block per massive body: the blocks' sums in order (mode 2), the massive
// bodies' pairs, and the number of its pairs with higher indices.
__global__ __launch_bounds__(RB) void k_tp_massive(TpDev a, int nb)
{
    __shared__ double sm[3][RB];
    __shared__ int64_t sc[RB / 64];
    const int tid = threadIdx.x, i = (int)blockIdx.x;
    double P[3] = {0.0, 0.0, 0.0};
    if (a.hc_part) tp_momentum(a.hc_part, a.hc_nb, sm, P);
    double f[3] = {0.0, 0.0, 0.0};
    if (a.back)
        for (int b = tid; b < nb; b += RB)
            for (int k = 0; k < 3; ++k) f[k] += a.part[((size_t)b * a.nm + i) * 3 + k];
    const double *x = a.x, *y = a.y, *z = a.z;
    if (a.hc_part) {
        x = a.xm;
        y = a.xm + TP_MAX;
        z = a.xm + 2 * TP_MAX;
    }
    const double X = x[i], Y = y[i], Z = z[i], rci = a.rc[i];
    bool inside = false;
    if (tid < a.nm && tid != i) {
        const double dx = x[tid] - X, dy = y[tid] - Y, dz = z[tid] - Z;
        const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
        if (r2 == 0.0) {
            atomicOr(a.status, ST_NONFINITE);
        } else {
            const double ir = rsq_full(r2), rho2 = rho2_of(rci, a.rc[tid]);
            double s = (ir * ir) * (a.m[tid] * ir);
            inside = r2 < rho2;
            if (inside) s *= tp_changeover(r2, rho2);
            f[0] = __builtin_fma(dx, s, f[0]);
            f[1] = __builtin_fma(dy, s, f[1]);
            f[2] = __builtin_fma(dz, s, f[2]);
        }
    }
    const uint64_t near = __ballot(inside && tid > i);   // (massive: the first wave)
    for (int k = 0; k < 3; ++k) sm[k][tid] = f[k];
    tp_sum3(sm, f);
    if (a.emit) {
        uint64_t *row = a.bits + (size_t)i * a.nw;
        int64_t c = 0, tot;
        for (int k = tid; k < a.nw; k += RB) {
            uint64_t b = row[k];
            if (k == 0) row[0] = b |= near;
            c += __popcll(b);
        }
        (void)block_excl_scan<RB>(c, &tot, sc);
        if (tid == 0) a.cnt[i] = (int32_t)tot;
    }
    if (tid != 0) return;
    for (int k = 0; k < 3; ++k) f[k] *= a.G;
    if (!(isfinite(f[0]) && isfinite(f[1]) && isfinite(f[2]))) atomicOr(a.status, ST_NONFINITE);
    if (a.h != 0.0 || a.mom) {
        double V[3] = {a.vx[i], a.vy[i], a.vz[i]};
        if (a.h != 0.0) {
            for (int k = 0; k < 3; ++k) V[k] = __builtin_fma(a.h, f[k], V[k]);
            a.vx[i] = V[0];
            a.vy[i] = V[1];
            a.vz[i] = V[2];
        }
        if (a.mom)
            for (int k = 0; k < 3; ++k) a.q0[k * RB + i] = a.m[i] * V[k];
    }
    if (a.ax) {
        a.ax[i] = f[0];
        a.ay[i] = f[1];
        a.az[i] = f[2];
    }
    if (a.hc_part) {
        a.x[i] = X + (a.hc_h * P[0]) / a.m_star;
        a.y[i] = Y + (a.hc_h * P[1]) / a.m_star;
        a.z[i] = Z + (a.hc_h * P[2]) / a.m_star;
    }
}

// The list of massive body `i` from the bitmaps and counts (one block).
__device__ __forceinline__ void tp_pairs_row(const TpDev &a, int i, const genga_pairs &out, int64_t *sc)
{
    const int tid = threadIdx.x;
    int64_t pos = 0;
    for (int r = 0; r < i; ++r) pos += a.cnt[r];
    if (i == a.nm - 1 && tid == 0) {
        const int64_t tot = pos + a.cnt[i];
        *out.count = tot;
        if (tot > out.capacity) atomicOr(a.status, ST_OVERFLOW);
    }
    for (int k0 = 0; k0 < a.nw; k0 += RB) {
        const int k = k0 + tid;
        uint64_t b = k < a.nw ? a.bits[(size_t)i * a.nw + k] : 0;
        int64_t tot;
        int64_t p = pos + block_excl_scan<RB>(__popcll(b), &tot, sc);
        while (b) {
            const int j = k * 64 + __ffsll((unsigned long long)b) - 1;
            b &= b - 1;
            if (p < out.capacity) {
                out.i[p] = i;
                out.j[p] = j;
            }
            ++p;
        }
        pos += tot;
    }
}

__global__ __launch_bounds__(RB) void k_tp_pairs(TpDev a, genga_pairs out)
{
    __shared__ int64_t sc[RB / 64];
    tp_pairs_row(a, (int)blockIdx.x, out, sc);
}

// Blocks [0, nb): HC(h), the drift and the momentum of the drifted bodies (as
// k_hc_drift; the first 256 bodies' momentum from a.q0).  Blocks [nb, nb + nm):
// the encounter list of the kick before, meanwhile.
__global__ __launch_bounds__(RB) void k_tp_drift(TpDev a, const double *hc_in, double h, double mu,
                                                 double *hc_out, int nb, genga_pairs out)
{
    __shared__ union {
        double red[3][RB];
        int64_t scan[RB / 64];
    } sm;
    if ((int)blockIdx.x >= nb) {
        tp_pairs_row(a, (int)blockIdx.x - nb, out, sm.scan);
        return;
    }
    const int t = threadIdx.x, i = (int)blockIdx.x * RB + t;
    double P[3], q[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < 3; ++k) sm.red[k][t] = a.q0[k * RB + t];
    tp_sum3(sm.red, P);
    for (int b = t; b < nb; b += RB)
        for (int k = 0; k < 3; ++k) q[k] += b == 0 ? P[k] : hc_in[(size_t)b * 3 + k];
    for (int k = 0; k < 3; ++k) sm.red[k][t] = q[k];
    tp_sum3(sm.red, P);
    q[0] = q[1] = q[2] = 0.0;
    if (i < a.n) {
        double X = a.x[i] + (h * P[0]) / a.m_star, Y = a.y[i] + (h * P[1]) / a.m_star,
               Z = a.z[i] + (h * P[2]) / a.m_star;
        double VX = a.vx[i], VY = a.vy[i], VZ = a.vz[i];
        const int st = kepler_uv(mu, a.dt, X, Y, Z, VX, VY, VZ);
        if (st) atomicOr(a.status, st);
        a.x[i] = X; a.y[i] = Y; a.z[i] = Z;
        a.vx[i] = VX; a.vy[i] = VY; a.vz[i] = VZ;
        if (i < a.nm) {
            a.xm[i] = X;
            a.xm[TP_MAX + i] = Y;
            a.xm[2 * TP_MAX + i] = Z;
        }
        if (a.back || i < a.nm) {
            const double mi = a.m[i];
            q[0] = mi * VX;
            q[1] = mi * VY;
            q[2] = mi * VZ;
        }
    }
    for (int k = 0; k < 3; ++k) sm.red[k][t] = q[k];
    tp_sum3(sm.red, q);
    if (t < 3) hc_out[(size_t)blockIdx.x * 3 + t] = q[t];
}

// The kick: the test particles with their shares, then the massive bodies.
static hipError_t launch_halves(const KickLaunch &k, TpDev &a, int nb, hipStream_t s)
{
    hipError_t e;
    if (k.ev0 && (e = hipEventRecord((hipEvent_t)k.ev0, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_tp_kick, dim3((unsigned)nb), dim3(RB), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (k.ev1 && (e = hipEventRecord((hipEvent_t)k.ev1, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_tp_massive, dim3((unsigned)a.nm), dim3(RB), 0, s, a, nb);
    return hipGetLastError();
}

static TpDev tp_dev(const KickLaunch &k, const KickCfg &c, const Layout &L, char *ws)
{
    TpDev a{};
    a.x = const_cast<double *>(k.x);
    a.y = const_cast<double *>(k.y);
    a.z = const_cast<double *>(k.z);
    a.vx = k.vx; a.vy = k.vy; a.vz = k.vz;
    a.m = k.m;
    a.rc = const_cast<double *>(k.rc);
    a.n = (int)k.n;
    a.nm = (int)c.nm;
    a.nw = (int)((k.n + 63) / 64);
    a.back = c.tp == 2;
    a.G = k.G;
    a.h = k.h;
    a.ax = k.ax; a.ay = k.ay; a.az = k.az;
    a.part = (double *)(ws + L.part);
    a.emit = k.pairs != nullptr;
    a.bits = (uint64_t *)(ws + L.stage);
    a.cnt = (int32_t *)(ws + L.cnt);
    a.status = (int32_t *)(ws + L.status);
    a.c53 = 5.0 / 3.0;
    return a;
}

// The blocks' sums (3 doubles per massive body and 256 bodies, then the step's
// 3 TP_MAX) lie in the partial-sum region (5 doubles per body) and the bitmaps (8 B per massive body and 64 bodies) in the
// staging region (1,536 B per wave of test-particle rows).
hipError_t launch_kick_tp(const KickLaunch &k, const KickCfg &c, const Layout &L, char *ws,
                          hipStream_t s)
{
    TpDev a = tp_dev(k, c, L, ws);
    hipError_t e = launch_halves(k, a, (int)L.nb, s);
    if (e != hipSuccess || !a.emit) return e;
    hipLaunchKernelGGL(k_tp_pairs, dim3((unsigned)a.nm), dim3(RB), 0, s, a, *k.pairs);
    return hipGetLastError();
}

hipError_t launch_step_tp(KickLaunch &k, genga_bodies *b, const genga_params *p, const KickCfg &c,
                          const Layout &L, char *ws, hipStream_t s)
{
    const double h = 0.5 * p->dt;
    const int nb = (int)L.nb;
    k.ev0 = p->prof_events[0];
    k.ev1 = p->prof_events[1];
    TpDev a = tp_dev(k, c, L, ws);
    a.rcrit = 1;
    a.m_star = p->m_star;
    a.dt = p->dt;
    a.n1 = p->n1;
    a.n2 = p->n2;
    a.mom = (double *)(ws + L.hc);
    a.q0 = (double *)(ws + L.gru);
    a.xm = a.part + 3 * TP_MAX * (size_t)nb;
    hipError_t e = launch_halves(k, a, nb, s);
    if (e != hipSuccess) return e;
    double *mom2 = (double *)(ws + L.hc2);
    hipLaunchKernelGGL(k_tp_drift, dim3((unsigned)(a.emit ? nb + a.nm : nb)), dim3(RB), 0, s, a,
                       (const double *)a.mom, h, p->G * p->m_star, mom2, nb,
                       k.pairs ? *k.pairs : genga_pairs{});
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k.ev0 = p->prof_events[2];
    k.ev1 = p->prof_events[3];
    a.rcrit = 0;
    a.emit = 0;
    a.mom = nullptr;
    a.q0 = nullptr;
    a.hc_part = mom2;
    a.hc_nb = nb;
    a.hc_h = h;
    return launch_halves(k, a, nb, s);
}

}  // namespace genga
