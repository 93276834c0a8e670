// One-sided binary64 kick of a small system (below SYM_MIN_N bodies) in one
// kernel, its encounter list, and the launches of the base step around it
// (GENGA II Sect. 2, eqs. Hb, Hc, rcrit; Appendix A).
//
// A small system is bound by latency and launches, not by its pairs (2,048
// bodies: 3 us of pair work per kick on the whole chip).  The tiled kick cuts
// the columns into slices, whose sums a second kernel adds; its diagonal
// waves enter the rare path once per column for the self pair (14 of the 15.6
// us of that kick).  Here a block owns 4 rows and every column
// (csrc/rows.h), so that the block ends with the accelerations themselves:
// the velocities, the rows' momentum and, in the second half kick, the Sun
// kick of the step are applied in the same kernel.
#include "device_common.h"
#include "genga_internal.h"
#include "kepler.h"
#include "rows.h"

namespace genga {

constexpr int ROWS_SEG = 16;       // pairs of a row kept as a list

struct RowsDev {
    RowsCols c;
    int n, nw;                     // bodies, bitmap words per row
    double G, h;                   // v += h a (h = 0: not)
    double *vx, *vy, *vz;
    double *ax, *ay, *az;          // optional
    double *mom;                   // optional: [row groups][3] sums of m v of the rows
    // optional (hc_part non-null): ox = x + hc_h P / hc_m_star, P the sum of the
    // hc_nb sums of 256 bodies; the columns are read from c, so ox must not be c.x
    double *ox, *oy, *oz;
    const double *hc_part;
    int hc_nb;
    double hc_h, hc_m_star;
    int emit;
    int32_t *cnt;                  // [n] pairs j > i of row i
    int32_t *seg;                  // [n][ROWS_SEG] their columns, rows with up to ROWS_SEG
    uint64_t *bits;                // [n][nw] bitmap of the columns, rows with more
    int32_t *status;
    double c53;
};

// The momentum P = sum m v of a small system is summed as a balanced binary
// tree in body order (padded with zeros), whoever sums it: a kick block the
// subtree of its row group, the drift and k_momentum_rows 256 bodies, and the
// top (at most 32 values) whoever applies P.
__device__ __forceinline__ double wave_tree(double v)
{
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    return v;
}

// Tree over the 256 threads of a block; the result in every thread.
__device__ __forceinline__ void block_tree(const double q[3], double (*sm)[4], double P[3])
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double v = wave_tree(q[c]);
        if (lane == 0) sm[c][w] = v;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) P[c] = (sm[c][0] + sm[c][1]) + (sm[c][2] + sm[c][3]);
}

constexpr int ROWS_NB = (int)(ROWS_MAX / RB);   // 256-body blocks of the largest system
static_assert(ROWS_NB <= 64, "the top of the tree is one wave's");

// Top of the tree: nb sums of 256 bodies, one per lane of a wave.
__device__ __forceinline__ double top_tree(const double *part, int nb, int c)
{
    const int lane = threadIdx.x & 63;
    return wave_tree(lane < nb ? part[(size_t)lane * 3 + c] : 0.0);
}

// One row group per block (fewer waves per group are slower at every size: step
// of 500 / 2,048 / 8,191 bodies with 1, 2 and 4 waves a group 34 / 28 / 24, 60 /
// 43 / 35 and 150 / 141 / 138 us).
__global__ __launch_bounds__(256) void k_kick_rows(RowsDev a)
{
    __shared__ RowsTeam sm;
    const int tid = threadIdx.x, grp = (int)blockIdx.x;
    const int r0 = grp * ROWS_G;
    // what the end of the block reads, loaded ahead of the columns (a round trip
    // to memory each, of which a block of a small system has few to hide: step of
    // 500 / 2,048 / 4,096 bodies 22.8 / 32.2 / 57.2 -> 21.7 / 31.1 / 55.9 us)
    const int i = r0 + tid;
    const bool real = tid < ROWS_G && i < a.n;
    const bool vel = real && (a.h != 0.0 || a.mom);
    double VX = 0.0, VY = 0.0, VZ = 0.0, mi = 0.0, X = 0.0, Y = 0.0, Z = 0.0;
    if (vel) {
        VX = a.vx[i];
        VY = a.vy[i];
        VZ = a.vz[i];
        mi = a.c.m[i];
    }
    double P[3] = {0.0, 0.0, 0.0};
    if (a.hc_part && tid < 64) {
        if (tid < a.hc_nb) {
#pragma unroll
            for (int c = 0; c < 3; ++c) P[c] = a.hc_part[(size_t)tid * 3 + c];
        }
        if (real) {
            X = a.c.x[i];
            Y = a.c.y[i];
            Z = a.c.z[i];
        }
    }
    double a3[3];
    rows_team(a.c, a.n, r0, tid, sm, a.status, a.c53, a3);
    if (a.emit) {
        // (rarely any: a row's pairs in order, by one wave)
        const int lane = tid & 63;
        const int q = tid >> 6, i = r0 + q;
        const int cnt = i < a.n ? sm.cnt[q] : 0;
        if (cnt > 0) {
            int at = 0;
            for (int k0 = 0; k0 < a.nw; k0 += 64) {
                const uint64_t word = k0 + lane < a.nw ? sm.bits[q][k0 + lane] : 0;
                if (cnt > ROWS_SEG) {
                    if (k0 + lane < a.nw) a.bits[(size_t)i * a.nw + k0 + lane] = word;
                    continue;
                }
                uint64_t some = __ballot(word != 0);
                while (some) {
                    const int k = __ffsll((unsigned long long)some) - 1;
                    some &= some - 1;
                    const uint64_t b = __shfl(word, k);
                    if ((b >> lane) & 1)
                        a.seg[(size_t)i * ROWS_SEG + at + __popcll(b & lanemask_lt())] =
                            (k0 + k) * 64 + lane;
                    at += __popcll(b);
                }
            }
        }
    }
    if (tid >= 64) return;
    if (a.hc_part) {
#pragma unroll
        for (int c = 0; c < 3; ++c) P[c] = wave_tree(P[c]);
    }
    if (tid >= ROWS_G) return;
    double q0 = 0.0, q1 = 0.0, q2 = 0.0;
    if (real) {
#pragma unroll
        for (int k = 0; k < 3; ++k) a3[k] *= a.G;
        if (!(isfinite(a3[0]) && isfinite(a3[1]) && isfinite(a3[2])))
            atomicOr(a.status, ST_NONFINITE);
        if (vel) {
            if (a.h != 0.0) {
                VX = __builtin_fma(a.h, a3[0], VX);
                VY = __builtin_fma(a.h, a3[1], VY);
                VZ = __builtin_fma(a.h, a3[2], VZ);
                a.vx[i] = VX;
                a.vy[i] = VY;
                a.vz[i] = VZ;
            }
            q0 = mi * VX;
            q1 = mi * VY;
            q2 = mi * VZ;
        }
        if (a.ax) {
            a.ax[i] = a3[0];
            a.ay[i] = a3[1];
            a.az[i] = a3[2];
        }
        if (a.hc_part) {
            a.ox[i] = X + (a.hc_h * P[0]) / a.hc_m_star;
            a.oy[i] = Y + (a.hc_h * P[1]) / a.hc_m_star;
            a.oz[i] = Z + (a.hc_h * P[2]) / a.hc_m_star;
        }
        if (a.emit) a.cnt[i] = sm.cnt[tid];
    }
    if (a.mom) {
        q0 += __shfl_xor(q0, 1);
        q1 += __shfl_xor(q1, 1);
        q2 += __shfl_xor(q2, 1);
        q0 += __shfl_xor(q0, 2);
        q1 += __shfl_xor(q1, 2);
        q2 += __shfl_xor(q2, 2);
        if (tid < 3) a.mom[(size_t)grp * 3 + tid] = tid == 0 ? q0 : (tid == 1 ? q1 : q2);
    }
}

// The encounter list from the rows' counts, lists and bitmaps: the blocks
// `blk` + nblk * part write the pairs of rows [256 blk, 256 blk + 256); every
// block adds the counts before its rows itself.  Part 0 writes the rows with a
// list and, in the last block, the true number of pairs; a row with a bitmap,
// whose words its wave takes one after another, is one wave's of all parts (kick
// of 4,096 bodies with about 20 / 160 partners each: 197 / 527 us with one
// part, 50 / 75 with 16, 39 / 54 with 64; few pairs: no difference).
constexpr int ROWS_PARTS = 64;
static_assert(ROWS_PARTS * (RB / 64) == RB, "a wave per row");

struct RowsPairs {
    const int32_t *cnt, *seg;
    const uint64_t *bits;
    int n, nw, nblk;
    int32_t *pi, *pj;
    int64_t capacity;
    int64_t *count;
    int32_t *status;
};

struct RowsPairsSmem {
    int64_t scan[RB / 64];
    int64_t pos[RB];
    int32_t cnt[RB];
};

__device__ __forceinline__ void pairs_rows_block(const RowsPairs &d, int slot, RowsPairsSmem &sm)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int blk = slot % d.nblk, part = slot / d.nblk;
    const int row0 = blk * RB, i = row0 + tid;
    const int32_t c = i < d.n ? d.cnt[i] : 0;
    if (part > 0 && !__syncthreads_or(c > ROWS_SEG)) return;
    int64_t before = 0, base, own;
    for (int k = tid; k < row0; k += RB) before += d.cnt[k];
    (void)block_excl_scan<RB>(before, &base, sm.scan);
    const int64_t off = block_excl_scan<RB>(c, &own, sm.scan);
    sm.pos[tid] = base + off;
    sm.cnt[tid] = c;
    if (part == 0 && blk == d.nblk - 1 && tid == 0) {
        *d.count = base + own;
        if (base + own > d.capacity) atomicOr(d.status, ST_OVERFLOW);
    }
    __syncthreads();
    // few pairs: the row's thread copies them (their loads in flight together)
    if (part == 0 && c > 0 && c <= ROWS_SEG) {
#pragma unroll
        for (int e = 0; e < ROWS_SEG; ++e) {
            if (e >= c) continue;
            const int32_t j = d.seg[(size_t)i * ROWS_SEG + e];
            if (base + off + e < d.capacity) {
                d.pi[base + off + e] = i;
                d.pj[base + off + e] = j;
            }
        }
    }
    const int t = part * (RB / 64) + __builtin_amdgcn_readfirstlane(tid >> 6);
    if (sm.cnt[t] <= ROWS_SEG) return;
    const int r = row0 + t;
    int64_t pos = sm.pos[t];
    for (int k0 = 0; k0 < d.nw; k0 += 64) {
        const uint64_t word = k0 + lane < d.nw ? d.bits[(size_t)r * d.nw + k0 + lane] : 0;
        uint64_t some = __ballot(word != 0);
        while (some) {
            const int k = __ffsll((unsigned long long)some) - 1;
            some &= some - 1;
            const uint64_t b = __shfl(word, k);
            if ((b >> lane) & 1) {
                const int64_t p = pos + __popcll(b & lanemask_lt());
                if (p < d.capacity) {
                    d.pi[p] = r;
                    d.pj[p] = (k0 + k) * 64 + lane;
                }
            }
            pos += __popcll(b);
        }
    }
}

__global__ __launch_bounds__(RB) void k_pairs_rows(RowsPairs d)
{
    __shared__ RowsPairsSmem sm;
    pairs_rows_block(d, (int)blockIdx.x, sm);
}

__global__ __launch_bounds__(RB) void k_momentum_rows(const double *vx, const double *vy,
                                                      const double *vz, const double *m, int64_t n,
                                                      double *out)
{
    __shared__ double sm[3][4];
    const int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x;
    const double mi = i < n ? m[i] : 0.0;
    const double q[3] = {i < n ? mi * vx[i] : 0.0, i < n ? mi * vy[i] : 0.0, i < n ? mi * vz[i] : 0.0};
    double P[3];
    block_tree(q, sm, P);
    if (threadIdx.x < 3) out[(size_t)blockIdx.x * 3 + threadIdx.x] = P[threadIdx.x];
}

__global__ __launch_bounds__(RB) void k_hc_apply_rows(double *x, double *y, double *z, int64_t n,
                                                      const double *part, int nb, double h,
                                                      double m_star)
{
    double P[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) P[c] = top_tree(part, nb, c);
    const int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x;
    if (i >= n) return;
    x[i] += (h * P[0]) / m_star;
    y[i] += (h * P[1]) / m_star;
    z[i] += (h * P[2]) / m_star;
}

// Blocks [0, nb): HC(h) with the row groups' momentum hc_in, the Kepler drift,
// the drifted positions to xs (the next kick reads them there and writes the
// state's after its Sun kick) and the momentum of 256 bodies to hc_out.
// The blocks behind them: the encounter list of the kick before, meanwhile.
__global__ __launch_bounds__(RB) void k_hc_drift_rows(const double *x, const double *y,
                                                      const double *z, double *vx, double *vy,
                                                      double *vz, const double *m, int64_t n,
                                                      const double *hc_in, double h, double m_star,
                                                      double mu, double dt, double *xs, double *ys,
                                                      double *zs, double *hc_out, int32_t *status,
                                                      int nb, RowsPairs pairs)
{
    __shared__ union {
        struct {
            double blk[64][3], wave[3][4];
        } mom;
        RowsPairsSmem pairs;
    } sm;
    if ((int)blockIdx.x >= nb) {
        pairs_rows_block(pairs, (int)blockIdx.x - nb, sm.pairs);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x;
    double X, Y, Z, VX, VY, VZ, mi = 0.0;
    if (i < n) {
        X = x[i]; Y = y[i]; Z = z[i];
        VX = vx[i]; VY = vy[i]; VZ = vz[i];
        mi = m[i];
    }
    // subtrees of 256 bodies (64 row groups, one per lane), a wave each
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int ng = (int)((n + ROWS_G - 1) / ROWS_G);
    for (int b = w; b < nb; b += 4) {
        const int g = b * (RB / ROWS_G) + lane;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double s = wave_tree(g < ng ? hc_in[(size_t)g * 3 + c] : 0.0);
            if (lane == 0) sm.mom.blk[b][c] = s;
        }
    }
    __syncthreads();
    double P[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) P[c] = top_tree(&sm.mom.blk[0][0], nb, c);
    double q[3] = {0.0, 0.0, 0.0};
    if (i < n) {
        X += (h * P[0]) / m_star;
        Y += (h * P[1]) / m_star;
        Z += (h * P[2]) / m_star;
        const int st = kepler_uv(mu, dt, X, Y, Z, VX, VY, VZ);
        if (st) atomicOr(status, st);
        xs[i] = X; ys[i] = Y; zs[i] = Z;
        vx[i] = VX; vy[i] = VY; vz[i] = VZ;
        q[0] = mi * VX;
        q[1] = mi * VY;
        q[2] = mi * VZ;
    }
    block_tree(q, sm.mom.wave, P);
    if (threadIdx.x < 3) hc_out[(size_t)blockIdx.x * 3 + threadIdx.x] = P[threadIdx.x];
}
static_assert(RB / ROWS_G == 64, "one lane per row group of 256 bodies");

// Up to ONE_MAX bodies in one workgroup: the whole chip would have one or two
// pairs per lane, and what counts is the chain of dependent steps and the
// launches.  Bodies and accelerations sit in LDS; a row's pairs are shared out
// over 1024 / n lanes (8 to 32), each evaluated where it stands, rare path
// included, and summed by a butterfly.
constexpr int ONE_NT = 1024;

struct OneSmem {
    double c[5][ONE_MAX];       // x, y, z, m, rc
    double a[3][ONE_MAX];
    double wave[3][2];
    unsigned long long bits[ONE_MAX][2];   // pairs j > i of row i
};

// Accelerations / G of all bodies into sm.a, their pairs into sm.bits.
__device__ __forceinline__ void one_forces(OneSmem &sm, int n, int32_t *status)
{
    const int t = threadIdx.x;
    const int lanes = n <= 32 ? 32 : (n <= 64 ? 16 : 8);
    const int i = t / lanes;
    if (t < 2 * ONE_MAX) sm.bits[t >> 1][t & 1] = 0;
    __syncthreads();
    double ax = 0.0, ay = 0.0, az = 0.0;
    if (i < n) {
        const double xi = sm.c[0][i], yi = sm.c[1][i], zi = sm.c[2][i], ri = sm.c[4][i];
        for (int j = t % lanes; j < n; j += lanes) {
            const double dx = sm.c[0][j] - xi, dy = sm.c[1][j] - yi, dz = sm.c[2][j] - zi;
            const double mj = sm.c[3][j];
            const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
            const double y = rsq_full(r2);
            double w = (y * y) * (mj * y);
            const double rho2 = rho2_of(ri, sm.c[4][j]);
            if (r2 < rho2 || r2 == 0.0) {
                if (r2 == 0.0) {
                    w = 0.0;
                    if (j != i) atomicOr(status, ST_NONFINITE);
                } else {
                    const double irho = rsq_full(rho2);
                    w *= changeover_of_y(__builtin_fma((r2 * y) * irho, 1.0 / 0.9, -1.0 / 9.0));
                    if (j > i) atomicOr(&sm.bits[i][j >> 6], 1ull << (j & 63));
                }
            }
            ax = __builtin_fma(dx, w, ax);
            ay = __builtin_fma(dy, w, ay);
            az = __builtin_fma(dz, w, az);
        }
    }
    for (int off = lanes / 2; off >= 1; off >>= 1) {
        ax += __shfl_xor(ax, off);
        ay += __shfl_xor(ay, off);
        az += __shfl_xor(az, off);
    }
    if (i < n && t % lanes == 0) {
        sm.a[0][i] = ax;
        sm.a[1][i] = ay;
        sm.a[2][i] = az;
    }
    __syncthreads();
}

// The list from sm.bits, by one wave: lane l writes the rows l and l + 64.
__device__ __forceinline__ void one_pairs(const OneSmem &sm, int n, int32_t *pi, int32_t *pj,
                                          int64_t capacity, int64_t *count, int32_t *status)
{
    const int lane = threadIdx.x & 63;
    int64_t before = 0;
    for (int r0 = 0; r0 < n; r0 += 64) {
        const int r = r0 + lane;
        const int64_t c = r < n ? __popcll(sm.bits[r][0]) + __popcll(sm.bits[r][1]) : 0;
        const int64_t inc = wave_incl_scan(c);
        int64_t at = before + inc - c;
        for (int k = 0; k < 2; ++k) {
            unsigned long long b = r < n ? sm.bits[r][k] : 0;
            while (b) {
                const int j = 64 * k + __ffsll(b) - 1;
                b &= b - 1;
                if (at < capacity) {
                    pi[at] = r;
                    pj[at] = j;
                }
                ++at;
            }
        }
        before += __shfl(inc, 63);
    }
    if (lane == 0) {
        *count = before;
        if (before > capacity) atomicOr(status, ST_OVERFLOW);
    }
}

// The momentum of the bodies (the first two waves' threads) as the balanced
// tree; the result in every thread.
__device__ __forceinline__ void one_momentum(OneSmem &sm, const double q[3], double P[3])
{
    const int t = threadIdx.x;
    if (t < ONE_MAX) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = wave_tree(q[c]);
            if ((t & 63) == 0) sm.wave[c][t >> 6] = v;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) P[c] = sm.wave[c][0] + sm.wave[c][1];
    __syncthreads();
}

// The kick alone.
__global__ __launch_bounds__(ONE_NT) void k_kick_one(RowsDev a, genga_pairs out)
{
    __shared__ OneSmem sm;
    const int i = threadIdx.x;
    if (i < a.n) {
        const double rc = a.c.rc[i];
        if (!(rc >= 0.0 && rc < INFINITY)) atomicOr(a.status, ST_RCRIT);
        sm.c[0][i] = a.c.x[i]; sm.c[1][i] = a.c.y[i]; sm.c[2][i] = a.c.z[i];
        sm.c[3][i] = a.c.m[i]; sm.c[4][i] = rc;
    }
    __syncthreads();
    one_forces(sm, a.n, a.status);
    if (i >= ONE_MAX && i < ONE_MAX + 64 && a.emit)
        one_pairs(sm, a.n, out.i, out.j, out.capacity, out.count, a.status);
    if (i >= a.n) return;
    double a3[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        a3[k] = sm.a[k][i] * a.G;
        if (!isfinite(a3[k])) atomicOr(a.status, ST_NONFINITE);
    }
    if (a.h != 0.0) {
        a.vx[i] = __builtin_fma(a.h, a3[0], a.vx[i]);
        a.vy[i] = __builtin_fma(a.h, a3[1], a.vy[i]);
        a.vz[i] = __builtin_fma(a.h, a3[2], a.vz[i]);
    }
    if (a.ax) {
        a.ax[i] = a3[0];
        a.ay[i] = a3[1];
        a.az[i] = a3[2];
    }
}

// The whole base step, one thread a body outside the kicks; a spare wave
// writes the list while the others drift.
struct StepOne {
    double *x, *y, *z, *vx, *vy, *vz;
    const double *m;
    double *rc;
    int n;
    double G, m_star, dt, n1, n2;
    genga_pairs out;               // count null: no list
    int32_t *status;
};

__global__ __launch_bounds__(ONE_NT) void k_step_one(StepOne a)
{
    __shared__ OneSmem sm;
    const int i = threadIdx.x, n = a.n;
    const double h = 0.5 * a.dt;
    double X[3], V[3], mi = 0.0, P[3], q[3] = {0.0, 0.0, 0.0};
    if (i < n) {
        X[0] = a.x[i]; X[1] = a.y[i]; X[2] = a.z[i];
        V[0] = a.vx[i]; V[1] = a.vy[i]; V[2] = a.vz[i];
        mi = a.m[i];
        const double rc = rcrit_of(X[0], X[1], X[2], V[0], V[1], V[2], mi, a.m_star, a.dt, a.n1, a.n2);
        if (!(rc >= 0.0 && rc < INFINITY)) atomicOr(a.status, ST_RCRIT);
        a.rc[i] = rc;
        sm.c[0][i] = X[0]; sm.c[1][i] = X[1]; sm.c[2][i] = X[2]; sm.c[3][i] = mi; sm.c[4][i] = rc;
    }
    __syncthreads();
    auto kick = [&]() {
        if (i >= n) return;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double acc = sm.a[k][i] * a.G;
            if (!isfinite(acc)) atomicOr(a.status, ST_NONFINITE);
            if (h != 0.0) V[k] = __builtin_fma(h, acc, V[k]);
            q[k] = mi * V[k];
        }
    };
    one_forces(sm, n, a.status);
    kick();
    one_momentum(sm, q, P);
    if (i < n) {
#pragma unroll
        for (int k = 0; k < 3; ++k) X[k] += (h * P[k]) / a.m_star;
        const int st = kepler_uv(a.G * a.m_star, a.dt, X[0], X[1], X[2], V[0], V[1], V[2]);
        if (st) atomicOr(a.status, st);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            sm.c[k][i] = X[k];
            q[k] = mi * V[k];
        }
    } else if (a.out.count && i >= ONE_MAX && i < ONE_MAX + 64) {
        one_pairs(sm, n, a.out.i, a.out.j, a.out.capacity, a.out.count, a.status);
    }
    one_momentum(sm, q, P);   // (its barriers end the drift)
    one_forces(sm, n, a.status);
    kick();
    if (i >= n) return;
    a.x[i] = X[0] + (h * P[0]) / a.m_star;
    a.y[i] = X[1] + (h * P[1]) / a.m_star;
    a.z[i] = X[2] + (h * P[2]) / a.m_star;
    a.vx[i] = V[0];
    a.vy[i] = V[1];
    a.vz[i] = V[2];
}

static RowsPairs rows_pairs(const KickLaunch &k, const Layout &L, char *ws)
{
    RowsPairs d{};
    if (!k.pairs) return d;
    d.cnt = (const int32_t *)(ws + L.cnt);
    d.seg = (const int32_t *)(ws + L.stage);
    d.bits = (const uint64_t *)(d.seg + (size_t)k.n * ROWS_SEG);
    d.n = (int)k.n;
    d.nw = (int)((k.n + 63) / 64);
    d.nblk = (int)L.nb;
    d.pi = k.pairs->i;
    d.pj = k.pairs->j;
    d.capacity = k.pairs->capacity;
    d.count = k.pairs->count;
    d.status = (int32_t *)(ws + L.status);
    return d;
}

// The rows' lists (64 B each) and bitmaps (8 B per 64 columns) share the staging
// region of the tiled kick: 1,536 B for every wave of 64 rows x 64 columns of
// its 256-row blocks, of which they take 512 B, and 4,096 B per 64 rows; with
// 4 waves to a block that fits from one slice on.
static hipError_t launch_rows(const KickLaunch &k, const Layout &L, char *ws, double *mom,
                              hipStream_t s)
{
    RowsDev a{};
    a.c = {k.x, k.y, k.z, k.m, k.rc};
    a.n = (int)k.n;
    a.nw = (int)((k.n + 63) / 64);
    a.G = k.G;
    a.h = k.h;
    a.vx = k.vx; a.vy = k.vy; a.vz = k.vz;
    a.ax = k.ax; a.ay = k.ay; a.az = k.az;
    a.mom = mom;
    a.ox = k.px; a.oy = k.py; a.oz = k.pz;
    a.hc_part = k.hc_part;
    a.hc_nb = (int)k.hc_nb;
    a.hc_h = k.hc_h;
    a.hc_m_star = k.hc_m_star;
    a.emit = k.pairs != nullptr;
    a.cnt = (int32_t *)(ws + L.cnt);
    a.seg = (int32_t *)(ws + L.stage);
    a.bits = (uint64_t *)(a.seg + (size_t)k.n * ROWS_SEG);
    a.status = (int32_t *)(ws + L.status);
    a.c53 = 5.0 / 3.0;
    hipError_t e;
    if (k.ev0 && (e = hipEventRecord((hipEvent_t)k.ev0, s)) != hipSuccess) return e;
    const unsigned grp = (unsigned)((k.n + ROWS_G - 1) / ROWS_G);
    // Up to ONE_MAX bodies in one workgroup (no Sun kick there: the step of
    // such a system is one kernel, or its operators).
    if (k.n <= ONE_MAX && !mom && !k.hc_part)
        hipLaunchKernelGGL(k_kick_one, dim3(1), dim3(ONE_NT), 0, s, a,
                           k.pairs ? *k.pairs : genga_pairs{});
    else
        hipLaunchKernelGGL(k_kick_rows, dim3(grp), dim3(256), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (k.ev1) e = hipEventRecord((hipEvent_t)k.ev1, s);
    return e;
}

hipError_t launch_kick_rows(const KickLaunch &k, const Layout &L, char *ws, hipStream_t s)
{
    hipError_t e = launch_rows(k, L, ws, nullptr, s);
    if (e != hipSuccess || !k.pairs || k.n <= ONE_MAX) return e;
    hipLaunchKernelGGL(k_pairs_rows, dim3((unsigned)(L.nb * ROWS_PARTS)), dim3(RB), 0, s,
                       rows_pairs(k, L, ws));
    return hipGetLastError();
}

hipError_t launch_hc_rows(genga_bodies *b, double m_star, double h, const Layout &L, char *ws,
                          hipStream_t s)
{
    double *part = (double *)(ws + L.hc);
    hipLaunchKernelGGL(k_momentum_rows, dim3((unsigned)L.nb), dim3(RB), 0, s, b->vx, b->vy, b->vz,
                       b->m, b->n, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_hc_apply_rows, dim3((unsigned)L.nb), dim3(RB), 0, s, b->x, b->y, b->z, b->n,
                       part, (int)L.nb, h, m_star);
    return hipGetLastError();
}

hipError_t launch_step_rows(KickLaunch &k, genga_bodies *b, const genga_params *p, const Layout &L,
                            char *ws, hipStream_t s)
{
    const double h = 0.5 * p->dt;
    hipError_t e;
    const bool events =
        p->prof_events[0] || p->prof_events[1] || p->prof_events[2] || p->prof_events[3];
    if (b->n <= ONE_MAX && !events) {
        StepOne a{};
        a.x = b->x; a.y = b->y; a.z = b->z;
        a.vx = b->vx; a.vy = b->vy; a.vz = b->vz;
        a.m = b->m;
        a.rc = b->rc;
        a.n = (int)b->n;
        a.G = p->G;
        a.m_star = p->m_star;
        a.dt = p->dt;
        a.n1 = p->n1;
        a.n2 = p->n2;
        if (k.pairs) a.out = *k.pairs;
        a.status = (int32_t *)(ws + L.status);
        hipLaunchKernelGGL(k_step_one, dim3(1), dim3(ONE_NT), 0, s, a);
        return hipGetLastError();
    }
    if ((e = launch_rcrit(b, p, ws, s)) != hipSuccess) return e;
    // (the row groups' momentum in the partial-sum region: 3 n / 4 of its at
    // least 5 npad doubles)
    double *mom = (double *)(ws + L.part), *mom2 = (double *)(ws + L.hc2);
    double *xs = (double *)(ws + L.gru);
    k.ev0 = p->prof_events[0];
    k.ev1 = p->prof_events[1];
    if ((e = launch_rows(k, L, ws, mom, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_hc_drift_rows, dim3((unsigned)(k.pairs ? L.nb * (1 + ROWS_PARTS) : L.nb)),
                       dim3(RB), 0, s, b->x, b->y, b->z, b->vx, b->vy, b->vz, b->m, b->n, mom, h, p->m_star,
                       p->G * p->m_star, p->dt, xs, xs + L.npad, xs + 2 * L.npad, mom2,
                       (int32_t *)(ws + L.status), (int)L.nb, rows_pairs(k, L, ws));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k.x = xs;
    k.y = xs + L.npad;
    k.z = xs + 2 * L.npad;
    k.pairs = nullptr;
    k.px = b->x; k.py = b->y; k.pz = b->z;
    k.hc_part = mom2;
    k.hc_nb = L.nb;
    k.hc_h = h;
    k.hc_m_star = p->m_star;
    k.ev0 = p->prof_events[2];
    k.ev1 = p->prof_events[3];
    return launch_rows(k, L, ws, nullptr, s);
}

}  // namespace genga
