// Kick of a small system by row groups: device code of csrc/rows.hip.
//
// A team of 256 threads (4 waves) owns ROWS_G = 4 rows and takes every column:
// thread t the columns t, t + 256, ..., each against the 4 rows, whose data
// sit in scalar registers (8 rows needed more of them than there are).  A lane
// loads 5 values per column (the next column's while it works on this one's)
// and evaluates 4 independent pairs, so no column is staged.
// Pairs inside the critical radius are marked in an LDS bitmap (row x column) and
// leave no term in the loop.  Afterwards a row's wave evaluates them: its words of
// 64 columns with at least ROWS_CROWD of them (neighbours in index, or a dense
// system) one after another, a pair per lane, its other words side by side, one
// or two per lane, whose pairs follow each other.  The bitmap, masked to j > i,
// is also the encounter list of the rows in canonical order.  The self pair
// (r^2 = 0) reaches the marking branch like a close pair and is dropped there:
// once per row, in one wave.
// Every sum runs in a fixed order that does not depend on the launch.
#pragma once

#include "device_common.h"
#include "genga_internal.h"

namespace genga {

// Whether any of the arrays of n doubles `out` lies over one of `in`: the row
// groups write a row's results while other blocks still read the columns, so
// such a call takes the forms that write in a second kernel.
template <int NO, int NI>
inline bool arrays_overlap(const double *const (&out)[NO], const double *const (&in)[NI], int64_t n)
{
    for (const double *o : out)
        for (const double *i : in)
            if (o && i && o < i + n && i < o + n) return true;
    return false;
}

// Whether any two of the arrays of n doubles `out` overlap: sums added to them one
// after another, as the two-kernel forms do, are not sums added to values read
// ahead.
template <int NO>
inline bool arrays_overlap(const double *const (&out)[NO], int64_t n)
{
    for (int a = 0; a < NO; ++a)
        for (int b = 0; b < a; ++b)
            if (out[a] < out[b] + n && out[b] < out[a] + n) return true;
    return false;
}

// Columns of a system (global memory or LDS).
struct RowsCols {
    const double *x, *y, *z, *m, *rc;
};

// Marked columns of a word from which on its row's wave takes it by itself, a
// pair per lane: such a word costs the wave one evaluation however many columns it
// has, while left to a lane each column is another chain of gathers and
// estimates.  Kick / VJP, us, with 4 / 6 / 10 / 16: 8,191 bodies of about 650
// scattered partners 224, 191, 155, 155 / 312, 254, 195, 193; a ring of 2,048 with
// 8 index neighbours on each side 18.0, 19.0, 19.8, 22.1 / 17.0, 17.2, 20.0, 22.6;
// 2,048 bodies that all meet 34, 34, 35, 38 / 38, 39, 40, 44.  With every word
// left to the lanes: ring of 32 neighbours 88 / 77 (now 19 / 20), 8,191 bodies that
// all meet 849 / 1,290 (278 / 388).
constexpr int ROWS_CROWD = 10;

// LDS of one team.
struct RowsTeam {
    uint64_t bits[ROWS_G][ROWS_MAX / 64];
    double part[4][3 * ROWS_G];
    double slow[ROWS_G][3];
    int32_t cnt[ROWS_G];
    double row[ROWS_G][4];   // x, y, z, rc of the rows
};

// a and b summed over the two halves of the wave: lanes 0-31 hold a's sums
// (l + (l + 32)), lanes 32-63 b's.
__device__ __forceinline__ double halve32(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// The same over neighbouring rows of 16 lanes: even rows hold a's sums, odd
// rows b's.
__device__ __forceinline__ double halve16(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 16 lanes of a row, in every lane of it up to rounding order
// (callers take lane 0's).
__device__ __forceinline__ double row16_sum(double v)
{
    v += dpp_f64<0x128>(v);   // row_ror:8
    v += dpp_f64<0x124>(v);   // row_ror:4
    v += dpp_f64<0x122>(v);   // row_ror:2
    v += dpp_f64<0x121>(v);   // row_ror:1
    return v;
}

static_assert(ROWS_G == 4, "12 sums: two halvings leave 3 per row of 16 lanes, one row group per wave");

// The crowded words of a row of the bitmap (nw <= ROWS_MAX / 64 words; all lanes
// of a wave pass): eval(j, column) by every lane whose column j = 64 k + lane is
// marked in such a word k, the words in order; the next one's columns are loaded
// meanwhile.
template <class Load, class Eval>
__device__ __forceinline__ void crowded_words(const uint64_t *bits, int nw, Load load, Eval eval)
{
    static_assert(ROWS_MAX / 64 <= 128, "two words a lane");
    const int lane = threadIdx.x & 63;
    auto pick = [&](int k) { return __ballot(k < nw && __popcll(bits[k < nw ? k : 0]) >= ROWS_CROWD); };
    uint64_t todo[2] = {pick(lane), nw > 64 ? pick(64 + lane) : 0};
    auto next = [&]() {
        const int h = todo[0] == 0;
        if (!todo[h]) return -1;
        const int k = __builtin_ctzll(todo[h]);
        todo[h] &= todo[h] - 1;
        return 64 * h + k;
    };
    int k = next();
    if (k < 0) return;
    auto cur = load(64 * k + lane);
    while (k >= 0) {
        const int kn = next();
        const auto nx = load(64 * (kn < 0 ? k : kn) + lane);
        if ((bits[k] >> lane) & 1) eval(64 * k + lane, cur);
        cur = nx;
        k = kn;
    }
}

// m K / r^3 of a pair inside its critical radius.
__device__ __forceinline__ double close_weight(double r2, double rho2, double m)
{
    const double yc = rsq_full(r2), irho = rsq_full(rho2);
    const double K = changeover_of_y(__builtin_fma((r2 * yc) * irho, 1.0 / 0.9, -1.0 / 9.0));
    return (m * K) * (yc * yc * yc);
}

// One column against the rows.
__device__ __forceinline__ void rows_column(RowsTeam &sm, const double (&xi)[ROWS_G],
                                            const double (&yi)[ROWS_G], const double (&zi)[ROWS_G],
                                            const double (&rc2i)[ROWS_G], double rg, int n, int r0,
                                            int j, double xj, double yj, double zj, double mj,
                                            double rcj, double c53, int word, int lane,
                                            int32_t &bad, double (&acc)[3 * ROWS_G])
{
    double dx[ROWS_G], dy[ROWS_G], dz[ROWS_G], r2[ROWS_G], sc[ROWS_G];
    const double m15 = 1.5 * mj, rc2j = rcj * rcj;
    double near = INFINITY;
#pragma unroll
    for (int q = 0; q < ROWS_G; ++q) {
        dx[q] = xj - xi[q];
        dy[q] = yj - yi[q];
        dz[q] = zj - zi[q];
        r2[q] = __builtin_fma(dz[q], dz[q], __builtin_fma(dy[q], dy[q], dx[q] * dx[q]));
        near = vmin_f64(near, r2[q]);
        // m r^-3 = (3/2 m) y^3 (5/3 - r^2 y^2) to first order, as in the other kicks
        const double y = __builtin_amdgcn_rsq(r2[q]);
        const double y2 = y * y;
        sc[q] = (m15 * (y2 * y)) * __builtin_fma(-r2[q], y2, c53);
    }
    // rare: some lane has a row inside the larger of the rows' and its own radius
    if (__any(near <= vmax_f64(rg, rc2j))) {
#pragma unroll
        for (int q = 0; q < ROWS_G; ++q) {
            const double rho2 = vmax_f64(rc2i[q], rc2j);
            if (!__any(r2[q] <= rho2)) continue;
            const bool same = r2[q] == 0.0;
            // (a column past the end repeats the last body without its mass)
            const bool inside = r2[q] < rho2 && !same && j < n;
            if (same && j < n && j != r0 + q) bad |= ST_NONFINITE;
            if (inside || same) sc[q] = 0.0;
            const uint64_t mask = __ballot(inside);
            if (mask && lane == 0) sm.bits[q][word] = mask;
        }
    }
#pragma unroll
    for (int q = 0; q < ROWS_G; ++q) {
        acc[3 * q + 0] = __builtin_fma(dx[q], sc[q], acc[3 * q + 0]);
        acc[3 * q + 1] = __builtin_fma(dy[q], sc[q], acc[3 * q + 1]);
        acc[3 * q + 2] = __builtin_fma(dz[q], sc[q], acc[3 * q + 2]);
    }
}

// A lane's column values; past the end, the last body's.
struct RowsColumn {
    double x, y, z, m, rc;
};

__device__ __forceinline__ RowsColumn rows_load(const RowsCols &c, int n, int j)
{
    // (32-bit byte offsets from scalar bases)
    const uint32_t o = (uint32_t)(j < n ? j : n - 1) * 8u;
    auto at = [o](const double *p) { return *(const double *)((const char *)p + o); };
    return {at(c.x), at(c.y), at(c.z), at(c.m), at(c.rc)};
}

// Accelerations / G of the rows [r0, r0 + ROWS_G) from the columns [0, n), and
// their encounter pairs j > i as sm.cnt and sm.bits; the lanes t < ROWS_G of
// the team's first wave return row r0 + t's sums in a3.  tid: thread of the
// team; every thread of the block passes here (block barriers).  Rows from n
// on are computed at a far place and are to be ignored.
__device__ __forceinline__ void rows_team(const RowsCols &c, int n, int r0, int tid, RowsTeam &sm,
                                          int32_t *status, double c53k, double a3[3])
{
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = (n + 63) >> 6;
    RowsColumn A = rows_load(c, n, tid), B;
    for (int q = 0; q < ROWS_G; ++q)
        for (int k = tid; k < nw; k += 256) sm.bits[q][k] = 0;
    // (an opaque zero keeps the constant in vector registers)
    const double c53 = c53k + (double)(int)__builtin_amdgcn_mbcnt_lo(0u, 0u);
    double xi[ROWS_G], yi[ROWS_G], zi[ROWS_G], rc2i[ROWS_G], rg = 0.0;
#pragma unroll
    for (int q = 0; q < ROWS_G; ++q) {
        const int i = r0 + q < n ? r0 + q : n - 1;
        const bool real = r0 + q < n;
        const double r = wave_uniform(c.rc[i]);
        xi[q] = wave_uniform(real ? c.x[i] : 1e18);
        yi[q] = wave_uniform(real ? c.y[i] : 1e18);
        zi[q] = wave_uniform(real ? c.z[i] : 1e18);
        rc2i[q] = wave_uniform(real ? r * r : 0.0);
        rg = rc2i[q] > rg ? rc2i[q] : rg;
        if (tid == 0) {
            sm.row[q][0] = xi[q];
            sm.row[q][1] = yi[q];
            sm.row[q][2] = zi[q];
            sm.row[q][3] = r;
        }
    }
    rg = wave_uniform(rg);
    double acc[3 * ROWS_G] = {};
    int32_t bad = 0;
    __syncthreads();

    auto column = [&](int j0, RowsColumn v) {
        const int j = j0 + tid;
        if (j >= n) v.m = 0.0;
        // (the rows of team 0 meet every column)
        if (r0 == 0 && !(v.rc >= 0.0 && v.rc < INFINITY)) bad |= ST_RCRIT;
        rows_column(sm, xi, yi, zi, rc2i, rg, n, r0, j, v.x, v.y, v.z, v.m, v.rc, c53,
                    (j0 >> 6) + w, lane, bad, acc);
    };
    for (int j0 = 0; j0 < n; j0 += 512) {
        B = rows_load(c, n, j0 + 256 + tid);
        column(j0, A);
        if (j0 + 256 >= n) break;
        A = rows_load(c, n, j0 + 512 + tid);
        column(j0 + 256, B);
    }
    if (bad) atomicOr(status, bad);
    // 12 sums over the wave: two halvings, then the 16 lanes of a row; row h
    // of the wave ends with the sums of row group member h
    double v[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = halve32(acc[k], acc[k + 6]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double s = row16_sum(halve16(v[k], v[k + 3]));
        if ((lane & 15) == 0) sm.part[w][(lane >> 4) * 3 + k] = s;
    }
    __syncthreads();
    // marked pairs: wave w takes row w, first its crowded words, then a lane the
    // words l, l + 64 of the others
    {
        const int q = w, i = r0 + w < n ? r0 + w : n - 1;
        const double Xi = sm.row[q][0], Yi = sm.row[q][1], Zi = sm.row[q][2], ri = sm.row[q][3];
        double sx = 0.0, sy = 0.0, sz = 0.0;
        int cnt = 0;
        bool seen = false;
        auto pair = [&](const RowsColumn &v) {
            const double dx = v.x - Xi, dy = v.y - Yi, dz = v.z - Zi;
            const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
            const double wk = close_weight(r2, rho2_of(ri, v.rc), v.m);
            sx = __builtin_fma(dx, wk, sx);
            sy = __builtin_fma(dy, wk, sy);
            sz = __builtin_fma(dz, wk, sz);
        };
        crowded_words(
            sm.bits[q], nw, [&](int j) { return rows_load(c, n, j); },
            [&](int, const RowsColumn &v) { pair(v); });
        for (int k = lane; k < nw; k += 64) {
            uint64_t b = sm.bits[q][k];
            if (!b) continue;
            seen = true;
            const int first = i + 1 - k * 64;   // bit of column i + 1
            const uint64_t after = first <= 0 ? b : (first > 63 ? 0 : b & (~0ull << first));
            sm.bits[q][k] = after;
            cnt += __popcll(after);
            if (__popcll(b) >= ROWS_CROWD) continue;
            while (b) {
                pair(rows_load(c, n, k * 64 + __ffsll((unsigned long long)b) - 1));
                b &= b - 1;
            }
        }
        if (__any(seen)) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                sx += __shfl_xor(sx, off);
                sy += __shfl_xor(sy, off);
                sz += __shfl_xor(sz, off);
                cnt += __shfl_xor(cnt, off);
            }
        }
        if (lane == 0) {
            sm.slow[q][0] = sx;
            sm.slow[q][1] = sy;
            sm.slow[q][2] = sz;
            sm.cnt[q] = cnt;
        }
    }
    __syncthreads();
    if (tid < ROWS_G) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double t = ((sm.part[0][3 * tid + k] + sm.part[1][3 * tid + k]) +
                              sm.part[2][3 * tid + k]) + sm.part[3][3 * tid + k];
            a3[k] = t + sm.slow[tid][k];
        }
    }
}

}  // namespace genga
