// Symplectic levels of the base step (GENGA II Sect. 6.2, higher-level
// changeover functions; Appendix A, the recursive encounter routine).
//
// The bodies of an encounter list are advanced, instead of their Kepler
// drift, by sub-steps of a shorter time step: new critical radii (eq. rcrit
// with the sub-step), a kick over the list's pairs with the level weight
//   W_l(r) = prod_{k<l} (1 - K(r; rho_k)) * K(r; rho_l),
// the drift of the list's bodies, and the same kick again; the pairs that are
// closer than the level's critical radius form the next level's list, whose
// bodies are advanced one level deeper instead of that drift.
//
// Everything is sparse over the lists and runs on the device with fixed grids
// that read the list sizes from device memory, so a step has a fixed launch
// sequence (no host synchronisation; capturable).  Lists stay in the
// canonical order (i ascending, then j): the next level's list is a
// stream compaction of the upper one (block counts, then ordered
// writes).  For the kicks every list gets an adjacency structure whose
// partners are sorted ascending per body, so each body adds its pair terms in
// a fixed order and no floating-point atomics are used.
#include <algorithm>
#include <climits>
#include <mutex>

#include "device_common.h"
#include "genga_internal.h"
#include "kepler.h"

namespace genga {

namespace {

constexpr int LT = 256;     // threads per block of the list kernels
constexpr int LG = 1024;    // blocks of the grid-stride list kernels
constexpr int GROUP_BLOCK = 512;   // largest group of the one-workgroup class
constexpr int DB = 256;     // blocks (and chunks) of the list compaction

__device__ __forceinline__ int64_t list_len(const int64_t *cnt, int64_t cap)
{
    const int64_t c = *cnt;
    return c < cap ? c : cap;
}

__device__ __forceinline__ double rho_of(const double *rc, int64_t i, int64_t j)
{
    return rc[i] > rc[j] ? rc[i] : rc[j];
}

// Squared separation with the encounter predicate's operation order.
__device__ __forceinline__ double sep2(const double *x, const double *y, const double *z,
                                       int64_t i, int64_t j)
{
    const double dx = x[j] - x[i], dy = y[j] - y[i], dz = z[j] - z[i];
    return __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
}

__global__ __launch_bounds__(64) void k_level_begin(int64_t *lcount, int L, const int64_t *cnt0,
                                                    int64_t *gstats, int64_t *coll_count)
{
    const int t = threadIdx.x;
    if (t < L) lcount[t] = t == 0 ? *cnt0 : 0;
    if (gstats && t < 2) gstats[t] = 0;
    if (coll_count && t == 0) *coll_count = 0;
}

// E_0 to the caller's list: min(count, capacities) entries and the true count.
__global__ __launch_bounds__(LT) void k_copy_pairs(const int32_t *si, const int32_t *sj,
                                                   const int64_t *scnt, int64_t scap, int32_t *di,
                                                   int32_t *dj, int64_t dcap, int64_t *dcnt,
                                                   int32_t *status)
{
    const int64_t c = *scnt;
    int64_t m = c < scap ? c : scap;
    if (m > dcap) m = dcap;
    const int64_t t0 = (int64_t)blockIdx.x * LT + threadIdx.x;
    for (int64_t p = t0; p < m; p += (int64_t)gridDim.x * LT) {
        di[p] = si[p];
        dj[p] = sj[p];
    }
    if (t0 == 0) {
        *dcnt = c;
        if (c > dcap) atomicOr(status, ST_OVERFLOW);
    }
}

// The bodies that a list kernel runs over: a list, or (bodies null) all n.
struct ListDev {
    const int32_t *bodies;
    const int32_t *nbod;
    int64_t n;
};

__device__ __forceinline__ int64_t list_count(const ListDev &a) { return a.bodies ? *a.nbod : a.n; }
__device__ __forceinline__ int32_t list_body(const ListDev &a, int64_t q)
{
    return a.bodies ? a.bodies[q] : (int32_t)q;
}

// ---------------------------------------------------------------------------
// Adjacency of a list: degrees, a segment of the partner array per body, fill
// in arrival order, and placement of each entry at its rank among the body's
// partners (so every segment is sorted ascending).
// ---------------------------------------------------------------------------
struct AdjDev {
    int32_t *deg;             // [n] degrees
    int32_t *start;           // [n] first entry of the body's segment; [n]: entries of the list
    int32_t *bodies, *nbod;   // the list's bodies
    int64_t n;
};

// Everything of the list is empty before its degrees are counted.
__device__ __forceinline__ void adj_begin(const AdjDev &A)
{
    A.start[A.n] = 0;
    *A.nbod = 0;
}

// atomicAdd(ctr + key, 1) by the active lanes, equal keys of neighbouring lanes
// (a list's pairs of one body i) by one atomic; returns such a slot.
__device__ __forceinline__ int32_t run_add(int32_t *ctr, int32_t key)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long on = __ballot(true);
    const int32_t prev = __shfl_up(key, 1, 64);
    const bool head = lane == 0 || !((on >> (lane - 1)) & 1) || prev != key;
    const unsigned long long heads = __ballot(head) | ~on;   // (an inactive lane ends a run)
    const unsigned long long upto = heads & on & (~0ull >> (63 - lane));
    const int lead = 63 - __builtin_clzll(upto);
    int32_t base = 0;
    if (head) {
        const unsigned long long next = lane == 63 ? 0 : heads >> (lane + 1);
        base = atomicAdd(ctr + key, next ? __builtin_ctzll(next) + 1 : 64 - lane);
    }
    return __shfl(base, lead, 64) + lane - lead;
}

__device__ __forceinline__ void adj_pair(const AdjDev &A, int32_t i, int32_t j)
{
    run_add(A.deg, i);
    atomicAdd(A.deg + j, 1);
}

__global__ __launch_bounds__(LT) void k_adj_begin(AdjDev A)
{
    const int64_t t0 = (int64_t)blockIdx.x * LT + threadIdx.x;
    for (int64_t k = t0; k < A.n; k += (int64_t)gridDim.x * LT) A.deg[k] = 0;
    if (t0 == 0) adj_begin(A);
}

__global__ __launch_bounds__(LT) void k_adj_count(const int32_t *pi, const int32_t *pj,
                                                  const int64_t *cnt, int64_t cap, AdjDev A)
{
    const int64_t m = list_len(cnt, cap);
    for (int64_t p = (int64_t)blockIdx.x * LT + threadIdx.x; p < m; p += (int64_t)gridDim.x * LT)
        adj_pair(A, pi[p], pj[p]);
}

// Segments and the list of bodies with a pair (a superset of them: `up`).
// Blocks take their shares of both by one atomic each, in the order in which they
// arrive: nothing reads the order of the bodies or of the segments.
__global__ __launch_bounds__(LT) void k_adj_alloc(ListDev up, AdjDev A)
{
    __shared__ int64_t sm[LT / 64];
    __shared__ int32_t base[2];
    const int64_t nb = list_count(up);
    for (int64_t k0 = (int64_t)blockIdx.x * LT; k0 < nb; k0 += (int64_t)gridDim.x * LT) {
        const int64_t k = k0 + threadIdx.x;
        const int32_t i = k < nb ? list_body(up, k) : 0;
        const int32_t d = k < nb ? A.deg[i] : 0;
        int64_t tot;   // (entries, bodies) in one scan
        const int64_t ex = block_excl_scan<LT>(((int64_t)d << 32) | (d > 0 ? 1 : 0), &tot, sm);
        if (threadIdx.x == 0) {
            base[0] = atomicAdd(A.start + A.n, (int32_t)(tot >> 32));
            base[1] = atomicAdd(A.nbod, (int32_t)tot);
        }
        __syncthreads();
        if (k < nb) {
            A.start[i] = base[0] + (int32_t)(ex >> 32);
            if (d > 0) A.bodies[base[1] + (int32_t)ex] = i;
            A.deg[i] = 0;   // fill counter of k_adj_fill
        }
        __syncthreads();
    }
}

// Each pair into both bodies' segments, in arrival order (owner recorded); the
// fill counters end as the degrees again.
__global__ __launch_bounds__(LT) void k_adj_fill(const int32_t *pi, const int32_t *pj,
                                                 const int64_t *cnt, int64_t cap, AdjDev A,
                                                 int32_t *tmp, int32_t *owner)
{
    const int64_t m = list_len(cnt, cap);
    for (int64_t p = (int64_t)blockIdx.x * LT + threadIdx.x; p < m; p += (int64_t)gridDim.x * LT) {
        const int32_t i = pi[p], j = pj[p];
        const int32_t si = A.start[i] + run_add(A.deg, i);
        tmp[si] = j;
        owner[si] = i;
        const int32_t sj = A.start[j] + atomicAdd(A.deg + j, 1);
        tmp[sj] = i;
        owner[sj] = j;
    }
}

// Sorted placement: an entry's rank among its body's partners (all distinct)
// is the number of smaller partners in the segment.
__global__ __launch_bounds__(LT) void k_adj_rank(AdjDev A, const int32_t *tmp, const int32_t *owner,
                                                 int32_t *adj)
{
    const int64_t total = A.start[A.n];
    for (int64_t e = (int64_t)blockIdx.x * LT + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * LT) {
        const int32_t b = owner[e], v = tmp[e];
        const int32_t s0 = A.start[b], s1 = s0 + A.deg[b];
        int32_t r = 0;
        for (int32_t q = s0; q < s1; ++q) r += tmp[q] < v;
        adj[s0 + r] = v;
    }
}

// ---------------------------------------------------------------------------
// Close-encounter groups of a list: connected components of its pair graph
// by a lock-free union-find (a root is hooked under the smaller root, so each
// group's root is its smallest body, whatever the order of the unions), then
// the sizes per root, each member's arrival number in its group, and a slot per
// group in the member array.  The solvers put a group's members into ascending
// order themselves, so no result depends on an order of arrival.
// ---------------------------------------------------------------------------
struct GroupDev {
    int32_t *parent;              // [n] union-find
    int32_t *flag;                // [n] body in the list
    int32_t *lab;                 // [n] its group's root
    int32_t *size;                // [n] members per root
    int32_t *slot;                // [n] the member's number in its group
    int32_t *start;               // [n] the root's first slot in mem
    int32_t *mem;                 // [n] members by group
    int32_t *root;                // [n] roots: of groups of 2 .. BS_GS from the front, of
                                  // GROUP_BLOCK from the back (k-th at n - 1 - k)
    int32_t *count;               // [0] small groups, [1] members, [2] medium groups
    int32_t *big;                 // optional: [0] larger groups, [1 ..] their roots
    unsigned long long *gsync;    // the grid solver's barrier state
    unsigned long long *gstats;   // groups integrated, largest of them
    int32_t limit;                // members of the largest group that a solver takes
    int64_t n;
};

// A parent read through the caches (workgroup scope) may be an older value:
// every value a body's parent ever held is still one of its ancestors (trees
// only merge) and a root's parent was itself until it was hooked, so an old
// value only makes a walk stop early, at a node that was a root; the hook's
// exchange then fails and returns the current parent.  (Reads at device
// scope, from memory, made the 65,536-body ring's unions 1.5 ms.)
__device__ __forceinline__ int32_t uf_load(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Root of x, halving the path on the way: a non-root's parent may be
// replaced by any of its ancestors (parents only point to smaller bodies and
// a non-root never becomes a root again), so plain atomic stores of the
// grandparent are safe under concurrent hooks and keep the chains short (a
// ring's chain is as long as the ring otherwise).
__device__ __forceinline__ int32_t uf_find(int32_t *parent, int32_t x)
{
    for (;;) {
        const int32_t p = uf_load(parent + x);
        if (p == x) return x;
        const int32_t gp = uf_load(parent + p);
        if (gp != p) __hip_atomic_store(parent + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = gp;
    }
}

// atomicAdd(ctr + key, 1) for every active lane; returns the old value, or
// such a slot.  While the first lane left shares its key with more than three others (the
// bodies of a large group), these take one atomic together; the rest of the
// wave then takes one each, all in flight at once.
__device__ __forceinline__ int32_t wave_add_by_key(int32_t *ctr, int32_t key, bool active)
{
    unsigned long long todo = __ballot(active);
    const int lane = threadIdx.x & 63;
    int32_t slot = 0;
    while (todo) {
        const int lead = __builtin_ctzll(todo);
        const int32_t k = __shfl(key, lead, 64);
        const unsigned long long same = __ballot(((todo >> lane) & 1) && key == k);
        if (__popcll(same) <= 4) break;
        int32_t base = 0;
        if (lane == lead) base = atomicAdd(ctr + k, __popcll(same));
        base = __shfl(base, lead, 64);
        if ((same >> lane) & 1) slot = base + __popcll(same & ((1ull << lane) - 1ull));
        todo &= ~same;
    }
    if ((todo >> lane) & 1) slot = atomicAdd(ctr + key, 1);
    return slot;
}

constexpr int BS_GS = 8;      // lanes of a small group in the direct solver

__device__ __forceinline__ void group_begin(const GroupDev &g, int32_t i)
{
    g.parent[i] = i;
    g.flag[i] = 0;
    g.size[i] = 0;
}

__device__ __forceinline__ void group_begin_all(const GroupDev &g)
{
    g.count[0] = g.count[1] = g.count[2] = 0;
    if (g.big) {
        // the grid solver's list and barrier state, fresh for its launch:
        // arrivals, abort flag, three maximum slots, three minimum slots
        g.big[0] = 0;
        for (int k = 0; k < 5; ++k) g.gsync[k] = 0;
        for (int k = 5; k < 8; ++k) g.gsync[k] = (unsigned long long)LLONG_MAX;
    }
}

__device__ __forceinline__ void group_union(const GroupDev &g, int32_t i, int32_t j)
{
    g.flag[i] = 1;
    g.flag[j] = 1;
    int32_t a0 = i, b0 = j;
    for (;;) {
        int32_t ra = uf_find(g.parent, a0), rb = uf_find(g.parent, b0);
        if (ra == rb) break;   // a common ancestor: one tree
        if (ra < rb) {
            const int32_t t = ra;
            ra = rb;
            rb = t;
        }
        // hook the larger root under the smaller (a root is the smallest
        // body of its tree, so rb < ra lies in another tree); a failed
        // exchange means ra was hooked meanwhile: go on from its current
        // parent, which the exchange returns
        const int32_t old = atomicCAS(g.parent + ra, ra, rb);
        if (old == ra) break;
        a0 = old;
        b0 = rb;
    }
}

__global__ __launch_bounds__(LT) void k_group_begin(GroupDev g)
{
    const int64_t t0 = (int64_t)blockIdx.x * LT + threadIdx.x;
    for (int64_t k = t0; k < g.n; k += (int64_t)gridDim.x * LT) group_begin(g, (int32_t)k);
    if (t0 == 0) group_begin_all(g);
}

__global__ __launch_bounds__(LT) void k_group_union(const int32_t *pi, const int32_t *pj,
                                                    const int64_t *cnt, int64_t cap, GroupDev g)
{
    const int64_t m = list_len(cnt, cap);
    for (int64_t p = (int64_t)blockIdx.x * LT + threadIdx.x; p < m; p += (int64_t)gridDim.x * LT)
        group_union(g, pi[p], pj[p]);
}

// Root of every listed body, members counted and numbered per root.
__global__ __launch_bounds__(LT) void k_group_root(ListDev up, GroupDev g)
{
    const int64_t nb = list_count(up);
    for (int64_t k0 = (int64_t)blockIdx.x * LT; k0 < nb; k0 += (int64_t)gridDim.x * LT) {
        const int64_t k = k0 + threadIdx.x;
        const int32_t i = k < nb ? list_body(up, k) : 0;
        const bool on = k < nb && g.flag[i];
        int32_t r = 0;
        if (on) {
            r = uf_find(g.parent, i);
            g.lab[i] = r;
        }
        const int32_t slot = wave_add_by_key(g.size, r, on);
        if (on) g.slot[i] = slot;
    }
}

// Slots of the groups in the member array and the lists of their roots, by one
// atomic per block and list.
__global__ __launch_bounds__(LT) void k_group_alloc(ListDev up, GroupDev g)
{
    __shared__ int64_t sm[LT / 64];
    __shared__ int32_t base[3];
    const int64_t nb = list_count(up);
    for (int64_t k0 = (int64_t)blockIdx.x * LT; k0 < nb; k0 += (int64_t)gridDim.x * LT) {
        const int64_t k = k0 + threadIdx.x;
        const int32_t i = k < nb ? list_body(up, k) : 0;
        const bool root = k < nb && g.flag[i] && g.lab[i] == i;
        const int32_t size = root ? g.size[i] : 0;
        const bool small = root && size <= BS_GS, large = size > GROUP_BLOCK;
        const bool medium = root && !small && !large;
        // (members, medium, small) in one scan
        int64_t tot;
        const int64_t ex = block_excl_scan<LT>(
            ((int64_t)size << 32) | (medium ? 1 << 16 : 0) | (small ? 1 : 0), &tot, sm);
        if (threadIdx.x == 0 && tot) {
            base[0] = atomicAdd(g.count, (int32_t)(tot & 0xffff));
            base[1] = atomicAdd(g.count + 1, (int32_t)(tot >> 32));
            base[2] = atomicAdd(g.count + 2, (int32_t)(tot >> 16 & 0xffff));
        }
        __syncthreads();
        if (root) {
            g.start[i] = base[1] + (int32_t)(ex >> 32);
            if (small) g.root[base[0] + (int32_t)(ex & 0xffff)] = i;
            if (medium) g.root[g.n - 1 - (base[2] + (int32_t)(ex >> 16 & 0xffff))] = i;
            if (large) {
                if (g.big) g.big[1 + atomicAdd(g.big, 1)] = i;
            }
        }
        // statistics of the groups that are integrated (a maximum that is
        // there already costs no atomic)
        const bool taken = root && size <= g.limit;
        if (taken && (unsigned long long)size > g.gstats[1])
            atomicMax(g.gstats + 1, (unsigned long long)size);
        const unsigned long long some = __ballot(taken);
        if (some && (threadIdx.x & 63) == 0)
            atomicAdd(g.gstats, (unsigned long long)__popcll(some));
        __syncthreads();
    }
}

// Per-body operators over a list's bodies.
struct BodyDev {
    const int32_t *bodies;
    const int32_t *nbod;
    double *x, *y, *z, *vx, *vy, *vz;
    const double *m;
    int32_t *status;
};

// What a level's pass does with its next list: nothing, its adjacency (a level
// follows) or its groups (the direct solver follows).
enum NextList { NEXT_NONE, NEXT_ADJ, NEXT_GROUPS };

// Start of a level's sub-step over the bodies of the upper list: their critical
// radii, and empty structures for the next list.
template <int NEXT>
__global__ __launch_bounds__(LT) void k_level_radii(BodyDev a, double *rc, double m_star, double dt,
                                                    double n1, double n2, AdjDev A, GroupDev g)
{
    const int64_t nb = *a.nbod;
    const int64_t t0 = (int64_t)blockIdx.x * LT + threadIdx.x;
    if (t0 == 0) {
        if (NEXT == NEXT_ADJ) adj_begin(A);
        if (NEXT == NEXT_GROUPS) group_begin_all(g);
    }
    for (int64_t q = t0; q < nb; q += (int64_t)gridDim.x * LT) {
        const int32_t i = a.bodies[q];
        const double r = __builtin_sqrt(a.x[i] * a.x[i] + a.y[i] * a.y[i] + a.z[i] * a.z[i]);
        const double v =
            __builtin_sqrt(a.vx[i] * a.vx[i] + a.vy[i] * a.vy[i] + a.vz[i] * a.vz[i]);
        const double rh = r * cbrt(a.m[i] / (3.0 * m_star));
        const double h1 = n1 * rh, h2 = n2 * fabs(dt) * v;
        const double out = h1 > h2 ? h1 : h2;
        if (!(out >= 0.0 && out < INFINITY)) atomicOr(a.status, ST_RCRIT);
        rc[i] = out;
        if (NEXT == NEXT_ADJ) A.deg[i] = 0;
        if (NEXT == NEXT_GROUPS) group_begin(g, i);
    }
}

// ---------------------------------------------------------------------------
// Next level's list: the pairs of list `in` closer than this level's
// critical radius, in the same order.  DB chunks of the input: counts (in the
// launch of the level's kick, which leaves positions and radii as they are), then
// ordered writes behind the counts of the chunks before.
// ---------------------------------------------------------------------------
struct DetectDev {
    const int32_t *in_i, *in_j;
    const int64_t *in_cnt;
    int32_t *out_i, *out_j;
    int64_t *out_cnt;
    int64_t *lcount;          // summed sizes of this level's lists
    int64_t cap;
    const double *x, *y, *z, *rc;
    int64_t *bcnt;            // [DB]
};

__device__ __forceinline__ bool detect_pair(const DetectDev &d, int32_t i, int32_t j)
{
    const double rho = rho_of(d.rc, i, j);
    return sep2(d.x, d.y, d.z, i, j) < rho * rho;
}

__device__ __forceinline__ void chunk_of(const DetectDev &d, int64_t &p0, int64_t &p1)
{
    const int64_t m = list_len(d.in_cnt, d.cap);
    const int64_t len = (m + DB - 1) / DB;
    p0 = min(m, (int64_t)blockIdx.x * len);
    p1 = min(m, p0 + len);
}

__device__ __forceinline__ void detect_count(const DetectDev &d)
{
    __shared__ int64_t sm[LT / 64];
    int64_t p0, p1;
    chunk_of(d, p0, p1);
    int64_t c = 0;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += LT) c += detect_pair(d, d.in_i[p], d.in_j[p]);
    int64_t tot;
    block_excl_scan<LT>(c, &tot, sm);
    if (threadIdx.x == 0) d.bcnt[blockIdx.x] = tot;
}

static_assert(DB == LT, "k_detect_write: a thread per chunk");

template <int NEXT>
__global__ __launch_bounds__(LT) void k_detect_write(DetectDev d, AdjDev A, GroupDev g)
{
    __shared__ int64_t sm[LT / 64];
    __shared__ int64_t before;
    int64_t p0, p1;
    chunk_of(d, p0, p1);
    int64_t all;
    const int64_t mine = block_excl_scan<DB>(d.bcnt[threadIdx.x], &all, sm);
    if (threadIdx.x == blockIdx.x) before = mine;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *d.out_cnt = all;
        *d.lcount += all;
    }
    __syncthreads();
    int64_t run = before;
    for (int64_t t0 = p0; t0 < p1; t0 += LT) {
        const int64_t p = t0 + threadIdx.x;
        const int32_t i = p < p1 ? d.in_i[p] : 0, j = p < p1 ? d.in_j[p] : 0;
        const bool f = p < p1 && detect_pair(d, i, j);
        int64_t tot;
        const int64_t ex = block_excl_scan<LT>(f ? 1 : 0, &tot, sm);
        if (f) {
            d.out_i[run + ex] = i;
            d.out_j[run + ex] = j;
            if (NEXT == NEXT_ADJ) adj_pair(A, i, j);
            if (NEXT == NEXT_GROUPS) group_union(g, i, j);
        }
        run += tot;
    }
}

// The drift of a level's bodies that no deeper list advances: the others start
// their sub-steps or their group's integration from the state they have.  (A
// group too large for every solver is drifted.)  Members go to their slots here.
template <int NEXT>
__global__ __launch_bounds__(LT) void k_drift_list(BodyDev a, double mu, double dt, AdjDev A,
                                                   GroupDev g)
{
    const int64_t nb = *a.nbod;
    for (int64_t q = (int64_t)blockIdx.x * LT + threadIdx.x; q < nb; q += (int64_t)gridDim.x * LT) {
        const int32_t i = a.bodies[q];
        if (NEXT == NEXT_ADJ && A.deg[i] > 0) continue;
        if (NEXT == NEXT_GROUPS && g.flag[i]) {
            const int32_t r = g.lab[i];
            g.mem[g.start[r] + g.slot[i]] = i;
            if (g.size[r] <= g.limit) continue;
        }
        double X = a.x[i], Y = a.y[i], Z = a.z[i], VX = a.vx[i], VY = a.vy[i], VZ = a.vz[i];
        const int st = kepler_uv(mu, dt, X, Y, Z, VX, VY, VZ);
        if (st) atomicOr(a.status, st);
        a.x[i] = X; a.y[i] = Y; a.z[i] = Z;
        a.vx[i] = VX; a.vy[i] = VY; a.vz[i] = VZ;
    }
}

// Members to their slots, their state to `shadow` (the whole system drifts next).
__global__ __launch_bounds__(LT) void k_group_place(BodyDev a, GroupDev g, double *shadow)
{
    const double *c[6] = {a.x, a.y, a.z, a.vx, a.vy, a.vz};
    for (int64_t i = (int64_t)blockIdx.x * LT + threadIdx.x; i < g.n; i += (int64_t)gridDim.x * LT) {
        if (!g.flag[i]) continue;
        g.mem[g.start[g.lab[i]] + g.slot[i]] = (int32_t)i;
#pragma unroll
        for (int k = 0; k < 6; ++k) shadow[(size_t)k * g.n + i] = c[k][i];
    }
}

// save = 1: shadow <- state; save = 0: state <- shadow (bodies of the list).
__global__ __launch_bounds__(LT) void k_state_list(BodyDev a, double *shadow, int64_t n, int save)
{
    const int64_t nb = *a.nbod;
    double *c[6] = {a.x, a.y, a.z, a.vx, a.vy, a.vz};
    for (int64_t q = (int64_t)blockIdx.x * LT + threadIdx.x; q < nb; q += (int64_t)gridDim.x * LT) {
        const int32_t i = a.bodies[q];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            if (save) shadow[(size_t)k * n + i] = c[k][i];
            else c[k][i] = shadow[(size_t)k * n + i];
        }
    }
}

// 1/x from v_rcp_f64 with a second-order correction (relative error a few
// 2^-53); a chain half as long as the IEEE division.
__device__ __forceinline__ double rcp_full(double x)
{
    const double t = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, t, 1.0);
    return __builtin_fma(t, __builtin_fma(e, e, e), t);
}

// 1 / rho for LevelWeight.  A radius of zero (a body at rest, or without mass,
// where n1 or n2 leaves nothing else) has K = 1 at every distance: its
// reciprocal is a number that takes y to 1, where rcp_full would give a NaN,
// which the clamp turns into y = 0.
__device__ __forceinline__ double rcp_radius(double rho)
{
    return rho > 1e-300 ? rcp_full(rho) : 1e300;
}

// The changeover K(y) = y^2 / (2 y^2 - 2 y + 1) of y = (r / rho - 0.1) / 0.9 in
// [0, 1], as num^2 / den: `up` takes y for a factor K and 1 - y for a factor
// 1 - K, so that a product over levels needs one reciprocal.
struct LevelWeight {
    double num = 1.0, den = 1.0;
    __device__ void add(double r, double irho, bool up)
    {
        double y = __builtin_fma(r * irho, 10.0 / 9.0, -1.0 / 9.0);
        y = vmin_f64(vmax_f64(y, 0.0), 1.0);
        num *= up ? y : 1.0 - y;
        den *= __builtin_fma(2.0 * y, y - 1.0, 1.0);
    }
    __device__ double value() const { return (num * num) * rcp_full(den); }
};

// Kick of level l over a list: v_b += h G sum_j m_j W_l(r_bj) (x_j - x_b) / r^3
// for every body b of the list.  A group of GL lanes takes one body: lane u
// adds the partners u, u + GL, ... of the body's ascending partner list, and
// the GL partial sums are combined by a fixed butterfly, so the result does
// not depend on scheduling.  Bound by its dependent loads (body, segment,
// partner, its state) and the chain of one pair, hence the corrected hardware
// estimates, the level as a template argument (all radii in flight at once)
// and one reciprocal for all levels (65,536 bodies, level 2 of 3 x 4: 8 -> 6-7
// us per launch; level 1, 235,000 pairs: 24-27 us, mostly gathers).
constexpr int GL = 8;
constexpr int KB_DETECT = DB;   // blocks in front that count the next list

struct LevelKickDev {
    BodyDev a;
    const int32_t *start, *deg, *adj;
    const double *rc[GENGA_MAX_LEVELS];   // rc[0]: level 0 (the bodies' rc)
    double G, h;
};

template <int LEVEL, bool DETECT>
__global__ __launch_bounds__(LT) void k_level_kick(LevelKickDev k, DetectDev d)
{
    if (DETECT && blockIdx.x < KB_DETECT) {
        detect_count(d);
        return;
    }
    const unsigned bx = DETECT ? blockIdx.x - KB_DETECT : blockIdx.x;
    const unsigned blocks = DETECT ? gridDim.x - KB_DETECT : gridDim.x;
    const BodyDev &a = k.a;
    const int64_t nb = *a.nbod;
    const int u = threadIdx.x & (GL - 1);
    const int64_t g0 = ((int64_t)bx * LT + threadIdx.x) / GL;
    const int64_t gstride = (int64_t)blocks * (LT / GL);
    // every lane of a group runs the same trip count (the body loop is
    // uniform per group), so the butterfly below sees all GL lanes
    for (int64_t q = g0; q < nb; q += gstride) {
        const int32_t b = a.bodies[q];
        const double xb = a.x[b], yb = a.y[b], zb = a.z[b];
        double rb[LEVEL + 1];
#pragma unroll
        for (int l = 0; l <= LEVEL; ++l) rb[l] = k.rc[l][b];
        double ax = 0.0, ay = 0.0, az = 0.0;
        const int32_t e0 = k.start[b], e1 = e0 + k.deg[b];
        for (int32_t e = e0 + u; e < e1; e += GL) {
            const int32_t j = k.adj[e];
            const double dx = a.x[j] - xb, dy = a.y[j] - yb, dz = a.z[j] - zb;
            double rho[LEVEL + 1];
#pragma unroll
            for (int l = 0; l <= LEVEL; ++l) rho[l] = vmax_f64(rb[l], k.rc[l][j]);
            const double mj = a.m[j];
            const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
            if (r2 == 0.0) {
                atomicOr(a.status, ST_NONFINITE);
                continue;
            }
            const double ir = rsq_full(r2), r = r2 * ir;
            LevelWeight w;
#pragma unroll
            for (int l = 0; l <= LEVEL; ++l)
                w.add(r, rcp_radius(rho[l]), l == LEVEL);
            const double s = (k.G * mj) * w.value() * (ir * ir * ir);
            ax = __builtin_fma(s, dx, ax);
            ay = __builtin_fma(s, dy, ay);
            az = __builtin_fma(s, dz, az);
        }
#pragma unroll
        for (int o = GL / 2; o > 0; o >>= 1) {
            ax += __shfl_xor(ax, o, GL);
            ay += __shfl_xor(ay, o, GL);
            az += __shfl_xor(az, o, GL);
        }
        if (u == 0) {
            a.vx[b] += k.h * ax;
            a.vy[b] += k.h * ay;
            a.vz[b] += k.h * az;
        }
    }
}

// ---------------------------------------------------------------------------
// Direct solver: one thread per member; groups of up to 8 bodies take 8 lanes
// of a wave each, larger ones a workgroup of 512 threads (Table 1 splits them
// into more classes up to 512 bodies; here they are rare, and 512 threads
// hold the extrapolation tableau in registers at 2 waves per SIMD with 125 KB
// of LDS).  The
// group's flow (Kepler force of the star plus the remainder R of the mutual
// forces) is integrated over H by Bulirsch-Stoer steps: the modified
// midpoint rule with n = 2, 4, ..., 2 KM sub-steps, polynomial extrapolation
// in (h/n)^2 (Neville), a step accepted when the last two extrapolations
// agree within eps (relative to each member's position and velocity
// magnitudes), else retried with half the step; after a step that converged
// early the next one doubles (never beyond what is left of H).
// ---------------------------------------------------------------------------
constexpr int KM = 8;
constexpr int BS_TRIES = 4096;

struct BsDev {
    int32_t *groot;                     // (each block of k_bs reorders its own medium ones)
    const int32_t *gstart, *gsize, *gmem, *gcount;
    const double *state[6];             // x, y, z, vx, vy, vz before the drift
    int64_t n;
    double *x, *y, *z, *vx, *vy, *vz;
    double *m;                          // written by mergers
    const double *rc[GENGA_MAX_LEVELS]; // levels 0 .. nlev - 1 weigh R
    int nlev;
    double G, mu, H, eps;
    int32_t *status;
    // collisions (radius non-null): radii (written by mergers), contact
    // tolerance, records (survivor, absorbed, lost energy)
    double *radius;
    double coll_tol;
    int32_t *coll_i, *coll_j;
    double *coll_du;
    unsigned long long *coll_count;
    int64_t coll_cap;
};

// R = prod_l (1 - K(r; rho_l)) with irho_l = 1 / rho_l = min(1 / rc_i, 1 / rc_j).
// The members' reciprocal critical radii are formed once per group (the radii
// do not change during the integration) and read from LDS: level l of member i at
// ia[l * sa], of member j at ib[l * sb].  NL: the number of levels (straight code:
// the serial chain of the group derivative is dominated by latency), or 0.
template <int NL>
__device__ __forceinline__ double bs_remainder(double r, const double *ia, int sa,
                                               const double *ib, int sb, int nlev)
{
    LevelWeight w;
    if constexpr (NL > 0) {
#pragma unroll
        for (int l = 0; l < NL; ++l) w.add(r, vmin_f64(ia[l * sa], ib[l * sb]), false);
    } else {
        for (int l = 0; l < nlev; ++l) w.add(r, vmin_f64(ia[l * sa], ib[l * sb]), false);
    }
    return w.value();
}

__device__ __forceinline__ double wave_min_all(double v)
{
    for (int d = 32; d > 0; d >>= 1) {
        const double o = __shfl_xor(v, d, 64);
        v = o < v ? o : v;
    }
    return v;
}

__device__ __forceinline__ double wave_max_all(double v)
{
    for (int d = 32; d > 0; d >>= 1) {
        const double o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Smallest and largest of a coordinate over the lanes that take part, as
// bounds in binary32 (rounded outwards) by DPP moves within the wave: a
// butterfly of binary64 shuffles costs ten times as much, and a box that is
// 2^-23 too large only keeps a tile whose terms are zeros.  NaN is ignored (a
// member at NaN fails the step by its own error).
__device__ __forceinline__ float wave_min_dpp(float v)
{
#define BS_DPP_MIN(ctrl, rows)                                                                     \
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(                                       \
                     __float_as_int(v), __float_as_int(v), ctrl, rows, 0xf, false)))
    BS_DPP_MIN(0x111, 0xf);   // row_shr:1, 2, 4, 8
    BS_DPP_MIN(0x112, 0xf);
    BS_DPP_MIN(0x114, 0xf);
    BS_DPP_MIN(0x118, 0xf);
    BS_DPP_MIN(0x142, 0xa);   // row_bcast:15, 31
    BS_DPP_MIN(0x143, 0xc);
#undef BS_DPP_MIN
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ void wave_bounds(double x, bool in, double &lo, double &hi)
{
    const float f = (float)x, e = fabsf(f) * 0x1p-23f + 1e-37f;
    lo = (double)wave_min_dpp(in ? f - e : INFINITY);
    hi = -(double)wave_min_dpp(in ? -f - e : INFINITY);
}

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Squared gap between the box (lo, hi) and the box B = (lo, hi) of another
// tile: a lower bound of the squared distance of any two of their members.
__device__ __forceinline__ double box_gap2(const double lo[3], const double hi[3], const double *B)
{
    double d2 = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double a1 = B[c] - hi[c], a2 = lo[c] - B[3 + c];
        const double gc = a1 > a2 ? a1 : a2;
        d2 += gc > 0.0 ? gc * gc : 0.0;
    }
    return d2;
}

// Pairs in reach that a wave keeps before it evaluates them.
constexpr int BS_ENT = 256;

template <int BT>
struct BsSmem {
    double px[BT], py[BT], pz[BT], m[BT];
    double pv[3][BT], R[BT];
    alignas(16) int32_t cell[BT];       // bs_cell of the positions
    uint32_t ent[BT / 64][BS_ENT];      // each wave's pairs in reach: member lane, partner
    double fo[BT / 64][3][BS_ENT];      // and their terms
    double box[BT / 64][8];             // each wave's box of its members' positions
    double trho[BT / 64];               // each wave's largest deepest-level rc
    int32_t idx[BT];
    double irc[GENGA_MAX_LEVELS][BT];   // 1 / rc of each level
    double red[BT / 64];
    long long ired[BT / 64];
};

// The partners in reach of 64 members are found first and evaluated after.
// Evaluated where they are found, a partner that any lane needs costs the
// whole wave a remainder (a chain of several hundred cycles): 15 us for an
// evaluation of 230 members with about 4 partners each.  Found as the bits of
// each lane and written down as (member, partner) entries, they are shared
// out over the lanes, one remainder per lane and pass, and each member then
// adds its terms in ascending order.
//
// The workgroup's search uses the group's x-y plane as a grid of 16,000 cells
// along its longer side, a pair of 16-bit coordinates per member: one
// difference, one 16-bit dot product and one compare per partner, four
// partners to an LDS read.  Rounding moves a coordinate by at most half a
// cell, and clamping to the frame only brings members closer, so a pair
// inside the larger deepest-level radius is within that radius plus 2 cells;
// beyond the radius R = 0 exactly, so the pairs found in vain add exact zeros.
typedef short bs_s16x2 __attribute__((ext_vector_type(2)));

struct BsFrame {
    double x0, y0, scale;
};

__device__ __forceinline__ int32_t bs_cell(const BsFrame &f, double x, double y)
{
    const double cx = __builtin_fmin(__builtin_fmax((x - f.x0) * f.scale, 0.0), 16000.0);
    const double cy = __builtin_fmin(__builtin_fmax((y - f.y0) * f.scale, 0.0), 16000.0);
    return (int)(cx + 0.5) | ((int)(cy + 0.5) << 16);
}

// `bits` with the test of one more partner shifted in from below: in reach iff
// d.d - (reach2 + 1) is negative, whose sign bit the funnel shift takes (three
// instructions a partner; compare, select and or into a 64-bit mask took 65 cycles).
__device__ __forceinline__ uint32_t bs_cell_test(uint32_t bits, int32_t a, int32_t b, int far2)
{
    const bs_s16x2 d = __builtin_bit_cast(bs_s16x2, a) - __builtin_bit_cast(bs_s16x2, b);
    const int q = __builtin_amdgcn_sdot2(d, d, far2, false);
    return __builtin_amdgcn_alignbit(bits, (uint32_t)q, 31);
}

// Exclusive sum over the lanes of a wave and the total (small counts).
__device__ __forceinline__ int wave_excl_sum(int v, int &total)
{
    int s = v;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xf, 0xf, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xf, 0xf, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xf, 0xf, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xa, 0xf, false);   // row_bcast:15, 31
    s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xc, 0xf, false);
    total = __builtin_amdgcn_readlane(s, 63);
    return s - v;
}

// A wave's entries.  Each round a lane adds up to 4; where they went is kept
// in `where` (base and count, 16 bits a round, up to 4 rounds).
struct BsEntries {
    int total = 0, rounds = 0;
    uint64_t where = 0;
};

// Partner sum of the wave's members (lane's member t, at position o) from the
// positions in LDS, over share `sub` of S: every partner wave's S-th part that
// `sub` names.  A partner wave whose box stays beyond the larger deepest-level
// critical radius of the two waves from the own wave's box holds no partner
// with R > 0 and is skipped.  All lanes of the wave pass here.
template <int BT, int NL>
__device__ __forceinline__ void bs_accel(const BsDev &a, BsSmem<BT> &sm, const BsFrame &fr, int t,
                                         int g, int S, int sub, double rcd, double acc[3])
{
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int t0 = t - lane;
    const double *BI = sm.box[t0 >> 6];
    const double lo[3] = {BI[0], BI[1], BI[2]}, hi[3] = {BI[3], BI[4], BI[5]};
    const int nw = (g + 63) >> 6;
    const double rhoI = sm.trho[t0 >> 6];
    const int32_t me = sm.cell[t < g ? t : 0];
    uint32_t *ent = sm.ent[w];
    double(*fo)[BS_ENT] = sm.fo[w];
    BsEntries E;
    auto flush = [&]() {
        wave_sync_lds();
        for (int p = lane; p < E.total; p += 64) {
            const uint32_t e = ent[p];
            const int i = t0 + (int)(e >> 16), q = (int)(e & 0xffffu);
            const double dx = sm.px[q] - sm.px[i], dy = sm.py[q] - sm.py[i],
                         dz = sm.pz[q] - sm.pz[i];
            const double r2 = dx * dx + dy * dy + dz * dz;
            const double ir = rsq_full(r2);
            const double R = bs_remainder<NL>(r2 * ir, &sm.irc[0][i], BT, &sm.irc[0][q], BT, a.nlev);
            const double s = a.G * sm.m[q] * R * (ir * ir * ir);
            fo[0][p] = s * dx;
            fo[1][p] = s * dy;
            fo[2][p] = s * dz;
        }
        wave_sync_lds();
        for (int r = 0; r < E.rounds; ++r) {
            const int at = (int)(E.where >> (16 * r)) & 0xffff;
            const int p0 = at >> 3, c = at & 7;
            for (int k = 0; k < c; ++k) {
                acc[0] += fo[0][p0 + k];
                acc[1] += fo[1][p0 + k];
                acc[2] += fo[2][p0 + k];
            }
        }
        wave_sync_lds();
        E = BsEntries();
    };
    // Up to 64 partners as the bits of one mask: a part of one tile, or the
    // parts of two tiles (S = 2, 4) in its halves
    const int per = 64 / S, u0 = sub * per;
    uint64_t mask = 0;
    int part = 0, first[2] = {0, 0};   // parts in the mask, first partner of each
    auto emit = [&]() {
        const int shift = first[1] - 32;
        while (__any(mask != 0)) {
            const int pc = __popcll(mask), c = pc < 4 ? pc : 4;
            int sum;
            const int off = wave_excl_sum(c, sum);
            if (E.rounds == 4 || E.total + sum > BS_ENT) flush();
            const int base = E.total + off;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (k < c) {
                    const int b = __builtin_ctzll(mask);
                    ent[base + k] = (uint32_t)(lane << 16) | (uint32_t)(b + (b < 32 ? first[0] : shift));
                    mask &= mask - 1;
                }
            }
            E.where |= (uint64_t)(base << 3 | c) << (16 * E.rounds);
            E.total += sum;
            ++E.rounds;
        }
        mask = 0;
        part = 0;
    };
    for (int J = 0; J < nw; ++J) {
        const double rr = rhoI > sm.trho[J] ? rhoI : sm.trho[J];
        if (box_gap2(lo, hi, sm.box[J]) > rr * rr * (1.0 + 0x1p-18)) continue;
        const double re = (rcd > sm.trho[J] ? rcd : sm.trho[J]) * fr.scale + 2.0;
        const int far2 = -1 - (int)__builtin_fmin(re * re + 1.0, 1e9);
        const int4 *cells = (const int4 *)&sm.cell[J * 64 + u0];
        // words of up to 32 partners, the first in the lowest bit
        auto word = [&](int v0, int cnt) {
            uint32_t bits = 0;
#pragma unroll 2
            for (int v = v0; v < v0 + cnt; v += 4) {
                const int4 c = cells[v >> 2];
                bits = bs_cell_test(bits, me, c.x, far2);
                bits = bs_cell_test(bits, me, c.y, far2);
                bits = bs_cell_test(bits, me, c.z, far2);
                bits = bs_cell_test(bits, me, c.w, far2);
            }
            bits = __brev(bits) >> (32 - cnt);
            const int j0 = J * 64 + u0 + v0;
            if (g - j0 < 32) bits &= g > j0 ? (1u << (g - j0)) - 1 : 0u;
            if (J * 64 == t0 && (unsigned)(t - j0) < 32u) bits &= ~(1u << (t - j0));
            return t < g ? bits : 0u;
        };
        first[part] = J * 64 + u0;
        if (S == 1) {
            mask = word(0, 32) | (uint64_t)word(32, 32) << 32;
            first[1] = first[0] + 32;
            emit();
        } else {
            mask |= (uint64_t)word(0, per) << (32 * part);
            if (++part == 2) emit();
        }
    }
    emit();
    if (E.total) flush();
}

// The same sums, term by term and in the same order, with each partner
// evaluated where it is met, for groups whose members want most of it: a search finds
// nearly every partner then, and an entry's way through LDS costs about as much as
// its remainder.  Rings whose members all meet, us a step, entries / in place:
// 40 bodies 260 / 212, 100 615 / 434, 150 1,357 / 870, 512 8,640 / 4,530.
template <int BT, int NL>
__device__ __forceinline__ void bs_accel_whole(const BsDev &a, const BsSmem<BT> &sm, int t, int g,
                                               int S, int sub, double rcd, double acc[3])
{
    const int t0 = t - (int)(threadIdx.x & 63), i = t < g ? t : 0;
    const double *BI = sm.box[t0 >> 6];
    const double lo[3] = {BI[0], BI[1], BI[2]}, hi[3] = {BI[3], BI[4], BI[5]};
    const double rhoI = sm.trho[t0 >> 6];
    const double x = sm.px[i], y = sm.py[i], z = sm.pz[i];
    const int per = 64 / S;
    for (int J = 0; J * 64 < g; ++J) {
        const double rJ = sm.trho[J], rr = rhoI > rJ ? rhoI : rJ;
        if (box_gap2(lo, hi, sm.box[J]) > rr * rr * (1.0 + 0x1p-18)) continue;
        const double re = rcd > rJ ? rcd : rJ;
        const double far2 = t < g ? re * re * (1.0 + 0x1p-18) : -1.0;
        const int q0 = J * 64 + sub * per, q1 = g < q0 + per ? g : q0 + per;
#pragma unroll 1
        for (int q = q0; q < q1; ++q) {
            const double dx = sm.px[q] - x, dy = sm.py[q] - y, dz = sm.pz[q] - z;
            const double r2 = dx * dx + dy * dy + dz * dz;
            if (q == t || r2 > far2) continue;
            const double ir = rsq_full(r2);
            const double R = bs_remainder<NL>(r2 * ir, &sm.irc[0][i], BT, &sm.irc[0][q], BT, a.nlev);
            const double s = a.G * sm.m[q] * R * (ir * ir * ir);
            acc[0] += s * dx;
            acc[1] += s * dy;
            acc[2] += s * dz;
        }
    }
}

// Publish positions (and each wave's box), then every member's derivative
// at them: the star's pull plus the S shares' partner sums, added in share
// order (the waves of a share hold copies of the same members; only share 0
// writes).  The shares' sums pass through pv, which no evaluation uses.
template <int BT, int NL, bool WHOLE>
__device__ __forceinline__ void bs_deriv(const BsDev &a, BsSmem<BT> &sm, const BsFrame &fr, int t,
                                         int g, int S, int sub, double rcd, const double z[6],
                                         double f[6])
{
    __syncthreads();   // the previous evaluation has finished reading
    const bool mem = t < g, own = mem && sub == 0;
    if (own) {
        sm.px[t] = z[0];
        sm.py[t] = z[1];
        sm.pz[t] = z[2];
        if (!WHOLE) sm.cell[t] = bs_cell(fr, z[0], z[1]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double lo, hi;
        wave_bounds(z[c], mem, lo, hi);
        if ((threadIdx.x & 63) == 0 && own) {
            sm.box[t >> 6][c] = lo;
            sm.box[t >> 6][3 + c] = hi;
        }
    }
    __syncthreads();
    f[0] = z[3];
    f[1] = z[4];
    f[2] = z[5];
    double p[3] = {0.0, 0.0, 0.0};
    if (t - (int)(threadIdx.x & 63) < g) {
        if constexpr (WHOLE)
            bs_accel_whole<BT, NL>(a, sm, t, g, S, sub, rcd, p);
        else
            bs_accel<BT, NL>(a, sm, fr, t, g, S, sub, rcd, p);
    }
    double k[3] = {0.0, 0.0, 0.0};
    if (mem) {
        const double r2s = z[0] * z[0] + z[1] * z[1] + z[2] * z[2];
        const double irs = rsq_full(r2s);
        const double ks = -a.mu * (irs * irs * irs);
        k[0] = ks * z[0];
        k[1] = ks * z[1];
        k[2] = ks * z[2];
    }
    if (S > 1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) sm.pv[c][threadIdx.x] = p[c];
        __syncthreads();
        const int w0 = (threadIdx.x >> 6) - sub, lane = threadIdx.x & 63;
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) k[c] += sm.pv[c][(w0 + s) * 64 + lane];
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) k[c] += p[c];
    }
    f[3] = k[0];
    f[4] = k[1];
    f[5] = k[2];
}

template <int BT>
__device__ __forceinline__ double bs_block_max(BsSmem<BT> &sm, double v)
{
    for (int d = 32; d > 0; d >>= 1) {
        const double o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm.red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = sm.red[0];
#pragma unroll
    for (int w = 1; w < BT / 64; ++w) r = sm.red[w] > r ? sm.red[w] : r;
    return r;
}

// How the members of a group see each other: a workgroup with the positions
// in LDS (BlockPol), or GS lanes of one wave exchanging them by shuffles
// (LanePol, several small groups per wave and no barriers).
// Both policies also expose, for the collision search and the merger: the
// whole state of member q after publish(), its mass, radius and body index,
// a group-wide minimum of an integer key, and updates of the own member's
// mass and radius.
template <int BT, int NL, bool WHOLE>
struct BlockPol {
    BsSmem<BT> &sm;
    int t, g;
    int S, sub;   // waves per member (the group's shares), this wave's share
    double rcd;   // own deepest-level rc
    BsFrame fr;   // the group's plane (bs_cell)
    __device__ void deriv(const BsDev &a, const double z[6], double f[6])
    {
        bs_deriv<BT, NL, WHOLE>(a, sm, fr, t, g, S, sub, rcd, z, f);
    }
    __device__ double gmax(double v) { return bs_block_max<BT>(sm, v); }
    __device__ bool member() const { return t < g; }
    __device__ bool owner() const { return t < g && sub == 0; }
    __device__ int self() const { return t; }
    __device__ long long overlap(const BsDev &a, const double z[6]);
    __device__ void publish(const double z[6])
    {
        __syncthreads();
        if (owner()) {
            sm.px[t] = z[0];
            sm.py[t] = z[1];
            sm.pz[t] = z[2];
            sm.pv[0][t] = z[3];
            sm.pv[1][t] = z[4];
            sm.pv[2][t] = z[5];
        }
        __syncthreads();
    }
    __device__ void get(int q, double o[6]) const
    {
        o[0] = sm.px[q];
        o[1] = sm.py[q];
        o[2] = sm.pz[q];
        o[3] = sm.pv[0][q];
        o[4] = sm.pv[1][q];
        o[5] = sm.pv[2][q];
    }
    __device__ double mass(int q) const { return sm.m[q]; }
    __device__ double rad(int q) const { return sm.R[q]; }
    __device__ int idx(int q) const { return sm.idx[q]; }
    __device__ void set_own(double m, double R)
    {
        if (owner()) {
            sm.m[t] = m;
            sm.R[t] = R;
        }
    }
    __device__ long long gmin(long long v)
    {
        for (int d = 32; d > 0; d >>= 1) {
            const long long o = __shfl_xor(v, d, 64);
            v = o < v ? o : v;
        }
        __syncthreads();
        if ((threadIdx.x & 63) == 0) sm.ired[threadIdx.x >> 6] = v;
        __syncthreads();
        long long r = sm.ired[0];
#pragma unroll
        for (int w = 1; w < BT / 64; ++w) r = sm.ired[w] < r ? sm.ired[w] : r;
        return r;
    }
};

template <int GS, int NL>
struct LanePol {
    int u, g;
    double m, R;
    int32_t bidx;
    double zc[6];
    const double *irc;   // 1 / rc of each level: LDS, level l at irc[l * stride]; lane q at + q - u
    static constexpr int stride = GROUP_BLOCK;
    __device__ bool member() const { return u < g; }
    __device__ bool owner() const { return true; }
    __device__ int self() const { return u; }
    __device__ long long overlap(const BsDev &a, const double z[6]);
    __device__ void publish(const double z[6])
    {
#pragma unroll
        for (int c = 0; c < 6; ++c) zc[c] = z[c];
    }
    __device__ void get(int q, double o[6]) const
    {
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = __shfl(zc[c], q, GS);
    }
    __device__ double mass(int q) const { return __shfl(m, q, GS); }
    __device__ double rad(int q) const { return __shfl(R, q, GS); }
    __device__ int idx(int q) const { return __shfl(bidx, q, GS); }
    __device__ void set_own(double mm, double RR)
    {
        if (u < g) {
            m = mm;
            R = RR;
        }
    }
    __device__ long long gmin(long long v)
    {
        for (int d = GS / 2; d > 0; d >>= 1) {
            const long long o = __shfl_xor(v, d, GS);
            v = o < v ? o : v;
        }
        return v;
    }
    // lane u takes the partners u + 1, u + 2, ... around the group, so that every
    // member works on each pass of the loop (a group of two: one pass); the
    // lanes beyond the group compute values that nothing reads
    __device__ void deriv(const BsDev &a, const double z[6], double f[6])
    {
        f[0] = z[3];
        f[1] = z[4];
        f[2] = z[5];
        const double irs = rsq_full(z[0] * z[0] + z[1] * z[1] + z[2] * z[2]);
        const double ks = -a.mu * (irs * irs * irs);
        double acc[3] = {ks * z[0], ks * z[1], ks * z[2]};
        for (int k = 1; k < g; ++k) {
            int q = u + k;
            q = q >= g ? q - g : q;
            const double xq = __shfl(z[0], q, GS), yq = __shfl(z[1], q, GS),
                         zq = __shfl(z[2], q, GS), mq = __shfl(m, q, GS);
            const double dx = xq - z[0], dy = yq - z[1], dz = zq - z[2];
            const double r2 = dx * dx + dy * dy + dz * dz;
            const double ir = rsq_full(r2);
            const double R = bs_remainder<NL>(r2 * ir, irc, stride, irc + (q - u), stride, a.nlev);
            const double s = a.G * mq * R * (ir * ir * ir);
            acc[0] += s * dx;
            acc[1] += s * dy;
            acc[2] += s * dz;
        }
        f[3] = acc[0];
        f[4] = acc[1];
        f[5] = acc[2];
    }
    __device__ double gmax(double v)
    {
        for (int d = GS / 2; d > 0; d >>= 1) {
            const double o = __shfl_xor(v, d, GS);
            v = o > v ? o : v;
        }
        return v;
    }
};

// One Bulirsch-Stoer step of length h from y: the modified midpoint rule
// with n = 2, 4, ..., 2 KM sub-steps and Neville's extrapolation (the tableau
// updated in place, the loop over the sequence unrolled so that it stays in
// registers).  Returns the number of extrapolations that met the tolerance
// (-1 if none did; yout then holds the last one).
template <class Pol>
__device__ int bs_step(const BsDev &a, Pol &P, const double y[6], double h, double yout[6])
{
    double f0[6];
    P.deriv(a, y, f0);
    const double sx = __builtin_sqrt(y[0] * y[0] + y[1] * y[1] + y[2] * y[2]) +
                      h * __builtin_sqrt(f0[0] * f0[0] + f0[1] * f0[1] + f0[2] * f0[2]);
    const double sv = __builtin_sqrt(y[3] * y[3] + y[4] * y[4] + y[5] * y[5]) +
                      h * __builtin_sqrt(f0[3] * f0[3] + f0[4] * f0[4] + f0[5] * f0[5]);
    double T[KM][6];
    int kdone = -1;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        const int nk = 2 * (k + 1);
        const double hh = h / nk;
        double z0[6], z1[6], fz[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            z0[c] = y[c];
            z1[c] = y[c] + hh * f0[c];
        }
#pragma unroll 1
        for (int q = 1; q < nk; ++q) {
            P.deriv(a, z1, fz);
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                const double z2 = z0[c] + 2.0 * hh * fz[c];
                z0[c] = z1[c];
                z1[c] = z2;
            }
        }
        P.deriv(a, z1, fz);
        // row k of the tableau: T[0] = the midpoint result, T[j] from T[j - 1]
        // (this row) and the previous row's T[j - 1]
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            double old = T[0][c];
            T[0][c] = 0.5 * (z0[c] + z1[c] + hh * fz[c]);
#pragma unroll
            for (int j = 1; j <= k; ++j) {
                // 1 / (ratio^2 - 1), ratio = nk / (nk - 2 j): a constant (with
                // divisions a launch of small groups took 26.2 us, now 24.9)
                const double rden = (double)((nk - 2 * j) * (nk - 2 * j)) /
                                    (double)(nk * nk - (nk - 2 * j) * (nk - 2 * j));
                const double oj = T[j][c];
                T[j][c] = T[j - 1][c] + (T[j - 1][c] - old) * rden;
                old = oj;
            }
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) yout[c] = T[k][c];
        if (k > 0) {
            double err = 0.0;
            if (P.member()) {
                double ex = 0.0, ev = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double dxc = fabs(T[k][c] - T[k - 1][c]);
                    const double dvc = fabs(T[k][c + 3] - T[k - 1][c + 3]);
                    // (written so that a NaN propagates into the error)
                    ex = (dxc > ex || dxc != dxc) ? dxc : ex;
                    ev = (dvc > ev || dvc != dvc) ? dvc : ev;
                }
                const double e1 = ex / (sx + 1e-300), e2 = ev / (sv + 1e-300);
                err = e1 > e2 ? e1 : e2;
                // a step through a singularity (two members passing through
                // each other) yields NaN: count it as not converged, so that
                // every member takes the same decision
                if (!(err <= INFINITY)) err = INFINITY;
            }
            err = P.gmax(err);
            if (err <= a.eps) {
                kdone = k;
                break;
            }
        }
    }
    return kdone;
}

// The first overlapping pair of the group at state z (a < b, encoded as
// a * KEY_BASE + b), or NO_PAIR.  Uniform over the group.
constexpr long long KEY_BASE = 65536;
constexpr long long NO_PAIR = LLONG_MAX;

template <class Pol>
__device__ long long bs_overlap(const BsDev &a, Pol &P, const double z[6])
{
    P.publish(z);
    long long key = NO_PAIR;
    const int u = P.self();
    const double ru = P.rad(u);
    for (int q = 0; q < P.g; ++q) {
        double o[6];
        P.get(q, o);
        const double rq = P.rad(q);
        if (!P.member() || q <= u) continue;
        const double rs = ru + rq;
        const double dx = o[0] - z[0], dy = o[1] - z[1], dz = o[2] - z[2];
        if (rs > 0.0 && dx * dx + dy * dy + dz * dz < rs * rs && key == NO_PAIR)
            key = (long long)u * KEY_BASE + q;
    }
    return P.gmin(key);
}

// (positions and radii only, the share's own partners)
template <int BT, int NL, bool WHOLE>
__device__ long long BlockPol<BT, NL, WHOLE>::overlap(const BsDev &a, const double z[6])
{
    publish(z);
    long long key = NO_PAIR;
    if (t < g) {
        const double ru = sm.R[t];
        for (int q = t + 1 + sub; q < g; q += S) {
            const double rs = ru + sm.R[q];
            const double dx = sm.px[q] - z[0], dy = sm.py[q] - z[1], dz = sm.pz[q] - z[2];
            if (rs > 0.0 && dx * dx + dy * dy + dz * dz < rs * rs) {
                key = (long long)t * KEY_BASE + q;
                break;
            }
        }
    }
    return gmin(key);
}

template <int GS, int NL>
__device__ long long LanePol<GS, NL>::overlap(const BsDev &a, const double z[6])
{
    return bs_overlap(a, *this, z);
}

// Distance of members ma, mb at state z (uniform).
template <class Pol>
__device__ double bs_sep(Pol &P, const double z[6], int ma, int mb)
{
    P.publish(z);
    double oa[6], ob[6];
    P.get(ma, oa);
    P.get(mb, ob);
    const double dx = ob[0] - oa[0], dy = ob[1] - oa[1], dz = ob[2] - oa[2];
    return __builtin_sqrt(dx * dx + dy * dy + dz * dz);
}

// Perfect merger of members ma, mb at state z (in place): the survivor (the
// more massive, the lower body index for equal masses) takes the mass-weighted
// position and velocity, the summed mass and the radius (R_a^3 + R_b^3)^(1/3);
// the absorbed body becomes a massless, sizeless ghost at rest at
// (1e6 + index, 0, 0); one record (survivor, absorbed, lost energy
// 1/2 m_a m_b / (m_a + m_b) |v_a - v_b|^2 - G m_a m_b / r).
template <class Pol>
__device__ void bs_merge(const BsDev &a, Pol &P, double z[6], int ma, int mb)
{
    P.publish(z);
    double ya[6], yb[6];
    P.get(ma, ya);
    P.get(mb, yb);
    const double m1 = P.mass(ma), m2 = P.mass(mb), R1 = P.rad(ma), R2 = P.rad(mb);
    const int i1 = P.idx(ma), i2 = P.idx(mb);
    const bool first = m1 > m2 || (m1 == m2 && i1 < i2);
    const int ms = first ? ma : mb, mg = first ? mb : ma;
    const double M = m1 + m2;
    const int u = P.self();
    if (u == ms) {
#pragma unroll
        for (int c = 0; c < 6; ++c) z[c] = (m1 * ya[c] + m2 * yb[c]) / M;
        P.set_own(M, cbrt(R1 * R1 * R1 + R2 * R2 * R2));
        double dv2 = 0.0, dx2 = 0.0;
        for (int c = 0; c < 3; ++c) {
            dx2 += (ya[c] - yb[c]) * (ya[c] - yb[c]);
            dv2 += (ya[c + 3] - yb[c + 3]) * (ya[c + 3] - yb[c + 3]);
        }
        const double du = 0.5 * m1 * m2 / M * dv2 - a.G * m1 * m2 / __builtin_sqrt(dx2);
        if (P.owner()) {
            const unsigned long long slot = atomicAdd(a.coll_count, 1ull);
            if ((int64_t)slot < a.coll_cap) {
                a.coll_i[slot] = first ? i1 : i2;
                a.coll_j[slot] = first ? i2 : i1;
                a.coll_du[slot] = du;
            }
        }
    } else if (u == mg) {
        z[0] = 1e6 + (double)(first ? i2 : i1);
        z[1] = z[2] = z[3] = z[4] = z[5] = 0.0;
        P.set_own(0.0, 0.0);
    }
}

// One group's flow over H from y (in place); returns true if it failed.
// With radii, each accepted step is searched for an overlapping pair; the
// contact is bisected on the step length until the overlap is below
// coll_tol of R_a + R_b, the pair merges there, and the flow continues from
// that time.
template <class Pol>
__device__ bool bs_run(const BsDev &a, Pol &P, double y[6])
{
    double tt = 0.0, h = a.H;
    int tries = 0;
    while (tt < a.H) {      // uniform over the group: every member holds the same tt, h
        const bool last = h >= a.H - tt;
        if (last) h = a.H - tt;
        double yn[6];
        const int kdone = bs_step(a, P, y, h, yn);
        if (kdone >= 0) {
            const long long key = a.radius ? P.overlap(a, yn) : NO_PAIR;
            if (key != NO_PAIR) {
                const int ma = (int)(key / KEY_BASE), mb = (int)(key % KEY_BASE);
                const double rs = P.rad(ma) + P.rad(mb);
                double lo = 0.0, hi = h;
                double yh[6];
#pragma unroll
                for (int c = 0; c < 6; ++c) yh[c] = yn[c];
                for (int it = 0; it < 60; ++it) {
                    if ((rs - bs_sep(P, yh, ma, mb)) / rs < a.coll_tol) break;
                    const double mid = 0.5 * (lo + hi);
                    double ym[6];
                    bs_step(a, P, y, mid, ym);
                    if (bs_sep(P, ym, ma, mb) < rs) {
                        hi = mid;
#pragma unroll
                        for (int c = 0; c < 6; ++c) yh[c] = ym[c];
                    } else {
                        lo = mid;
                    }
                }
                bs_merge(a, P, yh, ma, mb);
#pragma unroll
                for (int c = 0; c < 6; ++c) y[c] = yh[c];
                tt = (last && hi == h) ? a.H : tt + hi;
            } else {
#pragma unroll
                for (int c = 0; c < 6; ++c) y[c] = yn[c];
                tt = last ? a.H : tt + h;
                if (kdone < KM / 2) h *= 2.0;
            }
        } else {
            h *= 0.5;
        }
        if (++tries > BS_TRIES || h < a.H * 1e-12) return true;
    }
    return false;
}

__device__ __forceinline__ void bs_store(const BsDev &a, int32_t b, const double y[6])
{
    a.x[b] = y[0];
    a.y[b] = y[1];
    a.z[b] = y[2];
    a.vx[b] = y[3];
    a.vy[b] = y[4];
    a.vz[b] = y[5];
}

// Groups of at most GS bodies, GS lanes each (the many small groups): wave `w`
// of block `blk` of `blocks`, the groups eight at a time, first over the blocks.
// Bound by the dependent operations of the slowest group's evaluations (65,536
// bodies, 3 x 4 levels, 5,300 groups: 55 -> 25 us per launch, by lanes that go
// around the group, one reciprocal per remainder and shorter estimates).
template <int GS, int NL>
__device__ __forceinline__ void bs_lanes(const BsDev &a, double (*irc)[GROUP_BLOCK], int blk, int blocks)
{
    const int lane = threadIdx.x & 63, u = lane % GS;
    const int64_t ng = a.gcount[0];
    const int64_t wave = (int64_t)(threadIdx.x >> 6) * blocks + blk;
    const int64_t stride = (int64_t)blocks * (GROUP_BLOCK / 64) * (64 / GS);
    for (int64_t gi = wave * (64 / GS) + lane / GS; gi < ng; gi += stride) {
        const int32_t root = a.groot[gi];
        const int g = a.gsize[root];
        LanePol<GS, NL> P;
        P.u = u;
        P.g = g;
        P.m = 0.0;
        P.R = 0.0;
        for (int c = 0; c < 6; ++c) P.zc[c] = 0.0;
        P.irc = &irc[0][threadIdx.x];
        // members in ascending order: each to the lane of its rank
        int32_t b = u < g ? a.gmem[a.gstart[root] + u] : INT_MAX;
        int rank = 0;
#pragma unroll
        for (int q = 0; q < GS; ++q) {
            const int32_t o = __shfl(b, q, GS);
            rank += o < b || (o == b && q < u);
        }
        b = __builtin_amdgcn_ds_permute((lane - u + rank) * 4, b);
        P.bidx = b;
        double y[6] = {0, 0, 0, 0, 0, 0};
        if (u < g) {
#pragma unroll
            for (int c = 0; c < 6; ++c) y[c] = a.state[c][b];
            P.m = a.m[b];
            P.R = a.radius ? a.radius[b] : 0.0;
            for (int l = 0; l < a.nlev; ++l) irc[l][threadIdx.x] = rcp_radius(a.rc[l][b]);
        }
        wave_sync_lds();   // the partners' lanes read these
        const bool failed = bs_run(a, P, y);
        if (failed && u == 0) atomicOr(a.status, ST_NOCONV);
        if (u < g) {
            bs_store(a, b, y);
            if (a.radius) {
                a.m[b] = P.m;
                a.radius[b] = P.R;
            }
        }
    }
}

// Whether the members want more than half of the group, from one partner per
// thread, spread over the group; uniform over the block.  (The forms cross where they
// want about half: rings of 300 bodies and 120 partners each 2,240 us by entries and
// 2,260 in place, of 150 and 80 1,005 and 780.)
template <int BT>
__device__ __forceinline__ bool bs_crowded(BsSmem<BT> &sm, int t, int g, int S, bool owner,
                                           double rcd, const double y[6])
{
    if (owner) {
        sm.px[t] = y[0];
        sm.py[t] = y[1];
        sm.pz[t] = y[2];
    }
    __syncthreads();
    const int q = (int)((((uint32_t)threadIdx.x * 40503u & 0xffffu) * (uint32_t)g) >> 16);
    const double dx = sm.px[q] - y[0], dy = sm.py[q] - y[1], dz = sm.pz[q] - y[2];
    const double re = rcd > sm.trho[q >> 6] ? rcd : sm.trho[q >> 6];
    return 2 * __syncthreads_count(t < g && dx * dx + dy * dy + dz * dz <= re * re) > g * S;
}

// Groups of more than BS_GS and at most GROUP_BLOCK bodies, one workgroup each
// (larger ones are the grid solver's).  A group of fewer members than threads
// spreads each member over S waves (S = GROUP_BLOCK / 64 over the member waves, a
// power of two): the waves of member wave I are I * S ... I * S + S - 1, each
// taking one share of the partners, and the first of them (the owner) alone
// writes.
//
// The crowded ones (bs_crowded) wait for a second pass, WHOLE: the two forms in one
// loop share their registers out worse (2-4 % of the 8,192-body disk).  What
// a group is is decided once, before it moves: the first pass puts the roots of
// the crowded ones into the block's first slots and returns their count, the
// second takes those `count` slots.
template <int NL, bool WHOLE>
__device__ __forceinline__ int bs_medium(const BsDev &a, BsSmem<GROUP_BLOCK> &sm, int blk, int blocks,
                                         int count)
{
    // (the wave index is uniform: the partner loops then run on scalar registers)
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int32_t *slot = a.groot + (a.n - 1 - blk);   // the block's k-th group: slot[-k * blocks]
    int left = 0;
    for (int k = 0; k < count; ++k) {
        const int32_t root = slot[-(int64_t)k * blocks];
        const int g = a.gsize[root];
        const int nw = (g + 63) >> 6;
        int S = 1;
        while (nw * S * 2 <= GROUP_BLOCK / 64) S *= 2;
        const int t = (w / S) * 64 + lane, sub = w % S;
        BlockPol<GROUP_BLOCK, NL, WHOLE> P{sm, t, g, S, sub, 0.0, {}};
        // the member of rank t
        const int32_t start = a.gstart[root];
        if (P.owner()) sm.idx[t] = a.gmem[start + t];
        __syncthreads();
        int32_t b = t < g ? sm.idx[t] : 0, rank = 0;
        for (int q = 0; q < g; ++q) rank += sm.idx[q] < b;
        __syncthreads();
        if (P.owner()) sm.idx[rank] = b;
        __syncthreads();
        b = t < g ? sm.idx[t] : 0;
        double y[6] = {0, 0, 0, 0, 0, 0};
        double rcd = 0.0;
        if (t < g) {
#pragma unroll
            for (int c = 0; c < 6; ++c) y[c] = a.state[c][b];
            rcd = a.rc[a.nlev - 1][b];
        }
        P.rcd = rcd;
        if (P.owner()) {
            sm.m[t] = a.m[b];
            sm.R[t] = a.radius ? a.radius[b] : 0.0;
            for (int l = 0; l < a.nlev; ++l)
                sm.irc[l][t] = rcp_radius(a.rc[l][b]);
        }
        {
            const double tr = wave_max_all(rcd);
            if (lane == 0 && P.owner()) sm.trho[t >> 6] = tr;
        }
        if (!WHOLE) {
            // the group's frame: its x-y extent and what its members travel
            const bool in = t < g;
            const double far = bs_block_max(sm, in ? __builtin_fmax(fabs(y[3]), fabs(y[4])) : 0.0) *
                               fabs(a.H);
            const double x0 = -bs_block_max(sm, in ? -y[0] : -INFINITY) - far;
            const double x1 = bs_block_max(sm, in ? y[0] : -INFINITY) + far;
            const double y0 = -bs_block_max(sm, in ? -y[1] : -INFINITY) - far;
            const double y1 = bs_block_max(sm, in ? y[1] : -INFINITY) + far;
            const double side = x1 - x0 > y1 - y0 ? x1 - x0 : y1 - y0;
            P.fr.x0 = x0;
            P.fr.y0 = y0;
            P.fr.scale = side > 0.0 && side < 1e300 ? 16000.0 / side : 0.0;
        }
        if (!WHOLE && bs_crowded(sm, t, g, S, P.owner(), rcd, y)) {
            // (every thread has read its root, and LDS is free behind the count)
            if (threadIdx.x == 0) {
                slot[-(int64_t)k * blocks] = slot[-(int64_t)left * blocks];
                slot[-(int64_t)left * blocks] = root;
            }
            ++left;
            continue;
        }
        bool failed;
        [[clang::always_inline]] failed = bs_run(a, P, y);
        if (failed && threadIdx.x == 0) atomicOr(a.status, ST_NOCONV);
        if (P.owner()) {
            bs_store(a, b, y);
            if (a.radius) {
                a.m[b] = sm.m[t];
                a.radius[b] = sm.R[t];
            }
        }
        __syncthreads();   // LDS reuse by the next group
    }
    __syncthreads();   // the roots put forward
    return left;
}

// Both classes in one launch, so that the small groups run beside the medium
// ones and an empty class costs no launch: blocks [0, BS_MEDIUM) the medium groups (a
// compute unit holds one of them), the blocks behind them the small ones.
constexpr int BS_MEDIUM = 256, BS_SMALL = 256;

union BsLds {
    BsSmem<GROUP_BLOCK> medium;
    double irc[GENGA_MAX_LEVELS][GROUP_BLOCK];
    __device__ BsLds() {}
};

template <int NL>
__global__ __launch_bounds__(GROUP_BLOCK) void k_bs(BsDev a)
{
    __shared__ BsLds sm;
    if (blockIdx.x < BS_MEDIUM) {
        const int blk = (int)blockIdx.x, ng = a.gcount[2];
        const int count = ng > blk ? (ng - blk + BS_MEDIUM - 1) / BS_MEDIUM : 0;
        const int left = bs_medium<NL, false>(a, sm.medium, blk, BS_MEDIUM, count);
        if (left) bs_medium<NL, true>(a, sm.medium, blk, BS_MEDIUM, left);
    } else
        bs_lanes<BS_GS, NL>(a, sm.irc, (int)blockIdx.x - BS_MEDIUM, BS_SMALL);
}

// ---------------------------------------------------------------------------
// Groups of more than GROUP_BLOCK bodies (Sect. 6.1: the method that spreads
// one group over many thread blocks).  The paper drives each sub-step of
// that method from the host; here one persistent launch integrates the
// listed groups one after another, its workgroups meeting at a grid-wide
// barrier before every evaluation that reads other members' positions and
// at every group-wide maximum or minimum.  One thread per member (so a
// group may hold up to GENGA_GROUP_MAX bodies with the launch's workgroups
// all resident); the members are first ordered by a 64 x 64 cell grid over
// the group's x-y extent (cells along Hilbert's curve, members of a cell by their
// rank in the group), so that each wave's 64 members form a compact tile.
// A derivative then visits, per tile, only the tiles whose bounding boxes
// come within the larger deepest-level critical radius of the two tiles:
// every pair of the tiles left out has R = 0 exactly (the deepest level's
// factor 1 - K is zero at r >= rho), so its terms are exact zeros and the
// sums equal the all-pairs ones; a member's sum runs over its partners in
// ascending tile and slot order.
// ---------------------------------------------------------------------------
constexpr int GT = 256;             // threads per workgroup of the grid solver

// The grid solver's search runs in binary32, one 16-byte LDS read per partner: a position
// rounded to binary32 and the square of the radius widened by twice what two
// such neighbours can be off (2^-24 of each coordinate, 2^-23 of their
// difference), so that it misses no pair inside the radius.
__device__ __forceinline__ float4 bs_near(double x, double y, double z, double rcd)
{
    const double e = rcd + 0x1p-20 * (fabs(x) + fabs(y) + fabs(z) + rcd);
    return make_float4((float)x, (float)y, (float)z, (float)(e * e) * (1.0f + 0x1p-20f));
}

__device__ __forceinline__ bool bs_in_reach(const float4 &a, const float4 &b)
{
    const float dx = b.x - a.x, dy = b.y - a.y, dz = b.z - a.z;
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
    return !(r2 > (a.w > b.w ? a.w : b.w));   // (a NaN is evaluated)
}

constexpr int GCELL = 64;           // ordering cells per axis
// a barrier that has waited this long (wall clock, 100 MHz ticks: 2 s) gives up
constexpr uint64_t GWAIT_TICKS = 200000000ull;

struct GridDev {
    int32_t cap;                        // members per group the launch can hold
    const int32_t *big;                 // [0] listed groups, [1 ..] their roots
    double *pub;                        // [2][6][cap] published states (by parity)
    double *box;                        // [2][cap / 64][8] tile box lo, hi, max radius
    double *trho;                       // [cap / 64] largest deepest-level rc per tile
    double *mm, *mR;                    // [cap] member mass, radius
    double *mirc;                       // [GENGA_MAX_LEVELS][cap] 1 / rc per level
    double *mrc;                        // [cap] deepest-level rc
    int32_t *midx;                      // [cap] member body
    double *bpart;                      // [cap / 64][4] workgroup x-y extents
    int32_t *ccnt, *cfill;              // [GCELL^2] members per cell, fill counters
    int32_t *ctmp;                      // [cap] members by cell in arrival order
    unsigned long long *sync;           // [0] arrivals, [1] abort, [2..4] max slots
    long long *rmin;                    // [3] min slots
};

struct GridSmem {
    double sx[4][64], sy[4][64], sz[4][64], sm[4][64];
    float4 snear[4][64];                 // bs_near of the partners
    double sirc[4][GENGA_MAX_LEVELS][64];
    double oirc[GENGA_MAX_LEVELS][GT];   // own 1 / rc per level
    double part[4][3][64];               // partial sums of the split waves
    double red[4][4];
    int32_t cstart[GCELL * GCELL];
    double ext[4];
    int64_t scan[GT / 64];
    int dead;
};

// The grid solver's LDS (only k_bs_grid reaches it).  Declared at namespace
// scope so that the out-of-line evaluation addresses it as LDS.
static __shared__ GridSmem g_gsm;

// Position of cell (x, y) of the GCELL x GCELL grid along Hilbert's curve
// (the usual construction: at each scale s the quadrant's number goes into
// the index, then the coordinates are turned into that quadrant's frame),
// so that consecutive cells along the order are always neighbours.
__device__ __forceinline__ unsigned hilbert_cell(unsigned x, unsigned y)
{
    unsigned d = 0;
    for (unsigned s = GCELL / 2; s > 0; s >>= 1) {
        const unsigned rx = (x & s) ? 1u : 0u, ry = (y & s) ? 1u : 0u;
        d += s * s * ((3u * rx) ^ ry);
        if (ry == 0) {
            if (rx == 1) {
                x = GCELL - 1 - x;
                y = GCELL - 1 - y;
            }
            const unsigned tmp = x;
            x = y;
            y = tmp;
        }
    }
    return d;
}

struct GridPol {
    const GridDev &G;
    int t, g, nlev, nblk;
    int split, sub;             // waves per tile, this wave's share (0: the owner)
    unsigned long long nbar;    // barriers passed in this launch
    int par;                    // parity of the last publication
    int nred;                   // reductions done in this launch
    bool dead;
    double m, R;                // own mass and radius
    double rcd;                 // own deepest-level rc

    __device__ bool member() const { return t < g; }
    // the first wave of a tile writes; the others hold copies of its members
    __device__ bool owner() const { return t < g && sub == 0; }
    __device__ int self() const { return t; }

    // Grid-wide barrier of the nblk workgroups: every arrival is counted
    // once after a release fence; the wait polls with relaxed loads (an
    // acquire per poll would invalidate the L2 of the poller's XCD each
    // time) and ends with one acquire fence.  The wait is bounded in wall
    // clock time: a barrier that times out (or finds that another workgroup
    // gave up) marks the launch dead, after which no barrier waits and the
    // flow fails to converge.
    __device__ bool sync()
    {
        __syncthreads();
        ++nbar;
        if (threadIdx.x == 0) {
            int d = dead ? 1 : 0;
            if (!d) {
                unsigned long long *cnt = G.sync;
                const unsigned long long target = nbar * (unsigned long long)nblk;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                __hip_atomic_fetch_add(cnt, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint64_t t0 = wall_clock64();
                while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
                    if (__hip_atomic_load(cnt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        d = 1;
                        break;
                    }
                    if (wall_clock64() - t0 > GWAIT_TICKS) {
                        __hip_atomic_store(cnt + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        d = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(4);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            g_gsm.dead = d;
        }
        __syncthreads();
        dead = g_gsm.dead != 0;
        return !dead;
    }

    // the own tile's box (lo, hi) of positions z (members only)
    __device__ void tile_box(const double z[3], double lo[3], double hi[3]) const
    {
        const bool mem = member();
#pragma unroll
        for (int c = 0; c < 3; ++c) wave_bounds(z[c], mem, lo[c], hi[c]);
    }

    __device__ void publish_n(const double z[6], int nc, double lo[3], double hi[3])
    {
        par ^= 1;
        double *P = G.pub + (size_t)par * 6 * G.cap;
        if (owner())
            for (int c = 0; c < nc; ++c) P[(size_t)c * G.cap + t] = z[c];
        tile_box(z, lo, hi);
        const double rmax = wave_max_all(member() ? R : 0.0);
        if ((threadIdx.x & 63) == 0 && owner()) {
            double *B = G.box + ((size_t)par * (G.cap / 64) + (t >> 6)) * 8;
            B[0] = lo[0]; B[1] = lo[1]; B[2] = lo[2];
            B[3] = hi[0]; B[4] = hi[1]; B[5] = hi[2];
            B[6] = rmax;
        }
        sync();
    }

    __device__ void publish(const double z[6])
    {
        double lo[3], hi[3];
        publish_n(z, 6, lo, hi);
    }

    __device__ void get(int q, double o[6]) const
    {
        const double *P = G.pub + (size_t)par * 6 * G.cap;
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = P[(size_t)c * G.cap + q];
    }
    __device__ double mass(int q) const { return G.mm[q]; }
    __device__ double rad(int q) const { return G.mR[q]; }
    __device__ int idx(int q) const { return G.midx[q]; }
    __device__ void set_own(double mm, double RR)
    {
        if (member()) {
            m = mm;
            R = RR;
            if (owner()) {
                G.mm[t] = mm;
                G.mR[t] = RR;
            }
        }
    }


    // (one copy of the evaluation: bs_step reaches it from nine places; the
    // loop works on locals and LDS only).  A partner tile is visited if its
    // box comes within the larger deepest-level radius of the own tile's box
    // and of some member's own position (both tests skip only exact zeros).
    // The split waves of a tile take every split-th tile of its list each;
    // their partial sums are added in share order.
    __device__ __noinline__ void deriv(const BsDev &a, const double z[6], double f[6])
    {
        f[0] = z[3];
        f[1] = z[4];
        f[2] = z[5];
        double lo[3], hi[3];
        publish_n(z, 3, lo, hi);
        const double x0 = z[0], y0 = z[1], z0 = z[2];
        double ax = 0.0, ay = 0.0, az = 0.0;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const int me = t, ng = g, nl = nlev, S_ = split, mine = sub;
        const int t0 = me - lane;
        GridSmem &S = g_gsm;
        if (!dead && t0 < ng) {
            const double Gc = a.G, rcme = rcd;
            const float4 nme = bs_near(x0, y0, z0, rcme);
            const size_t cap = (size_t)G.cap;
            const int nt = (ng + 63) >> 6;
            const double *trho = G.trho, *mm = G.mm, *mrc = G.mrc, *mirc = G.mirc;
            const double rhoI = trho[t0 >> 6];
            const double *P = G.pub + (size_t)par * 6 * cap;
            const double *Bx = G.box + (size_t)par * (cap / 64) * 8;
            const double pos[3] = {x0, y0, z0};
            const bool mem = me < ng;
            int seen = 0;   // tiles of the list met so far (wave-uniform)
            for (int jb = 0; jb < nt; jb += 64) {
                const int Jl = jb + lane;
                bool near = false;
                double bj[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, rj = 0.0;
                if (Jl < nt) {
                    const double *B = Bx + (size_t)Jl * 8;
#pragma unroll
                    for (int c = 0; c < 6; ++c) bj[c] = B[c];
                    rj = trho[Jl];
                    const double rr = rhoI > rj ? rhoI : rj;
                    // (members at NaN are not in their tile's box: they fail the
                    // flow by their own error)
                    near = !(box_gap2(lo, hi, bj) > rr * rr * (1.0 + 0x1p-18));
                }
                unsigned long long mask = __ballot(near);
                while (mask) {
                    const int src = __builtin_ctzll(mask);
                    const int J = jb + src;
                    mask &= mask - 1;
                    // the same test for each member's own position: a tile whose
                    // box is large (members from distant cells) passes the box
                    // test against many tiles, of which few come near a member
                    double bJ[6];
#pragma unroll
                    for (int c = 0; c < 6; ++c) bJ[c] = __shfl(bj[c], src, 64);
                    const double rJ = __shfl(rj, src, 64);
                    const double rm = rcme > rJ ? rcme : rJ;
                    const bool close = mem && !(box_gap2(pos, pos, bJ) > rm * rm * (1.0 + 0x1p-18));
                    if (__ballot(close) == 0ull) continue;
                    if (seen++ % S_ != mine) continue;
                    const int jq = J * 64 + lane;
                    if (jq < ng) {
                        const double xq = P[jq], yq = P[cap + jq], zq = P[2 * cap + jq];
                        S.sx[w][lane] = xq;
                        S.sy[w][lane] = yq;
                        S.sz[w][lane] = zq;
                        S.snear[w][lane] = bs_near(xq, yq, zq, mrc[jq]);
                        S.sm[w][lane] = mm[jq];
                        for (int l = 0; l < nl; ++l) S.sirc[w][l][lane] = mirc[(size_t)l * cap + jq];
                    }
                    wave_sync_lds();
                    const int qn = ng - J * 64 < 64 ? ng - J * 64 : 64;
                    uint64_t reach = 0;
#pragma unroll 4
                    for (int q = 0; q < qn; ++q)
                        if (bs_in_reach(nme, S.snear[w][q])) reach |= 1ull << q;
                    if (J == me >> 6) reach &= ~(1ull << lane);
                    if (!mem) reach = 0;
                    while (reach) {
                        const int q = __builtin_ctzll(reach);
                        reach &= reach - 1;
                        const double dx = S.sx[w][q] - x0, dy = S.sy[w][q] - y0,
                                     dz = S.sz[w][q] - z0;
                        const double r2 = dx * dx + dy * dy + dz * dz;
                        const double ir = rsq_full(r2);
                        const double Rw = bs_remainder<0>(r2 * ir, &S.oirc[0][threadIdx.x], GT,
                                                          &S.sirc[w][0][q], 64, nl);
                        const double s = Gc * S.sm[w][q] * Rw * (ir * ir * ir);
                        ax += s * dx;
                        ay += s * dy;
                        az += s * dz;
                    }
                    wave_sync_lds();
                }
            }
        }
        // the star's pull, then the shares' partial sums in share order
        double kx = 0.0, ky = 0.0, kz = 0.0;
        if (member()) {
            const double r2s = x0 * x0 + y0 * y0 + z0 * z0;
            const double irs = rsq_full(r2s);
            const double ks = -a.mu * (irs * irs * irs);
            kx = ks * x0;
            ky = ks * y0;
            kz = ks * z0;
        }
        if (S_ > 1) {
            S.part[w][0][lane] = ax;
            S.part[w][1][lane] = ay;
            S.part[w][2][lane] = az;
            __syncthreads();
            const int w0 = w - mine;
            for (int k = 0; k < S_; ++k) {
                kx += S.part[w0 + k][0][lane];
                ky += S.part[w0 + k][1][lane];
                kz += S.part[w0 + k][2][lane];
            }
            __syncthreads();
        } else {
            kx += ax;
            ky += ay;
            kz += az;
        }
        f[3] = kx;
        f[4] = ky;
        f[5] = kz;
    }

    // group-wide reductions through rotating slots: slot nred % 3 collects
    // this reduction; after its barrier workgroup 0 resets slot
    // (nred + 2) % 3, whose last readers have all passed this barrier and
    // whose next writers come after the next one (the split waves hold the
    // same values: a maximum or minimum counts them once)
    __device__ void reset_slot()
    {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            const int s2 = (nred + 2) % 3;
            __hip_atomic_store(G.sync + 2 + s2, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(G.rmin + s2, NO_PAIR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ++nred;
    }

    __device__ double gmax(double v)
    {
        // non-negative (or +inf) values: their bit patterns order as integers
        v = wave_max_all(v);
        const int s = nred % 3;
        if ((threadIdx.x & 63) == 0 && !dead)
            __hip_atomic_fetch_max(G.sync + 2 + s, (unsigned long long)__double_as_longlong(v),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sync();
        double r = INFINITY;
        if (!dead)
            r = __longlong_as_double((long long)__hip_atomic_load(G.sync + 2 + s, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT));
        reset_slot();
        return r;
    }

    __device__ long long gmin(long long v)
    {
        for (int d = 32; d > 0; d >>= 1) {
            const long long o = __shfl_xor(v, d, 64);
            v = o < v ? o : v;
        }
        const int s = nred % 3;
        if ((threadIdx.x & 63) == 0 && !dead && v != NO_PAIR)
            __hip_atomic_fetch_min(G.rmin + s, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sync();
        long long r = NO_PAIR;
        if (!dead) r = __hip_atomic_load(G.rmin + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        reset_slot();
        return r;
    }

    __device__ long long overlap(const BsDev &a, const double z[6]);
};

// The grid solver's overlap search: tiles whose boxes stay apart by more
// than the sum of their largest radii hold no overlapping pair.
__device__ long long GridPol::overlap(const BsDev &a, const double z[6])
{
    double lo[3], hi[3];
    publish_n(z, 6, lo, hi);
    long long key = NO_PAIR;
    const int lane = threadIdx.x & 63;
    const int t0 = t - lane;
    if (!dead && t0 < g) {
        const int nt = (g + 63) >> 6;
        const double *Pp = G.pub + (size_t)par * 6 * G.cap;
        const double *Bx = G.box + (size_t)par * (G.cap / 64) * 8;
        const double rI = wave_max_all(member() ? R : 0.0);
        for (int jb = 0; jb < nt; jb += 64) {
            const int Jl = jb + lane;
            bool near = false;
            if (Jl < nt) {
                const double rs = rI + Bx[(size_t)Jl * 8 + 6];
                near = rs > 0.0 && !(box_gap2(lo, hi, Bx + (size_t)Jl * 8) > rs * rs * (1.0 + 0x1p-18));
            }
            unsigned long long mask = __ballot(near);
            while (mask) {
                const int J = jb + __builtin_ctzll(mask);
                mask &= mask - 1;
                const int qn = g - J * 64 < 64 ? g - J * 64 : 64;
                for (int qq = 0; qq < qn; ++qq) {
                    const int q = J * 64 + qq;
                    if (!member() || q <= t || key != NO_PAIR) continue;
                    const double rs = R + G.mR[q];
                    const double dx = Pp[q] - z[0], dy = Pp[(size_t)G.cap + q] - z[1],
                                 dz = Pp[2 * (size_t)G.cap + q] - z[2];
                    if (rs > 0.0 && dx * dx + dy * dy + dz * dz < rs * rs)
                        key = (long long)t * KEY_BASE + q;
                }
            }
        }
    }
    return gmin(key);
}

// Spatial order of the group's members (see above): by cell, then by body
// index, whatever the order of the group's slots; perm[k] = body of the k-th
// member in that order.  Four grid barriers; only the owners contribute.
__device__ void grid_order(const BsDev &a, GridPol &P, int32_t root, int32_t *perm)
{
    const GridDev &G = P.G;
    GridSmem &S = g_gsm;
    const int t = P.t;
    const bool own = P.owner();
    const int nthr = P.nblk * GT;
    const int tid = blockIdx.x * GT + threadIdx.x;
    const int32_t b = own ? a.gmem[a.gstart[root] + t] : 0;
    double x = 0.0, y = 0.0;
    if (own) {
        x = a.state[0][b];
        y = a.state[1][b];
    }
    for (int c = tid; c < GCELL * GCELL; c += nthr) {
        G.ccnt[c] = 0;
        G.cfill[c] = 0;
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    {
        const double v[4] = {wave_min_all(own ? x : INFINITY), wave_max_all(own ? x : -INFINITY),
                             wave_min_all(own ? y : INFINITY), wave_max_all(own ? y : -INFINITY)};
        if (lane == 0)
            for (int c = 0; c < 4; ++c) S.red[w][c] = v[c];
        __syncthreads();
        if (threadIdx.x < 4) {
            const int c = threadIdx.x;
            double r = S.red[0][c];
            for (int k = 1; k < 4; ++k) r = (c & 1) ? (S.red[k][c] > r ? S.red[k][c] : r)
                                                    : (S.red[k][c] < r ? S.red[k][c] : r);
            G.bpart[(size_t)blockIdx.x * 4 + c] = r;
        }
    }
    P.sync();
    // the group's extent (the same arithmetic in every workgroup)
    double *ext = S.ext;
    if (threadIdx.x < 4) {
        const int c = threadIdx.x;
        double r = G.bpart[c];
        for (int k = 1; k < P.nblk; ++k) {
            const double o = G.bpart[(size_t)k * 4 + c];
            r = (c & 1) ? (o > r ? o : r) : (o < r ? o : r);
        }
        ext[c] = r;
    }
    __syncthreads();
    unsigned cell = 0;
    if (own) {
        const double wx = ext[1] - ext[0], wy = ext[3] - ext[2];
        const double fx = wx > 0.0 ? (x - ext[0]) * (GCELL / wx) : 0.0;
        const double fy = wy > 0.0 ? (y - ext[2]) * (GCELL / wy) : 0.0;
        int cx = fx >= 0.0 ? (int)fx : 0, cy = fy >= 0.0 ? (int)fy : 0;
        cx = cx < GCELL - 1 ? cx : GCELL - 1;
        cy = cy < GCELL - 1 ? cy : GCELL - 1;
        // (NaN positions land in cell 0: the flow fails later anyway)
        cell = hilbert_cell((unsigned)cx, (unsigned)cy);
        atomicAdd(G.ccnt + cell, 1);
    }
    P.sync();
    // exclusive scan of the cell counts, in every workgroup
    {
        constexpr int PER = GCELL * GCELL / GT;
        int loc[PER], sum = 0;
        for (int k = 0; k < PER; ++k) {
            loc[k] = __hip_atomic_load(G.ccnt + threadIdx.x * PER + k, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            sum += loc[k];
        }
        int64_t tot;
        int64_t off = block_excl_scan<GT>((int64_t)sum, &tot, S.scan);
        for (int k = 0; k < PER; ++k) {
            S.cstart[threadIdx.x * PER + k] = (int32_t)off;
            off += loc[k];
        }
    }
    __syncthreads();
    if (own) G.ctmp[S.cstart[cell] + atomicAdd(G.cfill + cell, 1)] = b;
    P.sync();
    // within a cell by body index (the slots' arrival order is not fixed)
    if (own) {
        const int c0 = S.cstart[cell];
        const int cn = __hip_atomic_load(G.ccnt + cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int rank = 0;
        for (int k = c0; k < c0 + cn; ++k) rank += G.ctmp[k] < b;
        perm[c0 + rank] = b;
    }
    P.sync();
}

// Waves per tile for a group of g members when nb workgroups (of 4 waves)
// can take part: the most of 4, 2, 1 that fit in them (0: the group does not
// fit).
__device__ inline int grid_split(int g, int nb)
{
    const int nt = (g + 63) / 64;
    for (int s = 4; s >= 1; s >>= 1)
        if ((nt * s + 3) / 4 <= nb) return s;
    return 0;
}

// All listed groups of more than GROUP_BLOCK bodies, one after another.
// Launched with as many workgroups as are resident together (sized for two
// per compute unit); a group takes the most waves per tile that fit, and the
// workgroups beyond the largest group's need return at once.
__global__ __launch_bounds__(GT, 2) void k_bs_grid(BsDev a, GridDev G)
{
    GridSmem &S = g_gsm;
    const int nbig = G.big[0];
    int need = 0;
    for (int k = 0; k < nbig; ++k) {
        const int g = a.gsize[G.big[1 + k]];
        const int s = g <= G.cap ? grid_split(g, gridDim.x) : 0;
        if (s) {
            const int nb = ((g + 63) / 64 * s + 3) / 4;
            need = nb > need ? nb : need;
        } else if (blockIdx.x == 0 && threadIdx.x == 0) {
            atomicOr(a.status, ST_GROUP);
        }
    }
    if ((int)blockIdx.x >= need) return;
    GridPol P{G};
    P.nlev = a.nlev;
    P.nblk = need;
    P.nbar = 0;
    P.par = 0;
    P.nred = 0;
    P.dead = false;
    int32_t *perm = G.ctmp + G.cap;   // second half of the cell scratch
    const int gw = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int k = 0; k < nbig; ++k) {
        const int32_t root = G.big[1 + k];
        const int g = a.gsize[root];
        const int split = g <= G.cap ? grid_split(g, gridDim.x) : 0;
        if (!split) continue;
        P.g = g;
        P.split = split;
        P.sub = gw % split;
        P.t = gw / split * 64 + lane;
        grid_order(a, P, root, perm);
        const int t = P.t;
        const bool mem = t < g;
        const int32_t b = mem ? perm[t] : 0;
        double y[6] = {0, 0, 0, 0, 0, 0};
        P.m = 0.0;
        P.R = 0.0;
        P.rcd = 0.0;
        if (mem) {
#pragma unroll
            for (int c = 0; c < 6; ++c) y[c] = a.state[c][b];
            P.m = a.m[b];
            P.R = a.radius ? a.radius[b] : 0.0;
            P.rcd = a.rc[a.nlev - 1][b];
            for (int l = 0; l < a.nlev; ++l) {
                const double ir = rcp_radius(a.rc[l][b]);
                S.oirc[l][threadIdx.x] = ir;
                if (P.owner()) G.mirc[(size_t)l * G.cap + t] = ir;
            }
            if (P.owner()) {
                G.mm[t] = P.m;
                G.mR[t] = P.R;
                G.mrc[t] = P.rcd;
                G.midx[t] = b;
            }
        }
        const double tr = wave_max_all(mem ? P.rcd : 0.0);
        if (lane == 0 && P.owner()) G.trho[t >> 6] = tr;
        // (the first evaluation's barrier publishes these)
        const bool failed = bs_run(a, P, y);
        if (failed && t == 0) atomicOr(a.status, ST_NOCONV);
        if (P.owner()) {
            bs_store(a, b, y);
            if (a.radius) {
                a.m[b] = P.m;
                a.radius[b] = P.R;
            }
        }
        P.sync();   // scratch reuse by the next group
    }
}

// ---------------------------------------------------------------------------
// Host sequencing
// ---------------------------------------------------------------------------
struct LevelRun {
    genga_bodies *b;
    const genga_params *p;
    const LevelLayout *V;
    char *ws;
    hipStream_t s;

    template <typename T>
    T *at(size_t off) const { return (T *)(ws + off); }
    int32_t *status() const { return (int32_t *)ws; }
    unsigned list_blocks() const
    {
        return (unsigned)std::min<int64_t>(LG, (b->n + LT - 1) / LT);
    }
    ListDev all() const { return {nullptr, nullptr, b->n}; }
    BodyDev bodies_of(int l) const
    {
        BodyDev a;
        a.bodies = at<int32_t>(V->bodies[l]);
        a.nbod = at<int32_t>(V->nbod) + l;
        a.x = b->x; a.y = b->y; a.z = b->z;
        a.vx = b->vx; a.vy = b->vy; a.vz = b->vz;
        a.m = b->m;
        a.status = status();
        return a;
    }
};

static AdjDev adj_of(const LevelRun &R, int l)
{
    const LevelLayout &V = *R.V;
    AdjDev A{};
    if (l >= V.L - 1) return A;
    A.deg = R.at<int32_t>(V.deg[l]);
    A.start = R.at<int32_t>(V.start[l]);
    A.bodies = R.at<int32_t>(V.bodies[l]);
    A.nbod = R.at<int32_t>(V.nbod) + l;
    A.n = R.b->n;
    return A;
}

// Adjacency of list l, whose degrees are counted; its bodies are among `up`.
static hipError_t build_adj(const LevelRun &R, int l, const ListDev &up)
{
    const LevelLayout &V = *R.V;
    const AdjDev A = adj_of(R, l);
    const int32_t *pi = R.at<int32_t>(V.pi[l]), *pj = R.at<int32_t>(V.pj[l]);
    const int64_t *cnt = R.at<int64_t>(V.cnt) + l;
    int32_t *tmp = R.at<int32_t>(V.adj_tmp[l]), *owner = R.at<int32_t>(V.owner[l]);
    hipLaunchKernelGGL(k_adj_alloc, dim3(R.list_blocks()), dim3(LT), 0, R.s, up, A);
    hipLaunchKernelGGL(k_adj_fill, dim3(LG), dim3(LT), 0, R.s, pi, pj, cnt, V.cap, A, tmp, owner);
    hipLaunchKernelGGL(k_adj_rank, dim3(LG), dim3(LT), 0, R.s, A, tmp, owner,
                       R.at<int32_t>(V.adj[l]));
    return hipGetLastError();
}

template <int LEVEL>
static void launch_level_kick(const LevelKickDev &k, int l, const DetectDev *d, hipStream_t s)
{
    if constexpr (LEVEL < GENGA_MAX_LEVELS - 1) {
        if (l != LEVEL) return launch_level_kick<LEVEL + 1>(k, l, d, s);
    }
    if (d)
        hipLaunchKernelGGL((k_level_kick<LEVEL, true>), dim3(KB_DETECT + LG), dim3(LT), 0, s, k, *d);
    else
        hipLaunchKernelGGL((k_level_kick<LEVEL, false>), dim3(LG), dim3(LT), 0, s, k, DetectDev{});
}

// The kick of level l, 1 <= l < GENGA_MAX_LEVELS (d: and the count of its next list).
static hipError_t level_kick(const LevelRun &R, int l, double h, const DetectDev *d)
{
    const LevelLayout &V = *R.V;
    LevelKickDev k;
    k.a = R.bodies_of(l - 1);
    k.start = R.at<int32_t>(V.start[l - 1]);
    k.deg = R.at<int32_t>(V.deg[l - 1]);
    k.adj = R.at<int32_t>(V.adj[l - 1]);
    for (int q = 0; q < GENGA_MAX_LEVELS; ++q) k.rc[q] = nullptr;
    k.rc[0] = R.b->rc;
    for (int q = 1; q <= l; ++q) k.rc[q] = R.at<double>(V.rc[q]);
    k.G = R.p->G;
    k.h = h;
    launch_level_kick<1>(k, l, d, R.s);
    return hipGetLastError();
}

// Workgroups of k_bs_grid that the current device holds at once (queried
// once per device).
static hipError_t grid_resident_blocks(int *out)
{
    static std::mutex mu;
    static int cached[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!cached[dev]) {
        int per_cu = 0, cus = 0;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_bs_grid, GT, 0)) !=
            hipSuccess)
            return e;
        if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
            hipSuccess)
            return e;
        if (per_cu < 1 || cus < 1) return hipErrorLaunchFailure;
        cached[dev] = per_cu * cus;
    }
    *out = cached[dev];
    return hipSuccess;
}

// Workgroups of the grid solver's launch (as many as fit the capacity and are
// resident on the device together: the barriers need them all) and the members
// of the largest group it takes.
static hipError_t grid_size(const LevelLayout &V, int *nb, int32_t *cap)
{
    int resident = 0;
    const hipError_t e = grid_resident_blocks(&resident);
    if (e != hipSuccess) return e;
    *nb = (int)std::min<int64_t>(V.gcap / 64, resident);
    *cap = (int32_t)std::min<int64_t>(V.gcap, (int64_t)*nb * GT);
    return hipSuccess;
}

static hipError_t groups_of(const LevelRun &R, GroupDev *out)
{
    const LevelLayout &V = *R.V;
    GroupDev g{};
    if (V.direct) {
        g.parent = R.at<int32_t>(V.gtmp);
        g.flag = R.at<int32_t>(V.gflag);
        g.lab = R.at<int32_t>(V.glab);
        g.size = R.at<int32_t>(V.gsize);
        g.slot = R.at<int32_t>(V.gslot);
        g.start = R.at<int32_t>(V.gstart);
        g.mem = R.at<int32_t>(V.gmem);
        g.root = R.at<int32_t>(V.groot);
        g.count = R.at<int32_t>(V.gcount);
        g.big = V.gbig ? R.at<int32_t>(V.gbig) : nullptr;
        g.gsync = V.gbig ? R.at<unsigned long long>(V.gsync) : nullptr;
        g.gstats = R.at<unsigned long long>(V.gstats);
        g.limit = GROUP_BLOCK;
        g.n = R.b->n;
        if (V.gbig) {
            int nb = 0;
            const hipError_t e = grid_size(V, &nb, &g.limit);
            if (e != hipSuccess) return e;
        }
    }
    *out = g;
    return hipSuccess;
}

// Roots, sizes and slots of the groups whose pairs are joined; their members
// are among `up`.
static void build_groups(const LevelRun &R, const ListDev &up, const GroupDev &g)
{
    const dim3 nb(R.list_blocks());
    hipLaunchKernelGGL(k_group_root, nb, dim3(LT), 0, R.s, up, g);
    hipLaunchKernelGGL(k_group_alloc, nb, dim3(LT), 0, R.s, up, g);
}

// The groups of list l over dt_l from `state`, weights of levels 0..l.
static hipError_t direct_solve(const LevelRun &R, int l, double dt_l, const double *const *state)
{
    const LevelLayout &V = *R.V;
    BsDev a;
    a.groot = R.at<int32_t>(V.groot);
    a.gstart = R.at<int32_t>(V.gstart);
    a.gsize = R.at<int32_t>(V.gsize);
    a.gmem = R.at<int32_t>(V.gmem);
    a.gcount = R.at<int32_t>(V.gcount);
    for (int c = 0; c < 6; ++c) a.state[c] = state[c];
    a.n = R.b->n;
    a.x = R.b->x; a.y = R.b->y; a.z = R.b->z;
    a.vx = R.b->vx; a.vy = R.b->vy; a.vz = R.b->vz;
    a.m = R.b->m;
    for (int q = 0; q < GENGA_MAX_LEVELS; ++q) a.rc[q] = nullptr;
    a.rc[0] = R.b->rc;
    for (int q = 1; q <= l; ++q) a.rc[q] = R.at<double>(V.rc[q]);
    a.nlev = l + 1;
    a.G = R.p->G;
    a.mu = R.p->G * R.p->m_star;
    a.H = dt_l;
    a.eps = R.p->bs_eps > 0.0 ? R.p->bs_eps : 1e-12;
    a.status = R.status();
    a.radius = R.b->R;
    a.coll_tol = R.p->coll_tol > 0.0 ? R.p->coll_tol : 1e-6;
    a.coll_i = R.at<int32_t>(V.coll_i);
    a.coll_j = R.at<int32_t>(V.coll_j);
    a.coll_du = R.at<double>(V.coll_du);
    a.coll_count = R.at<unsigned long long>(V.coll_count);
    a.coll_cap = LEVEL_COLL_CAP;
    auto *bs = a.nlev == 1 ? k_bs<1> : a.nlev == 2 ? k_bs<2> : a.nlev == 3 ? k_bs<3> : k_bs<0>;
    hipLaunchKernelGGL(bs, dim3(BS_MEDIUM + BS_SMALL), dim3(GROUP_BLOCK), 0, R.s, a);
    if (!V.gbig) return hipGetLastError();
    // groups beyond one workgroup
    int nb = 0;
    GridDev G;
    const hipError_t e = grid_size(V, &nb, &G.cap);
    if (e != hipSuccess) return e;
    G.big = R.at<int32_t>(V.gbig);
    G.pub = R.at<double>(V.gpub);
    G.box = R.at<double>(V.gbox);
    G.trho = R.at<double>(V.gtrho);
    G.mm = R.at<double>(V.gmm);
    G.mR = R.at<double>(V.gmR);
    G.mrc = R.at<double>(V.gmrc);
    G.mirc = R.at<double>(V.gmirc);
    G.midx = R.at<int32_t>(V.gmidx);
    G.bpart = R.at<double>(V.gbpart);
    G.ccnt = R.at<int32_t>(V.gccnt);
    G.cfill = R.at<int32_t>(V.gcfill);
    G.ctmp = R.at<int32_t>(V.gctmp);
    G.sync = R.at<unsigned long long>(V.gsync);
    G.rmin = (long long *)(G.sync + 5);
    hipLaunchKernelGGL(k_bs_grid, dim3(nb), dim3(GT), 0, R.s, a, G);
    return hipGetLastError();
}

template <int NEXT>
static hipError_t sub_step(const LevelRun &R, int l, double dt_l, const AdjDev &A, const GroupDev &g);

// Level l >= 1 over list l - 1, sub-steps of dt_l.
static hipError_t advance(const LevelRun &R, int l, double dt_l)
{
    const LevelLayout &V = *R.V;
    const AdjDev A = adj_of(R, l);
    GroupDev g{};
    hipError_t e = groups_of(R, &g);
    for (int sub = 0; sub < R.p->substeps && e == hipSuccess; ++sub) {
        if (l < V.L - 1) e = sub_step<NEXT_ADJ>(R, l, dt_l, A, g);
        else if (V.direct) e = sub_step<NEXT_GROUPS>(R, l, dt_l, A, g);
        else e = sub_step<NEXT_NONE>(R, l, dt_l, A, g);
    }
    return e;
}

// A sub-step is bound by its launches, 4 to 7 us each whatever they do, so
// whatever has the same inputs shares one: 9 launches at the deepest level with
// the direct solver, 19 when each structure had its own (65,536 bodies, 3 x 4
// levels: 6.70 -> 5.39 ms per step with the solver's own change).
template <int NEXT>
static hipError_t sub_step(const LevelRun &R, int l, double dt_l, const AdjDev &A, const GroupDev &g)
{
    const LevelLayout &V = *R.V;
    const genga_params *p = R.p;
    const BodyDev up = R.bodies_of(l - 1);
    const ListDev list{up.bodies, up.nbod, R.b->n};
    hipError_t e;
    hipLaunchKernelGGL(k_level_radii<NEXT>, dim3(LG), dim3(LT), 0, R.s, up, R.at<double>(V.rc[l]),
                       p->m_star, dt_l, p->n1, p->n2, A, g);
    DetectDev d;
    d.in_i = R.at<int32_t>(V.pi[l - 1]);
    d.in_j = R.at<int32_t>(V.pj[l - 1]);
    d.in_cnt = R.at<int64_t>(V.cnt) + (l - 1);
    d.out_i = R.at<int32_t>(V.pi[l]);
    d.out_j = R.at<int32_t>(V.pj[l]);
    d.out_cnt = R.at<int64_t>(V.cnt) + l;
    d.lcount = R.at<int64_t>(V.lcount) + l;
    d.cap = V.cap;
    d.x = R.b->x; d.y = R.b->y; d.z = R.b->z;
    d.rc = R.at<double>(V.rc[l]);
    d.bcnt = R.at<int64_t>(V.bcnt);
    if ((e = level_kick(R, l, 0.5 * dt_l, &d)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_detect_write<NEXT>, dim3(DB), dim3(LT), 0, R.s, d, A, g);
    if (NEXT == NEXT_ADJ && (e = build_adj(R, l, list)) != hipSuccess) return e;
    if (NEXT == NEXT_GROUPS) build_groups(R, list, g);
    hipLaunchKernelGGL(k_drift_list<NEXT>, dim3(LG), dim3(LT), 0, R.s, up, p->G * p->m_star, dt_l, A,
                       g);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (NEXT == NEXT_ADJ && (e = advance(R, l + 1, dt_l / p->substeps)) != hipSuccess) return e;
    if (NEXT == NEXT_GROUPS) {
        const double *now[6] = {up.x, up.y, up.z, up.vx, up.vy, up.vz};
        if ((e = direct_solve(R, l, dt_l, now)) != hipSuccess) return e;
    }
    return level_kick(R, l, 0.5 * dt_l, nullptr);
}

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

LevelLayout make_level_layout(int64_t n, const genga_params *p, size_t base)
{
    LevelLayout V;
    if (!p || (p->slevels < 2 && !p->direct)) {
        V.total = base;
        return V;
    }
    V.L = p->slevels > 1 ? p->slevels : 1;
    V.direct = p->direct ? 1 : 0;
    V.cap = p->level_capacity;
    size_t off = align_up(base);
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    V.lcount = take(sizeof(int64_t) * V.L);
    V.cnt = take(sizeof(int64_t) * V.L);
    V.nbod = take(sizeof(int32_t) * V.L);
    V.bcnt = take(sizeof(int64_t) * DB);
    for (int l = 0; l < V.L; ++l) {
        V.pi[l] = take(sizeof(int32_t) * (size_t)V.cap);
        V.pj[l] = take(sizeof(int32_t) * (size_t)V.cap);
        if (l >= 1) V.rc[l] = take(sizeof(double) * (size_t)n);
        if (l < V.L - 1) {
            V.start[l] = take(sizeof(int32_t) * (size_t)(n + 1));
            V.adj[l] = take(sizeof(int32_t) * 2 * (size_t)V.cap);
            V.adj_tmp[l] = take(sizeof(int32_t) * 2 * (size_t)V.cap);
            V.owner[l] = take(sizeof(int32_t) * 2 * (size_t)V.cap);
            V.deg[l] = take(sizeof(int32_t) * (size_t)n);
            V.bodies[l] = take(sizeof(int32_t) * (size_t)n);
            if (l == 0) V.shadow[0] = take(sizeof(double) * 6 * (size_t)n);
        }
    }
    if (V.direct) {
        if (V.L == 1) V.shadow[0] = take(sizeof(double) * 6 * (size_t)n);
        V.glab = take(sizeof(int32_t) * (size_t)n);
        V.gflag = take(sizeof(int32_t) * (size_t)n);
        V.gsize = take(sizeof(int32_t) * (size_t)n);
        V.gslot = take(sizeof(int32_t) * (size_t)n);
        V.gstart = take(sizeof(int32_t) * (size_t)n);
        V.groot = take(sizeof(int32_t) * (size_t)n);
        V.gtmp = take(sizeof(int32_t) * (size_t)n);
        V.gmem = take(sizeof(int32_t) * (size_t)n);
        V.gcount = take(sizeof(int32_t) * 3);
        V.gstats = take(sizeof(int64_t) * 2);
        V.coll_count = take(sizeof(int64_t));
        V.coll_i = take(sizeof(int32_t) * LEVEL_COLL_CAP);
        V.coll_j = take(sizeof(int32_t) * LEVEL_COLL_CAP);
        V.coll_du = take(sizeof(double) * LEVEL_COLL_CAP);
        if (n > GROUP_BLOCK) {
            const int64_t gc = (n + GT - 1) / GT * GT;
            V.gcap = gc < GENGA_GROUP_MAX ? gc : GENGA_GROUP_MAX;
            const size_t c = (size_t)V.gcap;
            V.gbig = take(sizeof(int32_t) * (size_t)(2 + n / (GROUP_BLOCK + 1)));
            V.gsync = take(sizeof(uint64_t) * 8);
            V.gpub = take(sizeof(double) * 12 * c);
            V.gbox = take(sizeof(double) * 2 * (c / 64) * 8);
            V.gtrho = take(sizeof(double) * (c / 64));
            V.gmm = take(sizeof(double) * c);
            V.gmR = take(sizeof(double) * c);
            V.gmrc = take(sizeof(double) * c);
            V.gmirc = take(sizeof(double) * (size_t)V.L * c);
            V.gmidx = take(sizeof(int32_t) * c);
            V.gbpart = take(sizeof(double) * 4 * (c / 64));
            V.gccnt = take(sizeof(int32_t) * GCELL * GCELL);
            V.gcfill = take(sizeof(int32_t) * GCELL * GCELL);
            V.gctmp = take(sizeof(int32_t) * 2 * c);
        }
    }
    V.total = off;
    return V;
}

genga_pairs level0_pairs(const LevelLayout &V, char *ws)
{
    genga_pairs q;
    q.i = (int32_t *)(ws + V.pi[0]);
    q.j = (int32_t *)(ws + V.pj[0]);
    q.capacity = V.cap;
    q.count = (int64_t *)(ws + V.cnt);
    return q;
}

hipError_t levels_before_drift(const genga_bodies *b, const LevelLayout &V, genga_pairs *out,
                               char *ws, hipStream_t s)
{
    LevelRun R{const_cast<genga_bodies *>(b), nullptr, &V, ws, s};
    const int64_t *cnt0 = R.at<int64_t>(V.cnt);
    hipLaunchKernelGGL(k_level_begin, dim3(1), dim3(64), 0, s, R.at<int64_t>(V.lcount), V.L, cnt0,
                       V.direct ? R.at<int64_t>(V.gstats) : nullptr,
                       V.direct ? R.at<int64_t>(V.coll_count) : nullptr);
    if (out) {
        hipLaunchKernelGGL(k_copy_pairs, dim3(LG), dim3(LT), 0, s, R.at<int32_t>(V.pi[0]),
                           R.at<int32_t>(V.pj[0]), cnt0, V.cap, out->i, out->j, out->capacity,
                           out->count, R.status());
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int32_t *pi = R.at<int32_t>(V.pi[0]), *pj = R.at<int32_t>(V.pj[0]);
    const dim3 nb(R.list_blocks());
    if (V.L == 1) {
        // direct solver on E_0
        GroupDev g{};
        if ((e = groups_of(R, &g)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_group_begin, nb, dim3(LT), 0, s, g);
        hipLaunchKernelGGL(k_group_union, dim3(LG), dim3(LT), 0, s, pi, pj, cnt0, V.cap, g);
        build_groups(R, R.all(), g);
        hipLaunchKernelGGL(k_group_place, nb, dim3(LT), 0, s, R.bodies_of(0), g,
                           R.at<double>(V.shadow[0]));
        return hipGetLastError();
    }
    const AdjDev A = adj_of(R, 0);
    hipLaunchKernelGGL(k_adj_begin, nb, dim3(LT), 0, s, A);
    hipLaunchKernelGGL(k_adj_count, dim3(LG), dim3(LT), 0, s, pi, pj, cnt0, V.cap, A);
    if ((e = build_adj(R, 0, R.all())) != hipSuccess) return e;
    hipLaunchKernelGGL(k_state_list, dim3(LG), dim3(LT), 0, s, R.bodies_of(0),
                       R.at<double>(V.shadow[0]), b->n, 1);
    return hipGetLastError();
}

hipError_t levels_after_drift(genga_bodies *b, const genga_params *p, const LevelLayout &V,
                              char *ws, hipStream_t s)
{
    LevelRun R{b, p, &V, ws, s};
    if (V.L == 1) {
        const double *sh = R.at<double>(V.shadow[0]);
        const int64_t n = b->n;
        const double *saved[6] = {sh, sh + n, sh + 2 * n, sh + 3 * n, sh + 4 * n, sh + 5 * n};
        return direct_solve(R, 0, p->dt, saved);
    }
    hipLaunchKernelGGL(k_state_list, dim3(LG), dim3(LT), 0, s, R.bodies_of(0),
                       R.at<double>(V.shadow[0]), b->n, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return advance(R, 1, p->dt / p->substeps);
}

}  // namespace genga
