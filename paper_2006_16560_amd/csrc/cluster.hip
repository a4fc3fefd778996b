// Second-stage neighbour filter, clusters and SDAR groups (Sec. "Orbit-
// dependent neighbour criterion", Sec. "Clustering" and eq. rbin).
//
// Filter: a first-stage candidate j of i is kept iff the pericentre
// separation of the pair's two-body Kepler orbit is below c_v * r_nb,i.
// With r = x_j - x_i, v = v_j - v_i, mu = G (m_i + m_j): specific energy
// eps = v^2/2 - mu/|r|, angular momentum h = |r x v|, eccentricity
// e = sqrt(1 + 2 eps h^2/mu^2) and r_p = h^2 / (mu (1 + e)), over the whole
// orbit; r_p = 0 for coincident particles and |r x v|/|v| for two massless
// ones. FP64 without contraction, in this exact order, so that every
// decision is reproducible by any implementation of the same formula.
//
// Clusters: connected components of the kept pairs by a union-find whose
// roots are the smallest index of each component (so the result does
// not depend on the order of the unions).
#include <mutex>

#include "launch.h"

namespace petar {

namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(int64_t n, int threads, int64_t cap) {
    int64_t b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

__device__ double pericentre(double xi, double yi, double zi, double vxi, double vyi, double vzi,
                             double mi, double xj, double yj, double zj, double vxj, double vyj,
                             double vzj, double mj, double G) {
#pragma clang fp contract(off)
    double dx = xj - xi;
    double dy = yj - yi;
    double dz = zj - zi;
    double dvx = vxj - vxi;
    double dvy = vyj - vyi;
    double dvz = vzj - vzi;
    double d2 = (dx * dx + dy * dy) + dz * dz;
    double v2 = (dvx * dvx + dvy * dvy) + dvz * dvz;
    double hx = dy * dvz - dz * dvy;
    double hy = dz * dvx - dx * dvz;
    double hz = dx * dvy - dy * dvx;
    double h2 = (hx * hx + hy * hy) + hz * hz;
    double mu = G * (mi + mj);
    if (d2 == 0.0) return 0.0;
    if (mu > 0.0) {
        double d = sqrt(d2);
        double eps = 0.5 * v2 - mu / d;
        double e2 = 1.0 + ((2.0 * eps) * h2) / (mu * mu);
        double e = e2 > 0.0 ? sqrt(e2) : 0.0;
        return h2 / (mu * (1.0 + e));
    }
    return v2 > 0.0 ? sqrt(h2 / v2) : sqrt(d2);
}

// SDAR group relation (eq. rbin): r_ij < theta max(r_in,i, r_in,j), as
// d^2 < (theta R)^2 in FP64 without contraction, in this order.
__device__ bool group_pair(double xi, double yi, double zi, double ri, double xj, double yj,
                           double zj, double rj, double theta) {
#pragma clang fp contract(off)
    double dx = xj - xi;
    double dy = yj - yi;
    double dz = zj - zi;
    double d2 = sum_sq3(dx, dy, dz);
    double R = fmax(ri, rj);
    double g = theta * R;
    double g2 = g * g;
    return d2 < g2;
}

// CSR sanity: offsets start at 0 and never decrease (so every row range
// lies inside [0, offsets[n])); raises *bad otherwise.
__global__ __launch_bounds__(kThreads) void k_check_csr(const int64_t *offsets, int64_t n,
                                                        int32_t *bad) {
    int b = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (offsets[i + 1] < offsets[i]) b = 1;
        if (i == 0 && offsets[0] != 0) b = 1;
    }
    if (__ballot(b) && lane_id() == 0) atomicOr(bad, 1);
}

// The rows of a CSR by waves: a wave takes 64 consecutive rows, whose
// entries are consecutive, 64 entries at a time, one per lane. Rows differ
// widely (a massive star has a thousand neighbours, most have a few), and a
// thread per row took as long as the longest row: at 100k stars the passes
// of this file ran 20 to 260 us each, now 5 to 20.
struct RowLds {
    uint32_t head[kWave];  // row + 1 that starts at an entry of the chunk
};

struct RowWave {
    int64_t r0, e0, e1;  // first row, entry range
    int64_t beg, end;    // this lane's row
    uint32_t carry;      // last row + 1 seen so far
    RowLds *L;

    __device__ __forceinline__ void open(const int64_t *offsets, int64_t n, int64_t block,
                                         RowLds *l) {
        L = l;
        r0 = block * kWave;
        const int64_t r = r0 + lane_id();
        beg = offsets[r < n ? r : n];
        end = offsets[r + 1 < n ? r + 1 : n];
        const int64_t last = r0 + kWave < n ? r0 + kWave : n;
        e0 = offsets[r0];
        e1 = offsets[last];
        carry = 0;
    }
    // Row (0..63) of the entry base + lane; base goes from e0 to e1 by 64.
    // Lanes past the last entry get the last row.
    __device__ __forceinline__ int row(int64_t base) {
        wave_sync();
        L->head[lane_id()] = 0u;
        wave_sync();
        if (end > beg && beg >= base && beg < base + kWave)
            L->head[beg - base] = (uint32_t)lane_id() + 1u;
        wave_sync();
        uint32_t v = wave_incl_max(L->head[lane_id()]);
        v = v > carry ? v : carry;
        carry = last_lane(v);
        return (int)v - 1;
    }
};

inline unsigned row_grid(int64_t n) {
    return grid_for((n + kWave - 1) / kWave, kThreads / kWave, 16384);
}

// What the test reads of a star, in one record (64 B, or 32 B for the group
// relation) instead of seven (four) arrays: a candidate's partner is
// anywhere, and every array costs a memory transaction of its own. Packing reads
// and writes every star, so with fewer than one candidate in four stars the arrays
// are read instead (filter of three million stars with none, 0.10 and 0.25
// candidates a star: 186, 208 and 212 us from records, 78, 133 and 198 from the
// arrays; with 0.5: 227 and 296).
__device__ __forceinline__ bool packed(const FilterArgs &a) { return a.offsets[a.n] >= a.n / 4; }

__global__ __launch_bounds__(kThreads) void k_filter_pack(FilterArgs a, double4 *rec) {
    const int64_t n = a.n;
    if (!packed(a)) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double4 p = make_double4(a.pos[i], a.pos[n + i], a.pos[2 * n + i], a.r_nb[i]);
        if (a.mode == 1) {
            rec[i] = p;
        } else {
            rec[2 * i] = p;
            rec[2 * i + 1] = make_double4(a.vel[i], a.vel[n + i], a.vel[2 * n + i], a.mass[i]);
        }
    }
}

// Decision of every candidate entry: its bit in masks (one word per chunk of
// 64 entries, the chunks of row block b starting at word b + offsets[64 b] /
// 64) and the kept entries per row. An index outside [0, n) raises *bad.
// kRec: from the records of k_filter_pack, else from the arrays.
template <int MODE, bool kRec>
__device__ __forceinline__ void filter_test(const FilterArgs &a, const double4 *rec,
                                            uint64_t *masks, uint32_t *counts,
                                            FilterFlags *flags, RowLds *lds,
                                            uint32_t (*kept)[kWave]) {
    const int64_t n = a.n;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t nblk = (n + kWave - 1) / kWave;
    auto point = [&](int64_t i) {
        if constexpr (kRec) return rec[MODE == 1 ? i : 2 * i];
        return make_double4(a.pos[i], a.pos[n + i], a.pos[2 * n + i], a.r_nb[i]);
    };
    auto motion = [&](int64_t i) {
        if constexpr (kRec) return rec[2 * i + 1];
        return make_double4(a.vel[i], a.vel[n + i], a.vel[2 * n + i], a.mass[i]);
    };
    for (int64_t blk = (int64_t)blockIdx.x * (kThreads / kWave) + w; blk < nblk;
         blk += (int64_t)gridDim.x * (kThreads / kWave)) {
        RowWave rows;
        rows.open(a.offsets, n, blk, &lds[w]);
        wave_sync();
        kept[w][lane] = 0u;
        int64_t word = blk + rows.e0 / kWave;
        for (int64_t base = rows.e0; base < rows.e1; base += kWave, word++) {
            const int row = rows.row(base);
            const int64_t e = base + lane;
            bool keep = false;
            if (e < rows.e1) {
                const int64_t i = rows.r0 + row, j = a.idx[e];
                if (j < 0 || j >= n) {
                    atomicOr(&flags->bad, 1);
                } else {
                    const double4 pi = point(i), pj = point(j);
                    if constexpr (MODE == 1) {
                        keep = group_pair(pi.x, pi.y, pi.z, pi.w, pj.x, pj.y, pj.z, pj.w, a.c_v);
                    } else {
                        const double4 vi = motion(i), vj = motion(j);
                        keep = pericentre(pi.x, pi.y, pi.z, vi.x, vi.y, vi.z, vi.w, pj.x, pj.y,
                                          pj.z, vj.x, vj.y, vj.z, vj.w, a.G) < a.c_v * pi.w;
                    }
                }
                if (keep) atomicAdd(&kept[w][row], 1u);
            }
            const uint64_t m = __ballot(keep);
            if (lane == 0) masks[word] = m;
        }
        wave_sync();
        if (rows.r0 + lane < n) counts[rows.r0 + lane] = kept[w][lane];
    }
}

// When the CSR check failed or the words do not fit, flags->skip is all that is
// written. kRec: there are records, if k_filter_pack has packed them.
template <int MODE, bool kRec>
__global__ __launch_bounds__(kThreads) void k_filter_test(FilterArgs a, const double4 *rec,
                                                          uint64_t *masks, int64_t mask_cap,
                                                          uint32_t *counts, FilterFlags *flags) {
    __shared__ RowLds lds[kThreads / kWave];
    __shared__ uint32_t kept[kThreads / kWave][kWave];
    if (flags->csr_bad || filter_words(a.n, a.offsets[a.n]) > mask_cap) {
        if (blockIdx.x == 0 && threadIdx.x == 0) flags->skip = 1;
        return;
    }
    if constexpr (kRec) {
        if (packed(a)) {
            filter_test<MODE, true>(a, rec, masks, counts, flags, lds, kept);
            return;
        }
    }
    filter_test<MODE, false>(a, rec, masks, counts, flags, lds, kept);
}

// The kept entries of a row block are consecutive in the output too. Also
// the words the host reads: host[0] = kept entries, host[1] = candidates,
// host[2] = bad index, bad CSR.
__global__ __launch_bounds__(kThreads) void k_filter_write(FilterArgs a, const uint64_t *masks,
                                                           const int64_t *out_offsets,
                                                           int32_t *out_idx, int64_t capacity,
                                                           const FilterFlags *flags,
                                                           int64_t *host) {
    const int64_t n = a.n;
    const FilterFlags f = *flags;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        host[0] = f.skip ? 0 : out_offsets[n];
        host[1] = f.csr_bad ? 0 : a.offsets[n];
        host[2] = (f.bad ? 1 : 0) | (f.csr_bad ? 2 : 0);
    }
    if (f.skip || out_offsets[n] > capacity) return;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t nblk = (n + kWave - 1) / kWave;
    for (int64_t blk = (int64_t)blockIdx.x * (kThreads / kWave) + w; blk < nblk;
         blk += (int64_t)gridDim.x * (kThreads / kWave)) {
        const int64_t r0 = blk * kWave, last = r0 + kWave < n ? r0 + kWave : n;
        const int64_t e0 = a.offsets[r0], e1 = a.offsets[last];
        int64_t o = out_offsets[r0], word = blk + e0 / kWave;
        for (int64_t base = e0; base < e1; base += kWave, word++) {
            const unsigned long long m = masks[word];
            if (m >> lane & 1ull) out_idx[o + lanes_below(m)] = a.idx[base + lane];
            o += __popcll(m);
        }
    }
}

// ------------------------------------------------------------ components
// Union-find over the pairs. Every parent pointer goes to a smaller index
// (parent[v] <= v), so a root is the smallest index of its tree, and a union
// links the larger of two roots under the smaller with a compare-and-swap;
// after all unions each component is one tree whose root is its smallest
// index, whatever the order.
// The pairs are taken in three passes: each star's smallest neighbour (no
// swap needed; the start of ECL-CC, Jaiganesh and Burtscher 2018), its first and
// its last (neighbour sampling as in Afforest, Sutton et al. 2018), and then
// all, with the trees flattened in between. A pass reads the roots that the
// flattening left (a load inside a launch may return an older parent, since the
// L2 caches of the XCDs are not coherent within it) and goes on from there with
// loads and swaps at the coherence point. In one pass, every pair inside a
// percolating cluster climbed from its stars' old roots to the common root with
// swaps on the same few words, 2.7 ms at a million stars; after the sampling
// nearly all stars of such a cluster have the same root, and their pairs end
// with one comparison (0.1 ms).
// uf_root gives the root of v and leaves parent[v] there (where no swap runs at
// the same time). A chain is followed for kShallow steps; what is longer is
// shortened by all its stars at once: each star's pointer goes on to its parent's
// pointer, stored and read at the coherence point, until that is the root. (When
// each star walked the chain by itself, halving it behind it, three million stars
// in a row took 1 s, now 0.5 ms.)
constexpr int kShallow = 16;
__device__ __forceinline__ int32_t uf_root(int32_t *parent, int32_t v) {
    const int32_t first = parent[v];
    int32_t cur = first, next = parent[cur];
    for (int k = 0; k < kShallow && next != cur; k++) {
        cur = next;
        next = parent[cur];
    }
    if (next == cur) {
        if (cur != first) parent[v] = cur;
        return cur;
    }
    while (next != cur) {
        cur = next;
        __hip_atomic_store(parent + v, cur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        next = __hip_atomic_load(parent + cur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return cur;
}

// parent[v] = min(v, smallest in-range neighbour of v). Skipped when the
// CSR check failed (offsets could then reach outside the index array).
__global__ __launch_bounds__(kThreads) void k_uf_init(const int64_t *offsets, const int32_t *idx,
                                                      int64_t n, int32_t *parent,
                                                      const int32_t *csr_bad) {
    __shared__ RowLds lds[kThreads / kWave];
    __shared__ int32_t low[kThreads / kWave][kWave];
    if (*csr_bad) return;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t nblk = (n + kWave - 1) / kWave;
    for (int64_t blk = (int64_t)blockIdx.x * (kThreads / kWave) + w; blk < nblk;
         blk += (int64_t)gridDim.x * (kThreads / kWave)) {
        RowWave rows;
        rows.open(offsets, n, blk, &lds[w]);
        wave_sync();
        low[w][lane] = (int32_t)(rows.r0 + lane);
        for (int64_t base = rows.e0; base < rows.e1; base += kWave) {
            const int row = rows.row(base);
            if (base + lane < rows.e1) {
                const int32_t u = idx[base + lane];
                if (u >= 0 && u < rows.r0 + row) atomicMin(&low[w][row], u);
            }
        }
        wave_sync();
        if (rows.r0 + lane < n) parent[rows.r0 + lane] = low[w][lane];
    }
}

// Every particle straight to the end of its chain, so that the next pass
// starts from flat trees.
__global__ __launch_bounds__(kThreads) void k_uf_flatten(int32_t *parent, int64_t n,
                                                         const int32_t *csr_bad) {
    if (*csr_bad) return;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x)
        (void)uf_root(parent, (int32_t)v);
}

// Joins the trees of a and b, ancestors of two stars (or the stars). Trees that
// the pass itself has made deep are halved on the way from kJoinSteps on (a
// million stars of a lattice, each with its neighbours of larger index only: 0.95
// ms instead of 1.27); earlier, the stores slow every other climb down (lists of
// 20 neighbours: 1.45 ms from 8 on, 0.96 from 32 on).
constexpr int kJoinSteps = 32;
__device__ __forceinline__ void uf_join(int32_t *parent, int32_t a, int32_t b) {
    for (int k = 0; a != b; k++) {
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        int32_t p = __hip_atomic_load(parent + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (p == a) {
            p = atomicCAS(parent + a, a, b);
            if (p == a) return;
        } else if (k >= kJoinSteps) {
            const int32_t q =
                __hip_atomic_load(parent + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (q != p) {
                __hip_atomic_store(parent + a, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                p = q;
            }
        }
        a = p;  // a smaller ancestor of a
    }
}

// Two pairs per row: its first entry and its last.
__global__ __launch_bounds__(kThreads) void k_uf_sample(const int64_t *offsets, const int32_t *idx,
                                                        int64_t n, int32_t *parent,
                                                        const int32_t *csr_bad) {
    if (*csr_bad) return;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t beg = offsets[v], end = offsets[v + 1];
        if (beg == end) continue;
        const int32_t u = idx[beg], w = idx[end - 1], r = parent[v];
        if (u >= 0 && u < n) uf_join(parent, r, parent[u]);
        if (w != u && w >= 0 && w < n) uf_join(parent, r, parent[w]);
    }
}

__global__ __launch_bounds__(kThreads) void k_uf_union(const int64_t *offsets, const int32_t *idx,
                                                       int64_t n, int32_t *parent, int32_t *bad,
                                                       const int32_t *csr_bad) {
    __shared__ RowLds lds[kThreads / kWave];
    if (*csr_bad) return;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t nblk = (n + kWave - 1) / kWave;
    for (int64_t blk = (int64_t)blockIdx.x * (kThreads / kWave) + w; blk < nblk;
         blk += (int64_t)gridDim.x * (kThreads / kWave)) {
        RowWave rows;
        rows.open(offsets, n, blk, &lds[w]);
        for (int64_t base = rows.e0; base < rows.e1; base += kWave) {
            const int64_t v = rows.r0 + rows.row(base);
            if (base + lane < rows.e1) {
                const int32_t u = idx[base + lane];
                if (u < 0 || u >= n)
                    atomicOr(bad, 1);
                else
                    uf_join(parent, parent[v], parent[u]);
            }
        }
    }
}

// Labels from the final trees (every particle alone when the CSR check
// failed, so that the later passes stay in bounds before the error returns).
__global__ __launch_bounds__(kThreads) void k_uf_label(int32_t *parent, int64_t n, int32_t *label,
                                                       uint32_t *is_root, const int32_t *csr_bad) {
    const bool skip = *csr_bad != 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = skip ? (int32_t)v : uf_root(parent, (int32_t)v);
        label[v] = r;
        is_root[v] = r == (int32_t)v ? 1u : 0u;
    }
}

// Sort keys for the member lists: cluster index per particle (a stable
// radix sort by it keeps the members of each cluster ascending).
__global__ __launch_bounds__(kThreads) void k_cl_keys(const int32_t *label, int64_t n,
                                                      const uint32_t *root_pos, uint64_t *key,
                                                      uint32_t *val) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        key[i] = root_pos[label[i]];
        val[i] = (uint32_t)i;
    }
}

// Cluster offsets from the sorted cluster indices: a cluster starts where
// its index first appears; entries past the last cluster are n. Also the
// words the host reads: host[0] = clusters, host[1] = the two flags.
__global__ __launch_bounds__(kThreads) void k_cl_offsets(const uint64_t *key, int64_t n,
                                                         int64_t *cl_offsets,
                                                         const uint32_t *n_clusters,
                                                         const int32_t *flags, int64_t *host) {
    const int64_t nc = *n_clusters;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i >= nc) cl_offsets[i] = n;
        if (i < n && (i == 0 || key[i] != key[i - 1])) cl_offsets[key[i]] = i;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        host[0] = nc;
        host[1] = (flags[0] ? 1 : 0) | (flags[1] ? 2 : 0);
    }
}

__global__ __launch_bounds__(kThreads) void k_group_pairs(const int64_t *off, const int32_t *mem,
                                                          int64_t n_groups, const double *pos,
                                                          const double *vel, const double *mass,
                                                          int64_t n, double G, uint32_t *is_pair) {
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_groups;
         g += (int64_t)gridDim.x * blockDim.x) {
        uint32_t f = 0;
        if (off[g + 1] - off[g] == 2) {
            const int64_t i = mem[off[g]], j = mem[off[g] + 1];
            const double r[3] = {pos[j] - pos[i], pos[n + j] - pos[n + i],
                                 pos[2 * n + j] - pos[2 * n + i]};
            const double v[3] = {vel[j] - vel[i], vel[n + j] - vel[n + i],
                                 vel[2 * n + j] - vel[2 * n + i]};
            const double mu = G * (mass[i] + mass[j]);
            double rr;
            const double E = kepler_energy(r, v, mu, &rr);
            f = (rr > 0.0 && E < 0.0) ? 1u : 0u;
        }
        is_pair[g] = f;
    }
}

__global__ __launch_bounds__(kThreads) void k_group_pairs_write(const int64_t *off,
                                                                const int32_t *mem,
                                                                int64_t n_groups,
                                                                const uint32_t *is_pair,
                                                                const uint32_t *pos,
                                                                int32_t *pairs, int64_t cap,
                                                                int64_t *host) {
    if (blockIdx.x == 0 && threadIdx.x == 0) host[0] = pos[n_groups];
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_groups;
         g += (int64_t)gridDim.x * blockDim.x) {
        if (!is_pair[g]) continue;
        const int64_t k = pos[g];
        pairs[k] = mem[off[g]];
        pairs[cap + k] = mem[off[g] + 1];
    }
}

}  // namespace

void launch_group_pairs(const int64_t *grp_offsets, const int32_t *members, int64_t n_groups,
                        const double *pos, const double *vel, const double *mass, int64_t n,
                        double G, uint32_t *is_pair, hipStream_t s) {
    hipLaunchKernelGGL(k_group_pairs, dim3(grid_for(n_groups, kThreads, 8192)), dim3(kThreads), 0,
                       s, grp_offsets, members, n_groups, pos, vel, mass, n, G, is_pair);
}

void launch_group_pairs_write(const int64_t *grp_offsets, const int32_t *members, int64_t n_groups,
                              const uint32_t *is_pair, const uint32_t *pos, int32_t *pairs,
                              int64_t pair_cap, int64_t *host, hipStream_t s) {
    hipLaunchKernelGGL(k_group_pairs_write, dim3(grid_for(n_groups, kThreads, 8192)),
                       dim3(kThreads), 0, s, grp_offsets, members, n_groups, is_pair, pos, pairs,
                       pair_cap, host);
}

void launch_check_csr(const int64_t *offsets, int64_t n, int32_t *bad, hipStream_t s) {
    hipLaunchKernelGGL(k_check_csr, dim3(grid_for(n, kThreads, 8192)), dim3(kThreads), 0, s,
                       offsets, n, bad);
}

void launch_filter(const FilterArgs &a, double *rec, uint64_t *masks, int64_t mask_cap,
                   uint32_t *counts, FilterFlags *flags, hipStream_t s) {
    const dim3 g(row_grid(a.n)), b(kThreads);
    double4 *r = reinterpret_cast<double4 *>(rec);
    if (rec)
        hipLaunchKernelGGL(k_filter_pack, dim3(grid_for(a.n, kThreads, 8192)), b, 0, s, a, r);
#define TEST(MODE, REC)                                                                        \
    hipLaunchKernelGGL((k_filter_test<MODE, REC>), g, b, 0, s, a, (const double4 *)r, masks,   \
                       mask_cap, counts, flags)
    if (a.mode == 1) {
        if (rec)
            TEST(1, true);
        else
            TEST(1, false);
    } else {
        if (rec)
            TEST(0, true);
        else
            TEST(0, false);
    }
#undef TEST
}

void launch_filter_write(const FilterArgs &a, const uint64_t *masks, const int64_t *out_offsets,
                         int32_t *out_idx, int64_t capacity, const FilterFlags *flags,
                         int64_t *host, hipStream_t s) {
    hipLaunchKernelGGL(k_filter_write, dim3(row_grid(a.n)), dim3(kThreads), 0, s, a, masks,
                       out_offsets, out_idx, capacity, flags, host);
}

void launch_components(const int64_t *offsets, const int32_t *idx, int64_t n, int32_t *parent,
                       int32_t *label, uint32_t *is_root, int32_t *bad, const int32_t *csr_bad,
                       hipStream_t s) {
    // a thread per star: the stars of smaller indices, which chains lead to, start
    // first, so that a chain's halving begins at its root
    const dim3 g(grid_for(n, kThreads, INT32_MAX)), b(kThreads);
    const dim3 gr(row_grid(n));
    hipLaunchKernelGGL(k_uf_init, gr, b, 0, s, offsets, idx, n, parent, csr_bad);
    hipLaunchKernelGGL(k_uf_flatten, g, b, 0, s, parent, n, csr_bad);
    hipLaunchKernelGGL(k_uf_sample, g, b, 0, s, offsets, idx, n, parent, csr_bad);
    hipLaunchKernelGGL(k_uf_flatten, g, b, 0, s, parent, n, csr_bad);
    hipLaunchKernelGGL(k_uf_union, gr, b, 0, s, offsets, idx, n, parent, bad, csr_bad);
    hipLaunchKernelGGL(k_uf_label, g, b, 0, s, parent, n, label, is_root, csr_bad);
}

void launch_cluster_keys(const int32_t *label, int64_t n, const uint32_t *root_pos, uint64_t *key,
                         uint32_t *val, hipStream_t s) {
    hipLaunchKernelGGL(k_cl_keys, dim3(grid_for(n, kThreads, 8192)), dim3(kThreads), 0, s, label,
                       n, root_pos, key, val);
}

void launch_cluster_offsets(const uint64_t *sorted_key, int64_t n, int64_t *cl_offsets,
                            const uint32_t *n_clusters, const int32_t *flags, int64_t *host,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_cl_offsets, dim3(grid_for(n + 1, kThreads, 8192)), dim3(kThreads), 0, s,
                       sorted_key, n, cl_offsets, n_clusters, flags, host);
}

namespace {

// The scratch of petar_clusters_noalloc. Its name is a host-side stand-in
// in host code: kernels get the per-device address kept below.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];

}  // namespace

hipError_t noalloc_scratch(int device, void **out, size_t *bytes) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    *bytes = sizeof(scratch);
    return hipSuccess;
}

}  // namespace petar
