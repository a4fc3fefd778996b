// Long-range force kernels: group-wise tree walk fused with the interaction
// passes, persistent over per-XCD work queues; one wavefront per i-group
// (k_force) or, when there are too few groups to fill the chip that way, a
// team of waves (k_force_team), with the same result bit for bit.
//
// Per group the walk sorts every cell it reaches into
//   multipole (PC): the cell is inside the opening angle and no pair can be
//                   within search range -> monopole + quadrupole field;
//   far leaf:       opened leaf out of search range -> Newtonian pairs;
//   near leaf:      opened leaf within search range -> pairs weighted by
//                   the changeover functions (1 - K) and (1 - W)/r.
// Cells are buffered in LDS; a full buffer is staged as records relative to
// the group centre (FP32 in mixed mode, FP64 otherwise) and broadcast from
// LDS to all lanes. A lane holds up to IPL targets; small groups spread one
// target over S lanes that split the j loop. In mixed precision each tile of
// at most 64 sources is summed in FP32 and the tile partials are accumulated
// in FP64 (two instructions per component and tile; a Neumaier-compensated
// FP32 sum takes seven).
#include <algorithm>

#include "launch.h"
#include "walk.h"

namespace petar {

namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;
constexpr float kFarAway = 1e18f;  // position of padding records (zero mass)

template <typename R>
struct Vec;
template <>
struct Vec<float> {
    using v4 = float4;
    using v2 = float2;
};
template <>
struct Vec<double> {
    using v4 = double4;
    using v2 = double2;
};

// Tiles of up to 64 sources (plus padding); every read is an aligned
// 16/8/4-byte broadcast:
//   multipoles: a = (x, y, z, M), b = 2 (A'xx, A'yy, A'zz, A'xy), c = 2 (A'xz, A'yz)
//   particles:  a = (x, y, z, m), c = (r_in, r_out), k = index in Morton order
//               (far leaves use a only)
// Multipole entries are written by the walk as soon as a cell is accepted
// (its data are already in registers); particle entries are expanded from
// the buffered leaves when those are flushed.
constexpr int kTileCap = 72;  // 64 entries + padding up to a multiple of the loop step

template <typename R>
struct PcEntry {
    typename Vec<R>::v4 a, b;
    typename Vec<R>::v2 c, pad;
};
template <typename R>
struct PartEntry {
    typename Vec<R>::v4 a;
    typename Vec<R>::v2 c;
    uint32_t k, pad[sizeof(R) == 4 ? 1 : 3];
};
// Array of entries: one LDS base per tile, immediate offsets per field.
template <typename R>
struct PcTile {
    PcEntry<R> e[kTileCap];
};
template <typename R>
struct PartTile {
    PartEntry<R> e[kTileCap];
};

template <typename R>
struct WaveLds {
    uint32_t stack[kStackLds + kStackSlack];
    uint32_t far_start[kWave], far_pre[kWave];
    uint32_t near_start[kWave], near_pre[kWave];
    GroupGeom g;
    PcTile<R> pc;
    PartTile<R> part;
};

__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// FP64 reciprocal square root and reciprocal from the hardware's estimates
// (about 24 bits) and a third-order, respectively two second-order Newton
// corrections with exact residuals. Where the residual is not a number (0,
// infinity, NaN) the estimate is the result. Within 0.5005 and 0.5001 ulp of
// the exact results for arguments from 2^-980 to 2^980 and 2^-520 to 2^1000
// (1.0 / sqrt(x): 1.49), at about a quarter of the instructions.
__device__ __forceinline__ double rsq(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double h = x * y, hl = fma(x, y, -h);
    const double e = fma(-hl, y, fma(-h, y, 1.0));  // 1 - x y^2
    const double z = fma(y * e, fma(e, 0.375, 0.5), y);
    return e == e ? z : y;
}
__device__ __forceinline__ double rcp(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double z = fma(y, fma(-x, y, 1.0), y);
    const double e = fma(-x, z, 1.0);
    return e == e ? fma(z, e, z) : y;
}

// Accumulators: FP64 sums of the tile partials (FP32 partials in mixed
// precision, FP64 ones otherwise).
template <typename R>
struct Acc;
template <>
struct Acc<float> {
    double s[4];  // FP64 sums of the FP32 tile partials
    __device__ void zero() {
        for (int k = 0; k < 4; k++) s[k] = 0.0;
    }
    __device__ void add(int k, float v) { s[k] += (double)v; }
    __device__ double get(int k) const { return s[k]; }
};
template <>
struct Acc<double> {
    double s[4];
    __device__ void zero() {
        for (int k = 0; k < 4; k++) s[k] = 0.0;
    }
    __device__ void add(int k, double v) { s[k] += v; }
    __device__ double get(int k) const { return s[k]; }
};

template <typename R, int IPL>
struct Targets {
    R x[IPL], y[IPL], z[IPL], rin[IPL], rout[IPL];
    uint32_t k[IPL];  // index in Morton order, kNone for an empty slot
};

// Where a tile's sums go: into the FP64 accumulators of the wave that walks
// (AccSink), or into registers until the tile's turn (TileSums).
template <typename R, int IPL>
struct AccSink {
    Acc<R> acc[IPL];
    __device__ __forceinline__ void put(int u, int k, R v) { acc[u].add(k, v); }
    template <int U>
    __device__ __forceinline__ void rest() {}
};
template <typename R, int IPL>
struct TileSums {
    R v[IPL][4];
    __device__ __forceinline__ void put(int u, int k, R x) { v[u][k] = x; }
    // every loop sets every value, so that they stay in registers
    template <int U>
    __device__ __forceinline__ void rest() {
#pragma unroll
        for (int u = U; u < IPL; u++)
#pragma unroll
            for (int k = 0; k < 4; k++) v[u][k] = (R)0;
    }
};

// Work layout of a chunk of targets. nu target slots per lane are in use;
// W lanes hold one slot each of distinct targets, and S = 64 / W such lane
// sets split the source loop (lane = sl * W + il). Lanes past S * W idle:
// they mirror split 0 and their sums are dropped. Everything but sl, il and
// act is wave-uniform.
struct Layout {
    int nu, W, S;
    int sl, il;
    bool act;
};

// Chooses (nu, S) to keep as many lanes busy as possible: nu = 1 with
// S = 64 / active lanes per target, or, when the kernel holds two targets
// per lane and it is better, nu = 2 with S = 64 / ceil(active/2); chunks
// above 64 targets use nu = ceil(active / 64), S = 1. Splits up to
// kSplitFixed have loops of their own (fixed stride, unrolled, tiles padded
// to the step); wider ones (groups of at most 7 targets) share a loop with
// the stride in a register and no padding.
template <int IPL>
__device__ __forceinline__ Layout choose_layout(uint32_t active) {
    Layout ly;
    if (active > (uint32_t)kWave) {
        ly.nu = (int)((active + kWave - 1) / kWave);
        ly.W = kWave;
        ly.S = 1;
    } else {
        const int a = (int)active;
        const int S1 = kWave / a;
        ly.nu = 1;
        ly.W = a;
        ly.S = S1;
        if (IPL >= 2 && a >= 2) {
            const int W2 = (a + 1) / 2;
            const int S2 = kWave / W2;
            if (S2 > 2 * S1) {  // utilisation a * S / (64 * nu) is higher
                ly.nu = 2;
                ly.W = W2;
                ly.S = S2;
            }
        }
    }
    const int lane = lane_id();
    ly.sl = lane / ly.W;
    ly.il = lane - ly.sl * ly.W;
    ly.act = ly.sl < ly.S;
    if (!ly.act) ly.sl = 0;
    return ly;
}

// ---------------------------------------------------------------- loops
// Each loop runs uniformly over a tile padded to a multiple of its step
// F * S: S lanes share a target and take every S-th source, F sources per
// lane are unrolled per iteration.
enum { kTilePc = 0, kTileFar = 1, kTileNear = 2 };
constexpr int kSplitFixed = 8;  // widest split with a fixed-stride loop

__host__ __device__ constexpr int unroll_of(int kind, int S) {
    return kind == kTileFar ? (S >= 4 ? 1 : 4 / S) : (kind == kTilePc && S <= 4 ? 2 : 1);
}
__device__ __forceinline__ int pad_to(int m, int kind, int S) {
    if (S > kSplitFixed) return m;  // runtime stride: lanes past the end are masked
    const int q = unroll_of(kind, S) * S;
    return (m + q - 1) / q * q;
}

template <typename R, int U>
struct Partial {
    R ax[U], ay[U], az[U], ph[U];
    __device__ void zero() {
#pragma unroll
        for (int u = 0; u < U; u++) ax[u] = ay[u] = az[u] = ph[u] = (R)0;
    }
};

// Multipole term of one cell: with R the target minus the centre of mass,
// q = A'R and the tile holding 2A' (so q2 = 2q):
//   a   += (2/r^5) A'R - (M/r^3 + 5 R.A'R/r^7) R
//   phi -= M/r + R.A'R/r^5
template <typename R, int IPL, int U>
__device__ __forceinline__ void pc_one(const typename Vec<R>::v4 &a, const typename Vec<R>::v4 &b,
                                       const typename Vec<R>::v2 &c, const Targets<R, IPL> &T,
                                       Partial<R, U> &P) {
#pragma unroll
    for (int u = 0; u < U; u++) {
        R Rx = T.x[u] - a.x, Ry = T.y[u] - a.y, Rz = T.z[u] - a.z;
        R r2 = Rx * Rx + Ry * Ry + Rz * Rz;
        R ri = rsq(r2);
        R ri2 = ri * ri;
        R qx = b.x * Rx + b.w * Ry + c.x * Rz;  // 2 A'R
        R qy = b.w * Rx + b.y * Ry + c.y * Rz;
        R qz = c.x * Rx + c.y * Ry + b.z * Rz;
        R rqr = Rx * qx + Ry * qy + Rz * qz;    // 2 R.A'R
        R ri5 = ri * (ri2 * ri2);
        R mri = a.w * ri;                       // M/r
        R t2 = rqr * ri5;                       // 2 R.A'R / r^5
        R coef = ((R)2.5 * t2 + mri) * ri2;     // M/r^3 + 5 R.A'R/r^7
        P.ax[u] += ri5 * qx;
        P.ay[u] += ri5 * qy;
        P.az[u] += ri5 * qz;
        P.ax[u] -= coef * Rx;
        P.ay[u] -= coef * Ry;
        P.az[u] -= coef * Rz;
        P.ph[u] -= mri;
        P.ph[u] -= (R)0.5 * t2;
    }
}

template <typename R, int IPL, int U>
__device__ __forceinline__ void far_one(const typename Vec<R>::v4 &p, const Targets<R, IPL> &T,
                                        Partial<R, U> &P) {
#pragma unroll
    for (int u = 0; u < U; u++) {
        R dx = p.x - T.x[u], dy = p.y - T.y[u], dz = p.z - T.z[u];
        R r2 = dx * dx + dy * dy + dz * dz;
        R ri = rsq(r2);
        R mri = p.w * ri;
        R mri3 = mri * ri * ri;
        P.ax[u] += mri3 * dx;
        P.ay[u] += mri3 * dy;
        P.az[u] += mri3 * dz;
        P.ph[u] -= mri;
    }
}

template <typename R, int IPL, int U>
__device__ __forceinline__ void near_one(const typename Vec<R>::v4 &p,
                                         const typename Vec<R>::v2 &rr, uint32_t kj,
                                         const Targets<R, IPL> &T, Partial<R, U> &P) {
#pragma unroll
    for (int u = 0; u < U; u++) {
        R dx = p.x - T.x[u], dy = p.y - T.y[u], dz = p.z - T.z[u];
        R r2 = dx * dx + dy * dy + dz * dz;
        R rin = T.rin[u] > rr.x ? T.rin[u] : rr.x;
        R rout = T.rout[u] > rr.y ? T.rout[u] : rr.y;
        R ri = r2 > (R)0 ? rsq(r2) : (R)0;
        R r = r2 * ri;
        R dr = rout - rin;
        R sum = rout + rin;
        R x = (r - rin) * rcp(dr);
        R lam = dr * rcp(sum);
        R xc = x < (R)0 ? (R)0 : (x > (R)1 ? (R)1 : x);
        R x2 = xc * xc, x4 = x2 * x2;
        R xm = xc - (R)1, xm2 = xm * xm;
        // 1 - K(x) = x^4 [(35 - 84x + 70x^2 - 20x^3) - 35 Lambda (x-1)^4]
        R fw = x4 * (((R)35 + xc * ((R)-84 + xc * ((R)70 - (R)20 * xc))) -
                     (R)35 * lam * xm2 * xm2);
        // (1 - W)/r = 2/(r_in + r_out) - Lambda x^5 (14 - 28x + 20x^2 - 5x^3)/r
        R pw_in = (R)2 * rcp(sum) -
                  lam * x4 * xc * ((R)14 + xc * ((R)-28 + xc * ((R)20 - (R)5 * xc))) * ri;
        R pw = x >= (R)1 ? ri : pw_in;
        bool self = kj == T.k[u];
        fw = self ? (R)0 : fw;
        pw = self ? (R)0 : pw;
        R mf = p.w * fw * ri * ri * ri;
        P.ax[u] += mf * dx;
        P.ay[u] += mf * dy;
        P.az[u] += mf * dz;
        P.ph[u] -= p.w * pw;
    }
}

// mpad is a multiple of the step F * S.
template <int KIND, int U, int S, typename R, int IPL, typename TileT, typename Sink>
__device__ void loop_kind(const TileT &tile, int mpad, int sl, const Targets<R, IPL> &T,
                          Sink &sink) {
    constexpr int F = unroll_of(KIND, S);
    Partial<R, U> P;
    P.zero();
    for (int jj = 0; jj < mpad; jj += F * S) {
#pragma unroll
        for (int f = 0; f < F; f++) {
            const int j = jj + f * S + sl;
            if constexpr (KIND == kTilePc)
                pc_one<R, IPL, U>(tile.e[j].a, tile.e[j].b, tile.e[j].c, T, P);
            else if constexpr (KIND == kTileFar)
                far_one<R, IPL, U>(tile.e[j].a, T, P);
            else
                near_one<R, IPL, U>(tile.e[j].a, tile.e[j].c, tile.e[j].k, T, P);
        }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        sink.put(u, 0, P.ax[u]);
        sink.put(u, 1, P.ay[u]);
        sink.put(u, 2, P.az[u]);
        sink.put(u, 3, P.ph[u]);
    }
    sink.template rest<U>();
}

// Splits wider than kSplitFixed: the stride S is a register, each lane
// takes entries sl, sl + S, ... below m (no padding).
template <int KIND, int U, typename R, int IPL, typename TileT, typename Sink>
__device__ void loop_kind_wide(const TileT &tile, int m, int sl, int S, const Targets<R, IPL> &T,
                               Sink &sink) {
    Partial<R, U> P;
    P.zero();
    for (int j = sl; j < m; j += S) {
        if constexpr (KIND == kTilePc)
            pc_one<R, IPL, U>(tile.e[j].a, tile.e[j].b, tile.e[j].c, T, P);
        else if constexpr (KIND == kTileFar)
            far_one<R, IPL, U>(tile.e[j].a, T, P);
        else
            near_one<R, IPL, U>(tile.e[j].a, tile.e[j].c, tile.e[j].k, T, P);
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        sink.put(u, 0, P.ax[u]);
        sink.put(u, 1, P.ay[u]);
        sink.put(u, 2, P.az[u]);
        sink.put(u, 3, P.ph[u]);
    }
    sink.template rest<U>();
}

// Runs the loop of a staged tile for the chunk's layout (nu, S).
template <int KIND, typename R, int IPL, typename TileT, typename Sink>
__device__ __forceinline__ void run_tile(const TileT &tile, int mpad, const Layout &ly,
                                         const Targets<R, IPL> &T, Sink &sink) {
    if constexpr (IPL > 2) {
        if (ly.nu > 2) {
            loop_kind<KIND, IPL, 1>(tile, mpad, ly.sl, T, sink);
            return;
        }
    }
    if (ly.S > kSplitFixed) {
        if constexpr (IPL >= 2) {
            if (ly.nu == 2) {
                loop_kind_wide<KIND, 2>(tile, mpad, ly.sl, ly.S, T, sink);
                return;
            }
        }
        loop_kind_wide<KIND, 1>(tile, mpad, ly.sl, ly.S, T, sink);
        return;
    }
    if constexpr (IPL >= 2) {
        if (ly.nu == 2) {
            switch (ly.S) {
                case 1: loop_kind<KIND, 2, 1>(tile, mpad, ly.sl, T, sink); break;
                case 2: loop_kind<KIND, 2, 2>(tile, mpad, ly.sl, T, sink); break;
                case 3: loop_kind<KIND, 2, 3>(tile, mpad, ly.sl, T, sink); break;
                case 4: loop_kind<KIND, 2, 4>(tile, mpad, ly.sl, T, sink); break;
                case 5: loop_kind<KIND, 2, 5>(tile, mpad, ly.sl, T, sink); break;
                case 6: loop_kind<KIND, 2, 6>(tile, mpad, ly.sl, T, sink); break;
                case 7: loop_kind<KIND, 2, 7>(tile, mpad, ly.sl, T, sink); break;
                default: loop_kind<KIND, 2, 8>(tile, mpad, ly.sl, T, sink); break;
            }
            return;
        }
    }
    switch (ly.S) {
        case 1: loop_kind<KIND, 1, 1>(tile, mpad, ly.sl, T, sink); break;
        case 2: loop_kind<KIND, 1, 2>(tile, mpad, ly.sl, T, sink); break;
        case 3: loop_kind<KIND, 1, 3>(tile, mpad, ly.sl, T, sink); break;
        case 4: loop_kind<KIND, 1, 4>(tile, mpad, ly.sl, T, sink); break;
        case 5: loop_kind<KIND, 1, 5>(tile, mpad, ly.sl, T, sink); break;
        case 6: loop_kind<KIND, 1, 6>(tile, mpad, ly.sl, T, sink); break;
        case 7: loop_kind<KIND, 1, 7>(tile, mpad, ly.sl, T, sink); break;
        default: loop_kind<KIND, 1, 8>(tile, mpad, ly.sl, T, sink); break;
    }
}

// ---- multipole tile: entries [0, npc) were written by the walk; pads the
// tile to the loop's multiple and runs it.
template <typename R, int IPL>
__device__ void flush_pc(WaveLds<R> &L, int npc, const Layout &ly, const Targets<R, IPL> &T,
                         AccSink<R, IPL> &A) {
    const int mpad = pad_to(npc, kTilePc, ly.S);
    for (int t = npc + lane_id(); t < mpad; t += kWave) pad_entry(L.pc.e[t]);
    wave_sync();
    run_tile<kTilePc>(L.pc, mpad, ly, T, A);
    wave_sync();
}

// Multipole entry of cell data held in registers (relative to the group
// centre; traceless quadrupole A' = 3/2 S - 1/2 tr(S) I of the second
// moment S about the centre of mass). FP32: the doubled A' and M come
// rounded from the build (nd_q); FP64: from the second moments.
template <typename R>
struct CellQuad;
template <>
struct CellQuad<float> {
    float4 q0, q1;
    __device__ void load(const TreeDev &t, uint32_t nd) {
        q0 = t.nd_q[2 * (int64_t)nd];
        q1 = t.nd_q[2 * (int64_t)nd + 1];
    }
};
template <>
struct CellQuad<double> {
    double2 s01, s23, s45;
    __device__ void load(const TreeDev &t, uint32_t nd) {
        const double2 *Sp = reinterpret_cast<const double2 *>(t.nd_S) + (int64_t)nd * 3;
        s01 = Sp[0];
        s23 = Sp[1];
        s45 = Sp[2];
    }
};

__device__ __forceinline__ void stage_entry(PcEntry<float> &e, const double4 &cm,
                                            const CellQuad<float> &q, const GroupGeom &G) {
    e.a = {(float)(cm.x - G.c[0]), (float)(cm.y - G.c[1]), (float)(cm.z - G.c[2]), q.q1.z};
    e.b = q.q0;
    e.c = {q.q1.x, q.q1.y};
}
__device__ __forceinline__ void stage_entry(PcEntry<double> &e, const double4 &cm,
                                            const CellQuad<double> &q, const GroupGeom &G) {
    const double2 s01 = q.s01, s23 = q.s23, s45 = q.s45;
    const double tr = s01.x + s01.y + s23.x;
    e.a = {cm.x - G.c[0], cm.y - G.c[1], cm.z - G.c[2], cm.w};
    e.b = {2.0 * (1.5 * s01.x - 0.5 * tr), 2.0 * (1.5 * s01.y - 0.5 * tr),
           2.0 * (1.5 * s23.x - 0.5 * tr), 2.0 * (1.5 * s23.y)};
    e.c = {2.0 * (1.5 * s45.x), 2.0 * (1.5 * s45.y)};
}

// Padding: a source of zero mass far away.
template <typename R>
__device__ __forceinline__ void pad_entry(PcEntry<R> &e) {
    e.a = {(R)kFarAway, (R)kFarAway, (R)kFarAway, (R)0};
    e.b = {(R)0, (R)0, (R)0, (R)0};
    e.c = {(R)0, (R)0};
}
template <typename R>
__device__ __forceinline__ void pad_entry(PartEntry<R> &e) {
    e.a = {(R)kFarAway, (R)kFarAway, (R)kFarAway, (R)0};
    e.c = {(R)0, (R)1};
    e.k = kNone - 1;
}

// Binary search of the buffered leaf that holds expanded slot s.
__device__ __forceinline__ int find_leaf(const uint32_t *pre, int nleaf, uint32_t s) {
    int lo = 0, hi = nleaf;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (pre[mid] <= s)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Source particle k (position p) into an entry of the particle tile.
template <int KIND, typename R>
__device__ __forceinline__ void stage_particle(PartEntry<R> &e, const double4 &p, uint32_t k,
                                               const ForceLaunch &f, const GroupGeom &G) {
    e.a = {(R)(p.x - G.c[0]), (R)(p.y - G.c[1]), (R)(p.z - G.c[2]), (R)p.w};
    if (KIND == kTileNear) {
        const double2 rr = f.t.rr[k];
        e.c = {(R)rr.x, (R)rr.y};
        e.k = k;
    }
}

// Hands one flush of near leaves (lane l: start[l], c particles) of a group
// to the neighbour passes: a header and the flushed leaves.
__device__ __forceinline__ void record_leaves(const ForceLaunch &f, const uint32_t *start,
                                              uint32_t c, int nleaf, uint32_t gstart,
                                              uint32_t gn) {
    const int lane = lane_id();
    uint32_t hb = 0, lb = 0;
    if (lane == 0) {  // both counts in one claim (count is 8-byte aligned)
        const unsigned long long c2 =
            atomicAdd((unsigned long long *)f.nb.count,
                      1ull | ((unsigned long long)(uint32_t)nleaf << 32));
        hb = (uint32_t)c2;
        lb = (uint32_t)(c2 >> 32);
    }
    hb = (uint32_t)uniform((int)hb);
    lb = (uint32_t)uniform((int)lb);
    if (hb < f.nb.head_cap && (uint64_t)lb + (uint64_t)nleaf <= f.nb.leaf_cap) {
        if (lane < nleaf) f.nb.leaf[lb + lane] = make_uint2(start[lane], c);
        if (lane == 0) f.nb.head[hb] = make_uint4(gstart, gn, lb, (uint32_t)nleaf);
    }
}

// ---- leaves (far: Newtonian pairs; near: changeover pairs). On entry
// pre[] holds each buffered leaf's particle count; it is turned into an
// exclusive prefix and the particles are expanded in tiles of 64. Returns
// the number of source particles run. kSub: a force on a subset of targets
// (no neighbour lists), where particles of zero mass are dropped as sources
// (their terms are zero) and the rest packed to the front of the tile.
template <int KIND, bool kSub, typename R, int IPL>
__device__ uint32_t flush_leaves(WaveLds<R> &L, const uint32_t *start, uint32_t *pre, int nleaf,
                                 const ForceLaunch &f, const Layout &ly,
                                 const Targets<R, IPL> &T, AccSink<R, IPL> &A, bool record,
                                 uint32_t gstart, uint32_t gn) {
    wave_sync();
    const int lane = lane_id();
    uint32_t c = lane < nleaf ? pre[lane] : 0u;
    if (KIND == kTileNear && record) record_leaves(f, start, c, nleaf, gstart, gn);
    uint32_t incl = wave_incl_scan(c);
    uint32_t total = last_lane(incl);
    if (lane < nleaf) pre[lane] = incl - c;
    wave_sync();
    uint32_t kept = 0;
    for (uint32_t base = 0; base < total; base += kWave) {
        const uint32_t s = base + lane;
        int m = (int)(total - base < (uint32_t)kWave ? total - base : (uint32_t)kWave);
        bool have = false;
        if (s < total) {
            const int l = find_leaf(pre, nleaf, s);
            const uint32_t k = start[l] + (s - pre[l]);
            const double4 p = f.t.ps[k];
            have = p.w != 0.0;
            stage_particle<KIND>(L.part.e[lane], p, k, f, L.g);
        }
        if constexpr (kSub) {
            // move the entries with mass to the front of the tile
            const unsigned long long km = __ballot(have);
            if (km != (m == kWave ? ~0ull : (1ull << m) - 1ull)) {
                wave_sync();
                const typename Vec<R>::v4 a = L.part.e[lane].a;
                typename Vec<R>::v2 c = {(R)0, (R)0};
                uint32_t k = 0;
                if (KIND == kTileNear) {
                    c = L.part.e[lane].c;
                    k = L.part.e[lane].k;
                }
                wave_sync();
                if (have) {
                    const int e = lanes_below(km);
                    L.part.e[e].a = a;
                    if (KIND == kTileNear) {
                        L.part.e[e].c = c;
                        L.part.e[e].k = k;
                    }
                }
                m = __popcll(km);
            }
        }
        const int mpad = pad_to(m, KIND, ly.S);
        for (int t = m + lane; t < mpad; t += kWave) {
            L.part.e[t].a = {(R)kFarAway, (R)kFarAway, (R)kFarAway, (R)0};
            if (KIND == kTileNear) {
                L.part.e[t].c = {(R)0, (R)1};
                L.part.e[t].k = kNone - 1;
            }
        }
        wave_sync();
        run_tile<KIND>(L.part, mpad, ly, T, A);
        wave_sync();
        kept += (uint32_t)m;
    }
    return kept;
}

// Folds the partial sums of the S lanes that split one target's sources
// into the lane of split 0, in the fixed order of the splits (staged in the
// multipole tile, which is free once the walk of the chunk is done).
template <typename R>
__device__ __forceinline__ void fold_in(Acc<R> &a, const double *src, int k, int lane2) {
    a.s[k] += src[k * kWave + lane2];
}
template <typename R>
__device__ __forceinline__ void park(const Acc<R> &a, double *dst, int lane) {
    for (int k = 0; k < 4; k++) dst[k * kWave + lane] = a.s[k];
}

template <typename R, int IPL>
__device__ void combine_split(WaveLds<R> &L, AccSink<R, IPL> &A, const Layout &ly) {
    static_assert(sizeof(PcTile<R>) >= 4 * kWave * sizeof(double), "fold buffer");
    double *buf = reinterpret_cast<double *>(&L.pc);
    const int lane = lane_id();
#pragma unroll
    for (int u = 0; u < IPL; u++) {
        if (u >= ly.nu) break;
        wave_sync();
        park(A.acc[u], buf, lane);
        wave_sync();
        if (ly.act && ly.sl == 0) {
            for (int s2 = 1; s2 < ly.S; s2++) {
                const int lane2 = s2 * ly.W + ly.il;
#pragma unroll
                for (int k = 0; k < 4; k++) fold_in(A.acc[u], buf, k, lane2);
            }
        }
    }
    wave_sync();
}

enum { kKindNone = 0, kKindPc = 1, kKindFar = 2, kKindNear = 3, kKindOpen = 4 };

// Long-range kick fused into the output write (eq. lfmap: v += a_L dt with
// dt the half step), v + a dt rounded twice as written.
__device__ __forceinline__ void kick_add(double *v, double a, double dt) {
#pragma clang fp contract(off)
    *v = *v + a * dt;
}

// Queue q's groups: its eighth of the n_big large ones, which are listed
// first, then its eighth of the others.
__device__ __forceinline__ uint32_t eighths(uint32_t n, int q) {
    return (n >> 3) * (uint32_t)q + ((n & 7u) * (uint32_t)q >> 3);  // n q / 8
}
__device__ __forceinline__ uint32_t queue_size(uint32_t groups, uint32_t big, int q) {
    const uint32_t rest = groups - big;
    return eighths(big, q + 1) - eighths(big, q) + eighths(rest, q + 1) - eighths(rest, q);
}
__device__ __forceinline__ uint32_t queue_group(uint32_t groups, uint32_t big, int q, uint32_t v) {
    const uint32_t rest = groups - big;
    const uint32_t first = eighths(big, q), many = eighths(big, q + 1) - first;
    return v < many ? first + v : big + eighths(rest, q) + (v - many);
}

// Work queues, one per XCD: contiguous ranges of the groups (Morton order);
// a worker whose queue is empty goes on to the next one. A queue that may be
// empty is looked at before it is claimed from (a stale head costs one claim
// more): when every wave of the chip claimed from all eight queues before it
// stopped, those 32,768 adds on one cache line took 0.43 ms of a launch whose
// waves all end together (0.47 ms at a thousand stars); at ten million, where
// the ends are further apart than that, nothing. The heads lie in lines of
// their own.
// In the queues of the teams the workers take the first groups by their rank
// without a claim; with few groups there is no claim at all.
struct GroupQueue {
    uint32_t *heads;
    uint32_t n_groups, n_big;
    uint32_t rank;  // this worker's in its queue
    int q, moves;
    bool first, sure;

    __device__ __forceinline__ GroupQueue(uint32_t *h, const Status *s)
        : heads(h), n_groups((uint32_t)s->n_groups), n_big((uint32_t)s->n_big),
          rank(blockIdx.x >> 3), q((int)(blockIdx.x & 7u)), moves(0), first(true), sure(false) {}

    // Next group of this wave, -1 when all are taken.
    __device__ __forceinline__ int64_t next() {
        while (moves < 8) {
            const uint32_t size = queue_size(n_groups, n_big, q);
            const uint32_t nstat = (gridDim.x + 7u - (uint32_t)q) >> 3;
            uint32_t v = size;
            if (first) {
                v = rank;
            } else if (size > nstat) {
                uint32_t h = 0;
                if (lane_id() == 0) {
                    uint32_t *head = heads + q * kQueueStride;
                    if (!sure)
                        h = __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (sure || nstat + h < size) h = atomicAdd(head, 1u);
                }
                v = nstat + (uint32_t)uniform((int)h);
            }
            first = false;
            sure = v + 2 * nstat < size;  // not yet near the end
            if (v < size) return queue_group(n_groups, n_big, q, v);
            moves++;
            q = (q + 1) & 7;
        }
        return -1;
    }
};

// kSub: the targets are the listed subset (tpos, tidx) and cells and
// particles of zero mass are no sources; otherwise every particle is a
// target.
template <typename R, int IPL, bool kSub>
__global__ __launch_bounds__(kThreads, sizeof(R) == 4 && IPL == 2 ? 4 : 1) void k_force(ForceLaunch f) {
    __shared__ WaveLds<R> lds_all[kWavesPerBlock];
    const int w = threadIdx.x / kWave;
    WaveLds<R> &L = lds_all[w];
    const int lane = lane_id();
    const int64_t gwave = (int64_t)blockIdx.x * kWavesPerBlock + w;
    if (f.st_in->invalid_radii || f.st_in->cell_overflow) return;
    const uint32_t n_groups = (uint32_t)f.st_in->n_groups, n_big = (uint32_t)f.st_in->n_big;
    const int64_t n = f.t.n;
    WaveStack stk;
    stk.lds = L.stack;
    stk.spill = f.spill + gwave * kSpillCap;
    unsigned long long cnt_pc = 0, cnt_far = 0, cnt_near = 0;
    // theta^2 held in a vector register: as a scalar it shares a register
    // tuple with other kernel arguments, which the compiler spills and then
    // reloads whole at every walk step
    double th2 = f.th2;
    asm volatile("" : "+v"(th2));
    int q = blockIdx.x & 7;  // work queue of this XCD
    int moves = 0;
    const int CH = kWave * IPL;
    while (true) {
        const uint32_t size = queue_size(n_groups, n_big, q);
        uint32_t v = 0;
        if (lane == 0) {
            uint32_t *head = f.queue + q * kQueueStride;
            if (moves > 0)
                v = __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v < size) v = atomicAdd(head, 1u);
        }
        v = (uint32_t)uniform((int)v);
        const int64_t g = queue_group(n_groups, n_big, q, v);
        if (v >= size) {
            if (++moves >= 8) break;
            q = (q + 1) & 7;
            continue;
        }
        const uint32_t gnode = (uint32_t)uniform((int)f.groups[g]);
        const uint4 ginfo = f.t.nd_info[gnode];
        const uint32_t gstart = (uint32_t)uniform((int)ginfo.x);
        const uint32_t gn = (uint32_t)uniform((int)ginfo.y);
        // the group's targets: all its particles, or the listed subset
        uint32_t t0 = gstart, tn = gn;
        if constexpr (kSub) {
            t0 = (uint32_t)uniform((int)f.tpos[gstart]);
            tn = (uint32_t)uniform((int)f.tpos[gstart + gn]) - t0;
            if (tn == 0) continue;  // sources only: no walk
        }
        wave_sync();
        if (lane == 0) L.g = load_group(f.t.nd_lo, f.t.nd_hi, gnode);
        wave_sync();
        for (uint32_t chunk = 0; chunk < tn; chunk += CH) {
            const uint32_t active = tn - chunk < (uint32_t)CH ? tn - chunk : (uint32_t)CH;
            const Layout ly = choose_layout<IPL>(active);
            Targets<R, IPL> T;
            AccSink<R, IPL> A;
#pragma unroll
            for (int u = 0; u < IPL; u++) {
                uint32_t off = chunk + u * ly.W + ly.il;
                bool valid = ly.act && u < ly.nu && off < tn;
                uint32_t k = kSub ? f.tidx[t0 + (valid ? off : 0u)] : gstart + (valid ? off : 0u);
                double4 p = f.t.ps[k];
                double2 rr = f.t.rr[k];
                T.x[u] = (R)(p.x - L.g.c[0]);
                T.y[u] = (R)(p.y - L.g.c[1]);
                T.z[u] = (R)(p.z - L.g.c[2]);
                T.rin[u] = (R)rr.x;
                T.rout[u] = (R)rr.y;
                T.k[u] = valid ? k : kNone;
                A.acc[u].zero();
            }
            uint64_t n_pc = 0, n_far = 0, n_near = 0;
            int npc = 0, nfar = 0, nnear = 0;
            const bool record = f.nb.head != nullptr && chunk == 0;
            stk.init((uint32_t)uniform((int)root_of(f.t.nd_info, f.t.level_off, gstart)));
            bool ok = true;
            while (!stk.empty()) {
                const uint32_t node = stk.pop();
                // Lanes without a cell classify cell 0 (always present) and
                // are then marked idle: the wave issues these instructions
                // for all lanes anyway, and no default values are needed.
                const bool live = node != kNone;
                const uint32_t nd = live ? node : 0u;
                const double4 lo = f.t.nd_lo[nd], hi = f.t.nd_hi[nd];
                const double4 cm = f.t.nd_com[nd];
                CellQuad<R> quad;
                quad.load(f.t, nd);
                const uint4 info = f.t.nd_info[nd];
                double D2, R2;
                box_terms(L.g, lo, hi, &D2, &R2);
                const bool near = D2 < R2;
                const bool accept = mac_accept(L.g, cm, hi.w, th2) & !near;
                int kind = !live ? kKindNone
                                 : (accept ? kKindPc
                                           : ((info.z & kLeafFlag)
                                                  ? (near ? kKindNear : kKindFar)
                                                  : kKindOpen));
                // on a subset of targets (no neighbour lists), a cell of zero
                // mass is dropped with its subtree: it exerts no force
                if constexpr (kSub) {
                    if (cm.w == 0.0) kind = kKindNone;
                }
                int nc = kind == kKindOpen ? info_nchild(info.z) : 0;
                if (!stk.push(info.w, nc)) {
                    ok = false;
                    break;
                }
                unsigned long long m;
                int cnt;
                // Each buffer is filled to 64 entries before it is run: a
                // batch that does not fit completes it, the buffer is run,
                // and the rest of the batch (still in the lanes' registers)
                // starts the next one.
                m = __ballot(kind == kKindPc);
                cnt = __popcll(m);
                if (cnt) {
                    const int p = npc + lanes_below(m);
                    if (kind == kKindPc && p < kWave) stage_entry(L.pc.e[p], cm, quad, L.g);
                    if (npc + cnt >= kWave) {
                        flush_pc(L, kWave, ly, T, A);
                        n_pc += kWave;
                        if (kind == kKindPc && p >= kWave)
                            stage_entry(L.pc.e[p - kWave], cm, quad, L.g);
                        npc += cnt - kWave;
                    } else {
                        npc += cnt;
                    }
                }
                m = __ballot(kind == kKindFar);
                cnt = __popcll(m);
                if (cnt) {
                    const int p = nfar + lanes_below(m);
                    if (kind == kKindFar && p < kWave) {
                        L.far_start[p] = info.x;
                        L.far_pre[p] = info.y;
                    }
                    if (nfar + cnt >= kWave) {
                        n_far += flush_leaves<kTileFar, kSub>(L, L.far_start, L.far_pre, kWave,
                                                              f, ly, T, A, false, gstart,
                                                              gn);
                        if (kind == kKindFar && p >= kWave) {
                            L.far_start[p - kWave] = info.x;
                            L.far_pre[p - kWave] = info.y;
                        }
                        nfar += cnt - kWave;
                    } else {
                        nfar += cnt;
                    }
                }
                m = __ballot(kind == kKindNear);
                cnt = __popcll(m);
                if (cnt) {
                    const int p = nnear + lanes_below(m);
                    if (kind == kKindNear && p < kWave) {
                        L.near_start[p] = info.x;
                        L.near_pre[p] = info.y;
                    }
                    if (nnear + cnt >= kWave) {
                        n_near += flush_leaves<kTileNear, kSub>(L, L.near_start, L.near_pre,
                                                                kWave, f, ly, T, A, record, gstart,
                                                                gn);
                        if (kind == kKindNear && p >= kWave) {
                            L.near_start[p - kWave] = info.x;
                            L.near_pre[p - kWave] = info.y;
                        }
                        nnear += cnt - kWave;
                    } else {
                        nnear += cnt;
                    }
                }
            }
            if (!ok) {
                if (lane == 0) atomicAdd(&f.st->stack_overflow, 1);
                break;
            }
            if (npc) {
                wave_sync();
                flush_pc(L, npc, ly, T, A);
                n_pc += npc;
            }
            if (nfar)
                n_far += flush_leaves<kTileFar, kSub>(L, L.far_start, L.far_pre, nfar, f, ly, T,
                                                      A, false, gstart, gn);
            if (nnear)
                n_near += flush_leaves<kTileNear, kSub>(L, L.near_start, L.near_pre, nnear, f, ly,
                                                        T, A, record, gstart, gn);
            cnt_pc += n_pc * active;
            cnt_far += n_far * active;
            // minus the self pairs: every target's, or on a subset (massless
            // sources dropped) those of the targets with mass
            uint32_t n_self = active;
            if constexpr (kSub) {
                n_self = 0;
#pragma unroll
                for (int u = 0; u < IPL; u++) {
                    const bool own = T.k[u] != kNone && ly.sl == 0;
                    n_self += (uint32_t)__popcll(
                        __ballot(own && f.t.ps[own ? T.k[u] : 0u].w != 0.0));
                }
            }
            cnt_near += n_near * active - n_self;
            if (ly.S > 1) combine_split(L, A, ly);
#pragma unroll
            for (int u = 0; u < IPL; u++) {
                if (T.k[u] == kNone || ly.sl != 0) continue;
                uint32_t o = f.t.orig[T.k[u]];
                const double ax = f.G * A.acc[u].get(0), ay = f.G * A.acc[u].get(1),
                             az = f.G * A.acc[u].get(2);
                f.acc[o] = ax;
                f.acc[n + o] = ay;
                f.acc[2 * n + o] = az;
                f.pot[o] = f.G * A.acc[u].get(3);
                if (f.kick_vel) {
                    kick_add(f.kick_vel + o, ax, f.kick_dt);
                    kick_add(f.kick_vel + n + o, ay, f.kick_dt);
                    kick_add(f.kick_vel + 2 * n + o, az, f.kick_dt);
                }
                if (f.nb_bound) f.nb_bound[o] = (uint32_t)n_near;
                if (f.counts) {
                    f.counts[o] = (int32_t)n_pc;
                    f.counts[n + o] = (int32_t)n_far;
                    f.counts[2 * n + o] = (int32_t)n_near;
                    f.counts[3 * n + o] = (int32_t)gn;
                }
            }
        }
    }
    // one add per block and counter: the adds of a launch queue on one line
    __shared__ unsigned long long total[kWavesPerBlock][3];
    if (lane == 0) {
        total[w][0] = cnt_pc;
        total[w][1] = cnt_far;
        total[w][2] = cnt_near;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long v = 0;
        for (int k = 0; k < kWavesPerBlock; k++) v += total[k][threadIdx.x];
        if (v) atomicAdd(&f.st->inter[threadIdx.x], v);
    }
}

// ---------------------------------------------------------------- team
// One i-group by a workgroup of T waves. One wave walks the tree and
// publishes tiles (up to 64 accepted cells, or 64 particles of the listed
// leaves, as indices); every other wave, and the walker once its walk is
// done, claims tiles in turn, stages them in its own part of LDS and sums
// them, and each tile's FP32 sums are added to the FP64 accumulators in LDS
// in the order of the tiles, so the result is that of k_force bit for bit.
//
// Counters (LDS): pub = tiles published, with kTeamEnd when the walk is
// done; claim = tiles taken; done = tiles added. A wave waits for its tile
// to be published and, with its sums, for the tiles before it to be added:
// tile t - 1 was claimed earlier by a wave that waits for nothing later than
// t - 2. The walker waits only for places held by published tiles. So every
// wait ends.
constexpr int kTeamPc = 8;             // lists of accepted cells in flight
constexpr int kTeamTasks = 16;
constexpr uint32_t kTeamEnd = 0x80000000u;

template <typename R>
union TeamTile {
    PcTile<R> pc;
    PartTile<R> part;
};

template <typename R, int IPL, int T>
struct TeamLds {
    uint32_t stack[kStackLds + kStackSlack];
    uint32_t cell[kTeamPc][kWave];
    uint32_t leaf_start[4][kWave], leaf_pre[4][kWave];  // lists 0, 1: far; 2, 3: near
    TeamTile<R> tile[T];
    double acc[IPL][4][kWave];
    uint4 task[kTeamTasks];          // kind | list << 4, first place, leaves, entries
    uint32_t pub, claim, done;
    uint32_t kept[2];                // particles run, far and near (kSub)
    uint32_t chunk, fail;
    uint32_t n_pc, n_far, n_near;
    int64_t group;                   // -1: no more
};

__device__ __forceinline__ uint32_t lds_acquire(const uint32_t *p) {
    return (uint32_t)uniform(
        (int)__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
}
// Every lane stores the same value: a branch on the lane here, at the end of
// a loop whose head branches on the lane too, may be merged with that one,
// and the wave's lanes then go round the loop apart.
__device__ __forceinline__ void lds_release(uint32_t *p, uint32_t v) {
    wave_sync();
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
}

// The walker's side of the tiles. `seen` is a lower bound of `done`, so that
// the counter is read only when a place may still be in use.
template <typename R, int IPL, int T>
struct TeamFeed {
    TeamLds<R, IPL, T> &L;
    const ForceLaunch &f;
    uint32_t t, seen;       // tiles published; tiles known to be added
    uint32_t last[kTeamPc]; // tiles published when each list of cells was, oldest first
    uint32_t far_last, near_last;
    int pcs, farl, nearl;   // lists being filled
    uint32_t n_pc, n_far, n_near;

    __device__ __forceinline__ TeamFeed(TeamLds<R, IPL, T> &L_, const ForceLaunch &f_)
        : L(L_), f(f_), t(0), seen(0), far_last(0), near_last(0), pcs(0), farl(0), nearl(2),
          n_pc(0), n_far(0), n_near(0) {
#pragma unroll
        for (int k = 0; k < kTeamPc; k++) last[k] = 0;
    }
    __device__ __forceinline__ void need(uint32_t d) {
        while ((int32_t)(seen - d) < 0) {
            seen = lds_acquire(&L.done);
            if ((int32_t)(seen - d) < 0) __builtin_amdgcn_s_sleep(1);
        }
    }
    __device__ __forceinline__ void publish(const uint4 &task) {
        if (t >= (uint32_t)kTeamTasks) need(t - kTeamTasks + 1);
        if (lane_id() == 0) L.task[t % kTeamTasks] = task;
        lds_release(&L.pub, ++t);
    }
    // m accepted cells of the current list; goes on to the next one
    __device__ __forceinline__ void cells(int m) {
        publish(make_uint4(kTilePc | (uint32_t)pcs << 4, 0u, 0u, (uint32_t)m));
        n_pc += (uint32_t)m;
        pcs = (pcs + 1) % kTeamPc;
#pragma unroll
        for (int k = 0; k + 1 < kTeamPc; k++) last[k] = last[k + 1];
        last[kTeamPc - 1] = t;
        need(last[0]);
    }
    // nleaf buffered leaves of `list`: hands near ones over, turns the counts
    // into their exclusive prefix and publishes 64 particles at a time
    template <int KIND>
    __device__ __forceinline__ uint32_t leaves(int list, int nleaf, bool record, uint32_t gstart,
                                               uint32_t gn) {
        wave_sync();
        const int lane = lane_id();
        const uint32_t c = lane < nleaf ? L.leaf_pre[list][lane] : 0u;
        if (KIND == kTileNear && record)
            record_leaves(f, L.leaf_start[list], c, nleaf, gstart, gn);
        const uint32_t incl = wave_incl_scan(c);
        const uint32_t total = last_lane(incl);
        if (lane < nleaf) L.leaf_pre[list][lane] = incl - c;
        for (uint32_t base = 0; base < total; base += kWave) {
            const uint32_t m = total - base < (uint32_t)kWave ? total - base : (uint32_t)kWave;
            publish(make_uint4(KIND | (uint32_t)list << 4, base, (uint32_t)nleaf, m));
        }
        return total;
    }
    __device__ __forceinline__ void far(int nleaf, uint32_t gstart, uint32_t gn) {
        n_far += leaves<kTileFar>(farl, nleaf, false, gstart, gn);
        need(far_last);  // the other list's tiles
        far_last = t;
        farl ^= 1;
    }
    __device__ __forceinline__ void near(int nleaf, bool record, uint32_t gstart, uint32_t gn) {
        n_near += leaves<kTileNear>(nearl, nleaf, record, gstart, gn);
        need(near_last);
        near_last = t;
        nearl ^= 1;
    }
};

// What the walk reads of a cell.
struct CellData {
    double4 lo, hi, cm;
    uint4 info;
    __device__ __forceinline__ void load(const TreeDev &t, uint32_t nd) {
        lo = t.nd_lo[nd];
        hi = t.nd_hi[nd];
        cm = t.nd_com[nd];
        info = t.nd_info[nd];
    }
};

// The walk of one group (chunk); publishes every tile and ends with pub.
template <typename R, int IPL, int T, bool kSub>
__device__ void team_walk(TeamLds<R, IPL, T> &L, const ForceLaunch &f, const GroupGeom &G,
                          uint32_t gstart, uint32_t gn, bool record, uint32_t *spill,
                          double th2) {
    WaveStack stk;
    stk.lds = L.stack;
    stk.spill = spill;
    stk.init((uint32_t)uniform((int)root_of(f.t.nd_info, f.t.level_off, gstart)));
    TeamFeed<R, IPL, T> feed(L, f);
    int npc = 0, nfar = 0, nnear = 0;
    uint32_t node = stk.pop();
    CellData cell;
    cell.load(f.t, node != kNone ? node : 0u);
    while (true) {
        double D2, R2;
        box_terms(G, cell.lo, cell.hi, &D2, &R2);
        const bool is_near = D2 < R2;
        const bool accept = mac_accept(G, cell.cm, cell.hi.w, th2) & !is_near;
        int kind = node == kNone
                       ? kKindNone
                       : (accept ? kKindPc
                                 : ((cell.info.z & kLeafFlag) ? (is_near ? kKindNear : kKindFar)
                                                              : kKindOpen));
        if constexpr (kSub) {
            if (cell.cm.w == 0.0) kind = kKindNone;
        }
        const uint32_t nd = node, first = cell.info.x, count = cell.info.y;
        if (!stk.push(cell.info.w, kind == kKindOpen ? info_nchild(cell.info.z) : 0)) {
            if (lane_id() == 0) {
                atomicAdd(&f.st->stack_overflow, 1);
                L.fail = 1u;
            }
            break;
        }
        // the next cells are loaded while these are listed
        const bool more = !stk.empty();
        if (more) {
            node = stk.pop();
            cell.load(f.t, node != kNone ? node : 0u);
        }
        unsigned long long m = __ballot(kind == kKindPc);
        if (m) {
            const int p = npc + lanes_below(m);
            if (kind == kKindPc && p < kWave) L.cell[feed.pcs][p] = nd;
            npc += __popcll(m);
            if (npc >= kWave) {
                feed.cells(kWave);
                npc -= kWave;
                if (kind == kKindPc && p >= kWave) L.cell[feed.pcs][p - kWave] = nd;
            }
        }
        m = __ballot(kind == kKindFar);
        if (m) {
            const int p = nfar + lanes_below(m);
            if (kind == kKindFar && p < kWave) {
                L.leaf_start[feed.farl][p] = first;
                L.leaf_pre[feed.farl][p] = count;
            }
            nfar += __popcll(m);
            if (nfar >= kWave) {
                feed.far(kWave, gstart, gn);
                nfar -= kWave;
                if (kind == kKindFar && p >= kWave) {
                    L.leaf_start[feed.farl][p - kWave] = first;
                    L.leaf_pre[feed.farl][p - kWave] = count;
                }
            }
        }
        m = __ballot(kind == kKindNear);
        if (m) {
            const int p = nnear + lanes_below(m);
            if (kind == kKindNear && p < kWave) {
                L.leaf_start[feed.nearl][p] = first;
                L.leaf_pre[feed.nearl][p] = count;
            }
            nnear += __popcll(m);
            if (nnear >= kWave) {
                feed.near(kWave, record, gstart, gn);
                nnear -= kWave;
                if (kind == kKindNear && p >= kWave) {
                    L.leaf_start[feed.nearl][p - kWave] = first;
                    L.leaf_pre[feed.nearl][p - kWave] = count;
                }
            }
        }
        if (!more) {
            if (npc) feed.cells(npc);
            if (nfar) feed.far(nfar, gstart, gn);
            if (nnear) feed.near(nnear, record, gstart, gn);
            break;
        }
    }
    if (lane_id() == 0) {
        L.n_pc = feed.n_pc;
        L.n_far = feed.n_far;
        L.n_near = feed.n_near;
    }
    lds_release(&L.pub, feed.t | kTeamEnd);
}

// Entries [base, base + m) of a list of leaves into a particle tile; returns
// the entries (fewer than m when kSub drops particles of zero mass).
template <int KIND, bool kSub, typename R, typename Lds>
__device__ __forceinline__ int team_stage(const Lds &L, PartTile<R> &tile, int list,
                                          uint32_t base, int nleaf, int m, const ForceLaunch &f,
                                          const GroupGeom &G) {
    const int lane = lane_id();
    double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
    uint32_t k = 0;
    bool have = false;
    int e = lane;
    if (lane < m) {
        const uint32_t *pre = L.leaf_pre[list];
        const uint32_t s = base + (uint32_t)lane;
        const int l = find_leaf(pre, nleaf, s);
        k = L.leaf_start[list][l] + (s - pre[l]);
        p = f.t.ps[k];
        have = !kSub || p.w != 0.0;
    }
    if constexpr (kSub) {  // entries with mass to the front
        const unsigned long long km = __ballot(have);
        e = lanes_below(km);
        m = __popcll(km);
    }
    if (have) stage_particle<KIND>(tile.e[e], p, k, f, G);
    return m;
}

template <typename R, int IPL, int T, bool kSub>
__device__ void team_consume(TeamLds<R, IPL, T> &L, TeamTile<R> &buf, const ForceLaunch &f,
                             const GroupGeom &G, const Layout &ly, const Targets<R, IPL> &tg) {
    const int lane = lane_id();
    while (true) {
        uint32_t t = 0;
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) t = atomicAdd(&L.claim, 1u);
        __builtin_amdgcn_wave_barrier();
        t = (uint32_t)uniform((int)t);
        uint32_t pub;
        while (true) {
            pub = lds_acquire(&L.pub);
            if (t < (pub & ~kTeamEnd) || (pub & kTeamEnd)) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (t >= (pub & ~kTeamEnd)) return;
        const uint4 task = L.task[t % kTeamTasks];
        const int kind = uniform((int)task.x) & 15, list = uniform((int)task.x) >> 4;
        int m = uniform((int)task.w);
        TileSums<R, IPL> P;
        wave_sync();
        if (kind == kTilePc) {
            if (lane < m) {
                const uint32_t nd = L.cell[list][lane];
                CellQuad<R> quad;
                quad.load(f.t, nd);
                stage_entry(buf.pc.e[lane], f.t.nd_com[nd], quad, G);
            }
            const int mpad = pad_to(m, kTilePc, ly.S);
            if (m + lane < mpad) pad_entry(buf.pc.e[m + lane]);
            wave_sync();
            run_tile<kTilePc>(buf.pc, mpad, ly, tg, P);
        } else {
            const uint32_t base = (uint32_t)uniform((int)task.y);
            const int nleaf = uniform((int)task.z);
            const bool far = kind == kTileFar;
            if (far)
                m = team_stage<kTileFar, kSub>(L, buf.part, list, base, nleaf, m, f, G);
            else
                m = team_stage<kTileNear, kSub>(L, buf.part, list, base, nleaf, m, f, G);
            const int mpad = pad_to(m, kind, ly.S);
            if (m + lane < mpad) pad_entry(buf.part.e[m + lane]);
            wave_sync();
            if (far)
                run_tile<kTileFar>(buf.part, mpad, ly, tg, P);
            else
                run_tile<kTileNear>(buf.part, mpad, ly, tg, P);
            if (kSub && lane == 0) atomicAdd(&L.kept[far ? 0 : 1], (uint32_t)m);
        }
        while (lds_acquire(&L.done) != t) __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int u = 0; u < IPL; u++) {
            if (u >= ly.nu) break;
#pragma unroll
            for (int k = 0; k < 4; k++) L.acc[u][k][lane] += (double)P.v[u][k];
        }
        lds_release(&L.done, t + 1u);
    }
}

template <typename R, int IPL, int T, bool kSub, int MW>
__global__ __launch_bounds__(T *kWave, MW) void k_force_team(ForceLaunch f) {
    __shared__ TeamLds<R, IPL, T> L;
    if (f.st_in->invalid_radii || f.st_in->cell_overflow) return;
    const int w = uniform((int)(threadIdx.x / kWave));
    const int lane = lane_id();
    const int64_t n = f.t.n;
    // the walker's wave differs between the blocks of a CU (the grid's
    // quarters), so that the walks spread over its SIMDs
    const int walker = (int)((uint64_t)blockIdx.x * 4 / gridDim.x) % T;
    const uint32_t CH = kWave * IPL;
    unsigned long long cnt_pc = 0, cnt_far = 0, cnt_near = 0;
    for (int i = threadIdx.x; i < IPL * 4 * kWave; i += T * kWave) (&L.acc[0][0][0])[i] = 0.0;
    GroupQueue queue(f.queue, f.st_in);
    int64_t g = -1;
    uint32_t gnode = 0, gstart = 0, gn = 0, t0 = 0, tn = 0;
    auto group = [&](int64_t which) {
        gnode = (uint32_t)uniform((int)f.groups[which]);
        const uint4 ginfo = f.t.nd_info[gnode];
        gstart = (uint32_t)uniform((int)ginfo.x);
        gn = (uint32_t)uniform((int)ginfo.y);
        t0 = gstart;
        tn = gn;
        if constexpr (kSub) {
            t0 = (uint32_t)uniform((int)f.tpos[gstart]);
            tn = (uint32_t)uniform((int)f.tpos[gstart + gn]) - t0;
        }
    };
    // the next group that has targets (the walker's wave, between barriers)
    auto set_group = [&]() {
        do {
            g = queue.next();
            if (g >= 0) group(g);
        } while (kSub && g >= 0 && tn == 0);
    };
    auto set_item = [&](uint32_t at) {
        if (lane == 0) {
            L.pub = L.claim = L.done = 0u;
            L.group = g;
            L.chunk = at;
        }
    };
    if (w == walker) {
        set_group();
        set_item(0);
    }
    while (true) {
        __syncthreads();
        if (w != walker) {
            const int64_t mine = L.group;
            g = (int64_t)uniform((int)(mine >> 32)) << 32 | (uint32_t)uniform((int)mine);
            if (g >= 0) group(g);
        }
        if (g < 0) break;
        const uint32_t chunk = (uint32_t)uniform((int)L.chunk);
        const uint32_t active = tn - chunk < CH ? tn - chunk : CH;
        const Layout ly = choose_layout<IPL>(active);
        const GroupGeom G = load_group(f.t.nd_lo, f.t.nd_hi, gnode);
        if (w == walker) {
            if (lane == 0) L.kept[0] = L.kept[1] = L.fail = 0u;
            team_walk<R, IPL, T, kSub>(L, f, G, gstart, gn, f.nb.head != nullptr && chunk == 0,
                                       f.spill + (int64_t)blockIdx.x * kSpillCap, f.th2);
        }
        Targets<R, IPL> tg;
#pragma unroll
        for (int u = 0; u < IPL; u++) {
            const uint32_t off = chunk + u * ly.W + ly.il;
            const bool valid = ly.act && u < ly.nu && off < tn;
            const uint32_t k = kSub ? f.tidx[t0 + (valid ? off : 0u)]
                                    : gstart + (valid ? off : 0u);
            const double4 p = f.t.ps[k];
            const double2 rr = f.t.rr[k];
            tg.x[u] = (R)(p.x - G.c[0]);
            tg.y[u] = (R)(p.y - G.c[1]);
            tg.z[u] = (R)(p.z - G.c[2]);
            tg.rin[u] = (R)rr.x;
            tg.rout[u] = (R)rr.y;
            tg.k[u] = valid ? k : kNone;
        }
        team_consume<R, IPL, T, kSub>(L, L.tile[w], f, G, ly, tg);
        __syncthreads();
        // every tile has been added: each component's wave folds the splits
        // (in their order) and writes it
        const uint32_t n_pc = L.n_pc;
        const uint32_t n_far = kSub ? L.kept[0] : L.n_far, n_near = kSub ? L.kept[1] : L.n_near;
        const bool fail = L.fail != 0u;
#pragma unroll
        for (int u = 0; u < IPL; u++) {
            if (u >= ly.nu) break;
            const uint32_t off = chunk + u * ly.W + ly.il;
            const bool own = ly.act && ly.sl == 0 && off < tn;
            const uint32_t k = kSub ? f.tidx[t0 + (own ? off : 0u)] : gstart + (own ? off : 0u);
            if (kSub && w == walker)
                cnt_near -= (unsigned long long)__popcll(__ballot(own && f.t.ps[k].w != 0.0));
            const uint32_t o = f.t.orig[k];
            for (int c = w; c < 4; c += T) {
                double *a = L.acc[u][c];
                double v = a[lane];
                if (own)
                    for (int s2 = 1; s2 < ly.S; s2++) v += a[s2 * ly.W + ly.il];
                wave_sync();
                a[lane] = 0.0;
                if (!own || fail) continue;
                const double val = f.G * v;
                if (c < 3) {
                    f.acc[c * n + o] = val;
                    if (f.kick_vel) kick_add(f.kick_vel + c * n + o, val, f.kick_dt);
                } else {
                    f.pot[o] = val;
                    if (f.nb_bound) f.nb_bound[o] = n_near;
                    if (f.counts) {
                        f.counts[o] = (int32_t)n_pc;
                        f.counts[n + o] = (int32_t)n_far;
                        f.counts[2 * n + o] = (int32_t)n_near;
                        f.counts[3 * n + o] = (int32_t)gn;
                    }
                }
            }
        }
        if (w == walker) {
            cnt_pc += (unsigned long long)n_pc * active;
            cnt_far += (unsigned long long)n_far * active;
            cnt_near += (unsigned long long)n_near * active - (kSub ? 0u : active);
            uint32_t at = 0;
            if (chunk + CH < tn && !fail)
                at = chunk + CH;
            else
                set_group();
            wave_sync();
            set_item(at);
        }
    }
    if (w == walker && lane == 0) {
        if (cnt_pc) atomicAdd(&f.st->inter[0], cnt_pc);
        if (cnt_far) atomicAdd(&f.st->inter[1], cnt_far);
        if (cnt_near) atomicAdd(&f.st->inter[2], cnt_near);
    }
}

__global__ __launch_bounds__(kThreads) void k_target_flags(const uint8_t *target,
                                                            const uint32_t *orig, int64_t n,
                                                            uint32_t *flag, double *acc,
                                                            double *pot) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t o = orig[k];
        const bool t = target[o] != 0;
        flag[k] = t ? 1u : 0u;
        if (!t) {
            acc[o] = 0.0;
            acc[n + o] = 0.0;
            acc[2 * n + o] = 0.0;
            pot[o] = 0.0;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_target_compact(const uint32_t *flag,
                                                              const uint32_t *tpos, int64_t n,
                                                              uint32_t *tidx) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x)
        if (flag[k]) tidx[tpos[k]] = (uint32_t)k;
}

inline unsigned blocks_for(int64_t n) {
    int64_t b = (n + kThreads - 1) / kThreads;
    return (unsigned)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

int cus_of(int device) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        cus < 1)
        cus = 256;  // MI355X
    return cus;
}

template <typename K>
int resident_for(K kernel, int device) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, 0) != hipSuccess)
        per_cu = 1;
    if (per_cu < 1) per_cu = 1;
    return per_cu * cus_of(device) * kWavesPerBlock;
}

// Waves per SIMD that the teams are compiled for, and the teams a CU holds.
template <typename R>
constexpr int team_waves(int T) {
    if (T == 16) return 4;
    if (T == 8) return sizeof(R) == 4 ? 6 : 4;
    return sizeof(R) == 4 ? 5 : 3;
}

template <typename R, int IPL, int T>
void launch_team(const ForceLaunch &f, hipStream_t s) {
    constexpr int W = team_waves<R>(T);
    const dim3 grid(f.cus * (4 * W / T)), block(T * kWave);
    if (f.tidx)
        hipLaunchKernelGGL((k_force_team<R, IPL, T, true, W>), grid, block, 0, s, f);
    else
        hipLaunchKernelGGL((k_force_team<R, IPL, T, false, W>), grid, block, 0, s, f);
}

// A wave that walks alone (k_force) waits for the memory at every step of
// its walk, and a group of 64 targets runs its tiles one after the other: a
// launch takes no less than its slowest group, 0.1 to 0.5 ms, and fills the
// chip only with some ten groups per resident wave. Teams cut that time and
// pay for it with the walker's idle lanes and the hand-over of the tiles
// (4.9% more VALU instructions at a million stars). The lines lie by the
// groups to be had, about 3.4 n / group_size on clustered particles. Kernel
// times, two targets per lane, leaf 8, theta 0.5, ms:
//   n (group 64)   1k     4k     16k    64k    200k   500k   1m     2m
//   one wave       0.122  0.332  0.517  0.522  0.758  1.816  3.589  7.039
//   teams of 4     0.055  0.124  0.189  0.274  0.680  1.761  3.806  7.451
//   teams of 8     0.044  0.083  0.128  0.276  0.830  2.113
//   teams of 16    0.034  0.073  0.140  0.546
//   FP64, one wave 0.144  0.435  0.680  0.698  1.415  3.555
//   teams of 4     0.080  0.189  0.294  0.485  1.427  3.675
// The line above which one wave is better lies lower for smaller groups: they
// have fewer tiles for a team to share, and their times differ less, so that a
// launch of single waves ends together. n / group_size where the two are even at
// theta 0.5 (leaf 4 to 16, one or two targets per lane):
//   group          8      12     16     24     32     48     64     96     192
//   mixed          600    1300   1600   2300   3000   4500   9000   12000  above 7300
//   FP64           1200   1600   2000   2200   2900   3100   2800   4300   6000
// (At n / group_size of 12500, teams of 4 took 1.4 times as long at group 8,
// 1.25 times at 16; over theta 0.3 to 0.8, 0.93 to 1.4 times at 32.) From 64 on
// it goes either way, as theta and the cells' sizes have it: up to 20000, teams
// of 4 took 0.88 to 1.2 times as long at 64 and 0.81 to 1.09 times at 128. A leaf
// larger than group_size is a group as it is. With four targets per
// lane a team's waves pass their register bounds (31 to 121 VGPRs spilled) and
// none are built: teams of 4 would take what they take with two per lane (64k,
// group 64: 0.279 and 0.274 ms; one wave, four per lane, 0.484).
inline int64_t team_line(const ForceLaunch &f) {
    const int64_t group = std::max(f.group_size, f.leaf_size);
    return group * (group <= 32 ? 100 * group : std::min<int64_t>(525 * group - 13600, 20000));
}

template <typename R, int IPL>
void launch_t(const ForceLaunch &f, int resident_waves, hipStream_t s) {
    if constexpr (IPL <= 2) {
        const int64_t per = f.t.n / f.group_size;
        if (per <= 100) return launch_team<R, IPL, 16>(f, s);
        if (per <= 700) return launch_team<R, IPL, 8>(f, s);
        if (f.t.n <= team_line(f)) return launch_team<R, IPL, 4>(f, s);
    }
    const dim3 grid(resident_waves / kWavesPerBlock), block(kThreads);
    if (f.tidx)
        hipLaunchKernelGGL((k_force<R, IPL, true>), grid, block, 0, s, f);
    else
        hipLaunchKernelGGL((k_force<R, IPL, false>), grid, block, 0, s, f);
}

}  // namespace

int64_t force_spill_elems_per_wave() { return kSpillCap; }
int force_team_walkers(int device) { return 5 * cus_of(device); }

void launch_target_flags(const uint8_t *target, const TreeDev &t, uint32_t *flag, double *acc,
                         double *pot, hipStream_t s) {
    hipLaunchKernelGGL(k_target_flags, dim3(blocks_for(t.n)), dim3(kThreads), 0, s, target,
                       (const uint32_t *)t.orig, t.n, flag, acc, pot);
}

void launch_target_compact(const uint32_t *flag, const uint32_t *tpos, int64_t n, uint32_t *tidx,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_target_compact, dim3(blocks_for(n)), dim3(kThreads), 0, s, flag, tpos,
                       n, tidx);
}

int force_resident_waves(int precision, int ipl, int device) {
    if (precision == 1) {
        if (ipl == 4) return resident_for(k_force<double, 4, false>, device);
        if (ipl == 2) return resident_for(k_force<double, 2, false>, device);
        return resident_for(k_force<double, 1, false>, device);
    }
    if (ipl == 4) return resident_for(k_force<float, 4, false>, device);
    if (ipl == 2) return resident_for(k_force<float, 2, false>, device);
    return resident_for(k_force<float, 1, false>, device);
}

int force_cus(int device) { return cus_of(device); }

void launch_force(const ForceLaunch &f, int resident_waves, hipStream_t s) {
    if (f.precision == 1) {
        if (f.ipl == 4)
            launch_t<double, 4>(f, resident_waves, s);
        else if (f.ipl == 2)
            launch_t<double, 2>(f, resident_waves, s);
        else
            launch_t<double, 1>(f, resident_waves, s);
    } else {
        if (f.ipl == 4)
            launch_t<float, 4>(f, resident_waves, s);
        else if (f.ipl == 2)
            launch_t<float, 2>(f, resident_waves, s);
        else
            launch_t<float, 1>(f, resident_waves, s);
    }
}

}  // namespace petar
