// Exclusive prefix sums and fill kernels. Deterministic: integer sums in a
// fixed order.
//
// A launch costs 5 to 10 us on its own, more than a small scan's work, so the
// scan takes as few as its size allows: one block (up to kOneBlockTiles tiles
// in turn); block totals, then a scan in which every block adds up the totals
// before it (up to kSelfTotals, 10 KB a block at ten million counts); above
// that, a third launch scans the totals between the two.
#include "launch.h"

namespace petar {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kOneThreads = 1024;
constexpr int kOneBlockTiles = 4;   // of 4096 counts
constexpr int64_t kSelfTotals = 4096;

template <int Threads = kScanThreads>
__device__ int64_t block_excl_scan(int64_t v, int64_t *total) {
    __shared__ int64_t wsum[Threads / kWave];
    int64_t incl = wave_incl_scan(v);
    int w = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int64_t off = 0, tot = 0;
    for (int k = 0; k < Threads / kWave; k++) {
        if (k < w) off += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    *total = tot;
    return off + incl - v;
}

// What a scan makes of its counts: the counts themselves, or (Classes) flags
// 0, 1 and 2 of which the ones and the twos are counted side by side, in the
// halves of a word: every flagged element gets its position in its class,
// out[n] is the number of both and *second that of the twos.
struct Plain {
    __device__ static int64_t value(uint32_t f) { return (int64_t)f; }
    __device__ static int64_t place(int64_t, int64_t before) { return before; }
    __device__ static int64_t total(int64_t t, int64_t *) { return t; }
};
struct Classes {
    __device__ static int64_t value(uint32_t f) {
        return f == 2u ? (int64_t)1 << 32 : (int64_t)f;
    }
    __device__ static int64_t place(int64_t v, int64_t before) {
        return v >> 32 ? before >> 32 : before & 0xffffffffll;
    }
    __device__ static int64_t total(int64_t t, int64_t *second) {
        *second = t >> 32;
        return (t >> 32) + (t & 0xffffffffll);
    }
};

template <typename In, typename Map>
__global__ __launch_bounds__(kScanThreads) void k_block_totals(const In *in, int64_t n,
                                                               int64_t *bsum) {
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t v = 0;
    for (int k = 0; k < kScanItems; k++) {
        int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
        if (i < n) v += Map::value(in[i]);
    }
    int64_t tot;
    block_excl_scan(v, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Exclusive scan of nb block totals by one block, in chunks of kScanThreads.
__global__ __launch_bounds__(kScanThreads) void k_scan_totals(int64_t *bsum, int64_t nb) {
    int64_t carry = 0;
    for (int64_t c = 0; c < nb; c += kScanThreads) {
        int64_t i = c + threadIdx.x;
        int64_t v = i < nb ? bsum[i] : 0;
        int64_t tot;
        int64_t ex = block_excl_scan(v, &tot);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) bsum[nb] = carry;
}

// Block-local scan plus the sum of the earlier blocks: bsum holds the
// totals, added up here (kSelf), or already their prefix sums. kClear: the
// counts are set to 0 once read.
template <typename In, typename Out, typename Map, bool kSelf, bool kClear>
__global__ __launch_bounds__(kScanThreads) void k_block_scan(In *in, Out *out, int64_t n,
                                                             const int64_t *bsum, int64_t nb,
                                                             int64_t *second,
                                                             const int32_t *skip) {
    if (skip && *skip) return;
    int64_t before = 0;
    if constexpr (kSelf) {
        int64_t part = 0;
        for (int64_t k = threadIdx.x; k < (int64_t)blockIdx.x; k += kScanThreads) part += bsum[k];
        block_excl_scan(part, &before);
    } else {
        before = bsum[blockIdx.x];
    }
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int64_t vals[kScanItems];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        int64_t i = base + k;
        vals[k] = i < n ? Map::value(in[i]) : 0;
        s += vals[k];
    }
    if constexpr (kClear) {
#pragma unroll
        for (int k = 0; k < kScanItems; k++)
            if (base + k < n) in[base + k] = 0;
    }
    int64_t tot;
    int64_t off = block_excl_scan(s, &tot) + before;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        int64_t i = base + k;
        if (i < n) out[i] = (Out)Map::place(vals[k], off);
        off += vals[k];
    }
    if (blockIdx.x == nb - 1 && threadIdx.x == 0) out[n] = (Out)Map::total(before + tot, second);
}

// The whole scan by one block, kOneThreads * Items counts at a time.
template <typename In, typename Out, typename Map, bool kClear>
__global__ __launch_bounds__(kOneThreads) void k_scan_one(In *in, Out *out, int64_t n,
                                                          int64_t *second, const int32_t *skip) {
    constexpr int Items = 4;
    if (skip && *skip) return;
    int64_t carry = 0;
    for (int64_t c = 0; c < n; c += (int64_t)kOneThreads * Items) {
        const int64_t base = c + (int64_t)threadIdx.x * Items;
        int64_t vals[Items], s = 0;
#pragma unroll
        for (int k = 0; k < Items; k++) {
            vals[k] = base + k < n ? Map::value(in[base + k]) : 0;
            s += vals[k];
        }
        int64_t tot;
        int64_t off = carry + block_excl_scan<kOneThreads>(s, &tot);
#pragma unroll
        for (int k = 0; k < Items; k++) {
            if (base + k < n) {
                out[base + k] = (Out)Map::place(vals[k], off);
                if constexpr (kClear) in[base + k] = 0;
            }
            off += vals[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) out[n] = (Out)Map::total(carry, second);
}

template <typename T>
__global__ void k_fill(T *p, T v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Several buffers set to 0 in one launch (a row of blocks each).
struct FillList {
    uint32_t *p[kFillPieces];
    int64_t words[kFillPieces];
    int n;
};
__global__ void k_fill_words(FillList l) {
    uint32_t *p = l.p[blockIdx.y];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < l.words[blockIdx.y];
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

__global__ void k_words_out(const int64_t *words, int n, int64_t *host) {
    if ((int)threadIdx.x < n) host[threadIdx.x] = words[threadIdx.x];
}

template <typename In, typename Out, typename Map, bool kClear>
void scan_impl(In *in, Out *out, int64_t n, int64_t *ws, hipStream_t s,
               int64_t *second = nullptr, const int32_t *skip = nullptr) {
    int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb < 1) nb = 1;
    if (nb <= kOneBlockTiles) {
        hipLaunchKernelGGL((k_scan_one<In, Out, Map, kClear>), dim3(1), dim3(kOneThreads), 0, s,
                           in, out, n, second, skip);
        return;
    }
    const dim3 g((unsigned)nb), b(kScanThreads);
    hipLaunchKernelGGL((k_block_totals<In, Map>), g, b, 0, s, (const In *)in, n, ws);
    if (nb <= kSelfTotals) {
        hipLaunchKernelGGL((k_block_scan<In, Out, Map, true, kClear>), g, b, 0, s, in, out, n,
                           (const int64_t *)ws, nb, second, skip);
        return;
    }
    hipLaunchKernelGGL(k_scan_totals, dim3(1), b, 0, s, ws, nb);
    hipLaunchKernelGGL((k_block_scan<In, Out, Map, false, kClear>), g, b, 0, s, in, out, n,
                       (const int64_t *)ws, nb, second, skip);
}

template <typename T>
void fill_impl(T *p, T v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
}

}  // namespace

int64_t scan_ws_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 2; }

void scan_u32_to_i64(const uint32_t *in, int64_t *out, int64_t n, int64_t *ws, hipStream_t s,
                     const int32_t *skip) {
    scan_impl<uint32_t, int64_t, Plain, false>(const_cast<uint32_t *>(in), out, n, ws, s, nullptr,
                                               skip);
}
void scan_u32_to_i64_clear(uint32_t *in, int64_t *out, int64_t n, int64_t *ws, hipStream_t s) {
    scan_impl<uint32_t, int64_t, Plain, true>(in, out, n, ws, s);
}
void scan_u32_to_u32(const uint32_t *in, uint32_t *out, int64_t n, int64_t *ws, hipStream_t s) {
    scan_impl<uint32_t, uint32_t, Plain, false>(const_cast<uint32_t *>(in), out, n, ws, s);
}
void scan_classes(const uint32_t *flag, uint32_t *out, int64_t n, int64_t *second, int64_t *ws,
                  hipStream_t s) {
    scan_impl<uint32_t, uint32_t, Classes, false>(const_cast<uint32_t *>(flag), out, n, ws, s,
                                                  second);
}
void fill_words(std::initializer_list<FillWords> pieces, hipStream_t s) {
    FillList l{};
    unsigned most = 1;
    for (const FillWords &p : pieces) {
        l.p[l.n] = p.p;
        l.words[l.n++] = p.words;
        const unsigned blocks = (unsigned)((p.words + 255) / 256);
        most = blocks > most ? blocks : most;
    }
    hipLaunchKernelGGL(k_fill_words, dim3(most > 256 ? 256 : most, (unsigned)l.n), dim3(256), 0, s,
                       l);
}
void fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) { fill_impl(p, v, n, s); }
void fill_i64(int64_t *p, int64_t v, int64_t n, hipStream_t s) { fill_impl(p, v, n, s); }

void words_out(const int64_t *words, int n, int64_t *host, hipStream_t s) {
    hipLaunchKernelGGL(k_words_out, dim3(1), dim3(kWave), 0, s, words, n, host);
}

}  // namespace petar
