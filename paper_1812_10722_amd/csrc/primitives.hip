// Device primitives used by the geometry set-up: exclusive scan and a stable LSD radix sort
// of 64-bit keys carrying 32-bit values.  Both are hand-written for 64-wide wavefronts.
#include <algorithm>

#include "primitives.hpp"

namespace lspr {

namespace {

constexpr int SCAN_THREADS = 1024;

// Single-workgroup exclusive scan of n int64 counts (setup-time sizes, up to a few million).
// out[i] = sum_{k < i} in[k]; out[n] = total.  in and out may alias: each thread reads its
// SCAN_ITEMS consecutive elements of a chunk into registers and writes only those.  Per chunk,
// the thread sums are scanned in LDS, one wave's 64 by one thread, then the 16 wave sums by
// thread 0, which carries the running total from chunk to chunk (four barriers per chunk).
constexpr int SCAN_ITEMS = 8;
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_excl(const int64_t* in, int64_t* out,
                                                             int64_t n) {
    constexpr int NW = SCAN_THREADS / 64, CH = SCAN_THREADS * SCAN_ITEMS;
    __shared__ int64_t tsum[SCAN_THREADS];
    __shared__ int64_t wsum[NW];
    int64_t carry = 0;  // thread 0 only
    const int tid = threadIdx.x;
    for (int64_t base = 0; base < n; base += CH) {
        const int64_t first = base + static_cast<int64_t>(tid) * SCAN_ITEMS;
        int64_t v[SCAN_ITEMS], sum = 0;
#pragma unroll
        for (int e = 0; e < SCAN_ITEMS; ++e) {
            v[e] = first + e < n ? in[first + e] : 0;
            sum += v[e];
        }
        tsum[tid] = sum;
        __syncthreads();
        if (tid < NW) {
            int64_t a = 0;
            for (int l = 0; l < 64; ++l) {
                const int64_t t = tsum[64 * tid + l];
                tsum[64 * tid + l] = a;
                a += t;
            }
            wsum[tid] = a;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 0; w < NW; ++w) {
                const int64_t t = wsum[w];
                wsum[w] = carry;
                carry += t;
            }
        }
        __syncthreads();
        int64_t pre = wsum[tid >> 6] + tsum[tid];
#pragma unroll
        for (int e = 0; e < SCAN_ITEMS; ++e) {
            if (first + e < n) out[first + e] = pre;
            pre += v[e];
        }
        __syncthreads();
    }
    if (tid == 0) out[n] = carry;
}

constexpr int RS_THREADS = 256;               // 4 wavefronts
constexpr int RS_BINS = 256;                  // 8-bit digits
// Keys per thread per tile: 4 without a scan, 16 with one (a quarter of the counts: at 492032 keys the
// scan takes 28 us per pass instead of 106, the histogram and the scatter 28 instead of 15).
template <bool SCANNED>
constexpr int rs_rounds() { return SCANNED ? 16 : 4; }
template <bool SCANNED>
constexpr int rs_tile() { return RS_THREADS * rs_rounds<SCANNED>(); }

// Per-tile digit histogram, stored digit-major: hist[d * n_tiles + tile].
template <bool SCANNED>
__global__ void __launch_bounds__(RS_THREADS) k_rs_hist(const uint64_t* keys, int64_t n,
                                                        int shift, int64_t* hist, int n_tiles) {
    __shared__ int h[RS_BINS];
    for (int b = threadIdx.x; b < RS_BINS; b += RS_THREADS) h[b] = 0;
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * rs_tile<SCANNED>();
    for (int r = 0; r < rs_rounds<SCANNED>(); ++r) {
        const int64_t i = base + r * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & (RS_BINS - 1)], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < RS_BINS; b += RS_THREADS)
        hist[static_cast<int64_t>(b) * n_tiles + blockIdx.x] = h[b];
}

// Stable scatter.  Within a tile keys are visited round by round (key r*256 + t in round r),
// so rank order is round, then wavefront, then lane: the original order.  Lanes of a
// wavefront holding the same digit are found with one ballot per digit bit.
// SCANNED: offs holds the scanned histogram.  Otherwise offs is the histogram itself (up to
// RS_DIRECT tiles) and every block adds up its own offsets: thread b the counts of digit b over all
// tiles and over the tiles before its own, then a scan over the digits; that costs a few loads per
// thread instead of a launch of a single-workgroup scan per pass.  Tiles of 1024 keys: at 32768
// keys a pass takes 10 + 4 us in 32 blocks (scatter and histogram; 4096 keys in 8 blocks: 22 + 6.5
// us, and 5 us of the scan).
constexpr int RS_DIRECT = 256;
template <bool SCANNED>
__global__ void __launch_bounds__(RS_THREADS) k_rs_scatter(const uint64_t* keys_in,
                                                           const int32_t* vals_in,
                                                           uint64_t* keys_out,
                                                           int32_t* vals_out, int64_t n,
                                                           int shift, const int64_t* offs,
                                                           int n_tiles) {
    constexpr int WAVES = RS_THREADS / 64;
    static_assert(RS_BINS == RS_THREADS, "one thread per digit");
    __shared__ int64_t base_digit[RS_BINS];   // global start of each digit for this tile so far
    __shared__ int64_t wave_tot[WAVES];
    __shared__ int wave_cnt[WAVES][RS_BINS];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if constexpr (SCANNED) {
        base_digit[threadIdx.x] = offs[static_cast<int64_t>(threadIdx.x) * n_tiles + blockIdx.x];
    } else {
        const int64_t* h = offs + static_cast<int64_t>(threadIdx.x) * n_tiles;
        int64_t all = 0, before = 0;
#pragma unroll 8
        for (int t = 0; t < n_tiles; ++t) {
            const int64_t c = h[t];
            all += c;
            before += t < static_cast<int>(blockIdx.x) ? c : 0;
        }
        int64_t incl = all;  // inclusive scan over the digits, wave by wave
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t up = __shfl_up(incl, off, 64);
            incl += lane >= off ? up : 0;
        }
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        int64_t pre = incl - all + before;
        for (int w = 0; w < wave; ++w) pre += wave_tot[w];
        base_digit[threadIdx.x] = pre;
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * rs_tile<SCANNED>();
    for (int r = 0; r < rs_rounds<SCANNED>(); ++r) {
        for (int b = threadIdx.x; b < WAVES * RS_BINS; b += RS_THREADS)
            (&wave_cnt[0][0])[b] = 0;
        __syncthreads();
        const int64_t i = tile0 + r * RS_THREADS + threadIdx.x;
        const bool valid = i < n;
        const uint64_t key = valid ? keys_in[i] : 0;
        const int digit = static_cast<int>((key >> shift) & (RS_BINS - 1));
        uint64_t peers = __ballot(valid);
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t ones = __ballot(valid && ((digit >> bit) & 1));
            peers &= ((digit >> bit) & 1) ? ones : ~ones;
        }
        const int rank = __popcll(peers & below);
        if (valid && rank == 0) wave_cnt[wave][digit] = __popcll(peers);
        __syncthreads();
        // exclusive prefix over wavefronts for the digit of this key
        int64_t pos = 0;
        if (valid) {
            int before = 0;
            for (int w = 0; w < wave; ++w) before += wave_cnt[w][digit];
            pos = base_digit[digit] + before + rank;
        }
        __syncthreads();
        if (valid) {
            keys_out[pos] = key;
            vals_out[pos] = vals_in[i];
        }
        // advance the per-digit base by this round's totals
        for (int b = threadIdx.x; b < RS_BINS; b += RS_THREADS) {
            int tot = 0;
            for (int w = 0; w < WAVES; ++w) tot += wave_cnt[w][b];
            base_digit[b] += tot;
        }
        __syncthreads();
    }
}

// Blocks of bytes moved by one launch: blockIdx.y = block, 16 bytes per thread and step.  Latency-
// bound at set-up sizes (a copy per table cost a launch of 5-10 us each, 50 per 512-panel
// geometry); from pinned memory it streams at the link's rate.
constexpr int MOVES = 16;
struct MoveArgs {
    Move m[MOVES];
};
__global__ void __launch_bounds__(256) k_move(MoveArgs a) {
    const Move m = a.m[blockIdx.y];
    const size_t units = m.bytes / 16, step = static_cast<size_t>(gridDim.x) * 256;
    const size_t first = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    const uint4* src = static_cast<const uint4*>(m.src);
    uint4* dst = static_cast<uint4*>(m.dst);
    for (size_t u = first; u < units; u += step) dst[u] = src[u];
    const size_t rest = (m.bytes - 16 * units) / 4;  // the last, partial unit
    if (first < rest)
        reinterpret_cast<uint32_t*>(dst + units)[first] =
            reinterpret_cast<const uint32_t*>(src + units)[first];
}

}  // namespace

void move_blocks(const Move* m, size_t n, hipStream_t s) {
    for (size_t i = 0; i < n; i += MOVES) {
        MoveArgs a{};
        const size_t k = std::min<size_t>(MOVES, n - i);
        size_t most = 0;
        for (size_t q = 0; q < k; ++q) {
            a.m[q] = m[i + q];
            LSPR_REQUIRE((reinterpret_cast<uintptr_t>(a.m[q].dst) | reinterpret_cast<uintptr_t>(a.m[q].src)) % 16 == 0 &&
                             a.m[q].bytes % 4 == 0,
                         LSPR_E_INVALID, "misaligned block");
            most = std::max(most, a.m[q].bytes);
        }
        const unsigned gx = static_cast<unsigned>(std::min<size_t>(64, most / 4096 + 1));
        hipLaunchKernelGGL(k_move, dim3(gx, static_cast<unsigned>(k)), dim3(256), 0, s, a);
        LSPR_HIP(hipGetLastError());
    }
}

void scan_exclusive(const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_scan_excl, dim3(1), dim3(SCAN_THREADS), 0, s, in, out, n);
    LSPR_HIP(hipGetLastError());
}

void radix_sort_pairs(uint64_t* keys, int32_t* vals, int64_t n, int key_bits, hipStream_t s) {
    if (n <= 1) return;
    const bool scanned = n > static_cast<int64_t>(RS_DIRECT) * rs_tile<false>();
    const int tile = scanned ? rs_tile<true>() : rs_tile<false>();
    const int n_tiles = static_cast<int>((n + tile - 1) / tile);
    DevBuf<uint64_t> k2(n);
    DevBuf<int32_t> v2(n);
    DevBuf<int64_t> hist(static_cast<size_t>(RS_BINS) * n_tiles + 1);
    uint64_t* ka = keys;
    int32_t* va = vals;
    uint64_t* kb = k2.p;
    int32_t* vb = v2.p;
    const int passes = (key_bits + 7) / 8;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        if (!scanned) {
            hipLaunchKernelGGL(k_rs_hist<false>, dim3(n_tiles), dim3(RS_THREADS), 0, s, ka, n, shift,
                               hist.p, n_tiles);
            hipLaunchKernelGGL(k_rs_scatter<false>, dim3(n_tiles), dim3(RS_THREADS), 0, s, ka, va, kb,
                               vb, n, shift, hist.p, n_tiles);
        } else {
            hipLaunchKernelGGL(k_rs_hist<true>, dim3(n_tiles), dim3(RS_THREADS), 0, s, ka, n, shift,
                               hist.p, n_tiles);
            LSPR_HIP(hipGetLastError());
            scan_exclusive(hist.p, hist.p, static_cast<int64_t>(RS_BINS) * n_tiles, s);
            hipLaunchKernelGGL(k_rs_scatter<true>, dim3(n_tiles), dim3(RS_THREADS), 0, s, ka, va, kb,
                               vb, n, shift, hist.p, n_tiles);
        }
        LSPR_HIP(hipGetLastError());
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    if (ka != keys) {
        LSPR_HIP(hipMemcpyAsync(keys, ka, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
        LSPR_HIP(hipMemcpyAsync(vals, va, n * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    }
}

}  // namespace lspr
