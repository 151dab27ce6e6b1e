// Stable LSD radix sort of (key, u32 value) pairs with 8-bit digits.
//
// Used by the index build to order the entry segments (Sec. 4.2.1 sorts D by
// ascending start time and renumbers it), by the grid build to group the
// listings by cell, and by the trajectory merge.  Stability keeps equal keys in
// input order, which makes the renumbering deterministic.
//
//   rs_hist   the digit counts of every pass at once, one read of the keys;
//   rs_plan   exclusive sums of each digit's counts, and the digits to sort
//             by (a digit that is the same in every key is skipped);
//   rs_pass   one launch per digit: a workgroup takes the next tile of keys,
//             ranks them by digit (wave ballots, per-wave counts in LDS),
//             learns from the tiles before it where its keys go (decoupled
//             look-back: Merrill & Garland, "Single-pass Parallel Prefix Scan
//             with Decoupled Look-back", 2016; Adinets & Merrill, "Onesweep",
//             2022), orders the tile in LDS and writes each digit's keys as
//             one contiguous run.
//
// What bounds it: HBM traffic for large inputs (a pass reads and writes a key
// and a value once), launches for small ones (one per digit here).  Before, a
// pass was five launches (count, three scan steps, scatter), read the keys
// twice and wrote each key straight to its place from the lane that held it:
// 2.1-3.1 ms per pass at 171e6 pairs (now 0.9-1.0) and 40 us at 1e6 (now 22).
//
// Tiles are taken in order from a counter, so every tile before a waiting one
// is held by a workgroup that is running and publishes its counts without
// waiting for anything: each look-back ends.
#include <algorithm>

#include "radix_sort.hpp"

namespace tds {

namespace {

constexpr int kRadix = kSortRadix;
constexpr int kHistThreads = 512;

// Look-back status word of one (tile, digit): the pass it belongs to, whether
// it is the tile's own count or the sum up to and including the tile, and the
// count.  Words of an earlier pass read as "not yet published".
constexpr int kEpochShift = 56;
constexpr uint64_t kOwn = 1ull << 54, kSum = 2ull << 54, kFlags = 3ull << 54;
constexpr uint64_t kCount = (1ull << 54) - 1;

__device__ inline uint64_t lanemask_lt() {
    const uint32_t lane = __lane_id();
    return (lane == 0) ? 0ull : (~0ull >> (64 - lane));
}

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(256) void rs_clear(uint32_t* __restrict__ ctl,
                                                uint64_t* __restrict__ status, uint64_t words) {
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x, step = (uint64_t)gridDim.x * 256;
    for (uint64_t i = t; i < sizeof(SortControl) / 4; i += step) ctl[i] = 0u;
    for (uint64_t i = t; i < words; i += step) status[i] = 0ull;
}

// Digit counts of all passes.  A wave whose keys share a digit adds 64 to it
// at once (keys that come sorted, or high digits that hardly vary, would
// otherwise queue 64 atomics on one LDS address).
__global__ __launch_bounds__(kHistThreads) void rs_hist(const uint64_t* __restrict__ keys, uint64_t n,
                                                    int npass, SortControl* __restrict__ ctl) {
    __shared__ uint32_t h[8][kRadix];
    const uint32_t tid = threadIdx.x;
    for (int p = 0; p < npass; ++p)
        for (uint32_t d = tid; d < (uint32_t)kRadix; d += kHistThreads) h[p][d] = 0;
    __syncthreads();
    const PairPack pk = ctl->pack();
    const uint64_t step = (uint64_t)gridDim.x * kHistThreads;
    const uint64_t rounds = (n + step - 1) / step;
    for (uint64_t r = 0; r < rounds; ++r) {
        const uint64_t i = r * step + (uint64_t)blockIdx.x * kHistThreads + tid;
        const bool valid = i < n;
        const uint64_t key = valid ? pk.apply(keys[i]) : 0ull;
        const bool full = __ballot(valid) == ~0ull;
        for (int p = 0; p < npass; ++p) {
            const uint32_t d = (uint32_t)(key >> (8 * p)) & (kRadix - 1);
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, 0);
            const bool same = __ballot(d == d0) == ~0ull;
            if (full && same) {
                if (__lane_id() == 0) atomicAdd(&h[p][d], (uint32_t)kWave);
            } else if (valid) {
                atomicAdd(&h[p][d], 1u);
            }
        }
    }
    __syncthreads();
    for (int p = 0; p < npass; ++p)
        for (uint32_t d = tid; d < (uint32_t)kRadix; d += kHistThreads)
            if (h[p][d]) atomicAdd(&ctl->hist[p][d], h[p][d]);
}

// One workgroup of kRadix threads: exclusive sums per digit position, and the
// digit positions in use, in order (at least one, so that the values are
// written and the keys packed).
__global__ __launch_bounds__(kRadix) void rs_plan(SortControl* __restrict__ ctl, int npass,
                                                  uint32_t n) {
    __shared__ uint32_t wsum[kRadix / kWave];
    __shared__ uint32_t varies[8];
    const uint32_t t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    if (t < 8) varies[t] = 0;
    __syncthreads();
    for (int p = 0; p < npass; ++p) {
        const uint32_t v = ctl->hist[p][t];
        uint32_t x = v;
        for (uint32_t o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == kWave - 1) wsum[wv] = x;
        if (v && v != n) varies[p] = 1;
        __syncthreads();
        uint32_t before = 0;
        for (uint32_t k = 0; k < wv; ++k) before += wsum[k];
        ctl->hist[p][t] = before + x - v;
        __syncthreads();
    }
    if (t == 0) {
        uint32_t m = 0;
        for (int p = 0; p < npass; ++p)
            if (varies[p]) ctl->digit[m++] = (uint32_t)p;
        if (m == 0) {
            ctl->digit[0] = 0;
            m = 1;
        }
        ctl->npass = m;
    }
}

// One step back over kWide tiles from tile p on: adds the counts published so
// far up to the first one that is not, or that is a sum (then true: done).
template <int kWide>
__device__ __forceinline__ bool look_back(const uint64_t* status, uint32_t digit, uint32_t pass,
                                          int64_t& p, uint64_t& sum) {
    uint64_t w[kWide];
#pragma unroll
    for (int q = 0; q < kWide; ++q)
        w[q] = p >= q ? __hip_atomic_load(status + (uint64_t)(p - q) * kRadix + digit,
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                      : 0ull;
    bool more = true, done = false;
    int64_t back = 0;
#pragma unroll
    for (int q = 0; q < kWide; ++q) {
        more = more && !done && (w[q] >> kEpochShift) == (uint64_t)(pass + 1);
        if (more) {
            sum += w[q] & kCount;
            ++back;
            done = (w[q] & kFlags) == kSum;
        }
    }
    p -= back;
    return done;
}

// What pass 0 reads are the 64-bit keys as given.
template <class K, bool kFirst>
struct SortRaw {
    typedef K type;
};
template <class K>
struct SortRaw<K, true> {
    typedef uint64_t type;
};

// Pass number `pass` of the plan (a launch past the plan's end does nothing).
// Passes alternate between the two buffer pairs (k0, v0) and (k1, v1); pass 0
// reads its keys from `raw` (packed on the way) and its values from vinit or,
// without one, takes the positions.
//
// A tile is kThreads * kItems pairs, wave w holding its w-th contiguous part,
// item k of the part's lanes consecutive.  The keys and then the values go
// through one LDS buffer.  Keys past n are given digit 255: they come last in
// the last tile, whose counts no other tile reads.
template <class K, int kThreads, int kItems, bool kFirst>
__global__ __launch_bounds__(kThreads) void rs_pass(const uint64_t* __restrict__ raw,
                                                    const uint32_t* __restrict__ vinit, K* k0,
                                                    uint32_t* v0, K* k1, uint32_t* v1, uint32_t n,
                                                    uint32_t pass, SortControl* __restrict__ ctl,
                                                    uint64_t* __restrict__ status) {
    constexpr uint32_t kTile = kThreads * kItems;
    constexpr int kWaves = kThreads / kWave;
    static_assert(kThreads >= kRadix && kTile < 65536, "one thread per digit; 16-bit counts");
    __shared__ K s_buf[kTile];
    __shared__ uint16_t s_cnt[kWaves][kRadix];
    __shared__ uint32_t s_start[kRadix];  // first position of a digit in the tile
    __shared__ uint32_t s_dst[kRadix];    // its first position in the output, minus s_start
    __shared__ uint32_t s_wsum[kRadix / kWave];
    __shared__ uint32_t s_tile;
    if (pass >= ctl->npass) return;
    const uint32_t tid = threadIdx.x, lane = __lane_id(), wv = tid / kWave;
    const uint32_t dp = ctl->digit[pass];
    const int shift = 8 * (int)dp;
    const K* kin = (pass & 1) ? k1 : k0;
    const uint32_t* vin = (pass & 1) ? v1 : v0;
    K* kout = (pass & 1) ? k0 : k1;
    uint32_t* vout = (pass & 1) ? v0 : v1;
    if (tid == 0) s_tile = atomicAdd(&ctl->ticket[pass], 1u);
    for (uint32_t d = lane; d < (uint32_t)kRadix; d += kWave) s_cnt[wv][d] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    const uint64_t base = (uint64_t)tile * kTile;
    const uint64_t mine = base + (uint64_t)wv * (kWave * kItems) + lane;
    const uint32_t nvalid = (uint32_t)min((uint64_t)kTile, (uint64_t)n - base);
    K key[kItems];
    uint32_t val[kItems], rank[kItems];
    // all loads of the tile are issued before the first is used
    typename SortRaw<K, kFirst>::type in[kItems];
    if (nvalid == kTile) {
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint64_t i = mine + (uint64_t)k * kWave;
            if constexpr (kFirst) in[k] = raw[i];
            else in[k] = kin[i];
        }
    } else {
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const uint64_t i = mine + (uint64_t)k * kWave;
            in[k] = 0;
            if (i < n) {
                if constexpr (kFirst) in[k] = raw[i];
                else in[k] = kin[i];
            }
        }
    }
    if (kFirst && !vinit) {
#pragma unroll
        for (int k = 0; k < kItems; ++k) val[k] = (uint32_t)mine + (uint32_t)k * kWave;
    } else {
        const uint32_t* vsrc = kFirst ? vinit : vin;
        if (nvalid == kTile) {
#pragma unroll
            for (int k = 0; k < kItems; ++k) val[k] = vsrc[mine + (uint64_t)k * kWave];
        } else {
#pragma unroll
            for (int k = 0; k < kItems; ++k) {
                const uint64_t i = mine + (uint64_t)k * kWave;
                val[k] = i < n ? vsrc[i] : 0u;
            }
        }
    }
    {
        const PairPack pk = ctl->pack();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            if constexpr (kFirst) key[k] = (K)(pk.pairs ? pk.pack(in[k]) : in[k]);
            else key[k] = in[k];
            if (mine + (uint64_t)k * kWave >= n) key[k] = (K)~(K)0;
        }
    }
    // rank among the wave's keys of the same digit
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const uint32_t d = (uint32_t)(key[k] >> shift) & (kRadix - 1);
        uint64_t same = ~0ull;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool set = (d >> b) & 1u;
            const uint64_t m = __ballot(set);
            same &= set ? m : ~m;
        }
        const uint32_t below = (uint32_t)__popcll(same & lanemask_lt());
        const uint32_t c = s_cnt[wv][d];
        wave_sync();
        if (below == 0) s_cnt[wv][d] = (uint16_t)(c + (uint32_t)__popcll(same));
        wave_sync();
        rank[k] = c + below;
    }
    __syncthreads();
    uint32_t total = 0, before = 0;
    if (tid < (uint32_t)kRadix) {
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = s_cnt[w][tid];
            s_cnt[w][tid] = (uint16_t)total;
            total += c;
        }
        const uint64_t epoch = (uint64_t)(pass + 1) << kEpochShift;
        uint64_t* st = status + (uint64_t)tile * kRadix + tid;
        __hip_atomic_store(st, epoch | (tile ? kOwn : kSum) | total, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        // sum over the waves below (their scan of the digit totals follows)
        uint32_t x = total;
        for (uint32_t o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == kWave - 1) s_wsum[wv] = x;
        before = x - total;
        // look back over the tiles before this one: a few words at first
        // (enough once the tiles run staggered), then sixteen at a time (when
        // all tiles start together, tile t needs about sqrt(t / 8) such steps)
        uint64_t sum = 0;
        if (tile) {
            int64_t p = (int64_t)tile - 1;
            // the largest tile holds so many registers that sixteen more
            // spilled (171e6 pairs: 1.1 ms a pass, 0.9 with two and four)
            constexpr bool kFew = kItems >= 16;
            bool done = look_back<kFew ? 2 : 4>(status, tid, pass, p, sum);
            while (!done) done = look_back<kFew ? 4 : 16>(status, tid, pass, p, sum);
            __hip_atomic_store(st, epoch | kSum | (sum + total), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        s_dst[tid] = ctl->hist[dp][tid] + (uint32_t)sum;
    }
    __syncthreads();
    if (tid < (uint32_t)kRadix) {
        for (uint32_t w = 0; w < wv; ++w) before += s_wsum[w];
        s_start[tid] = before;
        s_dst[tid] -= before;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const uint32_t d = (uint32_t)(key[k] >> shift) & (kRadix - 1);
        rank[k] += s_start[d] + s_cnt[wv][d];  // position in the tile
        s_buf[rank[k]] = key[k];
    }
    __syncthreads();
    uint32_t dst[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const uint32_t p = (uint32_t)k * kThreads + tid;
        const K x = s_buf[p];
        dst[k] = s_dst[(uint32_t)(x >> shift) & (kRadix - 1)] + p;
        if (p < nvalid) kout[dst[k]] = x;
    }
    __syncthreads();
    uint32_t* s_val = reinterpret_cast<uint32_t*>(s_buf);
#pragma unroll
    for (int k = 0; k < kItems; ++k) s_val[rank[k]] = val[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const uint32_t p = (uint32_t)k * kThreads + tid;
        if (p < nvalid) vout[dst[k]] = s_val[p];
    }
}

// Exclusive scan of `len` u32 values in place, in three coalesced steps:
//   rs_scan_part  each block sums its tile of kScanTile values;
//   rs_scan_top   one block scans the tile sums (looping over them);
//   rs_scan_down  each block scans its tile again, offset by its tile's sum.
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 4;
constexpr int kScanTile = kScanThreads * kScanPer;

// Inclusive scan of one value per thread over a block of kScanThreads
// (Hillis-Steele in LDS); returns the inclusive prefix, *total the block sum.
__device__ inline uint32_t block_scan(uint32_t x, uint32_t* lds, uint32_t* total) {
    const uint32_t tid = threadIdx.x;
    lds[tid] = x;
    __syncthreads();
    for (uint32_t off = 1; off < kScanThreads; off <<= 1) {
        const uint32_t t = (tid >= off) ? lds[tid - off] : 0u;
        __syncthreads();
        lds[tid] += t;
        __syncthreads();
    }
    const uint32_t r = lds[tid];
    *total = lds[kScanThreads - 1];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kScanThreads) void rs_scan_part(const uint32_t* __restrict__ v,
                                                             uint32_t len,
                                                             uint32_t* __restrict__ part) {
    __shared__ uint32_t lds[kScanThreads];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int k = 0; k < kScanPer; ++k) {
        const uint64_t i = base + (uint64_t)k * kScanThreads + threadIdx.x;
        if (i < len) s += v[i];
    }
    uint32_t total;
    block_scan(s, lds, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void rs_scan_top(uint32_t* __restrict__ part,
                                                            uint32_t nparts) {
    __shared__ uint32_t lds[kScanThreads];
    uint32_t carry = 0;
    for (uint32_t b = 0; b < nparts; b += kScanThreads) {
        const uint32_t i = b + threadIdx.x;
        const uint32_t x = (i < nparts) ? part[i] : 0u;
        uint32_t total;
        const uint32_t inc = block_scan(x, lds, &total);
        if (i < nparts) part[i] = carry + inc - x;
        carry += total;
    }
    if (threadIdx.x == 0) part[nparts] = carry;  // the grand total
}

__global__ __launch_bounds__(kScanThreads) void rs_scan_down(uint32_t* __restrict__ v, uint32_t len,
                                                             const uint32_t* __restrict__ part) {
    __shared__ uint32_t lds[kScanThreads];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    // thread t scans kScanPer consecutive values: t's values are
    // base + t * kScanPer + [0, kScanPer)
    uint32_t x[kScanPer];
    uint32_t s = 0;
    for (int k = 0; k < kScanPer; ++k) {
        const uint64_t i = base + (uint64_t)threadIdx.x * kScanPer + k;
        x[k] = (i < len) ? v[i] : 0u;
        s += x[k];
    }
    uint32_t total;
    uint32_t run = block_scan(s, lds, &total) - s + part[blockIdx.x];
    for (int k = 0; k < kScanPer; ++k) {
        const uint64_t i = base + (uint64_t)threadIdx.x * kScanPer + k;
        if (i < len) v[i] = run;
        run += x[k];
    }
}

// Tile shapes.  A tile's number comes from one counter, and a returning
// atomic on one address takes the chip 30-48 ns, so large inputs take large
// tiles (tiles of 4,096 pairs at 171e6 pairs: 41,700 atomics, 1.26 ms a pass,
// whatever the bytes); small ones take tiles small enough to occupy the 256
// compute units.
struct TileShape {
    int threads, items;
};
constexpr TileShape kSmall{512, 2}, kMedium{512, 8}, kLarge{1024, 16}, kLargeWide{1024, 8};
constexpr uint32_t kMediumFrom = 1u << 18, kLargeFrom = 1u << 23;

TileShape shape_of(uint32_t n, bool narrow) {
    if (n < kMediumFrom) return kSmall;
    if (n < kLargeFrom) return kMedium;
    return narrow ? kLarge : kLargeWide;
}

uint32_t tiles_of(uint32_t n, bool narrow) {
    const TileShape t = shape_of(n, narrow);
    return ceil_div(n, (uint64_t)t.threads * t.items);
}

template <class K, bool kFirst>
auto pass_kernel(uint32_t n) {
    constexpr bool narrow = sizeof(K) == 4;
    constexpr TileShape L = narrow ? kLarge : kLargeWide;
    if (n < kMediumFrom) return rs_pass<K, kSmall.threads, kSmall.items, kFirst>;
    if (n < kLargeFrom) return rs_pass<K, kMedium.threads, kMedium.items, kFirst>;
    return rs_pass<K, L.threads, L.items, kFirst>;
}

template <class K>
void launch_pass(const SortJob& J, K* k0, K* k1, uint32_t p, hipStream_t s) {
    const auto kern = p == 0 ? pass_kernel<K, true>(J.n) : pass_kernel<K, false>(J.n);
    const bool narrow = sizeof(K) == 4;
    hipLaunchKernelGGL(kern, dim3(tiles_of(J.n, narrow)), dim3(shape_of(J.n, narrow).threads), 0,
                       s, J.raw, J.vinit, k0, J.v0, k1, J.v1, J.n, p, J.ctl, J.status);
}

}  // namespace

size_t sort_status_len(uint32_t n) {
    // the most tiles of any input up to n: each shape at its largest input
    uint32_t t = tiles_of(n, false);
    for (uint32_t top : {kMediumFrom - 1, kLargeFrom - 1}) t = std::max(t, tiles_of(std::min(n, top), false));
    return (size_t)kSortRadix * t;
}

int sort_clear(const SortJob& J, hipStream_t s) {
    const uint64_t words = (uint64_t)kSortRadix * tiles_of(J.n, false);  // the more of the two
    hipLaunchKernelGGL(rs_clear, dim3((uint32_t)std::min<uint64_t>((words + 255) / 256, 2048)),
                       dim3(256), 0, s, reinterpret_cast<uint32_t*>(J.ctl), J.status, words);
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

int sort_plan(const SortJob& J, int key_bits, hipStream_t s) {
    const int npass = (int)sort_npass(key_bits);
    const uint32_t blocks = std::min(ceil_div(J.n, (uint64_t)kHistThreads * 4), 1024u);
    hipLaunchKernelGGL(rs_hist, dim3(blocks), dim3(kHistThreads), 0, s, J.raw, (uint64_t)J.n, npass,
                       J.ctl);
    hipLaunchKernelGGL(rs_plan, dim3(1), dim3(kSortRadix), 0, s, J.ctl, npass, J.n);
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

int sort_passes(const SortJob& J, uint32_t npass, bool narrow, hipStream_t s) {
    for (uint32_t p = 0; p < npass; ++p) {
        if (narrow) {
            // two arrays of 32-bit keys in the space of the second 64-bit one
            uint32_t* a = reinterpret_cast<uint32_t*>(J.k1);
            launch_pass<uint32_t>(J, a + J.n, a, p, s);
        } else {
            launch_pass<uint64_t>(J, J.k0, J.k1, p, s);
        }
    }
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

int scan_u32(uint32_t* v, uint32_t len, uint32_t* part, hipStream_t s) {
    const uint32_t nparts = ceil_div(len, kScanTile);
    hipLaunchKernelGGL(rs_scan_part, dim3(nparts), dim3(kScanThreads), 0, s, v, len, part);
    hipLaunchKernelGGL(rs_scan_top, dim3(1), dim3(kScanThreads), 0, s, part, nparts);
    hipLaunchKernelGGL(rs_scan_down, dim3(nparts), dim3(kScanThreads), 0, s, v, len, part);
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

size_t scan_part_len(size_t len) { return (size_t)ceil_div(len, kScanTile) + 1; }

int exclusive_scan_u32(uint32_t* v, uint32_t len, uint32_t* total, hipStream_t stream) {
    return exclusive_scan_u32_with(v, len, total, stream, nullptr);
}

int exclusive_scan_u32_with(uint32_t* v, uint32_t len, uint32_t* total, hipStream_t stream,
                            uint32_t* scratch) {
    if (len == 0) {
        if (total) *total = 0;
        return TDS_OK;
    }
    const uint32_t nparts = ceil_div(len, kScanTile);
    uint32_t* part = scratch;
    if (!part) TDS_TRY(dmalloc(&part, (size_t)nparts + 1));
    int st = scan_u32(v, len, part, stream);
    if (st == TDS_OK && total) {
        if (hipMemcpyAsync(total, part + nparts, sizeof(uint32_t), hipMemcpyDeviceToHost, stream) !=
                hipSuccess ||
            hipStreamSynchronize(stream) != hipSuccess)
            st = TDS_E_DEVICE;
    }
    if (!total && hipStreamSynchronize(stream) != hipSuccess) st = TDS_E_DEVICE;
    if (!scratch) dfree(part);
    return st;
}

}  // namespace tds
