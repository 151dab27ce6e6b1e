// Trajectory-level output: segment-level result records merged into maximal
// time intervals per (q_traj, e_traj) pair (the trajectory-level answer to
// the motivating query of Sec. 1, built on the segment records of Sec. 3.1).
//
// One-pass form (pairs of at most kHalo records, every record an interval
// with t_lo <= t_hi):
//   1. k_pair_keys: the trajectory pair of every record, the largest ids and
//      whether a record is no interval;
//   2. a stable radix sort of the record positions by pair alone, the ids
//      packed into as many bits as they need (32-bit keys where that is
//      enough and the input large);
//   3. k_merge_tiles: a workgroup takes the runs (records of one pair) that
//      start in its tile of the sorted positions, reads their times once,
//      orders each run by t_lo in LDS, finds where an interval starts (t_lo
//      past every earlier t_hi of the run) and writes its intervals one after
//      another to a scratch place of its own; k_merge_place puts the tiles'
//      intervals together.
// No step needs a number on the host before it is launched, except that a
// large input (kHostPlanFrom) waits once for the id ranges, which pays for
// itself in passes not made.
//
// General form (a pair with more records than a tile's window, or a record
// whose t_lo <= t_hi does not hold), found out on the device and run instead:
//   1. stable radix sorts of the record positions by t_lo, then by pair;
//   2. k_run_heads / scan: one run per trajectory pair;
//   3. k_merge_runs<false>: one thread per run walks its records and counts
//      the merged intervals (an interval is extended while the next record
//      starts no later than the running end); scan of the counts;
//   4. k_merge_runs<true>: the same walk writes the intervals at their offsets
//      (only those below the capacity).
#include <algorithm>
#include <mutex>

#include "radix_sort.hpp"

namespace tds {

namespace {

constexpr int kMT = 256;

// Why the one-pass form does not apply (SortControl::odd).
constexpr uint32_t kOddRecord = 1, kOddRun = 2;

__device__ inline uint64_t order_key_f64(double t) {
    // order-preserving map of a double to u64 (-0 and +0 are equal)
    uint64_t u = (t == 0.0) ? 0ull : (uint64_t)__double_as_longlong(t);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Pair keys (q_traj << 32 | e_traj), the largest ids and the records that
// are no intervals.  Reads every record once (32 bytes) and writes 8: bound by
// HBM.  The workgroups loop and add to the control block once each: with one
// workgroup per 256 records and four atomics each on one line this step took
// 30 ms of the 73 ms of a merge of 171e6 records.
__global__ __launch_bounds__(kMT) void k_pair_keys(const tds_result* __restrict__ recs, uint32_t n,
                                                   uint64_t* __restrict__ keys,
                                                   SortControl* __restrict__ ctl) {
    __shared__ uint32_t s_q[kMT], s_e[kMT], s_o[kMT];
    uint32_t mq = 0, me = 0, odd = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * kMT + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * kMT) {
        const tds_result r = recs[i];
        keys[i] = ((uint64_t)r.q_traj << 32) | r.e_traj;
        mq = max(mq, r.q_traj);
        me = max(me, r.e_traj);
        if (!(r.t_lo <= r.t_hi)) odd = kOddRecord;
    }
    s_q[threadIdx.x] = mq;
    s_e[threadIdx.x] = me;
    s_o[threadIdx.x] = odd;
    __syncthreads();
    for (uint32_t off = kMT / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            s_q[threadIdx.x] = max(s_q[threadIdx.x], s_q[threadIdx.x + off]);
            s_e[threadIdx.x] = max(s_e[threadIdx.x], s_e[threadIdx.x + off]);
            s_o[threadIdx.x] |= s_o[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicMax(&ctl->max_high, s_q[0]);
        atomicMax(&ctl->max_low, s_e[0]);
        if (s_o[0]) atomicOr(&ctl->odd, s_o[0]);
        ctl->pairs = 1;  // the same value from every workgroup
    }
}

// Tiles of the one-pass merge: kPos sorted positions, whose runs may reach
// kHalo positions past the tile's end.  kHalo is the longest run that always
// fits; a pair of trajectories of n time steps has up to n records where their
// steps begin together, up to 2 n where each has a start time of its own.  Past
// it the general form takes over for all records: 2,000 pairs of 1,000 records
// take 2.4 ms, 10.0 million records 3.5 ms in pairs of 600, 0.9 in pairs of 40.
// Tiles of 1,024 need 38 KB of LDS with 32-bit keys: four workgroups of eight
// waves per compute unit; small inputs take tiles of 256, for four times the
// workgroups.
constexpr int kTileThreads = 512;
constexpr uint32_t kHalo = 512, kPosLarge = 1024, kPosSmall = 256;
constexpr uint32_t kSmallMerge = 1u << 18;  // records below which tiles are small
constexpr uint16_t kNoRun = 0xFFFFu;

// Exclusive prefix over the workgroup of one value per thread (op: max or +).
template <class Op>
__device__ inline uint32_t block_excl(uint32_t v, uint32_t id, Op op, uint32_t* s_w,
                                      uint32_t* total) {
    const uint32_t lane = __lane_id(), wv = threadIdx.x / kWave;
    uint32_t x = v;
    for (uint32_t o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o) x = op(x, y);
    }
    if (lane == kWave - 1) s_w[wv] = x;
    const uint32_t up = __shfl_up(x, 1);
    __syncthreads();
    uint32_t before = id, all = id;
    for (uint32_t k = 0; k < (uint32_t)(kTileThreads / kWave); ++k) {
        if (k < wv) before = op(before, s_w[k]);
        all = op(all, s_w[k]);
    }
    __syncthreads();
    *total = all;
    return lane ? op(before, up) : before;
}

// Runs that start in the tile, ordered and merged; the intervals go to `tmp`
// from the position of the tile's first run on (tiles own disjoint ranges of
// positions, and a range holds at least as many records as intervals), their
// number to cnt[tile].
//
// What bounds it: the gather of the records' times (16 bytes of a 32-byte
// record, at the record's place in the input) and, for long runs, the LDS
// reads of the ordering (each record compares itself with its run).  The
// intervals take a second trip (k_merge_place) because the alternative, a
// look-back over tiles numbered by a counter, made the counter's atomics the
// bound: 48 ns for each of 167,000 tiles, 8.06 ms at 171e6 records.
//
// Once a tile has found a run past its window the form is given up: that tile
// and those that start later end at once (2,000 pairs of 1,000 records: 517 us of
// ordering for nothing before).
template <class K, uint32_t kPos>
__global__ __launch_bounds__(kTileThreads) void k_merge_tiles(
    const tds_result* __restrict__ recs, const K* __restrict__ k0, const K* __restrict__ k1,
    const uint32_t* __restrict__ v0, const uint32_t* __restrict__ v1, uint32_t n,
    SortControl* __restrict__ ctl, uint32_t* __restrict__ cnt_out, uint32_t* __restrict__ at_out,
    tds_traj_interval* __restrict__ tmp) {
    constexpr uint32_t kWindow = kPos + kHalo;
    constexpr uint32_t kPer = (kWindow + kTileThreads - 1) / kTileThreads;
    constexpr uint32_t kSlots = kPer * kTileThreads;  // positions, whole threads
    __shared__ K s_key[kWindow];
    __shared__ double s_lo[kWindow], s_hi[kWindow];
    __shared__ uint16_t s_beg[kSlots];   // first position of the run, kNoRun: not this tile's
    __shared__ uint16_t s_end[kWindow];  // of a run's first position: its end
    __shared__ uint8_t s_first[kSlots];  // an interval starts here
    __shared__ uint32_t s_w[kTileThreads / kWave];
    __shared__ uint32_t s_low;           // the tile's first run
    __shared__ uint32_t s_odd;           // the general form will run
    const uint32_t tid = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * kPos;
    const uint32_t cnt = (uint32_t)min((uint64_t)kWindow, (uint64_t)n - base);
    const K* keys = ctl->side() ? k1 : k0;
    const uint32_t* vals = ctl->side() ? v1 : v0;
    uint32_t v[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t l = tid + j * kTileThreads;
        v[j] = 0;
        if (l < cnt) {
            s_key[l] = keys[base + l];
            v[j] = vals[base + l];
        }
    }
    const K prev = base ? keys[base - 1] : (K)0;
    if (tid == 0) {
        s_low = kWindow;
        s_odd = __hip_atomic_load(&ctl->odd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (s_odd) return;
    // run starts: thread t looks at kPer consecutive positions
    {
        const uint32_t l0 = tid * kPer;
        uint32_t h[kPer], last = 0;  // position + 1 of a run start, 0: none
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
            const uint32_t l = l0 + j;
            bool head = false;
            if (l < cnt) head = l ? s_key[l] != s_key[l - 1] : (base == 0 || s_key[0] != prev);
            h[j] = head ? l + 1 : 0u;
            last = max(last, h[j]);
        }
        uint32_t all;
        const uint32_t before = block_excl(
            last, 0u, [](uint32_t a, uint32_t b) { return max(a, b); }, s_w, &all);
        uint32_t run = before;
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
            const uint32_t l = l0 + j;
            if (h[j]) {
                if (run) s_end[run - 1] = (uint16_t)l;
                else s_low = l;  // one thread: the first run start of all
                run = h[j];
            }
            // runs that start in the halo are the next tile's
            s_beg[l] = (l < cnt && run && run <= kPos) ? (uint16_t)(run - 1) : kNoRun;
            s_first[l] = 0;
        }
        if (all && all <= kPos && base + cnt < n) {  // a run past the window
            if (tid == 0) atomicOr(&ctl->odd, kOddRun);
            return;
        }
        if (tid == 0 && all) s_end[all - 1] = (uint16_t)cnt;
    }
    __syncthreads();
    double lo[kPer], hi[kPer];
    uint32_t beg[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        beg[j] = s_beg[tid + j * kTileThreads];
        lo[j] = hi[j] = 0.0;
        if (beg[j] != kNoRun) {
            const tds_result& r = recs[v[j]];
            lo[j] = r.t_lo;
            hi[j] = r.t_hi;
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
        if (beg[j] != kNoRun) s_lo[tid + j * kTileThreads] = lo[j];
    __syncthreads();
    // order every run by t_lo (records that start together stay in input order)
    uint32_t to[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t l = tid + j * kTileThreads;
        to[j] = l;
        if (beg[j] == kNoRun) continue;
        const uint32_t e = s_end[beg[j]];
        uint32_t r = beg[j];
#pragma unroll 4
        for (uint32_t m = beg[j]; m < l; ++m) r += s_lo[m] <= lo[j] ? 1u : 0u;
#pragma unroll 4
        for (uint32_t m = l + 1; m < e; ++m) r += s_lo[m] < lo[j] ? 1u : 0u;
        to[j] = r;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
        if (beg[j] != kNoRun) {
            s_lo[to[j]] = lo[j];
            s_hi[to[j]] = hi[j];
        }
    __syncthreads();
    // a record starts an interval if it starts past all earlier ends of its run
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        if (beg[j] == kNoRun) continue;
        double most = -INFINITY;
#pragma unroll 4
        for (uint32_t m = beg[j]; m < to[j]; ++m) most = fmax(most, s_hi[m]);
        s_first[to[j]] = (to[j] == beg[j] || lo[j] > most) ? 1 : 0;
    }
    __syncthreads();
    const uint32_t l0 = tid * kPer;
    uint32_t c = 0, all;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) c += s_first[l0 + j];
    uint32_t at = block_excl(c, 0u, [](uint32_t a, uint32_t b) { return a + b; }, s_w, &all);
    const uint32_t low = s_low < kPos ? s_low : 0u;
    if (tid == 0) {
        cnt_out[blockIdx.x] = all;
        at_out[blockIdx.x] = (uint32_t)(base + low);
    }
    const PairPack pk = ctl->pack();
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t l = l0 + j;
        if (!s_first[l]) continue;
        const uint32_t e = s_end[s_beg[l]];
        double end = s_hi[l];
        for (uint32_t m = l + 1; m < e && !s_first[m]; ++m)
            if (s_hi[m] > end) end = s_hi[m];
        tds_traj_interval o;
        o.q_traj = pk.high((uint64_t)s_key[l]);
        o.e_traj = pk.low((uint64_t)s_key[l]);
        o.t_lo = s_lo[l];
        o.t_hi = end;
        tmp[base + low + at] = o;
        ++at;
    }
}

// The tiles' intervals one after another in `out` (those below the capacity).
// pre: exclusive sums of the tiles' counts with the total at [tiles], or, for
// inputs of few tiles (kSum), the counts themselves, which each workgroup adds
// up to its tile.  One workgroup per tile; bound by HBM (24 bytes in and out
// per interval, in 8-byte words next to each other).  Nothing is written where
// the general form takes over: it may find fewer intervals.
template <bool kSum>
__global__ __launch_bounds__(256) void k_merge_place(const uint32_t* __restrict__ pre,
                                                     const uint32_t* __restrict__ from,
                                                     uint32_t tiles,
                                                     const uint64_t* __restrict__ tmp,
                                                     uint64_t* __restrict__ out, uint64_t capacity,
                                                     SortControl* __restrict__ ctl) {
    if (ctl->odd) return;
    const uint32_t t = blockIdx.x;
    uint32_t first, n;
    if (kSum) {
        __shared__ uint32_t s_w[256 / kWave];
        uint32_t x = 0;
        for (uint32_t i = threadIdx.x; i < t; i += 256) x += pre[i];
        for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_xor(x, o);
        if (__lane_id() == 0) s_w[threadIdx.x / kWave] = x;
        __syncthreads();
        first = s_w[0] + s_w[1] + s_w[2] + s_w[3];
        n = pre[t];
    } else {
        first = pre[t];
        n = pre[t + 1] - first;
    }
    if (t == tiles - 1 && threadIdx.x == 0) ctl->total = first + n;
    if (first >= capacity) return;
    const uint32_t words = 3 * (uint32_t)min((uint64_t)n, capacity - first);
    const uint64_t src = 3 * (uint64_t)from[t], dst = 3 * (uint64_t)first;
    for (uint32_t i = threadIdx.x; i < words; i += 256) out[dst + i] = tmp[src + i];
}

// ------------------------------------------------------------ general form

__global__ __launch_bounds__(kMT) void k_keys_tlo(const tds_result* __restrict__ recs, uint32_t n,
                                                  uint64_t* __restrict__ keys) {
    const uint32_t i = blockIdx.x * kMT + threadIdx.x;
    if (i < n) keys[i] = order_key_f64(recs[i].t_lo);
}

// The first sort's values to v, and the pair keys in that order (which sort
// side holds it follows from the control block).
__global__ __launch_bounds__(kMT) void k_keys_pair(const tds_result* __restrict__ recs, uint32_t n,
                                                   const uint32_t* __restrict__ v0,
                                                   const uint32_t* __restrict__ v1,
                                                   const SortControl* __restrict__ ctl,
                                                   uint32_t* __restrict__ v,
                                                   uint64_t* __restrict__ keys) {
    const uint32_t i = blockIdx.x * kMT + threadIdx.x;
    if (i >= n) return;
    const uint32_t x = ctl->side() ? v1[i] : v0[i];
    const tds_result r = recs[x];
    v[i] = x;
    keys[i] = ((uint64_t)r.q_traj << 32) | r.e_traj;
}

// head[i] = 1 where a new trajectory pair starts in sorted order.
__global__ __launch_bounds__(kMT) void k_run_heads(const uint64_t* __restrict__ k0,
                                                   const uint64_t* __restrict__ k1,
                                                   const SortControl* __restrict__ ctl, uint32_t n,
                                                   uint32_t* __restrict__ head) {
    const uint64_t* keys = ctl->side() ? k1 : k0;
    const uint32_t i = blockIdx.x * kMT + threadIdx.x;
    if (i >= n) return;
    head[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1u : 0u;
}

// run_start[run index] = first sorted position of the run (from the
// exclusive scan of the heads and the heads themselves).
__global__ __launch_bounds__(kMT) void k_run_starts(const uint64_t* __restrict__ k0,
                                                    const uint64_t* __restrict__ k1,
                                                    const SortControl* __restrict__ ctl, uint32_t n,
                                                    const uint32_t* __restrict__ run_of,
                                                    uint32_t* __restrict__ run_start,
                                                    uint32_t n_runs) {
    const uint64_t* keys = ctl->side() ? k1 : k0;
    const uint32_t i = blockIdx.x * kMT + threadIdx.x;
    if (i >= n) return;
    if (i == 0 || keys[i] != keys[i - 1]) run_start[run_of[i]] = i;
    if (i == 0) run_start[n_runs] = n;
}

// One thread per run: the merged intervals of one trajectory pair, counted
// (kWrite false: cnt[r]) or written from offset cnt[r] (kWrite true).
//
// Bound by the latency of a run's records, which lie anywhere in the input: the
// loads of kAhead records are issued together (2,000 runs of 1,000 records, one
// at a time: 712 us to count and 1,125 to write).
constexpr uint32_t kAhead = 8;
template <bool kWrite>
__global__ __launch_bounds__(kMT) void k_merge_runs(const tds_result* __restrict__ recs,
                                                    const uint32_t* __restrict__ v0,
                                                    const uint32_t* __restrict__ v1,
                                                    const SortControl* __restrict__ ctl,
                                                    const uint32_t* __restrict__ run_start,
                                                    uint32_t n_runs, uint32_t* __restrict__ cnt,
                                                    tds_traj_interval* __restrict__ out,
                                                    uint64_t capacity) {
    const uint32_t r = blockIdx.x * kMT + threadIdx.x;
    if (r >= n_runs) return;
    const uint32_t* order = ctl->side() ? v1 : v0;
    const uint32_t b = run_start[r], e = run_start[r + 1];
    uint64_t pos = kWrite ? cnt[r] : 0u;
    uint32_t c = 0;
    const tds_result first = recs[order[b]];
    double lo = first.t_lo, hi = first.t_hi;
    const auto close = [&] {  // the current interval is complete
        if (kWrite && pos < capacity) {
            tds_traj_interval o;
            o.q_traj = first.q_traj;
            o.e_traj = first.e_traj;
            o.t_lo = lo;
            o.t_hi = hi;
            out[pos] = o;
        }
        ++pos;
        ++c;
    };
    for (uint32_t i = b + 1; i < e; i += min(kAhead, e - i)) {
        double nlo[kAhead], nhi[kAhead];
        uint32_t at[kAhead];
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) at[k] = order[k < e - i ? i + k : i];
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) {
            nlo[k] = recs[at[k]].t_lo;
            nhi[k] = recs[at[k]].t_hi;
        }
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) {
            if (k >= e - i) continue;
            if (nlo[k] > hi) {  // a gap
                close();
                lo = nlo[k];
                hi = nhi[k];
            } else if (nhi[k] > hi) {
                hi = nhi[k];
            }
        }
    }
    close();
    if (!kWrite) cnt[r] = c;
}

uint32_t merge_tiles(uint32_t n) { return ceil_div(n, n < kSmallMerge ? kPosSmall : kPosLarge); }

// Tiles up to which k_merge_place adds up the counts itself.
constexpr uint32_t kSumTiles = 1024;

// Device scratch of the merge, per device, grown on demand and kept until the
// process ends (the merge is called repeatedly on result sets of similar
// size; allocating and freeing per call cost more than the kernels).
struct MergeScratch {
    std::mutex mu;
    size_t cap = 0, rec_cap = 0, out_cap = 0, run_cap = 0;  // records each part holds
    tds_result* recs = nullptr;          // host input
    tds_traj_interval* stage = nullptr;  // host output
    tds_traj_interval* tmp = nullptr;    // the tiles' intervals, before they are put together
    uint64_t *k1 = nullptr, *k2 = nullptr, *status = nullptr;
    uint32_t *v1 = nullptr, *v2 = nullptr;
    uint32_t *tcnt = nullptr, *tfrom = nullptr, *tpart = nullptr;  // per tile
    // general form
    uint32_t *vfirst = nullptr, *runs = nullptr, *run_start = nullptr, *cnt = nullptr,
             *part = nullptr;
    SortControl* ctl = nullptr;
    SortControl* ctl_host = nullptr;  // pinned; the fields before the counts

    template <class... P>
    static void drop(size_t& c, P&... p) {
        (dfree(p), ...);
        ((p = nullptr), ...);
        c = 0;
    }

    int reserve(size_t n) {
        if (!ctl) TDS_TRY(dmalloc(&ctl, 1));
        if (!ctl_host) {
            if (hipHostMalloc(reinterpret_cast<void**>(&ctl_host), sizeof(SortControl),
                              hipHostMallocDefault) != hipSuccess) {
                (void)hipGetLastError();
                ctl_host = nullptr;
                return TDS_E_NOMEM;
            }
        }
        if (n <= cap) return TDS_OK;
        drop(cap, k1, k2, status, v1, v2, tmp, tcnt, tfrom, tpart);
        const size_t c = std::max<size_t>(n, 1024);
        int st = dmalloc(&k1, c);
        if (st == TDS_OK) st = dmalloc(&k2, c);
        if (st == TDS_OK) st = dmalloc(&v1, c);
        if (st == TDS_OK) st = dmalloc(&v2, c);
        if (st == TDS_OK) st = dmalloc(&status, sort_status_len((uint32_t)c));
        if (st == TDS_OK) st = dmalloc(&tmp, c);
        // tiles of either size
        const size_t t = std::max<size_t>(merge_tiles((uint32_t)c),
                                          merge_tiles((uint32_t)std::min<size_t>(c, kSmallMerge - 1)));
        if (st == TDS_OK) st = dmalloc(&tcnt, t + 1);
        if (st == TDS_OK) st = dmalloc(&tfrom, t);
        if (st == TDS_OK) st = dmalloc(&tpart, scan_part_len(t + 1));
        if (st != TDS_OK) {
            drop(cap, k1, k2, status, v1, v2, tmp, tcnt, tfrom, tpart);
            return st;
        }
        cap = c;
        return TDS_OK;
    }

    int reserve_recs(size_t n) {
        if (n <= rec_cap) return TDS_OK;
        drop(rec_cap, recs);
        TDS_TRY(dmalloc(&recs, n));
        rec_cap = n;
        return TDS_OK;
    }

    int reserve_out(size_t n) {
        if (n <= out_cap) return TDS_OK;
        drop(out_cap, stage);
        TDS_TRY(dmalloc(&stage, n));
        out_cap = n;
        return TDS_OK;
    }

    int reserve_runs(size_t n) {
        if (n <= run_cap) return TDS_OK;
        drop(run_cap, vfirst, runs, run_start, cnt, part);
        int st = dmalloc(&vfirst, n);
        if (st == TDS_OK) st = dmalloc(&runs, n);
        if (st == TDS_OK) st = dmalloc(&run_start, n + 1);
        if (st == TDS_OK) st = dmalloc(&cnt, n);
        if (st == TDS_OK) st = dmalloc(&part, scan_part_len(n));
        if (st != TDS_OK) {
            drop(run_cap, vfirst, runs, run_start, cnt, part);
            return st;
        }
        run_cap = n;
        return TDS_OK;
    }

    // the control block's fields before the digit counts, after the stream's work
    int read_ctl(hipStream_t s) {
        TDS_HIP(hipMemcpyAsync(ctl_host, ctl, offsetof(SortControl, hist), hipMemcpyDeviceToHost,
                               s));
        TDS_HIP(hipStreamSynchronize(s));
        return TDS_OK;
    }
};

// Waits for the stream at a merge's end unless it has (`idle`): parts of the
// scratch are reserved after work was queued on it, and when that fails the next
// merge, perhaps on another stream, must not find that work running.
struct MergeWait {
    hipStream_t s;
    bool idle = false;
    ~MergeWait() {
        if (!idle) (void)hipStreamSynchronize(s);
    }
};

constexpr int kMaxDevices = 64;
MergeScratch g_scratch[kMaxDevices];

// Records from which the host waits for the id ranges before the sort: then it
// launches the passes that they need instead of all eight (a launch that has
// nothing to do costs about 3 us; the wait about 40), and 32-bit keys are a
// third less traffic per pass.
constexpr uint32_t kHostPlanFrom = 1u << 20;

// The one-pass form on the sorted positions.
int merge_one_pass(MergeScratch& M, const tds_result* R, uint32_t nn, bool narrow,
                   tds_traj_interval* dst, uint64_t capacity, hipStream_t s) {
    const uint32_t tiles = merge_tiles(nn);
    const auto go = [&](auto kern, const auto* k0, const auto* k1) {
        hipLaunchKernelGGL(kern, dim3(tiles), dim3(kTileThreads), 0, s, R, k0, k1, M.v1, M.v2, nn,
                           M.ctl, M.tcnt, M.tfrom, M.tmp);
    };
    const uint32_t* a = reinterpret_cast<const uint32_t*>(M.k2);
    const uint64_t *w0 = M.k1, *w1 = M.k2;
    if (narrow) go(k_merge_tiles<uint32_t, kPosLarge>, a + nn, a);
    else if (nn < kSmallMerge) go(k_merge_tiles<uint64_t, kPosSmall>, w0, w1);
    else go(k_merge_tiles<uint64_t, kPosLarge>, w0, w1);
    const uint64_t* src = reinterpret_cast<const uint64_t*>(M.tmp);
    uint64_t* out = reinterpret_cast<uint64_t*>(dst);
    if (tiles <= kSumTiles) {
        hipLaunchKernelGGL(k_merge_place<true>, dim3(tiles), dim3(256), 0, s, M.tcnt, M.tfrom,
                           tiles, src, out, capacity, M.ctl);
    } else {
        // one entry more than tiles, so that the total ends up after the sums
        TDS_TRY(scan_u32(M.tcnt, tiles + 1, M.tpart, s));
        hipLaunchKernelGGL(k_merge_place<false>, dim3(tiles), dim3(256), 0, s, M.tcnt, M.tfrom,
                           tiles, src, out, capacity, M.ctl);
    }
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

// The general form; the records are on the device.  Leaves the first `keep` =
// min(total, capacity) intervals in dst.
int merge_general(MergeScratch& M, const tds_result* R, uint32_t nn, SortJob J,
                  tds_traj_interval* dst, uint64_t capacity, uint32_t* total, hipStream_t s) {
    TDS_TRY(M.reserve_runs(nn));
    const uint32_t nb = ceil_div(nn, kMT);
    TDS_TRY(sort_clear(J, s));
    hipLaunchKernelGGL(k_keys_tlo, dim3(nb), dim3(kMT), 0, s, R, nn, M.k1);
    TDS_TRY(sort_plan(J, 64, s));
    TDS_TRY(sort_passes(J, 8, false, s));
    hipLaunchKernelGGL(k_keys_pair, dim3(nb), dim3(kMT), 0, s, R, nn, M.v1, M.v2, M.ctl, M.vfirst,
                       M.k1);
    J.vinit = M.vfirst;
    TDS_TRY(sort_clear(J, s));
    TDS_TRY(sort_plan(J, 64, s));
    TDS_TRY(sort_passes(J, 8, false, s));
    // runs of equal pairs
    hipLaunchKernelGGL(k_run_heads, dim3(nb), dim3(kMT), 0, s, M.k1, M.k2, M.ctl, nn, M.runs);
    TDS_HIP(hipGetLastError());
    uint32_t n_runs = 0;
    TDS_TRY(exclusive_scan_u32_with(M.runs, nn, &n_runs, s, M.part));
    hipLaunchKernelGGL(k_run_starts, dim3(nb), dim3(kMT), 0, s, M.k1, M.k2, M.ctl, nn, M.runs,
                       M.run_start, n_runs);
    const uint32_t rb = ceil_div(n_runs, kMT);
    hipLaunchKernelGGL(k_merge_runs<false>, dim3(rb), dim3(kMT), 0, s, R, M.v1, M.v2, M.ctl,
                       M.run_start, n_runs, M.cnt, nullptr, 0ull);
    TDS_HIP(hipGetLastError());
    TDS_TRY(exclusive_scan_u32_with(M.cnt, n_runs, total, s, M.part));
    const uint64_t keep = std::min<uint64_t>(*total, capacity);
    if (keep) {
        hipLaunchKernelGGL(k_merge_runs<true>, dim3(rb), dim3(kMT), 0, s, R, M.v1, M.v2, M.ctl,
                           M.run_start, n_runs, M.cnt, dst, keep);
        TDS_HIP(hipGetLastError());
    }
    return TDS_OK;
}

}  // namespace

int merge_impl(const tds_result* recs, uint64_t n, bool recs_dev, tds_traj_interval* out,
               uint64_t capacity, bool out_dev, uint64_t* n_out, hipStream_t s) {
    if (!n_out) return TDS_E_INVALID;
    *n_out = 0;
    if (n == 0) return TDS_OK;
    if (!recs || (capacity && !out) || n >= 0xFFFFFFFFull) return TDS_E_INVALID;
    int dev = 0;
    TDS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return TDS_E_DEVICE;
    MergeScratch& M = g_scratch[dev];
    // one merge at a time per device: every call waits for its own work
    // before it returns, so the next call finds the scratch free
    std::lock_guard<std::mutex> lock(M.mu);
    TDS_TRY(M.reserve(n));
    MergeWait wait{s};
    const uint32_t nn = (uint32_t)n;
    const tds_result* R = recs;
    if (!recs_dev) {
        TDS_TRY(M.reserve_recs(n));
        TDS_HIP(hipMemcpyAsync(M.recs, recs, n * sizeof(tds_result), hipMemcpyHostToDevice, s));
        R = M.recs;
    }
    // at most one interval per record, so a staging buffer of n fits
    tds_traj_interval* dst = out;
    if (!out_dev && capacity) {
        TDS_TRY(M.reserve_out(std::min<uint64_t>(n, capacity)));
        dst = M.stage;
    }
    const uint64_t cap = std::min<uint64_t>(n, capacity);
    SortJob J{nn, M.k1, nullptr, M.k1, M.k2, M.v1, M.v2, M.ctl, M.status};
    TDS_TRY(sort_clear(J, s));
    hipLaunchKernelGGL(k_pair_keys, dim3(std::min(ceil_div(nn, kMT), 2048u)), dim3(kMT), 0, s, R,
                       nn, M.k1, M.ctl);
    TDS_HIP(hipGetLastError());
    int bits = 64;
    bool narrow = false, one_pass = true;
    if (nn >= kHostPlanFrom) {
        TDS_TRY(M.read_ctl(s));
        bits = (int)(bits_of(M.ctl_host->max_high) + bits_of(M.ctl_host->max_low));
        narrow = bits <= 32;
        one_pass = !M.ctl_host->odd;
    }
    if (one_pass) {
        TDS_TRY(sort_plan(J, bits, s));
        TDS_TRY(sort_passes(J, sort_npass(bits), narrow, s));
        TDS_TRY(merge_one_pass(M, R, nn, narrow, dst, cap, s));
        TDS_TRY(M.read_ctl(s));
        one_pass = !M.ctl_host->odd;
        if (one_pass) *n_out = M.ctl_host->total;
    }
    if (!one_pass) {
        uint32_t total = 0;
        TDS_TRY(merge_general(M, R, nn, J, dst, cap, &total, s));
        *n_out = total;
    }
    const uint64_t keep = std::min<uint64_t>(*n_out, capacity);
    if (keep && !out_dev)
        TDS_HIP(hipMemcpyAsync(out, M.stage, keep * sizeof(tds_traj_interval),
                               hipMemcpyDeviceToHost, s));
    if (keep && (!out_dev || !one_pass)) TDS_HIP(hipStreamSynchronize(s));
    wait.idle = true;
    return *n_out > capacity ? TDS_E_OVERFLOW : TDS_OK;
}

}  // namespace tds
