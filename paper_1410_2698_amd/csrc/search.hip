// Distance threshold search on the GPU (Sec. 3.1 problem, Sec. 4.2.2 search).
//
// Per search, on one stream:
//   k_zero       clear the header, bucket counters and request counters;
//   k_qprep      one thread per query segment: validate, velocity, clip to the
//                window, candidate range [lo, hi) by bisection of the bin
//                tables (the schedule S of Sec. 4.2.2, computed on the GPU),
//                FP32 filter sphere, bucket key = (first bin, bin span); its
//                filter record and its FP64 data, in query order;
//   k_bucket_scan  one block: bucket offsets, 64-segment groups per bucket,
//                the size of the candidate chunks and the work-item table;
//   k_scatter    the numbers of the query segments by bucket, and the
//                work-item table (item -> bucket);
//   k_distance   persistent waves take work items (64 query segments of one
//                bucket x one chunk of their common candidate range).  FP32
//                form: the lanes hold the chunk's candidates (coalesced loads)
//                and the boxes of its 64-entry blocks; each
//                block's box is tested against every query of the group (one
//                lane per query) and only the surviving queries are tested
//                against the block's candidates.  FP64 plain form: one query
//                segment per lane, candidates streamed through wave-uniform
//                scalar loads.  Pairs that pass are queued in LDS and
//                evaluated 64 at a time by the canonical FP64 code; results
//                of one request go to positions that the wave reserved, those
//                of several through a stage per wave;
//   k_fill       after one request: the results' positions made dense, and the
//                counters folded (k_stats_fold alone after several).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>

#include <hip/hip_ext.h>

#include "canon.hpp"
#include "schedule.hpp"
#include "tds_internal.hpp"

namespace tds {

namespace {

constexpr uint32_t kInactive = 0xFFFFFFFFu;

// The bucket slot counters are split into parts: about 1,500 returning
// atomics on one address serialize for ≈ 25 µs; 16 parts are the best
// balance between that and the bucket scan's work of adding up the parts
// (8 and 32 were slower).  Part p counts for the query-preparation workgroups
// [p * bpp, (p + 1) * bpp) (bpp = workgroups per part): the parts are laid
// out one after the other in each bucket, so its segments stay close to
// their input order, and the segments of one request (one d) stay together
// in the 64-segment groups.  The counters are stored part by part (bucket b
// of part p at p * buckets + b): the 64 lanes of a wave, whose keys are
// often consecutive, then hit a few cache lines, which the atomics of one
// instruction share (stored bucket by bucket, the same atomics took as long
// as without parts).  1 or kCountParts parts: kCountParts when parts *
// buckets fits the kMaxBuckets-entry tables.
constexpr uint32_t kCountParts = 16;

uint32_t count_parts(uint32_t nb) {
    return (uint64_t)nb * kCountParts <= kMaxBuckets ? kCountParts : 1u;
}

constexpr uint32_t kPartedBuckets = kMaxBuckets / kCountParts;  // most buckets with parts

constexpr uint32_t kChunkLevels = 4;  // chunk sizes k_bucket_scan chooses from

// Maximum over the kCountParts parts of bucket b (nb buckets).
__device__ __forceinline__ uint32_t parts_max(const uint32_t* c, uint32_t b, uint32_t nb) {
    uint32_t v[kCountParts];
#pragma unroll
    for (uint32_t p = 0; p < kCountParts; ++p) v[p] = c[p * nb + b];
    uint32_t m = 0;
#pragma unroll
    for (uint32_t p = 0; p < kCountParts; ++p) m = max(m, v[p]);
    return m;
}

// Candidates held per lane by the FP32 form: a wave works on tiles of
// kCpl * 64 candidates, so each query record fetched by a scalar load feeds
// kCpl * 64 pair tests.  kCpl is a launch choice (2 or 4, the autotuner's tile
// size); chunks are rounded to whole tiles of the larger one.
constexpr int kCplMax = 4;
constexpr uint32_t kTile = kCplMax * kWave;

// FP64 entry records are read through the constant address space with a
// wave-uniform index, so the compiler fetches them with scalar loads into
// SGPRs: one load serves the 64 lanes (query segments) of the wave.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) f64x4* ConstE64;

struct QueryView {
    const double* a[8];  // xs, ys, zs, ts, xe, ye, ze, te
    const uint32_t* traj;
    uint64_t n;
    // self-join: query segment k is index entry k (its FP64 record, input id
    // and trajectory); each unordered pair of entries of different
    // trajectories is then tested once, from its entry of lower position
    const EntryF64* ent;
    const uint32_t* ent_id;
    const uint32_t* ent_traj;
};

__device__ inline uint64_t lanemask_lt() {
    const uint32_t lane = __lane_id();
    return (lane == 0) ? 0ull : (~0ull >> (64 - lane));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Keeps LDS traffic of one wave in program order around cross-lane exchange.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Where the lanes meet again after a branch that only some of them took.  It
// emits nothing, but gives the meeting point a place of its own: without it
// the compiler merges it with a following loop latch, takes the loop's state
// (queue lengths, masks, counters) to differ between lanes, keeps it in
// vector registers and runs every loop around it under lane masks.  In the
// distance kernel that was all of them: 128 VGPRs with 20-90 spilled.
__device__ inline void rejoin() { __builtin_amdgcn_wave_barrier(); }

// The lane number, computed anew: what is derived from it (masks, addresses)
// is then not kept in registers from the kernel's start on.
__device__ inline uint32_t fresh_lane() {
    uint32_t l = __lane_id();
#if defined(__AMDGCN__)
    asm volatile("" : "+v"(l));
#endif
    return l;
}
__device__ inline uint64_t below(uint32_t lane) { return (1ull << lane) - 1ull; }

__device__ inline uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Lane 0's 64-bit value in every lane (the value need not be uniform).
__device__ inline uint64_t lane0_64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 0);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 0);
    return ((uint64_t)hi << 32) | lo;
}

// ------------------------------------------------------------ schedule

__device__ inline bool finite(double v) { return isfinite(v); }

// Request of query segment k: requests hold contiguous, ascending slices.
__device__ inline uint32_t request_of(const Request* req, uint32_t nreq, uint64_t k) {
    uint32_t l = 0, h = nreq;
    while (h - l > 1) {
        uint32_t mid = (l + h) >> 1;
        if (req[mid].q_begin <= k) l = mid;
        else h = mid;
    }
    return l;
}

// ------------------------------------------------------------ kernels

__global__ __launch_bounds__(kBlock) void k_zero(SearchHeader* hdr, uint32_t* b_count,
                                                 uint32_t* b_hi, uint32_t nb,
                                                 uint32_t nparts, ReqCounter* rc, uint32_t nreq,
                                                 unsigned long long* dyn_ctr,
                                                 unsigned long long dir_first) {
    // nreq: capacity of the request counters (all of them are cleared);
    // b_count and b_hi hold nparts parts for each of the nb buckets;
    // dir_first: first position of the direct output not given to a wave yet
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i == 0) {
        SearchHeader h = {};
        *hdr = h;
    }
    if (i < nb * nparts) {
        b_count[i] = 0;
        b_hi[i] = 0;
    }
    if (i < nreq) {
        rc[i].count = 0;
        rc[i].pad = 0;
    }
    if (i < kCtrSlots * kCtrStride) dyn_ctr[i] = i == kCtrDirect * kCtrStride ? dir_first : 0ull;
}

// Canonical FP64 data of query segment k of request r, from the query
// arrays (the same operations wherever it is needed, so bit-identical).
// Canonical query data from the segment's end points (the velocity of the
// segment as every search form computes it).
__device__ inline void query_canon_pts(double xs, double ys, double zs, double ts, double xe,
                                       double ye, double ze, double te, const Request& R,
                                       QCanon& q) {
    const double dt = te - ts;
    q.x = xs;
    q.y = ys;
    q.z = zs;
    q.vx = (xe - xs) / dt;
    q.vy = (ye - ys) / dt;
    q.vz = (ze - zs) / dt;
    q.ts = ts;
    q.aq = dmax(ts, R.t_start);
    q.bq = dmin(te, R.t_end);
    q.d = R.d;
}

__device__ inline void query_canon(const QueryView& Q, const Request& R, uint64_t k, QCanon& q) {
    if (!Q.ent) {
        query_canon_pts(Q.a[0][k], Q.a[1][k], Q.a[2][k], Q.a[3][k], Q.a[4][k], Q.a[5][k],
                        Q.a[6][k], Q.a[7][k], R, q);
        return;
    }
    double ts, te;
    {
        // the entry record holds the same velocity, computed the same way
        const EntryF64 e = Q.ent[k];
        q.x = e.x;
        q.y = e.y;
        q.z = e.z;
        q.vx = e.vx;
        q.vy = e.vy;
        q.vz = e.vz;
        ts = e.ts;
        te = e.te;
    }
    q.ts = ts;
    q.aq = dmax(ts, R.t_start);
    q.bq = dmin(te, R.t_end);
    q.d = R.d;
}

// One record per lane, the 64 of a wave consecutive in dst (cnt of them
// within the buffer): through LDS, so that each store
// of the wave is one run of 512 bytes.  Straight from the lanes, 88 or 64
// bytes apart, the two records' stores were most of the kernel.
template <class T>
__device__ inline void store_records(T* __restrict__ dst, const T& v, uint64_t* lds, uint32_t cnt) {
    static_assert(sizeof(T) % 8 == 0, "");
    constexpr uint32_t kW = sizeof(T) / 8;
    const uint32_t lane = __lane_id();
    wave_sync();
    __builtin_memcpy(lds + lane * kW, &v, sizeof(T));
    wave_sync();
    uint64_t* d = (uint64_t*)dst;
#pragma unroll
    for (uint32_t i = 0; i < kW; ++i)
        if (i * kWave + lane < cnt * kW) d[i * kWave + lane] = lds[i * kWave + lane];
}

__global__ __launch_bounds__(kBlock) void k_qprep(QueryView Q, const BatchDesc* __restrict__ desc,
                                                  const Request* __restrict__ req, IndexView I,
                                                  QF32* __restrict__ qf,
                                                  QEval* __restrict__ qev,
                                                  uint32_t* __restrict__ qkey,
                                                  uint32_t* __restrict__ qslot, uint32_t* b_count,
                                                  uint32_t* b_hi, uint32_t shift, uint32_t nb,
                                                  uint32_t bpp, SearchHeader* hdr) {
    // the first requests' starts in LDS: the request of a query segment is
    // then found without a chain of dependent global loads
    __shared__ uint64_t s_begin[kBlock];
    __shared__ uint64_t s_rec[kWavesPerBlock][kWave * sizeof(QEval) / 8];
    static_assert(sizeof(QF32) <= sizeof(QEval), "");
    const uint32_t nreq = desc->nreq;
    if (threadIdx.x < nreq) s_begin[threadIdx.x] = req[threadIdx.x].q_begin;
    __syncthreads();
    const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    // this workgroup's part of the bucket counters (k_scatter finds it the
    // same way)
    const uint32_t part = blockIdx.x / bpp;
    bool act = false;  // the segment gets a bucket slot
    uint32_t key = 0;
    QF32 f = {};
    QEval e = {};
    if (k < desc->nq) {
        uint32_t r;
        if (nreq <= kBlock) {
            uint32_t l = 0, h = nreq;
            while (h - l > 1) {
                const uint32_t mid = (l + h) >> 1;
                if (s_begin[mid] <= k) l = mid;
                else h = mid;
            }
            r = l;
        } else {
            r = request_of(req, nreq, k);
        }
        bool ok = true;  // index entries were validated when the index was built
        QCanon p;
        if (Q.ent) {
            query_canon(Q, req[r], k, p);
        } else {
            // the end points are read once, for the validation and the
            // canonical data
            const double xs = Q.a[0][k], ys = Q.a[1][k], zs = Q.a[2][k], ts = Q.a[3][k];
            const double xe = Q.a[4][k], ye = Q.a[5][k], ze = Q.a[6][k], te = Q.a[7][k];
            ok = finite(xs) && finite(ys) && finite(zs) && finite(ts) && finite(xe) &&
                 finite(ye) && finite(ze) && finite(te) && te > ts;
            if (ok) query_canon_pts(xs, ys, zs, ts, xe, ye, ze, te, req[r], p);
        }
        if (!ok) {
            atomicOr(&hdr->err, 1u);
        } else {
            const double ts = p.ts;
            if (p.aq < p.bq) {
                uint32_t lo, hi, j0, j1;
                cand_range(I, p.aq, p.bq, &lo, &hi, &j0, &j1);
                if (Q.ent) lo = max(lo, (uint32_t)k + 1u);  // self-join: entries after k
                if (lo < hi) {
                    const double pax = p.x + p.vx * (p.aq - ts), pay = p.y + p.vy * (p.aq - ts),
                                 paz = p.z + p.vz * (p.aq - ts);
                    const double pbx = p.x + p.vx * (p.bq - ts), pby = p.y + p.vy * (p.bq - ts),
                                 pbz = p.z + p.vz * (p.bq - ts);
                    query_sphere32(pax, pay, paz, pbx, pby, pbz, p.vx, p.vy, p.vz, p.d, f.cx, f.cy,
                                   f.cz, f.R);
                    f.box = seg_box32(pax, pay, paz, pbx, pby, pbz, p.d);
                    f.req = r;
                    f.pad = 0.f;
                    f.a32 = __double2float_rd(p.aq);
                    f.b32 = __double2float_ru(p.bq);
                    f.lo = lo;
                    f.hi = hi;
                    const uint32_t span = min(j1 - j0, kSpanClasses - 1);
                    key = (j0 * kSpanClasses + span) >> shift;
                    act = true;
                    qkey[k] = key;
                    // the bucket's range follows from its key unless it merges
                    // several first bins or spans an open number of bins
                    if (shift || span == kSpanClasses - 1) atomicMax(&b_hi[part * nb + key], hi);
                    e.c = p;
                    if (Q.ent) {
                        e.qid = Q.ent_id[k];
                        e.qtraj = Q.ent_traj[k];
                    } else {
                        e.qid = (uint32_t)(k - req[r].q_begin);
                        e.qtraj = Q.traj ? Q.traj[k] : 0u;
                    }
                }
            }
        }
    }
    const uint32_t wv = threadIdx.x / kWave;
    const uint64_t k0 = k - __lane_id(), nq = desc->nq;
    if (ballot(act)) {
        const uint32_t cnt = (uint32_t)(nq - k0 < kWave ? nq - k0 : kWave);
        store_records(qf + k0, f, s_rec[wv], cnt);
        store_records(qev + k0, e, s_rec[wv], cnt);
    }
    // bucket slots: one atomic per run of equal keys in consecutive lanes
    // (neighbouring query segments often share a bucket, e.g. in the
    // self-join, where a wave's segments are neighbours in one bin)
    const uint32_t lane = __lane_id();
    const uint32_t ke = act ? key : 0xFFFFFFFFu;
    const uint32_t prev = __shfl_up(ke, 1);
    const uint64_t bnd = __ballot(lane == 0 || prev != ke || !act);
    const uint64_t upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const uint32_t start = 63u - (uint32_t)__clzll(bnd & upto);
    const uint64_t above = bnd & ~upto;
    const uint32_t next = above ? (uint32_t)__ffsll((unsigned long long)above) - 1u : 64u;
    uint32_t base = 0;
    if (act && lane == start) base = atomicAdd(&b_count[part * nb + key], next - start);
    base = __shfl(base, start);
    if (k < desc->nq) qslot[k] = act ? base + (lane - start) : kInactive;
}

// Schedule only (tds_schedule): candidate range per query segment.
__global__ __launch_bounds__(kBlock) void k_schedule(QueryView Q, double t_start, double t_end,
                                                     IndexView I, uint32_t* __restrict__ lo_out,
                                                     uint32_t* __restrict__ hi_out,
                                                     uint32_t* err) {
    const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= Q.n) return;
    bool ok = true;
    for (int c = 0; c < 8; ++c) ok = ok && finite(Q.a[c][k]);
    const double ts = Q.a[3][k], te = Q.a[7][k];
    ok = ok && te > ts;
    uint32_t lo = 0, hi = 0;
    if (!ok) {
        atomicOr(err, 1u);
    } else {
        const double aq = dmax(ts, t_start), bq = dmin(te, t_end);
        if (aq < bq) {
            uint32_t j0, j1;
            cand_range(I, aq, bq, &lo, &hi, &j0, &j1);
            if (lo >= hi) lo = hi = 0;
        }
    }
    lo_out[k] = lo;
    hi_out[k] = hi;
}

// Inclusive sum of v over the wave's lanes up to this one.
__device__ inline uint32_t wave_scan(uint32_t v) {
    const uint32_t lane = __lane_id();
#pragma unroll
    for (uint32_t off = 1; off < (uint32_t)kWave; off <<= 1) {
        const uint32_t t = __shfl_up(v, off);
        if (lane >= off) v += t;
    }
    return v;
}

// Candidate range [lo, hi) of bucket b (not empty): first entry of its
// smallest first bin to the end of its last bin (from the key, or the
// members' maximum hi_max where the bucket merges several first bins or spans
// an open number of bins).
__device__ inline void bucket_range(uint32_t b, uint32_t shift, uint32_t m,
                                    const uint32_t* __restrict__ bin_first, uint32_t hi_max,
                                    uint32_t* lo, uint32_t* hi) {
    const uint32_t code = b << shift;  // smallest (j0 * classes + span) of the bucket
    const uint32_t j0 = code / kSpanClasses, span = code % kSpanClasses;
    *lo = bin_first[j0];
    *hi = (shift == 0 && span < kSpanClasses - 1) ? bin_first[min(j0 + span + 1, m)] : hi_max;
}

// Bucket offsets, groups and the work-item table, one block.  The parts of
// each bucket's slot counter become the parts' offsets within the bucket.
//
// Candidates per work item: with levels == 1, `chunk`.  Otherwise the largest
// of chunk, chunk / 2, ... chunk / 2^(levels - 1) that makes at least `target`
// items (about; the count is that of the unrounded chunks), or the smallest of
// them if none does: a search of few items leaves most waves idle while each
// of the others walks its whole chunk.  Each halving at most doubles that
// count, so a smaller chunk than the first never makes 2 target items or more.
//
// Where most items have mixed times (`mixed`, or their bucket spans several bins),
// the chunk is not halved again either where that takes them from at most `fit`
// to more (see item_fit).
__global__ __launch_bounds__(1024) void k_bucket_scan(uint32_t* __restrict__ b_count,
                                                      const uint32_t* __restrict__ b_hi,
                                                      const uint32_t* __restrict__ bin_first,
                                                      const double* __restrict__ min_te,
                                                      const double* __restrict__ max_ts,
                                                      uint32_t m, uint32_t shift,
                                                      uint32_t nb, uint32_t nparts, uint32_t chunk,
                                                      uint32_t levels, uint32_t target,
                                                      uint32_t fit, uint32_t mixed,
                                                      uint32_t* __restrict__ b_start,
                                                      uint32_t* __restrict__ b_nch,
                                                      BucketInfo* __restrict__ binfo,
                                                      SearchHeader* hdr) {
    __shared__ uint32_t s_cnt[kPartedBuckets], s_hi[kPartedBuckets];
    __shared__ uint32_t s_n0[kChunkLevels], s_mixed;
    __shared__ uint32_t s_c[1024 / kWave], s_i[1024 / kWave];
    const uint32_t tid = threadIdx.x, lane = __lane_id(), wv = tid / kWave;
    if (tid < kChunkLevels) s_n0[tid] = 0;
    if (tid == 0) s_mixed = 0;
    if (nparts == kCountParts) {
        // bucket totals and range maxima of the parts (nb <= kPartedBuckets),
        // each part's count replaced by its first slot in the bucket;
        // consecutive threads take consecutive buckets (coalesced)
        for (uint32_t b = tid; b < nb; b += 1024) {
            uint32_t v[kCountParts];
#pragma unroll
            for (uint32_t p = 0; p < kCountParts; ++p) v[p] = b_count[p * nb + b];
            uint32_t cnt = 0;
#pragma unroll
            for (uint32_t p = 0; p < kCountParts; ++p) {
                b_count[p * nb + b] = cnt;
                cnt += v[p];
            }
            s_cnt[b] = cnt;
            const uint32_t code = b << shift;
            s_hi[b] = (cnt && (shift || code % kSpanClasses == kSpanClasses - 1))
                          ? parts_max(b_hi, b, nb)
                          : 0u;
        }
    }
    __syncthreads();
    // each thread's consecutive buckets
    const uint32_t per = (nb + 1023) / 1024;
    const uint32_t b0 = tid * per, b1 = min(nb, b0 + per);
    if (levels > 1) {
        // chunk is a power of two; sums capped at the target, so that the
        // block's total fits 32 bits
        const uint32_t lg = (uint32_t)__builtin_ctz(chunk);
        uint32_t n0[kChunkLevels] = {}, nm = 0;
        const auto add = [&](uint32_t b, uint32_t cnt, uint32_t rmax) {
            uint32_t lo, hi;
            bucket_range(b, shift, m, bin_first, rmax, &lo, &hi);
            const uint64_t len = hi - (lo & ~(uint32_t)(kWave - 1));
#pragma unroll
            for (uint32_t l = 0; l < kChunkLevels; ++l) {
                const uint64_t n = (uint64_t)((cnt + kWave - 1) / kWave) *
                                   ((len + (chunk >> l) - 1) >> (lg - l));
                n0[l] = (uint32_t)min(n0[l] + n, (uint64_t)target);
                if (l == 0 && (mixed || shift || b % kSpanClasses))
                    nm = (uint32_t)min(nm + n, (uint64_t)target);
            }
        };
        if (nparts == kCountParts) {
#pragma unroll 1
            for (uint32_t b = tid; b < nb; b += 1024)
                if (s_cnt[b]) add(b, s_cnt[b], s_hi[b]);
        } else {
            // any order will do: consecutive threads take consecutive buckets, and a
            // few counts are asked for together (65,535 buckets, each thread's own
            // one after another: 20 us)
            constexpr uint32_t kAtOnce = 4;
            for (uint32_t bb = tid; bb < nb; bb += 1024 * kAtOnce) {
                uint32_t cnts[kAtOnce];
#pragma unroll
                for (uint32_t i = 0; i < kAtOnce; ++i)
                    cnts[i] = bb + 1024 * i < nb ? b_count[bb + 1024 * i] : 0u;
#pragma unroll
                for (uint32_t i = 0; i < kAtOnce; ++i)
                    if (cnts[i]) add(bb + 1024 * i, cnts[i], b_hi[bb + 1024 * i]);
            }
        }
        nm = wave_scan(nm);
        if (lane == kWave - 1 && nm) atomicAdd(&s_mixed, nm);
#pragma unroll
        for (uint32_t l = 0; l < kChunkLevels; ++l) {
            const uint32_t sum = wave_scan(n0[l]);
            if (lane == kWave - 1 && sum) atomicAdd(&s_n0[l], sum);
        }
        __syncthreads();
        if (2 * s_mixed <= s_n0[0]) fit = 0;
        uint32_t l = 0;
        while (l + 1 < levels && s_n0[l] < target &&
               !(l && s_n0[l] <= fit && s_n0[l + 1] > fit))
            ++l;
        chunk >>= l;
    }
    // the record of each bucket (all but its offsets), then the offsets after
    // the scan.  Items per bucket are kept in s_hi (parts) or b_nch for the
    // second pass.
    uint32_t sc = 0, si = 0;
    for (uint32_t b = b0; b < b1; ++b) {
        const uint32_t cnt = nparts == kCountParts ? s_cnt[b] : b_count[b];
        BucketInfo bi;
        bi.lo = 0xFFFFFFFFu;
        bi.hi = 0;
        bi.nch = 0;
        bi.clen = 0;
        bi.count = cnt;
        bi.start = 0;
        bi.item0 = 0;
        bi.pad = 0;
        bi.tmin_te = -INFINITY;  // unknown: the kernel keeps the per-pair time test
        bi.tmax_ts = INFINITY;
        bi.pad2[0] = bi.pad2[1] = 0.0;
        if (cnt) {
            const uint32_t code = b << shift;
            const uint32_t j0 = code / kSpanClasses, span = code % kSpanClasses;
            uint32_t lo, hi;
            bucket_range(b, shift, m, bin_first, nparts == kCountParts ? s_hi[b] : b_hi[b], &lo,
                         &hi);
            if (shift == 0 && span < kSpanClasses - 1) {
                // time bounds of the bins the bucket's range covers
                const uint32_t j1 = min(j0 + span, m - 1);
                double mn = INFINITY, mx = -INFINITY;
                for (uint32_t j = j0; j <= j1; ++j) {
                    mn = fmin(mn, min_te[j]);
                    mx = fmax(mx, max_ts[j]);
                }
                bi.tmin_te = mn;
                bi.tmax_ts = mx;
            }
            // balanced chunks of at most `chunk` candidates counted from the
            // 64-entry block of lo (chunk c covers [base + c clen, base +
            // (c + 1) clen) clipped to [lo, hi)), whole 64-candidate tiles
            // where possible, none empty
            const uint32_t len = hi - (lo & ~(uint32_t)(kWave - 1));
            const uint32_t n0 = (len + chunk - 1) / chunk;
            uint32_t clen = (len + n0 - 1) / n0;
            clen = (clen + kWave - 1) / kWave * kWave;
            if (clen > 2 * kTile) clen = (clen + kTile - 1) / kTile * kTile;
            bi.lo = lo;
            bi.hi = hi;
            bi.clen = clen;
            bi.nch = (len + clen - 1) / clen;
        }
        binfo[b] = bi;
        const uint32_t items = ((cnt + kWave - 1) / kWave) * bi.nch;
        if (nparts == kCountParts) s_hi[b] = items;
        else b_nch[b] = items;
        sc += cnt;
        si += items;
    }
    // sums over the threads before this one: within the wave, then the waves'
    // totals (two barriers)
    const uint32_t ic = wave_scan(sc), ii = wave_scan(si);
    if (lane == kWave - 1) {
        s_c[wv] = ic;
        s_i[wv] = ii;
    }
    __syncthreads();
    uint32_t rc = ic - sc, ri = ii - si;
    for (uint32_t w = 0; w < wv; ++w) {
        rc += s_c[w];
        ri += s_i[w];
    }
    if (tid == 1023) {
        hdr->n_items = ri + si;
        hdr->n_buckets = nb;
        hdr->active = rc + sc;  // every active query segment has a bucket slot
    }
    for (uint32_t b = b0; b < b1; ++b) {
        uint32_t cnt, items;
        if (nparts == kCountParts) {
            cnt = s_cnt[b];
            items = s_hi[b];
        } else {
            cnt = b_count[b];
            items = b_nch[b];
            b_count[b] = 0;  // the one part's first slot
        }
        b_start[b] = rc;
        binfo[b].start = rc;
        binfo[b].item0 = ri;
        rc += cnt;
        ri += items;
    }
}

// Workgroups [0, qblocks): one thread per query segment, whose number goes to
// its bucket position (bucket start + its counter part's offset + its slot in
// the part).  Only the number: copying the records along (64 to 152 bytes to
// scattered places) cost 15-50 us more than the distance kernel saves by not
// following the number.
// Workgroups [qblocks, qblocks + nb): item_bucket[i] = bucket of work item i,
// one workgroup per bucket.
__global__ __launch_bounds__(kBlock) void k_scatter(const BatchDesc* __restrict__ desc,
                                                    const uint32_t* __restrict__ qkey,
                                                    const uint32_t* __restrict__ qslot,
                                                    const uint32_t* __restrict__ b_start,
                                                    const uint32_t* __restrict__ b_part,
                                                    uint32_t nb, uint32_t bpp, uint32_t qblocks,
                                                    uint32_t* __restrict__ qsorted,
                                                    const BucketInfo* __restrict__ binfo,
                                                    uint32_t* __restrict__ item_bucket,
                                                    SearchHeader* hdr) {
    if (blockIdx.x < qblocks) {
        const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
        if (k >= desc->nq) return;
        const uint32_t s = qslot[k];
        if (s == kInactive) return;
        const uint32_t key = qkey[k];
        qsorted[b_start[key] + b_part[(blockIdx.x / bpp) * nb + key] + s] = (uint32_t)k;
        return;
    }
    const uint32_t b = blockIdx.x - qblocks;
    const BucketInfo bi = binfo[b];
    const uint32_t n = ((bi.count + kWave - 1) / kWave) * bi.nch;
    const uint32_t cap = desc->item_cap;
    if (threadIdx.x == 0 && n && (uint64_t)bi.item0 + n > cap) atomicOr(&hdr->err, 2u);
    for (uint32_t i = threadIdx.x; i < n; i += kBlock)
        if (bi.item0 + i < cap) item_bucket[bi.item0 + i] = b;
}

// Resets the per-pass request counters and the dynamic item counters of the
// distance kernel.
__global__ void k_reset_pass(ReqCounter* rc, uint32_t nreq, unsigned long long* dyn_ctr) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nreq) rc[i].count = 0;
    if (i < kCtrSlots * kCtrStride) dyn_ctr[i] = 0;
}

// Adds the per-workgroup counters of one distance-kernel launch to the
// header (one block of kThreads).
template <uint32_t kThreads>
__device__ inline void fold_stats(const BlockStats* __restrict__ bs, uint32_t nb,
                                  SearchHeader* hdr) {
    __shared__ uint64_t red[5][kThreads / kWave];
    uint64_t v[5] = {0, 0, 0, 0, 0};
    for (uint32_t i = threadIdx.x; i < nb; i += kThreads) {
        const BlockStats b = bs[i];
        v[0] += b.tests;
        v[1] += b.evals;
        v[2] += b.ftests;
        v[3] += b.btests;
        v[4] += b.flushes;
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        for (uint32_t off = kWave / 2; off; off >>= 1) v[k] += __shfl_xor(v[k], (int)off);
        if (__lane_id() == 0) red[k][threadIdx.x / kWave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 0; k < 5; ++k) v[k] = 0;
        for (uint32_t w = 0; w < kThreads / kWave; ++w)
            for (int k = 0; k < 5; ++k) v[k] += red[k][w];
        hdr->tests += v[0];
        hdr->evals += v[1];
        hdr->ftests += v[2];
        hdr->btests += v[3];
        hdr->flushes += (uint32_t)v[4];
    }
}
__global__ __launch_bounds__(256) void k_stats_fold(const BlockStats* __restrict__ bs, uint32_t nb,
                                                    SearchHeader* hdr) {
    fold_stats<256>(bs, nb, hdr);
}

// Waves of a distance-kernel launch that may use direct output (the fill
// plan keeps one 16-bit entry per chunk it looks at, at most one more than
// the waves, in LDS).
constexpr uint32_t kMaxDirectWaves = 16384;

// Exclusive prefix sums of f(0..n-1) into out[0..n] (out[n] = total) by one
// workgroup of 1024 threads, 1024 values per round.
template <class F>
__device__ void block_scan_1024(uint32_t n, F f, uint64_t* __restrict__ out) {
    __shared__ uint64_t wsum[1024 / kWave];
    __shared__ uint64_t carry_s;
    const uint32_t t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    if (t == 0) carry_s = 0;
    __syncthreads();
    for (uint32_t r0 = 0; r0 < n; r0 += 1024) {
        const uint32_t i = r0 + t;
        const uint64_t v = i < n ? f(i) : 0;
        uint64_t x = v;
        for (uint32_t o = 1; o < kWave; o <<= 1) {
            const uint64_t y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == kWave - 1) wsum[wv] = x;
        __syncthreads();
        uint64_t before = carry_s;
        for (uint32_t k = 0; k < wv; ++k) before += wsum[k];
        if (i < n) out[i] = before + x - v;
        __syncthreads();
        if (t == 1023) carry_s = before + x;
        __syncthreads();
    }
    if (t == 0) out[n] = carry_s;
}

// Direct output, after the distance kernel (one workgroup): the plan of the
// fill.  T = min(count, capacity) is the end of the dense output.  The
// holes are the unused tails of the waves' last chunks below T (at most one
// per wave, none of a wave that reserved nothing: ~0 in dlast); the sources
// are the results at positions at or past T, in position order, of which the
// first (total hole size) are moved.  Those lie within W (C - 1) positions of T
// (every hole is shorter than C), so the chunks c0 = T / C .. c0 + W are enough,
// and positions past the capacity within W C of it are in the scratch buffer.
// Writes the source prefix sums per chunk, the hole prefix sums and starts per
// wave, and (T, c0, chunks).
__global__ __launch_bounds__(1024) void k_fill_plan(const Request* __restrict__ req,
                                                    const ReqCounter* __restrict__ rc,
                                                    const unsigned long long* __restrict__ dir_ctr,
                                                    const uint64_t* __restrict__ dlast, uint32_t nw,
                                                    uint32_t C, uint64_t* __restrict__ s_pre,
                                                    uint64_t* __restrict__ d_pre,
                                                    uint64_t* __restrict__ d_start,
                                                    uint64_t* __restrict__ plan) {
    __shared__ uint16_t used[kMaxDirectWaves + 1];  // positions used of chunk c0 + i
    const uint32_t t = threadIdx.x;
    const uint64_t count = rc[0].count, cap = req[0].out_capacity, R = *dir_ctr;
    const uint64_t T = min(count, cap);
    const uint64_t c0 = T / C, nch = R / C;
    const uint32_t ns = nch > c0 ? (uint32_t)min(nch - c0, (uint64_t)nw + 1) : 0u;
    for (uint32_t i = t; i < ns; i += 1024) used[i] = (uint16_t)C;  // full unless a last chunk
    __syncthreads();
    for (uint32_t w = t; w < nw; w += 1024) {
        const uint64_t v = dlast[w];
        if (v == ~0ull) continue;
        const uint64_t k = v >> 16;
        if (k >= c0 && k - c0 < ns) used[k - c0] = (uint16_t)(v & 0xFFFFu);
    }
    __syncthreads();
    block_scan_1024(
        ns,
        [&](uint32_t i) -> uint64_t {
            const uint64_t cb = (c0 + i) * C, a = max(cb, T), e = cb + used[i];
            return e > a ? e - a : 0;
        },
        s_pre);
    block_scan_1024(
        nw,
        [&](uint32_t w) -> uint64_t {
            const uint64_t v = dlast[w];
            if (v == ~0ull) return 0;
            const uint64_t cb = (v >> 16) * C, a = cb + (v & 0xFFFFu), e = min(cb + C, T);
            d_start[w] = a;
            return e > a ? e - a : 0;
        },
        d_pre);
    if (t == 0) {
        plan[0] = T;
        plan[1] = c0;
        plan[2] = ns;
    }
}

// Direct output: moves source t of the plan to hole position t (any pairing
// of the two lists makes the output dense; a source is never a hole below T).
__global__ __launch_bounds__(256) void k_fill_copy(const uint64_t* __restrict__ plan,
                                                   const uint64_t* __restrict__ s_pre,
                                                   const uint64_t* __restrict__ d_pre,
                                                   const uint64_t* __restrict__ d_start,
                                                   uint32_t nw, uint32_t C,
                                                   const Request* __restrict__ req,
                                                   tds_result* __restrict__ out,
                                                   const tds_result* __restrict__ scratch) {
    const uint64_t T = plan[0], c0 = plan[1];
    const uint32_t ns = (uint32_t)plan[2];
    const uint64_t total = d_pre[nw];
    const Request R = req[0];
    for (uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x; t < total;
         t += (uint64_t)gridDim.x * 256) {
        uint32_t lo = 0, hi = nw;  // last hole with d_pre <= t
        while (hi - lo > 1) {
            const uint32_t m = (lo + hi) >> 1;
            if (d_pre[m] <= t) lo = m;
            else hi = m;
        }
        const uint64_t dst = d_start[lo] + (t - d_pre[lo]);
        uint32_t a = 0, b = ns;  // last source chunk with s_pre <= t
        while (b - a > 1) {
            const uint32_t m = (a + b) >> 1;
            if (s_pre[m] <= t) a = m;
            else b = m;
        }
        const uint64_t src = max((c0 + a) * C, T) + (t - s_pre[a]);
        const tds_result v =
            src < R.out_capacity ? out[R.out_offset + src] : scratch[src - R.out_capacity];
        out[R.out_offset + dst] = v;
    }
}

// A wave's last reservation in dlast: g chunks of C positions of which it used
// the first `used`, as (g - 1) << 56 | first chunk << 16 | used.
__device__ inline uint64_t pack_last(uint64_t first, uint32_t g, uint32_t used) {
    return (uint64_t)(g - 1) << 56 | first << 16 | used;
}
struct LastRes {
    uint64_t first;   // chunk
    uint64_t a, e;    // its unused positions [a, e)
};
__device__ inline LastRes unpack_last(uint64_t v, uint32_t C) {
    LastRes l;
    l.first = v >> 16 & ((1ull << 40) - 1);
    l.a = l.first * C + (v & 0xFFFFu);
    l.e = (l.first + (v >> 56) + 1) * C;
    return l;
}

// Direct output of a launch of up to kFillWaves waves, after the distance
// kernel: the number of results (positions reserved less the unused ones), the
// fill (see k_fill_plan: holes below T = min(count, capacity), sources at or
// past T) and, by the last workgroup, the fold of the launch's counters.
// Between T and the last source that is moved lie no more positions than all
// the unused ones together, U, so the chunks T / C .. T / C + U / C + 1 are
// enough, and positions past the capacity within U of it are in the scratch
// buffer.
//
// Bound by the latency of the chain launch, load of the waves' words, prefix
// sums, load of the records, store, at about 2 us for each access that comes
// from memory.  So every workgroup makes the plan for itself, in LDS: as two
// kernels (one workgroup's plan in memory, then the copy) and the fold it was
// three launches and 25 us for a small search, now 12.5 (dense walks, 8000
// items: 53 -> 16.5).  The sums fit 32 bits: U is
// at most the stage buffer's 2^23 records.
constexpr uint32_t kFillWaves = 4096;
constexpr uint32_t kFillBlocks = 128;  // and one for the fold
constexpr uint32_t kFillChunks = 4 * kFillWaves;  // most chunks of the waves' last reservations
__global__ __launch_bounds__(1024) void k_fill(const Request* __restrict__ req,
                                               ReqCounter* __restrict__ rc,
                                               const unsigned long long* __restrict__ dir_ctr,
                                               const uint64_t* __restrict__ dlast, uint32_t nw,
                                               uint32_t C, tds_result* __restrict__ out,
                                               const tds_result* __restrict__ scratch,
                                               const BlockStats* __restrict__ bs, uint32_t nb,
                                               SearchHeader* __restrict__ hdr) {
    __shared__ uint64_t last[kFillWaves];
    __shared__ uint32_t hpre[kFillWaves];       // hole positions before wave w's
    __shared__ uint32_t src[kFillChunks + 2];   // positions used of chunk c0 + i at or past T,
                                                // then the sources before them
    __shared__ uint32_t s_u[1024 / kWave], s_s[1024 / kWave], s_d[1024 / kWave];
    if (blockIdx.x == gridDim.x - 1) {
        fold_stats<1024>(bs, nb, hdr);
        return;
    }
    const uint32_t t = threadIdx.x, lane = __lane_id(), wv = t / kWave;
    const Request Rq = req[0];
    const uint64_t R = *dir_ctr;
    for (uint32_t w = t; w < nw; w += 1024) last[w] = dlast[w];
    __syncthreads();
    // consecutive waves, and below consecutive chunks, per thread: a prefix sum
    // is one step within the waves and one over them
    const uint32_t pw = (nw + 1023) / 1024, w0 = min(nw, t * pw), w1 = min(nw, w0 + pw);
    const auto over_c = [&](uint64_t v) {
        return C & (C - 1) ? v / C : v >> (uint32_t)__builtin_ctz(C);
    };
    uint32_t u = 0;
#pragma unroll 1
    for (uint32_t w = w0; w < w1; ++w) {
        const LastRes l = unpack_last(last[w], C);
        u += (uint32_t)(l.e - l.a);
    }
    u = wave_scan(u);
    if (lane == kWave - 1) s_u[wv] = u;
    __syncthreads();
    uint32_t unused = 0;
#pragma unroll 1
    for (uint32_t k = 0; k < 1024 / kWave; ++k) unused += s_u[k];
    const uint64_t count = R - unused, T = min(count, Rq.out_capacity);
    const uint64_t c0 = over_c(T), nch = over_c(R);
    const uint32_t skip = (uint32_t)(T - c0 * C);  // chunk c0's positions below T
    const uint32_t ns =
        nch > c0 ? (uint32_t)min(min(nch - c0, over_c(unused) + 2), (uint64_t)kFillChunks + 2)
                 : 0u;
    // full unless a wave's last
    for (uint32_t i = t; i < ns; i += 1024) src[i] = C - (i ? 0u : skip);
    __syncthreads();
    uint32_t dsum = 0;
#pragma unroll 1
    for (uint32_t w = w0; w < w1; ++w) {
        const LastRes l = unpack_last(last[w], C);
        const uint64_t e = min(l.e, T);
        if (e > l.a) dsum += (uint32_t)(e - l.a);
        uint64_t p = l.first * C;
        for (uint64_t k = l.first; p < l.e; ++k, p += C)
            if (p + C > l.a && k >= c0 && k - c0 < ns) {
                const uint64_t f = max(p, T);
                src[k - c0] = l.a > f ? (uint32_t)(l.a - f) : 0u;
            }
    }
    __syncthreads();
    const uint32_t ps = (ns + 1023) / 1024, i0 = min(ns, t * ps), i1 = min(ns, i0 + ps);
    uint32_t ssum = 0;
#pragma unroll 1
    for (uint32_t i = i0; i < i1; ++i) ssum += src[i];
    const uint32_t is = wave_scan(ssum), id = wave_scan(dsum);
    if (lane == kWave - 1) {
        s_s[wv] = is;
        s_d[wv] = id;
    }
    __syncthreads();
    uint32_t sp = is - ssum, dp = id - dsum, total = 0;
#pragma unroll 1
    for (uint32_t k = 0; k < 1024 / kWave; ++k) {
        if (k < wv) {
            sp += s_s[k];
            dp += s_d[k];
        }
        total += s_d[k];
    }
#pragma unroll 1
    for (uint32_t i = i0; i < i1; ++i) {
        const uint32_t n = src[i];
        src[i] = sp;
        sp += n;
    }
#pragma unroll 1
    for (uint32_t w = w0; w < w1; ++w) {
        const LastRes l = unpack_last(last[w], C);
        const uint64_t e = min(l.e, T);
        hpre[w] = dp;
        if (e > l.a) dp += (uint32_t)(e - l.a);
    }
    if (blockIdx.x == 0 && t == 0) rc[0].count = count;
    __syncthreads();
    // last entry of p[0 .. n) that is at most x (p[0] is 0)
    const auto find = [](const uint32_t* p, uint32_t n, uint32_t x) {
        uint32_t a = 0;
        while (n > 1) {
            const uint32_t h = n >> 1;
            if (p[a + h] <= x) a += h;
            n -= h;
        }
        return a;
    };
    for (uint32_t x = blockIdx.x * 1024 + t; x < total; x += (gridDim.x - 1) * 1024) {
        const uint32_t w = find(hpre, nw, x), a = find(src, ns, x);
        const uint64_t dst = unpack_last(last[w], C).a + (x - hpre[w]);
        const uint64_t from = max((c0 + a) * C, T) + (x - src[a]);
        const tds_result v =
            from < Rq.out_capacity ? out[Rq.out_offset + from] : scratch[from - Rq.out_capacity];
        out[Rq.out_offset + dst] = v;
    }
}

// The distance kernel's arguments.  Steps off the filter's walk take them from
// the kernel's argument block anew (cold_args), so that they are not held in
// scalar registers, which spilled by the dozen, across the walk.
struct DistArgs {
    IndexView I;
    uint32_t self;           // self-join (see QueryView)
    uint32_t keep;           // results stay staged from item to item (at most 64 requests)
    const uint32_t* qsorted; // query segments in bucket order
    const QF32* qf;          // their records in query order
    const QEval* qev;
    const BucketInfo* binfo;
    const uint32_t* item_bucket;
    const BatchDesc* desc;
    SearchHeader* hdr;
    BlockStats* bstats;
    const Request* req;
    ReqCounter* rc;
    tds_result* out;
    uint64_t win_lo;        // first request-local result position kept
    unsigned long long* dyn_ctr;  // per-XCD dynamic item counters (kCtrStride apart)
    uint32_t item_begin;    // work items [item_begin, item_end)
    uint32_t item_end;      // 0xFFFFFFFF: every item of the search
    uint32_t* item_count;   // results per work item, or nullptr
    tds_result* stage;      // per-wave result stages, stage_cap records each
    uint32_t* stage_meta;   // slot | index among the slot's staged results << 6
    uint32_t stage_cap;     // records per wave (a multiple of 64)
    uint32_t by_order;      // 1: a single-request item run whose results go to
                            // their order in the item (minus win_lo), no stage
    uint32_t cpl;           // FP32 form: candidates per lane per tile (2 or 4)
    uint32_t refine;        // FP32 form: TDS_REFINE_QUEUED or TDS_REFINE_INLINE
    uint32_t deal;          // TDS_DEAL_STATIC or TDS_DEAL_DYNAMIC
    // direct output (one request, not by_order): results go straight to the
    // request's output through per-wave reservations of dir_chunk positions
    uint32_t direct;
    uint32_t dir_chunk;
    uint32_t dir_max;       // most chunks of one reservation
    uint32_t dir_given;     // every wave starts with the chunk of its number (k_fill); else
                            // with none, and adds its results to the request's counter
    unsigned long long* dir_ctr;  // next free position (reservation counter)
    tds_result* dscratch;   // positions [cap, cap + dscratch_cap) (the stage buffer)
    uint64_t dscratch_cap;
    uint64_t* dlast;        // per wave: last reservation (pack_last)
};

#if defined(__AMDGCN__)
typedef const __attribute__((address_space(4))) DistArgs* ArgsPtr;
__device__ __forceinline__ ArgsPtr cold_args(const DistArgs&) {
    ArgsPtr p = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
#else
typedef const DistArgs* ArgsPtr;
inline ArgsPtr cold_args(const DistArgs& A) { return &A; }
#endif

// FP32 data of a query segment for the closest-approach refinement (one per
// group lane, refine32).
struct QRef {
    float ox, oy, oz;  // the sphere centre moved to time 0 (c - v t, t its time)
    float vx, vy, vz;  // velocity
    float d;           // d + 2^-17 times the query's part of the position scale
    float st;          // |a| + |b| + |t| + 1, [a, b] the clipped extent rounded outwards
};
static_assert(sizeof(QRef) == 32, "QRef layout");

// Results go through a stage of stage_cap records per wave in device memory
// and get their output positions when the stage is flushed: one device-scope
// atomic per request slot with staged results reserves exactly their number.  A
// returning atomic that every wave directs at its request's counter serialises
// across the chip, 14 ns each: one per 64 evaluations cost a search with 10^8
// results most of its time.  Positions within a request are unique and dense, in
// no fixed order.
//
// With up to 64 requests (keep) slot r is request r and results stay staged from
// item to item, until the next batch of evaluations might not fit or the wave has
// no more items; then the workgroup's waves reserve together.  Flushed at the end
// of every item, 10,000 items of dense walks took 142 us, 124 in a batch of three
// requests, of which 65 are the walk.  With more requests a slot is the
// first query of the group with the same request, which the next group shares
// nothing with: flushed at the end of every item.
//
// With by_order set (one request, one work item, re-run to fill successive
// windows of the host's buffer), a result's position is instead its order
// among the item's results, which a wave computes the same way on every run.
//
// Direct output (a one-request search's first pass): a wave writes its results
// straight to consecutive positions of the request that it reserved, first the
// dir_chunk positions of its own number, then twice as many chunks as the last
// time, up to dir_max (one atomic per reservation; whole aligned chunks),
// keeping its last reservation open from one item to the next.  In launches of more
// than kFillWaves waves it reserves a chunk when it has results: most waves have
// none, and the holes that their first chunks would leave took 10 to 24 us.  At the end it
// may be partly used; positions at or past the output capacity go to a scratch
// buffer.  A fill pass (k_fill, or k_fill_plan and k_fill_copy) then moves the
// results found past the final count (or the capacity) into the unused tails
// below it, so that the output is dense again.  No result takes the round trip
// through a stage.
// Filter data of a query segment as the wave keeps it in LDS: the sphere and
// the clipped extent of its QF32 record, apart, since most slots need only the
// sphere (the candidate range stays in the registers of the query's lane).
struct alignas(16) QSphere {
    float cx, cy, cz, R;
};
struct alignas(8) QTime {
    float a, b;
};

// The wave's LDS: 10,240 bytes, so that four workgroups of four waves fit in a
// compute unit's 160 KB.  Per-lane values of the group (the request of query
// j, its request slot, the staged results of a slot) live in the registers of
// lane j (ItemState) and are read across lanes by shuffles.
struct alignas(64) WaveLDS {
    uint32_t queue[2 * kWave];  // sphere survivors to refine: < 64 left over + one per lane
    uint32_t rq[2 * kWave];     // pairs awaiting the FP64 evaluation, likewise
    QSphere qs[kWave];          // filter data of the item's query group
    QTime qt[kWave];
    QRef qref[kWave];           // FP32 form: refinement data of the group's queries
    QEval qe[kWave];            // FP64 data of the group's queries
};
static_assert(sizeof(WaveLDS) == 10240, "WaveLDS size");

struct ItemState {
    uint32_t c0, c1, qbase, nq;
    uint32_t qn, rqn;  // pairs in the two queues
    uint32_t evals;
    uint32_t found;   // results of the item so far (their order in the item)
    uint32_t nst;     // results in the wave's stage
    uint64_t sbase;   // the wave's stage: records [sbase, sbase + stage_cap)
    uint64_t ftests, btests;
    uint32_t hits;    // without boxes: kAhead times the queries that had survivors in
                      // the last block, less its queries (kept across items)
    // direct output: the wave's open reservation [dpos, dend) (kept across
    // items) and its reservations so far
    uint64_t dpos, dend;
    uint32_t dg;      // chunks of the open reservation
    uint32_t nres;
    // per lane j of the group
    uint32_t qr;      // request of query j
    uint32_t rslot;   // its request slot (see DistArgs)
    uint32_t rcnt;    // staged results of request slot j (slot lanes only)
};

// Wave-wide ordering of device-memory accesses: stores of one lane are
// visible to loads of the other lanes after it (the stage is written by the
// lane that found a result and read back by the lane that copies it).
__device__ inline void wave_sync_mem() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
}

// Staged records each lane copies per round of a flush (their loads in
// flight together).
constexpr int kFlushUnroll = 2;

// Copies the wave's nst staged results to their positions.  Slot lane s knows
// where its results go: the n staged results of the slot have positions base + k of
// request r, and k is kept when that falls in the window [win_lo, win_lo +
// out_capacity), at out[dst + k].  The copy reads kFlushUnroll records per lane
// before it writes any, so it waits for about one memory round trip per 128
// records.
__device__ __forceinline__ void stage_copy(const ArgsPtr A, uint64_t sbase, uint32_t nst,
                                           uint32_t r, uint32_t n, uint64_t base) {
    const uint32_t lane = fresh_lane();
    int64_t dst = 0;
    uint32_t klo = 0, khi = 0;  // kept staged results of slot `lane`: [klo, khi)
    if (n) {
        const Request& R = A->req[r];
        const uint64_t w0 = A->win_lo, w1 = A->win_lo + R.out_capacity, nn = n;
        klo = (uint32_t)min(max(w0, base) - base, nn);
        khi = (uint32_t)min(max(w1, base) - base, nn);
        dst = (int64_t)R.out_offset + (int64_t)base - (int64_t)A->win_lo;
    }
    // (nothing to copy once the output is full)
    const uint32_t end = ballot(klo < khi) ? nst : 0u;
    for (uint32_t p0 = 0; p0 < end; p0 += kFlushUnroll * kWave) {
        uint32_t meta[kFlushUnroll];
        uint4 ra[kFlushUnroll], rb[kFlushUnroll];
#pragma unroll
        for (int u = 0; u < kFlushUnroll; ++u) {
            const uint32_t p = p0 + u * kWave + lane;
            meta[u] = 0xFFFFFFFFu;  // no record (a real one is below 2^17)
            ra[u] = rb[u] = make_uint4(0u, 0u, 0u, 0u);
            if (p < nst) {
                meta[u] = A->stage_meta[sbase + p];
                const uint4* src = reinterpret_cast<const uint4*>(A->stage + sbase + p);
                ra[u] = src[0];
                rb[u] = src[1];
            }
        }
#pragma unroll
        for (int u = 0; u < kFlushUnroll; ++u) {
            // every lane takes part in the shuffles
            const uint32_t slot = meta[u] & (kWave - 1);
            const uint32_t k = (meta[u] >> 6) & 0x3FFFFFFu;
            const int64_t d = __shfl((long long)dst, (int)slot);
            const uint32_t lo = (uint32_t)__shfl((int)klo, (int)slot);
            const uint32_t hi = (uint32_t)__shfl((int)khi, (int)slot);
            if (meta[u] != 0xFFFFFFFFu && k >= lo && k < hi) {
                uint4* o = reinterpret_cast<uint4*>(A->out + (d + (int64_t)k));
                o[0] = ra[u];
                o[1] = rb[u];
            }
            rejoin();
        }
    }
}

// Reserves the staged results of every request slot (one atomic each) and
// copies them from the stage to their positions; the stage is then empty.
__device__ __forceinline__ void stage_flush(WaveLDS& L, const DistArgs& A0, ItemState& S) {
    const uint32_t lane = fresh_lane();
    const ArgsPtr A = cold_args(A0);
    wave_sync_mem();
    const uint32_t r = A->keep ? lane : S.qr;
    uint64_t base = 0;
    if (S.rcnt) base = (uint64_t)atomicAdd(&A->rc[r].count, (unsigned long long)S.rcnt);
    stage_copy(A, S.sbase, S.nst, r, S.rcnt, base);
    S.rcnt = 0;
    S.nst = 0;
    wave_sync_mem();
}

// Evaluates the last min(rqn, 64) pairs of the refined queue (one per lane)
// with the canonical FP64 code and writes or stages the results.
__device__ __forceinline__ void drain(WaveLDS& L, ItemState& S, const DistArgs& A0) {
    const uint32_t lane = fresh_lane();
    const ArgsPtr A = cold_args(A0);
    const uint32_t cnt = min(S.rqn, (uint32_t)kWave);
    wave_sync();
    S.rqn -= cnt;
    const bool act = lane < cnt;
    const uint32_t pk = act ? L.rq[S.rqn + lane] : 0u;
    wave_sync();
    const uint32_t ql = pk & (kWave - 1);
    const uint32_t i = S.c0 + (pk >> 6);
    const uint32_t slot = (uint32_t)__shfl((int)S.rslot, (int)ql);  // every lane takes part
    double t_lo = 0.0, t_hi = 0.0;
    bool hit = false;
    uint32_t qid = 0, qtraj = 0, eid = 0, etraj = 0;
    if (act) {
        const EntryF64 e = A->I.e64[i];
        eid = A->I.seg_id[i];
        etraj = A->I.traj[i];
        const QCanon& q = L.qe[ql].c;
        qid = L.qe[ql].qid;
        qtraj = L.qe[ql].qtraj;
        hit = canon_eval<true>(q, e.x, e.y, e.z, e.vx, e.vy, e.vz, e.ts, e.te, &t_lo, &t_hi);
        if (A->self) {
            // self-join: pairs of one trajectory are not results, and a record
            // names the lower segment id first (its interval is symmetric)
            hit = hit && qtraj != etraj;
            if (qid > eid) {
                const uint32_t t0 = qid, t1 = qtraj;
                qid = eid;
                qtraj = etraj;
                eid = t0;
                etraj = t1;
            }
        }
    }
    tds_result rec;
    rec.q_seg = qid;
    rec.e_seg = eid;
    rec.q_traj = qtraj;
    rec.e_traj = etraj;
    rec.t_lo = t_lo;
    rec.t_hi = t_hi;
    const uint64_t hm = ballot(hit);
    const uint32_t nhit = (uint32_t)__popcll(hm);
    const uint32_t rank = (uint32_t)__popcll(hm & below(lane));
    S.evals += cnt;
    if (A->by_order) {
        const uint64_t pos = (uint64_t)S.found + rank;
        const Request& R = A->req[0];
        if (hit && pos >= A->win_lo && pos - A->win_lo < R.out_capacity)
            A->out[R.out_offset + (pos - A->win_lo)] = rec;
        rejoin();
        S.found += nhit;
        return;
    }
    if (A->direct) {
        if (!nhit) return;
        // nhit <= 64 <= dir_chunk: at most one new reservation, of twice the
        // last one's chunks
        const uint64_t room = S.dend - S.dpos;
        uint64_t pos = S.dpos + rank;
        if (nhit > room) {
            unsigned long long nb = 0;
            S.dg = min(2 * S.dg, A->dir_max);
            const uint32_t size = S.dg * A->dir_chunk;
            if (lane == 0) nb = atomicAdd(A->dir_ctr, (unsigned long long)size);
            const uint64_t b = lane0_64(nb);
            if (rank >= room) pos = b + (rank - room);
            S.dpos = b + (nhit - room);
            S.dend = b + size;
            ++S.nres;
        } else {
            S.dpos += nhit;
        }
        if (hit) {
            const Request& R = A->req[0];
            if (pos < R.out_capacity) A->out[R.out_offset + pos] = rec;
            else if (pos - R.out_capacity < A->dscratch_cap) A->dscratch[pos - R.out_capacity] = rec;
        }
        rejoin();
        S.found += nhit;
        return;
    }
    if (!nhit) return;
    if (S.nst + nhit > A->stage_cap) stage_flush(L, A0, S);
    // index of each result among the staged results of its request slot
    uint32_t idx = 0;
    uint64_t rem = hm;
    while (rem) {
        const uint32_t leader = (uint32_t)__ffsll((unsigned long long)rem) - 1u;
        const uint32_t sl = uniform((uint32_t)__shfl((int)slot, (int)leader));
        const uint64_t mm = ballot(hit && slot == sl);
        const uint32_t c = uniform((uint32_t)__builtin_amdgcn_readlane((int)S.rcnt, (int)sl));
        if (hit && slot == sl) idx = c + (uint32_t)__popcll(mm & below(lane));
        if (lane == sl) S.rcnt = c + (uint32_t)__popcll(mm);
        rem &= ~mm;
    }
    if (hit) {
        A->stage[S.sbase + S.nst + rank] = rec;
        A->stage_meta[S.sbase + S.nst + rank] = slot | (idx << 6);
    }
    rejoin();
    S.nst += nhit;
    S.found += nhit;
}

// Is this lane's bit set in m?
__device__ __forceinline__ bool in_mask(uint64_t m) {
    return __builtin_amdgcn_inverse_ballot_w64(m);
}

// Appends the pairs of the lanes of mask m to a queue.
__device__ __forceinline__ void enqueue(uint32_t* queue, uint32_t& n, uint64_t m, uint32_t pk) {
    if (in_mask(m)) queue[n + (uint32_t)__popcll(m & lanemask_lt())] = pk;
    rejoin();
    n += (uint32_t)__popcll(m);
}

// fmaxf / fminf as the one instruction they are: the compiler precedes it by
// one per operand that quiets signalling NaNs, of which none are made here.
__device__ __forceinline__ float max1(float a, float b) {
#if defined(__AMDGCN__)
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
#else
    return fmaxf(a, b);
#endif
}
__device__ __forceinline__ float min1(float a, float b) {
#if defined(__AMDGCN__)
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
#else
    return fminf(a, b);
#endif
}

// Closest-approach refinement of the FP32 filter, for a pair that passed the
// sphere and time tests: a lower bound, in FP32, on the smallest distance of
// the two moving points over their common extent.  The pair is dropped only
// when it exceeds d by more than the FP32 data and arithmetic can account
// for, so every pair the canonical FP64 evaluation accepts is kept.
//
// Query: position cq at time tq, velocity vq, clipped extent [qa, qb] rounded
// outwards; entry likewise (cl, vl, tl, [la, lb]).  Both positions moved to
// time 0 (oq = cq - vq tq, ol = cl - vl tl), on the common extent [a, b]
// (rounded outwards, so it contains the exact one), with tm = (a + b) / 2 and
// h = (b - a) / 2, the relative position is D(tau) = Dm + W tau for
// |tau| <= h, Dm = (oq - ol) + W tm, W = vq - vl.  Its distance from the
// origin is smallest at tau* = clamp(-Dm.W / |W|^2, -h, h); the pair is
// dropped when |D(tau)|^2 > R^2 for the computed tau, R = d + E.
//
// Error budget (u = 2^-24), with S0 = |cq|1 + |cl|1 + (|vq|1 + |vl|1)(|a| +
// |b| + |tq| + |tl| + 1) (L1 norms):
//  - rounding of the FP32 data to nearest (centres, velocities, mid times,
//    the positions moved to time 0) and the operations forming Dm, W, tm and h
//    move D(tau) by at most about 12 u S0, which also covers the FP64 rounding
//    of the canonical evaluation (its vertex clause accepts distances past d
//    by at most 0.7 u S0);
//  - the computed tau lies in [-h, h] whatever its error, so D(tau) is a
//    distance of the segment; that it is not the smallest one costs
//    |W|^2 (tau - tau*)^2 <= (9 u |Dm|)^2 (|tau - tau*| <= 9 u |Dm| / |W|
//    from the products' rounding, the reciprocal's 1 ulp and |tau*| <=
//    |Dm| / |W|), i.e. at most 9 u S0 of distance;
//  - |W|^2 may underflow when |W| < 2^-50; then D moves by at most 2 h |W|
//    over the whole extent, below the 2^-48 st that the query's part of E
//    always holds (qref_of).
// E = 2^-17 S = 128 u S with S = (sc_q + sc_l) + (sv_q + sv_l)(st_q + st_l) >=
// S0 (sc = |c|1, sv = |v|1, st = |a| + |b| + |t|, each side's own extent: |a| +
// |b| <= |qa| + |qb| + |la| + |lb| since a is qa or la and b is qb or lb), so
// E is at least six times the sum.  The relative rounding of R^2 and of
// |D|^2 (below 8 u each) is covered by the factor 1 + 2^-19.
//
// Range: tau is only as good as said while |W|^2 and its reciprocal are normal
// numbers and Dm.W is finite.  So a side whose speed sv reaches 2^60 (kFastest)
// has R infinite: a query's sphere is made unbounded (query_sphere32), which
// those past 1e18 < 2^60 are already, an entry's velocity infinite (motion32).
// Otherwise |W| < 2^61, hence |W|^2 < 2^122; each segment lies within 2^61 of
// the origin at all of the common extent, hence |Dm| < 2^63 up to its rounding
// of u S, which is small beside that where R^2 is finite (S < 2^81), so Dm.W and
// |D|^2 are finite too.  Where R is infinite nothing is dropped: the test is
// "value > bound", and an undefined tau (0 times infinity) becomes an end of the
// extent.
//
// One reciprocal and about 45 operations; the three separate bounds used
// before (triangle inequality, distance to the line of motion, the ends) took
// 75 and a square root for the same pairs kept.
__device__ __forceinline__ bool refine32(const QTime& f, const QRef& r, float olx, float oly,
                                         float olz, float vlx, float vly, float vlz, float la,
                                         float lb, float scl, float svl, float stl) {
    // sums of products are fused (fmaf): each has at most the rounding error
    // of the separate multiply and add it replaces
    const float a = max1(f.a, la), b = min1(f.b, lb);
    const float tm = 0.5f * (a + b), h = 0.5f * (b - a);
    const float wx = r.vx - vlx, wy = r.vy - vly, wz = r.vz - vlz;
    const float dx = fmaf(wx, tm, r.ox - olx);
    const float dy = fmaf(wy, tm, r.oy - oly);
    const float dz = fmaf(wz, tm, r.oz - olz);
    const float svq = (fabsf(r.vx) + fabsf(r.vy)) + fabsf(r.vz);
    const float R = fmaf(0x1p-17f, fmaf(svq + svl, r.st + stl, scl), r.d);
    const float R2 = (R * R) * (1.0f + 0x1p-19f);
    const float WW = fmaf(wz, wz, fmaf(wy, wy, wx * wx));
    const float DW = fmaf(dz, wz, fmaf(dy, wy, dx * wx));
    const float tau = min1(max1(-DW * __builtin_amdgcn_rcpf(WW), -h), h);
    const float px = fmaf(wx, tau, dx), py = fmaf(wy, tau, dy), pz = fmaf(wz, tau, dz);
    return !(fmaf(pz, pz, fmaf(py, py, px * px)) > R2);
}

// The query's refinement data, from its canonical data and filter record.
__device__ __forceinline__ QRef qref_of(const QCanon& q, const QF32& f) {
    QRef r;
    r.vx = __double2float_rn(q.vx);
    r.vy = __double2float_rn(q.vy);
    r.vz = __double2float_rn(q.vz);
    const float tq = __double2float_rn(0.5 * (q.aq + q.bq));
    r.ox = fmaf(-r.vx, tq, f.cx);
    r.oy = fmaf(-r.vy, tq, f.cy);
    r.oz = fmaf(-r.vz, tq, f.cz);
    r.st = ((fabsf(f.a32) + fabsf(f.b32)) + fabsf(tq)) + 1.0f;
    const float sc = (fabsf(f.cx) + fabsf(f.cy)) + fabsf(f.cz);
    // an unbounded sphere (stored centre 0): nothing is dropped
    r.d = f.R < INFINITY ? fmaf(0x1p-17f, fmaf(0x1p-30f, r.st, sc), __double2float_ru(q.d))
                         : INFINITY;
    return r;
}

// The candidate's side of the refinement: its position moved to time 0 and
// its parts of the error scale (see refine32).
struct ERef {
    float ox, oy, oz, vx, vy, vz;
    float sc, sv, st;
};
__device__ __forceinline__ ERef eref_of(float cx, float cy, float cz, float rad,
                                        const EntryV32& v, float ts, float te) {
    ERef e;
    e.vx = v.vx;
    e.vy = v.vy;
    e.vz = v.vz;
    e.ox = fmaf(-v.vx, v.tm, cx);
    e.oy = fmaf(-v.vy, v.tm, cy);
    e.oz = fmaf(-v.vz, v.tm, cz);
    // an unbounded sphere (stored centre 0): nothing is dropped, nor where the
    // velocity is infinite (motion32)
    e.sc = rad < INFINITY ? (fabsf(cx) + fabsf(cy)) + fabsf(cz) : INFINITY;
    e.sv = (fabsf(v.vx) + fabsf(v.vy)) + fabsf(v.vz);
    e.st = (fabsf(ts) + fabsf(te)) + fabsf(v.tm);
    return e;
}

// FP32 form: the closest-approach refinement (refine32) of the last
// min(qn, 64) queued sphere survivors, one per lane; the pairs it keeps go to
// the refined queue, which is evaluated when it holds 64.
__device__ __forceinline__ void refine_step(WaveLDS& L, ItemState& S, const DistArgs& A0) {
    const uint32_t lane = fresh_lane();
    const ArgsPtr A = cold_args(A0);
    const uint32_t cnt = min(S.qn, (uint32_t)kWave);
    wave_sync();
    S.qn -= cnt;
    const bool act = lane < cnt;
    const uint32_t pk = act ? L.queue[S.qn + lane] : 0u;
    wave_sync();
    bool keep = false;
    if (act) {
        const uint32_t ql = pk & (kWave - 1);
        const uint32_t i = S.c0 + (pk >> 6);
        const EntryF32 e = A->I.e32[i];
        const EntryV32 v = A->I.ev32[i];
        const ERef x = eref_of(e.cx, e.cy, e.cz, e.r, v, e.ts, e.te);
        keep = refine32(L.qt[ql], L.qref[ql], x.ox, x.oy, x.oz, x.vx, x.vy, x.vz, e.ts, e.te, x.sc,
                        x.sv, x.st);
    }
    enqueue(L.rq, S.rqn, ballot(keep), pk);
}

// The request slot of each query of the group: the first lane of the group
// with the same request.
__device__ __forceinline__ uint32_t request_slots(bool has, uint32_t r) {
    const uint32_t lane = __lane_id();
    uint32_t slot = lane;
    uint64_t rem = ballot(has);
    while (rem) {
        const uint32_t leader = (uint32_t)__ffsll((unsigned long long)rem) - 1u;
        const uint32_t rr = uniform((uint32_t)__shfl((int)r, (int)leader));
        const uint64_t mm = ballot(has && r == rr);
        if ((mm >> lane) & 1ull) slot = leader;
        rem &= ~mm;
    }
    return slot;
}

// Value of v in lane j (wave-uniform j): a register read, no memory access.
__device__ __forceinline__ float lane_val(float v, uint32_t j) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), (int)j));
}

// A candidate as a lane holds it; its motion with kRef other than queued.
struct Cand {
    float cx, cy, cz, r, ts, te;
    EntryV32 v;
};

// Candidate `lane` of a block; one outside the chunk gets an empty time extent
// (it never passes).
template <bool kMotion>
__device__ __forceinline__ Cand load_cand(const DistArgs& A, const ItemState& S, uint32_t blk) {
    const uint32_t cand = (blk << kBoxShift) + __lane_id();
    const bool valid = cand >= S.c0 && cand < S.c1;
    const uint32_t i = valid ? cand : S.c1 - 1;
    const EntryF32 e = A.I.e32[i];
    EntryV32 v = {0.f, 0.f, 0.f, 0.f};
    if (kMotion) v = A.I.ev32[i];
    return {e.cx, e.cy, e.cz, e.r, valid ? e.ts : INFINITY, valid ? e.te : -INFINITY, v};
}

// Without block boxes: the first query of mask mk (not 0) that has lanes whose
// candidate passes its sphere test and, with kTime, its time test: its number in
// j, those lanes as the result; 0 if no query has.  Takes it and those before it
// from mk.
//
// A block's entries lie anywhere, and where most queries have no survivors among
// them this loop is all that a query costs.  kAhead at a time: their records are
// read together, and the loop's scalar steps are shared (past the last one, the
// first again).  Taken where at most one query in kAhead of the last block had
// survivors, since the tests past one that has some are in vain.  200,000 uniform
// segments on the temporal layout: kernel 268 us with the older walk, a copy of the
// code per combination of time test and partial ranges, 447 with the one-query steps
// that block boxes take, 303 two at a time, 275 four.
constexpr uint32_t kAhead = 4;
template <bool kTime>
__device__ __forceinline__ uint64_t next_query(const WaveLDS& L, const Cand& c, uint64_t& mk,
                                               uint32_t& j) {
    constexpr int kN = (int)kAhead;
    for (;;) {
        uint64_t rest[kN + 1];
        uint32_t jn[kN];
        QSphere q[kN];
        QTime t[kN];
        rest[0] = mk;
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            jn[i] = (uint32_t)__builtin_ctzll(i && !rest[i] ? mk : rest[i]);
            rest[i + 1] = rest[i] & (rest[i] - 1u);
            q[i] = L.qs[jn[i]];
            if (kTime) t[i] = L.qt[jn[i]];
        }
        uint64_t m[kN], any = 0;
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            m[i] = ballot(sphere_pass(q[i].cx, q[i].cy, q[i].cz, q[i].R, c.cx, c.cy, c.cz, c.r));
            if (kTime) m[i] &= ballot(t[i].a < c.te) & ballot(c.ts < t[i].b);
            any |= m[i];
        }
        if (any) {
            j = jn[kN - 1];
            mk = rest[kN];
            uint64_t got = m[kN - 1];
#pragma unroll
            for (int i = kN - 2; i >= 0; --i)
                if (m[i]) {
                    j = jn[i];
                    mk = rest[i + 1];
                    got = m[i];
                }
            return got;
        }
        mk = rest[kN];
        if (!mk) {
            j = jn[0];
            return 0;
        }
    }
}

// Takes queued pairs on while a queue holds at least `from` of them (64 inside
// an item, 1 at its end): refinement, then FP64 evaluation.
__device__ __forceinline__ void take_queued(WaveLDS& L, ItemState& S, const DistArgs& A,
                                            uint32_t from) {
    while (S.qn >= from || S.rqn >= from) {
        if (S.qn >= from && S.rqn < kWave) refine_step(L, S, A);
        if (S.rqn >= from) drain(L, S, A);
    }
}

// FP32 form: the wave takes the chunk kCpl * 64 candidates at a time (kCpl
// per lane, coalesced vector loads issued together, tiles aligned to the
// 64-entry blocks).  Lane j holds the box of query j and the box of one of the
// next 64 blocks (broadcast from its registers by readlane; read by scalar
// loads, every read of LDS waited for them as well).  Each block's box is
// first tested against every query, and only the queries that pass are tested
// against the block's entries, one after another (a scalar walk over the
// mask), their records read from the wave's LDS copy of the group at
// wave-uniform addresses: the sphere and time test of every lane's candidate,
// then the closest-approach refinement of the pairs that passed, here or later
// from the queue (kRef); pairs that stay go on to the FP64 evaluation 64 at a
// time.  (The candidates' motion loaded only at a block's first refinement
// cost twelve register copies per query; candidates read again after an
// evaluation instead of held, a stall each.)  Queries whose candidate range
// covers a block only in part (`part`, from the lanes' qlo and qhi; none when
// `uni`) have their bounds checked per pair.  When every candidate of the bucket overlaps every
// query of the group in time (all_overlap), the per-pair time test is skipped:
// exact, since the outward-rounded FP32 times then overlap as well.
//
// One copy of each step per block of the tile, with the item's end as part of
// the last block: a copy per combination of partial ranges, skipped time test
// and item end made 70 KB of code and 22 to 103 spilled registers.
//
// Bound by instructions issued (about 23 vector and 26 scalar ones per query
// and block, 66 and 33 where pairs are refined), not by memory.  The kernel,
// before (queued refinement with three bounds, tile 4) and with this walk (one
// bound, in the walk, tile 2): two particle sets close by, 4.4 million
// evaluations, 1577 -> 904 us; the same overlapping, 171 million, 6507 -> 4438;
// 1 M uniform segments in a batch 145 -> 148; 89 k evaluations of a self-join
// of 1 M, 240 -> 231; 8000 items of dense walks 165 -> 143.
template <int kCpl, int kRef, bool kCull>
__device__ __forceinline__ void scan_chunk_fp32(WaveLDS& L, const DistArgs& A, ItemState& S,
                                                const Box32& qbox, uint32_t qlo, uint32_t qhi,
                                                bool uni, bool all_overlap) {
    const uint32_t lane = __lane_id();
    const uint64_t has_mask = ~0ull >> (kWave - S.nq);
    const uint32_t blk0 = S.c0 >> kBoxShift, blk1 = (S.c1 - 1) >> kBoxShift;
    Box32 wbox = {};  // box of block wb + lane
    uint32_t wb = blk0 - kWave;
    for (uint32_t tile = blk0; tile <= blk1; tile += kCpl) {
        Cand tc[kCpl];
#pragma unroll
        for (int k = 0; k < kCpl; ++k)
            tc[k] = load_cand<kRef != TDS_REFINE_QUEUED>(A, S, tile + k);
        if (kCull && tile + kCpl - 1 - wb >= kWave) {
            wb = tile;
            wbox = A.I.bbox[min(wb + lane, blk1)].b;
        }
#pragma unroll
        for (int k = 0; k < kCpl; ++k) {
            const uint32_t blk = tile + k;
            if (blk > blk1) break;
            const uint32_t b0 = blk << kBoxShift;  // first entry of the block
            uint64_t mk = has_mask, part = 0;
            if (!uni) {
                mk &= ballot(qlo < b0 + kWave) & ballot(qhi > b0);
                part = mk & ~(ballot(qlo <= b0) & ballot(qhi >= b0 + kWave));
            }
            if (kCull && mk) {
                const uint32_t l = blk - wb;
                const Box32 box = {lane_val(wbox.lx, l), lane_val(wbox.ly, l),
                                   lane_val(wbox.lz, l), lane_val(wbox.hx, l),
                                   lane_val(wbox.hy, l), lane_val(wbox.hz, l)};
                // box_overlap, a mask per comparison
                mk &= ballot(box.lx <= qbox.hx) & ballot(qbox.lx <= box.hx) &
                      ballot(box.ly <= qbox.hy) & ballot(qbox.ly <= box.hy) &
                      ballot(box.lz <= qbox.hz) & ballot(qbox.lz <= box.hz);
                S.btests += S.nq;
            }
            // at the item's end what is queued is taken on to the last pair
            const uint32_t from = blk == blk1 ? 1u : (uint32_t)kWave;
            if (!mk && from == kWave) continue;
            const uint32_t nv = min(S.c1, b0 + kWave) - max(S.c0, b0);
            S.ftests += (uint64_t)__popcll(mk) * (uint64_t)nv;
            const uint32_t cand = b0 + lane;
            const uint32_t code = (cand - S.c0) << 6;  // used where the candidate is in the chunk
            // the time test can be dropped only on full slots
            const bool timed = !all_overlap || nv < kWave;
            const Cand c = tc[k];
            const ERef ex = eref_of(c.cx, c.cy, c.cz, c.r, c.v, c.ts, c.te);
            // query j's survivors among the lanes go on (with block boxes most queries
            // have some, and asking for that before the range cost two particle sets
            // close by 943 -> 961 us)
            const auto pass = [&](uint32_t j, uint64_t m) {
                if (!kCull) S.hits += kAhead;
                if ((part >> j) & 1ull) {
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)qlo, (int)j);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)qhi, (int)j);
                    m &= ballot(cand >= lo) & ballot(cand < hi);
                }
                if (!m) return;
                if (kRef == TDS_REFINE_QUEUED) {
                    enqueue(L.queue, S.qn, m, code | j);
                    return;
                }
                const bool keep = refine32(L.qt[j], L.qref[j], ex.ox, ex.oy, ex.oz, ex.vx, ex.vy,
                                           ex.vz, c.ts, c.te, ex.sc, ex.sv, ex.st);
                enqueue(L.rq, S.rqn, m & ballot(keep), code | j);
            };
            const bool few = !kCull && (int32_t)S.hits <= 0;
            if (!kCull) S.hits = 0u - (uint32_t)__popcll(mk);
            for (;;) {
                if (few) {
                    while (mk && max(S.qn, S.rqn) < kWave) {
                        uint32_t j;
                        const uint64_t m =
                            timed ? next_query<true>(L, c, mk, j) : next_query<false>(L, c, mk, j);
                        if (m) pass(j, m);
                    }
                } else {
                    while (mk && max(S.qn, S.rqn) < kWave) {
                        const uint32_t j = (uint32_t)__builtin_ctzll(mk);
                        mk &= mk - 1u;
                        const QSphere q = L.qs[j];
                        uint64_t m =
                            ballot(sphere_pass(q.cx, q.cy, q.cz, q.R, c.cx, c.cy, c.cz, c.r));
                        if (timed) {
                            const QTime t = L.qt[j];
                            m &= ballot(t.a < c.te) & ballot(c.ts < t.b);
                        }
                        if (kCull || m) pass(j, m);
                    }
                }
                take_queued(L, S, A, mk ? (uint32_t)kWave : from);
                if (!mk) break;
            }
        }
    }
    wave_sync();
}

// Plain FP64 form: one query segment per lane, every candidate of the chunk
// streamed through scalar loads, each asked for one candidate ahead, and
// tested with the canonical predicate.
__device__ __forceinline__ void scan_chunk_fp64(WaveLDS& L, const DistArgs& A, ItemState& S,
                                                const QCanon& q, uint32_t qlo, uint32_t qhi,
                                                bool uni) {
    ConstE64 ce = (ConstE64)(A.I.e64);
    f64x4 n0 = ce[2 * S.c0], n1 = ce[2 * S.c0 + 1];
    for (uint32_t i = S.c0; i <= S.c1; ++i) {
        uint32_t from = 1;
        if (i < S.c1) {
            from = kWave;
            const f64x4 e0 = n0, e1 = n1;  // x, y, z, vx | vy, vz, ts, te
            const uint32_t i1 = min(i + 1, S.c1 - 1);
            n0 = ce[2 * i1];
            n1 = ce[2 * i1 + 1];
            bool pass = canon_eval<false>(q, e0[0], e0[1], e0[2], e0[3], e1[0], e1[1], e1[2],
                                          e1[3], nullptr, nullptr);
            if (!uni) pass = pass & (i >= qlo) & (i < qhi);
            const uint64_t m = ballot(pass);
            if (!m) continue;
            enqueue(L.rq, S.rqn, m, ((i - S.c0) << 6) | __lane_id());
        }
        if (S.rqn >= from) take_queued(L, S, A, from);
    }
    wave_sync();
}

template <int kPrec, int kCplT, int kRef, bool kCull>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_distance(DistArgs A) {
    __shared__ WaveLDS wl[kWavesPerBlock];
    const uint32_t wid = uniform(threadIdx.x / kWave);
    WaveLDS& L = wl[wid];
    const uint32_t lane = __lane_id();
    uint64_t tests = 0, evals_total = 0, ftests = 0, btests = 0;
    uint32_t flushes = 0;  // stage flushes at the end of an item (direct output: reservations)
    // direct output (see DistArgs): the wave's open reservation, at first the
    // chunk of its number or none
    const uint64_t dfirst =
        A.dir_given ? (uint64_t)(blockIdx.x * kWavesPerBlock + wid) * A.dir_chunk : 0ull;
    uint64_t dpos = dfirst, dend = dfirst + (A.dir_given ? A.dir_chunk : 0u);
    uint32_t dg = 1;
    uint64_t found_total = 0;
    // what stays staged between items (keep): nst results, request r's number of
    // them at queue[r], since the queue is empty then (in a register it was spilled,
    // one more trip to memory per item)
    uint32_t nst = 0;
    L.queue[lane] = 0u;
    uint32_t hits = 0;
    // all items of the search, unless a range is given (incremental passes)
    const uint32_t item_end = (A.item_end == 0xFFFFFFFFu)
                                  ? uniform(min(A.hdr->n_items, A.desc->item_cap))
                                  : A.item_end;
    // Items [item_begin, item_end) are split into 8 contiguous parts, one
    // per XCD (workgroups are dispatched to the XCDs round-robin, so
    // workgroup b runs on XCD b mod 8; consecutive items share buckets, hence
    // candidate ranges, which then stay under one XCD's L2).  Each wave first
    // takes one item of its XCD's part statically (item p0 + its index among
    // the XCD's waves: no atomic on the critical path of light searches,
    // where this round covers every item).  Items beyond that round are
    // taken dynamically from the part's counter, and a wave whose part is
    // used up takes from the next parts: item costs vary by orders of
    // magnitude where results cluster (a static deal left some XCDs idle for
    // more than half of a galaxy search).  The next item is asked for before
    // the current one's last evaluations, which hide most of the atomic's
    // latency (asked for at the item's start, it is bound to a wave that may
    // be busy for long: 8.6 against 6.4 ms on galaxy), and the counters are read
    // before an increment only by a wave that looks for another part: reading
    // all eight per item, next to the atomics, took the whole chip 30 ns per item
    // (1.9e6 items of 64 candidates: 57 ms).
    // The 9,600 items of three uniform1m searches: 279 us that way, 197 asked
    // ahead, 145 with the line that says all parts are used up, 137 dealt
    // statically.
    const uint64_t n_it = item_end > A.item_begin ? item_end - A.item_begin : 0u;
    // this wave's result stage
    const uint64_t sbase =
        (uint64_t)(blockIdx.x * kWavesPerBlock + wid) * A.stage_cap;
    const uint32_t ng = min(gridDim.x, kXcds);
    const uint32_t grp = blockIdx.x % ng;
    const uint32_t gw = (blockIdx.x / ng) * kWavesPerBlock + wid;
    // waves of the workgroups on XCD x
    auto waves_of = [&](uint32_t x) {
        return ((gridDim.x - x + ng - 1) / ng) * (uint32_t)kWavesPerBlock;
    };
    auto part_lo = [&](uint32_t x) { return n_it * x / ng; };
    // static deal (chosen per launch): every item round-robin over the
    // XCD's waves, no counter at all
    const bool stat = A.deal == TDS_DEAL_STATIC;
    bool dyn = false;  // does any part hold more items than its XCD has waves?
    if (!stat)
        for (uint32_t x = 0; x < ng; ++x) dyn = dyn || part_lo(x + 1) - part_lo(x) > waves_of(x);
    uint64_t k = part_lo(grp) + gw;
    bool have = k < part_lo(grp + 1);
    uint32_t xs = grp;  // the part dynamic items are taken from
    uint64_t ahead = 0;  // lane 0: its next number, asked for during the current item
    bool asked = false;
    for (;;) {
        if (!have) {
            if (!dyn) break;
            if (asked) {
                asked = false;
                const uint64_t v = lane0_64(ahead);
                const uint64_t ps = part_lo(xs) + waves_of(xs), pe = part_lo(xs + 1);
                if (ps + v < pe) {
                    k = ps + v;
                    have = true;
                }
            }
            // the next dynamic item: the parts' counters are read at once,
            // one part per lane in rotation from part xs, and the first part
            // with items left past its static round is taken from; losing
            // the race for a part's last items exhausts that part, so this
            // ends after at most ng + 1 rounds
            // (a wave that finds all parts used up says so on a line of its
            // own, which the other waves look at first)
            unsigned long long* done = A.dyn_ctr + (size_t)kCtrDone * kCtrStride;
            if (!have) {
                uint64_t over = 0;
                if (lane == 0)
                    over = __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (lane0_64(over)) break;
            }
            for (uint32_t round = 0; round <= ng && !have; ++round) {
                bool avail = false;
                if (lane < ng) {
                    const uint32_t x = (xs + lane) % ng;
                    const uint64_t ps = part_lo(x) + waves_of(x), pe = part_lo(x + 1);
                    if (ps < pe) {
                        const uint64_t v = __hip_atomic_load(A.dyn_ctr + (size_t)x * kCtrStride,
                                                             __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                        avail = ps + v < pe;
                    }
                }
                const uint64_t am = ballot(avail);
                if (!am) {  // every part is used up (every lane stores the same)
                    __hip_atomic_store(done, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                xs = (xs + (uint32_t)__ffsll((unsigned long long)am) - 1u) % ng;
                uint64_t v = 0;
                if (lane == 0) v = atomicAdd(A.dyn_ctr + (size_t)xs * kCtrStride, 1ull);
                v = lane0_64(v);
                const uint64_t ps = part_lo(xs) + waves_of(xs), pe = part_lo(xs + 1);
                if (ps + v < pe) {
                    k = ps + v;
                    have = true;
                }
            }
            if (!have) break;
        }
        have = false;
        const uint32_t it = A.item_begin + (uint32_t)k;
        const uint32_t b = uniform(A.item_bucket[it]);
        const BucketInfo bi = A.binfo[b];
        const uint32_t local = it - bi.item0;
        // chunk-major inside a bucket: the groups of one chunk are adjacent
        // items, so the waves of an XCD, which work through a contiguous
        // part of the item list, share the chunk's records in their L2
        const uint32_t ngr = (bi.count + kWave - 1) / kWave;
        const uint32_t c = local / ngr;
        const uint32_t g = local - c * ngr;
        ItemState S;
        S.sbase = sbase;
        S.nq = uniform(min((uint32_t)kWave, bi.count - g * kWave));
        const uint64_t base = (uint64_t)(bi.lo & ~(uint32_t)(kWave - 1)) + (uint64_t)c * bi.clen;
        S.c0 = uniform((uint32_t)max((uint64_t)bi.lo, base));
        S.c1 = uniform((uint32_t)min((uint64_t)bi.hi, base + bi.clen));
        S.qbase = uniform(bi.start + g * kWave);
        S.qn = 0;
        S.rqn = 0;
        S.evals = 0;
        S.found = 0;
        S.nst = nst;
        S.ftests = 0;
        S.btests = 0;
        S.hits = hits;
        S.dpos = dpos;
        S.dend = dend;
        S.dg = dg;
        S.nres = 0;
        // the group's data.  A lane without a query: an empty box (it never
        // passes a block), an unbounded window and range (it never stands in
        // the way of the whole-group shortcuts) and, in FP64, an empty extent
        // (never a member)
        const bool has = lane < S.nq;
        QF32 f = {0.f, 0.f, 0.f, 0.f, -INFINITY, INFINITY, 0u, 0xFFFFFFFFu,
                  {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY}, 0u, 0.f};
        QEval e = {{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0}, 0u, 0u};
        if (has) {
            const uint32_t q = A.qsorted[S.qbase + lane];
            f = A.qf[q];
            e = A.qev[q];
        }
        // does every query of the group cover the whole chunk?
        const bool all_cover = ballot(f.lo <= S.c0 && f.hi >= S.c1) == ~0ull;
        S.qr = f.req;
        S.rslot = A.keep ? f.req : request_slots(has, f.req);
        wave_sync();
        L.qe[lane] = e;
        if (kPrec == TDS_PREC_FP32_RECHECK) {
            L.qs[lane] = QSphere{f.cx, f.cy, f.cz, f.R};
            L.qt[lane] = QTime{f.a32, f.b32};
            L.qref[lane] = qref_of(e.c, f);
        }
        S.rcnt = L.queue[lane];
        wave_sync();
        if (kPrec == TDS_PREC_FP32_RECHECK)
            scan_chunk_fp32<kCplT, kRef, kCull>(
                L, A, S, f.box, f.lo, f.hi, all_cover,
                (ballot((double)f.a32 < bi.tmin_te) & ballot(bi.tmax_ts < (double)f.b32)) == ~0ull);
        else scan_chunk_fp64(L, A, S, e.c, f.lo, f.hi, all_cover);
        if (dyn) {
            if (lane == 0) ahead = atomicAdd(A.dyn_ctr + (size_t)xs * kCtrStride, 1ull);
            rejoin();
            asked = true;
        }
        // the item's results get their positions where the next item's group has
        // other request slots
        if (!A.keep && S.nst) {
            stage_flush(L, A, S);
            ++flushes;
        }
        nst = S.nst;
        L.queue[lane] = S.rcnt;
        dpos = S.dpos;
        dend = S.dend;
        dg = S.dg;
        flushes += S.nres;
        found_total += S.found;
        hits = S.hits;
        tests += (uint64_t)(S.c1 - S.c0) * S.nq;
        ftests += (kPrec == TDS_PREC_FP64) ? (uint64_t)(S.c1 - S.c0) * S.nq : S.ftests;
        btests += S.btests;
        evals_total += S.evals;
        if (A.item_count && lane == 0) A.item_count[it] = S.found;
        rejoin();
        if (stat) {
            // the wave's next item of its part
            k += waves_of(grp);
            have = k < part_lo(grp + 1);
        }
    }
    if (A.direct && lane == 0) {
        // the wave's last reservation (~0: none) and, where the fill does not
        // count them, its results
        const uint32_t size = dg * A.dir_chunk;
        A.dlast[blockIdx.x * kWavesPerBlock + wid] =
            dend ? pack_last((dend - size) / A.dir_chunk, dg, size - (uint32_t)(dend - dpos))
                 : ~0ull;
        if (!A.dir_given && found_total)
            atomicAdd(&A.rc[0].count, (unsigned long long)found_total);
    }
    if (A.keep && !A.direct && !A.by_order) {
        // what the workgroup's waves still have staged: lane r adds up request r's
        // results, and one wave reserves for all
        if (nst) ++flushes;
        const uint32_t rcnt = L.queue[lane];
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (uint32_t w = 0; w < (uint32_t)kWavesPerBlock; ++w) {
            const uint32_t c = wl[w].queue[lane];
            before += w < wid ? c : 0u;
            all += c;
        }
        unsigned long long* s_base = reinterpret_cast<unsigned long long*>(wl[0].rq);
        if (wid == 0) {
            unsigned long long base = 0;
            if (all) base = atomicAdd(&A.rc[lane].count, (unsigned long long)all);
            s_base[lane] = base;
        }
        __syncthreads();
        wave_sync_mem();
        stage_copy(cold_args(A), sbase, nst, lane, rcnt, s_base[lane] + before);
    }
    // the first reservation counts as one that was made, once it holds a result
    if (A.direct && A.dir_given && !(dpos == dfirst)) ++flushes;
    // per-workgroup counters (folded into the header by k_stats_fold), each
    // wave's in the front of its own LDS, which it no longer uses
    wave_sync();
    if (lane == 0) {
        BlockStats& w = *reinterpret_cast<BlockStats*>(wl[wid].queue);
        w.tests = tests;
        w.evals = evals_total;
        w.ftests = ftests;
        w.btests = btests;
        w.flushes = flushes;
        w.pad[0] = w.pad[1] = w.pad[2] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        BlockStats b = *reinterpret_cast<const BlockStats*>(wl[0].queue);
        for (int k = 1; k < kWavesPerBlock; ++k) {
            const BlockStats& w = *reinterpret_cast<const BlockStats*>(wl[k].queue);
            b.tests += w.tests;
            b.evals += w.evals;
            b.ftests += w.ftests;
            b.btests += w.btests;
            b.flushes += w.flushes;
        }
        A.bstats[blockIdx.x] = b;
    }
}

// ------------------------------------------------------------ host side

template <typename T>
int grow(T** p, size_t* cap, size_t need) {
    if (*cap >= need && *p) return TDS_OK;
    dfree(*p);
    *p = nullptr;
    *cap = 0;
    TDS_TRY(dmalloc(p, need));
    *cap = need;
    return TDS_OK;
}

}  // namespace

namespace {
struct PinPool {
    std::mutex mu;
    PinBlock* idle[kPinPool];
    size_t n = 0;
};
// never destroyed: at the program's end the runtime may be gone first
PinPool& pin_pool() {
    alignas(PinPool) static unsigned char mem[sizeof(PinPool)];
    static PinPool* pool = new (mem) PinPool();
    return *pool;
}
}  // namespace

int acquire_pin(PinBlock** b) {
    if (*b) return TDS_OK;
    {
        PinPool& P = pin_pool();
        std::lock_guard<std::mutex> l(P.mu);
        if (P.n) {
            *b = P.idle[--P.n];
            return TDS_OK;
        }
    }
    void* p = nullptr;
    TDS_HIP(hipHostMalloc(&p, sizeof(PinBlock), hipHostMallocPortable));
    *b = static_cast<PinBlock*>(p);
    return TDS_OK;
}

void release_pin(PinBlock* b) {
    if (!b) return;
    {
        PinPool& P = pin_pool();
        std::lock_guard<std::mutex> l(P.mu);
        if (P.n < kPinPool) {
            P.idle[P.n++] = b;
            return;
        }
    }
    (void)hipHostFree(b);
}

Workspace::~Workspace() {
    for (void* p : {(void*)qsorted, (void*)qkey, (void*)qslot, (void*)qf, (void*)qev, (void*)qstage,
                    (void*)qtraj_stage, (void*)ctl, (void*)b_count,
                    (void*)b_hi, (void*)b_start, (void*)b_nch,
                    (void*)binfo, (void*)item_bucket, (void*)item_count, (void*)res,
                    (void*)bstats, (void*)dyn_ctr,
                    (void*)dlast, (void*)fill_s, (void*)fill_d, (void*)fill_dstart,
                    (void*)fill_plan})
        dfree(p);
    if (ctl_host) (void)hipHostFree(ctl_host);
    release_block(&stage_block);
    release_pin(pin);  // nothing uses it: the releases above waited for the device
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
}

int ws_init(Workspace* w) {
    TDS_TRY(dmalloc(&w->b_count, kMaxBuckets));
    TDS_TRY(dmalloc(&w->b_hi, kMaxBuckets));
    TDS_TRY(dmalloc(&w->b_start, kMaxBuckets));
    TDS_TRY(dmalloc(&w->b_nch, kMaxBuckets));
    TDS_TRY(dmalloc(&w->binfo, kMaxBuckets));
    TDS_TRY(dmalloc(&w->bstats, kMaxDistBlocks));
    TDS_TRY(dmalloc(&w->dyn_ctr, (size_t)kCtrSlots * kCtrStride));
    TDS_HIP(hipEventCreate(&w->ev0));
    TDS_HIP(hipEventCreate(&w->ev1));
    return ws_reserve(w, 0, 1);
}

namespace {

// Byte offsets in the control block for r_cap requests (every part starts
// on a 64-B boundary: the four structures are multiples of 16 B, and
// BatchDesc and SearchHeader are 64-B aligned).
struct CtlLayout {
    size_t req, hdr, ctr, bytes;
};

CtlLayout ctl_layout(size_t r_cap) {
    auto up = [](size_t v) { return (v + 63) / 64 * 64; };
    CtlLayout L;
    L.req = up(sizeof(BatchDesc));
    L.hdr = up(L.req + r_cap * sizeof(Request));
    L.ctr = up(L.hdr + sizeof(SearchHeader));
    L.bytes = up(L.ctr + r_cap * sizeof(ReqCounter));
    return L;
}

}  // namespace

int ws_upload(Workspace* w, uint32_t nreq, hipStream_t s) {
    const CtlLayout L = ctl_layout(w->r_cap);
    TDS_HIP(hipMemcpyAsync(w->ctl, w->ctl_host, L.req + nreq * sizeof(Request),
                           hipMemcpyHostToDevice, s));
    return TDS_OK;
}

int ws_download(Workspace* w, uint32_t nreq, hipStream_t s) {
    const CtlLayout L = ctl_layout(w->r_cap);
    TDS_HIP(hipMemcpyAsync(w->ctl_host + L.hdr, w->ctl + L.hdr,
                           L.ctr - L.hdr + nreq * sizeof(ReqCounter), hipMemcpyDeviceToHost, s));
    return TDS_OK;
}

int ws_reserve(Workspace* w, size_t nq, size_t nreq) {
    if (w->q_cap < nq || !w->qf) {
        for (void* p : {(void*)w->qsorted, (void*)w->qkey, (void*)w->qslot, (void*)w->qf,
                        (void*)w->qev})
            dfree(p);
        w->qf = nullptr;
        w->qev = nullptr;
        w->qkey = w->qslot = w->qsorted = nullptr;
        w->q_cap = 0;
        TDS_TRY(dmalloc(&w->qsorted, nq));
        TDS_TRY(dmalloc(&w->qkey, nq));
        TDS_TRY(dmalloc(&w->qslot, nq));
        TDS_TRY(dmalloc(&w->qf, nq));
        TDS_TRY(dmalloc(&w->qev, nq));
        w->q_cap = nq;
    }
    if (w->r_cap < nreq || !w->ctl) {
        dfree(w->ctl);
        if (w->ctl_host) (void)hipHostFree(w->ctl_host);
        w->ctl = w->ctl_host = nullptr;
        w->desc = w->desc_host = nullptr;
        w->req = w->req_host = nullptr;
        w->hdr = w->hdr_host = nullptr;
        w->req_ctr = w->rc_host = nullptr;
        w->r_cap = 0;
        const size_t r_cap = std::max<size_t>(nreq, 16);
        const CtlLayout L = ctl_layout(r_cap);
        TDS_TRY(dmalloc(&w->ctl, L.bytes));
        TDS_HIP(hipHostMalloc((void**)&w->ctl_host, L.bytes, hipHostMallocDefault));
        std::memset(w->ctl_host, 0, L.bytes);
        for (int side = 0; side < 2; ++side) {
            char* base = side ? w->ctl_host : w->ctl;
            BatchDesc* desc = reinterpret_cast<BatchDesc*>(base);
            Request* req = reinterpret_cast<Request*>(base + L.req);
            SearchHeader* hdr = reinterpret_cast<SearchHeader*>(base + L.hdr);
            ReqCounter* ctr = reinterpret_cast<ReqCounter*>(base + L.ctr);
            (side ? w->desc_host : w->desc) = desc;
            (side ? w->req_host : w->req) = req;
            (side ? w->hdr_host : w->hdr) = hdr;
            (side ? w->rc_host : w->req_ctr) = ctr;
        }
        w->r_cap = r_cap;
    }
    return TDS_OK;
}

namespace {
uint32_t launch_blocks(uint32_t grid_waves);
size_t stage_total(uint32_t grid_waves);
}  // namespace

int ws_reserve_stage(Workspace* w, uint32_t grid_waves) {
    const size_t need = stage_total(grid_waves);
    const uint32_t waves = launch_blocks(grid_waves) * kWavesPerBlock;
    if (w->stage_waves < waves || !w->dlast) {
        for (void* p : {(void*)w->dlast, (void*)w->fill_s, (void*)w->fill_d,
                        (void*)w->fill_dstart, (void*)w->fill_plan})
            dfree(p);
        w->dlast = w->fill_s = w->fill_d = w->fill_dstart = w->fill_plan = nullptr;
        w->stage_waves = 0;
        TDS_TRY(dmalloc(&w->dlast, waves));
        if (waves > kFillWaves) {  // k_fill keeps its plan in LDS
            TDS_TRY(dmalloc(&w->fill_s, (size_t)waves + 2));
            TDS_TRY(dmalloc(&w->fill_d, (size_t)waves + 1));
            TDS_TRY(dmalloc(&w->fill_dstart, waves));
            TDS_TRY(dmalloc(&w->fill_plan, 4));
        }
        w->stage_waves = waves;
    }
    if (w->stage_recs >= need && w->stage) return TDS_OK;
    release_block(&w->stage_block);
    w->stage = nullptr;
    w->stage_meta = nullptr;
    w->stage_recs = 0;
    DeviceArena a;
    a.add(&w->stage, need);
    a.add(&w->stage_meta, need);
    TDS_TRY(a.alloc(&w->stage_block));
    w->stage_recs = need;
    return TDS_OK;
}

namespace {

// 4 waves per SIMD on all 256 CUs (the occupancy the distance kernel's register
// use allows).
constexpr uint32_t kDefaultWaves = 256 * 4 * 4;

uint32_t bucket_shift(uint32_t m) {
    uint32_t shift = 0;
    while ((((uint64_t)m * kSpanClasses - 1) >> shift) >= kMaxBuckets) ++shift;
    return shift;
}

uint32_t bucket_count(uint32_t m) {
    return (uint32_t)((((uint64_t)m * kSpanClasses - 1) >> bucket_shift(m)) + 1);
}

// Waves of a launch that run at a time, at most those of the default grid: items
// are not made for more (8,192 waves, dense walks: 172 us with chunks for 4,096, 236
// with chunks for 8,192; uniform walks 166 and 212).
uint32_t busy_waves(uint32_t grid_waves) {
    return std::min(launch_blocks(grid_waves) * kWavesPerBlock, kDefaultWaves);
}

// Candidates per work item, chosen by the item count (k_bucket_scan): from
// 4096 down to 512 (FP32 form) or 512 down to 128 (FP64 form), until there
// are 3 / 2 items per wave.  Small searches are bound by the longest item:
// with 4096 -> 512 the kernel takes 22 -> 12 us (201 -> 1005 items), 63 -> 26
// (98 -> 392), 95 -> 32 (ragged, 2806 items), FP64 with 512 -> 128 240 -> 200
// (2000 -> 8000).  With enough items each costs its own start, 8 to 10 us of
// latency: 512 instead of 4096 takes 225 instead of 148 us at 9600 items and
// 306 instead of 231 at 16000; 4800 items are better split (159 -> 143).
uint32_t chunk_levels(int prec, uint32_t chunk) {
    if (!(chunk & kChunkAuto)) return 1;
    return prec == TDS_PREC_FP64 ? 3 : 4;
}
uint32_t item_target(uint32_t grid_waves) {
    return busy_waves(grid_waves) * 3 / 2;
}

// Items that every wave has one of.  Where the entries of a bucket begin and end at
// times of their own, or a bin is much wider than a segment is long, most of an
// item's pairs fail the time test, items are light and alike, and a second round of
// smaller ones costs more than it evens out: walks with start times of their own,
// call at 2829, 5150 and 9786 items 163, 190 and 199 us, at 3071 and 6043 101 and
// 123 (but the first halving is made: 2833, 5420 and 10208 items 151, 144 and 150);
// 40 trajectories in 19 bins, kernel at 858, 1716, 3432 and 6798 items 38, 36, 32
// and 55.  Where all the entries of a bin share its times the items may be as
// uneven as space is: stars near 60 others at 3724 and 7429 items 650 and 464.  The
// FP64 form's items are long, and of one kind.
uint32_t item_fit(int prec, uint32_t grid_waves) {
    return prec == TDS_PREC_FP64 ? 0u : busy_waves(grid_waves);
}
// Whether that holds whatever the buckets: bins wider than segments, or more waves
// than have a first reservation given (dense walks in 8,192 waves, kernel at 2,500
// and 10,000 items 84 and 166 us).
uint32_t fit_always(const tds_index* idx, uint32_t grid_waves) {
    return idx->bw > 1.5 * idx->mean_dt || grid_waves > kFillWaves ? 1u : 0u;
}

// Upper bound of the work items of a batch of nq query segments: every
// non-empty bucket contributes ceil(count / 64) groups, each split into at
// most ceil((n + 63) / chunk) chunks (chunks count from a 64-entry block).
// With the chunk picked by the item count, twice the count aimed at bounds
// the items of the smaller chunks.
uint64_t item_bound(uint64_t nq, uint32_t nb, uint64_t n, uint32_t chunk, uint32_t grid_waves) {
    const uint64_t groups = (nq + kWave - 1) / kWave + std::min<uint64_t>(nq, nb);
    const uint64_t c = chunk & ~kChunkAuto;
    const uint64_t bound = groups * std::max<uint64_t>((n + kWave - 1 + c - 1) / c, 1);
    return chunk & kChunkAuto ? std::max<uint64_t>(bound, 2ull * item_target(grid_waves)) : bound;
}

constexpr uint64_t kMaxItemTable = 1ull << 26;  // entries (256 MiB) kept without an exact count

// Largest chunk: a queued pair packs its candidate's offset in the chunk
// (at most the chunk rounded up to whole tiles) above 6 bits of query lane,
// in 32 bits.
constexpr uint32_t kMaxChunk = 1u << 19;
static_assert((uint64_t)kMaxChunk + 2 * kTile < (1ull << 26), "packed queue entries");

uint32_t resolve_chunk(int prec, uint32_t chunk) {
    if (chunk) return std::min(std::max(chunk, 64u), kMaxChunk);
    return kChunkAuto | (prec == TDS_PREC_FP64 ? 512u : 4096u);
}

uint32_t resolve_grid(uint32_t grid_waves) {
    return std::min(grid_waves ? grid_waves : kDefaultWaves, kMaxDistBlocks * kWavesPerBlock);
}

// Waves of a distance-kernel launch of grid_waves (whole workgroups).
uint32_t launch_blocks(uint32_t grid_waves) {
    return std::min(kMaxDistBlocks, std::max(1u, ceil_div(grid_waves, kWavesPerBlock)));
}

// Result stage of each wave: up to kStageMax records, within a workspace
// total of at most kStageTotal (the stages of one launch never exceed about
// 300 MB; at the default grid every wave gets kStageMax).
constexpr uint32_t kStageMax = 2048;
constexpr size_t kStageTotal = size_t(1) << 23;

size_t stage_total(uint32_t grid_waves) {
    const size_t waves = (size_t)launch_blocks(grid_waves) * kWavesPerBlock;
    return std::min(kStageTotal, waves * kStageMax);
}

uint32_t stage_per_wave(size_t recs, uint32_t blocks) {
    const size_t per = recs / ((size_t)blocks * kWavesPerBlock);
    return (uint32_t)std::min<size_t>(kStageMax, per / kWave * kWave);
}

// Kernel variant and dealing of a launch, packed: candidates per lane per
// tile of the FP32 form (0 selects 2; 2 and 4 are built) in the low byte,
// the place of the closest-approach refinement (TDS_REFINE_*, 0 selects the
// walk) in the next, the dealing of the work items (TDS_DEAL_*, 0
// selects the dynamic tail) above; 0 if any of them is unknown.
uint32_t resolve_tile(uint32_t t, uint32_t refine = 0, uint32_t deal = 0) {
    if (t == 0) t = 2;
    if (t != 2 && t != 4) return 0;
    if (refine > TDS_REFINE_INLINE) return 0;
    if (refine == TDS_REFINE_DEFAULT) refine = TDS_REFINE_INLINE;
    if (deal == TDS_DEAL_DEFAULT) deal = TDS_DEAL_DYNAMIC;
    if (deal != TDS_DEAL_DYNAMIC && deal != TDS_DEAL_STATIC) return 0;
    return t | (refine << 8) | (deal << 16);
}

int resolve_prec(int p) {
    if (p == TDS_PREC_DEFAULT) return TDS_PREC_FP32_RECHECK;
    if (p != TDS_PREC_FP64 && p != TDS_PREC_FP32_RECHECK) return -1;
    return p;
}

// Device view of the query arrays; host arrays are copied into the staging
// buffers first, through the workspace's pinned block (`pin`, taken at its
// first use) where they fit and there is one.
int stage_queries(const tds_segments* Q, QueryView* V, hipStream_t s, double** stage_buf,
                  size_t* stage_cap, uint32_t** traj_buf, size_t* traj_cap, PinBlock** block) {
    V->n = Q->n;
    const double* src[8] = {Q->xs, Q->ys, Q->zs, Q->ts, Q->xe, Q->ye, Q->ze, Q->te};
    if (Q->on_device) {
        for (int k = 0; k < 8; ++k) V->a[k] = src[k];
        V->traj = Q->traj_id;
        return TDS_OK;
    }
    const hipMemcpyKind kind = hipMemcpyHostToDevice;
    if (block && Q->n <= kPinSegs && acquire_pin(block) == TDS_OK) {
        char* pin = (*block)->segs;
        const size_t col = Q->n * sizeof(double);
        for (int k = 0; k < 8; ++k) std::memcpy(pin + k * col, src[k], col);
        if (Q->traj_id) std::memcpy(pin + 8 * col, Q->traj_id, Q->n * sizeof(uint32_t));
        const size_t bytes = 8 * col + (Q->traj_id ? Q->n * sizeof(uint32_t) : 0);
        // the ids after the columns, in whole doubles
        TDS_TRY(grow(stage_buf, stage_cap, (bytes + sizeof(double) - 1) / sizeof(double)));
        TDS_HIP(hipMemcpyAsync(*stage_buf, pin, bytes, kind, s));
        for (int k = 0; k < 8; ++k) V->a[k] = *stage_buf + k * Q->n;
        V->traj = Q->traj_id ? reinterpret_cast<uint32_t*>(*stage_buf + 8 * Q->n) : nullptr;
        return TDS_OK;
    }
    TDS_TRY(grow(stage_buf, stage_cap, 8 * (size_t)Q->n));
    for (int k = 0; k < 8; ++k) {
        TDS_HIP(hipMemcpyAsync(*stage_buf + k * Q->n, src[k], Q->n * sizeof(double), kind, s));
        V->a[k] = *stage_buf + k * Q->n;
    }
    V->traj = nullptr;
    if (Q->traj_id) {
        TDS_TRY(grow(traj_buf, traj_cap, (size_t)Q->n));
        TDS_HIP(hipMemcpyAsync(*traj_buf, Q->traj_id, Q->n * sizeof(uint32_t), kind, s));
        V->traj = *traj_buf;
    }
    return TDS_OK;
}

// Positions per chunk of the direct output (a whole number of 64): a quarter
// of a wave's stage.  A wave's first chunk is given to it, the next
// reservations are of 2, 4, 4 ... chunks.  A returning atomic on one counter
// takes 30 ns of the chip's time: with reservations of 128, 256, 512 or 2048
// positions 71 million results take 16.7, 8.9, 5.0 or 4.4 ms, so they have to
// be large, but the holes that large first ones leave cost the fill 40 to 74 us
// where a wave has few results, and the first atomic of every wave at the
// search's end as much again (8000 items of dense walks: kernel 143 -> 114 us
// without it and without the waves' atomics on the number of results).
uint32_t direct_chunk(uint32_t stage_cap) {
    return std::max((uint32_t)kWave, stage_cap / 4 / kWave * kWave);
}

DistArgs dist_args(const tds_index* idx, const Workspace* w, const QueryView& Q, tds_result* out,
                   uint64_t win_lo, uint32_t item_begin, uint32_t item_end, uint32_t* item_count,
                   uint32_t grid_waves, bool by_order, uint32_t cpl, uint32_t r_cap,
                   bool direct = false) {
    DistArgs A;
    A.cpl = cpl & 0xFFu;
    A.refine = (cpl >> 8) & 0xFFu;
    A.deal = cpl >> 16;
    A.dyn_ctr = w->dyn_ctr;
    A.stage = w->stage;
    A.stage_meta = w->stage_meta;
    A.stage_cap = stage_per_wave(w->stage_recs, launch_blocks(grid_waves));
    A.by_order = by_order ? 1u : 0u;
    A.I = view_of(idx);
    A.self = Q.ent ? 1u : 0u;
    A.keep = r_cap <= (uint32_t)kWave ? 1u : 0u;
    A.qsorted = w->qsorted;
    A.qf = w->qf;
    A.qev = w->qev;
    A.binfo = w->binfo;
    A.item_bucket = w->item_bucket;
    A.desc = w->desc;
    A.hdr = w->hdr;
    A.bstats = w->bstats;
    A.req = w->req;
    A.rc = w->req_ctr;
    A.out = out;
    A.win_lo = win_lo;
    A.item_begin = item_begin;
    A.item_end = item_end;
    A.item_count = item_count;
    // direct output: reservations of up to a wave's stage size, the stage
    // buffer as the scratch for positions past the capacity
    const uint32_t waves = launch_blocks(grid_waves) * kWavesPerBlock;
    A.direct = (direct && !by_order && win_lo == 0 && waves <= kMaxDirectWaves &&
                waves <= w->stage_waves && A.stage_cap >= (uint32_t)kWave)
                   ? 1u
                   : 0u;
    const bool small = waves <= kFillWaves;
    A.dir_chunk = small ? direct_chunk(A.stage_cap) : A.stage_cap;
    A.dir_max = small ? std::min(A.stage_cap / A.dir_chunk, kFillChunks / waves) : 1u;
    A.dir_given = small ? 1u : 0u;
    A.dir_ctr = w->dyn_ctr + (size_t)kCtrDirect * kCtrStride;
    A.dscratch = w->stage;
    A.dscratch_cap = (uint64_t)waves * A.stage_cap;
    A.dlast = w->dlast;
    return A;
}

// The distance kernel, timed by the two events when both are given.
int launch_distance(int prec, const DistArgs& A, uint32_t grid_waves, hipStream_t s,
                    hipEvent_t ev_begin, hipEvent_t ev_end) {
    const uint32_t blocks = launch_blocks(grid_waves);
    // every wave must be able to stage a full batch of 64 evaluations
    if (!A.stage || A.stage_cap < (uint32_t)kWave) return TDS_E_DEVICE;
    constexpr int F32 = TDS_PREC_FP32_RECHECK, Q = TDS_REFINE_QUEUED, N = TDS_REFINE_INLINE;
    void (*kern)(DistArgs);
    const auto fp32 = [&](auto cull) -> void (*)(DistArgs) {
        constexpr bool C = decltype(cull)::value;
        if (A.refine == Q) return A.cpl == 2 ? k_distance<F32, 2, Q, C> : k_distance<F32, 4, Q, C>;
        return A.cpl == 2 ? k_distance<F32, 2, N, C> : k_distance<F32, 4, N, C>;
    };
    if (prec == TDS_PREC_FP64) kern = k_distance<TDS_PREC_FP64, 2, Q, false>;
    else kern = A.I.bbox ? fp32(std::true_type()) : fp32(std::false_type());
    if (ev_begin && ev_end) {
        // the events take the dispatch's own start and end times (no marker
        // packets around the kernel, so no bubbles before and after it)
        hipExtLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), 0, s, ev_begin, ev_end, 0u, A);
    } else {
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), 0, s, A);
    }
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

// After the distance kernel: the fold of its counters and, with direct output,
// the fill of the holes left by the waves' last reservations.
int launch_finish(const DistArgs& A, const Workspace* w, uint32_t grid_waves, hipStream_t s) {
    const uint32_t blocks = launch_blocks(grid_waves), nw = blocks * kWavesPerBlock;
    if (A.direct && A.dir_given) {
        hipLaunchKernelGGL(k_fill, dim3(kFillBlocks + 1), dim3(1024), 0, s, A.req, A.rc, A.dir_ctr,
                           A.dlast, nw, A.dir_chunk, A.out, A.dscratch, A.bstats, blocks, A.hdr);
        TDS_HIP(hipGetLastError());
        return TDS_OK;
    }
    hipLaunchKernelGGL(k_stats_fold, dim3(1), dim3(256), 0, s, A.bstats, blocks, A.hdr);
    if (A.direct) {
        hipLaunchKernelGGL(k_fill_plan, dim3(1), dim3(1024), 0, s, A.req, A.rc, A.dir_ctr,
                           A.dlast, nw, A.dir_chunk, w->fill_s, w->fill_d, w->fill_dstart,
                           w->fill_plan);
        hipLaunchKernelGGL(k_fill_copy, dim3(1024), dim3(256), 0, s, w->fill_plan, w->fill_s,
                           w->fill_d, w->fill_dstart, nw, A.dir_chunk, A.req, A.out, A.dscratch);
    }
    TDS_HIP(hipGetLastError());
    return TDS_OK;
}

// The whole search for the batch described by w->desc / w->req, as a fixed
// sequence of fixed-shape launches (capturable in a graph): clear, prepare
// queries, bucket table, ordering, item table, distance kernel over every
// item.  q_grid and r_cap are the capacities the launches are shaped for.
int enqueue_pipeline(const tds_index* idx, Workspace* w, const QueryView& Q, size_t q_grid,
                     uint32_t r_cap, int prec, uint32_t chunk, uint32_t grid_waves, uint32_t cpl,
                     tds_result* out, uint32_t* item_count, hipStream_t s, hipEvent_t ev_begin,
                     hipEvent_t ev_end, bool direct = false) {
    const IndexView I = view_of(idx);
    const uint32_t shift = bucket_shift(idx->m);
    const uint32_t nb = bucket_count(idx->m);
    const uint32_t nparts = count_parts(nb);
    const uint32_t zn = std::max(std::max(nb * nparts, r_cap), kCtrSlots * kCtrStride);
    const DistArgs A = dist_args(idx, w, Q, out, 0, 0, 0xFFFFFFFFu, item_count, grid_waves, false,
                                 cpl, r_cap, direct);
    // k_zero also clears the request counters the distance kernel appends with
    hipLaunchKernelGGL(k_zero, dim3(ceil_div(zn, kBlock)), dim3(kBlock), 0, s, w->hdr, w->b_count,
                       w->b_hi, nb, nparts, w->req_ctr, r_cap, w->dyn_ctr,
                       A.dir_given ? (unsigned long long)launch_blocks(grid_waves) * kWavesPerBlock *
                                         A.dir_chunk
                                   : 0ull);
    const uint32_t qblocks = std::max(1u, ceil_div(q_grid, kBlock));
    const uint32_t bpp = ceil_div(qblocks, nparts);  // workgroup b counts in part b / bpp < nparts
    hipLaunchKernelGGL(k_qprep, dim3(qblocks), dim3(kBlock), 0, s, Q, w->desc, w->req, I, w->qf,
                       w->qev, w->qkey, w->qslot, w->b_count, w->b_hi, shift, nb, bpp, w->hdr);
    hipLaunchKernelGGL(k_bucket_scan, dim3(1), dim3(1024), 0, s, w->b_count, w->b_hi,
                       idx->bin_first, idx->min_te, idx->max_ts, idx->m, shift, nb, nparts,
                       chunk & ~kChunkAuto, chunk_levels(prec, chunk), item_target(grid_waves),
                       item_fit(prec, grid_waves), fit_always(idx, grid_waves), w->b_start,
                       w->b_nch, w->binfo, w->hdr);
    hipLaunchKernelGGL(k_scatter, dim3(qblocks + nb), dim3(kBlock), 0, s, w->desc, w->qkey,
                       w->qslot, w->b_start, w->b_count, nb, bpp, qblocks, w->qsorted, w->binfo,
                       w->item_bucket, w->hdr);
    TDS_HIP(hipGetLastError());
    TDS_TRY(launch_distance(prec, A, grid_waves, s, ev_begin, ev_end));
    return launch_finish(A, w, grid_waves, s);
}

// Re-runs the distance kernel over work items [i0, i1) keeping result
// positions [win_lo, win_lo + capacity) (incremental processing).
// by_order: one item of a one-request search, its results placed by their
// order in the item (a window of an item larger than the device buffer).
int enqueue_range(const tds_index* idx, Workspace* w, const QueryView& Q, int prec, uint32_t r_cap,
                  tds_result* out, uint64_t win_lo, uint32_t i0, uint32_t i1, bool by_order,
                  uint32_t grid_waves, uint32_t cpl, hipStream_t s, hipEvent_t ev_begin,
                  hipEvent_t ev_end) {
    hipLaunchKernelGGL(k_reset_pass, dim3(ceil_div(std::max(r_cap, kCtrSlots * kCtrStride), 256)),
                       dim3(256), 0, s, w->req_ctr, r_cap, w->dyn_ctr);
    TDS_HIP(hipGetLastError());
    const DistArgs A = dist_args(idx, w, Q, out, win_lo, i0, i1, nullptr, grid_waves, by_order,
                                 cpl, r_cap);
    TDS_TRY(launch_distance(prec, A, grid_waves, s, ev_begin, ev_end));
    return launch_finish(A, w, grid_waves, s);
}

Workspace* acquire(tds_index* idx) {
    {
        std::lock_guard<std::mutex> g(idx->mu);
        if (!idx->pool.empty()) {
            Workspace* w = idx->pool.back();
            idx->pool.pop_back();
            return w;
        }
    }
    Workspace* w = new (std::nothrow) Workspace();
    if (!w) return nullptr;
    w->device = idx->device;
    if (ws_init(w) != TDS_OK) {
        delete w;
        return nullptr;
    }
    return w;
}

void release(tds_index* idx, Workspace* w) {
    std::lock_guard<std::mutex> g(idx->mu);
    idx->pool.push_back(w);
}

// Gives a call's workspace back.  Unless the call has waited for all it queued
// on its stream (`idle`: it has returned its results), that is done first: the
// next call may be on another stream, and the copy of the query arrays reads the
// workspace's pinned memory and writes its device memory.
struct WsGuard {
    tds_index* idx;
    Workspace* w;
    hipStream_t s;
    bool idle = false;
    ~WsGuard() {
        if (!idle) (void)hipStreamSynchronize(s);
        release(idx, w);
    }
};

bool valid_window(double d, double t0, double t1) {
    return d >= 0.0 && !std::isinf(d) && t0 < t1;
}

// Sizes the item table for the batch: from the bound when it is small enough,
// else from the exact count after the preparation launches (one extra sync).
int reserve_items(const tds_index* idx, Workspace* w, uint64_t nq, uint32_t chunk,
                  uint32_t grid_waves, uint64_t* cap_out) {
    const uint64_t bound = item_bound(nq, bucket_count(idx->m), idx->n, chunk, grid_waves);
    const uint64_t cap = std::min<uint64_t>(bound, kMaxItemTable);
    TDS_TRY(grow(&w->item_bucket, &w->item_bucket_cap, std::max<size_t>(cap, 1)));
    TDS_TRY(grow(&w->item_count, &w->item_cap, std::max<size_t>(cap, 1)));
    *cap_out = cap;
    return TDS_OK;
}

// Largest output that a one-request search stages unless told otherwise: 32
// records per wave, 4 MB in all at the default grid, so that the second trip of
// the records that are kept costs 2 us.  Small outputs are those of small
// searches, which are latency: staged they end with the last item, direct with
// one more kernel of 12.5 us (4,900 query segments, 6,000 records: the call 100
// direct, 93 staged; 201 query segments 88 and 82).  Large outputs lose by the second
// trip (174 million records 4.8 and 7.1 ms).  Where results stay staged from item to
// item the two meet past 466,000 records (186 and 177 us); flushed after every item,
// for which the line was drawn, they met before that (189 and 202).
uint64_t staged_room(uint32_t grid_waves) {
    return 32ull * launch_blocks(grid_waves) * kWavesPerBlock;
}

// One run of the pipeline for the batch whose requests the caller staged in
// w->req_host with an item table of `cap` entries: the descriptor and the
// requests go up, the launches are ordered on `s`, and the header and request
// counters come back into pinned memory.  Returns without waiting.
int enqueue_attempt(const tds_index* idx, Workspace* w, const QueryView& V, uint32_t nreq,
                    int prec, uint32_t chunk, uint32_t grid_waves, uint32_t cpl, uint32_t output,
                    tds_result* out, hipStream_t s, uint64_t cap, uint32_t peek = 0) {
    w->desc_host->nq = V.n;
    w->desc_host->nreq = nreq;
    w->desc_host->item_cap = (uint32_t)std::min<uint64_t>(cap, 0xFFFFFFFFull);
    TDS_TRY(ws_upload(w, nreq, s));
    const bool direct =
        nreq == 1 && (output == TDS_OUTPUT_DIRECT ||
                      (output == TDS_OUTPUT_DEFAULT &&
                       w->req_host->out_capacity > staged_room(grid_waves)));
    TDS_TRY(enqueue_pipeline(idx, w, V, V.n, nreq, prec, chunk, grid_waves, cpl, out,
                             w->item_count, s, w->ev0, w->ev1, direct));
    if (peek)
        TDS_HIP(hipMemcpyAsync(w->pin->peek, out, peek * sizeof(tds_result), hipMemcpyDeviceToHost, s));
    return ws_download(w, nreq, s);
}

// After an attempt has completed: its header and kernel time; returns TDS_OK,
// TDS_E_INVALID, or 1 when the item table was too small (it is then sized
// exactly for another attempt).
int finish_attempt(Workspace* w, tds_stats* st, SearchHeader* h_out, uint64_t* cap) {
    *h_out = *w->hdr_host;
    float ms = 0.f;
    TDS_HIP(hipEventElapsedTime(&ms, w->ev0, w->ev1));
    st->kernel_ms += ms;
    st->passes += 1;
    if (h_out->err & 1u) return TDS_E_INVALID;
    if (!(h_out->err & 2u)) return TDS_OK;
    *cap = h_out->n_items;
    TDS_TRY(grow(&w->item_bucket, &w->item_bucket_cap, std::max<size_t>(*cap, 1)));
    TDS_TRY(grow(&w->item_count, &w->item_cap, std::max<size_t>(*cap, 1)));
    return 1;
}

// Runs the pipeline once for the batch whose requests the caller staged in
// w->req_host (sent to the device here, with the descriptor), growing the
// item table and re-running if the bound was too small.
int run_batch(const tds_index* idx, Workspace* w, const QueryView& V, uint32_t nreq, int prec,
              uint32_t chunk, uint32_t grid_waves, uint32_t cpl, uint32_t output, tds_result* out,
              hipStream_t s, tds_stats* st, SearchHeader* h_out, uint32_t peek = 0) {
    uint64_t cap = 0;
    TDS_TRY(reserve_items(idx, w, V.n, chunk, grid_waves, &cap));
    TDS_TRY(ws_reserve_stage(w, grid_waves));
    for (int attempt = 0; attempt < 2; ++attempt) {
        TDS_TRY(enqueue_attempt(idx, w, V, nreq, prec, chunk, grid_waves, cpl, output, out, s,
                                cap, peek));
        TDS_HIP(hipStreamSynchronize(s));
        const int r = finish_attempt(w, st, h_out, &cap);
        if (r != 1) return r;
    }
    return TDS_E_DEVICE;
}

}  // namespace

int resolve_config(const tds_search_params* params, PipelineConfig* cfg) {
    tds_search_params P;
    tds_search_params_default(&P);
    if (params) P = *params;
    cfg->prec = resolve_prec(P.precision);
    if (cfg->prec < 0) return TDS_E_INVALID;
    cfg->chunk = resolve_chunk(cfg->prec, P.chunk);
    cfg->grid_waves = resolve_grid(P.grid_waves);
    cfg->cpl = resolve_tile(P.tile, P.refine, P.deal);
    if (!cfg->cpl) return TDS_E_INVALID;
    if (P.output > TDS_OUTPUT_STAGED) return TDS_E_INVALID;  // batches always stage
    return TDS_OK;
}

uint64_t item_table_bound(const tds_index* idx, uint64_t nq, const PipelineConfig& cfg) {
    return item_bound(nq, bucket_count(idx->m), idx->n, cfg.chunk, cfg.grid_waves);
}

int enqueue_search(const tds_index* idx, Workspace* w, const double* const* qarrays,
                   const uint32_t* qtraj, size_t q_grid, uint32_t r_cap,
                   const PipelineConfig& cfg, tds_result* out, hipStream_t s) {
    QueryView V{};
    for (int k = 0; k < 8; ++k) V.a[k] = qarrays[k];
    V.traj = qtraj;
    V.n = q_grid;
    return enqueue_pipeline(idx, w, V, q_grid, r_cap, cfg.prec, cfg.chunk, cfg.grid_waves,
                            cfg.cpl, out, w->item_count, s, nullptr, nullptr);
}

int schedule_impl(tds_index* idx, const tds_segments* Q, double t_start, double t_end,
                  uint32_t* lo, uint32_t* hi, hipStream_t s) {
    if (!idx || !lo || !hi) return TDS_E_INVALID;
    TDS_TRY(validate_segments_args(Q));
    if (!(t_start < t_end)) return TDS_E_INVALID;
    const uint64_t nq = Q->n;
    double* stage = nullptr;
    size_t scap = 0;
    uint32_t* tstage = nullptr;
    size_t tcap = 0;
    uint32_t *dlo = nullptr, *dhi = nullptr, *err = nullptr;
    int st = TDS_OK;
    QueryView V{};
    do {
        if ((st = stage_queries(Q, &V, s, &stage, &scap, &tstage, &tcap, nullptr))) break;
        if ((st = dmalloc(&dlo, nq))) break;
        if ((st = dmalloc(&dhi, nq))) break;
        if ((st = dmalloc(&err, 1))) break;
        if (hipMemsetAsync(err, 0, sizeof(uint32_t), s) != hipSuccess) { st = TDS_E_DEVICE; break; }
        hipLaunchKernelGGL(k_schedule, dim3(ceil_div(nq, kBlock)), dim3(kBlock), 0, s, V, t_start,
                           t_end, view_of(idx), dlo, dhi, err);
        uint32_t herr = 0;
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(lo, dlo, nq * sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipMemcpyAsync(hi, dhi, nq * sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipMemcpyAsync(&herr, err, sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            st = TDS_E_DEVICE;
            break;
        }
        if (herr) st = TDS_E_INVALID;
    } while (0);
    dfree(stage);
    dfree(tstage);
    dfree(dlo);
    dfree(dhi);
    dfree(err);
    return st;
}

namespace {
int search_core(tds_index* idx, const tds_segments* Q, bool self_join, double d, double t_start,
                double t_end, tds_result* out, uint64_t capacity, uint64_t* n_out,
                const tds_search_params* params, hipStream_t s, tds_stats* stats);
}  // namespace

int search_impl(tds_index* idx, const tds_segments* Q, double d, double t_start, double t_end,
                tds_result* out, uint64_t capacity, uint64_t* n_out,
                const tds_search_params* params, hipStream_t s, tds_stats* stats) {
    if (!idx || !n_out) return TDS_E_INVALID;
    *n_out = 0;
    TDS_TRY(validate_segments_args(Q));
    return search_core(idx, Q, false, d, t_start, t_end, out, capacity, n_out, params, s, stats);
}

int self_join_impl(tds_index* idx, double d, double t_start, double t_end, tds_result* out,
                   uint64_t capacity, uint64_t* n_out, const tds_search_params* params,
                   hipStream_t s, tds_stats* stats) {
    if (!idx || !n_out) return TDS_E_INVALID;
    *n_out = 0;
    return search_core(idx, nullptr, true, d, t_start, t_end, out, capacity, n_out, params, s,
                       stats);
}

namespace {
int search_core(tds_index* idx, const tds_segments* Q, bool self_join, double d, double t_start,
                double t_end, tds_result* out, uint64_t capacity, uint64_t* n_out,
                const tds_search_params* params, hipStream_t s, tds_stats* stats) {
    const auto t_begin = std::chrono::steady_clock::now();
    if (!valid_window(d, t_start, t_end)) return TDS_E_INVALID;
    if (capacity > 0 && !out) return TDS_E_INVALID;
    tds_search_params P;
    tds_search_params_default(&P);
    if (params) P = *params;
    const int prec = resolve_prec(P.precision);
    if (prec < 0) return TDS_E_INVALID;
    const uint32_t chunk = resolve_chunk(prec, P.chunk);
    const uint32_t grid_waves = resolve_grid(P.grid_waves);
    const uint32_t cpl = resolve_tile(P.tile, P.refine, P.deal);
    if (!cpl) return TDS_E_INVALID;
    if (P.output > TDS_OUTPUT_STAGED) return TDS_E_INVALID;
    const bool dev_out = P.out_on_device != 0;

    Workspace* w = acquire(idx);
    if (!w) return TDS_E_NOMEM;
    WsGuard guard{idx, w, s};
    const uint64_t nq = self_join ? idx->n : Q->n;
    TDS_TRY(ws_reserve(w, nq, 1));
    QueryView V{};
    if (self_join) {
        V.n = nq;
        V.ent = idx->e64;
        V.ent_id = idx->seg_id;
        V.ent_traj = idx->traj;
    } else {
        TDS_TRY(stage_queries(Q, &V, s, &w->qstage, &w->stage_cap, &w->qtraj_stage, &w->traj_cap,
                              &w->pin));
    }

    // result buffer
    uint64_t dev_cap;
    tds_result* res;
    if (dev_out) {
        dev_cap = capacity;
        res = out;
    } else {
        dev_cap = P.device_capacity ? P.device_capacity
                                    : std::min<uint64_t>(std::max<uint64_t>(capacity, 1), kDefaultDevCap);
        TDS_TRY(grow(&w->res, &w->res_cap, (size_t)std::max<uint64_t>(dev_cap, 1)));
        res = w->res;
    }
    Request R{};
    R.q_begin = 0;
    R.q_count = nq;
    R.d = d;
    R.t_start = t_start;
    R.t_end = t_end;
    R.out_offset = 0;
    R.out_capacity = dev_cap;
    *w->req_host = R;  // uploaded with the descriptor

    tds_stats st{};
    st.query_segments = nq;
    SearchHeader h{};
    // pass 1: every item, result window [0, dev_cap)
    uint32_t peek = 0;
    if (!dev_out && capacity && acquire_pin(&w->pin) == TDS_OK)
        peek = (uint32_t)std::min<uint64_t>(kPeek, dev_cap);
    TDS_TRY(run_batch(idx, w, V, 1, prec, chunk, grid_waves, cpl, P.output, res, s, &st, &h, peek));
    const ReqCounter rc = w->rc_host[0];
    const uint32_t n_items = h.n_items;
    st.active_segments = h.active;
    st.work_items = n_items;
    st.candidate_tests = h.tests;
    st.filter_tests = h.ftests;
    st.block_tests = h.btests;
    st.fp64_evals = h.evals;
    st.stage_flushes = h.flushes;
    const uint64_t total = rc.count;
    float ms = 0.f;
    int status = TDS_OK;
    if (dev_out) {
        status = (total > capacity) ? TDS_E_OVERFLOW : TDS_OK;
    } else if (total <= dev_cap) {
        const uint64_t k = std::min(total, capacity);
        if (k && k <= peek) {
            std::memcpy(out, w->pin->peek, k * sizeof(tds_result));
        } else if (k) {
            TDS_HIP(hipMemcpyAsync(out, res, k * sizeof(tds_result), hipMemcpyDeviceToHost, s));
            TDS_HIP(hipStreamSynchronize(s));
        }
        status = (total > capacity) ? TDS_E_OVERFLOW : TDS_OK;
    } else if (total > capacity) {
        const uint64_t k = std::min(dev_cap, capacity);
        if (k) TDS_HIP(hipMemcpyAsync(out, res, k * sizeof(tds_result), hipMemcpyDeviceToHost, s));
        TDS_HIP(hipStreamSynchronize(s));
        status = TDS_E_OVERFLOW;
    } else {
        // incremental processing: re-run consecutive work items whose results
        // fit the device buffer; an item larger than the buffer is re-run
        // alone with a sliding window (one wave processes an item, in a fixed
        // order, so its result order is the same on every run)
        std::vector<uint32_t> cnt(n_items);
        TDS_HIP(hipMemcpyAsync(cnt.data(), w->item_count, n_items * sizeof(uint32_t),
                               hipMemcpyDeviceToHost, s));
        TDS_HIP(hipStreamSynchronize(s));
        uint64_t written = 0;
        uint32_t i0 = 0;
        while (i0 < n_items) {
            uint32_t i1 = i0;
            uint64_t sum = 0;
            while (i1 < n_items && sum + cnt[i1] <= dev_cap) sum += cnt[i1++];
            std::vector<std::pair<uint64_t, uint64_t>> windows;  // (win_lo, expected)
            const bool by_order = i1 == i0;  // one item larger than the buffer
            if (i1 == i0) {
                i1 = i0 + 1;
                for (uint64_t wl = 0; wl < cnt[i0]; wl += dev_cap)
                    windows.push_back({wl, std::min<uint64_t>(dev_cap, cnt[i0] - wl)});
            } else {
                windows.push_back({0, sum});
            }
            for (auto& win : windows) {
                if (win.second == 0) continue;
                TDS_TRY(enqueue_range(idx, w, V, prec, 1, res, win.first, i0, i1, by_order,
                                      std::min(grid_waves, i1 - i0), cpl, s, w->ev0, w->ev1));
                TDS_HIP(hipMemcpyAsync(out + written, res, win.second * sizeof(tds_result),
                                       hipMemcpyDeviceToHost, s));
                TDS_HIP(hipStreamSynchronize(s));
                TDS_HIP(hipEventElapsedTime(&ms, w->ev0, w->ev1));
                st.kernel_ms += ms;
                st.passes += 1;
                written += win.second;
            }
            i0 = i1;
        }
        if (written != total) return TDS_E_DEVICE;
    }
    guard.idle = true;
    *n_out = total;
    st.results = total;
    st.total_ms =
        std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
    if (stats) *stats = st;
    {
        std::lock_guard<std::mutex> g(idx->mu);
        idx->last = st;
    }
    return status;
}
}  // namespace

// A search begun on a stream and not yet ended (tds_search_begin): it holds
// its workspace until tds_search_end.
struct PendingSearch {
    tds_index* idx = nullptr;
    Workspace* w = nullptr;
    hipStream_t s = nullptr;
    QueryView V{};
    tds_result* out = nullptr;
    uint64_t capacity = 0, cap_items = 0;
    int prec = 0;
    uint32_t chunk = 0, grid_waves = 0, cpl = 0, output = 0;
    hipEvent_t done = nullptr;
    std::chrono::steady_clock::time_point t0;
};

int search_begin_impl(tds_index* idx, const tds_segments* Q, double d, double t_start,
                      double t_end, tds_result* out, uint64_t capacity,
                      const tds_search_params* params, hipStream_t s, void** pending) {
    const auto t_begin = std::chrono::steady_clock::now();
    if (!idx || !pending) return TDS_E_INVALID;
    *pending = nullptr;
    TDS_TRY(validate_segments_args(Q));
    if (!valid_window(d, t_start, t_end)) return TDS_E_INVALID;
    if (capacity > 0 && !out) return TDS_E_INVALID;
    tds_search_params P;
    tds_search_params_default(&P);
    if (params) P = *params;
    if (!P.out_on_device) return TDS_E_INVALID;  // the output is device memory
    const int prec = resolve_prec(P.precision);
    if (prec < 0) return TDS_E_INVALID;
    const uint32_t cpl = resolve_tile(P.tile, P.refine, P.deal);
    if (!cpl || P.output > TDS_OUTPUT_STAGED) return TDS_E_INVALID;
    PendingSearch* ps = new (std::nothrow) PendingSearch();
    if (!ps) return TDS_E_NOMEM;
    ps->idx = idx;
    ps->s = s;
    ps->out = out;
    ps->capacity = capacity;
    ps->prec = prec;
    ps->chunk = resolve_chunk(prec, P.chunk);
    ps->grid_waves = resolve_grid(P.grid_waves);
    ps->cpl = cpl;
    ps->output = P.output;
    ps->t0 = t_begin;
    int st = TDS_OK;
    do {
        if (!(ps->w = acquire(idx))) { st = TDS_E_NOMEM; break; }
        Workspace* w = ps->w;
        if ((st = ws_reserve(w, Q->n, 1))) break;
        if ((st = stage_queries(Q, &ps->V, s, &w->qstage, &w->stage_cap, &w->qtraj_stage,
                                &w->traj_cap, &w->pin)))
            break;
        Request R{};
        R.q_begin = 0;
        R.q_count = Q->n;
        R.d = d;
        R.t_start = t_start;
        R.t_end = t_end;
        R.out_offset = 0;
        R.out_capacity = capacity;
        *w->req_host = R;
        if ((st = reserve_items(idx, w, Q->n, ps->chunk, ps->grid_waves, &ps->cap_items))) break;
        if ((st = ws_reserve_stage(w, ps->grid_waves))) break;
        if (hipEventCreateWithFlags(&ps->done, hipEventDisableTiming) != hipSuccess) {
            ps->done = nullptr;
            st = TDS_E_DEVICE;
            break;
        }
        if ((st = enqueue_attempt(idx, w, ps->V, 1, prec, ps->chunk, ps->grid_waves, cpl,
                                  ps->output, out, s, ps->cap_items)))
            break;
        if (hipEventRecord(ps->done, s) != hipSuccess) { st = TDS_E_DEVICE; break; }
    } while (0);
    if (st != TDS_OK) {
        if (ps->done) (void)hipEventDestroy(ps->done);
        if (ps->w) {
            (void)hipStreamSynchronize(s);  // nothing of it may still run
            release(idx, ps->w);
        }
        delete ps;
        return st;
    }
    *pending = ps;
    return TDS_OK;
}

int search_end_impl(void* pending, uint64_t* n_out, tds_stats* stats) {
    PendingSearch* ps = static_cast<PendingSearch*>(pending);
    if (!ps) return TDS_E_INVALID;
    Workspace* w = ps->w;
    tds_stats st{};
    st.query_segments = ps->V.n;
    SearchHeader h{};
    int status = TDS_OK;
    if (hipEventSynchronize(ps->done) != hipSuccess) {
        status = TDS_E_DEVICE;
    } else {
        int r = finish_attempt(w, &st, &h, &ps->cap_items);
        if (r == 1) {
            // the item table was too small: the search runs again, sized exactly
            r = enqueue_attempt(ps->idx, w, ps->V, 1, ps->prec, ps->chunk, ps->grid_waves,
                                ps->cpl, ps->output, ps->out, ps->s, ps->cap_items);
            if (r == TDS_OK)
                r = hipStreamSynchronize(ps->s) == hipSuccess
                        ? finish_attempt(w, &st, &h, &ps->cap_items)
                        : TDS_E_DEVICE;
            if (r == 1) r = TDS_E_DEVICE;
        }
        status = r;
    }
    if (status != TDS_OK) (void)hipStreamSynchronize(ps->s);  // a second attempt may still run
    if (status == TDS_OK) {
        const uint64_t total = w->rc_host[0].count;
        if (n_out) *n_out = total;
        st.active_segments = h.active;
        st.work_items = h.n_items;
        st.candidate_tests = h.tests;
        st.filter_tests = h.ftests;
        st.block_tests = h.btests;
        st.fp64_evals = h.evals;
        st.stage_flushes = h.flushes;
        st.results = total;
        st.total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() -
                                                                ps->t0)
                          .count();
        if (stats) *stats = st;
        status = total > ps->capacity ? TDS_E_OVERFLOW : TDS_OK;
    }
    (void)hipEventDestroy(ps->done);
    release(ps->idx, w);
    delete ps;
    return status;
}

// Checks that the requests tile [0, nq) in order and their output slices fit.
int validate_requests(const tds_request* reqs, uint32_t nreq, uint64_t nq, uint64_t out_cap) {
    if (!reqs || nreq == 0) return TDS_E_INVALID;
    uint64_t next = 0;
    for (uint32_t r = 0; r < nreq; ++r) {
        const tds_request& q = reqs[r];
        if (q.q_begin != next || q.q_count == 0) return TDS_E_INVALID;
        next += q.q_count;
        if (!valid_window(q.d, q.t_start, q.t_end)) return TDS_E_INVALID;
        if (q.out_offset > out_cap || q.out_capacity > out_cap - q.out_offset) return TDS_E_INVALID;
    }
    return next == nq ? TDS_OK : TDS_E_INVALID;
}

int batch_impl(tds_index* idx, const tds_segments* Q, const tds_request* reqs, uint32_t nreq,
               tds_result* out, uint64_t out_capacity, uint64_t* counts,
               const tds_search_params* params, hipStream_t s, tds_stats* stats) {
    const auto t_begin = std::chrono::steady_clock::now();
    if (!idx || !counts || (out_capacity && !out)) return TDS_E_INVALID;
    TDS_TRY(validate_segments_args(Q));
    TDS_TRY(validate_requests(reqs, nreq, Q->n, out_capacity));
    tds_search_params P;
    tds_search_params_default(&P);
    if (params) P = *params;
    const int prec = resolve_prec(P.precision);
    if (prec < 0) return TDS_E_INVALID;
    const uint32_t chunk = resolve_chunk(prec, P.chunk);
    const uint32_t grid_waves = resolve_grid(P.grid_waves);
    const uint32_t cpl = resolve_tile(P.tile, P.refine, P.deal);
    if (!cpl) return TDS_E_INVALID;
    if (P.output > TDS_OUTPUT_STAGED) return TDS_E_INVALID;
    const bool dev_out = P.out_on_device != 0;

    Workspace* w = acquire(idx);
    if (!w) return TDS_E_NOMEM;
    WsGuard guard{idx, w, s};
    TDS_TRY(ws_reserve(w, Q->n, nreq));
    QueryView V{};
    TDS_TRY(stage_queries(Q, &V, s, &w->qstage, &w->stage_cap, &w->qtraj_stage, &w->traj_cap,
                          &w->pin));
    tds_result* res = out;
    if (!dev_out) {
        TDS_TRY(grow(&w->res, &w->res_cap, (size_t)std::max<uint64_t>(out_capacity, 1)));
        res = w->res;
    }
    Request* R = w->req_host;
    for (uint32_t r = 0; r < nreq; ++r) {
        R[r].q_begin = reqs[r].q_begin;
        R[r].q_count = reqs[r].q_count;
        R[r].d = reqs[r].d;
        R[r].t_start = reqs[r].t_start;
        R[r].t_end = reqs[r].t_end;
        R[r].out_offset = reqs[r].out_offset;
        R[r].out_capacity = reqs[r].out_capacity;
        R[r].pad = 0;
    }
    tds_stats st{};
    st.query_segments = Q->n;
    SearchHeader h{};
    TDS_TRY(run_batch(idx, w, V, nreq, prec, chunk, grid_waves, cpl, P.output, res, s, &st,
                      &h));
    const ReqCounter* rc = w->rc_host;
    int status = TDS_OK;
    uint64_t total = 0;
    for (uint32_t r = 0; r < nreq; ++r) {
        counts[r] = rc[r].count;
        total += rc[r].count;
        if (rc[r].count > reqs[r].out_capacity) status = TDS_E_OVERFLOW;
        if (!dev_out) {
            const uint64_t k = std::min<uint64_t>(rc[r].count, reqs[r].out_capacity);
            if (k)
                TDS_HIP(hipMemcpyAsync(out + reqs[r].out_offset, res + reqs[r].out_offset,
                                       k * sizeof(tds_result), hipMemcpyDeviceToHost, s));
        }
    }
    if (!dev_out) TDS_HIP(hipStreamSynchronize(s));
    guard.idle = true;
    st.active_segments = h.active;
    st.work_items = h.n_items;
    st.candidate_tests = h.tests;
    st.filter_tests = h.ftests;
    st.block_tests = h.btests;
    st.fp64_evals = h.evals;
    st.stage_flushes = h.flushes;
    st.results = total;
    st.total_ms =
        std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_begin).count();
    if (stats) *stats = st;
    {
        std::lock_guard<std::mutex> g(idx->mu);
        idx->last = st;
    }
    return status;
}

}  // namespace tds
