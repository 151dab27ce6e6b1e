// Fixed spatial grid (FSG) index and search: the spatial method of Sec. 4.1
// (Alg. 1), built over the entries of a temporal index.
//
// Build: the entries' boxes (start and canonical end position, grown by a
// relative 1e-9) are reduced to the grid extent; each entry's cell range is
// counted, the counts scanned, and one (cell, entry position) listing written
// per overlapped cell; a radix sort by cell groups the listings, and a dense
// table gives each cell's first listing (cells are few enough, at most 2^24,
// for a dense table instead of the paper's searched array of non-empty cells).
//
// Search: a workgroup prepares a batch of query segments for each of its waves
// (canonical data, cells overlapped by the box grown by d, and the range of
// entry positions that may overlap in time).  A wave lays the runs of listings of
// its batch's cells (cells that are neighbours along x hold consecutive listings)
// end to end, tests them 64 at a time by entry position, queues the pairs that
// stay and evaluates them 64 at a time with the canonical FP64 code.  A pair listed
// in several of the visited cells is reported only from the lowest cell of the
// intersection of the two cell ranges, so no duplicates are produced (the paper
// removed them on the host afterwards).
#include <algorithm>
#include <chrono>
#include <cmath>

#include <hip/hip_ext.h>

#include "canon.hpp"
#include "radix_sort.hpp"
#include "schedule.hpp"
#include "tds_internal.hpp"

namespace tds {

namespace {

constexpr int kFT = 256;

struct Grid {
    uint32_t g[3];
    double lo[3], cw[3];
};

// Bounding box of an entry: its start point and its canonical end position,
// grown by a relative 1e-9 (covers the rounding of every position the
// canonical evaluation forms along the segment).
__device__ inline void entry_box(const EntryF64& e, double* lo, double* hi) {
    const double dt = e.te - e.ts;
    const double p0[3] = {e.x, e.y, e.z};
    const double p1[3] = {e.x + e.vx * dt, e.y + e.vy * dt, e.z + e.vz * dt};
    for (int a = 0; a < 3; ++a) {
        const double l = dmin(p0[a], p1[a]), h = dmax(p0[a], p1[a]);
        const double m = 1e-9 * (fabs(l) + fabs(h) + 1.0);
        lo[a] = l - m;
        hi[a] = h + m;
    }
}

__device__ inline uint32_t cell_of(double v, double lo, double cw, uint32_t g) {
    if (!(cw > 0.0)) return 0u;
    const double u = floor((v - lo) / cw);
    if (!(u > 0.0)) return 0u;
    if (u >= (double)(g - 1)) return g - 1;
    return (uint32_t)u;
}

// Cell range of a box; a NaN bound (a position formed from an infinite
// velocity times zero) widens the range to the edge of the grid.
__device__ inline void cell_range(const Grid& G, const double* lo, const double* hi, uint32_t* c0,
                                  uint32_t* c1) {
    for (int a = 0; a < 3; ++a) {
        c0[a] = isnan(lo[a]) ? 0u : cell_of(lo[a], G.lo[a], G.cw[a], G.g[a]);
        c1[a] = isnan(hi[a]) ? G.g[a] - 1 : cell_of(hi[a], G.lo[a], G.cw[a], G.g[a]);
    }
}

// Per-block partial extents of the entry boxes (min lo, max hi per axis).
__global__ __launch_bounds__(kFT) void k_fsg_extent(const EntryF64* __restrict__ e64, uint32_t n,
                                                    double* __restrict__ part) {
    __shared__ double sp[6][kFT];
    const uint32_t i = blockIdx.x * kFT + threadIdx.x;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (i < n) entry_box(e64[i], lo, hi);
    for (int a = 0; a < 3; ++a) {
        sp[a][threadIdx.x] = lo[a];
        sp[3 + a][threadIdx.x] = hi[a];
    }
    __syncthreads();
    for (uint32_t off = kFT / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off)
            for (int a = 0; a < 3; ++a) {
                sp[a][threadIdx.x] = fmin(sp[a][threadIdx.x], sp[a][threadIdx.x + off]);
                sp[3 + a][threadIdx.x] = fmax(sp[3 + a][threadIdx.x], sp[3 + a][threadIdx.x + off]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[6 * blockIdx.x + threadIdx.x] = sp[threadIdx.x][0];
}

// Number of cells each entry is listed in (kEmit false), or its listings
// written from its offset (kEmit true).
template <bool kEmit>
__global__ __launch_bounds__(kFT) void k_fsg_list(const EntryF64* __restrict__ e64, uint32_t n,
                                                  Grid G, uint32_t* __restrict__ cnt,
                                                  uint64_t* __restrict__ keys,
                                                  uint32_t* __restrict__ vals) {
    const uint32_t i = blockIdx.x * kFT + threadIdx.x;
    if (i >= n) return;
    double lo[3], hi[3];
    entry_box(e64[i], lo, hi);
    uint32_t c0[3], c1[3];
    cell_range(G, lo, hi, c0, c1);
    if (!kEmit) {
        cnt[i] = (c1[0] - c0[0] + 1) * (c1[1] - c0[1] + 1) * (c1[2] - c0[2] + 1);
        return;
    }
    uint32_t o = cnt[i];
    for (uint32_t z = c0[2]; z <= c1[2]; ++z)
        for (uint32_t y = c0[1]; y <= c1[1]; ++y)
            for (uint32_t x = c0[0]; x <= c1[0]; ++x) {
                keys[o] = ((uint64_t)z * G.g[1] + y) * G.g[0] + x;
                vals[o] = i;
                ++o;
            }
}

// first[c] = number of listings with a cell below c (c = 0..ncells): one
// thread per cell, a binary search of the sorted cell keys.
__global__ __launch_bounds__(kFT) void k_fsg_cell_first(const uint32_t* __restrict__ k0,
                                                        const uint32_t* __restrict__ k1,
                                                        const SortControl* __restrict__ ctl,
                                                        uint32_t nl, uint32_t ncells,
                                                        uint32_t* __restrict__ first) {
    const uint32_t* keys = ctl->side() ? k1 : k0;
    const uint32_t c = blockIdx.x * kFT + threadIdx.x;
    if (c > ncells) return;
    uint32_t l = 0, h = nl;
    while (l < h) {
        const uint32_t mid = l + (h - l) / 2;
        if (keys[mid] < c) l = mid + 1;
        else h = mid;
    }
    first[c] = l;
}

// The sorted listings, from the sort's side that holds them.
__global__ __launch_bounds__(kFT) void k_fsg_take(const uint32_t* __restrict__ v0,
                                                  const uint32_t* __restrict__ v1,
                                                  const SortControl* __restrict__ ctl, uint32_t nl,
                                                  uint32_t* __restrict__ list) {
    const uint64_t i = (uint64_t)blockIdx.x * kFT + threadIdx.x;
    if (i < nl) list[i] = ctl->side() ? v1[i] : v0[i];
}

constexpr uint32_t kFTested = 16, kFLine = 16;
constexpr uint32_t kFCounters = (1 + kFTested) * kFLine;

struct FsgArgs {
    Grid G;
    IndexView I;
    const uint32_t* cell_first;
    const uint32_t* list;
    const double* q[8];  // xs, ys, zs, ts, xe, ye, ze, te (device)
    const uint32_t* qtraj;
    uint32_t nq;
    uint32_t batch;      // query segments a wave takes at a time, at most kFQ
    double d, t_start, t_end;
    tds_result* out;
    uint64_t capacity;
    // [0] results, [1] invalid input; then on kFTested lines of their own parts
    // of the number of listings compared
    unsigned long long* counters;
};

__device__ inline uint64_t lanemask_below() {
    const uint32_t lane = __lane_id();
    return (lane == 0) ? 0ull : (~0ull >> (64 - lane));
}

// Keeps LDS traffic of one wave in program order around cross-lane exchange.
__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A query segment of the wave's batch: its canonical data, cell range and
// candidate range (positions of the entries that may overlap it in time).
struct FsgQuery {
    QCanon c;
    uint32_t q0[3], nx, ny;  // lowest cell; cells along x and y
    uint32_t lo, hi;
    uint32_t qid, qtraj;
    uint32_t rows;           // rows of cells along x (ny times its cells along z)
};

// A pair to evaluate: the entry, its listing and the row it was found in.
struct FsgPair {
    uint32_t pos, i, cell, q;  // cell: first of the grid's row; q: query of the batch
};

constexpr int kFS = 256;           // threads of the search's workgroups
constexpr uint32_t kFQ = 16;       // query segments of a batch
constexpr uint32_t kFU = 4;        // listings per lane in flight
constexpr uint32_t kFOut = 128;    // results a workgroup keeps until its end

struct FsgWave {
    FsgQuery q[kFQ];
    FsgPair pair[2 * kWave];
    uint32_t pre[kWave];                  // listings before row r of the step
    uint32_t first[kWave], cell[kWave];   // first listing of row r, first cell of its grid row
    uint32_t rq[kWave];                   // its query
    uint32_t qrow[kFQ];                   // rows before query j
};

struct FsgOut {
    tds_result r[kFOut];
    uint32_t n;
    unsigned long long tested, base;
};

// Evaluates the last min(n, 64) pairs.  An entry listed in several of the
// query's cells counts only in the lowest cell of the intersection of the two
// cell ranges.
__device__ inline void fsg_drain(const FsgArgs& A, FsgWave& W, FsgOut& O, uint32_t& n) {
    const uint32_t lane = __lane_id();
    const uint32_t cnt = min(n, (uint32_t)kWave);
    n -= cnt;
    wave_fence();
    bool hit = false;
    double t_lo = 0.0, t_hi = 0.0;
    FsgPair p = {0, 0, 0, 0};
    if (lane < cnt) {
        p = W.pair[n + lane];
        const FsgQuery& Q = W.q[p.q];
        const EntryF64 E = A.I.e64[p.pos];
        if (E.ts < Q.c.bq && E.te > Q.c.aq) {
            double el[3], eh[3];
            entry_box(E, el, eh);
            uint32_t e0[3], e1[3];
            cell_range(A.G, el, eh, e0, e1);
            const uint32_t row =
                (max(Q.q0[2], e0[2]) * A.G.g[1] + max(Q.q0[1], e0[1])) * A.G.g[0];
            if (row == p.cell) {
                const uint32_t c = row + max(Q.q0[0], e0[0]);
                hit = A.cell_first[c] <= p.i && p.i < A.cell_first[c + 1] &&
                      canon_eval<true>(Q.c, E.x, E.y, E.z, E.vx, E.vy, E.vz, E.ts, E.te, &t_lo,
                                       &t_hi);
            }
        }
    }
    const uint64_t hm = __ballot(hit);
    if (!hm) return;
    const uint32_t nh = (uint32_t)__popcll(hm), rank = (uint32_t)__popcll(hm & lanemask_below());
    tds_result r;
    if (hit) {
        r.q_seg = W.q[p.q].qid;
        r.e_seg = A.I.seg_id[p.pos];
        r.q_traj = W.q[p.q].qtraj;
        r.e_traj = A.I.traj[p.pos];
        r.t_lo = t_lo;
        r.t_hi = t_hi;
    }
    // into the workgroup's buffer, those past its end straight to the output
    uint32_t at = 0;
    if (lane == 0) at = *(volatile uint32_t*)&O.n < kFOut ? atomicAdd(&O.n, nh) : kFOut;
    at = __shfl(at, 0);
    if (hit && at + rank < kFOut) O.r[at + rank] = r;
    const uint32_t kept = min(nh, at < kFOut ? kFOut - at : 0u);
    if (kept == nh) return;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&A.counters[0], (unsigned long long)(nh - kept));
    base = __shfl(base, 0);
    if (hit && rank >= kept && base + (rank - kept) < A.capacity) A.out[base + (rank - kept)] = r;
}

// A workgroup takes `batch` consecutive query segments for each of its waves:
// first, one per thread, what is done once per segment, its canonical data,
// cell range, and the range of entry positions that may overlap it in time
// (from the index's bins), then a wave each its batch.  The cells of a query
// that are neighbours along x hold consecutive listings, so its cells
// are (cells along y) x (cells along z) runs of listings; the runs of the batch
// are laid end to end, 64 at a time, and their listings tested 64 at a time,
// full waves whatever the cells hold.  A listing is four bytes, read in order,
// and its entry position decides by the range whether the entry is read at all
// (one in a hundred where a segment lasts 1 / 400 of the data's time span).
// Pairs that stay are queued and evaluated 64 at a time.
//
// With a wave per query, one cell after another (three dependent loads each,
// the 64-byte entry for every listing), 200,000 segments in 50^3 cells of a
// million entries (13 million listings) took 311 us, nearly all latency; this
// takes 105, about 45 of it the latency of a workgroup's chain and the last
// ones' end, and the number of listings in flight, of workgroups and of query
// segments to a batch hardly change it.  Results are collected per workgroup:
// a returning atomic on one counter takes 30 ns of the chip's time, one per
// wave and evaluation would be most of the kernel.
__global__ __launch_bounds__(kFS) void k_fsg_search(FsgArgs A) {
    __shared__ FsgWave waves[kFS / kWave];
    __shared__ FsgOut O;
    if (threadIdx.x == 0) {
        O.n = 0;
        O.tested = 0;
    }
    __syncthreads();
    const uint32_t lane = __lane_id(), t = threadIdx.x;
    FsgWave& W = waves[t / kWave];
    const uint32_t per = A.batch * (kFS / kWave);  // query segments of the workgroup at a time
    unsigned long long tested = 0;
    for (uint64_t k0 = (uint64_t)blockIdx.x * per; k0 < A.nq; k0 += (uint64_t)gridDim.x * per) {
        const uint64_t kk = k0 + t;
        if (t < per) {
            const uint32_t k = (uint32_t)kk;
            uint32_t rows = 0;
            if (kk < A.nq) {
                const double xs = A.q[0][k], ys = A.q[1][k], zs = A.q[2][k], ts = A.q[3][k];
                const double xe = A.q[4][k], ye = A.q[5][k], ze = A.q[6][k], te = A.q[7][k];
                FsgQuery Q;
                QCanon& q = Q.c;
                if (!(isfinite(xs) && isfinite(ys) && isfinite(zs) && isfinite(ts) && isfinite(xe) &&
                      isfinite(ye) && isfinite(ze) && isfinite(te) && te > ts)) {
                    atomicAdd(&A.counters[1], 1ull);
                } else {
                    // the canonical query data (the same operations as every
                    // search form)
                    const double dt = te - ts;
                    q.x = xs;
                    q.y = ys;
                    q.z = zs;
                    q.vx = (xe - xs) / dt;
                    q.vy = (ye - ys) / dt;
                    q.vz = (ze - zs) / dt;
                    q.ts = ts;
                    q.aq = dmax(ts, A.t_start);
                    q.bq = dmin(te, A.t_end);
                    q.d = A.d;
                    if (q.aq < q.bq) {
                        // the query's box over its clipped extent, grown by d (+
                        // rounding room)
                        const double pa[3] = {q.x + q.vx * (q.aq - ts), q.y + q.vy * (q.aq - ts),
                                              q.z + q.vz * (q.aq - ts)};
                        const double pb[3] = {q.x + q.vx * (q.bq - ts), q.y + q.vy * (q.bq - ts),
                                              q.z + q.vz * (q.bq - ts)};
                        double lo[3], hi[3];
                        for (int a = 0; a < 3; ++a) {
                            const double l = dmin(pa[a], pb[a]), h = dmax(pa[a], pb[a]);
                            const double m = q.d + 1e-9 * (fabs(l) + fabs(h) + q.d + 1.0);
                            lo[a] = l - m;
                            hi[a] = h + m;
                        }
                        uint32_t q1[3], j0, j1;
                        cell_range(A.G, lo, hi, Q.q0, q1);
                        Q.nx = q1[0] - Q.q0[0] + 1;
                        Q.ny = q1[1] - Q.q0[1] + 1;
                        rows = Q.ny * (q1[2] - Q.q0[2] + 1);
                        cand_range(A.I, q.aq, q.bq, &Q.lo, &Q.hi, &j0, &j1);
                        Q.qid = k;
                        Q.qtraj = A.qtraj ? A.qtraj[k] : 0u;
                        Q.rows = rows;
                        waves[t / A.batch].q[t % A.batch] = Q;
                    }
                }
            }
            waves[t / A.batch].qrow[t % A.batch] = rows;
        }
        __syncthreads();
        const uint32_t rows = lane < A.batch ? W.qrow[lane] : 0u;
        wave_fence();
        // rows of the queries before each
        uint32_t inc = rows;
        for (uint32_t off = 1; off < kFQ; off <<= 1) {
            const uint32_t v = __shfl_up(inc, off);
            if (lane >= off) inc += v;
        }
        if (lane < kFQ) W.qrow[lane] = inc - rows;
        const uint32_t total = __shfl(inc, kFQ - 1);
        wave_fence();
        uint32_t np = 0;
        for (uint32_t r0 = 0; r0 < total;) {
            // up to 64 rows: their listings
            const uint32_t r = r0 + lane;
            uint32_t len = 0, first = 0, cell = 0, ql = 0;
            if (r < total) {
                for (uint32_t h = kFQ / 2; h; h >>= 1)
                    if (W.qrow[ql + h] <= r) ql += h;
                const FsgQuery& Q = W.q[ql];
                const uint32_t x = r - W.qrow[ql], z = x / Q.ny, y = x - z * Q.ny;
                cell = ((Q.q0[2] + z) * A.G.g[1] + Q.q0[1] + y) * A.G.g[0];
                first = A.cell_first[cell + Q.q0[0]];
                len = A.cell_first[cell + Q.q0[0] + Q.nx] - first;
            }
            uint64_t sum = len;
            for (uint32_t off = 1; off < (uint32_t)kWave; off <<= 1) {
                const uint64_t v = __shfl_up(sum, off);
                if (lane >= off) sum += v;
            }
            // all of them, or one if their listings' number passes 32 bits
            uint32_t step = kWave;
            uint64_t all = __shfl(sum, kWave - 1);
            if (all >> 31) {
                step = 1;
                all = __shfl(sum, 0);
                if (lane) sum = all + len;  // past the end
            }
            wave_fence();
            W.pre[lane] = (uint32_t)(sum - len);
            W.first[lane] = first;
            W.cell[lane] = cell;
            W.rq[lane] = ql;
            wave_fence();
            r0 += step;
            tested += all;
            for (uint64_t x0 = 0; x0 < all; x0 += kFU * kWave) {
                uint32_t row[kFU], li[kFU], pos[kFU];
                bool in[kFU];
#pragma unroll
                for (uint32_t u = 0; u < kFU; ++u) {
                    const uint64_t x = x0 + u * kWave + lane;
                    in[u] = x < all;
                    // the last row with at most x listings before it
                    row[u] = 0;
                    if (step == kWave)
                        for (uint32_t h = kWave / 2; h; h >>= 1)
                            if (W.pre[row[u] + h] <= (uint32_t)x) row[u] += h;
                    li[u] = in[u] ? W.first[row[u]] + (uint32_t)(x - W.pre[row[u]]) : 0u;
                }
#pragma unroll
                for (uint32_t u = 0; u < kFU; ++u) pos[u] = A.list[li[u]];
#pragma unroll
                for (uint32_t u = 0; u < kFU; ++u) {
                    const uint32_t ql = W.rq[row[u]];
                    in[u] = in[u] && pos[u] >= W.q[ql].lo && pos[u] < W.q[ql].hi;
                    const uint64_t m = __ballot(in[u]);
                    if (!m) continue;
                    if (in[u]) {
                        const FsgPair p = {pos[u], li[u], W.cell[row[u]], ql};
                        W.pair[np + (uint32_t)__popcll(m & lanemask_below())] = p;
                    }
                    np += (uint32_t)__popcll(m);
                    if (np >= (uint32_t)kWave) fsg_drain(A, W, O, np);
                }
            }
        }
        while (np) fsg_drain(A, W, O, np);
        __syncthreads();
    }
    // listings compared, and the workgroup's results
    if (lane == 0 && tested) atomicAdd(&O.tested, tested);
    __syncthreads();
    const uint32_t n = min(O.n, kFOut);
    if (threadIdx.x == 0) {
        if (O.tested)
            atomicAdd(&A.counters[(1 + blockIdx.x % kFTested) * kFLine], O.tested);
        if (n) O.base = atomicAdd(&A.counters[0], (unsigned long long)n);
    }
    __syncthreads();
    if (t < n && O.base + t < A.capacity) A.out[O.base + t] = O.r[t];
}

void free_scratch(FsgScratch& x) {
    dfree(x.ctr);
    if (x.ctr_host) (void)hipHostFree(x.ctr_host);
    if (x.e0) (void)hipEventDestroy(x.e0);
    if (x.e1) (void)hipEventDestroy(x.e1);
    x = {};
}

// A search's counters and events, from the grid's pool or new, given back (or
// freed, past kFsgPool) at the end: once the search has waited for its stream
// (`idle`), or after that wait here.
struct ScratchLease {
    const tds_fsg* f;
    hipStream_t s;
    FsgScratch x;
    bool idle = false;
    ScratchLease(const tds_fsg* g, hipStream_t stream) : f(g), s(stream) {
        std::lock_guard<std::mutex> l(f->mu);
        if (f->npool) x = f->pool[--f->npool];
    }
    int ready() {
        if (x.e1) return TDS_OK;
        TDS_TRY(dmalloc(&x.ctr, kFCounters));
        TDS_HIP(hipHostMalloc((void**)&x.ctr_host, kFCounters * sizeof(unsigned long long),
                              hipHostMallocDefault));
        TDS_HIP(hipEventCreate(&x.e0));
        TDS_HIP(hipEventCreate(&x.e1));
        return TDS_OK;
    }
    ~ScratchLease() {
        if (!idle) (void)hipStreamSynchronize(s);
        {
            std::lock_guard<std::mutex> l(f->mu);
            if (x.e1 && f->npool < kFsgPool) {
                f->pool[f->npool++] = x;
                return;
            }
        }
        free_scratch(x);
    }
};

struct Bufs {
    void* p[8] = {};
    ~Bufs() {
        for (void* q : p) dfree(q);
    }
};

}  // namespace

int fsg_build(const tds_index* idx, uint32_t gx, uint32_t gy, uint32_t gz, hipStream_t s,
              tds_fsg** out) {
    if (!idx || !out) return TDS_E_INVALID;
    *out = nullptr;
    const uint32_t g[3] = {gx ? gx : 50u, gy ? gy : 50u, gz ? gz : 50u};
    for (uint32_t v : g)
        if (v > 1024) return TDS_E_INVALID;
    const uint64_t ncells = (uint64_t)g[0] * g[1] * g[2];
    if (ncells > (1ull << 24)) return TDS_E_INVALID;
    const uint32_t n = (uint32_t)idx->n;
    const uint32_t nb = ceil_div(n, kFT);
    Bufs B;
    double* part = nullptr;
    TDS_TRY(dmalloc(&part, 6 * (size_t)nb));
    B.p[0] = part;
    hipLaunchKernelGGL(k_fsg_extent, dim3(nb), dim3(kFT), 0, s, idx->e64, n, part);
    TDS_HIP(hipGetLastError());
    std::vector<double> hp(6 * (size_t)nb);
    TDS_HIP(hipMemcpyAsync(hp.data(), part, hp.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    TDS_HIP(hipStreamSynchronize(s));
    Grid G;
    for (int a = 0; a < 3; ++a) {
        double lo = INFINITY, hi = -INFINITY;
        for (uint32_t b = 0; b < nb; ++b) {
            lo = std::fmin(lo, hp[6 * b + a]);
            hi = std::fmax(hi, hp[6 * b + 3 + a]);
        }
        G.g[a] = g[a];
        G.lo[a] = lo;
        const double w = (hi - lo) / (double)g[a];
        G.cw[a] = (std::isfinite(w) && w > 0.0) ? w : 0.0;
    }
    uint32_t* cnt = nullptr;
    TDS_TRY(dmalloc(&cnt, n));
    B.p[1] = cnt;
    hipLaunchKernelGGL(k_fsg_list<false>, dim3(nb), dim3(kFT), 0, s, idx->e64, n, G, cnt, nullptr,
                       nullptr);
    TDS_HIP(hipGetLastError());
    // the listing total must fit 32 bits: check with a 64-bit host sum
    {
        std::vector<uint32_t> hc(n);
        TDS_HIP(hipMemcpyAsync(hc.data(), cnt, n * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
        TDS_HIP(hipStreamSynchronize(s));
        uint64_t tot = 0;
        for (uint32_t c : hc) tot += c;
        if (tot >= 0xFFFFFFFFull) return TDS_E_NOMEM;
    }
    uint32_t nl = 0;
    TDS_TRY(exclusive_scan_u32(cnt, n, &nl, s));
    uint64_t *keys = nullptr, *keys2 = nullptr, *status = nullptr;
    uint32_t *vals = nullptr, *vals2 = nullptr, *list = nullptr;
    SortControl* ctl = nullptr;
    const uint32_t na = std::max<uint32_t>(nl, 1);
    TDS_TRY(dmalloc(&keys, na));
    B.p[2] = keys;
    TDS_TRY(dmalloc(&keys2, na));
    B.p[3] = keys2;
    TDS_TRY(dmalloc(&vals, na));
    B.p[4] = vals;
    TDS_TRY(dmalloc(&vals2, na));
    B.p[5] = vals2;
    TDS_TRY(dmalloc(&status, sort_status_len(na)));
    B.p[6] = status;
    TDS_TRY(dmalloc(&ctl, 1));
    B.p[7] = ctl;
    int bits = 1;
    while ((1ull << bits) < ncells) ++bits;
    // cell numbers fit 32 bits (at most 2^24 cells); an entry's listings are
    // written from its offset, so its position is the value to carry
    const SortJob sort{nl, keys, vals, keys, keys2, vals, vals2, ctl, status};
    TDS_TRY(sort_clear(sort, s));
    hipLaunchKernelGGL(k_fsg_list<true>, dim3(nb), dim3(kFT), 0, s, idx->e64, n, G, cnt, keys, vals);
    TDS_TRY(sort_plan(sort, bits, s));
    TDS_TRY(sort_passes(sort, sort_npass(bits), true, s));
    int st = dmalloc(&list, na);
    uint32_t* first = nullptr;
    if (st == TDS_OK) st = dmalloc(&first, ncells + 1);
    if (st == TDS_OK) {
        const uint32_t* k1 = reinterpret_cast<const uint32_t*>(keys2);
        hipLaunchKernelGGL(k_fsg_cell_first, dim3(ceil_div(ncells + 1, kFT)), dim3(kFT), 0, s,
                           k1 + nl, k1, ctl, nl, (uint32_t)ncells, first);
        hipLaunchKernelGGL(k_fsg_take, dim3(ceil_div(na, kFT)), dim3(kFT), 0, s, vals, vals2, ctl,
                           nl, list);
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            st = TDS_E_DEVICE;
    }
    tds_fsg* f = (st == TDS_OK) ? new (std::nothrow) tds_fsg() : nullptr;
    if (!f) {
        dfree(list);
        dfree(first);
        return st == TDS_OK ? TDS_E_NOMEM : st;
    }
    f->idx = idx;
    f->device = idx->device;
    for (int a = 0; a < 3; ++a) {
        f->g[a] = G.g[a];
        f->lo[a] = G.lo[a];
        f->cw[a] = G.cw[a];
    }
    f->cell_first = first;
    f->list = list;
    f->nlist = nl;
    *out = f;
    return TDS_OK;
}

void fsg_destroy(tds_fsg* f) {
    if (!f) return;
    for (size_t i = 0; i < f->npool; ++i) free_scratch(f->pool[i]);
    dfree(f->cell_first);
    dfree(f->list);
    delete f;
}

int fsg_search(const tds_fsg* f, const tds_segments* Q, double d, double t_start, double t_end,
               tds_result* out, uint64_t capacity, uint64_t* n_out, const tds_search_params* params,
               hipStream_t s, tds_stats* stats) {
    const auto t_begin = std::chrono::steady_clock::now();
    if (!f || !n_out) return TDS_E_INVALID;
    *n_out = 0;
    TDS_TRY(validate_segments_args(Q));
    if (!(d >= 0.0) || std::isinf(d) || !(t_start < t_end)) return TDS_E_INVALID;
    if (capacity > 0 && !out) return TDS_E_INVALID;
    tds_search_params P;
    tds_search_params_default(&P);
    if (params) P = *params;
    const bool dev_out = P.out_on_device != 0;
    const uint64_t nq = Q->n;
    Bufs B;
    FsgArgs A{};
    A.G.g[0] = f->g[0];
    A.G.g[1] = f->g[1];
    A.G.g[2] = f->g[2];
    for (int a = 0; a < 3; ++a) {
        A.G.lo[a] = f->lo[a];
        A.G.cw[a] = f->cw[a];
    }
    A.I = view_of(f->idx);
    A.cell_first = f->cell_first;
    A.list = f->list;
    const double* src[8] = {Q->xs, Q->ys, Q->zs, Q->ts, Q->xe, Q->ye, Q->ze, Q->te};
    if (Q->on_device) {
        for (int k = 0; k < 8; ++k) A.q[k] = src[k];
        A.qtraj = Q->traj_id;
    } else {
        double* stage = nullptr;
        TDS_TRY(dmalloc(&stage, 8 * nq));
        B.p[0] = stage;
        for (int k = 0; k < 8; ++k) {
            TDS_HIP(hipMemcpyAsync(stage + k * nq, src[k], nq * sizeof(double),
                                   hipMemcpyHostToDevice, s));
            A.q[k] = stage + k * nq;
        }
        A.qtraj = nullptr;
        if (Q->traj_id) {
            uint32_t* tr = nullptr;
            TDS_TRY(dmalloc(&tr, nq));
            B.p[1] = tr;
            TDS_HIP(hipMemcpyAsync(tr, Q->traj_id, nq * sizeof(uint32_t), hipMemcpyHostToDevice, s));
            A.qtraj = tr;
        }
    }
    A.nq = (uint32_t)nq;
    A.d = d;
    A.t_start = t_start;
    A.t_end = t_end;
    A.capacity = capacity;
    if (dev_out) {
        A.out = out;
    } else {
        tds_result* res = nullptr;
        TDS_TRY(dmalloc(&res, std::max<uint64_t>(capacity, 1)));
        B.p[2] = res;
        A.out = res;
    }
    ScratchLease lease(f, s);
    TDS_TRY(lease.ready());
    A.counters = lease.x.ctr;
    TDS_HIP(hipMemsetAsync(A.counters, 0, kFCounters * sizeof(unsigned long long), s));
    // batches of up to kFQ query segments, smaller ones while there are fewer
    // than the waves that the chip holds (4 to a workgroup of 24 KB of LDS)
    A.batch = (uint32_t)std::min<uint64_t>(kFQ, std::max<uint64_t>(1, nq / 8192));
    const uint32_t blocks =
        std::max(1u, std::min(ceil_div(ceil_div(nq, A.batch), kFS / kWave), 4096u));
    hipExtLaunchKernelGGL(k_fsg_search, dim3(blocks), dim3(kFS), 0, s, lease.x.e0,
                          lease.x.e1, 0u, A);
    const unsigned long long* h = lease.x.ctr_host;
    int st = (hipGetLastError() == hipSuccess) ? TDS_OK : TDS_E_DEVICE;
    if (st == TDS_OK &&
        hipMemcpyAsync(lease.x.ctr_host, A.counters, kFCounters * sizeof(unsigned long long),
                       hipMemcpyDeviceToHost, s) != hipSuccess)
        st = TDS_E_DEVICE;
    if (st == TDS_OK && hipStreamSynchronize(s) != hipSuccess) st = TDS_E_DEVICE;
    lease.idle = st == TDS_OK;
    float ms = 0.f;
    if (st == TDS_OK) (void)hipEventElapsedTime(&ms, lease.x.e0, lease.x.e1);
    TDS_TRY(st);
    if (h[1]) return TDS_E_INVALID;
    uint64_t tested = 0;
    for (uint32_t i = 1; i <= kFTested; ++i) tested += h[i * kFLine];
    *n_out = h[0];
    if (!dev_out) {
        const uint64_t k = std::min<uint64_t>(h[0], capacity);
        if (k) {
            TDS_HIP(hipMemcpyAsync(out, A.out, k * sizeof(tds_result), hipMemcpyDeviceToHost, s));
            TDS_HIP(hipStreamSynchronize(s));
        }
    }
    if (stats) {
        tds_stats st2{};
        st2.query_segments = nq;
        st2.candidate_tests = tested;
        st2.filter_tests = tested;
        st2.results = h[0];
        st2.passes = 1;
        st2.kernel_ms = ms;
        st2.total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() -
                                                                 t_begin)
                           .count();
        *stats = st2;
    }
    return h[0] > capacity ? TDS_E_OVERFLOW : TDS_OK;
}

}  // namespace tds
