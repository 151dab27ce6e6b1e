// Index build on the GPU: the temporal index of Sec. 4.2.1, optionally with
// every temporal bin subdivided in space (the idea of Sec. 4.3).
//
//   k_seg_prep    validate every segment, compute its velocity (IEEE FP64
//                 division), its FP32 bounding-sphere record, its sort key
//                 (order-preserving bits of t_start) and per-block partial
//                 min t_start / max t_end / sum of durations / extent of the
//                 sphere centres;
//   k_spatial_key (spatial layout) replace the key by (bin, Hilbert index of
//                 the sphere centre on a 1024^3 grid over the centres' extent);
//   radix sort    stable, by the key (radix_sort.hip);
//   k_gather      write the ordered AoS records, ids and trajectory ids;
//   k_bin_first   first position of every bin (boundary detection);
//   k_bin_stats   per-bin data extents (min/max t_start, min/max t_end);
//   k_bin_scan    running maximum of max t_end over bins, which makes the
//                 bins overlapping a query one contiguous, bisectable span,
//                 and the minimum t_start over the bins from j on;
//   k_block_box   (spatial layout) box of the segments of every aligned
//                 block of 64 entries.
#include <cmath>
#include <new>
#include <utility>

#include "hilbert.hpp"
#include "radix_sort.hpp"
#include "tds_internal.hpp"

namespace tds {

namespace {

constexpr int kBT = 256;

__device__ inline uint64_t order_key(double t) {
    // order-preserving map of a finite double to u64 (-0 and +0 are equal)
    uint64_t u = (t == 0.0) ? 0ull : (uint64_t)__double_as_longlong(t);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ inline bool finite(double v) { return isfinite(v); }

// Per-block partials written by k_seg_prep: min t_start, max t_end, sum of
// durations, then min and max of the sphere centres per axis.
constexpr int kPart = 9;

__global__ __launch_bounds__(kBT) void k_seg_prep(SegView S, EntryF64* __restrict__ tmp64,
                                                  EntryF32* __restrict__ tmp32,
                                                  uint64_t* __restrict__ keys,
                                                  double* __restrict__ part, uint32_t* err) {
    __shared__ double sp[kPart][kBT];
    const uint32_t tid = threadIdx.x;
    const uint64_t i = (uint64_t)blockIdx.x * kBT + tid;
    double v[kPart] = {INFINITY, -INFINITY, 0.0, INFINITY, -INFINITY,
                       INFINITY, -INFINITY, INFINITY, -INFINITY};
    if (i < S.n) {
        double xs = S.a[0][i], ys = S.a[1][i], zs = S.a[2][i], ts = S.a[3][i];
        double xe = S.a[4][i], ye = S.a[5][i], ze = S.a[6][i], te = S.a[7][i];
        bool ok = finite(xs) && finite(ys) && finite(zs) && finite(ts) && finite(xe) &&
                  finite(ye) && finite(ze) && finite(te) && te > ts;
        if (!ok) {
            atomicOr(err, 1u);
            ts = 0.0;
            te = 1.0;
        }
        double dt = te - ts;
        EntryF64 e;
        e.x = xs;
        e.y = ys;
        e.z = zs;
        e.vx = (xe - xs) / dt;
        e.vy = (ye - ys) / dt;
        e.vz = (ze - zs) / dt;
        e.ts = ts;
        e.te = te;
        tmp64[i] = e;
        EntryF32 f;
        sphere32(xs, ys, zs, xe, ye, ze, 0.0, f.cx, f.cy, f.cz, f.r);
        f.ts = __double2float_rd(ts);
        f.te = __double2float_ru(te);
        f.pad0 = 0.f;
        f.pad1 = 0.f;
        tmp32[i] = f;
        keys[i] = order_key(ts);
        v[0] = ts;
        v[1] = te;
        v[2] = dt;
        v[3] = v[4] = f.cx;
        v[5] = v[6] = f.cy;
        v[7] = v[8] = f.cz;
    }
    for (int k = 0; k < kPart; ++k) sp[k][tid] = v[k];
    __syncthreads();
    for (uint32_t off = kBT / 2; off > 0; off >>= 1) {
        if (tid < off) {
            sp[0][tid] = fmin(sp[0][tid], sp[0][tid + off]);
            sp[1][tid] = fmax(sp[1][tid], sp[1][tid + off]);
            sp[2][tid] = sp[2][tid] + sp[2][tid + off];
            for (int k = 3; k < kPart; k += 2) {
                sp[k][tid] = fmin(sp[k][tid], sp[k][tid + off]);
                sp[k + 1][tid] = fmax(sp[k + 1][tid], sp[k + 1][tid + off]);
            }
        }
        __syncthreads();
    }
    if (tid < kPart) part[kPart * blockIdx.x + tid] = sp[tid][0];
}

// Bin of a t_start: floor((ts - t_min) / b) clamped to [0, m-1].
__device__ inline uint32_t bin_of(double ts, double tmin, double bw, uint32_t m) {
    double u = floor((ts - tmin) / bw);
    if (!(u > 0.0)) return 0u;
    if (u >= (double)(m - 1)) return m - 1;
    return (uint32_t)u;
}

__device__ inline uint32_t cell10(float c, float lo, float scale) {
    const float u = (c - lo) * scale;
    if (!(u > 0.f)) return 0u;
    if (u >= 1023.f) return 1023u;
    return (uint32_t)u;
}

// Spatial layout key: bin in the high bits, then the Hilbert index of the
// sphere centre's cell.  Only the order inside a bin depends on the cell, so
// the bins, and every table derived from them, are those of the temporal
// layout.
__global__ __launch_bounds__(kBT) void k_spatial_key(uint64_t n, const EntryF64* __restrict__ tmp64,
                                                     const EntryF32* __restrict__ tmp32,
                                                     double tmin, double bw, uint32_t m,
                                                     float lx, float ly, float lz, float sx,
                                                     float sy, float sz,
                                                     uint64_t* __restrict__ keys) {
    const uint64_t i = (uint64_t)blockIdx.x * kBT + threadIdx.x;
    if (i >= n) return;
    const EntryF32 f = tmp32[i];
    const uint32_t h =
        hilbert3<10>(cell10(f.cx, lx, sx), cell10(f.cy, ly, sy), cell10(f.cz, lz, sz));
    keys[i] = ((uint64_t)bin_of(tmp64[i].ts, tmin, bw, m) << 30) | h;
}

__global__ __launch_bounds__(kBT) void k_gather(uint64_t n, const uint32_t* __restrict__ v0,
                                                const uint32_t* __restrict__ v1,
                                                const SortControl* __restrict__ ctl,
                                                const EntryF64* __restrict__ tmp64,
                                                const EntryF32* __restrict__ tmp32,
                                                const uint32_t* __restrict__ traj_in,
                                                EntryF64* __restrict__ e64,
                                                EntryF32* __restrict__ e32,
                                                EntryV32* __restrict__ ev32,
                                                uint32_t* __restrict__ seg_id,
                                                uint32_t* __restrict__ traj) {
    const uint64_t i = (uint64_t)blockIdx.x * kBT + threadIdx.x;
    if (i >= n) return;
    const uint32_t src = ctl->side() ? v1[i] : v0[i];
    const EntryF64 e = tmp64[src];
    e64[i] = e;
    e32[i] = tmp32[src];
    ev32[i] = motion32(e.vx, e.vy, e.vz, 0.5 * (e.ts + e.te));
    seg_id[i] = src;
    traj[i] = traj_in ? traj_in[src] : 0u;
}

__global__ __launch_bounds__(kBT) void k_bin_first(uint64_t n, const EntryF64* __restrict__ e64,
                                                   double tmin, double bw, uint32_t m,
                                                   uint32_t* __restrict__ bin_first) {
    const uint64_t i = (uint64_t)blockIdx.x * kBT + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = bin_of(e64[i].ts, tmin, bw, m);
    const int64_t jp = (i == 0) ? -1 : (int64_t)bin_of(e64[i - 1].ts, tmin, bw, m);
    for (int64_t k = jp + 1; k <= (int64_t)j; ++k) bin_first[k] = (uint32_t)i;
    if (i == n - 1)
        for (uint32_t k = j + 1; k <= m; ++k) bin_first[k] = (uint32_t)n;
}

// Per-bin extents: min and max of t_start and of t_end over the bin's
// entries (+inf / -inf when the bin is empty); one block per bin.
__global__ __launch_bounds__(kBT) void k_bin_stats(const EntryF64* __restrict__ e64,
                                                   const uint32_t* __restrict__ bin_first,
                                                   double* __restrict__ min_ts,
                                                   double* __restrict__ max_ts,
                                                   double* __restrict__ min_te,
                                                   double* __restrict__ max_te) {
    __shared__ double sp[4][kBT];
    const uint32_t j = blockIdx.x;
    const uint32_t f = bin_first[j], e = bin_first[j + 1];
    double v[4] = {INFINITY, -INFINITY, INFINITY, -INFINITY};
    for (uint32_t i = f + threadIdx.x; i < e; i += kBT) {
        const double ts = e64[i].ts, te = e64[i].te;
        v[0] = fmin(v[0], ts);
        v[1] = fmax(v[1], ts);
        v[2] = fmin(v[2], te);
        v[3] = fmax(v[3], te);
    }
    for (int k = 0; k < 4; ++k) sp[k][threadIdx.x] = v[k];
    __syncthreads();
    for (uint32_t off = kBT / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            for (int k = 0; k < 4; k += 2) {
                sp[k][threadIdx.x] = fmin(sp[k][threadIdx.x], sp[k][threadIdx.x + off]);
                sp[k + 1][threadIdx.x] = fmax(sp[k + 1][threadIdx.x], sp[k + 1][threadIdx.x + off]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        min_ts[j] = sp[0][0];
        max_ts[j] = sp[1][0];
        min_te[j] = sp[2][0];
        max_te[j] = sp[3][0];
    }
}

// Running extreme over len values with one block of 1024 threads: the
// maximum of v[0..i] (kMax, forward) or the minimum of v[i..len) (reverse).
template <bool kMax>
__global__ __launch_bounds__(1024) void k_bin_scan(const double* __restrict__ v,
                                                   double* __restrict__ out, uint32_t len) {
    __shared__ double part[1024];
    const double id = kMax ? -INFINITY : INFINITY;
    auto op = [](double a, double b) { return kMax ? fmax(a, b) : fmin(a, b); };
    // element k of the scan order: i = k (forward) or len - 1 - k (reverse)
    auto at = [&](uint32_t k) { return kMax ? k : len - 1 - k; };
    const uint32_t tid = threadIdx.x;
    const uint32_t per = (len + 1023) / 1024;
    const uint32_t b = tid * per, e = min(len, b + per);
    double acc = id;
    for (uint32_t k = b; k < e; ++k) acc = op(acc, v[at(k)]);
    part[tid] = acc;
    __syncthreads();
    for (uint32_t off = 1; off < 1024; off <<= 1) {
        const double t = (tid >= off) ? part[tid - off] : id;
        __syncthreads();
        part[tid] = op(part[tid], t);
        __syncthreads();
    }
    double run = (tid > 0) ? part[tid - 1] : id;
    for (uint32_t k = b; k < e; ++k) {
        run = op(run, v[at(k)]);
        out[at(k)] = run;
    }
}

// Box of each aligned block of 64 entries: the union of the entries' segment
// boxes (seg_box32 of the end points the canonical evaluation computes from
// the FP64 record), one wave per block (lanes past n contribute nothing).
__global__ __launch_bounds__(kBT) void k_block_box(uint64_t n, const EntryF64* __restrict__ e64,
                                                   BlockBox* __restrict__ box, uint32_t nblk) {
    const uint32_t blk = blockIdx.x * (kBT / kWave) + threadIdx.x / kWave;
    if (blk >= nblk) return;
    const uint64_t i = ((uint64_t)blk << kBoxShift) + __lane_id();
    Box32 v = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (i < n) {
        const EntryF64 e = e64[i];
        const double dt = e.te - e.ts;
        v = seg_box32(e.x, e.y, e.z, e.x + e.vx * dt, e.y + e.vy * dt, e.z + e.vz * dt, 0.0);
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        v.lx = fminf(v.lx, __shfl_xor(v.lx, off));
        v.ly = fminf(v.ly, __shfl_xor(v.ly, off));
        v.lz = fminf(v.lz, __shfl_xor(v.lz, off));
        v.hx = fmaxf(v.hx, __shfl_xor(v.hx, off));
        v.hy = fmaxf(v.hy, __shfl_xor(v.hy, off));
        v.hz = fmaxf(v.hz, __shfl_xor(v.hz, off));
    }
    if (__lane_id() == 0) {
        BlockBox b;
        b.b = v;
        b.pad0 = 0.f;
        b.pad1 = 0.f;
        box[blk] = b;
    }
}

struct Scratch {
    DeviceBlock block;
    ~Scratch() { release_block(&block); }
};

struct BlockPool {
    std::mutex mu;
    DeviceBlock idle[kPoolBlocks];  // in the order of their release
    size_t n = 0;
    DeviceBlock take(size_t i) {
        const DeviceBlock b = idle[i];
        std::copy(idle + i + 1, idle + n, idle + i);
        --n;
        return b;
    }
    // Takes the most recently released of the device's blocks with which, from
    // the newest on, they hold more than `keep` bytes.
    bool take_past(int device, size_t keep, DeviceBlock* b) {
        std::lock_guard<std::mutex> l(mu);
        size_t sum = 0;
        for (size_t i = n; i-- > 0;) {
            if (idle[i].device != device) continue;
            sum += idle[i].bytes;
            if (sum > keep) {
                *b = take(i);
                return true;
            }
        }
        return false;
    }
};
// never destroyed: at the program's end the runtime may be gone first
BlockPool& block_pool() {
    alignas(BlockPool) static unsigned char mem[sizeof(BlockPool)];
    static BlockPool* pool = new (mem) BlockPool();
    return *pool;
}

}  // namespace

int acquire_block(size_t bytes, DeviceBlock* b) {
    // whole 2 MB, so that about the same sizes fit
    bytes = (std::max<size_t>(bytes, 1) + (size_t(2) << 20) - 1) >> 21 << 21;
    int dev = 0;
    TDS_HIP(hipGetDevice(&dev));
    BlockPool& P = block_pool();
    {
        // the smallest idle block that holds it, unless most would lie idle
        std::lock_guard<std::mutex> l(P.mu);
        size_t best = P.n;
        for (size_t i = 0; i < P.n; ++i) {
            const DeviceBlock& x = P.idle[i];
            if (x.device == dev && x.bytes >= bytes && x.bytes / 2 <= bytes &&
                (best == P.n || x.bytes < P.idle[best].bytes))
                best = i;
        }
        if (best < P.n) {
            *b = P.take(best);
            return TDS_OK;
        }
    }
    TDS_TRY(dmalloc(&b->p, bytes));
    b->bytes = bytes;
    b->device = dev;
    return TDS_OK;
}

void release_block(DeviceBlock* b) {
    if (!b->p) return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(b->device);
    const bool idle = b->bytes <= kPoolBytes && hipDeviceSynchronize() == hipSuccess;
    (void)hipSetDevice(cur);
    DeviceBlock out;  // to free
    if (!idle) {
        (void)hipGetLastError();
        out = *b;
    } else {
        BlockPool& P = block_pool();
        std::lock_guard<std::mutex> l(P.mu);
        if (P.n == kPoolBlocks) out = P.take(0);
        P.idle[P.n++] = *b;
    }
    dfree(out.p);
    while (idle && block_pool().take_past(b->device, kPoolBytes, &out)) dfree(out.p);
    *b = DeviceBlock();
}

int trim_blocks(size_t* bytes) {
    *bytes = 0;
    int dev = 0;
    TDS_HIP(hipGetDevice(&dev));
    DeviceBlock out;
    while (block_pool().take_past(dev, 0, &out)) {
        dfree(out.p);
        *bytes += out.bytes;
    }
    return TDS_OK;
}

int validate_segments_args(const tds_segments* S) {
    if (!S) return TDS_E_INVALID;
    if (S->n == 0 || S->n >= 0xFFFFFFFFull) return TDS_E_INVALID;
    if (!S->xs || !S->ys || !S->zs || !S->ts || !S->xe || !S->ye || !S->ze || !S->te)
        return TDS_E_INVALID;
    return TDS_OK;
}

void destroy_index(tds_index* idx) {
    if (!idx) return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(idx->device);
    for (Workspace* w : idx->pool) delete w;
    idx->pool.clear();
    release_block(&idx->block);
    (void)hipSetDevice(cur);
    delete idx;
}

int build_impl(const tds_segments* D, const tds_build_params* p, hipStream_t stream,
               tds_index** out) {
    if (!out) return TDS_E_INVALID;
    *out = nullptr;
    TDS_TRY(validate_segments_args(D));
    const uint64_t n = D->n;
    const uint32_t req_bins = p ? p->num_bins : 0u;
    if (req_bins > kMaxBins) return TDS_E_INVALID;
    uint32_t layout = p ? p->layout : (uint32_t)TDS_LAYOUT_DEFAULT;
    if (layout == TDS_LAYOUT_DEFAULT) layout = TDS_LAYOUT_SPATIAL;
    if (layout != TDS_LAYOUT_TEMPORAL && layout != TDS_LAYOUT_SPATIAL) return TDS_E_INVALID;

    int dev = 0;
    TDS_HIP(hipGetDevice(&dev));
    // ---- everything that the build alone needs
    const uint32_t nb = ceil_div(n, kBT);
    double *stage = nullptr, *part = nullptr;
    EntryF64* tmp64 = nullptr;
    EntryF32* tmp32 = nullptr;
    uint64_t *keys = nullptr, *keys2 = nullptr, *status = nullptr;
    uint32_t *tr = nullptr, *vals = nullptr, *vals2 = nullptr, *err = nullptr;
    SortControl* ctl = nullptr;
    Scratch sc;
    {
        DeviceArena a;
        if (!D->on_device) {
            a.add(&stage, 8 * n);
            if (D->traj_id) a.add(&tr, n);
        }
        a.add(&tmp64, n);
        a.add(&tmp32, n);
        a.add(&keys, n);
        a.add(&keys2, n);
        a.add(&vals, n);
        a.add(&vals2, n);
        a.add(&part, kPart * (size_t)nb);
        a.add(&err, 1);
        a.add(&ctl, 1);
        a.add(&status, sort_status_len((uint32_t)n));
        TDS_TRY(a.alloc(&sc.block));
    }
    // ---- stage the input on the device
    SegView S{};
    S.n = n;
    const double* src[8] = {D->xs, D->ys, D->zs, D->ts, D->xe, D->ye, D->ze, D->te};
    if (D->on_device) {
        for (int k = 0; k < 8; ++k) S.a[k] = src[k];
        S.traj = D->traj_id;
    } else {
        for (int k = 0; k < 8; ++k) {
            TDS_HIP(hipMemcpyAsync(stage + k * n, src[k], n * sizeof(double), hipMemcpyHostToDevice,
                                   stream));
            S.a[k] = stage + k * n;
        }
        S.traj = nullptr;
        if (D->traj_id) {
            TDS_HIP(hipMemcpyAsync(tr, D->traj_id, n * sizeof(uint32_t), hipMemcpyHostToDevice,
                                   stream));
            S.traj = tr;
        }
    }
    // ---- per-segment preparation
    TDS_HIP(hipMemsetAsync(err, 0, sizeof(uint32_t), stream));
    hipLaunchKernelGGL(k_seg_prep, dim3(nb), dim3(kBT), 0, stream, S, tmp64, tmp32, keys,
                       part, err);
    TDS_HIP(hipGetLastError());
    std::vector<double> hpart(kPart * (size_t)nb);
    uint32_t herr = 0;
    TDS_HIP(hipMemcpyAsync(hpart.data(), part, hpart.size() * sizeof(double), hipMemcpyDeviceToHost,
                           stream));
    TDS_HIP(hipMemcpyAsync(&herr, err, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    TDS_HIP(hipStreamSynchronize(stream));
    if (herr) return TDS_E_INVALID;
    double tmin = INFINITY, tmax = -INFINITY, dsum = 0.0;
    double clo[3] = {INFINITY, INFINITY, INFINITY}, chi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (uint32_t b = 0; b < nb; ++b) {
        const double* q = &hpart[kPart * (size_t)b];
        tmin = std::fmin(tmin, q[0]);
        tmax = std::fmax(tmax, q[1]);
        dsum += q[2];
        for (int k = 0; k < 3; ++k) {
            clo[k] = std::fmin(clo[k], q[3 + 2 * k]);
            chi[k] = std::fmax(chi[k], q[4 + 2 * k]);
        }
    }
    uint32_t m = req_bins;
    const double mean = dsum / (double)n;
    if (m == 0) {
        double mm = std::nearbyint((tmax - tmin) / mean);
        if (!(mm >= 1.0)) mm = 1.0;
        if (mm > (double)kMaxBins) mm = (double)kMaxBins;
        m = (uint32_t)mm;
    }
    const double bw = (tmax - tmin) / (double)m;

    // ---- sort: by t_start, or by (bin, spatial cell)
    int key_bits = 64;
    if (layout == TDS_LAYOUT_SPATIAL) {
        float lo[3], sc[3];
        for (int k = 0; k < 3; ++k) {
            const double ext = chi[k] - clo[k];
            lo[k] = (float)clo[k];
            sc[k] = (ext > 0.0 && std::isfinite(ext)) ? (float)(1024.0 / ext) : 0.f;
        }
        hipLaunchKernelGGL(k_spatial_key, dim3(nb), dim3(kBT), 0, stream, n, tmp64, tmp32, tmin,
                           bw, m, lo[0], lo[1], lo[2], sc[0], sc[1], sc[2], keys);
        TDS_HIP(hipGetLastError());
        int bin_bits = 0;
        while ((1u << bin_bits) < m) ++bin_bits;
        key_bits = 30 + bin_bits;
    }
    const SortJob sort{(uint32_t)n, keys, nullptr, keys, keys2, vals, vals2, ctl, status};
    TDS_TRY(sort_clear(sort, stream));
    TDS_TRY(sort_plan(sort, key_bits, stream));
    TDS_TRY(sort_passes(sort, sort_npass(key_bits), false, stream));

    // ---- the index object
    tds_index* idx = new (std::nothrow) tds_index();
    if (!idx) return TDS_E_NOMEM;
    idx->device = dev;
    idx->n = n;
    idx->m = m;
    idx->t_min = tmin;
    idx->t_max = tmax;
    idx->bw = bw;
    idx->mean_dt = mean;
    idx->layout = layout;
    const uint32_t nblk = ceil_div(n, 1u << kBoxShift);
    DeviceArena arrays;
    arrays.add(&idx->e64, n);
    arrays.add(&idx->e32, n);
    arrays.add(&idx->ev32, n);
    arrays.add(&idx->seg_id, n);
    arrays.add(&idx->traj, n);
    arrays.add(&idx->bin_first, (size_t)m + 1);
    arrays.add(&idx->min_ts, m);
    arrays.add(&idx->max_te, m);
    arrays.add(&idx->min_te, m);
    arrays.add(&idx->cmax_te, m);
    arrays.add(&idx->lo_ts, m);
    arrays.add(&idx->max_ts, m);
    if (layout == TDS_LAYOUT_SPATIAL) arrays.add(&idx->bbox, nblk);
    const int st = arrays.alloc(&idx->block);
    if (st != TDS_OK) {
        destroy_index(idx);
        return st;
    }
    idx->device_bytes = n * (sizeof(EntryF64) + sizeof(EntryF32) + sizeof(EntryV32) + 8) +
                        (size_t)m * 52 + 4 +
                        (idx->bbox ? (size_t)nblk * sizeof(BlockBox) : 0);
    hipLaunchKernelGGL(k_gather, dim3(nb), dim3(kBT), 0, stream, n, vals, vals2, ctl, tmp64, tmp32, S.traj,
                       idx->e64, idx->e32, idx->ev32, idx->seg_id, idx->traj);
    hipLaunchKernelGGL(k_bin_first, dim3(nb), dim3(kBT), 0, stream, n, idx->e64, tmin, bw, m,
                       idx->bin_first);
    hipLaunchKernelGGL(k_bin_stats, dim3(m), dim3(kBT), 0, stream, idx->e64, idx->bin_first,
                       idx->min_ts, idx->max_ts, idx->min_te, idx->max_te);
    hipLaunchKernelGGL(k_bin_scan<true>, dim3(1), dim3(1024), 0, stream, idx->max_te, idx->cmax_te,
                       m);
    hipLaunchKernelGGL(k_bin_scan<false>, dim3(1), dim3(1024), 0, stream, idx->min_ts, idx->lo_ts,
                       m);
    if (idx->bbox)
        hipLaunchKernelGGL(k_block_box, dim3(ceil_div(nblk, kBT / kWave)), dim3(kBT), 0, stream, n,
                           idx->e64, idx->bbox, nblk);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(stream) != hipSuccess) {
        destroy_index(idx);
        return TDS_E_DEVICE;
    }
    *out = idx;
    return TDS_OK;
}

}  // namespace tds
