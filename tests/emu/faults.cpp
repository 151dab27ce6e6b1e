// The library's host paths on the CPU emulation of its kernels, with allocations
// that fail (see faults.hpp):
//
//   faults waits search|batch|begin   each allocation of a call without a
//       workspace fails in turn: "calls that failed, failures after something was queued,
//       calls that returned with work queued"
//   faults merge   each allocation of a merge of host records fails in turn: the
//       same three numbers, and the failed calls that gave a number of intervals
//   faults pools   device and pinned blocks are given back, and a grid search ends,
//       with no host memory to be had: 0 (an exception ends the program)
//   faults pinned  a search, a batch and a begun search of host arrays where the
//       index has a workspace and there is no more pinned memory: their statuses and
//       whether each found what it finds with it
//   faults trim    device allocations left after an index was closed, bytes given
//       back, allocations left then; the status of a build in a device that is full
//       but for idle blocks
//   faults grid    each copy of a grid search of device arrays fails in turn: the
//       same three numbers
#include <cstdio>
#include <new>
#include <string>
#include <vector>

#include "tds_internal.hpp"

long emu_launches = 0;

// As in the C ABI (capi.hip, not linked here).
extern "C" void tds_search_params_default(tds_search_params* p) {
    std::memset(p, 0, sizeof(*p));
    p->precision = TDS_PREC_FP32_RECHECK;
}

void* operator new(size_t n) {
    void* p = emu_faults.news ? nullptr : malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept {
    return emu_faults.news ? nullptr : malloc(n);
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

namespace {

struct Segs {
    std::vector<double> a[8];
    std::vector<uint32_t> traj;
    tds_segments s{};
    explicit Segs(size_t n, unsigned seed) {
        unsigned x = seed;
        const auto u = [&] { return (x = x * 1664525u + 1013904223u) / 4294967296.0; };
        for (auto& v : a) v.resize(n);
        for (size_t i = 0; i < n; ++i) {
            for (int k = 0; k < 3; ++k) a[k][i] = 10 * u(), a[4 + k][i] = a[k][i] + u();
            a[3][i] = 4 * u();
            a[7][i] = a[3][i] + 1;
            traj.push_back((uint32_t)i);
        }
        s.xs = a[0].data();
        s.ys = a[1].data();
        s.zs = a[2].data();
        s.ts = a[3].data();
        s.xe = a[4].data();
        s.ye = a[5].data();
        s.ze = a[6].data();
        s.te = a[7].data();
        s.traj_id = traj.data();
        s.n = n;
    }
};

tds_index* build(const Segs& D) {
    tds_build_params bp{};
    bp.num_bins = 2;
    tds_index* idx = nullptr;
    if (tds::build_impl(&D.s, &bp, nullptr, &idx) != TDS_OK) exit(3);
    return idx;
}

tds_search_params params() {
    tds_search_params p;
    tds_search_params_default(&p);
    p.grid_waves = 4;
    p.output = TDS_OUTPUT_STAGED;
    return p;
}

// One call of `entry`; what it returned.
int call(const std::string& entry, tds_index* idx, const Segs& Q, std::vector<tds_result>& out,
         uint64_t* n) {
    tds_search_params p = params();
    if (entry == "search")
        return tds::search_impl(idx, &Q.s, 2.0, -1e9, 1e9, out.data(), out.size(), n, &p, nullptr,
                                nullptr);
    if (entry == "batch") {
        const uint64_t h = Q.s.n / 2, room = out.size() / 2;
        const tds_request r[2] = {{0, h, 2.0, -1e9, 1e9, 0, room},
                                  {h, Q.s.n - h, 1.0, -1e9, 1e9, room, room}};
        uint64_t c[2] = {};
        const int st = tds::batch_impl(idx, &Q.s, r, 2, out.data(), out.size(), c, &p, nullptr, nullptr);
        *n = c[0] + c[1];
        return st;
    }
    p.out_on_device = 1;
    void* pending = nullptr;
    const int st = tds::search_begin_impl(idx, &Q.s, 2.0, -1e9, 1e9, out.data(), out.size(), &p,
                                          nullptr, &pending);
    return st == TDS_OK ? tds::search_end_impl(pending, n, nullptr) : st;
}

int run_waits(const std::string& entry) {
    const Segs D(200, 1), Q(70, 2);
    std::vector<tds_result> out(20000);
    int failed = 0, late = 0, unwaited = 0;
    tds_index* idx = build(D);
    for (int pinned = 0; pinned < 2; ++pinned)
        for (long k = 0;; ++k) {
            emu_faults.queued = emu_faults.failed = 0;
            const long launches = emu_launches;
            (pinned ? emu_faults.pinned : emu_faults.mallocs) = k;
            emu_faults.copies = 0;
            uint64_t n = 0;
            const int st = call(entry, idx, Q, out, &n);
            emu_faults.pinned = emu_faults.mallocs = -1;
            if (st != TDS_OK) {
                ++failed;
                late += emu_faults.copies > 0;
                unwaited += emu_faults.queued > 0;
            }
            const bool done = emu_faults.failed == 0;
            if (done && (st != TDS_OK || n == 0 || emu_launches == launches)) return 4;
            for (tds::Workspace* w : idx->pool) delete w;
            idx->pool.clear();
            if (done) break;
        }
    tds::destroy_index(idx);
    printf("%d %d %d\n", failed, late, unwaited);
    return 0;
}

int run_pools() {
    constexpr int kBlocks = 200;
    static tds::DeviceBlock b[kBlocks];
    static tds::PinBlock* pins[40];
    for (int i = 0; i < kBlocks; ++i)
        if (tds::acquire_block((size_t)(1 + i % 7) << 21, &b[i]) != TDS_OK) return 3;
    for (auto& p : pins)
        if (tds::acquire_pin(&p) != TDS_OK) return 3;
    emu_faults.news = true;
    for (auto& x : b) tds::release_block(&x);
    tds::DeviceBlock again;
    if (tds::acquire_block(3 << 20, &again) != TDS_OK) return 4;
    tds::release_block(&again);
    size_t freed = 0;
    if (tds::trim_blocks(&freed) != TDS_OK || freed == 0) return 4;
    for (auto* p : pins) tds::release_pin(p);
    emu_faults.news = false;
    if (emu_faults.live != 0) return 5;  // all blocks were freed
    const Segs D(200, 1), Q(70, 2);
    std::vector<tds_result> out(20000);
    tds_index* idx = build(D);
    tds_fsg* f = nullptr;
    if (tds::fsg_build(idx, 3, 3, 3, nullptr, &f) != TDS_OK) return 3;
    uint64_t n = 0;
    emu_faults.news_after_wait = true;
    const int st = tds::fsg_search(f, &Q.s, 2.0, -1e9, 1e9, out.data(), out.size(), &n, nullptr,
                                   nullptr, nullptr);
    emu_faults.news_after_wait = emu_faults.news = false;
    if (st != TDS_OK || n == 0) return 4;
    tds::fsg_destroy(f);
    tds::destroy_index(idx);
    printf("0\n");
    return 0;
}

int run_pinned() {
    const Segs D(200, 1), Q(70, 2);
    Segs dq(70, 3);
    dq.s.on_device = 1;
    std::vector<tds_result> out(20000);
    tds_index* idx = build(D);
    tds_search_params p = params();
    p.out_on_device = 1;
    const std::string entry[3] = {"search", "batch", "begin"};
    uint64_t want[3] = {}, n = 0;
    for (int i = 0; i < 3; ++i)
        if (call(entry[i], idx, Q, out, &want[i]) != TDS_OK || want[i] == 0) return 3;
    for (int i = 0; i < 3; ++i) {
        // a workspace as a search from and to device memory leaves it
        for (tds::Workspace* w : idx->pool) delete w;
        idx->pool.clear();
        if (tds::search_impl(idx, &dq.s, 2.0, -1e9, 1e9, out.data(), out.size(), &n, &p, nullptr,
                             nullptr) != TDS_OK)
            return 3;
        tds::PinBlock* idle[tds::kPinPool] = {};  // none in the pool either
        for (auto& x : idle) (void)tds::acquire_pin(&x);
        emu_faults.pinned = 0;
        n = 0;
        const int st = call(entry[i], idx, Q, out, &n);
        emu_faults.pinned = -1;
        for (auto* x : idle) tds::release_pin(x);
        printf("%d %d ", st, n == want[i]);
    }
    tds::destroy_index(idx);
    printf("\n");
    return 0;
}

int run_trim() {
    const Segs D(200, 1), Q(70, 2), large(90000, 3);
    std::vector<tds_result> out(20000);
    const auto search_and_close = [&] {
        tds_index* idx = build(D);
        uint64_t n = 0;
        const int st = call("search", idx, Q, out, &n);
        tds::destroy_index(idx);
        return st == TDS_OK && n;
    };
    if (!search_and_close()) return 3;
    const long left = emu_faults.live;
    size_t freed = 0;
    if (tds::trim_blocks(&freed) != TDS_OK) return 3;
    printf("%ld %zu %ld ", left, freed, emu_faults.live);
    if (!search_and_close()) return 3;
    emu_faults.most = emu_faults.live;  // only what the idle blocks make room for
    tds_build_params bp{};
    bp.num_bins = 2;
    tds_index* idx = nullptr;
    printf("%d\n", tds::build_impl(&large.s, &bp, nullptr, &idx));
    return 0;
}

int run_merge() {
    std::vector<tds_result> r(40);
    for (size_t i = 0; i < r.size(); ++i) {
        r[i] = {};
        r[i].q_traj = (uint32_t)i % 3;
        r[i].t_lo = (double)(i % 7);
        r[i].t_hi = r[i].t_lo + (i == 9 ? -1 : 2);  // one is no interval: the general form
    }
    std::vector<tds_traj_interval> out(r.size());
    int failed = 0, late = 0, unwaited = 0, counted = 0;
    for (long k = 0;; ++k) {
        emu_faults.queued = emu_faults.failed = emu_faults.copies = 0;
        emu_faults.mallocs = k;
        const long live = emu_faults.live;
        uint64_t n = 0;
        const int st = tds::merge_impl(r.data(), r.size(), false, out.data(), out.size(), false, &n,
                                       nullptr);
        emu_faults.mallocs = -1;
        if (emu_faults.failed == 0) {
            if (st != TDS_OK || n == 0) return 4;
            break;
        }
        failed += st != TDS_OK;
        late += emu_faults.copies > 0;
        unwaited += emu_faults.queued > 0;
        counted += n != 0;
        if (emu_faults.live > live) k = -1;  // a part of the scratch stays: on from the next
    }
    printf("%d %d %d %d\n", failed, late, unwaited, counted);
    return 0;
}

int run_grid() {
    const Segs D(200, 1);
    Segs Q(70, 2);
    Q.s.on_device = 1;
    std::vector<tds_result> out(20000);
    tds_index* idx = build(D);
    tds_fsg* f = nullptr;
    if (tds::fsg_build(idx, 3, 3, 3, nullptr, &f) != TDS_OK) return 3;
    tds_search_params p = params();
    p.out_on_device = 1;
    int failed = 0, late = 0, unwaited = 0;
    for (long k = 0;; ++k) {
        emu_faults.queued = emu_faults.failed = 0;
        emu_faults.copies_left = k;
        const long launches = emu_launches;
        uint64_t n = 0;
        const int st = tds::fsg_search(f, &Q.s, 2.0, -1e9, 1e9, out.data(), out.size(), &n, &p,
                                       nullptr, nullptr);
        emu_faults.copies_left = -1;
        if (emu_faults.failed == 0) {
            if (st != TDS_OK || n == 0) return 4;
            break;
        }
        failed += st != TDS_OK;
        late += emu_launches > launches;
        unwaited += emu_faults.queued > 0;
    }
    tds::fsg_destroy(f);
    tds::destroy_index(idx);
    printf("%d %d %d\n", failed, late, unwaited);
    return 0;
}

}  // namespace

int main(int argc, char** argv) {
    const std::string mode = argc > 1 ? argv[1] : "";
    if (mode == "waits" && argc > 2) return run_waits(argv[2]);
    if (mode == "pools") return run_pools();
    if (mode == "pinned") return run_pinned();
    if (mode == "trim") return run_trim();
    if (mode == "merge") return run_merge();
    if (mode == "grid") return run_grid();
    return 2;
}
