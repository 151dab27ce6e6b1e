// The index as the kernels see it, and the schedule: the candidate range of a
// query segment by bisection of the bin tables.
#pragma once

#include "canon.hpp"
#include "tds_internal.hpp"

namespace tds {

namespace {

struct IndexView {
    const EntryF64* e64;
    const EntryF32* e32;
    const uint32_t* seg_id;
    const uint32_t* traj;
    const uint32_t* bin_first;
    const double* cmax_te;
    const double* lo_ts;
    const EntryV32* ev32;  // FP32 motion of the entries (filter refinement)
    const BlockBox* bbox;  // block boxes (spatial layout) or nullptr
    double t_min, bw;      // bin origin and width (search starting points)
    uint32_t n, m;
};

inline IndexView view_of(const tds_index* idx) {
    IndexView v;
    v.e64 = idx->e64;
    v.e32 = idx->e32;
    v.seg_id = idx->seg_id;
    v.traj = idx->traj;
    v.bin_first = idx->bin_first;
    v.cmax_te = idx->cmax_te;
    v.lo_ts = idx->lo_ts;
    v.ev32 = idx->ev32;
    v.bbox = idx->bbox;
    v.t_min = idx->t_min;
    v.bw = idx->bw;
    v.n = (uint32_t)idx->n;
    v.m = idx->m;
    return v;
}

// Smallest j in [0, m] with pred(j), for a predicate that is monotone
// (false ... false true ... true) with pred(m) true.  The bins have equal
// widths, so the caller's guess g (the bin of the time searched for) is
// usually within one of the answer: four neighbouring values are loaded at
// once, and only if the answer lies outside them does the search gallop
// away from g and bisect the bracket found.
template <class Pred>
__device__ inline uint32_t first_true(Pred pred, uint32_t m, uint32_t g) {
    g = min(g, m);
    const uint32_t a = (g > 0) ? g - 1 : 0;
    bool w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = (a + k >= m) ? true : pred(a + k);
    uint32_t l, h;  // the answer lies in [l, h] and pred(h) holds
    if (w[0]) {
        if (a == 0) return 0;
        // answer <= a: gallop down from a
        h = a;
        uint32_t step = 1;
        for (;;) {
            if (h < step) {
                l = 0;
                break;
            }
            const uint32_t c = h - step;
            if (!pred(c)) {
                l = c + 1;
                break;
            }
            h = c;
            step *= 2;
        }
    } else {
#pragma unroll
        for (int k = 1; k < 4; ++k)
            if (w[k] && !w[k - 1]) return a + k;
        // answer > a + 3: gallop up
        l = a + 4;
        uint32_t step = 1;
        for (;;) {
            const uint32_t c = l - 1 + step;
            if (c >= m) {
                h = m;
                break;
            }
            if (pred(c)) {
                h = c;
                break;
            }
            l = c + 1;
            step *= 2;
        }
    }
    while (l < h) {
        const uint32_t mid = l + (h - l) / 2;
        if (pred(mid)) h = mid;
        else l = mid + 1;
    }
    return l;
}

// Two independent first_true searches whose first windows are loaded together.
template <class P1, class P2>
__device__ inline void first_true2(P1 p1, uint32_t g1, P2 p2, uint32_t g2, uint32_t m,
                                   uint32_t* r1, uint32_t* r2) {
    g1 = min(g1, m);
    g2 = min(g2, m);
    const uint32_t a1 = (g1 > 0) ? g1 - 1 : 0, a2 = (g2 > 0) ? g2 - 1 : 0;
    bool w1[4], w2[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        w1[k] = (a1 + k >= m) ? true : p1(a1 + k);
        w2[k] = (a2 + k >= m) ? true : p2(a2 + k);
    }
    // answer inside a window: the first true after a false (or a true at 0)
    auto inside = [](const bool (&w)[4], uint32_t a, uint32_t* r) {
        if (w[0]) {
            if (a == 0) {
                *r = 0;
                return true;
            }
            return false;
        }
#pragma unroll
        for (int k = 1; k < 4; ++k)
            if (w[k] && !w[k - 1]) {
                *r = a + k;
                return true;
            }
        return false;
    };
    if (!inside(w1, a1, r1)) *r1 = first_true(p1, m, g1);
    if (!inside(w2, a2, r2)) *r2 = first_true(p2, m, g2);
}

// Bin of time t for a search starting point (any value is correct).
__device__ inline uint32_t guess_bin(const IndexView& I, double t) {
    const double u = floor((t - I.t_min) / I.bw);
    if (!(u > 0.0)) return 0u;
    if (u >= (double)I.m) return I.m;
    return (uint32_t)u;
}

// Candidate range E_k of a clipped query [aq, bq] (Sec. 4.2.2): from the
// first entry of the first bin whose running max t_end exceeds aq (bin j0)
// to the last entry of the last non-empty bin whose smallest t_start is below
// bq (bin j1), as one contiguous span [lo, hi) of index positions.
__device__ inline void cand_range(const IndexView& I, double aq, double bq, uint32_t* lo,
                                  uint32_t* hi, uint32_t* j0o, uint32_t* j1o) {
    // j0 = first j with cmax_te[j] > aq (m if none); L = number of bins j for
    // which some entry of a bin >= j has t_start < bq (lo_ts, the minimum
    // t_start over bins >= j, is non-decreasing), i.e. the first j with
    // lo_ts[j] >= bq; entries before bin_first[L] are those of bins < L.
    // Both searches read their first windows before either decides.
    uint32_t j0, L;
    first_true2([&](uint32_t j) { return I.cmax_te[j] > aq; }, guess_bin(I, aq),
                [&](uint32_t j) { return I.lo_ts[j] >= bq; }, guess_bin(I, bq) + 1u, I.m, &j0, &L);
    *lo = (j0 < I.m) ? I.bin_first[j0] : I.n;
    *hi = I.bin_first[L];
    *j0o = j0;
    *j1o = (L > 0) ? L - 1 : 0;
}

}  // namespace

}  // namespace tds
