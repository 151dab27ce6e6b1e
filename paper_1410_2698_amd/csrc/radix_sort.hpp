// Device control block and host entry points of the radix sort
// (radix_sort.hip), shared with the kernels that feed it and read its result.
#pragma once

#include "tds_internal.hpp"

namespace tds {

constexpr int kSortRadix = 256;

// Keys as the sort sees them: the 64-bit key itself, or, for pair keys
// (first id << 32 | second id), the two ids next to each other with only as
// many bits for the second as its largest value needs.
struct PairPack {
    uint32_t pairs, low_bits;
    __host__ __device__ uint64_t apply(uint64_t k) const {
        return pairs ? pack(k) : k;
    }
    __host__ __device__ uint64_t pack(uint64_t k) const {
        return ((k >> 32) << low_bits) | (uint32_t)k;
    }
    __host__ __device__ uint32_t high(uint64_t packed) const {
        return (uint32_t)(packed >> low_bits);
    }
    __host__ __device__ uint32_t low(uint64_t packed) const {
        return (uint32_t)(packed & ((1ull << low_bits) - 1));
    }
};

__host__ __device__ inline uint32_t bits_of(uint32_t v) {
    uint32_t b = 0;
    for (; v; v >>= 1) ++b;
    return b;
}

// One sort's state in device memory, cleared before it starts.
struct SortControl {
    uint32_t npass;            // digits in use
    uint32_t digit[8];         // their positions, in sorting order
    uint32_t ticket[8];        // next tile of each pass
    // pair keys: set by the kernel that makes them
    uint32_t pairs;            // 1: pack (first, second) ids
    uint32_t max_high, max_low;
    // the trajectory merge
    uint32_t odd;              // why its one-pass form does not apply (kOdd*), 0: it does
    uint32_t total;            // intervals found
    uint32_t pad[5];
    uint32_t hist[8][kSortRadix];
    __host__ __device__ PairPack pack() const { return {pairs, bits_of(max_low)}; }
    // buffer (0 or 1) that holds the sorted data
    __host__ __device__ uint32_t side() const { return npass & 1u; }
};

// A sort of n (key, value) pairs: keys from `raw` (which may be k0), sorted
// keys and values in (k0, v0) or (k1, v1) by the control block's side(). With
// 32-bit keys (sort_passes, narrow) the sorted keys are u32 arrays in k1's
// space, side 1 at its start and side 0 n entries further.
struct SortJob {
    uint32_t n;
    const uint64_t* raw;
    const uint32_t* vinit;  // values of the pairs, or nullptr: their positions
    uint64_t *k0, *k1;
    uint32_t *v0, *v1;
    SortControl* ctl;
    uint64_t* status;  // sort_status_len(n) words
};

// Status words to allocate for sorts of up to n pairs.
size_t sort_status_len(uint32_t n);
// In this order, on one stream, nothing waiting: clear the control block and
// the status words; (make the keys); count digits over key_bits low bits and
// plan; up to npass passes (those past the plan's end do nothing).
int sort_clear(const SortJob& J, hipStream_t s);
int sort_plan(const SortJob& J, int key_bits, hipStream_t s);
int sort_passes(const SortJob& J, uint32_t npass, bool narrow, hipStream_t s);

// Exclusive scan of v in place, its sum to part[ceil(len / tile)] (part:
// scan_part_len(len) entries); waits for nothing.
int scan_u32(uint32_t* v, uint32_t len, uint32_t* part, hipStream_t s);

inline uint32_t sort_npass(int key_bits) {
    return (uint32_t)(key_bits < 1 ? 1 : key_bits > 64 ? 8 : (key_bits + 7) / 8);
}

}  // namespace tds
