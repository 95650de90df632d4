// Where the attention kernel's workgroups go: (query group, head) of each
// workgroup of the grid (host and device).
#pragma once

#include <hip/hip_runtime.h>

namespace iefwd {

constexpr int kAttnXcds = 8;

// Workgroups are dealt round-robin to the 8 XCDs: workgroup i is the (i / 8)th
// of XCD i % 8.  Of n_bh (batch, head) pairs, 8 F + r, XCD x takes the pairs
// 8 k + x (k < F) with all their query groups, so that their K and V are fetched
// into one L2 only; the last r pairs' groups, heaviest first, are dealt to the
// XCDs in turn, so that no XCD has more than one group more than another.  (As
// whole heads the last ones left XCDs idle or a head short: 2 heads x 8192
// positions 194 us on two XCDs against 146 on eight, 12 heads x 8192 373 on four
// of two heads and four of one against 285; causal 12 heads x 4000 72 against 71.)
//
// A causal group's work grows with its index, and an XCD's workgroups are
// mostly resident at once, one after the other on each of its CUs: they go
// heaviest first in rows of one per CU, every other row reversed, which pairs
// heavy with light ones.  (With the groups of a head next to each other, 4
// groups put every heaviest one on two of the XCDs: 8 x 16 heads x 512 positions
// 19.5 us against 16.0.  Causal 16 heads x 4001 on 64 CUs: 179 us in rows of 32,
// 164 in rows of the 8 that an XCD has there.)
struct AttnPlace {
    int n_bh, n_groups, cus;   // cus: CUs of an XCD

    __host__ __device__ int full() const { return n_bh / kAttnXcds; }
    __host__ __device__ int rest() const { return n_bh % kAttnXcds; }
    // groups of the last r pairs that XCD x takes of the `level` heaviest ones of each
    __host__ __device__ int dealt(int level, int x) const {
        return (level * rest() + kAttnXcds - 1 - x) / kAttnXcds;
    }
    // workgroups of XCD x before level `level` (level 0: the heaviest group of every pair)
    __host__ __device__ int before(int level, int x) const { return level * full() + dealt(level, x); }
    // workgroups of the grid; XCDs with fewer groups than XCD 0 leave their last one idle
    __host__ __device__ int grid() const { return kAttnXcds * before(n_groups, 0); }

    // Workgroup i -> query group and (batch, head) pair; false if it is idle.
    __host__ __device__ bool at(int i, bool causal, int &group, int &bh) const {
        const int x = i % kAttnXcds, p = i / kAttnXcds, n = before(n_groups, x);
        if (p >= n) return false;
        int s = p;   // position in the order of falling work
        if (causal) {
            const int row = p / cus, first = row * cus, last = (first + cus < n ? first + cus : n) - 1;
            if (row & 1) s = last - (p - first);
        }
        int level = kAttnXcds * s / n_bh;   // within a few levels: before(level) is level * n_bh / 8 within 1
        while (before(level, x) > s) --level;
        while (before(level + 1, x) <= s) ++level;
        const int in = s - before(level, x);
        group = n_groups - 1 - level;
        bh = in < full() ? in * kAttnXcds + x
                         : kAttnXcds * full() + kAttnXcds * (dealt(level, x) + in - full()) + x - level * rest();
        return true;
    }
};

// The placement of n_groups query groups of each of n_bh pairs on n_cu CUs.
inline AttnPlace attention_place(int n_bh, int n_groups, int n_cu) {
    return AttnPlace{n_bh, n_groups, n_cu < kAttnXcds ? 1 : n_cu / kAttnXcds};
}

}  // namespace iefwd
