// Where the attention kernel's workgroups go: (query group, head) of each
// workgroup of the grid (host and device).
#pragma once

#include <hip/hip_runtime.h>

namespace iefwd {

constexpr int kAttnXcds = 8;

// The grid is n_bh (batch, head) pairs by n_groups query groups, heaviest (last)
// group first; workgroups are dealt round-robin to the 8 XCDs in that order, so
// every XCD has an even share of each group's work.  Where 8 divides the pairs,
// an XCD takes whole heads, whose K and V are fetched into one L2 only;
// otherwise a head's groups move from XCD to XCD.  (Whole heads at any count
// left XCDs idle or a head short: 2 heads x 8192 positions 182 us on two XCDs
// against 137 on eight, 12 heads x 8192 349 on four of two heads and four of one
// against 272.)
//
// A causal group's work grows with its index, and an XCD's workgroups are
// mostly resident at once, one after the other on each of its CUs: they go
// heaviest first in rows of one per CU, every other row reversed, which pairs
// heavy with light ones.  (With the groups of a head next to each other, 4
// groups put every heaviest one on two of the XCDs: 8 x 16 heads x 512 positions
// 19.5 us against 16.0.  Causal 16 heads x 4001 on 64 CUs: 179 us in rows of 32,
// 164 in rows of the 8 that an XCD has there.)
//
// A launch of few chunks waits for this code to arrive: the grid's coordinates
// are the placement, and only reversed rows, which are a CU's second workgroup
// and later ones, divide (a search through a merged order of whole and dealt
// heads cost 4 x 12 heads x 256 positions 0.5 of 10.0 us).
struct AttnPlace {
    int n_bh, n_groups;
    int cus;              // CUs of an XCD
    uint32_t per_row;     // 2^32 / cus rounded up: p / cus = the high half of p * per_row for p * cus < 2^32

    // Workgroup (ix, iy) of the n_bh x n_groups grid -> query group and pair.
    __host__ __device__ void at(int ix, int iy, bool causal, int &group, int &bh) const {
        group = n_groups - 1 - iy;
        bh = ix;
        if (!causal) return;
        const int i = iy * n_bh + ix, x = i % kAttnXcds, p = i / kAttnXcds;
        const int row = (int)(((uint64_t)(uint32_t)p * per_row) >> 32);
        if (!(row & 1)) return;
        const int first = row * cus, n = (n_bh * n_groups - x + kAttnXcds - 1) / kAttnXcds;   // of XCD x
        const int j = kAttnXcds * ((first + cus < n ? first + cus : n) - 1 - (p - first)) + x;
        group = n_groups - 1 - j / n_bh;
        bh = j % n_bh;
    }
};

// The placement of n_groups query groups of each of n_bh pairs on n_cu CUs.
inline AttnPlace attention_place(int n_bh, int n_groups, int n_cu) {
    int cus = n_cu < kAttnXcds ? 1 : n_cu / kAttnXcds;
    const uint64_t most = (uint64_t)n_bh * n_groups / kAttnXcds + 1;
    // a row per CU as long as the row's number is exact; past that, one row, in order
    if (cus == 1 || most * cus >= (1ull << 32)) cus = 1 << 30;
    return AttnPlace{n_bh, n_groups, cus, (uint32_t)(((1ull << 32) + cus - 1) / cus)};
}

}  // namespace iefwd
