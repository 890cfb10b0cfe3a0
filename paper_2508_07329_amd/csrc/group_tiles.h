// Tiles of expert groups of a row tile or so each, dealt to work-groups.
#pragma once
#include "haq_common.h"

namespace haq {

struct GroupTile {
    int i;       // selected group
    int mi, mt;  // row tile of the group, its row tiles
    int u;       // channel tile
};

// Work-group ids go round the 8 XCDs (one L2 each): so do the channel tiles, all row tiles of one on the same XCD; a
// contiguous range would give each XCD an expert of its own.  The count goes on from group to group: begun anew for each,
// it left the last XCDs short whenever the `ntn` channel tiles are no multiple of 8 (17 row tiles x 12 channel tiles:
// 34 work-groups on four XCDs of 32 CUs and 17 on the others).
// A grid of round_up(ntn, 8) * (upper bound of the row tiles) reaches every XCD's last tile.  False past that.
// rows_of(i): rows of the i-th selected group.
template <int BM, class ROWS>
__host__ __device__ inline bool deal_group_tile(ROWS&& rows_of, int n_sel, int ntn, int block, GroupTile& t) {
    int slot = block >> 3, first = block & 7;  // first: this XCD's first channel tile of the group
    for (t.i = 0; t.i < n_sel; ++t.i) {
        t.mt = (rows_of(t.i) + BM - 1) / BM;
        if (t.mt == 0) continue;
        const int mine = (ntn - first + 7) >> 3;  // this XCD's channel tiles of the group
        if (slot < mine * t.mt) {
            t.u = first + 8 * (slot / t.mt);
            t.mi = slot % t.mt;
            return true;
        }
        slot -= mine * t.mt;
        first = (first - ntn) & 7;
    }
    return false;
}

#ifdef __HIPCC__
// The selected groups' experts and first and last rows, a group per lane: two loads one after the other for all of them
// (group by group it would be two for each).
struct GroupLanes {
    int e, lo, hi;
    __device__ __forceinline__ explicit GroupLanes(const GemmArgs& a) {
        const int i = threadIdx.x & 63;
        e = i < a.n_sel ? a.sel[i] : 0;
        lo = a.offsets[e];
        hi = a.offsets[e + 1];
    }
    static __device__ __forceinline__ int of(int v, int i) { return __builtin_amdgcn_readlane(v, i); }
    template <int BM>
    __device__ __forceinline__ bool deal(const GemmArgs& a, int ntn, GroupTile& t) const {
        const int rows = hi - lo;
        return deal_group_tile<BM>([&](int i) { return of(rows, i); }, a.n_sel, ntn, (int)blockIdx.x, t);
    }
};
#endif

}  // namespace haq
