// The tile tables of the grouped GEMMs, built by one wave from the permutation's offsets and order.
#pragma once
#include "common.h"
#include "ffn_internal.h"

namespace fate {

// tab_up / tab_down [E + n_shared + 1]: first tile, expert, first row and rows of every segment, in the order
// experts by rising number of rows, then the shared experts (the GEMMs read their table from its end).
__device__ __forceinline__ void wave_tile_tables(const int32_t* offsets, const int32_t* order, int E, int n_shared, int N,
                                                 const TileBlocks& nb, const PartSel& sel, int4* tab_up, int4* tab_down) {
    const int lane = threadIdx.x & 63;
    // tile tables: exclusive prefix sums over the segments, 64 segments per step of one wave
    const int nseg = E + n_shared;
    int ru = 0, rd = 0;
    for (int s0 = 0; s0 < nseg; s0 += 64) {
        const int s = s0 + lane;
        int cu = 0, cd = 0, e = 0, T = 0, row = 0;
        if (s < nseg) {
            // a piece holds the routed experts of its mask; the shared experts go with the first piece.
            // The table is read from its end: shared experts, then experts by falling number of rows
            e = s < E ? order[E - 1 - s] : s - E;
            const bool mine = s < E ? ((sel.mask[e >> 6] >> (e & 63)) & 1ull) != 0 : sel.first != 0;
            row = s < E ? offsets[e] : 0;
            T = !mine ? 0 : (s < E ? offsets[e + 1] - row : N);
            const int rl = s < E ? nb.rows_r : nb.rows_s, nt = (T + (1 << rl) - 1) >> rl;
            cu = nt * (s < E ? nb.r_up : nb.s_up);
            cd = nt * (s < E ? nb.r_down : nb.s_down);
        }
        int iu = cu, id = cd;
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) {
            const int pu = __shfl_up(iu, sh, 64), pd = __shfl_up(id, sh, 64);
            if (lane >= sh) { iu += pu; id += pd; }
        }
        if (s < nseg) {
            tab_up[s] = make_int4(ru + iu - cu, e, row, T);
            tab_down[s] = make_int4(rd + id - cd, e, row, T);
        }
        ru += __shfl(iu, 63, 64);
        rd += __shfl(id, 63, 64);
    }
    if (lane == 0) {
        tab_up[nseg] = make_int4(ru, 0, 0, 0);
        tab_down[nseg] = make_int4(rd, 0, 0, 0);
    }
}

}  // namespace fate
