// CPU build of the shares of workgroups that clear memory (pcr_common.h: fill_turn).  Test-only.
#include "../../paper_1911_00472_amd/csrc/pcr_common.h"

// The launch of `others` workgroups and about `groups` that fill: its size; out[b]: -1 - index for one that fills, else index.
extern "C" int fill_turns(unsigned others, unsigned groups, int* out) {
    const uint32_t rows = pcr::fill_rows(groups), period = pcr::fill_period(others, rows), total = others + pcr::kDies * rows;
    for (uint32_t b = 0; b < total; b++) {
        const pcr::FillTurn t = pcr::fill_turn(b, rows, period);
        out[b] = t.fills ? -1 - (int)t.index : (int)t.index;
    }
    return (int)total;
}
