// Bookkeeping of the members of a distillation team that another member does not wait for.  (No device code: what a
// member decides is the same function on the host, where it is tested.)
#pragma once

#include <cstdint>

namespace respec {

// A member whose words for a row have not come within the wait is given up for that row: its part is computed from
// the rows.  One that was given up on the row before is waited for a sixteenth as long, so that a work-group that is not
// running costs a team one wait and not one per row.  (Not at once: two members that were given up by one another would then
// go on in step, each computing a part that the other is just about to publish.)
struct KdAbsent {
    uint32_t known = 0;  // given up on the row before, a bit each
    uint32_t row = 0;    // given up on this row

    // Members given up now, of those whose words are missing (`late`) after `waited` of `spin` ticks.
    constexpr uint32_t give_up(uint32_t late, uint64_t waited, uint64_t spin) {
        const uint32_t now = waited >= spin ? late : waited >= spin / 16 ? late & known : 0u;
        row |= now;
        return now;
    }
    // Every word of the row is there or computed.
    constexpr void row_done() {
        known = row;
        row = 0;
    }
};

}  // namespace respec
