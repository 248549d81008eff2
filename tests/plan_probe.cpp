// The arithmetic of csrc/gt_plan.hpp on the CPU (tests/test_plan.py): the row
// kernels' plan of the classes and the host's choices, with the library's own
// functions.
#include <cstddef>
#include <cstdint>

#include "gt_attn.h"

namespace {
#include "gt_plan.hpp"
}

extern "C" {

// Batches of each XCD for rows[c] rows of each class c, P lane groups per
// wavefront, and the pieces of each class, as class_plan and row_loop have them;
// returns batch_bound of what the partition counts.
int64_t probe_batches(const RowCut* w, const uint32_t* rows, uint32_t P, uint32_t* nq, uint64_t* total,
                      uint64_t* asked) {
    uint64_t slots = 0;
    for (int c = 0; c < kClasses; ++c) {
        const uint32_t cap = class_capacity(*w, c);
        if (rows[c] > cap) return -1;
        nq[c] = cap ? class_pieces(*w, c) : 1;
        slots += nq[c] > 1 ? (uint64_t)rows[c] * nq[c] : 0;
    }
    if (slots > w->cap_slots) {
        uint32_t left = w->cap_slots;
        for (int c = kClasses - 1; c >= 0; --c) {
            nq[c] = fit_pieces(rows[c], nq[c], left);
            if (nq[c] > 1) left -= rows[c] * nq[c];
        }
    }
    uint64_t groups = 0;
    for (uint32_t x = 0; x < (uint32_t)kXcds; ++x) total[x] = 0;
    for (int c = 0; c < kClasses; ++c) {
        const uint64_t flat = (uint64_t)rows[c] * nq[c];
        for (uint32_t x = 0; x < (uint32_t)kXcds; ++x)
            total[x] += piece_batches(piece_share(flat, x + 1) - piece_share(flat, x), class_spread(*w, c, nq[c]), P);
        groups += rows[c] ? class_groups(*w, c, rows[c], P) : 0;
    }
    *asked = groups;  // (a 32-bit counter on the device)
    return batch_bound((uint32_t)groups, P);
}

void probe_rule(int64_t N, int64_t E, int slices, int gather_bytes, int piece_bytes, int P, const gt_tuning* tu,
                RowCut* w, RowRule* r) {
    *r = row_rule(N, E, slices, gather_bytes, piece_bytes, P, tu);
    w->N = N;
    w->E = (uint32_t)E;
    set_rule(*w, *r);
}

void probe_attn(const AttnShape* a, const gt_tuning* tu, int noalloc, AttnPlan* p) { *p = plan_attn(*a, tu, noalloc != 0); }

void probe_slots(const RowRule* r, int slices, int64_t slot_bytes, int64_t other_bytes, int bounded, SlotPlan* s) {
    *s = slot_plan(*r, slices, (size_t)slot_bytes, (size_t)other_bytes, bounded != 0);
}

void probe_grid(int64_t N, int64_t E, int groups, int slices, int tiles, int resident, const gt_tuning* tu, RowGrid* g) {
    *g = row_grid(N, E, groups, slices, tiles != 0, resident, tu);
}

int probe_wide(int64_t N, int64_t E, int64_t row_bytes) { return wide_slices(N, E, row_bytes); }

}  // extern "C"
