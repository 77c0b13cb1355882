// The host library (planner, host interpreter) without the HIP part, as a
// shared object for tests that build the planner with smaller limits or look
// into a plan.  The entry points that need a GPU answer EUNSUPPORTED.
#include <cstdint>

#include "reshard.h"

#include "../../paper_2211_05322_amd/csrc/planner.hpp"

namespace rs {
void release_device_table(const Plan &) {}
}  // namespace rs

extern "C" {
reshard_status_t reshard_plan_upload(const reshard_plan_t *) { return RESHARD_EUNSUPPORTED; }
reshard_status_t reshard_execute(const reshard_plan_t *, void *const *, void *const *, void *) {
    return RESHARD_EUNSUPPORTED;
}
reshard_status_t reshard_execute_noalloc(const reshard_plan_t *, void *const *, void *const *, void *) {
    return RESHARD_EUNSUPPORTED;
}

int64_t test_blocked_chunks(const reshard_plan_t *plan) {
    return int64_t(reinterpret_cast<const rs::Plan *>(plan)->n_blocked);
}
uint32_t test_transpose_launch_lds(const reshard_plan_t *plan, uint32_t user_lds) {
    return rs::transpose_launch_lds(*reinterpret_cast<const rs::Plan *>(plan), user_lds);
}
int test_transpose_plain(const reshard_plan_t *plan) {
    return reinterpret_cast<const rs::Plan *>(plan)->transpose_plain;
}
int64_t test_cached_limit(int64_t fanout, int64_t senders, int parts) {  // no senders: direct chunks
    return senders > 0 ? rs::cached_slots_limit(fanout, senders, parts != 0) : rs::cached_direct_limit(fanout);
}
int test_slots_of_parts(const reshard_plan_t *plan) {
    return reinterpret_cast<const rs::Plan *>(plan)->gather_u_parts;
}
int test_sets_in_turn(const reshard_plan_t *plan) { return reinterpret_cast<const rs::Plan *>(plan)->sets_in_turn; }
}
