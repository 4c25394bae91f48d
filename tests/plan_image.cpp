// Host view of what a plan uploads, for tests: the planner's sources compiled once more, with access to the
// device image that the library only ever copies to a GPU.
#include <cstring>

#include "planner.hpp"

namespace {
codec::PlanData plan;
}

extern "C" {

// Plans, then carries the plan over to `refreshed_len` if given (page lists as they are).  Returns a CODEC_* status.
int image_plan(const codec_tree *tree, const codec_head_config *head, const codec_plan_options *opt,
               const int32_t *refreshed_len)
{
    plan = codec::PlanData();
    if (int st = codec::build_best_plan(*tree, *head, *opt, plan)) return st;
    return refreshed_len ? codec::refresh_plan(plan, refreshed_len, tree->node_page_off, tree->page_ids) : 0;
}

// slot_recs, slot_off, num_slots, queue_off, queue_recs, num_entries, packs, single_parts, schedule, fused, makespan, part_rows
void image_layout(int64_t *v)
{
    const codec::DevLayout &L = plan.layout;
    const int64_t x[] = {int64_t(L.slot_recs), int64_t(L.slot_off), L.num_slots, int64_t(L.queue_off), int64_t(L.queue_recs),
                         L.num_entries, int64_t(plan.packs.size()), codec::single_parts(plan), plan.schedule, plan.fused,
                         plan.makespan, plan.part_rows};
    std::memcpy(v, x, sizeof x);
}

// per pack: first, step, tiles, rows, cost; then, per slot of the packs, its end in the list of pack indices
void image_packs(int64_t *packs, int32_t *slot_off, int32_t *slot_packs)
{
    for (const codec::DeviceTask &d : plan.packs) {
        const int64_t x[] = {d.first, d.step, d.tiles, d.rows, d.cost};
        std::memcpy(packs, x, sizeof x);
        packs += 5;
    }
    if (plan.packs.empty()) return;
    std::memcpy(slot_off, plan.pack_slots.off.data(), plan.pack_slots.off.size() * 4);
    std::memcpy(slot_packs, plan.pack_slots.tasks.data(), plan.pack_slots.tasks.size() * 4);
}

// which rows the kernels write through: bit 0 those with tasks to follow, bit 1 a workgroup's last ones
int image_rows_through(int32_t part_rows, int32_t kv_heads, int32_t head_dim)
{
    const bool early = int64_t(part_rows) * kv_heads * (head_dim * 4) > codec::kEarlyThroughBytes;
    return (early ? 1 : 0) | (codec::last_rows_through(kv_heads) ? 2 : 0);
}

const unsigned char *image_blob() { return plan.blob.data(); }
int64_t image_bytes() { return int64_t(plan.blob.size()); }

}
