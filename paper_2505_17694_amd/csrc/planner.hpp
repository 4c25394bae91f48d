// Host-side workload balancer: forest indexing, cost estimation, KV division and
// slot scheduling (paper Sec. 4.1 indexes, Sec. 5 Eq. 3-7).  Pure C++, no HIP.
#pragma once

#include <cstdint>
#include <vector>

#include "codec.h"

namespace codec {

// Profiled cost table with integer bilinear interpolation (Sec. 5.2, Eq. 6).
struct CostTable {
    std::vector<int32_t> row_grid;
    std::vector<int32_t> len_grid;
    std::vector<int64_t> cost;          // [row][len]

    int validate() const;
    int64_t estimate(int64_t rows, int64_t len) const;
};

// A task of at most kSoloMaxRows rows and kSoloMaxLen tokens may be run by a single wave; the kernels
// take runs of such tasks in a slot's list one wave each (see solo_run below).
constexpr int32_t kSoloMaxRows = 16;
// Most rows of a task with `head_dim` channels: 256 in the dense task shape, which exists for 128 channels;
// otherwise what the stream shape holds, two row tiles of 16 with 64 channels and one with 256.
constexpr int32_t max_task_rows(int32_t head_dim) { return head_dim == 128 ? 256 : head_dim == 64 ? 32 : 16; }
constexpr int32_t kSoloMaxLen = 2048;
// Most short tasks in one entry of the run-time queue (measured on cfg3/cfg4: 2 costs fetches, 8 and
// more make the last entries long).
constexpr int32_t kQueueBundle = 4;
// schedule = 2 takes the run-time queue from this many entries per slot on.
constexpr int32_t kAutoQueueEntriesPerSlot = 6;
// ... of packed row tiles.  Static time over queue time of 150 drawn plans with packs, geometric mean by entries
// per slot: 64 channels 1.05 at 3.5 .. 4.5, 1.15 at 4.5 .. 5.5, 1.08 beyond; 256 channels 1.00, 1.01 and 1.05.
constexpr int32_t kAutoQueueEntriesPerSlotPacked = 5;
// fused = 2 reduces inside the attention launch when the estimated makespan (ns) is below this: where a
// second launch (about 5 us with the gap in front of it) is a large part of the step.
constexpr int64_t kAutoFusedMakespanNs = 40000;
// ... and when the batch has at most this many query rows per KV head (requests x group).
constexpr int64_t kAutoFusedMaxRows = 64;

// Task record as the kernels read it (32 bytes).  The device image holds the records twice: in the
// order of the slots' lists and in the order of the run-time queue, so that a workgroup reads record
// i of its list directly instead of through an index (a task's start is a chain of dependent reads,
// each of which costs microseconds when the memory system is busy).
struct DevTask {
    int32_t page_off;       // index into the device copy of page_ids of the slice's first page
    int32_t kv_len;         // tokens in the slice
    int32_t q_off;          // first request of the task in node_q
    int32_t n_req;          // requests in the task
    int32_t part_row_base;  // first partial row
    int32_t solo_run;       // number of consecutive single-wave tasks in the slot's list from this one on
    int32_t flags;          // kTaskReadOnce: no other task reads this KV slice (its node has a single row
                            // tile); kTaskMasked: some request of the task has a visibility mask over this node;
                            // kTaskTiles: sibling row tiles packed into one task, of (flags >> kTaskTileShift)
                            // & 255 rows each; the last one may have fewer, its partial rows then start
                            // flags >> kTaskLastShift rows before their place by single_req
    int32_t single_req;     // n_req == 1: the request itself (saves the read of node_q); kTaskTiles: ~(distance
                            // of two tiles' first partial rows); else -1
};

enum : int32_t { kTaskReadOnce = 1, kTaskMasked = 2, kTaskTiles = 4, kTaskTileShift = 8, kTaskLastShift = 16 };
constexpr int32_t kTaskLastMax = 32767;
// Most rows of packed row tiles (64 and 256 channels): eight waves of 32 rows, four with 256 channels.
constexpr int32_t pack_max_rows(int32_t head_dim) { return head_dim == 64 ? 256 : 128; }

// Which partial rows of dense and packed tasks are written through to memory at once, instead of staying in L2 until
// the reduction reads them (MB: all partial rows of the plan, fp32; why, and what else was measured: RowStore in
// kernels.hip).  Time written through over plain, geometric mean and worst of drawn plans, both builds
// in turn on one card.
// Rows with tasks to follow in their workgroup, by MB of rows (260 plans, 158 of them with 128 channels):
//   128 channels:  3 .. 6 1.015 (1.049),  6 .. 8 1.002 (1.047),  8 .. 10 0.992 (1.046),  10 .. 14 0.973,  more 0.957
//   256 channels:  3 .. 6 1.002 (1.034),  6 .. 8 0.987,  8 .. 10 0.998 (1.018),  10 .. 14 0.982,  more 0.989
//    64 channels:  3 .. 8 0.996,  8 .. 10 0.989,  10 .. 14 0.986,  more 1.005 (1.019)
// (A constant, not a function as below: with the comparison in a function the compiler allocates the tile path of 256
// channels otherwise, 13 drawn plans 1.006 of the time.)
constexpr int64_t kEarlyThroughBytes = int64_t(8) << 20;
// A workgroup's last rows, with a number of KV heads that eight does not divide.  (Workgroups of KV head h run on XCD
// h % 8 if eight divides it, in the reduction too, which then finds the rows in that XCD's L2: they stay plain.)
//   more than 3 MB, up to seven heads:         128 channels 82 plans 0.991 (1.025), 256: 34 0.992 (1.014), 64: 35 0.993 (1.015)
//   more than 3 MB, from nine heads (9 .. 36): 128 channels 47 plans 0.997 (1.014), 256: 40 0.995 (1.007), 64: 22 1.002 (1.017)
//   up to 3 MB: 119 plans 1.006 (1.049); but groups of more than 16 heads of 128 channels, all of whose tasks are dense,
//   so that all rows are written through: 16 plans 0.979 (1.006)
// The rule knows neither size nor group all the same: with them (several forms, evaluated here or on the host) the small
// plans of smaller groups took 0.995 .. 1.002 of the time, and plans that the rule treats alike, of 128 channels and
// up to 6 MB, 1.003 .. 1.007, by where the kernel's code then lay; two copies of one build differ by 0.0005.
constexpr bool last_rows_through(int32_t kv_heads) { return (kv_heads & 7) != 0; }

// Two-launch plans whose stream tasks go round the KV heads on [token][head] pools (head_of in kernels.hip): plans of
// at least this estimated makespan and so many tasks per CU, in which tasks that go round read at least this much of all
// tokens that tasks read.  Rows of a head then lie in other L2s than the one of the XCD that reduces it, and a workgroup
// with a single task gains nothing: by tasks of all heads per CU, 444 drawn plans of 64 and 128 channels, time against
// fixed heads, one 1.020, 1.4 .. 2.8 0.990 .. 1.011 (up to 1.043), 4 .. 8 0.96 .. 1.00, more 0.81 .. 0.96.  Where nothing goes
// round (plans that read their slices several times) the kernels are only longer: of 717 drawn plans by the first two
// lines, 242 without such tasks 1.007 (up to 1.025), eight up to a tenth of the tokens 0.993 (up to 1.037), eleven up to a
// quarter 0.958, 456 beyond 0.931.  The 467 plans by this rule 0.931 (0.797 .. 1.022).  256 channels gain nothing (1.00).
constexpr int64_t kHeadsInTurnNs = 60000;
constexpr int64_t kHeadsInTurnTasks = 3 * 256;
constexpr int64_t kHeadsInTurnShare = 10;       // a tenth of the tokens
constexpr bool heads_in_turn(int64_t tasks, int32_t kv_heads, int64_t makespan, int64_t turning_tokens, int64_t tokens)
{
    return kv_heads > 1 && makespan >= kHeadsInTurnNs && tasks * kv_heads >= kHeadsInTurnTasks && turning_tokens * kHeadsInTurnShare >= tokens;
}

// Per request, the reduction kernel reads one 64-byte line: the number of partial rows on the request's
// path and, if there are at most kInlineParts of them, the rows themselves; longer lists are read
// from the CSR arrays.  One dependent read less than offset -> list -> partial rows.
constexpr int32_t kInlineParts = 15;

// Waves that share a list in the split form of the reduction (merge_split_kernel), the first fifteen rows and eight each
// round; less than four: one wave folds a list, see LONG of merge_kernel.  By the longest list and by the waves of the launch:
// the chip holds about 4096 of them at once, and a wave whose part of a list is empty still has to start.  Drawn plans, whole
// steps, time with the split form over time with one wave per list: lists of 16 .. 23 rows (two waves) 73 plans 0.997
// (0.915 .. 1.043); 24 .. 39 rows (four), up to 4096 waves 14 plans 0.930 (0.867 .. 0.981), up to 6143 14 plans 0.973 (0.913 ..
// 1.012), 7000 .. 9700 27 plans 1.007 (0.970 .. 1.034); more rows (eight), up to 5000 waves 14 plans 0.828 (0.667 .. 0.934), up to
// 8191 13 plans 0.913 (0.723 .. 0.992).  Beyond, where no plan was drawn, the reduction alone, its rows in L2, 0.02, 0.3 or
// all of the lists long: eight waves, 10600 waves 0.69 .. 1.18 of the time, 13100 waves 0.65 .. 1.27.
constexpr int32_t kSplitMinList = 24;
constexpr int64_t kSplitMaxWavesOfFour = 6143, kSplitMaxWavesOfEight = 8191;
// Most waves of a launch that reads rows sixteen to 23 beside the first fifteen.
constexpr int64_t kReadAheadMaxWaves = 16383;
constexpr int32_t split_rows(int32_t waves) { return kInlineParts + 8 * (waves - 1); }     // of a list, that a round reads
constexpr int32_t split_waves(int32_t longest_list, int32_t num_requests, int32_t h_q, int32_t group, int32_t head_dim)
{
    if (longest_list <= kInlineParts) return 0;
    const int32_t heads = 256 / head_dim > 1 && group % (256 / head_dim) == 0 ? 256 / head_dim : 1;  // rows of a wave
    const int64_t lists = int64_t(num_requests) * (h_q / heads);
    const int32_t waves = longest_list <= split_rows(4) ? 4 : 8;
    if (longest_list >= kSplitMinList && lists * waves <= (waves == 4 ? kSplitMaxWavesOfFour : kSplitMaxWavesOfEight)) return waves;
    return lists <= kReadAheadMaxWaves ? 1 : 2;
}
// Words of a request's line for the split form: its list's length and first rows.
constexpr int32_t split_line_words(int32_t waves) { return (1 + split_rows(waves) + 15) / 16 * 16; }

// Byte offsets of the arrays inside the device metadata blob.
struct DevLayout {
    size_t slot_recs = 0, slot_off = 0, node_q = 0, page_ids = 0,
           req_part_off = 0, req_part = 0, req_inline = 0, req_line = 0, queue_off = 0, queue_recs = 0, counters = 0,
           arrive = 0,      // [h_kv][num_requests] partial results arrived (single-launch mode), zero between launches
           nodeq_mask = 0,  // per entry of node_q: first word of that request's mask if the node ends the request, else -1
           mask_words = 0,
           total = 0;
    int32_t num_entries = 0;    // entries of the run-time queue as the kernels see it
    int32_t num_slots = 0;      // workgroups per KV head
    int32_t split_waves = 0;    // split_waves() of the plan
    int64_t tokens_read = 0;    // by all tasks
    int64_t turning_tokens = 0; // of those, by stream tasks that alone read their slice: they may go round the heads
};

// Lists of task indices with their offsets.
struct TaskLists {
    std::vector<int32_t> off, tasks;
};

// What the kernels run as one task: a task of the plan, or `tiles` sibling row tiles of one KV slice (64 and
// 256 channels, whose tasks hold at most 32 and 16 rows), tile k being the plan's task first + k * step.
struct DeviceTask {
    int32_t first, step, tiles, rows;
    int64_t cost;
};

struct PlanData {
    codec_head_config head{};
    int32_t group = 1;
    int32_t num_slots = 0, split_align = 0, max_rows = 0, share = 1, schedule = 0, fused = 0;
    int32_t num_nodes = 0, num_requests = 0;

    std::vector<int32_t> node_len, node_page_off, page_ids;
    std::vector<int32_t> node_q_off, node_q;
    std::vector<int32_t> req_node;                  // last node of every request
    std::vector<int32_t> req_mask_off;              // empty: no visibility masks
    std::vector<uint32_t> req_mask;
    std::vector<codec_item> items;
    std::vector<codec_task> tasks;
    std::vector<int32_t> slot_off, slot_tasks;
    std::vector<int32_t> queue_off, queue_tasks;    // run-time queue: entries in longest-first order
    std::vector<int32_t> req_part_off, req_part;
    int64_t cost_l = 0, makespan = 0;
    int32_t part_rows = 0;

    // Packed row tiles (empty: the kernels run the plan's tasks, slots and queue as they are)
    std::vector<DeviceTask> packs;
    TaskLists pack_slots;               // indices into packs, per workgroup of a KV head

    CostTable table;                    // the table the plan was estimated with (for refresh_plan)

    DevLayout layout;
    std::vector<unsigned char> blob;    // host image of the device metadata
};

const CostTable &builtin_cost_table(bool wide);

// Fills `plan` from the caller's forest; returns a CODEC_* status.
int build_plan(const codec_tree &tree, const codec_head_config &head,
               const codec_plan_options &opt, PlanData &plan);

// options.share == 2: builds the candidate plans named in codec.h and keeps the one with the lowest
// estimated makespan (ties: the earlier candidate).  Other values: build_plan.
int build_best_plan(const codec_tree &tree, const codec_head_config &head,
                    const codec_plan_options &opt, PlanData &plan);

// Carries `plan` over to new node lengths and page lists without dividing or scheduling again (the
// paper divides tasks only every few decoding steps: Implementation section, task division module):
// slices keep their boundaries, a node's last slice takes up the change in length, costs and the
// makespan are re-estimated, the device image is rebuilt.  On error `plan` is left as it was.
int refresh_plan(PlanData &plan, const int32_t *node_len, const int32_t *node_page_off, const int32_t *page_ids);

// Every request has one partial result and the kernels run nothing but tasks of at most 16 rows: the attention
// launch writes finished rows and there is nothing to reduce.  Packed row tiles hold more rows than that.
bool single_parts(const PlanData &plan);

}  // namespace codec
