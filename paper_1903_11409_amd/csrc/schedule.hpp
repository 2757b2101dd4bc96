// Host-side batch scheduler of libbspmm: bins operations by size, tiles the feature
// dimension, orders the work largest-first and maps it onto workgroups XCD-aware.
#pragma once

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <memory>
#include <utility>
#include <vector>

#include "../../include/bspmm.h"
#include "plan.hpp"

namespace bspmm {

// The operations of one direction (forward, or transposed with the roles swapped).
struct DirOps {
    std::vector<int32_t> m, k, nnz;
    std::vector<int64_t> rpt_off, nz_off, in_off, out_off;
    std::vector<int32_t> chan;   // empty, or per operation: channels of the fused front it carries
                                 // (an operation standing in for a set of summed channels)
    int channels(int i) const { return chan.empty() ? 1 : chan[i]; }
    int size() const { return (int)m.size(); }
};

// Scheduler knobs with defaults filled in.
struct Knobs {
    int force_bin = -1;       // -1 automatic, else BSPMM_BIN_*
    int lds_words = 6144;     // 24 KiB: six workgroups per CU
    int min_tile = 32;
    int min_odd_tile = 8;     // the same for widths that are no multiple of four
    int max_tile = 256;
    int target_wgs = 1024;
    bool target_given = false;   // the caller fixed target_wgs
    int compute_units = 256;
    int pad = 0;
    int max_passes = 1;
    int generic_rows = 8;
    bool generic_given = false;
    int wg_passes = 0;        // 0 automatic, >0 cap on passes of a workgroup item, <0 never cut
    int capacity_wgs = 1536;  // workgroups the chip holds at once (lean kernel variant)
    int capacity_wgs_slices = 1024;   // same for the kernel variant with 32/16-lane slots
    bool accumulate = false;  // operations naming one output block are summed (else an error)
    bool hubs = false;        // split hub rows across the workgroup (reserves LDS for it)
    int front = 0;            // > 0: columns of the layer input of bspmm_run_gcn (whole workgroups,
                              // tiles in multiples of 16 columns)
    bool symmetric = false;   // A_i == A_i^T promised: the transposed product reads the same CSR
    bool coo_direct = false;  // COO plans: run the direct kernel instead of converting to CSR
    int persistent_wgs = 0;   // > 0: launch only this many workgroups and let them stride
    bool wide_offsets = false;       // the transposed arrays outgrow the compact table's 32-bit offsets
    bool one_front_launch = false;   // layers: never the gather-first launch
    bool lds_given = false;   // the caller fixed lds_words
    bool whole_sets = false;  // a set of summed operations over the budget is an error (not a fused task)
    bool device_ok = false;   // planning may ask the current device (occupancy); false: dry runs
    bool need_both = false;   // planning: a transposed product that does not fit is an error too
};

// An item table whose memory is not cleared before it is written.
class ItemTable {
public:
    ItemTable() = default;
    ItemTable(ItemTable&& o) noexcept : p_(std::move(o.p_)), n_(o.n_), room_(o.room_) { o.n_ = o.room_ = 0; }
    ItemTable(const ItemTable& o) { *this = o; }
    ItemTable& operator=(ItemTable&& o) noexcept
    {
        p_ = std::move(o.p_);
        n_ = o.n_, room_ = o.room_;
        o.n_ = o.room_ = 0;
        return *this;
    }
    ItemTable& operator=(const ItemTable& o)
    {
        if (this == &o) return *this;
        n_ = 0;
        resize(o.n_);
        if (n_) std::memcpy(p_.get(), o.p_.get(), n_ * sizeof(LeanItem));
        return *this;
    }
    void resize(size_t n)      // keeps what is there, clears nothing
    {
        if (n > room_) {
            std::unique_ptr<LeanItem[]> q(new LeanItem[n]);
            if (n_) std::memcpy(q.get(), p_.get(), n_ * sizeof(LeanItem));
            p_ = std::move(q);
            room_ = n;
        }
        n_ = n;
    }
    void push_back(const LeanItem& t)
    {
        if (n_ == room_) {
            const size_t n = n_;
            resize(2 * n + 64);
            n_ = n;
        }
        p_[n_++] = t;
    }
    void clear() { n_ = 0; }
    bool empty() const { return n_ == 0; }
    size_t size() const { return n_; }
    LeanItem* data() const { return p_.get(); }
    LeanItem& operator[](size_t i) const { return p_[i]; }
    LeanItem* begin() const { return p_.get(); }
    LeanItem* end() const { return p_.get() + n_; }

private:
    std::unique_ptr<LeanItem[]> p_;
    size_t n_ = 0, room_ = 0;
};

struct Schedule {
    std::vector<WorkItem> items;     // device table, launch order, padded with empty items
    ItemTable compact;               // plain batches: the compact table instead of `items` and `view`
    std::vector<int32_t> item_op;    // operation of every entry of `items` or `compact` (-1: empty item)
    std::vector<bspmm_item> view;    // the non-empty items, for inspection (see items_of)
    int count = 0;                   // non-empty items
    int uncut_wgs = 0;               // workgroups without row cuts, at the first LDS budget
    bool row_blocks = false;         // `compact` has row blocks of the generic bin
    int32_t wg_end[kRanges] = {0, 0, 0, 0, 0};
    int32_t item_base[kRanges] = {0, 0, 0, 0, 0};
    int fused_stride = 1;            // item slots per fused task
    int fused_tasks = 0;
    std::vector<std::vector<int>> fused_sets;   // the sets of summed operations (members in order)
    std::vector<int> task_set;       // set of every fused task, in task order
    std::vector<std::vector<int>> merged_sets;  // sets that one operation with the summed matrix
                                     // stands in for; its index is first_stand_in + position
    int first_stand_in = 0;          // == number of operations of the batch
    int error = 0;                   // BSPMM_E* when the batch cannot be scheduled
    int grid = 0;                    // number of tasks
    int launch_grid = 0;             // workgroups of the persistent launch
    bool whole = false;              // every task is one whole-workgroup item: the launch runs from
                                     // the compact item table (lean kernel, bspmm_any_kernel)
    bool pow2 = false;               // ... on the float4 path with power-of-two tiles: it may take the
                                     // lean kernel
    bool has_slices = false;         // any 32- or 16-lane item: needs the larger kernel variant
    int tile = 0;
    int lds_words = 0;               // `whole` launches: LDS the launch asks for (its largest item)
    int budget_words = 0;            // LDS per workgroup the items were planned for
    int front_lds_words = 0;         // LDS the fused-front launch asks for (its largest item)
    int items_in_bin[BSPMM_NUM_BINS] = {0, 0, 0, 0, 0};
};

// Schedule of the direct COO kernel: one workgroup per item, largest first.
struct CooSchedule {
    std::vector<CooItem> items;
    std::vector<bspmm_item> view;
    int tile = 0;
    int error = 0;
    int lds_words = 0;     // what the launch asks for: the largest item's
};

// Positions 0 .. n-1, largest value first, equal ones in order.  Compared in 1024 steps of the
// largest value: the order only steers greedy placement, and one counting pass is a tenth of a
// comparison sort.
template <typename T>
void largest_first(const T* value, int n, std::vector<int32_t>& order)
{
    T top = 1;
    for (int i = 0; i < n; ++i) top = std::max(top, value[i]);
    int shift = 0;
    while ((top >> shift) > 1023) ++shift;
    uint32_t at[1025] = {0};
    for (int i = 0; i < n; ++i) ++at[1024 - (value[i] >> shift)];
    for (int v = 1; v <= 1024; ++v) at[v] += at[v - 1];
    order.resize(n);
    for (int i = 0; i < n; ++i) order[at[1023 - (value[i] >> shift)]++] = i;
}

int workgroups_per_cu(int front_features);
Knobs resolve_knobs(const bspmm_options* o);

// Items of the direct COO kernel for `ops` (rpt_off unused, nz_off = the caller's entry offsets).
CooSchedule make_coo_schedule(const DirOps& ops, int F, const Knobs& kn);

// The non-empty items of a schedule whose compact table is `compact`.
std::vector<bspmm_item> items_of(const Schedule& s, const ItemTable& compact);

// Build the single-launch schedule for `ops` at feature width F.
Schedule make_schedule(const DirOps& ops, int F, const Knobs& kn);

}  // namespace bspmm
