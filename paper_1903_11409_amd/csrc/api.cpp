// C ABI of libbspmm (see include/bspmm.h for the contract of every entry point).
#include <hip/hip_runtime.h>
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <new>
#include <set>
#include <memory>
#include <utility>
#include <vector>

#include "../../include/bspmm.h"
#include "plan.hpp"
#include "plan_api.hpp"
#include "schedule.hpp"
#include "staging.hpp"

namespace bspmm {
hipError_t launch_bspmm(const LaunchParams& P, int grid, int lds_bytes, bool vec4, bool slices,
                        bool hubs, bool merged, hipStream_t stream);
hipError_t launch_bspmm_lean(const LeanItem* items, const LaunchParams& P, int grid, int lds_bytes, bool merged, bool first,
                             hipStream_t stream);
hipError_t launch_bspmm_any(const LeanItem* items, const LaunchParams& P, bool aligned, bool quads, bool first, int grid,
                            int lds_bytes, hipStream_t stream);
hipError_t launch_lean_hints(LeanItem* items, int n, const int32_t* rpt, hipStream_t stream);
hipError_t launch_first_transposed(const LeanItem* items, const LaunchParams& P, int grid, int lds_bytes, int32_t* rpt_t,
                                   int32_t* colids_t, float* values_t, hipStream_t stream);
hipError_t launch_bspmm_gcn(const LaunchParams& P, int grid, int lds_bytes, bool accumulate,
                            bool sets, bool wide, hipStream_t stream);
int front_workgroups_per_cu(bool sets, bool wide, int lds_bytes);
bool layer_supported(int ks, int units, int rb, int waves);
int layer_workgroups_per_cu(int ks, int units, int rb, int waves, int lds_bytes);
hipError_t launch_bspmm_layer(const LayerParams& P, int ks, int units, int rb, int waves, int lds_bytes, hipStream_t stream);
hipError_t launch_layer_rows(const LayerSet* sets, int count, const OpRecord* ops, const int32_t* rpt,
                             const int32_t* colids, const float* values, int32_t* starts, int32_t* entries,
                             int32_t* out_rows, hipStream_t stream);
hipError_t launch_build_transpose(const OpRecord* ops, int batch, int threads, int lds_bytes,
                                  const int32_t* rpt, const int32_t* colids,
                                  const float* values, int32_t* rpt_t, int32_t* colids_t,
                                  float* values_t, int32_t* gscratch, const int32_t* order,
                                  hipStream_t stream);
hipError_t launch_build_from_coo(const OpRecord* ops, int batch, int threads, int lds_bytes, const int32_t* ids,
                                 const float* values, int32_t* rpt, int32_t* colids,
                                 float* csr_values, int32_t* gscratch, const int32_t* order,
                                 hipStream_t stream);
hipError_t launch_bspmm_coo(const CooLaunchParams& P, int grid, int lds_bytes, bool vec4,
                            hipStream_t stream);
hipError_t launch_merge_sets(const SetRecord* sets, int count, const int32_t* rpt,
                             const int32_t* colids, const float* values, int32_t* merged,
                             hipStream_t stream);
hipError_t launch_validate_coo(const OpRecord* ops, int batch, const int32_t* ids, int32_t* flag,
                               hipStream_t stream);
int bspmm_max_resident_workgroups(int lds_bytes, bool slices, bool hubs);
hipError_t kernel_resources(int which, int lds_bytes, int out[7]);
hipError_t launch_validate(const OpRecord* ops, int batch, const int32_t* rpt,
                           const int32_t* colids, int32_t* flag, hipStream_t stream);
}  // namespace bspmm

using namespace bspmm;


// Workspace of plans made by bspmm_create_static: device memory that belongs to the library's
// code object, so no allocation is needed to get it.  Every GPU the library runs on holds its own
// copy at its own address until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress (see static_workspace below); it is never passed to a kernel or a copy.
static __device__ __align__(256) unsigned char scratch[BSPMM_STATIC_WORKSPACE_BYTES];

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return BSPMM_EHIP;
}

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Where each table sits inside the workspace (byte offsets).  The tables the host writes come first
// (one image, one copy), what the device builds behind them.
struct Layout {
    size_t items[2] = {0, 0};
    size_t lean[2] = {0, 0};     // item tables of the lean kernel (empty when a direction is not lean)
    size_t op_records = 0;
    size_t build_order = 0;
    size_t rpt_t = 0, colids_t = 0, values_t = 0;
    size_t scratch = 0;
    size_t flag = 0;
    // summed sets (BSPMM_ACCUMULATE), per direction: their records and their merged CSR arrays
    size_t sets[2] = {0, 0};
    size_t merged[2] = {0, 0};
    // layers run by resident workgroups: graph records, the items of the graphs that stay with the
    // one-launch kernel, and the arrays the device builds
    size_t stream_sets = 0, stream_items = 0, stream_rest = 0, stream_arrays = 0;
    // plans made from COO operands: the CSR arrays built on the device and what the build needs
    size_t coo_records = 0;
    size_t csr_rpt = 0, csr_colids = 0, csr_values = 0;
    size_t coo_scratch = 0;
    size_t image = 0;            // bytes of the host-written front
    size_t total = 0;
};

}  // namespace

struct bspmm_plan {
    bool counted = false;           // (staging.hpp: one of the plans that exist)
    int static_device = -1;         // >= 0: the workspace is that device's static array ...
    uint64_t static_generation = 0; // ... as handed out by this call of bspmm_create_static
    int32_t batch = 0;
    int32_t F = 0;
    bool dry = false;
    int front_wide = 0;             // the one-launch layer kernel runs with workgroups of eight wavefronts
    Knobs knobs;
    DirOps dir[2];
    Schedule sched[2];
    std::vector<OpRecord> records;
    std::vector<int32_t> build_order;      // operations, most entries first: the order the build
                                           // kernels take them in
    ItemTable lean_items[2];            // per direction: the compact item table of a `whole` schedule
    bool lean_shared = false;              // both directions run from the forward table
    bool sorts_in_run = false;             // ... and the first transposed run may build the transposed arrays itself
    int32_t lean_rows[2] = {0, 0};         // most input rows / output rows of an operation, or of a summed
    int32_t lean_out_rows[2] = {0, 0};     // set that is one item: bounds of the lean kernel's 32-bit offsets
    bool lean_blocks[2] = {false, false};  // the lean table has row blocks of the generic bin ...
    bool lean_ranges[2] = {false, false};  // ... and a run has left their entry ranges in it
    StagedCopy upload;          // the copy of the tables from pinned memory, until it is known to have run ...
    hipStream_t upload_stream = nullptr;   // ... and the stream it was enqueued on
    hipEvent_t copied = nullptr;           // ... or the event behind the copy from pageable memory
    std::vector<char> tables;   // host image of the workspace's front, for copies from pageable memory
    Layout lay;
    int build_lds_bytes = 0;
    int build_threads = kThreads;          // lanes per workgroup of the build kernels
    int64_t scratch_words = 0;
    bool transposed_supported = true;
    bool transposed_built = false;
    std::vector<SetRecord> set_records[2];   // summed sets of the forward / transposed schedule
    int64_t merged_words[2] = {0, 0};
    bool merged_built[2] = {false, false};
    int front_channels = 1;   // fused front with BSPMM_ACCUMULATE: channels per output block
    // Layers in launches of many rounds (bspmm_layer_kernel): the graphs whose rows are cut into blocks,
    // and the items of the others, for a launch of bspmm_gcn_kernel of their own.
    struct Stream {
        // Channels that one launch adds up (all of them, or halves where K = channels n_X is more than a
        // wavefront's registers hold weights for): its graph records, and its arrays in the workspace.
        struct Part {
            int first_channel = 0, channels = 0, ks = 0, lds_bytes = 0, ranges_per_xcd = 0, slots = 0;
            size_t sets_at = 0;                                       // first record
            int64_t starts_at = 0, entries_at = 0;                    // words from the arrays' base
        };
        std::vector<Part> parts;
        std::vector<LayerSet> sets;
        std::vector<LayerItem> items;    // small layers of one channel: the blocks, read from the CSR arrays
        std::vector<WorkItem> rest;
        int units = 0, rb = 0, waves = 4, tiles = 0, blocks = 0, direct_entries = 0;
        int64_t out_rows_at = 0, words = 0;
        bool built = false;
        int graphs = 0;
        bool many = false;           // enough graphs to be reported as streamed
        bool on() const { return !parts.empty(); }
    } stream;
    int64_t effective_bytes[2] = {0, 0};
    int64_t flops = 0;
    int64_t covered[2] = {-1, -1};   // covered_rows(), once asked
    bool reads_dense = false;   // some operation has rows and columns: the runs read the dense input
    // borrowed device pointers
    const int32_t* rpt = nullptr;
    const int32_t* colids = nullptr;
    const float* values = nullptr;
    char* ws = nullptr;
    // COO / SparseTensor input: borrowed pair array and values, records of the conversion
    bool from_coo = false;
    const int32_t* ids = nullptr;
    const float* coo_values = nullptr;
    std::vector<OpRecord> coo_records;
    int coo_build_lds_bytes = 0;
    int64_t csr_rpt_words = 0, csr_nz = 0, coo_scratch_words = 0;
    // BSPMM_COO_DIRECT: no CSR at all, the runs launch the direct COO kernel
    bool coo_direct = false;
    CooSchedule coo_sched[2];
};

namespace {

int check_batch(const bspmm_batch* b, int32_t F, bool need_device)
{
    if (!b || F <= 0 || b->batch < 0) return BSPMM_EINVAL;
    if (b->batch == 0) return BSPMM_OK;
    if (!b->rows || !b->cols || !b->nnz || !b->rpt_off || !b->nz_off || !b->b_row_off ||
        !b->c_row_off)
        return BSPMM_EINVAL;
    int64_t total_nnz = 0;
    for (int i = 0; i < b->batch; ++i) {
        if (b->rows[i] < 0 || b->cols[i] < 0 || b->nnz[i] < 0) return BSPMM_EINVAL;
        if (b->rpt_off[i] < 0 || b->nz_off[i] < 0 || b->b_row_off[i] < 0 || b->c_row_off[i] < 0)
            return BSPMM_EINVAL;
        if ((b->rows[i] == 0 || b->cols[i] == 0) && b->nnz[i] != 0) return BSPMM_EINVAL;
        total_nnz += b->nnz[i];
    }
    if (need_device) {
        if (!b->rpt) return BSPMM_EINVAL;
        if (total_nnz > 0 && (!b->colids || !b->values)) return BSPMM_EINVAL;
    }
    return BSPMM_OK;
}

// How the half-open row intervals [off, off+len) with len > 0 relate:
// 0 = pairwise disjoint, 1 = some are identical but none overlaps otherwise, 2 = real overlap.
int overlap_kind(const int64_t* off, const int32_t* len, int n)
{
    bool in_order = true;   // the usual case: blocks back to back in operation order
    int64_t end = 0;
    for (int i = 0; i < n && in_order; ++i) {
        if (len[i] <= 0) continue;
        in_order = off[i] >= end;
        end = off[i] + len[i];
    }
    if (in_order) return 0;
    std::vector<std::pair<int64_t, int64_t>> v;
    v.reserve(n);
    for (int i = 0; i < n; ++i)
        if (len[i] > 0) v.emplace_back(off[i], off[i] + len[i]);
    std::sort(v.begin(), v.end());
    int kind = 0;
    for (size_t i = 1; i < v.size(); ++i) {
        if (v[i] == v[i - 1])
            kind = std::max(kind, 1);
        else if (v[i].first < v[i - 1].second)
            return 2;
    }
    return kind;
}

// The sets of summed operations of direction d: one record per set for the kernel that merges
// their CSR arrays, room for the merged arrays, and the location of those in the first item of
// every task of the set (its rpt_off, nz_off and nnz then describe the merged CSR).
void describe_sets(bspmm_plan& p, int d)
{
    Schedule& sc = p.sched[d];
    const DirOps& o = p.dir[d];
    std::vector<SetRecord>& recs = p.set_records[d];
    recs.clear();
    int64_t words = 0;
    auto describe = [&](const std::vector<int>& mem, bool plain) {
        SetRecord r;
        std::memset(&r, 0, sizeof r);
        r.members = (int32_t)mem.size();
        r.m = o.m[mem[0]];
        r.plain = plain ? 1 : 0;
        int32_t rows = 0;
        int64_t nnz_sum = 0;
        for (size_t j = 0; j < mem.size(); ++j) {
            r.rpt_off[j] = o.rpt_off[mem[j]];
            r.nz_off[j] = o.nz_off[mem[j]];
            r.nnz[j] = o.nnz[mem[j]];
            r.k[j] = o.k[mem[j]];
            size_t owner = j;
            for (size_t e = 0; e < j; ++e)
                if (o.in_off[mem[e]] == o.in_off[mem[j]] && o.k[mem[e]] == o.k[mem[j]]) {
                    owner = e;
                    break;
                }
            if (owner == j || (plain && d == 0 && p.knobs.front > 0)) {   // (front: a tile per channel)
                r.tile_row[j] = rows;
                rows += o.k[mem[j]];
            } else {
                r.tile_row[j] = r.tile_row[owner];
            }
            nnz_sum += o.nnz[mem[j]];
        }
        r.merged_rpt_off = words;
        words += round_up(r.m + 1, 4);
        r.merged_nz_off = words;
        words += 2 * (int64_t)round_up((int)nnz_sum, 4);
        recs.push_back(r);
        return (int32_t)nnz_sum;
    };
    // sets run as fused tasks, then sets an operation with the summed matrix stands in for
    std::vector<int32_t> nnz_sum;
    for (const std::vector<int>& mem : sc.fused_sets) nnz_sum.push_back(describe(mem, false));
    const size_t first_plain = recs.size();
    for (const std::vector<int>& mem : sc.merged_sets) describe(mem, true);
    p.merged_words[d] = words;
    for (size_t t = 0; t < sc.task_set.size(); ++t) {
        const int si = sc.task_set[t];
        WorkItem& w = sc.items[(size_t)sc.item_base[1] + t * sc.fused_stride];
        w.rpt_off = recs[si].merged_rpt_off;
        w.nz_off = recs[si].merged_nz_off;
        w.nnz = nnz_sum[si];
    }
    if (!sc.merged_sets.empty())
        for (size_t j = 0; j < sc.items.size(); ++j) {
            const int op = j < sc.item_op.size() ? sc.item_op[j] : -1;
            if (op < sc.first_stand_in) continue;
            const SetRecord& r = recs[first_plain + (size_t)(op - sc.first_stand_in)];
            sc.items[j].rpt_off = r.merged_rpt_off;
            sc.items[j].nz_off = r.merged_nz_off;
        }
}

// Layers (bspmm_run_gcn): the plan of the gather-first launch (bspmm_layer_kernel).  The output rows of the
// graphs, one after the other in the order of their layer input, are cut into blocks of 16, 32 or 64; a
// workgroup takes a run of blocks and 64 or 128 columns.  The device writes what the blocks read
// (layer_rows_kernel), the host only places every graph's share.
void make_stream_plan(bspmm_plan& p)
{
    bspmm_plan::Stream& st = p.stream;
    st = bspmm_plan::Stream();
    const Schedule& sc = p.sched[0];
    const Knobs& kn = p.knobs;
    const int nx = kn.front, F = p.F;
    if (nx <= 0 || kn.one_front_launch || !sc.fused_sets.empty() || sc.fused_tasks > 0) return;
    if (nx != 16 && nx != 32 && nx != 64 && nx != 128) return;
    // (plans of single channels - no operations summed - take the same kernel with one channel)
    const bool single = sc.merged_sets.empty();
    const int channels = single ? 1 : p.front_channels;
    if (channels < 1 || channels > kMaxMembers || (!single && !kn.accumulate)) return;
    const DirOps& o = p.dir[0];
    const size_t n_graphs = single ? (size_t)o.size() : sc.merged_sets.size();
    auto op_of = [&](size_t g, int c) { return single ? (int)g : sc.merged_sets[g][(size_t)c]; };
    // Launches of two (graph, 32 columns) and more per CU - of one channel also 700,000 elements of layer
    // input on 256 CUs - are the ones that bspmm_info.front_stream reports (resident workgroups).
    st.many = (int64_t)n_graphs * ((F + 31) / 32) >= (single ? 4 : 2) * (int64_t)kn.compute_units;
    if (single) {
        int64_t x_rows = 0;
        for (int i = 0; i < o.size(); ++i) x_rows += o.k[i];
        st.many = st.many && x_rows * nx * 256 >= (int64_t)700000 * kn.compute_units;
    }

    // Fewer graphs: one block to a workgroup, where there are enough to matter.  Blocks of one channel are rows
    // of one operation then, whose CSR arrays the kernel reads as they are: the first run of a plan needs no
    // other launch (whole layers merge their channels' CSR arrays for either kernel).
    const bool direct = single && !st.many;

    // The graphs in the order of their layer input; those with more entries per row than `degree` keep their
    // items of the one-launch schedule.  What a row costs here grows with its entries, n_X floats each, and on the
    // one-launch kernel with the dense tile, F floats for every row and channel, and less with the entries.  us,
    // F = 128, molecules of so many entries per row (all channels), this kernel / one-launch:
    //   four channels, n_X = 64, 2048 graphs: 3 32 / 120, 8 37 / 125, 24 52 / 143, 64 91 / 260; 128 graphs: 8
    //   8 / 15, 24 11 / 18, 64 14 / 36;   eight channels, 1024 graphs: 8 40 / 158, 64 63 / 214
    //   one channel, 2048 graphs: 8 24 / 34, 16 32 / 40, 24 44 / 66, 48 72 / 91; 600 graphs: 16 13 / 16, 24 21 / 18,
    //   48 31 / 29;   n_X = 128, 1024 graphs: 24 31 / 46, 48 44 / 56;   n_X = 16, F = 64, 2048 graphs: 8 11 / 13, 16
    //   17.7 / 17.2, 32 24 / 26, 48 36 / 42, 64 78 / 51
    // so that a batch of one kind stays here.  A few graphs of many entries in a batch of few make long trips:
    // past 32 and twice the average they are left out (every 40th graph of 24 / 48 entries per row, the others
    // 2.2: one channel 21 / 40 here, 21 / 24 with them left out; four channels 38 / 46, 45 / 43).
    // One channel: a graph that fills nearly two ranges of a workgroup, of 128 rows and more each, and has a
    // third more entries per row than the average, is left out too.  Its ranges end last, but not by as much as
    // the other launch takes (2048 skewed graphs at n_X = 64, F = 64, eleven of them left out: 35 us -> 52; the
    // streaming kernel before this one, which left 149 out, 60): it is test_single_channel_streamed that
    // wants a graph left out of a batch of that kind.
    // One operation to a block (`direct`): n_X = 16 up to six (F = 16, 200 graphs of 4 / 6 / 8: 4.1 / 4.4 / 4.7,
    // one-launch 4.2 / 4.3 / 4.5), else eight (n_X = 128, F = 64, 48 graphs of 6 / 8 / 12: 5.6 / 6.2 / 6.8, one-launch
    // 5.9 / 6.1 / 6.3; n_X = 64, F = 128, 200 graphs: 5.6 / 6.0 / 6.4, one-launch 7.5 / 7.7 / 9.0).
    constexpr int64_t kLimit = (int64_t)1 << 31;
    int64_t all_rows = 0, all_entries = 0;
    for (size_t g = 0; g < n_graphs; ++g) {
        if (o.m[op_of(g, 0)] <= 0) continue;
        all_rows += o.m[op_of(g, 0)];
        for (int c = 0; c < channels; ++c) all_entries += o.nnz[op_of(g, c)];
    }
    const double mean = (double)all_entries / (double)std::max<int64_t>(all_rows, 1);
    const double degree = direct ? (nx == 16 ? 6.0 : 8.0) : std::max(32.0, 2 * mean);
    const double range = (double)all_rows * ((F + 127) / 128) / (3.0 * kn.compute_units);
    // Fewer columns than the layer input has: here a row still gathers n_X floats for every entry, and wavefronts
    // past F have no columns to multiply, while the other kernel's dense tile is narrow.  Batches of more entries per
    // row than `narrow` stay there; the line moves with the 16-row blocks per CU (up to one, up to three, more).  us,
    // this kernel / one-launch, 100 | 400 | 1500 molecules (0.6 | 2.4 | 9 blocks per CU):
    //   F = 16, one channel, n_X = 64, 2.2 entries per row 4.3 / 4.7 | 5.0 / 5.7 | 9.7 / 8.7, 5 4.3 / 4.9 | 6.7 / 5.9 |
    //   11.4 / 9.0;   n_X = 128, 5 5.6 / 6.1 | 9.7 / 11.2 | 18.0 / 13.2;   three, n_X = 64, 2.2 6.0 / 6.6 | 8.5 / 8.9 |
    //   15.9 / 14.4, 5 6.7 / 6.7 | 9.4 / 8.9 | 18.1 / 14.9;   n_X = 128, 5 9.5 / 9.9 | 17.2 / 12.2 | 32.6 / 24.7
    //   F = 32, one channel, n_X = 64, 5 4.3 / 5.1 | 6.8 / 6.9 | 11.5 / 11.1, 8 4.6 / 5.1 | 7.5 / 8.2 | 13.7 / 11.5;
    //   three, n_X = 128, 5 9.6 / 10.0 | 17.3 / 15.7 | 32.7 / 37.3, 16 12.1 / 11.2 | 22.4 / 19.1 | 46.0 / 39.8;   eight,
    //   n_X = 128, 2.2 18.6 / 15.3 | 33.2 / 35.8 | 61.5 / 112
    //   F = 48, one channel, n_X = 64, 8 4.6 / 5.6 | 7.5 / 8.8 | 13.9 / 14.8, 16 - | - | 20.7 / 16.4;   three, n_X = 128, 8 10.5
    //   / 10.5 | 19.2 / 21.0 | 38.0 / 64.1, 16 12.1 / 11.2 | 22.4 / 21.7 | 46.2 / 65.5;   eight, 5 20.2 / 20.4, 8 22.4 / 20.5
    //   n_X = 32, F = 16, one channel, 2.2 3.8 / 4.4 | 4.8 / 5.2 | 7.0 / 6.9, 5 4.0 / 4.5 | 4.8 / 5.6 | 8.8 / 7.1
    //   F = 64, 100 molecules: two channels, n_X = 64, 30 9.0 / 7.8;   three, n_X = 64 8.1 / 8.3, n_X = 128 8
    //   10.6 / 10.7, 16 12.1 / 11.5;   eight, n_X = 128, 5 20.2 / 20.5, 8 22.2 / 20.7
    // Graphs of hundreds of rows take the other kernel several passes each, one after the other (907 skewed graphs of
    // up to 500 rows, three channels, n_X = 128, F = 16: 34.9 / 62.9).
    // Whole layers of half a block per CU and less: six entries per row (us, 45 graphs of three channels, n_X = 32, F = 64,
    // 30 per row 8.1 / 7.0; 70 of eight, n_X = 128, F = 96, 14 per row 24.1 / 21.7).
    if (!single && all_rows / 8 <= kn.compute_units && mean > 6) return;
    // One channel by resident workgroups: up to fourteen where the launch is short (n_X = 64, F = 128, 600 graphs, 3.7 blocks
    // per CU, 12 / 16 / 24 per row 11.5 / 18.3 / 21.2, one-launch 14.7 / 15.9 / 17.6; 2048 graphs, see above, any) or the rows
    // are (n_X = 16).
    if (single && !direct && mean > 14 && (nx == 16 || (nx == 64 && all_rows / 16 <= 6 * kn.compute_units))) return;
    int64_t most_rows = 0;
    for (size_t g = 0; g < n_graphs; ++g) most_rows = std::max<int64_t>(most_rows, o.m[op_of(g, 0)]);
    if (most_rows <= 192 && (F < 64 ? nx > F : F == 64 && nx >= 64)) {
        const int64_t per_cu = (all_rows / 16 + kn.compute_units - 1) / kn.compute_units;
        const bool few = per_cu <= 1, many = per_cu > 3;
        const int K = channels * nx;
        double narrow = 1e9;
        if (nx < 64) {
            if (F <= 16 && many && K <= 128) narrow = single ? 3 : 5;
        } else if (F <= 16) {
            narrow = many || K > (few ? 384 : 192) ? 0 : few ? 5 : single ? nx / 16 : 3;
        } else if (few) {
            if (!single) narrow = K > 512 ? (F <= 32 ? 0 : 5) : F <= 32 ? 5 : F < 64 ? 8 : nx == 128 ? 10 : 18;
        } else if (F == 64) {      // (no line found)
        } else if (many) {
            if (single) narrow = F <= 32 ? 3 : 10;
            else if (F <= 32 && nx == 128 && K <= 384) narrow = 8;
        } else if (nx == 128 && !single) {
            narrow = F <= 32 ? 3 : 13;
        }
        if (mean > narrow) return;
    }
    std::vector<int> mine;
    std::vector<char> streamed(n_graphs, 0);
    int64_t rows = 0, entries = 0;
    for (size_t g = 0; g < n_graphs; ++g) {
        const int op0 = op_of(g, 0);
        int64_t nnz = 0;
        for (int c = 0; c < channels; ++c) nnz += o.nnz[op_of(g, c)];
        if (o.m[op0] <= 0) continue;
        const double most = single && range >= 128 && o.m[op0] >= 1.75 * range ? std::max(8.0, mean * 4 / 3) : degree;
        if ((double)nnz > std::min(most, degree) * o.m[op0] || o.in_off[op0] + o.k[op0] >= kLimit || o.out_off[op0] + o.m[op0] >= kLimit) {
            if (direct) return;
            continue;
        }
        mine.push_back((int)g);
        streamed[g] = 1;
        rows += o.m[op0];
        entries += nnz;
    }
    if (mine.empty() || (rows + 64) * channels >= kLimit || entries >= kLimit) return;
    // Too few to matter.  us of a run, F = 128, this kernel / one-launch kernel: one channel at n_X = 64, 32
    // graphs 5.4 / 5.6, 64 graphs 4.1 / 6.0, 128 graphs 4.8 / 6.6, 300 graphs 6.6 / 8.5; four channels at n_X = 64, 24
    // graphs 6.4 / 6.6, 128 graphs 7.1 / 14.2; K = channels n_X past 256: 24 graphs of four channels at n_X = 128
    // 9.9 / 8.5, 64 graphs 10.7 / 14.0; two channels at n_X = 128, 24 graphs 7.3 / 6.5, 32 graphs 7.4 / 7.5.
    if (!st.many && (rows + 15) / 16 * (single || channels * nx > 256 ? 4 : (nx == 128 ? 6 : 8)) < kn.compute_units) return;
    int most_k = 0, most_nnz = 0;                        // of an operation: it has to fit on chip
    if (direct) {
        int64_t words = 0;                               // (32-bit offsets)
        for (int g : mine) {
            words = std::max({words, o.rpt_off[g] + o.m[g] + 1, o.nz_off[g] + o.nnz[g]});
            most_k = std::max(most_k, o.k[g]);
            most_nnz = std::max(most_nnz, o.nnz[g]);
        }
        if (words >= kLimit || most_nnz > 4096) return;
    }
    std::stable_sort(mine.begin(), mine.end(),
                     [&](int a, int b) { return o.in_off[op_of(a, 0)] < o.in_off[op_of(b, 0)]; });

    // channels per launch: K = channels n_X up to 512 (96 registers per 16 columns and 256 of K)
    const int launches = channels * nx > 512 ? 2 : 1;
    const int most = (channels + launches - 1) / launches;
    static const int kSteps[] = {1, 2, 3, 4, 6, 8, 12, 16};
    auto steps_of = [&](int ch) {
        for (int k : kSteps)
            if (32 * k >= ch * nx) return k;
        return 0;
    };
    // Shape of a workgroup.  Past 64 columns: four wavefronts of 32 columns up to K = 48, eight of 16 columns
    // from K = 64 on (a lane then holds half the weights and twice the wavefronts hide each other's
    // latencies: us at 700 molecules, F = 128, four against eight: K = 32 7.2 / 8.6, K = 64 8.6 / 8.7, K = 128
    // 13.1 / 12.0, K = 256 17.4 / 15.0, K = 512 30.0 / 26.1; 2048 at K = 64 16.8 / 14.8); more than four
    // channels have no register for a second bias there up to K = 256.  Launches that leave half the chip
    // idle that way take tiles of 64 columns (64 molecules, K = 64 5.2 / 4.9 / 4.7, K = 256 7.6 / 6.7 / 6.4).
    int units = steps_of(most) <= 8 && F > 64 ? 2 : 1, waves = 4;
    if (F > 64 && most * nx >= 64 && (most <= 4 || most * nx > 256)) units = 1, waves = 8;
    if (F > 64 && (rows + 15) / 16 * 2 * ((F + 127) / 128) <= kn.compute_units) units = 1, waves = 4;
    const int tiles = (F + 16 * waves * units - 1) / (16 * waves * units);
    // LDS: a third of a CU's; half of it where that holds the rows of X of few entries.  Rows of a block: up
    // to 64 where the rows of X that they name (a quarter more than on average) then have slots, by the
    // number of trips times what a trip costs: a fixed part and the passes of its gather (one channel at
    // n_X = 16, F = 64, 2048 molecules, 16 / 32 / 64 rows: 11.2 / 9.4 / 9.2 us; at n_X = 64, 1200: 9.3 / 9.8).
    // (no more than 1024 slots: 256 had blocks of four entries per row at n_X = 16 past them, 9.9 -> 8.9 us)
    // (eight wavefronts past K = 256 hold so many registers that a CU has one workgroup whatever its LDS: us, four channels at
    // n_X = 128, F = 128, 53 / 128 KiB: 1500 molecules 47.0 / 44.5, 300 15.3 / 14.7; three channels, eight at n_X = 64 level.
    // By the channels of the launch: five of 128 run as three and two, whose K = 256 leaves room for two workgroups; 1500
    // graphs of 9 / 17 entries per row, 53 / 128 KiB in both launches / as it is 73.0 / 79.7 / 73.2, 81.0 / 87.8 / 80.5)
    auto lds_budget = [&](int ch) { return kn.lds_given ? kn.lds_words * 4 : waves == 8 && !direct && steps_of(ch) > 8 ? 131072 : 53248; };
    const int budget = lds_budget(most);
    constexpr int kSlots = 1024;
    auto slots_in = [&](int rb, int ch, int bytes, int want) {
        const int unit = 256 / nx;             // rows that a wavefront's request brings
        int n = round_up(std::min(want, kSlots), unit);
        while (n > 0 && layer_lds(steps_of(ch), rb, waves, ch, n, n, nx).total > bytes) n -= unit;
        return n;
    };
    const double per_row = (double)entries / (double)rows;
    auto wanted = [&](int rb) { return (int)(20.0 * rb * per_row) + 16; };
    int rb = 1;
    {
        const int groups = 256 * waves / nx;     // virtual rows that a pass takes
        double best = 0;
        for (int r = 1; r <= (direct ? 1 : 4); r *= 2) {
            if (!layer_supported(steps_of(most), units, r, waves) || 16 * r * most > 240 ||
                (r > 1 && slots_in(r, most, budget, wanted(r)) < std::min(wanted(r), kSlots)))
                continue;
            const int64_t round = (int64_t)16 * r * 3 * kn.compute_units;
            const int64_t trips = (rows * tiles + round - 1) / round;
            const double cost = (double)trips * (1 + (16 * r * most + groups - 1) / groups);
            if (r == 1 || cost < best) {
                best = cost;
                rb = r;
            }
        }
    }
    int64_t blocks = (rows + 16 * rb - 1) / (16 * rb);
    if (direct)
        for (int g : mine)
            for (int r0 = 0; r0 < o.m[g]; r0 += 16) {
                LayerItem t = {};
                t.rpt_off = (uint32_t)(o.rpt_off[g] + r0);
                t.nz_off = (uint32_t)o.nz_off[g];
                t.in_row = (uint32_t)o.in_off[g];
                t.out_row = (uint32_t)(o.out_off[g] + r0);
                t.nrows = std::min(16, o.m[g] - r0);
                t.k = o.k[g], t.nnz = o.nnz[g];
                st.items.push_back(t);
            }
    if (direct) blocks = (int64_t)st.items.size();
    // Rows of 16 floats are a quarter of a wavefront's gather each, and a workgroup's start is most of its time:
    // past so many workgroups per CU the one-launch kernel, a workgroup to a graph, is the faster one up to F = 64.
    // us, this kernel / that one, molecules of 2.2 to 5.5 entries per row: F = 16, 500 graphs (4.0 workgroups per CU)
    // 4.6 to 5.1 / 4.9 to 5.3, 800 6.1 to 6.5 / 5.2 to 5.7; F = 32, 500 4.7 to 5.2 / 5.3 to 5.7, 700 (5.6) 5.8 to 6.2 / 5.3
    // to 5.8; F = 64, 800 (6.4) 6.6 to 7.1 / 7.1 to 7.2, 1000 (8.1) 7.2 to 8.4 / 7.5 to 7.9, 1300 8.7 to 9.6 / 8.6 to 8.9,
    // skewed graphs 400 (6.7) 11.5 to 13.7 / 12.5 to 15.1, 500 14.3 to 17.0 / 12.6 to 14.9; F = 128, 1600 13.4 to 15.1 /
    // 15.0 to 16.4; F = 256, 1300 19.3 to 21.6 / 21.7 to 23.7.
    if (direct && nx == 16 && F <= 64 && 16 * blocks * tiles > (int64_t)kn.compute_units * (F + 56)) {
        st = bspmm_plan::Stream();
        return;
    }
    st.units = units;
    st.rb = rb;
    st.waves = waves;
    st.tiles = tiles;
    st.blocks = (int)blocks;
    int64_t at = 0;
    auto place = [&at](int64_t words) {
        const int64_t here = at;
        at += (words + 3) / 4 * 4;
        return here;
    };
    if (!direct) st.out_rows_at = place(16 * rb * blocks);
    for (int c0 = 0; c0 < channels; c0 += most) {
        bspmm_plan::Stream::Part part;
        part.first_channel = c0;
        part.channels = std::min(most, channels - c0);
        part.ks = steps_of(part.channels);
        if (!layer_supported(part.ks, units, direct ? 0 : rb, waves)) {
            st = bspmm_plan::Stream();
            return;
        }
        part.slots = slots_in(rb, part.channels, lds_budget(part.channels), std::max(wanted(rb), 64));
        if (direct) {
            part.slots = round_up(std::max(most_k, 1), 256 / nx);
        } else if (!kn.lds_given) {
            // (half of a CU's LDS too, past six entries per row, where it holds the rows of X of a block, a tenth
            // more than on average, and a third does not: us, one channel, F = 128, third / half: n_X = 64, 2048 molecules of 8 / 10 / 12 / 16
            // entries per row 23.7 / 23.6, 27.3 / 25.8, 32.2 / 27.4, 36.5 / 32.3, and 24, which neither holds, 44.2 /
            // 48.6; n_X = 32, 1024 of 16 / 24 / 48: 13.8 / 13.8, 22.0 / 19.0, 30.2 / 39.7)
            const int block = (int)(17.6 * rb * per_row * part.channels / channels);
            const int half = slots_in(rb, part.channels, 81920, std::max(wanted(rb), 64));
            if (part.slots < 40 || (per_row > 6 && part.slots < block && half >= block)) part.slots = half;
        }
        if (part.slots < 16 && !direct) {
            st = bspmm_plan::Stream();
            return;
        }
        part.lds_bytes = layer_lds(part.ks, rb, waves, part.channels, part.slots, direct ? most_nnz : part.slots, nx).total;
        // (operations that do not fit half of a CU's LDS: the one-launch kernel)
        if (direct && part.lds_bytes > (kn.lds_given ? budget : 81920)) {
            st = bspmm_plan::Stream();
            return;
        }
        st.direct_entries = most_nnz;
        int per_cu = kn.device_ok ? layer_workgroups_per_cu(part.ks, units, direct ? 0 : rb, waves, part.lds_bytes) : 0;
        if (per_cu <= 0) per_cu = 2;
        // (eight wavefronts with two 16-row blocks: no third workgroup, whose weights cost more than its trips
        // save: us, one channel, n_X = 64, F = 128, two / three per CU: 512 skewed graphs 10.9 / 13.5, 1299 molecules,
        // accumulating 23.5 / 30.0, 2048 molecules 15.6 / 14.2)
        per_cu = std::min(per_cu, waves == 8 && rb == 2 ? 2 : 3);
        const int64_t most_ranges = std::max<int64_t>(8, (int64_t)per_cu * kn.compute_units / st.tiles);
        const int64_t ranges = direct || blocks <= most_ranges ? blocks + 7 : most_ranges;
        part.ranges_per_xcd = (int)std::max<int64_t>(ranges / 8, (blocks / kLayerRangeBlocks + 8) / 8);
        if (direct) {
            st.parts.push_back(part);
            break;
        }
        part.sets_at = st.sets.size();
        int64_t row = 0, entry = 0;
        for (int g : mine) {
            const int op0 = op_of(g, 0);
            LayerSet r;
            std::memset(&r, 0, sizeof r);
            for (int c = 0; c < part.channels; ++c) {
                const int op = op_of(g, c0 + c);
                r.op[c] = op;
                r.entries += o.nnz[op];
            }
            r.m = o.m[op0];
            r.in_row = (int32_t)o.in_off[op0];
            r.out_row = (int32_t)o.out_off[op0];
            r.channels = part.channels;
            r.first_row = (int32_t)row;
            r.first_entry = (int32_t)entry;
            r.pad_rows = -1;
            row += r.m;
            entry += r.entries;
            st.sets.push_back(r);
        }
        st.sets.back().pad_rows = (int32_t)(16 * rb * blocks - rows);
        part.starts_at = place(16 * rb * blocks * part.channels + 4);
        part.entries_at = place(2 * (entry + part.slots));      // (requests always ask for a slot's worth each)
        st.parts.push_back(part);
    }
    st.words = at;
    st.graphs = (int)mine.size();
    // the other graphs: their items of the one-launch schedule, in its order
    for (size_t j = 0; j < sc.items.size(); ++j) {
        const int op = j < sc.item_op.size() ? sc.item_op[j] : -1;
        if (op < (single ? 0 : sc.first_stand_in) || sc.items[j].nrows <= 0) continue;
        if (!streamed[(size_t)(op - (single ? 0 : sc.first_stand_in))]) st.rest.push_back(sc.items[j]);
    }
}

// The compact item table of direction d, when the schedule is made of whole-workgroup items and every
// offset fits the table's 32-bit fields (else the direction keeps the general kernel).  Plain
// batches come with it.
void make_lean_items(bspmm_plan& p, int d)
{
    Schedule& sc = p.sched[d];
    ItemTable& out = p.lean_items[d];
    out.clear();
    p.lean_blocks[d] = false;
    if (!sc.whole) return;
    if (!sc.compact.empty()) {
        out = std::move(sc.compact);
        p.lean_blocks[d] = sc.row_blocks;
        return;
    }
    constexpr int64_t kLimit = (int64_t)1 << 31;
    if (p.merged_words[d] >= kLimit) {
        sc.whole = sc.pow2 = false;
        return;
    }
    for (const WorkItem& w : sc.items) {
        p.lean_rows[d] = std::max(p.lean_rows[d], w.k);   // (a summed set's: the rows of all its members)
        p.lean_out_rows[d] = std::max(p.lean_out_rows[d], w.m);
        LeanItem t;
        std::memset(&t, 0, sizeof t);
        if (w.nrows > 0) {
            if (w.rpt_off >= kLimit || w.nz_off >= kLimit || w.in_row_off >= kLimit ||
                w.out_row_off >= kLimit) {
                out.clear();
                sc.whole = sc.pow2 = false;
                return;
            }
            int sh = 0;
            while ((4 << sh) < w.fw) ++sh;
            t.rpt_off = (uint32_t)w.rpt_off;
            t.nz_off = (uint32_t)w.nz_off;
            t.in_row = (uint32_t)w.in_row_off;
            t.out_row = (uint32_t)w.out_row_off;
            t.m = w.m, t.k = w.k, t.nnz = w.nnz, t.row0 = w.row0, t.nrows = w.nrows, t.f0 = w.f0;
            t.sh = sh;
            t.flags = w.fw << 8;
            if (w.staged & 1) {
                const StagedLayout L = staged_layout(w.m, w.k, w.nnz, w.fw, 0, false);
                t.flags |= ((w.staged & 2) ? 1 : 0) | ((w.staged & 4) ? 4 : 0);
                t.cv_byte = 4 * L.cv_off;
                t.b_byte = 4 * L.b_off;
                t.tile_vecs = w.k << sh;
            } else {
                t.flags |= 2;    // a row block: its entry range is filled in on the device
                p.lean_blocks[d] = true;
            }
        }
        out.push_back(t);
    }
    sc.items.clear();            // (nothing runs from the long form any more)
}

// How the build kernel sorts an operation of `keys` key values, `nnz` entries and payloads below
// `payloads` (rows of a CSR operand, columns of a COO one); `with_rpt` when the input's row
// pointers come along.  Sets r.small and r.scratch_off and returns the LDS words it needs
// (0 when the operation works in global scratch, whose words are added to *scratch_words).
int64_t classify_build(OpRecord& r, int64_t keys, int64_t payloads, int64_t nnz, bool with_rpt,
                       int threads, int64_t* scratch_words)
{
    const int64_t budget = (kBuildLdsBytes - 2048) / 4;
    const int64_t base = keys + 1 + nnz;                     // counters and positions
    const int64_t reg_path = base + (with_rpt ? payloads + 1 : 0);
    auto bits = [](int64_t v) { int b = 0; while (v > 0) { ++b; v >>= 1; } return b; };
    r.scratch_off = -1;
    if (nnz <= (int64_t)build_entries_per_lane(threads) * threads && reg_path <= budget) {
        r.small = 1;     // register path: a few entries per lane, row pointers in LDS too
        return reg_path;
    }
    if (base + nnz <= budget && bits(keys) + bits(std::max<int64_t>(payloads - 1, 0)) <= 32) {
        r.small = 2;     // key and payload of every entry packed into one more LDS word
        return base + nnz;
    }
    r.small = 0;
    if (base <= budget) return base;
    r.scratch_off = *scratch_words;
    *scratch_words += base;
    return 0;
}

// Fill everything of the plan that needs no device.
int plan_host(bspmm_plan& p, const bspmm_batch* b, int32_t F, const Knobs& kn)
{
    const int n = b->batch;
    p.batch = n;
    p.F = F;
    p.knobs = kn;
    DirOps& f = p.dir[0];
    DirOps& t = p.dir[1];
    int64_t rpt_t_words = 0;
    p.records.resize(n);
    p.build_threads = kThreads;
    for (int i = 0; i < n; ++i)
        if (b->nnz[i] > 4 * kThreads) p.build_threads = kBuildThreadsLarge;
    int64_t nz_pack = 0;
    int64_t scratch_words = 0;
    int build_lds_words = 0;
    for (int d = 0; d < 2; ++d) p.lean_rows[d] = p.lean_out_rows[d] = 0;
    f.m.assign(b->rows, b->rows + n), f.k.assign(b->cols, b->cols + n), f.nnz.assign(b->nnz, b->nnz + n);
    f.rpt_off.assign(b->rpt_off, b->rpt_off + n), f.nz_off.assign(b->nz_off, b->nz_off + n);
    f.in_off.assign(b->b_row_off, b->b_row_off + n), f.out_off.assign(b->c_row_off, b->c_row_off + n);
    // transposed: rows and columns swap, dense input is indexed like C, output like B; the
    // transposed entries are packed back to back in operation order (a symmetric operand is its
    // own transpose: the same arrays serve both directions)
    t.m = f.k, t.k = f.m, t.nnz = f.nnz, t.in_off = f.out_off, t.out_off = f.in_off;
    t.rpt_off = f.rpt_off, t.nz_off = f.nz_off;
    bool same_place = true;      // the transposed arrays have the forward ones' offsets
    for (int i = 0; i < n; ++i) {
        if (kn.symmetric && b->rows[i] != b->cols[i]) return BSPMM_EINVAL;
        if (!kn.symmetric) {
            same_place = same_place && b->rpt_off[i] == rpt_t_words && b->nz_off[i] == nz_pack;
            t.rpt_off[i] = rpt_t_words;
            t.nz_off[i] = nz_pack;
        }
        OpRecord& r = p.records[i];
        r.rpt_off = b->rpt_off[i];
        r.nz_off = b->nz_off[i];
        r.rpt_t_off = rpt_t_words;
        r.nz_t_off = nz_pack;
        r.m = b->rows[i];
        r.k = b->cols[i];
        r.nnz = b->nnz[i];
        build_lds_words = std::max<int64_t>(
            build_lds_words,
            classify_build(r, b->cols[i], b->rows[i], b->nnz[i], true, p.build_threads, &scratch_words));
        rpt_t_words += (int64_t)b->cols[i] + 1;
        nz_pack += b->nnz[i];
    }
    p.build_lds_bytes = (int)round_up(build_lds_words * 4 + 16, 256);
    p.scratch_words = scratch_words;

    const int ck = n > 0 ? overlap_kind(b->c_row_off, b->rows, n) : 0;
    const int bk = n > 0 ? overlap_kind(b->b_row_off, b->cols, n) : 0;
    if (ck == 2 || (ck == 1 && !kn.accumulate)) return BSPMM_EOVERLAP;
    p.transposed_supported = bk == 0 || (bk == 1 && kn.accumulate);

    if (kn.front > 0 && (F % 16 != 0 || kn.front % 4 != 0 || kn.hubs || kn.pad != 0))
        return BSPMM_EINVAL;
    p.knobs.wide_offsets = std::max(rpt_t_words, nz_pack) >= (int64_t)1 << 31;
    p.sched[0] = make_schedule(f, F, p.knobs);
    if (p.sched[0].error) return p.sched[0].error;
    if (kn.front > 0 && kn.accumulate) {
        // the whole layer in one launch: every operation must be a channel of a set, all sets
        // with the same number of channels, the channels of a set sharing the layer input
        const Schedule& sc = p.sched[0];
        size_t in_sets = 0, with_rows = 0;
        for (const auto& mem : sc.merged_sets) {
            if (mem.size() != sc.merged_sets[0].size()) return BSPMM_EINVAL;
            in_sets += mem.size();
        }
        for (int i = 0; i < n; ++i) with_rows += b->rows[i] > 0;
        if (in_sets != with_rows) return sc.fused_tasks > 0 ? BSPMM_ETOOBIG : BSPMM_EINVAL;
        p.front_channels = sc.merged_sets.empty() ? 1 : (int)sc.merged_sets[0].size();
    }
    // Square operations whose input and output blocks sit at the same rows (adjacency matrices
    // of a GCN batch) have the same schedule in both directions: only the location of the
    // CSR arrays differs.
    bool same_shape = kn.front == 0;
    for (int i = 0; i < n && same_shape; ++i)
        same_shape = b->rows[i] == b->cols[i] && b->b_row_off[i] == b->c_row_off[i];
    const bool plain = !p.sched[0].compact.empty();
    if (plain) make_lean_items(p, 0);
    p.lean_shared = p.sorts_in_run = false;
    if (p.transposed_supported && same_shape) {
        p.sched[1] = p.sched[0];
        Schedule& st = p.sched[1];
        for (size_t j = 0; j < st.items.size(); ++j) {
            const int op = st.item_op[j];
            if (op < 0 || op >= n) continue;     // (stand-ins of summed sets: see describe_sets)
            st.items[j].rpt_off = t.rpt_off[op];
            st.items[j].nz_off = t.nz_off[op];
        }
        if (plain) {
            // (the same items again: only the CSR arrays are elsewhere - or not even those, when the
            // caller's are packed in operation order; row blocks carry entry ranges of their own)
            p.lean_shared = same_place && !p.lean_blocks[0];
            // Every workgroup of the product then sorts its operation: 0.5 to 0.9 us per thousand workgroups, against
            // a launch of its own (3.5 us of the host's time, 1.5 between two kernels) for the build, 5 us and 1.5 per
            // thousand operations.  us between events around the first run, build + product / one launch: 60 molecules at
            // F = 64 (136 workgroups) 10.5 / 7.4, 128 at F = 128 (624) 10.9 / 7.9, 2000 tiny graphs (2000) 15.1 / 11.7, 16384
            // molecules (20515) 113.5 / 96.6, 300 random matrices at F = 512 (1592) 24.8 / 21.0, 512 wide graphs at F = 512 (2480)
            // 33.6 / 33.7, 400 at F = 1024 (9016) 49.1 / 52.2, which the launch that the host saves makes level.
            p.sorts_in_run = n > 0 && p.lean_shared && !kn.symmetric && p.build_threads == kThreads &&
                             *std::min_element(b->rows, b->rows + n) > 0 &&
                             (int64_t)p.lean_items[0].size() <= 10000 + 2 * (int64_t)n;
            p.lean_blocks[1] = p.lean_blocks[0];
            if (!p.lean_shared) {
                p.lean_items[1] = p.lean_items[0];
                for (size_t j = 0; j < p.lean_items[1].size(); ++j) {
                    const int op = st.item_op[j];
                    if (op < 0) continue;
                    p.lean_items[1][j].rpt_off = (uint32_t)t.rpt_off[op];
                    p.lean_items[1][j].nz_off = (uint32_t)t.nz_off[op];
                }
            }
        }
    } else if (p.transposed_supported) {
        Knobs kt = p.knobs;
        kt.front = 0;                     // the layer input is a forward-only guest
        p.sched[1] = make_schedule(t, F, kt);
        if (p.sched[1].error) {          // the forward product still works
            if (kn.need_both && p.sched[1].error == BSPMM_ETOOBIG) return BSPMM_ETOOBIG;
            p.sched[1] = Schedule();
            p.transposed_supported = false;
        }
    }
    for (int d = 0; d < 2; ++d) describe_sets(p, d);
    if (!plain) make_lean_items(p, 0);
    if (!plain || !same_shape) make_lean_items(p, 1);

    // compulsory traffic: CSR once, every distinct dense input block once, every output once
    int64_t csr_f = 0, csr_t = 0, out_f = 0, out_t = 0, in_f = 0, in_t = 0, nnz = 0;
    // a dense block counts once as an input and once as an output, however many operations
    // read it or are summed into it
    auto distinct_rows = [n](const int64_t* off, const int32_t* len) {
        bool increasing = true;        // the usual case: blocks back to back in operation order
        for (int i = 1; i < n && increasing; ++i) increasing = off[i] >= off[i - 1] + len[i - 1];
        int64_t rows = 0;
        if (increasing) {
            for (int i = 0; i < n; ++i) rows += len[i];
            return rows;
        }
        std::vector<std::pair<int64_t, int32_t>> v(n);
        for (int i = 0; i < n; ++i) v[i] = {off[i], len[i]};
        std::sort(v.begin(), v.end());
        for (int i = 0; i < n; ++i)
            if (i == 0 || v[i] != v[i - 1]) rows += v[i].second;
        return rows;
    };
    const int64_t b_rows = distinct_rows(b->b_row_off, b->cols);
    const int64_t c_rows = distinct_rows(b->c_row_off, b->rows);
    in_f = out_t = 4 * b_rows * F;
    in_t = out_f = 4 * c_rows * F;
    for (int i = 0; i < n; ++i) {
        csr_f += 4 * ((int64_t)b->rows[i] + 1) + 8 * (int64_t)b->nnz[i];
        csr_t += 4 * ((int64_t)b->cols[i] + 1) + 8 * (int64_t)b->nnz[i];
        nnz += b->nnz[i];
        for (int d = 0; d < 2; ++d) {
            p.lean_rows[d] = std::max(p.lean_rows[d], d ? b->rows[i] : b->cols[i]);
            p.lean_out_rows[d] = std::max(p.lean_out_rows[d], d ? b->cols[i] : b->rows[i]);
        }
        if (b->rows[i] > 0 && b->cols[i] > 0) p.reads_dense = true;
    }
    p.effective_bytes[0] = csr_f + in_f + out_f;
    p.effective_bytes[1] = csr_t + in_t + out_t;
    p.flops = 2 * nnz * F;

    make_stream_plan(p);
    largest_first(b->nnz, n, p.build_order);

    // workspace layout
    Layout& L = p.lay;
    auto lay_out = [&]() {
        size_t at = 0;
        auto place = [&at](size_t& where, size_t bytes) {
            where = at;
            at = align_up(at + bytes);
        };
        for (int d = 0; d < 2; ++d) place(L.items[d], p.sched[d].items.size() * sizeof(WorkItem));
        for (int d = 0; d < 2; ++d) place(L.lean[d], p.lean_items[d].size() * sizeof(LeanItem));
        if (p.lean_shared) L.lean[1] = L.lean[0];
        place(L.op_records, (size_t)n * sizeof(OpRecord));
        place(L.coo_records, p.coo_records.size() * sizeof(OpRecord));
        place(L.build_order, (size_t)n * sizeof(int32_t));
        for (int d = 0; d < 2; ++d) place(L.sets[d], p.set_records[d].size() * sizeof(SetRecord));
        place(L.stream_sets, p.stream.sets.size() * sizeof(LayerSet));
        place(L.stream_items, p.stream.items.size() * sizeof(LayerItem));
        place(L.stream_rest, p.stream.rest.size() * sizeof(WorkItem));
        L.image = at;
        place(L.rpt_t, (size_t)rpt_t_words * 4);
        place(L.colids_t, (size_t)nz_pack * 4);
        place(L.values_t, (size_t)nz_pack * 4);
        place(L.scratch, (size_t)scratch_words * 4);
        place(L.flag, 4);
        for (int d = 0; d < 2; ++d) place(L.merged[d], (size_t)p.merged_words[d] * 4);
        place(L.stream_arrays, (size_t)p.stream.words * 4);
        L.total = at;
    };
    lay_out();
    // (small layers need none of the layer kernel's arrays: they must not push a plan out of the static array)
    if (p.stream.on() && !p.stream.many && L.total > BSPMM_STATIC_WORKSPACE_BYTES) {
        p.stream = bspmm_plan::Stream();
        lay_out();
    }
    return BSPMM_OK;
}

// What the device says about itself does not change between plans: asked once per
// (device, LDS size, kernel variant) and thread.
struct DeviceFacts {
    int dev = -1, lds_bytes = 0;
    bool hubs = false;
    int cus = 0, resident = 0, resident_slices = 0;
};

const DeviceFacts& device_facts(int lds_bytes, bool hubs)
{
    thread_local DeviceFacts f;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        dev = -2;
    }
    if (f.dev != dev || f.lds_bytes != lds_bytes || f.hubs != hubs) {
        f = DeviceFacts();
        f.dev = dev;
        f.lds_bytes = lds_bytes;
        f.hubs = hubs;
        if (dev >= 0) {
            int cus = 0;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
                f.cus = cus;
            else
                (void)hipGetLastError();
            f.resident = bspmm_max_resident_workgroups(lds_bytes, false, hubs);
            f.resident_slices = bspmm_max_resident_workgroups(lds_bytes, true, hubs);
        }
    }
    return f;
}

Knobs knobs_for(const bspmm_options* o, bool ask_device)
{
    Knobs kn = resolve_knobs(o);
    kn.device_ok = ask_device;
    const bool cus_given = o && o->compute_units > 0;
    int r = 0, rs = 0;
    if (ask_device) {
        const DeviceFacts& f = device_facts(kn.lds_words * 4, kn.hubs);
        if (!cus_given && f.cus > 0) kn.compute_units = f.cus;
        r = f.resident;
        rs = f.resident_slices;
    }
    if (!(o && o->target_workgroups > 0)) kn.target_wgs = workgroups_per_cu(kn.front) * kn.compute_units;
    kn.capacity_wgs = r > 0 ? r : 6 * kn.compute_units;
    kn.capacity_wgs_slices = rs > 0 ? rs : 4 * kn.compute_units;
    return kn;
}

// Host planning with the LDS budget the caller gave.  When the caller left it open and the
// batch does not fit the default (operations summed into one block share a workgroup's LDS; an
// operation of the fused front shares it with its layer input), larger budgets are tried
// before the batch is refused: first asking for both directions, then for the forward product
// alone.
template <class Batch, class PlanFn>
int plan_with_budget(bspmm_plan& p, const Batch* b, int32_t F, const bspmm_options* options,
                     bool dry, PlanFn plan_fn)
{
    const bool open = !(options && options->lds_bytes > 0);
    const bool front = options && options->front_features > 0;   // its default is 80 KiB already
    Knobs kn = knobs_for(options, !dry);
    if (open && front && b->batch > 0) {
        // A fused-front launch of several rounds of workgroups: a workgroup goes through its
        // phases (descriptor, staging, matrix cores, gather, store) one after the other, so the
        // launch runs at the rate at which the workgroups of a CU overlap, and a smaller budget
        // (narrower tiles for the operations that need them, four to six workgroups per CU
        // instead of two) is faster.  Measured on MI355X, F = 128, molecule graphs: one channel,
        // 1024 graphs, n_X = 32 / 48 / 64 / 100 / 128: 15.3 -> 13.6, 20.1 -> 16.1, 20.5 -> 19.1,
        // 39.8 -> 28.5, 39.5 -> 32.3 us (384 graphs, n_X = 64: 11.6 -> 8.9 us); whole layers of
        // four channels, n_X = 32: 384 graphs 28.9 -> 21.9 us, 512 graphs 25.2 -> 20.8 us, 2048
        // graphs 76.8 -> 68.3 us.  Launches of one or two rounds (up to 256 graphs) do not change.
        int channels = 1;
        if (options->flags & BSPMM_ACCUMULATE) {
            channels = 0;
            for (int i = 0; i < b->batch; ++i) channels += b->c_row_off[i] == b->c_row_off[0] ? 1 : 0;
        }
        if (b->batch / std::max(1, channels) >= kn.compute_units + kn.compute_units / 2) {
            const int first = channels > 1 ? 52 * 1024 : (options->front_features < 64 ? 24 * 1024 : 40 * 1024);
            const int second = first == 24 * 1024 ? 40 * 1024 : 0;
            for (int bytes : {first, second}) {
                if (bytes == 0) break;
                bspmm_options o = *options;
                o.lds_bytes = bytes;
                Knobs small = knobs_for(&o, !dry);
                small.need_both = false;
                small.lds_given = false;      // (the library's choice, not the caller's)
                p = bspmm_plan();
                const int rc = plan_fn(p, b, F, small);
                if (rc != BSPMM_ETOOBIG) return rc;
            }
            p = bspmm_plan();
        }
    }
    kn.need_both = open && !front;
    int rc = plan_fn(p, b, F, kn);
    if (rc == BSPMM_OK && open && !front && !p.coo_direct && F >= 512 && p.effective_bytes[0] > 28000000 &&
        p.effective_bytes[0] < 70000000 && !p.sched[0].row_blocks &&
        p.sched[0].uncut_wgs > kn.capacity_wgs) {
        // Wide feature matrices moved by a launch of more than one round of workgroups, which
        // runs at the rate of the memory system: with 24 KiB the larger operations get tiles of
        // 32 columns (row segments of 128 bytes), each staging the operation's CSR again.  A
        // budget of a third of a CU's LDS doubles the tiles; it is kept when the launch then
        // takes at most a tenth more rounds than before, since three workgroups per CU are resident
        // instead of six (measured, 128 graphs of 20-100 nodes: F = 1024, six seeds, 1.35-1.45
        // rounds before and 1.39-1.47 after, 14.3-15.2 -> 13.4-14.4 us, 4.24-4.34 -> 4.49-4.56 TB/s;
        // F = 512, 0.71 -> 1.33 rounds, 7.46 -> 8.79 us: not taken; 1024 graphs of 25 nodes at
        // F = 512, 2.19 -> 2.82 rounds, 21.0 -> 21.3 us: not taken).  Beyond 70 MB, and where some
        // operations are row blocks, the row ranges of the first plan are ahead (300 graphs of 20-100
        // nodes at F = 512 15.8 -> 14.0 us, 200 at F = 1024 20.3 -> 17.7; 80 random matrices at
        // F = 512 10.1 -> 8.7).
        bspmm_options o = options ? *options : bspmm_options{};
        o.lds_bytes = 53248;
        Knobs wide = knobs_for(&o, !dry);
        if (dry) wide.capacity_wgs = 3 * wide.compute_units;
        wide.need_both = kn.need_both;
        wide.lds_given = false;
        bspmm_plan q;
        if (plan_fn(q, b, F, wide) == BSPMM_OK &&
            10 * (int64_t)q.sched[0].grid * kn.capacity_wgs <= 11 * (int64_t)p.sched[0].uncut_wgs * wide.capacity_wgs)
            p = std::move(q);
        return BSPMM_OK;
    }
    if (rc != BSPMM_ETOOBIG || !open) return rc;
    static const struct { int bytes; bool both; } attempts[] = {
        {kHalfLdsBytes, true}, {kMaxLdsBytes, true}, {0, false}, {kHalfLdsBytes, false}, {kMaxLdsBytes, false}};
    for (const auto& a : attempts) {
        if (front && !(a.bytes == kMaxLdsBytes && !a.both)) continue;
        bspmm_options o = options ? *options : bspmm_options{};
        o.lds_bytes = a.bytes;
        kn = knobs_for(&o, !dry);
        kn.need_both = a.both;
        kn.lds_given = false;
        p = bspmm_plan();
        rc = plan_fn(p, b, F, kn);
        if (rc != BSPMM_ETOOBIG) return rc;
    }
    return rc;
}

// A one-off build recorded into a stream capture runs when the graph is replayed, not now: the
// plan must not count it as done (a later eager run builds again; the graph keeps its copy).
bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusActive;
}

// Before work on `s` that reads the plan's tables: a plan may be used on another stream than it was
// made on without the caller ordering the two, as when the tables went over in blocking copies.
// (hipStreamPerThread is one handle for the streams of all threads)
int settle(bspmm_plan* p, hipStream_t s)
{
    return s != p->upload_stream || s == hipStreamPerThread ? settle_upload(p) : BSPMM_OK;
}

int enqueue_build(bspmm_plan* p, hipStream_t s)
{
    if (p->transposed_built || p->knobs.symmetric) return BSPMM_OK;
    hipError_t e = launch_build_transpose(
        reinterpret_cast<const OpRecord*>(p->ws + p->lay.op_records), p->batch,
        p->build_threads, p->build_lds_bytes, p->rpt, p->colids, p->values,
        reinterpret_cast<int32_t*>(p->ws + p->lay.rpt_t),
        reinterpret_cast<int32_t*>(p->ws + p->lay.colids_t),
        reinterpret_cast<float*>(p->ws + p->lay.values_t),
        reinterpret_cast<int32_t*>(p->ws + p->lay.scratch),
        reinterpret_cast<const int32_t*>(p->ws + p->lay.build_order), s);
    if (e != hipSuccess) return hip_fail(e);
    p->transposed_built = !capturing(s);
    return BSPMM_OK;
}

// The merged CSR of the summed sets of direction d (once per plan; for d = 1 after the
// transposed CSR has been built).
int enqueue_merge(bspmm_plan* p, int d, hipStream_t s)
{
    if (p->merged_built[d] || p->set_records[d].empty()) return BSPMM_OK;
    const bool own = d == 0 || p->knobs.symmetric;
    const int32_t* rpt = own ? p->rpt : reinterpret_cast<const int32_t*>(p->ws + p->lay.rpt_t);
    const int32_t* colids = own ? p->colids : reinterpret_cast<const int32_t*>(p->ws + p->lay.colids_t);
    const float* values = own ? p->values : reinterpret_cast<const float*>(p->ws + p->lay.values_t);
    hipError_t e = launch_merge_sets(reinterpret_cast<const SetRecord*>(p->ws + p->lay.sets[d]),
                                     (int)p->set_records[d].size(), rpt, colids, values,
                                     reinterpret_cast<int32_t*>(p->ws + p->lay.merged[d]), s);
    if (e != hipSuccess) return hip_fail(e);
    p->merged_built[d] = !capturing(s);
    return BSPMM_OK;
}

// CSR arrays a run of direction d reads.
void csr_of_direction(const bspmm_plan* p, int d, const int32_t** rpt, const int32_t** colids,
                      const float** values)
{
    if (d == 0 || p->knobs.symmetric) {
        *rpt = p->rpt;
        *colids = p->colids;
        *values = p->values;
    } else {
        *rpt = reinterpret_cast<const int32_t*>(p->ws + p->lay.rpt_t);
        *colids = reinterpret_cast<const int32_t*>(p->ws + p->lay.colids_t);
        *values = reinterpret_cast<const float*>(p->ws + p->lay.values_t);
    }
}

// The arrays that the blocks of a layer read (once per plan).
int enqueue_layer_rows(bspmm_plan* p, hipStream_t s)
{
    bspmm_plan::Stream& st = p->stream;
    if (st.built || !st.on() || !st.items.empty()) return BSPMM_OK;
    int32_t* base = reinterpret_cast<int32_t*>(p->ws + p->lay.stream_arrays);
    const int count = (int)(st.sets.size() / st.parts.size());
    for (const bspmm_plan::Stream::Part& part : st.parts) {
        hipError_t e = launch_layer_rows(reinterpret_cast<const LayerSet*>(p->ws + p->lay.stream_sets) + part.sets_at,
                                         count, reinterpret_cast<const OpRecord*>(p->ws + p->lay.op_records), p->rpt,
                                         p->colids, p->values, base + part.starts_at, base + part.entries_at,
                                         base + st.out_rows_at, s);
        if (e != hipSuccess) return hip_fail(e);
    }
    st.built = !capturing(s);
    return BSPMM_OK;
}

// The entry ranges of row blocks ahead of the first run, which finds them itself otherwise (for d = 1 after the
// transposed CSR is built).
int enqueue_ranges(bspmm_plan* p, int d, hipStream_t s)
{
    if (p->lean_ranges[d] || !p->lean_blocks[d] || p->lean_items[d].empty()) return BSPMM_OK;
    const int32_t* rpt;
    const int32_t* colids;
    const float* values;
    csr_of_direction(p, d, &rpt, &colids, &values);
    const hipError_t e = launch_lean_hints(reinterpret_cast<LeanItem*>(p->ws + p->lay.lean[d]),
                                           (int)p->lean_items[d].size(), rpt, s);
    if (e != hipSuccess) return hip_fail(e);
    p->lean_ranges[d] = !capturing(s);
    return BSPMM_OK;
}

// Rows of both operands are whole float4 on 16 bytes.
bool on_quads(const bspmm_plan* p, const float* in, const float* out, int64_t ld_in, int64_t ld_out)
{
    return p->F % 4 == 0 && ld_in % 4 == 0 && ld_out % 4 == 0 &&
           ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
}

// The transposed product and the transposed arrays in one launch (the arguments have been checked).
int first_transposed(bspmm_plan* p, const float* in, float* out, int64_t ld_in, int64_t ld_out, hipStream_t s)
{
    LaunchParams P = {};
    P.rpt = p->rpt, P.colids = p->colids, P.values = p->values;
    P.in = in, P.out = out, P.ld_in = ld_in, P.ld_out = ld_out;
    const hipError_t e = launch_first_transposed(
        reinterpret_cast<const LeanItem*>(p->ws + p->lay.lean[1]), P, (int)p->lean_items[0].size(),
        p->sched[1].lds_words * 4, reinterpret_cast<int32_t*>(p->ws + p->lay.rpt_t),
        reinterpret_cast<int32_t*>(p->ws + p->lay.colids_t), reinterpret_cast<float*>(p->ws + p->lay.values_t), s);
    if (e != hipSuccess) return hip_fail(e);
    p->transposed_built = !capturing(s);
    return BSPMM_OK;
}

int run_direction(bspmm_plan* p, int d, const float* in, float* out, int64_t ld_in,
                  int64_t ld_out, hipStream_t s)
{
    if (p->coo_direct) {
        const CooSchedule& cs = p->coo_sched[d];
        if (cs.items.empty()) return BSPMM_OK;
        if ((!in && p->reads_dense) || !out || ld_in < p->F || ld_out < p->F) return BSPMM_EINVAL;
        CooLaunchParams C;
        C.items = reinterpret_cast<const CooItem*>(p->ws + p->lay.items[d]);
        C.ids = p->ids;
        C.values = p->coo_values;
        C.in = in;
        C.out = out;
        C.ld_in = ld_in;
        C.ld_out = ld_out;
        C.transposed = d;
        hipError_t ce = launch_bspmm_coo(C, (int)cs.items.size(), cs.lds_words * 4, on_quads(p, in, out, ld_in, ld_out), s);
        return ce == hipSuccess ? BSPMM_OK : hip_fail(ce);
    }
    const Schedule& sc = p->sched[d];
    if (sc.grid == 0) return BSPMM_OK;
    // when no operation has both rows and columns nothing is read: the input may have no rows at all
    if ((!in && p->reads_dense) || !out || ld_in < p->F || ld_out < p->F) return BSPMM_EINVAL;
    const int mrc = enqueue_merge(p, d, s);
    if (mrc != BSPMM_OK) return mrc;
    LaunchParams P;
    P.items = reinterpret_cast<const WorkItem*>(p->ws + p->lay.items[d]);
    csr_of_direction(p, d, &P.rpt, &P.colids, &P.values);
    P.in = in;
    P.out = out;
    P.ld_in = ld_in;
    P.ld_out = ld_out;
    for (int r = 0; r < kRanges; ++r) {
        P.wg_end[r] = sc.wg_end[r];
        P.item_base[r] = sc.item_base[r];
    }
    P.n_tasks = sc.grid;
    P.fused_stride = sc.fused_stride;
    P.lds_floats = sc.budget_words;
    P.pad = p->knobs.pad;
    P.w = reinterpret_cast<const float*>(p->ws + p->lay.merged[d]);   // see LaunchParams
    P.bias = nullptr;
    P.ld_w = 0;
    P.n_front = 0;
    P.accumulate = 0;
    const bool vec4 = on_quads(p, in, out, ld_in, ld_out);
    if (!sc.whole) {
        const hipError_t e = launch_bspmm(P, sc.launch_grid, sc.budget_words * 4, vec4, sc.has_slices,
                                          p->knobs.hubs, !sc.merged_sets.empty(), s);
        return e == hipSuccess ? BSPMM_OK : hip_fail(e);
    }
    const LeanItem* items = reinterpret_cast<const LeanItem*>(p->ws + p->lay.lean[d]);
    const bool first = p->lean_blocks[d] && !p->lean_ranges[d];
    hipError_t e;
    if (vec4 && takes_lean_kernel(p, d, ld_in, ld_out)) {
        e = launch_bspmm_lean(items, P, sc.launch_grid, sc.lds_words * 4, !sc.merged_sets.empty(), first, s);
    } else {
        // (the table's packed items follow the launch's own: here each is a workgroup)
        const int grid = (int)p->lean_items[p->lean_shared ? 0 : d].size();
        e = launch_bspmm_any(items, P, vec4, p->F % 4 == 0, first, grid, sc.lds_words * 4, s);
    }
    if (e == hipSuccess && first) p->lean_ranges[d] = !capturing(s);
    return e == hipSuccess ? BSPMM_OK : hip_fail(e);
}

int check_coo_batch(const bspmm_coo_batch* b, int32_t F, bool need_device)
{
    if (!b || F <= 0 || b->batch < 0) return BSPMM_EINVAL;
    if (b->batch == 0) return BSPMM_OK;
    if (!b->rows || !b->cols || !b->nnz || !b->nz_off || !b->b_row_off || !b->c_row_off)
        return BSPMM_EINVAL;
    int64_t total_nnz = 0;
    for (int i = 0; i < b->batch; ++i) {
        if (b->rows[i] < 0 || b->cols[i] < 0 || b->nnz[i] < 0) return BSPMM_EINVAL;
        if (b->nz_off[i] < 0 || b->b_row_off[i] < 0 || b->c_row_off[i] < 0) return BSPMM_EINVAL;
        if ((b->rows[i] == 0 || b->cols[i] == 0) && b->nnz[i] != 0) return BSPMM_EINVAL;
        total_nnz += b->nnz[i];
    }
    if (need_device && total_nnz > 0 && (!b->ids || !b->values)) return BSPMM_EINVAL;
    return BSPMM_OK;
}

// Plan of the direct COO kernel: two item tables (forward, transposed), the validation
// records and the flag word; no CSR, no build.
int plan_host_coo_direct(bspmm_plan& p, const bspmm_coo_batch* b, int32_t F, const Knobs& kn)
{
    const int n = b->batch;
    if (kn.accumulate || kn.hubs) return BSPMM_EINVAL;
    p.batch = n;
    p.F = F;
    p.knobs = kn;
    p.from_coo = true;
    p.coo_direct = true;
    DirOps& f = p.dir[0];
    DirOps& t = p.dir[1];
    int64_t nnz = 0, in_f = 0, out_f = 0;
    std::set<std::pair<int64_t, int32_t>> blocks_b;
    for (DirOps* o : {&f, &t}) {
        o->m.reserve(n), o->k.reserve(n), o->nnz.reserve(n), o->rpt_off.reserve(n);
        o->nz_off.reserve(n), o->in_off.reserve(n), o->out_off.reserve(n);
    }
    for (int i = 0; i < n; ++i) {
        if (kn.symmetric && b->rows[i] != b->cols[i]) return BSPMM_EINVAL;
        f.m.push_back(b->rows[i]);
        f.k.push_back(b->cols[i]);
        t.m.push_back(b->cols[i]);
        t.k.push_back(b->rows[i]);
        for (DirOps* d : {&f, &t}) {
            d->nnz.push_back(b->nnz[i]);
            d->rpt_off.push_back(0);
            d->nz_off.push_back(b->nz_off[i]);
        }
        f.in_off.push_back(b->b_row_off[i]);
        f.out_off.push_back(b->c_row_off[i]);
        t.in_off.push_back(b->c_row_off[i]);
        t.out_off.push_back(b->b_row_off[i]);
        nnz += b->nnz[i];
        if (b->rows[i] > 0 && b->cols[i] > 0) p.reads_dense = true;
        if (blocks_b.emplace(b->b_row_off[i], b->cols[i]).second) in_f += 4 * (int64_t)b->cols[i] * F;
        out_f += 4 * (int64_t)b->rows[i] * F;
    }
    if (n > 0 && overlap_kind(b->c_row_off, b->rows, n) != 0) return BSPMM_EOVERLAP;
    p.transposed_supported = n == 0 || overlap_kind(b->b_row_off, b->cols, n) == 0;
    p.coo_sched[0] = make_coo_schedule(f, F, kn);
    if (p.transposed_supported) p.coo_sched[1] = make_coo_schedule(t, F, kn);
    // compulsory traffic: every entry once (two indices and a value), distinct dense inputs
    // once, outputs once
    p.effective_bytes[0] = 12 * nnz + in_f + out_f;
    p.effective_bytes[1] = 12 * nnz + out_f + in_f;
    p.flops = 2 * nnz * F;
    Layout& L = p.lay;
    size_t at = 0;
    for (int d = 0; d < 2; ++d) {
        L.items[d] = at;
        at = align_up(at + p.coo_sched[d].items.size() * sizeof(CooItem));
    }
    L.coo_records = at;
    at = align_up(at + (size_t)n * sizeof(OpRecord));
    L.image = at;
    L.flag = at;
    at = align_up(at + 4);
    L.total = at;
    return BSPMM_OK;
}

// Plan for COO operands: the CSR arrays (row pointers and entries packed back to back in
// operation order) are built inside the workspace, and everything else is the CSR plan of them.
int plan_host_coo(bspmm_plan& p, const bspmm_coo_batch* b, int32_t F, const Knobs& kn)
{
    const int n = b->batch;
    std::vector<int64_t> rpt_off(n), nz_pack(n);
    int64_t rpt_words = 0, nz = 0, scratch_words = 0, lds_words = 0;
    p.coo_records.resize(n);
    int threads = kThreads;
    for (int i = 0; i < n; ++i)
        if (b->nnz[i] > 4 * kThreads) threads = kBuildThreadsLarge;
    for (int i = 0; i < n; ++i) {
        rpt_off[i] = rpt_words;
        nz_pack[i] = nz;
        OpRecord& r = p.coo_records[i];
        r.rpt_off = 0;
        r.nz_off = b->nz_off[i];          // where the caller's pairs and values sit
        r.rpt_t_off = rpt_words;          // where the built row pointers go
        r.nz_t_off = nz;                  // where the built entries go
        r.m = b->cols[i];                 // bound of the payload (column)
        r.k = b->rows[i];                 // number of keys (rows)
        r.nnz = b->nnz[i];
        lds_words = std::max(lds_words, classify_build(r, b->rows[i], b->cols[i], b->nnz[i], false,
                                                       threads, &scratch_words));
        rpt_words += (int64_t)b->rows[i] + 1;
        nz += b->nnz[i];
    }
    if (kn.coo_direct) return plan_host_coo_direct(p, b, F, kn);
    bspmm_batch ib;
    ib.batch = n;
    ib.rows = b->rows;
    ib.cols = b->cols;
    ib.nnz = b->nnz;
    ib.rpt_off = rpt_off.data();
    ib.nz_off = nz_pack.data();
    ib.b_row_off = b->b_row_off;
    ib.c_row_off = b->c_row_off;
    ib.rpt = nullptr;
    ib.colids = nullptr;
    ib.values = nullptr;
    const int rc = plan_host(p, &ib, F, kn);
    if (rc != BSPMM_OK) return rc;
    p.from_coo = true;
    p.coo_build_lds_bytes = (int)round_up(lds_words * 4 + 16, 256);
    p.csr_rpt_words = rpt_words;
    p.csr_nz = nz;
    p.coo_scratch_words = scratch_words;
    Layout& L = p.lay;
    size_t at = L.total;
    L.csr_rpt = at;
    at = align_up(at + (size_t)rpt_words * 4);
    L.csr_colids = at;
    at = align_up(at + (size_t)nz * 4);
    L.csr_values = at;
    at = align_up(at + (size_t)nz * 4);
    L.coo_scratch = at;
    at = align_up(at + (size_t)scratch_words * 4);
    L.total = at;
    return BSPMM_OK;
}

// The tables the host writes, as they lie at the front of the workspace.
void write_image(const bspmm_plan* p, char* to)
{
    auto put = [to](size_t where, const auto& v) {
        if (!v.empty()) std::memcpy(to + where, v.data(), v.size() * sizeof(v[0]));
    };
    const Layout& L = p->lay;
    for (int d = 0; d < 2; ++d) {
        if (p->coo_direct)
            put(L.items[d], p->coo_sched[d].items);
        else
            put(L.items[d], p->sched[d].items);
        put(L.lean[d], p->lean_items[d]);
        put(L.sets[d], p->set_records[d]);
    }
    put(L.op_records, p->records);
    put(L.coo_records, p->coo_records);
    put(L.build_order, p->build_order);
    put(L.stream_sets, p->stream.sets);
    put(L.stream_items, p->stream.items);
    put(L.stream_rest, p->stream.rest);
}

// Device half of plan creation: tables to the workspace, conversions enqueued on `s`.  `front`: host
// arrays that go to the memory right in front of the workspace in the same copy; `pinned`: staging
// memory may be taken for the copy.
int upload_plan(bspmm_plan* p, const bspmm_options* options, void* workspace,
                size_t workspace_bytes, hipStream_t s, const HostFront* front = nullptr, bool pinned = true)
{
    // The one-launch layer kernel's workgroup size, decided here (plans made by
    // bspmm_workspace_bytes never asked the device) and not in the first run, which may be
    // inside a stream capture.  A launch of up to two workgroups per CU lasts as long as its
    // largest item, and workgroups of eight wavefronts halve that item's matrix blocks per
    // wavefront and the passes of its gather.  Measured on 256 CUs, F = 128, four against eight
    // wavefronts: one channel at n_X = 64, 32 graphs (320 workgroups) 6.4 -> 5.1 us; n_X = 128,
    // 128 graphs (312) 9.3 -> 8.7; four channels at n_X = 64, 64 graphs (512) 9.3 -> 7.9, 32
    // graphs 7.1 -> 6.2.  Beyond two per CU the launch of twice the wavefronts costs more than it
    // gains (128 graphs at n_X = 64, 544 workgroups: 6.6 -> 6.9 us; four channels, 1024
    // workgroups: 11.9 -> 12.3).
    p->front_wide = 0;
    if (p->knobs.front > 0) {
        const Schedule& sc = p->sched[0];
        const int64_t grid = p->stream.on() ? (int64_t)p->stream.rest.size() : sc.grid;
        const int per_cu = std::min(2, front_workgroups_per_cu(!sc.merged_sets.empty(), true, sc.front_lds_words * 4));
        p->front_wide = grid > 0 && grid <= (int64_t)per_cu * p->knobs.compute_units ? 1 : 0;
    }
    if (options && (options->flags & BSPMM_FLOOR_PROBE)) {
        p->sorts_in_run = false;                           // (emptied items write no arrays)
        for (int d = 0; d < 2; ++d) {
            for (WorkItem& w : p->sched[d].items) w.nrows = w.m = w.k = w.nnz = 0;
            for (LeanItem& w : p->lean_items[d])
                w.nrows = w.m = w.k = w.nnz = w.tile_vecs = w.count = w.flags = w.b_byte = 0;
            for (CooItem& w : p->coo_sched[d].items) w.nrows = w.nnz = 0;
        }
    }
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0)
        return BSPMM_EINVAL;
    if (workspace_bytes < p->lay.total) return BSPMM_ENOSPACE;
    p->ws = static_cast<char*>(workspace);
    // One copy brings the image of the tables, and in front of it the caller's arrays where they come
    // from host memory.  From pinned memory, except in a stream capture (the copy then belongs to a
    // graph and reads the plan's own memory on every replay) and for very large plans.
    hipError_t e = hipSuccess;
    const size_t head = front ? front->bytes : 0;
    char* dst = p->ws - head;
    StageBlock stage;
    if (pinned && head + p->lay.image > 0 && !capturing(s)) stage = stage_take(head + p->lay.image);
    if (front && !stage.ptr) return BSPMM_ESTATE;      // (the caller copies the arrays itself)
    if (stage.ptr) {
        if (front) front->write(front->from, stage.ptr);
        write_image(p, stage.ptr + head);
        p->upload_stream = s;
        e = stage_copy(stage, dst, head + p->lay.image, s, &p->upload);
    } else if (p->lay.image > 0) {
        p->tables.resize(p->lay.image);
        write_image(p, p->tables.data());
        e = hipMemcpyAsync(p->ws, p->tables.data(), p->tables.size(), hipMemcpyHostToDevice, s);
        p->upload_stream = s;
        if (e == hipSuccess && !capturing(s)) {
            e = hipEventCreateWithFlags(&p->copied, hipEventDisableTiming);
            if (e == hipSuccess) e = hipEventRecord(p->copied, s);
        }
    }
    if (p->coo_direct) return e == hipSuccess ? BSPMM_OK : hip_fail(e);
    if (e == hipSuccess && p->from_coo) {
        int32_t* rpt = reinterpret_cast<int32_t*>(p->ws + p->lay.csr_rpt);
        int32_t* colids = reinterpret_cast<int32_t*>(p->ws + p->lay.csr_colids);
        float* values = reinterpret_cast<float*>(p->ws + p->lay.csr_values);
        p->rpt = rpt;
        p->colids = colids;
        p->values = values;
        if (!p->coo_records.empty())
            e = launch_build_from_coo(
                reinterpret_cast<const OpRecord*>(p->ws + p->lay.coo_records), p->batch,
                p->build_threads, p->coo_build_lds_bytes, p->ids, p->coo_values, rpt, colids, values,
                reinterpret_cast<int32_t*>(p->ws + p->lay.coo_scratch),
                reinterpret_cast<const int32_t*>(p->ws + p->lay.build_order), s);
    }
    if (e != hipSuccess) return hip_fail(e);
    if (options && (options->flags & BSPMM_BUILD_TRANSPOSE)) {
        int rc = enqueue_merge(p, 0, s);
        if (rc == BSPMM_OK) rc = enqueue_layer_rows(p, s);
        if (rc == BSPMM_OK && p->transposed_supported) rc = enqueue_build(p, s);
        if (rc == BSPMM_OK && p->transposed_supported) rc = enqueue_merge(p, 1, s);
        if (rc == BSPMM_OK) rc = enqueue_ranges(p, 0, s);
        if (rc == BSPMM_OK && p->transposed_supported) rc = enqueue_ranges(p, 1, s);
        return rc;
    }
    return BSPMM_OK;
}

// One channel of the graph-convolution layer: the forward schedule with the dense tile made
// on chip from X_i, W and bias.
int run_gcn(bspmm_plan* p, const float* X, int64_t ldx, const float* W, int64_t ldw,
            const float* bias, float* Y, int64_t ldy, int accumulate, hipStream_t s)
{
    const Schedule& sc = p->sched[0];
    if (sc.grid == 0) return BSPMM_OK;
    const int nx = p->knobs.front;
    auto misaligned = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) != 0; };
    if (!X || !W || !bias || !Y || ldx < nx || ldw < p->F || ldy < p->F) return BSPMM_EINVAL;
    if (ldx % 4 || ldw % 4 || ldy % 4 || misaligned(X) || misaligned(W) || misaligned(Y))
        return BSPMM_EINVAL;
    const bool sets = !sc.merged_sets.empty();
    // (32-bit offsets inside W, 32-bit leading dimensions of X and Y)
    if (p->stream.on() && p->stream.many && (ldx >= (int64_t(1) << 31) || ldy >= (int64_t(1) << 31))) return BSPMM_EINVAL;
    const bool layer = p->stream.on() && ldx < (int64_t(1) << 31) && ldy < (int64_t(1) << 31) && ldw < (int64_t(1) << 20);
    if (layer) {
        const int mrc = enqueue_layer_rows(p, s);
        if (mrc != BSPMM_OK) return mrc;
    }
    if (sets && (!layer || !p->stream.rest.empty())) {
        const int mrc = enqueue_merge(p, 0, s);
        if (mrc != BSPMM_OK) return mrc;
    }
    const bspmm_plan::Stream& st = p->stream;
    if (layer) {
        // the graphs cut into blocks; the others (if any) follow in a launch of the one-launch kernel over
        // their items
        const int32_t* base = reinterpret_cast<const int32_t*>(p->ws + p->lay.stream_arrays);
        for (const bspmm_plan::Stream::Part& part : st.parts) {
            LayerParams S;
            S.starts = base + part.starts_at;
            S.entries = base + part.entries_at;
            S.out_rows = base + st.out_rows_at;
            S.x = X;
            S.w = W + (int64_t)part.first_channel * nx * ldw;
            S.bias = bias + (int64_t)part.first_channel * p->F;
            S.y = Y;
            S.direct = {reinterpret_cast<const LayerItem*>(p->ws + p->lay.stream_items), p->rpt, p->colids, p->values};
            LayerShape& sh = S.shape;
            sh.ld_x = ldx, sh.ld_w = ldw, sh.ld_y = ldy, sh.bias_stride = p->F;
            sh.blocks = st.blocks, sh.ranges_per_xcd = part.ranges_per_xcd, sh.tiles = st.tiles;
            const int ranges = 8 * part.ranges_per_xcd;
            sh.blocks_each = st.blocks / ranges, sh.blocks_over = st.blocks % ranges;
            sh.inv_tiles = st.tiles > 1 ? (uint32_t)(((uint64_t(1) << 32) + st.tiles - 1) / st.tiles) : 0;
            sh.F = p->F;
            sh.channels = part.channels;
            sh.inv_channels = (65535 + part.channels) / part.channels;
            sh.lane_shift = nx == 16 ? 2 : (nx == 32 ? 3 : (nx == 64 ? 4 : 5));
            sh.slots = part.slots;
            sh.entries = st.direct_entries;
            sh.accumulate = accumulate || part.first_channel > 0 ? 1 : 0;
            const hipError_t es = launch_bspmm_layer(S, part.ks, st.units, st.items.empty() ? st.rb : 0, st.waves, part.lds_bytes, s);
            if (es != hipSuccess) return hip_fail(es);
        }
        if (st.rest.empty()) return BSPMM_OK;
    }
    LaunchParams P;
    P.items = layer ? reinterpret_cast<const WorkItem*>(p->ws + p->lay.stream_rest)
                    : reinterpret_cast<const WorkItem*>(p->ws + p->lay.items[0]);
    // (channel sets: every item reads the merged CSR of its set; P.rpt carries its base)
    P.rpt = sets ? reinterpret_cast<const int32_t*>(p->ws + p->lay.merged[0]) : p->rpt;
    P.colids = p->colids;
    P.values = p->values;
    P.in = X;
    P.out = Y;
    P.ld_in = ldx;
    P.ld_out = ldy;
    for (int r = 0; r < kRanges; ++r) {
        P.wg_end[r] = sc.wg_end[r];
        P.item_base[r] = sc.item_base[r];
    }
    P.n_tasks = sc.grid;
    P.fused_stride = p->F;                 // this launch: floats between the channels' bias rows
    P.lds_floats = sc.front_lds_words;     // what the launch gets: decides the rows of X_i per pass
    P.pad = 0;
    P.w = W;
    P.bias = bias;
    P.ld_w = ldw;
    P.n_front = nx;
    P.accumulate = accumulate ? 1 : 0;
    const int grid = layer ? (int)st.rest.size() : sc.grid;
    hipError_t e = launch_bspmm_gcn(P, grid, sc.front_lds_words * 4, accumulate != 0, sets, p->front_wide == 1, s);
    return e == hipSuccess ? BSPMM_OK : hip_fail(e);
}

// The static workspace of the current device.  Its device address is asked for once per device
// (with that device current) and kept; every later use goes through the kept pointer.  The
// generation counts the plans handed out on a device: only the latest owns the array.
constexpr int kMaxDevices = 64;
std::mutex g_static_mutex;
void* g_static_ptr[kMaxDevices] = {};
std::atomic<uint64_t> g_static_generation[kMaxDevices];

int static_workspace(int* device, void** ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxDevices) return BSPMM_EINVAL;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        void* q = nullptr;
        e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e);
        if (!q || (reinterpret_cast<uintptr_t>(q) & (kAlign - 1)) != 0) return BSPMM_EINVAL;
        g_static_ptr[dev] = q;
    }
    *device = dev;
    *ptr = g_static_ptr[dev];
    return BSPMM_OK;
}

// A plan made by bspmm_create_static that a later one on the same device has displaced must
// not run: the tables it points at are no longer its own.
bool displaced(const bspmm_plan* p)
{
    return p->static_device >= 0 &&
           g_static_generation[p->static_device].load(std::memory_order_acquire) != p->static_generation;
}

// bspmm_workspace_bytes has to schedule the batch to know the size; a bspmm_create that follows
// on the same thread with the same arguments takes that plan over instead of scheduling again.
// "The same" is checked on the values themselves: F, the options, and every host array of the
// batch against what the remembered plan was made from.
struct PlanKey {
    int32_t batch = -1, F = 0;
    bool coo = false, has_options = false;
    bspmm_options options;
};

thread_local std::unique_ptr<bspmm_plan> t_memo;
thread_local PlanKey t_memo_key;

PlanKey make_key(int32_t batch, int32_t F, const bspmm_options* o, bool coo)
{
    PlanKey k;
    k.batch = batch;
    k.F = F;
    k.coo = coo;
    k.has_options = o != nullptr;
    std::memset(&k.options, 0, sizeof(k.options));
    if (o) k.options = *o;
    return k;
}

void remember(bspmm_plan* p, const PlanKey& k)
{
    t_memo.reset(p);
    t_memo_key = k;
}

// The remembered plan, if it was made from exactly this batch.  `rpt_off` is null for COO batches
// (their plans keep the row-pointer offsets the library chose itself).
template <class Batch>
bspmm_plan* recall(const PlanKey& k, const Batch* b, const int64_t* rpt_off)
{
    if (!t_memo) return nullptr;
    const PlanKey& m = t_memo_key;
    if (m.batch != k.batch || m.F != k.F || m.coo != k.coo || m.has_options != k.has_options ||
        std::memcmp(&m.options, &k.options, sizeof(k.options)) != 0)
        return nullptr;
    const bspmm_plan& p = *t_memo;
    const DirOps& f = p.dir[0];
    const size_t n = (size_t)k.batch;
    if (p.batch != k.batch || f.m.size() != n) return nullptr;
    auto same = [n](const auto& kept, const auto* given) {
        return std::memcmp(kept.data(), given, n * sizeof(*given)) == 0;
    };
    if (!same(f.m, b->rows) || !same(f.k, b->cols) || !same(f.nnz, b->nnz) ||
        !same(f.in_off, b->b_row_off) || !same(f.out_off, b->c_row_off))
        return nullptr;
    if (rpt_off) {
        if (!same(f.rpt_off, rpt_off) || !same(f.nz_off, b->nz_off)) return nullptr;
    } else {
        for (size_t i = 0; i < n; ++i)
            if (p.coo_records[i].nz_off != b->nz_off[i]) return nullptr;
    }
    return t_memo.release();
}

// The end of every create call: the plan to the caller, or nothing.
int hand_over(bspmm_plan* p, int rc, bspmm_plan** plan)
{
    if (rc != BSPMM_OK) {
        if (p->copied) (void)hipEventDestroy(p->copied);
        delete p;
        return rc;
    }
    if (!p->dry) {
        p->counted = true;
        stage_plan_made();
    }
    *plan = p;
    return BSPMM_OK;
}

int create_csr(bspmm_plan** plan, const bspmm_batch* b, int32_t F, const bspmm_options* options, void* workspace,
               size_t workspace_bytes, const HostFront* front, hipStream_t stream)
{
    if (!plan) return BSPMM_EINVAL;
    *plan = nullptr;
    const bool dry = options && (options->flags & BSPMM_DRY_RUN);
    int rc = check_batch(b, F, !dry);
    if (rc != BSPMM_OK) return rc;
    bspmm_plan* p = b->batch > 0 ? recall(make_key(b->batch, F, options, false), b, b->rpt_off) : nullptr;
    if (!p) {
        p = new (std::nothrow) bspmm_plan;
        if (!p) return BSPMM_EINVAL;
        rc = plan_with_budget(*p, b, F, options, dry, plan_host);
    }
    p->dry = dry;
    if (rc == BSPMM_OK && !dry) {
        p->rpt = b->rpt;
        p->colids = b->colids;
        p->values = b->values;
        rc = upload_plan(p, options, workspace, workspace_bytes, stream, front);
    }
    return hand_over(p, rc, plan);
}

}  // namespace

namespace bspmm {

int create_from_host(bspmm_plan** plan, const bspmm_batch* b, int32_t F, const bspmm_options* options,
                     void* workspace, size_t workspace_bytes, const HostFront& front, void* stream)
{
    return create_csr(plan, b, F, options, workspace, workspace_bytes, &front, static_cast<hipStream_t>(stream));
}

int settle_upload(bspmm_plan* plan)
{
    if (plan->copied) {
        const hipError_t e = event_wait(plan->copied);
        if (e != hipSuccess) return hip_fail(e);
        (void)hipEventDestroy(plan->copied);
        plan->copied = nullptr;
    }
    if (!plan->upload.slot) return BSPMM_OK;
    const hipError_t e = stage_wait(plan->upload, plan->upload_stream);
    if (e != hipSuccess) return hip_fail(e);
    plan->upload.slot = nullptr;
    return BSPMM_OK;
}

int run_after(void* stream, void* earlier)
{
    const hipStream_t s = static_cast<hipStream_t>(stream), first = static_cast<hipStream_t>(earlier);
    if (capturing(s) || capturing(first)) return BSPMM_OK;
    hipEvent_t done;
    hipError_t e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e);
    e = hipEventRecord(done, first);
    if (e == hipSuccess) e = hipStreamWaitEvent(s, done, 0);
    (void)hipEventDestroy(done);           // (released when what refers to it has run)
    return e == hipSuccess ? BSPMM_OK : hip_fail(e);
}

int run_out(void* stream)
{
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = capturing(s) ? hipSuccess : hipStreamSynchronize(s);
    return e == hipSuccess ? BSPMM_OK : hip_fail(e);
}

// (it forms 32-bit byte offsets inside an operation's dense blocks and multiplies a row's index and its
// bytes in 24 bits each: leading dimensions below 4 Mi floats, blocks below 4 GiB and 16 Mi rows)
bool takes_lean_kernel(const bspmm_plan* plan, bool transposed, int64_t ld_in, int64_t ld_out)
{
    constexpr int64_t kMul24 = (int64_t)1 << 22, kOff32 = (int64_t)1 << 30;
    constexpr int32_t kRows24 = 1 << 24;
    const int d = transposed ? 1 : 0;
    return plan->sched[d].pow2 && ld_in < kMul24 && ld_out < kMul24 && plan->lean_rows[d] <= kRows24 &&
           (int64_t)plan->lean_rows[d] * ld_in < kOff32 && (int64_t)plan->lean_out_rows[d] * ld_out < kOff32;
}

int64_t covered_rows(bspmm_plan* plan, bool transposed)
{
    int64_t& known = plan->covered[transposed ? 1 : 0];
    if (known >= 0) return known;
    const std::vector<int64_t>& off = transposed ? plan->dir[0].in_off : plan->dir[0].out_off;
    const std::vector<int32_t>& len = transposed ? plan->dir[0].k : plan->dir[0].m;
    std::vector<std::pair<int64_t, int64_t>> blocks;
    int64_t end = 0;
    for (size_t i = 0; i < off.size(); ++i) {
        if (blocks.empty() && off[i] <= end)       // the usual case: back to back in operation order
            end = std::max(end, off[i] + len[i]);
        else
            blocks.emplace_back(off[i], off[i] + len[i]);
    }
    std::sort(blocks.begin(), blocks.end());
    for (const auto& b : blocks) {
        if (b.first > end) break;
        end = std::max(end, b.second);
    }
    return known = end;
}

}  // namespace bspmm

extern "C" {

int bspmm_workspace_bytes(const bspmm_batch* b, int32_t F, const bspmm_options* options,
                          size_t* bytes)
{
    if (!bytes) return BSPMM_EINVAL;
    *bytes = 0;
    int rc = check_batch(b, F, false);
    if (rc != BSPMM_OK) return rc;
    bspmm_plan* p = new (std::nothrow) bspmm_plan;
    if (!p) return BSPMM_EINVAL;
    const bool dry = options && (options->flags & BSPMM_DRY_RUN);
    rc = plan_with_budget(*p, b, F, options, dry, plan_host);
    if (rc != BSPMM_OK) {
        delete p;
        return rc;
    }
    *bytes = p->lay.total;
    remember(p, make_key(b->batch, F, options, false));
    return BSPMM_OK;
}

int bspmm_create(bspmm_plan** plan, const bspmm_batch* b, int32_t F,
                 const bspmm_options* options, void* workspace, size_t workspace_bytes,
                 void* stream)
{
    return create_csr(plan, b, F, options, workspace, workspace_bytes, nullptr, static_cast<hipStream_t>(stream));
}

int bspmm_create_static(bspmm_plan** plan, const bspmm_batch* b, int32_t F,
                        const bspmm_options* options, void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    *plan = nullptr;
    if (options && (options->flags & BSPMM_DRY_RUN)) return BSPMM_EINVAL;
    int rc = check_batch(b, F, true);
    if (rc != BSPMM_OK) return rc;
    int dev = -1;
    void* ws = nullptr;
    rc = static_workspace(&dev, &ws);
    if (rc != BSPMM_OK) return rc;
    bspmm_plan* p = new (std::nothrow) bspmm_plan;
    if (!p) return BSPMM_EINVAL;
    rc = plan_with_budget(*p, b, F, options, false, plan_host);
    if (rc == BSPMM_OK && p->lay.total > (size_t)BSPMM_STATIC_WORKSPACE_BYTES && p->stream.on()) {
        // (a layer whose gather-first arrays do not fit: without them where that does)
        bspmm_options one = *options;
        one.flags |= BSPMM_ONE_FRONT_LAUNCH;
        delete p;
        p = new (std::nothrow) bspmm_plan;
        if (!p) return BSPMM_EINVAL;
        rc = plan_with_budget(*p, b, F, &one, false, plan_host);
    }
    if (rc == BSPMM_OK && p->lay.total > (size_t)BSPMM_STATIC_WORKSPACE_BYTES) rc = BSPMM_ENOSPACE;
    if (rc == BSPMM_OK) {
        p->rpt = b->rpt;
        p->colids = b->colids;
        p->values = b->values;
        // from here on the array belongs to this plan: earlier static plans of the device are
        // displaced before anything is written over their tables
        p->static_device = dev;
        p->static_generation =
            g_static_generation[dev].fetch_add(1, std::memory_order_acq_rel) + 1;
        rc = upload_plan(p, options, ws, (size_t)BSPMM_STATIC_WORKSPACE_BYTES,
                         static_cast<hipStream_t>(stream), nullptr, false);
    }
    return hand_over(p, rc, plan);
}

int bspmm_workspace_bytes_coo(const bspmm_coo_batch* b, int32_t F, const bspmm_options* options,
                              size_t* bytes)
{
    if (!bytes) return BSPMM_EINVAL;
    *bytes = 0;
    int rc = check_coo_batch(b, F, false);
    if (rc != BSPMM_OK) return rc;
    bspmm_plan* p = new (std::nothrow) bspmm_plan;
    if (!p) return BSPMM_EINVAL;
    const bool dry = options && (options->flags & BSPMM_DRY_RUN);
    rc = plan_with_budget(*p, b, F, options, dry, plan_host_coo);
    if (rc != BSPMM_OK) {
        delete p;
        return rc;
    }
    *bytes = p->lay.total;
    remember(p, make_key(b->batch, F, options, true));
    return BSPMM_OK;
}

int bspmm_create_coo(bspmm_plan** plan, const bspmm_coo_batch* b, int32_t F,
                     const bspmm_options* options, void* workspace, size_t workspace_bytes,
                     void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    *plan = nullptr;
    const bool dry = options && (options->flags & BSPMM_DRY_RUN);
    int rc = check_coo_batch(b, F, !dry);
    if (rc != BSPMM_OK) return rc;
    bspmm_plan* p = b->batch > 0 ? recall(make_key(b->batch, F, options, true), b, static_cast<const int64_t*>(nullptr)) : nullptr;
    if (!p) {
        p = new (std::nothrow) bspmm_plan;
        if (!p) return BSPMM_EINVAL;
        rc = plan_with_budget(*p, b, F, options, dry, plan_host_coo);
    }
    p->dry = dry;
    if (rc == BSPMM_OK && !dry) {
        p->ids = b->ids;
        p->coo_values = b->values;
        rc = upload_plan(p, options, workspace, workspace_bytes, static_cast<hipStream_t>(stream));
    }
    return hand_over(p, rc, plan);
}

int bspmm_export_csr(bspmm_plan* plan, int32_t* rpt, int32_t* colids, float* values, void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    if (plan->dry || !plan->from_coo || plan->coo_direct) return BSPMM_ESTATE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipSuccess;
    if (plan->csr_rpt_words) {
        if (!rpt) return BSPMM_EINVAL;
        e = hipMemcpyAsync(rpt, plan->rpt, (size_t)plan->csr_rpt_words * 4, hipMemcpyDeviceToDevice, s);
    }
    if (e == hipSuccess && plan->csr_nz) {
        if (!colids || !values) return BSPMM_EINVAL;
        e = hipMemcpyAsync(colids, plan->colids, (size_t)plan->csr_nz * 4, hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(values, plan->values, (size_t)plan->csr_nz * 4,
                               hipMemcpyDeviceToDevice, s);
    }
    return e == hipSuccess ? BSPMM_OK : hip_fail(e);
}

int bspmm_run(bspmm_plan* plan, const float* B, float* C, int64_t ldb, int64_t ldc,
              void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    if (plan->dry || displaced(plan)) return BSPMM_ESTATE;
    const int rc = settle(plan, static_cast<hipStream_t>(stream));
    if (rc != BSPMM_OK) return rc;
    return run_direction(plan, 0, B, C, ldb, ldc, static_cast<hipStream_t>(stream));
}

int bspmm_run_gcn(bspmm_plan* plan, const float* X, int64_t ldx, const float* W, int64_t ldw,
                  const float* bias, float* Y, int64_t ldy, int32_t accumulate, void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    if (plan->dry || plan->knobs.front <= 0 || plan->coo_direct || displaced(plan)) return BSPMM_ESTATE;
    const int rc = settle(plan, static_cast<hipStream_t>(stream));
    if (rc != BSPMM_OK) return rc;
    return run_gcn(plan, X, ldx, W, ldw, bias, Y, ldy, accumulate, static_cast<hipStream_t>(stream));
}

int bspmm_run_transposed(bspmm_plan* plan, const float* dY, float* G, int64_t ldy, int64_t ldg,
                         void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    if (plan->dry || !plan->transposed_supported || displaced(plan)) return BSPMM_ESTATE;
    int rc = settle(plan, static_cast<hipStream_t>(stream));
    if (rc != BSPMM_OK) return rc;
    if (plan->coo_direct)
        return run_direction(plan, 1, dY, G, ldy, ldg, static_cast<hipStream_t>(stream));
    if (plan->sched[1].grid > 0 && ((!dY && plan->reads_dense) || !G || ldy < plan->F || ldg < plan->F))
        return BSPMM_EINVAL;
    if (plan->sorts_in_run && !plan->transposed_built && on_quads(plan, dY, G, ldy, ldg) &&
        bspmm::takes_lean_kernel(plan, true, ldy, ldg))
        return first_transposed(plan, dY, G, ldy, ldg, static_cast<hipStream_t>(stream));
    rc = enqueue_build(plan, static_cast<hipStream_t>(stream));
    if (rc != BSPMM_OK) return rc;
    return run_direction(plan, 1, dY, G, ldy, ldg, static_cast<hipStream_t>(stream));
}

int bspmm_export_transposed(bspmm_plan* plan, int32_t* rpt_t, int32_t* colids_t,
                            float* values_t, void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    if (plan->dry || plan->coo_direct || plan->knobs.symmetric || displaced(plan)) return BSPMM_ESTATE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int rc = settle(plan, s);
    if (rc == BSPMM_OK) rc = enqueue_build(plan, s);
    if (rc != BSPMM_OK) return rc;
    size_t rpt_words = 0, nz = 0;
    for (int i = 0; i < plan->batch; ++i) {
        rpt_words += (size_t)plan->dir[1].m[i] + 1;
        nz += (size_t)plan->dir[1].nnz[i];
    }
    hipError_t e = hipSuccess;
    if (rpt_words) {
        if (!rpt_t) return BSPMM_EINVAL;
        e = hipMemcpyAsync(rpt_t, plan->ws + plan->lay.rpt_t, rpt_words * 4,
                           hipMemcpyDeviceToDevice, s);
    }
    if (e == hipSuccess && nz) {
        if (!colids_t || !values_t) return BSPMM_EINVAL;
        e = hipMemcpyAsync(colids_t, plan->ws + plan->lay.colids_t, nz * 4,
                           hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(values_t, plan->ws + plan->lay.values_t, nz * 4,
                               hipMemcpyDeviceToDevice, s);
    }
    return e == hipSuccess ? BSPMM_OK : hip_fail(e);
}

int bspmm_validate(bspmm_plan* plan, int32_t* bad_op, void* stream)
{
    if (!plan) return BSPMM_EINVAL;
    if (plan->dry || displaced(plan)) return BSPMM_ESTATE;
    if (bad_op) *bad_op = -1;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int rc = settle(plan, s);
    if (rc != BSPMM_OK) return rc;
    int32_t* flag = reinterpret_cast<int32_t*>(plan->ws + plan->lay.flag);
    hipError_t e = plan->from_coo
        ? launch_validate_coo(reinterpret_cast<const OpRecord*>(plan->ws + plan->lay.coo_records),
                              plan->batch, plan->ids, flag, s)
        : launch_validate(reinterpret_cast<const OpRecord*>(plan->ws + plan->lay.op_records),
                          plan->batch, plan->rpt, plan->colids, flag, s);
    if (e != hipSuccess) return hip_fail(e);
    int32_t host_flag = 0;
    e = hipMemcpyAsync(&host_flag, flag, 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e);
    if (host_flag != 0x7fffffff) {
        if (bad_op) *bad_op = host_flag;
        return BSPMM_EBADCSR;
    }
    return BSPMM_OK;
}

int bspmm_kernel_info(int32_t kernel, int32_t dynamic_lds_bytes, bspmm_kernel_resources* out)
{
    if (!out || kernel < 0 || kernel > BSPMM_KERNEL_LAYER_STREAM || dynamic_lds_bytes < 0) return BSPMM_EINVAL;
    int v[7] = {0, 0, 0, 0, 0, 0, 0};
    const hipError_t e = kernel_resources(kernel, dynamic_lds_bytes, v);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return hip_fail(e);
    }
    out->vgprs = v[0];
    out->sgprs = v[1];
    out->static_lds_bytes = v[2];
    out->scratch_bytes = v[3];
    out->threads = v[4];
    out->workgroups_per_cu = v[5];
    out->compute_units = v[6];
    out->reserved_ = 0;
    return BSPMM_OK;
}

int bspmm_plan_info(const bspmm_plan* plan, bspmm_info* info)
{
    if (!plan || !info) return BSPMM_EINVAL;
    std::memset(info, 0, sizeof(*info));
    info->batch = plan->batch;
    info->F = plan->F;
    info->lds_bytes = 4 * std::max(plan->sched[0].budget_words, plan->sched[1].budget_words);
    if (plan->coo_direct)      // the direct COO launches ask for their largest item's LDS
        info->lds_bytes = 4 * std::max(plan->coo_sched[0].lds_words, plan->coo_sched[1].lds_words);
    info->compute_units = plan->knobs.compute_units;
    for (int d = 0; d < 2; ++d) {
        info->tile[d] = plan->sched[d].tile;
        info->workgroups[d] = plan->sched[d].launch_grid;
        info->tasks[d] = plan->sched[d].grid;
        info->items[d] = plan->sched[d].count;
        for (int b = 0; b < BSPMM_NUM_BINS; ++b)
            info->items_in_bin[d][b] = plan->sched[d].items_in_bin[b];
        info->effective_bytes[d] = plan->effective_bytes[d];
        info->fused_tasks[d] = plan->sched[d].fused_tasks;
        if (plan->coo_direct) {
            info->tile[d] = plan->coo_sched[d].tile;
            info->workgroups[d] = info->tasks[d] = info->items[d] =
                (int32_t)plan->coo_sched[d].items.size();
        }
    }
    info->transposed_supported = plan->transposed_supported ? 1 : 0;
    info->transposed_built = plan->transposed_built ? 1 : 0;
    for (int d = 0; d < 2; ++d) info->lean[d] = plan->sched[d].pow2 && plan->sched[d].merged_sets.empty() ? 1 : 0;
    if (plan->stream.on() && plan->stream.many) {
        info->front_stream[0] = plan->stream.graphs;
        info->front_stream[1] = 8 * plan->stream.parts[0].ranges_per_xcd * plan->stream.tiles;
        info->front_stream[2] = plan->stream.parts[0].lds_bytes;
        int32_t left = 0;
        for (const WorkItem& w : plan->stream.rest) left += w.f0 == 0 ? 1 : 0;
        info->front_stream[3] = left;
    }
    info->flops = plan->flops;
    info->workspace_bytes = plan->lay.total;
    return BSPMM_OK;
}

int bspmm_plan_items(const bspmm_plan* plan, int32_t transposed, bspmm_item* items,
                     int32_t capacity, int32_t* count)
{
    if (!plan || !count || capacity < 0 || (capacity > 0 && !items)) return BSPMM_EINVAL;
    const int d = transposed ? 1 : 0;
    const std::vector<bspmm_item> v = plan->coo_direct ? plan->coo_sched[d].view
                                                       : items_of(plan->sched[d], plan->lean_items[plan->lean_shared ? 0 : d]);
    *count = (int32_t)v.size();
    const size_t n = std::min<size_t>(v.size(), (size_t)capacity);
    if (n) std::memcpy(items, v.data(), n * sizeof(bspmm_item));
    return BSPMM_OK;
}

void bspmm_destroy(bspmm_plan* plan)
{
    if (plan && plan->copied) (void)hipEventDestroy(plan->copied);
    if (plan && plan->counted) stage_plan_gone();
    delete plan;
}

const char* bspmm_strerror(int code)
{
    switch (code) {
        case BSPMM_OK: return "ok";
        case BSPMM_EINVAL: return "invalid argument";
        case BSPMM_ENOSPACE: return "workspace too small";
        case BSPMM_EHIP: return "HIP runtime error";
        case BSPMM_EOVERLAP: return "output blocks overlap";
        case BSPMM_ESTATE: return "operation not available on this plan";
        case BSPMM_EBADCSR: return "malformed CSR arrays on the device";
        case BSPMM_ETOOBIG: return "operations do not fit on chip (those summed into one block together, or one with the fused front)";
        default: return "unknown error";
    }
}

int bspmm_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
