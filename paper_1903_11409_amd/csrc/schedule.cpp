// Batch scheduler (host only).
//
// The paper's Batched SpMM for CSR (Sec. IV-C) sizes one launch from the batch maximum:
// max m_A * subWarp * batch [* p] threads, column blocking for all operations if any needs it,
// surplus threads exit.  Here every operation is scheduled from its own size instead:
//   * the feature dimension is cut into tiles (the column blocking of Fig. 5(d)); the
//     batch-wide tile is the widest one that still yields enough workgroups to fill the chip,
//     and an operation whose dense tile does not fit its LDS share gets narrower tiles;
//   * an (operation, tile) item runs on a 16/32-lane slice, a wavefront or a workgroup,
//     whichever is the smallest that finishes its rows in a few passes and holds its operands
//     in the slot's share of LDS; operations too large for LDS at the narrowest tile fall to
//     the generic bin, cut into row blocks that read global memory;
//   * work is ordered largest-first; items that read the same dense tile (row blocks of a
//     large operation, channels of one graph) are kept on one XCD, i.e. on workgroup indices
//     that are equal modulo 8, so the tile is fetched into one L2 only.
#include "schedule.hpp"

#include <algorithm>
#include <cstdint>
#include <initializer_list>
#include <map>
#include <numeric>
#include <utility>

namespace bspmm {

namespace {

constexpr int kXcds = 8;
constexpr int kFrontBlocks = 8;   // matrix-core blocks one workgroup of the fused front should make

struct Draft {           // one item before placement
    int op;
    int bin;
    int row0, nrows, f0, fw;
    int staged;
    int64_t cost;
    int group;           // items with one group read the same dense tile
    int fused;           // >= 0: index of the set of operations this task adds up
};

int bin_slot_lanes(int bin)
{
    switch (bin) {
        case BSPMM_BIN_WAVE: return 64;
        case BSPMM_BIN_SLICE32: return 32;
        case BSPMM_BIN_SLICE16: return 16;
        default: return kThreads;
    }
}

int bin_range(int bin)
{
    switch (bin) {
        case BSPMM_BIN_WAVE: return 2;
        case BSPMM_BIN_SLICE32: return 3;
        case BSPMM_BIN_SLICE16: return 4;
        default: return 0;
    }
}

int draft_range(const Draft& x) { return x.fused >= 0 ? 1 : bin_range(x.bin); }

// Whether these knobs leave every launch to bspmm_kernel (see Schedule::whole).
bool general_only(const Knobs& kn)
{
    return kn.front > 0 || kn.hubs || kn.pad != 0 || kn.persistent_wgs > 0 || kn.wide_offsets;
}

// Output rows of operation i that a whole workgroup has in flight (see bspmm_any_kernel; long rows off 16
// bytes take a lane per float); in launches that
// run in bspmm_kernel, which gives a row a power of two of lanes, at most four of its passes (200 operations
// of 1 to 220 rows with hub rows split: F = 17 10.2 -> 9.1 us, F = 50 10.5 -> 9.8, F = 127 17.6 -> 14.8; one
// pass instead of four: F = 17 8.3, but F = 127 18.3 and F = 301 37.0 against 26.4).
int rows_in_flight(const DirOps& o, int i, int fw, int vec, const Knobs& kn)
{
    const int per_lane = vec == 1 && o.nnz[i] > kLongRow * o.m[i] ? 1 : 4;
    const int rows = std::max(1, kThreads / std::max(1, (fw + per_lane - 1) / per_lane));
    return general_only(kn) ? std::min(rows, 4 * (kThreads / lanes_per_row(fw, vec))) : rows;
}

// Candidate tile widths, widest first.
std::vector<int> tile_candidates(int F, const Knobs& kn)
{
    std::vector<int> c;
    if (F % 4 != 0 && kn.front == 0) {
        // Widths that no 16-byte load divides gain nothing from powers of two: the columns are split evenly
        // (on even columns where F is even).  The launches of bspmm_kernel and of the direct COO kernel
        // take the same tiles: 200 operations of 1 to 220 rows from index pairs F = 17 16.0 -> 10.5 us, F = 50
        // 15.3 -> 11.5, F = 127 18.1 -> 17.6, F = 301 55.0 -> 46.7 against powers of two; 60 of them F = 50
        // 14.4 -> 8.8; 512 sums of four at F = 127 14.4 -> 8.5.  (On operands that stay in the caches F = 127
        // loses: 14.8 -> 15.6.)
        const int even = F % 2 == 0 ? 2 : 1;
        for (int parts = (F + kn.max_tile - 1) / kn.max_tile; ; parts += (parts + 2) / 3) {
            const int w = round_up((F + parts - 1) / parts, even);
            if (!c.empty() && w < kn.min_odd_tile) break;
            if (w <= kn.max_tile && (c.empty() || w < c.back())) c.push_back(w);
            if (w <= even) break;
        }
        return c;
    }
    int t = std::min(F, kn.max_tile);
    c.push_back(t);
    int p = 1;
    while (p * 2 < t) p *= 2;        // largest power of two below t
    if (p == t) p /= 2;
    for (; p >= kn.min_tile && p >= 4; p /= 2) c.push_back(p);
    return c;
}

struct Choice {
    int bin;
    int tile;
};

bool fits_slot(const DirOps& o, int i, int tile, int F, int vec, int lanes, int max_passes,
               const Knobs& kn)
{
    const int fw = std::min(tile, F);
    const int g = lanes_per_row(fw, vec);
    if (g > lanes) return false;
    const int64_t lanes_wanted = (int64_t)o.m[i] * g;
    if (max_passes > 0 && (lanes_wanted + lanes - 1) / lanes > max_passes) return false;
    const int64_t head = (int64_t)round_up(o.m[i] + 1, 2) + 2 * (int64_t)o.nnz[i];
    int64_t need = (head + 3) / 4 * 4 + (int64_t)o.k[i] * (round_up(fw, 4) + kn.pad);
    if (vec == 1) need = std::max(need, any_words(o.m[i], o.k[i], o.nnz[i], fw, false));
    if (kn.hubs && lanes == kThreads) need += hub_words(o.nnz[i] / kHubMin, fw);   // as staged_layout()
    if (kn.front > 0)   // a weight tile and a bias tile per channel and at least 16 rows of X_i ride along
        need += 16 * (int64_t)kn.front +
                o.channels(i) * ((int64_t)kn.front * round_up(fw, 4) + round_up(fw, 4));
    return need <= (int64_t)kn.lds_words * lanes / kThreads;
}

// Decide bin and tile of operation i given the batch-wide tile candidates from `first` on.
// `widest_fit` (optional): per operation, the index of the widest candidate whose whole-workgroup
// item fits LDS (cand.size() when none does).  Fitting is monotone in the tile width, so with it
// the plain case - no forced bin, no sub-workgroup slots - is answered without looking at the
// operation again, however often the search over tiles and row cuts asks.
Choice choose(const DirOps& o, int i, int F, int vec, const std::vector<int>& cand, size_t first,
              const Knobs& kn, bool allow_small, const std::vector<uint8_t>* widest_fit = nullptr)
{
    const int forced = kn.front > 0 ? BSPMM_BIN_WORKGROUP : kn.force_bin;   // the fused front runs on whole workgroups
    if (widest_fit && forced < 0 && !allow_small) {
        const size_t c = std::max<size_t>(first, (*widest_fit)[i]);
        return c < cand.size() ? Choice{BSPMM_BIN_WORKGROUP, cand[c]} : Choice{BSPMM_BIN_GENERIC, cand[0]};
    }
    if (forced == BSPMM_BIN_GENERIC) return {BSPMM_BIN_GENERIC, cand[0]};
    if (forced >= 0) {
        for (size_t c = first; c < cand.size(); ++c) {
            // fused front: a workgroup makes its whole dense tile on the matrix cores before it
            // can gather, and the launch lasts as long as its slowest workgroup, so a larger
            // operation takes a narrower tile (at most kFrontBlocks 16 x 16 blocks each)
            if (kn.front > 0 && c + 1 < cand.size() &&
                ((o.k[i] + 15) / 16) * ((std::min(cand[c], F) + 15) / 16) > kFrontBlocks)
                continue;
            if (fits_slot(o, i, cand[c], F, vec, bin_slot_lanes(forced), 0, kn))
                return {forced, cand[c]};
        }
    }
    const int tile = cand[first];
    static const int small_bins[3] = {BSPMM_BIN_SLICE16, BSPMM_BIN_SLICE32, BSPMM_BIN_WAVE};
    for (int b : small_bins)
        if (allow_small && fits_slot(o, i, tile, F, vec, bin_slot_lanes(b), kn.max_passes, kn))
            return {b, tile};
    for (size_t c = first; c < cand.size(); ++c)
        if (fits_slot(o, i, cand[c], F, vec, kThreads, 0, kn))
            return {BSPMM_BIN_WORKGROUP, cand[c]};
    return {BSPMM_BIN_GENERIC, cand[0]};
}

int64_t item_cost(const DirOps& o, int i, int nrows, int fw, bool staged)
{
    const int64_t dense_in = staged ? o.k[i] : std::min<int64_t>(o.k[i], (int64_t)nrows * 4);
    return 4 * (int64_t)fw * (dense_in + nrows) + 8 * (int64_t)o.nnz[i] * nrows / std::max(o.m[i], 1) +
           4 * (int64_t)nrows + 512;
}

// Where drafted items go.  Sizing the launch only needs to know how many items each launch
// range would get, so the search over tiles and row cuts runs on a sink that counts; the one
// draft that is kept is built with a sink that stores the items.
struct Sink {
    std::vector<Draft>* out = nullptr;     // null: count only
    int per_range[kRanges] = {0, 0, 0, 0, 0};
    int generic = 0;                       // items that read their operands from global memory
    int64_t tile_words = 0;                // counting only: dense-tile words the staged items copy
    const std::vector<int>* block_of_op = nullptr;   // dense-input block index of every operation
    int tiles_per_block = 1;               // group id = block * tiles_per_block + f0 / tile_unit
    int tile_unit = 4;
    void add(const DirOps& o, int i, int bin, int row0, int nrows, int f0, int fw, int staged,
             int fused)
    {
        per_range[fused >= 0 ? 1 : bin_range(bin)]++;
        generic += bin == BSPMM_BIN_GENERIC;
        if (!out) return;
        const int gid = fused >= 0 ? -1 : (*block_of_op)[i] * tiles_per_block + f0 / tile_unit;
        out->push_back({i, bin, row0, nrows, f0, fw, staged,
                        fused >= 0 ? 0 : item_cost(o, i, nrows, fw, staged != 0), gid, fused});
    }
    int workgroups() const
    {
        int wgs = per_range[0] + per_range[1];
        for (int r = 2; r < kRanges; ++r) {
            const int slots = kThreads >> range_log2_slot(r);
            wgs += (per_range[r] + slots - 1) / slots;
        }
        return wgs;
    }
};

// `cap` > 0 cuts a workgroup item into row ranges of at most `cap` passes each (every range
// stages the whole operation, so the cut costs on-chip traffic and buys parallelism).
void draft_op(const DirOps& o, int i, int F, int vec, const Choice& ch, const Knobs& kn, int cap,
              Sink& sink)
{
    if (o.m[i] <= 0) return;
    const int tile = ch.tile;
    if (!sink.out) {    // counting: the same items in closed form
        auto per_tile = [&](int fw) {
            if (ch.bin == BSPMM_BIN_WORKGROUP && cap > 0) {
                const int chunk = cap * rows_in_flight(o, i, fw, vec, kn);
                return (o.m[i] + chunk - 1) / chunk;
            }
            if (ch.bin != BSPMM_BIN_GENERIC) return 1;
            return (o.m[i] + kn.generic_rows - 1) / kn.generic_rows;
        };
        const int full = F / tile, tail = F % tile;
        const int n_full = full ? per_tile(tile) : 0, n_tail = tail ? per_tile(tail) : 0;
        const int n = full * n_full + n_tail;
        sink.per_range[bin_range(ch.bin)] += n;
        sink.generic += ch.bin == BSPMM_BIN_GENERIC ? n : 0;
        if (ch.bin != BSPMM_BIN_GENERIC)   // every piece of a cut item copies the whole tile
            sink.tile_words += (int64_t)o.k[i] * ((int64_t)full * n_full * tile + (int64_t)n_tail * tail);
        return;
    }
    for (int f0 = 0; f0 < F; f0 += tile) {
        const int fw = std::min(tile, F - f0);
        if (ch.bin == BSPMM_BIN_WORKGROUP && cap > 0) {
            const int chunk = cap * rows_in_flight(o, i, fw, vec, kn);
            for (int r0 = 0; r0 < o.m[i]; r0 += chunk)
                sink.add(o, i, ch.bin, r0, std::min(chunk, o.m[i] - r0), f0, fw, 1, -1);
        } else if (ch.bin != BSPMM_BIN_GENERIC) {
            sink.add(o, i, ch.bin, 0, o.m[i], f0, fw, 1, -1);
        } else {
            for (int r0 = 0; r0 < o.m[i]; r0 += kn.generic_rows)
                sink.add(o, i, ch.bin, r0, std::min(kn.generic_rows, o.m[i] - r0), f0, fw, 0, -1);
        }
    }
}

// LDS words a fused task needs: mirrors run_fused() in kernels.hip.
int64_t fused_words(const DirOps& o, const std::vector<int>& members, int fw)
{
    int64_t nnz_sum = 0;
    for (int i : members) nnz_sum += o.nnz[i];
    int64_t words = round_up(o.m[members[0]] + 1, 4) + 2 * ((nnz_sum + 1) / 2 * 2);
    for (size_t j = 0; j < members.size(); ++j) {
        bool owns = true;
        for (size_t e = 0; e < j; ++e)   // (the same block: same first row AND same row count)
            owns = owns && !(o.in_off[members[e]] == o.in_off[members[j]] && o.k[members[e]] == o.k[members[j]]);
        if (owns) words += (int64_t)o.k[members[j]] * round_up(fw, 4);
    }
    return words;
}

// Tasks of one set of operations that are summed into one output block.  The tile is the
// widest candidate (from `first` on, then 16, 8 and 4 floats) whose task fits LDS; returns false
// when none does.
bool draft_fused(const DirOps& o, const std::vector<int>& members, int fused_index, int F, int vec,
                 const std::vector<int>& cand, size_t first, const Knobs& kn, int cap,
                 Sink& sink)
{
    std::vector<int> tiles(cand.begin() + first, cand.end());
    for (int t : {16, 8, 4})
        if (t < tiles.back()) tiles.push_back(t);
    int tile = 0;
    for (int t : tiles)
        if (fused_words(o, members, std::min(t, F)) <= kn.lds_words) {
            tile = t;
            break;
        }
    if (!tile) return false;
    const int m = o.m[members[0]];
    for (int f0 = 0; f0 < F; f0 += tile) {
        const int fw = std::min(tile, F - f0);
        const int rows_per_pass = kThreads / lanes_per_row(fw, vec);
        const int chunk = cap > 0 ? cap * rows_per_pass : m;
        for (int r0 = 0; r0 < m; r0 += chunk) {
            const int nr = std::min(chunk, m - r0);
            sink.add(o, members[0], BSPMM_BIN_WORKGROUP, r0, nr, f0, fw, 1, fused_index);
            if (sink.out) {
                int64_t cost = 0;
                for (int i : members) cost += item_cost(o, i, nr, fw, true);
                sink.out->back().cost = cost;
            }
        }
    }
    return true;
}

// Operations grouped by the output block they name: a group of more than one is summed.
// Groups are listed in the order of their first operation, members in operation order; group g
// is member[start[g]] .. member[start[g + 1] - 1].
struct Groups {
    std::vector<int> start, member;
    int size() const { return (int)start.size() - 1; }
    int count(int g) const { return start[g + 1] - start[g]; }
    const int* begin(int g) const { return member.data() + start[g]; }
    std::vector<int> members(int g) const { return std::vector<int>(begin(g), begin(g) + count(g)); }
};

Groups output_groups(const DirOps& o)
{
    Groups out;
    const int n = o.size();
    out.member.reserve(n);
    out.start.reserve(n + 1);
    // the usual case: every operation has an output block of its own, later operations at
    // higher rows - nothing to sort
    bool separate = true;
    int64_t end = -1;
    for (int i = 0; i < n && separate; ++i) {
        if (o.m[i] <= 0) continue;
        separate = o.out_off[i] >= end;
        end = o.out_off[i] + o.m[i];
    }
    if (separate) {
        for (int i = 0; i < n; ++i)
            if (o.m[i] > 0) {
                out.start.push_back((int)out.member.size());
                out.member.push_back(i);
            }
        out.start.push_back((int)out.member.size());
        return out;
    }
    std::vector<int> idx;
    idx.reserve(n);
    for (int i = 0; i < n; ++i)
        if (o.m[i] > 0) idx.push_back(i);
    std::vector<int> sorted = idx;
    std::sort(sorted.begin(), sorted.end(), [&](int a, int b) {
        if (o.out_off[a] != o.out_off[b]) return o.out_off[a] < o.out_off[b];
        if (o.m[a] != o.m[b]) return o.m[a] < o.m[b];
        return a < b;
    });
    // leader[i] = first operation (lowest index) naming the same block as i; size[l] = members
    std::vector<int> leader(n, -1), size(n, 0);
    for (size_t a = 0; a < sorted.size();) {
        size_t b = a;
        while (b < sorted.size() && o.out_off[sorted[b]] == o.out_off[sorted[a]] &&
               o.m[sorted[b]] == o.m[sorted[a]])
            leader[sorted[b++]] = sorted[a];
        size[sorted[a]] = (int)(b - a);
        a = b;
    }
    // groups in the order of their leaders; a group's slots are filled in operation order
    std::vector<int> at(n, -1);
    int total = 0;
    for (int i : idx)
        if (leader[i] == i) {
            out.start.push_back(total);
            at[i] = total;
            total += size[i];
        }
    out.start.push_back(total);
    out.member.resize(total);
    for (int i : idx) out.member[at[leader[i]]++] = i;
    return out;
}

// Index of the dense-input block of every operation (operations reading the same first row
// share an index).
std::vector<int> input_blocks(const DirOps& o)
{
    std::vector<int> block(o.size(), 0);
    bool sorted = true;            // the usual case: blocks back to back in operation order
    for (int i = 1; i < o.size() && sorted; ++i) sorted = o.in_off[i] >= o.in_off[i - 1];
    if (sorted) {
        for (int i = 1; i < o.size(); ++i) block[i] = block[i - 1] + (o.in_off[i] != o.in_off[i - 1]);
        return block;
    }
    std::vector<int> order(o.size());
    std::iota(order.begin(), order.end(), 0);
    std::sort(order.begin(), order.end(),
              [&](int a, int b) { return o.in_off[a] != o.in_off[b] ? o.in_off[a] < o.in_off[b] : a < b; });
    int nb = -1;
    for (size_t t = 0; t < order.size(); ++t) {
        if (t == 0 || o.in_off[order[t]] != o.in_off[order[t - 1]]) ++nb;
        block[order[t]] = nb;
    }
    return block;
}

// Narrowest tile a stand-in may take: the narrowest batch-wide candidate, or half of it when
// only that fits (the members' tiles side by side are several times an operation's tile; 0 when
// neither fits).
int stand_in_tile(const DirOps& o, int v, int F, int vec, const std::vector<int>& cand, const Knobs& kn)
{
    if (fits_slot(o, v, cand.back(), F, vec, kThreads, 0, kn)) return cand.back();
    const int half = cand.back() / 2;
    if (half >= 16 && half % 4 == 0 && fits_slot(o, v, half, F, vec, kThreads, 0, kn)) return half;
    return 0;
}

// `stand_in[g]` >= 0: the operations of group g all read one dense block, so their sum is the
// product with the sum of their matrices: one operation (appended to `o` at that index, its CSR
// the set's merged one) stands in for them and is drafted as a workgroup item like any other.
void draft_all(const DirOps& o, int F, int vec, const std::vector<int>& cand, size_t first,
               const Knobs& kn, int cap, bool allow_small,
               const Groups& outs, const std::vector<int>& stand_in, bool* fits, Sink& sink,
               const std::vector<uint8_t>* widest_fit = nullptr)
{
    int nfused = 0;
    for (int g = 0; g < outs.size(); ++g) {
        if (outs.count(g) == 1) {
            const int i = *outs.begin(g);
            draft_op(o, i, F, vec, choose(o, i, F, vec, cand, first, kn, allow_small, widest_fit), kn, cap, sink);
        } else if (stand_in[g] >= 0) {
            const int v = stand_in[g];
            Choice ch = {BSPMM_BIN_WORKGROUP, stand_in_tile(o, v, F, vec, cand, kn)};
            for (size_t c = first; c < cand.size(); ++c)
                if (fits_slot(o, v, cand[c], F, vec, kThreads, 0, kn)) {
                    ch.tile = cand[c];
                    break;
                }
            draft_op(o, v, F, vec, ch, kn, cap, sink);
        } else if (!draft_fused(o, outs.members(g), nfused++, F, vec, cand, first, kn, cap, sink)) {
            *fits = false;
        }
    }
}

// The search over batch-wide tiles and row cuts (plain batches without a caller's knobs have a rule
// of their own: plain_shape).  count(first, cap) says how many workgroups the launch would get with
// candidate tiles from `first` on and workgroup items cut into row ranges of `cap` passes (0: not cut),
// and how many dense-tile words its staged items would copy.
struct Count {
    int wgs;
    int64_t tile_words;
    bool row_blocks;      // some operations are cut into row blocks that gather from memory
    int64_t in_words;     // of the dense blocks of all operations
    int blocked;          // operations in row blocks, and the dense blocks of those
    int64_t blocked_words;
};
// Whether the operations in row blocks are the tail of the others' sizes, not a few giants among small ones: at most
// six times their dense input on average (heavy-tailed graphs have 5, uniformly random matrices 2).
bool one_tail(const Count& t, int n)
{
    return t.blocked >= n || t.blocked_words * (n - t.blocked) <= 6 * (t.in_words - t.blocked_words) * t.blocked;
}
struct Shape {
    size_t chosen;
    int cap, wgs;
};

template <typename CountFn>
Shape search_shape(const Knobs& kn, int vec, size_t candidates, CountFn count)
{
    Shape s = {candidates - 1, kn.wg_passes > 0 ? kn.wg_passes : 0, 0};
    // (F % 4 != 0: the widest tile every operation can hold, and row ranges for parallelism - see below)
    const bool wide_first = vec == 1 && kn.front == 0;
    int64_t tile_words = 0;
    for (size_t c = 0; c < candidates; ++c) {
        const Count n = count(c, s.cap);
        s.wgs = n.wgs;
        tile_words = n.tile_words;
        if (wide_first || s.wgs >= kn.target_wgs || c + 1 == candidates) {
            s.chosen = c;
            break;
        }
    }
    if (kn.wg_passes != 0 || kn.front != 0) return s;
    if (wide_first) {
        // Widths off 16 bytes: a tile of whole rows is one run of memory, cheaper to copy several
        // times (out of L2) than column tiles whose rows start anywhere.  Ranges of at most eight
        // passes over the lane groups (200 operations of 1 to 220 rows, F = 127: uncut 16.5 us, sixteen
        // passes 12.3, eight 9.3), shorter until there are three and a half workgroups per CU (two per
        // CU: 100 operations 7.5 us instead of 6.6, 150 9.3 instead of 8.1; five: 6.9 and 8.1), but not in
        // launches bound by bandwidth.
        const int want = kn.target_given ? kn.target_wgs : 7 * kn.compute_units / 2;
        for (int c = 8; c >= 1; c /= 2) {
            const Count n = count(s.chosen, c);
            s.wgs = n.wgs;
            s.cap = c;
            if (n.wgs >= want || n.tile_words > 3500000) break;
        }
        return s;
    }
    // still too few workgroups at the narrowest tile: the batch is small, its time is set by
    // the slowest workgroup, so cut multi-pass workgroup items into row ranges
    // Likewise while the launch still fits the chip at once: the workgroups with several passes
    // are its critical path, and cutting them pays as long as no workgroup has to wait for a
    // free slot and the pieces, each of which copies the whole dense tile again, do not add
    // more than 60 % to the tile traffic (measured: 256 molecule graphs 4.9 -> 4.3 us, 512
    // graphs 5.9 -> 4.8 us; cut beyond what the chip holds, 384 graphs go from 4.9 to 5.9 us;
    // wide tiles of 100-row graphs cut to four rows each, 8.2 -> 9.2 us).
    const int uncut = s.wgs;                       // (the tile search ended on this very count)
    const int64_t uncut_words = tile_words;
    // (a launch that moves more than about 28 MB is bound by bandwidth, not by its slowest
    // workgroup: there the extra copies only cost)
    const bool latency_bound = uncut_words <= 3500000;
    for (int c = 1; c <= 4 && uncut <= kn.capacity_wgs && latency_bound; c *= 2) {
        const Count n = count(s.chosen, c);
        if (n.wgs <= kn.capacity_wgs && 5 * (n.tile_words - uncut_words) <= 3 * uncut_words) {
            s.cap = c;
            s.wgs = n.wgs;
            return s;
        }
    }
    if (uncut < kn.target_wgs)
        for (s.cap = 4; s.cap >= 1; s.cap /= 2) {
            s.wgs = count(s.chosen, s.cap).wgs;
            if (s.wgs >= kn.target_wgs || s.cap == 1) break;
        }
    return s;
}

WorkItem to_item(const DirOps& o, const Draft& x)
{
    WorkItem w;
    w.rpt_off = o.rpt_off[x.op];
    w.nz_off = o.nz_off[x.op];
    w.in_row_off = o.in_off[x.op];
    w.out_row_off = o.out_off[x.op];
    w.m = o.m[x.op];
    w.k = o.k[x.op];
    w.nnz = o.nnz[x.op];
    w.row0 = x.row0;
    w.nrows = x.nrows;
    w.f0 = x.f0;
    w.fw = x.fw;
    w.staged = x.staged;
    return w;
}

WorkItem empty_item()
{
    WorkItem w;
    w.rpt_off = w.nz_off = w.in_row_off = w.out_row_off = 0;
    w.m = w.k = w.nnz = w.row0 = w.nrows = w.f0 = w.fw = 0;
    w.staged = 1;
    return w;
}

// The rule for plain batches on the float4 path without a caller's knobs.  fit(words, c) plans the tiles for
// that LDS budget and row blocks for candidate c.  Row ranges copy their tile again and column tiles
// stage the CSR again.  Out of the caches the copies of a tile that row ranges make are cheap, on operands
// that come from memory they are not: the two orders disagree, and where they do the rule goes by the
// operands from memory.  Measured on MI355X over 110 batches (8 to 8192 graphs of molecule, 20-100-node,
// heavy-tailed and random-matrix sizes, F = 16 to 1024), times in us on operands from memory / out of
// the caches:
//  - A launch that fits the chip at once (six workgroups of 24 KiB per CU) lasts as long as its slowest
//    workgroup: ranges of 32 rows, of 64 if it then fits, at the narrowest tile at which it does (128
//    molecules at F = 128 2.93 / 2.78 in 32 columns, 3.10 / 2.61 in 128 columns cut to 8 rows; at F = 256
//    3.37 / 3.25 against 3.91 / 3.00; 384 of them at F = 128 3.79 / 3.53 in 64 columns, 4.29 / 3.34; 20
//    heavy-tailed graphs at F = 256 3.6 / 3.2 against 4.7 / 3.8), unless it moves more than 28 MB.  With
//    operations in row blocks: the narrowest tile only, and where at least half of the dense input is
//    staged (20 random matrices at F = 512 6.1 / 3.6 in 32 columns, 4.1 / 3.7 uncut in 128).  Up to F = 64
//    ranges of one pass, 16 rows at F = 64, or of two, if it then fits: the orders are within 4 % of each
//    other (512 molecules at F = 64 3.44 / 3.06, in 32 columns 3.30 / 3.20), and a fifth more items to
//    plan and send cost a data loader more (plan and two products from index pairs 50.1, 47.6).
//  - One that does not is not cut below 32 rows, and planned for 40 KiB where that saves a quarter of the
//    workgroups, none are row blocks and F >= 128 (1000 graphs of 20-100 nodes at F = 128 13.2 / 11.8,
//    ranges of 16 rows at 20 KiB 16.1 / 11.8, uncut at 24 14.3 / 12.8; 400 of them at F = 256 10.6 / 8.8
//    against 11.6 / 10.4), for 20 KiB, eight workgroups per CU, where that holds all of it at once (no row
//    blocks) or costs at most a twentieth more of them (4096 molecules at
//    F = 64 11.4 / 10.4, 12.8 / 11.9 at 24), else for 24 (2048 molecules at F = 128 11.4 / 9.9 uncut, 12.6 /
//    10.0 in ranges of 16 rows; 300 random matrices of 3 entries a row 10.6 / 7.7 against 12.9 / 7.7).  Past
//    88 MB of dense input, where input and output no longer stay in the 256 MB memory-side cache
//    together: ranges of four passes at 24 KiB (4096 molecules at F = 256 38.6 / 38.5, uncut 40.9 / 39.9).
//  - From F = 256 on with operations in row blocks that do not: uncut tiles and row blocks of 128 columns (150
//    heavy-tailed graphs at F = 512 10.5 / 10.2, ranges of one pass at 20 KiB 12.0 / 7.7, 32 columns
//    11.1 / 10.4; 700 at F = 256 19.4 / 19.0, 26.2 / 17.8, 19.7 / 18.9; 100 random matrices 8.0 / 5.6, 9.5 /
//    5.2, 8.9 / 8.4), past 48 MB of dense input of 256 columns at 40 KiB (1024 heavy-tailed graphs 27.3 /
//    26.6, in 128 columns 27.9 / 27.9, cut to one pass 33.1 / 24.4).
//  - Row blocks past 104 MB fetch what they gather from memory again: uncut at 40 KiB where that saves
//    a third of the workgroups (3000 heavy-tailed graphs at F = 256 107 at 20 KiB, 76.5 at 24, 75.1; 10000
//    random matrices at F = 32 90 -> 76).
//  - Dense blocks that several operations read (edge types as channels): ranges of four passes at 24 KiB,
//    the tiles come out of L2 (900 molecules of four channels at F = 128 10.0 / 9.7, uncut 10.3 / 10.0).
//  - Widths of whole 128-byte lines that are no power of two (96, 160, 192): one tile of the whole row keeps
//    part of the lanes idle but copies and stages once, which wins in launches of several rounds that stay
//    in cache (3000 molecules at F = 192 24.1 / 19.6 uncut, tiles of 64 22.7 / 22.2).  Tiles that are powers
//    of two win past 88 MB (2500 graphs of 20-100 nodes 49.3 -> 44.9), and where most operations are too
//    large for the whole row anyway (400 of them 9.4 -> 8.8).
//  - Rows off the 128-byte lines (F = 100): column tiles share lines, so operations that need them at 24 KiB
//    get 40 once the launch does not fit the chip at once anyway, where that saves a quarter of the
//    tiles and none are row blocks, and ranges of four passes (2000 graphs of 20-100 nodes 26.1 / 20.4
//    against 40.0 / 39.7; 2000 molecules, of which few need it, 9.7 -> 11.0: not taken).
// narrow: the first candidate from which on all tiles are powers of two (-1: none); ops: operations of the batch.
template <typename CountFn, typename FitFn>
Shape plain_shape(const Knobs& kn, int F, const std::vector<int>& cand, int narrow, int ops, bool shared, CountFn count, FitFn fit,
                  int* uncut_wgs)
{
    Shape s = {0, 0, 0};
    const Count n = count(0, 0);
    s.wgs = *uncut_wgs = n.wgs;
    auto take = [&](size_t first, int cap, int most) {
        const int w = count(first, cap).wgs;
        if (w > most) return false;
        s = {first, cap, w};
        return true;
    };
    auto cut = [&](int cap) {
        take(s.chosen, cap, INT32_MAX);
        return s;
    };
    const bool small = n.tile_words <= 3500000;
    const bool streams = F >= 128 && n.in_words > 22000000;
    const bool lines = F % 32 == 0;
    if (lines && F > 64 && small && s.wgs <= kn.capacity_wgs && 2 * n.tile_words >= n.in_words) {
        const int last = (int)cand.size() - 1;
        if (n.row_blocks) fit(kn.lds_words, last);
        for (int c = last; c >= (n.row_blocks ? last : 0); --c)
            for (int rows : {32, 64}) {    // (a pass of 32 columns is 32 rows)
                const int cap = std::max(1, rows * cand[c] / 1024);
                const int w = count((size_t)c, cap).wgs;
                if (w <= kn.capacity_wgs) return {(size_t)c, cap, w};
            }
        if (!n.row_blocks) return s;
        fit(kn.lds_words, 0);
    }
    bool pow2 = narrow == 0;
    // (with row blocks past 40 MB, where they are the tail of the others: 1167 heavy-tailed graphs at F = 192 62.8 -> 51.0 us both
    // directions, 2700 at F = 96 79 -> 64, 486 random matrices at F = 192 59 -> 54; 208 of them, 23 MB, 21.2 -> 24.6; one graph
    // of 400 nodes among 3000 molecules at F = 192 40.0 -> 47.9, among 6000 at F = 96 42.2 -> 51.3)
    if (narrow > 0 && lines && n.row_blocks && n.in_words > 10000000 && one_tail(n, ops)) {
        pow2 = true;
        fit(kn.lds_words, narrow);
        s = {(size_t)narrow, 0, count((size_t)narrow, 0).wgs};
        *uncut_wgs = s.wgs;
    }
    if (narrow > 0 && lines && !small && !n.row_blocks) {
        const Count t = count((size_t)narrow, 0);
        if (streams || 4 * (int64_t)t.wgs <= 5 * (int64_t)n.wgs) {
            pow2 = true;
            s = {(size_t)narrow, 0, t.wgs};
            *uncut_wgs = t.wgs;
        }
    }
    if (n.row_blocks && lines && n.in_words > 26000000) {
        fit(40 * 1024 / 4, (int)s.chosen);
        if (3 * (int64_t)count(s.chosen, 0).wgs <= 2 * (int64_t)s.wgs) return cut(0);
        fit(kn.lds_words, (int)s.chosen);
    }
    if (n.row_blocks && pow2 && F >= 256) {
        if (n.in_words > 12000000) {
            fit(40 * 1024 / 4, 0);
            return cut(0);
        }
        while (cand[s.chosen] > 128 && s.chosen + 1 < cand.size()) ++s.chosen;
        fit(kn.lds_words, (int)s.chosen);
        return cut(8);
    }
    const int eight = 8 * kn.compute_units;            // (other widths: the kernel's registers allow six)
    if (s.wgs <= kn.capacity_wgs) {
        if (!small || take(s.chosen, 1, kn.capacity_wgs) || take(s.chosen, 2, kn.capacity_wgs)) return s;
        if (!pow2) take(s.chosen, 4, kn.capacity_wgs);
        return s;
    }
    auto saves_at_40 = [&] {
        fit(40 * 1024 / 4, (int)s.chosen);
        if (4 * (int64_t)count(s.chosen, 0).wgs <= 3 * (int64_t)s.wgs) return true;
        fit(kn.lds_words, (int)s.chosen);
        return false;
    };
    if (!pow2 && !lines && !n.row_blocks) saves_at_40();
    if (streams || (shared && F >= 128)) return cut(4);
    if (!pow2) return cut(lines && F > 128 ? 8 : 4);
    if (F >= 128 && !n.row_blocks && saves_at_40()) return cut(0);
    fit(20 * 1024 / 4, (int)s.chosen);
    const int w20 = count(s.chosen, 0).wgs;
    const bool more = 20 * (int64_t)w20 > 21 * (int64_t)s.wgs;
    if (more && (w20 > eight || n.row_blocks)) fit(kn.lds_words, (int)s.chosen);
    if (w20 > eight || (more && n.row_blocks)) return cut(8);
    s.wgs = w20;
    for (int c : {2, 4, 8})
        if (32 * c >= cand[s.chosen] && take(s.chosen, c, eight - eight / 8)) break;
    return s;
}

// The plain batch - every operation an output block of its own, no forced bins, no sub-workgroup slots,
// nothing riding along - straight to the compact item table.  A data loader plans a batch per step,
// so this is on its critical path: no item is written twice, ordering and placement work on
// groups of items, and counting is closed form (128 molecules at F = 128: 33 us before, 10 now).
// Returns false when the batch needs the general planner below.
bool plain_schedule(const DirOps& o, int F, const Knobs& kn, int vec, const std::vector<int>& cand, Schedule& s)
{
    const int n = o.size();
    const int nc = (int)cand.size();
    if (nc > 64) return false;
    constexpr int64_t kLimit = (int64_t)1 << 31;       // the table's 32-bit fields
    for (int i = 0; i < n; ++i)
        if (o.rpt_off[i] >= kLimit || o.nz_off[i] >= kLimit || o.in_off[i] >= kLimit || o.out_off[i] >= kLimit)
            return false;

    // per candidate: its full tiles and the rest of the columns (width, columns of tiles, rows per pass
    // of a row in four-float lanes and of a long row in one-float lanes), words from row to row in LDS
    struct Columns {
        int width = 0, sh = 0, rows[2] = {1, 1};
        bool pow2 = true;
        explicit Columns(int w = 0) : width(w)
        {
            if (w <= 0) return;
            const int v = w >> 2;
            pow2 = w % 4 == 0 && v > 0 && v <= 64 && (v & (v - 1)) == 0;
            while ((4 << sh) < w) ++sh;
            rows[0] = std::max(1, kThreads / ((w + 3) / 4));
            rows[1] = std::max(1, kThreads / w);
        }
    };
    struct Tile {
        Columns full, tail;
        int nfull, stride;
    } tile[64];
    for (int c = 0; c < nc; ++c)
        tile[c] = {Columns(cand[c]), Columns(F % cand[c]), F / cand[c], tile_stride(cand[c], vec == 4)};
    // the widest candidate each operation can hold in LDS (nc: none, it is cut into row blocks)
    std::vector<uint8_t> fit(n);
    int lds_words = kn.lds_words;
    int blocks = 0;                                    // the candidate whose columns row blocks take ...
    int generic_rows = kn.generic_rows;                // ... and their rows
    auto fit_all = [&](int words, int block_tile) {
        lds_words = words;
        blocks = block_tile;
        // what the workgroup has in flight (2000 heavy-tailed graphs at F = 64: 16.8 us with eight rows, half
        // of the lanes idle, 15.7 with sixteen), sixty-four at most
        if (!kn.generic_given) generic_rows = std::max(kn.generic_rows, std::min(tile[blocks].full.rows[0], 64));
        for (int i = 0; i < n; ++i) {
            const int64_t room = words - ((int64_t)round_up(o.m[i] + 1, 2) + 2 * (int64_t)o.nnz[i] + 3) / 4 * 4 -
                                 (vec == 4 ? 0 : 4);   // (as fits_slot())
            int c = 0;
            while (c < nc && (int64_t)o.k[i] * tile[c].stride > room) ++c;
            fit[i] = (uint8_t)c;
        }
    };
    fit_all(kn.lds_words, 0);
    auto long_rows = [&](int i) { return vec == 1 && o.nnz[i] > kLongRow * o.m[i] ? 1 : 0; };
    // (exact below 2^31: x + 1/2 over d is at least 1/(2d) away from a whole number)
    auto pieces_of = [](int m, double inv_chunk, int chunk) { return (int)((m + chunk - 0.5) * inv_chunk); };
    auto count = [&](size_t first, int cap) {
        int chunk[64][2][2];
        double inv[64][2][2];
        for (int c = (int)first; c < nc && cap > 0; ++c)
            for (int l = 0; l < 2; ++l) {
                chunk[c][0][l] = cap * tile[c].full.rows[l], chunk[c][1][l] = cap * tile[c].tail.rows[l];
                for (int t = 0; t < 2; ++t) inv[c][t][l] = 1.0 / chunk[c][t][l];
            }
        Count t = {0, 0, false, 0, 0, 0};
        int64_t k_sum = 0;
        for (int i = 0; i < n; ++i) {
            const int m = o.m[i];
            if (m <= 0) continue;
            t.in_words += o.k[i];
            const int c = std::max((int)first, (int)fit[i]);
            if (c >= nc) {
                t.wgs += (tile[blocks].nfull + (tile[blocks].tail.width > 0)) * ((m + generic_rows - 1) / generic_rows);
                t.row_blocks = true;
                ++t.blocked;
                t.blocked_words += (int64_t)o.k[i] * F;
                continue;
            }
            const Tile& x = tile[c];
            if (cap <= 0) {
                t.wgs += x.nfull + (x.tail.width > 0);
                k_sum += o.k[i];
                continue;
            }
            const int l = long_rows(i);
            const int pf = x.nfull * pieces_of(m, inv[c][0][l], chunk[c][0][l]);
            const int pt = x.tail.width > 0 ? pieces_of(m, inv[c][1][l], chunk[c][1][l]) : 0;
            t.wgs += pf + pt;
            t.tile_words += (int64_t)o.k[i] * (pf * x.full.width + pt * x.tail.width);
        }
        t.tile_words += k_sum * F;
        t.in_words *= F;
        return t;
    };
    const std::vector<int> unit_of = input_blocks(o);
    int units = 0;
    bool in_order = true;
    for (int i = 0; i < n; ++i) {
        units = std::max(units, unit_of[i] + 1);
        in_order = in_order && (i == 0 || unit_of[i] >= unit_of[i - 1]);
    }
    const bool open = vec == 4 && kn.lds_words == Knobs().lds_words && !kn.lds_given && !kn.target_given && kn.wg_passes == 0;
    int narrow = -1;
    for (int c = std::min(nc, 2) - 1; c >= 0; --c)
        if (tile[c].full.pow2 && tile[c].tail.pow2) narrow = c;
    Shape shape = open ? plain_shape(kn, F, cand, narrow, n, 2 * units <= n, count, fit_all, &s.uncut_wgs)
                       : search_shape(kn, vec, (size_t)nc, count);
    // Longer row blocks where the launch does not fit the chip: from 24 rows on, four passes at most, no more than
    // make it seven eighths.  Where most of the dense input belongs to row blocks, whose gathers want every workgroup
    // there can be, two passes, if it then fits.  Not past 104 MB of dense input (48 at 40 KiB), which bounds either, nor
    // below F = 64 (a pass has 32 rows; 600 graphs at F = 32 9.1 -> 10.1).  us, both directions, operands from memory,
    // before / after, heavy-tailed graphs: 1333 at F = 64 24.8 / 22.2; 500 at F = 128 20.7 / 16.1, 2700 82.8 / 75.0; 240 at
    // F = 256 20.2 / 15.9; 200 at F = 512 27.2 / 25.5; 66 at F = 1024 20.7 / 16.1.  Random matrices of three entries a row
    // (most of the input in row blocks): 160 at F = 128 13.8 / 11.3, 41 at F = 512 13.9 / 11.3; four passes where two
    // do not fit lose: 100 at F = 512 23.8 -> 29.1.
    // Only where the large operations are the tail of the others, no more than six times their columns on average: a few
    // giants among small ones lose (30 of 500 rows among 400 of 60 at F = 128 15.8 -> 20.6, 60 of 400 among 1500 of 40 31.2
    // -> 37.5, 100 of 250 to 500 among 3000 molecules 47 -> 52), nor where the launch is between seven eighths of the chip
    // and all of it (239 heavy-tailed graphs at F = 128 11.3 -> 12.2).  A block's entries take half of the LDS on average:
    // what does not fit is read from memory entry by entry (60 of 400 rows of 60 entries among 1500 of 40 at F = 64 46
    // -> 80), and blocks of more entries are fewer workgroups than the gathers want (30 of 500 rows of 100 37 -> 44.6).
    const int short_rows = generic_rows;
    auto block_rows = [&](int i, int rows) {
        return std::min((int64_t)rows, std::max((int64_t)short_rows, (int64_t)lds_words / 2 * o.m[i] / (o.m[i] + 2 * (int64_t)o.nnz[i]) / 8 * 8));
    };
    if (open && F % 4 == 0 && F >= 64) {
        std::vector<int> blocked;
        Count t = {0, 0, true, 0, 0, 0};
        for (int i = 0; i < n; ++i) {
            t.in_words += (int64_t)o.k[i] * F;
            if (o.m[i] <= 0 || std::max((int)shape.chosen, (int)fit[i]) < nc) continue;
            blocked.push_back(i);
            t.blocked_words += (int64_t)o.k[i] * F;
        }
        t.blocked = (int)blocked.size();
        auto pieces = [&](int rows) {
            int64_t w = 0;
            for (int i : blocked) w += (o.m[i] + block_rows(i, rows) - 1) / block_rows(i, rows);
            return (int)w * (tile[blocks].nfull + (tile[blocks].tail.width > 0));
        };
        const int others = shape.wgs - pieces(generic_rows), most = std::min(64, 4 * tile[blocks].full.rows[0]);
        const int chip = tile[blocks].full.pow2 ? kMaxLdsBytes / 4 / lds_words * kn.compute_units : kn.capacity_wgs;
        const int room = 7 * (kMaxLdsBytes / 4 / lds_words) * kn.compute_units / 8;
        const int passes2 = std::min(64, 2 * tile[blocks].full.rows[0]);
        if (kn.generic_given || blocked.empty() || generic_rows >= 24 || shape.wgs <= chip || !one_tail(t, n)) {
        } else if (2 * t.blocked_words > t.in_words) {
            if (generic_rows < 16 && others + pieces(passes2) <= kn.capacity_wgs) generic_rows = std::max(generic_rows, passes2);
        } else if (t.in_words <= (lds_words > kn.lds_words ? 12000000 : 26000000)) {
            generic_rows = std::max(generic_rows, std::min(24, most));
            while (generic_rows + 8 <= most && others + pieces(generic_rows) > room) generic_rows += 8;
        }
        shape.wgs = others + pieces(generic_rows);
    }
    if (!open) s.uncut_wgs = shape.wgs;

    // A unit is a dense block and the operations that read it; the items of a unit that read the same
    // dense tile are a group and go to one XCD (rows that are no whole number of 128-byte lines: the
    // whole unit, because column tiles share the lines at their edges - 900 operations of 1 to 220 rows
    // at F = 127 fetched 122 MB and wrote 60 MB instead of 50 each, and took 34 us instead of 22, with
    // the tiles of an operation on different XCDs).
    const int columns = F % 32 != 0 ? std::max(4, F) : std::max(4, std::min(cand.back(), F));   // of a group
    std::vector<int32_t> first((size_t)units + 1, 0), member(in_order ? 0 : n);   // the operations of every unit
    for (int i = 0; i < n; ++i) ++first[unit_of[i] + 1];
    for (int u = 0; u < units; ++u) first[u + 1] += first[u];
    if (!in_order) {
        std::vector<int32_t> at(first.begin(), first.end() - 1);
        for (int i = 0; i < n; ++i) member[at[unit_of[i]]++] = i;
    }
    // bytes an item of one row range moves (as item_cost(), the entries spread evenly over the ranges)
    auto ranges_of = [](int m, int chunk) { return chunk >= m ? 1 : (int)((unsigned)(m + chunk - 1) / (unsigned)chunk); };
    auto chunk_of = [&](int i, const Columns& y, bool staged) {
        return !staged ? (int)block_rows(i, generic_rows) : (shape.cap > 0 ? shape.cap * y.rows[long_rows(i)] : o.m[i]);
    };
    auto cost_of = [&](int i, const Columns& y, int chunk, int ranges, bool staged) {
        const int nrows = std::min(chunk, o.m[i]);
        const int64_t entries = ranges == 1 ? o.nnz[i] : (unsigned)o.nnz[i] / (unsigned)ranges;
        const int64_t dense_in = staged ? o.k[i] : entries;      // (a row block gathers a row per entry)
        return 4 * (int64_t)y.width * (dense_in + nrows) + 8 * entries + 4 * (int64_t)nrows + 512;
    };
    auto choice_of = [&](int i) { return std::max((int)shape.chosen, (int)fit[i]); };
    std::vector<int64_t> cost((size_t)units, 0);
    for (int i = 0; i < n; ++i) {
        if (o.m[i] <= 0) continue;
        const int c = choice_of(i);
        const bool staged = c < nc;
        const Columns& y = tile[staged ? c : blocks].full;
        const int chunk = chunk_of(i, y, staged);
        cost[unit_of[i]] = std::max(cost[unit_of[i]], cost_of(i, y, chunk, ranges_of(o.m[i], chunk), staged));
    }
    std::vector<int32_t> order;
    largest_first(cost.data(), units, order);

    // units largest first: the groups of a unit go to neighbouring XCDs, from the one with the least
    // cost so far on (halves or quarters of the eight where the groups are four or two: the loads of a
    // half stay level); list x of the eight occupies workgroups x, x + 8, x + 16, ...
    static_assert(kXcds == 8, "the minimum below is a tree over eight loads");
    uint64_t load[kXcds];                             // cost so far << 3 | list: one minimum, no branches
    for (int x = 0; x < kXcds; ++x) load[x] = (uint64_t)x;
    int32_t used[kXcds] = {0};
    // Launches of many rounds at narrow widths are bound by the rate at which workgroups start (about
    // one a nanosecond): operations of at most two passes of a wavefront share a workgroup, one
    // wavefront each (16000 molecules at F = 16: 17.7 us one to a workgroup, 13.4 packed).
    std::vector<int32_t> packed;
    const bool pack = shape.wgs > 8 * kn.compute_units && tile[0].full.pow2 && tile[0].nfull == 1 && tile[0].tail.width == 0;
    const int wave_rows = pack ? 2 * 64 / (tile[0].full.width / 4) : 0;
    s.compact.resize((size_t)round_up(shape.wgs + shape.wgs / 8 + 64, kXcds));
    s.item_op.assign(s.compact.size(), -1);
    bool all_pow2 = vec == 4;
    int64_t lds = 0;
    auto item_of = [&](int i, bool staged) {
        LeanItem t = {};
        t.rpt_off = (uint32_t)o.rpt_off[i];
        t.nz_off = (uint32_t)o.nz_off[i];
        t.in_row = (uint32_t)o.in_off[i];
        t.out_row = (uint32_t)o.out_off[i];
        t.m = o.m[i], t.k = o.k[i], t.nnz = o.nnz[i];
        if (staged) {
            const int cv = round_up(t.m + 1, 2);
            t.cv_byte = 4 * cv;
            t.b_byte = 4 * round_up(cv + 2 * t.nnz, 4);
        }
        return t;
    };
    for (int32_t u : order) {
        const uint64_t la = std::min(std::min(load[0], load[1]), std::min(load[2], load[3]));
        const uint64_t lb = std::min(std::min(load[4], load[5]), std::min(load[6], load[7]));
        const int start = (int)(std::min(la, lb) & 7);
        for (int32_t j = first[u]; j < first[u + 1]; ++j) {
            const int i = in_order ? j : member[j];
            const int m = o.m[i];
            if (m <= 0) continue;
            const int c = choice_of(i);
            const bool staged = c < nc;
            const Tile& x = tile[staged ? c : blocks];
            if (m <= wave_rows && c == 0 && 4 * any_words(m, o.k[i], o.nnz[i], F, true) <= lds_words) {
                packed.push_back(i);
                continue;
            }
            LeanItem t = item_of(i, staged);
            if (staged) {
                lds = std::max(lds, any_words(m, t.k, t.nnz, x.nfull > 0 ? x.full.width : x.tail.width, vec == 4));
            } else {
                s.row_blocks = true;
            }
            const int groups = columns >= F ? 1 : x.nfull + (x.tail.width > 0);   // of this operation
            const int base = groups == 4 || groups == 2 ? start & ~(groups - 1) : start;
            const int next = columns >= F ? 0 : 1;
            int group = 0;
            const Columns* last = nullptr;
            int chunk = 0, ranges = 0;
            uint64_t here = 0;
            for (int f0 = 0; f0 < F; f0 += x.full.width, group += next) {
                const Columns& y = F - f0 >= x.full.width ? x.full : x.tail;
                if (&y != last) {
                    last = &y;
                    chunk = chunk_of(i, y, staged);
                    ranges = ranges_of(m, chunk);
                    here = (uint64_t)cost_of(i, y, chunk, ranges, staged) * (uint64_t)ranges << 3;
                    all_pow2 = all_pow2 && y.pow2;
                    t.sh = y.sh;
                    // bit 0: no other item reads the tile
                    const bool once = ranges == 1 && first[u + 1] - first[u] == 1 && (F % 32 == 0 || y.width == F);
                    t.flags = y.width << 8 | (staged ? (once ? 1 : 0) : 2);
                    t.tile_vecs = staged ? t.k << y.sh : 0;
                }
                const int list = (base + group) & 7;
                load[list] += here;
                size_t at = (size_t)used[list] * kXcds + (size_t)list;
                used[list] += ranges;
                if ((size_t)used[list] * kXcds > s.compact.size()) {
                    s.compact.resize(2 * (size_t)used[list] * kXcds);
                    s.item_op.resize(s.compact.size(), -1);
                }
                t.f0 = f0;
                for (int r0 = 0; r0 < m; r0 += chunk, at += kXcds) {
                    t.row0 = r0;
                    t.nrows = std::min(chunk, m - r0);
                    s.compact[at] = t;
                    s.item_op[at] = i;
                }
                s.count += ranges;
                s.items_in_bin[staged ? BSPMM_BIN_WORKGROUP : BSPMM_BIN_GENERIC] += ranges;
            }
        }
    }
    const int whole = kXcds * *std::max_element(used, used + kXcds);
    const int groups = ((int)packed.size() + kWaves - 1) / kWaves, grid = whole + groups;
    s.compact.resize((size_t)grid + packed.size());
    s.item_op.resize((size_t)grid + packed.size());
    for (int x = 0; x < kXcds; ++x)                   // the ends of the shorter lists: empty items
        for (int at = used[x] * kXcds + x; at < whole; at += kXcds) s.compact[at] = LeanItem();
    for (int j = 0; j < (int)packed.size(); ++j) {    // behind the launch's own items: the packed ones
        const int i = packed[j];
        LeanItem t = item_of(i, true);
        t.nrows = t.m;
        t.sh = tile[0].full.sh;
        t.tile_vecs = t.k << t.sh;
        t.flags = F << 8 | (first[unit_of[i] + 1] - first[unit_of[i]] == 1 ? 1 : 0);
        s.compact[grid + j] = t;
        s.item_op[grid + j] = i;
        lds = std::max(lds, kWaves * (int64_t)round_up((int)any_words(t.m, t.k, t.nnz, F, true), 4));
    }
    for (int g = 0; g < groups; ++g) {
        LeanItem t = {};
        t.flags = 8;
        t.tile_vecs = grid + g * kWaves;
        t.count = std::min(kWaves, (int)packed.size() - g * kWaves);
        s.compact[whole + g] = t;
        s.item_op[whole + g] = -1;
    }
    s.count += (int)packed.size();
    s.items_in_bin[BSPMM_BIN_WAVE] += (int)packed.size();
    s.tile = cand[shape.chosen];
    s.grid = s.launch_grid = grid;
    for (int r = 0; r < kRanges; ++r) s.wg_end[r] = grid;   // (the compact table's launches do not ask)
    s.whole = grid > 0;
    s.pow2 = s.whole && all_pow2;
    s.budget_words = lds_words;
    s.lds_words = s.row_blocks ? lds_words : (int)std::min<int64_t>(lds_words, round_up((int)lds, 64));
    return true;
}

}  // namespace

// Workgroups per CU a launch aims for.  Plain products: four (their time is latency).  The
// fused front stages X_i again for every feature tile, so it wants fewer, wider tiles the
// wider the layer input is: two per CU measured best up to 64 input columns, one from 128 on.
int workgroups_per_cu(int front)
{
    return front <= 0 ? 4 : (front < 128 ? 2 : 1);
}

Knobs resolve_knobs(const bspmm_options* o)
{
    Knobs k;
    if (!o) return k;
    if (o->force_bin > 0 && o->force_bin <= BSPMM_NUM_BINS) k.force_bin = o->force_bin - 1;
    if (o->lds_bytes > 0) k.lds_words = std::min(o->lds_bytes, kMaxLdsBytes) / 256 * 64;
    if (k.lds_words < 256) k.lds_words = 256;
    if (o->max_tile > 0) k.max_tile = std::min(std::max(o->max_tile, 4), 256) / 4 * 4;
    if (o->min_tile > 0) k.min_tile = k.min_odd_tile = std::min(std::max(o->min_tile, 4), k.max_tile);
    if (o->compute_units > 0) k.compute_units = o->compute_units;
    k.target_given = o->target_workgroups > 0;
    k.target_wgs = o->target_workgroups > 0 ? o->target_workgroups
                                            : workgroups_per_cu(o->front_features) * k.compute_units;
    if (o->lds_pad > 0) k.pad = std::min(o->lds_pad, 64) / 4 * 4;
    if (o->lds_pad < 0) k.pad = 0;
    if (o->max_passes > 0) k.max_passes = o->max_passes;
    if (o->generic_rows > 0) k.generic_rows = std::min(o->generic_rows, kThreads - 1);   // (a row pointer per lane)
    k.generic_given = o->generic_rows > 0;
    k.wg_passes = o->wg_passes;
    if (o->resident_workgroups > 0) k.persistent_wgs = o->resident_workgroups;
    k.hubs = (o->flags & BSPMM_SPLIT_HUB_ROWS) != 0;
    k.accumulate = (o->flags & BSPMM_ACCUMULATE) != 0;
    k.coo_direct = (o->flags & BSPMM_COO_DIRECT) != 0;
    k.symmetric = (o->flags & BSPMM_SYMMETRIC) != 0;
    k.one_front_launch = (o->flags & BSPMM_ONE_FRONT_LAUNCH) != 0;
    k.lds_given = o->lds_bytes > 0;
    if (o->front_features > 0) {   // the matrix-core blocks of the fused front are 16 columns wide
        k.front = o->front_features;
        // an item also holds X_i and a weight tile: take half the CU's LDS unless told otherwise
        // (the launch asks only for what its largest item needs)
        if (o->lds_bytes <= 0) k.lds_words = kHalfLdsBytes / 4;
        k.max_tile = std::max(16, k.max_tile / 16 * 16);
        k.min_tile = o->min_tile > 0 ? std::min(std::max(16, (k.min_tile + 15) / 16 * 16), k.max_tile) : 16;
    }
    return k;
}

std::vector<bspmm_item> items_of(const Schedule& s, const ItemTable& compact)
{
    if (!s.view.empty()) return s.view;
    std::vector<bspmm_item> v;
    v.reserve((size_t)s.count);
    auto add = [&](size_t j, int bin, int workgroup, int slot) {
        const LeanItem& t = compact[j];
        v.push_back({s.item_op[j], bin, t.row0, t.nrows, t.f0, t.flags >> 8, workgroup, slot});
    };
    for (int j = 0; j < s.launch_grid; ++j) {
        const LeanItem& t = compact[(size_t)j];
        if (t.flags & 8)
            for (int w = 0; w < t.count; ++w) add((size_t)(t.tile_vecs + w), BSPMM_BIN_WAVE, j, w);
        else if (s.item_op[(size_t)j] >= 0)
            add((size_t)j, (t.flags & 2) ? BSPMM_BIN_GENERIC : BSPMM_BIN_WORKGROUP, j, 0);
    }
    return v;
}

Schedule make_schedule(const DirOps& ops_in, int F, const Knobs& kn_in)
{
    Schedule s;
    Knobs kn = kn_in;
    if (!kn_in.target_wgs) kn.target_wgs = 4 * kn.compute_units;
    s.budget_words = kn.lds_words;
    const int vec = (F % 4 == 0) ? 4 : 1;
    const std::vector<int> cand = tile_candidates(F, kn);
    const Groups outs = output_groups(ops_in);
    s.first_stand_in = ops_in.size();
    if (kn.front == 0 && kn.force_bin < 0 && !kn.hubs && kn.pad == 0 && kn.persistent_wgs == 0 &&
        !kn.wide_offsets && outs.size() == (int)outs.member.size() && plain_schedule(ops_in, F, kn, vec, cand, s))
        return s;

    // Sets of summed operations whose dense blocks are one block (the same one, or blocks that
    // lie back to back in the packed input): an operation with the members' matrices side by
    // side stands in for the set when it fits a staged workgroup item at the narrowest tile.
    DirOps ext;
    std::vector<int> stand_in(outs.size(), -1);
    {
        bool copied = false, narrow = false, apart = false;   // a set over the budget; one of scattered blocks
        for (int g = 0; g < outs.size(); ++g) {
            const int cnt = outs.count(g);
            if (cnt < 2 || cnt > kMaxMembers || kn.force_bin == BSPMM_BIN_GENERIC) continue;
            const int* mem = outs.begin(g);
            // the members' dense blocks, each counted once in member order, must lie back to
            // back: laid end to end they are then one block of the packed input as it stands
            bool one_block = true;
            int64_t nnz = 0, rows = 0;
            for (int j = 0; j < cnt; ++j) {
                nnz += ops_in.nnz[mem[j]];
                bool seen = false;
                for (int e = 0; e < j && !seen; ++e)
                    seen = ops_in.in_off[mem[e]] == ops_in.in_off[mem[j]] && ops_in.k[mem[e]] == ops_in.k[mem[j]];
                if (kn.front > 0) {
                    // fused front: the channels of a set share the layer input X_i, and each
                    // makes a dense tile of its own from it (X_i W[ch] + bias[ch]) on chip:
                    // the tiles are side by side by construction
                    one_block = one_block && (j == 0 || seen);
                    rows += ops_in.k[mem[j]];
                    continue;
                }
                if (seen) continue;
                one_block = one_block && ops_in.in_off[mem[j]] == ops_in.in_off[mem[0]] + rows;
                rows += ops_in.k[mem[j]];
            }
            if (!one_block || nnz > INT32_MAX || rows > INT32_MAX) {
                apart = true;
                continue;
            }
            if (!copied) {
                ext = ops_in;
                copied = true;
            }
            const int v = ext.size();
            ext.m.push_back(ops_in.m[mem[0]]);
            ext.k.push_back((int32_t)rows);
            ext.nnz.push_back((int32_t)nnz);
            ext.rpt_off.push_back(0);       // the merged arrays are placed by the caller
            ext.nz_off.push_back(0);
            ext.in_off.push_back(ops_in.in_off[mem[0]]);
            ext.out_off.push_back(ops_in.out_off[mem[0]]);
            if (kn.front > 0) {
                ext.chan.resize(ext.size(), 1);
                ext.chan.back() = cnt;
            }
            if (stand_in_tile(ext, v, F, vec, cand, kn) > 0) {
                stand_in[g] = v;
                s.merged_sets.push_back(outs.members(g));
            } else {   // take it back: the set runs as a fused task (or does not fit at all)
                narrow = true;
                if (kn.whole_sets) break;
                ext.m.pop_back(), ext.k.pop_back(), ext.nnz.pop_back(), ext.rpt_off.pop_back();
                ext.nz_off.pop_back(), ext.in_off.pop_back(), ext.out_off.pop_back();
                if (!ext.chan.empty()) ext.chan.pop_back();
            }
        }
        if (narrow && kn.whole_sets) {
            s.error = BSPMM_ETOOBIG;
            return s;
        }
        // One set over the default budget takes the whole launch to the general kernel, its fused tasks with
        // narrow tiles that each stage the set's merged CSR again.  Where 40 KiB hold every set the launch
        // runs from compact items instead: us, four channels with dense blocks of their own, molecules: 300
        // graphs at F = 64 4.9 -> 3.6, 512 at F = 128 9.7 -> 7.0, at F = 50 9.5 -> 5.1, 2048 at F = 64 14.7
        // -> 12.7, at F = 128 24.6 -> 23.9; three channels, 1000 graphs at F = 128 11.9 -> 10.5.  Past 128 MB
        // of dense input memory bounds either (2048 graphs of four channels at F = 256, 210 MB: 46.5 before,
        // 48.5 at 40 KiB).
        if (narrow && !apart && kn.front == 0 && kn.force_bin < 0 && !kn.lds_given && kn.lds_words == Knobs().lds_words) {
            int64_t in_rows = 0;
            for (int i = 0; i < ops_in.size(); ++i) in_rows += ops_in.k[i];
            if (in_rows * F <= 32000000) {
                Knobs wide = kn_in;
                wide.lds_words = 40 * 1024 / 4;
                wide.capacity_wgs = std::min(kn.capacity_wgs, 4 * kn.compute_units);
                wide.whole_sets = true;
                Schedule t = make_schedule(ops_in, F, wide);
                // Options that keep a launch from compact items leave it to the general kernel, where 40 KiB are
                // the better budget too but for columns off 16 bytes (four channels, split hub rows, at 24 /
                // 40 KiB: 300 graphs at F = 64 4.7 / 4.2, at F = 128 5.9 / 6.7, 512 at F = 128 9.0 / 8.2, 2048 at F = 64
                // 13.8 / 13.3, 1000 of three at F = 128 11.0 / 10.8; 512 at F = 50 8.3 / 9.9, with lds_pad 7.7 / 8.9).
                if (!t.error && (t.whole || F % 4 == 0)) return t;
            }
        }
    }
    s.first_stand_in = ops_in.size();
    // the whole layer per item: M channels make M times the matrix-core work of a plain front
    // item, so the launch wants M times the workgroups (128 graphs of 4 channels, n_X = 64:
    // 15.5 us at 512 workgroups, 11.7 us at 1024)
    if (kn.front > 0 && !s.merged_sets.empty() && !kn.target_given)
        kn.target_wgs *= (int)s.merged_sets[0].size();
    const DirOps& ops = s.merged_sets.empty() ? ops_in : ext;

    // widest batch-wide tile that still gives the launch enough workgroups
    std::vector<Draft> d;
    const bool allow_small = kn.force_bin >= 0 && kn.front == 0;   // sub-workgroup slots: forced bins only
    size_t most_members = 1;
    for (int g = 0; g < outs.size(); ++g) most_members = std::max<size_t>(most_members, outs.count(g));
    if (most_members > (size_t)kMaxMembers) {
        s.error = BSPMM_ETOOBIG;
        return s;
    }
    bool fits = true;
    int64_t counted_tile_words = 0;
    std::vector<uint8_t> widest_fit(ops.size(), (uint8_t)std::min<size_t>(cand.size(), 255));
    if (kn.front == 0 && kn.force_bin < 0 && cand.size() < 255)
        for (int i = 0; i < ops.size(); ++i)
            for (size_t c = 0; c < cand.size(); ++c)
                if (fits_slot(ops, i, cand[c], F, vec, kThreads, 0, kn)) {
                    widest_fit[i] = (uint8_t)c;
                    break;
                }
    const std::vector<uint8_t>* fit_table = kn.front == 0 && kn.force_bin < 0 && cand.size() < 255 ? &widest_fit : nullptr;
    auto workgroups_of = [&](size_t first, int cap) {
        Sink counter;
        draft_all(ops, F, vec, cand, first, kn, cap, allow_small, outs, stand_in, &fits, counter, fit_table);
        counted_tile_words = counter.tile_words;
        return counter.workgroups();
    };
    const Shape shape = search_shape(kn, vec, cand.size(), [&](size_t first, int cap) {
        const int w = workgroups_of(first, cap);
        return Count{w, counted_tile_words, false};
    });
    const size_t chosen = shape.chosen;
    const int cap = shape.cap, wgs = shape.wgs;
    s.tile = cand[chosen];
    if (!fits) {   // a set of summed operations does not fit LDS together even at 4 columns
        s.error = BSPMM_ETOOBIG;
        return s;
    }
    if (kn.front > 0) {   // every operation must hold its layer input on chip
        Sink probe;
        draft_all(ops, F, vec, cand, chosen, kn, cap, allow_small, outs, stand_in, &fits, probe, fit_table);
        if (probe.per_range[1] || probe.generic) {
            s.error = BSPMM_ETOOBIG;
            return s;
        }
    }
    // the draft that is kept
    const std::vector<int> block_of_op = input_blocks(ops);
    Sink keep;
    keep.out = &d;
    keep.block_of_op = &block_of_op;
    keep.tile_unit = std::max(4, std::min(cand.back(), F));
    keep.tiles_per_block = (F + keep.tile_unit - 1) / keep.tile_unit;
    // (fused front: every feature tile of an operation reads the whole of X_i.  Rows that are no whole
    // number of 128-byte lines: column tiles share the lines at their edges - 900 operations of 1 to 220
    // rows at F = 127 fetched 122 MB and wrote 60 MB instead of 50 each, and took 34 us instead of 22,
    // with the tiles of an operation on different XCDs.)
    if (kn.front > 0 || F % 32 != 0) {
        keep.tile_unit = std::max(4, F);
        keep.tiles_per_block = 1;
    }
    d.reserve((size_t)wgs * 4 + 16);
    draft_all(ops, F, vec, cand, chosen, kn, cap, allow_small, outs, stand_in, &fits, keep, fit_table);

    // group costs, for ordering and XCD placement
    int ngroups = 0;
    for (int bi : block_of_op) ngroups = std::max(ngroups, (bi + 1) * keep.tiles_per_block);
    for (Draft& x : d)
        if (x.fused >= 0) x.group = ngroups++;                // fused tasks stand alone
    std::vector<int64_t> gcost(ngroups, 0);
    std::vector<int> gsize(ngroups, 0);
    for (const Draft& x : d) {
        gcost[x.group] = std::max(gcost[x.group], x.cost);
        ++gsize[x.group];
    }
    for (Draft& x : d)
        if (x.fused < 0 && x.staged && gsize[x.group] == 1) x.staged |= 2;   // tile read once

    // Largest group first, members of a group together, larger items first inside a group,
    // equal keys in draft order.  The order only steers the greedy placement below, so costs
    // are compared in 15 and 16 bits (scaled to the largest): the three keys then pack into one
    // 55-bit word and a stable radix sort (11-bit digits: the counters stay in L1; digits that
    // are equal in every key are skipped) replaces the comparison sort, which was the most
    // expensive step of planning a large batch.
    std::vector<std::vector<int>> by_range(kRanges);
    {
        int64_t top = 1;
        for (int64_t c : gcost) top = std::max(top, c);
        int shift = 0;
        while ((top >> shift) > 0x7fff) ++shift;
        size_t n_in[kRanges] = {0, 0, 0, 0, 0};
        for (const Draft& x : d) n_in[draft_range(x)]++;
        std::vector<uint64_t> key[kRanges], key_tmp;
        std::vector<int> idx_tmp;
        for (int r = 0; r < kRanges; ++r) {
            key[r].reserve(n_in[r]);
            by_range[r].reserve(n_in[r]);
        }
        const bool packable = ngroups < (1 << 24);
        for (int idx = 0; idx < (int)d.size(); ++idx) {
            const Draft& x = d[idx];
            const int r = draft_range(x);
            const uint64_t g15 = 0x7fff - (uint64_t)(gcost[x.group] >> shift);
            const uint64_t c16 = 0xffff - (uint64_t)(std::min(x.cost, gcost[x.group]) >> shift << 1);
            key[r].push_back(g15 << 40 | (uint64_t)x.group << 16 | c16);
            by_range[r].push_back(idx);
        }
        uint32_t count[1 << 11];
        for (int r = 0; r < kRanges; ++r) {
            std::vector<uint64_t>& k = key[r];
            std::vector<int>& v = by_range[r];
            const size_t n = k.size();
            if (n < 2) continue;
            if (packable && n < 4096) {   // few items: the counters of a radix pass would outweigh them
                std::vector<std::pair<uint64_t, int>> kv(n);
                for (size_t t = 0; t < n; ++t) kv[t] = {k[t], v[t]};
                std::sort(kv.begin(), kv.end());     // (equal keys: by draft index, as the stable sort)
                for (size_t t = 0; t < n; ++t) v[t] = kv[t].second;
                continue;
            }
            if (!packable) {   // more groups than the key holds: compare
                std::vector<int> order(n);
                std::iota(order.begin(), order.end(), 0);
                std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
                    const Draft &x = d[v[a]], &y = d[v[b]];
                    if ((k[a] >> 40) != (k[b] >> 40)) return k[a] < k[b];
                    if (x.group != y.group) return x.group < y.group;
                    return (k[a] & 0xffff) < (k[b] & 0xffff);
                });
                std::vector<int> sorted(n);
                for (size_t t = 0; t < n; ++t) sorted[t] = v[order[t]];
                v.swap(sorted);
                continue;
            }
            key_tmp.resize(n);
            idx_tmp.resize(n);
            for (int pass = 0; pass < 5; ++pass) {
                const int sh = 11 * pass;
                std::fill(count, count + (1 << 11), 0u);
                for (size_t t = 0; t < n; ++t) ++count[(k[t] >> sh) & 0x7ff];
                if (count[(k[0] >> sh) & 0x7ff] == n) continue;   // one digit everywhere
                uint32_t run = 0;
                for (uint32_t& c : count) {
                    const uint32_t here = c;
                    c = run;
                    run += here;
                }
                for (size_t t = 0; t < n; ++t) {
                    const uint32_t at = count[(k[t] >> sh) & 0x7ff]++;
                    key_tmp[at] = k[t];
                    idx_tmp[at] = v[t];
                }
                k.swap(key_tmp);
                v.swap(idx_tmp);
            }
        }
    }

    // range 0: one item per workgroup; groups dealt to the XCD with the least cost so far,
    // then the eight lists interleaved so that list x occupies workgroups x, x+8, x+16, ...
    std::vector<std::vector<int>> xcd(kXcds);
    {
        int64_t load[kXcds] = {0};
        const std::vector<int>& v = by_range[0];
        for (auto& l : xcd) l.reserve(v.size() / kXcds + 64);
        size_t a = 0;
        while (a < v.size()) {
            size_t b = a;
            int64_t total = 0;
            while (b < v.size() && d[v[b]].group == d[v[a]].group) total += d[v[b++]].cost;
            const int x = (int)(std::min_element(load, load + kXcds) - load);
            for (size_t t = a; t < b; ++t) xcd[x].push_back(v[t]);
            load[x] += total;
            a = b;
        }
    }
    size_t longest = 0;
    for (auto& l : xcd) longest = std::max(longest, l.size());
    const int grid0 = (int)(longest * kXcds);

    // Optional persistent launch (off by default: the hardware dispatcher balances uneven
    // tasks better than a static stride): W workgroups take tasks w, w+W, ...  With the lists
    // sorted largest-first, every second round of W tasks is laid out backwards (in whole
    // groups of eight, so a task keeps its XCD) and the workgroup that drew the largest task
    // of one round draws the smallest of the next.
    bool slices = false;
    for (const Draft& x : d) slices = slices || x.bin == BSPMM_BIN_SLICE32 || x.bin == BSPMM_BIN_SLICE16;
    s.has_slices = slices;
    const int capacity = slices ? kn.capacity_wgs_slices : kn.capacity_wgs;
    const int W = std::max(kXcds, (kn.persistent_wgs > 0 ? kn.persistent_wgs : capacity) / kXcds * kXcds);
    const size_t per_round = (size_t)W / kXcds;
    for (auto& l : xcd) {
        l.resize(longest, -1);
        for (size_t a = per_round; kn.persistent_wgs > 0 && a < longest; a += 2 * per_round) {
            const size_t b = std::min(longest, a + per_round);
            std::reverse(l.begin() + a, l.begin() + b);
        }
    }

    // Whole layers in a launch of several rounds of workgroups, up to 64 input features: the
    // dense tiles are made in 32 x 32 blocks (half the LDS reads per flop, a quarter of the
    // blocks).  Measured on MI355X, four channels, F = 128: 2048 graphs 88 -> 79 us at
    // n_X = 32 and 130 -> 122 us at 64, 512 graphs 27.6 -> 25.6 and 35.8 -> 34.6 us; at
    // n_X = 128 it is 4 % slower, and a launch of one round (128 graphs) gains nothing.
    const bool wide_blocks = kn.front > 0 && kn.front <= 64 && wgs > 6 * kn.compute_units;
    auto emit = [&](int draft_idx, int wg, int slot) {
        const Draft& x = d[draft_idx];
        s.item_op.resize(s.items.size(), -1);      // empty items before this one
        s.items.push_back(to_item(ops, x));
        s.item_op.push_back(x.op);
        s.items_in_bin[x.bin]++;
        if (x.op < s.first_stand_in) {
            s.view.push_back({x.op, x.bin, x.row0, x.nrows, x.f0, x.fw, wg, slot});
        } else {   // a stand-in: the view lists the operations it stands for
            s.items.back().staged |= 4 | (kn.front > 0 ? ops.channels(x.op) << 8 : 0) | (wide_blocks ? 8 : 0);
            const std::vector<int>& mem = s.merged_sets[x.op - s.first_stand_in];
            for (size_t j = 0; j < mem.size(); ++j)
                s.view.push_back({mem[j], x.bin, x.row0, x.nrows, x.f0, x.fw, wg, (int)j});
        }
    };

    s.items.reserve(longest * kXcds + d.size() * (most_members > 1 ? most_members : 1) + 64);
    s.view.reserve(d.size() * (most_members > 1 ? most_members : 1));
    s.item_base[0] = 0;
    for (size_t pos = 0; pos < longest; ++pos)
        for (int x = 0; x < kXcds; ++x) {
            if (xcd[x][pos] >= 0)
                emit(xcd[x][pos], (int)(pos * kXcds + x), 0);
            else
                s.items.push_back(empty_item());
        }
    s.wg_end[0] = grid0;

    // range 1: fused tasks, `fused_stride` item slots each (the members, then empty items)
    int wg = grid0;
    {
        std::vector<std::vector<int>>& fused_sets = s.fused_sets;
        for (int g = 0; g < outs.size(); ++g)
            if (outs.count(g) > 1 && stand_in[g] < 0) fused_sets.push_back(outs.members(g));
        s.fused_stride = (int)most_members;
        s.item_base[1] = (int)s.items.size();
        for (int idx : by_range[1]) {
            const Draft& x = d[idx];
            const std::vector<int>& mem = fused_sets[x.fused];
            for (size_t j = 0; j < mem.size(); ++j) {
                Draft y = x;
                y.op = mem[j];
                WorkItem w = to_item(ops, y);
                size_t owner = j;
                for (size_t e = 0; e < j; ++e)
                    if (ops.in_off[mem[e]] == ops.in_off[mem[j]] && ops.k[mem[e]] == ops.k[mem[j]]) {
                        owner = e;
                        break;
                    }
                w.staged = 1 | (j == 0 ? (int)mem.size() << 8 : 0) | ((int)owner << 16);
                s.item_op.resize(s.items.size(), -1);
                s.items.push_back(w);
                s.item_op.push_back(y.op);
                s.view.push_back({y.op, BSPMM_BIN_WORKGROUP, x.row0, x.nrows, x.f0, x.fw, wg, (int)j});
                s.items_in_bin[BSPMM_BIN_WORKGROUP]++;
            }
            for (size_t j = mem.size(); j < most_members; ++j) s.items.push_back(empty_item());
            s.task_set.push_back(x.fused);
            ++wg;
            ++s.fused_tasks;
        }
        s.wg_end[1] = wg;
    }
    for (int r = 2; r < kRanges; ++r) {
        const int slots = kThreads >> range_log2_slot(r);
        s.item_base[r] = (int)s.items.size();
        const std::vector<int>& v = by_range[r];
        for (size_t t = 0; t < v.size(); ++t) emit(v[t], wg + (int)(t / slots), (int)(t % slots));
        const int nwg = (int)((v.size() + slots - 1) / slots);
        while ((int)s.items.size() < s.item_base[r] + nwg * slots) s.items.push_back(empty_item());
        wg += nwg;
        s.wg_end[r] = wg;
    }
    s.item_op.resize(s.items.size(), -1);
    s.count = (int)s.view.size();
    s.uncut_wgs = wg;
    s.grid = wg;
    s.launch_grid = kn.persistent_wgs > 0 ? std::min(wg, W) : wg;
    // Launches made only of whole-workgroup items (staged operations and row blocks of the generic
    // bin) run from the compact item table; the lean kernel serves those on the float4 path whose
    // tile rows are a power-of-two number of float4.
    s.whole = kn.pad == 0 && !kn.hubs && !kn.wide_offsets && kn.front == 0 && kn.persistent_wgs == 0 &&
              s.wg_end[0] == wg && wg > 0;
    s.pow2 = s.whole && vec == 4;
    for (const WorkItem& w : s.items) {
        if (!s.pow2) break;
        if (w.nrows <= 0) continue;
        const int nvec = w.fw >> 2;
        s.pow2 = (w.fw & 3) == 0 && nvec > 0 && (nvec & (nvec - 1)) == 0 && nvec <= 64;
    }
    if (s.whole) {   // what the launch asks for: its largest item's LDS (row blocks: the whole budget)
        int64_t most = 0;
        for (const WorkItem& w : s.items) {
            if (w.nrows <= 0) continue;
            most = std::max<int64_t>(most, (w.staged & 1) ? any_words(w.m, w.k, w.nnz, w.fw, vec == 4) : kn.lds_words);
        }
        s.lds_words = (int)std::min<int64_t>(kn.lds_words, round_up((int)most, 64));
    }
    if (kn.front > 0) {
        int64_t most = 0;
        for (const WorkItem& w : s.items) {
            if (w.nrows <= 0) continue;
            const StagedLayout L = staged_layout(w.m, w.k, w.nnz, w.fw, 0, false);
            const int ch = std::max(1, (w.staged >> 8) & 0xff);     // channels of a stand-in
            most = std::max<int64_t>(most, (int64_t)L.total + (int64_t)(w.k / ch) * kn.front +
                                               ch * ((int64_t)kn.front * w.fw + w.fw));
        }
        s.front_lds_words = (int)std::min<int64_t>(kn.lds_words, round_up((int)most, 64));
    }
    return s;
}

// Direct COO kernel (the resource assignment of Sec. IV-C for SparseTensor operands, cases 1-3):
// an item keeps its whole output tile in LDS.  Where they fit beside it, the operation's dense
// tile and its entries are staged in LDS too (one bulk copy instead of one round trip to
// memory per entry); an operation that is too large for that at the batch-wide tile takes a
// narrower tile of its own, and one that fits at no width keeps only the output tile (and
// the entries, if they fit) on chip and is cut into row ranges, each of which scans all of the
// operation's entries and keeps its own (the paper falls back to atomics on global memory
// there).  As for CSR, the batch-wide tile is the widest one that still gives the launch
// enough workgroups.
namespace {

constexpr int kCooSortedRows = 128;   // rows of an item that sorts its entries and reads dense rows from memory

struct CooChoice {
    int fw;      // tile width of this operation
    int nr;      // rows per item
    int mode;
};

CooChoice coo_choice(const DirOps& o, int i, int F, size_t first, const std::vector<int>& cand,
                     const Knobs& kn)
{
    const int64_t W = kn.lds_words;
    // entries sorted by row on chip and the rows summed in registers (no output tile, no
    // atomics): with the dense tile beside them at the widest tile that fits, else with the
    // dense rows read from memory at the batch-wide tile
    for (size_t c = first; c < cand.size(); ++c) {
        const int fw = std::min(cand[c], F);
        if (coo_lds_words(o.m[i], o.k[i], o.nnz[i], fw, 7) <= W) return {fw, o.m[i], 7};
    }
    {
        // the dense rows come from memory entry by entry: narrow tiles and short row ranges, so
        // that a workgroup has many rows in flight and few to go through one after another
        const int fw = std::min(cand.back(), F);
        const int nr = std::min(o.m[i], kCooSortedRows);
        if (coo_lds_words(nr, o.k[i], o.nnz[i], fw, 6) <= W) return {fw, nr, 6};
    }
    for (size_t c = first; c < cand.size(); ++c) {
        const int fw = std::min(cand[c], F);
        if (coo_lds_words(o.m[i], o.k[i], o.nnz[i], fw, 3) <= W) return {fw, o.m[i], 3};
    }
    const int fw = std::min(cand[first], F);
    const int64_t stride = round_up(fw, 4);
    const int64_t ent = 3 * (int64_t)o.nnz[i] + 1;
    if (ent + 16 * stride <= W)
        return {fw, (int)std::min<int64_t>(o.m[i], (W - ent) / stride), 2};
    return {fw, (int)std::min<int64_t>(o.m[i], std::max<int64_t>(1, W / stride)), 0};
}

}  // namespace

namespace {
CooSchedule coo_schedule_at(const DirOps& ops, int F, const Knobs& kn_in);
}

// Without a budget from the caller the launch gets the smallest of a few LDS sizes at which
// every operation is sorted on chip (or has its entries and both tiles there): an operation that
// falls through to the row-range forms goes over all of its entries once per range and holds the
// whole launch up.
CooSchedule make_coo_schedule(const DirOps& ops, int F, const Knobs& kn)
{
    if (kn.lds_given) return coo_schedule_at(ops, F, kn);
    CooSchedule s;
    for (int words : {6144, 8192, 12288, 16384}) {
        Knobs k2 = kn;
        k2.lds_words = words;
        s = coo_schedule_at(ops, F, k2);
        bool ranges = false;
        for (const CooItem& it : s.items) ranges = ranges || (!(it.mode & 4) && it.mode != 3);
        if (!ranges) break;
    }
    return s;
}

namespace {

CooSchedule coo_schedule_at(const DirOps& ops, int F, const Knobs& kn_in)
{
    CooSchedule s;
    Knobs kn = kn_in;
    if (!kn.target_wgs) kn.target_wgs = 4 * kn.compute_units;
    const std::vector<int> cand = tile_candidates(F, kn);
    auto count = [&](size_t first) {
        int64_t n = 0;
        for (int i = 0; i < ops.size(); ++i)
            if (ops.m[i] > 0) {
                const CooChoice ch = coo_choice(ops, i, F, first, cand, kn);
                n += (int64_t)((F + ch.fw - 1) / ch.fw) * ((ops.m[i] + ch.nr - 1) / ch.nr);
            }
        return n;
    };
    size_t first = cand.size() - 1;
    for (size_t c = 0; c < cand.size(); ++c)
        if (count(c) >= kn.target_wgs) {
            first = c;
            break;
        }
    s.tile = std::min(cand[first], F);
    struct Key { int64_t work; int idx; };
    std::vector<CooItem> raw;
    for (int i = 0; i < ops.size(); ++i) {
        if (ops.m[i] <= 0) continue;
        const CooChoice ch = coo_choice(ops, i, F, first, cand, kn);
        const int parts = (ops.m[i] + ch.nr - 1) / ch.nr;
        const int per = (ops.m[i] + parts - 1) / parts;
        for (int f0 = 0; f0 < F; f0 += ch.fw)
            for (int r0 = 0; r0 < ops.m[i]; r0 += per) {
                CooItem it{};
                it.nz_off = ops.nz_off[i];
                it.in_row_off = ops.in_off[i];
                it.out_row_off = ops.out_off[i];
                it.nnz = ops.nnz[i];
                it.k = ops.k[i];
                it.row0 = r0;
                it.nrows = std::min(per, ops.m[i] - r0);
                it.f0 = f0;
                it.fw = std::min(ch.fw, F - f0);
                it.op = i;
                it.mode = ch.mode;
                raw.push_back(it);
            }
    }
    std::vector<Key> order(raw.size());
    for (size_t j = 0; j < raw.size(); ++j)
        order[j] = {(int64_t)raw[j].fw * ((int64_t)raw[j].nnz * ((raw[j].mode & 1) ? 1 : 4) +
                                          2 * raw[j].nrows + raw[j].k), (int)j};
    std::stable_sort(order.begin(), order.end(),
                     [](const Key& a, const Key& b) { return a.work > b.work; });
    s.items.reserve(raw.size());
    s.view.reserve(raw.size());
    for (const Key& kx : order) {
        const CooItem& it = raw[kx.idx];
        bspmm_item v;
        v.op = it.op;
        v.bin = BSPMM_BIN_COO;
        v.row0 = it.row0;
        v.nrows = it.nrows;
        v.f0 = it.f0;
        v.fw = it.fw;
        v.workgroup = (int32_t)s.items.size();
        v.slot = it.mode;
        s.items.push_back(it);
        s.view.push_back(v);
        s.lds_words = (int)std::max<int64_t>(s.lds_words, coo_lds_words(it.nrows, it.k, it.nnz, it.fw, it.mode));
    }
    s.lds_words = std::min(kn.lds_words, round_up(s.lds_words, 64));
    return s;
}

}  // namespace

}  // namespace bspmm
