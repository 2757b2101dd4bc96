// Device kernels of libbspmm for gfx950 (wave64).
//
// bspmm_kernel      one launch computes every work item of a schedule: per item, stage the
//                   operation's CSR arrays and the feature tile of its dense input in LDS
//                   (or, for the generic bin, read them from global memory), then give every
//                   output row a group of lanes that accumulates its stored entries in
//                   registers and writes the row once (the row-wise, atomic-free product of
//                   Fig. 4, batched as in Sec. IV-C, with the column blocking of Fig. 5(d)).
// bspmm_lean_kernel the same product for launches made only of whole-workgroup items on the
//                   float4 path: items carry what the general kernel derives, the dense tile
//                   goes global -> LDS directly.
// bspmm_first_transposed_kernel  the first transposed product of a plan, which sorts the operations itself.
// bspmm_gcn_kernel  the fused front of the graph-convolution layer (Fig. 7): the dense tile is
//                   made on the matrix cores from the layer input and the weights, for one
//                   channel or for all channels of the layer, and gathered as above.
// bspmm_layer_kernel  the same layer from a few dozen graphs on, gather first: workgroups with the
//                   weights in registers make blocks of 16 to 64 output rows.
// bspmm_coo_kernel  the direct product for COO / SparseTensor operands (Fig. 3, Fig. 5(a,b)).
// build_sorted      stable CSR -> transposed CSR of every operation (counting sort by column),
//                   and COO / SparseTensor -> CSR (the same sort by row).
// merge_sets        merged CSR of operations that are summed into one output block.
// validate_csr      structural check of the device CSR arrays.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "plan.hpp"

namespace bspmm {

// ---------------------------------------------------------------------------------------
// small vector helpers
// ---------------------------------------------------------------------------------------
template <int VEC> struct Vec;
template <> struct Vec<4> {
    using type = float4;
    static __device__ __forceinline__ type zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
    static __device__ __forceinline__ void fma(type& acc, float a, const type& b)
    {
        acc.x = fmaf(a, b.x, acc.x);
        acc.y = fmaf(a, b.y, acc.y);
        acc.z = fmaf(a, b.z, acc.z);
        acc.w = fmaf(a, b.w, acc.w);
    }
};
template <> struct Vec<1> {
    using type = float;
    static __device__ __forceinline__ type zero() { return 0.f; }
    static __device__ __forceinline__ void fma(type& acc, float a, const type& b)
    {
        acc = fmaf(a, b, acc);
    }
};

template <int VEC>
__device__ __forceinline__ typename Vec<VEC>::type load_vec(const float* p)
{
    return *reinterpret_cast<const typename Vec<VEC>::type*>(p);
}
template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const typename Vec<VEC>::type& v)
{
    *reinterpret_cast<typename Vec<VEC>::type*>(p) = v;
}

// Output rows are written once and never read by this launch: a non-temporal store keeps
// them from displacing the dense blocks that the generic bin re-reads out of L2.
template <int VEC>
__device__ __forceinline__ void store_out(float* p, const typename Vec<VEC>::type& v)
{
    if constexpr (VEC == 4) {
        typedef float native4 __attribute__((ext_vector_type(4)));
        native4 n = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(n, reinterpret_cast<native4*>(p));
    } else {
        __builtin_nontemporal_store(v, p);
    }
}

__device__ __forceinline__ int ilog2(int pow2) { return 31 - __clz(pow2); }

// How the S lanes of a slot split into row groups for a tile of fw columns.
template <int S, int VEC>
struct Split {
    int g_lanes;   // lanes per row (power of two, <= S and <= 64)
    int groups;    // rows in flight
    int g;         // this lane's row group
    int l;         // this lane's position inside the group
    int nvec;      // vectors per tile row
    __device__ __forceinline__ Split(int fw, int lane)
    {
        int gl = lanes_per_row(fw, VEC);
        if (gl > S) gl = S;
        g_lanes = gl;
        const int sh = ilog2(gl);
        groups = S >> sh;
        g = lane >> sh;
        l = lane & (gl - 1);
        nvec = (fw + VEC - 1) / VEC;
    }
};

// ---------------------------------------------------------------------------------------
// staging: global -> LDS.  The three copies (row pointers, entries, dense tile) do not depend
// on each other, and none depends on the contents of the CSR arrays.  What decides the time
// of a small item is the number of global-memory round trips on its critical path, so the
// first trip of every copy is issued before anything is waited for: one round trip stages a
// typical molecule-sized item completely; larger items finish in unrolled leftover loops.
// ---------------------------------------------------------------------------------------
// (the pointer travels in the slot of the front's weights, which such launches do not have: a
// field of its own made the argument block longer and the headline launch 1 % slower)
__device__ __forceinline__ const int32_t* merged_words(const LaunchParams& P)
{
    return reinterpret_cast<const int32_t*>(P.w);
}

template <int S, int VEC, bool HUBS, bool WITH_TILE = true, bool MERGED = false>
__device__ __forceinline__ void stage_item(const LaunchParams& P, const WorkItem& it, int* sm,
                                           int lane)
{
    using VT = typename Vec<VEC>::type;
    const StagedLayout L = staged_layout(it.m, it.k, it.nnz, it.fw, P.pad, HUBS && S == kThreads);
    if (HUBS && S == kThreads && lane == 0) sm[L.hub_off] = 0;   // no hub row found yet
    // (MERGED kernels, bit 2 of `staged`: the item is a set of summed operations that read one
    // dense block, i.e. the product with the sum of their matrices; its CSR is the set's
    // merged one in the workspace - row pointers at rpt_off, columns at nz_off, values behind
    // the columns.  A template parameter, not a run-time test alone: the three selects cost
    // the plain kernel 2 % of the headline launch.)
    const bool merged = MERGED && (it.staged & 4) != 0;
    const int32_t* __restrict__ rp = (merged ? merged_words(P) : P.rpt) + it.rpt_off;
    const int32_t* __restrict__ ci = (merged ? merged_words(P) : P.colids) + it.nz_off;
    const float* __restrict__ va =
        merged ? reinterpret_cast<const float*>(merged_words(P) + it.nz_off + round_up(it.nnz, 4))
               : P.values + it.nz_off;
    int2* cv = reinterpret_cast<int2*>(sm + L.cv_off);
    float* bs = reinterpret_cast<float*>(sm + L.b_off);
    const float* __restrict__ src = P.in + it.in_row_off * P.ld_in + it.f0;
    const Split<S, VEC> sp(it.fw, lane);
    const int step = sp.groups;
    const int m = it.m, nnz = it.nnz, k = it.k;

    // ---- first trip of every copy: loads only
    // (unconditional, from a clamped index: a load inside a branch drags the first use of its
    // value, and with it a wait for the whole round trip, in front of the loads that follow)
    const int rv = rp[min(lane, m)];
    int c0 = 0, c1 = 0;
    float a0 = 0.f, a1 = 0.f;
    if (lane < nnz) {
        c0 = ci[lane];
        a0 = va[lane];
    }
    if (lane + S < nnz) {
        c1 = ci[lane + S];
        a1 = va[lane + S];
    }
    // Dense tile.  Fast path: when a tile row is a power-of-two number of float4 and rows are
    // packed without padding, whole wavefronts copy 1 KiB at a time straight from global
    // memory into LDS (lane i lands at base + 16*i): no staging registers, and the entire
    // tile is in flight at once instead of four rows per lane group.
    const bool direct = WITH_TILE && VEC == 4 && S >= 64 && P.pad == 0 && (sp.nvec & (sp.nvec - 1)) == 0;
    if (direct) {
        const int sh = ilog2(sp.nvec);
        const int total = k << sh;                       // float4 in the tile
        const int wl = lane & 63;
        for (int e0 = (lane >> 6) << 6; e0 < total; e0 += S) {
            const int e = e0 + wl;
            if (e < total) {
                const float* gp = src + (int64_t)(e >> sh) * P.ld_in + ((e & (sp.nvec - 1)) << 2);
                // a dense tile that no other item reads is streamed (non-temporal) so that it
                // does not displace data other workgroups re-read from L2
                if (it.staged & 2)
                    __builtin_amdgcn_global_load_lds(
                        (const void __attribute__((address_space(1)))*)gp,
                        (void __attribute__((address_space(3)))*)(bs + (e0 << 2)), 16, 0, 2);
                else
                    __builtin_amdgcn_global_load_lds(
                        (const void __attribute__((address_space(1)))*)gp,
                        (void __attribute__((address_space(3)))*)(bs + (e0 << 2)), 16, 0, 0);
            }
        }
    }
    const bool col_ok = WITH_TILE && !direct && sp.l < sp.nvec;
    const int r0 = sp.g, r1 = sp.g + step, r2 = sp.g + 2 * step, r3 = sp.g + 3 * step;
    const float* colp = src + sp.l * VEC;
    VT t0 = Vec<VEC>::zero(), t1 = Vec<VEC>::zero(), t2 = Vec<VEC>::zero(), t3 = Vec<VEC>::zero();
    if (WITH_TILE && !direct) {     // the same for every lane: a scalar branch over the whole path
        if (col_ok && r0 < k) t0 = load_vec<VEC>(colp + (int64_t)r0 * P.ld_in);
        if (col_ok && r1 < k) t1 = load_vec<VEC>(colp + (int64_t)r1 * P.ld_in);
        if (col_ok && r2 < k) t2 = load_vec<VEC>(colp + (int64_t)r2 * P.ld_in);
        if (col_ok && r3 < k) t3 = load_vec<VEC>(colp + (int64_t)r3 * P.ld_in);
    }

    // No use of a loaded value may be scheduled above this line: the wait in front of it would
    // hold back the loads that have not been issued yet and cost a second round trip.
    __builtin_amdgcn_sched_barrier(0);

    // ---- first trip: LDS writes.  Row pointers are clamped to [0, nnz] and columns to
    // [0, k) so that malformed arrays cannot make a lane leave its slot.
    if (lane <= m) sm[lane] = min(max(rv, 0), nnz);
    // (entries carry the word offset of their dense row in the tile, not the column itself:
    // the multiplication is done once here instead of by every lane that gathers the entry)
    if (lane < nnz)
        cv[lane] = make_int2((unsigned)c0 < (unsigned)k ? c0 * L.stride : 0, __float_as_int(a0));
    if (lane + S < nnz)
        cv[lane + S] = make_int2((unsigned)c1 < (unsigned)k ? c1 * L.stride : 0, __float_as_int(a1));
    float* bcol = bs + sp.l * VEC;
    if (WITH_TILE && !direct) {
        if (col_ok && r0 < k) store_vec<VEC>(bcol + r0 * L.stride, t0);
        if (col_ok && r1 < k) store_vec<VEC>(bcol + r1 * L.stride, t1);
        if (col_ok && r2 < k) store_vec<VEC>(bcol + r2 * L.stride, t2);
        if (col_ok && r3 < k) store_vec<VEC>(bcol + r3 * L.stride, t3);
    }

    // ---- leftovers of larger items (each behind a condition that is the same for every
    // lane, so that a small item jumps over them instead of walking through masked-off code)
    if (m >= S)
        for (int i = lane + S; i <= m; i += S) sm[i] = min(max(rp[i], 0), nnz);
    if (nnz > 2 * S)
    for (int p = lane + 2 * S; p < nnz; p += 2 * S) {
        const int q = p + S;
        const int cc0 = ci[p];
        const float aa0 = va[p];
        int cc1 = 0;
        float aa1 = 0.f;
        if (q < nnz) {
            cc1 = ci[q];
            aa1 = va[q];
        }
        cv[p] = make_int2((unsigned)cc0 < (unsigned)k ? cc0 * L.stride : 0, __float_as_int(aa0));
        if (q < nnz)
            cv[q] = make_int2((unsigned)cc1 < (unsigned)k ? cc1 * L.stride : 0, __float_as_int(aa1));
    }
    if (WITH_TILE && !direct)
    for (int v = sp.l; v < sp.nvec; v += sp.g_lanes) {
        const float* cp = src + v * VEC;
        float* bp = bs + v * VEC;
        for (int row = (v == sp.l ? sp.g + 4 * step : sp.g); row < k; row += 4 * step) {
            const int q1 = row + step, q2 = row + 2 * step, q3 = row + 3 * step;
            VT u0 = load_vec<VEC>(cp + (int64_t)row * P.ld_in);
            VT u1 = Vec<VEC>::zero(), u2 = Vec<VEC>::zero(), u3 = Vec<VEC>::zero();
            if (q1 < k) u1 = load_vec<VEC>(cp + (int64_t)q1 * P.ld_in);
            if (q2 < k) u2 = load_vec<VEC>(cp + (int64_t)q2 * P.ld_in);
            if (q3 < k) u3 = load_vec<VEC>(cp + (int64_t)q3 * P.ld_in);
            store_vec<VEC>(bp + row * L.stride, u0);
            if (q1 < k) store_vec<VEC>(bp + q1 * L.stride, u1);
            if (q2 < k) store_vec<VEC>(bp + q2 * L.stride, u2);
            if (q3 < k) store_vec<VEC>(bp + q3 * L.stride, u3);
        }
    }
}

// ---------------------------------------------------------------------------------------
// split-row reduce.  A hub row (hundreds of entries) would keep one lane group busy long after
// the rest of the workgroup has finished, so its entries are dealt out to ALL lane groups of
// the workgroup; each lane then holds a partial sum for its columns, and the partial sums of the
// groups are added up: inside a wavefront with DPP row rotations (distance < 16),
// ds_swizzle (16) and ds_bpermute (32), across the four wavefronts through one tile row of LDS
// each, in a fixed order (the result does not depend on timing).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float add_from_lane_xor(float v, int off)
{
    switch (off) {
        case 1: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));
        case 2: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));
        case 4: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
        case 8: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));
        case 16: return v + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), (16 << 10) | 0x1f));
        default: return v + __shfl_xor(v, 32);
    }
}

// Sum over the lane groups of one wavefront: afterwards every lane holds the total of the
// lanes that share its position inside a group (rotations by g, 2g, ... inside rows of 16
// lanes visit every group of the row; 16 and 32 are true exchanges).
template <int VEC>
__device__ __forceinline__ void wave_group_sum(typename Vec<VEC>::type& a, int g_lanes)
{
    for (int off = g_lanes; off < 64; off <<= 1) {
        if constexpr (VEC == 4) {
            a.x = add_from_lane_xor(a.x, off);
            a.y = add_from_lane_xor(a.y, off);
            a.z = add_from_lane_xor(a.z, off);
            a.w = add_from_lane_xor(a.w, off);
        } else {
            a = add_from_lane_xor(a, off);
        }
    }
}

// One hub row computed by the whole workgroup.  `load_entry(p)` yields (column, value) of entry
// p, `bcol` addresses this lane's vector of dense row 0, `stride` is the dense row stride.
// Contains two barriers: every lane of the workgroup must call it.
template <int VEC, typename Entry>
__device__ __forceinline__ void hub_row(int p0, int p1, Entry load_entry, const float* bcol,
                                        int64_t stride, bool col_ok, int g_lanes, int groups,
                                        int g, int l, float* scratch, int fwp, float* out_row)
{
    using V = Vec<VEC>;
    using VT = typename V::type;
    VT acc = V::zero();
    if (col_ok) {
        int p = p0 + g;
        for (; p + 3 * groups < p1; p += 4 * groups) {
            const int2 e0 = load_entry(p), e1 = load_entry(p + groups),
                       e2 = load_entry(p + 2 * groups), e3 = load_entry(p + 3 * groups);
            const VT b0 = load_vec<VEC>(bcol + e0.x * stride);
            const VT b1 = load_vec<VEC>(bcol + e1.x * stride);
            const VT b2 = load_vec<VEC>(bcol + e2.x * stride);
            const VT b3 = load_vec<VEC>(bcol + e3.x * stride);
            V::fma(acc, __int_as_float(e0.y), b0);
            V::fma(acc, __int_as_float(e1.y), b1);
            V::fma(acc, __int_as_float(e2.y), b2);
            V::fma(acc, __int_as_float(e3.y), b3);
        }
        for (; p < p1; p += groups) {
            const int2 e = load_entry(p);
            V::fma(acc, __int_as_float(e.y), load_vec<VEC>(bcol + e.x * stride));
        }
    }
    wave_group_sum<VEC>(acc, g_lanes);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) < g_lanes && col_ok) store_vec<VEC>(scratch + wave * fwp + l * VEC, acc);
    __syncthreads();
    if (threadIdx.x < g_lanes && col_ok) {
        VT t = load_vec<VEC>(scratch + l * VEC);
#pragma unroll
        for (int w = 1; w < kThreads / 64; ++w) {
            const VT u = load_vec<VEC>(scratch + w * fwp + l * VEC);
            if constexpr (VEC == 4) {
                t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
            } else {
                t += u;
            }
        }
        store_out<VEC>(out_row + l * VEC, t);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------------
// row gather-FMA from LDS and store
// ---------------------------------------------------------------------------------------
// `tile_shift` moves the dense tile behind a guest that sits at its usual place (the layer
// input of the fused front); ACC adds the sums to the output instead of overwriting it.
template <int S, int VEC, bool HUBS, bool ACC = false>
__device__ __forceinline__ void compute_staged(const LaunchParams& P, const WorkItem& it,
                                               int* sm, int lane, int tile_shift = 0)
{
    using V = Vec<VEC>;
    constexpr bool kHubs = HUBS && S == kThreads;
    const StagedLayout L = staged_layout(it.m, it.k, it.nnz, it.fw, P.pad, kHubs);
    const int2* cv = reinterpret_cast<const int2*>(sm + L.cv_off);
    const float* bs = reinterpret_cast<const float*>(sm + L.b_off + tile_shift);
    const Split<S, VEC> sp(it.fw, lane);
    float* __restrict__ dst = P.out + it.out_row_off * P.ld_out + it.f0;
    // hub rows need one vector per lane (always true on the float4 path)
    const bool hubs_on = kHubs && sp.nvec <= sp.g_lanes;
    const int hub_deg = max(kHubMin, kHubRatio * ((it.nnz + it.m - 1) / max(it.m, 1)));
    int* hub = sm + L.hub_off;

    const int row_end = it.row0 + it.nrows;
    for (int r = it.row0 + sp.g; r < row_end; r += sp.groups) {
        const int p0 = sm[r];
        const int p1 = sm[r + 1];
        if (hubs_on && p1 - p0 >= hub_deg) {
            // left to the whole workgroup.  The list has room for nnz / kHubMin rows, which is
            // all there can be when the row pointers are monotone; malformed ones (clamped, but
            // going up and down) could name more: those rows stay out of the list, and so
            // inside the item's LDS (their output is not written; the arrays were malformed).
            if (sp.l == 0) {
                const int slot = atomicAdd(&hub[0], 1);
                if (slot < it.nnz / kHubMin) hub[1 + slot] = r;
            }
            continue;
        }
        for (int v = sp.l; v < sp.nvec; v += sp.g_lanes) {
            const float* bcol = bs + v * VEC;
            typename V::type acc = V::zero();
            int p = p0;
            for (; p + 3 < p1; p += 4) {
                const int2 e0 = cv[p], e1 = cv[p + 1], e2 = cv[p + 2], e3 = cv[p + 3];
                const typename V::type b0 = load_vec<VEC>(bcol + e0.x);
                const typename V::type b1 = load_vec<VEC>(bcol + e1.x);
                const typename V::type b2 = load_vec<VEC>(bcol + e2.x);
                const typename V::type b3 = load_vec<VEC>(bcol + e3.x);
                V::fma(acc, __int_as_float(e0.y), b0);
                V::fma(acc, __int_as_float(e1.y), b1);
                V::fma(acc, __int_as_float(e2.y), b2);
                V::fma(acc, __int_as_float(e3.y), b3);
            }
            for (; p < p1; ++p) {
                const int2 e = cv[p];
                V::fma(acc, __int_as_float(e.y), load_vec<VEC>(bcol + e.x));
            }
            if constexpr (ACC) {
                static_assert(VEC == 4, "accumulating stores are built for the float4 path");
                const float4 old = load_vec<4>(dst + (int64_t)r * P.ld_out + v * VEC);
                acc.x += old.x;
                acc.y += old.y;
                acc.z += old.z;
                acc.w += old.w;
            }
            store_out<VEC>(dst + (int64_t)r * P.ld_out + v * VEC, acc);
        }
    }
    if constexpr (kHubs) {
        if (!hubs_on) return;          // uniform: depends on the item only
        __syncthreads();               // the hub list is complete
        const int n_hub = min(hub[0], it.nnz / kHubMin);
        const int fwp = round_up(it.fw, 4);
        float* scratch = reinterpret_cast<float*>(hub + round_up(1 + it.nnz / kHubMin, 4));
        for (int h = 0; h < n_hub; ++h) {
            const int r = hub[1 + h];
            hub_row<VEC>(sm[r], sm[r + 1], [cv](int p) { return cv[p]; }, bs + sp.l * VEC,
                         (int64_t)1 /* entries hold row offsets already */, sp.l < sp.nvec, sp.g_lanes, sp.groups, sp.g, sp.l,
                         scratch, fwp, dst + (int64_t)r * P.ld_out);
        }
    }
}

// Generic bin: the operation's dense tile does not fit LDS, so a row block gathers it from
// global memory (L2 keeps the block while the row blocks of one operation run on one XCD).
// Only the block's slice of the CSR arrays is staged, in two dependent steps (row pointers,
// then the entries they delimit); after that every gather of a row is independent and up to
// four are in flight per lane (deeper
// unrolling costs registers, hence occupancy, and measured slower).
template <int VEC, bool HUBS>
__device__ __forceinline__ void run_generic(const LaunchParams& P, const WorkItem& it, int* sm,
                                            int tid)
{
    using V = Vec<VEC>;
    using VT = typename V::type;
    const int32_t* __restrict__ rp = P.rpt + it.rpt_off + it.row0;
    const int32_t* __restrict__ ci = P.colids + it.nz_off;
    const float* __restrict__ va = P.values + it.nz_off;
    const int nrows = it.nrows;
    for (int i = tid; i <= nrows; i += kThreads) sm[i] = min(max(rp[i], 0), it.nnz);
    __syncthreads();
    const int pbeg = __builtin_amdgcn_readfirstlane(sm[0]);
    const int cnt = max(__builtin_amdgcn_readfirstlane(sm[nrows]) - pbeg, 0);
    const int cv_off = round_up(nrows + 1, 2);
    const int hub_off = round_up(cv_off + 2 * cnt, 4);
    const bool fits = hub_off + (HUBS ? hub_words(nrows, it.fw) : 0) <= P.lds_floats;
    int2* cv = reinterpret_cast<int2*>(sm + cv_off);
    int* hub = sm + hub_off;
    if (fits) {
        if (HUBS && tid == 0) hub[0] = 0;
        for (int p = tid; p < cnt; p += 2 * kThreads) {
            const int q = p + kThreads;
            const int c0 = ci[pbeg + p];
            const float a0 = va[pbeg + p];
            int c1 = 0;
            float a1 = 0.f;
            if (q < cnt) {
                c1 = ci[pbeg + q];
                a1 = va[pbeg + q];
            }
            cv[p] = make_int2((unsigned)c0 < (unsigned)it.k ? c0 : 0, __float_as_int(a0));
            if (q < cnt) cv[q] = make_int2((unsigned)c1 < (unsigned)it.k ? c1 : 0, __float_as_int(a1));
        }
    }
    __syncthreads();

    const Split<kThreads, VEC> sp(it.fw, tid);
    const float* __restrict__ src = P.in + it.in_row_off * P.ld_in + it.f0;
    float* __restrict__ dst = P.out + (it.out_row_off + it.row0) * P.ld_out + it.f0;
    const bool hubs_on = HUBS && fits && sp.nvec <= sp.g_lanes;
    const int hub_deg = HUBS ? max(kHubMin, kHubRatio * ((it.nnz + it.m - 1) / max(it.m, 1))) : 0;
    for (int i = sp.g; i < nrows; i += sp.groups) {
        const int p0 = sm[i] - pbeg;
        const int p1 = sm[i + 1] - pbeg;
        if (hubs_on && p1 - p0 >= hub_deg) {
            if (sp.l == 0) hub[1 + atomicAdd(&hub[0], 1)] = i;   // left to the whole workgroup
            continue;
        }
        for (int v = sp.l; v < sp.nvec; v += sp.g_lanes) {
            const float* bcol = src + v * VEC;
            VT acc = V::zero();
            for (int p = p0; p < p1; p += 4) {
                int cc[4];
                float aa[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = min(p + u, p1 - 1);
                    if (fits) {
                        const int2 e = cv[q];
                        cc[u] = e.x;
                        aa[u] = __int_as_float(e.y);
                    } else {
                        const int c = ci[pbeg + q];
                        cc[u] = (unsigned)c < (unsigned)it.k ? c : 0;
                        aa[u] = va[pbeg + q];
                    }
                    if (p + u >= p1) aa[u] = 0.f;
                }
                VT b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    b[u] = V::zero();
                    if (p + u < p1) b[u] = load_vec<VEC>(bcol + (int64_t)cc[u] * P.ld_in);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) V::fma(acc, aa[u], b[u]);
            }
            store_out<VEC>(dst + (int64_t)i * P.ld_out + v * VEC, acc);
        }
    }
    if (!HUBS || !hubs_on) return;     // uniform: depends on the item and its row pointers
    __syncthreads();                   // the hub list is complete
    const int n_hub = hub[0];
    const int fwp = round_up(it.fw, 4);
    float* scratch = reinterpret_cast<float*>(hub + round_up(1 + nrows, 4));
    for (int h = 0; h < n_hub; ++h) {
        const int i = hub[1 + h];
        hub_row<VEC>(sm[i] - pbeg, sm[i + 1] - pbeg, [cv](int p) { return cv[p]; },
                     src + sp.l * VEC, P.ld_in, sp.l < sp.nvec, sp.g_lanes, sp.groups, sp.g, sp.l,
                     scratch, fwp, dst + (int64_t)i * P.ld_out);
    }
}


// ---------------------------------------------------------------------------------------
// Fused task: M operations with the same output rows whose products are added up (the channel
// sum of the graph-convolution layer, Fig. 6 / Fig. 7) in registers, so the block is written
// once instead of M times and never read back.  The set runs from its merged CSR (built once
// per plan by merge_sets_kernel below): the task is then an ordinary staged item whose dense
// tile is the members' tiles laid end to end.  Everything goes straight from global memory
// into LDS, 16 bytes per lane (the merged arrays are the library's own: aligned and padded).
// ---------------------------------------------------------------------------------------
// `vecs` 16-byte vectors global -> LDS by the whole workgroup, 1 KiB per wavefront instruction.
__device__ __forceinline__ void wg_copy_vec4(const int32_t* src, int* dst_lds, int vecs, int wave,
                                             int wl)
{
    for (int e0 = wave << 6; e0 < vecs; e0 += kThreads) {
        const int e = e0 + wl;
        if (e < vecs)
            __builtin_amdgcn_global_load_lds(
                (const void __attribute__((address_space(1)))*)(src + 4 * e),
                (void __attribute__((address_space(3)))*)(dst_lds + 4 * e0), 16, 0, 0);
    }
}

template <int VEC>
__device__ __forceinline__ void run_fused(const LaunchParams& P, int* sm, int first_item,
                                          int task)
{
    using V = Vec<VEC>;
    using VT = typename V::type;
    const int tid = threadIdx.x;
    // ---- member descriptors: lane j of every wavefront fetches member j's item, so all of
    // them arrive in one round trip; the uniform code below picks a member's fields out of
    // the lanes with v_readlane (no scalar load and no LDS per member).  The task's own
    // fields are member 0's; its rpt_off, nz_off and nnz describe the merged CSR of the set.
    const int wl = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WorkItem mine = P.items[first_item + min(wl, P.fused_stride - 1)];
    auto lane_i32 = [](int v, int j) { return __builtin_amdgcn_readlane(v, j); };
    auto lane_i64 = [](int64_t v, int j) {
        const unsigned lo = __builtin_amdgcn_readlane((int)(v & 0xffffffff), j);
        const unsigned hi = __builtin_amdgcn_readlane((int)(v >> 32), j);
        return (int64_t)(((uint64_t)hi << 32) | lo);
    };
    const int nrows = lane_i32(mine.nrows, 0);
    if (nrows <= 0) return;
    const int staged0 = lane_i32(mine.staged, 0);
    const int m = lane_i32(mine.m, 0);
    const int fw = lane_i32(mine.fw, 0);
    const int f0 = lane_i32(mine.f0, 0);
    const int row0 = lane_i32(mine.row0, 0);
    const int nnz_sum = lane_i32(mine.nnz, 0);
    const int64_t out_row_off = lane_i64(mine.out_row_off, 0);
    const int members = (staged0 >> 8) & 0xff;
    const FusedLayout L = fused_layout(m, nnz_sum);
    const int stride = round_up(fw, 4);
    const Split<kThreads, VEC> sp(fw, tid);
    const bool direct = VEC == 4 && (sp.nvec & (sp.nvec - 1)) == 0;

    // ---- stage the merged CSR
    wg_copy_vec4(merged_words(P) + lane_i64(mine.rpt_off, 0), sm, L.rs >> 2, wave, wl);
    wg_copy_vec4(merged_words(P) + lane_i64(mine.nz_off, 0), sm + L.rs, L.entry_words >> 2, wave, wl);
    // ---- and the dense tile of every member that does not share an earlier member's
    int tile_off = L.tile_off;
    for (int j = 0; j < members; ++j) {
        const int owner = (lane_i32(mine.staged, j) >> 16) & 0xff;
        if (owner != j) continue;
        const int k = lane_i32(mine.k, j);
        float* bs = reinterpret_cast<float*>(sm + tile_off);
        const float* __restrict__ src = P.in + lane_i64(mine.in_row_off, j) * P.ld_in + f0;
        if (direct) {
            const int sh = ilog2(sp.nvec);
            const int total = k << sh;
            for (int e0 = wave << 6; e0 < total; e0 += kThreads) {
                const int e = e0 + wl;
                if (e < total)
                    __builtin_amdgcn_global_load_lds(
                        (const void __attribute__((address_space(1)))*)(
                            src + (int64_t)(e >> sh) * P.ld_in + ((e & (sp.nvec - 1)) << 2)),
                        (void __attribute__((address_space(3)))*)(bs + (e0 << 2)), 16, 0, 0);
            }
        } else {
            for (int v = sp.l; v < sp.nvec; v += sp.g_lanes)
                for (int row = sp.g; row < k; row += sp.groups)
                    store_vec<VEC>(bs + row * stride + v * VEC,
                                   load_vec<VEC>(src + (int64_t)row * P.ld_in + v * VEC));
        }
        tile_off += k * stride;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
    __syncthreads();

    // ---- rows of the sum: the plain gather loop over the merged CSR, one store per row
    const int* crpt = sm;
    const int2* cv = reinterpret_cast<const int2*>(sm + L.rs);
    const int row_end = row0 + nrows;
    float* __restrict__ dst = P.out + out_row_off * P.ld_out + f0;
    const float* tiles = reinterpret_cast<const float*>(sm + L.tile_off);
    for (int r = row0 + sp.g; r < row_end; r += sp.groups) {
        const int p1 = min(max(crpt[r + 1], 0), nnz_sum);     // malformed pointers stay bounded
        const int p0 = min(max(crpt[r], 0), p1);
        for (int v = sp.l; v < sp.nvec; v += sp.g_lanes) {
            const float* bcol = tiles + v * VEC;
            VT acc = V::zero();
            int p = p0;
            for (; p + 3 < p1; p += 4) {
                const int2 e0 = cv[p], e1 = cv[p + 1], e2 = cv[p + 2], e3 = cv[p + 3];
                const VT b0 = load_vec<VEC>(bcol + e0.x * stride);
                const VT b1 = load_vec<VEC>(bcol + e1.x * stride);
                const VT b2 = load_vec<VEC>(bcol + e2.x * stride);
                const VT b3 = load_vec<VEC>(bcol + e3.x * stride);
                V::fma(acc, __int_as_float(e0.y), b0);
                V::fma(acc, __int_as_float(e1.y), b1);
                V::fma(acc, __int_as_float(e2.y), b2);
                V::fma(acc, __int_as_float(e3.y), b3);
            }
            for (; p < p1; ++p) {
                const int2 e = cv[p];
                V::fma(acc, __int_as_float(e.y), load_vec<VEC>(bcol + e.x * stride));
            }
            store_out<VEC>(dst + (int64_t)r * P.ld_out + v * VEC, acc);
        }
    }
}

// Merged CSR of one set of summed operations (one workgroup per set, once per plan and
// direction): row r of the set = row r of member 0, then of member 1, ...; an entry becomes (row of the
// concatenated dense tiles, value).  Row pointers are clamped to the member's entry count and columns
// outside a member's tile point at its row 0, so malformed input cannot make the product leave its LDS.
__global__ void __launch_bounds__(kThreads)
merge_sets_kernel(const SetRecord* __restrict__ sets, const int32_t* __restrict__ rpt,
                  const int32_t* __restrict__ colids, const float* __restrict__ values,
                  int32_t* __restrict__ merged)
{
    __shared__ int partial[kThreads];
    const SetRecord& g = sets[blockIdx.x];
    const int tid = threadIdx.x;
    const int m = g.m, members = g.members;
    const int per = (m + kThreads - 1) / kThreads;
    const int r0 = min(m, tid * per), r1 = min(m, r0 + per);
    auto row_range = [&](int j, int r, int& a, int& b) {
        const int32_t* rp = rpt + g.rpt_off[j];
        b = min(max(rp[r + 1], 0), g.nnz[j]);
        a = min(max(rp[r], 0), b);
    };
    int sum = 0;
    for (int r = r0; r < r1; ++r)
        for (int j = 0; j < members; ++j) {
            int a, b;
            row_range(j, r, a, b);
            sum += b - a;
        }
    partial[tid] = sum;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {     // inclusive scan over the lanes' sums
        const int add = tid >= off ? partial[tid - off] : 0;
        __syncthreads();
        partial[tid] += add;
        __syncthreads();
    }
    int pos = partial[tid] - sum;
    int32_t* mr = merged + g.merged_rpt_off;
    int2* mc = reinterpret_cast<int2*>(merged + g.merged_nz_off);
    // plain sets (one dense block): an ordinary CSR, columns and values in arrays of their own
    int nnz_sum = 0;
    for (int j = 0; j < members; ++j) nnz_sum += g.nnz[j];
    int32_t* pc = merged + g.merged_nz_off;
    float* pv = reinterpret_cast<float*>(pc + round_up(nnz_sum, 4));
    for (int r = r0; r < r1; ++r) {
        mr[r] = pos;
        for (int j = 0; j < members; ++j) {
            int a, b;
            row_range(j, r, a, b);
            const int32_t* ci = colids + g.nz_off[j];
            const float* va = values + g.nz_off[j];
            for (int p = a; p < b; ++p) {
                const int c = ci[p];
                const int row = g.tile_row[j] + ((unsigned)c < (unsigned)g.k[j] ? c : 0);
                if (g.plain) {
                    pc[pos] = row;
                    pv[pos] = va[p];
                } else {
                    mc[pos] = make_int2(row, __float_as_int(va[p]));
                }
                ++pos;
            }
        }
    }
    if (tid == kThreads - 1) mr[m] = pos;
}

// What the blocks of bspmm_layer_kernel read, once per plan: one workgroup per graph writes, for its
// output rows and their channels, where the entries start, the entries (row of X, value) and the row of
// Y; the last graph's workgroup also writes the empty rows that fill the last block.  Row pointers are
// clamped and columns outside the matrix point at the graph's first row of X, so malformed input stays
// inside the graph's share of the arrays.
__global__ void __launch_bounds__(kThreads)
layer_rows_kernel(const LayerSet* __restrict__ sets, const OpRecord* __restrict__ ops, const int32_t* __restrict__ rpt,
                  const int32_t* __restrict__ colids, const float* __restrict__ values, int32_t* __restrict__ starts,
                  int2* __restrict__ entries, int32_t* __restrict__ out_rows)
{
    __shared__ int partial[kThreads];
    const LayerSet& g = sets[blockIdx.x];
    const int tid = threadIdx.x;
    const int M = g.channels, m = g.m;
    const int per = (m + kThreads - 1) / kThreads;
    const int r0 = min(m, tid * per), r1 = min(m, r0 + per);
    auto row_range = [&](int j, int r, int& a, int& b) {
        const OpRecord& o = ops[g.op[j]];
        const int32_t* rp = rpt + o.rpt_off;
        b = min(max(rp[r + 1], 0), o.nnz);
        a = min(max(rp[r], 0), b);
    };
    int sum = 0;
    for (int r = r0; r < r1; ++r)
        for (int j = 0; j < M; ++j) {
            int a, b;
            row_range(j, r, a, b);
            sum += b - a;
        }
    partial[tid] = sum;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {     // inclusive scan over the lanes' sums
        const int add = tid >= off ? partial[tid - off] : 0;
        __syncthreads();
        partial[tid] += add;
        __syncthreads();
    }
    const int end = g.first_entry + g.entries;
    int pos = g.first_entry + partial[tid] - sum;
    for (int r = r0; r < r1; ++r) {
        const int row = g.first_row + r;
        out_rows[row] = g.out_row + r;
        for (int j = 0; j < M; ++j) {
            const OpRecord& o = ops[g.op[j]];
            int a, b;
            row_range(j, r, a, b);
            const int32_t* ci = colids + o.nz_off;
            const float* va = values + o.nz_off;
            starts[(int64_t)row * M + j] = min(pos, end);
            for (int p = a; p < b; ++p, ++pos) {
                const int c = ci[p];
                if (pos < end)
                    entries[pos] = make_int2(g.in_row + ((unsigned)c < (unsigned)o.k ? c : 0), __float_as_int(va[p]));
            }
        }
    }
    // (fewer entries than announced, malformed row pointers only: the rest adds nothing)
    for (int p = g.first_entry + partial[kThreads - 1] + tid; p < end; p += kThreads) entries[p] = make_int2(g.in_row, 0);
    if (g.pad_rows >= 0) {
        const int last = g.first_row + m;
        for (int i = tid; i < g.pad_rows; i += kThreads) out_rows[last + i] = -1;
        for (int i = tid; i < g.pad_rows * M + 4; i += kThreads) starts[(int64_t)last * M + i] = end;
    }
}

// One task of a sub-workgroup range: 256/S slots, one staged item each.
template <int LOG2S, int VEC, bool HUBS>
__device__ __forceinline__ void run_slots(const LaunchParams& P, int* sm, int first_item)
{
    constexpr int S = 1 << LOG2S;
    const int tid = threadIdx.x;
    const int slot = tid >> LOG2S;
    const int lane = tid & (S - 1);
    int idx = first_item + slot;
    if (LOG2S == 6) idx = __builtin_amdgcn_readfirstlane(idx);   // uniform inside a wavefront
    const WorkItem it = P.items[idx];
    int* slot_sm = sm + slot * (P.lds_floats >> (8 - LOG2S));
    if (it.nrows > 0) stage_item<S, VEC, HUBS>(P, it, slot_sm, lane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
    __syncthreads();
    if (it.nrows > 0) compute_staged<S, VEC, HUBS>(P, it, slot_sm, lane);
}


// One launch runs the whole schedule.  By default the grid has one workgroup per task (the
// hardware dispatcher balances uneven tasks, largest first); when the plan asks for fewer
// resident workgroups, workgroup w takes tasks w, w + gridDim.x, ... and fetches the next
// item's descriptor while it processes the current one.  Tasks below wg_end[0] are one item
// for the whole workgroup (bins workgroup and generic), tasks below wg_end[1] add up several
// operations into one output block, later tasks hold 4, 8 or 16 items for 64-, 32- or 16-lane
// slots.
// SLICES = false leaves out the 32- and 16-lane slot code (per-lane item descriptors cost
// registers, hence occupancy); the host launches it for schedules without such items.
// HUBS = true adds the split-row path for hub rows (an option of the plan: it costs a
// register-limited occupancy step and LDS for the reduction, which plain batches do not need).
template <int VEC, bool SLICES, bool HUBS, bool MERGED = false>
__global__ void __launch_bounds__(kThreads) bspmm_kernel(const LaunchParams P)
{
    extern __shared__ __align__(16) int sm[];
    const int tid = threadIdx.x;
    const int stride = gridDim.x;
    int t = blockIdx.x;
    if (t < P.wg_end[0]) {
        WorkItem it = P.items[P.item_base[0] + t];   // uniform address: scalar loads
        for (;;) {
            const int tn = t + stride;
            const bool more = tn < P.wg_end[0];
            WorkItem nx = it;
            if (more) nx = P.items[P.item_base[0] + tn];
            if (it.nrows > 0) {
                if (it.staged) {
                    stage_item<kThreads, VEC, HUBS, true, MERGED>(P, it, sm, tid);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
                    __syncthreads();
                    compute_staged<kThreads, VEC, HUBS>(P, it, sm, tid);
                } else {
                    run_generic<VEC, HUBS>(P, it, sm, tid);
                }
            }
            t = tn;
            if (!more) break;
            __syncthreads();   // the next item overwrites the LDS this one was read from
            it = nx;
        }
    }
    for (; t < P.n_tasks; t += stride) {
        __syncthreads();
        if (t < P.wg_end[1]) {
            run_fused<VEC>(P, sm, P.item_base[1] + (t - P.wg_end[0]) * P.fused_stride, t);
        } else if (t < P.wg_end[2]) {
            run_slots<6, VEC, HUBS>(P, sm, P.item_base[2] + (t - P.wg_end[1]) * 4);
        } else if (SLICES) {
            if (t < P.wg_end[3])
                run_slots<5, VEC, HUBS>(P, sm, P.item_base[3] + (t - P.wg_end[2]) * 8);
            else
                run_slots<4, VEC, HUBS>(P, sm, P.item_base[4] + (t - P.wg_end[3]) * 16);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Lean launch.  When every task of a schedule is one staged workgroup item whose dense tile is
// a power-of-two number of float4 wide (molecule-sized batches: the launch fits the chip at
// once and its time is the life of a workgroup, a chain of short latencies), the launch runs
// this kernel instead of bspmm_kernel: the same staging and the same gather (Fig. 4 per row,
// batched as in Sec. IV-C, column blocking of Fig. 5(d)), with nothing on the path that such
// an item does not need.  The dense tile is requested first (it is the part that comes from
// HBM), every lane group asks for the row pointers of its own first row directly, so the first
// pass over the rows starts from registers instead of a dependent LDS read, and the address
// arithmetic of the copies is scalar wherever the item decides it.
// Results are bit for bit those of bspmm_kernel: same order of the additions inside a row.
// ---------------------------------------------------------------------------------------
// The second to fourth entry of a trip, of which `left` are the row's own: each is added by the lanes that
// still have one.  (Adding the others with value zero would make a NaN of an infinite b.)  The three
// sets of lanes are each part of the one before, so three compares that write the execution mask
// and one move that restores it do, instead of a compare and a select per entry.
__device__ __forceinline__ void add_rest(float4& acc, int left, float v1, const float4& b1, float v2,
                                         const float4& b2, float v3, const float4& b3)
{
    uint64_t lanes;
    asm("s_mov_b64 %[lanes], exec\n\t"
        "v_cmpx_lt_i32_e32 vcc, 1, %[left]\n\t"
        "v_fmac_f32_e32 %[x], %[v1], %[b1x]\n\t"
        "v_fmac_f32_e32 %[y], %[v1], %[b1y]\n\t"
        "v_fmac_f32_e32 %[z], %[v1], %[b1z]\n\t"
        "v_fmac_f32_e32 %[w], %[v1], %[b1w]\n\t"
        "v_cmpx_lt_i32_e32 vcc, 2, %[left]\n\t"
        "v_fmac_f32_e32 %[x], %[v2], %[b2x]\n\t"
        "v_fmac_f32_e32 %[y], %[v2], %[b2y]\n\t"
        "v_fmac_f32_e32 %[z], %[v2], %[b2z]\n\t"
        "v_fmac_f32_e32 %[w], %[v2], %[b2w]\n\t"
        "v_cmpx_lt_i32_e32 vcc, 3, %[left]\n\t"
        "v_fmac_f32_e32 %[x], %[v3], %[b3x]\n\t"
        "v_fmac_f32_e32 %[y], %[v3], %[b3y]\n\t"
        "v_fmac_f32_e32 %[z], %[v3], %[b3z]\n\t"
        "v_fmac_f32_e32 %[w], %[v3], %[b3w]\n\t"
        "s_mov_b64 exec, %[lanes]"
        : [x] "+v"(acc.x), [y] "+v"(acc.y), [z] "+v"(acc.z), [w] "+v"(acc.w), [lanes] "=&s"(lanes)
        : [left] "v"(left), [v1] "v"(v1), [b1x] "v"(b1.x), [b1y] "v"(b1.y), [b1z] "v"(b1.z), [b1w] "v"(b1.w),
          [v2] "v"(v2), [b2x] "v"(b2.x), [b2y] "v"(b2.y), [b2z] "v"(b2.z), [b2w] "v"(b2.w), [v3] "v"(v3),
          [b3x] "v"(b3.x), [b3y] "v"(b3.y), [b3z] "v"(b3.z), [b3w] "v"(b3.w)
        : "vcc");
}

__device__ __forceinline__ float4 gather_row(const int2* cv, const char* bcol, int p0, int p1)
{
    using V = Vec<4>;
    float4 acc = V::zero();
    // Four entries per trip, all their LDS reads in flight together, also on the last trip of
    // a row: an entry past the end reads the row's last one and is not added.
    const int last = p1 - 1;
    for (int p = p0; p < p1; p += 4) {
        const int2 e0 = cv[p], e1 = cv[min(p + 1, last)], e2 = cv[min(p + 2, last)],
                   e3 = cv[min(p + 3, last)];
        const float4 b0 = *reinterpret_cast<const float4*>(bcol + e0.x);
        const float4 b1 = *reinterpret_cast<const float4*>(bcol + e1.x);
        const float4 b2 = *reinterpret_cast<const float4*>(bcol + e2.x);
        const float4 b3 = *reinterpret_cast<const float4*>(bcol + e3.x);
        V::fma(acc, __int_as_float(e0.y), b0);
        add_rest(acc, p1 - p, __int_as_float(e1.y), b1, __int_as_float(e2.y), b2, __int_as_float(e3.y), b3);
    }
    return acc;
}

// The same sum with the dense rows gathered from global memory (L2): `cv` holds (byte offset
// of the dense row inside the operation's block, value), `src_l` addresses this lane's float4 of
// the block's first row.  Four independent gathers are in flight per lane (eight measured the
// same: the gathers of a large operation are bound by what the L2 delivers, not by latency).
__device__ __forceinline__ float4 gather_row_global(const int2* cv, const char* __restrict__ src_l,
                                                    int p0, int p1)
{
    using V = Vec<4>;
    float4 acc = V::zero();
    const int last = p1 - 1;
    for (int p = p0; p < p1; p += 4) {
        int2 e[4];
        float4 b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = cv[min(p + u, last)];
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = *reinterpret_cast<const float4*>(src_l + (uint32_t)e[u].x);
        V::fma(acc, __int_as_float(e[0].y), b[0]);
        add_rest(acc, p1 - p, __int_as_float(e[1].y), b[1], __int_as_float(e[2].y), b[2], __int_as_float(e[3].y),
                 b[3]);
    }
    return acc;
}

// Entries of a row block: its first one and how many, as its item has them.  The first run of a plan and
// direction (FIRST) finds them in the row pointers, a round trip to memory more, and leaves them in the item (a
// launch of its own for that cost a batch that is new every step 3.5 us of the host's time for each direction:
// 239 graphs of 8 to 500 nodes at F = 256 62.5 -> 57.5 us, 100 at F = 128 38 -> 33).  A kernel of its own: one that asks
// its items whether they have been filled in costs later runs 2 to 6 % (1333 graphs at F = 32 14.7 -> 15.6).
__device__ __forceinline__ int2 row_block_range(const LeanItem& it, const int32_t* __restrict__ rpt)
{
    const int32_t* __restrict__ rp = rpt + it.rpt_off + (uint32_t)it.row0;
    const int from = min(max(rp[0], 0), it.nnz), to = min(max(rp[it.nrows], 0), it.nnz);
    return make_int2(from, max(to - from, 0));
}

template <bool FIRST>
__device__ __forceinline__ int2 block_entries(const LeanItem& it, const LeanItem* item, const int32_t* __restrict__ rpt)
{
    if constexpr (!FIRST) return make_int2(it.tile_vecs, it.count);
    const int2 range = row_block_range(it, rpt);
    if (threadIdx.x == 0) {
        LeanItem* const mine = const_cast<LeanItem*>(item);
        mine->tile_vecs = range.x;
        mine->count = range.y;
    }
    return range;
}

// Row block of the generic bin in a lean launch.  ONE round trip to memory brings the block's
// row pointers and its entries: their position comes with the item (see block_entries), where
// bspmm_kernel needs the row pointers before it can ask for the entries.
// (Fetching the block's share of the dense rows into L2 ahead of the gathers was measured and
// changed nothing: the gathers are bound by L2 throughput.)
template <bool FIRST>
__device__ __forceinline__ void lean_row_block(const LeanItem& it, const LeanItem* item, int* sm,
                                               const int32_t* __restrict__ rpt,
                                               const int32_t* __restrict__ colids,
                                               const float* __restrict__ values,
                                               const float* __restrict__ in, float* __restrict__ out,
                                               uint32_t ld_in, uint32_t ld_out, uint32_t lds_words)
{
    const uint32_t tid = threadIdx.x;
    const int nrows = it.nrows, k = it.k, nnz = it.nnz;
    const int sh = it.sh;
    const uint32_t nvec = 1u << sh;
    const uint32_t l = tid & (nvec - 1), g = tid >> sh, groups = kThreads >> sh;
    const int2 range = block_entries<FIRST>(it, item, rpt);
    const int pbeg = min(max(range.x, 0), nnz);
    const int cnt = min(max(range.y, 0), nnz - pbeg);
    const uint32_t row_bytes = ld_in << 2;
    const char* __restrict__ src =
        reinterpret_cast<const char*>(in + ((uint64_t)it.in_row * ld_in + (uint32_t)it.f0));
    const int32_t* __restrict__ rp = rpt + it.rpt_off + (uint32_t)it.row0;
    const int32_t* __restrict__ ci = colids + it.nz_off + (uint32_t)pbeg;
    const float* __restrict__ va = values + it.nz_off + (uint32_t)pbeg;
    const uint32_t cv_off = (uint32_t)round_up(nrows + 1, 2);
    const bool fits = cv_off + 2u * (uint32_t)cnt <= lds_words;   // entries of the block in LDS
    int2* cv = reinterpret_cast<int2*>(sm + cv_off);

    // ---- requests
    const uint32_t ri = min(tid, (uint32_t)nrows);
    const int rv = rp[ri];
    const uint32_t last = (uint32_t)max(cnt - 1, 0);
    const uint32_t i0 = min(tid, last), i1 = min(tid + kThreads, last);
    int c0 = 0, c1 = 0;
    float a0 = 0.f, a1 = 0.f;
    if (fits && cnt > 0) {
        c0 = ci[i0];
        a0 = va[i0];
    }
    if (fits && cnt > kThreads) {
        c1 = ci[i1];
        a1 = va[i1];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- LDS writes (clamped as in the staged path)
    sm[ri] = min(max(rv, 0), nnz);
    if (fits && cnt > 0)
        cv[i0] = make_int2((unsigned)c0 < (unsigned)k ? (int)__umul24((uint32_t)c0, row_bytes) : 0, __float_as_int(a0));
    if (fits && cnt > kThreads)
        cv[i1] = make_int2((unsigned)c1 < (unsigned)k ? (int)__umul24((uint32_t)c1, row_bytes) : 0, __float_as_int(a1));
    if (fits && cnt > 2 * kThreads)
        for (int p = tid + 2 * kThreads; p < cnt; p += kThreads) {
            const int c = ci[p];
            cv[p] = make_int2((unsigned)c < (unsigned)k ? (int)__umul24((uint32_t)c, row_bytes) : 0,
                              __float_as_int(va[p]));
        }
    __syncthreads();

    // ---- rows
    const char* src_l = src + (l << 4);
    char* __restrict__ dst = reinterpret_cast<char*>(
        out + (((uint64_t)it.out_row + (uint32_t)it.row0) * ld_out + (uint32_t)it.f0));
    const uint32_t out_row_bytes = ld_out << 2;
    for (uint32_t i = g; i < (uint32_t)nrows; i += groups) {
        const int p1 = min(max(sm[i + 1] - pbeg, 0), cnt);
        const int p0 = min(max(sm[i] - pbeg, 0), p1);
        float4 acc;
        if (fits) {
            acc = gather_row_global(cv, src_l, p0, p1);
        } else {
            // a block whose entries do not fit LDS (rows of thousands of entries): entry by
            // entry from global memory, four gathers in flight
            acc = Vec<4>::zero();
            for (int p = p0; p < p1; p += 4) {
                int cc[4];
                float aa[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = min(p + u, p1 - 1);
                    const int c = ci[q];
                    cc[u] = (unsigned)c < (unsigned)k ? c : 0;
                    aa[u] = va[q];
                }
                float4 b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    b[u] = *reinterpret_cast<const float4*>(src_l + __umul24((uint32_t)cc[u], row_bytes));
                Vec<4>::fma(acc, aa[0], b[0]);
                add_rest(acc, p1 - p, aa[1], b[1], aa[2], b[2], aa[3], b[3]);
            }
        }
        store_out<4>(reinterpret_cast<float*>(dst + (__umul24(i, out_row_bytes) + (l << 4))), acc);
    }
}

// ---------------------------------------------------------------------------------------
// The lean launch for every other width and alignment (tile rows that are no power-of-two number
// of float4, F % 4 != 0, operands or leading dimensions off 16 bytes, offsets beyond 32 bits):
// the same items, the same order of the additions inside a row.
//
// Staging.  Instruction issue is what such a tile costs (a wavefront instruction takes four
// cycles): copied word by word it is 25 instructions per 256 bytes, and 900 operations of 1 to
// 220 rows at F = 127 spent half of their 33 us there.  So every row of the tile is copied as the
// 16-byte words of memory it lies in, 1 KiB per wavefront instruction, straight into LDS: its
// first column then sits zero to three words into the row's place, which an entry's offset
// takes into account.  A tile that is whole rows of a packed matrix is one run of memory and is
// copied as such.  Only a dense input that does not start on 16 bytes is copied word by word.
//
// Rows.  A row takes ceil(fw / 4) lanes of four floats, no power of two; the last lane stores what
// is left of the row.  The additions of a row are a serial chain of LDS reads, so rows of more than kLongRow
// entries on average are different.  Where they are fewer than the lane groups, the groups share a row's entries
// (any_long_rows): a row of 660 entries otherwise keeps a launch waiting for 4 us.  Off 16 bytes a read of four
// floats costs a CU as much as four reads of one and more: long rows take a lane per float there, unless that leaves half
// of the lanes idle and a row has 2 kSharedEntries entries on average; groups then share it, kSharedEntries each at least.
// us, both directions, a lane per float / four floats, shared from sixteen entries on / as it is: F = 127, 2000 operations of 4 to
// 40 rows of 20 entries 68 / 80 / 68, 1500 of 2 to 30 rows of 100 195 / 233 / 195, 800 of 1 to 120 rows of 20 119 / 137 / 120;
// F = 50, the same 36 / 39 / 36, 119 / 112 / 97, 89 / 85 / 69; F = 17, the last two 94 / 52 / 45, 71 / 33 / 33; F = 1, 5000 of
// 4 to 40 rows of 20 17.9 / 22.5 / 19.3.  On 16 bytes groups share from sixteen entries on: F = 100, 2000 of 4 to 40 rows of 20
// 64 / 33, 1500 of 100 154 / 67.
// Bound: small launches the chain of item, staging and gather, large ones memory (900 operations of 1 to
// 220 rows, F = 127: 100 MB in 22 us).  200 of them at F = 50: forward 15.9 -> 6.0 us, transposed 33 -> 6.5 us against
// the general kernel's scalar path.  Both directions with operations of one to three columns among them (rows of up to
// 660 entries in the transposed one), a lane per float / shared: 200 at F = 50 17.4 / 13.3, 800 32.7 / 27.5, 200 at F =
// 127 23.7 / 19.9, 800 at F = 17 18.9 / 14.0.
// ---------------------------------------------------------------------------------------
enum AnyMode {
    kAnyWindows = 1,   // the dense input starts on 16 bytes: rows are copied as 16-byte words
    kAnyTight = 2      // no room for such words beside a row (F % 4 == 0; windows then need ld_in % 4 == 0 too)
};

// n / d for 0 <= n < 2^21 and 1 <= d <= 256: (n + 1/2) / d is at least 1/512 away from a whole
// number, further than the three roundings reach.
__device__ __forceinline__ uint32_t div_small(uint32_t n, float inv_d)
{
    return (uint32_t)(((float)n + 0.5f) * inv_d);
}

template <int VEC> struct Floats { typedef float type __attribute__((ext_vector_type(VEC))); };
template <int VEC> struct FloatsAt4 { typedef float type __attribute__((ext_vector_type(VEC), aligned(4))); };

template <int VEC, bool ALIGNED>
__device__ __forceinline__ typename Floats<VEC>::type any_load(const void* p)
{
    using VT = typename Floats<VEC>::type;
    if constexpr (ALIGNED)
        return *reinterpret_cast<const VT*>(p);
    else
        return *reinterpret_cast<const typename FloatsAt4<VEC>::type*>(p);
}

// Sum of a row's entries [p0, p1): entry(p) gives (key, value), dense(key) this lane's floats of the
// entry's dense row.  N entries in flight while there are as many, then four at a time with the
// entries past the end left out (see gather_row).
template <int VEC, typename Entry, typename Dense>
__device__ __forceinline__ typename Floats<VEC>::type any_row(int p0, int p1, Entry entry, Dense dense)
{
    using VT = typename Floats<VEC>::type;
    constexpr int N = VEC == 4 ? 8 : 16;
    VT acc = 0.f;
    int p = p0;
    auto fma = [&](float a, const VT& b) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = fmaf(a, b[i], acc[i]);
    };
    for (; p + N <= p1; p += N) {
        int2 e[N];
        VT b[N];
#pragma unroll
        for (int u = 0; u < N; ++u) e[u] = entry(p + u);
#pragma unroll
        for (int u = 0; u < N; ++u) b[u] = dense(e[u].x);
#pragma unroll
        for (int u = 0; u < N; ++u) fma(__int_as_float(e[u].y), b[u]);
    }
    const int last = p1 - 1;
    for (; p < p1; p += 4) {
        int2 e[4];
        VT b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = entry(min(p + u, last));
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = dense(e[u].x);
        fma(__int_as_float(e[0].y), b[0]);
        if constexpr (VEC == 4) {
            auto f4 = [](const VT& v) { return make_float4(v[0], v[1], v[2], v[3]); };
            float4 sum = f4(acc);
            add_rest(sum, p1 - p, __int_as_float(e[1].y), f4(b[1]), __int_as_float(e[2].y), f4(b[2]),
                     __int_as_float(e[3].y), f4(b[3]));
            acc[0] = sum.x, acc[1] = sum.y, acc[2] = sum.z, acc[3] = sum.w;
        } else {
#pragma unroll
            for (int u = 1; u < 4; ++u) {
                const VT old = acc;
                fma(__int_as_float(e[u].y), b[u]);
                if (p + u >= p1) acc = old;
            }
        }
    }
    return acc;
}

// The lane's `n` floats of an output row (n < VEC on the last lane of a row only).  Rows off 16
// bytes share lines with their neighbours, so only aligned rows are stored past the caches.
template <int VEC, bool ALIGNED>
__device__ __forceinline__ void any_store(float* p, const typename Floats<VEC>::type& v, int n)
{
    if constexpr (VEC == 1) {
        *p = v[0];
    } else if constexpr (ALIGNED) {
        __builtin_nontemporal_store(v, reinterpret_cast<typename Floats<VEC>::type*>(p));
    } else if (n >= VEC) {
        *reinterpret_cast<typename FloatsAt4<VEC>::type*>(p) = v;
    } else {
        p[0] = v[0];
        if (n > 1) p[1] = v[1];
        if (n > 2) p[2] = v[2];
    }
}

// Rows [0, nrows) of an item in lanes of VEC floats: row(i, p0, p1) gives row i's entries, entry(p) the
// (key, value) of one, dense(key, l, n) the floats at l of the dense row it names, n of them in the row.
template <int VEC, bool ALIGNED, typename Row, typename Entry, typename Dense>
__device__ __forceinline__ void any_rows(uint32_t fw, int nrows, float* __restrict__ dst, int64_t ld_out, Row row,
                                         Entry entry, Dense dense)
{
    const uint32_t nvec = (fw + VEC - 1) / VEC, groups = kThreads / nvec;
    const uint32_t g = div_small(threadIdx.x, 1.f / (float)nvec), l = threadIdx.x - g * nvec;
    if (g >= groups) return;
    const int n = (int)(fw - VEC * l);
    float* p = dst + (g * ld_out + VEC * l);
    const int64_t step = groups * ld_out;
    for (int i = g; i < nrows; i += groups, p += step) {
        int p0, p1;
        row(i, p0, p1);
        any_store<VEC, ALIGNED>(p, any_row<VEC>(p0, p1, entry, [&](int key) {
            return dense.template operator()<VEC>(key, (int)(VEC * l), n);
        }), n);
    }
}

// The same for few long rows: `parts` lane groups share a row, each with its share of the entries, and the
// first of them adds up the partial sums, in order, from `sums` (LDS that nobody reads any more once the
// workgroup has met).  Every lane of the workgroup comes here; nrows parts <= groups of lanes.
template <bool ALIGNED, typename Row, typename Entry, typename Dense>
__device__ __forceinline__ void any_long_rows(uint32_t fw, int nrows, int parts, float* __restrict__ dst, int64_t ld_out,
                                              float4* sums, Row row, Entry entry, Dense dense)
{
    const uint32_t nvec = (fw + 3) / 4;
    const uint32_t g = div_small(threadIdx.x, 1.f / (float)nvec), l = threadIdx.x - g * nvec;
    const uint32_t i = div_small(g, 1.f / (float)parts), part = g - i * parts;
    const int n = (int)(fw - 4 * l);
    typename Floats<4>::type acc = 0.f;
    const bool mine = i < (uint32_t)nrows;
    if (mine) {
        int p0, p1;
        row((int)i, p0, p1);
        const float share = (float)(p1 - p0) / (float)parts;
        const int from = p0 + (int)(share * (float)part);
        const int to = part + 1 == (uint32_t)parts ? p1 : p0 + (int)(share * (float)(part + 1));
        acc = any_row<4>(from, to, entry, [&](int key) { return dense.template operator()<4>(key, (int)(4 * l), n); });
    }
    __syncthreads();
    float4* const at = sums + threadIdx.x;
    if (mine) *at = make_float4(acc[0], acc[1], acc[2], acc[3]);
    __syncthreads();
    if (!mine || part != 0) return;
    for (int s = 1; s < parts; ++s) {
        const float4 more = at[s * nvec];
        acc[0] += more.x, acc[1] += more.y, acc[2] += more.z, acc[3] += more.w;
    }
    any_store<4, ALIGNED>(dst + ((int64_t)i * ld_out + 4 * l), acc, n);
}

// Lane groups to a row of an item of long rows (`entries` in `rows` of them): what the workgroup has, up to sixteen,
// off 16 bytes with kSharedEntries each; one where the partial sums have no room in `bytes` of LDS.
template <bool ALIGNED>
__device__ __forceinline__ int long_row_parts(uint32_t fw, int nrows, int entries, int rows, int bytes)
{
    if (entries <= kLongRow * rows || (!ALIGNED && (entries < 2 * kSharedEntries * rows || 2 * nrows * (int)fw > kThreads)) || bytes < (int)(kThreads * sizeof(float4)))
        return 1;
    const uint32_t groups = kThreads / ((fw + 3) / 4), most = ALIGNED ? 16u : min((uint32_t)(entries / (kSharedEntries * max(rows, 1))), 16u);
    return (int)min(groups / (uint32_t)max(nrows, 1), most);
}

// A lane's floats out of the LDS tile (the last lane of a row may read up to three words past
// the row: LDS of this item) and out of global memory (nothing past the row's end is read).
template <bool ALIGNED> struct TileRows {
    const char* tile;
    template <int VEC> __device__ __forceinline__ typename Floats<VEC>::type operator()(int off, int l, int) const
    {
        return any_load<VEC, ALIGNED>(tile + off + 4 * l);
    }
};
template <bool ALIGNED> struct GlobalRows {
    const float* src;
    int64_t ld;
    template <int VEC> __device__ __forceinline__ typename Floats<VEC>::type operator()(int c, int l, int n) const
    {
        const float* p = src + (c * ld + l);
        if (ALIGNED || n >= VEC) return any_load<VEC, ALIGNED>(p);
        typename Floats<VEC>::type v = 0.f;
        v[0] = p[0];
        if constexpr (VEC == 4) {
            if (n > 1) v[1] = p[1];
            if (n > 2) v[2] = p[2];
        }
        return v;
    }
};

// Row block of the generic bin (see lean_row_block): dense rows gathered from global memory.
template <bool ALIGNED, bool FIRST>
__device__ __forceinline__ void any_row_block(const LeanItem& it, const LeanItem* item, int* sm,
                                              const int32_t* __restrict__ rpt,
                                              const int32_t* __restrict__ colids,
                                              const float* __restrict__ values, const float* __restrict__ in,
                                              float* __restrict__ out, int64_t ld_in, int64_t ld_out,
                                              uint32_t lds_words)
{
    const uint32_t tid = threadIdx.x;
    const int nrows = it.nrows, k = it.k, nnz = it.nnz;
    const uint32_t fw = max((uint32_t)it.flags >> 8, 1u);
    const int2 range = block_entries<FIRST>(it, item, rpt);
    const int pbeg = min(max(range.x, 0), nnz);
    const int cnt = min(max(range.y, 0), nnz - pbeg);
    const int32_t* __restrict__ rp = rpt + it.rpt_off + (uint32_t)it.row0;
    const int32_t* __restrict__ ci = colids + it.nz_off + (uint32_t)pbeg;
    const float* __restrict__ va = values + it.nz_off + (uint32_t)pbeg;
    const uint32_t cv_off = (uint32_t)round_up(nrows + 1, 2);
    const bool fits = cv_off + 2u * (uint32_t)cnt <= lds_words;
    int2* cv = reinterpret_cast<int2*>(sm + cv_off);
    for (int i = tid; i <= nrows; i += kThreads) sm[i] = min(max(rp[i], 0), nnz);
    auto global_entry = [&](int p) {
        const int c = ci[p];
        return make_int2((unsigned)c < (unsigned)k ? c : 0, __float_as_int(va[p]));
    };
    if (fits)
        for (int p = tid; p < cnt; p += kThreads) cv[p] = global_entry(p);
    __syncthreads();
    float* __restrict__ dst = out + (((int64_t)it.out_row + it.row0) * ld_out + it.f0);
    const GlobalRows<ALIGNED> dense = {in + ((int64_t)it.in_row * ld_in + it.f0), ld_in};
    auto row = [&](int i, int& p0, int& p1) {
        p1 = min(max(sm[i + 1] - pbeg, 0), cnt);
        p0 = min(max(sm[i] - pbeg, 0), p1);
    };
    auto lds_entry = [&](int p) { return cv[p]; };
    const uint32_t sums = (uint32_t)round_up((int)cv_off, 4);
    const int parts = fits ? long_row_parts<ALIGNED>(fw, nrows, cnt, nrows, 4 * ((int)lds_words - (int)sums)) : 1;
    if (!fits)
        any_rows<4, ALIGNED>(fw, nrows, dst, ld_out, row, global_entry, dense);
    else if (parts > 1)
        any_long_rows<ALIGNED>(fw, nrows, parts, dst, ld_out, reinterpret_cast<float4*>(sm + sums), row, lds_entry, dense);
    else if (!ALIGNED && cnt > kLongRow * nrows)
        any_rows<1, false>(fw, nrows, dst, ld_out, row, lds_entry, dense);
    else
        any_rows<4, ALIGNED>(fw, nrows, dst, ld_out, row, lds_entry, dense);
}

// mode: kAnyWindows, kAnyTight (ALIGNED implies both).
template <bool ALIGNED, bool FIRST = false>
__global__ void __launch_bounds__(kThreads)
bspmm_any_kernel(const LeanItem* __restrict__ items, const int32_t* __restrict__ rpt,
                 const int32_t* __restrict__ colids, const float* __restrict__ values,
                 const float* __restrict__ in, float* __restrict__ out, int64_t ld_in, int64_t ld_out,
                 uint32_t lds_words, int mode, const int32_t* __restrict__ merged)
{
    extern __shared__ __align__(16) int sm[];
    const uint32_t tid = threadIdx.x;
    const LeanItem it = items[blockIdx.x];
    if (it.flags & 8) return;  // (small items packed for the lean kernel: this launch has a workgroup for each)
    if (it.flags & 2) {        // (the same for the whole workgroup)
        any_row_block<ALIGNED, FIRST>(it, items + blockIdx.x, sm, rpt, colids, values, in, out, ld_in, ld_out, lds_words);
        return;
    }
    const int m = it.m, k = it.k, nnz = it.nnz;
    const uint32_t fw = max((uint32_t)it.flags >> 8, 1u);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wl = tid & 63;
    char* lds = reinterpret_cast<char*>(sm);
    char* bs = lds + it.b_byte;
    typedef const void __attribute__((address_space(1)))* gptr;
    typedef void __attribute__((address_space(3)))* lptr;

    // ---- dense tile, global -> LDS: rows of `chunks` 16-byte words
    const int64_t at = (int64_t)it.in_row * ld_in + it.f0;
    const bool windows = ALIGNED || (mode & kAnyWindows);     // (the same for the whole launch)
    const uint32_t chunks = (uint32_t)tile_stride((int)fw, ALIGNED || (mode & kAnyTight)) >> 2;
    const bool run = !ALIGNED && windows && (int64_t)fw == ld_in;   // (f0 is 0 then)
    const uint32_t stride = run ? fw : chunks << 2;  // words from row to row in LDS
    if (run) {
        const uint32_t shift = k > 0 ? (uint32_t)at & 3 : 0;     // (no rows: nothing is read, `in` may be null)
        const float* __restrict__ src = in + (at - shift);
        const uint32_t words = (uint32_t)k * fw + shift, total = words >> 2, rest = words & 3;
        for (uint32_t e0 = wave << 6; e0 < total; e0 += kThreads)
            if (e0 + wl < total)
                __builtin_amdgcn_global_load_lds((gptr)(src + 4 * (e0 + wl)), (lptr)(bs + (e0 << 4)), 16, 0, 0);
        if (wave == 0 && wl < rest)
            __builtin_amdgcn_global_load_lds((gptr)(src + 4 * total + wl), (lptr)(bs + (total << 4)), 4, 0, 0);
    } else if (windows) {
        // the last chunk of the last row may reach past the operation's block: its words are
        // copied one by one
        const int64_t row_last = at + (int64_t)(k - 1) * ld_in;
        const int64_t base_last = row_last & ~(int64_t)3;
        const uint32_t full_last = (uint32_t)(row_last + fw - base_last) >> 2;      // whole chunks of the last row
        const uint32_t total = k > 0 ? (uint32_t)(k - 1) * chunks + (ALIGNED ? chunks : full_last) : 0;
        const float inv = 1.f / (float)chunks;
        for (uint32_t e0 = wave << 6; e0 < total; e0 += kThreads) {
            const uint32_t e = e0 + wl;
            const uint32_t r = div_small(e, inv), c = e - r * chunks;
            const int64_t row = at + r * ld_in;
            if (e < total)
                __builtin_amdgcn_global_load_lds((gptr)(in + ((ALIGNED ? row : row & ~(int64_t)3) + 4 * c)),
                                                 (lptr)(bs + (e0 << 4)), 16, 0, 0);
        }
        if (!ALIGNED && k > 0) {
            const uint32_t rest = (uint32_t)(row_last + fw - base_last) & 3;
            if (wave == 0 && wl < rest)
                __builtin_amdgcn_global_load_lds((gptr)(in + (base_last + 4 * full_last + wl)),
                                                 (lptr)(bs + (total << 4)), 4, 0, 0);
        }
    } else {
        const float inv = 1.f / (float)stride;
        const uint32_t total = (uint32_t)k * stride;
        for (uint32_t e0 = wave << 6; e0 < total; e0 += kThreads) {
            const uint32_t e = e0 + wl;
            const uint32_t r = div_small(e, inv), c = e - r * stride;
            if (e < total && c < fw)
                __builtin_amdgcn_global_load_lds((gptr)(in + (at + r * ld_in + c)), (lptr)(bs + (e0 << 2)), 4, 0, 0);
        }
    }

    // ---- CSR (as bspmm_lean_kernel; the first four entries of a lane in one round trip)
    const bool summed = (it.flags & 4) != 0;
    const int32_t* __restrict__ rp = (summed ? merged : rpt) + it.rpt_off;
    const int32_t* __restrict__ ci = (summed ? merged : colids) + it.nz_off;
    const float* __restrict__ va = summed ? reinterpret_cast<const float*>(ci + round_up(nnz, 4)) : values + it.nz_off;
    const uint32_t ri = min(tid, (uint32_t)m);
    const int rv = rp[ri];
    int c[4] = {0, 0, 0, 0};
    float a[4] = {0.f, 0.f, 0.f, 0.f};
    const uint32_t last = (uint32_t)max(nnz - 1, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (nnz > u * kThreads) {                    // (the same for every lane)
            const uint32_t i = min(tid + u * kThreads, last);
            c[u] = ci[i];
            a[u] = va[i];
        }
    __builtin_amdgcn_sched_barrier(0);

    // ---- LDS writes, clamped as in bspmm_lean_kernel; an entry carries the byte offset of its
    // dense row inside the tile
    int2* cv = reinterpret_cast<int2*>(lds + it.cv_byte);
    sm[ri] = min(max(rv, 0), nnz);
    const uint32_t at3 = windows ? (uint32_t)at : 0, ld3 = windows && !run ? (uint32_t)ld_in : 0;
    auto entry = [&](int col, float v) {
        const uint32_t r = (unsigned)col < (unsigned)k ? (uint32_t)col : 0;
        uint32_t off = __umul24(r, stride << 2);
        if (!ALIGNED) off += ((at3 + r * ld3) & 3) << 2;
        return make_int2((int)off, __float_as_int(v));
    };
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (nnz > u * kThreads) cv[min(tid + u * kThreads, last)] = entry(c[u], a[u]);
    if (m >= kThreads)
        for (int i = tid + kThreads; i <= m; i += kThreads) sm[i] = min(max(rp[i], 0), nnz);
    if (nnz > 4 * kThreads)
        for (int p = tid + 4 * kThreads; p < nnz; p += kThreads) cv[p] = entry(ci[p], va[p]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
    __syncthreads();

    // ---- rows
    float* __restrict__ dst = out + (((int64_t)it.out_row + it.row0) * ld_out + it.f0);
    auto row = [&](int i, int& p0, int& p1) {
        p0 = sm[it.row0 + i];
        p1 = sm[it.row0 + i + 1];
    };
    auto lds_entry = [&](int p) { return cv[p]; };
    const int sums = round_up(it.cv_byte, 16);
    const int parts = long_row_parts<ALIGNED>(fw, it.nrows, nnz, m, it.b_byte - sums + 4 * k * (int)stride);
    if (parts > 1)
        any_long_rows<ALIGNED>(fw, it.nrows, parts, dst, ld_out, reinterpret_cast<float4*>(lds + sums), row, lds_entry,
                               TileRows<ALIGNED>{bs});
    else if (!ALIGNED && nnz > kLongRow * m)
        any_rows<1, false>(fw, it.nrows, dst, ld_out, row, lds_entry, TileRows<false>{bs});
    else
        any_rows<4, ALIGNED>(fw, it.nrows, dst, ld_out, row, lds_entry, TileRows<ALIGNED>{bs});
}

// The entry range of every row block into its item, for plans whose builds are wanted ahead of the first run.
__global__ void lean_hints_kernel(LeanItem* items, int n, const int32_t* __restrict__ rpt)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    LeanItem& it = items[i];
    if ((it.flags & 2) == 0 || it.nrows <= 0) return;
    const int2 range = row_block_range(it, rpt);
    it.tile_vecs = range.x;
    it.count = range.y;
}

// A small operation on one wavefront of a lean launch (four of them share a workgroup, see plain_schedule):
// the staged path of bspmm_lean_kernel with 64 lanes and its own quarter of the LDS; the wavefront waits for
// itself only.
__device__ __forceinline__ void lean_wave_item(const LeanItem& it, char* lds, const int32_t* __restrict__ rpt,
                                               const int32_t* __restrict__ colids, const float* __restrict__ values,
                                               const float* __restrict__ in, float* __restrict__ out, uint32_t ld_in,
                                               uint32_t ld_out)
{
    const uint32_t lane = threadIdx.x & 63;
    const int m = it.m, k = it.k, nnz = it.nnz, sh = it.sh;
    const uint32_t nvec = 1u << sh;
    int* sm = reinterpret_cast<int*>(lds);
    {
        const char* __restrict__ src =
            reinterpret_cast<const char*>(in + ((uint64_t)it.in_row * ld_in + (uint32_t)it.f0));
        const uint32_t row_bytes = ld_in << 2, total = (uint32_t)it.tile_vecs;
        char* bs = lds + it.b_byte;
        for (uint32_t e0 = 0; e0 < total; e0 += 64) {
            const uint32_t e = e0 + lane;
            if (e < total)
                __builtin_amdgcn_global_load_lds(
                    (const void __attribute__((address_space(1)))*)(
                        src + (__umul24(e >> sh, row_bytes) + ((e & (nvec - 1)) << 4))),
                    (void __attribute__((address_space(3)))*)(bs + (e0 << 4)), 16, 0, 0);
        }
    }
    const int32_t* __restrict__ rp = rpt + it.rpt_off;
    const int32_t* __restrict__ ci = colids + it.nz_off;
    const float* __restrict__ va = values + it.nz_off;
    const uint32_t ri = min(lane, (uint32_t)m), last = (uint32_t)max(nnz - 1, 0);
    const int rv = rp[ri];
    int c[2] = {0, 0};
    float a[2] = {0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (nnz > u * 64) {
            c[u] = ci[min(lane + u * 64, last)];
            a[u] = va[min(lane + u * 64, last)];
        }
    __builtin_amdgcn_sched_barrier(0);
    const int lsh = sh + 4;
    int2* cv = reinterpret_cast<int2*>(lds + it.cv_byte);
    auto entry = [&](int col, float v) { return make_int2((unsigned)col < (unsigned)k ? col << lsh : 0, __float_as_int(v)); };
    sm[ri] = min(max(rv, 0), nnz);
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (nnz > u * 64) cv[min(lane + u * 64, last)] = entry(c[u], a[u]);
    for (int i = lane + 64; i <= m; i += 64) sm[i] = min(max(rp[i], 0), nnz);
    for (int p = lane + 128; p < nnz; p += 64) cv[p] = entry(ci[p], va[p]);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();

    const uint32_t l = lane & (nvec - 1);
    const char* bcol = lds + it.b_byte + (l << 4);
    char* __restrict__ dst = reinterpret_cast<char*>(out + ((uint64_t)it.out_row * ld_out + (uint32_t)it.f0));
    const uint32_t out_row_bytes = ld_out << 2;
    for (uint32_t r = lane >> sh; r < (uint32_t)m; r += 64u >> sh)
        store_out<4>(reinterpret_cast<float*>(dst + (__umul24(r, out_row_bytes) + (l << 4))),
                     gather_row(cv, bcol, sm[r], sm[r + 1]));
}

// Dense tile of a staged item, straight from global memory into LDS, 1 KiB per wavefront instruction
// (lane i lands at base + 16*i); a tile no other item reads is streamed.  Offsets inside the item's
// block are 32-bit (the host launches the lean kernels only when they fit).
__device__ __forceinline__ void lean_tile(const LeanItem& it, char* lds, const float* __restrict__ in, uint32_t ld_in,
                                          uint32_t wave, uint32_t wl)
{
    const char* __restrict__ src =
        reinterpret_cast<const char*>(in + ((uint64_t)it.in_row * ld_in + (uint32_t)it.f0));
    const uint32_t row_bytes = ld_in << 2, total = (uint32_t)it.tile_vecs, nvec = 1u << it.sh;
    const int sh = it.sh;
    char* bs = lds + it.b_byte;
    if (it.flags & 1) {
        for (uint32_t e0 = wave << 6; e0 < total; e0 += kThreads) {
            const uint32_t e = e0 + wl;
            if (e < total)
                __builtin_amdgcn_global_load_lds(
                    (const void __attribute__((address_space(1)))*)(
                        src + (__umul24(e >> sh, row_bytes) + ((e & (nvec - 1)) << 4))),
                    (void __attribute__((address_space(3)))*)(bs + (e0 << 4)), 16, 0, 2);
        }
    } else {
        for (uint32_t e0 = wave << 6; e0 < total; e0 += kThreads) {
            const uint32_t e = e0 + wl;
            if (e < total)
                __builtin_amdgcn_global_load_lds(
                    (const void __attribute__((address_space(1)))*)(
                        src + (__umul24(e >> sh, row_bytes) + ((e & (nvec - 1)) << 4))),
                    (void __attribute__((address_space(3)))*)(bs + (e0 << 4)), 16, 0, 0);
        }
    }
}

// MERGED: items with flag bit 2 read their CSR from the merged arrays of summed sets (a template
// parameter: the selects cost the plain kernel).  512 graphs of four channels with dense blocks of their
// own, F = 128, summed: 9.1 us, 10.0 through the general kernel.
template <bool MERGED, bool FIRST = false>
__global__ void __launch_bounds__(kThreads)
bspmm_lean_kernel(const LeanItem* __restrict__ items, const int32_t* __restrict__ rpt,
                  const int32_t* __restrict__ colids, const float* __restrict__ values,
                  const float* __restrict__ in, float* __restrict__ out, uint32_t ld_in,
                  uint32_t ld_out, uint32_t lds_words, const int32_t* __restrict__ merged)
{
    extern __shared__ __align__(16) int sm[];
    const uint32_t tid = threadIdx.x;
    // One clause of scalar loads fetches the whole item; there is no early exit for an empty
    // item (all its sizes are zero, so nothing below has a trip): a branch on one field would
    // split the fetch into two dependent round trips.  The output arguments are pulled in here
    // as well, not after the barrier where they are first used.
    const LeanItem it = items[blockIdx.x];
    asm volatile("" ::"s"(out), "s"(ld_out));
    if (it.flags & 10) {       // (the same for the whole workgroup)
        if (it.flags & 2) {
            lean_row_block<FIRST>(it, items + blockIdx.x, sm, rpt, colids, values, in, out, ld_in, ld_out, lds_words);
        } else {
            const int w = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
            if (w < it.count) {
                const LeanItem small = items[it.tile_vecs + w];
                lean_wave_item(small, reinterpret_cast<char*>(sm) + w * ((lds_words / kWaves) & ~3u) * 4, rpt, colids,
                               values, in, out, ld_in, ld_out);
            }
        }
        return;
    }
    const int m = it.m, k = it.k, nnz = it.nnz;
    const int sh = it.sh;
    const uint32_t nvec = 1u << sh;                  // float4 per tile row, <= 64
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wl = tid & 63;
    char* lds = reinterpret_cast<char*>(sm);

    lean_tile(it, lds, in, ld_in, wave, wl);
    // ---- CSR: the row pointers of this lane group's first row (they stay in registers), all
    // row pointers and the entries (on their way to LDS).  Indices are clamped instead of
    // predicated: a lane past the end reads, and later writes, what the last lane does.
    const bool summed = MERGED && (it.flags & 4) != 0;
    const int32_t* __restrict__ rp = (summed ? merged : rpt) + it.rpt_off;
    const int32_t* __restrict__ ci = (summed ? merged : colids) + it.nz_off;
    const float* __restrict__ va = summed ? reinterpret_cast<const float*>(ci + round_up(nnz, 4)) : values + it.nz_off;
    const uint32_t r_first = (uint32_t)it.row0 + (tid >> sh);
    const uint32_t um = (uint32_t)m;
    const int q0 = rp[min(r_first, um)];
    const int q1 = rp[min(r_first + 1, um)];
    const uint32_t ri = min(tid, um);
    const int rv = rp[ri];
    const uint32_t last = (uint32_t)max(nnz - 1, 0);
    const uint32_t i0 = min(tid, last), i1 = min(tid + kThreads, last);
    int c0 = 0, c1 = 0;
    float a0 = 0.f, a1 = 0.f;
    if (nnz > 0) {               // (the same for every lane: a scalar branch)
        c0 = ci[i0];
        a0 = va[i0];
    }
    if (nnz > kThreads) {
        c1 = ci[i1];
        a1 = va[i1];
    }
    // No use of a loaded value above this line (its wait would hold back later loads).
    __builtin_amdgcn_sched_barrier(0);

    // ---- LDS writes.  Row pointers are clamped to [0, nnz] and columns to [0, k): malformed
    // arrays cannot make a lane leave the item's LDS.  An entry carries the byte offset of its
    // dense row inside the tile.
    const int lsh = sh + 4;                          // log2 of the tile's row stride in bytes
    int2* cv = reinterpret_cast<int2*>(lds + it.cv_byte);
    sm[ri] = min(max(rv, 0), nnz);
    if (nnz > 0) cv[i0] = make_int2((unsigned)c0 < (unsigned)k ? c0 << lsh : 0, __float_as_int(a0));
    if (nnz > kThreads) cv[i1] = make_int2((unsigned)c1 < (unsigned)k ? c1 << lsh : 0, __float_as_int(a1));
    if (m >= kThreads)
        for (int i = tid + kThreads; i <= m; i += kThreads) sm[i] = min(max(rp[i], 0), nnz);
    if (nnz > 2 * kThreads)
        for (int p = tid + 2 * kThreads; p < nnz; p += kThreads) {
            const int c = ci[p];
            cv[p] = make_int2((unsigned)c < (unsigned)k ? c << lsh : 0, __float_as_int(va[p]));
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
    __syncthreads();

    // ---- rows: the first pass from the registers, later passes from the staged row pointers
    const uint32_t l = tid & (nvec - 1);
    const char* bcol = lds + it.b_byte + (l << 4);
    char* __restrict__ dst = reinterpret_cast<char*>(out + ((uint64_t)it.out_row * ld_out + (uint32_t)it.f0));
    const uint32_t out_row_bytes = ld_out << 2;
    const uint32_t row_end = (uint32_t)(it.row0 + it.nrows);
    const uint32_t groups = kThreads >> sh;          // rows in flight
    if (r_first < row_end)
        store_out<4>(reinterpret_cast<float*>(dst + (__umul24(r_first, out_row_bytes) + (l << 4))),
                     gather_row(cv, bcol, min(max(q0, 0), nnz), min(max(q1, 0), nnz)));
    for (uint32_t r = r_first + groups; r < row_end; r += groups)
        store_out<4>(reinterpret_cast<float*>(dst + (__umul24(r, out_row_bytes) + (l << 4))),
                     gather_row(cv, bcol, sm[r], sm[r + 1]));
}

// ---------------------------------------------------------------------------------------
// The first transposed product of a plan whose transposed CSR arrays do not exist yet.  A batch that is
// new every step used to pay for two launches here, the build (one workgroup per operation, a latency
// chain of 5 us) and the product, each 3.5 us of host time beside what the GPU takes.  Instead every
// workgroup of the product sorts its operation itself, in the LDS of its item: entries of
// A (a column, and the row that its row pointers give) are counted per column, the counts are scanned,
// the entries' positions are scattered in the order in which they were counted, and an entry's rank among its
// column's positions is its place - the stable order of build_sorted_kernel, whatever the order of arrival, so
// the sums are bit for bit those of the build and bspmm_lean_kernel.  Positions and rows of the
// entries take the two halves of the words that their (row offset, value) pairs take afterwards.  Every
// workgroup of an operation sorts, so hub nodes must not make it long: long columns keep their positions as one
// bit each, whose ranks are at most 32 words away, and a wavefront writes the rows of a long row's entries together.  The
// workgroup with the first rows and columns of an operation writes its transposed arrays, for every later run.
// 128 molecules, F = 128, GPU time of build and product 8.7 us, of this kernel 5.6; a step with a new batch (plan, both
// products) 29.7 -> 25.9 us, 512 from index pairs at F = 64 45.9 to 47.3 -> 42.1 to 44.4.  Bound: the chain of LDS round
// trips and barriers of the sort, which other workgroups of the CU hide in larger launches.
// Star graphs, between events around the first run, us, build and product / every lane through its row and column
// alone / as it is: 512 of 100 nodes at F = 64 27.4 / 26.2 / 14.9, at F = 512 55 / 100 / 53; 4000 of 150 at F = 64 121 /
// 186 / 84; 512 of 190 at F = 512 129 / 320 / 113; batches without hubs 0.2 us longer for it (128 molecules 11.2 / 7.6 / 7.9).
// (square operations, arrays of both directions at the same offsets: `it` describes either; at most four entries per lane)
// ---------------------------------------------------------------------------------------
constexpr int kHubEntries = 16;   // entries of a row or column that one lane goes through on its own

__global__ void __launch_bounds__(kThreads)
bspmm_first_transposed_kernel(const LeanItem* __restrict__ items, const int32_t* __restrict__ rpt,
                              const int32_t* __restrict__ colids, const float* __restrict__ values,
                              const float* __restrict__ in, float* __restrict__ out, uint32_t ld_in, uint32_t ld_out,
                              int32_t* __restrict__ rpt_t, int32_t* __restrict__ colids_t, float* __restrict__ values_t)
{
    extern __shared__ __align__(16) int sm[];
    const uint32_t tid = threadIdx.x;
    const LeanItem it = items[blockIdx.x];
    if (it.flags & 8) return;  // (small items packed for the lean kernel: this launch has a workgroup for each)
    const int m = it.m, nnz = min(it.nnz, 4 * kThreads), sh = it.sh;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wl = tid & 63;
    char* lds = reinterpret_cast<char*>(sm);
    lean_tile(it, lds, in, ld_in, wave, wl);

    // ---- requests: up to four entries per lane, the two pointers of this lane's first row
    const int32_t* __restrict__ rp = rpt + it.rpt_off;
    const int32_t* __restrict__ ci = colids + it.nz_off;
    const float* __restrict__ va = values + it.nz_off;
    const uint32_t last = (uint32_t)max(nnz - 1, 0);
    int key[4] = {-1, -1, -1, -1};
    float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (nnz > u * kThreads) {                    // (the same for every lane)
            const uint32_t i = min(tid + u * kThreads, last);
            key[u] = ci[i];
            a[u] = va[i];
        }
    int r0 = rp[min(tid, (uint32_t)m)], r1 = rp[min(tid + 1, (uint32_t)m)];
    __builtin_amdgcn_sched_barrier(0);

    int2* cv = reinterpret_cast<int2*>(lds + it.cv_byte);
    int* pos = reinterpret_cast<int*>(cv);           // positions in A, by column
    int* row_of = pos + nnz;                         // row of every entry of A
    for (int c = tid; c <= m; c += kThreads) sm[c] = 0;
    for (int i0 = (int)wave * 64; i0 < m; i0 += kThreads) {          // (the same for every lane of a wavefront)
        const int i = i0 + (int)wl;
        if (i0 >= kThreads) r0 = rp[min(i, m)], r1 = rp[min(i + 1, m)];
        // (entries outside what the row pointers cover: the first row and the last, as in the build)
        const int from = i > 0 ? max(r0, 0) : 0, end = i + 1 < m ? min(r1, nnz) : nnz;
        const bool hub = i < m && end - from > kHubEntries;
        if (i < m && !hub)
            for (int p = from; p < end; ++p) row_of[p] = i;
        for (uint64_t rows = __ballot(hub); rows != 0; rows &= rows - 1) {
            const int lane = __builtin_ctzll(rows), first = __shfl(from, lane), past = __shfl(end, lane);
            for (int p = first + (int)wl; p < past; p += 64) row_of[p] = i0 + lane;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)                      // (entries outside the matrix are skipped, as in the build)
        if ((int)(tid + u * kThreads) >= nnz || (unsigned)key[u] >= (unsigned)m) key[u] = -1;
    __syncthreads();
    int place[4], row[4];                            // (first: how many entries of its column came before)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        place[u] = row[u] = 0;
        if (key[u] >= 0) place[u] = atomicAdd(&sm[key[u] + 1], 1);
    }
    __syncthreads();

    // ---- inclusive scan of sm[0..m]: afterwards the first position of every column.  The wavefronts' sums go through
    // the words of the positions, of which an operation without four entries has too few: the items' LDS may be
    // all that a workgroup can have, so that there is none beside it.
    const bool writes = it.row0 == 0 && it.f0 == 0 && m > 0;
    const int chunk = (m + kThreads) / kThreads;
    const int lo = tid * chunk, hi = min(lo + chunk, m + 1);
    int sum = 0;
    for (int c = lo; c < hi; ++c) sum += sm[c];
    int incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int n = __shfl_up(incl, d);
        if ((int)wl >= d) incl += n;
    }
    const int words = (nnz + 31) >> 5, from_long = max(words + kWaves, kHubEntries);   // bits, and entries of a long column
    int before = 0;
    bool hubs = false;                               // a column is long
    if (nnz >= kWaves) {
        const bool mine = max(max(place[0], place[1]), max(place[2], place[3])) >= from_long - 1;
        const int bit = __ballot(mine) != 0 ? 1 << 16 : 0;
        if (wl == 63) pos[wave] = incl | bit;
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int of = pos[w];
            all |= of;
            before += w < (int)wave ? of & 0xffff : 0;
        }
        hubs = __builtin_amdgcn_readfirstlane(all) >> 16 != 0;
        if (hubs)                                    // (a long column's bits are its last words: not the sums')
            for (int p = kWaves + (int)tid; p < nnz; p += kThreads) pos[p] = 0;
    } else {
        const int front = min((int)wave * 64 * chunk, m + 1);
        for (int c = wl; c < front; c += 64) before += sm[c];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) before += __shfl_xor(before, d);
        __syncthreads();
    }
    int run = before + incl - sum;
    for (int c = lo; c < hi; ++c) {
        run += sm[c];
        sm[c] = run;
        if (writes) rpt_t[it.rpt_off + (uint32_t)c] = run;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (key[u] >= 0) {
            const int p = (int)(tid + u * kThreads), beg = sm[key[u]];
            int* at = pos + beg + place[u];
            if (hubs) {
                const int end = sm[key[u] + 1];
                if (end - beg >= from_long) at = nullptr, atomicOr(&pos[end - words + (p >> 5)], 1 << (p & 31));
            }
            if (at) *at = p;
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (key[u] < 0) continue;
        const int p = (int)(tid + u * kThreads);
        const int beg = sm[key[u]], end = sm[key[u] + 1];
        int rank = 0, t = beg;
        if (hubs && end - beg >= from_long) {
            const int last_word = end - words + (p >> 5);
            rank = __popc(pos[last_word] & ((1u << (p & 31)) - 1u));
            for (t = end - words; t < last_word; ++t) rank += __popc(pos[t]);
            t = end;
        }
        for (; t < end; ++t) rank += pos[t] < p ? 1 : 0;
        place[u] = beg + rank;
        row[u] = row_of[p];
        if ((unsigned)row[u] >= (unsigned)m) row[u] = 0;   // (decreasing row pointers may leave an entry out)
    }
    __syncthreads();                                 // everyone has read positions and rows
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (key[u] >= 0) cv[place[u]] = make_int2(row[u] << (sh + 4), __float_as_int(a[u]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
    __syncthreads();

    // ---- rows, as in bspmm_lean_kernel
    const uint32_t l = tid & ((1u << sh) - 1);
    const char* bcol = lds + it.b_byte + (l << 4);
    char* __restrict__ dst = reinterpret_cast<char*>(out + ((uint64_t)it.out_row * ld_out + (uint32_t)it.f0));
    const uint32_t out_row_bytes = ld_out << 2;
    const uint32_t row_end = (uint32_t)(it.row0 + it.nrows);
    for (uint32_t r = (uint32_t)it.row0 + (tid >> sh); r < row_end; r += kThreads >> sh)
        store_out<4>(reinterpret_cast<float*>(dst + (__umul24(r, out_row_bytes) + (l << 4))),
                     gather_row(cv, bcol, sm[r], sm[r + 1]));
    if (writes)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (key[u] >= 0) {
                colids_t[it.nz_off + (uint32_t)place[u]] = row[u];
                values_t[it.nz_off + (uint32_t)place[u]] = a[u];
            }
}

// ---------------------------------------------------------------------------------------
// transposed CSR build: one workgroup per operation.
//   count entries per column -> exclusive prefix sum (row pointers of A^T) -> scatter the
//   entry positions with atomic cursors (arrival order is arbitrary) -> every entry finds its
//   rank inside its column segment by counting the positions smaller than its own.
// The result does not depend on the arrival order: it is the stable transpose.
// `work` is k+1 counters followed by nnz positions (and, for small operations, the input's
// row pointers), in LDS when it fits, else in global scratch (both reached through flat
// addressing).
// ---------------------------------------------------------------------------------------
// FROM_COO = true sorts a SparseTensor / COO operation (index pairs as in Fig. 2:
// ids[2p] = row, ids[2p+1] = column, in any order) into CSR with the same machinery: the key is
// the row, the payload the column; `colids` is then the pair array, o.k the number of rows,
// o.m the number of columns, and the result is the stable sort by row (entries of a row keep
// their stored order).
template <bool FROM_COO, int T>
__global__ void __launch_bounds__(T)
build_sorted_kernel(const OpRecord* __restrict__ ops, const int32_t* __restrict__ rpt,
                    const int32_t* __restrict__ colids, const float* __restrict__ values,
                    int32_t* __restrict__ rpt_t, int32_t* __restrict__ colids_t,
                    float* __restrict__ values_t, int32_t* gscratch,
                    const int32_t* __restrict__ order)
{
    extern __shared__ __align__(16) int sm[];
    __shared__ int partial[T];
    // (operations are taken largest first: the launch lasts as long as its slowest workgroup)
    const OpRecord o = ops[order[blockIdx.x]];
    const int tid = threadIdx.x;
    const int k = o.k, m = o.m, nnz = o.nnz;
    int* cnt = o.scratch_off >= 0 ? gscratch + o.scratch_off : sm;   // k+1 ints
    int* pos = cnt + (k + 1);                                          // nnz ints
    const int32_t* ci = colids + (FROM_COO ? 2 * o.nz_off : o.nz_off);
    const int32_t* rp = rpt + o.rpt_off;
    int32_t* rt = rpt_t + o.rpt_t_off;
    // key of entry p, or -1 when the entry is malformed and must be skipped
    auto key_of = [&](int p) {
        if (FROM_COO) {
            const int r = ci[2 * p], c = ci[2 * p + 1];
            return ((unsigned)r < (unsigned)k && (unsigned)c < (unsigned)m) ? r : -1;
        }
        const int c = ci[p];
        return (unsigned)c < (unsigned)k ? c : -1;
    };
    // Pairs outside their matrix leave room behind the others: no column there, so that the transposed build, which
    // asks every entry that the operation was planned for, leaves them out too.
    auto close = [&](int placed) {
        if (FROM_COO)
            for (int p = placed + tid; p < nnz; p += T) {
                colids_t[o.nz_t_off + p] = -1;
                values_t[o.nz_t_off + p] = 0.f;
            }
    };

    // ---- small operations (flagged by the host: everything in LDS, at most four entries per
    // lane): one round trip to memory reads the operation into registers (and the row
    // pointers into LDS, which turns the search for an entry's row into LDS reads), the scan
    // runs on wavefront shuffles, and nothing is read twice.
    if (o.small == 1) {
        constexpr int E = build_entries_per_lane(T);
        int key[E], pay[E];
        float val[E];
        const float* va = values + o.nz_off;
        int* rps = pos + nnz;                              // CSR input only: m+1 row pointers
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int p = tid + u * T;
            key[u] = -1;
            pay[u] = 0;
            val[u] = 0.f;
            if (p < nnz) {
                if (FROM_COO) {
                    const int r = ci[2 * p], c = ci[2 * p + 1];
                    key[u] = ((unsigned)r < (unsigned)k && (unsigned)c < (unsigned)m) ? r : -1;
                    pay[u] = c;
                } else {
                    const int c = ci[p];
                    key[u] = (unsigned)c < (unsigned)k ? c : -1;
                }
                val[u] = va[p];
            }
        }
        if (!FROM_COO)
            for (int i = tid; i <= m; i += T) rps[i] = rp[i];
        for (int c = tid; c <= k; c += T) cnt[c] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < E; ++u)
            if (key[u] >= 0) atomicAdd(&cnt[key[u] + 1], 1);
        __syncthreads();

        // inclusive scan of cnt[0..k]: a lane sums its chunk, the wavefront scans the sums with
        // shuffles, the four wavefront totals go through LDS
        const int chunk = (k + 1 + T - 1) / T;
        const int lo = tid * chunk;
        const int hi = min(lo + chunk, k + 1);
        int sum = 0;
        for (int c = lo; c < hi; ++c) sum += cnt[c];
        int incl = sum;
        const int wl = tid & 63;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int n = __shfl_up(incl, d);
            if (wl >= d) incl += n;
        }
        if (wl == 63) partial[tid >> 6] = incl;
        __syncthreads();
        int run = incl - sum;
        for (int w = 0; w < (tid >> 6); ++w) run += partial[w];
        for (int c = lo; c < hi; ++c) {
            run += cnt[c];
            cnt[c] = run;
            rt[c] = run;
        }
        __syncthreads();

        // scatter positions; cnt[c] ends as the first position of column c+1
#pragma unroll
        for (int u = 0; u < E; ++u)
            if (key[u] >= 0) pos[atomicAdd(&cnt[key[u]], 1)] = tid + u * T;
        __syncthreads();

#pragma unroll
        for (int u = 0; u < E; ++u) {
            if (key[u] < 0) continue;
            const int p = tid + u * T;
            const int c = key[u];
            const int beg = c > 0 ? cnt[c - 1] : 0;
            const int end = cnt[c];
            int rank = 0;
            for (int t = beg; t < end; ++t) rank += pos[t] < p ? 1 : 0;
            int a = pay[u];
            if (!FROM_COO) {
                // row of entry p: the last r with rp[r] <= p
                a = 0;
                int b = m;
                while (b - a > 1) {
                    const int mid = (a + b) >> 1;
                    if (rps[mid] <= p) a = mid; else b = mid;
                }
            }
            colids_t[o.nz_t_off + beg + rank] = a;
            values_t[o.nz_t_off + beg + rank] = val[u];
        }
        close(cnt[k]);
        return;
    }

    // ---- operations of more than a thousand entries that still fit LDS (flagged 2 by the
    // host): every entry is read from memory ONCE, in order, with all loads of a lane in flight
    // together; its key and its payload - for CSR input the row, which a pass over the row
    // pointers ORs in - are packed into one LDS word, so the histogram, the scatter and the
    // ranking run out of LDS, and the last pass walks the entries in stored order again
    // (coalesced value loads; the scattered side is the stores, which nothing waits for).
    if (o.small == 2) {
        const int kb = 32 - __clz(k);                     // bits of a key; the value k marks a skipped entry
        const unsigned kmask = (1u << kb) - 1u;
        unsigned* keyrow = reinterpret_cast<unsigned*>(pos + nnz);
        for (int c = tid; c <= k; c += T) cnt[c] = 0;
        __syncthreads();
        for (int p0 = tid; p0 < nnz; p0 += 4 * T) {
            int key[4], pay[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * T;
                key[u] = k;
                pay[u] = 0;
                if (p < nnz) {
                    if (FROM_COO) {
                        const int r = ci[2 * p], c = ci[2 * p + 1];
                        if ((unsigned)r < (unsigned)k && (unsigned)c < (unsigned)m) key[u] = r;
                        pay[u] = c;
                    } else {
                        const int c = ci[p];
                        if ((unsigned)c < (unsigned)k) key[u] = c;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * T;
                if (p < nnz) {
                    keyrow[p] = (unsigned)key[u] | (key[u] < k ? (unsigned)pay[u] << kb : 0u);
                    if (key[u] < k) atomicAdd(&cnt[key[u] + 1], 1);
                }
            }
        }
        if (!FROM_COO) {
            __syncthreads();          // keys in place before the rows are ORed in
            for (int r = tid; r < m; r += T) {
                const int b = min(max(rp[r + 1], 0), nnz);
                const int a = min(max(rp[r], 0), b);
                for (int p = a; p < b; ++p) atomicOr(&keyrow[p], (unsigned)r << kb);
            }
        }
        __syncthreads();

        // inclusive scan of cnt[0..k] (as below)
        const int chunk = (k + 1 + T - 1) / T;
        const int lo = tid * chunk;
        const int hi = min(lo + chunk, k + 1);
        int sum = 0;
        for (int c = lo; c < hi; ++c) sum += cnt[c];
        int incl = sum;
        const int wl = tid & 63;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int n = __shfl_up(incl, d);
            if (wl >= d) incl += n;
        }
        if (wl == 63) partial[tid >> 6] = incl;
        __syncthreads();
        int run = incl - sum;
        for (int w = 0; w < (tid >> 6); ++w) run += partial[w];
        for (int c = lo; c < hi; ++c) {
            run += cnt[c];
            cnt[c] = run;
            rt[c] = run;
        }
        __syncthreads();

        // scatter positions; cnt[c] ends as the first position of key c+1
        for (int p = tid; p < nnz; p += T) {
            const int c = (int)(keyrow[p] & kmask);
            if (c < k) pos[atomicAdd(&cnt[c], 1)] = p;
        }
        __syncthreads();

        const float* va = values + o.nz_off;
        float v_next = tid < nnz ? va[tid] : 0.f;
        for (int p = tid; p < nnz; p += T) {
            const float v = v_next;
            if (p + T < nnz) v_next = va[p + T];     // in flight during this trip
            const unsigned kr = keyrow[p];
            const int c = (int)(kr & kmask);
            if (c >= k) continue;
            const int beg = c > 0 ? cnt[c - 1] : 0;
            const int end = cnt[c];
            int rank = 0;
            for (int t = beg; t < end; ++t) rank += pos[t] < p ? 1 : 0;
            colids_t[o.nz_t_off + beg + rank] = (int)(kr >> kb);
            values_t[o.nz_t_off + beg + rank] = v;
        }
        close(cnt[k]);
        return;
    }

    for (int c = tid; c <= k; c += T) cnt[c] = 0;
    __syncthreads();
    for (int p = tid; p < nnz; p += T) {
        const int c = key_of(p);
        if (c >= 0) atomicAdd(&cnt[c + 1], 1);
    }
    __syncthreads();

    // inclusive scan of cnt[0..k]: afterwards cnt[c] = first position of column c
    const int chunk = (k + 1 + T - 1) / T;
    const int lo = tid * chunk;
    const int hi = lo + chunk < k + 1 ? lo + chunk : k + 1;
    int sum = 0;
    for (int c = lo; c < hi; ++c) sum += cnt[c];
    partial[tid] = sum;
    __syncthreads();
    for (int d = 1; d < T; d <<= 1) {
        const int add = tid >= d ? partial[tid - d] : 0;
        __syncthreads();
        partial[tid] += add;
        __syncthreads();
    }
    int run = tid > 0 ? partial[tid - 1] : 0;
    for (int c = lo; c < hi; ++c) {
        run += cnt[c];
        cnt[c] = run;
        rt[c] = run;
    }
    __syncthreads();

    // scatter positions; cnt[c] ends as the first position of column c+1
    for (int p = tid; p < nnz; p += T) {
        const int c = key_of(p);
        if (c >= 0) pos[atomicAdd(&cnt[c], 1)] = p;
    }
    __syncthreads();

    const float* va = values + o.nz_off;
    const int placed = cnt[k];                      // entries that were not skipped
    for (int q = tid; q < placed; q += T) {
        const int p = pos[q];
        const int c = key_of(p);
        const int beg = c > 0 ? cnt[c - 1] : 0;
        const int end = cnt[c];
        int rank = 0;
        for (int t = beg; t < end; ++t) rank += pos[t] < p ? 1 : 0;
        int a;
        if (FROM_COO) {
            a = ci[2 * p + 1];                        // the payload is the column
        } else {
            // row of entry p: the last r with rp[r] <= p
            a = 0;
            int b = m;   // invariant: rp[a] <= p, and (b == m or rp[b] > p)
            while (b - a > 1) {
                const int mid = (a + b) >> 1;
                if (rp[mid] <= p) a = mid; else b = mid;
            }
        }
        colids_t[o.nz_t_off + beg + rank] = a;
        values_t[o.nz_t_off + beg + rank] = va[p];
    }
    close(placed);
}

// Index pairs of a COO operation inside their matrix?
__global__ void __launch_bounds__(kThreads)
validate_coo_kernel(const OpRecord* __restrict__ ops, const int32_t* __restrict__ ids, int32_t* flag)
{
    const OpRecord o = ops[blockIdx.x];
    const int32_t* id = ids + 2 * o.nz_off;
    bool bad = false;
    for (int p = threadIdx.x; p < o.nnz; p += kThreads)
        if ((unsigned)id[2 * p] >= (unsigned)o.k || (unsigned)id[2 * p + 1] >= (unsigned)o.m) bad = true;
    if (bad) atomicMin(flag, (int)blockIdx.x);
}

// ---------------------------------------------------------------------------------------
// One channel of the batched graph-convolution layer in one launch (Fig. 7: MatMul, Add,
// BatchedSpMM): Y_i (+)= A_i (X_i W + bias).  A workgroup stages A_i, the layer input X_i
// (k x n_front), the weight tile W[:, f0:f0+fw] and the bias tile in LDS in ONE round trip to
// memory (more when X_i does not fit at once), computes the dense tile B = X_i W + bias on the matrix cores out of LDS into the
// tile's usual place, and then runs the ordinary row gather over it: U, B and the per-channel
// C never exist in memory.
// The dense part is v_mfma_f32_16x16x4_f32 (fp32 in, fp32 accumulate).  The tile is cut into
// 16 x 16 blocks dealt to the four wavefronts.  Operand layout of the instruction: lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16] and receives rows 4*(l / 16) .. +3 of column
// l % 16.  A lane reads four consecutive k of its X row with one 16-byte LDS read and feeds
// them to four instructions together with the weights of the same four k, so the k order
// inside a step differs from memory order for both operands alike, which leaves the product
// unchanged.
// (Whole layers in launches of several rounds use v_mfma_f32_32x32x2_f32 on 32 x 32 blocks
// instead; see dense_rows32 in the kernel.)
// LDS, in words: the staged layout of the item (row pointers, entries, dense tile k x fw),
// then the weight tile (n_front x fw), the bias tile (fw) and as many rows of X_i as fit
// (a multiple of 16; operations with more rows take several passes).
// Needs F % 16 == 0, n_front % 4 == 0 and 16-byte aligned operands (checked on the host).
// ---------------------------------------------------------------------------------------

// rows x (4 * nvec) floats, global (leading dimension ld) -> LDS (rows packed).  Whole
// wavefronts copy 1 KiB per instruction straight into LDS when a row is a power-of-two number
// of float4; otherwise through registers, four rows per lane group in flight.
// `swz` != 0 (only with a power-of-two nvec, swz < nvec) stores the float4 with index v of row r
// in slot v ^ (r & swz): rows that are a multiple of 64 words apart then no longer fall on the
// same LDS banks when 16 lanes read the same column of 16 consecutive rows.
template <int THREADS = kThreads>
__device__ __forceinline__ void stage_tile4(float* dst, const float* __restrict__ src, int64_t ld,
                                            int rows, int nvec, int tid, int swz = 0)
{
    if ((nvec & (nvec - 1)) == 0) {
        const int sh = ilog2(nvec);
        const int total = rows << sh;
        const int wl = tid & 63;
        for (int e0 = (tid >> 6) << 6; e0 < total; e0 += THREADS) {
            const int e = e0 + wl;
            if (e < total) {
                const int r = e >> sh;
                const float* gp = src + (int64_t)r * ld + ((((e & (nvec - 1)) ^ (r & swz))) << 2);
                __builtin_amdgcn_global_load_lds(
                    (const void __attribute__((address_space(1)))*)gp,
                    (void __attribute__((address_space(3)))*)(dst + (e0 << 2)), 16, 0, 0);
            }
        }
    } else {
        const int gl = min(64, pow2_ceil(nvec));
        const int sh = ilog2(gl);
        const int g = tid >> sh, l = tid & (gl - 1), G = THREADS >> sh;
        if (l < nvec)
            for (int r0 = g; r0 < rows; r0 += 4 * G) {
                float4 t[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    t[u] = load_vec<4>(src + (int64_t)min(r0 + u * G, rows - 1) * ld + 4 * l);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (r0 + u * G < rows) store_vec<4>(dst + (r0 + u * G) * (nvec << 2) + 4 * l, t[u]);
            }
    }
}

// SETS = true: every item stands in for a set of M channel operations that share the layer
// input X_i and are summed into one output block (the whole layer of Fig. 7 in one launch):
// the dense tile is [X_i W[0] + bias[0]; ...; X_i W[M-1] + bias[M-1]] (M x kx rows), the CSR is
// the set's merged one, whose entries of channel c name rows c*kx ... of that tile; W is the M
// weight matrices one under the other (M*nx rows), bias M rows of P.fused_stride floats apart, and
// P.rpt is the base of the merged arrays.
// THREADS: 256, or 512 for launches of a single round of workgroups, whose time is the time of
// the largest item: twice the wavefronts halve its matrix blocks per wavefront and the passes
// of its gather.
template <bool ACC, bool SETS, int THREADS = kThreads>
__global__ void __launch_bounds__(THREADS) bspmm_gcn_kernel(const LaunchParams P)
{
    extern __shared__ __align__(16) int sm[];
    typedef float mfma4 __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x;
    const WorkItem it = P.items[blockIdx.x];
    if (it.nrows <= 0) return;
    const int nx = P.n_front;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wl = tid & 63;
    const int col = wl & 15, g = wl >> 4;
    const int nb_count = it.fw >> 4;
    const int M = SETS ? max(1, (it.staged >> 8) & 0xff) : 1;   // channels
    const int kx = SETS ? it.k / M : it.k;                       // rows of X_i

    const StagedLayout L = staged_layout(it.m, it.k, it.nnz, it.fw, 0, false);
    float* bt = reinterpret_cast<float*>(sm + L.b_off);      // dense tile k x fw, made below
    float* ws = bt + it.k * it.fw;                            // weight tiles, M x (nx x fw)
    float* bias_s = ws + M * nx * it.fw;                      // bias tiles, M x fw
    float* xs = bias_s + M * it.fw;                           // rows of X_i, R x nx
    // X_i is taken R rows at a time: all of them when the rest of the LDS holds them, else a
    // multiple of 16 (a 16 x 16 block needs 16 rows of X_i and all of their columns).  The
    // host has made sure of 16.
    const int x_room = (P.lds_floats - (int)(xs - reinterpret_cast<float*>(sm))) / nx;
    const int R = kx <= x_room ? kx : x_room & ~15;
    const int xvec = nx >> 2;
    const int swz = (xvec & (xvec - 1)) == 0 ? min(xvec, 16) - 1 : 0;
    const float* xg = P.in + it.in_row_off * P.ld_in;

    // dense tile rows r0 .. r0+rows on the matrix cores, LDS -> LDS
    auto dense_rows = [&](int r0, int rows) {
        const int per_channel = ((rows + 15) >> 4) * nb_count;
        const int blocks = per_channel * M;
        for (int blk = wave; blk < blocks; blk += THREADS / 64) {
            const int c = SETS ? blk / per_channel : 0;
            const int rem = blk - c * per_channel;
            const int mb = rem / nb_count, nb = rem - mb * nb_count;
            const float bv = bias_s[c * it.fw + 16 * nb + col];
            // four independent accumulators (one per k of a lane's four): a chain of
            // dependent matrix instructions would run at their latency, not their rate
            mfma4 acc = {bv, bv, bv, bv};
            mfma4 acc1 = {0.f, 0.f, 0.f, 0.f}, acc2 = acc1, acc3 = acc1;
            const int arow = min(16 * mb + col, rows - 1);     // rows past the end repeat the last
            const float* xrow = xs + arow * nx;
            const int xs_swz = arow & swz;
            const float* wcol = ws + (c * nx + 4 * g) * it.fw + 16 * nb + col;
            // Sixteen k per trip (four per lane group, one matrix instruction each).  The
            // operands of the next trip are read from LDS before the instructions of this one
            // are issued: read latency then hides behind the matrix pipeline instead of
            // adding to every trip.
            const int nfull = nx & ~15;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            float w0 = 0.f, w1 = 0.f, w2 = 0.f, w3 = 0.f;
            if (nfull > 0) {
                a = *reinterpret_cast<const float4*>(xrow + ((g ^ xs_swz) << 2));
                w0 = wcol[0], w1 = wcol[it.fw], w2 = wcol[2 * it.fw], w3 = wcol[3 * it.fw];
            }
            for (int k0 = 0; k0 < nfull; k0 += 16) {
                float4 an = a;
                float v0 = w0, v1 = w1, v2 = w2, v3 = w3;
                if (k0 + 16 < nfull) {
                    an = *reinterpret_cast<const float4*>(xrow + (((((k0 + 16) >> 2) + g) ^ xs_swz) << 2));
                    const float* wk = wcol + (k0 + 16) * it.fw;
                    v0 = wk[0], v1 = wk[it.fw], v2 = wk[2 * it.fw], v3 = wk[3 * it.fw];
                }
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, w0, acc, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, w1, acc1, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, w2, acc2, 0, 0, 0);
                acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, w3, acc3, 0, 0, 0);
                a = an;
                w0 = v0, w1 = v1, w2 = v2, w3 = v3;
            }
            if (nfull < nx) {
                // the last, partial trip: every lane takes part in the matrix instruction; a
                // lane group whose four k lie past the end (nx % 4 == 0: all four or none)
                // reads the last valid ones instead and contributes zeros
                const bool ok = nfull + 4 * g < nx;
                const int kc = ok ? nfull : nx - 4 - 4 * g;
                float4 at = *reinterpret_cast<const float4*>(xrow + ((((kc >> 2) + g) ^ xs_swz) << 2));
                if (!ok) at = make_float4(0.f, 0.f, 0.f, 0.f);
                const float* wk = wcol + kc * it.fw;
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(at.x, wk[0], acc, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(at.y, wk[it.fw], acc1, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(at.z, wk[2 * it.fw], acc2, 0, 0, 0);
                acc3 = __builtin_amdgcn_mfma_f32_16x16x4f32(at.w, wk[3 * it.fw], acc3, 0, 0, 0);
            }
            acc = (acc + acc1) + (acc2 + acc3);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * mb + 4 * g + i;
                if (row < rows) bt[(c * kx + r0 + row) * it.fw + 16 * nb + col] = acc[i];
            }
        }
    };

    // The same on 32 x 32 blocks (channel sets whose tile is a multiple of 32 columns wide, where
    // the host asks for it with bit 3 of `staged`): a
    // block-trip of 16 k is eight matrix instructions of 64 cycles each fed by two 16-byte
    // reads of X_i and eight reads of W per lane - half the LDS reads per flop of the 16 x 16
    // form, and four times the matrix time per trip to hide their latency behind.  The
    // instruction sums over k in any order: lane half h takes k0 + 8h ... k0 + 8h + 7, which
    // are contiguous in the row of X_i.
    auto dense_rows32 = [&](int r0, int rows) {
        typedef float mfma16 __attribute__((ext_vector_type(16)));
        const int nb32 = it.fw >> 5;
        const int per_channel = ((rows + 31) >> 5) * nb32;
        const int blocks = per_channel * M;
        const int c32 = wl & 31, h = wl >> 5;
        for (int blk = wave; blk < blocks; blk += THREADS / 64) {
            const int c = blk / per_channel;
            const int rem = blk - c * per_channel;
            const int mb = rem / nb32, nb = rem - mb * nb32;
            const float bv = bias_s[c * it.fw + 32 * nb + c32];
            mfma16 acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = bv;
            const int arow = min(32 * mb + c32, rows - 1);     // rows past the end repeat the last
            const float* xrow = xs + arow * nx;
            const int xs_swz = arow & swz;
            const float* wcol = ws + (c * nx + 8 * h) * it.fw + 32 * nb + c32;
            const int nfull = nx & ~15;
            float4 a0 = make_float4(0.f, 0.f, 0.f, 0.f), a1 = a0;
            float w[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (nfull > 0) {
                a0 = *reinterpret_cast<const float4*>(xrow + (((2 * h) ^ xs_swz) << 2));
                a1 = *reinterpret_cast<const float4*>(xrow + (((2 * h + 1) ^ xs_swz) << 2));
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = wcol[j * it.fw];
            }
            for (int k0 = 0; k0 < nfull; k0 += 16) {
                float4 n0 = a0, n1 = a1;
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = w[j];
                if (k0 + 16 < nfull) {      // the next trip's operands, before this trip's instructions
                    const int q = ((k0 + 16) >> 2) + 2 * h;
                    n0 = *reinterpret_cast<const float4*>(xrow + ((q ^ xs_swz) << 2));
                    n1 = *reinterpret_cast<const float4*>(xrow + (((q + 1) ^ xs_swz) << 2));
                    const float* wk = wcol + (k0 + 16) * it.fw;
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[j] = wk[j * it.fw];
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, w[0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, w[1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, w[2], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, w[3], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, w[4], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, w[5], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, w[6], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, w[7], acc, 0, 0, 0);
                a0 = n0, a1 = n1;
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = v[j];
            }
            if (nfull < nx) {
                // the last, partial trip (4, 8 or 12 k): a lane whose k lies past the end reads
                // the row's first element instead and contributes zero
                const int left = nx - nfull;
                for (int j = 0; j < min(8, left); ++j) {
                    const bool ok = 8 * h + j < left;
                    const int k = ok ? nfull + 8 * h + j : 0;
                    float av = xrow[(((k >> 2) ^ xs_swz) << 2) + (k & 3)];
                    if (!ok) av = 0.f;
                    const float wv = ws[(c * nx + k) * it.fw + 32 * nb + c32];
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, wv, acc, 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = 32 * mb + 8 * (i >> 2) + 4 * h + (i & 3);
                if (row < rows) bt[(c * kx + r0 + row) * it.fw + 32 * nb + c32] = acc[i];
            }
        }
    };
    const bool blocks32 = SETS && (it.staged & 8) != 0 && (it.fw & 31) == 0;

    // ---- first pass: everything read from memory is requested at once (the first rows of
    // X_i, the weights, the bias, A_i)
    stage_tile4<THREADS>(xs, xg, P.ld_in, min(R, kx), xvec, tid, swz);
    stage_tile4<THREADS>(ws, P.w + it.f0, P.ld_w, M * nx, it.fw >> 2, tid);
    float bias_v = 0.f;
    if (tid < it.fw) bias_v = P.bias[it.f0 + tid];
    if (SETS) {
        LaunchParams Q = P;                                   // CSR from the merged arrays
        Q.w = reinterpret_cast<const float*>(P.rpt);
        stage_item<THREADS, 4, false, false, true>(Q, it, sm, tid);
        for (int e = tid + it.fw; e < M * it.fw; e += THREADS) {   // the other channels' bias
            const int c = e / it.fw;
            bias_s[e] = P.bias[(int64_t)c * P.fused_stride + it.f0 + (e - c * it.fw)];
        }
    } else {
        stage_item<THREADS, 4, false, false>(P, it, sm, tid);    // A_i only
    }
    if (tid < it.fw) bias_s[tid] = bias_v;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // direct-to-LDS loads landed
    __syncthreads();
    if (blocks32)
        dense_rows32(0, min(R, kx));
    else
        dense_rows(0, min(R, kx));
    __syncthreads();         // the rows of X_i may be replaced; after the last pass: tile complete
    // ---- operations with more rows than fit: further passes
    for (int r0 = R; r0 < kx; r0 += R) {
        const int rows = min(R, kx - r0);
        stage_tile4<THREADS>(xs, xg + (int64_t)r0 * P.ld_in, P.ld_in, rows, xvec, tid, swz);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (blocks32)
            dense_rows32(r0, rows);
        else
            dense_rows(r0, rows);
        __syncthreads();
    }
    compute_staged<THREADS, 4, false, ACC>(P, it, sm, tid);
}

// ---------------------------------------------------------------------------------------
// The layer (Fig. 7: one channel, or all channels with the ElementWiseAdd), gather first.  The sum is
// taken in the order
//     Y_i = [A_i^0 X_i | A_i^1 X_i | ...] [W[0]; W[1]; ...] + (row sums of A_i^ch) bias[ch],
// so that the gather moves rows of n_X floats instead of one dense tile of F columns per channel, the
// channels are summed by the matrix instructions, their results leave the registers as output rows, and no
// output row depends on another: the work is cut into blocks of R = 16 RB output rows whatever graph they
// belong to, all alike.  A kernel that runs once per plan (layer_rows_kernel) writes what the blocks
// read: for every output row and channel ("virtual row" R b M + row M + ch of block b) where its entries
// start, and the entries (row of X, value) one after the other.
//
// The dense part, Z (R x K, K = M n_X) times W (K x F), runs on bf16 matrix instructions without giving
// up fp32: every fp32 number is the sum of three bf16 numbers (24 = 3 x 8 bits: the rounded number, the
// rounded rest, the rest of that), and six of the nine products (all but those below 2^-26) are added in
// fp32, the large ones (hi x hi) in an accumulator of their own.  For 16 x 16 x 128 products that is 384
// cycles of a SIMD's matrix pipe instead of 1024 with v_mfma_f32_16x16x4_f32.  Error against 64 bits,
// products of uniform numbers, K = 64 / 256 / 512: 4.5e-8 / 8.1e-8 / 1.2e-7 of the result's norm; the fp32
// instructions 1.1e-7 / 2.1e-7 / 2.9e-7.  The parts of a small number would be subnormal, or below that: the
// values of A are taken times 2^48, the weights and the bias times 2^24 and the results times 2^-72, all
// exactly.  Every fp32 weight then has parts of 2^-125 and more, and what a Z below 2^-150 loses - less than
// 2^-174, were subnormal parts zero to the instructions - comes, with 512 weights of at most 2^16, to no more
// than the smallest fp32 number.  A split number that is not finite is NaN: blocks with results past 2^55 or not
// finite, and those of a wavefront with weights past 2^16, are made once more without the split, and in the order
// A (X W + bias): A X can leave the range of fp32 where the layer does not.  (A larger factor for A moves both
// bounds: more weights and fewer results.)
//   * W in REGISTERS for the whole launch, split once: wavefront w owns U blocks of 16 columns (12
//     registers per 32 of K and block); no LDS for W.
//   * A trip is one block.  While the matrix instructions of block b run, the rows of X that block b + 1
//     names are on their way to LDS (one 16-byte request per lane, each from its own row: a gather by the
//     memory system, one slot per entry in entry order), and the starts and entries of block b + 2.
//   * Gather: n_X / 4 lanes per virtual row add up the slots in stored order with fused multiply-adds,
//     split the sum and write the three bf16 planes of Z to LDS (rows 16 bytes apart from a multiple of
//     64, which spreads a column of 16 rows over the banks).
//   * The matrix phase computes the transposed block (W^T Z^T): a lane then holds consecutive columns of
//     an output row.  Results wait in registers and are stored at the top of the next trip, so that the
//     wait there finds only requests and stores that are a whole trip old; stores write whole 128-byte
//     lines (half lines: one channel, 2048 graphs, n_X = 64 20.5 us instead of 16.4).  With U = 1 a wavefront
//     writes half lines; non-temporal there too: cached stores would let the L2 join them but cost more (2048
//     graphs, n_X = 64: four channels 28.6 -> 29.9, one channel 15.7 -> 16.8).
// DIRECT: small layers of one channel, a block of 16 rows of one operation to a workgroup.  X_i, the
// operation's entries and its row pointers are requested at once and no other launch is needed (128 graphs,
// n_X = 64, F = 128: 4.8 us; the one-launch kernel 6.6.  With four wavefronts, before it took eight: 5.3; row
// pointers, entries and rows of X one after the other 5.7; from arrays built once per plan 4.9, but the first run 8
// us longer).
// Two barriers a trip.  us of a launch, F = 128, molecules, against the kernel this replaces, which made the
// dense tiles graph by graph with fp32 matrix instructions: four channels at n_X = 64, 2048 graphs 43.4 ->
// 28.0, 512 15.4 -> 12.5, 128 11.6 -> 7.1; n_X = 128, 2048 graphs 85.6 -> 57.3; eight channels at n_X = 64, 1024
// graphs 39.7 -> 31.7; one channel at n_X = 64, 2048 graphs 21.2 -> 15.7, 512 10.0 -> 7.1.  Bound at four
// channels (counters): the matrix pipe is busy for a quarter of the launch, waves wait for 44 %; a trip is a chain
// of LDS round trips and two barriers that two workgroups per CU hide from each other only in part, and
// splitting the weights is a fifth of the launch.
// ---------------------------------------------------------------------------------------

// Global -> LDS copy of 16 bytes per lane (lane i lands at lds_addr + 16 i), issued from inline assembly:
// the compiler then does not know that LDS is written behind its back and does not put a wait for ALL
// outstanding memory operations in front of the next LDS read.  The kernel waits for its requests
// itself, where it needs them.  (Untracked requests can only make the waits the compiler computes for
// its own loads longer, never shorter: the counter runs in issue order.)
__device__ __forceinline__ void lds_dma16_to(const void* gp, int lds_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(gp), "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory", "m0");
}

__device__ __forceinline__ int lds_address(const void* lds)
{
    return (int)(uintptr_t)((const __attribute__((address_space(3))) char*)lds);
}

// Workgroup barrier that orders LDS accesses only (no wait for global stores or for requests
// in flight, which __syncthreads would add).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Two fp32 numbers as three pairs of bf16 numbers whose sum they are (the first of a pair in the low half).
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo)
{
    auto pair = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2)); };
    hi = pair(a, b);
    const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xffff0000u);
    mid = pair(ra, rb);
    lo = pair(ra - __uint_as_float(mid << 16), rb - __uint_as_float(mid & 0xffff0000u));
}

constexpr float kValueScale = 0x1p48f, kWeightScale = 0x1p24f;     // (see above)

template <int KS, int U, int RB, int WV, bool DIRECT>
__global__ void __launch_bounds__(64 * WV, WV == 8 ? (KS > 8 ? 2 : 4) : (KS * U > 8 || (KS > 2 && U * RB > 2) ? 2 : 3))
bspmm_layer_kernel(const int32_t* __restrict__ starts, const int2* __restrict__ entries,
                   const int32_t* __restrict__ out_rows, const float* __restrict__ x, const float* __restrict__ wgt,
                   const float* __restrict__ bias, float* __restrict__ y, const LayerDirect D, const LayerShape S)
{
    extern __shared__ __align__(16) int sm[];
    constexpr int T = 64 * WV;                                // lanes: four or eight wavefronts
    constexpr int R = 16 * RB;                                // rows of a block
    constexpr int BQ = WV == 8 && KS <= 8 ? 1 : 2;            // four channels each
    constexpr int ZP = layer_z_row(KS), PLANE = R * ZP;      // bytes of a row / of a plane of Z
    int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int wl = tid & 63, col = wl & 15, g = wl >> 4;
    // Workgroups go to the XCDs round robin (index mod 8): a range of blocks and its feature tiles sit
    // on one XCD, and neighbouring ranges too, so that its L2 fetches the rows of X once.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int pair = S.tiles == 1 ? slot : (int)__umulhi((uint32_t)slot, S.inv_tiles);
    const int tile = slot - pair * S.tiles, range = xcd * S.ranges_per_xcd + pair;
    const int b0 = DIRECT ? range : range * S.blocks_each + min(range, S.blocks_over);
    const int b1 = DIRECT ? min(range + 1, S.blocks) : b0 + S.blocks_each + (range < S.blocks_over ? 1 : 0);
    if (b0 >= b1) return;
    // DIRECT: one channel, one block to a workgroup, 16 rows of one operation.  Its row pointers, all of the
    // operation's entries and all of X_i are requested at once (the slots are the rows of X_i, in their
    // order): one trip to memory instead of one for the row pointers, one for the entries, one for the rows
    // of X.
    LayerItem it;
    if constexpr (DIRECT) it = D.items[b0];
    const int M = S.channels, V = R * M;                      // virtual rows of a block
    const int lsh = S.lane_shift, L = 1 << lsh;               // n_X / 4 lanes per virtual row
    const int G = T >> lsh;
    int l = tid & (L - 1), grp = tid >> lsh;
    const int row_sh = lsh + 4;                               // a row of X in LDS is 16 << lsh bytes

    // ---- this wavefront's weights.  Block u has the columns f0 + U i + u, i < 16 (a lane's loads of a row are U columns side by side, and its
    // results U float4): the A operand is W^T, lane (g, col) holds W[32 s + 8 g + j][f0 + U col + u], j < 8 (all
    // eight inside K or none: K is a multiple of 16; where none the weights of k = j stand in, the columns of Z
    // there are zero)
    const int K = M << (lsh + 2);
    const int f0 = (tile * WV + wave) * (16 * U);
    const int width = min(16 * U, S.F - f0);                  // columns of this wavefront (none: negative)
    const int w_col = width > 0 ? f0 + U * min(col, width / U - 1) : 0;
    float raw[KS][8][U];
    auto request_weights = [&]() {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 32 * s + 8 * g;
            const uint32_t off = ((uint32_t)(k < K ? k : 0) * (uint32_t)S.ld_w + (uint32_t)w_col) << 2;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const char* p = reinterpret_cast<const char*>(wgt + j * S.ld_w) + off;
                if constexpr (U == 2) {
                    const float2 t = *reinterpret_cast<const float2*>(p);
                    raw[s][j][0] = t.x, raw[s][j][1] = t.y;
                } else {
                    raw[s][j][0] = *reinterpret_cast<const float*>(p);
                }
            }
        }
    };
    const LayerLds at = layer_lds(KS, RB, WV, M, S.slots, DIRECT ? S.entries : S.slots, 4 << lsh);
    char* const lds = reinterpret_cast<char*>(sm);
    char* const xs = lds + at.slots;            // the rows of X that the entries name
    uint32_t* const marks = reinterpret_cast<uint32_t*>(lds + at.marks);
    int* const z_place = reinterpret_cast<int*>(marks + WV * kLayerRedoWords);     // of every virtual row, in bytes
    const int csr_lds = lds_address(lds + at.csr), xs_lds = csr_lds - (at.csr - at.slots);

    // what the gather of block b reads -> csr buffer; its first entry is number e0 (as many entries as there
    // are slots, the block's or not: the array is that much longer)
    auto request_csr = [&](int b, int e0, int buf) {
        const int to = csr_lds + buf * at.csr_bytes;
        const uint32_t v = (uint32_t)b * (uint32_t)V;
        if (wave == 0) {
            for (int i = 0; 2 * i < S.slots; i += 64)
                if (2 * (i + wl) < S.slots) lds_dma16_to(entries + (uint32_t)((e0 & ~1) + 2 * (i + wl)), to + at.entries + 16 * i);
        } else if (wave == 1) {
            if (4 * wl < V + 1) lds_dma16_to(starts + (v + 4 * wl), to);
        } else if (wave == 2) {
            if (4 * wl < R) lds_dma16_to(out_rows + (uint32_t)(R * b + 4 * wl), to + at.rows);
        }
    };
    // rows of X of a block whose entries are in csr buffer `buf`
    auto request_rows = [&](int e0, int e1, int buf) {
        const int2* ent = reinterpret_cast<const int2*>(lds + at.csr + buf * at.csr_bytes + at.entries);
        const int n = min(e1 - (e0 & ~1), S.slots), per = 64 >> lsh;
        // (a request past the last entry asks for its row again; the slots are a multiple of a request's rows)
        for (int i0 = wave * per; i0 < n; i0 += 4 * WV * per) {
            uint32_t row[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) row[t] = (uint32_t)ent[min(i0 + WV * t * per + (wl >> lsh), n - 1)].x;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (i0 + WV * t * per < n)
                    lds_dma16_to(x + ((uint64_t)row[t] * (uint32_t)S.ld_x + 4 * l), xs_lds + ((i0 + WV * t * per) << row_sh));
        }
    };
    auto start_in = [&](int buf, int vr) {       // of the block whose starts are in that buffer
        return __builtin_amdgcn_readfirstlane(*reinterpret_cast<const int*>(lds + at.csr + buf * at.csr_bytes + 4 * vr));
    };

    int e_cur = 0, e_next = 0;
    if constexpr (DIRECT) {
        const char* xi = reinterpret_cast<const char*>(x + ((uint64_t)it.in_row * (uint32_t)S.ld_x + 4 * l));
        for (int i0 = wave * (64 >> lsh); i0 < it.k; i0 += T >> lsh) {
            const int r = min(i0 + (wl >> lsh), it.k - 1);
            lds_dma16_to(xi + (uint64_t)(uint32_t)r * ((uint32_t)S.ld_x * 4ull), xs_lds + (i0 << row_sh));
        }
        const int rp = D.rpt[it.rpt_off + (uint32_t)min(tid, it.nrows)];
        const int n = max(it.nnz, 1) - 1;
        const int c0 = it.nnz > 0 ? D.colids[it.nz_off + (uint32_t)min(tid, n)] : 0;
        const float a0 = it.nnz > 0 ? D.values[it.nz_off + (uint32_t)min(tid, n)] : 0.f;
        request_weights();
        int* st = reinterpret_cast<int*>(lds + at.csr);
        int2* ent = reinterpret_cast<int2*>(lds + at.csr + at.entries);      // (place in the slots, value)
        auto place_of = [&](int c) { return ((unsigned)c < (unsigned)it.k ? c : 0) << row_sh; };
        if (tid <= 16) st[tid] = min(max(rp, 0), it.nnz);
        if (tid < 16) *reinterpret_cast<int*>(lds + at.csr + at.rows + 4 * tid) = tid < it.nrows ? (int)it.out_row + tid : -1;
        if (tid < it.nnz) ent[tid] = make_int2(place_of(c0), __float_as_int(a0));
        for (int i = tid + T; i < it.nnz; i += T)
            ent[i] = make_int2(place_of(D.colids[it.nz_off + (uint32_t)i]), __float_as_int(D.values[it.nz_off + (uint32_t)i]));
        if (tid < kLayerSpare) ent[it.nnz + tid] = make_int2(0, 0);
        e_next = it.nnz;
    } else {
        e_cur = starts[(uint32_t)b0 * V], e_next = starts[(uint32_t)(b0 + 1) * V];
        request_csr(b0, e_cur, 0);
        if (b0 + 1 < b1) request_csr(b0 + 1, e_next, 1);
    }
    for (int i = tid; i < WV * kLayerRedoWords; i += T) marks[i] = 0;
    for (int i = tid; i < V; i += T) {
        const int r = (i * S.inv_channels) >> 16;
        z_place[i] = r * ZP + ((i - r * M) << (lsh + 3));
    }
    // slots that no request has filled yet hold finite numbers (see the gather)
    if constexpr (!DIRECT)
    for (int i = 16 * tid; i < (S.slots + kLayerSpare) << row_sh; i += 16 * T)
        *reinterpret_cast<float4*>(xs + i) = make_float4(0.f, 0.f, 0.f, 0.f);
    // the columns of Z past K (K off a multiple of 32) stay zero
    if (K < 32 * KS)
        for (int i = tid; i < 3 * PLANE / 4; i += T) sm[i] = 0;
    if constexpr (!DIRECT) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        lds_barrier();
        request_rows(e_cur, e_next, 0);
    }

    // (behind the first rows of X, which would wait for them: four channels at n_X = 64, 512 graphs 13.4 us
    // instead of 12.5)
    if constexpr (!DIRECT) request_weights();
    // ---- the weights, split once
    bf16x8 wh[U][KS], wm[U][KS], wlo[U][KS];
    float bv[U][BQ];
    bool huge;                                                // weights past 2^16 in this wavefront
    {
        float most = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint32_t h[4], m[4], lo[4];
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    v[j] = kWeightScale * raw[s][j][u];
                    most = fmaxf(most, fabsf(v[j]));
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) split2(v[2 * j], v[2 * j + 1], h[j], m[j], lo[j]);
                wh[u][s] = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
                wm[u][s] = __builtin_bit_cast(bf16x8, make_uint4(m[0], m[1], m[2], m[3]));
                wlo[u][s] = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
            }
        huge = __builtin_amdgcn_ballot_w64(most > 0x1p16f * kWeightScale) != 0;
        // bias as the A operand of v_mfma_f32_16x16x4_f32 (k = channel), the row sums are B
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < BQ; ++q) {
                const float t = bias[(int64_t)min(4 * q + g, M - 1) * S.bias_stride + w_col + (width > 0 ? u : 0)];
                bv[u][q] = 4 * q + g < M ? kWeightScale * t : 0.f;
            }
    }
    // The lane's place once more, here and in every trip of the loop below, so that nothing derived from it
    // is kept in registers from trip to trip: the weights leave none to spare.
    auto place = [&]() {
        asm volatile("" : "+v"(tid));
        wl = tid & 63, col = wl & 15, g = wl >> 4, l = tid & (L - 1), grp = tid >> lsh;
    };
    place();

    // Results wait here for the top of the next trip.  A lane has 4 U columns of output row `col` of every 16;
    // with U = 2 lanes eight rows apart exchange halves, so that a store writes whole lines: 128 bytes of rows
    // 0..7, then of rows 8..15.
    f32x4 pend[RB][U];
    int pend_row[RB][U];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int u = 0; u < U; ++u) pend_row[rb][u] = -1;
    auto store_pending = [&]() {
        const int c0 = U == 2 ? 8 * g + 4 * (col >> 3) : 4 * g;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (pend_row[rb][u] < 0 || c0 >= width) continue;
                float* yp = y + ((uint64_t)(uint32_t)pend_row[rb][u] * (uint32_t)S.ld_y + (uint32_t)(f0 + c0));
                float4 v = make_float4(pend[rb][u][0], pend[rb][u][1], pend[rb][u][2], pend[rb][u][3]);
                if (S.accumulate) {
                    const float4 old = *reinterpret_cast<const float4*>(yp);
                    v.x += old.x, v.y += old.y, v.z += old.z, v.w += old.w;
                }
                store_out<4>(yp, v);
            }
    };

    // Z of one block, `Q` virtual rows per lane group at a time, `J` entries of each at once.  (Lane groups
    // past the last virtual row repeat it; entries past a row's end are taken with value zero - where
    // their slot holds an infinity the sum is NaN, and so is the result: see the check behind the matrix
    // instructions.)  J = 0: blocks of more entries than slots.
    auto gather = [&](auto q_tag, auto j_tag, int e0, const char* csr) {
        constexpr int Q = decltype(q_tag)::value, J = decltype(j_tag)::value;
        static_assert(J <= kLayerSpare, "reads past the last entry");
        const int* st = reinterpret_cast<const int*>(csr);
        const int ea = e0 & ~1;                               // the entry of slot 0
        const char* x0 = xs + 16 * l;
        const char* v0 = csr + at.entries + 4;                // the entries' values
        float* const sums = reinterpret_cast<float*>(lds + at.sums);
        int p[Q], pe[Q], to[Q];
        auto fetch = [&](int r0) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int vr = min(r0 + q * G + grp, V - 1);
                p[q] = st[vr] - ea;
                pe[q] = st[vr + 1] - ea;
                to[q] = z_place[vr];
            }
        };
        fetch(0);
        for (int r0 = 0; r0 < V; r0 += Q * G) {
            float4 acc[Q];
            float sum[Q];                                 // of the row's values: what the bias is taken times
            int longest = 0;
            char* zp[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                sum[q] = 0.f;
                zp[q] = lds + to[q] + 8 * l;
            }
            if constexpr (DIRECT) {
                const char* ep = csr + at.entries;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    int2 en[J];
                    float4 xv[J];
#pragma unroll
                    for (int t = 0; t < J; ++t) en[t] = *reinterpret_cast<const int2*>(ep + ((p[q] + t) << 3));
#pragma unroll
                    for (int t = 0; t < J; ++t) xv[t] = *reinterpret_cast<const float4*>(x0 + en[t].x);
#pragma unroll
                    for (int t = 0; t < J; ++t) {
                        const float vt = p[q] + t < pe[q] ? kValueScale * __int_as_float(en[t].y) : 0.f;
                        Vec<4>::fma(acc[q], vt, xv[t]);
                        sum[q] += vt;
                    }
                    for (int i = p[q] + J; i < pe[q]; ++i) {
                        const int2 e = *reinterpret_cast<const int2*>(ep + (i << 3));
                        const float vt = kValueScale * __int_as_float(e.y);
                        Vec<4>::fma(acc[q], vt, *reinterpret_cast<const float4*>(x0 + e.x));
                        sum[q] += vt;
                    }
                }
            } else if constexpr (J > 0) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const char* xp = x0 + (p[q] << row_sh);
                    const char* vp = v0 + (p[q] << 3);
                    longest = max(longest, pe[q] - p[q]);
                    float4 xv[J];
                    float v[J];
#pragma unroll
                    for (int t = 0; t < J; ++t) {
                        xv[t] = *reinterpret_cast<const float4*>(xp + (t << row_sh));
                        v[t] = *reinterpret_cast<const float*>(vp + 8 * t);
                    }
#pragma unroll
                    for (int t = 0; t < J; ++t) {
                        const float vt = p[q] + t < pe[q] ? kValueScale * v[t] : 0.f;
                        Vec<4>::fma(acc[q], vt, xv[t]);
                        sum[q] += vt;
                    }
                }
                if (__any(longest > J))
                    for (int q = 0; q < Q; ++q)
                        for (int i = p[q] + J; i < pe[q]; ++i) {
                            const float vt = kValueScale * *reinterpret_cast<const float*>(v0 + (i << 3));
                            Vec<4>::fma(acc[q], vt, *reinterpret_cast<const float4*>(x0 + (i << row_sh)));
                            sum[q] += vt;
                        }
            } else {
                // The entries without a slot straight from memory, where the graph's rows of X are in the CU's
                // cache or the L2.  The lanes of a group request as many entries at once and pass them round:
                // one wait for them, not one for each (us, one channel, n_X = 64, F = 128, 2048 molecules of 24 /
                // 48 entries per row: 57 -> 44 / 114 -> 72).
                static_assert(Q == 1, "one row of a group at a time");
                constexpr int E = WV == 8 && KS <= 8 ? (KS == 8 ? 1 : 2) : 4;     // what the registers beside the weights hold
                auto add = [&](int n, auto entry) {                // entries 0 .. n - 1: (value, row of X)
                    for (int t0 = 0; t0 < n; t0 += E) {
                        float4 xv[E];
                        float v[E];
#pragma unroll
                        for (int t = 0; t < E; ++t) entry(min(t0 + t, n - 1), v[t], xv[t]);
#pragma unroll
                        for (int t = 0; t < E; ++t) {
                            const float vt = t0 + t < n ? kValueScale * v[t] : 0.f;
                            Vec<4>::fma(acc[0], vt, xv[t]);
                            sum[0] += vt;
                        }
                    }
                };
                int lane = tid;                                    // (see place)
                asm volatile("" : "+v"(lane));
                lane &= L - 1;
                const int top = S.slots;
                add(min(pe[0], top) - p[0], [&](int i, float& v, float4& xv) {
                    xv = *reinterpret_cast<const float4*>(x0 + ((p[0] + i) << row_sh));
                    v = *reinterpret_cast<const float*>(v0 + ((p[0] + i) << 3));
                });
                for (int i0 = max(p[0], top); i0 < pe[0]; i0 += L) {
                    const int2 en = entries[(uint32_t)(ea + min(i0 + lane, pe[0] - 1))];
                    add(min(L, pe[0] - i0), [&](int i, float& v, float4& xv) {
                        const uint32_t row = (uint32_t)__shfl(en.x, i, L);
                        v = __int_as_float(__shfl(en.y, i, L));
                        xv = load_vec<4>(x + ((uint64_t)row * (uint32_t)S.ld_x + 4 * lane));
                    });
                }
            }
            if (l == 0)
#pragma unroll
                for (int q = 0; q < Q; ++q) sums[min(r0 + q * G + grp, V - 1)] = sum[q];
            if (Q > 1 && r0 + Q * G < V) fetch(r0 + Q * G);   // the next rows' starts while these are split
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                uint2 h, m, lo;
                split2(acc[q].x, acc[q].y, h.x, m.x, lo.x);
                split2(acc[q].z, acc[q].w, h.y, m.y, lo.y);
                *reinterpret_cast<uint2*>(zp[q]) = h;
                *reinterpret_cast<uint2*>(zp[q] + PLANE) = m;
                *reinterpret_cast<uint2*>(zp[q] + 2 * PLANE) = lo;
            }
            if (Q == 1 && r0 + Q * G < V) fetch(r0 + Q * G);
        }
    };

    for (int b = b0; b < b1; ++b) {
        const int buf = (b - b0) & 1;
        const char* csr = lds + at.csr + buf * at.csr_bytes;
        place();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's requests for block b
        lds_barrier();                                     // everyone's; everyone is done with block b - 1
        store_pending();
        const int e_then = !DIRECT && b + 1 < b1 ? start_in(buf ^ 1, V) : 0;
        // (virtual rows in flight per lane: what the registers beside the weights hold)
        constexpr int kRows = WV == 8 ? (KS == 8 ? 1 : 2) : (KS * U <= 6 ? 4 : 2);
        std::integral_constant<int, 1> one;
        std::integral_constant<int, 2> two;
        const bool past = !DIRECT && e_next - (e_cur & ~1) > S.slots;
        if constexpr (!DIRECT)
            if (past) gather(one, std::integral_constant<int, 0>(), e_cur, csr);
        if (past)
            ;
        else if (V <= G || kRows == 1)
            gather(one, std::integral_constant<int, kRows == 1 ? 2 : 4>(), e_cur, csr);
        else if (M == 1)
            gather(two, std::integral_constant<int, kRows == 4 ? 4 : 2>(), e_cur, csr);
        else if (V <= 2 * G)
            gather(two, two, e_cur, csr);
        else
            gather(std::integral_constant<int, kRows>(), two, e_cur, csr);
        // this lane's output rows
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int u = 0; u < U; ++u)
                pend_row[rb][u] = *reinterpret_cast<const int*>(csr + at.rows + 4 * (16 * rb + (U == 2 ? 8 * u + (col & 7) : col)));
        lds_barrier();                                     // Z complete, slots and this csr buffer free
        place();
        if (!DIRECT && b + 1 < b1) request_rows(e_next, e_then, buf ^ 1);
        if (!DIRECT && b + 2 < b1) request_csr(b + 2, e_then, buf);
        float poison = 0.f;                                // NaN if one is not finite
        {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                f32x4 big[U], small[U];
                // the row sums are the B operand of the bias (row col, channel g)
                float rs[BQ];
#pragma unroll
                for (int q = 0; q < BQ; ++q)
                    rs[q] = *reinterpret_cast<const float*>(lds + at.sums + 4 * ((16 * rb + col) * M + min(4 * q + g, M - 1)));
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    small[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                    big[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[u][0], rs[0], small[u], 0, 0, 0);
                    if constexpr (BQ == 2)
                        if (M > 4) big[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[u][1], rs[1], big[u], 0, 0, 0);
                }
                const char* zr = lds + (16 * rb + col) * ZP + 16 * g;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const bf16x8 zh = *reinterpret_cast<const bf16x8*>(zr + 64 * s);
                    const bf16x8 zm = *reinterpret_cast<const bf16x8*>(zr + 64 * s + PLANE);
                    const bf16x8 zl = *reinterpret_cast<const bf16x8*>(zr + 64 * s + 2 * PLANE);
                    auto all = [&](f32x4* acc, const bf16x8(&w)[U][KS], const bf16x8& zz) {
#pragma unroll
                        for (int u = 0; u < U; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][s], zz, acc[u], 0, 0, 0);
                    };
                    all(big, wh, zh);
                    all(small, wh, zm);
                    all(small, wm, zh);
                    all(small, wm, zm);
                    all(small, wh, zl);
                    all(small, wlo, zh);
                }
                f32x4 r[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    r[u] = big[u] + small[u];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        poison = fmaf(r[u][i], 0.f, poison);
                        r[u][i] *= 1.f / (kValueScale * kWeightScale);
                    }
                }
                if constexpr (U == 2) {
                    const f32x4 q0 = {r[0][0], r[1][0], r[0][1], r[1][1]}, q1 = {r[0][2], r[1][2], r[0][3], r[1][3]};
                    const bool low = col < 8;
                    f32x4 got;
#pragma unroll
                    for (int i = 0; i < 4; ++i)          // row_ror:8 within 16 lanes
                        got[i] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(low ? q1[i] : q0[i]), 0x128, 0xf, 0xf, true));
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        pend[rb][0][i] = low ? q0[i] : got[i];
                        pend[rb][1][i] = low ? got[i] : q1[i];
                    }
                } else {
                    pend[rb][0] = r[0];
                }
            }
        }
        // Split numbers that are not finite (or round to infinity) are NaN: results that are not finite are made
        // again without the split, when there are no more blocks.
        if (huge || __builtin_amdgcn_ballot_w64(poison != poison) != 0) {
            if (wl == 0) marks[wave * kLayerRedoWords + ((b - b0) >> 5)] |= 1u << ((b - b0) & 31);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int u = 0; u < U; ++u) pend_row[rb][u] = -1;
        }
        e_cur = e_next;
        e_next = e_then;
    }
    store_pending();
    lds_barrier();                                            // everyone's marks
    place();
    {
        static_assert(WV * kLayerRedoWords <= 64, "a word to a lane");
        if (__builtin_amdgcn_ballot_w64(marks[min(wl, WV * kLayerRedoWords - 1)] != 0) == 0) return;
    }
    // The blocks that the split or the order of the sums does not hold: A (X W + bias), as the layer is written,
    // on fp32 matrix instructions.  One 16 x 16 product makes 16 columns of X W[ch] + bias[ch] for the p-th
    // entry of each of 16 rows, so the lanes that hold a row's columns add them up in stored order; rows with
    // fewer entries in the channel leave theirs out.  (k is taken in the order in which a lane's float4 of X
    // has it.)  The wavefronts take the marked (block, columns) in turn, whoever marked them: one weight that is
    // not finite marks every block, but of one wavefront.  us, four channels at n_X = 64, F = 128, 2048 molecules:
    // nothing marked 32, one weight NaN 60, everything marked 204 (each lane on its own, one product after the
    // other: 977 and 1600; by the wavefront that marked them 156 and 245; two entries at once 62 and 202).  Bound
    // by the loads of X and W, a row of X and the channel's weights once more for every entry.
    for (int turn = 0, word = 0; word < WV * kLayerRedoWords; ++word)
    for (uint32_t left = __builtin_amdgcn_readfirstlane(marks[word]); left != 0; left &= left - 1, ++turn) {
        if (turn % WV != wave) continue;
        const int b = b0 + 32 * (word % kLayerRedoWords) + __builtin_ctz(left);
        const int f1 = (tile * WV + word / kLayerRedoWords) * (16 * U), columns = min(16 * U, S.F - f1);
        if (columns <= 0) continue;
        // (one sixteen of columns at a time: two at once would take registers, and so workgroups, from every launch)
#pragma unroll 1
        for (int part = 0; part < RB * U; ++part) {
            const int rb = part / U, c0 = f1 + 16 * (part % U);
            if (16 * (part % U) >= columns) continue;
            const int row = DIRECT ? *reinterpret_cast<const int*>(lds + at.csr + at.rows + 4 * col)
                                   : out_rows[(uint32_t)(R * b + 16 * rb + col)];
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
            for (int ch = 0; ch < M; ++ch) {
                const uint32_t vr = (uint32_t)b * V + (uint32_t)((16 * rb + col) * M + ch);
                const int* st = reinterpret_cast<const int*>(lds + at.csr);
                const int first = DIRECT ? st[col] : starts[vr], count = (DIRECT ? st[col + 1] : starts[vr + 1]) - first;
                if (__builtin_amdgcn_ballot_w64(count > 0) == 0) continue;
                auto entry = [&](int i) {                     // (row of X, value)
                    if constexpr (DIRECT) {
                        const int2 e = reinterpret_cast<const int2*>(lds + at.csr + at.entries)[i];
                        return make_int2((int)it.in_row + (e.x >> row_sh), e.y);
                    } else {
                        return entries[(uint32_t)i];
                    }
                };
                int2 en = make_int2(0, 0);
                if (count > 0) en = entry(first);
                f32x4 bias4;
#pragma unroll
                for (int i = 0; i < 4; ++i) bias4[i] = bias[ch * S.bias_stride + c0 + 4 * g + i];
                const float* wp = wgt + (int64_t)(ch * 4 * L + 4 * g) * S.ld_w + (c0 + col);
                for (int p = 0;; ++p) {
                    const bool mine = p < count;
                    const unsigned long long has = __builtin_amdgcn_ballot_w64(mine);
                    if (has == 0) break;
                    // (lanes without an entry: the row of X that another one names)
                    const int other = __builtin_amdgcn_readlane(en.x, __builtin_ctzll(has));
                    const float* xp = x + ((uint64_t)(uint32_t)(mine ? en.x : other) * (uint32_t)S.ld_x + 4 * g);
                    const float v = __int_as_float(en.y);
                    if (p + 1 < count) en = entry(first + p + 1);
                    f32x4 acc = bias4;
                    // (sixteen k a trip, the next ones requested before these are multiplied)
                    float4 xn = load_vec<4>(xp);
                    float wn[4];
                    auto weights_at = [&](int k) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) wn[j] = wp[(uint32_t)(k + j) * (uint32_t)S.ld_w];
                    };
                    weights_at(0);
#pragma unroll 1
                    for (int k = 16; k <= 4 * L; k += 16) {
                        const float4 xv = xn;
                        float w[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) w[j] = wn[j];
                        if (k < 4 * L) {
                            xn = load_vec<4>(xp + k);
                            weights_at(k);
                        }
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[0], xv.x, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[1], xv.y, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[2], xv.z, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[3], xv.w, acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (mine) sum[i] = fmaf(v, acc[i], sum[i]);
                }
            }
            if (row < 0) continue;
            float* yp = y + ((uint64_t)(uint32_t)row * (uint32_t)S.ld_y + (uint32_t)(c0 + 4 * g));
            float4 v = make_float4(sum[0], sum[1], sum[2], sum[3]);
            if (S.accumulate) {
                const float4 old = *reinterpret_cast<const float4*>(yp);
                v.x += old.x, v.y += old.y, v.z += old.z, v.w += old.w;
            }
            store_out<4>(yp, v);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Direct product for COO / SparseTensor operands (Fig. 3 with the output staged on chip as in
// Fig. 5(a,b)), in two forms per item (item.mode):
//  * sorted: the workgroup counts the operation's entries per output row (integer LDS atomics),
//    scans the counts, scatters (dense row, value) pairs into row order in LDS and sums each row
//    in registers, a lane group per row: no floating-point atomics and no output tile.  The
//    dense tile sits in LDS beside the pairs where the scheduler found room; otherwise the dense
//    rows are read from memory, eight in flight per group.
//  * the paper's form: the item's output tile lives in LDS; a group of L lanes takes one stored
//    entry at a time (L = the tile's vectors per row rounded up to a power of two, at most 64),
//    reads the dense row it names and adds value * row into the tile with LDS floating-point
//    atomics; the tile is then streamed out.  Four entries per group are in flight at once.
//    What the paper reads from global memory entry by entry - the index pairs, the values and
//    the dense rows - is first copied to LDS in bulk where the scheduler found room: a
//    workgroup then pays one round trip to memory instead of one per entry.
// Entries outside the item's row range (or outside the matrix) are skipped.
// ---------------------------------------------------------------------------------------
template <int VEC>
__global__ void __launch_bounds__(kThreads)
bspmm_coo_kernel(const CooLaunchParams P)
{
    extern __shared__ __align__(16) float tile[];
    using V = typename Vec<VEC>::type;
    const CooItem it = P.items[blockIdx.x];
    const int tid = threadIdx.x;
    const int stride = round_up(it.fw, 4);
    const int nvec = (it.fw + VEC - 1) / VEC;          // VEC == 4 implies fw % 4 == 0
    const bool st_b = (it.mode & 1) != 0, st_e = (it.mode & 2) != 0;
    const bool sorted = (it.mode & 4) != 0 && st_e;
    float* bt = sorted ? tile : tile + it.nrows * stride;
    int2* ent = reinterpret_cast<int2*>(bt + (st_b ? it.k * stride : 0));
    float* ev = reinterpret_cast<float*>(ent + it.nnz);

    const int log2L = ilog2(min(64, pow2_ceil(nvec)));
    const int L = 1 << log2L;
    const int lane = tid & (L - 1);
    const int grp = tid >> log2L;
    const int G = kThreads >> log2L;
    const int32_t* __restrict__ id = P.ids + 2 * it.nz_off;
    const float* __restrict__ va = P.values + it.nz_off;
    const int sel = P.transposed ? 1 : 0;
    const float* __restrict__ in = P.in + it.in_row_off * P.ld_in + it.f0;

    // Items the host marked so (mode bit 2) sort their entries by output row on chip - count
    // per row, scan, scatter of (dense row, value) pairs into row order - and then run the row
    // gather of the CSR kernels over them: no floating-point atomics and no output tile, a
    // row's sum is kept in registers and stored once.  The pairs take the place of the staged
    // entries; behind them sit the row counts and the row pointers.
    int2* sp = ent;
    int* s_cnt = reinterpret_cast<int*>(sp + it.nnz);
    int* s_rp = s_cnt + it.nrows + 1;

    // ---- staging: every load is issued before anything is waited for
    bool direct = false;
    if (st_b) {
        direct = VEC == 4 && (nvec & (nvec - 1)) == 0;      // then stride == fw: rows are packed
        if (direct) {
            const int sh = ilog2(nvec);
            const int total = it.k << sh;                    // float4 in the tile
            const int wl = tid & 63;
            for (int e0 = (tid >> 6) << 6; e0 < total; e0 += kThreads) {
                const int e = e0 + wl;
                if (e < total) {
                    const float* gp = in + (int64_t)(e >> sh) * P.ld_in + ((e & (nvec - 1)) << 2);
                    __builtin_amdgcn_global_load_lds(
                        (const void __attribute__((address_space(1)))*)gp,
                        (void __attribute__((address_space(3)))*)(bt + (e0 << 2)), 16, 0, 0);
                }
            }
        } else {
            for (int r0 = grp; r0 < it.k; r0 += 4 * G)
                for (int j = lane; j < nvec; j += L) {
                    V t[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (r0 + u * G < it.k)
                            t[u] = load_vec<VEC>(in + (int64_t)(r0 + u * G) * P.ld_in + j * VEC);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (r0 + u * G < it.k) store_vec<VEC>(bt + (r0 + u * G) * stride + j * VEC, t[u]);
                }
        }
    }
    if (sorted) {
        __shared__ int wave_sum[kThreads / 64];
        __shared__ int carry;
        // The first four entries of every lane stay in registers between the count and the
        // scatter; what lies beyond them is read again.
        constexpr int KEEP = 4;
        int kr[KEEP], kc[KEEP];
        float kv[KEEP];
        auto entry = [&](int p, int& r, int& c, float& v) {
            r = id[2 * p + sel] - it.row0;
            c = id[2 * p + 1 - sel];
            v = va[p];
        };
#pragma unroll
        for (int u = 0; u < KEEP; ++u) {
            const int p = tid + u * kThreads;
            kr[u] = -1;
            kc[u] = 0;
            kv[u] = 0.f;
            if (p < it.nnz) entry(p, kr[u], kc[u], kv[u]);
        }
        for (int i = tid; i <= it.nrows; i += kThreads) s_cnt[i] = 0;
        lds_barrier();
#pragma unroll
        for (int u = 0; u < KEEP; ++u) {
            if (!((unsigned)kr[u] < (unsigned)it.nrows && (unsigned)kc[u] < (unsigned)it.k)) kr[u] = -1;
            if (kr[u] >= 0) atomicAdd(&s_cnt[kr[u]], 1);
        }
        for (int p = tid + KEEP * kThreads; p < it.nnz; p += kThreads) {
            int r, c;
            float v;
            entry(p, r, c, v);
            if ((unsigned)r < (unsigned)it.nrows && (unsigned)c < (unsigned)it.k) atomicAdd(&s_cnt[r], 1);
        }
        if (tid == 0) carry = 0;
        lds_barrier();
        // exclusive scan over the rows, 256 at a time (the counts are cleared for the scatter)
        const int wv = tid >> 6, wlane = tid & 63;
        for (int base = 0; base < it.nrows; base += kThreads) {
            const int i = base + tid;
            const int c = i < it.nrows ? s_cnt[i] : 0;
            int x = c;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off);
                if (wlane >= off) x += y;
            }
            if (wlane == 63) wave_sum[wv] = x;
            lds_barrier();
            int before = carry;
            for (int q = 0; q < wv; ++q) before += wave_sum[q];
            if (i < it.nrows) {
                s_rp[i] = before + x - c;
                s_cnt[i] = 0;
            }
            lds_barrier();
            if (tid == kThreads - 1) carry = before + x;
            lds_barrier();
        }
        if (tid == 0) s_rp[it.nrows] = carry;
        // (dense row, value) pairs in row order (inside a row: the order the lanes get there)
#pragma unroll
        for (int u = 0; u < KEEP; ++u)
            if (kr[u] >= 0)
                sp[s_rp[kr[u]] + atomicAdd(&s_cnt[kr[u]], 1)] =
                    make_int2(st_b ? kc[u] * stride : kc[u], __float_as_int(kv[u]));
        for (int p = tid + KEEP * kThreads; p < it.nnz; p += kThreads) {
            int r, c;
            float v;
            entry(p, r, c, v);
            if ((unsigned)r < (unsigned)it.nrows && (unsigned)c < (unsigned)it.k)
                sp[s_rp[r] + atomicAdd(&s_cnt[r], 1)] = make_int2(st_b ? c * stride : c, __float_as_int(v));
        }
        if (direct) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
        __syncthreads();
        // row gather: one lane group per output row; four entries in flight from LDS, eight
        // from memory
        float* outp = P.out + (it.out_row_off + it.row0) * P.ld_out + it.f0;
        auto gather = [&](auto width) {
            constexpr int W = decltype(width)::value;
            for (int rr = grp; rr < it.nrows; rr += G) {
                const int q0 = s_rp[rr], q1 = s_rp[rr + 1];
                for (int j = lane; j < nvec; j += L) {
                    V acc = Vec<VEC>::zero();
                    for (int q = q0; q < q1; q += W) {
                        int2 e[W];
#pragma unroll
                        for (int u = 0; u < W; ++u) e[u] = sp[min(q + u, q1 - 1)];
                        V b[W];
#pragma unroll
                        for (int u = 0; u < W; ++u)
                            b[u] = st_b ? load_vec<VEC>(bt + e[u].x + j * VEC)
                                        : load_vec<VEC>(in + (int64_t)e[u].x * P.ld_in + j * VEC);
#pragma unroll
                        for (int u = 0; u < W; ++u) {
                            const float v = q + u < q1 ? __int_as_float(e[u].y) : 0.f;
                            float* af = reinterpret_cast<float*>(&acc);
                            const float* bf = reinterpret_cast<const float*>(&b[u]);
#pragma unroll
                            for (int c = 0; c < VEC; ++c) af[c] = fmaf(v, bf[c], af[c]);
                        }
                    }
                    store_out<VEC>(outp + (int64_t)rr * P.ld_out + j * VEC, acc);
                }
            }
        };
        if (st_b) gather(std::integral_constant<int, 4>{});
        else gather(std::integral_constant<int, 8>{});
        return;
    }

    if (st_e) {
        for (int p0 = tid; p0 < it.nnz; p0 += 2 * kThreads) {
            int r[2], c[2];
            float v[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int p = p0 + u * kThreads;
                if (p < it.nnz) {
                    r[u] = id[2 * p + sel] - it.row0;
                    c[u] = id[2 * p + 1 - sel];
                    v[u] = va[p];
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int p = p0 + u * kThreads;
                if (p < it.nnz) {
                    const bool ok = (unsigned)r[u] < (unsigned)it.nrows && (unsigned)c[u] < (unsigned)it.k;
                    ent[p] = make_int2(ok ? r[u] * stride : -1, st_b ? c[u] * stride : c[u]);
                    ev[p] = v[u];
                }
            }
        }
    }
    {
        float4* t4 = reinterpret_cast<float4*>(tile);
        const int n4 = it.nrows * (stride >> 2);
        for (int i = tid; i < n4; i += kThreads) t4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (direct) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // direct-to-LDS loads landed
    __syncthreads();

    // ---- one lane group per entry
    constexpr int U = 4;
    for (int p0 = grp; p0 < it.nnz; p0 += U * G) {
        int ro[U], co[U];
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = p0 + u * G;
            ro[u] = -1;
            co[u] = 0;
            v[u] = 0.f;
            if (p < it.nnz) {
                if (st_e) {
                    const int2 e = ent[p];
                    ro[u] = e.x;
                    co[u] = e.y;
                    v[u] = ev[p];
                } else {
                    const int r = id[2 * p + sel] - it.row0;
                    const int c = id[2 * p + 1 - sel];
                    v[u] = va[p];
                    if ((unsigned)r < (unsigned)it.nrows && (unsigned)c < (unsigned)it.k) {
                        ro[u] = r * stride;
                        co[u] = c;             // mode bit 0 is never set without bit 1
                    }
                }
            }
        }
        for (int j = lane; j < nvec; j += L) {
            V b[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (ro[u] >= 0)
                    b[u] = st_b ? load_vec<VEC>(bt + co[u] + j * VEC)
                                : load_vec<VEC>(in + (int64_t)co[u] * P.ld_in + j * VEC);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (ro[u] >= 0) {
                    float* dst = tile + ro[u] + j * VEC;
                    const float* bf = reinterpret_cast<const float*>(&b[u]);
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        __hip_atomic_fetch_add(dst + e, v[u] * bf[e], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
        }
    }
    __syncthreads();

    float* out = P.out + (it.out_row_off + it.row0) * P.ld_out + it.f0;
    for (int rr = grp; rr < it.nrows; rr += G)
        for (int j = lane; j < nvec; j += L)
            store_out<VEC>(out + (int64_t)rr * P.ld_out + j * VEC,
                           load_vec<VEC>(tile + rr * stride + j * VEC));
}

// ---------------------------------------------------------------------------------------
// structural check: *flag becomes the smallest index of a malformed operation.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
validate_csr_kernel(const OpRecord* __restrict__ ops, const int32_t* __restrict__ rpt,
                    const int32_t* __restrict__ colids, int32_t* flag)
{
    const OpRecord o = ops[blockIdx.x];
    const int tid = threadIdx.x;
    bool bad = false;
    if (o.m > 0) {
        const int32_t* rp = rpt + o.rpt_off;
        if (tid == 0 && (rp[0] != 0 || rp[o.m] != o.nnz)) bad = true;
        for (int r = tid; r < o.m; r += kThreads)
            if (rp[r + 1] < rp[r]) bad = true;
    } else if (o.nnz != 0) {
        bad = true;
    }
    const int32_t* ci = colids + o.nz_off;
    for (int p = tid; p < o.nnz; p += kThreads)
        if ((unsigned)ci[p] >= (unsigned)o.k) bad = true;
    if (bad) atomicMin(flag, (int)blockIdx.x);
}

__global__ void fill_i32_kernel(int32_t* p, int32_t v, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------------------
// host-side launchers (the only symbols the rest of the library sees)
// ---------------------------------------------------------------------------------------
using KernelFn = void (*)(const LaunchParams);

static KernelFn kernel_variant(bool vec4, bool slices, bool hubs, bool merged = false)
{
    static const KernelFn table[16] = {
        bspmm_kernel<1, false, false>, bspmm_kernel<1, false, true>,
        bspmm_kernel<1, true, false>,  bspmm_kernel<1, true, true>,
        bspmm_kernel<4, false, false>, bspmm_kernel<4, false, true>,
        bspmm_kernel<4, true, false>,  bspmm_kernel<4, true, true>,
        bspmm_kernel<1, false, false, true>, bspmm_kernel<1, false, true, true>,
        bspmm_kernel<1, true, false, true>,  bspmm_kernel<1, true, true, true>,
        bspmm_kernel<4, false, false, true>, bspmm_kernel<4, false, true, true>,
        bspmm_kernel<4, true, false, true>,  bspmm_kernel<4, true, true, true>};
    return table[(merged ? 8 : 0) + (vec4 ? 4 : 0) + (slices ? 2 : 0) + (hubs ? 1 : 0)];
}

// Workgroups of bspmm_kernel the current device holds at once (0 if it cannot be asked).
int bspmm_max_resident_workgroups(int lds_bytes, bool slices, bool hubs)
{
    int per_cu4 = 0, per_cu1 = 0, dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu4, kernel_variant(true, slices, hubs),
                                                         kThreads, (size_t)lds_bytes);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu1, kernel_variant(false, slices, hubs),
                                                         kThreads, (size_t)lds_bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    const int per_cu = per_cu4 < per_cu1 ? per_cu4 : per_cu1;
    return per_cu > 0 && cus > 0 ? per_cu * cus : 0;
}

// Copy from pinned host memory (plan creation, see staging.hpp): every workgroup copies its 16-byte words
// and then writes `mark` to its word of `done`, also pinned: the host may reuse what it has read.
// Bound: the round trip over PCIe (160 KB: about 6 us).
__global__ void __launch_bounds__(kThreads)
stage_copy_kernel(const uint4* __restrict__ from, uint4* __restrict__ to, uint32_t words, uint32_t* done, uint32_t mark)
{
    const uint32_t step = gridDim.x * kThreads;
    uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    for (; i + step < words; i += 2 * step) {
        const uint4 a = from[i], b = from[i + step];
        to[i] = a;
        to[i + step] = b;
    }
    if (i < words) to[i] = from[i];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(done + blockIdx.x, mark, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// hipLaunchKernel with its arguments in place: 0.15 us less host time than the <<< >>> form, which
// pushes and pops the launch configuration around it.
template <typename... P>
static hipError_t launch(void (*fn)(P...), int grid, int threads, int lds_bytes, hipStream_t stream,
                         typename std::common_type<P>::type... args)
{
    void* p[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3(grid), dim3(threads), p,
                                         (size_t)lds_bytes, stream);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}


// Registers, LDS and occupancy of kernel `which` (BSPMM_KERNEL_* of the public header) on the
// current device.  out: vgprs, sgprs, static LDS, scratch, lanes per workgroup, workgroups per CU
// at `lds_bytes` of dynamic LDS, compute units.
hipError_t kernel_resources(int which, int lds_bytes, int out[7])
{
    const void* fn = nullptr;
    int threads = kThreads;
    switch (which) {
        case 0: fn = reinterpret_cast<const void*>(&bspmm_lean_kernel<false>); break;
        case 1: fn = reinterpret_cast<const void*>(&bspmm_kernel<4, false, false, false>); break;
        case 2: fn = reinterpret_cast<const void*>(&bspmm_kernel<1, false, false, false>); break;
        case 3: fn = reinterpret_cast<const void*>(&bspmm_gcn_kernel<false, false>); break;
        case 4: fn = reinterpret_cast<const void*>(&bspmm_gcn_kernel<false, true>); break;
        case 5: fn = reinterpret_cast<const void*>(&build_sorted_kernel<false, kThreads>); break;
        case 6:
            fn = reinterpret_cast<const void*>(&build_sorted_kernel<false, kBuildThreadsLarge>);
            threads = kBuildThreadsLarge;
            break;
        case 7: fn = reinterpret_cast<const void*>(&bspmm_coo_kernel<4>); break;
        case 8:
            fn = reinterpret_cast<const void*>(&bspmm_layer_kernel<8, 1, 1, 8, false>);
            threads = 512;
            break;
        default: return hipErrorInvalidValue;
    }
    hipFuncAttributes a;
    hipError_t e = hipFuncGetAttributes(&a, fn);
    if (e != hipSuccess) return e;
    int per_cu = 0, dev = 0, cus = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, (size_t)lds_bytes);
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    out[0] = a.numRegs;
    out[1] = 0;
    out[2] = (int)a.sharedSizeBytes;
    out[3] = (int)a.localSizeBytes;
    out[4] = threads;
    out[5] = per_cu;
    out[6] = cus;
    return hipSuccess;
}

hipError_t launch_stage_copy(const void* from, void* to, size_t bytes, uint32_t* done, uint32_t mark, int grid,
                             hipStream_t stream)
{
    return launch(stage_copy_kernel, grid, kThreads, 0, stream, static_cast<const uint4*>(from),
                  static_cast<uint4*>(to), (uint32_t)(bytes / 16), done, mark);
}

hipError_t launch_bspmm(const LaunchParams& P, int grid, int lds_bytes, bool vec4, bool slices,
                        bool hubs, bool merged, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    return launch(kernel_variant(vec4, slices, hubs, merged), grid, kThreads, lds_bytes, stream, P);
}

// first: the row blocks of these items have no entry ranges yet (see block_entries).
hipError_t launch_bspmm_lean(const LeanItem* items, const LaunchParams& P, int grid, int lds_bytes, bool merged, bool first,
                             hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    auto* const fn = merged ? (first ? bspmm_lean_kernel<true, true> : bspmm_lean_kernel<true>)
                            : (first ? bspmm_lean_kernel<false, true> : bspmm_lean_kernel<false>);
    return launch(fn, grid, kThreads, lds_bytes, stream, items,
                  P.rpt, P.colids, P.values, P.in, P.out, (uint32_t)P.ld_in, (uint32_t)P.ld_out,
                  (uint32_t)(lds_bytes / 4), reinterpret_cast<const int32_t*>(P.w));
}

hipError_t launch_first_transposed(const LeanItem* items, const LaunchParams& P, int grid, int lds_bytes, int32_t* rpt_t,
                                   int32_t* colids_t, float* values_t, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    return launch(bspmm_first_transposed_kernel, grid, kThreads, lds_bytes, stream, items, P.rpt, P.colids, P.values,
                  P.in, P.out, (uint32_t)P.ld_in, (uint32_t)P.ld_out, rpt_t, colids_t, values_t);
}

// aligned: F % 4 == 0 and every row of every tile is float4 on 16 bytes; quads: F % 4 == 0 (the schedule
// then left no room for rows off 16 bytes in LDS).
hipError_t launch_bspmm_any(const LeanItem* items, const LaunchParams& P, bool aligned, bool quads, bool first, int grid,
                            int lds_bytes, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    const bool windows = (reinterpret_cast<uintptr_t>(P.in) & 15) == 0 && (!quads || P.ld_in % 4 == 0);
    auto* const fn = aligned ? (first ? bspmm_any_kernel<true, true> : bspmm_any_kernel<true>)
                             : (first ? bspmm_any_kernel<false, true> : bspmm_any_kernel<false>);
    return launch(fn, grid, kThreads, lds_bytes, stream, items,
                  P.rpt, P.colids, P.values, P.in, P.out, P.ld_in, P.ld_out, (uint32_t)(lds_bytes / 4),
                  (windows ? kAnyWindows : 0) | (quads ? kAnyTight : 0), reinterpret_cast<const int32_t*>(P.w));
}

hipError_t launch_lean_hints(LeanItem* items, int n, const int32_t* rpt, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    return launch(lean_hints_kernel, (n + 255) / 256, 256, 0, stream, items, n, rpt);
}

using FrontFn = void (*)(const LaunchParams);

static FrontFn front_variant(bool accumulate, bool sets, bool wide)
{
    static const FrontFn table[8] = {
        bspmm_gcn_kernel<false, false>, bspmm_gcn_kernel<true, false>,
        bspmm_gcn_kernel<false, true>, bspmm_gcn_kernel<true, true>,
        bspmm_gcn_kernel<false, false, 2 * kThreads>, bspmm_gcn_kernel<true, false, 2 * kThreads>,
        bspmm_gcn_kernel<false, true, 2 * kThreads>, bspmm_gcn_kernel<true, true, 2 * kThreads>};
    return table[(wide ? 4 : 0) + (sets ? 2 : 0) + (accumulate ? 1 : 0)];
}

// Workgroups of the one-launch layer kernel one CU of the current device holds (0 if it cannot
// be asked); wide: workgroups of eight wavefronts.
int front_workgroups_per_cu(bool sets, bool wide, int lds_bytes)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, front_variant(false, sets, wide),
                                                     wide ? 2 * kThreads : kThreads, (size_t)lds_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu;
}

hipError_t launch_bspmm_gcn(const LaunchParams& P, int grid, int lds_bytes, bool accumulate,
                            bool sets, bool wide, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    return launch(front_variant(accumulate, sets, wide), grid, wide ? 2 * kThreads : kThreads, lds_bytes, stream, P);
}

using LayerFn = void (*)(const int32_t*, const int2*, const int32_t*, const float*, const float*, const float*, float*,
                         const LayerDirect, const LayerShape);

// (steps of 32 of K, 16-column blocks per wavefront, 16-row blocks per trip - 0: from an operation's own CSR
// arrays -, wavefronts) -> kernel; null for what it is not built for
static LayerFn layer_variant(int ks, int units, int rb, int waves)
{
    static const struct { int ks, units, rb, waves; LayerFn fn; } table[] = {
#define BSPMM_LAYER(K, U, R, W) {K, U, R, W, bspmm_layer_kernel<K, U, R, W, false>}
#define BSPMM_LAYER_DIRECT(K, U, W) {K, U, 0, W, bspmm_layer_kernel<K, U, 1, W, true>}
        BSPMM_LAYER_DIRECT(1, 1, 4), BSPMM_LAYER_DIRECT(1, 2, 4), BSPMM_LAYER_DIRECT(2, 1, 4), BSPMM_LAYER_DIRECT(2, 1, 8),
        BSPMM_LAYER_DIRECT(4, 1, 4), BSPMM_LAYER_DIRECT(4, 1, 8),
        BSPMM_LAYER(1, 1, 1, 4), BSPMM_LAYER(1, 1, 2, 4), BSPMM_LAYER(1, 1, 4, 4), BSPMM_LAYER(1, 2, 1, 4),
        BSPMM_LAYER(1, 2, 2, 4), BSPMM_LAYER(1, 2, 4, 4), BSPMM_LAYER(2, 1, 1, 4), BSPMM_LAYER(2, 1, 2, 4),
        BSPMM_LAYER(2, 2, 1, 4), BSPMM_LAYER(2, 2, 2, 4), BSPMM_LAYER(3, 1, 1, 4), BSPMM_LAYER(3, 1, 2, 4),
        BSPMM_LAYER(3, 2, 1, 4), BSPMM_LAYER(3, 2, 2, 4), BSPMM_LAYER(4, 1, 1, 4), BSPMM_LAYER(4, 1, 2, 4),
        BSPMM_LAYER(4, 2, 1, 4), BSPMM_LAYER(4, 2, 2, 4), BSPMM_LAYER(6, 1, 1, 4), BSPMM_LAYER(6, 2, 1, 4),
        BSPMM_LAYER(8, 1, 1, 4), BSPMM_LAYER(8, 2, 1, 4), BSPMM_LAYER(12, 1, 1, 4), BSPMM_LAYER(16, 1, 1, 4),
        BSPMM_LAYER(2, 1, 1, 8), BSPMM_LAYER(2, 1, 2, 8),
        BSPMM_LAYER(3, 1, 1, 8), BSPMM_LAYER(3, 1, 2, 8), BSPMM_LAYER(4, 1, 1, 8), BSPMM_LAYER(4, 1, 2, 8),
        BSPMM_LAYER(6, 1, 1, 8), BSPMM_LAYER(8, 1, 1, 8), BSPMM_LAYER(12, 1, 1, 8), BSPMM_LAYER(16, 1, 1, 8)};
#undef BSPMM_LAYER
#undef BSPMM_LAYER_DIRECT
    for (const auto& v : table)
        if (v.ks == ks && v.units == units && v.rb == rb && v.waves == waves) return v.fn;
    return nullptr;
}

bool layer_supported(int ks, int units, int rb, int waves) { return layer_variant(ks, units, rb, waves) != nullptr; }

// Workgroups of the layer kernel one CU of the current device holds (0 if it cannot be asked).
int layer_workgroups_per_cu(int ks, int units, int rb, int waves, int lds_bytes)
{
    const LayerFn fn = layer_variant(ks, units, rb, waves);
    int per_cu = 0;
    if (!fn) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * waves, (size_t)lds_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu;
}

hipError_t launch_bspmm_layer(const LayerParams& P, int ks, int units, int rb, int waves, int lds_bytes, hipStream_t stream)
{
    const LayerFn fn = layer_variant(ks, units, rb, waves);
    if (!fn) return hipErrorInvalidValue;
    return launch(fn, 8 * P.shape.ranges_per_xcd * P.shape.tiles, 64 * waves, lds_bytes, stream, P.starts,
                  reinterpret_cast<const int2*>(P.entries), P.out_rows, P.x, P.w, P.bias, P.y, P.direct, P.shape);
}

hipError_t launch_layer_rows(const LayerSet* sets, int count, const OpRecord* ops, const int32_t* rpt,
                             const int32_t* colids, const float* values, int32_t* starts, int32_t* entries,
                             int32_t* out_rows, hipStream_t stream)
{
    if (count <= 0) return hipSuccess;
    return launch(layer_rows_kernel, count, kThreads, 0, stream, sets, ops, rpt, colids, values, starts,
                  reinterpret_cast<int2*>(entries), out_rows);
}

hipError_t launch_build_transpose(const OpRecord* ops, int batch, int threads, int lds_bytes,
                                  const int32_t* rpt, const int32_t* colids,
                                  const float* values, int32_t* rpt_t, int32_t* colids_t,
                                  float* values_t, int32_t* gscratch, const int32_t* order,
                                  hipStream_t stream)
{
    if (batch <= 0) return hipSuccess;
    auto* fn = threads == kBuildThreadsLarge ? build_sorted_kernel<false, kBuildThreadsLarge>
                                             : build_sorted_kernel<false, kThreads>;
    return launch(fn, batch, threads, lds_bytes, stream, ops, rpt, colids, values, rpt_t, colids_t, values_t, gscratch,
                  order);
}

hipError_t launch_merge_sets(const SetRecord* sets, int count, const int32_t* rpt,
                             const int32_t* colids, const float* values, int32_t* merged,
                             hipStream_t stream)
{
    if (count <= 0) return hipSuccess;
    return launch(merge_sets_kernel, count, kThreads, 0, stream, sets, rpt, colids, values, merged);
}

hipError_t launch_bspmm_coo(const CooLaunchParams& P, int grid, int lds_bytes, bool vec4,
                            hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    return launch(vec4 ? bspmm_coo_kernel<4> : bspmm_coo_kernel<1>, grid, kThreads, lds_bytes, stream, P);
}

// COO (index pairs `ids`, values) -> CSR arrays of every operation.
hipError_t launch_build_from_coo(const OpRecord* ops, int batch, int threads, int lds_bytes, const int32_t* ids,
                                 const float* values, int32_t* rpt, int32_t* colids,
                                 float* csr_values, int32_t* gscratch, const int32_t* order,
                                 hipStream_t stream)
{
    if (batch <= 0) return hipSuccess;
    auto* fn = threads == kBuildThreadsLarge ? build_sorted_kernel<true, kBuildThreadsLarge>
                                             : build_sorted_kernel<true, kThreads>;
    return launch(fn, batch, threads, lds_bytes, stream, ops, static_cast<const int32_t*>(nullptr), ids, values, rpt,
                  colids, csr_values, gscratch, order);
}

hipError_t launch_validate_coo(const OpRecord* ops, int batch, const int32_t* ids, int32_t* flag,
                               hipStream_t stream)
{
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, stream, flag, 0x7fffffff, 1);
    if (batch > 0)
        hipLaunchKernelGGL(validate_coo_kernel, dim3(batch), dim3(kThreads), 0, stream, ops, ids, flag);
    return hipGetLastError();
}

hipError_t launch_validate(const OpRecord* ops, int batch, const int32_t* rpt,
                           const int32_t* colids, int32_t* flag, hipStream_t stream)
{
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, stream, flag, 0x7fffffff, 1);
    if (batch > 0)
        hipLaunchKernelGGL(validate_csr_kernel, dim3(batch), dim3(kThreads), 0, stream, ops, rpt,
                           colids, flag);
    return hipGetLastError();
}

}  // namespace bspmm
