// Fused priority update + ingest: the learner's new priorities for the last
// batch (App. C Invariant 2) and then the actor's next transitions (Sec. 2.2
// off-policy ingestion), with the effects of conduit_update_priorities
// followed by conduit_ingest, in one launch whose parts run concurrently.
//
// In that order the ingest overwrites the leaf of every slot it evicts, so an
// update of such a slot changes nothing but the running maximum priority; and
// the new rows enter with the running maximum raised by the update's
// priorities, which is max(current, every valid update priority).  Hence:
//   * block 0 (1024 lanes) runs the update pass (update_dev.h) skipping the
//     slots the ingest evicts, flushes its LDS bins and raises the running
//     maximum (a list of more than 1,024 updates is split over several such
//     blocks by slot);
//   * every other block is four ingest sub-blocks of 256 lanes (ingest_dev.h):
//     the new rows' columns, leaves and per-wavefront tree deltas, each
//     wavefront (of a long list, each block) computing the raised running
//     maximum from the update list itself, and the payload copy; variable-length
//     rows take a block each instead (256 sequences of up to 4,096 tokens with
//     256 updates: 9.2 us as two launches, 5.6 as one).
// The two sets of leaves are disjoint and every tree change is an integer
// atomic add, so the result equals the two calls made one after the other.
#include <type_traits>

#include "ingest_dev.h"
#include "update_dev.h"

namespace conduit {

namespace {

constexpr int kSubs = kUpdateThreads / kIngestThreads;

struct Ragged {};  // in the place of the copied vector type: variable-length rows

// The largest valid priority of a list, by the whole workgroup.
__device__ uint32_t list_max(const RaiseList& u, int32_t* scratch) {
    uint32_t m = 0;
    for (int64_t base = 0; base < u.n; base += (int64_t)kUpdateThreads * kRaiseUnroll) {
        int64_t s[kRaiseUnroll];
        uint32_t p[kRaiseUnroll];
#pragma unroll
        for (int r = 0; r < kRaiseUnroll; ++r) {
            const int64_t k = base + (int64_t)r * kUpdateThreads + threadIdx.x;
            s[r] = k < u.n ? u.idx[k] : -1;
            p[r] = k < u.n ? u.prio[k] : 0u;
        }
#pragma unroll
        for (int r = 0; r < kRaiseUnroll; ++r)
            if (s[r] >= 0 && s[r] < u.size && p[r] > m) m = p[r];
    }
    m = wave_max_u32(m);
    if (lane_id() == 0) scratch[threadIdx.x / kWave] = (int32_t)m;
    __syncthreads();
    uint32_t r = 0;
    for (int i = 0; i < kUpdateThreads / kWave; ++i) {
        const uint32_t x = (uint32_t)scratch[i];
        r = x > r ? x : r;
    }
    return r;
}

// SPLIT: the first `groups` blocks share a long update list by slot, SPLIT
// entries per lane and pass; 0: the first block takes the list
template <typename V, int SPLIT>
__global__ __launch_bounds__(kUpdateThreads) void k_update_ingest(UpdateArgs u, IngestArgs a, int64_t meta_subs,
                                                                  int64_t copy_subs, int32_t groups) {
    __shared__ uint32_t keys[kTable];
    __shared__ int32_t owner[kTable];
    __shared__ unsigned long long bins[kBins];
    const uint32_t first = SPLIT > 0 ? (uint32_t)groups : 1u;  // the first ingest block
    if (blockIdx.x < first) {
        // one workgroup's atomics cost less than waiting for the stored maximum
        const uint32_t seen = SPLIT > 0 ? u.state->max_prio : 0u;
        uint32_t pmax;
        if constexpr (SPLIT > 0) pmax = update_part<SPLIT>(u, blockIdx.x, first, keys, owner, bins, a.head, a.n);
        else pmax = update_pass(u, keys, owner, bins, a.head, a.n);
        flush_bins(u.tree, bins);
        raise_max(u.state, seen, pmax);
        return;
    }
    if constexpr (std::is_same<V, Ragged>::value) {
        // whole workgroups of metadata, then one per sequence
        const int64_t meta_wgs = (meta_subs + kSubs - 1) / kSubs;
        const int64_t j = (int64_t)(blockIdx.x - first) - meta_wgs;
        if (j >= 0) {
            copy_ragged<kUpdateThreads, 1>(a, j, threadIdx.x);
            return;
        }
    }
    const int64_t sub0 = (int64_t)(blockIdx.x - first) * kSubs;
    const int64_t sub = sub0 + threadIdx.x / kIngestThreads;
    const int tid = (int)(threadIdx.x % kIngestThreads);
    RaiseList raise{u.idx, u.prio, u.n, u.size};
    if constexpr (SPLIT > 0) {
        if (sub0 < meta_subs && !a.src_prio) raise.known = list_max(raise, owner);  // uniform: read by the whole workgroup
    }
    if (sub < meta_subs) {
        // the update block may already have raised the stored maximum with the
        // same priorities: raised_max takes max() over both, so the order of
        // the two parts does not matter
        ingest_meta<SPLIT == 0 ? kRaiseRead : kRaiseKnown>(a, sub, tid, raise);
    } else if constexpr (!std::is_same<V, Ragged>::value) {
        if (sub - meta_subs < copy_subs) copy_dense<V>(a, sub - meta_subs, tid);
    }
}

}  // namespace

hipError_t launch_update_ingest(const UpdateArgs& u, const IngestArgs& a, hipStream_t s) {
    const int64_t lanes = [&] {
        const int64_t n1 = a.n < a.capacity - a.head ? a.n : a.capacity - a.head;
        return (n1 + kWave - 1) / kWave * kWave + (a.n - n1 + kWave - 1) / kWave * kWave;
    }();
    const int64_t meta_subs = (lanes + kIngestThreads - 1) / kIngestThreads;
    const uintptr_t al = reinterpret_cast<uintptr_t>(a.src_obs) | reinterpret_cast<uintptr_t>(a.obs) |
                         (uintptr_t)a.row_bytes;
    int vec = (al & 15) == 0 ? 16 : (al & 7) == 0 ? 8 : (al & 3) == 0 ? 4 : 1;
    if (a.row_bytes == 0) vec = 16;
    const int64_t total_vec = a.n * (a.row_bytes / vec);
    const int64_t copy_subs = (total_vec + kIngestThreads * kCopyUnroll - 1) / (kIngestThreads * kCopyUnroll);
    const int32_t groups = update_groups(u.n);
    const int64_t meta_wgs = (meta_subs + kSubs - 1) / kSubs;
    const dim3 grid((unsigned)(groups + (a.length ? meta_wgs + a.n : (meta_subs + copy_subs + kSubs - 1) / kSubs)));
    const dim3 block(kUpdateThreads);
    auto go = [&](auto v) {
        typedef decltype(v) V;
        if (groups == 1)
            hipLaunchKernelGGL((k_update_ingest<V, 0>), grid, block, 0, s, u, a, meta_subs, copy_subs, groups);
        else if (u.n <= 4 * kUpdateThreads)
            hipLaunchKernelGGL((k_update_ingest<V, 4>), grid, block, 0, s, u, a, meta_subs, copy_subs, groups);
        else
            hipLaunchKernelGGL((k_update_ingest<V, 8>), grid, block, 0, s, u, a, meta_subs, copy_subs, groups);
    };
    if (a.length) {
        go(Ragged{});
        return hipGetLastError();
    }
    switch (vec) {
        case 16: go(u32x4{}); break;
        case 8: go(u32x2{}); break;
        case 4: go(uint32_t{}); break;
        default: go(uint8_t{}); break;
    }
    return hipGetLastError();
}

}  // namespace conduit
