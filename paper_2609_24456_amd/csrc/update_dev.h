// Priority-update device code shared by the update kernel and the fused
// update + ingest kernel.
#pragma once
#include "common.h"

namespace conduit {

namespace {

constexpr int kUpdateThreads = 1024;
constexpr int kTable = 2048;   // power of two, at least 2x the chunk size
constexpr int kBins = 2048;    // u64 LDS bins for small tree levels

__device__ __forceinline__ uint32_t slot_hash(uint32_t key) { return (key * 0x9E3779B1u) >> (32 - 11); }

// whether an ingest of ring slots [ev_head, ev_head + ev_n) replaces `slot`
__device__ __forceinline__ bool evicted(const TreeView& tr, int64_t slot, int64_t ev_head, int64_t ev_n) {
    if (ev_n <= 0) return false;  // known when compiled where there is no ingest
    const int64_t back = slot - ev_head;
    return (back < 0 ? back + tr.nodes[0] : back) < ev_n;
}

// The leaf of priority p in place of `old` at `slot`, and the change added to
// the slot's ancestors (in `bins` for the levels kept in LDS).
__device__ __forceinline__ void put_leaf(const TreeView& tr, int64_t slot, uint32_t p, uint32_t old,
                                         unsigned long long* bins) {
    const uint32_t q = quantise_leaf(p, tr.alpha_num, tr.alpha_den, tr.frac_bits);
    tr.leaves[slot] = q;
    const uint64_t delta = (uint64_t)q - (uint64_t)old;  // modulo 2^64
    if (!delta) return;
    // unrolled over the largest depth: the per-level arguments are loaded
    // together rather than one level at a time
#pragma unroll
    for (int l = 1; l <= kMaxLevels; ++l) {
        if (l > tr.depth) break;
        const uint64_t node = (uint64_t)slot >> (kFanoutLog2 * l);
        const int off = tr.lds_offset[l];
        if (off >= 0) atomicAdd(&bins[off + node], (unsigned long long)delta);
        else atomicAdd(reinterpret_cast<unsigned long long*>(tr.level[l] + node), delta);
    }
}

// The table entry of `key` (slot + 1) takes the larger of its position and `pos`.
__device__ __forceinline__ uint32_t claim(uint32_t* keys, int32_t* owner, uint32_t key, int32_t pos) {
    uint32_t h = slot_hash(key);
    while (true) {
        const uint32_t prev = atomicCAS(&keys[h], 0u, key);
        if (prev == 0u || prev == key) break;
        h = (h + 1) & (kTable - 1);
    }
    atomicMax(&owner[h], pos);
    return h;
}

// The running maximum raised to the wavefronts' largest priorities.  `seen` is
// the maximum as read at the start (it only grows): a priority that does not
// exceed it needs no atomic.
__device__ __forceinline__ void raise_max(DeviceState* state, uint32_t seen, uint32_t pmax) {
    const uint32_t wm = wave_max_u32(pmax);
    if (lane_id() == 0 && wm > seen) atomicMax(&state->max_prio, wm);
}

// The update pass of one workgroup of kUpdateThreads lanes: leaves swapped,
// deltas of large levels sent as global atomics and those of levels kept in
// LDS (tree.lds_offset) accumulated in `bins` (zeroed here).  Returns the
// lane's largest priority; the caller flushes the bins and raises the running
// maximum.  Ends with an LDS-only barrier: the leaf writes are not waited for.
// Slots in the ring range [ev_head, ev_head + ev_n) are about to be
// overwritten by an ingest of the same launch: their leaf and tree work is
// skipped (the ingest replaces the leaf), their priority still counts.
__device__ uint32_t update_pass(const UpdateArgs& a, uint32_t* keys, int32_t* owner, unsigned long long* bins,
                                int64_t ev_head = 0, int64_t ev_n = 0) {
    const int tid = threadIdx.x;
    const TreeView& tr = a.tree;

    uint32_t pmax = 0;
    // the first chunk's index and priority loads are issued before the LDS set-up
    int64_t k = tid;
    int64_t slot_next = k < a.n ? a.idx[k] : -1;
    uint32_t p_next = k < a.n ? a.prio[k] : 0u;
    for (int i = tid; i < kBins; i += kUpdateThreads) bins[i] = 0ull;

    for (int64_t base = 0; base < a.n; base += kUpdateThreads) {
        for (int i = tid; i < kTable; i += kUpdateThreads) {
            keys[i] = 0u;
            owner[i] = -1;
        }
        // orders global memory too: a later chunk reads leaves this one's
        // predecessors wrote
        __syncthreads();
        k = base + tid;
        bool valid = k < a.n;
        const int64_t slot = slot_next;
        const uint32_t p = p_next;
        if (valid && (slot < 0 || slot >= a.size)) {
            flag_error(a.err, ERR_UPDATE_INDEX);
            valid = false;
        }
        // the old leaf is needed only by the winner, but its load is issued now so
        // it overlaps the LDS dedupe and the quantiser (chunks before this one
        // finished their leaf writes before the barrier above); unconditional,
        // from slot 0 for an invalid entry, so that no select of its value makes
        // the lane wait for it here
        const uint32_t old = tr.leaves[valid ? slot : 0];
        uint32_t h = 0;
        if (valid) {
            pmax = p > pmax ? p : pmax;
            h = claim(keys, owner, (uint32_t)slot + 1u, tid);  // key 0 marks an empty entry
        }
        // the next chunk's loads overlap this chunk's dedupe and leaf work
        const int64_t kn = base + kUpdateThreads + tid;
        slot_next = kn < a.n ? a.idx[kn] : -1;
        p_next = kn < a.n ? a.prio[kn] : 0u;
        lds_barrier();
        if (valid && owner[h] == tid && !evicted(tr, slot, ev_head, ev_n)) put_leaf(tr, slot, p, old, bins);
        lds_barrier();  // bins complete; the table may be cleared again
    }
    return pmax;
}

// Long update lists: `groups` workgroups (a power of two) of kUpdateThreads
// lanes split the SLOTS by a hash.  Each reads every index, UNROLL per
// lane and pass, and lists the entries of its own slots in LDS, one per lane;
// then the largest position of each slot wins in its LDS table as in
// update_pass.  No other workgroup touches those slots, so the last occurrence
// wins without any exchange between workgroups.  A pass with more entries for a
// workgroup than it has lanes (never expected of a hash, but any list has to
// work) goes through them kUpdateThreads list entries at a time instead.
// Passes run in order, a barrier ordering the leaves one writes before the next
// reads them.
//
// Bound by the chain index -> list -> priority and old leaf -> leaf, and by each
// workgroup reading the whole list.  Alone, on 1M slots: 2,048 updates 8.2 ->
// 6.1 us, 4,096 16.8 -> 7.2, 8,192 33 -> 8.1, 16,384 62 -> 12; 1,500 updates
// take 6.6 us unsplit and 6.1-6.8 split, so lists below kPartMinUpdates stay
// whole.  64, 128 or 256 entries per workgroup and up to 128 workgroups measure
// within 0.5 us of each other.
constexpr int64_t kPartMinUpdates = 2048;  // shorter lists are not split
constexpr int kPartMaxGroups = 64;
constexpr int kPartEntries = 128;          // of the list per workgroup, about

// workgroups for a list of n updates
inline int update_groups(int64_t n) {
    if (n < kPartMinUpdates) return 1;
    int g = 2;
    while (g < kPartMaxGroups && g * kPartEntries < n) g *= 2;
    return g;
}

// spreads neighbouring slots and whole tree nodes over the workgroups; full-rate
// instructions only, since every workgroup hashes the whole list
__device__ __forceinline__ uint32_t part_hash(uint32_t slot) { return slot ^ (slot >> 6) ^ (slot >> 12); }

// UNROLL: entries per lane and pass (4 or 8; 16 would not fit the 128 registers
// a lane of 1,024 has)
template <int UNROLL>
__device__ uint32_t update_part(const UpdateArgs& a, uint32_t wg, uint32_t groups, uint32_t* keys, int32_t* owner,
                                unsigned long long* bins, int64_t ev_head = 0, int64_t ev_n = 0) {
    __shared__ uint32_t s_count[2];
    __shared__ uint2 s_list[kUpdateThreads];  // slot, position in the pass
    constexpr int64_t kPass = (int64_t)kUpdateThreads * UNROLL;
    const int tid = threadIdx.x;
    const TreeView& tr = a.tree;
    uint32_t pmax = 0;
    // one entry per lane: its loads, its claim on the slot, and the winners'
    // leaves (the table clear before, LDS barriers inside)
    auto settle = [&](bool on, uint32_t slot, uint32_t pos, int64_t base) {
        const uint32_t p = on ? a.prio[base + pos] : 0u;
        const uint32_t old = tr.leaves[on ? slot : 0u];
        uint32_t h = 0;
        if (on) h = claim(keys, owner, slot + 1u, (int32_t)pos);
        lds_barrier();
        if (p > pmax) pmax = p;
        if (on && owner[h] == (int32_t)pos && !evicted(tr, slot, ev_head, ev_n)) put_leaf(tr, slot, p, old, bins);
    };
    int pass = 0;
    for (int64_t base = 0; base < a.n; base += kPass, pass ^= 1) {
        int64_t raw[UNROLL];
#pragma unroll
        for (int r = 0; r < UNROLL; ++r) {
            const int64_t k = base + r * kUpdateThreads + tid;
            raw[r] = a.idx[k < a.n ? k : a.n - 1];  // past the end: the last entry again, dropped below
        }
        if (base == 0) {
            for (int i = tid; i < kBins; i += kUpdateThreads) bins[i] = 0ull;
            if (tid < 2) s_count[tid] = 0;
        }
        for (int i = tid; i < kTable; i += kUpdateThreads) {
            keys[i] = 0u;
            owner[i] = -1;
        }
        __syncthreads();  // the table is clear; leaves of the pass before are written
        if (tid == 0) s_count[pass ^ 1] = 0;
        uint32_t own = 0, bad = 0;  // bit r: entry r is this workgroup's, is out of range
#pragma unroll
        for (int r = 0; r < UNROLL; ++r) {
            const bool ok = (uint64_t)raw[r] < (uint64_t)a.size;
            const bool mine = ok & (((part_hash((uint32_t)raw[r]) ^ wg) & (groups - 1)) == 0);
            bad |= (ok ? 0u : 1u) << r;
            own |= (mine ? 1u : 0u) << r;
        }
        // entries of the lane inside the list (all of them but in the last pass)
        const int64_t left = a.n - base - tid;
        const int64_t in = left <= 0 ? 0 : (left + kUpdateThreads - 1) / kUpdateThreads;
        if (in < UNROLL) own &= (1u << in) - 1u;
        if (bad && wg == 0 && in > 0) flag_error(a.err, ERR_UPDATE_INDEX);  // a repeated last entry is in the list too
        uint32_t at = own ? atomicAdd(&s_count[pass], __popc(own)) : 0;
#pragma unroll
        for (int r = 0; r < UNROLL; ++r) {
            if ((own >> r) & 1) {
                if (at < kUpdateThreads) s_list[at] = make_uint2((uint32_t)raw[r], r * kUpdateThreads + tid);
                ++at;
            }
        }
        lds_barrier();
        const uint32_t total = s_count[pass];
        if (total <= kUpdateThreads) {  // uniform
            const bool on = (uint32_t)tid < total;
            const uint2 e = s_list[on ? tid : 0];
            settle(on, e.x, e.y, base);
        } else {
            for (int r = 0; r < UNROLL; ++r) {
                const bool on = (own >> r) & 1;
                const uint32_t pos = r * kUpdateThreads + tid;
                settle(on, on ? (uint32_t)a.idx[base + pos] : 0u, pos, base);
                __syncthreads();  // the leaves are written, the table read
                for (int i = tid; i < kTable; i += kUpdateThreads) {
                    keys[i] = 0u;
                    owner[i] = -1;
                }
                lds_barrier();
            }
        }
        lds_barrier();  // the table and the list are read, bins complete
    }
    return pmax;
}

// Flush the LDS-accumulated levels into the tree (after an LDS barrier).
__device__ void flush_bins(const TreeView& tr, const unsigned long long* bins) {
#pragma unroll
    for (int l = 1; l <= kMaxLevels; ++l) {
        if (l > tr.depth) break;
        const int off = tr.lds_offset[l];
        if (off < 0) continue;
        const int nodes = (int)tr.nodes[l];
        for (int i = threadIdx.x; i < nodes; i += kUpdateThreads) {
            const unsigned long long v = bins[off + i];
            if (v) atomicAdd(reinterpret_cast<unsigned long long*>(tr.level[l] + i), v);
        }
    }
}


}  // namespace
}  // namespace conduit
