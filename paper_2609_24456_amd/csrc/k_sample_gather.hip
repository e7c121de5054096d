// Fused sampler + gather for dense buffers whose rows are a few work items
// (the frame-stack DQN shape), and fused sampler + token packing for ragged
// buffers (k_sample_pack, at the end): one launch delivers indices,
// importance weights and the learner batch (proportional prioritised replay,
// Schaul et al.; the paper's off-policy delivery samples and then materialises
// the batch, Sec. 2.2).
//
// Two kinds of 512-lane workgroup share the grid:
//   * gather workgroups (the head of the grid, one per sample, or up to four in
//     small batches): wavefront 0
//     runs tree_descend (descend.h) for the sample -- a few KB of tree reads
//     -- so the frame loads never wait for another workgroup or for the index
//     to make a round trip through memory; then the two 256-lane halves split
//     the row's work items (two each for a stack of four frames), and the
//     first half writes the scalar columns.
//   * sampler workgroups (the tail of the grid, eight samples each, one per
//     wavefront) run the same descent, write the indices and error flags, and
//     park each sampled leaf in the weight array.
// The DQN batch's 512 gather and 64 sampler workgroups are all resident at
// once (the kernel's registers allow seven wavefronts per SIMD).  One
// workgroup per sample rather than one per pair of frames halves the
// redundant descents and lets the whole row start as soon as its one descent
// ends (17.8 against 18.7 us per DQN batch).
//
// Importance weights need the smallest sampled leaf of the whole batch (or,
// normalised buffer-wide, of the whole buffer: then each sampler workgroup
// also folds the minimum of its share of the leaves into the device state
// with one agent-scope atomic).  Each sampler workgroup parks its leaves with
// agent-scope atomic stores, waits until they are acknowledged (visible
// device-wide), and takes a ticket with one agent-scope atomic add on the
// buffer's device state.  The workgroup that
// draws the last ticket reads every leaf back with agent-scope atomic loads,
// writes the weights (is_weights_block) and resets the ticket for the next
// call.  No workgroup waits for another, no release fence (which would write
// back the L2 under the frame stores) is needed, and the ticket latency stays
// off the frame workgroups.
#include <type_traits>

#include "descend.h"
#include "gae_packed_dev.h"
#include "gather_dev.h"
#include "nstep_dev.h"

namespace conduit {

namespace {

constexpr int kWg = 2 * kThreads;  // two 256-lane halves
constexpr int kSamplesPerSamplerWg = kWg / kWave;

// A sampler workgroup of NT lanes: NT / 64 samples, one per wavefront.
template <int NT, int PRE, int DEPTH>
__device__ void sampler_wg(const SampleArgs& sa, const DivB& dv, int64_t wg) {
    constexpr int64_t kPer = NT / kWave;
    __shared__ uint32_t s_last;
    const int64_t k = wg * kPer + threadIdx.x / kWave;
    if (k < sa.batch) {  // wave-uniform
        const Descent d = tree_descend<PRE, DEPTH>(sa.tree, sa.uniforms, k, dv);
        if (lane_id() == 0) {
            sa.idx_out[k] = d.slot;
            if (d.slot < 0 && k == 0) flag_error(sa.err, ERR_EMPTY_TREE);
            if (d.lost) flag_error(sa.err, ERR_DESCENT);
            if (sa.w_out)
                __hip_atomic_store(reinterpret_cast<uint32_t*>(sa.w_out) + k, d.leaf, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (!sa.w_out) return;  // kernel argument: uniform
    // buffer-wide normalisation: this workgroup's share of the leaf minimum,
    // folded in before the ticket like the parked leaves
    if (sa.leaf_min) fold_leaf_min<NT, false>(sa, wg, (sa.batch + kPer - 1) / kPer);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's parked leaves are acknowledged
    __syncthreads();                // ... and every wavefront's
    if (threadIdx.x == 0) {
        const uint32_t tickets = (uint32_t)((sa.batch + kPer - 1) / kPer);
        const uint32_t t = __hip_atomic_fetch_add(&sa.state->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = t == tickets - 1;
    }
    __syncthreads();
    if (s_last) {  // every leaf of the batch is parked and visible
        is_weights_block<NT, true>(WeightsArgs{sa.w_out, sa.batch, sa.beta, sa.leaf_min});
        if (threadIdx.x == 0) __hip_atomic_store(&sa.state->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// log2 of the workgroups per sample (1, 2 or 4), each descending on its own: a
// small batch shares its samples out while that leaves at most a workgroup per
// compute unit and every half an item (128 samples of four 84x84 frames to fp32
// 15.0 -> 13.9 us a step, with 3-step targets and bootstrap stacks 20.5 -> 16.7; 64
// of three 116x116 planes to bf16 14.0 -> 12.6).  Two workgroups a unit pay only
// for samples of many items (256 samples with the targets 24.2 -> 22.4; of four
// plain frames 14.4 -> 15.9), and with the bf16 table, which each workgroup
// builds, sharing stops at half a workgroup a unit (128 samples of four frames
// 12.8 -> 13.1).  Unshared samples have kernels of their own (SHARED false): the
// shared form's scalars cost 0.4 us (delivery of 100 samples with 1-step targets
// 8.7 us against 8.3).
inline int32_t log2_wgs_per_sample(int64_t batch, int64_t items, bool norm) {
    const int64_t cus = device_cus();
    int32_t l = 0;
    while (l < 2) {
        const int64_t wgs = batch << (l + 1);
        const bool few = wgs <= (norm ? cus / 2 : cus) && (4 << l) <= items;
        const bool long_rows = wgs <= 2 * cus && (7 << l) <= items;
        if (!few && !long_rows) break;
        ++l;
    }
    return l;
}

template <int XF, int PRE, int DEPTH, bool SHARED>
__global__ __launch_bounds__(kWg) void k_sample_gather(SampleArgs sa, GatherArgs a, DivB dv, int32_t bpf,
                                                       int32_t gather_wgs, int32_t log2_wgs, int32_t per_group) {
    __shared__ uint16_t lut[(XF == CONDUIT_XF_U8_BF16_NORM) ? 4 * 256 : 1];
    __shared__ int64_t s_slot;
    if (blockIdx.x >= (uint32_t)gather_wgs) {
        sampler_wg<kWg, PRE, DEPTH>(sa, dv, (int64_t)blockIdx.x - gather_wgs);
        return;
    }
    const uint32_t b = SHARED ? blockIdx.x >> log2_wgs : blockIdx.x, sub = SHARED ? blockIdx.x - (b << log2_wgs) : 0u;
    if (threadIdx.x < kWave) {
        const Descent d = tree_descend<PRE, DEPTH>(sa.tree, sa.uniforms, b, dv);
        if (threadIdx.x == 0) s_slot = d.slot;
    } else if constexpr (XF == CONDUIT_XF_U8_BF16_NORM) {
        build_lut(a, lut, kWave, kWg - kWave);
    }
    __syncthreads();
    // each half of the sample's workgroups takes its part of the row's items
    // (uniform in each wavefront: read from the first lane, so that the item's
    // output base stays a scalar)
    const int half = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kThreads));
    gather_row<XF, true>(a, b, (int)sub * 2 + half, per_group, bpf, s_slot, lut, (int)(threadIdx.x % kThreads));
}

// Rows of few units (vector observations, small frames): one wavefront per
// sample descends and copies the row itself, up to kRowUnroll units per lane, so
// that a workgroup delivers eight rows; a 512-lane workgroup per row left all
// but a few lanes idle.  Bound by the descent's dependent loads for small
// batches and by the wavefronts in flight for large ones.  With TICKET sampler
// workgroups beside the row ones write the indices and the weights, as in
// k_sample_gather: a small batch's critical path is the ticket's, and it should
// not wait for rows.  Without it the row wavefronts write the indices and park
// the leaves, one descent per sample, and the weights come by launches of their
// own (launch_weights).  Against 512 lanes per row: 256 rows of 8 floats 6.2 ->
// 6.0 us, 512 of 240 floats 8.9 -> 6.4, 16,384 of 48 floats 169 -> 15.4 + 7.1 for
// the weights.
// TICKET up to kRowsTicketMax samples: the workgroups' atomics run one after the
// other and the last workgroup computes every weight (1,024 samples 10.0 us
// against 7.1 + 3.2 + a launch, 4,096 of 240 floats 22.2 against 6.7 + 2.0 + 3.1).

template <int XF>
struct WaveRow {
    typename UnitOf<XF>::T v[kRowUnroll];
    uint32_t w[kRowUnroll];
    int32_t d[kRowUnroll], sj[kRowUnroll];
    uint32_t ej[kRowUnroll];
    int32_t si;
    uint32_t ei, sv, total;
    int64_t ii;
    bool ok;

    __device__ __forceinline__ void load(const GatherArgs& a, int64_t i, uint32_t units, const Div31& by_units) {
        typedef typename UnitOf<XF>::T V;
        const int lane = lane_id();
        bool words;
        const int ns = row_scalar_lanes(a, &words);
        ok = i >= 0 && i < a.limit;
        ii = ok ? i : 0;
        total = a.out ? units * (uint32_t)a.stack : 0u;
        si = 0;
        ei = 0;
        if (a.stack > 1) {  // kernel argument: uniform
            si = a.step[ii];
            ei = a.episode[ii];
        }
        sv = 0;
        if (lane < ns) sv = row_scalar_load(a, ii, lane, ns - 2, words);
#pragma unroll
        for (int r = 0; r < kRowUnroll; ++r) {
            sj[r] = 0;
            ej[r] = 0;
            d[r] = 0;
            w[r] = 0;
            v[r] = {};
            if ((uint32_t)r * kWave >= total) continue;  // uniform
            const uint32_t e = (uint32_t)(lane + r * kWave);
            const uint32_t u = e < total ? e : total - 1;  // every load is in range
            const uint32_t f = a.stack > 1 ? div31(u, by_units) : 0u;
            w[r] = u - f * units;
            d[r] = a.stack - 1 - (int32_t)f;
            int64_t j = ii - d[r];
            if (j < 0) j = ok ? j + a.capacity : 0;
            v[r] = *(reinterpret_cast<const V*>(a.src + j * a.row_bytes) + w[r]);
            if (a.stack > 1) {
                sj[r] = a.step[j];
                ej[r] = a.episode[j];
            }
        }
    }

    __device__ __forceinline__ void store(const GatherArgs& a, int64_t b, const uint16_t* lut) const {
        typedef typename OutUnit<XF>::T O;
        const int lane = lane_id();
        O* out = reinterpret_cast<O*>(a.out) + b * total;
#pragma unroll
        for (int r = 0; r < kRowUnroll; ++r) {
            const bool valid = ok & ((d[r] == 0) | ((d[r] <= si) & (ei == ej[r]) & (sj[r] == si - d[r])));
            const O o = convert_unit<XF>(a, w[r], v[r], lut);
            const uint32_t e = (uint32_t)(lane + r * kWave);
            if (e < total) out[e] = valid ? o : zero_unit<O>();
        }
        bool words;
        const int ns = row_scalar_lanes(a, &words);
        if (lane < ns) row_scalar_store(a, b, lane, ns - 2, words, ok ? sv : 0u);
        for (int t = lane + kWave; t < ns; t += kWave)  // rows of more than 64 scalar units
            row_scalar_store(a, b, t, ns - 2, words, ok ? row_scalar_load(a, ii, t, ns - 2, words) : 0u);
    }
};

template <int XF, int PRE, int DEPTH, bool TICKET>
__global__ __launch_bounds__(kWg) void k_sample_rows(SampleArgs sa, GatherArgs a, DivB dv, uint32_t units, Div31 by_units,
                                                     int32_t row_wgs) {
    __shared__ uint16_t lut[(XF == CONDUIT_XF_U8_BF16_NORM) ? 4 * 256 : 1];
    const int64_t wg = blockIdx.x;
    if (TICKET && wg >= row_wgs) {
        sampler_wg<kWg, PRE, DEPTH>(sa, dv, wg - row_wgs);
        return;
    }
    if constexpr (XF == CONDUIT_XF_U8_BF16_NORM) {
        build_lut(a, lut, 0, kWg);
        __syncthreads();
    }
    const int64_t k = wg * kSamplesPerSamplerWg + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (k < sa.batch) {  // wave-uniform
        const Descent d = tree_descend<PRE, DEPTH>(sa.tree, sa.uniforms, k, dv);
        if (!TICKET && lane_id() == 0) {
            sa.idx_out[k] = d.slot;
            if (sa.w_out) reinterpret_cast<uint32_t*>(sa.w_out)[k] = d.leaf;  // parked for launch_weights
            if (d.slot < 0 && k == 0) flag_error(sa.err, ERR_EMPTY_TREE);
            if (d.lost) flag_error(sa.err, ERR_DESCENT);
        }
        WaveRow<XF> row;
        row.load(a, d.slot, units, by_units);
        row.store(a, k, lut);
    }
    if (!TICKET && sa.leaf_min) fold_leaf_min<kWg, true>(sa, wg, row_wgs);  // buffer-wide normalisation
}

template <int XF>
struct RowsLaunch {
    const SampleArgs& sa;
    const GatherArgs& ga;
    DivB dv;
    uint32_t units;
    hipStream_t s;
    template <int PRE, int DEPTH>
    hipError_t operator()() const {
        const int64_t wgs = (sa.batch + kSamplesPerSamplerWg - 1) / kSamplesPerSamplerWg;
        const dim3 block(kWg);
        const Div31 du = make_div31(units);
        if (sa.batch <= kRowsTicketMax) {
            hipLaunchKernelGGL((k_sample_rows<XF, PRE, DEPTH, true>), dim3((unsigned)(2 * wgs)), block, 0, s, sa, ga, dv,
                               units, du, (int32_t)wgs);
            return hipGetLastError();
        }
        hipLaunchKernelGGL((k_sample_rows<XF, PRE, DEPTH, false>), dim3((unsigned)wgs), block, 0, s, sa, ga, dv, units, du,
                           (int32_t)wgs);
        const hipError_t e = hipGetLastError();
        return e != hipSuccess || !sa.w_out ? e : launch_weights(sa, s);
    }
};

template <int XF>
struct FusedLaunch {
    const SampleArgs& sa;
    const GatherArgs& ga;
    DivB dv;
    int64_t bpf;
    hipStream_t s;
    template <int PRE, int DEPTH>
    hipError_t operator()() const {
        const int64_t sampler_wgs = (sa.batch + kSamplesPerSamplerWg - 1) / kSamplesPerSamplerWg;
        const int32_t l = log2_wgs_per_sample(sa.batch, bpf * ga.stack, XF == CONDUIT_XF_U8_BF16_NORM);
        const dim3 grid((unsigned)(sampler_wgs + (sa.batch << l))), block(kWg);
        const int64_t groups = 2ll << l;
        const int32_t per_group = (int32_t)((bpf * ga.stack + groups - 1) / groups);
        if (l)
            hipLaunchKernelGGL((k_sample_gather<XF, PRE, DEPTH, true>), grid, block, 0, s, sa, ga, dv, (int32_t)bpf,
                               (int32_t)(sa.batch << l), l, per_group);
        else
            hipLaunchKernelGGL((k_sample_gather<XF, PRE, DEPTH, false>), grid, block, 0, s, sa, ga, dv, (int32_t)bpf,
                               (int32_t)sa.batch, 0, per_group);
        return hipGetLastError();
    }
};

template <int XF>
hipError_t launch_xf(const SampleArgs& sa, const GatherArgs& ga, hipStream_t s, int64_t bpf) {
    const int64_t units = ga.row_bytes >> UnitOf<XF>::kShift;
    if (units * ga.stack <= kRowMaxUnits)
        return with_descent_shape(sa.tree, descend_prefetch(sa.tree),
                                  RowsLaunch<XF>{sa, ga, make_divb((uint64_t)sa.batch), (uint32_t)units, s});
    return with_descent_shape(sa.tree, descend_prefetch(sa.tree),
                              FusedLaunch<XF>{sa, ga, make_divb((uint64_t)sa.batch), bpf, s});
}

// The fused sampler + gather with n-step targets: each gather workgroup's
// first wavefront descends for its sample and issues the loads of the
// sample's n-step window from the slot it found; once every wavefront knows
// the slot, the two halves issue the loads of their first frames of the union
// of the state stack and the bootstrap stack (UnionGather) while the first
// wavefront evaluates the window (lane 0 writes the targets), and after a
// second barrier, with the bootstrap slot known, they convert and store every
// frame once into the stacks it belongs to.  Sampler workgroups as in
// k_sample_gather.
//
// NT: frames of a ring beyond the last-level cache come from HBM and are not read
// again soon; loaded non-temporally they leave that cache to the outputs (steps in
// turn on three replays: 512 samples of four 84x84 frames, 3 steps, out of 200,000
// 41.3 -> 39.7 us; 8,192 single 48x48 frames out of 160,000 150.7 -> 115.1).  A ring
// the cache holds is read through it (8,192 of 50,000: 117 us, 136
// non-temporally).
constexpr int64_t kNtMinRing = 256ll << 20;

template <int XF, int PRE, int DEPTH, bool SHARED, bool NT>
__global__ __launch_bounds__(kWg) void k_sample_gather_nstep(SampleArgs sa, GatherArgs a, NstepArgs na,
                                                             void* next_out, DivB dv, int32_t bpf,
                                                             int32_t gather_wgs, int32_t log2_wgs) {
    __shared__ uint16_t lut[(XF == CONDUIT_XF_U8_BF16_NORM) ? 4 * 256 : 1];
    __shared__ int64_t s_slot, s_next;
    if (blockIdx.x >= (uint32_t)gather_wgs) {
        sampler_wg<kWg, PRE, DEPTH>(sa, dv, (int64_t)blockIdx.x - gather_wgs);
        return;
    }
    const uint32_t b = SHARED ? blockIdx.x >> log2_wgs : blockIdx.x;
    const int sub = SHARED ? (int)(blockIdx.x - (b << log2_wgs)) : 0;
    WindowLoads win;
    if (threadIdx.x < kWave) {
        const Descent d = tree_descend<PRE, DEPTH>(sa.tree, sa.uniforms, b, dv);
        const int64_t slot = __builtin_amdgcn_readfirstlane((uint32_t)d.slot) |
                             ((int64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)d.slot >> 32)) << 32);
        win = nstep_window_load(na, slot);  // in flight across the barrier
        if (threadIdx.x == 0) s_slot = slot;
    } else if constexpr (XF == CONDUIT_XF_U8_BF16_NORM) {
        build_lut(a, lut, kWave, kWg - kWave);
    }
    __syncthreads();  // the slot is known
    UnionRow r = union_row(a, b, s_slot, na.n, next_out != nullptr);
    const int half = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kThreads));
    const int part = sub * 2 + half, tid = (int)(threadIdx.x % kThreads);
    UnionGather<XF, NT> g;
    g.start(a, r, part, bpf, tid);  // the first frames' loads, while the window is evaluated
    if (threadIdx.x < kWave) {
        const int64_t next = nstep_window_finish(na, b, win, sub == 0);
        if (threadIdx.x == 0) s_next = next;
    }
    __syncthreads();  // the bootstrap slot is known
    r.jn = r.S > 0 ? s_next : -1;
    g.run(a, r, part, SHARED ? 2 << log2_wgs : 2, bpf, next_out, lut, tid);
}

template <int XF>
struct FusedNstepLaunch {
    const SampleArgs& sa;
    const GatherArgs& ga;
    const NstepArgs& na;
    void* next_out;
    DivB dv;
    int64_t bpf;
    hipStream_t s;
    template <int PRE, int DEPTH>
    hipError_t operator()() const {
        const int64_t sampler_wgs = (sa.batch + kSamplesPerSamplerWg - 1) / kSamplesPerSamplerWg;
        const int64_t frames = ga.stack + (next_out ? (na.n < ga.stack ? na.n : ga.stack) : 0);
        const int32_t l = log2_wgs_per_sample(sa.batch, bpf * frames, XF == CONDUIT_XF_U8_BF16_NORM);
        const dim3 grid((unsigned)(sampler_wgs + (sa.batch << l))), block(kWg);
        auto go = [&](auto shared, auto nt) {
            hipLaunchKernelGGL((k_sample_gather_nstep<XF, PRE, DEPTH, shared.value, nt.value>), grid, block, 0, s, sa, ga,
                               na, next_out, dv, (int32_t)bpf, (int32_t)(sa.batch << l), l);
        };
        const std::true_type yes;
        const std::false_type no;
        if (l) go(yes, no);
        else if (ga.limit * ga.row_bytes > kNtMinRing) go(no, yes);
        else go(no, no);
        return hipGetLastError();
    }
};

template <int XF>
hipError_t launch_nstep_xf(const SampleArgs& sa, const GatherArgs& ga, const NstepArgs& na, void* next_out,
                           hipStream_t s, int64_t bpf) {
    return with_descent_shape(sa.tree, descend_prefetch(sa.tree),
                              FusedNstepLaunch<XF>{sa, ga, na, next_out, make_divb((uint64_t)sa.batch), bpf, s});
}

// Sampler + token packing in one launch (ragged buffers): one pack workgroup
// per sample at the head of the grid, whose first wavefront descends for the
// sample before the workgroup packs the row (pack_row), and sampler workgroups
// of the same width (one sample per wavefront) at the tail for the indices and
// the importance weights, as in k_sample_gather.
//
// With GAE, each pack workgroup then runs the GAE of its packed row from the
// length and reward it has just written (gae_packed_row), as
// conduit_gae_packed would over the packed batch.
//
// Widths: the pack alone takes 256 lanes ([256, 4096]: 7.4 us; 7.8-8.3 us with
// 512).  Pack + GAE take the row in one pass of at most 2 vectors per lane: 256
// lanes up to 1,024 elements ([1000, 256] 12.0 us against 13.4 with 512 lanes), 512
// up to 4,096 ([256, 4096] 9.8 us; 11.6 with 256, 12.0 with 1,024), 1,024 beyond
// ([200, 8192] 12.1 us against 13.9).
template <int NT, int PRE, int DEPTH, bool GAE>
__global__ __launch_bounds__(NT) void k_sample_pack(SampleArgs sa, PackArgs pa, GaePackedArgs ga, DivB dv,
                                                    int32_t sampler_wgs) {
    __shared__ int64_t s_slot;
    const int64_t pack_wgs = (int64_t)gridDim.x - sampler_wgs;
    if ((int64_t)blockIdx.x >= pack_wgs) {
        sampler_wg<NT, PRE, DEPTH>(sa, dv, (int64_t)blockIdx.x - pack_wgs);
        return;
    }
    const int64_t b = blockIdx.x;
    if (threadIdx.x < kWave) {
        const Descent d = tree_descend<PRE, DEPTH>(sa.tree, sa.uniforms, b, dv);
        if (threadIdx.x == 0) s_slot = d.slot;
    }
    __syncthreads();
    const PackedRow row = pack_row<NT>(pa, b, s_slot);
    if constexpr (GAE) gae_packed_row<NT, NT == kThreads ? 1 : 2, NT != 1024>(ga, b, row.L, (double)row.R);
}

struct PackLaunch {
    const SampleArgs& sa;
    const PackArgs& pa;
    const GaePackedArgs* ga;  // NULL: no GAE
    DivB dv;
    hipStream_t s;
    template <int NT, bool GAE, int PRE, int DEPTH>
    hipError_t launch() const {
        const int64_t sampler_wgs = (sa.batch + NT / kWave - 1) / (NT / kWave);
        const dim3 grid((unsigned)(sampler_wgs + sa.batch)), block(NT);
        hipLaunchKernelGGL((k_sample_pack<NT, PRE, DEPTH, GAE>), grid, block, 0, s, sa, pa, ga ? *ga : GaePackedArgs{},
                           dv, (int32_t)sampler_wgs);
        return hipGetLastError();
    }
    template <int PRE, int DEPTH>
    hipError_t operator()() const {
        if (!ga) return launch<kThreads, false, PRE, DEPTH>();
        if (pa.max_len <= 1024) return launch<kThreads, true, PRE, DEPTH>();
        if (pa.max_len <= 4096) return launch<512, true, PRE, DEPTH>();
        return launch<1024, true, PRE, DEPTH>();
    }
};

}  // namespace

hipError_t launch_sample_gather(const SampleArgs& sa, const GatherArgs& ga, hipStream_t s) {
    const bool c16 = copy16(ga);
    const int64_t units = ga.row_bytes >> (c16 ? 4 : 2);
    const int64_t bpf = ga.out && units > 0 ? (units + kUnitsPerBlock - 1) / kUnitsPerBlock : 0;
    const int64_t per_row = bpf * ga.stack;
    if (sa.batch <= 0 || ga.ncols != 0 || per_row > kFusedMaxItemsPerRow) return hipErrorNotSupported;
    // large batches of plain single frames that a wavefront does not take: the
    // sampler and the flat gather, without a descent and 512 lanes per row (4,096
    // rows of 4,000 floats: 52.7 us as one launch)
    if (ga.stack == 1 && ga.xform != CONDUIT_XF_U8_BF16_NORM && units > kRowMaxUnits && sa.batch > kRowsTicketMax)
        return hipErrorNotSupported;
    if (c16) return launch_xf<kXfCopy16>(sa, ga, s, bpf);
    switch (ga.xform) {
        case CONDUIT_XF_NONE: return launch_xf<CONDUIT_XF_NONE>(sa, ga, s, bpf);
        case CONDUIT_XF_U8_F32: return launch_xf<CONDUIT_XF_U8_F32>(sa, ga, s, bpf);
        case CONDUIT_XF_U8_BF16_NORM: return launch_xf<CONDUIT_XF_U8_BF16_NORM>(sa, ga, s, bpf);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sample_gather_nstep(const SampleArgs& sa, const GatherArgs& ga, const NstepArgs& na,
                                      void* next_out, hipStream_t s) {
    const bool c16 = copy16(ga);
    const int64_t units = ga.row_bytes >> (c16 ? 4 : 2);
    const int64_t bpf = ga.out && units > 0 ? (units + kUnitsPerBlock - 1) / kUnitsPerBlock : 0;
    const int64_t frames = ga.stack + (next_out ? (na.n < ga.stack ? na.n : ga.stack) : 0);
    if (sa.batch <= 0 || na.batch != sa.batch || ga.ncols != 0 || bpf < 1 ||
        bpf * frames > kFusedNstepMaxItemsPerRow)
        return hipErrorNotSupported;
    // large batches of small rows: the wavefront-per-sample delivery, then the
    // targets and the flat gather (a step of 1,025 rows of 8 floats, n = 3, 25.0 us
    // in one launch and 23.3 in these, 2,048 39.6 and 23.2, 16,384 303 and 38.8; of
    // 240 floats 25.4 and 24.0, 40.6 and 24.2, 310 and 45)
    if (units * ga.stack <= kRowMaxUnits && sa.batch > kRowsTicketMax) return hipErrorNotSupported;
    if (c16) return launch_nstep_xf<kXfCopy16>(sa, ga, na, next_out, s, bpf);
    switch (ga.xform) {
        case CONDUIT_XF_NONE: return launch_nstep_xf<CONDUIT_XF_NONE>(sa, ga, na, next_out, s, bpf);
        case CONDUIT_XF_U8_F32: return launch_nstep_xf<CONDUIT_XF_U8_F32>(sa, ga, na, next_out, s, bpf);
        case CONDUIT_XF_U8_BF16_NORM: return launch_nstep_xf<CONDUIT_XF_U8_BF16_NORM>(sa, ga, na, next_out, s, bpf);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sample_pack(const SampleArgs& sa, const PackArgs& pa, const GaePackedArgs* ga, hipStream_t s) {
    if (sa.batch <= 0 || pa.n != sa.batch || (ga && ga->B != sa.batch)) return hipErrorNotSupported;
    return with_descent_shape(sa.tree, descend_prefetch(sa.tree),
                              PackLaunch{sa, pa, ga, make_divb((uint64_t)sa.batch), s});
}

}  // namespace conduit
