// Stratified inverse-CDF sampling over the 64-ary integer sum tree, with
// importance weights (off-policy delivery draws from the replay dataset, paper
// Sec. 2.2; proportional prioritised replay, Schaul et al.).
//
// k_sample: one wavefront per sample runs tree_descend (descend.h): the exact
// stratified target, then one coalesced 64-child load, wavefront prefix scan
// and ballot per tree level.
//
// k_is_weights: the weights need the smallest sampled leaf of the batch.  Each
// sample's wavefront parks its leaf in the output weight slot; one workgroup
// then reduces the minimum in LDS and overwrites every slot with
// (q_min / q_i)^beta computed in fp64 (is_weights_block); batches of more than
// kWeightsOneWg samples take k_batch_min and k_is_weights_split.  The sample + gather
// call instead computes the weights inside its one launch (k_sample_gather.hip),
// or, for shapes that kernel does not take, in one extra workgroup of the
// gather launch.
#include "descend.h"

namespace conduit {

namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * kWave;

template <int PRE, int DEPTH>
__global__ __launch_bounds__(kThreads) void k_sample(SampleArgs a, DivB dv) {
    const int64_t k = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave;
    if (k < a.batch) {  // wave-uniform
        const Descent d = tree_descend<PRE, DEPTH>(a.tree, a.uniforms, k, dv);
        if (lane_id() == 0) {
            a.idx_out[k] = d.slot;
            // the sampled leaf is parked in the weight slot for the weights block
            if (a.w_out) reinterpret_cast<uint32_t*>(a.w_out)[k] = d.leaf;
            if (d.slot < 0 && k == 0) flag_error(a.err, ERR_EMPTY_TREE);
            if (d.lost) flag_error(a.err, ERR_DESCENT);
        }
    }
    // buffer-wide normalisation: this workgroup's share of the leaf minimum
    if (a.leaf_min) fold_leaf_min<kThreads, true>(a, blockIdx.x, gridDim.x);
}

constexpr int kWThreads = 1024;
constexpr int64_t kWeightsOneWg = 2048;  // batches up to here take their weights from one workgroup

__global__ __launch_bounds__(kWThreads) void k_is_weights(WeightsArgs a) { is_weights_block<kWThreads>(a); }

// The weights of a large batch in two launches: one workgroup finds the smallest
// parked leaf (or takes it over from leaf_min), then every lane of up to kSplitWgs workgroups turns leaves into
// weights.  The fp64 powers bound the one-workgroup kernel (16,384 weights 32.7
// us, 4,096 9.2, 2,048 5.3); the pair takes 5.8, 5.1 and about 5.  Folding the minimum in
// the sampler instead costs more: its workgroups' atomics (or even reads) of one
// line run one after the other, about 5 ns each (16,384 samples: 8.3 -> 22-27
// us).
constexpr int kSplitWgs = 64;
constexpr int kSplitThreads = 256;

// leaf_min (buffer-wide normalisation): the sampler has folded the minimum there
// already; it is moved, and reset for the next call.
__global__ __launch_bounds__(kWThreads) void k_batch_min(const uint32_t* parked, int64_t batch, uint32_t* leaf_min,
                                                         DeviceState* st) {
    if (leaf_min) {  // kernel argument: uniform
        if (threadIdx.x == 0) {
            st->batch_min = *leaf_min;
            *leaf_min = 0xffffffffu;
        }
        return;
    }
    __shared__ uint32_t s_min[kWThreads / kWave];
    uint32_t m = 0xffffffffu;
    constexpr int kU = 8;  // loads in flight
    for (int64_t base = 0; base < batch; base += kWThreads * kU) {
        uint32_t q[kU];
#pragma unroll
        for (int r = 0; r < kU; ++r) {
            const int64_t k = base + r * kWThreads + threadIdx.x;
            q[r] = parked[k < batch ? k : batch - 1];
        }
#pragma unroll
        for (int r = 0; r < kU; ++r) m = q[r] && q[r] < m ? q[r] : m;
    }
    m = wave_min_u32(m);
    if (lane_id() == 0) s_min[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kWThreads / kWave; ++i) m = s_min[i] < m ? s_min[i] : m;
        st->batch_min = m;
    }
}

__global__ __launch_bounds__(kSplitThreads) void k_is_weights_split(WeightsArgs a, const DeviceState* st) {
    const double qmin = (double)st->batch_min;
    for (int64_t k = (int64_t)blockIdx.x * kSplitThreads + threadIdx.x; k < a.batch;
         k += (int64_t)gridDim.x * kSplitThreads) {
        const uint32_t q = reinterpret_cast<const uint32_t*>(a.w)[k];
        a.w[k] = q ? (float)pow(qmin / (double)q, a.beta) : 0.0f;
    }
}

// the sampler grid for a tree of PRE prefetched groups and depth DEPTH
struct DescendLaunch {
    const SampleArgs& a;
    DivB dv;
    hipStream_t s;
    template <int PRE, int DEPTH>
    hipError_t operator()() const {
        const int64_t blocks = (a.batch + kWaves - 1) / kWaves;
        hipLaunchKernelGGL((k_sample<PRE, DEPTH>), dim3((unsigned)blocks), dim3(kThreads), 0, s, a, dv);
        return hipGetLastError();
    }
};

}  // namespace

hipError_t launch_descend(const SampleArgs& a, hipStream_t s) {
    return with_descent_shape(a.tree, descend_prefetch(a.tree), DescendLaunch{a, make_divb((uint64_t)a.batch), s});
}

hipError_t launch_weights(const SampleArgs& a, hipStream_t s) {
    const WeightsArgs wa{a.w_out, a.batch, a.beta, a.leaf_min};
    if (a.batch <= kWeightsOneWg) {
        hipLaunchKernelGGL(k_is_weights, dim3(1), dim3(kWThreads), 0, s, wa);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_batch_min, dim3(1), dim3(kWThreads), 0, s, reinterpret_cast<const uint32_t*>(a.w_out), a.batch,
                       a.leaf_min, a.state);
    const int64_t wgs = (a.batch + kSplitThreads - 1) / kSplitThreads;
    hipLaunchKernelGGL(k_is_weights_split, dim3((unsigned)(wgs < kSplitWgs ? wgs : kSplitWgs)), dim3(kSplitThreads), 0, s,
                       wa, a.state);
    return hipGetLastError();
}

hipError_t launch_sample(const SampleArgs& a, hipStream_t s) {
    const hipError_t e = launch_descend(a, s);
    return e != hipSuccess || a.w_out == nullptr ? e : launch_weights(a, s);
}

}  // namespace conduit
