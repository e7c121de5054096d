// Gather / transform: materialise the learner batch (off-policy delivery
// builds it from the drawn transitions and changes its layout, paper Sec. 2.2;
// concat/stack, reshape, batching and padding/packing are the processing
// operators it lists).  The same kernels
// serve the on-policy minibatch shuffle-gather (K = 1, rows of a rollout).
//
// Three shapes: single frames and small ones as one flat run of units
// (k_gather_flat); stacked and bf16 frames as the work items of gather_dev.h,
// walked double-buffered by four persistent workgroups per compute unit
// (k_gather_pipe, outputs up to 128 MB) or one per workgroup (k_gather_rows,
// larger outputs).
// Scalar columns (action, reward, done, extra float columns) are produced by
// workgroups at the head of the grid, one lane per output row, so that their
// dependent loads (index, then the columns) start with the first dispatched
// workgroups and finish under the frame traffic.  When the indices were just
// sampled, one more workgroup there computes the batch's importance weights
// (is_weights_block).
#include <type_traits>

#include "gather_dev.h"

namespace conduit {

namespace {

// an index outside [0, limit): the row is zero-filled; err_kind < 0 (indices
// produced by the library, where -1 stands for "no row") raises no flag
__device__ __forceinline__ void flag_index(const GatherArgs& a) {
    if (a.err_kind >= 0) flag_error(a.err, a.err_kind);
}

// outputs up to this size use the persistent pipelined kernel
constexpr int64_t kPipeMaxOutBytes = 128ll << 20;

// The flat kernel (below) takes, of the batches whose units a 31-bit number
// counts:
//   * every frame of up to kFlatMaxUnits units: an item of 1,792 units would
//     leave most of its lanes idle (24,576 rows of 48 floats, 12 units each:
//     42.2 us as items, 6.3 us flat; 4,096 40x40 frames to fp32: 10.7 and 7.4);
//   * single frames of any size, unless normalised to bf16: its even split beats
//     items with a remainder, and large outputs leave faster (88x88 50 -> 32 us;
//     65,536 rows of 4 KB 114 -> 98 us; 16,384 images of 3x84x84 to fp32 322 -> 310
//     us), except
//       - frames to fp32 that fill their items, from HBM (a source beyond
//         kFlatMaxSource) or of a sampled batch, into up to kItemsMaxOutBytes: the
//         persistent kernel has more loads in flight (566 84x84 frames of 60,941 5.8
//         us, 7.1 flat; 2,267 14.9, 18.3; 2,900 25.0, 22.5; 566 of 2,264 in the last-level
//         cache 5.6, 4.6; a step of 216 sampled 3x152x152 23.0, 26.3, of 324 33.9, 33.1);
//       - rows of 4-byte units that fill half of their items, into more than
//         kPipeMaxOutBytes (57,429 rows of 1,023 floats 96.2 us, 108.8 flat; of 601
//         floats, a third, 134.7 and 110);
//       - such frames of a sampled batch into more than kPipeMaxOutBytes, its rows in
//         address order (a step of 694 4x120x120 46.1 us, 48.8 flat; 498 3x224x224
//         73.3, 77.7);
//   * single frames of up to kFlatMaxNormUnits units normalised to bf16 (4,096
//     64x64 frames 15.3 -> 11.8 us); larger ones spend more on finding each
//     unit's row than they save (1,024 images of 3x224x224: 83 us as items, 98
//     flat).
// Stacks of larger frames stay with the item kernels, which look each frame's
// validity up once per item (512 stacks of four 84x84 frames to bf16: 10.8 us,
// 12.9 flat).
constexpr int64_t kFlatMaxUnits = 512;
constexpr int64_t kFlatMaxNormUnits = 1024;
constexpr int64_t kFlatMaxSource = 256ll << 20;
constexpr int64_t kItemsMaxOutBytes = 64ll << 20;
constexpr int kFlatUnroll = 4;         // its most units per lane
constexpr int64_t kFlatWgsPerCu = 4;   // workgroups per compute unit before a lane takes more units
constexpr int64_t kFlatLoopWgs = 16;   // bf16: workgroups per compute unit, each looping with its table

// Blocks [0, tail): scalar columns, then the weights block (if any).
__device__ __forceinline__ bool tail_block(const GatherArgs& a, int64_t tail) {
    const int64_t blk = blockIdx.x;
    if (blk >= tail) return false;
    if (a.weights.w && blk == tail - 1) is_weights_block<kThreads>(a.weights);
    else gather_scalars(a, blk);
    return true;
}

// One work item per workgroup, all of the grid's loads before its stores: the
// shape for large outputs, where many resident workgroups keep the most bytes
// in flight.

template <int XF>
__global__ __launch_bounds__(kThreads) void k_gather_rows(GatherArgs a, int32_t bpf, int32_t tail) {
    __shared__ uint16_t lut[(XF == CONDUIT_XF_U8_BF16_NORM) ? 4 * 256 : 1];
    if (tail_block(a, tail)) return;
    const int64_t it = (int64_t)blockIdx.x - tail;
    if constexpr (XF == CONDUIT_XF_U8_BF16_NORM) {
        build_lut(a, lut);
        __syncthreads();
    }
    const int64_t i = a.idx[it / ((int64_t)bpf * a.stack)];
    const Item t = decode(a, it, bpf, i);
    if (!t.ok && threadIdx.x == 0 && t.part == 0 && t.k == a.stack - 1) flag_index(a);
    typename UnitOf<XF>::T v[kUnroll];
    int32_t si = 0, sj = 0;
    uint32_t ei = 0, ej = 0;
    issue<XF>(a, t, i, v, si, sj, ei, ej, threadIdx.x);
    finish<XF, kStoreNT, true>(a, t, v, si, sj, ei, ej, lut, threadIdx.x);
}

// Persistent workgroups walk the items with a stride of the grid.  Two register
// sets alternate: the loads of the next item are issued before the stores of
// the current one, so reads of one item overlap the writes of the previous one
// instead of the whole GPU reading first and writing afterwards.  The sample
// index of the item after next is fetched one step ahead as well.
template <int XF>
__global__ __launch_bounds__(kThreads) void k_gather_pipe(GatherArgs a, int32_t bpf, int64_t n_items, int32_t frame_grid,
                                                          int32_t tail) {
    __shared__ uint16_t lut[(XF == CONDUIT_XF_U8_BF16_NORM) ? 4 * 256 : 1];
    if (tail_block(a, tail)) return;
    if constexpr (XF == CONDUIT_XF_U8_BF16_NORM) {
        build_lut(a, lut);
        __syncthreads();
    }
    const int64_t G = frame_grid;
    const int64_t per_row = (int64_t)bpf * a.stack;
    auto clampi = [&](int64_t x) { return x < n_items ? x : n_items - 1; };
    int64_t it = (int64_t)blockIdx.x - tail;
    const int64_t i0 = a.idx[it / per_row];
    int64_t itn = it + G;
    int64_t i1 = a.idx[clampi(itn) / per_row];
    typename UnitOf<XF>::T va[kUnroll], vb[kUnroll];
    int32_t sia = 0, sja = 0, sib = 0, sjb = 0;
    uint32_t eia = 0, eja = 0, eib = 0, ejb = 0;
    Item ta = decode(a, it, bpf, i0), tb;
    if (!ta.ok && threadIdx.x == 0 && ta.part == 0 && ta.k == a.stack - 1) flag_index(a);
    issue<XF>(a, ta, i0, va, sia, sja, eia, eja, threadIdx.x);
    while (true) {
        tb = decode(a, clampi(itn), bpf, i1);
        issue<XF>(a, tb, i1, vb, sib, sjb, eib, ejb, threadIdx.x);
        int64_t itnn = itn + G;
        int64_t i2 = a.idx[clampi(itnn) / per_row];
        finish<XF, kStoreWT, false>(a, ta, va, sia, sja, eia, eja, lut, threadIdx.x);
        if (itn >= n_items) break;
        if (!tb.ok && threadIdx.x == 0 && tb.part == 0 && tb.k == a.stack - 1) flag_index(a);
        itn = itnn;
        i1 = i2;
        ta = decode(a, clampi(itn), bpf, i1);
        issue<XF>(a, ta, i1, va, sia, sja, eia, eja, threadIdx.x);
        itnn = itn + G;
        i2 = a.idx[clampi(itnn) / per_row];
        finish<XF, kStoreWT, false>(a, tb, vb, sib, sjb, eib, ejb, lut, threadIdx.x);
        if (itn >= n_items) break;
        if (!ta.ok && threadIdx.x == 0 && ta.part == 0 && ta.k == a.stack - 1) flag_index(a);
        itn = itnn;
        i1 = i2;
    }
}

// The batch as one flat run of n * stack * units units, U per lane and kThreads
// apart, so that a workgroup takes as many rows as its lanes cover and a
// wavefront's store is contiguous whatever the row size.  Each lane finds its
// units' frames with a multiply (div31) and reads their sample indices itself:
// two dependent rounds of loads (index, then payload and frame metadata), all U
// of each in flight.  Bound by those two rounds for small batches and by HBM for
// large ones.  Non-temporal stores: written through at agent scope the same
// kernel takes 336 us instead of 310 for 16,384 images of 3x84x84 to fp32, and
// 16.8 instead of 14.5 us for 4,096 64x64 frames.  With the bf16 table a
// workgroup loops over tiles, so that the table is built once per workgroup.
template <int XF, int U>
__global__ __launch_bounds__(kThreads) void k_gather_flat(GatherArgs a, uint32_t units, Div31 by_units, Div31 by_stack,
                                                          uint32_t total, int32_t tail) {
    __shared__ uint16_t lut[(XF == CONDUIT_XF_U8_BF16_NORM) ? 4 * 256 : 1];
    if (tail_block(a, tail)) return;
    typedef typename UnitOf<XF>::T V;
    typedef typename OutUnit<XF>::T O;
    constexpr uint32_t kTile = kThreads * U;
    if constexpr (XF == CONDUIT_XF_U8_BF16_NORM) {
        build_lut(a, lut);
        __syncthreads();
    }
    const uint32_t step = (gridDim.x - (uint32_t)tail) * kTile;
    for (uint32_t first = (blockIdx.x - (uint32_t)tail) * kTile; first < total; first += step) {
        uint32_t w[U], d[U];  // unit of the frame, frames back
        int64_t i[U];
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const uint32_t e = first + r * kThreads + threadIdx.x;
            const uint32_t u = e < total ? e : total - 1;  // every load is in range
            const uint32_t f = div31(u, by_units);
            const uint32_t b = div31(f, by_stack);
            w[r] = u - f * units;
            d[r] = (uint32_t)a.stack - 1 - (f - b * (uint32_t)a.stack);
            i[r] = a.idx[b];
        }
        bool ok[U];
        V v[U];
        int32_t si[U], sj[U];
        uint32_t ei[U], ej[U];
#pragma unroll
        for (int r = 0; r < U; ++r) {
            ok[r] = i[r] >= 0 && i[r] < a.limit;
            if (!ok[r] && w[r] == 0 && d[r] == 0) flag_index(a);
            const int64_t ii = ok[r] ? i[r] : 0;
            int64_t j = ii - d[r];
            if (j < 0) j = ok[r] ? j + a.capacity : 0;
            v[r] = *(reinterpret_cast<const V*>(a.src + j * a.row_bytes) + w[r]);
            si[r] = sj[r] = 0;
            ei[r] = ej[r] = 0;
            if (a.stack > 1) {  // kernel argument: uniform
                si[r] = a.step[ii];
                sj[r] = a.step[j];
                ei[r] = a.episode[ii];
                ej[r] = a.episode[j];
            }
        }
        O o[U];
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const int32_t dr = (int32_t)d[r];
            const bool valid = ok[r] & ((dr == 0) | ((dr <= si[r]) & (ei[r] == ej[r]) & (sj[r] == si[r] - dr)));
            o[r] = convert_unit<XF>(a, w[r], v[r], lut);
            if (!valid) o[r] = zero_unit<O>();
            asm volatile("" : "+v"(o[r]));  // conversions ahead of the stores, as in finish()
        }
        O* out = reinterpret_cast<O*>(a.out) + first;
        const uint32_t n = total - first < kTile ? total - first : kTile;  // the tile's units
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const uint32_t e = r * kThreads + threadIdx.x;
            if (e < n) __builtin_nontemporal_store(o[r], out + e);
        }
    }
}

// ragged token packing: one workgroup per sample; each lane handles up to 4
// quads (16 elements) per pass, all loads issued before the stores
__global__ __launch_bounds__(kThreads) void k_pack(PackArgs a) {
    const int64_t b = blockIdx.x;
    if (b >= a.n) {  // the weights workgroup
        is_weights_block<kThreads>(a.weights);
        return;
    }
    pack_row<kThreads>(a, b, a.idx[b]);
}

}  // namespace

int device_cus() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cached[dev]) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
        cached[dev] = cus;
    }
    return cached[dev];
}

// Stores: the persistent kernel writes through at agent scope (outputs of at
// most 128 MB: no dirty L2 lines left for the end-of-kernel write-back; the
// DQN gather 15.2 -> 14.9 us), the one-item-per-workgroup kernel writes
// non-temporal (larger outputs stream: PPO minibatch 325 us against 342 us
// written through and 344 us with plain stores; large bf16 86 against 93 and
// 94 us).
template <int XF>
hipError_t launch_gather_xf(const GatherArgs& a, hipStream_t s, int64_t tail_blocks) {
    const int64_t units = a.row_bytes >> UnitOf<XF>::kShift;
    const int64_t bpf = a.out && units > 0 ? (units + kUnitsPerBlock - 1) / kUnitsPerBlock : 0;
    const int64_t n_items = a.n * a.stack * bpf;
    if (n_items + tail_blocks == 0) return hipSuccess;
    const int64_t out_bytes = a.n * a.stack * a.row_bytes *
                              (XF == CONDUIT_XF_U8_F32 ? 4 : XF == CONDUIT_XF_U8_BF16_NORM ? 2 : 1);
    const bool norm = XF == CONDUIT_XF_U8_BF16_NORM;
    // frames to fp32 that fill at least 3/4 of their items
    const bool full = XF == CONDUIT_XF_U8_F32 && units * 4 >= bpf * kUnitsPerBlock * 3;
    const bool rows4 = XF == CONDUIT_XF_NONE && units * 2 >= bpf * kUnitsPerBlock && out_bytes > kPipeMaxOutBytes;
    const bool sampled = a.weights.w != nullptr;
    const bool few = out_bytes <= kItemsMaxOutBytes && (sampled || a.limit * a.row_bytes > kFlatMaxSource);
    const bool items = rows4 || (full && (few || (sampled && out_bytes > kPipeMaxOutBytes)));
    const bool flat = units <= kFlatMaxUnits || (a.stack == 1 && !items && (!norm || units <= kFlatMaxNormUnits));
    const int64_t total = a.n * a.stack * units;
    if (n_items > 0 && flat && total < (1ll << 31) - kThreads * kFlatUnroll) {
        // the most units per lane that still gives every compute unit
        // kFlatWgsPerCu workgroups
        const int64_t per = total / (kThreads * kFlatWgsPerCu * (int64_t)device_cus());
        const Div31 du = make_div31((uint32_t)units), ds = make_div31((uint32_t)a.stack);
        auto go = [&](auto U) {
            const int64_t wgs = (total + kThreads * U.value - 1) / (kThreads * U.value);
            const int64_t cap = norm ? kFlatLoopWgs * device_cus() : wgs;
            hipLaunchKernelGGL((k_gather_flat<XF, U.value>), dim3((unsigned)((wgs < cap ? wgs : cap) + tail_blocks)),
                               dim3(kThreads), 0, s, a, (uint32_t)units, du, ds, (uint32_t)total, (int32_t)tail_blocks);
        };
        if (per >= 4) go(std::integral_constant<int, 4>{});
        else if (per >= 2) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 1>{});
        return hipGetLastError();
    }
    if (out_bytes <= kPipeMaxOutBytes) {
        // small batches: persistent pipelined workgroups
        const int64_t frame_grid = n_items < 4LL * device_cus() ? n_items : 4LL * device_cus();
        hipLaunchKernelGGL((k_gather_pipe<XF>), dim3((unsigned)(frame_grid + tail_blocks)), dim3(kThreads), 0,
                           s, a, (int32_t)bpf, n_items, (int32_t)frame_grid, (int32_t)tail_blocks);
    } else {
        // large batches: one workgroup per item
        hipLaunchKernelGGL((k_gather_rows<XF>), dim3((unsigned)(n_items + tail_blocks)), dim3(kThreads), 0, s,
                           a, (int32_t)bpf, (int32_t)tail_blocks);
    }
    return hipGetLastError();
}

bool copy16(const GatherArgs& a) {
    return a.xform == CONDUIT_XF_NONE &&
           ((reinterpret_cast<uintptr_t>(a.src) | reinterpret_cast<uintptr_t>(a.out) | (uintptr_t)a.row_bytes) & 15) == 0;
}

hipError_t launch_gather(const GatherArgs& a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    const bool scalars = a.out_action || a.out_reward || a.out_done || a.ncols > 0;
    // scalar-column workgroups and the weights workgroup, at the head of the grid
    const int64_t tail_blocks = (scalars ? (a.n + kThreads - 1) / kThreads : 0) + (a.weights.w ? 1 : 0);
    if (copy16(a)) return launch_gather_xf<kXfCopy16>(a, s, tail_blocks);
    switch (a.xform) {
        case CONDUIT_XF_NONE: return launch_gather_xf<CONDUIT_XF_NONE>(a, s, tail_blocks);
        case CONDUIT_XF_U8_F32: return launch_gather_xf<CONDUIT_XF_U8_F32>(a, s, tail_blocks);
        case CONDUIT_XF_U8_BF16_NORM: return launch_gather_xf<CONDUIT_XF_U8_BF16_NORM>(a, s, tail_blocks);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pack(const PackArgs& a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)(a.n + (a.weights.w ? 1 : 0))), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace conduit
