// Generalised advantage estimation over packed (right-padded) sequences, one
// workgroup per sequence: shared by the packed GAE kernel and the fused sampler +
// packing + GAE kernel (its pack workgroup as it is).
#pragma once
#include "common.h"

namespace conduit {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kRsrcRaw32 = 0x00020000;  // raw buffer descriptor, 32-bit data format
constexpr int kAgentScopeStore = 16;    // cache policy SC1: written through at agent scope

// A double moved by one DPP control; lanes with no source keep `id`.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double x, double id) {
    const uint64_t b = (uint64_t)__double_as_longlong(x), o = (uint64_t)__double_as_longlong(id);
    const uint32_t lo =
        (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(b >> 32),
                                                              CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One step of a wavefront prefix scan of affine maps whose lanes run backwards
// in time: the source lane (lower) covers later steps than this one.
template <int CTRL, int ROWS>
__device__ __forceinline__ void later_scan_step(double& P, double& S) {
    const double p2 = dpp_f64<CTRL, ROWS>(P, 1.0);
    const double s2 = dpp_f64<CTRL, ROWS>(S, 0.0);
    S = S + P * s2;
    P = P * p2;
}

constexpr int kDppWaveShr1 = 0x138;  // lane i reads lane i - 1 across the whole wavefront

// g^e (e >= 0) by binary exponentiation in fp64
__device__ __forceinline__ double pow_int(double g, int64_t e) {
    double r = 1.0;
    for (; e; e >>= 1, g *= g)
        if (e & 1) r *= g;
    return r;
}

// A packed row without values (V = 0): the only non-zero TD residual is the
// last live element's reward R, so A_t = R (gamma lambda)^(L-1-t) for t < L,
// 0 beyond, and R_t = A_t.  Each lane takes 16-byte vectors of the row: the
// vector's last live element from the closed form, the ones before it by the
// recursion's own step A_t = gamma lambda A_{t+1}.  No element waits for
// another lane: no scan, no barrier, no LDS.
template <int NT>
__device__ void gae_packed_row_novalue(const GaePackedArgs& a, int64_t b, int64_t L, double R) {
    const int64_t Lmax = a.Lmax;
    float* adv = a.adv + b * Lmax;
    float* ret = a.ret + b * Lmax;
    const double gl = a.gamma * a.lambda;
    // the values of elements [t, t + 4): o[i] for t + i
    auto quad = [&](int64_t t, f32x4& o) {
        const int64_t hi = (t + 3 < L - 1 ? t + 3 : L - 1);  // last live element of the quad
        double A = hi >= t ? R * pow_int(gl, L - 1 - hi) : 0.0;
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            if (t + i > hi) {
                o[i] = 0.0f;
            } else {
                if (t + i < hi) A = gl * A;
                o[i] = (float)A;
            }
        }
    };
    const bool vec = ((reinterpret_cast<uintptr_t>(adv) | reinterpret_cast<uintptr_t>(ret)) & 15) == 0 &&
                     (Lmax & 3) == 0 && Lmax * 4 <= 0x7fffffffll;  // uniform
    if (vec) {
        const int nb = __builtin_amdgcn_readfirstlane((int)(Lmax * 4));
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(adv, 0, nb, kRsrcRaw32);
        const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(ret, 0, nb, kRsrcRaw32);
        for (int64_t t = (int64_t)threadIdx.x * 4; t < Lmax; t += (int64_t)NT * 4) {
            f32x4 o;
            quad(t, o);
            // write-through at agent scope, as the scanned path stores its rows
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), ra, (int)(t * 4), 0, kAgentScopeStore);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rr, (int)(t * 4), 0, kAgentScopeStore);
        }
    } else {
        for (int64_t t = (int64_t)threadIdx.x * 4; t < Lmax; t += (int64_t)NT * 4) {
            f32x4 o;
            quad(t, o);
            for (int i = 0; i < 4 && t + i < Lmax; ++i) {
                adv[t + i] = o[i];
                ret[t + i] = o[i];
            }
        }
    }
}

// 16 bytes at a 4-byte aligned address
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Powers of gamma lambda for the scan of a block whose lanes all have the same
// map, A_start = (gamma lambda)^4 A_end + S: only the S parts move then.
struct LanePowers {
    double p1, p2, p4, p8;  // of 1, 2, 4, 8 lanes
    double row, half;       // of the lanes up to this one in its row of 16, its half of 32
    double later, block;    // of the lanes before this one (later in time), of all 64
    __device__ __forceinline__ LanePowers(double gl, int lane) {
        p1 = (gl * gl) * (gl * gl);
        p2 = p1 * p1;
        p4 = p2 * p2;
        p8 = p4 * p4;
        const double p16 = p8 * p8, p32 = p16 * p16;
        const double in_row = ((lane & 1) ? p1 : 1.0) * ((lane & 2) ? p2 : 1.0) * ((lane & 4) ? p4 : 1.0) *
                              ((lane & 8) ? p8 : 1.0);
        const double in_half = in_row * ((lane & 16) ? p16 : 1.0);
        row = in_row * p1;
        half = in_half * p1;
        later = in_half * ((lane & 32) ? p32 : 1.0);
        block = p32 * p32;
    }
};

// GAE of packed row b, of L live elements (0 <= L <= Lmax) with reward R on
// the last one, by one workgroup of NT lanes, in passes of 4 NT J elements from
// the row's end.  A wavefront owns 256 J consecutive elements of a pass, as J
// blocks of one 16-byte vector per lane, so values and outputs stay in registers
// and every access is contiguous over the wavefront.  Lanes run backwards in
// time (lane 0 holds a block's last vector), so the suffix composition of the
// lanes' affine maps is a DPP prefix scan; the blocks' maps compose in scalar
// order, the wavefronts' through LDS with one barrier per pass.  A block that
// ends before the sequence's last element has the same coefficient everywhere,
// so only the S parts of its maps are scanned (LanePowers): the fp64 arithmetic
// bounds the kernel as much as the chain of its latencies does.  The next pass's
// values load before the current one is worked on; padding is not read.  Outputs
// may take the values' place: a wavefront stores only elements it has loaded
// itself, and the one value it needs of another's span is used before that
// wavefront stores (or comes through LDS, from the later pass's first wavefront).
// Against staging each row through LDS, 4,096 elements at a time: [256, 8192] 9.3
// -> 8.0 us, [244, 16384] 16.0 -> 11.4, rows off 16 bytes [244, 16383] 23.0 ->
// 11.2, [1024, 1024] 10.2 -> 5.8, [1024, 4096] 14.0 -> 11.8; the fused sample +
// pack + GAE of [1024, 1024] 21.3 -> 19.2.
// ONE: one pass takes the row (Lmax <= 4 NT J); compiled without the next pass's
// registers ([1000, 4000] 10.4 -> 9.1 us, [1024, 2000] 8.2 -> 7.2).
template <int NT, int J, bool ONE>
__device__ void gae_packed_row(const GaePackedArgs& a, int64_t b, int64_t L, double R) {
    if (!a.value) {  // kernel argument: uniform
        gae_packed_row_novalue<NT>(a, b, L, R);
        return;
    }
    constexpr int kWaves = NT / kWave;
    constexpr int64_t kWaveSpan = 4 * kWave * J;  // elements of a wavefront and pass
    constexpr int64_t kPass = kWaveSpan * kWaves;
    __shared__ double sWP[2][kWaves], sWS[2][kWaves];
    __shared__ float sV[2][kWaves];  // the wavefronts' first values
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = lane_id();
    const int64_t Lmax = a.Lmax;
    const float* val = a.value + b * Lmax;  // may be adv or ret
    float* adv = a.adv + b * Lmax;
    float* ret = a.ret + b * Lmax;
    const double gl = a.gamma * a.lambda;
    const int own = (kWave - 1 - lane) * 4;  // the lane's vector in a block
    // the lane's vectors of the pass at `base`, and the value after the
    // wavefront's span (0 where nothing live lies there, and for the last
    // wavefront, whose next value is the later pass's)
    auto load = [&](int64_t base, f32x4 (&v)[J], float& after) {
        const int64_t w0 = base + wv * kWaveSpan;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int64_t t = w0 + j * 4 * kWave + own;
            v[j] = (f32x4)(0.0f);
            if (t < L) {
                if (t + 3 < Lmax) {
                    v[j] = *reinterpret_cast<const f32x4u*>(val + t);
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) v[j][i] = t + i < Lmax ? val[t + i] : 0.0f;
                }
            }
        }
        const int64_t e = w0 + kWaveSpan;
        after = wv < kWaves - 1 && e < L ? val[e] : 0.0f;
    };
    auto put = [&](int64_t t, const f32x4& x, const f32x4& y) {
        if (t + 3 < Lmax) {
            *reinterpret_cast<f32x4u*>(adv + t) = x;
            *reinterpret_cast<f32x4u*>(ret + t) = y;
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (t + i < Lmax) {
                    adv[t + i] = x[i];
                    ret[t + i] = y[i];
                }
            }
        }
    };
    // a block whose elements all come before the sequence's last one
    auto inside = [&](int64_t b0) { return b0 + 4 * kWave < L; };
    const LanePowers pw(gl, lane);
    int64_t base = (Lmax + kPass - 1) / kPass * kPass - kPass;
    for (; base >= L && base >= 0; base -= kPass) {  // passes of padding only (uniform)
#pragma unroll
        for (int j = 0; j < J; ++j) put(base + wv * kWaveSpan + j * 4 * kWave + own, (f32x4)(0.0f), (f32x4)(0.0f));
    }
    f32x4 v[J], vn[J];
    float after = 0.0f, after_n = 0.0f;
    if (base >= 0) load(base, v, after);
    double carry = 0.0;  // A at the start of the later pass
    for (int par = 0; base >= 0; base -= kPass, par ^= 1) {
        if (!ONE && base > 0) load(base - kPass, vn, after_n);
        const int64_t w0 = base + wv * kWaveSpan;
        double end[J];            // V after the lane's vector
        double eP[J], eS[J];      // the block's later lanes
        double bP[J], bS[J];      // the wavefront's later blocks
        double wP = 1.0, wS = 0.0;
#pragma unroll
        for (int j = J - 1; j >= 0; --j) {
            const int64_t b0 = w0 + j * 4 * kWave, t = b0 + own;
            bP[j] = wP;
            bS[j] = wS;
            eP[j] = 1.0;
            eS[j] = 0.0;
            end[j] = 0.0;
            if (b0 >= L) continue;  // padding only (uniform)
            const float next = j + 1 < J ? __uint_as_float(__builtin_amdgcn_readlane(
                                               __float_as_uint(v[j + 1 < J ? j + 1 : j][0]), kWave - 1))
                                         : after;
            const float up = __uint_as_float(dpp_u32<kDppWaveShr1, 0xf>(__float_as_uint(v[j][0]), __float_as_uint(next)));
            double S = 0.0, tP;
            if (inside(b0)) {  // uniform
                end[j] = (double)up;
                double v_next = end[j];
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const double x = (double)v[j][i];
                    S = (a.gamma * v_next - x) + gl * S;
                    v_next = x;
                }
                S += pw.p1 * dpp_f64<kDppRowShr + 1, 0xf>(S, 0.0);
                S += pw.p2 * dpp_f64<kDppRowShr + 2, 0xf>(S, 0.0);
                S += pw.p4 * dpp_f64<kDppRowShr + 4, 0xf>(S, 0.0);
                S += pw.p8 * dpp_f64<kDppRowShr + 8, 0xf>(S, 0.0);
                S += pw.row * dpp_f64<kDppRowBcast15, 0xa>(S, 0.0);
                S += pw.half * dpp_f64<kDppRowBcast31, 0xc>(S, 0.0);
                eP[j] = pw.later;
                tP = pw.block;
            } else {
                end[j] = t + 4 < L ? (double)up : 0.0;  // what lies past the sequence is never used
                double v_next = end[j];
                double P = 1.0;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (t + i < L) {
                        const double x = (double)v[j][i];
                        const bool last = t + i == L - 1;
                        S = last ? R - x : (a.gamma * v_next - x) + gl * S;
                        P = last ? 0.0 : gl * P;
                        v_next = x;
                    }
                }
                // shifts by 1, 2, 4, 8 in a row, then the row broadcasts
                later_scan_step<kDppRowShr + 1, 0xf>(P, S);
                later_scan_step<kDppRowShr + 2, 0xf>(P, S);
                later_scan_step<kDppRowShr + 4, 0xf>(P, S);
                later_scan_step<kDppRowShr + 8, 0xf>(P, S);
                later_scan_step<kDppRowBcast15, 0xa>(P, S);
                later_scan_step<kDppRowBcast31, 0xc>(P, S);
                eP[j] = dpp_f64<kDppWaveShr1, 0xf>(P, 1.0);
                tP = __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(P), kWave - 1));
            }
            eS[j] = dpp_f64<kDppWaveShr1, 0xf>(S, 0.0);
            const double tS = __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(S), kWave - 1));
            wS = tS + tP * wS;
            wP = tP * wP;
        }
        if (lane == kWave - 1) {  // holds the span's first vector
            sWP[par][wv] = wP;
            sWS[par][wv] = wS;
            if (!ONE) sV[par][wv] = v[0][0];
        }
        lds_barrier();  // the pass before used the other half
        double lP = 1.0, lS = 0.0;  // the later wavefronts
        double tP = 1.0, tS = 0.0;  // the whole pass
#pragma unroll
        for (int w = kWaves - 1; w >= 0; --w) {
            if (w == wv) {
                lP = tP;
                lS = tS;
            }
            tS = sWS[par][w] + sWP[par][w] * tS;
            tP = sWP[par][w] * tP;
        }
        const double A_w = lP * carry + lS;  // A at the end of the wavefront's span
#pragma unroll
        for (int j = J - 1; j >= 0; --j) {
            const int64_t b0 = w0 + j * 4 * kWave, t = b0 + own;
            double A = eP[j] * (bP[j] * A_w + bS[j]) + eS[j];
            double v_next = end[j];
            f32x4 oa = (f32x4)(0.0f), orr = (f32x4)(0.0f);
            if (inside(b0)) {
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const double x = (double)v[j][i];
                    A = (a.gamma * v_next - x) + gl * A;
                    oa[i] = (float)A;
                    orr[i] = (float)(A + x);
                    v_next = x;
                }
            } else if (b0 < L) {
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (t + i < L) {
                        const double x = (double)v[j][i];
                        A = t + i == L - 1 ? R - x : (a.gamma * v_next - x) + gl * A;
                        oa[i] = (float)A;
                        orr[i] = (float)(A + x);
                        v_next = x;
                    }
                }
            }
            put(t, oa, orr);
        }
        if constexpr (ONE) break;
        carry = tP * carry + tS;
#pragma unroll
        for (int j = 0; j < J; ++j) v[j] = vn[j];
        after = wv == kWaves - 1 ? sV[par][0] : after_n;
    }
}

}  // namespace
}  // namespace conduit
