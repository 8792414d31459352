// Sequence-parallel form of the decayed linear-attention pass (arXiv 2307.14995, Sec. 3.3:
// the recurrence kv_t = lambda kv_{t-1} + k_t^T v_t is linear in the state, so a chain cut
// into segments needs only each segment's end state from a zero start and a scan over
// them).  This file holds the scan: with L[g] the end state of segment g computed from a
// zero state and len(g) its token count,
//
//     S[0] = initial state,     S[g+1] = lambda^len(g) S[g] + L[g].
//
// The states array [count][chains][segs][D*D] is rewritten in place from L[.] to S[.] (the
// state at each segment's start); the state after the last segment goes to kv_out.
#include <type_traits>
#include "ltn_kernels.h"

namespace ltn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kThreads = 256;
constexpr int kAhead = 8;                // segments whose end states a thread has in flight

// A thread owns four adjacent elements of one (pass, chain)'s state and walks the segments in
// order.  Bound by the latency of the loads, then by bytes (each state read and written once):
// what a step needs from the one before it is one fmaf, so the end states of eight segments are
// fetched together, ahead of the powers of lambda.  One element per thread with each load behind
// the previous segment's store took 8.4 us for 32 chains x 5 segments of 128 x 128 (21 MB), 12.7
// for 32 x 8; this form 6.0 and 7.8.
__global__ __launch_bounds__(kThreads)
void segment_scan_kernel(float* states, const float* __restrict__ kv_in, float* __restrict__ kv_out,
                         const float* __restrict__ decay, int chains, int H, int segs,
                         int seg_len, long long N, int DD) {
    const int per = DD / (4 * kThreads);                       // workgroups per state
    const int pc = blockIdx.x / per;                           // pass * chains + chain
    const int e = (blockIdx.x % per * kThreads + threadIdx.x) * 4;
    const int pass = pc / chains, chain = pc % chains;
    float* s = states + (size_t)pc * segs * DD + e;
    const bool final_state = pass == 0 && kv_out;
    // the last segment's end state exists only if someone asked for the final state
    const int have = kv_out ? segs : segs - 1;
    f32x4 run = (pass == 0 && kv_in) ? *(const f32x4*)(kv_in + (size_t)chain * DD + e) : f32x4{0.f, 0.f, 0.f, 0.f};
    float lam_full = 0.f, lam_last = 0.f;
    bool flushed = false;                // lambda^len is zero although lambda is not
    for (int g0 = 0; g0 < segs; g0 += kAhead) {
        f32x4 local[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            local[i] = g0 + i < have ? *(const f32x4*)(s + (size_t)(g0 + i) * DD) : f32x4{0.f, 0.f, 0.f, 0.f};
        if (g0 == 0) {
            const float lam = decay[chain % H];
            lam_full = decay_pow(lam, seg_len);
            lam_last = final_state ? decay_pow(lam, (int)(N - (long long)(segs - 1) * seg_len)) : 0.f;
            flushed = lam > 0.f && lam_full == 0.f;
        }
        // keep_inf: an infinite entry stays infinite, as it does under the whole-chain pass's one
        // factor per block, instead of becoming 0 x Inf.  A loop of its own: tested per segment it
        // cost 0.5 us of an 8 us scan.
        auto walk = [&](auto keep_inf) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                if (g0 + i >= segs) break;
                *(f32x4*)(s + (size_t)(g0 + i) * DD) = run;
                const float f = g0 + i + 1 < segs ? lam_full : lam_last;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    run[j] = fmaf(decltype(keep_inf)::value && __builtin_isinf(run[j]) ? 1.f : f, run[j], local[i][j]);
            }
        };
        if (flushed) walk(std::true_type{});
        else walk(std::false_type{});
    }
    if (final_state) *(f32x4*)(kv_out + (size_t)chain * DD + e) = run;
}

// The scan of a backward's three passes from the end states of two: dV = pass(K, Q, dO) and dK = pass(V, dO, Q) walk the
// tokens together, and their states, sums of q_t^T dO_t and of dO_t^T q_t, are each other's transposes.  So no
// sweep is run for dK; its states are written here.  A workgroup has a tile of kTile x kTile elements of a (dV and dK, or
// dQ) state of one chain and walks the segments; dK's tile is turned round in LDS.
constexpr int kTile = 32;

__global__ __launch_bounds__(kTile * kTile / 4)
void segment_scan_pair_kernel(const ScanStates s, const float* __restrict__ decay, int chains, int H, int segs, int seg_len,
                              long long N, int D) {
    constexpr int PITCH = kTile + 4;       // whole 16-byte pieces
    __shared__ __attribute__((aligned(16))) float tile[2][kTile * PITCH];
    const int per = (D / kTile) * (D / kTile);
    const int uc = blockIdx.x / per, t = blockIdx.x % per;
    const int unit = uc / chains, chain = uc % chains;         // 0: dV and dK, 1: dQ
    const int row0 = t / (D / kTile) * kTile, col0 = t % (D / kTile) * kTile;
    const int r = threadIdx.x / (kTile / 4), c = threadIdx.x % (kTile / 4) * 4;
    const int pass = unit ? 2 : 0;
    auto seg_off = [&](int g) -> size_t {
        if (!s.rows) return (size_t)g * D * D;
        const long long start = (long long)g * seg_len, n = g + 1 == segs ? N - start : seg_len;
        return (size_t)(s.rev[pass] ? N - start - n : start) * D;
    };
    float* const own = s.p[pass] + (size_t)chain * s.chain_stride + (size_t)(row0 + r) * D + col0 + c;
    float* const turned = s.p[1] + (size_t)chain * s.chain_stride + (size_t)(col0 + r) * D + row0 + c;
    f32x4 run = {0.f, 0.f, 0.f, 0.f};
    float lam_full = 0.f;
    bool flushed = false;
    for (int g0 = 0; g0 < segs; g0 += kAhead) {
        f32x4 local[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            local[i] = g0 + i + 1 < segs ? *(const f32x4*)(own + seg_off(g0 + i)) : f32x4{0.f, 0.f, 0.f, 0.f};
        if (g0 == 0) {
            const float lam = decay[chain % H];
            lam_full = decay_pow(lam, seg_len);
            flushed = lam > 0.f && lam_full == 0.f;
        }
        auto walk = [&](auto keep_inf) {                       // (as above)
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                const int g = g0 + i;
                if (g >= segs) break;
                *(f32x4*)(own + seg_off(g)) = run;
                if (unit == 0) {
                    // two tiles in turn: the barrier of the next segment separates these reads from the writes after it
                    float* const lds = tile[i & 1];
                    *(f32x4*)(lds + r * PITCH + c) = run;
                    __syncthreads();
                    f32x4 x;
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = lds[(c + j) * PITCH + r];
                    *(f32x4*)(turned + seg_off(g)) = x;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    run[j] = fmaf(decltype(keep_inf)::value && __builtin_isinf(run[j]) ? 1.f : lam_full, run[j], local[i][j]);
            }
        };
        if (flushed) walk(std::true_type{});
        else walk(std::false_type{});
    }
}

}  // namespace

hipError_t launch_segment_scan_pair(const ScanStates& s, const float* decay, int chains, int H, int segs, long long seg_len,
                                    long long N, int D, hipStream_t stream) {
    if (chains < 1 || segs < 1 || seg_len <= 0 || seg_len > 0x7fffffffLL || D % kTile != 0) return hipErrorInvalidValue;
    const long long wgs = 2LL * chains * (D / kTile) * (D / kTile);
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(segment_scan_pair_kernel, dim3((unsigned)wgs), dim3(kTile * kTile / 4), 0, stream, s, decay, chains, H,
                       segs, (int)seg_len, N, D);
    return hipGetLastError();
}

hipError_t launch_segment_scan(float* states, const float* kv_in, float* kv_out, const float* decay,
                               int count, int chains, int H, int segs, long long seg_len, long long N,
                               int D, hipStream_t stream, int DC) {
    if (DC == 0) DC = D;
    if (count < 1 || chains < 1 || segs < 1 || seg_len <= 0 || seg_len > 0x7fffffffLL) return hipErrorInvalidValue;
    if (D * DC % (4 * kThreads) != 0) return hipErrorInvalidValue;     // every state width of the library is a multiple
    const long long wgs = (long long)count * chains * (D * DC / (4 * kThreads));
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(segment_scan_kernel, dim3((unsigned)wgs), dim3(kThreads), 0, stream,
                       states, kv_in, kv_out, decay, chains, H, segs, (int)seg_len, N, D * DC);
    return hipGetLastError();
}

}  // namespace ltn
