// Gated SimpleRMSNorm on rows (arXiv 2307.14995, Sec. 3.1.2 Eq. 3: O = Norm(.) (.) U, with
// the SimpleRMSNorm of Sec. 3.1.3 taken per head over its D features):
//
//     y = x / sqrt(mean(x^2) + eps) (.) u
//
// and its derivative.  The forward of this map is normally fused into the attention
// forward (the gated epilogue of the pass kernels); these stand-alone kernels serve the
// backward (which needs the stored attention output x) and callers that hold x already.
// The forward may run in place (y = x's memory: a lane reads its piece before it writes it).
// Streaming kernels, HBM-bound: every lane owns 16 bytes of one row, a row's lanes are
// neighbours in one wave and reduce with cross-lane shuffles (rows of 96 features take 16 or 32
// lanes of which 12 or 24 hold data); fp32 arithmetic.
// ONCE, from kOnceBytes a tensor on: loads that leave the caches first, and a derivative's du stored so, which a projection's
// gradient reads later.  dx is stored plainly, for the attention's backward, which reads it next, and so is y, for the
// output projection, up to kOnceYBytes.  us, rotating inputs.
//   no hints / loads / loads and du / everything.  Derivative, attention backward, copies of
//     dq, dk, dv, du: 32 chains x 2048 x 128 (16 MiB a tensor) 117.5 / 117.5 / 118.5 / 118.9, 48 x 2048 145.6 / 145.6 /
//     144.4 / 144.4, 64 x 2048 177.5 / 175.1 / 171.5 / 173.4, 128 x 2048 332 / 332 / 327 / 338, 128 x 8192 1291 / 1294 / 1268
//     / 1275; the copy of du before the attention 96 x 2048 186.8 / 177.0 / 174.0 / 187.0, 128 x 2048 222.7 / 217.5 / 217.7 /
//     225.7; no copies 128 x 2048 184.0 / 182.5 / 180.1 / 188.3
//   y plain / once.  Mixer step with copies of what it returns: 96 x 2048 (48 MiB) 329.9 / 331.2, 128 x 2048 (64) 396 / 398 and
//     400.7 / 401.6, 160 x 2048 492 / 493, 180 x 2500 (110) 709 / 705, 128 x 4096 790 / 778, 96 x 4096 x 256 (192) 1558 / 1545,
//     102 x 25568 x 64 2163 / 2151; without them 128 x 2048 261 / 253, 128 x 4096 522 / 504, 102 x 25568 x 64 1557 / 1510.
//     Forward and copy of y: 64 x 3000 (47) 92.8 / 94.4, 96 x 1500 (35) 64.6 / 67.0, 128 x 2048 107.7 / 109.3 (no hints
//     109.4), 160 x 2048 139 / 142 (144), 64 x 8192 253.5 / 253.6 (266), 128 x 8192 457 / 449 (463)
//   The kernels alone, 2^18 rows of 128, no hints and so, outputs in other memory each time (in one place): forward 38.5 and 34.3
//     (34.0 and 34.5), derivative 64.3 and 54.6 (62.8 and 54.7)
#include "ltn_cache.h"
#include "ltn_kernels.h"

namespace ltn {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(float)))) float f32x8;

constexpr long long kOnceBytes = 24 << 20, kOnceYBytes = 64 << 20;

template <bool ONCE> __device__ __forceinline__ u32x4 load16(const void* p) {
    if constexpr (ONCE) return load16_once(p);
    else return *(const u32x4*)p;
}
template <bool ONCE> __device__ __forceinline__ void store16(void* p, u32x4 v) {
    if constexpr (ONCE) store16_once(p, v);
    else *(u32x4*)p = v;
}

template <bool BF16> struct Vec;            // the 16 bytes of one lane as fp32 values
template <> struct Vec<true> {
    static constexpr int N = 8;
    float v[8];
    template <bool ONCE>
    __device__ __forceinline__ void load(const void* p) {
        union { u32x4 u; bf16x8 h; } c;
        c.u = load16<ONCE>(p);
        const f32x8 f = __builtin_convertvector(c.h, f32x8);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = f[i];
    }
    template <bool ONCE>
    __device__ __forceinline__ void store(void* p) const {
        f32x8 f;
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = v[i];
        union { u32x4 u; bf16x8 h; } c;
        c.h = __builtin_convertvector(f, bf16x8);
        store16<ONCE>(p, c.u);
    }
};
template <> struct Vec<false> {
    static constexpr int N = 4;
    float v[4];
    template <bool ONCE>
    __device__ __forceinline__ void load(const void* p) {
        const u32x4 u = load16<ONCE>(p);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(u[i]);
    }
    template <bool ONCE>
    __device__ __forceinline__ void store(void* p) const {
        u32x4 u;
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = __float_as_uint(v[i]);
        store16<ONCE>(p, u);
    }
};

template <int LPR>
__device__ __forceinline__ float row_sum(float x) {   // sum over the LPR neighbouring lanes of a row
#pragma unroll
    for (int m = LPR / 2; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

constexpr int kThreads = 256;

template <int D, bool BF16, bool BWD, bool ONCE, bool ONCE_Y>
__global__ __launch_bounds__(kThreads)
void gate_kernel(const char* x, const char* __restrict__ u, const char* __restrict__ dy,
                 char* o0, char* __restrict__ o1, float eps, long long rows) {
    using V = Vec<BF16>;
    constexpr int ACT = D / V::N;                 // lanes that hold a piece of the row
    constexpr int LPR = ACT <= 8 ? 8 : (ACT <= 16 ? 16 : (ACT <= 32 ? 32 : 64));   // lanes given to a row (96 features: 12 of 16, 24 of 32)
    constexpr int RPW = kThreads / LPR;           // rows per workgroup step
    static_assert(D % V::N == 0 && ACT <= 64, "a row's lanes sit in one wave");
    const int sub = threadIdx.x % LPR;
    const bool live = sub < ACT;                  // idle lanes of a row contribute zeros and store nothing
    long long r = (long long)blockIdx.x * RPW + threadIdx.x / LPR;
    const long long stride = (long long)gridDim.x * RPW;
    // every lane of a wave runs the same number of steps (the shuffles need all of a
    // row's lanes); rows past the end are skipped as whole rows
    for (; r < rows; r += stride) {
        const size_t off = ((size_t)r * ACT + (live ? sub : 0)) * 16;
        V xv, uv;
        xv.template load<ONCE>(x + off);
        uv.template load<ONCE>(u + off);
        if (!live) {
#pragma unroll
            for (int i = 0; i < V::N; ++i) xv.v[i] = 0.f;
        }
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < V::N; ++i) ss = fmaf(xv.v[i], xv.v[i], ss);
        if constexpr (!BWD) {
            ss = row_sum<LPR>(ss);
            const float rstd = 1.0f / sqrtf(ss * (1.0f / D) + eps);
            V yv;
#pragma unroll
            for (int i = 0; i < V::N; ++i) yv.v[i] = xv.v[i] * rstd * uv.v[i];
            if (live) yv.template store<ONCE_Y>(o0 + off);
        } else {
            V gv;
            gv.template load<ONCE>(dy + off);
            float dot = 0.f;
#pragma unroll
            for (int i = 0; i < V::N; ++i) dot = fmaf(gv.v[i] * uv.v[i], xv.v[i], dot);
            ss = row_sum<LPR>(ss);
            dot = row_sum<LPR>(dot);
            const float rstd = 1.0f / sqrtf(ss * (1.0f / D) + eps);
            const float mean = dot * rstd * (1.0f / D);       // mean of (dy u) (.) (x rstd)
            V dx, du;
#pragma unroll
            for (int i = 0; i < V::N; ++i) {
                const float n = xv.v[i] * rstd;
                du.v[i] = gv.v[i] * n;
                dx.v[i] = (gv.v[i] * uv.v[i] - n * mean) * rstd;
            }
            if (live) {
                dx.template store<false>(o0 + off);
                du.template store<ONCE>(o1 + off);
            }
        }
    }
}

template <int D, bool BF16, bool BWD>
hipError_t launch_gate_t(const void* x, const void* u, const void* dy, void* o0, void* o1, float eps,
                         long long rows, hipStream_t stream) {
    constexpr int ACT = D / Vec<BF16>::N;
    constexpr int RPW = kThreads / (ACT <= 8 ? 8 : (ACT <= 16 ? 16 : (ACT <= 32 ? 32 : 64)));
    long long wgs = (rows + RPW - 1) / RPW;
    if (wgs > 256 * 16) wgs = 256 * 16;           // grid-stride beyond 16 workgroups per compute unit
    if (wgs <= 0) return hipSuccess;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(kThreads), 0, stream,
                           (const char*)x, (const char*)u, (const char*)dy, (char*)o0, (char*)o1, eps, rows);
    };
    const long long bytes = rows * ACT * 16;
    if (!BWD && bytes >= kOnceYBytes) launch(gate_kernel<D, BF16, BWD, true, !BWD>);
    else if (bytes >= kOnceBytes) launch(gate_kernel<D, BF16, BWD, true, false>);
    else launch(gate_kernel<D, BF16, BWD, false, false>);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gate(const void* x, const void* u, const void* dy, void* o0, void* o1, float eps,
                       long long rows, int D, int is_bf16, int is_bwd, hipStream_t stream) {
#define LTN_GATE_CASE(d, b, w) \
    if (D == d && (is_bf16 != 0) == b && (is_bwd != 0) == w) return launch_gate_t<d, b, w>(x, u, dy, o0, o1, eps, rows, stream)
    LTN_GATE_CASE(128, true, false); LTN_GATE_CASE(128, true, true);
    LTN_GATE_CASE(128, false, false); LTN_GATE_CASE(128, false, true);
    LTN_GATE_CASE(64, true, false); LTN_GATE_CASE(64, true, true);
    LTN_GATE_CASE(64, false, false); LTN_GATE_CASE(64, false, true);
    LTN_GATE_CASE(96, true, false); LTN_GATE_CASE(96, true, true);
    LTN_GATE_CASE(96, false, false); LTN_GATE_CASE(96, false, true);
    LTN_GATE_CASE(256, true, false); LTN_GATE_CASE(256, true, true);
    LTN_GATE_CASE(256, false, false); LTN_GATE_CASE(256, false, true);
#undef LTN_GATE_CASE
    return hipErrorInvalidValue;
}

}  // namespace ltn
