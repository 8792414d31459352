// Recurrent decode of Lightning Attention (arXiv 2307.14995, Sec. 3.3, Algorithm 2), per
// (batch, head), for S >= 1 consecutive tokens in one call:
//     kv <- lambda kv + k_s^T v_s   (fp32),   o_s = q_s kv   (the updated state),  s = 0..S-1
// The state is read once, kept in registers over the S iterations and written once, so a
// call moves 2 D^2 fp32 values per chain whatever S is; with S = 1 (one token per call) the
// step is bound by HBM bandwidth (about half a FLOP per byte), with few chains by latency.  Plain
// fp32 vector code with 16-byte accesses; one workgroup per chain (or per 32 value columns of
// one, below), each thread owns four adjacent state
// columns of a strided set of rows, and the partial dot products per column are reduced
// through LDS.  Queries and keys have DK features, values and outputs DV (the state is
// [DK x DV]); the two differ only behind the LRPE-d expansion of Eq. 1.
#include "ltn_cache.h"
#include "ltn_kernels.h"

namespace ltn {
namespace {

// Threads per workgroup, at least max(DK, DV) (one thread per q/k/v feature).  128 threads
// per 128 x 128 state: measured best on MI355X for the 2048-chain decode workload (39.4 us
// per step against 41.9 with 256 and 39.9 with 1024); larger states keep the same number of
// state values per thread, smaller ones the 128 threads.
constexpr int threads_for(int DK, int DV) {
    return (DK == 96 && DV == 96) ? 96 : (DK * DV / 128 < 128 ? 128 : DK * DV / 128);   // 96: 24 threads per row
}

__device__ __forceinline__ float bf16_bits_to_f32(unsigned short h) {
    return __uint_as_float(((unsigned int)h) << 16);
}

__device__ __forceinline__ unsigned short f32_to_bf16_bits(float f) {   // round to nearest even
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40);  // NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// A state is read once and written once, and the next call that wants it comes after every other layer's.  Loads and
// stores that leave the caches first, or are written through, keep the lines from being written back
// in the middle of the reads.  us a call, plain / once / read once and written through; states of many layers (1.2 GiB in
// turn), of three, and one repeated (in the memory-side cache, below 85 MiB a state):
//     128 x 128    512 chains (32 MiB)   15.8 / 11.2 / 11.4     11.2 / 10.3 / 10.6      8.4 /  8.3 / 10.5
//                  640 (40)              21.0 / 14.3 / 15.3     12.6 / 13.2 / 12.5     11.1 / 10.9 / 12.5
//                  768 (48)              23.5 / 17.3 / 17.7     14.8 / 15.9 / 14.8     12.9 / 12.5 / 14.8
//                  896 (56)              26.7 / 21.0 / 22.0     16.8 / 20.2 / 17.3     16.8 / 18.1 / 17.2
//                 1024 (64)              29.4 / 22.3 / 23.6     19.6 / 21.7 / 19.6     19.6 / 18.8 / 19.5
//                 1280 (80)              37.1 / 30.9 / 31.9     24.6 / 30.4 / 25.3     24.5 / 27.8 / 25.3
//                 2048 (128)             56.9 / 50.2 / 50.9                            39.8 / 47.8 / 41.3
//     64 x 64     1200 (19)               9.3 /  6.7 /  7.1      7.2 /  6.2 /  6.5      5.6 /  5.4 /  6.5
//                 1536 (24)              12.1 /  9.3 /  9.8      8.7 /  8.3 /  8.4      6.4 /  6.0 /  8.4
//                 2048 (32), six sets    15.1 / 12.3 / 12.4     10.7 / 11.8 / 10.2      8.2 /  9.1 / 10.2
//     96 x 96     1000 (35)              17.7 / 12.8 / 13.2     11.5 / 11.7 / 11.2     10.1 /  9.8 / 11.1
//                 1140 (40)              19.9 / 16.3 / 17.4     12.4 / 15.4 / 13.4     11.8 / 13.0 / 13.3
//                 2000 (70)              32.5 / 27.3 / 29.0     22.3 / 26.3 / 23.2     22.3 / 24.8 / 23.2
//     128 x 64    1280 (40)              19.5 / 14.1 / 14.9     13.1 / 13.0 / 12.5     12.8 / 10.8 / 12.5
//                 1600 (50), four sets   24.8 / 19.6 / 20.5     15.7 / 19.0 / 16.4     15.7 / 16.3 / 16.4
//     256 x 128    192 (24), seven sets  11.9 /  9.2 /  9.3      9.2 /  8.8 /  8.8      7.6 /  7.7 /  8.8
//                  256 (32), six sets    16.6 / 12.8 / 13.6     10.7 / 12.4 / 11.0      8.2 /  8.6 / 10.9
//                  512 (64)              29.2 / 25.0 / 26.9     20.8 / 24.4 / 20.8     20.8 / 23.3 / 20.8
//     256 x 256     96 (24)              12.1 /  9.2 /  9.5      9.4 /  8.4 /  8.6      6.8 /  6.5 /  8.6
//                  160 (40)              21.1 / 16.6 / 17.7     13.3 / 15.9 / 13.3     13.2 / 14.3 / 13.1
// A model's many layers gain a fifth to a third either way.  Past the line (through_bytes) a program of few layers would lose up
// to a fifth without writing through, which costs the many up to 8 %; with it the few are within 4 % of plain (96 x 96
// 8), and a single layer's state, repeated, loses up to a third at the line and nothing from 64 MiB on.
union Bits { u32x4 u; float4 f; };
__device__ __forceinline__ float4 load_state(const float4* p) {
    Bits b;
    b.u = load16_once(p);
    return b.f;
}
template <bool THROUGH>
__device__ __forceinline__ void store_state(float4* p, float4 v) {      // (by reference: 256 registers, not 200)
    Bits b;
    b.f = v;
    if constexpr (THROUGH) store16_through(p, b.u);
    else store16_once(p, b.u);
}
constexpr long long through_bytes(int DK) { return (DK == 256 || DK == 64 ? 24LL : 40) << 20; }
bool write_through(int chains, int DK, int DV) { return (long long)chains * DK * DV * 4 >= through_bytes(DK); }

// Order of an output's sum, the same in both kernels below, so that a sequence's output does not depend on
// how many others are in the call: rows in DK / 8 classes (row mod DK / 8) of eight, each summed in the
// rows' order; the classes pairwise, neighbours first, in groups of eight (96 features: in threes); the
// groups one after another.  A thread here has adjacent classes, whose queries and keys are one 16-byte
// read.  One token, us a call, sums over every fourth or eighth row a thread as before, and so: 128 x 128, 400 / 2048
// chains 10.2 / 56.2 and 9.9 / 55.6, 256 x 128, 3000 chains 148.8 and 146.6, 96 x 96, 1024 chains 12.8 and 12.9,
// 256 x 256, 2048 chains 204 and 206.  Classes that lie apart, so that a wave reads adjacent rows: 10.0 /
// 55.8, 146.9, 12.9 and 206.
template <int DK, int DV, bool BF16, bool THROUGH>
__global__ __launch_bounds__(threads_for(DK, DV))
void decode_kernel(const void* __restrict__ q, const void* __restrict__ k, const void* __restrict__ v,
                   void* __restrict__ o, float* __restrict__ kv, const float* __restrict__ decay, int H,
                   int steps) {
    constexpr int kThreads = threads_for(DK, DV);
    constexpr int TX = DV / 4;            // threads across one state row (float4 each)
    constexpr int TY = kThreads / TX;     // rows in flight per sweep
    constexpr int IT = DK / TY;           // rows of a thread
    constexpr int CL = DK / 8, G = CL / TY;   // classes, and those of a thread: G ty .. G ty + G - 1
    constexpr int PG = G == 3 ? 1 : 8 / G;    // threads whose partial sums make a group's
    static_assert(kThreads >= DK && kThreads >= DV && kThreads % TX == 0 && IT == 8 * G && CL == G * TY &&
                  (G == 3 || 8 % G == 0) && TY % PG == 0, "thread layout");
    __shared__ __attribute__((aligned(16))) float qs[DK], ks[DK], vs[DV];
    __shared__ float4 part[TY][TX];

    const int chain = blockIdx.x;
    const int tid = threadIdx.x;
    const float lam = decay[chain % H];
    const int tx = tid % TX, ty = tid / TX;
    float4* S = (float4*)(kv + (size_t)chain * DK * DV) + G * ty * TX + tx;     // row G ty, and from there:
    auto row = [](int it) { return CL * (it / G) + it % G; };
    float4 s[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) s[it] = load_state(S + row(it) * TX);

    for (int step = 0; step < steps; ++step) {
        if (tid < DK) {
            const size_t e = ((size_t)chain * steps + step) * DK + tid;
            if (BF16) {
                qs[tid] = bf16_bits_to_f32(((const unsigned short*)q)[e]);
                ks[tid] = bf16_bits_to_f32(((const unsigned short*)k)[e]);
            } else {
                qs[tid] = ((const float*)q)[e];
                ks[tid] = ((const float*)k)[e];
            }
        }
        if (tid < DV) {
            const size_t e = ((size_t)chain * steps + step) * DV + tid;
            vs[tid] = BF16 ? bf16_bits_to_f32(((const unsigned short*)v)[e]) : ((const float*)v)[e];
        }
        __syncthreads();
        const float4 vv = *(const float4*)(&vs[4 * tx]);
        float4 acc[G];
#pragma unroll
        for (int j = 0; j < G; ++j) acc[j] = float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const float ki = ks[G * ty + row(it)], qi = qs[G * ty + row(it)];
            float4& a = acc[it % G];
            s[it].x = fmaf(lam, s[it].x, ki * vv.x);
            s[it].y = fmaf(lam, s[it].y, ki * vv.y);
            s[it].z = fmaf(lam, s[it].z, ki * vv.z);
            s[it].w = fmaf(lam, s[it].w, ki * vv.w);
            a.x = fmaf(qi, s[it].x, a.x);
            a.y = fmaf(qi, s[it].y, a.y);
            a.z = fmaf(qi, s[it].z, a.z);
            a.w = fmaf(qi, s[it].w, a.w);
        }
#pragma unroll
        for (int m = 1; m < G; m *= 2)
#pragma unroll
            for (int j = 0; j + m < G; j += 2 * m) {           // (three: 0 and 1, then 2)
                acc[j].x += acc[j + m].x;
                acc[j].y += acc[j + m].y;
                acc[j].z += acc[j + m].z;
                acc[j].w += acc[j + m].w;
            }
        part[ty][tx] = acc[0];
        __syncthreads();                  // also: everyone is done with qs/ks/vs of this step
        if (tid < DV) {
            const int cx = tid / 4, comp = tid % 4;
            float sum = 0.f;
#pragma unroll
            for (int y = 0; y < TY; y += PG) {
                float t[PG];
#pragma unroll
                for (int i = 0; i < PG; ++i) t[i] = ((const float*)&part[y + i][cx])[comp];
#pragma unroll
                for (int m = 1; m < PG; m *= 2)
#pragma unroll
                    for (int i = 0; i < PG; i += 2 * m) t[i] += t[i + m];
                sum += t[0];
            }
            const size_t e = ((size_t)chain * steps + step) * DV + tid;
            if (BF16) ((unsigned short*)o)[e] = f32_to_bf16_bits(sum);
            else ((float*)o)[e] = sum;
        }
        // the next step's first barrier separates these reads of `part` from its next writes
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) store_state<THROUGH>(S + row(it) * TX, s[it]);
}

// The same with a chain's value columns split over DV / 32 workgroups: columns are independent of each
// other, and a workgroup a chain waits for a whole state to cross one unit's load path (and leaves units
// idle where chains are few).  A thread holds a class of eight rows of four columns; a wave's classes meet by
// lane swaps, the waves (96 features, a wave and a half: the classes) through LDS.  One token, us of GPU time a call, whole
// state and slices, one state repeated (and states that come from HBM): 128 x 128, 32 / 128 / 384 chains 4.05 /
// 4.96 / 7.71 and 3.10 / 4.34 / 7.40 (4.93 / 6.56 / 12.7 and 3.41 / 6.10 / 12.7); 256 x 256, 32 / 256 / 1024 chains
// 7.77 / 21.5 / 83.4 and 4.35 / 21.2 / 81.9 (10.9 / 29.5 / 107.5 and 6.11 / 30.0 / 106.4).
constexpr int kSliceCols = 32;

template <int DK, int DV, bool BF16, bool THROUGH>
__global__ __launch_bounds__(DK)
void decode_slice_kernel(const void* __restrict__ q, const void* __restrict__ k, const void* __restrict__ v,
                         void* __restrict__ o, float* __restrict__ kv, const float* __restrict__ decay, int H,
                         int steps) {
    constexpr int TX = kSliceCols / 4, TY = DK / TX, IT = DK / TY;       // threads = DK
    constexpr int NS = DV / kSliceCols;
    constexpr bool WHOLE = DK % 64 == 0;  // whole waves: eight classes of rows in each, summed by lane swaps
    constexpr int NP = WHOLE ? DK / 64 : TY;
    static_assert(DV % kSliceCols == 0 && DK % TX == 0 && IT == 8 && (WHOLE || TY % 3 == 0), "thread layout");
    __shared__ float qs[DK], ks[DK], vs[kSliceCols];
    __shared__ float4 part[NP][TX];

    const int chain = blockIdx.x / NS, col0 = (blockIdx.x - chain * NS) * kSliceCols;
    const int tid = threadIdx.x;
    const float lam = decay[chain % H];
    const int tx = tid % TX, ty = tid / TX;
    float4* S = (float4*)(kv + (size_t)chain * DK * DV + col0);
    float4 s[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) s[it] = load_state(S + (size_t)(ty + TY * it) * (DV / 4) + tx);

    auto load = [](const void* p, size_t e) {
        return BF16 ? bf16_bits_to_f32(((const unsigned short*)p)[e]) : ((const float*)p)[e];
    };
    for (int step = 0; step < steps; ++step) {
        const size_t row = (size_t)chain * steps + step;
        qs[tid] = load(q, row * DK + tid);
        ks[tid] = load(k, row * DK + tid);
        if (tid < kSliceCols) vs[tid] = load(v, row * DV + col0 + tid);
        __syncthreads();
        const float4 vv = *(const float4*)(&vs[4 * tx]);
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int i = ty + TY * it;
            const float ki = ks[i], qi = qs[i];
            s[it].x = fmaf(lam, s[it].x, ki * vv.x);
            s[it].y = fmaf(lam, s[it].y, ki * vv.y);
            s[it].z = fmaf(lam, s[it].z, ki * vv.z);
            s[it].w = fmaf(lam, s[it].w, ki * vv.w);
            acc[0] = fmaf(qi, s[it].x, acc[0]);
            acc[1] = fmaf(qi, s[it].y, acc[1]);
            acc[2] = fmaf(qi, s[it].z, acc[2]);
            acc[3] = fmaf(qi, s[it].w, acc[3]);
        }
        if constexpr (WHOLE) {
#pragma unroll
            for (int m = TX; m < 64; m *= 2)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] += __shfl_xor(acc[c], m, 64);
        }
        if (!WHOLE || (tid & 63) < TX) part[WHOLE ? tid / 64 : ty][tx] = float4{acc[0], acc[1], acc[2], acc[3]};
        __syncthreads();                  // also: everyone is done with qs/ks/vs of this step
        if (tid < kSliceCols) {
            auto p = [&](int i) { return ((const float*)&part[i][tid / 4])[tid % 4]; };
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < NP; i += WHOLE ? 1 : 3) sum += WHOLE ? p(i) : (p(i) + p(i + 1)) + p(i + 2);
            const size_t e = row * DV + col0 + tid;
            if (BF16) ((unsigned short*)o)[e] = f32_to_bf16_bits(sum);
            else ((float*)o)[e] = sum;
        }
        // the next step's first barrier separates these reads of `part` from its next writes
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) store_state<THROUGH>(S + (size_t)(ty + TY * it) * (DV / 4) + tx, s[it]);
}

// Slices up to which a call is split; past them the units are full either way, and a slice reads rows
// of 128 bytes where a whole state is one piece (bf16 tokens, slower beyond: 128 x 128, 512 chains 13.5 and
// 14.8 us for 4 tokens; 128 x 64, 1024 chains 14.1 and 15.0 for 4; 96 x 96, 1024 chains 15.8 and 17.3 for 4; 256 x 256,
// 2048 chains 205 and 214 for 1).  Just below the lines the two are within 3 %, but for 256 x 256, 128 and 192 chains out
// of HBM (16.6 and 18.0, 22.4 and 23.4; 384 to 1024 chains: slices ahead by 1 to 6 %).  64 x 64: never, a wave
// a slice has nothing to overlap (1 chain 2.37 and 2.61 us, 4.08 and 4.69 for 4).
constexpr int split_limit(int DK, int DV) {
    return DK == 256 ? 8192 : DK == 64 ? 0 : DK * DV == 128 * 64 ? 1024 : 1536;
}

// A state of this width, as slices or whole.  (Slices are written through only where their sizes reach that line: 256 rows.)
template <int DK, int DV, bool BF16, bool THROUGH>
hipError_t launch_t(const void* q, const void* k, const void* v, void* o, float* kv, const float* decay, int chains, int H,
                    int steps, hipStream_t stream) {
    constexpr int PER = DV / kSliceCols, MOST = split_limit(DK, DV) / PER;      // slices of a chain, chains that are split
    if constexpr (MOST > 0 && (!THROUGH || 4LL * MOST * DK * DV >= through_bytes(DK))) {
        if (chains <= MOST) {
            hipLaunchKernelGGL((decode_slice_kernel<DK, DV, BF16, THROUGH>), dim3((unsigned)(chains * PER)), dim3(DK), 0, stream,
                               q, k, v, o, kv, decay, H, steps);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((decode_kernel<DK, DV, BF16, THROUGH>), dim3((unsigned)chains), dim3(threads_for(DK, DV)), 0, stream,
                       q, k, v, o, kv, decay, H, steps);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(const void* q, const void* k, const void* v, void* o, float* kv,
                         const float* decay, int chains, int H, int steps, int DK, int DV, int is_bf16,
                         hipStream_t stream) {
    if (chains <= 0 || steps <= 0) return hipSuccess;
    const bool through = write_through(chains, DK, DV);
    auto launch = [&](auto kernel) { return kernel(q, k, v, o, kv, decay, chains, H, steps, stream); };
#define LTN_DECODE(dk, dv)                                                                              \
    if (DK == dk && DV == dv) {                                                                         \
        if (is_bf16) return through ? launch(launch_t<dk, dv, true, true>) : launch(launch_t<dk, dv, true, false>);    \
        return through ? launch(launch_t<dk, dv, false, true>) : launch(launch_t<dk, dv, false, false>);               \
    }
    LTN_DECODE(128, 128) LTN_DECODE(64, 64) LTN_DECODE(96, 96) LTN_DECODE(256, 256) LTN_DECODE(256, 128) LTN_DECODE(128, 64)
#undef LTN_DECODE
    return hipErrorInvalidValue;
}

}  // namespace ltn
