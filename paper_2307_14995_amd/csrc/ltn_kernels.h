// Internal launcher interface between the C-ABI layer and the gfx950 kernels.
// Not installed; the public boundary is include/ltn_attn.h.
#pragma once
#include <hip/hip_runtime.h>

namespace ltn {

// One "decayed linear-attention pass":
//   out[t,:] = sum_{s<=t} lambda^(t-s) (a_t . b_s) c_s  (+ lambda^(t+1) a_t state_in)
// evaluated blockwise with a running state  S <- lambda^len S + (decayed b)^T c.
// With rev = 1 the token axis is traversed from the last token to the first, which
// turns the sum into  sum_{s>=t} lambda^(s-t) (a_t . b_s) c_s  (the anti-causal pass
// the gradients dK and dV need).  The forward pass and the three gradients of
// Lightning Attention (arXiv 2307.14995, Sec. 3.2.1 / App. B) are four such passes:
//   O  = pass(Q,  K,  V)        dQ = pass(dO, V,  K)
//   dV = pass(K,  Q,  dO, rev)  dK = pass(V,  dO, Q, rev)
struct PassArgs {
    const void* a;        // [chains, N, D]  "query-like" operand
    const void* b;        // [chains, N, D]  "key-like" operand
    const void* c;        // [chains, N, D]  "value-like" operand
    void* out;            // [chains, N, D]
    const float* state_in;  // [chains, D, D] fp32 or nullptr (zero)
    float* state_out;       // [chains, D, D] fp32 or nullptr
    int rev;              // 0: first token -> last; 1: last -> first
    // Gated, normalised epilogue (arXiv 2307.14995 Eq. 3 with the SimpleRMSNorm of
    // Sec. 3.1.3 per head): when gate != nullptr the pass also writes
    //   gated_out[t,:] = out[t,:] / sqrt(mean(out[t,:]^2) + eps) (.) gate[t,:]
    // and `out` itself may be nullptr.  Needs full-width slices (dv = D), one pass.
    const void* gate;     // [chains, N, D] or nullptr
    void* gated_out;      // [chains, N, D]
    float eps;
    // fp32 kernel, sequence-parallel form: [chains, N, DC] buffer (the output) in the first D
    // rows of whose segments the segments' states live between the launches; nullptr otherwise
    float* seg_rows;
};

// Cache hints of a bf16 launch; results do not depend on them.  kOnce*: an operand's tiles are loaded
// non-temporally, so that they leave the caches first.  kPast: outputs are stored past the caches, which then
// keep what will be read again.
enum { kOnceA = 1, kOnceB = 2, kOnceC = 4, kPast = 8 };
constexpr int kOnce = kOnceA | kOnceB | kOnceC;

struct PassBatch {
    PassArgs p[3];
    int count;            // 1..3 passes run concurrently in one launch
    const float* decay;   // [H]
    int chains;           // Bt * H
    int H;
    long long N;
    // Sequence-parallel form: every chain is cut into `segs` segments of seg_len tokens
    // (a multiple of 64; the last may be shorter) along the pass's own token order, each
    // handled by its own workgroups.  state_in / state_out then hold one state per
    // (chain, segment): [chains * segs, D, D].  segs = 1: the whole chain, seg_len unused.
    int segs;
    long long seg_len;
    int state_only;       // 1: compute only each segment's end state from a zero state
    int need_last;        // state_only: also for the last segment of a chain
    // count == 3 only: passes 0 and 1 read the same token rows at the same time (same direction,
    // two shared operands) and pass 2 does not; lets the bf16 kernel order workgroup ids for that
    int pairs_first;
    // Passes in more workgroups than compute units (launch_pass_cut_bf16): the last pass of chains
    // 0 .. cut_chains - 1 runs as two workgroups per slice, tokens [0, cut_len) and the rest, the second
    // starting from the state the first leaves.  cut_ids: workgroup ids where the whole passes but the
    // last, the whole last passes and the second parts begin.  Read by the cut kernels only.
    int cut_chains;
    int cut_ids[3];
    long long cut_len;
    int hints;            // those of the kernels that have them (launch_pass_bf16, launch_pass_cut_bf16)
};

// What the workgroup that goes by id `id` of a cut launch does.  part: 0 a whole pass, 1 the first and 2 the
// second part of the last pass of a cut chain; split: column slice, of NS.  Ids [0, cut_ids[0]) are first parts,
// from cut_ids[2] (a multiple of 8) on second parts, in the same order.  The workgroups of either go by an id
// that they draw when they start (cut_id): the next one of those congruent mod 8 to their own (one XCD's), first
// parts first.  So whoever gets a second part knows that its first part has started, whatever the order in which
// the GPU starts workgroups.
struct CutRole { int part, pass, chain, split; };

// fills in cut_ids; returns the workgroups of the launch
inline long long cut_launch_ids(PassBatch& pb, int NS) {
    const long long cut = (long long)pb.cut_chains * NS, others = (long long)pb.chains * (pb.count - 1) * NS,
                    whole = (long long)(pb.chains - pb.cut_chains) * NS;
    const long long second = (cut + others + whole + 7) / 8 * 8;       // congruent mod 8 to the first parts
    pb.cut_ids[0] = (int)cut;
    pb.cut_ids[1] = (int)(cut + others);
    pb.cut_ids[2] = (int)second;
    return second + cut;
}

__host__ __device__ inline bool cut_draws(const PassBatch& pb, int wg) {
    return wg < pb.cut_ids[0] || wg >= pb.cut_ids[2];
}
// first parts (and second parts) of the ids congruent to c mod 8
__host__ __device__ inline int cut_parts_of(const PassBatch& pb, int c) { return (pb.cut_ids[0] - c + 7) / 8; }
// chain and slice of part w; xcd: chains are dealt to XCDs (their number and cut_chains are multiples of 8)
template <int NS>
__host__ __device__ inline void cut_part(int w, int xcd, int& chain, int& split) {
    const int slot = xcd ? w >> 3 : w, q = slot / NS;
    chain = xcd ? q * 8 + (w & 7) : q;
    split = slot - q * NS;
}
// the part that the last workgroup of the ids congruent to c mod 8 to draw gets (if they have parts)
__host__ __device__ inline int cut_last_part(const PassBatch& pb, int c) { return c + 8 * (cut_parts_of(pb, c) - 1); }

// number: how many of those that draw with ids congruent to wg mod 8 drew before it
__host__ __device__ inline int cut_id(const PassBatch& pb, int wg, int number) {
    const int c = wg & 7, n = cut_parts_of(pb, c);
    return c + 8 * number + (number < n ? 0 : pb.cut_ids[2] - 8 * n);
}

// chain >= pb.chains: a padding workgroup
template <int NS>
__host__ __device__ inline CutRole cut_role(const PassBatch& pb, int xcd, int id) {
    const int last = pb.count - 1;
    const bool others = id >= pb.cut_ids[0] && id < pb.cut_ids[1];     // (count - 1 is 1 or 2 then: no divisions)
    CutRole r;
    r.part = id < pb.cut_ids[0] ? 1 : (id >= pb.cut_ids[2] ? 2 : 0);
    const int w = id - (r.part == 1 ? 0 : (others ? pb.cut_ids[0] : (r.part == 2 ? pb.cut_ids[2] : pb.cut_ids[1])));
    const unsigned slot = xcd ? (unsigned)w >> 3 : (unsigned)w;
    const unsigned q = others ? (last == 1 ? slot / NS : slot / (2 * NS)) : slot / NS;
    const int within = (int)(slot - q * (others ? (unsigned)(last * NS) : NS));
    r.chain = (int)(xcd ? q * 8 + (w & 7) : q) + (r.part == 0 && !others ? pb.cut_chains : 0);
    r.pass = others ? within / NS : last;
    r.split = others ? within % NS : within;
    return r;
}

// bf16 MFMA kernel, block length 64.  D in {64,96,128,256}; dv = value columns per workgroup
// (D, D/2 or, for D = 128, D/4; 64 or 32 for D = 256 and 32 for D = 96, plain pass only).
// DC (0: = D): features per token of c and out when they differ from those of a and b
// (the LRPE-d expansion of Eq. 1 doubles the query/key width): a, b [chains, N, D];
// c, out [chains, N, DC]; states [chains, D, DC]; dv slices DC.  Plain pass, or the state-only
// sweep with dv = 64 (128 for (128,256)).  (D, DC) in {(256,128), (128,256), (128,64), (64,128)}.
hipError_t launch_pass_bf16(const PassBatch& pb, int D, int dv, hipStream_t stream, int DC = 0);
// The same for plain and gated passes at their widest slices (DC columns up to 128; 64 where D = 256 or
// DC = 2 D = 128) with cut_chains and cut_len set and cut_ids to be filled in: two launches, as the flags that the
// second parts wait for and the counters are cleared first.  cut_len is a multiple of 64, at least cut_state_rows(D) tokens less than N.
inline long long cut_state_rows(int D) { return 2 * D + 64; }
hipError_t launch_pass_cut_bf16(PassBatch& pb, int D, hipStream_t stream, int DC = 0);
// Forward by the quadratic tiling of App. B Algorithm 3 (comparison kernel), bf16, zero
// initial state, D in {64,128}.
hipError_t launch_tiled_fwd_bf16(const void* q, const void* k, const void* v, void* o, const float* decay,
                                 int chains, int H, long long N, int D, hipStream_t stream);
// Gradients by the tiling of App. B Algorithm 4 (comparison kernel), bf16, D in {64,128}: one
// workgroup per key/value block (dK, dV) and one per query block (dQ), in one launch.
hipError_t launch_tiled_bwd_bf16(const void* q, const void* k, const void* v, const void* d_o, void* dq, void* dk,
                                 void* dv, const float* decay, int chains, int H, long long N, int D,
                                 hipStream_t stream);
// fp32 MFMA kernel.  D in {64,96,128,256}, block in {16,32,64}, D*block <= 4096 (96 counts as 128),
// the (dv, block) combinations f32_has_slice() accepts; gated: dv = D in {64,128}.  (D, DC) as for bf16.
bool f32_has_slice(int D, int DC, int dv, int block);
hipError_t launch_pass_f32(const PassBatch& pb, int D, int dv, int block, hipStream_t stream, int DC = 0);
// The scan below for fp32 passes, whose segment states live in PassArgs::seg_rows.
hipError_t launch_segment_scan_rows(const PassBatch& pb, const float* kv_in, float* kv_out, int D, hipStream_t stream,
                                    int DC = 0);
// Turns the segment-local end states L[pass][chain][g] in `states` (as written by a
// state_only launch) into the states at each segment's start, in place:
//   S[0] = kv_in (pass 0 only) or 0,   S[g+1] = lambda^len(g) S[g] + L[g],
// and writes the state after the last segment to kv_out (pass 0) when given.
hipError_t launch_segment_scan(float* states, const float* kv_in, float* kv_out, const float* decay,
                               int count, int chains, int H, int segs, long long seg_len, long long N,
                               int D, hipStream_t stream, int DC = 0 /* 0: = D; states are [D x DC] */);
// The same for the three passes of a backward of D features, of which dV's and dQ's (p[0], p[2]) have been swept; dK's
// states (p[1]) are dV's transposed.  A chain's states of pass i begin at p[i] + chain * chain_stride, segment after
// segment, or, with `rows`, in the first D rows of the segments of a [N, D] buffer (as in PassArgs::seg_rows).
struct ScanStates { float* p[3]; size_t chain_stride; int rev[3]; int rows; };
hipError_t launch_segment_scan_pair(const ScanStates& s, const float* decay, int chains, int H, int segs, long long seg_len,
                                    long long N, int D, hipStream_t stream);
// kv[c] (or zeros if null) -> kv_out[c], n floats.
hipError_t launch_state_copy(const float* kv_in, float* kv_out, size_t n, hipStream_t stream);
// `steps` consecutive decode steps per chain (q, k: [chains, steps, DK]; v, o: [chains,
// steps, DV]; kv: [chains, DK, DV]), see ltn_attn_decode_steps.  (DK, DV) in {(64,64), (96,96),
// (128,128), (256,256), (128,64), (256,128)}.
hipError_t launch_decode(const void* q, const void* k, const void* v, void* o, float* kv,
                         const float* decay, int chains, int H, int steps, int DK, int DV, int is_bf16,
                         hipStream_t stream);

// Input side of the token mixer for queries and keys (see ltn_prologue.hip): swish (Eq. 2)
// and the LRPE-d expansion of Eq. 1.  is_bwd = 0: y from x.  is_bwd = 1: dx from (x, dy)
// and, with theta and dtheta given, dtheta[H, D] through `partials` (device scratch of
// prologue_partial_count(N) * H * D doubles).
long long prologue_partial_count(long long N);
hipError_t launch_prologue(const void* x, const float* theta, const void* dy, void* out, float* dtheta,
                           double* partials, int act, int Bt, int H, long long N, int D, long long pos0,
                           int is_bf16, int is_bwd, hipStream_t stream);

// Gated SimpleRMSNorm on `rows` rows of D features (see ltn_gate.hip).  is_bwd = 0:
// o0 = y (dy, o1 unused); is_bwd = 1: o0 = dx, o1 = du.
hipError_t launch_gate(const void* x, const void* u, const void* dy, void* o0, void* o1, float eps,
                       long long rows, int D, int is_bf16, int is_bwd, hipStream_t stream);

// Streaming-read probe (see ltn_probe.hip): wgs workgroups each read their own per_wg bytes
// (a multiple of 64 KB) of `buf` `iters` times, to LDS directly or to registers.
hipError_t launch_probe_stream(const void* buf, size_t per_wg, int wgs, int iters, int to_registers, unsigned* sink,
                               hipStream_t stream);

// lambda^n, n >= 0, by binary powering in fp64 (only multiplications: exact up to
// rounding, lambda = 0 gives 0^0 = 1, no transcendental).  Never called with n < 0.
__device__ __forceinline__ float decay_pow(float lam, int n) {
    double base = (double)lam, r = 1.0;
    while (n > 0) {
        if (n & 1) r *= base;
        base *= base;
        n >>= 1;
    }
    return (float)r;
}

// Workgroup index -> (pass, chain, split).  Consecutive workgroup ids are dealt
// round-robin to the 8 XCDs, each with a private L2; all workgroups that read the
// same chain's tokens (its passes and value-column splits) are therefore given
// ids that are congruent mod 8, so re-reads of a chain's tiles hit one L2.
__device__ __forceinline__ void map_workgroup(int wg, int per_chain, int chains,
                                              int& chain, int& within) {
    if ((chains & 7) == 0) {
        const int xcd = wg & 7, slot = wg >> 3;
        chain = (slot / per_chain) * 8 + xcd;
        within = slot % per_chain;
    } else {
        chain = wg / per_chain;
        within = wg % per_chain;
    }
}

// The same dealing for a number of chains that is no multiple of 8: the launch is padded to
// 8 * ceil(chains / 8) chain slots and the workgroups of the empty ones leave at once.  That
// puts ceil(chains / 8) * per_chain workgroups on the first XCDs, so it is used only while
// those fit an XCD's 32 compute units (xcd_ids_fit); otherwise ids stay chain-major.
inline bool xcd_ids_fit(long long chains, int per_chain) {
    return per_chain > 1 && ((chains & 7) == 0 || (chains + 7) / 8 * per_chain <= 32);
}
inline long long launch_chain_slots(long long chains, int per_chain) {
    return xcd_ids_fit(chains, per_chain) ? (chains + 7) / 8 * 8 : chains;
}
// xcd_ids: xcd_ids_fit(chains, per_chain), computed by the host.  False: the workgroup is a
// padding one and has nothing to do.
__device__ __forceinline__ bool map_workgroup_padded(int wg, int per_chain, int chains, int xcd_ids,
                                                     int& chain, int& within) {
    if (xcd_ids) {
        const int xcd = wg & 7, slot = wg >> 3;
        chain = (slot / per_chain) * 8 + xcd;
        within = slot % per_chain;
    } else {
        chain = wg / per_chain;
        within = wg % per_chain;
    }
    return chain < chains;
}

}  // namespace ltn
