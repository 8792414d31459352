// C-ABI layer of the Lightning Attention library: argument validation (host only,
// before any launch), choice of block length and value-column split, and dispatch
// to the gfx950 kernels.  See include/ltn_attn.h for the contract.
#include "../../include/ltn_attn.h"
#include "ltn_kernels.h"

#include <atomic>
#include <cstdint>
#include <mutex>

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Test-only overrides of the launch plan (ltn_attn_set_debug_plan); 0 = the library's choice.
std::atomic<int> g_debug_dv{0};
std::atomic<int> g_debug_segs{0};

// A tensor argument as a byte range.  Outputs are written while inputs are still being
// read (tile loads run up to three blocks ahead of the stores), so any overlap between an
// output and an input, or between two outputs, is rejected, not only equal base pointers.
struct Span { const void* p; size_t bytes; };

bool spans_overlap(const Span& a, const Span& b) {
    if (!a.p || !b.p || a.bytes == 0 || b.bytes == 0) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a.p), b0 = reinterpret_cast<uintptr_t>(b.p);
    return a0 < b0 + b.bytes && b0 < a0 + a.bytes;
}

// true when some output overlaps an input or another output
bool outputs_alias(const Span* outs, int n_out, const Span* ins, int n_in) {
    for (int a = 0; a < n_out; ++a) {
        for (int b = 0; b < n_in; ++b)
            if (spans_overlap(outs[a], ins[b])) return true;
        for (int b = a + 1; b < n_out; ++b)
            if (spans_overlap(outs[a], outs[b])) return true;
    }
    return false;
}

size_t esize_of(ltn_dtype dtype) { return dtype == LTN_BF16 ? 2 : 4; }

// Value columns handled per workgroup.  Every value-column slice of a chain recomputes
// that chain's score tiles and re-reads its first two operands through L2, and a compute
// unit holds one workgroup: the split is the deepest one whose workgroups still fit one
// round of the 256 compute units; when even full-width slices need more than one round,
// full width (fewest re-reads).  Among the splits that fit one round, bf16 takes the deepest
// whose workgroups of one chain can be given ids on one XCD (count passes x slices per chain,
// ltn::xcd_ids_fit): slices that meet in one L2 beat a deeper split that does not (20 chains,
// backward: 32-column slices 0.101 ms, 64-column 0.066 ms; 42 chains: 64-column 0.120 ms,
// full width 0.110 ms).  Measured on MI355X for 8..256 chains, forward and backward.
// ltn_attn_set_debug_plan (test only) overrides the choice.
// chain_passes = chains (x segments) x count; count = passes per chain in the launch.
int pick_dv(long long chain_passes, int D, int count = 1) {
    if (D == 96) {                         // three 32-column slices, or all 96 columns in one workgroup
        if (const int v = g_debug_dv.load(std::memory_order_relaxed)) {
            if (v == 32 || v == 96) return v;
        }
        // three slices per pass while a chain's workgroups can share an XCD within one round
        return (chain_passes * 3 <= 256 && ltn::xcd_ids_fit(chain_passes / count, count * 3)) ? 32 : 96;
    }
    // D = 256: the state copies of more than 64 columns do not fit the LDS
    const int lo = 32, hi = (D == 256) ? 64 : D;
    if (const int v = g_debug_dv.load(std::memory_order_relaxed)) {
        if ((v == D || v == D / 2 || v == D / 4 || v == D / 8) && v >= lo && v <= hi) return v;
    }
    int fits = 0;
    for (int dv = lo; dv <= hi; dv *= 2) {
        if (chain_passes * (D / dv) > 256) continue;
        if (count * (D / dv) == 1 || ltn::xcd_ids_fit(chain_passes / count, count * (D / dv))) return dv;
        if (!fits) fits = dv;
    }
    return fits ? fits : hi;               // more than one round even at full width: fewest re-reads
}

// The same rule for a pass whose value side has DC columns and whose kernels exist for
// slices of lo .. hi columns (powers of two).
int pick_dv_range(long long chain_passes, int DC, int lo, int hi) {
    for (int dv = lo; dv <= hi; dv *= 2)
        if (chain_passes * (DC / dv) <= 256) return dv;
    return hi;
}

// Launch plan of the fp32 kernel: value columns per workgroup and segments per chain, the pair
// with the least estimated time.  The kernel is bound by the fp32 matrix rate, so the estimate
// counts the MFMAs a SIMD issues per block (its slots), times blocks, times rounds of 256 units:
// a slice of dv columns costs its share of the state products plus the whole score tiles (a
// narrower slice repeats those); a cut into segments adds the state-only sweep at full width
// and two more launches.  kF32Launch and kF32Block are a launch and the latencies of a block in
// units of one MFMA (32 cycles), fitted to forced plans (128 features, 64 chains x 2048 tokens:
// 32 / 64 / 128 columns 1.9 / 3.0 / 5.0 us a block; the choice was the fastest plan, or within 8 %
// of it, at 30 shapes of 2 .. 256 chains x 100 .. 2048 tokens, 64 .. 256 features).  The gated pass adds
// its epilogue, kF32Gate a block per 64 columns (6.6 us a block of 128), and, as it has only one width
// and so is cut where plain passes take narrower slices, kF32State per element of the segments' states
// (96 chains x 512 tokens, 64 features, cut 8 ways: 44 us, 32 in two steps; in the plain passes'
// estimate that term chose worse: 64 x 700 forward 29 -> 33 us).
struct F32Plan { int dv, segs; long long seg_len; double t; };
constexpr double kF32Launch = 250.0, kF32Block = 30.0, kF32Gate = 40.0, kF32State = 2e-4;

F32Plan pick_f32(long long chains, int count, long long N, int D, int DC, int blk, bool gated) {
    if (blk > 32) blk = 32;
    const int forced_dv = g_debug_dv.load(std::memory_order_relaxed), forced_segs = g_debug_segs.load(std::memory_order_relaxed);
    const int ts = blk / 16;
    const double scores = ts * (ts + 1) / 2 * (D / 4) / 4.0;                 // per SIMD, whatever the slice
    auto slice_cost = [&](int dv) {
        const double c = scores + dv / 16 / 4.0 * (2.0 * ts * (D / 4) + 2.0 * ts * (ts + 1)) + kF32Block +
                         (gated ? kF32Gate * dv / 64 : 0.0);
        return D == 96 && dv == 32 ? c + 40.0 : c;                           // four waves, one per SIMD: latencies exposed
    };
    const int full = DC == 256 ? 128 : DC;                                   // columns of a sweep's workgroup
    const double sweep_cost = full / 16 / 4.0 * ts * (D / 4) + kF32Block;
    F32Plan best = {0, 1, 0, 0.0}, paired = best;
    // `sweeps` passes of a piece are swept; `states`: with the bytes of the segments' states
    auto estimate = [&](int dv, int segs, long long len, int sweeps, bool states) {
        const long long pieces = chains * segs, wgs = pieces * count * (DC / dv), blocks = ((segs > 1 ? len : N) + blk - 1) / blk;
        double t = (double)((wgs + 255) / 256) * blocks * slice_cost(dv);
        if (segs > 1) t += (double)((pieces * sweeps * (DC / full) + 255) / 256) * blocks * sweep_cost + 2 * kF32Launch;
        if (segs > 1 && states) t += kF32State * D * DC * pieces * count;
        return t;
    };
    auto consider = [&](int dv, int segs, long long len) {
        const double t = estimate(dv, segs, len, count, gated), t2 = estimate(dv, segs, len, count - 1, gated);
        if (!best.dv || t < best.t) best = F32Plan{dv, segs, len, t};
        if (!paired.dv || t2 < paired.t) paired = F32Plan{dv, segs, len, t2};
    };
    int dvs[5], n_dv = 0;
    if (gated) dvs[n_dv++] = DC;
    else {
        for (const int dv : {128, 96, 64, 32})
            if (ltn::f32_has_slice(D, DC, dv, blk)) {
                if (dv == forced_dv) {
                    n_dv = 0;
                    dvs[n_dv++] = dv;
                    break;
                }
                dvs[n_dv++] = dv;
            }
    }
    // the sweep exists for the library's own block length of each shape
    const bool can_cut = forced_segs != 1 && N >= 2 * D && blk == (D == 256 || DC == 256 ? 16 : 32);
    for (int i = 0; i < n_dv; ++i) {
        if (!(forced_segs > 1 && can_cut)) consider(dvs[i], 1, 0);
        if (!can_cut) continue;
        const long long at_least = N / 256 > D ? 256 : D;
        for (long long want = 2; want <= 64 && N / want >= at_least; want += want < 8 ? 1 : want / 4) {
            long long w = forced_segs > 1 ? forced_segs : want;
            // every segment holds a whole state in its rows: at least D tokens, the last one too
            for (; w > 1; --w) {
                const long long len = ((N + w - 1) / w + 63) / 64 * 64, segs = (N + len - 1) / len;
                if (segs > 1 && len >= D && N - (segs - 1) * len >= D) {
                    if (chains * count * segs * (DC / full) <= 1024 || forced_segs > 1) consider(dvs[i], (int)segs, len);
                    break;
                }
            }
            if (forced_segs > 1) break;
        }
        if (forced_segs > 1 && !best.dv) consider(dvs[i], 1, 0);
    }
    // A backward sweeps two passes of three (swept_passes), which makes more and shorter cuts look worth it than are: the
    // segments' states, 64 KiB a piece, are no part of that estimate.  So the plan it leads to is taken only where
    // it is ahead of the other by 1 % with them counted.  At the 154 ends of the ranges of 1 .. 129 chains x 640 .. 16384
    // tokens where the two differ the choice is at most 1.1 % slower than the plan for three sweeps and up to 8 faster (us:
    // 24 x 8192 593 and 552, 52 x 16384 2611 and 2410); the other plan, always taken, lost up to 18 (16 x 1024 67 and 75, 32 x
    // 1024 102 and 120, 56 x 1500 240 and 269, 64 x 4096 654 and 693).  Other widths keep the plan for three
    // (20 x 2048 x 64 56 and 64, 12 x 1999 x 96 78 and 82, 16 x 2048 x 256 332 and 354).
    if (count == 3 && D == 128 && (paired.dv != best.dv || paired.segs != best.segs) &&
        estimate(paired.dv, paired.segs, paired.seg_len, 2, true) < 0.99 * estimate(best.dv, best.segs, best.seg_len, 2, true))
        return paired;
    return best;
}

// The passes of `pb` that a state-only sweep is run for: all, or of a backward's three dV's and dQ's, since dK's
// states are dV's transposed (launch_segment_scan_pair).  In fp32, where a sweep is bound by its products (us a backward,
// three sweeps and two: 32 chains x 2048 tokens of 128 features 222 and 198, 32 x 2000 of 64 84.8 and 77.3, 16 x 2048 of 96
// 92.4 and 84.5), and for 256 features in bf16 (4 x 8192 121 and 116).  The other bf16 sweeps of dV and dK share their loads, and
// take no longer for being two (4 x 32768 of 128 106.0 and 106.9, 2 x 4000 22.4 and 23.2, 4 x 8192 of 96 42.6 and 44.0).
int backward_sweeps(long long chains, int segs, int D, ltn_dtype dtype) {
    if (segs <= 1) return 0;
    if (dtype == LTN_BF16) return D == 256 ? 2 : 3;
    // (a third sweep that its units would be idle for costs nothing: 2 chains x 1952 x 64 28.1 with three, 29.0)
    const long long swept = chains * segs * (D == 256 ? 2 : 1);
    return (3 * swept + 255) / 256 > (2 * swept + 255) / 256 ? 2 : 3;
}

int swept_passes(const ltn::PassBatch& pb, int segs, int D, ltn_dtype dtype, int (&pass)[3]) {
    const bool pair = pb.count == 3 && pb.pairs_first && backward_sweeps(pb.chains, segs, D, dtype) == 2;
    for (int i = 0; i < 3; ++i) pass[i] = pair ? 2 * i : i;
    return pair ? 2 : pb.count;
}

// One launch of fp32 passes of one shape, cut into segments (state-only sweep, scan, per-segment
// pass) when the plan says so; the segments' states live in the output's rows.
ltn_status run_f32(ltn::PassBatch& pb, int D, int DC, int blk, hipStream_t stream, bool gated = false) {
    if (blk > 32) blk = 32;               // a block of 64 tokens is two tiles of 32 on chip
    const F32Plan plan = pick_f32(pb.chains, pb.count, pb.N, D, DC, blk, gated);
    if (!plan.dv) return LTN_ERR_UNSUPPORTED;
    pb.segs = plan.segs;
    pb.seg_len = plan.seg_len;
    if (plan.segs > 1) {
        float* const kv_out = pb.p[0].state_out;
        for (int i = 0; i < pb.count; ++i) pb.p[i].seg_rows = static_cast<float*>(pb.p[i].out ? pb.p[i].out : pb.p[i].gated_out);
        ltn::PassBatch sweep = pb;
        sweep.state_only = 1;
        sweep.need_last = kv_out != nullptr;
        int pass[3];
        sweep.count = swept_passes(pb, pb.segs, D, LTN_F32, pass);
        for (int i = 0; i < sweep.count; ++i) {
            sweep.p[i] = pb.p[pass[i]];
            sweep.p[i].gate = nullptr;
            sweep.p[i].state_in = nullptr;
        }
        if (ltn::launch_pass_f32(sweep, D, DC == 256 ? 128 : DC, blk, stream, DC) != hipSuccess) return LTN_ERR_LAUNCH;
        if (sweep.count != pb.count) {
            const ltn::ScanStates s = {{pb.p[0].seg_rows, pb.p[1].seg_rows, pb.p[2].seg_rows}, (size_t)pb.N * D,
                                       {pb.p[0].rev, pb.p[1].rev, pb.p[2].rev}, 1};
            if (ltn::launch_segment_scan_pair(s, pb.decay, pb.chains, pb.H, pb.segs, pb.seg_len, pb.N, D, stream) != hipSuccess)
                return LTN_ERR_LAUNCH;
        } else if (ltn::launch_segment_scan_rows(pb, pb.p[0].state_in, kv_out, D, stream, DC) != hipSuccess) {
            return LTN_ERR_LAUNCH;
        }
        pb.p[0].state_out = nullptr;
    }
    return ltn::launch_pass_f32(pb, D, plan.dv, blk, stream, DC) == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

ltn_status check_common(int Bt, int H, long long N, int D, int block, ltn_dtype dtype, int* blk_out) {
    if (Bt < 0 || H < 0 || N < 0 || D <= 0 || block < 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (D != 64 && D != 96 && D != 128 && D != 256) return LTN_ERR_UNSUPPORTED;
    const int blk = block ? block : ltn_attn_pick_block(D, dtype);
    if (dtype == LTN_BF16) {
        if (blk != 64) return LTN_ERR_UNSUPPORTED;
    } else {
        if (blk != 16 && blk != 32 && blk != 64) return LTN_ERR_UNSUPPORTED;
        if ((long long)(D == 96 ? 128 : D) * blk > 4096) return LTN_ERR_UNSUPPORTED;   // 96 takes the blocks of 128
    }
    if ((long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    *blk_out = blk;
    return LTN_OK;
}

// Sequence-parallel plan.  With few chains even the deepest value-column split leaves
// compute units idle and makes every workgroup re-read A and B; cutting each chain into
// segments instead gives full-width workgroups to all compute units at the price of one
// extra read of B and C (the state-only sweep) and two more launches.  Measured on MI355X
// (2 .. 64 chains, N = 2048 .. 65536, forward and backward, every segment count): pays when a
// chain can be cut at least 8 ways into segments of at least 512 tokens without exceeding one
// round of compute units, from 5 ways on when the segments are at least 1024 tokens long
// (33 .. 51 passes of long chains: the forward of 36 .. 48 chains at N = 8192 runs 17-29 % faster
// cut 5 .. 7 ways, the backward of 12 .. 16 chains 11-16 %), and 4 ways in the backward of about
// 20 chains with segments of at least 2048 tokens (13-19 %); shorter segments than these only where
// finer_pays() says so.
// bf16 kernels only.  Heads of 256 features always need four 64-column workgroups per chain
// and segment, heads of 96 three of 32; there the form pays from 3 segments of at least 512
// tokens on (measured: 2 .. 32 chains, N = 2048 .. 32768, forward and backward; heads of 96
// features have a second cut for their 96-column workgroups, in place), for the gated
// pass from 4 segments of at least 512 tokens on, and from 2 when they are at least 2048 tokens
// long (measured: 4 .. 100 chains, N = 2048 .. 16384, 64 / 96 / 128 features).
// ltn_attn_set_debug_plan (test only) forces a segment count.
struct SegPlan { int segs; long long seg_len; };
constexpr long long kMinSegsFullWidth = 4;   // measured: 2 segments lose to one workgroup per chain

SegPlan cut_chain(long long N, long long want) {
    SegPlan plan = {1, 0};
    if (want <= 1) return plan;
    long long len = (N + want - 1) / want;
    len = (len + 63) / 64 * 64;
    const long long segs = (N + len - 1) / len;
    if (segs <= 1 || segs > 0x7fff) return plan;
    plan.segs = (int)segs;
    plan.seg_len = len;
    return plan;
}

// Estimated time, in us, of a bf16 pass of DA query/key and DC value features under a plan, for
// sequences that the rules above cut fewer than 8 ways.  Whole chains: a start and `whole` a block of
// 64 tokens.  Cut: the sweep's and the scan's launches more, `block` per block of a segment (as cut_chain
// rounds it; sweep and pass), and per segment its state, written, scanned and read, at about
// 4.6 TB/s; and no less than `issue`, in which the binding issues three launches and allocates the
// scratch.  Fitted for the choice below to forced plans, 1 .. 64 chains x 520 .. 4095 tokens, every width.
struct BlockCost { double whole, block; };
constexpr double kIssue = 16.2, kIssueBwd = 19.1;
BlockCost block_cost(int DA, int DC, bool gated) {
    if (gated) return DA == 64 ? BlockCost{0.92, 1.17} : BlockCost{1.89, 1.81};
    if (DA == 64) return BlockCost{0.47, DC == 128 ? 0.63 : 0.74};
    if (DA == 96) return BlockCost{0.70, 0.95};
    if (DA == 128) return BlockCost{0.69, DC == 256 ? 1.53 : DC == 128 ? 1.7 : 1.43};
    return BlockCost{1.46, 2.23};
}
double plan_time(const SegPlan& plan, long long chain_passes, long long N, int DA, int DC, bool gated, double issue = kIssue) {
    constexpr double kStart = 4.2, kCut = 7.5, kStateElement = 3.5e-6;
    const BlockCost c = block_cost(DA, DC, gated);
    if (plan.segs == 1) return kStart + c.whole * ((N + 63) / 64);
    const double state = kStateElement * (DA == 96 ? 128 : DA) * (DC == 96 ? 128 : DC);
    const double t = kStart + kCut + c.block * (plan.seg_len / 64) + state * chain_passes * plan.segs;
    return t < issue ? issue : t;
}

// Shorter segments than those rules allow (`finer` of them, down to 256 tokens, about 160 in the gated
// pass): where they are estimated 1.5 % faster than the plan the rules give, cut or whole.  Over the
// 1880 forced shapes where a finer cut is possible this takes 0.854 of the rules' time on average, 0.3 %
// more than the better of each pair, and loses more than 3 % at 17 shapes.  Taking every finer cut
// from 5 segments on (4 of 1536 tokens for unequal widths) lost that at 190: 20-34 % at 64 chains x
// 1537 .. 2000 tokens of (128, 64), 6 % at 51 gated chains x 800, 11 % at backwards of 1 .. 4 chains x
// 1537 of 64 features.
bool finer_pays(long long finer, long long want, long long chain_passes, long long N, int DA, int DC, bool gated, double issue) {
    return plan_time(cut_chain(N, finer), chain_passes, N, DA, DC, gated, issue) <
           0.985 * plan_time(cut_chain(N, want), chain_passes, N, DA, DC, gated, issue);
}

// paired_chains: the number of chains when the passes are the three of a backward (whose
// (dV, dK) workgroups sit side by side on one XCD at full width), else 0.
SegPlan pick_segments(long long chain_passes, long long N, int D, ltn_dtype dtype, bool full_width = false,
                      long long paired_chains = 0) {
    SegPlan plan = {1, 0};
    if (dtype != LTN_BF16 || chain_passes <= 0 || N <= 64) return plan;
    // D = 256: every (chain, segment) still needs four 64-column workgroups; D = 96: three of 32
    const long long per_seg = (D == 256) ? 4 : ((D == 96 && !full_width) ? 3 : 1);
    long long want = 256 / (per_seg * chain_passes);
    bool whole_rows = per_seg == 1;        // one workgroup per chain, pass and segment
    const bool bwd = paired_chains > 0;
    long long finer = N / (full_width ? 160 : 256) < want ? N / (full_width ? 160 : 256) : want;
    if (D == 96 && !full_width)               // an XCD's share of three-slice segments, as below
        while (finer > 1 && (chain_passes * finer + 7) / 8 * 3 > 32) --finer;
    // a pass that must keep full-width slices has no column split to fall back on
    if (want > N / 512) want = N / 512;       // segments of at least 512 tokens
    // finer cuts: from 5 segments on (6 and 7 where a whole chain splits its columns four ways), not for
    // the gated pass of 96 features (three workgroups per segment in its sweep)
    const long long least = full_width || per_seg > 1 ? 5 : (D == 128 && !bwd ? 7 : 6);
    const bool try_finer = want < 8 && finer > want && finer >= least && !(D == 96 && full_width);
    if (full_width) {
        // from 4 ways on; 2 or 3 ways when the segments stay at least 2048 tokens long (not for 96
        // features, whose state-only sweep runs three workgroups per segment; for 128 features
        // only when that leaves an eighth of the compute units free: at 128 chains the second
        // read of K and V costs more than the idle half of the chip)
        const bool few_ok = D != 96 && want >= 2 && N / want >= 2048 && (D == 64 || chain_passes * want <= 224);
        if (want < kMinSegsFullWidth && !few_ok) want = 1;
    } else if (per_seg > 1) {
        if (want < 3) want = 1;
        if (D == 96) {
            // Workgroup ids deal (chain, segment) pairs to the 8 XCDs of 32 compute units and keep
            // a pair's three slices on one XCD: an XCD's share must not exceed its units (11
            // pairs per XCD -- 252 workgroups -- ran 30 % slower than 10).
            while (want > 1 && (chain_passes * want + 7) / 8 * 3 > 32) --want;
            if (want < 3) want = 1;
            // Heads of 96 features also have one 96-column workgroup per chain and segment
            // (pick_dv takes it when three 32-column slices each would need more than one round).
            // From 12 chain passes on, cutting for that width pays from 8 segments on -- of at
            // least 768 tokens, or 512 where the rule above finds nothing to cut -- and from 5
            // segments of at least 1024 tokens (measured: 4 .. 32 chains, N = 4096 .. 32768,
            // forward and backward, every segment count).
            if (chain_passes >= 12) {
                long long all = 256 / chain_passes;
                if (all > N / 512) all = N / 512;
                if (all >= 5) {
                    const long long len = N / all;
                    if ((all >= 8 && (len >= 768 || want == 1)) || len >= 1024) {
                        want = all;
                        whole_rows = true;
                    }
                }
            }
        }
    } else if (want < 8) {
        // 5 .. 7 ways: segments of at least 1024 tokens; 4 ways: the backward alone, segments of at
        // least 2048 tokens, when its (dV, dK) pairs can sit side by side (chains x 4 a multiple of 8)
        // (heads of 64 features, whose blocks cost half as much: 512 and 1024 tokens)
        const long long few_len = D == 64 ? 512 : 1024;
        const bool few = want >= 5 && N / want >= few_len;
        const bool four = want == 4 && paired_chains > 0 && (paired_chains * 4) % 8 == 0 && N / want >= 2 * few_len;
        if (!few && !four) want = 1;
    }
    if (try_finer && !(D == 96 && whole_rows) && finer_pays(finer, want, chain_passes, N, D, D, full_width, bwd ? kIssueBwd : kIssue))
        want = finer;
    if (paired_chains > 0 && want >= 6 && whole_rows) {
        // The backward's workgroup ids pair a chain's (dV, dK) passes on one XCD only when
        // chains x segments is a multiple of 8: up to a quarter fewer segments for that
        // (measured, 4 / 5 / 6 / 12 chains: 21 -> 20, 17 -> 16, 14 -> 12, 7 -> 6 segments run
        // 9-15 % faster).
        for (long long w = want; w >= 2 && 4 * w >= 3 * want; --w) {
            const SegPlan p = cut_chain(N, w);
            if (p.segs > 1 && (paired_chains * p.segs) % 8 == 0) {
                want = w;
                break;
            }
        }
    }
    if (const int v = g_debug_segs.load(std::memory_order_relaxed)) want = v;
    return cut_chain(N, want);
}

// How the gated forward runs: fused, or as the plain forward followed by the gate kernel on its
// stored output (store_o: the caller wants that output).  256 features (and 96 in fp32): no kernel
// holds a complete output row of these widths in one workgroup.
//
// The fused epilogue needs complete output rows in one workgroup, i.e. full-width slices
// (one workgroup per chain, or per chain segment).  With few chains that can leave
// compute units idle; when the caller wants the attention output stored anyway
// (training), the plain forward at its usual split followed by the gate kernel on the
// stored output is then the faster way to the same result (bf16, measured on MI355X: below
// about 192 chains).  fp32 loses nothing by storing o, so there y's own memory can hold it on
// the way, and two steps are taken, whether o is wanted or not, where they are estimated 3 % faster
// (the gate kernel's three tensors at about 5 TB/s, two launches no faster than they are issued).
// Measured fused and in two steps, 128 features: 8 chains x 300 tokens 59 and 26 us, 96 x 512 82
// and 65, 128 x 1000 155 and 135, but 32 x 2048 86 and 96.
// (64 features: a full-width workgroup is a quarter of the work, and the fused form is the faster
// one where it is at most 512 tokens long, where the second launch counts -- 15.5 us in two steps,
// 13 fused -- or cut into 3 or more segments and estimated faster: 32 x 2048 tokens 26.5 and
// 21.5, 64 x 8192 123 and 104, but 8 x 800 14.6 and 17.5; uncut and longer the split pays
// again, 80 x 2048 36 and 48.  The gate kernel streams three tensors at 5 TB/s behind 3 us; two
// launches and the call's allocations take 14.6 us to issue.)
bool gated_in_two_steps(long long chains, long long N, int D, ltn_dtype dtype, int blk, bool store_o) {
    if (D == 256 || (D == 96 && dtype != LTN_BF16)) return true;
    if (dtype == LTN_F32) {
        // (whether o is wanted does not enter: y has the same bits with and without it)
        constexpr double kSlotsPerValue = 3 * 4 / 5e12 * 2.4e9 / 32, kIssueTwo = 700.0;
        double two = pick_f32(chains, 1, N, D, D, blk, false).t + kF32Launch + (double)chains * N * D * kSlotsPerValue;
        if (two < kIssueTwo) two = kIssueTwo;
        return two < 0.97 * pick_f32(chains, 1, N, D, D, blk, true).t;
    }
    if (!store_o || chains >= 192) return false;
    if (D != 64) return true;
    if (N <= 512) return false;
    const SegPlan fused = pick_segments(chains, N, D, dtype, true), plain = pick_segments(chains, N, D, dtype);
    double two_us = plan_time(plain, chains, N, D, D, false) + 3.0 + chains * N * D * (3 * 2 / 5e6);
    if (two_us < 14.6) two_us = 14.6;
    return fused.segs < 3 || plan_time(fused, chains, N, D, D, true) + 1.5 >= two_us;
}

// Passes in more workgroups than the 256 units hold at once: are those that would be alone in the last round to be
// cut in two (launch_pass_cut_bf16), at half a chain?  chains = 0: no.
// Up to four rounds: beyond, workgroups end so far apart that the last round fills up by itself (time cut over
// time whole 0.97 .. 1.10).  Up to half a round alone: with more, the second parts take more than the units that
// are left (1.01 .. 1.08).  Shorter than 12 blocks the launch that clears the flags takes what the cut gains.  And
// inputs of at least least_cut_mib: while they stay in the 256 MiB memory-side cache, workgroups that are alone in
// the last round find them there and run faster than those of a full round, so that half of a short last round is
// less than what two parts and the clearing cost.
// Measured at 17800 shapes of 20 .. 1024 chains x 700 .. 6000 tokens on two cards, every width, kernels alone and
// in training and mixer steps.  Time cut over time whole of those that are cut, mean: training and mixer steps of
// 64 / 96 / 128 / 256 features 0.96 / 0.96 / 0.96 / 0.93, forward 0.95 / 0.93 / 0.94 / 0.87, gated 0.94 / 0.93 /
// 0.93, with o 0.92; 0.8 % of them lose more than 1 %, none 6 %.
// Chains of 512 KiB (to within 1 KiB: 2048 tokens of 128 features, 4096 of 64, 2731 of 96): the distance from
// chain to chain costs the cut 3 .. 6 % (not the inputs' total size: 112 x 2340 and 120 x 2180 x 128 are 256 MiB
// as well and gain 7 and 5 %; which addresses collide has not been traced), so backwards of more than 7/16 of a
// round alone lose (training and mixer step 128 x 2048 x 128 1.03 and 1.04, 213 x 2048 1.02 and 1.03, 126 x 2048
// 0.98 and 1.02, 213 x 2731 x 96 1.03 and 1.01) where 8 KiB more or fewer a chain gain (128 x 2016 0.98 and 1.00,
// x 2080 0.985 and 0.99, x 1984 0.96 and 0.98, 213 x 1500 0.98 and 0.99); with less alone the cut gains there too
// (120 x 2048 0.95 and 0.97).
// widest: value columns of the widest slices that DC columns have here, the only ones that are cut.
struct Cut { int chains; long long len; };

// Inputs, each read once, from which on the cut pays, in MiB.  rounds: full ones (1 .. 3); alone: workgroups in
// the last one, of `units`; xcd: ids deal chains to XCDs (whole passes that share tokens then meet in one L2, and
// a cut gains less).
// Time cut over whole below and above each line:
//   forward: 64 features 1.00 .. 1.03 at 90 .. 120 MiB, 0.95 .. 0.99 at 120 .. 150; more than 7/16 alone 1.03 and
//     1.00
//   backward, three passes of full width, xcd: up to a quarter of a round alone 1.01 below 40 MiB, 0.97 .. 1.00
//     from there; 5/16 1.01 at 64 .. 90, 1.00 at 90 .. 150; 7/16 1.02 at 90 .. 120, 0.98 .. 0.99 at 150 .. 180;
//     8/16 1.02 at 120 .. 150, 0.99 at 150 .. 180; two and three full rounds 1.00 .. 1.03 below 150, 0.97 from 200
//   backward, not xcd: one full round 0.95 .. 1.00 from 45, two 0.97 .. 1.00 from 120, three 0.97 .. 1.00 from 180
//   dK and dQ of unequal widths, xcd: one full round 1.03 below 40 and 0.98 above (up to a quarter alone 0.99 there
//     too), two 1.01 at 90 .. 120 and 0.97 at 150 .. 180, three 0.99 .. 1.03; not xcd 0.92 .. 1.01 everywhere
// 256-feature and gated passes, whose blocks take longest, gain at every size (0.80 .. 1.00).
long long least_cut_mib(int count, int slices, bool gated, bool xcd, long long rounds, long long alone, long long units) {
    constexpr long long kNever = 1LL << 40;
    if (gated || (slices > 1 && count != 2)) return 0;
    if (count == 1) return 16 * alone <= 7 * units ? 120 : 150;
    const long long past_quarter = 16 * alone > 4 * units ? 16 * alone - 4 * units : 0;
    if (count == 2) {
        if (!xcd) return 0;
        return rounds == 1 ? (past_quarter ? 45 : 0) : (rounds == 2 ? 140 : kNever);
    }
    if (xcd) return rounds == 1 ? 45 + 32 * past_quarter / units : 175;
    return rounds == 1 ? 45 : (rounds == 2 ? 120 : 180);
}

Cut pick_cut(int chains, int count, long long N, int D, int DC, int dv, int widest, bool gated = false) {
    constexpr long long kRounds = 4, kHalf = 6, kKiB = 1024;
    const Cut none = {0, 0};
    if (dv != widest || g_debug_segs.load(std::memory_order_relaxed) == 1) return none;
    const int slices = DC / dv;
    const long long per_chain = (long long)count * slices;
    // one XCD's workgroups and units where ids deal chains to XCDs, else all of them
    const bool xcd = (chains & 7) == 0;
    const long long wgs = xcd ? chains / 8 * per_chain : chains * per_chain, units = xcd ? 32 : 256;
    const long long cut_chains = (wgs % units + slices - 1) / slices, alone = cut_chains * slices;
    if (wgs < units || wgs > kRounds * units || alone == 0 || alone > units / 2) return none;
    const long long first = ((N + 63) / 64 + 1) / 2;                   // of a chain's blocks
    if (N - 64 * first <= 64 * (kHalf - 1) || N - 64 * first < ltn::cut_state_rows(D)) return none;
    const long long row_bytes = count == 3 ? 8LL * D : 2 * (2LL * D + DC);       // of every input
    const long long least = least_cut_mib(count, slices, gated, xcd, wgs / units, alone, units) * kKiB * kKiB;
    if (row_bytes * chains * N < least) return none;
    const long long chain_bytes = 2LL * D * N;
    if (count == 3 && slices == 1 && 16 * alone > 7 * units && chain_bytes > 511 * kKiB && chain_bytes < 513 * kKiB) return none;
    const Cut cut = {(int)(xcd ? 8 * cut_chains : cut_chains), 64 * first};
    return cut.chains <= chains ? cut : none;
}

// Cache hints of a launch of `pb` in slices of dv value columns.  Launches of these sizes are bound by memory (with
// every product taken out of the kernels they take 0 .. 6 % less), and what they read once goes through an L2 of 4 MiB
// an XCD and a memory-side cache of 256 MiB on its way, where it takes the place of what another pass is about to read
// again.  Measured without and with, us, rotating inputs:
//   backward, full width, each pass's A once and outputs past the caches, which keep what dQ's pass reads again; after its
//     forward: 128 features 128 chains x 2048 / 8192 tokens 184.5 and 172.7, 713 and 688, 200 x 3000 414 and 402, 16 x
//     16384 (segments) 265 and 257; 96 features 544 x 928 299 and 282; 64 features 320 x 2048 227 and 216, 128 x 6000 269
//     and 256, but 180 x 2829 (249 MiB) 187 and 193.  Inputs that the memory-side cache holds lose (alone: 64 x 1000
//     34.0 and 36.6, 128 x 1000 65.4 and 69.2), and so do 64-column slices (32 x 16301 322 and 334).
//     With the gradients read next (forward, backward, copies of dQ, dK, dV): 128 features 128 x 2048 269 and 262, 128 x 8192
//     1017 and 975, 200 x 3000 589 and 576; 96 features 544 x 928 411 and 393; 64 features 320 x 2048 334 and 320, 600 x 2048
//     (600 MiB) 627 and 621, but from 650 MiB on most with 128 chains or more lose (512 x 2600 666 and 671, 640 x 2200 699 and 709,
//     640 x 3000 948 and 966, 1024 x 2048 1011 and 1025, 2500 x 1024 1146 and 1179; 250 x 8192 982 and 971), not with
//     fewer (102 x 25568 1385 and 1372, 64 x 25000 925 and 915).  Just past the lines, where the last round of workgroups
//     is partly filled, up to 2 % are lost (100 x 2476 269 and 273, 260 x 1500 x 96 332 and 338; beside them 128 x 2000 254 and 249,
//     200 x 1300 265 and 258, 256 x 1000 252 and 247).  96 features in segments: nothing (16 x 24000 440 and 440)
//   forward in segments, all once in the pass after the sweep and outputs past the caches, so that K and V of the sweep
//     stay: 32 x 16301 and its backward 501 and 475; alone 176 and 140, 8 x 65536 179 and 154.  With a gate that reads O, and
//     the backward: 16 x 16384 (256 MiB) 297 and 307, 16 x 20000 359 and 367, 32 x 12000 (375) 407 and 404, 32 x 13000
//     (406) 453 and 449, 32 x 16301 571 and 554 (O kept 550; with a copy of O and no backward 235, 201 and 206)
//   gated forward without o (inference), all once, outputs through the caches: 128 features 256 x 500 38.9 and 34.8, 512 x
//     1000 139 and 131, segments 32 x 8192 103 and 92, 64 x 3000 79 and 76; 64 features 320 x 2048 92 and 87; 96
//     features 320 x 2000 139 and 129, but rows of 192 bytes, whose lines two loads share, need a nearly full chip (x 2000:
//     128 chains 60.3 and 62.4, 160 68.1 and 67.8, 192 78.1 and 76.4, 224 88.3 and 83.9).  Below 64 MiB (192 in
//     segments) nothing
// The plain forward of whole chains gains alone (all once: 256 x 4096 207 and 180) and loses with the backward that finds
// less of Q, K and V in the memory-side cache (fwd and bwd 320 x 2048 x 64 216 and 227, 200 x 3000 402 and 414, 256 x 1000
// 168 and 172; 256 x 4096 684 and 672).  256 features: nothing within 1 %.  Unequal widths, the first layer's step with copies of
// its gradients: forward and dV nothing; dK and dQ with C once and past 4 x 16 x 2048 x 128 338 and 332, 4 x 32 x 4096 1159
// and 1136, 1 x 32 x 30000 nothing, 4 x 32 x 4096 x 64 569 and 574: no hints.
void set_hints(ltn::PassBatch& pb, int D, int DC, int dv, bool segmented) {
    constexpr long long kMiB = 1 << 20;
    const long long tokens = pb.chains * pb.N;
    pb.hints = 0;
    if (D == 256 || D != DC || dv != D) return;
    if (pb.count == 3) {
        const long long bytes = 8LL * D * tokens;
        const bool pays = D == 64 ? bytes >= 288 * kMiB && (segmented || pb.chains < 128 || bytes < 640 * kMiB) : bytes >= 240 * kMiB && !(segmented && D == 96);
        if (pays) pb.hints = ltn::kOnceA | ltn::kPast;
    } else if (pb.p[0].gate) {
        const bool fills = D != 96 || (!segmented && pb.chains >= 192);
        if (!pb.p[0].out && fills && 10LL * D * tokens >= (segmented ? 192 : 64) * kMiB) pb.hints = ltn::kOnce;
    } else if (segmented && D == 128 && 8LL * D * tokens >= 400 * kMiB) {
        pb.hints = ltn::kOnce | ltn::kPast;
    }
}

// the passes of `pb` in whole chains, dv value columns a workgroup, or cut in two
ltn_status launch_whole_or_cut(ltn::PassBatch& pb, int D, int DC, int dv, int widest, hipStream_t stream) {
    const Cut cut = pick_cut(pb.chains, pb.count, pb.N, D, DC, dv, widest, pb.p[0].gate != nullptr);
    pb.cut_chains = cut.chains;
    pb.cut_len = cut.len;
    set_hints(pb, D, DC, dv, false);
    const hipError_t e = cut.chains ? ltn::launch_pass_cut_bf16(pb, D, stream, DC)
                                    : ltn::launch_pass_bf16(pb, D, dv, stream, DC);
    return e == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

int widest_dv(int D) { return D == 256 ? 64 : D; }

// full_width: the pass carries the gated epilogue, which needs complete output rows in one
// workgroup (slices of all D value columns).
ltn_status run_passes(ltn::PassBatch& pb, int D, int blk, ltn_dtype dtype, void* workspace, hipStream_t stream,
                      bool full_width = false) {
    if (dtype != LTN_BF16) return run_f32(pb, D, D, blk, stream, full_width);
    const long long chain_passes = (long long)pb.chains * pb.count;
    const SegPlan plan = pick_segments(chain_passes, pb.N, D, dtype, full_width,
                                       (pb.pairs_first && pb.count == 3) ? pb.chains : 0);
    pb.segs = 1;
    if (plan.segs == 1) {
        const int dv = full_width ? D : pick_dv(chain_passes, D, pb.count);
        return launch_whole_or_cut(pb, D, D, dv, widest_dv(D), stream);
    }
    // three launches: segment end states from zero, scan, then the pass proper per segment
    if (!workspace) return LTN_ERR_NULL;
    float* states = static_cast<float*>(workspace);
    const size_t per_pass = (size_t)pb.chains * plan.segs * D * D;
    const float* kv_in = pb.p[0].state_in;
    float* kv_out = pb.p[0].state_out;
    ltn::PassBatch sweep = pb;
    sweep.segs = plan.segs;
    sweep.seg_len = plan.seg_len;
    sweep.state_only = 1;
    sweep.need_last = kv_out != nullptr;
    int pass[3];
    sweep.count = swept_passes(pb, plan.segs, D, dtype, pass);
    for (int i = 0; i < sweep.count; ++i) {
        sweep.p[i] = pb.p[pass[i]];
        sweep.p[i].out = nullptr;
        sweep.p[i].gate = nullptr;
        sweep.p[i].gated_out = nullptr;
        sweep.p[i].state_in = nullptr;
        sweep.p[i].state_out = states + pass[i] * per_pass;
    }
    // one full-width workgroup per segment; narrower slices while those fit one round of compute
    // units (128 features, full width, 64 and 32 columns: forward of 2 chains x 8192 tokens 24.9, 22.4
    // and 21.9 us, 8 x 8000 32.5 and 29.7; 64 features, 64 and 32 columns: 17.7 and 17.1; same values)
    int sweep_dv = D == 256 ? 64 : D == 96 ? 32 : D;
    while ((D == 64 || D == 128) && sweep_dv > 32 && (long long)pb.chains * sweep.count * plan.segs * (2 * D / sweep_dv) <= 256) sweep_dv /= 2;
    if (ltn::launch_pass_bf16(sweep, D, sweep_dv, stream) != hipSuccess) return LTN_ERR_LAUNCH;
    if (sweep.count != pb.count) {
        const ltn::ScanStates s = {{states, states + per_pass, states + 2 * per_pass}, (size_t)plan.segs * D * D, {0, 0, 0}, 0};
        if (ltn::launch_segment_scan_pair(s, pb.decay, pb.chains, pb.H, plan.segs, plan.seg_len, pb.N, D, stream) != hipSuccess)
            return LTN_ERR_LAUNCH;
    } else if (ltn::launch_segment_scan(states, kv_in, kv_out, pb.decay, pb.count, pb.chains, pb.H, plan.segs,
                                        plan.seg_len, pb.N, D, stream) != hipSuccess) {
        return LTN_ERR_LAUNCH;
    }
    ltn::PassBatch main = pb;
    main.segs = plan.segs;
    main.seg_len = plan.seg_len;
    for (int i = 0; i < pb.count; ++i) {
        main.p[i].state_in = states + i * per_pass;
        main.p[i].state_out = nullptr;
    }
    const int dv = full_width ? D : pick_dv(chain_passes * plan.segs, D, pb.count);
    set_hints(main, D, D, dv, true);
    return ltn::launch_pass_bf16(main, D, dv, stream) == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

// Scratch of ltn_attn_fwd_static: device memory that belongs to the library's code object,
// so that entry point needs no allocation and no caller workspace.  Every GPU the library
// runs on holds its own copy at its own address until the process ends; in host code the
// array's name is only a handle for hipGetSymbolAddress, never an address to pass on.
constexpr size_t kScratchBytes = (size_t)LTN_ATTN_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
ltn_status scratch_on_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LTN_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return LTN_ERR_LAUNCH;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return LTN_OK;
}

}  // namespace

extern "C" {

ltn_status ltn_attn_set_debug_plan(int dv, int segs) {
    if (dv != 0 && dv != 16 && dv != 32 && dv != 64 && dv != 96 && dv != 128 && dv != 256) return LTN_ERR_SHAPE;
    if (segs < 0 || segs > 4096) return LTN_ERR_SHAPE;
    g_debug_dv.store(dv, std::memory_order_relaxed);
    g_debug_segs.store(segs, std::memory_order_relaxed);
    return LTN_OK;
}

ltn_status ltn_attn_query_plan(int Bt, int H, long long N, int D, ltn_dtype dtype, int call,
                               int* dv_out, int* segs_out) {
    if (!dv_out || !segs_out) return LTN_ERR_NULL;
    if (Bt <= 0 || H <= 0 || N <= 0 || call < 0 || call > 2) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (D != 64 && D != 96 && D != 128 && D != 256) return LTN_ERR_UNSUPPORTED;
    const long long chains = (long long)Bt * H;
    const int count = call == 1 ? 3 : 1, blk = ltn_attn_pick_block(D, dtype);
    const bool fused = call == 2 && !gated_in_two_steps(chains, N, D, dtype, blk, false);
    if (dtype == LTN_F32) {
        const F32Plan f = pick_f32(chains, count, N, D, D, blk, fused);
        *segs_out = f.segs;
        *dv_out = f.dv;
        return LTN_OK;
    }
    const SegPlan plan = pick_segments(chains * count, N, D, dtype, fused, call == 1 ? chains : 0);
    *segs_out = plan.segs;
    *dv_out = fused ? D : pick_dv(chains * count * plan.segs, D, count);
    return LTN_OK;
}

ltn_status ltn_attn_query_sweeps(int Bt, int H, long long N, int D, ltn_dtype dtype, int* sweeps_out) {
    if (!sweeps_out) return LTN_ERR_NULL;
    int dv, segs;
    const ltn_status s = ltn_attn_query_plan(Bt, H, N, D, dtype, 1, &dv, &segs);
    if (s == LTN_OK) *sweeps_out = backward_sweeps((long long)Bt * H, segs, D, dtype);
    return s;
}

int ltn_attn_pick_block(int D, ltn_dtype dtype) {
    if (D != 64 && D != 96 && D != 128 && D != 256) return 0;
    if (dtype == LTN_BF16) return 64;
    if (dtype == LTN_F32) return D == 64 ? 64 : (D == 256 ? 16 : 32);
    return 0;
}

size_t ltn_attn_workspace_bytes(int Bt, int H, long long N, int D, int block, ltn_dtype dtype, int call) {
    (void)block;
    if (Bt <= 0 || H <= 0 || N <= 0 || (D != 64 && D != 96 && D != 128 && D != 256) || call < 0 || call > 2) return 0;
    const long long chains = (long long)Bt * H;
    const int count = (call == 1) ? 3 : 1;
    const size_t state = (size_t)D * D * sizeof(float);                                   // one fp32 state per segment
    const SegPlan plan = pick_segments(chains * count, N, D, dtype, call == 2, call == 1 ? chains : 0);
    size_t need = plan.segs == 1 ? 0 : (size_t)count * (size_t)chains * (size_t)plan.segs * state;
    if (call == 2) {
        // the gated forward may run as the plain forward followed by the gate kernel (when the
        // attention output is stored anyway): room for whichever plan needs more
        const SegPlan plain = pick_segments(chains, N, D, dtype, false);
        const size_t alt = plain.segs == 1 ? 0 : (size_t)chains * (size_t)plain.segs * state;
        if (alt > need) need = alt;
    }
    return need;
}

ltn_status ltn_attn_check_decay(const float* decay_host, int H) {
    if (!decay_host) return LTN_ERR_NULL;
    if (H < 0) return LTN_ERR_SHAPE;
    for (int h = 0; h < H; ++h)
        if (!(decay_host[h] >= 0.0f && decay_host[h] <= 1.0f)) return LTN_ERR_DECAY;
    return LTN_OK;
}

const char* ltn_status_str(ltn_status s) {
    switch (s) {
        case LTN_OK: return "LTN_OK";
        case LTN_ERR_NULL: return "LTN_ERR_NULL: a required pointer is NULL";
        case LTN_ERR_SHAPE: return "LTN_ERR_SHAPE: bad size or workspace too small";
        case LTN_ERR_UNSUPPORTED: return "LTN_ERR_UNSUPPORTED: shape/dtype/block not supported, or an output overlaps an input or another output";
        case LTN_ERR_ALIGN: return "LTN_ERR_ALIGN: tensor pointer not 16-byte aligned";
        case LTN_ERR_DECAY: return "LTN_ERR_DECAY: decay value outside [0, 1]";
        case LTN_ERR_LAUNCH: return "LTN_ERR_LAUNCH: HIP launch failed";
        case LTN_ERR_SCRATCH: return "LTN_ERR_SCRATCH: the call needs more scratch than the library's static buffer holds";
        default: break;
    }
    return "LTN_ERR_?: unknown status";
}

// Shared body of ltn_attn_fwd and ltn_attn_fwd_gated (u == nullptr: plain forward).
static ltn_status fwd_common(const void* q, const void* k, const void* v, const void* u, void* o, void* y,
                             const float* decay, const float* kv_in, float* kv_out, float eps,
                             int Bt, int H, long long N, int D, int block, ltn_dtype dtype,
                             void* workspace, size_t workspace_bytes, void* stream, bool gated) {
    const bool empty = (Bt == 0 || H == 0 || N == 0);   // no token is read or written
    if (!decay || (!empty && (!q || !k || !v || (gated ? (!u || !y) : !o)))) return LTN_ERR_NULL;
    int blk = 0;
    const ltn_status cs = check_common(Bt, H, N, D, block, dtype, &blk);
    if (cs != LTN_OK) return cs;
    if (gated && !(eps >= 0.0f)) return LTN_ERR_SHAPE;
    // 256 features (and 96 in fp32): no kernel holds a complete output row of these widths in one
    // workgroup, so the epilogue is applied to the stored attention output by the gate kernel; a
    // caller that does not want o stored has no fused form to fall back on
    const bool unfused_only = gated && (D == 256 || (D == 96 && dtype != LTN_BF16));
    if (unfused_only && !o && !empty) return LTN_ERR_UNSUPPORTED;
    const size_t need_ws = ltn_attn_workspace_bytes(Bt, H, N, D, block, dtype, gated ? 2 : 0);
    if (workspace_bytes < need_ws) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(u) || !aligned16(y) ||
        !aligned16(kv_in) || !aligned16(kv_out) || !aligned16(workspace) ||
        (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    const long long chains = (long long)Bt * H;
    if (!empty) {
        const size_t tb = (size_t)chains * (size_t)N * D * esize_of(dtype), sb = (size_t)chains * D * D * sizeof(float);
        // kv_out may be kv_in itself (a state updated in place); any other overlap is refused
        const Span ins[5] = {{q, tb}, {k, tb}, {v, tb}, {u, tb}, {kv_in == kv_out ? nullptr : kv_in, sb}};
        const Span outs[4] = {{o, tb}, {y, tb}, {kv_out, sb}, {workspace, need_ws}};
        if (outputs_alias(outs, 4, ins, 5)) return LTN_ERR_UNSUPPORTED;
    }
    if (chains == 0) return LTN_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (N == 0) {
        if (!kv_out) return LTN_OK;
        if (kv_in && kv_in != kv_out && spans_overlap({kv_in, (size_t)chains * D * D * sizeof(float)},
                                                      {kv_out, (size_t)chains * D * D * sizeof(float)}))
            return LTN_ERR_UNSUPPORTED;
        return ltn::launch_state_copy(kv_in, kv_out, (size_t)chains * D * D, st) == hipSuccess
                   ? LTN_OK : LTN_ERR_LAUNCH;
    }
    ltn::PassBatch pb = {};
    pb.segs = 1;
    pb.count = 1;
    pb.decay = decay;
    pb.chains = (int)chains;
    pb.H = H;
    pb.N = N;
    pb.p[0] = ltn::PassArgs{q, k, v, o, kv_in, kv_out, 0, gated ? u : nullptr, gated ? y : nullptr, eps};
    if (!gated) return run_passes(pb, D, blk, dtype, workspace, st);
    const bool two_steps = gated_in_two_steps(chains, N, D, dtype, blk, o != nullptr);
    if (two_steps) {
        void* const dst = o ? o : y;
        pb.p[0].out = dst;
        pb.p[0].gate = nullptr;
        pb.p[0].gated_out = nullptr;
        const ltn_status s1 = run_passes(pb, D, blk, dtype, workspace, st);
        if (s1 != LTN_OK) return s1;
        return ltn::launch_gate(dst, u, nullptr, y, nullptr, eps, chains * N, D, dtype == LTN_BF16, 0, st) == hipSuccess
                   ? LTN_OK : LTN_ERR_LAUNCH;
    }
    return run_passes(pb, D, blk, dtype, workspace, st, true);
}

ltn_status ltn_attn_fwd(const void* q, const void* k, const void* v, void* o,
                        const float* decay, const float* kv_in, float* kv_out,
                        int Bt, int H, long long N, int D, int block, ltn_dtype dtype,
                        void* workspace, size_t workspace_bytes, void* stream) {
    return fwd_common(q, k, v, nullptr, o, nullptr, decay, kv_in, kv_out, 0.0f, Bt, H, N, D, block, dtype,
                      workspace, workspace_bytes, stream, false);
}

ltn_status ltn_attn_fwd_static(const void* q, const void* k, const void* v, void* o,
                               const float* decay, const float* kv_in, float* kv_out,
                               int Bt, int H, long long N, int D, int block, ltn_dtype dtype, void* stream) {
    // the plan (and so the scratch it needs) is the one ltn_attn_fwd would take
    if (ltn_attn_workspace_bytes(Bt, H, N, D, block, dtype, 0) > kScratchBytes) return LTN_ERR_SCRATCH;
    void* ws = nullptr;
    const ltn_status s = scratch_on_current_device(&ws);
    if (s != LTN_OK) return s;
    // Nothing in the scratch has to start at zero: the scan reads exactly the segment end
    // states that the state-only sweep of the same call has written.
    return fwd_common(q, k, v, nullptr, o, nullptr, decay, kv_in, kv_out, 0.0f, Bt, H, N, D, block, dtype,
                      ws, kScratchBytes, stream, false);
}

ltn_status ltn_attn_fwd_gated(const void* q, const void* k, const void* v, const void* u, void* o, void* y,
                              const float* decay, const float* kv_in, float* kv_out, float eps,
                              int Bt, int H, long long N, int D, int block, ltn_dtype dtype,
                              void* workspace, size_t workspace_bytes, void* stream) {
    return fwd_common(q, k, v, u, o, y, decay, kv_in, kv_out, eps, Bt, H, N, D, block, dtype,
                      workspace, workspace_bytes, stream, true);
}

ltn_status ltn_attn_fwd_tiled(const void* q, const void* k, const void* v, void* o, const float* decay,
                              int Bt, int H, long long N, int D, ltn_dtype dtype, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || N == 0);
    if (!decay || (!empty && (!q || !k || !v || !o))) return LTN_ERR_NULL;
    if (Bt < 0 || H < 0 || N < 0 || D <= 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_BF16 || (D != 64 && D != 128)) return LTN_ERR_UNSUPPORTED;
    if ((long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
        (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    if (!empty) {
        const size_t tb = (size_t)Bt * H * (size_t)N * D * esize_of(dtype);
        const Span ins[3] = {{q, tb}, {k, tb}, {v, tb}};
        const Span outs[1] = {{o, tb}};
        if (outputs_alias(outs, 1, ins, 3)) return LTN_ERR_UNSUPPORTED;
    }
    if (empty) return LTN_OK;
    return ltn::launch_tiled_fwd_bf16(q, k, v, o, decay, Bt * H, H, N, D, static_cast<hipStream_t>(stream)) ==
                   hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

ltn_status ltn_attn_bwd_tiled(const void* q, const void* k, const void* v, const void* d_o,
                              void* dq, void* dk, void* dv, const float* decay,
                              int Bt, int H, long long N, int D, ltn_dtype dtype, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || N == 0);
    if (!decay || (!empty && (!q || !k || !v || !d_o || !dq || !dk || !dv))) return LTN_ERR_NULL;
    if (Bt < 0 || H < 0 || N < 0 || D <= 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_BF16 || (D != 64 && D != 128)) return LTN_ERR_UNSUPPORTED;
    if ((long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o) || !aligned16(dq) ||
        !aligned16(dk) || !aligned16(dv) || (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    if (empty) return LTN_OK;
    const size_t tb = (size_t)Bt * H * (size_t)N * D * esize_of(dtype);
    const Span ins[4] = {{q, tb}, {k, tb}, {v, tb}, {d_o, tb}};
    const Span outs[3] = {{dq, tb}, {dk, tb}, {dv, tb}};
    if (outputs_alias(outs, 3, ins, 4)) return LTN_ERR_UNSUPPORTED;
    return ltn::launch_tiled_bwd_bf16(q, k, v, d_o, dq, dk, dv, decay, Bt * H, H, N, D,
                                      static_cast<hipStream_t>(stream)) == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

static ltn_status gate_common(const void* x, const void* u, const void* d_y, void* o0, void* o1, float eps,
                              long long rows, int D, ltn_dtype dtype, void* stream, bool bwd) {
    if (rows < 0 || D <= 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (D != 64 && D != 96 && D != 128 && D != 256) return LTN_ERR_UNSUPPORTED;
    if (!(eps >= 0.0f)) return LTN_ERR_SHAPE;
    if (rows == 0) return LTN_OK;
    if (!x || !u || !o0 || (bwd && (!d_y || !o1))) return LTN_ERR_NULL;
    if (!aligned16(x) || !aligned16(u) || !aligned16(d_y) || !aligned16(o0) || !aligned16(o1)) return LTN_ERR_ALIGN;
    {
        const size_t tb = (size_t)rows * D * esize_of(dtype);
        const Span ins[3] = {{x, tb}, {u, tb}, {d_y, tb}};
        const Span outs[2] = {{o0, tb}, {bwd ? o1 : nullptr, tb}};
        if (outputs_alias(outs, 2, ins, 3)) return LTN_ERR_UNSUPPORTED;
    }
    const hipError_t e = ltn::launch_gate(x, u, d_y, o0, o1, eps, rows, D, dtype == LTN_BF16, bwd,
                                          static_cast<hipStream_t>(stream));
    return e == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

ltn_status ltn_gate_fwd(const void* x, const void* u, void* y, float eps,
                        long long rows, int D, ltn_dtype dtype, void* stream) {
    return gate_common(x, u, nullptr, y, nullptr, eps, rows, D, dtype, stream, false);
}

ltn_status ltn_gate_bwd(const void* x, const void* u, const void* d_y, void* d_x, void* d_u, float eps,
                        long long rows, int D, ltn_dtype dtype, void* stream) {
    return gate_common(x, u, d_y, d_x, d_u, eps, rows, D, dtype, stream, true);
}

ltn_status ltn_attn_bwd(const void* q, const void* k, const void* v, const void* d_o,
                        void* dq, void* dk, void* dv, const float* decay,
                        int Bt, int H, long long N, int D, int block, ltn_dtype dtype,
                        void* workspace, size_t workspace_bytes, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || N == 0);
    if (!decay || (!empty && (!q || !k || !v || !d_o || !dq || !dk || !dv))) return LTN_ERR_NULL;
    int blk = 0;
    const ltn_status cs = check_common(Bt, H, N, D, block, dtype, &blk);
    if (cs != LTN_OK) return cs;
    const size_t need_ws = ltn_attn_workspace_bytes(Bt, H, N, D, block, dtype, 1);
    if (workspace_bytes < need_ws) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o) || !aligned16(dq) ||
        !aligned16(dk) || !aligned16(dv) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    const long long chains = (long long)Bt * H;
    if (!empty) {
        const size_t tb = (size_t)chains * (size_t)N * D * esize_of(dtype);
        const Span ins[4] = {{q, tb}, {k, tb}, {v, tb}, {d_o, tb}};
        const Span outs[4] = {{dq, tb}, {dk, tb}, {dv, tb}, {workspace, need_ws}};
        if (outputs_alias(outs, 4, ins, 4)) return LTN_ERR_UNSUPPORTED;
    }
    if (chains == 0 || N == 0) return LTN_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // The three gradients are three decayed linear-attention passes with permuted
    // operands (derivative of O = ((Q K^T)(.)M) V; App. B Algorithm 4 corrected):
    //   dQ = ((dO V^T)(.)M)   K   -> pass(dO, V, K), first token -> last
    //   dV = ((Q K^T)(.)M)^T  dO  -> pass(K, Q, dO), last token -> first
    //   dK = ((dO V^T)(.)M)^T Q   -> pass(V, dO, Q), last token -> first
    ltn::PassBatch pb = {};
    pb.segs = 1;
    pb.count = 3;
    pb.decay = decay;
    pb.chains = (int)chains;
    pb.H = H;
    pb.N = N;
    pb.p[0] = ltn::PassArgs{k, q, d_o, dv, nullptr, nullptr, 1};
    pb.p[1] = ltn::PassArgs{v, d_o, q, dk, nullptr, nullptr, 1};
    pb.p[2] = ltn::PassArgs{d_o, v, k, dq, nullptr, nullptr, 0};
    pb.pairs_first = 1;
    return run_passes(pb, D, blk, dtype, workspace, st);
}

ltn_status ltn_attn_decode_steps(const void* q, const void* k, const void* v, void* o,
                                 float* kv, const float* decay,
                                 int Bt, int H, int S, int D, ltn_dtype dtype, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || S == 0);   // no token is read, the state is not touched
    if (!decay || (!empty && (!q || !k || !v || !o || !kv))) return LTN_ERR_NULL;
    if (Bt < 0 || H < 0 || S < 0 || D <= 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (D != 64 && D != 96 && D != 128 && D != 256) return LTN_ERR_UNSUPPORTED;
    if ((long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(kv) ||
        (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    const int chains = Bt * H;
    if (!empty) {
        const size_t tb = (size_t)chains * S * D * esize_of(dtype);
        const Span ins[3] = {{q, tb}, {k, tb}, {v, tb}};
        const Span outs[2] = {{o, tb}, {kv, (size_t)chains * D * D * sizeof(float)}};
        if (outputs_alias(outs, 2, ins, 3)) return LTN_ERR_UNSUPPORTED;
    }
    if (empty) return LTN_OK;
    const hipError_t e = ltn::launch_decode(q, k, v, o, kv, decay, chains, H, S, D, D, dtype == LTN_BF16,
                                            static_cast<hipStream_t>(stream));
    return e == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

ltn_status ltn_attn_decode_step(const void* q, const void* k, const void* v, void* o,
                                float* kv, const float* decay,
                                int Bt, int H, int D, ltn_dtype dtype, void* stream) {
    return ltn_attn_decode_steps(q, k, v, o, kv, decay, Bt, H, 1, D, dtype, stream);
}

// ---------------------------------------------------------------------------------------
// Query/key width Dk = 2 Dv (behind the LRPE-d expansion) and the input side itself.
// ---------------------------------------------------------------------------------------

static ltn_status check_dkdv(int Bt, int H, long long N, int Dk, int Dv, int block, ltn_dtype dtype, int* blk_out) {
    if (Bt < 0 || H < 0 || N < 0 || Dk <= 0 || Dv <= 0 || block < 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (!((Dk == 256 && Dv == 128) || (Dk == 128 && Dv == 64))) return LTN_ERR_UNSUPPORTED;
    int blk = block;
    if (dtype == LTN_BF16) {
        if (blk == 0) blk = 64;
        if (blk != 64) return LTN_ERR_UNSUPPORTED;
    } else {
        if (blk == 0) blk = Dk == 256 ? 16 : 32;
        if (blk != 16 && !(blk == 32 && Dk == 128)) return LTN_ERR_UNSUPPORTED;
    }
    if ((long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    *blk_out = blk;
    return LTN_OK;
}

// Slices the bf16 kernels exist for behind a DA-wide query/key side: 32..64 for 256 (its state
// copies fill the LDS beyond that) and for 64, 32..min(DC,128) otherwise; the state-only sweep
// of the sequence-parallel form uses the widest of them.
static int dkdv_hi(int DA, int DC) { return (DA == 256 || DA == 64) ? 64 : (DC < 128 ? DC : 128); }

// Sequence-parallel plan of a launch of `chain_passes` passes of shape (DA, DC): as for equal
// widths (pick_segments), with DC / hi workgroups per chain segment.  bf16 only.
static SegPlan pick_segments_dkdv(long long chain_passes, long long N, int DA, int DC, ltn_dtype dtype) {
    SegPlan plan = {1, 0};
    if (dtype != LTN_BF16 || chain_passes <= 0 || N <= 64) return plan;
    const long long per_seg = DC / dkdv_hi(DA, DC);
    long long want = 256 / (per_seg * chain_passes);
    const long long finer = N / 256 < want ? N / 256 : want;
    if (want > N / 512) want = N / 512;       // segments of at least 512 tokens (measured: 2 .. 32 chains, N = 2048 .. 16384)
    const bool try_finer = want < 8 && finer > want && finer >= 4;
    if (want < kMinSegsFullWidth) want = 1;
    // (DA < DC: the second launch of a backward, issued while the first one runs)
    if (try_finer && finer_pays(finer, want, chain_passes, N, DA, DC, false, DA < DC ? 0.0 : kIssue)) want = finer;
    if (const int v = g_debug_segs.load(std::memory_order_relaxed)) want = v;
    return cut_chain(N, want);
}

// One launch of `pb` (passes of one shape): a, b with DA features, c and out with DC; cut into
// segments (state-only sweep, scan, per-segment pass) when the plan says so.
static ltn_status run_dkdv(ltn::PassBatch& pb, int DA, int DC, int blk, ltn_dtype dtype, void* workspace, hipStream_t st) {
    const long long chain_passes = (long long)pb.chains * pb.count;
    pb.segs = 1;
    if (dtype != LTN_BF16) return run_f32(pb, DA, DC, blk, st);
    const int hi = dkdv_hi(DA, DC);
    const SegPlan plan = pick_segments_dkdv(chain_passes, pb.N, DA, DC, dtype);
    if (plan.segs == 1) return launch_whole_or_cut(pb, DA, DC, pick_dv_range(chain_passes, DC, 32, hi), hi, st);
    if (!workspace) return LTN_ERR_NULL;
    float* states = static_cast<float*>(workspace);
    const size_t per_pass = (size_t)pb.chains * plan.segs * DA * DC;
    const float* kv_in = pb.p[0].state_in;
    float* kv_out = pb.p[0].state_out;
    ltn::PassBatch sweep = pb;
    sweep.segs = plan.segs;
    sweep.seg_len = plan.seg_len;
    sweep.state_only = 1;
    sweep.need_last = kv_out != nullptr;
    for (int i = 0; i < pb.count; ++i) {
        sweep.p[i].out = nullptr;
        sweep.p[i].state_in = nullptr;
        sweep.p[i].state_out = states + i * per_pass;
    }
    if (ltn::launch_pass_bf16(sweep, DA, hi, st, DC) != hipSuccess) return LTN_ERR_LAUNCH;
    if (ltn::launch_segment_scan(states, kv_in, kv_out, pb.decay, pb.count, pb.chains, pb.H, plan.segs, plan.seg_len,
                                 pb.N, DA, st, DC) != hipSuccess)
        return LTN_ERR_LAUNCH;
    ltn::PassBatch main = pb;
    main.segs = plan.segs;
    main.seg_len = plan.seg_len;
    for (int i = 0; i < pb.count; ++i) {
        main.p[i].state_in = states + i * per_pass;
        main.p[i].state_out = nullptr;
    }
    const int dv = pick_dv_range(chain_passes * plan.segs, DC, 32, hi);
    return ltn::launch_pass_bf16(main, DA, dv, st, DC) == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

size_t ltn_attn_workspace_bytes_dkdv(int Bt, int H, long long N, int Dk, int Dv, ltn_dtype dtype, int call) {
    if (Bt <= 0 || H <= 0 || N <= 0 || call < 0 || call > 1) return 0;
    if (!((Dk == 256 && Dv == 128) || (Dk == 128 && Dv == 64))) return 0;
    const long long chains = (long long)Bt * H;
    const size_t state = (size_t)Dk * Dv * sizeof(float);
    // forward and the dV pass: (Dk, Dv), one pass per chain; dK and dQ: (Dv, Dk), two; the two
    // launches of the backward follow each other on the stream and share the workspace
    const SegPlan a = pick_segments_dkdv(chains, N, Dk, Dv, dtype);
    size_t need = a.segs > 1 ? (size_t)chains * a.segs * state : 0;
    if (call == 1) {
        const SegPlan b = pick_segments_dkdv(2 * chains, N, Dv, Dk, dtype);
        const size_t nb = b.segs > 1 ? (size_t)2 * chains * b.segs * state : 0;
        if (nb > need) need = nb;
    }
    return need;
}

ltn_status ltn_attn_query_cut(int Bt, int H, long long N, int Dk, int Dv, ltn_dtype dtype, int call,
                              int* chains_out, long long* tokens_out) {
    if (!chains_out || !tokens_out) return LTN_ERR_NULL;
    if (Bt <= 0 || H <= 0 || N <= 0 || call < 0 || call > 2 || (long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    int blk = 0;
    const ltn_status s = Dk == Dv ? check_common(Bt, H, N, Dk, 0, dtype, &blk)
                                  : check_dkdv(Bt, H, N, Dk, Dv, 0, dtype, &blk);
    if (s != LTN_OK) return s;
    if (Dk != Dv && call == 2) return LTN_ERR_UNSUPPORTED;
    const int chains = Bt * H;
    Cut cut = {0, 0};
    if (dtype == LTN_BF16 && Dk == Dv) {
        const int count = call == 1 ? 3 : 1;
        const bool fused = call == 2 && !gated_in_two_steps(chains, N, Dk, dtype, blk, false);
        if (pick_segments((long long)chains * count, N, Dk, dtype, fused, call == 1 ? chains : 0).segs == 1)
            cut = pick_cut(chains, count, N, Dk, Dk, fused ? Dk : pick_dv((long long)chains * count, Dk, count),
                           widest_dv(Dk), fused);
    } else if (dtype == LTN_BF16) {        // of a backward: the launch of dK and dQ
        const int count = call == 1 ? 2 : 1, DA = call == 1 ? Dv : Dk, DC = call == 1 ? Dk : Dv, hi = dkdv_hi(DA, DC);
        if (pick_segments_dkdv((long long)chains * count, N, DA, DC, dtype).segs == 1)
            cut = pick_cut(chains, count, N, DA, DC, pick_dv_range((long long)chains * count, DC, 32, hi), hi);
    }
    *chains_out = cut.chains;
    *tokens_out = cut.len;
    return LTN_OK;
}

ltn_status ltn_attn_fwd_dkdv(const void* q, const void* k, const void* v, void* o,
                             const float* decay, const float* kv_in, float* kv_out,
                             int Bt, int H, long long N, int Dk, int Dv, int block, ltn_dtype dtype,
                             void* workspace, size_t workspace_bytes, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || N == 0);
    if (!decay || (!empty && (!q || !k || !v || !o))) return LTN_ERR_NULL;
    int blk = 0;
    const ltn_status cs = check_dkdv(Bt, H, N, Dk, Dv, block, dtype, &blk);
    if (cs != LTN_OK) return cs;
    const size_t need_ws = ltn_attn_workspace_bytes_dkdv(Bt, H, N, Dk, Dv, dtype, 0);
    if (workspace_bytes < need_ws) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(kv_in) ||
        !aligned16(kv_out) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    const long long chains = (long long)Bt * H;
    if (!empty) {
        const size_t qb = (size_t)chains * (size_t)N * Dk * esize_of(dtype), vb = (size_t)chains * (size_t)N * Dv * esize_of(dtype);
        const size_t sb = (size_t)chains * Dk * Dv * sizeof(float);
        const Span ins[4] = {{q, qb}, {k, qb}, {v, vb}, {kv_in == kv_out ? nullptr : kv_in, sb}};
        const Span outs[3] = {{o, vb}, {kv_out, sb}, {workspace, need_ws}};
        if (outputs_alias(outs, 3, ins, 4)) return LTN_ERR_UNSUPPORTED;
    }
    if (chains == 0) return LTN_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (N == 0) {
        if (!kv_out) return LTN_OK;
        return ltn::launch_state_copy(kv_in, kv_out, (size_t)chains * Dk * Dv, st) == hipSuccess
                   ? LTN_OK : LTN_ERR_LAUNCH;
    }
    ltn::PassBatch pb = {};
    pb.segs = 1;
    pb.count = 1;
    pb.decay = decay;
    pb.chains = (int)chains;
    pb.H = H;
    pb.N = N;
    pb.p[0] = ltn::PassArgs{q, k, v, o, kv_in, kv_out, 0};
    return run_dkdv(pb, Dk, Dv, blk, dtype, workspace, st);
}

ltn_status ltn_attn_bwd_dkdv(const void* q, const void* k, const void* v, const void* d_o,
                             void* dq, void* dk, void* dv, const float* decay,
                             int Bt, int H, long long N, int Dk, int Dv, int block, ltn_dtype dtype,
                             void* workspace, size_t workspace_bytes, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || N == 0);
    if (!decay || (!empty && (!q || !k || !v || !d_o || !dq || !dk || !dv))) return LTN_ERR_NULL;
    int blk = 0;
    const ltn_status cs = check_dkdv(Bt, H, N, Dk, Dv, block, dtype, &blk);
    if (cs != LTN_OK) return cs;
    const size_t need_ws = ltn_attn_workspace_bytes_dkdv(Bt, H, N, Dk, Dv, dtype, 1);
    if (workspace_bytes < need_ws) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(d_o) || !aligned16(dq) ||
        !aligned16(dk) || !aligned16(dv) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    const long long chains = (long long)Bt * H;
    if (!empty) {
        const size_t qb = (size_t)chains * (size_t)N * Dk * esize_of(dtype), vb = (size_t)chains * (size_t)N * Dv * esize_of(dtype);
        const Span ins[4] = {{q, qb}, {k, qb}, {v, vb}, {d_o, vb}};
        const Span outs[4] = {{dq, qb}, {dk, qb}, {dv, vb}, {workspace, need_ws}};
        if (outputs_alias(outs, 4, ins, 4)) return LTN_ERR_UNSUPPORTED;
    }
    if (chains == 0 || N == 0) return LTN_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // The same three passes as ltn_attn_bwd; they come in two shapes, hence two launches:
    //   dV = pass(K, Q, dO), last token -> first:  Dk-wide a, b;  Dv-wide c, out
    //   dK = pass(V, dO, Q) (last -> first), dQ = pass(dO, V, K):  Dv-wide a, b;  Dk-wide c, out
    ltn::PassBatch pb = {};
    pb.segs = 1;
    pb.decay = decay;
    pb.chains = (int)chains;
    pb.H = H;
    pb.N = N;
    pb.count = 1;
    pb.p[0] = ltn::PassArgs{k, q, d_o, dv, nullptr, nullptr, 1};
    const ltn_status s1 = run_dkdv(pb, Dk, Dv, blk, dtype, workspace, st);
    if (s1 != LTN_OK) return s1;
    pb.count = 2;
    pb.p[0] = ltn::PassArgs{v, d_o, q, dk, nullptr, nullptr, 1};
    pb.p[1] = ltn::PassArgs{d_o, v, k, dq, nullptr, nullptr, 0};
    return run_dkdv(pb, Dv, Dk, blk, dtype, workspace, st);
}

ltn_status ltn_attn_decode_steps_dkdv(const void* q, const void* k, const void* v, void* o,
                                      float* kv, const float* decay,
                                      int Bt, int H, int S, int Dk, int Dv, ltn_dtype dtype, void* stream) {
    const bool empty = (Bt == 0 || H == 0 || S == 0);
    if (!decay || (!empty && (!q || !k || !v || !o || !kv))) return LTN_ERR_NULL;
    if (Bt < 0 || H < 0 || S < 0 || Dk <= 0 || Dv <= 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (!((Dk == 256 && Dv == 128) || (Dk == 128 && Dv == 64))) return LTN_ERR_UNSUPPORTED;
    if ((long long)Bt * H > 0x3fffffffLL) return LTN_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(kv) ||
        (reinterpret_cast<uintptr_t>(decay) & 3u))
        return LTN_ERR_ALIGN;
    if (!empty) {
        const size_t qb = (size_t)Bt * H * S * Dk * esize_of(dtype), vb = (size_t)Bt * H * S * Dv * esize_of(dtype);
        const Span ins[3] = {{q, qb}, {k, qb}, {v, vb}};
        const Span outs[2] = {{o, vb}, {kv, (size_t)Bt * H * Dk * Dv * sizeof(float)}};
        if (outputs_alias(outs, 2, ins, 3)) return LTN_ERR_UNSUPPORTED;
    }
    if (empty) return LTN_OK;
    const hipError_t e = ltn::launch_decode(q, k, v, o, kv, decay, Bt * H, H, S, Dk, Dv, dtype == LTN_BF16,
                                            static_cast<hipStream_t>(stream));
    return e == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

ltn_status ltn_probe_stream_read(const void* buf, size_t buf_bytes, size_t bytes_per_workgroup, int workgroups,
                                 int iters, int to_registers, unsigned* sink, void* stream) {
    if (!buf || !sink) return LTN_ERR_NULL;
    if (workgroups <= 0 || iters <= 0 || bytes_per_workgroup == 0 || bytes_per_workgroup % 65536 != 0) return LTN_ERR_SHAPE;
    if (bytes_per_workgroup > buf_bytes / (size_t)workgroups) return LTN_ERR_SHAPE;      // every region inside the buffer
    if (!aligned16(buf) || (reinterpret_cast<uintptr_t>(sink) & 3u)) return LTN_ERR_ALIGN;
    return ltn::launch_probe_stream(buf, bytes_per_workgroup, workgroups, iters, to_registers, sink,
                                    static_cast<hipStream_t>(stream)) == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

size_t ltn_prologue_workspace_bytes(int Bt, int H, long long N, int D) {
    if (Bt <= 0 || H <= 0 || N <= 0 || D <= 0) return 0;
    return (size_t)ltn::prologue_partial_count(N) * (size_t)H * (size_t)D * sizeof(double);
}

static ltn_status prologue_common(const void* x, const float* theta, const void* d_y, void* out, float* d_theta,
                                  int act, int Bt, int H, long long N, int D, long long pos0, ltn_dtype dtype,
                                  void* workspace, size_t workspace_bytes, void* stream, bool bwd) {
    if (Bt < 0 || H < 0 || N < 0 || D <= 0 || pos0 < 0) return LTN_ERR_SHAPE;
    if (dtype != LTN_F32 && dtype != LTN_BF16) return LTN_ERR_UNSUPPORTED;
    if (D != 64 && D != 128) return LTN_ERR_UNSUPPORTED;
    if ((long long)Bt * H > 0x3fffffffLL || pos0 + N > (1LL << 40)) return LTN_ERR_SHAPE;
    const bool empty = (Bt == 0 || H == 0 || N == 0);
    if (d_theta && !theta) return LTN_ERR_NULL;
    if (!empty && (!x || !out || (bwd && !d_y))) return LTN_ERR_NULL;
    const bool want_dtheta = bwd && theta && d_theta;
    if (want_dtheta && !empty) {
        if (workspace_bytes < ltn_prologue_workspace_bytes(Bt, H, N, D)) return LTN_ERR_SHAPE;
        if (!workspace) return LTN_ERR_NULL;
    }
    if (!aligned16(x) || !aligned16(d_y) || !aligned16(out) || !aligned16(workspace) ||
        (reinterpret_cast<uintptr_t>(theta) & 3u) || (reinterpret_cast<uintptr_t>(d_theta) & 3u))
        return LTN_ERR_ALIGN;
    if (!empty) {
        // x and d_x have D features per token; y and d_y have 2D behind the expansion, D without it
        const size_t xb = (size_t)Bt * H * (size_t)N * D * esize_of(dtype), yb = theta ? 2 * xb : xb;
        const size_t hb = (size_t)H * D * sizeof(float);
        const Span ins[3] = {{x, xb}, {d_y, yb}, {theta, hb}};
        const Span outs[3] = {{out, bwd ? xb : yb}, {d_theta, hb},
                              {want_dtheta ? workspace : nullptr, ltn_prologue_workspace_bytes(Bt, H, N, D)}};
        if (outputs_alias(outs, 3, ins, 3)) return LTN_ERR_UNSUPPORTED;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (empty) {
        // no token contributes: the angle gradient is zero
        if (want_dtheta && H > 0)
            return ltn::launch_state_copy(nullptr, d_theta, (size_t)H * D, st) == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
        return LTN_OK;
    }
    const hipError_t e = ltn::launch_prologue(x, theta, d_y, out, d_theta, static_cast<double*>(workspace), act != 0,
                                              Bt, H, N, D, pos0, dtype == LTN_BF16, bwd, st);
    return e == hipSuccess ? LTN_OK : LTN_ERR_LAUNCH;
}

ltn_status ltn_prologue_fwd(const void* x, const float* theta, void* y, int act,
                            int Bt, int H, long long N, int D, long long pos0, ltn_dtype dtype, void* stream) {
    return prologue_common(x, theta, nullptr, y, nullptr, act, Bt, H, N, D, pos0, dtype, nullptr, 0, stream, false);
}

ltn_status ltn_prologue_bwd(const void* x, const float* theta, const void* d_y, void* d_x, float* d_theta, int act,
                            int Bt, int H, long long N, int D, long long pos0, ltn_dtype dtype,
                            void* workspace, size_t workspace_bytes, void* stream) {
    return prologue_common(x, theta, d_y, d_x, d_theta, act, Bt, H, N, D, pos0, dtype, workspace, workspace_bytes,
                           stream, true);
}

}  // extern "C"
