// fp32 kernel for one decayed linear-attention pass on gfx950: the same block recurrence as the
// bf16 kernel (arXiv 2307.14995, Sec. 3.2.1 / Eq. 1; Sec. 3.3 Algorithm 2 in block form), every
// product on the matrix cores in full fp32 (v_mfma_f32_16x16x4_f32: fp32 operands and
// accumulation -- no reduced-precision step anywhere):
//
//   P    = (A_i B_i^T) (.) M,       M[r,c] = lambda^(r-c) for r >= c else 0
//   O_i  = P C_i + diag(lambda^(r+1)) A_i S_i
//   S_i+1 = lambda^len S_i + sum_c lambda^(len-1-c) b_c^T c_c
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s, a sixteenth of the bf16 rate).  So the
// layout is chosen to keep every SIMD's matrix pipe fed by two waves that do the same work:
//
//   * A workgroup (one per chain, pass and slice of DV value columns) has NT x KH waves, NT = DV/16:
//     wave (ct, kh) keeps rows [kh D/KH, (kh+1) D/KH) of the 16 state columns of tile ct in
//     accumulators for the whole sequence.  KH > 1 (narrow slices) keeps eight waves on the unit.
//   * The state never leaves the registers: the accumulator layout of S (lane = value column,
//     registers = key features 4g .. 4g+3) is the A operand of the next product with the
//     contraction index permuted (k-slot g of step j <-> feature 4g + j), so O^T = S^T A^T takes
//     it as it stands.  The same holds for the transposed scores P^T, which go through LDS once,
//     from the wave that formed them to all others.
//   * One barrier per block.  Between two of them a wave forms its score tiles of block i (the
//     causal 16x16 tiles, each split KS ways along the features, dealt over the waves), its part
//     of O^T = S^T A^T of block i and the state update of block i, and finishes the output of
//     block i - 1 (C^T P^T on top, a lane holding four consecutive features of a token: 16-byte
//     stores), whose scores -- and with KH > 1 the other waves' parts of S^T A^T -- came through
//     LDS at the last barrier.  The next block's tiles are fetched into registers at the start
//     and go to the other LDS stage towards the end.
//   * Operands contracted over a feature index are read 16 bytes per lane (one read feeds four
//     MFMAs), those contracted over the token index 4 bytes per lane; row pitches of 4 floats
//     more than a multiple of 32 keep both conflict-free.
// Measured (MI355X, 128 features, 32-token blocks): 5.0 / 3.0 / 1.9 us a block at 128 / 64 / 32
// columns, of which the MFMAs alone take 4.05 / 2.24 / 1.39; the rest are LDS latencies, which the
// two waves of a SIMD expose because they walk in step.  With the state copy published to LDS and
// two wave roles (the form before): 6.3 / 4.5 / 2.8; with plain multiply-adds (then the form of the
// gated pass, the unequal widths and 96 and 256 features) 28 at full width.
// Only non-negative powers of lambda are formed.
//
// Variants: the gated epilogue (full-width slices; the token mixer's y = SRMSNorm(o) (.) u of
// Eq. 3, row sums of squares exchanged through LDS) and the state-only sweep of the
// sequence-parallel form.  That form keeps its segment states in the output's own rows: a
// segment's D x DC start state sits in the first D of its output rows, column by column where
// the slice that reads it will write, so no scratch memory is needed.
#include <type_traits>
#include "ltn_kernels.h"

namespace ltn {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

enum { kPlain = 0, kGated = 1, kStateOnly = 2 };

__device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, int DV, int B, int KH>
struct FCfg {
    static constexpr int TS = B / 16;              // token strips of a block
    static constexpr int NT = DV / 16;             // 16-column tiles of the slice
    static constexpr int NW = NT * KH;             // waves
    static constexpr int THREADS = 64 * NW;
    static constexpr int MR = D / 16 / KH;         // 16-row state tiles of a wave
    // GR tiles interleave their rows: row m of tile t of a group stands for feature GR m + t, so one
    // GR-float LDS read per lane feeds GR tiles of the state update (and the S^T A^T operand of
    // a group is 4 GR consecutive features per lane, still read 16 bytes at a time)
    static constexpr int GR = MR % 4 == 0 ? 4 : (MR % 2 == 0 ? 2 : 1);
    // score units: TRI causal tiles x KS feature ranges
    static constexpr int TRI = TS * (TS + 1) / 2;
    static constexpr int KS = TS == 2 || D % 64 ? 2 : 4;
    static constexpr int PA = D + 4, PC = DV + 4, PP = B + 4;     // row pitches (floats)
    static constexpr int A_OFF = 0, B_OFF = B * PA, C_OFF = 2 * B * PA, STAGE = C_OFF + B * PC;
    // doubled: written while the previous block's are read
    static constexpr int P_OFF = 2 * STAGE, P_SIZE = KS * B * PP; // KS partial score blocks [token][key]
    static constexpr int X_ONE = 64 * 4, X_SIZE = NT * TS * (KH - 1) * X_ONE;
    static constexpr int X_OFF = P_OFF + 2 * P_SIZE;              // S^T A^T parts on their way to the strip's owner
    static constexpr int Q_OFF = X_OFF + 2 * X_SIZE, Q_SIZE = NT * B;      // gated: sums of squares [NT][B]
    static constexpr int PW_OFF = Q_OFF + 2 * Q_SIZE;
    static constexpr int FLOATS = PW_OFF + B + 4;
    static_assert(B == 16 || B == 32, "block lengths");
    static_assert(D % (16 * KH) == 0 && MR >= 1 && DV % 16 == 0, "state tiles");
    static_assert((D / 16) % KS == 0, "score feature ranges");
    static_assert(PA % 32 == 4 && PC % 16 == 4, "conflict-free pitches");
    static_assert(FLOATS * 4 <= 163840, "LDS per workgroup");
    static_assert(THREADS <= 1024, "workgroup size");
    // prefetch: 16-byte pieces per thread and tile (the last round of a tile may be partial)
    static constexpr int EA = B * (D / 4), EC = B * (DV / 4);
    static constexpr int LA = (EA + THREADS - 1) / THREADS, LC = (EC + THREADS - 1) / THREADS;
};

template <int D, int DV, int B, int KH, int DC, int MODE>
__global__ __launch_bounds__(64 * (DV / 16) * KH)
void pass_f32_kernel(const PassBatch pb, const int nsplit, const int xcd_ids) {
    using C = FCfg<D, DV, B, KH>;
    constexpr bool GATED = MODE == kGated, SO = MODE == kStateOnly;
    static_assert(!GATED || DV == DC, "the gated epilogue needs complete output rows");
    constexpr int TS = C::TS, NT = C::NT, NW = C::NW, MR = C::MR, GR = C::GR, KS = C::KS, PA = C::PA, PC = C::PC, PP = C::PP;
    typedef float vg __attribute__((ext_vector_type(GR)));
    __shared__ __attribute__((aligned(16))) float smem[C::FLOATS];
    float* pw = smem + C::PW_OFF;         // lambda^0 .. lambda^B

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, g = lane >> 4, i16 = lane & 15;
    const int ct = wave % NT, kh = wave / NT;      // waves w and w + 4 (one SIMD) differ in kh, or hold different tiles

    int vchain, within;
    if (!map_workgroup_padded(blockIdx.x, pb.count * nsplit, pb.chains * pb.segs, xcd_ids, vchain, within)) return;
    const int chain = vchain / pb.segs;
    const int seg = vchain - chain * pb.segs;
    if (SO && seg + 1 == pb.segs && !pb.need_last) return;      // nobody consumes this end state
    const int pi = within / nsplit;
    const int split = within - pi * nsplit;
    const PassArgs P = pb.p[pi];
    const int rev = P.rev;
    const float lam = pb.decay[chain % pb.H];

    // the segment's tokens [seg_start, seg_start + N) of the pass's (possibly reversed) token
    // axis are rows [row0, row0 + N) of the tensors
    const long long seg_start = (long long)seg * pb.seg_len;
    const long long N = (pb.segs > 1 && pb.N - seg_start > pb.seg_len) ? pb.seg_len : pb.N - seg_start;
    const size_t row0 = (size_t)chain * (size_t)pb.N + (size_t)(rev ? (pb.N - seg_start - N) : seg_start);
    const float* Ap = (const float*)P.a + row0 * D;
    const float* Bp = (const float*)P.b + row0 * D;
    const float* Cp = (const float*)P.c + row0 * DC + (size_t)split * DV;
    float* Op = P.out ? (float*)P.out + row0 * DC + (size_t)split * DV : nullptr;
    const float* Up = GATED ? (const float*)P.gate + row0 * DC : nullptr;
    float* Yp = GATED ? (float*)P.gated_out + row0 * DC : nullptr;
    const size_t state_off = (size_t)chain * D * DC + (size_t)split * DV;
    float* rows = P.seg_rows ? P.seg_rows + row0 * DC + (size_t)split * DV : nullptr;
    const float* sin_p = SO ? nullptr : (rows ? rows : (P.state_in ? P.state_in + state_off : nullptr));
    float* sout_p = SO ? rows : (P.state_out ? P.state_out + state_off : nullptr);

    for (int n = tid; n <= B; n += C::THREADS) pw[n] = decay_pow(lam, n);

    // running state: st[q GR + t][j] = S[state_row(q, t, j)][16ct + i16]
    auto state_row = [&](int q, int t, int j) { return 16 * (kh * MR + q * GR) + GR * (4 * g + j) + t; };
    v4f st[MR];
#pragma unroll
    for (int mt = 0; mt < MR; ++mt) st[mt] = v4f{0.f, 0.f, 0.f, 0.f};
    if (sin_p) {
#pragma unroll
        for (int mt = 0; mt < MR; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) st[mt][j] = sin_p[(size_t)state_row(mt / GR, mt % GR, j) * DC + 16 * ct + i16];
    }

    v4f ra[SO ? 1 : C::LA], rb[C::LA], rc[C::LC];
    // A block's rows are addressed from the lowest of them, a wave-uniform base, with 32-bit lane
    // offsets that are the same for every full block.  Rows past the end of a short last block
    // re-read its last row (every address stays inside the segment) and are cleared in LDS.
    const int T = (int)((N + B - 1) / B), tail = (int)(N - (long long)(T - 1) * B);
    auto row_at = [&](int r, int len) { return rev ? len - 1 - r : r; };
    auto first_low = [&](int len) { return rev ? N - len : 0; };
    auto at = [](const float* base, unsigned bytes) { return (const v4f*)((const char*)base + bytes); };
    const int dir = rev ? -B : B;          // from one block's lowest row to the next one's
    const float *pa, *pb_, *pc;            // the block to fetch
    unsigned oa[C::LA], oc[C::LC];
    auto set_offsets = [&](int len) {
#pragma unroll
        for (int i = 0; i < C::LA; ++i) {
            const int e = min(tid + i * C::THREADS, C::EA - 1);
            oa[i] = (row_at(min(e / (D / 4), len - 1), len) * D + 4 * (e % (D / 4))) * 4;
        }
#pragma unroll
        for (int i = 0; i < C::LC; ++i) {
            const int e = min(tid + i * C::THREADS, C::EC - 1);
            oc[i] = (row_at(min(e / (DV / 4), len - 1), len) * DC + 4 * (e % (DV / 4))) * 4;
        }
    };
    // One load site, reached by every block (past the end it re-reads the last block): loads on two
    // paths, or on one that may be skipped, meet in register copies that wait for them at once.
    auto fetch = [&]() {
#pragma unroll
        for (int i = 0; i < C::LA; ++i) {
            if constexpr (!SO) ra[i] = *at(pa, oa[i]);
            rb[i] = *at(pb_, oa[i]);
        }
#pragma unroll
        for (int i = 0; i < C::LC; ++i) rc[i] = *at(pc, oc[i]);
    };
    auto advance = [&](int b) {            // make b the block to fetch
        if (b >= T) return;
        pa += dir * D;
        pb_ += dir * D;
        pc += dir * DC;
        if (b == T - 1 && tail != B) {
            asm volatile("" ::: "memory"); // a branch, not a dozen selects in every block
            set_offsets(tail);
            if (rev) {
                pa += (B - tail) * D;
                pb_ += (B - tail) * D;
                pc += (B - tail) * DC;
            }
        }
    };
    auto commit = [&](float* stage) {
#pragma unroll
        for (int i = 0; i < C::LA; ++i) {
            const int e = tid + i * C::THREADS, r = e / (D / 4), c4 = e % (D / 4);
            if (C::EA % C::THREADS == 0 || e < C::EA) {
                if constexpr (!SO) *(v4f*)&stage[C::A_OFF + r * PA + 4 * c4] = ra[i];
                *(v4f*)&stage[C::B_OFF + r * PA + 4 * c4] = rb[i];
            }
        }
#pragma unroll
        for (int i = 0; i < C::LC; ++i) {
            const int e = tid + i * C::THREADS, r = e / (DV / 4), c4 = e % (DV / 4);
            if (C::EC % C::THREADS == 0 || e < C::EC) *(v4f*)&stage[C::C_OFF + r * PC + 4 * c4] = rc[i];
        }
    };
    // Rows past the end of a short last block, cleared by the threads that have just stored them: a
    // zero decay factor times an infinity of the row they repeat would be NaN in the state and in
    // that row's own output.  (Of A they reach only outputs that are not stored.)
    auto clear_tail = [&](float* stage) {
        const v4f z = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < C::LA; ++i) {
            const int e = tid + i * C::THREADS, r = e / (D / 4), c4 = e % (D / 4);
            if (e < C::EA && r >= tail) *(v4f*)&stage[C::B_OFF + r * PA + 4 * c4] = z;
        }
#pragma unroll
        for (int i = 0; i < C::LC; ++i) {
            const int e = tid + i * C::THREADS, r = e / (DV / 4), c4 = e % (DV / 4);
            if (e < C::EC && r >= tail) *(v4f*)&stage[C::C_OFF + r * PC + 4 * c4] = z;
        }
    };

    {
        const int len0 = T == 1 ? tail : B;
        set_offsets(len0);
        pa = Ap + first_low(len0) * D;
        pb_ = Bp + first_low(len0) * D;
        pc = Cp + first_low(len0) * DC;
    }
    fetch();
    commit(smem);
    if (T == 1 && tail != B) clear_tail(smem);
    advance(1);
    __syncthreads();

    float w[TS][4];                        // lambda^(len-1-key), zero from the block's end on
    float lam_len = pw[B];
    auto set_len = [&](int len) {
#pragma unroll
        for (int q = 0; q < TS; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int key = 16 * q + 4 * g + j;
                const float v = pw[max(len - 1 - key, 0)];
                w[q][j] = key < len ? v : 0.0f;
            }
        lam_len = pw[len];
    };
    set_len(B);

    // score units of this wave (causal tile: key tile kt <= token strip s; feature range ks): operand
    // and result offsets, and the decay factors of the lane's four entries
    constexpr int UNITS = C::TRI * KS, UPW = (UNITS + NW - 1) / NW, KC = D / 16 / KS;
    int ua[UPW], ub[UPW], up[UPW], ue[UPW];
    v4f um[UPW];
    float qscale[TS];
    unsigned oo[TS];                       // byte offsets of this lane's output pieces in a full block
    if constexpr (!SO) {
#pragma unroll
        for (int n = 0; n < UPW; ++n) {
            const int u = min(wave + n * NW, UNITS - 1), tile = u / KS, ks = u % KS;
            int s = 0;
            while ((s + 1) * (s + 2) / 2 <= tile) ++s;
            const int kt = tile - s * (s + 1) / 2;
            ua[n] = C::A_OFF + (16 * s + i16) * PA + 16 * KC * ks + 4 * g;
            ub[n] = C::B_OFF + (16 * kt + i16) * PA + 16 * KC * ks + 4 * g;
            up[n] = C::P_OFF + (ks * B + 16 * s + i16) * PP + 16 * kt + 4 * g;
            ue[n] = 16 * (s - kt) + i16 - 4 * g;                   // token - key at j = 0
#pragma unroll
            for (int j = 0; j < 4; ++j) um[n][j] = pw[max(ue[n] - j, 0)];
        }
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            qscale[s] = pw[16 * s + i16 + 1];
            oo[s] = (row_at(16 * s + i16, B) * DC + 16 * ct + 4 * g) * 4;
        }
    }

    // What a block leaves for the next step: its C values, the strips of S^T A^T this wave owns, where
    // its rows go, and (gated) the gate values of its rows.
    float cv[2][TS][4];                    // C[key 16q + 4g + j][16ct + i16]
    v4f oe[2][SO ? 1 : TS];
    v4f uq[GATED ? TS : 1];

    // Output of block i (S^T A^T in oe[i & 1], rows at `low`): adds the other waves' parts and C^T P^T.
    auto finish = [&](v4f (&o)[SO ? 1 : TS], const float (&c)[TS][4], int odd, long long low, int len) {
        if constexpr (!SO) {
            const float* pp = smem + C::P_OFF + odd * C::P_SIZE;
            const float* xp = smem + C::X_OFF + odd * C::X_SIZE;
#pragma unroll
            for (int s = 0; s < TS; ++s) {
                if (KH > 1 && s % KH != kh) continue;
                if constexpr (KH > 1) {
#pragma unroll
                    for (int x = 0; x < KH - 1; ++x) o[s] += *(const v4f*)&xp[((ct * TS + s) * (KH - 1) + x) * C::X_ONE + 4 * lane];
                }
                o[s] *= qscale[s];
#pragma unroll
                for (int kt = 0; kt <= s; ++kt) {
                    v4f p4 = *(const v4f*)&pp[(16 * s + i16) * PP + 16 * kt + 4 * g];
#pragma unroll
                    for (int ks = 1; ks < KS; ++ks) p4 += *(const v4f*)&pp[(ks * B + 16 * s + i16) * PP + 16 * kt + 4 * g];
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[s] = mfma4(c[kt][j], p4[j], o[s]);
                }
                if constexpr (GATED) {     // this tile's share of the token's sum of squares
                    float ss = o[s][0] * o[s][0] + o[s][1] * o[s][1] + o[s][2] * o[s][2] + o[s][3] * o[s][3];
                    ss += __shfl_xor(ss, 16, 64);
                    ss += __shfl_xor(ss, 32, 64);
                    if (g == 0) smem[C::Q_OFF + odd * C::Q_SIZE + ct * B + 16 * s + i16] = ss;
                    uq[s] = *at(Up + low, oo[s]);
                }
                if (Op && (len == B || 16 * s + i16 < len)) *(v4f*)((char*)(Op + low) + oo[s]) = o[s];
            }
        }
    };
    // Gated output of a finished block, one barrier later: every wave's share of the row norms is there.
    auto gate = [&](const v4f (&o)[SO ? 1 : TS], int odd, long long low, int len) {
        if constexpr (GATED) {
#pragma unroll
            for (int s = 0; s < TS; ++s) {
                if (KH > 1 && s % KH != kh) continue;
                float ss = 0.0f;
#pragma unroll
                for (int n = 0; n < NT; ++n) ss += smem[C::Q_OFF + odd * C::Q_SIZE + n * B + 16 * s + i16];
                const float rstd = 1.0f / sqrtf(ss * (1.0f / DC) + P.eps);
                if (len == B || 16 * s + i16 < len) *(v4f*)((char*)(Yp + low) + oo[s]) = o[s] * rstd * uq[s];
            }
        }
    };

    const long long ostep = (long long)dir * DC;
    long long low = first_low(T == 1 ? tail : B) * DC;    // elements to the lowest row of the block to finish next
    auto step = [&](int i, auto odd_c) {
        constexpr int odd = decltype(odd_c)::value;
        const bool more = i + 1 < T;
        const float* stage = smem + odd * C::STAGE;
        fetch();
        advance(i + 2);
        if (!more && tail != B) set_len(tail);
        if constexpr (GATED) if (i >= 2) gate(oe[odd], odd, low - ostep, B);

#pragma unroll
        for (int q = 0; q < TS; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) cv[odd][q][j] = stage[C::C_OFF + (16 * q + 4 * g + j) * PC + 16 * ct + i16];
        if constexpr (!SO) {
            // -------- masked score tiles, and S^T A^T with the state of the block's start
#pragma unroll
            for (int n = 0; n < UPW; ++n) {
                if (UNITS % NW != 0 && n == UPW - 1 && wave + n * NW >= UNITS) break;
                v4f p0 = v4f{0.f, 0.f, 0.f, 0.f}, p1 = p0;
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    const v4f a4 = *(const v4f*)&stage[ua[n] + 16 * c], b4 = *(const v4f*)&stage[ub[n] + 16 * c];
                    p0 = mfma4(b4[0], a4[0], p0);
                    p1 = mfma4(b4[1], a4[1], p1);
                    p0 = mfma4(b4[2], a4[2], p0);
                    p1 = mfma4(b4[3], a4[3], p1);
                }
                p0 = (p0 + p1) * um[n];
                // a select, not a zero factor: an infinite score with a later key stays masked
#pragma unroll
                for (int j = 0; j < 4; ++j) p0[j] = ue[n] >= j ? p0[j] : 0.0f;
                *(v4f*)&smem[up[n] + odd * C::P_SIZE] = p0;
            }
#pragma unroll
            for (int s = 0; s < TS; ++s) oe[odd][s] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < MR; ++c)
#pragma unroll
                for (int s = 0; s < TS; ++s) {
                    // features 4x .. 4x+3 of this lane's 4 GR of the group (x = c % GR): j = y / GR, t = y % GR, y = 4x + i
                    const int x = c % GR;
                    const v4f a4 = *(const v4f*)&stage[C::A_OFF + (16 * s + i16) * PA + 16 * (kh * MR + c - x) + 4 * GR * g + 4 * x];
#pragma unroll
                    for (int y = 0; y < 4; ++y) oe[odd][s] = mfma4(st[c - x + (4 * x + y) % GR][(4 * x + y) / GR], a4[y], oe[odd][s]);
                }
            if constexpr (KH > 1) {
#pragma unroll
                for (int s = 0; s < TS; ++s) {
                    const int own = s % KH;                        // the wave (ct, own) finishes strip s
                    if (kh != own) {
                        const int slot = kh < own ? kh : kh - 1;
                        *(v4f*)&smem[C::X_OFF + odd * C::X_SIZE + ((ct * TS + s) * (KH - 1) + slot) * C::X_ONE + 4 * lane] = oe[odd][s];
                    }
                }
            }
            if (i > 0) {
                finish(oe[odd ^ 1], cv[odd ^ 1], odd ^ 1, low, B);
                low += ostep;
            }
        }
        if (more || sout_p) {
#pragma unroll
            for (int mt = 0; mt < MR; ++mt) st[mt] *= lam_len;
            // B^T values of the next key step are read while the current one's MFMAs run
            vg bv[2][MR / GR];
            const float* bp = stage + C::B_OFF + 4 * g * PA + 16 * kh * MR + GR * i16;
            auto load_b = [&](vg (&x)[MR / GR], int key) {
#pragma unroll
                for (int q = 0; q < MR / GR; ++q) x[q] = *(const vg*)&bp[(16 * (key / 4) + key % 4) * PA + 16 * GR * q];
            };
            load_b(bv[0], 0);
            __builtin_amdgcn_sched_group_barrier(0x100, MR / GR, 0);
#pragma unroll
            for (int key = 0; key < 4 * TS; ++key) {
                if (key + 1 < 4 * TS) load_b(bv[(key + 1) & 1], key + 1);
                const float cw = cv[odd][key / 4][key % 4] * w[key / 4][key % 4];
#pragma unroll
                for (int mt = 0; mt < MR; ++mt) st[mt] = mfma4(bv[key & 1][mt / GR][mt % GR], cw, st[mt]);
                if (key + 1 < 4 * TS) __builtin_amdgcn_sched_group_barrier(0x100, MR / GR, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, MR, 0);
            }
        }
        if (more) {
            commit(smem + (odd ^ 1) * C::STAGE);
            if (i + 2 == T && tail != B) clear_tail(smem + (odd ^ 1) * C::STAGE);
        }
        __syncthreads();
    };
    for (int i = 0; i < T; i += 2) {
        step(i, std::integral_constant<int, 0>{});
        if (i + 1 < T) step(i + 1, std::integral_constant<int, 1>{});
    }
    if constexpr (!SO) {                   // the last block's output
        auto last = [&](auto odd_c) {
            constexpr int odd = decltype(odd_c)::value;
            if constexpr (GATED) if (T >= 2) gate(oe[odd ^ 1], odd ^ 1, low - ostep, B);
            if (tail != B) {
                if (rev && T > 1) low += (B - tail) * DC;
#pragma unroll
                for (int s = 0; s < TS; ++s) oo[s] = (row_at(min(16 * s + i16, tail - 1), tail) * DC + 16 * ct + 4 * g) * 4;
            }
            finish(oe[odd], cv[odd], odd, low, tail);
            if constexpr (GATED) {
                __syncthreads();
                gate(oe[odd], odd, low, tail);
            }
        };
        if (T & 1) last(std::integral_constant<int, 0>{});
        else last(std::integral_constant<int, 1>{});
    }

    if (sout_p) {
#pragma unroll
        for (int mt = 0; mt < MR; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                sout_p[(size_t)state_row(mt / GR, mt % GR, j) * DC + 16 * ct + i16] = st[mt][j];
    }
}

template <int D, int DV, int B, int KH, int DC, int MODE>
hipError_t launch_t(const PassBatch& pb, hipStream_t stream) {
    static_assert(DC % DV == 0, "value-column slices tile the C operand");
    const int nsplit = DC / DV;
    const long long nch = (long long)pb.chains * pb.segs;
    const int per_chain = pb.count * nsplit;
    const long long wgs = launch_chain_slots(nch, per_chain) * per_chain;
    if (wgs <= 0 || wgs > 0x7fffffffLL || pb.segs < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((pass_f32_kernel<D, DV, B, KH, DC, MODE>), dim3((unsigned)wgs), dim3(FCfg<D, DV, B, KH>::THREADS), 0,
                       stream, pb, nsplit, (int)xcd_ids_fit(nch, per_chain));
    return hipGetLastError();
}

// States at the segments' starts, in place in the first D rows of each segment's output rows
// (layout of PassArgs::seg_rows): with L[g] the end state of segment g from a zero start,
//     S[0] = initial state,     S[g+1] = lambda^len(g) S[g] + L[g].
// One thread per four columns of a state row; the end states of eight segments are read at a
// time, ahead of the chain of multiply-adds over them.
struct ScanArgs { float* rows[3]; int rev[3]; };

__global__ __launch_bounds__(256)
void segment_scan_rows_kernel(const ScanArgs s, const float* __restrict__ kv_in, float* __restrict__ kv_out,
                              const float* __restrict__ decay, int count, int chains, int H, int segs,
                              long long seg_len, long long N, int D, int DC) {
    const int q = DC / 4, per = D * q;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long long)count * chains * per) return;
    const int e = (int)(idx % per), row = e / q, c4 = e % q;
    const long long pc = idx / per;
    const int chain = (int)(pc % chains), pass = (int)(pc / chains);
    const int rev = s.rev[pass];
    const float lam = decay[chain % H], lam_full = decay_pow(lam, (int)seg_len);
    float* base = s.rows[pass] + (size_t)chain * N * DC + (size_t)row * DC + 4 * c4;
    const long long last_n = N - (long long)(segs - 1) * seg_len;
    auto at = [&](int g) -> v4f* {
        const long long start = (long long)g * seg_len, n = g + 1 == segs ? last_n : seg_len;
        return (v4f*)(base + (size_t)(rev ? N - start - n : start) * DC);
    };
    const bool final_state = pass == 0 && kv_out;
    const size_t so = ((size_t)chain * D + row) * DC + 4 * c4;
    v4f run = (pass == 0 && kv_in) ? *(const v4f*)(kv_in + so) : v4f{0.f, 0.f, 0.f, 0.f};
    for (int g0 = 0; g0 < segs; g0 += 8) {
        v4f l[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            l[i] = (g0 + i + 1 < segs || (g0 + i + 1 == segs && final_state)) ? *at(g0 + i) : v4f{0.f, 0.f, 0.f, 0.f};
        // keep_inf as in the bf16 passes' scan
        auto walk = [&](auto keep_inf) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int g = g0 + i;
                if (g < segs) {
                    *at(g) = run;
                    const float f = g + 1 < segs ? lam_full : decay_pow(lam, (int)last_n);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        run[j] = run[j] * (decltype(keep_inf)::value && __builtin_isinf(run[j]) ? 1.f : f) + l[i][j];
                }
            }
        };
        if (lam > 0.f && lam_full == 0.f) walk(std::true_type{});
        else walk(std::false_type{});
    }
    if (final_state) *(v4f*)(kv_out + so) = run;
}

__global__ void state_copy_kernel(const float* __restrict__ in, float* __restrict__ out, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) out[i] = in ? in[i] : 0.0f;
}

}  // namespace

// (D, DC, value columns per workgroup, block length, KH) of the plain pass.
#define LTN_F32_SLICES(X)                                                                          \
    X(64, 64, 64, 32, 2) X(64, 64, 32, 32, 4) X(64, 64, 64, 16, 2) \
    X(96, 96, 96, 32, 2) X(96, 96, 32, 32, 2) X(96, 96, 32, 16, 2)                                 \
    X(128, 128, 128, 32, 1) X(128, 128, 64, 32, 2) X(128, 128, 32, 32, 4) X(128, 128, 64, 16, 2)   \
    X(256, 256, 128, 16, 1) X(256, 256, 64, 16, 2) X(256, 256, 32, 16, 4)                          \
    X(256, 128, 128, 16, 1) X(256, 128, 64, 16, 2) X(256, 128, 32, 16, 4)                          \
    X(128, 256, 128, 16, 1) X(128, 256, 64, 16, 2) X(128, 256, 32, 16, 4)                          \
    X(128, 64, 64, 32, 2) X(128, 64, 32, 32, 4) X(128, 64, 64, 16, 2)                              \
    X(64, 128, 128, 32, 1) X(64, 128, 64, 32, 2) X(64, 128, 32, 32, 4) X(64, 128, 64, 16, 2)

bool f32_has_slice(int D, int DC, int dv, int block) {
#define LTN_F32_HAS(d, c, v, b, kh) if (D == d && DC == c && dv == v && block == b) return true;
    LTN_F32_SLICES(LTN_F32_HAS)
#undef LTN_F32_HAS
    return false;
}

hipError_t launch_pass_f32(const PassBatch& pb, int D, int dv, int block, hipStream_t stream, int DC) {
    if (DC == 0) DC = D;
    const bool gated = pb.p[0].gate != nullptr;
    for (int i = 0; i < pb.count; ++i)
        if (!(pb.state_only ? (const void*)pb.p[i].seg_rows : pb.p[i].out) && !gated) return hipErrorInvalidValue;
    if (gated && (pb.count != 1 || dv != DC || !pb.p[0].gated_out || pb.state_only)) return hipErrorInvalidValue;
    if (pb.segs > 1)
        for (int i = 0; i < pb.count; ++i)
            if (!pb.p[i].seg_rows || pb.seg_len < D || pb.N - (pb.segs - 1) * pb.seg_len < D) return hipErrorInvalidValue;
    const int mode = pb.state_only ? kStateOnly : (gated ? kGated : kPlain);
    // 64 features, more workgroups than units: four waves without the exchange between row halves take
    // 72 KB of LDS (88 with it), so two workgroups share a unit, out of step with each other.  Backward of
    // 1024 chains x 64 tokens 71 -> 52 us, 512 x 512 201 -> 172, 128 x 2048 248 -> 219, forward of 300 x
    // 2048 247 -> 220; up to 256 workgroups a unit holds one, and its four waves would be alone there.
    if (mode == kPlain && D == 64 && DC == 64 && dv == 64 && block == 32 && (long long)pb.chains * pb.segs * pb.count > 256)
        return launch_t<64, 64, 32, 1, 64, kPlain>(pb, stream);
#define LTN_F32(m, d, c, v, b, kh) if (mode == m && D == d && DC == c && dv == v && block == b) return launch_t<d, v, b, kh, c, m>(pb, stream)
#define LTN_F32_PLAIN(d, c, v, b, kh) LTN_F32(kPlain, d, c, v, b, kh);
    LTN_F32_SLICES(LTN_F32_PLAIN)
#undef LTN_F32_PLAIN
    // gated epilogue: one pass, complete output rows
    LTN_F32(kGated, 64, 64, 64, 32, 2); LTN_F32(kGated, 64, 64, 64, 16, 2);
    LTN_F32(kGated, 128, 128, 128, 32, 1); LTN_F32(kGated, 128, 128, 128, 16, 1);
    // segment end states
    LTN_F32(kStateOnly, 64, 64, 64, 32, 2); LTN_F32(kStateOnly, 96, 96, 96, 32, 2); LTN_F32(kStateOnly, 128, 128, 128, 32, 1);
    LTN_F32(kStateOnly, 256, 256, 128, 16, 1); LTN_F32(kStateOnly, 256, 128, 128, 16, 1);
    LTN_F32(kStateOnly, 128, 256, 128, 16, 1); LTN_F32(kStateOnly, 128, 64, 64, 32, 2); LTN_F32(kStateOnly, 64, 128, 128, 32, 1);
#undef LTN_F32
    return hipErrorInvalidValue;
}

hipError_t launch_segment_scan_rows(const PassBatch& pb, const float* kv_in, float* kv_out, int D, hipStream_t stream, int DC) {
    if (DC == 0) DC = D;
    const long long total = (long long)pb.count * pb.chains * D * (DC / 4);
    if (total <= 0 || pb.segs < 1 || pb.seg_len <= 0 || pb.seg_len > 0x7fffffffLL) return hipErrorInvalidValue;
    const long long wgs = (total + 255) / 256;
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    ScanArgs s = {};
    for (int i = 0; i < pb.count; ++i) {
        s.rows[i] = pb.p[i].seg_rows;
        s.rev[i] = pb.p[i].rev;
    }
    hipLaunchKernelGGL(segment_scan_rows_kernel, dim3((unsigned)wgs), dim3(256), 0, stream, s, kv_in, kv_out, pb.decay,
                       pb.count, pb.chains, pb.H, pb.segs, pb.seg_len, pb.N, D, DC);
    return hipGetLastError();
}

hipError_t launch_state_copy(const float* kv_in, float* kv_out, size_t n, hipStream_t stream) {
    if (n == 0 || kv_in == kv_out) return hipSuccess;
    const unsigned grid = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    hipLaunchKernelGGL(state_copy_kernel, dim3(grid), dim3(256), 0, stream, kv_in, kv_out, n);
    return hipGetLastError();
}

}  // namespace ltn
