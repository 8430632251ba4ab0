// Chunked prefill for bf16 tensors, as in prefill_bf16.hip (same evaluation, same arithmetic, same operand layouts), with the work of a
// chunk in stages that run side by side on different waves of the workgroup, one barrier per chunk:
//   conv waves      raw x -> X (LDS, [channel][token]);
//   weight waves    dt's prefix sums and the weights (a further chunk ahead), the weighted B (head and tail, transposed), M^T;
//   consumer waves  own the state (accumulator registers, as there): h C^T, M X, the update, the gate and the outputs, of the chunk that
//                   the others prepared in the step before.
// Nothing that the first two do depends on the state.  In the other kernel a wave does all of it in turn, with three barriers: that keeps a
// compute unit busy if two to four workgroups share it, but one that is alone takes 1.9 us per chunk (128 x 64), 1.0-1.2 here, three
// waves per SIMD of one workgroup filling each other's waits.  The step is bound by the chain of a stage: LDS round trips, conversions,
// dependent products (weight waves alone 0.9 us, consumers alone 0.9, 0.2 for an empty step).
// Each stage requests everything it reads from LDS at the top of its step: left in place, a read would queue up behind the stores of the
// part before it, which the compiler cannot tell apart from it.  Raw inputs come straight into LDS, DIST chunks ahead, and are waited
// for by count.  Outputs leave a step late, as whole rows of the head.
// Who shares a SIMD with whom, and who goes first: wave w is on SIMD w % 4, and the stage that a step waits for is a chain of short
// instructions beside others' long ones.  Where the state is split the waves of the second half of n, which have no M X, gate and outputs, come
// first, so that they share with the conv waves (0.98 of the time at 32 x 128 and 64 x 128).  The weight waves have priority where that pays, the conv waves
// where they have a SiLU and it does.  Time over that without either, with the halves in the old order; means of 24 calls each, 16 to 210 pairs,
// 300 to 1985 tokens, one length and spread:
//             no SiLU, no gate     gate                 SiLU                             SiLU and gate
//             none  weights        none  weights        none  weights  conv  both        none  weights  conv  both
//    32 x 64  1.00  1.01           1.00  1.04           1.00  1.00     1.03  1.00        1.00  1.01     1.03  1.02
//    32 x 128 0.97  0.96           0.96  1.00           0.98  0.98     1.03  0.98        0.96  1.00     1.00  1.00
//    64 x 64  1.00  0.99           1.00  1.02           1.00  1.01     1.00  1.00        1.00  1.00     1.00  1.00
//    64 x 128 0.99  0.96           0.99  1.05           0.98  0.99     1.02  0.95        0.95  0.98     0.98  0.97
//   128 x 64  1.00  0.98           1.00  1.01           1.00  1.00     0.96  0.94        1.00  1.00     0.99  0.97
//   128 x 128 1.00  0.99           1.00  1.01           1.00  1.00     0.97  1.01        1.00  0.98     0.97  1.00
//   128 x 32  1.00  0.97           1.00  0.99           1.00  1.00     1.01  0.97        1.00  1.00     1.02  0.97
//    64 x 32  1.00  1.00           1.00  1.00           1.00  1.00     0.97  0.97        1.00  1.00     0.97  0.97
//    32 x 32  nothing does anything
// The worst of weights first with a gate was 1.12 (32 x 64, 6 x 35 pairs, 1985 tokens: 80 -> 89 us).
// Which launches are served: prefill_pipe_serves.  A split state (NSPL = 2): both waves of a tile scale their share of h C^T by exp(cum_t),
// and the second's goes to the first through LDS a step later.
#include "prefill_bf16_ops.h"
#include "prefill_split.h"

namespace ssmv {
namespace {

constexpr int kQ = kPrefillChunk;

template <int P, int N>
struct PipeLds {              // byte offsets of the LDS arrays (bf16 unless said)
    static constexpr int XS = kQ * 2 + 16;                 // row stride of the arrays indexed [..][token]
    static constexpr int NP = P / 32;                      // 32-channel tiles of the head
    static constexpr int NSPL = prefill_nsplit(P, N);
    static constexpr int NC = NP * NSPL;                   // consumer waves
    static constexpr int NWT = N >= 64 ? 4 : 2;            // weight waves
    static constexpr int NCV = P / 32;                     // conv waves
    static constexpr int NW = NC + NWT + NCV;
    // chunks that raw inputs are requested ahead of their use: one where two of them take the LDS of a further workgroup (64 x 64) or
    // more than there is (128 x 128)
    static constexpr int DIST = (P >= 128 && N >= 128) || (P == 64 && N == 64) ? 1 : 2;
    static constexpr int XB = DIST + 1, CB = DIST + 2;     // copies of the raw x and B, of C (the consumers read it, a chunk later)
    static constexpr int PX = P * XS, PB = N * XS, PM = kQ * XS;
    static constexpr int oX = 0;                           // [2][P][Q]  conv output x_s
    static constexpr int oBh = oX + 2 * PX;                // [2][N][Q]  head of w_s B_s, transposed
    static constexpr int oBl = oBh + 2 * PB;               // [2][N][Q]  tail of w_s B_s, transposed
    static constexpr int oM = oBl + 2 * PB;                // [2][Q][Q]  M^T, rows t
    static constexpr int YS = 32 * 2 + 16;                 // row stride of an output tile [token][32 channels]
    static constexpr int YT = kQ * YS + 64;                // stride of the tiles: a row of all tiles then covers the banks
    static constexpr int oY = oM + 2 * PM;                 // [2][NP][Q][32]  the output tiles
    static constexpr int oZ = oY + 2 * NP * YT;            // fp32 [2][NP][16][64]  h C^T over the second half of n, for the tile's first wave
    static constexpr int PXR = kQ * P * 2, PBC = kQ * N * 2;
    static constexpr int oXraw = oZ + (NSPL - 1) * 2 * NP * 4096;   // [XB][Q][P]  raw conv inputs, pieces swizzled
    static constexpr int oB = oXraw + XB * PXR;            // [XB][Q][N]
    static constexpr int oC = oB + XB * PBC;               // [CB][Q][N]
    static constexpr int oDtr = oC + CB * PBC;             // [4][64] raw dt, a word each (tokens twice)
    static constexpr int oCar = oDtr + 4 * 256;     // [2][P][4]  the last four raw inputs of a chunk, for the next one's conv
    static constexpr int oCum = oCar + 2 * P * 8;          // fp32 [NWT][2][Q]  log2 e times the inclusive prefix of dt*A (a copy per wave)
    static constexpr int oDt = oCum + NWT * 2 * kQ * 4;    // fp32 [NWT][2][Q]  dt
    static constexpr int oW = oDt + NWT * 2 * kQ * 4;      // fp32 [NWT][2][Q]  exp(cum_Q - cum_s) dt_s
    static constexpr int oAt = oW + NWT * 2 * kQ * 4;      // fp32 [4][Q]  exp(cum_t), for the consumers
    static constexpr int total = oAt + 4 * kQ * 4;
    // Workgroups that fit a compute unit by their LDS, and the waves per SIMD that the registers have to leave room for then.  The fullest SIMD
    // counts: a workgroup of six waves puts two on the same ones as the next does (32 x 64 with registers for three waves, which would do if
    // they were dealt out evenly, 512 workgroups, 1024 tokens: 46 -> 61 us).  32 x 64, 64 x 64 and 64 x 128 spill 1 to 4 registers for
    // it, outside the chunk loop.
    static constexpr int fit = 160 * 1024 / total;
    static constexpr int WPE = fit * ((NW + 3) / 4);
};

template <int P, int N, bool SEG>
__global__ __launch_bounds__((64 * PipeLds<P, N>::NW)) __attribute__((amdgpu_waves_per_eu((PipeLds<P, N>::WPE))))
void prefill_pipe_kernel(const PrefillParams p)
{
    using Ld = PipeLds<P, N>;
    constexpr int Q = kQ, W = SSMV_CONV_WIDTH, NSPL = Ld::NSPL, NC = Ld::NC, NWT = Ld::NWT, NCV = Ld::NCV, NP = Ld::NP, DIST = Ld::DIST, XB = Ld::XB, CB = Ld::CB;
    constexpr int TN = N / 32, TNL = TN / NSPL;          // state tiles of the head, of a consumer wave
    constexpr int QS = Q * P / (64 * NCV);               // consecutive tokens a conv thread takes per chunk
    constexpr int XS = Ld::XS, PIECES = N / 8;
    static_assert(P % 32 == 0 && P <= 128 && N % 32 == 0 && W == 4 && QS % 8 == 0, "tile shapes");

    extern __shared__ float4 lds_raw[];
    char *lds = reinterpret_cast<char *>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int li = lane & 31, lh = lane >> 5;            // MFMA: row/column index and k half of this lane
    const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
    SSMV_TRACE_BEGIN();
    const int H = p.H, G = p.G;
    const PrefillItem item = prefill_item<SEG>(p);
    const int hd = item.hd, b = item.b;
    const int Ls = p.L;                                  // token stride of the arrays
    const int L = item.L;                                // this sequence's prompt length
    if (L == 0) return;                                  // nothing to feed: state, ring and outputs stay as they are
    Segment seg = {0, (L + Q - 1) / Q, 0, true, true, true};
    if constexpr (SEG) {
        seg = segment_of(p, L, item.slot);
        if (!seg.work) return;
    }
    const int c_beg = SEG ? seg.c0 : 0, c_end = seg.c1;  // the chunks of this workgroup
    const bool emit = !SEG || seg.emit;                  // whether it writes outputs
    const int HP = H * P, GN = G * N;
    const int g = hd / (H / G);
    const int mask = p.ring_len - 1;
    // an element offset from a sequence's (or chunk's) first row, in bytes; and a chunk's first row (uniform)
    auto off = [](int token, int stride, int rest) { return 2u * (__umul24(token, stride) + (unsigned)rest); };
    auto chunk_of = [](const void *base, int c, int stride) { return static_cast<const char *>(base) + (size_t)c * Q * stride * 2; };
    char *y_b = reinterpret_cast<char *>(p.y) + (size_t)b * Ls * HP * 2;

    int xb = 0, xi = DIST % XB;                          // copies of the raw inputs: of the chunk, of the one to request
    if (wave_u >= NC + NWT) {
        // =================================================== conv waves ==================================================
        const int pw = wave_u - NC - NWT, ptid = tid - 64 * (NC + NWT);
        // (the last pass of a segmented prompt runs behind the launch that has moved conv_head on already)
        const int conv_head = (p.conv_head[b] - (SEG && p.seg_pass == 1 ? L : 0)) & mask;
        const bool silu = p.conv_act == SSMV_ACT_SILU;
        uint2 *sCar = reinterpret_cast<uint2 *>(lds + Ld::oCar);
        const uint16_t *x_b = reinterpret_cast<const uint16_t *>(p.x_raw) + (size_t)b * Ls * HP;
        constexpr int LR = P / 8;                        // lanes per row of x, 64 / LR rows per instruction, P / 16 instructions
        constexpr int XPW = (P / 16) / NCV;              // of them per wave
        uint32_t ox[XPW];
        auto lane_offsets = [&](int last) {              // last: the chunk's last row that is there
#pragma unroll
            for (int k = 0; k < XPW; ++k) {
                const int row = (pw + k * NCV) * (64 / LR) + lane / LR;
                ox[k] = off(min(row, last), HP, hd * P + ((lane % LR) ^ key_x<P>(row)) * 8);
            }
        };
        lane_offsets(Q - 1);
        auto issue = [&](int c, int to) {
            if (c * Q + Q > L) lane_offsets(L - 1 - c * Q);
            const char *xc = chunk_of(x_b, c, HP);
#pragma unroll
            for (int k = 0; k < XPW; ++k) load_to_lds16(xc, ox[k], lds + Ld::oXraw + to * Ld::PXR + (pw + k * NCV) * 1024);
        };
        issue(c_beg, 0);
        if (DIST > 1 && c_beg + 1 < c_end) issue(c_beg + 1, 1);
        const int pc = ptid % P;                         // this thread's channel, and the first of its tokens
        const int s0 = (P >= 64 ? __builtin_amdgcn_readfirstlane(ptid / P) : ptid / P) * QS;
        const unsigned ch = hd * P + pc;
        uint2 wraw = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(p.wgt) + (size_t)ch * W);
        float cbias = p.bias ? load_io(p.bias, ch, SSMV_BF16) : 0.f;
        auto raw_bits = [&](int tg) { return (uint32_t)(x_b + (size_t)min(max(tg, 0), L - 1) * HP)[ch]; };
        if (ptid < P) {                                  // the W-1 raw inputs ahead of the first chunk (newest last)
            uint32_t hist[W - 1];
#pragma unroll
            for (int j = 0; j < W - 1; ++j) {
                if (SEG && c_beg > 0) hist[j] = raw_bits(c_beg * Q - (W - 1) + j);
                else hist[j] = reinterpret_cast<const uint16_t *>(p.ring)[((size_t)b * p.ring_len + ((conv_head + 1 - (W - 1) + j) & mask)) * HP + ch];
            }
            sCar[((c_beg + 1) & 1) * P + pc] = make_uint2(hist[0] << 16, hist[1] | (hist[2] << 16));
        }
        // transposing reads (read_tr16): lane j of 16 is in row j / 4 of four, 8 bytes j % 4 of the 32 of its 16 channels
        const int trow = (lane & 15) >> 2, tpiece = (lane >> 1) & 1, tbyte = (lane & 1) * 8;
        const char *xtr = lds + Ld::oXraw + trow * (2 * P) + ((((pc >> 4) * 2 + tpiece) ^ key_x<P>(trow)) * 16) + tbyte;
        // every value loaded so far is here before the loop: the compiler would wait for it at its first use in there, for all loads
        // under way, the direct ones for the chunks to come among them
        asm volatile("" : "+v"(wraw.x), "+v"(wraw.y), "+v"(cbias));
        auto wait_next = [&](bool newer) {               // the next chunk's rows have landed; `newer`: a further chunk's may be under way
            if (DIST > 1 && newer) wait_direct_loads_but<XPW>();
            else wait_direct_loads();
        };
        wait_next(c_beg + 1 < c_end);
        __syncthreads();
        // (in the head of this file.  Not ahead of the first loads: a branch there waits for conv_head)
        if (silu && !(P == 32 && N >= 64) && !(P == 64 && (N == 64 || (N == 128 && p.z)))) __builtin_amdgcn_s_setprio(2);
        for (int c = c_beg; c < c_end; ++c) {
            const bool more = c + DIST < c_end;
            if (more) issue(c + DIST, xi);
            // raw x as packed pairs of adjacent tokens of this channel: e[0], e[1] the four tokens ahead of s0 (in the chunk's first tokens
            // what the chunk before left), then the thread's own; o the pairs in between
            uint32_t e[QS / 2 + 2], o[QS / 2 + 1];
            const char *xr = xtr + xb * Ld::PXR;
            uint2 ahead;
            if constexpr (P >= 64) {
                if (s0 != 0) ahead = read_tr16(xr + (s0 - 4) * (2 * P));
                else ahead = sCar[((c + 1) & 1) * P + pc];
            } else {                                     // both kinds of threads in one wave
                const uint2 here = read_tr16(xr + max(s0 - 4, 0) * (2 * P)), before = sCar[((c + 1) & 1) * P + pc];
                ahead = s0 != 0 ? here : before;
            }
            e[0] = ahead.x;
            e[1] = ahead.y;
#pragma unroll
            for (int j = 0; j < QS / 4; ++j) {
                const uint2 r = read_tr16(xr + (s0 + 4 * j) * (2 * P));
                e[2 + 2 * j] = r.x;
                e[3 + 2 * j] = r.y;
            }
            if (s0 + QS == Q) sCar[(c & 1) * P + pc] = make_uint2(e[QS / 2], e[QS / 2 + 1]);     // for the next chunk
#pragma unroll
            for (int i = 0; i < QS / 2 + 1; ++i) o[i] = __builtin_amdgcn_alignbit(e[i + 1], e[i], 16);
            char *to = lds + Ld::oX + (c & 1) * Ld::PX + pc * XS + s0 * 2;
#pragma unroll
            for (int v = 0; v < QS / 8; ++v) {
                float xv[8];
                conv8(xv, o + 4 * v, e + 1 + 4 * v, wraw.x, wraw.y, cbias);
                if (silu) conv_silu8(xv);
                // the rounding to the storage type
                *reinterpret_cast<uint4 *>(to + 16 * v) =
                    make_uint4(pack_bf16x2(xv[0], xv[1]), pack_bf16x2(xv[2], xv[3]), pack_bf16x2(xv[4], xv[5]), pack_bf16x2(xv[6], xv[7]));
            }
            wait_next(more);
            __syncthreads();
            xb = xb + 1 == XB ? 0 : xb + 1;
            xi = xi + 1 == XB ? 0 : xi + 1;
        }
        __syncthreads();
        if ((!SEG || seg.last) && ptid < P) {            // the newest W-1 raw inputs into the ring behind conv_head
            for (int tg = (L - (W - 1) > 0 ? L - (W - 1) : 0); tg < L; ++tg)
                IoVec<SSMV_BF16>::store_raw1(p.ring, ((size_t)b * p.ring_len + ((conv_head + 1 + tg) & mask)) * HP + ch, raw_bits(tg));
        }
        return;
    }
    int cb = 0, ci = DIST % CB;                          // the same of C, which the consumers read a chunk later
    if (wave_u >= NC) {
        // =================================================== weight waves ===================================================
        const int pw = wave_u - NC, ptid = tid - 64 * NC;
        const float A2_h = p.A[hd] * kLog2e, D_h = p.D[hd];
        float dtb_h = p.dt_bias ? p.dt_bias[hd] : 0.f;
        float *sCum = reinterpret_cast<float *>(lds + Ld::oCum) + pw * 2 * Q;
        float *sDt = reinterpret_cast<float *>(lds + Ld::oDt) + pw * 2 * Q;
        float *sW = reinterpret_cast<float *>(lds + Ld::oW) + pw * 2 * Q;
        float *sAt = reinterpret_cast<float *>(lds + Ld::oAt);
        const char *sDtr = lds + Ld::oDtr;
        const uint16_t *B_b = reinterpret_cast<const uint16_t *>(p.Bm) + (size_t)b * Ls * GN + (size_t)g * N;
        const uint16_t *C_b = reinterpret_cast<const uint16_t *>(p.Cm) + (size_t)b * Ls * GN + (size_t)g * N;
        const uint16_t *dt_b = reinterpret_cast<const uint16_t *>(p.dt) + (size_t)b * Ls * H + hd;

        // ---- raw inputs, straight into LDS (1 KB per wave and instruction), DIST chunks ahead.  Every address is the chunk's
        // first row (uniform) plus a lane offset that stays the same over the chunks; a last chunk that is not full reads its last
        // token again for the rows behind it (they carry dt = 0 and thereby weight 0 everywhere) -------------------------------
        constexpr int BT = N / 16;                       // instructions for the 32 rows of B, and as many for C
        constexpr int BPW = BT / NWT;
        static_assert(BT % NWT == 0, "loads per wave");
        uint32_t obc[BPW];
        auto lane_offsets = [&](int last) {              // last: the chunk's last row that is there
#pragma unroll
            for (int k = 0; k < BPW; ++k) {
                const int row = ((pw + k * NWT) % BT) * (64 / PIECES) + lane / PIECES;
                obc[k] = off(min(row, last), GN, ((lane % PIECES) ^ key_bc<N>(row)) * 8);
            }
        };
        lane_offsets(Q - 1);
        constexpr int kLoads = 2 * BPW, kLoadsState = BPW;      // of a wave and chunk, at least (dt ahead of them); without outputs
        // dt of a chunk comes with the rows of the one before it: its decay factors are worked out a step ahead of the rest
        auto issue_dt = [&](int c) { if (pw == 0) load_to_lds2(dt_b, off(min(c * Q + li, L - 1), H, 0), sDtr + (c & 3) * 256); };
        auto issue = [&](int c, int tob, int toc) {      // which copies
            if (c * Q + Q > L) lane_offsets(L - 1 - c * Q);
            const char *Bc = chunk_of(B_b, c, GN), *Cc = chunk_of(C_b, c, GN);
            char *dB = lds + Ld::oB + tob * Ld::PBC, *dC = lds + Ld::oC + toc * Ld::PBC;
            issue_dt(c + 1);
#pragma unroll
            for (int k = 0; k < BPW; ++k) {
                const int idx = (pw + k * NWT) % BT;
                load_to_lds16(Bc, obc[k], dB + idx * 1024);
                if (emit) load_to_lds16(Cc, obc[k], dC + idx * 1024);
            }
        };
        issue_dt(c_beg);
        issue(c_beg, 0, 0);
        if (DIST > 1 && c_beg + 1 < c_end) issue(c_beg + 1, 1, 1);

        // ---- what stays over the chunks ----
        const int l16 = lane & 15, k4 = lane >> 4;
        float dadd[4];
        bool keep[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            keep[v] = 4 * k4 + v <= l16;
            dadd[v] = 4 * k4 + v == l16 ? D_h : 0.f;
        }
        // the quadrant t < 16 <= s of both copies of M^T stays zero
        if (ptid < 64) *reinterpret_cast<uint4 *>(lds + Ld::oM + (ptid >> 5) * Ld::PM + ((ptid & 31) >> 1) * XS + 32 + (ptid & 1) * 16) = make_uint4(0u, 0u, 0u, 0u);
        // transposing reads (read_tr16): lane j of 16 is in row j / 4 of four, 8 bytes j % 4 of the 32 of its 16 columns: of
        // the rows of B, per unit, tokens 4 h .. 4 h + 3 of its eight
        constexpr int UI = 4 * N / (64 * NWT);           // (n, eight tokens) units of the transposed B per thread
        static_assert(4 * N % (64 * NWT) == 0, "units per thread");
        const int trow = l16 >> 2, tpiece = (l16 >> 1) & 1, tbyte = (l16 & 1) * 8;
        int btr[UI][2];
#pragma unroll
        for (int i = 0; i < UI; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int u = ptid + i * (64 * NWT), row = 8 * (u / N) + 4 * h + trow;
                btr[i][h] = row * (2 * N) + ((((u % N) >> 4) * 2 + tpiece) ^ key_bc<N>(row)) * 16 + tbyte;
            }
        // quadrants (0,0), (1,0), (1,1) of M^T go round the waves; of four the last makes one too that it does not store
        constexpr int QPW = (3 + NWT - 1) / NWT;
        auto qi_of = [&](int i) { return pw + i * NWT >= 1 ? 1 : 0; };
        auto qj_of = [&](int i) { return pw + i * NWT == 2 ? 1 : 0; };
        float cum_all = 0.f;                             // SEG: log2 of the segment's decay

        // dt of a chunk, its prefix sums and the decay factors: every wave for itself (32 tokens, both halves alike)
        auto decays = [&](int c) {
            const uint32_t dt_bits = reinterpret_cast<const uint32_t *>(sDtr + (c & 3) * 256)[lane];
            float dv = __uint_as_float(dt_bits << 16) + dtb_h;
            if (p.dt_softplus) dv = softplus_fast(dv);
            if (c * Q + li >= L) dv = 0.f;               // padding: no decay, no input
            const float cum = prefix32(dv * A2_h);
            const float cq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cum), Q - 1));
            if constexpr (SEG) cum_all += cq;
            if (lh == 0) {
                const int o = (c & 1) * Q + li;
                sCum[o] = cum;
                sDt[o] = dv;
                sW[o] = __builtin_amdgcn_exp2f(cq - cum) * dv;
                if (pw == 0) sAt[(c & 3) * Q + li] = __builtin_amdgcn_exp2f(cum);
            }
        };
        auto produce = [&](int c) {
            const int buf = c & 1;
            char *sBh = lds + Ld::oBh + buf * Ld::PB, *sBl = lds + Ld::oBl + buf * Ld::PB;
            char *sM = lds + Ld::oM + buf * Ld::PM;
            const char *sB = lds + Ld::oB + xb * Ld::PBC, *sC = lds + Ld::oC + cb * Ld::PBC;
            // ---- every read of the raw inputs first: left in place they would queue up behind the stores of the stage before (which the
            // compiler cannot tell apart from them), a trip to LDS each ----
            uint4 gb[QPW][N / 32], gc[QPW][N / 32];      // operands of the wave's quadrants of G^T = B C^T
            if (emit) {
#pragma unroll
                for (int i = 0; i < QPW; ++i)
#pragma unroll
                    for (int kk = 0; kk < N / 32; ++kk) {
                        const int o = l16 * (N * 2) + (((4 * kk + k4) ^ key_bc<N>(l16)) * 16);
                        gb[i][kk] = *reinterpret_cast<const uint4 *>(sB + (qj_of(i) * (16 * N * 2) + o));
                        gc[i][kk] = *reinterpret_cast<const uint4 *>(sC + (qi_of(i) * (16 * N * 2) + o));
                    }
            }
            uint2 br[UI][2];
#pragma unroll
            for (int i = 0; i < UI; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) br[i][h] = read_tr16(sB + btr[i][h]);
            float4 w0[UI], w1[UI];                       // the weights of a unit's eight tokens
#pragma unroll
            for (int i = 0; i < UI; ++i) {
                const int u = ptid + i * (64 * NWT), oct = N >= 64 ? __builtin_amdgcn_readfirstlane(u / N) : u / N;
                w0[i] = *reinterpret_cast<const float4 *>(sW + buf * Q + 8 * oct);
                w1[i] = *reinterpret_cast<const float4 *>(sW + buf * Q + 8 * oct + 4);
            }
            float ct[QPW];
            float4 cs[QPW], ds[QPW];
            f4v gacc[QPW];
            if (emit) {
#pragma unroll
                for (int i = 0; i < QPW; ++i) {
                    ct[i] = sCum[buf * Q + 16 * qi_of(i) + l16];
                    cs[i] = *reinterpret_cast<const float4 *>(sCum + buf * Q + 16 * qj_of(i) + 4 * k4);
                    ds[i] = *reinterpret_cast<const float4 *>(sDt + buf * Q + 16 * qj_of(i) + 4 * k4);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (c + 1 < c_end) decays(c + 1);
            if (emit) {
#pragma unroll
                for (int i = 0; i < QPW; ++i) {
                    gacc[i] = f4v{0};
#pragma unroll
                    for (int kk = 0; kk < N / 32; ++kk) gacc[i] = mfma16(as_bf8(gb[i][kk]), as_bf8(gc[i][kk]), gacc[i]);
                }
            }
            // ---- w_s B_s transposed, head and tail: eight tokens of one n per unit ----
#pragma unroll
            for (int i = 0; i < UI; ++i) {
                const int u = ptid + i * (64 * NWT), n = u % N, oct = u / N;
                const float wv[8] = {w0[i].x, w0[i].y, w0[i].z, w0[i].w, w1[i].x, w1[i].y, w1[i].z, w1[i].w};
                uint32_t bh[4], bl[4];
                const uint32_t bb[4] = {br[i][0].x, br[i][0].y, br[i][1].x, br[i][1].y};
#pragma unroll
                for (int j2 = 0; j2 < 4; ++j2)
                    split2(wv[2 * j2] * __uint_as_float(bb[j2] << 16), wv[2 * j2 + 1] * __uint_as_float(bb[j2] & 0xffff0000u), bh[j2], bl[j2]);
                *reinterpret_cast<uint4 *>(sBh + n * XS + oct * 16) = make_uint4(bh[0], bh[1], bh[2], bh[3]);
                *reinterpret_cast<uint4 *>(sBl + n * XS + oct * 16) = make_uint4(bl[0], bl[1], bl[2], bl[3]);
            }
            // ---- this wave's quadrants of M^T: decayed, scaled, masked, D on the diagonal ----
            if (emit) {
#pragma unroll
                for (int i = 0; i < QPW; ++i) {
                    if (pw + i * NWT >= 3) break;
                    const float csv[4] = {cs[i].x, cs[i].y, cs[i].z, cs[i].w}, dsv[4] = {ds[i].x, ds[i].y, ds[i].z, ds[i].w};
                    float m[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float dec = __builtin_amdgcn_exp2f(ct[i] - csv[v]) * dsv[v];      // may overflow where s > t: selected away
                        const bool off_diagonal = pw + i * NWT == 1;
                        m[v] = off_diagonal ? gacc[i][v] * dec : keep[v] ? fmaf(gacc[i][v], dec, dadd[v]) : 0.f;
                    }
                    *reinterpret_cast<uint2 *>(sM + (16 * qi_of(i) + l16) * XS + (16 * qj_of(i) + 4 * k4) * 2) =
                        make_uint2(pack_bf16x2(m[0], m[1]), pack_bf16x2(m[2], m[3]));
                }
            }
        };
        auto wait_next = [&](bool newer) {               // the next chunk's rows have landed; `newer`: a further chunk's may be under way
            if (DIST == 1 || !newer) wait_direct_loads();
            else if (emit) wait_direct_loads_but<kLoads>();
            else wait_direct_loads_but<kLoadsState>();
        };
        // (as in the conv waves)
        asm volatile("" : "+v"(dtb_h));
        wait_next(c_beg + 1 < c_end);
        __syncthreads();
        // (in the head of this file)
        const bool gated = p.z != nullptr, silu = p.conv_act == SSMV_ACT_SILU;
        const bool first = N == 32 || (N == 128 ? !gated && (P < 128 || !silu) : P == 128 && (!gated || silu));
        if (first) __builtin_amdgcn_s_setprio(2);
        decays(c_beg);                                   // (read by this wave only, but for the consumers' share, a barrier later)
        for (int c = c_beg; c < c_end; ++c) {
            const bool more = c + DIST < c_end;
            if (more) issue(c + DIST, xi, ci);
            produce(c);
            wait_next(more);
            __syncthreads();
            xb = xb + 1 == XB ? 0 : xb + 1;
            xi = xi + 1 == XB ? 0 : xi + 1;
            cb = cb + 1 == CB ? 0 : cb + 1;
            ci = ci + 1 == CB ? 0 : ci + 1;
        }
        __syncthreads();
        if constexpr (SEG) {
            if (!seg.last && p.seg_pass == 0 && c_beg > 0 && ptid == 0)
                *reinterpret_cast<float *>(y_b + seg_piece<2>(P * N / 4, P, seg.area, HP, hd)) = cum_all;
        }
        return;
    }

    // ===================================================== consumers =====================================================
    const int lperm = swap23(li);
    const int pt = wave_u % NP, nh = NSPL - 1 - wave_u / NP;        // the wave's 32-channel tile, and its share of n (0 unless the state is split)
    const bool gated = p.z != nullptr;
    const int cur = (int)((unsigned)p.cur_slot[b] % 3u);
    float *state = p.state + (size_t)cur * p.slot_stride + ((size_t)b * H + hd) * P * N;
    const char *z_b = reinterpret_cast<const char *>(p.z) + (size_t)b * Ls * HP * 2;
    // a segment's state between the passes: the lane's float4 number q of tile tn in the rows of y from the segment's area on
    auto seg_at = [&](int tn, int q) {
        return reinterpret_cast<float4 *>(y_b + seg_piece<2>(((wave_u * TNL + tn) * 4 + q) * 64 + lane, P, seg.area, HP, hd));
    };
    // state -> accumulator registers, transposed tiles [n][p]: register 4 q + e of tile tn holds
    // h[p = 32 pt + li][n = 32 (TNL nh + tn) + 16 (q/2) + 8 lh + 4 (q%2) + e]
    f16v hacc[TNL];
    const int prow = pt * 32 + li, scol0 = 32 * TNL * nh + 8 * lh;
    auto state_at = [&](int tn, int q) { return state + state_off4(p.tiled, prow, scol0 + 32 * tn + 16 * (q / 2) + 4 * (q % 2), N); };
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!SEG || c_beg == 0) v = *reinterpret_cast<const float4 *>(state_at(tn, q));
            else if (p.seg_pass == 1) v = *seg_at(tn, q);
            hacc[tn][4 * q + 0] = v.x; hacc[tn][4 * q + 1] = v.y; hacc[tn][4 * q + 2] = v.z; hacc[tn][4 * q + 3] = v.w;
        }
    // outputs leave a chunk late: as whole rows of the head, dealt out over the waves (all 32-channel tiles side by side); with a
    // split state as rows of the tile's first wave, which then has the other's share of h C^T
    constexpr int LPT = NSPL == 1 ? 4 * NP : 4, TPI = 64 / LPT;          // lanes per token row, tokens per instruction
    int ytok[2], ylds[2];
    uint32_t oy[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int piece = lane % LPT;
        ytok[r] = (NSPL == 1 ? 2 * wave_u + r : r) * TPI + lane / LPT;
        ylds[r] = Ld::oY + (NSPL == 1 ? piece >> 2 : pt) * Ld::YT + ytok[r] * Ld::YS + (piece & 3) * 16;
        oy[r] = off(ytok[r], HP, hd * P + (NSPL == 1 ? 0 : pt * 32) + piece * 8);
    }
    auto store_rows = [&](int c) {
        char *yc = y_b + (size_t)c * Q * HP * 2;
        const char *from = lds + (c & 1) * (NP * Ld::YT);
        const int live = L - c * Q;
        uint4 v[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) v[r] = *reinterpret_cast<const uint4 *>(from + ylds[r]);
        if (live >= Q) {
#pragma unroll
            for (int r = 0; r < 2; ++r) *reinterpret_cast<uint4 *>(yc + oy[r]) = v[r];
        } else {
#pragma unroll
            for (int r = 0; r < 2; ++r)
                if (ytok[r] < live) *reinterpret_cast<uint4 *>(yc + oy[r]) = v[r];
        }
    };
    using QV = XVec<SSMV_BF16, 4>;                       // four adjacent channels
    typename QV::Raw zraw[4];
    auto load_gate = [&](int c) {
        const char *zc = chunk_of(z_b, c, HP) + off(min(li, L - 1 - c * Q), HP, hd * P + pt * 32 + 4 * lh);
#pragma unroll
        for (int q = 0; q < 4; ++q) zraw[q] = *reinterpret_cast<const typename QV::Raw *>(zc + 16 * q);
    };
    auto gate_and_round = [&](int c, f16v &yacc) {       // into the tile [token][channel]
        if (gated) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float zf[4];
                QV::decode(zraw[q], zf);
#pragma unroll
                for (int e = 0; e < 4; ++e) yacc[4 * q + e] *= silu_fast(zf[e]);
            }
        }
        char *sY = lds + Ld::oY + (c & 1) * (NP * Ld::YT) + pt * Ld::YT;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<uint2 *>(sY + li * Ld::YS + (8 * q + 4 * lh) * 2) =
                make_uint2(pack_bf16x2(yacc[4 * q], yacc[4 * q + 1]), pack_bf16x2(yacc[4 * q + 2], yacc[4 * q + 3]));
    };
    auto zsum_at = [&](int c) { return reinterpret_cast<float *>(lds + Ld::oZ) + ((c & 1) * NP + pt) * 1024 + lane * 4; };
    f16v yacc;
    auto finish = [&](int c) {                           // the outputs of chunk c, behind the barrier that ended it
        if constexpr (NSPL == 2) {
            if (nh == 1) return;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 z4 = *reinterpret_cast<const float4 *>(zsum_at(c) + q * 256);
                yacc[4 * q] += z4.x; yacc[4 * q + 1] += z4.y; yacc[4 * q + 2] += z4.z; yacc[4 * q + 3] += z4.w;
            }
            gate_and_round(c, yacc);
            __builtin_amdgcn_wave_barrier();             // the wave's own LDS traffic stays in program order
        }
        store_rows(c);
    };
    __syncthreads();                                     // the first raw inputs
    __syncthreads();                                     // the first chunk's operands
    for (int c = c_beg; c < c_end; ++c) {
        const int buf = c & 1;
        const char *sX = lds + Ld::oX + buf * Ld::PX, *sBh = lds + Ld::oBh + buf * Ld::PB, *sBl = lds + Ld::oBl + buf * Ld::PB;
        const char *sM = lds + Ld::oM + buf * Ld::PM, *sC = lds + Ld::oC + cb * Ld::PBC;
        const float *sAt = reinterpret_cast<const float *>(lds + Ld::oAt) + (c & 3) * Q;
        // ---- every operand of the chunk is requested first ----
        constexpr bool kAhead = TNL <= 2 && Ld::WPE < 4;                // (four state tiles in a wave leave no registers for the operands of the update)
        uint4 cop[2 * TNL], mop[2], bop[TNL][4];
        auto load_bop = [&](int tn) {
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const int o = (32 * (TNL * nh + tn) + lperm) * XS + (16 * st + 8 * lh) * 2;
                bop[tn][2 * st] = *reinterpret_cast<const uint4 *>(sBh + o);
                bop[tn][2 * st + 1] = *reinterpret_cast<const uint4 *>(sBl + o);
            }
        };
        auto load_cop = [&](int st) { cop[st] = *reinterpret_cast<const uint4 *>(sC + li * (N * 2) + (((2 * (2 * TNL * nh + st) + lh) ^ key_bc<N>(li)) * 16)); };
        if (emit && kAhead) {
#pragma unroll
            for (int st = 0; st < 2 * TNL; ++st) load_cop(st);
        }
        const float at_t = sAt[li], aq = sAt[Q - 1];
        uint4 xop[2];                                    // X of the wave's channels: A operand of X^T M^T, B operand of the update
#pragma unroll
        for (int st = 0; st < 2; ++st) xop[st] = *reinterpret_cast<const uint4 *>(sX + prow * XS + (16 * st + 8 * lh) * 2);
        if (kAhead) {
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn) load_bop(tn);
        }
        if (emit) {
#pragma unroll
            for (int st = 0; st < 2; ++st) mop[st] = *reinterpret_cast<const uint4 *>(sM + li * XS + (16 * st + 8 * lh) * 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (emit && c > c_beg) finish(c - 1);
        if (emit && gated && nh == 0) load_gate(c);
        if (emit) {
            // ---- Y^T = h C^T, scaled by exp(cum_t): the state registers are the A operand (heads only: this ends in outputs) ----
            yacc = f16v{0};
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    uint32_t ah[4];
                    if (!kAhead) load_cop(2 * tn + st);
#pragma unroll
                    for (int d = 0; d < 4; ++d) ah[d] = pack_bf16x2(hacc[tn][8 * st + 2 * d], hacc[tn][8 * st + 2 * d + 1]);
                    yacc = mfma(as_bf8(ah[0], ah[1], ah[2], ah[3]), as_bf8(cop[2 * tn + st]), yacc);
                }
        }
        // ---- h^T <- exp(cum_Q) h^T + (diag(w) B)^T X ----
#pragma unroll
        for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) hacc[tn][v] *= aq;
        if (kAhead) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int tn = 0; tn < TNL; ++tn) hacc[tn] = mfma(as_bf8(bop[tn][j]), as_bf8(xop[j / 2]), hacc[tn]);
        } else {
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn) {
                load_bop(tn);
#pragma unroll
                for (int j = 0; j < 4; ++j) hacc[tn] = mfma(as_bf8(bop[tn][j]), as_bf8(xop[j / 2]), hacc[tn]);
            }
        }
        if (emit) {
#pragma unroll
            for (int v = 0; v < 16; ++v) yacc[v] *= at_t;
            if (NSPL == 2 && nh == 1) {                  // the second half of n: for the tile's first wave
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(zsum_at(c) + q * 256) = make_float4(yacc[4 * q], yacc[4 * q + 1], yacc[4 * q + 2], yacc[4 * q + 3]);
            } else {
                // ---- Y^T += X^T M^T ----
#pragma unroll
                for (int st = 0; st < 2; ++st) yacc = mfma(as_bf8(xop[st]), as_bf8(mop[st]), yacc);
            }
        }
        if (NSPL == 1 && emit) gate_and_round(c, yacc);
        __syncthreads();
        cb = cb + 1 == CB ? 0 : cb + 1;
    }
    if (emit) finish(c_end - 1);
    if constexpr (SEG) {
        if (!seg.last) {
            if (p.seg_pass == 1) {                       // the next segment has its state already
                SSMV_TRACE_END(tid == 0);
                return;
            }
            // a segment's state on its way to the combining launch
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *seg_at(tn, q) = make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
            SSMV_TRACE_END(tid == 0);
            return;
        }
    }
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(state_at(tn, q)) =
                make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
    SSMV_TRACE_END(tid == 0);
}

template <int P, int N, bool SEG>
int launch_pn(const PrefillParams &p, hipStream_t stream)
{
    const size_t lds = PipeLds<P, N>::total;
    static_assert(PipeLds<P, N>::total <= 160 * 1024, "LDS");
    const dim3 grid((unsigned)(p.H * p.batch) * (SEG ? p.seg_count - 1 : 1)), block(64 * PipeLds<P, N>::NW);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&prefill_pipe_kernel<P, N, SEG>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL((prefill_pipe_kernel<P, N, SEG>), grid, block, lds, stream, p);
    return (int)hipGetLastError();
}

template <int P>
int launch_p(const PrefillParams &p, hipStream_t stream)
{
    switch (p.N) {
        case 32: return p.seg_count ? launch_pn<P, 32, true>(p, stream) : launch_pn<P, 32, false>(p, stream);
        case 64: return p.seg_count ? launch_pn<P, 64, true>(p, stream) : launch_pn<P, 64, false>(p, stream);
        case 128: return p.seg_count ? launch_pn<P, 128, true>(p, stream) : launch_pn<P, 128, false>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

}  // namespace

// Up to how many workgroups ((sequence, head) pairs) this kernel is the faster one: what fits the chip side by side, a second round where
// the other kernel gains little from company (measured at 1024 tokens, 64 to 1280 workgroups; us of the other kernel, of this one):
//   128 x 64   256: 59, 47;  384: 70, 78;  512: 84, 90;  1024: 165, 173      128 x 32   256: 50, 44;  384: 59, 77;  512: 75, 82
//   64 x 128   256: 70, 54;  384: 82, 92;  512: 84, 94;  1024: 167, 184      64 x 32    512: 57, 43;  768: 60, 70;  1024: 86, 110
//   32 x 128   512: 99, 90;  768: 103, 133;  1024: 181, 175                  32 x 64    768: 81, 66;  1024: 84, 102
//   32 x 32    768: 58, 42;  1024: 58, 63
//   64 x 64    512: 76, 52;  1024: 101, 100;  1280: 170, 129    128 x 128  256: 88, 64;  512: 171, 122;  1024: 341, 239 (all)
// A second round starts all over (LDS, the state's way in), which short prompts do not give back (us of the other kernel, of this one):
// 640 workgroups of 64 x 64, 1 token 10.2, 12.2;  64: 14.1, 15.7;  200: 0.97 of the other's;  768 of 32 x 64, 32: 11.1, 12.6;  128: 1.03;
// 200: 0.94;  512 of 32 x 128, 33: 13.9, 14.9;  128: 1.02;  200: 0.97.  With 64 x 64 the line depends on whether the other kernel's
// last round is a full one (four workgroups to a compute unit; this one's times over the other's):
//   one length  640: 128 tokens 1.02, 200 0.97;  1024: 400 1.05, 1024 0.99;  1280: 64 1.00, 96 0.96, 200 0.90;  1600: 64 1.04, 96 1.01, 200 0.98;
//               2048: 64 1.04, 200 1.03, 700 0.96
//   different   640: 128 1.08, 200 0.90;  1024: 200 1.08, 400 0.97;  1280: 200 1.16, 400 1.10, 700 1.00;  2048: 400 1.13, 512 1.11, 700 1.01
// Prompts of different lengths (drawn from 1 up) are bound by the longest, which is alone at its end: twice as many and less (same
// lengths at most: 128 x 64  512: 61, 53;  768: 85, 88;  64 x 128  512: 73, 63;  768: 84, 99;  64 x 32  768: 52, 45;  1024: 55, 57;  32 x 64  1024:
// 80, 61;  32 x 128  768: 92, 89;  1024: 94, 111), if they are long enough for that to outweigh the start of a second round of workgroups
// (512 workgroups of 128 x 64, 200 tokens each: 26, 31).  The host sees only that lengths are given: a call that gives equal ones is taken
// for one of these (64 x 128, 512 pairs of one length: 84, 94).
bool prefill_pipe_serves(const PrefillParams &p)
{
    const long pairs = (long)p.batch * p.H;
    auto pick = [&](int n32, int n64, int n128) { return p.N == 32 ? n32 : p.N == 64 ? n64 : n128; };
    const bool mixed = p.seq_len && p.L >= 512;
    if ((p.P == 128 && p.N == 128) || pairs <= 256 * prefill_pipe_resident(p.P, p.N)) return true;
    if (p.P == 64 && p.N == 64) {
        if (pairs <= 768) return p.L >= 160;
        if (pairs <= 1024) return p.L >= (p.seq_len ? 400 : 1024);
        return p.L >= (p.seq_len ? 700 : 65);
    }
    if (p.P == 32) return p.L >= 128 && pairs <= (mixed ? pick(1024, 1024, 768) : pick(768, 768, 512));
    return mixed && pairs <= (p.P == 64 && p.N == 32 ? 768 : 512);
}

int prefill_pipe_resident(int P, int N)
{
    auto pick = [&](int n32, int n64, int n128) { return N == 32 ? n32 : N == 64 ? n64 : n128; };
    if (P == 32) return pick(PipeLds<32, 32>::fit, PipeLds<32, 64>::fit, PipeLds<32, 128>::fit);
    if (P == 64) return pick(PipeLds<64, 32>::fit, PipeLds<64, 64>::fit, PipeLds<64, 128>::fit);
    return pick(PipeLds<128, 32>::fit, PipeLds<128, 64>::fit, PipeLds<128, 128>::fit);
}

// One workgroup to a compute unit, most units idle; slope between prompts of 1500 and 3000 tokens (64 x 32: 300 and 1024).  With a workgroup on
// every unit a chunk takes 0.86 to 1.01 (N <= 64) and 1.33 to 1.39 us.  Counted with those, choose_segments cuts more, and prompts of different
// lengths lose by it (288 pairs of 32 x 32, 1500 tokens at most: 41 whole, 54 cut).
double prefill_pipe_chunk_us(int P, int N, bool silu)
{
    // the conv waves are the longest stage then: 1.1 to 1.6 times (64 x 64, counted with 1.1: 176 pairs, 4096 tokens 175 uncut, 200 cut)
    const double conv = !silu || (P == 64 && N == 64) ? 1.0 : P == 128 ? 1.5 : P == 64 ? 1.3 : 1.1;
    if (N == 128) return conv * (P == 128 ? 1.38 : 1.25);
    return conv * (P == 128 ? 1.0 : P == 64 && N == 32 ? 0.91 : 0.78);
}

#ifdef SSMV_TRACE
int set_trace_prefill_pipe(long long *buf) { return (int)hipMemcpyToSymbol(HIP_SYMBOL(pf_trace_buf_), &buf, sizeof(buf)); }
#endif

int launch_prefill_pipe(const PrefillParams &p, hipStream_t stream)
{
    switch (p.P) {
        case 32: return launch_p<32>(p, stream);
        case 64: return launch_p<64>(p, stream);
        case 128: return launch_p<128>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

}  // namespace ssmv
