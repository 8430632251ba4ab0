// Chunked prefill for fp32 tensors: the evaluation and the operand layouts of prefill.hip, with the work of a chunk on different waves of the
// workgroup, side by side, one barrier per chunk.  (The sums are taken in another order, and a token's weight in the state comes from a
// sum of its own instead of the difference of two prefix sums: the last bits of the results are not those of the other kernel.)
//   consumer waves  own the state (accumulator registers, as there): C h^T, M X, the update, the gate and the outputs, of the chunk that
//                   the others prepared in the step before;
//   weight waves    one 16x16 quadrant of M each: B and C come from memory as operands of their product (a lane has the same 16 bytes of
//                   its row of C and of B, so that slot k of instruction 4 j + e is n = 16 j + 4 (lane/16) + e in both) and go to LDS from
//                   there, C scaled by exp(cum_t);
//   a decay wave    dt's prefix sums and the decays, a further step ahead;
//   conv waves      raw x -> X.
// Two copies of everything that is staged, in the order in which 16-byte reads of it are operands: slot lk of a product's kk-th instruction
// over the tokens is token 16 lk + kk.  In the other kernel the four waves stage a chunk and then multiply: 5.7 us a chunk alone on a compute
// unit (128 x 64).  Here 3.7, or 2.2 as two parts on two compute units (the figures that the plan in prefill.hip counts with).  Of a part's chunk
// the products take 2560 clock cycles of each SIMD and those of G 384 on average, 58 % of the launch below by the counters; the rest is the
// barrier, the LDS round trips behind it and the two steps that fill the stages.  4 x 1021 tokens of 32 heads x 128 x 64, with the ring and
// the state: 128 -> 82 us.
// Where the consumers split n (NSPL > 1) each takes a share of the tokens of M X too, and finishes a share of the tile's channels: the
// others' sums for these come through LDS, a step later.
//
// A head of P channels may be taken as p.parts heads of P / p.parts channels that share dt, A, D, B and C: p.H and p.P are those of the parts.
#include "prefill_split.h"

namespace ssmv {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kQ = kPrefillChunk;

template <int P, int N>
struct F32Pipe {                                         // float offsets of the LDS arrays
    static constexpr int TP = P / 32, TN = N / 32, SPL = 4 / TP;
    static constexpr int TNL = TN > SPL ? TN / SPL : 1;  // state tiles of a consumer wave
    static constexpr int NSPL = TN / TNL;                // consumer waves per 32-channel tile
    static constexpr int NC = TP * NSPL, NWT = 3, NCV = 4, NW = NC + NWT + 1 + NCV;
    static constexpr int NP = N + 4, QP = kQ + 4;        // row strides of C, and of what is indexed [..][token]: 16-byte rows, all banks
    static constexpr int oX = 0;                         // [2][P][QP]   conv output
    static constexpr int oB = oX + 2 * P * QP;           // [2][N][QP]   w_s B_s, w_s = exp(cum_Q - cum_s) dt_s
    static constexpr int oC = oB + 2 * N * QP;           // [2][Q][NP]   exp(cum_t) C_t
    static constexpr int oZ = oC + 2 * kQ * NP;          // [2][TP][NSPL][16][64]  a consumer's sums
    static constexpr int oW = oZ + (NSPL > 1 ? 2 * NC * 1024 : 0);      // [4][Q]  w_s
    static constexpr int oAt = oW + 4 * kQ;              // [4][Q]  exp(cum_t): decay from the chunk's start to after token t
    static constexpr int oCum = oAt + 4 * kQ;            // [4][Q]  inclusive prefix of dt*A
    static constexpr int oDt = oCum + 4 * kQ;            // [4][Q]  dt
    static constexpr int oM = oDt + 4 * kQ;              // [2][Q][QP]
    static constexpr int floats = oM + 2 * kQ * QP;
};

// SEG: the workgroup owns one segment of the prompt instead of all of it (prefill_split.h); in the first pass every segment but the
// first one forms its share of the state only
template <int P, int N, bool SEG>
__global__ __launch_bounds__((64 * F32Pipe<P, N>::NW)) void prefill_f32_pipe_kernel(const PrefillParams p)
{
    using Ld = F32Pipe<P, N>;
    using Vec = IoVec<SSMV_F32>;
    constexpr int Q = kQ, W = SSMV_CONV_WIDTH;
    constexpr int NP = Ld::NP, QP = Ld::QP, TP = Ld::TP, TNL = Ld::TNL, NSPL = Ld::NSPL, NC = Ld::NC, NWT = Ld::NWT, NCV = Ld::NCV;
    static_assert(P % 32 == 0 && P <= 128 && N % 32 == 0 && N <= 128 && W == 4, "tile shapes");

    extern __shared__ float4 lds_raw[];
    float *lds = reinterpret_cast<float *>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const PrefillItem item = prefill_item<SEG>(p);
    const int hd = item.hd, b = item.b;
    const int L = item.L;                                // this sequence's prompt length
    if (L == 0) return;                                  // nothing to feed: state, ring and outputs stay as they are
    Segment seg = {0, (L + Q - 1) / Q, 0, true, true, true};
    if constexpr (SEG) {
        seg = segment_of(p, L, item.slot);
        if (!seg.work) return;
    }
    const int c_beg = SEG ? seg.c0 : 0, c_end = seg.c1;  // the chunks of this workgroup
    const bool emit = !SEG || seg.emit;                  // whether it writes outputs
    const int Ls = p.L, HP = p.H * P;
    // addresses: a base pointer per sequence and a 32-bit element offset from the 24-bit multiplier (the host refuses prompts whose tensors
    // would not fit)
    auto off = [](int token, int stride, int rest) { return (size_t)(unsigned)(__umul24(token, stride) + rest); };
    char *y_b = reinterpret_cast<char *>(p.y) + (size_t)b * Ls * HP * 4;

    if (wave > NC + NWT) {
        // =================================================== conv waves ==================================================
        constexpr int XG = 64 * NCV / P, QS = Q / XG;    // thread groups along the tokens, consecutive tokens per thread
        const int ptid = tid - 64 * (NC + NWT + 1), pc = ptid % P, s0 = ptid / P * QS;
        const int ch = hd * P + pc, mask = p.ring_len - 1;
        // (the last pass of a segmented prompt runs behind the launch that has moved conv_head on already)
        const int conv_head = (p.conv_head[b] - (SEG && p.seg_pass == 1 ? L : 0)) & mask;
        const char *x_b = reinterpret_cast<const char *>(p.x_raw) + (size_t)b * Ls * HP * 4;
        const bool silu = p.conv_act == SSMV_ACT_SILU;
        float wgt[W];
#pragma unroll
        for (int w = 0; w < W; ++w) wgt[w] = load_io(p.wgt, (size_t)ch * W + w, SSMV_F32);
        const float cbias = p.bias ? load_io(p.bias, ch, SSMV_F32) : 0.f;
        auto raw_bits = [&](int tg) { return Vec::load_raw1(x_b, off(min(max(tg, 0), L - 1), HP, ch)); };
        float hist[W - 1];                               // the raw inputs ahead of the prompt (newest last)
#pragma unroll
        for (int j = 0; j < W - 1; ++j) hist[j] = load_io(p.ring, ((size_t)b * p.ring_len + ((conv_head + 1 - (W - 1) + j) & mask)) * HP + ch, SSMV_F32);
        uint32_t raw[QS + W - 1];
        auto fetch = [&](int c) {
#pragma unroll
            for (int j = 0; j < QS + W - 1; ++j) raw[j] = raw_bits(c * Q + s0 - (W - 1) + j);
        };
        auto stage = [&](int c) {
            float *sX = lds + Ld::oX + (c & 1) * (P * QP) + pc * QP + s0;
            const int t0 = c * Q + s0;
            float r[QS + W - 1];
#pragma unroll
            for (int j = 0; j < QS + W - 1; ++j) r[j] = j < W - 1 && t0 - (W - 1) + j < 0 ? hist[j < W - 1 ? j : 0] : Vec::decode1(raw[j]);
#pragma unroll
            for (int j0 = 0; j0 < QS; j0 += 4) {
                f4v x;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // same fp32 order and rounding as conv1d_state_update
                    float acc = cbias;
#pragma unroll
                    for (int w = 0; w < W; ++w) acc = fmaf(wgt[w], r[j0 + j + w], acc);
                    x[j] = acc;
                }
                if (silu) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = x[j] / (1.f + expf(-x[j]));
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = t0 + j0 + j < L ? x[j] : 0.f;
                *reinterpret_cast<f4v *>(sX + j0) = x;
            }
        };
        fetch(c_beg);
        __syncthreads();
        for (int c = c_beg; c < c_end; ++c) {
            stage(c);
            if (c + 1 < c_end) fetch(c + 1);
            __syncthreads();
        }
        __syncthreads();
        if ((!SEG || seg.last) && ptid < P) {            // the newest W-1 raw inputs into the ring behind conv_head
            for (int tg = max(L - (W - 1), 0); tg < L; ++tg)
                Vec::store_raw1(p.ring, ((size_t)b * p.ring_len + ((conv_head + 1 + tg) & mask)) * HP + ch, raw_bits(tg));
        }
        return;
    }
    const int heads = p.H / p.parts, hr = hd / p.parts;  // dt, A, D, B and C know the head, not its parts
    if (wave == NC + NWT) {
        // =================================================== the decay wave ==================================================
        const int li = lane & 31;                        // both halves alike
        const char *dt_b = reinterpret_cast<const char *>(p.dt) + ((size_t)b * Ls * heads + hr) * 4;
        const float A_h = p.A[hr], dtb_h = p.dt_bias ? p.dt_bias[hr] : 0.f;
        uint32_t dt_raw;
        auto fetch = [&](int c) { dt_raw = Vec::load_raw1(dt_b, off(min(c * Q + li, L - 1), heads, 0)); };
        float cum_all = 0.f;                             // SEG: log of the segment's decay
        auto decays = [&](int c) {
            float d = Vec::decode1(dt_raw) + dtb_h;
            if (c + 1 < c_end) fetch(c + 1);
            if (p.dt_softplus) d = softplus_fast(d);
            if (c * Q + li >= L) d = 0.f;                // padding: no decay, no input
            float v = d * A_h;
            // the decay from a token to the chunk's end as a sum of its own: as the difference of two prefix sums it has their rounding,
            // which under a strong decay is large beside what the last tokens add up to (state against 64 bits, 4 x 1021 tokens of 32 heads x
            // 128 x 64: 1.1e-7 of the norm; 2.1e-7 to 2.4e-7 in the other kernel, the outputs 5.2e-8 in both)
            float after = __shfl_down(v, 1, 32);
            if (li == Q - 1) after = 0.f;
#pragma unroll
            for (int o = 1; o < Q; o <<= 1) {
                const float u = __shfl_up(v, o, 32), w = __shfl_down(after, o, 32);
                if (li >= o) v += u;
                if (li + o < Q) after += w;
            }
            const float cq = __shfl(v, Q - 1, 64);
            if constexpr (SEG) cum_all += cq;
            float *to = lds + (c & 3) * Q + li;
            to[Ld::oDt] = d;
            to[Ld::oCum] = v;
            to[Ld::oAt] = expf(v);
            to[Ld::oW] = expf(after) * d;
        };
        fetch(c_beg);
        decays(c_beg);
        __syncthreads();
        for (int c = c_beg; c < c_end; ++c) {
            if (c + 1 < c_end) decays(c + 1);
            __syncthreads();
        }
        __syncthreads();
        if constexpr (SEG) {
            if (!seg.last && p.seg_pass == 0 && c_beg > 0 && lane == 0)
                *reinterpret_cast<float *>(y_b + seg_piece<4>(P * N / 4, P, seg.area, HP, hd)) = cum_all * 1.4426950408889634f;
        }
        return;
    }
    if (wave >= NC) {
        // =================================================== weight waves ===================================================
        const int pw = wave - NC, qi = pw >= 1, qj = pw == 2;       // rows t in [16 qi, +16), columns s in [16 qj, +16)
        const int l16 = lane & 15, k4 = lane >> 4;
        const int GN = p.G * N, g = hr / (heads / p.G);
        const char *B_b = reinterpret_cast<const char *>(p.Bm) + ((size_t)b * Ls * GN + (size_t)g * N) * 4;
        const char *C_b = reinterpret_cast<const char *>(p.Cm) + ((size_t)b * Ls * GN + (size_t)g * N) * 4;
        constexpr int NV = N / 16;                       // 16-byte pieces of a row per lane
        f4v bv[NV], cv[NV];
        auto fetch = [&](int c) {
            const int tb = min(c * Q + 16 * qj + l16, L - 1), tc = min(c * Q + 16 * qi + l16, L - 1);
#pragma unroll
            for (int j = 0; j < NV; ++j) bv[j] = *reinterpret_cast<const f4v *>(B_b + 4 * off(tb, GN, 16 * j + 4 * k4));
            if (emit) {
#pragma unroll
                for (int j = 0; j < NV; ++j) cv[j] = *reinterpret_cast<const f4v *>(C_b + 4 * off(tc, GN, 16 * j + 4 * k4));
            }
        };
        auto stage = [&](int c) {
            const int buf = c & 1, t0 = c * Q;
            const float *dec = lds + (c & 3) * Q;
            const f4v ct = *reinterpret_cast<const f4v *>(dec + Ld::oCum + 16 * qi + 4 * k4);
            const float cs = dec[Ld::oCum + 16 * qj + l16], ds = dec[Ld::oDt + 16 * qj + l16], a = dec[Ld::oAt + 16 * qi + l16], ws = dec[Ld::oW + 16 * qj + l16];
            if (t0 + Q > L) {                            // rows behind the prompt's end
                const bool dead_b = t0 + 16 * qj + l16 >= L, dead_c = t0 + 16 * qi + l16 >= L;
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    if (dead_b) bv[j] = f4v{0};
                    if (dead_c) cv[j] = f4v{0};
                }
            }
            if (pw != 1) {
                float *sB = lds + Ld::oB + buf * (N * QP) + 4 * k4 * QP + 16 * qj + l16;
#pragma unroll
                for (int j = 0; j < NV; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sB[(16 * j + e) * QP] = bv[j][e] * ws;
            }
            if (!emit) return;
            f4v gacc = {0};
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) gacc = __builtin_amdgcn_mfma_f32_16x16x4f32(cv[j][e], bv[j][e], gacc, 0, 0, 0);
            if (pw != 1) {                               // on C, not on the sums: these may leave fp32's range where y does not
                float *sC = lds + Ld::oC + buf * (Q * NP) + (16 * qi + l16) * NP + 4 * k4;
#pragma unroll
                for (int j = 0; j < NV; ++j) *reinterpret_cast<f4v *>(sC + 16 * j) = cv[j] * a;
            }
            float *sM = lds + Ld::oM + buf * (Q * QP) + (16 * qi + 4 * k4) * QP + 16 * qj + l16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool keep = pw == 1 || l16 <= 4 * k4 + i;
                const float m = gacc[i] * expf(keep ? ct[i] - cs : 0.f) * ds;
                sM[i * QP] = keep ? m : 0.f;
            }
        };
        // the quadrant t < 16 <= s of both copies of M stays zero
        if (pw == 1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) lds[Ld::oM + (i >> 2) * (Q * QP) + (4 * (i & 3) + k4) * QP + 16 + l16] = 0.f;
        }
        fetch(c_beg);
        __syncthreads();                                 // the first chunk's decays
        for (int c = c_beg; c < c_end; ++c) {
            stage(c);
            if (c + 1 < c_end) fetch(c + 1);
            __syncthreads();
        }
        __syncthreads();
        return;
    }

    // ===================================================== consumers =====================================================
    const int li = lane & 31, lk = lane >> 5;            // MFMA: row/column index and k index of this lane
    const int pt = wave % TP, nh = wave / TP;            // the wave's channel tile, and its share of n
    const bool gated = p.z != nullptr;
    const float D_h = p.D[hr];
    const int cur = (int)((unsigned)p.cur_slot[b] % 3u);
    float *state = p.state + (size_t)cur * p.slot_stride + ((size_t)b * p.H + hd) * P * N;
    const char *z_b = reinterpret_cast<const char *>(p.z) + (size_t)b * Ls * HP * 4;
    // the lane's channel in the tile: such that the channels which the wave finishes are its first rows
    constexpr int KQ = 4 / NSPL, KX = Q / 2 / NSPL;
    const int lch = li ^ (8 * KQ * nh);
    // state -> registers, transposed tiles [n][p]: register 4 q + e of tile tn holds h[p = 32 pt + lch][n = 32 (TNL nh + tn) + 8 q + 4 lk + e].
    // From the live slot, from what the combining launch left in the segment's rows of y, or zeros
    f16v hacc[TNL];
    auto state_at = [&](int tn, int q) { return state + state_off4(p.tiled, pt * 32 + lch, 32 * (TNL * nh + tn) + 8 * q + 4 * lk, N); };
    auto seg_at = [&](int tn, int q) {
        return reinterpret_cast<float4 *>(y_b + seg_piece<4>(((wave * TNL + tn) * 4 + q) * 64 + lane, P, seg.area, HP, hd));
    };
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!SEG || c_beg == 0) v = *reinterpret_cast<const float4 *>(state_at(tn, q));
            else if (p.seg_pass == 1) v = *seg_at(tn, q);
            hacc[tn][4 * q + 0] = v.x; hacc[tn][4 * q + 1] = v.y; hacc[tn][4 * q + 2] = v.z; hacc[tn][4 * q + 3] = v.w;
        }
    // here before the loop: the compiler would wait for it at its first use in there, and with it for the outputs on their way
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn) asm volatile("" : "+v"(hacc[tn]));
    // The output tile is accumulated TRANSPOSED (rows = the wave's 32 channels, columns = the chunk's tokens): register 4 q + e of a lane is
    // channel 8 (q ^ KQ nh) + 4 lk + e of token li.  The wave finishes q < KQ, and multiplies M X over KX pairs of tokens from KX nh on
    float ykeep[KQ][4], xkeep[KQ][4];
    float4 zin[KQ];
    auto channel = [&](int k) { return pt * 32 + 8 * (KQ * nh + k) + 4 * lk; };       // first of four, inside the head
    auto load_gate = [&](int c) {
#pragma unroll
        for (int k = 0; k < KQ; ++k) zin[k] = *reinterpret_cast<const float4 *>(z_b + 4 * off(min(c * Q + li, L - 1), HP, hd * P + channel(k)));
    };
    auto zsum = [&](int c, int share, int q) { return lds + Ld::oZ + ((c & 1) * NC + pt * NSPL + share) * 1024 + q * 256 + lane * 4; };
    auto finish = [&](int c) {
        if constexpr (NSPL > 1) {
#pragma unroll
            for (int u = 1; u < NSPL; ++u)
#pragma unroll
                for (int k = 0; k < KQ; ++k) {
                    const f4v o = *reinterpret_cast<const f4v *>(zsum(c, nh ^ u, KQ * nh + k));
#pragma unroll
                    for (int e = 0; e < 4; ++e) ykeep[k][e] += o[e];
                }
        }
#pragma unroll
        for (int k = 0; k < KQ; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) ykeep[k][e] = fmaf(D_h, xkeep[k][e], ykeep[k][e]);       // last: one rounding at the size of the output
        if (gated) {
#pragma unroll
            for (int k = 0; k < KQ; ++k) {
                const float zf[4] = {zin[k].x, zin[k].y, zin[k].z, zin[k].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) ykeep[k][e] *= silu_fast(zf[e]);
            }
        }
        if (c * Q + li < L) {
#pragma unroll
            for (int k = 0; k < KQ; ++k)
                *reinterpret_cast<float4 *>(y_b + 4 * off(c * Q + li, HP, hd * P + channel(k))) = make_float4(ykeep[k][0], ykeep[k][1], ykeep[k][2], ykeep[k][3]);
        }
    };
    __syncthreads();                                     // the first chunk's decays
    __syncthreads();                                     // the first chunk's operands
    f16v sacc = {0};                                     // the last state tile's update by the chunk before, and that chunk's decay
    float aq = 1.f;
    auto take_in = [&](int tn) {                         // the chunk's own sum, then ONE rounding against the state (prefill.hip)
#pragma unroll
        for (int v = 0; v < 16; ++v) hacc[tn][v] = fmaf(aq, hacc[tn][v], sacc[v]);
    };
    for (int c = c_beg; c < c_end; ++c) {
        const int buf = c & 1;
        // slot lk of a product's kk-th instruction is token 16 lk + kk
        const float *sX = lds + Ld::oX + buf * (P * QP) + pt * 32 * QP, *sB = lds + Ld::oB + buf * (N * QP) + (32 * TNL * nh + li) * QP + 16 * lk;
        const float *sC = lds + Ld::oC + buf * (Q * NP) + li * NP + 32 * TNL * nh + 4 * lk, *sM = lds + Ld::oM + buf * (Q * QP) + li * QP + 16 * lk;
        auto read4 = [](const float *from) { return *reinterpret_cast<const f4v *>(from); };
        f4v x4[4], m4[KX / 4], xm4[KX / 4], op[4], next[4];
        auto request_c = [&](int tn, f4v (&to)[4]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) to[q] = read4(sC + 32 * tn + 8 * q);
        };
        auto request_b = [&](int tn, f4v (&to)[4]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) to[q] = read4(sB + 32 * tn * QP + 4 * q);
        };
        // Every operand is requested a group of products ahead of its own; what is left of the chunk before, and of these outputs, goes
        // between the products
        if (emit) request_c(0, op);
        else request_b(0, op);
        take_in(TNL - 1);
        aq = lds[Ld::oAt + (c & 3) * Q + Q - 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) x4[i] = read4(sX + lch * QP + 16 * lk + 4 * i);
        f16v yacc = {0};
        if (emit) {
#pragma unroll
            for (int i = 0; i < KX / 4; ++i) {
                m4[i] = read4(sM + KX * nh + 4 * i);
                xm4[i] = NSPL == 1 ? x4[i] : read4(sX + lch * QP + 16 * lk + KX * nh + 4 * i);
            }
            // ---- C h^T: the state registers are the A operand ----
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn) {
                __builtin_amdgcn_sched_barrier(0);
                if (tn + 1 < TNL) request_c(tn + 1, next);
                else request_b(0, next);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    yacc = __builtin_amdgcn_mfma_f32_32x32x2f32(hacc[tn][i], op[i / 4][i % 4], yacc, 0, 0, 0);
                    if (tn == 0 && i == 3) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (NSPL > 1 && c > c_beg) finish(c - 1);
                        if (gated) load_gate(c);
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) op[q] = next[q];
            }
            // ---- + X^T M^T ----
#pragma unroll
            for (int j = 0; j < KX; ++j) yacc = __builtin_amdgcn_mfma_f32_32x32x2f32(xm4[j / 4][j % 4], m4[j / 4][j % 4], yacc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- h^T <- exp(cum_Q) h^T + B^T (diag(w) X), in the registers ----
#pragma unroll
        for (int tn = 0; tn < TNL; ++tn) {
            if (tn + 1 < TNL) request_b(tn + 1, next);
            f16v acc = {0};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(op[i / 4][i % 4], x4[i / 4][i % 4], acc, 0, 0, 0);
                if (tn == 0 && i == 3 && emit) {
                    __builtin_amdgcn_sched_barrier(0);
                    // what the wave finishes, the sums of the other channels to their waves
#pragma unroll
                    for (int k = 0; k < KQ; ++k)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            ykeep[k][e] = yacc[4 * k + e];
                            xkeep[k][e] = sX[(channel(k) - pt * 32 + e) * QP + li];
                        }
#pragma unroll
                    for (int q = KQ; q < 4; ++q)
                        *reinterpret_cast<f4v *>(zsum(c, nh, q ^ (KQ * nh))) = f4v{yacc[4 * q], yacc[4 * q + 1], yacc[4 * q + 2], yacc[4 * q + 3]};
                    if (NSPL == 1) finish(c);
                }
            }
            sacc = acc;
            if (tn + 1 < TNL) take_in(tn);
#pragma unroll
            for (int q = 0; q < 4; ++q) op[q] = next[q];
        }
        __syncthreads();
    }
    take_in(TNL - 1);
    if (NSPL > 1 && emit) finish(c_end - 1);
    if constexpr (SEG) {
        if (!seg.last) {
            if (p.seg_pass == 1) return;                 // the next segment has its state already
            // a segment's state on its way to the combining launch
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *seg_at(tn, q) = make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
            return;
        }
    }
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(state_at(tn, q)) = make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
}

template <int P, int N, bool SEG>
int launch_pn(const PrefillParams &p, hipStream_t stream)
{
    const size_t lds = F32Pipe<P, N>::floats * sizeof(float);
    static_assert(F32Pipe<P, N>::floats * sizeof(float) <= 160 * 1024, "LDS");
    const dim3 grid((unsigned)(p.H * p.batch) * (SEG ? p.seg_count - 1 : 1)), block(64 * F32Pipe<P, N>::NW);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&prefill_f32_pipe_kernel<P, N, SEG>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL((prefill_f32_pipe_kernel<P, N, SEG>), grid, block, lds, stream, p);
    return (int)hipGetLastError();
}

template <int P, int N>
int launch_n(const PrefillParams &p, hipStream_t stream) { return p.seg_count ? launch_pn<P, N, true>(p, stream) : launch_pn<P, N, false>(p, stream); }

}  // namespace

// (128 x 128 is taken as two parts, or by the other kernel)
int launch_prefill_f32_pipe(const PrefillParams &p, hipStream_t stream)
{
    switch (p.P * 1000 + p.N) {
        case 32032: return launch_n<32, 32>(p, stream);
        case 32064: return launch_n<32, 64>(p, stream);
        case 32128: return launch_n<32, 128>(p, stream);
        case 64032: return launch_n<64, 32>(p, stream);
        case 64064: return launch_n<64, 64>(p, stream);
        case 64128: return launch_n<64, 128>(p, stream);
        case 128032: return launch_n<128, 32>(p, stream);
        case 128064: return launch_n<128, 64>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

}  // namespace ssmv
