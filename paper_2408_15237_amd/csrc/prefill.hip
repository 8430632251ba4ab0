// Chunked prefill of a scalar-decay (Mamba-2 style) layer with fp32 tensors, in large launches and where a cut prompt is faster this way
// (plan_f32; the others: prefill_f32_pipe.hip; bf16 tensors: prefill_bf16.hip, same evaluation on the bf16 matrix cores): all L prompt tokens through the recurrence of
// Section 2.1 Eq. 1 (with the discretisation of Section 2.2), producing every y_t and leaving the cached state and
// the conv ring as if the L tokens had been verified and accepted.  This is where the path has a dense
// contraction, so it runs on the matrix cores (fp32 MFMA: the state and the outputs keep fp32 accuracy).
//
// Per chunk of Q = 32 tokens, with cum_t = A * (dt_0 + .. + dt_t) inside the chunk and h the state before it:
//   G      = C B^T                                            [Q x Q]   contraction over N
//   M_ts   = G_ts exp(cum_t - cum_s) dt_s   for s <= t, else 0
//   Y      = M X  +  diag(exp(cum_t)) C h^T  +  D X           [Q x P]   contractions over Q and over N
//   h     <- exp(cum_Q) h  +  (diag(w) X)^T B,  w_s = exp(cum_Q - cum_s) dt_s      [P x N]   contraction over Q
// which is Eq. 1 unrolled over the chunk and regrouped (the "chunked" or "state-space dual" evaluation of the
// scan; the paper's own prefill uses the hardware-aware scan of its reference [Mamba]).  One workgroup of four
// waves owns one (sequence, head).  The state stays in the accumulator registers across the chunks, transposed (rows = n,
// columns = channel): a lane's register of a tile is then directly the A operand of C h^T (its two k slots are rows n and n + 4)
// and the update ends in place; the chunk's X, B, C are in LDS as fp32, X is read once for both of its products.
// (With the state in LDS, read for C h^T and read and written back for the update, a chunk took 256 instead of about 90 LDS
// instructions per wave.  16 x 512 tokens of 32 heads x 128 x 128: 473 -> 238 us; 8 x 512 of 80 x 64 x 128: 283 -> 236; 32 x 512 of 32 x
// 128 x 64: 311 -> 295.  Scaling C by exp(cum_t) ahead of the product and not the sums behind it is 1 to 3 % of that: 229, 233, 291.)
// (The products alone, 80 of 64 cycles each per wave and chunk at 128 x 64, would take 0.6 of that time.)
// v_mfma_f32_32x32x2_f32 operands: A[i = lane%32][k = lane/32], B[k = lane/32][j = lane%32]; result register v of
// a lane is D[8*(v/4) + 4*(lane/32) + v%4][lane%32]; v_mfma_f32_16x16x4_f32 (used for the Q x Q product, one
// quadrant per wave): A[i = lane%16][k = lane/16], B[k = lane/16][j = lane%16], D[4*(lane/16) + v][lane%16].  Rows of
// the LDS arrays that are read with the lane as the ROW index are padded, by one float (M) or by four (B, C: 16-byte reads),
// so that the lanes hit different banks.
// The global loads of chunk c+1 are issued (as raw bits, unconditionally, from clamped addresses) right after the
// barrier that ends the staging of chunk c and are decoded into LDS after chunk c's arithmetic: one chunk of
// latency hiding for a kernel that would otherwise wait for memory once per chunk.
#include "prefill_split.h"

namespace ssmv {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));

constexpr int kQ = kPrefillChunk;

// How the four waves share a head: wave w owns the 32 channels [32 (w % TP), +32) and, of the state's 32-wide tiles along n, the
// TNL from TNL (w / TP) on (narrow heads split n; where there are fewer tiles than waves the last ones only stage).
template <int P, int N>
struct F32Shape {
    static constexpr int TP = P / 32, TN = N / 32, SPL = 4 / TP;
    static constexpr int TNL = TN > SPL ? TN / SPL : 1;
    static constexpr int NSPL = TN / TNL;                // waves per channel tile that own state
    static constexpr int NP = N + 4, QP = kQ + 1;        // row strides of B, C and of M: 16-byte rows, all banks
    static constexpr int floats = kQ * P + 2 * kQ * NP + kQ * QP + 3 + 4 * kQ + (NSPL - 1) * TP * 1024;
};

// SEG: the workgroup owns one segment of the prompt instead of all of it (prefill_split.h); in the first pass every segment
// but the first one forms its share of the state only: no Q x Q product, no outputs, one barrier less per chunk.
template <int P, int N, int IO, bool SEG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void prefill_kernel(const PrefillParams p)
{
    constexpr int Q = kQ;
    constexpr int W = SSMV_CONV_WIDTH;
    using Sh = F32Shape<P, N>;
    constexpr int NP = Sh::NP, QP = Sh::QP, TP = Sh::TP, TNL = Sh::TNL, NSPL = Sh::NSPL;
    constexpr int XG = 256 / P;          // thread groups along the tokens of a chunk
    constexpr int QS = Q / XG;           // consecutive tokens one thread convolves per chunk
    using Vec = IoVec<IO>;
    constexpr int EV = Vec::EV;
    static_assert(P % 32 == 0 && P <= 128 && N % 32 == 0, "tile shapes");

    extern __shared__ float4 lds_raw[];
    float *sX = reinterpret_cast<float *>(lds_raw);     // [Q][P]    conv output of the chunk (rounded to the I/O type)
    float *sB = sX + Q * P;                             // [Q][N+4]
    float *sC = sB + Q * NP;                            // [Q][N+4]
    float *sDt = sC + Q * NP;                           // [Q]
    float *sCum = sDt + Q;                              // [Q]  inclusive prefix of dt*A
    float *sAt = sCum + Q;                              // [Q]  exp(cum_t): decay from the chunk's start to after token t
    float *sW = sAt + Q;                                // [Q]  exp(cum_Q - cum_s) dt_s: weight of token s in the chunk's state update
    float *sM = sW + Q;                                 // [Q][Q+1]
    float *sZ = sM + ((Q * QP + 3) & ~3);               // [NSPL-1][TP][16][64]  C h^T over the later shares of n

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lk = lane >> 5;           // MFMA: row/column index and k index of this lane
    const int pt = wave % TP, nh = wave / TP;           // the wave's channel tile, and its share of n
    const bool owns = nh < NSPL;
    const int H = p.H, G = p.G;
    const PrefillItem item = prefill_item<SEG>(p);
    const int hd = item.hd, b = item.b;
    const int Ls = p.L;                                 // token stride of the arrays
    const int L = item.L;                               // this sequence's prompt length
    if (L == 0) return;                                 // nothing to feed: state, ring and outputs stay as they are
    Segment seg = {0, (L + Q - 1) / Q, 0, true, true, true};
    if constexpr (SEG) {
        seg = segment_of(p, L, item.slot);
        if (!seg.work) return;
    }
    const int c_beg = SEG ? seg.c0 : 0, c_end = seg.c1; // the chunks of this workgroup
    const bool emit = !SEG || seg.emit;                 // whether it writes outputs
    const int HP = H * P, GN = G * N;
    const int g = hd / (H / G);
    const int cur = (int)((unsigned)p.cur_slot[b] % 3u);
    const int mask = p.ring_len - 1;
    // (the last pass of a segmented prompt runs behind the launch that has moved conv_head on already)
    const int conv_head = (p.conv_head[b] - (SEG && p.seg_pass == 1 ? L : 0)) & mask;
    const float A_h = p.A[hd], D_h = p.D[hd];
    const float dtb_h = p.dt_bias ? p.dt_bias[hd] : 0.f;
    const bool gated = p.z != nullptr;
    float *state = p.state + (size_t)cur * p.slot_stride + ((size_t)b * H + hd) * P * N;

    constexpr size_t ES = IO == SSMV_BF16 ? 2 : 4;
    char *y_b = reinterpret_cast<char *>(p.y) + (size_t)b * Ls * HP * ES;
    // state -> registers, transposed tiles [n][p]: register 4 q + e of tile tn holds h[p = 32 pt + li][n = 32 (TNL nh + tn) + 8 q + 4 lk + e].
    // From the live slot, from what the combining launch left in the segment's rows of y, or zeros
    f16v hacc[TNL];
    auto state_at = [&](int tn, int q) { return state + state_off4(p.tiled, pt * 32 + li, 32 * (TNL * nh + tn) + 8 * q + 4 * lk, N); };
    auto seg_at = [&](int tn, int q) {
        return reinterpret_cast<float4 *>(y_b + seg_piece<ES>((((nh * TP + pt) * TNL + tn) * 4 + q) * 64 + lane, P, seg.area, HP, hd));
    };
    if (owns) {
#pragma unroll
        for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (!SEG || c_beg == 0) v = *reinterpret_cast<const float4 *>(state_at(tn, q));
                else if (p.seg_pass == 1) v = *seg_at(tn, q);
                hacc[tn][4 * q + 0] = v.x; hacc[tn][4 * q + 1] = v.y; hacc[tn][4 * q + 2] = v.z; hacc[tn][4 * q + 3] = v.w;
            }
    }
    // this thread's conv channel: weights and bias stay in registers for the whole prompt
    const int pc = tid % P, sg = tid / P;
    const int ch = hd * P + pc;
    float wgt[W];
#pragma unroll
    for (int w = 0; w < W; ++w) wgt[w] = load_io(p.wgt, (size_t)ch * W + w, IO);
    const float cbias = p.bias ? load_io(p.bias, ch, IO) : 0.f;
    // raw conv input of prompt token tg for this channel (bits), from a clamped address: a token before the prompt is
    // replaced by the ring history below, one past the end is zeroed when it is used.  (One base pointer only: a
    // select between two gets compiled into two loads and a select of their results, with a wait on the spot.)
    // Addresses: a base pointer per sequence that is uniform over the workgroup plus a 32-bit element offset from the
    // 24-bit multiplier (the host refuses prompts whose tensors would not fit), so that no load needs 64-bit or
    // quarter-rate integer arithmetic.
    const char *x_b = reinterpret_cast<const char *>(p.x_raw) + (size_t)b * Ls * HP * ES;
    const char *z_b = reinterpret_cast<const char *>(p.z) + (size_t)b * Ls * HP * ES;
    const char *B_b = reinterpret_cast<const char *>(p.Bm) + ((size_t)b * Ls * GN + (size_t)g * N) * ES;
    const char *C_b = reinterpret_cast<const char *>(p.Cm) + ((size_t)b * Ls * GN + (size_t)g * N) * ES;
    const char *dt_b = reinterpret_cast<const char *>(p.dt) + ((size_t)b * Ls * H + hd) * ES;
    auto off = [](int token, int stride, int rest) { return (size_t)(unsigned)(__umul24(token, stride) + rest); };
    auto raw_bits = [&](int tg) {
        const int tc = tg < 0 ? 0 : (tg < L ? tg : L - 1);
        return Vec::load_raw1(x_b, off(tc, HP, ch));
    };
    // the W-1 raw inputs ahead of the prompt (newest last)
    float hist[W - 1];
#pragma unroll
    for (int j = 0; j < W - 1; ++j)
        hist[j] = SEG && c_beg > 0 ? Vec::decode1(raw_bits(c_beg * Q - (W - 1) + j))
                                   : load_io(p.ring, ((size_t)b * p.ring_len + ((conv_head + 1 - (W - 1) + j) & mask)) * HP + ch, IO);
    constexpr int BI = (Q * (N / EV) + 255) / 256;      // 16-byte B (and C) vectors per thread and chunk
    struct Fetch { uint32_t x[QS + W - 1]; uint4 bv[BI], cv[BI]; uint32_t dt; };
    auto prefetch = [&](int c, Fetch &f) {
        const int t0 = c * Q, s0 = sg * QS;
#pragma unroll
        for (int j = 0; j < QS + W - 1; ++j) f.x[j] = raw_bits(t0 + s0 - (W - 1) + j);
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int item = tid + i * 256;
            const int s_ = item / (N / EV), n = (item % (N / EV)) * EV;
            const int tg = t0 + (s_ < Q ? s_ : Q - 1);
            const size_t o = off(tg < L ? tg : L - 1, GN, n);
            f.bv[i] = Vec::load_raw(B_b, o);
            f.cv[i] = Vec::load_raw(C_b, o);
        }
        const int tq = t0 + (tid & (Q - 1));
        f.dt = Vec::load_raw1(dt_b, off(tq < L ? tq : L - 1, H, 0));
    };
    float cum_all = 0.f;                                // SEG, threads 0 .. Q - 1: log of the segment's decay
    auto consume = [&](int c, const Fetch &f) {
        const int t0 = c * Q, s0 = sg * QS;
        float tap[W - 1];
#pragma unroll
        for (int j = 0; j < W - 1; ++j) {
            const int tg = t0 + s0 - (W - 1) + j;       // < 0 only in the prompt's first chunk: -(W-1)+j, i.e. hist[j]
            tap[j] = tg < 0 ? hist[j] : Vec::decode1(f.x[j]);
        }
        float t1 = tap[0], t2 = tap[1], t3 = tap[2];
#pragma unroll
        for (int j = 0; j < QS; ++j) {
            const int tg = t0 + s0 + j;
            const float r = Vec::decode1(f.x[j + W - 1]);
            // same fp32 order and rounding as conv1d_state_update
            float acc = cbias;
            acc = fmaf(wgt[0], t1, acc);
            acc = fmaf(wgt[1], t2, acc);
            acc = fmaf(wgt[2], t3, acc);
            acc = fmaf(wgt[3], r, acc);
            if (p.conv_act == SSMV_ACT_SILU) acc = acc / (1.f + expf(-acc));
            if (IO == SSMV_BF16) acc = bf16_bits_to_f32(f32_to_bf16_bits(acc));
            sX[(s0 + j) * P + pc] = tg < L ? acc : 0.f;
            t1 = t2; t2 = t3; t3 = r;
        }
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int item = tid + i * 256;
            if (item < Q * (N / EV)) {
                const int s_ = item / (N / EV), n = (item % (N / EV)) * EV;
                const bool live = t0 + s_ < L;
                float bv[EV], cv[EV];
                Vec::decode(f.bv[i], bv);
                Vec::decode(f.cv[i], cv);
#pragma unroll
                for (int e = 0; e < EV; e += 4) {
                    *reinterpret_cast<v4f_t *>(sB + s_ * NP + n + e) = live ? v4f_t{bv[e], bv[e + 1], bv[e + 2], bv[e + 3]} : v4f_t{0.f, 0.f, 0.f, 0.f};
                    *reinterpret_cast<v4f_t *>(sC + s_ * NP + n + e) = live ? v4f_t{cv[e], cv[e + 1], cv[e + 2], cv[e + 3]} : v4f_t{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
        if (tid < Q) {
            float d = Vec::decode1(f.dt) + dtb_h;
            if (p.dt_softplus) d = softplus_fast(d);
            if (t0 + tid >= L) d = 0.f;                                                      // padding: no decay, no input
            float v = d * A_h;
#pragma unroll
            for (int off = 1; off < Q; off <<= 1) {
                const float u = __shfl_up(v, off, 64);
                if (tid >= off) v += u;
            }
            const float cq = __shfl(v, Q - 1, 64);
            if constexpr (SEG) cum_all += cq;
            sDt[tid] = d;
            sCum[tid] = v;
            sAt[tid] = expf(v);
            sW[tid] = expf(cq - v) * d;
        }
    };

    Fetch fetch;
    prefetch(c_beg, fetch);
    for (int c = c_beg; c < c_end; ++c) {
        const int t0 = c * Q;
        consume(c, fetch);
        __syncthreads();
        if (c + 1 < c_end) prefetch(c + 1, fetch);
        __builtin_amdgcn_sched_barrier(0);              // the loads stay here, a whole chunk of arithmetic ahead of their use

        // ---- G = C B^T, one 16x16 quadrant per wave, masked and scaled into M; Y <- diag(exp(cum)) C h^T -----------
        if (emit) {
            const int qi = wave >> 1, qj = wave & 1;        // rows t in [16 qi, +16), columns s in [16 qj, +16)
            const int l16 = lane & 15, k4 = lane >> 4;
            const int srow = qj * 16 + l16;
            if (qj <= qi) {                                 // the upper-right quadrant is all s > t
                f4v gacc = {0};
#pragma unroll
                for (int kk = 0; kk < N / 4; ++kk) {
                    const int n = 4 * kk + k4;
                    gacc = __builtin_amdgcn_mfma_f32_16x16x4f32(sC[(qi * 16 + l16) * NP + n], sB[srow * NP + n], gacc, 0, 0, 0);
                }
                const float cs = sCum[srow], ds = sDt[srow];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int t = qi * 16 + 4 * k4 + v;
                    const bool keep = srow <= t;
                    const float dec = expf(keep ? sCum[t] - cs : 0.f);
                    sM[t * QP + srow] = keep ? gacc[v] * dec * ds : 0.f;
                }
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) sM[(qi * 16 + 4 * k4 + v) * QP + srow] = 0.f;
            }
        }
        // The output tile is accumulated TRANSPOSED (rows = the wave's 32 channels, columns = the chunk's tokens): a lane
        // then holds, for its token, runs of four adjacent channels, which leave as 8- or 16-byte stores and meet the
        // gate inputs and the skip term in the same shape, with no trip through LDS.
        f16v yacc = {0};
        if (emit && owns) {                                 // the state registers are the A operand: rows p, contraction over the wave's n
            const float at = sAt[li];                       // on C, not on the sums: these may leave fp32's range where y does not
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4f_t c4 = *reinterpret_cast<const v4f_t *>(sC + li * NP + 32 * (TNL * nh + tn) + 8 * q + 4 * lk);
#pragma unroll
                    for (int e = 0; e < 4; ++e) yacc = __builtin_amdgcn_mfma_f32_32x32x2f32(hacc[tn][4 * q + e], c4[e] * at, yacc, 0, 0, 0);
                }
            if (NSPL > 1 && nh > 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<v4f_t *>(sZ + ((nh - 1) * TP + pt) * 1024 + q * 256 + lane * 4) =
                        v4f_t{yacc[4 * q], yacc[4 * q + 1], yacc[4 * q + 2], yacc[4 * q + 3]};
            }
        }
        // X of the wave's channels, token 2 kk + lk: A operand of X^T M^T, and, weighted, B operand of the state update
        float xop[Q / 2];
#pragma unroll
        for (int kk = 0; kk < Q / 2; ++kk) xop[kk] = sX[(2 * kk + lk) * P + pt * 32 + li];
        if (emit) __syncthreads();     // M is complete, and the shares of C h^T

        // ---- Y^T += X^T M^T, + D X, gate, store ---------------------------------------------------------
        if (emit && nh == 0) {
            const int t = li;                                   // this lane's token within the chunk
            const bool live = t0 + t < L;
            const int tc = live ? t0 + t : L - 1;
            using QV = XVec<IO, 4>;                             // four adjacent channels in the I/O type
            typename QV::Raw zraw[4];
            if (gated) {                                        // requested ahead of the matrix products
#pragma unroll
                for (int q = 0; q < 4; ++q) zraw[q] = QV::load(z_b, off(tc, HP, hd * P + pt * 32 + 8 * q + 4 * lk));
            }
#pragma unroll
            for (int u = 0; u < NSPL - 1; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4f_t z4 = *reinterpret_cast<const v4f_t *>(sZ + (u * TP + pt) * 1024 + q * 256 + lane * 4);
                    yacc[4 * q] += z4.x; yacc[4 * q + 1] += z4.y; yacc[4 * q + 2] += z4.z; yacc[4 * q + 3] += z4.w;
                }
#pragma unroll
            for (int kk = 0; kk < Q / 2; ++kk) yacc = __builtin_amdgcn_mfma_f32_32x32x2f32(xop[kk], sM[li * QP + 2 * kk + lk], yacc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int pl = pt * 32 + 8 * q + 4 * lk;        // first of the four channels (inside the head)
                const v4f_t xs = *reinterpret_cast<const v4f_t *>(sX + t * P + pl);
                float yv[4] = {fmaf(D_h, xs.x, yacc[4 * q + 0]), fmaf(D_h, xs.y, yacc[4 * q + 1]), fmaf(D_h, xs.z, yacc[4 * q + 2]),
                               fmaf(D_h, xs.w, yacc[4 * q + 3])};
                if (gated) {
                    float zf[4];
                    QV::decode(zraw[q], zf);
#pragma unroll
                    for (int e = 0; e < 4; ++e) yv[e] *= silu_fast(zf[e]);
                }
                if (live) QV::store(y_b, off(t0 + t, HP, hd * P + pl), QV::encode(yv));
            }
        }
        // ---- h^T <- exp(cum_Q) h^T + B^T (diag(w) X), in the registers ------------------------------------------
        if (owns) {
            const float aq = sAt[Q - 1];
#pragma unroll
            for (int kk = 0; kk < Q / 2; ++kk) xop[kk] *= sW[2 * kk + lk];
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn) {
                // the chunk's own sum first, then ONE rounding against the state: accumulated straight into it, its sixteen
                // partial sums are rounded at the state's size (state error 2.3e-7 instead of 1.3e-7 under a slow decay)
                f16v sacc = {0};
#pragma unroll
                for (int kk = 0; kk < Q / 2; ++kk)
                    sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(sB[(2 * kk + lk) * NP + 32 * (TNL * nh + tn) + li], xop[kk], sacc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 16; ++v) hacc[tn][v] = fmaf(aq, hacc[tn][v], sacc[v]);
                if constexpr (TNL >= 4) __builtin_amdgcn_sched_barrier(0);       // one tile's sum at a time (128 x 128 spills 4 registers so, 7 cut)
            }
        }
        __syncthreads();     // the next chunk overwrites X, B, C, M
    }

    if constexpr (SEG) {
        if (!seg.last) {
            if (p.seg_pass == 1) return;                // the next segment has its state already
            // a segment's state on its way to the combining launch
            if (owns) {
#pragma unroll
                for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *seg_at(tn, q) = make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
            }
            if (c_beg > 0 && tid == 0) *reinterpret_cast<float *>(y_b + seg_piece<ES>(P * N / 4, P, seg.area, HP, hd)) = cum_all * 1.4426950408889634f;
            return;
        }
    }
    // ---- state back in place; the newest W-1 raw inputs into the ring behind conv_head -----------------------
    if (owns) {
#pragma unroll
        for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4 *>(state_at(tn, q)) = make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
    }
    if (tid < P) {
        for (int tg = (L - (W - 1) > 0 ? L - (W - 1) : 0); tg < L; ++tg)
            Vec::store_raw1(p.ring, ((size_t)b * p.ring_len + ((conv_head + 1 + tg) & mask)) * HP + ch, raw_bits(tg));
    }
}

// pos += L, conv_head += L; a prefill on a cache with pending tokens or an uncommitted verify is a sequencing error
__device__ __forceinline__ void finish_sequence(const PrefillParams &p, int b)
{
    const int L = p.seq_len ? min(max(p.seq_len[b], 0), p.L) : p.L;
    if (p.pend[b] != 0 || p.last_k[b] != 0) *p.err_flag = 1;
    p.pos[b] += L;
    p.conv_head_rw[b] = (p.conv_head_rw[b] + L) & (p.ring_len - 1);
}

__global__ void prefill_finish_kernel(const PrefillParams p)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < p.batch) finish_sequence(p, b);
}

// Between the two passes of a segmented prompt: (u, d) of the segments -> the states ahead of them, in place, one thread per
// 16 bytes of a state (an element only ever meets itself).  grid = (P N / 1024, H, batch).  The loads of up to eight
// segments are under way together: as a chain of load, multiply-add and store per segment it would be that many round
// trips to memory long.
template <int ES>
__global__ __launch_bounds__(256) void prefill_combine_kernel(const PrefillParams p)
{
    const int hd = blockIdx.y, b = blockIdx.z, i = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 0 && hd == 0 && threadIdx.x == 0) finish_sequence(p, b);
    const int L = p.seq_len ? min(max(p.seq_len[b], 0), p.L) : p.L;
    if (L == 0) return;
    const int n = (L + kPrefillChunk - 1) / kPrefillChunk, ns = segments_of(p.seg_chunks, n), HP = p.H * p.P;
    if (ns < 3) return;                                  // one segment: done; two: the state ahead of the second is in its place already
    char *y_b = static_cast<char *>(p.y) + (size_t)b * p.L * HP * ES;
    auto area = [&](int s, int piece) { return y_b + seg_piece<ES>(piece, p.P, segment_begin(p.seg_chunks, n, s) * kPrefillChunk, HP, hd); };
    constexpr int U = 8;
    v4f_t h = *reinterpret_cast<const v4f_t *>(area(ns - 1, i));       // the state behind segment 0
    for (int s0 = 1; s0 < ns - 1; s0 += U) {
        v4f_t u[U];
        float d[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int s = min(s0 + j, ns - 2);
            u[j] = *reinterpret_cast<const v4f_t *>(area(s, i));
            d[j] = *reinterpret_cast<const float *>(area(s, p.P * p.N / 4));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (s0 + j < ns - 1) {
                *reinterpret_cast<v4f_t *>(area(s0 + j, i)) = h;
                const float a = __builtin_amdgcn_exp2f(d[j]);
                h.x = fmaf(a, h.x, u[j].x); h.y = fmaf(a, h.y, u[j].y); h.z = fmaf(a, h.z, u[j].z); h.w = fmaf(a, h.w, u[j].w);
            }
        }
    }
    *reinterpret_cast<v4f_t *>(area(ns - 1, i)) = h;
}

// fp32 tensors only: bf16 tensors take the bf16 matrix cores (prefill_bf16.hip)
template <int P, int N, bool SEG>
static int launch_pn(const PrefillParams &p, hipStream_t stream)
{
    const size_t lds = F32Shape<P, N>::floats * sizeof(float);
    const dim3 grid((unsigned)(p.H * p.batch) * (SEG ? p.seg_count - 1 : 1)), block(256);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&prefill_kernel<P, N, SSMV_F32, SEG>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL((prefill_kernel<P, N, SSMV_F32, SEG>), grid, block, lds, stream, p);
    return (int)hipGetLastError();
}

template <int P>
static int launch_p(const PrefillParams &p, hipStream_t stream)
{
    switch (p.N) {
        case 32: return p.seg_count ? launch_pn<P, 32, true>(p, stream) : launch_pn<P, 32, false>(p, stream);
        case 64: return p.seg_count ? launch_pn<P, 64, true>(p, stream) : launch_pn<P, 64, false>(p, stream);
        case 128:
            if constexpr (P > 32) if (p.seg_count) return launch_pn<P, 128, true>(p, stream);      // (plan_f32)
            return launch_pn<P, 128, false>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

// workgroups that fit a compute unit side by side: one wave per SIMD each, two or three of them by their registers
template <int P, int N>
static constexpr int resident()
{
    constexpr int by_lds = 160 * 1024 / (F32Shape<P, N>::floats * 4), by_registers = P * N <= 4096 ? 3 : 2;
    return by_lds < by_registers ? by_lds : by_registers;
}
static int resident_f32(int P, int N)
{
    auto pick = [&](int n32, int n64, int n128) { return N == 32 ? n32 : N == 64 ? n64 : n128; };
    if (P == 32) return pick(resident<32, 32>(), resident<32, 64>(), resident<32, 128>());
    if (P == 64) return pick(resident<64, 32>(), resident<64, 64>(), resident<64, 128>());
    return pick(resident<128, 32>(), resident<128, 64>(), resident<128, 128>());
}

bool prefill_shape_supported(int P, int N)
{
    return (P == 32 || P == 64 || P == 128) && (N == 32 || N == 64 || N == 128);
}

// What a cut costs a kernel.  The unit of time is one chunk of a workgroup that has its compute unit to itself.
struct CutCosts {
    int resident;        // workgroups that fit a compute unit side by side
    double company;      // with all of them there a chunk takes 1 + company, linearly less below; five and more are counted as four
    double share;        // a chunk of a segment's share of the state alone
    double launches;     // the two further launches
    double trip;         // a segment's state through memory, four times
    double worth;        // asked for: this much of the uncut time at most
};

// The segments of a prompt, or none.  More workgroups than fit at once would run as a second round, which always lost (320 heads x 1500
// tokens at 128 x 64: 150 us cut in three, 118 us uncut): not cut.
// Returns the time of the cut, in units.
static double choose_segments(PrefillParams &p, const CutCosts &k)
{
    constexpr int kCUs = 256;
    const long pairs = (long)p.batch * p.H;
    const int n = (p.L + kPrefillChunk - 1) / kPrefillChunk;
    // the last segment may end with a chunk of one token, and has to hold a state in its rows
    const int shortest = (4 * p.N / (p.io == SSMV_BF16 ? 2 : 4) + kPrefillChunk - 1 + kPrefillChunk - 1) / kPrefillChunk;
    const int r = k.resident;
    auto chunk_time = [&](long wgs) { return r > 1 ? 1.0 + k.company * ((wgs + kCUs - 1) / kCUs - 1) / ((r < 4 ? r : 4) - 1) : 1.0; };
    p.seg_chunks = p.seg_count = 0;
    double best = k.worth * n * chunk_time(pairs);
    const long most = kCUs * r / pairs + 1 < segments_of(shortest, n) ? kCUs * r / pairs + 1 : segments_of(shortest, n);
    for (int ns = (int)most; ns >= 3; --ns) {
        // the segment lengths l that make ns segments; the time max(n - (ns - 1) l, share l) + l falls and then rises with l
        int lo = (n - 1) / ns + 1, hi = (n - 1) / (ns - 1);
        if (lo < shortest) lo = shortest;
        if (hi < lo) continue;
        const int turn = (int)(n / (ns - 1 + k.share));
        for (int l = turn; l <= turn + 1; ++l) {
            const int len = l < lo ? lo : l > hi ? hi : l, first = n - (ns - 1) * len;
            const double t = ((first > k.share * len ? first : k.share * len) + len) * chunk_time(pairs * (ns - 1)) + k.launches + k.trip * pairs * (ns - 1);
            if (t < best) { best = t; p.seg_chunks = len; p.seg_count = ns; }
        }
    }
    return best;
}

// Whether a bf16 prompt that the pipelined kernel would take whole or cut is cut by the other kernel instead.  That one fits more workgroups
// (prefill_bf16_resident), so that it can cut a prompt into more segments where the pipelined kernel has room for a few or none: worth it
// from so many tokens on, between two numbers of (sequence, head) pairs.  Lines from times of both at 260 to 4096 tokens, 4 to 512
// pairs, prompts of one length and of different ones (drawn from 1 up).  The pipelined kernel's choice, this one's (us):
//   one length  128 x 32  96 pairs, 4096 tokens: 104, 74;  144, 3000: 104, 88     64 x 32  176, 3000: 89, 66
//               32 x 32  288, 4096: 110, 83                                       32 x 128  384, 4096: 319, 253
//   different   128 x 32  80, 4096: 95, 60;  96, 1500: 56, 38     64 x 32  176, 4096: 118, 75     32 x 32  288, 4096: 113, 74     32 x 128  96, 3000: 96, 76
//   outside     128 x 32  192, 4096: 140, 152;  208, 1024: 43, 51   64 x 32  352, 3000: 106, 126    32 x 128  288, 3000, different: 113, 189
static bool prefill_bf16_cuts(const PrefillParams &p)
{
    if (!prefill_bf16_resident(p.P, p.N)) return false;
    const long pairs = (long)p.batch * p.H;
    auto between = [&](int tokens, int from, int to) { return p.L >= tokens && pairs >= from && pairs <= to; };
    if (p.seq_len) {
        if (p.P == 32) return p.N == 32 ? between(1500, 112, 256) || between(2048, 80, 384) : between(3000, 64, 144);
        return p.P == 64 ? between(1024, 80, 224) : between(1024, 80, 144) || between(1500, 32, 208);
    }
    if (p.P == 32) return p.N == 32 ? between(3000, 112, 448) : between(1500, 288, 384) || between(3000, 80, 192);
    return p.P == 64 ? between(2048, 144, 256) : between(1500, 48, 176);
}

// y carries states between the launches of a cut prompt: not if it overlaps anything that is still to be read
static bool y_is_apart(const PrefillParams &p)
{
    const int es = p.io == SSMV_BF16 ? 2 : 4;
    const char *y0 = static_cast<const char *>(p.y), *y1 = y0 + (size_t)p.batch * p.L * p.H * p.P * es;
    auto overlaps = [&](const void *t, size_t bytes) {
        const char *a = static_cast<const char *>(t);
        return a && a < y1 && y0 < a + bytes;
    };
    const size_t tok = (size_t)p.batch * p.L, ch = (size_t)p.H * p.P;
    return !(overlaps(p.x_raw, tok * ch * es) || overlaps(p.z, tok * ch * es) || overlaps(p.dt, tok * p.H * es) ||
             overlaps(p.Bm, tok * p.G * p.N * es) || overlaps(p.Cm, tok * p.G * p.N * es) || overlaps(p.wgt, ch * SSMV_CONV_WIDTH * es) ||
             overlaps(p.bias, ch * es) || overlaps(p.A, p.H * sizeof(float)) || overlaps(p.D, p.H * sizeof(float)) ||
             overlaps(p.dt_bias, p.H * sizeof(float)) || overlaps(p.seq_len, p.batch * sizeof(int32_t)));
}

// Whether and how a bf16 prompt is cut, and by which kernel: the return value says whether by the pipelined one.
// Uncut and cut (us; one sequence unless said):
//   128 x 64, 32 heads:  700 tokens 29 -> 26, 1500: 54 -> 34, 3000: 100 -> 41;  4 sequences, 3000: 99 -> 85;  8 heads, 1500: 52 -> 24
//   64 x 128, 80 heads:  1500 tokens 69 -> 52, 3000: 130 -> 78;   64 x 64, 80 heads, 1500: 48 -> 37
// Over nine tiles, 4 to 512 pairs and 260 to 4096 tokens of one length: never more than 4 % slower than uncut, 13 % faster on average.  Of
// prompts of different lengths only the device knows them: one sequence that is far shorter than L pays for the launches (32 heads of
// 128 x 64, 700 tokens given, one there: 8 -> 11 us).
static bool plan_bf16(PrefillParams &p)
{
    p.seg_chunks = p.seg_count = 0;
    if (!prefill_pipe_serves(p)) return false;
    if (!y_is_apart(p)) return true;
    if (prefill_bf16_cuts(p)) {                          // unit 1.3 to 2.4 us; of full compute units 1.5 of it, the launches with the states' trips 5
        choose_segments(p, {prefill_bf16_resident(p.P, p.N), 0.5, 0.6, 5.0, 0.0, 0.85});
        if (p.seg_count) return false;
    }
    // with SiLU (us)  4 heads of 128 x 64, 550 tokens: 37 uncut, 27 cut;  48 pairs of 128 x 32, 550: 35, 28;  of lengths that differ as many
    // calls lost by it as gained (96 pairs of 64 x 128, 1024 at most: 54, 64)
    // the launches 8 us, the states' trips at 4.7 TB/s
    const double unit = prefill_pipe_chunk_us(p.P, p.N, p.conv_act == SSMV_ACT_SILU && !p.seq_len);
    choose_segments(p, {prefill_pipe_resident(p.P, p.N), 0.3, 0.5, 8.0 / unit, 4.0 * p.P * p.N * sizeof(float) / 4.7e6 / unit, 0.9});
    return true;
}

// fp32: which kernel, into how many parts a head goes (the pipelined kernel only, prefill_f32_pipe.hip), and whether and how the prompt
// is cut: what a model of the times says is fastest.  The model's figures are the times of both kernels at 512 tokens, 64 to 1024 pairs; those
// of several rounds of the pipelined one, and of a cut's launches, are the ones whose choices over 2148 measured calls took the least time (nine
// tiles, 20 to 2048 pairs, 24 to 3000 tokens, with and without SiLU, gate and softplus).  Time of the choice over the other kernel's, whole or cut, mean
// and slowest: 900 calls of 20 to 1300 pairs, one length 0.83, 1.04, lengths that spread 0.78, 1.08, lengths given and all the same 0.86, 1.27;
// 1248 calls of 512 to 2048 pairs 0.93, 1.05;  0.91, 1.06;  0.93, 1.21.
// Up to the (sequence, head) pairs at which the other kernel has two workgroups on every compute unit the pipelined one is the faster, with
// as many parts as the chip has room for; in large launches those of its shapes whose products outweigh the start of each round.
// us with the other kernel alone -> with this choice, one length, one sequence unless said:
//   128 x 64, 32 heads:   4 sequences, 512 tokens 78 -> 45, 1021: 126 -> 81;  8, 512: 101 -> 74;  12: 144 -> 114
//                         16, 700: 226 -> 219, with SiLU, gate and softplus 264 -> 231;  32, 2000: 1126 -> 1072, 1347 -> 1167
//   128 x 128, 32 heads:  4 sequences, 512 tokens 116 -> 70;  12: 222 -> 186;  16: 232 (the other; this one 256)
//   64 x 128, 80 heads:   8 sequences, 512 tokens 237 -> 185;   64 x 64, 80 heads: 2 sequences, 1024 tokens 107 -> 78
// A conv SiLU, a gate and a softplus are not in it: they cost the other kernel more than the pipelined one, which has other waves for the
// first and the last.
// Lengths that are given are the device's to know: they may spread from 1 up or all be the longest, and what is fast for the one can be slow
// for the other (22 x 7 x 64 x 32, 2324 tokens, all that long: two parts 306 us, the other kernel 182).  The fastest for lengths that spread is
// taken of what loses at most kLoss times as much (and kSlack) where all are equal as it gains there.  Without that condition the choice lost up
// to 69 % on equal lengths; with it up to 27 % (10 x 57 x 32 x 32, 340 tokens, 70 -> 90 us;  16 x 32 x 128 x 128, 2000 tokens, 882 -> 1013, for 715 -> 568
// where they spread); at kLoss = 1 it gives up too much on lengths that spread (24 x 30 x 32 x 32, 2364 tokens at most, SiLU: 313 us, 208 at 2).
static bool plan_f32(PrefillParams &p)
{
    // per chunk (us): the other kernel with a compute unit to itself, what company adds to it (CutCosts), the pipelined kernel in a launch of
    // one round of workgroups, and in each of several
    struct Times { double unit, company, pipe, pipe_rounds; };
    constexpr Times kTimes[3][3] = {{{3.5, 0.21, 1.6, 1.78}, {4.0, 0.43, 1.85, 1.90}, {4.7, 0.32, 2.35, 2.25}},
                                    {{3.7, 0.60, 2.0, 2.23}, {4.4, 0.65, 2.20, 2.01}, {5.9, 0.50, 3.75, 3.98}},
                                    {{4.3, 0.50, 2.95, 2.50}, {5.7, 0.56, 3.7, 3.76}, {8.5, 0.64, 0.0, 0.0}}};
    auto times = [&](int P, int N) { return kTimes[P == 32 ? 0 : P == 64 ? 1 : 2][N == 32 ? 0 : N == 64 ? 1 : 2]; };
    constexpr double kStart = 6.5, kStartPipe = 7.5, kTurn = 2.0, kLaunches = 8.0;      // of a launch, of a further round of workgroups, of a cut prompt's two further launches
    // of lengths that spread: several rounds of the pipelined kernel (the last workgroups have the chip to themselves), a prompt that the other
    // kernel cuts (the long sequences' segments share compute units while others rest)
    constexpr double kSpread = 1.2, kCutSpread = 1.15;
    constexpr double kLoss = 2.0, kSlack = 2.5;          // (us: the model is not better than that)
    constexpr int kCUs = 256;
    const int n = (p.L + kPrefillChunk - 1) / kPrefillChunk, r = resident_f32(p.P, p.N);
    const bool may_cut = y_is_apart(p);
    // of lengths that spread: the first sequence's and half of the others' chunks, the longest alone at its end
    const double half = 0.05 + (1.0 + (p.batch - 1) * 0.5 * (n + 1) / n) / p.batch;
    auto rounds = [&](double mean, double first, double all) { return mean * all < first ? first : mean * all; };
    p.seg_chunks = p.seg_count = 0;
    const PrefillParams whole = p;
    const Times k = times(p.P, p.N);
    const long wgs = (long)p.batch * p.H, rest = wgs % (kCUs * r);
    auto shared = [&](long w) { return r > 1 ? 1.0 + k.company * ((w + kCUs - 1) / kCUs - 1) / (r - 1) : 1.0; };
    struct Cost { double same, spread; };                // of one length, of lengths that spread
    // the other kernel, whole or cut
    const double first = shared(wgs < kCUs * r ? wgs : kCUs * r), all = wgs / (kCUs * r) * shared(kCUs * r) + (rest ? shared(rest) : 0.0);
    Cost other = {kStart + n * k.unit * rounds(1.0, first, all), kStart + n * k.unit * rounds(half, first, 0.5 * (all + wgs / (double)(kCUs * r) * shared(kCUs * r)))};
    if (may_cut && !(p.P == 32 && p.N == 128)) {         // (of 32 x 128 the pipelined kernel's is always the faster)
        const double t = kStart + k.unit * choose_segments(p, {r, k.company < 0.5 ? k.company : 0.5, 0.5, 1.5, 0.0, 0.85});
        if (p.seg_count) other = {t, kCutSpread * t};
    }
    bool pipe = false;
    double best = p.seq_len ? other.spread : other.same;
    auto better = [&](const PrefillParams &q, Cost t) {
        const double at = p.seq_len ? t.spread : t.same;
        const bool safe = !p.seq_len || t.same - other.same - kSlack <= kLoss * (other.spread - t.spread);
        if (at < best && safe) { best = at; p = q; pipe = true; }
    };
    for (int parts = 1; whole.P / parts >= 32; parts *= 2) {
        PrefillParams q = whole;
        q.parts = parts;
        q.H *= parts;
        q.P /= parts;
        if (q.P == 128 && q.N == 128) continue;          // never the fastest: its waves lack registers
        const double unit = times(q.P, q.N).pipe, turns = (wgs * parts + kCUs - 1) / kCUs;
        auto time = [&](double mean, double turns) {
            return kStartPipe + n * (turns > 1.0 ? times(q.P, q.N).pipe_rounds : unit) * rounds(mean, 1.0, turns) + kTurn * (turns - 1.0);
        };
        // of lengths that spread a workgroup starts as another ends
        const double spread = turns > 1.0 ? kSpread * time(half, n > 1 ? wgs * parts / (double)kCUs : turns) : time(half, turns);
        better(q, {time(1.0, turns), spread});
        if (may_cut) {
            const double t = kStartPipe + unit * choose_segments(q, {1, 0.0, 0.6, kLaunches / unit, 4.0 * q.P * q.N * sizeof(float) / 4.7e6 / unit, 0.9});
            if (q.seg_count) better(q, {t, t});
        }
    }
    return pipe;
}

static int launch_pass(const PrefillParams &p, bool pipe, hipStream_t stream)
{
    if (p.io == SSMV_BF16) return pipe ? launch_prefill_pipe(p, stream) : launch_prefill_bf16(p, stream);
    if (pipe) return launch_prefill_f32_pipe(p, stream);
    switch (p.P) {
        case 32: return launch_p<32>(p, stream);
        case 64: return launch_p<64>(p, stream);
        case 128: return launch_p<128>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

int launch_prefill(const PrefillParams &p_in, hipStream_t stream)
{
    PrefillParams p = p_in;
    p.parts = 1;
    p.seg_pass = 0;
    const bool pipe = p.io == SSMV_BF16 ? plan_bf16(p) : plan_f32(p);
    int rc = launch_pass(p, pipe, stream);
    if (rc != 0) return rc;
    if (p.seg_count) {
        const dim3 grid(p.P * p.N / 1024, p.H, p.batch);
        if (p.io == SSMV_BF16) hipLaunchKernelGGL(prefill_combine_kernel<2>, grid, dim3(256), 0, stream, p);
        else hipLaunchKernelGGL(prefill_combine_kernel<4>, grid, dim3(256), 0, stream, p);
        if ((rc = (int)hipGetLastError()) != 0) return rc;
        p.seg_pass = 1;
        return launch_pass(p, pipe, stream);
    }
    hipLaunchKernelGGL(prefill_finish_kernel, dim3((p.batch + 63) / 64), dim3(64), 0, stream, p);
    return (int)hipGetLastError();
}

}  // namespace ssmv
