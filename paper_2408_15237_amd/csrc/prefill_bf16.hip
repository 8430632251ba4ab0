// Chunked prefill for bf16 tensors on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16, 16 times the fp32 MFMA rate).
// Same evaluation of Section 2.1 Eq. 1 (discretisation of Section 2.2) as prefill.hip, chunk by chunk:
//   G = C B^T,  M_ts = G_ts exp(cum_t - cum_s) dt_s (s <= t) + [s = t] D,
//   Y = M X + diag(exp(cum_t)) C h^T,   h <- exp(cum_Q) h + X^T diag(w) B,   w_s = exp(cum_Q - cum_s) dt_s,
// with the operands arranged so that fp32 accuracy survives the 8-bit mantissa of the multiplier inputs:
//   * B, C and the conv output X ARE bf16 (the tensors' storage type; the conv output is rounded to it by
//     definition), so they enter exactly;
//   * the fp32 operand of the product that UPDATES THE STATE (the weighted rows w_s B_s) is split into a bf16 head and a
//     bf16 tail, v = hi + lo + O(2^-17 |v|), and contributes two products into the same fp32 accumulator: the state
//     carries over the whole prompt and stays at fp32 accuracy;
//   * the fp32 operands of the two products that end in OUTPUTS only (the state h in h C^T, the masked matrix M in M X)
//     enter as their bf16 head alone: a relative 2^-9 per term, the size of the rounding the outputs get anyway when
//     they are stored as bf16, and nothing of it feeds back into the state.  (Their tails cost a fifth of the kernel's
//     vector and matrix instructions: 0.41 -> 0.36 ms for 32 x 2048 tokens of a 32 x 128 x 64 layer; the largest output
//     error against the fp64 scan went from 0.0058 to 0.0075 of the largest output.)
// One workgroup owns one (sequence, head); wave w owns the 32 channels [32 w, 32 w + 32).  The state lives in the
// accumulator registers for the whole prompt, TRANSPOSED (tile rows = state index n, columns = channel p): in that
// shape the registers of a lane (its channel, 16 of the 32 n of a tile) are directly the k-slots of the A operand of
// h C^T, so the state never visits LDS; the result tile comes out as [channel][token], a lane holding runs of four
// adjacent channels of its token (the wave turns the tile through a patch of LDS of its own into 64-byte rows for the
// stores).  G^T comes in 16 x 16 quadrants on v_mfma_f32_16x16x32_bf16: the three that are not above the diagonal go round the
// waves, each finishes its own into M^T (mask, decay, dt_s, D on the diagonal) and shares it through LDS.
// What a chunk costs is its instructions, vector ones above all (two waves per SIMD, neither the matrix pipe nor LDS nor memory
// more than half busy).  So: raw inputs and B leave LDS through the transposing read (read_tr16), four tokens of a channel per lane
// and instruction, already paired for the conv's dot products; the addend of those is an operand (conv8); G is computed once, not by
// every wave; lane offsets of all global accesses stay the same over the chunks.  With single 16-bit
// LDS reads, pairs put together by shifts, G in every wave and 64-bit addresses formed per access a
// wave took 334 vector, 18 matrix and 67 LDS instructions per chunk at 128 x 64 (no SiLU; counters, start and end of a prompt included), so
// 237, 15.5 and 42.
// 32 x 2048 tokens of 32 heads x 128 x 64: 348 -> 298 us; 16 x 1024: 64 heads x 32 x 64 102 -> 83, 64 x 32 x 32 73 -> 58.
// Operand layout (checked on the hardware): A[i = lane%32][k = 8 (lane/32) + j], B[k = 8 (lane/32) + j][col = lane%32],
// j = 0..7 the elements of the lane's 16-byte operand; result register v of a lane is row 8 (v/4) + 4 (lane/32) + v%4,
// column lane%32.  Registers 8 st .. 8 st + 7 of a result tile, used as the operand of step st of a following
// product, are therefore rows 16 st + 8 (j/4) + 4 (lane/32) + j%4.  Rows of the state tiles (the index n) are stored
// under the permutation "swap bits 2 and 3" of the row index: then those eight registers hold the CONSECUTIVE indices
// 16 st + 8 (lane/32) + j, and the other operand of h C^T is one 16-byte LDS read; X serves M X and the update with
// one read.
// The chunk's raw x, B and C rows travel from global memory straight into LDS (no registers, 1 KB per wave and
// instruction), one chunk ahead: they are requested right after the barrier that ends the staging of chunk c, land
// during its arithmetic, and the barrier at its end publishes them.
// LDS rows that the kernel writes itself are padded by 16 bytes: a row stride that is an odd multiple of 16 bytes
// spreads 16-byte reads of consecutive rows over all banks; the rows of B and C, which the direct loads fill without
// gaps, have their 16-byte pieces XOR-swizzled instead (by the choice of the global address each lane fetches).
#include "prefill_bf16_ops.h"
#include "prefill_split.h"

namespace ssmv {
namespace {

constexpr int kQ = kPrefillChunk;

__host__ __device__ constexpr bool cuts(int P, int N) { return N == 32 || (P == 32 && N == 128); }      // see prefill_bf16_resident

template <int P, int N>
struct PfLds {              // byte offsets of the LDS arrays (bf16 unless said)
    static constexpr int XS = kQ * 2 + 16;                 // row stride of the arrays indexed [..][token]
    static constexpr int NP = P / 32;                      // 32-channel tiles of the head
    static constexpr int NSPL = prefill_nsplit(P, N);
    static constexpr int NW = NP * NSPL;                   // waves
    static constexpr int oX = 0;                           // [P][Q]  conv output x_s
    static constexpr int oBh = oX + P * XS;                // [N][Q]  head of w_s B_s, transposed
    static constexpr int oBl = oBh + N * XS;               // [N][Q]  tail of w_s B_s, transposed
    static constexpr int oMh = oBl + N * XS;               // [Q][Q]  M^T, rows t (rounded to bf16: it only feeds outputs)
    static constexpr int YS = 32 * 2 + 16;                 // row stride of a wave's output tile [token][32 channels]
    static constexpr int oY = oMh + kQ * XS;               // [NP][Q][32]  the output tiles, for stores of whole 64-byte rows
    // filled by loads that go from global memory straight into LDS (1 KB per wave and instruction, lane l at byte 16 l):
    static constexpr int YT = kQ * YS + 64;                // stride of the tiles: a row of all tiles then covers the banks
    static constexpr int oZ = oY + NP * YT;           // fp32 [NP][16][64]  h C^T over the second half of n, for the tile's first wave
    static constexpr int oXraw = oZ + (NSPL - 1) * NP * 4096;        // [Q][P]  raw conv inputs of the chunk, rows of 2 P bytes
    static constexpr int BCS = kQ * N * 2;                 // one copy of B or C: [Q][N], rows of 2 N bytes, 16-byte pieces swizzled
    // Two copies of B and C (chunks alternate; the next chunk's are requested at the start of this one's arithmetic) where
    // that does not cost a workgroup per CU; else one copy, and the next chunk's B and C are requested only once this
    // chunk's have been read (after the barrier in the middle): narrow heads (few waves per workgroup: 48 KB -> 40 KB
    // is a fourth workgroup per CU).
    static constexpr int BCC = P >= 128 ? 2 : 1;
    static constexpr int oB = oXraw + kQ * P * 2;
    static constexpr int oC = oB + BCC * BCS;
    static constexpr int oCar = oC + BCC * BCS;              // [2][P][4]  the last four raw inputs of a chunk, for the next one's conv
    static constexpr int oCum = oCar + 2 * P * 8;          // fp32 [NW][Q]  log2 e times the inclusive prefix of dt*A (a copy per wave)
    static constexpr int oDt = oCum + NW * kQ * 4;         // fp32 [NW][Q]  dt
    static constexpr int oW = oDt + NW * kQ * 4;           // fp32 [NW][Q]  exp(cum_Q - cum_s) dt_s
    static constexpr int total = oW + NW * kQ * 4;
    static constexpr int PIECES = N / 8;
};

}  // namespace

// Two waves per SIMD (256 registers each, and then the compiler keeps the accumulators in ordinary registers: no copies
// between the two register files around every use).  The tile of 128 x 128 is not built: prefill_pipe.hip takes all of it.
// A state of N = 128 under a narrow head (P <= 64) is split over two waves per 32-channel tile, each with half of n: the
// second adds its share of h C^T through LDS, both update their own half of the state, and the workgroup has twice the
// threads for the staging.
// SEG: the workgroup owns one segment of the prompt instead of all of it (prefill_split.h); in the first pass of such a
// prompt every segment but the first one only needs its share of the state: no C, no Q x Q product, no outputs, and one
// barrier less per chunk.
// SILU: of the conv.  As a branch on the argument its code cost the launches without it 3 % (32 x 2048 tokens of 32 heads x 128 x 64).
template <int P, int N, bool SEG, bool SILU>
__global__ __launch_bounds__(2 * P * prefill_nsplit(P, N)) __attribute__((amdgpu_waves_per_eu(2)))
void prefill_bf16_kernel(const PrefillParams p)
{
    using Ld = PfLds<P, N>;
    constexpr int Q = kQ;
    constexpr int W = SSMV_CONV_WIDTH;
    constexpr int NSPL = Ld::NSPL;
    constexpr int NT = 2 * P * NSPL;     // threads: one wave per 32 channels (and per half of n where the state is split)
    constexpr int TN = N / 32;
    constexpr int TNL = TN / NSPL;       // state tiles of a wave
    constexpr int QS = Q * P / NT;       // consecutive tokens one thread convolves per chunk (NT / P threads per channel)
    constexpr int XS = Ld::XS, PIECES = Ld::PIECES;
    using Vec = IoVec<SSMV_BF16>;
    static_assert(P % 32 == 0 && P <= 128 && N % 32 == 0 && W == 4, "tile shapes");

    extern __shared__ float4 lds_raw[];
    char *lds = reinterpret_cast<char *>(lds_raw);
    char *sX = lds + Ld::oX, *sBh = lds + Ld::oBh, *sBl = lds + Ld::oBl, *sMh = lds + Ld::oMh, *sXraw = lds + Ld::oXraw;
    uint2 *sCar = reinterpret_cast<uint2 *>(lds + Ld::oCar);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    SSMV_TRACE_BEGIN();
    const int li = lane & 31, lh = lane >> 5;           // MFMA: row/column index and k half of this lane
    const int lperm = swap23(li);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int pt = Ld::NSPL == 1 ? wave_u : wave_u % Ld::NP;   // the wave's 32-channel tile
    const int nh = Ld::NSPL == 1 ? 0 : wave_u / Ld::NP;        // and its half of n (0 unless the state is split)
    char *sY = lds + Ld::oY + pt * Ld::YT;
    float *sCum = reinterpret_cast<float *>(lds + Ld::oCum) + wave * Q;
    float *sDt = reinterpret_cast<float *>(lds + Ld::oDt) + wave * Q;
    float *sW = reinterpret_cast<float *>(lds + Ld::oW) + wave * Q;
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
    const float A2_h = p.A[hd] * kLog2e, D_h = p.D[hd];
    const float dtb_h = p.dt_bias ? p.dt_bias[hd] : 0.f;
    const bool gated = p.z != nullptr;
    float *state = p.state + (size_t)cur * p.slot_stride + ((size_t)b * H + hd) * P * N;

    char *y_b = reinterpret_cast<char *>(p.y) + (size_t)b * Ls * HP * 2;
    // a segment's state between the passes: the lane's float4 number q of tile tn in the rows of y from the segment's area on
    auto seg_at = [&](int tn, int q) {
        return reinterpret_cast<float4 *>(y_b + seg_piece<2>(((wave_u * TNL + tn) * 4 + q) * 64 + lane, P, seg.area, HP, hd));
    };
    // state -> accumulator registers, transposed tiles [n][p]: register 4 q + e of tile tn holds
    // h[p = 32 pt + li][n = 32 (TNL nh + tn) + 16 (q/2) + 8 lh + 4 (q%2) + e]
    f16v hacc[TNL];
    // (row, first column) of the lane's float4 number q of tile tn; the slot is row-major or tiled (state_off4)
    const int srow_ = pt * 32 + li, scol0 = 32 * TNL * nh + 8 * lh;
    auto state_at = [&](int tn, int q) { return state + state_off4(p.tiled, srow_, scol0 + 32 * tn + 16 * (q / 2) + 4 * (q % 2), N); };
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!SEG || c_beg == 0) v = *reinterpret_cast<const float4 *>(state_at(tn, q));
            else if (p.seg_pass == 1) v = *seg_at(tn, q);
            hacc[tn][4 * q + 0] = v.x; hacc[tn][4 * q + 1] = v.y; hacc[tn][4 * q + 2] = v.z; hacc[tn][4 * q + 3] = v.w;
        }
    // G^T and M^T in 16 x 16 quadrants (tokens t of the first or second half of the chunk, s likewise; lane: t = 16 qi + lane % 16,
    // s = 16 qj + 4 (lane / 16) + v): (0,0), (1,0) and (1,1) go round the waves, the fourth is all s > t and stays zero.
    // In the diagonal ones the causal mask, and the skip term D where s = t:
    const int l16 = lane & 15, k4 = lane >> 4;
    float dadd[4];
    bool keep[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        keep[v] = 4 * k4 + v <= l16;
        dadd[v] = 4 * k4 + v == l16 ? D_h : 0.f;
    }
    if (tid < 32) *reinterpret_cast<uint4 *>(sMh + (tid >> 1) * XS + 32 + (tid & 1) * 16) = make_uint4(0u, 0u, 0u, 0u);
    // this thread's conv channel: weights and bias stay in registers for the whole prompt
    const int pc = tid % P;
    const int sg = P >= 64 ? __builtin_amdgcn_readfirstlane(tid / P) : tid / P;      // uniform over a wave when P >= 64
    const unsigned ch = hd * P + pc;
    // the four taps as two packed pairs (they are bf16 in memory): the conv is two bf16 dot products per token
    const uint2 wraw = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(p.wgt) + (size_t)ch * W);
    const float cbias = p.bias ? load_io(p.bias, ch, SSMV_BF16) : 0.f;
    // One base pointer per tensor that is uniform over the workgroup plus an element offset; tokens are clamped into
    // the prompt, so every load is unconditional: a token before the prompt is replaced by the ring history, tokens past
    // its end carry dt = 0 and thereby weight 0 everywhere (their rows of X, B, C are the last token's: finite).
    const uint16_t *x_b = reinterpret_cast<const uint16_t *>(p.x_raw) + (size_t)b * Ls * HP;
    const char *z_b = reinterpret_cast<const char *>(p.z) + (size_t)b * Ls * HP * 2;
    const uint16_t *B_b = reinterpret_cast<const uint16_t *>(p.Bm) + (size_t)b * Ls * GN + (size_t)g * N;
    const uint16_t *C_b = reinterpret_cast<const uint16_t *>(p.Cm) + (size_t)b * Ls * GN + (size_t)g * N;
    const uint16_t *dt_b = reinterpret_cast<const uint16_t *>(p.dt) + (size_t)b * Ls * H + hd;
    auto off = [](int token, int stride, int rest) { return 2u * (__umul24(token, stride) + (unsigned)rest); };     // in bytes
    // the same for a chunk's first row (uniform)
    auto chunk_of = [](const void *base, int c, int stride) { return static_cast<const char *>(base) + (size_t)c * Q * stride * 2; };
    auto clampL = [&](int tg) { return tg < 0 ? 0 : (tg < L ? tg : L - 1); };
    auto raw_bits = [&](int tg) { return (uint32_t)(x_b + (size_t)clampL(tg) * HP)[ch]; };    // uniform row pointer, 32-bit lane offset
    // the W-1 raw inputs ahead of the first chunk (newest last), where the conv finds those of the chunk before
    if (tid < P) {
        uint32_t hist[W - 1];                           // as bits
#pragma unroll
        for (int j = 0; j < W - 1; ++j) {
            if (SEG && c_beg > 0) hist[j] = raw_bits(c_beg * Q - (W - 1) + j);
            else hist[j] = reinterpret_cast<const uint16_t *>(p.ring)[((size_t)b * p.ring_len + ((conv_head + 1 - (W - 1) + j) & mask)) * HP + ch];
        }
        sCar[((c_beg + 1) & 1) * P + pc] = make_uint2(hist[0] << 16, hist[1] | (hist[2] << 16));
    }

    constexpr int UI = (4 * N + NT - 1) / NT;           // (n, eight tokens) units of the transposed B per thread and chunk
    // The chunk's raw x, B and C rows go from global memory straight into LDS, 1 KB per wave and instruction (lane l's 16
    // bytes land at byte 16 l of the destination): no registers hold them while they are under way, and a chunk costs a
    // wave 4 to 6 load instructions instead of 30.  dt (one value per lane) takes the ordinary way.
    // Every address is the chunk's first row (uniform) plus a lane offset that stays the same over the chunks; a last chunk that is
    // not full reads its last token again for the rows behind it.
    constexpr int LR = P / 8;                           // lanes per row of x, 64 / LR rows per instruction, P / 16 instructions
    constexpr int XPW = 2 / NSPL;                       // of them per wave
    constexpr int BPW = (PIECES / 2 + Ld::NW - 1) / Ld::NW;      // PIECES / 2 instructions cover the 32 rows of B, and of C
    uint32_t ox[XPW], obc[BPW], odt;
    auto lane_offsets = [&](int last) {                 // last: the chunk's last row that is there
#pragma unroll
        for (int k = 0; k < XPW; ++k) {
            const int row = (XPW * wave_u + k) * (64 / LR) + lane / LR;
            ox[k] = off(min(row, last), HP, hd * P + ((lane % LR) ^ key_x<P>(row)) * 8);
        }
#pragma unroll
        for (int k = 0; k < BPW; ++k) {
            const int row = (wave_u + k * Ld::NW) * (64 / PIECES) + lane / PIECES;
            obc[k] = off(min(row, last), GN, ((lane % PIECES) ^ key_bc<N>(row)) * 8);
        }
        odt = off(min(li, last), H, 0);
    };
    lane_offsets(Q - 1);
    auto issue_x_loads = [&](int c, uint32_t &dt_bits) {
        if (c * Q + Q > L) lane_offsets(L - 1 - c * Q);
        const char *xc = chunk_of(x_b, c, HP);
#pragma unroll
        for (int k = 0; k < XPW; ++k) load_to_lds16(xc, ox[k], sXraw + (XPW * wave_u + k) * 1024);
        dt_bits = *reinterpret_cast<const uint16_t *>(chunk_of(dt_b, c, H) + odt);
    };
    auto issue_bc_loads = [&](int c) {                  // behind issue_x_loads of the same chunk
        const char *Bc = chunk_of(B_b, c, GN), *Cc = chunk_of(C_b, c, GN);
        char *dB = lds + Ld::oB + (c & (Ld::BCC - 1)) * Ld::BCS, *dC = lds + Ld::oC + (c & (Ld::BCC - 1)) * Ld::BCS;
#pragma unroll
        for (int k = 0; k < BPW; ++k) {
            const int idx = wave_u + k * Ld::NW;
            if (idx < PIECES / 2) {
                load_to_lds16(Bc, obc[k], dB + idx * 1024);
                if (emit) load_to_lds16(Cc, obc[k], dC + idx * 1024);
            }
        }
    };
    // transposing reads (read_tr16): lane j of 16 is in row j / 4 of four, 8 bytes j % 4 of the 32 of its 16 columns.  Of the raw
    // x rows from token 0 on, this thread's channel; of the rows of B, per unit, tokens 4 h .. 4 h + 3 of its eight
    const int trow = l16 >> 2, tpiece = (l16 >> 1) & 1, tbyte = (l16 & 1) * 8;
    const char *xtr = sXraw + trow * (2 * P) + ((((pc >> 4) * 2 + tpiece) ^ key_x<P>(trow)) * 16) + tbyte;
    int btr[UI][2];
#pragma unroll
    for (int i = 0; i < UI; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int u = tid + i * NT, row = 8 * (u / N) + 4 * h + trow;
            btr[i][h] = row * (2 * N) + ((((u % N) >> 4) * 2 + tpiece) ^ key_bc<N>(row)) * 16 + tbyte;
        }
    // Per chunk: exp(cum_t) of this lane's token t = li, and exp(cum_Q) (the same in every lane).
    float at_t, aq;
    float cum_all = 0.f;                                // SEG: log2 of the segment's decay
    auto consume = [&](int c, uint32_t dt_bits) {
        const int t0 = c * Q, s0 = sg * QS;
        const char *sB = lds + Ld::oB + (c & (Ld::BCC - 1)) * Ld::BCS;
        // ---- dt, its prefix sums and the decay factors: every wave for itself (32 tokens, both halves alike) ----
        {
            float d = Vec::decode1(dt_bits) + dtb_h;
            if (p.dt_softplus) d = softplus_fast(d);
            if (t0 + li >= L) d = 0.f;                  // padding: no decay, no input
            float v = d * A2_h;
            v = prefix32(v);
            const float cq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), Q - 1));
            at_t = __builtin_amdgcn_exp2f(v);
            aq = __builtin_amdgcn_exp2f(cq);
            if constexpr (SEG) cum_all += cq;
            if (lh == 0) {
                sCum[li] = v;
                sDt[li] = d;
                sW[li] = __builtin_amdgcn_exp2f(cq - v) * d;
            }
            __builtin_amdgcn_wave_barrier();            // the wave's own LDS traffic stays in program order
        }
        // ---- conv of this thread's QS tokens, rows [p][token] ----
        {
            // raw inputs, as packed pairs of adjacent tokens of this channel: e[0], e[1] the four tokens ahead of s0 (in the chunk's first
            // tokens what the chunk before left), then the thread's own; o the pairs in between
            uint32_t e[QS / 2 + 2], o[QS / 2 + 1];
            uint2 ahead;
            if constexpr (P >= 64) {
                if (s0 != 0) ahead = read_tr16(xtr + (s0 - 4) * (2 * P));
                else ahead = sCar[((c + 1) & 1) * P + pc];
            } else {                                    // both kinds of threads in one wave
                const uint2 here = read_tr16(xtr + max(s0 - 4, 0) * (2 * P)), before = sCar[((c + 1) & 1) * P + pc];
                ahead = s0 != 0 ? here : before;
            }
            e[0] = ahead.x;
            e[1] = ahead.y;
#pragma unroll
            for (int j = 0; j < QS / 4; ++j) {
                const uint2 r = read_tr16(xtr + (s0 + 4 * j) * (2 * P));
                e[2 + 2 * j] = r.x;
                e[3 + 2 * j] = r.y;
            }
            if (s0 + QS == Q) sCar[(c & 1) * P + pc] = make_uint2(e[QS / 2], e[QS / 2 + 1]);     // for the next chunk
#pragma unroll
            for (int i = 0; i < QS / 2 + 1; ++i) o[i] = __builtin_amdgcn_alignbit(e[i + 1], e[i], 16);
#pragma unroll
            for (int v = 0; v < QS / 8; ++v) {
                float xv[8];
                conv8(xv, o + 4 * v, e + 1 + 4 * v, wraw.x, wraw.y, cbias);
                if constexpr (SILU) conv_silu8(xv);
                // the rounding to the storage type
                *reinterpret_cast<uint4 *>(sX + pc * XS + s0 * 2 + 16 * v) =
                    make_uint4(pack_bf16x2(xv[0], xv[1]), pack_bf16x2(xv[2], xv[3]), pack_bf16x2(xv[4], xv[5]), pack_bf16x2(xv[6], xv[7]));
            }
        }
        // ---- w_s B_s transposed, head and tail: eight tokens of one n per unit ----
#pragma unroll
        for (int i = 0; i < UI; ++i) {
            const int u = tid + i * NT;
            if (u < 4 * N) {
                const int n = u % N;
                const int oct = N >= 64 ? __builtin_amdgcn_readfirstlane(u / N) : u / N;
                const float4 w0 = *reinterpret_cast<const float4 *>(sW + 8 * oct), w1 = *reinterpret_cast<const float4 *>(sW + 8 * oct + 4);
                const float wv[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
                uint32_t bh[4], bl[4];
                const uint2 r0 = read_tr16(sB + btr[i][0]), r1 = read_tr16(sB + btr[i][1]);
                const uint32_t bb[4] = {r0.x, r0.y, r1.x, r1.y};
#pragma unroll
                for (int j2 = 0; j2 < 4; ++j2)
                    split2(wv[2 * j2] * __uint_as_float(bb[j2] << 16), wv[2 * j2 + 1] * __uint_as_float(bb[j2] & 0xffff0000u), bh[j2], bl[j2]);
                *reinterpret_cast<uint4 *>(sBh + n * XS + oct * 16) = make_uint4(bh[0], bh[1], bh[2], bh[3]);
                *reinterpret_cast<uint4 *>(sBl + n * XS + oct * 16) = make_uint4(bl[0], bl[1], bl[2], bl[3]);
            }
        }
    };

    // The output tile [token][32 channels] of a chunk goes into the wave's own LDS patch and leaves as 64-byte rows or wider
    // (four lanes a row: a store instruction then touches 16 cache lines, not 32 with 16 bytes in each), one chunk LATE, next
    // to the issue of the following chunk's loads: loads and stores share one counter and complete in no fixed order
    // among each other, so the wait for the loads at the top of a chunk also waits for every store issued before it -
    // which by then is a whole chunk old instead of a few cycles.
    // By then every wave's tile of that chunk is complete (the barrier at the chunk's end lies in between), so the rows are
    // dealt out again: a wave stores whole rows of the head (all its 32-channel tiles side by side: whole cache lines
    // from one instruction instead of 64-byte halves from two waves at different times) for its share of the tokens.
    // 4 to 8 % on the 64- and 128-channel heads.
    constexpr bool kWholeRows = NSPL == 1 && Ld::NP > 1;
    constexpr int LPT = kWholeRows ? 4 * Ld::NP : 4, TPI = 64 / LPT;      // lanes per token row, tokens per instruction
    int ytok[2], ylds[2];
    uint32_t oy[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int piece = lane % LPT;
        ytok[r] = (kWholeRows ? 2 * wave_u + r : r) * TPI + lane / LPT;
        ylds[r] = Ld::oY + (kWholeRows ? piece >> 2 : pt) * Ld::YT + ytok[r] * Ld::YS + (piece & 3) * 16;
        oy[r] = off(ytok[r], HP, hd * P + (kWholeRows ? 0 : pt * 32) + piece * 8);
    }
    auto flush_outputs = [&](int c) {
        char *yc = y_b + (size_t)c * Q * HP * 2;
        const int live = L - c * Q;
        if (live >= Q) {
#pragma unroll
            for (int r = 0; r < 2; ++r) *reinterpret_cast<uint4 *>(yc + oy[r]) = *reinterpret_cast<const uint4 *>(lds + ylds[r]);
        } else {
#pragma unroll
            for (int r = 0; r < 2; ++r)
                if (ytok[r] < live) *reinterpret_cast<uint4 *>(yc + oy[r]) = *reinterpret_cast<const uint4 *>(lds + ylds[r]);
        }
    };
    const int prow = pt * 32 + li;                      // this lane's channel (inside the head) as an operand row
    float *sZ = reinterpret_cast<float *>(lds + Ld::oZ) + pt * 1024;
    // Of the workgroups on a compute unit the one that stages goes first on two kinds of heads, all of whose waves wait for the staging.  Time over
    // that without, means of 96 to 1500 tokens with and without SiLU and gate:
    //   128 x 64   with a gate 0.94 to 1.01 at any number of workgroups.  Without one, where the last round fills more than a workgroup a compute
    //              unit, 0.97 at 258 and 512 workgroups, 0.98 at 896, 0.99 at 1024, 1536 and 2048; where it does not it loses, 1.01 at 520, 600, 1088 and 1280,
    //              1.03 at 700 and 768; of lengths that differ from about 640 workgroups on, 1.02 at 520, 0.98 at 900.
    //              Three chunks 0.99, with SiLU 1.01.  32 x 32 heads, 2048 tokens 294 -> 287 us, 700 with SiLU, gate, softplus 184 -> 167
    //   32 channels, one length   1100 to 2240 workgroups 0.97 to 0.98 (N = 32), 0.96 to 0.99 (64), 0.99 (128), and never more than 1.01; of lengths that
    //              differ up to 1.03.  (The products first: the same, but up to 1.03 at N = 128)
    // Not on the others: staging or products first, means of 24 calls each, 280 to 2048 workgroups, 0.98 to 1.01, single calls up to 1.08.
    const unsigned wgs = gridDim.x;
    const bool staging_first = P == 32 ? !p.seq_len : P == 128 && N == 64 && p.L > 4 * Q && (p.z || (p.seq_len ? wgs >= 640 : (wgs - 1) % 512 >= 256));
    uint32_t dt_bits;
    issue_x_loads(c_beg, dt_bits);
    issue_bc_loads(c_beg);
    wait_direct_loads();
    __syncthreads();
    for (int c = c_beg; c < c_end; ++c) {
        const int t0 = c * Q;
        const char *sB = lds + Ld::oB + (c & (Ld::BCC - 1)) * Ld::BCS, *sC = lds + Ld::oC + (c & (Ld::BCC - 1)) * Ld::BCS;
        if (staging_first) __builtin_amdgcn_s_setprio(1);
        consume(c, dt_bits);
        if (staging_first) __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        // the stores ahead of the loads on the wide tiles (2 % there; the other way round on the narrow ones)
        constexpr bool kStoresFirst = P >= 128 && N >= 64;
        if (kStoresFirst && c > c_beg && nh == 0 && emit) {
            flush_outputs(c - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (c + 1 < c_end) {                            // under way for the whole chunk
            issue_x_loads(c + 1, dt_bits);
            if (Ld::BCC == 2) issue_bc_loads(c + 1);
        }
        if (!kStoresFirst && c > c_beg && nh == 0 && emit) flush_outputs(c - 1);
        __builtin_amdgcn_sched_barrier(0);              // the loads and stores stay here, a chunk of arithmetic ahead of the next wait

        const int t = li;                               // this lane's token within the chunk
        using QV = XVec<SSMV_BF16, 4>;                  // four adjacent channels
        typename QV::Raw zraw[4];
        if (gated && nh == 0 && emit) {                 // requested ahead of the matrix products
            const char *zc = chunk_of(z_b, c, HP) + off(min(t, L - 1 - t0), HP, hd * P + pt * 32 + 4 * lh);
#pragma unroll
            for (int q = 0; q < 4; ++q) zraw[q] = *reinterpret_cast<const typename QV::Raw *>(zc + 16 * q);
        }
        f16v yacc = {0};
        if (emit) {
            // C of this lane's token: the B operand of h C^T over the wave's own tiles
            uint4 cop[2 * TNL];
#pragma unroll
            for (int st = 0; st < 2 * TNL; ++st) cop[st] = *reinterpret_cast<const uint4 *>(sC + t * (N * 2) + (((2 * (2 * TNL * nh + st) + lh) ^ key_bc<N>(t)) * 16));
            // ---- this wave's quadrants of G^T = B C^T, and of M^T: decayed, scaled, masked, D on the diagonal; to LDS ----
            auto quadrant = [&](int qi, int qj) {
                f4v gacc = {0};
                const int rs = 16 * qj + l16, rt = 16 * qi + l16;
#pragma unroll
                for (int kk = 0; kk < N / 32; ++kk)
                    gacc = mfma16(as_bf8(*reinterpret_cast<const uint4 *>(sB + rs * (N * 2) + (((4 * kk + k4) ^ key_bc<N>(rs)) * 16))),
                                  as_bf8(*reinterpret_cast<const uint4 *>(sC + rt * (N * 2) + (((4 * kk + k4) ^ key_bc<N>(rt)) * 16))), gacc);
                const int s0 = 16 * qj + 4 * k4;
                const float ct = sCum[rt];
                const float4 cs = *reinterpret_cast<const float4 *>(sCum + s0), ds = *reinterpret_cast<const float4 *>(sDt + s0);
                const float csv[4] = {cs.x, cs.y, cs.z, cs.w}, dsv[4] = {ds.x, ds.y, ds.z, ds.w};
                float m[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float dec = __builtin_amdgcn_exp2f(ct - csv[v]) * dsv[v];      // may overflow where s > t: selected away
                    if (qi == qj) m[v] = keep[v] ? fmaf(gacc[v], dec, dadd[v]) : 0.f;
                    else m[v] = gacc[v] * dec;
                }
                *reinterpret_cast<uint2 *>(sMh + rt * XS + s0 * 2) = make_uint2(pack_bf16x2(m[0], m[1]), pack_bf16x2(m[2], m[3]));
            };
            if (wave_u == 0) quadrant(0, 0);
            if (wave_u == 1 % Ld::NW) quadrant(1, 0);
            if (wave_u == 2 % Ld::NW) quadrant(1, 1);
            // ---- Y^T = h C^T, scaled by exp(cum_t): the state registers are the A operand ----
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    uint32_t ah[4];                          // heads only: these products end in outputs, not in the state
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        ah[d] = pack_bf16x2(hacc[tn][8 * st + 2 * d], hacc[tn][8 * st + 2 * d + 1]);
                    }
                    yacc = mfma(as_bf8(ah[0], ah[1], ah[2], ah[3]), as_bf8(cop[2 * tn + st]), yacc);
                }
            if constexpr (NSPL == 2) {
                if (nh == 1) {                              // the second half of n: hand the sum to the tile's first wave
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<float4 *>(sZ + q * 256 + lane * 4) = make_float4(yacc[4 * q], yacc[4 * q + 1], yacc[4 * q + 2], yacc[4 * q + 3]);
                }
            }
        }
        // ---- Y^T += X^T M^T;  h^T <- exp(cum_Q) h^T + (diag(w) B)^T X: X is the A operand of one, the B operand of the other ----
        uint4 xop[2];
#pragma unroll
        for (int st = 0; st < 2; ++st) xop[st] = *reinterpret_cast<const uint4 *>(sX + prow * XS + (16 * st + 8 * lh) * 2);
        if (emit) __syncthreads();     // M^T is complete; nobody reads this chunk's B and C rows any more
        if (Ld::BCC == 1 && c + 1 < c_end) issue_bc_loads(c + 1);
        if (nh == 0 && emit) {
            if constexpr (NSPL == 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 z4 = *reinterpret_cast<const float4 *>(sZ + q * 256 + lane * 4);
                    yacc[4 * q] += z4.x; yacc[4 * q + 1] += z4.y; yacc[4 * q + 2] += z4.z; yacc[4 * q + 3] += z4.w;
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) yacc[v] *= at_t;
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const int o = t * XS + (16 * st + 8 * lh) * 2;
                yacc = mfma(as_bf8(xop[st]), as_bf8(*reinterpret_cast<const uint4 *>(sMh + o)), yacc);
            }
        }
#pragma unroll
        for (int tn = 0; tn < TNL; ++tn) {
#pragma unroll
            for (int v = 0; v < 16; ++v) hacc[tn][v] *= aq;
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const int o = (32 * (TNL * nh + tn) + lperm) * XS + (16 * st + 8 * lh) * 2;
                hacc[tn] = mfma(as_bf8(*reinterpret_cast<const uint4 *>(sBh + o)), as_bf8(xop[st]), hacc[tn]);
                hacc[tn] = mfma(as_bf8(*reinterpret_cast<const uint4 *>(sBl + o)), as_bf8(xop[st]), hacc[tn]);
            }
        }
        // ---- gate, store ----
        if (nh == 0 && emit) {
            if (gated) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float zf[4];
                    QV::decode(zraw[q], zf);
#pragma unroll
                    for (int e = 0; e < 4; ++e) yacc[4 * q + e] *= silu_fast(zf[e]);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2 *>(sY + t * Ld::YS + (8 * q + 4 * lh) * 2) =
                    make_uint2(pack_bf16x2(yacc[4 * q], yacc[4 * q + 1]), pack_bf16x2(yacc[4 * q + 2], yacc[4 * q + 3]));
        }
        __builtin_amdgcn_wave_barrier();                // the tile waits in the wave's LDS patch: flush_outputs
        wait_direct_loads();                            // this wave's share of the next chunk's inputs has landed ...
        __syncthreads();     // ... and so has everybody's; the next chunk overwrites X, B^T, M
    }

    if (nh == 0 && emit) flush_outputs(c_end - 1);
    if constexpr (SEG) {
        if (!seg.last) {
            if (p.seg_pass == 1) {                      // the next segment has its state already
                SSMV_TRACE_END(tid == 0);
                return;
            }
            // a segment's state on its way to the combining launch
#pragma unroll
            for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *seg_at(tn, q) = make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
            if (c_beg > 0 && tid == 0) *reinterpret_cast<float *>(y_b + seg_piece<2>(P * N / 4, P, seg.area, HP, hd)) = cum_all;
            SSMV_TRACE_END(tid == 0);
            return;
        }
    }
    // ---- state back in place; the newest W-1 raw inputs into the ring behind conv_head -----------------------
#pragma unroll
    for (int tn = 0; tn < TNL; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(state_at(tn, q)) =
                make_float4(hacc[tn][4 * q + 0], hacc[tn][4 * q + 1], hacc[tn][4 * q + 2], hacc[tn][4 * q + 3]);
    if (tid < P) {
        for (int tg = (L - (W - 1) > 0 ? L - (W - 1) : 0); tg < L; ++tg)
            Vec::store_raw1(p.ring, ((size_t)b * p.ring_len + ((conv_head + 1 + tg) & mask)) * HP + ch, raw_bits(tg));
    }
    SSMV_TRACE_END(tid == 0);
}

template <int P, int N, bool SEG, bool SILU>
static int launch_pn(const PrefillParams &p, hipStream_t stream)
{
    const size_t lds = PfLds<P, N>::total;
    const dim3 grid((unsigned)(p.H * p.batch) * (SEG ? p.seg_count - 1 : 1)), block(2 * P * PfLds<P, N>::NSPL);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&prefill_bf16_kernel<P, N, SEG, SILU>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL((prefill_bf16_kernel<P, N, SEG, SILU>), grid, block, lds, stream, p);
    return (int)hipGetLastError();
}

template <int P, int N, bool SILU>
static int launch_n(const PrefillParams &p, hipStream_t stream)
{
    if constexpr (P == 128 && N == 128) return (int)hipErrorInvalidConfiguration;
    else if constexpr (cuts(P, N)) return p.seg_count ? launch_pn<P, N, true, SILU>(p, stream) : launch_pn<P, N, false, SILU>(p, stream);
    else return p.seg_count ? (int)hipErrorInvalidConfiguration : launch_pn<P, N, false, SILU>(p, stream);
}

template <int P>
static int launch_p(const PrefillParams &p, hipStream_t stream)
{
    const bool silu = p.conv_act == SSMV_ACT_SILU;
    switch (p.N) {
        case 32: return silu ? launch_n<P, 32, true>(p, stream) : launch_n<P, 32, false>(p, stream);
        case 64: return silu ? launch_n<P, 64, true>(p, stream) : launch_n<P, 64, false>(p, stream);
        case 128: return silu ? launch_n<P, 128, true>(p, stream) : launch_n<P, 128, false>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

template <int P, int N>
static constexpr int resident()
{
    constexpr int by_lds = 160 * 1024 / PfLds<P, N>::total, by_waves = 12 / PfLds<P, N>::NW;      // three waves per SIMD by their registers
    return by_lds < by_waves ? by_lds : by_waves;
}

// The tiles whose prompts this kernel cuts, under prefill_bf16_cuts: those of which it fits more than twice as many workgroups on a compute
// unit as the pipelined kernel does (8 to 3, 5 to 2, 3 to 1, 3 to 1), at 1.4 to 2.1 times its time per chunk
int prefill_bf16_resident(int P, int N)
{
    if (!cuts(P, N)) return 0;
    return P == 64 ? resident<64, 32>() : P == 128 ? resident<128, 32>() : N == 32 ? resident<32, 32>() : resident<32, 128>();
}

#ifdef SSMV_TRACE
int set_trace_prefill_bf16(long long *buf) { return (int)hipMemcpyToSymbol(HIP_SYMBOL(pf_trace_buf_), &buf, sizeof(buf)); }
#endif

// large launches (prefill_pipe_serves), and a pass over a prompt that is cut; the caller appends the bookkeeping or the combining launch
int launch_prefill_bf16(const PrefillParams &p, hipStream_t stream)
{
    switch (p.P) {
        case 32: return launch_p<32>(p, stream);
        case 64: return launch_p<64>(p, stream);
        case 128: return launch_p<128>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

}  // namespace ssmv
