// The fused multi-step verification kernel for diagonal A (Mamba-1 style: A[channel][n], one channel per head).
//
// One verify moves little (8192 channels x 16: half a megabyte) and takes up to 32 tokens one after the other, so what
// counts is the chain of latencies and the number of instructions, not bytes.  Layout (gfx950, wave64):
//   * a QUAD of lanes owns R adjacent channels for the whole launch: lane `sub` of the quad holds n = 16 v + 4 sub .. + 3 of
//     their state rows and of A, 16 bytes an access;
//   * the tokens of a channel live in the same quad, lane `sub` having fetched and prepared token 4 j + sub of group j (conv,
//     softplus, dt x); a step hands a token round its quad with a DPP broadcast.  x and dt so need neither LDS nor a barrier,
//     each is loaded once, and the conv's three older inputs are quad rotations of what is there.  Only B and C, which all
//     channels share, go through LDS;
//   * four outputs of a channel are summed over the quad and land one per lane (a transposing reduction: nine instructions for
//     four tokens), which is where they are scaled, gated and stored;
//   * what does not depend on the cache's integers (this call's tokens, taps, A) is requested ahead of them, the rest right
//     behind: two round trips to memory before the first step.
// Measured (all layers of a round, conv fused, bf16): one sequence, 8192 channels x 16, k = 8, 24 layers 193 -> 117 us; 24
// sequences x 5120 channels, ragged k = 6, softplus and SiLU, four layers 63 -> 47 us (500 vector instructions for a wave's 32
// channels, where verify_impl.h took 404 for 16).  What is left: at small batch two round trips to memory and the launch itself, at
// large batch the vector instructions (about half of them exp, softplus and SiLU).
// (verify_impl.h, which stages the tokens in LDS as fp32 and walks them one at a time, keeps ssmv_materialize of these caches and
// explicitly chosen launch shapes.)
#include <type_traits>

#include "verify_impl.h"

namespace ssmv {
namespace {

typedef unsigned u4v __attribute__((ext_vector_type(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ T *at(void *base, unsigned idx) { return reinterpret_cast<T *>(static_cast<char *>(base) + (size_t)(idx * (unsigned)sizeof(T))); }
template <typename T>
__device__ __forceinline__ const T *at(const void *base, unsigned idx) { return at<T>(const_cast<void *>(base), idx); }

// one value of R adjacent channels in the I/O type
template <int IO, int R>
struct ChanVec {
    static constexpr int NW = IO == SSMV_BF16 ? 1 : R;      // 32-bit words
    uint32_t w[NW];
    // element idx behind a base that is the same in all lanes: a 32-bit lane offset, no 64-bit address arithmetic
    static __device__ __forceinline__ ChanVec load(const void *base, unsigned idx)
    {
        ChanVec r;
        if constexpr (IO == SSMV_BF16) {
            const uint16_t *s = at<uint16_t>(base, idx);
            if constexpr (R == 1) r.w[0] = *s;
            else r.w[0] = *reinterpret_cast<const uint32_t *>(s);
        } else {
            const uint32_t *s = at<uint32_t>(base, idx);
            if constexpr (R == 1) r.w[0] = *s;
            else { const u2v t = *reinterpret_cast<const u2v *>(s); r.w[0] = t.x; r.w[1] = t.y; }
        }
        return r;
    }
    __device__ __forceinline__ void store(void *base, unsigned idx) const
    {
        if constexpr (IO == SSMV_BF16) {
            uint16_t *d = at<uint16_t>(base, idx);
            if constexpr (R == 1) *d = (uint16_t)w[0];
            else *reinterpret_cast<uint32_t *>(d) = w[0];
        } else {
            uint32_t *d = at<uint32_t>(base, idx);
            if constexpr (R == 1) *d = w[0];
            else *reinterpret_cast<u2v *>(d) = u2v{w[0], w[1]};
        }
    }
    __device__ __forceinline__ float get(int r) const
    {
        if constexpr (IO == SSMV_BF16) return __uint_as_float(r == 0 ? w[0] << 16 : w[0] & 0xffff0000u);
        else return __uint_as_float(w[r]);
    }
    static __device__ __forceinline__ ChanVec encode(const float (&v)[R])
    {
        ChanVec r;
        if constexpr (IO == SSMV_BF16) {
            r.w[0] = R == 1 ? pack_bf16x2(v[0], 0.f) : pack_bf16x2(v[0], v[R - 1]);
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) r.w[i] = __float_as_uint(v[i]);
        }
        return r;
    }
};

template <int CTRL>
__device__ __forceinline__ uint32_t quad_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float quad_movef(float v) { return __uint_as_float(quad_move<CTRL>(__float_as_uint(v))); }
// the value lane i of the quad holds
__device__ __forceinline__ float quad_get(float v, int i)
{
    return i == 0 ? quad_movef<0x00>(v) : i == 1 ? quad_movef<0x55>(v) : i == 2 ? quad_movef<0xAA>(v) : quad_movef<0xFF>(v);
}

// GP, GK: groups of four pending tokens and of four drafts that the launch may meet
template <int V, int R, int GP, int GK, int IO, bool CONV, bool EXTRA>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
void verify_diag_kernel(const int32_t *a_cur, const int32_t *a_pend, const int32_t *a_par, const int64_t *a_pos, const int32_t *a_head,
                        const VerifyParams p)
{
    constexpr int N = 16 * V;
    constexpr int W = SSMV_CONV_WIDTH;
    constexpr float LOG2E = 1.4426950408889634f;
    using CV = ChanVec<IO, R>;
    using Vec = IoVec<IO>;
    constexpr int EV = Vec::EV, VN = N / EV;             // 16-byte vectors per token of B or C
    constexpr int NB = 4 * (GP + GK) * VN, NC = 4 * GK * VN;
    __shared__ __attribute__((aligned(16))) float sB[4 * (GP + GK) * N];      // pending tokens from row 0, drafts from row 4 GP
    __shared__ __attribute__((aligned(16))) float sC[4 * GK * N];

    const unsigned tid = threadIdx.x, sub = tid & 3u;
    const int tile = blockIdx.x, b = blockIdx.y, k = p.k, H = p.H, nthreads = blockDim.x;
    // all of the cache's integers at once (clamped: a corrupted cache cannot index out of bounds)
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    int cur_raw = uni(a_cur[b]), pd_raw = uni(a_pend[b]), par_raw = uni(a_par[0]), pos_raw = uni((int)a_pos[b]), ch_raw = 0, ks_raw = k;
    if constexpr (CONV) ch_raw = uni(a_head[b]);
    if constexpr (EXTRA) if (p.k_seq) ks_raw = uni(p.k_seq[b]);

    const int c0 = (int)((tile * nthreads + tid) >> 2) * R;          // first channel of the quad
    const bool have = c0 < H;
    const int cc = have ? c0 : H - R;                    // quads past the end read the last channels again and store nothing
    // this sequence's part of every array: uniform bases, behind which all lane offsets fit 32 bits of bytes (the host refuses
    // rows of 2^22 elements and more, and longer conv rings do not get here: ring_fits), row numbers the 24-bit multiplier
    constexpr size_t ES = IO == SSMV_BF16 ? 2 : 4;
    const size_t tok_in = (size_t)b * k, tok_win = (size_t)b * p.win_tokens;
    auto seq = [&](const void *base, size_t rows, int len) { return const_cast<char *>(static_cast<const char *>(base) + rows * len * ES); };
    auto row_at = [&](int row, int len, int col) { return (unsigned)__mul24(row, len) + (unsigned)col; };

    // ---- this call's tokens, the conv's parameters, A and D: nothing here depends on the integers -------------------------
    CV xr[GK], dr[GK], zr[EXTRA ? GK : 1];
    const char *x_b = seq(CONV ? p.x_raw : p.xc, tok_in, H), *dt_b = seq(p.dt, tok_in, H), *z_b = seq(p.z, tok_in, H);
    const bool gated = EXTRA && p.z != nullptr;
#pragma unroll
    for (int j = 0; j < GK; ++j) {
        if (4 * j < k) {
            const unsigned o = row_at(min(4 * j + (int)sub, k - 1), H, cc);
            xr[j] = CV::load(x_b, o);
            dr[j] = CV::load(dt_b, o);
            if constexpr (EXTRA) if (gated) zr[j] = CV::load(z_b, o);
        }
    }
    u4v wraw[IO == SSMV_BF16 ? 1 : R];
    CV braw;
    if constexpr (CONV) {
        if constexpr (IO == SSMV_BF16) {
            const uint16_t *ws = at<uint16_t>(p.wgt, (unsigned)cc * W);
            if constexpr (R == 2) wraw[0] = *reinterpret_cast<const u4v *>(ws);
            else { const u2v t = *reinterpret_cast<const u2v *>(ws); wraw[0] = u4v{t.x, t.y, 0u, 0u}; }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) wraw[r] = *reinterpret_cast<const u4v *>(at<float>(p.wgt, (unsigned)(cc + r) * W));
        }
        if (p.bias) braw = CV::load(p.bias, cc);
    }
    v4f a2[R][V];
    float Dv[R], dtb[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int v = 0; v < V; ++v) a2[r][v] = *reinterpret_cast<const v4f *>(at<float>(p.A, (unsigned)cc * N + 4 * sub) + r * N + 16 * v) * LOG2E;
        Dv[r] = at<float>(p.D, cc)[r];
        dtb[r] = 0.f;
        if constexpr (EXTRA) if (p.dt_bias) dtb[r] = at<float>(p.dt_bias, cc)[r];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- what the integers decide: state, pending tokens, the conv's history, B and C -------------------------------------
    const int t0 = EXTRA ? p.tok0 : 0;
    const int cur = (int)((unsigned)cur_raw % 3u);
    const int pd = min(max(pd_raw, 0), p.pend_max) & (EXTRA ? p.pend_mask : ~0);
    const int src_slot = EXTRA ? (cur + p.src_add) % 3 : cur;
    const int par = par_raw & 1, wp = pos_raw & (SSMV_WINDOW - 1);
    const int kb = min(max(ks_raw, 1), k);
    const bool wring = p.win_ring != 0;
    auto slot_in = [&](int tt) { return wring ? (wp + tt) & (SSMV_WINDOW - 1) : tt; };               // pending token tt
    auto slot_out = [&](int t) { return wring ? (wp + pd + t) & (SSMV_WINDOW - 1) : t0 + t; };       // token t of this call
    // both halves of the window are kernel arguments: a select, not an indexed load that would wait for `par`
    auto half = [&](void *const (&w2)[2], int which) { return which ? w2[1] : w2[0]; };
    const char *winB = seq(half(p.win_B, par), tok_win, N), *winX = seq(half(p.win_xc, par), tok_win, H), *winDt = seq(half(p.win_dt, par), tok_win, H);
    char *winB_out = seq(half(p.win_B, par ^ 1), tok_win, N), *winX_out = seq(half(p.win_xc, par ^ 1), tok_win, H),
         *winDt_out = seq(half(p.win_dt, par ^ 1), tok_win, H);
    v4f h[R][V];
    float *state_b = p.state + (size_t)b * H * N;        // slot 0
    const unsigned srow = (unsigned)cc * N + 4 * sub;
    const float *src = state_b + (size_t)src_slot * p.slot_stride;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int v = 0; v < V; ++v)
            h[r][v] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(at<float>(src, srow) + r * N + 16 * v));
    CV xp[GP], dp[GP];
#pragma unroll
    for (int j = 0; j < GP; ++j) {
        if (4 * j < pd) {
            const unsigned o = row_at(slot_in(min(4 * j + (int)sub, pd - 1)), H, cc);
            xp[j] = CV::load(winX, o);
            dp[j] = CV::load(winDt, o);
        }
    }
    const int ring_mask = p.ring_len - 1, conv_head = (ch_raw + t0) & ring_mask;       // newest raw input fed so far
    char *ring_b = seq(p.ring, (size_t)b * p.ring_len, H);
    CV hist;
    if constexpr (CONV) hist = CV::load(ring_b, row_at((conv_head - 3 + (int)sub) & ring_mask, H, cc));   // token sub - 4
    // B rows and C rows into LDS as fp32 (rows of no token are not read back)
    const char *B_b = seq(p.Bm, tok_in, N), *C_b = seq(p.Cm, tok_in, N);
    auto bc_item = [&](int i, uint4 &raw, int &t, bool &is_c) {
        is_c = i >= NB;
        const int q = is_c ? i - NB : i, row = q / VN, n = (q % VN) * EV;
        t = is_c ? row : row - 4 * GP;                   // draft number, or (< 0) pending token t + 4 GP
        const bool on = t >= 0 ? t < kb : row < pd;
        raw = make_uint4(0, 0, 0, 0);
        if (on) raw = Vec::load_raw(is_c ? C_b : t >= 0 ? B_b : winB, (t >= 0 ? t : slot_in(row)) * N + n);
        return on;
    };
    auto bc_use = [&](int i, uint4 raw, int t, bool is_c, bool on) {
        float f[EV];
        Vec::decode(raw, f);
        float *d = is_c ? sC + (i - NB) * EV : sB + i * EV;
#pragma unroll
        for (int e = 0; e < EV; e += 4) *reinterpret_cast<v4f *>(d + e) = v4f{f[e], f[e + 1], f[e + 2], f[e + 3]};
        if (on && !is_c && t >= 0 && tile == 0) Vec::store_raw(winB_out, slot_out(t) * N + (i % VN) * EV, raw);
    };
    {
        uint4 raw;
        int t;
        bool is_c, on = false;
        if ((int)tid < NB + NC) on = bc_item(tid, raw, t, is_c);
        __builtin_amdgcn_sched_barrier(0);
        if ((int)tid < NB + NC) bc_use(tid, raw, t, is_c, on);
        for (int i = tid + nthreads; i < NB + NC; i += nthreads) {
            on = bc_item(i, raw, t, is_c);
            bc_use(i, raw, t, is_c, on);
        }
    }
    if (tile == 0 && tid == 0) p.last_k[b] = t0 + kb;

    // ---- the tokens: conv, step size, dt x -------------------------------------------------------------------------------
    auto dt_fix = [&](float d, int r) {
        if constexpr (EXTRA) {
            d += dtb[r];
            if (p.dt_softplus) d = softplus_fast(d);
        }
        return d;
    };
    float dtp[GP][R], dxp[GP][R], dtk[GK][R], dxk[GK][R], skip[GK][R];
#pragma unroll
    for (int j = 0; j < GP; ++j) {
        if (4 * j < pd) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dtp[j][r] = dt_fix(dp[j].get(r), r);
                dxp[j][r] = dtp[j][r] * xp[j].get(r);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < GK; ++j) {
        if (4 * j < kb) {
            const int t = 4 * j + (int)sub;
            const bool on = t < kb;
            CV xc = xr[j];
            if constexpr (CONV) {
                // width-4 causal depthwise conv, fp32 accumulate in tap order, rounded to the I/O type.  Input t - s sits s
                // lanes back in the quad, in the group before for the first s lanes
                const CV &before = j == 0 ? hist : xr[j > 0 ? j - 1 : 0];
                CV t1, t2, t3;
#pragma unroll
                for (int i = 0; i < CV::NW; ++i) {
                    t1.w[i] = quad_move<0x93>(sub == 3 ? before.w[i] : xr[j].w[i]);        // from lane (sub + 3) & 3
                    t2.w[i] = quad_move<0x4E>(sub >= 2 ? before.w[i] : xr[j].w[i]);        // (sub + 2) & 3
                    t3.w[i] = quad_move<0x39>(sub >= 1 ? before.w[i] : xr[j].w[i]);        // (sub + 1) & 3
                }
                float s[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float wv[W];
                    if constexpr (IO == SSMV_BF16) {
                        const uint32_t lo = r == 0 ? wraw[0].x : wraw[0].z, hi = r == 0 ? wraw[0].y : wraw[0].w;
                        wv[0] = __uint_as_float(lo << 16); wv[1] = __uint_as_float(lo & 0xffff0000u);
                        wv[2] = __uint_as_float(hi << 16); wv[3] = __uint_as_float(hi & 0xffff0000u);
                    } else {
                        wv[0] = __uint_as_float(wraw[r].x); wv[1] = __uint_as_float(wraw[r].y);
                        wv[2] = __uint_as_float(wraw[r].z); wv[3] = __uint_as_float(wraw[r].w);
                    }
                    float acc = p.bias ? braw.get(r) : 0.f;
                    acc = fmaf(wv[0], t3.get(r), acc);
                    acc = fmaf(wv[1], t2.get(r), acc);
                    acc = fmaf(wv[2], t1.get(r), acc);
                    acc = fmaf(wv[3], xr[j].get(r), acc);
                    if (p.conv_act == SSMV_ACT_SILU) acc = acc / (1.f + expf(-acc));
                    s[r] = acc;
                }
                xc = CV::encode(s);                      // what is fed on is what is stored
                if (on && have) xr[j].store(ring_b, row_at((conv_head + 1 + t) & ring_mask, H, cc));
            }
            if (on && have) {
                const unsigned o = row_at(slot_out(t), H, cc);
                xc.store(winX_out, o);
                dr[j].store(winDt_out, o);               // the raw dt: replay applies dt_fix again
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dtk[j][r] = dt_fix(dr[j].get(r), r);
                dxk[j][r] = dtk[j][r] * xc.get(r);
                skip[j][r] = Dv[r] * xc.get(r);
            }
        }
    }
    __syncthreads();

    // ---- one recurrence step: h <- exp(dt A) h + (dt x) B ------------------------------------------------------------------
    auto step = [&](int row, int i, const float (&dt)[R], const float (&dx)[R]) {
        v4f Bv[V];
#pragma unroll
        for (int v = 0; v < V; ++v) Bv[v] = *reinterpret_cast<const v4f *>(sB + row * N + 16 * v + 4 * sub);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float d = quad_get(dt[r], i), x = quad_get(dx[r], i);
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int e = 0; e < 4; ++e) h[r][v][e] = fmaf(x, Bv[v][e], h[r][v][e] * __builtin_amdgcn_exp2f(d * a2[r][v][e]));
        }
    };
    auto store_state = [&](int slot) {
        if (!have) return;
        float *dst = at<float>(state_b + (size_t)slot * p.slot_stride, srow);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < V; ++v) __builtin_nontemporal_store(h[r][v], reinterpret_cast<v4f *>(dst + r * N + 16 * v));
    };
    // (i) replay the pending tokens, (ii) snapshot h_j
#pragma unroll
    for (int j = 0; j < GP; ++j) {
        if (4 * j < pd) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * j + i < pd) step(4 * j + i, i, dtp[j], dxp[j]);
        }
    }
    if (pd > p.pend_hi) store_state((cur + 1) % 3);
    // (iii) the drafts, four at a time
#pragma unroll
    for (int j = 0; j < GK; ++j) {
        if (4 * j < k) {
            const int t = 4 * j + (int)sub;
            float y[R];
#pragma unroll
            for (int r = 0; r < R; ++r) y[r] = 0.f;      // tokens not taken: zeros
            if (4 * j < kb) {
                float acc[R][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r][i] = 0.f;
                    if (4 * j + i >= kb) continue;
                    step(4 * (GP + j) + i, i, dtk[j], dxk[j]);
                    v4f Cv[V];
#pragma unroll
                    for (int v = 0; v < V; ++v) Cv[v] = *reinterpret_cast<const v4f *>(sC + (4 * j + i) * N + 16 * v + 4 * sub);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
#pragma unroll
                        for (int v = 0; v < V; ++v)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[r][i] = fmaf(Cv[v][e], h[r][v][e], acc[r][i]);
                    }
                }
                const bool b0 = sub & 1u, b1 = sub & 2u;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float u = (b0 ? acc[r][1] : acc[r][0]) + quad_movef<0xB1>(b0 ? acc[r][0] : acc[r][1]);
                    const float w = (b0 ? acc[r][3] : acc[r][2]) + quad_movef<0xB1>(b0 ? acc[r][2] : acc[r][3]);
                    float yv = (b1 ? w : u) + quad_movef<0x4E>(b1 ? u : w) + skip[j][r];
                    if constexpr (EXTRA) if (gated) yv *= silu_fast(zr[j].get(r));       // y <- y * z * sigmoid(z), ahead of the rounding
                    if (t < kb) y[r] = yv;
                }
            }
            if (t < k && have) CV::encode(y).store(seq(p.y, tok_in, H), row_at(t, H, cc));
        }
    }
    // (iv) snapshot h_k (Algorithm 2), unless every accepted token is to stay pending
    if (p.write_hk) store_state((cur + 2) % 3);
}

template <int V, int R, int GP, int GK, int IO>
void launch_one(const VerifyParams &p, int waves, hipStream_t stream)
{
    const int per_wg = waves * 16 * R;
    const dim3 grid((p.H + per_wg - 1) / per_wg, p.batch), block(64 * waves);
    const bool extra = p.tok0 > 0 || p.dt_softplus || p.dt_bias || p.z || p.k_seq;
    auto go = [&](auto conv, auto ex) {
        hipLaunchKernelGGL((verify_diag_kernel<V, R, GP, GK, IO, conv.value, ex.value>), grid, block, 0, stream, p.cur_slot, p.pend, p.win_par,
                           p.pos, p.conv_head, p);
    };
    const std::true_type yes;
    const std::false_type no;
    if (p.x_raw) { if (extra) go(yes, yes); else go(yes, no); }
    else { if (extra) go(no, yes); else go(no, no); }
}

template <int V, int R, int IO>
int launch_groups(const VerifyParams &p, int waves, hipStream_t stream)
{
    const int pend_max = p.pend_mask ? p.pend_max : 0, most = pend_max > p.k ? pend_max : p.k;
    if (most <= 4) launch_one<V, R, 1, 1, IO>(p, waves, stream);
    else if (most <= 8) launch_one<V, R, 2, 2, IO>(p, waves, stream);
    else launch_one<V, R, 4, 4, IO>(p, waves, stream);
    return (int)hipGetLastError();
}

}  // namespace

// The ring's length is the caller's choice, and here a sequence's ring has to lie within 32 bits of bytes and its row
// numbers within the (signed) 24-bit multiplier.  verify_impl.h takes any: a ring of 4 GiB or 2^23 rows goes there.  (64-bit
// offsets of a full product here instead: rotating over 600 MB of caches, k up to 4, 3.61 -> 3.83, 3.71 -> 3.92 us.)
static bool ring_fits(const VerifyParams &p)
{
    return !p.x_raw || (p.ring_len <= 1 << 23 && (size_t)p.ring_len * p.H * (p.io == SSMV_BF16 ? 2 : 4) <= (size_t)1 << 32);
}

// Two channels per quad with bf16 tokens and 16 states (one 4-byte access then serves both): 24 sequences x 5120 channels,
// ragged k = 6, four layers 45.4 against 50.3 us, one sequence of 8192 channels, k = 8, 24 layers 116.7 against 119.3.  With fp32 tokens
// or 32 states one channel is faster (51.2 against 51.8, 40.3 against 42.7 us).  Four waves per workgroup share B and C where
// there are workgroups for every compute unit even so, fewer where the chip would not fill.
int launch_verify_diag(const VerifyParams &p, VerifyShape shape, hipStream_t stream)
{
    if (shape.forced || p.h_out || !ring_fits(p)) return launch_verify_any<true>(p, shape, stream);
    const bool bf16 = p.io == SSMV_BF16, two = bf16 && p.N == 16 && p.H % 2 == 0;
    const long quads = (long)p.batch * p.H / (two ? 2 : 1);
    const int waves = quads >= 32768 ? 4 : quads >= 8192 ? 2 : 1;
    if (two) return launch_groups<1, 2, SSMV_BF16>(p, waves, stream);
    switch (p.N) {
        case 16: return bf16 ? launch_groups<1, 1, SSMV_BF16>(p, waves, stream) : launch_groups<1, 1, SSMV_F32>(p, waves, stream);
        case 32: return bf16 ? launch_groups<2, 1, SSMV_BF16>(p, waves, stream) : launch_groups<2, 1, SSMV_F32>(p, waves, stream);
        case 64: return bf16 ? launch_groups<4, 1, SSMV_BF16>(p, waves, stream) : launch_groups<4, 1, SSMV_F32>(p, waves, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

}  // namespace ssmv
