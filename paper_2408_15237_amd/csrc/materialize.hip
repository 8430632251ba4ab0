// ssmv_materialize of the scalar-A modes: the live slot with the pending tokens folded in, row-major into the caller's buffer.
// A copy in the common case (a cache just prefilled, or handed over between rounds, has nothing pending), so it is built as one:
// a wave owns 16 rows, reads them in 1 KiB accesses (a tile each, or the rows as they are) and writes 1 KiB accesses of whole
// rows; tiles change into rows through a patch of LDS of the wave's own.  (Out of the tiles in 16-byte pieces, as the vector
// verify kernel reads them, 32 x 32 x 128 x 64 took 21.8 us, so 10.1; 5 x 80 x 64 x 128: 6.0, 4.3; 1 x 32 x 128 x 64: 3.0, 2.3.)
// Row-major slots with N > 64: as many rows as make 4 KiB, so that a launch has workgroups enough and wastes few rows on a headdim
// that 64 does not divide.  (fp32, 31 x 13 x 70 x 256: 14.1 us with 16 rows, 10.9 on the vector verify kernel, 10.1 so; 28 x 2 x 128 x 256: 3.8, 3.8, 3.1.)
// The pending tokens: h <- 2^(A sum dt) h + sum_s w_s x_s (x) B_s with w_s = dt_s 2^(A sum_{u > s} dt_u), all in fp32, taken
// backwards so that the exponent is a running sum - of A dt, not A times a sum that starts at 0: a head with A = -inf (or A log2 e
// beyond fp32's range) keeps its newest token with weight dt, as exp(dt A) = 0 of the stepwise form has it.
#include "ssmv_internal.h"

namespace ssmv {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

template <int N, bool TILED, int IO>
__global__ __launch_bounds__(256) void materialize_kernel(const VerifyParams p)
{
    using Vec = IoVec<IO>;
    constexpr int RW = TILED || N <= 64 ? 16 : 1024 / N, RG = 4 * RW;     // rows of a wave, of the workgroup
    constexpr int NQ = RW * N / 256;                     // 16-byte accesses per lane for the wave's rows
    constexpr int EV = Vec::EV, VN = N / EV;             // 16-byte vectors per token of B
    constexpr int XJ = RG / 16, BJ = (16 * VN + 255) / 256;               // loads of x and of B per thread
    constexpr int TS = N + 4;                            // row stride of the patch in which tiles become rows
    constexpr int TOK = 16 * RG + 16 * N + 16;           // pending tokens: x [16][RG], B [16][N], dt [16]
    constexpr int FL = TILED && RG * TS > TOK ? RG * TS : TOK;
    static_assert(SSMV_KMAX_LIMIT <= 16 && SSMV_WINDOW <= 16, "pending tokens");
    __shared__ __attribute__((aligned(16))) float lds[FL];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hd = blockIdx.y, b = blockIdx.z, H = p.H, P = p.P;
    const int row_wg = blockIdx.x * RG, row_w = row_wg + wave * RW;
    const int cur = (int)((unsigned)p.cur_slot[b] % 3u), pd = min(max(p.pend[b], 0), p.pend_max);
    const int par = p.win_par[0] & 1, wp = (int)p.pos[b] & (SSMV_WINDOW - 1);
    const size_t head = ((size_t)b * H + hd) * P * N;
    const float *src = p.state + (size_t)cur * p.slot_stride + head;
    // lane: float4 number 64 q + lane of the wave's rows, row-major; or, in tile q, columns 16 q + 4 (lane / 16) of row lane % 16
    auto row_of = [&](int q) { return TILED ? lane & 15 : (64 * q + lane) / (N / 4); };
    auto col_of = [&](int q) { return TILED ? 16 * q + 4 * (lane >> 4) : (64 * q + lane) % (N / 4) * 4; };
    v4f h[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const size_t o = TILED ? (((size_t)(row_w >> 4) * NQ + q) << 8) + lane * 4 : (size_t)min(row_w + row_of(q), P - 1) * N + col_of(q);
        h[q] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(src + o));
    }
    if (pd > 0) {
        float *sX = lds, *sB = sX + 16 * RG, *sDt = sB + 16 * N;
        const size_t tok = (size_t)b * p.win_tokens;
        auto entry = [&](int s) { return tok + (p.win_ring ? (wp + s) & (SSMV_WINDOW - 1) : s); };
        const int g = hd / (H / p.G), GN = p.G * N, HP = H * P;
        const void *wX = par ? p.win_xc[1] : p.win_xc[0], *wB = par ? p.win_B[1] : p.win_B[0], *wD = par ? p.win_dt[1] : p.win_dt[0];
        float x[XJ], d;
        uint4 bv[BJ];
#pragma unroll
        for (int j = 0; j < XJ; ++j) {
            const int i = tid + 256 * j, s = min(i / RG, pd - 1);
            x[j] = load_io(wX, entry(s) * HP + (size_t)hd * P + min(row_wg + i % RG, P - 1), IO);
        }
#pragma unroll
        for (int j = 0; j < BJ; ++j) {
            const int i = min(tid + 256 * j, 16 * VN - 1), s = min(i / VN, pd - 1);
            bv[j] = Vec::load_raw(wB, entry(s) * GN + (size_t)g * N + i % VN * EV);
        }
        d = load_io(wD, entry(min(tid & 15, pd - 1)) * H + hd, IO) + (p.dt_bias ? p.dt_bias[hd] : 0.f);
        if (p.dt_softplus) d = softplus_fast(d);
#pragma unroll
        for (int j = 0; j < XJ; ++j) sX[tid + 256 * j] = x[j];
#pragma unroll
        for (int j = 0; j < BJ; ++j) {
            const int i = tid + 256 * j;
            float f[EV];
            Vec::decode(bv[j], f);
            if (i < 16 * VN) {
#pragma unroll
                for (int e = 0; e < EV; e += 4) *reinterpret_cast<v4f *>(sB + i * EV + e) = v4f{f[e], f[e + 1], f[e + 2], f[e + 3]};
            }
        }
        if (tid < 16) sDt[tid] = d;
        __syncthreads();
        constexpr float LOG2E = 1.4426950408889634f;
        const float A = p.A[hd];
        v4f u[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) u[q] = v4f{0.f, 0.f, 0.f, 0.f};
        float after = 0.f;                               // sum of the later tokens' A dt
#pragma unroll 1
        for (int s = pd - 1; s >= 0; --s) {
            const float dt = sDt[s], w = dt * __builtin_amdgcn_exp2f(after * LOG2E);
            after = fmaf(A, dt, after);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const float wx = w * sX[s * RG + wave * RW + row_of(q)];
                const v4f B4 = *reinterpret_cast<const v4f *>(sB + s * N + col_of(q));
#pragma unroll
                for (int e = 0; e < 4; ++e) u[q][e] = fmaf(wx, B4[e], u[q][e]);
            }
        }
        const float a = __builtin_amdgcn_exp2f(after * LOG2E);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) h[q][e] = fmaf(a, h[q][e], u[q][e]);
        __syncthreads();                                 // the patches take the tokens' place
    }
    float *dst = p.h_out + head;
    if constexpr (TILED) {
        float *patch = lds + wave * RW * TS;
#pragma unroll
        for (int q = 0; q < NQ; ++q) *reinterpret_cast<v4f *>(patch + row_of(q) * TS + col_of(q)) = h[q];
        __builtin_amdgcn_wave_barrier();                 // the wave's own LDS traffic stays in program order
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int i = 64 * q + lane;
            h[q] = *reinterpret_cast<const v4f *>(patch + i / (N / 4) * TS + i % (N / 4) * 4);
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int i = 64 * q + lane, row = row_w + i / (N / 4);
        if (row < P) __builtin_nontemporal_store(h[q], reinterpret_cast<v4f *>(dst + (size_t)row * N + i % (N / 4) * 4));
    }
}

template <int N>
int launch_n(const VerifyParams &p, hipStream_t stream)
{
    const int rg = p.tiled || N <= 64 ? 64 : 4096 / N;  // rows of a workgroup, as in the kernel
    const dim3 grid((p.P + rg - 1) / rg, p.H, p.batch), block(256);
    if constexpr (N == 32 || N == 64 || N == 128) {
        if (p.tiled) {                                   // bf16 tokens, P a multiple of 64
            hipLaunchKernelGGL((materialize_kernel<N, true, SSMV_BF16>), grid, block, 0, stream, p);
            return (int)hipGetLastError();
        }
    }
    if (p.tiled) return (int)hipErrorInvalidConfiguration;
    if (p.io == SSMV_BF16) hipLaunchKernelGGL((materialize_kernel<N, false, SSMV_BF16>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((materialize_kernel<N, false, SSMV_F32>), grid, block, 0, stream, p);
    return (int)hipGetLastError();
}

}  // namespace

int launch_materialize(const VerifyParams &p, hipStream_t stream)
{
    switch (p.N) {
        case 16: return launch_n<16>(p, stream);
        case 32: return launch_n<32>(p, stream);
        case 64: return launch_n<64>(p, stream);
        case 128: return launch_n<128>(p, stream);
        case 256: return launch_n<256>(p, stream);
        default: return (int)hipErrorInvalidConfiguration;
    }
}

}  // namespace ssmv
