// Small kernels around the fused verification kernel: the conv roll over the circular buffer
// (Section 4.3 footnote of arXiv 2408.15237), the integer commit/rollback of Algorithm 2,
// FirstConflict, cache reset, and a plain copy kernel for bandwidth calibration.
#include "ssmv_internal.h"

namespace ssmv {

// one element at a time, for channel counts that are no multiple of the 16-byte vector
template <int IO>
struct IoOne {
    static constexpr int EV = 1;
    static __device__ __forceinline__ void load(const void *base, size_t idx, float (&v)[1]) { v[0] = load_io(base, idx, IO); }
    static __device__ __forceinline__ void store(void *base, size_t idx, const float (&v)[1]) { store_io(base, idx, v[0], IO); }
};

// ---- conv roll -----------------------------------------------------------------------------------
// One thread owns VEC adjacent channels of one sequence for all k tokens: it reads the W-1 newest
// committed ring entries, then per new token appends the raw input to the ring and emits the
// width-4 causal dot product.  Ring slots written are head+1..head+k, slots read are
// head-2..head, disjoint because R >= W-1+kmax.
template <int IO, typename VT>
__global__ __launch_bounds__(256) void conv_kernel(const ConvParams p)
{
    constexpr int W = SSMV_CONV_WIDTH;
    constexpr int VEC = VT::EV;
    const int chunks = p.Cx / VEC;
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (long)p.batch * chunks) return;
    const int b = (int)(gid / chunks);
    const int c0 = (int)(gid - (long)b * chunks) * VEC;
    const int head = p.conv_head[b];
    const int mask = p.R - 1;

    float hist[W - 1][VEC];
#pragma unroll
    for (int i = 0; i < W - 1; ++i)
        VT::load(p.ring, ((size_t)b * p.R + ((head - (W - 2) + i) & mask)) * p.Cx + c0, hist[i]);

    float w[VEC][W];
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
        for (int i = 0; i < W; ++i) w[c][i] = load_io(p.wgt, (size_t)(c0 + c) * W + i, IO);
    float bias[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) bias[c] = p.bias ? load_io(p.bias, c0 + c, IO) : 0.f;

    for (int t = 0; t < p.k; ++t) {
        float x[VEC], out[VEC];
        VT::load(p.x_raw, ((size_t)b * p.k + t) * p.Cx + c0, x);
        VT::store(p.ring, ((size_t)b * p.R + ((head + 1 + t) & mask)) * p.Cx + c0, x);
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            float s = bias[c];
            s = fmaf(w[c][0], hist[0][c], s);
            s = fmaf(w[c][1], hist[1][c], s);
            s = fmaf(w[c][2], hist[2][c], s);
            s = fmaf(w[c][3], x[c], s);
            if (p.act == SSMV_ACT_SILU) s = s / (1.f + expf(-s));
            out[c] = s;
            hist[0][c] = hist[1][c];
            hist[1][c] = hist[2][c];
            hist[2][c] = x[c];
        }
        VT::store(p.xc, ((size_t)b * p.k + t) * p.Cx + c0, out);
    }
}

int launch_conv(const ConvParams &p, hipStream_t stream)
{
    const int vec = p.io == SSMV_BF16 ? 8 : 4;
    const bool vec_ok = (p.Cx % vec) == 0;
    const long threads = (long)p.batch * (vec_ok ? p.Cx / vec : p.Cx);
    const int block = 256;
    const unsigned grid = (unsigned)((threads + block - 1) / block);
    if (p.io == SSMV_BF16) {
        if (vec_ok) hipLaunchKernelGGL((conv_kernel<SSMV_BF16, IoVec<SSMV_BF16>>), dim3(grid), dim3(block), 0, stream, p);
        else hipLaunchKernelGGL((conv_kernel<SSMV_BF16, IoOne<SSMV_BF16>>), dim3(grid), dim3(block), 0, stream, p);
    } else {
        if (vec_ok) hipLaunchKernelGGL((conv_kernel<SSMV_F32, IoVec<SSMV_F32>>), dim3(grid), dim3(block), 0, stream, p);
        else hipLaunchKernelGGL((conv_kernel<SSMV_F32, IoOne<SSMV_F32>>), dim3(grid), dim3(block), 0, stream, p);
    }
    return (int)hipGetLastError();
}

// ---- commit / rollback (Algorithm 2: "return h_k if k'=k else h_j", lazily advanced cache) -----------
// grid.y = cache (layer), one thread per sequence.  Every load is issued before the first use:
// the kernel is a chain of memory latencies and nothing else.
__global__ __launch_bounds__(256) void commit_kernel(const CommitParams p)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= p.batch) return;
    const CacheInts &c = p.c[blockIdx.y];
    const int lk = c.last_k[b];
    int a = p.accepted[b];
    const int cur = c.cur_slot[b];
    const int pd = c.pend[b];
    const int head = c.conv_head[b];
    const int64_t pos = c.pos[b];
    const int par = b == 0 ? *c.win_par : 0;
    if (lk == 0) {                       // nothing was verified: leave everything, flag it
        *c.err_flag = 1;
        return;
    }
    if (a < 0 || a > lk) {
        *c.err_flag = 1;
        a = a < 0 ? 0 : lk;
    }
    if (p.mode == SSMV_SNAP_DEFER) {     // deferred advance: the live slot moves only when the verify stored h_j
        if (pd > p.pend_hi) {
            c.cur_slot[b] = (cur + 1) % 3;
            c.pos[b] = pos + pd;
            c.pend[b] = a;
        } else {
            c.pend[b] = pd + a;
        }
    } else if (a == lk && p.mode == SSMV_SNAP_BOTH) {   // every draft accepted: h_k becomes the live state
        c.cur_slot[b] = (cur + 2) % 3;
        c.pos[b] = pos + pd + a;
        c.pend[b] = 0;
    } else if (pd > 0) {                 // rejection: fall back to h_j, the accepted prefix stays pending
        c.cur_slot[b] = (cur + 1) % 3;
        c.pos[b] = pos + pd;
        c.pend[b] = a;
    } else {                             // rejection with nothing pending: the live slot already is h_j
        c.pend[b] = a;
    }
    c.conv_head[b] = (head + a) & (p.R - 1);
    c.last_k[b] = 0;
    if (b == 0) *c.win_par = par ^ 1;
}

int launch_commit(const CommitParams &p, hipStream_t stream)
{
    const int block = 256;
    hipLaunchKernelGGL(commit_kernel, dim3((p.batch + block - 1) / block, p.n_caches), dim3(block), 0, stream, p);
    return (int)hipGetLastError();
}

// ---- FirstConflict ----------------------------------------------------------------------------------
// A lane per token: a wave compares the tokens of as many whole sequences as fit 64 lanes (longer ones a wave each, 64 tokens at
// a time and no further than the first conflict), in coalesced requests, and a sequence's count is the position of the first set
// bit of its share of the ballot.  In large launches a wave takes U such shares and requests all of them at once.
// (Launches back to back in a graph, operands in the L2, us.  A lane per sequence, one token after the other: a round trip per
// agreement; eight tokens a lane at once: accesses k tokens apart, also where the first token already disagrees.
//   k = 8, 32 sequences:     all agree 2.23 / 1.83 / so 1.86, first disagrees 1.84 / 1.82 / 1.87
//   k = 16, 512 sequences:   all agree 4.80 / 4.79 / 1.98,    first disagrees 1.84 / 3.09 / 1.98
//   k = 8, 10^6 sequences:   all agree 34.2 / 30.0 / 13.4,    first disagrees 10.7 / 30.1 / 13.4)
// per = sequences of a wave's share, 0 = longer than 64 tokens; inv = 2^16 / k rounded up: lane * inv >> 16 = lane / k
template <int U>
__global__ __launch_bounds__(256) void first_conflict_kernel(const int32_t *draft, const int32_t *target, int batch, int k, int per, int inv,
                                                             long shares, int32_t *accepted)
{
    const int lane = threadIdx.x & 63;
    const long first = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * U, stride = (long)gridDim.x * 4 * U;
    if (per > 0) {
        const int s = lane * inv >> 16, t = lane - s * k;                 // the lane's sequence of the share, and its token
        for (long share = first; share < shares; share += stride) {
            bool wrong[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const long b = (share + u) * per + s;
                wrong[u] = false;
                if (s < per && b < batch) wrong[u] = draft[(size_t)b * k + t] != target[(size_t)b * k + t];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const long b = (share + u) * per + s;
                const unsigned long long w = __ballot(wrong[u]) >> (s * k);
                if (s < per && b < batch && t == 0) accepted[b] = w ? min(__builtin_ctzll(w), k) : k;
            }
        }
        return;
    }
    for (long b = first; b < batch; b += stride) {                        // U = 1
        unsigned n = 0;
        unsigned long long w;
        do {
            const unsigned t = n + lane;
            w = __ballot(t < (unsigned)k && draft[(size_t)b * k + t] != target[(size_t)b * k + t]);
            n += 64;
        } while (!w && n < (unsigned)k);
        if (lane == 0) accepted[b] = w ? (int)(n - 64) + __builtin_ctzll(w) : k;
    }
}

int launch_first_conflict(const int32_t *draft, const int32_t *target, int batch, int k, int32_t *accepted, hipStream_t stream)
{
    const int per = k <= 64 ? 64 / k : 0, inv = per ? (65536 + k - 1) / k : 0;
    const long shares = per ? (batch + (per - 1L)) / per : batch;
    const bool many = per && shares >= 32768;                             // eight waves per SIMD even so
    const long per_wg = many ? 16 : 4, wgs = (shares + per_wg - 1) / per_wg;
    const dim3 grid((unsigned)(wgs < 65536 ? wgs : 65536));
    if (many) hipLaunchKernelGGL(first_conflict_kernel<4>, grid, dim3(256), 0, stream, draft, target, batch, k, per, inv, shares, accepted);
    else hipLaunchKernelGGL(first_conflict_kernel<1>, grid, dim3(256), 0, stream, draft, target, batch, k, per, inv, shares, accepted);
    return (int)hipGetLastError();
}

// ---- reset (a fill kernel, so that a caller may capture it in a graph) ------------------------------------
// One launch: the first `state_wgs` workgroups fill the state, eight 16-byte vectors a thread, the others the ring, a vector a
// thread.  An empty start (no h0, no history) is a plain fill: no index arithmetic, whatever the layout.
// (32 x 32 x 128 x 64 and its ring: 12.6 us as two kernels with the layout worked out per vector, 6.9 so; 1 x 32 x 128 x 64: 4.0, 2.2.)
constexpr int kResetVecs = 8;

template <int IO>
__global__ __launch_bounds__(256) void reset_kernel(const ResetParams p, unsigned state_wgs)
{
    typedef float v4 __attribute__((ext_vector_type(4)));
    const unsigned wg = blockIdx.x, tid = threadIdx.x;
    if (wg < state_wgs) {
        const unsigned n4 = (unsigned)(p.state_elems / 4);       // N is a multiple of 4, so is the slot size; < 2^31 (host)
        const unsigned base = wg * (256 * kResetVecs) + tid;
        if (!p.h0) {
#pragma unroll
            for (int u = 0; u < kResetVecs; ++u)
                if (base + u * 256 < n4) reinterpret_cast<v4 *>(p.state)[base + u * 256] = v4{0.f, 0.f, 0.f, 0.f};
            return;
        }
        v4 v[kResetVecs];
#pragma unroll
        for (int u = 0; u < kResetVecs; ++u) v[u] = reinterpret_cast<const v4 *>(p.h0)[min(base + u * 256, n4 - 1)];
        const unsigned blk4 = (unsigned)p.P * p.N / 4, row4 = (unsigned)p.N / 4;
#pragma unroll
        for (int u = 0; u < kResetVecs; ++u) {
            const unsigned i = base + u * 256;
            if (i >= n4) continue;
            size_t o = (size_t)i * 4;
            if (p.tiled) {                         // h0 is row-major; the slot keeps each (sequence, head) block in tiles
                const unsigned head = i / blk4, e = i - head * blk4;
                o = (size_t)head * blk4 * 4 + state_off4(true, (int)(e / row4), (int)(e % row4) * 4, p.N);
            }
            *reinterpret_cast<v4 *>(p.state + o) = v[u];
        }
        return;
    }
    using Vec = IoVec<IO>;
    constexpr int EV = Vec::EV;
    const unsigned i = (wg - state_wgs) * 256 + tid;               // 16-byte vector of the ring
    const size_t n = (size_t)p.batch * p.R * p.Cx;
    const size_t e0 = (size_t)i * EV;
    if (e0 < n) {
        if (e0 + EV <= n && (!p.conv_init || p.Cx % EV == 0)) {    // a whole vector, of one row of the ring
            uint4 v = make_uint4(0, 0, 0, 0);
            if (p.conv_init) {
                const unsigned br = (unsigned)(e0 / (unsigned)p.Cx), c = (unsigned)(e0 - (size_t)br * p.Cx);
                const unsigned b = br / (unsigned)p.R, slot = br - b * p.R;
                if ((int)slot < p.W - 1) v = Vec::load_raw(p.conv_init, ((size_t)b * (p.W - 1) + slot) * p.Cx + c);
            }
            Vec::store_raw(p.ring, e0, v);
        } else {
            float v[EV];
#pragma unroll
            for (int u = 0; u < EV; ++u) {                         // requested together; past the end the last element again
                const size_t e = e0 + u < n ? e0 + u : n - 1;
                const unsigned br = (unsigned)(e / (unsigned)p.Cx), c = (unsigned)(e - (size_t)br * p.Cx);
                const unsigned b = br / (unsigned)p.R, slot = br - b * p.R;
                v[u] = 0.f;
                if (p.conv_init && (int)slot < p.W - 1) v[u] = load_io(p.conv_init, ((size_t)b * (p.W - 1) + slot) * p.Cx + c, IO);
            }
#pragma unroll
            for (int u = 0; u < EV; ++u)
                if (e0 + u < n) store_io(p.ring, e0 + u, v[u], IO);
        }
    }
    if (i < (unsigned)p.batch) {                   // the ring has at least four elements per sequence, but a vector holds eight
        p.cur_slot[i] = 0;
        p.pend[i] = 0;
        p.pos[i] = 0;
        p.conv_head[i] = p.W - 2;
        p.last_k[i] = 0;
    }
    if (i == 0) {
        *p.win_par = 0;
        *p.err_flag = 0;
    }
}

int launch_reset(const ResetParams &p, hipStream_t stream)
{
    const unsigned per_wg = 256 * kResetVecs;
    const unsigned state_wgs = (unsigned)((p.state_elems / 4 + per_wg - 1) / per_wg);
    const size_t ring = (size_t)p.batch * p.R * p.Cx, ev = p.io == SSMV_BF16 ? 8 : 4;
    size_t vecs = (ring + ev - 1) / ev;
    if (vecs < (size_t)p.batch) vecs = p.batch;
    const dim3 grid(state_wgs + (unsigned)((vecs + 255) / 256));
    if (p.io == SSMV_BF16) hipLaunchKernelGGL(reset_kernel<SSMV_BF16>, grid, dim3(256), 0, stream, p, state_wgs);
    else hipLaunchKernelGGL(reset_kernel<SSMV_F32>, grid, dim3(256), 0, stream, p, state_wgs);
    return (int)hipGetLastError();
}

// ---- plain copy: read n bytes, write them once or twice ----------------------------------------------
typedef float copy_v4f __attribute__((ext_vector_type(4)));

// A workgroup copies contiguous tiles of 8 x 256 float4 (32 KiB): eight loads in flight per thread, then the
// stores - the verify kernel's shape - with the same streaming hints as its state traffic.
__global__ __launch_bounds__(256) void copy_probe_kernel(const copy_v4f *__restrict__ src, copy_v4f *__restrict__ dst0,
                                                         copy_v4f *__restrict__ dst1, size_t n16)
{
    constexpr int U = 8;
    const size_t tiles = (n16 + U * 256 - 1) / (U * 256);
    for (size_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const size_t base = tile * (U * 256) + threadIdx.x;
        copy_v4f v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t i = base + u * 256;
            v[u] = __builtin_nontemporal_load(src + (i < n16 ? i : n16 - 1));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t i = base + u * 256;
            if (i < n16) {
                __builtin_nontemporal_store(v[u], dst0 + i);
                if (dst1) __builtin_nontemporal_store(v[u], dst1 + i);
            }
        }
    }
}

// sum over the 64 lanes, the same in every lane (row shifts, then row totals handed on; lanes shifted in from outside add 0)
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v = dpp_add<0x111, 0xf>(v);     // row_shr:1, 2, 4, 8: lane 15 of a row holds the row's sum
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);     // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Gated RMS norm of a Mamba-2 block: g = y * z * sigmoid(z) (or y without z); out = g * rsqrt(mean_group(g^2) + eps) * w.
// `gt` threads (64, 128 or 256) per (token row, group), as many groups of a row per workgroup as fit 256 threads; a thread takes
// MV 16-byte vectors of its group in each of ROWS token rows.  Everything is requested before the first wait, the weights too: a
// small launch is one round trip to memory and a reduction, and behind the reduction the weights were a second round trip.  The
// sum of squares goes through DPP row operations, over the waves of a group through LDS; a group of one wave needs neither
// LDS nor a barrier.  (128 x 4096, one group, bf16, against the weights behind the reduction and shuffles: 2.92 -> 2.33 us on buffers
// in the L2, 4.34 -> 3.19 rotating over 1 GiB.)
template <int IO, int MV, int ROWS>
__global__ __launch_bounds__(256) void gated_rmsnorm_kernel(const void *y, const void *z, const float *weight, int rows, int channels,
                                                            int group, int gt, float eps, void *out)
{
    using Vec = IoVec<IO>;
    constexpr int EV = Vec::EV;
    __shared__ float partial[ROWS][4];
    const int sub = threadIdx.x / gt, tid = threadIdx.x % gt, gpb = blockDim.x / gt, nvec = group / EV;
    const int grp = min(blockIdx.y * gpb + sub, channels / group - 1);        // the last workgroup of a row may hold fewer groups:
    const bool have = blockIdx.y * gpb + sub == grp;                          // the rest repeat its last one and store nothing
    const int row0 = blockIdx.x * ROWS;
    // rows and vectors past the end read the last one again
    auto at = [&](int r, int v) { return (size_t)min(row0 + r, rows - 1) * channels + (size_t)grp * group + (size_t)min(v, nvec - 1) * EV; };
    uint4 yr[ROWS][MV], zr[ROWS][MV];
    float4 w[MV][EV / 4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            yr[r][i] = Vec::load_raw(y, at(r, tid + i * gt));
            if (z) zr[r][i] = Vec::load_raw(z, at(r, tid + i * gt));
        }
#pragma unroll
    for (int i = 0; i < MV; ++i)
#pragma unroll
        for (int e = 0; e < EV / 4; ++e)
            w[i][e] = reinterpret_cast<const float4 *>(weight + (size_t)grp * group + (size_t)min(tid + i * gt, nvec - 1) * EV)[e];
    __builtin_amdgcn_sched_barrier(0);
    float g[ROWS][MV][EV], ss[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        ss[r] = 0.f;
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            Vec::decode(yr[r][i], g[r][i]);
            if (z) {
                float zv[EV];
                Vec::decode(zr[r][i], zv);
#pragma unroll
                for (int e = 0; e < EV; ++e) g[r][i][e] *= silu_fast(zv[e]);
            }
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < EV; ++e) s = fmaf(g[r][i][e], g[r][i][e], s);
            ss[r] += tid + i * gt < nvec ? s : 0.f;
        }
        ss[r] = wave_sum(ss[r]);
    }
    if (gt > 64) {
        const int wv = threadIdx.x >> 6, first = sub * (gt >> 6);
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) partial[r][wv] = ss[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            ss[r] = partial[r][first] + partial[r][first + 1];
            if (gt > 128) ss[r] += partial[r][2] + partial[r][3];
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const float scale = rsqrtf(ss[r] / (float)group + eps);
#pragma unroll
        for (int i = 0; i < MV; ++i) {
            float o[EV];
#pragma unroll
            for (int e = 0; e < EV; ++e) {
                const float4 w4 = w[i][e / 4];
                o[e] = g[r][i][e] * scale * (e % 4 == 0 ? w4.x : e % 4 == 1 ? w4.y : e % 4 == 2 ? w4.z : w4.w);
            }
            if (have && row0 + r < rows && tid + i * gt < nvec) Vec::store(out, at(r, tid + i * gt), o);
        }
    }
}

// Four rows per workgroup only for groups that leave lanes of their wave idle, in launches of sixteen waves and more per compute
// unit: more bytes under way per wave, and the weights (fp32, for bf16 tensors twice the bytes of a row of y) fetched once for the
// four.  A full wave is slower so (bf16 with z, rotating over 500 MB: 16 of 64 lanes, 2048 x 1024 in groups of 128, 7.84 us with
// one row and 7.27 with four, 32768 rows 87 and 69; 64 lanes, 4096 x 2048 in groups of 512, 12.0 and 13.0; 128 vectors on
// 64 lanes, 4096 x 1024 in one group, 7.4 and 9.0).
template <int IO>
static int launch_norm_io(const void *y, const void *z, const float *weight, int rows, int channels, int group, float eps, void *out, hipStream_t stream)
{
    const int nvec = group / IoVec<IO>::EV, ngroups = channels / group;
    const int gt = nvec > 256 ? 256 : nvec > 128 ? 128 : 64;           // threads per group: two vectors each beat one and another wave
    const int mv = (nvec + gt - 1) / gt;                                // 1 .. 4
    const int rows_wg = nvec < 64 && (long)rows * ngroups >= 16384 ? 4 : 1;
    // groups of a row per workgroup: as many as fit 256 threads, spread evenly, and no threads for groups that there are not
    // (2048 x 1280 in one group, bf16 with z: 4.6 us with its 128 threads, 6.4 with 128 idle ones beside them)
    const int tiles = (ngroups + 256 / gt - 1) / (256 / gt), gpb = (ngroups + tiles - 1) / tiles;
    const dim3 grid((rows + rows_wg - 1) / rows_wg, tiles), block(gt * gpb);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, y, z, weight, rows, channels, group, gt, eps, out); };
    if (rows_wg == 4) go(gated_rmsnorm_kernel<IO, 1, 4>);
    else if (mv <= 1) go(gated_rmsnorm_kernel<IO, 1, 1>);
    else if (mv <= 2) go(gated_rmsnorm_kernel<IO, 2, 1>);
    else go(gated_rmsnorm_kernel<IO, 4, 1>);
    return (int)hipGetLastError();
}

int launch_gated_rmsnorm(const void *y, const void *z, const float *weight, int rows, int channels, int group, float eps, int io,
                         void *out, hipStream_t stream)
{
    return io == SSMV_BF16 ? launch_norm_io<SSMV_BF16>(y, z, weight, rows, channels, group, eps, out, stream)
                           : launch_norm_io<SSMV_F32>(y, z, weight, rows, channels, group, eps, out, stream);
}

// ---- bandwidth probe: what the memory system gives a plain stream of a given direction and shape --------------------------
// MODE 0 read only, 1 write only, 2 read 1 / write 1, 3 read 1 / write 2, 4 nothing (the floor of a launch).  A workgroup of
// 256 threads takes contiguous pieces of U x 4 KiB (a wave instruction = 1 KiB), non-temporal as the verify kernel's state.
template <int MODE, int U>
__global__ __launch_bounds__(256) void stream_probe_kernel(const copy_v4f *__restrict__ src, copy_v4f *__restrict__ dst0,
                                                           copy_v4f *__restrict__ dst1, size_t n16)
{
    if (MODE == 4) return;
    const size_t tiles = n16 / (U * 256);
    for (size_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const size_t base = tile * (U * 256) + threadIdx.x;
        copy_v4f v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = MODE == 1 ? copy_v4f{(float)tile, 1.f, 2.f, 3.f} : __builtin_nontemporal_load(src + base + u * 256);
        if (MODE == 0) {
            float a = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) a += v[u].x + v[u].y + v[u].z + v[u].w;
            if (a == 123.456f) dst0[base] = v[0];            // keeps the loads alive; practically never taken
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                __builtin_nontemporal_store(v[u], dst0 + base + u * 256);
                if (MODE == 3) __builtin_nontemporal_store(v[u], dst1 + base + u * 256);
            }
        }
    }
}

template <int MODE>
static void launch_probe_u(int u, unsigned grid, const copy_v4f *s, copy_v4f *d0, copy_v4f *d1, size_t n16, hipStream_t stream)
{
    if (u == 1) hipLaunchKernelGGL((stream_probe_kernel<MODE, 1>), dim3(grid), dim3(256), 0, stream, s, d0, d1, n16);
    else if (u == 2) hipLaunchKernelGGL((stream_probe_kernel<MODE, 2>), dim3(grid), dim3(256), 0, stream, s, d0, d1, n16);
    else hipLaunchKernelGGL((stream_probe_kernel<MODE, 8>), dim3(grid), dim3(256), 0, stream, s, d0, d1, n16);
}

int launch_stream_probe(int mode, const void *src, void *dst0, void *dst1, size_t n_bytes, int piece_kib, int grid, hipStream_t stream)
{
    const size_t n16 = n_bytes / 16;
    const int u = piece_kib / 4;
    const size_t tiles = n16 / ((size_t)u * 256);
    const unsigned g = grid > 0 ? (unsigned)grid : (unsigned)(tiles > 0x7fffffff ? 0x7fffffff : tiles);
    const copy_v4f *s = reinterpret_cast<const copy_v4f *>(src);
    copy_v4f *d0 = reinterpret_cast<copy_v4f *>(dst0), *d1 = reinterpret_cast<copy_v4f *>(dst1);
    switch (mode) {
        case 0: launch_probe_u<0>(u, g, s, d0, d1, n16, stream); break;
        case 1: launch_probe_u<1>(u, g, s, d0, d1, n16, stream); break;
        case 2: launch_probe_u<2>(u, g, s, d0, d1, n16, stream); break;
        case 3: launch_probe_u<3>(u, g, s, d0, d1, n16, stream); break;
        default: launch_probe_u<4>(u, g, s, d0, d1, n16, stream); break;
    }
    return (int)hipGetLastError();
}

int launch_copy_probe(const void *src, void *dst0, void *dst1, size_t n_bytes, hipStream_t stream)
{
    const size_t n16 = n_bytes / 16;
    const size_t tiles = (n16 + 8 * 256 - 1) / (8 * 256);
    const unsigned grid = (unsigned)(tiles > 65536 ? 65536 : tiles);
    hipLaunchKernelGGL(copy_probe_kernel, dim3(grid), dim3(256), 0, stream, reinterpret_cast<const copy_v4f *>(src),
                       reinterpret_cast<copy_v4f *>(dst0), reinterpret_cast<copy_v4f *>(dst1), n16);
    return (int)hipGetLastError();
}

}  // namespace ssmv
