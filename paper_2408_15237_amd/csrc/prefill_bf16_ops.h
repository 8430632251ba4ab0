// What the two bf16 prefill kernels (prefill_bf16.hip, prefill_pipe.hip) have in common: loads into LDS, the operand layouts, the conv.
#pragma once

#include "ssmv_internal.h"

namespace ssmv {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr float kLog2e = 1.4426950408889634f;

// waves per 32-channel tile: a large state under a narrow head is split over n
__host__ __device__ constexpr int prefill_nsplit(int P, int N) { return (N >= 128 && P <= 64) ? 2 : 1; }

// Direct loads into LDS fill rows without padding, so the 16-byte pieces of row r of x, B and C sit at piece index (logical index ^
// key(r)).  A cycle serves 256 bytes: 16 lanes that read one logical piece out of 16 consecutive rows (operands of the
// products; B and C only), or 32 lanes of a transposing read, four adjacent pieces out of each of four rows.  So the rows that
// fall onto the same banks take different keys, and in the key's upper bits, which move groups of four pieces, if they
// are among the same four rows.
template <int N>
__device__ __forceinline__ constexpr int key_bc(int r)
{
    return N == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : N == 64 ? ((r & 2) << 1) | ((r & 4) >> 1) | ((r & 8) >> 3) : (r >> 2) & 3;
}
template <int P>
__device__ __forceinline__ constexpr int key_x(int r) { return P == 128 ? (r & 3) << 2 : P == 64 ? (r & 2) << 1 : 0; }

typedef __attribute__((address_space(3))) char lds_char_t;

// 16 bytes per lane from global memory straight into LDS: lane l's data lands at LDS address `dst` + 16 l (dst is the
// same in all lanes and travels in M0).  Issued from assembly, so that the compiler does not count these loads: it would
// otherwise wait for them before the next LDS read that it cannot prove to be disjoint from their target, and at every
// workgroup barrier.  The kernel waits for them itself (wait_direct_loads) ahead of the barrier that publishes the data.
// The address is a base that is the same in all lanes plus an unsigned byte offset.
// The base is copied by a scalar instruction: a vector memory access may read a scalar five wait states after a vector instruction wrote
// it (v_readfirstlane, or v_readlane of a spilled one), for which the compiler does not look in here, but at any time after a scalar
// instruction did, and that one waits for the vector instruction by itself.  The copy is also the wait state that M0 asks for.
// (Five wait states by s_nop cost 1 to 2 % of launches that fill the chip: 2048 pairs of 32 x 64, 1024 tokens, 189 us with two, 193 with five,
// 189 so.)
__device__ __forceinline__ void load_to_lds16(const void *base, uint32_t offset, const char *dst)
{
    const unsigned lds_addr = (unsigned)(size_t)(lds_char_t *)dst;
    const void *copy;
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0" : "=&s"(copy) : "v"(offset), "s"(base), "s"(lds_addr) : "memory", "m0");
}
// the same with 16 bits per lane, zero-extended: lane l's word at `dst` + 4 l
__device__ __forceinline__ void load_to_lds2(const void *base, uint32_t offset, const char *dst)
{
    const unsigned lds_addr = (unsigned)(size_t)(lds_char_t *)dst;
    const void *copy;
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_ushort %1, %0" : "=&s"(copy) : "v"(offset), "s"(base), "s"(lds_addr) : "memory", "m0");
}
// until at most COUNT of the wave's memory accesses are under way
template <int COUNT>
__device__ __forceinline__ void wait_direct_loads_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"i"(COUNT) : "memory"); }
__device__ __forceinline__ void wait_direct_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Transposing LDS read: in every 16 lanes, lane i gets element i % 4 of the 8 bytes at the address of each of the lanes i / 4,
// 4 + i / 4, 8 + i / 4, 12 + i / 4 (checked on the hardware).  With lane j's address in row j / 4, 8 bytes j % 4 of 32, that is
// column i of four rows.
__device__ __forceinline__ uint2 read_tr16(const char *at)
{
    typedef short s4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s4 lds_s4;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(lds_char_t *)at));
}

// Eight outputs of the conv from packed pairs of raw inputs (e: even-aligned, o: odd-aligned): x_(2i) = bias + w01 . o[i] + w23 .
// o[i + 1], x_(2i+1) = bias + w01 . e[i] + w23 . e[i + 1]; products exact, sums in fp32, the pair (w0, w1) first.  In assembly for the
// form with an addend of its own: the compiler takes the accumulating one and copies the bias ahead of each (16 of a chunk's
// 92 instructions for the conv).  A result of a dot product may be read three instructions later at the earliest: s_nop.
__device__ __forceinline__ void conv8(float (&x)[8], const uint32_t *o, const uint32_t *e, uint32_t w01, uint32_t w23, float bias)
{
    asm("v_dot2_f32_bf16 %0, %18, %8, %20\n\t"
        "v_dot2_f32_bf16 %1, %18, %13, %20\n\t"
        "v_dot2_f32_bf16 %2, %18, %9, %20\n\t"
        "v_dot2_f32_bf16 %3, %18, %14, %20\n\t"
        "v_dot2_f32_bf16 %4, %18, %10, %20\n\t"
        "v_dot2_f32_bf16 %5, %18, %15, %20\n\t"
        "v_dot2_f32_bf16 %6, %18, %11, %20\n\t"
        "v_dot2_f32_bf16 %7, %18, %16, %20\n\t"
        "v_dot2_f32_bf16 %0, %19, %9, %0\n\t"
        "v_dot2_f32_bf16 %1, %19, %14, %1\n\t"
        "v_dot2_f32_bf16 %2, %19, %10, %2\n\t"
        "v_dot2_f32_bf16 %3, %19, %15, %3\n\t"
        "v_dot2_f32_bf16 %4, %19, %11, %4\n\t"
        "v_dot2_f32_bf16 %5, %19, %16, %5\n\t"
        "v_dot2_f32_bf16 %6, %19, %12, %6\n\t"
        "v_dot2_f32_bf16 %7, %19, %17, %7\n\t"
        "s_nop 2"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
        : "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]), "v"(o[4]), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(w01), "v"(w23), "v"(bias));
}

// SiLU of eight conv outputs on their way to bf16: the bits of v / (1 + expf(-v)), rounded, which every other kernel's conv takes (a token's
// conv output is the same whichever call it comes through), for less than half of its instructions.  silu_fast is within 9 fp32 steps
// of that for every v >= -8 (all of them tried); rounding to bf16 gives the same then unless it is that close to the middle between two bf16
// numbers.  Such a result, and any v below -8 (silu_fast is off by 18 steps at -20 and gives 0 from -87.3 on), is computed as there: one
// in 3000 for values of order 1, so every sixth call of a wave.
// 1024 tokens with SiLU, gate and softplus (us), silu_fast alone, v / (1 + expf(-v)) alone, and so:  256 pairs of 128 x 64 57, 72, 65;  1024: 230, 293,
// 265;  256 of 64 x 128 58, 71, 63;  256 of 32 x 64 40, 51, 43.
__device__ __forceinline__ void conv_silu8(float (&v)[8])
{
    constexpr uint32_t kSteps = 10, kClose = 2 * kSteps << 16;
    constexpr float kLowest = -8.f;
    float f[8], lowest = v[0];
    uint32_t dist[8], closest = ~0u;                     // dist at most kClose: within kSteps of the middle
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        f[j] = silu_fast(v[j]);
        dist[j] = (__float_as_uint(f[j]) + (0x8000u + kSteps)) << 16;
        closest = min(closest, dist[j]);
        lowest = fminf(lowest, v[j]);
    }
    if (closest <= kClose || lowest < kLowest) {
        // One value of a lane after the other (two different ones are rare; the rows behind a prompt's end are all the same): the code for it
        // is there once and short, since the first wave that gets here waits for it to be fetched
        if (lowest < kLowest) {
#pragma unroll
            for (int j = 0; j < 8; ++j) dist[j] = v[j] < kLowest ? 0u : dist[j];
        }
        bool left;
        do {
            float a = v[7];
#pragma unroll
            for (int j = 6; j >= 0; --j) a = dist[j] <= kClose ? v[j] : a;
            const float exact = a / (1.f + expf(-a));
            left = false;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool hard = dist[j] <= kClose, same = __float_as_uint(v[j]) == __float_as_uint(a);
                f[j] = hard && same ? exact : f[j];
                dist[j] = same ? ~0u : dist[j];
                left = left || (hard && !same);
            }
        } while (left);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = f[j];
}

// two fp32 values -> packed bf16 heads and packed bf16 tails (first value in the low half)
__device__ __forceinline__ void split2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    hi = pack_bf16x2(a, b);
    lo = pack_bf16x2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

__device__ __forceinline__ bf8 as_bf8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    const uint4 u = make_uint4(a, b, c, d);
    return __builtin_bit_cast(bf8, u);
}
__device__ __forceinline__ bf8 as_bf8(uint4 u) { return __builtin_bit_cast(bf8, u); }

typedef float f4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4v mfma16(bf8 a, bf8 b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f16v mfma(bf8 a, bf8 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }

// inclusive prefix sums over lanes 0..31 and, separately, over lanes 32..63 (rows of 16 lanes: shifts inside a row,
// then the first row's total into the second); a lane shifted in from outside its row contributes 0
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or_zero(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float prefix32(float v)
{
    v += dpp_or_zero<0x111, 0xf>(v);     // row_shr:1
    v += dpp_or_zero<0x112, 0xf>(v);     // row_shr:2
    v += dpp_or_zero<0x114, 0xf>(v);     // row_shr:4
    v += dpp_or_zero<0x118, 0xf>(v);     // row_shr:8
    v += dpp_or_zero<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
    return v;
}

__device__ __forceinline__ int swap23(int i) { return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1); }

// Profiling builds only: per workgroup that has work, the shader-clock and the 100 MHz wall-clock ticks from its start to its end (the
// kernel of either file has a buffer pointer of its own; the last launch counts).
#ifdef SSMV_TRACE
__device__ long long *pf_trace_buf_ = nullptr;
#define SSMV_TRACE_BEGIN() const long long tr_c0 = clock64(), tr_w0 = wall_clock64()
#define SSMV_TRACE_END(one_thread)                                  \
    do {                                                            \
        if (pf_trace_buf_ && (one_thread)) {                        \
            pf_trace_buf_[2 * blockIdx.x] = clock64() - tr_c0;      \
            pf_trace_buf_[2 * blockIdx.x + 1] = wall_clock64() - tr_w0; \
        }                                                           \
    } while (0)
#else
#define SSMV_TRACE_BEGIN() (void)0
#define SSMV_TRACE_END(one_thread) (void)0
#endif

}  // namespace
}  // namespace ssmv
