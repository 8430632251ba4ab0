// A prompt cut into segments.  One workgroup per (sequence, head) walks the chunks of a prompt one after the other, so a
// launch with fewer (sequence, head) pairs than the chip holds workgroups leaves most of it idle however long the prompt
// is.  Eq. 1 is linear in the state: a segment of the prompt maps the state h before it to  2^d h + u,  with d the segment's
// summed decay exponent and u its state when it starts from zero.  So such a prompt takes three launches:
//   pass 0   segment 0 starts from the live slot and does everything; segments 1 .. n-2 form (u, d) only, side by side;
//   combine  the states ahead of segments 1 .. n-1, one after the other but each element on its own (prefill.hip); also moves
//            pos and conv_head on, which no launch of pass 0 is still reading;
//   pass 1   segments 1 .. n-1 start from those states and write their outputs; the last one leaves the state in the live
//            slot and the ring.
// The library owns no memory, so (u, d) and the states travel in rows of y that nobody has written yet: a segment's own, and
// for segment 0 (which does write its own in pass 0) the last segment's, whose u nobody needs.  A state is P N floats, that
// is 4 N / sizeof(element) rows of a head's share of y, which bounds a segment's length from below.  The host takes this path
// only if y overlaps none of the inputs.
#pragma once

#include "ssmv_internal.h"

namespace ssmv {

constexpr int kPrefillChunk = 32;      // tokens per chunk

struct Segment {
    int c0, c1;          // its chunks
    int area;            // first token of the rows of y that hold its state between the launches
    bool work;           // there is something to do in this pass
    bool emit;           // it writes outputs in this pass
    bool last;           // it ends the prompt
};

// a prompt of n chunks: every segment has seg_chunks chunks, but the first one has what is left
__host__ __device__ inline int segments_of(int seg_chunks, int n_chunks) { return 1 + (n_chunks - 1) / seg_chunks; }
__host__ __device__ inline int segment_begin(int seg_chunks, int n_chunks, int s)
{
    return s == 0 ? 0 : n_chunks - (segments_of(seg_chunks, n_chunks) - s) * seg_chunks;
}

// what workgroup number `slot` (0 .. seg_count - 2) of a (sequence, head) does in this pass; L >= 1
__device__ __forceinline__ Segment segment_of(const PrefillParams &p, int L, int slot)
{
    const int n = (L + kPrefillChunk - 1) / kPrefillChunk, ns = segments_of(p.seg_chunks, n);
    const int s = slot + p.seg_pass;
    Segment g;
    g.last = s == ns - 1;
    g.work = p.seg_pass ? s < ns : (s == 0 || s < ns - 1);
    g.emit = p.seg_pass || s == 0;
    g.c0 = segment_begin(p.seg_chunks, n, s);
    g.c1 = segment_begin(p.seg_chunks, n, s + 1);
    g.area = (s == 0 ? segment_begin(p.seg_chunks, n, ns - 1) : g.c0) * kPrefillChunk;
    return g;
}

// Which (sequence, head[, segment slot]) a workgroup takes.  Prompts of one length: the heads of a sequence on one XCD
// (xcd_contiguous), B and C then come out of its L2.  Prompts of different lengths: consecutive workgroups over all XCDs, and where
// prompts are of more than two chunks and some compute unit gets more than one, the longest first.  Contiguous ranges would give an
// XCD nothing but one long prompt's heads and another nothing but a short one's, and a long prompt that starts last ends alone.
// (Lengths drawn from 1 up, bf16: 32 sequences x 32 heads x 128 x 64, 2048 tokens at most 453-515 -> 313-377 us; 20 x 80 x 64 x 128,
// 700 at most 238-275 -> 179-205; 5 x 80: 102 -> 80.  The ranking costs 0.3 us, one round trip and a count over the batch, which
// nothing gives back on short prompts and small launches: 20 x 80 x 64 x 128, 64 at most, contiguous 38-41, ranked 38-40, spread
// only 34-38; 12 x 12 x 128 x 64, 128 at most: 14.1, 14.4, 14.1.)
struct PrefillItem { int hd, b, L, slot; };
template <bool SEG>
__device__ __forceinline__ PrefillItem prefill_item(const PrefillParams &p)
{
    PrefillItem w;
    auto take = [&](unsigned item) {
        const unsigned q = item / (unsigned)p.H;
        w.hd = (int)(item - q * p.H);
        w.slot = SEG ? (int)(q / (unsigned)p.batch) : 0;
        w.b = (int)(q - w.slot * (unsigned)p.batch);
    };
    if (!p.seq_len) {
        take(xcd_contiguous(blockIdx.x, gridDim.x));
        w.L = p.L;
        return w;
    }
    take(blockIdx.x);
    if (p.batch <= 64 && p.L > 2 * kPrefillChunk && p.H * p.batch > 256) {
        // lane j knows sequence j: the one with w.b longer ones ahead of it.
        // (len, lane) as one number, all different: a rank is a count of greater ones.  Eight at a time: lanes without a sequence
        // hold numbers below all others
        const int lane = threadIdx.x & 63;
        const int len = lane < p.batch ? min(max(p.seq_len[lane], 0), p.L) : -1, key = len * 64 + (63 - lane);
        int ahead = 0;
        for (int j0 = 0; j0 < p.batch; j0 += 8) {
#pragma unroll
            for (int j = 0; j < 8; ++j) ahead += __builtin_amdgcn_readlane(key, j0 + j) > key;
        }
        w.b = __builtin_ctzll(__ballot(lane < p.batch && ahead == w.b));
        w.L = __builtin_amdgcn_readlane(len, w.b);
    } else {
        w.L = min(max(p.seq_len[w.b], 0), p.L);
    }
    return w;
}

// byte offset, from the sequence's first row of y, of 16-byte piece i of a state kept in head hd's rows from token t on;
// ES = bytes of an element of y.  Piece P N / 4, behind the state, holds d.
template <int ES>
__device__ __forceinline__ size_t seg_piece(int i, int P, int t, int HP, int hd)
{
    const int ppr = P * ES / 16;                         // pieces per row
    return ((size_t)(t + i / ppr) * HP + (size_t)hd * P) * ES + (size_t)(i % ppr) * 16;
}

}  // namespace ssmv
