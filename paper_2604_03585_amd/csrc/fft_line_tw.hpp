// fft_line_tw.hpp -- the line transform with twiddles applied ahead of each
// butterfly, the radix-16 ones as products of two table entries or (TAB) all from
// the table.
//
// The first serves data that are about to be stored as FP16.  The transform of
// fft_line.hpp has its radix-16 twiddles inside the butterflies' FMAs and rounds
// differently in the last FP32 bits.  Where the result is rounded to FP16 next
// (half storage: the range output and the range-Doppler rows) such a last-bit
// change moves a few values by a whole FP16 step (2^-11 relative; 2.3e-5 relative
// L2 of a 4096^2 image, against 2.5e-4 from the FP16 rounding itself), so those
// two passes keep this form, whose stored bits callers have.  They are bound by
// memory, not by the instruction count (range pass of 4096^2: 66 us against 54 us
// for a plain copy of its FP32 input and output).
// The second is the autotuner's table-twiddle variant of the FP32 line kernels
// (relative L2 of Gaussian noise 0.95e-7 at 256 points, 1.22e-7 at 4096, 1.32e-7 at
// 16384).
#pragma once

#include "fft_line.hpp"

namespace sar {
namespace tw_first {

// Radix-16 pass: W^1 and W^4 come from the table, the other powers are
// products (at most four roundings deep, ~3e-7 relative).  Thirteen complex
// products replace thirteen table reads, for kernels bound by vector-memory
// issue rather than by VALU.  w[i-1] = W^i, w[0] and w[3] given.
__device__ __forceinline__ void tw_products16(float2* w)
{
    w[1] = c_mul(w[0], w[0]);
    w[2] = c_mul(w[1], w[0]);
    w[4] = c_mul(w[3], w[0]);
    w[5] = c_mul(w[3], w[1]);
    w[6] = c_mul(w[3], w[2]);
    w[7] = c_mul(w[3], w[3]);
#pragma unroll
    for (int i = 8; i < 15; ++i) w[i] = c_mul(w[7], w[i - 8]);
}

// TAB: every twiddle from the table, no products.
template <int N, int P, bool TAB>
__device__ __forceinline__ void load_tw(PassTw<N, P>& pt, const float2* __restrict__ tw, int t)
{
    using G = LineGeom<N>;
    if constexpr (!TAB && PassTw<N, P>::ANY && G::radix(P) == 16) {
        constexpr int NS = G::span(P);
        const int jm = t & (NS - 1);
        pt.w[0] = tw_ld<N, P>(tw, jm, 0);
        pt.w[3] = tw_ld<N, P>(tw, jm, 3 * NS);
        tw_products16(pt.w);
    } else {
        read_tw<N, P>(pt, tw, t);
    }
}

// The table reads of a radix-16 pass (W^1, W^4), issued one pass ahead so that
// their latency overlaps the previous pass and its LDS exchange; other passes
// read their twiddles when they start.
template <int N, int P, bool TAB> struct TwAhead {
    static constexpr bool ON = !TAB && PassTw<N, P>::ANY && LineGeom<N>::radix(P) == 16;
    float2 w1, w4;
};

template <int N, int P, bool TAB>
__device__ __forceinline__ void tw_issue(TwAhead<N, P, TAB>& a, const float2* __restrict__ tw, int t)
{
    if constexpr (TwAhead<N, P, TAB>::ON) {
        using G = LineGeom<N>;
        constexpr int NS = G::span(P);
        const int jm = t & (NS - 1);
        a.w1 = tw_ld<N, P>(tw, jm, 0);
        a.w4 = tw_ld<N, P>(tw, jm, 3 * NS);
    }
}

template <int N, int P, bool TAB>
__device__ __forceinline__ void tw_form(PassTw<N, P>& pt, const TwAhead<N, P, TAB>& a,
                                        const float2* __restrict__ tw, int t)
{
    if constexpr (TwAhead<N, P, TAB>::ON) {
        pt.w[0] = a.w1;
        pt.w[3] = a.w4;
        tw_products16(pt.w);
    } else {
        load_tw<N, P, TAB>(pt, tw, t);
    }
}

// AHEAD: a radix-16 pass's table reads are issued one pass early.
template <int N, bool INV, int P, bool AHEAD, bool TAB, bool SPLIT, class F>
__device__ __forceinline__ void fft_from(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last,
                                         const TwAhead<N, P, TAB>& ahead)
{
    if constexpr (P < LineGeom<N>::NP) {
        if constexpr (P == LineGeom<N>::NP - 1) before_last();
        PassTw<N, P> cur;
        TwAhead<N, P + 1, TAB> next;
        if constexpr (AHEAD) {
            tw_form<N, P, TAB>(cur, ahead, tw, t);
            tw_issue<N, P + 1, TAB>(next, tw, t);
        } else {
            load_tw<N, P, TAB>(cur, tw, t);
        }
        tw_butterflies<N, P, INV>(x, cur);
        if constexpr (P < LineGeom<N>::NP - 1) line_exchange<N, P, SPLIT>(x, lds, t);
        fft_from<N, INV, P + 1, AHEAD, TAB, SPLIT>(x, lds, tw, t, before_last, next);
    }
}

template <int N, bool INV, bool TAB = false, bool SPLIT = false, class F = NoOp>
__device__ __forceinline__ void fft_line(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last = F())
{
    TwAhead<N, 0, TAB> first;
    fft_from<N, INV, 0, false, TAB, SPLIT>(x, lds, tw, t, before_last, first);
}

template <int N, bool INV, class F = NoOp>
__device__ __forceinline__ void fft_line_ahead(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                               const float2* __restrict__ tw, int t,
                                               F&& before_last = F())
{
    TwAhead<N, 0, false> first;
    tw_issue<N, 0, false>(first, tw, t);
    fft_from<N, INV, 0, true, false, false>(x, lds, tw, t, before_last, first);
}

}  // namespace tw_first
}  // namespace sar
