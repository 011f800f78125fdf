// fft_line_tw.hpp -- the line transform with twiddles applied ahead of each
// butterfly, for data that are about to be stored as FP16.
//
// The transform of fft_line.hpp has its twiddles inside the butterflies' FMAs
// and rounds differently in the last FP32 bits.  Where the result is rounded to
// FP16 next (half storage: the range output and the range-Doppler rows) such a
// last-bit change moves a few values by a whole FP16 step (2^-11 relative;
// 2.3e-5 relative L2 of a 4096^2 image, against 2.5e-4 from the FP16 rounding
// itself), so those two passes keep this form, whose stored bits callers have.
// So does the trailing pass of the split-BF16 lines (see mfma_fft.hpp).
// They are bound by memory, not by the instruction count (range pass of
// 4096^2: 66 us against 54 us for a plain copy of its FP32 input and output).
#pragma once

#include "fft_line.hpp"

namespace sar {
namespace tw_first {

// a * exp(-+ j 3pi/4) = a * (-1 -+ j)/sqrt(2)
template <bool INV>
__device__ __forceinline__ float2 c_mul_w8_3(float2 a)
{
    constexpr float r = 0.70710678118654752440f;
    return INV ? make_float2(-r * (a.x + a.y), r * (a.x - a.y))
               : make_float2(r * (a.y - a.x), -r * (a.x + a.y));
}

// a * (c, -+ s)
template <bool INV>
__device__ __forceinline__ float2 c_mul_cs(float2 a, float c, float s)
{
    return c_mul(a, make_float2(c, INV ? s : -s));
}

// ---------------------------------------------------------- small DFTs
// All take natural-order input in v[] and leave natural-order output.
template <bool INV>
__device__ __forceinline__ void dft2(float2& a, float2& b)
{
    float2 t = a;
    a = c_add(t, b);
    b = c_sub(t, b);
}

template <bool INV>
__device__ __forceinline__ void dft4(float2& a0, float2& a1, float2& a2, float2& a3)
{
    float2 s0 = c_add(a0, a2), d0 = c_sub(a0, a2);
    float2 s1 = c_add(a1, a3), d1 = c_mul_mj<INV>(c_sub(a1, a3));
    a0 = c_add(s0, s1);
    a2 = c_sub(s0, s1);
    a1 = c_add(d0, d1);
    a3 = c_sub(d0, d1);
}

template <int R, bool INV> struct Dft;

template <bool INV> struct Dft<2, INV> {
    __device__ __forceinline__ static void run(float2* v) { dft2<INV>(v[0], v[1]); }
};

template <bool INV> struct Dft<4, INV> {
    __device__ __forceinline__ static void run(float2* v) { dft4<INV>(v[0], v[1], v[2], v[3]); }
};

// DFT8 = DFT2 (stride 4) x twiddle W8^{n2 k1} x DFT4.
template <bool INV> struct Dft<8, INV> {
    __device__ __forceinline__ static void run(float2* v)
    {
        dft2<INV>(v[0], v[4]);
        dft2<INV>(v[1], v[5]);
        dft2<INV>(v[2], v[6]);
        dft2<INV>(v[3], v[7]);
        v[5] = c_mul_w8<INV>(v[5]);
        v[6] = c_mul_mj<INV>(v[6]);
        v[7] = c_mul_w8_3<INV>(v[7]);
        // y[n2][k1] sits in v[n2 + 4 k1]; DFT4 over n2 gives X[k1 + 2 k2]
        float2 a0 = v[0], a1 = v[1], a2 = v[2], a3 = v[3];
        float2 b0 = v[4], b1 = v[5], b2 = v[6], b3 = v[7];
        dft4<INV>(a0, a1, a2, a3);
        dft4<INV>(b0, b1, b2, b3);
        v[0] = a0; v[2] = a1; v[4] = a2; v[6] = a3;
        v[1] = b0; v[3] = b1; v[5] = b2; v[7] = b3;
    }
};

// DFT16 = DFT4 (stride 4) x twiddle W16^{n2 k1} x DFT4.
template <bool INV> struct Dft<16, INV> {
    __device__ __forceinline__ static void run(float2* v)
    {
        constexpr float c1 = 0.92387953251128675613f;   // cos(pi/8)
        constexpr float s1 = 0.38268343236508977173f;   // sin(pi/8)
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) dft4<INV>(v[n2], v[n2 + 4], v[n2 + 8], v[n2 + 12]);
        // y[n2][k1] is in v[n2 + 4 k1]
        v[5] = c_mul_cs<INV>(v[5], c1, s1);     // n2=1 k1=1: W16^1
        v[9] = c_mul_w8<INV>(v[9]);             // n2=1 k1=2: W16^2
        v[13] = c_mul_cs<INV>(v[13], s1, c1);   // n2=1 k1=3: W16^3
        v[6] = c_mul_w8<INV>(v[6]);             // n2=2 k1=1: W16^2
        v[10] = c_mul_mj<INV>(v[10]);           // n2=2 k1=2: W16^4
        v[14] = c_mul_w8_3<INV>(v[14]);         // n2=2 k1=3: W16^6
        v[7] = c_mul_cs<INV>(v[7], s1, c1);     // n2=3 k1=1: W16^3
        v[11] = c_mul_w8_3<INV>(v[11]);         // n2=3 k1=2: W16^6
        v[15] = c_mul_cs<INV>(v[15], -c1, -s1); // n2=3 k1=3: W16^9 = (-c1, +s1)
        float2 o[16];
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            float2 a0 = v[4 * k1], a1 = v[4 * k1 + 1], a2 = v[4 * k1 + 2], a3 = v[4 * k1 + 3];
            dft4<INV>(a0, a1, a2, a3);
            o[k1] = a0; o[k1 + 4] = a1; o[k1 + 8] = a2; o[k1 + 12] = a3;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = o[i];
    }
};

// Twiddles a thread needs in pass P: for butterfly q (j = t + q*T) and
// i = 1..R-1, exp(-2 pi i * (j mod Ns) * i / (Ns * R)), read from this N's
// table (entry tw_off(P) + (i-1)*Ns + (j mod Ns)); passes with Ns == 1 need
// none.
template <int N, int P> struct PassTw {
    using G = LineGeom<N>;
    static constexpr bool ANY = P < G::NP && G::span(P) > 1;
    static constexpr int COUNT = ANY ? (line_e(N) / G::radix(P)) * (G::radix(P) - 1) : 1;
    float2 w[COUNT];
};

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

template <int N, int P>
__device__ __forceinline__ void load_tw(PassTw<N, P>& pt, const float2* __restrict__ tw, int t)
{
    using G = LineGeom<N>;
    if constexpr (PassTw<N, P>::ANY && G::radix(P) == 16) {
        constexpr int NS = G::span(P), B = line_e(N) / 16, OFF = G::tw_off(P);
#pragma unroll
        for (int q = 0; q < B; ++q) {
            const int jm = (t + q * G::T) & (NS - 1);
            float2* w = pt.w + q * 15;
            w[0] = tw[OFF + jm];
            w[3] = tw[OFF + 3 * NS + jm];
            tw_products16(w);
        }
    } else if constexpr (PassTw<N, P>::ANY) {
        constexpr int R = G::radix(P), NS = G::span(P), B = line_e(N) / R, OFF = G::tw_off(P);
#pragma unroll
        for (int q = 0; q < B; ++q) {
            const int jm = (t + q * G::T) & (NS - 1);
#pragma unroll
            for (int i = 1; i < R; ++i) pt.w[q * (R - 1) + i - 1] = tw[OFF + (i - 1) * NS + jm];
        }
    }
}

// The table reads of a radix-16 pass (W^1, W^4 per butterfly), issued
// one pass ahead so that their latency overlaps the previous pass and its
// LDS exchange; other passes read their twiddles when they start.
template <int N, int P> struct TwAhead {
    static constexpr bool ON = PassTw<N, P>::ANY && LineGeom<N>::radix(P) == 16;
    static constexpr int B = ON ? line_e(N) / 16 : 1;
    float2 w1[B], w4[B];
};

template <int N, int P>
__device__ __forceinline__ void tw_issue(TwAhead<N, P>& a, const float2* __restrict__ tw, int t)
{
    if constexpr (TwAhead<N, P>::ON) {
        using G = LineGeom<N>;
        constexpr int NS = G::span(P), OFF = G::tw_off(P);
#pragma unroll
        for (int q = 0; q < TwAhead<N, P>::B; ++q) {
            const int jm = (t + q * G::T) & (NS - 1);
            a.w1[q] = tw[OFF + jm];
            a.w4[q] = tw[OFF + 3 * NS + jm];
        }
    }
}

template <int N, int P>
__device__ __forceinline__ void tw_form(PassTw<N, P>& pt, const TwAhead<N, P>& a,
                                        const float2* __restrict__ tw, int t)
{
    if constexpr (TwAhead<N, P>::ON) {
#pragma unroll
        for (int q = 0; q < TwAhead<N, P>::B; ++q) {
            float2* w = pt.w + q * 15;
            w[0] = a.w1[q];
            w[3] = a.w4[q];
            tw_products16(w);
        }
    } else {
        load_tw<N, P>(pt, tw, t);
    }
}

// One Stockham pass P of an N-point line (see the header comment), with its
// twiddles already loaded.
template <int N, int P, bool INV>
__device__ __forceinline__ void fft_pass(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const PassTw<N, P>& pt, int t)
{
    using G = LineGeom<N>;
    constexpr int E = line_e(N);
    constexpr int R = G::radix(P);
    constexpr int NS = G::span(P);
    constexpr int B = E / R;
    constexpr bool LAST = (P == G::NP - 1);
#pragma unroll
    for (int q = 0; q < B; ++q) {
        float2 v[R];
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = x[q + i * B];
        const int j = t + q * G::T;
        const int jm = j & (NS - 1);
        if constexpr (NS > 1) {
#pragma unroll
            for (int i = 1; i < R; ++i) {
                float2 w = pt.w[q * (R - 1) + i - 1];
                if (INV) w.y = -w.y;
                v[i] = c_mul(v[i], w);
            }
        }
        Dft<R, INV>::run(v);
        if constexpr (LAST) {
#pragma unroll
            for (int i = 0; i < R; ++i) x[q + i * B] = v[i];
        } else {
            const int base = (j / NS) * NS * R + jm;
#pragma unroll
            for (int i = 0; i < R; ++i) lds[lds_out<NS, P>(base, i)] = v[i];
        }
    }
    if constexpr (!LAST) {
        wg_barrier();
#pragma unroll
        for (int m = 0; m < E; ++m) x[m] = lds[lds_in<G::T, P>(t, m)];
        wg_barrier();
    }
}

// AHEAD: a radix-16 pass's table reads are issued one pass early.
template <int N, bool INV, int P, bool AHEAD, class F>
__device__ __forceinline__ void fft_from(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last,
                                         const TwAhead<N, P>& ahead)
{
    if constexpr (P < LineGeom<N>::NP) {
        if constexpr (P == LineGeom<N>::NP - 1) before_last();
        PassTw<N, P> cur;
        TwAhead<N, P + 1> next;
        if constexpr (AHEAD) {
            tw_form<N, P>(cur, ahead, tw, t);
            tw_issue<N, P + 1>(next, tw, t);
        } else {
            load_tw<N, P>(cur, tw, t);
        }
        fft_pass<N, P, INV>(x, lds, cur, t);
        fft_from<N, INV, P + 1, AHEAD>(x, lds, tw, t, before_last, next);
    }
}

template <int N, bool INV, class F = NoOp>
__device__ __forceinline__ void fft_line(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last = F())
{
    TwAhead<N, 0> first;
    fft_from<N, INV, 0, false>(x, lds, tw, t, before_last, first);
}

template <int N, bool INV, class F = NoOp>
__device__ __forceinline__ void fft_line_ahead(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                               const float2* __restrict__ tw, int t,
                                               F&& before_last = F())
{
    TwAhead<N, 0> first;
    tw_issue<N, 0>(first, tw, t);
    fft_from<N, INV, 0, true>(x, lds, tw, t, before_last, first);
}

}  // namespace tw_first
}  // namespace sar
