// fft_line.hpp -- register/LDS line FFT building blocks for gfx950.
//
// One line of N complex64 points (64 <= N <= 16384, power of two) is held by
// T = N/16 threads, 16 points per thread, in the "strided" register layout:
//
//     thread t, register m  <->  element t + m*T .
//
// The transform is a sequence of self-sorting (Stockham) passes: radix-16
// passes followed by at most one smaller power-of-two pass (N = 16^a * r).
// A pass with radix R and span Ns (product of the earlier radices) computes,
// for every butterfly j in [0, N/R),
//
//     v_i = x[j + i*N/R] * W_{Ns*R}^{(j mod Ns)*i},   i = 0..R-1
//     y[(j/Ns)*Ns*R + (j mod Ns) + k*Ns] = DFT_R(v)_k,
//
// and thread t owns butterflies j = t + q*T (q < 16/R), whose inputs are its
// own registers q + i*(16/R).  Between passes the data go through LDS once
// (scatter write, barrier, strided read).  The last pass writes y in natural
// order straight back to the same registers, so a forward transform ends in
// the layout in which the next step (filter multiply, inverse transform,
// store) starts: FFT -> x H -> IFFT needs no extra exchange.
//
// The inverse transform (INV = true) uses conjugated twiddles and butterflies,
// i.e. computes sum_k X[k] exp(+2 pi i k n / N) without the 1/N, which the
// callers fold into the filter.  This equals the paper's conj(FFT(conj(.)))
// form of the IFFT (Sec. II.C) up to rounding.
#pragma once

#include <hip/hip_runtime.h>

namespace sar {

// Workgroup barrier for LDS exchanges.  The compiler models the barrier and
// its fences as side effects that do not write memory, so LDS reads issued
// before a barrier may be sunk below it into a following branch, where they
// race with other waves' writes of the next exchange.  The empty asm that
// clobbers memory counts as a store and keeps every memory access on its
// side of the barrier.
__device__ __forceinline__ void wg_barrier()
{
    __syncthreads();
    asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------- complex
__device__ __forceinline__ float2 c_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 c_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 c_mul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 c_scale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 c_conj(float2 a) { return make_float2(a.x, -a.y); }

// a * (-j) for the forward transform, a * (+j) for the inverse.
template <bool INV>
__device__ __forceinline__ float2 c_mul_mj(float2 a)
{
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// a * exp(-+ j pi/4) = a * (1 -+ j)/sqrt(2)
template <bool INV>
__device__ __forceinline__ float2 c_mul_w8(float2 a)
{
    constexpr float r = 0.70710678118654752440f;
    return INV ? make_float2(r * (a.x - a.y), r * (a.y + a.x))
               : make_float2(r * (a.x + a.y), r * (a.y - a.x));
}

// ---------------------------------------------------------- butterflies
// A thread's 16 points are transformed as radix-2 levels whose twiddles ride
// inside the fused multiply-adds: (a, b) -> (a + w b, a - w b) takes four FMAs
// for t = a + w b and two for 2 a - t.  A pass of radix R on inputs
// v_i = x_i w^i is the evaluation of sum_i x_i z^i at z = w W_R^k, level by
// level (even and odd powers), so the input twiddles cost nothing of their
// own: 12 FMAs per point and radix-16 pass, where a radix-16 butterfly after
// fifteen twiddle multiplies took 10.5 + 3.8 instructions, and eight distinct
// twiddles per pass instead of fifteen.
template <bool INV>
__device__ __forceinline__ void bfly(float2& a, float2& b, float2 w)
{
    if (INV) w.y = -w.y;
    float2 t, u;
    t.x = fmaf(-w.y, b.y, fmaf(w.x, b.x, a.x));
    t.y = fmaf(w.y, b.x, fmaf(w.x, b.y, a.y));
    u.x = fmaf(2.0f, a.x, -t.x);
    u.y = fmaf(2.0f, a.y, -t.y);
    a = t;
    b = u;
}

// The same with the twiddle -j w (forward; +j conj(w) inverse).
template <bool INV>
__device__ __forceinline__ void bfly_mj(float2& a, float2& b, float2 w)
{
    if (INV) w.y = -w.y;
    float2 t, u;
    if (INV) {                                    // a + j w b
        t.x = fmaf(-w.y, b.x, fmaf(-w.x, b.y, a.x));
        t.y = fmaf(-w.y, b.y, fmaf(w.x, b.x, a.y));
    } else {                                      // a - j w b
        t.x = fmaf(w.y, b.x, fmaf(w.x, b.y, a.x));
        t.y = fmaf(w.y, b.y, fmaf(-w.x, b.x, a.y));
    }
    u.x = fmaf(2.0f, a.x, -t.x);
    u.y = fmaf(2.0f, a.y, -t.y);
    a = t;
    b = u;
}

// Butterfly with the constant twiddle W16^M (M = 0..7): additions only for
// M = 0 and 4, one rotation by 45 degrees for M = 2 and 6.
template <bool INV, int M>
__device__ __forceinline__ void bfly_c(float2& a, float2& b)
{
    constexpr float c1 = 0.92387953251128675613f;   // cos(pi/8)
    constexpr float s1 = 0.38268343236508977173f;   // sin(pi/8)
    constexpr float r2 = 0.70710678118654752440f;
    if constexpr (M == 0 || M == 4) {
        const float2 t = M == 0 ? b : c_mul_mj<INV>(b);
        b = c_sub(a, t);
        a = c_add(a, t);
    } else if constexpr (M == 2 || M == 6) {
        // W8 b = r2 (x + y, y - x) forward, r2 (x - y, y + x) inverse
        float2 t = INV ? make_float2(b.x - b.y, b.y + b.x) : make_float2(b.x + b.y, b.y - b.x);
        if (M == 6) t = c_mul_mj<INV>(t);
        b = make_float2(fmaf(-r2, t.x, a.x), fmaf(-r2, t.y, a.y));
        a = make_float2(fmaf(r2, t.x, a.x), fmaf(r2, t.y, a.y));
    } else if constexpr (M == 1 || M == 3) {
        bfly<INV>(a, b, M == 1 ? make_float2(c1, -s1) : make_float2(s1, -c1));
    } else {
        bfly_mj<INV>(a, b, M == 5 ? make_float2(c1, -s1) : make_float2(s1, -c1));
    }
}

// ------------------------------------------------------------ pass plan
__host__ __device__ constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }

// Points per thread for a line of length N.  16 (radix-16 passes) needs one
// LDS exchange fewer per transform than 8 at N = 4096 and measured faster.
__host__ __device__ constexpr int line_e(int n) { return n > 0 ? 16 : 16; }

template <int N> struct LineGeom {
    static_assert(N >= 64 && N <= 16384 && (N & (N - 1)) == 0, "line length");
    static constexpr int T = N / 16;                       // threads per line
    static constexpr int LOG = ilog2(N);
    static constexpr int NFULL = LOG / 4;                  // radix-16 passes
    static constexpr int REM = 1 << (LOG % 4);             // trailing radix (1 = none)
    static constexpr int NP = NFULL + (REM > 1 ? 1 : 0);   // number of passes
    __host__ __device__ static constexpr int radix(int p) { return p < NFULL ? 16 : REM; }
    __host__ __device__ static constexpr int span(int p)   // Ns of pass p
    {
        return p == 0 ? 1 : span(p - 1) * radix(p - 1);
    }
    // offset of pass p's twiddles in the per-N table (pass 0 has none)
    __host__ __device__ static constexpr int tw_off(int p)
    {
        return p <= 1 ? 0 : tw_off(p - 1) + (radix(p - 1) - 1) * span(p - 1);
    }
    static constexpr int TW_SIZE = tw_off(NP);
    // LDS words (float2) per line, with up to one pad slot per 16 points
    static constexpr int LDS = N + N / 16;
};

// LDS slot of point i in the exchange after pass P: 1 (P = 0) or 2 (later
// passes) pad slots every 32.  LDS serves 8-byte accesses 32 lanes at a time
// from 32 slots' worth of banks.  The reads take 32 consecutive points, which
// no pad splits, so they are free of conflicts; the writes of pass 0 (16
// points apart) need an odd pad, those of pass 1 (two runs of 16 points 256
// apart) an even one.  With one pad every 16 for all passes the reads had a
// two-way conflict (0.5 conflict cycles per active LDS cycle).
template <int P> __host__ __device__ constexpr int lds_pads() { return P == 0 ? 1 : 2; }

template <int P> __device__ __forceinline__ int lds_slot(int i)
{
    return i + lds_pads<P>() * (i >> 5);
}

// lds_slot(t + m * T) for t < T, and lds_slot(base + i * NS) for the outputs of
// radix-16 pass P of span NS (base = 16 t, or 16 NS (t / NS) + t % NS), as one
// address per thread plus a constant, which becomes the instruction's offset:
// the sums carry nothing from their low five bits into the pad term.
template <int T, int P> __device__ __forceinline__ int lds_in(int t, int m)
{
    if constexpr (T >= 32) return lds_slot<P>(t) + m * (T + lds_pads<P>() * (T / 32));
    else return t + (m * T + lds_pads<P>() * (m * T / 32));
}
template <int NS, int P> __device__ __forceinline__ int lds_out(int base, int i)
{
    return lds_slot<P>(base) + i * NS + lds_pads<P>() * (i * NS / 32);
}

// The twiddles of one thread in one pass.  The thread's 16 / R butterflies of
// a radix-R pass (q = 0 .. 16/R - 1, j = t + q T) and their levels need
// w^e W16^(e r), e a power of two below R, r < 8 / e; with -j factored out
// (r >= 4 / e) eight values remain: w W16^r, w^2 W8^r, w^4, w^8, where w is
// the twiddle of butterfly q = 0 (in a trailing pass the span is N / R, so
// butterfly q's is w W16^q).
struct TwSet {
    float2 r[4];         // w, w W16, w W16^2, w W16^3
    float2 s[2];         // w^2, w^2 W8
    float2 w4, w8;
};

__device__ __forceinline__ float2 c_sqr(float2 a)
{
    return make_float2(fmaf(a.x, a.x, -a.y * a.y), 2.0f * a.x * a.y);
}

// The constant multiples of w and w^2 (set r[0], s[0] first).
template <int R>
__device__ __forceinline__ void tw_rotate(TwSet& p)
{
    constexpr float c1 = 0.92387953251128675613f;
    constexpr float s1 = 0.38268343236508977173f;
    const float2 w = p.r[0];
    p.r[1] = c_mul(w, make_float2(c1, -s1));
    p.r[2] = c_mul_w8<false>(w);
    p.r[3] = c_mul(w, make_float2(s1, -c1));
    if constexpr (R >= 4) p.s[1] = c_mul_w8<false>(p.s[0]);
}

// Twiddle table reads of pass P of virtual thread t (one of N / 16): w, and
// for radix 8 and 16 w^4 (TWP: the other powers are squares of these two) or
// w^2, w^4 and w^8 as well (!TWP: table reads instead of squares).  Row i - 1
// of the pass's table holds w^i.
template <int N, int P, bool TWP> struct TwReads {
    using G = LineGeom<N>;
    static constexpr bool ANY = P < G::NP && G::span(P) > 1;
    static constexpr int R = ANY ? G::radix(P) : 1;
    float2 w1, w2, w4, w8;
};

template <int N, int P, bool TWP>
__device__ __forceinline__ void tw_issue(TwReads<N, P, TWP>& a, const float2* __restrict__ tw, int t)
{
    using Rd = TwReads<N, P, TWP>;
    if constexpr (Rd::ANY) {
        using G = LineGeom<N>;
        constexpr int NS = G::span(P), OFF = G::tw_off(P), R = Rd::R;
        const int jm = t & (NS - 1);
        a.w1 = tw[OFF + jm];
        if constexpr (R >= 8) a.w4 = tw[OFF + 3 * NS + jm];
        if constexpr (!TWP && R >= 4) a.w2 = tw[OFF + NS + jm];
        if constexpr (!TWP && R >= 16) a.w8 = tw[OFF + 7 * NS + jm];
    }
}

template <int N, int P, bool TWP>
__device__ __forceinline__ void tw_form(TwSet& p, const TwReads<N, P, TWP>& a)
{
    using Rd = TwReads<N, P, TWP>;
    if constexpr (Rd::ANY) {
        constexpr int R = Rd::R;
        p.r[0] = a.w1;
        if constexpr (R >= 4) p.s[0] = TWP ? c_sqr(a.w1) : a.w2;
        if constexpr (R >= 8) p.w4 = a.w4;
        if constexpr (R >= 16) p.w8 = TWP ? c_sqr(a.w4) : a.w8;
        tw_rotate<R>(p);
    }
}

// Level E (inputs E apart within a butterfly) of a thread's 16 / R butterflies
// of radix R: point i of butterfly q, partial output k, sits at
// q + (16 / R) (i + 2 E k) before and q + (16 / R) (i + E k) after.
template <int R, int E, bool INV, bool TW>
__device__ __forceinline__ void fft_level(float2 (&v)[16], const TwSet& p)
{
    constexpr int B = 16 / R, K = R / (2 * E);
    float2 o[16];
#pragma unroll
    for (int q = 0; q < B; ++q)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            constexpr int J = 4 / E > 0 ? 4 / E : 1;      // r >= J carries the factor -j
            const int r = q + k * B;
#pragma unroll
            for (int i = 0; i < E; ++i) {
                float2 a = v[q + B * (i + 2 * E * k)], b = v[q + B * (i + E + 2 * E * k)];
                if constexpr (TW) {
                    const float2 w = E == 8 ? p.w8 : E == 4 ? p.w4 : E == 2 ? p.s[r & 1] : p.r[r & 3];
                    if (E < 8 && r >= J) bfly_mj<INV>(a, b, w);
                    else bfly<INV>(a, b, w);
                } else {
                    switch (E * r) {
                    case 0: bfly_c<INV, 0>(a, b); break;
                    case 1: bfly_c<INV, 1>(a, b); break;
                    case 2: bfly_c<INV, 2>(a, b); break;
                    case 3: bfly_c<INV, 3>(a, b); break;
                    case 4: bfly_c<INV, 4>(a, b); break;
                    case 5: bfly_c<INV, 5>(a, b); break;
                    case 6: bfly_c<INV, 6>(a, b); break;
                    default: bfly_c<INV, 7>(a, b); break;
                    }
                }
                o[q + B * (i + E * k)] = a;
                o[q + B * (i + E * (k + K))] = b;
            }
        }
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = o[i];
}

// All butterflies of pass P of one virtual thread, in registers.
template <int N, int P, bool INV>
__device__ __forceinline__ void pass_butterflies(float2 (&x)[16], const TwSet& p)
{
    using G = LineGeom<N>;
    constexpr int R = G::radix(P);
    constexpr bool TW = G::span(P) > 1;
    if constexpr (R >= 16) fft_level<R, 8, INV, TW>(x, p);
    if constexpr (R >= 8) fft_level<R, 4, INV, TW>(x, p);
    if constexpr (R >= 4) fft_level<R, 2, INV, TW>(x, p);
    fft_level<R, 1, INV, TW>(x, p);
}

// One Stockham pass P of an N-point line (see the header comment), with its
// twiddles already formed.
// SPLIT: the exchange keeps real and imaginary parts in two float arrays of
// the line's LDS (re[0, LDS), im[LDS, 2 LDS)), two 4-byte accesses per point
// instead of one 8-byte access, so that the two layouts can be compared.
template <int N, int P, bool INV, bool SPLIT = false>
__device__ __forceinline__ void fft_pass(float2 (&x)[16], float2* __restrict__ lds,
                                         const TwSet& p, int t)
{
    using G = LineGeom<N>;
    constexpr int R = G::radix(P);
    constexpr int NS = G::span(P);
    constexpr int B = 16 / R;
    pass_butterflies<N, P, INV>(x, p);
    if constexpr (P < G::NP - 1) {
        static_assert(B == 1, "only the last pass is smaller than radix 16");
        const int base = (t / NS) * NS * R + (t & (NS - 1));
        if constexpr (SPLIT) {
            float* re = (float*)lds;
            float* im = re + G::LDS;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                re[lds_out<NS, P>(base, i)] = x[i].x;
                im[lds_out<NS, P>(base, i)] = x[i].y;
            }
            wg_barrier();
#pragma unroll
            for (int m = 0; m < 16; ++m)
                x[m] = make_float2(re[lds_in<G::T, P>(t, m)], im[lds_in<G::T, P>(t, m)]);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) lds[lds_out<NS, P>(base, i)] = x[i];
            wg_barrier();
#pragma unroll
            for (int m = 0; m < 16; ++m) x[m] = lds[lds_in<G::T, P>(t, m)];
        }
        wg_barrier();
    }
}

// Passes P.. of the line.  `before_last` runs just before the last pass
// (callers use it to request data needed right after the transform, e.g.
// the matched filter, so that its latency overlaps the last pass).
struct NoOp {
    __device__ __forceinline__ void operator()() const {}
};

// AHEAD: a pass's table reads are issued one pass early, so they are in
// flight during the previous pass and its exchange (and, for the last pass,
// ahead of the `before_last` loads), at the cost of a few registers across
// the previous pass.
// FRESH: bit P set = pass P's twiddles are read and formed anew even where an
// earlier transform of the same thread has them (its index is hidden from the
// compiler); a bit left clear lets the compiler keep them in registers.
template <int N, bool INV, bool TWP, int P, bool SPLIT, bool AHEAD, int FRESH, class F>
__device__ __forceinline__ void fft_from(float2 (&x)[16], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last,
                                         const TwReads<N, P, TWP>& ahead)
{
    if constexpr (P < LineGeom<N>::NP) {
        if constexpr (P == LineGeom<N>::NP - 1) before_last();
        TwSet cur;
        TwReads<N, P + 1, TWP> next;
        int ti = t;
        constexpr int READ = AHEAD ? P + 1 : P;           // the pass whose reads are issued here
        if constexpr ((FRESH >> READ) & 1) asm volatile("" : "+v"(ti));
        if constexpr (AHEAD) {
            tw_form<N, P, TWP>(cur, ahead);
            tw_issue<N, P + 1, TWP>(next, tw, ti);
        } else {
            TwReads<N, P, TWP> now;
            tw_issue<N, P, TWP>(now, tw, ti);
            tw_form<N, P, TWP>(cur, now);
        }
        fft_pass<N, P, INV, SPLIT>(x, lds, cur, t);
        fft_from<N, INV, TWP, P + 1, SPLIT, AHEAD, FRESH>(x, lds, tw, t, before_last, next);
    }
}

// TWP selects twiddles by products (fewer loads, more VALU) or table reads;
// SPLIT the split real/imaginary exchange layout (see fft_pass).
template <int N, bool INV, bool TWP = true, bool SPLIT = false, int FRESH = 0, class F = NoOp>
__device__ __forceinline__ void fft_line(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last = F())
{
    TwReads<N, 0, TWP> first;
    fft_from<N, INV, TWP, 0, SPLIT, false, FRESH>(x, lds, tw, t, before_last, first);
}

// The same transform with every pass's table reads issued one pass ahead.
template <int N, bool INV, bool TWP = true, bool SPLIT = false, int FRESH = 0, class F = NoOp>
__device__ __forceinline__ void fft_line_ahead(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                               const float2* __restrict__ tw, int t,
                                               F&& before_last = F())
{
    TwReads<N, 0, TWP> first;
    fft_from<N, INV, TWP, 0, SPLIT, true, FRESH>(x, lds, tw, t, before_last, first);
}

// The value is in its registers here: a pending load has been waited for, and
// what is computed from it later is not moved ahead of this point (out of a
// loop over lines, where it would stay in registers).
__device__ __forceinline__ void pin(float2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

__device__ __forceinline__ void pin_line(float2 (&x)[16])
{
#pragma unroll
    for (int m = 0; m < 16; ++m) pin(x[m]);
}

__device__ __forceinline__ void copy_line(float2 (&to)[16], const float2 (&from)[16])
{
#pragma unroll
    for (int m = 0; m < 16; ++m) to[m] = from[m];
}

// The same value under a new name: addresses formed from it are formed where
// they are used instead of staying in registers through a loop.
__device__ __forceinline__ int fresh(int t)
{
    asm volatile("" : "+v"(t));
    return t;
}

// The twiddle reads of every pass (at most five values), held in registers by a
// thread that transforms line after line: the transforms between then read
// nothing from memory, so no wait of theirs covers loads of the next line.
template <int N> struct TwAll {
    TwReads<N, 1, true> p1;
    TwReads<N, 2, true> p2;
    TwReads<N, 3, true> p3;
    __device__ __forceinline__ void read(const float2* __restrict__ tw, int t)
    {
        tw_issue<N, 1, true>(p1, tw, t);
        tw_issue<N, 2, true>(p2, tw, t);
        tw_issue<N, 3, true>(p3, tw, t);
    }
    template <int P> static __device__ __forceinline__ void pin_pass(TwReads<N, P, true>& r)
    {
        if constexpr (TwReads<N, P, true>::ANY) {
            pin(r.w1);
            if constexpr (TwReads<N, P, true>::R >= 8) pin(r.w4);
        }
    }
    __device__ __forceinline__ void hold()
    {
        pin_pass<1>(p1);
        pin_pass<2>(p2);
        pin_pass<3>(p3);
    }
};

template <int N, bool INV, int P, class F>
__device__ __forceinline__ void fft_held_from(float2 (&x)[16], float2* __restrict__ lds,
                                              const TwAll<N>& tw, int t, F&& before_last)
{
    if constexpr (P < LineGeom<N>::NP) {
        // ahead of the last radix-16 pass (its butterflies and exchange cover
        // the latency of the loads; a trailing smaller pass is too short)
        if constexpr (P == LineGeom<N>::NFULL - 1) before_last();
        TwSet cur;
        if constexpr (P == 1) tw_form<N, 1, true>(cur, tw.p1);
        if constexpr (P == 2) tw_form<N, 2, true>(cur, tw.p2);
        if constexpr (P == 3) tw_form<N, 3, true>(cur, tw.p3);
        fft_pass<N, P, INV>(x, lds, cur, t);
        fft_held_from<N, INV, P + 1>(x, lds, tw, t, before_last);
    }
}

// fft_line with held twiddle reads.
// (before_last runs before the last radix-16 pass)
template <int N, bool INV, class F = NoOp>
__device__ __forceinline__ void fft_line_held(float2 (&x)[16], float2* __restrict__ lds,
                                              const TwAll<N>& tw, int t, F&& before_last = F())
{
    fft_held_from<N, INV, 0>(x, lds, tw, t, before_last);
}

// ---------------------------------------------------- half-LDS exchange
// The same transform with half the LDS: the real parts of a line go through N
// floats first, then the imaginary parts through the same floats.  It costs
// four barriers per exchange instead of two and buys twice the lines per CU
// (with 64 registers per thread, 32 waves): for the column strips, whose loads
// wait long, that is worth more.
//
// Slot of point i after pass P: 4-byte accesses are served 64 lanes at a time
// from 64 banks; pass 0's writes are 16 points apart (an odd pad every 64
// points keeps them apart), pass 1's are runs of 16 points 256 apart (a pad of
// 4 every 64).
template <int P> __host__ __device__ constexpr int half_pads() { return P == 0 ? 1 : 4; }

template <int P> __device__ __forceinline__ int half_slot(int i)
{
    return i + half_pads<P>() * (i >> 6);
}
// half_slot(t + m * T), t < T, and half_slot(base + i * NS), as in lds_in / lds_out.
template <int T, int P> __device__ __forceinline__ int half_in(int t, int m)
{
    if constexpr (T >= 64) return half_slot<P>(t) + m * (T + half_pads<P>() * (T / 64));
    else return t + (m * T + half_pads<P>() * (m * T / 64));
}
template <int NS, int P> __device__ __forceinline__ int half_out(int base, int i)
{
    return half_slot<P>(base) + i * NS + half_pads<P>() * (i * NS / 64);
}

template <int N, int P>
__device__ __forceinline__ void half_exchange(float2 (&x)[16], float* __restrict__ lds, int t)
{
    constexpr int NS = LineGeom<N>::span(P), T = LineGeom<N>::T;
    const int base = (t / NS) * NS * 16 + (t & (NS - 1));
#pragma unroll
    for (int i = 0; i < 16; ++i) lds[half_out<NS, P>(base, i)] = x[i].x;
    wg_barrier();
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m].x = lds[half_in<T, P>(t, m)];
    wg_barrier();
#pragma unroll
    for (int i = 0; i < 16; ++i) lds[half_out<NS, P>(base, i)] = x[i].y;
    wg_barrier();
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m].y = lds[half_in<T, P>(t, m)];
    wg_barrier();
}

template <int N, bool INV, int P>
__device__ __forceinline__ void fft_half_from(float2 (&x)[16], float* __restrict__ lds,
                                              const float2* __restrict__ tw, int t)
{
    if constexpr (P < LineGeom<N>::NP) {
        TwReads<N, P, true> now;
        tw_issue<N, P, true>(now, tw, fresh(t));
        TwSet cur;
        tw_form<N, P, true>(cur, now);
        pass_butterflies<N, P, INV>(x, cur);
        if constexpr (P < LineGeom<N>::NP - 1) half_exchange<N, P>(x, lds, t);
        fft_half_from<N, INV, P + 1>(x, lds, tw, t);
    }
}

template <int N, bool INV>
__device__ __forceinline__ void fft_line_half(float2 (&x)[16], float* __restrict__ lds,
                                              const float2* __restrict__ tw, int t)
{
    fft_half_from<N, INV, 0>(x, lds, tw, t);
}

}  // namespace sar
