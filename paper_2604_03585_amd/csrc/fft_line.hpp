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

#include <cstdint>

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

// Buffer resource over `bytes` bytes (less than 4 GiB) from a wave-uniform base:
// reads beyond its end return zero and writes there are dropped.  A buffer
// access takes a vector offset plus a scalar one, so the 16 accesses of a line
// share one address register instead of 16 64-bit sums.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
}
__device__ __forceinline__ float2 buf_ld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

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

// ------------------------------------------------------ FMA butterflies
// Radix-2 levels whose twiddles ride inside the fused multiply-adds: (a, b) ->
// (a + w b, a - w b) takes four FMAs for t = a + w b and two for 2 a - t.  A pass
// of radix R on inputs v_i = x_i w^i is the evaluation of sum_i x_i z^i at
// z = w W_R^k, level by level (even and odd powers), so the input twiddles cost
// nothing of their own: 12 FMAs per point and radix-16 pass, where a radix-16
// butterfly after fifteen twiddle multiplies takes 10.5 + 3.8 instructions and
// 3.3 more to form the twiddles from two table reads.
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

// LDS slot of point i in the exchange after pass P: 1 (P = 0) or 2 (later passes)
// pad slots every 32.  LDS serves 8-byte reads 32 lanes and 8-byte writes 16 lanes at
// a time (2 and 4 cycles per wave and instruction, SQ_LDS_IDX_ACTIVE of each pattern
// alone), so 32 lanes of a read must differ in the slot's low five bits and 16 lanes
// of a write in its low four.  The reads take 32 consecutive points, which no pad
// splits, and are free of conflicts; so are the writes of pass 1 (runs of 16 points
// 256 apart).  The writes of pass 0 (16 points apart) have a two-way conflict and
// take 8 cycles; a pad every 16 would move it to the reads (4 + 4 cycles).
template <int P> __host__ __device__ constexpr int lds_pads() { return P == 0 ? 1 : 2; }

template <int P>
__host__ __device__ constexpr int lds_slot(int i)
{
    return i + lds_pads<P>() * (i >> 5);
}

// lds_slot(t + m * T) for t < T, and lds_slot(base + i * NS) for the outputs of
// radix-16 pass P of span NS (base = 16 t, or 16 NS (t / NS) + t % NS), as one
// address per thread plus a constant, which becomes the instruction's offset:
// the sums carry nothing from their low five bits into the pad term.
template <int T, int P>
__host__ __device__ constexpr int lds_in(int t, int m)
{
    if constexpr (T >= 32) return lds_slot<P>(t) + m * (T + lds_pads<P>() * (T / 32));
    else return t + (m * T + lds_pads<P>() * (m * T / 32));
}
template <int NS, int P>
__host__ __device__ constexpr int lds_out(int base, int i)
{
    return lds_slot<P>(base) + i * NS + lds_pads<P>() * (i * NS / 32);
}

// ------------------------------------------------------------- twiddles
// Where a pass's twiddles enter, chosen so that no transform is further from its
// value in 64 bits than with twiddles ahead of every butterfly and the powers of
// radix-16 passes as products of two table entries (tw_first).  Relative L2 of
// Gaussian noise, 1e-7, here (there): 64 points 0.80 (0.81), 256 1.12 (1.15), 512
// 1.18 (1.21), 1024 1.23 (1.26), 2048 1.29 (1.32), 4096 1.46 (1.53), 8192 1.52
// (1.58), 16384 1.57 (1.62).
//   NONE  pass 0 has none; its butterflies are plain DFTs (the FMA butterflies'
//         u = 2a - t carries t's rounding: 0.82 at 64 points);
//   FMA   radix-16 passes: inside the butterflies, w, w^2, w^4 and w^8 read from
//         the table (with w^2 and w^8 as squares 4096 points have 1.61, with one
//         of them 1.55 and 1.53);
//   PRE   trailing passes of up to 4096 points: every twiddle from the table,
//         ahead of the butterfly (ROT there: 1.26 at 1024 points, 1.33 at 2048);
//   ROT   those of longer lines: inside the butterflies, butterfly q's w W16^q
//         from the table too (as products 1.66 at 16384 points; PRE's twelve
//         twiddles would spill in the persistent kernel).
// Against squares and products in every pass (0.99 at 64 points, 1.46 at 1024, 1.62
// at 4096) this costs two reads more per radix-16 pass and up to thirteen in a
// trailing one: 3001 lines of 1024 points 9.6 -> 10.0 us, 1024 x 2048 azimuth step
// 19.9 -> 20.6, 4096 x 4096 hyperbolic scene 180.7 -> 182.3.
enum PassForm { PASS_NONE, PASS_FMA, PASS_PRE, PASS_ROT };
template <int N, int P> __host__ __device__ constexpr PassForm pass_form()
{
    if (P >= LineGeom<N>::NP || LineGeom<N>::span(P) == 1) return PASS_NONE;
    if (LineGeom<N>::radix(P) == 16) return PASS_FMA;
    return N <= 4096 ? PASS_PRE : PASS_ROT;
}

// Twiddles ahead of the butterflies of pass P: for butterfly q (j = t + q*T) and
// i = 1..R-1, exp(-2 pi i * (j mod Ns) * i / (Ns * R)), read from this N's
// table (entry tw_off(P) + (i-1)*Ns + (j mod Ns)); passes with Ns == 1 need
// none.
template <int N, int P> struct PassTw {
    using G = LineGeom<N>;
    static constexpr bool ANY = P < G::NP && G::span(P) > 1;
    static constexpr int PER = ANY ? G::radix(P) - 1 : 0;      // per butterfly
    static constexpr int COUNT = ANY ? line_e(N) / G::radix(P) * PER : 1;
    float2 w[COUNT];
};

// Entry jm + k (k a constant) of pass P's part of the table.
template <int N, int P>
__device__ __forceinline__ float2 tw_ld(const float2* __restrict__ tw, int jm, int k)
{
    constexpr int OFF = LineGeom<N>::tw_off(P);
    return buf_ld(buf_rsrc(tw, LineGeom<N>::TW_SIZE * 8u), (uint32_t)jm * 8u, (uint32_t)(OFF + k) * 8u);
}

// The twiddles of butterfly q.
template <int N, int P>
__device__ __forceinline__ void read_tw(PassTw<N, P>& pt, const float2* __restrict__ tw, int t, int q)
{
    using G = LineGeom<N>;
    constexpr int R = G::radix(P), NS = G::span(P), PER = PassTw<N, P>::PER;
    // radix 16: one butterfly, one of NS twiddle sets; trailing passes: j = t + q T < NS
    const int jm = R == 16 ? t & (NS - 1) : t, at = R == 16 ? 0 : q * G::T;
#pragma unroll
    for (int i = 0; i < PER; ++i) pt.w[q * PER + i] = tw_ld<N, P>(tw, jm, at + i * NS);
}

template <int N, int P>
__device__ __forceinline__ void read_tw(PassTw<N, P>& pt, const float2* __restrict__ tw, int t)
{
    if constexpr (PassTw<N, P>::ANY) {
#pragma unroll
        for (int q = 0; q < 16 / LineGeom<N>::radix(P); ++q) read_tw<N, P>(pt, tw, t, q);
    }
}

// Butterfly q of pass P with its twiddles (if any) ahead of it.
template <int N, int P, bool INV>
__device__ __forceinline__ void tw_butterfly(float2 (&x)[16], const PassTw<N, P>& pt, int q)
{
    constexpr int R = LineGeom<N>::radix(P), B = 16 / R;
    float2 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = x[q + i * B];
    if constexpr (PassTw<N, P>::ANY) {
#pragma unroll
        for (int i = 1; i < R; ++i) {
            float2 w = pt.w[q * (R - 1) + i - 1];
            if (INV) w.y = -w.y;
            v[i] = c_mul(v[i], w);
        }
    }
    Dft<R, INV>::run(v);
#pragma unroll
    for (int i = 0; i < R; ++i) x[q + i * B] = v[i];
}

template <int N, int P, bool INV>
__device__ __forceinline__ void tw_butterflies(float2 (&x)[16], const PassTw<N, P>& pt)
{
#pragma unroll
    for (int q = 0; q < 16 / LineGeom<N>::radix(P); ++q) tw_butterfly<N, P, INV>(x, pt, q);
}

// The same in little room: the butterflies take turns, six to eight twiddles read
// at a time (all of them together would spill in the strips' 64 registers, one
// butterfly at a time waits too often: batch of 24 scenes 33.8 us against 34.6).
template <int N, int P, bool INV>
__device__ __forceinline__ void tw_butterflies_in_turn(float2 (&x)[16], const float2* __restrict__ tw, int t)
{
    constexpr int R = LineGeom<N>::radix(P), TURN = R == 2 ? 8 : (R == 4 ? 2 : 1);
    PassTw<N, P> pt;
#pragma unroll
    for (int q = 0; q < 16 / R; q += TURN) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TURN; ++i) read_tw<N, P>(pt, tw, t, q + i);
#pragma unroll
        for (int i = 0; i < TURN; ++i) tw_butterfly<N, P, INV>(x, pt, q + i);
    }
}

// The twiddles of one thread inside the butterflies of one pass.  The thread's
// 16 / R butterflies of a radix-R pass (q = 0 .. 16/R - 1, j = t + q T) and their
// levels need w^e W16^(e r), e a power of two below R, r < 8 / e; with -j factored
// out (r >= 4 / e) eight values remain: w W16^r, w^2 W8^r, w^4, w^8, where w is
// the twiddle of butterfly q = 0 (in a trailing pass the span is N / R, so
// butterfly q's is w W16^q).
struct TwSet {
    float2 r[4];         // w, w W16, w W16^2, w W16^3
    float2 s[2];         // w^2, w^2 W8
    float2 w4, w8;
};

// Twiddle table reads of pass P of virtual thread t (one of N / 16); row i - 1
// of the pass's table holds w^i.
//   FMA: w, w^2, w^4, w^8;  ROT: w W16^q (q < 4), for radix 4 also w^2 W8^q
//   (q < 2), the others being -j times these;  PRE: see PassTw.
template <int N, int P, PassForm F = pass_form<N, P>()> struct TwReads {
    static constexpr int COUNT = F == PASS_FMA ? 4 : F == PASS_ROT ? (LineGeom<N>::radix(P) == 2 ? 4 : 6) : 0;
    float2 w[COUNT ? COUNT : 1];
};
template <int N, int P> struct TwReads<N, P, PASS_PRE> : PassTw<N, P> {};

template <int N, int P>
__device__ __forceinline__ void tw_issue(TwReads<N, P>& a, const float2* __restrict__ tw, int t)
{
    using G = LineGeom<N>;
    constexpr PassForm F = pass_form<N, P>();
    if constexpr (F == PASS_FMA) {
        constexpr int NS = G::span(P);
        const int jm = t & (NS - 1);
        a.w[0] = tw_ld<N, P>(tw, jm, 0);
        a.w[1] = tw_ld<N, P>(tw, jm, NS);
        a.w[2] = tw_ld<N, P>(tw, jm, 3 * NS);
        a.w[3] = tw_ld<N, P>(tw, jm, 7 * NS);
    } else if constexpr (F == PASS_ROT) {
        constexpr int NS = G::span(P);
        static_assert(G::radix(P) <= 4 && 4 * G::T <= NS, "w W16^q lie in the first row");
#pragma unroll
        for (int q = 0; q < 4; ++q) a.w[q] = tw_ld<N, P>(tw, t, q * G::T);
        if constexpr (G::radix(P) == 4) {
#pragma unroll
            for (int q = 0; q < 2; ++q) a.w[4 + q] = tw_ld<N, P>(tw, t, NS + q * G::T);
        }
    } else if constexpr (F == PASS_PRE) {
        read_tw<N, P>(a, tw, t);
    }
}

template <int N, int P>
__device__ __forceinline__ void tw_form(TwSet& p, const TwReads<N, P>& a)
{
    if constexpr (pass_form<N, P>() == PASS_FMA) {
        constexpr float c1 = 0.92387953251128675613f;
        constexpr float s1 = 0.38268343236508977173f;
        const float2 w = a.w[0];
        p.r[0] = w;
        p.r[1] = c_mul(w, make_float2(c1, -s1));
        p.r[2] = c_mul_w8<false>(w);
        p.r[3] = c_mul(w, make_float2(s1, -c1));
        p.s[0] = a.w[1];
        p.s[1] = c_mul_w8<false>(a.w[1]);
        p.w4 = a.w[2];
        p.w8 = a.w[3];
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) p.r[q] = a.w[q];
        if constexpr (LineGeom<N>::radix(P) == 4) {
            p.s[0] = a.w[4];
            p.s[1] = a.w[5];
        }
    }
}

// Level E (inputs E apart within a butterfly) of a thread's 16 / R butterflies
// of radix R: point i of butterfly q, partial output k, sits at
// q + (16 / R) (i + 2 E k) before and q + (16 / R) (i + E k) after.
template <int R, int E, bool INV>
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
            const float2 w = E == 8 ? p.w8 : E == 4 ? p.w4 : E == 2 ? p.s[r & 1] : p.r[r & 3];
#pragma unroll
            for (int i = 0; i < E; ++i) {
                float2 a = v[q + B * (i + 2 * E * k)], b = v[q + B * (i + E + 2 * E * k)];
                if (E < 8 && r >= J) bfly_mj<INV>(a, b, w);
                else bfly<INV>(a, b, w);
                o[q + B * (i + E * k)] = a;
                o[q + B * (i + E * (k + K))] = b;
            }
        }
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = o[i];
}

// All butterflies of pass P of one virtual thread, in registers.
template <int N, int P, bool INV>
__device__ __forceinline__ void pass_butterflies(float2 (&x)[16], const TwReads<N, P>& a)
{
    constexpr PassForm F = pass_form<N, P>();
    if constexpr (F == PASS_NONE) {
        Dft<16, INV>::run(x);
    } else if constexpr (F == PASS_PRE) {
        tw_butterflies<N, P, INV>(x, a);
    } else {
        constexpr int R = LineGeom<N>::radix(P);
        TwSet p;
        tw_form<N, P>(p, a);
        if constexpr (R >= 16) fft_level<R, 8, INV>(x, p);
        if constexpr (R >= 16) fft_level<R, 4, INV>(x, p);
        if constexpr (R >= 4) fft_level<R, 2, INV>(x, p);
        fft_level<R, 1, INV>(x, p);
    }
}

// The LDS exchange after radix-16 pass P: outputs of the butterflies to the
// strided layout.
// SPLIT: real and imaginary parts in two float arrays of the line's LDS
// (re[0, LDS), im[LDS, 2 LDS)), two 4-byte accesses per point instead of one
// 8-byte access, so that the two layouts can be compared.
template <int N, int P, bool SPLIT>
__device__ __forceinline__ void line_exchange(float2 (&x)[16], float2* __restrict__ lds, int t)
{
    using G = LineGeom<N>;
    static_assert(G::radix(P) == 16, "only the last pass is smaller than radix 16");
    constexpr int NS = G::span(P);
    const int base = (t / NS) * NS * 16 + (t & (NS - 1));
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

// One Stockham pass P of an N-point line (see the header comment), with its
// twiddles already read.
template <int N, int P, bool INV, bool SPLIT = false>
__device__ __forceinline__ void fft_pass(float2 (&x)[16], float2* __restrict__ lds,
                                         const TwReads<N, P>& a, int t)
{
    pass_butterflies<N, P, INV>(x, a);
    if constexpr (P < LineGeom<N>::NP - 1) line_exchange<N, P, SPLIT>(x, lds, t);
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
template <int N, bool INV, int P, bool SPLIT, bool AHEAD, int FRESH, class F>
__device__ __forceinline__ void fft_from(float2 (&x)[16], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last,
                                         const TwReads<N, P>& ahead)
{
    if constexpr (P < LineGeom<N>::NP) {
        TwReads<N, P + 1> next;
        int ti = t;
        constexpr int READ = AHEAD ? P + 1 : P;           // the pass whose reads are issued here
        if constexpr ((FRESH >> READ) & 1) asm volatile("" : "+v"(ti));
        if constexpr (AHEAD) {
            if constexpr (P == LineGeom<N>::NP - 1) before_last();
            tw_issue<N, P + 1>(next, tw, ti);
            fft_pass<N, P, INV, SPLIT>(x, lds, ahead, t);
        } else {
            TwReads<N, P> now;
            tw_issue<N, P>(now, tw, ti);
            // after the reads that the pass waits for, so that it need not wait for these
            if constexpr (P == LineGeom<N>::NP - 1) before_last();
            fft_pass<N, P, INV, SPLIT>(x, lds, now, t);
        }
        fft_from<N, INV, P + 1, SPLIT, AHEAD, FRESH>(x, lds, tw, t, before_last, next);
    }
}

// SPLIT: the split real/imaginary exchange layout (see line_exchange).
template <int N, bool INV, bool SPLIT = false, int FRESH = 0, class F = NoOp>
__device__ __forceinline__ void fft_line(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, int t, F&& before_last = F())
{
    TwReads<N, 0> first;
    fft_from<N, INV, 0, SPLIT, false, FRESH>(x, lds, tw, t, before_last, first);
}

// The same transform with every pass's table reads issued one pass ahead.
template <int N, bool INV, bool SPLIT = false, int FRESH = 0, class F = NoOp>
__device__ __forceinline__ void fft_line_ahead(float2 (&x)[line_e(N)], float2* __restrict__ lds,
                                               const float2* __restrict__ tw, int t,
                                               F&& before_last = F())
{
    TwReads<N, 0> first;
    fft_from<N, INV, 0, SPLIT, true, FRESH>(x, lds, tw, t, before_last, first);
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

// The twiddle reads of every pass (at most fourteen values), held in registers by
// a thread that transforms line after line: the transforms between then read
// nothing from memory, so no wait of theirs covers loads of the next line.
template <int N> struct TwAll {
    TwReads<N, 1> p1;
    TwReads<N, 2> p2;
    TwReads<N, 3> p3;
    __device__ __forceinline__ void read(const float2* __restrict__ tw, int t)
    {
        tw_issue<N, 1>(p1, tw, t);
        tw_issue<N, 2>(p2, tw, t);
        tw_issue<N, 3>(p3, tw, t);
    }
    template <int P> static __device__ __forceinline__ void pin_pass(TwReads<N, P>& r)
    {
#pragma unroll
        for (int i = 0; i < TwReads<N, P>::COUNT; ++i) pin(r.w[i]);
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
        if constexpr (P == 0) fft_pass<N, 0, INV>(x, lds, TwReads<N, 0>(), t);
        if constexpr (P == 1) fft_pass<N, 1, INV>(x, lds, tw.p1, t);
        if constexpr (P == 2) fft_pass<N, 2, INV>(x, lds, tw.p2, t);
        if constexpr (P == 3) fft_pass<N, 3, INV>(x, lds, tw.p3, t);
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
// Slot of point i after pass P: 4-byte accesses are served 32 lanes at a time (2
// cycles per wave and instruction), which must differ in the slot's low five bits.
// The reads take consecutive points, pass 1's writes runs of 16 points 256 apart (a
// pad of 4 every 64): free of conflicts.  Pass 0's writes are 16 points apart and with
// a pad every 64 have a two-way conflict (4 cycles); a pad every 32 avoids it, but
// with that and the strips' lines 32 / C apart the back-turned 1024 x 2048 scene took
// 28.1 us instead of 27.4 and no other scene less.
template <int P> __host__ __device__ constexpr int half_pads() { return P == 0 ? 1 : 4; }

template <int P>
__host__ __device__ constexpr int half_slot(int i)
{
    return i + half_pads<P>() * (i >> 6);
}
// half_slot(t + m * T), t < T, and half_slot(base + i * NS), as in lds_in / lds_out.
template <int T, int P>
__host__ __device__ constexpr int half_in(int t, int m)
{
    if constexpr (T >= 64) return half_slot<P>(t) + m * (T + half_pads<P>() * (T / 64));
    else return t + (m * T + half_pads<P>() * (m * T / 64));
}
template <int NS, int P>
__host__ __device__ constexpr int half_out(int base, int i)
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
        if constexpr (pass_form<N, P>() == PASS_PRE) {
            tw_butterflies_in_turn<N, P, INV>(x, tw, fresh(t));
        } else {
            TwReads<N, P> now;
            tw_issue<N, P>(now, tw, fresh(t));
            pass_butterflies<N, P, INV>(x, now);
        }
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
